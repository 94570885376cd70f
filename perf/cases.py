"""The work that users of this library have it do, as measurable cases.

A case is one call pattern through the public entry points on one seeded synthetic game.  The
listed cases are the shapes of this repository's own configurations, benchmark legs and tests, from
a 5151-point lattice (launch latency) to a streamed sweep of millions of candidates, in fp32 and
bf16 storage, on shapes that fill the matrix-core tiles and on shapes that do not.  `draw` gives
more of the same: every call pattern over its range of sizes.

Call patterns (`"call"`):
  lattice    bsse_lattice, bsse_sweep of that set, bsse_sweep_best_row (the commitment itself)
  sweep      bsse_sweep of a device buffer of candidate rows
  generated  bsse_sweep_dirichlet: seeded rows swept without the caller ever holding them;
             bsse_sweep_best_row
  streamed   reset; per chunk bsse_dirichlet into one buffer and bsse_sweep_chunk; bsse_sweep_result;
             bsse_sweep_best_row
  topk       bsse_sweep_topk of a buffer
  priors     bsse_sweep_priors of a buffer
  solve      one game from scratch: bsse_dirichlet, bsse_sweep, bsse_polish, bsse_refine,
             bsse_solve_realised
"""
import math

import numpy as np
import torch

from paper_2605_18856_amd import bsse, workloads


def listed():
    return [
        # the tiny game: every point of a simplex lattice; nothing but launches and waits
        {"name": "lattice_tiny", "call": "lattice", "m": 3, "n": 3, "K": 2, "storage": "f32",
         "payoffs": "uniform", "N": 100},
        # a handful of rows against an ordinary game: an interactive query, latency again
        {"name": "sweep_small_batch", "call": "sweep", "m": 32, "n": 32, "K": 16, "storage": "f32",
         "payoffs": "structured", "count": 1000},
        # the 8x8 game over seeded rows, the second configuration
        {"name": "generated_m8n8K4", "call": "generated", "m": 8, "n": 8, "K": 4, "storage": "f32",
         "payoffs": "normal", "count": 1 << 20},
        # the same game over rows that sit in memory: bound by reading them
        {"name": "sweep_stream_m8n8K4", "call": "sweep", "m": 8, "n": 8, "K": 4, "storage": "f32",
         "payoffs": "normal", "count": 1 << 24},
        # the misalignment-structured game, the third configuration, a quarter of its rows
        {"name": "generated_m32n32K16", "call": "generated", "m": 32, "n": 32, "K": 16, "storage": "f32",
         "payoffs": "structured", "count": 1 << 22},
        # the large dense game in bf16, the fourth configuration, streamed chunk by chunk
        {"name": "streamed_m64n128K64_bf16", "call": "streamed", "m": 64, "n": 128, "K": 64,
         "storage": "bf16", "payoffs": "uniform", "count": 1 << 21, "chunks": 2},
        # the widest game, small integer payoffs, the fifth configuration, a part of its rows
        {"name": "sweep_m128n256K256_int", "call": "sweep", "m": 128, "n": 256, "K": 256, "storage": "f32",
         "payoffs": "int", "count": 1 << 17},
        # games as they come, with no dimension a multiple of anything: fp32 and bf16 storage
        {"name": "sweep_ragged_f32", "call": "sweep", "m": 30, "n": 50, "K": 20, "storage": "f32",
         "payoffs": "normal", "count": 100003},
        {"name": "sweep_ragged_bf16", "call": "sweep", "m": 50, "n": 100, "K": 24, "storage": "bf16",
         "payoffs": "uniform", "count": 70001},
        # the best 64 of a million candidates (starting points of a local search)
        {"name": "topk_m8n8K4", "call": "topk", "m": 8, "n": 8, "K": 4, "storage": "f32",
         "payoffs": "normal", "count": 1 << 20, "k": 64},
        # how the best commitment moves over a hundred priors
        {"name": "priors_m8n8K4", "call": "priors", "m": 8, "n": 8, "K": 4, "storage": "f32",
         "payoffs": "normal", "count": 1 << 20, "P": 101},
        # one game solved end to end: sweep, polish, local refinement, programs of realised profiles
        {"name": "solve_m16n16K4", "call": "solve", "m": 16, "n": 16, "K": 4, "storage": "f32",
         "payoffs": "normal", "count": 1 << 16, "k": 8, "rounds": 2, "cloud": 4096, "programs": 200},
    ]


def _log_int(rng, lo, hi):
    """An integer in lo..hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _capped_count(rng, lo, hi, per_row, cap):
    """A row count in lo..hi (over its logarithm) whose work stays below `cap` operations."""
    return _log_int(rng, lo, max(lo, min(hi, int(cap / per_row))))


#: Operations of a drawn sweep of any shape, and of one whose shape fills the matrix-core tiles.
ANY_SHAPE_FLOPS, TILED_FLOPS = 6.0e9, 2.0e12


def draw(rng):
    call = rng.choice(["lattice", "any", "any", "any", "small", "generated", "tiled", "topk", "priors", "solve"])
    if call == "lattice":
        m = rng.randint(2, 6)
        payoffs = rng.choice(["uniform", "normal", "dup"])
        sizes = [N for N in range(4, 1200) if 500 <= bsse.bsse_lattice_count(m, N) <= 1 << 18]
        if payoffs == "dup":              # integer payoffs, dyadic points: every sum and every tie is exact
            sizes = [N for N in sizes if N & (N - 1) == 0] or [8]
        return {"call": "lattice", "m": m, "n": rng.randint(2, 12), "K": rng.randint(1, 6), "storage": "f32",
                "payoffs": payoffs, "N": rng.choice(sizes)}
    if call == "any":                     # any shape, either storage type
        m, n, K = _log_int(rng, 3, 128), _log_int(rng, 3, 256), _log_int(rng, 1, 128)
        storage = rng.choice(["f32", "bf16"])
        return {"call": rng.choice(["sweep", "sweep", "generated"]), "m": m, "n": n, "K": K, "storage": storage,
                "payoffs": rng.choice(["normal", "uniform"]),
                "count": _capped_count(rng, 200, 1 << 20, K * 2.0 * m * (n + 1), ANY_SHAPE_FLOPS)}
    if call == "small":                   # the 8x8 games over rows in memory
        return {"call": "sweep", "m": 8, "n": 8, "K": rng.choice([4, 8, 12, 16]), "storage": "f32",
                "payoffs": rng.choice(["normal", "uniform"]), "count": _log_int(rng, 1000, 1 << 24)}
    if call == "generated":
        if rng.random() < 0.5:
            m, n, K = 8, 8, rng.choice([4, 8, 12, 16])
            return {"call": "generated", "m": m, "n": n, "K": K, "storage": "f32", "payoffs": "normal",
                    "count": _log_int(rng, 1 << 14, 1 << 22)}
        m, n, K = rng.randint(17, 32), rng.choice([32, 64]), rng.randint(2, 16)
        return {"call": "generated", "m": m, "n": n, "K": K, "storage": "f32", "payoffs": "structured",
                "count": _log_int(rng, 1 << 14, 1 << 21)}
    if call == "tiled":
        if rng.random() < 0.5:
            m, K = rng.randint(33, 64), rng.randint(8, 64)
            return {"call": "streamed", "m": m, "n": 128, "K": K, "storage": "bf16", "payoffs": "uniform",
                    "count": _capped_count(rng, 1 << 12, 1 << 20, K * 2.0 * m * 129, TILED_FLOPS), "chunks": rng.randint(1, 3)}
        m, K = rng.randint(65, 128), rng.randint(16, 256)
        return {"call": "sweep", "m": m, "n": 256, "K": K, "storage": "f32", "payoffs": "int",
                "count": _capped_count(rng, 1 << 10, 1 << 17, K * 2.0 * m * 257, TILED_FLOPS)}
    if call in ("topk", "priors"):
        m, n, K = (8, 8, rng.choice([4, 8, 16])) if rng.random() < 0.5 else (
            rng.randint(4, 32), rng.choice([7, 12, 16, 24, 32]), rng.randint(2, 16))
        c = {"call": call, "m": m, "n": n, "K": K, "storage": "f32", "payoffs": "normal",
             "count": _capped_count(rng, 3000, 1 << 20, K * 2.0 * m * (n + 1), ANY_SHAPE_FLOPS)}
        c["k" if call == "topk" else "P"] = _log_int(rng, 1, 256) if call == "topk" else _log_int(rng, 2, 256)
        return c
    m, n, K = rng.randint(4, 16), rng.randint(4, 16), rng.randint(2, 4)
    return {"call": "solve", "m": m, "n": n, "K": K, "storage": "f32", "payoffs": "normal",
            "count": _log_int(rng, 1 << 12, 1 << 16), "k": rng.randint(2, 8), "rounds": rng.randint(1, 2),
            "cloud": _log_int(rng, 512, 4096), "programs": _log_int(rng, 10, 200)}


def _game(case, seed):
    m, n, K = case["m"], case["n"], case["K"]
    if case["payoffs"] != "structured":
        return workloads.small_game(m, n, K, seed, case["payoffs"], case["storage"])
    # follower payoffs correlated with the leader's, one correlation per type
    g = workloads.small_game(m, n, K, seed, "normal", case["storage"])
    rho = np.random.Generator(np.random.PCG64(seed + 1)).uniform(-1.0, 1.0, size=(K, 1, 1))
    g.B = (rho * g.A + np.sqrt(1.0 - rho ** 2) * g.B).astype(np.float32)
    return g


def prepare(case, seed):
    """The game's handle (payoffs packed on the device, as a program that uses the game keeps it),
    the candidate rows where the caller owns them, and the seed of generated rows."""
    game = _game(case, seed)
    storage = bsse.BSSE_STORAGE_BF16 if case["storage"] == "bf16" else bsse.BSSE_STORAGE_F32
    g = bsse.bsse_create(game.m, game.n, game.K, game.A, game.B, game.prior, storage=storage)
    state = {"case": case, "g": g, "seed": 7919 * seed + 1}
    if case["call"] in ("sweep", "topk", "priors", "streamed"):
        state["X"] = torch.empty((case["count"], game.m), dtype=torch.float32, device="cuda")
        if case["call"] != "streamed":
            bsse.bsse_dirichlet(g, state["seed"], 0, case["count"], state["X"])
    if case["call"] == "priors":
        rng = np.random.Generator(np.random.PCG64(seed + 2))
        p = rng.dirichlet(np.ones(game.K), size=case["P"])
        p = p.astype(np.float32).astype(np.float64)
        state["priors"] = (p / p.sum(axis=1, keepdims=True)).astype(np.float32)
    return state


def _sweep_outputs(out):
    # (the count of exact fp32 ties is left out here: with real-valued payoffs it depends on the order in
    # which a dot product is summed)
    return {"value": out.best_value, "index": out.best_index, "response": out.best_response, "evals": out.n_evals}


def run(state):
    case, g = state["case"], state["g"]
    call, count = case["call"], case.get("count", 0)
    if call == "lattice":
        bsse.bsse_lattice(g, case["N"])
        out = bsse.bsse_sweep(g)
        outputs = dict(_sweep_outputs(out), x=bsse.bsse_sweep_best_row(g))
        if case["payoffs"] == "dup":
            outputs["ties"] = out.n_tie_evals
        return outputs
    if call == "sweep":
        return _sweep_outputs(bsse.bsse_sweep(g, state["X"], count))
    if call == "generated":
        out = bsse.bsse_sweep_dirichlet(g, state["seed"], 0, count)
        return dict(_sweep_outputs(out), x=bsse.bsse_sweep_best_row(g))
    if call == "streamed":
        bsse.bsse_sweep_reset(g)
        for c in range(case["chunks"]):
            bsse.bsse_dirichlet(g, state["seed"], c * count, count, state["X"])
            bsse.bsse_sweep_chunk(g, state["X"], count, c * count)
        return dict(_sweep_outputs(bsse.bsse_sweep_result(g)), x=bsse.bsse_sweep_best_row(g))
    if call == "topk":
        values, indices, responses = bsse.bsse_sweep_topk(g, case["k"], state["X"], count)
        return {"values": values, "indices": indices, "responses": responses}
    if call == "priors":
        outs = bsse.bsse_sweep_priors(g, state["priors"], state["X"], count)
        return {"values": np.array([o.best_value for o in outs]), "indices": np.array([o.best_index for o in outs]),
                "responses": np.stack([o.best_response for o in outs])}
    bsse.bsse_dirichlet(g, state["seed"], 0, count)
    swept = bsse.bsse_sweep(g)
    polished = bsse.bsse_polish(g)
    value, x, profile, _, _ = bsse.bsse_solve_realised(g, max_profiles=case["programs"])
    xr, vr, br, _ = bsse.bsse_refine(g, case["k"], case["rounds"], cloud_count=case["cloud"], seed=state["seed"])
    return {"swept": _sweep_outputs(swept), "polished": polished.value, "polished_x": polished.x,
            "program_value": polished.lp_value, "realised": value, "realised_x": x, "realised_profile": profile,
            "refined": vr, "refined_x": xr, "refined_response": br}


def work(case):
    m, n, K = case["m"], case["n"], case["K"]
    rows = case.get("count", 0) * case.get("chunks", 1)
    if case["call"] == "lattice":
        rows = bsse.bsse_lattice_count(m, case["N"])
    if case["call"] == "solve":            # the sweep, the realised profiles' evaluation, the rounds' clouds
        rows = 3 * rows + case["k"] * case["rounds"] * case["cloud"]
    evals = float(rows) * K
    flops = evals * (2.0 * m * n + 2.0 * m)
    payoffs = 2.0 * K * m * n * (2 if case["storage"] == "bf16" else 4)
    # rows that the caller owns are read once; generated rows need never exist; a lattice or a
    # handle-owned set is written by its call, for the caller to have, and read by the next
    bytes_ = payoffs
    if case["call"] in ("sweep", "topk", "priors"):
        bytes_ += 4.0 * m * rows
    if case["call"] in ("lattice", "streamed"):
        bytes_ += 8.0 * m * rows
    if case["call"] == "solve":
        bytes_ += 8.0 * m * case["count"]
    if case["call"] == "priors":
        flops += 2.0 * evals * case["P"]
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # fp32 sums of at most 128 + 256 terms in some order (bf16 storage too: its products are exact in
    # fp32, and what is rounded to bf16 is rounded before any sum).  Two candidates of a sorted list
    # of survivors whose values differ by less than that may change places.
    t = {"rel": 1e-5}
    if case["call"] in ("topk", "priors"):
        t["differ"] = 0.01
    if case["call"] == "solve":
        # a vertex is reached through fp64 pivots, then a point of a segment is chosen by fp32 values
        t["rel"] = 1e-4
    return t
