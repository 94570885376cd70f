"""How one matrix instruction adds its terms, which the margins of the filters rest on: terms set so that they lose all
that they can beside a greater one, with the sum and against it, and sums that cancel.

In half precision and bf16 (two passes of eight products): a term loses up to 2^-24 of the greatest product of its pass
or 2^-26 of the sum it is added to, and each pass rounds once.  In units of 2^-24 that is at most eight times the sum of
the absolute products and six times the greater of both sums.  The scaled instruction on e2m3 numbers loses up to 5.1
units of the greatest of terms and sums on these; the six-bit kernel counts with 65/4 + 1."""
import ctypes

import numpy as np
import pytest

from paper_2605_18856_amd import bsse

pytestmark = pytest.mark.gpu
COUNT = 16
UNIT = 2.0 ** -24
ROWS = np.array([[(r & 3) + 8 * (r >> 2) + 4 * h for r in range(16)] for h in range(2)])       # of a lane's accumulator


def _run(kind, a, b, scales, C):
    """One instruction per problem: words of the operands [count][64][8], C and the result [count][row][column]."""
    import torch
    f = bsse.lib()._ZN4bsse11matrix_unitEiiPKjS1_PKiPKfPfP12ihipStream_t
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 6
    lanes = np.concatenate([C[:, ROWS[h], :].transpose(0, 2, 1) for h in range(2)], axis=1)
    dev = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (a.view(np.int32), b.view(np.int32), scales.astype(np.int32), lanes)]
    out = torch.empty((len(a), 64, 16), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    assert f(kind, len(a), *[t.data_ptr() for t in dev], out.data_ptr(), None) == 0
    torch.cuda.synchronize()
    d, D = out.cpu().numpy(), np.empty_like(C)
    for h in range(2):
        D[:, ROWS[h], :] = d[:, 32 * h:32 * h + 32].transpose(0, 2, 1)
    return D


def _words(v16):
    """16-bit operands [count][row][k] as a lane's words: lane 32 h + row holds k from 8 h on."""
    out = np.zeros((len(v16), 64, 16), np.uint16)
    for h in range(2):
        out[:, 32 * h:32 * h + 32, :8] = v16[:, :, 8 * h:8 * h + 8]
    return out.view(np.uint32)


def _sixteen_bit(kind, A, B):
    if kind == 0:                                        # (rounded towards zero: any bf16 numbers will do)
        A, B = [(v.astype(np.float32).view(np.uint32) & 0xFFFF0000).view(np.float32) for v in (A, B)]
        return A, B, *[_words((v.view(np.uint32) >> 16).astype(np.uint16)) for v in (A, B)]
    A, B = A.astype(np.float16), B.astype(np.float16)
    return A, B, _words(A.view(np.uint16)), _words(B.view(np.uint16))


@pytest.mark.parametrize("kind", [0, 1], ids=["bf16", "half"])
@pytest.mark.parametrize("terms", ["great_0", "great_9", "great_sum", "spread", "subnormal"])
@pytest.mark.parametrize("sign", [1.0, -1.0, 0.0], ids=["same", "against", "mixed"])
def test_terms_of_sixteen(kind, terms, sign):
    rng = np.random.default_rng(600 + kind)
    shape, bits = (COUNT, 32, 16), 10 if kind else 7
    worst = 0.0
    for size in range(18, 30):
        A = (2.0 - (1 + rng.integers(0, 3, shape)) * 2.0 ** -bits) * 2.0 ** -(size // 2)
        B = (2.0 - (1 + rng.integers(0, 3, shape)) * 2.0 ** -bits) * 2.0 ** -(size - size // 2)
        B *= sign if sign else rng.choice([-1.0, 1.0], shape)
        C = np.zeros((COUNT, 32, 32), np.float32)
        if terms.startswith("great_") and terms != "great_sum":
            A[:, :, int(terms[6:])] = B[:, :, int(terms[6:])] = 1.0
        elif terms == "great_sum":
            C[:] = 1.0
        elif terms == "subnormal":
            if kind == 0:
                continue
            A, B = np.ldexp(rng.integers(-1023, 1024, shape), -24), B * 2.0 ** (size - size // 2)
        else:
            A *= 2.0 ** rng.integers(0, size // 2 + 1, shape)
            B *= 2.0 ** rng.integers(0, size // 2 + 1, shape)
            C = (rng.uniform(1.0, 2.0, C.shape) * 2.0 ** rng.integers(-25, 3, C.shape)).astype(np.float32)
        A, B, a, b = _sixteen_bit(kind, A, B)
        D = _run(kind, a, b, np.zeros((COUNT, 64)), C).astype(np.float64)
        T = A.astype(np.float64)[:, :, None, :] * B.astype(np.float64)[:, None, :, :]
        S = T.sum(axis=-1) + C
        bound = 8 * np.abs(T).sum(axis=-1) + 6 * np.maximum(np.abs(C), np.abs(S))
        worst = max(worst, (np.abs(D - S) / (UNIT * np.where(bound > 0, bound, 1))).max())
    assert worst <= 1.0, worst


def _e2m3(q):
    e, f = (q >> 3) & 3, q & 7
    return np.where(q & 32, -1.0, 1.0) * np.where(e == 0, f / 8.0, (1 + f / 8.0) * 2.0 ** (e - 1.0))


def _codes(q):
    """Codes [count][row][64] as a lane's words: lane 32 h + row holds k from 32 h on, six bits each."""
    out = np.zeros((len(q), 64, 8), np.uint32)
    bits = ((q[..., None] >> np.arange(6)) & 1).astype(np.uint8)
    for h in range(2):
        packed = np.packbits(bits[:, :, 32 * h:32 * h + 32].reshape(len(q), 32, 192), axis=-1, bitorder="little")
        out[:, 32 * h:32 * h + 32, :6] = np.ascontiguousarray(packed).view(np.uint32)
    return out


@pytest.mark.parametrize("terms", ["great_term", "great_sum", "spread"])
@pytest.mark.parametrize("sign", [0, 32, 63], ids=["same", "against", "mixed"])
def test_terms_of_the_scaled_instruction(terms, sign):
    rng = np.random.default_rng(610)
    shape = (COUNT, 32, 64)
    worst = 0.0
    for size in range(8, 36):
        low = 24 if terms == "great_term" else 1
        a, b = rng.integers(low, 32, shape), rng.integers(low, 32, shape)
        b |= sign & 32 if sign != 63 else 32 * rng.integers(0, 2, shape)
        e = np.zeros((COUNT, 64), int)
        C = np.zeros((COUNT, 32, 32), np.float32)
        if terms == "great_term":                        # one product of 1 in the first half, the other half smaller
            a[:, :, :32] = b[:, :, :32] = 0
            a[:, :, 3] = b[:, :, 3] = 8
            e[:, 32:] = -size
        elif terms == "great_sum":
            C[:] = 2.0 ** size
            e[:, 32:] = -rng.integers(0, 12, (COUNT, 32))
        else:
            e = rng.integers(-size // 2, size // 2 + 1, e.shape)
            C = (rng.uniform(1.0, 2.0, C.shape) * 2.0 ** rng.integers(-20, 20, C.shape)).astype(np.float32)
        D = _run(2, _codes(a), _codes(b), 127 + e, C).astype(np.float64)
        scale = np.repeat(np.ldexp(1.0, e).reshape(COUNT, 2, 32).transpose(0, 2, 1), 32, axis=2)       # [count][column][k]
        T = _e2m3(a)[:, :, None, :] * (_e2m3(b) * scale)[:, None, :, :]
        S = T.sum(axis=-1) + C
        great = np.maximum(np.maximum(np.abs(T).max(axis=-1), np.abs(C)), np.abs(S))
        worst = max(worst, (np.abs(D - S) / (UNIT * great)).max())
    assert worst <= 65 / 4 + 1, worst
