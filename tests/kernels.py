"""Which kernel the library picks for a game where the path name does not say: the rules that bsse_create asks, which run
on the host (internal functions of the library, called by their mangled names; no GPU needed)."""
import ctypes

import numpy as np

from paper_2605_18856_amd import bsse


def _rule(symbol, game, *payoffs):
    f = getattr(bsse.lib(), symbol)
    f.restype = ctypes.c_bool
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p] * len(payoffs)
    arrays = [np.ascontiguousarray(p, np.float32) for p in payoffs]
    return f(game.m, game.n, game.K, *[a.ctypes.data for a in arrays])


def six_bit(game):
    """bsse::six_bit_suits: bf16 payoffs, n = 256 on the six-bit matrix instruction."""
    return _rule("_ZN4bsse13six_bit_suitsEiiiPKfS1_", game, game.A, game.B)


def half_parts(game):
    """bsse::any_half_suits: fp32 payoffs that are no bf16 numbers in half-precision parts."""
    return _rule("_ZN4bsse14any_half_suitsEiiiPKf", game, game.B)
