"""The launch shapes of the top-k and of the sort behind it, over all sizes a call may have: host rules of the library,
asked for by their C++ names."""
import ctypes

import pytest

from paper_2502_16927_amd import binding as B


class Chunks(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("threads", "tokens", "parts", "count")]


class Grid(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("workgroups", "threads", "tokens")]


def rule(symbol, result, args):
    f = getattr(B.lib(), symbol)
    f.restype, f.argtypes = result, args
    return f


ci = ctypes.c_int
topk_counts = rule("_ZN6bigmac11topk_countsEiii", ctypes.c_bool, [ci] * 3)
topk_grid = rule("_ZN6bigmac9topk_gridEiiib", Grid, [ci] * 3 + [ctypes.c_bool])
permutation_ws_bytes = rule("_ZN6bigmac20permutation_ws_bytesEiiib", ctypes.c_size_t, [ci] * 3 + [ctypes.c_bool])
sort_chunks = rule("_ZN6bigmac11sort_chunksEiiib", Chunks, [ci] * 3 + [ctypes.c_bool])

SIZES = [(T, k, N) for T in (1, 2, 31, 32, 64, 65, 500, 512, 1024, 1025, 3001, 4096, 4097, 8192, 16384, 32768, 65536, 131072, 1 << 20)
         for N in (1, 8, 40, 64, 65, 96, 128, 129, 256, 512, 513, 1024) for k in (1, 2, 3, 6, 8, 17, 64) if k <= N]


def test_topk_spreads_over_the_chip():
    """Whoever counts the pairs: half of the 256 CUs have a workgroup, or no wavefront has a second round of two tokens."""
    for T, k, N in SIZES:
        g = topk_grid(T, k, N, topk_counts(T, k, N))
        assert g.workgroups * g.tokens >= T and 64 <= g.threads <= (1024 if N <= 128 else 256), (T, k, N)
        assert g.workgroups >= 128 or g.tokens <= 2 * (g.threads // 64), (T, k, N, g.workgroups)
        assert not topk_counts(T, k, N) or (N <= 128 and T * k > 4096)


@pytest.mark.parametrize("counting", [False, True])
def test_no_wavefront_of_the_topk_sorts_for_nothing(counting):
    """A wavefront takes two tokens at a time where it counts and one elsewhere: as many wavefronts as have tokens to take."""
    for T, k, N in SIZES:
        if not counting or topk_counts(T, k, N):
            g = topk_grid(T, k, N, counting)
            assert g.threads // 64 == (min(16, -(-g.tokens // 2)) if counting else g.tokens), (T, k, N)


@pytest.mark.parametrize("counted", [False, True])
def test_sort_chunks_hold_whole_tokens_and_every_token(counted):
    for T, k, N in SIZES:
        if counted and not topk_counts(T, k, N):
            continue
        c = sort_chunks(T, k, N, counted)
        if not c.threads:
            continue
        pairs = c.tokens * c.parts * k
        assert 0 < pairs <= c.threads and c.count * pairs >= T * k > (c.count - 1) * pairs, (T, k, N)
        assert c.threads == 1024 or N <= 64                      # the tile maps of more experts take 1024 threads
        rows = c.count * c.parts
        need = -(-rows * N * 4 // 256) * 256
        assert permutation_ws_bytes(T, k, N, counted) == need and rows <= 512, (T, k, N)
        if not counted:      # bigmac_dispatch, whose counts are its own, does not ask for the rows that a layer call's top-k counts
            assert B.workspace_bytes(B.make_dims(T, 64, 64, N, k, 64), B.WS_DISPATCH) == need, (T, k, N)
        if counted:
            g = topk_grid(T, k, N, True)
            assert (g.workgroups, g.tokens) == (rows, c.tokens)
