"""The plans behind the calls, on the host: which kernels and layouts the sizes choose, that the
GPU tests' cases reach all of them, and that a plan's workspace holds what it writes."""
import ctypes
import math
import random

import pytest

import test_gpu_attention_tiles
import test_gpu_lmhead_instances


@pytest.fixture(scope="module")
def lib():
    from paper_2606_08411_amd import _lib
    return _lib.library()


def attn_plan(lib, L, B, P, Hq, Hkv, D, n_ref):
    """[lane pass, refresh pass], each (wavefront split, key splits, query tiles, fp32 partials, lane
    blocks dealt to the splits)."""
    out = (ctypes.c_int32 * 10)()
    assert lib.al_internal_attn_plan(L, B, P, Hq, Hkv, D, n_ref, out) == 0
    return tuple(out[:5]), tuple(out[5:])


def _attn_sizes(n, seed):
    r = random.Random(seed)
    for _ in range(n):
        Hkv, g = r.choice([1, 2, 4, 8, 16, 32]), r.choice([1, 1, 2, 4, 7])
        P, D = r.choice([0, 1, 65, 130, 200, 449, 700, 1300, 3000]), r.choice([64, 128])
        L = r.choice([0, 1, 2, 3, 5, 8, 9, 16, 17, 20, 33, 40, 64])
        n_ref = r.randint(0 if L else 1, P) if P else 0
        if L or n_ref:
            yield L, r.choice([16, 32, 48, 80]), P, Hkv * g, Hkv, D, n_ref


def test_attention_cases_reach_every_plan(lib):
    """(pass, key splits, query tiles, fp32 partials, dealt) of the 8-tile kernel."""
    def kinds(case):
        lane, ref = attn_plan(lib, *case)
        if case[0] and not lane[0]:
            yield ("lane",) + lane[1:]
        if case[6] and not ref[0]:
            yield ("refresh",) + ref[1:]
    met = {k for c in _attn_sizes(40000, 1) for k in kinds(c)}
    tested = {k for c in test_gpu_attention_tiles.CASES for k in kinds(c)}
    # refreshed rows split otherwise than below take thousands of keys times heads: they run the
    # instances that the lanes' cases run, the workgroup does not know which pass it is in
    met = {k for k in met if k[0] == "lane" or ("lane",) + k[1:] not in tested}
    assert met <= tested, sorted(met - tested)


def test_attention_workspace_holds_the_partials(lib):
    """Splits write [n_split][rows][Hq] x (D bf16 or fp32 + 2 fp32); fp32 only with fewer splits than
    the workspace is sized for."""
    n = 0
    for c in _attn_sizes(40000, 2):
        L, B, P, Hq, Hkv, D, n_ref = c
        ws = lib.lane_attn_workspace_size(*c)
        for (wsplit, ns, tpw, f32, deal), rows in zip(attn_plan(lib, *c), (L * B, n_ref)):
            if rows and ns > 1:
                assert not wsplit
                assert ns * rows * Hq * ((4 if f32 else 2) * D + 8) <= ws, c
                n += f32
            else:
                assert not f32
    assert n > 100


def lmhead_plan(lib, N, d, V, packed):
    """(RA, CBT, vocabulary tiles, column tiles, ragged, non-temporal, two barriers per stage, fits)."""
    out = (ctypes.c_int32 * 8)()
    assert lib.al_internal_lmhead_plan(N, d, V, int(packed), out) == 0
    return tuple(out)


def _lmhead_kind(plan):
    """The kernel that runs: (RA, CBT, two barriers, ragged, non-temporal)."""
    return plan[0], plan[1], plan[6], plan[4], plan[5]


def _log_int(r, lo, hi):
    return int(round(math.exp(r.uniform(math.log(lo), math.log(hi)))))


def test_lmhead_every_size_has_a_layout(lib):
    """Some instance's partials always fit the workspace that the size query names, also where the
    no-alloc twin's fixed array is the workspace."""
    r = random.Random(4)
    for _ in range(30000):
        N, V = _log_int(r, 1, 100000), _log_int(r, 1, 1 << 30)
        assert lmhead_plan(lib, N, 4096, V, r.random() < 0.5)[7], (N, V)
    for V in (1, 31, 32, 33, 511, 513, 126464, 152064):
        for N in range(1, 1300):
            assert lmhead_plan(lib, N, 64, V, N & 1)[7], (N, V)


def test_lmhead_ragged_k_loads_w_like_full_k(lib):
    """A packed weight past the memory-side cache that is read once is loaded non-temporally whatever
    d % 64 is (only the hidden rows' loads differ): V = 126464, N = 96 took 191 us cached."""
    for N in (1, 64, 96, 128, 205):
        for d in (4096, 4072, 4104, 3000):
            for V in (64000, 126464, 152064):
                p = lmhead_plan(lib, N, d, V, True)
                assert p[4] == (d % 64 != 0) and p[5] == (p[3] == 1 and 2 * V * d > 384000000)
                assert not lmhead_plan(lib, N, d, V, False)[5]


def test_lmhead_few_rows_keep_loads_in_flight(lib):
    """Tiles of 512 rows have two K stages in LDS.  Where they leave compute units idle (85000 rows of V:
    167 tiles) one barrier a stage let the W stream drain: 85000 x 4096 packed, 1 row 103 -> 127 us."""
    for V, N, packed, two in ((85000, 1, True, 1), (85000, 40, True, 1), (85000, 1, False, 1),
                              (118000, 64, True, 1), (126464, 1, True, 0), (126464, 64, True, 0),
                              (126464, 77, True, 1), (126464, 77, False, 1), (126464, 1, False, 0),
                              (126464, 32, False, 1), (200000, 1, True, 1)):
        p = lmhead_plan(lib, N, 4096, V, packed)
        assert p[0] >= 6 and p[6] == two, (V, N, packed, p)
    for N in (77, 96):
        assert lmhead_plan(lib, N, 4096, 85000, True)[:2] == (6, 6)


def test_lmhead_narrow_tiles_for_few_rows(lib):
    """32 rows or fewer do not compute 64 columns where 320-row tiles fill one or two rounds
    (V = 134000 as given, 1 row: 209 us before the tile kernel, 219 with 64 columns, 189 with 32)."""
    for N in (1, 32):
        for V in (66000, 81900, 134000, 140000, 152064, 163000):
            for packed in (False, True):
                assert lmhead_plan(lib, N, 4096, V, packed)[:2] == (5, 2), (N, V)
        for V in (200000, 256000, 330000):
            assert lmhead_plan(lib, N, 4096, V, True)[:2] == (8, 2), (N, V)


def test_lmhead_cases_reach_every_instance(lib):
    """Every built (RA, CBT) in each of its stage forms, ragged and not, packed and as given, with one
    tile a workgroup and (from 256 rows of V a tile on) several; every non-temporal kernel."""
    T = test_gpu_lmhead_instances
    pairs = (ctypes.c_int32 * 400)()
    built = {(pairs[2 * i], pairs[2 * i + 1])
             for i in range(lib.al_internal_lmhead_instances(pairs, 200))}
    tested, several, nt = set(), set(), set()
    for N, d, V in T.SIZES:
        for packed in (False, True):
            p = lmhead_plan(lib, N, d, V, packed)
            (several if p[2] * p[3] > 256 else tested).add((packed,) + _lmhead_kind(p))
    for N, d, V in T.NT_SIZES:
        p = lmhead_plan(lib, N, d, V, True)
        assert p[5]
        nt.add(_lmhead_kind(p))
    assert {k[1:3] for k in tested} == built
    r = random.Random(6)
    for _ in range(60000):   # what the sizes in use reach
        d = 8 * _log_int(r, 1, 2048)
        N, V, packed = _log_int(r, 1, 1200), _log_int(r, 64, 260000), r.random() < 0.6
        p = lmhead_plan(lib, N, d, V, packed)
        k = (packed,) + _lmhead_kind(p)
        if p[5]:
            assert k[1:] in nt, (N, d, V, k)
        else:
            k = k[:5] + (0,)
            assert k in tested, (N, d, V, k)
            if p[2] * p[3] > 256 and p[0] >= 4:
                assert k in several, (N, d, V, k)
