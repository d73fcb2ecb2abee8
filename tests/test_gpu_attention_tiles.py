"""The 8-tile attention kernel at the edges of its key-tile ring: 0 to 9 prefix
tiles of 64 keys (odd and even, full and ragged), lane blocks of 1 and 2 tiles,
workgroups of 8 and of 4 query tiles, with and without key splits.

Against the fp64 oracle; outputs are bf16 (half a step of the largest values
met, below 4, is 2^-8) and P is rounded to bf16 (relative 2^-9 of a convex
combination of values below 5): within 2e-2.  LSE within 2e-3.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import f32
from test_gpu_attention import TOL_LSE, TOL_O, _run

pytestmark = pytest.mark.gpu

CASES = [  # L, B, P, Hq, Hkv, D, refreshed rows
    (0, 16, 40, 130, 130, 64, 40), (0, 16, 64, 130, 130, 128, 64), (0, 16, 65, 100, 100, 128, 65),
    (0, 16, 128, 65, 65, 64, 128), (0, 16, 129, 64, 64, 128, 129), (0, 16, 193, 56, 56, 128, 193),
    (0, 16, 257, 40, 40, 64, 257), (0, 16, 320, 32, 32, 128, 320), (0, 16, 385, 28, 4, 128, 385),
    (0, 16, 577, 16, 16, 128, 577), (0, 16, 300, 64, 4, 128, 300), (0, 16, 600, 8, 8, 64, 600),
    (6, 48, 0, 32, 32, 128, 0), (6, 48, 1, 32, 32, 64, 0), (5, 64, 64, 32, 32, 128, 0),
    (5, 80, 130, 28, 4, 128, 13), (9, 32, 200, 32, 32, 128, 20), (9, 96, 320, 16, 16, 64, 0),
    (33, 16, 190, 8, 8, 128, 0), (20, 32, 449, 16, 16, 128, 44), (64, 16, 513, 8, 1, 128, 5),
    # blocks that end at and past half a key tile, many lanes (dealt depth first)
    (17, 32, 200, 16, 16, 128, 0), (17, 48, 200, 16, 16, 64, 0), (40, 80, 70, 8, 8, 128, 0),
    (40, 96, 70, 8, 8, 64, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_key_tile_edges(case):
    L, B, P, Hq, Hkv, D, n_ref = case
    step = synth.make_step("tiny", 5, with_weight=False, D=D, B=B, L=max(L, 1), tree="random",
                           Hq=Hq, Hkv=Hkv, P=P, refresh_frac=n_ref / P if P else 0.0, depth_max=4,
                           V=64, d=64)
    assert step.n_ref == n_ref
    if L == 0:
        import paper_2606_08411_amd as al
        import torch
        from gpu_util import dev, dev_bf16, host_bf16_f32
        kp, vp = dev_bf16(step.k_pre), dev_bf16(step.v_pre)
        _, _, o, lse = al.lane_attn_forward(
            None, None, None, kp, vp, [], B, refresh_idx=dev(step.refresh_idx),
            q_ref=dev_bf16(step.q_ref), k_ref=dev_bf16(step.k_ref), v_ref=dev_bf16(step.v_ref))
        torch.cuda.synchronize()
        k, v = oracle.attention.refresh_scatter(f32(step.k_pre), f32(step.v_pre), step.refresh_idx,
                                                f32(step.k_ref), f32(step.v_ref))
        ro, rl = oracle.attention.refresh_attention(f32(step.q_ref), k, v)
        assert np.abs(host_bf16_f32(o) - ro).max() < TOL_O
        assert np.abs(lse.cpu().numpy() - rl).max() < TOL_LSE
        return
    out = _run(step)
    ref = oracle.attention.decode_attention(
        f32(step.q), f32(step.k_lane), f32(step.v_lane), f32(step.k_pre), f32(step.v_pre),
        step.parent, step.B, step.refresh_idx, f32(step.q_ref), f32(step.k_ref), f32(step.v_ref))
    assert np.abs(out["o"] - ref["o"]).max() < TOL_O
    assert np.abs(out["lse"] - ref["lse"]).max() < TOL_LSE
    if n_ref:
        assert np.abs(out["o_ref"] - ref["o_ref"]).max() < TOL_O
        assert np.abs(out["lse_ref"] - ref["lse_ref"]).max() < TOL_LSE


def test_rounding_does_not_depend_on_the_other_lanes():
    """With key splits, which keys a partial holds is a matter of the call's sizes: the result of a
    lane that only sees itself has the same bits whatever the other lanes of its workgroup see."""
    import paper_2606_08411_amd as al
    import torch
    from gpu_util import dev_bf16
    L, B = 20, 32
    step = synth.make_step("tiny", 5, with_weight=False, D=128, B=B, L=L, tree="linear", Hq=16,
                           Hkv=16, P=449, V=64, d=64)
    a = [dev_bf16(x) for x in (step.q, step.k_lane, step.v_lane, step.k_pre, step.v_pre)]
    got = []
    for parent in ([-1] * L, list(range(-1, L - 2)) + [-1]):   # alone / a chain, the last lane alone
        o, lse, _, _ = al.lane_attn_forward(*a, parent, B)
        got.append((o[-B:].clone(), lse[-B:].clone()))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
