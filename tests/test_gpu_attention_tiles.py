"""The 8-tile attention kernel at the edges of its key-tile ring: 0 to 47 prefix
tiles of 64 keys (odd and even, full and ragged), lane blocks of 1 and 2 tiles,
and every number of key splits and of query tiles per workgroup that the plan
chooses, for lanes and for refreshed rows (test_plans_host.py checks that).

Against the fp64 oracle; outputs are bf16 (half a step of the largest values
met, below 4, is 2^-8) and P is rounded to bf16 (relative 2^-9 of a convex
combination of values below 5): within 2e-2.  LSE within 2e-3: a rounded P moves it
by at most 2^-8 of that key's share, and the smallest case has 40 keys.
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
    # 8 query tiles unsplit; 2 to 16 splits of lanes, some starting inside the lane
    # tiles; refreshed rows with 8 query tiles, with 2 and with 4 splits
    (5, 16, 65, 224, 32, 64, 0), (16, 16, 65, 28, 4, 64, 0), (33, 16, 130, 16, 16, 64, 0),
    (64, 16, 65, 16, 16, 64, 0), (17, 16, 65, 16, 16, 64, 0), (33, 48, 65, 2, 2, 64, 0),
    (8, 80, 1300, 1, 1, 128, 0), (33, 16, 1300, 2, 2, 64, 0), (64, 16, 65, 4, 4, 64, 0),
    (33, 16, 1300, 4, 2, 128, 0), (33, 16, 1300, 1, 1, 64, 0), (40, 16, 1300, 2, 2, 64, 0),
    (9, 16, 65, 32, 16, 128, 0), (0, 16, 200, 224, 32, 64, 129), (0, 16, 1000, 14, 2, 64, 669),
    (0, 16, 1000, 56, 8, 64, 129), (0, 16, 1500, 112, 16, 128, 65),
    # lane blocks in contiguous shares and dealt to the splits
    (57, 80, 1357, 6, 6, 64, 0), (60, 16, 450, 16, 16, 64, 0), (46, 16, 1096, 12, 6, 64, 0),
    (64, 80, 3000, 4, 4, 64, 0), (5, 16, 700, 56, 8, 64, 0), (10, 48, 1409, 1, 1, 64, 0),
    (9, 16, 3000, 16, 16, 64, 0), (1, 16, 3000, 1, 1, 64, 0), (17, 16, 3000, 4, 2, 64, 0),
    (16, 32, 700, 4, 4, 128, 0), (0, 16, 3000, 8, 2, 64, 914), (0, 16, 3000, 28, 4, 64, 294),
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


@pytest.mark.parametrize("case", [(20, 449, 16), (16, 2048, 32)], ids=["dealt", "contiguous"])
def test_rounding_does_not_depend_on_the_other_lanes(case):
    """With key splits, which keys a partial holds is a matter of the call's sizes: the result of a
    lane that only sees itself has the same bits whatever the other lanes of its workgroup see."""
    import paper_2606_08411_amd as al
    import torch
    from gpu_util import dev_bf16
    L, P, H = case
    B = 32
    step = synth.make_step("tiny", 5, with_weight=False, D=128, B=B, L=L, tree="linear", Hq=H,
                           Hkv=H, P=P, V=64, d=64)
    a = [dev_bf16(x) for x in (step.q, step.k_lane, step.v_lane, step.k_pre, step.v_pre)]
    got = []
    for parent in ([-1] * L, list(range(-1, L - 2)) + [-1]):   # alone / a chain, the last lane alone
        o, lse, _, _ = al.lane_attn_forward(*a, parent, B)
        got.append((o[-B:].clone(), lse[-B:].clone()))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("case", [(9, 32, 3333, 32, 8, 128), (12, 64, 1500, 8, 2, 128)], ids=str)
def test_fewer_splits_keep_fp32_partials(case):
    """Rounding P (bf16) and the output (bf16) each give a relative error of about 2^-9 / sqrt(1.4) =
    1.65e-3, 2.33e-3 together (2-norms); bf16 partials would add a third, 2.85e-3 in all."""
    import paper_2606_08411_amd as al
    import torch
    L, B, P, Hq, Hkv, D = case
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    mk = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    q, kl, vl, kp, vp = mk(L * B, Hq, D), mk(L * B, Hkv, D), mk(L * B, Hkv, D), mk(P, Hkv, D), mk(P, Hkv, D)
    o, _, _, _ = al.lane_attn_forward(q, kl, vl, kp, vp, list(range(-1, L - 1)), B)   # a chain
    see = torch.ones((L, L), device="cuda").tril().bool().repeat_interleave(B, 0).repeat_interleave(B, 1)
    see = torch.cat([torch.ones((L * B, P), dtype=torch.bool, device="cuda"), see], 1)
    num = den = 0.0
    for h in range(Hq):
        k = torch.cat([kp[:, h // (Hq // Hkv)], kl[:, h // (Hq // Hkv)]]).double()
        v = torch.cat([vp[:, h // (Hq // Hkv)], vl[:, h // (Hq // Hkv)]]).double()
        z = torch.mm(q[:, h].double(), k.t().contiguous()) / D ** 0.5
        ref = torch.mm(torch.softmax(z.masked_fill(~see, -float("inf")), 1), v)
        num += float((o[:, h].double() - ref).pow(2).sum())
        den += float(ref.pow(2).sum())
    assert (num / den) ** 0.5 < 2.6e-3
