"""Every built instance of the LM-head tile kernel (test_plans_host.py checks that the cases reach
them all): one and several tiles per workgroup, over 9 K stages of 64 (so that every ring of stages
wraps) and over a ragged K, W packed and as given, with rows of W ragged against its 8-row pieces;
and the packed variants that load W non-temporally, on weights larger than 384 MB.

Against torch in 64 bits.  Tolerance: a logit is an fp32 sum of d products (|h| < 25, |w| ~ 1/sqrt(d),
|z| up to ~30), whose partial sums round with random signs: about 2^-24 30 sqrt(d / 32) = 4e-5 at d =
16384 (32 products a matrix instruction); the exponent's argument is rounded at ~1e-5: conf and lse
within 1.5e-4.  argmax exact where the top-2 gap exceeds
1e-3.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # N, V at d = 576 and, ragged, V - 3 at d = 568
    (1, 72), (1349, 328), (1271, 328), (1217, 520), (133, 10960), (1301, 648), (67, 16480), (97, 16480), (131, 16480),
    (195, 16480), (1, 33000), (1, 131200), (33, 33040), (33, 163880), (67, 33000), (211, 20600), (100, 82400),
    (133, 33160), (131, 84200), (292, 18280), (294, 43760), (326, 21920), (165, 83400), (180, 41400),
    (180, 82400), (197, 36200), (197, 83400), (213, 41160), (213, 82200), (229, 41400), (229, 82200), (487, 21880),
    (490, 43920), (1, 65680), (40, 65680), (1, 133400), (40, 133400), (1, 178000), (518, 10880), (265, 43760), (197, 33240), (330, 43840), (389, 22000),
    (390, 43680), (440, 22800), (580, 33040), (326, 33200), (328, 65800), (545, 21920), (356, 66040), (785, 16560),
    (398, 65800), (70, 82400), (70, 166200), (1, 107200), (1, 122400), (1, 214800), (1, 244000), (2, 82400),
    (2, 197000), (40, 123000), (40, 246000), (40, 82400), (70, 98600), (270, 83200),
]
SIZES = [(N, d, v) for N, V in CASES for d, v in ((576, V), (568, V - 3))] + [
    (70, 1152, 166320), (77, 1144, 166317), (34, 64, 204144), (34, 40, 204141)]
NT_CASES = [  # N, V at d = 4096 and, ragged, V - 3 at d = 4072
    (1, 47520), (40, 47520), (70, 47520), (100, 47520), (135, 47600), (150, 48000), (165, 48400), (180, 47800),
    (200, 47800), (213, 47800), (230, 47600), (245, 48200), (1, 65800), (40, 65800), (70, 66000), (100, 65900), (135, 66200),
    (150, 65900), (165, 65900), (180, 66200), (200, 65900), (70, 82400), (2, 122400), (2, 82400), (40, 122600),
    (40, 82400), (70, 99200),
]
NT_WIDE = [  # narrow tiles: V at d = 8192 and V - 3 at d = 8152; at twice those d
    (1, 30000, 1), (40, 30000, 1), (70, 30000, 1), (100, 28000, 1), (150, 30000, 1), (200, 28000, 1),
    (1, 14000, 2), (40, 14000, 2), (70, 14000, 2), (140, 14000, 2),
]
NT_SIZES = [(N, d, v) for N, V in NT_CASES for d, v in ((4096, V), (4072, V - 3))] + [
    (N, d * m, v) for N, V, m in NT_WIDE for d, v in ((8192, V), (8152, V - 3))]


def _check(N, d, V, packed):
    import paper_2606_08411_amd as al
    g = torch.Generator(device="cuda")
    g.manual_seed(N * 1000003 + d * 1009 + V)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = torch.empty((V, d), dtype=torch.bfloat16, device="cuda")
    for i in range(0, V, 16384):
        W[i:i + 16384] = rnd(min(16384, V - i), d) / d ** 0.5
    H = (rnd(N + 3, d) * (1 + 5 * torch.rand((N + 3, 1), generator=g, device="cuda"))).bfloat16()
    rows = torch.randperm(N + 3, generator=g, device="cuda")[:N].to(torch.int32)
    sup = (torch.rand(N, generator=g, device="cuda") < 0.5).to(torch.uint8)
    kw = dict(row_idx=rows, suppress_eos=sup, eos_id=V // 3)
    if packed:
        conf, arg, lse = al.lmhead_confidence_packed(H, al.lmhead_pack_weight(W), V, **kw)
    else:
        conf, arg, lse = al.lmhead_confidence(H, W, **kw)
    h = H[rows.long()].double()
    z = torch.cat([torch.mm(h, w.double().t().contiguous()) for w in W.split(16384)], 1)
    z[sup.bool(), V // 3] = -float("inf")
    top, idx = z.topk(2, dim=1)
    ref = torch.logsumexp(z, 1)
    clear = top[:, 0] - top[:, 1] >= 1e-3
    assert (~clear).sum() <= max(2, N // 50)
    assert torch.equal(arg[clear].long(), idx[clear, 0])
    assert (lse - ref).abs().max() < 1.5e-4
    assert (conf - torch.exp(top[:, 0] - ref)).abs().max() < 1.5e-4


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("size", SIZES, ids=str)
def test_instance(size, packed):
    _check(*size, packed)


@pytest.mark.parametrize("size", NT_SIZES, ids=str)
def test_non_temporal(size):
    N, d, V = size
    _check(N, d, V, True)
