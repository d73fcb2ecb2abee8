"""The LM-head tile kernel at the edges of its tiles: row counts around each column-tile width,
one and several column tiles, one and several tiles per workgroup, K ragged against the 64-element
stages, vocabularies ragged against the 32-row units and the 8-row pieces of W as given, down to one
row, one token and 8 elements.  (test_gpu_lmhead_instances.py runs every built instance.)

Against the fp64 oracle.  Tolerance: a logit is an fp32 sum of d <= 320 products
(|h| < 25, |w| ~ 1/sqrt(d), |z| up to ~30; rounding error about
sqrt(d) 2^-24 30 = 3e-5), the exponent's argument is rounded at ~1e-5: conf
and lse within 1.5e-4.  argmax exact where the oracle's top-2 gap exceeds 1e-3.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, dev_bf16, f32

pytestmark = pytest.mark.gpu

CASES = [  # N, d, V
    (1, 8, 1), (2, 64, 31), (15, 56, 33), (16, 64, 64), (17, 72, 65), (32, 128, 257),
    (33, 192, 1000), (64, 200, 2047), (65, 64, 4096), (96, 136, 5001), (97, 320, 3333),
    (128, 64, 8200), (129, 64, 70001), (144, 72, 70008), (145, 128, 70000), (161, 64, 66001),
    (177, 64, 82000), (193, 72, 90001), (205, 192, 70003), (208, 64, 70016), (209, 64, 70007),
    (224, 8, 70000), (225, 64, 70001), (241, 136, 66000), (256, 64, 131080), (257, 64, 2000),
    (273, 64, 33000), (416, 72, 66008), (417, 64, 20000), (614, 64, 40001), (625, 128, 9000),
    (77, 64, 152064), (128, 64, 152064), (160, 128, 152064), (200, 64, 152064),
]


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_tile_edges(case, packed):
    import paper_2606_08411_amd as al
    N, d, V = case
    g = np.random.default_rng([N, d, V])
    n_rows = N + 3
    scale = g.uniform(1, 6, n_rows).astype(np.float32)
    H = synth.f32_to_bf16_bits(g.standard_normal((n_rows, d), dtype=np.float32) * scale[:, None])
    W = synth.f32_to_bf16_bits(g.standard_normal((V, d), dtype=np.float32) / np.float32(np.sqrt(d)))
    rows = g.permutation(n_rows)[:N].astype(np.int32)
    eos = int(g.integers(V)) if V > 1 else -1
    sup = (g.random(N) < 0.5).astype(np.uint8)
    Wd = dev_bf16(W)
    kw = dict(row_idx=dev(rows), suppress_eos=dev(sup), eos_id=eos)
    if packed:
        conf, arg, lse = al.lmhead_confidence_packed(dev_bf16(H), al.lmhead_pack_weight(Wd), V, **kw)
    else:
        conf, arg, lse = al.lmhead_confidence(dev_bf16(H), Wd, **kw)
    torch.cuda.synchronize()
    ref = oracle.lmhead.lmhead_confidence_full(f32(H), rows, f32(W), sup, eos)
    ok = ref["gap"] >= 1e-3
    assert (~ok).sum() <= max(2, N // 50)
    assert np.array_equal(arg.cpu().numpy()[ok], ref["argmax"][ok])
    assert np.abs(conf.cpu().numpy() - ref["conf"]).max() < 1.5e-4
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() < 1.5e-4
