"""Wide experts at 65 to 400 rows against the oracle: QKV and gate/up (or the
plain up product) split along k with a reduction kernel of their own, or not,
on both sides of the rule; several streams, whose time-MLP rows go through the
same rule.  Tolerance: the suite's 1e-2 of the largest value (bf16)."""
import numpy as np
import pytest

import synth
from gpu_util import Case, dev, rel_err, tol

pytestmark = pytest.mark.gpu

# (width, heads, kv heads, head_dim, mlp_dim, gated, streams, chunks, actions)
CASES = [(1152, 2, 1, 64, 128, True, 1, 5, 13),      # 65 rows, 18 k-tiles: unsplit
         (1536, 4, 2, 64, 256, False, 2, 5, 19),     # 190 rows, 24 k-tiles: 4 splits
         (1536, 8, 1, 256, 1024, True, 1, 10, 32),   # 320 rows, 2304 and 2048 columns: unsplit
         (1920, 2, 1, 64, 192, True, 40, 2, 1),      # 80 rows, 78 of them FiLM rows of their own
         (1920, 4, 1, 128, 512, True, 8, 5, 10),     # 400 rows: unsplit
         (2048, 2, 1, 64, 128, False, 1, 9, 9)]      # 81 rows, 8 splits of 32 k-tiles


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_wide_experts(shape):
    W, hq, hkv, dh, F, gated, B, K, C = shape
    w = synth.Workload("wide", n_layers=1, width=W, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh,
                       mlp_dim=F, action_dim=8, chunk_len=C, n_chunks=K, prefix_len=(0, 50),
                       batch=B, dtype=synth.BF16, mlp_gated=gated)
    case = Case(w)
    try:
        # every stream at noise levels of its own: every FiLM row is computed
        case.t = (case.t - np.arange(B, dtype=np.float32)[:, None] * 0.01 / B).astype(np.float32)
        case.td = dev(case.t)
        v = case.gpu_velocity()
        for b in sorted({0, B // 2, B - 1}):
            ref = case.oracle_velocity(b)
            errs = [rel_err(v[b, k], ref[k]) for k in range(K)]
            print(shape, b, max(errs))
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()


# (layers, chunks = FiLM rows of width 512, dtype): wide FiLM products on both
# sides of 32 rows and 16384 columns, and of the fp32 kernel's four column groups
FILM = [(4, 33, synth.BF16), (5, 33, synth.BF16), (6, 64, synth.BF16), (6, 32, synth.BF16),
        (5, 48, synth.FP32), (7, 17, synth.FP32), (7, 32, synth.FP32), (7, 16, synth.FP32)]


@pytest.mark.parametrize("shape", FILM, ids=lambda s: "x".join(map(str, s)))
def test_wide_film_products(shape):
    L, K, dtype = shape
    w = synth.Workload("film", n_layers=L, width=512, n_q_heads=2, n_kv_heads=1, head_dim=64,
                       mlp_dim=128, action_dim=8, chunk_len=2, n_chunks=K, prefix_len=9, batch=1,
                       dtype=dtype)
    case = Case(w)
    try:
        v, ref = case.gpu_velocity(), case.oracle_velocity(0)
        errs = [rel_err(v[0, k], ref[k]) for k in range(K)]
        print(shape, max(errs))
        assert max(errs) < tol(w), errs
    finally:
        case.close()
