"""Few-row passes (at most 64 token rows: one-pass GEMMs straight into MFMA
registers, key-split attention on 16-row tiles, tiled activations) against the
oracle, at the edges of their row tiles and wave splits.  Tolerances are the
suite's: 1e-2 of the largest value for bf16 operands, 1e-4 for fp32."""
import numpy as np
import pytest

import synth
from gpu_util import Case, dev, rel_err, tol

pytestmark = pytest.mark.gpu


def _shape(name, dtype, **kw):
    base = dict(n_layers=2, width=128, n_q_heads=2, n_kv_heads=1, head_dim=64, mlp_dim=128,
                action_dim=8, chunk_len=4, n_chunks=4, prefix_len=40, batch=1)
    base.update(kw)
    return synth.Workload(name, dtype=dtype, **base)


CASES = [
    # rows 1 and 2 with fewer k blocks than waves; one query row tile, partly filled
    dict(chunk_len=1, n_chunks=1, n_q_heads=1, head_dim=128, prefix_len=2),
    dict(chunk_len=1, n_chunks=2, prefix_len=1),
    # row tiles exactly full, one row over, one short (16, 17, 32, 33, 48, 49, 63, 64) ...
    dict(chunk_len=8, n_chunks=2),
    dict(chunk_len=17, n_chunks=1, head_dim=192, n_q_heads=4, n_kv_heads=2),
    dict(chunk_len=8, n_chunks=4, width=256, mlp_dim=576, n_q_heads=4, head_dim=128, prefix_len=33),
    dict(chunk_len=11, n_chunks=3, n_q_heads=6, n_kv_heads=2, head_dim=64, width=384),
    dict(chunk_len=12, n_chunks=4, n_q_heads=8, head_dim=256, prefix_len=70),
    dict(chunk_len=7, n_chunks=7, mlp_gated=False, prefix_len=130),
    dict(chunk_len=21, n_chunks=3, n_q_heads=4, head_dim=64, prefix_len=500),
    dict(chunk_len=16, n_chunks=4, width=1024, n_q_heads=8, head_dim=128, mlp_dim=2048, prefix_len=97),
    # ... and the first row count of the tiled kernels
    dict(chunk_len=13, n_chunks=5),
    # ragged streams in one row tile; FiLM rows 33..64 with more waves than k
    # blocks and two column groups per workgroup (8 layers of width 128)
    dict(batch=3, chunk_len=5, n_chunks=3, prefix_len=(0, 60), n_kv_heads=2),
    dict(batch=6, chunk_len=1, n_chunks=10, n_layers=8, prefix_len=(3, 30)),
    # the widest expert: two column groups per thread in the reductions
    dict(chunk_len=9, n_chunks=2, width=2048, mlp_dim=192, n_layers=1),
]


@pytest.mark.parametrize("dtype", [synth.BF16, synth.FP32])
@pytest.mark.parametrize("kw", CASES, ids=lambda k: "-".join(f"{a}{b}" for a, b in k.items())
                         .replace(" ", ""))
def test_few_row_velocity(kw, dtype):
    w = _shape("few", dtype, **kw)
    case = Case(w)
    try:
        # every stream at noise levels of its own, so that all FiLM rows are computed
        case.t = (case.t - np.arange(w.batch, dtype=np.float32)[:, None] * 0.01 / w.batch
                  ).astype(np.float32)
        case.td = dev(case.t)
        v = case.gpu_velocity()
        for b in range(w.batch):
            ref = case.oracle_velocity(b)
            errs = [rel_err(v[b, k], ref[k]) for k in range(w.n_chunks)]
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()
