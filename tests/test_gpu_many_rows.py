"""Many-row passes at the edges of their rules, against the oracle: the
embedding and velocity head on the matrix units (from 1024 rows on, partly
filled 16-row tiles, action dims that are no multiple of 4), QKV on 64x128
tiles in one round (1300 rows), gate/up on 256x256 tiles from 2048 rows on.
The step's Euler update, fused into the head or (an action dim that is no
multiple of 4) the queue update kernel, equals the host's on the same velocities
bit for bit, and its refill the oracle's Philox draw.  Tolerances are the suite's: 1e-2 of the largest value for bf16 operands,
1e-4 for fp32."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Case, host, rel_err, tol

pytestmark = pytest.mark.gpu

# (streams, chunks, actions, width, heads, kv heads, head_dim, mlp_dim, action_dim, dtype)
CASES = [(11, 3, 31, 128, 2, 1, 64, 128, 8, synth.BF16),      # 1023 rows: the smaller kernels
         (16, 4, 16, 256, 4, 2, 128, 256, 32, synth.BF16),    # 1024, whole tiles
         (5, 5, 41, 384, 6, 2, 64, 192, 14, synth.BF16),      # 1025, head not fused
         (13, 4, 25, 256, 8, 1, 256, 256, 4, synth.BF16),     # 1300
         (16, 3, 43, 256, 2, 1, 192, 3072, 20, synth.BF16),   # 2064
         (8, 3, 43, 128, 2, 1, 64, 128, 12, synth.FP32)]      # 1032


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_many_rows(shape):
    B, K, C, W, hq, hkv, dh, F, A, dtype = shape
    w = synth.Workload("many", n_layers=1, width=W, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh,
                       mlp_dim=F, action_dim=A, chunk_len=C, n_chunks=K, prefix_len=(0, 50),
                       batch=B, dtype=dtype)
    case = Case(w)
    try:
        v = case.gpu_velocity().copy()
        for b in sorted({0, B // 2, B - 1}):
            ref = case.oracle_velocity(b)
            errs = [rel_err(v[b, k], ref[k]) for k in range(K)]
            print(shape, b, max(errs))
            assert max(errs) < tol(w), (b, errs)
        case.ex.decode_step(case.xd, case.td, case.out)
        new, out = host(case.xd), host(case.out)
        t = case.t.astype(np.float32)
        dt = t - np.concatenate([np.zeros((B, 1), np.float32), t[:, :-1]], axis=1)
        x = case.x.astype(np.float32) - dt[:, :, None, None] * v
        assert np.array_equal(out, x[:, 0])
        assert np.array_equal(new[:, :-1], x[:, 1:])
        z = np.stack([oracle.gaussian_chunk(case.noise_seed + b, 0, C, A) for b in range(B)])
        assert np.max(np.abs(new[:, -1] - z)) <= 1e-6
        assert np.count_nonzero(new[:, -1] != z) <= 2  # fp64 libm ties only
    finally:
        case.close()
