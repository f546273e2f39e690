"""Softmax references of the few-row attention (passes of at most 64 token
rows), whose waves take key tiles of their own, rescale in the loop and merge
once: scores that rise by 100 from block to block of keys, far past the
headroom, so that a wave rescales again and again, and that stay at their
maximum in every fourth block of the last third, so that waves and splits end
on different references and several of them carry weight.  Equal keys within a
block have equal scores, so the weights do not hang on rounding, and the
tolerances are the suite's: 1e-2 of the largest value in bf16, 1e-4 in fp32."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Case, dev_prefix, rel_err, tol

pytestmark = pytest.mark.gpu

# (head_dim, heads, kv heads, chunks, actions, prefix, streams): prefixes of
# several tiles a wave, and (the last three) of fewer tiles than waves
CASES = [(64, 2, 1, 4, 4, 2900, 1), (128, 8, 2, 4, 16, 1500, 1), (192, 4, 2, 3, 7, 1300, 2),
         (256, 8, 1, 5, 10, 2000, 1), (256, 2, 2, 2, 1, 3000, 30), (64, 2, 1, 4, 5, 5, 3),
         (256, 8, 1, 4, 4, 33, 1), (128, 2, 1, 1, 3, 1, 2)]


@pytest.mark.parametrize("mode", ["causal", "isolated"])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.FP32])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_rising_scores(shape, dtype, mode):
    dh, heads, kv, K, C, P, B = shape
    w = synth.Workload("softmax_few", n_layers=1, width=256, n_q_heads=heads, n_kv_heads=kv,
                       head_dim=dh, mlp_dim=256, action_dim=8, chunk_len=C, n_chunks=K,
                       prefix_len=P, batch=B, dtype=dtype)
    W = synth.make_weights(w, 0)
    W["b_mod"][0][w.width:2 * w.width] = 3.0       # the normalised input is near 3 ...
    W["wq"][0][:, dh - 1::dh] = 0.0625             # ... and this query feature near 48, its
    case = Case(w, weights=W)                      # rotary angle small at every position
    try:
        case.ex.set_mask_mode(mode)
        case.k[:] = 0.0
        block = np.arange(case.k.shape[2]) // 24
        last = int(block.max(initial=0))
        level = np.where((block > 2 * last // 3) & (block % 4 == last % 4), last, block * 2 // 3)
        case.k[..., dh - 1] = synth.round_to_bf16(
            (100.0 / 48.0 * np.sqrt(dh) * level).astype(np.float32))[None, None, :, None]
        kd, vd = dev_prefix(w, case.k, case.v)
        case.ex.set_prefix(kd, vd, case.lens)
        v = case.gpu_velocity()
        assert np.isfinite(v).all()
        for b in sorted({0, B - 1}):
            ref = oracle.velocity(case.x[b], case.t[b], case.k[:, b], case.v[:, b],
                                  int(case.lens[b]), case.W, case.w, mask=mode)
            errs = [rel_err(v[b, k], ref[k]) for k in range(K)]
            print(shape, dtype, mode, b, max(errs))
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()
