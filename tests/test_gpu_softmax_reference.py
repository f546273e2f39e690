"""Softmax references of the 16-row attention kernels: scores that pass a row's
reference by far more than the headroom, again and again in later key tiles,
and rows that see no key in the first tiles of a split, against the oracle.
Every query has one large, almost equal component and the prefix keys have
nothing else, in blocks of equal keys whose score rises by 100 from block to
block: the scores are far apart between blocks and equal within one, so the
weights do not hang on the rounding of a score, and the tolerance is the
suite's 1e-2 of the largest value for bf16 operands."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Case, dev_prefix, rel_err, tol

pytestmark = pytest.mark.gpu


def _shape(dh, heads, kv, tokens, prefix, batch):
    return synth.Workload("softmax_ref", n_layers=1, width=256, n_q_heads=heads, n_kv_heads=kv,
                          head_dim=dh, mlp_dim=256, action_dim=8, chunk_len=tokens // 4,
                          n_chunks=4, prefix_len=prefix, batch=batch, dtype=synth.BF16)


# (head_dim, heads, kv heads, tokens, prefix, streams): both kernels (64/192
# staged through registers, 128/256 direct to LDS); more than 64 rows, with
# splits that start in the prefix, at its end and in the buffer, and without
CASES = [(256, 8, 1, 100, 300, 1), (128, 8, 2, 132, 97, 1), (64, 4, 2, 200, 160, 1),
         (192, 4, 1, 100, 70, 2), (256, 8, 1, 260, 40, 16), (64, 2, 1, 260, 5, 40)]


@pytest.mark.parametrize("mode", ["causal", "isolated"])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_rising_scores(shape, mode):
    w = _shape(*shape)
    W = synth.make_weights(w, 0)
    dh = w.head_dim
    W["b_mod"][0][w.width:2 * w.width] = 3.0       # the normalised input is near 3 ...
    W["wq"][0][:, dh - 1::dh] = 0.0625             # ... and this query feature near 48, its
    case = Case(w, weights=W)                      # rotary angle below 0.1 at every position
    try:
        case.ex.set_mask_mode(mode)
        case.k[:] = 0.0
        block = np.arange(case.k.shape[2]) // 24
        case.k[..., dh - 1] = synth.round_to_bf16(
            (100.0 / 48.0 * np.sqrt(dh) * block).astype(np.float32))[None, None, :, None]
        kd, vd = dev_prefix(w, case.k, case.v)
        case.ex.set_prefix(kd, vd, case.lens)
        v = case.gpu_velocity()
        assert np.isfinite(v).all()
        for b in sorted({0, w.batch - 1}):
            ref = oracle.velocity(case.x[b], case.t[b], case.k[:, b], case.v[:, b],
                                  int(case.lens[b]), case.W, case.w, mask=mode)
            errs = [rel_err(v[b, k], ref[k]) for k in range(w.n_chunks)]
            print(shape, mode, b, max(errs))
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()
