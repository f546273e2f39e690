"""Scores that are not finite, in every attention kernel: keys whose product
with every query overflows to -inf weigh nothing, also where a row's first
tiles hold nothing else; a NaN or an infinity in one stream's buffer stays in
that stream, bit for bit; one in the prefix makes its stream's velocities NaN,
as the oracle's softmax does."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Case, dev_prefix, rel_err, tol

pytestmark = pytest.mark.gpu

# (head_dim, heads, kv heads, tokens, streams, dtype): few-row passes, then the
# register-staged, the direct-to-LDS and the fp32 kernel
CASES = [(64, 2, 1, 12, 2, synth.BF16), (256, 8, 1, 20, 3, synth.BF16), (128, 4, 2, 16, 2, synth.FP32),
         (64, 4, 2, 100, 2, synth.BF16), (192, 4, 1, 100, 2, synth.BF16),
         (128, 8, 2, 132, 2, synth.BF16), (256, 8, 1, 100, 3, synth.BF16),
         (64, 4, 2, 100, 2, synth.FP32), (256, 4, 2, 60, 2, synth.FP32)]
P = 150


def _case(shape):
    dh, heads, kv, tokens, B, dtype = shape
    w = synth.Workload("softmax_ext", n_layers=1, width=256, n_q_heads=heads, n_kv_heads=kv,
                       head_dim=dh, mlp_dim=256, action_dim=8, chunk_len=tokens // 4,
                       n_chunks=4, prefix_len=P, batch=B, dtype=dtype)
    W = synth.make_weights(w, 0)
    W["b_mod"][0][w.width:2 * w.width] = 3.0
    W["wq"][0][:, dh - 1::dh] = 0.0625  # this query feature is near 48 in every row
    return Case(w, weights=W)


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_minus_infinity(shape):
    case = _case(shape)
    w = case.w
    try:
        dh = w.head_dim
        huge = synth.round_to_bf16(np.array([-2.0 ** 127], np.float32))[0]
        for b in range(w.batch):  # the first tiles, a tile in between, the last keys
            for lo, hi in ((0, 70), (90, 100), (P - 3 - b, P)):
                case.k[:, b, lo:hi, :, dh - 1] = huge
        kd, vd = dev_prefix(w, case.k, case.v)
        case.ex.set_prefix(kd, vd, case.lens)
        v = case.gpu_velocity()
        assert np.isfinite(v).all()
        for b in range(w.batch):
            ref = case.oracle_velocity(b)
            errs = [rel_err(v[b, k], ref[k]) for k in range(w.n_chunks)]
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_not_finite_stays_in_its_stream(shape, bad):
    case = _case(shape)
    w = case.w
    try:
        clean = case.gpu_velocity().copy()
        x = case.x.copy()
        x[0, 1, 0, 2] = bad
        v = case.gpu_velocity(x)
        assert np.array_equal(v[1:], clean[1:])
        assert np.isnan(v[0, 1:, 0]).all()  # its own token, and the later chunks' attention
        k = case.k.copy()
        k[:, 0, 5, :, w.head_dim - 1] = bad
        kd, vd = dev_prefix(w, k, case.v)
        case.ex.set_prefix(kd, vd, case.lens)
        v = case.gpu_velocity()
        assert np.isnan(v[0]).all()
        assert np.array_equal(v[1:], clean[1:])
    finally:
        case.close()


@pytest.mark.parametrize("shape", [(256, 8, 1, 100, 3, synth.BF16), (128, 8, 2, 132, 2, synth.BF16),
                                   (256, 8, 1, 20, 3, synth.BF16), (64, 4, 2, 100, 2, synth.FP32)],
                         ids=lambda s: "x".join(map(str, s)))
def test_prefix_shorter_than_the_handle_allows(shape):
    """The key splits are planned from max_prefix: prefixes far below it (0,
    1, a few tiles) leave splits and waves without keys."""
    dh, heads, kv, tokens, B, dtype = shape
    w = synth.Workload("short_prefix", n_layers=2, width=256, n_q_heads=heads, n_kv_heads=kv,
                       head_dim=dh, mlp_dim=256, action_dim=8, chunk_len=tokens // 4, n_chunks=4,
                       prefix_len=4000, batch=B, dtype=dtype)
    case = Case(w, lens=[(0, 1, 70)[b % 3] for b in range(B)])
    try:
        v = case.gpu_velocity()
        for b in range(B):
            ref = case.oracle_velocity(b)
            errs = [rel_err(v[b, k], ref[k]) for k in range(w.n_chunks)]
            assert max(errs) < tol(w), (b, errs)
    finally:
        case.close()
