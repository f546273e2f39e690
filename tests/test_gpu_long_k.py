"""An MLP so wide that the down projection leaves the direct-to-LDS tiles (from
2^22 k on, where their 32-bit byte offsets end), and the widest that stays on
them.  All but 256 of the hidden features have zero weights, spread to both
ends of k, so the oracle runs the 256 alone; their outputs are scaled up until
the velocity hangs on them.  Tolerance: the suite's 1e-2 of the largest value."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Case, rel_err, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [(1 << 22) - 128, 1 << 22])
def test_long_k(F):
    w = synth.Workload("longk", n_layers=1, width=128, n_q_heads=2, n_kv_heads=1, head_dim=64,
                       mlp_dim=256, action_dim=8, chunk_len=11, n_chunks=6, prefix_len=20, batch=1,
                       dtype=synth.BF16, mlp_gated=False)
    small = synth.make_weights(w, 0)
    small["wd"][0] = synth.round_to_bf16(small["wd"][0] * 50.0)
    small["b_mod"][1][2 * w.width:] = 1.0  # the MLP's gate
    idx = np.concatenate([np.arange(64), F // 2 + np.arange(64) * 131,
                          np.arange(F - 4096, F, 64), np.arange(F - 64, F)])
    assert len(set(idx)) == 255  # the stride and the tail share one
    idx = np.unique(np.append(idx, F // 3))
    W = dict(small)
    W["wu"], W["wd"] = [np.zeros((w.width, F), np.float32)], [np.zeros((F, w.width), np.float32)]
    W["wu"][0][:, idx] = small["wu"][0]
    W["wd"][0][idx] = small["wd"][0]
    case = Case(w.replace(mlp_dim=F), weights=W)
    try:
        v = case.gpu_velocity()

        def ref(weights):
            return oracle.velocity(case.x[0], case.t[0], case.k[:, 0], case.v[:, 0],
                                   int(case.lens[0]), weights, w)

        without = dict(small, wd=[np.zeros_like(small["wd"][0])])
        r = ref(small)
        assert rel_err(ref(without), r) > 20 * tol(w)
        errs = [rel_err(v[0, k], r[k]) for k in range(w.n_chunks)]
        print(F, errs)
        assert max(errs) < tol(w), errs
    finally:
        case.close()
