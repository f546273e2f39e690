"""Sequential decode: the FiLM maps of up to 16 Euler steps come from one
product.  Against a loop of velocity passes (maps made per pass) with the
Euler update on the host, bit for bit: a map row does not depend on the rows
computed with it, and the update is a rounded product and a rounded
difference in fp32.  Step counts at the edges of a group of maps."""
import numpy as np
import pytest

import synth
from gpu_util import Case, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 16, 17, 33])
@pytest.mark.parametrize("dtype,width,batch", [(synth.BF16, 512, 1), (synth.BF16, 384, 3),
                                               (synth.BF16, 1024, 20), (synth.FP32, 128, 2)])
def test_equals_velocity_passes(steps, dtype, width, batch):
    w = synth.Workload("seqmaps", n_layers=2, width=width, n_q_heads=2, n_kv_heads=1, head_dim=64,
                       mlp_dim=256, action_dim=8, chunk_len=7, n_chunks=1, prefix_len=(3, 40),
                       batch=batch, dtype=dtype)
    case = Case(w)
    try:
        noise = np.ascontiguousarray(case.x[:, 0])
        out = dev(np.zeros_like(noise))
        for _ in range(3):  # the captured graph replays
            case.ex.sequential_decode(dev(noise), steps, out)
        got = host(out)
        x = case.x.astype(np.float32).copy()
        ts = [np.float32((steps - j) / steps) for j in range(steps + 1)]
        for j in range(steps):
            case.td = dev(np.full((batch, 1), ts[j], np.float32))
            v = case.gpu_velocity(x)
            x = x - (ts[j] - ts[j + 1]) * v
        assert np.array_equal(got, x[:, 0])
    finally:
        case.close()
