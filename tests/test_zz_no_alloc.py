"""fv_decode_step_noalloc (scratch in the library's static device array)
against fv_decode_step (scratch owned by the handle), through the C ABI.

Same kernels in the same order: the emitted chunk, the buffer and the noise
state must be bit-identical, on two calls in a row, the second with a smaller
input (fewer streams, or a shorter prefix).  The static array keeps the
previous call's contents, so the second call also shows that nothing in it
has to start at zero.  A step whose scratch exceeds the array is rejected
before anything is enqueued.
"""
import numpy as np
import pytest

import synth
from paper_2608_27384_amd import flashvla as fvb
from tests.gpu_util import Case, dev, host

pytestmark = pytest.mark.gpu


def _stream():
    import torch
    return int(torch.cuda.current_stream().cuda_stream)


def _noalloc(case):
    st = fvb.lib().fv_decode_step_noalloc(case.ex.handle, case.xd.data_ptr(),
                                          case.td.data_ptr(), case.out.data_ptr(), _stream())
    assert st == fvb.FV_OK, fvb.lib().fv_last_error(case.ex.handle)


def _same_step(a, r):
    _noalloc(a)
    r.ex.decode_step(r.xd, r.td, r.out)
    assert np.array_equal(host(a.out), host(r.out))
    assert np.array_equal(host(a.xd), host(r.xd))
    assert a.ex.noise_state == r.ex.noise_state


def _set_batch(case, nb, lens=None):
    """Installs the first nb streams of the case's prefix (smaller input)."""
    lens = [int(x) for x in (case.lens[:nb] if lens is None else lens)]
    case.ex.set_prefix(case.kd[:, :nb].contiguous(), case.vd[:, :nb].contiguous(), lens)
    case.xd = dev(host(case.xd)[:nb])
    case.td = dev(case.t[:nb])
    case.out = case.out[:nb].contiguous()


def test_noalloc_matches_decode_step_then_smaller_batch():
    w = synth.workload("small_bf16_b3")
    a, r = Case(w, noise_seed=4), Case(w, noise_seed=4)
    try:
        assert a.ex.attn_split(3) > 1   # the attention partials live in the static array
        assert 0 < a.ex.noalloc_scratch_bytes(3) <= fvb.FV_NOALLOC_SCRATCH_BYTES
        _same_step(a, r)                # batch 3
        _set_batch(a, 1)
        _set_batch(r, 1)
        _same_step(a, r)                # batch 1: smaller input, same array
    finally:
        a.close()
        r.close()


def test_noalloc_matches_decode_step_pi05_then_shorter_prefix():
    w = synth.workload("pi05_b1")
    a, r = Case(w, noise_seed=6), Case(w, noise_seed=6)
    try:
        need = a.ex.noalloc_scratch_bytes(1)
        print(f"pi05_b1: {need} bytes of static scratch "
              f"(split partials and split-K tiles), limit {fvb.FV_NOALLOC_SCRATCH_BYTES}")
        assert 0 < need <= fvb.FV_NOALLOC_SCRATCH_BYTES
        _same_step(a, r)
        _set_batch(a, 1, [300])         # a shorter observation prefix
        _set_batch(r, 1, [300])
        _same_step(a, r)
    finally:
        a.close()
        r.close()


def test_noalloc_rejects_a_step_larger_than_the_array():
    w = synth.Workload("noalloc_big", n_layers=1, width=128, n_q_heads=8, n_kv_heads=1,
                       head_dim=256, mlp_dim=256, action_dim=8, chunk_len=50, n_chunks=10,
                       prefix_len=64, batch=2, dtype=synth.BF16)
    case = Case(w, noise_seed=1)
    try:
        need = case.ex.noalloc_scratch_bytes(2)
        assert need > fvb.FV_NOALLOC_SCRATCH_BYTES
        x0, ns = host(case.xd).copy(), case.ex.noise_state
        st = fvb.lib().fv_decode_step_noalloc(case.ex.handle, case.xd.data_ptr(),
                                              case.td.data_ptr(), case.out.data_ptr(), _stream())
        assert st == fvb.FV_ERR_INVALID_ARG
        assert b"scratch" in fvb.lib().fv_last_error(case.ex.handle)
        assert np.array_equal(host(case.xd), x0) and case.ex.noise_state == ns
        ref = Case(w, noise_seed=1)
        try:
            _set_batch(case, 1)
            _set_batch(ref, 1)
            assert case.ex.noalloc_scratch_bytes(1) <= fvb.FV_NOALLOC_SCRATCH_BYTES
            _same_step(case, ref)
        finally:
            ref.close()
    finally:
        case.close()


def test_noalloc_counts_the_film_products_of_several_streams():
    """Streams at noise levels of their own compute their FiLM maps in
    products of K and (batch - 1) K rows, which the plan may split where one of
    batch K rows is not: at width 896 in fp32, time-MLP products of 4600 rows
    in 2 splits of 33 MB together, of 4800 rows unsplit.  With t the step asks
    for them and is refused; with a schedule it computes none and runs."""
    w = synth.Workload("noalloc_film", n_layers=1, width=896, n_q_heads=2, n_kv_heads=1,
                       head_dim=64, mlp_dim=128, action_dim=8, chunk_len=4, n_chunks=200,
                       prefix_len=8, batch=24, dtype=synth.FP32)
    a, r = Case(w, noise_seed=2), Case(w, noise_seed=2)
    try:
        assert a.ex.noalloc_scratch_bytes(24) >= 2 * 23 * 200 * 896 * 4
        st = fvb.lib().fv_decode_step_noalloc(a.ex.handle, a.xd.data_ptr(), a.td.data_ptr(),
                                              a.out.data_ptr(), _stream())
        assert st == fvb.FV_ERR_INVALID_ARG
        for c in (a, r):
            c.ex.set_schedule(c.td)
            c.td = None
        st = fvb.lib().fv_decode_step_noalloc(a.ex.handle, a.xd.data_ptr(), None,
                                              a.out.data_ptr(), _stream())
        assert st == fvb.FV_OK, fvb.lib().fv_last_error(a.ex.handle)
        r.ex.decode_step(r.xd, None, r.out)
        assert np.array_equal(host(a.out), host(r.out))
        assert np.array_equal(host(a.xd), host(r.xd))
    finally:
        a.close()
        r.close()
