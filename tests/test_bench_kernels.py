"""The benchmark's stage-to-kernel map and the counter summaries name kernels
that the library has, by the library's own rules (at most 64 rows, 1024 rows
and more, the fused Euler update)."""
import subprocess

import pytest

import bench
import synth
from paper_2608_27384_amd import counters
from paper_2608_27384_amd.flashvla import LIB_PATH


@pytest.fixture(scope="module")
def symbols():
    return subprocess.run(["nm", "-C", LIB_PATH], capture_output=True, text=True,
                          check=True).stdout


def _workloads():
    p = synth.workload("pi05_b1")
    return list(synth.WORKLOADS.values()) + [
        p.replace(name="wide", width=2048), p.replace(name="b3", batch=3),
        p.replace(name="adim", action_dim=14), p.replace(name="adim48", action_dim=48, batch=4),
        p.replace(name="fp32", dtype=synth.FP32, head_dim=64, batch=2, mlp_gated=False)]


@pytest.mark.parametrize("w", _workloads(), ids=lambda w: w.name)
@pytest.mark.parametrize("splits", [1, 4])
def test_every_stage_names_a_kernel_of_the_library(w, splits, symbols):
    for stage, (label, match) in bench.stage_kernels(w, splits, splits).items():
        assert match in symbols, (stage, match)


def test_kernels_by_the_rows_of_a_pass():
    few = bench.stage_kernels(synth.workload("short_chunk"), 4, 8)
    assert [few[s][1] for s in ("attention", "qkv_gemm", "gate_up_gemm", "o_proj_gemm", "time_mlp1",
                                "euler_shift")] == [
        "attn_few_kernel", "FewQkv", "FewGeglu", "FewPartial", "FewBiasSilu",
        "final_small_kernel<true>"]
    b1 = bench.stage_kernels(synth.workload("pi05_b1"), 4, 8)
    assert [b1[s][1] for s in ("attention", "qkv_gemm", "o_proj_gemm", "time_mlp1", "embed")] == [
        "attn16d_kernel", "EpiQkv", "EpiNone", "FewBiasSilu", "embed_adarms_small_kernel"]
    b64 = bench.stage_kernels(synth.workload("batched64"), 1, 1)
    assert [b64[s][1] for s in ("o_proj_gemm", "embed", "head", "euler_shift")] == [
        "EpiGatedResid", "embed_adarms_mma_kernel", "final_mma_kernel", "final_mma_kernel<true>"]


@pytest.mark.parametrize("w", _workloads(), ids=lambda w: w.name)
def test_a_step_ends_at_its_euler_update(w):
    """The counter summaries cut a trace into steps there."""
    stages = bench.stage_kernels(w, 4, 4)
    ends = [s for s, (_, match) in stages.items() if counters._step_end(match)]
    assert ends == ["euler_shift"]


def test_a_change_of_any_kernel_source_makes_the_summaries_stale():
    import glob
    import os
    src = {"csrc/" + os.path.basename(p)
           for p in glob.glob(os.path.join(counters.PKG, "csrc", "*.hip"))}
    assert src <= set(counters.ALL_SRC)
