"""The benchmark's summaries of profiler output, on made-up rows (CPU)."""
import pytest

import bench


@pytest.mark.parametrize("prep", ["void prep_kernel<float>(float const*, int const*)",
                                  "void prep4_kernel<unsigned short>(unsigned short const*, int const*)"])
def test_act_steps_start_at_either_frame_prep_kernel(prep):
    """The act loop's launches are cut into steps at the frame prep: either
    form of it, and not the core's prep kernel."""
    step = [prep, "void gemm_kernel<ConvFwdUProb<float>, float, 64, 64, 2, 2, false>(...)",
            "act_core_prep_kernel(...)", "act_head_kernel(...)"]
    rows = [{"Kernel_Name": n, "Grid_Size_X": 256, "Grid_Size_Y": 1} for n in 6 * step]
    out = "\n".join(bench.act_step_positions(rows, lambda r: 2.0))
    assert "(4 launches, 3 steps averaged): kernel sum 8.0 us" in out


def test_counters_list_the_stems_weight_gradient_by_itself(tmp_path):
    """Of the learner probe's launches the first weight gradient is the stem's."""
    rows = ["Dispatch_Id,Kernel_Name,Grid_Size,Counter_Name,Counter_Value", "1,copyBuffer,1,X,7",
            "2,cast_bf16_kernel,256,X,1", "3,gemm_kernel<ConvFwdUProb>,1,X,1", "4,gemm_kernel<ConvWgradQProb>,1,X,2",
            "5,gemm_kernel<ConvDgradProb>,1,X,3", "6,gemm_kernel<ConvWgradQProb>,1,X,4",
            "7,gemm_kernel<ConvWgradProb>,1,X,5"]
    csv = tmp_path / "counters.csv"
    csv.write_text("\n".join(rows))
    out = bench.summarize_counters(str(csv))
    assert out["copy_calibration"] == [{"X": 7.0}]
    assert {k: (v["dispatches"], v["X"]) for k, v in out["classes"].items()} == {
        "conv forward GEMM": (1, 1.0), "stem conv weight-gradient GEMM": (1, 2.0), "conv data-gradient GEMM": (1, 3.0),
        "conv weight-gradient GEMM": (2, 9.0)}
