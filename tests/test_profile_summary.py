"""The matrix-core summary counts FLOP by the hardware's operation counter, so that kernels which mix
MFMA shapes (16,384 and 32,768 FLOP per instruction) are counted right (CPU only, synthetic counters)."""
import csv
import json

import pytest

from paper_2608_15171_amd import profile_summary as P


@pytest.mark.parametrize("kernel,name", [("attn_step_kernel", "void attn_step_kernel<4>(StepArgs)"),
                                         ("attn_step_kernel", "void attn_step_kernel<8>(StepArgs)"),
                                         ("gateup_kernel", "void gateup_kernel<256, false>(GemmArgs)"),
                                         ("gateup_any_kernel", "void gateup_any_kernel<false>(GemmArgs)")])
def test_mfma_flop_of_mixed_shapes(tmp_path, monkeypatch, kernel, name):
    big, small = 300, 700                                     # 32x32x16 and 16x16x32 instructions
    flop = big * 32768 + small * 16384
    values = {c: 1000 for c in P.MFMA_COUNTERS}
    values.update(SQ_INSTS_MFMA=big + small, SQ_INSTS_VALU_MFMA_MOPS_BF16=flop // 512)
    (tmp_path / "MFMA").mkdir()
    (tmp_path / "profiles").mkdir()
    with open(tmp_path / "MFMA" / "run_counter_collection.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value", "Start_Timestamp", "End_Timestamp"])
        for d in (1, 2):
            for c, v in values.items():
                w.writerow([d, name, c, v, 0, 1000])
    (tmp_path / "MFMA_bench.json").write_text(json.dumps(
        {"config": {"workload": "w"}, "roofline": {"per_launch": {"flop": 1e6}}}))
    monkeypatch.setattr(P, "ROOT", str(tmp_path))
    monkeypatch.setitem(P.DESCRIPTION, kernel, "synthetic")
    P.mfma_summary("w", str(tmp_path), kernel)
    text = (tmp_path / "profiles" / f"{kernel}.w.mfma.md").read_text()
    assert f"| FLOP of the MFMAs | {flop / 1e9:.1f} GFLOP |" in text
    assert f"| MFMA rate at the run's clock | {flop / 1e-6 / 1e12:.0f} TFLOP/s |" in text
