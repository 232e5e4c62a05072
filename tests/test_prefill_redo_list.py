"""Behind the first variant of the bf16 prefill every wave looks whether the workgroup's list of items to redo is empty, and wave 0
then takes entries off that list: a barrier has to lie between the two, or a wave that looks late finds the list empty and
leaves. Read from the code that the compiler makes of the kernels (no GPU: no run shows it reliably)."""
import os
import re
import subprocess

from paper_2506_11104_amd import build as hip_build


def test_no_entry_is_taken_before_every_wave_has_looked(tmp_path):
    out = tmp_path / "dam_prefill.s"
    src = os.path.join(hip_build.CSRC, "dam_prefill.hip")
    subprocess.run(["hipcc", "--cuda-device-only", "-S", src, "-o", str(out)] + hip_build.FLAGS, check=True, capture_output=True, timeout=300)
    kernels = re.findall(r"\n(_ZN\S*k_prefill_bf16_pipe\S*):(.*?)s_endpgm", out.read_text(), re.S)
    calls = {name: code.split("s_swappc_b64")[0] for name, code in kernels if "s_swappc_b64" in code}
    assert len(kernels) == 8 and len(calls) == 4, [name for name, _ in kernels]  # (the variant with a reference alone has no list)
    for name, code in calls.items():
        looked = code.rindex("ds_read")
        assert re.search(r"\n\s*s_cbranch", code[looked:]) and "s_barrier" in code[looked:], name
