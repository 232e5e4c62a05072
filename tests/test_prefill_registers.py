"""The bf16 prefill kernels keep their scalar values in scalar registers (all but one or two): a spilled one travels through vector lanes, which cost
a prefill of a ragged length 1 to 2 % when the kernels' arguments were held through the work items. Read from the compiler's
own resource figures (no GPU)."""
import os
import re
import subprocess

from paper_2506_11104_amd import build as hip_build


def test_bf16_prefill_kernels_spill_no_scalar_registers(tmp_path):
    out = tmp_path / "dam_prefill.s"
    src = os.path.join(hip_build.CSRC, "dam_prefill.hip")
    subprocess.run(["hipcc", "--cuda-device-only", "-S", src, "-o", str(out)] + hip_build.FLAGS, check=True, capture_output=True, timeout=300)
    kernels = re.findall(r"\.name: +(\S+)\n(?:.*\n)*?.*\.sgpr_spill_count: +(\d+)", out.read_text())
    pipe = {name: int(n) for name, n in kernels if "k_prefill_bf16_pipe" in name}
    assert len(pipe) == 8, sorted(pipe)
    assert all(n <= 4 for n in pipe.values()), pipe  # 42 to 102 with the arguments held
