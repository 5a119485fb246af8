"""The prefix prefill kernel switches between its two LDS buffers by one address
bit: with static LDS in the kernel (none today; a copy of the source with some
added) the dynamic LDS behind it has to begin at a multiple of two buffers."""
import os
import re
import subprocess

from paper_2605_20600_amd.build import CSRC, HIPCC_FLAGS, ROOT, hipcc

LARGEST = 2 * 2 * 64 * 256  # two buffers of 64 K and V rows of d = 128, in bytes


def _fixed_lds(text, tmp_path):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(text.replace("../../include", os.path.join(ROOT, "include")))
    subprocess.run([hipcc(), *HIPCC_FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(src),
                    "-o", str(asm)], check=True, capture_output=True,
                   env={**os.environ, "TMPDIR": str(tmp_path)})
    return [int(x) for x in re.findall(r"amdhsa_group_segment_fixed_size (\d+)", asm.read_text())]


def test_dynamic_lds_is_aligned_to_two_buffers(tmp_path):
    with open(os.path.join(CSRC, "prefill_attn.hip")) as f:
        text = f.read()
    head = "    const int tid = threadIdx.x, lane = tid & 63;\n"
    assert text.count(head) == 1
    text = text.replace(head, "    __shared__ int pad[5];\n    pad[threadIdx.x % 5] = C;\n"
                              "    if (C == 77) out[0] = pad[0];\n" + head)
    sizes = _fixed_lds(text, tmp_path)
    assert len(sizes) == 6 and all(n > 0 and n % LARGEST == 0 for n in sizes), sizes
