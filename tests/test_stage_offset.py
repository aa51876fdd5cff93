"""Where a stage's bytes start in a chunk of the one-wave leaf kernels: the
helper both kernels take it from, compiled for the host, up to the last stage
of the longest chunk (2^37 bytes), and no other stage offset in their sources.
On the CPU: the chain of a chunk beyond 4 GiB takes a lane minutes."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_23938_amd", "csrc")
STAGES = [0, 1, (1 << 25) - 1, 1 << 25, (1 << 25) + 1, (1 << 30) - 1]


def test_offsets(tmp_path):
    src = tmp_path / "stage.cpp"
    src.write_text('#include <stdio.h>\n#include "stage.h"\nint main() {\n' + "".join(
        f'    printf("%llu\\n", (unsigned long long)hv::stage_offset({s}u));\n' for s in STAGES) + "}\n")
    exe = tmp_path / "stage"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-std=c++17",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    assert got == [128 * s for s in STAGES]


def test_every_stage_offset_comes_from_it():
    for name in ("sha256_leaves.hip", "sha384_leaves.hip"):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        # the next stage's loads, aligned and at any alignment
        assert len(re.findall(r"const uint64_t off = stage_offset\(nx\);", text)) == 2, name
        assert not re.search(r"kStageBytes \* n?x\b", text), name
