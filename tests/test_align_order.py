"""The aligner's wavefronts exchange carries through LDS without waiting for each access: what the compiled loop of the row
wavefront leaves there must be covered by a wait that the source states, not by one that the compiler happens to place (CPU:
the kernel's assembly, built from its source)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_11076_amd", "csrc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "align.s")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S", "-o", out,
                    os.path.join(CSRC, "ss_align.hip")], check=True, stderr=subprocess.DEVNULL, timeout=300)
    return open(out).read()


def loops_of_rows(text):
    """instructions (stated in an asm statement or not) of every loop that does 32 row steps"""
    found = []
    for kernel in re.findall(r"^_ZN\w*ss_align_rows_kernel\w*:.*?s_endpgm", text, flags=re.S | re.M):
        lines, label_at, stated = [], {}, False
        for line in kernel.splitlines():
            line = line.strip()
            if line.startswith(";;#ASM"):
                stated = "START" in line
            elif re.match(r"\.LBB\w+:", line):
                label_at[line.split(":")[0]] = len(lines)
            elif line and not line.startswith((";", ".")):
                lines.append((line, stated))
                m = re.match(r"s_cbranch_\w+ (\.LBB\w+)", line)
                if m and m.group(1) in label_at:
                    body = lines[label_at[m.group(1)]:]
                    if sum(x.startswith("v_bitop3") for x, _ in body) == 32:
                        found.append(body)
    return found


def test_a_strips_words_are_in_lds_a_block_later(assembly):
    loops = [b for b in loops_of_rows(assembly) if any(x.startswith("ds_write") for x, _ in b)]
    assert len(loops) == 2                                     # 16-bit and wide ids
    for body in loops:
        on_its_way, passed = [], 0                             # LDS operations, oldest first: number of the barrier they precede
        for line, stated in 3 * body:
            assert not line.startswith("s_load")               # would count as well, and end out of order
            if line.startswith("ds_"):
                on_its_way.append((line.startswith("ds_write"), passed))
            elif stated and "lgkmcnt" in line:
                n = int(re.search(r"lgkmcnt\((\d+)\)", line).group(1))
                on_its_way = on_its_way[max(0, len(on_its_way) - n):]
            elif line.startswith("s_barrier"):
                assert not any(store and at < passed for store, at in on_its_way)
                passed += 1
        assert passed == 3
