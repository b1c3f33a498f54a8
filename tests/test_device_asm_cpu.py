"""Inline assembly of the device code: what the compiler does not see of a statement
has to be written in it.  A statement that writes m0 names it as clobbered; the
buffer resources that buffer-to-LDS loads read from scalar registers are written by
vector instructions (v_readfirstlane), after which gfx9 needs 5 wait states, so the
statement that makes a resource leaves them, and the code built from the base kernels
keeps them and spills no scalar register (whose reload is such a write).
"""
import glob
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_11240_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\(", text):
            depth, end = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
            yield os.path.basename(path), text[m.end():end - 1]


def test_m0_is_a_named_clobber():
    writes = [(p, s) for p, s in statements() if re.search(r'(?:"|\\n\\t)s_\w+ m0\b', s)]
    assert writes
    for path, stmt in writes:
        assert '"m0"' in stmt.rsplit(":", 1)[1], (path, stmt)


def test_resources_are_made_with_their_wait_states():
    text = open(os.path.join(CSRC, "lora_base.hip")).read()
    body = text[text.index("u32x4 rsrc_words("):]
    body = body[:body.index("\n}\n")]
    nop = re.search(r'asm volatile\("s_nop (\d+)" : "\+s"\(', body)
    assert nop and int(nop.group(1)) + 1 >= 5


def registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="ROCm compilers missing")
def test_built_base_kernels_keep_the_wait_states(tmp_path):
    from paper_2401_11240_amd import build as B
    out = str(tmp_path / "base.s")
    subprocess.run([HIPCC, f"--offload-arch={B.ARCH}", "-O3", "-std=c++17", "-fPIC", f"-I{B.INCLUDE}", f"-I{CSRC}"] +
                   B.DEVICE_FLAGS + ["--cuda-device-only", "-S", os.path.join(CSRC, "lora_base.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    spills = re.findall(r"\.sgpr_spill_count:\s*(\d+)", text)
    assert spills and set(spills) == {"0"}
    code = [ln.split(";")[0].strip() for ln in text.splitlines()]
    code = [ln for ln in code if ln and not ln.startswith(".") and not ln.endswith(":")]
    loads = [i for i, ln in enumerate(code) if ln.startswith("buffer_load") and ln.endswith(" lds")]
    assert loads
    for i in loads:
        used = registers(re.split(r",\s*", code[i].split(None, 1)[1])[1])
        assert len(used) == 4, code[i]
        states, j = 0, i - 1
        while states < 5:
            op, _, args = code[j].partition(" ")
            if op.startswith("v_"):               # its scalar results come first
                written = set().union(*(registers(a) for a in re.split(r",\s*", args.strip())[:2]))
                assert not (written & used and op.startswith(("v_readfirstlane", "v_readlane", "v_cmp"))), code[j:i + 1]
            states += 1 + int(args) if op == "s_nop" else 1
            j -= 1
