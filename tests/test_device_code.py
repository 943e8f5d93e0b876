"""What the compiler makes of the attention kernels: those of 16-bit pools that run units of either row-tile class read a plan's tables and fp8
scales as the kernels of one class do, by scalar loads, and none needs scratch memory."""
import os
import re
import subprocess

import pytest

from paper_2401_06761_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _compiled(tmp_path_factory, source):
    """Per kernel of a source, by its mangled name: vector loads of one or two words, bytes of scratch."""
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    asm = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    csrc = os.path.join(ROOT, "paper_2401_06761_amd", "csrc")
    done = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-x", "hip", "--cuda-device-only", "-S",
                           os.path.join(csrc, source), "-o", asm], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr[-3000:]
    text = open(asm).read()
    found = {}
    for name in re.findall(r"^\s*\.amdhsa_kernel (\S+)", text, re.M):
        body = re.search(rf"^{re.escape(name)}:.*?^\.Lfunc_end", text, re.S | re.M).group(0)
        scratch = re.search(rf"\.amdhsa_kernel {re.escape(name)}.*?private_segment_fixed_size (\d+)", text, re.S).group(1)
        found[name] = (len(re.findall(r"^\s+global_load_dword(?:x2)? ", body, re.M)), int(scratch))
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return _compiled(tmp_path_factory, "kernels_attn_bf16.hip")


def _one(kernels, pattern):
    return next(v for k, v in kernels.items() if pattern in k)


@pytest.mark.parametrize("f8,split,inline", [(0, 0, 0), (0, 1, 0), (0, 1, 1), (1, 0, 0), (1, 1, 0), (1, 1, 1)])
def test_kernels_of_both_classes_load_as_those_of_one_do(kernels, f8, split, inline):
    rest = f"ELb{f8}ELb{split}ELb{inline}EE"
    both = _one(kernels, f"attention_bf16_bothILb{f8}ELb{split}ELb{inline}EE")
    one, two = (_one(kernels, f"attention_bf16ILi{nt}{rest}") for nt in (1, 2))
    # (the words of a list that each lane reads for itself are vector loads in all of them)
    assert both[0] <= one[0] + two[0]


def test_no_kernel_needs_scratch(kernels):
    assert len(kernels) == 18 and all(scratch == 0 for _, scratch in kernels.values()), kernels


@pytest.mark.parametrize("source,n", [("kernels_few_bf16.hip", 16), ("kernels_attn_f32.hip", 6)])
def test_no_kernel_of_other_sources_needs_scratch(tmp_path_factory, source, n):
    found = _compiled(tmp_path_factory, source)
    assert len(found) == n and all(scratch == 0 for _, scratch in found.values()), found


def test_matrix_kernels(tmp_path_factory):
    found = _compiled(tmp_path_factory, "kernels_matrix_bf16.hip")
    assert len(found) == 3 and all(scratch == 0 for _, scratch in found.values()), found
    # a unit's workgroup reads its list of blocks by scalar loads: left are a lane's thread and the last block's fill count
    assert _one(found, "attention_units_bf16")[0] <= 2


def test_statements_say_that_they_write_m0():
    """Inline assembly that sets M0 names it among what it overwrites: the compiler may keep a value of its own there."""
    csrc = os.path.join(ROOT, "paper_2401_06761_amd", "csrc")
    setting = 0
    for name in sorted(os.listdir(csrc)):
        for body in re.findall(r"\basm(?:\s+volatile)?\s*\((.*?)\);", open(os.path.join(csrc, name)).read(), re.S):
            if re.search(r"\bs_mov_b32 m0\b", body):
                setting += 1
                assert '"m0"' in body.rsplit(":", 1)[1], (name, body)
    assert setting >= 2
