"""What the kernel sources ask of the compiler (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2606_23419_amd import build as b


@pytest.mark.parametrize("src", ["vmm_mm.hip"])
def test_inline_asm_compiles_without_warnings(src, tmp_path):
    # an asm block that names a reserved register (m0) as a clobber is undefined
    flags = [f for f in b.HIPCC_FLAGS if f != "-Werror=inline-asm"]
    r = subprocess.run([b.hipcc(), *flags, *b.SOURCE_FLAGS.get(src, []), "-c", os.path.join(b.CSRC, src),
                        "-o", str(tmp_path / "o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "warning" not in r.stderr, r.stderr[:2000]


def _code(src):
    """A kernel source without its comments."""
    with open(os.path.join(b.CSRC, src)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def test_lut_copies_are_waited_for_before_the_barrier():
    # no register depends on a copy to LDS, and a barrier alone does not wait
    # for copies in flight: the source has to ask for it
    after = _code("vmm_lut.hip").split("__builtin_amdgcn_global_load_lds(")[-1]
    assert "s_waitcnt vmcnt(0)" in after.split("__syncthreads()")[0]


def test_decode_adds_are_one_instruction_each():
    # the copies are waited for by counting the memory instructions behind them:
    # the adds of a column are written as the one instruction that is counted
    code = _code("vmm_mm.hip")
    columns = code.split("wait_copies(nlate")[1].split("float lost")[0]
    assert "add_to(yo" in columns and not re.search(r"\batomicAdd\b|__hip_atomic|unsafeAtomicAdd", columns)
    assert re.search(r'asm volatile\("global_atomic_add_f32 %0, %1, off"', code)


def test_lut_channels_are_loaded_at_once(tmp_path):
    # the run's x and level bytes all go out before the first wait
    out = tmp_path / "lut.s"
    r = subprocess.run([b.hipcc(), *b.HIPCC_FLAGS, *b.SOURCE_FLAGS.get("vmm_lut.hip", []), "--cuda-device-only", "-S",
                        os.path.join(b.CSRC, "vmm_lut.hip"), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = re.split(r"\n(?=_ZN\S*k_vmm_lut\S*:)", out.read_text())[1:]
    assert len(kernels) == 6
    for k in kernels:
        name, body = k.split("\n", 1)
        prologue = body.split("s_barrier")[0]
        before = re.split(r"s_waitcnt[^\n]*vmcnt", prologue)[0]
        loads = r"global_load_u(?:short|byte)"
        assert len(re.findall(loads, before)) == len(re.findall(loads, prologue)) >= 4, name
