"""The checks that build() makes on the device assembly: they hold for the kernels as they are, and each refuses the mistake
it is there for."""
import os
import re
import subprocess
import tempfile

import pytest

import __graft_entry__ as build

UNITS = ["k_stream.hip", "k_prefill.hip"]


@pytest.fixture(scope="module")
def device_asm():
    """Device assembly of the units the checks are about, with the flags of the build."""
    flags = [f for f in build.FLAGS if not f.startswith("-save-temps")]
    with tempfile.TemporaryDirectory() as d:
        out = {u: os.path.join(d, u + ".s") for u in UNITS}
        jobs = [subprocess.Popen([build.HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(build.CSRC, u), "-o", out[u]],
                                 stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL) for u in UNITS]
        assert all(j.wait() == 0 for j in jobs)
        yield out


def _plant(tmp_path, text):
    p = tmp_path / "planted.s"
    p.write_text(text)
    return str(p)


def test_range_checked_accesses_have_no_scalar_offset(device_asm):
    for u, path in device_asm.items():
        build._check_buffer_offsets(u, path)


@pytest.mark.parametrize("line,ok", [
    ("\tbuffer_load_dword v11, v14, s[8:11], s33 offen", False),
    ("\tbuffer_load_dword v11, v14, s[8:11], s33 offen offset:64", False),
    ("\tbuffer_store_dword v11, v14, s[8:11], s33 offen", False),
    ("\tbuffer_load_dwordx4 v[4:7], v14, s[8:11], 0 offen offset:1024 nt", True),
    ("\tbuffer_load_dwordx4 v14, s[8:11], s33 offen lds", True)])
def test_scalar_offset_check(tmp_path, line, ok):
    path = _plant(tmp_path, line + "\n")
    if ok:
        build._check_buffer_offsets("x", path)
    else:
        with pytest.raises(RuntimeError, match="scalar offset"):
            build._check_buffer_offsets("x", path)


def test_products_of_the_pipelined_gemm_keep_their_registers(device_asm):
    path = device_asm["k_prefill.hip"]
    with open(path) as f:
        kernels = re.findall(r"^_ZN2bd\w*pf_gemm_pipe_kernel\w*:", f.read(), re.M)
    assert kernels and build._check_accumulators("k_prefill.hip", path) == len(kernels)


GOOD = """\
\t; BD_ACC_BEGIN
\tv_add_u32_e32 v0, s0, v9
\tds_read_b128 v[0:3], v0
\tds_read_b128 v[4:7], v21
\ts_waitcnt lgkmcnt(0)
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]
\tv_mfma_f32_16x16x32_bf16 v[12:15], v[0:3], v[4:7], v[12:15]
\tbuffer_load_dwordx4 v0, s[8:11], s33 offen lds
\ts_nop 15
\ts_nop 15
\t; BD_ACC_END
\tv_accvgpr_read_b32 v0, a0
"""


@pytest.mark.parametrize("old,new,what", [
    ("", "", None),
    ("a[0:3], v[0:3], v[4:7], a[0:3]", "a[0:3], v[0:3], v[4:7], a[4:7]", "not in place"),
    ("\tbuffer", "\tv_accvgpr_read_b32 v30, a2\n\tbuffer", "moved, read or spilled"),
    ("\tbuffer", "\tv_mov_b32_e32 v30, v13\n\tbuffer", "moved, read or spilled"),
    ("\tbuffer", "\tv_add_f32_e32 v15, v15, v30\n\tbuffer", "moved, read or spilled"),
    ("\tbuffer", "\tscratch_store_dwordx4 off, v[40:43], off\n\tbuffer", "moved, read or spilled"),
    ("\tv_mfma_f32_16x16x32_bf16 a", "\tv_mov_b32_e32 v5, v30\n\tv_mfma_f32_16x16x32_bf16 a", "written by v_mov"),
    ("\ts_nop 15\n\ts_nop 15\n", "\ts_nop 15\n", "no wait"),
    ("\t; BD_ACC_END\n", "", "missing")])
def test_accumulator_check(tmp_path, old, new, what):
    assert old in GOOD
    path = _plant(tmp_path, GOOD.replace(old, new, 1))
    if what is None:
        assert build._check_accumulators("x", path) == 1
    else:
        with pytest.raises(RuntimeError, match=what):
            build._check_accumulators("x", path)
