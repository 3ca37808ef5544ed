"""The checks that build() makes on the device assembly: they hold for the kernels as they are, and each refuses the mistake
it is there for."""
import os
import subprocess
import tempfile

import pytest

import __graft_entry__ as build

UNITS = ["k_stream.hip"]


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
