"""The host's own rules (csrc/plan.h and the headers beside it): sizes of buffers, waits, choices of kernels.  tests/host_rules_check.cpp
includes those headers; it is compiled for the host only and needs no GPU."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no ROCm compiler here")
    out = str(tmp_path_factory.mktemp("host_rules") / "host_rules_check")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-value",
                    os.path.join(ROOT, "tests", "host_rules_check.cpp"), "-o", out], check=True)
    return out


def _run(program, name):
    r = subprocess.run([program, name], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-3000:]


def test_decode_buffers_hold_every_forward_that_uses_them(program):
    """A quadratic step of B (B + 1) <= 32 rows runs on the decode kernels, also where max_block is smaller than that."""
    _run(program, "decode_rows")


def test_barriers_wait_whatever_the_number_of_barriers_before(program):
    """The epochs of a context run through 2^31 and 2^32: no barrier may count as passed when its launch starts."""
    _run(program, "barrier_words")


def test_down_projection_takes_tiles_that_measured_well_at_every_ffn(program):
    """The rule weighs a round's fixed part and its part per k-step: what is right for FFN 11008 is not for 2816."""
    _run(program, "down_plan")


def test_norm_kernel_by_rows_and_hidden_size(program):
    _run(program, "norm")


def test_lm_head_product_only_where_its_offsets_reach(program):
    """Vocabularies of 4 GiB and more keep the decode path's LM head, which has no such limit; so do contexts without a forward of
    more than 32 rows, which would never read the copy of the weights."""
    _run(program, "lm_product")


def test_every_reason_to_give_up_has_its_own_text(program):
    _run(program, "device_errors")


def test_phase_trace_leaves_out_two_token_tiles(program):
    _run(program, "trace")


def test_down_phase_has_a_flag_for_every_row_tile(program):
    _run(program, "down_flags")


def test_timeline_of_17_to_32_rows_is_refused_before_anything_runs():
    for block in ("17", "32"):
        r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--timeline", "--block", block], stdout=subprocess.PIPE,
                           stderr=subprocess.STDOUT, text=True, timeout=120)
        assert r.returncode == 2 and "at most 16" in r.stdout, r.stdout[-2000:]
