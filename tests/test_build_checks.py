"""What the build says about device code (no GPU): faults stop it, what only costs speed does not."""
import pathlib
import warnings

import pytest

from paper_2505_05856_amd import build as bld

STEP = ["ds_read_b128 v[0:3], v9", "v_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[0:3], v[4:7]"]
WAIT = ["#ASMSTART", "s_waitcnt vmcnt(4)", "#ASMEND"]


def check(monkeypatch, lines, src="gemm_pair.hip"):
    monkeypatch.setattr(bld, "device_asm", lambda _, asm: pathlib.Path(asm).write_text("\n".join([".LBB0_1:"] + lines) + "\n"))
    with warnings.catch_warnings(record=True) as said:
        warnings.simplefilter("always")
        bld._check_device_asm(src)
    return [str(w.message) for w in said]


@pytest.fixture(autouse=True)
def scratch(monkeypatch, tmp_path):
    monkeypatch.setattr(bld, "OBJ", str(tmp_path))


def test_one_wait_a_step_is_what_the_build_expects(monkeypatch):
    assert check(monkeypatch, STEP + WAIT + ["s_barrier"]) == []


def test_a_second_wait_is_said_and_built(monkeypatch):
    said = check(monkeypatch, STEP + ["s_waitcnt vmcnt(0)"] + WAIT + ["s_barrier"])
    assert len(said) == 1 and "gemm_pair.hip" in said[0] and "1 k-steps" in said[0]


def test_a_step_without_a_wait_stops_the_build(monkeypatch):
    with pytest.raises(RuntimeError, match="does not wait"):
        check(monkeypatch, STEP + ["s_barrier"])


def test_m0_outside_the_inline_asm_stops_the_build(monkeypatch):
    assert check(monkeypatch, ["#ASMSTART", "s_mov_b32 m0, s4", "#ASMEND"]) == []
    with pytest.raises(RuntimeError, match="M0"):
        check(monkeypatch, ["s_mov_b32 m0, s4"])
