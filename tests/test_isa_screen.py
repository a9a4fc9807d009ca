"""The kernels over bytes issue their LDS fragment reads like those of lookup_mfma.hip: the same check on the generated ISA
(CPU only: hipcc cross-compiles)."""

import shutil

import pytest

import isa_check


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_fragment_reads_in_flight_and_private_memory():
    asm = isa_check.device_asm("screen.hip")
    checked = 0
    for name, lines in isa_check.kernels(asm).items():
        if any(l.startswith("ds_read_b128") and "hand-scheduled" in l for l in lines):
            bad = isa_check.inflight_violations(lines)
            assert not bad, f"{name}: {bad[:3]}"
            checked += 1
    assert checked >= 3  # two lookups and the pair search
    spilled = {k: v for k, v in isa_check.private_segment_sizes(asm).items() if v}
    assert not spilled, spilled
