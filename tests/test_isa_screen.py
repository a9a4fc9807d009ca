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


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_private_memory_stays_out_of_the_products_of_small_lookups():
    """Up to 32 queries everything is in registers; beyond, what a wave keeps in scratch memory is written before its rounds and read outside their products."""
    asm = isa_check.device_asm("lookup_bytes.hip")
    sizes = isa_check.private_segment_sizes(asm)
    few = {k: l for k, l in isa_check.kernels(asm).items() if "k_bytes_few" in k}
    assert len(few) == 21
    for name, lines in few.items():
        products = [i for i, l in enumerate(lines) if l.startswith("v_mfma_i32")]
        scratch = [i for i, l in enumerate(lines) if l.startswith("scratch_")]
        assert not any(products[0] < i < products[-1] for i in scratch), name
        assert not any(i > products[0] and lines[i].startswith("scratch_store") for i in scratch), name
        assert "ELi2ELi8EE" in name or sizes[name] == 0, name
        assert sizes[name] <= 64, (name, sizes[name])
