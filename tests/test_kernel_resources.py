"""Registers and scratch of the built kernels (code object metadata, no GPU)."""
import os
import random
import re

import pytest

from paper_2608_02134_amd import binding as B

from .code_objects import kernels

CSRC = os.path.join(os.path.dirname(B.LIB_PATH), "csrc")


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libgmc.so is not built; run __graft_entry__.build()")
    return kernels(B.LIB_PATH)


def _find(built, pattern):
    found = {n: k for n, k in built.items() if re.search(pattern, n)}
    assert found, pattern
    return found


def test_head_gram_keeps_its_registers(built):
    """No probe rank (1..8, with and without 16-byte runs) spills to scratch."""
    found = _find(built, r"headgram_kernelILi\dELb[01]")
    assert len(found) == 16
    assert {n: k[".private_segment_fixed_size"] for n, k in found.items() if k[".private_segment_fixed_size"]} == {}


def test_audit_keeps_its_registers(built):
    """No head dimension (32..256) spills to scratch, in either type."""
    found = _find(built, r"audit_(full|compact)_kernel")
    assert len(found) == 32
    assert {n: k[".private_segment_fixed_size"] for n, k in found.items() if k[".private_segment_fixed_size"]} == {}


# --- selections that run side by side ----------------------------------------------
# A selection's blocks wait for each other.  Two may be in flight on a device:
# one of the context, one of the static entry point.
CU_REGS, CU_LDS, CUS = 512, 160 * 1024, 48   # (as many CUs as a quick simulation takes)


def _regs(k):
    return (k[".vgpr_count"] + 7) // 8 * 8   # the unified file is given out in eights


@pytest.fixture(scope="module")
def limits():
    text = open(os.path.join(CSRC, "gmc_select.h")).read()
    return {n: eval(v) for n, v in re.findall(r"\b(k[A-Z]\w*) = ([0-9 *]+)[,;]", text)}


def _variants(built):
    """(name, registers, static LDS, half) of every selection kernel."""
    out = []
    for name, k in _find(built, r"select_(stream|wide|split|hold)_kernel").items():
        hold = re.search(r"select_hold_kernelILi(\d+)ELi(\d+)ELb([01])", name)
        half = not hold or (hold.group(3) == "0" and int(hold.group(1)) * int(hold.group(2)) <= 20)
        out.append((name, _regs(k), k[".group_segment_fixed_size"], half))
    return out


def test_selection_blocks_leave_the_room_they_count_on(built, limits):
    gate, = _find(built, r"bank_gate_kernel").values()
    assert _regs(gate) <= limits["kGateRegs"] and gate[".group_segment_fixed_size"] == 0
    cluster, = _find(built, r"cluster_kernel").values()
    assert _regs(cluster) + limits["kHalfRegs"] + limits["kGateRegs"] <= CU_REGS
    assert cluster[".group_segment_fixed_size"] + limits["kHalfLdsStatic"] <= CU_LDS
    for k in _find(built, r"take_turn_kernel|zero_fill_kernel").values():
        assert _regs(k) <= limits["kWaitRegs"] and k[".group_segment_fixed_size"] == 0
    assert limits["kWholeRegs"] + limits["kGateRegs"] + limits["kWaitRegs"] <= CU_REGS
    assert 2 * limits["kHalfRegs"] + limits["kGateRegs"] <= CU_REGS
    assert limits["kHalfLds"] + limits["kHalfLdsStatic"] <= CU_LDS
    for name, regs, lds, half in _variants(built):
        assert regs <= limits["kHalfRegs" if half else "kWholeRegs"], name
        assert lds <= limits["kSelStaticLds"], name


def _stuck(rng, a, b, gate):
    """Blocks (registers, LDS) of two grids of one block per CU each start in any
    order on any CU with room: True if both can end up partly resident."""
    regs, lds = [0] * CUS, [0] * CUS
    regs[0] = gate
    left = [CUS, CUS]
    for step in range(8 * CUS):
        g = rng.choice([0, 1]) if step < 6 * CUS else step & 1
        fits = [c for c in range(CUS) if regs[c] + (a, b)[g][0] <= CU_REGS and lds[c] + (a, b)[g][1] <= CU_LDS]
        if left[g] and fits:
            # mostly where the other fits no longer or is already: the worst orders
            c = rng.choice(fits) if rng.random() < 0.5 else max(fits, key=lambda c: regs[c])
            regs[c] += (a, b)[g][0]
            lds[c] += (a, b)[g][1]
            left[g] -= 1
    return left[0] > 0 and left[1] > 0


def test_selections_side_by_side_never_wait_for_each_others_room(built, limits):
    """Every pair that the plan lets run together becomes resident, at least one
    grid at a time; a pair that it does not may get stuck."""
    rng = random.Random(1)
    half = sorted({r for _, r, _, h in _variants(built) if h})
    for a in half:
        for b in half:
            for lds_b in (limits["kHalfLds"], limits["kHalfLdsStatic"]):
                for _ in range(3):
                    assert not _stuck(rng, (a, limits["kHalfLds"]), (b, lds_b), limits["kGateRegs"]), (a, b, lds_b)
    whole = max(r for _, r, _, h in _variants(built) if not h)
    assert any(_stuck(rng, (whole, limits["kHalfLds"]), (half[-1], limits["kHalfLds"]), 0) for _ in range(3))
