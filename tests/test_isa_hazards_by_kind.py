"""Wait states of the hand-written vector instructions that tests/test_isa_hazards.py does not look at: the 16-pass fp32
MFMAs, whose results take longer than those of the 8-pass ones, and scalar registers that a vector instruction writes
(comparison masks, lane reads) and a hand-written one reads, in the selection kernels as well."""
import functools
import os
import re

import pytest

from tests import test_isa_hazards as hz

# one compilation of a source serves both files
hz._isa = functools.lru_cache(maxsize=None)(hz._isa)

MFMA_WAIT_STATES = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x2_f32": 20}   # passes + 3, + 1 on gfx950
SGPR_WAIT_STATES = 2   # a vector instruction's scalar result as the operand or carry of another one


def scalar_results_and_operands(text):
    """SGPRs that a vector instruction writes, and those that it reads."""
    op, _, rest = text.partition(" ")
    ops = [o.strip() for o in rest.split(",")]
    n_dst = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_", op) else 1
    wrote = set().union(*[hz._sregs(o) for o in ops[:n_dst]])
    read = set().union(*[hz._sregs(o) for o in ops[n_dst:]]) if len(ops) > n_dst else set()
    return wrote, read


def hand_written_readers_of_fresh_sgprs(ins, need):
    """In straight-line order, as the compiler lays the code out."""
    found = []
    for i, (text, by_hand) in enumerate(ins):
        if not by_hand or not text.startswith("v_"):
            continue
        read, ws = scalar_results_and_operands(text)[1], 0
        for j in range(i - 1, -1, -1):
            if ws >= need or not read:
                break
            u = ins[j][0]
            if u.startswith("v_") and scalar_results_and_operands(u)[0] & read:
                found.append((ws, u, text))
                break
            m = re.match(r"s_nop (\d+)", u)
            ws += int(m.group(1)) + 1 if m else 1
    return found


def test_the_checkers_find_planted_exposures():
    ins = [("v_mfma_f32_32x32x2_f32 v[0:15], v20, v21, v[0:15]", False)] + [("s_nop 7", False), ("s_nop 4", False)] + \
          [("v_max3_f32 v30, v0, v1, v2", True), ("s_endpgm", False)]
    is_fp32 = lambda t: t.startswith("v_mfma_f32_32x32x2_f32")
    assert [h[0] for h in hz.exposed_readers(ins, {}, is_fp32, MFMA_WAIT_STATES["v_mfma_f32_32x32x2_f32"])] == [13]
    assert hz.exposed_readers(ins, {}, is_fp32, 12) == []
    cmp, add = "v_cmp_le_u32_e64 s[4:5], s8, v1", "v_addc_co_u32_e64 v2, s[4:5], 0, v2, s[4:5]"
    other = ("v_cmp_le_u32_e64 s[6:7], s9, v1", True)
    assert hand_written_readers_of_fresh_sgprs([(cmp, True), other, (add, True)], 2) == [(1, cmp, add)]
    assert hand_written_readers_of_fresh_sgprs([(cmp, True), other, other, (add, True)], 2) == []
    lane = "v_readfirstlane_b32 s8, v9"
    assert hand_written_readers_of_fresh_sgprs([(lane, False), (cmp, True)], 2) == [(0, lane, cmp)]


@pytest.mark.parametrize("source,masks", [("topk.hip", True), ("select_ragged.hip", True), ("compact.hip", True),
                                          ("score_mfma.hip", False), ("patch_attn.hip", False)])
def test_no_hand_written_instruction_reads_too_early(source, masks):
    if not os.path.exists(hz.HIPCC):
        pytest.skip("hipcc not present")
    n_mfma, n_masks = 0, 0
    for name, ins, labels in hz._kernels(hz._isa(source)):
        early = hand_written_readers_of_fresh_sgprs(ins, SGPR_WAIT_STATES)
        assert not early, (name, early[:3])
        n_masks += sum(by_hand and t.startswith("v_addc_co_u32_e64") for t, by_hand in ins)
        kinds = {t.split()[0] for t, _ in ins if t.startswith("v_mfma")}
        assert kinds <= set(MFMA_WAIT_STATES), (name, kinds)
        for kind in kinds:
            n_mfma += 1
            hits = hz.exposed_readers(ins, labels, lambda t: t.startswith(kind + " "), MFMA_WAIT_STATES[kind])
            assert not hits, (name, hits[:3])
    assert (n_masks > 0) == masks and (n_mfma > 0) == (not masks)
