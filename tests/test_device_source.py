"""Rules of the device source that no result shows reliably, checked on its text (no GPU)."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1402_6601_amd", "csrc")
HIP = sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _asm_statements(path):
    """The instruction lists of the inline assembly statements of a source file."""
    text = open(path).read()
    out = []
    for m in re.finditer(r'\basm\s+volatile\s*\(\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', text):
        body = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1)))
        out.append([i.strip() for i in re.split(r"\\n(?:\\t)?|;", body) if i.strip()])
    return out


def _wait_states(ins):
    m = re.match(r"s_nop\s+(\w+)", ins)
    return int(m.group(1), 0) + 1 if m else 1


@pytest.mark.parametrize("path", HIP, ids=os.path.basename)
def test_wait_states_before_lds_transfers(path):
    """What the compiler sees to in its own code, but not inside assembly: a
    scalar write of M0 and the transfer into LDS that reads it are one wait state
    apart; and a transfer's scalar base, which a vector instruction
    (readfirstlane, the restore of a spilled scalar) may have written right before
    the statement, is copied by a scalar instruction of the statement or read
    five wait states after its start."""
    found = 0
    for ins in _asm_statements(path):
        for at, b in enumerate(ins):
            if "_lds_" not in b:
                continue
            found += 1
            before = ins[:at]
            m0 = [k for k, a in enumerate(before) if re.match(r"s_\w+\s+m0\b", a)]
            assert m0 and sum(_wait_states(a) for a in before[m0[-1] + 1:]) >= 1, ins
            base = b.split(",")[-1].strip()
            if base != "off":
                copied = any(re.match(r"s_\w+\s+%s\b" % re.escape(base), a) for a in before)
                assert copied or sum(_wait_states(a) for a in before) >= 5, ins
    if path.endswith("tchol_device.hip"):
        assert found >= 5  # the transfers are still found


def test_claim_words_have_one_writer():
    """Every wavefront reads the words of a claim after its barrier, at its own
    time: nothing but the claim stores them, so that no wavefront can find a word
    that another one has gone on to overwrite."""
    text = open(os.path.join(CSRC, "tchol_device.hip")).read()
    stores = re.findall(r"\bs_claim\[(\w+)\]\s*=(?!=)", text)
    assert len(stores) >= 6 and sorted(set(stores)) == sorted(stores), stores


def test_wavefronts_agree_on_skipping():
    """Whether a work item is skipped is read once per workgroup, by the claim: a
    load by every wavefront could find a failure word that another workgroup
    changes in between, and the wavefronts' barriers would not match.  (The
    compact instance may load it anywhere: its systems' tasks follow each other.)"""
    text = open(os.path.join(CSRC, "tchol_device.hip")).read()
    loads = [l.strip() for l in text.splitlines() if re.search(r"ld_relaxed\(&a\.sinfo\[", l)]
    assert loads
    for at in re.finditer(r"ld_relaxed\(&a\.sinfo\[", text):
        guard = text[max(0, at.start() - 60):at.start()]
        assert re.search(r"if \((wave == 0|COMPACT)\) \{\s*[^{}]*$", guard), guard


def test_no_kernel_is_chosen_by_a_fixed_order():
    """A system's order is compared with nothing but sizes of its own: which
    kernel runs follows from tile sizes, types and alignment."""
    text = open(os.path.join(CSRC, "tchol_device.hip")).read()
    assert re.findall(r"\bsn\s*[<>]=?\s*(?:\d+|[A-Z][A-Z_0-9]+)\b", text) == []
