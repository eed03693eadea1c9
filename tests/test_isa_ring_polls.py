"""The polls of the forward exchange's ring, checked in the compiled code (no GPU
needed).  A slot of the ring is rewritten every four steps and any value that is
not all ones is taken for the current h, so its loads must be non-temporal (nt),
which leaves no line in the L1, and carry no scope bits, which would send them
past the L2; the flags' polls too."""

import re

from tests.test_isa_waits import _assembly


def _body(lines, start):
    for line in lines[start + 1:]:
        s = line.split(";")[0].strip()
        if s.startswith(".Lfunc_end"):
            return
        yield s


def test_ring_polls_are_non_temporal_loads(tmp_path):
    lines = _assembly(tmp_path)
    heads = [(i, m) for i, l in enumerate(lines)
             if (m := re.match(r"^(_Z\w*lstm_fwd_xcdILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)\w*):", l))]
    rings = 0
    for i, m in heads:
        mt, ks, staged = int(m.group(2)), int(m.group(3)), m.group(5) == "1"
        loads = [s for s in _body(lines, i) if re.match(r"(global|flat|buffer)_load_", s) and "lds" not in s]
        nt = [s for s in loads if re.search(r"\bnt\b", s)]
        assert nt and all(not re.search(r"\bsc[01]\b", s) for s in nt), m.group(1)
        wide = [s for s in nt if s.startswith("global_load_dwordx4")]
        if mt == 1 and staged:
            # a wave polls a quarter of the row's lines, 8 rows at a time
            per_poll = -(-ks // 4)
            assert len(wide) >= per_poll and len(wide) % per_poll == 0, (m.group(1), len(wide), per_poll)
            rings += 1
        else:
            assert not wide, m.group(1)
    assert rings >= 20
