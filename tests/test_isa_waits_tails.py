"""The same check as test_isa_waits.py for the chunks of every size: hidden
sizes that are odd multiples of 64 leave a wave's k-slice with a chunk of two
k-steps or one after its chunks of four.  Each chunk's wait must leave in
flight only operations issued after the chunk's last direct load."""

import re

from tests.test_isa_waits import _assembly, _events


def _chunks(kw):
    rem = kw % 4
    return [4] * (kw // 4) + {0: [], 1: [1], 2: [2], 3: [2, 1]}[rem]


def test_every_chunk_wait_leaves_only_later_operations_in_flight(tmp_path):
    lines = _assembly(tmp_path)
    heads = [(i, m) for i, l in enumerate(lines)
             if (m := re.match(r"^(_Z\w*lstm_bwd_xcdILi(\d+)ELi(\d+)ELi(\d+)E\w*):", l))]
    assert {int(m.group(4)) % 4 for _, m in heads} == {0, 1, 2, 3}
    for i, m in heads:
        mt, kw = int(m.group(2)), int(m.group(4))
        loads = [mt * c for c in _chunks(kw)]  # direct loads of each chunk
        ends = [sum(loads[:k + 1]) for k in range(len(loads))]
        ops, waits, sections = None, 0, 0
        for e in _events(lines, i):
            if ops is None:
                if e[0] == "D":
                    ops, waits = [e], 0
                continue
            if e[0] != "W":
                ops.append(e)
                continue
            d = [j for j, o in enumerate(ops) if o[0] == "D"]
            assert len(d) >= ends[waits], (m.group(1), waits, len(d))
            after = len(ops) - d[ends[waits] - 1] - 1
            assert after >= e[1], (m.group(1), waits, after, e[1])
            waits += 1
            if waits == len(loads):
                sections += 1
                ops = None
        assert sections >= 1, m.group(1)
