"""Every stage that cola_trace_stage_name lists is recorded by some launch in the sources
(host-only)."""
import os
import re

import paper_1301_0322_amd as cola


def test_every_listed_stage_is_recorded():
    src = open(os.path.join(cola.HERE, "csrc", "cola_api.cpp")).read()
    enum = re.search(r"enum Stage : int \{(.*?)kNumStages", src, re.S).group(1)
    ids = re.findall(r"kSt\w+", enum)
    lib = cola.lib()
    assert lib.cola_trace_stage_count() == len(ids)
    names = [lib.cola_trace_stage_name(k) for k in range(len(ids))]
    assert all(names) and len(set(names)) == len(names) and lib.cola_trace_stage_name(len(ids)) is None
    rest = src.replace(enum, "")
    assert [i for i in ids if not re.search(rf"\b{i}\b", rest)] == []
