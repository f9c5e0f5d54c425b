"""The counted waits of the prompt GEMM's pipeline (csrc/sdfp_prefill_plan.h), compiled on their own and played through a model
of a wave's memory queue: requests in the kernel's order, answered in order, a wait for at most n on their way.  The pieces of a
slab have landed, for every wave, before it is read; nothing is on its way to LDS when the workgroup ends; and it holds whether
or not the compiler keeps weight loads that bring nothing that is multiplied, unless the kernel itself keeps them."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_prefill_plan.h"
extern "C" int depth(int nt) { return sdfp::pf_weight_depth(nt); }
extern "C" int one_ahead(int nt, int wj) { return sdfp::pf_one_ahead(nt, wj); }
extern "C" int fetched(int jt, int f) { return sdfp::pf_fetched(jt, f); }
extern "C" int wait_first(int nt, int jt, int wj) { return sdfp::pf_wait_first(nt, jt, wj); }
extern "C" int wait_slab(int nt, int jt, int wj) { return sdfp::pf_wait_slab(nt, jt, wj); }
"""
# NT, JT, WJ of every instance that is launched
INSTANCES = [(3, 4, 1), (4, 4, 1), (4, 4, 2), (2, 4, 2), (2, 2, 2), (1, 1, 1)]
WAVES, STEPS, FRAGMENTS = 8, 4, 48


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("pipe")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


class Early(Exception):
    pass


def _walk(plan, nt, jt, wj, n, wave, tail_requests=False, dead_loads=True, drain=True):
    """One wave over n slabs.  tail_requests: the tail fetches and waits like any slab; dead_loads: weight loads that bring nothing
    that is multiplied are issued."""
    wd, one = plan.depth(nt), bool(plan.one_ahead(nt, wj))
    frags = sum(plan.fetched(jt, f) for f in range(wave, FRAGMENTS, WAVES))
    queue, landed, last, tail_from = [], {}, n - 1, n // wd * wd

    def fetch(i, buf):
        landed.pop(buf, None)
        queue.extend([("piece", min(i, last), buf)] * frags)

    def weights(i, count=nt):
        if dead_loads or i <= last:
            queue.extend([("weight", i)] * count)

    def wait(count):
        while len(queue) > count:
            r = queue.pop(0)
            if r[0] == "piece" and r not in queue:
                landed[r[2]] = r[1]

    fetch(0, 0)
    weights(0, nt * STEPS)
    if not one:
        fetch(1, 1)
    for w in range(1, wd):
        weights(w, nt * STEPS)
    wait(plan.wait_first(nt, jt, wj))
    buf = 0
    for i in range(n):
        tail = i >= tail_from
        if frags and landed.get(buf) != i:
            raise Early((nt, jt, wj, n, wave, i))
        requests = not tail or tail_requests
        if not one and requests:
            fetch(i + 2, (buf + 2) % 3)
        for s in range(STEPS):
            if requests:
                weights(i + wd)
            if one and s == 0 and requests:
                fetch(i + 1, buf ^ 1)
        wait(plan.wait_slab(nt, jt, wj) if requests else 0)
        buf = buf ^ 1 if one else (buf + 1) % 3
    if drain:
        wait(0)
    if any(r[0] == "piece" for r in queue):
        raise Early((nt, jt, wj, n, wave, "end"))


@pytest.mark.parametrize("nt,jt,wj", INSTANCES)
def test_slabs_have_landed_when_they_are_read(plan, nt, jt, wj):
    # loads without a use: the kernel gives every load of the loop one where the waits count them (more than one slab ahead)
    for dead_loads in ([True] if plan.depth(nt) > 1 else [True, False]):
        for n in range(1, 26):
            for wave in range(WAVES):
                _walk(plan, nt, jt, wj, n, wave, dead_loads=dead_loads)


def test_the_model_sees_a_tail_that_waits_by_count(plan):
    """A tail that requests like any slab, without the weight loads that nothing uses, reads pieces too early."""
    with pytest.raises(Early):
        for n in range(1, 26):
            _walk(plan, 1, 1, 1, n, 0, tail_requests=True, dead_loads=False)
    with pytest.raises(Early):
        _walk(plan, 2, 4, 2, 8, 0, drain=False)   # pieces past the end still on their way
