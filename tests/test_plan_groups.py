"""Plans of the group path (host side, no GPU): a work item holds a fair share of a group's index entries
whatever the k-mer length, so that plan tables, launches and host time stay in proportion; and a plan takes
the path where the measurements say that it pays."""
import ctypes as C
import os
import subprocess
import sys

import pytest

import paper_2510_23679_amd as pdp
from paper_2510_23679_amd import binding as B


def _dicts(n, genes, per, k, alphabet):
    out, base = [], 256
    for _ in range(n):
        arena, _ = pdp.dict_size(genes, genes * per, k, alphabet)
        d = B.pdp_dict()
        B.check(pdp.lib().pdp_dict_bind(base, arena, genes, genes * per, k, B.alphabet_id(alphabet), 0, C.byref(d)), "bind")
        base += (arena + 4095) // 4096 * 4096
        out.append(d)
    return out


def _items(dicts, **prm):
    n = len(dicts)
    prm = pdp.params(**prm)
    tasks = (B.pdp_task * (n * (n - 1) // 2))()
    for t, (i, j) in zip(tasks, [(i, j) for i in range(n) for j in range(i)]):
        t.a, t.b, t.flags = C.pointer(dicts[i]), C.pointer(dicts[j]), pdp.PDP_TASK_BBH
    h, info = B.vp(), B.pdp_plan_info()
    B.check(pdp.lib().pdp_plan_create(tasks, len(tasks), C.byref(prm), C.byref(h)), "plan")
    B.check(pdp.lib().pdp_plan_info_get(h, C.byref(info)), "info")
    pdp.lib().pdp_plan_destroy(h)
    return info.join_groups


@pytest.mark.parametrize("alphabet,k", [("aa", k) for k in range(6, 13)] + [("nt", k) for k in (15, 17, 21, 23, 24, 25, 26, 31)])
@pytest.mark.parametrize("n,genes", [(16, 200), (12, 1270), (10, 3000), (40, 4000)])
def test_items_are_in_proportion_to_the_entries(n, genes, alphabet, k):
    per = 300 if alphabet == "aa" else 900
    buckets = 160000 if alphabet == "aa" else 262144
    entries = n * (genes * per + 1)
    # about 1536 entries an item (fewer in small plans: at least 256), half of that for a narrow
    # identity, and whole buckets: an item's share is rounded down by at most half
    assert _items(_dicts(n, genes, per, k, alphabet)) <= min(buckets, 4 * max(entries // 1536, min(1024, entries // 256)) + 8)


@pytest.mark.parametrize("n,genes,filters,grouped", [
    (9, 300, False, True), (7, 300, True, True), (6, 300, False, False),       # launches either way
    (7, 1000, False, False), (10, 1000, False, False), (12, 1000, False, True),
    (7, 1000, True, False), (10, 1000, True, True),
    (8, 2000, False, False), (10, 2000, False, True), (6, 2000, True, False), (8, 2000, True, True),
    (6, 4000, False, False), (8, 4000, False, True), (5, 4000, True, False), (7, 4000, True, True),
    (50, 4000, False, True)])
def test_a_group_is_taken_where_it_pays(n, genes, filters, grouped):
    prm = {"theta": (1, 2), "tau": (1, 6)} if filters else {}
    dicts = _dicts(n, genes, 340, 6, "aa")
    assert (_items(dicts, **prm) != _items(dicts, persistent=True, **prm)) == grouped


def test_a_plan_past_the_host_memory_is_an_error():
    # 150,000 tasks of two genomes of 3000 genes: some 2 GB of join items, in a process that may have 1 GB
    code = """
import ctypes as C, resource, sys
sys.path.insert(0, %r)
import test_plan_groups as T
import paper_2510_23679_amd as pdp
from paper_2510_23679_amd import binding as B
a, b = T._dicts(2, 3000, 300, 6, "aa")
tasks = (B.pdp_task * 150000)()
for t in tasks:
    t.a, t.b, t.flags = C.pointer(a), C.pointer(b), pdp.PDP_TASK_AB
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (1 << 30),) * 2)
h = B.vp()
rc = pdp.lib().pdp_plan_create(tasks, len(tasks), None, C.byref(h))
assert rc == pdp.PDP_E_INVAL and not h.value, rc
print(pdp.lib().pdp_last_error().decode())
""" % os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), timeout=120)
    assert r.returncode == 0 and "out of host memory" in r.stdout, (r.returncode, r.stderr[-500:])
