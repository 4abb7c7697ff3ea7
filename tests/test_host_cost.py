"""Small submissions are bound by the host: a call's planning and launch
building may not take more heap allocations than before.  Counted, as times
on a shared machine are not reproducible: a preloaded operator new counts the
allocations of gdy_plan and gdy_dispatch_map (plan, launches and launch block,
as gdy_execute makes them) on a host-only context."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TABLE = os.path.join(ROOT, "paper_2409_02227_amd", "tables", "gfx950.table")
COUNTER = r"""
#include <cstdlib>
#include <new>
static long n;
extern "C" long counted_news() { return n; }
void* operator new(std::size_t s) { ++n; void* p = std::malloc(s ? s : 1); if (!p) std::abort(); return p; }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""


def counts():
    """Allocations of one call of each, per submission; runs in the preloaded process."""
    from paper_2409_02227_amd import gdy
    from tests.test_dispatch_map import _desc
    news = ctypes.CDLL(None).counted_news
    news.restype = ctypes.c_long
    ctx = gdy.Context(-1, table=TABLE)
    for sizes, dtype in (([(256, 256, 256)] * 2, 1), ([(64, 4096, 1024)] * 4, 2)):
        descs = [_desc(m, n, k, dtype, j) for j, (m, n, k) in enumerate(sizes)]
        arr, n = (gdy.GemmDesc * len(descs))(*descs), len(descs)
        plan, grid = gdy.Plan(), ctypes.c_int32()
        wg, items = (ctypes.c_int32 * 1)(), (ctypes.c_int64 * n)()
        a = news()
        assert ctx.lib.gdy_plan(ctx.h, arr, n, gdy.SELECTOR, 0, ctypes.byref(plan)) == 0
        b = news()
        assert ctx.lib.gdy_dispatch_map(ctx.h, arr, n, gdy.SELECTOR, 0, 0, 0, ctypes.byref(grid), wg, wg, wg, items) == 0
        assert plan.n_dispatches == 1
        print(b - a, news() - b)


def test_allocations_of_a_small_submission(tmp_path):
    if not shutil.which("g++") or not os.path.exists(TABLE):
        pytest.skip("no host compiler or table")
    src, lib = tmp_path / "news.cpp", tmp_path / "libnews.so"
    src.write_text(COUNTER)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    env = dict(os.environ, LD_PRELOAD=":".join(filter(None, [str(lib), os.environ.get("LD_PRELOAD")])), PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", "from tests.test_host_cost import counts; counts()"], env=env, cwd=ROOT,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    got = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    # no more than the selector's lists, the split offsets and (four members) XCD placement took before launches could
    # be joint; the joint launches came with (31, 47) and (36, 76)
    assert len(got) == 2
    for (plan, launch), (most_plan, most_launch) in zip(got, ((30, 36), (35, 58))):
        assert plan <= most_plan and launch <= most_launch, got
