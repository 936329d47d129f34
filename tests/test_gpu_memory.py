"""What a context asks of the device's memory (needs an MI355X): hipMalloc
goes through a small host library that counts the library's allocations and
refuses those beyond a set number of bytes, as a card that is nearly full
would.  A child process each, so that the library binds to it."""
import json
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
#include <stdint.h>
#define CAP (1 << 17)
typedef int (*malloc_fn)(void**, size_t);
typedef int (*free_fn)(void*);
static malloc_fn real_malloc;
static free_fn real_free;
static struct { uintptr_t p; size_t n; } tab[CAP];
static long long live, peak, calls, limit = -1;
void shim_init(void* m, void* f) { real_malloc = (malloc_fn)m; real_free = (free_fn)f; }
/* further bytes allowed from now on; < 0: no limit.  Restarts the peak and the count. */
void shim_limit(long long more) { limit = more < 0 ? -1 : live + more; peak = live; calls = 0; }
long long shim_live(void) { return live; }
long long shim_peak(void) { return peak; }
long long shim_calls(void) { return calls; }
static unsigned slot(uintptr_t p) { return (unsigned)((p >> 12) * 2654435761u) % CAP; }
int hipMalloc(void** p, size_t n) {
    ++calls;
    if (!real_malloc) return 1;
    /* the runtime's own refusal, with the error state that it leaves */
    if (limit >= 0 && live + (long long)n > limit) return real_malloc(p, (size_t)1 << 50);
    int e = real_malloc(p, n);
    if (e) return e;
    unsigned i = slot((uintptr_t)*p);
    while (tab[i].p > 1) i = (i + 1) % CAP;
    tab[i].p = (uintptr_t)*p;
    tab[i].n = n;
    live += (long long)n;
    if (live > peak) peak = live;
    return 0;
}
int hipFree(void* p) {
    if (!real_free) return 1;
    unsigned i = slot((uintptr_t)p);
    while (tab[i].p && tab[i].p != (uintptr_t)p) i = (i + 1) % CAP;
    if (tab[i].p) { live -= (long long)tab[i].n; tab[i].p = 1; }
    return real_free(p);
}
"""

PRELUDE = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import torch
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
hip = ctypes.CDLL(path)
for f in ("shim_live", "shim_peak", "shim_calls"):
    getattr(shim, f).restype = ctypes.c_longlong
shim.shim_limit.argtypes = [ctypes.c_longlong]
shim.shim_init.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
shim.shim_init(ctypes.cast(hip.hipMalloc, ctypes.c_void_p), ctypes.cast(hip.hipFree, ctypes.c_void_p))
from paper_2411_15897_amd import ElasticHelmholtz
from paper_2411_15897_amd.solver import EhelmError

def medium(n, seed=3):
    rng = np.random.default_rng(seed)
    vp = rng.uniform(2.0, 3.5, tuple(reversed(n)))
    return vp, 0.5 * vp, rng.uniform(1.0, 2.0, vp.shape)

def context(n, more=-1, **kw):
    # a context under `more` further bytes, and (live, peak, calls) of its creation
    live = shim.shim_live()
    shim.shim_limit(more)
    try:
        s = ElasticHelmholtz(n, (1.0,) * len(n), *medium(n), 0.7, levels=1, alpha=0.3, abc_width=4, mg_precision=64, **kw)
    finally:
        calls, peak = shim.shim_calls(), shim.shim_peak()
        shim.shim_limit(-1)
    return s, (shim.shim_live() - live, peak - live, calls)

def blocks(s, nrhs=2):
    # the direct solves of every block for fixed right-hand sides
    out = []
    for b in range(s.dim + 1):
        N = int(np.prod(s.block_dims(b, 0)))
        g = torch.Generator("cuda").manual_seed(b)
        out.append(s.block_cycle(b, torch.randn(nrhs, N, dtype=torch.complex128, device="cuda", generator=g)))
    return out

def worst(xs, ys):
    return max(float((x - y).norm() / y.norm()) for x, y in zip(xs, ys))

def done(**kw):
    print("RESULT " + json.dumps(kw), flush=True)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.c").write_text(SHIM)
    so = str(d / "libshim.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, str(d / "shim.c")], check=True)

    def child(code):
        res = subprocess.run([sys.executable, "-c", PRELUDE + code, so], cwd=ROOT, capture_output=True, text=True,
                             timeout=100)
        assert res.returncode == 0, res.stdout + res.stderr
        print(res.stderr, file=sys.stderr, flush=True)
        return json.loads(next(l for l in res.stdout.splitlines() if l.startswith("RESULT "))[7:])

    return child


def test_dense_inverses_one_after_the_other(run):
    """Every block's matrix side by side needs more than one block's with
    the right half of Gauss-Jordan on [X | I] at the end, the least this
    solver has asked for: with that much, the same inverses, bitwise."""
    r = run("""
s, (steady, peak, _) = context((40, 32), coarse_solver="dense")
N = max(int(np.prod(s.block_dims(b, 0))) for b in range(3))
ref = blocks(s)
more = steady + 2 * 16 * N * N + (1 << 20)
t, (steady2, peak2, _) = context((40, 32), more, coarse_solver="dense")
done(more=more, steady=steady, peak=peak, steady2=steady2, peak2=peak2, diff=worst(blocks(t), ref))
""")
    assert r["peak"] > r["more"] >= r["peak2"]
    assert r["steady"] == r["steady2"] and r["diff"] == 0.0


def test_eliminations_that_fit_only_in_the_smaller_order(run):
    """Removing every other group stores five matrices per group here, the
    groups one after the other three, and needs every group's blocks at
    once.  Whatever room there is beyond the smaller factors of all blocks
    (and a tenth), the context is made -- also where the first blocks' larger
    factors fit and would leave too little for the last one's smaller ones --
    and its solves stay as accurate."""
    r = run("""
n = (15, 6, 120)                                   # groups: planes of 90 to 105 points
s, (steady, peak, _) = context(n, coarse_solver="bt")
ref = blocks(s)
dims = [tuple(int(v) for v in s.block_dims(b, 0)) for b in range(4)]
s.close()
one = sum(16 * 3 * (m[0] * m[1]) ** 2 * m[2] for m in dims)
out = []
for more in (1.1, 1.2, 1.25, 1.33, 1.4, 1.5, 2.0):
    try:
        t, (steady2, peak2, _) = context(n, int(more * one), coarse_solver="bt")
    except EhelmError as e:
        out.append((more, str(e), 0, 1.0))
        continue
    out.append((more, "", peak2, worst(blocks(t), ref)))
    t.close()
done(one=one, steady=steady, peak=peak, out=out)
""")
    print(r)
    assert r["peak"] > 2.0 * r["one"]
    for more, err, peak, diff in r["out"]:
        assert not err and peak <= more * r["one"] and diff <= 1e-11, more


def test_refused_context_leaves_others_alone(run):
    """A creation refused for memory is EH_ERR_OOM, and neither a context
    that exists nor the next creation meets its error."""
    r = run("""
s, (steady, _, _) = context((40, 32), coarse_solver="dense")
ref = blocks(s)
status = None
try:
    context((40, 32), steady // 2, coarse_solver="dense")
except EhelmError as e:
    status = e.status
after = worst(blocks(s), ref)
try:
    context((40, 32), 1000, coarse_solver="bt")
except EhelmError:
    pass
t, _ = context((40, 32), coarse_solver="dense")
done(status=status, after=after, new=worst(blocks(t), ref), live=shim.shim_live())
""")
    assert r["status"] == -3 and r["after"] == 0.0 and r["new"] == 0.0


def test_long_chain_in_few_allocations(run):
    """6000 groups of 4 points: their matrices do not take an allocation
    each (three per group and more)."""
    r = run("""
s, (steady, peak, calls) = context((6000, 4), coarse_solver="bt")
done(calls=calls, steady=steady, peak=peak)
""")
    print(r)
    assert r["calls"] < 1000
