"""Reads of a code (export, export_nodes, pack) and the library's waits: a
child process puts its own hipStreamSynchronize and hipEventSynchronize before
the runtime's, which count the waits and can report one of them as failed
(after it has really ended, so nothing is left in flight)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r'''
#define _GNU_SOURCE
#include <dlfcn.h>
int waits_seen, waits_fail_at;   /* fail_at: number of the wait to report as failed, 0: none */
static int through(const char* name, void* arg) {
  static void* lib;
  if (!lib) lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  int (*fn)(void*) = lib ? (int (*)(void*))dlsym(lib, name) : 0;
  if (!fn) return 999;
  const int rc = fn(arg);
  return ++waits_seen == waits_fail_at ? 999 : rc;
}
int hipStreamSynchronize(void* s) { return through("hipStreamSynchronize", s); }
int hipEventSynchronize(void* e) { return through("hipEventSynchronize", e); }
'''

COMMON = r'''
import ctypes, sys
root, shim = sys.argv[1:3]
sys.path.insert(0, root)
shim = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)      # before the library is loaded
seen, fail_at = ctypes.c_int.in_dll(shim, "waits_seen"), ctypes.c_int.in_dll(shim, "waits_fail_at")
import numpy as np, torch
from paper_2605_09190_amd import aqmp as A
from workloads import piecewise_image
dic = A.Dictionary(8, 32)
def code_of(h, w, **kw):
    img = torch.from_numpy(piecewise_image(h, w, seed=51)).float().cuda()
    prm = dict(tol=1e-4, max_atoms=24, n_min=8, n_max=32, **kw)
    return img, A.Code(dic, [img], [prm], [(0, 0)], precision=A.PREC_BF16, schedule=A.SCHED_BATCHED)
'''

FAILING = COMMON + r'''
def buffers(n, na):
    return [np.full(n, 0x5a, np.uint8) for n in (n * A.LEAF_DTYPE.itemsize, 4 * na, 8 * na)]
def call(fn, code, b, n, na):
    return fn(code.h, *[x.ctypes.data for x in b], n, na)
for h, w in ((64, 64), (1024, 1024)):
    img, code = code_of(h, w)
    for fn, all_nodes in ((A.lib.aqmp_code_export, False), (A.lib.aqmp_code_export_nodes, True)):
        if all_nodes:
            n, na = int(sum(code.stats()["nodes"])), int(code.stats()["iters_executed"])
        else:
            n, na = code.sizes()
        code.reencode([img])
        want = buffers(n, na)
        assert call(fn, code, want, n, na) == 0
        clean, failed = buffers(n, na), 0
        for k in range(1, 64):
            code.reencode([img])
            torch.cuda.synchronize()
            got = buffers(n, na)
            seen.value, fail_at.value = 0, k
            rc = call(fn, code, got, n, na)
            fail_at.value = 0
            assert (rc == 0) == (seen.value < k), (rc, seen.value, k)
            if rc == 0:
                break
            failed += 1
            assert all((a == b).all() for a, b in zip(got, clean)), ("buffers touched", h, all_nodes, k)
            assert call(fn, code, got, n, na) == 0     # and the next call is whole again
            assert all((a == b).all() for a, b in zip(got, want)), (h, all_nodes, k)
        assert rc == 0 and all((a == b).all() for a, b in zip(got, want))
        print("ok", h, w, all_nodes, "bytes", sum(x.size for x in want), "failed waits", failed, flush=True)
        assert failed >= 2
    code.free()
dic.free()
print("done", flush=True)
'''

AGAIN = COMMON + r'''
def waits(f):
    seen.value = 0
    r = f()
    return seen.value, r
def same(a, b):
    return all(x.tobytes() == y.tobytes() for x, y in ((a.leaves, b.leaves), (a.atom_idx, b.atom_idx), (a.coef, b.coef)))
for h, w in ((96, 64), (512, 512)):
    img, code = code_of(h, w)
    leaves = code.export()
    assert leaves.leaves["atom_off"][-1] + leaves.leaves["n_atoms"][-1] == len(leaves.coef)
    n0, nodes = waits(code.export_nodes)
    packed = code.pack([0], level=-1)
    print("nodes", len(nodes.leaves), "leaves", len(leaves.leaves), "waits of the first reading of all", n0, flush=True)
    assert len(nodes.leaves) > len(leaves.leaves) and n0 >= 1     # a stale count would hide the others
    reads = [code.export, code.export_nodes, code.export, lambda: code.pack([0], level=-1), code.export, code.sizes, code.stats]
    for start in (None, code.export_nodes, code.export):
        if start:                                                  # another encode, read in another order
            code.reencode([img])
            start()
            code.export_nodes()
        for k, f in enumerate(reads):
            n, r = waits(f)
            assert n == 0, (h, k, n)
            if isinstance(r, A.Export):
                assert same(r, nodes if f == code.export_nodes else leaves), (h, k)
            elif isinstance(r, bytes):
                assert r == packed
    code.free()
dic.free()
print("done", flush=True)
'''


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = tmp_path_factory.mktemp("shim")
    src, lib = d / "waits.c", d / "libwaits.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    return str(lib)


def _child(script, shim):
    out = subprocess.run([sys.executable, "-u", "-c", script, ROOT, shim], capture_output=True, text=True, timeout=100)
    print(out.stdout, out.stderr[-2000:], flush=True)
    assert out.returncode == 0 and out.stdout.strip().endswith("done"), out.stderr[-2000:]


def test_failed_wait_leaves_buffers_untouched(shim):
    """Every wait of an export reported as failed in turn: the caller's buffers
    keep their bytes, of a result that the gather writes to host memory and of
    one that is copied (several MB)."""
    _child(FAILING, shim)


def test_nodes_serve_every_later_read(shim):
    """Once all nodes of an encode are read, leaves, nodes, streams, sizes and
    statistics of it need the device no more, in any order, and are the same."""
    _child(AGAIN, shim)
