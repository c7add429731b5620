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
