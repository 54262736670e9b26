"""C-ABI surface and host-side planning of top-k (no GPU, no kernel launch)."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

from paper_2605_28213_amd import build as gl_build
from paper_2605_28213_amd import gemm, topk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def _built():
    gl_build.build()


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "topk_lineage.h")).read()
    body = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(topk_[a-z_0-9]+)\s*\(", body))
    assert {"topk_run", "topk_query", "topk_variant_name"} <= names
    L = ctypes.CDLL(gemm.LIB_PATH)
    for n in sorted(names):
        assert hasattr(L, n), f"{n} declared in the header but not exported"
    assert topk.topk_variant_count() == topk.TOPK_VARIANT_COUNT == 3
    assert [topk.topk_variant_name(v) for v in range(3)] == ["T0_selection", "T1_radix_select", "T2_resident_coarse_refine"]
    for name, bit in topk.COND_BITS.items():
        assert topk.topk_cond_name(bit) == name
    assert topk.topk_variant_intent(1) == "radix_select" and "coarse + refine" in topk.topk_variant_intent(2)


def test_struct_layout_matches_the_header_as_plain_c(tmp_path):
    fields_d = [f[0] for f in topk.topk_desc_t._fields_]
    fields_q = [f[0] for f in topk.topk_query_t._fields_]
    prog = ['#include <stdio.h>', '#include <stddef.h>', '#include "topk_lineage.h"', 'int main(void){',
            'printf("%zu %zu\\n", sizeof(topk_desc_t), sizeof(topk_query_t));']
    prog += [f'printf("%zu\\n", offsetof(topk_desc_t, {f}));' for f in fields_d]
    prog += [f'printf("%zu\\n", offsetof(topk_query_t, {f}));' for f in fields_q]
    prog += ['return 0;}']
    src = tmp_path / "layout.c"
    src.write_text("\n".join(prog))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(out[0]), int(out[1])] == [ctypes.sizeof(topk.topk_desc_t), ctypes.sizeof(topk.topk_query_t)]
    want = [getattr(topk.topk_desc_t, f).offset for f in fields_d] + [getattr(topk.topk_query_t, f).offset for f in fields_q]
    assert [int(x) for x in out[2:]] == want


@pytest.mark.parametrize("n", [4097, 8192, 16384, 100000])
@pytest.mark.parametrize("batch", [(1 << 22) - 1, 1 << 22, (1 << 24) - 1])
def test_rows_of_the_streaming_state_fit_a_launch(n, batch):
    """A launch holds fewer than 2^32 threads: long rows in such numbers that 1024 lanes each exceed that run on 256."""
    q = topk.topk_query(1, topk.make_desc(batch, n, 7))
    assert q.status == gemm.GEMM_OK and q.grid == batch and q.grid * q.threads < 1 << 32


def test_which_long_rows_go_to_which_form():
    """256 lanes share the CUs better where there are many rows; the filter's two reads pay on long rows only."""
    of = lambda b, n, k: topk.topk_query(1, topk.make_desc(b, n, k))
    for b, n, k, threads, passes in [(1, 4096, 9, 256, 5), (512, 4097, 9, 1024, 5), (513, 4097, 9, 256, 5), (513, 5000, 2100, 256, 5), (513, 5001, 9, 1024, 5),
                                     (8, 12288, 9, 1024, 5), (8, 12289, 2048, 1024, 2), (8, 12289, 2049, 1024, 5), (4096, 20000, 1, 1024, 2)]:
        q = of(b, n, k)
        assert (q.threads, q.passes, "filter" in q.path) == (threads, passes, passes == 2), (b, n, k, q)


def test_plans_and_refusals():
    d = topk.make_desc(64, 4096, 512)
    q0, q1, q2 = (topk.topk_query(v, d) for v in range(3))
    assert all(q.status == gemm.GEMM_OK and q.grid == 64 for q in (q0, q1, q2))
    assert (q0.threads, q0.passes) == (256, 512) and (q1.threads, q1.passes) == (256, 5) and (q2.threads, q2.passes) == (1024, 4)
    assert "11+11+10" in q2.path and "4 keys/lane" in q2.path
    assert "16 keys/lane" in topk.topk_query(2, topk.make_desc(2, 4097, 5, ld=4100)).path
    big = topk.make_desc(2, 70001, 300)
    assert topk.Query.names(topk.topk_query(0, big).violated) == ["ROW_IN_LDS"]
    assert topk.topk_query(1, big).status == gemm.GEMM_OK
    q = topk.topk_query(2, big)
    assert q.status == gemm.GEMM_ERR_PRECONDITION and "ROW_IN_REGISTERS" in topk.Query.names(q.violated)
    assert topk.Query.names(topk.topk_query(2, topk.make_desc(2, 1000, 5, ld=1001)).violated) == ["ALIGN16"]
    assert topk.Query.names(topk.topk_query(2, d, 256 + 4).violated) == ["ALIGN16"]
    assert topk.topk_run(2, d, 256 + 4, 256, 256) == gemm.GEMM_ERR_PRECONDITION


def test_argument_validation():
    def st(variant=1, **kw):
        a = dict(batch=2, n=100, k=10)
        a.update(kw)
        return topk.topk_query(variant, topk.make_desc(a["batch"], a["n"], a["k"], ld=a.get("ld", 0), flags=a.get("flags", 0))).status
    assert st() == gemm.GEMM_OK
    assert st(variant=3) == gemm.GEMM_ERR_BAD_VARIANT
    for bad in (dict(batch=-1), dict(n=-1), dict(k=-1), dict(k=101), dict(ld=99), dict(flags=1), dict(n=1 << 31, k=1)):
        assert st(**bad) == gemm.GEMM_ERR_BAD_ARG, bad
    assert st(k=0) == gemm.GEMM_OK and st(batch=0) == gemm.GEMM_OK and st(n=0, k=0) == gemm.GEMM_OK
    assert topk.topk_query(1, topk.make_desc(2, 100, 0)).grid == 0
    assert topk.topk_run(1, topk.make_desc(2, 100, 10), None, 256, 256) == gemm.GEMM_ERR_BAD_ARG


LAUNCHES = r'''
#include <stdint.h>
#include <stddef.h>
typedef struct { uint32_t x, y, z; } dim3_t;
static dim3_t g, b; static size_t shm; static void* st; static int error;
int launches, fail_at; uint32_t grids[8]; const void* kernels[8]; void* streams[8];
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t s, void* stream) { g = grid; b = block; shm = s; st = stream; return 0; }
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* s, void** stream) { *grid = g; *block = b; *s = shm; *stream = st; return 0; }
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t s, void* stream)
{
    (void)block; (void)args; (void)s;
    kernels[launches] = f; grids[launches] = grid.x; streams[launches] = stream;
    if (++launches != fail_at) return 0;
    error = 1;
    return 1;
}
int hipGetLastError(void) { const int e = error; error = 0; return e; }
'''
CALLER = r'''
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)        # found before the runtime's own launch calls
lib = ctypes.CDLL(sys.argv[2])
class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("batch", "n", "k", "ld")] + [("stream", ctypes.c_void_p), ("flags", ctypes.c_uint32), ("reserved", ctypes.c_uint32)]
lib.topk_run.argtypes = [ctypes.c_int, ctypes.POINTER(Desc), ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
count, fail_at = ctypes.c_int.in_dll(stub, "launches"), ctypes.c_int.in_dll(stub, "fail_at")
for fail in (0, 1, 2, 3):
    count.value, fail_at.value = 0, fail
    rc = lib.topk_run(1, ctypes.byref(Desc(3, 20000, 9, 20000, 0x77, 0, 0)), 4096, 1 << 20, 2 << 20)
    n = count.value
    print(fail, rc, n, *(ctypes.c_uint32 * 8).in_dll(stub, "grids")[:n], len(set((ctypes.c_void_p * 8).in_dll(stub, "kernels")[:n])),
          set((ctypes.c_void_p * 8).in_dll(stub, "streams")[:n]) == {0x77})
'''


def test_a_launch_that_fails_leaves_no_slot_of_cut_rows_claimed(tmp_path):
    """Rows in parts take two launches.  The second is not made where the first fails, and where it fails itself a third kernel
    gives the slots back, one workgroup per row.  The runtime's launch calls are replaced in a process of its own: no GPU."""
    (tmp_path / "launches.c").write_text(LAUNCHES)
    stub = tmp_path / "liblaunches.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-Wall", "-Werror", str(tmp_path / "launches.c"), "-o", str(stub)], check=True)
    r = subprocess.run([sys.executable, "-c", CALLER, str(stub), gemm.LIB_PATH], check=True, capture_output=True, text=True)
    ok, bad = gemm.GEMM_OK, gemm.GEMM_ERR_LAUNCH
    assert r.stdout.split("\n")[:4] == [f"0 {ok} 2 15 3 2 True", f"1 {bad} 1 15 1 True", f"2 {bad} 3 15 3 3 3 True", f"3 {ok} 2 15 3 2 True"]


def test_reported_lds_is_what_the_kernels_were_built_with():
    """Every form's lds_bytes against the compiler's record of its kernel; the larger of two where a call launches two."""
    kernels = gl_build.resources()["kernels"]
    for v, b, n, k, names in [(0, 2, 1000, 9, ["topk_selection"]), (1, 2, 1000, 9, ["topk_radix<256, 1, false"]), (1, 40, 12000, 9, ["topk_long"]),
                              (1, 40, 70000, 9, ["topk_long"]), (1, 2, 70000, 9, ["topk_parts", "topk_merge"]), (2, 2, 4096, 9, ["topk_radix<1024, 4, true"]),
                              (2, 2, 5000, 9, ["topk_radix<1024, 16, true"])]:
        q = topk.topk_query(v, topk.make_desc(b, n, k))
        built = [f["lds_bytes"] for name, f in kernels.items() if any(x in name for x in names)]
        assert q.status == gemm.GEMM_OK and len(built) == len(names) and q.lds_bytes == max(built), (v, b, n, k, q, built)
