"""Which kernel values a sweep reads, from the arguments of its launches: on the host, with a HIP runtime that runs no kernels
(fake_hip.c)."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2006_10350_amd", "libknm.so")

# the sums over a fit's kept values by their first arguments: values, points of the two sides (KeptArgs); how many sums over a product's slabs
RECORD = """
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
enum { kFunctions = 4096, kLaunches = 4096 };
static const void *functions[kFunctions];
static int known, reads;
static int64_t sizes[kLaunches][2];
static const void *values[kLaunches];
static const void *slab_sums[64];
static int slab_kinds, slabs;
int kept_reads(void) { return reads; }
int kept_slabs(void) { return slabs; }
static const void *slab;
const void *kept_slab(void) { return slab; } /* values of the last sum over a slab */
int64_t kept_size(int launch, int side) { return sizes[launch][side]; }
int kept_blocks(void) /* different blocks of values */
{
    int count = 0;
    for (int i = 0; i < reads; ++i) {
        int seen = 0;
        for (int j = 0; j < i; ++j) seen |= values[i] == values[j];
        count += !seen;
    }
    return count;
}
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *size)
{
    (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
    if (strstr(name, "kept_over_") && known < kFunctions) functions[known++] = host;
    if (strstr(name, "kept_rows_kernel") && slab_kinds < 64) slab_sums[slab_kinds++] = host;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)grid; (void)block; (void)lds; (void)stream;
    for (int i = 0; i < slab_kinds; ++i)
        if (slab_sums[i] == f) {
            ++slabs;
            memcpy(&slab, args[0], 8);
        }
    for (int i = 0; i < known; ++i)
        if (functions[i] == f && reads < kLaunches) {
            memcpy(&values[reads], args[0], 8);
            memcpy(sizes[reads++], (char *)args[0] + 8, 16);
        }
    return 0;
}
"""

HEAD = """
import ctypes as c
rec, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
lib = c.CDLL({lib!r})
P, L, I, F, D, Z = c.c_void_p, c.c_int64, c.c_int, c.c_float, c.c_double, c.c_size_t
rec.kept_size.restype = c.c_int64
rec.kept_slab.restype = P
hip.fake_set_budget.argtypes = hip.fake_set_total.argtypes = [Z]
hip.fake_inside.argtypes = [P, Z]
hip.fake_live.restype = hip.fake_peak.restype = lib.knm_workspace_held.restype = Z
lib.knm_workspace_held.argtypes = lib.knm_release_workspace.argtypes = lib.knm_destroy.argtypes = [P]
lib.logfalkon_fit.argtypes = [P, P, L, I, L, P, P, L, L, P, F, P, P, I, D, P, P]
lib.falkon_fit.argtypes = [P, P, L, I, L, P, I, P, L, L, F, D, D, I, P, P]
lib.knm_prod.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P, P]
ctx = P()
assert lib.knm_create(c.byref(ctx), 0, None) == 0
created = hip.fake_live()
x, cen, y, yc, alpha, v, u = (P(0x7f0000000000 + (i << 40)) for i in range(7))  # never read: kernels do not run


def prod(n, M, d, t):
    return lib.knm_prod(ctx, x, n, d, d, cen, M, d, 1.0, v, t, None, u)


def fit(n, d, M, t):
    return lib.falkon_fit(ctx, x, n, d, d, y, t, cen, M, d, 1.0, 1e-6, 1e-6, 3, alpha, None)
"""


def _run(shims, body):
    """In a process of its own: the fake runtime must come before the real one."""
    r = subprocess.run([sys.executable, "-c", HEAD.format(shims=shims, lib=LIB) + textwrap.dedent(body)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.fixture(scope="module")
def shims(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("hip")
    (tmp / "record.c").write_text(RECORD)
    out = []
    for name, src in (("record", str(tmp / "record.c")), ("fakehip", os.path.join(HERE, "fake_hip.c"))):
        out.append(str(tmp / f"lib{name}.so"))
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", f"-Wl,-soname,lib{name}.so", "-o", out[-1], src], check=True)
    return out


# Centres of their own, every tenth row of X, the first rows of X, X among the centres, X itself: the values are those of n x M pairs (M x n
# formed by columns), and no sweep of k(C, C) takes them for its own unless the two sets are one.
@pytest.mark.parametrize("n,M,step,shared", [(3000, 300, 1, False), (3000, 300, 10, True), (3000, 300, 1, True), (300, 1000, 1, True),
                                             (3000, 3000, 2, True), (400, 400, 1, True)])
@pytest.mark.parametrize("cross", [0, 1])
def test_logistic_fit_reads_the_values_of_its_pair(shims, n, M, step, shared, cross):
    d = 500
    _run(shims, f"""
        assert lib.knm_set_cross_term(ctx, {cross}) == 0
        if {shared}:
            cen = x
        lambdas, iters = (c.c_double * 2)(1e-2, 1e-3), (c.c_int * 2)(4, 5)
        st = lib.logfalkon_fit(ctx, x, {n}, {d}, {d}, y, cen, {M}, {step * d}, yc, 1.0, lambdas, iters, 2, 1e-6, alpha, None)
        assert st == 0, st
        reads = [(rec.kept_size(i, 0), rec.kept_size(i, 1)) for i in range(rec.kept_reads())]
        print(len(reads), set(reads))
        assert set(reads) in ({{({n}, {M})}}, {{({M}, {n})}})
        assert rec.kept_blocks() == 1
        # in each of two Newton steps a sweep by rows, one by columns and two for each iteration; and one of k(C, C)
        own = {shared} and {n} == {M} and {step} == 1
        assert len(reads) == 2 * 2 + 2 * 9 + (2 if own else 0)
        """)


# slabs of 4 GiB of values: one, three, many of the fewest rows (1024), fewer rows than that (two sweeps); few features, many columns and
# the other arithmetic (two sweeps)
@pytest.mark.parametrize("n,M,d,t,cross,slabs", [(40000, 20000, 784, 10, 1, 1), (40000, 50000, 784, 1, 1, 3), (20480, 1 << 20, 300, 1, 1, 20),
                                                 (20480, (1 << 20) + 128, 300, 1, 1, 0), (1000, 3 << 20, 300, 1, 1, 0), (256, 3 << 20, 300, 1, 1, 1),
                                                 (40000, 20000, 200, 1, 1, 0), (40000, 20000, 784, 13, 1, 0), (40000, 20000, 784, 1, 0, 0)])
def test_slabs_of_a_product(shims, n, M, d, t, cross, slabs):
    _run(shims, f"""
        assert lib.knm_set_cross_term(ctx, {cross}) == 0
        for k in (1, 2):
            assert prod({n}, {M}, {d}, {t}) == 0
            assert rec.kept_slabs() == k * {slabs}, rec.kept_slabs()
        """)


# The shapes of the GPU tests that are to go by kept values do
@pytest.mark.parametrize("n,M,d,t,cross,kind", [(1100, 130, 400, 1, 1, 0), (900, 257, 784, 20, 1, 0), (256, 128, 700, 16, 1, 0), (1537, 33, 705, 17, 1, 0),
                                                (1, 1, 700, 1, 1, 0), (700, 100, 300, 3, 1, 1), (513, 255, 301, 9, 1, 3), (1025, 128, 90, 2, 0, 0),
                                                (257, 31, 91, 32, 0, 1)])
def test_fits_that_read_kept_values(shims, n, M, d, t, cross, kind):
    _run(shims, f"""
        assert lib.knm_set_cross_term(ctx, {cross}) == 0 and lib.knm_set_kernel(ctx, {kind}) == 0
        assert lib.falkon_fit(ctx, x, {n}, {d}, {d}, y, {t}, cen, {M}, {d}, 1.0, 1e-4, 1e-6, 8, alpha, None) == 0
        assert rec.kept_reads() == 2 * 8 + 1 and rec.kept_blocks() == 1, rec.kept_reads()
        """)


@pytest.mark.parametrize("n,M,d,t", [(1, 1, 700, 1), (33, 127, 700, 2), (255, 257, 330, 12), (256, 128, 401, 7), (1000, 511, 784, 10), (2049, 31, 305, 9),
                                     (1537, 1025, 784, 1), (40001, 300, 320, 3), (55003, 25000, 400, 10), (40000, 36000, 400, 2)])
def test_products_that_keep_slabs(shims, n, M, d, t):
    _run(shims, f"""
        assert prod({n}, {M}, {d}, {t}) == 0
        assert rec.kept_slabs() > 0
        """)


# bench.py prices a product by whether it forms its values once: its rule is the library's
def test_the_benchmarks_rule_for_slabs(shims):
    shapes = [(n, d, M, t, cross, kind) for n, M in ((2_000_000, 50_000), (30_000, 3000), (20_480, 1 << 20), (20_480, (1 << 20) + 128), (1000, 3 << 20),
                                                     (256, 3 << 20))
              for d in (28, 233, 234, 239, 240, 260, 261, 304, 305, 784) for t in (1, 4, 6, 8, 10, 12, 13, 40) for cross, kind in ((1, 0), (0, 0), (1, 1))]
    _run(shims, f"""
        import os, sys, types
        sys.path.insert(0, {os.path.dirname(HERE)!r})
        import bench
        for n, d, M, t, cross, kind in {shapes!r}:
            assert lib.knm_set_cross_term(ctx, cross) == 0 and lib.knm_set_kernel(ctx, kind) == 0
            before = rec.kept_slabs()
            assert prod(n, M, d, t) == 0
            w = types.SimpleNamespace(n=n, d=d, M=M, t=t)
            once = bench.forms_values_once(w, "f16x3" if cross else "f32", "laplacian" if kind else "gaussian")
            assert once == (rec.kept_slabs() > before), (n, d, M, t, cross, kind, once)
        """)


# A captured product holds pointers into its slab: no other call frees that or moves it, and none is allocated while the stream is captured
def test_slab_of_a_captured_product_stays(shims):
    _run(shims, """
        n, M, d, t = 40000, 20000, 784, 10
        hip.fake_set_capturing(1)
        lib.knm_prod(ctx, x, n, 784, d, cen, M, d, 1.0, v, t, None, u)
        assert rec.kept_slabs() == 0  # two sweeps: nothing to take it from
        hip.fake_set_capturing(0)
        assert prod(n, M, d, t) == 0 and rec.kept_slabs() == 1
        slab, held = rec.kept_slab(), lib.knm_workspace_held(ctx)
        hip.fake_set_capturing(1)
        assert prod(n, M, d, t) == 0 and rec.kept_slabs() == 2 and rec.kept_slab() == slab
        assert lib.knm_workspace_held(ctx) == held and hip.fake_live() == created + held
        hip.fake_set_capturing(0)
        assert fit(1_000_000, 400, 2000, 10) == 0 and fit(5_000_000, 300, 3000, 1) == 0  # idle blocks of 16 GiB and more
        assert hip.fake_inside(slab, 4 * n * M)
        hip.fake_set_budget(hip.fake_live() + (1 << 20))
        assert fit(3_000_000, 784, 3000, 12) in (0, -3)
        hip.fake_set_budget(1 << 50)
        assert hip.fake_inside(slab, 4 * n * M)
        assert prod(n // 2, M // 2, d, t) == 0 and rec.kept_slab() == slab
        assert lib.knm_release_workspace(ctx) == 0 and hip.fake_live() == created
        """)


# One that was not is given up when a fit finds no room, and comes back with the next product
def test_slab_is_given_up_when_a_fit_needs_the_room(shims):
    _run(shims, """
        assert fit(3_000_000, 28, 3000, 1) == 0
        need = hip.fake_peak()
        lib.knm_release_workspace(ctx)
        assert prod(40000, 20000, 784, 10) == 0 and rec.kept_slabs() == 1
        slab = rec.kept_slab()
        hip.fake_set_budget(need + (1 << 30))
        assert fit(3_000_000, 28, 3000, 1) == 0
        assert not hip.fake_inside(slab, 1 << 30)
        hip.fake_set_budget(1 << 50)
        assert prod(40000, 20000, 784, 10) == 0 and rec.kept_slabs() == 2
        assert hip.fake_live() == created + lib.knm_workspace_held(ctx)
        lib.knm_destroy(ctx)
        assert hip.fake_live() == 0
        """)


# What is for speed alone (a fit's values, a slab) leaves a sixteenth of the card to the rest of the program, and beyond 4 GiB of idle blocks
# so does the pool
def test_kept_values_leave_room(shims):
    _run(shims, """
        import time
        def others_leave(bytes):
            hip.fake_set_budget(bytes)
            time.sleep(0.06)  # the pool asks that often
        card = 288 << 30
        hip.fake_set_total(card)
        for n, d, M, t in ((500_000, 400, 3000, 10), (1_000_000, 400, 2000, 1)):
            others_leave(card)
            reads, slabs = rec.kept_reads(), rec.kept_slabs()
            assert fit(n, d, M, t) == 0 and rec.kept_reads() == reads + 7
            assert prod(n, M, d, t) == 0 and rec.kept_slabs() > slabs
            assert lib.knm_workspace_held(ctx) > 5 << 30
            lib.knm_release_workspace(ctx)
            others_leave(card // 16 + (3 << 30))  # the rest is others'
            reads, slabs = rec.kept_reads(), rec.kept_slabs()
            assert fit(n, d, M, t) == 0 and rec.kept_reads() == reads
            assert lib.knm_workspace_held(ctx) < 5 << 30
            assert prod(n, M, d, t) == 0 and rec.kept_slabs() == slabs
            lib.knm_release_workspace(ctx)
            others_leave(card)
            assert fit(n, d, M, t) == 0 and lib.knm_workspace_held(ctx) > 5 << 30
            others_leave(hip.fake_live() + (1 << 30))
            assert fit(n, d, M, t) == 0 and lib.knm_workspace_held(ctx) < 5 << 30
            lib.knm_release_workspace(ctx)
        """)
