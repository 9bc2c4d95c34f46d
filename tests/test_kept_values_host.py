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
    for (int i = 0; i < slab_kinds; ++i) slabs += slab_sums[i] == f;
    for (int i = 0; i < known; ++i)
        if (functions[i] == f && reads < kLaunches) {
            memcpy(&values[reads], args[0], 8);
            memcpy(sizes[reads++], (char *)args[0] + 8, 16);
        }
    return 0;
}
"""


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
    body = f"""
        import ctypes as c
        rec, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
        lib = c.CDLL({LIB!r})
        rec.kept_size.restype = c.c_int64
        P, L, I, F, D = c.c_void_p, c.c_int64, c.c_int, c.c_float, c.c_double
        lib.logfalkon_fit.argtypes = [P, P, L, I, L, P, P, L, L, P, F, P, P, I, D, P, P]
        ctx = P()
        assert lib.knm_create(c.byref(ctx), 0, None) == 0
        assert lib.knm_set_cross_term(ctx, {cross}) == 0
        x, cen, y, yc, alpha = (P(0x7f0000000000 + (i << 36)) for i in range(5))  # never read: kernels do not run
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
        """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(body)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


# slabs of 4 GiB of values: one, three, many of the fewest rows (1024), fewer rows than that (two sweeps); few features, many columns and
# the other arithmetic (two sweeps)
@pytest.mark.parametrize("n,M,d,t,cross,slabs", [(40000, 20000, 784, 10, 1, 1), (40000, 50000, 784, 1, 1, 3), (20480, 1 << 20, 300, 1, 1, 20),
                                                 (20480, (1 << 20) + 128, 300, 1, 1, 0), (1000, 3 << 20, 300, 1, 1, 0), (256, 3 << 20, 300, 1, 1, 1),
                                                 (40000, 20000, 200, 1, 1, 0), (40000, 20000, 784, 13, 1, 0), (40000, 20000, 784, 1, 0, 0)])
def test_slabs_of_a_product(shims, n, M, d, t, cross, slabs):
    body = f"""
        import ctypes as c
        rec, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
        lib = c.CDLL({LIB!r})
        P, L, I, F = c.c_void_p, c.c_int64, c.c_int, c.c_float
        lib.knm_prod.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P, P]
        ctx = P()
        assert lib.knm_create(c.byref(ctx), 0, None) == 0
        assert lib.knm_set_cross_term(ctx, {cross}) == 0
        x, cen, v, u = (P(0x7f0000000000 + (i << 40)) for i in range(4))  # never read: kernels do not run
        for k in (1, 2):
            assert lib.knm_prod(ctx, x, {n}, {d}, {d}, cen, {M}, {d}, 1.0, v, {t}, None, u) == 0
            assert rec.kept_slabs() == k * {slabs}, rec.kept_slabs()
        """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(body)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
