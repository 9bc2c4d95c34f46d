"""Which kernels a call launches, by their names: on the host, with a HIP runtime that runs no kernels (fake_hip.c)."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2006_10350_amd", "libknm.so")

RECORD = """
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
enum { kFunctions = 4096 };
static const void *functions[kFunctions];
static const char *names[kFunctions];
static long counts[kFunctions];
static int known;
static size_t live; /* device memory held at most when a leaf of a factorisation was launched */
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *size)
{
    (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
    if (known == kFunctions) return;
    functions[known] = host;
    names[known++] = name;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)grid; (void)block; (void)args; (void)lds; (void)stream;
    for (int i = 0; i < known; ++i)
        if (functions[i] == f) {
            ++counts[i];
            size_t (*held)(void) = (size_t (*)(void))dlsym(RTLD_DEFAULT, "fake_live");
            if (strstr(names[i], "leaf") && held() > live) live = held();
        }
    return 0;
}
long launched(const char *part) /* launches of kernels with this in their (mangled) name */
{
    long n = 0;
    for (int i = 0; i < known; ++i)
        if (strstr(names[i], part)) n += counts[i];
    return n;
}
size_t live_at_most(void) { return live; }
void forget(void)
{
    memset(counts, 0, sizeof counts);
    live = 0;
}
"""

HEAD = """
import ctypes as c
rec, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
lib = c.CDLL({lib!r})
P, L, I, F, D, Z = c.c_void_p, c.c_int64, c.c_int, c.c_float, c.c_double, c.c_size_t
hip.fake_set_budget.argtypes = hip.fake_set_total.argtypes = [Z]
hip.fake_live.restype = hip.fake_peak.restype = lib.knm_workspace_held.restype = Z
lib.knm_workspace_held.argtypes = lib.knm_release_workspace.argtypes = lib.knm_destroy.argtypes = [P]
lib.knm_last_error.restype = c.c_char_p
lib.knm_last_error.argtypes = [P]
lib.knm_set_pack_limit.argtypes = [P, Z]
lib.knm_prod.argtypes = lib.knm_prod_static.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P, P]
ctx = P()
assert lib.knm_create(c.byref(ctx), 0, None) == 0
x, cen, v, u, w = (P(0x7f0000000000 + (i << 40)) for i in range(5))  # never read: kernels do not run


def launched(name):
    return rec.launched(name.encode())


def prod(n, M, d, t):
    rec.forget()
    return lib.knm_prod(ctx, x, n, d, d, cen, M, d, 1.0, v, t, None, u)


def prod_static(n, M, d, t):
    rec.forget()
    return lib.knm_prod_static(ctx, x, n, d, d, cen, M, d, 1.0, v, t, w, u)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("hip")
    (tmp / "record.c").write_text(RECORD)
    shims = []
    for name, src in (("record", str(tmp / "record.c")), ("fakehip", os.path.join(HERE, "fake_hip.c"))):
        shims.append(str(tmp / f"lib{name}.so"))
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", f"-Wl,-soname,lib{name}.so", "-o", shims[-1], src], check=True)

    def go(body):
        """In a process of its own: the fake runtime must come before the real one."""
        r = subprocess.run([sys.executable, "-c", HEAD.format(shims=shims, lib=LIB) + textwrap.dedent(body)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr

    return go


# Sums over kept values run on the matrix cores: only products whose sweeps' sums do too, in every group of 160 columns, go by them, and
# bench.py prices them by the same rule
def test_products_with_many_columns_that_keep_values(run):
    shapes = [(n, M, d, t) for n, M in ((60_000, 10_000), (9_000, 11_000), (1_500, 3 << 20))
              for d in (179, 180, 209, 210, 319, 320, 449, 450, 784)
              for t in (12, 13, 16, 17, 32, 33, 64, 65, 128, 129, 160, 161, 167, 168, 172, 173, 176, 177, 320, 321, 330)]
    run(f"""
        import sys, types
        sys.path.insert(0, {os.path.dirname(HERE)!r})
        import bench
        kept = 0
        for n, M, d, t in {shapes!r}:
            assert prod(n, M, d, t) == 0
            once = launched("kept_many_kernel") > 0
            groups = [160] * (t // 160) + [t % 160] * (t % 160 > 0)
            mc = all(g > 16 or (g >= 8 and 4 * (3 + g) >= 3 * ((d + 15) // 16) + 1) for g in groups)
            assert mc or not once, (n, M, d, t)
            assert once == bench.sums_many_columns(types.SimpleNamespace(n=n, M=M, d=d, t=t), "f16x3", "gaussian"), (n, M, d, t)
            kept += once
        assert 0 < kept < {len(shapes)}
        """)


# bench.py names the engine that the library takes
def test_the_engine_that_the_benchmark_names(run):
    shapes = [(n, M, d, t, cross, kind) for n, M in ((5_900_000, 100_000), (60_000, 2000), (9000, 9000), (2000, 500)) for d in (1, 8, 14, 15, 28, 29, 44, 45, 64, 65)
              for t in (1, 2) for cross, kind in ((1, 0), (0, 0), (1, 1), (0, 1))]
    run(f"""
        import sys, types
        sys.path.insert(0, {os.path.dirname(HERE)!r})
        import bench
        for n, M, d, t, cross, kind in {shapes!r}:
            assert lib.knm_set_cross_term(ctx, cross) == 0 and lib.knm_set_kernel(ctx, kind) == 0
            assert prod_static(n, M, d, t) == 0 or prod(n, M, d, t) == 0
            name = bench.engine_of(types.SimpleNamespace(n=n, M=M, d=d, t=t), "f16x3" if cross else "f32", "laplacian" if kind else "gaussian")[0]
            assert launched(name) > 0, (n, M, d, t, cross, kind, name)
        """)


# The image of three-part numbers is for speed alone: it leaves a sixteenth of the card free and every other buffer where it is, and a call that
# does without it has no error to report
def test_three_part_images_leave_room(run):
    run("""
        import time
        n, M, d, t = 4_000_000, 20_000, 9, 1
        card = 288 << 30
        hip.fake_set_total(card)
        assert lib.knm_set_cross_term(ctx, 0) == 0

        def others_leave(bytes):
            hip.fake_set_budget(hip.fake_live() + bytes)
            time.sleep(0.06)

        def engines():
            return launched("gauss_sweep_b16_kernel"), launched("gauss_sweep_kernel")

        others_leave(card // 16 + (256 << 20))  # W and the partials, but not 512 MB of image as well
        assert prod(n, M, d, t) == 0
        assert launched("gauss_sweep_b16_kernel") == 1  # the sweep over the rows packs the 20000 centres: 2.5 MB
        assert launched("gauss_sweep_kernel") == 1
        assert lib.knm_last_error(ctx) == b"" and lib.knm_workspace_held(ctx) < 256 << 20
        # nothing is allocated under capture, not even where there is room by then
        others_leave(card)
        held = lib.knm_workspace_held(ctx)
        hip.fake_set_capturing(1)
        assert prod(n, M, d, t) == 0 and engines() == (1, 1) and lib.knm_workspace_held(ctx) == held
        hip.fake_set_capturing(0)
        assert prod(n, M, d, t) == 0 and engines() == (2, 0)
        hip.fake_set_capturing(1)
        assert prod(n, M, d, t) == 0 and engines() == (2, 0)
        """)


def test_a_static_call_without_room_for_a_three_part_image(run):
    run("""
        assert lib.knm_set_cross_term(ctx, 0) == 0
        without = 0
        for n in range(16_300_000, 16_777_216, 8192):
            st = prod_static(n, 3000, 9, 1)
            assert st in (0, -2)
            if st == 0:
                assert lib.knm_last_error(ctx) == b"", n
                without += launched("gauss_sweep_kernel") > 0
        assert without > 0
        """)


# A fit in the fp32 mode keeps its images only where there is room to spare
def test_three_part_images_of_a_fit_leave_room(run):
    run("""
        lib.falkon_fit.argtypes = [P, P, L, I, L, P, I, P, L, L, F, D, D, I, P, P]
        card, n, d, M = 288 << 30, 20_000_000, 9, 1000
        hip.fake_set_total(card)
        assert lib.knm_set_cross_term(ctx, 0) == 0
        for left, b16 in ((card, 7), (card // 16 + (1 << 30), 3)):  # 2.5 GB of image for the sums over the rows
            hip.fake_set_budget(left)
            lib.knm_release_workspace(ctx)
            rec.forget()
            assert lib.falkon_fit(ctx, x, n, d, d, v, 1, cen, M, d, 1.0, 1e-4, 1e-6, 3, u, None) == 0
            assert launched("gauss_sweep_b16_kernel") == b16 and launched("gauss_sweep_kernel") == 7 - b16, launched("gauss_sweep_b16_kernel")
            assert lib.knm_last_error(ctx) == b""
        """)


# Factorisations: by residues from the sizes that residue_pays says, where the card has room to spare; by fp64 products elsewhere, and then none of the
# room that was found for a part of the arrays is held while the factorisation runs
def test_factorisations_by_residues(run):
    run("""
        import time
        pays = lib._ZN3knm12residue_paysEllb
        pays.argtypes, pays.restype = [L, L, c.c_bool], c.c_bool
        lib.precond_build.argtypes = [P, P, L, I, L, F, D, D, P, P]
        lib.precond_free.argtypes = [P]
        rec.live_at_most.restype = Z

        def build(M):
            rec.forget()
            p = P()
            assert lib.precond_build(ctx, cen, M, 8, 8, 1.0, 1e-6, 1e-6, c.byref(p), None) == 0
            assert lib.precond_free(p) == 0
            return launched("residue_gemm_kernel")

        def width(M):  # of a block row
            return min(((M + 7) // 8 + 255) // 256 * 256, 4096)

        tri = next(M for M in range(1000, 9000) if pays(M, M, True))
        rows = next(M for M in range(1000, 9000) if pays(M - width(M), width(M), False))
        assert 3000 < tri < 4500 < rows < 6000, (tri, rows)
        assert build(tri - 1) == 0 and build(tri) == 1 and build(rows - 1) == 1
        assert build(rows) >= 3  # and a block row of each factor

        M, card = 20000, 288 << 30
        hip.fake_set_total(card)
        assert build(M) > 10
        lib.knm_release_workspace(ctx)
        full = 8 * (M + 3) * M + 2 * 8 * 2048 * (M + 2048) + (256 << 20)  # factors, inverted blocks, some vectors
        hip.fake_set_budget(card // 16 + full + (900 << 20))  # room for planes of one block row (0.76 GB), not for those of two
        time.sleep(0.06)
        assert build(M) == 0 and launched("rank_k_upper_kernel") > 0
        assert rec.live_at_most() < full
        assert lib.knm_last_error(ctx) == b""
        """)
