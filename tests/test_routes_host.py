"""Which kernels a call launches, by their names: on the host, with a HIP runtime that runs no kernels (fake_hip.c)."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2006_10350_amd", "libknm.so")

RECORD = """
#include <stdint.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
enum { kFunctions = 4096 };
static const void *functions[kFunctions];
static const char *names[kFunctions];
static long counts[kFunctions];
static int known;
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
        if (functions[i] == f) ++counts[i];
    return 0;
}
long launched(const char *part) /* launches of kernels with this in their (mangled) name */
{
    long n = 0;
    for (int i = 0; i < known; ++i)
        if (strstr(names[i], part)) n += counts[i];
    return n;
}
void forget(void) { memset(counts, 0, sizeof counts); }
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
