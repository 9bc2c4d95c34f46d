"""Launches stay within what the runtime takes (fewer than 2^32 work-items in a dimension), whatever the size of a product: on the
host, with a HIP runtime that only counts (fake_hip.c)."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2006_10350_amd", "libknm.so")

CHECK = """
#include <stddef.h>
#include <stdint.h>
typedef struct { uint32_t x, y, z; } dim3;
static long launches, beyond;
long checked_launches(void) { return launches; }
long launches_beyond(void) { return beyond; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *stream)
{
    (void)lds; (void)stream;
    ++launches;
    if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || (uint64_t)g.z * b.z >> 32 || b.x * b.y * b.z > 1024 || g.y > 65535 || g.z > 65535) ++beyond;
    return 0;
}
"""


@pytest.fixture(scope="module")
def shims(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("hip")
    (tmp / "check.c").write_text(CHECK)
    out = []
    for name, src in (("check", str(tmp / "check.c")), ("fakehip", os.path.join(HERE, "fake_hip.c"))):
        out.append(str(tmp / f"lib{name}.so"))
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", f"-Wl,-soname,lib{name}.so", "-o", out[-1], src], check=True)
    return out


# several columns: partial results of n t = 2^29 entries and more in 8 chunks and more
@pytest.mark.parametrize("n,d,M,t", [(11_000_000, 28, 100_000, 64), (4_000_000, 28, 40_000, 144), (600_000, 28, 32_768, 1024),
                                     (2_000_000, 784, 50_000, 10), (1_000_000_000, 9, 100_000, 1)])
def test_products_of_many_outputs(shims, n, d, M, t):
    body = f"""
        import ctypes as c
        check, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
        lib = c.CDLL({LIB!r})
        P, L, I, F = c.c_void_p, c.c_int64, c.c_int, c.c_float
        lib.knm_prod.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P, P]
        lib.knm_t_y.argtypes = lib.knm_v.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P]
        ctx = P()
        assert lib.knm_create(c.byref(ctx), 0, None) == 0
        x, cen, v, u = (P(0x7f0000000000 + (i << 40)) for i in range(4))  # never read: kernels do not run
        assert lib.knm_prod(ctx, x, {n}, {d}, {d}, cen, {M}, {d}, 1.0, v, {t}, None, u) == 0
        assert lib.knm_v(ctx, x, {n}, {d}, {d}, cen, {M}, {d}, 1.0, v, {t}, u) == 0
        assert lib.knm_t_y(ctx, x, {n}, {d}, {d}, cen, {M}, {d}, 1.0, v, {t}, u) == 0
        check.checked_launches.restype = check.launches_beyond.restype = c.c_long
        assert check.checked_launches() > 6
        assert check.launches_beyond() == 0
        """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(body)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


# A small prediction is one launch (two where its rows are split), but not one of hundreds of thousands of workgroups with next to nothing
# to do each: few centres or many columns against many rows, which took up to 30 times as long as the engines
@pytest.mark.parametrize("n,M,d,t,cross,launches", [(200, 1000, 8, 1, 1, 1), (1, 50_001, 5, 1, 1, 2), (20_000, 1000, 8, 1, 1, 1), (5000, 300, 8, 8, 1, 1),
                                                    (20_000, 10, 8, 1, 0, 1), (100_000, 100, 8, 1, 1, None), (20_000, 300, 8, 3, 1, None),
                                                    (60_000, 30, 12, 5, 1, None), (10_000, 20, 4, 16, 0, None), (1_000_000, 1, 8, 16, 1, None),
                                                    (1_000_000, 10, 2, 3, 1, None), (1_000_000, 1, 2, 1, 0, None)])
def test_small_predictions_have_few_workgroups(shims, n, M, d, t, cross, launches):
    body = f"""
        import ctypes as c
        check, hip = (c.CDLL(s, mode=c.RTLD_GLOBAL) for s in {shims!r})
        lib = c.CDLL({LIB!r})
        P, L, I, F = c.c_void_p, c.c_int64, c.c_int, c.c_float
        lib.knm_v.argtypes = [P, P, L, I, L, P, L, L, F, P, I, P]
        lib.knm_set_cross_term.argtypes = [P, I]
        check.checked_launches.restype = c.c_long
        ctx = P()
        assert lib.knm_create(c.byref(ctx), 0, None) == 0 and lib.knm_set_cross_term(ctx, {cross}) == 0
        x, cen, v, u = (P(0x7f0000000000 + (i << 40)) for i in range(4))  # never read: kernels do not run
        before = check.checked_launches()
        assert lib.knm_v(ctx, x, {n}, {d}, {d}, cen, {M}, {d}, 1.0, v, {t}, u) == 0
        count = check.checked_launches() - before
        assert count == {launches} if {launches} else count > 1, count  # (shift and sweep at least; no rows are split here)
        """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(body)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
