"""How a sweep's stream is cut into chunks, and which workgroup takes which of them (host code, no GPU needed)."""
import ctypes
import itertools
import os
import random
import subprocess

import pytest

GAUSSIAN, LAPLACIAN, MATERN52 = 0, 1, 3
F32, F16X3 = 0, 1


@pytest.fixture(scope="module")
def plan():
    import paper_2006_10350_amd as pkg

    lib = ctypes.CDLL(pkg.LIB_PATH)
    choose = lib._ZN3knm13choose_chunksElliiiiPl
    choose.restype = ctypes.c_int64
    choose.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    for name in ("_ZN3knm17gemm_stage_pointsEv", "_ZN3knm12stage_pointsEv", "_ZN3knm20gemm_fixed_per_blockEv",
                 "_ZN3knm16f16_stage_pointsEii", "_ZN3knm15fixed_per_blockEi"):
        getattr(lib, name).restype = ctypes.c_int64

    class Plan:
        @staticmethod
        def chunks(nF, nS, d, t, cross, kind):
            length = ctypes.c_int64()
            return choose(nF, nS, d, t, cross, kind, ctypes.byref(length)), length.value

        @staticmethod
        def fp32_mfma_chunks(nF, nS, d):
            length = ctypes.c_int64()
            chunks = lib._ZN3knm17choose_chunks_forElliiiibPl
            chunks.restype = ctypes.c_int64
            chunks.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_void_p]
            return chunks(nF, nS, d, 1, F32, GAUSSIAN, False, ctypes.byref(length)), length.value

        @staticmethod
        def engine(d, t, cross, kind):
            """(K-loop engine?, points per stage, fixed points per block, sums through a chunk in fp32?)"""
            if lib._ZN3knm15use_gemm_engineEiiii(d, t, cross, kind) & 1:
                fp32 = lib._ZN3knm18gemm_f16_fp32_sumsEiii(d, t, kind) & 1 if cross == F16X3 else lib._ZN3knm14gemm_fp32_sumsEi(t) & 1
                return True, lib._ZN3knm17gemm_stage_pointsEv(), lib._ZN3knm20gemm_fixed_per_blockEv(), bool(fp32)
            stage = lib._ZN3knm16f16_stage_pointsEii(d, kind) if cross == F16X3 else lib._ZN3knm12stage_pointsEv()
            return False, stage, lib._ZN3knm15fixed_per_blockEi(d), True

    return Plan


def _shapes():
    rng = random.Random(3)
    sizes = [1, 127, 128, 129, 2047, 2049, 60_000, 262_144, 262_145, 11_000_000]
    yield from itertools.product(sizes, sizes, [8, 45, 784], [1, 10, 13, 144], [F32, F16X3], [GAUSSIAN, MATERN52])
    for _ in range(2000):
        nF, nS = (int(10 ** rng.uniform(0, 7.2)) for _ in range(2))
        yield (nF, nS, int(10 ** rng.uniform(0, 3)), rng.choice([1, 1, 2, 8, 12, 13, 16, 17, 60, 160, 161, 400]),
               rng.choice([F32, F16X3]), rng.choice([GAUSSIAN, LAPLACIAN, MATERN52]))


def test_chunks_cover_the_stream_within_their_bounds(plan):
    for shape in _shapes():
        nF, nS, d, t, cross, kind = shape
        chunks, length = plan.chunks(*shape)
        gemm, stage, block, fp32_sums = plan.engine(d, t, cross, kind)
        assert 1 <= chunks <= 65535 and length % stage == 0, shape
        assert (chunks - 1) * length < nS <= chunks * length, shape
        assert length <= (1 << 18) + stage, shape
        # 4096 workgroups, at least 2048 points per chunk: what calls with limited workspace use.  fp32 sums are never longer, and
        # partials of more than 48 MB are only made where that rule has as many
        blocks = -(-nF // block)
        want = -(-4096 // blocks)
        if gemm:
            want = max(want, 16)
        want = max(min(want, -(-nS // (16 * stage if gemm else 2048))), -(-nS // (1 << 18)))
        compact = -(-(-(-nS // want)) // stage) * stage
        if fp32_sums:
            assert length <= compact, shape
        if 4 * chunks * nF * t > 48 << 20:
            assert chunks <= max(-(-nS // compact), 1), shape


def test_sums_of_three_part_products_are_no_longer_than_the_fp32_engines(plan):
    rng = random.Random(4)
    shapes = [(120_000, 3000), (3000, 120_000), (40_000, 9000), (9000, 40_000), (1_000_003, 20_001), (20_001, 1_000_003)]
    shapes += [tuple(int(10 ** rng.uniform(2, 7.2)) for _ in range(2)) for _ in range(500)]
    for nF, nS in shapes:
        for d in range(1, 18):
            chunks, length = plan.chunks(nF, nS, d, 1, F32, GAUSSIAN)
            assert length <= plan.fp32_mfma_chunks(nF, nS, d)[1], (nF, nS, d)


def test_every_workgroup_pair_is_taken_once(tmp_path):
    """The numbering of the K-loop engine's workgroups over the XCDs: every (fixed block, chunk) once, none outside."""
    import paper_2006_10350_amd as pkg

    csrc = os.path.join(os.path.dirname(pkg.LIB_PATH), "csrc")
    (tmp_path / "map.cpp").write_text("""
        #include "knm_patch_map.h"
        #include <cstdio>
        #include <vector>
        int main()
        {
            for (int64_t blocks = 1; blocks <= 700; blocks += blocks < 140 ? 1 : 37)
                for (int64_t chunks = 1; chunks <= 70; ++chunks) {
                    const knm::PatchMap pm = knm::PatchMap::make(blocks, chunks);
                    std::vector<int> seen((size_t)(blocks * chunks), 0);
                    int64_t per_xcd[8] = {0};
                    for (int64_t wg = 0; wg < pm.workgroups(); ++wg) {
                        int64_t f, c;
                        if (!pm.find(wg, f, c)) continue;
                        if (f < 0 || f >= blocks || c < 0 || c >= chunks || seen[(size_t)(f * chunks + c)]++) return 1;
                        ++per_xcd[wg & 7];
                    }
                    int64_t most = 0, total = 0;
                    for (int64_t n : per_xcd) {
                        most = n > most ? n : most;
                        total += n;
                    }
                    if (total != blocks * chunks) return 2;
                    // no XCD more than one above the even share per group of 8 chunks
                    if (8 * most > total + 8 * ((chunks + 7) / 8)) return 3;
                }
            return 0;
        }
        """)
    exe = str(tmp_path / "map")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", csrc, "-I", "/opt/rocm/include", "-o", exe,
                    str(tmp_path / "map.cpp")], check=True)
    assert subprocess.run([exe], timeout=100).returncode == 0
