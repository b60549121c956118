"""Rules that the library decides on the host, asked of its internal functions by a small program
that links against it: nothing is launched, so no GPU is needed."""
import os
import subprocess

import pytest

from paper_2501_08697_amd import build

PRELUDE = r"""
#include "columns_plane.hpp"
#include "gemm.hpp"
#include "local.hpp"
#include <cstdio>
using namespace apw;
namespace apw {
size_t heev_part_bytes(int n, int nw);   // dense_large.hip
}
// the fields of a plan that the rules read: a sphere of a quarter of the grid length
static void fill(Plan &P, int n1, int n2, int n3) {
    P.N1 = n1; P.N2 = n2; P.N3 = n3;
    P.N = (int64_t)n1 * n2 * n3;
    P.nslab = n1 / 2 + 1;
    P.max_ncol = n1 * n2 / 5;
    P.ldc = (P.max_ncol + 15) / 16 * 16;
    P.zero_band[0] = P.zero_band[1] = P.zero_band[2] = true;
}
"""


@pytest.fixture
def ask(tmp_path):
    """Compiles and runs `body` as main; returns the numbers it prints."""
    def f(body):
        src, exe = tmp_path / "t.cpp", tmp_path / "t"
        src.write_text(PRELUDE + "int main() {\n" + body + "\nfflush(stdout); _Exit(0); }\n")
        libdir = os.path.dirname(build.LIB)
        r = subprocess.run([build.HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-O1",
                            f"-I{build.ROOT}/include", f"-I{build.CSRC}", str(src), "-o", str(exe), f"-L{libdir}",
                            f"-l:{os.path.basename(build.LIB)}", f"-Wl,-rpath,{libdir}"], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return [int(v) for v in subprocess.run([str(exe)], capture_output=True, text=True, check=True,
                                               timeout=60).stdout.split()]
    return f


def test_fp32_columns_refuse_lengths_without_a_kernel(ask):
    """An FP32 z pass of a length that has only an FP64 kernel is an internal error (-10), never the FP64
    kernel on FP32 data, and the rule that chooses the columns looks at all three lengths."""
    got = ask("""
    for (int n3 : {90, 96, 128}) {
        Plan P;
        fill(P, 72, 72, n3);
        ColumnsCall c{&P, 0, 1, BatchArgs{1, 0, 0, 1}, nullptr, nullptr, nullptr, 1};
        printf("%d %d %d\\n", (int)local_uses_columns(P, 1, 1), columns_inverse(c, nullptr, nullptr),
               columns_forward(c, nullptr, nullptr));
    }
    Plan P;
    fill(P, 72, 72, 72);
    printf("%d\\n", (int)local_uses_columns(P, 1, 1));
    """)
    assert got == [0, -10, -10] * 3 + [1]


def test_overlap_keeps_its_batches(ask):
    """With the projector GEMMs on a second stream the local term runs in batches of at most 64 bands, so
    that their accumulation can begin; without it the columns take every band that their work space holds."""
    got = ask("""
    Plan P;
    fill(P, 72, 72, 72);
    for (int ov : {0, 1, 2}) {
        g_overlap = ov;
        printf("%d %d\\n", local_band_batch(P, 0, 0, 1, 128), local_band_batch(P, 0, 0, 1, 40));
    }
    g_overlap = 1;
    g_band_batch = 100;
    printf("%d\\n", local_band_batch(P, 0, 0, 1, 128));
    """)
    assert got == [128, 40, 64, 40, 128, 40, 100]


def test_batched_products_fit_a_grid(ask):
    """Several k-points in one launch: their K splits and their column tiles add up in the grid's z and y,
    which hold 65,536 work-groups each (a 128^3 grid has spheres of up to 2,048,383 plane waves)."""
    got = ask("""
    for (int K : {100, 24000, 161235, 1100000, 2048383})
        for (int M : {1, 500})
            for (int hint : {0, 16, 64, 1024}) {
                const int n = gemm_batch_limit(M, 16, K, 16, hint);
                const int splits = hint ? ceil_div(K, hint) : std::max(512, ceil_div(K, 1024));
                printf("%d ", n == 1 || (n >= 1 && n <= kGemmMaxBatch && n * splits <= 65536));
            }
    for (int G : {100, 24000, 161235, 524000, 1100000, 2048383})
        printf("%d ", gemm_nn_batch_limit(G));
    printf("%d %d", gemm_batch_limit(63, 37, 4000, 16, 0), gemm_batch_limit(1, 1, 1100000, 16, 0));
    """)
    assert got[:40] == [1] * 40
    for g, n in zip((100, 24000, 161235, 524000, 1100000, 2048383), got[40:46]):
        assert 1 <= n <= 8 and n * -(-g // 64) <= 65536
    assert got[40:44] == [8, 8, 8, 8] and got[46:] == [8, 8]


def test_eigensolver_partial_sums_fit(ask):
    """The region the eigensolver sets aside for partial sums holds those of every product that uses it, also
    where fewer eigenvectors than a reflector block's 32 are wanted (at one vector of order 300 the Gram matrices
    of the blocks need 32 times the sums of V^H coef, and ran on into the next region)."""
    got = ask("""
    for (int n : {257, 300, 1024, 4096})
        for (int nw : {1, 20, 31, 32, 33, 200})
            for (int m : {1, 5, 32})
                printf("%d ", heev_part_bytes(n, nw) >= gemm_cn_part_bytes(m, m, n, 16, 0) &&
                                  heev_part_bytes(n, nw) >= gemm_cn_part_bytes(m, nw, n, 16, 0));
    printf("%d", gemm_cn_part_bytes(32, 1, 300, 16, 0) < gemm_cn_part_bytes(32, 32, 300, 16, 0));
    """)
    assert got == [1] * (4 * 6 * 3) + [1]


def test_a_plane_alone_on_its_cu_takes_all_its_threads(ask):
    """Threads and LDS (KB) of a plane work-group: two of 256 threads to a CU, or one of 512, never one of 256."""
    got = ask("""
    for (int n : {45, 64, 72, 80, 81, 90, 96, 108})
        for (int rows : {n / 2 + 1, n / 2 + 5, 2 * n / 3, 4 * n / 5}) {
            Plan P;
            fill(P, n, n, n);
            P.nslab = rows;
            const PlaneShape s = plane_shape(P, 0);
            printf("%d %d %d ", s.C, s.NT, (int)(s.lds / 1024));
        }
    """)
    for c, nt, kb in zip(got[::3], got[1::3], got[2::3]):
        assert c == 0 or (kb < 160 and nt <= 512 and (nt > 256 if kb >= 80 else nt <= 512)), (c, nt, kb)


def test_bands_of_a_plane_work_group(ask):
    """Bands per work-group (planes, bands, work-groups a compute unit holds) whose last round is not left part
    empty: the choices within 5% of the fastest of 1 to 8 in timings of the plane pass."""
    good = {(72, 48, 3): {2, 3, 5}, (72, 100, 3): {2, 3, 5}, (72, 16, 2): {1, 3}, (64, 100, 3): {1, 2, 3, 5},
            (32, 200, 4): {7}, (81, 39, 2): {1, 2, 7}, (96, 48, 1): {3, 6}, (108, 48, 1): {7}, (120, 4, 1): {2}}
    got = ask("".join(f'printf("%d ", plane_bands({n}, {nb}, {q}));' for n, nb, q in good))
    for g, (case, ok) in zip(got, good.items()):
        assert g in ok, (case, g)


def test_columns_of_wide_spheres(ask):
    """Which spheres take the column passes, by their columns' share of the slab (per cent): planes from 72 x 72
    on, of those that the slab passes hold whole in LDS, only up to a share at which they are not slower. (At 108 and 68 the plane does not fit.)"""
    def uses(n, prec, share):
        return f"""{{ Plan P; fill(P, {n}, {n}, {n}); P.nslab = (int)({n} * {share} / 78.5) | 1;
                    P.max_ncol = {share} * P.nslab * {n} / 100; P.ldc = (P.max_ncol + 15) / 16 * 16;
                    printf("%d ", (int)local_uses_columns(P, {prec}, {prec})); }}"""
    table = {(72, 0): (1, 1, 1, 0), (81, 0): (1, 1, 0, 0), (96, 0): (1, 1, 0, 0), (108, 0): (1, 1, 1, 0),
             (48, 0): (1, 1, 1, 1), (72, 1): (1, 0, 0, 0), (80, 1): (1, 0, 0, 0), (64, 1): (1, 1, 1, 1)}
    got = ask("".join(uses(n, prec, share) for n, prec in table for share in (41, 51, 58, 68)))
    assert [tuple(got[i:i + 4]) for i in range(0, len(got), 4)] == list(table.values())
