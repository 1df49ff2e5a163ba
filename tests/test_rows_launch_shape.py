"""The launch shapes of the matrix-core forward kernel, walked on the CPU over the sizes the entry points accept: the
choice (apb_rows_shape.h) is compiled with the host compiler and must end, and give a grid that exists and covers every
tile and column, for each of them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include "apb_rows_shape.h"
using namespace apb;

static long long seen = 0, bad = 0;
static void check(int N, int K, int M, int bits, bool general, bool packed_out, bool from_float) {
    if ((long long)N * M >= (1LL << 40) || (long long)N * K >= (1LL << 31)) return;
    if (from_float && (packed_out || !rows_from_float(N, K, M))) return;
    if (K > 8192 && !general) return;
    for (long long nnz : {0LL, 1LL * N, 5LL * N, 11LL * N, 18LL * N})     // (a layer gets the operands of the kernel it may be given to)
        if (columns_kernel_better(N, K, nnz, M, packed_out) && !columns_kernel_possible(N, K, nnz) && ++bad <= 20)
            std::printf("no tile runs: N=%d K=%d M=%d nnz=%lld\n", N, K, M, nnz);
    const RowsProblem q{N, M, (K + 127) / 128, bits, general, packed_out, from_float};
    const RowsShape h = pick_rows_shape(q);
    ++seen;
    const int tiles = rows_tiles(N);
    const char* why = nullptr;
    if (!(h.groups == 1 || h.groups == 2 || h.groups == 4)) why = "groups";
    else if (h.chunk <= 0 || h.nt <= 0 || h.chunk % h.nt || tiles % h.nt) why = "chunk";
    else if (h.ncw <= 0 || h.groups % h.ncw) why = "column groups of an item";
    else if (h.waves <= 0 || h.waves > 8 || h.waves % (h.groups / h.ncw) || h.waves % std::min(h.waves, h.groups)) why = "waves";
    else {
        const int chunk = std::min(h.chunk, tiles);
        const long long parts = ((long long)tiles + chunk - 1) / chunk, cols = packed_out ? (M + 63LL) / 64 * 64 : M;
        const long long wgs = (cols + 16 * h.groups - 1) / (16 * h.groups) * parts;
        if (wgs <= 0 || wgs > 0x7fffffffLL) why = "grid";
        else if (rows_lds_bytes(q, h.groups, chunk) > LDS_LIMIT) why = "LDS";
    }
    if (why && ++bad <= 20)
        std::printf("%s: N=%d K=%d M=%d bits=%d general=%d packed_out=%d from_float=%d: groups %d chunk %d waves %d nt %d ncw %d\n", why, N, K, M,
                    bits, general, packed_out, from_float, h.groups, h.chunk, h.waves, h.nt, h.ncw);
}

int main() {
    const int Ns[] = {1, 10, 16, 31, 32, 33, 48, 64, 65, 96, 100, 128, 129, 256, 512, 1000, 1024, 2048, 4096, 8192, 32000, 100000};
    const int Ks[] = {1, 31, 32, 64, 128, 288, 512, 576, 1152, 2304, 2432, 2433, 4096, 4608, 4864, 4865, 6600, 8192, 8193, 9216, 9217, 18432};
    const int Ms[] = {1, 15, 16, 17, 63, 64, 100, 256, 333, 1024, 2048, 4096, 8192, 12544, 16384, 16385, 16400, 25088, 32736, 32737, 50176, 131072,
                      1 << 20, (1 << 28) - 64};
    for (int N : Ns) for (int K : Ks) for (int M : Ms)
        for (int v = 0; v < 16; ++v) check(N, K, M, 1 + (v & 1), v & 2, v & 4, v & 8);
    unsigned long long x = 88172645463325252ULL;                  // (xorshift: sizes spread over their logarithm)
    auto pick = [&](double hi) {
        x ^= x << 13; x ^= x >> 7; x ^= x << 17;
        return (int)std::exp(std::log(hi) * (double)(x >> 11) / 9007199254740992.0);
    };
    for (int i = 0; i < 200000; ++i) {
        const int N = pick(60000), K = pick(18433), M = pick(1 << 21);
        for (int v = 0; v < 16; ++v) check(N, K, M, 1 + (v & 1), v & 2, v & 4, v & 8);
    }
    std::printf("%lld shapes, %lld bad\n", seen, bad);
    return bad != 0 || seen < 1000000;
}
"""


def walk(tmp_path, lds_limit):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-ftrapv", f"-DLDS_LIMIT={lds_limit}",
                    "-I", os.path.join(ROOT, "paper_2306_08960_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=120)
    assert p.returncode == 0, p.stdout


def test_every_accepted_size_has_a_grid_that_covers_it(tmp_path):
    walk(tmp_path, "(1LL << 40)")


def test_no_accepted_size_asks_for_more_lds_than_a_workgroup_has(tmp_path):
    walk(tmp_path, 160 * 1024)
