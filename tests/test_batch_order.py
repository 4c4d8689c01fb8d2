"""Which particles a workgroup's batches start at (batch_order, batch_start and batch_begins of
pic_types.hpp, built here with the host compiler): every particle in one batch for all orders,
and whole starts up to the 2^40 particles that pic_init takes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "pic_types.hpp"
using namespace pic;
static int fails = 0;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s, n %lld\n", __LINE__, #c, (long long)n); ++fails; } } while (0)

// a small run: each batch of each workgroup, as the passes' loops visit them
template <bool MASKS> static void small(long long n, int batch, int nblocks, bool interleave, bool reverse)
{
    int64_t chunk = (n + nblocks - 1) / nblocks;
    chunk = (chunk + 63) / 64 * 64;
    nblocks = (int)((n + chunk - 1) / chunk);
    std::vector<int> seen(n, 0);
    for (int b = 0; b < nblocks; ++b) {
        const int64_t p0 = b * chunk, p1 = interleave ? n : (p0 + chunk < n ? p0 + chunk : n);
        const BatchOrder o = batch_order<MASKS>(p0, batch, interleave, b, nblocks, n, reverse);
        for (int k = 0; batch_begins(batch_start(o, k), p1); ++k)
            for (int64_t p = batch_start(o, k); p < batch_start(o, k) + batch && p < p1; ++p)
                ++seen[p];
        // the batches claimed past the end begin nowhere either
        int k = 0;
        while (batch_begins(batch_start(o, k), p1))
            ++k;
        for (int j = 0; j < 16; ++j)
            CHECK(!batch_begins(batch_start(o, k + j), p1));
    }
    for (int v : seen)
        CHECK(v == 1);
}

template <bool MASKS> static void run()
{
    const long long sizes[] = {1, 63, 64, 65, 127, 128, 129, 1000, 8191, 8192, 8193};
    for (long long n : sizes)
        for (int batch : {64, 128, 256})
            for (int nblocks : {1, 2, 7, 256})
                for (int how = 0; how < 3; ++how)
                    small<MASKS>(n, batch, nblocks, how > 0, how == 2);
    // large runs: the chunks of 256 workgroups, first and last batches of every order
    for (int e = 30; e <= 40; ++e)
        for (long long d : {-65LL, 0LL, 64LL}) {
            const long long n = (1LL << e) + (e == 40 && d > 0 ? 0 : d);
            const int64_t chunk = ((n + 255) / 256 + 63) / 64 * 64;
            const int nb = (int)((n + chunk - 1) / chunk);
            for (int b : {0, 1, nb / 2, nb - 1}) {
                const int64_t p0 = b * chunk;
                CHECK(batch_start(batch_order<MASKS>(p0, 128, false, b, nb, n, false), 0) == p0);
                const int last = (int)(((n - 1) / 128 - b) / nb);      // its last batch
                const BatchOrder f = batch_order<MASKS>(p0, 128, true, b, nb, n, false);
                const BatchOrder r = batch_order<MASKS>(p0, 128, true, b, nb, n, true);
                CHECK(batch_start(f, 0) == 128LL * b && batch_begins(batch_start(f, last), n));
                CHECK(!batch_begins(batch_start(f, last + 1), n));
                CHECK(batch_start(r, 0) == ((n - 1) / 128 - b) * 128 && batch_begins(batch_start(r, 0), n));
                CHECK(batch_begins(batch_start(r, last), n) && batch_start(r, last) / 128 < nb);
                CHECK(!batch_begins(batch_start(r, last + 1), n));
            }
        }
}

int main()
{
    run<false>();
    run<true>();
    std::printf(fails ? "failed\n" : "ok\n");
    return fails != 0;
}
"""


def test_batches_cover_the_particles(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    src, exe = tmp_path / "order.cpp", str(tmp_path / "order")
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2411_09605_amd", "csrc"),
                    "-o", exe, str(src)], check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
