"""Host rules of the library's dispatch that no call small enough for a test
reaches, checked on the CPU: a program that includes the internal header is
compiled for the host and compares each rule with the same one in wider
arithmetic (or with the sizes it has to cover)."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1409_5981_amd", "csrc")


def _host_program(tmp_path, body):
    """Output of a host program with `body` in main."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "pmmm_internal.h"\nusing namespace pmmm;\n'
                   "int main() {\n" + body + "\nreturn 0;\n}\n")
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    r = subprocess.run([hipcc, "-std=c++17", "-x", "hip", "--offload-host-only", "-I", CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.stdout, r.stderr)
    return r.stdout


def test_near_rule_holds_for_every_particle_count(tmp_path):
    """near_pairs_reach, which chooses the near field's kernels on the host and
    the kind of a row on the GPU, is (2c+1) np around >= pairs nx^2 for all
    counts up to 2^31 - 1, and where it holds for a row it holds for the host's
    question, which has all particles for both counts."""
    out = _host_program(tmp_path, """
    long long bad = 0, seen = 0, first = -1;
    unsigned long long seed = 1;
    auto rnd = [&]() { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return seed >> 33; };
    for (int c = 1; c <= 2; ++c)
        for (int nx = 1; nx <= 128; ++nx)
            for (int64_t pairs : {kNearLight, kNearHeavy}) {
                auto check = [&](int64_t np, int64_t around) {
                    if (np < 0 || around < np || around > INT32_MAX) return;
                    const bool want = (__int128)(2 * c + 1) * np * around >= (__int128)pairs * nx * nx;
                    ++seen;
                    const bool got = near_pairs_reach(np, around, nx, c, pairs);
                    if (got != want || (got && !near_pairs_reach(around, around, nx, c, pairs))) {
                        if (bad == 0) first = np;
                        ++bad;
                    }
                };
                for (int64_t np = 0; np < 20000; ++np) check(np, np);
                for (int e = 0; e < 32; ++e)
                    for (int k = 0; k < 32; ++k)
                        for (int64_t d = -1; d <= 1; ++d) check((int64_t(1) << e) + d, (int64_t(1) << k) + d);
                for (int64_t np = 1000003; np <= INT32_MAX; np += 9999991) check(np, np);
                for (int k = 0; k < 5000; ++k) check(rnd() >> (rnd() % 31), rnd() >> (rnd() % 31));
            }
    printf("%lld %lld %lld\\n", bad, seen, first);""")
    bad, seen, first = (int(v) for v in out.split())
    assert seen > 10 ** 7 and bad == 0, (bad, first)


def test_sort_scratch_holds_every_smaller_count(tmp_path):
    """bin_hist_ints of a capacity covers the partition's histograms, the bucket
    starts and a row of low-bit histograms per chunk (a bucket of c > kLocalTile
    particles makes at most 2 c / kLocalTile) for every count up to it, and
    never shrinks."""
    out = _host_program(tmp_path, """
    long long bad = 0;
    for (int n : {3, 4, 5, 8, 9, 16, 24, 32, 40, 64, 128}) {
        const int64_t K = (int64_t)n * n * n;
        int64_t prev = 0;
        for (int64_t np = 1; np < (int64_t(1) << 31); np += np < 10000 ? 1 : np / 1000) {
            const int hb = bin_high_bits(np, K), lb = bin_key_bits(K) - hb;
            const int64_t rows = np > kLocalTile ? 2 * np / kLocalTile : 0;
            const int64_t have = bin_hist_ints(np, K);
            if ((bin_tiles(np) << hb) + (int64_t(1) << hb) + (lb > 0 ? rows << lb : 0) > have) ++bad;
            if (have < prev) ++bad;
            prev = have;
        }
    }
    printf("%lld\\n", bad);""")
    assert int(out) == 0
