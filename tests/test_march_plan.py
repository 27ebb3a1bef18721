"""Host arithmetic of the marching kernels' launches (csrc/march_plan.hpp),
compiled by the host compiler and checked against direct enumeration."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_05668_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


def run(tmp_path, body):
    """Compile body as main() with the header; undefined arithmetic ends the program."""
    src = tmp_path / "plan.cpp"
    src.write_text('#include <cstdio>\n#include "march_plan.hpp"\nint main()\n{\n' + body + "\n    return 0;\n}\n")
    exe = str(tmp_path / "plan")
    cc = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I" + CSRC,
                         str(src), "-o", exe], capture_output=True, text=True, timeout=120)
    assert cc.returncode == 0, cc.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_rows_taken_lie_within_the_descriptor(tmp_path):
    """Around the limit of every field count, lattice and element size: a row
    that march_fits takes ends within 2^31 - 1 bytes of its first tile, from
    whichever cell of the tile it begins, and nothing is refused that is more
    than two tiles below the limit."""
    out = run(tmp_path, r"""
    for (int q : {5, 9})
        for (int k = 1; k <= 18; ++k)
            for (int e : {2, 4, 8}) {
                const long long bytes = (long long)k * q * e, top = 0x7fffffff / bytes;
                for (long long nx = top - 400; nx <= top + 10; ++nx) {
                    const bool fits = march_fits(nx, 1, k * q, e);
                    for (long long b = 0; b < 64; ++b) {
                        const long long end = ((b + nx - 1) / 64 + 1) * 64 * bytes;
                        if (fits && end > 0x7fffffff) { printf("nx %lld first cell %lld, %lld bytes a cell\n", nx, b, bytes); return 1; }
                    }
                    if (!fits && nx < top - 200) { printf("refused nx %lld, %lld bytes a cell\n", nx, bytes); return 1; }
                }
            }
    puts("ok");""")
    assert out == "ok\n"


def test_segments_cover_every_row_once(tmp_path):
    """Rows of a segment, the number of segments and their ends, up to the
    tallest grids an int holds: consecutive, none empty, the last one ends with
    the grid (the sanitizer ends the program on an overflow)."""
    out = run(tmp_path, r"""
    const int most = 0x7fffffff - kMarchLanes;
    for (int ny : {1, 2, 3, 64, 1023, 1024, 1025, 2048, 43400, 1 << 20, 1 << 30, (1 << 30) + 1, most - 1024, most - 1, most})
        for (int nx : {1, 2, 56, 57, 58, 59, 64, 150, 1024, 2048, 130001})
            for (int halo = 1; halo <= 4; ++halo)
                for (int lds : {2568, 7688, 20744, 30728})
                    for (int populations : {5, 27, 63}) {
                        const int rows = march_rows(halo, lds, populations, nx, ny), n = march_segments(ny, rows);
                        bool ok = rows >= 1 && n >= 1 && (long long)(n - 1) * rows < ny && (long long)n * rows >= ny;
                        for (int g : {0, n / 2, n - 2, n - 1}) {
                            if (!ok || g < 0) continue;
                            const int y0 = g * rows, y1 = segment_end(y0, rows, ny);
                            ok = y1 > y0 && y1 <= ny && (g == n - 1 ? y1 == ny : y1 == y0 + rows);
                        }
                        if (!ok) { printf("%d rows of %d, halo %d: %d segments of %d\n", ny, nx, halo, n, rows); return 1; }
                    }
    puts("ok");""")
    assert out == "ok\n"


# us per step on an MI355X: storage code, fields, velocities, steps of a march,
# rows, columns, one step a launch, the march
MEASURED = [
    (1, 3, 9, 4, 512, 512, 9.61, 6.95), (1, 3, 9, 4, 1024, 1024, 32.57, 15.61), (1, 3, 9, 4, 2048, 2048, 149.3, 58.08),
    (1, 3, 9, 4, 200000, 1, 8.94, 120.5), (1, 3, 9, 4, 43400, 3, 5.77, 29.03), (1, 3, 9, 4, 300000, 5, 55.21, 178.8),
    (1, 3, 9, 4, 20000, 65, 48.34, 28.23), (1, 3, 9, 4, 20, 40000, 26.03, 14.40), (1, 4, 5, 4, 1500, 1500, 60.05, 24.38),
    (2, 3, 9, 4, 512, 512, 6.32, 8.42), (2, 3, 9, 4, 640, 640, 9.11, 10.98), (2, 3, 9, 4, 1024, 1024, 18.07, 20.74),
    (2, 3, 9, 4, 2048, 2048, 77.75, 50.07), (2, 3, 9, 4, 200000, 1, 5.96, 119.3), (2, 3, 9, 4, 20000, 65, 21.33, 28.66),
    (2, 6, 9, 4, 300, 700, 10.69, 14.08), (2, 6, 9, 4, 2048, 2048, 150.9, 100.2), (0, 4, 5, 3, 800, 800, 30.52, 21.11),
    (0, 4, 5, 3, 1500, 1500, 129.0, 66.90), (0, 4, 5, 3, 200000, 1, 13.11, 252.0), (0, 4, 5, 3, 43400, 3, 8.98, 59.17),
    (3, 3, 9, 4, 2048, 2048, 110.8, 68.55), (3, 6, 9, 2, 2048, 2048, 224.3, 153.2), (3, 12, 5, 2, 2048, 40, 12.50, 16.45),
]


def test_marches_are_taken_where_they_were_measured_faster(tmp_path):
    rows = []
    for st, k, q, t, ny, nx, single, march in MEASURED:
        slots, e = (9 if q == 9 else 5), {0: 8, 1: 4, 2: 2, 3: 4}[st]
        lds = [((n if st == 3 else n - 1) * slots * k * 64 + 2) * e for n in (t, 2)]
        rows.append(f"{{{st}, {k}, {q}, {t}, {lds[0]}, {lds[1]}, {ny}, {nx}, {int(march < single)}}}")
    out = run(tmp_path, "const int m[][9] = {" + ", ".join(rows) + "};" + r"""
    int wrong = 0;
    for (auto &r : m) {
        const StepState s = {r[0], r[1], r[2], false, false};
        auto halo = [&](int T) { return r[0] == 3 ? T : T - 1; };
        const int n = march_steps(s, r[3], r[4], r[5], halo, 40, 40, r[7], r[6]);
        if ((n > 1) != (r[8] != 0) || (n > 1 && n != r[3] && n != 2)) {
            printf("storage %d, %d fields, %d x %d: %d steps a launch\n", r[0], r[1], r[6], r[7], n);
            ++wrong;
        }
        // one step left, and what the kernels do not hold
        if (march_steps(s, r[3], r[4], r[5], halo, 1, 1, r[7], r[6]) != 1) ++wrong;
        if (march_steps(s, r[3], r[4], r[5], halo, 40, 40, 0x7fffffff / 8, 4) != 1) ++wrong;
    }
    // the recomputation of a 512^2 rollout, with topography and history: 8.6 us per
    // step in the march, 10.4 by single steps
    const StepState rollout = {1, 3, 9, false, true};
    if (march_steps(rollout, 4, 20744, 6920, [](int T) { return T - 1; }, 40, 40, 512, 512) != 4) ++wrong;
    // advection-diffusion with two rates in double, 600 x 512: 19.4 and 21.8 us
    const StepState rates = {0, 3, 9, true, false};
    if (march_steps(rates, 2, 13840, 13840, [](int T) { return T - 1; }, 40, 40, 512, 600) != 2) ++wrong;
    printf("%d\n", wrong);""")
    assert out == "0\n", out


def test_launches_of_one_step_come_last(tmp_path):
    """Every run of up to 70 steps of every state and many grids: its launches
    add up, and none of one step comes before a larger one."""
    out = run(tmp_path, r"""
    for (int storage = 0; storage < 4; ++storage)
        for (int q : {5, 9})
            for (int k = 1; k <= (storage == 3 ? 12 : 7); ++k)
                for (int most = 2; most <= 4; ++most)
                    for (int ny : {3, 60, 200, 450, 512, 1000, 2048, 100000})
                        for (int nx : {20, 64, 300, 512, 1100, 2048}) {
                            const StepState s = {storage, k, q, false, false};
                            const int e = storage == 0 ? 8 : storage == 2 ? 2 : 4, extra = storage == 3 ? 0 : -1;
                            auto lds = [&](int T) { return ((T + extra) * (q == 9 ? 9 : 5) * k * 64 + 2) * e; };
                            if (lds(most) > kLdsPerCu / 5) continue;
                            auto halo = [&](int T) { return storage == 3 ? T : T - 1; };
                            for (int n = 1; n <= 70; ++n) {
                                int left = n, last = most + 1;
                                while (left > 0) {
                                    const int m = march_steps(s, most, lds(most), lds(2), halo, left, n, nx, ny);
                                    const bool late = last == 1 && m > 1;
                                    if (m < 1 || m > left || late) {
                                        printf("storage %d, %d fields, %d velocities, %d x %d, run of %d, %d left: %d steps after %d\n",
                                               storage, k, q, ny, nx, n, left, m, last);
                                        return 1;
                                    }
                                    last = m, left -= m;
                                }
                            }
                        }
    // a run of three that gains little from its march takes single steps
    const StepState s = {0, 3, 9, false, false};
    for (int left = 3; left > 0; --left)
        if (march_steps(s, 2, 13840, 13840, [](int T) { return T - 1; }, left, 3, 512, 512) != 1) return 1;
    puts("ok");""")
    assert out == "ok\n"
