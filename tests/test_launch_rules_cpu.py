"""The host rules that pick a launch's shape (csrc/spd_sched.h), compiled on their
own with the host compiler and checked at the sizes on either side of each rule's
line, where both sides were timed."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1611_09704_amd", "csrc")
MAX_ITEMS = 0xFFFFFFFF

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "spd_sched.h"
// one call per line of input: rule name and its arguments; one line of results each
int main()
{
    char name[64];
    long long v[8];
    while (std::scanf("%63s", name) == 1) {
        auto get = [&](int n) { for (int i = 0; i < n; ++i) if (std::scanf("%lld", v + i) != 1) std::exit(2); };
        if (!std::strcmp(name, "stream_shape")) {
            get(3);
            const spd::StreamShape f = spd::stream_shape(v[0], v[1], v[2] != 0);
            std::printf("%d %d %lld %d\n", f.steps, f.waves, (long long)f.tiles_per_row, (int)f.aligned);
        } else if (!std::strcmp(name, "stream_once")) {
            get(1);
            std::printf("%d\n", (int)spd::stream_once(v[0]));
        } else if (!std::strcmp(name, "window_pays")) {
            get(2);
            std::printf("%d\n", (int)spd::window_pays((int)v[0], v[1] != 0));
        } else if (!std::strcmp(name, "mf_shape")) {
            get(7);
            const bool fits[3] = {v[3] != 0, v[4] != 0, v[5] != 0};
            const spd::MfShape f = spd::mf_shape((int)v[0], (int)v[1], v[2], fits, (int)v[6]);
            std::printf("%d %d\n", f.k, f.ns);
        } else {
            return 3;
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(d / "main.cpp"), "-o", exe],
                   check=True)

    def call(calls):
        text = "\n".join(" ".join(str(int(a)) if not isinstance(a, str) else a for a in c) for c in calls)
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        return [tuple(int(x) for x in line.split()) for line in out]
    return call


@pytest.mark.parametrize("rows,nout,steps,waves,aligned", [
    (50000, 600, 8, 1, 0),            # rows of one run: one wave a work-group, walked from their first start
    (200000, 100, 8, 1, 0),
    (20000, 1024, 4, 1, 0),
    (100, 1024, 2, 1, 0),             # two steps, and no third for an offset that is not used
    (100, 1025, 2, 2, 0),
    (100, 2047, 2, 2, 0),             # the last length without the outputs' boundaries
    (100, 2048, 2, 3, 1),             # 4 steps and up to 15 starts before the row
    (64, 65521, 2, 4, 1),
    (512, 262129, 8, 4, 1),
    (2048, 524266, 8, 4, 1),
])
def test_stream_shape(rule, rows, nout, steps, waves, aligned):
    (s, w, tiles, a), = rule([("stream_shape", rows, nout, 1)])
    assert (s, w, a) == (steps, waves, aligned)
    runs = -(-(-(-(nout + 15 * a) // 512)) // s)
    assert tiles == -(-runs // w)


@pytest.mark.parametrize("rows,nout,outputs,steps", [(2048, 262000, 1, 8), (2048, 262000, 0, 16),
                                                     (1024, 262000, 0, 16), (1023, 262000, 0, 8)])
def test_stream_runs_are_longer_without_outputs(rule, rows, nout, outputs, steps):
    assert rule([("stream_shape", rows, nout, outputs)])[0][0] == steps


def test_stream_shape_covers_every_row_and_fits_a_launch(rule):
    rng = random.Random(5)
    cases = [(1, 1 << 40), (1 << 24, 1), (1 << 24, 512), (1 << 24, 9000), (16776960, 32768 * 1), (1 << 23, 70000)]
    cases += [(int(2 ** rng.uniform(0, 22)), int(2 ** rng.uniform(0, 30))) for _ in range(400)]
    cases = [(r, n, len(str(n)) % 2) for r, n in cases if r * -(-n // (4 * 16 * 512)) * 256 <= MAX_ITEMS]     # what a plan takes
    for (r, n, _), (s, w, tiles, a) in zip(cases, rule([("stream_shape",) + c for c in cases])):
        assert s >= 2 and 1 <= w <= 4
        assert tiles * w * s * 512 >= n + 15 * a
        assert r * tiles * w * 64 <= MAX_ITEMS


@pytest.mark.parametrize("mb,once", [(32, 0), (128, 0), (192, 0), (256, 0), (320, 1), (400, 1), (2048, 1)])
def test_stream_loads_past_the_caches_only_from_planes_they_cannot_hold(rule, mb, once):
    assert rule([("stream_once", mb << 20)]) == [(once,)]


@pytest.mark.parametrize("n", range(1, 30))
def test_short_lists_keep_the_strided_form_on_one_plane(rule, n):
    assert rule([("window_pays", n, 0), ("window_pays", n, 1)]) == [(int(n > 16 or n in (8, 16)),), (1,)]


@pytest.mark.parametrize("C,n_dm,n_out,fits,shape", [
    (4096, 6000, 1 << 17, 7, (2, 4)), (256, 200, 50001, 7, (2, 4)), (128, 100, 10000, 7, (1, 2)),
    (512, 500, 20000, 3, (1, 2)), (33, 36, 900, 1, (0, 2)), (4096, 6000, 1 << 17, 0, (-1, 2)),
    (256, 33, 1 << 20, 7, (2, 4)), (256, 32, 1 << 20, 7, (1, 4)), (256, 24, 1 << 18, 7, (1, 2)),   # few trials
    (256, 16, 1 << 20, 7, (0, 2)), (256, 16, 1 << 18, 7, (1, 2)), (256, 17, 1 << 20, 7, (1, 4)),
    (16, 1, 1024 * 512, 7, (0, 2)), (16, 1, 1023 * 512, 7, (1, 4)),
    (16, 64, 1 << 20, 7, (2, 4)), (15, 64, 1 << 20, 7, (1, 4)), (2, 64, 1 << 20, 7, (1, 4)),       # few channels
    (1, 64, 1 << 20, 7, (-1, 2)),
])
def test_dedispersion_work_groups(rule, C, n_dm, n_out, fits, shape):
    got, = rule([("mf_shape", C, n_dm, n_out, fits & 1, fits >> 1 & 1, fits >> 2 & 1, 256)])
    assert got[0] == shape[0] and (got[0] < 0 or got == shape)
