"""Slices of served queries (csrc/slices.hpp), without a device: a program that serves one
query from given times per root and prints each iteration's time over its target."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "slices.hpp"
// argv: roots, split roots, ways, seconds of the first and of the last root, target,
// whether slices know the query's end
int main(int argc, char** a) {
    const int64_t roots = atoll(a[1]), split_roots = atoll(a[2]);
    gpint::TaskSplit sp;
    sp.ways = atoi(a[3]);
    sp.tasks = split_roots * sp.ways;
    const double t0 = atof(a[4]), t1 = atof(a[5]), target = atof(a[6]);
    const int64_t n_tasks = roots + split_roots * (sp.ways - 1);
    std::vector<double> end(n_tasks + 1, 0.0);  // seconds of the tasks before each
    for (int64_t t = 0; t < n_tasks; ++t) {
        const int64_t r = t < sp.tasks ? t / sp.ways : t - sp.tasks + split_roots;
        const double s = t0 + (t1 - t0) * (double)r / (double)roots;
        end[t + 1] = end[t] + (t < sp.tasks ? s / sp.ways : s);
    }
    // tasks and roots agree, also across the end of the split roots
    for (int64_t first = 0; first < n_tasks; first += 1 + n_tasks / 50)
        for (int64_t n = 1; first + n <= n_tasks; n += 1 + n_tasks / 40)
            if (llabs(sp.tasks_of(first, sp.roots(first, n) + 1e-9) - n) > 1) return 1;
    int64_t at = 0, slice = std::min<int64_t>(8192, n_tasks), iterations = 0;
    while (at < n_tasks) {
        const int64_t n = std::min(slice, n_tasks - at);
        const double s = end[at + n] - end[at];
        printf("%.4f\n", s / target);
        slice = gpint::next_slice(sp, at, n, s, at + n, target, argc > 7 ? n_tasks : 0);
        at += n;
        if (++iterations > 10000) return 2;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("slices")
    (d / "serve.cpp").write_text(PROGRAM)
    exe = str(d / "serve")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{ROOT}/paper_2009_10955_amd/csrc", str(d / "serve.cpp"), "-o", exe],
                   check=True)
    return exe


def _serve(program, *args):
    r = subprocess.run([program] + [str(x) for x in args], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.returncode
    return [float(x) for x in r.stdout.split()]


@pytest.mark.parametrize("roots,split,ways", [(400_000, 10_000, 16), (100_000, 20_000, 4), (50_000, 0, 1),
                                              (30_000, 30_000, 16), (2_000_000, 600, 64)])
def test_even_roots_keep_the_iteration_at_its_target(program, roots, split, ways):
    """Every root takes as long: no iteration after the first takes longer than its target,
    also the one in which the split roots end (their shares take a 16th of a root's
    time: a slice measured in tasks took 6 to 16 targets there)."""
    times = _serve(program, roots, split, ways, 1e-5, 1e-5, 0.025)
    assert max(times[1:], default=0) <= 1.01
    # and it does not crawl either: all but the first few and the last are on target
    assert all(t >= 0.99 for t in times[4:-1])


def test_lighter_roots_come_later(program):
    """Roots get lighter, so rates err low and iterations fall short of their target, never
    past it."""
    times = _serve(program, 1_000_000, 5_000, 16, 4e-5, 1e-7, 0.025)
    assert max(times[1:]) <= 1.01 and len(times) < 2000


@pytest.mark.parametrize("roots,split,ways", [(10_000, 256, 16), (9_000, 0, 1), (400_000, 10_000, 16)])
def test_a_short_rest_goes_at_once(program, roots, split, ways):
    """A rest of up to two shares is one slice: the last iteration takes between one and two
    targets where two would have run, and no other goes past its own."""
    cut = _serve(program, roots, split, ways, 1e-5, 1e-5, 0.025)
    times = _serve(program, roots, split, ways, 1e-5, 1e-5, 0.025, 1)
    assert sum(times) == pytest.approx(sum(cut), abs=1e-3 * len(cut))
    assert max(times[1:-1], default=0) <= 1.01 and times[-1] <= 2.01
    # the last two of the cut iterations are one, unless the first slice was all there is to one target
    assert len(times) == len(cut) - (1 if len(cut) > 2 else 0)
