"""The traversal's own source, compiled for the host: the functions of build_kernels.hip that clip, count and walk rays
are IEEE operations on doubles in a fixed order, so what they give here is what they give on the GPU.  For every ray the
chords of the general walk (which divides) are compared exactly with those of the dense walk and of the walk in
parts, and their number with the count by faces: rays at random, from lattice points, with equal, integer and almost
equal slopes, parallel to axes, ending on a face or next to one."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2006_03512_amd", "csrc")

HEAD = """
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::isfinite; using std::min; using std::max;
namespace mrf {
constexpr int kBrick = 8;
"""

TAIL = """
struct Chord { int k, i, j, kz; double tin, tout; };
struct Keep {
    std::vector<Chord>* v;
    void operator()(int k, int i, int j, int kz, double a, double b) const { v->push_back({k, i, j, kz, a, b}); }
    void operator()(int k, int i, int j, int kz, int lin, double a, double b) const
    {
        v->push_back({k, i, j, kz, a, b});
        if (lin != i + nx * (j + ny * kz)) v->back().k = -1;
    }
    int nx, ny;
};
static bool same(const std::vector<Chord>& a, const std::vector<Chord>& b)
{
    if (a.size() != b.size()) return false;
    for (size_t x = 0; x < a.size(); ++x)
        if (a[x].k != b[x].k || a[x].i != b[x].i || a[x].j != b[x].j || a[x].kz != b[x].kz ||
            !(a[x].tin == b[x].tin) || !(a[x].tout == b[x].tout)) return false;   // equal bits but for a zero's sign
    return true;
}
}  // namespace mrf
using namespace mrf;
// rays r: centre c, direction w, end: 0 at the grid's exit, > 0 that share of the way, < 0 on face -end of the
// crossed ones (with the last bit of the time moved by `ulp`).  stat: rays in the grid, counted, split, by division,
// and the ray and check of the first failure (0 none).
extern "C" void check(int64_t n, const int* dims, double h, const double* o, const double* c, const double* w,
                      const double* end, const int* ulp, int64_t* stat)
{
    SceneDev sd{};
    sd.W = sd.H = 1;
    sd.fx = sd.fy = 1.0;
    for (int a = 0; a < 3; ++a) sd.n[a] = dims[a], sd.o[a] = o[a], sd.nb[a] = (dims[a] + 7) / 8;
    sd.h = h;
    BuildDev bp{};
    bp.z_max = 1e300;
    for (int q = 0; q < 6; ++q) stat[q] = 0;
    std::vector<Chord> ref, got;
    const Keep keep{&got, dims[0], dims[1]};
    for (int64_t r = 0; r < n; ++r) {
        double T[16] = {0};
        for (int a = 0; a < 3; ++a) T[4 * a + 2] = w[3 * r + a], T[4 * a + 3] = c[3 * r + a];
        Ray ray;
        double ts, te;
        if (!clip_ray(sd, bp, T, 1.0f, 0, 0, ray, ts, te) || !(te > ts) || !std::isfinite(te)) continue;
        ray.ts = ts;
        ray.te = te;
        if (end[r] > 0.0) ray.te = ts + end[r] * (te - ts);
        if (end[r] < 0.0) {
            got.clear();
            walk(sd, ray, (const uint8_t*)nullptr, keep);
            ray.te = got.empty() ? te : got[(size_t)(-end[r]) % got.size()].tout;
        }
        for (int u = 0; u < std::abs(ulp[r]); ++u) ray.te = std::nextafter(ray.te, ulp[r] > 0 ? te : ts);
        if (ray.te > te) ray.te = te;
        if (!(ray.te > ray.ts)) continue;
        ++stat[0];
        got.clear();
        walk(sd, ray, (const uint8_t*)nullptr, keep);
        ref = got;
        const bool quots = times_by_quot(sd, ray);
        stat[3] += !quots;
        int bad = 0;
        got.clear();
        if (walk_dense<false>(sd, ray, keep) != (int)ref.size() || !same(ref, got)) bad = 1;
        got.clear();
        if (!bad && (walk_dense(sd, ray, keep) != (int)ref.size() || !same(ref, got))) bad = 2;
        const int cnt = quots ? count_dense(sd, ray) : -1;
        stat[1] += cnt >= 0;
        if (!bad && cnt >= 0 && cnt != (int)ref.size()) bad = 3;
        got.clear();
        size_t first = 0;
        for (int p = 0; p < kEmitParts; ++p) {
            walk_part(sd, ray, p, keep);
            if (p == 0) first = got.size();
        }
        stat[2] += first < got.size();
        if (!bad && !same(ref, got)) bad = 4;
        if (bad && !stat[5]) stat[4] = r, stat[5] = bad;
    }
}
"""


def _section(text, begin, end):
    a = text.index(begin)
    return text[a:text.index(end, a)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    with open(os.path.join(CSRC, "mrf_internal.hpp")) as f:
        hpp = f.read()
    with open(os.path.join(CSRC, "build_kernels.hip")) as f:
        hip = f.read()
    src = HEAD + _section(hpp, "struct SceneDev {", "struct FrameDev {") + _section(hpp, "struct BuildDev {", "\n\n")
    src += _section(hip, "struct Ray {", "// Pixel (u, v) of thread t of block b") + TAIL
    assert not re.search(r"threadIdx|__shared__|asm", src)   # plain functions alone
    d = tmp_path_factory.mktemp("traversal")
    (d / "t.cpp").write_text(src)
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-fPIC", "-shared", "-w", str(d / "t.cpp"),
                        "-o", str(d / "t.so"), "-lm"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return C.CDLL(str(d / "t.so"))


KINDS = ("random", "lattice", "equal slopes", "almost parallel", "almost shared", "parallel", "few bits", "near two")


def _rays(rng, kind, N, n, h, o):
    n, o = np.array(n), np.array(o)
    c = o + rng.uniform(-0.3, 1.3, (N, 3)) * n * h
    w = rng.uniform(-1, 1, (N, 3))
    sign = lambda *s: rng.choice((-1.0, 1.0), s)
    half = rng.random(N) < 0.5
    c[half] = o + rng.uniform(0, 1, (half.sum(), 3)) * n * h   # half of the centres inside
    if kind == "lattice":
        c = o + h * rng.integers(-2, n + 3, (N, 3))
        w = rng.choice((1.0, 0.5, 0.25, 0.75), (N, 3)) * sign(N, 3)
    elif kind == "equal slopes":
        w[:, 1] = sign(N) * w[:, 0]
        c[:, 1] = o[1] + sign(N) * (c[:, 0] - o[0])
        w[rng.random(N) < 0.3, 2] = 0.0
        twice = rng.random(N) < 0.3
        w[twice, 2] = w[twice, 0] * rng.choice((2.0, 3.0, 0.5, -2.0), twice.sum())
        c[twice, 2] = o[2] + (c[twice, 0] - o[0])
    elif kind == "almost parallel":
        w[np.arange(N), rng.integers(0, 3, N)] *= 2.0 ** -rng.integers(5, 60, N).astype(float)
    elif kind == "almost shared":
        e = 2.0 ** -rng.choice((18, 20, 21, 22, 24, 30, 40, 50, 52), (2, N)).astype(float)
        a, b = rng.permutation(3)[:2]
        w[:, b] = w[:, a] * (1 + rng.integers(-4, 5, N) * e[0])
        c[:, b] = o[b] + (c[:, a] - o[a]) * (1 + rng.integers(-4, 5, N) * e[1])
    elif kind == "parallel":
        for a in range(3):
            w[rng.random(N) < 0.45, a] = 0.0
        snap = rng.random((N, 3)) < 0.5
        c = np.where(snap, o + h * np.round((c - o) / h), c)
    elif kind == "few bits":
        c = o + h * rng.integers(-8, 8 * n + 8, (N, 3)) / 8.0
        w = rng.integers(-32, 33, (N, 3)) / 16.0
    elif kind == "near two":   # significands at the edge of the reciprocal quotient's range
        k = rng.integers(0, 40, (N, 3))
        w = (2.0 - k * 2.0 ** -52 * rng.choice((1, 4), (N, 3))) * 2.0 ** rng.integers(-4, 2, (N, 3)) * sign(N, 3)
    end = rng.choice((0.0, 1.0, -1.0), N) * np.where(rng.random(N) < 0.3, 1.0, rng.random(N))
    tiny = rng.random(N) < 0.05
    end[tiny] = 2.0 ** -rng.integers(1, 53, tiny.sum()).astype(float)
    end = np.where(end < 0, -rng.integers(1, 500, N).astype(float), end)
    ulp = np.where(end < 0, rng.integers(-2, 3, N), 0).astype(np.int32)
    return c, w, end, ulp


GRIDS = [((25, 25, 15), 0.2, (-2.5, -2.5, -0.3)), ((250, 240, 150), 0.02, (-2.5, 1.1, 0.0)),
         ((1, 7, 64), 0.25, (0.0, -0.875, 8.0)), ((2000, 3, 3), 0.01, (100.0, -0.01, 0.0)),
         ((64, 64, 64), 0.05, (0.0, 0.0, 0.0)), ((40, 33, 21), 0.1, (-123456.7, 3e5, 0.1)), ((1, 1, 1), 1.0, (0.0, 0.0, 0.0))]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("g", range(len(GRIDS)))
def test_counts_and_parts_are_the_general_walk(lib, g, kind):
    n, h, o = GRIDS[g]
    rng = np.random.default_rng([g, KINDS.index(kind)])
    N = 40000 if g in (1, 3) else 100000
    c, w, end, ulp = (np.ascontiguousarray(x) for x in _rays(rng, kind, N, n, h, o))
    stat = np.zeros(6, np.int64)
    p = lambda a: a.ctypes.data_as(C.c_void_p)
    lib.check(C.c_int64(N), p(np.array(n, np.int32)), C.c_double(h), p(np.array(o, np.float64)), p(c), p(w), p(end),
              p(ulp), p(stat))
    inside, counted, split, divided, ray, bad = stat.tolist()
    assert bad == 0, (("walk with divisions", "dense walk", "count by faces", "walk in parts")[bad - 1], ray,
                      [x.hex() for x in c[ray]], [x.hex() for x in w[ray]], end[ray], int(ulp[ray]))
    assert inside > 0.002 * N
    if kind == "random" and max(n) < 1024 and g != 5:   # the shortcuts are taken
        assert counted > 0.98 * inside and (split > 0.5 * inside or max(n) == 1) and divided == 0
    if kind in ("lattice", "equal slopes") and min(n) > 1 and max(n) < 1024:   # and shared times leave them
        assert counted < 0.9 * inside
    if kind == "near two":
        assert divided > 0.1 * inside
