// Graph construction on gfx950: ray clipping and 3D-DDA traversal
// (Amanatides-Woo, the traversal Sec. IV-A names; truncation 3 sigma past the
// measurement, Sec. IV-B), device exclusive scans, a stable LSD radix sort
// for the voxel->ray incidence, and the work lists of the message kernels.
//
// The traversal is FP64 and compiled with -ffp-contract=off: every rounding
// step is an IEEE-754 operation on doubles in a fixed order, so the voxel
// ids and chord end points are reproducible bit for bit by any FP64
// implementation that performs the same operations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "dev_common.hpp"
#include "mrf_internal.hpp"

namespace mrf {

// ============================================================== traversal

struct Ray {
    double c[3], w[3];
    double Z, ts, te;
};

// Ray of pixel (u, v): centre c, direction R (x_n, y_n, 1) (t is z-depth),
// clipped to the grid box: [ts, texit].  False when the pixel has no usable
// measurement or the ray misses the grid.
__device__ bool clip_ray(const SceneDev& sd, const BuildDev& bp, const double* T, float zf, int v, int u,
                         Ray& r, double& ts_out, double& texit_out)
{
    const double Z = (double)zf;
    if (!isfinite(Z) || Z < bp.z_min || Z > bp.z_max) return false;
    const double xn = ((double)u - sd.cx) / sd.fx;
    const double yn = ((double)v - sd.cy) / sd.fy;
    double ts = 0.0, texit = __builtin_huge_val();
    for (int a = 0; a < 3; ++a) {
        r.c[a] = T[4 * a + 3];
        double wa = T[4 * a + 0] * xn;
        wa = wa + T[4 * a + 1] * yn;
        wa = wa + T[4 * a + 2];
        r.w[a] = wa;
        if (!isfinite(wa) || !isfinite(r.c[a])) return false;   // unusable pose
        const double lo = sd.o[a];
        const double hi = sd.o[a] + (double)sd.n[a] * sd.h;
        if (wa != 0.0) {
            const double t0 = (lo - r.c[a]) / wa;
            const double t1 = (hi - r.c[a]) / wa;
            const double tmn = t0 < t1 ? t0 : t1;
            const double tmx = t0 < t1 ? t1 : t0;
            if (tmn > ts) ts = tmn;
            if (tmx < texit) texit = tmx;
        } else if (r.c[a] < lo || r.c[a] >= hi) {
            return false;
        }
    }
    r.Z = Z;
    ts_out = ts;
    texit_out = texit;
    return true;
}

// The graph's ray: the clipped ray of a surface inside the grid, walked to
// Z + nsig * sigma_tr(Z) or the grid exit.
__device__ bool setup_ray(const SceneDev& sd, const BuildDev& bp, const double* T, float zf,
                          int v, int u, Ray& r)
{
    double ts, texit;
    if (!clip_ray(sd, bp, T, zf, v, u, r, ts, texit)) return false;
    const double Z = r.Z;
    if (Z >= texit) return false;   // surface outside the grid
    double sig = bp.c2 * Z;
    sig = sig * Z;
    sig = bp.c0 + sig;
    if (sig < bp.smin) sig = bp.smin;
    double te = Z + bp.nsig * sig;
    if (te > texit) te = texit;
    if (te <= ts) return false;
    r.ts = ts;
    r.te = te;
    return true;
}

__device__ __forceinline__ double face(const SceneDev& sd, int a, int idx)
{
    return sd.o[a] + (double)idx * sd.h;
}

// Boundary time of voxel index i along axis a in the walk's direction (the
// face the ray leaves voxel i through), +inf when the ray is parallel to it.
__device__ __forceinline__ double tmax_at(const SceneDev& sd, const Ray& r, int a, int i)
{
    if (r.w[a] > 0.0) return (face(sd, a, i + 1) - r.c[a]) / r.w[a];
    if (r.w[a] < 0.0) return (face(sd, a, i) - r.c[a]) / r.w[a];
    return __builtin_huge_val();
}

// The last voxel along axis a inside brick b in the walk's direction (the
// grid's last voxel for a partial brick); cur when the ray is parallel to a.
__device__ __forceinline__ int brick_last(const SceneDev& sd, const Ray& r, int a, int b, int cur)
{
    if (r.w[a] > 0.0) return min(b * kBrick + kBrick - 1, sd.n[a] - 1);
    if (r.w[a] < 0.0) return b * kBrick;
    return cur;
}

// Walk voxels from ts to te; emit(k, i, j, kz, tin, tout) for each chord of
// positive length (voxel (i, j, kz)) in an allocated brick (every brick when
// bricks is null); ties between axes step the lowest axis.  Returns count.
//
// Empty-space skip (Sec. IV-B: rays skip unallocated bricks), when skip is
// set: from a voxel of an unallocated brick the walk steps brick by brick.  The ray leaves a brick
// along an axis at the boundary time of its last voxel there (the expression
// the voxel walk evaluates at that voxel), so stepping the axis with the
// earliest such time (ties: lowest axis) visits the bricks in the voxel walk's
// order.  On entering an allocated brick across axis a at time t, every other
// axis has crossed exactly the voxel boundaries earlier than t (and one at t
// if it is the lower axis); its index is estimated from the entry point and
// settled by those comparisons.  The state then -- indices, boundary times,
// entry time -- is bit for bit the one the voxel-by-voxel walk reaches, so the
// emitted chords are unchanged.
template <class Emit>
__device__ int walk(const SceneDev& sd, const Ray& r, const uint8_t* bricks, Emit&& emit, bool skip = false)
{
    int idx[3];
    double tmax[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double p = r.c[a] + r.ts * r.w[a];
        double q = floor((p - sd.o[a]) / sd.h);
        if (q < 0.0) q = 0.0;
        if (q > (double)(sd.n[a] - 1)) q = (double)(sd.n[a] - 1);
        idx[a] = (int)q;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (r.w[a] > 0.0)
            tmax[a] = (face(sd, a, idx[a] + 1) - r.c[a]) / r.w[a];
        else if (r.w[a] < 0.0)
            tmax[a] = (face(sd, a, idx[a]) - r.c[a]) / r.w[a];
        else
            tmax[a] = __builtin_huge_val();
    }
    double tin = r.ts;
    const double inv_h = 1.0 / sd.h;
    int k = 0;
    for (;;) {
        const bool unalloc = bricks && !bricks[(idx[0] >> 3) + sd.nb[0] * ((idx[1] >> 3) + sd.nb[1] * (idx[2] >> 3))];
        if (unalloc && skip) {
            // walk brick by brick until an allocated brick, the ray's end or the grid's exit
            int bi[3], last[3];
            double tb[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                bi[a] = idx[a] >> 3;
                last[a] = brick_last(sd, r, a, bi[a], idx[a]);
                tb[a] = last[a] == idx[a] ? tmax[a] : tmax_at(sd, r, a, last[a]);
            }
            int a;
            double tm;
            bool stop = false;
            for (;;) {
                a = (tb[0] <= tb[1] && tb[0] <= tb[2]) ? 0 : (tb[1] <= tb[2] ? 1 : 2);
                tm = tb[a];
                if (tm >= r.te) {   // the ray ends in unallocated space
                    stop = true;
                    break;
                }
                bi[a] += r.w[a] > 0.0 ? 1 : -1;
                if (bi[a] < 0 || bi[a] >= sd.nb[a]) {   // it leaves the grid
                    stop = true;
                    break;
                }
                if (bricks[bi[0] + sd.nb[0] * (bi[1] + sd.nb[1] * bi[2])]) break;
                last[a] = brick_last(sd, r, a, bi[a], -1);
                tb[a] = tmax_at(sd, r, a, last[a]);
            }
            if (stop) break;
            // the voxel walk's state as it enters brick bi across axis a at time tm
            idx[a] = r.w[a] > 0.0 ? bi[a] * kBrick : min(bi[a] * kBrick + kBrick - 1, sd.n[a] - 1);
            tmax[a] = tmax_at(sd, r, a, idx[a]);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                if (b == a || r.w[b] == 0.0) continue;
                const int sg = r.w[b] > 0.0 ? 1 : -1;
                // b has crossed every boundary earlier than tm, and one at tm if it is the lower axis
                auto stepped = [&](double t) { return t < tm || (t == tm && b < a); };
                const int blo = bi[b] * kBrick, bhi = min(blo + kBrick - 1, sd.n[b] - 1);
                int first = sg > 0 ? blo : bhi;
                if ((idx[b] >> 3) == bi[b]) first = idx[b];   // still in the brick it started in
                const int lastb = sg > 0 ? bhi : blo;
                const double q = floor((r.c[b] + tm * r.w[b] - sd.o[b]) * inv_h);   // estimate only
                const int lo = min(first, lastb), hi = max(first, lastb);
                int i = (int)fmin(fmax(q, (double)lo), (double)hi);
                double ti = tmax_at(sd, r, b, i);
                while (i != lastb && stepped(ti)) {
                    i += sg;
                    ti = tmax_at(sd, r, b, i);
                }
                while (i != first) {
                    const double tp = tmax_at(sd, r, b, i - sg);
                    if (stepped(tp)) break;
                    i -= sg;
                    ti = tp;
                }
                idx[b] = i;
                tmax[b] = ti;   // the first boundary of b not yet crossed
            }
            if (tm > tin) tin = tm;
            continue;
        }
        const int a = (tmax[0] <= tmax[1] && tmax[0] <= tmax[2]) ? 0 : (tmax[1] <= tmax[2] ? 1 : 2);
        const double tm = tmax[a];
        const double tout = tm < r.te ? tm : r.te;
        if (tout > tin && !unalloc) {
            emit(k, idx[0], idx[1], idx[2], tin, tout);
            ++k;
        }
        if (tm >= r.te) break;
        if (tm > tin) tin = tm;
        idx[a] += r.w[a] > 0.0 ? 1 : -1;
        if (idx[a] < 0 || idx[a] >= sd.n[a]) break;
        if (r.w[a] > 0.0)
            tmax[a] = (face(sd, a, idx[a] + 1) - r.c[a]) / r.w[a];
        else
            tmax[a] = (face(sd, a, idx[a]) - r.c[a]) / r.w[a];
    }
    return k;
}

// ------------------------------------------------------------ dense walk
//
// A quotient n / w with fixed w, rounded once as the division is, from the
// correctly rounded reciprocal y = 1 / w (Markstein's theorem): q0 = n y is within
// 2 ulp of the quotient; q1 = q0 + (n - w q0) y is within half an ulp and 2^-51 of
// one, so n - w q1 is exact in an FMA and q1 + (n - w q1) y rounds to the rounded
// quotient, unless w's significand lies within 4 ulp of 2 (no quotient is a rounding
// tie, and the correction's error, at most (1/2 + 2^-51) ulp(q) w |y - 1/w|, stays
// below the distance of n / w from the nearest tie for every other w).  Nothing may
// underflow or overflow: quot_exact checks the ray and its grid.  Five operations
// where the division takes eleven, one of them a quarter-rate reciprocal.
__device__ __forceinline__ double quot(double n, double w, double y)
{
    const double q0 = n * y;
    const double q1 = __builtin_fma(__builtin_fma(-w, q0, n), y, q0);
    return __builtin_fma(__builtin_fma(-w, q1, n), y, q1);
}

// x is 0 or 2^lo <= |x| < 2^hi
__device__ __forceinline__ bool exponent_in(double x, int lo, int hi)
{
    const int e = (int)((__builtin_bit_cast(uint64_t, x) >> 52) & 2047u) - 1023;
    return x == 0.0 || (e >= lo && e < hi);
}

// Whether quot() gives every boundary time of the ray along one axis: faces o + i h and
// their distances to c are 0 or of magnitude in [2^-900, 2^900) (sums of multiples of
// 2^-852), w of magnitude in [2^-100, 2^100) with a significand below 2 - 2^-48.
__device__ __forceinline__ bool quot_exact(double o, double h, double c, double w)
{
    if (w == 0.0) return true;   // never divided by
    const uint64_t m = __builtin_bit_cast(uint64_t, w) & ((1ull << 52) - 1);
    return exponent_in(w, -100, 100) && m < (1ull << 52) - 16 && exponent_in(o, -500, 500) &&
           exponent_in(h, -500, 500) && exponent_in(c, -800, 800);
}

// One axis of the walk: the next boundary's time t and number f (boundary f lies at
// o + f h; the voxel index plus one when the ray runs upwards), and its constants.
struct WalkAxis {
    double t, f, s, c, w, y;
    int dl, di;   // steps of the linear voxel id and of the index
    template <bool FAST>
    __device__ __forceinline__ void time(double o, double h)
    {
        const double n = (o + f * h) - c;
        t = FAST ? quot(n, w, y) : n / w;
    }
    template <bool FAST>
    __device__ __forceinline__ void step(double o, double h)
    {
        f += s;
        time<FAST>(o, h);
    }
};

template <bool FAST>
__device__ __forceinline__ WalkAxis walk_axis(const SceneDev& sd, const Ray& r, int a, int idx, int stride)
{
    WalkAxis x;
    const bool up = r.w[a] > 0.0;
    x.w = r.w[a];
    x.c = r.c[a];
    x.y = FAST ? 1.0 / x.w : 0.0;
    x.s = up ? 1.0 : -1.0;
    x.di = up ? 1 : -1;
    x.dl = up ? stride : -stride;
    x.f = (double)(up ? idx + 1 : idx);
    if (x.w != 0.0)
        x.time<FAST>(sd.o[a], sd.h);
    else
        x.t = __builtin_huge_val();
    return x;
}

// walk() on a dense grid: the same voxels, chords and order, with the axes in named
// registers (arrays indexed by the stepped axis were placed in LDS: several dependent
// LDS accesses per step) and quot() for the boundary times.  The walk needs no test of
// the grid's end: the ray's end te is at most the grid exit, which is the smallest of
// the axes' last boundary times (the same expression), so it stops there first; the
// test of the linear id only keeps an index out of range from ever being used.
// emit(k, i, j, kz, lin, t_in, t_out).  5e8 steps (8 VGA frames at 2 cm): the bare walk
// 1.18 ms with walk() and 0.78 (VALU-bound), emit pass 1.89 and 1.82 (with its stores of 4,
// 4 and 1 bytes a step; 1.72 with its bins by quot() too); the metric's walk of 4 frames to
// the grid exit 1.15 and 0.70.
struct WalkState {
    WalkAxis X, Y, Z;
    int i, j, kz, lin, k;   // voxel, its linear id, chords so far
    double tin;
};

template <bool FAST>
__device__ __forceinline__ WalkState walk_start(const SceneDev& sd, const Ray& r)
{
    int idx[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double p = r.c[a] + r.ts * r.w[a];
        double q = floor((p - sd.o[a]) / sd.h);
        if (q < 0.0) q = 0.0;
        if (q > (double)(sd.n[a] - 1)) q = (double)(sd.n[a] - 1);
        idx[a] = (int)q;
    }
    const int nx = sd.n[0], nxy = sd.n[0] * sd.n[1];
    WalkState w;
    w.i = idx[0], w.j = idx[1], w.kz = idx[2];
    w.lin = w.i + nx * w.j + nxy * w.kz;
    w.X = walk_axis<FAST>(sd, r, 0, w.i, 1);
    w.Y = walk_axis<FAST>(sd, r, 1, w.j, nx);
    w.Z = walk_axis<FAST>(sd, r, 2, w.kz, nxy);
    w.tin = r.ts;
    w.k = 0;
    return w;
}

// the chords from a state on (PART: that end by tend); returns their number with those before
template <bool FAST, bool PART, class Emit>
__device__ __forceinline__ int walk_from(const SceneDev& sd, const Ray& r, const WalkState& w, double tend, Emit&& emit)
{
    const uint32_t nvox = (uint32_t)(sd.n[0] * sd.n[1]) * (uint32_t)sd.n[2];
    WalkAxis X = w.X, Y = w.Y, Z = w.Z;
    int i = w.i, j = w.j, kz = w.kz, lin = w.lin, k = w.k;
    const double ox = sd.o[0], oy = sd.o[1], oz = sd.o[2], h = sd.h;
    double tin = w.tin;
    for (;;) {
        const bool ax = X.t <= Y.t && X.t <= Z.t;   // ties step the lowest axis
        const bool ay = !ax && Y.t <= Z.t;
        const double tm = ax ? X.t : ay ? Y.t : Z.t;
        if (PART && tm > tend) break;
        const double tout = fmin(tm, r.te);
        if (tout > tin) {
            emit(k, i, j, kz, lin, tin, tout);
            ++k;
        }
        if (tm >= r.te) break;
        tin = fmax(tin, tm);
        // one branch per axis: lanes that step different axes run them one after the
        // other, still fewer instructions than selecting every operand by axis
        if (ax) {
            lin += X.dl;
            i += X.di;
            X.step<FAST>(ox, h);
        } else if (ay) {
            lin += Y.dl;
            j += Y.di;
            Y.step<FAST>(oy, h);
        } else {
            lin += Z.dl;
            kz += Z.di;
            Z.step<FAST>(oz, h);
        }
        if ((uint32_t)lin >= nvox) break;
    }
    return k;
}

template <bool FAST, class Emit>
__device__ __forceinline__ int walk_dense(const SceneDev& sd, const Ray& r, Emit&& emit)
{
    return walk_from<FAST, false>(sd, r, walk_start<FAST>(sd, r), 0.0, emit);
}

__device__ __forceinline__ bool times_by_quot(const SceneDev& sd, const Ray& r)
{
    bool fast = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) fast = fast && quot_exact(sd.o[a], sd.h, r.c[a], r.w[a]);
    return fast;
}

template <class Emit>
__device__ __forceinline__ int walk_dense(const SceneDev& sd, const Ray& r, Emit&& emit)
{
    if (times_by_quot(sd, r)) return walk_dense<true>(sd, r, emit);
    return walk_dense<false>(sd, r, emit);
}

// The number of voxels walk_dense visits, from the faces crossed along each axis: every
// boundary time in (ts, te) that no other axis shares ends one chord, and te the last.
// Along an axis boundary k has the walk's time of f0 + k s, which does not fall with k, so
// their number is the face position of te, settled by the times next to it.
//
// No two axes may share a time.  With T the times in exact arithmetic, boundary f of axis p
// lies at G = (c + T(f) w - o) / h on axis q's face numbers, and every rounded time within
// 2^-50 M / |w| of T (M bounds the faces and the centre), so a shared time needs G within
// 2^-50 (M_p |w_q / w_p| + M_q) / h of an integer.  G advances by w_q / |w_p| a boundary: its
// fraction is followed in units of 2^-32 (truncated, at most 2^-22 off after 1024
// boundaries) over the axis of fewer faces, and any value within 2^-21 of an integer, for
// which the bound above, the start's own error and the drift add up to less, gives the ray
// to the walk (-1), as do axes of more than 1024 boundaries and grids far from the origin.
// Two integer operations a boundary instead of the walk's 40 FP64 ones: the count pass of
// 8 VGA frames at 2 cm (5e8 voxels) 0.165 ms, 0.83 by walking; of one 64x48 frame 7.7 us
// and 24.
constexpr uint32_t kTieBand = 2048;   // 2^-21
constexpr int kMaxFaces = 1024;

__device__ __forceinline__ bool shares_time(const SceneDev& sd, const Ray& r, int p, int q, const int (&n)[3],
                                            const double (&t0)[3], const double (&y)[3], const double (&mh)[3],
                                            double rh)
{
    const bool sw = n[q] < n[p];
    const int np = sw ? n[q] : n[p];
    if (np <= 0) return false;   // an axis without faces
    const double tp = sw ? t0[q] : t0[p], yp = fabs(sw ? y[q] : y[p]);
    const double wq = sw ? r.w[p] : r.w[q], cq = sw ? r.c[p] : r.c[q], oq = sw ? sd.o[p] : sd.o[q];
    const double a = wq * yp;
    if (!((sw ? mh[q] : mh[p]) * fabs(a) + (sw ? mh[p] : mh[q]) < 0x1p25)) return true;
    const double g = ((cq + tp * wq) - oq) * rh;
    uint32_t x = (uint32_t)((g - floor(g)) * 0x1p32) + kTieBand;
    const uint32_t dx = (uint32_t)((a - floor(a)) * 0x1p32);
    uint32_t least = x;
    for (int k = 0; k < np; k += 8) {   // up to 8 faces too many: at worst a walk for nothing
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            least = min(least, x);
            x += dx;
        }
    }
    return least <= 2 * kTieBand;
}

__device__ int count_dense(const SceneDev& sd, const Ray& r)
{
    int n[3];
    double t0[3], y[3], mh[3];
    const double h = sd.h, rh = 1.0 / h;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double o = sd.o[a], c = r.c[a], w = r.w[a];
        n[a] = 0;
        t0[a] = y[a] = 0.0;
        mh[a] = (fabs(o) + fabs(c)) * rh + (double)(sd.n[a] + 2);
        if (!(mh[a] < 0x1p25)) return -1;
        if (w == 0.0) continue;
        double q = floor((c + r.ts * w - o) / h);   // the walk's first voxel
        if (q < 0.0) q = 0.0;
        if (q > (double)(sd.n[a] - 1)) q = (double)(sd.n[a] - 1);
        const double s = w > 0.0 ? 1.0 : -1.0, f0 = w > 0.0 ? q + 1.0 : q;
        y[a] = 1.0 / w;
        auto time = [&](double f) { return quot((o + f * h) - c, w, y[a]); };
        const double e = ceil((((c + r.te * w) - o) * rh - f0) * s);
        if (!(e <= (double)kMaxFaces)) return -1;
        int m = (int)fmax(e, 0.0);
        if (m > 0 && time(f0 + s * (double)(m - 1)) >= r.te)
            --m;
        else if (time(f0 + s * (double)m) < r.te)
            ++m;
        if (m == 0) continue;
        double f = f0;
        t0[a] = time(f);
        if (t0[a] <= r.ts) {   // on the start
            --m;
            f += s;
            t0[a] = time(f);
            if (t0[a] <= r.ts) return -1;
        }
        n[a] = m;
    }
    if (shares_time(sd, r, 0, 1, n, t0, y, mh, rh) || shares_time(sd, r, 0, 2, n, t0, y, mh, rh) ||
        shares_time(sd, r, 1, 2, n, t0, y, mh, rh))
        return -1;
    return n[0] + n[1] + n[2] + 1;
}

// one axis of a state moved past its faces up to time t
__device__ __forceinline__ void walk_axis_to(const SceneDev& sd, const Ray& r, int a, double t, WalkAxis& x, int& idx,
                                             WalkState& w)
{
    if (x.w == 0.0) return;
    const double o = sd.o[a], h = sd.h, f0 = x.f;
    auto time = [&](double f) { return quot((o + f * h) - x.c, x.w, x.y); };
    // faces passed: as many as lie at or before the ray's position at t, settled by their times
    const double e = floor((((x.c + t * x.w) - o) / h - f0) * x.s) + 1.0;
    int m = (int)fmin(fmax(e, 0.0), (double)kMaxFaces);
    if (m > 0 && time(f0 + x.s * (double)(m - 1)) > t)
        --m;
    else if (time(f0 + x.s * (double)m) <= t)
        ++m;
    if (m == 0) return;
    w.k += x.t <= r.ts ? m - 1 : m;   // a face on the start ends no chord
    w.tin = fmax(w.tin, time(f0 + x.s * (double)(m - 1)));
    w.lin += x.dl * m;
    idx += x.di * m;
    x.f = f0 + x.s * (double)m;
    x.t = time(x.f);
}

// Part `part` of a ray's chords, those that end in its quarter of (ts, te]; every part starts
// from the faces before it.  Rays that count_dense does not count stay whole (part 0).
constexpr int kEmitParts = 4;

template <class Emit>
__device__ __forceinline__ void walk_part(const SceneDev& sd, const Ray& r, int part, Emit&& emit)
{
    auto cut = [&](int p) { return r.ts + (r.te - r.ts) * ((double)p * (1.0 / kEmitParts)); };
    if (!times_by_quot(sd, r) || !(cut(1) > r.ts && cut(kEmitParts - 1) < r.te) || count_dense(sd, r) < 0) {
        if (part == 0) walk_dense(sd, r, emit);
        return;
    }
    WalkState w = walk_start<true>(sd, r);
    if (part > 0) {
        const double t = cut(part);
        walk_axis_to(sd, r, 0, t, w.X, w.i, w);
        walk_axis_to(sd, r, 1, t, w.Y, w.j, w);
        walk_axis_to(sd, r, 2, t, w.Z, w.kz, w);
    }
    walk_from<true, true>(sd, r, w, part < kEmitParts - 1 ? cut(part + 1) : __builtin_huge_val(), emit);
}

// Pixel (u, v) of thread t of block b: 16 x 16 pixels a block, 8 x 8 a wave, so that a
// wave's rays are of like length and cross the same voxels.
__device__ __forceinline__ bool block_pixel(const SceneDev& sd, int b, int t, int& u, int& v)
{
    const int nbx = (sd.W + 15) / 16;
    const int by = b / nbx, bx = b - by * nbx;
    u = bx * 16 + ((t >> 6) & 1) * 8 + (t & 7);
    v = by * 16 + (t >> 7) * 8 + ((t >> 3) & 7);
    return u < sd.W && v < sd.H;
}

// most blocks of 16 x 16 pixels of any scene's image
static int pixel_blocks(const mrf_ctx* c)
{
    int n = 0;
    for (const auto& sd : c->scenes_h) n = std::max(n, ((sd.W + 15) / 16) * ((sd.H + 15) / 16));
    return n;
}

__device__ __forceinline__ const uint8_t* scene_bricks(const BuildDev& bp, const SceneDev& sd)
{
    return bp.bricks ? bp.bricks + sd.brick_off : nullptr;
}

// Sparse grid (Sec. IV-B: bricks are allocated around the reprojected depth
// points): one thread per pixel of one frame (blockIdx.y).  The measured
// surface point c + Z w of a usable measurement marks every brick within
// bp.radius bricks (per axis) of the brick of its voxel; points outside the
// grid mark nothing.  Bytes are only ever set to 1, so the mask does not
// depend on the order of the stores.
__global__ __launch_bounds__(256) void brick_mark_k(const SceneDev* __restrict__ scenes,
                                                    const FrameDev* __restrict__ frames, BuildDev bp,
                                                    uint8_t* __restrict__ bricks)
{
    const FrameDev fr = frames[blockIdx.y];
    const SceneDev& sd = scenes[fr.scene];
    const int pix = blockIdx.x * 256 + threadIdx.x;
    if (pix >= sd.W * sd.H) return;
    const int v = pix / sd.W, u = pix - v * sd.W;
    const double Z = (double)fr.depth[pix];
    if (!isfinite(Z) || Z < bp.z_min || Z > bp.z_max) return;
    const double xn = ((double)u - sd.cx) / sd.fx;
    const double yn = ((double)v - sd.cy) / sd.fy;
    const double* T = fr.T;
    int b[3];
    for (int a = 0; a < 3; ++a) {
        double wa = T[4 * a + 0] * xn;
        wa = wa + T[4 * a + 1] * yn;
        wa = wa + T[4 * a + 2];
        const double pa = T[4 * a + 3] + Z * wa;
        const double q = floor((pa - sd.o[a]) / sd.h);
        if (!(q >= 0.0 && q < (double)sd.n[a])) return;
        b[a] = (int)q / kBrick;
    }
    const int r = bp.radius;
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = max(b[a] - r, 0);
        hi[a] = min(b[a] + r, sd.nb[a] - 1);
    }
    uint8_t* m = bricks + sd.brick_off;
    for (int bk = lo[2]; bk <= hi[2]; ++bk)
        for (int bj = lo[1]; bj <= hi[1]; ++bj)
            for (int bi = lo[0]; bi <= hi[0]; ++bi) m[bi + (int64_t)sd.nb[0] * (bj + (int64_t)sd.nb[1] * bk)] = 1;
}

struct NoEmit {
    __device__ void operator()(int, int, int, int, double, double) const {}
    __device__ void operator()(int, int, int, int, int, double, double) const {}
};

template <bool DENSE>
__global__ __launch_bounds__(256) void trace_count_k(const SceneDev* __restrict__ scenes,
                                                     const FrameDev* __restrict__ frames,
                                                     BuildDev bp, int32_t* __restrict__ counts)
{
    const FrameDev fr = frames[blockIdx.y];
    const SceneDev& sd = scenes[fr.scene];
    int u, v;
    if (!block_pixel(sd, blockIdx.x, threadIdx.x, u, v)) return;
    const int pix = v * sd.W + u;
    Ray r;
    int m = 0;
    if (setup_ray(sd, bp, fr.T, fr.depth[pix], v, u, r)) {
        if constexpr (DENSE) {
            m = times_by_quot(sd, r) ? count_dense(sd, r) : -1;
            if (m < 0) m = walk_dense(sd, r, NoEmit{});
        } else {
            m = walk(sd, r, scene_bricks(bp, sd), NoEmit{}, bp.skip);
        }
    }
    counts[fr.ray_base + pix] = m >= bp.min_vox ? m : 0;
}

// brick-major key of voxel (i, j, k) of a scene
__device__ __forceinline__ uint32_t brick_key(const SceneDev& sd, int i, int j, int k)
{
    const int64_t brick = ((int64_t)(k >> 3) * sd.nb[1] + (j >> 3)) * sd.nb[0] + (i >> 3);
    return (uint32_t)(sd.key_base + brick * 512 + ((k & 7) * 8 + (j & 7)) * 8 + (i & 7));
}

template <bool KEY>
struct EdgeEmit {
    int32_t* col;
    uint32_t* key;
    float* delta;
    uint8_t* bin;
    double* tin;
    double* tout;
    float* wlen;          // chord length per edge (per-keyframe averaging), or null
    const SceneDev* sd;
    int64_t base;
    int32_t vbase;
    double Z, dbin;
    double wn;            // |w| of the ray: chord length = (t_out - t_in) |w|
    double rbin;          // 1 / dbin, correctly rounded
    bool by_quot;         // quot() gives d / dbin
    // The bin is floor(d / dbin) with the quotient rounded once, as in the oracle: by
    // quot(), seven operations with the clamp below (a quotient of 128 and one of more are
    // the last bin alike; chord midpoints are not negative).  Where that is not exact the
    // division is behind a barrier that keeps the compiler from forming it on every step,
    // which took 25.  Emit pass of 8 VGA frames at 2 cm 1.83 -> 1.72 ms, of one at 4 cm 92
    // -> 87 us.
    __device__ int bin_of(double d) const
    {
        d = fmin(d, 128.0 * dbin);
        double q = quot(d, dbin, rbin);
        if (!by_quot) {
            asm volatile("");
            q = d / dbin;
        }
        return min(max((int)q, 0), 63);
    }
    __device__ void operator()(int k, int vi, int vj, int vk, double ti, double to) const
    {
        (*this)(k, vi, vj, vk, vi + sd->n[0] * (vj + sd->n[1] * vk), ti, to);
    }
    __device__ void operator()(int k, int vi, int vj, int vk, int lin, double ti, double to) const
    {
        const int64_t e = base + (int64_t)kTile * k;   // step k of this ray's tile lane
        const double d = (ti + to) * 0.5;   // voxel depth: chord midpoint
        col[e] = vbase + lin;
        if constexpr (KEY) key[e] = brick_key(*sd, vi, vj, vk);
        delta[e] = (float)(Z - d);
        bin[e] = (uint8_t)bin_of(d);
        if (tin) {
            tin[e] = ti;
            tout[e] = to;
        }
        if (wlen) wlen[e] = (float)((to - ti) * wn);
    }
};

// Threads are grouped by tile: the 16 lanes 16t..16t+15 of a block trace the 16 pixels
// of tile t, so at every traversal step they write one whole 64-byte line of each
// per-slot array (a row-major pixel order would write 16-byte pieces of 16 lines).
// Each lane then marks its column's slots past its ray, up to the tile's length, as
// padding (no voxel, no bin, sort key pad_key past every voxel); lanes of pixels
// outside the image pad their whole column.  Sort keys are written where the
// slots themselves are sorted (KEY).
template <bool DENSE, bool KEY, int PARTS>
__global__ __launch_bounds__(256) void trace_emit_k(const SceneDev* __restrict__ scenes,
                                                    const FrameDev* __restrict__ frames, BuildDev bp,
                                                    const int32_t* __restrict__ counts,
                                                    const int64_t* __restrict__ tbase,
                                                    const TileDev* __restrict__ tiles, uint32_t pad_key,
                                                    int32_t* col, uint32_t* key, float* delta, uint8_t* bin,
                                                    double* tin, double* tout, float* wlen)
{
    const FrameDev fr = frames[blockIdx.y];
    const SceneDev& sd = scenes[fr.scene];
    const int nty = (sd.H + kTileW - 1) / kTileW;
    // PARTS > 1: wave w of a block takes part w of the rays of its four tiles
    const int th = PARTS > 1 ? threadIdx.x & 63 : threadIdx.x, part = PARTS > 1 ? threadIdx.x >> 6 : 0;
    const int lt = blockIdx.x * (256 / PARTS / kTile) + th / kTile;
    if (lt >= fr.ntx * nty) return;
    const int ty = lt / fr.ntx, tx = lt - ty * fr.ntx;
    const int q = th % kTile;
    const int v = ty * kTileW + q / kTileW, u = tx * kTileW + q % kTileW;
    const int64_t t = fr.tile_base + lt;
    const int64_t slot0 = tbase[t] + q;
    const int len = tiles[t].len;
    int m = 0;
    if (v < sd.H && u < sd.W) {
        const int pix = v * sd.W + u;
        m = counts[fr.ray_base + pix];
        if (m > 0) {
            Ray ray;
            setup_ray(sd, bp, fr.T, fr.depth[pix], v, u, ray);
            double wn = ray.w[0] * ray.w[0];
            wn = wn + ray.w[1] * ray.w[1];
            wn = wn + ray.w[2] * ray.w[2];
            const double dbin = bp.dmax / 64.0;
            EdgeEmit<KEY> em{col,   key,   delta, bin, tin, tout, wlen, &sd, slot0, (int32_t)sd.voxel_base, ray.Z,
                        dbin,  sqrt(wn), 1.0 / dbin, dbin > 0.0 && quot_exact(0.0, 0.0, 0.0, dbin)};
            if constexpr (PARTS > 1)
                walk_part(sd, ray, part, em);
            else if constexpr (DENSE)
                walk_dense(sd, ray, em);
            else
                walk(sd, ray, scene_bricks(bp, sd), em, bp.skip);
        }
    }
    for (int k = m + part; k < len; k += PARTS) {
        const int64_t e = slot0 + (int64_t)kTile * k;
        col[e] = -1;
        if constexpr (KEY) key[e] = pad_key;
        delta[e] = 0.0f;
        bin[e] = 255;
    }
}

// tile lt of frame f: its rays, extent inside the image and longest ray
__device__ __forceinline__ TileDev tile_of(const SceneDev& sd, const FrameDev& fr, int f, int lt,
                                           const int32_t* __restrict__ counts)
{
    const int ty = lt / fr.ntx, tx = lt - ty * fr.ntx;
    TileDev td;
    td.ray0 = (int32_t)(fr.ray_base + (int64_t)(ty * kTileW) * sd.W + tx * kTileW);
    td.W = sd.W;
    td.nu = min(kTileW, sd.W - tx * kTileW);
    td.nv = min(kTileW, sd.H - ty * kTileW);
    int len = 0;
    for (int a = 0; a < td.nv; ++a)
        for (int b = 0; b < td.nu; ++b) len = max(len, counts[td.ray0 + a * sd.W + b]);
    td.len = len;
    td.base = 0;
    td.frame = f;
    return td;
}

// one thread per tile
__global__ void tile_init_k(const SceneDev* __restrict__ scenes, const FrameDev* __restrict__ frames, int f0,
                            const int32_t* __restrict__ counts, TileDev* __restrict__ tiles,
                            int32_t* __restrict__ slots16, int64_t t0)
{
    const FrameDev fr = frames[f0 + blockIdx.y];
    const SceneDev& sd = scenes[fr.scene];
    const int nty = (sd.H + kTileW - 1) / kTileW;
    const int lt = blockIdx.x * blockDim.x + threadIdx.x;
    if (lt >= fr.ntx * nty) return;
    const TileDev td = tile_of(sd, fr, f0 + (int)blockIdx.y, lt, counts);
    tiles[fr.tile_base + lt] = td;
    slots16[fr.tile_base + lt - t0] = kTile * td.len;
}

__global__ void tile_base_k(TileDev* __restrict__ tiles, const int64_t* __restrict__ tbase, int64_t T)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) tiles[t].base = tbase[t];
}

__global__ void fill_u32_k(uint32_t* __restrict__ p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_brick_mask(mrf_ctx* c, hipStream_t s)
{
    hipError_t e = launch_fill_u32((uint32_t*)c->b_bricks.p, 0u, (c->n_bricks + 3) / 4, s);
    if (e != hipSuccess) return e;
    dim3 grid((c->max_hw + 255) / 256, c->n_frames);
    hipLaunchKernelGGL(brick_mark_k, grid, dim3(256), 0, s, (const SceneDev*)c->b_scenes.p,
                       (const FrameDev*)c->b_frames.p, c->bp, (uint8_t*)c->b_bricks.p);
    return hipGetLastError();
}

hipError_t launch_trace_count(mrf_ctx* c, hipStream_t s, int f0, int nf)
{
    if (nf < 0) nf = c->n_frames - f0;
    if (nf <= 0) return hipSuccess;
    const dim3 grid(pixel_blocks(c), nf);
    const SceneDev* sc = (const SceneDev*)c->b_scenes.p;
    const FrameDev* fr = (const FrameDev*)c->b_frames.p + f0;
    int32_t* counts = (int32_t*)c->b_counts.p;
    if (c->bp.bricks)
        hipLaunchKernelGGL(trace_count_k<false>, grid, dim3(256), 0, s, sc, fr, c->bp, counts);
    else
        hipLaunchKernelGGL(trace_count_k<true>, grid, dim3(256), 0, s, sc, fr, c->bp, counts);
    return hipGetLastError();
}

hipError_t launch_tiles(mrf_ctx* c, int32_t* slots16, hipStream_t s, int f0, int nf)
{
    if (nf < 0) nf = c->n_frames - f0;
    if (nf <= 0) return hipSuccess;
    int max_tiles = 0;
    for (const auto& sd : c->scenes_h)
        max_tiles = std::max(max_tiles, ((sd.W + kTileW - 1) / kTileW) * ((sd.H + kTileW - 1) / kTileW));
    dim3 grid((max_tiles + 255) / 256, nf);
    hipLaunchKernelGGL(tile_init_k, grid, dim3(256), 0, s, (const SceneDev*)c->b_scenes.p,
                       (const FrameDev*)c->b_frames.p, f0, (const int32_t*)c->b_counts.p, (TileDev*)c->b_tiles.p,
                       slots16, c->frames_h[f0].tile_base);
    return hipGetLastError();
}

hipError_t launch_tile_bases(mrf_ctx* c, hipStream_t s, int64_t t0)
{
    if (c->T > t0)
        hipLaunchKernelGGL(tile_base_k, dim3((unsigned)((c->T - t0 + 255) / 256)), dim3(256), 0, s,
                           (TileDev*)c->b_tiles.p + t0, (const int64_t*)c->b_tbase.p + t0, c->T - t0);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(fill_u32_k, dim3((unsigned)b), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

__global__ void scatter_by_slot_k(const uint32_t* __restrict__ slot, const float* __restrict__ in, int64_t n,
                                  float* __restrict__ out)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        out[slot[j]] = in[j];
}

hipError_t launch_scatter_by_slot(const uint32_t* slot, const float* in, int64_t n, float* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(scatter_by_slot_k, dim3((unsigned)b), dim3(256), 0, s, slot, in, n, out);
    return hipGetLastError();
}

template <bool DENSE, bool KEY, int PARTS>
static void launch_emit_t(mrf_ctx* c, hipStream_t s, int f0, int nf)
{
    constexpr int per = 256 / PARTS / kTile;   // tiles of a block
    const dim3 grid((unsigned)((c->max_tpf + per - 1) / per), nf);
    hipLaunchKernelGGL((trace_emit_k<DENSE, KEY, PARTS>), grid, dim3(256), 0, s, (const SceneDev*)c->b_scenes.p,
                       (const FrameDev*)c->b_frames.p + f0, c->bp, (const int32_t*)c->b_counts.p,
                       (const int64_t*)c->b_tbase.p, (const TileDev*)c->b_tiles.p, (uint32_t)c->Vk,
                       (int32_t*)c->b_col.p, (uint32_t*)c->b_g.p, (float*)c->b_delta.p, (uint8_t*)c->b_bin.p,
                       c->keep_chords ? (double*)c->b_tin.p : nullptr,
                       c->keep_chords ? (double*)c->b_tout.p : nullptr, c->kf ? (float*)c->b_kflen.p : nullptr);
}

// Whether rays are walked in parts: where they are few, the pass lasts as long as its longest
// chain of steps, and a part's is a quarter; many fill the chip by themselves, and the parts'
// starts are added work.  Build in us, whole and in parts: 16 tiles 165 and 156, 192 (64x48)
// 218 and 192, 1200 282 and 270, 4800 (320x240) 418 and 411; 14400 504 and 511, 19200 (VGA)
// 510 and 535; the emit pass of 8 VGA frames at 2 cm 1.84 ms and 1.95 (in other scenes of
// that size the build is 5% faster in parts).
static bool emit_in_parts(int64_t tiles) { return tiles <= 8192; }

hipError_t launch_trace_emit(mrf_ctx* c, bool keys, hipStream_t s, int f0, int nf)
{
    if (nf < 0) nf = c->n_frames - f0;
    if (nf <= 0) return hipSuccess;
    const bool split = emit_in_parts((int64_t)c->max_tpf * nf);
    if (c->bp.bricks)
        keys ? launch_emit_t<false, true, 1>(c, s, f0, nf) : launch_emit_t<false, false, 1>(c, s, f0, nf);
    else if (split)
        keys ? launch_emit_t<true, true, kEmitParts>(c, s, f0, nf) : launch_emit_t<true, false, kEmitParts>(c, s, f0, nf);
    else
        keys ? launch_emit_t<true, true, 1>(c, s, f0, nf) : launch_emit_t<true, false, 1>(c, s, f0, nf);
    return hipGetLastError();
}

// ============================================================== scans

constexpr int SC_T = 256, SC_IPT = 8, SC_TILE = SC_T * SC_IPT;

struct LoadI32 {
    const int32_t* p;
    __device__ int64_t operator()(int64_t i) const { return p[i]; }
};
struct LoadI64 {
    const int64_t* p;
    __device__ int64_t operator()(int64_t i) const { return p[i]; }
};

__device__ int64_t block_excl_scan_i64(int64_t x, int64_t* total)
{
    __shared__ int64_t wsum[SC_T / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int64_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int64_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < SC_T / 64; ++i) {
        if (i < w) off += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + incl - x;
}

template <class Load>
__global__ __launch_bounds__(SC_T) void scan_reduce_k(Load ld, int64_t n, int64_t* __restrict__ bsum)
{
    const int64_t base = (int64_t)blockIdx.x * SC_TILE;
    int64_t acc = 0;
#pragma unroll
    for (int k = 0; k < SC_IPT; ++k) {
        const int64_t i = base + k * SC_T + threadIdx.x;
        if (i < n) acc += ld(i);
    }
    int64_t tot;
    block_excl_scan_i64(acc, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

template <class Load, class Out>
__global__ __launch_bounds__(SC_T) void scan_apply_k(Load ld, int64_t n, const int64_t* __restrict__ boff,
                                                     Out* __restrict__ out)
{
    const int64_t base = (int64_t)blockIdx.x * SC_TILE + (int64_t)threadIdx.x * SC_IPT;
    int64_t v[SC_IPT];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SC_IPT; ++k) {
        const int64_t i = base + k;
        v[k] = i < n ? ld(i) : 0;
        s += v[k];
    }
    int64_t tot;
    int64_t ex = block_excl_scan_i64(s, &tot) + (boff ? boff[blockIdx.x] : 0);
#pragma unroll
    for (int k = 0; k < SC_IPT; ++k) {
        const int64_t i = base + k;
        if (i < n) out[i] = (Out)ex;
        ex += v[k];
        if (i == n - 1) out[n] = (Out)ex;
    }
}

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

size_t scan_tmp_bytes(int64_t n)
{
    size_t words = 0;
    int64_t m = n;
    while (cdiv(m, SC_TILE) > 1) {
        const int64_t nb = cdiv(m, SC_TILE);
        words += 2 * nb + 1;
        m = nb;
    }
    return (words + 8) * sizeof(int64_t);
}

template <class Out>
__global__ void zero_k(Out* p) { *p = 0; }

// Exclusive scan of ld(0..n-1) into out[0..n] (out[n] = the total), written as
// Out (the caller guarantees the total fits); tmp holds scan_tmp_bytes(n).
template <class Load, class Out = int64_t>
static hipError_t scan_rec(Load ld, int64_t n, Out* out, int64_t* tmp, hipStream_t s)
{
    if (n == 0) {
        hipLaunchKernelGGL(zero_k<Out>, dim3(1), dim3(1), 0, s, out);
        return hipGetLastError();
    }
    const int64_t nb = cdiv(n, SC_TILE);
    if (nb == 1) {
        hipLaunchKernelGGL((scan_apply_k<Load, Out>), dim3(1), dim3(SC_T), 0, s, ld, n, (const int64_t*)nullptr,
                           out);
        return hipGetLastError();
    }
    int64_t* bsum = tmp;
    int64_t* boff = tmp + nb;
    hipLaunchKernelGGL(scan_reduce_k<Load>, dim3((unsigned)nb), dim3(SC_T), 0, s, ld, n, bsum);
    hipError_t e = scan_rec(LoadI64{bsum}, nb, boff, tmp + 2 * nb + 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((scan_apply_k<Load, Out>), dim3((unsigned)nb), dim3(SC_T), 0, s, ld, n, (const int64_t*)boff,
                       out);
    return hipGetLastError();
}

hipError_t scan_exclusive_i32(const int32_t* in, int64_t* out, int64_t n, void* tmp, size_t tmp_bytes,
                              hipStream_t s)
{
    if (tmp_bytes < scan_tmp_bytes(n)) return hipErrorInvalidValue;
    return scan_rec(LoadI32{in}, n, out, (int64_t*)tmp, s);
}

// ============================================================== radix sort

#ifndef MRF_RS_T
#define MRF_RS_T 256
#define MRF_RS_IPT 16
#endif
constexpr int RS_T = MRF_RS_T, RS_IPT = MRF_RS_IPT, RS_TILE = RS_T * RS_IPT;
static_assert(RS_T == 256 && RS_IPT % 4 == 0, "radix tile shape: one thread per digit");

// Tiles per chunk of the digit-offset scan: each chunk is a serial walk of its tiles,
// so short chunks keep more blocks busy (one VGA frame's 4e6 runs, 1000 tiles: chunks of
// 256 took 39 us per pass, of 32 take 9).
constexpr int RS_CB = 32;

size_t radix_hist_entries(int64_t n) { return (size_t)256 * (size_t)cdiv(n > 0 ? n : 1, RS_TILE); }

size_t radix_tmp_bytes(int64_t n)
{
    const int64_t nch = cdiv(cdiv(n > 0 ? n : 1, RS_TILE), RS_CB);
    return sizeof(int64_t) * (size_t)(2 * 256 * nch + 256);
}

// Lanes of a wave holding digit d (of valid items): 8 ballots.  Per bit, with
// s the bit sign-extended (all ones when set, 0 when clear) and m the lanes
// whose bit is set, the lanes that agree with this lane are ~(m ^ s); each
// 32-bit half is updated with one three-input bit operation, p & ~(m ^ s)
// (truth table 0x90 over (p, m, s)), instead of a select of the 64-bit mask.
__device__ __forceinline__ uint64_t rs_peers(int d, bool valid)
{
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t sb = (uint32_t)((int32_t)((uint32_t)d << (31 - b)) >> 31);   // 0 or all ones
        const uint64_t m = __ballot(sb != 0u);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, sb, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), sb, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Digit counts of one tile of RS_TILE keys.  Thread t takes RS_IPT
// consecutive keys (vector loads) and adds each run of equal digits with one
// LDS atomic: keys in slot order come in runs (the rays of a tile cross the
// same voxels at the same step), which would otherwise serialise the atomics
// of a wave on a few addresses.  RS_TILE is a multiple of 16 and n of 4 is
// not assumed: the tile's tail is read key by key.
__global__ __launch_bounds__(RS_T) void rs_hist_k(const uint32_t* __restrict__ keys, int64_t n, int shift,
                                                  int32_t* __restrict__ hist, int64_t nblocks)
{
    __shared__ int32_t h[256];
    h[threadIdx.x] = 0;
    const int64_t i0 = (int64_t)blockIdx.x * RS_TILE + (int64_t)threadIdx.x * RS_IPT;
    uint32_t kr[RS_IPT];
    if (i0 + RS_IPT <= n) {
        const uint4* p = (const uint4*)(keys + i0);   // keys and RS_IPT * 4 bytes: 16-byte aligned
#pragma unroll
        for (int q = 0; q < RS_IPT / 4; ++q) {
            const uint4 w = p[q];
            kr[4 * q] = w.x;
            kr[4 * q + 1] = w.y;
            kr[4 * q + 2] = w.z;
            kr[4 * q + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < RS_IPT; ++j) kr[j] = i0 + j < n ? keys[i0 + j] : 0u;
    }
    const int nv = (int)(n - i0 < RS_IPT ? (n - i0 > 0 ? n - i0 : 0) : RS_IPT);
    __syncthreads();
    if (nv > 0) {
        int cur = (kr[0] >> shift) & 255, cnt = 1;
#pragma unroll
        for (int j = 1; j < RS_IPT; ++j) {
            const int d = (kr[j] >> shift) & 255;
            if (j < nv) {
                if (d == cur) {
                    ++cnt;
                } else {
                    atomicAdd(&h[cur], cnt);
                    cur = d;
                    cnt = 1;
                }
            }
        }
        atomicAdd(&h[cur], cnt);
    }
    __syncthreads();
    hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// Digit offsets from the tile-major (tile, digit) counts, of few tiles by the scatter's
// blocks themselves, else in three steps: per-chunk column sums (coalesced rows), an exclusive scan of each digit's
// chunk sums (one block per digit), and per-tile running sums inside each
// chunk on top of the digit's base (the exclusive scan of the digit totals).
__global__ __launch_bounds__(256) void rs_colsum_k(const int32_t* __restrict__ hist, int64_t nb,
                                                   int64_t* __restrict__ csum)
{
    const int64_t b0 = (int64_t)blockIdx.x * RS_CB;
    const int64_t b1 = b0 + RS_CB < nb ? b0 + RS_CB : nb;
    int64_t acc = 0;
#pragma unroll 8
    for (int64_t b = b0; b < b1; ++b) acc += hist[b * 256 + threadIdx.x];
    csum[(int64_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

// block d: coff[c][d] = items of digit d in chunks < c; dtot[d] = all of them
__global__ __launch_bounds__(256) void rs_colscan_k(const int64_t* __restrict__ csum, int64_t nch,
                                                    int64_t* __restrict__ coff, int64_t* __restrict__ dtot)
{
    const int d = blockIdx.x;
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < nch; c0 += 256) {
        const int64_t c = c0 + threadIdx.x;
        const int64_t x = c < nch ? csum[c * 256 + d] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan_i64(x, &tot);
        if (c < nch) coff[c * 256 + d] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) dtot[d] = carry;
}

// offs[b][d]: output position of tile b's first item of digit d
__global__ __launch_bounds__(256) void rs_offsets_k(const int32_t* __restrict__ hist, int64_t nb,
                                                    const int64_t* __restrict__ coff,
                                                    const int64_t* __restrict__ dtot, int64_t* __restrict__ offs)
{
    const int64_t b0 = (int64_t)blockIdx.x * RS_CB;
    const int64_t b1 = b0 + RS_CB < nb ? b0 + RS_CB : nb;
    int64_t total;
    const int64_t base = block_excl_scan_i64(dtot[threadIdx.x], &total);
    int64_t run = base + coff[(int64_t)blockIdx.x * 256 + threadIdx.x];
    for (int64_t b = b0; b < b1; ++b) {
        offs[b * 256 + threadIdx.x] = run;
        run += hist[b * 256 + threadIdx.x];
    }
}

// Stable scatter of one tile of RS_TILE items.  Wave w owns items
// [w RS_IPT 64, (w + 1) RS_IPT 64) of the tile, RS_IPT rounds of 64; equal
// digits inside a round are matched with wave ballots.  A first walk counts
// each wave's digits, the per-wave bases follow in digit-major, wave-minor
// order (index order, hence stable), and a second walk places every item in
// an LDS copy of the tile grouped by digit: two barriers in all.  The copy is
// then written out as contiguous runs, one per digit, at the digit's global
// offset for this tile (coalesced stores in place of scattered words).  Tile
// t's run of a digit ends where tile t+1's begins, so consecutive tiles run on
// one XCD (block remap) and their shared lines merge in its L2.  hist
// and offs hold the tile's digit counts and output offsets (tile-major rows
// of 256); offs null: every block adds up the counts of all tiles.  MASK: items carry a second value of 16 bits.
template <bool MASK>
__global__ __launch_bounds__(RS_T) void rs_scatter_k(const uint32_t* __restrict__ keys_in,
                                                     const uint32_t* __restrict__ vals_in, int64_t n,
                                                     int shift, const int32_t* __restrict__ hist,
                                                     const int64_t* __restrict__ offs,
                                                     uint32_t* __restrict__ keys_out,
                                                     uint32_t* __restrict__ vals_out, const SlotGroups groups,
                                                     const uint16_t* __restrict__ masks_in,
                                                     uint16_t* __restrict__ masks_out)
{
    constexpr int NW = RS_T / 64;
    constexpr int WI = RS_IPT * 64;   // items per wave
    __shared__ uint32_t lk[RS_TILE];
    __shared__ uint32_t lv[RS_TILE];
    __shared__ uint16_t lm[MASK ? RS_TILE : 1];
    __shared__ int64_t boff[256];
    __shared__ int32_t dstart[256];
    __shared__ int32_t wcnt[NW][256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform across the wave
    const int64_t tile = xcd_block(blockIdx.x, gridDim.x);   // neighbouring tiles on one XCD
    const int64_t start = tile * RS_TILE;
    const int64_t wstart = start + (int64_t)w * WI;
    // items of this wave below n: item r * 64 + lane is valid iff it is < nvw
    const int64_t rem = n - wstart;
    const int nvw = rem <= 0 ? 0 : (rem < WI ? (int)rem : WI);
    uint32_t kr[RS_IPT], vr[RS_IPT];
    uint16_t mr[MASK ? RS_IPT : 1];
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const int64_t i = wstart + r * 64 + lane;
        const int64_t ic = i < n ? i : n - 1;
        kr[r] = keys_in[ic];
        if (MASK || vals_in) vr[r] = vals_in[ic];
        if constexpr (MASK) mr[r] = masks_in[ic];
    }
    if (!MASK && !vals_in) {   // first pass: the values are the slots, relative to their group's first slot
        if (groups.n > 1) {
#pragma unroll
            for (int r = 0; r < RS_IPT; ++r) {
                const int64_t i = wstart + r * 64 + lane;
                vr[r] = (uint32_t)(i - group_slot_base_of_slot(groups, i));
            }
        } else {
#pragma unroll
            for (int r = 0; r < RS_IPT; ++r) vr[r] = (uint32_t)(wstart + r * 64 + lane);
        }
    }
    int64_t o0;
    if (offs) {
        o0 = offs[tile * 256 + tid];
    } else {
        int before = 0, all = 0;   // the thread's digit in the tiles before this one, and in all
        const int nb = (int)gridDim.x;
#pragma unroll 16
        for (int b = 0; b < nb; ++b) {
            const int x = hist[(int64_t)b * 256 + tid];
            before += b < tile ? x : 0;
            all += x;
        }
        int64_t total;
        o0 = block_excl_scan_i64(all, &total) + before;
    }
    const int64_t cnt = hist[tile * 256 + tid];
    boff[tid] = o0;
#pragma unroll
    for (int q = 0; q < NW; ++q) wcnt[q][tid] = 0;
    int64_t total;
    dstart[tid] = (int32_t)block_excl_scan_i64(cnt, &total);   // synchronises the block
    const uint64_t below = lane ? ((~0ull) >> (64 - lane)) : 0ull;
    // walk 1: digit counts of this wave (the lowest lane of each digit adds;
    // the digits of one round are distinct, so no two lanes share an address).
    // Each item keeps its rank among equal digits of its round and their
    // count, packed as rank | count << 8 (both <= 64).
    int rc[RS_IPT];
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const bool valid = r * 64 + lane < nvw;
        const int d = (kr[r] >> shift) & 255;
        const uint64_t peers = rs_peers(d, valid);
        const int rank = __popcll(peers & below), num = __popcll(peers);
        rc[r] = rank | (num << 8);
        if (valid && rank == 0) wcnt[w][d] += num;
    }
    __syncthreads();
    {   // thread = digit: wave bases inside the tile's LDS copy
        int acc = dstart[tid];
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int t = wcnt[q][tid];
            wcnt[q][tid] = acc;
            acc += t;
        }
    }
    __syncthreads();
    // walk 2: place the items; a round's lanes read their digit's base before
    // the lowest lane of each digit advances it (LDS operations of a wave
    // complete in order)
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const bool valid = r * 64 + lane < nvw;
        const int d = (kr[r] >> shift) & 255;
        const int rank = rc[r] & 255;
        const int b = wcnt[w][d];
        if (valid) {
            lk[b + rank] = kr[r];
            lv[b + rank] = vr[r];
            if constexpr (MASK) lm[b + rank] = mr[r];
        }
        if (valid && rank == 0) wcnt[w][d] = b + (rc[r] >> 8);
    }
    __syncthreads();
    const int tn = (int)(n - start < RS_TILE ? n - start : RS_TILE);
    for (int j = tid; j < tn; j += RS_T) {
        const uint32_t key = lk[j];
        const int d = (key >> shift) & 255;
        const int64_t pos = boff[d] + (j - dstart[d]);
        keys_out[pos] = key;
        vals_out[pos] = lv[j];
        if constexpr (MASK) masks_out[pos] = lm[j];
    }
}

// n sort passes from keys / vals (/ masks) A into B, B into A, ...; tables: hist and
// offs (radix_hist_entries(n)), tmp (radix_tmp_bytes(n)).
struct RadixTables {
    int32_t* hist;
    int64_t* offs;
    int64_t* tmp;
};

// Most tiles whose offsets the scatter's blocks add up themselves: the three kernels
// between the counts and the scatter take 13 us whatever the size, a block's pass over the
// counts grows with the tiles.  Build of a frame of 1.2e5 slots (31 tiles) 226 us, 251 with
// the three kernels; of 6.2e5 (152 tiles) 247 and 258; of 9.1e5 (222 tiles) 252 and 257.
// 256 tiles hold the 2^20 slots that are sorted one by one.
constexpr int64_t kRsFewTiles = 256;

template <bool MASK>
static hipError_t radix_pass(const uint32_t* sk, const uint32_t* sv, const uint16_t* sm, uint32_t* dk, uint32_t* dv,
                             uint16_t* dm, int64_t n, int shift, const RadixTables& t, const SlotGroups& groups,
                             hipStream_t s)
{
    if ((uintptr_t)sk % 16 != 0) return hipErrorInvalidValue;   // rs_hist_k's 16-byte loads
    const int64_t nb = cdiv(n, RS_TILE);
    const int64_t nch = cdiv(nb, RS_CB);
    int64_t* csum = t.tmp;
    int64_t* coff = csum + 256 * nch;
    int64_t* dtot = coff + 256 * nch;
    const bool few = nb <= kRsFewTiles;
    hipLaunchKernelGGL(rs_hist_k, dim3((unsigned)nb), dim3(RS_T), 0, s, sk, n, shift, t.hist, nb);
    if (!few) {
        hipLaunchKernelGGL(rs_colsum_k, dim3((unsigned)nch), dim3(256), 0, s, (const int32_t*)t.hist, nb, csum);
        hipLaunchKernelGGL(rs_colscan_k, dim3(256), dim3(256), 0, s, (const int64_t*)csum, nch, coff, dtot);
        hipLaunchKernelGGL(rs_offsets_k, dim3((unsigned)nch), dim3(256), 0, s, (const int32_t*)t.hist, nb,
                           (const int64_t*)coff, (const int64_t*)dtot, t.offs);
    }
    hipLaunchKernelGGL(rs_scatter_k<MASK>, dim3((unsigned)nb), dim3(RS_T), 0, s, sk, sv, n, shift,
                       (const int32_t*)t.hist, few ? nullptr : (const int64_t*)t.offs, dk, dv, groups, sm, dm);
    return hipGetLastError();
}

hipError_t radix_sort_pairs(const uint32_t* keys_in, uint32_t* keys_a, uint32_t* vals_a, uint32_t* keys_b,
                            uint32_t* vals_b, uint32_t* keys_out, uint32_t* vals_out, int64_t n,
                            int key_bits, int32_t* hist, int64_t* offs, void* tmp, size_t tmp_bytes,
                            hipStream_t s, const SlotGroups& groups)
{
    if (n == 0) return hipSuccess;
    const int passes = key_bits <= 8 ? 1 : (key_bits + 7) / 8;
    if (tmp_bytes < radix_tmp_bytes(n)) return hipErrorInvalidValue;
    const RadixTables t{hist, offs, (int64_t*)tmp};
    const uint32_t* sk = keys_in;
    const uint32_t* sv = nullptr;
    for (int p = 0; p < passes; ++p) {
        uint32_t* dk = (p == passes - 1) ? keys_out : ((p & 1) ? keys_b : keys_a);
        uint32_t* dv = (p == passes - 1) ? vals_out : ((p & 1) ? vals_b : vals_a);
        const hipError_t e = radix_pass<false>(sk, sv, nullptr, dk, dv, nullptr, n, 8 * p, t, groups, s);
        if (e != hipSuccess) return e;
        sk = dk;
        sv = dv;
    }
    return hipSuccess;
}

// ------------------------------------------------------------ runs
//
// The 16 rays of a tile cross the same few voxels at a step: a row of 16 slots
// holds few different voxels (1.4 on average for VGA at 5 cm, 1.7 at 2 cm, 5 for 64x48 at
// 5 cm).  Sorting one item per (row, voxel) -- a run:
// its key, row and the 16-bit mask of its lanes -- instead of one per slot, and
// writing the runs out as list entries afterwards, gives the same lists: a
// (row, voxel) pair is one run, so runs of a voxel in row order, lanes
// ascending inside, are its slots in order.  Padding slots make no run.
// Three passes over 5.2e8 slots (8 VGA frames at 2 cm) took 7.6 ms of HBM-bound
// sorting; finding, packing, sorting and expanding their runs takes 4.8.

constexpr int kRunRows = 256;                   // rows per block of runs_find_k, 64 per wave
constexpr int kRunSlots = kTile * kRunRows;

// The scene whose voxels, or keys (BASE: its first), hold id x: the last with BASE <= x.  By
// halves, since a batch may hold thousands of scenes (2500 of 16x12 pixels: build 1.02 ms, 11.5 with
// a walk along them for every run).
template <int64_t SceneDev::*BASE>
__device__ __forceinline__ const SceneDev& scene_of(const SceneDev* __restrict__ scenes, int ns, int64_t x)
{
    int lo = 0, hi = ns;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (scenes[mid].*BASE <= x)
            lo = mid;
        else
            hi = mid;
    }
    return scenes[lo];
}

__device__ __forceinline__ uint32_t voxel_key32(const SceneDev* __restrict__ scenes, int ns, uint32_t v)
{
    const SceneDev& sd = scene_of<&SceneDev::voxel_base>(scenes, ns, v);
    const uint32_t local = v - (uint32_t)sd.voxel_base;
    const uint32_t nx = (uint32_t)sd.n[0], nxy = nx * (uint32_t)sd.n[1];
    const uint32_t k = local / nxy, rem = local - k * nxy;
    const uint32_t j = rem / nx, i = rem - j * nx;
    const uint32_t brick = ((k >> 3) * (uint32_t)sd.nb[1] + (j >> 3)) * (uint32_t)sd.nb[0] + (i >> 3);
    return (uint32_t)sd.key_base + brick * 512u + ((k & 7) * 8 + (j & 7)) * 8 + (i & 7);
}

// lanes (of four rows) that hold the value of a lower lane of their row; x not 0 in the
// lanes that matter (a lane without a lane J below it compares with 0)
template <int... J>
__device__ __forceinline__ uint64_t row_repeats(uint32_t x, std::integer_sequence<int, J...>)
{
    return (__ballot(x == (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111 + J, 0xF, 0xF, true)) | ...);   // row_shr
}

// The runs of kRunRows rows, in row order, at [block * kRunSlots, + bcnt[block])
// of gkey / ginfo (lane mask | row of the block << 16).  VALU-bound if every lane
// forms its mask (15 comparisons and bits, 104 instructions per 64 slots: 1.32 ms for
// 5.2e8 slots, 2.5 GB of traffic).  So the lanes only learn whether a lower one holds
// their voxel (the comparisons' lane masks are joined by scalar operations); masks, from
// the row's values in LDS, and keys are formed once the runs' first lanes are compacted:
// 0.92 ms (1.02 with eight comparisons, every pair once: more scalar work than it saves).
__global__ __launch_bounds__(256) void runs_find_k(const int32_t* __restrict__ col, int64_t n,
                                                   const SceneDev* __restrict__ scenes, int ns,
                                                   uint32_t* __restrict__ gkey, uint32_t* __restrict__ ginfo,
                                                   int32_t* __restrict__ bcnt)
{
    constexpr int NR = kRunRows / 16;   // rounds of 4 rows per wave
    __shared__ __attribute__((aligned(16))) uint32_t lv[4][64 * NR];
    __shared__ uint16_t li[4][64 * NR];
    __shared__ int wcnt[4];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t b0 = (int64_t)blockIdx.x * kRunSlots;
    const int64_t w0 = b0 + w * 64 * NR;
    uint32_t v[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int64_t at = w0 + r * 64 + lane;   // n is a multiple of 16: a row lies wholly inside or outside
        v[r] = at < n ? (uint32_t)col[at] : 0xffffffffu;
    }
    const uint64_t below = lane ? (~0ull) >> (64 - lane) : 0ull;
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint64_t b =
            __ballot((int32_t)v[r] >= 0) & ~row_repeats(v[r] + 1u, std::make_integer_sequence<int, 15>{});
        lv[w][r * 64 + lane] = v[r];
        if ((b >> lane) & 1u) li[w][cnt + __popcll(b & below)] = (uint16_t)(r * 64 + lane);
        cnt += __popcll(b);
    }
    if (lane == 0) wcnt[w] = cnt;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < w) off += wcnt[q];
        tot += wcnt[q];
    }
    for (int j = lane; j < cnt; j += 64) {
        const int at = li[w][j], row = at >> 4;
        const uint32_t x = lv[w][at];
        const uint4* rv = (const uint4*)&lv[w][row * 16];
        uint32_t mask = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 y = rv[q];
            mask |= (x == y.x ? 1u : 0u) << (4 * q) | (x == y.y ? 2u : 0u) << (4 * q) |
                    (x == y.z ? 4u : 0u) << (4 * q) | (x == y.w ? 8u : 0u) << (4 * q);
        }
        gkey[b0 + off + j] = voxel_key32(scenes, ns, x);
        ginfo[b0 + off + j] = mask | (uint32_t)(w * (kRunRows / 4) + row) << 16;
    }
    if (threadIdx.x == 0) bcnt[blockIdx.x] = tot;
}

// the blocks' runs, one after the other
__global__ __launch_bounds__(256) void runs_pack_k(const uint32_t* __restrict__ gkey,
                                                   const uint32_t* __restrict__ ginfo,
                                                   const int32_t* __restrict__ bcnt, const int64_t* __restrict__ boff,
                                                   uint32_t* __restrict__ key, uint32_t* __restrict__ row,
                                                   uint16_t* __restrict__ mask)
{
    const int64_t g = (int64_t)blockIdx.x * kRunSlots, d = boff[blockIdx.x];
    const int cnt = bcnt[blockIdx.x];
    for (int j = threadIdx.x; j < cnt; j += 256) {
        const uint32_t x = ginfo[g + j];
        key[d + j] = gkey[g + j];
        row[d + j] = (uint32_t)blockIdx.x * kRunRows + (x >> 16);
        mask[d + j] = (uint16_t)(x & 0xffffu);
    }
}

struct LoadPop {
    const uint16_t* p;
    __device__ int64_t operator()(int64_t i) const { return __popc((uint32_t)p[i]); }
};

// Sorted runs written out as list entries: a block takes SC_TILE runs (boff[block]
// entries before them), a wave 64 of them at a time through LDS, so that the
// entries leave as contiguous stores.  The first run of a key sets vptr[key].
__global__ __launch_bounds__(256) void runs_expand_k(const uint32_t* __restrict__ key,
                                                     const uint32_t* __restrict__ row,
                                                     const uint16_t* __restrict__ mask, int64_t n,
                                                     const int64_t* __restrict__ boff, const SlotGroups groups,
                                                     uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                     int64_t* __restrict__ vptr)
{
    constexpr int NR = SC_TILE / 256;   // rounds of 64 runs per wave
    __shared__ uint32_t lv[4][64 * kTile], lk[4][64 * kTile];
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r0 = (int64_t)blockIdx.x * SC_TILE + w * 64 * NR;
    uint32_t k[NR], rw[NR], m[NR];
    bool first[NR];
    int sum = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int64_t at = r0 + r * 64 + lane, ic = at < n ? at : n - 1;
        k[r] = key[ic];
        rw[r] = row[ic];
        m[r] = at < n ? mask[ic] : 0u;
        first[r] = at < n && (ic == 0 || key[ic - 1] != k[r]);
        sum += __popc(m[r]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) wsum[w] = sum;
    __syncthreads();
    int64_t out = boff[blockIdx.x];
    for (int q = 0; q < w; ++q) out += wsum[q];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        int incl = __popc(m[r]);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        int at = incl - __popc(m[r]);
        if (first[r]) vptr[k[r]] = out + at;
        const int64_t slot0 = (int64_t)rw[r] * kTile;
        const uint32_t rel = (uint32_t)(slot0 - (groups.n > 1 ? group_slot_base_of_slot(groups, slot0) : 0));
        for (uint32_t x = m[r]; x; x &= x - 1, ++at) {
            lv[w][at] = rel + (uint32_t)__ffs(x) - 1u;
            lk[w][at] = k[r];
        }
        // LDS accesses of one wave complete in order: the fences keep the compiler
        // from moving the reads above the writes, and the next round's writes above them
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int tot = __shfl(incl, 63, 64);
        for (int j = lane; j < tot; j += 64) {
            vals[out + j] = lv[w][j];
            keys[out + j] = lk[w][j];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        out += tot;
    }
}

// The first run of a key sets vptr[key] (its first entry) and rptr[key] (the run).
__global__ __launch_bounds__(SC_T) void runs_mark_k(const uint32_t* __restrict__ key,
                                                    const uint16_t* __restrict__ mask, int64_t n,
                                                    const int64_t* __restrict__ boff, int64_t* __restrict__ vptr,
                                                    uint32_t* __restrict__ rptr)
{
    const int64_t base = (int64_t)blockIdx.x * SC_TILE + (int64_t)threadIdx.x * SC_IPT;
    uint32_t k[SC_IPT + 1];
    int pc[SC_IPT], sum = 0;
    k[0] = base > 0 && base - 1 < n ? key[base - 1] : 0xffffffffu;   // no voxel's key
#pragma unroll
    for (int q = 0; q < SC_IPT; ++q) {
        const int64_t i = base + q;
        k[q + 1] = i < n ? key[i] : 0u;
        pc[q] = i < n ? __popc((uint32_t)mask[i]) : 0;
        sum += pc[q];
    }
    int64_t tot;
    int64_t at = boff[blockIdx.x] + block_excl_scan_i64(sum, &tot);
#pragma unroll
    for (int q = 0; q < SC_IPT; ++q) {
        if (base + q < n && k[q] != k[q + 1]) {
            vptr[k[q + 1]] = at;
            rptr[k[q + 1]] = (uint32_t)(base + q);
        }
        at += pc[q];
    }
}

// vptr of the keys without a run (all ones so far): that of the next key with one, or the
// number of entries; rptr (may be null) likewise.  A wave takes 1024 keys from the last to
// the first, 64 at a time: the next key with a run is found in the lanes' mask, or is the
// one that the keys before left, at first the first run past all of them (a search among
// the sorted runs).  9.4e6 keys, half of them without a run: 39 us, with a search for
// each of those 175; 1.2e6 keys 10.8 and 15.4.
__global__ __launch_bounds__(256) void vptr_gaps_k(const uint32_t* __restrict__ key, int64_t n, int64_t V,
                                                   int64_t entries, int64_t* __restrict__ vptr,
                                                   uint32_t* __restrict__ rptr)
{
    constexpr int NR = 16;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t v0 = ((int64_t)blockIdx.x * 4 + w) * 64 * NR, v1 = v0 + 64 * NR;   // keys up to V
    if (v0 > V) return;   // whole wave
    int64_t x[NR];
    uint32_t rp[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int64_t v = v0 + r * 64 + lane;
        x[r] = v <= V ? vptr[v] : -1;
        rp[r] = v <= V && rptr ? rptr[v] : 0u;
    }
    int64_t lo = 0, hi = n;   // the first run of a key of v1 or more
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)key[mid] < v1)
            lo = mid + 1;
        else
            hi = mid;
    }
    int64_t nx = entries;
    uint32_t nr = (uint32_t)lo;
    if (lo < n) nx = vptr[key[lo]];   // a key with a run: no wave changes it
#pragma unroll
    for (int r = NR - 1; r >= 0; --r) {
        const int64_t v = v0 + r * 64 + lane;
        const uint64_t has = __ballot(x[r] != -1);
        const uint64_t up = has >> lane;   // from this lane on
        const int src = up ? lane + __ffsll((unsigned long long)up) - 1 : lane;
        const int64_t sx = __shfl(x[r], src, 64);
        const uint32_t sr = __shfl(rp[r], src, 64);
        if (v <= V && x[r] == -1) {
            vptr[v] = up ? sx : nx;
            if (rptr) rptr[v] = up ? sr : nr;
        }
        if (has) {
            const int f = __ffsll((unsigned long long)has) - 1;
            nx = __shfl(x[r], f, 64);
            nr = __shfl(rp[r], f, 64);
        }
    }
}

// Slots are sorted one by one, and lists kept per edge, where there are few of them: the runs
// cost six more launches and a readback of their number, and sweeps gain from them.  The
// line lies where a build with three sweeps takes as long either way.  One frame in 100x100x60
// voxels in us, by slots and by runs: 6.2e5 slots, build 245 and 257, build with 3 sweeps and
// marginals 327 and 336, 10 sweeps alone 170 and 155; 9.1e5, 254 and 258, 335 and 341, 184 and
// 170; 1.08e6, 286 and 286, 378 and 370, 196 and 182; 2.9e6, 286 and 275, 398 and 382, 286 and
// 282.  With keyframe pairs, 1.2e6: build 389 and 394, three sweeps and their reverse 229 and
// 225.  A 640x480 frame (2.4e7) 2075 and 1922 with its sweeps, at 2 cm (6e7) 4427 and 3855.
bool incidence_by_runs(int64_t n) { return n >= (int64_t(1) << 20); }

static int key_bits(int64_t maxval)
{
    int b = 1;
    while (b < 63 && (int64_t(1) << b) <= maxval) ++b;
    return b;
}

hipError_t build_incidence(mrf_ctx* c, int64_t n, int64_t edges, uint32_t* keys, uint32_t* vals, int64_t* vptr,
                           const SlotGroups& groups, bool keep_runs, hipStream_t s)
{
    hipError_t e;
    const int bits = key_bits(c->Vk);
    if (!incidence_by_runs(n)) {
        const int64_t nh = (int64_t)radix_hist_entries(n);
        if ((e = ensure(c->b_tmp64, sizeof(int64_t) * (size_t)(nh + 1) + sizeof(int32_t) * (size_t)nh)) != hipSuccess)
            return e;
        int64_t* offs = (int64_t*)c->b_tmp64.p;
        const size_t tb = (radix_tmp_bytes(n) + 255) / 256 * 256;   // then the sort's spare values
        if ((e = ensure(c->b_misc, tb + sizeof(uint32_t) * (size_t)n)) != hipSuccess) return e;
        e = radix_sort_pairs((const uint32_t*)c->b_g.p, (uint32_t*)c->b_lam.p, (uint32_t*)c->b_ell.p,
                             (uint32_t*)c->b_ellbar.p, (uint32_t*)((char*)c->b_misc.p + tb), keys, vals, n, bits,
                             (int32_t*)(offs + nh + 1), offs, c->b_misc.p, tb, s, groups);
        return e == hipSuccess ? launch_vptr_from_sorted(keys, n, c->Vk, vptr, s) : e;
    }
    // runs are found per block (b_g and a buffer outside the first list), packed into a
    // list and sorted between the lists (b_lam, b_ell) and (b_lambar, b_gsum), masks in the
    // halves of b_ellbar; the first list is the one from which the passes end in (b_lam, b_ell)
    const int passes = (bits + 7) / 8;
    const int64_t nb = cdiv(n, kRunSlots);
    const size_t cnt_bytes = sizeof(int64_t) * (size_t)(nb + 1) + sizeof(int32_t) * (size_t)nb;
    const int64_t nh = (int64_t)radix_hist_entries(n);   // as if every slot were a run
    const size_t tab_bytes = sizeof(int64_t) * (size_t)(nh + 1) + sizeof(int32_t) * (size_t)nh;
    if ((e = ensure(c->b_tmp64, std::max(cnt_bytes, tab_bytes))) != hipSuccess) return e;
    const int64_t nb2 = cdiv(n, SC_TILE);
    const size_t sb = std::max(std::max(scan_tmp_bytes(nb), radix_tmp_bytes(n)),
                               sizeof(int64_t) * (size_t)(2 * nb2 + 1) + scan_tmp_bytes(nb2));
    if ((e = ensure(c->b_misc, sb)) != hipSuccess) return e;
    int64_t* boff = (int64_t*)c->b_tmp64.p;
    int32_t* bcnt = (int32_t*)(boff + nb + 1);
    uint32_t* lk[2] = {(uint32_t*)c->b_lam.p, (uint32_t*)c->b_lambar.p};
    uint32_t* lr[2] = {(uint32_t*)c->b_ell.p, (uint32_t*)c->b_gsum.p};
    uint16_t* lm[2] = {(uint16_t*)c->b_ellbar.p, (uint16_t*)c->b_ellbar.p + n};
    const int first = passes & 1;
    uint32_t* gkey = (uint32_t*)c->b_g.p;
    uint32_t* ginfo = first ? lk[0] : lr[1];
    hipLaunchKernelGGL(runs_find_k, dim3((unsigned)nb), dim3(256), 0, s, (const int32_t*)c->b_col.p, n,
                       (const SceneDev*)c->b_scenes.p, c->n_scenes, gkey, ginfo, bcnt);
    if ((e = scan_exclusive_i32(bcnt, boff, nb, c->b_misc.p, c->b_misc.cap, s)) != hipSuccess) return e;
    int64_t nr = 0;
    if ((e = read_back(c, &nr, boff + nb, sizeof(int64_t), s)) != hipSuccess) return e;
    // more runs than rptr's 32 bits number (a batch of several slot groups; fewer bits for
    // tests, as the groups'): lists of edges after all
    if (keep_runs && nr >= (int64_t(1) << c->group_log2)) {
        if ((e = ensure(c->b_vedge, sizeof(uint32_t) * (size_t)n + 16)) != hipSuccess) return e;
        vals = (uint32_t*)c->b_vedge.p;
        keep_runs = false;
        c->by_runs = 0;
    }
    if (keep_runs) {
        const size_t nrr = (size_t)((double)nr * c->room);
        if ((e = ensure(c->b_runrow, sizeof(uint32_t) * nrr)) != hipSuccess) return e;
        if ((e = ensure(c->b_runmask, sizeof(uint16_t) * nrr)) != hipSuccess) return e;
        if ((e = ensure(c->b_rptr, sizeof(uint32_t) * (size_t)(c->Vk + 1))) != hipSuccess) return e;
        c->n_runs = nr;
    }
    uint32_t* rptr = keep_runs ? (uint32_t*)c->b_rptr.p : nullptr;
    if ((e = launch_fill_u32((uint32_t*)vptr, 0xffffffffu, 2 * (c->Vk + 1), s)) != hipSuccess) return e;
    if (nr > 0) {
        hipLaunchKernelGGL(runs_pack_k, dim3((unsigned)nb), dim3(256), 0, s, (const uint32_t*)gkey,
                           (const uint32_t*)ginfo, (const int32_t*)bcnt, (const int64_t*)boff, lk[first], lr[first],
                           lm[first]);
        const int64_t nhr = (int64_t)radix_hist_entries(nr);
        int64_t* offs = (int64_t*)c->b_tmp64.p;
        const RadixTables t{(int32_t*)(offs + nhr + 1), offs, (int64_t*)c->b_misc.p};
        int at = first;
        for (int p = 0; p < passes; ++p, at ^= 1) {
            if (keep_runs && p == passes - 1) {   // the last pass: to where they stay (at ^ 1 is 0)
                lr[0] = (uint32_t*)c->b_runrow.p;
                lm[0] = (uint16_t*)c->b_runmask.p;
            }
            if ((e = radix_pass<true>(lk[at], lr[at], lm[at], lk[at ^ 1], lr[at ^ 1], lm[at ^ 1], nr, 8 * p, t,
                                      SlotGroups{}, s)) != hipSuccess)
                return e;
        }
        const int64_t nbr = cdiv(nr, SC_TILE);
        int64_t* bsum = (int64_t*)c->b_misc.p;
        int64_t* eoff = bsum + nbr;
        hipLaunchKernelGGL(scan_reduce_k<LoadPop>, dim3((unsigned)nbr), dim3(SC_T), 0, s, LoadPop{lm[0]}, nr, bsum);
        if ((e = scan_rec(LoadI64{bsum}, nbr, eoff, eoff + nbr + 1, s)) != hipSuccess) return e;
        if (keep_runs)
            hipLaunchKernelGGL(runs_mark_k, dim3((unsigned)nbr), dim3(SC_T), 0, s, (const uint32_t*)lk[0],
                               (const uint16_t*)lm[0], nr, (const int64_t*)eoff, vptr, rptr);
        else
            hipLaunchKernelGGL(runs_expand_k, dim3((unsigned)nbr), dim3(256), 0, s, (const uint32_t*)lk[0],
                               (const uint32_t*)lr[0], (const uint16_t*)lm[0], nr, (const int64_t*)eoff, groups, keys,
                               vals, vptr);
    }
    hipLaunchKernelGGL(vptr_gaps_k, dim3((unsigned)cdiv(c->Vk + 1, 4096)), dim3(256), 0, s, (const uint32_t*)lk[0], nr,
                       c->Vk, edges, vptr, rptr);
    return hipGetLastError();
}

// vptr[v] = first position whose key >= v (binary search), v in [0, V]
__global__ void vptr_k(const uint32_t* __restrict__ keys, int64_t n, int64_t V, int64_t* __restrict__ vptr)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > V) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    vptr[v] = lo;
}

hipError_t launch_vptr_from_sorted(const uint32_t* sorted_keys, int64_t n, int64_t V, int64_t* vptr,
                                   hipStream_t s)
{
    hipLaunchKernelGGL(vptr_k, dim3((unsigned)cdiv(V + 1, 256)), dim3(256), 0, s, sorted_keys, n, V, vptr);
    return hipGetLastError();
}

// ============================================================== work lists

// linear voxel id of a brick-major key (keys of padding voxels never appear)
__device__ uint32_t key_to_voxel(const SceneDev* __restrict__ scenes, int ns, uint32_t key)
{
    const SceneDev& sd = scene_of<&SceneDev::key_base>(scenes, ns, key);
    const int64_t local = (int64_t)key - sd.key_base;
    const int64_t brick = local >> 9;
    const int l = (int)(local & 511);
    const int bx = (int)(brick % sd.nb[0]);
    const int by = (int)((brick / sd.nb[0]) % sd.nb[1]);
    const int bz = (int)(brick / ((int64_t)sd.nb[0] * sd.nb[1]));
    const int i = bx * 8 + (l & 7), j = by * 8 + ((l >> 3) & 7), k = bz * 8 + (l >> 6);
    return (uint32_t)(sd.voxel_base + i + (int64_t)sd.n[0] * (j + (int64_t)sd.n[1] * k));
}

// brick-major key of a linear voxel id
__device__ uint32_t voxel_to_key(const SceneDev* __restrict__ scenes, int ns, int64_t v)
{
    const SceneDev& sd = scene_of<&SceneDev::voxel_base>(scenes, ns, v);
    const int64_t local = v - sd.voxel_base;
    const int64_t nxy = (int64_t)sd.n[0] * sd.n[1];
    const int k = (int)(local / nxy);
    const int64_t rem = local - k * nxy;
    const int j = (int)(rem / sd.n[0]), i = (int)(rem - (int64_t)j * sd.n[0]);
    return brick_key(sd, i, j, k);
}

// canonical incidence: degree per linear voxel, then each voxel's edge list
__global__ void canon_degree_k(const SceneDev* __restrict__ scenes, int ns, const int64_t* __restrict__ vptr,
                               int64_t V, int32_t* __restrict__ deg)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const uint32_t k = voxel_to_key(scenes, ns, v);
    deg[v] = (int32_t)(vptr[k + 1] - vptr[k]);
}

// first slot of ray r (its tile's base plus its lane)
__device__ int64_t ray_slot0(const FrameDev* __restrict__ frames, int nf, const SceneDev* __restrict__ scenes,
                             const int64_t* __restrict__ tbase, int64_t r)
{
    int lo = 0, hi = nf;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (frames[mid].ray_base <= r)
            lo = mid;
        else
            hi = mid;
    }
    const FrameDev fr = frames[lo];
    const int W = scenes[fr.scene].W;
    const int64_t pix = r - fr.ray_base;
    const int v = (int)(pix / W), u = (int)(pix - (int64_t)v * W);
    return tbase[fr.tile_base + (int64_t)(v / kTileW) * fr.ntx + u / kTileW] + (v % kTileW) * kTileW + u % kTileW;
}

template <class T>
__global__ void canon_edges_k(const FrameDev* __restrict__ frames, int nf, const SceneDev* __restrict__ scenes,
                              const int64_t* __restrict__ tbase, const int64_t* __restrict__ row_ptr, int64_t R,
                              const T* __restrict__ in, T* __restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    const int64_t d = row_ptr[r], m = row_ptr[r + 1] - d;
    if (m == 0) return;
    const int64_t s0 = ray_slot0(frames, nf, scenes, tbase, r);
    for (int64_t k = 0; k < m; ++k) out[d + k] = in[s0 + kTile * k];
}

}  // namespace mrf

namespace mrf {

// Stable partition of items 0 .. n-1 into classes 0 .. NC-1 (class 255: left
// out), class-major, ascending inside a class: a count per block and class, a
// scan of each class over the blocks, and a placement that classifies again.
// A block takes 256 R items, each of its waves a contiguous quarter in
// rounds of 64; ranks inside a round are wave ballots.  F gives the items of a
// block (range), an item's class (cls), takes its statistics (note, with the
// block's LDS counters) and places it (put).  One read of the items per kernel
// and no host step between: partitioning class by class (a flag scan of every
// item, a readback and a compaction each, 25 times per build) took 1.05 of the
// 1.34 ms of a 64x48 frame's build and inference and 1.9 of 24 ms at 8 VGA
// keyframes and 9.4e6 voxels.
// A wave takes R rounds: 16 where there are blocks enough (fewer block counts to
// scan), 2 below 2^20 items, whose few blocks would each walk serially (the tiles of a
// VGA frame, 19200 items: 155 us with 16 rounds, 23 with 2).
template <int R>
constexpr int part_items() { return 256 * R; }
static int part_rounds(int64_t n) { return n < (int64_t(1) << 20) ? 2 : 16; }
constexpr int kPartMaxClasses = 16;

// Statistics of the work lists: items, edges and rays per class, log2
// histograms and maxima of ray lengths and voxel degrees.
struct ListStats {
    unsigned long long tiles[kPartMaxClasses], tile_edges[kPartMaxClasses], tile_rays[kPartMaxClasses];
    unsigned long long voxels[kPartMaxClasses];
    unsigned long long ray_hist[16], deg_hist[24], max_ray, max_deg, pieces;
};

struct PartLds {
    unsigned long long edges[kPartMaxClasses];
    uint32_t rays[kPartMaxClasses], hist[24], top, pieces;
};

__device__ __forceinline__ int64_t seg_pieces(int64_t m, int piece) { return (m + piece - 1) / piece; }

__device__ __forceinline__ int vox_class(int64_t m)
{
    if (m <= 0) return 255;
    if (m > 2147483647LL) return kVoxClasses;   // reported as an error by the host
    int c = kVoxClasses - 1;
#pragma unroll
    for (int k = kVoxClasses - 2; k >= 0; --k)
        if (m <= kVoxCap[k]) c = k;
    return c;
}

// tiles of rays by their longest ray; blocks do not span frames (bpf blocks each)
struct TileItems {
    static constexpr int NC = kRayClasses + 1;   // and tiles that are too long
    static_assert(NC <= kPartMaxClasses, "classes");
    const TileDev* tiles;
    const int32_t* counts;
    const FrameDev* frames;
    int64_t T;
    int nf, bpf;
    uint32_t* list;
    ListStats* st;
    __device__ void range(int64_t b, int items, int64_t& i0, int64_t& i1) const
    {
        const int f = (int)(b / bpf);
        i0 = frames[f].tile_base + (b - (int64_t)f * bpf) * items;
        i1 = f + 1 < nf ? frames[f + 1].tile_base : T;
    }
    __device__ int cls(int64_t i) const
    {
        const int n = tiles[i].len;
        if (n <= 0) return 255;
        int c = kRayClasses;   // too long: reported as an error by the host
#pragma unroll
        for (int k = kRayClasses - 1; k >= 0; --k)
            if (n <= kRayCap[k]) c = k;
        return c;
    }
    __device__ void note(int64_t i, int c, PartLds& l) const
    {
        const TileDev td = tiles[i];
        uint32_t e = 0, nr = 0, mx = 0;
        for (int a = 0; a < td.nv; ++a)
            for (int b = 0; b < td.nu; ++b) {
                const int x = counts[td.ray0 + a * td.W + b];
                if (x <= 0) continue;
                e += (uint32_t)x;
                ++nr;
                mx = max(mx, (uint32_t)x);
                atomicAdd(&l.hist[min(15, 31 - __clz(x))], 1u);
            }
        atomicAdd(&l.edges[c], (unsigned long long)e);
        atomicAdd(&l.rays[c], nr);
        atomicMax(&l.top, mx);
    }
    __device__ void flush(const PartLds& l, int t) const
    {
        if (t < NC && l.edges[t]) atomicAdd(&st->tile_edges[t], l.edges[t]);
        if (t < NC && l.rays[t]) atomicAdd(&st->tile_rays[t], (unsigned long long)l.rays[t]);
        if (t < 16 && l.hist[t]) atomicAdd(&st->ray_hist[t], (unsigned long long)l.hist[t]);
        if (t == 0 && l.top) atomicMax(&st->max_ray, (unsigned long long)l.top);
    }
    __device__ void put(int64_t at, int64_t i, int c) const
    {
        if (c < kRayClasses) list[at] = (uint32_t)i;
    }
};

// class by number of runs
__device__ __forceinline__ int run_class(int64_t m)
{
    int k = kVoxClasses - 1;
#pragma unroll
    for (int q = kRunClasses - 1; q >= 0; --q)
        if (m <= kRunCap[q]) k = q;
    return k;
}

// brick-major voxel keys by degree, or by number of runs (rptr not null)
struct VoxItems {
    static constexpr int NC = kVoxClasses + 1;   // and voxels of too many edges
    static_assert(NC <= kPartMaxClasses, "classes");
    const int64_t* vptr;
    const uint32_t* rptr;
    int64_t n;
    const SceneDev* scenes;
    int ns;
    VoxDev* desc;
    ListStats* st;
    __device__ void range(int64_t b, int items, int64_t& i0, int64_t& i1) const
    {
        i0 = b * items;
        i1 = n;
    }
    __device__ int cls(int64_t i) const
    {
        const int c = vox_class(vptr[i + 1] - vptr[i]);
        if (!rptr || c >= kVoxClasses) return c;   // 255, or too many edges
        return run_class((int64_t)rptr[i + 1] - rptr[i]);
    }
    __device__ void note(int64_t i, int c, PartLds& l) const
    {
        const int64_t m = vptr[i + 1] - vptr[i];
        const int64_t items = rptr ? (int64_t)rptr[i + 1] - rptr[i] : m;
        const int piece = rptr ? kRunPiece : kSegPiece;
        if (items > piece) atomicAdd(&l.pieces, (uint32_t)min(seg_pieces(items, piece), (int64_t)1 << 22));
        atomicAdd(&l.hist[min(23, 63 - __clzll(m))], 1u);
        atomicMax(&l.top, (uint32_t)min(m, (int64_t)0xffffffffLL));
    }
    __device__ void flush(const PartLds& l, int t) const
    {
        if (t == 1 && l.pieces) atomicAdd(&st->pieces, (unsigned long long)l.pieces);
        if (t < 24 && l.hist[t]) atomicAdd(&st->deg_hist[t], (unsigned long long)l.hist[t]);
        if (t == 0 && l.top) atomicMax(&st->max_deg, (unsigned long long)l.top);
    }
    __device__ void put(int64_t at, int64_t i, int c) const
    {
        if (c >= kVoxClasses) return;
        const int64_t s = rptr ? (int64_t)rptr[i] : vptr[i];
        const int64_t e = rptr ? (int64_t)rptr[i + 1] : vptr[i + 1];
        desc[at] = VoxDev{s, (int32_t)(e - s), key_to_voxel(scenes, ns, (uint32_t)i)};
    }
};

// (keyframe, voxel) pairs by edge count, or by number of runs
struct PairItems {
    static constexpr int NC = kVoxClasses;
    const uint32_t* pstart;
    int64_t n;
    int runs;
    VoxDev* desc;
    __device__ void range(int64_t b, int items, int64_t& i0, int64_t& i1) const
    {
        i0 = b * items;
        i1 = n;
    }
    __device__ int cls(int64_t i) const
    {
        const int64_t m = (int64_t)pstart[i + 1] - pstart[i];
        return runs ? run_class(m) : vox_class(m);
    }
    unsigned long long* pieces;
    __device__ void note(int64_t i, int, PartLds& l) const
    {
        const int64_t m = (int64_t)pstart[i + 1] - pstart[i];
        const int piece = runs ? kRunPiece : kSegPiece;
        if (m > piece) atomicAdd(&l.pieces, (uint32_t)seg_pieces(m, piece));
    }
    __device__ void flush(const PartLds& l, int t) const
    {
        if (t == 0 && l.pieces) atomicAdd(pieces, (unsigned long long)l.pieces);
    }
    __device__ void put(int64_t at, int64_t i, int) const
    {
        desc[at] = VoxDev{(int64_t)pstart[i], (int32_t)(pstart[i + 1] - pstart[i]), (uint32_t)i};
    }
};

template <int R, class F>
__device__ __forceinline__ void part_count(const F& f, int64_t block, int64_t nb, uint32_t* __restrict__ bcnt,
                                           PartLds& l, uint32_t (&wc)[4][kPartMaxClasses])
{
    for (int i = threadIdx.x; i < (int)(sizeof(PartLds) / 4); i += 256) ((uint32_t*)&l)[i] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t i0, i1;
    f.range(block, part_items<R>(), i0, i1);
    i0 += (int64_t)w * R * 64;
    int cl[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = i0 + r * 64 + lane;
        cl[r] = i < i1 ? f.cls(i) : 255;
    }
    uint32_t cnt[F::NC] = {0};
#pragma unroll 2
    for (int r = 0; r < R; ++r) {
        if (cl[r] < F::NC) f.note(i0 + r * 64 + lane, cl[r], l);
#pragma unroll
        for (int k = 0; k < F::NC; ++k) cnt[k] += (uint32_t)__popcll(__ballot(cl[r] == k));
    }
#pragma unroll
    for (int k = 0; k < F::NC; ++k)
        if (lane == k) wc[w][k] = cnt[k];
    __syncthreads();
    if (threadIdx.x < F::NC) {
        uint32_t t = 0;
        for (int q = 0; q < 4; ++q) t += wc[q][threadIdx.x];
        bcnt[(int64_t)threadIdx.x * nb + block] = t;
    }
    f.flush(l, threadIdx.x);
}

// the blocks of f's items, then those of g's
template <class F, int R, class G, int Q>
__global__ __launch_bounds__(256) void part_count_k(const F f, int64_t nf, uint32_t* __restrict__ fcnt, const G g,
                                                    int64_t ng, uint32_t* __restrict__ gcnt)
{
    __shared__ PartLds l;
    __shared__ uint32_t wc[4][kPartMaxClasses];
    if (blockIdx.x < nf)
        part_count<R>(f, blockIdx.x, nf, fcnt, l, wc);
    else
        part_count<Q>(g, (int64_t)blockIdx.x - nf, ng, gcnt, l, wc);
}

// exclusive scan over the blocks of each class (one wave per class, in place),
// the class totals, and with fo the value at every bpf-th block (a frame's first)
struct PartScan {
    uint32_t* bcnt;
    int64_t nb;
    int nc;
    unsigned long long* tot;
    int64_t* fo;
    int bpf, nf;
};

__global__ __launch_bounds__(64 * kPartMaxClasses) void part_scan_k(const PartScan a, const PartScan b2)
{
    const PartScan& l = blockIdx.x == 0 ? a : b2;
    uint32_t* bcnt = l.bcnt;
    const int64_t nb = l.nb;
    const int nc = l.nc, bpf = l.bpf, nf = l.nf;
    unsigned long long* tot = l.tot;
    int64_t* fo = l.fo;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (k >= nc) return;
    uint32_t* p = bcnt + (int64_t)k * nb;
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += 256) {
        uint32_t x[4], t = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t b = b0 + 4 * lane + q;
            x[q] = b < nb ? p[b] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) t += x[q];
        uint32_t incl = t;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        uint32_t run = carry + incl - t;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t b = b0 + 4 * lane + q;
            if (b < nb) {
                p[b] = run;
                if (fo && b % bpf == 0) fo[(int64_t)k * (nf + 1) + b / bpf] = run;
            }
            run += x[q];
        }
        carry += __shfl(incl, 63, 64);
    }
    if (lane == 0) {
        tot[k] = carry;
        if (fo) fo[(int64_t)k * (nf + 1) + nf] = carry;
    }
}

template <int R, class F>
__device__ __forceinline__ void part_place(const F& f, int64_t block, int64_t nb, const uint32_t* __restrict__ boff,
                                           const unsigned long long* __restrict__ tot,
                                           uint32_t (&wc)[4][kPartMaxClasses])
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t i0, i1;
    f.range(block, part_items<R>(), i0, i1);
    i0 += (int64_t)w * R * 64;
    int cl[R];
    uint32_t cnt[F::NC] = {0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = i0 + r * 64 + lane;
        cl[r] = i < i1 ? f.cls(i) : 255;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < F::NC; ++k) cnt[k] += (uint32_t)__popcll(__ballot(cl[r] == k));
#pragma unroll
    for (int k = 0; k < F::NC; ++k)
        if (lane == k) wc[w][k] = cnt[k];
    __syncthreads();
    // the ballots of the second walk are taken again: kept from the first (R NC masks)
    // they would spill
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(cl[r]));
    uint32_t at[F::NC];   // next position of this wave's items of class k (totals are below 2^32)
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < F::NC; ++k) {
        at[k] = base + boff[(int64_t)k * nb + block];
        for (int q = 0; q < w; ++q) at[k] += wc[q][k];
        base += (uint32_t)tot[k];
    }
    const uint64_t below = lane ? (~0ull) >> (64 - lane) : 0ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t pos = 0;
#pragma unroll
        for (int k = 0; k < F::NC; ++k) {
            const uint64_t m = __ballot(cl[r] == k);
            if (cl[r] == k) pos = at[k] + (uint32_t)__popcll(m & below);
            at[k] += (uint32_t)__popcll(m);
        }
        if (cl[r] < F::NC) f.put(pos, i0 + r * 64 + lane, cl[r]);
    }
}

template <class F, int R, class G, int Q>
__global__ __launch_bounds__(256) void part_place_k(const F f, int64_t nf, const uint32_t* __restrict__ foff,
                                                    const unsigned long long* __restrict__ ftot, const G g,
                                                    int64_t ng, const uint32_t* __restrict__ goff,
                                                    const unsigned long long* __restrict__ gtot)
{
    __shared__ uint32_t wc[4][kPartMaxClasses];
    if (blockIdx.x < nf)
        part_place<R>(f, blockIdx.x, nf, foff, ftot, wc);
    else
        part_place<Q>(g, (int64_t)blockIdx.x - nf, ng, goff, gtot, wc);
}

// Two lists partitioned in the same three launches (sf, sg: their scans)
template <class F, int R, class G, int Q>
static hipError_t partition_r(const F& f, const PartScan& sf, const G& g, const PartScan& sg, hipStream_t s)
{
    const unsigned nb = (unsigned)(sf.nb + sg.nb);
    if (nb > 0)
        hipLaunchKernelGGL((part_count_k<F, R, G, Q>), dim3(nb), dim3(256), 0, s, f, sf.nb, sf.bcnt, g, sg.nb, sg.bcnt);
    hipLaunchKernelGGL(part_scan_k, dim3(2), dim3(64 * kPartMaxClasses), 0, s, sf, sg);
    if (nb > 0)
        hipLaunchKernelGGL((part_place_k<F, R, G, Q>), dim3(nb), dim3(256), 0, s, f, sf.nb, (const uint32_t*)sf.bcnt,
                           (const unsigned long long*)sf.tot, g, sg.nb, (const uint32_t*)sg.bcnt,
                           (const unsigned long long*)sg.tot);
    return hipGetLastError();
}

template <class F, class G>
static hipError_t partition(const F& f, int fr, const PartScan& sf, const G& g, int gr, const PartScan& sg,
                            hipStream_t s)
{
    if (fr == 2) return gr == 2 ? partition_r<F, 2, G, 2>(f, sf, g, sg, s) : partition_r<F, 2, G, 16>(f, sf, g, sg, s);
    return gr == 2 ? partition_r<F, 16, G, 2>(f, sf, g, sg, s) : partition_r<F, 16, G, 16>(f, sf, g, sg, s);
}

// A list that is not there
struct NoItems {
    static constexpr int NC = 1;
    __device__ void range(int64_t, int, int64_t& i0, int64_t& i1) const { i0 = i1 = 0; }
    __device__ int cls(int64_t) const { return 255; }
    __device__ void note(int64_t, int, PartLds&) const {}
    __device__ void flush(const PartLds&, int) const {}
    __device__ void put(int64_t, int64_t, int) const {}
};

// The hub segments hubs[0, n) cut into pieces of `piece` items (one block): the
// pieces in order, then per hub its range of them (at[np + i]).
__global__ __launch_bounds__(SC_T) void hub_pieces_k(const VoxDev* __restrict__ hubs, int64_t n, int64_t np,
                                                     int piece, VoxDev* __restrict__ at)
{
    int64_t carry = 0;
    for (int64_t i0 = 0; i0 < n; i0 += SC_T) {
        const int64_t i = i0 + threadIdx.x;
        const VoxDev d = hubs[i < n ? i : n - 1];
        const int64_t k = i < n ? seg_pieces(d.m, piece) : 0;
        int64_t tot;
        const int64_t first = carry + block_excl_scan_i64(k, &tot);
        carry += tot;
        if (i >= n) continue;
        at[np + i] = VoxDev{first, (int32_t)k, d.v};
        for (int64_t p = 0; p < k; ++p) {
            const int64_t left = d.m - p * piece;
            at[first + p] = VoxDev{d.start + p * piece, (int32_t)(left < piece ? left : piece), (uint32_t)(first + p)};
        }
    }
}

// class sizes of a partitioned list, and its hubs' pieces
static hipError_t finish_segments(mrf_ctx* c, SegList& l, const unsigned long long* cnt, int64_t pieces, int piece,
                                  hipStream_t s)
{
    int64_t off = 0;
    for (int k = 0; k < kVoxClasses; ++k) {
        l.off[k] = off;
        off += l.cnt[k] = (int64_t)cnt[k];
    }
    const int64_t nh = l.cnt[kVoxClasses - 1];
    l.n_pieces = pieces;
    if (nh == 0) return hipSuccess;
    hipError_t e = ensure(l.hub, sizeof(VoxDev) * (size_t)(pieces + nh));
    if (e == hipSuccess) e = ensure(c->b_hubsum, sizeof(double) * (size_t)pieces);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(hub_pieces_k, dim3(1), dim3(SC_T), 0, s, (const VoxDev*)l.desc.p + l.off[kVoxClasses - 1], nh,
                       pieces, piece, (VoxDev*)l.hub.p);
    return hipGetLastError();
}

hipError_t build_classes(mrf_ctx* c, hipStream_t s)
{
    hipError_t e;
    const int nf = c->n_frames;
    const int tr = part_rounds(c->T), vr = part_rounds(c->Vk);
    const int bpf = (int)std::max<int64_t>(1, cdiv(c->max_tpf, 256 * tr));
    const int64_t tb = (int64_t)bpf * nf, vb = cdiv(c->Vk, 256 * vr);
    // statistics | frame offsets of every tile class | per-block counts
    const size_t fo_bytes = sizeof(int64_t) * (size_t)TileItems::NC * (nf + 1);
    const size_t head = sizeof(ListStats) + fo_bytes;
    if ((e = ensure(c->b_part, head + sizeof(uint32_t) * (size_t)(TileItems::NC * tb + VoxItems::NC * vb))) !=
        hipSuccess)
        return e;
    const int64_t nvox = std::min(c->V, c->E);   // at most this many touched voxels
    if ((e = ensure(c->b_ray_list, sizeof(uint32_t) * (size_t)c->T)) != hipSuccess) return e;
    if ((e = ensure(c->vox.desc, sizeof(VoxDev) * (size_t)nvox)) != hipSuccess) return e;
    ListStats* st = (ListStats*)c->b_part.p;
    int64_t* fo = (int64_t*)(st + 1);
    uint32_t* tcnt = (uint32_t*)((char*)c->b_part.p + head);
    uint32_t* vcnt = tcnt + (size_t)TileItems::NC * tb;
    if ((e = launch_fill_u32((uint32_t*)st, 0u, (int64_t)(sizeof(ListStats) / 4), s)) != hipSuccess) return e;
    const TileItems ti{(const TileDev*)c->b_tiles.p, (const int32_t*)c->b_counts.p, (const FrameDev*)c->b_frames.p,
                       c->T, nf, bpf, (uint32_t*)c->b_ray_list.p, st};
    const VoxItems vi{(const int64_t*)c->b_vptr.p, c->by_runs ? (const uint32_t*)c->b_rptr.p : nullptr, c->Vk, (const SceneDev*)c->b_scenes.p, c->n_scenes,
                      (VoxDev*)c->vox.desc.p, st};
    e = partition(ti, tr, PartScan{tcnt, tb, TileItems::NC, st->tiles, fo, bpf, nf}, vi, vr,
                  PartScan{vcnt, vb, VoxItems::NC, st->voxels, nullptr, 1, 0}, s);
    if (e != hipSuccess) return e;

    // one readback: class sizes, statistics, and per-frame offsets of the tile lists (plain schedule)
    std::vector<char> hb(head);
    if ((e = read_back(c, hb.data(), st, head, s)) != hipSuccess) return e;
    const ListStats& h = *(const ListStats*)hb.data();
    if (h.tiles[kRayClasses] > 0) {
        set_error("a ray crosses more than 2048 voxels");
        return hipErrorInvalidConfiguration;
    }
    if (h.voxels[kVoxClasses] > 0) {
        set_error("a voxel is crossed by more than 2^31 - 1 rays");
        return hipErrorInvalidConfiguration;
    }
    int64_t off = 0;
    for (int k = 0; k < kRayClasses; ++k) {
        c->ray_off[k] = off;
        off += c->ray_cnt[k] = (int64_t)h.tiles[k];
        c->ray_cls_edges[k] = (int64_t)h.tile_edges[k];
        c->ray_cls_rays[k] = (int64_t)h.tile_rays[k];
    }
    if ((e = finish_segments(c, c->vox, h.voxels, (int64_t)h.pieces, c->by_runs ? kRunPiece : kSegPiece, s)) != hipSuccess) return e;
    const int64_t* hfo = (const int64_t*)(hb.data() + sizeof(ListStats));
    c->frame_ray_off.assign(hfo, hfo + (size_t)(nf + 1) * kRayClasses);
    for (int i = 0; i < 16; ++i) c->stats.ray_len_hist[i] = (int64_t)h.ray_hist[i];
    for (int i = 0; i < 24; ++i) c->stats.voxel_degree_hist[i] = (int64_t)h.deg_hist[i];
    c->stats.max_ray_len = (int64_t)h.max_ray;
    c->stats.max_voxel_degree = (int64_t)h.max_deg;
    return hipSuccess;
}

// the pairs [pstart[p], pstart[p + 1]) of the lists (edges or runs) by size
static hipError_t partition_pairs(mrf_ctx* c, const uint32_t* pstart, int64_t P, hipStream_t s)
{
    hipError_t e;
    const int rounds = part_rounds(P);
    const int64_t nb = cdiv(P, 256 * rounds);
    const size_t head = sizeof(unsigned long long) * (kPartMaxClasses + 1);   // class sizes, hub pieces
    if ((e = ensure(c->b_part, head + sizeof(uint32_t) * (size_t)(PairItems::NC * nb))) != hipSuccess) return e;
    unsigned long long* tot = (unsigned long long*)c->b_part.p;
    if ((e = launch_fill_u32((uint32_t*)tot, 0u, (int64_t)(head / 4), s)) != hipSuccess) return e;
    const PairItems f{pstart, P, c->by_runs, (VoxDev*)c->pair.desc.p, tot + kPartMaxClasses};
    const PartScan sf{(uint32_t*)((char*)c->b_part.p + head), nb, PairItems::NC, tot, nullptr, 1, 0}, none{};
    e = rounds == 2 ? partition_r<PairItems, 2, NoItems, 2>(f, sf, NoItems{}, none, s)
                    : partition_r<PairItems, 16, NoItems, 2>(f, sf, NoItems{}, none, s);
    unsigned long long h[kPartMaxClasses + 1];
    if (e == hipSuccess) e = read_back(c, h, tot, head, s);
    if (e != hipSuccess) return e;
    return finish_segments(c, c->pair, h, (int64_t)h[kPartMaxClasses], c->by_runs ? kRunPiece : kSegPiece, s);
}

// ============================================================== adding keyframes
//
// Frames appended to the last scene add tiles and slots after every existing one; the
// voxel -> ray lists are sorted anew.

__global__ void slot_keys_k(const SceneDev* __restrict__ scenes, int ns, const int32_t* __restrict__ col, int64_t n,
                            uint32_t pad_key, uint32_t* __restrict__ keys)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        keys[j] = col[j] < 0 ? pad_key : voxel_key32(scenes, ns, (uint32_t)col[j]);
}

__global__ void add_i64_k(int64_t* __restrict__ p, int64_t v, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        p[k] += v;
}

hipError_t read_back(mrf_ctx* c, void* dst, const void* src, size_t bytes, hipStream_t s)
{
    const bool fits = bytes <= kPinnedBytes;
    hipError_t e = hipMemcpyAsync(fits ? c->pinned : dst, src, bytes, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess && fits) std::memcpy(dst, c->pinned, bytes);
    return e;
}

static unsigned grid_of(int64_t n)
{
    int64_t b = cdiv(n, 256);
    if (b > 65536) b = 65536;
    return (unsigned)(b > 0 ? b : 1);
}

hipError_t launch_add_i64(int64_t* p, int64_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(add_i64_k, dim3(grid_of(n)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_slot_keys(const mrf_ctx* c, hipStream_t s)
{
    if (c->S <= 0) return hipSuccess;
    hipLaunchKernelGGL(slot_keys_k, dim3(grid_of(c->S)), dim3(256), 0, s, (const SceneDev*)c->b_scenes.p, c->n_scenes,
                       (const int32_t*)c->b_col.p, c->S, (uint32_t)c->Vk, (uint32_t*)c->b_g.p);
    return hipGetLastError();
}

// ============================================================== keyframe pairs
//
// Per-keyframe averaged messages (Sec. IV-A): the rays of one keyframe that
// cross a voxel send it one message, the average of theirs weighted by the
// length each travels in the voxel.  A voxel's list (slots ascending) is grouped by
// keyframe, since slots are frame-major; each stretch of one keyframe inside one
// voxel's list is a (keyframe, voxel) pair.  A list of runs (16 slots of a row, so of
// one keyframe) has a tenth of the entries of one of edges: lists and pairs of 4 VGA
// frames at 4 cm (1.14e8 slots, the last one added) take 4.5 ms so, and 5.5 over the
// list of edges.

// first slot of every frame (frames occupy consecutive slot ranges in order);
// fs[nf] = S
__global__ void frame_slots_k(const FrameDev* __restrict__ frames, int nf, const int64_t* __restrict__ tbase,
                              int64_t T, int64_t* __restrict__ fs)
{
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < nf) fs[f] = tbase[frames[f].tile_base];
    if (f == nf) fs[nf] = tbase[T];
}

// frame holding slot x: the last f with fs[f] <= x (frames without edges
// share their successor's first slot and are skipped)
__device__ __forceinline__ int slot_frame(const int64_t* __restrict__ fs, int nf, int64_t x)
{
    int lo = 0, hi = nf;   // fs[lo] <= x < fs[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (fs[mid] <= x)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// the frame (keyframe) of every entry of the voxel -> ray list (slots: a slot's, 1, or a row's, 16)
__global__ void entry_frame_k(const uint32_t* __restrict__ entry, int slots, int64_t n,
                              const int64_t* __restrict__ fs, int nf, uint16_t* __restrict__ fr)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        fr[j] = (uint16_t)slot_frame(fs, nf, (int64_t)entry[j] * slots);
}

// 1 where entry j of the voxel -> ray list starts a (keyframe, voxel) pair
struct LoadPairStart {
    const uint16_t* fr;     // frame of each entry
    const uint32_t* keys;   // sorted voxel keys, aligned with the list
    __device__ int64_t operator()(int64_t j) const
    {
        if (j == 0) return 1;
        if (keys[j] != keys[j - 1]) return 1;
        return fr[j] != fr[j - 1] ? 1 : 0;
    }
};

// pair p (starting at entry j): its first entry and the index of its message
// in the per-keyframe buffers, xb[f] + linear voxel id
__global__ void pair_init_k(const LoadPairStart ld, int64_t E, const uint32_t* __restrict__ pos,
                            const SceneDev* __restrict__ scenes, int ns, const int64_t* __restrict__ xb,
                            uint32_t* __restrict__ pstart, uint32_t* __restrict__ px)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j > E) return;
    if (j == E) {
        pstart[pos[E]] = (uint32_t)E;
        return;
    }
    if (!ld(j)) return;
    const uint32_t p = pos[j];
    pstart[p] = (uint32_t)j;
    const int f = ld.fr[j];
    px[p] = (uint32_t)(xb[f] + (int64_t)key_to_voxel(scenes, ns, ld.keys[j]));
}

// the pairs of every touched voxel (work item of the voxel phase): [pos[start], pos[start + m])
__global__ void kf_vox_k(const VoxDev* __restrict__ vox, int64_t n, const uint32_t* __restrict__ pos,
                         VoxDev* __restrict__ desc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const VoxDev d = vox[i];
    const uint32_t p0 = pos[d.start], p1 = pos[d.start + d.m];
    desc[i] = VoxDev{(int64_t)p0, (int32_t)(p1 - p0), d.v};
}

// weight of entry j = chord length / its pair's summed chord length (equal
// weights should every chord of the pair have rounded to zero length)
__global__ void pair_weight_k(const uint32_t* __restrict__ vedge, const uint32_t* __restrict__ pos, int64_t E,
                              const uint32_t* __restrict__ pstart, const float* __restrict__ wlen,
                              const double* __restrict__ wsum, float* __restrict__ w)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < E; j += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = pos[j + 1] - 1;   // inclusive count of pair starts, less one
        const double sw = wsum[p];
        w[j] = sw > 0.0 ? (float)((double)wlen[vedge[j]] / sw) : (float)(1.0 / (double)(pstart[p + 1] - pstart[p]));
    }
}

// The same over runs, in slot order: lane l of a 16-lane group takes lane l of a run's row.
__global__ __launch_bounds__(256) void pair_weight_runs_k(const uint32_t* __restrict__ rows,
                                                          const uint16_t* __restrict__ masks,
                                                          const uint32_t* __restrict__ pos, int64_t n,
                                                          const uint32_t* __restrict__ pstart,
                                                          const float* __restrict__ len,
                                                          const double* __restrict__ wsum, float* __restrict__ w)
{
    const int l = threadIdx.x & 15;
    for (int64_t j = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); j < n; j += (int64_t)gridDim.x * 16) {
        if (!((masks[j] >> l) & 1u)) continue;
        const uint32_t p = pos[j + 1] - 1;   // inclusive count of pair starts, less one
        const double sw = wsum[p];
        const int64_t at = (int64_t)rows[j] * kTile + l;
        int m = 0;
        if (!(sw > 0.0))
            for (uint32_t r = pstart[p]; r < pstart[p + 1]; ++r) m += __popc((uint32_t)masks[r]);
        w[at] = sw > 0.0 ? (float)((double)len[at] / sw) : (float)(1.0 / (double)m);
    }
}

hipError_t build_keyframe_pairs(mrf_ctx* c, hipStream_t s)
{
    hipError_t e;
    const int64_t E = c->E;
    const int nf = c->n_frames;
    // per-keyframe message buffers: frame f's entries follow the frames before it
    std::vector<int64_t> xb(nf);
    int64_t nx = 0;
    for (int f = 0; f < nf; ++f) {
        const SceneDev& sd = c->scenes_h[c->frames_h[f].scene];
        xb[f] = nx - sd.voxel_base;
        nx += (int64_t)sd.n[0] * sd.n[1] * sd.n[2];
    }
    if (nx >= (int64_t(1) << 32)) {
        set_error("per-keyframe message buffers of 2^32 or more entries");
        return hipErrorInvalidConfiguration;
    }
    c->n_kfx = nx;
    if ((e = ensure(c->b_kfxb, sizeof(int64_t) * (size_t)(nf + 1) * 2)) != hipSuccess) return e;
    int64_t* d_xb = (int64_t*)c->b_kfxb.p;
    int64_t* d_fs = d_xb + nf + 1;
    if ((e = hipMemcpyAsync(d_xb, xb.data(), sizeof(int64_t) * nf, hipMemcpyHostToDevice, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(frame_slots_k, dim3((unsigned)cdiv(nf + 1, 64)), dim3(64), 0, s,
                       (const FrameDev*)c->b_frames.p, nf, (const int64_t*)c->b_tbase.p, c->T, d_fs);
    if ((e = ensure(c->b_kfx, sizeof(float) * (size_t)(nx > 0 ? nx : 1))) != hipSuccess) return e;

    // Pair starts: exclusive count over the entries (pos, n + 1 of them) from the sorted keys
    // and each entry's frame, in per-slot arrays free during the build.  Lists of edges: keys
    // in b_lambar, count in b_lam, pair starts in b_ell; runs: b_lam, b_ell, b_ellbar.
    const bool runs = c->by_runs != 0;
    const int64_t n = runs ? c->n_runs : E;
    const uint32_t* entry = (const uint32_t*)(runs ? c->b_runrow.p : c->b_vedge.p);
    uint16_t* fr = (uint16_t*)c->b_gsum.p;   // 2 n bytes
    const unsigned nblocks = (unsigned)std::min<int64_t>(cdiv(n, 256), 65536);
    if (n > 0)
        hipLaunchKernelGGL(entry_frame_k, dim3(nblocks), dim3(256), 0, s, entry, runs ? kTile : 1, n,
                           (const int64_t*)d_fs, nf, fr);
    const LoadPairStart ld{fr, (const uint32_t*)(runs ? c->b_lam.p : c->b_lambar.p)};
    uint32_t* pos = (uint32_t*)(runs ? c->b_ell.p : c->b_lam.p);
    const size_t sb = scan_tmp_bytes(n);
    if ((e = ensure(c->b_misc, sb > c->b_misc.cap ? sb : c->b_misc.cap)) != hipSuccess) return e;
    if ((e = scan_rec(ld, n, pos, (int64_t*)c->b_misc.p, s)) != hipSuccess) return e;
    uint32_t P32 = 0;
    if ((e = read_back(c, &P32, pos + n, sizeof(uint32_t), s)) != hipSuccess) return e;
    const int64_t P = P32;
    c->n_pairs = P;
    uint32_t* pstart = (uint32_t*)(runs ? c->b_ellbar.p : c->b_ell.p);   // P + 1 <= n + 1 entries
    if ((e = ensure(c->b_pair_x, sizeof(uint32_t) * (size_t)(P > 0 ? P : 1))) != hipSuccess) return e;
    if ((e = ensure(c->b_pair_m, sizeof(double) * (size_t)(P > 0 ? P : 1))) != hipSuccess) return e;
    hipLaunchKernelGGL(pair_init_k, dim3((unsigned)cdiv(n + 1, 256)), dim3(256), 0, s, ld, n, (const uint32_t*)pos,
                       (const SceneDev*)c->b_scenes.p, c->n_scenes, (const int64_t*)d_xb, pstart,
                       (uint32_t*)c->b_pair_x.p);

    // pairs by size, as VoxDev work items of the voxel-phase kernels
    if ((e = ensure(c->pair.desc, (size_t)(P > 0 ? P : 1) * sizeof(VoxDev))) != hipSuccess) return e;
    if ((e = partition_pairs(c, pstart, P, s)) != hipSuccess) return e;

    // touched voxels with their pair ranges, in the voxel lists' order
    int64_t nv = 0;
    for (int k = 0; k < kVoxClasses; ++k) nv += c->vox.cnt[k];
    c->n_kf_vox = nv;
    if ((e = ensure(c->b_kf_vox, (size_t)(nv > 0 ? nv : 1) * sizeof(VoxDev))) != hipSuccess) return e;
    if (nv > 0)
        hipLaunchKernelGGL(kf_vox_k, dim3((unsigned)cdiv(nv, 256)), dim3(256), 0, s, (const VoxDev*)c->vox.desc.p,
                           nv, (const uint32_t*)pos, (VoxDev*)c->b_kf_vox.p);

    // weights: chord length over the pair's summed chord length, which the pair phase
    // forms from the chord lengths (slot order, b_kflen).  Lists of edges keep them in list
    // order (b_kfw), runs in slot order (b_kfws, where the reverse pass reads them too).
    double* wsum = (double*)c->b_pair_m.p;
    if ((e = launch_pair_phase(c, (const float*)c->b_kflen.p, nullptr, wsum, s)) != hipSuccess) return e;
    if (runs) {
        if ((e = ensure(c->b_kfws, sizeof(float) * (size_t)c->S)) != hipSuccess) return e;
        if ((e = launch_fill((float*)c->b_kfws.p, 0.0f, c->S, s)) != hipSuccess) return e;
        if (n > 0)
            hipLaunchKernelGGL(pair_weight_runs_k, dim3((unsigned)std::min<int64_t>(cdiv(n, 16), 65536)), dim3(256), 0,
                               s, entry, (const uint16_t*)c->b_runmask.p, (const uint32_t*)pos, n,
                               (const uint32_t*)pstart, (const float*)c->b_kflen.p, (const double*)wsum,
                               (float*)c->b_kfws.p);
        c->kfws_ready = 1;
        return hipGetLastError();
    }
    if ((e = ensure(c->b_kfw, sizeof(float) * (size_t)(E > 0 ? E : 1))) != hipSuccess) return e;
    if (E > 0)
        hipLaunchKernelGGL(pair_weight_k, dim3(nblocks), dim3(256), 0, s, entry, (const uint32_t*)pos, E,
                           (const uint32_t*)pstart, (const float*)c->b_kflen.p, (const double*)wsum,
                           (float*)c->b_kfw.p);
    return hipGetLastError();
}

}  // namespace mrf

namespace mrf {

hipError_t export_canonical_incidence(const mrf_ctx* c, int64_t* vptr, uint32_t* vedge, hipStream_t s)
{
    hipError_t e;
    mrf_ctx* m = const_cast<mrf_ctx*>(c);
    const SceneDev* sc = (const SceneDev*)c->b_scenes.p;
    if (vptr) {
        // canonical vptr: exclusive scan of the degree of every linear voxel id
        if ((e = ensure(m->b_tmp64, sizeof(int32_t) * (size_t)(c->V + 1))) != hipSuccess) return e;
        const size_t sb = scan_tmp_bytes(c->V + 1);
        if ((e = ensure(m->b_misc, sb)) != hipSuccess) return e;
        int32_t* deg = (int32_t*)c->b_tmp64.p;
        if (c->V > 0)
            hipLaunchKernelGGL(canon_degree_k, dim3((unsigned)cdiv(c->V, 256)), dim3(256), 0, s, sc, c->n_scenes,
                               (const int64_t*)c->b_vptr.p, c->V, deg);
        if ((e = scan_rec(LoadI32{deg}, c->V, vptr, (int64_t*)m->b_misc.p, s)) != hipSuccess) return e;
    }
    if (vedge && c->E > 0) {
        // canonical vedge: stable radix sort of canonical edge ids by linear voxel id
        // (O(E) temporaries: this export is a checking facility)
        const size_t E = (size_t)c->E;
        const size_t Ep = (E + 63) & ~(size_t)63;   // 256-byte aligned sub-arrays (vector loads)
        if ((e = ensure(m->b_export, 5 * Ep * sizeof(uint32_t))) != hipSuccess) return e;
        uint32_t* keys = (uint32_t*)c->b_export.p;
        uint32_t *ka = keys + Ep, *va = keys + 2 * Ep, *kb = keys + 3 * Ep, *vb = keys + 4 * Ep;
        if ((e = export_canonical_edges(c, c->b_col.p, keys, 4, s)) != hipSuccess) return e;
        const int64_t nh = (int64_t)radix_hist_entries(c->E);
        if ((e = ensure(m->b_tmp64, sizeof(int64_t) * (size_t)(nh + 1) + sizeof(int32_t) * (size_t)nh)) != hipSuccess)
            return e;
        int64_t* offs = (int64_t*)c->b_tmp64.p;
        int32_t* hist = (int32_t*)(offs + nh + 1);
        const size_t sb2 = radix_tmp_bytes(c->E);
        if ((e = ensure(m->b_misc, sb2 > m->b_misc.cap ? sb2 : m->b_misc.cap)) != hipSuccess) return e;
        int bits = 1;
        while (bits < 31 && (int64_t(1) << bits) <= c->V - 1) ++bits;
        const int passes = bits <= 8 ? 1 : (bits + 7) / 8;
        uint32_t* kout = passes == 1 ? kb : keys;   // the first pass is the only reader of `keys`
        if ((e = radix_sort_pairs(keys, ka, va, kb, vb, kout, vedge, c->E, bits, hist, offs, m->b_misc.p,
                                  m->b_misc.cap, s)) != hipSuccess)
            return e;
    }
    return hipGetLastError();
}

hipError_t export_canonical_edges(const mrf_ctx* c, const void* in_slots, void* out, int elem_bytes, hipStream_t s)
{
    if (c->R <= 0 || c->E <= 0) return hipSuccess;
    const dim3 g((unsigned)cdiv(c->R, 256)), b(256);
    const FrameDev* fr = (const FrameDev*)c->b_frames.p;
    const SceneDev* sc = (const SceneDev*)c->b_scenes.p;
    const int64_t* tb = (const int64_t*)c->b_tbase.p;
    const int64_t* rp = (const int64_t*)c->b_rowptr.p;
    switch (elem_bytes) {
        case 1:
            hipLaunchKernelGGL(canon_edges_k<uint8_t>, g, b, 0, s, fr, c->n_frames, sc, tb, rp, c->R,
                               (const uint8_t*)in_slots, (uint8_t*)out);
            break;
        case 4:
            hipLaunchKernelGGL(canon_edges_k<uint32_t>, g, b, 0, s, fr, c->n_frames, sc, tb, rp, c->R,
                               (const uint32_t*)in_slots, (uint32_t*)out);
            break;
        case 8:
            hipLaunchKernelGGL(canon_edges_k<uint64_t>, g, b, 0, s, fr, c->n_frames, sc, tb, rp, c->R,
                               (const uint64_t*)in_slots, (uint64_t*)out);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}


// ============================================================== per-frame counts

__device__ __forceinline__ void frame_count(const FrameDev& fr, const SceneDev* scenes, const int64_t* tbase,
                                            const int64_t* rowptr, int64_t* out)
{
    const SceneDev& sd = scenes[fr.scene];
    const int64_t nt = (int64_t)fr.ntx * ((sd.H + kTileW - 1) / kTileW);
    const int64_t hw = (int64_t)sd.W * sd.H;
    out[0] = tbase[fr.tile_base + nt] - tbase[fr.tile_base];
    out[1] = rowptr[fr.ray_base + hw] - rowptr[fr.ray_base];
}

__global__ void frame_counts_k(const FrameDev* __restrict__ frames, const SceneDev* __restrict__ scenes, int nf,
                               const int64_t* __restrict__ tbase, const int64_t* __restrict__ rowptr,
                               int64_t* __restrict__ out)
{
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < nf) frame_count(frames[f], scenes, tbase, rowptr, out + 2 * f);
}

// What follows the count pass of a few rays, by one block: row pointers, tiles with their
// first slots, and every frame's slots and edges; a thread takes consecutive rays and tiles.
__device__ int64_t block1024_excl_scan(int64_t x, int64_t* wsum, int64_t* total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int64_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i < w) off += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + incl - x;
}

__global__ __launch_bounds__(1024) void count_finish_k(const SceneDev* __restrict__ scenes,
                                                       const FrameDev* __restrict__ frames, int nf,
                                                       const int32_t* __restrict__ counts, int R, int T,
                                                       int64_t* rowptr, TileDev* tiles, int64_t* tbase,
                                                       int64_t* __restrict__ out)
{
    __shared__ int64_t wsum[16];
    const int rper = (R + 1023) / 1024, tper = (T + 1023) / 1024;
    const int r0 = min((int)threadIdx.x * rper, R), r1 = min(r0 + rper, R);
    int64_t sum = 0, total;
    for (int r = r0; r < r1; ++r) sum += counts[r];
    int64_t at = block1024_excl_scan(sum, wsum, &total);
    for (int r = r0; r < r1; ++r) {
        rowptr[r] = at;
        at += counts[r];
    }
    if (threadIdx.x == 0) rowptr[R] = total;

    const int t0 = min((int)threadIdx.x * tper, T), t1 = min(t0 + tper, T);
    int f = 0;
    if (t0 < t1) {
        int hi = nf;   // tile_base of f <= t0 < that of hi
        while (hi - f > 1) {
            const int mid = (f + hi) >> 1;
            if (frames[mid].tile_base <= t0)
                f = mid;
            else
                hi = mid;
        }
    }
    sum = 0;
    for (int t = t0; t < t1; ++t) {
        while (f + 1 < nf && frames[f + 1].tile_base <= t) ++f;
        const TileDev td = tile_of(scenes[frames[f].scene], frames[f], f, t - (int)frames[f].tile_base, counts);
        tiles[t] = td;
        sum += (int64_t)kTile * td.len;
    }
    at = block1024_excl_scan(sum, wsum, &total);
    for (int t = t0; t < t1; ++t) {
        tiles[t].base = at;
        tbase[t] = at;
        at += (int64_t)kTile * tiles[t].len;
    }
    if (threadIdx.x == 0) tbase[T] = total;
    __syncthreads();   // the block's writes of rowptr and tbase
    for (int i = threadIdx.x; i < nf; i += 1024) frame_count(frames[i], scenes, tbase, rowptr, out + 2 * i);
}

// Most rays of a batch finished by one block: its time grows with them, that of the seven
// launches it replaces hardly.  Build of 256 rays 172 us and 200, of 3072 (64x48) 226 and
// 258, of 12288 266 and 282, of 16384 303 and 308.
constexpr int64_t kFinishRays = int64_t(1) << 14;

bool launch_count_finish(mrf_ctx* c, int64_t* out, hipStream_t s)
{
    if (c->R > kFinishRays || c->n_frames <= 0) return false;
    hipLaunchKernelGGL(count_finish_k, dim3(1), dim3(1024), 0, s, (const SceneDev*)c->b_scenes.p,
                       (const FrameDev*)c->b_frames.p, c->n_frames, (const int32_t*)c->b_counts.p, (int)c->R,
                       (int)c->T, (int64_t*)c->b_rowptr.p, (TileDev*)c->b_tiles.p, (int64_t*)c->b_tbase.p, out);
    return true;
}

hipError_t launch_frame_counts(const mrf_ctx* c, int64_t* out, hipStream_t s)
{
    if (c->n_frames <= 0) return hipSuccess;
    hipLaunchKernelGGL(frame_counts_k, dim3((unsigned)cdiv(c->n_frames, 256)), dim3(256), 0, s,
                       (const FrameDev*)c->b_frames.p, (const SceneDev*)c->b_scenes.p, c->n_frames,
                       (const int64_t*)c->b_tbase.p, (const int64_t*)c->b_rowptr.p, out);
    return hipGetLastError();
}

// ============================================================== accuracy metric

// Sec. III-D: a voxel is a region of constant occlusion density alpha, chosen
// so that crossing one voxel side h blocks a ray with the voxel's occupancy
// probability: alpha = -ln(1 - p) / h = softplus(L) / h for log-odds L.  Per
// voxel of one scene, FP64: (alpha, log alpha), one 16-byte gather per step.
__global__ void metric_alpha_k(const float* __restrict__ logit, int64_t n, double inv_h, double2* __restrict__ alpha)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = (double)logit[i];
        const double sp = (x > 0.0 ? x : 0.0) + log1p(exp(-fabs(x)));
        const double a = sp * inv_h;
        alpha[i] = make_double2(a, log(a));
    }
}

// Along a ray (Euclidean length s) vis(s) = exp(-integral of alpha) and the
// density of the generating surface omega(s) = alpha(s) vis(s) decays inside
// a voxel, so its maximum is at the entry of the voxel maximising
// log alpha_n - sum_{i<n} alpha_i l_i (the first on ties).
struct MetricEmit {
    const double2* alpha;    // of the scene's voxels
    double wn;               // |w|: Euclidean length per unit of z-depth
    double acc = 0.0;        // sum of alpha_i l_i so far
    double best = -__builtin_huge_val();
    double btin = 0.0, btout = 0.0;

    __device__ void operator()(int, int, int, int, int lin, double tin, double tout)
    {
        const double2 al = alpha[lin];
        const double a = al.x;
        const double lw = al.y - acc;
        if (lw > best) {
            best = lw;
            btin = tin;
            btout = tout;
        }
        acc += a * ((tout - tin) * wn);
    }
};

// One thread per pixel of one frame (blockIdx.y): the ray clipped to the grid
// box and walked to the grid exit.  Exit visibility of at least vis_min (log:
// lvmin) means the map leaves the ray visible, and the ray is accurate iff its
// measurement lies beyond the exit; otherwise iff the measurement lies inside
// the chord [t_in, t_out) of the voxel of the most likely surface, or, with
// tol > 0 (the paper's evaluation rule), iff that surface (the voxel's entry)
// lies within tol sigma(Z) of Z, sigma(Z) = max(c0 + c2 Z^2, smin).  The
// measurement is the built frame's, or ref[global ray] when ref is given
// (e.g. noise-free depth from the same poses).  code: 1
// accurate, 0 not, -1 not evaluated; surf: z-depth of the chosen voxel's
// entry, +inf when the surface is taken to lie beyond the map, NaN when not
// evaluated.  Per-scene counts (evaluated, accurate) by block counts and one
// atomic per block.
__global__ __launch_bounds__(256) void accuracy_k(const SceneDev* __restrict__ scenes,
                                                  const FrameDev* __restrict__ frames, BuildDev bp,
                                                  const double2* __restrict__ alpha, double lvmin,
                                                  const float* __restrict__ ref, double tol,
                                                  int8_t* __restrict__ code, double* __restrict__ surf,
                                                  unsigned long long* __restrict__ counts)
{
    const FrameDev fr = frames[blockIdx.y];
    const SceneDev& sd = scenes[fr.scene];
    int ev = 0, ok = 0, u, v;
    if (block_pixel(sd, blockIdx.x, threadIdx.x, u, v)) {
        const int pix = v * sd.W + u;
        Ray r;
        double ts, texit;
        int8_t cd = -1;
        double sf = __builtin_nan("");
        const float zm = ref ? ref[fr.ray_base + pix] : fr.depth[pix];
        if (clip_ray(sd, bp, fr.T, zm, v, u, r, ts, texit) && ts < texit) {
            r.ts = ts;
            r.te = texit;
            MetricEmit m;
            m.alpha = alpha + sd.voxel_base;
            m.wn = sqrt(r.w[0] * r.w[0] + r.w[1] * r.w[1] + r.w[2] * r.w[2]);
            walk_dense(sd, r, m);   // the metric walks the whole grid
            if (-m.acc >= lvmin) {
                cd = r.Z > texit ? 1 : 0;
                sf = __builtin_huge_val();
            } else if (tol > 0.0) {
                double sig = bp.c2 * r.Z;
                sig = sig * r.Z;
                sig = bp.c0 + sig;
                if (sig < bp.smin) sig = bp.smin;
                cd = fabs(m.btin - r.Z) <= tol * sig ? 1 : 0;
                sf = m.btin;
            } else {
                cd = (m.btin <= r.Z && r.Z < m.btout) ? 1 : 0;
                sf = m.btin;
            }
            ev = 1;
            ok = cd;
        }
        const int64_t gr = fr.ray_base + pix;
        if (code) code[gr] = cd;
        if (surf) surf[gr] = sf;
    }
    const int nev = __syncthreads_count(ev);
    const int nok = __syncthreads_count(ok);
    if (counts && threadIdx.x == 0 && nev > 0) {
        atomicAdd(&counts[2 * fr.scene], (unsigned long long)nev);
        atomicAdd(&counts[2 * fr.scene + 1], (unsigned long long)nok);
    }
}

hipError_t launch_accuracy(mrf_ctx* c, const float* logit, double vis_min, const float* ref, double tol,
                           int8_t* code, double* surf, int64_t* counts, double* work, hipStream_t s)
{
    double2* alpha = (double2*)work;
    for (const SceneDev& sd : c->scenes_h) {
        const int64_t n = (int64_t)sd.n[0] * sd.n[1] * sd.n[2];
        int64_t b = (n + 255) / 256;
        if (b > 65536) b = 65536;
        hipLaunchKernelGGL(metric_alpha_k, dim3((unsigned)b), dim3(256), 0, s, logit + sd.voxel_base, n, 1.0 / sd.h,
                           alpha + sd.voxel_base);
    }
    if (counts) {
        hipError_t e = launch_fill_u32((uint32_t*)counts, 0u, 4 * (int64_t)c->n_scenes, s);
        if (e != hipSuccess) return e;
    }
    const dim3 grid(pixel_blocks(c), c->n_frames);
    hipLaunchKernelGGL(accuracy_k, grid, dim3(256), 0, s, (const SceneDev*)c->b_scenes.p,
                       (const FrameDev*)c->b_frames.p, c->bp, (const double2*)alpha, std::log(vis_min), ref, tol, code,
                       surf, (unsigned long long*)counts);
    return hipGetLastError();
}

// ------------------------------------------------------------ static scratch
//
// The accuracy metric's per-voxel alpha and log alpha for callers that cannot
// allocate device memory (mrf_accuracy_static): a file-scope device array of
// kStaticMetricVoxels voxels (two doubles each, 32 MiB), one copy per GPU,
// held until the process ends.  Host code never passes the array's name to a
// kernel (on the host it is a stand-in, not a device address): its device
// address is looked up once per device, with that device current, and kept.
static __device__ __align__(256) double scratch[2 * kStaticMetricVoxels];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {nullptr};
hipError_t g_scratch_err[kMaxDevices] = {hipSuccess};
bool g_scratch_done[kMaxDevices] = {false};
}  // namespace

hipError_t static_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_done[device]) {
        void* ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));   // the current device's copy
        g_scratch_ptr[device] = e == hipSuccess ? (double*)ptr : nullptr;
        g_scratch_err[device] = e;
        g_scratch_done[device] = true;
        if (e != hipSuccess) hipGetLastError();
    }
    return g_scratch_err[device];
}

hipError_t static_scratch(int device, double** out)
{
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_done[device]) return hipErrorNotInitialized;
    *out = g_scratch_ptr[device];
    return g_scratch_err[device];
}

}  // namespace mrf
