// Forward message passing on gfx950 (Sec. III-B/C, IV-A of MRFMap).
//
// Messages to binary occupancy variables are log-odds, so every message is
// normalised by construction (supplement, Sec. II-A).  Per edge e (one ray
// crossing one voxel):
//   lam_e  voxel -> ray factor  (Eq. node_to_factor: prior plus every other
//          ray's message into the voxel)
//   ell_e  ray factor -> voxel  (Eqs. pos and neg)
//   g_e    log nu(d_e) = log N(Z; d_e, sigma(d_e))   (Eq. noise)
//
// Voxel phase: per touched voxel the total tot_v = theta_v + sum of every
// incoming ray message, a fixed-order FP64 reduction over its edge list kept
// as the FP32 pair (hi, lo).  Eq. node_to_factor (every incoming message but
// the receiving ray's own) is then lam_e = (hi_v(e) - ell_e) + lo_v(e), which
// the ray kernels form as they stage their tiles: no per-edge scatter.  When
// the edge's own message is most of the total (a message of 1e9 against
// others summing to a few units), hi - ell_e is exact and lam_e keeps the
// accuracy of the FP64 sum.
// Ray phase: one group of lanes per ray.  With P_i = sum_{k<i} log mu_k(0),
//   S_i = LSE_{j<i} (log mu_j(1) + g_j + P_j)
//   Q_i = LSE(log mu_{i+1}(1) + g_{i+1}, log mu_{i+1}(0) + Q_{i+1})
//   ell_i = LSE(S_i, g_i + P_i) - LSE(S_i, P_i + Q_i)
// is Eq. pos over Eq. neg with the second sum of Eq. neg in its division-free
// form (sum over j > i of the product over k < j, k != i).  The kernels carry
// R_i = S_i - P_i instead of S and P (see ray_body).
#include <hip/hip_runtime.h>

#include <array>
#include <utility>

#include "dev_common.hpp"
#include "mrf_internal.hpp"
#include "tile_lds.hpp"

namespace mrf {

static inline unsigned nblk(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// ------------------------------------------------------------ elementwise

__global__ void fill_k(float* __restrict__ p, float v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void copy_k(float* __restrict__ d, const float* __restrict__ s, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = s[i];
}

__global__ void excl_k(const int32_t* __restrict__ col, ExclDev x, float* __restrict__ out, int64_t E)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E; i += (int64_t)gridDim.x * blockDim.x)
    {
        const int32_t v = col[i];
        out[i] = excl_value(v, x.tot[v < 0 ? 0 : v], x.own[i], x.has_own);
    }
}

__global__ void marginals_k(const float* __restrict__ L, float* __restrict__ p, float* __restrict__ logit, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float l = L[i];
        if (p) p[i] = 1.0f / (1.0f + __expf(-l));
        if (logit) logit[i] = l;
    }
}

// An inference's inputs in one launch instead of six copies of 2 us each: the prior
// (as theta, as the first sweep's total pairs and as the beliefs of voxels that no ray
// touches) and the sensor tables (bias null: zero).
__global__ void infer_inputs_k(const float* __restrict__ prior, int64_t V, float* __restrict__ theta,
                               float2* __restrict__ theta2, float* __restrict__ L, const float* __restrict__ sigma_in,
                               const float* __restrict__ bias_in, int64_t nt, float* __restrict__ sigma,
                               float* __restrict__ bias)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
        const float x = prior[i];
        theta[i] = x;
        theta2[i] = make_float2(x, 0.0f);
        L[i] = x;
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nt; i += stride) {
        sigma[i] = sigma_in[i];
        bias[i] = bias_in ? bias_in[i] : 0.0f;
    }
}

// The reverse pass's seed d loss / d L: the start of d / d theta, and as total pairs
__global__ void reverse_seed_k(const float* __restrict__ dlogit, float* __restrict__ thetabar,
                               float2* __restrict__ seed, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float x = dlogit[i];
        thetabar[i] = x;
        seed[i] = make_float2(x, 0.0f);
    }
}

// g_e = log N(Z; d_e + mu_b, sigma_b) = -((delta_e - mu_b) / sigma_b)^2 / 2 -
// log sigma_b - log(2 pi) / 2, delta_e = Z - d_e, mu_b the learnt depth bias
// (the predicted mean measurement at depth d is d + mu(d)).  A lane takes 4
// consecutive slots and consecutive lanes consecutive groups, so every load
// (4 bins, 4 deltas) and store (4 g) instruction of a wave covers one
// contiguous run; S is a multiple of 16, so a group lies wholly inside or
// outside [0, S).  Grid-stride, so each block builds its tables once.
// Padding slots (bin 255) are left as they are.
__device__ __forceinline__ float potential(float delta, float inv, float cst, float mu)
{
    const float x = (delta - mu) * inv;   // residual about the predicted mean d + mu
    return -0.5f * x * x - cst;
}

constexpr int kPotGroups = 4;   // potentials: groups of 4 slots in flight per lane

__global__ __launch_bounds__(256) void potentials_k(const float* __restrict__ delta, const uint8_t* __restrict__ bin,
                                                    int64_t S, const float* __restrict__ sigma,
                                                    const float* __restrict__ bias, float* __restrict__ g)
{
    __shared__ float inv[kBins], cst[kBins], mu[kBins];
    if (threadIdx.x < kBins) {
        const float s = sigma[threadIdx.x];
        inv[threadIdx.x] = 1.0f / s;
        cst[threadIdx.x] = logf(s) + 0.91893853320467274f;
        mu[threadIdx.x] = bias[threadIdx.x];
    }
    __syncthreads();
    const int64_t ng = S / 4;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g0 = (int64_t)blockIdx.x * blockDim.x * kPotGroups + threadIdx.x; g0 < ng;
         g0 += stride * kPotGroups) {
        uint32_t bw[kPotGroups];
        float4 dv[kPotGroups];
#pragma unroll
        for (int u = 0; u < kPotGroups; ++u) {
            const int64_t gi = g0 + (int64_t)u * blockDim.x;
            const int64_t at = gi < ng ? gi : ng - 1;
            bw[u] = ((const uint32_t*)bin)[at];
            dv[u] = ((const float4*)delta)[at];
        }
#pragma unroll
        for (int u = 0; u < kPotGroups; ++u) {
            const int64_t gi = g0 + (int64_t)u * blockDim.x;
            if (gi >= ng) break;
            float out[4];
            bool all = true;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int b = (int)((bw[u] >> (8 * j)) & 255u);
                const float dj = j == 0 ? dv[u].x : j == 1 ? dv[u].y : j == 2 ? dv[u].z : dv[u].w;
                const int bb = b < kBins ? b : 0;
                out[j] = potential(dj, inv[bb], cst[bb], mu[bb]);
                all = all && b < kBins;
            }
            if (all) {
                ((float4*)g)[gi] = make_float4(out[0], out[1], out[2], out[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (((bw[u] >> (8 * j)) & 255u) < kBins) g[4 * gi + j] = out[j];
            }
        }
    }
}

// potentials_k with per-region tables: one block per tile (grid-stride), the
// region's row staged in LDS, the tile's 16 len slots in groups of 4 with the
// same arithmetic as potentials_k.
__global__ __launch_bounds__(256) void potentials_cells_k(const TileDev* __restrict__ tiles, int64_t T,
                                                          const FrameDev* __restrict__ frames, int cp,
                                                          const float* __restrict__ delta,
                                                          const uint8_t* __restrict__ bin,
                                                          const float* __restrict__ sigma,
                                                          const float* __restrict__ bias, float* __restrict__ g)
{
    __shared__ float inv[kBins], cst[kBins], mu[kBins];
    for (int64_t ti = blockIdx.x; ti < T; ti += gridDim.x) {
        const TileDev t = tiles[ti];
        const int64_t row = tile_cell(t, frames, cp) * kBins;
        __syncthreads();   // the previous tile's readers are done
        if (threadIdx.x < kBins) {
            const float s = sigma[row + threadIdx.x];
            inv[threadIdx.x] = 1.0f / s;
            cst[threadIdx.x] = logf(s) + 0.91893853320467274f;
            mu[threadIdx.x] = bias[row + threadIdx.x];
        }
        __syncthreads();
        const int64_t g0 = t.base / 4, ng = 4 * (int64_t)t.len;
        for (int64_t k = threadIdx.x; k < ng; k += blockDim.x) {
            const int64_t gi = g0 + k;
            const uint32_t bw = ((const uint32_t*)bin)[gi];
            const float4 dv = ((const float4*)delta)[gi];
            float out[4];
            bool all = true;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int b = (int)((bw >> (8 * j)) & 255u);
                const float dj = j == 0 ? dv.x : j == 1 ? dv.y : j == 2 ? dv.z : dv.w;
                const int bb = b < kBins ? b : 0;
                out[j] = potential(dj, inv[bb], cst[bb], mu[bb]);
                all = all && b < kBins;
            }
            if (all) {
                ((float4*)g)[gi] = make_float4(out[0], out[1], out[2], out[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (((bw >> (8 * j)) & 255u) < kBins) g[4 * gi + j] = out[j];
            }
        }
    }
}

static unsigned grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    return (unsigned)(b > 0 ? b : 1);
}

hipError_t launch_fill(float* p, float v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_k, dim3(grid_for(n)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_copy(float* d, const float* src, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_k, dim3(grid_for(n)), dim3(256), 0, s, d, src, n);
    return hipGetLastError();
}

hipError_t launch_infer_inputs(mrf_ctx* c, const float* prior, const float* sigma, const float* bias, hipStream_t s)
{
    const int64_t nt = table_entries(c);
    hipLaunchKernelGGL(infer_inputs_k, dim3(grid_for(c->V > nt ? c->V : nt)), dim3(256), 0, s, prior, c->V,
                       (float*)c->b_theta.p, (float2*)c->b_theta2.p, (float*)c->b_L.p, sigma, bias, nt,
                       (float*)c->b_sigma.p, (float*)c->b_bias.p);
    return hipGetLastError();
}

hipError_t launch_reverse_seed(const float* dlogit, float* thetabar, float2* seed, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(reverse_seed_k, dim3(grid_for(n)), dim3(256), 0, s, dlogit, thetabar, seed, n);
    return hipGetLastError();
}

hipError_t launch_excl(const mrf_ctx* c, ExclSrc x, float* out, hipStream_t s)
{
    if (c->S <= 0) return hipSuccess;
    hipLaunchKernelGGL(excl_k, dim3(grid_for(c->S)), dim3(256), 0, s, (const int32_t*)c->b_col.p, excl_dev(c, x),
                       out, c->S);
    return hipGetLastError();
}

hipError_t launch_marginals(const float* L, float* p, float* logit, int64_t n, hipStream_t s)
{
    if (n <= 0 || (!p && !logit)) return hipSuccess;
    hipLaunchKernelGGL(marginals_k, dim3(grid_for(n)), dim3(256), 0, s, L, p, logit, n);
    return hipGetLastError();
}

hipError_t launch_potentials(mrf_ctx* c, hipStream_t s)
{
    if (c->S <= 0) return hipSuccess;
    ProfScope ps(c, KID_POT, s);
    if (c->cell_px > 0) {
        const int64_t blocks = c->T < 65536 ? c->T : 65536;
        hipLaunchKernelGGL(potentials_cells_k, dim3((unsigned)blocks), dim3(256), 0, s, (const TileDev*)c->b_tiles.p,
                           c->T, (const FrameDev*)c->b_frames.p, c->cell_px, (const float*)c->b_delta.p,
                           (const uint8_t*)c->b_bin.p, (const float*)c->b_sigma.p, (const float*)c->b_bias.p,
                           (float*)c->b_g.p);
        return hipGetLastError();
    }
    int64_t blocks = nblk(c->S / 4, 256 * kPotGroups);
    if (blocks > 4096) blocks = 4096;   // grid-stride over at most 16 blocks per CU
    hipLaunchKernelGGL(potentials_k, dim3((unsigned)blocks), dim3(256), 0, s, (const float*)c->b_delta.p,
                       (const uint8_t*)c->b_bin.p, c->S, (const float*)c->b_sigma.p,
                       (const float*)c->b_bias.p, (float*)c->b_g.p);
    return hipGetLastError();
}

// ------------------------------------------------------------ voxel phase
//
// The voxel phase reduces: for every touched voxel v, sum_v = the sum of its
// incoming per-edge values (ray messages forward, d/d lambda in reverse), in a
// fixed order and in FP64 (every FP32 term is exact there), written as VoxOut
// describes.  The voxel -> ray message of edge e is then formed from the total
// pair and the edge's own term by the ray kernels as they stage their tiles
// (no per-edge scatter here).

__device__ __forceinline__ void vox_store(uint32_t v, double sum, const VoxOut& o)
{
    const double t = (o.base ? (double)o.base[v] : 0.0) + sum;
    if (o.tot2) o.tot2[v] = split_pair(t);
    if (o.totf) o.totf[v] = (float)t;
    if (o.acc) o.acc[v] += (float)sum;
    if (o.dsum) o.dsum[v] = sum;
}

// How a segment (a voxel's edge list, or a keyframe pair's) is summed, by class:
//   0, 1  at most G = 16 or 32 edges: 64 / G lane groups per wave, each walking
//         kVoxVPW consecutive segments (lane l holds edge l of each);
//   2..5  at most 64, 128, 256, 1024 edges: one wave walks kVoxVPW consecutive
//         segments, 64 edges a round;
//   6     at most 4096: the four waves of a block, 1024 edges each;
//   7     more: pieces of 4096 edges (b_*_hub), each summed as a class-6 segment
//         into psum, then added in order by hub_sum_k.
// Every class issues all its loads before the first wait (indices clamped inside
// the list): the phase waits on its gathers, so bytes in flight count.  Segments
// come in brick-major order and each XCD takes a contiguous range of a class's
// blocks.  All classes run in one launch, the longest first: with a launch each, a
// 640x480 frame's sweep spent 144 us in ten kernels that each drained before the
// next, 63 of them in one 1024-thread block walking the camera's voxel (3e5 edges);
// one launch with the hubs in pieces takes 47 us, and at 5e8 edges 1.13 ms (3.6 TB/s of
// list and messages) instead of 1.19.  Eight waves per SIMD are asked for where the
// registers allow it without spills: with the 82 registers that the compiler takes by
// itself the unweighted kernel runs 1.27 ms.

template <int G, int VPG, bool WT, bool MG>
__device__ __forceinline__ void seg_group(int64_t lb, const VoxDev* __restrict__ vd, int64_t n,
                                          const uint32_t* __restrict__ vedge, const float* __restrict__ in,
                                          const VoxOut& out, const float* __restrict__ w, const SlotGroups& sg)
{
    constexpr int GPB = 256 / G;   // groups per block
    if (lb * GPB * VPG >= n) return;   // whole block
    const int64_t v0 = (lb * GPB + (int)threadIdx.x / G) * VPG;
    const int l = (int)threadIdx.x % G;
    VoxDev d[VPG];
#pragma unroll
    for (int u = 0; u < VPG; ++u) d[u] = vd[min(v0 + u, n - 1)];   // past the list: a repeat, not stored
    uint32_t e[VPG];
    float x[VPG], wt[VPG];
#pragma unroll
    for (int u = 0; u < VPG; ++u) e[u] = vedge[d[u].start + min(l, d[u].m - 1)];
    if constexpr (WT) {
#pragma unroll
        for (int u = 0; u < VPG; ++u) wt[u] = w[d[u].start + min(l, d[u].m - 1)];
    }
#pragma unroll
    for (int u = 0; u < VPG; ++u) x[u] = in[(MG ? group_slot_base(sg, d[u].start) : 0) + e[u]];
#pragma unroll
    for (int u = 0; u < VPG; ++u) {
        const double t = WT ? (double)x[u] * (double)wt[u] : (double)x[u];
        const double sum = dgroup_sum_d<G>(l < d[u].m ? t : 0.0);   // at group lane 0
        if (l == 0 && v0 + u < n) vox_store(d[u].v, sum, out);
    }
}

constexpr int kSegRed = 8 * 64;   // doubles of LDS per wave

template <int IPL, int VPW, bool WT, bool MG>
__device__ __forceinline__ void seg_wave(int64_t lb, const VoxDev* __restrict__ vd, int64_t n,
                                         const uint32_t* __restrict__ vedge, const float* __restrict__ in,
                                         const VoxOut& out, const float* __restrict__ w, const SlotGroups& sg,
                                         double* red)
{
    // the wave index is uniform across the wave: said so, the descriptors below
    // become scalar loads and their address and group arithmetic scalar
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int64_t v0 = (lb * 4 + wv) * VPW;
    if (v0 >= n) return;   // whole wave
    VoxDev d[VPW];
#pragma unroll
    for (int u = 0; u < VPW; ++u) d[u] = vd[min(v0 + u, n - 1)];   // past the list: a repeat, not stored
    uint32_t e[VPW][IPL];
    float x[VPW][IPL], wt[VPW][IPL];
#pragma unroll
    for (int u = 0; u < VPW; ++u)
#pragma unroll
        for (int k = 0; k < IPL; ++k) e[u][k] = vedge[d[u].start + min(k * 64 + l, d[u].m - 1)];
    if constexpr (WT) {
#pragma unroll
        for (int u = 0; u < VPW; ++u)
#pragma unroll
            for (int k = 0; k < IPL; ++k) wt[u][k] = w[d[u].start + min(k * 64 + l, d[u].m - 1)];
    }
#pragma unroll
    for (int u = 0; u < VPW; ++u) {
        const float* ing = in + (MG ? group_slot_base(sg, d[u].start) : 0);
#pragma unroll
        for (int k = 0; k < IPL; ++k) x[u][k] = ing[e[u][k]];
    }
    double a[VPW];
#pragma unroll
    for (int u = 0; u < VPW; ++u) {
        a[u] = 0.0;
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            const double t = WT ? (double)x[u][k] * (double)wt[u][k] : (double)x[u][k];
            a[u] += k * 64 + l < d[u].m ? t : 0.0;
        }
    }
    if constexpr (VPW == 1) {
        const double t = dgroup_sum_d<64>(a[0]);
        if (l == 0) vox_store(d[0].v, t, out);
    } else {
        // the wave's VPW x 64 lane sums transposed through LDS: segment u goes to
        // the LG = 64 / VPW lanes [u LG, (u + 1) LG), lane p of them adding the
        // sums of lanes [p VPW, (p + 1) VPW) in order, then a group sum over the LG
        // lanes (one reduction for all segments)
        constexpr int LG = 64 / VPW;
        static_assert((LG == 8 || LG == 16) && VPW * 64 <= kSegRed, "four or eight segments per wave");
        double* r = red + wv * kSegRed;
#pragma unroll
        for (int u = 0; u < VPW; ++u) r[u * 64 + l] = a[u];
        // LDS accesses of one wave complete in order: the fences only keep the
        // compiler from moving the reads above the writes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int u = l / LG, p = l % LG;
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < VPW; ++j) t += r[u * 64 + p * VPW + j];
        t = dgroup_sum_d<LG>(t);   // at the group's first lane
        if (p == 0 && v0 + u < n) vox_store(vd[v0 + u].v, t, out);
    }
}

// one segment of at most 4096 edges by the block's four waves
template <bool WT, bool MG>
__device__ __forceinline__ void seg_block(int64_t lb, const VoxDev* __restrict__ vd, int64_t n,
                                          const uint32_t* __restrict__ vedge, const float* __restrict__ in,
                                          const VoxOut& out, const float* __restrict__ w, const SlotGroups& sg,
                                          double* red)
{
    constexpr int IPL = kSegPiece / 256;
    if (lb >= n) return;   // whole block
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const VoxDev d = vd[lb];
    const float* ing = in + (MG ? group_slot_base(sg, d.start) : 0);
    const int base = wv * 64 * IPL;
    uint32_t e[IPL];
    float x[IPL], wt[IPL];
#pragma unroll
    for (int k = 0; k < IPL; ++k) e[k] = vedge[d.start + min(base + k * 64 + l, d.m - 1)];
    if constexpr (WT) {
#pragma unroll
        for (int k = 0; k < IPL; ++k) wt[k] = w[d.start + min(base + k * 64 + l, d.m - 1)];
    }
#pragma unroll
    for (int k = 0; k < IPL; ++k) x[k] = ing[e[k]];
    double a = 0.0;
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const double t = WT ? (double)x[k] * (double)wt[k] : (double)x[k];
        a += base + k * 64 + l < d.m ? t : 0.0;
    }
    a = dgroup_sum_d<64>(a);
    if (l == 0) red[wv] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int q = 0; q < 4; ++q) tot += red[q];
        vox_store(d.v, tot, out);
    }
}

// Work of one launch: class k's segments are desc[off[k], off[k] + cnt[k]) (class 7:
// the hub pieces), its blocks [blk[k], blk[k + 1]) counted from class 7 downwards;
// every blk is a multiple of 8, so a block's XCD is that of its place in the class.
struct SegWork {
    const VoxDev* desc;
    const VoxDev* pieces;
    double* psum;
    int64_t off[kVoxClasses], cnt[kVoxClasses];
    uint32_t blk[kVoxClasses + 1];
};

template <bool WT, bool MG>
__global__ __launch_bounds__(256, WT ? 6 : 8) void seg_sum_k(const SegWork s, const uint32_t* __restrict__ vedge,
                                                             const float* __restrict__ in, VoxOut out,
                                                             const float* __restrict__ w, const SlotGroups sg)
{
    __shared__ double red[4 * kSegRed];
    int k = kVoxClasses - 1;   // uniform: the class whose blocks hold this one
    while (k > 0 && blockIdx.x >= s.blk[kVoxClasses - k]) --k;
    const uint32_t b0 = s.blk[kVoxClasses - 1 - k], nb = s.blk[kVoxClasses - k] - b0;
    const int64_t lb = xcd_block(blockIdx.x - b0, nb);
    const VoxDev* d = s.desc + s.off[k];
    const int64_t n = s.cnt[k];
    switch (k) {
        case 0: seg_group<kVoxCap[0], kVoxVPW[0], WT, MG>(lb, d, n, vedge, in, out, w, sg); break;
        case 1: seg_group<kVoxCap[1], kVoxVPW[1], WT, MG>(lb, d, n, vedge, in, out, w, sg); break;
        case 2: seg_wave<kVoxCap[2] / 64, kVoxVPW[2], WT, MG>(lb, d, n, vedge, in, out, w, sg, red); break;
        case 3: seg_wave<kVoxCap[3] / 64, kVoxVPW[3], WT, MG>(lb, d, n, vedge, in, out, w, sg, red); break;
        case 4: seg_wave<kVoxCap[4] / 64, kVoxVPW[4], WT, MG>(lb, d, n, vedge, in, out, w, sg, red); break;
        case 5: seg_wave<kVoxCap[5] / 64, kVoxVPW[5], WT, MG>(lb, d, n, vedge, in, out, w, sg, red); break;
        case 6: seg_block<WT, MG>(lb, d, n, vedge, in, out, w, sg, red); break;
        default: {
            const VoxOut po{nullptr, nullptr, nullptr, nullptr, s.psum};
            seg_block<WT, MG>(lb, s.pieces, n, vedge, in, po, w, sg, red);
        }
    }
}

// the hubs' sums from their pieces' (one wave a hub: lane l adds pieces l, l + 64, ...
// in order, then the lanes)
__global__ __launch_bounds__(256) void hub_sum_k(const VoxDev* __restrict__ hubs, int64_t n,
                                                 const double* __restrict__ psum, VoxOut out)
{
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;   // whole wave
    const int l = threadIdx.x & 63;
    const VoxDev d = hubs[i];
    double a = 0.0;
    for (int p = l; p < d.m; p += 64) a += psum[d.start + p];
    a = dgroup_sum_d<64>(a);
    if (l == 0) vox_store(d.v, a, out);
}

// ------------------------------------------------------------ voxel phase over runs
//
// Large graphs keep the voxel -> ray lists as runs (a row of 16 slots, the mask of its
// lanes that lie in the voxel): 6 bytes for the 8 to 12 edges of a run where the
// list of edges takes 4 each, and a run's messages are one 64-byte line, loaded by 16
// lanes at once instead of gathered.  A 16-lane group takes 16 runs at a time: lane l
// loads run l's row and mask, and step j broadcasts run j's to the group (a DPP move),
// whose lane l then loads message l of that row and adds it if its bit is set.  By
// class (number of runs):
//   0  at most 4: four segments per group;   1  at most 8: two per group;
//   2  at most 16: one per group, two in turn;   3  at most 32: one per half-wave, two in turn;
//   4  at most 64: one per wave, two in turn;   5  at most 256: one per wave;
//   6  at most 1024: the four waves of a block;   7  more: pieces of 1024 runs.
// Bound by HBM: 5e8 edges (8 VGA frames at 2 cm) in 0.84 ms where seg_sum_k takes
// 1.13, 1.3e8 (3 rooms) in 0.173 and 0.275.  With weights (keyframe pairs) a run takes a
// second line: 1e8 edges in 0.39 ms where the sums without weights take 0.21; sweeps and
// their reverse 3.72 ms against 3.76 by the list of edges.

template <int J>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + J, 0xF, 0xF, false);   // row_newbcast:J
}

// Messages of the group's 16 runs: x[j] = lane l's message of run j
template <int... J>
__device__ __forceinline__ void run_load(const float* __restrict__ in, uint32_t row, float (&x)[16],
                                         std::integer_sequence<int, J...>)
{
    const int l = threadIdx.x & 15;
    ((x[J] = in[(uint64_t)row_bcast<J>(row) * kTile + l]), ...);
}

// a[J / PER] += the messages whose mask bit is set (WT: each times its weight)
template <int PER, bool WT, int N, int... J>
__device__ __forceinline__ void run_add(uint32_t mask, const float (&x)[16], const float (&w)[WT ? 16 : 1],
                                        double (&a)[N], std::integer_sequence<int, J...>)
{
    const int l = threadIdx.x & 15;
    ((a[J / PER] += (row_bcast<J>(mask) >> l) & 1u ? (WT ? (double)x[J] * (double)w[WT ? J : 0] : (double)x[J]) : 0.0),
     ...);
}

constexpr auto kRunSteps = std::make_integer_sequence<int, 16>{};

// classes 0 and 1: 16 / PER segments of at most PER runs per group
template <int PER, bool WT>
__device__ __forceinline__ void run_parts(int64_t lb, const VoxDev* __restrict__ vd, int64_t n,
                                          const uint32_t* __restrict__ rows, const uint16_t* __restrict__ masks,
                                          const float* __restrict__ in, const float* __restrict__ w,
                                          const VoxOut& out)
{
    constexpr int NS = 16 / PER;
    const int l = threadIdx.x & 15, q = l % PER;
    const int64_t vi = (lb * 16 + (int)(threadIdx.x >> 4)) * NS + l / PER;
    const VoxDev d = vd[min(vi, n - 1)];   // past the list: a repeat, not stored
    const int64_t at = d.start + min(q, d.m - 1);
    const uint32_t row = rows[at];
    const uint32_t mask = vi < n && q < d.m ? masks[at] : 0u;
    float x[16], wx[WT ? 16 : 1];
    run_load(in, row, x, kRunSteps);
    if constexpr (WT) run_load(w, row, wx, kRunSteps);
    double a[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) a[u] = 0.0;
    run_add<PER, WT>(mask, x, wx, a, kRunSteps);
    double t = 0.0;   // at the segment's first lane
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const double s = __shfl(dgroup_sum_d<16>(a[u]), 0, 16);
        t = l / PER == u ? s : t;
    }
    if (q == 0 && vi < n) vox_store(d.v, t, out);
}

// classes 2 to 4: one segment of at most G runs per G lanes, two in turn (weighted: one,
// for the registers that its weights take)
template <int G, bool WT>
__device__ __forceinline__ void run_group(int64_t lb, const VoxDev* __restrict__ vd, int64_t n,
                                          const uint32_t* __restrict__ rows, const uint16_t* __restrict__ masks,
                                          const float* __restrict__ in, const float* __restrict__ w,
                                          const VoxOut& out)
{
    constexpr int U = WT ? 1 : 2;
    const int64_t v0 = (lb * (256 / G) + (int)(threadIdx.x / G)) * U;
    const int l = threadIdx.x & (G - 1);
    VoxDev d[U];
    uint32_t row[U], mask[U];
    float x[U][16], wx[U][WT ? 16 : 1];
#pragma unroll
    for (int u = 0; u < U; ++u) d[u] = vd[min(v0 + u, n - 1)];   // past the list: a repeat, not stored
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t at = d[u].start + min(l, d[u].m - 1);
        row[u] = rows[at];
        mask[u] = l < d[u].m ? masks[at] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        run_load(in, row[u], x[u], kRunSteps);
        if constexpr (WT) run_load(w, row[u], wx[u], kRunSteps);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        double a[1] = {0.0};
        run_add<16, WT>(mask[u], x[u], wx[u], a, kRunSteps);
        const double t = dgroup_sum_d<G>(a[0]);
        if (l == 0 && v0 + u < n) vox_store(d[u].v, t, out);
    }
}

// 64 runs of a segment by a wave, lane i holding run base + i
template <bool WT>
__device__ __forceinline__ double run_wave64(int64_t start, int m, int base, const uint32_t* __restrict__ rows,
                                             const uint16_t* __restrict__ masks, const float* __restrict__ in,
                                             const float* __restrict__ w)
{
    const int i = base + (int)(threadIdx.x & 63);
    const int64_t at = start + min(i, m - 1);
    const uint32_t row = rows[at];
    const uint32_t mask = i < m ? masks[at] : 0u;
    float x[16], wx[WT ? 16 : 1];
    run_load(in, row, x, kRunSteps);
    if constexpr (WT) run_load(w, row, wx, kRunSteps);
    double a[1] = {0.0};
    run_add<16, WT>(mask, x, wx, a, kRunSteps);
    return a[0];
}

// runs [base, base + 256) of a segment by a wave
template <bool WT>
__device__ __forceinline__ double run_wave256(const VoxDev& d, int base, const uint32_t* __restrict__ rows,
                                              const uint16_t* __restrict__ masks, const float* __restrict__ in,
                                              const float* __restrict__ w)
{
    double a = 0.0;
    for (int t = base; t < base + 256 && t < d.m; t += 64) a += run_wave64<WT>(d.start, d.m, t, rows, masks, in, w);
    return dgroup_sum_d<64>(a);
}

template <bool WT>
__global__ __launch_bounds__(256, 8) void run_sum_k(const SegWork s, const uint32_t* __restrict__ rows,
                                                             const uint16_t* __restrict__ masks,
                                                             const float* __restrict__ in,
                                                             const float* __restrict__ w, VoxOut out)
{
    __shared__ double red[4];
    int k = kVoxClasses - 1;   // uniform: the class whose blocks hold this one
    while (k > 0 && blockIdx.x >= s.blk[kVoxClasses - k]) --k;
    const uint32_t b0 = s.blk[kVoxClasses - 1 - k], nb = s.blk[kVoxClasses - k] - b0;
    const int64_t lb = xcd_block(blockIdx.x - b0, nb);
    const VoxDev* d = k == kVoxClasses - 1 ? s.pieces : s.desc + s.off[k];
    const int64_t n = s.cnt[k];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    switch (k) {
        case 0: run_parts<4, WT>(lb, d, n, rows, masks, in, w, out); break;
        case 1: run_parts<8, WT>(lb, d, n, rows, masks, in, w, out); break;
        case 2: run_group<16, WT>(lb, d, n, rows, masks, in, w, out); break;
        case 3: run_group<32, WT>(lb, d, n, rows, masks, in, w, out); break;
        case 4: run_group<64, WT>(lb, d, n, rows, masks, in, w, out); break;
        case 5: {
            const int64_t v = lb * 4 + wv;
            if (v >= n) return;   // whole wave
            const double t = run_wave256<WT>(d[v], 0, rows, masks, in, w);
            if ((threadIdx.x & 63) == 0) vox_store(d[v].v, t, out);
            break;
        }
        default: {
            if (lb >= n) return;   // whole block
            const double t = run_wave256<WT>(d[lb], wv * 256, rows, masks, in, w);
            if ((threadIdx.x & 63) == 0) red[wv] = t;
            __syncthreads();
            if (threadIdx.x == 0) {
                const double sum = ((red[0] + red[1]) + red[2]) + red[3];
                const VoxOut po{nullptr, nullptr, nullptr, nullptr, s.psum};
                vox_store(d[lb].v, sum, k == kVoxClasses - 1 ? po : out);
            }
        }
    }
}

// segments per block of class k
static int64_t seg_per_block(int k)
{
    if (k >= kVoxClasses - 2) return 1;
    return kVoxCap[k] <= 32 ? (int64_t)(256 / kVoxCap[k]) * kVoxVPW[k] : 4 * kVoxVPW[k];
}

static int64_t run_per_block(int k)
{
    constexpr int64_t per[kRunClasses] = {64, 32, 32, 16, 8, 4, 1};
    return k < kRunClasses ? per[k] : 1;
}

static int64_t run_per_block_weighted(int k)   // one in turn
{
    return k >= 2 && k <= 4 ? run_per_block(k) / 2 : run_per_block(k);
}

// the work of one launch; returns its blocks
static int64_t seg_work(const mrf_ctx* c, const SegList& l, int64_t (*per_block)(int), SegWork& k)
{
    k = SegWork{};
    k.desc = (const VoxDev*)l.desc.p;
    k.pieces = (const VoxDev*)l.hub.p;
    k.psum = (double*)c->b_hubsum.p;
    int64_t blocks = 0;
    for (int q = kVoxClasses - 1; q >= 0; --q) {
        k.off[q] = l.off[q];
        k.cnt[q] = q == kVoxClasses - 1 ? l.n_pieces : l.cnt[q];
        blocks += (nblk(k.cnt[q], (int)per_block(q)) + 7) / 8 * 8;
        k.blk[kVoxClasses - q] = (uint32_t)blocks;
    }
    return blocks;
}

// the hubs of a launched segment list
static hipError_t hub_sum(mrf_ctx* c, const SegList& l, const VoxOut& out, hipStream_t s)
{
    const int64_t nh = l.cnt[kVoxClasses - 1];
    if (nh > 0)
        hipLaunchKernelGGL(hub_sum_k, dim3(nblk(nh, 4)), dim3(256), 0, s, (const VoxDev*)l.hub.p + l.n_pieces, nh,
                           (const double*)c->b_hubsum.p, out);
    return hipGetLastError();
}

static hipError_t seg_sum(mrf_ctx* c, const SegList& l, const float* in, const VoxOut& out, const float* w,
                          hipStream_t s)
{
    SegWork k;
    const int64_t blocks = seg_work(c, l, seg_per_block, k);
    if (blocks == 0) return hipSuccess;
    const dim3 g((unsigned)blocks), b(256);
    const uint32_t* ve = (const uint32_t*)c->b_vedge.p;
    if (w)   // weights: keyframe pairs, whose builds have one slot group
        hipLaunchKernelGGL((seg_sum_k<true, false>), g, b, 0, s, k, ve, in, out, w, c->sg);
    else if (c->sg.n > 1)
        hipLaunchKernelGGL((seg_sum_k<false, true>), g, b, 0, s, k, ve, in, out, w, c->sg);
    else
        hipLaunchKernelGGL((seg_sum_k<false, false>), g, b, 0, s, k, ve, in, out, w, c->sg);
    return hub_sum(c, l, out, s);
}

// w (slot order, may be null): every message times its weight
static hipError_t run_sum(mrf_ctx* c, const SegList& l, const float* in, const VoxOut& out, const float* w,
                          hipStream_t s)
{
    SegWork k;
    const int64_t blocks = seg_work(c, l, w ? run_per_block_weighted : run_per_block, k);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(w ? run_sum_k<true> : run_sum_k<false>, dim3((unsigned)blocks), dim3(256), 0, s, k,
                       (const uint32_t*)c->b_runrow.p, (const uint16_t*)c->b_runmask.p, in, w, out);
    return hub_sum(c, l, out, s);
}

hipError_t launch_voxel_phase(mrf_ctx* c, const float* in, VoxOut out, hipStream_t s)
{
    ProfScope ps(c, KID_VOX, s);
    return c->by_runs ? run_sum(c, c->vox, in, out, nullptr, s) : seg_sum(c, c->vox, in, out, nullptr, s);
}

// ------------------------------------------------------------ keyframe pairs
//
// Per-keyframe averaged messages (Sec. IV-A): keyframe f sends voxel v the
// average M_fv = sum_j w_j ell_j of its rays' messages, w_j the edge's chord
// length over the pair's summed chord length, and a ray of keyframe f
// receives theta_v plus the other keyframes' averages.  The pair phase forms
// every M (FP64, fixed order); the voxel step sums them per voxel and writes,
// per pair, x = fl(T - M_fv) into keyframe f's message buffer.

hipError_t launch_pair_phase(mrf_ctx* c, const float* in, const float* w, double* M, hipStream_t s)
{
    ProfScope ps(c, KID_PAIR, s);
    const VoxOut out{nullptr, nullptr, nullptr, nullptr, M};
    return c->by_runs ? run_sum(c, c->pair, in, out, w, s) : seg_sum(c, c->pair, in, out, w, s);
}

// One 16-lane group per touched voxel: T = theta_v + the sum of the voxel's
// pair averages (FP64; lane-strided partial sums added in a fixed order), then
// every pair's message x = fl(T - M) into its keyframe's buffer, and L_v = fl(T).
// M null: every average is 0 (x = theta).
__global__ __launch_bounds__(256) void kf_voxel_k(const VoxDev* __restrict__ vd, int64_t n,
                                                  const double* __restrict__ M, const uint32_t* __restrict__ px,
                                                  const float* __restrict__ theta, float* __restrict__ x,
                                                  float* __restrict__ L)
{
    const int64_t vi = (int64_t)xcd_block(blockIdx.x, gridDim.x) * 16 + (int)(threadIdx.x >> 4);
    if (vi >= n) return;   // whole group
    const int l = (int)(threadIdx.x & 15);
    const VoxDev d = vd[vi];
    double a = 0.0;
    if (M)
        for (int q = l; q < d.m; q += 16) a += M[d.start + q];
    a = dgroup_sum_d<16>(a);
    const double T = (double)theta[d.v] + __shfl(a, (int)(threadIdx.x & 48), 64);
    if (x)
        for (int q = l; q < d.m; q += 16) x[px[d.start + q]] = (float)(T - (M ? M[d.start + q] : 0.0));
    if (L && l == 0) L[d.v] = (float)T;
}

hipError_t launch_kf_voxel(mrf_ctx* c, const double* M, const float* theta, float* x, float* L, hipStream_t s)
{
    if (c->n_kf_vox <= 0) return hipSuccess;
    ProfScope ps(c, KID_KFVOX, s);
    hipLaunchKernelGGL(kf_voxel_k, dim3(nblk(c->n_kf_vox, 16)), dim3(256), 0, s, (const VoxDev*)c->b_kf_vox.p,
                       c->n_kf_vox, M, (const uint32_t*)c->b_pair_x.p, theta, x, L);
    return hipGetLastError();
}

// Reverse of kf_voxel_k: with s_p the pair sums of d/d lambda (FP64), S_v =
// their sum over the voxel's pairs (the same fixed order); acc_v += fl(S_v)
// (d/d theta) and, when y is given, y = fl(S_v - s_p) into the pair's keyframe
// buffer: the derivative reaching the pair's average through every other
// keyframe's incoming message.
__global__ __launch_bounds__(256) void kf_voxel_rev_k(const VoxDev* __restrict__ vd, int64_t n,
                                                      const double* __restrict__ sp, const uint32_t* __restrict__ px,
                                                      float* __restrict__ acc, float* __restrict__ y)
{
    const int64_t vi = (int64_t)xcd_block(blockIdx.x, gridDim.x) * 16 + (int)(threadIdx.x >> 4);
    if (vi >= n) return;   // whole group
    const int l = (int)(threadIdx.x & 15);
    const VoxDev d = vd[vi];
    double a = 0.0;
    for (int q = l; q < d.m; q += 16) a += sp[d.start + q];
    a = dgroup_sum_d<16>(a);
    const double S = __shfl(a, (int)(threadIdx.x & 48), 64);
    if (y)
        for (int q = l; q < d.m; q += 16) y[px[d.start + q]] = (float)(S - sp[d.start + q]);
    if (l == 0) acc[d.v] += (float)S;
}

hipError_t launch_kf_voxel_rev(mrf_ctx* c, const double* sp, float* acc, float* y, hipStream_t s)
{
    if (c->n_kf_vox <= 0) return hipSuccess;
    ProfScope ps(c, KID_KFVOX, s);
    hipLaunchKernelGGL(kf_voxel_rev_k, dim3(nblk(c->n_kf_vox, 16)), dim3(256), 0, s, (const VoxDev*)c->b_kf_vox.p,
                       c->n_kf_vox, sp, (const uint32_t*)c->b_pair_x.p, acc, y);
    return hipGetLastError();
}

// ------------------------------------------------------------ ray phase

// Messages of one ray held by a group of G lanes, blocked: lane l holds steps
// [i0, i0 + IPL), i0 = l IPL, as base-2 log mu(0) (al), log mu(1) (be) and g,
// with neutral padding past the ray's m steps.  With c_i = log mu_i(1) + g_i
// the kernel carries P-free quantities (P_i, the log visibility up to voxel i,
// can reach 1e6 and would leak its rounding into every message):
//   R_i = S_i - P_i:  R_0 = log 0,  R_{i+1} = LSE(R_i, c_i) - log mu_i(0)
//   Q_i:              Q_{m-1} = log 0,  Q_{i-1} = LSE(c_i, log mu_i(0) + Q_i)
//   ell_i = LSE(R_i, g_i) - LSE(R_i, Q_i)
// Both recurrences are maps x -> LSE(c, a + x), scanned once across the group
// on the lane aggregates and walked sequentially inside the lane.
// put(j, ok, ell) receives the natural-log message of step i0 + j (meaningful
// when ok, i.e. i0 + j < m).
template <int G, int IPL, class Put>
__device__ __forceinline__ void ray_body(const float (&al)[IPL], const float (&be)[IPL], const float (&gg)[IPL],
                                         int m, int i0, Put&& put)
{
    // lane aggregate Cl = LSE_j (c_j + lp_j), lp_j the lane-local prefix of
    // log mu(0), a the lane sum: the lane's R map is (-a, Cl - a) and its Q
    // map (a, Cl)
    float c[IPL], cw[IPL];
    float a = 0.0f;
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        c[j] = be[j] + gg[j];
        cw[j] = c[j] + a;
        a += al[j];
    }
    const float Cl = lse_items<IPL>(cw);
    float R[IPL];
    {
        const LMap left = dscan_lmap<G>(LMap{-a, Cl - a});
        float r = dexcl<G>(left.c, MRF_NINF);
#pragma unroll
        for (int j = 0; j < IPL; ++j) {
            R[j] = r;
            r = lse(r, c[j]) - al[j];
        }
    }
    const LMap right = drscan_lmap<G>(LMap{a, Cl});
    float Q = drexcl<G>(right.c, MRF_NINF);
#pragma unroll
    for (int j = IPL - 1; j >= 0; --j) {
        put(j, i0 + j < m, lse_diff(R[j], gg[j], Q) * kLn2);
        Q = lse(c[j], al[j] + Q);
    }
}

// Direct variant: each group reads its ray's steps from global memory (one
// 64-byte row per step holds the 16 rays of the tile); lambda_e = tot[col_e] -
// own_e.  Step indices are clamped to the ray (m >= 1) so that every load is
// issued before the first wait.
// With KF (per-keyframe averaged messages, Sec. IV-A) lambda_e is the message
// of the ray's keyframe, kf.x[kf.xb[frame] + col_e], instead.
template <int G, int IPL, bool KF>
__global__ __launch_bounds__(256) void ray_k(const uint32_t* __restrict__ list, int64_t ntiles,
                                             const TileDev* __restrict__ tiles, const int32_t* __restrict__ counts,
                                             const int32_t* __restrict__ col, ExclDev lam, KfSrc kf,
                                             const float* __restrict__ g, float* __restrict__ ell)
{
    static_assert(G == 64 || IPL == 1, "16-lane groups hold a whole ray");
    int64_t s;
    int m, frame = 0;
    if (!tile_ray<G>(list, ntiles, tiles, counts, s, m, &frame)) return;
    const int i0 = (int)(threadIdx.x & (G - 1)) * IPL;
    int32_t cv[IPL];
    float ov[IPL], gv[IPL], lv[IPL];
    float2 tv[IPL];
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        const int64_t at = s + kTile * (int64_t)min(i0 + j, m - 1);
        cv[j] = col[at];
        if constexpr (!KF) ov[j] = lam.own[at];
        gv[j] = g[at];
    }
    if constexpr (KF) {
        const float* xf = kf.x + kf.xb[frame];
#pragma unroll
        for (int j = 0; j < IPL; ++j) lv[j] = cv[j] >= 0 ? xf[cv[j]] : 0.0f;
    } else {
#pragma unroll
        for (int j = 0; j < IPL; ++j) tv[j] = lam.tot[max(cv[j], 0)];
#pragma unroll
        for (int j = 0; j < IPL; ++j) lv[j] = excl_value(cv[j], tv[j], ov[j], lam.has_own);
    }
    float al[IPL], be[IPL], gg[IPL];
#pragma unroll
    for (int j = 0; j < IPL; ++j) load_step(lv[j], gv[j], i0 + j < m, al[j], be[j], gg[j]);
    ray_body<G, IPL>(al, be, gg, m, i0, [&](int j, bool ok, float v) {
        if (ok) ell[s + kTile * (i0 + j)] = v;
    });
}

// Tile-staged variant for tiles of at most G*IPL steps: one block of 16 groups
// per tile.  The block reads the tile's col, own and g (16 rays x len steps,
// contiguous) with coalesced loads, gathers the voxel totals, and puts lambda
// = tot[col] - own and g into LDS; every group runs the scans of its own ray
// on its LDS column and writes ell back into that column (0 past the ray),
// and the block stores the tile coalesced.
// Where a ray phase's messages come from: per-edge exclusion from the voxel totals, the
// per-keyframe message buffers, or (FIRST) the prior, with the potentials still to be
// computed.
enum RayMode { RAY_EXCL, RAY_KF, RAY_FIRST };

// The potentials of this thread's slots of the tile into vg and, for later sweeps, into
// p.g (padding slots: any value).  The tile's table row is staged in tab (3 kBins words
// of the LDS image, which is still unused).
// In the first sweep's ray kernels they cost 5 bytes an edge read and 4 written beside
// its col and ell; a pass of their own reads 5, writes 4 and has the sweep read 4 more:
// 8 VGA frames at 2 cm (5.2e8 slots), potentials and first sweep 2.66 ms in two
// passes and 2.03 in one.
template <int NT, int NR>
struct TilePotentials {
    static constexpr int W = tile_vec<NR>();
    float vd[NR];
    uint32_t vb[NR / W];

    __device__ __forceinline__ void fetch(const TileDev& td, int nf, const PotSrc& p)
    {
        tile_fetch<NT, NR>(p.delta, td.base, nf, vd);
        const uint8_t* bp = p.bin + td.base;
#pragma unroll
        for (int q = 0; q < NR / W; ++q) {
            const int iw = min((int)threadIdx.x + q * NT, nf / W - 1);
            if constexpr (W == 4) vb[q] = *(const uint32_t*)(bp + (uint32_t)iw * 4u);
            if constexpr (W == 2) vb[q] = *(const uint16_t*)(bp + (uint32_t)iw * 2u);
            if constexpr (W == 1) vb[q] = bp[(uint32_t)iw];
        }
    }

    __device__ __forceinline__ void compute(const TileDev& td, int nf, const PotSrc& p, float* tab, float (&vg)[NR])
    {
        if (threadIdx.x < kBins) {
            const int64_t row = p.cp > 0 ? tile_cell(td, p.frames, p.cp) * kBins : 0;
            const float s = p.sigma[row + threadIdx.x];
            tab[threadIdx.x] = 1.0f / s;
            tab[kBins + threadIdx.x] = logf(s) + 0.91893853320467274f;
            tab[2 * kBins + threadIdx.x] = p.bias[row + threadIdx.x];
        }
        __syncthreads();
        float* gp = p.g + td.base;
#pragma unroll
        for (int q = 0; q < NR / W; ++q) {
            VecT<W, float> o;
#pragma unroll
            for (int b = 0; b < W; ++b) {
                const uint32_t k = (vb[q] >> (8 * b)) & 255u;
                const int kk = k < kBins ? (int)k : 0;
                o.v[b] = vg[W * q + b] = potential(vd[W * q + b], tab[kk], tab[kBins + kk], tab[2 * kBins + kk]);
            }
            const int iw = (int)threadIdx.x + q * NT;
            if (W * iw < nf) vec_at<W>(gp, iw) = o;
        }
        __syncthreads();   // tab is free again
    }
};

template <int G, int IPL, RayMode MODE>
__device__ __forceinline__ void ray_tile(const TileDev& td, const int32_t* __restrict__ counts,
                                         const int32_t* __restrict__ col, const ExclDev& lam, const KfSrc& kf,
                                         const PotSrc& pot, const float* __restrict__ g, float* __restrict__ ell,
                                         float* sl, float* sg)
{
    constexpr bool KF = MODE == RAY_KF, FIRST = MODE == RAY_FIRST;
    constexpr int NT = kTile * G;
    const int nf = kTile * td.len;   // 1 <= td.len <= G * IPL by class
    const int i = (int)threadIdx.x / G;   // this group's ray: lane i of the tile
    const int gl = (int)threadIdx.x % G;
    const int i0 = gl * IPL;
    const int cb = lds_col(i0, gl, i);
    const int m = tile_ray_len(td, counts, i);
    {
        int32_t vc[IPL];
        float vo[IPL], vg[IPL], vt[IPL];
        float2 vp[IPL];
        tile_fetch_i<NT, IPL>(col, td.base, nf, vc);
        if constexpr (MODE == RAY_EXCL) tile_fetch<NT, IPL>(lam.own, td.base, nf, vo);
        TilePotentials<NT, IPL> tp;
        if constexpr (FIRST)
            tp.fetch(td, nf, pot);
        else
            tile_fetch<NT, IPL>(g, td.base, nf, vg);
        if constexpr (KF) {
            const float* xf = kf.x + kf.xb[td.frame];
#pragma unroll
            for (int r = 0; r < IPL; ++r) vt[r] = vc[r] >= 0 ? xf[vc[r]] : 0.0f;
        } else {
#pragma unroll
            for (int r = 0; r < IPL; ++r) vp[r] = lam.tot[max(vc[r], 0)];
#pragma unroll
            for (int r = 0; r < IPL; ++r)
                vt[r] = FIRST ? excl_value(vc[r], vp[r], 0.0f, 0) : excl_value(vc[r], vp[r], vo[r], lam.has_own);
        }
        if constexpr (FIRST) tp.compute(td, nf, pot, sl, vg);
        tile_to_lds<NT, IPL, IPL>(sl, vt);
        tile_to_lds<NT, IPL, IPL>(sg, vg);
    }
    __syncthreads();
    if (__ballot(m > 0)) {   // skip waves whose rays are all empty
        float al[IPL], be[IPL], gg[IPL];
#pragma unroll
        for (int j = 0; j < IPL; ++j)   // column rows are inside the LDS tile even past the ray
            load_step(sl[cb + kTile * j], sg[cb + kTile * j], i0 + j < m, al[j], be[j], gg[j]);
        ray_body<G, IPL>(al, be, gg, m, i0, [&](int j, bool ok, float v) { sl[cb + kTile * j] = ok ? v : 0.0f; });
    }
    __syncthreads();
    tile_store<NT, IPL, IPL>(ell, td.base, nf, [&](int, int at) { return sl[at]; });
}

template <int G, int IPL, RayMode MODE>
__global__ __launch_bounds__(kTile * G) void ray_lds_k(const uint32_t* __restrict__ list, int64_t ntiles,
                                                       const TileDev* __restrict__ tiles,
                                                       const int32_t* __restrict__ counts,
                                                       const int32_t* __restrict__ col, ExclDev lam, KfSrc kf, PotSrc pot,
                                                       const float* __restrict__ g, float* __restrict__ ell)
{
    __shared__ float sl[kTile * G * IPL];
    __shared__ float sg[kTile * G * IPL];
    const int64_t ti = xcd_block(blockIdx.x, gridDim.x);
    if (ti >= ntiles) return;   // whole block
    const TileDev td = tiles[list[ti]];
    ray_tile<G, IPL, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg);
}

// The short classes of a small graph in one launch, a block per tile.  Such a phase is
// a few microseconds of launch, dependent loads and scans whatever its tiles: one launch
// of them instead of one per class.
template <RayMode MODE>
__global__ __launch_bounds__(256) void ray_small_k(const SmallTiles st, const TileDev* __restrict__ tiles,
                                                   const int32_t* __restrict__ counts,
                                                   const int32_t* __restrict__ col, ExclDev lam, KfSrc kf, PotSrc pot,
                                                   const float* __restrict__ g, float* __restrict__ ell)
{
    constexpr int CAP = kRayCap[kSmallClasses - 1];
    __shared__ float sl[kTile * CAP];
    __shared__ float sg[kTile * CAP];
    int k = 0;   // uniform: the class whose blocks hold this one
    while (k + 1 < kSmallClasses && blockIdx.x >= st.blk[k + 1]) ++k;
    const int q = kSmallClasses - 1 - k;
    const int64_t lt = xcd_block(blockIdx.x - st.blk[k], st.blk[k + 1] - st.blk[k]);
    if (lt >= st.cnt[q]) return;   // whole block
    const TileDev td = tiles[st.list[st.off[q] + lt]];
    switch (q) {
        case 0: ray_tile<16, kRayCap[0] / 16, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg); break;
        case 1: ray_tile<16, kRayCap[1] / 16, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg); break;
        case 2: ray_tile<16, kRayCap[2] / 16, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg); break;
        case 3: ray_tile<16, kRayCap[3] / 16, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg); break;
        default: ray_tile<16, kRayCap[4] / 16, MODE>(td, counts, col, lam, kf, pot, g, ell, sl, sg);
    }
}

// The sources of one ray-phase launch.
struct RaySrc {
    ExclDev lam;
    KfSrc kf;
    PotSrc pot;
    RayMode mode;
};

template <int Q, int I, RayMode MODE>
static void launch_ray_shape_t(const mrf_ctx* c, int64_t off, int64_t n, const RaySrc& src, float* ell, hipStream_t s)
{
    constexpr int G = kFwdShapes[Q][I].g;
    if constexpr (G != 0) {
        constexpr int CAP = kRayCap[Q];
        const uint32_t* list = (const uint32_t*)c->b_ray_list.p + c->ray_off[Q] + off;
        if constexpr (ray_class_lds(Q)) {
            hipLaunchKernelGGL((ray_lds_k<G, CAP / G, MODE>), dim3((unsigned)n), dim3(kTile * G), 0, s, list, n,
                               (const TileDev*)c->b_tiles.p, (const int32_t*)c->b_counts.p,
                               (const int32_t*)c->b_col.p, src.lam, src.kf, src.pot, (const float*)c->b_g.p, ell);
        } else {   // the potentials have their own pass where direct classes run
            hipLaunchKernelGGL((ray_k<G, CAP / G, MODE == RAY_KF>), dim3((unsigned)(n * tile_blocks<G>())), dim3(256),
                               0, s, list, n, (const TileDev*)c->b_tiles.p, (const int32_t*)c->b_counts.p,
                               (const int32_t*)c->b_col.p, src.lam, src.kf, (const float*)c->b_g.p, ell);
        }
    }
}

template <int Q, int I>
static void launch_ray_shape(const mrf_ctx* c, int64_t off, int64_t n, const RaySrc& src, float* ell, hipStream_t s)
{
    switch (src.mode) {
        case RAY_KF: launch_ray_shape_t<Q, I, RAY_KF>(c, off, n, src, ell, s); break;
        case RAY_FIRST: launch_ray_shape_t<Q, I, RAY_FIRST>(c, off, n, src, ell, s); break;
        default: launch_ray_shape_t<Q, I, RAY_EXCL>(c, off, n, src, ell, s);
    }
}

template <int Q, int... I>
static void launch_ray_sel(int sel, const mrf_ctx* c, int64_t off, int64_t n, const RaySrc& src, float* ell,
                           hipStream_t s, std::integer_sequence<int, I...>)
{
    ((sel == I ? launch_ray_shape<Q, I>(c, off, n, src, ell, s) : void()), ...);
}

// class Q of the ray phase with launch shape sel, over n tiles of its list from off
template <int Q>
static void launch_ray_class(const mrf_ctx* c, int sel, int64_t off, int64_t n, const RaySrc& src, float* ell,
                             hipStream_t s)
{
    if (n <= 0) return;
    ProfScope ps(c, KID_RAY0 + Q, s);
    launch_ray_sel<Q>(sel, c, off, n, src, ell, s, std::make_integer_sequence<int, kNShapes>{});
}

// The untuned shape of the plain schedule: one 64-lane wave per ray where the
// class has such a shape (the 16-step class holds a ray in 16 lanes).
constexpr int plain_shape(int q)
{
    for (int i = 0; i < ray_shape_count(q, false); ++i)
        if (kFwdShapes[q][i].g == 64) return i;
    return 0;
}

template <int... Q>
static void ray_classes(std::integer_sequence<int, Q...>, const mrf_ctx* c, const int64_t* off, const int64_t* cnt,
                        const RaySrc& src, float* ell, bool plain, hipStream_t s)
{
    (launch_ray_class<Q>(c, plain ? plain_shape(Q) : c->fwd_sel[Q], off[Q], cnt[Q], src, ell, s), ...);
}

static void ray_classes(const mrf_ctx* c, const int64_t* off, const int64_t* cnt, const RaySrc& src, float* ell,
                        bool plain, hipStream_t s)
{
    ray_classes(std::make_integer_sequence<int, kRayClasses>{}, c, off, cnt, src, ell, plain, s);
}

using RayClassFn = void (*)(const mrf_ctx*, int, int64_t, int64_t, const RaySrc&, float*, hipStream_t);
template <int... Q>
static constexpr std::array<RayClassFn, kRayClasses> ray_class_fns(std::integer_sequence<int, Q...>)
{
    return {&launch_ray_class<Q>...};
}

static hipError_t ray_class_shape(const mrf_ctx* c, int q, int sel, const RaySrc& src, float* ell, hipStream_t s)
{
    static constexpr std::array<RayClassFn, kRayClasses> fns =
        ray_class_fns(std::make_integer_sequence<int, kRayClasses>{});
    if (q < 0 || q >= kRayClasses || sel < 0 || sel >= ray_shape_count(q, false)) return hipErrorInvalidValue;
    fns[q](c, sel, 0, c->ray_cnt[q], src, ell, s);
    return hipGetLastError();
}

hipError_t launch_ray_class_shape(const mrf_ctx* c, int q, int sel, ExclSrc lam, float* ell, hipStream_t s)
{
    return ray_class_shape(c, q, sel, RaySrc{excl_dev(c, lam), KfSrc{}, PotSrc{}, RAY_EXCL}, ell, s);
}

hipError_t launch_ray_class_shape_kf(const mrf_ctx* c, int q, int sel, KfSrc lam, float* ell, hipStream_t s)
{
    return ray_class_shape(c, q, sel, RaySrc{excl_dev(c, ExclSrc{nullptr, nullptr}), lam, PotSrc{}, RAY_KF}, ell, s);
}

static hipError_t ray_phase(mrf_ctx* c, const RaySrc& src, float* ell, bool plain, hipStream_t s)
{
    int64_t off[kRayClasses] = {0}, cnt[kRayClasses];
    if (!plain) {
        SmallTiles st;
        const int64_t blocks = small_tiles(c, c->fwd_sel, kSmallTilesFwd, st);
        for (int k = 0; k < kRayClasses; ++k)
            cnt[k] = k < kSmallClasses && st.cnt[k] > 0 ? 0 : c->ray_cnt[k];
        if (blocks > 0) {
            ProfScope ps(c, KID_RAYS, s);
            const auto kernel = src.mode == RAY_KF      ? ray_small_k<RAY_KF>
                                : src.mode == RAY_FIRST ? ray_small_k<RAY_FIRST>
                                                        : ray_small_k<RAY_EXCL>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, st, (const TileDev*)c->b_tiles.p,
                               (const int32_t*)c->b_counts.p, (const int32_t*)c->b_col.p, src.lam, src.kf, src.pot,
                               (const float*)c->b_g.p, ell);
        }
        ray_classes(c, off, cnt, src, ell, false, s);
    } else {
        // the plain per-frame schedule: one launch per frame (per class), untuned shapes
        const int nf = c->n_frames;
        for (int f = 0; f < nf; ++f) {
            for (int k = 0; k < kRayClasses; ++k) {
                const int64_t* fo = c->frame_ray_off.data() + (size_t)k * (nf + 1);
                off[k] = fo[f];
                cnt[k] = fo[f + 1] - fo[f];
            }
            ray_classes(c, off, cnt, src, ell, true, s);
        }
    }
    return hipGetLastError();
}

hipError_t launch_ray_phase(mrf_ctx* c, ExclSrc lam_src, float* ell, bool plain, hipStream_t s)
{
    return ray_phase(c, RaySrc{excl_dev(c, lam_src), KfSrc{}, PotSrc{}, RAY_EXCL}, ell, plain, s);
}

hipError_t launch_first_sweep(mrf_ctx* c, float* ell, bool plain, hipStream_t s)
{
    const ExclSrc theta{(const float2*)c->b_theta2.p, nullptr};
    bool fused = !plain;   // and no tiles longer than the LDS classes hold
    for (int q = 0; q < kRayClasses; ++q) fused = fused && (ray_class_lds(q) || c->ray_cnt[q] == 0);
    if (!fused) {
        const hipError_t e = launch_potentials(c, s);
        return e == hipSuccess ? launch_ray_phase(c, theta, ell, plain, s) : e;
    }
    const PotSrc p{(const float*)c->b_delta.p, (const uint8_t*)c->b_bin.p, (const float*)c->b_sigma.p,
                   (const float*)c->b_bias.p, (float*)c->b_g.p, (const FrameDev*)c->b_frames.p, c->cell_px};
    return ray_phase(c, RaySrc{excl_dev(c, theta), KfSrc{}, p, RAY_FIRST}, ell, false, s);
}

hipError_t launch_ray_phase_kf(mrf_ctx* c, KfSrc lam, float* ell, bool plain, hipStream_t s)
{
    return ray_phase(c, RaySrc{excl_dev(c, ExclSrc{nullptr, nullptr}), lam, PotSrc{}, RAY_KF}, ell, plain, s);
}

// lambda_e of the per-keyframe messages on every slot (exports)
__global__ void excl_kf_k(const int32_t* __restrict__ col, const int64_t* __restrict__ fs, int nf, KfSrc x,
                          float* __restrict__ out, int64_t S)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < S; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = col[i];
        int lo = 0, hi = nf;   // frame of slot i: the last f with fs[f] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (fs[mid] <= i)
                lo = mid;
            else
                hi = mid;
        }
        out[i] = v >= 0 ? x.x[x.xb[lo] + v] : 0.0f;
    }
}

hipError_t launch_excl_kf(const mrf_ctx* c, KfSrc x, float* out, hipStream_t s)
{
    if (c->S <= 0) return hipSuccess;
    const int64_t* fs = (const int64_t*)c->b_kfxb.p + c->n_frames + 1;
    hipLaunchKernelGGL(excl_kf_k, dim3(grid_for(c->S)), dim3(256), 0, s, (const int32_t*)c->b_col.p, fs, c->n_frames,
                       x, out, c->S);
    return hipGetLastError();
}

}  // namespace mrf

namespace mrf {

// ------------------------------------------------------------ depth messages
//
// The ray factor's message to its depth variable (Eq. depth_message, Sec.
// III-C): the measurement came from voxel i's depth with weight
// nu(d_i) mu_i(1) prod_{k<i} mu_k(0), mu the voxel -> ray messages of the last
// sweep, normalised over the ray (the all-empty configuration has potential
// zero).  With the log2 weights W_i = log2 mu_i(1) + log2 nu_i + P_i, the
// visibility P_i summed in FP64, the mode is the first largest W_i,
// q_i = 2^(W_i - max) / sum, and the mean depth sum_i q_i d_i, d_i = Z - delta_i.

// Depth messages of one ray held by a group of G lanes, blocked as in ray_body (lane l
// holds steps [i0, i0 + IPL), i0 = l IPL).  step(j, al, be, gg) gives the base-2 logs of step
// i0 + j (load_step); ready() is called once all of them have been taken, then delta(j) gives
// its Z - d_i.  Returns the probabilities of the lane's steps (0 past the ray), and in every
// lane the most probable step and, with want_mean, the expected depth.
template <int G, int IPL, class Step, class Ready, class Delta>
__device__ __forceinline__ void depth_body(int m, int i0, bool want_mean, double Z, Step&& step, Ready&& ready,
                                           Delta&& delta, float (&prob)[IPL], int& best, double& mean)
{
    double W[IPL];
    double P = 0.0;
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        float al, be, gg;
        step(j, al, be, gg);
        W[j] = ((double)be + (double)gg) + P;   // past the ray: log 0
        P += (double)al;
    }
    ready();
    const double before = dexcl_scan_d<G>(P);   // log2 visibility up to the lane's first step
    double M = -__builtin_huge_val();
    best = 0;
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        W[j] += before;
        if (i0 + j < m && W[j] > M) {
            M = W[j];
            best = i0 + j;
        }
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
        const double oM = __shfl_xor(M, d, G);
        const int ob = __shfl_xor(best, d, G);
        if (oM > M || (oM == M && ob < best)) {
            M = oM;
            best = ob;
        }
    }
    double S = 0.0;
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        prob[j] = i0 + j < m ? ex2((float)(W[j] - M)) : 0.0f;
        S += (double)prob[j];
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1) S += __shfl_xor(S, d, G);
    const double inv = 1.0 / S;
    mean = 0.0;
    if (want_mean) {
#pragma unroll
        for (int j = 0; j < IPL; ++j)
            if (i0 + j < m) mean += ((double)prob[j] * inv) * (Z - (double)delta(j));
#pragma unroll
        for (int d = 1; d < G; d <<= 1) mean += __shfl_xor(mean, d, G);
    }
#pragma unroll
    for (int j = 0; j < IPL; ++j) prob[j] = (float)((double)prob[j] * inv);
}

// One group of G lanes per ray, one block per tile, staged through LDS like
// ray_lds_k; lane l holds steps [l IPL, (l + 1) IPL).  The probabilities go back
// through the ray's LDS column and leave as contiguous runs in canonical edge
// order.  Bound by its five accesses of 4 bytes an edge: 1.1e8 edges (2 VGA
// frames at 2 cm) in 576 us, 3.9 TB/s; a thread per ray walking its steps twice, and a
// gather from slot to canonical order after it, took 4036.
template <int G, int IPL, bool KF>
__global__ __launch_bounds__(kTile * G) void depth_lds_k(const uint32_t* __restrict__ list, int64_t ntiles,
                                                         const TileDev* __restrict__ tiles,
                                                         const FrameDev* __restrict__ frames,
                                                         const int32_t* __restrict__ counts,
                                                         const int64_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col, ExclDev lam, KfSrc kf,
                                                         const float* __restrict__ g,
                                                         const float* __restrict__ delta, float* __restrict__ prob,
                                                         int32_t* __restrict__ mode, float* __restrict__ mean)
{
    constexpr int NT = kTile * G;
    __shared__ float sl[kTile * G * IPL];
    __shared__ float sg[kTile * G * IPL];
    const int64_t ti = xcd_block(blockIdx.x, gridDim.x);
    if (ti >= ntiles) return;   // whole block
    const TileDev td = tiles[list[ti]];
    const int nf = kTile * td.len;   // 1 <= td.len <= G * IPL by class
    const int i = (int)threadIdx.x / G;   // this group's ray: lane i of the tile
    const int gl = (int)threadIdx.x % G;
    const int i0 = gl * IPL;
    const int cb = lds_col(i0, gl, i);
    const int m = tile_ray_len(td, counts, i);
    float vd[IPL];
    {
        int32_t vc[IPL];
        float vo[IPL], vg[IPL], vt[IPL];
        float2 vp[IPL];
        tile_fetch_i<NT, IPL>(col, td.base, nf, vc);
        if constexpr (!KF) tile_fetch<NT, IPL>(lam.own, td.base, nf, vo);
        tile_fetch<NT, IPL>(g, td.base, nf, vg);
        tile_fetch<NT, IPL>(delta, td.base, nf, vd);
        if constexpr (KF) {
            const float* xf = kf.x + kf.xb[td.frame];
#pragma unroll
            for (int r = 0; r < IPL; ++r) vt[r] = vc[r] >= 0 ? xf[vc[r]] : 0.0f;
        } else {
#pragma unroll
            for (int r = 0; r < IPL; ++r) vp[r] = lam.tot[max(vc[r], 0)];
#pragma unroll
            for (int r = 0; r < IPL; ++r) vt[r] = excl_value(vc[r], vp[r], vo[r], lam.has_own);
        }
        tile_to_lds<NT, IPL, IPL>(sl, vt);
        tile_to_lds<NT, IPL, IPL>(sg, vg);
    }
    __syncthreads();
    const int64_t r = td.ray0 + (int64_t)(i / kTileW) * td.W + (i & (kTileW - 1));
    const int64_t at = m > 0 ? row_ptr[r] : 0;
    double Z = 0.0, mq;
    if (mean && m > 0) {
        const FrameDev fr = frames[td.frame];
        Z = (double)fr.depth[r - fr.ray_base];
    }
    float q[IPL];
    int best;
    depth_body<G, IPL>(
        m, i0, mean != nullptr, Z,
        [&](int j, float& al, float& be, float& gg) {   // column rows are inside the LDS tile even past the ray
            load_step(sl[cb + kTile * j], sg[cb + kTile * j], i0 + j < m, al, be, gg);
        },
        [&] {
            __syncthreads();   // every group has its g: reuse sg for delta
            tile_to_lds<NT, IPL, IPL>(sg, vd);
            __syncthreads();
        },
        [&](int j) { return sg[cb + kTile * j]; }, q, best, mq);
    if (m > 0 && gl == 0) {
        if (mode) mode[r] = best;
        if (mean) mean[r] = (float)mq;
    }
    if (!prob) return;
#pragma unroll
    for (int j = 0; j < IPL; ++j) sl[cb + kTile * j] = q[j];
    // the group reads back its own column: accesses of one wave complete in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        const int k = j * G + gl;
        if (k < m) prob[at + k] = sl[lds_at<IPL>(k, i)];
    }
}

// Tiles longer than a block's LDS holds: one wave per ray, read in place as ray_k does.  The
// probabilities go through the wave's LDS row (a word more every 32, for the blocked writes)
// and leave as contiguous runs.  3.2e7 edges in rays of up to 1109 steps: 554 us; a thread per
// ray took 9.84 ms when it stored its ray's run word by word, and 4.09 with a pass of its own
// from slot to canonical order.
template <int IPL, bool KF>
__global__ __launch_bounds__(256) void depth_wave_k(const uint32_t* __restrict__ list, int64_t ntiles,
                                                    const TileDev* __restrict__ tiles,
                                                    const FrameDev* __restrict__ frames,
                                                    const int32_t* __restrict__ counts,
                                                    const int64_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col, ExclDev lam, KfSrc kf,
                                                    const float* __restrict__ g, const float* __restrict__ delta,
                                                    float* __restrict__ prob, int32_t* __restrict__ mode,
                                                    float* __restrict__ mean)
{
    constexpr int G = 64, BPT = tile_blocks<G>();
    __shared__ float row[4][G * IPL + 2 * IPL];
    const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
    const int64_t ti = lb / BPT;
    if (ti >= ntiles) return;   // whole block
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int i = (int)(lb % BPT) * 4 + w;   // this wave's ray: lane i of the tile
    const TileDev td = tiles[list[ti]];
    const int m = tile_ray_len(td, counts, i);
    if (m == 0) return;   // whole wave
    const int i0 = l * IPL;
    const int64_t s = td.base + i;
    int32_t cv[IPL];
    float ov[IPL], gv[IPL], lv[IPL], dv[IPL];
    float2 tv[IPL];
#pragma unroll
    for (int j = 0; j < IPL; ++j) {   // indices clamped to the ray: every load before the first wait
        const int64_t at = s + kTile * (int64_t)min(i0 + j, m - 1);
        cv[j] = col[at];
        if constexpr (!KF) ov[j] = lam.own[at];
        gv[j] = g[at];
        dv[j] = delta[at];
    }
    if constexpr (KF) {
        const float* xf = kf.x + kf.xb[td.frame];
#pragma unroll
        for (int j = 0; j < IPL; ++j) lv[j] = cv[j] >= 0 ? xf[cv[j]] : 0.0f;
    } else {
#pragma unroll
        for (int j = 0; j < IPL; ++j) tv[j] = lam.tot[max(cv[j], 0)];
#pragma unroll
        for (int j = 0; j < IPL; ++j) lv[j] = excl_value(cv[j], tv[j], ov[j], lam.has_own);
    }
    const int64_t r = td.ray0 + (int64_t)(i / kTileW) * td.W + (i & (kTileW - 1));
    double Z = 0.0, mq;
    if (mean) {
        const FrameDev fr = frames[td.frame];
        Z = (double)fr.depth[r - fr.ray_base];
    }
    float q[IPL];
    int best;
    depth_body<G, IPL>(
        m, i0, mean != nullptr, Z,
        [&](int j, float& al, float& be, float& gg) { load_step(lv[j], gv[j], i0 + j < m, al, be, gg); }, [] {},
        [&](int j) { return dv[j]; }, q, best, mq);
    if (l == 0) {
        if (mode) mode[r] = best;
        if (mean) mean[r] = (float)mq;
    }
    if (!prob) return;
    float* o = row[w];
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        const int k = i0 + j;
        o[k + (k >> 5)] = q[j];
    }
    // LDS accesses of one wave complete in order: the fences keep the compiler from moving
    // the reads above the writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int64_t at = row_ptr[r];
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
        const int k = j * G + l;
        if (k < m) prob[at + k] = o[k + (k >> 5)];
    }
}

// rays without voxels
__global__ void depth_none_k(const int32_t* __restrict__ counts, int64_t R, int32_t* __restrict__ mode,
                             float* __restrict__ mean)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R || counts[r] > 0) return;
    if (mode) mode[r] = -1;
    if (mean) mean[r] = __builtin_nanf("");
}

// The depth messages of one class's tiles; classes of LDS tiles take the class's
// default forward shape, longer ones a wave per ray.
template <int Q, bool KF>
static void launch_depth_class(const mrf_ctx* c, const ExclDev& lam, const KfSrc& kf, float* prob, int32_t* mode,
                               float* mean, hipStream_t s)
{
    const int64_t n = c->ray_cnt[Q];
    if (n <= 0) return;
    const uint32_t* list = (const uint32_t*)c->b_ray_list.p + c->ray_off[Q];
    const TileDev* tiles = (const TileDev*)c->b_tiles.p;
    const FrameDev* frames = (const FrameDev*)c->b_frames.p;
    const int32_t* counts = (const int32_t*)c->b_counts.p;
    const int64_t* rp = (const int64_t*)c->b_rowptr.p;
    const int32_t* col = (const int32_t*)c->b_col.p;
    const float *g = (const float*)c->b_g.p, *delta = (const float*)c->b_delta.p;
    if constexpr (kRayCap[Q] <= kLdsMaxCap) {
        constexpr int G = kFwdShapes[Q][0].g;
        hipLaunchKernelGGL((depth_lds_k<G, kRayCap[Q] / G, KF>), dim3((unsigned)n), dim3(kTile * G), 0, s, list, n,
                           tiles, frames, counts, rp, col, lam, kf, g, delta, prob, mode, mean);
    } else {
        hipLaunchKernelGGL((depth_wave_k<kRayCap[Q] / 64, KF>), dim3((unsigned)(n * tile_blocks<64>())), dim3(256), 0, s,
                           list, n, tiles, frames, counts, rp, col, lam, kf, g, delta, prob, mode, mean);
    }
}

template <bool KF, int... Q>
static void depth_classes(std::integer_sequence<int, Q...>, const mrf_ctx* c, const ExclDev& lam, const KfSrc& kf,
                          float* prob, int32_t* mode, float* mean, hipStream_t s)
{
    (launch_depth_class<Q, KF>(c, lam, kf, prob, mode, mean, s), ...);
}

hipError_t launch_depth_distribution(const mrf_ctx* c, ExclSrc lam, const KfSrc* kf, float* prob, int32_t* mode,
                                     float* mean, hipStream_t s)
{
    if (c->R > 0 && (mode || mean))
        hipLaunchKernelGGL(depth_none_k, dim3(nblk(c->R, 256)), dim3(256), 0, s, (const int32_t*)c->b_counts.p, c->R,
                           mode, mean);
    constexpr auto classes = std::make_integer_sequence<int, kRayClasses>{};
    if (kf)
        depth_classes<true>(classes, c, excl_dev(c, lam), *kf, prob, mode, mean, s);
    else
        depth_classes<false>(classes, c, excl_dev(c, lam), KfSrc{nullptr, nullptr}, prob, mode, mean, s);
    return hipGetLastError();
}

}  // namespace mrf
