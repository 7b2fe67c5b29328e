// Omega-masked TV primal-dual regulariser over hashed 8^3 blocks (gfx950).
//
// Section III-B/C of the paper: masked forward-difference gradient (Eq. 3),
// its negative adjoint as divergence (Eq. 4), and the Chambolle-Pock
// iteration (Eqs. 7-9) on the weighted ROF energy.  Two implementations of
// one iteration:
//   - two-pass: a dual kernel and a primal kernel, in place (60 B/voxel);
//   - fused: one kernel per iteration; each workgroup stages its block's
//     ubar with a one-voxel halo in LDS, recomputes the new dual on the -1
//     halo faces (so no second pass is needed) and ping-pongs ubar and p
//     between two buffers (48 B/voxel of algorithmic traffic).
// The fused body is shared with a persistent kernel that runs many
// sub-maps and all iterations in one launch, separated by grid barriers.
// Energies are accumulated in float64 with a fixed reduction order.
#include <cstring>
#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <cstdlib>
#include <cmath>
#include <map>
#include <mutex>
#include <vector>

#include "cp_kernel.h"
#include "dn_internal.h"

namespace dn {

// W waves of 64 lanes per block, 8 / W planes each.
template <class S, bool kRefine, bool kStream, bool kStill, int W>
__global__ __launch_bounds__(64 * W) void k_cp_fused(CPArgs<S> A)
{
    __shared__ CPShared<W> sh;
    const int64_t slot = xcd_slot(blockIdx.x, A.nb);
    if (slot >= A.nb) return;
    const int32_t b = A.order ? as_scalar(A.order)[slot] : int32_t(slot);
    cp_block<S, kRefine, kStream, kStill, W>(A, b, sh, wave_index(), threadIdx.x & 63u);
}

// The first iteration from the zero state, four voxels per thread: ubar and p
// are zero, so the dual stays zero, and each voxel takes the data term's step
// from u = 0.  Reads f, w and the masks, writes u, ubar and p: 29 bytes per
// FP32 voxel, where clearing the state (20) and a general iteration (48) were
// before; the result has the same bits.  A whole solve before and now: 202195
// blocks, 30 iterations FP32 28.1 and 27.0 ms; 60001 blocks, 50 iterations
// BF16 (whose zeros were also converted) 9.50 and 8.84 ms.
template <class S>
__global__ __launch_bounds__(256) void k_cp_first(int64_t n4, int64_t ps, const uint32_t *__restrict__ em,
                                                  const float4 *__restrict__ f, const float4 *__restrict__ w,
                                                  typename S::T *__restrict__ u, typename S::T *__restrict__ ubar,
                                                  typename S::T *__restrict__ p, float tl, float theta, int l1,
                                                  uint32_t seed)
{
    typedef typename S::T T4 __attribute__((ext_vector_type(4)));
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const uint32_t m = em[i];
    const float4 fv = f[i], wv = w[i];
    const float fs[4] = {fv.x, fv.y, fv.z, fv.w}, ws[4] = {wv.x, wv.y, wv.z, wv.w};
    T4 a, b;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float un = data_prox(0.0f, fs[k], ws[k], tl, l1);
        un = (m >> (8 * k)) & 1u ? un : 0.0f;
        const float ubn = un + theta * un;
        const uint32_t r = S::kLow ? voxel_bits(4 * i + k, 2, seed) : 0u;
        a[k] = S::sr(un, r);
        b[k] = S::sr(ubn, r >> 16);
    }
    const T4 zero = T4(0);
    reinterpret_cast<T4 *>(u)[i] = a;
    reinterpret_cast<T4 *>(ubar)[i] = b;
    for (int c = 0; c < 3; ++c) reinterpret_cast<T4 *>(p + c * ps)[i] = zero;
}

// ----------------------------------------------------- two-pass variant
__global__ __launch_bounds__(512) void k_dual(int64_t nb, int64_t ps, const int32_t *__restrict__ nbr,
                                              const uint8_t *__restrict__ emask, const float *__restrict__ ubar,
                                              float *__restrict__ p, float sigma)
{
    const int64_t b = blockIdx.x;
    if (b >= nb) return;
    const int t = threadIdx.x, lx = t & 7, ly = (t >> 3) & 7, lz = t >> 6;
    const int64_t gi = b * kBlockVox + t;
    const int32_t *nb27 = nbr + b * kNbr;
    const uint8_t m = emask[gi];
    const float u0 = ubar[gi];
    float g[3] = {0.f, 0.f, 0.f};
    if (m & 2) g[0] = ubar[lx < 7 ? gi + 1 : halo_index(nb27, 8, ly, lz)] - u0;
    if (m & 4) g[1] = ubar[ly < 7 ? gi + 8 : halo_index(nb27, lx, 8, lz)] - u0;
    if (m & 8) g[2] = ubar[lz < 7 ? gi + 64 : halo_index(nb27, lx, ly, 8)] - u0;
    float a = p[gi] + sigma * g[0], c1 = p[gi + ps] + sigma * g[1], c2 = p[gi + 2 * ps] + sigma * g[2];
    const float n = sqrtf((a * a + c1 * c1) + c2 * c2);
    if (n > 1.0f) { a = a / n; c1 = c1 / n; c2 = c2 / n; }
    p[gi] = a; p[gi + ps] = c1; p[gi + 2 * ps] = c2;
}

__global__ __launch_bounds__(512) void k_primal(int64_t nb, int64_t ps, const int32_t *__restrict__ nbr,
                                                const uint8_t *__restrict__ emask, const float *__restrict__ p,
                                                const float *__restrict__ f, const float *__restrict__ w,
                                                float *__restrict__ u, float *__restrict__ ubar, float tau,
                                                float lambda, float theta, int l1)
{
    const int64_t b = blockIdx.x;
    if (b >= nb) return;
    const int t = threadIdx.x, lx = t & 7, ly = (t >> 3) & 7, lz = t >> 6;
    const int64_t gi = b * kBlockVox + t;
    const int32_t *nb27 = nbr + b * kNbr;
    const uint8_t m = emask[gi];
    const float uo = u[gi];
    float un = uo;
    if (m & 1) {
        float dv = 0.0f;
        for (int a = 0; a < 3; ++a) {
            int64_t jm;
            if (a == 0) jm = lx > 0 ? gi - 1 : halo_index(nb27, -1, ly, lz);
            else if (a == 1) jm = ly > 0 ? gi - 8 : halo_index(nb27, lx, -1, lz);
            else jm = lz > 0 ? gi - 64 : halo_index(nb27, lx, ly, -1);
            const uint8_t bit = uint8_t(2 << a);
            float fwd = (m & bit) ? p[gi + a * ps] : 0.0f;
            float bwd = (jm >= 0 && (emask[jm] & bit)) ? p[jm + a * ps] : 0.0f;
            dv += fwd - bwd;
        }
        float ut = uo + tau * dv;
        float tlw = tau * lambda * w[gi];
        if (l1) {
            float r = ut - f[gi];
            r = r > tlw ? r - tlw : (r < -tlw ? r + tlw : 0.0f);
            un = fminf(fmaxf(f[gi] + r, -1.0f), 1.0f);
        } else {
            un = (ut + tlw * f[gi]) / (1.0f + tlw);
        }
    }
    u[gi] = un;
    ubar[gi] = un + theta * (un - uo);
}

// ------------------------------------------------------------- masks
// emask bit0 = Omega(g) (block allocated and w > 0); bit 1+a = m_a(g) =
// Omega(g) and Omega(g + e_a)  (Eq. 3's cases where the difference is kept).
// em4 holds the same four bits for the fused kernel, a word per (x, y):
// bits 4z .. 4z + 3 of em4[block][x + 8 y].
__global__ __launch_bounds__(512) void k_masks(int64_t nb, const int32_t *__restrict__ nbr,
                                               const float *__restrict__ w, uint8_t *__restrict__ emask,
                                               uint32_t *__restrict__ em4)
{
    __shared__ uint8_t sm[kBlockVox];
    const int64_t b = blockIdx.x;
    if (b >= nb) return;
    const int t = threadIdx.x, lx = t & 7, ly = (t >> 3) & 7, lz = t >> 6;
    const int64_t gi = b * kBlockVox + t;
    const int32_t *nb27 = nbr + b * kNbr;
    uint8_t m = 0;
    if (w[gi] > 0.0f) {
        m = 1;
        int64_t jx = halo_index(nb27, lx + 1, ly, lz);
        int64_t jy = halo_index(nb27, lx, ly + 1, lz);
        int64_t jz = halo_index(nb27, lx, ly, lz + 1);
        if (jx >= 0 && w[jx] > 0.0f) m |= 2;
        if (jy >= 0 && w[jy] > 0.0f) m |= 4;
        if (jz >= 0 && w[jz] > 0.0f) m |= 8;
    }
    emask[gi] = m;
    sm[t] = m;
    __syncthreads();
    if (t < 64) {
        uint32_t word = 0;
        for (int z = 0; z < 8; ++z) word |= uint32_t(sm[t + 64 * z]) << (4 * z);
        em4[b * 64 + t] = word;
    }
}

__device__ __forceinline__ uint64_t spread3(uint64_t v)
{
    v &= 0x1FFFFF;
    v = (v | (v << 32)) & 0x1F00000000FFFFull;
    v = (v | (v << 16)) & 0x1F0000FF0000FFull;
    v = (v | (v << 8)) & 0x100F00F00F00F00Full;
    v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

__global__ void k_morton(const int32_t *__restrict__ coords, int64_t nb, uint64_t *__restrict__ code,
                         int32_t *__restrict__ ids)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= nb) return;
    uint64_t x = uint64_t(int64_t(coords[4 * i]) + (1 << 20));
    uint64_t y = uint64_t(int64_t(coords[4 * i + 1]) + (1 << 20));
    uint64_t z = uint64_t(int64_t(coords[4 * i + 2]) + (1 << 20));
    code[i] = spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
    ids[i] = int32_t(i);
}

// ---------------------------------------------------------- energies
template <int kCtrl> __device__ __forceinline__ double dpp_add(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xF, 0xF, true);
    return v + __hiloint2double(hi, lo);
}
// A wave's sums of two values: of e in lane 0, of d in lane 32.  The halves
// of the wave take one value each, then four steps inside rows of 16 lanes
// (quads, mirrors) without LDS, and one across.
__device__ __forceinline__ double wave_sum2(double e, double d)
{
    const bool low = (threadIdx.x & 32u) == 0;
    double v = (low ? e : d) + __shfl_xor(low ? d : e, 32, 64);
    v = dpp_add<0xB1>(v);      // lane ^ 1
    v = dpp_add<0x4E>(v);      // lane ^ 2
    v = dpp_add<0x141>(v);     // the other quad of 8
    v = dpp_add<0x140>(v);     // the other 8 of 16
    return v + __shfl_xor(v, 16, 64);
}

// Per-block partial sums of E(u) and D(p) (Eq. 2 with the weight of the
// proximal step, Eq. 6), float64.  256 threads, two voxels each; u with its
// +1 faces, p and the edge masks with their -1 faces are staged in LDS.  Bound
// by latency and the float64 units: every load is issued before the barrier,
// nothing branches on the masks, and the sums stay in registers down to 16
// lanes: 5777 blocks 23.9 -> 19.8 us, 60001 269 -> 192.
// Fixed reduction order: wave_sum2, then the 4 wave sums in wave order.
template <class S>
__global__ __launch_bounds__(256) void k_energy_partial(int64_t nb, int64_t ps, const int32_t *__restrict__ nbr,
                                                        const uint8_t *__restrict__ emask,
                                                        const typename S::T *__restrict__ u,
                                                        const typename S::T *__restrict__ p,
                                                        const float *__restrict__ f, const float *__restrict__ w,
                                                        double lambda, int l1, double *__restrict__ partials)
{
    __shared__ float su[729];        // u on [0, 8]^3, index ((z*9)+y)*9+x
    __shared__ float sp[3][729];     // p on [-1, 7]^3, index i9
    __shared__ uint8_t sm[729];      // edge masks on [-1, 7]^3, index i9
    __shared__ double se[4], sd[4];
    const int64_t b = blockIdx.x;
    if (b >= nb) return;
    const int t = threadIdx.x;
    const int32_t *nb27 = nbr + b * kNbr;
    auto iu = [](int x, int y, int z) { return (z * 9 + y) * 9 + x; };
    float u2[2], f2[2], w2[2], q0[2], q1[2], q2[2];
    uint8_t m2[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int64_t gi = b * kBlockVox + t + 256 * k;
        u2[k] = S::ld(u[gi]);
        m2[k] = emask[gi];
        q0[k] = S::ld(p[gi]); q1[k] = S::ld(p[gi + ps]); q2[k] = S::ld(p[gi + 2 * ps]);
        f2[k] = f[gi];
        w2[k] = w[gi];
    }
    // wave a < 3: the +1 face of u along axis a, and on the -1 face the
    // component of p along it and the edge mask (of the block itself, and then
    // 0, where the neighbour is not allocated)
    const int a = __builtin_amdgcn_readfirstlane(t >> 6), c0 = t & 7, c1 = (t >> 3) & 7;
    if (a < 3) {
        const int32_t up = nb27[a == 0 ? 14 : (a == 1 ? 16 : 22)], low = nb27[a == 0 ? 12 : (a == 1 ? 10 : 4)];
        const int at = a == 0 ? 8 * c0 + 64 * c1 : (a == 1 ? c0 + 64 * c1 : c0 + 8 * c1);
        const int64_t ju = (up >= 0 ? up : b) * kBlockVox + at;
        const int64_t jl = (low >= 0 ? low : b) * kBlockVox + at + (a == 0 ? 7 : (a == 1 ? 56 : 448));
        const float uf = S::ld(u[ju]), pf = S::ld(p[jl + a * ps]);
        const uint8_t mf = emask[jl];
        su[a == 0 ? iu(8, c0, c1) : (a == 1 ? iu(c0, 8, c1) : iu(c0, c1, 8))] = up >= 0 ? uf : 0.0f;
        const int q = a == 0 ? i9(-1, c0, c1) : (a == 1 ? i9(c0, -1, c1) : i9(c0, c1, -1));
        sm[q] = low >= 0 ? mf : uint8_t(0);
        sp[a][q] = low >= 0 ? pf : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int v = t + 256 * k, lx = v & 7, ly = (v >> 3) & 7, lz = v >> 6;
        const int q = i9(lx, ly, lz);
        su[iu(lx, ly, lz)] = u2[k];
        sm[q] = m2[k];
        sp[0][q] = q0[k]; sp[1][q] = q1[k]; sp[2][q] = q2[k];
    }
    __syncthreads();
    double e = 0.0, d = 0.0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int v = t + 256 * k, lx = v & 7, ly = (v >> 3) & 7, lz = v >> 6;
        const int q = i9(lx, ly, lz);
        // (no branch on the masks: each would hold up the LDS reads after it)
        const uint32_t m = m2[k];
        const int qx = i9(lx - 1, ly, lz), qy = i9(lx, ly - 1, lz), qz = i9(lx, ly, lz - 1);
        const float ux = su[iu(lx + 1, ly, lz)], uy = su[iu(lx, ly + 1, lz)], uz = su[iu(lx, ly, lz + 1)];
        const float px = sp[0][qx], py = sp[1][qy], pz = sp[2][qz];
        const uint32_t mx = sm[qx], my = sm[qy], mz = sm[qz];
        const double u0 = u2[k], fv = f2[k], wv = w2[k], r = u0 - fv;
        const double g0 = double(m & 2 ? ux : u2[k]) - u0, g1 = double(m & 4 ? uy : u2[k]) - u0,
                     g2 = double(m & 8 ? uz : u2[k]) - u0;
        const double ev = sqrt((g0 * g0 + g1 * g1) + g2 * g2) + (l1 ? lambda * wv * fabs(r) : 0.5 * lambda * wv * r * r);
        double dv = 0.0, db;
        dv += double(m & 2 ? q0[k] : 0.0f) - double(mx & 2 ? px : 0.0f);
        dv += double(m & 4 ? q1[k] : 0.0f) - double(my & 4 ? py : 0.0f);
        dv += double(m & 8 ? q2[k] : 0.0f) - double(mz & 8 ? pz : 0.0f);
        if (l1) {
            // minimum over u in [-1, 1] of -u d + lambda w |u - f|: at -1, f or 1
            const double lw = lambda * wv;
            const double c0 = -fv * dv, c1 = -dv + lw * fabs(1.0 - fv), c2 = dv + lw * fabs(1.0 + fv);
            db = fmin(fmin(c0, c1), c2);
        } else {
            db = -fv * dv - dv * dv / (2.0 * lambda * wv);
        }
        e += m & 1 ? ev : 0.0;
        d += m & 1 ? db : 0.0;
    }
    const double v = wave_sum2(e, d);
    if ((t & 31) == 0) (t & 32 ? sd : se)[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        partials[2 * b] = ((se[0] + se[1]) + se[2]) + se[3];
        partials[2 * b + 1] = ((sd[0] + sd[1]) + sd[2]) + sd[3];
    }
}

// Fixed-order reduction of n (E, D) pairs: workgroup g sums pairs
// [1024 g, 1024 g + 1024): each thread adds 4 consecutive pairs, then a
// tree over the 256 threads.
__global__ __launch_bounds__(256) void k_energy_reduce(int64_t n, const double *__restrict__ in,
                                                       double *__restrict__ out)
{
    __shared__ double se[256], sd[256];
    const int t = threadIdx.x;
    const int64_t base = int64_t(blockIdx.x) * 1024 + 4 * t;
    double e = 0.0, d = 0.0;
    for (int k = 0; k < 4; ++k)
        if (base + k < n) { e += in[2 * (base + k)]; d += in[2 * (base + k) + 1]; }
    se[t] = e; sd[t] = d;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) { se[t] += se[t + h]; sd[t] += sd[t + h]; }
        __syncthreads();
    }
    if (t == 0) { out[2 * blockIdx.x] = se[0]; out[2 * blockIdx.x + 1] = sd[0]; }
}

// The last step: n <= kFinalPairs pairs by one workgroup, in a fixed order
// (each thread every 1024th pair, then a tree), to the call's report.
constexpr int64_t kFinalPairs = 16384;
__global__ __launch_bounds__(1024) void k_energy_final(int n, const double *__restrict__ in, double *__restrict__ out)
{
    __shared__ double se[16], sd[16];
    const int t = threadIdx.x;
    double e = 0.0, d = 0.0;
    const double2 *pairs = reinterpret_cast<const double2 *>(in);
    int k = t;
    for (; k + 3 * 1024 < n; k += 4 * 1024) {
        const double2 a = pairs[k], b = pairs[k + 1024], c = pairs[k + 2048], f = pairs[k + 3072];
        e += (a.x + b.x) + (c.x + f.x);
        d += (a.y + b.y) + (c.y + f.y);
    }
    for (; k < n; k += 1024) { e += pairs[k].x; d += pairs[k].y; }
    const double v = wave_sum2(e, d);
    if ((t & 31) == 0) (t & 32 ? sd : se)[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        e = d = 0.0;
        for (int w = 0; w < 16; ++w) { e += se[w]; d += sd[w]; }
        out[0] = e;
        out[1] = d;
    }
}

// ------------------------------------------------------- helpers
template <class T> __global__ void k_fill(T *__restrict__ a, int64_t n, T v)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

// A given dual into the state; *off = 1 if it is not zero outside Omega.
__global__ __launch_bounds__(256) void k_copy_dual(int64_t n4, int64_t ps4, const uint32_t *__restrict__ em,
                                                   const float4 *__restrict__ p0, float4 *__restrict__ p,
                                                   int64_t *__restrict__ off)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const uint32_t m = em[i];
    bool bad = false;
    for (int c = 0; c < 3; ++c) {
        const float4 q = p0[c * n4 + i];
        p[c * ps4 + i] = q;
        bad = bad || (!(m & 1u) && q.x != 0.0f) || (!(m & 0x100u) && q.y != 0.0f) || (!(m & 0x10000u) && q.z != 0.0f) ||
              (!(m & 0x1000000u) && q.w != 0.0f);
    }
    if (bad) *off = 1;
}

__global__ __launch_bounds__(256) void k_zero_state(int64_t n4, int64_t ps, float *__restrict__ u,
                                                    float *__restrict__ ubar, float *__restrict__ p)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    reinterpret_cast<float4 *>(u)[i] = zero;
    reinterpret_cast<float4 *>(ubar)[i] = zero;
    for (int c = 0; c < 3; ++c) reinterpret_cast<float4 *>(p + c * ps)[i] = zero;
}

template <class S> __global__ void k_demote(const float *__restrict__ a, typename S::T *__restrict__ b, int64_t n, int rz)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) b[i] = rz ? S::rz(a[i]) : S::rn(a[i]);
}

template <class S> __global__ void k_promote(const typename S::T *__restrict__ b, float *__restrict__ a, int64_t n)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) a[i] = S::ld(b[i]);
}

static inline unsigned grid1(int64_t n, int bs = 256) { return unsigned((n + bs - 1) / bs); }

template <class T> static int fill(hipStream_t st, T *a, int64_t n, T v)
{
    if (n <= 0) return DN_OK;
    hipLaunchKernelGGL(k_fill<T>, dim3(grid1(n)), dim3(256), 0, st, a, n, v);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

struct MaskScratch {
    uint64_t *code, *code2;
    int32_t *ids;
    void *tmp;
    size_t tmp_bytes;
};
static MaskScratch carve_masks(Bump &b, int64_t nb)
{
    MaskScratch x;
    x.code = b.take<uint64_t>(size_t(nb));
    x.code2 = b.take<uint64_t>(size_t(nb));
    x.ids = b.take<int32_t>(size_t(nb));
    x.tmp_bytes = tmp_sort(size_t(nb), 12);
    x.tmp = b.take<char>(x.tmp_bytes);
    return x;
}

size_t masks_scratch(int64_t n_blocks)
{
    Bump b(nullptr, 0);
    carve_masks(b, n_blocks);
    return b.off;
}

int build_masks(dn_volume *v)
{
    if (v->emask_nb == v->nb) return DN_OK;
    hipStream_t st = v->stream;
    if (v->nb > 0) {
        hipLaunchKernelGGL(k_masks, dim3(unsigned(v->nb)), dim3(512), 0, st, v->nb, v->nbr, v->w, v->emask,
                           v->em4);
        DN_HIP(hipGetLastError());
        // Morton processing order of the blocks
        Bump bump(v->scratch, v->scratch_bytes);
        MaskScratch x = carve_masks(bump, v->nb);
        if (!bump.fits()) { set_error("scratch too small for the block order"); return DN_E_CAPACITY; }
        hipLaunchKernelGGL(k_morton, dim3(grid1(v->nb)), dim3(256), 0, st, v->coords, v->nb, x.code, x.ids);
        DN_HIP(hipGetLastError());
        size_t tbytes = x.tmp_bytes;
        DN_HIP(rocprim::radix_sort_pairs(x.tmp, tbytes, x.code, x.code2, x.ids, v->order, size_t(v->nb), 0, 63, st));
    }
    v->emask_nb = v->nb;
    return DN_OK;
}

template <class S>
static int energy_launch(dn_volume *v, double lambda, int l1, const typename S::T *u, const typename S::T *p)
{
    hipStream_t st = v->stream;
    const int64_t ps = v->cap_blocks * kBlockVox;
    if (v->nb == 0) {
        hipLaunchKernelGGL(k_fill<double>, dim3(1), dim3(256), 0, st, reinterpret_cast<double *>(report(v)), int64_t(2),
                           0.0);
        DN_HIP(hipGetLastError());
        return DN_OK;
    }
    hipLaunchKernelGGL((k_energy_partial<S>), dim3(unsigned(v->nb)), dim3(256), 0, st, v->nb, ps, v->nbr,
                       v->emask, u, p, v->f, v->w, lambda, l1, v->partials);
    DN_HIP(hipGetLastError());
    return reduce_pairs(v, v->nb);
}

// Fixed-order sum of the n per-block pairs in v->partials, into the call's
// report: sums of 1024 pairs until one workgroup takes the rest.
int reduce_pairs(dn_volume *v, int64_t n)
{
    hipStream_t st = v->stream;
    double *src = v->partials;
    double *bufs[2] = {v->partials + 2 * v->cap_blocks, v->partials + 2 * v->cap_blocks + 2 * ((v->cap_blocks + 1023) / 1024 + 1)};
    int which = 0;
    while (n > kFinalPairs) {
        const int64_t g = (n + 1023) / 1024;
        hipLaunchKernelGGL(k_energy_reduce, dim3(unsigned(g)), dim3(256), 0, st, n, src, bufs[which]);
        DN_HIP(hipGetLastError());
        src = bufs[which];
        which ^= 1;
        n = g;
    }
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(1024), 0, st, int(n), src, reinterpret_cast<double *>(report(v)));
    DN_HIP(hipGetLastError());
    return DN_OK;
}

// Energies of the current state into the call's report (read_energy).
int energy_current(dn_volume *v, double lambda, bool use_f32, int data_term)
{
    const int l1 = data_term == DN_DATA_L1;
    int rc = build_masks(v);
    if (rc) return rc;
    switch (use_f32 ? DN_F32 : v->state_storage) {
    case DN_F16:
        return energy_launch<SF16>(v, lambda, l1, (const uint16_t *)v->u16, (const uint16_t *)v->p16[v->cur]);
    case DN_BF16:
        return energy_launch<SBF16>(v, lambda, l1, (const uint16_t *)v->u16, (const uint16_t *)v->p16[v->cur]);
    default:
        return energy_launch<SF32>(v, lambda, l1, v->u, v->p[v->cur]);
    }
}

int read_energy(dn_volume *v, double out[2])
{
    int rc = fetch_report(v, 2);
    if (rc) return rc;
    memcpy(out, v->host_stage, 16);
    return DN_OK;
}

template <class S>
static CPArgs<S> make_args(dn_volume *v, const dn_reg_params *prm, typename S::T *u, typename S::T *ub_in,
                           typename S::T *ub_out, typename S::T *p_in, typename S::T *p_out)
{
    CPArgs<S> A;
    A.nb = v->nb;
    A.pstride = v->cap_blocks * kBlockVox;
    A.nbr = v->nbr;
    A.em4 = v->em4;
    A.order = v->layout & 1 ? nullptr : v->order;
    A.f = v->f; A.w = v->w;
    A.u = u; A.ubar_in = ub_in; A.ubar_out = ub_out; A.p_in = p_in; A.p_out = p_out;
    A.u32 = nullptr; A.ubar32 = nullptr; A.p32 = nullptr;
    A.sigma = float(prm->sigma); A.tau = float(prm->tau); A.lambda = float(prm->lambda);
    A.theta = float(prm->theta);
    A.l1 = prm->data_term == DN_DATA_L1;
    A.seed = 0u;
    return A;
}

// Off Omega an iteration leaves u and p as they are and sets ubar to u, as
// long as p is zero there (it is projected with the rest).  Two iterations
// that write everything put the same values into both sets of buffers; after
// those (true here), iterations may leave empty lines alone.  Counts the
// iteration about to run.
static bool still_state(dn_volume *v) { return v->p_off_zero && v->full_iters++ >= 2; }

static unsigned fused_grid(int64_t nb) { return unsigned(((nb + 7) / 8) * 8); }

template <class S, bool kRefine, bool kStream, bool kStill>
static void launch_fused_w(hipStream_t st, const CPArgs<S> &A, int kernel)
{
    const dim3 grid(fused_grid(A.nb));
    switch (kernel) {
    case DN_K_FUSED64: hipLaunchKernelGGL((k_cp_fused<S, kRefine, kStream, kStill, 1>), grid, dim3(64), 0, st, A); break;
    case DN_K_FUSED128: hipLaunchKernelGGL((k_cp_fused<S, kRefine, kStream, kStill, 2>), grid, dim3(128), 0, st, A); break;
    case DN_K_FUSED256: hipLaunchKernelGGL((k_cp_fused<S, kRefine, kStream, kStill, 4>), grid, dim3(256), 0, st, A); break;
    default: hipLaunchKernelGGL((k_cp_fused<S, kRefine, kStream, kStill, 8>), grid, dim3(512), 0, st, A);
    }
}

// `still`: see still_state.  Not with 8 waves per block (a wait for the masks
// for a single plane each: no faster) and not in 16 bits, where a line is a
// whole plane and the waits cost more than the few empty planes give (60001
// blocks BF16: 179 and 232 us).
template <class S, bool kRefine> static void launch_fused(hipStream_t st, const CPArgs<S> &A, int kernel, bool still)
{
    if constexpr (!kRefine) {
        if (!streams_state(A.nb, sizeof(typename S::T))) {
            launch_fused_w<S, false, false, false>(st, A, kernel);
            return;
        }
        if constexpr (!S::kLow)
            if (still && kernel != DN_K_FUSED) {
                launch_fused_w<S, false, true, true>(st, A, kernel);
                return;
            }
    }
    launch_fused_w<S, kRefine, true, false>(st, A, kernel);
}

// One FP32 iteration with the chosen kernel.
static int step_f32(dn_volume *v, const dn_reg_params *prm, int kernel)
{
    hipStream_t st = v->stream;
    const int64_t ps = v->cap_blocks * kBlockVox;
    if (kernel == DN_K_TWOPASS) {
        hipLaunchKernelGGL(k_dual, dim3(unsigned(v->nb)), dim3(512), 0, st, v->nb, ps, v->nbr, v->emask,
                           v->ubar[v->cur], v->p[v->cur], float(prm->sigma));
        DN_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_primal, dim3(unsigned(v->nb)), dim3(512), 0, st, v->nb, ps, v->nbr, v->emask,
                           v->p[v->cur], v->f, v->w, v->u, v->ubar[v->cur], float(prm->tau), float(prm->lambda),
                           float(prm->theta), int(prm->data_term == DN_DATA_L1));
        DN_HIP(hipGetLastError());
        return DN_OK;
    }
    const int c = v->cur, n = 1 - c;
    auto A = make_args<SF32>(v, prm, v->u, v->ubar[c], v->ubar[n], v->p[c], v->p[n]);
    launch_fused<SF32, false>(st, A, kernel, still_state(v));
    DN_HIP(hipGetLastError());
    v->cur = n;
    return DN_OK;
}

template <class S>
static int step_lowp(dn_volume *v, const dn_reg_params *prm, bool refine, int kernel)
{
    const int c = v->cur, n = 1 - c;
    using T = typename S::T;
    auto A = make_args<S>(v, prm, (T *)v->u16, (T *)v->ubar16[c], (T *)v->ubar16[n], (T *)v->p16[c],
                          (T *)v->p16[n]);
    A.seed = uint32_t(v->lowp_iter++);
    if (refine) {
        A.u32 = v->u; A.ubar32 = v->ubar[n]; A.p32 = v->p[n];
        launch_fused<S, true>(v->stream, A, kernel, false);
    } else {
        launch_fused<S, false>(v->stream, A, kernel, false);
    }
    DN_HIP(hipGetLastError());
    v->cur = n;
    return DN_OK;
}

// Copy the FP32 state into the 16-bit buffers (u, ubar round to nearest,
// p toward zero so |p| <= 1 survives the rounding).
template <class S> static int demote_state(dn_volume *v)
{
    hipStream_t st = v->stream;
    const int64_t n = v->nb * kBlockVox, ps = v->cap_blocks * kBlockVox;
    using T = typename S::T;
    if (n == 0) return DN_OK;
    hipLaunchKernelGGL((k_demote<S>), dim3(grid1(n)), dim3(256), 0, st, v->u, (T *)v->u16, n, 0);
    hipLaunchKernelGGL((k_demote<S>), dim3(grid1(n)), dim3(256), 0, st, v->ubar[v->cur], (T *)v->ubar16[v->cur], n, 0);
    for (int a = 0; a < 3; ++a)
        hipLaunchKernelGGL((k_demote<S>), dim3(grid1(n)), dim3(256), 0, st, v->p[v->cur] + a * ps,
                           (T *)v->p16[v->cur] + a * ps, n, 1);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

static int validate(const dn_reg_params *prm)
{
    DN_REQUIRE(prm, "null params");
    DN_REQUIRE(prm->lambda > 0 && prm->tau > 0 && prm->sigma > 0, "lambda, tau, sigma must be > 0");
    DN_REQUIRE(prm->tau * prm->sigma * 12.0 <= 1.0 + 1e-9,
               "step sizes violate tau*sigma*|grad|^2 <= 1 (|grad|^2 <= 12 in 3-D)");
    DN_REQUIRE(prm->theta >= 0 && prm->theta <= 1, "theta must be in [0, 1]");
    DN_REQUIRE(prm->iters >= 0 && prm->gap_every >= 0, "iters, gap_every must be >= 0");
    int s = prm->storage;
    DN_REQUIRE(s == DN_F32 || s == DN_F16 || s == DN_BF16, "bad storage");
    DN_REQUIRE(prm->init >= DN_INIT_ZERO && prm->init <= DN_INIT_CONTINUE, "bad init");
    DN_REQUIRE(prm->kernel >= DN_K_AUTO && prm->kernel <= DN_K_FUSED256, "bad kernel");
    DN_REQUIRE(prm->refine_every >= 0, "refine_every must be >= 0");
    DN_REQUIRE(prm->gamma >= 0 && std::isfinite(prm->gamma), "gamma must be >= 0");
    DN_REQUIRE(prm->data_term == DN_DATA_L2 || prm->data_term == DN_DATA_L1, "bad data_term");
    DN_REQUIRE(prm->data_term == DN_DATA_L2 || prm->gamma == 0.0,
               "the accelerated variant needs the uniformly convex (L2) data term");
    return DN_OK;
}

// Copy the 16-bit state (exactly) into the FP32 buffers, so that a 16-bit
// run that stopped between refinement sweeps leaves its current state
// where the extraction and an FP32 continuation read it.
template <class S> static int promote_state(dn_volume *v)
{
    hipStream_t st = v->stream;
    const int64_t n = v->nb * kBlockVox, ps = v->cap_blocks * kBlockVox;
    using T = typename S::T;
    if (n == 0) return DN_OK;
    hipLaunchKernelGGL((k_promote<S>), dim3(grid1(n)), dim3(256), 0, st, (const T *)v->u16, v->u, n);
    hipLaunchKernelGGL((k_promote<S>), dim3(grid1(n)), dim3(256), 0, st, (const T *)v->ubar16[v->cur],
                       v->ubar[v->cur], n);
    for (int a = 0; a < 3; ++a)
        hipLaunchKernelGGL((k_promote<S>), dim3(grid1(n)), dim3(256), 0, st, (const T *)v->p16[v->cur] + a * ps,
                           v->p[v->cur] + a * ps, n);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

int zero_state(dn_volume *v)
{
    const int64_t n4 = v->nb * kBlockVox / 4, ps = v->cap_blocks * kBlockVox;
    from_zero(v);
    if (n4 == 0) return DN_OK;
    hipLaunchKernelGGL(k_zero_state, dim3(grid1(n4)), dim3(256), 0, v->stream, n4, ps, v->u, v->ubar[v->cur],
                       v->p[v->cur]);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

void from_zero(dn_volume *v)
{
    v->p_off_zero = true;
    v->full_iters = 0;
    v->state_storage = DN_F32;
}

int first_iteration(dn_volume *v, float tau, float lambda, float theta, int l1)
{
    const int64_t n4 = v->nb * kBlockVox / 4, ps = v->cap_blocks * kBlockVox;
    const int n = 1 - v->cur;
    if (n4 == 0) return DN_OK;
    hipLaunchKernelGGL(k_cp_first<SF32>, dim3(grid1(n4)), dim3(256), 0, v->stream, n4, ps,
                       reinterpret_cast<const uint32_t *>(v->emask), reinterpret_cast<const float4 *>(v->f),
                       reinterpret_cast<const float4 *>(v->w), v->u, v->ubar[n], v->p[n], tau * lambda, theta, l1, 0u);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

template <class S> static int first_lowp(dn_volume *v, const dn_reg_params *prm)
{
    using T = typename S::T;
    const int64_t n4 = v->nb * kBlockVox / 4, ps = v->cap_blocks * kBlockVox;
    const int n = 1 - v->cur;
    hipLaunchKernelGGL(k_cp_first<S>, dim3(grid1(n4)), dim3(256), 0, v->stream, n4, ps,
                       reinterpret_cast<const uint32_t *>(v->emask), reinterpret_cast<const float4 *>(v->f),
                       reinterpret_cast<const float4 *>(v->w), (T *)v->u16, (T *)v->ubar16[n], (T *)v->p16[n],
                       float(prm->tau) * float(prm->lambda), float(prm->theta),
                       int(prm->data_term == DN_DATA_L1), uint32_t(v->lowp_iter++));
    DN_HIP(hipGetLastError());
    v->cur = n;
    return DN_OK;
}

// Kernel choice for DN_K_AUTO: measured once per size bucket.  A choice is
// (kernel variant, layout) with layout bit 0 = pool order instead of Morton
// order.
struct AutoChoice { int kernel; int layout; };
// The candidates: 8, 4, 2 and 1 waves per block in Morton and in pool order,
// in XCD chunks.  Many waves are best where blocks are few (503 blocks: 4.9
// us with 8, 6.6 with 1), one wave where the 16-bit state leaves the vector
// units busy (60001 blocks: 169 us with 1, 174 with 4, 236 with 8).  The
// two-pass kernels (1.95 against 0.96 ms at 202195 blocks, 8.2 against 4.9
// us at 503) and the plain workgroup map (never more than 1 % ahead, up to
// 12 % behind) are not tried.
constexpr int kTuned[] = {DN_K_FUSED, DN_K_FUSED256, DN_K_FUSED128, DN_K_FUSED64};
// Keyed by (device, size bucket); the tuners of all threads share them.
static std::map<int64_t, AutoChoice> g_auto_kernel, g_auto_lowp;     // FP32 state, 16-bit state
static std::mutex g_auto_mutex;

static int size_bucket(int64_t nb)
{
    int b = 0;
    while ((int64_t(1) << b) < nb) ++b;
    return b;
}

static int64_t tune_key(const dn_volume *v, int64_t sub) { return (int64_t(v->device) << 32) | sub; }

// Long enough for the events' own time not to decide between small maps.
static int trial_iterations(int64_t nb) { return int(std::min<int64_t>(48, std::max<int64_t>(6, 24576 / nb))); }

// A later candidate has to be ahead by more than that: where the host issues
// the launches of a small map more slowly than they run (a profiler does that)
// all candidates look alike, and many waves, the first, are the safe choice
// (503 blocks: 4.6 us with 8, 6.8 with 1).
static float needed_lead(int64_t nb) { return nb < 4096 ? 0.97f : 1.0f; }

static bool find_choice(std::map<int64_t, AutoChoice> &m, int64_t key, AutoChoice *out)
{
    std::lock_guard<std::mutex> lk(g_auto_mutex);
    auto it = m.find(key);
    if (it == m.end()) return false;
    *out = it->second;
    return true;
}

void remember_choice(const dn_volume *v, int storage, int kernel, int layout)
{
    const bool low = storage != DN_F32;
    std::lock_guard<std::mutex> lk(g_auto_mutex);
    (low ? g_auto_lowp : g_auto_kernel)[tune_key(v, (low ? storage * 64 : 0) + size_bucket(v->nb))] = AutoChoice{kernel, layout};
}

static int autotune_single(dn_volume *v, const dn_reg_params *prm, int *choice)
{
    const int64_t key = tune_key(v, size_bucket(v->nb));
    AutoChoice found;
    if (find_choice(g_auto_kernel, key, &found)) {
        *choice = found.kernel;
        v->layout = found.layout;
        return DN_OK;
    }
    // time a few iterations of each candidate from the zero state
    hipEvent_t e0, e1;
    DN_HIP(hipEventCreate(&e0));
    DN_HIP(hipEventCreate(&e1));
    float best_ms = 1e30f;
    AutoChoice best{DN_K_FUSED, 0};
    const int trial = trial_iterations(v->nb);
    const float lead = needed_lead(v->nb);
    for (int k : kTuned)
        for (int layout = 0; layout < 2; ++layout) {
            v->layout = layout;
            int rc = zero_state(v);
            if (rc) return rc;
            for (int i = 0; i < 2; ++i)
                if ((rc = step_f32(v, prm, k))) return rc;  // warm up
            DN_HIP(hipEventRecord(e0, v->stream));
            for (int i = 0; i < trial; ++i)
                if ((rc = step_f32(v, prm, k))) return rc;
            DN_HIP(hipEventRecord(e1, v->stream));
            DN_HIP(hipEventSynchronize(e1));
            float ms = 0;
            DN_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (getenv("DN_VERBOSE"))
                fprintf(stderr, "[denser] tune: kernel %d layout %d: %.4f ms per iteration\n", k, layout, ms / trial);
            if (ms < best_ms * lead) { best_ms = ms; best = AutoChoice{k, layout}; }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    remember_choice(v, DN_F32, best.kernel, best.layout);
    *choice = best.kernel;
    v->layout = best.layout;
    return zero_state(v);
}

// The same choice for 16-bit state storage, timed on the 16-bit kernels.
// It runs only on a state just demoted from FP32, or zero (the trials
// overwrite the 16-bit buffers, which are then demoted again).

template <class S> static int autotune_lowp(dn_volume *v, const dn_reg_params *prm, bool zero, int *choice)
{
    const int storage = prm->storage;
    const int64_t key = tune_key(v, storage * 64 + size_bucket(v->nb));
    AutoChoice found;
    if (find_choice(g_auto_lowp, key, &found)) {
        *choice = found.kernel;
        v->layout = found.layout;
        return DN_OK;
    }
    hipEvent_t e0, e1;
    DN_HIP(hipEventCreate(&e0));
    DN_HIP(hipEventCreate(&e1));
    const int cur = v->cur;
    const uint64_t seed_iter = v->lowp_iter;   // the trials are discarded, so are their seeds
    float best_ms = 1e30f;
    AutoChoice best{DN_K_FUSED, 0};
    const int trial = trial_iterations(v->nb);
    const float lead = needed_lead(v->nb);
    int rc = DN_OK;
    if (zero) {                 // (the solve's own first iteration does without)
        if ((rc = zero_state(v)) || (rc = demote_state<S>(v))) return rc;
        v->state_storage = storage;
    }
    for (int k : kTuned)
        for (int layout = 0; layout < 2 && !rc; ++layout) {
            v->layout = layout;
            if ((rc = step_lowp<S>(v, prm, false, k))) break;   // warm up
            DN_HIP(hipEventRecord(e0, v->stream));
            for (int i = 0; i < trial && !rc; ++i) rc = step_lowp<S>(v, prm, false, k);
            DN_HIP(hipEventRecord(e1, v->stream));
            DN_HIP(hipEventSynchronize(e1));
            float ms = 0;
            DN_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (getenv("DN_VERBOSE"))
                fprintf(stderr, "[denser] tune16: kernel %d layout %d: %.4f ms per iteration\n", k, layout, ms / trial);
            if (ms < best_ms * lead) { best_ms = ms; best = AutoChoice{k, layout}; }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    v->cur = cur;
    v->lowp_iter = seed_iter;
    if (rc) return rc;
    remember_choice(v, storage, best.kernel, best.layout);
    *choice = best.kernel;
    v->layout = best.layout;
    return demote_state<S>(v);
}

}  // namespace dn

using namespace dn;

extern "C" {

int dn_energy(dn_volume *v, double lambda, int32_t data_term, double out[2])
{
    DN_REQUIRE(v && out && lambda > 0, "bad argument");
    DN_REQUIRE(data_term == DN_DATA_L2 || data_term == DN_DATA_L1, "bad data_term");
    int rc = energy_current(v, lambda, false, data_term);
    if (rc) return rc;
    return read_energy(v, out);
}

int dn_regularize(dn_volume *v, const dn_reg_params *prm, const float *u0, const float *p0, dn_reg_stats *out)
{
    DN_REQUIRE(v, "null volume");
    int rc = validate(prm);
    if (rc) return rc;
    DN_REQUIRE(prm->init != DN_INIT_GIVEN || u0, "init GIVEN needs u0");
    DN_REQUIRE(prm->storage == DN_F32 || v->prm.state16, "16-bit storage needs a volume created with state16");
    hipStream_t st = v->stream;
    if ((rc = build_masks(v))) return rc;
    const int64_t n = v->nb * kBlockVox, ps = v->cap_blocks * kBlockVox;
    const int storage = prm->storage;
    // initial state
    constexpr int kOffWord = 7;     // of the report (energies take the first two)
    bool look = false;
    // from zero, the first iteration need not find the zeros in memory, unless
    // it is the two-pass kernels' or a refinement sweep
    const bool first = prm->init == DN_INIT_ZERO && prm->iters > 0 && v->nb > 0 &&
                       (storage == DN_F32 ? prm->kernel != DN_K_TWOPASS : prm->iters > 1 && prm->refine_every != 1);
    if (first) {
        from_zero(v);
    } else if (prm->init == DN_INIT_ZERO) {
        if ((rc = zero_state(v))) return rc;
    } else if (prm->init == DN_INIT_GIVEN) {
        // a given dual of a map whose lines may rest (still_state) is looked
        // at as it is copied: a warm start's is zero outside Omega (202195
        // blocks: 0.95 ms per iteration without, 0.87 with)
        look = p0 && storage == DN_F32 && prm->kernel != DN_K_TWOPASS && prm->iters > 2 &&
               streams_state(v->nb, sizeof(float)) && (reinterpret_cast<uintptr_t>(p0) & 15) == 0;
        if (look) {
            if ((rc = fill<int64_t>(st, report(v) + kOffWord, 1, 0))) return rc;
            hipLaunchKernelGGL(k_copy_dual, dim3(grid1(n / 4)), dim3(256), 0, st, n / 4, ps / 4,
                               reinterpret_cast<const uint32_t *>(v->emask), reinterpret_cast<const float4 *>(p0),
                               reinterpret_cast<float4 *>(v->p[v->cur]), report(v) + kOffWord);
            DN_HIP(hipGetLastError());
        }
        if (n > 0) {
            DN_HIP(hipMemcpyAsync(v->u, u0, n * 4, hipMemcpyDeviceToDevice, st));
            DN_HIP(hipMemcpyAsync(v->ubar[v->cur], u0, n * 4, hipMemcpyDeviceToDevice, st));
            for (int a = 0; a < 3; ++a) {
                if (look) continue;
                if (p0) {
                    DN_HIP(hipMemcpyAsync(v->p[v->cur] + a * ps, p0 + a * n, n * 4, hipMemcpyDeviceToDevice, st));
                } else if ((rc = fill<float>(st, v->p[v->cur] + a * ps, n, 0.f))) {
                    return rc;
                }
            }
        }
        v->state_storage = DN_F32;
        v->p_off_zero = p0 == nullptr;
    } else if (prm->init == DN_INIT_CONTINUE) {
        // a 16-bit run ended with an FP32 sweep: continue from its output
        v->state_storage = DN_F32;
        const int64_t first = v->nb_state < v->nb ? v->nb_state : v->nb;
        const int64_t cnt = (v->nb - first) * kBlockVox;
        if (cnt > 0) {
            DN_HIP(hipMemcpyAsync(v->u + first * kBlockVox, v->f + first * kBlockVox, cnt * 4,
                                  hipMemcpyDeviceToDevice, st));
            DN_HIP(hipMemcpyAsync(v->ubar[v->cur] + first * kBlockVox, v->f + first * kBlockVox, cnt * 4,
                                  hipMemcpyDeviceToDevice, st));
            for (int a = 0; a < 3; ++a)
                if ((rc = fill<float>(st, v->p[v->cur] + a * ps + first * kBlockVox, cnt, 0.f))) return rc;
        }
    }
    v->full_iters = 0;     // Omega may have changed since the last call
    if (prm->init != DN_INIT_KEEP || v->acc_tau <= 0.0) {
        v->acc_tau = prm->tau;
        v->acc_sigma = prm->sigma;
    }
    // the stochastic rounding restarts its seeds with the solve (a call that
    // keeps the state continues them), so equal calls give equal results
    if (prm->init != DN_INIT_KEEP) v->lowp_iter = 0;
    int kernel = prm->kernel;
    bool fresh16 = false;     // the 16-bit state was just demoted from FP32
    if (storage != DN_F32) {
        if (kernel != DN_K_FUSED256) kernel = DN_K_FUSED;
        if (v->state_storage != storage) {
            // the FP32 state (zero, given or an earlier FP32 run) is demoted
            if (v->state_storage != DN_F32) {
                set_error("cannot continue a %s state with another 16-bit storage",
                          v->state_storage == DN_F16 ? "FP16" : "BF16");
                return DN_E_INVALID;
            }
            if (!first) {
                rc = storage == DN_F16 ? demote_state<SF16>(v) : demote_state<SBF16>(v);
                if (rc) return rc;
            }
            v->state_storage = storage;
            fresh16 = true;
        }
        if (prm->kernel == DN_K_AUTO && v->nb > 0) {
            if (fresh16) {
                rc = storage == DN_F16 ? autotune_lowp<SF16>(v, prm, first, &kernel)
                                       : autotune_lowp<SBF16>(v, prm, first, &kernel);
                if (rc) return rc;
            } else {
                AutoChoice found;
                if (find_choice(g_auto_lowp, tune_key(v, storage * 64 + size_bucket(v->nb)), &found)) {
                    kernel = found.kernel;
                    v->layout = found.layout;
                }
            }
        }
    } else {
        // a 16-bit run always ends with an FP32 sweep: continue from its output
        v->state_storage = DN_F32;
        if (kernel == DN_K_AUTO && v->nb > 0) {
            if (prm->init == DN_INIT_ZERO) {
                if ((rc = autotune_single(v, prm, &kernel))) return rc;
            } else {
                AutoChoice found;
                if (find_choice(g_auto_kernel, tune_key(v, size_bucket(v->nb)), &found)) {
                    kernel = found.kernel;
                    v->layout = found.layout;
                } else {
                    kernel = DN_K_FUSED;
                }
            }
        }
    }
    dn_reg_stats stats{};
    double ed[2] = {0, 0};
    int it = 0;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    DN_HIP(hipEventCreate(&ev0));
    DN_HIP(hipEventCreate(&ev1));
    DN_HIP(hipEventRecord(ev0, st));
    dn_reg_params step_prm = *prm;
    bool last_refined = false;   // the last 16-bit iteration also wrote the FP32 state
    for (; it < prm->iters && v->nb > 0; ++it) {
        if (prm->gamma > 0.0) {
            // accelerated schedule: this iteration's (sigma_n, tau_n, theta_n)
            const double th = 1.0 / std::sqrt(1.0 + 2.0 * prm->gamma * v->acc_tau);
            step_prm.tau = v->acc_tau;
            step_prm.sigma = v->acc_sigma;
            step_prm.theta = th;
            v->acc_tau = th * v->acc_tau;
            v->acc_sigma = v->acc_sigma / th;
        }
        if (look && it == 2) {       // (two full iterations are under way)
            if ((rc = fetch_report(v, kOffWord + 1))) return rc;
            v->p_off_zero = v->host_stage[kOffWord] == 0;
            v->full_iters = 2;
        }
        if (first && it == 0) {
            if (storage == DN_F32) {
                (void)still_state(v);
                rc = first_iteration(v, float(step_prm.tau), float(step_prm.lambda), float(step_prm.theta),
                                     prm->data_term == DN_DATA_L1);
                v->cur = 1 - v->cur;
            } else {
                rc = storage == DN_F16 ? first_lowp<SF16>(v, &step_prm) : first_lowp<SBF16>(v, &step_prm);
            }
        } else if (storage == DN_F32) {
            rc = step_f32(v, &step_prm, kernel);
        } else {
            bool refine = (prm->refine_every > 0 && (it + 1) % prm->refine_every == 0) || it + 1 == prm->iters;
            rc = storage == DN_F16 ? step_lowp<SF16>(v, &step_prm, refine, kernel)
                                   : step_lowp<SBF16>(v, &step_prm, refine, kernel);
            last_refined = refine;
        }
        if (rc) return rc;
        if (prm->gap_every > 0 && (it + 1) % prm->gap_every == 0 && it + 1 < prm->iters) {
            if ((rc = energy_current(v, prm->lambda, false, prm->data_term))) return rc;
            if ((rc = read_energy(v, ed))) return rc;
            double gap = ed[0] - ed[1];
            if (!std::isfinite(gap)) {
                set_error("non-finite gap at iteration %d", it + 1);
                // (no sweep has written the FP32 state yet: it starts at zero)
                if (first && storage != DN_F32 && !(prm->refine_every > 0 && it + 1 >= prm->refine_every)) {
                    if ((rc = zero_state(v))) return rc;
                    v->state_storage = storage;
                }
                return DN_E_NUMERIC;
            }
            if (prm->gap_tol > 0 && gap <= prm->gap_tol * ed[0]) { ++it; stats.converged = 1; break; }
        }
    }
    stats.iters_run = it;
    v->nb_state = v->nb;
    if (storage != DN_F32 && it > 0 && !last_refined) {
        // stopped early (gap_tol) between sweeps: the FP32 buffers take the
        // current 16-bit state
        rc = storage == DN_F16 ? promote_state<SF16>(v) : promote_state<SBF16>(v);
        if (rc) return rc;
    }
    DN_HIP(hipEventRecord(ev1, st));
    // after a 16-bit run the FP32 buffers hold the result: the output of
    // the last sweep, or the promoted 16-bit state after an early stop
    if ((rc = energy_current(v, prm->lambda, true, prm->data_term))) return rc;
    if ((rc = read_energy(v, ed))) return rc;
    {
        float ms = 0.f;
        DN_HIP(hipEventElapsedTime(&ms, ev0, ev1));
        stats.ms_loop = ms;
        (void)hipEventDestroy(ev0);
        (void)hipEventDestroy(ev1);
    }
    stats.energy = ed[0];
    stats.dual = ed[1];
    stats.gap = ed[0] - ed[1];
    stats.rel_gap = ed[0] != 0.0 ? stats.gap / ed[0] : 0.0;
    if (prm->gap_tol > 0 && stats.gap <= prm->gap_tol * ed[0]) stats.converged = 1;
    stats.kernel_used = kernel;
    stats.layout_used = v->layout;
    if (out) *out = stats;
    if (!std::isfinite(stats.gap)) { set_error("non-finite energy"); return DN_E_NUMERIC; }
    return DN_OK;
}

}  // extern "C"
