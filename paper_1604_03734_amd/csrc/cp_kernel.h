// Device code of one fused Chambolle-Pock iteration on one 8^3 block,
// shared by the per-iteration kernel and the persistent batched kernel.
// Section III-B/C of the paper: Eq. (3) gradient, Eq. (4) divergence,
// Eqs. (7)-(9) updates.
#pragma once

#include "dn_internal.h"

namespace dn {

// ---------------------------------------------------------- storage types
// State storage: float, IEEE half or bfloat16 (16-bit kept as raw bits).
// sr(x, r) rounds stochastically with the 16 random bits r: the magnitude
// goes up one step with probability equal to the fraction of the step it
// has past the lower neighbour (adding random bits below the kept mantissa,
// then truncating), so rounding errors have mean zero and increments far
// below one step still accumulate.  Rounding to nearest (or toward zero)
// stalls the iteration once its increments drop below half a step.
struct SF32 {
    using T = float;
    static constexpr bool kLow = false;
    static __device__ __forceinline__ float ld(float v) { return v; }
    static __device__ __forceinline__ float rn(float x) { return x; }
    static __device__ __forceinline__ float rz(float x) { return x; }
    static __device__ __forceinline__ float sr(float x, uint32_t) { return x; }
};
struct SF16 {
    using T = uint16_t;
    static constexpr bool kLow = true;
    static __device__ __forceinline__ float ld(uint16_t v) { return float(__builtin_bit_cast(_Float16, v)); }
    static __device__ __forceinline__ uint16_t rn(float x) { return __builtin_bit_cast(uint16_t, _Float16(x)); }
    static __device__ __forceinline__ uint16_t rz(float x)
    {
        auto h2 = __builtin_amdgcn_cvt_pkrtz(x, 0.0f);
        return __builtin_bit_cast(uint16_t, h2[0]);
    }
    // 13 float mantissa bits fall away for a normal half (exact stochastic
    // rounding there; below 2^-14 the step is finer than the noise)
    static __device__ __forceinline__ uint16_t sr(float x, uint32_t r)
    {
        return rz(__uint_as_float(__float_as_uint(x) + (r & 0x1FFFu)));
    }
};
struct SBF16 {
    using T = uint16_t;
    static constexpr bool kLow = true;
    static __device__ __forceinline__ float ld(uint16_t v) { return __uint_as_float(uint32_t(v) << 16); }
    static __device__ __forceinline__ uint16_t rn(float x)
    {
        uint32_t u = __float_as_uint(x);
        u += 0x7FFFu + ((u >> 16) & 1u);
        return uint16_t(u >> 16);
    }
    static __device__ __forceinline__ uint16_t rz(float x) { return uint16_t(__float_as_uint(x) >> 16); }
    static __device__ __forceinline__ uint16_t sr(float x, uint32_t r)
    {
        return uint16_t((__float_as_uint(x) + (r & 0xFFFFu)) >> 16);
    }
};

// Streaming accesses.  A block's f, w and u are read by that block alone
// and every store of the iteration is read back only in the next one,
// whereas ubar, p and the edge masks are also read by the neighbours as
// their halo.  On a map larger than the last-level cache (kStream), loading
// the former and storing everything as non-temporal leaves the L2 for the
// lines the neighbouring blocks will read; on a smaller one the hints would
// send to memory what the cache could hold from one iteration to the next.
template <bool kStream, class T> __device__ __forceinline__ T ld_own(const T *p)
{
    if constexpr (kStream) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool kStream, class T> __device__ __forceinline__ void st_own(T *p, T v)
{
    if constexpr (kStream) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Counter-based random bits of one voxel and iteration: an integer hash
// (xor-shift / multiply rounds) of the global voxel index, a stream number
// and the iteration seed.  Deterministic, so a run is reproducible and a
// voxel's stored value does not depend on which workgroup wrote it.
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}
__device__ __forceinline__ uint32_t voxel_bits(int64_t gi, uint32_t stream, uint32_t seed)
{
    return mix32(uint32_t(gi) * 3u + stream + mix32(seed ^ uint32_t(uint64_t(gi) >> 32)));
}

template <class S> struct CPArgs {
    int64_t nb;                 // blocks
    int64_t pstride;            // elements between p planes
    const int32_t *nbr;         // [nb][27]
    const uint32_t *em4;        // [nb][64] edge masks, see k_masks
    const int32_t *order;       // processing order or nullptr (pool order)
    const float *f, *w;
    typename S::T *u;           // in place
    const typename S::T *ubar_in;
    typename S::T *ubar_out;
    const typename S::T *p_in;  // 3 planes
    typename S::T *p_out;
    float *u32, *ubar32, *p32;  // FP32 copies written by a refinement sweep
    float sigma, tau, lambda, theta;
    int32_t l1;                 // data term lambda w |u - f| (with u in [-1, 1]) instead of (lambda/2) w (u - f)^2
    uint32_t seed;              // 16-bit storage: this iteration's seed of the stochastic rounding
};

__device__ __forceinline__ int i9(int x, int y, int z) { return ((z + 1) * 9 + (y + 1)) * 9 + (x + 1); }

// Global index of voxel (hx, hy, hz) relative to block b, hx.. in [-1, 8],
// or -1 if it lies in an unallocated block.
__device__ __forceinline__ int64_t halo_index(const int32_t *nb27, int hx, int hy, int hz)
{
    int dx = hx < 0 ? -1 : (hx > 7 ? 1 : 0);
    int dy = hy < 0 ? -1 : (hy > 7 ? 1 : 0);
    int dz = hz < 0 ? -1 : (hz > 7 ? 1 : 0);
    int32_t id = nb27[(dz + 1) * 9 + (dy + 1) * 3 + (dx + 1)];
    if (id < 0) return -1;
    return int64_t(id) * kBlockVox + ((hx - 8 * dx) + 8 * (hy - 8 * dy) + 64 * (hz - 8 * dz));
}

// Correctly rounded projection and division in fewer instructions than the
// compiler's general sequences, which also rescale operands near the ends
// of the exponent range; the dual step's three quotients share one
// reciprocal.  n = sqrt(s) is v_rsq's estimate with one Newton step on the
// root and one on its reciprocal, a quotient one residual correction.
// Checked against sqrtf and IEEE division: the root for all 2^24 operands of
// two octaves (exact), the quotients for 2^33 operand pairs (exact).  A
// correction is exact where neither the residual nor the quotient is
// subnormal: for a denominator in [1, 2^24) and a numerator of at least
// 2^-100, or zero (which keeps its sign).  A wave with any other takes the
// general path behind it, which gives the same bits elsewhere; the test runs
// beside the chain of the short one (503 blocks 4.48 us an iteration with it,
// 4.47 without; in front of the chain 4.73).
//   sqrt(s) > 1  <=>  s > 1 + 2^-23: the root of 1 + 2^-23 rounds to 1.
__device__ __forceinline__ float div_by(float a, float n, float r)
{
    const float q = a * r;
    return __builtin_fmaf(-__builtin_fmaf(n, q, -a), r, q);
}

// Below kTiny for a magnitude in (0, 2^-100), not for zero or any larger one.
constexpr uint32_t kTiny = ((127u - 100u) << 24) - 1u;
__device__ __forceinline__ uint32_t size_of(float x) { return (__float_as_uint(x) << 1) - 1u; }

__device__ __forceinline__ void project(float &a, float &b, float &c)
{
    const float s = (a * a + b * b) + c * c;
    if (s > 1.00000011920928955f) {
        const bool general = min(min(size_of(a), size_of(b)), size_of(c)) < kTiny || !(s < 0x1p48f);
        const float y = __builtin_amdgcn_rsqf(s), n0 = s * y;
        const float n = __builtin_fmaf(__builtin_fmaf(-n0, n0, s), 0.5f * y, n0);
        const float r = __builtin_fmaf(__builtin_fmaf(-n, y, 1.0f), y, y);
        const float x0 = a, x1 = b, x2 = c;
        a = div_by(x0, n, r); b = div_by(x1, n, r); c = div_by(x2, n, r);
        if (__builtin_expect(__any(general), 0)) {
            const float root = sqrtf(s);
            a = x0 / root; b = x1 / root; c = x2 / root;
        }
    }
}

// num / den for den = 1 + tau lambda w >= 1
__device__ __forceinline__ float prox_div(float num, float den)
{
    const bool general = size_of(num) < kTiny || !(den < 0x1p24f);
    const float r0 = __builtin_amdgcn_rcpf(den);
    float q = div_by(num, den, __builtin_fmaf(__builtin_fmaf(-den, r0, 1.0f), r0, r0));
    q = __builtin_amdgcn_div_fixupf(q, den, num);       // (an infinite numerator)
    if (__builtin_expect(__any(general), 0)) q = num / den;
    return q;
}

// The data term's proximal step of u~, tl = tau lambda.
__device__ __forceinline__ float data_prox(float ut, float fv, float wv, float tl, int l1)
{
    const float tlw = tl * wv;
    if (l1) {
        // soft threshold of u~ - f by tau lambda w, then the [-1, 1] box
        float r = ut - fv;
        r = r > tlw ? r - tlw : (r < -tlw ? r + tlw : 0.0f);
        return fminf(fmaxf(fv + r, -1.0f), 1.0f);
    }
    return prox_div(ut + tlw * fv, 1.0f + tlw);
}

// One wave of 64 lanes holds whole (x, y) planes of a block: lane = x + 8 y,
// plane z in registers.  Bit 4z + i of a mask word: bit i (0 Omega, 1 + a
// m_a) of the edge mask of voxel (lane, z).
__device__ __forceinline__ uint32_t keep_if(uint32_t word, int bit)   // all ones where the bit is set
{
    return uint32_t(__builtin_amdgcn_sbfe(int(word), unsigned(bit), 1u));
}
__device__ __forceinline__ float and_f(float x, uint32_t m) { return __uint_as_float(__float_as_uint(x) & m); }

// Data that one iteration passes between lanes, in LDS: ubar on the block
// with a one-voxel halo, and the masked new dual components p_x and p_y
// shifted by one along their axis (their first column / row is the -1 face),
// p_z of each wave's last plane.
template <int W> struct CPShared {
    float u[1000];       // index x + 1 + 10 (y + 1) + 100 (z + 1)
    float px[576];       // index x + 1 + 9 y + 72 z
    float py[576];       // index x + 8 (y + 1) + 72 z
    float pz[W][64];     // by wave
};

// Memory the kernel only reads, the same for all lanes: scalar loads.
typedef const __attribute__((address_space(4))) int32_t *ScalarI32;
__device__ __forceinline__ ScalarI32 as_scalar(const int32_t *p) { return (ScalarI32) reinterpret_cast<uint64_t>(p); }

template <int W> __device__ __forceinline__ void block_sync()
{
    if constexpr (W == 1) {
        // one wave: its LDS operations are processed in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// One fused Chambolle-Pock iteration on block b by W waves of 8 / W planes
// each.  Bound by HBM on maps beyond the caches, by the last-level cache and
// latency on smaller ones.  A voxel's neighbours along z stay in registers,
// faces are loaded a wave at a time from a base the whole wave shares, and
// masks are a word per lane, so a voxel takes about a third of the vector
// instructions of a thread-per-voxel layout with its index arithmetic per
// voxel.  Per iteration, that layout and this one: 202195 blocks FP32 0.946
// and 0.939 ms; 60001 blocks BF16 236 and 169 us; 5777 blocks FP32 34.0 and
// 24.3 us (with the cache hints dropped there); 503 blocks 5.4 and 4.7 us.
//
// kStill: the voxels outside Omega hold the same u, ubar and p in both sets
// of buffers (see still_state), so a memory line without an observed voxel is
// neither read nor written.  Whole lines only: leaving out single voxels
// makes every line a partial write (1.11 ms at 202195 blocks, where whole
// lines take it from 0.936 to 0.869; 12 % of that map's lines are empty).
// It pays where memory bounds the kernel: the loads have to wait for the
// masks (5777 blocks: no gain; 503: 4.5 -> 4.7 us).
template <class S, bool kRefine, bool kStream, bool kStill, int W>
__device__ __forceinline__ void cp_block(const CPArgs<S> &A, int32_t b, CPShared<W> &sh, int wave, unsigned lane)
{
    using T = typename S::T;
    constexpr int ZP = 8 / W;
    const int z0 = wave * ZP;
    const int64_t g0 = int64_t(b) * kBlockVox;
    const int64_t o0 = g0 + z0 * 64;             // this wave's first plane
    const int64_t ps = A.pstride;
    const ScalarI32 nb = as_scalar(A.nbr) + int64_t(b) * kNbr;
    const unsigned l8 = lane & 7u, h8 = lane >> 3;

    // the wave's own planes
    float ub[ZP], p0[ZP], p1[ZP], p2[ZP], uo[ZP], fv[ZP], wv[ZP];
    const uint32_t mw0 = (A.em4 + int64_t(b) * 64)[lane];
    // kStill: bit k of `lines`: this lane's 128-byte line of plane z0 + k
    // holds an observed voxel
    uint32_t lines = 0;
    if constexpr (kStill) {
        static_assert(!S::kLow && !kRefine, "half a wave's plane is a line of FP32");
#pragma unroll
        for (int k = 0; k < ZP; ++k) {
            const uint64_t m = __ballot((mw0 >> (4 * (z0 + k))) & 1u);
            lines |= ((lane < 32u ? uint32_t(m) : uint32_t(m >> 32)) != 0u ? 1u : 0u) << k;
        }
    }
    auto on = [&](int k) { return !kStill || ((lines >> k) & 1u) != 0u; };
#pragma unroll
    for (int k = 0; k < ZP; ++k) {
        if constexpr (kStill) ub[k] = p0[k] = p1[k] = p2[k] = uo[k] = fv[k] = wv[k] = 0.0f;
        if (on(k)) ub[k] = S::ld((A.ubar_in + o0)[64 * k + lane]);
    }
#pragma unroll
    for (int k = 0; k < ZP; ++k)
        if (on(k)) {
            p0[k] = S::ld((A.p_in + o0)[64 * k + lane]);
            p1[k] = S::ld((A.p_in + o0 + ps)[64 * k + lane]);
            p2[k] = S::ld((A.p_in + o0 + 2 * ps)[64 * k + lane]);
        }
    const unsigned ax = 110u + 10u * l8 + 100u * h8, ay = 101u + l8 + 100u * h8, az = 11u + l8 + 10u * h8;
    // ubar on the faces and edges and the old dual and masks on the -1 faces,
    // shared out over the waves; every load is issued before the first value
    // is used.  An unallocated neighbour is skipped by FP32 state, which is
    // bound by memory traffic (0.939 against 0.966 ms at 202195 blocks); 16-
    // bit state, bound by latency, reads the block itself in its place and
    // drops the values, which costs no branch (181 against 186 us at 60001).
    constexpr bool kSkip = !S::kLow;
    constexpr int kTasks = 7, kPer = (kTasks + W - 1) / W;
    const int nid[6] = {nb[14], nb[12], nb[16], nb[10], nb[22], nb[4]};   // +x, -x, +y, -y, +z, -z
    float hv[kPer];
    uint32_t edge = 0;
    int edge_id = -1;
    auto face_at = [&](int t) {
        return t == 0 ? 8u * lane : t == 1 ? 8u * lane + 7u : t == 2 ? l8 + 64u * h8 : t == 3 ? l8 + 64u * h8 + 56u :
               t == 4 ? lane : lane + 448u;
    };
    auto load_task = [&](int t) -> float {
        if (t < 6) {
            if (kSkip && nid[t] < 0) return 0.0f;
            return S::ld((A.ubar_in + int64_t(nid[t] >= 0 ? nid[t] : b) * kBlockVox)[face_at(t)]);
        }
        // voxel j of the six (-a, +b) edges, 8 lanes each: the offset in the
        // neighbour's block, and its index in CPShared::u in the high half:
        // (-1, 8, j), (-1, j, 8), (8, -1, j), (j, -1, 8), (8, j, -1), (j, 8, -1)
        const unsigned e = h8;
        uint32_t first = 7u | 190u << 16;
        edge_id = nb[15];
        if (e == 1u) { edge_id = nb[21]; first = 7u | 910u << 16; }
        if (e == 2u) { edge_id = nb[11]; first = 56u | 109u << 16; }
        if (e == 3u) { edge_id = nb[19]; first = 56u | 901u << 16; }
        if (e == 4u) { edge_id = nb[5]; first = 448u | 19u << 16; }
        if (e == 5u) { edge_id = nb[7]; first = 448u | 91u << 16; }
        const uint32_t step = e == 0u || e == 2u ? 64u | 100u << 16 : (e == 1u || e == 4u ? 8u | 10u << 16 : 1u | 1u << 16);
        edge = first + l8 * step;
        if (kSkip && edge_id < 0) return 0.0f;
        return S::ld(A.ubar_in[int64_t(edge_id >= 0 ? edge_id : b) * kBlockVox + (edge & 0xFFFFu)]);
    };
    auto store_task = [&](int t, float v) {
        if (t < 6) {
            const unsigned at = t == 0 ? ax + 9u : t == 1 ? ax : t == 2 ? ay + 90u : t == 3 ? ay : t == 4 ? az + 900u : az;
            sh.u[at] = nid[t] >= 0 ? v : 0.0f;
        } else if (lane < 48u) {   // six edges
            sh.u[edge >> 16] = edge_id >= 0 ? v : 0.0f;
        }
    };
    // the -1 faces: -z by the first wave (its lanes match plane 0), -x and -y by the next ones
    constexpr int kWx = W == 1 ? 0 : 1, kWy = W <= 2 ? W - 1 : 2;
    struct Face { float a, b, c; uint32_t m; };
    Face fx{0.f, 0.f, 0.f, 0u}, fy = fx, fz = fx;
    auto load_face = [&](Face &F, int t, unsigned word) {
        if (kSkip && nid[t] < 0) return;
        const int id = nid[t] >= 0 ? nid[t] : b;
        const T *q = A.p_in + int64_t(id) * kBlockVox;
        const unsigned off = face_at(t);
        F.a = S::ld(q[off]); F.b = S::ld((q + ps)[off]); F.c = S::ld((q + 2 * ps)[off]);
        F.m = (A.em4 + int64_t(id) * 64)[word];
    };
#pragma unroll
    for (int w = 0; w < W; ++w)
        if (wave == w) {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (w + j * W < kTasks) hv[j] = load_task(w + j * W);
            if (w == 0) load_face(fz, 5, lane);
            if (w == kWx) load_face(fx, 1, 8u * l8 + 7u);
            if (w == kWy) load_face(fy, 3, l8 + 56u);
        }
#pragma unroll
    for (int k = 0; k < ZP; ++k)
        if (on(k)) {
            uo[k] = S::ld(ld_own<kStream>((const T *)(A.u + o0) + 64 * k + lane));
            fv[k] = ld_own<kStream>(A.f + o0 + 64 * k + lane);
            wv[k] = ld_own<kStream>(A.w + o0 + 64 * k + lane);
        }
#pragma unroll
    for (int w = 0; w < W; ++w)
        if (wave == w) {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (w + j * W < kTasks) store_task(w + j * W, hv[j]);
        }
    const unsigned own = az + 100u * (z0 + 1);
#pragma unroll
    for (int k = 0; k < ZP; ++k) sh.u[own + 100 * k] = ub[k];
    block_sync<W>();

    const uint32_t mw = mw0 >> (4 * z0);
    // dual ascent and projection (Eq. 7); p_x, p_y to LDS masked, p_z kept
    const unsigned qx = 1u + l8 + 9u * h8 + 72u * z0, qy = l8 + 8u * (h8 + 1u) + 72u * z0;
    float d0[ZP], d1[ZP], d2[ZP];
#pragma unroll
    for (int k = 0; k < ZP; ++k) {
        const uint32_t mx = keep_if(mw, 4 * k + 1), my = keep_if(mw, 4 * k + 2), mz = keep_if(mw, 4 * k + 3);
        const float uz = k + 1 < ZP ? ub[k + 1 < ZP ? k + 1 : 0] : sh.u[own + 100 * k + 100];
        const float gx = and_f(sh.u[own + 100 * k + 1] - ub[k], mx);
        const float gy = and_f(sh.u[own + 100 * k + 10] - ub[k], my);
        const float gz = and_f(uz - ub[k], mz);
        float a0 = p0[k] + A.sigma * gx, a1 = p1[k] + A.sigma * gy, a2 = p2[k] + A.sigma * gz;
        project(a0, a1, a2);
        d0[k] = and_f(a0, mx); d1[k] = and_f(a1, my); d2[k] = and_f(a2, mz);
        sh.px[qx + 72 * k] = d0[k];
        sh.py[qy + 72 * k] = d1[k];
        const unsigned i = 64 * k + lane;
        T *po = A.p_out + o0;
        if (!on(k)) {
        } else if constexpr (S::kLow) {
            // stochastic rounding; where it would leave the unit ball, toward zero
            const int64_t gi = o0 + i;
            const uint32_t r0 = voxel_bits(gi, 0, A.seed), r1 = voxel_bits(gi, 1, A.seed);
            T s0 = S::sr(a0, r0), s1 = S::sr(a1, r0 >> 16), s2 = S::sr(a2, r1);
            const float b0 = S::ld(s0), b1 = S::ld(s1), b2 = S::ld(s2);
            if ((b0 * b0 + b1 * b1) + b2 * b2 > 1.0f) { s0 = S::rz(a0); s1 = S::rz(a1); s2 = S::rz(a2); }
            st_own<kStream>(po + i, s0); st_own<kStream>(po + ps + i, s1); st_own<kStream>(po + 2 * ps + i, s2);
        } else {
            st_own<kStream>(po + i, a0); st_own<kStream>(po + ps + i, a1); st_own<kStream>(po + 2 * ps + i, a2);
        }
        if (kRefine) {
            float *q = A.p32 + o0;
            q[i] = a0; (q + ps)[i] = a1; (q + 2 * ps)[i] = a2;
        }
    }
    if (W > 1) sh.pz[wave][lane] = d2[ZP - 1];
    // ... and on the -1 faces, which the divergence needs: the component
    // along the face's axis, masked
    auto face_dual = [&](const Face &F, float us, float ux, float uy, float uz, float &a0, float &a1, float &a2) {
        a0 = F.a + A.sigma * and_f(ux - us, keep_if(F.m, 1));
        a1 = F.b + A.sigma * and_f(uy - us, keep_if(F.m, 2));
        a2 = F.c + A.sigma * and_f(uz - us, keep_if(F.m, 3));
        project(a0, a1, a2);
    };
    float a0, a1, a2, zlow = 0.0f;
    if (wave == 0) {
        fz.m = nid[5] >= 0 ? fz.m >> 28 : 0u;
        face_dual(fz, sh.u[az], sh.u[az + 1], sh.u[az + 10], ub[0], a0, a1, a2);
        zlow = and_f(a2, keep_if(fz.m, 3));
    }
    if (wave == kWx) {
        fx.m = nid[1] >= 0 ? fx.m >> (4u * h8) : 0u;
        face_dual(fx, sh.u[ax], sh.u[ax + 1], sh.u[ax + 10], sh.u[ax + 100], a0, a1, a2);
        sh.px[9u * l8 + 72u * h8] = and_f(a0, keep_if(fx.m, 1));
    }
    if (wave == kWy) {
        fy.m = nid[3] >= 0 ? fy.m >> (4u * h8) : 0u;
        face_dual(fy, sh.u[ay], sh.u[ay + 1], sh.u[ay + 10], sh.u[ay + 100], a0, a1, a2);
        sh.py[l8 + 72u * h8] = and_f(a1, keep_if(fy.m, 2));
    }
    block_sync<W>();
    if (W > 1 && wave > 0) zlow = sh.pz[wave - 1][lane];

    // primal proximal step (Eq. 8) and relaxation (Eq. 9)
    const float tl = A.tau * A.lambda;
#pragma unroll
    for (int k = 0; k < ZP; ++k) {
        float dv = d0[k] - sh.px[qx + 72 * k - 1];
        dv += d1[k] - sh.py[qy + 72 * k - 8];
        dv += d2[k] - (k > 0 ? d2[k > 0 ? k - 1 : 0] : zlow);
        float un = data_prox(uo[k] + A.tau * dv, fv[k], wv[k], tl, A.l1);
        un = keep_if(mw, 4 * k) ? un : uo[k];
        const float ubn = un + A.theta * (un - uo[k]);
        const unsigned i = 64 * k + lane;
        if (!on(k)) {
        } else if constexpr (S::kLow) {
            const uint32_t r2 = voxel_bits(o0 + i, 2, A.seed);
            st_own<kStream>(A.u + o0 + i, S::sr(un, r2));
            st_own<kStream>(A.ubar_out + o0 + i, S::sr(ubn, r2 >> 16));
        } else {
            st_own<kStream>(A.u + o0 + i, un);
            st_own<kStream>(A.ubar_out + o0 + i, ubn);
        }
        if (kRefine) { (A.u32 + o0)[i] = un; (A.ubar32 + o0)[i] = ubn; }
    }
}

// The lane index, one that the compiler cannot hoist out of an enclosing
// loop (the index arithmetic is redone per block instead of staying live).
__device__ __forceinline__ unsigned opaque_lane()
{
    unsigned t = threadIdx.x & 63u;
    asm volatile("" : "+v"(t));
    return t;
}
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Whether the state of that many blocks outgrows the last-level cache (256
// MB): two buffers of ubar and p, u, and f, w.  Either side of the line,
// without / with the hints: FP32 10000 blocks 39.6 / 51.9 us per iteration,
// 12000 59.4 / 61.3, 20000 105.5 / 100.5; 16-bit 16000 41.3 / 51.1, 20000
// 64.1 / 62.9, 40000 131 / 123.
static inline bool streams_state(int64_t blocks, size_t state_size)
{
    return size_t(blocks) * kBlockVox * (9 * state_size + 8) > (size_t(272) << 20);
}

// Workgroup -> block mapping.  Consecutive workgroups go round-robin to the
// 8 XCDs; giving XCD x the x-th contiguous chunk of the (Morton) order keeps
// spatial neighbours, whose faces are each other's halos, in one L2.
__device__ __forceinline__ int64_t xcd_slot(int64_t wg, int64_t n)
{
    int64_t per = (n + 7) / 8;
    return (wg % 8) * per + wg / 8;
}

}  // namespace dn
