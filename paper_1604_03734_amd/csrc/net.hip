// Learned warm start: a 3-layer 3x3x3 convolutional network on 10^3 tiles
// (an 8^3 block plus a one-voxel halo), 2 -> 16 -> 16 -> 1 channels, ReLU,
// "same" zero padding inside the tile.
//
// Forward pass of given tiles: k_net_tiles, one launch on
// v_mfma_f32_16x16x16_bf16 (bfloat16 operands, float32 accumulation; one
// MFMA = 16 voxels x 16 output channels x 16 input channels of one tap).
//
// Inference path (warm start) and the forward half of a training step: one
// fused launch, k_net_fwd, on v_mfma_f32_16x16x32_bf16 with all activations
// in LDS and the weights in registers.
#include <cstring>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "dn_internal.h"

namespace dn {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kT = 1000;      // voxels of a 10^3 tile
constexpr int kC = 16;        // channels of a stored activation
constexpr int kTaps = 27;
constexpr int kWPack = kTaps * kC * kC;   // one packed layer: [tap][co][ci]
constexpr int kMT = 63;       // 16-voxel row tiles covering 1000 voxels
// Training layouts: an activation on the tile's 10^3 grid padded by one zero
// voxel on every side (12^3 = 1728 entries, index (x+1) + 12 (y+1) +
// 144 (z+1)); a gradient on the compact rows of that grid (the 100 rows
// (y, z) of 12 entries, padding entries x = -1 and x = 10 zero, index
// (x+1) + 12 (10 z + y), 1216 entries with the tail zero).  The 16 channels of
// an entry are contiguous; the layer-1 input has its two channels one after
// the other, and d3 has one.
constexpr int kPadVox = 1728;
// offsets of the layers in the canonical 8241-float parameter vector
constexpr int kW1 = 0, kB1 = 16 * 2 * 27, kW2 = kB1 + 16, kB2 = kW2 + 16 * 16 * 27, kW3 = kB2 + 16,
              kB3 = kW3 + 16 * 27;
constexpr int kRowVox = 1216;

__device__ __forceinline__ uint16_t f2bf(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float(uint32_t(v) << 16); }

__device__ __forceinline__ int64_t halo_vox(const int32_t *nb27, int hx, int hy, int hz)
{
    int dx = hx < 0 ? -1 : (hx > 7 ? 1 : 0);
    int dy = hy < 0 ? -1 : (hy > 7 ? 1 : 0);
    int dz = hz < 0 ? -1 : (hz > 7 ? 1 : 0);
    int32_t id = nb27[(dz + 1) * 9 + (dy + 1) * 3 + (dx + 1)];
    if (id < 0) return -1;
    return int64_t(id) * kBlockVox + ((hx - 8 * dx) + 8 * (hy - 8 * dy) + 64 * (hz - 8 * dz));
}

// Input tiles of the n listed blocks, float [n][2][1000]: channel 0 f,
// channel 1 log(1 + w) / log(101); 0 for voxels of unallocated neighbours.
// perm exchanges the tile's x axis with the volume's y (1) or z (2) axis.
__global__ void k_gather(const int32_t *__restrict__ nbr, const float *__restrict__ f, const float *__restrict__ w,
                         const int32_t *__restrict__ blocks, int64_t n, float *__restrict__ tiles, int perm)
{
    int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= n * kT) return;
    int64_t i = k / kT;
    int v = int(k % kT);
    int64_t b = blocks[i];
    int x = v % 10, y = (v / 10) % 10, z = v / 100;
    if (perm == 1) { int s = x; x = y; y = s; }
    if (perm == 2) { int s = x; x = z; z = s; }
    int64_t j = halo_vox(nbr + b * kNbr, x - 1, y - 1, z - 1);
    float fv = 0.f, wv = 0.f;
    if (j >= 0) {
        fv = f[j];
        wv = float(log(1.0 + double(w[j])) / log(101.0));
    }
    tiles[i * 2 * kT + v] = fv;
    tiles[i * 2 * kT + kT + v] = wv;
}


// The gradient of all 8241 parameters from the per-workgroup partials of
// the three layers, written to the
// canonical parameter layout and scaled by 1 / N (the partials are of the
// loss before its division by N: every entry is linear in d3).  The sum over p has a fixed order: a
// workgroup takes 32 consecutive partial entries (contiguous reads across
// its threads), its 8 thread groups add consecutive eighths of the
// partials (each in order, eight loads in flight), then the eight group
// sums are added in group order.
constexpr int kFinalEntries = 32, kFinalGroups = 8;
// a workgroup's partial of each layer: weights [tap][co][ci], then biases
constexpr int kPart1 = kTaps * kC * 2 + kC, kPart2 = kWPack + kC, kPart3 = kTaps * kC + 1;
__global__ __launch_bounds__(256) void k_grad_final(const float *__restrict__ parts, int nparts,
                                                    const double *__restrict__ tile_loss,
                                                    const double *__restrict__ tile_count, int64_t ntiles,
                                                    double *__restrict__ loss, double *__restrict__ host_loss,
                                                    float *__restrict__ grad)
{
    __shared__ float sg[kFinalGroups][kFinalEntries];
    __shared__ double sl[256], sc[256];
    // N = max(1, sum of the mask) and the loss, the same fixed-order sums
    // in every workgroup; workgroup 0 writes loss[0] = squared errors / N,
    // loss[1] = 1 / N
    {
        double l = 0.0, c = 0.0;
        for (int64_t k = threadIdx.x; k < ntiles; k += 256) {
            l += tile_loss[k];
            c += tile_count[k];
        }
        sl[threadIdx.x] = l;
        sc[threadIdx.x] = c;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (threadIdx.x < h) {
                sl[threadIdx.x] += sl[threadIdx.x + h];
                sc[threadIdx.x] += sc[threadIdx.x + h];
            }
            __syncthreads();
        }
    }
    const double N = sc[0] > 1.0 ? sc[0] : 1.0, inv_n = 1.0 / N;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        loss[0] = sl[0] / N;
        loss[1] = inv_n;
        if (host_loss) *host_loss = sl[0] / N;
    }
    const int el = threadIdx.x % kFinalEntries, grp = threadIdx.x / kFinalEntries;
    const int k = blockIdx.x * kFinalEntries + el;
    const bool live = k < kPart1 + kPart2 + kPart3;
    const int layer = k < kPart1 ? 0 : (k < kPart1 + kPart2 ? 1 : 2);
    const int idx = layer == 0 ? k : (layer == 1 ? k - kPart1 : k - kPart1 - kPart2);
    const int size = layer == 0 ? kPart1 : (layer == 1 ? kPart2 : kPart3);
    const int per = (nparts + kFinalGroups - 1) / kFinalGroups;
    const int p0 = grp * per, p1 = min(nparts, p0 + per);
    float a = 0.f;
    if (live) {
        const float *src = parts + int64_t(layer) * nparts * (kWPack + kC) + idx;
        int p = p0;
        for (; p + 8 <= p1; p += 8) {
            float q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) q[e] = src[int64_t(p + e) * size];
#pragma unroll
            for (int e = 0; e < 8; ++e) a += q[e];
        }
        for (; p < p1; ++p) a += src[int64_t(p) * size];
    }
    sg[grp][el] = a;
    __syncthreads();
    if (grp != 0 || !live) return;
    float sum = sg[0][el];
    for (int q = 1; q < kFinalGroups; ++q) sum += sg[q][el];
    sum = float(double(sum) * inv_n);
    const int cout = layer == 2 ? 1 : 16, cin = layer == 0 ? 2 : 16;
    const int wbase = layer == 0 ? kW1 : (layer == 1 ? kW2 : kW3);
    const int bbase = layer == 0 ? kB1 : (layer == 1 ? kB2 : kB3);
    const int weights = kTaps * cin * cout;
    if (idx < weights) {
        const int t = idx / (cin * cout), co = (idx / cin) % cout, ci = idx % cin;
        grad[wbase + (co * cin + ci) * kTaps + t] = sum;
    } else {
        grad[bbase + idx - weights] = sum;
    }
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       int64_t n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= n) return;
    float gk = g[k];
    float mk = b1 * m[k] + (1.f - b1) * gk;
    float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// p0 = P(grad(u0) / delta) with the masked forward differences of Eq. (3)
__global__ __launch_bounds__(512) void k_warm_p(int64_t nb, int64_t ps, const int32_t *__restrict__ nbr,
                                                const uint8_t *__restrict__ emask, const float *__restrict__ u0,
                                                float inv_delta, float *__restrict__ p0)
{
    const int64_t b = blockIdx.x;
    const int t = threadIdx.x, lx = t & 7, ly = (t >> 3) & 7, lz = t >> 6;
    const int64_t gi = b * kBlockVox + t;
    const int32_t *nb27 = nbr + b * kNbr;
    const uint8_t m = emask[gi];
    const float u = u0[gi];
    float g0 = (m & 2) ? u0[lx < 7 ? gi + 1 : halo_vox(nb27, 8, ly, lz)] - u : 0.f;
    float g1 = (m & 4) ? u0[ly < 7 ? gi + 8 : halo_vox(nb27, lx, 8, lz)] - u : 0.f;
    float g2 = (m & 8) ? u0[lz < 7 ? gi + 64 : halo_vox(nb27, lx, ly, 8)] - u : 0.f;
    g0 *= inv_delta; g1 *= inv_delta; g2 *= inv_delta;
    float nrm = sqrtf((g0 * g0 + g1 * g1) + g2 * g2);
    if (nrm > 1.f) { g0 /= nrm; g1 /= nrm; g2 /= nrm; }
    p0[gi] = g0; p0[gi + ps] = g1; p0[gi + 2 * ps] = g2;
}

// p0 onto the unit ball; u0 = f on Omega, 0 elsewhere
__global__ void k_warm_finish(int64_t n, int64_t ps, const uint8_t *__restrict__ emask, const float *__restrict__ f,
                              float *__restrict__ p0, float *__restrict__ u0)
{
    int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= n) return;
    float a = p0[g], b = p0[g + ps], c = p0[g + 2 * ps];
    float nrm = sqrtf((a * a + b * b) + c * c);
    if (nrm > 1.f) { a /= nrm; b /= nrm; c /= nrm; }
    p0[g] = a; p0[g + ps] = b; p0[g + 2 * ps] = c;
    u0[g] = (emask[g] & 1) ? f[g] : 0.f;
}


static inline unsigned grid1(int64_t n, int bs = 256) { return unsigned((n + bs - 1) / bs); }


// ---------------------------------------------------------------------------
// Fused inference: gather, three layers and the warm-start epilogue of one
// tile per iteration of a workgroup, activations in LDS only.  Every layer
// is an implicit GEMM on v_mfma_f32_16x16x32_bf16 (16 voxels x 16 output
// channels x 32 products of (tap, input channel)); the weights of all three
// layers stay in registers for the whole launch.

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kL1M = 3;       // layer 1: per lane group a (y, z) tap pair, its 3 x taps + 1 zero slot x 2 channels
constexpr int kL2M = 14;      // layer 2: 27 taps x 16 channels, two taps per MFMA
constexpr int kL3M = 2;       // layer 3: rows = the 9 (y, z) tap pairs, K = 3 x taps x 16 channels
// layer 1 runs on the weight pair hi + lo (bfloat16(W) and bfloat16(W -
// bfloat16(W))): its few input channels make the layer's output sensitive to
// the rounding of W1, and the second MFMA per K step costs little
constexpr int kLaneW = (2 * kL1M + kL2M + kL3M) * 64 * 8;

// The workspace of one network call (caller device memory): packed
// weights, activations of n tiles and, for training, their gradients and
// the weight-gradient partial sums.
struct NetWS {
    // training step (dn_net_loss_grad)
    uint16_t *lanew, *lanef, *gates, *x1cf, *h1cf, *h2cf, *d3cf, *d2cf, *d1cf;
    float *d3, *parts;
    double *misc, *tl, *tc;
    int nparts;
};
constexpr int kMaxWgradGroups = 256;
static NetWS carve_net(Bump &b, int64_t n, bool training)
{
    NetWS x{};
    if (!training) {
        const size_t act = size_t(n) * kT * kC;
        // the forward pass keeps its activations in LDS; the size callers
        // allocate by stays what it was
        b.take<uint16_t>(size_t(4) * kWPack);
        for (int k = 0; k < 3; ++k) b.take<uint16_t>(act);
        b.take<float>(size_t(n) * kT);
        return x;
    }
    x.lanew = b.take<uint16_t>(size_t(kLaneW));
    x.lanef = b.take<uint16_t>(size_t(kL2M) * 64 * 8);
    x.gates = b.take<uint16_t>(size_t(n) * 2 * kT);
    x.x1cf = b.take<uint16_t>(size_t(n) * 2 * kPadVox);
    x.h1cf = b.take<uint16_t>(size_t(n) * 16 * kPadVox);
    x.h2cf = b.take<uint16_t>(size_t(n) * 16 * kPadVox);
    x.d3 = b.take<float>(size_t(n) * kBlockVox);
    x.d3cf = b.take<uint16_t>(size_t(n) * kRowVox);
    x.d2cf = b.take<uint16_t>(size_t(n) * 16 * kRowVox);
    x.d1cf = b.take<uint16_t>(size_t(n) * 16 * kRowVox);
    x.nparts = int(n < kMaxWgradGroups ? n : kMaxWgradGroups);
    x.parts = b.take<float>(size_t(3) * x.nparts * (kWPack + kC));
    x.misc = b.take<double>(8);
    x.tl = b.take<double>(size_t(n));
    x.tc = b.take<double>(size_t(n));
    return x;
}

static bool ws_ok(const void *ws) { return ws && (reinterpret_cast<uintptr_t>(ws) & 255) == 0; }

// Lane-ready weights [mfma][lane][8] (bfloat16).  The K slots of lane
// group g = lane / 16, entry j, of MFMA m: layer 1 -> x tap j/2 (3: zero) of
// the (y, z) tap pair 4m + g, channel j%2; layer 2 -> tap 2m + g/2, channel 8(g%2) + j; the output
// column (output channel) is lane % 16.  Layer 3 has one output channel, so
// its rows are taps instead: row n = 3 kz + ky (n < 9) is the (y, z) tap
// pair, and the K slots of MFMA m, group g are x tap kx = 2m + g/2 (kx < 3),
// channel 8(g%2) + j.  The activation operand uses the same map, so the
// products pair up whatever order the hardware sums them in.
__device__ void pack_lane(const float *__restrict__ params, int k, uint16_t *__restrict__ out)
{
    const int j = k & 7, lane = (k >> 3) & 63, m = k >> 9;
    const int g = lane >> 4, n = lane & 15;
    float val = 0.f;
    if (m < kL1M || m >= kL1M + kL2M + kL3M) {
        const int ml = m < kL1M ? m : m - (kL1M + kL2M + kL3M);
        const int pr = 4 * ml + g, e = j >> 1, ci = j & 1;   // (y, z) pair, x slot, channel
        if (pr < 9 && e < 3) val = params[kW1 + (n * 2 + ci) * kTaps + e + 3 * pr];
        if (m >= kL1M) val -= bf2f(f2bf(val));
    } else if (m < kL1M + kL2M) {
        const int t = 2 * (m - kL1M) + (g >> 1), ci = 8 * (g & 1) + j;
        if (t < kTaps) val = params[kW2 + (n * 16 + ci) * kTaps + t];
    } else {
        const int kx = 2 * (m - kL1M - kL2M) + (g >> 1), ci = 8 * (g & 1) + j;
        if (kx < 3 && n < 9) val = params[kW3 + ci * kTaps + 3 * n + kx];
    }
    out[k] = f2bf(val);
}

__global__ void k_pack_lanes(const float *__restrict__ params, uint16_t *__restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kLaneW) pack_lane(params, k, out);
}

// LDS activation: two halves of 8 channels, a 16-byte cell per voxel of the
// tile on a grid whose rows and planes share one zero cell or row with the
// next (11 cells per row, 11 rows per plane, 10 planes: 79 KB for two
// activations, so two workgroups fit a compute unit), kLead zero cells before
// the first.  Every tap inside a plane is a fixed offset; a tap outside the
// planes 0 and 9 is left out.  The 16 lanes of a 16-byte read take consecutive
// cells, four groups of them from the two halves; the halves are 0 modulo 256
// bytes apart: a pass of the read takes cells 0-3 and 12-15 of one half with
// 4-11 of the other (128 apart they met: twice the bank conflicts, 466 against
// 448 us for the warm start of 5777 blocks).
constexpr int kRowS = 11, kPlaneS = 121, kLead = 12;
constexpr int kHalf = 1232 * 16;           // bytes per half: cells up to kLead + 9 * kPlaneS + 111 + 12, and padding
static_assert(kLead + 9 * kPlaneS + 111 + 12 < kHalf / 16 && kHalf % 256 == 0, "activation layout");
constexpr int kCols = 7;                   // columns of 16 plane positions covering 10 rows of 11
constexpr int kPieces = 10 * kCols;        // (column, plane) pieces of 16 positions, columns outermost

__device__ __forceinline__ int cell_of(int x, int y, int z) { return kLead + x + kRowS * y + kPlaneS * z; }
__device__ __forceinline__ int tile_cell(int v) { return cell_of(v % 10, (v / 10) % 10, v / 100); }
__device__ __forceinline__ int act_byte(int cell, int half) { return half * kHalf + cell * 16; }
// plane position (< 112) that is a voxel, not border
__device__ __forceinline__ bool pos_voxel(int pos) { return pos < 10 * kRowS && pos % kRowS < 10; }

__device__ __forceinline__ v8bf as_v8bf(v4u q) { return __builtin_bit_cast(v8bf, q); }

__device__ __forceinline__ v4u lds_row(const uint16_t *h, int byte)
{
    return *reinterpret_cast<const v4u *>(reinterpret_cast<const char *>(h) + byte);
}

// A wave's share of the pieces.
template <int W> __device__ __forceinline__ void piece_range(int wave, int &first, int &last)
{
    first = kPieces * wave / W;
    last = kPieces * (wave + 1) / W;
}

// The next run of a wave's pieces in one column: its planes z0 .. z1.
__device__ __forceinline__ void next_run(int &first, int last, int &c, int &z0, int &z1)
{
    c = first / 10;
    z0 = first % 10;
    z1 = min(9, z0 + (last - first) - 1);
    first += z1 - z0 + 1;
}

// The 16 -> 16 channel layer on the pieces first .. last - 1: store(c, z, acc)
// gets the sums of column c, plane z (this lane's position 16 c + lane % 16,
// its output channels 4g .. 4g + 3).  W2 holds the 14 operands of two taps
// each; lanes of par = 0 take tap 2m, the others tap 2m + 1.
//
// A wave walks down a column: what it reads of a plane serves the plane's own
// sums (their taps of kz = 1: O[0..3]) and those of the next and the previous
// (kz = 0 and 2: E[0..3]; M holds tap 8 and, for the MFMA that straddles two
// planes, the next plane's tap 0), 9 operand reads for 14 MFMAs.  Each sum
// still gets its operands in the order m = 0 .. 13, its three parts as the
// `nxt`, `cur` and `prv` of three steps, which also gives a wave three chains
// of MFMAs in flight; the reads of the next plane are issued as this one's
// operands are used.
template <class Store>
__device__ __forceinline__ void conv_columns(const uint16_t *h, const v8bf (&W2)[kL2M], int lane, int first, int last,
                                             Store store)
{
    const int i = lane & 15, half = (lane >> 4) & 1, par = lane >> 5;
    const v4u zero = {0u, 0u, 0u, 0u};
    const v4f none = {0.f, 0.f, 0.f, 0.f};
    auto mfma = [](v8bf w, v4u a, v4f acc) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, as_v8bf(a), acc, 0, 0, 0);
    };
    while (first < last) {
        int c, z0, z1;
        next_run(first, last, c, z0, z1);
        const int at = act_byte(kLead + 16 * c + i, half);
        // the taps of the two lane halves lie 1, 9 or 97 cells apart
        const int a1 = at + 16 * par, a9 = at + 16 * 9 * par, a97 = at + 16 * 97 * par;
        v4u E[4], O[4], M;
        auto load_e = [&](int k, int z) {
            const int zb = z * (16 * kPlaneS);
            E[k] = k == 0 ? lds_row(h, a1 + zb - 16 * 12) : k == 1 ? lds_row(h, a9 + zb - 16 * 10)
                 : k == 2 ? lds_row(h, a1 + zb) : lds_row(h, a1 + zb + 16 * 10);
        };
        auto load_o = [&](int k, int z) {
            const int zb = z * (16 * kPlaneS);
            O[k] = k == 0 ? lds_row(h, a1 + zb - 16 * 11) : k == 1 ? lds_row(h, a1 + zb - 16)
                 : k == 2 ? lds_row(h, a9 + zb + 16) : lds_row(h, a1 + zb + 16 * 11);
        };
        // (no plane 10: its tap 0 is not used, and not read)
        auto load_m = [&](int z) { M = lds_row(h, (z < 9 ? a97 : at) + z * (16 * kPlaneS) + 16 * 12); };
        v4f prv = none, cur = none, nxt = none;
        if (z0 > 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) load_e(k, z0 - 1);
            load_m(z0 - 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) nxt = mfma(W2[k], E[k], nxt);
        } else {
            M = lds_row(h, at - 16 * 12);            // tap 0 of plane 0; nothing below it
            M = par ? M : zero;
        }
        nxt = mfma(W2[4], M, nxt);
#pragma unroll
        for (int k = 0; k < 4; ++k) { load_e(k, z0); load_o(k, z0); }
        load_m(z0);
        auto step = [&](int z, auto has_prv, auto has_nxt) {
            const int zl = min(z + 1, 9);            // (after plane 9: read again, not used)
            cur = nxt;
            nxt = none;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (decltype(has_nxt)::value) nxt = mfma(W2[k], E[k], nxt);
                cur = mfma(W2[5 + k], O[k], cur);
                if constexpr (decltype(has_prv)::value) prv = mfma(W2[9 + k], E[k], prv);
                load_e(k, zl);
                load_o(k, zl);
            }
            if constexpr (decltype(has_nxt)::value) nxt = mfma(W2[4], M, nxt);
            if constexpr (decltype(has_prv)::value) prv = mfma(W2[13], par ? zero : M, prv);
            load_m(zl);
            if constexpr (decltype(has_prv)::value) store(c, z - 1, prv);
            prv = cur;
        };
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        if (z0 == z1) {
            step(z0, no, no);
        } else {
            step(z0, no, yes);
#pragma unroll 1
            for (int z = z0 + 1; z < z1; ++z) step(z, yes, yes);
            step(z1, yes, no);
        }
        if (z1 < 9) {
#pragma unroll
            for (int k = 0; k < 4; ++k) prv = mfma(W2[9 + k], E[k], prv);
            prv = mfma(W2[13], par ? zero : M, prv);
        }
        store(c, z1, prv);
    }
}

// Products are taken as W x A^T, so a lane holds 4 output channels
// (4g .. 4g+3) of voxel i of the row tile: bias + ReLU, then one 8-byte
// store per lane.
// (bias + ReLU rounded to bfloat16 by the hardware's round-to-nearest-even
// pair conversion, the same rounding as f2bf for these finite values)
typedef float v2f_t __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_act(uint16_t *h, int cell, uint32_t voxel, int g, v4f acc, const float *bias4)
{
    float y[4];
    for (int r = 0; r < 4; ++r) y[r] = fmaxf(acc[r] + bias4[r], 0.f);
    uint2 pk = make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(v2f_t{y[0], y[1]}, v2bf_t)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f_t{y[2], y[3]}, v2bf_t)));
    pk.x &= voxel;      // (all bits of a voxel, none of a border cell, which keeps its zeros)
    pk.y &= voxel;
    *reinterpret_cast<uint2 *>(reinterpret_cast<char *>(h) + act_byte(cell, g >> 1) + 8 * (g & 1)) = pk;
}

// Layer-1 input word of every voxel of the pool: the bfloat16 pair
// (f, log(1 + w) / log(101)), computed once for the three axes; the
// inference kernel reads its tiles from it through the neighbour table.
__global__ void k_voxel_pairs(const float *__restrict__ f, const float *__restrict__ w, int64_t n,
                              uint32_t *__restrict__ pair)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float wv = float(log(1.0 + double(w[i])) / log(101.0));
    pair[i] = uint32_t(f2bf(f[i])) | (uint32_t(f2bf(wv)) << 16);
}

// kDual: out = p0, component perm written on the centre (kept where m_perm =
// 1), for the three axes of every tile; kPrimal (perm 0): out = u0 =
// clamp(f + r, -1, 1) on Omega, 0 elsewhere.  Workgroups loop over (tile,
// axis) items; the layer-1 input of the next one is loaded while the current
// one is computed.  4 waves per workgroup and two workgroups per compute unit
// where items are many; a training step has few tiles, so 8 waves share each.
//
// Bound by what a tile's waves issue: per item 1437 MFMAs (5.9k cycles of a
// compute unit's four matrix cores), LDS reads (8.7k cycles of its one port)
// and some 4800 vector instructions, with two waves per SIMD to overlap them.
// Row tiles in linear order (a tap mask per voxel, an LDS read per MFMA, one
// chain of MFMAs at a time) and a launch per axis: warm start of 5777 blocks
// 588 us, now 448; a training step's forward at 256 tiles 27.2 us, now 20.6 (21.4
// with the loss, which was a launch of 3.9).
//
// kTraining: the forward pass of a training step on n given tiles (f holds the
// float tiles [n][2][1000]); the layer inputs are also written to global
// memory on the zero-padded 12^3 grid for the backward pass (x1cf: the two
// input channels channel-first, [n][2][1728]; h1cf, h2cf channel-last,
// [n][1728][16]), and the residual on the centre goes into the loss at once
// (loss_of_tile), not to memory (out is null).
__device__ __forceinline__ int pad_index(int x, int y, int z) { return (x + 1) + 12 * (y + 1) + 144 * (z + 1); }

// Channel-last copy of an LDS activation (two planes of 8 channels) onto the
// padded grid: dst[1728][16], 32 bytes per padded voxel, zero on the padding.
template <int kThreads>
__device__ __forceinline__ void copy_act_cl(const uint16_t *h, uint16_t *__restrict__ dst, int tid)
{
    for (int p = tid; p < kPadVox; p += kThreads) {
        const int x = p % 12 - 1, y = (p / 12) % 12 - 1, z = p / 144 - 1;
        uint4 lo = make_uint4(0, 0, 0, 0), hi = lo;
        if (x >= 0 && x < 10 && y >= 0 && y < 10 && z >= 0 && z < 10) {
            const int v = cell_of(x, y, z);
            lo = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(h) + act_byte(v, 0));
            hi = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(h) + act_byte(v, 1));
        }
        reinterpret_cast<uint4 *>(dst)[2 * p] = lo;
        reinterpret_cast<uint4 *>(dst)[2 * p + 1] = hi;
    }
}

// Bit ch of dst[v] set when channel ch of the LDS activation is positive at
// tile voxel v (the open ReLUs the backward pass gates with).
template <int kThreads>
__device__ __forceinline__ void gate_bits(const uint16_t *h, uint16_t *__restrict__ dst, int tid)
{
    for (int v = tid; v < kT; v += kThreads) {
        const int cell = tile_cell(v);
        const uint4 lo = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(h) + act_byte(cell, 0));
        const uint4 hi = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(h) + act_byte(cell, 1));
        const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        uint32_t m = 0;
        for (int k = 0; k < 8; ++k) {
            const uint32_t a = w[k] & 0xFFFFu, c = w[k] >> 16;
            if (!(a & 0x8000u) && (a & 0x7FFFu)) m |= 1u << (2 * k);
            if (!(c & 0x8000u) && (c & 0x7FFFu)) m |= 1u << (2 * k + 1);
        }
        dst[v] = uint16_t(m);
    }
}

enum NetUse { kPrimal, kDual, kTraining };
// what a training step reads and writes beside the tiles
struct TrainIO {
    uint16_t *x1cf, *h1cf, *h2cf, *gates;    // for the backward pass
    const float *targets, *mask;             // [n][512]
    int kind;
    float *d3;                               // the loss's gradient, see loss_of_tile
    uint16_t *d3cf;
    double *tile_loss, *tile_count;
};
// Layer-1 input words: the planes -1 .. 10 of a grid with rows of 16 (10 and
// zeros) and 11 rows a plane (10 and one of zeros), kInLead zeros before; the
// (y, z) tap pairs of the four lane groups are then 16 banks apart.
constexpr int kInRow = 16, kInPlane = 176, kInLead = 20, kInWords = 2148;
static_assert(kInLead > kInRow && kInWords % 4 == 0 &&
                  kInWords > kInLead + 10 + 10 * kInRow + 10 * kInPlane + kInRow + kInPlane + 2, "layer-1 input grid");
__device__ __forceinline__ int in_word(int x, int y, int z) { return kInLead + x + kInRow * y + kInPlane * (z + 1); }
// Compact-row index of tile voxel (x, y, z), and its decoding (false for
// padding entries).
__device__ __forceinline__ int row_index(int x, int y, int z) { return (x + 1) + 12 * (10 * z + y); }
__device__ __forceinline__ bool row_voxel(int c, int &x, int &y, int &z)
{
    if (c >= 1200) return false;
    const int xr = c % 12, r = c / 12;
    x = xr - 1; y = r % 10; z = r / 10;
    return xr >= 1 && xr <= 10;
}

// Masked squared loss of a tile, r of this thread's centre voxel given (512
// threads), before the division by N = max(1, sum of the mask), which
// k_grad_final forms and applies: d3 = N dL/dr on the centre (float [n][512])
// and the same in the compact-row layout for the weight gradient of layer 3
// (d3cf [n][1216], bfloat16, zero off the centre), the tile's sum of squared
// errors and of the mask.  (A launch of its own took 3.9 us for 256 tiles.)
__device__ __forceinline__ void loss_of_tile(const float *__restrict__ tiles, const TrainIO &io, int64_t tile, int v,
                                             float r, uint8_t *lds /* 16-byte aligned, 2176 bytes */)
{
    double *sl = reinterpret_cast<double *>(lds), *sc = sl + 8;         // [8] each
    uint16_t *sg = reinterpret_cast<uint16_t *>(lds + 128);             // [1024]
    const int tv = ((v & 7) + 1) + 10 * (((v >> 3) & 7) + 1) + 100 * ((v >> 6) + 1);
    const double m = io.mask[tile * 512 + v];
    const double e = (io.kind == 0 ? double(tiles[tile * 2 * kT + tv]) : 0.0) + double(r) -
                     double(io.targets[tile * 512 + v]);
    double l = m != 0.0 ? e * e : 0.0, c = m;
    const float gv = m != 0.0 ? float(2.0 * e) : 0.f;
    io.d3[tile * 512 + v] = gv;
    for (int k = v; k < kT; k += 512) sg[k] = 0;
    __syncthreads();
    sg[tv] = f2bf(gv);
    for (int o = 32; o > 0; o >>= 1) {
        l += __shfl_xor(l, o, 64);
        c += __shfl_xor(c, o, 64);
    }
    if ((v & 63) == 0) {
        sl[v >> 6] = l;
        sc[v >> 6] = c;
    }
    __syncthreads();
    uint16_t *dst = io.d3cf + tile * kRowVox;
    for (int k = v; k < kRowVox; k += 512) {
        uint16_t val = 0;
        int x, y, z;
        if (row_voxel(k, x, y, z)) val = sg[x + 10 * y + 100 * z];
        dst[k] = val;
    }
    if (v == 0) {
        double s = 0.0, t = 0.0;
        for (int k = 0; k < 8; ++k) {
            s += sl[k];
            t += sc[k];
        }
        io.tile_loss[tile] = s;
        io.tile_count[tile] = t;
    }
}

template <NetUse kUse, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_net_fwd(
    const int32_t *__restrict__ nbr, const uint32_t *__restrict__ pair, const float *__restrict__ f,
    const uint8_t *__restrict__ emask, int64_t nb, const uint16_t *__restrict__ lw, const float *__restrict__ params, int64_t ps,
    float *__restrict__ out, TrainIO io)
{
    constexpr bool kTrain = kUse == kTraining;
    constexpr int kAxes = kUse == kDual ? 3 : 1;
    constexpr int kThreads = 64 * W;
    __shared__ __align__(16) uint16_t h1[kHalf];    // (two halves of kHalf bytes)
    __shared__ __align__(16) uint16_t h2[kHalf];
    // the layer-1 input words lie where layer 2 writes its result later
    uint32_t *x0 = reinterpret_cast<uint32_t *>(h2);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int i = lane & 15, g = lane >> 4;
    const int half = g & 1, par = g >> 1;      // channel half and tap parity of this lane's K slots
    int p_first, p_last;
    piece_range<W>(wave, p_first, p_last);
    const v4u *lw4 = reinterpret_cast<const v4u *>(lw);
    v8bf W1[kL1M], W1l[kL1M], W2[kL2M], W3[kL3M];
    for (int m = 0; m < kL1M; ++m) W1[m] = as_v8bf(lw4[m * 64 + lane]);
    for (int m = 0; m < kL1M; ++m) W1l[m] = as_v8bf(lw4[(kL1M + kL2M + kL3M + m) * 64 + lane]);
    for (int m = 0; m < kL2M; ++m) W2[m] = as_v8bf(lw4[(kL1M + m) * 64 + lane]);
    for (int m = 0; m < kL3M; ++m) W3[m] = as_v8bf(lw4[(kL1M + kL2M + m) * 64 + lane]);
    float bias1[4], bias2[4];
    for (int r = 0; r < 4; ++r) {
        bias1[r] = params[kB1 + 4 * g + r];
        bias2[r] = params[kB2 + 4 * g + r];
    }
    const float bias3 = params[kB3];
    // the border cells of h1 that no layer writes: before the first plane and
    // the rest of the row below each plane (its first two cells come with the
    // last column)
    auto clear_border = [&]() {
        for (int k = tid; k < 2 * (kLead + 10 * 12); k += kThreads) {
            const int e = k >> 1;
            const int cell = e < kLead ? e : kLead + ((e - kLead) / 12) * kPlaneS + 112 + (e - kLead) % 12;
            if (e < kLead || (e - kLead) % 12 < 9 || (e - kLead) / 12 == 9)
                *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(h1) + act_byte(cell, k & 1)) = make_uint4(0, 0, 0, 0);
        }
    };
    clear_border();
    // (or every loop below waits for these loads, and so for the prefetch)
    __builtin_amdgcn_s_waitcnt(0);

    // the layer-1 input of a tile and axis: the words of its voxels, read from
    // the pool's pair words through the neighbour table (voxels of unallocated
    // blocks give 0), the next one's while this one is computed; all loads of a
    // thread are issued together.  where: x + 7, y + 7, z + 7 in three bytes
    // (so that bits 3.. are the block, bits 0-2 the voxel in it), 0 past the
    // tile's voxels, where some voxel is read and not used
    constexpr int kGet = (kT + kThreads - 1) / kThreads;
    uint32_t nxt[kGet], where[kGet];
    int to[kGet];
    for (int e = 0; e < kGet; ++e) {
        const int k = tid + kThreads * e, x = k % 10, y = (k / 10) % 10, z = k / 100;
        where[e] = k < kT ? uint32_t((x + 7) | ((y + 7) << 8) | ((z + 7) << 16)) : 0u;
        to[e] = in_word(x, y, z);
    }
    auto clear_input = [&]() {
        for (int k = tid; k < kInWords / 4; k += kThreads) reinterpret_cast<uint4 *>(x0)[k] = make_uint4(0, 0, 0, 0);
    };
    clear_input();
    __syncthreads();
    // (in two parts: the table entries, or the given tile's f and weight
    // channel, [n][2][1000], then the pair words)
    uint32_t more[kGet];
    auto fetch_table = [&](int64_t item) {
        const int64_t bb = item / kAxes;
        const int perm = int(item - kAxes * bb);
        for (int e = 0; e < kGet; ++e) {
            if constexpr (kTrain) {
                const int k = min(tid + kThreads * e, kT - 1);
                nxt[e] = __float_as_uint(f[bb * 2 * kT + k]);
                more[e] = __float_as_uint(f[bb * 2 * kT + kT + k]);
            } else {
                // weights of the tile's x, y, z in the neighbour slot; axis 1
                // or 2 in the place of axis 0 and the reverse
                const uint32_t ws = perm == 0 ? 0x090301u : (perm == 1 ? 0x090103u : 0x010309u);
                const uint32_t slot = __builtin_amdgcn_udot4((where[e] >> 3) & 0x030303u, ws, 0u, false);
                more[e] = uint32_t(nbr[bb * kNbr + (where[e] ? slot : 13u)]);
            }
        }
    };
    auto fetch_words = [&](int64_t item) {
        if constexpr (kTrain) return;
        const int perm = int(item % kAxes);
        const uint32_t wo = perm == 0 ? 0x400801u : (perm == 1 ? 0x400108u : 0x010840u);
        for (int e = 0; e < kGet; ++e) {
            const uint32_t o = __builtin_amdgcn_udot4(where[e] & 0x070707u, wo, 0u, false);
            nxt[e] = pair[int64_t(int32_t(more[e]) < 0 ? 0u : more[e]) * kBlockVox + o];
        }
    };
    auto fetched = [&](int e) {
        if constexpr (kTrain)
            return uint32_t(f2bf(__uint_as_float(nxt[e]))) | (uint32_t(f2bf(__uint_as_float(more[e]))) << 16);
        else return int32_t(more[e]) >= 0 ? nxt[e] : 0u;
    };
    const int64_t items = nb * kAxes;
    if (blockIdx.x < items) {
        fetch_table(blockIdx.x);
        fetch_words(blockIdx.x);
    }

    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const int64_t b = item / kAxes;
        const int perm = int(item - kAxes * b);
        for (int e = 0; e < kGet; ++e)
            if (where[e]) x0[to[e]] = fetched(e);
        __syncthreads();
        const int64_t next = item + gridDim.x;
        if (next < items) fetch_table(next);
        if constexpr (kTrain)
            for (int e = tid; e < 2 * kPadVox; e += kThreads) {
                const int ch = e / kPadVox, p = e - ch * kPadVox;
                const int x = p % 12 - 1, y = (p / 12) % 12 - 1, z = p / 144 - 1;
                const bool in = x >= 0 && x < 10 && y >= 0 && y < 10 && z >= 0 && z < 10;
                io.x1cf[b * (2 * kPadVox) + e] = in ? uint16_t(x0[in_word(x, y, z)] >> (16 * ch)) : uint16_t(0);
            }

        // layer 1: 2 -> 16, ReLU.  Lane group g of MFMA m takes the (y, z)
        // tap pair 4m + g: the input words of its x taps -1, 0, +1 (and +2,
        // whose weights are zero) are 4 consecutive words, zero wherever the
        // tap leaves the tile.  Two planes at a time: two chains of MFMAs.
        for (int first = p_first; first < p_last;) {
            int c, z0, z1;
            next_run(first, p_last, c, z0, z1);
            const int pos = 16 * c + i;
            const uint32_t voxel = pos_voxel(pos) ? ~0u : 0u;
            int at[kL1M], step[kL1M];          // words of plane z0, and from plane to plane
            for (int m = 0; m < kL1M; ++m) {
                const int pr = 4 * m + g;
                step[m] = pr < 9 ? kInPlane : 0;   // (past the 9th pair: zeros, and zero weights)
                at[m] = pr < 9 ? in_word(pos % kRowS - 1, pos / kRowS + pr % 3 - 1, z0 + pr / 3 - 1) : 0;
            }
#pragma unroll 1
            for (int z = z0; z <= z1; z += 2) {
                v4f acc[2];
                const int odd = z < z1 ? 1 : 0;    // (a last single plane is computed twice)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    acc[k] = v4f{0.f, 0.f, 0.f, 0.f};
                    for (int m = 0; m < kL1M; ++m) {
                        const int a = at[m] + k * odd * step[m];
                        const v4u q = {x0[a], x0[a + 1], x0[a + 2], x0[a + 3]};
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W1[m], as_v8bf(q), acc[k], 0, 0, 0);
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W1l[m], as_v8bf(q), acc[k], 0, 0, 0);
                    }
                }
                for (int m = 0; m < kL1M; ++m) at[m] += 2 * step[m];
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    store_act(h1, kLead + pos + kPlaneS * (z + k * odd), voxel, g, acc[k], bias1);
            }
        }
        __syncthreads();
        if constexpr (kTrain) {
            // layer inputs for the backward pass (read-only use of h1 until
            // the barrier after layer 2), and which ReLUs are open
            copy_act_cl<kThreads>(h1, io.h1cf + b * (16 * kPadVox), tid);
            gate_bits<kThreads>(h1, io.gates + b * (2 * kT), tid);
        }

        if (next < items) fetch_words(next);

        // layer 2: 16 -> 16, ReLU
        conv_columns(h1, W2, lane, p_first, p_last, [&](int c, int z, v4f acc) {
            const int pos = 16 * c + i;
            store_act(h2, kLead + pos + kPlaneS * z, pos_voxel(pos) ? ~0u : 0u, g, acc, bias2);
        });
        __syncthreads();
        if constexpr (kTrain) {
            copy_act_cl<kThreads>(h2, io.h2cf + b * (16 * kPadVox), tid);
            gate_bits<kThreads>(h2, io.gates + b * (2 * kT) + kT, tid);
        }

        // the centre voxels this thread will write, and whether it does
        constexpr int kOwn = kBlockVox / kThreads;
        int64_t own[kOwn];
        float own_f[kOwn];
        bool on[kOwn];
        if constexpr (!kTrain)
#pragma unroll
            for (int e = 0; e < kOwn; ++e) {
                const int c = tid + kThreads * e;
                int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
                if (perm == 1) { const int sw = x; x = y; y = sw; }
                if (perm == 2) { const int sw = x; x = z; z = sw; }
                own[e] = b * kBlockVox + x + 8 * y + 64 * z;
                on[e] = (emask[own[e]] >> (kUse == kDual ? perm + 1 : 0)) & 1;
                own_f[e] = kUse == kPrimal ? f[own[e]] : 0.f;
            }

        // layer 3: 16 -> 1 on the centre 8^3, as partial sums over the x taps.
        // P[n][u] = sum over kx, ci of W3[ci][3n + kx] h2[u + kx - 1][ci] for
        // the 9 (y, z) tap pairs n and the 800 voxels u with x in 1..8 (rows
        // r = 10 z + y, 8 voxels each), one 16-voxel tile (two rows) per pair
        // of MFMAs; P goes to h1, which layer 2 has finished reading.
        // (the lane groups' P rows are 32 banks apart)
        constexpr int kPRow = 808, kGroup = W == 4 ? 4 : 2;
        float *P = reinterpret_cast<float *>(h1);
        const int u0 = act_byte(cell_of((i & 7) + par, i >> 3, 0), half);        // kx = par
        const int u2 = act_byte(cell_of((i & 7) + 2, i >> 3, 0), half);          // kx = 2
        for (int mt0 = 50 * wave / W; mt0 < 50 * (wave + 1) / W; mt0 += kGroup) {
            v4f sum[kGroup];
#pragma unroll
            for (int k = 0; k < kGroup; ++k) {
                const int mt = min(mt0 + k, 50 * (wave + 1) / W - 1);
                const int row2 = 16 * (2 * kRowS * (mt % 5) + kPlaneS * (mt / 5));
                const v4u q0 = lds_row(h2, u0 + row2);
                const v4u q1 = lds_row(h2, par ? 0 : u2 + row2);   // (cell 0 is zero: layer 2 writes none below kLead)
                v4f acc = {0.f, 0.f, 0.f, 0.f};
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W3[0], as_v8bf(q0), acc, 0, 0, 0);
                sum[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W3[1], as_v8bf(q1), acc, 0, 0, 0);
            }
            // lane: rows (tap pairs) 4g .. 4g+3 of column i
            auto p_at = [&](int k) { return 4 * g * kPRow + i + 16 * min(mt0 + k, 50 * (wave + 1) / W - 1); };
            if (g < 3)
#pragma unroll
                for (int k = 0; k < kGroup; ++k) P[p_at(k)] = sum[k][0];
            if (g < 2)
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
                    for (int e = 1; e < 4; ++e) P[p_at(k) + e * kPRow] = sum[k][e];
        }
        __syncthreads();

        // the 9 pair sums of each centre voxel, then the epilogue (and layer
        // 1's zeros again where h2 was)
        clear_input();
#pragma unroll
        for (int e = 0; e < kOwn; ++e) {
            const int c = tid + kThreads * e, cx = c & 7, cy = (c >> 3) & 7, cz = c >> 6;
            float acc = 0.f;
            for (int n = 0; n < 9; ++n) {
                const int row = (cz + n / 3) * 10 + (cy + n % 3);   // (z + kz - 1 + 1, y + ky - 1 + 1)
                acc += P[n * kPRow + 8 * row + cx];
            }
            const float rv = acc + bias3;
            if constexpr (kTrain) {
                static_assert(!kTrain || kOwn == 1, "one centre voxel per thread");
                loss_of_tile(f, io, b, tid, rv, reinterpret_cast<uint8_t *>(h1) + 4 * 9 * kPRow);
            } else {
                float y1 = rv;
                if constexpr (kUse == kPrimal) {
                    y1 = own_f[e] + rv;
                    y1 = y1 < -1.f ? -1.f : (y1 > 1.f ? 1.f : y1);
                }
                out[perm * ps + own[e]] = on[e] ? y1 : 0.f;
            }
        }
        __syncthreads();
        clear_border();      // P lay there
    }
}

// ---------------------------------------------------------------------------
// Training step kernels (after k_net_fwd<kTraining>).

// Lane-ready weights of a training step: the forward's (as k_pack_lanes)
// and those of the input gradient of layer 2, d1 = conv(d2, W') with
// W'[ci][co][t] = W2[co][ci][26 - t] (the layer-2 map of k_pack_lanes).
__global__ void k_pack_train(const float *__restrict__ params, uint16_t *__restrict__ lw, uint16_t *__restrict__ out)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kLaneW) {
        pack_lane(params, k, lw);
        return;
    }
    k -= kLaneW;
    if (k >= kL2M * 64 * 8) return;
    const int j = k & 7, lane = (k >> 3) & 63, m = k >> 9;
    const int g = lane >> 4, n = lane & 15;
    const int t = 2 * m + (g >> 1), c = 8 * (g & 1) + j;
    float val = 0.f;
    if (t < kTaps) val = params[kW2 + (c * 16 + n) * kTaps + (kTaps - 1 - t)];
    out[k] = f2bf(val);
}

__device__ __forceinline__ bool bf_pos(uint16_t h) { return !(h & 0x8000u) && (h & 0x7FFFu) != 0; }

// Backward through layers 3 and 2 of one tile per iteration of a
// workgroup, on MFMA: d2 = (W3 applied backwards to d3) gated by [h2 > 0],
// as one 16 (channels) x 16 (voxels) x 32 (taps) product per row tile (the
// lane's 8 taps read d3 shifted back by the tap), then d1 = conv(d2, W')
// gated by [h1 > 0] as layer 2 of k_net_fwd (conv_columns, flipped weights W'
// in registers, d2 in LDS; 256 tiles 23.5 us with its row tiles and 4 waves,
// now 15.4).  d2 and d1 go to global memory on the compact
// rows, channel-last ([n][1216][16] bfloat16, 32 bytes per entry).
constexpr int kD3Words = 1472;     // the planes -1 .. 10 of the activations' grid
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_net_bwd(
    const float *__restrict__ d3, const uint16_t *__restrict__ gates, int64_t n, const uint16_t *__restrict__ lwf,
    const float *__restrict__ params, uint16_t *__restrict__ d2cf, uint16_t *__restrict__ d1cf)
{
    constexpr int kThreads = 64 * W;
    __shared__ __align__(16) uint16_t dd[kHalf];     // (two halves of kHalf bytes)
    __shared__ uint16_t s3[kD3Words];        // d3 (bfloat16) on the planes -1 .. 10 of the grid, zero off the centre
    __shared__ __align__(16) uint16_t sg[2 * kT];    // open ReLUs of layers 1 and 2 (bit = channel)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    for (int k = tid; k < 2 * kHalf / 16; k += kThreads) reinterpret_cast<uint4 *>(dd)[k] = make_uint4(0, 0, 0, 0);
    for (int k = tid; k < kD3Words; k += kThreads) s3[k] = 0;
    const int i = lane & 15, g = lane >> 4;
    int p_first, p_last;
    piece_range<W>(wave, p_first, p_last);
    const v4u *lw4 = reinterpret_cast<const v4u *>(lwf);
    v8bf W2[kL2M];
    for (int m = 0; m < kL2M; ++m) W2[m] = as_v8bf(lw4[m * 64 + lane]);
    // W3 as the first operand: row ci = i, K slots = taps 8g .. 8g + 7
    v8bf W3r;
    {
        uint16_t w[8];
        for (int j = 0; j < 8; ++j) {
            const int t = 8 * g + j;
            w[j] = t < kTaps ? f2bf(params[kW3 + i * kTaps + t]) : uint16_t(0);
        }
        W3r = as_v8bf(*reinterpret_cast<const v4u *>(&w[0]));
    }
    // d3 of a voxel shifted back by the lane's taps (one past the 27th reads
    // word 0, a border word)
    int toff[8];
    for (int j = 0; j < 8; ++j) {
        const int t = 8 * g + j;
        toff[j] = t < kTaps ? (t % 3 - 1) + kRowS * ((t / 3) % 3 - 1) + kPlaneS * (t / 9 - 1) : 0;
    }
    // the next tile's d3 (2 centre values per thread) and gate words (one
    // 16-byte chunk per thread) are loaded while the current one is computed
    static_assert(kThreads >= 256, "the loads of a tile take 256 threads");
    float2 nd3 = make_float2(0.f, 0.f);
    uint4 ngt = make_uint4(0, 0, 0, 0);
    auto fetch = [&](int64_t bb) {
        if (tid < 256) nd3 = reinterpret_cast<const float2 *>(d3 + bb * 512)[tid];
        if (tid < 2 * kT / 8) ngt = reinterpret_cast<const uint4 *>(gates + bb * (2 * kT))[tid];
    };
    __builtin_amdgcn_s_waitcnt(0);
    if (blockIdx.x < n) fetch(blockIdx.x);
    __syncthreads();
    for (int64_t b = blockIdx.x; b < n; b += gridDim.x) {
        if (tid < 256) {
            const int c0 = 2 * tid;       // centre voxels c0, c0 + 1 (same x row)
            const int at = cell_of((c0 & 7) + 1, ((c0 >> 3) & 7) + 1, (c0 >> 6) + 2);
            s3[at] = f2bf(nd3.x);
            s3[at + 1] = f2bf(nd3.y);
            if (tid < 2 * kT / 8) reinterpret_cast<uint4 *>(sg)[tid] = ngt;
        }
        const int64_t bn = b + gridDim.x;
        if (bn < n) fetch(bn);
        __syncthreads();
        uint16_t *o2 = d2cf + b * (16 * kRowVox);
        uint16_t *o1 = d1cf + b * (16 * kRowVox);
        // d2 = W3^T d3 (shifted back), gated by [h2 > 0]
        for (int id = p_first; id < p_last; ++id) {
            const int pos = 16 * (id / 10) + i, z = id % 10, cell = kLead + pos + kPlaneS * z;
            const bool voxel = pos_voxel(pos);
            uint16_t q[8];
            for (int j = 0; j < 8; ++j) q[j] = s3[8 * g + j < kTaps ? cell + kPlaneS - toff[j] : 0];
            v4f acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W3r, as_v8bf(*reinterpret_cast<const v4u *>(&q[0])), acc,
                                                         0, 0, 0);
            if (voxel) {
                // lane: voxel (x, y, z), channels 4g .. 4g + 3
                const int x = pos % kRowS, y = pos / kRowS;
                const uint32_t open2 = sg[kT + x + 10 * y + 100 * z];
                uint16_t r4[4];
                for (int r = 0; r < 4; ++r) r4[r] = ((open2 >> (4 * g + r)) & 1u) ? f2bf(acc[r]) : uint16_t(0);
                const uint2 pk = *reinterpret_cast<const uint2 *>(&r4[0]);
                *reinterpret_cast<uint2 *>(reinterpret_cast<char *>(dd) + act_byte(cell, g >> 1) + 8 * (g & 1)) = pk;
                reinterpret_cast<uint2 *>(o2 + row_index(x, y, z) * 16)[g] = pk;
            }
        }
        for (int c = tid; c < kRowVox; c += kThreads) {
            int x, y, z;
            if (!row_voxel(c, x, y, z)) {
                reinterpret_cast<uint4 *>(o2)[2 * c] = make_uint4(0, 0, 0, 0);
                reinterpret_cast<uint4 *>(o2)[2 * c + 1] = make_uint4(0, 0, 0, 0);
                reinterpret_cast<uint4 *>(o1)[2 * c] = make_uint4(0, 0, 0, 0);
                reinterpret_cast<uint4 *>(o1)[2 * c + 1] = make_uint4(0, 0, 0, 0);
            }
        }
        __syncthreads();
        // d1 = conv(d2, W') gated by [h1 > 0]
        conv_columns(dd, W2, lane, p_first, p_last, [&](int c, int z, v4f acc) {
            const int pos = 16 * c + i;
            if (!pos_voxel(pos)) return;
            const int x = pos % kRowS, y = pos / kRowS;
            const uint32_t open1 = sg[x + 10 * y + 100 * z];
            uint16_t q[4];
            for (int r = 0; r < 4; ++r) q[r] = ((open1 >> (4 * g + r)) & 1u) ? f2bf(acc[r]) : uint16_t(0);
            reinterpret_cast<uint2 *>(o1 + row_index(x, y, z) * 16)[g] = *reinterpret_cast<const uint2 *>(&q[0]);
        });
        __syncthreads();
    }
}

// LDS rows: X channel rows of 1928 entries (8 + 1728 + zero margin; 964
// words, 4 modulo 64 banks, so the 16 lanes of a 16-byte read start on 16
// distinct groups of 4 banks), dY rows of 1224 entries (612 words, 36 modulo
// 64, likewise).
constexpr int kXRow = 1928;
constexpr int kDRow = 1224;

// Eight channel values (one 16-byte chunk of a channel-last entry) into
// eight channel rows of an LDS tile: row0[j * stride + pos] = channel j.
__device__ __forceinline__ void scatter8(uint16_t *row0, int stride, int pos, uint4 v)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        row0[(2 * j) * stride + pos] = uint16_t(w[j] & 0xFFFFu);
        row0[(2 * j + 1) * stride + pos] = uint16_t(w[j] >> 16);
    }
}

// The three x shifts of a run of 8 channel-row entries starting at p
// (p 8-byte aligned): bm = p[-1 .. 6], b0 = p[0 .. 7], bp = p[1 .. 8], from
// four aligned 8-byte reads of p[-4 .. 11] and 16-bit funnel shifts (an
// LDS read at a 2-byte offset is split by the hardware and costs several
// times an aligned one).
__device__ __forceinline__ void x_shifts(const uint16_t *p, v4u &bm, v4u &b0, v4u &bp)
{
    const uint2 *q = reinterpret_cast<const uint2 *>(p - 4);
    const uint2 l0 = q[0], l1 = q[1], l2 = q[2], l3 = q[3];
    const uint32_t s1 = __builtin_amdgcn_alignbit(l1.y, l1.x, 16), s2 = __builtin_amdgcn_alignbit(l2.x, l1.y, 16),
                   s3 = __builtin_amdgcn_alignbit(l2.y, l2.x, 16);
    bm = v4u{__builtin_amdgcn_alignbit(l1.x, l0.y, 16), s1, s2, s3};
    b0 = v4u{l1.x, l1.y, l2.x, l2.y};
    bp = v4u{s1, s2, s3, __builtin_amdgcn_alignbit(l3.x, l2.y, 16)};
}

// The shift s in {-1, 0, +1} of that run (p[s .. s + 7]), s per lane.
__device__ __forceinline__ v4u x_shift(const uint16_t *p, int s)
{
    v4u bm, b0, bp;
    x_shifts(p, bm, b0, bp);
    return s < 0 ? bm : (s > 0 ? bp : b0);
}

// Eight entries p[0 .. 7] at an 8-byte aligned p, as two aligned reads.
__device__ __forceinline__ v4u lds8_a8(const uint16_t *p)
{
    const uint2 *q = reinterpret_cast<const uint2 *>(p);
    const uint2 l1 = q[0], l2 = q[1];
    return v4u{l1.x, l1.y, l2.x, l2.y};
}

// Weight and bias gradient of layer 3 (one output channel):
//   dW3[ci][t] = sum over tile voxels v of h2[ci][v] d3[v - off(t)],
// as (taps, 16 rows) x (input channels, 16 columns) x (32 voxels) MFMAs:
// the rows read d3, kept on the padded grid, shifted back by their own tap
// (x shifts per lane from x_shift), the columns read h2 unshifted.  Two MFMAs per
// 32 voxels instead of 27 with one used row.  Partials in the
// [tap][co][ci] layout (co = 0), bias db3 = sum of d3.
constexpr int kD3Row = 2080;   // LDS entries of d3: 168 zero margin + 1728 + margin
constexpr int kWgrad3Lds = 2 * 16 * kXRow + 2 * kD3Row + 4 * 512;
static_assert(4 * 8 * 32 * 16 <= 2 * 16 * kXRow, "the waves' sums lie where the tiles did");
__device__ __forceinline__ void wgrad3_body(const uint16_t *__restrict__ X, const uint16_t *__restrict__ d3cf,
                                            int64_t n, float *__restrict__ partials, int wg, int ngroups,
                                            uint8_t *lds)
{
    uint16_t *sx = reinterpret_cast<uint16_t *>(lds);                  // [16][kXRow]
    uint16_t *sd = sx + 16 * kXRow;                                     // [kD3Row]
    float *sb = reinterpret_cast<float *>(sd + kD3Row);                 // [512]
    float(*red)[32][16] = reinterpret_cast<float(*)[32][16]>(sx);       // [8][32][16], after the last tile
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i = lane & 15, g = lane >> 4;
    for (int k = tid; k < 16 * kXRow / 8; k += 512) reinterpret_cast<uint4 *>(sx)[k] = make_uint4(0, 0, 0, 0);
    for (int k = tid; k < kD3Row / 8; k += 512) reinterpret_cast<uint4 *>(sd)[k] = make_uint4(0, 0, 0, 0);
    v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
    float bsum = 0.f;
    __syncthreads();
    constexpr int kXc = kPadVox / 8;
    constexpr int kPer = (16 * kXc + 511) / 512;
    constexpr int kDPer = (kRowVox + 511) / 512;
    uint4 nxt[kPer];
    uint16_t nd[kDPer];
    auto fetch = [&](int64_t tl) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 512 * e;
            if (k < 16 * kXc) nxt[e] = reinterpret_cast<const uint4 *>(X + tl * 16 * kPadVox)[k];
        }
#pragma unroll
        for (int e = 0; e < kDPer; ++e) {
            const int c = tid + 512 * e;
            nd[e] = c < kRowVox ? d3cf[tl * kRowVox + c] : uint16_t(0);
        }
    };
    if (wg < n) fetch(wg);
    for (int64_t tile = wg; tile < n; tile += ngroups) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 512 * e;
            if (k < 16 * kXc) scatter8(sx + (k & 1) * 8 * kXRow + 8, kXRow, k >> 1, nxt[e]);
        }
        // d3 from its compact rows onto the padded grid (zero elsewhere)
#pragma unroll
        for (int e = 0; e < kDPer; ++e) {
            const int c = tid + 512 * e;
            int x, y, z;
            if (c < kRowVox && row_voxel(c, x, y, z)) {
                sd[168 + pad_index(x, y, z)] = nd[e];
                bsum += bf2f(nd[e]);
            }
        }
        __syncthreads();
        if (tile + ngroups < n) fetch(tile + ngroups);
        // wave w takes the 32-voxel chunks w, w + 8, ...
        for (int c0 = 32 * wave; c0 < kRowVox; c0 += 256) {
            const int c = c0 + 8 * g;
            const int plane = c / 120, within = c - 120 * plane;
            const int pc = within + 12 + 144 * (plane + 1);          // padded index of entry c
            const v8bf b = as_v8bf(lds8_a8(sx + i * kXRow + 8 + pc));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = 16 * h + i;
                v4u q = {0u, 0u, 0u, 0u};
                if (t < kTaps)
                    q = x_shift(sd + 168 + pc - 12 * ((t / 3) % 3 - 1) - 144 * (t / 9 - 1), 1 - t % 3);
                acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_v8bf(q), b, acc[h], 0, 0, 0);
            }
        }
        __syncthreads();
        for (int c = tid; c < kRowVox; c += 512) {      // clear d3's entries for the next tile
            int x, y, z;
            if (row_voxel(c, x, y, z)) sd[168 + pad_index(x, y, z)] = 0;
        }
    }
    // the eight waves' sums of each (tap, ci), then one partial per workgroup
    for (int h = 0; h < 2; ++h)
        for (int r = 0; r < 4; ++r) red[wave][16 * h + 4 * g + r][i] = acc[h][r];
    sb[tid] = bsum;
    __syncthreads();
    float *out = partials + int64_t(wg) * kPart3;
    for (int e = tid; e < kTaps * kC; e += 512) {
        float v = 0.f;
        for (int w = 0; w < 8; ++w) v += red[w][e / kC][e % kC];
        out[e] = v;
    }
    if (wave == 7) {
        float v = 0.f;
        for (int w = 0; w < 8; ++w) v += sb[64 * w + lane];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) out[kTaps * kC] = v;
    }
}

// Weight and bias gradient of layer 1 (two input channels):
//   dW1[co][ci][t] = sum over v of d1[co][v] x[ci][v + off(t)],
// as (output channels) x (54 (ci, t) columns in four MFMAs) x (32 voxels):
// each column reads the input channel shifted by its own tap (the y and z
// shifts keep the reads 8-byte aligned, x shifts per lane from x_shift).
constexpr int kWgrad1Lds = 2 * 2 * kXRow + 2 * 16 * kDRow + 4 * 512;
static_assert(4 * 8 * 16 * 64 <= 2 * 16 * kDRow, "the waves' sums lie where the tiles did");
__device__ __forceinline__ void wgrad1_body(const uint16_t *__restrict__ X, const uint16_t *__restrict__ dY,
                                            int64_t n, float *__restrict__ partials, int wg, int ngroups,
                                            uint8_t *lds)
{
    uint16_t *sx = reinterpret_cast<uint16_t *>(lds);                  // [2][kXRow]
    uint16_t *sd = sx + 2 * kXRow;                                      // [16][kDRow]
    float *sb = reinterpret_cast<float *>(sd + 16 * kDRow);             // [512]
    float(*red)[16][64] = reinterpret_cast<float(*)[16][64]>(sd);       // [8][16][64], after the last tile
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i = lane & 15, g = lane >> 4;
    for (int k = tid; k < 2 * kXRow / 8; k += 512) reinterpret_cast<uint4 *>(sx)[k] = make_uint4(0, 0, 0, 0);
    for (int k = tid; k < 16 * kDRow / 8; k += 512) reinterpret_cast<uint4 *>(sd)[k] = make_uint4(0, 0, 0, 0);
    v4f acc[4];
    for (int q = 0; q < 4; ++q) acc[q] = v4f{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    int coff[4], ckx[4];             // column 16 q + i: channel row + (y, z) tap shift, and its x shift
    bool cuse[4];
    for (int q = 0; q < 4; ++q) {
        const int col = 16 * q + i, ci = col / kTaps, t = col % kTaps;
        cuse[q] = col < 2 * kTaps;
        coff[q] = cuse[q] ? ci * kXRow + 8 + 12 * ((t / 3) % 3 - 1) + 144 * (t / 9 - 1) : 8;
        ckx[q] = t % 3 - 1;
    }
    __syncthreads();
    constexpr int kXc = kPadVox / 8, kDc = kRowVox / 8;
    constexpr int kChunks = 2 * kXc + 16 * kDc;
    constexpr int kPer = (kChunks + 511) / 512;
    uint4 nxt[kPer];
    auto fetch = [&](int64_t tl) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 512 * e;
            if (k < 2 * kXc) nxt[e] = reinterpret_cast<const uint4 *>(X + tl * 2 * kPadVox)[k];
            else if (k < kChunks) nxt[e] = reinterpret_cast<const uint4 *>(dY + tl * 16 * kRowVox)[k - 2 * kXc];
        }
    };
    if (wg < n) fetch(wg);
    for (int64_t tile = wg; tile < n; tile += ngroups) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 512 * e;
            if (k < 2 * kXc) {
                const int ch = k / kXc, r = k - ch * kXc;
                reinterpret_cast<uint4 *>(sx + ch * kXRow + 8)[r] = nxt[e];
            } else if (k < kChunks) {
                const int kk = k - 2 * kXc;
                scatter8(sd + (kk & 1) * 8 * kDRow, kDRow, kk >> 1, nxt[e]);
            }
        }
        __syncthreads();
        if (tile + ngroups < n) fetch(tile + ngroups);
        for (int c = tid >> 4; c < kRowVox; c += 32) bsum += bf2f(sd[(tid & 15) * kDRow + c]);
        for (int c0 = 32 * wave; c0 < kRowVox; c0 += 256) {
            const int c = c0 + 8 * g;
            const v8bf a = as_v8bf(*reinterpret_cast<const v4u *>(sd + i * kDRow + c));
            const int plane = c / 120, within = c - 120 * plane;
            const int pc = within + 12 + 144 * (plane + 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4u bq = {0u, 0u, 0u, 0u};
                if (cuse[q]) bq = x_shift(sx + coff[q] + pc, ckx[q]);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_v8bf(bq), acc[q], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // D[co][col]: lane holds column 16 q + i, rows co = 4g .. 4g + 3; the
    // eight waves' sums, then one partial per workgroup in [tap][co][ci]
    for (int q = 0; q < 4; ++q)
        for (int r = 0; r < 4; ++r) red[wave][4 * g + r][16 * q + i] = acc[q][r];
    sb[tid] = bsum;
    __syncthreads();
    float *out = partials + int64_t(wg) * kPart1;
    for (int e = tid; e < kTaps * kC * 2; e += 512) {
        const int col = (e & 1) * kTaps + e / (2 * kC), co = (e >> 1) % kC;
        float v = 0.f;
        for (int w = 0; w < 8; ++w) v += red[w][co][col];
        out[e] = v;
    }
    if (tid < kC) {
        float v = 0.f;
        for (int k = 0; k < 32; ++k) v += sb[k * 16 + tid];
        out[kTaps * kC * 2 + tid] = v;
    }
}

// The layer-1 and layer-3 weight gradients in one launch: workgroups
// [0, g1) take layer 1, the rest layer 3.  Each is latency-bound with one
// workgroup per compute unit; sharing one LDS allocation (the larger of the
// two) lets a unit hold one of each, so the two run side by side.  8 waves
// each: with 4, and partials in layer 2's shape, 17.8 us for 256 tiles, now
// 11.9.
constexpr int kWgrad13Lds = kWgrad1Lds > kWgrad3Lds ? kWgrad1Lds : kWgrad3Lds;
__global__ __launch_bounds__(512) void k_wgrad13(const uint16_t *__restrict__ X1, const uint16_t *__restrict__ d1,
                                                 const uint16_t *__restrict__ X3, const uint16_t *__restrict__ d3,
                                                 int64_t n, float *__restrict__ parts1, float *__restrict__ parts3,
                                                 int g1)
{
    __shared__ __align__(16) uint8_t lds[kWgrad13Lds];
    const int wg = int(blockIdx.x);
    if (wg < g1) wgrad1_body(X1, d1, n, parts1, wg, g1, lds);
    else wgrad3_body(X3, d3, n, parts3, wg - g1, int(gridDim.x) - g1, lds);
}

// LDS rows of the layer-2 weight gradient.  Its X reads are 8-byte reads
// by 16 channel rows x 4 lane groups whose runs are 64 entries (32 banks)
// apart: a row stride of 2 banks modulo 64 (1924 entries) puts the 32 lanes
// of each half-wave pass on 64 distinct banks.  dY rows of 1288 entries (4
// banks modulo 64) keep its 16-byte reads conflict-free, and hold the 1280
// entries the K steps cover (the compact rows' 1216 and zeros).
constexpr int kXRow2 = 1924;
constexpr int kDRow2 = 1288;
constexpr int kRowVox2 = 1280;

// Weight and bias gradient of layer 2 on MFMA (X = h1 channel-last on the
// padded grid, dY = d2 channel-last on the compact rows, both turned
// channel-first as they enter LDS):
//   dW[co][ci][t] = sum over tile voxels v of dY[co][v] X[ci][v + off(t)],
//   db[co] = sum over v of dY[co][v],
// the products as 16 (co) x 16 (ci) x 32 (voxels) MFMAs: 32 consecutive
// compact-row entries of dY (aligned 16-byte reads) against the same
// entries of the padded X shifted by the tap (a run of 8 entries never
// leaves its z plane, where the two layouts are contiguous alike; the y and
// z shifts keep X 8-byte aligned, the x shifts come from x_shifts).  One
// workgroup per compute unit loops over tiles and keeps every tap's 16 x 16
// block in registers, 8 waves for the first half of the K steps and 8 for the
// second (8 waves for all: 17.5 us for 256 tiles, now 15.9); one partial
// [27][16][16] + [16] per workgroup.
template <int CI, int CO>
__global__ __launch_bounds__(1024) void k_wgrad_mfma(const uint16_t *__restrict__ X, const uint16_t *__restrict__ dY,
                                                    int64_t n, float *__restrict__ partials)
{
    __shared__ __align__(16) uint16_t sx[16 * kXRow2];
    __shared__ __align__(16) uint16_t sd[16 * kDRow2];
    __shared__ float sb[1024];
    const int tid = threadIdx.x, wave = (tid >> 6) & 7, part = tid >> 9, lane = tid & 63;
    const int i = lane & 15, g = lane >> 4;
    // wave w: the taps t = 3w .. 3w + 2 of the (y, z) offset pair w (x
    // offsets -1, 0, +1, one read for the three); waves 0..2 also tap
    // 24 + w of pair 8 (y and z offsets +1)
    const int ky = wave % 3 - 1, kz = wave / 3 - 1;
    for (int k = tid; k < 16 * kXRow2 / 8; k += 1024) reinterpret_cast<uint4 *>(sx)[k] = make_uint4(0, 0, 0, 0);
    for (int k = tid; k < 16 * kDRow2 / 8; k += 1024) reinterpret_cast<uint4 *>(sd)[k] = make_uint4(0, 0, 0, 0);
    v4f acc[4];
    for (int j = 0; j < 4; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    __syncthreads();
    // 16-byte chunks of a tile: X (CI channels) then dY (CO channels), the
    // next tile's held in registers while the current one is computed
    constexpr int kXc = kPadVox / 8, kDc = kRowVox / 8;
    constexpr int kChunks = CI * kXc + CO * kDc;
    constexpr int kPer = (kChunks + 1023) / 1024;
    uint4 nxt[kPer];
    auto fetch = [&](int64_t tl) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 1024 * e;
            if (k < CI * kXc) nxt[e] = reinterpret_cast<const uint4 *>(X + tl * CI * kPadVox)[k];
            else if (k < kChunks) nxt[e] = reinterpret_cast<const uint4 *>(dY + tl * CO * kRowVox)[k - CI * kXc];
        }
    };
    if (blockIdx.x < n) fetch(blockIdx.x);
    for (int64_t tile = blockIdx.x; tile < n; tile += gridDim.x) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int k = tid + 1024 * e;
            if (k < CI * kXc) {
                scatter8(sx + (k & 1) * 8 * kXRow2 + 8, kXRow2, k >> 1, nxt[e]);
            } else if (k < kChunks) {
                const int kk = k - CI * kXc;
                scatter8(sd + (kk & 1) * 8 * kDRow2, kDRow2, kk >> 1, nxt[e]);
            }
        }
        __syncthreads();
        if (tile + gridDim.x < n) fetch(tile + gridDim.x);
        for (int c = tid >> 4; c < kRowVox; c += 64) bsum += bf2f(sd[(tid & 15) * kDRow2 + c]);
        const uint16_t *xrow = sx + i * kXRow2;
        // K steps: runs of 8 entries 64 apart for the four lane groups
        // (c = cb + j + 64 g over 1280 entries, the last 64 zero in dY)
        for (int step = part * (kRowVox2 / 64); step < (part + 1) * (kRowVox2 / 64); ++step) {
            const int c = 256 * (step >> 3) + 8 * (step & 7) + 64 * g;
            const v8bf a = as_v8bf(*reinterpret_cast<const v4u *>(sd + i * kDRow2 + c));
            const int plane = c / 120, within = c - 120 * plane;
            const int pc = 8 + within + 12 + 144 * (plane + 1);
            v4u bm, b0, bp;
            x_shifts(xrow + pc + 12 * ky + 144 * kz, bm, b0, bp);
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_v8bf(bm), acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_v8bf(b0), acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_v8bf(bp), acc[2], 0, 0, 0);
            if (wave < 3) {
                x_shifts(xrow + pc + 12 + 144, bm, b0, bp);
                acc[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_v8bf(wave == 0 ? bm : (wave == 1 ? b0 : bp)),
                                                                 acc[3], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // the second half's sums to the first, through LDS
    float *other = reinterpret_cast<float *>(sx);
    if (part == 1)
        for (int j = 0; j < 4; ++j) *reinterpret_cast<v4f *>(other + ((tid & 511) * 4 + j) * 4) = acc[j];
    sb[tid] = bsum;
    __syncthreads();
    float *out = partials + int64_t(blockIdx.x) * (kWPack + kC);
    if (part == 0) for (int j = 0; j < 4; ++j) acc[j] += *reinterpret_cast<const v4f *>(other + (tid * 4 + j) * 4);
    // lane: column ci = i, rows co = 4g .. 4g + 3
    for (int j = 0; j < 4; ++j) {
        const int t = j < 3 ? 3 * wave + j : 24 + wave;
        if (part == 0 && (j < 3 || wave < 3))
            for (int r = 0; r < 4; ++r) out[(t * kC + 4 * g + r) * kC + i] = acc[j][r];
    }
    if (tid < kC) {
        float sum = 0.f;
        for (int k = 0; k < 64; ++k) sum += sb[k * 16 + tid];
        out[kWPack + tid] = sum;
    }
}

// Forward pass of n given tiles, every layer as 27 products of 16 voxels x 16
// output channels x 16 input channels (v_mfma_f32_16x16x16_bf16), one per
// tap in order (layer 1 its weights' high and low parts), so each output is
// the same sum in the same order whatever the batch.  One workgroup takes a
// tile at a time; all activations lie in LDS on the zero-bordered 12^3 grid,
// where every tap is a fixed offset, and the weights are rounded and packed
// there once per workgroup: one launch and no scratch.  Bound by the latency
// of a tile up to one tile per compute unit, then by the LDS operand reads.
// With a launch per layer, index arithmetic per tap and five launches to pack
// the weights and the tiles, 32 tiles took 172 us and 1024 357; now 25 and 88.
typedef short v4s __attribute__((ext_vector_type(4)));
constexpr int kFwdWaves = 16, kFwdRows = (kMT + kFwdWaves - 1) / kFwdWaves;   // row tiles per wave
constexpr int kFwdTap2 = kC * kC + 4, kFwdTap1 = kC * 4 + 4;
struct FwdLds {
    alignas(16) uint16_t h1[kPadVox * kC], h2[kPadVox * kC];     // [padded voxel][channel]
    // weights by tap, the taps 2 (mod 64) LDS banks apart so that packing
    // them in parameter order (taps fastest) meets no bank twice
    alignas(16) uint16_t w2[kTaps * kFwdTap2];                   // [tap][output][input channel]
    alignas(16) uint16_t w1[kTaps * kFwdTap1], w1l[kTaps * kFwdTap1];   // [tap][output][4 inputs, 2 used], high, low parts
    alignas(16) uint16_t w3[kTaps * kC];                         // [tap][input channel]
    uint32_t x0[kPadVox];                                        // the two input channels
};
__global__ __launch_bounds__(64 * kFwdWaves) void k_net_tiles(const float *__restrict__ tiles, int64_t n,
                                                              const float *__restrict__ params,
                                                              float *__restrict__ out)
{
    __shared__ FwdLds sh;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    constexpr int kThreads = 64 * kFwdWaves;
    // a thread's voxel of the tile, if it has one, and its input, loaded a tile ahead
    float nf = 0.f, nw = 0.f;
    auto fetch = [&](int64_t tile) {
        if (tid < kT) {
            nf = tiles[tile * 2 * kT + tid];
            nw = tiles[tile * 2 * kT + kT + tid];
        }
    };
    static_assert(kThreads >= kT, "one voxel per thread");
    if (blockIdx.x < n) fetch(blockIdx.x);
    for (int k = tid; k < kPadVox * kC / 8; k += kThreads) {
        reinterpret_cast<uint4 *>(sh.h1)[k] = make_uint4(0, 0, 0, 0);
        reinterpret_cast<uint4 *>(sh.h2)[k] = make_uint4(0, 0, 0, 0);
    }
    for (int k = tid; k < kPadVox; k += kThreads) sh.x0[k] = 0u;
    for (int k = tid; k < kTaps * kC * kC; k += kThreads) {      // parameter order: coalesced reads
        const int t = k % kTaps, ci = (k / kTaps) % kC, co = k / (kTaps * kC);
        sh.w2[t * kFwdTap2 + co * kC + ci] = f2bf(params[kW2 + k]);
    }
    for (int k = tid; k < kTaps * kC * 2; k += kThreads) {
        const int t = k % kTaps, ci = (k / kTaps) % 2, co = k / (kTaps * 2);
        const float w = params[kW1 + k];
        const int at = t * kFwdTap1 + co * 4 + ci;
        sh.w1[at] = f2bf(w);
        sh.w1l[at] = f2bf(w - bf2f(f2bf(w)));
        sh.w1[at + 2] = 0;
        sh.w1l[at + 2] = 0;
    }
    for (int k = tid; k < kTaps * kC; k += kThreads) sh.w3[(k % kTaps) * kC + k / kTaps] = f2bf(params[kW3 + k]);
    const int i = lane & 15, kg = lane >> 4;
    const float b1 = params[kB1 + i], b2 = params[kB2 + i], b3 = params[kB3];
    // the wave's row tiles: wave, wave + 16, ...; this lane's row (an operand)
    // and its four rows of the result, on the padded grid
    int row[kFwdRows], res[kFwdRows][4];
#pragma unroll
    for (int q = 0; q < kFwdRows; ++q) {
        const int mt = wave + q * kFwdWaves;
        auto padded = [](int v) { return v < kT ? pad_index(v % 10, (v / 10) % 10, v / 100) : -1; };
        const int v = padded(mt * 16 + i);
        row[q] = v < 0 ? pad_index(0, 0, 0) : v;         // (a row past the tile: computed, not stored)
        for (int r = 0; r < 4; ++r) res[q][r] = padded(mt * 16 + 4 * kg + r);
    }
    const v4s zero = {0, 0, 0, 0};
    const int own = tid < kT ? pad_index(tid % 10, (tid / 10) % 10, tid / 100) : 0;
    for (int64_t tile = blockIdx.x; tile < n; tile += gridDim.x) {
        if (tid < kT) sh.x0[own] = uint32_t(f2bf(nf)) | (uint32_t(f2bf(nw)) << 16);
        __syncthreads();
        if (tile + gridDim.x < n) fetch(tile + gridDim.x);
        v4f acc[kFwdRows];
        auto clear = [&]() {
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q) acc[q] = v4f{0.f, 0.f, 0.f, 0.f};
        };
        auto store = [&](uint16_t *h, float bias) {
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float y = acc[q][r] + bias;
                    y = y > 0.f ? y : 0.f;
                    if (res[q][r] >= 0) h[res[q][r] * kC + i] = f2bf(y);
                }
        };
        // (the taps of a (y, z) pair unrolled, the nine pairs not: the
        // operands of a whole layer would not fit the registers)
        auto layer = [&](auto product) {
            clear();
#pragma unroll 1
            for (int pair = 0; pair < 9; ++pair) {
                const int at = 12 * (pair % 3 - 1) + 144 * (pair / 3 - 1) - 1;
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) product(3 * pair + kx, at + kx);
            }
        };
        layer([&](int t, int off) {
            v4s bh = zero, bl = zero;
            if (kg == 0) {
                bh = *reinterpret_cast<const v4s *>(&sh.w1[t * kFwdTap1 + i * 4]);
                bl = *reinterpret_cast<const v4s *>(&sh.w1l[t * kFwdTap1 + i * 4]);
            }
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q) {
                const uint32_t x = kg == 0 ? sh.x0[row[q] + off] : 0u;
                const v4s a = {short(x & 0xFFFFu), short(x >> 16), 0, 0};
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bh, acc[q], 0, 0, 0);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bl, acc[q], 0, 0, 0);
            }
        });
        store(sh.h1, b1);
        __syncthreads();
        layer([&](int t, int off) {
            const v4s b = *reinterpret_cast<const v4s *>(&sh.w2[t * kFwdTap2 + i * kC + 4 * kg]);
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q) {
                const v4s a = *reinterpret_cast<const v4s *>(&sh.h1[(row[q] + off) * kC + 4 * kg]);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[q], 0, 0, 0);
            }
        });
        store(sh.h2, b2);
        __syncthreads();
        layer([&](int t, int off) {
            const v4s b = i == 0 ? *reinterpret_cast<const v4s *>(&sh.w3[t * kC + 4 * kg]) : zero;
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q) {
                const v4s a = *reinterpret_cast<const v4s *>(&sh.h2[(row[q] + off) * kC + 4 * kg]);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[q], 0, 0, 0);
            }
        });
        if (i == 0)
#pragma unroll
            for (int q = 0; q < kFwdRows; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (res[q][r] >= 0) out[tile * kT + (wave + q * kFwdWaves) * 16 + 4 * kg + r] = acc[q][r] + b3;
        // the next tile's x0 is not read before the next barrier, and no wave
        // writes h1 or h2 again before all have passed two
    }
}

static int forward_tiles(const float *tiles, int64_t n, const float *params, float *out, hipStream_t st)
{
    int dev = 0, cus = 0;
    DN_HIP(hipGetDevice(&dev));
    DN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    hipLaunchKernelGGL(k_net_tiles, dim3(unsigned(std::min<int64_t>(n, std::max(cus, 1)))), dim3(64 * kFwdWaves), 0, st,
                       tiles, n, params, out);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

}  // namespace dn

using namespace dn;

extern "C" {

int dn_net_gather(dn_volume *v, const int32_t *blocks, int64_t n, int32_t perm, float *tiles)
{
    DN_REQUIRE(v && blocks && tiles && n >= 0 && perm >= 0 && perm <= 2, "bad argument");
    if (n == 0) return DN_OK;
    hipLaunchKernelGGL(k_gather, dim3(grid1(n * kT)), dim3(256), 0, v->stream, v->nbr, v->f, v->w, blocks,
                       n, tiles, int(perm));
    DN_HIP(hipGetLastError());
    return DN_OK;
}

size_t dn_net_bytes(int64_t n_tiles, int32_t training)
{
    if (n_tiles < 0 || (training != 0 && training != 1)) return 0;
    Bump b(nullptr, 0);
    carve_net(b, n_tiles, training != 0);
    return (b.off + 255) & ~size_t(255);
}

int dn_net_forward(const float *tiles, int64_t n, const float *params, float *out, void *workspace,
                   size_t workspace_bytes, void *stream)
{
    DN_REQUIRE(tiles && params && out && n >= 0, "bad argument");
    if (n == 0) return DN_OK;
    DN_REQUIRE(ws_ok(workspace), "the workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < dn_net_bytes(n, 0)) {
        set_error("workspace of %zu bytes is short: %zu needed (dn_net_bytes)", workspace_bytes, dn_net_bytes(n, 0));
        return DN_E_CAPACITY;
    }
    return forward_tiles(tiles, n, params, out, static_cast<hipStream_t>(stream));
}

int dn_net_forward_static(const float *tiles, int64_t n, const float *params, float *out, void *stream)
{
    DN_REQUIRE(tiles && params && out && n >= 0, "bad argument");
    if (n > DN_NET_STATIC_TILES) {
        set_error("dn_net_forward_static takes at most %d tiles per call (%lld given)", DN_NET_STATIC_TILES,
                  (long long)n);
        return DN_E_CAPACITY;
    }
    if (n == 0) return DN_OK;
    return forward_tiles(tiles, n, params, out, static_cast<hipStream_t>(stream));
}

int dn_net_loss_grad(const float *tiles, int64_t n, const float *params, const float *targets, const float *mask,
                     int32_t kind, float *grad, void *workspace, size_t workspace_bytes, double *loss_host,
                     void *stream)
{
    DN_REQUIRE(tiles && params && targets && mask && grad && n > 0 && (kind == 0 || kind == 1), "bad argument");
    DN_REQUIRE(ws_ok(workspace), "the workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < dn_net_bytes(n, 1)) {
        set_error("workspace of %zu bytes is short: %zu needed (dn_net_bytes)", workspace_bytes, dn_net_bytes(n, 1));
        return DN_E_CAPACITY;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    Bump bump(workspace, workspace_bytes);
    const NetWS ws = carve_net(bump, n, true);
    int dev = 0, cus = 0;
    DN_HIP(hipGetDevice(&dev));
    DN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // a workgroup of 8 waves per compute unit (two of 4 waves leave half the
    // units' waves idle at 256 tiles: 20.6 and 15.4 us for the two kernels
    // against 27.2 and 23.5; where every unit has two tiles the whole step is
    // within 2 %: 512 tiles 130 us with 8, 129 with 4, 4096 696 and 710)
    const unsigned grid1w = unsigned(std::min<int64_t>(n, std::max(cus, 1)));
    // a loss word that the device can write (pinned) spares the copy: with that
    // and the loss in the forward pass a step of 256 tiles 141.6 -> 103 to 114 us (it differs by process)
    double *host_loss = nullptr;
    if (loss_host) {
        hipPointerAttribute_t at{};
        if (hipPointerGetAttributes(&at, loss_host) == hipSuccess && at.type == hipMemoryTypeHost)
            host_loss = static_cast<double *>(at.devicePointer);
        else (void)hipGetLastError();
    }
    double *lsum = ws.misc;   // [0] loss, [1] 1 / N (written by k_grad_final)
    const TrainIO io{ws.x1cf, ws.h1cf, ws.h2cf, ws.gates, targets, mask, int(kind), ws.d3, ws.d3cf, ws.tl, ws.tc};
    // weights; forward with the layer inputs kept, loss and its gradient on the centre
    hipLaunchKernelGGL(k_pack_train, dim3(grid1(kLaneW + kL2M * 64 * 8)), dim3(256), 0, st, params, ws.lanew,
                       ws.lanef);
    hipLaunchKernelGGL((k_net_fwd<kTraining, 8>), dim3(grid1w), dim3(512), 0, st, (const int32_t *)nullptr,
                       (const uint32_t *)nullptr, tiles, (const uint8_t *)nullptr, n, ws.lanew, params, int64_t(0),
                       (float *)nullptr, io);
    DN_HIP(hipGetLastError());
    // input gradients of layers 3 and 2
    hipLaunchKernelGGL(k_net_bwd<8>, dim3(grid1w), dim3(512), 0, st, ws.d3, ws.gates, n, ws.lanef, params, ws.d2cf,
                       ws.d1cf);
    DN_HIP(hipGetLastError());
    // weight gradients, one partial per workgroup and layer, summed in a fixed order
    const unsigned gw = unsigned(ws.nparts);
    const size_t lp = size_t(ws.nparts) * (kWPack + kC);
    hipLaunchKernelGGL(k_wgrad13, dim3(2 * gw), dim3(512), 0, st, ws.x1cf, ws.d1cf, ws.h2cf, ws.d3cf, n, ws.parts,
                       ws.parts + 2 * lp, int(gw));
    hipLaunchKernelGGL((k_wgrad_mfma<16, 16>), dim3(gw), dim3(1024), 0, st, ws.h1cf, ws.d2cf, n, ws.parts + lp);
    hipLaunchKernelGGL(k_grad_final, dim3((kPart1 + kPart2 + kPart3 + kFinalEntries - 1) / kFinalEntries), dim3(256), 0, st,
                       ws.parts, ws.nparts, ws.tl, ws.tc, n, lsum, host_loss, grad);
    DN_HIP(hipGetLastError());
    if (host_loss) {
        DN_HIP(hipStreamSynchronize(st));
    } else if (loss_host) {
        double h = 0.0;
        DN_HIP(hipMemcpyAsync(&h, lsum, 8, hipMemcpyDeviceToHost, st));
        DN_HIP(hipStreamSynchronize(st));
        *loss_host = h;
    }
    return DN_OK;
}

int dn_net_adam(float *params, const float *grad, float *m, float *v, int64_t n, float lr, float beta1, float beta2,
                float eps, int32_t step, void *stream)
{
    DN_REQUIRE(params && grad && m && v && n > 0 && step >= 1, "bad argument");
    hipStream_t st = static_cast<hipStream_t>(stream);
    float c1 = 1.f - std::pow(beta1, float(step)), c2 = 1.f - std::pow(beta2, float(step));
    hipLaunchKernelGGL(k_adam, dim3(grid1(n)), dim3(256), 0, st, params, grad, m, v, n, lr, beta1, beta2, eps, c1, c2);
    DN_HIP(hipGetLastError());
    return DN_OK;
}

size_t dn_warm_start_bytes(int64_t n_blocks)
{
    if (n_blocks < 0) return 0;
    Bump b(nullptr, 0);
    b.take<uint16_t>(size_t(kLaneW));
    b.take<uint32_t>(size_t(n_blocks) * kBlockVox);
    return (b.off + 255) & ~size_t(255);
}

int dn_net_warm_start(dn_volume *v, const float *params, int32_t mode, double delta, float *u0, float *p0,
                      void *workspace, size_t workspace_bytes)
{
    DN_REQUIRE(v && params && u0 && (mode == DN_WARM_PRIMAL || mode == DN_WARM_DUAL), "bad argument");
    DN_REQUIRE(mode == DN_WARM_DUAL ? p0 != nullptr : delta > 0, "dual mode needs p0; primal mode needs delta > 0");
    hipStream_t st = v->stream;
    int rc;
    if ((rc = build_masks(v))) return rc;
    if (v->nb == 0) return DN_OK;
    DN_REQUIRE(ws_ok(workspace), "the workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < dn_warm_start_bytes(v->nb)) {
        set_error("workspace of %zu bytes is short: %zu needed (dn_warm_start_bytes)", workspace_bytes,
                  dn_warm_start_bytes(v->nb));
        return DN_E_CAPACITY;
    }
    Bump bump(workspace, workspace_bytes);
    uint16_t *lanew = bump.take<uint16_t>(size_t(kLaneW));
    uint32_t *vp = bump.take<uint32_t>(size_t(v->nb) * kBlockVox);
    hipLaunchKernelGGL(k_pack_lanes, dim3(grid1(kLaneW)), dim3(256), 0, st, params, lanew);
    DN_HIP(hipGetLastError());
    int cus = 0;
    DN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, v->device));
    // two workgroups fit a compute unit (77 KiB of LDS each); each loops over tiles and axes
    const int axes = mode == DN_WARM_DUAL ? 3 : 1;
    const unsigned grid = unsigned(std::min<int64_t>(v->nb * axes, int64_t(2) * (cus > 0 ? cus : 1)));
    const int64_t ps = v->nb * int64_t(kBlockVox);
    hipLaunchKernelGGL(k_voxel_pairs, dim3(grid1(ps)), dim3(256), 0, st, v->f, v->w, ps, vp);
    auto fwd = mode == DN_WARM_DUAL ? k_net_fwd<kDual, 4> : k_net_fwd<kPrimal, 4>;
    hipLaunchKernelGGL(fwd, dim3(grid), dim3(256), 0, st, v->nbr, vp, v->f, v->emask, v->nb, lanew, params, ps,
                       mode == DN_WARM_DUAL ? p0 : u0, TrainIO{});
    DN_HIP(hipGetLastError());
    if (mode == DN_WARM_DUAL) {
        hipLaunchKernelGGL(k_warm_finish, dim3(grid1(ps)), dim3(256), 0, st, ps, ps, v->emask, v->f, p0, u0);
        DN_HIP(hipGetLastError());
    } else if (p0) {
        hipLaunchKernelGGL(k_warm_p, dim3(unsigned(v->nb)), dim3(512), 0, st, v->nb, ps, v->nbr, v->emask, u0,
                           float(1.0 / delta), p0);
        DN_HIP(hipGetLastError());
    }
    return DN_OK;
}

}  // extern "C"
