// Extraction of the volume's parts and of the zero-crossing surface of u
// (the model handed to consumers, Section II / Fig. 2 of the paper).
#include <cstring>
#include <rocprim/rocprim.hpp>

#include "dn_internal.h"

namespace dn {

static inline unsigned grid1(int64_t n, int bs = 256) { return unsigned((n + bs - 1) / bs); }

// One workgroup of 256 threads takes a block, two voxels per thread (v and
// v + 256).  u on the block and its +1 faces, edges and corner is staged in
// LDS, and for each of its 81 rows along x which voxels are observed (bits 0
// to 8) and which have u < 0 (bits 16 to 24): a voxel's neighbours are then
// a fixed offset or a shift away, without a neighbour lookup and two loads
// per corner.
constexpr int kTile = 729;                 // index x + 9 y + 81 z, 0..8 each
__device__ __forceinline__ int tile_at(int v) { return (v & 7) + 9 * ((v >> 3) & 7) + 81 * (v >> 6); }

struct Tile {
    float u[kTile];
    uint32_t row[81];                      // index y + 9 z
    uint8_t x8[81];                        // the row's voxel at x = 8: observed, u < 0
};

__device__ __forceinline__ void load_tile(Tile &sh, int64_t b, const int32_t *__restrict__ nbr,
                                          const uint32_t *__restrict__ em4, const float *__restrict__ u, int t)
{
    const int i = t & 63, p = i & 7, q = i >> 3;
    // the bits of a wave whose lanes are x + 8 k: row k of them
    auto rows = [&](uint32_t c, int at) {
        const uint64_t o = __ballot(c & 1u), n = __ballot(c & 2u);
        if (i < 8) sh.row[at] = uint32_t(o >> (8 * i)) & 255u | (uint32_t(n >> (8 * i)) & 255u) << 16;
    };
    auto get = [&](int at, int64_t block, int v) {
        const float x = u[block * kBlockVox + v];
        sh.u[at] = x;
        return ((em4[block * 64 + (v & 63)] >> (4 * (v >> 6))) & 1u) | (x < 0.0f ? 2u : 0u);
    };
    rows(get(tile_at(t), b, t), i + 9 * (t >> 6));
    rows(get(tile_at(t + 256), b, t + 256), i + 9 * (t >> 6) + 36);
    // by wave: the +x, +y and +z faces; then the edges along z, y and x (8
    // lanes each) and the corner
    int x, y, z;
    if (t < 64) { x = 8; y = p; z = q; }
    else if (t < 128) { x = p; y = 8; z = q; }
    else if (t < 192) { x = p; y = q; z = 8; }
    else if (i < 8) { x = 8; y = 8; z = p; }
    else if (i < 16) { x = 8; y = p; z = 8; }
    else if (i < 24) { x = p; y = 8; z = 8; }
    else { x = 8; y = 8; z = 8; }
    uint32_t c = 0;
    if (t < 217) {
        const int at = x + 9 * y + 81 * z;
        const int32_t id = nbr[b * kNbr + 13 + (x >> 3) + 3 * (y >> 3) + 9 * (z >> 3)];
        if (id >= 0) c = get(at, id, (x & 7) + 8 * (y & 7) + 64 * (z & 7));
        else sh.u[at] = 0.0f;
        if (x == 8) sh.x8[y + 9 * z] = uint8_t(c);
    }
    if (t >= 64 && t < 128) rows(c, 8 + 9 * i);
    if (t >= 128 && t < 192) rows(c, i + 72);
    if (t >= 192) {
        const uint64_t o = __ballot(c & 1u), n = __ballot(c & 2u);
        if (i == 0) sh.row[80] = uint32_t(o >> 16) & 255u | (uint32_t(n >> 16) & 255u) << 16;
    }
    __syncthreads();
    if (t < 81) sh.row[t] |= (sh.x8[t] & 1u) << 8 | (sh.x8[t] >> 1) << 24;
    __syncthreads();
}

// Observed (bits 0, 1) and negative (16, 17) of voxel v + (0 or 1, dy, dz).
__device__ __forceinline__ uint32_t pair_at(const Tile &sh, int v, int dy, int dz)
{
    return sh.row[((v >> 3) & 7) + dy + 9 * ((v >> 6) + dz)] >> (v & 7);
}

// Exclusive prefix, in voxel order, of the counts (below 16) of the
// workgroup's two voxels per thread, and their total.
__device__ __forceinline__ int prefix_counts(int c0, int c1, int &p0, int &p1, int *wave_sum /* [8] */)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t below = (uint64_t(1) << lane) - 1;
    auto prefix = [&](int c, int &sum) {
        int p = 0;
        sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t m = __ballot((c >> k) & 1);
            p += __popcll(m & below) << k;
            sum += __popcll(m) << k;
        }
        return p;
    };
    int s0, s1;
    p0 = prefix(c0, s0);
    p1 = prefix(c1, s1);
    if (lane == 0) {
        wave_sum[wave] = s0;
        wave_sum[4 + wave] = s1;
    }
    __syncthreads();
    int total = 0;
    for (int k = 0; k < 8; ++k) {
        if (k == wave) p0 += total;
        if (k == 4 + wave) p1 += total;
        total += wave_sum[k];
    }
    return total;
}

// Zero crossings of voxel v: axes a with both v and v + e_a observed and
// u(v) < 0 differing from u(v + e_a) < 0.
__device__ __forceinline__ int crossing_bits(const Tile &sh, int v)
{
    const uint32_t c = pair_at(sh, v, 0, 0), y = pair_at(sh, v, 1, 0), z = pair_at(sh, v, 0, 1);
    // bit 0: both observed and different signs
    const uint32_t ox = c & (c >> 1) & ((c >> 16) ^ (c >> 17)), oy = c & y & ((c ^ y) >> 16), oz = c & z & ((c ^ z) >> 16);
    return int((ox & 1u) | (oy & 1u) << 1 | (oz & 1u) << 2);
}

__global__ __launch_bounds__(256) void k_surface_count(const int32_t *__restrict__ nbr, const uint32_t *__restrict__ em4,
                                                       const float *__restrict__ u, int64_t *__restrict__ counts)
{
    __shared__ Tile sh;
    __shared__ int wave_sum[8];
    const int64_t b = blockIdx.x;
    const int t = threadIdx.x;
    load_tile(sh, b, nbr, em4, u, t);
    int p0, p1;
    const int n = prefix_counts(__popc(crossing_bits(sh, t)), __popc(crossing_bits(sh, t + 256)), p0, p1, wave_sum);
    if (t == 0) counts[b] = n;
}

__global__ __launch_bounds__(256) void k_surface_write(const int32_t *__restrict__ coords,
                                                       const int32_t *__restrict__ nbr, const uint32_t *__restrict__ em4,
                                                       const float *__restrict__ u, const int64_t *__restrict__ offsets,
                                                       double s, float *__restrict__ out)
{
    __shared__ Tile sh;
    __shared__ int wave_sum[8];
    const int64_t b = blockIdx.x, first = offsets[b];
    if (offsets[b + 1] == first) return;
    const int t = threadIdx.x;
    load_tile(sh, b, nbr, em4, u, t);
    const int bits[2] = {crossing_bits(sh, t), crossing_bits(sh, t + 256)};
    int p[2];
    prefix_counts(__popc(bits[0]), __popc(bits[1]), p[0], p[1], wave_sum);
    const int4 c4 = reinterpret_cast<const int4 *>(coords)[b];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int v = t + 256 * j, at = tile_at(v);
        const int step[3] = {1, 9, 81};
        int64_t pos = first + p[j];
        const double centre[3] = {(double(8 * c4.x + (v & 7)) + 0.5) * s, (double(8 * c4.y + ((v >> 3) & 7)) + 0.5) * s,
                                  (double(8 * c4.z + (v >> 6)) + 0.5) * s};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (!(bits[j] & (1 << a))) continue;
            const double u0 = sh.u[at], u1 = sh.u[at + step[a]];
            const double tt = u0 / (u0 - u1);
#pragma unroll
            for (int i = 0; i < 3; ++i) out[3 * pos + i] = float(centre[i] + (i == a ? tt * s : 0.0));
            ++pos;
        }
    }
}

// ------------------------------------------------------------------ mesh
// Zero level set of u as triangles (Section II; Tables III and IV report
// the area of this surface).  Cubes are voxel g and g + {0,1}^3 (corner
// k = x + 2y + 4z), meshed only when all eight corners are observed (bit 0
// of the edge mask).  Each cube is cut into six tetrahedra along its main
// diagonal, corners 0, e_a0, e_a0 + e_a1, 7 for the axis orders below, so
// neighbouring cubes cut their shared faces alike.  One vertex alone on
// its side of zero gives the triangle on its three edges (increasing
// tetrahedron order); two and two (negative a < b, positive c < d) give
// (ac, ad, bd) and (ac, bd, bc).  Edge points are taken from the corner
// with the smaller k, so a shared edge is computed identically everywhere;
// a triangle is turned when its normal points against r = n_neg *
// sum(positive offsets) - n_pos * sum(negative offsets).  Double precision
// throughout; the output rounds to float.  Order: pool id, voxel,
// tetrahedron, triangle.
//
// A cube's signs decide its triangles, so a block first lists them (cube,
// tetrahedron, which of two) in order in LDS, then every thread computes
// triangles of the list: all lanes work, where a thread per voxel left seven
// of eight idle beside the few on the surface, and no array is indexed by a
// variable outside LDS.  5777 blocks, 1.28 million triangles: area 190 -> 40
// us, writing 222 -> 39 (the triangles alone are 46 MB), counting 55 -> 11.

// The tetrahedra's corners (a nibble each, first to last), by tables that the
// compiler fills.
struct MeshTables {
    uint16_t corners[6];
    uint8_t count[256];        // triangles of a cube by its corners' signs
    uint32_t edges[16][2];     // by the tetrahedron's signs and which triangle: 3 edges (two nibbles each)
    constexpr MeshTables() : corners{}, count{}, edges{}
    {
        const int axes[6][2] = {{0, 1}, {0, 2}, {1, 0}, {1, 2}, {2, 0}, {2, 1}};
        for (int t = 0; t < 6; ++t) {
            const int k1 = 1 << axes[t][0], k2 = k1 | (1 << axes[t][1]);
            corners[t] = uint16_t(k1 << 4 | k2 << 8 | 7 << 12);
        }
        for (int m = 0; m < 256; ++m) {
            int n = 0;
            for (int t = 0; t < 6; ++t) {
                int neg = 0;
                for (int q = 0; q < 4; ++q) neg += (m >> ((corners[t] >> (4 * q)) & 7)) & 1;
                n += neg == 2 ? 2 : (neg == 1 || neg == 3 ? 1 : 0);
            }
            count[m] = uint8_t(n);
        }
        for (int m = 0; m < 16; ++m) {
            int ng[4] = {}, ps[4] = {}, nn = 0, np = 0;
            for (int q = 0; q < 4; ++q) {
                if ((m >> q) & 1) ng[nn++] = q;
                else ps[np++] = q;
            }
            auto edge = [](int a, int b) { return uint32_t(a | b << 4); };
            if (nn == 1) edges[m][0] = edge(ng[0], ps[0]) | edge(ng[0], ps[1]) << 8 | edge(ng[0], ps[2]) << 16;
            if (nn == 3) edges[m][0] = edge(ps[0], ng[0]) | edge(ps[0], ng[1]) << 8 | edge(ps[0], ng[2]) << 16;
            if (nn == 2) {
                edges[m][0] = edge(ng[0], ps[0]) | edge(ng[0], ps[1]) << 8 | edge(ng[1], ps[1]) << 16;
                edges[m][1] = edge(ng[0], ps[0]) | edge(ng[1], ps[1]) << 8 | edge(ng[1], ps[0]) << 16;
            }
        }
    }
};
static __constant__ MeshTables kMesh{};

// The signs of the cube at voxel v (bit k: u < 0 at corner k); 0 (no
// triangle) unless all eight corners are observed.
__device__ __forceinline__ uint32_t cube_signs(const Tile &sh, int v)
{
    const uint32_t a = pair_at(sh, v, 0, 0), b = pair_at(sh, v, 1, 0), c = pair_at(sh, v, 0, 1), d = pair_at(sh, v, 1, 1);
    if ((a & b & c & d & 3u) != 3u) return 0u;
    return ((a >> 16) & 3u) | ((b >> 16) & 3u) << 2 | ((c >> 16) & 3u) << 4 | ((d >> 16) & 3u) << 6;
}

__device__ __forceinline__ int tet_signs(uint32_t corners, uint32_t neg)
{
    return int((neg & 1u) | ((neg >> ((corners >> 4) & 7u)) & 1u) << 1 | ((neg >> ((corners >> 8) & 7u)) & 1u) << 2 |
               ((neg >> 7) & 1u) << 3);
}

struct MeshShared {
    Tile tile;
    uint16_t list[kBlockVox * 12];         // voxel | tetrahedron << 9 | triangle << 12
    uint32_t edges[16][2];
    uint16_t corners[6];
    uint8_t count[256];
    int wave_sum[8];
};

// The block's triangles, listed in order; returns their number.
__device__ __forceinline__ int list_triangles(MeshShared &sh, int64_t b, const int32_t *__restrict__ nbr,
                                              const uint32_t *__restrict__ em4, const float *__restrict__ u, int t)
{
    sh.count[t] = kMesh.count[t];
    if (t < 32) sh.edges[t >> 1][t & 1] = kMesh.edges[t >> 1][t & 1];
    if (t < 6) sh.corners[t] = kMesh.corners[t];
    load_tile(sh.tile, b, nbr, em4, u, t);
    const uint32_t neg[2] = {cube_signs(sh.tile, t), cube_signs(sh.tile, t + 256)};
    int p[2];
    const int n = prefix_counts(sh.count[neg[0]], sh.count[neg[1]], p[0], p[1], sh.wave_sum);
    for (int j = 0; j < 2; ++j) {
        if (sh.count[neg[j]] == 0) continue;
        int at = p[j];
        for (int tt = 0; tt < 6; ++tt) {
            const int k = __popc(tet_signs(sh.corners[tt], neg[j]));
            if (k == 0 || k == 4) continue;
            const int e = (t + 256 * j) | tt << 9;
            sh.list[at++] = uint16_t(e);
            if (k == 2) sh.list[at++] = uint16_t(e | 1 << 12);
        }
    }
    __syncthreads();
    return n;
}

// Triangle e of the list: fn(A, B, C, area) with the oriented vertices.
template <class F>
__device__ __forceinline__ void triangle(const MeshShared &sh, int e, const int4 c4, double s, F fn)
{
    const int entry = sh.list[e], v = entry & 511, at = tile_at(v);
    const uint32_t corners = sh.corners[(entry >> 9) & 7];
    auto corner_at = [&](int k) { return at + (k & 1) + 9 * ((k >> 1) & 1) + 81 * (k >> 2); };
    int r[3] = {0, 0, 0};
    const int m = tet_signs(corners, cube_signs(sh.tile, v));
    const int nneg = __popc(m);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int comp = 0; comp < 3; ++comp)
            r[comp] += ((m >> q) & 1 ? nneg - 4 : nneg) * int((corners >> (4 * q + comp)) & 1u);
    const uint32_t edges = sh.edges[m][entry >> 12];
    const int base[3] = {8 * c4.x + (v & 7), 8 * c4.y + ((v >> 3) & 7), 8 * c4.z + (v >> 6)};
    double P[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int ki = int(corners >> (4 * ((edges >> (8 * k)) & 15u))) & 7;
        int kj = int(corners >> (4 * ((edges >> (8 * k + 4)) & 15u))) & 7;
        if (ki > kj) { const int x = ki; ki = kj; kj = x; }
        const double ui = sh.tile.u[corner_at(ki)], uj = sh.tile.u[corner_at(kj)];
        const double tt = ui / (ui - uj);
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            const double pi = (double(base[comp] + ((ki >> comp) & 1)) + 0.5) * s;
            const double pj = (double(base[comp] + ((kj >> comp) & 1)) + 0.5) * s;
            P[k][comp] = pi + tt * (pj - pi);
        }
    }
    const double ab[3] = {P[1][0] - P[0][0], P[1][1] - P[0][1], P[1][2] - P[0][2]};
    const double ac[3] = {P[2][0] - P[0][0], P[2][1] - P[0][1], P[2][2] - P[0][2]};
    const double nx = ab[1] * ac[2] - ab[2] * ac[1];
    const double ny = ab[2] * ac[0] - ab[0] * ac[2];
    const double nz = ab[0] * ac[1] - ab[1] * ac[0];
    const bool flip = (nx * double(r[0]) + ny * double(r[1])) + nz * double(r[2]) < 0.0;
    fn(P[0], flip ? P[2] : P[1], flip ? P[1] : P[2], 0.5 * sqrt((nx * nx + ny * ny) + nz * nz));
}

__global__ __launch_bounds__(256) void k_mesh_count(const int32_t *__restrict__ nbr, const uint32_t *__restrict__ em4,
                                                    const float *__restrict__ u, int64_t *__restrict__ counts)
{
    __shared__ Tile sh;
    __shared__ uint8_t count[256];
    __shared__ int wave_sum[8];
    const int64_t b = blockIdx.x;
    const int t = threadIdx.x;
    count[t] = kMesh.count[t];
    load_tile(sh, b, nbr, em4, u, t);
    int p0, p1;
    const int n = prefix_counts(count[cube_signs(sh, t)], count[cube_signs(sh, t + 256)], p0, p1, wave_sum);
    if (t == 0) counts[b] = n;
}

__global__ __launch_bounds__(256) void k_mesh_write(const int32_t *__restrict__ coords, const int32_t *__restrict__ nbr,
                                                    const uint32_t *__restrict__ em4, const float *__restrict__ u,
                                                    const int64_t *__restrict__ offsets, double s,
                                                    float *__restrict__ out)
{
    __shared__ MeshShared sh;
    const int64_t b = blockIdx.x, first = offsets[b];
    if (offsets[b + 1] == first) return;
    const int n = list_triangles(sh, b, nbr, em4, u, threadIdx.x);
    const int4 c4 = reinterpret_cast<const int4 *>(coords)[b];
    for (int e = threadIdx.x; e < n; e += 256)
        triangle(sh, e, c4, s, [&](const double *A, const double *B, const double *C, double) {
            float *o = out + 9 * (first + e);
            for (int i = 0; i < 3; ++i) {
                o[i] = float(A[i]);
                o[3 + i] = float(B[i]);
                o[6 + i] = float(C[i]);
            }
        });
}

// Per-block (area, triangle count) pairs, float64, fixed order: each thread
// its triangles in list order, lanes by xor butterflies, waves in order.
__global__ __launch_bounds__(256) void k_mesh_area(const int32_t *__restrict__ coords, const int32_t *__restrict__ nbr,
                                                   const uint32_t *__restrict__ em4, const float *__restrict__ u,
                                                   double s, double *__restrict__ partials)
{
    __shared__ MeshShared sh;
    __shared__ double wa[4];
    const int64_t b = blockIdx.x;
    const int t = threadIdx.x;
    const int n = list_triangles(sh, b, nbr, em4, u, t);
    const int4 c4 = reinterpret_cast<const int4 *>(coords)[b];
    double a = 0.0;
    for (int e = t; e < n; e += 256)
        triangle(sh, e, c4, s, [&](const double *, const double *, const double *, double ar) { a += ar; });
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if ((t & 63) == 0) wa[t >> 6] = a;
    __syncthreads();
    if (t == 0) {
        partials[2 * b] = ((wa[0] + wa[1]) + wa[2]) + wa[3];
        partials[2 * b + 1] = double(n);
    }
}

__global__ void k_fill_zero_i64(int64_t *a) { *a = 0; }

// Offsets of nb counts and their total (ofs[nb], also reported), by one
// workgroup: quicker than a device-wide scan's launches up to kScanBlocks.
constexpr int64_t kScanBlocks = 32768;
__global__ __launch_bounds__(1024) void k_scan_counts(const int64_t *__restrict__ cnt, int nb, int64_t *__restrict__ ofs,
                                                      int64_t *__restrict__ total)
{
    __shared__ int64_t wave_sum[16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int64_t carry = 0;
    int64_t ahead[4];
    auto fetch = [&](int i0) {
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + 4 * t + k;
            ahead[k] = i < nb ? cnt[i] : 0;
        }
    };
    fetch(0);
    for (int i0 = 0; i0 < nb; i0 += 4096) {
        int64_t c[4];
        for (int k = 0; k < 4; ++k) c[k] = ahead[k];
        fetch(i0 + 4096);
        const int64_t mine = (c[0] + c[1]) + (c[2] + c[3]);
        int64_t inc = mine;
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t other = __shfl_up(inc, d, 64);
            if (lane >= d) inc += other;
        }
        if (lane == 63) wave_sum[wave] = inc;
        __syncthreads();
        int64_t at = carry + inc - mine;
        for (int k = 0; k < 16; ++k) {
            if (k < wave) at += wave_sum[k];
            carry += wave_sum[k];
        }
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + 4 * t + k;
            if (i < nb) ofs[i] = at;
            at += c[k];
        }
        __syncthreads();
    }
    if (t == 0) {
        ofs[nb] = carry;
        *total = carry;
    }
}

__global__ void k_copy_coords(const int32_t *__restrict__ c4, int64_t nb, int32_t *__restrict__ out)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < nb * 3) out[i] = c4[4 * (i / 3) + i % 3];
}

__global__ void k_unpack_keys(const uint64_t *__restrict__ k, int64_t n, int32_t *__restrict__ out)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t m = (uint64_t(1) << 21) - 1;
    const int64_t off = int64_t(1) << 20;
    out[3 * i] = int32_t(int64_t((k[i] >> 42) & m) - off);
    out[3 * i + 1] = int32_t(int64_t((k[i] >> 21) & m) - off);
    out[3 * i + 2] = int32_t(int64_t(k[i] & m) - off);
}

struct ScanScratch {
    int64_t *cnt, *ofs;
    void *tmp;
    size_t tmp_bytes;
};
static ScanScratch carve_scan(Bump &b, int64_t nb)
{
    ScanScratch x;
    x.cnt = b.take<int64_t>(size_t(nb) + 1);
    x.ofs = b.take<int64_t>(size_t(nb) + 1);
    x.tmp_bytes = tmp_light(size_t(nb) + 1);
    x.tmp = b.take<char>(x.tmp_bytes);
    return x;
}

size_t extract_scratch(int64_t n_blocks)
{
    Bump b(nullptr, 0);
    carve_scan(b, n_blocks);
    return b.off;
}

// Per-block counts (count_kernel) -> offsets -> total, in the scratch.
template <class CountK>
static int count_and_scan(dn_volume *v, CountK count_kernel, ScanScratch &x, int64_t *total)
{
    hipStream_t st = v->stream;
    const int64_t nb = v->nb;
    Bump bump(v->scratch, v->scratch_bytes);
    x = carve_scan(bump, nb);
    if (!bump.fits()) { set_error("scratch too small for the extraction"); return DN_E_CAPACITY; }
    if (nb > 0) {
        hipLaunchKernelGGL(count_kernel, dim3(unsigned(nb)), dim3(256), 0, st, v->nbr, v->em4, v->u, x.cnt);
        DN_HIP(hipGetLastError());
    }
    if (nb > 0 && nb <= kScanBlocks) {
        hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, st, x.cnt, int(nb), x.ofs, report(v));
        DN_HIP(hipGetLastError());
        const int rc = fetch_report(v, 1);
        *total = v->host_stage[0];
        return rc;
    }
    hipLaunchKernelGGL(k_fill_zero_i64, dim3(1), dim3(1), 0, st, x.cnt + nb);
    DN_HIP(hipGetLastError());
    size_t tbytes = x.tmp_bytes;
    DN_HIP(rocprim::exclusive_scan(x.tmp, tbytes, x.cnt, x.ofs, int64_t(0), size_t(nb + 1), rocprim::plus<int64_t>(),
                                   st));
    int rc = read_back(v, x.ofs + nb, 8);
    if (rc) return rc;
    *total = v->host_stage[0];
    return DN_OK;
}

}  // namespace dn

using namespace dn;

extern "C" int dn_extract(dn_volume *v, int32_t what, void *out, size_t out_bytes, int64_t *n_out)
{
    DN_REQUIRE(v && n_out, "null argument");
    hipStream_t st = v->stream;
    const int64_t nb = v->nb, nv = nb * kBlockVox, ps = v->cap_blocks * kBlockVox;
    int64_t items = 0;
    size_t need = 0;
    int rc;
    uint64_t *uniq = nullptr;
    switch (what) {
    case DN_X_COORDS: items = nb; need = size_t(nb) * 12; break;
    case DN_X_HASH: items = v->hash_slots; need = size_t(items) * 16; break;
    case DN_X_NBR: items = nb; need = size_t(nb) * kNbr * 4; break;
    case DN_X_F: case DN_X_W: case DN_X_U: case DN_X_UBAR: items = nb; need = size_t(nv) * 4; break;
    case DN_X_P: items = nb; need = size_t(nv) * 12; break;
    case DN_X_EMASK: items = nb; need = size_t(nv); break;
    case DN_X_CANDIDATES:
        if ((rc = build_candidates(v, &uniq, &items))) return rc;
        need = size_t(items) * 12;
        break;
    case DN_X_SURFACE: {
        if ((rc = build_masks(v))) return rc;
        ScanScratch x;
        if ((rc = count_and_scan(v, k_surface_count, x, &items))) return rc;
        need = size_t(items) * 12;
        *n_out = items;
        if (items == 0) return DN_OK;
        if (!out || out_bytes < need) { set_error("output too small: need %zu bytes", need); return DN_E_CAPACITY; }
        hipLaunchKernelGGL(k_surface_write, dim3(unsigned(nb)), dim3(256), 0, st, v->coords, v->nbr, v->em4, v->u,
                           x.ofs, v->prm.voxel_size, static_cast<float *>(out));
        DN_HIP(hipGetLastError());
        DN_HIP(hipStreamSynchronize(st));
        return DN_OK;
    }
    case DN_X_MESH: {
        if ((rc = build_masks(v))) return rc;
        ScanScratch x;
        if ((rc = count_and_scan(v, k_mesh_count, x, &items))) return rc;
        need = size_t(items) * 36;
        *n_out = items;
        if (items == 0) return DN_OK;
        if (!out || out_bytes < need) { set_error("output too small: need %zu bytes", need); return DN_E_CAPACITY; }
        hipLaunchKernelGGL(k_mesh_write, dim3(unsigned(nb)), dim3(256), 0, st, v->coords, v->nbr, v->em4, v->u,
                           x.ofs, v->prm.voxel_size, static_cast<float *>(out));
        DN_HIP(hipGetLastError());
        DN_HIP(hipStreamSynchronize(st));
        return DN_OK;
    }
    default:
        set_error("unknown extract target %d", what);
        return DN_E_INVALID;
    }
    *n_out = items;
    if (need == 0) return DN_OK;
    if (!out || out_bytes < need) { set_error("output too small: need %zu bytes", need); return DN_E_CAPACITY; }
    switch (what) {
    case DN_X_COORDS:
        hipLaunchKernelGGL(k_copy_coords, dim3(grid1(nb * 3)), dim3(256), 0, st, v->coords, nb, static_cast<int32_t *>(out));
        DN_HIP(hipGetLastError());
        break;
    case DN_X_HASH: DN_HIP(hipMemcpyAsync(out, v->hash[v->cur_hash], need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_NBR: DN_HIP(hipMemcpyAsync(out, v->nbr, need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_F: DN_HIP(hipMemcpyAsync(out, v->f, need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_W: DN_HIP(hipMemcpyAsync(out, v->w, need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_U: DN_HIP(hipMemcpyAsync(out, v->u, need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_UBAR: DN_HIP(hipMemcpyAsync(out, v->ubar[v->cur], need, hipMemcpyDeviceToDevice, st)); break;
    case DN_X_P:
        for (int a = 0; a < 3; ++a)
            DN_HIP(hipMemcpyAsync(static_cast<float *>(out) + a * nv, v->p[v->cur] + a * ps, size_t(nv) * 4,
                                  hipMemcpyDeviceToDevice, st));
        break;
    case DN_X_EMASK:
        if ((rc = build_masks(v))) return rc;
        DN_HIP(hipMemcpyAsync(out, v->emask, need, hipMemcpyDeviceToDevice, st));
        break;
    case DN_X_CANDIDATES:
        hipLaunchKernelGGL(k_unpack_keys, dim3(grid1(items)), dim3(256), 0, st, uniq, items,
                           static_cast<int32_t *>(out));
        DN_HIP(hipGetLastError());
        break;
    }
    DN_HIP(hipStreamSynchronize(st));
    return DN_OK;
}

// Total area (float64) and number of the mesh's triangles.
extern "C" int dn_mesh_area(dn_volume *v, double *area, int64_t *n_tris)
{
    DN_REQUIRE(v && area, "null argument");
    int rc;
    if ((rc = build_masks(v))) return rc;
    double ed[2] = {0.0, 0.0};
    if (v->nb > 0) {
        hipLaunchKernelGGL(k_mesh_area, dim3(unsigned(v->nb)), dim3(256), 0, v->stream, v->coords, v->nbr, v->em4,
                           v->u, v->prm.voxel_size, v->partials);
        DN_HIP(hipGetLastError());
        if ((rc = reduce_pairs(v, v->nb))) return rc;
        if ((rc = read_energy(v, ed))) return rc;
    }
    *area = ed[0];
    if (n_tris) *n_tris = int64_t(ed[1]);
    return DN_OK;
}
