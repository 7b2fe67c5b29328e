// Volume lifecycle, block allocation (grid traversal, dedupe, canonical
// hash), projective TSDF fusion and plain extraction for gfx950.
//
// Section III-A of the paper (hashing voxel grid, Eq. 1).  Discrete
// decisions (block keys, pixel choice, truncation test) are taken in
// float64 with contraction disabled, so they are reproducible bit for bit.
#include <cstring>  // rocprim needs memset declared before its headers
#include <rocprim/rocprim.hpp>

#include <cstdarg>
#include <algorithm>
#include <cmath>

#include "dn_internal.h"

namespace dn {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int read_back(dn_volume *v, const void *dev, size_t bytes)
{
    if (bytes > sizeof(v->host_stage)) { set_error("read-back too large"); return DN_E_INVALID; }
    DN_HIP(hipMemcpyAsync(v->host_stage, dev, bytes, hipMemcpyDeviceToHost, v->stream));
    DN_HIP(hipStreamSynchronize(v->stream));
    return DN_OK;
}

int64_t *report(dn_volume *v) { return v->report ? v->report : v->misc + kMiscReport; }

int fetch_report(dn_volume *v, int words)
{
    if (!v->report) return read_back(v, v->misc + kMiscReport, size_t(words) * 8);
    DN_HIP(hipStreamSynchronize(v->stream));
    memcpy(v->host_stage, v->report_host, size_t(words) * 8);
    return DN_OK;
}

int volume_sync(dn_volume *v)
{
    DN_HIP(hipStreamSynchronize(v->stream));
    return DN_OK;
}

// ------------------------------------------------------------ block keys
constexpr int64_t kKeyOff = int64_t(1) << 20;   // 21 bits per axis

__host__ __device__ inline uint64_t pack_key(int32_t x, int32_t y, int32_t z)
{
    return (uint64_t(int64_t(x) + kKeyOff) << 42) | (uint64_t(int64_t(y) + kKeyOff) << 21) |
           uint64_t(int64_t(z) + kKeyOff);
}

__host__ __device__ inline void unpack_key(uint64_t k, int32_t &x, int32_t &y, int32_t &z)
{
    const uint64_t m = (uint64_t(1) << 21) - 1;
    x = int32_t(int64_t((k >> 42) & m) - kKeyOff);
    y = int32_t(int64_t((k >> 21) & m) - kKeyOff);
    z = int32_t(int64_t(k & m) - kKeyOff);
}

__device__ inline uint32_t bucket_of(int32_t x, int32_t y, int32_t z, uint32_t cap)
{
    uint32_t h = (uint32_t(x) * 73856093u) ^ (uint32_t(y) * 19349669u) ^ (uint32_t(z) * 83492791u);
    return h & (cap - 1u);
}

// Probe forward from the bucket until the key or an empty slot; the table
// never wraps, so the walk is bounded by the slot count.
__device__ inline int32_t hash_lookup(const int4 *slots, int64_t nslots, uint32_t cap, int32_t x,
                                      int32_t y, int32_t z)
{
    for (int64_t pos = bucket_of(x, y, z, cap); pos < nslots; ++pos) {
        int4 sl = slots[pos];
        if (sl.w < 0) return -1;
        if (sl.x == x && sl.y == y && sl.z == z) return sl.w;
    }
    return -1;
}

struct Geo {
    double fx, fy, cx, cy;
    double T[16];
    double s, mu, maxd;
    int32_t W, H;
};

__device__ inline bool depth_ok(float d, double maxd)
{
    return isfinite(d) && d > 0.0f && double(d) <= maxd;
}

// Amanatides-Woo traversal of a -> b on the unit grid (ties x before y
// before z, only axes with steps left towards the end cell); nothing is
// visited if an end point lies beyond `limit` cells (at most 1e9, so that
// cells and step counts fit 32 bits).  Shared by the depth band, the laser
// band and the laser fusion walks.
struct Walk {
    int32_t k[3], e[3], step[3];     // cell, end cell
    double tmax[3], tdel[3];         // an axis without steps left has tmax = infinity
    // false: nothing to visit
    __device__ __forceinline__ bool start(const double a[3], const double b[3], double limit)
    {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (!(fabs(a[i]) < limit && fabs(b[i]) < limit)) return false;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            k[i] = int32_t(floor(a[i]));
            e[i] = int32_t(floor(b[i]));
            const double dir = b[i] - a[i];
            if (e[i] != k[i]) {
                step[i] = e[i] > k[i] ? 1 : -1;
                tmax[i] = (double(e[i] > k[i] ? k[i] + 1 : k[i]) - a[i]) / dir;
                tdel[i] = double(step[i]) / dir;
            } else {
                step[i] = 0; tmax[i] = HUGE_VAL; tdel[i] = 0.0;
            }
        }
        return true;
    }
    __device__ __forceinline__ int64_t cells() const
    {
        return int64_t(abs(e[0] - k[0])) + abs(e[1] - k[1]) + abs(e[2] - k[2]) + 1;
    }
    // On to the next cell; false at the end cell.  `at` receives the segment's
    // parameter where it leaves the cell, `moved` the bits of the coordinate
    // that changed.  No branches: lanes of a wave step along different axes.
    __device__ __forceinline__ bool next(double &at, int32_t &moved)
    {
        const bool by = tmax[1] < tmax[0];
        const double t = by ? tmax[1] : tmax[0];
        const bool bz = tmax[2] < t;
        at = bz ? tmax[2] : t;
        const bool go = at < HUGE_VAL;
        const bool sel[3] = {go && !by && !bz, by && !bz, bz};
        moved = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int32_t kn = k[i] + (sel[i] ? step[i] : 0);
            moved |= kn ^ k[i];
            k[i] = kn;
            tmax[i] += sel[i] ? tdel[i] : 0.0;
            if (sel[i] && kn == e[i]) tmax[i] = HUGE_VAL;
        }
        return go;
    }
    __device__ __forceinline__ bool next()
    {
        double at;
        int32_t moved;
        return next(at, moved);
    }
};

template <class Emit>
__device__ int64_t walk_segment(const double a[3], const double b[3], double limit, Emit emit)
{
    Walk w;
    if (!w.start(a, b, limit)) return 0;
    int64_t n = 0;
    do {
        emit(n, w.k[0], w.k[1], w.k[2]);
        ++n;
    } while (w.next());
    return n;
}

// Grid traversal of one pixel's band [max(d - mu, 1e-3), d + mu] over the
// block grid (edge 8 s).  Emits the visited block keys through `emit` and
// returns how many were visited.
template <class Emit>
__device__ int dda_pixel(const Geo &g, int px, int py, float d, Emit emit)
{
    const double bs = 8.0 * g.s;
    double rx = (double(px) - g.cx) / g.fx;
    double ry = (double(py) - g.cy) / g.fy;
    double z0 = double(d) - g.mu;
    if (z0 < 1e-3) z0 = 1e-3;
    double z1 = double(d) + g.mu;
    double a[3], b[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double pa = ((g.T[4 * i + 0] * (z0 * rx) + g.T[4 * i + 1] * (z0 * ry)) + g.T[4 * i + 2] * z0) + g.T[4 * i + 3];
        double pb = ((g.T[4 * i + 0] * (z1 * rx) + g.T[4 * i + 1] * (z1 * ry)) + g.T[4 * i + 2] * z1) + g.T[4 * i + 3];
        a[i] = pa / bs;
        b[i] = pb / bs;
    }
    return int(walk_segment(a, b, 1e6, [&](int64_t j, int32_t x, int32_t y, int32_t z) { emit(int(j), x, y, z); }));
}

// The cells of one point's band, for the allocation kernel below.
struct DepthBand {
    Geo g;
    const float *depth;
    template <class Emit> __device__ int64_t operator()(int64_t i, Emit emit) const
    {
        const float d = depth[i];
        if (!depth_ok(d, g.maxd)) return 0;
        return dda_pixel(g, int(i % g.W), int(i / g.W), d,
                         [&](int, int32_t x, int32_t y, int32_t z) { emit(pack_key(x, y, z)); });
    }
};

__global__ void k_pack_coords(const int32_t *__restrict__ c3, int64_t n, uint64_t *__restrict__ out)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = pack_key(c3[3 * i], c3[3 * i + 1], c3[3 * i + 2]);
}

// flag[i] = 1 when raw candidate i (repeats allowed) is not in the table.
__global__ void k_flag_unknown(const uint64_t *__restrict__ cand, int64_t n, const int4 *__restrict__ slots,
                               int64_t nslots, uint32_t cap, uint8_t *__restrict__ flag)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t x, y, z;
    unpack_key(cand[i], x, y, z);
    flag[i] = hash_lookup(slots, nslots, cap, x, y, z) < 0 ? 1 : 0;
}

// Append the sorted new keys after the existing pool; clear their fields.
__global__ void k_append(const uint64_t *__restrict__ newk, int64_t n_new, int64_t nb_old,
                         int32_t *__restrict__ coords, uint64_t *__restrict__ keys)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n_new) return;
    int32_t x, y, z;
    unpack_key(newk[i], x, y, z);
    int64_t b = nb_old + i;
    keys[b] = newk[i];
    coords[4 * b + 0] = x; coords[4 * b + 1] = y; coords[4 * b + 2] = z; coords[4 * b + 3] = 0;
}

// The per-voxel fields of blocks [first, first + count) in several arrays
// at once (the new blocks of an allocation: f, w, u, both ubar and both
// sets of dual planes), one launch instead of one per array.
struct FieldSet {
    float *a[16];
    int n;
};
__device__ __forceinline__ void zero_fields(const FieldSet &fs, int64_t first, int64_t i)   // 4 voxels
{
    for (int k = 0; k < fs.n; ++k)
        reinterpret_cast<float4 *>(fs.a[k] + first * kBlockVox)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void k_zero_fields(FieldSet fs, int64_t first, int64_t count)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count * (kBlockVox / 4)) zero_fields(fs, first, i);
}

__global__ void k_iota(int32_t *__restrict__ a, int64_t n)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) a[i] = int32_t(i);
}

__global__ void k_bucket_of_keys(const uint64_t *__restrict__ keys, int64_t n, uint32_t cap,
                                 uint32_t *__restrict__ home)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t x, y, z;
    unpack_key(keys[i], x, y, z);
    home[i] = bucket_of(x, y, z, cap);
}

// d[i] = home_sorted[i] - i (as int64), scanned later with max
__global__ void k_home_minus_rank(const uint32_t *__restrict__ home, int64_t n, int64_t *__restrict__ d)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) d[i] = int64_t(home[i]) - i;
}

__global__ void k_zero_i32(int32_t *a) { *a = 0; }

__global__ void k_fill_empty(int4 *__restrict__ slots, int64_t n)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) slots[i] = make_int4(0, 0, 0, -1);
}

// Canonical slot of the i-th key in (bucket, key) order:
// pos = max_{j<=i}(home_j - j) + i  (sequential linear probing, unrolled);
// the last key's is the end of the occupied slots.
__global__ void k_scatter_slots(const int64_t *__restrict__ runmax, const int32_t *__restrict__ ids,
                                const int32_t *__restrict__ coords, int64_t n, int64_t nslots,
                                int4 *__restrict__ slots, int32_t *__restrict__ overflow, int64_t *__restrict__ end)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int64_t pos = runmax[i] + i;
    if (i == n - 1) *end = pos;
    if (pos >= nslots) { atomicOr(overflow, 1); return; }
    int32_t id = ids[i];
    slots[pos] = make_int4(coords[4 * id], coords[4 * id + 1], coords[4 * id + 2], id);
}

__global__ void k_nbr_table(const int32_t *__restrict__ coords, int64_t nb, const int4 *__restrict__ slots,
                            int64_t nslots, uint32_t cap, int32_t *__restrict__ nbr)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= nb * kNbr) return;
    int64_t b = i / kNbr;
    int o = int(i % kNbr);
    int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
    nbr[i] = (o == kCentre) ? int32_t(b)
                            : hash_lookup(slots, nslots, cap, coords[4 * b] + dx,
                                          coords[4 * b + 1] + dy, coords[4 * b + 2] + dz);
}

static inline unsigned grid1(int64_t n, int bs = 256) { return unsigned((n + bs - 1) / bs); }

static int bits_for(uint64_t v)
{
    int b = 1;
    while (b < 64 && (v >> b)) ++b;
    return b;
}

InsertScratch carve_insert(Bump &b, int64_t n_cand, int64_t n_blocks)
{
    InsertScratch x;
    x.flags = b.take<uint8_t>(size_t(n_cand));
    x.newraw = b.take<uint64_t>(size_t(n_cand));
    x.sorted = b.take<uint64_t>(size_t(n_cand));
    x.newk = b.take<uint64_t>(size_t(n_cand));
    x.pos0 = b.take<int32_t>(size_t(n_cand));
    x.pos1 = b.take<int32_t>(size_t(n_cand));
    x.ksorted = b.take<uint64_t>(size_t(n_blocks));
    x.ids0 = b.take<int32_t>(size_t(n_blocks));
    x.ids1 = b.take<int32_t>(size_t(n_blocks));
    x.home = b.take<uint32_t>(size_t(n_blocks));
    x.dm = b.take<int64_t>(size_t(n_blocks));
    x.runmax = b.take<int64_t>(size_t(n_blocks));
    x.tmp_bytes = std::max(std::max(tmp_sort(size_t(n_cand), 12), tmp_light(size_t(n_cand))),
                           std::max(tmp_sort(size_t(n_blocks), 12), tmp_light(size_t(n_blocks))));
    x.tmp = b.take<char>(x.tmp_bytes);
    return x;
}

// flags[i] = 1 where sorted[i] starts a run of equal keys
__global__ void k_run_heads(const uint64_t *__restrict__ sorted, int64_t n, uint8_t *__restrict__ flags)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) flags[i] = (i == 0 || sorted[i] != sorted[i - 1]) ? 1 : 0;
}

__global__ void k_gather_keys(const uint64_t *__restrict__ keys, const int32_t *__restrict__ pos, int64_t n,
                              uint64_t *__restrict__ out)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = keys[pos[i]];
}

static FieldSet field_set(const dn_volume *v)
{
    FieldSet fs{};
    float *fields[] = {v->f, v->w, v->u, v->ubar[0], v->ubar[1]};
    for (float *a : fields) fs.a[fs.n++] = a;
    for (int pp = 0; pp < 2; ++pp)
        for (int a = 0; a < 3; ++a) fs.a[fs.n++] = v->p[pp] + size_t(a) * v->cap_blocks * kBlockVox;
    return fs;
}

// -------------------------------------------------- allocation of one frame
// A frame's band cells name few distinct blocks, and after the first frames
// hardly any new one.  One kernel walks the bands; each workgroup keeps the
// distinct keys of its points in an LDS set, and each of those is
// looked up once; the unknown ones meet in a small set in global memory,
// whose first inserter lists the key.  The host reads the counts (the call's
// one wait); new blocks then take three more launches, none of which sorts
// or scans more than the new keys and the list of occupied slots.  Bound by
// latency: 12 frames of 1242 x 375 take 0.78 ms, 3.72 ms with a full sort of
// the pool and four waits per frame; four of 320 x 96 0.29 ms, 1.18 before.
// Points (threads) per workgroup: each workgroup adds to the same counters,
// so on a large frame fewer, larger ones are quicker (1242 x 375: 256 points
// 50 us, 512 30 us, 1024 28 us); a small frame needs them spread over the
// chip.
constexpr int64_t kBandSmall = int64_t(1) << 17;
constexpr int kBandSet = 1024;          // slots of its LDS set
constexpr int kBandList = 512;          // distinct keys it lists; more go on one by one
constexpr uint64_t kNoKey = ~uint64_t(0);

struct BandOut {
    uint64_t *cand;                     // distinct keys of each workgroup (repeats between them)
    int64_t cand_cap;
    uint64_t *set;                      // [kNewSet], kNoKey at rest
    uint64_t *new_key;                  // [kMaxNew]
    uint32_t *new_home, *new_slot;
    int64_t *misc;
    int64_t *host;                      // report: total cells, listed keys, new keys, overflow, table end
};

__device__ __forceinline__ uint32_t key_mix(uint64_t k)
{
    return uint32_t((k * 0x9E3779B97F4A7C15ull) >> 32);
}

// A key that its workgroup met first: look it up; if it is in no block yet,
// list it once for all workgroups.  Probing is bounded: a set that fills up
// sends the frame to the general path.
__device__ void band_key(const BandOut &o, uint64_t key, const int4 *slots, int64_t nslots, uint32_t cap)
{
    int32_t x, y, z;
    unpack_key(key, x, y, z);
    if (hash_lookup(slots, nslots, cap, x, y, z) >= 0) return;
    unsigned long long *set = reinterpret_cast<unsigned long long *>(o.set);
    uint32_t h = key_mix(key) & (kNewSet - 1);
    for (int probe = 0; probe < 64; ++probe, h = (h + 1) & (kNewSet - 1)) {
        const unsigned long long old = atomicCAS(set + h, (unsigned long long)kNoKey, (unsigned long long)key);
        if (old == key) return;
        if (old != kNoKey) continue;
        const unsigned long long at = atomicAdd(reinterpret_cast<unsigned long long *>(o.misc + kMiscNew), 1ull);
        if (at < kMaxNew) {
            o.new_key[at] = key;
            o.new_home[at] = bucket_of(x, y, z, cap);
            o.new_slot[at] = h;
        } else {
            atomicOr(reinterpret_cast<unsigned long long *>(o.misc + kMiscFull), 1ull);
        }
        return;
    }
    atomicOr(reinterpret_cast<unsigned long long *>(o.misc + kMiscFull), 1ull);
}

// The last workgroup's done count shares a word with the cells.
constexpr int kDoneShift = 40;

template <class Band, int kBandPoints>
__global__ __launch_bounds__(kBandPoints) void k_band(Band band, int64_t n, const int4 *__restrict__ slots,
                                                      int64_t nslots, uint32_t cap, BandOut o)
{
    __shared__ unsigned long long set[kBandSet];
    __shared__ uint64_t list[kBandList];
    __shared__ unsigned n_list;
    __shared__ unsigned long long cells, base;
    const int tid = threadIdx.x;
    for (int k = tid; k < kBandSet; k += kBandPoints) set[k] = kNoKey;
    if (tid == 0) { n_list = 0; cells = 0; }
    __syncthreads();
    unsigned long long mine = 0;
    const int64_t i = int64_t(blockIdx.x) * kBandPoints + tid;
    unsigned long long *listed_all = reinterpret_cast<unsigned long long *>(o.misc + kMiscListed);
    if (i < n)
        mine = (unsigned long long)band(i, [&](uint64_t key) {
            uint32_t h = key_mix(key) & (kBandSet - 1);
            for (int probe = 0; probe < 32; ++probe, h = (h + 1) & (kBandSet - 1)) {
                // (other waves fill slots meanwhile: a key is read as one)
                unsigned long long old = __hip_atomic_load(set + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (old == kNoKey) old = atomicCAS(set + h, (unsigned long long)kNoKey, (unsigned long long)key);
                if (old == key) return;
                if (old == kNoKey) break;
            }
            // first met here (or the set is crowded: a repeat does no harm)
            const unsigned at = atomicAdd(&n_list, 1u);
            if (at < kBandList) {
                list[at] = key;
            } else {
                const unsigned long long to = atomicAdd(listed_all, 1ull);
                if (to < (unsigned long long)o.cand_cap) o.cand[to] = key;
                band_key(o, key, slots, nslots, cap);
            }
        });
    for (int d = 32; d > 0; d >>= 1) mine += __shfl_xor(mine, d, 64);
    if ((tid & 63) == 0 && mine) atomicAdd(&cells, mine);
    __syncthreads();
    const unsigned listed = min(n_list, unsigned(kBandList));
    if (listed) {
        if (tid == 0) base = atomicAdd(listed_all, (unsigned long long)listed);
        for (unsigned k = tid; k < listed; k += kBandPoints) band_key(o, list[k], slots, nslots, cap);
        __syncthreads();
        for (unsigned k = tid; k < listed; k += kBandPoints)
            if (base + k < (unsigned long long)o.cand_cap) o.cand[base + k] = list[k];
    }
    // The last workgroup hands the counts to the host and clears them.  The
    // counts are atomics of device scope, complete before their workgroup's
    // cells are added; a release fence per workgroup, which would write back
    // the L2 each time, cost 100 us a frame.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid != 0) return;
    const unsigned long long one = 1ull << kDoneShift;
    const unsigned long long before = atomicAdd(reinterpret_cast<unsigned long long *>(o.misc + kMiscCells), cells + one);
    if ((before >> kDoneShift) + 1ull != gridDim.x) return;
    const int which[4] = {kMiscListed, kMiscNew, kMiscFull, kMiscEnd};
    o.host[0] = int64_t((before + cells) & (one - 1ull));
    for (int k = 0; k < 4; ++k)
        o.host[1 + k] = __hip_atomic_load(o.misc + which[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int k = 0; k < 3; ++k) o.misc[which[k]] = 0;
    o.misc[kMiscCells] = 0;
    __threadfence_system();
}

// A new volume's counters (all 32 words) and its set of new keys.
__global__ void k_init_misc(int64_t *__restrict__ misc, uint64_t *__restrict__ set)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 32) misc[i] = 0;
    if (i < kNewSet) set[i] = kNoKey;
}

__global__ void k_fill_keys(uint64_t *__restrict__ a, int64_t n)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) a[i] = kNoKey;
}

// Append n <= kMaxNew listed keys to the pool in ascending order, list them
// in (home bucket, key) order too, empty their slots of the set, and (the
// workgroups past the first `rank_groups`) empty the table to be built.  A
// key's place in either order is the number of keys before it: 16 lanes
// count for each.
__global__ __launch_bounds__(256) void k_append_ranked(const uint64_t *__restrict__ key, const uint32_t *__restrict__ home,
                                                       const uint32_t *__restrict__ slot, int n, int rank_groups,
                                                       int64_t nb_old, uint64_t *__restrict__ set,
                                                       int32_t *__restrict__ coords, uint64_t *__restrict__ keys,
                                                       uint32_t *__restrict__ s_home, uint64_t *__restrict__ s_key,
                                                       int32_t *__restrict__ s_id, int4 *__restrict__ table,
                                                       int64_t nslots)
{
    if (int(blockIdx.x) >= rank_groups) {
        const int64_t stride = int64_t(gridDim.x - rank_groups) * 256;
        for (int64_t i = int64_t(blockIdx.x - rank_groups) * 256 + threadIdx.x; i < nslots; i += stride)
            table[i] = make_int4(0, 0, 0, -1);
        return;
    }
    const int sub = threadIdx.x & 15, i = int(blockIdx.x) * 16 + (threadIdx.x >> 4);
    if (i >= n) return;
    const uint64_t k = key[i];
    const uint32_t h = home[i];
    int by_key = 0, by_home = 0;
    for (int j = sub; j < n; j += 16) {
        const uint64_t kj = key[j];
        const uint32_t hj = home[j];
        by_key += kj < k;
        by_home += hj < h || (hj == h && kj < k);
    }
    for (int d = 8; d > 0; d >>= 1) {
        by_key += __shfl_xor(by_key, d, 16);
        by_home += __shfl_xor(by_home, d, 16);
    }
    if (sub != 0) return;
    const int64_t b = nb_old + by_key;
    int32_t x, y, z;
    unpack_key(k, x, y, z);
    keys[b] = k;
    reinterpret_cast<int4 *>(coords)[b] = make_int4(x, y, z, 0);
    s_home[by_home] = h;
    s_key[by_home] = k;
    s_id[by_home] = int32_t(b);
    set[slot[i]] = kNoKey;
}

// The canonical table of the old blocks (listed in (home, key) order) and n
// new ones, by one workgroup: merge the two lists (each key's place is its
// own rank plus the number of the other list's keys before it), then each
// key's slot as in k_scatter_slots.  Bound by the latency of its few
// dependent steps: both lists and the merged one stay in LDS where they fit,
// and go through global memory up to kMergeBlocks, where one workgroup is
// quicker than the launches of a device-wide sort or scan.
constexpr int64_t kMergeBlocks = 65536;
template <bool kLds>
__global__ __launch_bounds__(1024) void k_merge_table(const uint32_t *__restrict__ o_home, const int32_t *__restrict__ o_ids,
                                                      int nb_old, const uint32_t *__restrict__ s_home,
                                                      const uint64_t *__restrict__ s_key,
                                                      const int32_t *__restrict__ s_id, int n,
                                                      const uint64_t *__restrict__ keys, uint32_t *g_home,
                                                      int32_t *g_ids, const int32_t *__restrict__ coords,
                                                      int4 *__restrict__ table, int64_t nslots,
                                                      int64_t *__restrict__ end, int32_t *__restrict__ overflow)
{
    extern __shared__ uint32_t lds[];
    __shared__ int wave_max[16];
    uint32_t *nh = lds;                                              // [n]
    uint32_t *oh = lds + n;                                          // [nb_old], kLds
    uint32_t *m_home = kLds ? oh + nb_old : g_home;                  // [nb_old + n]
    int32_t *m_ids = kLds ? reinterpret_cast<int32_t *>(m_home + nb_old + n) : g_ids;
    const int t = threadIdx.x;
    for (int k = t; k < n; k += 1024) nh[k] = s_home[k];
    if constexpr (kLds)
        for (int k = t; k < nb_old; k += 1024) oh[k] = o_home[k];
    if (t == 0) *overflow = 0;
    const uint32_t *oldh = kLds ? oh : o_home;
    __syncthreads();
    // the first position of a list whose bucket is h or more
    auto lower = [](const uint32_t *a, int len, uint32_t h) {
        int lo = 0, hi = len;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (a[mid] < h) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    for (int i = t; i < nb_old; i += 1024) {
        const uint32_t h = oldh[i];
        const int id = o_ids[i];
        int c = lower(nh, n, h);
        if (c < n && nh[c] == h) {
            const uint64_t k = keys[id];
            while (c < n && nh[c] == h && s_key[c] < k) ++c;
        }
        m_home[i + c] = h;
        m_ids[i + c] = id;
    }
    for (int r = t; r < n; r += 1024) {
        const uint32_t h = nh[r];
        int c = lower(oldh, nb_old, h);
        if (c < nb_old && oldh[c] == h) {
            const uint64_t k = s_key[r];
            while (c < nb_old && oldh[c] == h && keys[o_ids[c]] < k) ++c;
        }
        m_home[r + c] = h;
        m_ids[r + c] = s_id[r];
    }
    __syncthreads();
    const int nb = nb_old + n;
    if constexpr (kLds)
        for (int i = t; i < nb; i += 1024) {
            g_home[i] = m_home[i];
            g_ids[i] = m_ids[i];
        }
    // tiles of 1024 keys, the running maximum carried from one to the next;
    // the first tiles' coordinates are on their way before the scan starts
    constexpr int kAhead = 4;
    int4 ahead[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
        if (k * 1024 + t < nb) ahead[k] = reinterpret_cast<const int4 *>(coords)[m_ids[k * 1024 + t]];
    int carry = INT32_MIN;
    for (int i0 = 0; i0 < nb; i0 += 1024) {
        const int i = i0 + t;
        int4 q = ahead[0];
#pragma unroll
        for (int k = 1; k < kAhead; ++k) ahead[k - 1] = ahead[k];
        int run = INT32_MIN, id = 0;
        if (i < nb) {
            id = m_ids[i];
            run = int(m_home[i]) - i;
        }
        if (i + kAhead * 1024 < nb)
            ahead[kAhead - 1] = reinterpret_cast<const int4 *>(coords)[m_ids[i + kAhead * 1024]];
        for (int d = 1; d < 64; d <<= 1) {
            const int other = __shfl_up(run, d, 64);
            if ((t & 63) >= d) run = max(run, other);
        }
        if ((t & 63) == 63) wave_max[t >> 6] = run;
        __syncthreads();
        int top = carry;
        for (int w = 0; w < 16; ++w) {
            if (w == (t >> 6)) run = max(run, top);
            top = max(top, wave_max[w]);
        }
        carry = top;
        __syncthreads();
        if (i >= nb) continue;
        const int64_t pos = int64_t(run) + i;
        if (i == nb - 1) *end = pos;
        if (pos < nslots) table[pos] = make_int4(q.x, q.y, q.z, id);
        else *overflow = 1;
    }
}

// Neighbours of the n new blocks, both ways, and their zeroed fields (the
// workgroups past the first `nbr_groups`).
__global__ __launch_bounds__(256) void k_commit_new(const int32_t *__restrict__ coords, int64_t nb_old, int64_t n,
                                                    const int4 *__restrict__ slots, int64_t nslots, uint32_t cap,
                                                    int nbr_groups, int32_t *__restrict__ nbr, FieldSet fs)
{
    if (int(blockIdx.x) >= nbr_groups) {
        const int64_t i = int64_t(blockIdx.x - nbr_groups) * 256 + threadIdx.x;
        if (i < n * (kBlockVox / 4)) zero_fields(fs, nb_old, i);
        return;
    }
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n * kNbr) return;
    const int64_t b = nb_old + i / kNbr;
    const int o = int(i % kNbr);
    const int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
    const int32_t id = o == kCentre ? int32_t(b)
                                    : hash_lookup(slots, nslots, cap, coords[4 * b] + dx, coords[4 * b + 1] + dy,
                                                  coords[4 * b + 2] + dz);
    nbr[b * kNbr + o] = id;
    if (id >= 0 && id < nb_old) nbr[int64_t(id) * kNbr + (kNbr - 1 - o)] = int32_t(b);
}

// Empty the set of new keys after a frame that did not consume it.
static int reset_new_set(dn_volume *v)
{
    hipLaunchKernelGGL(k_fill_keys, dim3(grid1(kNewSet)), dim3(256), 0, v->stream, v->new_set, int64_t(kNewSet));
    DN_HIP(hipGetLastError());
    return DN_OK;
}

// The n_new <= kMaxNew keys that k_band listed become blocks.
static int insert_listed(dn_volume *v, int64_t n_new, int64_t table_end, int32_t *n_new_out)
{
    hipStream_t st = v->stream;
    const int64_t nb_old = v->nb, nb_new = nb_old + n_new;
    const int other = 1 - v->cur_hash;
    int4 *dst = reinterpret_cast<int4 *>(v->hash[other]);
    int32_t *d_ovf = reinterpret_cast<int32_t *>(v->misc + 2);
    const int rank_groups = int((n_new + 15) / 16);
    const int clear_groups = int(std::min<int64_t>(1024, (v->hash_slots + 1023) / 1024));
    hipLaunchKernelGGL(k_append_ranked, dim3(unsigned(rank_groups + clear_groups)), dim3(256), 0, st, v->new_key,
                       v->new_home, v->new_slot, int(n_new), rank_groups, nb_old, v->new_set, v->coords, v->keys,
                       v->sort_home, v->sort_key, v->sort_id, dst, v->hash_slots);
    const size_t lds_all = (size_t(n_new) + size_t(nb_old) + 2 * size_t(nb_new)) * 4;
    const bool in_lds = lds_all <= (size_t(60) << 10);
    const size_t lds = in_lds ? lds_all : size_t(n_new) * 4;
    hipLaunchKernelGGL(in_lds ? k_merge_table<true> : k_merge_table<false>, dim3(1), dim3(1024), lds, st, v->hord_home[v->cur_hash], v->hord_ids[v->cur_hash],
                       int(nb_old), v->sort_home, v->sort_key, v->sort_id, int(n_new), v->keys, v->hord_home[other],
                       v->hord_ids[other], v->coords, dst, v->hash_slots, v->misc + kMiscEnd, d_ovf);
    DN_HIP(hipGetLastError());
    // each key moves the end of the occupied slots by one at most: only near
    // the end of the tail does the table have to be checked before it is used
    if (std::max<int64_t>(table_end, int64_t(v->hash_cap) - 1) + n_new >= v->hash_slots) {
        int rc = read_back(v, d_ovf, sizeof(int32_t));
        if (rc) return rc;
        if (int32_t(v->host_stage[0] & 0xFFFFFFFF) != 0) {
            // the old table stays, and with it the end of its slots
            const int64_t keep = table_end;
            DN_HIP(hipMemcpyAsync(v->misc + kMiscEnd, &keep, sizeof(keep), hipMemcpyHostToDevice, st));
            DN_HIP(hipStreamSynchronize(st));
            set_error("hash table full: %lld keys do not fit 2^%d buckets + %d tail slots", (long long)nb_new,
                      v->prm.hash_cap_log2, v->prm.hash_tail);
            return DN_E_CAPACITY;
        }
    }
    v->cur_hash = other;
    v->nb = nb_new;
    v->emask_nb = -1;
    v->state_storage = DN_F32;
    const int nbr_groups = int(grid1(n_new * kNbr));
    hipLaunchKernelGGL(k_commit_new, dim3(unsigned(nbr_groups) + grid1(n_new * (kBlockVox / 4))), dim3(256), 0, st,
                       v->coords, nb_old, n_new, dst, v->hash_slots, v->hash_cap, nbr_groups, v->nbr, field_set(v));
    DN_HIP(hipGetLastError());
    if (n_new_out) *n_new_out = int32_t(n_new);
    return DN_OK;
}

// Insert a packed candidate list (device, n_cand entries, repeats allowed).
// Appends the keys not yet present in ascending order (keep_order: in the
// order of their first occurrence in the list), rebuilds hash +
// neighbours.  The raw list is first filtered against the table, so only
// candidates of new blocks are sorted (after the first frames of a sequence
// almost every candidate is a block that exists); the ascending list of all
// distinct candidates is built from the same raw list only when it is
// extracted (build_candidates).  All buffers come from the volume's scratch.
static int insert_packed(dn_volume *v, uint64_t *cand, int64_t n_cand, int32_t *n_new_out, bool keep_order = false)
{
    hipStream_t st = v->stream;
    if (n_new_out) *n_new_out = 0;
    v->cand_n = n_cand;
    if (n_cand == 0) return DN_OK;
    Bump bump(v->scratch, v->scratch_bytes);
    InsertScratch x = carve_insert(bump, n_cand, v->cap_blocks);
    if (!bump.fits()) { set_error("scratch too small for %lld candidates", (long long)n_cand); return DN_E_CAPACITY; }
    int64_t *d_nraw = v->misc;
    int64_t *d_nnew = d_nraw + 1;
    size_t tbytes;
    // 1) the candidates of blocks not in the table (repeats kept)
    const int4 *slots = reinterpret_cast<const int4 *>(v->hash[v->cur_hash]);
    hipLaunchKernelGGL(k_flag_unknown, dim3(grid1(n_cand)), dim3(256), 0, st, cand, n_cand, slots,
                       v->hash_slots, v->hash_cap, x.flags);
    DN_HIP(hipGetLastError());
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::select(x.tmp, tbytes, cand, x.flags, x.newraw, d_nraw, size_t(n_cand), st));
    int rc = read_back(v, d_nraw, sizeof(int64_t));
    if (rc) return rc;
    const int64_t n_raw = v->host_stage[0];
    if (n_raw == 0) return DN_OK;
    // 2) the distinct new keys, ascending (keep_order: in first-occurrence
    // order: a stable sort of (key, position), the first position of each
    // run of equal keys, those positions sorted, the keys gathered)
    if (!keep_order) {
        tbytes = x.tmp_bytes;
        DN_HIP(rocprim::radix_sort_keys(x.tmp, tbytes, x.newraw, x.sorted, size_t(n_raw), 0, 63, st));
        tbytes = x.tmp_bytes;
        DN_HIP(rocprim::unique(x.tmp, tbytes, x.sorted, x.newk, d_nnew, size_t(n_raw), rocprim::equal_to<uint64_t>(),
                               st));
    } else {
        hipLaunchKernelGGL(k_iota, dim3(grid1(n_raw)), dim3(256), 0, st, x.pos0, n_raw);
        DN_HIP(hipGetLastError());
        tbytes = x.tmp_bytes;
        DN_HIP(rocprim::radix_sort_pairs(x.tmp, tbytes, x.newraw, x.sorted, x.pos0, x.pos1, size_t(n_raw), 0, 63, st));
        hipLaunchKernelGGL(k_run_heads, dim3(grid1(n_raw)), dim3(256), 0, st, x.sorted, n_raw, x.flags);
        DN_HIP(hipGetLastError());
        tbytes = x.tmp_bytes;
        DN_HIP(rocprim::select(x.tmp, tbytes, x.pos1, x.flags, x.pos0, d_nnew, size_t(n_raw), st));
    }
    if ((rc = read_back(v, d_nnew, sizeof(int64_t)))) return rc;
    const int64_t n_new = v->host_stage[0];
    if (keep_order && n_new > 0) {
        tbytes = x.tmp_bytes;
        DN_HIP(rocprim::radix_sort_keys(x.tmp, tbytes, x.pos0, x.pos1, size_t(n_new), 0, bits_for(uint64_t(n_raw)),
                                        st));
        hipLaunchKernelGGL(k_gather_keys, dim3(grid1(n_new)), dim3(256), 0, st, x.newraw, x.pos1, n_new, x.newk);
        DN_HIP(hipGetLastError());
    }
    if (v->nb + n_new > v->cap_blocks) {
        set_error("block pool full: %lld + %lld new blocks > max_blocks %lld", (long long)v->nb,
                  (long long)n_new, (long long)v->cap_blocks);
        return DN_E_CAPACITY;
    }
    // 3) tentatively append (beyond nb; not committed until the hash fits)
    const int64_t nb_old = v->nb, nb_new = v->nb + n_new;
    hipLaunchKernelGGL(k_append, dim3(grid1(n_new)), dim3(256), 0, st, x.newk, n_new, nb_old, v->coords, v->keys);
    DN_HIP(hipGetLastError());
    // 4) canonical table: sort (key -> id), then stable sort by bucket
    hipLaunchKernelGGL(k_iota, dim3(grid1(nb_new)), dim3(256), 0, st, x.ids0, nb_new);
    DN_HIP(hipGetLastError());
    const int hbits = bits_for(v->hash_cap - 1);
    const int other = 1 - v->cur_hash;
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::radix_sort_pairs(x.tmp, tbytes, v->keys, x.ksorted, x.ids0, x.ids1, size_t(nb_new), 0, 63, st));
    hipLaunchKernelGGL(k_bucket_of_keys, dim3(grid1(nb_new)), dim3(256), 0, st, x.ksorted, nb_new, v->hash_cap, x.home);
    DN_HIP(hipGetLastError());
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::radix_sort_pairs(x.tmp, tbytes, x.home, v->hord_home[other], x.ids1, v->hord_ids[other],
                                     size_t(nb_new), 0, hbits, st));
    hipLaunchKernelGGL(k_home_minus_rank, dim3(grid1(nb_new)), dim3(256), 0, st, v->hord_home[other], nb_new, x.dm);
    DN_HIP(hipGetLastError());
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::inclusive_scan(x.tmp, tbytes, x.dm, x.runmax, size_t(nb_new), rocprim::maximum<int64_t>(), st));
    int4 *dst = reinterpret_cast<int4 *>(v->hash[other]);
    int32_t *d_ovf = reinterpret_cast<int32_t *>(d_nraw + 2);
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(1), 0, st, d_ovf);
    hipLaunchKernelGGL(k_fill_empty, dim3(grid1(v->hash_slots)), dim3(256), 0, st, dst, v->hash_slots);
    DN_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_scatter_slots, dim3(grid1(nb_new)), dim3(256), 0, st, x.runmax, v->hord_ids[other], v->coords,
                       nb_new, v->hash_slots, dst, d_ovf, v->misc + kMiscEnd);
    DN_HIP(hipGetLastError());
    if ((rc = read_back(v, d_ovf, sizeof(int32_t)))) return rc;
    if (int32_t(v->host_stage[0] & 0xFFFFFFFF) != 0) {
        // the old table stays; its end is unknown now, so the next frame's is checked
        const int64_t unknown = v->hash_slots;
        DN_HIP(hipMemcpyAsync(v->misc + kMiscEnd, &unknown, sizeof(unknown), hipMemcpyHostToDevice, st));
        DN_HIP(hipStreamSynchronize(st));
        set_error("hash table full: %lld keys do not fit 2^%d buckets + %d tail slots", (long long)nb_new,
                  v->prm.hash_cap_log2, v->prm.hash_tail);
        return DN_E_CAPACITY;
    }
    // 5) commit: new table, zeroed fields of the new blocks, neighbours
    v->cur_hash = other;
    hipLaunchKernelGGL(k_zero_fields, dim3(grid1(n_new * (kBlockVox / 4))), dim3(256), 0, st, field_set(v), nb_old,
                       n_new);
    DN_HIP(hipGetLastError());
    v->nb = nb_new;
    v->emask_nb = -1;
    v->state_storage = DN_F32;
    hipLaunchKernelGGL(k_nbr_table, dim3(grid1(nb_new * kNbr)), dim3(256), 0, st, v->coords, nb_new, dst,
                       v->hash_slots, v->hash_cap, v->nbr);
    DN_HIP(hipGetLastError());
    if (n_new_out) *n_new_out = int32_t(n_new);
    return DN_OK;
}

// ---------------------------------------------------------------- fusion
// Eq. 1 for voxels k0, k0 + step, ... (x fastest) of block b: project the
// centre, take the depth of the pixel it falls in, and average the
// truncated signed distance in with weight 1.  Voxels behind the camera,
// outside the image, with an invalid depth or more than mu behind the
// observed surface keep their values; free space in front of the surface
// is updated with the truncated value 1.
template <int N>
__device__ inline void fuse_voxels(const Geo &g, const float *__restrict__ depth, const int32_t *__restrict__ coords,
                                   int64_t b, int k0, int step, float *__restrict__ f, float *__restrict__ w)
{
    const int4 c = reinterpret_cast<const int4 *>(coords)[b];
    // every load is issued before its value is known to matter: the map's
    // overlap the projection, the voxels' depths each other
    float fo[N], wo[N], d[N];
    double zc[N];
    bool in[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int64_t i = b * kBlockVox + k0 + j * step;
        fo[j] = f[i];
        wo[j] = w[i];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int k = k0 + j * step;
        const int vx = k & 7, vy = (k >> 3) & 7, vz = (k >> 6) & 7;
        double d0 = (double(8 * c.x + vx) + 0.5) * g.s - g.T[3];
        double d1 = (double(8 * c.y + vy) + 0.5) * g.s - g.T[7];
        double d2 = (double(8 * c.z + vz) + 0.5) * g.s - g.T[11];
        double xc = (g.T[0] * d0 + g.T[4] * d1) + g.T[8] * d2;
        double yc = (g.T[1] * d0 + g.T[5] * d1) + g.T[9] * d2;
        zc[j] = (g.T[2] * d0 + g.T[6] * d1) + g.T[10] * d2;
        double X = g.fx * (xc / zc[j]) + g.cx;
        double Y = g.fy * (yc / zc[j]) + g.cy;
        double px = X + 0.5, py = Y + 0.5;
        in[j] = zc[j] > 0.0 && px >= 0.0 && px < double(g.W) && py >= 0.0 && py < double(g.H);
        const int ix = int(floor(px)), iy = int(floor(py));
        d[j] = depth[in[j] ? int64_t(iy) * g.W + ix : 0];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double eta = double(d[j]) - zc[j];
        if (!in[j] || !depth_ok(d[j], g.maxd) || eta < -g.mu) continue;
        double psi = eta / g.mu;
        if (psi > 1.0) psi = 1.0;
        const int64_t i = b * kBlockVox + k0 + j * step;
        const float wn = wo[j] + 1.0f;
        f[i] = (float(psi) + wo[j] * fo[j]) / wn;
        w[i] = wn;
    }
}

// Visibility culling for fusion: can any voxel centre of the block pass
// the camera tests of fuse_voxels?  The centres span a box whose image in
// camera coordinates is a parallelepiped (the pose is affine), so depth
// ranges over the corners' depths; if all corners lie in front of the
// camera the box projects into the convex hull of the projected corners.
// Conservative: margins of 1e-6 m in depth and one pixel in the image
// absorb rounding differences from the per-voxel evaluation, and a box
// reaching behind the camera counts as visible.  A block is skipped only if
// every centre is behind the camera, beyond max_depth + mu (where no valid
// depth can put it within mu of a surface) or outside the image (all corners
// past one of its sides, tested without the division by their depths).
__device__ inline bool block_in_view(const Geo &g, const int4 c)
{
    double zmin = 1e300, zmax = -1e300;
    int left = 0, right = 0, up = 0, down = 0;
    for (int k = 0; k < 8; ++k) {
        const double d0 = (double(8 * c.x + ((k & 1) ? 7 : 0)) + 0.5) * g.s - g.T[3];
        const double d1 = (double(8 * c.y + ((k & 2) ? 7 : 0)) + 0.5) * g.s - g.T[7];
        const double d2 = (double(8 * c.z + ((k & 4) ? 7 : 0)) + 0.5) * g.s - g.T[11];
        const double x = (g.T[0] * d0 + g.T[4] * d1) + g.T[8] * d2;
        const double y = (g.T[1] * d0 + g.T[5] * d1) + g.T[9] * d2;
        const double z = (g.T[2] * d0 + g.T[6] * d1) + g.T[10] * d2;
        zmin = fmin(zmin, z);
        zmax = fmax(zmax, z);
        // X + 1/2 = fx x / z + cx + 1/2 against -1 and W + 1, times z
        const double X = g.fx * x + (g.cx + 0.5) * z, Y = g.fy * y + (g.cy + 0.5) * z;
        left += X < -z;
        right += X >= (double(g.W) + 1.0) * z;
        up += Y < -z;
        down += Y >= (double(g.H) + 1.0) * z;
    }
    const double eps = 1e-6;
    if (zmax <= -eps || zmin > g.maxd + g.mu + eps) return false;
    if (zmin <= eps) return true;
    return left < 8 && right < 8 && up < 8 && down < 8;
}

// Eq. 1 over the blocks in view.  Bound by launches and latency: a frame
// touches a few MB.  Each block is tested once: lane t of workgroup g takes
// block g + t G of a grid of G workgroups, so that blocks in view, which lie
// together in the pool, are spread over the chip, and the workgroup updates
// those of its up to 256 blocks that passed.  (XCD x takes the x-th eighth of
// the g: the blocks of one line of `coords` are tested beside one L2.)  Times
// of a frame, against a test and a list in launches of their own, and against
// one launch in which every workgroup tested a whole group of 64 blocks for
// itself: 503 blocks 11.5, 6.9 and now 6.0 us; 5370 13.9, 13.8 and 8.6; 187950
// 18.7, 33.6 and 13.7; 375900 24.7, 59.4 and 17.6.
__global__ __launch_bounds__(256) void k_fuse(Geo g, const float *__restrict__ depth,
                                              const int32_t *__restrict__ coords, int64_t nb,
                                              float *__restrict__ f, float *__restrict__ w)
{
    __shared__ uint64_t seen[4];
    const int tid = threadIdx.x;
    const int64_t first = int64_t(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;      // (the grid is a multiple of 8)
    const int64_t mb = first + int64_t(tid) * gridDim.x;
    const uint64_t mine = __ballot(mb < nb && block_in_view(g, reinterpret_cast<const int4 *>(coords)[min(mb, nb - 1)]));
    if ((tid & 63) == 0) seen[tid >> 6] = mine;
    __syncthreads();
    for (int q = 0; q < 4; ++q)
        for (uint64_t m = uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(seen[q] >> 32))) << 32 |
                          uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(seen[q])));
             m; m &= m - 1) {
            const int at = 64 * q + __ffsll((unsigned long long)m) - 1;
            fuse_voxels<2>(g, depth, coords, first + int64_t(at) * gridDim.x, tid, 256, f, w);
        }
}
// (375900 blocks: 1024 workgroups 17.4 us, 4096 18.6, 8192 22.6; 5370: 8.4, 11.9, 14.4)
constexpr int64_t kFuseGrid = 2048;

static int make_geo(const dn_volume *v, const dn_intrinsics *K, const double *T, Geo &g)
{
    DN_REQUIRE(K && T, "null intrinsics or pose");
    DN_REQUIRE(K->width > 0 && K->height > 0 && K->fx != 0.0 && K->fy != 0.0, "bad intrinsics");
    for (int i = 0; i < 16; ++i) DN_REQUIRE(std::isfinite(T[i]), "non-finite pose");
    g.fx = K->fx; g.fy = K->fy; g.cx = K->cx; g.cy = K->cy;
    for (int i = 0; i < 16; ++i) g.T[i] = T[i];
    g.s = v->prm.voxel_size; g.mu = v->prm.mu; g.maxd = v->prm.max_depth;
    g.W = K->width; g.H = K->height;
    return DN_OK;
}

// ------------------------------------------------------------------ laser
// Laser range data (Section III-A: the projective update extends to laser
// sensors by updating only the voxels along each ray from the sensor to mu
// behind the observed surface).  A return is a point p in the sensor frame
// (T: sensor -> world), range r = |p|, valid iff finite, 0 < r <= max_depth,
// direction d = p / r; the point at range rho is
// ((T_i0 (rho d_x) + T_i1 (rho d_y)) + T_i2 (rho d_z)) + T_i3.
//   Allocation: the blocks met by the band rho in [max(r - mu, 1e-3), r + mu].
//   Fusion: the voxels met by rho in [0, r + mu] in allocated blocks with
//   eta = r - (c - o) . D >= -mu give psi = min(1, eta / mu); one scan's
//   observations are applied together, f <- (w f + sum psi) / (w + k),
//   w <- w + k, the sum in fixed point on maps of up to kAccumBlocks blocks
//   (LaserSums), else in float64 (a segmented reduction over the observations
//   sorted by voxel).
struct LGeo {
    double T[16];
    double s, mu, maxd;
};

__device__ inline bool laser_ray(const float *p, double maxd, double &r, double d[3])
{
    if (!(isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]))) return false;
    const double x = p[0], y = p[1], z = p[2];
    const double rr = sqrt((x * x + y * y) + z * z);
    if (!(rr > 0.0 && rr <= maxd)) return false;
    r = rr;
    d[0] = x / rr; d[1] = y / rr; d[2] = z / rr;
    return true;
}

__device__ inline void ray_point(const double *T, const double d[3], double rho, double out[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
        out[i] = ((T[4 * i + 0] * (rho * d[0]) + T[4 * i + 1] * (rho * d[1])) + T[4 * i + 2] * (rho * d[2])) +
                 T[4 * i + 3];
}

template <class Emit>
__device__ int64_t laser_band(const LGeo &g, const float *p, Emit emit)
{
    double r, d[3], pa[3], pb[3], a[3], b[3];
    if (!laser_ray(p, g.maxd, r, d)) return 0;
    double r0 = r - g.mu;
    if (r0 < 1e-3) r0 = 1e-3;
    ray_point(g.T, d, r0, pa);
    ray_point(g.T, d, r + g.mu, pb);
    const double bs = 8.0 * g.s;
#pragma unroll
    for (int i = 0; i < 3; ++i) { a[i] = pa[i] / bs; b[i] = pb[i] / bs; }
    return walk_segment(a, b, 1e9, emit);
}

struct LaserBand {
    LGeo g;
    const float *pts;
    template <class Emit> __device__ int64_t operator()(int64_t i, Emit emit) const
    {
        return laser_band(g, pts + 3 * i, [&](int64_t, int32_t x, int32_t y, int32_t z) { emit(pack_key(x, y, z)); });
    }
};

// The observations of one return: emit(j, voxel index, psi) for each visited
// voxel of an allocated block with eta >= -mu; returns their number.
template <class Emit>
__device__ int64_t laser_obs(const LGeo &g, const float *p, const int4 *slots, int64_t nslots, uint32_t cap,
                             Emit emit)
{
    double r, d[3], pa[3], pb[3], a[3], b[3], D[3];
    if (!laser_ray(p, g.maxd, r, d)) return 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) D[i] = (g.T[4 * i + 0] * d[0] + g.T[4 * i + 1] * d[1]) + g.T[4 * i + 2] * d[2];
    ray_point(g.T, d, 0.0, pa);
    ray_point(g.T, d, r + g.mu, pb);
#pragma unroll
    for (int i = 0; i < 3; ++i) { a[i] = pa[i] / g.s; b[i] = pb[i] / g.s; }
    int64_t m = 0;
    int32_t kb[3] = {INT32_MIN, 0, 0};
    int32_t id = -1;
    walk_segment(a, b, 1e9, [&](int64_t, int32_t x, int32_t y, int32_t z) {
        const int32_t bx = x >> 3, by = y >> 3, bz = z >> 3;   // floor division
        if (bx != kb[0] || by != kb[1] || bz != kb[2]) {
            kb[0] = bx; kb[1] = by; kb[2] = bz;
            id = hash_lookup(slots, nslots, cap, bx, by, bz);
        }
        if (id < 0) return;
        const double gg[3] = {double(x), double(y), double(z)};
        double rho = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) rho += ((gg[i] + 0.5) * g.s - g.T[4 * i + 3]) * D[i];
        const double eta = r - rho;
        if (eta < -g.mu) return;
        double psi = eta / g.mu;
        if (psi > 1.0) psi = 1.0;
        const int64_t v = int64_t(id) * kBlockVox + ((x - 8 * bx) + 8 * (y - 8 * by) + 64 * (z - 8 * bz));
        emit(m, v, psi);
        ++m;
    });
    return m;
}

__global__ void k_laser_obs_count(LGeo g, const float *__restrict__ pts, int64_t n, const int4 *__restrict__ slots,
                                  int64_t nslots, uint32_t cap, int64_t *__restrict__ counts)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    counts[i] = laser_obs(g, pts + 3 * i, slots, nslots, cap, [](int64_t, int64_t, double) {});
}

__global__ void k_laser_obs_emit(LGeo g, const float *__restrict__ pts, int64_t n, const int4 *__restrict__ slots,
                                 int64_t nslots, uint32_t cap, const int64_t *__restrict__ offsets,
                                 uint32_t *__restrict__ keys, double *__restrict__ vals, int64_t total)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t base = offsets[i];
    laser_obs(g, pts + 3 * i, slots, nslots, cap, [&](int64_t j, int64_t v, double psi) {
        if (base + j < total) {
            keys[base + j] = uint32_t(v);
            vals[base + j] = psi;
        }
    });
}

// Fusion of a scan into a map of up to kAccumBlocks blocks: every voxel has
// an accumulator in the scratch: a count of its observations and the sum of
// 1 - psi over those in the band (in free space psi = 1), in fixed point, so
// that the result does not depend on the order of the additions (LaserSums).
// Bound by latency along each ray: one lane walks a ray
// and looks a block up when it enters it, in LDS, where a map of up to
// kSeenAll blocks lies whole (a larger one's table keeps the blocks that its
// workgroup met: neighbouring rays pass the same ones, but each costs one
// wait for memory), and lanes in the same voxel add to its count once.
// Against two walks with a lookup in memory per block and a sort of all
// observations, 65536 returns into 1400 blocks: 0.90 ms a scan before
// (allocation included), 0.22 ms now.
constexpr int64_t kAccumBlocks = 16384;

// The two words of a voxel's accumulator.  `fine` is the sum with F bits after
// the point, modulo 2^64; `coarse` the count in its upper b bits (n < 2^b
// returns) and below it the sum of the same terms cut to q bits after the
// point.  Each term, in [0, 2], loses less than one unit there, so the whole
// sum is the coarse one plus less than n units, and `fine` tells how much: it
// is exact.  With 60 bits (56 for the largest scans) a term keeps the digits
// of psi in float64 up to the rounding of the distances; one word of 63 - b
// bits lost them (f near the surface had 3 of float32's 7 digits after a scan
// of 10^6 returns), and was 4 us of 130 quicker for 65536 returns.  Coarse
// parts are added up over a run of lanes first: an atomic per observation for
// them cost 4 us more.
// (Sums of mu - eta, divided by mu once per voxel, take 132 us, but round f the
// other way now and then, as psi is not rounded by itself.)
struct LaserSums {
    int b, q, F;
    static constexpr int kMaxB = 23;
    explicit LaserSums(int64_t n)
    {
        b = 1;
        while ((n >> b) > 0) ++b;
        F = std::min(60, 125 - 3 * b);      // n units of the coarse sum are less than 2^63 fine ones
        q = std::min(24, 63 - 2 * b);       // n terms (each up to 2) of the coarse sum fit its 64 - b bits, 64 of them 32
    }
    // (not negative: psi < 1)
    __device__ __forceinline__ unsigned long long term(double psi) const
    {
        return (1ull << F) - (unsigned long long)(int64_t)(psi * double(1ull << F));
    }
    __device__ __forceinline__ uint32_t cut(unsigned long long term) const { return uint32_t(term >> (F - q)); }
    // of up to 64 observations, given the sum of their cut terms
    __device__ __forceinline__ unsigned long long coarse(unsigned count, uint32_t cuts) const
    {
        return (unsigned long long)count << (64 - b) | cuts;
    }
    __device__ __forceinline__ uint32_t count(unsigned long long c) const { return uint32_t(c >> (64 - b)); }
    // the sum of psi over all observations
    __device__ __forceinline__ double psi(unsigned long long c, unsigned long long fine) const
    {
        const unsigned long long cut = c & ((1ull << (64 - b)) - 1ull);
        const int64_t a = (int64_t(count(c)) << q) - int64_t(cut);          // at least the sum, in 2^-q
        const int64_t less = int64_t(fine - (cut << (F - q)));              // by that, in 2^-F
        const int64_t top = int64_t(1) << (62 - (F - q));
        const double unit = 1.0 / double(1ull << F);
        if (a < top && a > -top) return double((a << (F - q)) - less) * unit;
        return double(a) / double(1ull << q) - double(less) * unit;
    }
};
constexpr int kSeen = 8192, kSeenAll = kSeen / 2;   // entries of the table
constexpr double kSeenRange = 500.0;                // blocks from the sensor that its tags tell apart

// Inclusive prefix sums over the lanes of a wave, without LDS.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // from the lane 1, 2, 4 and 8 before, in rows of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // the row before, to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // the half before, to rows 2 and 3
    return v;
}

// (sums: coarse and fine word of each voxel)
__global__ void k_laser_clear(ulonglong2 *__restrict__ sums, int64_t nvox, int64_t *__restrict__ total)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;   // 4 voxels
    if (i == 0) *total = 0;
    if (4 * i >= nvox) return;
    for (int k = 0; k < 4; ++k) sums[k * (nvox / 4) + i] = make_ulonglong2(0, 0);
}

template <bool kAll>
__global__ __launch_bounds__(256) void k_laser_accumulate(LGeo g, const float *__restrict__ pts, int64_t n,
                                                          const int4 *__restrict__ slots, int64_t nslots, uint32_t cap,
                                                          const int4 *__restrict__ coords, int nb, LaserSums ls,
                                                          ulonglong2 *__restrict__ sums, int64_t *__restrict__ total)
{
    __shared__ unsigned long long seen[kSeen];      // block relative to the sensor's (high half) and its id
    __shared__ unsigned long long s_total;
    const int tid = threadIdx.x, lane = tid & 63;
    constexpr unsigned long long kNone = ~0ull;
    const int32_t sx = int32_t(floor(g.T[3] / (8.0 * g.s))), sy = int32_t(floor(g.T[7] / (8.0 * g.s))),
                  sz = int32_t(floor(g.T[11] / (8.0 * g.s)));
    // the block's tag, ~0 out of the table's range; its place in the table
    auto tag_of = [&](int32_t bx, int32_t by, int32_t bz) {
        const uint32_t rx = uint32_t(bx) - uint32_t(sx) + 512u, ry = uint32_t(by) - uint32_t(sy) + 512u,
                       rz = uint32_t(bz) - uint32_t(sz) + 512u;
        return (rx | ry | rz) < 1024u ? rx << 20 | ry << 10 | rz : ~0u;
    };
    auto place = [](uint32_t tag) { return (tag * 2654435761u) >> 19; };
    static_assert(kSeen == 1 << 13, "place() gives 13 bits");
    for (int k = tid; k < kSeen; k += 256) seen[k] = kNone;
    if (tid == 0) s_total = 0;
    __syncthreads();
    if constexpr (kAll) {
        for (int k = tid; k < nb; k += 256) {
            const int4 c = coords[k];
            const uint32_t tag = tag_of(c.x, c.y, c.z);
            if (tag == ~0u) continue;
            for (uint32_t h = place(tag);; h = (h + 1) & (kSeen - 1))
                if (atomicCAS(seen + h, kNone, (unsigned long long)tag << 32 | uint32_t(k)) == kNone) break;
        }
        __syncthreads();
    }
    const int64_t i = int64_t(blockIdx.x) * 256 + tid;
    double r = 0.0, d[3], pa[3], pb[3], a[3], b[3], D[3] = {0.0, 0.0, 0.0};
    Walk w{};
    bool alive = i < n && laser_ray(pts + 3 * i, g.maxd, r, d);
    if (alive) {
#pragma unroll
        for (int q = 0; q < 3; ++q) D[q] = (g.T[4 * q + 0] * d[0] + g.T[4 * q + 1] * d[1]) + g.T[4 * q + 2] * d[2];
        ray_point(g.T, d, 0.0, pa);
        ray_point(g.T, d, r + g.mu, pb);
#pragma unroll
        for (int q = 0; q < 3; ++q) { a[q] = pa[q] / g.s; b[q] = pb[q] / g.s; }
        alive = w.start(a, b, 1e9);
    }
    // gridDim.y workgroups share a ray by step numbers; each walks up to its own
    int steps = 0;
    if (alive) {
        const int64_t all = w.cells();
        const int64_t first = all * blockIdx.y / gridDim.y, end = all * (blockIdx.y + 1) / gridDim.y;
        steps = int(end - first);
        for (int64_t k = 0; k < first; ++k) w.next();
        alive = steps > 0;
    }
    // Up to the parameter `safe` a cell's centre, at most 0.87 s from the
    // ray, is more than mu in front of the surface: psi = 1 without its
    // distance.  At the parameter t the ray is t (r + mu) |D|^2 along D, and
    // |D| is 1 for a rigid pose only.
    const double dd = (D[0] * D[0] + D[1] * D[1]) + D[2] * D[2];
    const double safe = (r - g.mu - 2.0 * g.s * fmax(1.0, sqrt(dd))) / ((r + g.mu) * dd);
    double now = 2.0;                    // the parameter at which the ray entered the cell (2: unknown)
    int32_t id = -1, moved = ~7;         // ~7: not in this block yet
    unsigned mine = 0;
    while (__any(alive)) {
        uint32_t vox = 0, cut = 0;
        bool hit = false;
        if (alive) {
            if ((moved & ~7) != 0) {
                const int32_t bx = w.k[0] >> 3, by = w.k[1] >> 3, bz = w.k[2] >> 3;   // floor division
                const uint32_t tag = tag_of(bx, by, bz);
                if constexpr (kAll) {
                    id = -1;
                    for (uint32_t h = place(tag);; h = (h + 1) & (kSeen - 1)) {
                        const unsigned long long e = seen[h];
                        if (uint32_t(e >> 32) == tag) id = int32_t(uint32_t(e));
                        if (e == kNone || id >= 0) break;
                    }
                } else if (tag != ~0u) {
                    // (waves replace each other's entries at any time: an
                    // entry's two halves are read and written as one)
                    unsigned long long *at = seen + place(tag);
                    const unsigned long long e =
                        __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (uint32_t(e >> 32) == tag) {
                        id = int32_t(uint32_t(e));
                    } else {
                        id = hash_lookup(slots, nslots, cap, bx, by, bz);
                        __hip_atomic_store(at, (unsigned long long)tag << 32 | uint32_t(id), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                } else {
                    id = hash_lookup(slots, nslots, cap, bx, by, bz);
                }
            }
            if (id >= 0) {
                vox = uint32_t(id) * uint32_t(kBlockVox) + uint32_t((w.k[0] & 7) + 8 * (w.k[1] & 7) + 64 * (w.k[2] & 7));
                hit = now < safe;
                if (!hit) {
                    double rho = 0.0;
#pragma unroll
                    for (int q = 0; q < 3; ++q) rho += ((double(w.k[q]) + 0.5) * g.s - g.T[4 * q + 3]) * D[q];
                    const double eta = r - rho;
                    hit = eta >= g.mu;
                    if (!hit && eta >= -g.mu) {
                        const unsigned long long term = ls.term(eta / g.mu);
                        atomicAdd(&sums[vox].y, term);
                        cut = ls.cut(term);
                        hit = true;
                    }
                }
                if (hit) ++mine;
            }
            alive = w.next(now, moved) && --steps > 0;
        }
        // one addition per run of neighbouring lanes in the same voxel
        const uint64_t hits = __ballot(hit);
        if (hits == 0) continue;
        const uint32_t before = uint32_t(__builtin_amdgcn_update_dpp(0, int(vox), 0x138, 0xF, 0xF, false));   // lane - 1
        const bool head = hit && (lane == 0 || !((hits >> (lane - 1)) & 1ull) || before != vox);
        const uint64_t ends = (__ballot(head) | ~hits) >> lane >> 1;      // where a run after this lane ends
        const int len = ends ? __ffsll((unsigned long long)ends) : 64 - lane;
        uint32_t run = 0;
        if (__any(cut != 0)) {
            const uint32_t to = wave_prefix(cut);
            run = __shfl(to, lane + len - 1, 64) - (to - cut);
        }
        if (head) atomicAdd(&sums[vox].x, ls.coarse(unsigned(len), run));
    }
    if (mine) atomicAdd(&s_total, (unsigned long long)mine);
    __syncthreads();
    if (tid == 0 && s_total) atomicAdd(reinterpret_cast<unsigned long long *>(total), s_total);
}

// Apply the accumulators (unless the scan has more observations than the
// volume takes) and hand their number to the host.
__global__ void k_laser_apply_sums(const ulonglong2 *__restrict__ sums, int64_t nvox, LaserSums ls,
                                   const int64_t *__restrict__ total, int64_t most, int64_t *host,
                                   float *__restrict__ f, float *__restrict__ w)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t m = *total;
    if (i == 0) *host = m;
    if (m > most || i >= nvox) return;
    const ulonglong2 q = sums[i];
    const uint32_t c = ls.count(q.x);
    if (c == 0) return;
    const double w0 = w[i], wn = w0 + double(c);
    f[i] = float((w0 * double(f[i]) + ls.psi(q.x, q.y)) / wn);
    w[i] = float(wn);
}

// One scan's update of each observed voxel, from the per-voxel sums and
// counts of its observations (a segmented reduction of the sorted list).
__global__ void k_laser_apply(const uint32_t *__restrict__ uniq, const double *__restrict__ sums,
                              const uint32_t *__restrict__ counts, const uint32_t *__restrict__ nruns, int64_t m,
                              float *__restrict__ f, float *__restrict__ w)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= m || i >= int64_t(*nruns)) return;
    const uint32_t v = uniq[i];
    const double w0 = w[v];
    const double wn = w0 + double(counts[i]);
    f[v] = float((w0 * double(f[v]) + sums[i]) / wn);
    w[v] = float(wn);
}

static int make_lgeo(const dn_volume *v, const double *T, LGeo &g)
{
    DN_REQUIRE(T, "null pose");
    for (int i = 0; i < 16; ++i) DN_REQUIRE(std::isfinite(T[i]), "non-finite pose");
    for (int i = 0; i < 16; ++i) g.T[i] = T[i];
    g.s = v->prm.voxel_size; g.mu = v->prm.mu; g.maxd = v->prm.max_depth;
    return DN_OK;
}

// Scratch of one laser fusion call: per-return counts and offsets, the
// observation lists (voxel key, psi) and their sorted copies, the per-voxel
// counts and the rocprim storage.
struct LaserScratch {
    int64_t *counts, *offs;
    uint32_t *k_in, *k_out, *counts32, *nruns;
    double *v_in, *v_out;
    void *tmp;
    size_t tmp_bytes;
};
static LaserScratch carve_laser(Bump &b, int64_t n, int64_t m)
{
    LaserScratch x;
    x.counts = b.take<int64_t>(size_t(n));
    x.offs = b.take<int64_t>(size_t(n) + 1);
    x.k_in = b.take<uint32_t>(size_t(m));
    x.k_out = b.take<uint32_t>(size_t(m));
    x.counts32 = b.take<uint32_t>(size_t(m));
    x.nruns = b.take<uint32_t>(1);
    x.v_in = b.take<double>(size_t(m));
    x.v_out = b.take<double>(size_t(m));
    x.tmp_bytes = std::max(std::max(tmp_light(size_t(n)), tmp_light(size_t(m))), tmp_sort(size_t(m), 12));
    x.tmp = b.take<char>(x.tmp_bytes);
    return x;
}

struct CandScratch {
    uint64_t *sorted, *uniq;
    void *tmp;
    size_t tmp_bytes;
};
static CandScratch carve_cand(Bump &b, int64_t n)
{
    CandScratch x;
    x.sorted = b.take<uint64_t>(size_t(n));
    x.uniq = b.take<uint64_t>(size_t(n));
    x.tmp_bytes = std::max(tmp_sort(size_t(n), 8), tmp_light(size_t(n)));
    x.tmp = b.take<char>(x.tmp_bytes);
    return x;
}

size_t candidates_scratch(int64_t n_cand)
{
    Bump b(nullptr, 0);
    carve_cand(b, n_cand);
    return b.off;
}

// The ascending distinct keys of the last candidate list, built in the
// scratch on request (*uniq points into it until the next call uses it).
int build_candidates(dn_volume *v, uint64_t **uniq, int64_t *n_uniq)
{
    *uniq = nullptr;
    *n_uniq = 0;
    const int64_t n = v->cand_n;
    if (n == 0) return DN_OK;
    hipStream_t st = v->stream;
    Bump bump(v->scratch, v->scratch_bytes);
    CandScratch x = carve_cand(bump, n);
    if (!bump.fits()) { set_error("scratch too small for the candidate list"); return DN_E_CAPACITY; }
    int64_t *d_n = v->misc + 3;
    size_t tbytes = x.tmp_bytes;
    DN_HIP(rocprim::radix_sort_keys(x.tmp, tbytes, v->cand, x.sorted, size_t(n), 0, 63, st));
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::unique(x.tmp, tbytes, x.sorted, x.uniq, d_n, size_t(n), rocprim::equal_to<uint64_t>(), st));
    int rc = read_back(v, d_n, sizeof(int64_t));
    if (rc) return rc;
    *uniq = x.uniq;
    *n_uniq = v->host_stage[0];
    return DN_OK;
}

// Placement of everything a volume keeps in its arena (base == nullptr:
// measure only).  Returns the arena size; with v != nullptr the volume's
// pointers are set.
static size_t volume_layout(const dn_volume_params &p, void *base, dn_volume *v)
{
    const size_t mb = size_t(p.max_blocks), vox = mb * kBlockVox;
    const size_t slots = (size_t(1) << p.hash_cap_log2) + size_t(p.hash_tail);
    Bump b(base, ~size_t(0));
    int32_t *coords = b.take<int32_t>(mb * 4);
    uint64_t *keys = b.take<uint64_t>(mb);
    int32_t *h0 = b.take<int32_t>(slots * 4);
    int32_t *h1 = b.take<int32_t>(slots * 4);
    uint32_t *oh0 = b.take<uint32_t>(mb), *oh1 = b.take<uint32_t>(mb);
    int32_t *oi0 = b.take<int32_t>(mb), *oi1 = b.take<int32_t>(mb);
    uint64_t *nset = b.take<uint64_t>(kNewSet), *nkey = b.take<uint64_t>(kMaxNew), *skey = b.take<uint64_t>(kMaxNew);
    uint32_t *nhome = b.take<uint32_t>(kMaxNew), *nslot = b.take<uint32_t>(kMaxNew), *shome = b.take<uint32_t>(kMaxNew);
    int32_t *sid = b.take<int32_t>(kMaxNew);
    int32_t *nbr = b.take<int32_t>(mb * kNbr);
    float *f = b.take<float>(vox);
    float *w = b.take<float>(vox);
    float *u = b.take<float>(vox);
    float *ub0 = b.take<float>(vox);
    float *ub1 = b.take<float>(vox);
    float *p0 = b.take<float>(vox * 3);
    float *p1 = b.take<float>(vox * 3);
    uint8_t *emask = b.take<uint8_t>(vox);
    uint32_t *em4 = b.take<uint32_t>(mb * 64);
    int32_t *order = b.take<int32_t>(mb);
    double *partials = b.take<double>(mb * 2 + 2 * ((mb + 1023) / 1024 + 1) * 2 + 8);
    int64_t *misc = b.take<int64_t>(32);
    uint64_t *cand = b.take<uint64_t>(size_t(p.max_candidates));
    void *u16 = nullptr, *ub16a = nullptr, *ub16b = nullptr, *p16a = nullptr, *p16b = nullptr;
    if (p.state16) {
        u16 = b.take<uint16_t>(vox);
        ub16a = b.take<uint16_t>(vox);
        ub16b = b.take<uint16_t>(vox);
        p16a = b.take<uint16_t>(vox * 3);
        p16b = b.take<uint16_t>(vox * 3);
    }
    // scratch: the largest of the per-call needs
    size_t need = 0;
    auto upd = [&](size_t n) { need = std::max(need, n); };
    {
        Bump m(nullptr, 0);
        carve_insert(m, std::max<int64_t>(p.max_candidates, 1), p.max_blocks);
        upd(m.off);
    }
    upd(candidates_scratch(std::max<int64_t>(p.max_candidates, 1)));
    upd(masks_scratch(p.max_blocks));
    upd(extract_scratch(p.max_blocks));
    if (p.max_observations > 0) {
        Bump m(nullptr, 0);
        carve_laser(m, p.max_points, p.max_observations);
        upd(m.off);
        // the accumulators (16 bytes a voxel) of every map that three quarters of
        // them fit beside the other needs
        const size_t blocks = std::min({mb, size_t(kAccumBlocks), need / (12 * kBlockVox)});
        upd(blocks * kBlockVox * 16);
    }
    char *scratch = b.take<char>(need);
    if (v) {
        v->coords = coords; v->keys = keys; v->hash[0] = h0; v->hash[1] = h1; v->nbr = nbr;
        v->f = f; v->w = w; v->u = u; v->ubar[0] = ub0; v->ubar[1] = ub1; v->p[0] = p0; v->p[1] = p1;
        v->emask = emask; v->em4 = em4; v->order = order; v->partials = partials; v->misc = misc;
        v->cand = cand;
        v->hord_home[0] = oh0; v->hord_home[1] = oh1; v->hord_ids[0] = oi0; v->hord_ids[1] = oi1;
        v->new_set = nset; v->new_key = nkey; v->sort_key = skey; v->new_home = nhome; v->new_slot = nslot;
        v->sort_home = shome; v->sort_id = sid;
        v->u16 = u16; v->ubar16[0] = ub16a; v->ubar16[1] = ub16b; v->p16[0] = p16a; v->p16[1] = p16b;
        v->scratch = scratch;
        v->scratch_bytes = need;
    }
    return (b.off + 255) & ~size_t(255);
}

static bool params_ok(const dn_volume_params *p)
{
    return p && p->voxel_size > 0 && p->mu > 0 && p->max_depth > 0 && p->max_blocks >= 1 &&
           p->hash_cap_log2 >= 4 && p->hash_cap_log2 <= 30 && p->hash_tail >= 0 &&
           (p->state16 == 0 || p->state16 == 1) && p->max_points >= 0 && p->max_candidates >= 0 &&
           p->max_observations >= 0 && p->max_points < (int64_t(1) << 31) &&
           p->max_candidates < (int64_t(1) << 40) && p->max_observations < (int64_t(1) << 32) &&
           std::isfinite(p->voxel_size) && std::isfinite(p->mu) && std::isfinite(p->max_depth);
}

// The rocprim calls' own storage figures at the largest sizes this volume
// can ask for, against the bounds its scratch was sized with.
static int verify_tmp_bounds(dn_volume *v)
{
    const dn_volume_params &p = v->prm;
    hipStream_t st = v->stream;
    const size_t nc = size_t(std::max<int64_t>(p.max_candidates, 1)), mb = size_t(p.max_blocks);
    const size_t np = size_t(std::max<int64_t>(p.max_points, 1)), no = size_t(std::max<int64_t>(p.max_observations, 1));
    struct Q { const char *what; size_t need, have; };
    std::vector<Q> q;
    size_t t = 0;
    int32_t *i32 = nullptr; int64_t *i64 = nullptr; uint64_t *u64 = nullptr; uint32_t *u32 = nullptr;
    uint8_t *u8 = nullptr; double *f64 = nullptr;
    DN_HIP(rocprim::select(nullptr, t, u64, u8, u64, i64, nc, st));
    q.push_back({"candidate selection", t, tmp_light(nc)});
    t = 0;
    DN_HIP(rocprim::radix_sort_keys(nullptr, t, u64, u64, nc, 0, 63, st));
    q.push_back({"candidate sort", t, tmp_sort(nc, 8)});
    t = 0;
    DN_HIP(rocprim::unique(nullptr, t, u64, u64, i64, nc, rocprim::equal_to<uint64_t>(), st));
    q.push_back({"candidate unique", t, tmp_light(nc)});
    t = 0;
    DN_HIP(rocprim::radix_sort_pairs(nullptr, t, u64, u64, i32, i32, nc, 0, 63, st));
    q.push_back({"candidate sort with positions", t, tmp_sort(nc, 12)});
    t = 0;
    DN_HIP(rocprim::select(nullptr, t, i32, u8, i32, i64, nc, st));
    q.push_back({"first-occurrence selection", t, tmp_light(nc)});
    t = 0;
    DN_HIP(rocprim::radix_sort_keys(nullptr, t, i32, i32, nc, 0, 31, st));
    q.push_back({"position sort", t, tmp_sort(nc, 12)});
    t = 0;
    DN_HIP(rocprim::radix_sort_pairs(nullptr, t, u64, u64, i32, i32, mb, 0, 63, st));
    q.push_back({"key sort", t, tmp_sort(mb, 12)});
    t = 0;
    DN_HIP(rocprim::radix_sort_pairs(nullptr, t, u32, u32, i32, i32, mb, 0, 31, st));
    q.push_back({"bucket sort", t, tmp_sort(mb, 8)});
    t = 0;
    DN_HIP(rocprim::inclusive_scan(nullptr, t, i64, i64, mb, rocprim::maximum<int64_t>(), st));
    q.push_back({"slot scan", t, tmp_light(mb)});
    t = 0;
    DN_HIP(rocprim::exclusive_scan(nullptr, t, i64, i64, int64_t(0), mb + 1, rocprim::plus<int64_t>(), st));
    q.push_back({"extraction scan", t, tmp_light(mb + 1)});
    if (p.max_observations > 0) {
        t = 0;
        DN_HIP(rocprim::exclusive_scan(nullptr, t, i64, i64, int64_t(0), np, rocprim::plus<int64_t>(), st));
        q.push_back({"return scan", t, tmp_light(np)});
        t = 0;
        DN_HIP(rocprim::radix_sort_pairs(nullptr, t, u32, u32, f64, f64, no, 0, 32, st));
        q.push_back({"observation sort", t, tmp_sort(no, 12)});
        t = 0;
        DN_HIP(rocprim::reduce_by_key(nullptr, t, u32, f64, no, u32, f64, u32, rocprim::plus<double>(),
                                      rocprim::equal_to<uint32_t>(), st));
        q.push_back({"observation sums", t, tmp_light(no)});
        t = 0;
        DN_HIP(rocprim::run_length_encode(nullptr, t, u32, no, u32, u32, u32, st));
        q.push_back({"observation counts", t, tmp_light(no)});
    }
    for (const Q &e : q)
        if (e.need > e.have) {
            set_error("rocprim %s needs %zu bytes of storage, the scratch bound is %zu", e.what, e.need, e.have);
            return DN_E_CAPACITY;
        }
    return DN_OK;
}

// Allocation for n points (depth pixels or laser returns): walk their
// bands, check the limits, turn the new keys into blocks.  A frame with more
// new keys than k_band lists, or a pool past kMergeBlocks, takes the general
// insertion of the listed keys.
template <class Band> static int alloc_points(dn_volume *v, int64_t n, const Band &band, int32_t *n_new_out)
{
    if (n_new_out) *n_new_out = 0;
    v->cand_n = 0;
    if (n == 0) return DN_OK;
    if (n > v->prm.max_points) {
        set_error("%lld points exceed the volume's max_points %lld", (long long)n, (long long)v->prm.max_points);
        return DN_E_CAPACITY;
    }
    hipStream_t st = v->stream;
    BandOut o{v->cand, v->prm.max_candidates, v->new_set, v->new_key, v->new_home, v->new_slot, v->misc, report(v)};
    const int4 *slots = reinterpret_cast<const int4 *>(v->hash[v->cur_hash]);
    if (n <= kBandSmall)
        hipLaunchKernelGGL((k_band<Band, 256>), dim3(grid1(n, 256)), dim3(256), 0, st, band, n, slots, v->hash_slots,
                           v->hash_cap, o);
    else
        hipLaunchKernelGGL((k_band<Band, 1024>), dim3(grid1(n, 1024)), dim3(1024), 0, st, band, n, slots,
                           v->hash_slots, v->hash_cap, o);
    DN_HIP(hipGetLastError());
    int rc = fetch_report(v, 5);
    if (rc) return rc;
    const int64_t total = v->host_stage[0], listed = v->host_stage[1], n_new = v->host_stage[2], end = v->host_stage[4];
    const bool full = v->host_stage[3] != 0;
    if (total > v->prm.max_candidates) {
        if ((n_new > 0 || full) && (rc = reset_new_set(v))) return rc;
        set_error("%lld band cells exceed the volume's max_candidates %lld", (long long)total,
                  (long long)v->prm.max_candidates);
        return DN_E_CAPACITY;
    }
    v->cand_n = listed;
    if (n_new == 0 && !full) return DN_OK;
    if (!full && v->nb + n_new <= v->cap_blocks && v->nb + n_new <= kMergeBlocks)
        return insert_listed(v, n_new, end, n_new_out);
    if ((rc = reset_new_set(v))) return rc;
    return insert_packed(v, v->cand, listed, n_new_out);
}

}  // namespace dn

using namespace dn;

// ================================================================== C ABI
extern "C" {

const char *dn_last_error(void) { return g_err; }

size_t dn_volume_bytes(const dn_volume_params *p)
{
    if (!params_ok(p)) return 0;
    return volume_layout(*p, nullptr, nullptr);
}

int dn_volume_create(const dn_volume_params *p, void *arena, size_t arena_bytes, void *hip_stream, dn_volume **out)
{
    DN_REQUIRE(p && out, "null argument");
    *out = nullptr;
    DN_REQUIRE(p->voxel_size > 0 && p->mu > 0 && p->max_depth > 0, "voxel_size, mu, max_depth must be > 0");
    DN_REQUIRE(p->max_blocks >= 1, "max_blocks must be >= 1");
    DN_REQUIRE(p->hash_cap_log2 >= 4 && p->hash_cap_log2 <= 30, "hash_cap_log2 must be in [4, 30]");
    DN_REQUIRE(p->hash_tail >= 0, "hash_tail must be >= 0");
    DN_REQUIRE(params_ok(p), "bad limits (state16 0/1; max_points, max_candidates, max_observations >= 0 and in range)");
    DN_REQUIRE(arena, "null arena");
    DN_REQUIRE((reinterpret_cast<uintptr_t>(arena) & 255) == 0, "the arena must be 256-byte aligned");
    const size_t need = volume_layout(*p, nullptr, nullptr);
    if (arena_bytes < need) {
        set_error("arena of %zu bytes is short: the volume needs %zu (dn_volume_bytes)", arena_bytes, need);
        return DN_E_CAPACITY;
    }
    dn_volume *v = new dn_volume();
    v->prm = *p;
    v->stream = static_cast<hipStream_t>(hip_stream);
    v->cap_blocks = p->max_blocks;
    v->hash_cap = 1u << p->hash_cap_log2;
    v->hash_slots = int64_t(v->hash_cap) + p->hash_tail;
    v->arena = arena;
    v->arena_bytes = arena_bytes;
    volume_layout(*p, arena, v);
    auto fail = [&](int rc) { delete v; return rc; };
    if (hipGetDevice(&v->device) != hipSuccess) { set_error("hipGetDevice failed"); return fail(DN_E_DEVICE); }
    int rc = verify_tmp_bounds(v);
    if (rc) return fail(rc);
    hipStream_t st = v->stream;
    // (a block's fields are zeroed when it is allocated)
    hipLaunchKernelGGL(k_init_misc, dim3(grid1(kNewSet)), dim3(256), 0, st, v->misc, v->new_set);
    hipLaunchKernelGGL(k_fill_empty, dim3(grid1(v->hash_slots)), dim3(256), 0, st,
                       reinterpret_cast<int4 *>(v->hash[0]), v->hash_slots);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
        set_error("initialisation failed");
        return fail(DN_E_DEVICE);
    }
    *out = v;
    return DN_OK;
}

void dn_volume_destroy(dn_volume *v)
{
    if (!v) return;
    (void)hipStreamSynchronize(v->stream);
    delete v;
}

int dn_volume_clear(dn_volume *v)
{
    DN_REQUIRE(v, "null volume");
    hipStream_t st = v->stream;
    hipLaunchKernelGGL(k_fill_empty, dim3(grid1(v->hash_slots)), dim3(256), 0, st,
                       reinterpret_cast<int4 *>(v->hash[v->cur_hash]), v->hash_slots);
    DN_HIP(hipGetLastError());
    v->nb = 0;
    v->p_off_zero = true;
    v->nb_state = 0;
    v->emask_nb = -1;
    v->cand_n = 0;
    v->state_storage = DN_F32;
    return DN_OK;
}

int dn_set_stream(dn_volume *v, void *hip_stream)
{
    DN_REQUIRE(v, "null volume");
    v->stream = static_cast<hipStream_t>(hip_stream);
    return DN_OK;
}

int dn_set_report_buffer(dn_volume *v, void *pinned, size_t bytes)
{
    DN_REQUIRE(v, "null volume");
    DN_HIP(hipStreamSynchronize(v->stream));
    if (!pinned) {
        v->report = v->report_host = nullptr;
        return DN_OK;
    }
    DN_REQUIRE(bytes >= DN_REPORT_BYTES && (reinterpret_cast<uintptr_t>(pinned) & 7) == 0,
               "the report buffer must hold DN_REPORT_BYTES, 8-byte aligned");
    void *dev = nullptr;
    if (hipHostGetDevicePointer(&dev, pinned, 0) != hipSuccess || !dev) {
        (void)hipGetLastError();
        set_error("the report buffer is not pinned host memory");
        return DN_E_INVALID;
    }
    v->report = static_cast<int64_t *>(dev);
    v->report_host = static_cast<int64_t *>(pinned);
    return DN_OK;
}

int64_t dn_num_blocks(const dn_volume *v) { return v ? v->nb : -1; }

int dn_sync(dn_volume *v)
{
    DN_REQUIRE(v, "null volume");
    return volume_sync(v);
}

int dn_alloc_blocks(dn_volume *v, const float *depth, const dn_intrinsics *K, const double T[16],
                    int32_t *n_new_out)
{
    DN_REQUIRE(v && depth, "null argument");
    Geo g;
    int rc = make_geo(v, K, T, g);
    if (rc) return rc;
    return alloc_points(v, int64_t(g.W) * g.H, DepthBand{g, depth}, n_new_out);
}

static int insert_keys(dn_volume *v, const int32_t *coords, int64_t n, int32_t *n_new_out, bool keep_order)
{
    DN_REQUIRE(v && (coords || n == 0) && n >= 0, "bad argument");
    if (n_new_out) *n_new_out = 0;
    v->cand_n = 0;
    if (n == 0) return DN_OK;
    if (n > v->prm.max_candidates) {
        set_error("%lld keys exceed the volume's max_candidates %lld", (long long)n, (long long)v->prm.max_candidates);
        return DN_E_CAPACITY;
    }
    hipLaunchKernelGGL(k_pack_coords, dim3(grid1(n)), dim3(256), 0, v->stream, coords, n, v->cand);
    DN_HIP(hipGetLastError());
    return insert_packed(v, v->cand, n, n_new_out, keep_order);
}

int dn_insert_blocks(dn_volume *v, const int32_t *coords, int64_t n, int32_t *n_new_out)
{
    return insert_keys(v, coords, n, n_new_out, false);
}

int dn_insert_blocks_ordered(dn_volume *v, const int32_t *coords, int64_t n, int32_t *n_new_out)
{
    DN_REQUIRE(n < (int64_t(1) << 31), "at most 2^31 - 1 keys per call");
    return insert_keys(v, coords, n, n_new_out, true);
}

int dn_fuse_depth(dn_volume *v, const float *depth, const dn_intrinsics *K, const double T[16])
{
    DN_REQUIRE(v && depth, "null argument");
    Geo g;
    int rc = make_geo(v, K, T, g);
    if (rc) return rc;
    if (v->nb == 0) return DN_OK;
    const int64_t grid = (std::max(std::min(v->nb, kFuseGrid), (v->nb + 255) / 256) + 7) / 8 * 8;
    hipLaunchKernelGGL(k_fuse, dim3(unsigned(grid)), dim3(256), 0, v->stream, g, depth, v->coords, v->nb, v->f, v->w);
    DN_HIP(hipGetLastError());
    v->emask_nb = -1;
    return DN_OK;
}

int dn_load_fused(dn_volume *v, const float *f, const float *w)
{
    DN_REQUIRE(v && f && w, "null argument");
    if (v->nb == 0) return DN_OK;
    size_t bytes = size_t(v->nb) * kBlockVox * 4;
    DN_HIP(hipMemcpyAsync(v->f, f, bytes, hipMemcpyDeviceToDevice, v->stream));
    DN_HIP(hipMemcpyAsync(v->w, w, bytes, hipMemcpyDeviceToDevice, v->stream));
    v->p_off_zero = false;      // (until a solve starts from p = 0)
    v->emask_nb = -1;
    return DN_OK;
}

int dn_alloc_laser(dn_volume *v, const float *pts, int64_t n, const double T[16], int32_t *n_new_out)
{
    DN_REQUIRE(v && (pts || n == 0) && n >= 0, "bad argument");
    LGeo g;
    int rc = make_lgeo(v, T, g);
    if (rc) return rc;
    return alloc_points(v, n, LaserBand{g, pts}, n_new_out);
}

int dn_fuse_laser(dn_volume *v, const float *pts, int64_t n, const double T[16])
{
    DN_REQUIRE(v && (pts || n == 0) && n >= 0, "bad argument");
    LGeo g;
    int rc = make_lgeo(v, T, g);
    if (rc) return rc;
    if (n == 0 || v->nb == 0) return DN_OK;
    if (n > v->prm.max_points) {
        set_error("%lld returns exceed the volume's max_points %lld", (long long)n, (long long)v->prm.max_points);
        return DN_E_CAPACITY;
    }
    if (v->prm.max_observations <= 0) { set_error("the volume was created without laser observations"); return DN_E_CAPACITY; }
    DN_REQUIRE(v->nb * int64_t(kBlockVox) < (int64_t(1) << 32), "volume too large for 32-bit voxel keys");
    hipStream_t st = v->stream;
    const int4 *slots = reinterpret_cast<const int4 *>(v->hash[v->cur_hash]);
    Bump bump(v->scratch, v->scratch_bytes);
    const int64_t nvox = v->nb * int64_t(kBlockVox);
    ulonglong2 *sums = bump.take<ulonglong2>(size_t(nvox));
    const LaserSums ls(n);
    if (v->nb <= kAccumBlocks && ls.b <= LaserSums::kMaxB && bump.fits()) {
        int64_t *total = v->misc + kMiscObs;
        hipLaunchKernelGGL(k_laser_clear, dim3(grid1(nvox / 4)), dim3(256), 0, st, sums, nvox, total);
        // (the whole map in the table: every block that a ray can observe has a tag.  A
        // voxel that observes is within r + mu of the sensor, whatever the pose: with
        // k = |D|, the ray ends at k (r + mu), and eta >= -mu only up to (r + mu) / k)
        const bool all = v->nb <= kSeenAll && (g.maxd + g.mu) / (8.0 * g.s) <= kSeenRange;
        hipLaunchKernelGGL(all ? k_laser_accumulate<true> : k_laser_accumulate<false>, dim3(grid1(n), 2), dim3(256), 0,
                           st, g, pts, n, slots, v->hash_slots, v->hash_cap, reinterpret_cast<const int4 *>(v->coords),
                           int(v->nb), ls, sums, total);
        hipLaunchKernelGGL(k_laser_apply_sums, dim3(grid1(nvox)), dim3(256), 0, st, sums, nvox, ls, total,
                           v->prm.max_observations, report(v), v->f, v->w);
        DN_HIP(hipGetLastError());
        if ((rc = fetch_report(v, 1))) return rc;
        const int64_t m = v->host_stage[0];
        if (m > v->prm.max_observations) {
            set_error("%lld laser observations exceed the volume's max_observations %lld", (long long)m,
                      (long long)v->prm.max_observations);
            return DN_E_CAPACITY;
        }
        if (m > 0) v->emask_nb = -1;
        return DN_OK;
    }
    bump = Bump(v->scratch, v->scratch_bytes);
    LaserScratch x = carve_laser(bump, n, v->prm.max_observations);
    if (!bump.fits()) { set_error("scratch too small for the laser observations"); return DN_E_CAPACITY; }
    hipLaunchKernelGGL(k_laser_obs_count, dim3(grid1(n)), dim3(256), 0, st, g, pts, n, slots, v->hash_slots,
                       v->hash_cap, x.counts);
    DN_HIP(hipGetLastError());
    size_t tbytes = x.tmp_bytes;
    DN_HIP(rocprim::exclusive_scan(x.tmp, tbytes, x.counts, x.offs, int64_t(0), size_t(n),
                                   rocprim::plus<int64_t>(), st));
    DN_HIP(hipMemcpyAsync(v->host_stage, x.offs + n - 1, 8, hipMemcpyDeviceToHost, st));
    DN_HIP(hipMemcpyAsync(v->host_stage + 1, x.counts + n - 1, 8, hipMemcpyDeviceToHost, st));
    DN_HIP(hipStreamSynchronize(st));
    const int64_t m = v->host_stage[0] + v->host_stage[1];
    if (m == 0) return DN_OK;
    if (m > v->prm.max_observations) {
        set_error("%lld laser observations exceed the volume's max_observations %lld", (long long)m,
                  (long long)v->prm.max_observations);
        return DN_E_CAPACITY;
    }
    hipLaunchKernelGGL(k_laser_obs_emit, dim3(grid1(n)), dim3(256), 0, st, g, pts, n, slots, v->hash_slots,
                       v->hash_cap, x.offs, x.k_in, x.v_in, m);
    DN_HIP(hipGetLastError());
    int bits = 1;
    while ((int64_t(1) << bits) < v->nb * int64_t(kBlockVox)) ++bits;
    // sort by voxel, then the sum and the count of each voxel's observations
    // (distinct voxels into k_in / v_in, counts into counts32)
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::radix_sort_pairs(x.tmp, tbytes, x.k_in, x.k_out, x.v_in, x.v_out, size_t(m), 0, bits, st));
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::reduce_by_key(x.tmp, tbytes, x.k_out, x.v_out, size_t(m), x.k_in, x.v_in, x.nruns,
                                  rocprim::plus<double>(), rocprim::equal_to<uint32_t>(), st));
    tbytes = x.tmp_bytes;
    DN_HIP(rocprim::run_length_encode(x.tmp, tbytes, x.k_out, size_t(m), x.k_in, x.counts32, x.nruns, st));
    hipLaunchKernelGGL(k_laser_apply, dim3(grid1(m)), dim3(256), 0, st, x.k_in, x.v_in, x.counts32, x.nruns, m,
                       v->f, v->w);
    DN_HIP(hipGetLastError());
    v->emask_nb = -1;
    return DN_OK;
}

}  // extern "C"
