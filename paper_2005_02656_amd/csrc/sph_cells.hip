// sph_cells.hip -- sph_build_cells: keep particles in the depth-first (Morton)
// order of the octree (section 4.3).
//
//   1. bounding box of the open axes and largest h (each workgroup's extrema;
//      min/max are exact and order-free, so the result is deterministic);
//   2. from them the domain record (key domain, 2^21 scale per axis, cell level)
//      and 63-bit keys (21 bits per axis, x highest in each bit triplet) + iota;
//   3. stable LSD radix sort of (key, slot), 8 bits a pass.  Per pass:
//      LDS tile histogram -> exclusive scan of the digit-major counts ->
//      stable LDS-local ranking (wave ballots) -> tile reordered in LDS and
//      written digit run by digit run (coalesced);
//   4. dense cell table (start/end per Morton cell at the chosen level), and
//      every state array gathered through the permutation into workspace
//      scratch and copied back.
#include "sph_common.h"

namespace sph {
namespace {

constexpr int kSortItems = 16;                      // keys per thread per tile
constexpr int kSortTile = kBlock * kSortItems;      // 4096
constexpr int kWaves = kBlock / 64;
constexpr int kWaveItems = kSortTile / kWaves;      // 1024 consecutive keys per wave
// workgroups of the bounding box: 256, and from 1 M particles on one per 4,096 up to
// 1,024 (256 leave too few loads in flight there: a whole cell build of 4.1, 15.6 and
// 64 M particles took 0.774, 2.865 and 11.12 ms with 256, 0.730, 2.70 and 10.38 now.
// 1,024 at 262,144 cost this launch and the next 23.4 us against 20.0)
constexpr int64_t kRedGrid = 256, kRedGridMax = 1024;
static_assert(kRedGridMax <= kSumBlocks, "the partial extrema share the sums' area");
#ifndef SPH_CELL_FACTOR
#define SPH_CELL_FACTOR 0.5
#endif
// cell edge >= kCellFactor * hmax: cells smaller than the kernel reach, walked
// with a per-target stencil and per-cell distance culling
constexpr double kCellFactor = SPH_CELL_FACTOR;

__global__ void k_clear_domain(Domain* d)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        Domain z = {};
        *d = z;
    }
}

__device__ __forceinline__ double wave_min(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// the key domain along an axis, from the extrema of the positions
__device__ __forceinline__ void key_axis(const Params& P, int k, const double (&r)[7], double& lo,
                                         double& hi, double& scale)
{
    lo = P.periodic[k] ? P.box_lo[k] : r[k];
    hi = P.periodic[k] ? P.box_hi[k] : r[3 + k];
    const double D = hi - lo;
    scale = D > 0.0 ? 2097152.0 / D : 0.0;
}

// The domain record, from the extrema of the open axes and the largest h.  Nothing
// in it but the error word outlives a cell build.
__device__ void domain_record(const Params& P, Domain* d, const double (&r)[7], bool mv, bool uv)
{
    double hm = r[6];
    if (!(hm > 0.0)) hm = 0.0;
    double D[3], ext = 0.0;
    for (int k = 0; k < 3; ++k) {
        key_axis(P, k, r, d->lo[k], d->hi[k], d->scale[k]);
        D[k] = d->hi[k] - d->lo[k];
        ext = fmax(ext, D[k]);
    }
    // the walk's unit: ext is 1/2 .. 1 of it (1 where ext is 0 or no finite number)
    int e = 0;
    if (ext > 0.0 && ext < INFINITY) frexp(ext, &e);
    const double sc = ldexp(1.0, -max(-1022, min(1022, e)));
    d->walk_scale = sc;
    d->walk_slack = (float)(ext * sc * 0x1p-20);
    for (int k = 0; k < 3; ++k) {
        d->wrap[k] = P.periodic[k] ? (float)(P.L[k] * sc) : 0.0f;
        d->wrap_inv[k] = P.periodic[k] ? (float)(1.0 / (P.L[k] * sc)) : 0.0f;
    }
    int level = 0;
    for (int l = P.lcap; l >= 0; --l) {
        bool ok = true;
        for (int k = 0; k < 3; ++k)
            if (D[k] > 0.0 && D[k] / (double)(1 << l) < kCellFactor * hm) ok = false;
        if (ok) { level = l; break; }
    }
    d->level = level;
    d->shift = 3 * (kKeyBits - level);
    d->ncell_axis = 1 << level;
    for (int k = 0; k < 3; ++k) d->cell[k] = (D[k] > 0.0) ? D[k] / (double)(1 << level) : 0.0;
    d->hmax = hm;
    d->mass_varies = mv ? 1u : 0u;
    d->u_varies = uv ? 1u : 0u;
    d->reach_level = reach_level(*d, 2.0 * P.kappa * hm);
    d->arrived = 0u;
    d->built_n = P.n;
}

// Extrema over the first `waves` (at most kWaves) wavefronts of a workgroup into r,
// mv and uv of thread 0
__device__ __forceinline__ void block_extrema(double (&r)[7], bool& mv, bool& uv, int waves)
{
    __shared__ double s[kWaves][7];
    __shared__ uint32_t flags[kWaves];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w < waves) {
        for (int k = 0; k < 3; ++k) r[k] = wave_min(r[k]);
        for (int k = 3; k < 7; ++k) r[k] = wave_max(r[k]);
        const uint32_t f = (__ballot(mv) ? 1u : 0u) | (__ballot(uv) ? 2u : 0u);
        if (lane == 0) {
            for (int k = 0; k < 7; ++k) s[w][k] = r[k];
            flags[w] = f;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t all = 0u;
    for (int ww = 0; ww < waves; ++ww) {
        for (int k = 0; k < 3; ++k) r[k] = fmin(r[k], s[ww][k]);
        for (int k = 3; k < 7; ++k) r[k] = fmax(r[k], s[ww][k]);
        all |= flags[ww];
    }
    mv = (all & 1u) != 0u;
    uv = (all & 2u) != 0u;
}

// Bounding box of the open axes, largest h, and whether the masses and the
// internal energies are all slot 0's (the passes then take the mass from there,
// or the shorter momentum records).  Each workgroup leaves its extrema in `part`;
// the next launch combines them.  With atomics on one line instead 262,144
// particles took 63 us and 1 M 66, and a launch for the record 9 more.
__global__ __launch_bounds__(kBlock) void k_bbox(Params P, const double* __restrict__ x,
                                                 const double* __restrict__ y,
                                                 const double* __restrict__ z,
                                                 const double* __restrict__ h,
                                                 const double* __restrict__ m,
                                                 const double* __restrict__ u,
                                                 double* __restrict__ part)
{
    double r[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY};
    const double* pos[3] = {x, y, z};
    const double m0 = m[0], u0 = u[0];
    bool mv = false, uv = false;
    const int64_t step = (int64_t)gridDim.x * kBlock;
#pragma unroll 2
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < P.n; i += step) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (P.periodic[k]) continue;
            const double v = pos[k][i];
            r[k] = fmin(r[k], v);
            r[3 + k] = fmax(r[3 + k], v);
        }
        r[6] = fmax(r[6], h[i]);
        mv |= m[i] != m0;
        uv |= u[i] != u0;
    }
    block_extrema(r, mv, uv, kWaves);
    if (threadIdx.x != 0) return;
    double* out = part + blockIdx.x * 10;
    for (int k = 0; k < 7; ++k) out[k] = r[k];
    out[7] = mv ? 1.0 : 0.0;
    out[8] = uv ? 1.0 : 0.0;
}

// keys and the digit counts of the sort's first pass, tile by tile; the cell
// table and the blocks' largest h start from nothing here too (three launches
// before).  1,024 threads a tile: with 256 the 64 tiles of 262,144 particles took
// 22 us, now 10.  Every workgroup combines the extrema for itself, the first one
// leaves the domain record: no workgroup waits for another, and no counter has to
// hold a known value when a call begins.  The grid is bounded, as that takes some
// microseconds each time, and the registers are held to two workgroups per CU (15.6
// M particles, 3,815 tiles: 221 us without either, 177 with the first, 116 with
// both).  With the record by the last workgroup of the launch before, the
// two launches took 12.4 us at 1,000 particles and 24.6 at 262,144; now 11.2 and 20.0.
constexpr int kKeyThreads = 1024;
constexpr int64_t kKeyGrid = 1024;
__global__ __launch_bounds__(kKeyThreads) SPH_WAVES_EXACT(8) void k_keys(Params P, const double* __restrict__ x,
                                                 const double* __restrict__ y,
                                                 const double* __restrict__ z, Domain* d,
                                                 const double* __restrict__ part, int nparts,
                                                 uint64_t* __restrict__ keys,
                                                 uint32_t* __restrict__ idx, int shift,
                                                 uint32_t* __restrict__ hist, int64_t nb,
                                                 CellRange* __restrict__ cells, int64_t ncells,
                                                 uint64_t* __restrict__ reach, int64_t nreach)
{
    __shared__ uint32_t hh[256];
    __shared__ double lo[3], scale[3];
    const int64_t n = P.n;
    double r[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY};
    bool mv = false, uv = false;
    if (threadIdx.x < kBlock) {
        for (int i = threadIdx.x; i < nparts; i += kBlock) {
            const double* in = part + i * 10;
#pragma unroll
            for (int k = 0; k < 3; ++k) r[k] = fmin(r[k], in[k]);
#pragma unroll
            for (int k = 3; k < 7; ++k) r[k] = fmax(r[k], in[k]);
            mv |= in[7] != 0.0;
            uv |= in[8] != 0.0;
        }
    }
    block_extrema(r, mv, uv, min((nparts + 63) / 64, kWaves));
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) {
            double hi;
            key_axis(P, k, r, lo[k], hi, scale[k]);
        }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) domain_record(P, d, r, mv, uv);
    for (int64_t tile = blockIdx.x; tile < nb; tile += gridDim.x) {
        if (threadIdx.x < 256) hh[threadIdx.x] = 0;
        __syncthreads();
        const int64_t base = tile * kSortTile;
#pragma unroll
        for (int i = 0; i < kSortTile / kKeyThreads; ++i) {
            const int64_t g = base + i * kKeyThreads + threadIdx.x;
            if (g >= n) continue;
            const uint32_t qx = quantize(x[g], lo[0], scale[0]);
            const uint32_t qy = quantize(y[g], lo[1], scale[1]);
            const uint32_t qz = quantize(z[g], lo[2], scale[2]);
            const uint64_t key = morton3(qx, qy, qz);
            keys[g] = key;
            idx[g] = (uint32_t)g;
            if (shift < 64) atomicAdd(&hh[(uint32_t)(key >> shift) & 255u], 1u);
            if (g < ncells) cells[g] = CellRange{0, 0, 0.0};
            if (g < nreach) reach[g] = reach[nreach + g] = 0ull;   // and the fullest cells
        }
        __syncthreads();
        if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * nb + tile] = hh[threadIdx.x];
    }
}

// ------------------------------------------------------------------ radix sort
__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint64_t* __restrict__ keys,
                                                       int64_t n, int shift,
                                                       uint32_t* __restrict__ hist, int64_t nb)
{
    __shared__ uint32_t hh[256];
    hh[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = blockIdx.x * (int64_t)kSortTile;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        int64_t g = base + i * kBlock + threadIdx.x;
        if (g < n) atomicAdd(&hh[(uint32_t)(keys[g] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nb + blockIdx.x] = hh[threadIdx.x];
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive scan over the block (kBlock threads); lds needs kWaves+1 entries
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t& total)
{
    uint32_t inc = wave_incl_scan(v);
    int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int i = 0; i < kWaves; ++i) {
            uint32_t t = lds[i];
            lds[i] = acc;
            acc += t;
        }
        lds[kWaves] = acc;
    }
    __syncthreads();
    uint32_t r = lds[w] + inc - v;
    total = lds[kWaves];
    __syncthreads();
    return r;
}

// sums of consecutive chunks of kSortTile entries
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t* __restrict__ a,
                                                        int64_t len, uint32_t* __restrict__ part)
{
    __shared__ uint32_t lds[kWaves + 1];
    int64_t base = blockIdx.x * (int64_t)kSortTile + threadIdx.x * kSortItems;
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i)
        if (base + i < len) s += a[base + i];
    uint32_t total;
    block_excl_scan(s, lds, total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// exclusive scan of the chunk sums, one block, chunks of kBlock with a carry
__global__ __launch_bounds__(kBlock) void k_scan_top(uint32_t* part, int64_t np)
{
    __shared__ uint32_t lds[kWaves + 1];
    uint32_t carry = 0;
    for (int64_t base = 0; base < np; base += kBlock) {
        int64_t i = base + threadIdx.x;
        uint32_t v = i < np ? part[i] : 0u;
        uint32_t total;
        uint32_t ex = block_excl_scan(v, lds, total);
        if (i < np) part[i] = carry + ex;
        carry += total;
    }
}

// exclusive scan of each chunk, offset by the chunk's prefix, in place
__global__ __launch_bounds__(kBlock) void k_scan_down(uint32_t* __restrict__ a, int64_t len,
                                                      const uint32_t* __restrict__ part)
{
    __shared__ uint32_t lds[kWaves + 1];
    int64_t base = blockIdx.x * (int64_t)kSortTile + threadIdx.x * kSortItems;
    uint32_t v[kSortItems];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        v[i] = (base + i < len) ? a[base + i] : 0u;
        s += v[i];
    }
    uint32_t total;
    uint32_t ex = block_excl_scan(s, lds, total) + part[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        if (base + i < len) a[base + i] = ex;
        ex += v[i];
    }
}

// the same three steps in one workgroup, for up to kScanOne entries (131,072
// particles): each thread sums a run of them, the runs' starts follow from one
// scan of the 1,024 sums.  2 us against 3 x 2 at 1,000 particles; at 262,144
// (16,384 entries) its one workgroup takes 24 us, the three launches 14.
constexpr int kScanThreads = 1024;
constexpr int64_t kScanOne = 8192;
__global__ __launch_bounds__(kScanThreads) void k_scan_one(uint32_t* __restrict__ a, int64_t len)
{
    __shared__ uint32_t waves[kScanThreads / 64];
    const int t = threadIdx.x, per = (int)((len + kScanThreads - 1) / kScanThreads);
    const int64_t base = (int64_t)t * per;
    uint32_t sum = 0;
    for (int i = 0; i < per; ++i)
        if (base + i < len) sum += a[base + i];
    const uint32_t inc = wave_incl_scan(sum);
    if ((t & 63) == 63) waves[t >> 6] = inc;
    __syncthreads();
    uint32_t ex = inc - sum;
    for (int w = 0; w < (t >> 6); ++w) ex += waves[w];
    for (int i = 0; i < per; ++i) {
        if (base + i < len) {
            const uint32_t v = a[base + i];
            a[base + i] = ex;
            ex += v;
        }
    }
}

// stable scatter of one tile by the digit at `shift`
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const uint64_t* __restrict__ kin, const uint32_t* __restrict__ iin,
    uint64_t* __restrict__ kout, uint32_t* __restrict__ iout, int64_t n, int shift,
    const uint32_t* __restrict__ offs, int64_t nb)
{
    __shared__ uint32_t wcount[kWaves][256];   // running digit counts per wave
    __shared__ uint32_t bstart[256];           // digit start in the reordered tile
    __shared__ uint32_t gofs[256];             // global start of the digit for this tile
    __shared__ uint32_t lds[kWaves + 1];
    __shared__ uint64_t skey[kSortTile];
    __shared__ uint32_t sidx[kSortTile];

    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int ww = 0; ww < kWaves; ++ww) wcount[ww][t] = 0;
    gofs[t] = offs[(int64_t)t * nb + blockIdx.x];
    __syncthreads();

    const int64_t tile = blockIdx.x * (int64_t)kSortTile;
    const int64_t base = tile + (int64_t)w * kWaveItems;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t k[kSortItems];
    uint32_t v[kSortItems], r[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        int64_t g = base + (int64_t)i * 64 + lane;
        bool ok = g < n;
        uint64_t key = ok ? kin[g] : 0ull;
        uint32_t d = (uint32_t)(key >> shift) & 255u;
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t rank = __popcll(peers & below);
        uint32_t before = wcount[w][d];
        // lanes of one wavefront run in lockstep: every peer has read `before`
        // when the lowest peer stores the advanced count
        if (ok && (peers & below) == 0) wcount[w][d] = before + (uint32_t)__popcll(peers);
        k[i] = key;
        v[i] = ok ? iin[g] : 0u;
        r[i] = ok ? before + rank : 0xffffffffu;
    }
    __syncthreads();
    {
        uint32_t c[kWaves], tot = 0;
        for (int ww = 0; ww < kWaves; ++ww) {
            c[ww] = wcount[ww][t];
            wcount[ww][t] = tot;
            tot += c[ww];
        }
        uint32_t total;
        bstart[t] = block_excl_scan(tot, lds, total);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        if (r[i] != 0xffffffffu) {
            uint32_t d = (uint32_t)(k[i] >> shift) & 255u;
            uint32_t pos = bstart[d] + wcount[w][d] + r[i];
            skey[pos] = k[i];
            sidx[pos] = v[i];
        }
    }
    __syncthreads();
    int64_t rem = n - tile;
    int cnt = rem < kSortTile ? (int)rem : kSortTile;
    for (int p = t; p < cnt; p += kBlock) {
        uint64_t key = skey[p];
        uint32_t d = (uint32_t)(key >> shift) & 255u;
        int64_t dst = (int64_t)gofs[d] + (p - (int64_t)bstart[d]);
        kout[dst] = key;
        iout[dst] = sidx[p];
    }
}

// ------------------------------------------------------------------ cell table
// start and end of slot i's cell, where the sorted keys change cells
__device__ __forceinline__ void fill_cell(const Domain* __restrict__ d,
                                          const uint64_t* __restrict__ keys, int64_t i, int64_t n,
                                          CellRange* __restrict__ cells)
{
    const int sh = d->shift;
    uint64_t c = (sh >= 64) ? 0ull : (keys[i] >> sh);
    uint64_t cp = (i > 0) ? ((sh >= 64) ? 0ull : (keys[i - 1] >> sh)) : ~0ull;
    uint64_t cn = (i + 1 < n) ? ((sh >= 64) ? 0ull : (keys[i + 1] >> sh)) : ~0ull;
    if (cp != c) cells[c].s = (int32_t)i;
    if (cn != c) cells[c].e = (int32_t)(i + 1);
}

// ------------------------------------------------------------------ permutation
struct PermSet {
    uint64_t* f[kMaxPermFields];
    int nf;
};

// every state array gathered into the sorted order, and the cell table
__global__ __launch_bounds__(kBlock) void k_gather(PermSet S, const uint32_t* __restrict__ perm,
                                                   uint64_t* __restrict__ tmp, int64_t n,
                                                   const Domain* __restrict__ dom,
                                                   const uint64_t* __restrict__ keys,
                                                   CellRange* __restrict__ cells)
{
    int64_t nb = (n + kBlock - 1) / kBlock;
    int64_t lb = xcd_block(nb);
    if (lb < 0) return;
    int64_t i = lb * kBlock + threadIdx.x;
    if (i >= n) return;
    fill_cell(dom, keys, i, n, cells);
    uint32_t src = perm[i];
    for (int f = 0; f < S.nf; ++f) tmp[(int64_t)f * n + i] = S.f[f][src];
}

// copy back, and pack positions and h (fields 0, 1, 2 and 9 of the set); with
// pf, also the FP32 walk records of the fused candidate pass
__global__ __launch_bounds__(kBlock) void k_scatter_back(PermSet S,
                                                         const uint64_t* __restrict__ tmp,
                                                         int64_t n, const Domain* __restrict__ dom,
                                                         Pos4* __restrict__ p4,
                                                         Pos4f* __restrict__ pf, float k2s)
{
    int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i >= n) return;
    for (int f = 0; f < S.nf; ++f) S.f[f][i] = tmp[(int64_t)f * n + i];
    Pos4 q;
    q.x = __builtin_bit_cast(double, tmp[i]);
    q.y = __builtin_bit_cast(double, tmp[n + i]);
    q.z = __builtin_bit_cast(double, tmp[2 * n + i]);
    q.h = __builtin_bit_cast(double, tmp[9 * n + i]);
    p4[i] = q;
    if (pf) pf[i] = walk_record(dom, q, k2s);
}

__global__ __launch_bounds__(kBlock) void k_pack_p4(const double* __restrict__ x,
                                                    const double* __restrict__ y,
                                                    const double* __restrict__ z,
                                                    const double* __restrict__ h, int64_t n,
                                                    Pos4* __restrict__ p4)
{
    int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i >= n) return;
    p4[i] = Pos4{x[i], y[i], z[i], h[i]};
}

}  // namespace

// The kernel tables (section 4.5): entry i holds the values at nodes i and
// i+1 of v_i = 2i/(N-1), from the same fitted polynomials as the direct
// evaluation; dS_n/dv = (v dS_n/dv) / v, 0 at v = 0 (S_n is even in v).
__global__ __launch_bounds__(kBlock) void k_fill_tables(Params P, double2* __restrict__ tS,
                                                        double2* __restrict__ tD,
                                                        float2* __restrict__ tSf,
                                                        float2* __restrict__ tDf)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= P.tab_n - 1) return;
    double S[2], D[2];
    for (int k = 0; k < 2; ++k) {
        const double v = (double)(i + k) / P.tab_inv_dv;
        double vdS;
        sinc_terms(kPiHalfSq * v * v, P.sinc_n, S[k], vdS);
        D[k] = v > 0.0 ? vdS / v : 0.0;
    }
    tS[i] = make_double2(S[0], S[1]);
    tD[i] = make_double2(D[0], D[1]);
    tSf[i] = make_float2((float)S[0], (float)S[1]);
    tDf[i] = make_float2((float)D[0], (float)D[1]);
}

hipError_t launch_clear_domain(const Ws& W, hipStream_t s)
{
    k_clear_domain<<<1, 64, 0, s>>>(W.dom);
    return hipGetLastError();
}

hipError_t launch_build_cells(const Params& P, const Layout& L, const Ws& W,
                              const sph_particles* p, hipStream_t s)
{
    const int64_t n = P.n;
    const int64_t nb = (n + kBlock - 1) / kBlock;
    if (P.tab_n > 0)
        k_fill_tables<<<(P.tab_n + kBlock - 1) / kBlock, kBlock, 0, s>>>(P, W.tabS, W.tabD,
                                                                          W.tabSf, W.tabDf);
    const int64_t wanted = nb / 16 < kRedGrid ? kRedGrid : nb / 16 < kRedGridMax ? nb / 16 : kRedGridMax;
    const int64_t rg = nb < wanted ? nb : wanted;
    k_bbox<<<rg, kBlock, 0, s>>>(P, p->x, p->y, p->z, p->h, p->m, p->u, W.sums);

    // Stable LSD radix sort by the key's prefix of lcap levels (3 lcap bits, 8
    // bits a pass): the depth-first order of the octree down to its finest
    // cells (section 4.3), every cell level the step uses being at most lcap.
    // Inside a finest cell the particles keep the order they came in, so the
    // order is updated, not rebuilt: only particles that changed cells move.
    // The first buffers are those from which the last pass ends in keys0/idx0.
    const int s0 = 3 * (kKeyBits - L.lcap);
    const int passes = (3 * L.lcap + 7) / 8;
    uint64_t* kin = passes & 1 ? W.keys1 : W.keys0;
    uint64_t* kout = passes & 1 ? W.keys0 : W.keys1;
    uint32_t* iin = passes & 1 ? W.idx1 : W.idx0;
    uint32_t* iout = passes & 1 ? W.idx0 : W.idx1;
    const int64_t kg = L.nsort_blocks < kKeyGrid ? L.nsort_blocks : kKeyGrid;
    k_keys<<<kg, kKeyThreads, 0, s>>>(P, p->x, p->y, p->z, W.dom, W.sums, (int)rg, kin,
                                             iin, s0, W.hist,
                                             L.nsort_blocks, W.cells, L.ncells_cap, W.reach,
                                             L.nreach);
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = s0 + 8 * pass;
        if (pass > 0)
            k_radix_hist<<<L.nsort_blocks, kBlock, 0, s>>>(kin, n, shift, W.hist, L.nsort_blocks);
        if (L.hist_len <= kScanOne) {
            k_scan_one<<<1, kScanThreads, 0, s>>>(W.hist, L.hist_len);
        } else {
            k_scan_reduce<<<L.scan_blocks, kBlock, 0, s>>>(W.hist, L.hist_len, W.scanpart);
            k_scan_top<<<1, kBlock, 0, s>>>(W.scanpart, L.scan_blocks);
            k_scan_down<<<L.scan_blocks, kBlock, 0, s>>>(W.hist, L.hist_len, W.scanpart);
        }
        k_radix_scatter<<<L.nsort_blocks, kBlock, 0, s>>>(kin, iin, kout, iout, n, shift, W.hist,
                                                         L.nsort_blocks);
        uint64_t* tk = kin; kin = kout; kout = tk;
        uint32_t* ti = iin; iin = iout; iout = ti;
    }

    PermSet S{};
    uint64_t* fields[] = {(uint64_t*)p->x, (uint64_t*)p->y, (uint64_t*)p->z,
                          (uint64_t*)p->vx, (uint64_t*)p->vy, (uint64_t*)p->vz,
                          (uint64_t*)p->vhx, (uint64_t*)p->vhy, (uint64_t*)p->vhz,
                          (uint64_t*)p->h, (uint64_t*)p->m, (uint64_t*)p->u,
                          (uint64_t*)p->du_m1, (uint64_t*)p->id,
                          (uint64_t*)p->p_ref, (uint64_t*)p->rho_ref};
    for (uint64_t* f : fields)
        if (f) S.f[S.nf++] = f;
    k_gather<<<grid_xcd(nb), kBlock, 0, s>>>(S, W.idx0, (uint64_t*)W.tmp, n, W.dom, W.keys0,
                                             W.cells);
    k_scatter_back<<<nb, kBlock, 0, s>>>(S, (const uint64_t*)W.tmp, n, W.dom, W.p4,
                                         P.cand_cap > 0 ? W.pf : nullptr,
                                         short_reach_f32(P.kappa));
    return hipGetLastError();
}

hipError_t launch_pack_p4(const Params& P, const Ws& W, const sph_particles* p, hipStream_t s)
{
    const int64_t nb = (P.n + kBlock - 1) / kBlock;
    k_pack_p4<<<nb, kBlock, 0, s>>>(p->x, p->y, p->z, p->h, P.n, W.p4);
    return hipGetLastError();
}

}  // namespace sph
