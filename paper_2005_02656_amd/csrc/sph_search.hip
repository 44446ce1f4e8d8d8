// sph_search.hip -- smoothing-length Newton update and neighbour search.
//
// Cells are smaller than the kernel reach (edge >= h_max/2).  The walks of groups
// of 16 neighbouring targets test FP32 records of positions and reaches (below);
// the walks of one target per thread, over the packed 32-byte records, take their
// own stencil and skip cells whose box is out of reach, with a margin covering the
// rounding of the key quantisation.  Consecutive slots are Morton-consecutive, so
// the lanes of a wavefront sit in a few neighbouring cells and walk mostly the same
// ones (same-address loads across lanes, served from L1/L2).
//
// Three compositions use these kernels:
//  * the fused step: ONE walk, by groups of neighbouring targets, collects
//    candidates within 2 kappa max(h0_a, h0_b) (a superset of every set the step
//    needs, since the Newton clamp keeps h <= kappa h0), the Newton iterations sum
//    over the candidate list, and a filter pass writes the exact lists from the
//    candidates with the final h;
//  * the stage entry points: the same, a walk each for Newton (its reach chosen
//    by a sample) and for the lists;
//  * one target per lane by cell walks, for targets that the candidates of a stage
//    call do not serve and where the order of the sums has to stand.
//    The neighbour sets are identical; only the visiting order differs.
#include <cmath>

#include "sph_common.h"
#include "sph_walk_cell.h"

namespace sph {
namespace {

constexpr double kCullMargin = 1e-9;  // relative to the cell edge
// particles of a cell that a refit by a wavefront takes with all lanes together: a
// lane by itself needs some 150 cycles a particle, all together some 600 for each
// of up to 64 cells
constexpr uint32_t kRefitFat = 128;

// particle records of one cell loaded together by the cell walk (a batch may
// read up to kCellBatch - 1 records past the cell's end: the record arrays keep
// kWalkPad spare entries), and cell
// records of one row (along z) loaded together
#ifndef SPH_CELL_BATCH
#define SPH_CELL_BATCH 2
#endif
static_assert(SPH_CELL_BATCH - 1 <= kWalkPad, "cell-walk batch overruns the record padding");
#ifndef SPH_CELL_ROW
#define SPH_CELL_ROW 2
#endif

// spread the low 10 bits of v to every third bit (cell coordinates, level <= 9)
__device__ __forceinline__ uint32_t spread10(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

struct AxisWalk {
    int lo, hi;      // offsets (or absolute cells when `all`)
    bool all;        // every cell of a periodic axis, no culling
    bool empty;      // zero-extent axis: only cell 0
    int c0;          // target's cell
    double f;        // target position inside its cell
    double ce;       // cell edge
};

__device__ __forceinline__ AxisWalk axis_walk(const Params& P, const Domain& D, int k, double pos,
                                              double R)
{
    AxisWalk a;
    const int nax = D.ncell_axis;
    const int sh = kKeyBits - D.level;
    uint32_t q = quantize(pos, D.lo[k], D.scale[k]);
    a.c0 = (int)(q >> sh);
    a.ce = D.cell[k];
    a.all = false;
    a.empty = !(a.ce > 0.0);
    if (a.empty) {
        a.lo = a.hi = 0;
        a.f = 0.0;
        return a;
    }
    a.f = (pos - D.lo[k]) - (double)a.c0 * a.ce;
    double Kd = ceil(R / a.ce);
    int K = (Kd < (double)nax) ? (int)Kd : nax;
    if (P.periodic[k]) {
        if (2 * K + 1 >= nax) {
            a.all = true;
            a.lo = 0;
            a.hi = nax - 1;
        } else {
            a.lo = -K;
            a.hi = K;
        }
    } else {
        a.lo = (-K > -a.c0) ? -K : -a.c0;
        a.hi = (K < nax - 1 - a.c0) ? K : nax - 1 - a.c0;
    }
    return a;
}

// lower bound of the distance along one axis from the target to the cell at
// offset o, reduced by the rounding margin
__device__ __forceinline__ double axis_gap(const AxisWalk& a, int o)
{
    if (a.all || a.empty || o == 0) return 0.0;
    double d = (o > 0) ? (double)o * a.ce - a.f : a.f - (double)(o + 1) * a.ce;
    d -= kCullMargin * a.ce;
    return d > 0.0 ? d : 0.0;
}

__device__ __forceinline__ uint32_t axis_cell(const AxisWalk& a, int o, int nax)
{
    if (a.all || a.empty) return (uint32_t)o;
    int c = a.c0 + o;
    if (c < 0) c += nax;
    else if (c >= nax) c -= nax;
    return (uint32_t)c;
}

// Visit every particle of every cell whose box may hold a point closer than R
// to the target and that `want(cell, gap2)` accepts; body(b, record_of_b).
// Row by row, x outermost and rows along z: z takes the lowest bit of each
// coordinate triple of the Morton code, so the cells of a row pair are
// adjacent in the table and in particle order, and the lists the walk writes
// follow the particle order closely; the 64 lanes of a wavefront, whose
// targets are neighbours, then read the same records at about the same time in
// every later pass over the lists.  (Rows along x, the same walk with z
// outermost, made every list pass 5-15% slower at 64 M particles, and a walk
// block by block in Morton order made the walk itself 25% slower.)  The cell
// records of one row (up to kRow cells) are loaded together, then each cell's
// particle records in batches: independent loads in flight instead of one
// dependent load per candidate.
template <class Rec, class Want, class Body>
__device__ __forceinline__ void walk_cells(const Params& P, const Domain& D,
                                           const CellRange* __restrict__ cells,
                                           const Rec* __restrict__ recs, double xa, double ya,
                                           double za, double R, Want&& want, Body&& body)
{
    constexpr int kRow = SPH_CELL_ROW;
    constexpr int kCellBatch = SPH_CELL_BATCH;
    const int nax = D.ncell_axis;
    AxisWalk wx = axis_walk(P, D, 0, xa, R);
    AxisWalk wy = axis_walk(P, D, 1, ya, R);
    AxisWalk wz = axis_walk(P, D, 2, za, R);
    const AxisWalk& wo = wx;   // outer axis and its Morton bit offset
    const AxisWalk& wi = wz;   // row axis
    constexpr int so = 2, si = 0;
    const double R2 = R * R;
    for (int oo = wo.lo; oo <= wo.hi; ++oo) {
        double go = axis_gap(wo, oo);
        double go2 = go * go;
        if (go2 >= R2) continue;
        uint32_t mo = spread10(axis_cell(wo, oo, nax)) << so;
        for (int oy = wy.lo; oy <= wy.hi; ++oy) {
            double gy = axis_gap(wy, oy);
            double goy2 = go2 + gy * gy;
            if (goy2 >= R2) continue;
            uint32_t moy = mo | (spread10(axis_cell(wy, oy, nax)) << 1);
            for (int oi0 = wi.lo; oi0 <= wi.hi; oi0 += kRow) {
                uint32_t cid[kRow];
                double g2[kRow];
                bool in[kRow];
#pragma unroll
                for (int i = 0; i < kRow; ++i) {
                    const int oi = oi0 + i;
                    double gi = (oi <= wi.hi) ? axis_gap(wi, oi) : 0.0;
                    g2[i] = goy2 + gi * gi;
                    in[i] = (oi <= wi.hi) && g2[i] < R2;
                    cid[i] = in[i] ? (moy | (spread10(axis_cell(wi, oi, nax)) << si)) : 0u;
                }
                CellRange cr[kRow];
#pragma unroll
                for (int i = 0; i < kRow; ++i) cr[i] = cells[cid[i]];
#pragma unroll
                for (int i = 0; i < kRow; ++i) {
                    if (!in[i] || !want(cr[i], g2[i])) continue;
                    const int32_t e = cr[i].e;
                    for (int32_t b0 = cr[i].s; b0 < e; b0 += kCellBatch) {
                        Rec q[kCellBatch];
#pragma unroll
                        for (int u = 0; u < kCellBatch; ++u) q[u] = recs[b0 + u];
#pragma unroll
                        for (int u = 0; u < kCellBatch; ++u)
                            if (b0 + u < e) body(b0 + u, q[u]);
                    }
                }
            }
        }
    }
}


__device__ __forceinline__ double newton_step(const Params& P, double hc, double h0, double sS,
                                              double sV)
{
    const double k3 = (32.0 * kPi / 3.0) * P.bn;
    const double kap = P.kappa;
    double F = k3 * sS - P.n_target;
    double Fp = -(k3 / hc) * sV;
    double hn = (Fp > 0.0) ? hc - F / Fp : kap * h0;
    if (hn < h0 / kap) hn = h0 / kap;
    if (hn > kap * h0) hn = kap * h0;
    return hn;
}

__device__ __forceinline__ void check_cell_range(const Params& P, Domain* dom, double h)
{
    for (int k = 0; k < 3; ++k)
        if (P.periodic[k] && !(4.0 * h < P.L[k])) set_err(dom, SPH_ERRBIT_CELL_RANGE);
}

// ---------------------------------------------------------------- cell-walk forms
// (flag: only the targets it marks with 2, if any is marked, unless the stage call
// has no reach and leaves all to this walk)
__global__ __launch_bounds__(kBlock) void k_update_h(Params P, const Domain* __restrict__ dom,
                                                     const CellRange* __restrict__ cells,
                                                     const Pos4* __restrict__ p4,
                                                     double* __restrict__ h,
                                                     const uint8_t* __restrict__ flag)
{
    const bool some = flag && dom->stage_reach > 0.0;
    if (some && dom->refit == 0u) return;
    const int64_t nb = (P.n + kBlock - 1) / kBlock;
    const int64_t lb = xcd_block(nb);
    if (lb < 0) return;
    const int64_t a = lb * kBlock + threadIdx.x;
    if (a >= P.n || (some && flag[a] != 2)) return;
    const Domain D = *dom;
    const Pos4 pa = p4[a];
    const double xa = pa.x, ya = pa.y, za = pa.z;
    const double h0 = flag ? pa.h : h[a];
    double hc = h0;
    for (int it = 0; it < P.newton_iters; ++it) {
        const double h2 = 2.0 * hc;
        const double R2 = h2 * h2;
        const double tsc = kPiHalfSq / (hc * hc);
        double sS = 0.0, sV = 0.0;
        walk_cells(P, D, cells, p4, xa, ya, za, h2,
                   [](const CellRange&, double) { return true; },
                   [&](int32_t b, const Pos4& q) {
                       double dx, dy, dz;
                       double r2 = disp(P, xa, ya, za, q.x, q.y, q.z, dx, dy, dz);
                       if (r2 < R2) {
                           double S, vdS;
                           kern_terms(P, r2 * tsc, S, vdS);
                           sS += S;
                           sV += vdS;
                       }
                   });
        hc = newton_step(P, hc, h0, sS, sV);
    }
    h[a] = hc;
}

__global__ void k_hmax_begin(Domain* d) { d->hmax_new_bits = ord_bits(0.0); }

// The reach of sph_update_h's group walk is a bet on how far h moves: a walk at
// 1.03 h0 serves converged smoothing lengths, at up to 1.25 h0 those that still
// move, and where they move farther, or hold more candidates than fit, the targets
// walk by themselves and a group walk before that is lost.  Losing it cost up to
// twice the call: 1 M random particles with h 1.7 times too large 25 -> 52 ms, with
// h 4% short 3.3 -> 4.5 ms.  So a sample of the targets takes its first Newton step
// beforehand, in the launch that looks for the cells' largest h, a workgroup a
// target with its lanes on the cells (12 us of a converged call; 2,048 samples of a
// wavefront each 20).
constexpr int kSamples = 512;
inline int stage_samples(int64_t n) { return n < kSamples ? (int)n : kSamples; }
// One sampled target in kMissed without room for its candidates, or in kLost that
// grows past the largest reach, and all walk by themselves.  (Targets that grow lie
// together, at the edge of a clump, and the rest gains more than their walks cost;
// where candidates do not fit, h is too large and the group walk itself dear.  An h
// that is too large with room for its candidates stays: clumped sets from 1.7 h,
// twelve iterations by targets -> by the group walk: 30,000 particles 42 -> 49 ms,
// 100,000 25 -> 30, 400,000 64 -> 42, 1 M 102 -> 62.)
constexpr int kMissed = 64, kLost = 8;
// the largest reach of a group walk of the call, and the one to try first
__host__ __device__ inline double stage_wide(const Params& P)
{
    return P.kappa < kFusedKappaMax ? P.kappa : kFusedKappaMax;
}
__host__ __device__ inline double stage_short(const Params& P)
{
    return P.kappa <= kFusedKappaMax ? fmin(kFusedReach, P.kappa) : kFusedKappaMax;
}
// The call's reach.  With a clamp inside the largest reach no h can leave that:
// it is taken where more than one sampled h in 512 leaves the short one (by walks
// of their own that many would cost as much again); its lists hold 1.8 times
// the candidates (1 M random particles: 1.41 ms at the short reach, 2.41 at 1.25).
__device__ __forceinline__ double stage_reach(const Params& P, const Domain* dom, int ns)
{
    const int grown = (int)dom->stage_grown, crowded = (int)dom->stage_crowded;
    if (crowded * kMissed > ns) return 0.0;
    if (P.kappa <= kFusedKappaMax) return grown * 512 > ns ? stage_wide(P) : stage_short(P);
    return grown * kLost > ns ? 0.0 : stage_wide(P);
}

// one sampled target, by the whole workgroup: bit 0 if its first Newton step leaves
// the short reach, bit 1 if its candidates there would not fit (estimated from those
// within 2 h)
__device__ __forceinline__ uint32_t sample_target(const Params& P, const Domain& D,
                                                  const CellRange* __restrict__ cells,
                                                  const Pos4* __restrict__ p4, int cap, int64_t a)
{
    const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const Pos4 pa = p4[a];
    const double R = 2.0 * pa.h, R2 = R * R;
    const double tsc = kPiHalfSq / (pa.h * pa.h);
    const AxisWalk wx = axis_walk(P, D, 0, pa.x, R);
    const AxisWalk wy = axis_walk(P, D, 1, pa.y, R);
    const AxisWalk wz = axis_walk(P, D, 2, pa.z, R);
    const int nx = wx.hi - wx.lo + 1, ny = wy.hi - wy.lo + 1, nz = wz.hi - wz.lo + 1;
    const float ryz1 = 1.0f / (float)(ny * nz), rz1 = 1.0f / (float)nz;
    const int ncells = nx > 0 && ny > 0 && nz > 0 ? nx * ny * nz : 0;
    double sS = 0.0, sV = 0.0;
    int cnt = 0;
    auto add = [&](const Pos4& q) {
        double dx, dy, dz;
        const double r2 = disp(P, pa.x, pa.y, pa.z, q.x, q.y, q.z, dx, dy, dz);
        if (r2 < R2) {
            double S, vdS;
            kern_terms(P, r2 * tsc, S, vdS);
            sS += S;
            sV += vdS;
            ++cnt;
        }
    };
    // What it takes is the latency of its loads, one after the other: a lane's
    // cells are loaded together, then the first particles of all of them, then the
    // rest in fours (the records have spare entries past the last slot); a wavefront
    // shares what its fullest cells hold beyond 32.
    constexpr int kU = 4, kFirst = 2, kOwn = 32;
    for (int q0 = 0; q0 < ncells; q0 += kBlock * kU) {
        CellRange cr[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int q = q0 + kBlock * u + (int)threadIdx.x;
            cr[u] = CellRange{0, 0, 0.0};
            if (q >= ncells) continue;
            int ix, iy, iz;
            box_cell(q, nx, ny, nz, ryz1, rz1, ix, iy, iz);
            const double gx = axis_gap(wx, wx.lo + ix), gy = axis_gap(wy, wy.lo + iy);
            const double gz = axis_gap(wz, wz.lo + iz);
            if (gx * gx + gy * gy + gz * gz < R2)
                cr[u] = cells[(spread10(axis_cell(wx, wx.lo + ix, D.ncell_axis)) << 2) |
                              (spread10(axis_cell(wy, wy.lo + iy, D.ncell_axis)) << 1) |
                              spread10(axis_cell(wz, wz.lo + iz, D.ncell_axis))];
        }
        Pos4 first[kU][kFirst];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int v = 0; v < kFirst; ++v) first[u][v] = p4[cr[u].s + v];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
#pragma unroll
            for (int v = 0; v < kFirst; ++v)
                if (cr[u].s + v < cr[u].e) add(first[u][v]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t own = min(cr[u].e, cr[u].s + kOwn);
            for (int32_t b = cr[u].s + kFirst; b < own; b += 4) {
                Pos4 q[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) q[v] = p4[b + v];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (b + v < own) add(q[v]);
            }
            uint64_t full = __ballot(cr[u].e - cr[u].s > kOwn);
            while (full != 0u) {
                const int l = __ffsll((unsigned long long)full) - 1;
                full &= full - 1u;
                const int32_t e = __builtin_amdgcn_readlane(cr[u].e, l);
                for (int32_t b = __builtin_amdgcn_readlane(cr[u].s, l) + kOwn + lane; b < e; b += 64)
                    add(p4[b]);
            }
        }
    }
    sS = group_sum<64>(sS);
    sV = group_sum<64>(sV);
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    __shared__ double part[kBlock / 64][2];
    __shared__ int count[kBlock / 64];
    if (lane == 0) {
        part[wv][0] = sS;
        part[wv][1] = sV;
        count[wv] = cnt;
    }
    __syncthreads();
    sS = sV = 0.0;
    cnt = 0;
    for (int w = 0; w < kBlock / 64; ++w) {
        sS += part[w][0];
        sV += part[w][1];
        cnt += count[w];
    }
    const double lam = stage_short(P);
    return (newton_step(P, pa.h, pa.h, sS, sV) > lam * pa.h ? 1u : 0u) |
           ((double)cnt * (lam * lam * lam) > (double)cap ? 2u : 0u);
}

// largest h per cell (for the symmetric search) and overall
// (h is read from the slot-ordered array: consecutive cells read consecutive
// runs of it); one atomic per workgroup of a bounded grid of `blocks`; each
// workgroup past it takes one of sph_update_h's samples
constexpr int kHmaxGrid = 512;
template <bool kSample>
__global__ __launch_bounds__(kBlock) void k_cells_max(Params P, Domain* __restrict__ dom,
                                                      CellRange* __restrict__ cells,
                                                      const double* __restrict__ h, int64_t cap,
                                                      const Pos4* __restrict__ p4, int blocks)
{
    if (kSample && (int)blockIdx.x >= blocks) {
        const int i = (int)blockIdx.x - blocks, ns = (int)gridDim.x - blocks;
        const uint32_t bits =
            sample_target(P, *dom, cells, p4, P.cand_cap, (2 * i + 1) * P.n / (2 * ns));
        if (threadIdx.x < 2 && (bits >> threadIdx.x & 1u) != 0u) {
            uint32_t* to = threadIdx.x == 0 ? &dom->stage_grown : &dom->stage_crowded;
            // (past the decision the count does not matter)
            if ((int)__hip_atomic_load(to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * kLost <= ns)
                atomicAdd(to, 1u);
        }
        return;
    }
    const int64_t ncell = min(int64_t(1) << (3 * dom->level), cap);
    double all = 0.0;
    for (int64_t c = blockIdx.x * (int64_t)kBlock + threadIdx.x; c < ncell;
         c += (int64_t)blocks * kBlock) {
        double hm = 0.0;
        const CellRange cr = cells[c];
        for (int32_t b = cr.s; b < cr.e; ++b) hm = fmax(hm, h[b]);
        cells[c].hmax = hm;
        all = fmax(all, hm);
    }
    for (int o = 32; o > 0; o >>= 1) all = fmax(all, __shfl_xor(all, o, 64));
    __shared__ double part[kBlock / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = all;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) all = fmax(all, part[w]);
        ord_max_to(&dom->hmax_new_bits, all);
    }
}

// the neighbour search's condition on the largest h
__global__ void k_check_range(Params P, Domain* dom)
{
    const double hm = ord_value(dom->hmax_new_bits);
    if (hm > 0.0) check_cell_range(P, dom, hm);
}

// ---------------------------------------------------------------- walk reach
// The fused walk's stencil must hold every b within 2 kap max(h_a, h_b) of its
// target.  With one global bound (the largest h) the free surfaces and the
// thin outskirts of a cluster size every target's stencil.  Instead: blocks of
// the Morton octree at a level whose edge E exceeds 2 kappa h_max (plus the
// rounding of the keys and of the walk's FP32 test; chosen with the domain
// record) bound h_b by the largest h of the target's block and its 26 neighbours
// (periodic axes wrap).  A b outside those blocks is at least one block edge
// away, E > 2 kap max(h_a, h_b), so it can be no candidate; a b inside has h_b at
// most that bound.  Each walk then reaches 2 kap max(h_a, bound).
__device__ __forceinline__ uint32_t compact10(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030c30c3u;
    v = (v | (v >> 4)) & 0x0300f00fu;
    v = (v | (v >> 8)) & 0x030000ffu;
    v = (v | (v >> 16)) & 0x3ffu;
    return v;
}

// entry of a blocks' table for the i-th of block c and its 26 neighbours at the
// reach level, i = 0 .. 26 (wrapped on periodic axes, 0 beyond the edge of open ones)
__device__ __forceinline__ uint64_t block_neighbor(const Params& P, int level, uint32_t c, int i,
                                                   const uint64_t* __restrict__ table)
{
    const int nb = 1 << level;
    int q[3] = {(int)compact10(c >> 2) + i / 9 - 1, (int)compact10(c >> 1) + i / 3 % 3 - 1,
                (int)compact10(c) + i % 3 - 1};
    bool in = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (q[k] < 0 || q[k] >= nb) {
            if (P.periodic[k]) q[k] = (q[k] + nb) & (nb - 1);
            else in = false;
        }
    }
    if (!in) return 0u;
    const uint32_t cc = (spread10((uint32_t)q[0]) << 2) | (spread10((uint32_t)q[1]) << 1) |
                        spread10((uint32_t)q[2]);
    return table[cc];
}
// its largest h
__device__ __forceinline__ double reach_neighbor(const Params& P, int level, uint32_t c, int i,
                                                 const uint64_t* __restrict__ reach)
{
    return __builtin_bit_cast(double, block_neighbor(P, level, c, i, reach));
}

// The stage entry points walk by groups too, at the h of the call: packed
// positions, with the blocks' table and the call's words cleared
__global__ __launch_bounds__(kBlock) void k_stage_begin(Params P, Domain* __restrict__ dom,
                                                        const double* __restrict__ x,
                                                        const double* __restrict__ y,
                                                        const double* __restrict__ z,
                                                        const double* __restrict__ h,
                                                        Pos4* __restrict__ p4,
                                                        uint64_t* __restrict__ reach,
                                                        int64_t nreach)
{
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i == 0) {
        dom->hmax_new_bits = ord_bits(0.0);
        dom->refit = 0u;
        dom->stage_grown = dom->stage_crowded = 0u;
    }
    if (i >= P.n) return;
    p4[i] = Pos4{x[i], y[i], z[i], h[i]};
    if (i < nreach) reach[i] = 0ull;
}

// The call's reach (the lists' own, or chosen by the ns samples), the walk records
// for it, and the blocks' largest h from the cells' at the level for it
__global__ __launch_bounds__(kBlock) void k_stage_reach(Params P, Domain* __restrict__ dom,
                                                        const CellRange* __restrict__ cells,
                                                        int64_t cap, int ns,
                                                        const Pos4* __restrict__ p4,
                                                        Pos4f* __restrict__ pf,
                                                        uint64_t* __restrict__ reach)
{
    const int64_t c = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    const double kap = ns > 0 ? stage_reach(P, dom, ns) : 1.0;
    if (c == 0) dom->stage_reach = kap;
    if (!(kap > 0.0)) return;
    if (c < P.n) pf[c] = walk_record(dom, p4[c], up_f32(2.0 * kap));
    const int level = dom->level;
    const int rl = reach_level(*dom, 2.0 * kap * ord_value(dom->hmax_new_bits));
    if (c == 0) dom->reach_level = rl;
    const int64_t ncell = min(int64_t(1) << (3 * level), cap);
    double hm = c < ncell ? cells[c].hmax : 0.0;
    for (int o = 32; o > 0; o >>= 1) hm = fmax(hm, __shfl_xor(hm, o, 64));
    if ((threadIdx.x & 63) == 0 && c < ncell && hm > 0.0) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, hm);
        uint64_t* at = &reach[c >> (3 * (level - rl))];
        if (bits > __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax((unsigned long long*)at, (unsigned long long)bits);
    }
}

// The fused step's largest h per cell and per block of the reach level, the
// particles of each block's fullest cell (tables that the cell build cleared), and
// the step's flags.  h is still the cell
// build's, so its largest value is known and no word is shared by all
// workgroups: 262,144 particles 46 -> 5 us, and eleven launches fewer than with a
// level-by-level reduction, its bounds and the flags' resets.  h >= 0, so its bits
// order as integers; a wavefront's 64 cells lie in one block.
__global__ __launch_bounds__(kBlock) void k_cells_reach(Params P, Domain* __restrict__ dom,
                                                        CellRange* __restrict__ cells,
                                                        const double* __restrict__ h, int64_t cap,
                                                        uint64_t* __restrict__ reach,
                                                        uint64_t* __restrict__ fullest)
{
    const int64_t c = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    const int level = dom->level;
    const int64_t ncell = min(int64_t(1) << (3 * level), cap);
    double hm = 0.0;
    int cnt = 0;
    if (c < ncell) {
        const CellRange cr = cells[c];
        for (int32_t b = cr.s; b < cr.e; ++b) hm = fmax(hm, h[b]);
        cells[c].hmax = hm;
        cnt = cr.e - cr.s;
    }
    for (int o = 32; o > 0; o >>= 1) hm = fmax(hm, __shfl_xor(hm, o, 64));
    const uint64_t most = (uint64_t)wave_max_i(cnt);
    if ((threadIdx.x & 63) == 0 && c < ncell && hm > 0.0) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, hm);
        const int64_t block = c >> (3 * (level - dom->reach_level));
        uint64_t* at = &reach[block];
        if (bits > __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax((unsigned long long*)at, (unsigned long long)bits);
        at = &fullest[block];
        if (most > kRefitFat &&
            most > __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax((unsigned long long*)at, (unsigned long long)most);
    }
    if (c == 0) {
        dom->refit = 0u;
        dom->dtmin_bits = ord_bits(INFINITY);
        // equal sound speeds: equal internal energies, or the weakly
        // compressible EOS (c = c0)
        dom->nonuniform =
            dom->mass_varies | (P.eos == SPH_EOS_IDEAL ? dom->u_varies : 0u);
        if (dom->hmax > 0.0) check_cell_range(P, dom, dom->hmax);
    }
}

// symmetric neighbour lists: gather members of N(a) from the front of the
// tile row, members of N_s(a) \ N(a) from the back
__global__ __launch_bounds__(kBlock) void k_find_neighbors(Params P, Domain* __restrict__ dom,
                                                           const CellRange* __restrict__ cells,
                                                           const Pos4* __restrict__ p4,
                                                           int32_t* __restrict__ nc,
                                                           int32_t* __restrict__ ns,
                                                           int32_t* __restrict__ list,
                                                           const int32_t* __restrict__ nk, int cap)
{
    // (nk: only the targets with more candidates than their capacity, if any)
    if (nk && dom->refit == 0u) return;
    const int64_t nb = (P.n + kBlock - 1) / kBlock;
    const int64_t lb = xcd_block(nb);
    if (lb < 0) return;
    const int64_t a = lb * kBlock + threadIdx.x;
    if (a >= P.n || (nk && nk[a] <= cap)) return;
    const Domain D = *dom;
    const Pos4 pa = p4[a];
    const double xa = pa.x, ya = pa.y, za = pa.z, ha = pa.h;
    const double hnew = ord_value(D.hmax_new_bits);
    const double ha2 = 2.0 * ha;
    const double Ra2 = ha2 * ha2;
    const int ng = P.ng_max;
    int cg = 0, co = 0;
    walk_cells(
        P, D, cells, p4, xa, ya, za, 2.0 * fmax(ha, hnew),
        [&](const CellRange& cr, double g2) {
            double hc = 2.0 * fmax(ha, cr.hmax);
            return g2 < hc * hc;
        },
        [&](int32_t b, const Pos4& q) {
            if (b == a) return;
            double dx, dy, dz;
            double r2 = disp(P, xa, ya, za, q.x, q.y, q.z, dx, dy, dz);
            if (r2 < Ra2) {
                if (cg < ng) list[lpos(a, cg, ng)] = b;
                ++cg;
            } else {
                double hb2 = 2.0 * fmax(ha, q.h);
                if (r2 < hb2 * hb2) {
                    if (co < ng) list[lpos(a, ng - 1 - co, ng)] = b;
                    ++co;
                }
            }
        });
    nc[a] = cg;
    ns[a] = cg + co;
    if (cg + co > ng) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
}

// squared FP32 distance of two walk records, minimum image on the axes of kPer.
// It may fuse multiply-adds: the widening factor of the reach covers its FP32
// rounding either way
template <int kPer>
__device__ __forceinline__ float walk_r2(const Domain& D, float xa, float ya, float za, float xb,
                                         float yb, float zb)
{
#pragma clang fp contract(fast)
    // minimum image without branches: the shift is 0 on open axes
    float d[3] = {xb - xa, yb - ya, zb - za};
#pragma unroll
    for (int c = 0; c < 3; ++c)
        if (kPer & (1 << c)) d[c] = fmaf(-D.wrap[c], rintf(d[c] * D.wrap_inv[c]), d[c]);
    return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
}

// ---------------------------------------------------------------- fused step
// Candidates: every b != a with r^2 < (2 kap max(h0_a, h0_b))^2 (kap: the reach
// factor of this pass), by walks of the cells over 16-byte FP32 records.  The test
// runs in FP32 on offsets from the domain's low corner, with
// the reach widened by a bound on their rounding (the cell build stores each
// particle's widened squared reach in its record): each offset is within
// 2^-24 ext of its FP64 value (ext: the largest extent of the key domain); the
// difference, the FP32 box length and the shift by it each add at most as much
// again, and where d/L rounds across +-1/2 the other image is taken, at most
// 2^-24 L farther.  Every displacement component is then within 6 * 2^-24 ext
// and the distance within sqrt(3) times that, below the slack 2^-20 ext added
// to the reach; the factor 1 + 2^-18 on the squared reach covers the FP32
// rounding of r^2 and of the reach itself.  The extras are at most a relative 1e-4 beyond the reach at
// the benchmark sizes, and the passes after this one test every candidate in
// FP64.
//
// Two walks make them.  The short-reach pass over every target (k_candidates)
// shares the tests between neighbouring targets, below; the full-reach refits
// (k_candidates_full) of the few targets whose h left the short reach walk by
// themselves.
//
// A refit has one target or some, and the targets that they mark lie together: a
// target per lane took the serial walk's latency twice over.  A wavefront per
// target has its lanes test a cell each; the flags of 512 slots go to 8 or 64
// wavefronts, so that neighbours go to different ones.  Both launches, with some
// targets grown: 30,011 random particles 296 -> 79 us; the 8 M blob 314 -> 245.  A
// wavefront per target costs several times a lane's share of the machine, so it
// is for 512 slots with few flagged ones (refit_few), a lane each for the others
// (a whole step with all particles grown, by lanes over an unbounded grid and now:
// lattices of 262,144 1.62, 1.49 ms, 1 M 6.04, 5.77; 262,144 random 3.20, 2.61).
// Where a cell near by holds more than kRefitFat particles, as in a clump whose
// cells are sized for its surroundings, a lane's walk takes milliseconds and the
// wavefront's lanes share such cells.
// Both walk a target's cells, and write its candidates, in the same order.
//
// kMode 1: the targets whose h left the short reach (flag 2), marking every
// candidate not so flagged (flag 1); 2: the marked targets (flag 1)
template <int kPer, int kMode>   // bit k of kPer set: axis k periodic
__device__ __forceinline__ void refit_target(
    const Params& P, Domain* __restrict__ dom, const CellRange* __restrict__ cells,
    const Pos4* __restrict__ p4, const Pos4f* __restrict__ pf, int32_t* __restrict__ nk,
    int32_t* __restrict__ cand, double kap, float sc, uint8_t* __restrict__ flag,
    const uint64_t* __restrict__ keys, const uint64_t* __restrict__ reach, int64_t a)
{
    const int lane = (int)threadIdx.x & 63;
    const Pos4 pa = p4[a];
    const Pos4f fa = pf[a];
    const uint32_t far2 = __float_as_uint(fa.r2 * sc);
    const Domain& D = *dom;
    const int nax = D.ncell_axis;
    const uint32_t block = (uint32_t)(keys[a] >> (3 * (kKeyBits - D.reach_level)));
    double hreach = lane < 27 ? reach_neighbor(P, D.reach_level, block, lane, reach) : 0.0;
    for (int o = 16; o > 0; o >>= 1) hreach = fmax(hreach, __shfl_xor(hreach, o, 64));
    hreach = __shfl(hreach, 0, 64);
    const double R = 2.0 * kap * fmax(pa.h, hreach);
    const AxisWalk wx = axis_walk(P, D, 0, pa.x, R);
    const AxisWalk wy = axis_walk(P, D, 1, pa.y, R);
    const AxisWalk wz = axis_walk(P, D, 2, pa.z, R);
    const int ny = wy.hi - wy.lo + 1, nz = wz.hi - wz.lo + 1;
    const int ncells = __builtin_amdgcn_readfirstlane((wx.hi - wx.lo + 1) * ny * nz);
    const int cap = P.cand_cap;
    int k = 0;
    for (int q0 = 0; q0 < ncells; q0 += 64) {
        // this lane's cell, x outermost and rows along z; an empty range out of reach
        const int q = q0 + lane;
        int32_t b0 = 0, e = 0;
        if (q < ncells) {
            const int iz = q % nz, iy = q / nz % ny, ix = q / nz / ny;
            const double gx = axis_gap(wx, wx.lo + ix), gy = axis_gap(wy, wy.lo + iy);
            const double gz = axis_gap(wz, wz.lo + iz);
            const double g2 = gx * gx + gy * gy + gz * gz;
            if (g2 < R * R) {
                const CellRange cr = cells[(spread10(axis_cell(wx, wx.lo + ix, nax)) << 2) |
                                           (spread10(axis_cell(wy, wy.lo + iy, nax)) << 1) |
                                           spread10(axis_cell(wz, wz.lo + iz, nax))];
                const double hc = 2.0 * kap * fmax(pa.h, cr.hmax);
                if (g2 < hc * hc) {
                    b0 = cr.s;
                    e = cr.e;
                }
            }
        }
        // full cells (a clump in cells sized for its surroundings): one after the
        // other, all lanes on its particles, in the same order
        if (__ballot(e - b0 > (int32_t)kRefitFat) != 0u) {
            uint64_t cells_left = __ballot(e > b0);
            while (cells_left != 0u) {
                const int l = __ffsll((unsigned long long)cells_left) - 1;
                cells_left &= cells_left - 1u;
                const int32_t end = __builtin_amdgcn_readlane(e, l);
                for (int32_t s = __builtin_amdgcn_readlane(b0, l); s < end; s += 64) {
                    const int32_t b = s + lane;
                    const Pos4f r = pf[b < end ? b : s];
                    const float r2 = walk_r2<kPer>(D, fa.x, fa.y, fa.z, r.x, r.y, r.z);
                    const bool near = b < end && b != (int32_t)a &&
                                      __float_as_uint(r2) < max(far2, __float_as_uint(r.r2 * sc));
                    const uint64_t m = __ballot(near);
                    const int at = k + __popcll(m & ((uint64_t(1) << lane) - 1u));
                    if (near) {
                        if (kMode == 1 && flag[b] == 0) flag[b] = 1;
                        if (at < cap) cand[lpos8(a, at & ~7, cap) + (at & 7)] = b;
                    }
                    k += __popcll(m);
                }
            }
            continue;
        }
        // its accepted particles: counted first, for their places, then written
        auto each = [&](auto&& take) {
            for (int32_t b = b0; b < e; b += 4) {
                Pos4f r[4];   // (the records have spare entries past the last slot)
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = pf[b + u];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float r2 = walk_r2<kPer>(D, fa.x, fa.y, fa.z, r[u].x, r[u].y, r[u].z);
                    if (b + u < e && b + u != (int32_t)a &&
                        __float_as_uint(r2) < max(far2, __float_as_uint(r[u].r2 * sc)))
                        take(b + u);
                }
            }
        };
        int cnt = 0;
        each([&](int32_t) { ++cnt; });
        int inc = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(inc, o, 64);
            if (lane >= o) inc += up;
        }
        int at = k + inc - cnt;
        each([&](int32_t b) {
            // a neighbour of a grown h redoes its own walk at full reach
            if (kMode == 1 && flag[b] == 0) flag[b] = 1;
            if (at < cap) cand[lpos8(a, at & ~7, cap) + (at & 7)] = b;
            ++at;
        });
        k += __builtin_amdgcn_readlane(inc, 63);
    }
    if (lane == 0) {
        nk[a] = k;
        if (k > cap) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
    }
}

// flagged targets among 512 up to which each has a wavefront: about 16,000 of them
// in all, or half; near full cells 96, where the lanes' walks of 512 targets take as
// long (8 wavefronts, 150 cycles a particle) as so many wavefronts' (600 cycles a
// cell and 9 a particle, some 100 cells of 20,000 particles)
constexpr int kRefitFewFat = 96;
__device__ inline int refit_few(const Params& P)
{
    const int64_t t = (int64_t(1) << 23) / P.n;
    return t > 256 ? 256 : t < 4 ? 4 : (int)t;
}

// wavefronts that share the flags of 512 slots: above a million particles 64 would
// read them for more rounds than they save
__host__ __device__ inline int refit_share(const Params& P)
{
    return P.n <= (int64_t(1) << 20) ? 64 : 8;
}

template <int kPer, int kMode>   // bit k of kPer set: axis k periodic
__global__ __launch_bounds__(kBlock) SPH_WAVES_EXACT(5) void k_candidates_full(
    Params P, Domain* __restrict__ dom, const CellRange* __restrict__ cells,
    const Pos4* __restrict__ p4, const Pos4f* __restrict__ pf, int32_t* __restrict__ nk,
    int32_t* __restrict__ cand, double kap, float sc, uint8_t* __restrict__ flag,
    const uint64_t* __restrict__ keys, const uint64_t* __restrict__ reach,
    const uint64_t* __restrict__ fullest)
{
    if (dom->refit == 0u) return;
    // a bounded grid: a launch that finds nothing to do costs its workgroups'
    // start (31,250 of them at 8 M particles: 110-190 us); an XCD's workgroups
    // take neighbouring slots, which share its L2
    constexpr uint32_t kWant = kMode == 1 ? 2u : 1u;
    const int64_t nt = (P.n + 511) / 512;
    const int share = refit_share(P);
    const int lane = (int)threadIdx.x & 63;
    // candidates are staged in LDS, column per lane, and written out in
    // whole chunks of 8 (two 16-byte stores per lane)
    __shared__ int32_t stage[8][kBlock];
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    const int64_t w0 = xcd_block(gridDim.x) * (kBlock / 64) +
                       __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int64_t it = w0; it < nt * share; it += waves) {
        const int64_t s0 = it / share * 512;
        const int g = (int)(it % share);
        // this lane's 8 of the 512 flags (the array has room for whole words)
        uint64_t f = 0u;
        if (s0 + 8 * lane + 8 <= P.n) {
            f = *(const uint64_t*)(flag + s0 + 8 * lane);
        } else {
            for (int i = 0; i < 8; ++i)
                if (s0 + 8 * lane + i < P.n) f |= (uint64_t)flag[s0 + 8 * lane + i] << (8 * i);
        }
        int mine = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) mine += ((uint32_t)(f >> (8 * i)) & 0xffu) == kWant ? 1 : 0;
        const uint64_t any = __ballot(mine > 0);
        if (any == 0u) continue;
        int found = mine;
        for (int o = 32; o > 0; o >>= 1) found += __shfl_xor(found, o, 64);
        const int one = __ffsll((unsigned long long)any) - 1;   // a lane with a flagged target
        const uint32_t near = (uint32_t)(keys[s0 + 8 * one] >> (3 * (kKeyBits - dom->reach_level)));
        const bool fat = lane < 27 && block_neighbor(P, dom->reach_level, near, lane, fullest) > 0u;
        if (found <= (__ballot(fat) != 0u ? max(refit_few(P), kRefitFewFat) : refit_few(P))) {
            // one target after the other, the wavefront's lanes on its cells
            uint64_t todo = __ballot(((uint32_t)(f >> (8 * (g & 7))) & 0xffu) == kWant &&
                                     (share == 8 || (lane & 7) == g >> 3));
            while (todo != 0u) {
                const int l = __ffsll((unsigned long long)todo) - 1;
                todo &= todo - 1u;
                refit_target<kPer, kMode>(P, dom, cells, p4, pf, nk, cand, kap, sc, flag, keys,
                                          reach, s0 + 8 * l + (g & 7));
            }
            continue;
        }
        // a lane each: 8 of the wavefronts take 64 slots, others from round to round
        // (a round advances a wavefront by waves / share sets of 512)
        const int64_t per = waves / share, turn = it / share % per + it / share / per;
        if (share != 8 && ((g ^ (int)turn) & 7) != 0) continue;
        const int64_t a = s0 + 64 * (share != 8 ? g >> 3 : g) + lane;
        if (a >= P.n || flag[a] != kWant) continue;
        const Domain D = *dom;
        const Pos4 pa = p4[a];
        const Pos4f fa = pf[a];
        const uint32_t far2 = __float_as_uint(fa.r2 * sc);
        // the largest h the target's candidates can have (its block's bound)
        const uint32_t block = (uint32_t)(keys[a] >> (3 * (kKeyBits - D.reach_level)));
        double hreach = 0.0;
        for (int i = 0; i < 27; ++i)
            hreach = fmax(hreach, reach_neighbor(P, D.reach_level, block, i, reach));
        const int cap = P.cand_cap;
        const int t = threadIdx.x;
        const int32_t self = (int32_t)a;
        int k = 0;
        walk_cells(
            P, D, cells, pf, pa.x, pa.y, pa.z, 2.0 * kap * fmax(pa.h, hreach),
            [&](const CellRange& cr, double g2) {
                double hc = 2.0 * kap * fmax(pa.h, cr.hmax);
                return g2 < hc * hc;
            },
            [&](int32_t b, const Pos4f& q) {
                // r < 2 kap max(h_a, h_b) (+ slack): r^2 below either widened
                // squared reach (the records hold the short ones, scaled up by sc).
                // All three are non-negative floats, whose order is that of their
                // bit patterns as unsigned integers: one integer max and one
                // compare (a float max quiets NaNs first, one more instruction).
                const float r2 = walk_r2<kPer>(D, fa.x, fa.y, fa.z, q.x, q.y, q.z);
                const bool near = __float_as_uint(r2) < max(far2, __float_as_uint(q.r2 * sc));
                if (near & (b != self)) {
                    // a neighbour of a grown h redoes its own walk at full reach
                    if (kMode == 1 && flag[b] == 0) flag[b] = 1;
                    if (k < cap) {
                        stage[k & 7][t] = b;
                        if ((k & 7) == 7) {
                            int4* dst = (int4*)(cand + lpos8(a, k & ~7, cap));
                            dst[0] = make_int4(stage[0][t], stage[1][t], stage[2][t], stage[3][t]);
                            dst[1] = make_int4(stage[4][t], stage[5][t], stage[6][t], stage[7][t]);
                        }
                    }
                    ++k;
                }
            });
        if (k < cap && (k & 7) != 0) {   // the partial last chunk
            int4* dst = (int4*)(cand + lpos8(a, k & ~7, cap));
            dst[0] = make_int4(stage[0][t], stage[1][t], stage[2][t], stage[3][t]);
            dst[1] = make_int4(stage[4][t], stage[5][t], stage[6][t], stage[7][t]);
        }
        nk[a] = k;
        if (k > cap) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
    }
}

// ------------------------------------------------ the short-reach pass
// A wavefront takes 16 consecutive targets (neighbours in Morton order) and
// walks the cells around their bounding box once for all of them.  The lanes
// test 64 cells at a time and queue the particles of the cells in reach; every
// 128 queued particles are tested against the 16 targets by matrix
// instructions: with positions relative to the group's centre,
//   r^2 - R^2 = -2 a.b + (|b|^2 [- R_b^2]) + (|a|^2 [- R_a^2])
// is a product over k = (x, y, z, 1) plus the accumulator's start, so two
// v_mfma_f32_16x16x4_f32 give 256 pairs' r^2 - R_b^2 and r^2 - R_a^2; the sign
// bit of either accepts the pair (two vector instructions per pair-register).
//
// Lanes: j = lane % 16 is the target, s = lane / 16 one of four streams of the
// queue.  In the product's result lane (j, s) holds rows 4 s .. 4 s + 3 of the
// tile for target j.  A window's entry u takes position p = 32 s + i, stream
// s = (u / 4) % 4: runs of 4 spread the accepted entries, which cluster along
// the queue, over the streams (a lane's bit loop runs ~45 times per group so,
// 60 with runs of 8; 23 is the mean).
//
// What bounds it: vector instructions (about two thirds of its time at four
// wavefronts per SIMD, which is what its 9.9 KB of LDS and 128 registers
// allow; three wavefronts 10.5 ms, four 9.0 at 15.6 M particles).  One target
// per lane spent ~12 instructions on each of ~930 record slots per target,
// lanes idling while a neighbour finished a longer cell, and left small sizes
// with too few wavefronts.  Before -> now, per walk: 1,000 particles 266 -> 44
// us, 8,000 281 -> 37 us, 1 M (3.8 per cell) 953 -> 490 us, 8 M clustered 8.1
// -> 5.4 ms, 15.6 M (7.4 per cell) 9.3 -> 9.0 ms.  32 targets per wavefront
// tests fewer particles per target but fits half the wavefronts (9.7 ms).
//
// Rounding of the expanded form: every term is at most M^2 in size, M the
// largest distance from the centre (half the bounding box's diagonal, the reach
// and a cell's diagonal), and fewer than 32 roundings of 2^-24 enter; the
// squared reach is widened by 2^-18 M^2.  Where that is not small against it
// (more than 2^-10 of it), or where a periodic box is so narrow that the image
// nearest to the centre need not be the one nearest to the target, the wavefront
// tests its pairs by differences as the refit walk does.
//
// kSplit wavefronts share a group where the chip would be idle (a wavefront alone
// waits for its loads and LDS for most of its time): each takes a quarter of the
// cells in order and keeps what it accepts in its own LDS, and the lists are the
// shares one after the other.  If one share does not fit, the first wavefront
// does the group over by itself.  One wavefront -> four, per walk: lattices of
// 1,000 / 4,096 / 8,000 / 13,824 particles 45.7 -> 19.5, 22.3 -> 13.5, 37.7 ->
// 20.5, 35.2 -> 27.4 us, random 3,001 / 10,007 / 20,011: 87 -> 35, 49 -> 27, 57 ->
// 42 us; a lattice of 32,768 32.5 -> 39.9 us (the wavefronts exceed the slots):
// the line lies between.  Two: 61 us at 1,000 (shares that do not fit), eight: 18.1
// there, but 27 at 8,000.  Queues of 640 and 136 places per target made 30,011
// random particles do most groups twice (98 us, 56 with 1,024 and 168).
constexpr int kWalkSplit = 4;
constexpr int64_t kWalkSplitN = 24576;
constexpr int kWalkT = 16;              // targets per wavefront
constexpr int kWalkWin = 128;           // queue entries tested at a time
constexpr int kWalkRow = 36;            // LDS stride of a stream's 32 records
constexpr int kWalkComp = 4 * kWalkRow; // and of a component: both conflict-free

template <int kSplit>
struct alignas(16) WalkLds {
    // entries kept before the lists are written out, and accepted ones staged per
    // target; wavefronts that share a group hold all of theirs
    static constexpr int kWalkQueue = kSplit > 1 ? 1024 : 640;
    static constexpr int kWalkList = kSplit > 1 ? 168 : kWalkWin + 8;
    uint16_t list[kWalkT][kWalkList];   // accepted entries, as queue indices
    uint32_t queue[kWalkQueue];         // particle slots, in queue order
    float rec[5][kWalkComp];   // x, y, z, |b|^2 - R_b^2 (or R_b^2), |b|^2 (or 1)
    int32_t self[kWalkT];      // window position of the target itself, or -1
};

// the window entry at position p = 32 s + i; kOrder: entry p itself, so that the
// lists keep the queue's order
template <bool kOrder>
__device__ __forceinline__ int walk_entry(int p)
{
    const int s = p >> 5, i = p & 31;
    return kOrder ? p : ((i >> 2) << 4) | (s << 2) | (i & 3);
}

template <int kCtrl>
__device__ __forceinline__ float row_ror(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                         0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
// minimum / maximum over the 16 lanes of a row (row rotations by 8, 4, 2, 1)
__device__ __forceinline__ float row_min(float v)
{
    v = fminf(v, row_ror<0x128>(v));
    v = fminf(v, row_ror<0x124>(v));
    v = fminf(v, row_ror<0x122>(v));
    return fminf(v, row_ror<0x121>(v));
}
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, row_ror<0x128>(v));
    v = fmaxf(v, row_ror<0x124>(v));
    v = fmaxf(v, row_ror<0x122>(v));
    return fmaxf(v, row_ror<0x121>(v));
}

__device__ __forceinline__ float uniform(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

template <int kPer, bool kOrder, int kSplit>
__global__ __launch_bounds__(64 * kSplit) SPH_WAVES_EXACT(kSplit > 1 ? 3 : SPH_WAVES_CAND) void k_candidates(
    Params P, Domain* __restrict__ dom, const CellRange* __restrict__ cells,
    const Pos4* __restrict__ p4, const Pos4f* __restrict__ pf, int32_t* __restrict__ nk,
    int32_t* __restrict__ cand, double kap, const uint64_t* __restrict__ keys,
    const uint64_t* __restrict__ reach, bool stage)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    constexpr int kWalkQueue = WalkLds<kSplit>::kWalkQueue, kWalkList = WalkLds<kSplit>::kWalkList;
    __shared__ WalkLds<kSplit> lds[kSplit];
    __shared__ int parts_k[kSplit][kWalkT];
    const int64_t nb = (P.n + kWalkT - 1) / kWalkT;
    const int64_t lb = xcd_block(nb);
    if (lb < 0) return;
    if (stage) kap = dom->stage_reach;
    if (!(kap > 0.0)) return;
    const int wv = kSplit > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
    WalkLds<kSplit>& S = lds[wv];
    const int lane = (int)threadIdx.x & 63, j = lane & 15, s = lane >> 4;
    const int64_t a0 = lb * kWalkT;
    const bool live = a0 + j < P.n;
    const int64_t a = live ? a0 + j : P.n - 1;
    const int cap = P.cand_cap;
    const int nax = dom->ncell_axis, level = dom->level;
    // (every FP32 length here is in the walk's unit)
    const float slack = dom->walk_slack;
    const double unit = dom->walk_scale;
    float ce[3], inv[3], wl[3], wi[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        ce[x] = (float)(dom->cell[x] * unit);
        inv[x] = ce[x] > 0.0f ? 1.0f / ce[x] : 0.0f;
        wl[x] = dom->wrap[x];
        wi[x] = dom->wrap_inv[x];
    }
    const Pos4f fa = pf[a];
    const float k2 = up_f32(2.0 * kap);
    const float ha = up_f32(p4[a].h * unit);
    // targets of one block of 4 x 4 x 4 cells are walked together
    const int glevel = level > 2 ? level - 2 : 0, rlevel = dom->reach_level;
    const uint32_t block = (uint32_t)(keys[a] >> (3 * (kKeyBits - glevel)));

    int k = 0;         // accepted candidates of target j (the same in its four lanes)
    int flushed = 0;   // of them written out (whole chunks)
    int qbase = 0;     // start of the open window in the queue
    int fill = 0;      // entries in it
    int parts = kSplit;   // wavefronts that share the cells
    bool over = false;    // more than this one's share of the LDS holds

    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); };
    // writes the staged entries out in chunks of 8 (two 16-byte stores per
    // lane); an incomplete chunk only at the end, else it stays staged
    auto flush = [&](bool last) {
        fence();
        uint16_t* list = S.list[j];
        const int pend = k - flushed;
        const int full = pend >> 3, nch = last ? (pend + 7) >> 3 : full;
        for (int c = s; c < nch; c += 4) {
            const uint4 v = *(const uint4*)&list[8 * c];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            int32_t id[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // (entries past the end: any index)
                id[2 * e] = (int32_t)S.queue[min(w[e] & 0xffffu, (uint32_t)kWalkQueue - 1u)];
                id[2 * e + 1] = (int32_t)S.queue[min(w[e] >> 16, (uint32_t)kWalkQueue - 1u)];
            }
            const int at = flushed + 8 * c;
            if (at < cap) {
                int4* dst = (int4*)(cand + lpos8(a, at, cap));
                dst[0] = make_int4(id[0], id[1], id[2], id[3]);
                dst[1] = make_int4(id[4], id[5], id[6], id[7]);
            }
        }
        if (last) return;
        fence();
        if (full > 0)
            for (int e = s; e < pend - 8 * full; e += 4) list[e] = list[8 * full + e];
        flushed += 8 * full;
        fence();
    };

again:
    uint32_t todo = (uint32_t)__ballot(live) & 0xffffu;
    while (todo != 0u) {
        // the group: the targets left that share the first one's block
        const int lead = __ffs((int)todo) - 1;
        const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)block, lead);
        const bool member = ((todo >> j) & 1u) && block == mine;
        todo &= ~((uint32_t)__ballot(member) & 0xffffu);
        const float hm = uniform(row_max(member ? ha : 0.0f));
        const float r2min = uniform(row_min(member ? fa.r2 : INFINITY));
        // the largest h that the targets' candidates can have: of the group's
        // block at the reach level (no finer than the group's) and its neighbours
        float hb = lane < 27 ? up_f32(unit * reach_neighbor(
                                                 P, rlevel, mine >> (3 * (glevel - rlevel)), lane,
                                                 reach))
                             : 0.0f;
        hb = row_max(hb);
        hb = fmaxf(uniform(hb), __builtin_bit_cast(float, __builtin_amdgcn_readlane(
                                                              __builtin_bit_cast(int, hb), 16)));
        const float R = k2 * fmaxf(hm, hb) + 2.0f * slack;
        const float pos[3] = {fa.x, fa.y, fa.z};
        float lo[3], hi[3], ctr[3];
        int c0[3], nc[3];
        bool all[3], wide = false;
        float half2 = 0.0f, diag2 = 0.0f;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            lo[x] = uniform(row_min(member ? pos[x] : INFINITY));
            hi[x] = uniform(row_max(member ? pos[x] : -INFINITY));
            ctr[x] = 0.5f * (lo[x] + hi[x]);
            const float half = 0.5f * (hi[x] - lo[x]);
            half2 += half * half;
            diag2 += ce[x] * ce[x];
            // cells that can hold a point within R of the box (clamped to ints
            // first: positions may be anything)
            int b0 = (int)fminf(fmaxf(floorf((lo[x] - R) * inv[x]), -4096.0f), 4096.0f);
            int b1 = (int)fminf(fmaxf(floorf((hi[x] + R) * inv[x]), -4096.0f), 4096.0f);
            all[x] = false;
            if (!(ce[x] > 0.0f)) {
                b0 = b1 = 0;
                all[x] = true;
            } else if (kPer & (1 << x)) {
                if (b1 - b0 + 1 >= nax) {
                    b0 = 0;
                    b1 = nax - 1;
                    all[x] = true;
                }
                b0 = max(b0, -nax);
                b1 = min(b1, 2 * nax - 1);
                // the nearest image to the centre is the nearest to every
                // target when no pair in reach spans half the box
                wide = wide || !(half + R < 0.49f * wl[x]);
            } else {
                b0 = min(max(b0, 0), nax - 1);
                b1 = min(max(b1, 0), nax - 1);
            }
            c0[x] = __builtin_amdgcn_readfirstlane(b0);
            nc[x] = __builtin_amdgcn_readfirstlane(b1 - b0 + 1);
        }
        const float M = sqrtf(half2) + R + sqrtf(diag2);
        const float e2 = M * M * 0x1p-18f;
        const bool product = __builtin_amdgcn_readfirstlane(!wide && e2 < 0x1p-10f * r2min) != 0;
        // this lane's share of the targets' matrix, and the accumulators' starts (a
        // target at no position is infinitely far: the products hold no NaN, whose
        // sign bit would accept)
        const float ax = fa.x - ctr[0], ay = fa.y - ctr[1], az = fa.z - ctr[2];
        const float r2a = ax * ax + ay * ay + az * az;
        const bool placed = r2a < INFINITY;
        const float a2 = placed ? r2a : INFINITY;
        const float comp = s == 0 ? -2.0f * ax : s == 1 ? -2.0f * ay : -2.0f * az;
        const float bmat = s == 3 ? 1.0f : placed ? comp : 0.0f;
        const float accA = a2 - (fa.r2 + e2);

        // tests the open window's first nv entries against the targets
        auto test = [&](int nv) {
            if (lane < kWalkT) S.self[lane] = -1;
            fence();
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int p = lane + 64 * half;
                const int u = walk_entry<kOrder>(p);
                const bool ok = u < nv;
                const int32_t id = ok ? (int32_t)S.queue[qbase + u] : 0;
                const Pos4f q = pf[id];
                float x = q.x, y = q.y, z = q.z, w = q.r2, w2 = ok ? 1.0f : 0.0f;
                if (product) {
                    x -= ctr[0];
                    y -= ctr[1];
                    z -= ctr[2];
                    if (kPer & 1) x = fmaf(-wl[0], rintf(x * wi[0]), x);
                    if (kPer & 2) y = fmaf(-wl[1], rintf(y * wi[1]), y);
                    if (kPer & 4) z = fmaf(-wl[2], rintf(z * wi[2]), z);
                    w2 = fmaf(z, z, fmaf(y, y, x * x));
                    w = w2 - (w + e2);
                    // past the end, and at no position: an infinite distance,
                    // which no reach of any size accepts (an accepted place past
                    // the end would name whatever the queue holds there)
                    const bool there = ok && w2 < INFINITY;
                    x = there ? x : 0.0f;
                    y = there ? y : 0.0f;
                    z = there ? z : 0.0f;
                    w = there ? w : INFINITY;
                    w2 = there ? w2 : INFINITY;
                }
                const int at = (p >> 5) * kWalkRow + (p & 31);
                S.rec[0][at] = x;
                S.rec[1][at] = y;
                S.rec[2][at] = z;
                S.rec[3][at] = w;
                S.rec[4][at] = w2;
                const uint32_t own = (uint32_t)(id - (int32_t)a0);
                if (ok && own < (uint32_t)kWalkT) S.self[own] = p;
            }
            fence();
            uint32_t m = 0u;
            if (product) {
                // row j of tile t: stream j / 4, entry 4 t + j % 4; component s
                const float* col = &S.rec[s][(j >> 2) * kWalkRow + (j & 3)];
                const float* col4 = &S.rec[4][(j >> 2) * kWalkRow + (j & 3)];
                const v4f startB = {a2, a2, a2, a2};
                const v4f startA = {accA, accA, accA, accA};
#pragma unroll 4
                for (int t = 0; t < kWalkWin / 16; ++t) {
                    const float b1 = col[4 * t];
                    const float b2 = s == 3 ? col4[4 * t] : b1;
                    const v4f dB =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(b1, bmat, startB, 0, 0, 0);
                    const v4f dA =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(b2, bmat, startA, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        m = __builtin_amdgcn_alignbit(
                            m, __float_as_uint(dA[r]) | __float_as_uint(dB[r]), 31);
                }
            } else {
                const uint32_t far2 = __float_as_uint(fa.r2);
#pragma unroll 2
                for (int e = 0; e < 32; ++e) {
                    const int at = s * kWalkRow + e;
                    const float r2 = walk_r2<kPer>(*dom, fa.x, fa.y, fa.z, S.rec[0][at],
                                                   S.rec[1][at], S.rec[2][at]);
                    const bool near =
                        __float_as_uint(r2) < max(far2, __float_as_uint(S.rec[3][at])) &&
                        S.rec[4][at] != 0.0f;
                    m = (m << 1) | (near ? 1u : 0u);
                }
            }
            const int own = S.self[j];
            if (own >= 0 && (own >> 5) == s) m &= ~(0x80000000u >> (own & 31));
            if (!member) m = 0u;
            // places: the target's streams one after the other
            if (kSplit > 1 && over) m = 0u;
            const int c = __popc(m);
            const int n0 = __shfl(c, j, 64), n1 = __shfl(c, j + 16, 64);
            const int n2 = __shfl(c, j + 32, 64), n3 = __shfl(c, j + 48, 64);
            int tot = n0 + n1 + n2 + n3;
            if (__ballot(k - flushed + tot > kWalkList)) {
                if (kSplit > 1 && parts > 1) {
                    over = true;
                    m = 0u;
                    tot = 0;
                } else {
                    flush(false);
                }
            }
            uint16_t* put = &S.list[j][k - flushed + (s > 0 ? n0 : 0) + (s > 1 ? n1 : 0) +
                                       (s > 2 ? n2 : 0)];
            while (m != 0u) {
                const int b = __clz((int)m);
                m &= ~(0x80000000u >> b);
                *put++ = (uint16_t)(qbase + walk_entry<kOrder>(32 * s + b));
            }
            k += tot;
            qbase += nv;
            if (kSplit > 1 && parts > 1 && qbase + kWalkWin > kWalkQueue) {
                over = true;
                qbase = 0;
            } else if (qbase + kWalkWin > kWalkQueue) {
                // the queue starts over: what is staged (fewer than 8 per
                // target) moves to its front
                flush(false);
                const int rem = k - flushed;
                uint32_t id[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    id[h] = s + 4 * h < rem ? S.queue[S.list[j][s + 4 * h]] : 0u;
                fence();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int e = s + 4 * h;
                    if (e < rem) {
                        S.queue[8 * j + e] = id[h];
                        S.list[j][e] = (uint16_t)(8 * j + e);
                    }
                }
                qbase = 8 * kWalkT;
            }
            fence();
        };

        // the cell of this lane in the round of 64 that starts at q0: x
        // outermost and rows along z; an empty range if it is out of reach
        const int ncells = nc[0] * nc[1] * nc[2];
        // (of them this wavefront's: qb .. qe - 1)
        const int qb = parts > 1 ? ncells * wv / kSplit : 0;
        const int qe = parts > 1 ? ncells * (wv + 1) / kSplit : ncells;
        const float ryz1 = 1.0f / (float)(nc[1] * nc[2]), rz1 = 1.0f / (float)nc[2];
        auto load_cell = [&](int q0, CellRange& cr, float& g2) {
            const int q = q0 + lane;
            int ix, iy, iz;
            box_cell(q, nc[0], nc[1], nc[2], ryz1, rz1, ix, iy, iz);
            const int at[3] = {c0[0] + ix, c0[1] + iy, c0[2] + iz};
            uint32_t code = 0u;
            g2 = 0.0f;
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                int c = at[x];
                if (!all[x]) {
                    // distance from the targets' box to the cell along the axis,
                    // less the slack of the FP32 offsets
                    const float l = (float)c * ce[x], h = (float)(c + 1) * ce[x];
                    const float g = fmaxf(fmaxf(l - hi[x], lo[x] - h) - 2.0f * slack, 0.0f);
                    g2 = fmaf(g, g, g2);
                    if (kPer & (1 << x)) {
                        if (c < 0) c += nax;
                        else if (c >= nax) c -= nax;
                    }
                }
                code |= spread10((uint32_t)c) << (2 - x);
            }
            cr = CellRange{0, 0, 0.0};
            if (q < qe && g2 < R * R) cr = cells[code];
        };
        CellRange next;
        float next_g2;
        load_cell(qb, next, next_g2);
        for (int q0 = qb; q0 < qe; q0 += 64) {
            const CellRange cr = next;
            const float Rc = fmaf(k2, fmaxf(hm, up_f32(cr.hmax * unit)), slack);
            const int cnt = next_g2 < Rc * Rc ? cr.e - cr.s : 0;
            if (q0 + 64 < qe) load_cell(q0 + 64, next, next_g2);   // meanwhile
            // places in the queue: an inclusive scan over the lanes
            int inc = cnt;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(inc, o, 64);
                if (lane >= o) inc += up;
            }
            const int total = __builtin_amdgcn_readlane(inc, 63);
            const int start = fill + inc - cnt;
            int w0 = 0;   // the windows completed by this round's cells
            for (;;) {
                const int have = fill + total - w0;
                // (in fours: one cell may fill windows by itself, and its lane alone
                // queues them)
                int i = max(0, w0 - start);
                const int i1 = min(cnt, w0 + kWalkWin - start);
                uint32_t* to = &S.queue[qbase + start - w0];
                for (; i + 4 <= i1; i += 4) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) to[i + v] = (uint32_t)(cr.s + i + v);
                }
                for (; i < i1; ++i) to[i] = (uint32_t)(cr.s + i);
                if (have < kWalkWin && (have == 0 || q0 + 64 < qe)) {
                    fill = have;
                    break;
                }
                test(min(have, kWalkWin));   // a part window after the last cells
                w0 += kWalkWin;
                if (have < kWalkWin) {
                    fill = 0;
                    break;
                }
            }
        }
    }
    if (kSplit > 1 && parts > 1) {
        // the wavefronts' shares one after the other, or the first one alone
        // once more if one of them did not fit
        if (s == 0) parts_k[wv][j] = over ? -1 : k;
        __syncthreads();
        int before = 0, total = 0;
        bool redo = false;
#pragma unroll
        for (int w = 0; w < kSplit; ++w) {
            const int c = parts_k[w][j];
            redo = redo || c < 0;
            before += w < wv ? c : 0;
            total += c;
        }
        if (!redo) {
            if (live)
                for (int e = s; e < k; e += 4)
                    if (before + e < cap)
                        cand[lpos8(a, (before + e) & ~7, cap) + ((before + e) & 7)] =
                            (int32_t)S.queue[S.list[j][e]];
            if (wv == 0 && s == 0 && live) {
                nk[a] = total;
                if (total > cap && !stage) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
            }
            return;
        }
        if (wv != 0) return;
        k = flushed = qbase = fill = 0;
        over = false;
        parts = 1;
        goto again;
    }
    flush(true);
    if (s == 0 && live) {
        nk[a] = k;
        // (a stage call redoes such a target by its own walk)
        if (k > cap && !stage) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
    }
}

// workgroups of the refit walks, as many as are resident at once (with 2,048 a part
// waited for the others to end: 262,144 lattice particles grown, a step of 1.37 ms
// took 1.59 in mixed precision); a multiple of 16, so that a wavefront's share of
// 512 slots stays the same from round to round
constexpr int64_t kRefitGrid = 1280;
// and of the Newton pass after them
constexpr int64_t kRefitNewtonGrid = 2048;

// the candidate pass for the periodic axes of P: mode 0 short reach, 1 and 2
// the full-reach refits
static void launch_candidates(int mode, const Params& P, const Ws& W, double kap, hipStream_t s,
                              bool stage = false)
{
    const int64_t waves = (P.n + 511) / 512 * refit_share(P);
    const int64_t blocks = (waves * 64 + kBlock - 1) / kBlock;
    const int few = (int)(blocks < kRefitGrid ? (blocks + 15) / 16 * 16 : kRefitGrid);
    // the records hold the squared short reach; the full pass scales it by
    // at least (kap / lambda)^2 (the slack scales with it, which only widens)
    const double lam = fmin(kFusedReach, P.kappa);
    const double q = (kap / lam) * (kap / lam) * (1.0 + 0x1p-20);
    float sc = (float)q;
    if ((double)sc < q) sc = nextafterf(sc, INFINITY);
    with_periodic(P, [&](auto per) {
        constexpr int kPer = decltype(per)::value;
        if (mode == 1)
            k_candidates_full<kPer, 1><<<few, kBlock, 0, s>>>(
                P, W.dom, W.cells, W.p4, W.pf, W.nk, W.cand, kap, sc, W.flag, W.keys0, W.reach,
                W.fullest);
        else if (mode == 2)
            k_candidates_full<kPer, 2><<<few, kBlock, 0, s>>>(
                P, W.dom, W.cells, W.p4, W.pf, W.nk, W.cand, kap, sc, W.flag, W.keys0, W.reach,
                W.fullest);
        else if (in_order(P))
            k_candidates<kPer, true, 1><<<grid_xcd((P.n + kWalkT - 1) / kWalkT), 64, 0, s>>>(
                P, W.dom, W.cells, W.p4, W.pf, W.nk, W.cand, kap, W.keys0, W.reach, stage);
        else if (P.n <= kWalkSplitN)
            k_candidates<kPer, false, kWalkSplit>
                <<<grid_xcd((P.n + kWalkT - 1) / kWalkT), 64 * kWalkSplit, 0, s>>>(
                    P, W.dom, W.cells, W.p4, W.pf, W.nk, W.cand, kap, W.keys0, W.reach, stage);
        else
            k_candidates<kPer, false, 1><<<grid_xcd((P.n + kWalkT - 1) / kWalkT), 64, 0, s>>>(
                P, W.dom, W.cells, W.p4, W.pf, W.nk, W.cand, kap, W.keys0, W.reach, stage);
    });
}

// ------------------------------------------------ lanes per target
// The passes over a target's list give it kG neighbouring lanes (4, or 16 at
// small sizes), each taking every kG-th entry or pair of entries, and add the
// lanes' sums up at the end.  A wavefront then runs to the longest of 64 / kG
// lists instead of 64 (in a clumped distribution the longest of 64 is 1.6 times
// the mean), and small problems have enough wavefronts: 8,000 targets make 125
// with one lane each and 2,000 with 16.
//
// one chunk of 8 candidates of slot a (entries at or past cnt read as a itself)
__device__ __forceinline__ void load_chunk(const int32_t* __restrict__ cand, int64_t a, int j0,
                                           int cap, int cnt, int32_t (&bb)[8])
{
    const int4* src = (const int4*)(cand + lpos8(a, j0, cap));
    const int4 lo = src[0], hi = src[1];
    const int32_t v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
    for (int u = 0; u < 8; ++u) bb[u] = (j0 + u < cnt) ? v[u] : (int32_t)a;
}

// This lane's entries of the step that starts at entry j0 of target a: kE in a
// row, those at or past cnt read as a itself
template <int kG>
struct GroupStep {
    static constexpr int kE = kG < 8 ? 8 / kG : 1;   // entries per lane
    static constexpr int kStep = kG * kE;            // entries per target
};
template <int kG>
__device__ __forceinline__ void group_entries(const int32_t* __restrict__ cand, int64_t a, int j0,
                                              int g, int cap, int cnt,
                                              int32_t (&e)[GroupStep<kG>::kE])
{
    constexpr int kE = GroupStep<kG>::kE;
    const int j = j0 + kE * g;
    if constexpr (kG == 1) {
        if (j0 < cnt) {
            load_chunk(cand, a, j0, cap, cnt, e);
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = (int32_t)a;
        }
    } else if constexpr (kE == 2) {
        const int2 v = j < cnt ? *(const int2*)(cand + lpos8(a, j, cap)) : make_int2(0, 0);
        e[0] = j < cnt ? v.x : (int32_t)a;
        e[1] = j + 1 < cnt ? v.y : (int32_t)a;
    } else {
        static_assert(kE == 1, "one or two entries per lane");
        e[0] = j < cnt ? cand[lpos8(a, j, cap)] : (int32_t)a;
    }
}

// x, y, z of candidate b of this lane, gathered by the two lanes of a pair
// together: one 16-byte load per lane fetches the even lane's record (x, y to
// the even lane, z, h to the odd one) and a second the odd lane's, so the two
// loads of a pair touch one line each instead of two per lane; a swap then
// completes each lane's own position.  Both lanes of the pair must be active.
// kNarrow (the records span under 4 GiB): the byte offsets fit 32 bits, so
// each address is one shift-or on a scalar base instead of a 64-bit
// sign-extend, shift and add (Newton 27.0 -> 26.0 ms at 64 M particles; the
// same form in the list filter made it slower, 21.9 -> 29.0 ms).
template <bool kNarrow>
__device__ __forceinline__ void pair_gather_xyz(const Pos4* __restrict__ p4, int32_t b, int odd,
                                                double& x, double& y, double& z)
{
    const int32_t o = pair_swap(b);
    const int32_t rA = odd ? o : b;   // the even lane's candidate
    const int32_t rB = odd ? b : o;   // the odd lane's candidate
    double2 A, B;
    if constexpr (kNarrow) {
        const char* base = (const char*)p4;
        A = *(const double2*)(base + (((uint32_t)rA << 5) | (uint32_t)(odd << 4)));
        B = *(const double2*)(base + (((uint32_t)rB << 5) | (uint32_t)(odd << 4)));
    } else {
        const double2* half = (const double2*)p4;
        A = half[2 * (int64_t)rA + odd];
        B = half[2 * (int64_t)rB + odd];
    }
    // even lane: A = (x, y) of its own record, B = (x, y) of the odd lane's;
    // odd lane: A = (z, h) of the even lane's record, B = (z, h) of its own
    const double r0 = pair_swap(odd ? A.x : B.x);
    const double r1 = pair_swap(B.y);
    x = odd ? r0 : A.x;
    y = odd ? r1 : A.y;
    z = odd ? B.x : r0;
}

// Newton iterations summing over the candidate list (self term added: S(0) = 1).
// The first kHold candidates of a target are gathered once, their r^2 kept in
// registers for every iteration; longer lists gather the rest again each time.
// Bound by vector FP64 instructions (two fits of 10 and 11 terms per candidate
// and iteration); three wavefronts per SIMD hold the 64 registers of r^2.
// Before (one lane per target, a gather per iteration) -> now: 1,000 particles
// 56 -> 7 us, 1 M 502 -> 402 us, 15.6 M 7.3 -> 6.1 ms, 8 M clustered 5.3 -> 5.0
// ms (8 lanes at four wavefronts: 407 us, 6.5 and 4.5 ms).
constexpr int kHold = 128;
// the fused step's short pass, its refit of the flagged targets, and a stage call
enum { kNewtonStep, kNewtonRefit, kNewtonStage };
template <int kPer, bool kTab, int kG>
__device__ __forceinline__ void update_h_list(const Params& P, Domain* __restrict__ dom,
                                              const int32_t* __restrict__ nk,
                                              const int32_t* __restrict__ cand,
                                              const Pos4* __restrict__ p4, double* __restrict__ h,
                                              double lam, uint8_t* __restrict__ flag, int mode,
                                              int64_t lb)
{
    const bool full = mode == kNewtonRefit;
    constexpr int kE = GroupStep<kG>::kE, kStep = GroupStep<kG>::kStep;
    constexpr int kRuns = kE < 4 ? 4 / kE : 1;   // steps gathered together,
    constexpr int kRecs = kRuns * kE;            // records of a lane
    constexpr int kBat = kRuns * kStep;          // and of its target in them
    constexpr int kHeld = kG > 1 ? kHold : 0;    // (one lane has no room for them)
    constexpr int kTargets = kBlock / kG;
    // lanes past the end shadow the last particle with no candidates, so that
    // both lanes of every pair run the gathers together; in the full-reach pass
    // only the targets whose h left the short reach (flag 2) are live
    const int64_t a0 = lb * kTargets + (int)threadIdx.x / kG;
    const int g = (int)threadIdx.x % kG;
    const int64_t a = a0 < P.n ? a0 : P.n - 1;
    const bool live = a0 < P.n && (!full || flag[a] == 2);
    const int odd = threadIdx.x & 1;
    const Pos4 pa = p4[a];
    const double xa = pa.x, ya = pa.y, za = pa.z;
    const double h0 = pa.h;
    const int cap = P.cand_cap;
    const int cnt = live ? min(nk[a], cap) : 0;
    const int most = wave_max_i(cnt);   // the wavefront's longest list
    // the candidates reach 2 lam max(h0_a, h0_b): exact as long as every
    // iterate stays at or below lam h0 (2 (lam h0) == (2 lam) h0 in FP64)
    const double hlim = lam * h0;
    // (a stage call redoes targets with more candidates than fit, too)
    bool over = mode == kNewtonStage && live && nk[a] > cap;
    double hc = h0;
    auto run = [&](auto narrow) {
        constexpr bool kNarrow = decltype(narrow)::value;
        auto entries = [&](int j0, int32_t (&e)[kRuns][kE]) {
#pragma unroll
            for (int r = 0; r < kRuns; ++r) group_entries<kG>(cand, a, j0 + r * kStep, g, cap, cnt, e[r]);
        };
        // r^2 of this lane's entries from j0, infinite past the end
        auto distances = [&](int j0, const int32_t (&e)[kRuns][kE], double* r2) {
            double qx[kRecs], qy[kRecs], qz[kRecs];
#pragma unroll
            for (int u = 0; u < kRecs; ++u)
                pair_gather_xyz<kNarrow>(p4, e[u / kE][u % kE], odd, qx[u], qy[u], qz[u]);
#pragma unroll
            for (int u = 0; u < kRecs; ++u) {
                double dx, dy, dz;
                const double v = disp_p<kPer>(P, xa, ya, za, qx[u], qy[u], qz[u], dx, dy, dz);
                r2[u] = j0 + (u / kE) * kStep + kE * g + u % kE < cnt ? v : INFINITY;
            }
        };
        double held[kHeld > 0 ? kHeld / kG : 1];
        int32_t e[kRuns][kE];
        if (kHeld > 0) entries(0, e);
#pragma unroll
        for (int i = 0; i < kHeld / kBat; ++i) {
            if (i * kBat >= most) continue;
            int32_t nx[kRuns][kE];
            entries((i + 1) * kBat, nx);   // (past the longest list: no loads)
            distances(i * kBat, e, &held[kRecs * i]);
#pragma unroll
            for (int u = 0; u < kRecs; ++u) e[u / kE][u % kE] = nx[u / kE][u % kE];
        }
        for (int it = 0; it < P.newton_iters; ++it) {
            const double h2 = 2.0 * hc;
            const double R2 = h2 * h2;
            const double tsc = kPiHalfSq / (hc * hc);
            double sS = kG == 1 ? 1.0 : 0.0, sV = 0.0;
            auto add = [&](double r2) {
                if (r2 < R2) {
                    double S, vdS;
                    kern_terms_t<kTab>(P, r2 * tsc, S, vdS);
                    sS += S;
                    sV += vdS;
                }
            };
#pragma unroll
            for (int i = 0; i < kHeld / kBat; ++i) {
                if (i * kBat >= most) continue;
#pragma unroll
                for (int u = 0; u < kRecs; ++u) add(held[kRecs * i + u]);
            }
            for (int j0 = kHeld; j0 < most; j0 += kBat) {
                double r2[kRecs];
                entries(j0, e);
                distances(j0, e, r2);
#pragma unroll
                for (int u = 0; u < kRecs; ++u) add(r2[u]);
            }
            if constexpr (kG > 1) {
                sS = group_sum<kG>(sS) + 1.0;
                sV = group_sum<kG>(sV);
            }
            hc = newton_step(P, hc, h0, sS, sV);
            over = over || hc > hlim;
        }
    };
    if ((uint64_t)P.n * sizeof(Pos4) <= 0xffffffffull) run(std::true_type{});
    else run(std::false_type{});
    if (!live || g != 0) return;
    h[a] = hc;
    // the short pass flags the targets whose h may have missed candidates
    // (2) and clears the others (0); the full-reach pass recomputes the former
    if (!full) flag[a] = over ? 2 : 0;
    if (over) {
        flag_or(&dom->refit, 1u);
    } else if (mode != kNewtonStage) {
        check_cell_range(P, dom, hc);
    }
}

template <int kPer, bool kTab, int kG>
__global__ __launch_bounds__(kBlock) SPH_WAVES_EXACT(kG == 1 ? 4 : 3) void k_update_h_list(
    Params P, Domain* __restrict__ dom, const int32_t* __restrict__ nk,
    const int32_t* __restrict__ cand, const Pos4* __restrict__ p4, double* __restrict__ h,
    double lam, uint8_t* __restrict__ flag, int mode)
{
    constexpr int kTargets = kBlock / kG;
    const int64_t lb = xcd_block((P.n + kTargets - 1) / kTargets);
    if (mode == kNewtonStage) {
        lam = dom->stage_reach;
        if (!(lam > 0.0)) return;
    }
    if (lb >= 0) update_h_list<kPer, kTab, kG>(P, dom, nk, cand, p4, h, lam, flag, mode, lb);
}
// After the refits: the grown targets redo Newton over their full candidates,
// and the packed positions take the new h (their other fields stand).  A target
// reads only its own packed h, as h0, so each can be replaced as it is done.
template <int kPer, bool kTab, int kG>
__global__ __launch_bounds__(kBlock) SPH_WAVES_EXACT(kG == 1 ? 4 : 3) void k_update_h_list_full(
    Params P, Domain* __restrict__ dom, const int32_t* __restrict__ nk,
    const int32_t* __restrict__ cand, Pos4* p4, double* h, double lam,
    uint8_t* __restrict__ flag)
{
    constexpr int kTargets = kBlock / kG;
    const int64_t nb = (P.n + kTargets - 1) / kTargets;
    if constexpr (kG == 1) {
        // (a workgroup per 256 targets: in a loop 27 registers spill, 680 -> 950 us
        // with all of a 1 M patch grown)
        const int64_t lb = xcd_block(nb);
        const int64_t a = lb * kBlock + threadIdx.x;
        if (lb < 0) return;
        if (dom->refit != 0u && lam > kFusedReach)
            update_h_list<kPer, kTab, 1>(P, dom, nk, cand, p4, h, lam, flag, kNewtonRefit, lb);
        if (a < P.n) p4[a].h = h[a];
        return;
    }
    if (dom->refit != 0u && lam > kFusedReach) {
        for (int64_t bid = blockIdx.x; bid < grid_xcd(nb); bid += gridDim.x) {
            const int64_t lb = xcd_block(nb, bid);
            if (lb < 0) continue;
            const int64_t a = lb * kTargets + (int)threadIdx.x / kG;
            update_h_list<kPer, kTab, kG>(P, dom, nk, cand, p4, h, lam, flag, kNewtonRefit, lb);
            if (a < P.n && (int)threadIdx.x % kG == 0) p4[a].h = h[a];
        }
        return;
    }
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < P.n;
         i += (int64_t)gridDim.x * kBlock)
        p4[i].h = h[i];
}

// exact lists from the candidates with the final h (same layout as k_find_neighbors)
// kDens: also the density sums over the gather members, then rho, Omega and
// the EOS.  Four lanes per target at four wavefronts per SIMD; before (one lane)
// -> now: 1,000 particles 43 -> 7 us, 1 M 540 -> 450 us, 15.6 M 8.0 -> 6.8 ms, 8
// M clustered 8.0 -> 6.0 ms (8 lanes: 491 us, 7.5 and 5.5 ms).
template <bool kDens, int kPer, bool kTab, int kG>
__global__ __launch_bounds__(kBlock) SPH_WAVES_CAP(kG == 1 ? 3 : 4) void k_filter(Params P, Domain* __restrict__ dom,
                                                   const int32_t* __restrict__ nk,
                                                   const int32_t* __restrict__ cand,
                                                   const Pos4* __restrict__ p4,
                                                   int32_t* __restrict__ nc,
                                                   int32_t* __restrict__ ns,
                                                   int32_t* __restrict__ list, DensOut O,
                                                   double* __restrict__ vol,
                                                   PosV* __restrict__ pv)
{
    constexpr int kE = GroupStep<kG>::kE, kStep = GroupStep<kG>::kStep;
    constexpr int kRuns = kE < 4 ? 4 / kE : 1;
    constexpr int kBat = kRuns * kStep;
    constexpr int kTargets = kBlock / kG;
    const int64_t nb = (P.n + kTargets - 1) / kTargets;
    const int64_t lb = xcd_block(nb);
    if (lb < 0) return;
    // lanes past the end shadow the last particle with no candidates, so that
    // both lanes of every pair run the gathers together
    const int64_t a0 = lb * kTargets + (int)threadIdx.x / kG;
    const int g = (int)threadIdx.x % kG;
    const bool live = a0 < P.n;
    const int64_t a = live ? a0 : P.n - 1;
    const int odd = threadIdx.x & 1;
    const Pos4 pa = p4[a];
    const double xa = pa.x, ya = pa.y, za = pa.z, ha = pa.h;
    const double ha2 = 2.0 * ha;
    const double Ra2 = ha2 * ha2;
    const int cap = P.cand_cap;
    const int cnt = live ? min(nk[a], cap) : 0;
    const int most = wave_max_i(cnt);
    const int ng = P.ng_max;
    const double tsc = kPiHalfSq / (ha * ha);
    // self term: S = 1, v dS/dv = 0
    double sS = kDens && kG == 1 ? O.m[a] : 0.0, sD = 3.0 * sS;
    // with equal masses (flagged by the cell build) the mass of every
    // neighbour is slot 0's: no gather
    const bool mvar = !kDens || dom->mass_varies != 0u;
    const double m0 = kDens ? O.m[0] : 0.0;
    int cg = 0, co = 0;   // the target's entries so far (the same in its lanes)
    const int first = (int)(threadIdx.x & 63u) & ~(kG - 1);   // the group's first lane
    const uint32_t below = (1u << g) - 1u;
    auto group_bits = [&](bool v) {
        return (uint32_t)(__ballot(v) >> first) & ((1u << kG) - 1u);
    };
    int32_t e[kRuns][kE];
#pragma unroll
    for (int r = 0; r < kRuns; ++r) group_entries<kG>(cand, a, r * kStep, g, cap, cnt, e[r]);
    for (int j0 = 0; j0 < most; j0 += kBat) {
        Pos4 q[kRuns][kE];
        double mb[kRuns][kE];
        int32_t bb[kRuns][kE];
        // one straight run of loads per case (a test per load would split the
        // batch into blocks and serialise its gathers)
        if (mvar) {
#pragma unroll
            for (int r = 0; r < kRuns; ++r)
#pragma unroll
                for (int u = 0; u < kE; ++u) {
                    q[r][u] = pair_gather32(p4, e[r][u], odd);
                    if (kDens) mb[r][u] = O.m[e[r][u]];
                }
        } else {
#pragma unroll
            for (int r = 0; r < kRuns; ++r)
#pragma unroll
                for (int u = 0; u < kE; ++u) {
                    q[r][u] = pair_gather32(p4, e[r][u], odd);
                    mb[r][u] = m0;
                }
        }
#pragma unroll
        for (int r = 0; r < kRuns; ++r) {
#pragma unroll
            for (int u = 0; u < kE; ++u) bb[r][u] = e[r][u];
            group_entries<kG>(cand, a, j0 + kBat + r * kStep, g, cap, cnt, e[r]);
        }
#pragma unroll
        for (int r = 0; r < kRuns; ++r) {
            bool in[kE], sym[kE];
            double r2[kE];
            bool anysym = false;
#pragma unroll
            for (int u = 0; u < kE; ++u) {
                const bool ok = j0 + r * kStep + kE * g + u < cnt;
                double dx, dy, dz;
                r2[u] = disp_p<kPer>(P, xa, ya, za, q[r][u].x, q[r][u].y, q[r][u].z, dx, dy, dz);
                const double hb2 = 2.0 * fmax(ha, q[r][u].h);
                in[u] = ok && r2[u] < Ra2;
                sym[u] = ok && !in[u] && r2[u] < hb2 * hb2;
                anysym = anysym || sym[u];
            }
            // places in candidate order: entry (g, u) follows those of the
            // lanes before it
            auto put = [&](const bool (&yes)[kE], int base, bool front) {
                uint32_t bits[kE];
                int before = 0, tot = 0;
#pragma unroll
                for (int u = 0; u < kE; ++u) {
                    bits[u] = group_bits(yes[u]);
                    before += __popc(bits[u] & below);
                    tot += __popc(bits[u]);
                }
#pragma unroll
                for (int u = 0; u < kE; ++u) {
                    if (yes[u]) {
                        const int k = base + before++;
                        if (k < ng) {
                            list[lpos(a, front ? k : ng - 1 - k, ng)] = bb[r][u];
                            if (front && kDens) {
                                double S, vdS;
                                kern_terms_t<kTab>(P, r2[u] * tsc, S, vdS);
                                sS += mb[r][u] * S;
                                sD += mb[r][u] * (3.0 * S + vdS);
                            }
                        }
                    }
                }
                return tot;
            };
            cg += put(in, cg, true);
            if (__ballot(anysym)) co += put(sym, co, false);
        }
    }
    if constexpr (kDens && kG > 1) {
        sS = group_sum<kG>(sS) + O.m[a];
        sD = group_sum<kG>(sD) + 3.0 * O.m[a];
    }
    if (!live || g != 0) return;
    nc[a] = cg;
    ns[a] = cg + co;
    // (a stage call redoes targets with more candidates than fit)
    if (!kDens && nk[a] > cap) flag_or(&dom->refit, 1u);
    if (cg + co > ng) set_err(dom, SPH_ERRBIT_NEIGHBOR_OVERFLOW);
    if (kDens) {
        const double rho = finish_density(P, dom, O, a, ha, sS, sD);
        if (pv) {   // the IAD pass's records
            const double v = O.m[a] / rho;
            vol[a] = v;
            pv[a] = PosV{xa, ya, za, v};
        }
    }
}

}  // namespace

int candidate_capacity(int ng_max)
{
    // the candidate reach is at most kFusedKappaMax times the list reach:
    // kFusedKappaMax^3 times the volume, with 25% headroom
    double c = ng_max * kFusedKappaMax * kFusedKappaMax * kFusedKappaMax * 1.25;
    int cap = ((int)ceil(c) + 7) & ~7;   // whole chunks of 8
    return cap > 8192 ? 8192 : cap;
}

// The group walk of a stage call at the present h, in Q's capacity: the candidates
// within 2 max(h_a, h_b), or (ns samples) within the reach that the samples choose.
static hipError_t stage_candidates(const Params& Q, const Layout& L, const Ws& W,
                                   const sph_particles* p, int ns, hipStream_t s)
{
    const int64_t nb = (Q.n + kBlock - 1) / kBlock;
    const int64_t cb = (L.ncells_cap + kBlock - 1) / kBlock;
    const int mb = (int)(cb < kHmaxGrid ? cb : kHmaxGrid);
    k_stage_begin<<<nb, kBlock, 0, s>>>(Q, W.dom, p->x, p->y, p->z, p->h, W.p4, W.reach,
                                        L.nreach);
    if (ns > 0)
        k_cells_max<true><<<mb + ns, kBlock, 0, s>>>(Q, W.dom, W.cells, p->h, L.ncells_cap, W.p4,
                                                     mb);
    else
        k_cells_max<false><<<mb, kBlock, 0, s>>>(Q, W.dom, W.cells, p->h, L.ncells_cap, W.p4, mb);
    k_stage_reach<<<nb, kBlock, 0, s>>>(Q, W.dom, W.cells, L.ncells_cap, ns, W.p4, W.pf, W.reach);
    launch_candidates(0, Q, W, 1.0, s, true);
    return hipGetLastError();
}

// Newton over one walk's candidates, at the reach that stage_reach chooses, and by
// cell walks for the targets it flags: those whose h left that reach, or with more
// candidates than fit.  The call with a walk per iteration and target -> now, two
// iterations: lattices of 4,096 317 -> 51 us (64 wavefronts), 262,144 523 -> 300,
// 1 M random 3.49 -> 1.48 ms; all h short by 4%: 293 -> 63, 442 -> 427 us, 3.31 ->
// 2.20 ms.  Where the order of the sums shows (in_order) every target keeps the
// cell walks.
hipError_t launch_update_h(const Params& P, const Layout& L, const Ws& W, sph_particles* p,
                           hipStream_t s, bool pack)
{
    if (P.newton_iters == 0) return hipSuccess;
    const int64_t nb = (P.n + kBlock - 1) / kBlock;
    if (in_order(P)) {
        if (pack) {
            hipError_t e = launch_pack_p4(P, W, p, s);
            if (e != hipSuccess) return e;
        }
        k_update_h<<<grid_xcd(nb), kBlock, 0, s>>>(P, W.dom, W.cells, W.p4, p->h, nullptr);
        return hipGetLastError();
    }
    Params Q = P;
    Q.cand_cap = L.cand_cap;
    hipError_t e = stage_candidates(Q, L, W, p, stage_samples(P.n), s);
    if (e != hipSuccess) return e;
    with_periodic(Q, [&](auto per) {
        with_table(Q, [&](auto tab) {
            constexpr int kPer = decltype(per)::value;
            constexpr bool kTab = decltype(tab)::value;
            with_lanes<4>(Q, [&](auto lanes) {
                constexpr int kG = decltype(lanes)::value;
                k_update_h_list<kPer, kTab, kG><<<grid_lanes(Q, kG), kBlock, 0, s>>>(
                    Q, W.dom, W.nk, W.cand, W.p4, p->h, 0.0, W.flag, kNewtonStage);
            });
        });
    });
    k_update_h<<<grid_xcd(nb), kBlock, 0, s>>>(P, W.dom, W.cells, W.p4, p->h, W.flag);
    return hipGetLastError();
}

// Lists from one walk's candidates at h (always repacked: h may have changed since
// the cell build), and by a cell walk each for targets with more candidates than
// fit, whose counts must be true all the same.  One target per lane took 613 us at
// 125,000 random particles and 198 us at 4,096 on a lattice; this takes 200 and 50.
hipError_t launch_find_neighbors(const Params& P, const Layout& L, const Ws& W,
                                 const sph_particles* p, hipStream_t s)
{
    const int64_t nb = (P.n + kBlock - 1) / kBlock;
    if (in_order(P)) {
        hipError_t e = launch_pack_p4(P, W, p, s);
        if (e != hipSuccess) return e;
        k_hmax_begin<<<1, 1, 0, s>>>(W.dom);
        const int64_t cb = (L.ncells_cap + kBlock - 1) / kBlock;
        const int mb = (int)(cb < kHmaxGrid ? cb : kHmaxGrid);
        k_cells_max<false><<<mb, kBlock, 0, s>>>(P, W.dom, W.cells, p->h, L.ncells_cap, W.p4, mb);
        k_check_range<<<1, 1, 0, s>>>(P, W.dom);
        k_find_neighbors<<<grid_xcd(nb), kBlock, 0, s>>>(P, W.dom, W.cells, W.p4, W.nc, W.ns,
                                                         W.list, nullptr, 0);
        return hipGetLastError();
    }
    Params Q = P;
    Q.cand_cap = L.cand_cap;
    hipError_t e = stage_candidates(Q, L, W, p, 0, s);
    if (e != hipSuccess) return e;
    k_check_range<<<1, 1, 0, s>>>(P, W.dom);
    with_periodic(Q, [&](auto per) {
        constexpr int kPer = decltype(per)::value;
        with_lanes<4>(Q, [&](auto lanes) {
            constexpr int kG = decltype(lanes)::value;
            k_filter<false, kPer, false, kG><<<grid_lanes(Q, kG), kBlock, 0, s>>>(
                Q, W.dom, W.nk, W.cand, W.p4, W.nc, W.ns, W.list, DensOut{}, nullptr, nullptr);
        });
    });
    k_find_neighbors<<<grid_xcd(nb), kBlock, 0, s>>>(P, W.dom, W.cells, W.p4, W.nc, W.ns, W.list,
                                                     W.nk, L.cand_cap);
    return hipGetLastError();
}

// fused: candidates at h0, Newton over candidates, exact lists and densities at
// the new h.  Expects the packed positions and walk records of the cell build
// (h0 in them).
hipError_t launch_fused_step(const Params& P, const Layout& L, const Ws& W, sph_particles* p,
                             hipStream_t s, const Marks& mk)
{
    const int64_t cb = (L.ncells_cap + kBlock - 1) / kBlock;
    k_cells_reach<<<cb, kBlock, 0, s>>>(P, W.dom, W.cells, p->h, L.ncells_cap, W.reach, W.fullest);
    mk.at(0, s);
    // short reach first; the full-reach pair runs only if an h left it (the
    // kernels read the device flag and return at once when it is clear)
    const double lam = fmin(kFusedReach, P.kappa);
    launch_candidates(0, P, W, lam, s);
    mk.at(1, s);
    if (P.newton_iters > 0) {
        with_periodic(P, [&](auto per) {
            with_table(P, [&](auto tab) {
                constexpr int kPer = decltype(per)::value;
                constexpr bool kTab = decltype(tab)::value;
                with_lanes_m<4>(P, [&](auto lanes) {
                    constexpr int kG = decltype(lanes)::value;
                    k_update_h_list<kPer, kTab, kG><<<grid_lanes(P, kG), kBlock, 0, s>>>(
                        P, W.dom, W.nk, W.cand, W.p4, p->h, lam, W.flag, kNewtonStep);
                });
            });
        });
        if (lam < P.kappa) {
            // targets whose h left the short reach walk again at full reach
            // and mark their candidates, whose symmetric sets may now hold
            // them; the marked targets walk again too (their own h stands),
            // then the grown ones redo Newton over their full candidates
            launch_candidates(1, P, W, P.kappa, s);
            launch_candidates(2, P, W, P.kappa, s);
        }
        const int64_t nb = (P.n + kBlock - 1) / kBlock;
        const int64_t grid = in_order(P) ? grid_xcd(nb) : nb < kRefitNewtonGrid ? nb : kRefitNewtonGrid;
        with_periodic(P, [&](auto per) {
            with_table(P, [&](auto tab) {
                constexpr int kPer = decltype(per)::value;
                constexpr bool kTab = decltype(tab)::value;
                if (in_order(P))
                    k_update_h_list_full<kPer, kTab, 1><<<grid, kBlock, 0, s>>>(
                        P, W.dom, W.nk, W.cand, W.p4, p->h, P.kappa, W.flag);
                else
                    k_update_h_list_full<kPer, kTab, 4><<<grid, kBlock, 0, s>>>(
                        P, W.dom, W.nk, W.cand, W.p4, p->h, P.kappa, W.flag);
            });
        });
    }
    mk.at(2, s);
    const DensOut O{p->m, p->u, p->p_ref, p->rho_ref, p->rho, p->omega, p->p, p->c};
    PosV* const pv = P.precision == SPH_FP64 ? W.pv : nullptr;
    with_periodic(P, [&](auto per) {
        with_table(P, [&](auto tab) {
            constexpr int kPer = decltype(per)::value;
            constexpr bool kTab = decltype(tab)::value;
            with_lanes_m<4>(P, [&](auto lanes) {
                constexpr int kG = decltype(lanes)::value;
                k_filter<true, kPer, kTab, kG><<<grid_lanes(P, kG), kBlock, 0, s>>>(
                    P, W.dom, W.nk, W.cand, W.p4, W.nc, W.ns, W.list, O, W.vol, pv);
            });
        });
    });
    return hipGetLastError();
}

}  // namespace sph
