// One wave per workgroup.  Lane u owns a unit: a product x^a y^b and up to
// four consecutive powers z^c0 .. z^(c0+3) of the same (a, b), so its terms
// share one product x^a (y^b z^c0), each added by one fused multiply-add with
// z^0 .. z^3 (61 units cover the 165 terms of order 8).  Particles are staged
// kChunk = 32 at a time: double x^k and y^b z^c0 in LDS, one row per power, z in
// the lane's register.  In a run the offsets of kBatch = 4 chunks are loaded
// together, in a piece those of the next chunk while the current one is summed.
//
//   k_mp_plan     the first cell of every run, and the pieces of the big cells
//   k_multipoles  a run of consecutive cells of bounded cost (particles plus
//                 a fixed cost per cell) per workgroup; each lane adds its
//                 terms over the run's particles in sorted order and writes a
//                 cell's moments as it passes the cell's end.  Cells of more
//                 than kBig particles are skipped: one workgroup summing them
//                 alone would set the kernel's length; their pieces of kBig
//                 particles, moments in double, are the kernel's first
//                 workgroups.
//   k_mp_combine  adds a cell's pieces in piece order and writes its moments.
// Every moment is a fixed sequence of double operations, so the moments are
// reproducible.
//
// Bound by FP64 issue for about 60 % of the time (counted, 2.1M particles: 15.5 VALU
// instructions a particle, 9 of them its sums, at 4.4 clocks of a SIMD; it spends
// 7.4 on one, with 3.8 waves a SIMD, the rest waiting for LDS, stores and
// barriers).  A particle takes 9 clocks of a CU of LDS; with the four z powers read
// from LDS too that was 24 and set the time.
// 6 KB of LDS a workgroup, so that registers limit the waves (five per SIMD), and
// short runs, so that the last ones even out.  64^3 cells, 2.1M clustered
// particles, order 8 (173 MB of moments), the whole call: 151 -> 107 us; 50k
// particles of 18^3 cells 45 -> 28.
#include "nf_internal.h"
#include "nf_kernels.h"

namespace nf {
namespace {

constexpr int kMaxOrder = 8;
constexpr int kUnitTerms = 4;       // consecutive z powers per lane
constexpr int kChunk = 32;          // particles staged per round (one per lane)
// rows of staged powers: x^0..8, then y^b z^c0 for c0 = 0 (b = 0..8), 4 (0..4)
// and 8 (0); a row holds one double per particle and one of padding, which
// spreads the rows over the LDS banks
constexpr int yz_row(int b, int c0) {
    return kMaxOrder + 1 + b + (c0 >= 4 ? kMaxOrder + 1 : 0) + (c0 >= 8 ? kMaxOrder - 4 + 1 : 0);
}
constexpr int kRows = yz_row(0, 8) + 1;
constexpr int kRowLen = kChunk + 1;
static_assert(kMaxOrder == 8 && kUnitTerms == 4, "the rows above");
// Work partition: cell c costs its particles plus kCellCost (its T stores);
// workgroup w takes the cells whose cumulative cost
//   cost(c) = cell_start[c] + kCellCost * c
// lies in [w kRange, (w + 1) kRange).  cost is increasing in c, so the first
// cell of every range is found by one pass over the cells.
constexpr int kCellCost = 8;
constexpr int kRange = 128;
constexpr int kBatch = 4;           // chunks whose offsets are loaded together: a load waits
                                    // for the stores before it (they return in order)
constexpr int kBig = 256;           // larger cells are summed in pieces of kBig
constexpr int kMaxTerms = (kMaxOrder + 1) * (kMaxOrder + 2) * (kMaxOrder + 3) / 6;

__device__ __forceinline__ int64_t cell_cost(const int32_t *cs, int c) {
    return (int64_t)cs[c] + (int64_t)kCellCost * c;
}

// Storage index of term (a, b, c), n = a + b + c: the terms of lower degree,
// then a descending, then b descending within degree n.
constexpr int term_index(int a, int b, int c) {
    const int n = a + b + c;
    return n * (n + 1) * (n + 2) / 6 + (n - a) * (n - a + 1) / 2 + (n - a - b);
}

// first[w] = smallest c with cost(c) >= w kRange, for w = 0 .. nrange - 1,
// and first[nrange] = ncell.  The pieces of each cell of more than kBig
// particles, in order from wherever the count of pieces stands (total, zeroed
// by the descriptor upload): no moment depends on the place.  PER cells a
// thread, NT apart.  A block draws from the count once, and a cell of many ranges
// or pieces is written by its whole wave: strongly clustered, a draw and a thread
// a big cell took 75 us of 16.8M particles' call, a draw per 256 cells 52 (and 392
// of 134M), this 16 (72).
template <int NT, int PER>
__global__ void __launch_bounds__(NT)
k_mp_plan(const DevBox *__restrict__ boxes, const int64_t *__restrict__ range_base,
          int32_t *__restrict__ first, uint32_t *__restrict__ total,
          MpPiece *__restrict__ pieces, int64_t max_pieces) {
    const DevBox &B = boxes[blockIdx.y];
    const int64_t c0 = (int64_t)blockIdx.x * (NT * PER) + threadIdx.x;
    if (c0 - threadIdx.x > B.ncell) return;   // whole workgroup
    int32_t *f = first + range_base[blockIdx.y] + blockIdx.y;   // nrange + 1 entries per box
    const int nrange = (int)(range_base[blockIdx.y + 1] - range_base[blockIdx.y]);
    const int lane = threadIdx.x & 63;
    int q[PER], np[PER], n[PER], all = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = (int)min(c0 + i * NT, (int64_t)B.ncell);
        int lo = 0, hi = -1;   // the ranges whose first cell is c
        q[i] = n[i] = 0;
        if (c0 + i * NT <= B.ncell) {
            if (c == 0) {
                f[0] = 0;
                f[nrange] = B.ncell;
            } else {
                lo = (int)(cell_cost(B.cell_start, c - 1) / kRange) + 1;
                hi = min((int)(cell_cost(B.cell_start, c) / kRange), nrange - 1);
            }
            if (c < B.ncell) {
                q[i] = B.cell_start[c];
                n[i] = B.cell_start[c + 1] - q[i];
            }
        }
        if (hi - lo < 8)
            for (int w = lo; w <= hi; ++w) f[w] = c;
        for (uint64_t m = __ballot(hi - lo >= 8); m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1;
            const int a = __builtin_amdgcn_readlane(lo, l), b = __builtin_amdgcn_readlane(hi, l);
            const int v = __builtin_amdgcn_readlane(c, l);
            for (int w = a + lane; w <= b; w += 64) f[w] = v;
        }
        np[i] = n[i] > kBig ? (n[i] - 1) / kBig + 1 : 0;
        all += np[i];
    }
    if (!__syncthreads_or(all)) return;
    __shared__ uint32_t block_pieces, block_at;
    if (threadIdx.x == 0) block_pieces = 0u;
    __syncthreads();
    int at = all ? (int)atomicAdd(&block_pieces, (uint32_t)all) : 0;
    __syncthreads();
    if (threadIdx.x == 0) block_at = atomicAdd(total, block_pieces);
    __syncthreads();
    at += (int)block_at;
    auto put = [&](int64_t to, int cell, int q0, int cnt, int k, int k1) {
        if (to + k < max_pieces)
            pieces[to + k] = MpPiece{(int32_t)blockIdx.y, cell, q0 + k * kBig,
                                     q0 + min(cnt, (k + 1) * kBig), k, k1};
    };
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = (int)(c0 + i * NT);
        if (np[i] <= 16)
            for (int k = 0; k < np[i]; ++k) put(at, c, q[i], n[i], k, np[i]);
        for (uint64_t m = __ballot(np[i] > 16); m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1;
            const int cell = __builtin_amdgcn_readlane(c, l);
            const int q0 = __builtin_amdgcn_readlane(q[i], l);
            const int cnt = __builtin_amdgcn_readlane(n[i], l);
            const int k1 = __builtin_amdgcn_readlane(np[i], l);
            const int to = __builtin_amdgcn_readlane(at, l);
            for (int k = lane; k < k1; k += 64) put(to, cell, q0, cnt, k, k1);
        }
        at += np[i];
    }
}

// The lanes' units for every order p: (a, b) pairs in order, each cut into
// runs of <= 4 z powers of which the first uk are terms.  ia and iyz are the rows
// of their staged powers; idx are the storage indices of the unit's terms,
// and for j >= uk idx[j] repeats idx[0], so that a lane stores all four slots
// without a branch (the extra stores rewrite term 0 with its own value).
// Lanes without a unit repeat lane 0's: they compute and store the same
// values at the same places.  Built at compile time, read once per workgroup.
struct LaneUnit {
    int16_t ia, iyz, uk;
    int16_t idx[kUnitTerms];
};
struct UnitTable {
    LaneUnit u[kMaxOrder + 1][64];
};
constexpr UnitTable make_units() {
    UnitTable T{};
    for (int p = 0; p <= kMaxOrder; ++p) {
        int n = 0;
        for (int a = 0; a <= p; ++a)
            for (int b = 0; a + b <= p; ++b)
                for (int c = 0; a + b + c <= p; c += kUnitTerms, ++n) {
                    LaneUnit L{(int16_t)a, (int16_t)yz_row(b, c),
                               (int16_t)(p - a - b - c + 1 < kUnitTerms ? p - a - b - c + 1
                                                                        : kUnitTerms),
                               {0, 0, 0, 0}};
                    for (int j = 0; j < kUnitTerms; ++j)
                        L.idx[j] = (int16_t)term_index(a, b, j < L.uk ? c + j : c);
                    T.u[p][n] = L;
                }
        for (int t = n; t < 64; ++t) T.u[p][t] = T.u[p][0];
    }
    return T;
}
constexpr int count_units(int p) {
    int n = 0;
    for (int a = 0; a <= p; ++a)
        for (int b = 0; a + b <= p; ++b)
            for (int c = 0; a + b + c <= p; c += kUnitTerms) ++n;
    return n;
}
static_assert(count_units(kMaxOrder) <= 64, "one unit per lane");
__constant__ UnitTable kUnits = make_units();

__device__ __forceinline__ LaneUnit lane_unit(int p, int t) { return kUnits.u[p][t]; }

// Lane t < cnt writes the powers of its particle's offset o, up to the largest
// order: straight-line code, cheaper than a loop to the call's order.
__device__ __forceinline__ void stage_powers(double (*pw)[kRowLen], int t, int cnt, float4 o) {
    if (t < cnt) {
        const double x = o.x, y = o.y, z = o.z, z2 = z * z, z4 = z2 * z2;
        double px = 1.0, py = 1.0;
#pragma unroll
        for (int k = 0; k <= kMaxOrder; ++k) {
            pw[k][t] = px;
            pw[yz_row(k, 0)][t] = py;
            if (k + 4 <= kMaxOrder) pw[yz_row(k, 4)][t] = py * z4;
            px *= x;
            py *= y;
        }
        pw[yz_row(0, 8)][t] = z4 * z4;
    }
}

// acc[j] += sum over the cnt staged particles, in order, of x^a y^b z^(c0 + j);
// z: lane l's is particle l's.  at(l) runs before particle l is added.  The
// powers of the next four particles are read while four are added, also
// across at().  Terms past the unit's last one are computed and never stored.
template <class At>
__device__ __forceinline__ void add_staged(const double (*pw)[kRowLen], int cnt, float z,
                                           const LaneUnit &U, double (&acc)[kUnitTerms], At at) {
    constexpr int kAhead = 4;
    static_assert(kChunk % kAhead == 0, "whole groups");
    const double *xa = pw[U.ia], *yz = pw[U.iyz];
    double x[kAhead], w[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        x[u] = xa[u];
        w[u] = yz[u];
    }
    for (int l0 = 0; l0 < cnt; l0 += kAhead) {
        double m[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) m[u] = x[u] * w[u];
        const int next = l0 + kAhead < cnt ? l0 + kAhead : l0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            x[u] = xa[next + u];
            w[u] = yz[next + u];
        }
        double z1[kAhead], z2[kAhead], z3[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            z1[u] = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), l0 + u));
            z2[u] = z1[u] * z1[u];
            z3[u] = z2[u] * z1[u];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (l0 + u >= cnt) break;
            at(l0 + u);
            acc[0] += m[u];
            acc[1] = __builtin_fma(m[u], z1[u], acc[1]);
            acc[2] = __builtin_fma(m[u], z2[u], acc[2]);
            acc[3] = __builtin_fma(m[u], z3[u], acc[3]);
        }
    }
}

// The offset of sorted slot i (x, y, z) through a global pointer.
__device__ __forceinline__ float4 ld_off(gptr<const float> off, int i) {
    const gptr<const float> q = off + 4 * (int64_t)i;   // 4 i passes 2^31 for i >= 2^29
    return make_float4(q[0], q[1], q[2], 0.f);
}

// The moments of piece w of a big cell, in double.
__device__ __forceinline__ void piece_moments(const DevBox *__restrict__ boxes, const MpPiece &pc,
                                              double *__restrict__ partial, int p,
                                              double (*pw)[kRowLen]) {
    const int t = threadIdx.x;
    const LaneUnit U = lane_unit(p, t);
    const gptr<const float> off = gp((const float *)boxes[pc.box].off);
    double acc[kUnitTerms] = {0.0, 0.0, 0.0, 0.0};
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (pc.q0 + t < pc.q1) o = ld_off(off, pc.q0 + t);
    for (int s = pc.q0; s < pc.q1; s += kChunk) {
        const int e = min(s + kChunk, pc.q1);
        __syncthreads();
        stage_powers(pw, t, e - s, o);
        const float z = o.z;
        if (e + t < pc.q1) o = ld_off(off, e + t);
        __syncthreads();
        add_staged(pw, e - s, z, U, acc, [](int) {});
    }
#pragma unroll
    for (int j = 0; j < kUnitTerms; ++j) gp(partial)[U.idx[j]] = j < U.uk ? acc[j] : acc[0];
}

// Workgroups in row-major order: the pieces of all boxes (most calls have more
// such workgroups than pieces, and these end at once), then the runs of box 0, of
// box 1, ...  One flat list: a row of the grid per box, as long as the longest,
// held mostly idle workgroups for uneven boxes (63 boxes of 1000 particles beside
// one of 2.1M: 577 us a call, 145 so).
__global__ void __launch_bounds__(64)
k_multipoles(const DevBox *__restrict__ boxes, int nbox, const int64_t *__restrict__ range_base,
             const int32_t *__restrict__ first, int p, int nterms,
             const MpPiece *__restrict__ pieces, const uint32_t *__restrict__ total,
             int64_t max_pieces, double *__restrict__ partial) {
    __shared__ __align__(16) double pw[kRows][kRowLen];   // powers of the staged particles
    static_assert(kChunk == 32, "one staged particle per lane");
    const int64_t i = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (i < max_pieces) {
        if (i < (int64_t)*total) piece_moments(boxes, pieces[i], partial + i * kMaxTerms, p, pw);
        return;
    }
    const int64_t run = i - max_pieces;
    if (run >= range_base[nbox]) return;   // whole workgroup
    // the last box whose runs start here or before, 64 candidates by one load
    int box = 0;
    for (int len = nbox; len > 1;) {
        const int step = (len + 63) >> 6, at = (int)threadIdx.x * step;
        const bool from = at < len && range_base[box + at] <= run;
        const int k = (__popcll(__ballot(from)) - 1) * step;
        box += k;
        len = min(step, len - k);
    }
    box = __builtin_amdgcn_readfirstlane(box);
    const int w = (int)(run - range_base[box]);
    const DevBox &B = boxes[box];
    const int32_t *f = first + range_base[box] + box;
    const int t = threadIdx.x;
    const LaneUnit U = lane_unit(p, t);
    const gptr<const int32_t> cs = gp(B.cell_start);
    const gptr<const float> off = gp((const float *)B.off);
    const gptr<float> out = gp(B.out);
    static_assert(kRange % kCellCost == 0, "range bound");
    const int c0 = f[w], c1 = f[w + 1];
    if (c0 >= c1) return;
    // each cell costs >= kCellCost, so a range holds at most kRange / kCellCost
    // = 16 cells: lane k holds the start and end of the range's cell k, read
    // back with readlane (uniform index, no memory wait)
    static_assert(kRange / kCellCost <= 64, "one cell of the range per lane");
    const int cbeg_l = t < c1 - c0 ? cs[c0 + t] : 0;
    const int cend_l = t < c1 - c0 ? cs[c0 + t + 1] : 0;
    auto cbeg = [&](int cell) { return __builtin_amdgcn_readlane(cbeg_l, cell - c0); };
    auto cend_of = [&](int cell) { return __builtin_amdgcn_readlane(cend_l, cell - c0); };
    double acc[kUnitTerms] = {0.0, 0.0, 0.0, 0.0};
    uint32_t at_byte[kUnitTerms];
#pragma unroll
    for (int j = 0; j < kUnitTerms; ++j) at_byte[j] = 4u * (uint32_t)U.idx[j];
    auto flush = [&](int cell) {
        // (scalar base, 32-bit byte offsets)
        const gptr<char> o = (gptr<char>)(out + (int64_t)cell * nterms);
        const float v0 = (float)acc[0];
#pragma unroll
        for (int j = 0; j < kUnitTerms; ++j) {
            *(gptr<float>)(o + at_byte[j]) = j < U.uk ? (float)acc[j] : v0;
            acc[j] = 0.0;
        }
    };
    // runs [ca, cb) of cells of at most kBig particles (bounds are uniform)
    for (int ca = c0; ca < c1;) {
        if (cend_of(ca) - cbeg(ca) > kBig) {
            ++ca;
            continue;
        }
        int cb = ca + 1;
        while (cb < c1 && cend_of(cb) - cbeg(cb) <= kBig) ++cb;
        const int p0 = cbeg(ca), p1 = cend_of(cb - 1);
        int cell = ca;
        int cend = cend_of(ca);
        float4 o[kBatch];
        for (int s = p0, q = 0; s < p1; s += kChunk, q = (q + 1) % kBatch) {
            const int e = min(s + kChunk, p1);
            if (q == 0) {
#pragma unroll
                for (int k = 0; k < kBatch; ++k) o[k] = ld_off(off, min(s + k * kChunk + t, p1 - 1));
            }
            __syncthreads();   // the previous chunk is consumed
            stage_powers(pw, t, e - s, o[0]);
            const float z = o[0].z;
#pragma unroll
            for (int k = 0; k + 1 < kBatch; ++k) o[k] = o[k + 1];
            __syncthreads();
            add_staged(pw, e - s, z, U, acc, [&](int l) {
                while (s + l >= cend) {   // cells that end at or before the particle
                    flush(cell);
                    ++cell;
                    cend = cend_of(cell);
                }
            });
        }
        for (; cell < cb; ++cell) flush(cell);   // the run's last cells (and empty ones)
        ca = cb;
    }
}

// The first piece of each big cell adds the cell's pieces in order, a thread a
// term, kAhead loads in flight: one by one they cost 0.9 us a piece.  16.8M strongly
// clustered particles 193 -> 25 us; 2.1M in one cell 7.3 -> 0.4 ms a call.
constexpr int kCombineThreads = 192;
static_assert(kMaxTerms <= kCombineThreads, "a thread a term");
__global__ void __launch_bounds__(kCombineThreads)
k_mp_combine(const DevBox *__restrict__ boxes, const MpPiece *__restrict__ pieces,
             const uint32_t *__restrict__ total, const double *__restrict__ partial,
             int nterms, int64_t max_pieces) {
    const int t = threadIdx.x;
    if (t >= nterms) return;
    constexpr int kAhead = 16;
    const int all = (int)min((int64_t)*total, max_pieces);
    for (int w = blockIdx.x; w < all; w += gridDim.x) {
        const MpPiece pc = pieces[w];
        if (pc.k != 0) continue;
        const int np = min(pc.np, all - w);
        const gptr<const double> from = gp(partial) + (int64_t)w * kMaxTerms + t;
        double sum = 0.0, v[kAhead];
        for (int k = 0; k < np; k += kAhead) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) v[u] = from[(int64_t)min(k + u, np - 1) * kMaxTerms];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (k + u < np) sum += v[u];
        }
        gp(boxes[pc.box].out)[(int64_t)pc.cell * nterms + t] = (float)sum;
    }
}

}  // namespace

int multipole_max_order() { return kMaxOrder; }

int multipole_terms(int p) { return (p + 1) * (p + 2) * (p + 3) / 6; }

int64_t multipole_ranges(int64_t n, int64_t ncell) {
    return (n + (int64_t)kCellCost * ncell) / kRange + 1;
}

int multipole_big() { return kBig; }

// Sum over big cells of ceil(n_c / kBig) <= n / kBig + (big cells) < 2 n / kBig.
int64_t multipole_max_pieces(int64_t n) { return 2 * (n / kBig) + 1; }

namespace {

// The grid of k_multipoles.  A dimension of a launch holds fewer than 2^32 work
// items, which the largest calls pass (K = 1024 needs 2^26 workgroups of 64):
// rows of at most kMaxRow workgroups.
constexpr int64_t kMaxRow = (int64_t)1 << 25;
constexpr int64_t grid_rows(int64_t workgroups) {
    return workgroups > kMaxRow ? (workgroups + kMaxRow - 1) / kMaxRow : 1;
}
constexpr int64_t grid_cols(int64_t workgroups) {
    return workgroups > 0 ? (workgroups + grid_rows(workgroups) - 1) / grid_rows(workgroups) : 1;
}
constexpr bool grid_fits(int64_t n, int64_t ncell, int64_t nbox) {
    const int64_t pieces = 2 * (n / kBig) + nbox;
    const int64_t all = (n + kCellCost * ncell) / kRange + nbox + pieces;
    return grid_cols(all) * 64 < (int64_t)1 << 32 && grid_rows(all) < 65536 &&
           grid_cols(all) * grid_rows(all) >= all && pieces <= INT32_MAX;
}
static_assert(grid_fits(0, 125, 1) && grid_fits(1 << 20, 1024 * 1024 * 1024, 1) &&
                  grid_fits(INT32_MAX, 1290 * 1290 * 1290, 1) &&
                  grid_fits(INT32_MAX, INT32_MAX, 4096),
              "every call that is accepted can be launched");

}  // namespace

constexpr int64_t kFineCells = (int64_t)1 << 20;   // from here 4096 cells a planning block

hipError_t multipole_launch(const DevBox *d_boxes, int nbox, const MpPlan &mp, int p,
                            hipStream_t s) {
    // The one count takes 87 M draws a second, so a block of a fine grid covers many
    // cells; a coarse one would leave CUs idle (64^3 cells: 64 blocks).
    const bool fine = mp.max_ncell >= kFineCells;
    const int nt = fine ? 1024 : 256, per = fine ? 4 : 1;
    hipLaunchKernelGGL((fine ? k_mp_plan<1024, 4> : k_mp_plan<256, 1>),
                       dim3((unsigned)(mp.max_ncell / (nt * per) + 1), (unsigned)nbox), dim3(nt),
                       0, s, d_boxes, mp.range_base, mp.first, mp.total, mp.pieces,
                       mp.max_pieces);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t all = mp.max_pieces + mp.ranges;
    hipLaunchKernelGGL(k_multipoles, dim3((unsigned)grid_cols(all), (unsigned)grid_rows(all)),
                       dim3(64), 0, s, d_boxes, nbox, mp.range_base, (const int32_t *)mp.first, p,
                       multipole_terms(p), (const MpPiece *)mp.pieces,
                       (const uint32_t *)mp.total, mp.max_pieces, mp.partial);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_mp_combine,
                       dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(mp.max_pieces, 16384))),
                       dim3(kCombineThreads), 0, s, d_boxes, (const MpPiece *)mp.pieces,
                       (const uint32_t *)mp.total, (const double *)mp.partial, multipole_terms(p),
                       mp.max_pieces);
    return hipGetLastError();
}

}  // namespace nf
