// nf_bin.hip -- binning of particles into the K^3 cell grid (Sec. 2.1):
// cell index + centre offset in double precision, then a stable sort by cell.
//
// All boxes of one call are binned together: box b's keys live in their own
// range [cellbase_b, cellbase_b + K_b^3) of one concatenated key space, so a
// single stable LSD radix sort over the concatenation of all boxes leaves
// every box's particles in its own slice, sorted by cell, ties in input order.
#include "nf_internal.h"
#include "nf_kernels.h"

namespace nf {

// ---------------------------------------------------------------- utilities

__global__ void k_fill_u32(uint32_t *p, int64_t count, uint32_t value) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) p[i] = value;
}

// Block-wide exclusive scan of NT thread values; returns this thread's prefix
// and the block total.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t &total) {
    __shared__ uint32_t wsum[NT / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t wpre = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
        uint32_t s = wsum[q];
        if (q < w) wpre += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return wpre + x - v;
}

// The box of concatenated element g: the last one that starts at or before it
// (empty boxes share the start of the next one).
__device__ __forceinline__ int box_of(const DevBox *boxes, int nbox, int64_t g) {
    int lo = 0, hi = nbox;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (boxes[mid].base <= g) lo = mid; else hi = mid;
    }
    return lo;
}

// ------------------------------------------------------------- cell keys

// Cell id and offsets of a particle of box B; false for one that has no cell
// (cell 0, offsets 0).
__device__ __forceinline__ bool particle_cell(const DevBox &B, const double (&x)[3], int &cell,
                                              float (&o)[3]) {
    int c[3];
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double od;
        ok &= cell_coord(x[a], B.kappa, B.K, c[a], od);
        o[a] = (float)od;
    }
    if (!ok) {
        c[0] = c[1] = c[2] = 0;
        o[0] = o[1] = o[2] = 0.0f;
    }
    cell = (c[0] * B.K + c[1]) * B.K + c[2];
    return ok;
}

// The cell keys (cell id in the box's key range) of a tile of the concatenated
// particles and the tile's histogram of the first digit, hist[d * pitch + tile].
// Reading the keys back for that histogram took 10 us of 2.1M particles.
template <int BITS>
__global__ void __launch_bounds__(kSortThreads)
k_bin_keys(const DevBox *__restrict__ boxes, int nbox, BinScratch sc, int64_t N, int pitch) {
    constexpr int R = 1 << BITS;
    __shared__ uint32_t cnt[R];
    const int t = threadIdx.x;
    for (int d = t; d < R; d += kSortThreads) cnt[d] = 0;
    __syncthreads();
    const int64_t tile0 = (int64_t)blockIdx.x * kSortTile;
    const int64_t last = min(tile0 + kSortTile, N) - 1;
    const int b0 = box_of(boxes, nbox, tile0), b1 = box_of(boxes, nbox, last);
    double x[kSortItems][3];
    auto load = [&](const DevBox &B, int64_t g, double (&p)[3]) {
        const gptr<const double> q = gp(B.pos) + 3 * (g - B.base);
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = q[a];
    };
    auto key = [&](const DevBox &B, int b, int64_t g, const double (&p)[3]) {
        int cell;
        float o[3];
        if (!particle_cell(B, p, cell, o)) atomicAdd(&sc.bad[b], 1u);
        const uint32_t k = (uint32_t)B.cellbase + (uint32_t)cell;
        gp(sc.keys[0])[g] = k;
        atomicAdd(&cnt[k & (R - 1)], 1u);
    };
    if (b0 == b1) {   // the common tile: one box, its descriptor in scalar registers
        const DevBox &B = boxes[b0];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int64_t g = tile0 + k * kSortThreads + t;
            load(B, min(g, last), x[k]);
        }
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int64_t g = tile0 + k * kSortThreads + t;
            if (g <= last) key(B, b0, g, x[k]);
        }
    } else {
        for (int k = 0; k < kSortItems; ++k) {
            const int64_t g = tile0 + k * kSortThreads + t;
            if (g > last) break;
            const int b = box_of(boxes, nbox, g);
            load(boxes[b], g, x[0]);
            key(boxes[b], b, g, x[0]);
        }
    }
    __syncthreads();
    for (int d = t; d < R; d += kSortThreads)
        gp(sc.hist)[(int64_t)d * pitch + blockIdx.x] = cnt[d];
}

// ------------------------------------------------------------- radix sort

// The histogram of a later digit; the count does not depend on the order
// within the tile, so a thread takes four consecutive keys by one load.
template <int BITS>
__global__ void __launch_bounds__(kSortThreads)
k_radix_hist(const uint32_t *__restrict__ keys, int64_t N, int shift, int pitch,
             uint32_t *__restrict__ hist) {
    constexpr int R = 1 << BITS;
    static_assert(kSortItems == 4, "one 16-byte load per thread");
    __shared__ uint32_t cnt[R];
    const int t = threadIdx.x;
    for (int d = t; d < R; d += kSortThreads) cnt[d] = 0;
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * kSortTile + 4 * t;
    if (g + 4 <= N) {
        const uint4 q = *reinterpret_cast<const uint4 *>(keys + g);
        atomicAdd(&cnt[(q.x >> shift) & (R - 1)], 1u);
        atomicAdd(&cnt[(q.y >> shift) & (R - 1)], 1u);
        atomicAdd(&cnt[(q.z >> shift) & (R - 1)], 1u);
        atomicAdd(&cnt[(q.w >> shift) & (R - 1)], 1u);
    } else {
        for (int64_t i = g; i < N; ++i) atomicAdd(&cnt[(keys[i] >> shift) & (R - 1)], 1u);
    }
    __syncthreads();
    for (int d = t; d < R; d += kSortThreads) hist[(int64_t)d * pitch + blockIdx.x] = cnt[d];
}

// One workgroup per digit: its row of tile counts to exclusive prefixes over
// the tiles, and its total.  (A scan over all counts takes two launches.)
__global__ void __launch_bounds__(kScanThreads)
k_scan_rows(uint32_t *__restrict__ hist, int nblk, int pitch, uint32_t *__restrict__ total) {
    constexpr int kPer = 4;
    uint32_t *row = hist + (int64_t)blockIdx.x * pitch;
    uint32_t run = 0;
    for (int b0 = 0; b0 < nblk; b0 += kPer * kScanThreads) {
        const int b = b0 + kPer * (int)threadIdx.x;
        uint32_t v[kPer], s = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            v[i] = b + i < nblk ? row[b + i] : 0u;
            s += v[i];
        }
        uint32_t all;
        uint32_t x = block_exclusive<kScanThreads>(s, all) + run;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (b + i < nblk) row[b + i] = x;
            x += v[i];
        }
        run += all;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = run;
}

// The tile of workgroup b when each of the 8 XCDs (workgroups are dealt to
// them round-robin by id) takes one contiguous range of the nb tiles.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
    const int x = b % 8, j = b / 8, per = nb / 8, rem = nb % 8;
    return x * per + min(x, rem) + j;
}

// Rank of a wave's key among the wave's keys of the same digit so far:
// "earlier round, then lower lane" is input order.  cnt: the wave's counters.
template <int BITS>
__device__ __forceinline__ uint32_t wave_rank(uint16_t *cnt, bool valid, uint32_t d, int lane,
                                              uint64_t below) {
    const uint64_t m = match_digit<BITS>(valid, d);
    const uint32_t before = cnt[d];
    __builtin_amdgcn_wave_barrier();
    if (valid && lane == 63 - __clzll(m)) cnt[d] = (uint16_t)(before + (uint32_t)__popcll(m));
    __builtin_amdgcn_wave_barrier();
    return before + (uint32_t)__popcll(m & below);
}

// Stable scatter of one tile, workgroup b taking tile xcd_tile(b): the
// neighbouring output runs of a digit (consecutive tiles) then meet whole in
// one XCD's L2 instead of as line fragments in several.  Wave w owns a
// contiguous part of the tile and walks it in rounds of 64, so "earlier round,
// then lower lane, then lower wave" is input order; that gives every key its
// rank within the tile's run of its digit.  The tile is then reordered by digit
// in LDS and written out slot by slot, so that the lanes of a wave store
// consecutive addresses of one output run.
//
// A key travels with its particle's record: the three offsets and the
// concatenated index.  The first pass makes the records from the positions,
// the last one writes the boxes' offsets and order.  Moving 16 bytes a pass in
// runs is cheaper than gathering them once at the end, a random line per
// particle, of which the last kernel took 44 us: binning 2.1M clustered particles
// 148 -> 86 us, 16.8M (three passes) 947 -> 758.
//
// total null: few tiles, and every workgroup adds up the digits' counts (rows
// of hist) itself; else hist holds the scanned rows and total their sums.
// 50 KB of LDS, three workgroups a CU.
template <int BITS, bool FIRST, bool LAST>
__global__ void __launch_bounds__(kSortThreads)
k_radix_scatter(const DevBox *__restrict__ boxes, int nbox, const uint32_t *__restrict__ keys_in,
                const float4 *__restrict__ rec_in, uint32_t *__restrict__ keys_out,
                float4 *__restrict__ rec_out, int64_t N, int shift, int nblk, int pitch,
                const uint32_t *__restrict__ hist, const uint32_t *__restrict__ total) {
    constexpr int R = 1 << BITS;
    constexpr int kWaves = kSortThreads / 64, kWaveKeys = kSortTile / kWaves;
    static_assert(R <= kSortThreads, "a thread per digit in the digit scan");
    __shared__ uint32_t gshift[R];   // output slot of the tile's local slot 0, per digit
    __shared__ uint16_t wcnt[kWaves][R];
    __shared__ uint32_t skey[kSortTile];
    __shared__ float4 srec[kSortTile];
    const int t = threadIdx.x;
    const int w = t >> 6, lane = t & 63;
    for (int d = t; d < R; d += kSortThreads) {
#pragma unroll
        for (int q = 0; q < kWaves; ++q) wcnt[q][d] = 0;
    }
    __syncthreads();

    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int tile = xcd_tile((int)blockIdx.x, nblk);
    const int64_t tile0 = (int64_t)tile * kSortTile;
    const int64_t last = min(tile0 + kSortTile, N) - 1;
    const int64_t base = tile0 + w * kWaveKeys + lane;
    uint32_t kk[kSortItems], rk[kSortItems];
    float4 rec[kSortItems];
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) kk[k] = gp(keys_in)[min(base + k * 64, last)];
    if constexpr (FIRST) {
        const int b0 = box_of(boxes, nbox, tile0), b1 = box_of(boxes, nbox, last);
        auto load = [&](const DevBox &B, int64_t g, double (&x)[3]) {
            const gptr<const double> q = gp(B.pos) + 3 * (g - B.base);
#pragma unroll
            for (int a = 0; a < 3; ++a) x[a] = q[a];
        };
        auto record = [&](const DevBox &B, int64_t g, const double (&x)[3]) {
            float o[3];
            bool ok = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double od, f;
                ok &= cell_offset(x[a], B.kappa, f, od);
                o[a] = (float)od;
            }
            return make_float4(ok ? o[0] : 0.f, ok ? o[1] : 0.f, ok ? o[2] : 0.f,
                               __uint_as_float((uint32_t)g));
        };
        if (b0 == b1) {
            const DevBox &B = boxes[b0];
            double x[kSortItems][3];
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) load(B, min(base + k * 64, last), x[k]);
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) rec[k] = record(B, min(base + k * 64, last), x[k]);
        } else {
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                const int64_t g = min(base + k * 64, last);
                const DevBox &B = boxes[box_of(boxes, nbox, g)];
                double x[3];
                load(B, g, x);
                rec[k] = record(B, g, x);
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const nf_v4f r = ld_g4(rec_in, (uint64_t)min(base + k * 64, last));
            rec[k] = make_float4(r.x, r.y, r.z, r.w);
        }
    }
#pragma unroll
    for (int k = 0; k < kSortItems; ++k)
        rk[k] = wave_rank<BITS>(wcnt[w], base + k * 64 <= last, (kk[k] >> shift) & (R - 1), lane,
                                below);
    __syncthreads();
    {   // per digit: exclusive prefix over the waves, then over the digits
        uint32_t sum = 0, before = 0, all = 0;
        const int d = t;
        if (d < R) {
#pragma unroll
            for (int q = 0; q < kWaves; ++q) sum += wcnt[q][d];
            const uint32_t *row = hist + (int64_t)d * pitch;
            if (total) {
                before = row[tile];
                all = total[d];
            } else {
                for (int b = 0; b < nblk; b += 4) {   // rows are padded to whole groups
                    const uint4 c = *reinterpret_cast<const uint4 *>(row + b);
                    const uint32_t v[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (b + i < nblk) all += v[i];
                        if (b + i < tile) before += v[i];
                    }
                }
            }
        }
        uint32_t unused;
        uint32_t run = block_exclusive<kSortThreads>(sum, unused);
        const uint32_t first = block_exclusive<kSortThreads>(all, unused);
        if (d < R) {
            gshift[d] = first + before - run;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                const uint32_t c = wcnt[q][d];
                wcnt[q][d] = (uint16_t)run;
                run += c;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        if (base + k * 64 <= last) {
            const uint32_t slot = wcnt[w][(kk[k] >> shift) & (R - 1)] + rk[k];
            skey[slot] = kk[k];
            srec[slot] = rec[k];
        }
    }
    __syncthreads();
    const int cnt = (int)(last - tile0) + 1;
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const int j = t + k * kSortThreads;
        if (j >= cnt) break;
        const uint32_t key = skey[j];
        const float4 r = srec[j];
        const uint32_t dst = gshift[(key >> shift) & (R - 1)] + (uint32_t)j;
        if (dst >= (uint64_t)N) continue;   // never for a consistent histogram
        gp(keys_out)[dst] = key;
        if constexpr (LAST) {
            const DevBox &B = boxes[box_of(boxes, nbox, (int64_t)dst)];
            const int64_t i = (int64_t)__float_as_uint(r.w) - B.base;
            const int64_t slot = (int64_t)dst - B.base;
            if (slot < B.n) {   // always true for a consistent sort
                const int z = (int)((key - (uint32_t)B.cellbase) % (uint32_t)B.K);
                st_g4(B.off, (uint64_t)slot, r.x, r.y, r.z, (float)z);
                gp(B.order)[slot] = (i >= 0 && i < B.n) ? (int)i : 0;   // likewise
            }
        } else {
            st_g4(rec_out, dst, r.x, r.y, r.z, r.w);
        }
    }
}

// ------------------------------------------------------------- exclusive scan

// Per-tile sums.
__global__ void __launch_bounds__(kScanThreads)
k_scan_reduce(const uint32_t *__restrict__ in, int64_t M, uint32_t *__restrict__ sums) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < M) s += in[i];
    }
    uint32_t tot;
    block_exclusive<kScanThreads>(s, tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Exclusive scan of tile blockIdx.x plus `offset`.  In-place (in == out) is
// allowed.
__device__ __forceinline__ void scan_tile(const uint32_t *in, uint32_t *out, int64_t M,
                                          uint32_t offset) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        v[k] = (i < M) ? in[i] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_exclusive<kScanThreads>(s, tot) + offset;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < M) out[i] = run;
        run += v[k];
    }
}

// Exclusive scan of each tile plus the tile's scanned offset (offsets may be
// null for a single tile).
__global__ void __launch_bounds__(kScanThreads)
k_scan_down(const uint32_t *in, uint32_t *out, int64_t M, const uint32_t *__restrict__ offsets) {
    scan_tile(in, out, M, offsets ? offsets[blockIdx.x] : 0u);
}

// The same with unscanned tile sums: each block adds up the sums of the tiles
// before it (few enough that every block can: at most kScanTile tiles).
__global__ void __launch_bounds__(kScanThreads)
k_scan_down_sums(uint32_t *data, int64_t M, const uint32_t *__restrict__ sums) {
    uint32_t part = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) part += sums[i];
    uint32_t before;
    block_exclusive<kScanThreads>(part, before);
    scan_tile(data, data, M, before);
}

// ------------------------------------------------------------- cell starts

// cell_start[c] = the first slot whose cell is >= c, for c = 0 .. ncell: slot s
// (0 .. n) writes the cells in (cell of slot s-1, cell of slot s], slot n the
// cells after the last one.  Every c is written exactly once.  The lanes of a
// wave call this together (slots above n write nothing); a long run of empty cells is
// written by the whole wave.
template <class CellOf>
__device__ __forceinline__ void write_cell_starts(int32_t *cell_start, int n, int ncell,
                                                  int64_t slot, CellOf cell_of) {
    const int lane = threadIdx.x & 63, s = (int)min(slot, (int64_t)n);
    int lo = 0, hi = -1;
    if (slot <= n) {
        lo = s == 0 ? 0 : cell_of(s - 1) + 1;
        hi = s == n ? ncell : cell_of(s);
    }
    gptr<int32_t> out = gp(cell_start);
    uint64_t longs = __ballot(hi - lo >= 8);
    if (hi - lo < 8)
        for (int c = lo; c <= hi; ++c) out[c] = s;
    while (longs) {
        const int l = __ffsll((unsigned long long)longs) - 1;
        longs &= longs - 1;
        const int a = __builtin_amdgcn_readlane(lo, l), b = __builtin_amdgcn_readlane(hi, l);
        const int v = __builtin_amdgcn_readlane(s, l);
        for (int64_t c = (int64_t)a + lane; c <= b; c += 64) out[c] = v;
    }
}

// Per box: cell_start from the sorted keys, and the count of bad particles.
__global__ void __launch_bounds__(256)
k_bin_cells(const DevBox *__restrict__ boxes, const uint32_t *__restrict__ keys,
            const uint32_t *__restrict__ bad) {
    const DevBox &B = boxes[blockIdx.y];
    if ((int64_t)blockIdx.x * 256 > B.n) return;
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const gptr<const uint32_t> k = gp(keys) + B.base;
    const uint32_t c0 = (uint32_t)B.cellbase;
    write_cell_starts(B.cell_start, B.n, B.ncell, s, [&](int i) { return (int)(k[i] - c0); });
    if (s == 0 && B.nbad) B.nbad[0] = (int32_t)bad[blockIdx.y];
}

// ------------------------------------------------------------- small boxes

// A whole box of at most kBinSmallN particles and kBinSmallCells cells by one
// workgroup: the same stable sort with the keys in LDS.  The descriptors come as
// a kernel argument (d_boxes null) or from memory.  Such a call was bound by its
// eight launches: 1000 particles 32 -> 8 us (14 by the tiled sort in four
// launches), 4096 29 -> 15 (17); one workgroup is slower above.
template <int BITS>
__device__ __forceinline__ void small_pass(int shift, int n, int rounds, int first, int lane,
                                           uint64_t below, uint16_t *wcnt,
                                           uint32_t *skey, uint16_t *sidx,
                                           uint32_t (&kk)[kBinSmallItems],
                                           uint32_t (&ix)[kBinSmallItems]) {
    constexpr int R = 1 << BITS, kWaves = kBinSmallThreads / 64;
    const int t = threadIdx.x, w = t >> 6;
    for (int d = t; d < R * kWaves; d += kBinSmallThreads) wcnt[d] = 0;
    __syncthreads();
    uint32_t rk[kBinSmallItems];
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k)
        if (k < rounds)
            rk[k] = wave_rank<BITS>(wcnt + w * R, first + k * 64 < n, (kk[k] >> shift) & (R - 1), lane,
                                    below);
    __syncthreads();
    uint32_t sum = 0, all;
    if (t < R)
#pragma unroll
        for (int q = 0; q < kWaves; ++q) sum += wcnt[q * R + t];
    uint32_t run = block_exclusive<kBinSmallThreads>(sum, all);
    if (t < R)
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t c = wcnt[q * R + t];
            wcnt[q * R + t] = (uint16_t)run;
            run += c;
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k)
        if (k < rounds && first + k * 64 < n) {
            const uint32_t slot = wcnt[w * R + ((kk[k] >> shift) & (R - 1))] + rk[k];
            skey[slot] = kk[k];
            sidx[slot] = (uint16_t)ix[k];
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k)
        if (k < rounds && first + k * 64 < n) {
            kk[k] = skey[first + k * 64];
            ix[k] = sidx[first + k * 64];
        }
}

__global__ void __launch_bounds__(kBinSmallThreads)
k_bin_small(Chunk c, const DevBox *__restrict__ d_boxes) {
    constexpr int kBits = 8, kWaves = kBinSmallThreads / 64;
    __shared__ uint16_t wcnt[kWaves << (kBits + 1)];
    __shared__ uint32_t skey[kBinSmallN];
    __shared__ uint16_t sidx[kBinSmallN], slot_of[kBinSmallN];
    __shared__ int nbad;
    const DevBox &B = d_boxes ? d_boxes[blockIdx.x]
                              : reinterpret_cast<const DevBox *>(c.bytes)[blockIdx.x];
    const int n = B.n, t = threadIdx.x, lane = t & 63;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // wave w owns the particles [64 w rounds, 64 (w + 1) rounds)
    const int rounds = (n + kBinSmallThreads - 1) / kBinSmallThreads;
    const int first = (t >> 6) * 64 * rounds + lane;
    if (t == 0) nbad = 0;
    __syncthreads();
    uint32_t kk[kBinSmallItems], ix[kBinSmallItems];
    float off[kBinSmallItems][3];
    int z[kBinSmallItems];
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k) {
        const int i = first + k * 64;
        kk[k] = ix[k] = 0u;
        if (k < rounds && i < n) {
            const gptr<const double> p = gp(B.pos) + 3 * (int64_t)i;
            const double x[3] = {p[0], p[1], p[2]};
            int cell;
            if (!particle_cell(B, x, cell, off[k])) atomicAdd(&nbad, 1);
            kk[k] = (uint32_t)cell;
            ix[k] = (uint32_t)i;
            z[k] = cell % B.K;
        }
    }
    if ((B.ncell - 1) >> kBits == 1)   // one pass of nine bits
        small_pass<kBits + 1>(0, n, rounds, first, lane, below, wcnt, skey, sidx, kk, ix);
    else
        for (int shift = 0; shift == 0 || (B.ncell - 1) >> shift; shift += kBits)
            small_pass<kBits>(shift, n, rounds, first, lane, below, wcnt, skey, sidx, kk, ix);
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k) {
        const int s = first + k * 64;
        if (k < rounds && s < n) {
            gp(B.order)[s] = (int)ix[k];
            slot_of[ix[k]] = (uint16_t)s;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kBinSmallItems; ++k) {
        const int i = first + k * 64;
        if (k < rounds && i < n)
            st_g4(B.off, slot_of[i], off[k][0], off[k][1], off[k][2], (float)z[k]);
    }
    for (int s0 = 0; s0 <= n; s0 += kBinSmallThreads)
        write_cell_starts(B.cell_start, n, B.ncell, s0 + t, [&](int i) { return (int)skey[i]; });
    if (t == 0 && B.nbad) B.nbad[0] = nbad;
}

// ------------------------------------------------------------- host driver

int64_t scan_scratch_words(int64_t M) {
    // words needed by scan_exclusive(M): the sums of each level, recursively
    int64_t words = 0;
    while (M > kScanTile) {
        int64_t nb = (M + kScanTile - 1) / kScanTile;
        words += nb;
        M = nb;
    }
    return words + 64;
}

hipError_t scan_exclusive(uint32_t *data, int64_t M, uint32_t *scratch, hipStream_t s) {
    if (M <= kScanTile) {
        hipLaunchKernelGGL(k_scan_down, dim3(1), dim3(kScanThreads), 0, s, data, data, M,
                           (const uint32_t *)nullptr);
        return hipGetLastError();
    }
    int64_t nb = (M + kScanTile - 1) / kScanTile;
    uint32_t *sums = scratch;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, M, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (nb <= kScanTile) {   // two launches: each block adds up its predecessors
        hipLaunchKernelGGL(k_scan_down_sums, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data,
                           M, (const uint32_t *)sums);
        return hipGetLastError();
    }
    e = scan_exclusive(sums, nb, scratch + nb, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, data, M,
                       (const uint32_t *)sums);
    return hipGetLastError();
}

hipError_t fill_u32(uint32_t *p, int64_t count, uint32_t value, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>(4096, (count + 255) / 256);
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(256), 0, s, p, count, value);
    return hipGetLastError();
}

template <int BITS>
static hipError_t sort_passes(const DevBox *d_boxes, int nbox, const BinPlan &p, hipStream_t s) {
    hipError_t e;
    const dim3 tiles((unsigned)p.nblk), threads(kSortThreads);
    const int pitch = (int)p.pitch;
    // The scatter of few tiles adds up the rows itself instead of a scan: 32768
    // particles 29 -> 25 us, 131k (64 tiles) equal, 262k 33 -> 39.
    const bool scan = p.nblk > kRowTiles;
    int src = 0;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int shift = pass * BITS;
        const bool first = pass == 0, last = pass + 1 == p.passes;
        if (first)
            hipLaunchKernelGGL(k_bin_keys<BITS>, tiles, threads, 0, s, d_boxes, nbox, p.sc, p.N,
                               pitch);
        else
            hipLaunchKernelGGL(k_radix_hist<BITS>, tiles, threads, 0, s,
                               (const uint32_t *)p.sc.keys[src], p.N, shift, pitch, p.sc.hist);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (scan) {
            hipLaunchKernelGGL(k_scan_rows, dim3(1 << BITS), dim3(kScanThreads), 0, s, p.sc.hist,
                               (int)p.nblk, pitch, p.sc.total);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        auto *scatter = first ? (last ? k_radix_scatter<BITS, true, true>
                                      : k_radix_scatter<BITS, true, false>)
                              : (last ? k_radix_scatter<BITS, false, true>
                                      : k_radix_scatter<BITS, false, false>);
        hipLaunchKernelGGL(scatter, tiles, threads, 0, s, d_boxes, nbox,
                           (const uint32_t *)p.sc.keys[src], (const float4 *)p.sc.rec[src ^ 1],
                           p.sc.keys[src ^ 1], p.sc.rec[src], p.N, shift, (int)p.nblk, pitch,
                           (const uint32_t *)p.sc.hist,
                           scan ? (const uint32_t *)p.sc.total : (const uint32_t *)nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        src ^= 1;
    }
    return hipSuccess;
}

bool bin_is_small(int64_t max_n, int64_t max_ncell) {
    return max_n <= kBinSmallN && max_ncell <= kBinSmallCells;
}

hipError_t bin_small_launch(const Chunk &c, const DevBox *d_boxes, int nbox, hipStream_t s) {
    hipLaunchKernelGGL(k_bin_small, dim3((unsigned)nbox), dim3(kBinSmallThreads), 0, s, c,
                       d_boxes);
    return hipGetLastError();
}

// Boxes that share their word nbad: each writes the sum over its sharers.
__global__ void __launch_bounds__(256)
k_bin_shared_bad(const DevBox *__restrict__ boxes, int nbox, const uint32_t *__restrict__ bad) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= nbox || !boxes[b].nbad) return;
    uint32_t sum = 0;
    for (int q = 0; q < nbox; ++q) sum += boxes[q].nbad == boxes[b].nbad ? bad[q] : 0u;
    boxes[b].nbad[0] = (int32_t)sum;
}

hipError_t bin_launch(const DevBox *d_boxes, int nbox, const BinPlan &p, hipStream_t s) {
    hipError_t e;
    if (p.N > 0) {
        e = p.radix_bits == 9 ? sort_passes<9>(d_boxes, nbox, p, s)
                              : sort_passes<8>(d_boxes, nbox, p, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_bin_cells, dim3((unsigned)(p.max_n / 256 + 1), (unsigned)nbox), dim3(256),
                       0, s, d_boxes, (const uint32_t *)p.sc.keys[p.passes & 1],
                       (const uint32_t *)p.sc.bad);
    if ((e = hipGetLastError()) != hipSuccess || !p.shared_bad) return e;
    hipLaunchKernelGGL(k_bin_shared_bad, dim3((unsigned)(nbox + 255) / 256), dim3(256), 0, s,
                       d_boxes, nbox, (const uint32_t *)p.sc.bad);
    return hipGetLastError();
}

}  // namespace nf
