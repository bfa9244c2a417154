// nf_tile.hip -- tiled near-field kernels for gfx950: a device-side planner
// that cuts the cell grid into work items, and persistent kernels that
// sum the pair forces of Eq. 2 (Sec. 4.3) over the 5x5x5 cell block of
// Sec. 2.1.
//
// The sinks of a cell are cut into chunks of 64.  Work items:
//   * dense  -- a full 64-sink chunk, or the last chunk when it holds at
//               least dense_min sinks (41 by default); one wave per item, one
//               sink per lane.  Every lane needs the same source at the same
//               time, so sources are read from the cell-sorted array with
//               scalar loads and enter the arithmetic as SGPR operands, and
//               the sink is shifted into each source cell's frame.  No LDS, so
//               many waves fit on a CU and hide the load latency.  Items run
//               heaviest neighbourhood first; the heaviest ones of a call of
//               few items by a whole workgroup each.
//   * light  -- a smaller last chunk (all sinks of a cell of fewer than
//               dense_min particles), one item per 4-wave workgroup.  The 125
//               source cells are staged in LDS in the sink cell's own frame,
//               (o_x + dx, o_y + dy, o_z + dz), the 27 cells with |d| <= 1
//               first, then the 98 outer cells, so the sum is two contiguous
//               segments; the g sinks are spread over the 256 threads as
//               (sink a, source slice b), thread = a + g b, P = 256 / g
//               slices, summed at the end by a fixed-order pairwise tree.
//   * narrow -- a light item of fewer than narrow_max sinks (12 by default):
//               the same kernel on one wave per workgroup (P = 64 / g), so the
//               per-item costs that do not shrink with g (item setup, the
//               per-wave header, the slice tree) are paid by one wave instead
//               of four.
// Small calls run all three classes in one launch (k_small).
// The class boundaries (dense_min, narrow_max), the staging windows of the
// light and narrow kernels and the compensated partial-sum length are tile
// choices of the caller (nf_box), picked by the autotuner.
// In both paths a source of the sink's own cell is used unshifted, so the
// closest pairs are formed from the exact float offsets, and a cell of the
// outer shell of the block (some |d| = 2) is at r >= 1 and takes the Newton
// branch directly when eps <= 1.  The Plummer law is the Newton branch with
// eps_p^2 as the floor on r^2, for every pair.
#include <climits>
#include <mutex>
#include <vector>

#include "nf_internal.h"
#include "nf_kernels.h"

namespace nf {

namespace {

constexpr int kUnit = 64;            // sinks per wave
constexpr int kQueues = 32;          // light-item queues (a multiple of the 8 XCDs)
constexpr int kXcds = 8;             // workgroups are dealt to the XCDs round-robin by id
constexpr int kXcdBlock = 256;       // consecutive light items kept on one XCD, at most
constexpr int kDenseBlock = 16;      // consecutive dense items kept on one XCD, at most
constexpr int kQueueStride = 32;     // words between queue counters (own 128-byte line)
constexpr int kLightWaves = 4;       // waves sharing one light item
constexpr int kLightThreads = 64 * kLightWaves;
constexpr int kNarrowThreads = 64;   // one wave per narrow item
constexpr int kRows = 25;            // (dx, dy) rows of the 5x5x5 block

__device__ __forceinline__ int wrapk(int c, int K) { return c < 0 ? c + K : (c >= K ? c - K : c); }
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// The place of an item in its block, as a mask: a block is the consecutive items
// that stay on one XCD, `most` (a power of two), or less so that every XCD gets at
// least eight blocks (blocks of 256 left 463 light items on two of the eight XCDs).
__device__ __forceinline__ int xcd_block_mask(int nitems, int most) {
    int b = 31 - __builtin_clz(most);
    while (b > 0 && nitems < 8 * kXcds << b) --b;
    return (1 << b) - 1;
}
// Item number of claim t of XCD x's queue: XCD x takes the items of the blocks x,
// x + 8, ... in order.  (Shifts by the block's logarithm instead took two to
// four vector registers more, which cost the narrow kernels a wave per SIMD.)
__device__ __forceinline__ int xcd_item(int t, int x, int mask) {
    return t + (t & ~mask) * (kXcds - 1) + x * (mask + 1);
}

// Inclusive prefix sums over the lanes of a wave (all 64 lanes active): a
// Kogge-Stone scan inside each row of 16 lanes by DPP row shifts (one
// v_add_u32_dpp per step), then the row totals read back with readlane.
// scan_lanes<32> is exact on lanes 0..31 only.
template <int W>
__device__ __forceinline__ int scan_lanes(int x) {
    static_assert(W == 32 || W == 64, "one or two halves of the wave");
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    const int row = (threadIdx.x & 63) >> 4;
    const int t15 = __builtin_amdgcn_readlane(x, 15);
    if constexpr (W == 32) return x + ((row & 1) ? t15 : 0);
    const int t31 = __builtin_amdgcn_readlane(x, 31), t47 = __builtin_amdgcn_readlane(x, 47);
    return x + (row >= 1 ? t15 : 0) + (row >= 2 ? t31 : 0) + (row >= 3 ? t47 : 0);
}

// ------------------------------------------------------------------ planner

// Sources of row r = (dx+2)*5 + (dy+2) of the 5x5x5 block of cell (cx, cy, cz).
__device__ __forceinline__ int row_sources(gptr<const int32_t> cs, int K, int cx, int cy, int cz,
                                           int r) {
    const int rb = (wrapk(cx + r / 5 - 2, K) * K + wrapk(cy + r % 5 - 2, K)) * K;
    const int lo = cz - 2, hi = cz + 2;
    if (lo < 0) return (cs[rb + K] - cs[rb + lo + K]) + (cs[rb + hi + 1] - cs[rb]);
    if (hi >= K) return (cs[rb + K] - cs[rb + lo]) + (cs[rb + hi - K + 1] - cs[rb]);
    return cs[rb + hi + 1] - cs[rb + lo];
}

// Buckets, placed highest first: dense items by cost (quarter octaves of
// their block's source count S, heaviest first); light and narrow items by
// spatial slab (128 slabs of consecutive cells, in cell order).
constexpr int kBuckets = 128;
constexpr int kKinds = 3;                  // 0: dense, 1: light, 2: narrow
__device__ __forceinline__ int cost_bucket(float pairs) {
    const float l = __log2f(fmaxf(pairs, 1.0f));
    return min(kBuckets - 1, (int)(4.0f * l));
}

// Items of a cell of n particles: n / 64 full dense chunks, and the last
// n % 64 sinks as one more dense chunk if they are at least dense_min, else as
// one light item (a narrow one below narrow_max sinks).  cellinfo packs
// (dense bucket + 1) | (light bucket + 1) << 16, 0 for none; the item counts
// per (kind, bucket) are summed in LDS first so that each block adds one value
// per non-empty bucket.
struct CellItems {
    int ndense;     // dense chunks
    int light;      // kind of the remainder's item: 0 none, 1 light, 2 narrow
};
__device__ __forceinline__ CellItems cell_items(int n, int dense_min, int narrow_max) {
    const int full = n / kUnit, rem = n % kUnit;
    const int lk = (rem > 0 && rem < dense_min) ? (rem < narrow_max ? 2 : 1) : 0;
    return CellItems{full + (rem >= dense_min ? 1 : 0), lk};
}

// Blocks [0, cell_blocks): the items of 256 cells of box blockIdx.y.  S ranks
// dense items only, and few cells hold one: the block lists them and its
// threads take their (cell, row) pairs (one thread per cell walking its 25
// rows kept nearly every wave in that loop for a lane or two: 24 us for 64^3
// cells).  The remaining blocks gather the VJP's source records (gather_cot),
// which need nothing of the plan.  (The descriptors are __restrict__: beside the
// stores of the records the compiler read them by vector loads, each waited for:
// 16.8M cells 440 us, 306 so.)
__global__ void __launch_bounds__(256)
k_plan_count(const DevBox *__restrict__ boxes, uint32_t *cellinfo, uint32_t *bucket_cnt,
             int cell_blocks, float4 *cot_sorted) {
    const DevBox &B = boxes[blockIdx.y];
    if ((int)blockIdx.x >= cell_blocks) {
        gather_cot(B, cot_sorted, (int64_t)(blockIdx.x - cell_blocks) * 256 + threadIdx.x);
        return;
    }
    __shared__ uint32_t h[kKinds * kBuckets];
    __shared__ int dcell[256], dsum[256];
    __shared__ int nd;
    for (int t = threadIdx.x; t < kKinds * kBuckets; t += 256) h[t] = 0;
    dsum[threadIdx.x] = 0;
    if (threadIdx.x == 0) nd = 0;
    __syncthreads();
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int K = B.K;
    const gptr<const int32_t> cs = gp(B.cell_start);
    CellItems it{0, 0};
    int at = 0;
    if (c < B.ncell) {
        it = cell_items(cs[c + 1] - cs[c], B.dense_min, B.narrow_max);
        if (it.ndense) {
            at = atomicAdd(&nd, 1);
            dcell[at] = c;
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nd * kRows; t += 256) {
        const int d = dcell[t / kRows];
        atomicAdd(&dsum[t / kRows],
                  row_sources(cs, K, d / (K * K), (d / K) % K, d % K, t % kRows));
    }
    __syncthreads();
    if (c < B.ncell) {
        uint32_t info = 0;
        if (it.ndense) {
            const int b = cost_bucket((float)dsum[at]);
            atomicAdd(&h[b], (uint32_t)it.ndense);
            info |= (uint32_t)(b + 1);
        }
        if (it.light) {
            // light items run in spatial order (slabs of consecutive cells):
            // neighbouring items share their sources in L2
            const int b = kBuckets - 1 - (int)((int64_t)c * kBuckets / B.ncell);
            atomicAdd(&h[it.light * kBuckets + b], 1u);
            info |= (uint32_t)(b + 1) << 16;
        }
        cellinfo[B.cellbase + c] = info;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kKinds * kBuckets; t += 256)
        if (h[t]) atomicAdd(&bucket_cnt[t], h[t]);
}

// Heavy dense items, the first of the list: those of more than 1 / share of all
// dense items' sources, which one wave each would still be summing when the rest
// of the call is done.  A lane's buckets b0 and b0 - 1 hold c0 and c1 items.
// Whole calls with half the share / this / twice, us, of clustered boxes (particles a
// cell and spread of ln density 8 and 1.0; 8 and 1.5; 8 and 2.0; 14 and 1.5): plain 100k 131 / 132 / 131, 170 / 173 / 176,
// 291 / 221 / 240, 272 / 222 / 238; 200k 195 / 198 / 199, 315 / 285 / 306, 351 / 333 / 352,
// 363 / 329 / 383; 340k 262 / 275 / 275, 352 / 300 / 322, 496 / 471 / 428, 543 / 487 / 494.
// Compensated VJP 100k 187 / 186 / 187, 269 / 251 / 253, 436 / 341 / 351, 420 / 346 / 347; 200k
// 290 / 292 / 292, 559 / 450 / 460, 952 / 522 / 516, 724 / 543 / 583; 340k 405 / 405 / 404, 614 /
// 503 / 525, 1034 / 825 / 763, 1082 / 831 / 845.
constexpr float kHeavyShareAccel = 1000.0f, kHeavyShareVjp = 1400.0f;
__device__ __forceinline__ uint32_t heavy_items(int b0, int c0, int c1, float share) {
    const float s0 = exp2f(0.25f * (float)b0), s1 = exp2f(0.25f * (float)(b0 - 1));
    float all = (float)c0 * s0 + (float)c1 * s1;
    for (int o = 32; o >= 1; o >>= 1) all += __shfl_xor(all, o, 64);
    const float least = all / share;
    uint32_t n = (s0 > least ? (uint32_t)c0 : 0u) + (s1 > least ? (uint32_t)c1 : 0u);
    for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);
    return n;
}

// Items into their bucket ranges: each block adds up the bucket counts of all
// blocks (highest bucket first), reserves one range per non-empty bucket with a
// global atomic and places its cells by LDS ranks.  The order inside a bucket
// depends on timing; every item's result does not.  Narrow items follow the
// light ones in the same array.
__global__ void __launch_bounds__(256)
k_plan_emit(const DevBox *__restrict__ boxes, const uint32_t *__restrict__ cellinfo,
            const uint32_t *__restrict__ bucket_cnt, uint32_t *bucket_cur, uint32_t *totals,
            Item *dense, Item *light, float heavy_share) {
    __shared__ uint32_t h[kKinds * kBuckets];
    __shared__ uint32_t base[kKinds * kBuckets];
    __shared__ uint32_t tot[kKinds];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave < kKinds) {   // one wave per kind, two buckets per lane
        static_assert(kBuckets == 128 && kKinds < 4, "two buckets per lane");
        const int b0 = wave * kBuckets + kBuckets - 1 - 2 * lane;
        const int c0 = (int)bucket_cnt[b0], c1 = (int)bucket_cnt[b0 - 1];
        const int x = scan_lanes<64>(c0 + c1);
        base[b0] = (uint32_t)(x - c0 - c1);
        base[b0 - 1] = (uint32_t)(x - c1);
        if (lane == 63) {
            tot[wave] = (uint32_t)x;
            if (blockIdx.x == 0 && blockIdx.y == 0) totals[wave] = (uint32_t)x;
        }
        if (wave == 0 && blockIdx.x == 0 && blockIdx.y == 0) {
            const uint32_t heavy = heavy_items(b0, c0, c1, heavy_share);
            if (lane == 0) totals[3] = heavy;
        }
    }
    for (int t = threadIdx.x; t < kKinds * kBuckets; t += 256) h[t] = 0;
    __syncthreads();
    const DevBox &B = boxes[blockIdx.y];
    const int c = blockIdx.x * 256 + threadIdx.x;
    uint32_t info = 0, rd = 0, rl = 0;
    int n = 0, bd = 0, bl = 0;
    CellItems it{0, 0};
    if (c < B.ncell) {
        info = cellinfo[B.cellbase + c];
        if (info) {
            n = gp(B.cell_start)[c + 1] - gp(B.cell_start)[c];
            it = cell_items(n, B.dense_min, B.narrow_max);
            bd = (int)(info & 0xffffu) - 1;
            bl = (int)(info >> 16) - 1;
            if (it.ndense) rd = atomicAdd(&h[bd], (uint32_t)it.ndense);
            if (it.light) rl = atomicAdd(&h[it.light * kBuckets + bl], 1u);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kKinds * kBuckets; t += 256)
        if (h[t]) base[t] += atomicAdd(&bucket_cur[t], h[t]);
    __syncthreads();
    if (it.ndense) {
        const uint32_t at = base[bd] + rd;
        for (int k = 0; k < it.ndense; ++k) dense[at + k] = Item{(int)blockIdx.y, c, 1, k};
    }
    if (it.light) {
        const uint32_t at = (it.light == 2 ? tot[1] : 0u) + base[it.light * kBuckets + bl] + rl;
        light[at] = Item{(int)blockIdx.y, c, 1, n / kUnit};
    }
}

// ------------------------------------------------------------------ pair arithmetic

struct Acc {
    float x = 0.f, y = 0.f, z = 0.f;
    float cx = 0.f, cy = 0.f, cz = 0.f;   // Kahan compensation (negated low parts)
};

__device__ __forceinline__ void kahan(float &s, float &c, float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

template <bool COMP>
__device__ __forceinline__ void fold(Acc &a, float px, float py, float pz) {
    if constexpr (COMP) {
        kahan(a.x, a.cx, px);
        kahan(a.y, a.cy, py);
        kahan(a.z, a.cz, pz);
    } else {
        a.x += px;
        a.y += py;
        a.z += pz;
    }
}

struct Coef {
    float cA, cB, cC, cC2, eps2;
    float floor;   // added to r^2 (DevBox::r2floor)
};

// Keep a uniform value in a vector register: an FP32 operation that reads a
// scalar register issues at half the rate of one that reads vector registers
// only (measured 4.4 against 2.4 clocks per wave instruction).
__device__ __forceinline__ void in_vector(float &x) { asm volatile("" : "+v"(x)); }

// One pair of the acceleration sum; SPLINE selects Eq. 2's single-min form,
// otherwise the pair is known to lie outside eps (Newton branch).  Outside
// eps the spline lies above r^-3 (their difference is 10 (r/eps - 1)^3 in
// units of eps^-3), so the min form is evaluated only when some lane of the
// wave has r^2 < eps^2, which few pairs do: a compare per pair instead of
// the polynomial and the min.  (The empty volatile asm keeps the rare branch
// a branch instead of letting the compiler evaluate both sides.)
template <bool SPLINE>
__device__ __forceinline__ void pair_accel(float sx, float sy, float sz, float xi, float yi,
                                           float zi, const Coef &k, float &px, float &py,
                                           float &pz) {
    const float rx = sx - xi, ry = sy - yi, rz = sz - zi;
    float r2 = __builtin_fmaf(rx, rx, k.floor);
    r2 = __builtin_fmaf(ry, ry, r2);
    r2 = __builtin_fmaf(rz, rz, r2);
    const float q = __builtin_amdgcn_rsqf(r2);
    float f = q * q * q;
    if constexpr (SPLINE) {
        const bool in = r2 < k.eps2;
        if (__any(in)) {
            asm volatile("");
            const float rho = r2 * q;
            const float g = fminf(__builtin_fmaf(__builtin_fmaf(k.cC, rho, k.cB), rho, k.cA), f);
            f = in ? g : f;
        }
    }
    px = __builtin_fmaf(f, rx, px);
    py = __builtin_fmaf(f, ry, py);
    pz = __builtin_fmaf(f, rz, pz);
}

// N pairs of the acceleration sum from their separations r, added in order; the
// spline's branch is taken once for all of them.
template <bool SPLINE, int N>
__device__ __forceinline__ void pair_accelN(const float (&rx)[N], const float (&ry)[N],
                                            const float (&rz)[N], const Coef &k, float &px,
                                            float &py, float &pz) {
    float r2[N], q[N], f[N];
    bool in = false;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        r2[u] = __builtin_fmaf(rx[u], rx[u], k.floor);
        r2[u] = __builtin_fmaf(ry[u], ry[u], r2[u]);
        r2[u] = __builtin_fmaf(rz[u], rz[u], r2[u]);
        q[u] = __builtin_amdgcn_rsqf(r2[u]);
        f[u] = q[u] * q[u] * q[u];
        if constexpr (SPLINE) in |= r2[u] < k.eps2;
    }
    if constexpr (SPLINE) {
        if (__any(in)) {
            asm volatile("");
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float rho = r2[u] * q[u];
                const float g =
                    fminf(__builtin_fmaf(__builtin_fmaf(k.cC, rho, k.cB), rho, k.cA), f[u]);
                f[u] = r2[u] < k.eps2 ? g : f[u];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        px = __builtin_fmaf(f[u], rx[u], px);
        py = __builtin_fmaf(f[u], ry[u], py);
        pz = __builtin_fmaf(f[u], rz[u], pz);
    }
}

// The same from the sources' offsets sx, sy, sz.
template <bool SPLINE>
__device__ __forceinline__ void pair_accel4(const float (&sx)[4], const float (&sy)[4],
                                            const float (&sz)[4], float xi, float yi, float zi,
                                            const Coef &k, float &px, float &py, float &pz) {
    float rx[4], ry[4], rz[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        rx[u] = sx[u] - xi;
        ry[u] = sy[u] - yi;
        rz[u] = sz[u] - zi;
    }
    pair_accelN<SPLINE, 4>(rx, ry, rz, k, px, py, pz);
}

// N pairs of the VJP, added in order: xbar_i += g (v_j - v_i) + h (r .
// (v_j - v_i)) r, with g = F/r and h = g'(rho)/rho, written as
// xbar_i += A (u + W r) with u = v_j - v_i, A = g and W = h (r . u) / g.
// Outside eps (Newton, or Plummer through the r^2 floor) A = q^3 and
// W = -3 q^2 (r . u): 23 VALU.  Inside eps g = cA + cB rho + cC rho^2 > 0 and
// h = cB / rho + 2 cC = cB q + 2 cC.  With SPLINE the inside coefficients
// replace the Newton ones only when some lane of the wave has one of the N
// pairs inside eps (a compare per pair otherwise), as in pair_accel; the
// branch rewrites A and W only, so the sums are updated outside it.
template <bool SPLINE, int N>
__device__ __forceinline__ void pair_vjp_sum(const float (&rx)[N], const float (&ry)[N],
                                             const float (&rz)[N], const float (&ux)[N],
                                             const float (&uy)[N], const float (&uz)[N],
                                             const Coef &k, float &px, float &py, float &pz) {
    float r2[N], q[N], rdu[N], A[N], W[N];
    bool in = false;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        r2[u] = __builtin_fmaf(rx[u], rx[u], k.floor);
        r2[u] = __builtin_fmaf(ry[u], ry[u], r2[u]);
        r2[u] = __builtin_fmaf(rz[u], rz[u], r2[u]);
        q[u] = __builtin_amdgcn_rsqf(r2[u]);
        rdu[u] = rx[u] * ux[u];
        rdu[u] = __builtin_fmaf(ry[u], uy[u], rdu[u]);
        rdu[u] = __builtin_fmaf(rz[u], uz[u], rdu[u]);
        const float q2 = q[u] * q[u];
        A[u] = q2 * q[u];
        W[u] = (-3.0f * q2) * rdu[u];
        if constexpr (SPLINE) in |= r2[u] < k.eps2;
    }
    if constexpr (SPLINE) {
        if (__any(in)) {
            asm volatile("");   // keep the rare branch a branch
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float rho = r2[u] * q[u];
                const float g = __builtin_fmaf(__builtin_fmaf(k.cC, rho, k.cB), rho, k.cA);
                const float h = __builtin_fmaf(k.cB, q[u], k.cC2);
                const bool inside = r2[u] < k.eps2;
                A[u] = inside ? g : A[u];
                W[u] = inside ? (h * rdu[u]) / g : W[u];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        px = __builtin_fmaf(A[u], __builtin_fmaf(W[u], rx[u], ux[u]), px);
        py = __builtin_fmaf(A[u], __builtin_fmaf(W[u], ry[u], uy[u]), py);
        pz = __builtin_fmaf(A[u], __builtin_fmaf(W[u], rz[u], uz[u]), pz);
    }
}

// The same from the sources' offsets and cotangents.
template <bool SPLINE, int N>
__device__ __forceinline__ void pair_vjpN(const float (&sx)[N], const float (&sy)[N],
                                          const float (&sz)[N], const float (&vx)[N],
                                          const float (&vy)[N], const float (&vz)[N], float xi,
                                          float yi, float zi, float vxi, float vyi, float vzi,
                                          const Coef &k, float &px, float &py, float &pz) {
    float rx[N], ry[N], rz[N], ux[N], uy[N], uz[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        rx[u] = sx[u] - xi;
        ry[u] = sy[u] - yi;
        rz[u] = sz[u] - zi;
        ux[u] = vx[u] - vxi;
        uy[u] = vy[u] - vyi;
        uz[u] = vz[u] - vzi;
    }
    pair_vjp_sum<SPLINE, N>(rx, ry, rz, ux, uy, uz, k, px, py, pz);
}

template <bool SPLINE>
__device__ __forceinline__ void pair_vjp(float sx, float sy, float sz, float vx, float vy,
                                         float vz, float xi, float yi, float zi, float vxi,
                                         float vyi, float vzi, const Coef &k, float &px,
                                         float &py, float &pz) {
    const float ax[1] = {sx}, ay[1] = {sy}, az[1] = {sz}, bx[1] = {vx}, by[1] = {vy},
                bz[1] = {vz};
    pair_vjpN<SPLINE, 1>(ax, ay, az, bx, by, bz, xi, yi, zi, vxi, vyi, vzi, k, px, py, pz);
}

// Final value of a lane's sum (compensation folded in).
template <bool COMP>
__device__ __forceinline__ float3 value(const Acc &a) {
    if constexpr (COMP) return make_float3(a.x - a.cx, a.y - a.cy, a.z - a.cz);
    return make_float3(a.x, a.y, a.z);
}

// Scaled result of sorted slot `slot` to caller index i = order[slot] (read
// by the caller early, so that its latency hides behind the sum).
__device__ __forceinline__ void store(const DevBox &B, int i, float3 f) {
    if (i >= 0 && i < B.n) {   // always true for a consistent binning
        gptr<float> o = gp(B.out) + 3 * (int64_t)i;
        o[0] = f.x * B.scale;
        o[1] = f.y * B.scale;
        o[2] = f.z * B.scale;
    }
}

// ------------------------------------------------------------------ dense path

typedef const __attribute__((address_space(4))) float cfloat;
typedef const __attribute__((address_space(1))) float gfloat;

// Float4 number i of a global array through a global-address-space pointer
// (plain pointers loaded from a descriptor compile to flat loads).  The index
// is 64-bit: VJP records are addressed by 2 (base + slot), which exceeds 2^31
// once the boxes of a call hold more than 2^30 particles.
__device__ __forceinline__ float4 ld_global4(gfloat *p, int64_t i) {
    gfloat *q = p + 4 * i;
    return make_float4(q[0], q[1], q[2], q[3]);
}

// N sources' records (16 bytes each, 32 for the VJP) from p on, by scalar loads
// of up to 64 bytes (one s_load_dwordx16 instead of a load per coordinate).
typedef float rec4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float rec8 __attribute__((ext_vector_type(8), aligned(4)));
typedef float rec16 __attribute__((ext_vector_type(16), aligned(4)));
template <int WORDS>
struct Rec {
    float w[WORDS];
};
template <int WORDS>
__device__ __forceinline__ Rec<WORDS> load_rec(cfloat *p) {
    Rec<WORDS> r;
    if constexpr (WORDS > 16) {
#pragma unroll
        for (int k = 0; k < WORDS / 16; ++k) {
            const rec16 v = *(const __attribute__((address_space(4))) rec16 *)(p + 16 * k);
#pragma unroll
            for (int i = 0; i < 16; ++i) r.w[16 * k + i] = v[i];
        }
    } else if constexpr (WORDS == 16) {
        const rec16 v = *(const __attribute__((address_space(4))) rec16 *)p;
#pragma unroll
        for (int i = 0; i < 16; ++i) r.w[i] = v[i];
    } else if constexpr (WORDS == 8) {
        const rec8 v = *(const __attribute__((address_space(4))) rec8 *)p;
#pragma unroll
        for (int i = 0; i < 8; ++i) r.w[i] = v[i];
    } else {
        const rec4 v = *(const __attribute__((address_space(4))) rec4 *)p;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.w[i] = v[i];
    }
    return r;
}

// The lane's separations from N sources (and the cotangent differences): the
// only operations that read the scalar registers of a group.
template <int MODE, int N>
struct Sep {
    float x[N], y[N], z[N], u[MODE == 1 ? N : 1], v[MODE == 1 ? N : 1], w[MODE == 1 ? N : 1];
};
template <int MODE, int N>
__device__ __forceinline__ Sep<MODE, N> separations(const Rec<N * (MODE == 0 ? 4 : 8)> &r, float xs,
                                                    float ys, float zs, const float4 &vi) {
    constexpr int W = MODE == 0 ? 4 : 8;
    Sep<MODE, N> d;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        d.x[i] = r.w[W * i] - xs;
        d.y[i] = r.w[W * i + 1] - ys;
        d.z[i] = r.w[W * i + 2] - zs;
        if constexpr (MODE == 1) {
            d.u[i] = r.w[W * i + 4] - vi.x;
            d.v[i] = r.w[W * i + 5] - vi.y;
            d.w[i] = r.w[W * i + 6] - vi.z;
        }
    }
    return d;
}
template <int MODE, bool SPLINE, int N>
__device__ __forceinline__ void sum_sep(const Sep<MODE, N> &d, const Coef &k, float &px, float &py,
                                        float &pz) {
    if constexpr (MODE == 0)
        pair_accelN<SPLINE, N>(d.x, d.y, d.z, k, px, py, pz);
    else
        pair_vjp_sum<SPLINE, N>(d.x, d.y, d.z, d.u, d.v, d.w, k, px, py, pz);
}

// Sources [j0, j1) of one cell through scalar loads, in groups of kGroup, then
// 2 and 1.  A group's registers are read by the separations alone; the next
// group's load is issued right behind them (scalar loads return out of order,
// so there is no waiting for one while a later one is in flight) and completes
// while this group is summed.  With eight loads per group and none ahead the
// kernel waited on them: 128^3 clustered particles, 1.55e9 pairs in dense items,
// alone 690 -> 556 us (plain), 1259 -> 1044 us (VJP, two sources a group: four
// take 86 registers, five waves per SIMD instead of seven).
template <int MODE, bool SPLINE, bool COMP>
__device__ __forceinline__ void run_scalar(cfloat *__restrict__ src, int j0, int j1, float xs,
                                           float ys, float zs, float4 vi, const Coef &k, int flush,
                                           Acc &acc) {
    // the block's first source through a 64-bit address (4 j0 passes 2^31 for
    // j0 >= 2^29); inside a block 32-bit offsets
    constexpr int W = MODE == 0 ? 4 : 8;   // floats per source
    constexpr int kGroup = MODE == 0 ? 4 : 2;
    cfloat *p = src + (int64_t)W * j0;
    int j = j0;
    while (j < j1) {
        // compensated: plain partials of at most flush terms; plain: one run
        const int blk = COMP ? min(j1 - j, flush) : j1 - j;
        float px = 0.f, py = 0.f, pz = 0.f;
        if constexpr (!COMP) {
            px = acc.x;
            py = acc.y;
            pz = acc.z;
        }
        int left = blk;
        if (left >= kGroup) {
            Rec<kGroup * W> r = load_rec<kGroup * W>(p);
            for (;;) {
                const Sep<MODE, kGroup> d = separations<MODE, kGroup>(r, xs, ys, zs, vi);
                __builtin_amdgcn_sched_barrier(0);
                left -= kGroup;
                p += W * kGroup;
                // (after the last group: some group of this run again, unused)
                r = load_rec<kGroup * W>(left >= kGroup ? p : p - W * kGroup);
                __builtin_amdgcn_sched_barrier(0);
                sum_sep<MODE, SPLINE, kGroup>(d, k, px, py, pz);
                if (left < kGroup) break;
            }
        }
        if (kGroup > 2 && (left & 2)) {
            const Sep<MODE, 2> d = separations<MODE, 2>(load_rec<2 * W>(p), xs, ys, zs, vi);
            sum_sep<MODE, SPLINE, 2>(d, k, px, py, pz);
            p += 2 * W;
        }
        if (left & 1) {
            const Sep<MODE, 1> d = separations<MODE, 1>(load_rec<W>(p), xs, ys, zs, vi);
            sum_sep<MODE, SPLINE, 1>(d, k, px, py, pz);
            p += W;
        }
        j += blk;
        if constexpr (COMP) {
            fold<true>(acc, px, py, pz);
        } else {
            acc.x = px;
            acc.y = py;
            acc.z = pz;
        }
    }
}

// Dense items by one wave each, drawn from the queues at counter.
template <int MODE, bool COMP>
__device__ __forceinline__ void dense_items(const int lane, const DevBox *__restrict__ boxes,
                                            const Item *__restrict__ items, int nitems,
                                            uint32_t *counter,
                                            const float4 *__restrict__ cot_sorted) {
    // one queue per XCD (workgroup w runs on XCD w % 8): XCD x takes the
    // blocks of up to kDenseBlock consecutive items c = x, x + 8, ... in order, so
    // the chunks of one cell, which share every source, meet in one L2, and
    // the heaviest items still come first everywhere (the map is one-to-one
    // and increasing, so only the locality depends on the placement)
    const int x = (int)(blockIdx.x % kXcds);
    const int mask = xcd_block_mask(nitems, kDenseBlock);
    uint32_t *dq = counter + kQueueStride * x;
    for (;;) {
        int t = 0;
        if (lane == 0)
            t = (int)__hip_atomic_fetch_add(gp(dq), 1u, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
        const int itx = xcd_item(uni(t), x, mask);
        if (itx >= nitems) break;
        const gptr<const Item> ip = gp(items) + itx;
        const Item I{ip->box, ip->cell0, ip->m, ip->chunk};
        const DevBox &B = boxes[I.box];
        const int K = B.K;
        const int cx = I.cell0 / (K * K), cy = (I.cell0 / K) % K, z = I.cell0 % K;
        const gptr<const int32_t> cs = gp(B.cell_start);
        const int s0 = uni(cs[I.cell0] + kUnit * I.chunk);
        const int g = uni(min(cs[I.cell0 + 1] - s0, kUnit));
        // Lanes beyond the g sinks repeat sink 0 and are dropped at the store:
        // the loop below stays convergent, so every lane holds its row's cell
        // ranges when they are read back with readlane.
        const bool active = lane < g;
        const int slot = s0 + (active ? lane : 0);
        const float4 oi = ld_global4((gfloat *)B.off, slot);
        const int dst = gp(B.order)[slot];
        float4 vi = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (MODE == 1) vi = ld_global4((gfloat *)cot_sorted, 2 * (B.base + slot) + 1);
        Coef k{B.cA, B.cB, B.cC, 2.0f * B.cC, B.eps * B.eps, B.r2floor};
        in_vector(k.floor);
        const bool fast = B.outer_newton != 0;
        const bool plummer = B.plummer != 0;   // Plummer law: one branch for every pair
        const int flush = uni(B.flush);
        // pair symmetry: the sinks of a symmetric cell skip the sources of
        // their symmetric partner cells (summed once by the pair kernel) and
        // leave their sum in partial slot 0
        const int nX = uni(cs[I.cell0 + 1] - cs[I.cell0]);
        const bool f4sink = MODE == 0 && B.f4tot != nullptr && uni((int)gp(B.f4tot)[0]) != 0 &&
                            f4_symmetric_cell(nX, B.dense_min);
        cfloat *src = (cfloat *)B.off;
        // the VJP reads sources from the 32-byte records (offset, cotangent)
        cfloat *cot = (cfloat *)(cot_sorted + 2 * B.base);
        if constexpr (MODE == 1) src = cot;
        // cell ranges of the 125 source cells: lane r < 25 holds row r's five
        // (start, end) pairs, read back with readlane (uniform, no memory wait)
        int cb[5], ce[5];
        {
            const int r = lane < kRows ? lane : 0;
            const int rb = (wrapk(cx + r / 5 - 2, K) * K + wrapk(cy + r % 5 - 2, K)) * K;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int c = rb + wrapk(z + q - 2, K);
                cb[q] = cs[c];
                ce[q] = cs[c + 1];
            }
        }
        Acc acc;
        {
            for (int r = 0; r < kRows; ++r) {
                const int dx = r / 5 - 2, dy = r % 5 - 2;
                const bool in_row = dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1;
                const float xs = oi.x - (float)dx, ys = oi.y - (float)dy;
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const int dz = q - 2;
                    const int cbq = __builtin_amdgcn_readlane(cb[q], r);
                    const int ceq = __builtin_amdgcn_readlane(ce[q], r);
                    const int j0 = max(cbq, 0);
                    const int j1 = min(ceq, B.n);
                    if (j0 >= j1) continue;
                    if (f4sink && !(r == 12 && q == 2) && f4_symmetric_cell(ceq - cbq, B.dense_min))
                        continue;
                    const float zs = oi.z - (float)dz;
                    if (!plummer && (!fast || (in_row && dz >= -1 && dz <= 1)))
                        run_scalar<MODE, true, COMP>(src, j0, j1, xs, ys, zs, vi, k, flush, acc);
                    else
                        run_scalar<MODE, false, COMP>(src, j0, j1, xs, ys, zs, vi, k, flush, acc);
                }
            }
        }
        if (f4sink) {
            if (active) {
                const int64_t gX = B.cellbase + I.cell0;
                const uint64_t idx = (uint64_t)gp(B.f4off)[gX] + (uint64_t)(kUnit * I.chunk + lane);
                if constexpr (COMP) {
                    st_g4(B.f4part, 2 * idx, acc.x, acc.y, acc.z);
                    st_g4(B.f4part, 2 * idx + 1, -acc.cx, -acc.cy, -acc.cz);
                } else {
                    st_g4(B.f4part, idx, acc.x, acc.y, acc.z);
                }
            }
        } else if (active) {
            store(B, dst, value<COMP>(acc));
        }
    }
}

// Workgroups from the cap on leave at once where there are many items
// (launch_dense).
constexpr int kCapItems = 2048;
template <int MODE, bool COMP>
__global__ void __launch_bounds__(kUnit)
k_dense(const DevBox *__restrict__ boxes, const Item *__restrict__ items,
        const uint32_t *__restrict__ totals, uint32_t *counter,
        const float4 *__restrict__ cot_sorted, int cap) {
    const int nitems = (int)totals[0];
    if ((int)blockIdx.x >= cap && nitems >= kCapItems) return;
    dense_items<MODE, COMP>((int)threadIdx.x, boxes, items, nitems, counter, cot_sorted);
}

// ------------------------------------------------------------------ dense path, few items

// A dense item by a whole workgroup, for calls with too few dense items to fill
// the card: k_dense walks an item's sources on one wave, which alone on its
// SIMD issues an operation every 5-7 clocks, so the call lasts as long as its
// heaviest item (13 operations times up to thousands of sources).  A sink's sum
// has to run through its sources in order, but only its last operation does:
// P waves compute the pairs' factors f and vectors e (F = f e: e = r,
// or W r + u for the VJP) of groups of four sources, 64 sinks in the lanes as in
// k_dense, and leave them in LDS; three consumer waves, one per component, add
// them in order, each pair one fused multiply-add with the operands, the order
// and the compensated folds of k_dense, so the sums are the same bit for bit.
// Producers work one round of P groups ahead of the consumers, in two
// buffers, with one barrier per round.  A pair costs more than k_dense's (10 KB of
// LDS traffic and the consumers' operations per 256 pairs), so k_dense_wide (five
// producers, three workgroups a CU) takes only the heavy items this way and the
// rest a wave each; k_small (thirteen producers, one workgroup a CU) all of them.
//
// What a group is (its sources, its cell's direction, whether it ends a partial
// sum) is worked out by one thread a group, a window of groups at a time, and
// read back as two words: worked out by each producer for itself it took 87 scalar
// operations a group, more than the 75 vector operations of its pairs (65k
// particles 226 -> 184 us, VJP 268 -> 238).
template <int P>
struct WideSmem {
    static constexpr int kThreads = 64 * (P + 3);
    static constexpr int kWindow = kThreads / P * P;   // whole rounds
    float4 terms[2][P][4][64];   // per buffer and group: f, then the components of e,
                                 // four pairs a lane
    int beg[128], cnt[128], end[128];   // source cells in order: first slot, sources,
                                        // groups up to and with the cell
    int2 group[kThreads];               // first slot, and what Group unpacks
    int item;
};

// The source cells of an item in order (c = 25 (dx+2) + 5 (dy+2) + dz+2) are cut
// into groups of at most four sources of one cell, and of one partial sum in
// the compensated mode (gpb groups in a full one).
template <bool COMP>
__device__ __forceinline__ int groups_of(int n, int flush, int gpb) {
    if constexpr (!COMP) return (n + 3) >> 2;
    const int full = n / flush;
    return full * gpb + ((n - full * flush + 3) >> 2);
}

// Group k, by one thread.
template <bool COMP, int P>
__device__ __forceinline__ int2 pack_group(const WideSmem<P> &sm, int k, int flush, int gpb) {
    int c = 0;   // the cell: the first with end > k
#pragma unroll
    for (int step = 64; step >= 1; step >>= 1)
        if (sm.end[c + step - 1] <= k) c += step;
    const int cnt = sm.cnt[c];
    const int i = k - (sm.end[c] - groups_of<COMP>(cnt, flush, gpb));
    int at = 4 * i, upto = cnt;
    if constexpr (COMP) {
        const int b = i / gpb, from = b * flush;
        at = from + 4 * (i - b * gpb);
        upto = min(cnt, from + flush);
    }
    const int r = c / 5, dx = r / 5 - 2, dy = r % 5 - 2, dz = c % 5 - 2;
    const bool inner = dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
    return make_int2(sm.beg[c] + at, (min(4, upto - at) - 1) | (at + 4 >= upto ? 4 : 0) |
                                         (inner ? 8 : 0) | (dx + 2) << 4 | (dy + 2) << 8 |
                                         (dz + 2) << 12);
}
struct Group {
    int count;
    bool ends, inner;
    int dx, dy, dz;
    __device__ __forceinline__ explicit Group(int w)
        : count((w & 3) + 1), ends(w & 4), inner(w & 8), dx(((w >> 4) & 15) - 2),
          dy(((w >> 8) & 15) - 2), dz((w >> 12) - 2) {}
};

// Four records from slot j on; past the array's end the last valid slot again.
// Accelerations by vector loads of one address (zero: a lane register that
// holds 0): operations on scalar registers issue at half the rate.  The VJP's 32
// registers would cost it a workgroup a CU: scalar loads.
template <int MODE>
__device__ __forceinline__ Rec<4 * (MODE == 0 ? 4 : 8)> load_group(cfloat *src, int j, int n,
                                                                   int zero) {
    constexpr int W = MODE == 0 ? 4 : 8;
    Rec<4 * W> r;
    if constexpr (MODE == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            gfloat *p = (gfloat *)src + (int64_t)W * min(j + u, n - 1) + zero;
            // (only what is used: a dead register of a load in flight would be
            // taken for something else, which waits for the load)
#pragma unroll
            for (int i = 0; i < 3; ++i) r.w[W * u + i] = p[i];
        }
    } else {
        if (j + 4 <= n) return load_rec<4 * W>(src + (int64_t)W * j);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const Rec<W> x = load_rec<W>(src + (int64_t)W * min(j + u, n - 1));
#pragma unroll
            for (int i = 0; i < W; ++i) r.w[W * u + i] = x.w[i];
        }
    }
    return r;
}

// f and e of four pairs: the terms of pair_accelN and pair_vjp_sum without their
// last operation.
template <int MODE, bool SPLINE>
__device__ __forceinline__ void pair_terms(const Sep<MODE, 4> &d, const Coef &k, float (&f)[4],
                                           float (&ex)[4], float (&ey)[4], float (&ez)[4]) {
    float r2[4], q[4], W[4], rdu[4];
    bool in = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        r2[u] = __builtin_fmaf(d.x[u], d.x[u], k.floor);
        r2[u] = __builtin_fmaf(d.y[u], d.y[u], r2[u]);
        r2[u] = __builtin_fmaf(d.z[u], d.z[u], r2[u]);
        q[u] = __builtin_amdgcn_rsqf(r2[u]);
        if constexpr (MODE == 0) {
            f[u] = q[u] * q[u] * q[u];
        } else {
            rdu[u] = d.x[u] * d.u[u];
            rdu[u] = __builtin_fmaf(d.y[u], d.v[u], rdu[u]);
            rdu[u] = __builtin_fmaf(d.z[u], d.w[u], rdu[u]);
            const float q2 = q[u] * q[u];
            f[u] = q2 * q[u];
            W[u] = (-3.0f * q2) * rdu[u];
        }
        if constexpr (SPLINE) in |= r2[u] < k.eps2;
    }
    if constexpr (SPLINE) {
        if (__any(in)) {
            asm volatile("");
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float rho = r2[u] * q[u];
                const float g = __builtin_fmaf(__builtin_fmaf(k.cC, rho, k.cB), rho, k.cA);
                const bool inside = r2[u] < k.eps2;
                if constexpr (MODE == 0) {
                    f[u] = inside ? fminf(g, f[u]) : f[u];
                } else {
                    const float h = __builtin_fmaf(k.cB, q[u], k.cC2);
                    f[u] = inside ? g : f[u];
                    W[u] = inside ? (h * rdu[u]) / g : W[u];
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if constexpr (MODE == 0) {
            ex[u] = d.x[u];
            ey[u] = d.y[u];
            ez[u] = d.z[u];
        } else {
            ex[u] = __builtin_fmaf(W[u], d.x[u], d.u[u]);
            ey[u] = __builtin_fmaf(W[u], d.y[u], d.v[u]);
            ez[u] = __builtin_fmaf(W[u], d.z[u], d.w[u]);
        }
    }
}

// The queue's items, by a workgroup of P + 3 waves.
template <int MODE, bool COMP, int P>
__device__ __forceinline__ void wide_items(WideSmem<P> &sm, const DevBox *__restrict__ boxes,
                                           const Item *__restrict__ items, int nitems,
                                           uint32_t *counter,
                                           const float4 *__restrict__ cot_sorted) {
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const int x = (int)(blockIdx.x % kXcds);   // one queue per XCD, as k_dense
    uint32_t *dq = counter + kQueueStride * x;
    for (;;) {
        if (threadIdx.x == 0) {
            const int t = (int)__hip_atomic_fetch_add(gp(dq), 1u, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
            sm.item = t * kXcds + x;   // few items: dealt singly
        }
        __syncthreads();
        const int itx = uni(sm.item);
        __syncthreads();
        if (itx >= nitems) break;
        const gptr<const Item> ip = gp(items) + itx;
        const Item I{ip->box, ip->cell0, ip->m, ip->chunk};
        const DevBox &B = boxes[I.box];
        const int K = B.K;
        const int cx = I.cell0 / (K * K), cy = (I.cell0 / K) % K, z = I.cell0 % K;
        const gptr<const int32_t> cs = gp(B.cell_start);
        const int s0 = uni(cs[I.cell0] + kUnit * I.chunk);
        const int g = uni(min(cs[I.cell0 + 1] - s0, kUnit));
        const bool active = lane < g;   // lanes past the g sinks repeat sink 0
        const int slot = s0 + (active ? lane : 0);
        const int flush = uni(B.flush), gpb = (flush + 3) >> 2;
        if (wave == 0) {
            int ng[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = min(lane + 64 * h, 124), r = c / 5;
                const int cell = (wrapk(cx + r / 5 - 2, K) * K + wrapk(cy + r % 5 - 2, K)) * K +
                                 wrapk(z + c % 5 - 2, K);
                const int b = max(cs[cell], 0), e = min(cs[cell + 1], B.n);
                const int cnt = lane + 64 * h < 125 ? max(e - b, 0) : 0;
                sm.beg[lane + 64 * h] = b;
                sm.cnt[lane + 64 * h] = cnt;
                ng[h] = groups_of<COMP>(cnt, flush, gpb);
            }
            const int e0 = scan_lanes<64>(ng[0]), e1 = scan_lanes<64>(ng[1]);
            sm.end[lane] = e0;
            sm.end[lane + 64] = e1 + __builtin_amdgcn_readlane(e0, 63);
        }
        const bool producer = wave < P;
        const int comp = wave - P;   // of a consumer
        const float4 oi = ld_global4((gfloat *)B.off, slot);
        const int dst = gp(B.order)[slot];
        float4 vi = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (MODE == 1) vi = ld_global4((gfloat *)cot_sorted, 2 * (B.base + slot) + 1);
        Coef k{B.cA, B.cB, B.cC, 2.0f * B.cC, B.eps * B.eps, B.r2floor};
        in_vector(k.floor);
        const bool fast = B.outer_newton != 0, plummer = B.plummer != 0;
        cfloat *src = MODE == 0 ? (cfloat *)B.off : (cfloat *)(cot_sorted + 2 * B.base);
        int zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        float p = 0.f, sum = 0.f, low = 0.f;
        __syncthreads();
        const int ngroups = uni(sm.end[127]);
        for (int w0 = 0; w0 < ngroups; w0 += sm.kWindow) {
            sm.group[threadIdx.x] = pack_group<COMP, P>(
                sm, min(w0 + (int)threadIdx.x, ngroups - 1), flush, gpb);
            __syncthreads();
            const int last = min(sm.kWindow, ngroups - w0) - 1;   // the window's last group
            const int rounds = last / P + 1;
            if (producer) {
                // (past the last group a producer repeats it, and nobody reads that)
                int kg = wave;
                int2 w = sm.group[min(kg, last)], next = sm.group[min(kg + P, last)];
                auto rec = load_group<MODE>(src, uni(w.x), B.n, zero);
                for (int t = 0; t < rounds; ++t) {
                    const Group gr(uni(w.y));
                    const float xs = oi.x - (float)gr.dx, ys = oi.y - (float)gr.dy,
                                zs = oi.z - (float)gr.dz;
                    const Sep<MODE, 4> d = separations<MODE, 4>(rec, xs, ys, zs, vi);
                    w = next;
                    __builtin_amdgcn_sched_barrier(0);
                    rec = load_group<MODE>(src, uni(w.x), B.n, zero);
                    kg += P;
                    next = sm.group[min(kg + P, last)];
                    __builtin_amdgcn_sched_barrier(0);
                    float f[4], ex[4], ey[4], ez[4];
                    if (!plummer && (!fast || gr.inner))
                        pair_terms<MODE, true>(d, k, f, ex, ey, ez);
                    else
                        pair_terms<MODE, false>(d, k, f, ex, ey, ez);
                    // past the group's sources: 0 times 0 (a finite e would do
                    // for the sum, but another cell's cotangent may not be)
                    if (gr.count < 4) {
#pragma unroll
                        for (int u = 1; u < 4; ++u)
                            if (u >= gr.count) f[u] = ex[u] = ey[u] = ez[u] = 0.f;
                    }
                    float4(*o)[64] = sm.terms[t & 1][wave];
                    o[0][lane] = make_float4(f[0], f[1], f[2], f[3]);
                    o[1][lane] = make_float4(ex[0], ex[1], ex[2], ex[3]);
                    o[2][lane] = make_float4(ey[0], ey[1], ey[2], ey[3]);
                    o[3][lane] = make_float4(ez[0], ez[1], ez[2], ez[3]);
                    __syncthreads();
                }
                __syncthreads();
            } else {
                for (int t = 0; t <= rounds; ++t) {
                    if (t > 0) {
                        const int buf = (t - 1) & 1, at = (t - 1) * P;
                        const int ends = COMP ? sm.group[at + min(lane, P - 1)].y : 0;
                        constexpr int kAhead = 5;   // groups read ahead
                        float4 f[P], e[P];
                        auto read = [&](int i) {
                            f[i] = sm.terms[buf][i][0][lane];
                            e[i] = sm.terms[buf][i][1 + comp][lane];
                        };
#pragma unroll
                        for (int i = 0; i < min(P, kAhead); ++i) read(i);
#pragma unroll
                        for (int i = 0; i < P; ++i) {
                            if (i + kAhead < P) read(i + kAhead);
                            if (at + i <= last) {
                                p = __builtin_fmaf(f[i].x, e[i].x, p);
                                p = __builtin_fmaf(f[i].y, e[i].y, p);
                                p = __builtin_fmaf(f[i].z, e[i].z, p);
                                p = __builtin_fmaf(f[i].w, e[i].w, p);
                                if constexpr (COMP) {
                                    if (__builtin_amdgcn_readlane(ends, i) & 4) {
                                        kahan(sum, low, p);
                                        p = 0.f;
                                    }
                                }
                            }
                        }
                    }
                    __syncthreads();
                }
            }
        }
        if (!producer && active && dst >= 0 && dst < B.n)
            gp(B.out)[3 * (int64_t)dst + comp] = (COMP ? sum - low : p) * B.scale;
    }
}

constexpr int kProducers = 5;
constexpr int kWideThreads = 64 * (kProducers + 3);
template <int MODE, bool COMP>
__global__ void __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(6)))
k_dense_wide(const DevBox *__restrict__ boxes, const Item *__restrict__ items,
             const uint32_t *__restrict__ totals, uint32_t *counter,
             const float4 *__restrict__ cot_sorted) {
    __shared__ WideSmem<kProducers> sm;
    const int nitems = (int)totals[0], heavy = (int)totals[3];
    wide_items<MODE, COMP, kProducers>(sm, boxes, items, heavy, counter, cot_sorted);
    // Nothing heavy: all items are alike, or few.  A workgroup's waves then claim one
    // after another (1.3 us apart), so that the first waves of all workgroups take
    // the largest items; else the workgroups that start first took eight each and
    // left CUs idle.  Uniform, compensated VJP, us: 100k particles of 463 a cell 11200
    // / 6250, 262k of 152 a cell 4880 / 3670; accelerations 4590 / 3470, 2200 / 1900.
    if (heavy == 0)
        for (int i = uni(threadIdx.x >> 6); i > 0; --i) __builtin_amdgcn_s_sleep(48);
    dense_items<MODE, COMP>((int)(threadIdx.x & 63), boxes, items + heavy, nitems - heavy,
                            counter + 1, cot_sorted);
}

// ------------------------------------------------------------------ light path

// Pieces of the staged union: per row r = (dx+2)*5 + (dy+2) up to four
// contiguous global ranges.  Slots 0-1: the |dz| <= 1 part of an inner row
// (|dx|, |dy| <= 1); slots 2-3: the rest of the row (dz = -2 and +2 for an
// inner row, dz = -2..2 split at the periodic wrap for an outer row).
constexpr int kSlots = 4;
constexpr int kPiece = kRows * kSlots;

template <int MODE, int CAP, int NT>
struct LightSmem {
    union {
        float4 sx[CAP];                  // (o_x + dx, o_y + dy, o_z + dz, v_x)
        float red[6][NT];                // after the sum: slice partials (sum, compensation)
    };
    float2 sv[MODE == 1 ? CAP : 1];  // (v_y, v_z) for the VJP
    int rs[128];                     // staged start of each non-empty piece (run), ascending,
                                     // then INT_MAX
    float4 rd[kPiece];               // per run: (global minus staged index, dx, dy, z bias)
    uint32_t bm[CAP / 32];           // staging window: bit e set when a run starts at u0 + e
    int cum[CAP / 32];               // runs starting before word w of the window
    int item;                        // current item and its (box, cell)
    int ibox, icell, ichunk;
    int inner;                       // staged particles of the 27 inner cells
    int total;
};

// Sum over staged sources [lo, hi) for one lane's sink, the lane taking
// indices lo + b, lo + b + P, ...
template <int MODE, bool SPLINE, bool COMP>
__device__ __forceinline__ void segment(const float4 *__restrict__ sx, const float2 *__restrict__ sv,
                                        int lo, int hi, int b, int P, float xi, float yi,
                                        float zi, float4 vi, const Coef &k, int flush, Acc &acc) {
    const int n = hi - lo;
    const int nfull = n / P;
    int j = lo + b;
    int it = 0;
    while (it < nfull) {
        // compensated: plain partials of at most flush terms; plain: one run
        const int blk = COMP ? min(nfull - it, flush) : nfull - it;
        float px = 0.f, py = 0.f, pz = 0.f;
        if constexpr (!COMP) {
            px = acc.x;
            py = acc.y;
            pz = acc.z;
        }
        if constexpr (MODE == 0) {
            int t = 0;
            for (; t + 4 <= blk; t += 4) {
                float ax[4], ay[4], az[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 s = sx[j + u * P];
                    ax[u] = s.x;
                    ay[u] = s.y;
                    az[u] = s.z;
                }
                pair_accel4<SPLINE>(ax, ay, az, xi, yi, zi, k, px, py, pz);
                j += 4 * P;
            }
            for (; t < blk; ++t) {
                const float4 s = sx[j];
                pair_accel<SPLINE>(s.x, s.y, s.z, xi, yi, zi, k, px, py, pz);
                j += P;
            }
        } else {
            int t = 0;
            for (; t + 2 <= blk; t += 2) {
                float ax[2], ay[2], az[2], bx[2], by[2], bz[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float4 s = sx[j + u * P];
                    const float2 v = sv[j + u * P];
                    ax[u] = s.x;
                    ay[u] = s.y;
                    az[u] = s.z;
                    bx[u] = s.w;
                    by[u] = v.x;
                    bz[u] = v.y;
                }
                pair_vjpN<SPLINE, 2>(ax, ay, az, bx, by, bz, xi, yi, zi, vi.x, vi.y, vi.z, k, px,
                                     py, pz);
                j += 2 * P;
            }
            for (; t < blk; ++t) {
                const float4 s = sx[j];
                const float2 v = sv[j];
                pair_vjp<SPLINE>(s.x, s.y, s.z, s.w, v.x, v.y, xi, yi, zi, vi.x, vi.y, vi.z, k,
                                 px, py, pz);
                j += P;
            }
        }
        it += blk;
        if constexpr (COMP) {
            fold<true>(acc, px, py, pz);
        } else {
            acc.x = px;
            acc.y = py;
            acc.z = pz;
        }
    }
    if (b < n - nfull * P) {
        float px = 0.f, py = 0.f, pz = 0.f;
        const float4 s = sx[j];
        if constexpr (MODE == 0) {
            pair_accel<SPLINE>(s.x, s.y, s.z, xi, yi, zi, k, px, py, pz);
        } else {
            const float2 v = sv[j];
            pair_vjp<SPLINE>(s.x, s.y, s.z, s.w, v.x, v.y, xi, yi, zi, vi.x, vi.y, vi.z, k, px,
                             py, pz);
        }
        fold<COMP>(acc, px, py, pz);
    }
}

// Items of one class by NT threads an item (256 for light items, 64 for narrow
// ones), lane 0 .. NT-1, drawing from queue q; sync() is a barrier of the NT
// threads.  cls selects the item class: 1 light (items from the start of the
// array), 2 narrow (after the light ones).
template <int MODE, bool COMP, int CAP, int NT, class Sync>
__device__ __forceinline__ void light_items(LightSmem<MODE, CAP, NT> &sm, const int lane,
                                            const int q, Sync &sync,
                                            const DevBox *__restrict__ boxes,
                                            const Item *__restrict__ all_items,
                                            const uint32_t *__restrict__ totals, uint32_t *counter,
                                            const float4 *__restrict__ cot_sorted, int cls) {
    static_assert(CAP % NT == 0, "a staging window is whole rounds of the workgroup");
    static_assert(NT % 64 == 0 && NT <= kLightThreads, "whole waves");
    const int nitems = (int)totals[cls];
    const gptr<const Item> items = gp(all_items) + (cls == 2 ? totals[1] : 0u);

    // kQueues interleaved queues: workgroup w of k_light draws from queue q = w % kQueues
    // (a single counter would cap the item rate at what one address sustains
    // for atomics).  The workgroups of queue q run on XCD q % 8, and the
    // queues of one XCD share blocks of up to kXcdBlock consecutive items (items
    // are in spatial order, so neighbours share their sources in that XCD's
    // L2): XCD x takes the blocks c = x, x + 8, ..., its four queues taking
    // its items in turn.  (q, k) -> item is one-to-one and increasing in k,
    // so the results do not depend on where the workgroups actually run;
    // only the L2 locality does.
    uint32_t *qc = counter + kQueueStride * q;
    const int x = q % kXcds, nth = q / kXcds;
    const int mask = xcd_block_mask(nitems, kXcdBlock);
    auto queue_item = [x, nth, mask](int kth) {
        // the XCD's t-th item
        return xcd_item(kth * (kQueues / kXcds) + nth, x, mask);
    };
    if (lane == 0) {
        const int first = queue_item((int)__hip_atomic_fetch_add(gp(qc), 1u, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT));
        sm.item = first;
        if (first < nitems) {
            sm.ibox = items[first].box;
            sm.icell = items[first].cell0;
            sm.ichunk = items[first].chunk;
        }
    }
    for (;;) {
        sync();
        const int itx = uni(sm.item);
        if (itx >= nitems) break;
        const int ibox = uni(sm.ibox), cell0 = uni(sm.icell), chunk = uni(sm.ichunk);
        // claim the next item now (lane 0); its record is fetched once the setup
        // below is done, and both complete while this item runs
        int nxt = 0;
        if (lane == 0)
            nxt = queue_item((int)__hip_atomic_fetch_add(gp(qc), 1u, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT));
        const DevBox &B = boxes[ibox];
        const int K = B.K;
        const int cx = cell0 / (K * K), cy = (cell0 / K) % K, z = cell0 % K;
        const gptr<const int32_t> cs = gp(B.cell_start);
        gfloat *goff = (gfloat *)B.off;
        gfloat *gcot = (gfloat *)cot_sorted;
        const int s0 = uni(cs[cell0]) + kUnit * chunk;
        const int g = min(uni(cs[cell0 + 1]) - s0, kUnit);

        // ---- this lane's sink (sink a, source slice b), loaded before the setup
        // (the floor stays in a scalar register: in a vector one it costs the narrow
        // kernels a wave per SIMD, and putting it there waits for it before the item's
        // loads are issued.  4.2M particles plain 1956 / 1888 us, compensated VJP
        // 3245 / 3057)
        const Coef k{B.cA, B.cB, B.cC, 2.0f * B.cC, B.eps * B.eps, B.r2floor};
        const bool fast = B.outer_newton != 0;
        const int flush = uni(B.flush);
        const int P = NT / g;
        const bool active = lane < g * P;
        const int a = active ? lane % g : 0;
        const int b = active ? lane / g : 0;
        const float4 oi = ld_global4((gfloat *)B.off, s0 + a);
        const int dst = lane < g ? gp(B.order)[s0 + lane] : 0;   // lane < g stores sink lane
        float4 vi = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (MODE == 1) vi = ld_global4((gfloat *)cot_sorted, 2 * (B.base + s0 + a) + 1);

        // ---- pieces and run table: wave 0, one lane per row.  Staged layout: the
        //      inner parts of rows 0..24, then their outer parts; the non-empty
        //      pieces in that order are the runs.
        if (lane < 64) {
            const int r = lane;
            int pg[kSlots] = {0, 0, 0, 0}, pn[kSlots] = {0, 0, 0, 0};
            float pb[kSlots] = {0.f, 0.f, 0.f, 0.f};
            if (r < kRows) {
                const int dx = r / 5 - 2, dy = r % 5 - 2;
                const bool in_row = dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1;
                const int rb = (wrapk(cx + dx, K) * K + wrapk(cy + dy, K)) * K;
                // a run of z cells [za, zb] relative to the sink (za <= zb), split at the wrap
                auto run = [&](int q, int za, int zb) {
                    const int lo = z + za, hi = z + zb;
                    if (lo < 0) {   // [lo+K, K-1] then [0, hi]
                        pg[q] = cs[rb + lo + K];
                        pn[q] = cs[rb + K] - pg[q];
                        pb[q] = -(float)(z + K);
                        pg[q + 1] = cs[rb];
                        pn[q + 1] = cs[rb + hi + 1] - pg[q + 1];
                        pb[q + 1] = -(float)z;
                    } else if (hi >= K) {   // [lo, K-1] then [0, hi-K]
                        pg[q] = cs[rb + lo];
                        pn[q] = cs[rb + K] - pg[q];
                        pb[q] = -(float)z;
                        pg[q + 1] = cs[rb];
                        pn[q + 1] = cs[rb + hi - K + 1] - pg[q + 1];
                        pb[q + 1] = (float)(K - z);
                    } else {
                        pg[q] = cs[rb + lo];
                        pn[q] = cs[rb + hi + 1] - pg[q];
                        pb[q] = -(float)z;
                    }
                };
                if (in_row) {
                    run(0, -1, 1);
                    // the two single cells at dz = -2 and dz = +2
                    const int zm = z - 2, zp = z + 2;
                    const int cm = rb + wrapk(zm, K), cp = rb + wrapk(zp, K);
                    pg[2] = cs[cm];
                    pn[2] = cs[cm + 1] - pg[2];
                    pb[2] = -(float)z + (zm < 0 ? -(float)K : 0.f);
                    pg[3] = cs[cp];
                    pn[3] = cs[cp + 1] - pg[3];
                    pb[3] = -(float)z + (zp >= K ? (float)K : 0.f);
                } else {
                    run(2, -2, 2);
                }
            }
            // exclusive prefixes over rows of the inner and outer counts and of
            // the non-empty piece counts (inner | outer << 16), by a wave scan
            const int ca = pn[0] + pn[1], ce = pn[2] + pn[3];
            const int cn = ((pn[0] > 0) + (pn[1] > 0)) | (((pn[2] > 0) + (pn[3] > 0)) << 16);
            static_assert(kRows <= 32, "the row scans use lanes 0..31");
            const int ia = scan_lanes<32>(ca), ie = scan_lanes<32>(ce), in_ = scan_lanes<32>(cn);
            const int tin = __builtin_amdgcn_readlane(ia, kRows - 1);
            const int tout = __builtin_amdgcn_readlane(ie, kRows - 1);
            const int tn = __builtin_amdgcn_readlane(in_, kRows - 1);
            const int kin = tn & 0xffff, kout = tn >> 16;
            if (r < kRows) {
                const int n0 = in_ - cn;
                int start[kSlots], rank[kSlots];
                start[0] = ia - ca;
                start[1] = start[0] + pn[0];
                start[2] = tin + (ie - ce);
                start[3] = start[2] + pn[2];
                rank[0] = n0 & 0xffff;
                rank[1] = rank[0] + (pn[0] > 0);
                rank[2] = kin + (n0 >> 16);
                rank[3] = rank[2] + (pn[2] > 0);
                const float dxf = (float)(r / 5 - 2), dyf = (float)(r % 5 - 2);
#pragma unroll
                for (int q = 0; q < kSlots; ++q) {
                    if (pn[q] > 0) {
                        sm.rs[rank[q]] = start[q];
                        sm.rd[rank[q]] = make_float4(__int_as_float(pg[q] - start[q]), dxf, dyf,
                                                     pb[q]);
                    }
                }
            }
            // pad the run starts: the search reads any index below 128
            if (r >= kin + kout) sm.rs[r] = INT_MAX;
            if (r + 64 >= kin + kout) sm.rs[r + 64] = INT_MAX;
            if (r == 0) {
                sm.inner = tin;
                sm.total = tin + tout;
            }
        }
        sync();
        int nbox = 0, ncell = 0, nchunk = 0;
        if (lane == 0 && nxt < nitems) {
            nbox = items[nxt].box;
            ncell = items[nxt].cell0;
            nchunk = items[nxt].chunk;
        }
        const int total = uni(sm.total);
        const int inner = uni(sm.inner);
        const bool single = total <= CAP;

        // stage the union window [u0, u1): thread t takes elements u0 + t + NT i.
        // Wave 0 first marks the run starts inside the window in a bitmap and
        // counts, per 32-element word, the runs that start before it; the run
        // of element d is then (runs starting at or before d) - 1, one word
        // lookup and a popcount.  Every thread issues all its loads before
        // any LDS store.
        auto stage = [&](int u0, int u1) {
            constexpr int kPer = CAP / NT;
            constexpr int kWords = CAP / 32;
            static_assert(CAP % 32 == 0 && kWords <= 64, "one bitmap word per lane of wave 0");
            if (lane < 64) {
                if (lane < kWords) sm.bm[lane] = 0u;
                __builtin_amdgcn_wave_barrier();
                int before = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int v = sm.rs[lane + 64 * h];   // INT_MAX past the last run
                    if (v < u0)
                        ++before;
                    else if (v < u1)
                        atomicOr(&sm.bm[(v - u0) >> 5], 1u << ((v - u0) & 31));
                }
                __builtin_amdgcn_wave_barrier();
                const int kb = (int)__popcll(__ballot(before >= 1)) +
                               (int)__popcll(__ballot(before >= 2));
                const int c = lane < kWords ? __popc(sm.bm[lane]) : 0;
                const int x = scan_lanes<(kWords <= 32 ? 32 : 64)>(c);
                if (lane < kWords) sm.cum[lane] = kb + x - c;
            }
            sync();
            int pos[kPer], d[kPer];
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                d[i] = u0 + lane + NT * i;
                const int e = lane + NT * i;   // < CAP
                const uint32_t w = sm.bm[e >> 5];
                pos[i] = sm.cum[e >> 5] + __popc(w & (0xffffffffu >> (31 - (e & 31)))) - 1;
            }
            float4 buf[kPer], cb[kPer];
            float sh[kPer][3];
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (d[i] < u1) {
                    const float4 dsc = sm.rd[pos[i]];
                    const int gsrc = d[i] + __float_as_int(dsc.x);
                    if constexpr (MODE == 1) {   // the source's 32-byte record
                        buf[i] = ld_global4(gcot, 2 * (B.base + gsrc));
                        cb[i] = ld_global4(gcot, 2 * (B.base + gsrc) + 1);
                    } else {
                        buf[i] = ld_global4(goff, gsrc);
                    }
                    sh[i][0] = dsc.y;
                    sh[i][1] = dsc.z;
                    sh[i][2] = dsc.w;
                }
            }
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (d[i] < u1) {
                    const float4 o = buf[i];
                    float4 v = make_float4(o.x + sh[i][0], o.y + sh[i][1], o.z + (o.w + sh[i][2]),
                                           0.f);
                    if constexpr (MODE == 1) {
                        v.w = cb[i].x;
                        sm.sv[d[i] - u0] = make_float2(cb[i].y, cb[i].z);
                    }
                    sm.sx[d[i] - u0] = v;
                }
            }
            sync();
        };

        if (single) stage(0, total);

        Acc acc;
        for (int u0 = 0; u0 < total; u0 += CAP) {
            const int u1 = min(total, u0 + CAP);
            if (!single) {
                sync();
                stage(u0, u1);
            }
            if (active) {
                // Eq. 2 branch for [0, split), f = q^3 (Newton, or Plummer
                // through the r^2 floor) for [split, total)
                const int split = B.plummer ? 0 : (fast ? inner : total);
                const int mid = min(max(split, u0), u1) - u0, hi = u1 - u0;
                if (mid > 0)
                    segment<MODE, true, COMP>(sm.sx, sm.sv, 0, mid, b, P, oi.x, oi.y, oi.z, vi, k,
                                              flush, acc);
                if (hi > mid)
                    segment<MODE, false, COMP>(sm.sx, sm.sv, mid, hi, b, P, oi.x, oi.y, oi.z, vi,
                                               k, flush, acc);
            }
        }
        // ---- fixed-order pairwise sum over slices: slice b adds slice b + half
        //      (TwoSum-compensated in the compensated mode); red overlays sx
        sync();
        if constexpr (COMP) {
            sm.red[0][lane] = acc.x;
            sm.red[1][lane] = acc.y;
            sm.red[2][lane] = acc.z;
            sm.red[3][lane] = -acc.cx;
            sm.red[4][lane] = -acc.cy;
            sm.red[5][lane] = -acc.cz;
        } else {
            sm.red[0][lane] = acc.x;
            sm.red[1][lane] = acc.y;
            sm.red[2][lane] = acc.z;
        }
        sync();
        for (int span = P; span > 1;) {
            const int half = (span + 1) >> 1;
            if (active && b < span - half) {
                const int o = lane + half * g;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if constexpr (COMP) {
                        const float x = sm.red[c][lane], y = sm.red[c][o];
                        const float t = x + y;
                        const float yp = t - x;
                        const float e = (x - (t - yp)) + (y - yp);
                        sm.red[c][lane] = t;
                        sm.red[c + 3][lane] = sm.red[c + 3][lane] + sm.red[c + 3][o] + e;
                    } else {
                        sm.red[c][lane] = sm.red[c][lane] + sm.red[c][o];
                    }
                }
            }
            sync();
            span = half;
        }
        if (lane < g) {
            float3 f;
            if constexpr (COMP)
                f = make_float3(sm.red[0][lane] + sm.red[3][lane], sm.red[1][lane] + sm.red[4][lane],
                                sm.red[2][lane] + sm.red[5][lane]);
            else
                f = make_float3(sm.red[0][lane], sm.red[1][lane], sm.red[2][lane]);
            store(B, dst, f);
        }
        sync();
        if (lane == 0) {
            sm.item = nxt;
            sm.ibox = nbox;
            sm.icell = ncell;
            sm.ichunk = nchunk;
        }
    }
}

struct WorkgroupSync {
    __device__ __forceinline__ void operator()() { __syncthreads(); }
};

template <int MODE, bool COMP, int CAP, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(MODE == 0 ? 8 : 7)))
k_light(const DevBox *__restrict__ boxes, const Item *__restrict__ all_items,
        const uint32_t *__restrict__ totals, uint32_t *counter,
        const float4 *__restrict__ cot_sorted, int cls) {
    __shared__ LightSmem<MODE, CAP, NT> sm;
    WorkgroupSync sync;
    light_items<MODE, COMP, CAP, NT>(sm, (int)threadIdx.x, (int)(blockIdx.x % kQueues), sync, boxes,
                                     all_items, totals, counter, cot_sorted, cls);
}

// ------------------------------------------------------------------ small calls

// The three item classes of a small call in one launch: workgroups of sixteen
// waves take dense items (thirteen producers), then, each four waves by
// themselves, light items, then, each wave by itself, narrow items, with the
// windows, the threads an item and so the sums of the separate kernels.
constexpr int kSmallProducers = 13;
constexpr int kSmallThreads = 64 * (kSmallProducers + 3);
constexpr int kQuarters = kSmallThreads / kLightThreads;

// Barrier of the kLightThreads / 64 waves of a quarter, all of one workgroup
// and so all resident: arrivals are counted in LDS, and each waits for the last
// one of its own barrier (every wave passes the same barriers in order).
struct QuarterSync {
    uint32_t *arrived;
    uint32_t expected = 0;
    __device__ __forceinline__ void operator()() {
        expected += kLightThreads / 64;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if ((threadIdx.x & 63) == 0)
            __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <
               expected)
            __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
};
// One wave: its LDS operations complete in order.
struct WaveSync {
    __device__ __forceinline__ void operator()() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

template <int MODE>
struct SmallSmem {
    static constexpr int kLightCap = MODE == 0 ? 1024 : 768, kNarrowCap = MODE == 0 ? 256 : 192;
    union {
        WideSmem<kSmallProducers> wide;
        union {
            LightSmem<MODE, kLightCap, kLightThreads> light;
            LightSmem<MODE, kNarrowCap, kNarrowThreads> narrow[kLightThreads / kNarrowThreads];
        } part[kQuarters];
    };
    uint32_t arrived[kQuarters];
};

template <int MODE, bool COMP>
__global__ void __launch_bounds__(kSmallThreads)
k_small(const DevBox *__restrict__ boxes, const Item *__restrict__ dense,
        const Item *__restrict__ light, const uint32_t *__restrict__ totals, uint32_t *counter,
        const float4 *__restrict__ cot_sorted) {
    typedef SmallSmem<MODE> Smem;
    __shared__ __align__(16) char raw[sizeof(Smem)];
    Smem &sm = *reinterpret_cast<Smem *>(raw);
    if (threadIdx.x < kQuarters) sm.arrived[threadIdx.x] = 0u;
    // (the barriers that end this also order the zeros before the quarters')
    wide_items<MODE, COMP, kSmallProducers>(sm.wide, boxes, dense, (int)totals[0], counter,
                                            cot_sorted);
    const int quarter = uni(threadIdx.x / kLightThreads), wave = uni(threadIdx.x >> 6);
    const int x = (int)(blockIdx.x % kXcds);   // queues x, x + 8, ... are XCD x's
    auto &part = sm.part[quarter];
    QuarterSync qsync{&sm.arrived[quarter]};
    uint32_t *q = counter + kQueueStride * kXcds;
    light_items<MODE, COMP, Smem::kLightCap, kLightThreads>(
        part.light, (int)threadIdx.x % kLightThreads, x + kXcds * (quarter % (kQueues / kXcds)),
        qsync, boxes, light, totals, q, cot_sorted, 1);
    qsync();   // the light items' shared memory is free
    WaveSync wsync;
    light_items<MODE, COMP, Smem::kNarrowCap, kNarrowThreads>(
        part.narrow[wave % (kLightThreads / kNarrowThreads)], (int)(threadIdx.x & 63),
        x + kXcds * (wave % (kQueues / kXcds)), wsync, boxes, light, totals,
        q + kQueueStride * kQueues, cot_sorted, 2);
}

// ------------------------------------------------------------------ launches

// As many workgroups as the card holds, of at most `most` a CU.
template <typename Kern>
int persistent_grid(Kern kern, int threads, int most = 1 << 20) {
    int dev = 0, ncu = 0, per = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, threads, 0);
    return std::max(1, ncu) * std::max(1, std::min(per, most));
}

// A persistent grid of `most` workgroups, or fewer where the call cannot have
// that many items (every workgroup ends with one claim that finds its queue
// empty, and one counter takes about 87 M claims a second: 7168 idle workgroups
// of k_dense on eight counters took 16 us).  A multiple of the queues.
int grid_for(int most, int64_t items, int queues) {
    return (int)std::min<int64_t>(most, (items + queues - 1) / queues * queues);
}

// The dense, light and narrow kernels of one call run concurrently: the
// light and narrow kernels go to two library streams of the same device
// (default priority), forked from and joined back to the caller's stream with
// events, so the kernels share the CUs (the dense kernel uses no LDS and
// waits on scalar loads, the light kernels lean on LDS) and no kernel's tail
// runs alone.  Under graph capture the fork and joins become graph
// dependencies.  The sequence is enqueued under a lock: the events are shared
// by all calls on the device.
struct SideStream {
    hipStream_t s[2] = {nullptr, nullptr};
    hipEvent_t fork = nullptr, join[2] = {nullptr, nullptr};
};
std::mutex g_side_mu;
std::vector<SideStream> g_side;

hipError_t side_stream(SideStream &out) {   // caller holds g_side_mu
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if ((int)g_side.size() <= dev) g_side.resize(dev + 1);
    SideStream &ss = g_side[dev];
    if (!ss.join[1]) {   // created in this order, so the last one marks completion
        if (!ss.fork &&
            (e = hipEventCreateWithFlags(&ss.fork, hipEventDisableTiming)) != hipSuccess)
            return e;
        for (int k = 0; k < 2; ++k) {
            if (!ss.s[k] &&
                (e = hipStreamCreateWithFlags(&ss.s[k], hipStreamNonBlocking)) != hipSuccess)
                return e;
            if (!ss.join[k] &&
                (e = hipEventCreateWithFlags(&ss.join[k], hipEventDisableTiming)) != hipSuccess)
                return e;
        }
    }
    out = ss;
    return hipSuccess;
}

// One light-kernel instance (NT threads per item, CAP staged sources per
// round) on its persistent grid: every queue needs at least one workgroup,
// so the grid is a multiple of kQueues.
template <int MODE, bool COMP, int CAP, int NT>
hipError_t launch_light_inst(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                             uint32_t *counter, int cls, hipStream_t s) {
    static const int most =
        (persistent_grid(k_light<MODE, COMP, CAP, NT>, NT) + kQueues - 1) / kQueues * kQueues;
    const int grid = grid_for(most, tp.max_light, kQueues);
    hipLaunchKernelGGL((k_light<MODE, COMP, CAP, NT>), dim3(grid), dim3(NT), 0, s, d_boxes,
                       (const Item *)tp.light, (const uint32_t *)tp.totals, counter, cot, cls);
    return hipGetLastError();
}

// Light items: windows of 512 / 1024 / 2048 sources (the VJP, whose staged
// sources take 24 bytes instead of 16: 512 / 768 / 1536).
template <int MODE, bool COMP>
hipError_t launch_light(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                        hipStream_t s) {
    uint32_t *q = tp.counter + kQueueStride * kXcds;
    switch (tp.light_window) {
        case 512: return launch_light_inst<MODE, COMP, 512, kLightThreads>(d_boxes, tp, cot, q, 1, s);
        case 2048:
            return launch_light_inst<MODE, COMP, MODE == 0 ? 2048 : 1536, kLightThreads>(
                d_boxes, tp, cot, q, 1, s);
        default:
            return launch_light_inst<MODE, COMP, MODE == 0 ? 1024 : 768, kLightThreads>(
                d_boxes, tp, cot, q, 1, s);
    }
}

// Narrow items: windows of 128 / 256 / 512 sources (VJP: 128 / 192 / 384).
template <int MODE, bool COMP>
hipError_t launch_narrow(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                         hipStream_t s) {
    uint32_t *q = tp.counter + kQueueStride * (kXcds + kQueues);
    switch (tp.narrow_window) {
        case 128: return launch_light_inst<MODE, COMP, 128, kNarrowThreads>(d_boxes, tp, cot, q, 2, s);
        case 512:
            return launch_light_inst<MODE, COMP, MODE == 0 ? 512 : 384, kNarrowThreads>(
                d_boxes, tp, cot, q, 2, s);
        default:
            return launch_light_inst<MODE, COMP, MODE == 0 ? 256 : 192, kNarrowThreads>(
                d_boxes, tp, cot, q, 2, s);
    }
}

// k_dense_wide takes the dense items of calls of at most this many particles
// (over all boxes): above, the card is full with one wave an item and nothing
// waits for the heaviest one.  Whole force calls with k_dense / k_dense_wide, us, of
// the boxes named at kHeavyShareAccel: plain 100k 140 / 132, 228 / 173, 325 / 221, 252 / 222; 200k 188 / 198, 462 /
// 285, 388 / 333, 339 / 329; 340k 248 / 275, 286 / 300, 509 / 471, 556 / 487.
// Compensated VJP 200k 357 / 292, 927 / 450, 773 / 522, 694 / 543; 340k 398 / 405, 521 /
// 503, 1069 / 825, 1094 / 831; 420k 461 / 496, 820 / 655, 894 / 897, 1049 / 1255; 500k
// 566 / 572, 598 / 708, 1491 / 1242, 1323 / 1450; 590k 595 / 624, 764 / 790, 1581 / 1541,
// 1088 / 1244 (another draw of 8 and 1.5: 420k 608 / 564, 590k 962 / 794).
constexpr int64_t kWideMaxAccel = 350000, kWideMaxVjp = 450000;
constexpr int64_t kDenseCapAccel = 5000000, kDenseCapVjp = 2500000;   // see launch_dense

template <int MODE, bool COMP>
hipError_t launch_dense_wide(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                             hipStream_t s) {
    static const int most =
        (persistent_grid(k_dense_wide<MODE, COMP>, kWideThreads) + kXcds - 1) / kXcds * kXcds;
    const int grid = grid_for(most, tp.max_dense, kXcds);
    hipLaunchKernelGGL((k_dense_wide<MODE, COMP>), dim3(grid), dim3(kWideThreads), 0, s, d_boxes,
                       (const Item *)tp.dense, (const uint32_t *)tp.totals, tp.counter, cot);
    return hipGetLastError();
}

template <int MODE, bool COMP>
hipError_t launch_dense(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot, bool f4,
                        bool concurrent, hipStream_t s) {
    if (!f4 && tp.particles <= (MODE == 0 ? kWideMaxAccel : kWideMaxVjp))
        return launch_dense_wide<MODE, COMP>(d_boxes, tp, cot, s);
    // Beside the light kernels twelve waves a CU (VJP sixteen) are enough, and
    // leave them the slots; where dense items last after the light ones, which
    // they do in the largest boxes, they need all.  Full / capped, clustered, us:
    // accelerations 1M 762 / 739, 2.1M 1391 / 1365, 4M 2532 / 2506 (more clustered
    // 3266 / 3232, 8M 6755 / 7082); VJP 1M 1134 / 1077, 2.1M 2186 / 2161, 4M 4173 /
    // 4203.  Not with fewer than kCapItems items: a short dense kernel on few waves
    // lets the light kernels start together, and their workgroups then share the CUs
    // unevenly (full / capped, compensated: 1M uniform of 0.5 a cell 1015 / 1083, 2M
    // of 3.5 a cell 1005 / 1071, 4M of 5 a cell 1789 / 1904).  Every XCD queue needs at
    // least one workgroup: multiples of kXcds.
    static const int full =
        (persistent_grid(k_dense<MODE, COMP>, kUnit) + kXcds - 1) / kXcds * kXcds;
    static const int few =
        (persistent_grid(k_dense<MODE, COMP>, kUnit, MODE == 0 ? 12 : 16) + kXcds - 1) / kXcds *
        kXcds;
    const int grid = grid_for(full, tp.max_dense, kXcds);
    const bool capped =
        concurrent && !f4 && tp.particles <= (MODE == 0 ? kDenseCapAccel : kDenseCapVjp);
    hipLaunchKernelGGL((k_dense<MODE, COMP>), dim3(grid), dim3(kUnit), 0, s, d_boxes,
                       (const Item *)tp.dense, (const uint32_t *)tp.totals, tp.counter, cot,
                       capped ? few : grid);
    return hipGetLastError();
}

// k_small takes small calls (with the default windows, which it is built for): they
// are bound by the host, and a fork to two streams and the joins take 50 us of it.
// Small is at most kSmallOne particles, a full dense chunk for every CU, or at most
// kSmallMax of which uniform boxes would form at most kSmallPairs pairs: with more
// work, one workgroup a CU is too few for the dense items.  Whole calls, three
// kernels / k_small, us, plain, compensated and compensated VJP: 1000 particles 67 /
// 27, 67 / 28, 70 / 38; 10k of 80 a cell 270 / 181, 261 / 231, 342 / 257; 40k of 8 a
// cell (4e7 pairs) uniform 84 / 56, 87 / 59, 109 / 84, spread of ln density 1.5 101 / 89,
// 102 / 99, 139 / 133; of 14 (7e7) 149 / 161, 146 / 183, 209 / 244; 59k of 8 (6e7) uniform 95 /
// 67, 98 / 71, 125 / 101, spread 1.5 130 / 131, 136 / 151, 187 / 199; of 14 (1e8) 175 / 192,
// 181 / 223, 251 / 292; of 44 (3e8) uniform 380 / 464, 391 / 559, 550 / 724 (414, 437, 797
// before there was either).
constexpr int64_t kSmallOne = 16384;
constexpr double kSmallPairs = 6.5e7;
constexpr int64_t kSmallMax = 60000;

template <int MODE, bool COMP>
hipError_t launch_small(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                        hipStream_t s) {
    static const int most =
        (persistent_grid(k_small<MODE, COMP>, kSmallThreads) + kXcds - 1) / kXcds * kXcds;
    const int grid = grid_for(most, tp.max_dense + tp.max_light, kXcds);
    hipLaunchKernelGGL((k_small<MODE, COMP>), dim3(grid), dim3(kSmallThreads), 0, s, d_boxes,
                       (const Item *)tp.dense, (const Item *)tp.light,
                       (const uint32_t *)tp.totals, tp.counter, cot);
    return hipGetLastError();
}

template <int MODE, bool COMP>
hipError_t launch_force(const DevBox *d_boxes, const TilePlan &tp, const float4 *cot,
                        bool concurrent, hipStream_t s, const F4Plan *f4) {
    hipError_t e;
    if (!concurrent) {   // the kernels in turn on the caller's stream
        if ((e = launch_light<MODE, COMP>(d_boxes, tp, cot, s)) != hipSuccess) return e;
        if ((e = launch_narrow<MODE, COMP>(d_boxes, tp, cot, s)) != hipSuccess) return e;
        if ((e = launch_dense<MODE, COMP>(d_boxes, tp, cot, f4 != nullptr, concurrent, s)) != hipSuccess) return e;
        if (f4 && (e = f4_ring_launch(d_boxes, *f4, COMP, s)) != hipSuccess) return e;
        return hipSuccess;
    }
    const bool small = tp.particles <= kSmallOne ||
                       (tp.particles <= kSmallMax && tp.uniform_pairs <= kSmallPairs);
    if (!f4 && small && tp.light_window == kDefaultLightWindow &&
        tp.narrow_window == kDefaultNarrowWindow)
        return launch_small<MODE, COMP>(d_boxes, tp, cot, s);
    std::lock_guard<std::mutex> lk(g_side_mu);
    SideStream ss;
    if ((e = side_stream(ss)) != hipSuccess) return e;
    if ((e = hipEventRecord(ss.fork, s)) != hipSuccess) return e;
    for (int k = 0; k < 2; ++k)
        if ((e = hipStreamWaitEvent(ss.s[k], ss.fork, 0)) != hipSuccess) return e;
    if ((e = launch_dense<MODE, COMP>(d_boxes, tp, cot, f4 != nullptr, concurrent, s)) != hipSuccess) return e;
    if ((e = launch_light<MODE, COMP>(d_boxes, tp, cot, ss.s[0])) != hipSuccess) return e;
    if ((e = hipEventRecord(ss.join[0], ss.s[0])) != hipSuccess) return e;
    if ((e = launch_narrow<MODE, COMP>(d_boxes, tp, cot, ss.s[1])) != hipSuccess) return e;
    if ((e = hipEventRecord(ss.join[1], ss.s[1])) != hipSuccess) return e;
    if (f4 && (e = f4_ring_launch(d_boxes, *f4, COMP, s)) != hipSuccess) return e;
    for (int k = 0; k < 2; ++k)
        if ((e = hipStreamWaitEvent(s, ss.join[k], 0)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace

// bucket counts, then their fill cursors
int plan_buckets() { return 2 * kKinds * kBuckets; }
// dense queues (one per XCD), light queues, narrow queues, the pair kernel's
int queue_words() { return (kXcds + 2 * kQueues + 1) * kQueueStride; }

namespace {
__global__ void __launch_bounds__(256)
k_plan_export(const uint32_t *__restrict__ totals, const Item *__restrict__ dense,
              const Item *__restrict__ light, int32_t *__restrict__ out, int64_t max_items,
              int64_t *__restrict__ counts) {
    const int64_t nd = totals[0], nl = totals[1], nn = totals[2];
    const int64_t total = min(nd + nl + nn, max_items);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 3) counts[t] = t == 0 ? nd : (t == 1 ? nl : nn);
    for (int64_t i = t; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        // narrow items follow the light ones in the same array
        const Item it = i < nd ? dense[i] : light[i - nd];
        const int32_t cls = i < nd ? 0 : (i < nd + nl ? 1 : 2);
        int32_t *o = out + 4 * i;
        o[0] = it.box;
        o[1] = it.cell0;
        o[2] = it.chunk;
        o[3] = cls;
    }
}
}  // namespace

hipError_t plan_export_launch(const TilePlan &tp, int32_t *items, int64_t max_items,
                              int64_t *counts, hipStream_t s) {
    const unsigned blocks = (unsigned)std::max<int64_t>(
        1, std::min<int64_t>(4096, (max_items + 255) / 256));
    hipLaunchKernelGGL(k_plan_export, dim3(blocks), dim3(256), 0, s,
                       (const uint32_t *)tp.totals, (const Item *)tp.dense,
                       (const Item *)tp.light, items, max_items, counts);
    return hipGetLastError();
}

// The bucket counts, the fill cursors and the queue counters are zeroed by the
// call's descriptor upload.
hipError_t plan_launch(const DevBox *d_boxes, int nbox, const TilePlan &tp, float4 *cot,
                       int64_t max_n, hipStream_t s) {
    const unsigned cb = (unsigned)((tp.max_cells + 255) / 256);
    const unsigned gb = cot ? (unsigned)((max_n + 255) / 256) : 0u;
    hipLaunchKernelGGL(k_plan_count, dim3(cb + gb, (unsigned)nbox), dim3(256), 0, s, d_boxes,
                       tp.cellinfo, tp.bucket_cnt, (int)cb, cot);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_plan_emit, dim3(cb, (unsigned)nbox), dim3(256), 0, s, d_boxes,
                       (const uint32_t *)tp.cellinfo, (const uint32_t *)tp.bucket_cnt,
                       tp.bucket_cnt + kKinds * kBuckets, tp.totals, tp.dense, tp.light,
                       cot ? kHeavyShareVjp : kHeavyShareAccel);
    return hipGetLastError();
}

hipError_t tile_launch(const DevBox *d_boxes, int mode, bool compensated, const TilePlan &tp,
                       const float4 *cot, bool concurrent, hipStream_t s, const F4Plan *f4) {
    if (mode == 0)
        return compensated ? launch_force<0, true>(d_boxes, tp, cot, concurrent, s, f4)
                           : launch_force<0, false>(d_boxes, tp, cot, concurrent, s, f4);
    return compensated ? launch_force<1, true>(d_boxes, tp, cot, concurrent, s, nullptr)
                       : launch_force<1, false>(d_boxes, tp, cot, concurrent, s, nullptr);
}

}  // namespace nf
