// Exhaustive filtered k-NN (Def. 2 of the paper) on gfx950, used as ground
// truth for the approximate search.
//
//   1. Planning (bf_init ... bf_items, all on the device): each query's rank
//      interval [l, r] (Sec 4); queries ordered by octave of range size, then
//      by l, and grouped into tiles of 32, so a tile's rows are the union of
//      32 overlapping intervals of like size.  Each tile's union is cut at
//      multiples of a chunk of rows that is the same for all tiles; (tile,
//      chunk) is a work item, and the items are ordered by chunk, so that the
//      wavefronts at work at one time read the same rows (from L2).
//   2. Passes of bf_scan_kernel over the blocks of 16 rows: every 16^p-th
//      block (few enough rows to list them all), then every 16^(p-1)-th and so
//      on, each block once, to the pass over the remaining 15/16 of them.  A
//      wavefront multiplies its tile's 32 queries with a block on the fp32
//      matrix cores (v_mfma_f32_16x16x4_f32, K = 4 per instruction; the query
//      operand stays in VGPRs for d <= 128) and appends the rows whose
//      approximate squared distance |q|^2 + |x|^2 - 2 q.x lies below the
//      query's threshold to the query's list.  After each sampling pass
//      bf_select_kernel sets each query's threshold from its list: the value
//      that about 4 K' rows of the whole interval lie below, K' = 2k rounded
//      up (64 to 512), as estimated from the part scanned (more in the coarser
//      passes).  So the tests almost never hold and the scan is a stream of
//      matrix products.
//   3. bf_merge_kernel, one wavefront per query: the K' smallest of the list,
//      re-ranked with the exact canonical distance (double accumulation,
//      rounded once to float); the k smallest (distance, rank) are the result.
//      Every row not re-ranked has an approximate distance at or above the
//      last threshold or the K'-th value kept; if that minus the approximation
//      bound exceeds the k-th exact distance, the result is certified exact
//      (reported per query).
//   4. Queries whose list overflowed, because the rows follow a pattern in rank
//      order that the sampled blocks are in step with, go through 1 to 3 once
//      more with sampled blocks drawn by a hash.
//   5. Queries the margin test leaves uncertified (near-tied distances that
//      the fp32 approximation cannot separate, e.g. vectors with large norms
//      close to each other; or more ties than a list holds) are recomputed
//      exhaustively: every rank of the interval with the exact canonical
//      distance (launch_exact_ranges), so every returned row is the exact
//      filtered k-NN.
//
// The approximation bound: with unit roundoff u = 2^-24, fp32 |q|^2 and |x|^2
// (d terms each), the fp32 dot product (d products) and the final two
// operations err by at most (2d + 4) u (|q|^2 + |x|^2); the kernel uses twice
// that with |x|^2 replaced by the largest squared norm in the index.
//
// The number of uncertified queries is read back to the host, so this entry
// point synchronises `stream`; it is a ground-truth tool, not the search path.

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "ws_pool.h"
#include "search_common.h"

namespace frog {
namespace {

using namespace topk;

constexpr int kBQ = 32;          // queries per tile: two MFMA row blocks share each row block loaded
constexpr int kBBins = 512;      // buckets of l per octave of range size
constexpr int kBBands = 32;      // octaves
constexpr int kBG = 4096;        // chunks of rows at most
constexpr int kBItems = 16384;   // work items of the last pass at most (and up to two more per tile)
constexpr int kBBuf = 1024;      // candidates a wavefront buffers in LDS
constexpr int kBPasses = 7;      // at most: 2^31 rows sampled down to 16^6 times fewer
constexpr int64_t kBBatch = 16384;   // queries planned at a time at most
constexpr int64_t kBBytes = (int64_t)256 << 20;   // their lists at most
constexpr int kBTiles = (int)(kBBatch / kBQ) + kBBands;   // tiles at most
static_assert(kBTiles <= 1024, "one thread per tile");

struct BTile {
    int32_t q[kBQ];   // query index, -1 = unused
    int32_t l[kBQ];
    int32_t r[kBQ];
    int32_t ul, ur;   // union of the intervals
    int32_t lo[2], hi[2];    // per half of 16: union of the intervals (lo > hi: no query)
    int32_t ilo[2], ihi[2];  // per half of 16: intersection of the intervals
};

struct BMeta {
    unsigned long long rows;      // rows of all tiles' unions
    uint32_t places;              // places in the order, a multiple of kBQ
    uint32_t nfail;               // uncertified queries
    uint32_t nredo;               // queries to be scanned again
    uint32_t counter[kBPasses];   // work counters of the passes
    uint32_t nitems[kBPasses];
    int64_t chunk[kBPasses];      // rows per work item of each pass
};

struct BFParams {
    DevIndex ix;
    const float* Q;       // [nq][d]
    const double* lo;
    const double* hi;
    int64_t nq;
    int k;
    float maxnorm;        // largest |x|^2 in the index
    int cap;              // entries per query's list
    int64_t tmax;         // tiles at most
    int64_t imax;         // work items at most
    int npass;            // pass p scans every 16^p-th block, or one drawn of each 16^p
    bool again;           // the second time, for the queries marked in redo
    BMeta* meta;
    uint32_t* hist;       // [kBBands kBBins] queries per bucket, then the bucket's first place
    int32_t* lr;          // [nq][2] rank intervals
    uint32_t* place;      // [nq] bucket and place within it
    uint32_t* bucket;
    int32_t* order;       // [kBQ tmax] queries by bucket, each octave padded to a multiple of kBQ with -1
    BTile* tiles;         // [tmax]
    uint2* items[kBPasses];   // (tile, chunk)
    float* Qp;            // [nq][dp] zero-padded queries
    uint64_t* list;       // [nq][cap] (orderable bits of the approximate distance << 32 | row)
    int32_t* cnt;         // [nq] entries offered to the list (more than cap: it overflowed)
    float* thr;           // [nq] rows at or above it are not listed
    int32_t* redo;        // [nq] 1: the list overflowed, to be scanned again
    int32_t* fail;        // [nq][3] uncertified queries: index, l, r
    int32_t* ids;
    float* dists;
    int32_t* cert;        // or NULL
};

// ------------------------------------------------------------------ planning

__global__ void bf_init_kernel(BFParams P) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        P.meta->rows = 0ull;
        if (!P.again) P.meta->nfail = P.meta->nredo = 0u;
        for (int p = 0; p < kBPasses; ++p) P.meta->counter[p] = 0u;
    }
    if (i < kBBands * kBBins) P.hist[i] = 0u;
    if (i < kBQ * P.tmax) P.order[i] = -1;
    if (i < P.nq) {
        P.cnt[i] = 0;
        P.thr[i] = __int_as_float(0x7f800000);
        if (!P.again) P.redo[i] = 0;
    }
}

// One wavefront per query: its rank interval and a place in the bucket of
// (octave of the range size, l); the padded row of an empty range.
__global__ __launch_bounds__(kBlock) void bf_plan_kernel(BFParams P) {
    const int64_t q = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (q >= P.nq || (P.again && P.redo[q] == 0)) return;   // wave-uniform
    const int lane = lane_id();
    int64_t l, r;
    rank_interval(P.ix, P.lo[q], P.hi[q], l, r);
    for (int c = lane; c < P.ix.dp; c += 64) P.Qp[q * P.ix.dp + c] = c < P.ix.d ? P.Q[q * P.ix.d + c] : 0.f;
    if (l > r) {
        for (int j = lane; j < P.k; j += 64) {
            P.ids[q * P.k + j] = -1;
            P.dists[q * P.k + j] = __int_as_float(0x7f800000);
        }
        if (P.cert && lane == 0) P.cert[q] = 1;
    }
    if (lane == 0) {
        P.lr[2 * q] = (int32_t)l;
        P.lr[2 * q + 1] = (int32_t)r;
        if (l <= r) {
            const int band = 63 - __builtin_clzll((uint64_t)(r - l + 1));
            // the largest octaves first: their work items are the longest
            const uint32_t b = (uint32_t)((kBBands - 1 - band) * kBBins) + (uint32_t)(l * kBBins / P.ix.n);
            P.bucket[q] = b;
            P.place[q] = atomicAdd(P.hist + b, 1u);
        }
    }
}

// One workgroup: the buckets' first places, each octave padded to a multiple
// of kBQ so that no tile mixes two.
__global__ __launch_bounds__(1024) void bf_bins_kernel(BFParams P) {
    constexpr int kPer = kBBands * kBBins / 1024;   // buckets per thread
    static_assert(kBBins / kPer == 32, "an octave is 32 threads");
    __shared__ uint32_t tot[kBBands];
    const int t = threadIdx.x;
    uint32_t v[kPer], s = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        v[i] = P.hist[t * kPer + i];
        s += v[i];
    }
    uint32_t inc = s;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 32);
        if ((t & 31) >= o) inc += u;
    }
    if ((t & 31) == 31) tot[t >> 5] = (inc + kBQ - 1) / kBQ * kBQ;
    __syncthreads();
    uint32_t run = inc - s, all = 0;
    for (int b = 0; b < kBBands; ++b) {
        if (b < (t >> 5)) run += tot[b];
        all += tot[b];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        P.hist[t * kPer + i] = run;
        run += v[i];
    }
    if (t == 0) P.meta->places = all;
}

__global__ void bf_order_kernel(BFParams P) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= P.nq || P.lr[2 * q] > P.lr[2 * q + 1] || (P.again && P.redo[q] == 0)) return;
    P.order[P.hist[P.bucket[q]] + P.place[q]] = (int32_t)q;
}

// One wavefront per tile.
__global__ __launch_bounds__(kBlock) void bf_tile_kernel(BFParams P) {
    const int lane = lane_id();
    const int64_t t = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (t * kBQ >= P.meta->places) return;   // wave-uniform
    const int32_t q = lane < kBQ ? P.order[t * kBQ + lane] : -1;
    const int32_t l = q >= 0 ? P.lr[2 * (int64_t)q] : 0, r = q >= 0 ? P.lr[2 * (int64_t)q + 1] : -1;
    BTile* T = P.tiles + t;
    if (lane < kBQ) {
        T->q[lane] = q;
        T->l[lane] = l;
        T->r[lane] = r;
    }
    int32_t lo = q >= 0 ? l : INT32_MAX, hi = r, ilo = q >= 0 ? l : -1, ihi = q >= 0 ? r : INT32_MAX;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
        ilo = max(ilo, __shfl_xor(ilo, o));
        ihi = min(ihi, __shfl_xor(ihi, o));
    }
    if (lane == 0 || lane == 16) {
        T->lo[lane >> 4] = lo;
        T->hi[lane >> 4] = hi;
        T->ilo[lane >> 4] = ilo;
        T->ihi[lane >> 4] = ihi;
    }
    const int32_t ul = min(lo, __shfl(lo, 16)), ur = max(hi, __shfl(hi, 16));
    if (lane == 0) {
        T->ul = ul;
        T->ur = ur;
        atomicAdd(&P.meta->rows, (unsigned long long)((int64_t)ur - ul + 1));
    }
}

// One workgroup per pass: the rows per work item (about kBItems items in the
// last pass, a multiple of 256 rows; 4^p times that in pass p, which touches
// every 16^p-th block) and the pass's items, ordered by chunk: a counting
// sort in LDS.
__global__ __launch_bounds__(1024) void bf_items_kernel(BFParams P) {
    __shared__ uint32_t bins[kBG];
    __shared__ uint32_t wsum[16];
    __shared__ int32_t sul[kBTiles], sur[kBTiles];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = P.ix.n;
    const int ntiles = (int)(P.meta->places / kBQ);
    if (tid < ntiles) {
        sul[tid] = P.tiles[tid].ul;
        sur[tid] = P.tiles[tid].ur;
    }
    int64_t chunk = ((int64_t)P.meta->rows / kBItems + 256) / 256 * 256;
    const int64_t least = (n / kBG + 256) / 256 * 256;   // at most kBG chunks
    if (chunk < least) chunk = least;
    const int p = blockIdx.x;
    const int64_t ch = chunk << (2 * p);
    for (int i = tid; i < kBG; i += 1024) bins[i] = 0u;
    __syncthreads();
    for (int t = wave; t < ntiles; t += 16) {
        const int64_t ul = sul[t], ur = sur[t];
        for (int g = (int)(ul / ch) + lane; g <= (int)(ur / ch); g += 64) atomicAdd(&bins[g], 1u);
    }
    __syncthreads();
    // exclusive scan of the 4096 bins: four per thread
    uint32_t v[kBG / 1024], s = 0;
#pragma unroll
    for (int i = 0; i < kBG / 1024; ++i) {
        v[i] = bins[tid * (kBG / 1024) + i];
        s += v[i];
    }
    uint32_t inc = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o);
        if (lane >= o) inc += u;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t run = inc - s, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) run += wsum[w];
        all += wsum[w];
    }
#pragma unroll
    for (int i = 0; i < kBG / 1024; ++i) {
        bins[tid * (kBG / 1024) + i] = run;
        run += v[i];
    }
    __syncthreads();
    for (int t = wave; t < ntiles; t += 16) {
        const int64_t ul = sul[t], ur = sur[t];
        for (int g = (int)(ul / ch) + lane; g <= (int)(ur / ch); g += 64) {
            const uint32_t at = atomicAdd(&bins[g], 1u);
            P.items[p][at] = make_uint2((uint32_t)t, (uint32_t)g);
        }
    }
    if (tid == 0) {
        P.meta->nitems[p] = all;
        P.meta->chunk[p] = ch;
    }
}

// ------------------------------------------------------------------ scan

// The blocks (16 rows, block b = rows 16 b ..) of a pass: the multiples of
// 16^pass; but16: those of 16^(pass + 1), which an earlier pass scanned, left
// out.  DRAWN: in place of every 16th element of a pass the next coarser one
// takes one of each 16, drawn by a hash, so that no pattern of the rows is in
// step with them (it costs the scan 1 to 3 % more scalar work per block, so
// only queries that need it pay: 4,000 queries of 300k x 128 whose every 16th
// block of rows lies far away took 14.9 ms when the 2,829 lists that overflowed
// went to the exact pass at once, 2.6 ms so).
template <bool DRAWN>
struct Blocks {
    int pass;
    bool but16;
    // the drawn one of elements 16 g .. 16 g + 15 of pass p
    __device__ static __forceinline__ int32_t drawn(int32_t g, int p) {
        uint32_t x = ((uint32_t)g + ((uint32_t)p << 28)) * 0x9E3779B1u;
        x = (x ^ (x >> 15)) * 0x85EBCA77u;
        return 16 * g + (int32_t)(x >> 28);
    }
    // DRAWN: the block of element m (in [m, m + 1) 16^pass), and of the first
    // element from m on that the pass scans
    __device__ __forceinline__ int32_t block(int32_t m) const {
        for (int p = pass - 1; p >= 0; --p) m = drawn(m, p);
        return m;
    }
    __device__ __forceinline__ int32_t from(int32_t m) const {
        while (but16 && m == drawn(m >> 4, pass)) ++m;
        return block(m);
    }
    // the first block of the pass at or behind b
    __device__ __forceinline__ int32_t first(int32_t b) const {
        const int sh = 4 * pass;
        if constexpr (DRAWN) {
            const int32_t m = b >> sh;
            return from(block(m) < b ? m + 1 : m);
        }
        int32_t m = (b + (1 << sh) - 1) >> sh;
        if (but16 && (m & 15) == 0) ++m;
        return m << sh;
    }
    // the one behind block b of the pass
    __device__ __forceinline__ int32_t next(int32_t b) const {
        const int sh = 4 * pass;
        if constexpr (DRAWN) return from((b >> sh) + 1);
        b += 1 << sh;
        return but16 && ((b >> sh) & 15) == 0 ? b + (1 << sh) : b;
    }
};

// One wavefront, persistent: takes work items of the pass.  KT = dp / 16
// float4 chunks of the 32 queries' operand in registers (d <= 128: at d = 128
// 64 VGPRs and two row buffers of 32, two wavefronts per SIMD); KT = 0 streams
// queries and rows, four blocks at a time, so that six 16-byte loads feed 32
// matrix instructions.
//
// Bound by the fp32 matrix cores: at 300k x 128, 4,000 queries (log-uniform
// selectivity on [2^-10, 1]) the last pass's products take 0.38 ms at the
// peak rate and the pass 0.75 ms, all passes 1.0 ms; lists kept in order by
// insertion, 16 queries per row block and no thresholds from a sample took
// 8.0 ms.  With one row buffer at three wavefronts per SIMD the last pass
// took 0.86 ms (its loads wait for the products to have read the buffer).
// Work items grouped by XCD, a raised priority during the products and four
// accumulation chains changed nothing.
template <int KT, bool DRAWN>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KT > 4 || KT == 0 ? 2 : 3)))
void bf_scan_kernel(BFParams P, int pass, bool but16) {
    const Blocks<DRAWN> S{pass, but16};
    __shared__ uint64_t s_key[kBBuf];
    __shared__ uint8_t s_slot[kBBuf];
    __shared__ uint16_t s_off[kBBuf];
    __shared__ int32_t s_cnt[kBQ];
    __shared__ int32_t s_q[kBQ], s_l[kBQ], s_r[kBQ];
    __shared__ float s_qn[kBQ];
    constexpr int NB = KT > 0 ? 1 : 4;   // blocks at a time
    const int lane = lane_id();
    const int ii = lane & 15, kk = lane >> 4;
    const int dp = P.ix.dp, dp4 = dp >> 2;
    const int32_t n32 = (int32_t)P.ix.n;
    const float4* X4 = reinterpret_cast<const float4*>(P.ix.X);
    const uint32_t nitems = P.meta->nitems[pass];
    const int64_t chunk = P.meta->chunk[pass];
    const float inf = __int_as_float(0x7f800000);
    int fill = 0;
    // the buffered candidates to their queries' lists: each one's place among
    // its slot's in LDS, one global counter step per slot, then the stores
    // (a counter step per candidate made each block of a sampling pass, where
    // every row is a candidate, wait for eight of them in turn)
    auto flush = [&]() {
        if (fill == 0) return;
        if (lane < kBQ) s_cnt[lane] = 0;
        wave_sync();
        for (int i = lane; i < fill; i += 64) s_off[i] = (uint16_t)atomicAdd(&s_cnt[s_slot[i]], 1);
        wave_sync();
        if (lane < kBQ && s_cnt[lane] > 0) s_cnt[lane] = atomicAdd(P.cnt + s_q[lane], s_cnt[lane]);
        wave_sync();
        for (int i = lane; i < fill; i += 64) {
            const int sl = s_slot[i];
            const int32_t at = s_cnt[sl] + s_off[i];
            if (at < P.cap) P.list[(int64_t)s_q[sl] * P.cap + at] = s_key[i];
        }
        fill = 0;
        wave_sync();
    };
    for (;;) {
        uint32_t item = 0;
        if (lane == 0) item = atomicAdd(&P.meta->counter[pass], 1u);
        item = (uint32_t)uniform((int)item);
        if (item >= nitems) break;
        const uint2 it = P.items[pass][item];
        const BTile& T = P.tiles[uniform((int)it.x)];
        const int64_t c0 = (int64_t)uniform((int)it.y) * chunk;
        const int64_t row0 = c0 > T.ul ? c0 : T.ul;
        const int64_t row1 = c0 + chunk - 1 < T.ur ? c0 + chunk - 1 : T.ur;
        const int32_t bend = (int32_t)(row1 >> 4);
        int32_t b = S.first((int32_t)(row0 >> 4));
        if (b > bend) continue;
        if (lane < kBQ) {
            s_q[lane] = T.q[lane];
            s_l[lane] = T.l[lane];
            s_r[lane] = T.r[lane];
        }
        // MFMA operand mapping (16x16x4 f32): A[i][kk] in lane i + 16 kk,
        // B[kk][j] in lane j + 16 kk, D[4 (lane/16) + e][lane % 16] in
        // element e.  Lane group kk takes dimensions 16 t + 4 kk + {0..3}.
        float4 qa[2][KT > 0 ? KT : 1];
        const float4* qrow4[2] = {nullptr, nullptr};
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int32_t q = T.q[16 * g + ii];
            float qs = 0.f;
            const float4* Q4 = reinterpret_cast<const float4*>(P.Qp) + (int64_t)(q >= 0 ? q : 0) * dp4 + kk;
            if constexpr (KT > 0) {
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    const float4 v = Q4[4 * t];
                    qa[g][t] = v;
                    qs += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                }
            } else {
                qrow4[g] = Q4;
                for (int t = 0; t < dp / 16; ++t) {
                    const float4 v = Q4[4 * t];
                    qs += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                }
            }
            qs += __shfl_xor(qs, 16);
            qs += __shfl_xor(qs, 32);
            if (kk == 0) s_qn[16 * g + ii] = qs;
        }
        wave_sync();
        float qn[2][4], th[2][4];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int sl = 16 * g + 4 * kk + e;
                const int32_t q = s_q[sl];
                qn[g][e] = s_qn[sl];
                th[g][e] = q >= 0 ? P.thr[q] : -inf;
            }
        int32_t glo[2], ghi[2], gilo[2], gihi[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            glo[g] = T.lo[g];
            ghi[g] = T.hi[g];
            gilo[g] = T.ilo[g];
            gihi[g] = T.ihi[g];
        }
        // the candidates of one block and half: lane holds D[4kk + e][ii],
        // query 16 g + 4 kk + e and row 16 b + ii
        auto candidates = [&](const floatx4_t& acc, float xn, int g, int32_t blk) {
            const int32_t r0 = blk * 16, row = r0 + ii;
            float ap[4];
            bool c[4];
            bool any = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ap[e] = qn[g][e] + xn - 2.f * acc[e];
                c[e] = ap[e] < th[g][e];
                any |= c[e];
            }
            if (ballot(any) == 0) return;
            const bool inside = r0 >= gilo[g] && r0 + 15 <= gihi[g];   // within every query's interval
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int sl = 16 * g + 4 * kk + e;
                if (!inside) c[e] = c[e] & (row >= s_l[sl]) & (row <= s_r[sl]);
                const uint64_t m = ballot(c[e]);
                if (m == 0) continue;
                if (c[e]) {
                    const int at = fill + mbcnt(m);
                    s_key[at] = ((uint64_t)ord_bits(ap[e]) << 32) | (uint32_t)row;
                    s_slot[at] = (uint8_t)sl;
                }
                fill += __popcll(m);
            }
        };
        if constexpr (KT > 0) {
            auto load_rows = [&](int32_t blk, float4 (&x)[KT]) {
                const int32_t at = blk * 16 + ii;   // a block holds a row of some interval, so 16 blk < n
                const int64_t row = at < n32 ? at : n32 - 1;
#pragma unroll
                for (int t = 0; t < KT; ++t) x[t] = X4[row * dp4 + 4 * t + kk];
            };
            auto process = [&](int32_t blk, const float4 (&x)[KT]) {
                const int32_t r0 = blk * 16;
                floatx4_t acc[2];
                bool live[2];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    live[g] = r0 <= ghi[g] && r0 + 15 >= glo[g];   // uniform
                    floatx4_t a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
                    if (live[g]) {
#pragma unroll
                        for (int t = 0; t < KT; ++t) {
                            a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[g][t].x, x[t].x, a0, 0, 0, 0);
                            a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[g][t].y, x[t].y, a1, 0, 0, 0);
                            a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[g][t].z, x[t].z, a0, 0, 0, 0);
                            a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[g][t].w, x[t].w, a1, 0, 0, 0);
                        }
                    }
                    acc[g] = a0 + a1;
                }
                float xn = 0.f;
#pragma unroll
                for (int t = 0; t < KT; ++t)
                    xn = __builtin_fmaf(x[t].x, x[t].x, __builtin_fmaf(x[t].y, x[t].y, __builtin_fmaf(x[t].z, x[t].z, __builtin_fmaf(x[t].w, x[t].w, xn))));
                xn += __shfl_xor(xn, 16);
                xn += __shfl_xor(xn, 32);
                if (fill > kBBuf - kBQ * 16) flush();
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    if (live[g]) candidates(acc[g], xn, g, blk);
            };
            // two row buffers in turn: the next block's loads are issued on
            // every step (past the last block they read it again) before the
            // current block is used, so its wait leaves them in flight
            float4 xa[KT], xb[KT];
            load_rows(b, xa);
            for (;;) {
                const int32_t nb = S.next(b);
                load_rows(nb <= bend ? nb : b, xb);
                process(b, xa);
                if (nb > bend) break;
                b = S.next(nb);
                load_rows(b <= bend ? b : nb, xa);
                process(nb, xb);
                if (b > bend) break;
            }
        } else {
            // NB blocks against halves G0 .. G1 - 1 of the tile's queries
            auto blocks = [&](const int32_t (&blk)[NB], auto g0, auto g1) {
                constexpr int G0 = decltype(g0)::value, G1 = decltype(g1)::value;
                const float4* xr[NB];
                floatx4_t acc[2][NB];
                float xn[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int32_t at = (blk[i] <= bend ? blk[i] : bend) * 16 + ii;
                    const int64_t row = at < n32 ? at : n32 - 1;
                    xr[i] = X4 + row * dp4 + kk;
                    acc[0][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
                    acc[1][i] = acc[0][i];
                    xn[i] = 0.f;
                }
                float4 qc[2][2], xc[2][NB];
                auto load = [&](int t, int s) {
                    const int tt = t < dp / 16 ? t : dp / 16 - 1;
#pragma unroll
                    for (int g = G0; g < G1; ++g) qc[s][g] = qrow4[g][4 * tt];
#pragma unroll
                    for (int i = 0; i < NB; ++i) xc[s][i] = xr[i][4 * tt];
                };
                auto mul = [&](int s) {
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        const float4 v = xc[s][i];
                        xn[i] = __builtin_fmaf(v.x, v.x, __builtin_fmaf(v.y, v.y, __builtin_fmaf(v.z, v.z, __builtin_fmaf(v.w, v.w, xn[i]))));
                    }
#pragma unroll
                    for (int w = 0; w < 4; ++w)
#pragma unroll
                        for (int i = 0; i < NB; ++i)
#pragma unroll
                            for (int g = G0; g < G1; ++g) {
                                const float4 a = qc[s][g], v = xc[s][i];
                                const float aw = w == 0 ? a.x : (w == 1 ? a.y : (w == 2 ? a.z : a.w));
                                const float xw = w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
                                acc[g][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(aw, xw, acc[g][i], 0, 0, 0);
                            }
                };
                // dp is a multiple of 32: an even number of steps of 16
                load(0, 0);
                for (int t = 0; t < dp / 16; t += 2) {
                    load(t + 1, 1);
                    mul(0);
                    load(t + 2, 0);
                    mul(1);
                }
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    float s = xn[i];
                    s += __shfl_xor(s, 16);
                    s += __shfl_xor(s, 32);
                    if (blk[i] > bend) continue;   // uniform
                    if (fill > kBBuf - kBQ * 16) flush();
#pragma unroll
                    for (int g = G0; g < G1; ++g) candidates(acc[g][i], s, g, blk[i]);
                }
            };
            // the halves that hold queries whose intervals meet the blocks (40k
            // x 960, one query: 576 us with both multiplied, 523 so; 40 queries:
            // 826, 677)
            const std::integral_constant<int, 0> h0{};
            const std::integral_constant<int, 1> h1{};
            const std::integral_constant<int, 2> h2{};
            while (b <= bend) {
                int32_t blk[NB], last = b;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    blk[i] = b;
                    if (b <= bend) last = b;
                    b = S.next(b);
                }
                const bool live0 = uniform(blk[0] * 16 <= ghi[0] && last * 16 + 15 >= glo[0]);
                const bool live1 = uniform(blk[0] * 16 <= ghi[1] && last * 16 + 15 >= glo[1]);
                if (live0 && live1) blocks(blk, h0, h2);
                else if (live0) blocks(blk, h0, h1);
                else if (live1) blocks(blk, h1, h2);
            }
        }
        flush();   // before the slots' queries change
    }
}

// ------------------------------------------------------------------ thresholds

// One wavefront per query: the threshold after a sampling pass, the value of
// the list's j-th smallest entry (or a little above: between j and 5j/4
// entries at or below it), and the list without the entries above it.  Lists
// with fewer than j entries keep their threshold.
__global__ __launch_bounds__(64) void bf_select_kernel(BFParams P, int j) {
    extern __shared__ __attribute__((aligned(16))) uint32_t s_v[];   // [cap]
    const int64_t q = blockIdx.x;
    const int lane = lane_id();
    const int f = uniform(P.cnt[q]);
    if (f < j) return;
    if (f > P.cap) {   // overflowed: nothing more is listed, the exact pass takes the query
        if (lane == 0) P.thr[q] = -__int_as_float(0x7f800000);
        return;
    }
    uint64_t* L = P.list + q * P.cap;
    uint32_t vmin = 0xFFFFFFFFu, vmax = 0u;
    for (int i = lane; i < f; i += 64) {
        const uint32_t v = (uint32_t)(L[i] >> 32);
        s_v[i] = v;
        vmin = v < vmin ? v : vmin;
        vmax = v > vmax ? v : vmax;
    }
    wave_sync();
    wave_minmax_u32(vmin, vmax);
    uint32_t lo = vmin, hi = vmax;
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        int c = 0;
        for (int i0 = 0; i0 < f; i0 += 64) {
            const int i = i0 + lane;
            c += __popcll(ballot(i < f && s_v[i < f ? i : 0] <= mid));
        }
        if (c < j) {
            lo = mid + 1;
        } else {
            hi = mid;
            if (c <= j + j / 4) break;
        }
    }
    const uint32_t x = hi;
    int kept = 0;
    for (int i0 = 0; i0 < f; i0 += 64) {
        const int i = i0 + lane;
        const uint64_t key = i < f ? L[i] : ~0ull;
        const bool keep = i < f && (uint32_t)(key >> 32) <= x;
        const uint64_t m = ballot(keep);
        if (keep) L[kept + mbcnt(m)] = key;   // at or before the entries read
        kept += __popcll(m);
    }
    if (lane == 0) {
        P.cnt[q] = kept;
        P.thr[q] = ord_value(x + 1u);   // the next value above x (x < +inf)
    }
}

// ------------------------------------------------------------------ results

// One wavefront per query.  MK: list entries re-ranked (2k rounded up); C, LP
// as for the search.
template <int C, int LP, int MK>
__global__ __launch_bounds__(64) void bf_merge_kernel(BFParams P) {
    __shared__ uint64_t s_list[2 * MK];
    __shared__ int32_t s_st[2];
    __shared__ uint64_t s_pk[64 * LP];
    __shared__ uint32_t s_pf[64 * LP];
    const int64_t q = blockIdx.x;
    const int lane = lane_id();
    const DevIndex& ix = P.ix;
    const int64_t l = uniform(P.lr[2 * q]), r = uniform(P.lr[2 * q + 1]);
    if (l > r) return;   // padded by bf_plan_kernel
    if (P.again && uniform(P.redo[q]) == 0) return;   // its result stands
    const float* qrow = P.Q + q * ix.d;
    float4 qv[C > 0 ? C : 1];
    if constexpr (C > 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int b = chunk_dim<float>(lane & 7, c);
            qv[c].x = b < ix.d ? qrow[b] : 0.f;
            qv[c].y = b + 1 < ix.d ? qrow[b + 1] : 0.f;
            qv[c].z = b + 2 < ix.d ? qrow[b + 2] : 0.f;
            qv[c].w = b + 3 < ix.d ? qrow[b + 3] : 0.f;
        }
    }
    const int f0 = uniform(P.cnt[q]);
    bool ok = f0 <= P.cap;
    if (!ok && !P.again) {
        // overflowed: to be scanned again, unless most of the list is tied at
        // its largest value, which another sample would not change
        const uint64_t* L = P.list + q * P.cap;
        uint32_t vmin = 0xFFFFFFFFu, vmax = 0u;
        for (int i = lane; i < P.cap; i += 64) {
            const uint32_t v = (uint32_t)(L[i] >> 32);
            vmin = v < vmin ? v : vmin;
            vmax = v > vmax ? v : vmax;
        }
        wave_minmax_u32(vmin, vmax);
        int tied = 0;
        for (int i = lane; i < P.cap; i += 64) tied += (uint32_t)(L[i] >> 32) == vmax ? 1 : 0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) tied += __shfl_xor(tied, o);
        if (2 * tied < P.cap) {
            if (lane == 0) {
                P.redo[q] = 1;
                atomicAdd(&P.meta->nredo, 1u);
            }
            return;
        }
    }
    Pool<LP> pool;
#pragma unroll
    for (int s = 0; s < LP; ++s) { pool.key[s] = kEmpty; pool.flag[s] = 0u; }
    pool.np = 0;
    if (ok) {
        const BufList Lst{s_list, s_st};
        buf_init(Lst);
        const uint64_t* L = P.list + q * P.cap;
        for (int i0 = 0; i0 < f0; i0 += 64) {
            const int i = i0 + lane;
            const uint64_t key = L[i < f0 ? i : f0 - 1];
            const float v = ord_value((uint32_t)(key >> 32));
            const uint64_t gm = ballot(i < f0 && v < __int_as_float(Lst.st[1]));
            if (gm) buf_offer<MK>(Lst, gm, v, (int32_t)(uint32_t)key);
        }
        buf_cut<MK>(Lst);
        // every row not re-ranked is at or above this
        const float texcl = fminf(P.thr[q], __int_as_float(Lst.st[1]));
        const int f = uniform(Lst.st[0]);
        for (int j0 = 0; j0 < f; j0 += 64) {
            const int nb = f - j0 < 64 ? f - j0 : 64;
            const int32_t id = (int32_t)(uint32_t)Lst.key[lane < nb ? j0 + lane : j0];
            float dd;
            if constexpr (C > 0) dd = eval_pipelined<C, float>(ix.X, ix.dp, qv, nb, id);
            else dd = eval_large(ix.X, ix.dp, qrow, ix.d, nb, id);
            uint64_t key = lane < nb ? make_key(dd, id) : kEmpty;
            if (LP == 1 && f <= 64) {
                // one key per lane: a bitonic sort over the wavefront
#pragma unroll
                for (int kb = 2; kb <= 64; kb <<= 1) {
#pragma unroll
                    for (int jb = kb >> 1; jb > 0; jb >>= 1) {
                        const uint64_t other = (uint64_t)__shfl_xor((long long)key, jb);
                        const bool up = (lane & kb) == 0;
                        const bool low = (lane & jb) == 0;
                        key = (low == up) ? (other < key ? other : key) : (other > key ? other : key);
                    }
                }
                pool.key[0] = lane < P.k ? key : kEmpty;
                pool.np = f < P.k ? f : P.k;
            } else {
                merge<LP>(pool, key, nb, P.k, s_pk, s_pf);
            }
        }
        double qn = 0.0;
        for (int c = lane; c < ix.d; c += 64) qn += (double)qrow[c] * (double)qrow[c];
        qn = sum64(qn);
        const double norms = qn + (double)P.maxnorm;
        const double eps = 2.0 * (2.0 * ix.d + 4.0) * 5.9604644775390625e-08 * norms;
        ok = norms < 1e37;   // the approximation cannot have overflowed
        if (!(texcl == __int_as_float(0x7f800000))) {   // rows were left out
            uint64_t kk = 0;
#pragma unroll
            for (int s = 0; s < LP; ++s)
                if (s == ((P.k - 1) >> 6)) kk = readlane64(pool.key[s], (P.k - 1) & 63);
            const double kth = (double)__uint_as_float((uint32_t)(kk >> 32));
            ok = ok && pool.np == P.k && (double)texcl - eps > kth;
        }
    }
#pragma unroll
    for (int s = 0; s < LP; ++s) {
        const int p = s * 64 + lane;
        if (p < P.k) {
            const bool have = p < pool.np;
            P.ids[q * P.k + p] = have ? ix.perm[(uint32_t)pool.key[s]] : -1;
            P.dists[q * P.k + p] = have ? __uint_as_float((uint32_t)(pool.key[s] >> 32)) : __int_as_float(0x7f800000);
        }
    }
    if (lane == 0) {
        if (P.cert) P.cert[q] = ok ? 1 : 0;
        if (!ok) {
            const uint32_t at = atomicAdd(&P.meta->nfail, 1u);
            P.fail[3 * (int64_t)at] = (int32_t)q;
            P.fail[3 * (int64_t)at + 1] = (int32_t)l;
            P.fail[3 * (int64_t)at + 2] = (int32_t)r;
        }
    }
}

template <int C>
void (*pick_bf_merge_c(int k))(BFParams) {
    if (k <= 32) return bf_merge_kernel<C, 1, 64>;
    if (k <= 64) return bf_merge_kernel<C, 1, 128>;
    if (k <= 128) return bf_merge_kernel<C, 2, 256>;
    return bf_merge_kernel<C, 4, 512>;
}

void (*pick_bf_merge(int dp, int k))(BFParams) {
    switch (dp) {
        case 32: return pick_bf_merge_c<1>(k);
        case 64: return pick_bf_merge_c<2>(k);
        case 96: return pick_bf_merge_c<3>(k);
        case 128: return pick_bf_merge_c<4>(k);
        default: return pick_bf_merge_c<0>(k);
    }
}

template <bool DRAWN>
void (*pick_bf_scan(int dp))(BFParams, int, bool) {
    switch (dp) {
        case 32: return bf_scan_kernel<2, DRAWN>;
        case 64: return bf_scan_kernel<4, DRAWN>;
        case 96: return bf_scan_kernel<6, DRAWN>;
        case 128: return bf_scan_kernel<8, DRAWN>;
        default: return bf_scan_kernel<0, DRAWN>;
    }
}

// entries re-ranked per query, as bf_merge_kernel's instances, and per list
int bf_kept(int k) { return k <= 32 ? 64 : (k <= 64 ? 128 : (k <= 128 ? 256 : 512)); }
int bf_cap(int k) { return std::max(2048, 16 * bf_kept(k)); }

// One batch of at most kBBatch queries.
int bruteforce_batch(const frog_index* ix, const float* Q, int64_t nq, const double* lo, const double* hi, int k,
                     int32_t* ids, float* dists, int32_t* cert, hipStream_t stream) {
    const DevIndex dix{ix->dX, ix->dXh, ix->dENC, ix->dattr, ix->dperm, ix->n, ix->d, ix->dp, ix->H, ix->m,
                       ix->storage};
    const int mk = bf_kept(k);
    BFParams P{};
    P.ix = dix;
    P.Q = Q;
    P.lo = lo;
    P.hi = hi;
    P.nq = nq;
    P.k = k;
    P.maxnorm = ix->maxnorm;
    P.cap = bf_cap(k);
    // the first pass lists every row it scans: at most 3/4 of the cap
    P.npass = 1;
    while (P.npass < kBPasses && (dix.n >> (4 * (P.npass - 1))) > P.cap * 3 / 4) ++P.npass;
    P.tmax = (nq + kBQ - 1) / kBQ + kBBands;
    // an interval of R rows meets at most R / chunk + 2 chunks, and the tiles'
    // rows make at most kBItems chunks in all
    P.imax = kBItems + 2 * P.tmax;
    auto align = [](size_t x) { return (x + 255) / 256 * 256; };
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += align(bytes); return o; };
    const size_t o_meta = take(sizeof(BMeta));
    const size_t o_hist = take((size_t)kBBands * kBBins * 4);
    const size_t o_lr = take((size_t)nq * 8);
    const size_t o_place = take((size_t)nq * 4);
    const size_t o_bucket = take((size_t)nq * 4);
    const size_t o_order = take((size_t)P.tmax * kBQ * 4);
    const size_t o_tiles = take((size_t)P.tmax * sizeof(BTile));
    size_t o_items[kBPasses];
    for (int p = 0; p < P.npass; ++p) o_items[p] = take((size_t)P.imax * sizeof(uint2));
    const size_t o_qp = take((size_t)nq * dix.dp * 4);
    const size_t o_list = take((size_t)nq * P.cap * 8);
    const size_t o_cnt = take((size_t)nq * 4);
    const size_t o_thr = take((size_t)nq * 4);
    const size_t o_redo = take((size_t)nq * 4);
    const size_t o_fail = take((size_t)nq * 12);
    void* ws = nullptr;
    hipError_t e = ws_alloc(&ws, off, stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();   // not to be reported by the next launch
        return fail(FROG_ENOMEM, "bruteforce workspace: %s", hipGetErrorString(e));
    }
    char* base = reinterpret_cast<char*>(ws);
    P.meta = reinterpret_cast<BMeta*>(base + o_meta);
    P.hist = reinterpret_cast<uint32_t*>(base + o_hist);
    P.lr = reinterpret_cast<int32_t*>(base + o_lr);
    P.place = reinterpret_cast<uint32_t*>(base + o_place);
    P.bucket = reinterpret_cast<uint32_t*>(base + o_bucket);
    P.order = reinterpret_cast<int32_t*>(base + o_order);
    P.tiles = reinterpret_cast<BTile*>(base + o_tiles);
    for (int p = 0; p < P.npass; ++p) P.items[p] = reinterpret_cast<uint2*>(base + o_items[p]);
    P.Qp = reinterpret_cast<float*>(base + o_qp);
    P.list = reinterpret_cast<uint64_t*>(base + o_list);
    P.cnt = reinterpret_cast<int32_t*>(base + o_cnt);
    P.thr = reinterpret_cast<float*>(base + o_thr);
    P.redo = reinterpret_cast<int32_t*>(base + o_redo);
    P.fail = reinterpret_cast<int32_t*>(base + o_fail);
    P.ids = ids;
    P.dists = dists;
    P.cert = cert;
    const int64_t ninit = std::max<int64_t>(std::max<int64_t>(kBBands * kBBins, P.tmax * kBQ), nq);
    const unsigned qwaves = (unsigned)((nq + kWavesPerBlock - 1) / kWavesPerBlock);
    // {uncertified, to be scanned again}, read back after each time
    static_assert(offsetof(BMeta, nredo) == offsetof(BMeta, nfail) + 4, "read together");
    uint32_t left[2] = {0, 0};
    hipError_t es = hipSuccess;
    for (int time = 0; time < 2; ++time) {
        P.again = time > 0;
        hipLaunchKernelGGL(bf_init_kernel, dim3((unsigned)((ninit + 255) / 256)), dim3(256), 0, stream, P);
        hipLaunchKernelGGL(bf_plan_kernel, dim3(qwaves), dim3(kBlock), 0, stream, P);
        hipLaunchKernelGGL(bf_bins_kernel, dim3(1), dim3(1024), 0, stream, P);
        hipLaunchKernelGGL(bf_order_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, stream, P);
        hipLaunchKernelGGL(bf_tile_kernel, dim3((unsigned)((P.tmax + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(kBlock), 0,
                           stream, P);
        hipLaunchKernelGGL(bf_items_kernel, dim3((unsigned)P.npass), dim3(1024), 0, stream, P);
        auto scan = P.again ? pick_bf_scan<true>(dix.dp) : pick_bf_scan<false>(dix.dp);
        const int blocks = max_blocks((const void*)scan, 0, 64);
        // The thresholds' places in the sampled lists: about 16 j of the rows the
        // next pass scans lie below the j-th smallest, with a spread of
        // 1/sqrt(j); the last list is then about 4 K' long.
        for (int p = P.npass - 1; p >= 0; --p) {
            hipLaunchKernelGGL(scan, dim3(blocks), dim3(64), 0, stream, P, p, p < P.npass - 1);
            if (p > 0)
                hipLaunchKernelGGL(bf_select_kernel, dim3((unsigned)nq), dim3(64), (size_t)P.cap * 4, stream, P,
                                   p > 1 ? mk / 8 : mk / 4);
        }
        hipLaunchKernelGGL(pick_bf_merge(dix.dp, k), dim3((unsigned)nq), dim3(64), 0, stream, P);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(left, &P.meta->nfail, 8, hipMemcpyDeviceToHost, stream);
        es = hipStreamSynchronize(stream);
        if (e != hipSuccess || es != hipSuccess || left[1] == 0) break;
    }
    const uint32_t nf = left[0];
    std::vector<int32_t> ff, fq, flr;
    if (e == hipSuccess && es == hipSuccess && nf > 0) {
        ff.resize((size_t)nf * 3);
        e = hipMemcpyAsync(ff.data(), P.fail, (size_t)nf * 12, hipMemcpyDeviceToHost, stream);
        es = hipStreamSynchronize(stream);
    }
    (void)ws_free(ws, stream);
    if (e != hipSuccess || es != hipSuccess)
        return fail(FROG_EHIP, "bruteforce launch: %s", hipGetErrorString(e != hipSuccess ? e : es));
    if (nf == 0) return FROG_OK;
    // the rest: every rank of the interval, exactly
    for (uint32_t i = 0; i < nf; ++i) {
        fq.push_back(ff[3 * (size_t)i]);
        flr.push_back(ff[3 * (size_t)i + 1]);
        flr.push_back(ff[3 * (size_t)i + 2]);
    }
    return launch_exact_ranges(dix, Q, fq.data(), flr.data(), (int64_t)nf, k, ids, dists, cert, stream);
}

}  // namespace

int launch_bruteforce(const frog_index* ix, const float* Q, int64_t nq, const double* lo,
                      const double* hi, int k, int32_t* ids, float* dists, int32_t* cert, void* stream_v) {
    // equal batches whose lists (16 KB a query at k <= 64, 32 at k <= 128, 64
    // above) fit kBBytes, and smaller ones on a device that has no such room
    // left (16,384 queries of 300k x 64, k = 256: 1.07 GB in one batch and
    // 3.2 ms, 4.7 in four; k <= 64 as before)
    const int64_t most = std::min(kBBatch, kBBytes / (8 * (int64_t)bf_cap(k)));
    const int64_t parts = (nq + most - 1) / most;
    int64_t batch = parts > 1 ? ((nq + parts - 1) / parts + kBQ - 1) / kBQ * kBQ : nq;
    for (int64_t q0 = 0; q0 < nq;) {
        const int64_t c = std::min(batch, nq - q0);
        const int rc = bruteforce_batch(ix, Q + q0 * ix->d, c, lo + q0, hi + q0, k, ids + q0 * k, dists + q0 * k,
                                        cert ? cert + q0 : nullptr, (hipStream_t)stream_v);
        if (rc == FROG_ENOMEM && c > 256) {
            batch = (c / 2 + kBQ - 1) / kBQ * kBQ;
            continue;
        }
        if (rc != FROG_OK) return rc;
        q0 += c;
    }
    return FROG_OK;
}

}  // namespace frog
