// cs_bin.hip -- binning of one species into collision cells (the grouping of
// particles by cell that precedes pairing, Sec. 3.1): a stable sort of the
// particles by cell id that writes the species' arrays in cell order, and
// the CSR offsets of the cells.
//
// The sort is a least-significant-digit radix sort of the cell ids with
// the fewest digits of at most 9 bits, as even as they come out, that moves
// the particles' values along with their keys, so that every access to the
// values is a run of consecutive elements (never a gather from random
// positions).  Every pass is stable, so the result is the stable sort;
// nothing depends on the timing of atomics, so the output is the same on
// every run.  Ids outside [0, n_cells) get the key n_cells, which sorts them
// after every valid particle.
//
//   up to kBinOne particles: k_bin_one, every pass by one workgroup in LDS
//   more: per pass (tiles by the particle count and the digit, see BinShape):
//   k_bin_hist    per tile, the digit counts (LDS atomics)
//   k_bin_scan    (more than kBinRows tiles) one workgroup per digit: exclusive prefix over the tiles of
//                 that digit's counts, and the digit's total
//   k_bin_scatter per tile: digit bases from the totals and the tile
//                 prefixes; each wave takes its consecutive keys in chunks
//                 of 64, in order, and ranks each key among the chunk's keys
//                 of the same digit by one ballot per digit bit; the tile,
//                 ordered by digit in LDS, is then written out run by run
//                 with the particles' four values
//   k_bin_offsets off[c] = first sorted position with key >= c, c = 0 ..
//                 n_cells; off[n_cells] counts the valid particles
// The passes alternate between a scratch copy of the values and the output
// arrays so that the last one writes the output.
#include <hip/hip_runtime.h>

#include "cs_block.h"
#include "cs_internal.h"

namespace cs {

constexpr int kBinThreads = 256;                          // scans and offsets
constexpr int kBinDigitBits = 9;  // at most
constexpr int kBinDigits = 1 << kBinDigitBits;

// Tile shape: WAVES waves of CHUNKS 64-key chunks.  The larger the tile, the
// longer each digit's run of consecutive output positions (8-bit digits: ~16
// keys per digit and tile of 4096, 64 bytes per FP32 value array), and the fewer
// workgroups a compute unit holds to read, rank and write side by side.
template <typename T, int WAVES, int CHUNKS, int LOTS>
struct BinShape {
    static constexpr int kThreads = 64 * WAVES;
    static constexpr int kWaveKeys = 64 * CHUNKS;
    static constexpr int kTile = WAVES * kWaveKeys;
    struct alignas(LOTS * sizeof(T)) Lot {  // what of a particle's values passes through LDS at once
        T v[LOTS];
    };
};

template <typename T>
struct BinArrays {
    const T *x, *y, *z, *w;
};
template <typename T>
struct BinOut {
    T *x, *y, *z, *w;
};

// Pass key of particle i: its cell id, or n_cells for an id outside
// [0, n_cells); read from the cell ids on the first pass.
__device__ __forceinline__ uint32_t bin_raw(const uint32_t* keys, const int32_t* cell, int64_t i) {
    return keys ? keys[i] : (uint32_t)cell[i];
}
__device__ __forceinline__ uint32_t bin_clamp(uint32_t c, int64_t n_cells) {
    return (int64_t)c < n_cells ? c : (uint32_t)n_cells;  // (negative ids are beyond every n_cells)
}
__device__ __forceinline__ uint32_t bin_key(const uint32_t* keys, const int32_t* cell, int64_t n_cells, int64_t i) {
    const uint32_t c = bin_raw(keys, cell, i);
    return keys ? c : bin_clamp(c, n_cells);
}

// Digit of pass ps when `bits` key bits are shared out over `passes`: even, the
// last ones (wide_first: the first ones) a bit wider where they do not come out
// even.
struct BinDigit {
    int shift, bits;
};
__host__ __device__ __forceinline__ BinDigit bin_digit(int bits, int passes, int ps, bool wide_first) {
    const int each = bits / passes, wide = bits % passes, first = wide_first ? 0 : passes - wide;
    const int before = ps < first ? 0 : (ps - first < wide ? ps - first : wide);  // wide ones before it
    return {ps * each + before, each + (ps >= first && ps < first + wide ? 1 : 0)};
}

// The lanes of `act` whose digit equals this lane's (a lane of act): per digit
// bit one ballot and one three-operand bit operation per half.
__device__ __forceinline__ uint64_t bin_match(uint64_t act, uint32_t d, int dbits) {
    uint32_t lo = (uint32_t)act, hi = (uint32_t)(act >> 32);
#pragma unroll
    for (int b = 0; b < 9; ++b) {
        if (b < dbits) {
            const uint32_t t = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // the bit, in every place
            const uint64_t m = __builtin_amdgcn_ballot_w64(t != 0);
            lo &= ~((uint32_t)m ^ t);
            hi &= ~((uint32_t)(m >> 32) ^ t);
        }
    }
    return (uint64_t)hi << 32 | lo;
}

// hist[d d_stride + t t_stride] = keys of tile t (TILE keys, THREADS threads)
// whose digit is d
template <int THREADS, int TILE>
__global__ __launch_bounds__(THREADS) void k_bin_hist(const uint32_t* keys, const int32_t* cell, int64_t n,
                                                      int64_t n_cells, int shift, int dbits, int64_t d_stride,
                                                      int64_t t_stride, uint32_t* hist) {
    __shared__ uint32_t s_cnt[kBinDigits];
    const int tid = threadIdx.x;
    const uint32_t mask = (1u << dbits) - 1u;
    const int nd = 1 << dbits;
    for (int d = tid; d < kBinDigits; d += THREADS) s_cnt[d] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * TILE;
#pragma unroll
    for (int j = 0; j < TILE / THREADS; ++j) {
        const int64_t i = t0 + (int64_t)j * THREADS + tid;
        if (i < n) atomicAdd(&s_cnt[(bin_key(keys, cell, n_cells, i) >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int d = tid; d < nd; d += THREADS) hist[d * d_stride + blockIdx.x * t_stride] = s_cnt[d];
}

// Workgroup d: exclusive prefix of hist[d][0 .. n_tiles) in place, the sum to
// totals[d].  The tiles are taken in blocks of 256 x 16, each thread owning
// 16 consecutive entries of a block.
__global__ __launch_bounds__(kBinThreads) void k_bin_scan(uint32_t* hist, int64_t n_tiles, uint32_t* totals) {
    __shared__ int s_scan[kBinThreads / 64 + 1];
    constexpr int kPer = 16;
    uint32_t* h = hist + (int64_t)blockIdx.x * n_tiles;
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < n_tiles; b0 += (int64_t)kBinThreads * kPer) {
        const int64_t i0 = b0 + (int64_t)threadIdx.x * kPer;
        uint32_t v[kPer];
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            v[k] = i0 + k < n_tiles ? h[i0 + k] : 0u;
            const uint32_t c = v[k];
            v[k] = run;
            run += c;
        }
        int block_total;
        const uint32_t ex = carry + (uint32_t)block_exclusive_scan((int)run, s_scan, &block_total);
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (i0 + k < n_tiles) h[i0 + k] = ex + v[k];
        carry += (uint32_t)block_total;
        __syncthreads();  // s_scan reused by the next block
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Stable scatter of tile t: key i goes to base(digit) + (keys of the same
// digit before it in the tile), base = (keys of smaller digits in all tiles)
// + (keys of this digit in earlier tiles); the particle's values go with it.
// The two sums come from k_bin_scan, or (SCAN false, few tiles) from the tiles'
// counts themselves, in rows of digits.
// The tile is first ordered by digit in LDS (keys and tile-local source
// indices) and written out in that order, so that consecutive threads write
// consecutive positions of a digit's run; each value array passes through
// LDS the same way (read in order, written in digit order), so every global
// access is coalesced.
//
// Its phases add up -- reading the tile, ranking, passing the values through
// LDS, writing: without the value stores it is 39.6 us long, with them 43 (2^22
// FP32 particles, 168 MB).  The keys are read first, so that they are ranked
// while the values arrive; a thread keeps its keys' places in registers and puts
// two FP32 values at a time through LDS.  4096-key tiles 43.7 -> 41.2 us by the
// latter, 16384-key tiles 46 -> 44 by the former.
template <typename T, int WAVES, int CHUNKS, int LOTS, bool SCAN>
__global__ __launch_bounds__(64 * WAVES) void k_bin_scatter(const uint32_t* keys_in, const int32_t* cell, int64_t n,
                                                            int64_t n_cells, int shift, int dbits, int64_t n_tiles,
                                                            const uint32_t* hist, const uint32_t* totals,
                                                            BinArrays<T> src, uint32_t* keys_out, BinOut<T> dst) {
    typedef BinShape<T, WAVES, CHUNKS, LOTS> Shape;
    constexpr int kThreads = Shape::kThreads, kTile = Shape::kTile, kWaves = WAVES, kBinWaveKeys = Shape::kWaveKeys;
    typedef typename Shape::Lot Lot;
    constexpr int kLots = LOTS;
    constexpr int kPer = kTile / kThreads;            // outputs per thread
    constexpr int kDigPer = kBinDigits / kThreads > 2 ? kBinDigits / kThreads : 2;  // digits of a thread in the scans
    __shared__ uint32_t s_cnt[kWaves][kBinDigits];    // per wave counts, then running local bases
    __shared__ uint32_t s_toff[kBinDigits];           // tile-local start of each digit's run
    __shared__ uint32_t s_gbase[kBinDigits];          // global start of each digit's run
    __shared__ Lot s_buf[kTile];                      // the tile's keys, then its values lot by lot
    __shared__ int s_scan[kWaves + 1];
    uint32_t* s_key = (uint32_t*)s_buf;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t t = blockIdx.x;
    const int64_t t0 = t * kTile;
    const int64_t rem = n - t0;
    const int len = rem < kTile ? (int)rem : kTile;
    const int wl0 = wave * kBinWaveKeys;  // this wave's first key in the tile
    const uint32_t mask = (1u << dbits) - 1u;
    const int nd = 1 << dbits;
    // thread t < kBinDigits / kDigPer looks after digits kDigPer t onwards in
    // the scans below; the others add nothing to them
    const bool dig = tid < kBinDigits / kDigPer;
    const int d0 = dig ? kDigPer * tid : 0;
    uint32_t key[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int li = wl0 + c * 64 + lane;
        key[c] = li < len ? bin_raw(keys_in, cell, t0 + li) : 0u;
    }
    // of each digit the keys in all tiles and in the tiles before this one
    uint32_t tot[kDigPer], pre[kDigPer];
#pragma unroll
    for (int k = 0; k < kDigPer; ++k) {
        const bool in = dig && d0 + k < nd;
        if constexpr (SCAN) {
            tot[k] = in ? totals[d0 + k] : 0u;
            pre[k] = in ? hist[(int64_t)(d0 + k) * n_tiles + t] : 0u;
        } else {
            tot[k] = pre[k] = 0u;
            if (in) {
                for (int i0 = 0; i0 < (int)n_tiles; i0 += 8) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int i = i0 + r;
                        const uint32_t v = hist[(i < (int)n_tiles ? i : 0) * nd + d0 + k];
                        tot[k] += i < (int)n_tiles ? v : 0u;
                        pre[k] += i < (int)t ? v : 0u;
                    }
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // the tile's four value arrays, read in order (coalesced) into registers;
    // non-temporal, as every value is read once per pass (the stores stay
    // ordinary: a digit's run rarely fills whole lines, and the cache
    // merges the pieces that neighbouring tiles write)
    const T* srcs[4] = {src.x, src.y, src.z, src.w};
    T val[4][CHUNKS];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int li = wl0 + c * 64 + lane;
            val[a][c] = li < len ? __builtin_nontemporal_load(&srcs[a][t0 + li]) : (T)0;
        }
    __builtin_amdgcn_sched_barrier(0);
    for (int i = tid; i < kWaves * kBinDigits; i += kThreads) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        if (!keys_in) key[c] = bin_clamp(key[c], n_cells);
        if (wl0 + c * 64 + lane < len) atomicAdd(&s_cnt[wave][(key[c] >> shift) & mask], 1u);
    }
    // digit base over all tiles: exclusive prefix of the totals
    {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kDigPer; ++k) {
            const uint32_t v = tot[k];
            tot[k] = sum;
            sum += v;
        }
        int unused;
        const uint32_t ex = (uint32_t)block_exclusive_scan((int)sum, s_scan, &unused);
        if (dig) {
#pragma unroll
            for (int k = 0; k < kDigPer; ++k) s_gbase[d0 + k] = ex + tot[k] + pre[k];
        }
    }
    __syncthreads();
    // the tile-local start of each digit's run, then each wave's running
    // base inside it (waves in key order)
    {
        uint32_t tc[kDigPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kDigPer; ++k) {
            tc[k] = 0;
            if (dig) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) tc[k] += s_cnt[w][d0 + k];
            }
            sum += tc[k];
        }
        int unused;
        uint32_t run = (uint32_t)block_exclusive_scan((int)sum, s_scan, &unused);
        if (dig) {
#pragma unroll
            for (int k = 0; k < kDigPer; ++k) {
                s_toff[d0 + k] = run;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const uint32_t v = s_cnt[w][d0 + k];
                    s_cnt[w][d0 + k] = run;
                    run += v;
                }
            }
        }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t lp[CHUNKS];  // tile-local output of each key
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const bool act = wl0 + c * 64 + lane < len;
        const uint32_t d = (key[c] >> shift) & mask;
        const uint64_t eq = bin_match(__ballot(act), d, dbits);
        lp[c] = s_cnt[wave][d] + (uint32_t)__popcll(eq & below);
        if (act) s_key[lp[c]] = key[c];
        // the lowest lane of each digit group advances that digit's base (the
        // reads above precede these writes in the wave's LDS order)
        if (act && (eq & below) == 0) s_cnt[wave][d] += (uint32_t)__popcll(eq);
    }
    __syncthreads();
    // keys, in digit order; each output's global position kept for the values
    uint32_t pos[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int j = tid + q * kThreads;
        pos[q] = 0;
        if (j < len) {
            const uint32_t k = s_key[j];
            const uint32_t d = (k >> shift) & mask;
            pos[q] = s_gbase[d] + ((uint32_t)j - s_toff[d]);
            keys_out[pos[q]] = k;
        }
    }
    T* dsts[4] = {dst.x, dst.y, dst.z, dst.w};
#pragma unroll
    for (int a = 0; a < 4; a += kLots) {
        __syncthreads();  // s_buf free
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            Lot v;
#pragma unroll
            for (int k = 0; k < kLots; ++k) v.v[k] = val[a + k][c];
            if (wl0 + c * 64 + lane < len) s_buf[lp[c]] = v;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int j = tid + q * kThreads;
            if (j < len) {
                const Lot v = s_buf[j];
#pragma unroll
                for (int k = 0; k < kLots; ++k) dsts[a + k][pos[q]] = v.v[k];
            }
        }
    }
}

// Cells up to which 16 lanes each search (2^22 particles, whole call: 16384 cells
// 101 us, 104 with one lane; 65536 cells 113, 112; 262144 cells 169, 149).
constexpr int64_t kBinLanesMax = 1 << 15;

// off[c] = lower bound of c in the sorted keys, c = 0 .. n_cells, by L lanes
// each (L = 1: a binary search; else L + 1 parts per step, one memory round
// trip: 2^22 keys take 6 of them with 16 lanes, 22 with one); the first lane
// of c = n_cells also reports the particles with no valid cell.
template <int L>
__global__ __launch_bounds__(kBinThreads) void k_bin_offsets(const uint32_t* keys, int64_t n, int64_t n_cells,
                                                             int64_t* off, int64_t* n_invalid) {
    const int64_t c = ((int64_t)blockIdx.x * kBinThreads + threadIdx.x) / L;
    if (c > n_cells) return;
    int64_t lo = 0, hi = n;  // first position with key >= c is in [lo, hi]
    if constexpr (L == 1) {
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)keys[mid] < c)
                lo = mid + 1;
            else
                hi = mid;
        }
    } else {
        const int l = lane_id() & (L - 1), g0 = lane_id() & ~(L - 1);
        while (lo < hi) {  // (the same for the lanes of c)
            // probe l at lo + (l + 1) part - 1, the last key of part l
            const int64_t part = (hi - lo + L) / (L + 1);
            const int64_t i = lo + (l + 1) * part - 1;
            const bool less = i < hi && (int64_t)keys[i] < c;
            const int k = __popcll((__ballot(less) >> g0) & ((1ull << L) - 1ull));  // parts wholly below c
            lo += k * part;
            hi = lo + part - 1 < hi && k < L ? lo + part - 1 : hi;
        }
    }
    if ((threadIdx.x & (L - 1)) == 0) {
        off[c] = lo;
        if (c == n_cells && n_invalid) *n_invalid = n - lo;
    }
}

// Up to kBinOne particles: the whole sort by one workgroup, keys and source
// indices in LDS, the values gathered at the end.
constexpr int kBinOneWaves = 16, kBinOneChunks = 4;
constexpr int64_t kBinOne = 64 * kBinOneWaves * kBinOneChunks;  // 4096

template <typename T>
__global__ __launch_bounds__(64 * kBinOneWaves) void k_bin_one(const int32_t* cell, int n, int64_t n_cells, int bits,
                                                               int passes, BinArrays<T> src, uint32_t* keys_out,
                                                               BinOut<T> dst) {
    constexpr int kThreads = 64 * kBinOneWaves;
    __shared__ uint32_t s_cnt[kBinOneWaves][kBinDigits];
    __shared__ uint32_t s_key[kBinOne];
    __shared__ uint16_t s_src[kBinOne];
    __shared__ int s_scan[kBinOneWaves + 1];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int wl0 = wave * 64 * kBinOneChunks;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t key[kBinOneChunks], from[kBinOneChunks];
#pragma unroll
    for (int c = 0; c < kBinOneChunks; ++c) {
        const int i = wl0 + c * 64 + lane;
        key[c] = i < n ? (uint32_t)cell[i] : 0u;
        from[c] = (uint32_t)i;
    }
#pragma unroll
    for (int c = 0; c < kBinOneChunks; ++c) key[c] = bin_clamp(key[c], n_cells);
    const bool dig = tid < kBinDigits;
    for (int ps = 0; ps < passes; ++ps) {
        const BinDigit dg = bin_digit(bits, passes, ps, false);
        const int shift = dg.shift, dbits = dg.bits;
        const uint32_t mask = (1u << dbits) - 1u;
        if (ps > 0) {
#pragma unroll
            for (int c = 0; c < kBinOneChunks; ++c) {
                const int i = wl0 + c * 64 + lane;
                key[c] = s_key[i];
                from[c] = s_src[i];
            }
        }
        for (int i = tid; i < kBinOneWaves * kBinDigits; i += kThreads) (&s_cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kBinOneChunks; ++c)
            if (wl0 + c * 64 + lane < n) atomicAdd(&s_cnt[wave][(key[c] >> shift) & mask], 1u);
        __syncthreads();
        uint32_t sum = 0;
        if (dig) {
#pragma unroll
            for (int w = 0; w < kBinOneWaves; ++w) sum += s_cnt[w][tid];
        }
        int unused;
        uint32_t run = (uint32_t)block_exclusive_scan((int)sum, s_scan, &unused);
        if (dig) {
#pragma unroll
            for (int w = 0; w < kBinOneWaves; ++w) {
                const uint32_t v = s_cnt[w][tid];
                s_cnt[w][tid] = run;
                run += v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kBinOneChunks; ++c) {
            const bool act = wl0 + c * 64 + lane < n;
            const uint32_t d = (key[c] >> shift) & mask;
            const uint64_t eq = bin_match(__ballot(act), d, dbits);
            if (act) {
                const uint32_t lp = s_cnt[wave][d] + (uint32_t)__popcll(eq & below);
                s_key[lp] = key[c];
                s_src[lp] = (uint16_t)from[c];
            }
            if (act && (eq & below) == 0) s_cnt[wave][d] += (uint32_t)__popcll(eq);
        }
        __syncthreads();
    }
    const T* srcs[4] = {src.x, src.y, src.z, src.w};
    T* dsts[4] = {dst.x, dst.y, dst.z, dst.w};
    for (int j = tid; j < n; j += kThreads) {
        keys_out[j] = s_key[j];
        const int i = s_src[j];
        T v[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) v[a] = srcs[a][i];
#pragma unroll
        for (int a = 0; a < 4; ++a) dsts[a][j] = v[a];
    }
}

// Tiles of 4096 keys; of 1024 for fewer particles (more workgroups, and shorter
// ones); of 16384 (8192 FP64) for many and digits of 8 bits or more, whose runs
// are too short otherwise.  FP32, whole call, 16384 cells: 65536 particles 32 us
// with 1024 keys (40 with 4096, 76 with 16384), 500000 44 (49, 85), 2^20 65 (51,
// 88), 2^22 179 (107, 117; 100 with the two mixed); 65536 cells, 2^22 particles:
// 111 with 16384, 147 with 4096, 136 with 8192.
constexpr int64_t kBinSmallMax = 3 << 18;
constexpr int64_t kBinLargeMin = 3 << 20;
constexpr int kBinLargeBits = 8;
template <typename T>
using BinSmall = BinShape<T, 4, 4, 8 / sizeof(T)>;
template <typename T>
using BinMedium = BinShape<T, 8, 8, 8 / sizeof(T)>;
template <typename T>
using BinLarge = BinShape<T, 16, sizeof(T) == 4 ? 16 : 8, 1>;

// Tiles up to which each scatter workgroup adds up the tiles' counts itself
// (20000 particles 24.7 us, 28.5 with a scan; 40000 27.9, 29.3; 65536 32.3, 29.2).
constexpr int64_t kBinRows = 48;

static int64_t bin_tiles(int64_t n) {
    const int64_t tile = n < kBinSmallMax ? BinSmall<float>::kTile : BinMedium<float>::kTile;
    return (n + tile - 1) / tile;
}

// scratch: two key arrays (uint32), one copy of the four value arrays (8 B
// elements, enough for either storage type), digit counts of every tile and
// the digit totals
size_t bin_workspace_bytes(int64_t n) {
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int64_t nn = n > 0 ? n : 1;
    return 2 * al(4 * (size_t)nn) + 4 * al(8 * (size_t)nn) + al(4 * (size_t)kBinDigits * bin_tiles(nn)) +
           al(4 * (size_t)kBinDigits);
}

struct BinRun {
    const int32_t* cell;
    int64_t n, n_cells;
    const void* const* in;
    void* const* out;
    uint32_t* const* keys;
    void* const* tmp;
    uint32_t *hist, *totals;
    int bits, passes;
};

// One pass: keys kin (null: the cell ids) and values src to kout and dst.
template <typename T, int WAVES, int CHUNKS, int LOTS>
static void launch_pass(const BinRun& r, BinShape<T, WAVES, CHUNKS, LOTS>, BinDigit dg, const uint32_t* kin,
                        BinArrays<T> src, uint32_t* kout, BinOut<T> dst, hipStream_t st) {
    typedef BinShape<T, WAVES, CHUNKS, LOTS> Shape;
    constexpr int kThreads = Shape::kThreads, kTile = Shape::kTile;
    const int64_t n_tiles = (r.n + kTile - 1) / kTile;
    const bool rows = n_tiles <= kBinRows;
    k_bin_hist<kThreads, kTile><<<(unsigned)n_tiles, kThreads, 0, st>>>(
        kin, r.cell, r.n, r.n_cells, dg.shift, dg.bits, rows ? 1 : n_tiles, rows ? (int64_t)1 << dg.bits : 1, r.hist);
    if (!rows) k_bin_scan<<<1u << dg.bits, kBinThreads, 0, st>>>(r.hist, n_tiles, r.totals);
    (rows ? k_bin_scatter<T, WAVES, CHUNKS, LOTS, false> : k_bin_scatter<T, WAVES, CHUNKS, LOTS, true>)
        <<<(unsigned)n_tiles, kThreads, 0, st>>>(kin, r.cell, r.n, r.n_cells, dg.shift, dg.bits, n_tiles, r.hist,
                                                 r.totals, src, kout, dst);
}

template <typename T>
static void launch_passes(const BinRun& r, hipStream_t st) {
    const BinArrays<T> in_a = {(const T*)r.in[0], (const T*)r.in[1], (const T*)r.in[2], (const T*)r.in[3]};
    const BinOut<T> out_a = {(T*)r.out[0], (T*)r.out[1], (T*)r.out[2], (T*)r.out[3]};
    const BinOut<T> tmp_a = {(T*)r.tmp[0], (T*)r.tmp[1], (T*)r.tmp[2], (T*)r.tmp[3]};
    // narrow digits first, but for those that stay below the large tile beside
    // others that take it (15 bits as 7 + 8 and 8 + 7: 2^21 particles 67 and 73
    // us, 2^22 106 and 100; 17 bits as 8 + 9 and 9 + 8: 2^22 111 and 117)
    const bool wide_first = r.n >= kBinLargeMin && r.bits / r.passes == kBinLargeBits - 1;
    for (int ps = 0; ps < r.passes; ++ps) {
        const BinDigit dg = bin_digit(r.bits, r.passes, ps, wide_first);
        const uint32_t* kin = ps == 0 ? nullptr : r.keys[(ps - 1) & 1];
        // the last pass writes the output; before it the passes alternate
        // between the scratch copy and the output
        const BinOut<T> dst = ((r.passes - 1 - ps) & 1) == 0 ? out_a : tmp_a;
        const BinOut<T> prev = ((r.passes - ps) & 1) == 0 ? out_a : tmp_a;
        const BinArrays<T> src = ps == 0 ? in_a : BinArrays<T>{prev.x, prev.y, prev.z, prev.w};
        uint32_t* kout = r.keys[ps & 1];
        if (r.n < kBinSmallMax)
            launch_pass<T>(r, BinSmall<T>{}, dg, kin, src, kout, dst, st);
        else if (r.n < kBinLargeMin || dg.bits < kBinLargeBits)
            launch_pass<T>(r, BinMedium<T>{}, dg, kin, src, kout, dst, st);
        else
            launch_pass<T>(r, BinLarge<T>{}, dg, kin, src, kout, dst, st);
    }
}

template <typename T>
static void launch_sort(const BinRun& r, hipStream_t st) {
    if (r.n <= kBinOne) {
        const BinArrays<T> in_a = {(const T*)r.in[0], (const T*)r.in[1], (const T*)r.in[2], (const T*)r.in[3]};
        const BinOut<T> out_a = {(T*)r.out[0], (T*)r.out[1], (T*)r.out[2], (T*)r.out[3]};
        k_bin_one<T><<<1, 64 * kBinOneWaves, 0, st>>>(r.cell, (int)r.n, r.n_cells, r.bits, r.passes, in_a,
                                                      r.keys[(r.passes - 1) & 1], out_a);
        return;
    }
    launch_passes<T>(r, st);
}

hipError_t launch_bin(cs_dtype dtype, const int32_t* cell, int64_t n, int64_t n_cells, const void* const in[4],
                      void* const out[4], int64_t* off, int64_t* n_invalid, void* ws, hipStream_t st) {
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int64_t nn = n > 0 ? n : 1;
    char* p = (char*)ws;
    uint32_t* keys[2];
    keys[0] = (uint32_t*)p;
    p += al(4 * (size_t)nn);
    keys[1] = (uint32_t*)p;
    p += al(4 * (size_t)nn);
    void* tmp[4];
    for (int a = 0; a < 4; ++a) {
        tmp[a] = p;
        p += al(8 * (size_t)nn);
    }
    uint32_t* hist = (uint32_t*)p;
    p += al(4 * (size_t)kBinDigits * bin_tiles(nn));
    uint32_t* totals = (uint32_t*)p;

    // the largest key is n_cells (the mark of an invalid id); at least one
    // pass, which also writes the keys the offsets are read from
    int bits = 1;
    while (bits < 32 && ((uint64_t)n_cells >> bits) != 0) ++bits;
    const int passes = (bits + kBinDigitBits - 1) / kBinDigitBits;
    const BinRun run = {cell, n, n_cells, in, out, keys, tmp, hist, totals, bits, passes};
    if (n > 0) {
        if (dtype == CS_F32)
            launch_sort<float>(run, st);
        else
            launch_sort<double>(run, st);
    }
    const uint32_t* sorted = keys[(passes - 1) & 1];
    if (n_cells < kBinLanesMax) {
        const unsigned blocks = (unsigned)(((n_cells + 1) * 16 + kBinThreads - 1) / kBinThreads);
        k_bin_offsets<16><<<blocks, kBinThreads, 0, st>>>(sorted, n, n_cells, off, n_invalid);
    } else {
        const unsigned blocks = (unsigned)((n_cells + 1 + kBinThreads - 1) / kBinThreads);
        k_bin_offsets<1><<<blocks, kBinThreads, 0, st>>>(sorted, n, n_cells, off, n_invalid);
    }
    return hipGetLastError();
}

}  // namespace cs
