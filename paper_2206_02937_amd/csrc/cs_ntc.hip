// cs_ntc.hip -- no-time-counter candidate selection (the NTC method of Bird
// that Sec. 3.1 names to shorten each cell's pair list) with the probability
// and bound of Sec. 3.2.
//
// Per cell c with N_e electrons, N_g photons and W the largest valid weight
// among them: P_max = 2 dt n W bounds the pair probability
// P = dt n max(w_e, w_g) s(x) flux (s <= 1, flux <= 2); the cell draws
// N_e N_g P_max candidates rounded stochastically, each an electron and a
// photon picked uniformly with replacement and accepted with probability
// P / P_max.  The candidates of a cell are taken in order, each on the
// momenta the earlier collisions of its cell left (Bird's sequential scheme).
//
// Data-parallel form.  A candidate's outcome depends only on its own two
// particles, so candidates that share no particle commute, and any order
// in which each candidate follows every earlier candidate of its cell that
// shares a particle with it gives the sequential result.  The step:
//   k_ntc_count    64 or 16 lanes per cell: W, P_max, the count
//   k_ntc_scan     the candidates before each few cells and the total, which
//                  stays on the device, which cells are large ones and the
//                  list of them (see kNtcLow), and whether the step proceeds (a step
//                  with more candidates than the capacity fixed before it, the
//                  context's grown one or a graph's, changes nothing and flags
//                  its stats record)
//   k_ntc_cells    the other cells, a few whole ones per wave: picks, then
//                  rounds of ready candidates (evaluation, and the accepted
//                  ones' scattering, on full waves), all state in LDS, until
//                  none is left
//   the large cells (an eager step that has no such cell, after one that had
//   none, queues none of these; in a graph they find an empty list):
//   k_ntc_pick     a workgroup per cell: its candidates' electrons, photons and
//                  acceptance uniforms; every candidate registers for round 0
//                  in the particles' "first toucher" words (atomicMax of
//                  (round tag << 32 | ~candidate): each word ends up holding
//                  the earliest candidate that touches the particle)
//   k_ntc_eval     round 0, one lane per candidate, one workgroup per
//                  segment of 1024 candidates (so the FP64 evaluation runs
//                  on full waves): the candidates that are the earliest
//                  registered toucher of both their particles are evaluated
//                  (probability, accept); the accepted ones are compacted
//                  into the segment's collide list, the others register for
//                  round 1 and are compacted into its round-1 list
//   k_ntc_collide_list  round 0's accepted candidates, one per lane:
//                  scattering and write-back
//   k_ntc_round t  rounds 1 and 2 over the segments' lists: ready
//                  candidates are evaluated and, when accepted, collide in
//                  place (few are left); the others register for round 2 in
//                  the other word set (two sets alternate, so a round never
//                  reads a word that the same round writes) and go to the
//                  segment's round-2 list or, after round 2, their cell to
//                  the list of cells with candidates left
//   k_ntc_serial   one wave per such cell: the remaining candidates in order,
//                  a window at a time, in rounds as in k_ntc_cells
//   k_ntc_reduce   fixed-order partial sums
//   k_ntc_final    fixed-order sums of both paths into cs_stats
// Compaction stays inside a workgroup (a prefix over its waves' ballots), and
// waves past a segment's list length return at once, so the waves that work
// are nearly full.  (The lists of cells are in no particular order; nothing
// that they lead to depends on it.)
// Tags grow by one per round and never repeat (an epoch kept on the device
// beside the touch words and advanced by the last kernel of each step), so
// the touch words are cleared only when the epoch would wrap.  No kernel
// depends on a value read back by the host, so a step can be captured in a
// HIP graph; the step index then comes from a device word that each replay
// advances.
//
// Random numbers: Philox4x32-10 as elsewhere; the count from
// (cell, kNtcCount), candidate l of cell c from index (c << 32) | l with
// kNtcPick (electron (r0 N_e) >> 32, photon (r1 N_g) >> 32, acceptance
// uniform from r2, r3), kNtcScatter (u_mu, u_phi) and kNtcWeight.
#include <hip/hip_runtime.h>

#include "cs_block.h"
#include "cs_device.h"
#include "cs_internal.h"
#include "cs_pair.h"

namespace cs {

constexpr int kNtcThreads = 256;
constexpr int kNtcRounds = 3;  // round 0 (k_ntc_eval), rounds 1 and 2 (k_ntc_round)
constexpr int kNtcScanPer = 4;                            // cells per thread in the scan
constexpr int kNtcScanBlock = kNtcThreads * kNtcScanPer;  // cells per scan workgroup
constexpr int kNtcPiece = 16;                             // cells per piece: 64 pieces per scan workgroup
static_assert(kNtcScanBlock == 64 * kNtcPiece, "a wave reads a scan workgroup's pieces at once");

// Which cells are resolved by one wave each (k_ntc_cells), which by the kernels
// of the large cells.  A wave takes a cell's candidates 64 at a time in turn, those
// kernels take all at once over the chip, in seven launches more.  Up to kNtcLow
// candidates a wave is the quicker, beyond kNtcMidMax it has no room.  The cells
// between go to waves if there are kNtcMidMin of them, which keep the chip busy
// (whole step, us, by waves / by the launches, cells x candidates: 455 x 255 115
// / 99, 699 x 167 86 / 100, 1823 x 255 163 / 190), or if none has more than
// kNtcMidHigh and the launches are not needed for others either (16 x 111 55 /
// 68, but 2 x 167 71 / 52; 6956 cells of a few candidates and denser ones up to 330
// 185 / 119), and there are not fewer cells than kNtcFew (4 x 111 64 / 52 in a
// graph).  Where the launches are needed and all cells together are fewer than
// kNtcMidMin, they take every cell (100 x 35 and 4 denser ones: 107 -> 92).  By the
// candidates alone, so that an eager step and a graph resolve a cell the same way.
constexpr int kNtcLow = 64, kNtcMidHigh = 128, kNtcMidMax = 256;
constexpr int kNtcMidMin = 640, kNtcFew = 8;
constexpr int kNtcRedPer = 2;                               // candidates per thread in the reduction
constexpr int64_t kNtcMaxCand = 2147483647;                 // candidates per step: below 2^31 - 1

// Control words of a step: the candidate total and flags.  Zero at the
// start of every step: zeroed when allocated and by k_ntc_final at the end
// of the previous step (they sit at the start of the per-cell scratch,
// whatever the cell count).
struct NtcCtl {
    long long total;    // candidates of the step
    long long total_l;  // those in the large cells
    int32_t layout_bad;
    int32_t too_many;   // 2^31 - 1 or more candidates
    int32_t overflow;   // more candidates than the launches were sized for
    int32_t go;         // none of the above: the step proceeds
    uint32_t n_large;   // large cells (all cells where local is 0)
    uint32_t n_over;    // cells of more than kNtcMidMax candidates
    uint32_t n_mid;     // cells of more than kNtcLow, up to kNtcMidMax
    uint32_t n_high;    // those of them of more than kNtcMidHigh
    uint32_t n_pend;    // cells left to k_ntc_serial
    uint32_t done;      // workgroups of k_ntc_scan that have finished
    int32_t local;      // candidates of a cell up to which it is not a large one
    uint32_t pad;
};
// Candidates per segment: the evaluation kernel takes one segment per
// workgroup and compacts the segment's accepted candidates and the ones left
// for round 1 into the segment's part of two lists (no global counters).
constexpr int kNtcSeg = 1024;
constexpr int kNtcSub = kNtcSeg / kNtcThreads;  // collide and round workgroups per segment

// Persistent words at the start of the touch-word allocation (zeroed with
// the words): the tag epoch and the step index of graph replays.
struct NtcHead {
    uint32_t epoch;
    uint32_t pad;
    uint64_t step;
};
constexpr size_t kNtcHeadBytes = 256;

struct NtcPart {
    double prob, eb, ea;
    long long coll, inv, clip;
};

template <typename T>
struct NtcArgs {
    Particles<T> pt;
    const int64_t *off_e, *off_g;
    int64_t n_cells;
    int64_t total;   // candidates of the large cells; filled on the device by ntc_live
    double dt, dn;
    uint64_t seed, step;  // step: the host's, or the device word's (dev_step)
    uint32_t epoch;       // filled on the device by ntc_live
    int32_t dev_step;
    NtcCtl* ctl;
    const NtcHead* head;
    const int64_t* count;     // [n_cells] candidates of each cell
    int64_t* cand_full;       // [n_cells] first candidate of each large cell (written by k_ntc_pick)
    const double* p_max;      // [n_cells]
    int32_t *c_ie, *c_ig, *c_cell, *c_local;
    double* c_u;              // acceptance uniform of each candidate
    const long long* bsum;    // [3 b], [3 b + 1]: small and large cells' candidates before scan workgroup b
    int64_t n_bsum;           // scan workgroups
    const int4* piece;        // per piece of kNtcPiece cells the candidates before it within its scan workgroup, in
                              // cells up to the low limit (x), between the limits (y), beyond (z)
    const int32_t* large;     // [n_cells] in no particular order: cells beyond the upper limit from the start on,
                              // those between the limits from the end back
    int32_t* pend;            // the cells left to k_ntc_serial, likewise
    uint8_t* status;  // bit 0 resolved; 2 collided, 4 invalid, 8 P > P_max
    double *r_ratio, *r_eb, *r_ea;
    unsigned long long *touch_e, *touch_g;  // [2][cap_e], [2][cap_g]
    int64_t cap_e, cap_g;
    int32_t* pending;    // [n_cells] whether the cell is in pend
    // per segment of kNtcSeg candidates: round 0's accepted candidates and
    // round 1's list (kNtcSeg entries each) with their lengths; round 2's
    // list in chunks of kNtcThreads (kNtcSub per segment) with theirs
    int32_t *lst_c, *lst_1, *lst_2;
    int32_t *cnt_c, *cnt_1, *cnt_2;
    int64_t n_seg;  // segments of the capacity
    int64_t cap;    // candidates the arrays hold
};

// The kernels below issue every read that does not depend on another one
// (the control words, the live values, their own inputs -- speculatively,
// clamped into the arrays) before they wait for any, and only then test
// whether the step proceeds: each read chain costs a memory round trip, and
// the waves of a launch run in few generations, so the round trips, not the
// arithmetic, set the kernels' length.

// The step's values that live on the device: the large cells' candidates, the tag
// epoch and (graph replays) the step index.
template <typename T>
__device__ __forceinline__ NtcArgs<T> ntc_live(const NtcArgs<T>& in) {
    NtcArgs<T> a = in;
    a.total = in.ctl->total_l;
    a.epoch = in.head->epoch;
    if (in.dev_step) a.step = in.head->step;
    return a;
}

__device__ __forceinline__ unsigned long long ntc_tag(uint32_t round_tag, int64_t j) {
    return ((unsigned long long)round_tag << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)j);
}

__device__ __forceinline__ long long wave_incl_scan64(long long v) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan of the thread values of a workgroup of THREADS (fixed
// order), and the total.
template <int THREADS>
__device__ __forceinline__ long long block_excl_scan64(long long v, long long* lds, long long* total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const long long inc = wave_incl_scan64(v);
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    long long before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        if (w < wave) before += lds[w];
        tot += lds[w];
    }
    __syncthreads();
    *total = tot;
    return before + inc - v;
}

// Marks in place of a cell's count: a bad layout, or 2^31 - 1 or more
// candidates.
constexpr long long kNtcBadCount = -1, kNtcBadLayout = -2;

// The largest finite non-negative weight of electrons [e0, e0 + nec) and
// photons [g0, g0 + ngc) (both not empty) that lane l of `n` finds (a maximum does
// not depend on the order; past a species' end its first weight is read again).
template <typename T>
__device__ __forceinline__ T ntc_largest_weight(const T* ew, const T* gw, int64_t e0, int64_t nec, int64_t g0,
                                                int64_t ngc, int l, int n) {
    T w = (T)0;
    const int64_t most = nec > ngc ? nec : ngc;
    for (int64_t b = 0; b < most; b += 4 * n) {
        T v[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = b + n * q + l;
            v[q] = ew[e0 + (i < nec ? i : 0)];
            v[4 + q] = gw[g0 + (i < ngc ? i : 0)];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) w = isfinite(v[q]) && v[q] > w ? v[q] : w;
    }
    return w;
}

// L lanes per cell: the largest valid weight, the bound and the candidate
// count; bound by reading the weights once (8 per lane in flight).  With 16
// lanes per cell, cells of kNtcCountLong of a species or more are read by the whole
// wave, one after another (100000 cells of 16 and one of a million: the step
// 8.6 ms without, 4.3 ms so).
constexpr uint32_t kNtcCountLong = 512;

template <typename T, int L>
__global__ __launch_bounds__(kNtcThreads) void k_ntc_count(const T* ew, const T* gw, const int64_t* off_e,
                                                         const int64_t* off_g, int64_t n_cells, int64_t ne,
                                                         int64_t ng, double dt, double dn, uint64_t seed,
                                                         uint64_t step_host, const NtcHead* head, int dev_step,
                                                         int64_t* count, double* p_max, int32_t* pending) {
    static_assert(L == 16 || L == 64, "lanes of a cell");
    const int l = lane_id() & (L - 1);
    const int64_t c = ((int64_t)blockIdx.x * kNtcThreads + threadIdx.x) / L;
    if (c >= n_cells) return;  // (whole cells, the last ones of the last workgroup)
    const uint64_t step = dev_step ? head->step : step_host;
    const int64_t e0 = off_e[c], e1 = off_e[c + 1], g0 = off_g[c], g1 = off_g[c + 1];
    const bool bad = e0 < 0 || e1 < e0 || e1 > ne || g0 < 0 || g1 < g0 || g1 > ng ||
                     (c == 0 && (e0 != 0 || g0 != 0)) || (c == n_cells - 1 && (e1 != ne || g1 != ng));
    const int64_t nec = bad ? 0 : e1 - e0, ngc = bad ? 0 : g1 - g0;
    T w = (T)0;
    const bool is_long = L < 64 && ((uint32_t)nec | (uint32_t)ngc) >= kNtcCountLong;
    if (nec > 0 && ngc > 0 && !is_long) w = ntc_largest_weight(ew, gw, e0, nec, g0, ngc, l, L);
    if (L < 64 && any_lane(is_long)) {
        const int n = __popcll(lanes(true));  // (the lanes of the wave's cells)
        for (uint64_t m = lanes(is_long && l == 0 && nec > 0 && ngc > 0); m; m &= m - 1) {
            const int src = (int)__ffsll((unsigned long long)m) - 1;  // the cell's first lane
            T v = ntc_largest_weight(ew, gw, __shfl((long long)e0, src, 64), __shfl((long long)nec, src, 64),
                                     __shfl((long long)g0, src, 64), __shfl((long long)ngc, src, 64), lane_id(), n);
#pragma unroll
            for (int o = L / 2; o > 0; o >>= 1) {
                const T x = __shfl_xor(v, o, 64);
                v = x > v ? x : v;
            }
            for (int o = 0; o < n; o += L) {
                const T x = __shfl(v, o, 64);
                if (lane_id() - l == src) w = x > w ? x : w;
            }
        }
    }
#pragma unroll
    for (int o = L / 2; o > 0; o >>= 1) {
        const T v = __shfl_xor(w, o, 64);
        w = v > w ? v : w;
    }
    if (l == 0) {
        long long n = 0;
        double pm = 0.0;
        if (bad) {
            n = kNtcBadLayout;
        } else if (nec > 0 && ngc > 0) {
            pm = 2.0 * dt * dn * (double)w;
            const double n_exp = (double)nec * (double)ngc * pm;
            if (!(n_exp < (double)kNtcMaxCand)) {
                n = kNtcBadCount;
            } else {
                const double fl = floor(n_exp);
                const u32x4 r = draw(seed, (uint64_t)c, step, kNtcCount);
                n = (long long)fl + (uniform53(r.a, r.b) < n_exp - fl ? 1 : 0);
            }
        }
        pending[c] = 0;
        count[c] = n;
        p_max[c] = pm;
    }
}

// The candidates before each piece of cells, the lists of the cells beyond the
// limits, and, by the workgroup that finishes last, which of them are large ones,
// the small and the large cells' candidates before each workgroup, the totals, and
// whether the step proceeds (a valid layout, fewer than 2^31 - 1 candidates, at
// most `cap` of them).  When the tag epoch is about to wrap, it clears the touch
// words and restarts the epoch at 0.  With `host` set the control words go there
// too.
__global__ __launch_bounds__(kNtcThreads) void k_ntc_scan(const int64_t* count, int64_t n_cells, int4* piece,
                                                        long long* bsum, int32_t* large, int64_t cap,
                                                        NtcCtl* ctl, NtcHead* head, unsigned long long* touch,
                                                        int64_t n_touch, NtcCtl* host) {
    __shared__ long long s[kNtcThreads / 64];
    __shared__ int s_last;
    constexpr long long kBadCount = 1ll << 60, kBadLayout = 1ll << 61;  // marks in a workgroup's word
    const int64_t base = (int64_t)blockIdx.x * kNtcScanBlock + (int64_t)threadIdx.x * kNtcScanPer;
    long long small = 0, lots = 0;  // small: cells up to the low limit, and those between the limits 32 bits up
    int marks = 0;
    int64_t v[kNtcScanPer];
#pragma unroll
    for (int q = 0; q < kNtcScanPer; ++q) v[q] = base + q < n_cells ? count[base + q] : 0;
#pragma unroll
    for (int q = 0; q < kNtcScanPer; ++q) {
        if (v[q] < 0) {
            marks |= v[q] == kNtcBadLayout ? 2 : 1;
        } else if (v[q] <= kNtcLow) {
            small += v[q];
        } else if (v[q] <= kNtcMidMax) {
            small += (long long)v[q] << 32;
            if (v[q] > kNtcMidHigh) atomicAdd(&ctl->n_high, 1u);
            large[n_cells - 1 - atomicAdd(&ctl->n_mid, 1u)] = (int32_t)(base + q);
        } else {
            lots += v[q];
            large[atomicAdd(&ctl->n_over, 1u)] = (int32_t)(base + q);
        }
    }
    long long sum_s, sum_l;
    const long long ex_s = block_excl_scan64<kNtcThreads>(small, s, &sum_s);
    const long long ex_l = block_excl_scan64<kNtcThreads>(lots, s, &sum_l);
    if (base % kNtcPiece == 0 && base < n_cells)
        piece[base / kNtcPiece] = make_int4((int)ex_s, (int)(ex_s >> 32),
                                            ex_l < kNtcMaxCand ? (int)ex_l : 0, 0);  // (else too many in all)
    const bool bad_c = __syncthreads_or(marks & 1), bad_l = __syncthreads_or(marks & 2);
    if (threadIdx.x == 0) {
        // the three words, past every cache, before the ticket (they are all
        // that the last workgroup reads of this one, so that no cache has to
        // be written back for it)
        const long long w = (sum_s & 0xFFFFFFFFll) | (bad_c ? kBadCount : 0) | (bad_l ? kBadLayout : 0);
        long long* mine = bsum + 3 * (int64_t)blockIdx.x;
        __hip_atomic_store(&mine[0], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mine[1], sum_s >> 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mine[2], sum_l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const uint32_t before = __hip_atomic_fetch_add(&ctl->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = before == gridDim.x - 1 ? 1 : 0;
    }
    __syncthreads();
    if (!s_last) return;  // (uniform in the workgroup)
    const uint32_t n_mid = __hip_atomic_load(&ctl->n_mid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t n_over = __hip_atomic_load(&ctl->n_over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t n_high = __hip_atomic_load(&ctl->n_high, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool launches = n_over + n_high > 0 || (n_cells < kNtcFew && n_mid > 0);
    const int local = !launches || n_mid >= kNtcMidMin ? kNtcMidMax : (n_cells < kNtcMidMin ? 0 : kNtcLow);
    const int64_t n_blocks = gridDim.x;
    long long total_s = 0, total_l = 0;
    bool bad_layout = false, bad_count = false;
    for (int64_t b0 = 0; b0 < n_blocks; b0 += kNtcThreads) {
        const int64_t b = b0 + threadIdx.x;
        long long ws = 0, wm = 0, wl = 0, sum;
        if (b < n_blocks) {
            ws = __hip_atomic_load(&bsum[3 * b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wm = __hip_atomic_load(&bsum[3 * b + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wl = __hip_atomic_load(&bsum[3 * b + 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        bad_layout = __syncthreads_or((ws & kBadLayout) != 0) || bad_layout;
        bad_count = __syncthreads_or((ws & kBadCount) != 0) || bad_count;
        ws &= kBadCount - 1;
        const long long bs = block_excl_scan64<kNtcThreads>(
            (local >= kNtcLow ? ws : 0) + (local >= kNtcMidMax ? wm : 0), s, &sum);
        if (b < n_blocks) bsum[3 * b] = total_s + bs;
        total_s += sum;
        const long long bl = block_excl_scan64<kNtcThreads>(
            wl + (local < kNtcMidMax ? wm : 0) + (local < kNtcLow ? ws : 0), s, &sum);
        if (b < n_blocks) bsum[3 * b + 1] = total_l + bl;
        total_l += sum;
    }
    const bool wrap = head->epoch > 0xFFFFFFFFu - 2 * kNtcRounds;  // (uniform)
    if (wrap) {
        for (int64_t i = threadIdx.x; i < n_touch; i += kNtcThreads) touch[i] = 0ull;
        __syncthreads();  // every thread has read the epoch
    }
    if (threadIdx.x == 0) {
        if (wrap) head->epoch = 0;
        const long long total = total_s + total_l;
        NtcCtl z = {};
        z.total = total;
        z.total_l = total_l;
        z.layout_bad = bad_layout ? 1 : 0;
        z.too_many = bad_count || total >= kNtcMaxCand ? 1 : 0;
        z.overflow = total > cap ? 1 : 0;
        z.go = (z.layout_bad | z.too_many | z.overflow) ? 0 : 1;
        z.n_large = local == 0 ? (uint32_t)n_cells : n_over + (local < kNtcMidMax ? n_mid : 0);
        z.n_over = n_over;
        z.n_mid = n_mid;
        z.n_high = n_high;
        z.local = local;
        *ctl = z;
        if (host) *host = z;
    }
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ long long wave_sum_ll(long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum a workgroup's per-thread partials in a fixed order (butterfly in each
// wave, then the waves in order); thread 0 gets the result.
__device__ __forceinline__ NtcPart block_sum_part(NtcPart v, NtcPart* lds) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    v.prob = wave_sum_d(v.prob);
    v.eb = wave_sum_d(v.eb);
    v.ea = wave_sum_d(v.ea);
    v.coll = wave_sum_ll(v.coll);
    v.inv = wave_sum_ll(v.inv);
    v.clip = wave_sum_ll(v.clip);
    if (lane == 0) lds[wave] = v;
    __syncthreads();
    NtcPart r = {0.0, 0.0, 0.0, 0, 0, 0};
    if (threadIdx.x == 0)
        for (int w = 0; w < kNtcThreads / 64; ++w) {
            r.prob += lds[w].prob;
            r.eb += lds[w].eb;
            r.ea += lds[w].ea;
            r.coll += lds[w].coll;
            r.inv += lds[w].inv;
            r.clip += lds[w].clip;
        }
    return r;
}

// Compaction inside a workgroup of THREADS threads: the position of this
// thread among those with `take` set (in thread order) and their number.
template <int THREADS>
__device__ __forceinline__ int compact_slot(bool take, int* lds, int* total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const unsigned long long m = __ballot(take);
    if (lane == 0) lds[wave] = __popcll(m);
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        before += w < wave ? lds[w] : 0;
        tot += lds[w];
    }
    *total = tot;
    return before + __popcll(m & ((1ull << lane) - 1));
}
__device__ __forceinline__ int seg_slot(bool take, int* lds, int* total) { return compact_slot<kNtcSeg>(take, lds, total); }
__device__ __forceinline__ int block_slot(bool take, int* lds, int* total) {
    return compact_slot<kNtcThreads>(take, lds, total);
}

// The large cells, a workgroup each time: their candidates' electrons, photons
// and acceptance uniforms; every candidate registers for round 0.
template <typename T>
__global__ __launch_bounds__(kNtcThreads) void k_ntc_pick(const NtcArgs<T> a_in) {
    if (!a_in.ctl->go) return;  // (uniform) the step does not proceed
    const uint32_t n_large = a_in.ctl->n_large, n_over = a_in.ctl->n_over;
    const int local = a_in.ctl->local;
    const NtcArgs<T> a = ntc_live(a_in);
    const int lane = lane_id();
    for (uint32_t i = blockIdx.x; i < n_large; i += gridDim.x) {
        const int64_t c = local == 0 ? (int64_t)i : a.large[i < n_over ? (int64_t)i : a.n_cells - 1 - (i - n_over)];
        const int64_t n = a.count[c];
        // the large cells' candidates before this cell's
        const int64_t cp = c / kNtcPiece * kNtcPiece;
        long long v = lane < (int)(c - cp) ? a.count[cp + lane] : 0;
        v = v > local ? v : 0;
#pragma unroll
        for (int o = kNtcPiece / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        const int4 pc = a.piece[c / kNtcPiece];
        const int64_t j0 = a.bsum[3 * (c / kNtcScanBlock) + 1] + pc.z + (local < kNtcMidMax ? pc.y : 0) +
                           (local < kNtcLow ? pc.x : 0) + __shfl(v, 0, 64);
        const int64_t e0 = a.off_e[c], e1 = a.off_e[c + 1], g0 = a.off_g[c], g1 = a.off_g[c + 1];
        if (threadIdx.x == 0) a.cand_full[c] = j0;
        const uint64_t nec = (uint64_t)(e1 - e0), ngc = (uint64_t)(g1 - g0);
        for (int64_t j = j0 + threadIdx.x; j < j0 + n; j += kNtcThreads) {
            const u32x4 r = draw(a.seed, ((uint64_t)c << 32) | (uint64_t)(j - j0), a.step, kNtcPick);
            const int32_t ie = (int32_t)(e0 + (int64_t)(((uint64_t)r.a * nec) >> 32));
            const int32_t ig = (int32_t)(g0 + (int64_t)(((uint64_t)r.b * ngc) >> 32));
            a.c_local[j] = (int32_t)(j - j0);
            a.c_u[j] = uniform53(r.c, r.d);
            a.c_ie[j] = ie;
            a.c_ig[j] = ig;
            a.c_cell[j] = (int32_t)c;
            const unsigned long long tag = ntc_tag(a.epoch, j);
            atomicMax(a.touch_e + ie, tag);
            atomicMax(a.touch_g + ig, tag);
        }
    }
}

// A candidate's probability on the current momenta and its accept/reject
// decision: the status bits (1 resolved; 2 collides, 4 invalid, 8 P > P_max),
// and P / P_max (-1 when invalid).
template <typename T>
__device__ __forceinline__ uint8_t ntc_probability(const NtcArgs<T>& a, double p_max, const PairRaw<T>& v, double u_c,
                                                   double* ratio_out) {
    const d3 p = {(double)v.p[0], (double)v.p[1], (double)v.p[2]}, k = {(double)v.k[0], (double)v.k[1], (double)v.k[2]};
    const double we = (double)v.we, wg = (double)v.wg;
    uint8_t st = 1;
    double ratio = -1.0;
    if (!finite_pair(p, we, k, wg)) {
        st |= 4;
    } else {
        const XFlux xf = x_flux(p, k, dot(p, p), dot(k, k));
        const double wmax = we > wg ? we : wg;
        const double P = xf.x > 0.0 ? a.dt * a.dn * wmax * sigma_ratio(xf.x) * xf.flux : 0.0;
        ratio = P / p_max;
        if (ratio > 1.0) st |= 8;
        if (u_c < ratio) st |= 2;
    }
    *ratio_out = ratio;
    return st;
}

// The values of the particles ie, ig.
template <typename T>
__device__ __forceinline__ PairRaw<T> ntc_load(const NtcArgs<T>& a, int32_t ie, int32_t ig) {
    return pair_load_all<T>(a.pt, PairSlot{ie, ig, 0, true});
}

// Resolve an accepted candidate (draws of index idx): scattering angle from
// the plain sampler, both momenta updated under the weight rule; the pair's
// energies before and after.  Its values come from src twice, before and
// after the sampler, so that they are not held across it.
template <typename T, typename Src>
__device__ __forceinline__ void ntc_scatter(const NtcArgs<T>& a, uint64_t step, uint64_t idx, const Src& src,
                                            double* eb, double* ea) {
    int32_t ie, ig;
    d3 p, k;
    double we, wg;
    src.get(a.pt, ie, ig, p, k, we, wg);
    const double x = pair_invariants(p, k).x;
    const u32x4 s = draw(a.seed, idx, step, kNtcScatter);
    const double v = angle_icdf_v(uniform53(s.a, s.b), x);
    asm volatile("" ::: "memory");
    src.get(a.pt, ie, ig, p, k, we, wg);
    const Scattered sc = scatter(p, k, pair_invariants(p, k), v, uniform53(s.c, s.d));
    bool upd_e = true, upd_g = true;
    if (we != wg) {
        const u32x4 q = draw(a.seed, idx, step, kNtcWeight);
        const double wmin = we < wg ? we : wg, wmax = we < wg ? wg : we;
        const bool heavier_moves = uniform53(q.a, q.b) < wmin / wmax;
        if (we > wg)
            upd_e = heavier_moves;
        else
            upd_g = heavier_moves;
    }
    if (upd_e) {
        a.pt.ex[ie] = (T)sc.p1.x;
        a.pt.ey[ie] = (T)sc.p1.y;
        a.pt.ez[ie] = (T)sc.p1.z;
    }
    if (upd_g) {
        a.pt.gx[ig] = (T)sc.k1.x;
        a.pt.gy[ig] = (T)sc.k1.y;
        a.pt.gz[ig] = (T)sc.k1.z;
    }
    *eb = sc.e_before;
    *ea = sc.e_after;
}

// Candidate j of a large cell (cell c): its status and P / P_max to the
// records; whether it collides (the collision itself: ntc_collide).
template <typename T>
__device__ __forceinline__ bool ntc_evaluate(const NtcArgs<T>& a, int64_t j, int32_t c, int32_t ie, int32_t ig) {
    double ratio;
    const uint8_t st = ntc_probability<T>(a, a.p_max[c], ntc_load<T>(a, ie, ig), a.c_u[j], &ratio);
    a.r_ratio[j] = ratio;
    a.status[j] = st;
    return (st & 2) != 0;
}

template <typename T>
__device__ __forceinline__ void ntc_collide(const NtcArgs<T>& a, int64_t j, int32_t c, int32_t ie, int32_t ig) {
    double eb, ea;
    ntc_scatter<T>(a, a.step, ((uint64_t)c << 32) | (uint64_t)a.c_local[j], FromArrays<T>{ie, ig}, &eb, &ea);
    a.r_eb[j] = eb;
    a.r_ea[j] = ea;
}

// A window of candidates that one wave resolves in rounds: whole small cells,
// or some of a large cell's that are left.  Once per window a candidate finds
// the last earlier one of its cell with its electron and the last with its
// photon, comparing itself with them; it is ready in a round when both were
// resolved in former rounds.  Ready candidates are evaluated, the accepted ones
// staged with their values and scattered on full waves, the others stay for
// the next round (the earliest open one of all is ready in every round, so that
// the rounds end).
constexpr int kNtcWin = 256;
static_assert(kNtcMidMax <= kNtcWin && kNtcWin <= 256, "8-bit indices of a window");

template <typename T>
struct NtcWindow {
    int2 eg[kNtcWin];                    // electron, photon
    double u[kNtcWin];                   // acceptance uniform
    uint16_t done[kNtcWin];              // 1 + the round that resolved it (0: open)
    uint8_t pe[kNtcWin], pg[kNtcWin];    // the last earlier one with its electron, photon (itself: none)
    uint8_t open[2][kNtcWin];
    StagedPair<T> pool[2 * 64];          // accepted; < 64 before 64 candidates add to them
    uint8_t pool_q[2 * 64];
};

// Resolve the window's m candidates, whose eg and u are set.  own(): the
// arguments (by scalar loads where they are used, not held in registers);
// cell0(q): the first candidate of q's cell in the window; p_max(q): its bound;
// index(q): its draws'; evaluated(q, st, ratio) and scattered(q, eb, ea) take
// the results (by lanes with q's candidate; evaluated by the whole wave, st = 0
// for lanes without one).  Called by one wave, a workgroup by itself.
template <typename T, typename Own, typename Cell0, typename PMax, typename Index, typename Ev, typename Sc>
__device__ __forceinline__ void ntc_resolve(NtcWindow<T>& w, int m, uint64_t step, const Own& own, const Cell0& cell0,
                                            const PMax& p_max, const Index& index, const Ev& evaluated,
                                            const Sc& scattered) {
    const int lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    __syncthreads();  // (one wave: the order of its LDS accesses)
    for (int q = lane; q < m; q += 64) {
        const int2 eg = w.eg[q];
        const int q0 = cell0(q);
        int pe = q, pg = q;
        for (int k = q - 1; k >= q0; k -= 4) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int p = k - r >= q0 ? k - r : q;  // (past the first: itself)
                const int2 o = w.eg[p];
                pe = pe == q && o.x == eg.x ? p : pe;
                pg = pg == q && o.y == eg.y ? p : pg;
            }
        }
        w.pe[q] = (uint8_t)pe;
        w.pg[q] = (uint8_t)pg;
        w.open[0][q] = (uint8_t)q;
        w.done[q] = 0;
    }
    __syncthreads();
    int set = 0;
    uint32_t round = 0;
    for (int n = m; n > 0; set ^= 1, ++round) {  // a round over the n open candidates
        const uint8_t* was = w.open[set];
        uint8_t* still = w.open[set ^ 1];
        const NtcArgs<T>& a = *own();
        int n_pool = 0, n_open = 0;
        // (the particles of the next 64 are read ahead)
        auto fetch = [&](int i, int& q, int2& eg, PairRaw<T>& raw) {
            q = i < n ? (int)was[i] : -1;
            eg = w.eg[q < 0 ? 0 : q];
            raw = ntc_load<T>(a, eg.x, eg.y);
        };
        int q_n;
        int2 eg_n;
        PairRaw<T> raw_n;
        fetch(lane, q_n, eg_n, raw_n);
        for (int b = 0;; b += 64) {
            const bool last = b >= n;
            if (!last) {
                const int q = q_n;
                const int2 eg = eg_n;
                const PairRaw<T> raw = raw_n;
                if (b + 64 < n) fetch(b + 64 + lane, q_n, eg_n, raw_n);
                bool open = false;
                uint8_t st = 0;
                double ratio = 0.0;
                if (q >= 0) {
                    const int pe = w.pe[q], pg = w.pg[q];
                    const uint32_t de = w.done[pe], dg = w.done[pg];  // (1 + a former round)
                    open = (pe != q && (de == 0 || de > round)) || (pg != q && (dg == 0 || dg > round));
                    if (!open) {
                        w.done[q] = (uint16_t)(round + 1);
                        st = ntc_probability<T>(a, p_max(q), raw, w.u[q], &ratio);
                    }
                }
                evaluated(q, st, ratio);
                const bool acc = (st & 2) != 0;
                const uint64_t m_acc = lanes(acc), m_open = lanes(open);
                if (acc) {
                    const int i = n_pool + __popcll(m_acc & below);
                    w.pool[i] = {eg.x, eg.y, {raw.p[0], raw.p[1], raw.p[2]}, {raw.k[0], raw.k[1], raw.k[2]}, raw.we,
                                 raw.wg};
                    w.pool_q[i] = (uint8_t)q;
                }
                if (open) still[n_open + __popcll(m_open & below)] = (uint8_t)q;
                n_pool += __popcll(m_acc);
                n_open += __popcll(m_open);
            }
            // (ready candidates share no particle: those of a round may
            // scatter in any order, also before its last are evaluated)
            if (n_pool >= 64 || (last && n_pool > 0)) {
                __syncthreads();
                const NtcArgs<T>& as = *own();
                const int n_now = n_pool < 64 ? n_pool : 64;
                n_pool -= n_now;
                if (lane < n_now) {
                    const int i = n_pool + lane, q = w.pool_q[i];
                    double eb, ea;
                    ntc_scatter<T>(as, step, index(q), FromStaged<T>{&w.pool[i]}, &eb, &ea);
                    scattered(q, eb, ea);
                }
                __syncthreads();
            }
            if (last) break;
        }
        n = n_open;
        __syncthreads();
    }
}

// The kernel's first argument, by scalar loads where it is used: its address
// is made opaque, so that the arguments are not held in scalar registers (and,
// past those, in lanes of vector registers) from one use to the next.
template <typename T>
__device__ __forceinline__ const NtcArgs<T>* ntc_own_args() {
    auto p = (const __attribute__((address_space(4))) NtcArgs<T>*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (const NtcArgs<T>*)p;
}

// The small cells, one wave per group of consecutive
// cells: those whose first candidate is among the group's share of the small
// cells' candidates (the share follows from the step's totals alone, so that
// eager steps and graphs of any capacity add their sums in the same order; by
// candidates, not by cells, because a dense region's cells would fall to a few
// waves).
// FP32 storage, 443 k candidates in 16384 cells of 256: 68 us, of which the
// groups, picks and readiness take 14, the particles' memory lines (nearly all
// of the arrays) 16, the first round's scattering 15 and its writes 7, the
// later rounds 19.  As kernels of their own -- picks, evaluation, collisions,
// two rounds, the serial rest, the sums -- it was 112 us.  Workgroups of four
// waves with windows of 512 and barriers between the phases: 96.  With shares of
// 104 or 128 candidates it takes 9 and 3 % longer than with 160.
constexpr int kNtcCellBlocks = 4096;
constexpr int kNtcShare = 160;  // most candidates of a share
static_assert(kNtcShare <= 256, "8-bit indices of a group's cells");

template <typename T>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? 4 : 3) void k_ntc_cells(const NtcArgs<T> args, NtcPart* part) {
    __shared__ NtcWindow<T> s_w;
    __shared__ uint8_t s_c[kNtcWin];       // cell within the group
    __shared__ int32_t s_cell[kNtcShare];  // the group's cells (one candidate each at least)
    __shared__ int s_pre[kNtcShare + 1];   // and the group's candidates before each
    const int lane = threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint64_t step = args.dev_step ? args.head->step : args.step;
    const auto own = [] { return ntc_own_args<T>(); };
    const NtcArgs<T>& a = *own();
    const long long total_s = a.ctl->total - a.ctl->total_l;
    const int local = a.ctl->local;
    if (!a.ctl->go) return;  // (uniform) the step does not proceed
    // a share of kNtcShare candidates, less where the chip would be left idle;
    // cells of more than half a share get one each, lest some waves take two
    long long W = total_s / 2048;
    W = W < 16 ? 16 : (W > kNtcShare ? kNtcShare : W);
    const long long mean = total_s / a.n_cells;
    if (2 * mean > W && mean >= 16) {
        W = mean - mean / 8;
        W = W > kNtcShare ? kNtcShare : W;
    }
    const long long n_groups = (total_s + W - 1) / W;
    double sum_p = 0.0, sum_eb = 0.0, sum_ea = 0.0;
    long long n_coll = 0, n_inv = 0, n_clip = 0;  // (of the wave)
    for (long long grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
        const NtcArgs<T>& a = *own();
        const long long w0 = grp * W, w1 = w0 + W;
        // the last scan workgroup with at most w0 small candidates before it,
        // by 64 probes at a time, and its last such piece
        int64_t b_lo = 0, b_n = a.n_bsum;  // it is one of [b_lo, b_lo + b_n)
        while (b_n > 1) {
            const int64_t stride = (b_n + 63) / 64, b = b_lo + lane * stride;
            const int k = __popcll(lanes(b < b_lo + b_n && a.bsum[3 * (b < b_lo + b_n ? b : b_lo)] <= w0)) - 1;
            b_n = b_n - k * stride < stride ? b_n - k * stride : stride;
            b_lo += k * stride;
        }
        long long before = a.bsum[3 * b_lo];
        const int64_t n_pieces = (a.n_cells + kNtcPiece - 1) / kNtcPiece, p_l = 64 * b_lo + lane;
        const int4 pc = a.piece[p_l < n_pieces ? p_l : 64 * b_lo];
        const int in_block = pc.x + (local >= kNtcMidMax ? pc.y : 0);
        const int p = __popcll(lanes(p_l < n_pieces && before + in_block <= w0)) - 1;
        before += __builtin_amdgcn_readlane(in_block, p);
        // the group's cells, 64 cells at a time
        __syncthreads();  // (one wave: the order of its LDS accesses)
        int n_c = 0, n_cand = 0;
        for (int64_t cb = (64 * b_lo + p) * kNtcPiece; cb < a.n_cells && before < w1; cb += 64) {
            const int64_t c = cb + lane;
            const long long nn = c < a.n_cells ? a.count[c] : 0;
            const int n = nn <= local ? (int)nn : 0;
            int inc = n;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(inc, o, 64);
                if (lane >= o) inc += t;
            }
            const long long start = before + inc - n;
            const bool in = n > 0 && start >= w0 && start < w1;
            const uint64_t m_in = lanes(in);
            if (m_in) {
                // (their candidates are consecutive: those before the first of
                // them are the first one's start)
                const int first_l = (int)__ffsll((unsigned long long)m_in) - 1;
                const int last_l = 63 - __clzll((long long)m_in);
                const int s0 = __builtin_amdgcn_readlane(inc - n, first_l);
                if (in) {
                    const int i = n_c + __popcll(m_in & below);
                    s_cell[i] = (int32_t)c;
                    s_pre[i] = n_cand + inc - n - s0;
                }
                n_c += __popcll(m_in);
                n_cand += __builtin_amdgcn_readlane(inc, last_l) - s0;
            }
            before += __builtin_amdgcn_readlane(inc, 63);
        }
        if (lane == 0) s_pre[n_c] = n_cand;
        __syncthreads();
        for (int lo = 0; lo < n_c;) {
            // the window: cells lo .. hi - 1, as many as fit (one at least)
            const int first = wave_uniform(s_pre[lo]);
            int hi = lo;
            for (;;) {
                const int i = hi + lane;
                const int k = __popcll(lanes(i < n_c && s_pre[i < n_c ? i + 1 : n_c] - first <= kNtcWin));
                hi += k;
                if (k < 64) break;
            }
            const int m = wave_uniform(s_pre[hi]) - first;
            // picks
            for (int q = lane; q < m; q += 64) {
                int i = lo, top = hi - 1;
                while (i < top) {
                    const int mid = (i + top + 1) >> 1;
                    if (s_pre[mid] - first <= q)
                        i = mid;
                    else
                        top = mid - 1;
                }
                const int32_t c = s_cell[i];
                const int64_t e0 = a.off_e[c], g0 = a.off_g[c];
                const uint64_t nec = (uint64_t)(a.off_e[c + 1] - e0), ngc = (uint64_t)(a.off_g[c + 1] - g0);
                const uint64_t idx = ((uint64_t)c << 32) | (uint64_t)(uint32_t)(q + first - s_pre[i]);
                const u32x4 r = draw(a.seed, idx, step, kNtcPick);
                s_w.eg[q] = make_int2((int32_t)(e0 + (int64_t)(((uint64_t)r.a * nec) >> 32)),
                                      (int32_t)(g0 + (int64_t)(((uint64_t)r.b * ngc) >> 32)));
                s_w.u[q] = uniform53(r.c, r.d);
                s_c[q] = (uint8_t)i;
            }
            ntc_resolve<T>(
                s_w, m, step, own, [&](int q) { return s_pre[s_c[q]] - first; },
                [&](int q) { return own()->p_max[s_cell[s_c[q]]]; },
                [&](int q) {
                    const int i = s_c[q];
                    return ((uint64_t)s_cell[i] << 32) | (uint64_t)(uint32_t)(q + first - s_pre[i]);
                },
                [&](int, uint8_t st, double ratio) {
                    sum_p += st & 4 ? 0.0 : ratio;
                    n_coll += __popcll(lanes((st & 2) != 0));
                    n_inv += __popcll(lanes((st & 4) != 0));
                    n_clip += __popcll(lanes((st & 8) != 0));
                },
                [&](int, double eb, double ea) {
                    sum_eb += eb;
                    sum_ea += ea;
                });
            lo = hi;
        }
    }
    NtcPart r;
    r.prob = wave_sum_d(sum_p);
    r.eb = wave_sum_d(sum_eb);
    r.ea = wave_sum_d(sum_ea);
    r.coll = n_coll;
    r.inv = n_inv;
    r.clip = n_clip;
    if (lane == 0) part[blockIdx.x] = r;
}

// Round 0 of the large cells, one workgroup per segment of kNtcSeg
// candidates, one lane per candidate: the earliest registered toucher of both
// its particles is evaluated, and the accepted ones compacted into the
// segment's collide list; the others register for round 1 and are compacted
// into the segment's round-1 list.
template <typename T>
__global__ __launch_bounds__(kNtcSeg) void k_ntc_eval(const NtcArgs<T> a_in) {
    __shared__ int s_acc[kNtcSeg / 64], s_later[kNtcSeg / 64];
    const int64_t base = (int64_t)blockIdx.x * kNtcSeg;
    const int64_t j = base + threadIdx.x;
    const int64_t jc = j < a_in.cap ? j : a_in.cap - 1;
    const int32_t go = a_in.ctl->go;
    const NtcArgs<T> a = ntc_live(a_in);
    const int32_t ie = a.c_ie[jc], ig = a.c_ig[jc], cell = a.c_cell[jc];
    if (!go || base >= a.total) return;  // (uniform) no step, or past the candidates
    bool acc = false, later = false;
    if (j < a.total) {
        const unsigned long long mine = ntc_tag(a.epoch, j);
        const bool ready = a.touch_e[ie] == mine && a.touch_g[ig] == mine;
        if (!ready) {
            const unsigned long long next = ntc_tag(a.epoch + 1u, j);
            atomicMax(a.touch_e + a.cap_e + ie, next);
            atomicMax(a.touch_g + a.cap_g + ig, next);
            later = true;
            a.status[j] = 0;
        }
        if (ready) acc = ntc_evaluate<T>(a, j, cell, ie, ig);
    }
    int n_acc, n_later;
    const int pa = seg_slot(acc, s_acc, &n_acc);
    const int pl = seg_slot(later, s_later, &n_later);
    if (acc) a.lst_c[base + pa] = (int32_t)j;
    if (later) a.lst_1[base + pl] = (int32_t)j;
    if (threadIdx.x == 0) {
        a.cnt_c[blockIdx.x] = n_acc;
        a.cnt_1[blockIdx.x] = n_later;
    }
}

// Round 0's accepted candidates, one per lane (they share no particle, so
// their order does not matter).  Workgroups of kNtcThreads, kNtcSub per
// segment: a small workgroup whose waves have nothing to do frees its
// place at once, so the few waves that work spread over the chip.
// Workgroup b takes part b / n_seg of segment b % n_seg: the first parts
// (the ones most often busy, as lists fill from their start) are
// consecutive workgroups, which the dispatcher deals out over all XCDs.
template <typename T>
__global__ __launch_bounds__(kNtcThreads) void k_ntc_collide_list(const NtcArgs<T> a_in) {
    const int64_t seg = blockIdx.x % a_in.n_seg;
    const int i = (int)(blockIdx.x / a_in.n_seg) * kNtcThreads + (int)threadIdx.x;
    const int32_t go = a_in.ctl->go;
    const NtcArgs<T> a = ntc_live(a_in);
    const int32_t n = a.cnt_c[seg];
    const int64_t j = a.lst_c[seg * kNtcSeg + i];  // (read whatever the count: i < kNtcSeg)
    if (!go || seg * kNtcSeg >= a.total || i >= n) return;
    ntc_collide<T>(a, j, a.c_cell[j], a.c_ie[j], a.c_ig[j]);
}

// Round t (1 or 2), one lane per list entry, workgroups of kNtcThreads:
// round 1 over the segments' round-1 lists (kNtcSub workgroups per
// segment, mapped as in k_ntc_collide_list), round 2 over the chunks of
// kNtcThreads entries that round 1 wrote.  A candidate that is the earliest registered toucher of both its
// particles is evaluated and, when accepted, collides in place (few
// candidates are left after round 0); in round 1 the others register for
// round 2 and are compacted into the workgroup's chunk of the round-2 list,
// in round 2 they mark their cell for the serial pass.
template <typename T>
__global__ __launch_bounds__(kNtcThreads) void k_ntc_round(const NtcArgs<T> a_in, int t) {
    __shared__ int s_later[kNtcThreads / 64];
    const int64_t seg = blockIdx.x % a_in.n_seg;
    const int sub = (int)(blockIdx.x / a_in.n_seg) * kNtcThreads;
    const int64_t chunk = (int64_t)blockIdx.x * kNtcThreads;  // this workgroup's chunk of the lists
    const int32_t go = a_in.ctl->go;
    const NtcArgs<T> a = ntc_live(a_in);
    // entries of this workgroup: round 1, the part [sub, sub + kNtcThreads)
    // of the segment's list; round 2, its own chunk (read whatever the count)
    const int32_t cnt = t == 1 ? a.cnt_1[seg] : a.cnt_2[blockIdx.x];
    const int64_t j_l = t == 1 ? a.lst_1[seg * kNtcSeg + sub + threadIdx.x] : a.lst_2[chunk + threadIdx.x];
    if (!go || seg * kNtcSeg >= a.total) return;  // (uniform) no step, or past the candidates
    const int n = t == 1 ? min(cnt - sub, kNtcThreads) : cnt;
    if (n <= 0) {
        if (t == 1 && threadIdx.x == 0) a.cnt_2[blockIdx.x] = 0;
        return;  // (uniform)
    }
    bool later = false;
    int64_t j = 0;
    if ((int)threadIdx.x < n) {
        j = j_l;
        const int32_t ie = a.c_ie[j], ig = a.c_ig[j], c = a.c_cell[j];
        const unsigned long long* te = a.touch_e + (t & 1) * a.cap_e;
        const unsigned long long* tg = a.touch_g + (t & 1) * a.cap_g;
        const unsigned long long mine = ntc_tag(a.epoch + (uint32_t)t, j);
        if (te[ie] == mine && tg[ig] == mine) {
            if (ntc_evaluate<T>(a, j, c, ie, ig)) ntc_collide<T>(a, j, c, ie, ig);
        } else if (t + 1 < kNtcRounds) {
            const unsigned long long next = ntc_tag(a.epoch + (uint32_t)(t + 1), j);
            atomicMax(a.touch_e + ((t + 1) & 1) * a.cap_e + ie, next);
            atomicMax(a.touch_g + ((t + 1) & 1) * a.cap_g + ig, next);
            later = true;
        } else {
            if (atomicExch(&a.pending[c], 1) == 0) a.pend[atomicAdd(&a.ctl->n_pend, 1u)] = c;
        }
    }
    if (t + 1 < kNtcRounds) {  // (uniform: t == 1)
        int n_later;
        const int pl = block_slot(later, s_later, &n_later);
        if (later) a.lst_2[chunk + pl] = (int32_t)j;
        if (threadIdx.x == 0) a.cnt_2[blockIdx.x] = n_later;
    }
}

// The large cells with candidates left, one wave each time: the candidates not
// yet resolved, in order, a window of them at a time (in order one by one, by
// one lane, they were most of the step on dense plasmas: the whole step on
// 2796 cells of 1500 particles and 3000 candidates 6.13 -> 4.01 ms, on 3000
// cells of uneven filling, 1000 on average, 3.22 -> 0.76 ms).
template <typename T>
__global__ __launch_bounds__(64) void k_ntc_serial(const NtcArgs<T> args) {
    __shared__ NtcWindow<T> s_w;
    __shared__ int32_t s_l[kNtcWin];  // candidate within the cell
    if (!args.ctl->go) return;  // (uniform)
    const uint32_t n_pend = args.ctl->n_pend;
    const int lane = threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint64_t step = args.dev_step ? args.head->step : args.step;
    const auto own = [] { return ntc_own_args<T>(); };
    for (uint32_t k = blockIdx.x; k < n_pend; k += gridDim.x) {
        const NtcArgs<T>& a = *own();
        const int32_t c = wave_uniform(a.pend[k]);
        const int64_t j0 = a.cand_full[c], j1 = j0 + a.count[c];
        for (int64_t jb = j0; jb < j1;) {
            __syncthreads();  // (one wave: the order of its LDS accesses)
            int m = 0;
            for (; jb < j1 && m <= kNtcWin - 64; jb += 64) {
                const int64_t j = jb + lane;
                const bool left = j < j1 && !(a.status[j < j1 ? j : j0] & 1);
                const uint64_t m_left = lanes(left);
                if (left) {
                    const int q = m + __popcll(m_left & below);
                    s_l[q] = (int32_t)(j - j0);
                    s_w.eg[q] = make_int2(a.c_ie[j], a.c_ig[j]);
                    s_w.u[q] = a.c_u[j];
                }
                m += __popcll(m_left);
            }
            ntc_resolve<T>(
                s_w, m, step, own, [](int) { return 0; }, [&](int) { return own()->p_max[c]; },
                [&](int q) { return ((uint64_t)(uint32_t)c << 32) | (uint64_t)(uint32_t)s_l[q]; },
                [&](int q, uint8_t st, double ratio) {
                    if (st) {
                        const NtcArgs<T>& r = *own();
                        r.r_ratio[j0 + s_l[q]] = ratio;
                        r.status[j0 + s_l[q]] = st;
                    }
                },
                [&](int q, double eb, double ea) {
                    const NtcArgs<T>& r = *own();
                    r.r_eb[j0 + s_l[q]] = eb;
                    r.r_ea[j0 + s_l[q]] = ea;
                });
        }
    }
}

__global__ __launch_bounds__(kNtcThreads) void k_ntc_reduce(const uint8_t* status, const double* ratio,
                                                          const double* eb, const double* ea, const NtcCtl* ctl,
                                                          int64_t cap, NtcPart* part) {
    __shared__ NtcPart s[kNtcThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kNtcThreads * kNtcRedPer + threadIdx.x;
    const int64_t total = ctl->total_l;
    const int32_t go = ctl->go;
    uint8_t st[kNtcRedPer];
    double rt[kNtcRedPer], b[kNtcRedPer], e[kNtcRedPer];
#pragma unroll
    for (int q = 0; q < kNtcRedPer; ++q) {  // (clamped into the arrays; used below the total only)
        const int64_t j = base + (int64_t)q * kNtcThreads;
        const int64_t jc = j < cap ? j : cap - 1;
        st[q] = status[jc];
        rt[q] = ratio[jc];
        b[q] = eb[jc];
        e[q] = ea[jc];
    }
    // (uniform) the step did not proceed, or a workgroup past the candidates
    if (!go || (int64_t)blockIdx.x * kNtcThreads * kNtcRedPer >= total) return;
    NtcPart v = {0.0, 0.0, 0.0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < kNtcRedPer; ++q) {
        const int64_t j = base + (int64_t)q * kNtcThreads;
        if (j >= total) break;
        if (st[q] & 4) {
            v.inv += 1;
            continue;
        }
        v.prob += rt[q];
        v.clip += (st[q] & 8) ? 1 : 0;
        if (st[q] & 2) {
            v.coll += 1;
            v.eb += b[q];
            v.ea += e[q];
        }
    }
    const NtcPart r = block_sum_part(v, s);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// The stats record from both paths' partials (n_cell of the workgroups of
// k_ntc_cells), the control words cleared for the next step, the epoch and
// the step word advanced.
__global__ __launch_bounds__(kNtcThreads) void k_ntc_final(const NtcPart* cell_part, int64_t n_cell,
                                                         const NtcPart* part, cs_stats* stats, NtcCtl* ctl,
                                                         NtcHead* head) {
    __shared__ NtcPart s[kNtcThreads / 64];
    const NtcCtl c = *ctl;
    const int64_t n_part = (c.total_l + kNtcThreads * kNtcRedPer - 1) / (kNtcThreads * kNtcRedPer);
    NtcPart v = {0.0, 0.0, 0.0, 0, 0, 0};
    auto add = [&](const NtcPart& p) {
        v.prob += p.prob;
        v.eb += p.eb;
        v.ea += p.ea;
        v.coll += p.coll;
        v.inv += p.inv;
        v.clip += p.clip;
    };
    if (c.go) {
        // four records in flight per thread, added in order
        for (int64_t b0 = threadIdx.x; b0 < n_cell; b0 += 4 * kNtcThreads) {
            NtcPart p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t b = b0 + (int64_t)q * kNtcThreads;
                p[q] = cell_part[b < n_cell ? b : 0];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (b0 + (int64_t)q * kNtcThreads < n_cell) add(p[q]);
        }
        for (int64_t b = threadIdx.x; b < n_part; b += kNtcThreads) add(part[b]);
    }
    const NtcPart r = block_sum_part(v, s);
    if (threadIdx.x == 0) {
        NtcCtl z = {};
        *ctl = z;
        head->epoch += kNtcRounds;
        head->step += 1;
    }
    if (threadIdx.x == 0 && stats) {
        cs_stats o = {};
        if (c.layout_bad) {
            o.layout_error = 1;
        } else if (!c.go) {  // too many candidates: nothing was changed
            o.n_pairs = c.too_many ? kNtcMaxCand : c.total;
            o.overflow = 1;
        } else {
            o.n_pairs = c.total;
            o.n_collided = r.coll;
            o.n_clipped = r.clip;
            o.n_invalid = r.inv;
            o.sum_prob = r.prob;
            o.energy_before = r.eb;
            o.energy_after = r.ea;
        }
        *stats = o;
    }
}

__global__ void k_ntc_stats_layout(cs_stats* stats) {
    cs_stats o = {};
    o.layout_error = 1;
    *stats = o;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Device scratch of a step, laid out from sizes the host knows before the
// step: the cell count, the candidate capacity and the particle counts.
struct NtcLayout {
    int64_t nb, n_cell, n_pb, n_seg, n_part;  // scan, cell, pick, segment and reduction workgroups
    size_t b_count, b_off, b_pmax, b_i32c, b_piece, b_bsum, b_ctl, b_cpart, cell;
    size_t b_i32, b_u8, b_d, b_part, b_lst, b_cnt, cand;
};

static NtcLayout ntc_layout(int64_t n_cells, int64_t cap) {
    NtcLayout l;
    l.nb = (n_cells + kNtcScanBlock - 1) / kNtcScanBlock;
    if (l.nb < 1) l.nb = 1;  // (a step without cells too)
    // (a small cell has at most kNtcMidMax candidates, a share 14 or more; waves
    // take groups in grid strides, so that any number of them is right)
    constexpr int64_t kSharesPerCell = kNtcMidMax / 16;
    l.n_cell = n_cells < kNtcCellBlocks / kSharesPerCell ? n_cells * kSharesPerCell : kNtcCellBlocks;
    l.n_pb = n_cells < 2048 ? n_cells : 2048;
    l.n_seg = (cap + kNtcSeg - 1) / kNtcSeg;
    l.n_part = (cap + kNtcThreads * kNtcRedPer - 1) / (kNtcThreads * kNtcRedPer);
    const size_t nc = (size_t)(n_cells > 0 ? n_cells : 1);
    l.b_count = align256(8 * nc);
    l.b_off = l.b_count;
    l.b_pmax = l.b_count;
    l.b_i32c = align256(4 * nc);
    l.b_piece = align256(sizeof(int4) * ((nc + kNtcPiece - 1) / kNtcPiece));
    l.b_bsum = align256(24 * (size_t)l.nb);
    l.b_cpart = align256(sizeof(NtcPart) * (size_t)(l.n_cell > 0 ? l.n_cell : 1));
    l.b_ctl = align256(sizeof(NtcCtl));
    l.cell = l.b_ctl + l.b_count + l.b_off + l.b_pmax + 3 * l.b_i32c + l.b_piece + l.b_bsum + l.b_cpart;
    const size_t tc = (size_t)(cap > 0 ? cap : 1);
    l.b_i32 = align256(4 * tc);
    l.b_u8 = align256(tc);
    l.b_d = align256(8 * tc);
    l.b_part = align256(sizeof(NtcPart) * (size_t)(l.n_part > 0 ? l.n_part : 1));
    l.b_lst = align256(4 * (size_t)(l.n_seg > 0 ? l.n_seg : 1) * kNtcSeg);
    l.b_cnt = align256(4 * (size_t)(l.n_seg > 0 ? l.n_seg : 1) * kNtcSub);
    l.cand = 4 * l.b_i32 + l.b_u8 + 4 * l.b_d + l.b_part + 3 * l.b_lst + 3 * l.b_cnt;
    return l;
}

static size_t touch_bytes(int64_t cap_e, int64_t cap_g) { return kNtcHeadBytes + 2 * 8 * (size_t)(cap_e + cap_g); }

static hipError_t grow(void** buf, size_t* bytes, size_t want, hipStream_t st, bool* fresh = nullptr) {
    if (fresh) *fresh = false;
    if (*bytes >= want) return hipSuccess;
    hipError_t e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    if (*buf) {
        e = hipFree(*buf);
        *buf = nullptr;
        *bytes = 0;
        if (e != hipSuccess) return e;
    }
    const size_t g = want + want / 4;
    e = hipMalloc(buf, g);
    if (e != hipSuccess) {
        *buf = nullptr;
        return e;
    }
    *bytes = g;
    if (fresh) *fresh = true;
    return hipSuccess;
}

void ntc_free(NtcState& s) {
    if (s.cell_ws) (void)hipFree(s.cell_ws);
    if (s.cand_ws) (void)hipFree(s.cand_ws);
    if (s.touch) (void)hipFree(s.touch);
    if (s.host) (void)hipHostFree(s.host);
    if (s.ev) (void)hipEventDestroy(s.ev);
    s = NtcState{};
}

// Scratch for a step of n_cells cells, `cap` candidates and ne / ng
// particles: the per-cell area (zeroed when fresh: its control words start
// at zero), the per-candidate area, and the touch words with their head
// (zeroed when (re)allocated).  Synchronises `st` when a buffer grows.
static hipError_t ntc_reserve(NtcState& s, int64_t n_cells, int64_t cap, int64_t ne, int64_t ng, hipStream_t st) {
    const NtcLayout l = ntc_layout(n_cells, cap);
    bool fresh = false;
    hipError_t err = grow(&s.cell_ws, &s.cell_bytes, l.cell, st, &fresh);
    if (err != hipSuccess) return err;
    if (fresh) {
        err = hipMemsetAsync(s.cell_ws, 0, s.cell_bytes, st);
        if (err != hipSuccess) return err;
    }
    if (cap > 0 || s.cand_ws == nullptr) {
        err = grow(&s.cand_ws, &s.cand_bytes, l.cand, st);
        if (err != hipSuccess) return err;
    }
    if (cap > s.cand_cap) s.cand_cap = cap;
    if (s.cap_e < ne || s.cap_g < ng || s.touch == nullptr) {
        err = hipStreamSynchronize(st);
        if (err != hipSuccess) return err;
        if (s.touch) (void)hipFree(s.touch);
        s.touch = nullptr;
        s.cap_e = ne > s.cap_e ? ne + ne / 4 : s.cap_e;
        s.cap_g = ng > s.cap_g ? ng + ng / 4 : s.cap_g;
        if (s.cap_e < 1) s.cap_e = 1;
        if (s.cap_g < 1) s.cap_g = 1;
        err = hipMalloc(&s.touch, touch_bytes(s.cap_e, s.cap_g));
        if (err != hipSuccess) {
            s.touch = nullptr;
            s.cap_e = s.cap_g = 0;
            return err;
        }
        err = hipMemsetAsync(s.touch, 0, touch_bytes(s.cap_e, s.cap_g), st);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// A step for the candidate capacity s.cand_cap, queued in three parts (no
// host synchronisation, no allocation, no memset: capturable): the counts,
// the small cells, with `host` set the control words written there by the
// first and `ev` recorded behind it; the large cells; the stats record.
template <typename T>
struct NtcQueue {
    NtcArgs<T> a;
    NtcLayout l;
    int64_t cap;
    NtcCtl* ctl;
    NtcHead* head;
    NtcPart *cell_part, *part;
    hipStream_t st;

    hipError_t start(const NtcState& s, const cs_species& e, const cs_species& g, const int64_t* off_e,
                     const int64_t* off_g, int64_t n_cells, double dt, double dn, uint64_t seed, uint64_t step,
                     bool dev_step, hipStream_t stream, void* host, hipEvent_t ev) {
        st = stream;
        cap = s.cand_cap;
        l = ntc_layout(n_cells, cap);
        char* cw = (char*)s.cell_ws;
        ctl = (NtcCtl*)cw;
        int64_t* count = (int64_t*)(cw += l.b_ctl);
        int64_t* cand_full = (int64_t*)(cw += l.b_count);
        double* p_max = (double*)(cw += l.b_off);
        int32_t* pending = (int32_t*)(cw += l.b_pmax);
        int32_t* large = (int32_t*)(cw += l.b_i32c);
        int32_t* pend = (int32_t*)(cw += l.b_i32c);
        int4* piece = (int4*)(cw += l.b_i32c);
        long long* bsum = (long long*)(cw += l.b_piece);
        cell_part = (NtcPart*)(cw += l.b_bsum);
        head = (NtcHead*)s.touch;
        unsigned long long* touch = (unsigned long long*)((char*)s.touch + kNtcHeadBytes);
        if (n_cells > 0) {
            // a wave per cell; 16 lanes each for cells of at most 32 of a
            // species on average (262144 cells of 16: 27 us, with
            // a wave each 102)
            const bool few = e.n <= 32 * n_cells && g.n <= 32 * n_cells;
            const int64_t per = kNtcThreads / (few ? 16 : 64);
            (few ? k_ntc_count<T, 16> : k_ntc_count<T, 64>)<<<(unsigned)((n_cells + per - 1) / per), kNtcThreads, 0, st>>>(
                (const T*)e.w, (const T*)g.w, off_e, off_g, n_cells, e.n, g.n, dt, dn, seed, step, head,
                dev_step ? 1 : 0, count, p_max, pending);
        }
        k_ntc_scan<<<(unsigned)l.nb, kNtcThreads, 0, st>>>(count, n_cells, piece, bsum, large, cap, ctl, head, touch,
                                                           2 * (s.cap_e + s.cap_g), (NtcCtl*)host);
        if (host) {
            const hipError_t err = hipEventRecord(ev, st);
            if (err != hipSuccess) return err;
        }
        a.pt = {(T*)e.x, (T*)e.y, (T*)e.z, (T*)e.w, (T*)g.x, (T*)g.y, (T*)g.z, (T*)g.w};
        a.off_e = off_e;
        a.off_g = off_g;
        a.n_cells = n_cells;
        a.total = 0;
        a.dt = dt;
        a.dn = dn;
        a.seed = seed;
        a.step = step;
        a.epoch = 0;
        a.dev_step = dev_step ? 1 : 0;
        a.ctl = ctl;
        a.head = head;
        a.count = count;
        a.bsum = bsum;
        a.n_bsum = l.nb;
        a.piece = piece;
        a.large = large;
        a.pend = pend;
        a.cand_full = cand_full;
        a.p_max = p_max;
        char* q = (char*)s.cand_ws;
        a.c_ie = (int32_t*)q;
        a.c_ig = (int32_t*)(q += l.b_i32);
        a.c_cell = (int32_t*)(q += l.b_i32);
        a.c_local = (int32_t*)(q += l.b_i32);
        a.status = (uint8_t*)(q += l.b_i32);
        a.r_ratio = (double*)(q += l.b_u8);
        a.r_eb = (double*)(q += l.b_d);
        a.r_ea = (double*)(q += l.b_d);
        a.c_u = (double*)(q += l.b_d);
        part = (NtcPart*)(q += l.b_d);
        a.lst_c = (int32_t*)(q += l.b_part);
        a.lst_1 = (int32_t*)(q += l.b_lst);
        a.lst_2 = (int32_t*)(q += l.b_lst);
        a.cnt_c = (int32_t*)(q += l.b_lst);
        a.cnt_1 = (int32_t*)(q += l.b_cnt);
        a.cnt_2 = (int32_t*)(q += l.b_cnt);
        a.n_seg = l.n_seg > 0 ? l.n_seg : 1;
        a.cap = cap > 0 ? cap : 1;
        a.touch_e = touch;
        a.touch_g = touch + 2 * s.cap_e;
        a.cap_e = s.cap_e;
        a.cap_g = s.cap_g;
        a.pending = pending;
        if (n_cells > 0) k_ntc_cells<T><<<(unsigned)l.n_cell, 64, 0, st>>>(a, cell_part);
        return hipGetLastError();
    }

    void large() {
        if (a.n_cells <= 0 || cap <= kNtcLow) return;  // (no cell can have more than the capacity: none is large)
        k_ntc_pick<T><<<(unsigned)l.n_pb, kNtcThreads, 0, st>>>(a);
        // one workgroup per segment, up to the capacity; kNtcSub smaller ones per segment
        k_ntc_eval<T><<<(unsigned)l.n_seg, kNtcSeg, 0, st>>>(a);
        const unsigned grid = (unsigned)(l.n_seg * kNtcSub);
        k_ntc_collide_list<T><<<grid, kNtcThreads, 0, st>>>(a);
        for (int t = 1; t < kNtcRounds; ++t) k_ntc_round<T><<<grid, kNtcThreads, 0, st>>>(a, t);
        k_ntc_serial<T><<<(unsigned)l.n_pb, 64, 0, st>>>(a);
        k_ntc_reduce<<<(unsigned)l.n_part, kNtcThreads, 0, st>>>(a.status, a.r_ratio, a.r_eb, a.r_ea, ctl, a.cap,
                                                                 part);
    }

    hipError_t finish(cs_stats* stats) {
        k_ntc_final<<<1, kNtcThreads, 0, st>>>(cell_part, l.n_cell, part, stats, ctl, head);
        return hipGetLastError();
    }
};

template <typename T>
static hipError_t ntc_launch(NtcState& s, const cs_species& e, const cs_species& g, const int64_t* off_e,
                             const int64_t* off_g, int64_t n_cells, double dt, double dn, uint64_t seed,
                             uint64_t step, cs_stats* stats, hipStream_t st, NtcOutcome* out) {
    *out = NtcOutcome::kOk;
    if (n_cells == 0 && (e.n != 0 || g.n != 0)) {
        *out = NtcOutcome::kLayout;
        if (stats) k_ntc_stats_layout<<<1, 1, 0, st>>>(stats);
        return hipGetLastError();
    }
    hipError_t err = ntc_reserve(s, n_cells, s.cand_cap, e.n, g.n, st);
    if (err != hipSuccess) return err;
    if (!s.host) {
        err = hipHostMalloc(&s.host, sizeof(NtcCtl), hipHostMallocDefault);
        if (err != hipSuccess) {
            s.host = nullptr;
            return err;
        }
    }
    if (!s.ev) {
        err = hipEventCreateWithFlags(&s.ev, hipEventDisableTiming);
        if (err != hipSuccess) {
            s.ev = nullptr;
            return err;
        }
    }
    // The counts and the small cells are queued at once; the host then waits
    // only for the counts' control words (the small cells run meanwhile) and
    // queues the large cells if there are any (or does so before it waits, if
    // the step before had some: their kernels leave where there are none, and
    // the chip does not idle meanwhile).  A step with more candidates than the
    // capacity changed nothing: the scratch grows and the step is queued again
    // (same inputs, same candidates).
    NtcQueue<T> q;
    err = q.start(s, e, g, off_e, off_g, n_cells, dt, dn, seed, step, false, st, s.host, s.ev);
    const bool ahead = s.had_large;
    if (err == hipSuccess && ahead) q.large();
    if (err == hipSuccess) err = hipEventSynchronize(s.ev);
    if (err != hipSuccess) return err;
    const NtcCtl h = *(const NtcCtl*)s.host;
    s.had_large = h.total_l > 0;
    if (h.go && h.total_l > 0 && !ahead) q.large();
    err = q.finish(stats);
    if (err != hipSuccess) return err;
    if (h.layout_bad) {
        *out = NtcOutcome::kLayout;
        return hipSuccess;
    }
    if (h.too_many) {
        *out = NtcOutcome::kTooMany;
        return hipSuccess;
    }
    if (h.overflow) {
        err = ntc_reserve(s, n_cells, h.total + h.total / 4, e.n, g.n, st);
        if (err == hipSuccess)
            err = q.start(s, e, g, off_e, off_g, n_cells, dt, dn, seed, step, false, st, nullptr, nullptr);
        if (err != hipSuccess) return err;
        if (h.total_l > 0) q.large();
        err = q.finish(stats);
    }
    return err;
}

hipError_t ntc_step(NtcState& s, cs_dtype dtype, const cs_species& e, const cs_species& g, const int64_t* off_e,
                    const int64_t* off_g, int64_t n_cells, double dt, double dn, uint64_t seed, uint64_t step,
                    cs_stats* stats, hipStream_t st, NtcOutcome* out) {
    if (dtype == CS_F64) return ntc_launch<double>(s, e, g, off_e, off_g, n_cells, dt, dn, seed, step, stats, st, out);
    return ntc_launch<float>(s, e, g, off_e, off_g, n_cells, dt, dn, seed, step, stats, st, out);
}

hipError_t ntc_prepare_graph(NtcState& s, int64_t n_cells, int64_t cap, int64_t ne, int64_t ng, hipStream_t st) {
    hipError_t err = ntc_reserve(s, n_cells, cap, ne, ng, st);
    if (err == hipSuccess) err = hipStreamSynchronize(st);
    return err;
}

template <typename T>
static hipError_t ntc_capture_t(const NtcState& s, const cs_species& e, const cs_species& g, const int64_t* off_e,
                                const int64_t* off_g, int64_t n_cells, double dt, double dn, uint64_t seed,
                                cs_stats* stats, hipStream_t st) {
    NtcQueue<T> q;
    const hipError_t err = q.start(s, e, g, off_e, off_g, n_cells, dt, dn, seed, 0, true, st, nullptr, nullptr);
    if (err != hipSuccess) return err;
    q.large();
    return q.finish(stats);
}

hipError_t ntc_capture(const NtcState& s, cs_dtype dtype, const cs_species& e, const cs_species& g,
                       const int64_t* off_e, const int64_t* off_g, int64_t n_cells, double dt, double dn,
                       uint64_t seed, cs_stats* stats, hipStream_t st) {
    if (dtype == CS_F64) return ntc_capture_t<double>(s, e, g, off_e, off_g, n_cells, dt, dn, seed, stats, st);
    return ntc_capture_t<float>(s, e, g, off_e, off_g, n_cells, dt, dn, seed, stats, st);
}

__global__ void k_ntc_set_step(NtcHead* head, uint64_t step) {
    if (threadIdx.x == 0 && blockIdx.x == 0) head->step = step;
}

hipError_t ntc_set_step(const NtcState& s, uint64_t step, hipStream_t st) {
    k_ntc_set_step<<<1, 64, 0, st>>>((NtcHead*)s.touch, step);
    return hipGetLastError();
}

}  // namespace cs
