// cs_fused.hip -- the step as a scan kernel, a persistent step kernel and a
// finalize kernel.
//
//   k_prep_scan  one pass over the cells: validate offsets, pairs per cell
//                (min(N_e, N_g)), pairing keys, exclusive scan of the pair
//                counts by decoupled look-back, and the first cell of every
//                256-pair chunk (64-pair wave for the compact strategy).
//   k_step       persistent over chunks: each workgroup evaluates `chunks`
//                consecutive 256-pair chunks (pairing, x, s(x), P, accept),
//                each wave appends its accepted pairs to a queue in LDS and
//                drains it densely (all lanes busy) whenever it holds a full
//                wave of pairs, the workgroup what is left at the end;
//                per-workgroup partial sums go to the workspace.
//   k_finalize_step  one workgroup reduces the partial sums in a fixed order
//                into cs_stats and advances the step epoch and device step.
//
// Step-to-step state lives in a small control block of the workspace (epoch,
// done counter, layout flag, device step).  The look-back status words and
// the layout flag carry the epoch of the step that wrote them, so nothing
// needs clearing between steps.
#include <hip/hip_runtime.h>

#include "cs_block.h"
#include "cs_device.h"
#include "cs_internal.h"
#include "cs_lookback.h"
#include "cs_pair.h"

namespace cs {

// ---------------------------------------------------------------------------
// k_prep_scan
// ---------------------------------------------------------------------------
constexpr int kPrepThreads = 256;
constexpr int kPrepPerThread = 1;
constexpr int kPrepCells = kPrepThreads * kPrepPerThread;
// Cell-map entries of one cell: up to kPrepOwn its lane writes one by one, up to
// kPrepLong (and more, where more than kPrepFew cells of a wave have more) four at
// a time; those of a few large cells the whole wave writes, one cell after
// the other.  (581 cells of 15 entries on average: 9.0 us with every cell of
// more than 8 by the wave, 4.6 so; 64 cells of 256: 13.6, 4.9; two cells of 256: 3.1
// by the wave, 4.3 by their lanes.)
constexpr int kPrepOwn = 8, kPrepLong = 32, kPrepFew = 4;

struct PrepArgs {
    const int64_t *off_e, *off_g;
    int64_t n_cells, ne, ng;
    uint64_t seed, step;
    int use_device_step;  // 1: take the step from ctrl (graph replay)
    int32_t* pair_off;    // [n_cells + 1]
    uint32_t* keys;       // [4 n_cells]
    int32_t* cell_map;    // [n_units + 1]: first cell of every `unit` pairs
    int64_t n_units;
    int unit_log2;
    uint64_t* status;     // [n_prep_blocks]
    StepControl* ctrl;
};

__global__ __launch_bounds__(kPrepThreads) void k_prep_scan(const PrepArgs a) {
    __shared__ int s_scan[kPrepThreads / 64 + 1];
    __shared__ int s_prefix;
    // (not ctrl_view: block 0 may write the step word during this kernel)
    const uint32_t E = a.ctrl->epoch;
    const uint64_t step = a.use_device_step ? a.ctrl->step : a.step;
    const int64_t base = (int64_t)blockIdx.x * kPrepCells + (int64_t)threadIdx.x * kPrepPerThread;
    int cnt[kPrepPerThread];
    bool bad = false;
    int tsum = 0;
#pragma unroll
    for (int r = 0; r < kPrepPerThread; ++r) {
        const int64_t c = base + r;
        cnt[r] = 0;
        if (c < a.n_cells) {
            const int64_t a0 = a.off_e[c], a1 = a.off_e[c + 1], b0 = a.off_g[c], b1 = a.off_g[c + 1];
            bool b = a1 < a0 || b1 < b0;
            if (c == 0) b = b || a0 != 0 || b0 != 0;
            if (c == a.n_cells - 1) b = b || a1 != a.ne || b1 != a.ng;
            if (b) {
                bad = true;
            } else {
                const int64_t nmin = (a1 - a0) < (b1 - b0) ? (a1 - a0) : (b1 - b0);
                cnt[r] = (int)nmin;
                if (nmin > 0) {
                    const u32x4 k = draw(a.seed, (uint64_t)c, step, kPair);
                    a.keys[4 * c + 0] = k.a;
                    a.keys[4 * c + 1] = k.b;
                    a.keys[4 * c + 2] = k.c;
                    a.keys[4 * c + 3] = k.d;
                }
            }
        }
        tsum += cnt[r];
    }
    if (bad) atomicMax(&a.ctrl->layout_epoch, E);
    if (blockIdx.x == 0 && threadIdx.x == 0 && !a.use_device_step) a.ctrl->step = a.step;
    int block_total;
    const int tex = block_exclusive_scan(tsum, s_scan, &block_total);
    if (threadIdx.x < 64) {
        const uint32_t ex =
            lookback_exclusive_wave(a.status, blockIdx.x, E, (uint32_t)block_total, &a.ctrl->scan_fault_epoch);
        if (threadIdx.x == 0) s_prefix = (int)ex;
    }
    __syncthreads();
    int run = s_prefix + tex;
#pragma unroll
    for (int r = 0; r < kPrepPerThread; ++r) {
        const int64_t c = base + r;
        if (c < a.n_cells) {
            a.pair_off[c] = run;
        }
        // units whose first pair lies in this cell start here
        const int up = (1 << a.unit_log2) - 1;
        const int64_t u0 = ((int64_t)run + up) >> a.unit_log2, u1 = ((int64_t)run + cnt[r] + up) >> a.unit_log2;
        // (an invalid layout's counts can add up to more than the map holds)
        const int32_t n_map = (int32_t)a.n_units + 1;
        int32_t j0 = u0 < 0 ? 0 : (int32_t)(u0 < n_map ? u0 : n_map);
        const int32_t j1 = u1 < 0 ? 0 : (int32_t)(u1 < n_map ? u1 : n_map);
        const uint64_t longs = __builtin_amdgcn_ballot_w64(j1 - j0 > kPrepLong);
        if (__popcll(longs) <= kPrepFew) {
            for (uint64_t m = longs; m; m &= m - 1) {
                const int l = (int)__ffsll((unsigned long long)m) - 1;
                const int32_t b0 = __builtin_amdgcn_readlane(j0, l), b1 = __builtin_amdgcn_readlane(j1, l);
                const int32_t bc = (int32_t)(base - (int64_t)lane_id() * kPrepPerThread + (int64_t)l * kPrepPerThread + r);
                for (int32_t j = b0 + lane_id(); j < b1; j += 64) a.cell_map[j] = bc;
            }
            if (j1 - j0 > kPrepLong) j0 = j1;
        }
        if (j1 - j0 > kPrepOwn) {
            for (; j0 & 3; ++j0) a.cell_map[j0] = (int32_t)c;
            const int4 c4 = make_int4((int32_t)c, (int32_t)c, (int32_t)c, (int32_t)c);
            for (; j0 + 4 <= j1; j0 += 4) *(int4*)(a.cell_map + j0) = c4;
        }
        for (; j0 < j1; ++j0) a.cell_map[j0] = (int32_t)c;
        run += cnt[r];
    }
    if (blockIdx.x == gridDim.x - 1) {
        // this block's inclusive prefix is the total pair count T
        const int T = s_prefix + block_total;
        if (threadIdx.x == 0) a.pair_off[a.n_cells] = T;
        int64_t jt = ((int64_t)T + (1 << a.unit_log2) - 1) >> a.unit_log2;
        if (jt < 0) jt = 0;  // (the same: T may have wrapped)
        for (int64_t j = jt + threadIdx.x; j <= a.n_units; j += kPrepThreads)
            a.cell_map[j] = (int32_t)(a.n_cells - 1);
    }
}

// ---------------------------------------------------------------------------
// k_step
// ---------------------------------------------------------------------------
constexpr int kWaveCap = 2 * 64;  // a wave's queue: holds < 64 before 64 pairs add at most as many

template <typename T>
struct FusedArgs {
    Particles<T> pt;
    const int64_t *off_e, *off_g;
    int64_t n_cells, n_chunks;
    int chunks_per_block;
    const int32_t* pair_off;
    const uint32_t* keys;
    const int32_t* chunk_cell;
    double dt, density_norm;
    uint64_t seed;
    StepControl* ctrl;
    BlockPartials part;
    cs_stats* stats;
    MlpDev mlp;  // network samplers only
};

// The wave's step over its lanes' staged pairs e (`active` in at least one
// lane): the plain sampler, or the network (every pair of the main stack lies
// in the network's domain).
template <typename T, int SAMP>
__device__ __forceinline__ void drain(const FusedArgs<T>& a, bool active, const StagedPair<T>* e, uint64_t step,
                                      NetLds<SAMP>& s_net, CollideSums& sums) {
    if constexpr (SAMP == CS_SAMPLER_PLAIN)
        collide_staged<T>(a.pt, active, e, a.seed, step, sums);
    else
        collide_net<T, SAMP>(a.pt, active, FromStaged<T>{e}, s_net, a.mlp, a.seed, step, sums);
}

// Network samplers: staged pairs outside the network's domain, with the
// plain sampler.
template <typename T>
__device__ __forceinline__ void drain_fallback(const FusedArgs<T>& a, bool active, const StagedPair<T>* e,
                                               uint64_t step, CollideSums& sums) {
    collide_staged<T>(a.pt, active, e, a.seed, step, sums);
    sums.n_fallback += active ? 1 : 0;
}

// The pairing and the particle reads of the wave's pairs of one chunk, cells
// c_lo (of the chunk's first pair) to c_hi: the first and the last cell of
// the wave's own 64 pairs come from one coalesced read of the chunk's pair
// offsets and two votes.
template <typename T, bool O32>
__device__ __forceinline__ void step_fetch(const FusedArgs<T>& a, int32_t t_wave, int32_t T_total, int c_lo, int c_hi,
                                           PairSlot& sl, PairRaw<T>& raw) {
    sl = PairSlot{0, 0, 0, false};
    if (t_wave < T_total) {  // uniform
        const int nc = c_hi - c_lo + 1;
        if (nc > 1 && nc <= 64) {
            const int l = lane_id() < nc ? lane_id() : nc - 1;
            const int32_t po = a.pair_off[c_lo + l];
            const int32_t t_last = t_wave + 63 < T_total ? t_wave + 63 : T_total - 1;
            const uint64_t in = ~0ull >> (64 - nc);
            c_hi = c_lo + __popcll(lanes(po <= t_last) & in) - 1;
            c_lo += __popcll(lanes(po <= t_wave) & in) - 1;
        }
        sl = pair_slots(a, t_wave, T_total, c_lo, c_hi);
    }
    raw = pair_load_all<T, O32>(a.pt, sl);
}

// Each wave takes its 64 pairs of every chunk and keeps its own queue, so
// that no wave waits for another until the end.  The pairing and the particle
// reads of a chunk are issued before the physics of the one before it, which
// reads nothing from global memory (the s(x) table is in LDS).  Bound by the
// vector instructions of the pairs and of the sampler.  FP32 storage, plain
// sampler, against one queue per workgroup, three barriers per chunk and
// nothing read ahead: 2^22 pairs in 256-pair cells 119.8 -> 63.4 us, in
// 64-pair cells of uneven filling 168 -> 93 us, 2^20 pairs 41.1 -> 24.9 us,
// 2^24 pairs 416 -> 258 us; FP64 storage 142.9 -> 81.6 us at 2^22 pairs; BF16
// network 139 -> 98 us.  With the plain sampler on FP32 storage four waves
// per SIMD are asked for (126 registers; the 143 it takes by itself allow
// three: 76 us where four take 62; five, with spills, 75).
template <typename T, int SAMP, bool O32>
__global__ __launch_bounds__(kChunk, SAMP == CS_SAMPLER_PLAIN && sizeof(T) == 4 ? 4 : 1) void k_step(
    const FusedArgs<T> args) {
    __shared__ double s_sig[kSigTabSegments * kSigTabTerms];
    __shared__ StagedPair<T> s_queue[kChunk / 64][kWaveCap];
    __shared__ NetLds<SAMP> s_net;
    __shared__ int s_left[2][kChunk / 64];
    __shared__ double s_red_d[3 * (kChunk / 64)];
    __shared__ long long s_red_i[4 * (kChunk / 64)];
    constexpr bool NET = SAMP != CS_SAMPLER_PLAIN;
    // The arguments by scalar loads where they are used: `own` makes their
    // address opaque, so that they are not held in scalar registers from one
    // use to the next (there are too few for the sampler's constants as well,
    // and what does not fit is kept in lanes of vector registers).
    const auto own = [] {
        auto p = (const __attribute__((address_space(4))) FusedArgs<T>*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return (const FusedArgs<T>*)p;
    };
    (void)args;  // (the kernel's only argument: at the segment's start)
    const FusedArgs<T>& a = *own();
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = wave_uniform(tid >> 6);
    // The s(x) table, the control words, the pair count and the first chunk's
    // cells are read together, and the table stored to LDS behind them: one
    // after another they are three memory round trips at the start of every
    // workgroup (this kernel at 2^20 pairs: FP32 25.6 -> 24.9 us, FP64 28.3 ->
    // 27.5 us; at 2^22 FP64 82.5 -> 81.6 us; the rest unchanged).
    constexpr int kSigRounds = kSigTabSegments * kSigTabTerms / kChunk;
    static_assert(kSigRounds * kChunk == kSigTabSegments * kSigTabTerms, "whole rounds");
    double sig_v[kSigRounds];
#pragma unroll
    for (int r = 0; r < kSigRounds; ++r) sig_v[r] = kSigTab[tid + r * kChunk];
    const int64_t j_begin = (int64_t)blockIdx.x * a.chunks_per_block;
    const int64_t j_read = j_begin < a.n_chunks ? j_begin : a.n_chunks;  // (n_chunks + 1 entries)
    const int c_first = ld_uniform(a.chunk_cell, j_read);
    int c_next = ld_uniform(a.chunk_cell, j_read < a.n_chunks ? j_read + 1 : j_read);
    StepControl* ctrl = a.ctrl;
    const int32_t T_read = a.pair_off[a.n_cells];
    const CtrlView cv = ctrl_view(ctrl);
    const uint64_t step = cv.step;
    double sum_p = 0.0;
    long long n_clip = 0, n_inv = 0, n_coll = 0;  // wave-uniform
    CollideSums sums;
    net_load<SAMP>(s_net, a.mlp);
#pragma unroll
    for (int r = 0; r < kSigRounds; ++r) s_sig[tid + r * kChunk] = sig_v[r];
    // (no pair at all under a layout error; reads past the map then too)
    const int32_t T_total = cv.layout_ok ? T_read : 0;
    const int64_t n_used = ((int64_t)T_total + kChunk - 1) / kChunk;
    int64_t j_end = j_begin + a.chunks_per_block;
    if (j_end > a.n_chunks) j_end = a.n_chunks;
    if (j_end > n_used) j_end = n_used;
    // two stacks in the wave's queue: from the bottom, and (network samplers,
    // x outside the network's domain) from the top
    StagedPair<T>* queue = s_queue[wave];
    int qn = 0, qf = 0;  // wave-uniform
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    __syncthreads();
    PairSlot sl = {0, 0, 0, false};
    PairRaw<T> raw = {};
    if (j_begin < j_end)
        step_fetch<T, O32>(a, (int32_t)(j_begin * kChunk) + 64 * wave, T_total, c_first, c_next, sl, raw);
    for (int64_t j = j_begin;; ++j) {
        const FusedArgs<T>& a = *own();
        const bool last = j >= j_end;  // uniform over the block
        // the entries to resolve now: n_main of the main stack (lane q's at
        // e_main), n_fb of the other (the waves' leftovers in the last round)
        const StagedPair<T>*e_main = queue, *e_fb = queue;
        uint64_t main_m = 0, fb_m = 0;  // lanes with an entry
        if (!last) {
            const PairSlot s = sl;
            const PairRaw<T> r = raw;
            if (j + 1 < j_end) {
                const int c_lo = c_next;
                c_next = ld_uniform(a.chunk_cell, j + 2);
                step_fetch<T, O32>(a, (int32_t)((j + 1) * kChunk) + 64 * wave, T_total, c_lo, c_next, sl, raw);
            }
            const PairOutcome o = pair_physics<T>(s, r, a.dt, a.density_norm, a.seed, step, s_sig);
            sum_p += o.P;
            n_clip += __popcll(lanes(o.clipped));
            n_inv += __popcll(lanes(o.invalid));
            bool to_fb = false;
            if constexpr (NET) to_fb = o.accept && !in_range((float)o.x, a.mlp.dom);
            const uint64_t acc = lanes(o.accept), mask_fb = NET ? lanes(to_fb) : 0, mask = acc & ~mask_fb;
            n_coll += __popcll(acc);
            if (o.accept) {
                StagedPair<T>& e = to_fb ? queue[kWaveCap - 1 - (qf + __popcll(mask_fb & lanes_below))]
                                         : queue[qn + __popcll(mask & lanes_below)];
                e.ie = s.ie;
                e.ig = s.ig;
                e.p[0] = r.p[0];
                e.p[1] = r.p[1];
                e.p[2] = r.p[2];
                e.k[0] = r.k[0];
                e.k[1] = r.k[1];
                e.k[2] = r.k[2];
                e.we = r.we;
                e.wg = r.wg;
            }
            qn += __popcll(mask);
            qf += __popcll(mask_fb);
            if (qn + qf < 64) continue;
            // both stacks hold < 64 entries together before 64 pairs add at
            // most 64, so they never meet; a stack of 64 or more gives its top
            // 64, and where neither has as many both give all they have
            if (qn >= 64 || qf < 64) {
                const int n = qn < 64 ? qn : 64;
                qn -= n;
                main_m = n > 0 ? ~0ull >> (64 - n) : 0;
                e_main = queue + qn + (lane < n ? lane : 0);
            }
            if (NET && qf > 0 && (qf >= 64 || qn == 0)) {
                const int n = qf < 64 ? qf : 64;
                qf -= n;
                fb_m = ~0ull >> (64 - n);
                e_fb = queue + (kWaveCap - 1 - qf - (lane < n ? lane : 0));
            }
            wave_lds_sync();
        } else {
            // what the waves have left (fewer than 64 each), together: lane q
            // of the workgroup takes entry q
            if (lane == 0) {
                s_left[0][wave] = qn;
                s_left[1][wave] = qf;
            }
            __syncthreads();
            int w = 0, q = tid, w_fb = 0, q_fb = tid;
#pragma unroll
            for (int i = 0; i < kChunk / 64 - 1; ++i) {
                const int l = s_left[0][i], l_fb = s_left[1][i];
                if (w == i && q >= l) ++w, q -= l;
                if (w_fb == i && q_fb >= l_fb) ++w_fb, q_fb -= l_fb;
            }
            const bool in = q < s_left[0][w], in_fb = q_fb < s_left[1][w_fb];
            main_m = lanes(in);
            fb_m = lanes(in_fb);
            e_main = &s_queue[w][in ? q : 0];
            e_fb = &s_queue[w_fb][kWaveCap - 1 - (in_fb ? q_fb : 0)];
        }
        const FusedArgs<T>& ad = *own();
        if (main_m) drain<T, SAMP>(ad, main_m >> lane & 1, e_main, step, s_net, sums);
        if constexpr (NET)
            if (fb_m) drain_fallback<T>(ad, fb_m >> lane & 1, e_fb, step, sums);
        if (last) break;
        wave_lds_sync();
    }
    // per-workgroup partials, fixed order: lanes (butterfly), then waves
    const double w_p = wave_sum(sum_p), w_eb = wave_sum(sums.e_before), w_ea = wave_sum(sums.e_after);
    const long long w_fb = NET ? wave_sum_i(sums.n_fallback) : 0;
    if (lane == 0) {
        s_red_d[3 * wave + 0] = w_p;
        s_red_d[3 * wave + 1] = w_eb;
        s_red_d[3 * wave + 2] = w_ea;
        s_red_i[4 * wave + 0] = n_clip;
        s_red_i[4 * wave + 1] = n_inv;
        s_red_i[4 * wave + 2] = n_coll;
        s_red_i[4 * wave + 3] = w_fb;
    }
    __syncthreads();
    if (tid == 0) {
        double p = 0.0, eb = 0.0, ea = 0.0;
        long long cl = 0, in = 0, co = 0, fb = 0;
        for (int w = 0; w < kChunk / 64; ++w) {
            p += s_red_d[3 * w + 0];
            eb += s_red_d[3 * w + 1];
            ea += s_red_d[3 * w + 2];
            cl += s_red_i[4 * w + 0];
            in += s_red_i[4 * w + 1];
            co += s_red_i[4 * w + 2];
            fb += s_red_i[4 * w + 3];
        }
        const int b = blockIdx.x;
        a.part.prob[b] = p;
        a.part.e_before[b] = eb;
        a.part.e_after[b] = ea;
        a.part.clipped[b] = cl;
        a.part.invalid[b] = in;
        a.part.collided[b] = co;
        a.part.fallback[b] = fb;
    }
}

// ---------------------------------------------------------------------------
// k_finalize_step: one workgroup reduces the per-unit partial sums in a fixed
// order (thread stride, then lanes, then waves), writes cs_stats and advances
// the epoch and the device step counter.  Small on purpose: one accumulator
// per quantity keeps everything in registers.
// ---------------------------------------------------------------------------
constexpr int kFinalThreads = 256;

__global__ __launch_bounds__(kFinalThreads) void k_finalize_step(const FinalArgs a) {
    __shared__ double s_d[3][kFinalThreads / 64];
    __shared__ long long s_i[4][kFinalThreads / 64];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    StepControl* ctrl = a.ctrl;
    const CtrlView cv = ctrl_view(ctrl);
    const uint32_t E = cv.epoch;
    const uint64_t step = cv.step;
    const int32_t np_read = a.pair_off[a.n_cells];  // (allocated for n_cells = 0 too)
    const int32_t n_pairs_raw = a.n_cells > 0 ? np_read : 0;
    const uint32_t n_acc_raw = ctrl->n_accepted;
    double sp = 0.0, eb = 0.0, ea = 0.0;
    long long cl = 0, in = 0, co = 0, fb = 0;
    // both partial sets in one pass, four entries of each per thread at a
    // time, every read of a batch issued before its sums (entries past an
    // array's end read as zeros, which leaves the sums unchanged: each thread
    // still adds its entries of an array in increasing order)
    const int64_t n_ab = a.n_a > a.n_b ? a.n_a : a.n_b;
    for (int64_t base = tid; base < n_ab; base += 4 * kFinalThreads) {
        double vp[4], ve[4], va[4];
        long long vc[4], vi[4], vo[4], vf[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + (int64_t)k * kFinalThreads;
            const bool ia = i < a.n_a, ib = i < a.n_b;
            vp[k] = ia ? a.a_prob[i] : 0.0;
            vc[k] = ia ? a.a_clip[i] : 0;
            vi[k] = ia ? a.a_inv[i] : 0;
            vo[k] = ia && a.a_coll ? a.a_coll[i] : 0;
            ve[k] = ib ? a.b_eb[i] : 0.0;
            va[k] = ib ? a.b_ea[i] : 0.0;
            vf[k] = ib && a.b_fb ? a.b_fb[i] : 0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sp += vp[k];
            cl += vc[k];
            in += vi[k];
            co += vo[k];
            eb += ve[k];
            ea += va[k];
            fb += vf[k];
        }
    }
    const bool layout_ok = cv.layout_ok;
    sp = wave_sum(sp);
    eb = wave_sum(eb);
    ea = wave_sum(ea);
    cl = wave_sum_i(cl);
    in = wave_sum_i(in);
    co = wave_sum_i(co);
    fb = wave_sum_i(fb);
    if (lane == 0) {
        s_d[0][wave] = sp;
        s_d[1][wave] = eb;
        s_d[2][wave] = ea;
        s_i[0][wave] = cl;
        s_i[1][wave] = in;
        s_i[2][wave] = co;
        s_i[3][wave] = fb;
    }
    __syncthreads();
    if (tid == 0) {
        cs_stats s = {};
        for (int w = 0; w < kFinalThreads / 64; ++w) {
            s.sum_prob += s_d[0][w];
            s.energy_before += s_d[1][w];
            s.energy_after += s_d[2][w];
            s.n_clipped += s_i[0][w];
            s.n_invalid += s_i[1][w];
            s.n_collided += s_i[2][w];
            s.n_fallback += s_i[3][w];
        }
        if (!a.a_coll) s.n_collided = (int64_t)n_acc_raw;
        s.n_pairs = n_pairs_raw;
        if (!layout_ok) {
            // no particle was touched: report the layout error only
            s = cs_stats{};
            s.layout_error = 1;
        }
        if (a.stats) *a.stats = s;
        ctrl->n_accepted = 0;
        ctrl->step = step + 1;
        ctrl->epoch = E + 1;
    }
}

hipError_t launch_finalize(const FinalArgs& f, hipStream_t st) {
    k_finalize_step<<<1, kFinalThreads, 0, st>>>(f);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// workspace and launcher
// ---------------------------------------------------------------------------
int64_t fused_prep_blocks(int64_t n_cells) { return (n_cells + kPrepCells - 1) / kPrepCells; }

static size_t al(size_t v) { return (v + 255) & ~(size_t)255; }

// Entries of each partial-sum array: the workgroups, and room for 16 chunks
// each at least (what a step needs of a bounded workspace does not depend on
// the split).
static int64_t fused_part_len(const StepShape& s) {
    const int64_t n = (s.n_chunks + 15) / 16;
    return s.n_step_blocks > n ? s.n_step_blocks : n;
}

size_t fused_workspace_bytes(const StepShape& s) {
    size_t b = 0;
    b += al(sizeof(int32_t) * (s.n_cells + 1));
    b += al(sizeof(uint32_t) * 4 * (s.n_cells > 0 ? s.n_cells : 1));
    b += al(sizeof(int32_t) * (s.n_chunks + 1));
    b += 7 * al(8 * fused_part_len(s));
    return b;
}

void carve_fused_buffers(const Workspace& w, const StepShape& s, FusedBuffers* b) {
    b->ctrl = ws_control(w);
    b->status = ws_status(w);
    char* p = (char*)ws_step_area(w);
    auto take = [&](size_t n) {
        char* r = p;
        p += al(n);
        return (void*)r;
    };
    b->pair_off = (int32_t*)take(sizeof(int32_t) * (s.n_cells + 1));
    b->cell_keys = (uint32_t*)take(sizeof(uint32_t) * 4 * (s.n_cells > 0 ? s.n_cells : 1));
    b->chunk_cell = (int32_t*)take(sizeof(int32_t) * (s.n_chunks + 1));
    b->part.prob = (double*)take(8 * fused_part_len(s));
    b->part.e_before = (double*)take(8 * fused_part_len(s));
    b->part.e_after = (double*)take(8 * fused_part_len(s));
    b->part.clipped = (int64_t*)take(8 * fused_part_len(s));
    b->part.invalid = (int64_t*)take(8 * fused_part_len(s));
    b->part.collided = (int64_t*)take(8 * fused_part_len(s));
    b->part.fallback = (int64_t*)take(8 * fused_part_len(s));
}

hipError_t launch_prep(const StepShape& sh, StepControl* ctrl, uint64_t* status, int32_t* pair_off, uint32_t* keys,
                       int32_t* cell_map, int unit, const StepParams& p, hipStream_t st) {
    if (sh.n_cells <= 0) return hipSuccess;
    PrepArgs pa;
    pa.off_e = p.off_e;
    pa.off_g = p.off_g;
    pa.n_cells = sh.n_cells;
    pa.ne = sh.ne;
    pa.ng = sh.ng;
    pa.n_units = sh.n_chunks * (kChunk / unit);
    pa.unit_log2 = __builtin_ctz((unsigned)unit);
    pa.seed = p.seed;
    pa.step = p.step;
    pa.use_device_step = p.use_device_step;
    pa.pair_off = pair_off;
    pa.keys = keys;
    pa.cell_map = cell_map;
    pa.status = status;
    pa.ctrl = ctrl;
    k_prep_scan<<<(unsigned)fused_prep_blocks(sh.n_cells), kPrepThreads, 0, st>>>(pa);
    return hipGetLastError();
}

Resident resident_of(ResidentCache& cache, const void* kernel, int threads) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return {0, 0};
    return cache.get(dev, [&]() -> Resident {
        int n_cu = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess)
            return {0, 0};
        return {per_cu, n_cu};
    });
}

// Workgroups of k_step<T, SAMP, true> resident at once on the current device,
// at most kFusedMaxBlocks (what the partial sums of a small step have room
// for).
constexpr int64_t kFusedMaxBlocks = 1024;

template <typename T, int SAMP>
static int64_t step_resident_blocks() {
    static ResidentCache cache;
    const Resident r = resident_of(cache, reinterpret_cast<const void*>(&k_step<T, SAMP, true>), kChunk);
    const int64_t n = r.per_cu * r.cus;
    return n <= 0 ? 512 : (n < kFusedMaxBlocks ? n : kFusedMaxBlocks);
}

template <typename T>
static int64_t step_resident_blocks(cs_sampler sampler) {
    switch (sampler) {
        case CS_SAMPLER_MLP_F32:
            return step_resident_blocks<T, CS_SAMPLER_MLP_F32>();
        case CS_SAMPLER_MLP_BF16:
            return step_resident_blocks<T, CS_SAMPLER_MLP_BF16>();
        case CS_SAMPLER_MLP_FP8:
            return step_resident_blocks<T, CS_SAMPLER_MLP_FP8>();
        default:
            return step_resident_blocks<T, CS_SAMPLER_PLAIN>();
    }
}

// One round of resident workgroups, at most 32 chunks each.  Plain sampler,
// FP32 storage (1024 resident): 4096 chunks take 26.1 us at 4 each and 29.5 at
// 8; 16384 chunks 62.2 at 16, 68.4 at 8, 73.7 at 24.  Beyond 32 the rounds
// stop counting (65536 chunks: 266 us at 16, 255 at 32, 251 at 64).
int64_t fused_fit_chunks(cs_dtype dtype, cs_sampler sampler, int64_t n_chunks) {
    const int64_t r = dtype == CS_F64 ? step_resident_blocks<double>(sampler) : step_resident_blocks<float>(sampler);
    int64_t g = (n_chunks + r - 1) / r;
    if (g > 32) g = 32;
    return g < 1 ? 1 : g;
}

template <typename T, int SAMP>
static hipError_t launch_fused_t(const StepShape& sh, const FusedBuffers& b, const StepParams& p, hipStream_t st) {
    auto mark = [&](int i) {
        if (p.events) (void)hipEventRecord(p.events[i], st);
    };
    mark(0);
    hipError_t e = launch_prep(sh, b.ctrl, b.status, b.pair_off, b.cell_keys, b.chunk_cell, kChunk, p, st);
    if (e != hipSuccess) return e;
    mark(1);
    FusedArgs<T> fa;
    fa.pt = {(T*)p.e.x, (T*)p.e.y, (T*)p.e.z, (T*)p.e.w, (T*)p.g.x, (T*)p.g.y, (T*)p.g.z, (T*)p.g.w};
    fa.off_e = p.off_e;
    fa.off_g = p.off_g;
    fa.n_cells = sh.n_cells;
    fa.n_chunks = sh.n_chunks;
    fa.chunks_per_block = sh.chunks_per_block;
    fa.pair_off = b.pair_off;
    fa.keys = b.cell_keys;
    fa.chunk_cell = b.chunk_cell;
    fa.dt = p.dt;
    fa.density_norm = p.density_norm;
    fa.seed = p.seed;
    fa.ctrl = b.ctrl;
    fa.part = b.part;
    fa.stats = p.stats;
    fa.mlp = p.net;
    // 32-bit byte offsets whenever both species fit them (see pair_load_all)
    constexpr int64_t kO32Max = ((int64_t)1 << 32) / (int64_t)sizeof(T);
    if (!p.wide_index && sh.ne <= kO32Max && sh.ng <= kO32Max)
        k_step<T, SAMP, true><<<(unsigned)sh.n_step_blocks, kChunk, 0, st>>>(fa);
    else
        k_step<T, SAMP, false><<<(unsigned)sh.n_step_blocks, kChunk, 0, st>>>(fa);
    mark(2);
    mark(3);
    mark(4);
    FinalArgs f = {};
    f.ctrl = b.ctrl;
    f.pair_off = b.pair_off;
    f.n_cells = sh.n_cells;
    f.a_prob = b.part.prob;
    f.a_clip = b.part.clipped;
    f.a_inv = b.part.invalid;
    f.a_coll = b.part.collided;
    f.n_a = sh.n_step_blocks;
    f.b_eb = b.part.e_before;
    f.b_ea = b.part.e_after;
    f.b_fb = b.part.fallback;
    f.n_b = sh.n_step_blocks;
    f.stats = p.stats;
    e = launch_finalize(f, st);
    mark(5);
    return e == hipSuccess ? hipGetLastError() : e;
}

template <typename T>
static hipError_t launch_fused_s(const StepShape& sh, const FusedBuffers& b, const StepParams& p, hipStream_t st) {
    switch (p.sampler) {
        case CS_SAMPLER_MLP_F32:
            return launch_fused_t<T, CS_SAMPLER_MLP_F32>(sh, b, p, st);
        case CS_SAMPLER_MLP_BF16:
            return launch_fused_t<T, CS_SAMPLER_MLP_BF16>(sh, b, p, st);
        case CS_SAMPLER_MLP_FP8:
            return launch_fused_t<T, CS_SAMPLER_MLP_FP8>(sh, b, p, st);
        default:
            return launch_fused_t<T, CS_SAMPLER_PLAIN>(sh, b, p, st);
    }
}

hipError_t launch_fused(const StepShape& sh, const FusedBuffers& b, const StepParams& p, hipStream_t st) {
    if (p.dtype == CS_F64) return launch_fused_s<double>(sh, b, p, st);
    return launch_fused_s<float>(sh, b, p, st);
}

// ---------------------------------------------------------------------------
// k_cell_baseline: the straightforward mapping, one workgroup per cell
// walking its pairs 256 at a time and resolving each accepted pair in the
// lane that found it (no compaction, so the sampler runs on mostly idle
// waves).  A baseline for the batched strategies; same per-pair code, so the
// same results.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kChunk) void k_cell_baseline(const FusedArgs<T> a) {
    __shared__ double s_red_d[3 * (kChunk / 64)];
    __shared__ long long s_red_i[3 * (kChunk / 64)];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    const int64_t c = blockIdx.x;
    StepControl* ctrl = a.ctrl;
    const CtrlView cv = ctrl_view(ctrl);
    const uint64_t step = cv.step;
    const bool layout_ok = cv.layout_ok;
    double sum_p = 0.0;
    long long n_clip = 0, n_inv = 0, n_coll = 0;
    CollideSums sums;
    if (layout_ok && c < a.n_cells) {
        const int32_t np = a.pair_off[c + 1] - a.pair_off[c];
        const int64_t e0 = a.off_e[c], e1 = a.off_e[c + 1], g0 = a.off_g[c], g1 = a.off_g[c + 1];
        for (int32_t base = 0; base < np; base += kChunk) {
            const int32_t i = base + tid;
            const bool active = i < np;
            const PairOutcome o = pair_eval<T>(a.pt, active, e0, e1, g0, g1, a.keys + 4 * c, (uint32_t)(active ? i : 0),
                                               a.dt, a.density_norm, a.seed, step);
            sum_p += o.P;
            n_clip += o.clipped ? 1 : 0;
            n_inv += o.invalid ? 1 : 0;
            n_coll += o.accept ? 1 : 0;
            collide_plain<T>(a.pt, o.accept, o.ie, o.ig, a.seed, step, sums);
        }
    }
    const double w_p = wave_sum(sum_p), w_eb = wave_sum(sums.e_before), w_ea = wave_sum(sums.e_after);
    const long long w_cl = wave_sum_i(n_clip), w_in = wave_sum_i(n_inv), w_co = wave_sum_i(n_coll);
    if (lane == 0) {
        s_red_d[3 * wave + 0] = w_p;
        s_red_d[3 * wave + 1] = w_eb;
        s_red_d[3 * wave + 2] = w_ea;
        s_red_i[3 * wave + 0] = w_cl;
        s_red_i[3 * wave + 1] = w_in;
        s_red_i[3 * wave + 2] = w_co;
    }
    __syncthreads();
    if (tid == 0) {
        double p = 0.0, eb = 0.0, ea = 0.0;
        long long cl = 0, in = 0, co = 0;
        for (int w = 0; w < kChunk / 64; ++w) {
            p += s_red_d[3 * w + 0];
            eb += s_red_d[3 * w + 1];
            ea += s_red_d[3 * w + 2];
            cl += s_red_i[3 * w + 0];
            in += s_red_i[3 * w + 1];
            co += s_red_i[3 * w + 2];
        }
        const int64_t b = blockIdx.x;
        a.part.prob[b] = p;
        a.part.e_before[b] = eb;
        a.part.e_after[b] = ea;
        a.part.clipped[b] = cl;
        a.part.invalid[b] = in;
        a.part.collided[b] = co;
        a.part.fallback[b] = 0;
    }
}

template <typename T>
static hipError_t launch_cell_t(const StepShape& sh, const FusedBuffers& b, const StepParams& p, hipStream_t st) {
    auto mark = [&](int i) {
        if (p.events) (void)hipEventRecord(p.events[i], st);
    };
    mark(0);
    hipError_t e = launch_prep(sh, b.ctrl, b.status, b.pair_off, b.cell_keys, b.chunk_cell, kChunk, p, st);
    if (e != hipSuccess) return e;
    mark(1);
    FusedArgs<T> fa = {};
    fa.pt = {(T*)p.e.x, (T*)p.e.y, (T*)p.e.z, (T*)p.e.w, (T*)p.g.x, (T*)p.g.y, (T*)p.g.z, (T*)p.g.w};
    fa.off_e = p.off_e;
    fa.off_g = p.off_g;
    fa.n_cells = sh.n_cells;
    fa.n_chunks = sh.n_chunks;
    fa.chunks_per_block = 1;
    fa.pair_off = b.pair_off;
    fa.keys = b.cell_keys;
    fa.chunk_cell = b.chunk_cell;
    fa.dt = p.dt;
    fa.density_norm = p.density_norm;
    fa.seed = p.seed;
    fa.ctrl = b.ctrl;
    fa.part = b.part;
    fa.stats = p.stats;
    if (sh.n_cells > 0) k_cell_baseline<T><<<(unsigned)sh.n_cells, kChunk, 0, st>>>(fa);
    mark(2);
    mark(3);
    mark(4);
    FinalArgs f = {};
    f.ctrl = b.ctrl;
    f.pair_off = b.pair_off;
    f.n_cells = sh.n_cells;
    f.a_prob = b.part.prob;
    f.a_clip = b.part.clipped;
    f.a_inv = b.part.invalid;
    f.a_coll = b.part.collided;
    f.n_a = sh.n_cells > 0 ? sh.n_cells : 0;
    f.b_eb = b.part.e_before;
    f.b_ea = b.part.e_after;
    f.b_fb = b.part.fallback;
    f.n_b = f.n_a;
    f.stats = p.stats;
    e = launch_finalize(f, st);
    mark(5);
    return e == hipSuccess ? hipGetLastError() : e;
}

hipError_t launch_cell(const StepShape& sh, const FusedBuffers& b, const StepParams& p, hipStream_t st) {
    if (p.dtype == CS_F64) return launch_cell_t<double>(sh, b, p, st);
    return launch_cell_t<float>(sh, b, p, st);
}

}  // namespace cs
