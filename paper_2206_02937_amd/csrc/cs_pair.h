// cs_pair.h -- the per-pair work of a Compton step, shared by every kernel
// strategy (multi-kernel baseline and fused persistent kernel) so that all of
// them compute bitwise-identical results.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cs_device.h"
#include "cs_net.h"

namespace cs {

template <typename T>
struct Particles {
    T *ex, *ey, *ez, *ew;
    T *gx, *gy, *gz, *gw;
};

// The step's control words that every kernel after the scan reads at its
// start (epoch, step counter, layout and scan-fault epochs), all in one
// memory round trip: read one by one, with the layout test's short-circuit
// between two of them, they took several round trips in a row.
struct CtrlView {
    uint32_t epoch;
    uint64_t step;
    bool layout_ok;  // no layout error and no scan time-out in this step
};

__device__ __forceinline__ CtrlView ctrl_view(const StepControl* ctrl) {
    const uint32_t epoch = ctrl->epoch, layout_epoch = ctrl->layout_epoch, fault_epoch = ctrl->scan_fault_epoch;
    const uint64_t step = ctrl->step;
    CtrlView v;
    v.epoch = epoch;
    v.step = step;
    v.layout_ok = (layout_epoch != epoch) & (fault_epoch != epoch);
    return v;
}

struct PairOutcome {
    int32_t ie, ig;  // electron / photon index of the pair
    double x;        // rest-frame photon energy (0 when invalid)
    double P;        // collision probability (0 when invalid)
    bool accept;
    bool clipped;
    bool invalid;
};

__device__ __forceinline__ bool finite_pair(d3 p, double we, d3 k, double wg) {
    return isfinite(p.x) && isfinite(p.y) && isfinite(p.z) && isfinite(k.x) && isfinite(k.y) && isfinite(k.z) &&
           isfinite(we) && isfinite(wg) && we >= 0.0 && wg >= 0.0;
}

// The three phases of a pair's evaluation, split so that a kernel can issue
// the memory accesses of several pairs before it needs any of them:
//   pair_index   pairing (keyed in-cell bijection) -> electron/photon index
//   pair_load    the two particles' momenta and weights (storage type)
//   pair_physics rest-frame photon energy, Klein-Nishina cross-section,
//                probability, accept/reject
// pair_eval runs the three in a row.
struct PairSlot {
    int32_t ie, ig;  // particle indices (0 when inactive)
    uint32_t M;      // larger species count of the cell
    bool active;
};

template <typename T>
struct PairRaw {
    T p[3], k[3], we, wg;
};

// Pair number i of the cell with particle ranges [e0, e1), [g0, g1) and
// pairing key key4.
__device__ __forceinline__ PairSlot pair_index(bool active, int64_t e0, int64_t e1, int64_t g0, int64_t g1,
                                               uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3, uint32_t i) {
    PairSlot s;
    s.ie = 0;
    s.ig = 0;
    s.M = 0;
    s.active = active;
    if (active) {
        const uint32_t ne = (uint32_t)(e1 - e0), ng = (uint32_t)(g1 - g0);
        s.M = ne > ng ? ne : ng;
        FeistelKey key;
        key.k[0] = k0;
        key.k[1] = k1;
        key.k[2] = k2;
        key.k[3] = k3;
        key.bits = ceil_log2(s.M);
        if (ne <= ng) {
            s.ie = (int32_t)(e0 + i);
            s.ig = (int32_t)(g0 + shuffle_index(i, ng, key));
        } else {
            s.ig = (int32_t)(g0 + i);
            s.ie = (int32_t)(e0 + shuffle_index(i, ne, key));
        }
    }
    return s;
}

// s_waitcnt immediate that waits for vmcnt 0 only (gfx9 encoding: vmcnt in
// bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 at their maxima).
constexpr int kWaitVmcnt0 = 0x0F70;

// Read-only data at a wave-uniform index through the constant address space,
// so that the read is one scalar load (the data do not change while the
// kernel runs).
template <typename X>
__device__ __forceinline__ X ld_uniform(const X* p, int64_t i) {
    return ((const __attribute__((address_space(4))) X*)p)[i];
}

// The pairing of a wave of 64 consecutive pairs.  (Args: off_e, off_g,
// pair_off, keys as the scan kernel left them.)

// A cell as the pairing needs it (its ranges start below 2^31).
struct CellMeta {
    int32_t e0, g0;
    uint32_t ne, ng;
    FeistelKey key;
    int32_t po;  // its first pair
};

__device__ __forceinline__ uint32_t larger(const CellMeta& m) { return m.ne > m.ng ? m.ne : m.ng; }

// Cell c's metadata by scalar loads (c wave-uniform).
template <typename Args>
__device__ __forceinline__ CellMeta cell_meta(const Args& a, int c) {
    CellMeta m;
    const int64_t e0 = ld_uniform(a.off_e, c), g0 = ld_uniform(a.off_g, c);
    m.e0 = (int32_t)e0;
    m.g0 = (int32_t)g0;
    m.ne = (uint32_t)(ld_uniform(a.off_e, c + 1) - e0);
    m.ng = (uint32_t)(ld_uniform(a.off_g, c + 1) - g0);
    m.key.k[0] = ld_uniform(a.keys, 4 * (int64_t)c);
    m.key.k[1] = ld_uniform(a.keys, 4 * (int64_t)c + 1);
    m.key.k[2] = ld_uniform(a.keys, 4 * (int64_t)c + 2);
    m.key.k[3] = ld_uniform(a.keys, 4 * (int64_t)c + 3);
    m.key.bits = ceil_log2(larger(m));
    m.po = ld_uniform(a.pair_off, c);
    return m;
}

// b in the lanes with take set, else a.
__device__ __forceinline__ CellMeta pick(bool take, const CellMeta& a, const CellMeta& b) {
    CellMeta m;
    m.e0 = take ? b.e0 : a.e0;
    m.g0 = take ? b.g0 : a.g0;
    m.ne = take ? b.ne : a.ne;
    m.ng = take ? b.ng : a.ng;
#pragma unroll
    for (int r = 0; r < 4; ++r) m.key.k[r] = take ? b.key.k[r] : a.key.k[r];
    m.key.bits = take ? b.key.bits : a.key.bits;
    m.po = take ? b.po : a.po;
    return m;
}

// Pair i of cell m with the larger species' index v.
__device__ __forceinline__ PairSlot slot_of(bool act, const CellMeta& m, uint32_t i, uint32_t v) {
    const bool e_first = m.ne <= m.ng;
    PairSlot s;
    s.M = larger(m);
    s.active = act;
    s.ie = act ? m.e0 + (int32_t)(e_first ? i : v) : 0;
    s.ig = act ? m.g0 + (int32_t)(e_first ? v : i) : 0;
    return s;
}

// The pairing of a wave whose pairs lie in cell a, or (TWO) in the cells a
// and b (in_b: the lane's pair is b's).  The cycle-walk of a lane leaves
// [0, M) for points of [M, 2^b) only: when the wave's cells have at most 64 of
// those together, one lane each evaluates them, and the walk is a chain of
// lane reads instead of passes through the network that the wave repeats
// until its last lane is done (five on average for 64-pair cells: on the uneven
// plasma, whose pair kernel took 84.0 us, the pairing was 32 us of it).
template <bool TWO>
__device__ __forceinline__ PairSlot pair_wave(bool act, uint32_t t, const CellMeta& a, const CellMeta& b, bool in_b) {
    const CellMeta m = TWO ? pick(in_b, a, b) : a;
    const uint32_t M = larger(m);
    const uint32_t i = act ? t - (uint32_t)m.po : 0u;
    uint32_t v = feistel(i, m.key);
    const uint64_t act_m = lanes(act);
    uint64_t out_m = act_m & lanes(v >= M);
    if (out_m) {
        const uint32_t n_a = (1u << a.key.bits) - larger(a), n_b = TWO ? (1u << b.key.bits) - larger(b) : 0u;
        if (n_a + n_b <= 64u && n_a <= 64u) {
            const uint32_t l = (uint32_t)lane_id();
            const bool tab_b = TWO && l >= n_a;
            uint32_t o;
            if (TWO) {
                FeistelKey k;
#pragma unroll
                for (int r = 0; r < 4; ++r) k.k[r] = tab_b ? b.key.k[r] : a.key.k[r];
                k.bits = tab_b ? b.key.bits : a.key.bits;
                o = feistel(tab_b ? larger(b) + (l - n_a) : larger(a) + l, k);
            } else {
                o = feistel(larger(a) + l, a.key);
            }
            // entry of point v: v - M, after a's entries for b
            const uint32_t base = M - (TWO && in_b ? n_a : 0u);
            do {
                const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((v - base) << 2), (int)o);
                v = v >= M ? w : v;  // (an inactive lane's value is not used)
                out_m = act_m & lanes(v >= M);
            } while (out_m);
        } else {
            bool out = act && v >= M;
            while (out) {
                v = feistel(v, m.key);
                out = v >= M;
            }
        }
    }
    return slot_of(act, m, i, v);
}

// The pairing of one lane whose wave's pairs lie in more than two cells, ma
// (cell cs0) to cell ch.
template <typename Args>
__device__ __forceinline__ PairSlot pair_cells(const Args& a, bool act, int32_t t, const CellMeta& ma, int cs0, int ch,
                                               int32_t po_next) {
    const int nc = ch - cs0 + 1;
    CellMeta m = ma;
    if (nc <= 64) {
        // lane l reads cell cs0 + l's metadata (one coalesced round trip);
        // each lane finds its cell among them by a binary search over the
        // wave's pair offsets and takes that cell's values by lane shuffles
        const int cl = cs0 + (lane_id() < nc ? lane_id() : nc - 1);
        const int32_t po_l = a.pair_off[cl];
        const int64_t e0_l = a.off_e[cl], g0_l = a.off_g[cl];
        const int32_t ne_l = (int32_t)(a.off_e[cl + 1] - e0_l), ng_l = (int32_t)(a.off_g[cl + 1] - g0_l);
        const uint4 key_l = *(const uint4*)(a.keys + 4 * (int64_t)cl);
        int lo = 0, hi = nc - 1;
#pragma unroll
        for (int it = 0; it < 6; ++it) {  // nc <= 64 = 2^6
            const int mid = (lo + hi + 1) >> 1;
            if (__shfl(po_l, mid, 64) <= t)
                lo = mid;
            else
                hi = mid - 1;
        }
        // (shuffles by the whole wave)
        m.e0 = __shfl((int32_t)e0_l, lo, 64);
        m.g0 = __shfl((int32_t)g0_l, lo, 64);
        m.ne = (uint32_t)__shfl(ne_l, lo, 64);
        m.ng = (uint32_t)__shfl(ng_l, lo, 64);
        m.key.k[0] = __shfl(key_l.x, lo, 64);
        m.key.k[1] = __shfl(key_l.y, lo, 64);
        m.key.k[2] = __shfl(key_l.z, lo, 64);
        m.key.k[3] = __shfl(key_l.w, lo, 64);
        m.po = __shfl(po_l, lo, 64);
        m.key.bits = ceil_log2(larger(m));
    } else if (act && t >= po_next) {
        // more than 64 cells: a binary search per lane
        int lo = cs0 + 1, hi = ch;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.pair_off[mid] <= t)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int64_t e0 = a.off_e[lo], g0 = a.off_g[lo];
        const uint4 key = *(const uint4*)(a.keys + 4 * (int64_t)lo);
        m.e0 = (int32_t)e0;
        m.g0 = (int32_t)g0;
        m.ne = (uint32_t)(a.off_e[lo + 1] - e0);
        m.ng = (uint32_t)(a.off_g[lo + 1] - g0);
        m.key.k[0] = key.x;
        m.key.k[1] = key.y;
        m.key.k[2] = key.z;
        m.key.k[3] = key.w;
        m.po = a.pair_off[lo];
        m.key.bits = ceil_log2(larger(m));
    }
    // complete these reads inside the branch, so that no read of it is still
    // counted as possibly in flight after it (which would make later waits
    // include the particle reads)
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    const uint32_t i = act ? (uint32_t)(t - m.po) : 0u;
    return slot_of(act, m, i, act ? shuffle_index(i, larger(m), m.key) : 0u);
}

// The wave's pairs t_wave .. t_wave + 63 below T_total, lane by lane; cs0 is
// the cell of the first, ch that of the last or a later one.  They lie in one
// cell, in two, or in more: the metadata of up to two cells come by scalar
// loads (with 64-pair cells 95 % of the waves; one lane per cell and a search
// by lane reads for all that spanned two, before).
template <typename Args>
__device__ __forceinline__ PairSlot pair_slots(const Args& a, int32_t t_wave, int32_t T_total, int cs0, int ch) {
    const int32_t t = t_wave + lane_id();
    const bool act = t < T_total;
    const CellMeta ma = cell_meta(a, cs0);
    const int32_t po_next = ld_uniform(a.pair_off, cs0 + 1);
    const int32_t t_last = t_wave + 63 < T_total ? t_wave + 63 : T_total - 1;
    if (t_last < po_next) return pair_wave<false>(act, (uint32_t)t, ma, ma, false);
    if (ch == cs0 + 1) return pair_wave<true>(act, (uint32_t)t, ma, cell_meta(a, ch), t >= po_next);
    return pair_cells(a, act, t, ma, cs0, ch, po_next);
}

template <typename T>
__device__ __forceinline__ PairRaw<T> pair_load(const Particles<T>& a, const PairSlot& s) {
    PairRaw<T> r;
    if (s.active) {
        r.p[0] = a.ex[s.ie];
        r.p[1] = a.ey[s.ie];
        r.p[2] = a.ez[s.ie];
        r.k[0] = a.gx[s.ig];
        r.k[1] = a.gy[s.ig];
        r.k[2] = a.gz[s.ig];
        r.we = a.ew[s.ie];
        r.wg = a.gw[s.ig];
    } else {
        r.p[0] = r.p[1] = r.p[2] = r.k[0] = r.k[1] = r.k[2] = r.we = r.wg = (T)0;
    }
    return r;
}

// The reads of pair_load issued by every lane: inactive lanes read element 0
// (which exists whenever a pair does; pair_index leaves index 0 in inactive
// slots) and leave the values unused (the physics reads them only for active
// slots), so that the number of reads in flight does not depend on which
// lanes are active and no lane waits for them before they are used.  With
// O32 the byte offsets are formed as unsigned 32-bit values (one multiply
// instead of a 64-bit shift-add per array; the loads take the array base in
// scalar registers), valid while every species has at most 2^32 / sizeof(T)
// elements -- the caller checks that.
template <typename T, bool O32 = false>
__device__ __forceinline__ PairRaw<T> pair_load_all(const Particles<T>& a, const PairSlot& s) {
    PairRaw<T> r;
    if constexpr (O32) {
        uint32_t oe = (uint32_t)s.ie * (uint32_t)sizeof(T), og = (uint32_t)s.ig * (uint32_t)sizeof(T);
        // (opaque here, so that the offsets are not widened before they reach
        // the loads and the bases stay in scalar registers)
        asm("" : "+v"(oe), "+v"(og));
        auto at = [](const T* b, uint32_t o) { return *(const T*)((const char*)b + (uint64_t)o); };
        r.p[0] = at(a.ex, oe);
        r.p[1] = at(a.ey, oe);
        r.p[2] = at(a.ez, oe);
        r.k[0] = at(a.gx, og);
        r.k[1] = at(a.gy, og);
        r.k[2] = at(a.gz, og);
        r.we = at(a.ew, oe);
        r.wg = at(a.gw, og);
    } else {
        r.p[0] = a.ex[s.ie];
        r.p[1] = a.ey[s.ie];
        r.p[2] = a.ez[s.ie];
        r.k[0] = a.gx[s.ig];
        r.k[1] = a.gy[s.ig];
        r.k[2] = a.gz[s.ig];
        r.we = a.ew[s.ie];
        r.wg = a.gw[s.ig];
    }
    return r;
}

// A weight the pair can use: finite and not negative.
__device__ __forceinline__ bool weight_ok(float w) { return __builtin_isfpclass(w, 0x1E0); }
__device__ __forceinline__ bool weight_ok(double w) { return __builtin_isfpclass(w, 0x1E0); }

// `sig_tab`: kSigTab or a copy of it (see sigma_ratio_tab).
//
// Every lane evaluates every step, and what an inactive or invalid lane gets
// is replaced at the end: kept in branches of their own, the steps cost the
// initial values and selects of everything they define (with it the
// pair kernel takes 224 vector instructions per 64 pairs in 256-pair cells, 292
// before).  (1 + p.p) k.k in
// [1e-300, 1e300] implies finite momenta, so one range test per lane stands
// for the six finiteness tests and for x_flux's own; a wave with an active
// lane outside it (or with an unusable weight) takes the general form, whose
// result for the other lanes is the same bit for bit.
template <typename T>
__device__ __forceinline__ PairOutcome pair_physics(const PairSlot& s, const PairRaw<T>& r, double dt,
                                                    double density_norm, uint64_t seed, uint64_t step,
                                                    const double* sig_tab = kSigTab) {
    const d3 p = {(double)r.p[0], (double)r.p[1], (double)r.p[2]};
    const d3 k = {(double)r.k[0], (double)r.k[1], (double)r.k[2]};
    const double pp = dot(p, p), kk = dot(k, k);
    const double a = (1.0 + pp) * kk;
    const uint64_t plain =
        lanes(weight_ok(r.we)) & lanes(weight_ok(r.wg)) & lanes(a >= kFluxNormalMin) & lanes(a <= kFluxNormalMax);
    bool valid = s.active;
    XFlux xf;
    if ((lanes(s.active) & ~plain) == 0) {
        xf = x_flux_impl<true>(p, k, pp, kk);
    } else {
        valid = s.active && finite_pair(p, (double)r.we, k, (double)r.wg);
        xf = valid ? x_flux(p, k, pp, kk) : XFlux{0.0, 0.0};
    }
    const double wmax = (double)(r.we > r.wg ? r.we : r.wg);
    const double tau = dt * density_norm * (double)s.M;
    double P = tau * wmax * sigma_ratio_tab(xf.x, sig_tab) * xf.flux;
    P = valid && xf.x > 0.0 ? P : 0.0;
    PairOutcome o;
    o.ie = s.ie;
    o.ig = s.ig;
    o.x = valid ? xf.x : 0.0;
    o.clipped = P > 1.0;
    o.P = o.clipped ? 1.0 : P;
    o.invalid = s.active && !valid;
    const u32x4 u = draw(seed, (uint64_t)(uint32_t)s.ie, step, kCollide);
    o.accept = uniform53(u.a, u.b) < o.P;  // (P = 0 where the pair is not valid)
    return o;
}

template <typename T>
__device__ __forceinline__ PairOutcome pair_eval(const Particles<T>& a, bool active, int64_t e0, int64_t e1,
                                                 int64_t g0, int64_t g1, const uint32_t* key4, uint32_t i,
                                                 double dt, double density_norm, uint64_t seed, uint64_t step) {
    uint32_t k0 = 0, k1 = 0, k2 = 0, k3 = 0;
    if (active) {
        k0 = key4[0];
        k1 = key4[1];
        k2 = key4[2];
        k3 = key4[3];
    }
    const PairSlot s = pair_index(active, e0, e1, g0, g1, k0, k1, k2, k3, i);
    return pair_physics<T>(s, pair_load<T>(a, s), dt, density_norm, seed, step);
}

struct CollideSums {
    double e_before = 0.0, e_after = 0.0;
    long long n_fallback = 0;  // network samplers: samples the plain sampler answered
};

template <typename T>
__device__ __forceinline__ d3 load_p(const Particles<T>& a, int32_t i) {
    return {(double)a.ex[i], (double)a.ey[i], (double)a.ez[i]};
}
template <typename T>
__device__ __forceinline__ d3 load_k(const Particles<T>& a, int32_t i) {
    return {(double)a.gx[i], (double)a.gy[i], (double)a.gz[i]};
}

// Write back a resolved collision under the weight rule.
template <typename T>
__device__ __forceinline__ void write_back(const Particles<T>& a, int32_t ie, int32_t ig, double we, double wg,
                                           const Scattered& s, uint64_t seed, uint64_t step) {
    bool upd_e = true, upd_g = true;
    if (we != wg) {
        const u32x4 rc = draw(seed, (uint64_t)ie, step, kCollide);
        const double wmin = we < wg ? we : wg, wmx = we < wg ? wg : we;
        const bool heavier_moves = uniform53(rc.c, rc.d) < wmin / wmx;
        if (we > wg)
            upd_e = heavier_moves;
        else
            upd_g = heavier_moves;
    }
    if (upd_e) {
        a.ex[ie] = (T)s.p1.x;
        a.ey[ie] = (T)s.p1.y;
        a.ez[ie] = (T)s.p1.z;
    }
    if (upd_g) {
        a.gx[ig] = (T)s.k1.x;
        a.gy[ig] = (T)s.k1.y;
        a.gz[ig] = (T)s.k1.z;
    }
}

// Resolve the accepted pair (ie, ig) with particle values raw = (p, k, we, wg)
// in their storage type with the plain sampler and write it back.  Lanes
// with active == false run the sampler on a dummy x = 0 (the quickest case)
// and write nothing.
template <typename T>
__device__ __forceinline__ void collide_raw(const Particles<T>& a, bool active, int32_t ie, int32_t ig,
                                            const T (&raw)[8], uint64_t seed, uint64_t step, CollideSums& sums) {
    double x = 0.0;
    if (active) {
        const d3 p = {(double)raw[0], (double)raw[1], (double)raw[2]};
        const d3 k = {(double)raw[3], (double)raw[4], (double)raw[5]};
        x = x_flux(p, k, dot(p, p), dot(k, k)).x;
    }
    const u32x4 r = draw(seed, (uint64_t)ie, step, kScatter);
    const double v = angle_icdf_v(active ? uniform53(r.a, r.b) : 0.5, x);
    if (!active) return;
    const double u_phi = uniform53(r.c, r.d);
    const d3 p = {(double)raw[0], (double)raw[1], (double)raw[2]};
    const d3 k = {(double)raw[3], (double)raw[4], (double)raw[5]};
    const PairInv inv = pair_invariants(p, k);
    const Scattered s = scatter(p, k, inv, v, u_phi);
    write_back<T>(a, ie, ig, (double)raw[6], (double)raw[7], s, seed, step);
    sums.e_before += s.e_before;
    sums.e_after += s.e_after;
}

// The same with the particle values read from the arrays (once, before the
// sampler, kept in their storage type across it: 8 registers for FP32).
template <typename T>
__device__ __forceinline__ void collide_plain(const Particles<T>& a, bool active, int32_t ie, int32_t ig,
                                              uint64_t seed, uint64_t step, CollideSums& sums) {
    T raw[8] = {};
    if (active) {
        raw[0] = a.ex[ie];
        raw[1] = a.ey[ie];
        raw[2] = a.ez[ie];
        raw[3] = a.gx[ig];
        raw[4] = a.gy[ig];
        raw[5] = a.gz[ig];
        raw[6] = a.ew[ie];
        raw[7] = a.gw[ig];
    }
    collide_raw<T>(a, active, ie, ig, raw, seed, step, sums);
}

// An accepted pair kept in global memory between the pair and the collide
// kernels: its indices and the particle values the pair kernel read, in 16-
// byte units (3 for FP32, 5 for FP64), so that the collide kernel reads them
// in a few wide loads instead of gathering eight scattered elements.
template <typename T>
struct alignas(16) StashPair {
    T p[3], we;
    T k[3], wg;
    int32_t ie, ig, pad0, pad1;
};

template <typename T>
__device__ __forceinline__ StashPair<T> make_stash(const PairSlot& s, const PairRaw<T>& r) {
    StashPair<T> e;
    e.p[0] = r.p[0];
    e.p[1] = r.p[1];
    e.p[2] = r.p[2];
    e.we = r.we;
    e.k[0] = r.k[0];
    e.k[1] = r.k[1];
    e.k[2] = r.k[2];
    e.wg = r.wg;
    e.ie = s.ie;
    e.ig = s.ig;
    e.pad0 = 0;
    e.pad1 = 0;
    return e;
}

// collide_raw with the pair taken from a stash entry.
template <typename T>
__device__ __forceinline__ void collide_stash(const Particles<T>& a, bool active, const StashPair<T>* e,
                                              uint64_t seed, uint64_t step, CollideSums& sums) {
    T raw[8] = {};
    int32_t ie = 0, ig = 0;
    if (active) {
        const StashPair<T> v = *e;
        raw[0] = v.p[0];
        raw[1] = v.p[1];
        raw[2] = v.p[2];
        raw[3] = v.k[0];
        raw[4] = v.k[1];
        raw[5] = v.k[2];
        raw[6] = v.we;
        raw[7] = v.wg;
        ie = v.ie;
        ig = v.ig;
    }
    collide_raw<T>(a, active, ie, ig, raw, seed, step, sums);
}

// An accepted pair staged in LDS with its particle values.
template <typename T>
struct alignas(8) StagedPair {
    int32_t ie, ig;
    T p[3], k[3], we, wg;
};

// The same as collide_plain with the particle values taken from LDS.
template <typename T>
__device__ __forceinline__ void collide_staged(const Particles<T>& a, bool active, const StagedPair<T>* e,
                                               uint64_t seed, uint64_t step, CollideSums& sums) {
    double x = 0.0;
    int32_t ie = 0;
    if (active) {
        ie = e->ie;
        const d3 p = {(double)e->p[0], (double)e->p[1], (double)e->p[2]};
        const d3 k = {(double)e->k[0], (double)e->k[1], (double)e->k[2]};
        x = pair_invariants(p, k).x;
    }
    const u32x4 r = draw(seed, (uint64_t)ie, step, kScatter);
    const double v = angle_icdf_v(active ? uniform53(r.a, r.b) : 0.5, x);
    if (!active) return;
    const double u_phi = uniform53(r.c, r.d);
    const d3 p = {(double)e->p[0], (double)e->p[1], (double)e->p[2]};
    const d3 k = {(double)e->k[0], (double)e->k[1], (double)e->k[2]};
    const PairInv inv = pair_invariants(p, k);
    const Scattered s = scatter(p, k, inv, v, u_phi);
    write_back<T>(a, ie, e->ig, (double)e->we, (double)e->wg, s, seed, step);
    sums.e_before += s.e_before;
    sums.e_after += s.e_after;
}

// Where a collision's particle values come from: an LDS queue entry, a stash
// entry or the particle arrays.
template <typename T>
struct FromStaged {
    const StagedPair<T>* e;
    __device__ __forceinline__ void get(const Particles<T>&, int32_t& ie, int32_t& ig, d3& p, d3& k, double& we,
                                        double& wg) const {
        ie = e->ie;
        ig = e->ig;
        p = {(double)e->p[0], (double)e->p[1], (double)e->p[2]};
        k = {(double)e->k[0], (double)e->k[1], (double)e->k[2]};
        we = (double)e->we;
        wg = (double)e->wg;
    }
};
template <typename T>
struct FromStash {
    const StashPair<T>* e;
    __device__ __forceinline__ void get(const Particles<T>&, int32_t& ie, int32_t& ig, d3& p, d3& k, double& we,
                                        double& wg) const {
        const StashPair<T> v = *e;
        ie = v.ie;
        ig = v.ig;
        p = {(double)v.p[0], (double)v.p[1], (double)v.p[2]};
        k = {(double)v.k[0], (double)v.k[1], (double)v.k[2]};
        we = (double)v.we;
        wg = (double)v.wg;
    }
};
template <typename T>
struct FromArrays {
    int32_t ie, ig;
    __device__ __forceinline__ void get(const Particles<T>& a, int32_t& ie_, int32_t& ig_, d3& p, d3& k,
                                        double& we, double& wg) const {
        ie_ = ie;
        ig_ = ig;
        p = load_p(a, ie);
        k = load_k(a, ig);
        we = (double)a.ew[ie];
        wg = (double)a.gw[ig];
    }
};

// Resolve an accepted pair with the sampler network: the network maps the
// FP32-rounded (x, u) to (cos theta, eps'/eps), read as v = 1 - cos theta by
// net_reading_v; outside the network's x range the plain sampler answers
// (counted in n_fallback).  The
// same Philox draw as the plain sampler supplies u and the azimuth.  Must be
// called by the whole wave; lanes with active == false write nothing.
template <typename T, int SAMP, typename Src>
__device__ __forceinline__ void collide_net(const Particles<T>& a, bool active, const Src& src, NetLds<SAMP>& s_net,
                                            const MlpDev& m, uint64_t seed, uint64_t step, CollideSums& sums) {
    // Three phases, so that little is live while the network runs: (1) x and
    // the Philox draw from the pair's values, (2) the network for the wave,
    // (3) the pair's values fetched again (the same source: LDS, a stash entry
    // in cache, or the particle arrays) for the sampler's fallback and the
    // scatter.
    double x = 0.0;
    int32_t ie = 0, ig = 0;
    {
        d3 p = {0.0, 0.0, 0.0}, k = {0.0, 0.0, 0.0};
        double we = 0.0, wg = 0.0;
        if (active) {
            src.get(a, ie, ig, p, k, we, wg);
            x = pair_invariants(p, k).x;
        }
    }
    const u32x4 r = draw(seed, (uint64_t)ie, step, kScatter);
    const double u = uniform53(r.a, r.b);
    const float xf = (float)x, uf = (float)u;
    const bool inside = active && in_range(xf, m.dom);
    const bool fallback = active && !inside;
    float f1 = 0.0f, f2 = 0.0f;
    if (inside) features(xf, uf, m.dom, f1, f2);
    const float2 y = net_outputs<SAMP>(s_net, m, inside, f1, f2);
    double v = 0.0;
    if (__builtin_expect(__any(fallback), 0)) {
        const double vf = angle_icdf_v(fallback ? u : 0.5, fallback ? x : 0.0);
        if (fallback) v = vf;
    }
    if (!active) return;
    if (inside) v = net_reading_v(xf, y.x, y.y);
    d3 p, k;
    double we, wg;
    src.get(a, ie, ig, p, k, we, wg);
    const PairInv inv = pair_invariants(p, k);
    const Scattered s = scatter(p, k, inv, v, uniform53(r.c, r.d));
    write_back<T>(a, ie, ig, we, wg, s, seed, step);
    sums.e_before += s.e_before;
    sums.e_after += s.e_after;
    sums.n_fallback += fallback ? 1 : 0;
}

}  // namespace cs
