// tas_sim.hip - the iteration-level serving simulation, one wavefront per
// instance (one trace x one policy setting), for gfx950.
//
// What each iteration computes (arXiv 2606.18431, Algorithm 1; Phase 2
// unified key and hysteresis; Phase 3 MemGuard; Phase 4 adaptive gamma):
//   0. with adaptive gamma, gamma follows the tail of the recent end-to-end
//      latencies, and the boost table that of its nearest grid point;
//   1. arrivals with a_i <= t join the waiting set;
//   2. every waiting or resident request has a key; candidates are taken in
//      ascending (key, idx) order;
//   3. greedy batch formation under max_seqs, max_tokens and the KV budget;
//      when the KV budget is exceeded the worst eligible resident outside the
//      batch is evicted (recompute preemption); a resident candidate with no
//      eligible victim forces out the worst other resident or itself; a
//      waiting candidate that does not fit closes admissions;
//   4. the step costs base + tok*sum(n) + floor(sum(kv+n)/div) us; tokens are
//      emitted, first/last token times and the max inter-token gap recorded.
//
// Design (MI355X): instances are independent, so one 64-lane wavefront owns
// one instance and needs no workgroup barrier. The active requests live in
// LDS as one array sorted by the packed key (key + 2^42) << 21 | idx, with
// their state in structure-of-arrays form, so the batch-formation pass is a
// sequence of 64-wide chunks with DPP prefix sums (token budget, KV blocks,
// sequence count) and a ballot to find the first candidate that does not
// fit; only that candidate takes the sequential eviction path. Keys of
// waiting requests never change (MemGuard recomputes a key only when the
// quantized signal moves, Phase 3), so the list is repaired incrementally:
// finished entries stay behind as holes until a compaction pass, entries whose
// key moved are extracted and merged back. Waiting requests beyond the
// on-chip capacity spill to HBM with the invariant that every spilled key
// exceeds every waiting key on chip; a radix select over the spill refills
// the list.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tas_internal.h"

namespace tas {
namespace {

#define DEV __device__ __forceinline__

// The checking build (a library of its own, compiled with
// TAS_CHECK_INVARIANTS=1) verifies the batch of every iteration that is
// formed, the members of every run of repeated iterations before it is
// applied, and the state of every instance after each step (an iteration, or
// the runs up to the next event). It fails the instance with S_ESTATE at the
// first violation; its results are otherwise those of the ordinary build.
#ifndef TAS_CHECK_INVARIANTS
#define TAS_CHECK_INVARIANTS 0
#endif
constexpr bool kCheck = TAS_CHECK_INVARIANTS != 0;
#define UNLIKELY(x) __builtin_expect(!!(x), 0)
#define LIKELY(x) __builtin_expect(!!(x), 1)

// record flag word (gs)
constexpr uint32_t G_GUARD = 0x1fu;      // MemGuard level at the latest dispatch
constexpr uint32_t G_RES = 1u << 5;      // resident: holds KV
constexpr uint32_t G_FIRST = 1u << 6;    // first token emitted
constexpr uint32_t G_INB = 1u << 7;      // in this iteration's batch
constexpr uint32_t G_EVI = 1u << 8;      // evicted during this iteration
constexpr uint32_t G_DONE = 1u << 9;     // completed: a hole until compaction
constexpr uint32_t G_DIRTY = 1u << 10;   // key moved: re-insert
constexpr uint32_t G_MARK = 1u << 11;    // selected for spilling
constexpr int G_LVL_SHIFT = 12;          // current MemGuard level (5 bits)
constexpr uint32_t G_LVL = 0x1fu << G_LVL_SHIFT;
constexpr uint32_t G_FLAGS = 0x1ffffu;   // the flags and levels: bits 0..16
constexpr int kLeftShift = 17;           // compact slots: left - 1 in bits 17..31
// LTR+ (which has no MemGuard level, and never uses compact slots): the
// level's lowest bit marks a promoted request, bits 17..31 hold its
// starvation count, or while promoted the quantum left
constexpr uint32_t G_PROMO = 1u << G_LVL_SHIFT;
constexpr int kLtrShift = 17;
constexpr int kHoleLimit = 16;           // compact once this many holes accumulate

enum { S_OK = 0, S_EOVERFLOW = -5, S_ELIVELOCK = -6, S_ESTATE = -7, S_ECAPACITY = -8 };
// Policies: the paper's boosted priority (BOOST), its comparators FCFS and
// oracle-length SRPT, and the further comparison policies of its Table 1 and
// evaluation baselines: shortest prompt first (SPF), shortest job first with
// perfect output-length knowledge (SJF), least attained service (LAS) and
// SRPT with TRAIL's swap-prevention threshold (TRAIL); and the Phase 1
// strawman DistBoost (DIST).
enum { P_FCFS = 0, P_SRPT = 1, P_BOOST = 2, P_SPF = 3, P_SJF = 4, P_LAS = 5, P_TRAIL = 6,
       P_DIST = 7, P_SARATHI = 8, P_LTR = 9 };
// LTR+ ranks a promoted request ahead of every unpromoted one (SJF keys are
// D >= 1): key j - 2^42 for a promotion at the end of iteration j.
constexpr int64_t kPromotedOff = int64_t(1) << 42;
// DistBoost ranks its decode queue (key: the time a request entered it, its
// first-token time) ahead of its prefill queue: decode keys are shifted down
// by 2^42, below every prefill key a - bt (boost tables are capped at 2^40).
constexpr int64_t kDecodeQueueOff = int64_t(1) << 42;

// ------------------------------------------------------------ wave helpers

DEV int lane() { return (int)__lane_id(); }
DEV uint64_t ballot(bool p) { return (uint64_t)__ballot(p); }
DEV int popc(uint64_t m) { return __popcll(m); }
DEV int ffs0(uint64_t m) { return __ffsll((unsigned long long)m) - 1; }
DEV int fls0(uint64_t m) { return 63 - __clzll((unsigned long long)m); }
DEV int mbcnt(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
DEV int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
DEV int rl(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
DEV uint64_t rlu(uint64_t x, int l) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
DEV int64_t rl64(int64_t x, int l) { return (int64_t)rlu((uint64_t)x, l); }
DEV uint64_t uniu(uint64_t x) { return rlu(x, __builtin_amdgcn_readfirstlane(lane())); }
// A wave-uniform 64-bit value in scalar registers: 64-bit comparisons, and the
// selects on them, have no scalar form, and a value that came out of one would
// otherwise stay in vector registers around the whole loop.
DEV uint64_t sgpr64(uint64_t x) {
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)x), hi = (uint32_t)uni((int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}
// A wave-uniform value kept in a vector register: state and constants that a
// step uses once or twice. Scalar registers are what the simulator runs out
// of, and a spilled scalar costs a lane write and a lane read where the
// compiler chooses; most builds have vector registers to spare at the
// occupancy the LDS allows (see sim_kernel). `v` serves lane arithmetic as it
// is, the conversion gives the scalar.
template <typename T_>
struct Held {
    T_ v;
    DEV Held &operator=(T_ x) {
        v = x;
        __asm__("" : "+v"(v));
        return *this;
    }
    DEV operator T_() const {
        if constexpr (sizeof(T_) == 8) return (T_)sgpr64((uint64_t)v);
        else return (T_)uni((int)v);
    }
};
// x with lane LANE set to the wave-uniform v. The intrinsic, not inline
// assembly: v is often reloaded by a lane read just before, a vector
// instruction may read that scalar only two wait states later, and the
// compiler inserts them for instructions it knows, not inside assembly text.
__device__ int llvm_writelane(int v, int l, int x) __asm("llvm.amdgcn.writelane.i32");
template <int LANE>
DEV int set_lane(int x, int v) {
    return llvm_writelane(uni(v), LANE, x);
}
// x < y for wave-uniform values whose difference fits 63 bits, in scalar
// instructions.
DEV bool less64(int64_t x, int64_t y) { return (int)((uint64_t)(x - y) >> 63) != 0; }
// min(d, 2^31 - 1) for d >= 0, likewise
DEV int sat31(int64_t d) { return ((uint64_t)d >> 31) ? INT32_MAX : (int)d; }
// One wavefront is the whole workgroup and its LDS operations execute in
// issue order, so ordering LDS traffic between lanes only needs the compiler
// not to move memory operations across this point.
DEV void wsync() { __asm__ volatile("" ::: "memory"); }
// Before reading back HBM this wavefront wrote (spill, overflow, timestamps).
DEV void hbm_fence() { __builtin_amdgcn_s_waitcnt(0); __asm__ volatile("" ::: "memory"); }

// DPP lane moves (GFX9 encodings): row_shr:n shifts within 16-lane rows,
// row_bcast:15 / :31 carry a row's last lane into the next row(s), wave_shr:1
// shifts across the whole wavefront. Disabled or out-of-range lanes take `old`.
constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118;
constexpr int kBc15 = 0x142, kBc31 = 0x143, kWShr1 = 0x138;

template <int CTRL, int RM = 0xf>
DEV int dpp(int old, int x) {
    return __builtin_amdgcn_update_dpp(old, x, CTRL, RM, 0xf, false);
}
template <int CTRL, int RM = 0xf>
DEV uint64_t dppu(uint64_t old, uint64_t x) {
    const uint32_t lo = (uint32_t)dpp<CTRL, RM>((int)(uint32_t)old, (int)(uint32_t)x);
    const uint32_t hi = (uint32_t)dpp<CTRL, RM>((int)(uint32_t)(old >> 32), (int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// inclusive prefix sum over the wavefront
DEV int scan_add(int x) {
    x += dpp<kShr1>(0, x);
    x += dpp<kShr2>(0, x);
    x += dpp<kShr4>(0, x);
    x += dpp<kShr8>(0, x);
    x += dpp<kBc15, 0xa>(0, x);
    x += dpp<kBc31, 0xc>(0, x);
    return x;
}
DEV int wsum(int x) { return rl(scan_add(x), 63); }
// the same for values from 0 to 2^31 - 1 whose sum may pass them
DEV int64_t wsum_wide(int x) {
    return (int64_t)wsum(x & 0xffff) + ((int64_t)wsum(x >> 16) << 16);
}
DEV int wmin(int x) {
    x = min(x, dpp<kShr1>(INT32_MAX, x));
    x = min(x, dpp<kShr2>(INT32_MAX, x));
    x = min(x, dpp<kShr4>(INT32_MAX, x));
    x = min(x, dpp<kShr8>(INT32_MAX, x));
    x = min(x, dpp<kBc15, 0xa>(INT32_MAX, x));
    x = min(x, dpp<kBc31, 0xc>(INT32_MAX, x));
    return rl(x, 63);
}
DEV uint64_t scan_maxu(uint64_t x) {
    uint64_t y;
    y = dppu<kShr1>(0ull, x), x = y > x ? y : x;
    y = dppu<kShr2>(0ull, x), x = y > x ? y : x;
    y = dppu<kShr4>(0ull, x), x = y > x ? y : x;
    y = dppu<kShr8>(0ull, x), x = y > x ? y : x;
    y = dppu<kBc15, 0xa>(0ull, x), x = y > x ? y : x;
    y = dppu<kBc31, 0xc>(0ull, x), x = y > x ? y : x;
    return x;
}
DEV uint64_t scan_minu(uint64_t x) {
    uint64_t y;
    y = dppu<kShr1>(~0ull, x), x = y < x ? y : x;
    y = dppu<kShr2>(~0ull, x), x = y < x ? y : x;
    y = dppu<kShr4>(~0ull, x), x = y < x ? y : x;
    y = dppu<kShr8>(~0ull, x), x = y < x ? y : x;
    y = dppu<kBc15, 0xa>(~0ull, x), x = y < x ? y : x;
    y = dppu<kBc31, 0xc>(~0ull, x), x = y < x ? y : x;
    return x;
}
DEV uint64_t wminu(uint64_t x) { return rlu(scan_minu(x), 63); }
// the value of the previous lane (lane 0 gets `fill`)
DEV uint64_t prev_lane_u64(uint64_t x, uint64_t fill) { return dppu<kWShr1>(fill, x); }

// ------------------------------------------------------------ keys

DEV uint64_t pack(int64_t key, int idx) {
    return ((uint64_t)(key + kKeyOff) << kIdxBits) | (uint64_t)(uint32_t)idx;
}
DEV int64_t key_of(uint64_t pk) { return (int64_t)(pk >> kIdxBits) - kKeyOff; }
DEV int idx_of(uint64_t pk) { return (int)(pk & kIdxMask); }

// MemGuard level floor(log2(max(w,k)/k)) capped at 23, without a division:
// with e = floor(log2 w) - floor(log2 k), the level is e when w >= k 2^e and
// e - 1 otherwise (Eq. memguard_level). Branch-free (lanes with w < k take 0
// by a select), so a wave evaluates it without splitting.
DEV int level_of(int w, int k, int lk) {
    const int e = (31 - __clz(w | 1)) - lk;
    const int L = ((w >> (e & 31)) >= k) ? e : e - 1;
    return w < k ? 0 : (L < kLevels - 1 ? L : kLevels - 1);
}

// ------------------------------------------------------------ LDS layout

// LDS holds the candidate list as three parallel arrays: the slot state
// {gs, w, kv, left} (what formation reads, one load per lane), the packed
// key (searches and merges) and the pair {tl, gm} of the last token time and
// the largest inter-token gap so far (emission only). The gap maximum stays
// on chip until the request completes, so the per-token work touches no HBM.
// The slot state takes 16 bytes, or 8 in the compact layout used when every
// request has P + D < 2^16 and D <= 2^15: w and kv in 16 bits each, left - 1
// in the flag word's bits 17..31 (the flags use bits 0..16). An entry is then
// 24 bytes instead of 32, which lets 16 instead of 12 instances share a
// compute unit's LDS at the large sweep's list size.
struct Lds {
    uint4 *q;   // four-word slots
    uint2 *q2;  // compact slots
    uint64_t *k;
    uint2 *tg;
    int64_t *bt;
    uint64_t *ty;  // Tally
    struct AdaLds *as;  // adaptive gamma: state, then the window in completion
    uint32_t *wr, *ws;  // order (a ring) and sorted
};

// Counters of one instance, kept in LDS (of a replica: in its router block).
enum Tally { TY_REQITERS, TY_TOKENS, TY_EVVOL, TY_EVFORCED, TY_WORK, TY_IDLE };

// Adaptive-gamma state of one instance (LDS, written by lane 0).
struct AdaLds {
    double gamma, ghat;      // current gamma, latest estimate
    int32_t wn, whead;       // latencies in the window, ring slot of the oldest
    int32_t cell, wnew;      // grid cell in use; 1: the window changed since ghat
    int64_t switches;        // grid-cell changes
    int32_t window, min_samples;
};
static_assert(sizeof(AdaLds) == kAdaStateBytes, "adaptive-gamma LDS block");

struct R {  // one candidate-list record in registers
    uint64_t pk = 0;
    int w = 0, left = 0, kv = 0;
    uint32_t gs = 0, tl = 0, gm = 0;
};

DEV R from_rec(const Rec &r) {
    R x;
    x.pk = r.pk, x.w = r.w, x.left = r.left, x.kv = r.kv, x.gs = r.gs, x.tl = r.tl, x.gm = r.gm;
    return x;
}
DEV Rec to_rec(const R &x) {
    Rec r;
    r.pk = x.pk, r.w = x.w, r.left = x.left, r.kv = x.kv, r.gs = x.gs, r.tl = x.tl, r.gm = x.gm;
    return r;
}
DEV R shfl_rec(const R &x, int src) {
    R y;
    y.pk = (uint64_t)__shfl((unsigned long long)x.pk, src);
    y.w = __shfl(x.w, src);
    y.left = __shfl(x.left, src);
    y.kv = __shfl(x.kv, src);
    y.gs = (uint32_t)__shfl((int)x.gs, src);
    y.tl = (uint32_t)__shfl((int)x.tl, src);
    y.gm = (uint32_t)__shfl((int)x.gm, src);
    return y;
}
DEV bool is_waiting(uint32_t g) { return (g & (G_RES | G_DONE)) == 0; }

// Destination lanes of a wavefront permutation: the lanes in m go, in order,
// to lanes base, base + 1, ...; the other lanes fill the remaining slots in
// order. Requires base + popc(m) <= 64.
DEV int place_dest(uint64_t m, int base) {
    const int before = mbcnt(m);
    if ((m >> lane()) & 1ull) return base + before;
    const int k = lane() - before;  // rank among the lanes outside m
    return k < base ? k : k + popc(m);
}
DEV uint32_t perm32(int dest, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_permute(dest * 4, (int)v);
}
// Move a record across lanes (a register transpose: no LDS storage is used).
// Every lane must be active, and dest must be a permutation.
DEV R permute_rec(const R &x, int dest) {
    R y;
    const uint32_t lo = perm32(dest, (uint32_t)x.pk), hi = perm32(dest, (uint32_t)(x.pk >> 32));
    y.pk = ((uint64_t)hi << 32) | lo;
    y.w = (int)perm32(dest, (uint32_t)x.w);
    y.left = (int)perm32(dest, (uint32_t)x.left);
    y.kv = (int)perm32(dest, (uint32_t)x.kv);
    y.gs = perm32(dest, x.gs);
    y.tl = perm32(dest, x.tl);
    y.gm = perm32(dest, x.gm);
    return y;
}

// ------------------------------------------------------------ the simulator

// BSH: log2 of the KV block size when it is a power of two (the common
// 16-token block gets its own instantiation), -1 otherwise. The policy is a
// run-time value: one copy of the code serves every policy, so workgroups of
// different policies on one compute unit share the instruction cache.
// CL: one replica of a cluster behind a join-shortest-queue router; its
// arrivals are the global requests the router has dispatched to it so far.
// CP: compact slots (see Lds).
template <int BSH, bool EXT, bool CL = false, bool CP = false>
struct Sim {
    const SimArgs &A;
    Lds S;
    // instance constants (memguard and delta are zero unless pol is BOOST)
    Held<int> inst, trace, N, c, base, tok, div, k, lk;
    int M, T, Kb, bs, pol, memguard, lcap;
    int ltr_s, ltr_q;  // LTR+: starvation threshold and quantum (iterations)
    Held<int64_t> delta, max_iters;
    Held<uint64_t> kargs;  // address of the kernel's arguments
    Held<uint64_t> div_magic;  // ceil(2^64 / div) for div >= 2
    // state. It has to stay in scalar registers through every loop: the
    // compiler copies all of it wherever paths meet, and what does not fit is
    // moved to vector lanes and back. So the counters live in LDS (Tally),
    // 64-bit values see no comparison or select, and addresses used now and
    // then are read from the kernel arguments each time (args).
    int64_t t;
    int U, L, nW, nR, n_holes, lo_hole, spill_n, next, pf, completed, status;
    uint64_t spill_min;
    int64_t pa;
    int pP, pD;
    Held<int64_t> iters;
    Held<int> maxU;
    int ev_vol, ev_forced, fpass;  // evictions and passes of the latest formation
    // CL: the replica (wave) index, the global indices dispatched to it in
    // order (HBM, written and read by this wave only, through L2), how many,
    // the prefetched global index of each lane, and the completions of the
    // latest iteration
    int wv, Nk, pidx, last_done;
    // per-iteration formation results
    int cnt, used;
    int64_t sum_ctx;  // KV tokens of the batch, this iteration's included
    int64_t kv_res;   // KV tokens of all residents
    // per lane: iterations to the next completion of the batch's members (under
    // LTR+ also promotion or demotion), and to the next level crossing
    int evl, evx;
    // nothing waits and the batch repeats; the latest run of repeated
    // iterations reached an arrival or its limit
    bool alone, due;
    // The next iteration takes every resident, one token each, and all that
    // arrived, whole chunks of which have new_tok tokens and new_blk blocks
    bool join;
    int new_tok, new_blk;
    uint64_t emit_chunks;  // 64-entry chunks holding batch members or evictions
    bool emit_all;         // ranks moved during formation: visit every chunk
    // Repeated batch: the next iteration's formation would select the same
    // residents again, one token each, and nothing else (see step), so it is
    // skipped: the first `nb` residents of the list, up to rank `last`
    // (INT32_MAX: all of them). Emission reports whether every batch member
    // emitted a token.
    bool rep, all_emit;
    int nb, last;
    int n_chunks;  // chunks the latest emission visited
    int nmoved;  // entries whose key the latest emission or streak moved
    // the key of the waiting candidate that closed admissions in the latest
    // formation (~0: none), the smallest keys of the arrivals taken since
    // (per lane, ~0: none) and a count of spill_excess calls
    uint64_t close_pk, arr_pk;
    int n_spilled;
    // victim masks, lane c = chunk c: residents, and those a voluntary
    // eviction may take (MemGuard). Kept across iterations: bits change in
    // place on admission, eviction and completion; any edit that moves ranks
    // clears vm_ok and the next victim search rebuilds them.
    uint64_t vm_res, vm_ev;
    bool vm_ok;
    // adaptive gamma (null without): constants, and lane j < grid - 1 holds
    // the midpoint above grid point j (+infinity beyond)
    const DevAda *ad;
    double bnd;
    bool phase_signal;  // BOOST with Algorithm 2's signal: P in prefill, dec after
    bool cache_signal;  // BOOST with the cache-aware signal P - h + dec

    // The kernel's arguments, read again where they are used: addresses
    // needed a few times per request are not worth registers all the time.
    typedef const __attribute__((address_space(4))) SimArgs KArgs;
    DEV KArgs *args() const {
        uint64_t p = kargs;
        __asm__ volatile("" : "+s"(p));  // a new value each time: nothing to keep
        return (KArgs *)p;
    }
    DEV size_t toff() const { return (size_t)trace * (size_t)N; }
    DEV size_t ioff() const { return (size_t)inst * (size_t)N; }
    DEV size_t slot() const {
        return CL ? (size_t)inst * (size_t)args()->replicas + (size_t)wv : (size_t)inst;
    }
    DEV const int64_t *arr() const { return args()->arrival + toff(); }
    DEV const int32_t *Pp() const { return args()->prompt + toff(); }
    DEV const int32_t *Dp() const { return args()->decode + toff(); }
    // expected prefix-cache hits of the trace (cache_signal)
    DEV const int32_t *Hp() const { return args()->cached + toff(); }
    DEV int64_t *tfirst() const { return args()->tfirst + ioff(); }
    DEV int64_t *tlast() const { return args()->tlast + ioff(); }
    // the instance's max-gap outputs, written at completion
    DEV uint32_t *tbo() const { return args()->tbtmax + ioff(); }
    DEV Rec *spill() const { return args()->spill + slot() * (size_t)scap(); }
    DEV int scap() const { return args()->spill_cap; }
    DEV Rec *ovf() const { return args()->ovf + slot() * (size_t)args()->ovf_stride; }
    DEV int32_t *jl() const { return args()->jidx + slot() * (size_t)N; }

    DEV Sim(const SimArgs &a, const DevSetting &st, int i, unsigned char *smem, uint64_t *tally,
            int w = 0)
        : A(a) {
        inst = i;
        trace = st.trace;
        kargs = sgpr64((uint64_t)__builtin_amdgcn_kernarg_segment_ptr());
        N = a.n_req;
        c = a.c;
        M = a.M, T = a.T, Kb = a.Kb, bs = a.bs, lcap = a.list_cap;
        base = a.base;
        tok = a.tok;
        div = a.div;
        div_magic = a.div_magic;
        max_iters = a.max_iters;
        const int k0 = st.k > 0 ? st.k : 1;
        k = k0;
        lk = 31 - __clz(k0);
        pol = st.policy;
        ltr_s = st.ltr_s, ltr_q = st.ltr_q;
        memguard = st.memguard;
        delta = st.delta;
        wv = w, Nk = 0, pidx = 0, last_done = 0;
        S.ty = tally;
        if (lane() < kTally) S.ty[lane()] = 0;
        const int cap = lcap + kStage;  // the list may use its overflow region during formation
        size_t o = 0;
        S.q = nullptr, S.q2 = nullptr;
        if constexpr (CP) S.q2 = (uint2 *)(smem + o), o += (size_t)cap * 8;
        else S.q = (uint4 *)(smem + o), o += (size_t)cap * 16;
        S.k = (uint64_t *)(smem + o), o += (size_t)cap * 8;
        S.tg = (uint2 *)(smem + o), o += (size_t)cap * 8;
        S.bt = (int64_t *)(smem + o), o += (size_t)kLevels * 8;
        if (lane() < kLevels) S.bt[lane()] = st.bt[lane()];
        ad = nullptr;
        bnd = 0.0;
        phase_signal = EXT && st.signal == 1;
        cache_signal = EXT && st.signal == 2;
        if constexpr (EXT) {
            S.as = (AdaLds *)(smem + o), o += kAdaStateBytes;
            S.wr = (uint32_t *)(smem + o), o += (size_t)a.ada_window * 4;
            S.ws = (uint32_t *)(smem + o);
            ad = st.ada >= 0 ? a.ada + st.ada : nullptr;
        }
        if (EXT && ad) {  // the table of the first cell is st.bt
            bnd = ad->bound[lane()];
            if (lane() == 0) {
                AdaLds &G = *S.as;
                G.gamma = ad->gamma0, G.ghat = 0.0;
                G.wn = G.whead = G.wnew = 0;
                G.cell = ad->cell0;
                G.switches = 0;
                G.window = ad->window, G.min_samples = ad->min_samples;
            }
        }
        t = 0;
        U = L = nW = nR = n_holes = spill_n = next = pf = completed = status = 0;
        lo_hole = INT32_MAX;
        spill_min = ~0ull;
        iters = 0;
        maxU = 0;
        ev_vol = ev_forced = fpass = 0;
        cnt = used = 0;
        sum_ctx = kv_res = 0;
        evl = evx = INT32_MAX;
        alone = due = join = false;
        new_tok = new_blk = 0;
        emit_chunks = 0;
        emit_all = false;
        rep = all_emit = false;
        nb = 0, last = INT32_MAX;
        nmoved = 0, n_chunks = 0;
        close_pk = arr_pk = ~0ull;
        n_spilled = 0;
        vm_res = vm_ev = 0;
        vm_ok = false;
        wsync();
    }

    // Adds to the counters in LDS (per step: below 2^32 each): lane j adds to
    // counter j, nothing waits for it.
    DEV void tally(int req, int tok_, int work) const {
        int v = 0;
        v = set_lane<TY_REQITERS>(v, req);
        v = set_lane<TY_TOKENS>(v, tok_);
        v = set_lane<TY_WORK>(v, work);
        if (ev_vol + ev_forced) {
            v = set_lane<TY_EVVOL>(v, ev_vol);
            v = set_lane<TY_EVFORCED>(v, ev_forced);
        }
        if (lane() <= TY_WORK)
            __hip_atomic_fetch_add(&S.ty[lane()], (uint64_t)(uint32_t)v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    DEV void fail(int code) {
        if (status == 0) status = code;
    }

    // ---------------------------------------------------------- slots

    // The state of slot i as loaded: the flag word in .x (compact: with
    // left - 1 above the flags), the rest unpacked by sw / skv / sleft.
    DEV uint4 ldq(int i) const {
        if constexpr (CP) {
            const uint2 v = S.q2[i];
            return make_uint4(v.x, v.y, 0u, 0u);
        } else {
            return S.q[i];
        }
    }
    DEV int sw(const uint4 &v) const { return CP ? (int)(v.y & 0xffffu) : (int)v.y; }
    DEV int skv(const uint4 &v) const { return CP ? (int)(v.y >> 16) : (int)v.z; }
    DEV int sleft(const uint4 &v) const {
        return CP ? (int)(v.x >> kLeftShift) + 1 : (int)v.w;
    }
    DEV void stq(int i, uint32_t x, int w, int kv, int left) const {
        if constexpr (CP) {
            S.q2[i] = make_uint2((x & G_FLAGS) | ((uint32_t)(left - 1) << kLeftShift),
                                 (uint32_t)w | ((uint32_t)kv << 16));
        } else {
            S.q[i] = make_uint4(x, (uint32_t)w, (uint32_t)kv, (uint32_t)left);
        }
    }
    // the flag word alone (flag edits keep the compact layout's left bits)
    DEV uint32_t ldx(int i) const { return CP ? S.q2[i].x : S.q[i].x; }
    DEV void stx(int i, uint32_t x) const {
        if constexpr (CP) S.q2[i].x = x;
        else S.q[i].x = x;
    }
    // the flag word (as loaded, flags edited) and kv of a slot whose w is w
    DEV void stxkv(int i, uint32_t x, int w, int kv) const {
        if constexpr (CP) {
            S.q2[i] = make_uint2(x, (uint32_t)w | ((uint32_t)kv << 16));
        } else {
            S.q[i].x = x;
            S.q[i].z = (uint32_t)kv;
        }
    }
    DEV void ldr(int i, R &x) const {
        const uint4 q = ldq(i);
        x.gs = q.x, x.w = sw(q), x.kv = skv(q), x.left = sleft(q);
        x.pk = S.k[i];
        const uint2 tg = S.tg[i];
        x.tl = tg.x, x.gm = tg.y;
    }
    DEV void str(int i, const R &x) const {
        stq(i, x.gs, x.w, x.kv, x.left);
        S.k[i] = x.pk;
        S.tg[i] = make_uint2(x.tl, x.gm);
    }
    // Entries the list keeps before spilling waiting ones. The adaptive build
    // sizes the waiting window from the residents (max(M, residents) + 128,
    // within lcap): its grid changes let residents outside the batch pile up,
    // and a list padded with waiting entries costs every pass over it.
    DEV int cap_now() const {
        if constexpr (EXT) {
            if (pol == P_LTR) return lcap;  // LTR+ keeps every request on chip
            return min(lcap, max(M, nR) + 128);
        } else {
            return lcap;
        }
    }
    // floor(s / div). Below 2^32 a multiply by the rounded-up reciprocal is
    // exact: s * ceil(2^64/div) / 2^64 exceeds s/div by less than 2^-32 <= 1/div.
    DEV uint64_t ctx_quot(uint64_t s) const {
        if (s >> 32) return s / (uint64_t)(int)div;
        return ctx_quot32((uint32_t)s);
    }
    DEV uint32_t ctx_quot32(uint32_t x) const {
        if (div == 1) return x;
        return (uint32_t)(((uint64_t)x * (div_magic >> 32) + __umulhi(x, (uint32_t)div_magic)) >> 32);
    }
    // the cost of an iteration of `tokens` tokens without its context term
    DEV int64_t fixed_cost(int tokens) const { return (int64_t)base + (int64_t)tok * tokens; }
    // The signal at which level `lvl` ends, k 2^(lvl+1) (signals stay below
    // 2^24: INT32_MAX for a threshold beyond, and above the last level).
    DEV int next_level(int lvl) const {
        return k.v <= (0xffffff >> (lvl + 1)) ? k.v << (lvl + 1) : INT32_MAX;
    }
    DEV int blocks(int x) const {
        if constexpr (BSH >= 0) {
            return (x + (1 << BSH) - 1) >> BSH;
        } else {
            return (x + bs - 1) / bs;
        }
    }

    // New KV blocks of the members (one per lane; kv tokens each) for r more
    // tokens each, over the wave: with power-of-two blocks r / bs each, and
    // one more where r mod bs exceeds what is free in the last block.
    DEV int growth(bool memb, int kv, int r) const {
        if constexpr (BSH >= 0) {
            const int m = (1 << BSH) - 1;
            const uint64_t all = ballot(memb), more = ballot(memb && ((-kv) & m) < (r & m));
            return popc(all) * (r >> BSH) + popc(more);
        } else {
            return wsum(memb ? blocks(kv + r) - blocks(kv) : 0);
        }
    }

    // The sum over the wave of each lane's KV tokens of up to 64 requests:
    // below 2^16 tokens each with compact slots, 2^24 otherwise.
    DEV int64_t ctx_sum(int x) const {
        if constexpr (CP) return wsum(x);
        return wsum_wide(x);
    }

    // ---------------------------------------------------------- arrivals

    // requests this instance (replica) may take: the trace, or those
    // dispatched to the replica so far
    DEV int n_known() const { return CL ? Nk : N; }

    // Without a branch on the lane: the compiler merges the join of such a
    // branch with the caller's, and then takes scalar state (pf, next and all
    // that follows from them) for lane-dependent and keeps it in vector
    // registers.
    DEV void load_pf() {
        const int n = n_known(), r = pf + lane();
        const bool in = r < n;
        int at = min(r, n - 1);
        if constexpr (CL) {
            if (n == 0) {  // nothing dispatched yet
                pa = INT64_MAX, pP = 1, pD = 1, pidx = 0;
                return;
            }
            at = __hip_atomic_load(&jl()[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pidx = in ? at : 0;
        }
        const int64_t a = arr()[at];
        const int p = Pp()[at], d = Dp()[at];
        pa = in ? a : INT64_MAX, pP = in ? p : 1, pD = in ? d : 1;
    }

    DEV R new_record(int idx, int64_t a, int P, int D) const {
        R x;
        x.w = P, x.left = D;
        int64_t key;
        uint32_t lvl = 0;
        if (pol == P_FCFS || (EXT && pol == P_SARATHI)) {
            key = a;  // Sarathi: prefills wait in arrival order
        } else if (pol == P_SRPT || pol == P_TRAIL) {
            key = (int64_t)P + D - 1;  // remaining computed tokens
        } else if (pol == P_SPF || pol == P_LAS) {
            key = P;  // prompt length; the attained service P + dec at dec = 0
        } else if (pol == P_SJF || (EXT && pol == P_LTR)) {
            key = D;  // output length (LTR+: until a promotion)
        } else {
            int sig = P;  // the signal before the first token
            if constexpr (EXT) {
                // cached tokens are not work (lanes past the trace hold no request)
                if (cache_signal && idx < N.v) sig = P - Hp()[idx];
            }
            lvl = (uint32_t)level_of(sig, k.v, lk.v);
            key = a - S.bt[lvl];
        }
        x.gs = lvl << G_LVL_SHIFT;
        x.pk = pack(key, idx);
        return x;
    }

    // Arrivals with a <= t join the waiting set, up to 64 per round.
    DEV void take_arrivals() {
        for (int round = 0; round <= (N >> 6) + 1 && status == 0; round++) {
            int off = next - pf;
            if (off >= kWave) {
                pf = next;
                load_pf();
                off = 0;
            }
            const int r = pf + lane();
            const bool arrive = lane() >= off && r < n_known() && pa <= t;
            const int n_arr = popc(ballot(arrive));
            if (LIKELY(n_arr == 0)) return;
            const R x = new_record(CL ? pidx : r, pa, pP, pD);
            const R y = off ? shfl_rec(x, min(off + lane(), kWave - 1)) : x;
            arr_pk = min(arr_pk, lane() < n_arr ? y.pk : ~0ull);
            const int n0 = lane() < n_arr ? min(y.w, c.v) : 0, b0 = blocks(n0);
            new_tok += n_arr == 1 ? rl(n0, 0) : wsum(n0);
            new_blk += n_arr == 1 ? rl(b0, 0) : wsum(b0);
            nW += n_arr;
            next += n_arr;
            add_entries(y, n_arr);
            if (off + n_arr < kWave) return;
        }
    }

    // ---------------------------------------------------------- list edits

    // Number of list entries with pk < x (x wave-uniform): the last key of
    // every 64-entry chunk, then one chunk. Requires L <= 64 * 64.
    DEV int lower_bound(uint64_t x) const {
        if (L == 0) return 0;
        const int nch = (L + kWave - 1) >> 6;
        const int probe = min(lane() * kWave + kWave - 1, L - 1);
        const uint64_t cm = lane() < nch ? S.k[probe] : ~0ull;
        const int c0 = popc(ballot(lane() < nch && cm < x));
        if (c0 >= nch) return L;
        const int r = c0 * kWave + lane();
        const uint64_t v = r < L ? S.k[r] : ~0ull;
        return c0 * kWave + popc(ballot(r < L && v < x));
    }

    // Merge K records held by lanes [0, K) into the sorted list.
    // Requires L + K <= lcap + kStage (the list's overflow region).
    DEV void merge_new(const R &x, int K) {
        if (K <= 0) return;
        const bool act = lane() < K;
        int rn = 0;
        for (int j = 0; j < K; j++) rn += (act && rlu(x.pk, j) < x.pk) ? 1 : 0;
        const uint64_t xmin = wminu(act ? x.pk : ~0ull);
        const int minpos = lower_bound(xmin);
        int pos_in = 0;  // lane j < K: list entries at ranks >= minpos smaller than x_j
        if (minpos < L) {
            for (int b = ((L - 1) >> 6) << 6; b >= 0 && b + kWave > minpos; b -= kWave) {
                const int r = b + lane();
                const bool mv = r >= minpos && r < L;
                const uint64_t pr = mv ? S.k[r] : ~0ull;
                int sh = 0;
                for (int j = 0; j < K; j++) {
                    const uint64_t xj = rlu(x.pk, j);
                    sh += (mv && xj < pr) ? 1 : 0;
                    const int cj = popc(ballot(mv && pr < xj));
                    if (lane() == j) pos_in += cj;
                }
                const bool go = mv && sh > 0;
                if (ballot(go)) vm_ok = false;
                R y;
                if (go) ldr(r, y);
                wsync();
                if (go) str(r + sh, y);
                wsync();
            }
        }
        if (act) str(minpos + pos_in + rn, x);
        wsync();
        L += K;
    }

    // Remove the entries whose flags intersect `mask`, from rank `from` on.
    DEV void compact_remove(int from, uint32_t mask) {
        vm_ok = false;
        int out = from;
        for (int b = (from >> 6) << 6; b < L; b += kWave) {
            const int r = b + lane();
            const bool v = r >= from && r < L;
            R y;
            if (v) ldr(r, y);
            const bool keep = v && !(y.gs & mask);
            const uint64_t km = ballot(keep);
            wsync();
            if (keep) {
                const int d = out + mbcnt(km);
                if (d != r) str(d, y);
            }
            wsync();
            out += popc(km);
        }
        L = out;
    }

    DEV void drop_holes() {
        if (n_holes == 0) return;
        compact_remove(lo_hole, G_DONE);
        n_holes = 0;
        lo_hole = INT32_MAX;
    }

    // Keep at most cap_now() entries: drop holes, then spill the largest
    // waiting entries to HBM.
    DEV void spill_excess() {
        const int cap = cap_now();
        if (L <= cap) return;
        drop_holes();
        const int E = L - cap;
        if (E <= 0) return;
        n_spilled++;
        if (EXT && pol == P_LTR) {
            // a spilled request's starvation count would have to advance in
            // HBM every iteration: an LTR+ instance keeps every request on
            // chip, and one that outgrows the list reruns with a larger one
            fail(S_ECAPACITY);
            return;
        }
        if (spill_n + E > scap()) {
            fail(S_ECAPACITY);
            return;
        }
        int found = 0, lowest = L;
        for (int b = ((L - 1) >> 6) << 6; b >= 0 && found < E; b -= kWave) {
            const int r = b + lane();
            const bool isw = r < L && is_waiting(ldx(r));
            const uint64_t m = ballot(isw);
            const int above = popc(m) - mbcnt(m) - 1;
            const bool take = isw && above < E - found;
            if (take) {
                R y;
                ldr(r, y);
                spill()[spill_n + found + above] = to_rec(y);
                stx(r, y.gs | G_MARK);
            }
            const uint64_t tm = ballot(take);
            found += popc(tm);
            if (tm) lowest = b + ffs0(tm);
        }
        wsync();
        if (found < E) {
            fail(S_ECAPACITY);
            return;
        }
        const uint64_t mn = uniu(S.k[lowest]);
        spill_min = sgpr64((spill_n == 0 || mn < spill_min) ? mn : spill_min);
        spill_n += E;
        nW -= E;
        compact_remove(lowest, G_MARK);
    }

    // Add K records (lanes [0, K)) to the list; waiting ones whose key exceeds
    // the spill's minimum go straight to the spill. L <= cap_now() on entry.
    DEV void add_entries(R y, int K) {
        if (spill_n > 0) {
            const bool toS = lane() < K && is_waiting(y.gs) && y.pk > spill_min;
            const uint64_t sm = ballot(toS);
            const int ns = popc(sm);
            if (ns) {
                if (spill_n + ns > scap()) {
                    fail(S_ECAPACITY);
                    return;
                }
                if (toS) spill()[spill_n + mbcnt(sm)] = to_rec(y);
                spill_n += ns;
                nW -= ns;
                const uint64_t km = ballot(lane() < K && !toS);
                y = permute_rec(y, place_dest(km, 0));
                K -= ns;
            }
        }
        if (K > 0) merge_new(y, K);
        if (L > cap_now()) spill_excess();
    }

    // The want-th smallest spilled key: radix select over 4-bit digits, the
    // 16 bin counts held one per lane (no LDS histogram).
    DEV uint64_t select_kth(int want) {
        hbm_fence();
        Rec *const spill = this->spill();
        uint64_t prefix = 0;
        int rank = want;
        for (int d = 15; d >= 0; d--) {
            const int sh = 4 * d;
            int cnt = 0;  // lane b < 16: matching entries whose digit is b
            for (int rd = 0; rd < spill_n; rd += kWave) {
                const int i = rd + lane();
                uint64_t key = 0;
                bool match = false;
                if (i < spill_n) {
                    key = spill[i].pk;
                    match = d == 15 || (key >> (sh + 4)) == (prefix >> (sh + 4));
                }
                if (!ballot(match)) continue;
                const int dig = (int)((key >> sh) & 15u);
                for (int b = 0; b < 16; b++) {
                    const int nb = popc(ballot(match && dig == b));
                    if (lane() == b) cnt += nb;
                }
            }
            const int inc = scan_add(lane() < 16 ? cnt : 0);
            const int exc = inc - cnt;
            const uint64_t hm = ballot(lane() < 16 && exc < rank && rank <= inc);
            if (hm == 0) {
                fail(S_ESTATE);
                return 0;
            }
            const int bin = ffs0(hm);
            rank -= rl(exc, bin);
            prefix |= (uint64_t)bin << sh;
        }
        return prefix;
    }

    // Bring the smallest spilled entries back on chip (as many as fit).
    DEV void refill() {
        drop_holes();
        refill_into(cap_now() - L);
    }

    DEV void refill_into(int room) {
        const int want = min(spill_n, room);
        if (want <= 0) return;
        Rec *const spill = this->spill();
        const uint64_t theta = want < spill_n ? select_kth(want) : ~0ull;
        if (status) return;
        hbm_fence();
        int wr = 0, got = 0;
        uint64_t newmin = ~0ull;
        const int n0 = spill_n;
        for (int rd = 0; rd < n0; rd += kWave) {
            const int i = rd + lane();
            const bool v = i < n0;
            Rec s = {};
            if (v) s = spill[i];
            const bool sel = v && s.pk <= theta;
            const bool keep = v && !sel;
            const uint64_t km = ballot(keep), sm = ballot(sel);
            if (keep) {
                const int d = wr + mbcnt(km);
                if (d != i) spill[d] = s;
                if (s.pk < newmin) newmin = s.pk;
            }
            wr += popc(km);
            const int ks = popc(sm);
            if (ks) {
                const R x = permute_rec(from_rec(s), place_dest(sm, 0));
                merge_new(x, ks);
                got += ks;
            }
        }
        if (got != want) fail(S_ESTATE);
        spill_n = wr;
        nW += got;
        spill_min = wminu(newmin);
    }

    // ---------------------------------------------------------- formation

    // Victim masks for the whole list: one LDS read and two ballots per chunk.
    // Batch members below the candidate are excluded by rank (victims lie
    // above it, where nothing is in the batch yet), so the masks ignore INB.
    DEV void build_victim_masks() {
        const int nch = (L + kWave - 1) >> 6;
        vm_res = vm_ev = 0;
        for (int c = 0; c < nch; c++) {
            const int r = c * kWave + lane();
            const uint32_t g = r < L ? ldx(r) : 0u;
            const bool rs = (g & G_RES) != 0;
            bool ev = rs;
            if (memguard) ev = rs && ((g >> G_LVL_SHIFT) & 31u) > (g & G_GUARD);
            if (pol == P_TRAIL && ballot(rs)) {
                // swap prevention: a request that emitted at least 0.6 D of its
                // D tokens is not a voluntary victim (5 (D - left) >= 3 D)
                int64_t Dv = 0, lv = 0;
                if (rs) {
                    const int idx = idx_of(S.k[r]);
                    Dv = idx < N.v ? Dp()[idx] : 0;
                    lv = CP ? (int)(g >> kLeftShift) + 1 : (int)S.q[r].w;
                }
                ev = rs && !(2 * Dv >= 5 * lv);
            }
            const uint64_t m1 = ballot(rs), m2 = ballot(ev);
            if (lane() == c) vm_res = m1, vm_ev = m2;
        }
        vm_ok = true;
    }

    // A request at rank r became resident (dispatch: MemGuard keeps it
    // non-evictable until its level moves) or stopped being one.
    DEV void vm_set(int r, bool resident) {
        if (!vm_ok) return;
        if (resident && pol == P_TRAIL) {  // eligibility depends on progress: rebuild
            vm_ok = false;
            return;
        }
        const uint64_t bit = 1ull << (r & 63);
        if (lane() == (r >> 6)) {
            if (resident) {
                vm_res |= bit;
                if (!memguard) vm_ev |= bit;
            } else {
                vm_res &= ~bit;
                vm_ev &= ~bit;
            }
        }
    }

    // Highest rank > q set in the per-chunk mask vm, or -1.
    DEV int top_above(uint64_t vm, int q) const {
        const int qc = q >> 6, qb = q & 63;
        uint64_t m = vm;
        if (lane() < qc) m = 0;
        else if (lane() == qc) m &= qb == 63 ? 0ull : (~0ull << (qb + 1));
        const uint64_t nz = ballot(m != 0);
        if (!nz) return -1;
        const int ch = fls0(nz);
        return ch * kWave + fls0(rlu(m, ch));
    }

    // Highest rank > q holding a resident outside the batch that may be
    // evicted for candidate q (voluntary: MemGuard and hysteresis apply).
    // The list is sorted, so the highest such rank is the worst (key, idx).
    DEV int find_victim(int q, bool voluntary) {
        if constexpr (EXT) {
            if (voluntary && pol == P_SARATHI) return -1;  // no preemption by priority
        }
        if (UNLIKELY(!vm_ok)) build_victim_masks();
        const int v = top_above(voluntary ? vm_ev : vm_res, q);
        if (voluntary && v >= 0 && delta > 0) {
            // the worst eligible key fails the hysteresis test => all fail
            const uint64_t pv = uniu(S.k[v]), pkq = uniu(S.k[q]);
            const int64_t kd = key_of(pv) - delta, kq = key_of(pkq);
            if (!(kd > kq || (kd == kq && idx_of(pv) > idx_of(pkq)))) return -1;
        }
        return v;
    }

    DEV void do_evict(int v) {
        const uint4 qv = ldq(v);
        const int kvv = uni(skv(qv)), wv_ = uni(sw(qv));
        const uint32_t g = (uint32_t)uni((int)qv.x);
        wsync();
        if (lane() == 0)
            stxkv(v, (g & ~G_RES) | G_EVI | (pol == P_SRPT || pol == P_TRAIL ? G_DIRTY : 0u), wv_, 0);
        wsync();
        U -= blocks(kvv);
        kv_res -= kvv;
        nW++;
        nR--;
        emit_chunks |= 1ull << (v >> 6);
        vm_set(v, false);
    }

    // Admission of candidate q with n tokens: its KV advances now (emission
    // finds the tokens scheduled this iteration already counted).
    DEV void admit_one(int q, uint32_t g, int n, int du, int kvv, int wq, int64_t &ctx_one) {
        const bool res = (g & G_RES) != 0;
        const int kv2 = uni(kvv + n);  // (wave-uniform also after the masked store)
        uint32_t g2 = g | G_INB;
        if (!res) g2 = (g2 & ~G_GUARD) | G_RES | ((g >> G_LVL_SHIFT) & 31u);
        if (lane() == 0) stxkv(q, g2, wq, kv2);
        wsync();
        cnt++;
        used += n;
        U += du;
        ctx_one += kv2;
        if (!res) {
            nW--, nR++;
            vm_set(q, true);
        }
        emit_chunks |= 1ull << (q >> 6);
    }

    // Candidate q did not fit: evictions, or closing admissions. r_ahead
    // counts residents at ranks > q.
    // (g, n, du, kvv, wq: its flag word, chunk size, KV blocks, KV tokens and w)
    DEV void slow_path(int q, uint32_t g, int n, int du, int kvv, int wq, bool &closed,
                       int &r_ahead, int64_t &ctx_one) {
        const bool res = (g & G_RES) != 0;
        for (int it = 0; it <= L + 1; it++) {
            if (U + du <= Kb) {
                admit_one(q, g, n, du, kvv, wq, ctx_one);
                return;
            }
            int v = find_victim(q, true);
            if (v >= 0) {
                do_evict(v);
                r_ahead--;
                ev_vol++;
                continue;
            }
            if (res) {
                v = find_victim(q, false);
                if (v >= 0) {
                    do_evict(v);
                    r_ahead--;
                    ev_forced++;
                    continue;
                }
                do_evict(q);
                ev_forced++;
                return;
            }
            closed = true;
            close_pk = uniu(S.k[q]);
            return;
        }
        fail(S_ESTATE);
    }

    // Spilled entries come next in the candidate order (formation reached
    // the first on-chip key above the spill's minimum with admissions open):
    // bring the smallest of them on chip. Every entry below rank p has been
    // processed and keeps its rank; every on-chip waiting key is below p.
    DEV void mid_refill(int p) {
        if (n_holes > 0) {
            const int from = max(p, lo_hole);
            const int L0 = L;
            compact_remove(from, G_DONE);
            n_holes -= L0 - L;
            if (n_holes == 0) lo_hole = INT32_MAX;
        }
        int room = cap_now() + kStage - L;  // may use the overflow region
        if (room <= 0) room = lcap + kStage - L;
        if (room <= 0) {
            fail(S_ECAPACITY);
            return;
        }
        refill_into(room);
        emit_all = true;
    }

    // Bound by its dependent chain (loads, ballots, scans), so a chunk whose
    // candidates all fit skips the prefix sums: at most one of them computes
    // more than one token nearly always, and ballots then give the totals.
    // The batch's context is the residents' (kept up to date as they change)
    // unless some are left out.
    DEV void formation() {
        // a formation that closed admissions is followed by others that do:
        // no use in adding up the candidates before the closing one
        const bool tight = close_pk != ~0ull;
        close_pk = ~0ull;
        ev_vol = ev_forced = fpass = 0;
        cnt = 0, used = 0;
        emit_chunks = 0;
        emit_all = false;
        bool closed = false;
        int r_ahead = nR;  // residents at ranks >= p
        int p = 0;
        int vctx = 0;         // per lane: KV tokens of the members admitted by chunk,
        int64_t ctx_one = 0;  // and of those admitted one by one
        int bstar = spill_n > 0 ? lower_bound(spill_min) : INT32_MAX;
        // the next chunk's records, loaded while this one is processed; valid
        // while formation walks whole chunks without touching the list
        const int lim = lcap + kStage;
        const uint32_t max_pass = (uint32_t)lim + (uint32_t)spill_n + 2u;
        uint4 nx = make_uint4(0u, 0u, 0u, 0u);
        bool have_nx = false;
        // every pass advances p or refills from the spill, so the walk ends
        // within L + spill_n passes; a walk that does not is a broken state
        for (;;) {
            if (UNLIKELY(!closed && p >= bstar)) {  // bstar <= L: spilled entries come next
                if (UNLIKELY((uint32_t)++fpass > max_pass)) {
                    fail(S_ESTATE);
                    return;
                }
                mid_refill(p);
                if (status) return;
                bstar = spill_n > 0 ? lower_bound(spill_min) : INT32_MAX;
                have_nx = false;
                continue;
            }
            if (p >= L) break;
            if (UNLIKELY((uint32_t)++fpass > max_pass)) {
                fail(S_ESTATE);
                return;
            }
            const int end = closed ? L : min(L, bstar);
            const int r = p + lane();
            const bool valid = r < end;
            // (lanes past the slots read the last one; they are not valid)
            uint4 qr = nx;
            if (!have_nx) qr = ldq(min(r, lim - 1));
            nx = ldq(min(r + kWave, lim - 1));
            const uint32_t g = valid ? qr.x : 0u;
            const int w = sw(qr);
            const int kvv = skv(qr);
            const bool res = (g & G_RES) != 0;
            const bool cand = valid && !(g & (G_EVI | G_DONE)) && (res || !closed);
            const int m = cand ? min(w - kvv, c.v) : 0;
            const int d = cand ? blocks(kvv + m) - blocks(kvv) : 0;
            const uint64_t cm = ballot(cand), resm = ballot(res);
            int mt = 0, dt = 0;  // tokens and blocks of the lanes admitted
            int path = 1;  // 0: all fit, 1: count lanes, 2: prefix sums
            if (closed || !tight) {  // do all candidates fit?
                const uint64_t big = ballot(m > 1);
                if (UNLIKELY((big & (big - 1)) != 0)) {
                    // several long chunks: their totals take the sums anyway
                    // (LAS under KV pressure, where most formations have
                    // such: 3 to 6 % of a step against summing twice)
                    path = 2;
                } else {
                    mt = popc(cm), dt = popc(ballot(d > 0));
                    if (big) {
                        const int l = ffs0(big), db = rl(d, l);
                        mt += rl(m, l) - 1;
                        dt += db > 0 ? db - 1 : 0;
                    }
                    path = cnt + popc(cm) <= M && mt <= T - used && dt <= Kb - U ? 0 : 1;
                }
            }
            uint64_t okm = cm, bad = 0;
            int n = m, du = d;
            bool scan = path != 0;
            if (path == 1) {
                // Up to the first candidate that computes more than a token,
                // counting lanes gives the prefix sums (two chains of six
                // dependent lane moves). Where the KV budget binds, the
                // candidate that does not fit is nearly always among those,
                // the first waiting one at the latest: 1 % off the chat,
                // large and comparator sweeps and the clusters, 2 % off the
                // ragged engine, 0.3 % off the reasoning sweep.
                const uint64_t big = ballot(m > 1), dm = ballot(d > 0);
                const uint64_t upto = big ? big ^ (big - 1) : ~0ull;
                const uint64_t over = ballot(mbcnt(dm) + d > Kb - U) & upto;
                if (over) {
                    const int ql = ffs0(over);
                    const uint64_t before = cm & ((1ull << ql) - 1ull);
                    const int k = popc(before);
                    if (cnt + k < M && rl(m, ql) <= T - used - k) {
                        bad = over, okm = before;
                        mt = k, dt = popc(dm & before);
                        scan = false;
                    }
                }
            }
            if (scan) {
                // the candidates admitted from this chunk are a prefix of
                // its candidates, and only the last of them can be clipped
                // by the token budget
                const int ub = used + scan_add(m) - m;
                const int dfi = scan_add(d);
                const bool adm = cand && cnt + mbcnt(cm) < M && ub < T;
                n = adm ? min(m, T - ub) : 0;
                du = adm ? blocks(kvv + n) - blocks(kvv) : 0;
                const int dui = dfi - d + du;
                bad = ballot(adm && U + dui > Kb);
                const uint64_t am = ballot(adm);
                okm = bad ? (am & ((1ull << ffs0(bad)) - 1ull)) : am;
                if (okm) {
                    const int last_ = fls0(okm);
                    mt = rl(ub + n, last_) - used, dt = rl(dui, last_);
                }
            }
            const bool ok = ((okm >> lane()) & 1ull) != 0;
            if (ok) {  // admitted: the KV advances by this iteration's chunk now
                uint32_t g2 = g | G_INB;
                if (!res) g2 = (g2 & ~G_GUARD) | G_RES | ((g >> G_LVL_SHIFT) & 31u);
                stxkv(r, g2, w, kvv + n);
                vctx += kvv + n;
            }
            if (okm) {
                const uint64_t nm = okm & ~resm;
                const int nadm_w = popc(nm);
                cnt += popc(okm);
                used += mt;
                U += dt;
                nW -= nadm_w;
                nR += nadm_w;
                if (pol == P_TRAIL && nadm_w) vm_ok = false;  // eligibility depends on progress
                if (UNLIKELY(vm_ok && nadm_w)) {  // dispatched waiting entries become residents
                    // lanes of this chunk land in aligned chunks p>>6 and (p>>6)+1
                    const int c0 = p >> 6, sh = p & 63;
                    const uint64_t lo = nm << sh, hi = sh ? (nm >> (64 - sh)) : 0ull;
                    const bool ev_too = !memguard;
                    if (lane() == c0) vm_res |= lo, vm_ev |= ev_too ? lo : 0ull;
                    if (lane() == c0 + 1) vm_res |= hi, vm_ev |= ev_too ? hi : 0ull;
                }
                emit_chunks |= (1ull << ((p + ffs0(okm)) >> 6)) | (1ull << ((p + fls0(okm)) >> 6));
            }
            wsync();
            if (bad) {
                const int ql = ffs0(bad);
                // residents among lanes [0, ql] are passed (q included if resident);
                // waiting entries admitted in this chunk sit below q
                r_ahead -= popc(resm & (ql == 63 ? ~0ull : ((2ull << ql) - 1ull)));
                slow_path(p + ql, (uint32_t)rl((int)g, ql), rl(n, ql), rl(du, ql), rl(kvv, ql),
                          rl(w, ql), closed, r_ahead, ctx_one);
                if (status) return;
                p = p + ql + 1;
                have_nx = false;
            } else {
                r_ahead -= popc(resm);
                const int p2 = min(p + kWave, end);
                have_nx = p2 == p + kWave;
                p = p2;
            }
            if (cnt >= M || used >= T || (closed && r_ahead <= 0)) break;
        }
        kv_res += used;
        sum_ctx = kv_res;
        if (cnt != nR)  // residents outside the batch
            sum_ctx = ctx_one + ctx_sum(vctx);
    }

    // ---------------------------------------------------------- execute

    // Returns the lowest rank whose key moved (INT32_MAX if none). `all_in`:
    // there was no formation, every live entry is a member (see join) and is
    // admitted here.
    DEV int emission(int64_t t_end, bool all_in) {
        int lo = INT32_MAX, lohole = INT32_MAX, nd = 0, ufree = 0, kfree = 0, nmv = 0;
        nmoved = 0, n_chunks = 0;
        evl = evx = INT32_MAX;
        int64_t it_end = 0;
        if constexpr (EXT) it_end = (int64_t)sgpr64((uint64_t)(iters + 1));
        int opened = 0;  // all_in: blocks that residents opened
        bool bad_idx = false;
        uint64_t noemit = 0;  // batch members that emitted no token
        const uint32_t t32 = (uint32_t)t_end;
        const int nch = (L + kWave - 1) >> 6;
        // LTR+ updates every candidate's starvation count: visit every chunk
        if (all_in || emit_all || (EXT && pol == P_LTR))
            emit_chunks = nch >= 64 ? ~0ull : ((1ull << nch) - 1ull);
        uint64_t todo = emit_chunks;
        if (!todo) return INT32_MAX;
        n_chunks = popc(todo);
        // chunks are visited in ascending order, the next one's records loaded
        // while this one is processed (a chunk's edits stay inside it). Lanes
        // past the list end read its last slot and are masked out.
        int b = ffs0(todo) * kWave;
        todo &= todo - 1;
        uint4 q;
        uint64_t pk;
        uint2 tg;
        {
            const int i0 = min(b + lane(), L - 1);
            q = ldq(i0), pk = S.k[i0], tg = S.tg[i0];
        }
        for (;;) {
            const int bn = todo ? ffs0(todo) * kWave : -1;
            todo &= todo - 1;
            uint4 qn = make_uint4(0u, 0u, 0u, 0u);
            uint64_t pkn = 0;
            uint2 tgn = make_uint2(0u, 0u);
            if (bn >= 0) {
                const int i1 = min(bn + lane(), L - 1);
                qn = ldq(i1), pkn = S.k[i1], tgn = S.tg[i1];
            }
            const int r = b + lane();
            uint32_t g = r < L ? q.x : 0u;
            int kv = skv(q);  // includes this iteration's chunk (added at admission)
            int now = uni(all_in ? 1 : 0);
            __asm__("" : "+s"(now));  // (the loop is not to be compiled twice)
            if (now) {
                const bool live = r < L && !(g & G_DONE), res = (g & G_RES) != 0;
                opened += popc(ballot(res && blocks(kv + 1) != blocks(kv)));
                kv += live ? min(sw(q) - kv, c.v) : 0;
                if (!res) g = (g & ~G_GUARD) | ((g >> G_LVL_SHIFT) & 31u);
                g |= live ? G_INB | G_RES : 0u;
            }
            // Per lane, as selects: the flag tests below are lane-dependent,
            // and a branch on them would cost scalar exec-mask work in every
            // chunk. Members advance; entries evicted in
            // this iteration lose the eviction mark.
            const bool memb = (g & G_INB) != 0;
            const bool evi = !memb && (g & G_EVI) != 0;
            int w = sw(q), left = sleft(q);
            const int idx = idx_of(pk);
            bad_idx = bad_idx || (memb && idx >= N.v);
            const bool emit = memb && kv == w && idx < N.v;
            const bool first = emit && !(g & G_FIRST);
            // times are kept modulo 2^32: a gap of 2^32 us or more overflows
            // the request's TTLT too
            const uint32_t gap = t32 - tg.x;
            const uint32_t gm = emit && !first && gap > tg.y ? gap : tg.y;
            w += emit ? 1 : 0;
            left -= emit ? 1 : 0;
            const bool fin = emit && left == 0;
            uint32_t gs = (memb ? g & ~G_INB : g & ~G_EVI) | (first ? G_FIRST : 0u);
            gs = fin ? (gs | G_DONE) & ~G_RES : gs;
            ufree += fin ? blocks(kv) : 0;
            kfree += fin ? kv : 0;
            if (first) tfirst()[idx] = t_end;
            if (fin) {
                tlast()[idx] = t_end;
                tbo()[idx] = gm;
            }
            kv = fin ? 0 : kv;
            const bool live = emit && !fin;  // emitted and has tokens left
            bool chg = false;
            uint64_t pk2 = pk;
            int ev = left;  // iterations to this member's next event
            if (pol == P_LAS) {
                // the attained service grew by one token
                chg = live;
                pk2 = chg ? pack((int64_t)w, idx) : pk;
            } else if (pol == P_SRPT || pol == P_TRAIL) {
                // remaining computed tokens (an evicted entry holds no KV)
                chg = (memb && !fin) || evi;
                pk2 = chg ? pack((int64_t)w + left - 1 - kv, idx) : pk;
            } else if (pol == P_BOOST) {
                const int lo_ = (int)((gs >> G_LVL_SHIFT) & 31u);
                int sig = w;  // P + dec
                int ln = lo_;
                if constexpr (EXT) {
                    // every lane reads: keep non-member lanes in bounds
                    const int ix = min(idx, N.v - 1);
                    if (phase_signal) sig = w - Pp()[ix];  // dec >= 1 after this token
                    if (cache_signal) sig = w - Hp()[ix];  // P - h + dec
                    if (phase_signal) ln = level_of(sig, k.v, lk.v);  // may fall at the first token
                }
                // the signal grows by one a token: the level follows when it
                // reaches the next threshold
                int thr = next_level(ln);
                const bool up = sig >= thr;
                ln += up ? 1 : 0;
                chg = live && ln != lo_;
                if (live) evx = min(evx, (thr << (up ? 1 : 0)) - sig);
                if (chg) {  // a level crossing (rare): re-key by the table step
                    pk2 = pack(key_of(pk) + S.bt[lo_] - S.bt[ln], idx);
                    gs = (gs & ~G_LVL) | ((uint32_t)ln << G_LVL_SHIFT);
                }
            }
            if constexpr (EXT) {
                if (pol == P_DIST && first && left > 0) {  // enters DistBoost's decode queue
                    pk2 = pack(t_end - kDecodeQueueOff, idx);
                    chg = true;
                } else if (pol == P_SARATHI && live) {
                    // round robin: back of the decode queue after each token
                    pk2 = pack(t_end - kDecodeQueueOff, idx);
                    chg = true;
                }
                if (pol == P_LTR && memb && !fin) {  // it ran: the count resets, or
                    if (!(gs & G_PROMO)) {           // a promotion spends its quantum
                        gs &= G_FLAGS;
                    } else if ((gs >> kLtrShift) <= 1u) {
                        gs = (gs & G_FLAGS & ~G_PROMO) | G_DIRTY;  // back to key D
                        pk2 = pack((int64_t)(w - Pp()[idx]) + left, idx);
                        chg = true;
                    } else {
                        gs -= 1u << kLtrShift;
                    }
                    if (gs & G_PROMO) ev = min(ev, max((int)(gs >> kLtrShift), 1));
                }
            }
            // SRPT's and TRAIL's re-keyed entries carry no re-insertion mark:
            // compaction extracts those that fall out of order
            const bool dirty = chg && pol != P_SRPT && pol != P_TRAIL;
            gs |= dirty ? G_DIRTY : 0u;
            const bool mute = memb && !emit;
            if (live) evl = min(evl, ev);
            if (memb || evi) {
                stq(r, gs, w, kv, left);
                if (chg) S.k[r] = pk2;
                S.tg[r] = make_uint2(emit ? t32 : tg.x, gm);
            }
            if constexpr (EXT) {
                // LTR+: a candidate that did not run starves one more
                // iteration; at the threshold it is promoted for a quantum
                if (pol == P_LTR && !memb && r < L && !(g & (G_DONE | G_PROMO))) {
                    const uint32_t cnt = (g >> kLtrShift) + 1u;
                    uint32_t gx = (g & G_FLAGS & ~G_EVI) | (cnt << kLtrShift);
                    if ((int)cnt >= ltr_s) {
                        gx = (g & G_FLAGS & ~G_EVI) | G_PROMO | G_DIRTY |
                             ((uint32_t)ltr_q << kLtrShift);
                        pk2 = pack(it_end - kPromotedOff, idx);
                        S.k[r] = pk2;
                        chg = true;
                    } else {
                        evl = min(evl, ltr_s - (int)cnt);
                    }
                    stx(r, gx);
                }
            }
            const uint64_t cm = ballot(chg), fm = ballot(fin);
            noemit |= ballot(mute);
            if (cm) {
                nmv += popc(cm);
                if (lo == INT32_MAX) lo = b + ffs0(cm);
            }
            if (fm) {
                if (lohole == INT32_MAX) lohole = b + ffs0(fm);
                nd += popc(fm);
                if (vm_ok && lane() == (b >> 6)) vm_res &= ~fm, vm_ev &= ~fm;
                if constexpr (EXT) {
                    if (ad) {  // end-to-end latencies enter the window in batch order
                        uint32_t lat = 0;
                        if (fin) {
                            const int64_t e2e = t_end - arr()[idx_of(pk)];
                            lat = e2e > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)e2e;
                        }
                        for (uint64_t m = fm; m; m &= m - 1)
                            ada_push((uint32_t)rl((int)lat, ffs0(m)));
                    }
                }
            }
            if (bn < 0) break;
            b = bn, q = qn, pk = pkn, tg = tgn;
        }
        wsync();
        if (ballot(bad_idx)) fail(S_ESTATE);
        all_emit = noemit == 0;
        nmoved = nmv;
        if (all_in) U += opened + new_blk;
        maxU = max(maxU.v, U);
        if (nd) {
            const int64_t kf = ctx_sum(kfree);
            U -= wsum(ufree);
            sum_ctx -= kf, kv_res -= kf;
            completed += nd;
            nR -= nd;
            n_holes += nd;
            lo_hole = min(lo_hole, lohole);
        }
        return lo;
    }

    // How many members of a repeated batch complete in its r-th iteration.
    DEV int completing(int r) const {
        int n = 0;
        for (uint64_t todo = emit_chunks; todo; todo &= todo - 1) {
            const int i = ffs0(todo) * kWave + lane();
            const uint4 q = ldq(min(i, L - 1));
            n += popc(ballot(i < L && i <= last && (q.x & G_RES) && sleft(q) == r));
        }
        return n;
    }

    // A run of repeated iterations (rep): the members are the first nb
    // residents, each takes one token per iteration, and nothing else changes until the
    // first event - a completion, a key that moves otherwise than with all
    // the others (an LTR+ promotion or demotion, with requests waiting also a
    // level crossing), an
    // arrival, a KV budget that the next blocks would exceed, `limit`
    // (CL), a new grid cell (adaptive gamma) or the iteration limit. The
    // outcome of r such iterations has a closed form per member, so they are
    // applied in one pass instead of r. The iterations' costs differ only in
    // the context sum, which grows by the members each time: lane j computes
    // the j-th cost and a prefix sum their end times, so the run is at most
    // 64 long. The events of the r-th iteration itself are applied too.
    // Returns r (0: the next iteration needs a formation, or the list an
    // insertion; nothing was done) and sets `lo` to the lowest rank that must
    // be re-inserted. `unsorted`: an earlier run moved keys, and the entries
    // were not re-inserted since.
    //
    // What bounds an instance is its own chain of iterations (about 10,000
    // cycles each for one formation and emission, on an idle or a full chip
    // alike), so fewer steps are worth more than cheaper ones: 64 to 97 % of
    // the iterations of the sweeps below the KV limit repeat the batch before
    // them, 5 to 25 in a row. Eight instances of 1,000 requests went from
    // 147 ms to 11.4 ms, 16,384 instances of 8,000 from 1,181 to 658 ms.
    DEV int streak(int64_t limit, bool unsorted, int &lo) {
        lo = INT32_MAX;
        nmoved = 0;
        // time: the r-th iteration starts before the next arrival and `limit`
        int room = sat31(limit - t);
        if (next < n_known()) {
            int off = next - pf;
            if (off >= kWave) {
                pf = next;
                load_pf();
                off = 0;
            }
            room = min(room, sat31(rl64(pa, off) - t));
        }
        const int64_t fixed = fixed_cost(nb);
        const int64_t top = sum_ctx + (int64_t)kWave * nb;  // the context of iteration 64
        if (UNLIKELY(((uint64_t)fixed >> 24) || (top >> 32))) return 0;
        const uint32_t qt = ctx_quot32((uint32_t)sum_ctx + (uint32_t)((lane() + 1) * nb));
        if (UNLIKELY((uint32_t)rl((int)qt, 63) >= (1u << 24))) return 0;
        const int cost = (int)fixed + (int)qt;
        const int tend = scan_add(cost);  // below 64 * 2^25
        int r = kWave;
        const uint64_t late = ballot(tend >= room);  // (a saturated room is never reached)
        if (late) r = ffs0(late) + 1;
        r = min(r, sat31(max_iters - iters));
        // (while nothing waits, the order of the members decides nothing but
        // the order in which latencies enter gamma's window: keys move at the
        // end of the run, and entries are re-inserted later)
        r = min(r, wmin(alone ? evl : min(evl, evx)));
        if constexpr (EXT) {
            // Latencies of one iteration enter the window in the order of the
            // keys it started with. Where a key moved before it, two requests
            // that complete in it need the list sorted first: the run ends an
            // iteration short of them. The adaptive sweep of 4,000 requests
            // takes 59.5 ms so, 66.1 ms with every run ended at a crossing
            // (58.2 ms in list order, which is wrong).
            if (ad && alone && (unsorted || wmin(evx) < r) && completing(r) > 1) r--;
        }
        if (r <= 0) return 0;
        // KV: every iteration's new blocks fit (the growth only adds up, so the
        // last one's total decides); halved until they do
        while (UNLIKELY(nb * blocks(r) > Kb - U)) {
            int grow = 0;
            for (uint64_t todo = emit_chunks; todo; todo &= todo - 1) {
                const int i = ffs0(todo) * kWave + lane();
                const uint4 q = ldq(min(i, L - 1));
                grow += growth(i < L && i <= last && (q.x & G_RES), skv(q), r);
            }
            if (grow <= Kb - U) break;
            r >>= 1;
            if (r == 0) return 0;
        }
        if constexpr (EXT) {
            if (ad) {
                r = ada_hold(r);
                if (r == 0) return 0;
            }
        }
        if constexpr (kCheck) {
            check_run(r);
            if (status) return 0;
        }
        // apply r iterations (counted before the loop: a sum the compiler also finds
        // in a lane's branch would make the count lane-dependent)
        const int64_t it_end = (int64_t)sgpr64((uint64_t)(iters + r));
        due = rl(tend, r - 1) >= room;
        const int64_t t_end = t + rl(tend, r - 1);
        const uint32_t t32 = (uint32_t)t_end, gap = (uint32_t)rl(cost, r - 1);  // costs never shrink
        int lohole = INT32_MAX, nd = 0, grow = 0, ufree = 0, kfree = 0;
        // LTR+ counts every candidate's starvation: visit every chunk
        const int nch = (L + kWave - 1) >> 6;
        const uint64_t chunks =
            EXT && pol == P_LTR ? (nch >= 64 ? ~0ull : ((1ull << nch) - 1ull)) : emit_chunks;
        evl = evx = INT32_MAX;
        for (uint64_t todo = chunks; todo; todo &= todo - 1) {
            const int b = ffs0(todo) * kWave;
            const int i = b + lane(), i0 = min(i, L - 1);
            const uint4 q = ldq(i0);
            const uint2 tg = S.tg[i0];
            const uint32_t g = i < L ? q.x : 0u;
            const bool memb = (g & G_RES) != 0 && i <= last;
            const int w = sw(q) + r, left = sleft(q) - r;
            int kv = skv(q);
            grow += growth(memb, kv, r);
            kv += r;
            int ev = left;
            const bool fin = memb && left == 0;
            ufree += fin ? blocks(kv) : 0;
            kfree += fin ? kv : 0;
            uint32_t gs = fin ? (g | G_DONE) & ~G_RES : g;
            const uint32_t gm = gap > tg.y ? gap : tg.y;
            const uint64_t fm = ballot(fin);
            if (fm) {
                const int idx = idx_of(S.k[i0]);
                if (fin) {
                    tlast()[idx] = t_end;
                    tbo()[idx] = gm;
                }
                if (lohole == INT32_MAX) lohole = b + ffs0(fm);
                nd += popc(fm);
                if (vm_ok && lane() == (b >> 6)) vm_res &= ~fm, vm_ev &= ~fm;
                if constexpr (EXT) {
                    if (ad) {
                        uint32_t lat = 0;
                        if (fin) {
                            const int64_t e2e = t_end - arr()[idx];
                            lat = e2e > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)e2e;
                        }
                        for (uint64_t m = fm; m; m &= m - 1)
                            ada_push((uint32_t)rl((int)lat, ffs0(m)));
                    }
                }
            }
            uint64_t cm = 0;  // entries to re-insert
            if (pol == P_BOOST) {
                const int ol = (int)((g >> G_LVL_SHIFT) & 31u);
                int sig = w;
                if constexpr (EXT) {
                    if (phase_signal || cache_signal) {
                        const int ix = min(idx_of(S.k[i0]), N.v - 1);
                        sig -= phase_signal ? Pp()[ix] : Hp()[ix];
                    }
                }
                int thr = next_level(ol);
                const bool chg = memb && !fin && sig >= thr;
                cm = ballot(chg);
                if (cm) {
                    const uint64_t pk = S.k[i0];
                    if (chg) {
                        const int nl = level_of(sig, k.v, lk.v);
                        thr = next_level(nl);
                        S.k[i] = pack(key_of(pk) + S.bt[ol] - S.bt[nl], idx_of(pk));
                        gs = (gs & ~G_LVL) | ((uint32_t)nl << G_LVL_SHIFT) | G_DIRTY;
                    }
                }
                if (memb && !fin) evx = min(evx, thr - sig);
            } else if (pol == P_SRPT || pol == P_TRAIL || pol == P_LAS) {
                // every member's key moves by r; holes among them move along, so
                // that the residents and holes stay in order
                const uint64_t d = (uint64_t)(uint32_t)r << kIdxBits;
                const uint64_t pk = S.k[i0];
                if (memb || ((g & G_DONE) && i <= last)) S.k[i] = pol == P_LAS ? pk + d : pk - d;
                // past a waiting entry, perhaps: compaction finds those
                if (pol != P_LAS && nW > 0) cm = ballot(memb && !fin);
            }
            if constexpr (EXT) {
                if (pol == P_SARATHI) {  // all to the same, latest key: they stay in order
                    const int idx = idx_of(S.k[i0]);
                    if (memb && !fin) S.k[i] = pack(t_end - kDecodeQueueOff, idx);
                    wsync();  // (joins the lanes before the branches on the policy do)
                } else if (pol == P_LTR) {
                    bool chg = false;
                    const uint64_t pk = S.k[i0];
                    if (memb && !fin) {
                        const int quota = (int)(g >> kLtrShift);
                        if (!(g & G_PROMO)) {
                            gs &= G_FLAGS;
                        } else if (quota <= r) {  // the quantum ends: back to key D
                            gs = (gs & G_FLAGS & ~G_PROMO) | G_DIRTY;
                            const int idx = idx_of(pk);
                            S.k[i] = pack((int64_t)(w - Pp()[idx]) + left, idx);
                            chg = true;
                        } else {
                            gs -= (uint32_t)r << kLtrShift;
                        }
                        if (gs & G_PROMO) ev = min(ev, max((int)(gs >> kLtrShift), 1));
                    } else if (i < L && !memb && !(g & (G_DONE | G_PROMO))) {
                        const uint32_t c2 = (g >> kLtrShift) + (uint32_t)r;
                        uint32_t gx = (g & G_FLAGS) | (c2 << kLtrShift);
                        if ((int)c2 >= ltr_s) {  // promoted at the end of the r-th iteration
                            gx = (g & G_FLAGS) | G_PROMO | G_DIRTY |
                                 ((uint32_t)ltr_q << kLtrShift);
                            S.k[i] = pack(it_end - kPromotedOff, idx_of(pk));
                            chg = true;
                        } else {
                            evl = min(evl, ltr_s - (int)c2);
                        }
                        stx(i, gx);
                    }
                    cm = ballot(chg);
                }
            }
            if (memb) {
                stq(i, gs, w, fin ? 0 : kv, left);
                S.tg[i] = make_uint2(t32, gm);
                if (!fin) evl = min(evl, ev);
            }
            if (cm) {
                nmoved += popc(cm);
                if (lo == INT32_MAX) lo = b + ffs0(cm);
            }
        }
        wsync();
        if (pol == P_TRAIL) vm_ok = false;  // eligibility depends on progress
        iters = it_end;
        ev_vol = ev_forced = 0;
        tally(r * nb, r * nb, 4 + 3 * popc(chunks));
        sum_ctx += r * nb, kv_res += r * nb;
        U += grow;
        maxU = max(maxU.v, U);
        if (nd) {
            const int64_t kf = ctx_sum(kfree);
            U -= wsum(ufree);
            sum_ctx -= kf, kv_res -= kf;
            completed += nd;
            nR -= nd;
            n_holes += nd;
            lo_hole = min(lo_hole, lohole);
        }
        t = t_end;
        return r;
    }

    // From rank `from` on: remove holes; extract entries whose key moved
    // (flagged, or below the running maximum of the entries kept before them)
    // into `stage` (lanes [0, min(count, 64))) and, beyond 64, the HBM
    // overflow. Returns the number extracted. No holes lie below `from`.
    DEV int compact_extract(int from, R &stage) {
        vm_ok = false;
        const int start = (from >> 6) << 6;
        uint64_t pmax = start > 0 ? uniu(S.k[start - 1]) : 0ull;
        int out = start, nx = 0;
        for (int b = start; b < L; b += kWave) {
            const int r = b + lane();
            const bool v = r < L;
            R y;
            if (v) ldr(r, y);
            const bool dead = v && (y.gs & G_DONE);
            const bool dirty = v && (y.gs & G_DIRTY);
            const uint64_t val = (v && !dead && !dirty) ? y.pk : 0ull;
            const uint64_t inc = scan_maxu(val);
            uint64_t exc = prev_lane_u64(inc, 0ull);
            if (pmax > exc) exc = pmax;
            const bool ext = v && !dead && (dirty || y.pk < exc);
            const bool keep = v && !dead && !ext;
            const uint64_t km = ballot(keep), xm = ballot(ext);
            wsync();
            if (keep) {
                const int d = out + mbcnt(km);
                if (d != r) str(d, y);
            }
            if (ext) {
                y.gs &= ~G_DIRTY;
                const int xi = nx + mbcnt(xm);
                if (xi >= kStage) ovf()[xi - kStage] = to_rec(y);
            }
            wsync();
            if (xm && nx < kStage) {  // the first kStage extracted stay in registers
                const uint64_t sm = ballot(ext && nx + mbcnt(xm) < kStage);
                const R z = permute_rec(y, place_dest(sm, nx));
                if (lane() >= nx && lane() < nx + popc(sm)) stage = z;
            }
            const uint64_t cm = rlu(inc, 63);
            if (cm > pmax) pmax = cm;
            out += popc(km);
            nx += popc(xm);
        }
        L = out;
        n_holes = 0;
        lo_hole = INT32_MAX;
        return nx;
    }

    // Whether the entries from rank `from` on, completed ones aside, are in
    // ascending order; if so, their re-keyed entries stay where they are
    // (their flags are cleared). No holes lie below `from`.
    DEV bool settle_in_place(int from) {
        const int start = (from >> 6) << 6;
        uint64_t pmax = start > 0 ? uniu(S.k[start - 1]) : 0ull;
        for (int b = start; b < L; b += kWave) {
            const int r = b + lane();
            const bool v = r < L && !(ldx(r) & G_DONE);
            const uint64_t pk = r < L ? S.k[r] : 0ull;
            const uint64_t inc = scan_maxu(v ? pk : 0ull);
            uint64_t exc = prev_lane_u64(inc, 0ull);
            if (pmax > exc) exc = pmax;
            if (ballot(v && pk < exc)) return false;
            const uint64_t cm = rlu(inc, 63);
            if (cm > pmax) pmax = cm;
        }
        for (int b = start; b < L; b += kWave) {
            const int r = b + lane();
            if (r < L) {
                const uint32_t g = ldx(r);
                if (g & G_DIRTY) stx(r, g & ~G_DIRTY);
            }
        }
        wsync();
        return true;
    }

    // The list is in key order except for the resident entry at rank r, whose
    // key moved: put it at its rank among the others, shifting the entries
    // in between by one slot (one pass over them, instead of extracting the
    // tail of the list and merging it back). Holes keep their stale keys,
    // which are in order, and move with the others.
    DEV void move_one(int r) {
        vm_ok = false;
        R x;
        ldr(r, x);  // every lane reads the entry (one address)
        x.gs &= ~G_DIRTY;
        const uint64_t key = x.pk;
        // its new rank: the entries other than it with smaller keys. Entries
        // before r had keys below its old key and after r above it, so only
        // one side is counted, chunk by chunk, until a chunk lies beyond.
        int to;
        const bool right = r + 1 < L && uniu(S.k[r + 1]) < key;
        if (right) {
            to = r;
            for (int b = ((r + 1) >> 6) << 6; b < L; b += kWave) {
                const int i = b + lane();
                const bool lt = i > r && i < L && S.k[i] < key;
                const uint64_t m = ballot(lt);
                to += popc(m);
                if (popc(m) < min(L, b + kWave) - max(b, r + 1)) break;
            }
        } else {
            to = r;
            for (int b = ((r - 1) >> 6) << 6; b >= 0 && r > 0; b -= kWave) {
                const int i = b + lane();
                const bool gt = i < r && S.k[i] > key;
                const uint64_t m = ballot(gt);
                to -= popc(m);
                if (popc(m) < min(r, b + kWave) - b) break;
            }
        }
        wsync();
        if (to > r) {  // entries r+1 .. to move down one slot, in ascending chunks
            for (int b = ((r + 1) >> 6) << 6; b <= to; b += kWave) {
                const int i = b + lane();
                const bool mv = i > r && i <= to;
                R y;
                if (mv) ldr(i, y);
                wsync();
                if (mv) str(i - 1, y);
                wsync();
            }
            if (lo_hole > r && lo_hole <= to) lo_hole--;
        } else if (to < r) {  // entries to .. r-1 move up one slot, in descending chunks
            for (int b = ((r - 1) >> 6) << 6; b >= 0 && b + kWave > to; b -= kWave) {
                const int i = b + lane();
                const bool mv = i >= to && i < r;
                R y;
                if (mv) ldr(i, y);
                wsync();
                if (mv) str(i + 1, y);
                wsync();
            }
            if (lo_hole >= to && lo_hole < r) lo_hole++;
        }
        if (lane() == 0) str(to, x);
        wsync();
    }

    // The members of a repeated batch: emit_chunks := the 64-entry chunks
    // holding the first nb residents; returns the rank of the last of them.
    DEV int find_members() {
        uint64_t m = 0;
        int left = nb, at = -1;
        for (int b = 0; b < L; b += kWave) {
            const int r = b + lane();
            const bool res = r < L && (ldx(r) & G_RES);
            const uint64_t rm = ballot(res);
            if (!rm) continue;
            m |= 1ull << (b >> 6);
            if (popc(rm) >= left) {
                at = b + ffs0(ballot(res && mbcnt(rm) == left - 1));
                break;
            }
            left -= popc(rm);
        }
        emit_chunks = m;
        return at;
    }

    // Returns whether entries may have moved to other ranks.
    DEV bool maintenance(int lo_mod) {
        bool edited = false;
        if constexpr (EXT) {
            // Sarathi moves every decode that emitted to the same, latest key:
            // when all decodes were in the batch (steady decoding) the list
            // is still in order and nothing needs re-inserting
            if (pol == P_SARATHI && lo_mod < L && n_holes < kHoleLimit && L <= cap_now() &&
                settle_in_place(min(lo_mod, lo_hole)))
                lo_mod = L;
        }
        if (nmoved == 1 && lo_mod < L && n_holes < kHoleLimit && L <= cap_now() &&
            (ldx(lo_mod) & G_RES)) {
            move_one(lo_mod);  // one resident re-keyed (a level crossing, say)
            lo_mod = L;
            edited = true;
        }
        if (UNLIKELY(lo_mod < L || n_holes >= kHoleLimit || L > cap_now())) {
            R stage;
            edited = true;
            const int nx = compact_extract(min(min(lo_mod, lo_hole), L), stage);
            if (nx > kStage) hbm_fence();
            if (L > cap_now()) spill_excess();  // a refill during formation used the overflow region
            if (nx > 0 && status == 0) {
                add_entries(stage, min(nx, kStage));
                for (int b = kStage; b < nx && status == 0; b += kStage) {
                    const int kb = min(nx - b, kStage);
                    R x;
                    if (lane() < kb) x = from_rec(ovf()[b - kStage + lane()]);
                    add_entries(x, kb);
                }
            }
        }
        if (status == 0) take_arrivals();
        return edited;
    }

    // ---------------------------------------------------------- adaptive gamma

    // Entries of the sorted window (n of them) below x.
    DEV int window_below(uint32_t x, int n) const {
        int c = 0;
        for (int b = 0; b < n; b += kWave) {
            const int r = b + lane();
            c += popc(ballot(r < n && S.ws[r] < x));
        }
        return c;
    }

    // UpdateStats (Algorithm 1): the end-to-end latency x (wave-uniform) of a
    // completed request enters the window; when it is full the oldest leaves.
    // The ring keeps completion order, the sorted copy serves the percentiles.
    DEV void ada_push(uint32_t x) {
        AdaLds &G = *S.as;
        int n = uni(G.wn);
        const int W = uni(G.window), head = uni(G.whead);
        if (n == W) {  // drop the oldest: close the gap at its first copy
            const uint32_t old = (uint32_t)uni((int)S.wr[head]);
            const int po = window_below(old, n);
            for (int b = ((po + 1) >> 6) << 6; b < n; b += kWave) {
                const int r = b + lane();
                const bool mv = r > po && r < n;
                uint32_t v = 0;
                if (mv) v = S.ws[r];
                wsync();
                if (mv) S.ws[r - 1] = v;
                wsync();
            }
            n--;
        }
        const int pn = window_below(x, n);  // open a slot at the insertion rank
        for (int b = ((n - 1) >> 6) << 6; b >= 0 && b + kWave > pn; b -= kWave) {
            const int r = b + lane();
            const bool mv = r >= pn && r < n;
            uint32_t v = 0;
            if (mv) v = S.ws[r];
            wsync();
            if (mv) S.ws[r + 1] = v;
            wsync();
        }
        if (lane() == 0) {
            S.ws[pn] = x;
            S.wr[head] = x;
            G.whead = head + 1 == W ? 0 : head + 1;
            G.wn = n + 1;
            G.wnew = 1;
        }
        wsync();
    }

    // gamma_hat for the window of wn >= min_samples latencies (the stored
    // estimate while the window has not changed).
    DEV double ada_ghat(int wn) const {
#pragma clang fp contract(off)
        const AdaLds &G = *S.as;
        if (!uni(G.wnew)) return G.ghat;
        const int r95 = (95 * wn + 99) / 100, r99 = (99 * wn + 99) / 100;
        const uint32_t t95 = S.ws[r95 - 1], t99 = S.ws[r99 - 1];
        double d = (double)(t99 - t95);
        if (d < ad->eps) d = ad->eps;
        return ad->num / d;
    }

    // UpdateGamma over up to r iterations in which no request completes:
    // every update is the one ada_update makes, until one would move to
    // another grid cell. Returns how many stay in the cell (at most r) and
    // stores the state after them.
    DEV int ada_hold(int r) {
#pragma clang fp contract(off)
        AdaLds &G = *S.as;
        const int wn = uni(G.wn);
        if (wn < uni(G.min_samples)) return r;
        const double gh = ada_ghat(wn);
        const int cell = uni(G.cell);
        const double keep = 1.0 - ad->beta, pull = ad->beta * gh;
        const double gmin = ad->gmin, gmax = ad->gmax;
        double g = G.gamma;
        int j = 0;
        for (; j < r; j++) {
            double x = keep * g + pull;
            if (x < gmin) x = gmin;
            if (x > gmax) x = gmax;
            if (popc(ballot(x >= bnd)) != cell) break;
            if (!ballot(x != g)) {  // a fixed point: every later update gives it again
                j = r;
                break;
            }
            g = x;
        }
        wsync();
        if (j > 0 && lane() == 0) G.gamma = g, G.ghat = gh, G.wnew = 0;
        wsync();
        return j;
    }

    // UpdateGamma (Phase 4, Algorithm 2), before the keys of every iteration:
    // with at least min_samples latencies in the window, gamma_hat =
    // tau ln 5 / max(t99 - t95, eps) from the nearest-rank t95, t99 (only
    // recomputed when the window changed), then gamma = clip((1 - beta) gamma
    // + beta gamma_hat); each is one rounded double operation (no contraction).
    // A new grid cell re-keys every waiting and resident request.
    DEV void ada_update() {
#pragma clang fp contract(off)
        AdaLds &G = *S.as;
        const int wn = uni(G.wn);
        if (wn < uni(G.min_samples)) return;
        const double gh = ada_ghat(wn);
        double g = (1.0 - ad->beta) * G.gamma + ad->beta * gh;
        if (g < ad->gmin) g = ad->gmin;
        if (g > ad->gmax) g = ad->gmax;
        const int cell = popc(ballot(g >= bnd));
        const int old = uni(G.cell);
        wsync();
        if (lane() == 0) {
            G.ghat = gh, G.wnew = 0;
            G.gamma = g;
            if (cell != old) G.cell = cell, G.switches++;
        }
        wsync();
        if (cell != old) ada_rekey(cell);
    }

    // The boost table changes to that of `cell`: keys a - bt[level] of the
    // spilled, waiting and resident entries shift by bt_old - bt_new of their
    // level; every on-chip entry is then re-inserted, so waiting entries above
    // the new spill minimum move to the spill and the list is sorted again.
    DEV void ada_rekey(int cell) {
        const int64_t *nt = ad->table[cell];
        hbm_fence();
        Rec *const spill = this->spill();
        uint64_t mn = ~0ull;
        for (int b = 0; b < spill_n; b += kWave) {
            const int i = b + lane();
            if (i < spill_n) {
                const uint64_t pk = spill[i].pk;
                const int lv = min((int)((spill[i].gs >> G_LVL_SHIFT) & 31u), kLevels - 1);
                const uint64_t pk2 = pack(key_of(pk) + S.bt[lv] - nt[lv], idx_of(pk));
                spill[i].pk = pk2;
                mn = pk2 < mn ? pk2 : mn;
            }
        }
        spill_min = wminu(mn);
        for (int b = 0; b < L; b += kWave) {
            const int r = b + lane();
            if (r < L) {
                const uint32_t g = ldx(r);
                if (!(g & G_DONE)) {
                    const int lv = min((int)((g >> G_LVL_SHIFT) & 31u), kLevels - 1);
                    const uint64_t pk = S.k[r];
                    S.k[r] = pack(key_of(pk) + S.bt[lv] - nt[lv], idx_of(pk));
                    stx(r, g | G_DIRTY);
                }
            }
        }
        int64_t v = 0;
        if (lane() < kLevels) v = nt[lane()];
        wsync();
        if (lane() < kLevels) S.bt[lane()] = v;
        wsync();
        R stage;
        const int nx = compact_extract(0, stage);  // every live entry is flagged
        if (nx > kStage) hbm_fence();
        if (nx > 0 && status == 0) {
            add_entries(stage, min(nx, kStage));
            for (int b = kStage; b < nx && status == 0; b += kStage) {
                const int kb = min(nx - b, kStage);
                R x;
                if (lane() < kb) x = from_rec(ovf()[b - kStage + lane()]);
                add_entries(x, kb);
            }
        }
    }

    // ---------------------------------------------------------- checks

    // The batch just formed respects the sequence cap, the token budget and
    // the KV budget, and every member computes at least one token.
    // Before a run of r repeated iterations is applied: its members are the
    // first nb residents, all within the chunks that the run visits, each
    // needs one token at a time and has r left; the batch respects its caps
    // and the blocks it grows by the KV budget; and, with adaptive gamma,
    // those that complete stand in the order of the keys that the r-th
    // iteration starts with.
    DEV void check_run(int r) {
        bool bad = r < 1 || r > kWave || nb < 1 || nb > M || nb > T;
        int n = 0, grow = 0;
        uint64_t top = 0;  // 1 + the largest key of those that complete so far (0: none)
        for (int b = 0; b < L && !bad; b += kWave) {
            const int i = b + lane();
            const uint4 q = ldq(min(i, L - 1));
            const uint32_t g = i < L ? q.x : 0u;
            const bool memb = (g & G_RES) != 0 && i <= last;
            const int w = sw(q), kv = skv(q), left = sleft(q);
            n += popc(ballot(memb));
            grow += growth(memb, kv, r);
            bad = bad || ballot(memb && (kv + 1 != w || left < r || (g & (G_INB | G_EVI)))) != 0;
            bad = bad || (ballot(memb) && !((emit_chunks >> (b >> 6)) & 1ull));
            if constexpr (EXT) {
                if (ad) {
                    const uint64_t pk = S.k[min(i, L - 1)];
                    const int ix = min(idx_of(pk), N.v - 1);
                    int sig = w + r - 1;
                    if (phase_signal) sig -= Pp()[ix];
                    if (cache_signal) sig -= Hp()[ix];
                    const int ol = (int)((g >> G_LVL_SHIFT) & 31u), nl = level_of(sig, k.v, lk.v);
                    const uint64_t at = pack(key_of(pk) + S.bt[ol] - S.bt[nl], ix);
                    for (uint64_t m = ballot(memb && left == r); m; m &= m - 1) {
                        const uint64_t x = rlu(at, ffs0(m)) + 1;
                        bad = bad || x <= top;
                        top = x;
                    }
                }
            }
        }
        if (bad || n != nb || grow > Kb - U) fail(S_ESTATE);
    }

    DEV void check_batch() {
        if (cnt < 1 || cnt > M || used < cnt || used > T || U < 0 || U > Kb) fail(S_ESTATE);
    }

    // The state between steps: the list's residents, waiting entries
    // and holes match their counts; the KV in use is the residents' blocks,
    // within the budget, and their tokens the running sum; the keys of the entries other than holes ascend
    // strictly; holes lie at or after lo_hole; no mark of an iteration (in
    // the batch, evicted, selected for spilling, key moved) survives it; an
    // entry's KV lies within its signal and a waiting entry holds none; the
    // spill holds waiting entries only, its minimum is exact; and every
    // request taken so far is done, on chip or spilled.
    DEV void check_state() {
        bool bad = U < 0 || U > Kb || L < 0 || L > cap_now() || spill_n < 0 || spill_n > scap();
        int nres = 0, nwait = 0, nhole = 0, blk = 0;
        uint32_t kvs = 0;
        uint64_t pmax = 0;  // 1 + the largest key of the live entries so far (0: none)
        for (int b = 0; b < L && !bad; b += kWave) {
            const int r = b + lane();
            const bool v = r < L;
            const int i = min(r, L - 1);  // lanes past the list read its last slot
            const uint4 q = ldq(i);
            const uint32_t g = q.x;
            const uint64_t pk = S.k[i];
            const bool done = v && (g & G_DONE) != 0;
            const bool live = v && !done;
            const bool rs = live && (g & G_RES) != 0;
            const bool wt = live && (g & G_RES) == 0;
            const int w = sw(q), kv = skv(q), left = sleft(q);
            nres += rs ? 1 : 0;
            nwait += wt ? 1 : 0;
            nhole += done ? 1 : 0;
            blk += rs ? blocks(kv) : 0;
            kvs += rs ? (uint32_t)kv : 0u;
            const uint64_t inc = scan_maxu(live ? pk + 1 : 0ull);
            uint64_t exc = prev_lane_u64(inc, 0ull);
            if (pmax > exc) exc = pmax;
            bool e = v && (g & (G_INB | G_EVI | G_MARK)) != 0;
            e = e || (live && (g & G_DIRTY) != 0);
            e = e || (live && pk + 1 <= exc);  // not above a live key before it
            e = e || (done && r < lo_hole);
            e = e || (live && (kv < 0 || kv > w || left < 1 || idx_of(pk) >= N.v));
            e = e || (wt && kv != 0);
            bad = bad || ballot(e) != 0;
            const uint64_t cm = rlu(inc, 63);
            if (cm > pmax) pmax = cm;
        }
        if (!bad) {
            nres = wsum(nres), nwait = wsum(nwait), nhole = wsum(nhole), blk = wsum(blk);
            bad = nres != nR || nwait != nW || nhole != n_holes || blk != U ||
                  (uint32_t)wsum((int)kvs) != (uint32_t)kv_res ||
                  completed + nR + nW + spill_n != next;
        }
        if (!bad && spill_n > 0) {
            hbm_fence();
            uint64_t mn = ~0ull;
            bool e = false;
            for (int b = 0; b < spill_n; b += kWave) {
                const int i = b + lane();
                if (i < spill_n) {
                    const Rec x = spill()[i];
                    if (x.pk < mn) mn = x.pk;
                    e = e || (x.gs & (G_RES | G_DONE | G_INB | G_EVI | G_MARK | G_DIRTY)) != 0 ||
                        x.kv != 0 || x.left < 1 || idx_of(x.pk) >= N.v;
                }
            }
            bad = ballot(e) != 0 || wminu(mn) != spill_min;
        }
        if (bad) fail(S_ESTATE);
    }

    // ---------------------------------------------------------- driver

    // TRAIL: whether the token budget clips, or could come to clip, the chunk
    // of the waiting request that closed admissions, the first on the list,
    // as members that ranked behind it come to rank before it.
    DEV bool may_clip() const {
        for (int b = 0; b < L; b += kWave) {
            const int i = b + lane();
            const uint4 q = ldq(min(i, L - 1));
            const uint64_t wm = ballot(i < L && is_waiting(q.x));
            if (wm) return min(rl(sw(q), ffs0(wm)), (int)c) > T - nb;
        }
        return false;
    }

    // Whether a batch that repeats but for the requests that arrived since
    // `next0` still does: those are met after admissions close, or not at
    // all because the batch is full before them, or nothing arrived. Finds
    // the members again where ranks may have moved (`moved`).
    DEV bool arrivals_keep(int next0, bool moved) {
        const bool full = nb == M;
        if constexpr (EXT) {
            if (pol == P_LTR && next != next0) evl = min(evl, ltr_s);  // they start to starve
        }
        last = INT32_MAX;
        uint64_t bar = close_pk;
        if (moved || full) {
            const int at = find_members();
            if (full && at >= 0) {
                last = at;
                const uint64_t pk = uniu(S.k[at]);
                bar = sgpr64(pk < bar ? pk : bar);
            }
        }
        if (next != next0 && (bar == ~0ull || ballot(arr_pk <= bar))) return false;
        return pol != P_TRAIL || close_pk == ~0ull || !may_clip();
    }

    // Sarathi: the first live entry of the list is a resident, so no waiting
    // request that emitted tokens (whose older decode-queue key ranks ahead
    // of every resident served just now) is met before them.
    DEV bool resident_first() const {
        for (int b = 0; b < L; b += kWave) {
            const int i = b + lane();
            const uint32_t g = i < L ? ldx(i) : G_DONE;
            const uint64_t live = ballot(!(g & G_DONE)), res = ballot((g & G_RES) != 0);
            if (live)
                return ((res >> ffs0(live)) & 1ull) &&
                       (spill_n == 0 || spill_min > uniu(S.k[b + ffs0(live)]));
        }
        return false;
    }

    // Nothing waited and every resident needs one token; then requests
    // arrived. If they all fit beside the residents, the next iteration
    // takes everything, in whatever order: emission admits it in its pass and
    // no formation is needed.
    DEV void plan_join() {
        join = nW > 0 && spill_n == 0 && nR + nW <= M && new_tok <= T - nR &&
               nR + new_blk <= Kb - U;
    }

    // One iteration, or a run of repeated ones; then the list's maintenance
    // and the arrivals. `limit`: see streak.
    DEV void step(int64_t limit) {
        const int c0 = completed;
        int lo_mod;
        // Does the next iteration repeat this one's batch? `again`: every
        // member emitted a token, so each needs exactly one next; `whole`:
        // the members are all the residents; `stays`: formation evicted
        // nothing, refilled nothing and stopped short of the token budget.
        bool again = true, whole = last == INT32_MAX || nb == nR, stays = true;
        bool run = false;
        int lo_pend = INT32_MAX, nm_pend = 0;  // entries to re-insert: lowest rank, how many
        while (rep) {
            const int c1 = completed;
            int lo;
            if (streak(limit, lo_pend != INT32_MAX, lo) == 0) break;
            run = true;
            lo_pend = min(lo_pend, lo);
            nm_pend += nmoved;
            last_done = completed - c1;
            // nothing waits or arrived: straight on, the order can wait
            if (!alone || due || nR == 0 || n_holes >= kHoleLimit) break;
            nb = nR;
        }
        if constexpr (kCheck) {
            if (status) return;
        }
        if (run) {
            lo_mod = lo_pend, nmoved = nm_pend;
        } else {
            if constexpr (EXT) {
                if (ad) {
                    ada_update();
                    if (status) return;
                }
            }
            if (join) {
                cnt = nR + nW, used = nR + new_tok;
                nR += nW, nW = 0;
                kv_res += used;
                sum_ctx = kv_res;
                close_pk = ~0ull;
                ev_vol = ev_forced = fpass = 0;
                emit_all = vm_ok = false;
            } else {
                formation();
                if (status) return;
                if (cnt == 0) {
                    fail(S_ESTATE);
                    return;
                }
            }
            if constexpr (kCheck) {
                check_batch();
                if (status) return;
            }
            whole = cnt == nR;
            nb = cnt;
            stays = ev_vol + ev_forced == 0 && !emit_all && used < T;
            const int64_t dt = fixed_cost(used) + (int64_t)ctx_quot((uint64_t)sum_ctx);
            const int64_t t_end = t + dt;
            const int c1 = completed;
            lo_mod = emission(t_end, join);
            last_done = completed - c1;
            join = false;
            again = all_emit;
            t = t_end;
            iters = iters.v + 1;
            tally(cnt, used, 4 + 5 * fpass + 3 * n_chunks);
            if (less64(max_iters, iters)) {
                fail(S_ELIVELOCK);
                return;
            }
        }
        const int next0 = next, sp0 = n_spilled;
        const bool none = nW == 0 && spill_n == 0;  // nothing waited before the arrivals
        arr_pk = ~0ull;
        new_tok = new_blk = 0;
        const bool edited = maintenance(lo_mod);
        // A member in its prefill: nothing below applies. Out before the
        // state that the tests need comes back from spilled scalars: 5 % off
        // LTR+ and 3 % off Sarathi on the reasoning law, 1 % off the
        // reasoning sweep, 2 % off LAS trading residents at a full budget.
        if (!again) {
            rep = alone = false;
            if constexpr (kCheck) {
                if (status == 0) check_state();
            }
            return;
        }
        // A whole batch repeats (as far as the KV budget allows: see streak)
        // if nothing waits. With requests waiting, or residents left out of
        // a full batch, it repeats if nothing completed, no key moved and
        // the list kept its waiting entries: a waiting candidate the next
        // formation meets with admissions open met them in this formation
        // too, did not fit and found no eligible victim; the KV held before
        // it has not shrunk, its own chunk has not shrunk, and the residents
        // after it are the same with the same keys and eligibility, so it
        // closes admissions again. A full batch (max_seqs) ends the
        // formation at its last member. Keys that all fall together (SRPT,
        // TRAIL) only take residents from behind a waiting candidate to
        // before it, where they hold the same KV and are no victims, so those
        // batches repeat too. But they also take a token each there, and the
        // token budget may then clip the candidate's chunk to one that fits:
        // under TRAIL, whose protected residents stay behind a candidate that
        // found no victim (SRPT's do not), its chunk must fit beside the
        // whole batch (see may_clip). Sarathi's batches, which all move to the
        // latest time, repeat as long as no resident is left out and no
        // waiting request ranks before them (it takes no victims by
        // priority). LAS's keys grow, past the waiting ones: excluded.
        alone = whole && nW == 0 && spill_n == 0;
        bool ok = stays && completed == c0 && pol != P_LAS && n_spilled == sp0 &&
                  (whole || nb == M);
        if (lo_mod != INT32_MAX && pol != P_SRPT && pol != P_TRAIL) {
            if constexpr (EXT) ok = ok && pol == P_SARATHI;
            else ok = false;
        }
        if constexpr (EXT) {
            if (ok && pol == P_SARATHI && !alone) ok = whole && resident_first();
        }
        rep = nR > 0 && (alone || ok);
        if (rep) {
            if (alone) {
                nb = nR, last = INT32_MAX;
                if (edited || emit_all || next != next0) find_members();
            } else {
                rep = arrivals_keep(next0, edited || emit_all || next != next0);
            }
        }
        alone = alone && rep;
        if (!rep && whole && none) plan_join();
        if constexpr (kCheck) {
            if (status == 0) check_state();
        }
    }

    DEV void run() {
        load_pf();
        take_arrivals();
        for (;;) {
            if (status) break;
            if (UNLIKELY(nW + nR == 0)) {
                if (spill_n > 0) {
                    refill();
                    if (status) break;
                    if (nW + nR == 0) {
                        fail(S_ESTATE);
                        break;
                    }
                    continue;
                }
                if (next >= N) break;
                int off = next - pf;
                if (off >= kWave) {
                    pf = next;
                    load_pf();
                    off = 0;
                }
                const int64_t an = rl64(pa, off);
                if (lane() == 0) S.ty[TY_IDLE] += (uint64_t)(an - t);
                t = an;
                take_arrivals();
                continue;
            }
            step(INT64_MAX);
        }
        finish();
    }

    // CL: simulate while the replica has work and its clock is below `limit`,
    // the next arrival time of the global trace (an iteration that starts
    // before it is formed without that request); then wait for the router.
    // With limit = INT64_MAX it runs to the end of what was dispatched.
    DEV void run_until(int64_t limit) {
        if (status) return;
        const int next0 = next, sp0 = n_spilled;
        arr_pk = ~0ull;
        if (!join) new_tok = new_blk = 0;
        take_arrivals();  // the router may have dispatched since the last call
        if (next != next0) {
            const bool free_ = alone || join;  // every resident needs one token
            // (LAS: members' keys grow past a request that ranks behind the
            // last of a full batch, which then takes a place in it; see step)
            rep = rep && pol != P_LAS && n_spilled == sp0 && arrivals_keep(next0, true);
            alone = false;
            if (!rep && free_) plan_join();
        }
        for (;;) {
            if (status) return;
            if (UNLIKELY(nW + nR == 0)) {
                if (spill_n > 0) {
                    refill();
                    if (status) return;
                    if (nW + nR == 0) {
                        fail(S_ESTATE);
                        return;
                    }
                    continue;
                }
                if (next >= Nk) return;  // idle: nothing dispatched yet
                int off = next - pf;
                if (off >= kWave) {
                    pf = next;
                    load_pf();
                    off = 0;
                }
                const int64_t an = rl64(pa, off);  // <= limit: dispatched requests have arrived
                if (lane() == 0) S.ty[TY_IDLE] += (uint64_t)(an - t);
                t = an;
                take_arrivals();
                continue;
            }
            if (!less64(t, limit)) return;
            step(limit);
        }
    }

    // CL: requests the replica holds at time aj (dispatched and not completed
    // by aj). Only the latest iteration can end after aj, and its
    // completions then have not happened yet.
    DEV int held_at(int64_t aj) const { return Nk - completed + (t > aj ? last_done : 0); }

    // CL: the router sends global request j to this replica.
    DEV void dispatch(int j) {
        if (lane() == 0) {
            __hip_atomic_store(&jl()[Nk], j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            A.assign[(size_t)inst * (size_t)N + (size_t)j] = wv;
        }
        // the prefetch window [pf, pf + 64) takes the new entry now, as a
        // reload from the list would (pf <= next <= Nk)
        if (lane() == Nk - pf) pidx = j, pa = arr()[j], pP = Pp()[j], pD = Dp()[j];
        Nk++;
        hbm_fence();
    }

    // CL: latencies of the replica's requests in global order, its counters
    // (HBM, and in `cn` for the instance's totals) and status (`st`).
    DEV void finish_cl(int64_t *cn, int32_t *st) {
        hbm_fence();
        const int64_t *const arr = this->arr(), *const tfirst = this->tfirst(),
                      *const tlast = this->tlast();
        if (status == 0 && completed != Nk) fail(S_ESTATE);
        if (status == 0) {
            const size_t ioff = (size_t)inst * (size_t)N;
            bool bad = false;
            for (int b = 0; b < Nk; b += kWave) {
                const int kk = b + lane();
                if (kk < Nk) {
                    const int i = __hip_atomic_load(&jl()[kk], __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
                    const int64_t a = arr[i];
                    const int64_t f = tfirst[i] - a, l = tlast[i] - a;
                    if (f < 0 || f > 0xFFFFFFFFll || l < 0 || l > 0xFFFFFFFFll) bad = true;
                    A.ttft[ioff + i] = (uint32_t)f;
                    A.ttlt[ioff + i] = (uint32_t)l;
                }
            }
            if (ballot(bad)) fail(S_EOVERFLOW);
        }
        if (lane() == 0) {
            const int64_t v[8] = {iters, (int64_t)S.ty[TY_REQITERS], (int64_t)S.ty[TY_TOKENS],
                                  (int64_t)S.ty[TY_EVVOL], (int64_t)S.ty[TY_EVFORCED], t,
                                  (int64_t)maxU, (int64_t)S.ty[TY_IDLE]};
            const size_t slot = (size_t)inst * (size_t)A.replicas + (size_t)wv;
            int64_t *rc = A.rcounters + slot * 8;
            for (int q = 0; q < 8; q++) rc[q] = v[q], cn[q] = v[q];
            A.rgamma[slot] = ad ? S.as->gamma : 0.0;
            A.rswitches[slot] = ad ? S.as->switches : 0;
            *st = status;
        }
    }

    DEV void finish() {
        hbm_fence();
        const int64_t *const arr = this->arr(), *const tfirst = this->tfirst(),
                      *const tlast = this->tlast();
        if (status == 0 && completed != N) fail(S_ESTATE);
        if (status == 0) {
            const size_t ioff = (size_t)inst * (size_t)N;
            bool bad = false;
            for (int b = 0; b < N; b += kWave) {
                const int i = b + lane();
                if (i < N) {
                    const int64_t a = arr[i];
                    const int64_t f = tfirst[i] - a, l = tlast[i] - a;
                    if (f < 0 || f > 0xFFFFFFFFll || l < 0 || l > 0xFFFFFFFFll) bad = true;
                    A.ttft[ioff + i] = (uint32_t)f;
                    A.ttlt[ioff + i] = (uint32_t)l;
                }
            }
            if (ballot(bad)) fail(S_EOVERFLOW);
        }
        if (lane() == 0) {
            int64_t *cn = A.counters + (size_t)inst * 8;
            cn[0] = iters, cn[1] = (int64_t)S.ty[TY_REQITERS], cn[2] = (int64_t)S.ty[TY_TOKENS];
            cn[3] = (int64_t)S.ty[TY_EVVOL], cn[4] = (int64_t)S.ty[TY_EVFORCED], cn[5] = t;
            cn[6] = maxU, cn[7] = (int64_t)S.ty[TY_IDLE];
            // the next launch's order key: the loop steps this wave ran,
            // weighted by their measured cost (a step's fixed work 4, a
            // formation pass over up to 64 candidates 5, an emission chunk
            // 3), and far below them, to part equals, the iterations, which a
            // run of repeated ones takes at once. Unlike wall-clock time it
            // does not depend on the slot the instance ran in. The full-size
            // chat, reasoning, bursty and large workloads take 140, 2,220,
            // 1,076 and 7,520 ms so, 140, 2,219, 1,078 and 7,547 by the steps
            // alone, 142, 3,046, 1,306 and 8,363 by the iterations.
            if (A.work) A.work[inst] = 4 * iters + 64 * (int64_t)S.ty[TY_WORK];
            if constexpr (EXT) {  // (zero from tas_create for the other build)
                A.gamma_out[inst] = ad ? S.as->gamma : 0.0;
                A.switch_out[inst] = ad ? S.as->switches : 0;
            }
            A.status[inst] = status;
        }
    }
};

template <int BSH, bool EXT, bool CP>
DEV void run_instance(const SimArgs &a, const DevSetting &st, int inst, unsigned char *smem) {
    Sim<BSH, EXT, false, CP> s(a, st, inst, smem + kTallyBytes, (uint64_t *)smem);
    s.run();
}

// A cluster of replicas behind a join-shortest-queue router (global dispatch
// policies): one wavefront per replica, all in one workgroup. For every
// request of the global trace, in order, each replica first simulates the
// iterations that start before its arrival; then the request goes to the
// replica holding the fewest requests at that instant (ties to the lowest
// replica). Every wave passes the same barrier once per request, whatever
// its own state, so the workgroup cannot split at a barrier.
struct JsqLds {
    int32_t held[2][kMaxReplicas];  // by the parity of the global request index
    int32_t status[kMaxReplicas];
    int64_t cn[kMaxReplicas][8];
};
static_assert(sizeof(JsqLds) == kJsqLdsBytes, "router block size");

template <int BSH>
DEV void run_cluster(const SimArgs &a, const DevSetting &st, int inst, unsigned char *smem) {
    JsqLds *J = (JsqLds *)smem;
    const int R = a.replicas, N = a.n_req;
    const int w = uni((int)(threadIdx.x >> 6));  // (scalar: the state follows from it)
    Sim<BSH, true, true> s(a, st, inst, smem + kJsqLdsBytes + (size_t)w * (size_t)a.wave_lds,
                           (uint64_t *)J->cn[w], w);
    const int64_t *arr = a.arrival + (size_t)st.trace * (size_t)N;
    s.load_pf();  // nothing dispatched yet: an empty window, kept current by dispatch
    for (int j = 0;; j++) {  // j = N: run what was dispatched to the end
        const int64_t aj = j < N ? arr[j] : INT64_MAX;
        s.run_until(aj);
        if (j == N) break;
        // One barrier per request: the counts alternate between two
        // buffers. A wave that runs ahead writes the other one, and it
        // comes back to this one only after passing the next request's
        // barrier, which every wave reaches after reading this one.
        int32_t *held = J->held[j & 1];
        if (lane() == 0) held[w] = s.held_at(aj);
        __syncthreads();
        int best = 0, bn = held[0];
        for (int r = 1; r < R; r++) {
            const int h = held[r];
            if (h < bn) best = r, bn = h;
        }
        if (best == w) s.dispatch(j);
    }
    s.finish_cl(J->cn[w], &J->status[w]);
    __syncthreads();
    if (w == 0) {  // instance totals: sums, the latest clock, the largest KV peak
        const int q = lane();
        if (q < 8) {
            int64_t v = 0;
            for (int r = 0; r < R; r++) {
                const int64_t x = J->cn[r][q];
                v = (q == 5 || q == 6) ? (x > v ? x : v) : v + x;
            }
            a.counters[(size_t)inst * 8 + q] = v;
        }
        if (q == 0) {
            int32_t e = 0;
            for (int r = 0; r < R && e == 0; r++) e = J->status[r];
            a.status[inst] = e;
        }
    }
}

// EXT: the extended build (adaptive gamma, the phase-aware and cache-aware signals,
// DistBoost, Sarathi), launched when some instance uses one of them (its extra state
// and code cost the other policies registers). CP: compact list slots. BSH: see Sim.
// At 64 sequences the LDS holds 16 instances a compute unit, four a SIMD: 128
// vector registers each. Only the extended four-word build would take one or
// two more, and is told to stay within them (0: nothing asked). 4,096
// instances of 1,500 requests, ms a step, 3 and 4 waves: LTR+ on chat 30.8 and
// 22.7, on reasoning 514 and 507; eight policies mixed on chat 42.2 and 40.0,
// on reasoning 1,532 and 1,514.
template <bool EXT, bool CP, int BSH>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(EXT && !CP ? 4 : 0))) void sim_kernel(SimArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    if ((int)blockIdx.x >= a.n_inst) return;
    const int inst = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    if (a.retry && a.status[inst] != S_ECAPACITY) return;
    const DevSetting &st = a.inst[inst];
    run_instance<BSH, EXT, CP>(a, st, inst, smem);
}

// MAXW: the largest number of waves (replicas) the build serves; 8 leaves
// each wave twice the registers of 16.
template <int BSH, int MAXW>
__global__ __launch_bounds__(64 * MAXW) void cluster_kernel(SimArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int inst = blockIdx.x;
    if (inst >= a.n_inst) return;
    if (a.retry && a.status[inst] != S_ECAPACITY) return;
    run_cluster<BSH>(a, a.inst[inst], inst, smem);
}

}  // namespace
}  // namespace tas

int tas_launch_cluster(const tas::SimArgs &a, int64_t lds_bytes, void *stream) {
    if (a.n_inst <= 0) return 0;
    if (a.replicas < 2 || a.replicas > tas::kMaxReplicas) return -4;
    hipStream_t s = (hipStream_t)stream;
    const bool small = a.replicas <= 8, b16 = a.bs == 16;
    const void *fn = small ? (b16 ? (const void *)tas::cluster_kernel<4, 8>
                                  : (const void *)tas::cluster_kernel<-1, 8>)
                           : (b16 ? (const void *)tas::cluster_kernel<4, tas::kMaxReplicas>
                                  : (const void *)tas::cluster_kernel<-1, tas::kMaxReplicas>);
    if (lds_bytes > 65536) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return -4;
    }
    const dim3 grid((unsigned)a.n_inst), block((unsigned)(64 * a.replicas));
    if (small && b16)
        hipLaunchKernelGGL((tas::cluster_kernel<4, 8>), grid, block, (size_t)lds_bytes, s, a);
    else if (small)
        hipLaunchKernelGGL((tas::cluster_kernel<-1, 8>), grid, block, (size_t)lds_bytes, s, a);
    else if (b16)
        hipLaunchKernelGGL((tas::cluster_kernel<4, tas::kMaxReplicas>), grid, block,
                           (size_t)lds_bytes, s, a);
    else
        hipLaunchKernelGGL((tas::cluster_kernel<-1, tas::kMaxReplicas>), grid, block,
                           (size_t)lds_bytes, s, a);
    return hipGetLastError() == hipSuccess ? 0 : -4;
}

int tas_launch_sim(const tas::SimArgs &a, int64_t lds_bytes, void *stream) {
    if (a.n_inst <= 0) return 0;
    hipStream_t s = (hipStream_t)stream;
    void (*const fns[2][2][2])(tas::SimArgs) = {
        {{tas::sim_kernel<false, false, -1>, tas::sim_kernel<false, false, 4>},
         {tas::sim_kernel<false, true, -1>, tas::sim_kernel<false, true, 4>}},
        {{tas::sim_kernel<true, false, -1>, tas::sim_kernel<true, false, 4>},
         {tas::sim_kernel<true, true, -1>, tas::sim_kernel<true, true, 4>}}};
    void (*fn)(tas::SimArgs) = fns[a.ext ? 1 : 0][a.cp ? 1 : 0][a.bs == 16 ? 1 : 0];
    if (lds_bytes > 65536) {
        if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return -4;
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)a.n_inst), dim3(64), (size_t)lds_bytes, s, a);
    return hipGetLastError() == hipSuccess ? 0 : -4;
}
