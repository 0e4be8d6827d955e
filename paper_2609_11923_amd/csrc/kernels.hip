// kernels.hip -- gfx950 kernels of one compiled CFR iteration.
//
// Iteration (paper Algorithm 'alg:iteration', Table 'tab:opsteps'):
//   reach    : per slot, seq(I, a) = seq(last own slot before I) * sigma(I, a): the acting player's
//              reach (eqs. reach, lanes) of every node whose last own slot is (I, a).  Chance and
//              the other player multiply by 1, so a node's two reaches are those of two slots,
//              and by perfect recall a set has one own reach.
//   backward : per depth level, v(h) = sum_children m(c) v(c), m = sigma(slot) below decisions,
//              1 below chance (eqs. cfv, opbwd); terminal entries of v hold the template and
//              are never overwritten, so no per-iteration template copy is needed
//   update   : per information set I of player i with members h,
//              r(I,a) = sum_h s_i pi_{-i}(h) (v(h.a) - v(h))         (eqs. regret, instregret)
//              R <- R + r, CFR+ clamps at 0; sbar += w_t pi_i(I) sigma^t (FP64, Prop. 4);
//              then sigma^{t+1} = regret matching of R (eq. rm) for the next iteration.
// The state type T (reach, values, regrets, strategy) is float -- the paper's
// configured dtype -- or double; strategy sums are double in both.  Every
// reduction runs in a fixed order inside one thread, so results are bitwise
// reproducible run to run (no float atomics).
//
// The update's instantiations take most of the compile time, so this file is compiled once per CFR_PART
// (build.py): 0 everything that is not listed here, 1 / 2 the level launches in FP32 / FP64, 3 / 4 the
// persistent and LDS-resident launches in FP32 / FP64.
#include "common.hpp"
#include "compiler.hpp"
#include "device.hpp"

namespace cfrx {

// the pieces compiled per state type
hipError_t level_f32(const DevGame &g, int d, IterFlags f, hipStream_t s);
hipError_t level_f64(const DevGame &g, int d, IterFlags f, hipStream_t s);
hipError_t persistent_f32(const DevGame &g, const PersistentPlan &p, int32_t T_, IterFlags f, int alt, hipStream_t s);
hipError_t persistent_f64(const DevGame &g, const PersistentPlan &p, int32_t T_, IterFlags f, int alt, hipStream_t s);
const void *persistent_fn_f32(const DevGame &g);
const void *persistent_fn_f64(const DevGame &g);
hipError_t lds_f32(const DevGame &g, const int32_t *gr, int32_t n_cuts, int32_t T_, IterFlags f, int alt, hipStream_t s,
                   size_t bytes, bool prepare);
hipError_t lds_f64(const DevGame &g, const int32_t *gr, int32_t n_cuts, int32_t T_, IterFlags f, int alt, hipStream_t s,
                   size_t bytes, bool prepare);
#if CFR_PART == 1 || CFR_PART == 3
using PartT = float;
#define LEVEL_OF level_f32
#define PERSISTENT_OF persistent_f32
#define PERSISTENT_FN_OF persistent_fn_f32
#define LDS_OF lds_f32
#elif CFR_PART == 2 || CFR_PART == 4
using PartT = double;
#define LEVEL_OF level_f64
#define PERSISTENT_OF persistent_f64
#define PERSISTENT_FN_OF persistent_fn_f64
#define LDS_OF lds_f64
#endif

static_assert(reach_tile(true) % BLOCK == 0 && reach_tile(false) % BLOCK == 0, "slots per thread of k_reach");
// one thread per set of an update group; uint8 member-to-set indices
static_assert(GROUP_SETS_MAX <= BLOCK && GROUP_SETS_MAX <= 256, "update group sets");

// The reach of the sequence that ends in slot p: the strategies along it multiplied from the root on,
// as ((1 * s1) * s2) * ....  Slots below S0 are finished (seq holds their reach; seq[-1] = 1 is the empty
// sequence); above, the walk collects the strategies on the way up: at most REACH_WALK of them, which stay
// in registers (plan_reach and one_launch_ranges choose S0 so that no walk is longer).
template <typename T>
__device__ __forceinline__ T seq_reach(int32_t p, int32_t S0, const int32_t *slot_par, const T *sigma, const T *seq) {
    T s[REACH_WALK];
    int n = 0;
#pragma unroll
    for (int k = 0; k < REACH_WALK; k++) {
        s[k] = T(1);
        if (p >= S0) {
            s[k] = sigma[p];
            p = slot_par[p];
            n = k + 1;
        }
    }
    T acc = seq[p];
#pragma unroll
    for (int k = REACH_WALK - 1; k >= 0; k--)
        if (k < n) acc = acc * s[k];
    return acc;
}

// What the update of iteration t does (paper Sec. 6, update rules; see cfr.h).
struct RuleArgs {
    int rule;          // CFR_RULE_*
    int upd;           // players whose sets are updated: bit 0 player 1, bit 1 player 2
    double w;          // average weight (t or 1 for CFR and CFR+, t^2 for PCFR+, 1 for DCFR)
    double pos, neg;   // DCFR: discounts of positive and of other regrets
    double sdisc;      // DCFR: strategy-sum discount
};

__device__ __forceinline__ RuleArgs rule_args(int rule, int linear, int upd, int32_t t) {
    RuleArgs r;
    r.rule = rule;
    r.upd = upd;
    const double td = (double)t;
    r.w = rule == CFR_RULE_DCFR ? 1.0 : rule == CFR_RULE_PCFR_PLUS ? td * td : linear ? td : 1.0;
    r.pos = r.neg = r.sdisc = 1.0;
    if (rule == CFR_RULE_DCFR) {
        const double ta = pow(td, DCFR_ALPHA), tb = pow(td, DCFR_BETA);
        r.pos = ta / (ta + 1.0);
        r.neg = tb / (tb + 1.0);
        r.sdisc = pow(td / (td + 1.0), DCFR_GAMMA);
    }
    return r;
}

// The reach of slots [lo, hi), SPT per thread (strided by the block size, so each wave's accesses stay
// contiguous).  Bound by memory: 12 bytes per slot in FP32, and the parents' reaches, which siblings and
// neighbouring sets share.  WALK launches hold depths that depend on one another (plan_reach) and are
// narrow, bound by the latency of the walk: one slot per thread, so that the walks of more waves
// overlap.  Measured, FP32: 220M-node card game, 5 launches, 28.0M slots in 0.085 ms (5.3 TB/s); a pass
// over the 76M internal nodes, a launch per depth, took 0.30 ms.  26-card Leduc, one launch of 45,864
// slots instead of ten over its nodes: an iteration 93 -> 69 us.
template <typename T, bool WALK>
__global__ void __launch_bounds__(BLOCK) k_reach(int32_t lo, int32_t hi, int32_t S0,
                                                 const int32_t *__restrict__ slot_par, const T *__restrict__ sigma,
                                                 T *seq, int32_t *tick, double *weights, int rule, int linear,
                                                 const int32_t *__restrict__ tiles) {
    constexpr int SPT = reach_tile(WALK) / BLOCK;
    if (tick && blockIdx.x == 0 && threadIdx.x == 0) {
        // the iteration's weight and discounts, for its levels (DCFR's powers cost a level's blocks more than
        // the loads they wait for)
        const int32_t t = tick[0] + 1;
        tick[0] = t;
        const RuleArgs r = rule_args(rule, linear, 3, t);
        weights[0] = r.w; weights[1] = r.pos; weights[2] = r.neg; weights[3] = r.sdisc;
    }
    if (hi <= lo) return;
    // with retired games only the listed tiles run (a tile shared with a retired game rewrites that
    // game's reach with the same values: its strategy no longer changes)
    const int32_t tile = tiles ? tiles[blockIdx.x] : (int32_t)blockIdx.x;
    const int32_t base = lo + tile * (BLOCK * SPT) + (int32_t)threadIdx.x;
    int32_t p[SPT];
    T sv[SPT], up[SPT];
#pragma unroll
    for (int i = 0; i < SPT; i++) {
        const int32_t q = min(base + i * BLOCK, hi - 1);
        p[i] = slot_par[q];
        sv[i] = sigma[q];
    }
#pragma unroll
    for (int i = 0; i < SPT; i++) {
        if constexpr (WALK) up[i] = seq_reach<T>(p[i], S0, slot_par, sigma, seq);
        else up[i] = seq[p[i]];
    }
#pragma unroll
    for (int i = 0; i < SPT; i++)
        if (base + i * BLOCK < hi) seq[base + i * BLOCK] = up[i] * sv[i];
}

// Arrays read and written by the backward/update level.
template <typename T>
struct LevelArgs {
    const int32_t *grp_iset_off, *slot_off, *mem_off;
    const int2 *mem;
    const int8_t *iset_player;
    const int32_t *kid_off, *kid, *chance_node, *bigc_node;
    const int32_t *grp_list, *chance_list, *bigc_list;   // batches with retired games (nullptr: all)
    const int32_t *iset_seq, *slot_par;  // last own slot before a set, and before the set of a slot
    const int32_t *mem_seq;        // the other player's last slot before each member (order of mem)
    const int32_t *koff;           // affine layouts: per-slot child offset, and DevGame's group headers,
    const int4 *ghdr;              // set records and member records
    const int2 *srec, *mwide;
    const uint32_t *mrec;
    const uint16_t *mpos;
    T *v;
    T *seq;       // reach of every slot's sequence; seq[-1] = 1
    T *R;
    double *sbar;
    T *sigma;
    T *pred;      // PCFR+ prediction buffer, nullptr for the other rules
    const int32_t *mem_words, *player_words;   // mem and iset_player as words (games staged whole in LDS)
};

// The reach of set i's slots, all of which continue the same sequence: a walk per set, where k_reach has one per slot
// to keep its accesses contiguous.
template <typename T, int MAXA>
__device__ __forceinline__ void set_reach(int32_t i, int32_t S0, const LevelArgs<T> &a) {
    const int32_t s0 = a.slot_off[i], nA = a.slot_off[i + 1] - s0, p = a.iset_seq[i];
    constexpr int U = MAXA < 4 ? MAXA : 4;
    T own = T(0);
    for (int32_t k0 = 0; k0 < nA; k0 += U) {
        T x[U];
#pragma unroll
        for (int k = 0; k < U; k++) x[k] = a.sigma[s0 + min(k0 + k, nA - 1)];
        if (k0 == 0) own = seq_reach<T>(p, S0, a.slot_par, a.sigma, a.seq);
#pragma unroll
        for (int k = 0; k < U; k++)
            if (k0 + k < nA) a.seq[s0 + k0 + k] = own * x[k];
        if constexpr (MAXA <= 4) break;
    }
}

// Value of an internal chance node: the sum of its children (chance folded into the template).
template <typename T, bool EXPLICIT>
__device__ __forceinline__ void chance_value(int32_t h, const LevelArgs<T> &a) {
    const int32_t b = a.kid_off[h], e = a.kid_off[h + 1];
    T acc = T(0);
    // eight children per step, loads unconditional (past the last child they repeat it) so they
    // are in flight together; the sum keeps child order
    constexpr int U = 8;
    for (int32_t c0 = b; c0 < e; c0 += U) {
        int32_t ch[U];
        T x[U];
#pragma unroll
        for (int i = 0; i < U; i++) ch[i] = child_of<EXPLICIT>(a.kid, min(c0 + i, e - 1));
#pragma unroll
        for (int i = 0; i < U; i++) x[i] = a.v[ch[i]];
#pragma unroll
        for (int i = 0; i < U; i++) acc = c0 + i < e ? acc + x[i] : acc;
    }
    a.v[h] = acc;
}

// Value of a chance node with large fan-out, by a whole block: each thread sums a strided slice
// of the children in order, then a fixed-shape tree reduction over the block (deterministic).
// Must be called by every thread of the block.
template <typename T, bool EXPLICIT>
__device__ void big_chance_value(int32_t h, const LevelArgs<T> &a, T *red) {
    const int tid = threadIdx.x;
    const int32_t b = a.kid_off[h], e = a.kid_off[h + 1];
    T acc = T(0);
    // this thread's children b + tid, b + tid + BLOCK, ... summed in that order, eight loads in
    // flight at a time (past the last child the index is clamped and the value not added)
    constexpr int U = 8;
    for (int32_t c0 = b + tid; c0 < e; c0 += U * BLOCK) {
        int32_t ch[U];
        T x[U];
#pragma unroll
        for (int i = 0; i < U; i++) ch[i] = child_of<EXPLICIT>(a.kid, min(c0 + i * BLOCK, e - 1));
#pragma unroll
        for (int i = 0; i < U; i++) x[i] = a.v[ch[i]];
#pragma unroll
        for (int i = 0; i < U; i++) acc = c0 + i * BLOCK < e ? acc + x[i] : acc;
    }
    red[tid] = acc;
    __syncthreads();
    for (int w = BLOCK / 2; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0) a.v[h] = red[0];
    __syncthreads();
}

// The update of one information set from its instantaneous regrets r (already summed over the
// members, player 1's sign) and its state as loaded (R, sigma^t, sbar): R <- R + sign r with the
// rule's clamp or discount, sbar += w pi_i(I) sigma^t (FP64; DCFR discounts it), then
// sigma^{t+1} = regret matching of R (PCFR+: of R plus the prediction, which becomes this
// iteration's instantaneous regret and is stored here).  Rk and sb are updated in place and the
// new strategy is returned in sn.
template <typename T, int MAXA, bool EXT>
__device__ __forceinline__ void set_update_compute(const RuleArgs &ru, const LevelArgs<T> &a, int32_t s0, int32_t nA,
                                                   int pl, double pown, const T (&r)[MAXA], T (&Rk)[MAXA],
                                                   const T (&sk)[MAXA], double (&sb)[MAXA], T (&sn)[MAXA]) {
    const T sign = pl == 1 ? T(1) : T(-1);
    T tot = T(0);
    T Rn[MAXA];
    if constexpr (!EXT) {
        const bool clamp = ru.rule != CFR_RULE_CFR;
#pragma unroll
        for (int k = 0; k < MAXA; k++)
            if (k < nA) {
                sb[k] += ru.w * pown * (double)sk[k];
                T y = fma_t(sign, r[k], Rk[k]);
                if (clamp) y = max_t(y, T(0));
                Rk[k] = y;
                Rn[k] = max_t(y, T(0));
                tot += Rn[k];
            }
    } else {
        if (ru.rule == CFR_RULE_DCFR) {
            const T pos = (T)ru.pos, neg = (T)ru.neg;
#pragma unroll
            for (int k = 0; k < MAXA; k++)
                if (k < nA) {
                    sb[k] = (sb[k] + pown * (double)sk[k]) * ru.sdisc;
                    T y = fma_t(sign, r[k], Rk[k]);
                    y = y > T(0) ? y * pos : y * neg;
                    Rk[k] = y;
                    Rn[k] = max_t(y, T(0));
                    tot += Rn[k];
                }
        } else if (ru.rule == CFR_RULE_PCFR_PLUS) {
#pragma unroll
            for (int k = 0; k < MAXA; k++)
                if (k < nA) {
                    sb[k] += ru.w * pown * (double)sk[k];
                    const T y = max_t(fma_t(sign, r[k], Rk[k]), T(0));
                    const T m = sign * r[k];
                    Rk[k] = y;
                    a.pred[s0 + k] = m;
                    Rn[k] = max_t(y + m, T(0));
                    tot += Rn[k];
                }
        } else {
            const bool clamp = ru.rule != CFR_RULE_CFR;
#pragma unroll
            for (int k = 0; k < MAXA; k++)
                if (k < nA) {
                    sb[k] += ru.w * pown * (double)sk[k];
                    T y = fma_t(sign, r[k], Rk[k]);
                    if (clamp) y = max_t(y, T(0));
                    Rk[k] = y;
                    Rn[k] = max_t(y, T(0));
                    tot += Rn[k];
                }
        }
    }
    const T inv = tot > T(0) ? T(1) / tot : T(0);
    const T uni = T(1) / (T)nA;
#pragma unroll
    for (int k = 0; k < MAXA; k++) sn[k] = tot > T(0) ? Rn[k] * inv : uni;
}

// set_update_compute, then the set's new regrets, strategy sums and strategy stored in place.
template <typename T, int MAXA, bool EXT>
__device__ __forceinline__ void set_update_from(const RuleArgs &ru, const LevelArgs<T> &a, int32_t s0, int32_t nA,
                                                int pl, double pown, const T (&r)[MAXA], T (&Rk)[MAXA],
                                                const T (&sk)[MAXA], double (&sb)[MAXA]) {
    T sn[MAXA];
    set_update_compute<T, MAXA, EXT>(ru, a, s0, nA, pl, pown, r, Rk, sk, sb, sn);
#pragma unroll
    for (int k = 0; k < MAXA; k++)
        if (k < nA) {
            a.R[s0 + k] = Rk[k];
            a.sbar[s0 + k] = sb[k];
            a.sigma[s0 + k] = sn[k];
        }
}

// Load the set's state, then set_update_from.
template <typename T, int MAXA>
__device__ __forceinline__ void load_set_state(const LevelArgs<T> &a, int32_t s0, int32_t nA, T (&Rk)[MAXA],
                                               T (&sk)[MAXA], double (&sb)[MAXA]) {
    // unconditional loads (past the last action they repeat it): all in flight at once
#pragma unroll
    for (int k = 0; k < MAXA; k++) {
        const int32_t q = s0 + min(k, nA - 1);
        Rk[k] = a.R[q];
        sk[k] = a.sigma[q];
        sb[k] = a.sbar[q];
    }
}

template <typename T, int MAXA, bool EXT>
__device__ __forceinline__ void set_update(const RuleArgs &ru, const LevelArgs<T> &a, int32_t s0, int32_t nA, int pl,
                                           double pown, const T (&r)[MAXA]) {
    T Rk[MAXA], sk[MAXA];
    double sb[MAXA];
    load_set_state<T, MAXA>(a, s0, nA, Rk, sk, sb);
    set_update_from<T, MAXA, EXT>(ru, a, s0, nA, pl, pown, r, Rk, sk, sb);
}

// Phase 2 of a group: a set's instantaneous regrets r(I, a) += po(h) * diff(h, a) over its staged
// members [k0, k1) in ascending order, one fused multiply-add chain per action.  The LDS reads of
// U members are issued before their multiply-adds (the order of the chain is unchanged), so a set
// with many members does not wait one LDS round trip per member.  The first NA columns are
// accumulated (NA bounds the group's action counts): past a set's actions the columns hold repeats
// that are never read afterwards.
template <typename T, int MAXA, int NA = MAXA>
__device__ __forceinline__ void reduce_members(const T *po, const T *diff, int32_t k0, int32_t k1, T (&r)[MAXA]) {
    constexpr int U = NA <= 4 ? (sizeof(T) == 4 ? 8 : 4) : 2;
    int32_t k = k0;
    for (; k + U <= k1; k += U) {
        T p[U], d[U][NA];
#pragma unroll
        for (int i = 0; i < U; i++) {
            p[i] = po[k + i];
#pragma unroll
            for (int q = 0; q < NA; q++) d[i][q] = diff[(k + i) * MAXA + q];
        }
#pragma unroll
        for (int i = 0; i < U; i++)
#pragma unroll
            for (int q = 0; q < NA; q++) r[q] = fma_t(p[i], d[i][q], r[q]);
    }
    for (; k < k1; k++) {
        const T p = po[k];
#pragma unroll
        for (int q = 0; q < NA; q++) r[q] = fma_t(p, diff[k * MAXA + q], r[q]);
    }
}

// LDS staging of one update group (members of a chunk, the group's set offsets)
template <typename T, int MAXA, int MPT>
struct GroupLds {
    T po[MPT * BLOCK];
    alignas(16) T diff[MPT * BLOCK * MAXA];
    int32_t moff[BLOCK + 1];
    int32_t slot[BLOCK + 1];
};

// One update group: consecutive information sets of one depth with at most MPT * BLOCK members
// and GROUP_SETS sets.  Phase 1 (one thread per member h, coalesced over the member list):
//   v(h) = sum_a sigma^t(I, a) v(h.a)   -- written to v: the backward value pass at h
//   stage pi_{-i}(h) and v(h.a) - v(h) in LDS.
// Phase 2 (one thread per set I): reduce the set's members from LDS in ascending member order,
//   r(I,a) = sum_h s_i pi_{-i}(h) (v(h.a) - v(h)), then R <- R + r (CFR+: max(R, 0)),
//   sbar += w_t pi_i(I) sigma^t (FP64), sigma^{t+1} = regret matching of R.
// Only this group reads sigma(I) during the backward pass (all members of I are here), and the
// reach pass has already consumed it, so overwriting sigma(I) with sigma^{t+1} is safe.
// Sets with more members than a chunk are streamed through LDS chunk by chunk.  Must be called by
// every thread of the block (it synchronises the block).
template <typename T, int MAXA, int MPT, bool EXPLICIT, bool EXT>
__device__ void group_update(int32_t g, const RuleArgs &ru, const LevelArgs<T> &a, GroupLds<T, MAXA, MPT> &L) {
    // EXT: the discounted and predictive rules (DCFR, PCFR+); otherwise CFR or CFR+ (lean tail)
    constexpr int CHUNK = MPT * BLOCK;
    const int tid = threadIdx.x;
    const int32_t i0 = a.grp_iset_off[g], i1 = a.grp_iset_off[g + 1];
    const int32_t nsets = i1 - i0;
    if (tid < nsets) {
        L.moff[tid] = a.mem_off[i0 + tid];
        L.slot[tid] = a.slot_off[i0 + tid];
    }
    if (tid == 0) {
        L.moff[nsets] = a.mem_off[i1];
        L.slot[nsets] = a.slot_off[i1];
    }
    __syncthreads();
    const int32_t mbeg = L.moff[0], mend = L.moff[nsets];
    const bool has_set = tid < nsets;
    int32_t s0 = 0, nA = 0, m0 = 0, m1 = 0, pl = 1;
    if (has_set) {
        s0 = L.slot[tid];
        nA = L.slot[tid + 1] - s0;
        m0 = L.moff[tid];
        m1 = L.moff[tid + 1];
        pl = a.iset_player[i0 + tid];
    }
    T r[MAXA];
#pragma unroll
    for (int k = 0; k < MAXA; k++) r[k] = T(0);
    for (int32_t cb = mbeg; cb < mend; cb += CHUNK) {
        const int32_t ce = min(cb + CHUNK, mend);
        // loads first and unconditional (past the chunk's end a lane repeats its first member, past
        // a set's last action the last child and slot), then the arithmetic and the masked stores
        bool in[MPT];
        int32_t sb[MPT], na[MPT], hh[MPT];
        T po[MPT], sg[MPT][MAXA], cv[MPT][MAXA];
#pragma unroll
        for (int u = 0; u < MPT; u++) {
            const int32_t j = u * BLOCK + tid;
            in[u] = cb + j < ce;
            const int32_t m = cb + (in[u] ? j : 0);
            // the set of member m: the last k with moff[k] <= m
            int32_t lo = 0, hi = nsets - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (L.moff[mid] <= m) lo = mid; else hi = mid - 1;
            }
            sb[u] = L.slot[lo];
            na[u] = L.slot[lo + 1] - sb[u];
            const int2 x = a.mem[m];
            hh[u] = x.x & MEMBER_NODE_MASK;
            po[u] = a.seq[a.mem_seq[m]];
#pragma unroll
            for (int k = 0; k < MAXA; k++) {
                const int32_t kk = min(k, na[u] - 1);
                cv[u][k] = a.v[child_of<EXPLICIT>(a.kid, x.y + kk)];
                sg[u][k] = a.sigma[sb[u] + kk];
            }
        }
#pragma unroll
        for (int u = 0; u < MPT; u++) {
            T vh = T(0);
#pragma unroll
            for (int k = 0; k < MAXA; k++) vh = k < na[u] ? fma_t(sg[u][k], cv[u][k], vh) : vh;
            if (!in[u]) continue;
            const int32_t j = u * BLOCK + tid;
            a.v[hh[u]] = vh;
            L.po[j] = po[u];
#pragma unroll
            for (int k = 0; k < MAXA; k++) L.diff[j * MAXA + k] = cv[u][k] - vh;
        }
        __syncthreads();
        if (has_set) reduce_members<T, MAXA>(L.po, L.diff, max(m0, cb) - cb, min(m1, ce) - cb, r);
        __syncthreads();
    }
    if (!has_set) return;
    // alternating order: the other player's half leaves this set's state alone (values only)
    if (!((ru.upd >> (pl - 1)) & 1)) return;
    set_update<T, MAXA, EXT>(ru, a, s0, nA, pl, (double)a.seq[a.iset_seq[i0 + tid]], r);
}

// LDS staging of one update group in an affine layout: the member values of group_update, each set's first
// slot and each member's set, and (FP32 state, up to 16 actions) the child offsets and strategy of the
// group's slots.  These hold GS sets, the game's group bound (128 or 256): with 128 an FP32 block's LDS fits
// six per compute unit instead of five.  For FP64 they would cost a resident block per compute unit
// (measured slower), so members read them through the cache instead.
template <typename T, int MAXA, int MPT, int GS>
struct GroupLdsA {
    static constexpr bool ROWS = MAXA <= 16 && sizeof(T) == 4;
    static constexpr int SLOTS = ROWS ? GS * MAXA : 1;
    T po[MPT * BLOCK];
    alignas(16) T diff[MPT * BLOCK * MAXA];
    alignas(16) int32_t ko[SLOTS];
    T sg[SLOTS];
    uint16_t slot[GS + 1];
    alignas(4) uint8_t mset[MPT * BLOCK];
};

// set tid's first slot and members [m0, m1) (relative to the group's) into LDS: the member -> set map covers
// one chunk (a group of several sets fits it, and a larger one is a single set)
template <typename T, int MAXA, int MPT, int GS>
__device__ __forceinline__ void map_set(GroupLdsA<T, MAXA, MPT, GS> &L, int tid, int32_t nsets, int32_t slot,
                                        int32_t nslots, int32_t m0, int32_t m1) {
    L.slot[tid] = (uint16_t)slot;
    if (tid == nsets - 1) L.slot[nsets] = (uint16_t)nslots;
    int32_t m = m0;
    const int32_t e = min(m1, MPT * BLOCK);
    for (; m < e && (m & 3); m++) L.mset[m] = (uint8_t)tid;
    for (; m + 4 <= e; m += 4) *(uint32_t *)&L.mset[m] = (uint32_t)tid * 0x01010101u;
    for (; m < e; m++) L.mset[m] = (uint8_t)tid;
}

// group_update for affine layouts (child a of member h is h + koff[slot a]): the same arithmetic
// in the same order, so the results are bitwise those of group_update.  What changes is what is loaded
// and when.  Large levels are bound by memory traffic, small ones by the chain of dependent loads (a
// launch holds a few groups per compute unit at most), so both are kept short:
//  * the group's header gives its sets, members and slots, so every further load but two depends on the
//    header alone: set records, member records, and the child offsets and strategy of its slots (into LDS,
//    coalesced) are requested together; the opponent's reach follows the member record (requested before the
//    first barrier as well) and the child values follow the offsets;
//  * a member record is four bytes: its node and the opponent's last sequence relative to the group's
//    bases, split where the group's nodes need it (GRP_WIDE groups, whose spans need more than 32 bits
//    together or whose single set has more members than a chunk, keep them in eight);
//  * a set record is eight bytes: its first member, first slot and player in one word, its own sequence;
//  * the slots' regrets and strategy sums are requested right after the child values, so that nothing waits
//    for them before the reduction is done.
// The member pass has no branch: past a set's last action loads repeat its last child (an address already
// read), lanes past the group's end repeat its first member and store what that member's lane stores, slots
// past the last one repeat it into rows nobody reads, and a group that updates nothing reads the empty
// sequence's reach.  A guard compiles to a branch, and what a branch holds is neither issued with the loads
// around it nor waited for apart from them.  The number of child loads per member
// is the group's widest set, bucketed (with_action_bound; the public-state layout orders states by
// action count, so most groups are uniform), and where a group's sets interleave -- a player-2 set's
// members are strided by the opponent's hand count -- the host lists the group's members in node order
// (GRP_PERM) with each one's set-major position: consecutive lanes then touch consecutive nodes, children
// and values instead of one cache line each, and the staging stays set-major, so the reduction, and every
// result, is unchanged.  Both are choices of the header, made once per group.  In alternating order a group
// without sets of the updated player only needs its values.
// Measured, FP32 state, all levels of an iteration, against set and member arrays read one after another (8-byte
// members, 13-byte sets, slots loaded after the reduction): 220M-node card game 0.74 -> 0.63 ms (2.75 GB of
// design bytes, 4.4 TB/s), 256 subgames 103 -> 97 us, 26-card Leduc 61 -> 56 us in 11 launches; DCFR in FP64
// on the 10.0M-node card game, with the discounts' powers out of the blocks, 12.7 -> 11.2 us per launch.
// The guards taken out: five iterations of the 37.6M-node card game 1.40 -> 1.29 ms, ten of 256 subgames
// 1.00 -> 0.95 ms, ten of Leduc with 3 ranks in FP64 0.43 -> 0.41 ms.  (Requesting the slots' state with the
// group's records instead makes the child values wait for it: 1.44 ms for the first.)
template <typename T, int MAXA, int MPT, bool EXT, int GS, int NA, bool PERM>
__device__ __forceinline__ void group_body(const int4 &h0, const int4 &hb, const int4 &h1, const RuleArgs &ru,
                                           const LevelArgs<T> &a, GroupLdsA<T, MAXA, MPT, GS> &L) {
    constexpr bool ROWS = GroupLdsA<T, MAXA, MPT, GS>::ROWS;
    constexpr bool SLOT_PASS = ROWS && MAXA <= 4;
    constexpr int SPT = (GS * MAXA + BLOCK - 1) / BLOCK;   // slots per thread
    const int tid = threadIdx.x;
    const int32_t i0 = h0.x, nsets = h1.x - i0, mbeg = h0.y, mend = h1.y, S0 = h0.z, nslots = h1.z - S0;
    const bool update = (h0.w >> GRP_PLAYERS) & ru.upd;
    const bool has_set = tid < nsets;
    int32_t h[MPT], ms[MPT], pj[MPT];
#pragma unroll
    for (int u = 0; u < MPT; u++) {
        const int32_t j = u * BLOCK + tid, jj = mbeg + j < mend ? j : 0;
        const uint32_t x = a.mrec[mbeg + jj];
        h[u] = hb.x + (int32_t)(x & ((1u << hb.w) - 1));
        ms[u] = hb.y + (int32_t)(x >> hb.w);
        if constexpr (PERM) pj[u] = a.mpos[mbeg + jj];
        else pj[u] = jj;
    }
    const int32_t ti = i0 + (has_set ? tid : nsets - 1);
    const int2 sr = a.srec[ti];
    const int32_t next = a.srec[min(ti + 1, h1.x - 1)].x;
    if constexpr (ROWS) {
        // Up to four actions all slots are loaded at once.  Up to sixteen a group has a few hundred slots as a rule
        // and 4,096 at most: four loads in flight at a time, and no rounds past the group's last slot (a load and a
        // dependent store in each of sixteen rounds made an iteration of a 6-action game of 259 nodes 20.2 us;
        // now 17.2, the child lists 16.5; a 5-action game of 19,531 nodes 42.5, 36.2 and 38.5).
        constexpr int UNROLL = SLOT_PASS ? SPT : 4;
        static_assert(SPT % UNROLL == 0, "whole rounds");
        int32_t k[UNROLL];
        T s[UNROLL];
#pragma unroll 1
        for (int u0 = 0; u0 < SPT && (SLOT_PASS || u0 * BLOCK < nslots); u0 += UNROLL) {
#pragma unroll
            for (int u = 0; u < UNROLL; u++) {
                const int32_t q = S0 + min((u0 + u) * BLOCK + tid, nslots - 1);
                k[u] = a.koff[q];
                s[u] = a.sigma[q];
            }
#pragma unroll
            for (int u = 0; u < UNROLL; u++) {
                L.ko[(u0 + u) * BLOCK + tid] = k[u];
                L.sg[(u0 + u) * BLOCK + tid] = s[u];
            }
        }
    }
    const bool last = ti + 1 == h1.x;
    const int32_t m0 = mbeg + (sr.x & SREC_MEMBER_MASK), m1 = last ? mend : mbeg + (next & SREC_MEMBER_MASK);
    const int32_t sl = (sr.x >> SREC_SLOT_SHIFT) & SREC_SLOT_MASK;
    const int32_t nA = (last ? nslots : (next >> SREC_SLOT_SHIFT) & SREC_SLOT_MASK) - sl;
    const int pl = (sr.x >> SREC_PLAYER_SHIFT) + 1;
    T po[MPT];
#pragma unroll
    for (int u = 0; u < MPT; u++) po[u] = a.seq[update ? ms[u] : -1];
    const T pown = a.seq[sr.y];
    if (has_set) map_set<T, MAXA, MPT, GS>(L, tid, nsets, sl, nslots, m0 - mbeg, m1 - mbeg);
    __syncthreads();
    double sbp[SLOT_PASS ? SPT : 1];
    T Rp[SLOT_PASS ? SPT : 1];
    {
        T cv[MPT][NA], sg[MPT][ROWS ? 1 : NA];
        int32_t sb[MPT], na[MPT];
#pragma unroll
        for (int u = 0; u < MPT; u++) {
            const int32_t st = L.mset[pj[u]];
            sb[u] = L.slot[st];
            na[u] = L.slot[st + 1] - sb[u];
            int32_t ko[NA];
#pragma unroll
            for (int k = 0; k < NA; k++) {
                const int32_t q = sb[u] + min(k, na[u] - 1);
                if constexpr (ROWS) {
                    ko[k] = L.ko[q];
                } else {
                    ko[k] = a.koff[S0 + q];
                    sg[u][k] = a.sigma[S0 + q];
                }
            }
#pragma unroll
            for (int k = 0; k < NA; k++) cv[u][k] = a.v[h[u] + ko[k]];
        }
        if constexpr (SLOT_PASS) {
            const int32_t last_slot = update ? nslots - 1 : 0;
#pragma unroll
            for (int u = 0; u < SPT; u++) {
                const int32_t q = S0 + min(u * BLOCK + tid, last_slot);
                sbp[u] = a.sbar[q];
                Rp[u] = a.R[q];
            }
        }
#pragma unroll
        for (int u = 0; u < MPT; u++) {
            T vh = T(0);
#pragma unroll
            for (int k = 0; k < NA; k++) {
                T sk;
                if constexpr (ROWS) sk = L.sg[sb[u] + min(k, na[u] - 1)];
                else sk = sg[u][k];
                vh = k < na[u] ? fma_t(sk, cv[u][k], vh) : vh;
            }
            const int32_t j = pj[u];
            a.v[h[u]] = vh;
            L.po[j] = po[u];
#pragma unroll
            for (int k = 0; k < NA; k++) L.diff[j * MAXA + k] = cv[u][k] - vh;
        }
    }
    if (!update) return;
    __syncthreads();
    T r[MAXA];
#pragma unroll
    for (int k = 0; k < MAXA; k++) r[k] = T(0);
    if (has_set) reduce_members<T, MAXA, NA>(L.po, L.diff, m0 - mbeg, m1 - mbeg, r);
    if constexpr (SLOT_PASS) {
        // The group's slots are contiguous: their regrets, strategy sums and strategy move through LDS (the
        // member staging is free now) with coalesced passes of the whole block, instead of each set thread
        // loading and storing its few slots.  Slots of sets this half leaves alone are written back
        // unchanged.
        constexpr int CHUNK = MPT * BLOCK;
        double *sbs = reinterpret_cast<double *>(L.diff);   // [<= CHUNK]
        T *Rs = reinterpret_cast<T *>(sbs + CHUNK);         // [<= CHUNK]
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SPT; u++) {
            sbs[u * BLOCK + tid] = sbp[u];
            Rs[u * BLOCK + tid] = Rp[u];
        }
        __syncthreads();
        if (has_set && ((ru.upd >> (pl - 1)) & 1)) {
            T Rk[MAXA], sk[MAXA], sn[MAXA];
            double sb[MAXA];
#pragma unroll
            for (int k = 0; k < MAXA; k++) {
                const int32_t q = sl + min(k, nA - 1);
                Rk[k] = Rs[q];
                sk[k] = L.sg[q];
                sb[k] = sbs[q];
            }
            set_update_compute<T, MAXA, EXT>(ru, a, S0 + sl, nA, pl, (double)pown, r, Rk, sk, sb, sn);
#pragma unroll
            for (int k = 0; k < MAXA; k++)
                if (k < nA) {
                    Rs[sl + k] = Rk[k];
                    sbs[sl + k] = sb[k];
                    L.sg[sl + k] = sn[k];
                }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SPT; u++) {
            const int32_t q = u * BLOCK + tid;
            if (q < nslots) {
                a.sbar[S0 + q] = sbs[q];
                a.R[S0 + q] = Rs[q];
                a.sigma[S0 + q] = L.sg[q];
            }
        }
    } else if (has_set && ((ru.upd >> (pl - 1)) & 1)) {
        set_update<T, MAXA, EXT>(ru, a, S0 + sl, nA, pl, (double)pown, r);
    }
}

// group_body for GRP_WIDE groups: full member records, a chunk of members at a time (only a group of a
// single set has several), a member of each thread after another.
template <typename T, int MAXA, int MPT, bool EXT, int GS>
__device__ void group_wide(const int4 &h0, const int4 &hb, const int4 &h1, const RuleArgs &ru, const LevelArgs<T> &a,
                           GroupLdsA<T, MAXA, MPT, GS> &L) {
    constexpr int CHUNK = MPT * BLOCK;
    const int tid = threadIdx.x;
    const int32_t i0 = h0.x, nsets = h1.x - i0, mbeg = h0.y, mend = h1.y, S0 = h0.z, nslots = h1.z - S0;
    const bool has_set = tid < nsets;
    const int32_t ti = i0 + (has_set ? tid : nsets - 1);
    const int2 sr = a.srec[ti];
    const int32_t next = a.srec[min(ti + 1, h1.x - 1)].x;
    const bool last = ti + 1 == h1.x;
    const int32_t m0 = mbeg + (sr.x & SREC_MEMBER_MASK), m1 = last ? mend : mbeg + (next & SREC_MEMBER_MASK);
    const int32_t sl = (sr.x >> SREC_SLOT_SHIFT) & SREC_SLOT_MASK;
    const int32_t nA = (last ? nslots : (next >> SREC_SLOT_SHIFT) & SREC_SLOT_MASK) - sl;
    const int pl = (sr.x >> SREC_PLAYER_SHIFT) + 1;
    if (has_set) map_set<T, MAXA, MPT, GS>(L, tid, nsets, sl, nslots, m0 - mbeg, m1 - mbeg);
    __syncthreads();
    T r[MAXA];
#pragma unroll
    for (int k = 0; k < MAXA; k++) r[k] = T(0);
    for (int32_t cb = mbeg; cb < mend; cb += CHUNK) {
        const int32_t ce = min(cb + CHUNK, mend);
#pragma unroll 1
        for (int32_t m = cb + tid; m < ce; m += BLOCK) {
            const int2 x = a.mwide[hb.z + (m - mbeg)];
            const int32_t pos = nsets == 1 ? m - cb : a.mpos[m], st = nsets == 1 ? 0 : L.mset[pos];
            const int32_t q0 = S0 + L.slot[st], na = S0 + L.slot[st + 1] - q0;
            T cv[MAXA], sg[MAXA];
            const T po = a.seq[x.y];
#pragma unroll
            for (int k = 0; k < MAXA; k++) {
                const int32_t q = q0 + min(k, na - 1);
                cv[k] = a.v[x.x + a.koff[q]];
                sg[k] = a.sigma[q];
            }
            T vh = T(0);
#pragma unroll
            for (int k = 0; k < MAXA; k++) vh = k < na ? fma_t(sg[k], cv[k], vh) : vh;
            a.v[x.x] = vh;
            L.po[pos] = po;
#pragma unroll
            for (int k = 0; k < MAXA; k++) L.diff[pos * MAXA + k] = cv[k] - vh;
        }
        __syncthreads();
        if (has_set) reduce_members<T, MAXA>(L.po, L.diff, max(m0, cb) - cb, min(m1, ce) - cb, r);
        __syncthreads();
    }
    if (has_set && ((ru.upd >> (pl - 1)) & 1))
        set_update<T, MAXA, EXT>(ru, a, S0 + sl, nA, pl, (double)a.seq[sr.y], r);
}

// Must be called by every thread of the block; a block that updates several groups synchronises between
// them.
template <typename T, int MAXA, int MPT, bool EXT, int GS>
__device__ void group_update_affine(int32_t g, const RuleArgs &ru, const LevelArgs<T> &a,
                                    GroupLdsA<T, MAXA, MPT, GS> &L) {
    const int4 h0 = a.ghdr[2 * g], hb = a.ghdr[2 * g + 1], h1 = a.ghdr[2 * g + 2];
    if (h0.w & GRP_WIDE) {
        group_wide<T, MAXA, MPT, EXT, GS>(h0, hb, h1, ru, a, L);
        return;
    }
    // (the positions of a set-major list are the identity, so the node-order form is right for any group:
    // those of more than four actions, which are rare, have only that)
    with_action_bound<MAXA>((h0.w >> GRP_ACTIONS) & 0xff, [&](auto na) {
        constexpr int NA = decltype(na)::value;
        if (MAXA > 4 || (h0.w & GRP_PERM)) group_body<T, MAXA, MPT, EXT, GS, NA, true>(h0, hb, h1, ru, a, L);
        else group_body<T, MAXA, MPT, EXT, GS, NA, false>(h0, hb, h1, ru, a, L);
    });
}

// AF: 0 the child-list update, 1 the affine update with rows for 256 sets per group, 2 the affine
// update with rows for 128 (FP32 state, at most 4 actions)
constexpr int aff_sets(int AF) { return AF == 2 ? 128 : GROUP_SETS_MAX; }

template <typename T, int MAXA, int MPT, bool EXPLICIT, int AF>
using LevelLds = std::conditional_t<AF != 0, GroupLdsA<T, MAXA, MPT, aff_sets(AF)>, GroupLds<T, MAXA, MPT>>;

template <typename T, int MAXA, int MPT, bool EXPLICIT, bool EXT, int AF>
__device__ __forceinline__ void update_group(int32_t g, const RuleArgs &ru, const LevelArgs<T> &a,
                                             LevelLds<T, MAXA, MPT, EXPLICIT, AF> &L) {
    if constexpr (AF != 0) group_update_affine<T, MAXA, MPT, EXT, aff_sets(AF)>(g, ru, a, L);
    else group_update<T, MAXA, MPT, EXPLICIT, EXT>(g, ru, a, L);
}

// FP64 state with at most 4 actions and the lean rule tail: ask for 6 waves per SIMD (78 registers, no
// spills; the LDS of 6 workgroups fits) instead of the 5 that 86 registers allow.  The discounted and
// predictive tails would spill under that bound.  FP32 needs no bound: its registers allow 6 and its
// LDS too with 128-set groups (5 with 256).
template <typename T, int MAXA, bool EXT, int AF>
constexpr int level_min_waves() {
    if (MAXA > 4) return 1;
    if (sizeof(T) == 8) return EXT ? 1 : 6;
    return AF == 2 ? (EXT ? 5 : 6) : AF == 1 ? 5 : 1;
}
template <typename T, int MAXA, int MPT, bool EXPLICIT, bool EXT, int AF>
__global__ void __launch_bounds__(BLOCK, (level_min_waves<T, MAXA, EXT, AF>())) k_level(int32_t gbeg, int32_t ngroups, int32_t bbeg, int32_t nbig,
                                                 int32_t cbeg, int32_t nchance, LevelArgs<T> a,
                                                 const double *__restrict__ weights, int rule, int upd) {
    __shared__ LevelLds<T, MAXA, MPT, EXPLICIT, AF> L;
    const int32_t blk = (int32_t)blockIdx.x;
    // with retired games in a batch the ranges index lists of the work that still runs (a retired
    // game's values feed only its own parents)
    if (blk >= ngroups + nbig) {
        const int32_t j = (blk - ngroups - nbig) * BLOCK + (int32_t)threadIdx.x;
        if (j < nchance) chance_value<T, EXPLICIT>(a.chance_node[a.chance_list ? a.chance_list[cbeg + j] : cbeg + j], a);
        return;
    }
    if (blk >= ngroups) {
        const int32_t b = bbeg + blk - ngroups;
        big_chance_value<T, EXPLICIT>(a.bigc_node[a.bigc_list ? a.bigc_list[b] : b], a, L.po);
        return;
    }
    const int32_t x = gbeg + xcd_tile(blk, ngroups);
    const int32_t grp = a.grp_list ? a.grp_list[x] : x;
    const RuleArgs ru{rule, upd, weights[0], weights[1], weights[2], weights[3]};
    update_group<T, MAXA, MPT, EXPLICIT, EXT, AF>(grp, ru, a, L);
}

// Per-game barrier among the W blocks of one game.  Thread 0 publishes the block's writes
// (device-scope release), arrives on the game's counter and waits, with a bounded spin, until all
// W blocks of this epoch arrived; on time-out it raises the error flag and stops waiting, so every
// wave still exits.  Returns false once the error flag is up.
__device__ __forceinline__ bool game_barrier(int32_t *ctr, int32_t W, int32_t &epoch, int32_t *err,
                                             int64_t timeout_ticks) {
    __shared__ int32_t s_ok;
    if (W == 1) {
        __syncthreads();
        return true;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        epoch += 1;
        __threadfence();
        atomicAdd(ctr, 1);
        // Arrivals are counted modulo 2^32 and compared by signed difference, so the count may wrap
        // over a long launch.  The poll is a relaxed load: an acquiring load per poll would
        // invalidate this compute unit's caches on every spin.  One fence after the count is
        // reached makes the other blocks' writes visible.
        const uint32_t target = (uint32_t)epoch * (uint32_t)W;
        const int64_t t_start = (int64_t)wall_clock64();
        int32_t ok = 1;
        while ((int32_t)((uint32_t)__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
            if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                (int64_t)wall_clock64() - t_start > timeout_ticks) {
                atomicExch(err, 1);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        __threadfence();
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

// The work of one (game, rank): n_iter whole iterations of game gm as rank `rank` of its W workgroups,
// which stride over the game's slots (reach) and over each backward level's update groups and chance
// nodes and meet at the game's barrier between levels.  Iteration t0 + k (k = 1..n_iter) uses the
// same arithmetic, in the same order per set, as the level-synchronous kernels.  Returns false once
// a barrier reported an error.
template <typename T, int MAXA, int MPT, bool EXPLICIT, bool EXT, int AF>
__device__ bool persistent_game(int32_t gm, int32_t rank, int32_t W, const int32_t *__restrict__ game_range,
                                const int32_t *__restrict__ game_depth, int32_t MD, int32_t n_iter,
                                const LevelArgs<T> &a, int32_t t0, int32_t *barrier,
                                int32_t *err, int64_t timeout_ticks, int rule, int linear, int alternating,
                                LevelLds<T, MAXA, MPT, EXPLICIT, AF> &L) {
    const int32_t *gr = game_range + (size_t)gm * (MD + 1) * DR_FIELDS;
    const int32_t Ds = game_depth[gm];
    const int tid = threadIdx.x;
    int32_t epoch = 0;
    const int halves = alternating ? 2 : 1;
    for (int32_t it = 1; it <= n_iter; it++) {
        for (int half = 0; half < halves; half++) {
            const RuleArgs ru = rule_args(rule, linear, alternating ? 1 << half : 3, t0 + it);
            // A game's only workgroup synchronises for less than a walk's first step costs: its pass goes depth by
            // depth, a lookup per slot.  Several meet at a barrier of about 2 us, so they walk (one_launch_ranges):
            // once per set, since a thread has many.  Measured, us an iteration: 8 games of one workgroup in which
            // each player moves m times in a row, FP32, m = 8 49 (57 with a walk per slot or set), m = 50 280 (327 and
            // 338; 2,730 with whole sequences); game of 7 workgroups and 8 actions in which one move in seven goes
            // on, FP64, 199 (217 with a walk per slot).
            if (W == 1) {
                for (int32_t d = 0; d < Ds; d++) {
                    const int32_t *r = gr + d * DR_FIELDS;
                    const int32_t lo = r[0], hi = r[1] & ~REACH_CUT;
                    if (lo == hi) continue;
                    for (int32_t q = lo + tid; q < hi; q += BLOCK) a.seq[q] = a.seq[a.slot_par[q]] * a.sigma[q];
                    __syncthreads();
                }
            } else {
                int32_t S0 = 0;
                for (int32_t d = 0; d < Ds; d++) {
                    const int32_t *r = gr + d * DR_FIELDS;
                    if (r[1] & REACH_CUT) {
                        if (!game_barrier(barrier + gm, W, epoch, err, timeout_ticks)) return false;
                        S0 = r[0];
                    }
                    for (int32_t i = r[8] + rank * BLOCK + tid; i < r[9]; i += W * BLOCK) set_reach<T, MAXA>(i, S0, a);
                }
            }
            if (!game_barrier(barrier + gm, W, epoch, err, timeout_ticks)) return false;
            for (int32_t d = Ds - 1; d >= 0; d--) {
                const int32_t *r = gr + d * DR_FIELDS;
                for (int32_t g = r[2] + rank; g < r[3]; g += W) {
                    update_group<T, MAXA, MPT, EXPLICIT, EXT, AF>(g, ru, a, L);
                    __syncthreads();
                }
                for (int32_t b = r[6] + rank; b < r[7]; b += W) big_chance_value<T, EXPLICIT>(a.bigc_node[b], a, L.po);
                for (int32_t j = r[4] + rank * BLOCK + tid; j < r[5]; j += W * BLOCK) chance_value<T, EXPLICIT>(a.chance_node[j], a);
                if (!game_barrier(barrier + gm, W, epoch, err, timeout_ticks)) return false;
            }
        }
    }
    return true;
}

// The batched persistent form: one launch runs n_iter whole iterations of every game of a forest.
// The work is a list of tickets (game, rank, W), one queue per XCD: a game's W ranks are consecutive
// tickets of one queue.  A workgroup claims tickets of the queue of the XCD it runs on (the hardware
// XCC id), in order, runs each claimed rank to the end, then takes the other queues' remaining
// tickets.  A game's barrier therefore waits only for ranks claimed by workgroups already running,
// and the others are claimed next by whichever workgroup frees up: the launch needs one game's
// workgroups resident at once, not the whole grid, and any grid size is correct.
template <typename T, int MAXA, int MPT, bool EXPLICIT, bool EXT, int AF>
__global__ void __launch_bounds__(BLOCK) k_persistent(const int4 *__restrict__ tickets, const int32_t *__restrict__ q_off,
                                                      int32_t *claim, const int32_t *__restrict__ game_range,
                                                      const int32_t *__restrict__ game_depth, int32_t MD, int32_t n_iter,
                                                      LevelArgs<T> a,
                                                      const int32_t *__restrict__ tcount, int32_t *barrier,
                                                      int32_t *err, int64_t timeout_ticks, int rule, int linear,
                                                      int alternating) {
    __shared__ LevelLds<T, MAXA, MPT, EXPLICIT, AF> L;
    __shared__ int32_t s_ticket;
    const int32_t t0 = tcount[0];
    // XCC_ID hardware register (bits 3:0): the XCD this workgroup runs on
    const int home = (int)(__builtin_amdgcn_s_getreg((20) | (0 << 6) | ((4 - 1) << 11)) & (PERSISTENT_QUEUES - 1));
    for (int k = 0; k < PERSISTENT_QUEUES; k++) {
        const int q = (home + k) & (PERSISTENT_QUEUES - 1);
        const int32_t qlo = q_off[q], qn = q_off[q + 1] - qlo;
        for (;;) {
            if (threadIdx.x == 0) s_ticket = atomicAdd(claim + q, 1);
            __syncthreads();
            const int32_t t = s_ticket;
            __syncthreads();
            if (t >= qn) break;
            const int4 wt = tickets[qlo + t];
            if (!persistent_game<T, MAXA, MPT, EXPLICIT, EXT, AF>(wt.x, wt.y, wt.z, game_range, game_depth, MD, n_iter,
                                                                a, t0, barrier, err, timeout_ticks, rule, linear,
                                                                alternating, L))
                return;
        }
    }
}

// ---- the LDS-resident schedule for tiny standalone games --------------------------------------
//
// One workgroup runs n_iter whole iterations of a game whose state fits in LDS: the values (with
// the terminal template), the slots' reach, strategy, regrets, strategy sums and (PCFR+) the
// prediction are staged in, every level of every iteration runs between block barriers, and the
// state is written back at the end.  No launch per level and no trip to HBM inside the loop.  Where the
// structure arrays fit as well they are staged too (STAGED), since each level is a chain of dependent
// lookups in them.  One thread
// per information set walks its members in ascending order with the level kernels' arithmetic,
// so the iterates are bitwise those of the level launches.

// The update of one set by one thread: member values v(h) = sum_a sigma v(h.a), the set's
// instantaneous regrets summed over its members in ascending order, then set_update.
template <typename T, int MAXA, bool EXPLICIT, bool EXT, bool STAGED>
__device__ void set_serial(int32_t i, const RuleArgs &ru, const LevelArgs<T> &a) {
    const int32_t s0 = a.slot_off[i], nA = a.slot_off[i + 1] - s0;
    const int32_t m0 = a.mem_off[i], m1 = a.mem_off[i + 1];
    const int pl = STAGED ? a.player_words[i] : (int)a.iset_player[i];
    T sg[MAXA], r[MAXA];
#pragma unroll
    for (int k = 0; k < MAXA; k++) {
        sg[k] = a.sigma[s0 + min(k, nA - 1)];
        r[k] = T(0);
    }
    for (int32_t m = m0; m < m1; m++) {
        const int2 x = STAGED ? make_int2(a.mem_words[2 * m], a.mem_words[2 * m + 1]) : a.mem[m];
        const int32_t h = x.x & MEMBER_NODE_MASK;
        const T po = a.seq[a.mem_seq[m]];
        T cv[MAXA];
#pragma unroll
        for (int k = 0; k < MAXA; k++) cv[k] = a.v[child_of<EXPLICIT>(a.kid, x.y + min(k, nA - 1))];
        T vh = T(0);
#pragma unroll
        for (int k = 0; k < MAXA; k++) vh = k < nA ? fma_t(sg[k], cv[k], vh) : vh;
        a.v[h] = vh;
#pragma unroll
        for (int q = 0; q < MAXA; q++) r[q] = fma_t(po, cv[q] - vh, r[q]);
    }
    if (!((ru.upd >> (pl - 1)) & 1)) return;
    set_update<T, MAXA, EXT>(ru, a, s0, nA, pl, (double)a.seq[a.iset_seq[i]], r);
}

// The LDS a game is admitted by: strategy sums (double), then values and two words per node and
// strategy, regrets (and the PCFR+ prediction) per slot in the state type, then BLOCK reduction slots
// for big chance nodes.  k_lds uses less: instead of the two words per node it keeps A + 1 for the
// slots' reach (a game has fewer slots than nodes).
#if CFR_PART == 0
size_t lds_schedule_bytes(int32_t N, int32_t A, int fp64, int pred) {
    const size_t es = fp64 ? 8 : 4;
    return 8 * (size_t)A + es * (3 * (size_t)N + (pred ? 3 : 2) * (size_t)A + BLOCK);
}
#endif

// Sizes of the structure arrays that a staged game keeps in LDS, in 4-byte words.
struct LdsSizes {
    int32_t I, Ndec, E, C, B;   // sets, members, listed children, chance nodes, big chance nodes
};
__host__ __device__ inline size_t lds_structure_words(const LdsSizes &z, int32_t N, int32_t A, int32_t D) {
    return (size_t)A + 2 * ((size_t)z.I + 1) + 2 * (size_t)z.I + 3 * (size_t)z.Ndec + z.E + (N + 1) + z.C + z.B + 6 * (size_t)D;
}

template <typename T, int MAXA, bool EXPLICIT, bool EXT, bool STAGED>
__global__ void __launch_bounds__(BLOCK) k_lds(const int32_t *__restrict__ gr, int32_t n_cuts, int32_t D, int32_t N,
                                               int32_t A, LdsSizes z, int32_t n_iter, LevelArgs<T> g, int32_t *tcount, int rule,
                                               int linear, int alternating) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *sb = reinterpret_cast<double *>(smem);
    T *v = reinterpret_cast<T *>(sb + A);
    T *seq = v + N + 1, *sig = seq + A, *R = sig + A;   // seq[-1] = 1
    T *pred = g.pred ? R + A : nullptr;
    T *red = R + A + (g.pred ? A : 0);
    const int tid = threadIdx.x;
    const int32_t t0 = tcount[0];
    LevelArgs<T> a = g;
    // per depth: first set and the end, chance and big chance node ranges
    const int32_t *lv = nullptr;
    if constexpr (STAGED) {
        int32_t *w = reinterpret_cast<int32_t *>(red + BLOCK);
        auto take = [&](const int32_t *src, int32_t n) {
            int32_t *dst = w;
            for (int32_t i = tid; i < n; i += BLOCK) dst[i] = src[i];
            w += n;
            return dst;
        };
        int32_t *ranges = w;
        for (int32_t d = tid; d < D; d += BLOCK) {
            const int32_t *r = gr + d * DR_FIELDS;
            ranges[6 * d] = g.grp_iset_off[r[2]];
            ranges[6 * d + 1] = g.grp_iset_off[r[3]];
            for (int k = 0; k < 4; k++) ranges[6 * d + 2 + k] = r[4 + k];
        }
        w += 6 * D;
        lv = ranges;
        a.slot_par = take(g.slot_par, A);
        a.slot_off = take(g.slot_off, z.I + 1);
        a.mem_off = take(g.mem_off, z.I + 1);
        a.iset_seq = take(g.iset_seq, z.I);
        a.mem_seq = take(g.mem_seq, z.Ndec);
        a.kid_off = take(g.kid_off, N + 1);
        if (EXPLICIT) a.kid = take(g.kid, z.E);
        a.chance_node = take(g.chance_node, z.C);
        a.bigc_node = take(g.bigc_node, z.B);
        // members as two words each, players as one
        int32_t *mw = w;
        for (int32_t m = tid; m < z.Ndec; m += BLOCK) {
            const int2 x = g.mem[m];
            mw[2 * m] = x.x;
            mw[2 * m + 1] = x.y;
        }
        w += 2 * z.Ndec;
        for (int32_t i = tid; i < z.I; i += BLOCK) w[i] = g.iset_player[i];
        a.mem_words = mw;
        a.player_words = w;
    }
    for (int32_t i = tid; i < N; i += BLOCK) v[i] = g.v[i];
    if (tid == 0) seq[-1] = T(1);
    for (int32_t q = tid; q < A; q += BLOCK) {
        sb[q] = g.sbar[q];
        sig[q] = g.sigma[q];
        R[q] = g.R[q];
        if (pred) pred[q] = g.pred[q];
    }
    __syncthreads();
    a.v = v; a.seq = seq; a.sigma = sig; a.R = R; a.sbar = sb; a.pred = pred;
    const int halves = alternating ? 2 : 1;
    const int32_t *cuts = gr + (D + 1) * DR_FIELDS;
    // a walk per slot while every slot has a thread, then one per set (FP32, us an iteration: Kuhn's 24 slots 3.9
    // and 4.1; 1,696 slots of a 16-action game in which one move in ten goes on 35 and 27)
    const bool by_set = A > BLOCK;
    for (int32_t it = 1; it <= n_iter; it++) {
        for (int half = 0; half < halves; half++) {
            const RuleArgs ru = rule_args(rule, linear, alternating ? 1 << half : 3, t0 + it);
            // one part, unless sequences are longer than a walk
            auto part = [&](int32_t S0, int32_t S1, int32_t i0, int32_t i1) {
                if (by_set)
                    for (int32_t i = i0 + tid; i < i1; i += BLOCK) set_reach<T, MAXA>(i, S0, a);
                else
                    for (int32_t q = S0 + tid; q < S1; q += BLOCK)
                        seq[q] = seq_reach<T>(a.slot_par[q], S0, a.slot_par, sig, seq) * sig[q];
                __syncthreads();
            };
            int32_t S0 = 0, i0 = 0;
            for (int32_t c = 0; c < n_cuts; c++) {
                part(S0, cuts[2 * c], i0, cuts[2 * c + 1]);
                S0 = cuts[2 * c];
                i0 = cuts[2 * c + 1];
            }
            part(S0, A, i0, z.I);
            for (int32_t d = D - 1; d >= 0; d--) {
                int32_t ib, ie, cb, ce, bb, be;
                if constexpr (STAGED) {
                    const int32_t *r = lv + 6 * d;
                    ib = r[0]; ie = r[1]; cb = r[2]; ce = r[3]; bb = r[4]; be = r[5];
                } else {
                    const int32_t *r = gr + d * DR_FIELDS;
                    ib = g.grp_iset_off[r[2]]; ie = g.grp_iset_off[r[3]];
                    cb = r[4]; ce = r[5]; bb = r[6]; be = r[7];
                }
                for (int32_t i = ib + tid; i < ie; i += BLOCK) set_serial<T, MAXA, EXPLICIT, EXT, STAGED>(i, ru, a);
                for (int32_t j = cb + tid; j < ce; j += BLOCK) chance_value<T, EXPLICIT>(a.chance_node[j], a);
                for (int32_t b = bb; b < be; b++) big_chance_value<T, EXPLICIT>(a.bigc_node[b], a, red);
                __syncthreads();
            }
        }
    }
    if (tid == 0) tcount[0] = t0 + n_iter;
    for (int32_t i = tid; i < N; i += BLOCK) g.v[i] = v[i];
    for (int32_t q = tid; q < A; q += BLOCK) {
        g.sbar[q] = sb[q];
        g.sigma[q] = sig[q];
        g.R[q] = R[q];
        if (pred) g.pred[q] = pred[q];
    }
}

#if CFR_PART == 0
__global__ void k_fill_int(int32_t n, int32_t *p, int32_t value) {
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = value;
}

__global__ void k_add_counter(int32_t *t, int32_t n) {
    if (threadIdx.x == 0) t[0] += n;
}

template <typename T>
__global__ void __launch_bounds__(BLOCK) k_regret_matching(int32_t I, const int32_t *__restrict__ slot_off,
                                                           const T *__restrict__ R, const T *__restrict__ pred,
                                                           T *__restrict__ sigma) {
    int32_t i = (int32_t)(blockIdx.x * BLOCK + threadIdx.x);
    if (i >= I) return;
    int32_t s0 = slot_off[i], s1 = slot_off[i + 1];
    // PCFR+: regret matching of R + prediction
    auto x = [&](int32_t q) { return pred ? R[q] + pred[q] : R[q]; };
    T tot = T(0);
    for (int32_t q = s0; q < s1; q++) tot += max_t(x(q), T(0));
    const T inv = tot > T(0) ? T(1) / tot : T(0);
    const T uni = T(1) / (T)(s1 - s0);
    for (int32_t q = s0; q < s1; q++) sigma[q] = tot > T(0) ? max_t(x(q), T(0)) * inv : uni;
}

__global__ void k_tick(int32_t *t) {
    if (threadIdx.x == 0) t[0] += 1;
}

// dst[map i] = src[i] (map == nullptr: identity)
template <typename S, typename D>
__global__ void __launch_bounds__(BLOCK) k_scatter(int32_t n, const int32_t *__restrict__ map,
                                                   const S *__restrict__ src, D *__restrict__ dst) {
    int32_t i = (int32_t)(blockIdx.x * BLOCK + threadIdx.x);
    if (i < n) dst[map ? map[i] : i] = (D)src[i];
}

// dst[map i] += src[i]
template <typename S, typename D>
__global__ void __launch_bounds__(BLOCK) k_scatter_add(int32_t n, const int32_t *__restrict__ map,
                                                       const S *__restrict__ src, D *__restrict__ dst) {
    int32_t i = (int32_t)(blockIdx.x * BLOCK + threadIdx.x);
    if (i < n) {
        const int32_t j = map ? map[i] : i;
        dst[j] = dst[j] + (D)src[i];
    }
}

// ---- in-place re-solve: the chance-folded template of a game's terminals ---------------------
__global__ void __launch_bounds__(BLOCK) k_gather_payoffs(int64_t lo, int64_t hi, const int32_t *__restrict__ in,
                                                          const double *__restrict__ pay, double *__restrict__ u) {
    const int64_t j = lo + (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (j < hi) u[j] = pay[in[j]];
}

template <typename T>
__global__ void __launch_bounds__(BLOCK) k_template(int64_t lo, int64_t hi, const int32_t *__restrict__ node,
                                                    const int32_t *__restrict__ branch, const double *__restrict__ u,
                                                    const double *__restrict__ pic, const double *__restrict__ root,
                                                    T *__restrict__ v, double *__restrict__ v0) {
    const int64_t j = lo + (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (j >= hi) return;
    const double c = root ? root[branch[j]] * pic[j] : pic[j];
    const double t = c * u[j];
    v[node[j]] = (T)t;
    v0[node[j]] = t;
}

// The template under new root ranges.  A game's call is bound by its fixed costs, so the ranges are kernel
// arguments (a block keeps them in LDS, since arguments may lie in host memory) and every terminal computes
// its own root chance: no copy of the root's chances before the launch.  64 subgames, a call each:
// 18.6 us a call instead of 23.1, most of them the wait for the stream.
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_template_ranges(int64_t lo, int64_t hi, const int32_t *__restrict__ node,
                                                           const int32_t *__restrict__ branch,
                                                           const double *__restrict__ u, const double *__restrict__ pic,
                                                           const int2 *__restrict__ hands, int64_t n, RangeArgs a,
                                                           double *__restrict__ root, T *__restrict__ v,
                                                           double *__restrict__ v0) {
    __shared__ double r[RANGE_MAX];
    for (int k = threadIdx.x; k < a.n1 + a.n2; k += BLOCK) r[k] = a.r[k];
    __syncthreads();
    const int64_t k = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    auto chance = [&](int64_t b) {
        const int2 h = hands[b];
        return r[h.x] * r[a.n1 + h.y] / a.total;
    };
    if (k < n) root[k] = chance(k);
    const int64_t j = lo + k;
    if (j >= hi) return;
    const double c = chance(branch[j]) * pic[j];
    const double t = c * u[j];
    v[node[j]] = (T)t;
    v0[node[j]] = t;
}
#endif

// ---- launchers ------------------------------------------------------------

#if CFR_PART == 0
template <typename T>
static hipError_t reach_t(const DevGame &g, int32_t lo, int32_t hi, bool walk, int32_t *tick, IterFlags f,
                          const int32_t *tiles, int64_t n_tiles, hipStream_t s) {
    // one block still runs the counter bump
    if (tiles && n_tiles == 0) hi = lo;
    const int32_t tile = reach_tile(walk);
    const unsigned blocks = hi <= lo ? 1u : tiles ? (unsigned)n_tiles : (unsigned)(((int64_t)hi - lo + tile - 1) / tile);
    if (walk)
        hipLaunchKernelGGL((k_reach<T, true>), dim3(blocks), dim3(BLOCK), 0, s, lo, hi, lo, g.slot_par,
                           (const T *)g.sigma, (T *)g.seq, tick, g.weights, f.rule, f.linear, tiles);
    else
        hipLaunchKernelGGL((k_reach<T, false>), dim3(blocks), dim3(BLOCK), 0, s, lo, hi, lo, g.slot_par,
                           (const T *)g.sigma, (T *)g.seq, tick, g.weights, f.rule, f.linear, tiles);
    return hipGetLastError();
}

hipError_t launch_reach(const DevGame &g, int k, int32_t lo, int32_t hi, bool walk, int32_t *tick, IterFlags f,
                        hipStream_t s) {
    if (hi <= lo && !tick) return hipSuccess;
    const int32_t *tiles = g.use_lists ? g.reach_list + g.reach_off[k] : nullptr;
    const int64_t nt = g.use_lists ? g.reach_off[k + 1] - g.reach_off[k] : 0;
    if (g.use_lists && nt == 0 && !tick) return hipSuccess;
    return g.fp64 ? reach_t<double>(g, lo, hi, walk, tick, f, tiles, nt, s) : reach_t<float>(g, lo, hi, walk, tick, f, tiles, nt, s);
}
#endif

#if CFR_PART == 0
// launch k of the reach pass on the average strategy (sigbar into seqbar)
hipError_t launch_reach_average(const DevGame &g, int32_t lo, int32_t hi, bool walk, hipStream_t s) {
    if (hi <= lo) return hipSuccess;
    const unsigned blocks = (unsigned)(((int64_t)hi - lo + reach_tile(walk) - 1) / reach_tile(walk));
    if (walk)
        hipLaunchKernelGGL((k_reach<double, true>), dim3(blocks), dim3(BLOCK), 0, s, lo, hi, lo, g.slot_par, g.sigbar,
                           g.seqbar, nullptr, nullptr, 0, 0, nullptr);
    else
        hipLaunchKernelGGL((k_reach<double, false>), dim3(blocks), dim3(BLOCK), 0, s, lo, hi, lo, g.slot_par, g.sigbar,
                           g.seqbar, nullptr, nullptr, 0, 0, nullptr);
    return hipGetLastError();
}
#endif

template <typename T>
static LevelArgs<T> level_args(const DevGame &g) {
    LevelArgs<T> a;
    a.grp_iset_off = g.grp_iset_off; a.slot_off = g.slot_off; a.mem_off = g.mem_off; a.mem = g.mem;
    a.iset_player = g.iset_player; a.kid_off = g.kid_off; a.kid = g.kid; a.chance_node = g.chance_node;
    a.bigc_node = g.bigc_node;
    a.iset_seq = g.iset_seq; a.slot_par = g.slot_par; a.mem_seq = g.mem_seq;
    a.koff = g.koff; a.ghdr = g.ghdr; a.srec = g.srec; a.mwide = g.mwide; a.mrec = g.mrec; a.mpos = g.mpos;
    a.grp_list = g.use_lists ? g.grp_list : nullptr;
    a.chance_list = g.use_lists ? g.chance_list : nullptr;
    a.bigc_list = g.use_lists ? g.bigc_list : nullptr;
    a.v = (T *)g.v;
    a.seq = (T *)g.seq;
    a.R = (T *)g.R; a.sbar = g.sbar; a.sigma = (T *)g.sigma;
    a.pred = (T *)g.pred;
    return a;
}

template <typename T, int MAXA, int MPT, bool EX, bool XT, int AF>
static hipError_t level_t(const DevGame &g, int d, IterFlags f, hipStream_t s) {
    // all work of depth d, or with retired games the listed part of it
    const int32_t gbeg = g.use_lists ? (int32_t)g.grp_off[d] : g.grp_depth_off[d];
    const int32_t ng = g.use_lists ? (int32_t)(g.grp_off[d + 1] - g.grp_off[d]) : g.grp_depth_off[d + 1] - gbeg;
    const int32_t cbeg = g.use_lists ? (int32_t)g.chance_off_l[d] : g.chance_off[d];
    const int32_t nc = g.use_lists ? (int32_t)(g.chance_off_l[d + 1] - g.chance_off_l[d]) : g.chance_off[d + 1] - cbeg;
    const int32_t bbeg = g.use_lists ? (int32_t)g.bigc_off_l[d] : g.bigc_off[d];
    const int32_t nb = g.use_lists ? (int32_t)(g.bigc_off_l[d + 1] - g.bigc_off_l[d]) : g.bigc_off[d + 1] - bbeg;
    const unsigned blocks = (unsigned)ng + (unsigned)nb + grid_for(nc);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((k_level<T, MAXA, MPT, EX, XT, AF>), dim3(blocks), dim3(BLOCK), 0, s,
                       gbeg, ng, bbeg, nb, cbeg, nc, level_args<T>(g), g.weights, f.rule, f.upd);
    return hipGetLastError();
}

// the discounted and predictive rules get their own instantiation, so CFR and CFR+ keep a lean update
inline bool ext_rule(int rule) { return rule == CFR_RULE_DCFR || rule == CFR_RULE_PCFR_PLUS; }

// Instantiation selector shared by the level and persistent launches: state type, action bound
// (members per thread must match the group capacity the compiler used, group_members: four for
// FP32 state with at most 4 actions, two for FP64, else one), child addressing (implicit,
// explicit, affine; AF, see aff_sets) and rule class.
template <typename T, bool EX, bool XT, int AF, typename F>
static auto by_actions(const DevGame &g, F &&f) {
    static_assert(AF != 2 || sizeof(T) == 4, "128-set rows are an FP32 instantiation");
    if constexpr (AF == 2) {
        return f.template operator()<T, 4, 4, EX, XT, 2>();
    } else {
        if (g.max_actions <= 4) return f.template operator()<T, 4, sizeof(T) == 4 ? 4 : 2, EX, XT, AF>();
        if (g.max_actions <= 16) return f.template operator()<T, 16, 1, EX, XT, AF>();
        return f.template operator()<T, 64, 1, EX, XT, AF>();
    }
}

template <typename T, typename F>
static auto by_kind(const DevGame &g, int rule, F &&f) {
    const bool x = ext_rule(rule);
    if (g.affine) {
        // FP32 state, at most 4 actions, groups of at most 128 sets: the instantiation with 128-set rows
        if constexpr (sizeof(T) == 4)
            if (g.max_actions <= 4 && g.group_sets == 128)
                return x ? by_actions<T, true, true, 2>(g, f) : by_actions<T, true, false, 2>(g, f);
        return x ? by_actions<T, true, true, 1>(g, f) : by_actions<T, true, false, 1>(g, f);
    }
    if (g.explicit_kids) return x ? by_actions<T, true, true, 0>(g, f) : by_actions<T, true, false, 0>(g, f);
    return x ? by_actions<T, false, true, 0>(g, f) : by_actions<T, false, false, 0>(g, f);
}

struct LevelLaunch {
    const DevGame &g; int d; IterFlags f; hipStream_t s;
    template <typename T, int MAXA, int MPT, bool EX, bool XT, int AF>
    hipError_t operator()() const { return level_t<T, MAXA, MPT, EX, XT, AF>(g, d, f, s); }
};

#if CFR_PART == 1 || CFR_PART == 2
hipError_t LEVEL_OF(const DevGame &g, int d, IterFlags f, hipStream_t s) {
    return by_kind<PartT>(g, f.rule, LevelLaunch{g, d, f, s});
}
#endif

struct PersistentLaunch {
    const DevGame &g; const PersistentPlan &p; int32_t T_; IterFlags f; int alt; hipStream_t s;
    template <typename T, int MAXA, int MPT, bool EX, bool XT, int AF>
    hipError_t operator()() const {
        hipLaunchKernelGGL((k_persistent<T, MAXA, MPT, EX, XT, AF>), dim3(p.blocks), dim3(BLOCK), 0, s, p.tickets,
                           p.q_off, p.claim, p.game_range, p.game_depth, p.max_depth, T_, level_args<T>(g), g.t,
                           p.barrier, p.err, p.timeout_ticks, f.rule, f.linear, alt);
        return hipGetLastError();
    }
};

#if CFR_PART == 3 || CFR_PART == 4
hipError_t PERSISTENT_OF(const DevGame &g, const PersistentPlan &p, int32_t T_, IterFlags f, int alt, hipStream_t s) {
    return by_kind<PartT>(g, f.rule, PersistentLaunch{g, p, T_, f, alt, s});
}
#endif

struct LdsLaunch {
    const DevGame &g; const int32_t *gr; int32_t n_cuts, T_; IterFlags f; int alt; hipStream_t s; size_t bytes;
    bool prepare;   // true: only raise the kernel's dynamic LDS limit to bytes
    template <typename T, int MAXA, int MPT, bool EX, bool XT, int AF>
    hipError_t operator()() const {
        if constexpr (MAXA > 16) {
            return hipErrorInvalidValue;
        } else if (MAXA == 4 && g.max_actions <= 2) {
            // a tiny game is bound by the instructions of its few busy waves: half the columns take Kuhn's 20
            // iterations from 84 to 73 us
            return operator()<T, 2, MPT, EX, XT, AF>();
        } else {
            const LdsSizes z{g.I, g.Ndec, EX ? g.E : 0, g.chance_off[g.max_depth + 1], g.bigc_off[g.max_depth + 1]};
            const size_t whole = bytes + 4 * lds_structure_words(z, g.N, g.A, g.max_depth);
            const bool staged = whole <= (size_t)g.lds_limit;
            auto fn = staged ? k_lds<T, MAXA, EX, XT, true> : k_lds<T, MAXA, EX, XT, false>;
            if (prepare)
                return hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(staged ? whole : bytes));
            hipLaunchKernelGGL(fn, dim3(1), dim3(BLOCK), staged ? whole : bytes, s, gr, n_cuts, g.max_depth, g.N, g.A, z, T_,
                               level_args<T>(g), g.t, f.rule, f.linear, alt);
            return hipGetLastError();
        }
    }
};

// the serial update reads the child list when the layout has one (affine offsets serve only the
// member-parallel form)
template <typename T>
static hipError_t lds_dispatch(const DevGame &g, const LdsLaunch &L) {
    const bool x = ext_rule(L.f.rule);
    if (g.explicit_kids) return x ? by_actions<T, true, true, 0>(g, L) : by_actions<T, true, false, 0>(g, L);
    return x ? by_actions<T, false, true, 0>(g, L) : by_actions<T, false, false, 0>(g, L);
}

#if CFR_PART == 3 || CFR_PART == 4
hipError_t LDS_OF(const DevGame &g, const int32_t *gr, int32_t n_cuts, int32_t T_, IterFlags f, int alt, hipStream_t s,
                  size_t bytes, bool prepare) {
    return lds_dispatch<PartT>(g, LdsLaunch{g, gr, n_cuts, T_, f, alt, s, bytes, prepare});
}
#endif

struct PersistentFn {
    template <typename T, int MAXA, int MPT, bool EX, bool XT, int AF>
    const void *operator()() const { return reinterpret_cast<const void *>(&k_persistent<T, MAXA, MPT, EX, XT, AF>); }
};

#if CFR_PART == 3 || CFR_PART == 4
const void *PERSISTENT_FN_OF(const DevGame &g) { return by_kind<PartT>(g, g.rule, PersistentFn{}); }
#endif

#if CFR_PART == 0
hipError_t launch_level(const DevGame &g, int d, IterFlags f, hipStream_t s) {
    return g.fp64 ? level_f64(g, d, f, s) : level_f32(g, d, f, s);
}

hipError_t launch_persistent(const DevGame &g, const PersistentPlan &p, int32_t T_, IterFlags f, int alt,
                             hipStream_t s) {
    // the barrier counters and, right after them, the queues' claim counters start at zero
    const int32_t nz = p.n_games + PERSISTENT_QUEUES;
    hipLaunchKernelGGL(k_fill_int, dim3((nz + 255) / 256), dim3(256), 0, s, nz, p.barrier, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = g.fp64 ? persistent_f64(g, p, T_, f, alt, s) : persistent_f32(g, p, T_, f, alt, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_add_counter, dim3(1), dim3(64), 0, s, g.t, T_);
    return hipGetLastError();
}

hipError_t prepare_lds(const DevGame &g, int rule, size_t *bytes) {
    *bytes = lds_schedule_bytes(g.N, g.A, g.fp64, g.pred != nullptr);
    if (g.max_actions > 16) return hipErrorInvalidValue;
    const IterFlags f{rule, 0, 3};
    return g.fp64 ? lds_f64(g, nullptr, 0, 0, f, 0, nullptr, *bytes, true) : lds_f32(g, nullptr, 0, 0, f, 0, nullptr, *bytes, true);
}

hipError_t launch_lds(const DevGame &g, const int32_t *ranges, int32_t n_cuts, int32_t T_, IterFlags f, int alt,
                      hipStream_t s) {
    const size_t bytes = lds_schedule_bytes(g.N, g.A, g.fp64, g.pred != nullptr);
    return g.fp64 ? lds_f64(g, ranges, n_cuts, T_, f, alt, s, bytes, false)
                  : lds_f32(g, ranges, n_cuts, T_, f, alt, s, bytes, false);
}

// the instantiation launch_persistent uses for this game
hipError_t persistent_occupancy(const DevGame &g, int *blocks_per_cu) {
    const void *fn = g.fp64 ? persistent_fn_f64(g) : persistent_fn_f32(g);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, BLOCK, 0);
}

hipError_t launch_regret_matching(const DevGame &g, hipStream_t s) {
    if (g.I == 0) return hipSuccess;
    if (g.fp64)
        hipLaunchKernelGGL(k_regret_matching<double>, dim3(grid_for(g.I)), dim3(BLOCK), 0, s, g.I, g.slot_off,
                           (const double *)g.R, (const double *)g.pred, (double *)g.sigma);
    else
        hipLaunchKernelGGL(k_regret_matching<float>, dim3(grid_for(g.I)), dim3(BLOCK), 0, s, g.I, g.slot_off,
                           (const float *)g.R, (const float *)g.pred, (float *)g.sigma);
    return hipGetLastError();
}

hipError_t launch_tick(const DevGame &g, hipStream_t s) {
    hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, s, g.t);
    return hipGetLastError();
}

hipError_t launch_regrets_from_float(const DevGame &g, const float *src, hipStream_t s) {
    if (g.A == 0) return hipSuccess;
    if (g.fp64)
        hipLaunchKernelGGL((k_scatter<float, double>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map, src,
                           (double *)g.R);
    else
        hipLaunchKernelGGL((k_scatter<float, float>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map, src,
                           (float *)g.R);
    return hipGetLastError();
}

hipError_t launch_regrets_add_float(const DevGame &g, const float *src, hipStream_t s) {
    if (g.A == 0) return hipSuccess;
    if (g.fp64)
        hipLaunchKernelGGL((k_scatter_add<float, double>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map,
                           src, (double *)g.R);
    else
        hipLaunchKernelGGL((k_scatter_add<float, float>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map,
                           src, (float *)g.R);
    return hipGetLastError();
}

// dst[map q] <- src[q] for a canonical FP64 source: into the state type (R, prediction) or into the FP64
// strategy sums
hipError_t launch_scatter_double(const DevGame &g, const double *src, void *dst, bool state_type, hipStream_t s) {
    if (g.A == 0) return hipSuccess;
    if (!state_type)
        hipLaunchKernelGGL((k_scatter<double, double>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map, src,
                           (double *)dst);
    else if (g.fp64)
        hipLaunchKernelGGL((k_scatter<double, double>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map, src,
                           (double *)dst);
    else
        hipLaunchKernelGGL((k_scatter<double, float>), dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, g.slot_map, src,
                           (float *)dst);
    return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(BLOCK) k_zero(int32_t n, T *__restrict__ p) {
    const int32_t i = (int32_t)(blockIdx.x * BLOCK + threadIdx.x);
    if (i < n) p[i] = T(0);
}

// A slots of the state type set to zero (a fill kernel, so it may sit in a captured graph)
hipError_t launch_fill_state(const DevGame &g, void *dst, hipStream_t s) {
    if (g.A == 0) return hipSuccess;
    if (g.fp64) hipLaunchKernelGGL(k_zero<double>, dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, (double *)dst);
    else hipLaunchKernelGGL(k_zero<float>, dim3(grid_for(g.A)), dim3(BLOCK), 0, s, g.A, (float *)dst);
    return hipGetLastError();
}

hipError_t launch_gather_payoffs(int64_t lo, int64_t hi, const int32_t *in, const double *payoff_in, double *u,
                                 hipStream_t s) {
    if (hi <= lo) return hipSuccess;
    hipLaunchKernelGGL(k_gather_payoffs, dim3((unsigned)((hi - lo + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, lo, hi,
                       in, payoff_in, u);
    return hipGetLastError();
}

hipError_t launch_template(const DevGame &g, int64_t lo, int64_t hi, const int32_t *node, const int32_t *branch,
                           const double *u, const double *pic, const double *root, hipStream_t s) {
    if (hi <= lo) return hipSuccess;
    const dim3 grid((unsigned)((hi - lo + BLOCK - 1) / BLOCK));
    if (g.fp64)
        hipLaunchKernelGGL(k_template<double>, grid, dim3(BLOCK), 0, s, lo, hi, node, branch, u, pic, root,
                           (double *)g.v, g.val[0]);
    else
        hipLaunchKernelGGL(k_template<float>, grid, dim3(BLOCK), 0, s, lo, hi, node, branch, u, pic, root,
                           (float *)g.v, g.val[0]);
    return hipGetLastError();
}

hipError_t launch_template_ranges(const DevGame &g, int64_t lo, int64_t hi, const int32_t *node, const int32_t *branch,
                                  const double *u, const double *pic, const int2 *hands, int64_t n,
                                  const RangeArgs &ranges, double *root, hipStream_t s) {
    const int64_t work = std::max(hi - lo, n);
    if (work <= 0) return hipSuccess;
    const dim3 grid((unsigned)((work + BLOCK - 1) / BLOCK));
    if (g.fp64)
        hipLaunchKernelGGL(k_template_ranges<double>, grid, dim3(BLOCK), 0, s, lo, hi, node, branch, u, pic, hands, n,
                           ranges, root, (double *)g.v, g.val[0]);
    else
        hipLaunchKernelGGL(k_template_ranges<float>, grid, dim3(BLOCK), 0, s, lo, hi, node, branch, u, pic, hands, n,
                           ranges, root, (float *)g.v, g.val[0]);
    return hipGetLastError();
}

#endif  // CFR_PART == 0

}  // namespace cfrx
