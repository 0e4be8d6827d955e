// evaluate.hip -- what a solve hands out: the current and average strategy in canonical order, and the
// exploitability of the average profile (eq. exploitability) in FP64.
//
// Exploitability needs three values per node: v0 under the average profile, and vi where player i plays
// his best response to it (i = 1, 2).  One sweep over the compiled levels computes all three: below a set
// of player i, v0 and the other player's vj are averages over the set's actions, and vi takes the action a
// that maximises Q(I, a) = sum_h q(h) s_i vi(h.a), lowest index on ties, with q(h) the other player's reach
// of member h, that is of his last sequence (k_reach on the average strategy).  Terminals hold their
// template once, in v0.
#include "common.hpp"
#include "compiler.hpp"
#include "device.hpp"

namespace cfrx {
namespace {

// dst <- the strategy sums over their set's total (uniform where that is 0).  A block takes 256 sets of one
// order, whose slots are contiguous in that order: device order (map == nullptr), or the canonical order
// with the device slots in map.  They go through LDS, all loads of a thread in flight together and
// coalesced where the orders agree, where at most NORM_SLOTS (1024: up to four actions per set) are there; else
// each thread reads its set's own (contiguous in both orders).  A pass in device order, a gather into
// canonical order and a copy took 128 us for the 11.2M slots of the 37.6M-node card game, this
// takes 54 us (20 bytes per slot and the lines that the map scatters over).
constexpr int NORM_SLOTS = 1024;
template <typename D>
__global__ void __launch_bounds__(BLOCK) k_normalise(int32_t I, const int32_t *__restrict__ off,
                                                     const int32_t *__restrict__ map, const double *__restrict__ sbar,
                                                     D *__restrict__ dst) {
    __shared__ double sb[NORM_SLOTS];
    const int32_t i0 = (int32_t)blockIdx.x * BLOCK, i1 = min(I, i0 + BLOCK);
    const int32_t S0 = off[i0], S1 = off[i1];
    const int32_t i = i0 + (int32_t)threadIdx.x;
    const int32_t s0 = off[min(i, i1 - 1)], n = off[min(i, i1 - 1) + 1] - s0;
    const double uni = 1.0 / (double)n;
    if (S1 - S0 > NORM_SLOTS) {
        if (i >= i1) return;
        const double *x = sbar + (map ? map[s0] : s0);
        double tot = 0.0;
        for (int32_t k = 0; k < n; k++) tot += x[k];
        for (int32_t k = 0; k < n; k++) dst[s0 + k] = (D)(tot > 0.0 ? x[k] / tot : uni);
        return;
    }
    constexpr int P = NORM_SLOTS / BLOCK;
    int32_t q[P];
#pragma unroll
    for (int u = 0; u < P; u++) {
        q[u] = min(S0 + u * BLOCK + (int32_t)threadIdx.x, S1 - 1);
        if (map) q[u] = map[q[u]];
    }
    double x[P];
#pragma unroll
    for (int u = 0; u < P; u++) x[u] = sbar[q[u]];
#pragma unroll
    for (int u = 0; u < P; u++) sb[u * BLOCK + threadIdx.x] = x[u];
    __syncthreads();
    if (i < i1) {
        double tot = 0.0;
        for (int32_t k = 0; k < n; k++) tot += sb[s0 - S0 + k];
        for (int32_t k = 0; k < n; k++) sb[s0 - S0 + k] = tot > 0.0 ? sb[s0 - S0 + k] / tot : uni;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < P; u++)
        if (S0 + u * BLOCK + (int32_t)threadIdx.x < S1)
            dst[S0 + u * BLOCK + threadIdx.x] = (D)sb[u * BLOCK + threadIdx.x];
}

// dst[i] = src[map i] as float (map == nullptr: identity), four per thread in flight together
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_gather(int32_t n, const int32_t *__restrict__ map, const T *__restrict__ src,
                                                  float *__restrict__ dst) {
    constexpr int P = 4;
    const int32_t base = (int32_t)blockIdx.x * (BLOCK * P) + (int32_t)threadIdx.x;
    int32_t q[P];
    T x[P];
#pragma unroll
    for (int u = 0; u < P; u++) {
        q[u] = min(base + u * BLOCK, n - 1);
        if (map) q[u] = map[q[u]];
    }
#pragma unroll
    for (int u = 0; u < P; u++) x[u] = src[q[u]];
#pragma unroll
    for (int u = 0; u < P; u++)
        if (base + u * BLOCK < n) dst[base + u * BLOCK] = (float)x[u];
}

struct EvalArgs {
    const int32_t *grp_iset_off, *slot_off, *mem_off, *mem_seq, *kid_off, *kid, *koff;
    const int4 *ghdr;
    const int2 *mwide;
    const uint32_t *mrec;
    const int2 *mem;
    const uint16_t *mpos;
    const int8_t *iset_player;
    const uint8_t *slot_kids;            // KIDS_* bits of the children below each slot
    const int32_t *chance_node, *bigc_node;
    const uint8_t *chance_kids, *bigc_kids;
    const double *sigbar, *seqbar;
    double *v0, *v1, *v2;
};

// how a member's child is found: numbered (breadth-first layout), listed, or at an offset per slot
enum { ADDR_IMPLICIT = 0, ADDR_LIST = 1, ADDR_OFFSET = 2 };

constexpr uint8_t KIDS_MIXED = KIDS_TERMINAL | KIDS_INTERNAL;

// whether child c, below a slot or chance node with children of `kinds`, is a terminal (a lookup only
// where the kinds are mixed)
__device__ __forceinline__ bool is_leaf(uint8_t kinds, int32_t c, const int32_t *__restrict__ kid_off) {
    return kinds == KIDS_TERMINAL || (kinds == KIDS_MIXED && kid_off[c] == kid_off[c + 1]);
}

// the three values of child c; a terminal's are its template, and the loads stay unconditional
struct Three { double x0, x1, x2; };
__device__ __forceinline__ Three three(const EvalArgs &a, int32_t c, bool leaf) {
    const double *p1 = leaf ? a.v0 : a.v1, *p2 = leaf ? a.v0 : a.v2;
    return {a.v0[c], p1[c], p2[c]};
}

// the sums of the values of children b, b + step, ... below e of a chance node, four loads of each in flight
template <int ADDR, bool MIXED>
__device__ __forceinline__ Three chance_slice(const EvalArgs &a, int32_t b, int32_t e, int32_t step, uint8_t kinds) {
    constexpr int U = 4;
    Three s{0.0, 0.0, 0.0};
    for (int32_t c0 = b; c0 < e; c0 += U * step) {
        int32_t c[U];
        Three t[U];
#pragma unroll
        for (int i = 0; i < U; i++) {
            const int32_t x = c0 + i * step < e ? c0 + i * step : c0;
            c[i] = ADDR == ADDR_IMPLICIT ? x : a.kid[x];
        }
#pragma unroll
        for (int i = 0; i < U; i++)
            t[i] = three(a, c[i], MIXED ? is_leaf(kinds, c[i], a.kid_off) : kinds == KIDS_TERMINAL);
#pragma unroll
        for (int i = 0; i < U; i++)
            if (c0 + i * step < e) { s.x0 += t[i].x0; s.x1 += t[i].x1; s.x2 += t[i].x2; }
    }
    return s;
}
template <int ADDR>
__device__ __forceinline__ Three chance_sum(const EvalArgs &a, int32_t b, int32_t e, int32_t step, uint8_t kinds) {
    return kinds == KIDS_MIXED ? chance_slice<ADDR, true>(a, b, e, step, kinds)
                               : chance_slice<ADDR, false>(a, b, e, step, kinds);
}

// lanes that share a chance node of at most BIG_FANOUT children
constexpr int CHANCE_LANES = 8;

template <int MAXA, int MPT>
struct EvalLds {
    double diff[MPT * BLOCK * MAXA];
    int32_t slot[BLOCK + 1], moff[BLOCK + 1];
    int8_t pl[BLOCK];
    uint8_t best[BLOCK];
    int32_t wide[BLOCK / 64], mixed;
    uint8_t mset[GROUP_MEMBERS_MAX];
};

// One level of the sweep: update groups as the iteration's (blocks [0, ngroups)), big chance nodes (a block
// each), chance nodes (eight lanes each).  A group's members go through LDS in chunks: each thread takes MPT
// members, stores their averages and stages their weighted child values; a thread per set sums them in
// member order and picks the action; a second pass over the members, whose lines are in the cache, stores
// the best responder's value.  A chunk holds every group of several sets, so affine layouts take the
// members in their listed order (node order where sets interleave) as the iteration does.  Bound by
// memory for large games and by the launches for small ones.
// Measured (three sweeps with separate reach, argmax and value launches before): 256 subgames of 28.1M
// nodes 13.5 -> 0.37 ms, of which 11 ms were root deals of up to 11,000 pairs summed by one thread; card
// game of 10.0M nodes 0.92 -> 0.29 ms.
template <int MAXA, int MPT, int ADDR>
__global__ void __launch_bounds__(BLOCK) k_eval_level(int32_t gbeg, int32_t ngroups, int32_t bbeg, int32_t nbig,
                                                      int32_t cbeg, int32_t nchance, EvalArgs a) {
    __shared__ EvalLds<MAXA, MPT> L;
    constexpr int CHUNK = MPT * BLOCK;
    const int tid = threadIdx.x;
    const int32_t blk = (int32_t)blockIdx.x;
    if (blk >= ngroups + nbig) {
        // each lane of a node sums a strided slice of its children, then the lanes add up in a fixed tree
        const int32_t j = (blk - ngroups - nbig) * (BLOCK / CHANCE_LANES) + tid / CHANCE_LANES;
        const int32_t jj = min(j, nchance - 1);
        const int32_t h = a.chance_node[cbeg + jj];
        const int32_t b = a.kid_off[h], e = a.kid_off[h + 1];
        Three s = chance_sum<ADDR>(a, b + tid % CHANCE_LANES, e, CHANCE_LANES, a.chance_kids[cbeg + jj]);
#pragma unroll
        for (int off = CHANCE_LANES / 2; off >= 1; off >>= 1) {
            s.x0 += __shfl_xor(s.x0, off);
            s.x1 += __shfl_xor(s.x1, off);
            s.x2 += __shfl_xor(s.x2, off);
        }
        if (j < nchance && tid % CHANCE_LANES == 0) { a.v0[h] = s.x0; a.v1[h] = s.x1; a.v2[h] = s.x2; }
        return;
    }
    if (blk >= ngroups) {
        // each thread sums a strided slice of the children in order, then a tree over the block
        const int32_t j = bbeg + blk - ngroups, h = a.bigc_node[j];
        const int32_t b = a.kid_off[h], e = a.kid_off[h + 1];
        const Three s = chance_sum<ADDR>(a, b + tid, e, BLOCK, a.bigc_kids[j]);
        double *red = L.diff;   // 3 * BLOCK
        red[tid] = s.x0; red[BLOCK + tid] = s.x1; red[2 * BLOCK + tid] = s.x2;
        __syncthreads();
        for (int w = BLOCK / 2; w > 0; w >>= 1) {
            if (tid < w)
                for (int k = 0; k < 3; k++) red[k * BLOCK + tid] += red[k * BLOCK + tid + w];
            __syncthreads();
        }
        if (tid == 0) { a.v0[h] = red[0]; a.v1[h] = red[BLOCK]; a.v2[h] = red[2 * BLOCK]; }
        return;
    }
    const int32_t g = gbeg + xcd_tile(blk, ngroups);
    const int32_t i0 = a.grp_iset_off[g], nsets = a.grp_iset_off[g + 1] - i0;
    const int32_t mbeg = a.mem_off[i0], mend = a.mem_off[i0 + nsets];
    int32_t nact = 0;
    bool mix = false;
    if (tid == 0) L.mixed = 0;
    if (tid < nsets) {
        const int32_t m0 = a.mem_off[i0 + tid], m1 = a.mem_off[i0 + tid + 1];
        L.moff[tid] = m0;
        L.slot[tid] = a.slot_off[i0 + tid];
        nact = a.slot_off[i0 + tid + 1] - L.slot[tid];
        for (int32_t k = 0; k < nact; k++) mix |= a.slot_kids[L.slot[tid] + k] == KIDS_MIXED;
        L.pl[tid] = a.iset_player[i0 + tid];
        if (tid == nsets - 1) {
            L.moff[nsets] = m1;
            L.slot[nsets] = a.slot_off[i0 + nsets];
        }
        // a group of several sets holds at most GROUP_MEMBERS_MAX members; a larger one is a single set
        const int32_t e = min(m1, mbeg + GROUP_MEMBERS_MAX);
        for (int32_t m = m0; m < e; m++) L.mset[m - mbeg] = (uint8_t)tid;
    }
    // the group's widest set, and whether some slot of it has children of both kinds
    int32_t wide = nact;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) wide = max(wide, __shfl_xor(wide, off));
    if ((tid & 63) == 0) L.wide[tid >> 6] = wide;
    __syncthreads();
    if (mix) L.mixed = 1;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < BLOCK / 64; w++) wide = max(wide, L.wide[w]);
    const bool mixed = L.mixed != 0;
    int4 hf = make_int4(0, 0, 0, 0), hb = hf;
    if constexpr (ADDR == ADDR_OFFSET) {
        hf = a.ghdr[2 * g];
        hb = a.ghdr[2 * g + 1];
    }
    const bool perm = (hf.w & GRP_PERM) != 0, wide_rec = (hf.w & GRP_WIDE) != 0;
    // the member listed at m: its node, the opponent's last sequence and its first edge; its set-major
    // position in the group
    auto member = [&](int32_t m) -> int3 {
        if constexpr (ADDR == ADDR_OFFSET) {
            if (wide_rec) {
                const int2 x = a.mwide[hb.z + (m - mbeg)];
                return make_int3(x.x, x.y, 0);
            }
            const uint32_t x = a.mrec[m];
            return make_int3(hb.x + (int32_t)(x & ((1u << hb.w) - 1)), hb.y + (int32_t)(x >> hb.w), 0);
        } else {
            const int2 x = a.mem[m];
            return make_int3(x.x & MEMBER_NODE_MASK, a.mem_seq[m], x.y);
        }
    };
    auto place = [&](int32_t m) { return perm ? (int32_t)a.mpos[m] : m - mbeg; };
    auto set_at = [&](int32_t pos) { return pos < GROUP_MEMBERS_MAX ? (int32_t)L.mset[pos] : 0; };
    auto child = [&](const int3 &x, int32_t q, int32_t k) -> int32_t {
        if constexpr (ADDR == ADDR_OFFSET) return x.x + a.koff[q];
        else if constexpr (ADDR == ADDR_LIST) return a.kid[x.z + k];
        else return x.z + k;
    };
    double Q[MAXA];
#pragma unroll
    for (int k = 0; k < MAXA; k++) Q[k] = 0.0;
    // values and staging of the members [cb, ce): at most NA actions per set
    auto members = [&](int32_t cb, int32_t ce, auto nac, auto mixc) {
        constexpr int NA = decltype(nac)::value;
        constexpr bool MIXED = decltype(mixc)::value;
        auto leaf_at = [&](uint8_t kinds, int32_t c) {
            if constexpr (MIXED) return is_leaf(kinds, c, a.kid_off);
            else return kinds == KIDS_TERMINAL;
        };
        if constexpr (NA <= 4) {
            // two members at a time, every load of a stage issued before the next: lanes past the end
            // repeat the chunk's first member, actions past a set's last repeat it
            constexpr int P = MPT >= 2 ? 2 : 1;
#pragma unroll
            for (int u0 = 0; u0 < MPT; u0 += P) {
                bool in[P], one[P];
                int32_t pos[P], s0[P], nA[P];
                int3 x[P];
#pragma unroll
                for (int u = 0; u < P; u++) {
                    const int32_t j = (u0 + u) * BLOCK + tid;
                    in[u] = cb + j < ce;
                    const int32_t m = in[u] ? cb + j : cb;
                    pos[u] = place(m);
                    x[u] = member(m);
                }
                double q[P], sg[P][NA];
                int32_t c[P][NA];
                uint8_t kinds[P][NA];
#pragma unroll
                for (int u = 0; u < P; u++) {
                    const int32_t st = set_at(pos[u]);
                    s0[u] = L.slot[st];
                    nA[u] = L.slot[st + 1] - s0[u];
                    one[u] = L.pl[st] == 1;
                    q[u] = a.seqbar[x[u].y];
#pragma unroll
                    for (int k = 0; k < NA; k++) {
                        const int32_t kk = min(k, nA[u] - 1);
                        c[u][k] = child(x[u], s0[u] + kk, kk);
                        kinds[u][k] = a.slot_kids[s0[u] + kk];
                        sg[u][k] = a.sigbar[s0[u] + kk];
                    }
                }
                Three t[P][NA];
#pragma unroll
                for (int u = 0; u < P; u++)
#pragma unroll
                    for (int k = 0; k < NA; k++) t[u][k] = three(a, c[u][k], leaf_at(kinds[u][k], c[u][k]));
#pragma unroll
                for (int u = 0; u < P; u++) {
                    double va = 0.0, vo = 0.0;
                    const double w = one[u] ? q[u] : -q[u];
#pragma unroll
                    for (int k = 0; k < NA; k++) {
                        va = k < nA[u] ? fma(sg[u][k], t[u][k].x0, va) : va;
                        vo = k < nA[u] ? fma(sg[u][k], one[u] ? t[u][k].x2 : t[u][k].x1, vo) : vo;
                    }
                    if (!in[u]) continue;
#pragma unroll
                    for (int k = 0; k < NA; k++)
                        L.diff[(pos[u] - (cb - mbeg)) * MAXA + k] = w * (one[u] ? t[u][k].x1 : t[u][k].x2);
                    a.v0[x[u].x] = va;
                    (one[u] ? a.v2 : a.v1)[x[u].x] = vo;
                }
            }
        } else {
            for (int32_t m = cb + tid; m < ce; m += BLOCK) {
                const int32_t pos = place(m), st = set_at(pos), s0 = L.slot[st], nA = L.slot[st + 1] - s0;
                const bool one = L.pl[st] == 1;
                const int3 x = member(m);
                const double q = a.seqbar[x.y], w = one ? q : -q;
                double va = 0.0, vo = 0.0;
#pragma unroll 4
                for (int k = 0; k < nA; k++) {
                    const int32_t c = child(x, s0 + k, k);
                    const Three t = three(a, c, leaf_at(a.slot_kids[s0 + k], c));
                    const double sg = a.sigbar[s0 + k];
                    va = fma(sg, t.x0, va);
                    vo = fma(sg, one ? t.x2 : t.x1, vo);
                    L.diff[(pos - (cb - mbeg)) * MAXA + k] = w * (one ? t.x1 : t.x2);
                }
                a.v0[x.x] = va;
                (one ? a.v2 : a.v1)[x.x] = vo;
            }
        }
    };
    for (int32_t cb = mbeg; cb < mend; cb += CHUNK) {
        const int32_t ce = min(cb + CHUNK, mend);
        with_action_bound<MAXA>(wide, [&](auto nac) {
            if (mixed) members(cb, ce, nac, std::true_type{});
            else members(cb, ce, nac, std::false_type{});
        });
        __syncthreads();
        if (tid < nsets) {
            const int32_t k0 = max(L.moff[tid], cb) - cb, k1 = min(L.moff[tid + 1], ce) - cb;
            // several members' columns are read ahead of their additions; past a set's actions they hold
            // other columns' leftovers, which are never compared
            constexpr int U = MAXA <= 4 ? 4 : 1;
            int32_t m = k0;
            for (; m + U <= k1; m += U) {
                double d[U][MAXA];
#pragma unroll
                for (int i = 0; i < U; i++)
#pragma unroll
                    for (int k = 0; k < MAXA; k++) d[i][k] = L.diff[(m + i) * MAXA + k];
#pragma unroll
                for (int i = 0; i < U; i++)
#pragma unroll
                    for (int k = 0; k < MAXA; k++) Q[k] += d[i][k];
            }
            for (; m < k1; m++) {
#pragma unroll
                for (int k = 0; k < MAXA; k++) Q[k] += L.diff[m * MAXA + k];
            }
        }
        __syncthreads();
    }
    if (tid < nsets) {
        const int32_t nA = L.slot[tid + 1] - L.slot[tid];
        int best = 0;
        double bq = Q[0];
#pragma unroll
        for (int k = 1; k < MAXA; k++)
            if (k < nA && Q[k] > bq) { bq = Q[k]; best = k; }
        L.best[tid] = (uint8_t)best;
    }
    __syncthreads();
    for (int32_t m = mbeg + tid; m < mend; m += BLOCK) {
        const int32_t st = set_at(place(m)), k = L.best[st], s = L.slot[st] + k;
        const int3 x = member(m);
        const int32_t c = child(x, s, k);
        const bool one = L.pl[st] == 1;
        double *own = one ? a.v1 : a.v2;
        own[x.x] = (is_leaf(a.slot_kids[s], c, a.kid_off) ? a.v0 : own)[c];
    }
}

// out[k * n + s] <- value k of game s's root (the first n nodes)
__global__ void __launch_bounds__(BLOCK) k_eval_roots(int32_t n, const int32_t *__restrict__ kid_off, EvalArgs a,
                                                      double *__restrict__ out) {
    const int32_t s = (int32_t)(blockIdx.x * BLOCK + threadIdx.x);
    if (s >= n) return;
    const Three t = three(a, s, kid_off[s] == kid_off[s + 1]);
    out[s] = t.x0; out[n + s] = t.x1; out[2 * n + s] = t.x2;
}

EvalArgs eval_args(const DevGame &g) {
    EvalArgs a;
    a.grp_iset_off = g.grp_iset_off; a.slot_off = g.slot_off; a.mem_off = g.mem_off; a.mem_seq = g.mem_seq;
    a.kid_off = g.kid_off; a.kid = g.kid; a.koff = g.koff; a.ghdr = g.ghdr; a.mwide = g.mwide; a.mrec = g.mrec;
    a.mpos = g.mpos; a.mem = g.mem; a.iset_player = g.iset_player;
    a.slot_kids = g.slot_kids; a.chance_node = g.chance_node; a.bigc_node = g.bigc_node;
    a.chance_kids = g.chance_kids; a.bigc_kids = g.bigc_kids; a.sigbar = g.sigbar; a.seqbar = g.seqbar;
    a.v0 = g.val[0]; a.v1 = g.val[1]; a.v2 = g.val[2];
    return a;
}

template <int MAXA, int MPT>
hipError_t eval_level(const DevGame &g, int d, hipStream_t s) {
    const int32_t gb = g.grp_depth_off[d], ng = g.grp_depth_off[d + 1] - gb;
    const int32_t cb = g.chance_off[d], nc = g.chance_off[d + 1] - cb;
    const int32_t bb = g.bigc_off[d], nb = g.bigc_off[d + 1] - bb;
    const unsigned blocks = (unsigned)ng + (unsigned)nb + grid_for((int64_t)nc * CHANCE_LANES);
    if (blocks == 0) return hipSuccess;
    const EvalArgs a = eval_args(g);
    if (g.affine) k_eval_level<MAXA, MPT, ADDR_OFFSET><<<blocks, BLOCK, 0, s>>>(gb, ng, bb, nb, cb, nc, a);
    else if (g.explicit_kids) k_eval_level<MAXA, MPT, ADDR_LIST><<<blocks, BLOCK, 0, s>>>(gb, ng, bb, nb, cb, nc, a);
    else k_eval_level<MAXA, MPT, ADDR_IMPLICIT><<<blocks, BLOCK, 0, s>>>(gb, ng, bb, nb, cb, nc, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_average(const DevGame &g, hipStream_t s) {
    if (g.I == 0) return hipSuccess;
    k_normalise<double><<<grid_for(g.I), BLOCK, 0, s>>>(g.I, g.slot_off, nullptr, g.sbar, g.sigbar);
    return hipGetLastError();
}

hipError_t launch_strategy(const DevGame &g, const int32_t *canon_off, bool average, float *dst, hipStream_t s) {
    if (g.I == 0) return hipSuccess;
    const unsigned slots = (unsigned)(((int64_t)g.A + 4 * BLOCK - 1) / (4 * BLOCK));
    if (average) k_normalise<float><<<grid_for(g.I), BLOCK, 0, s>>>(g.I, canon_off, g.slot_map, g.sbar, dst);
    else if (g.fp64) k_gather<double><<<slots, BLOCK, 0, s>>>(g.A, g.slot_map, (const double *)g.sigma, dst);
    else k_gather<float><<<slots, BLOCK, 0, s>>>(g.A, g.slot_map, (const float *)g.sigma, dst);
    return hipGetLastError();
}

// members per thread: the group capacity over the block (group_members), so that a chunk holds a group
hipError_t launch_eval_level(const DevGame &g, int d, hipStream_t s) {
    if (g.max_actions <= 4) return g.fp64 ? eval_level<4, 2>(g, d, s) : eval_level<4, 4>(g, d, s);
    if (g.max_actions <= 16) return eval_level<16, 1>(g, d, s);
    return eval_level<64, 1>(g, d, s);
}

hipError_t launch_eval_roots(const DevGame &g, int32_t n, double *out, hipStream_t s) {
    k_eval_roots<<<grid_for(n), BLOCK, 0, s>>>(n, g.kid_off, eval_args(g), out);
    return hipGetLastError();
}

}  // namespace cfrx
