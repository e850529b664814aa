// phase_small.hip -- whole 6D subtree of a small node inside one workgroup.
//
// Nodes of at most 64 members belong to one wavefront (wave_subtree): a
// member per lane, nodes as 64-bit lane masks, no LDS and no barriers.
//
// A larger node (at most MAXN members) is split by a workgroup, whose
// members stay in global memory (they are its own and L2-resident) while LDS
// holds what the pair searches read.  Per node:
//   1. exact integer moments (wave reductions + LDS atomics) -> a, c
//   2. normalised coordinates X = sqrt(a) (x - centre), sqrt(c) (v - mean)
//      and their squared norms, as rows of an LDS table
//   3. nearest neighbours: |Xi|^2 + |Xj|^2 - 2 Xi.Xj of 64 x 16 pairs at a
//      time by fp32 matrix instructions (two 16x16x4 products a tile).  The
//      norms are scaled so that the value never exceeds the pair's d^2 as the
//      method defines it (see LB_EPS): the lane keeps the smallest value, its
//      member and the second smallest; the pair's own d^2 is then evaluated
//      exactly and accepted when it does not exceed the second smallest
//      bound.  The few other members are searched exactly; where they are
//      many, or the node percolates, every pair is evaluated, here and in 5.
//   4. l^2 = k-th smallest d^2 by a 4-pass 8-bit radix select in LDS
//   5. links: the same products over the members with d_i^2 <= l^2 (others
//      cannot link), tiles above the diagonal; pairs whose bound admits them
//      are queued per wavefront and evaluated exactly 64 at a time, then
//      united in a lock-free union-find in LDS
//   6. components -> children (>= min_sub, not the whole node): node records
//      get global slots, members are regrouped so each child is a contiguous
//      range, children are pushed, those of at most 64 members on a list that
//      the wavefronts share out at the end
// Every result is decided by the exact fp32 evaluation; the products only
// choose the pairs that need one.
//
// What bounds it: the matrix products of step 3 (64 cycles per 256 pairs and
// SIMD, beside 48 vector instructions of bookkeeping), where evaluating
// every pair exactly took some 25 dependent vector instructions per 64
// pairs.  512^3 workload, kernel time of a step: 2048-member bucket 291 ->
// 20 ms, 1024 338 -> 10 ms, 256 59 -> 4 ms; one 2048-member subtree alone on
// its CU 2.4 -> 0.7 ms.
#include <type_traits>

#include "phase_common.h"

namespace rs {

// LDS scalars
enum { SH_SP, SH_NSMALL, SH_NEXT, SH_NC, SH_NCH, SH_BASE, SH_OK, SH_TOT, SH_BUCKET, SH_KK,
       SH_NOWRAP, SH_NQ, SH_N };

// a pushed node: members perm[s0, s0 + size), ref = member of smallest index,
// depth below the workgroup's item (whose own level has no such bound; every
// split loses a member, so a depth stays below the item's size)
struct StackEntry {
    int32_t slot;
    uint16_t s0, size, ref, depth;
};

constexpr int WAVE_MAX = 64;      // nodes one wavefront splits by itself
constexpr int QCAP = 128;         // queued pairs per wavefront
constexpr int N_ROWS = 7;         // X of x y z u v w, squared norm
// The screening decides next to nothing where nearest distances are tied
// (lattices, coinciding members) or tiny beside the node (two compact clumps
// far apart).  With more than half of the members undecided, every pair is
// evaluated instead, as for a node that percolates: a listed member costs a
// wavefront a pass over the node, all pairs together less than a listed half.
// 195 nodes of 2048 members, listed one by one and this way: lattices 3.4 and
// 2.1 ms, two clumps 4.1 and 2.0, points of a uniform box 6.3 and 2.7; sets with
// a third of duplicates 1.9, with the limit at an eighth 2.4.
constexpr int EXACT_PART = 2;

constexpr int n_stride(int maxn) { return maxn + 16; }   // rows on different banks

// Per member 36 bytes: the seven rows (whose space holds the component
// counts and minima and the child table in step 6), d^2 or union-find parent,
// two 16-bit member lists.  At the default min_sub two 2048-member
// workgroups of eight wavefronts and four 1024-member ones fit per CU.
static size_t small_lds_bytes(int maxn, int nt, int min_sub) {
    const int capn = maxn / min_sub + 1;
    return (size_t)N_ROWS * n_stride(maxn) * 4 + (size_t)maxn * 8 +
           (size_t)capn * sizeof(StackEntry) + (size_t)(nt / 64) * QCAP * 4;
}

template <int CTRL, int ROWS>
RS_DEV uint64_t dpp_add_u64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf,
                                                              false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL,
                                                              ROWS, 0xf, false);
    return v + (((uint64_t)hi << 32) | lo);
}

// sum over the 64 lanes, uniform (as wave_min_u32, with identity 0)
RS_DEV uint64_t wave_sum_u64(uint64_t v) {
    v = dpp_add_u64<0xB1, 0xf>(v);
    v = dpp_add_u64<0x4E, 0xf>(v);
    v = dpp_add_u64<0x124, 0xf>(v);
    v = dpp_add_u64<0x128, 0xf>(v);
    v = dpp_add_u64<0x142, 0xa>(v);
    v = dpp_add_u64<0x143, 0xc>(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// sum of a 128-bit quantity below 2^90 over the 64 lanes
RS_DEV u128 wave_sum_u128(u128 v) {
    return ((u128)wave_sum_u64((uint64_t)(v >> 32)) << 32) +
           wave_sum_u64((uint64_t)v & 0xffffffffu);
}

RS_DEV int64_t lane_i64(int64_t v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// one member's phase-space coordinates and particle index
struct Member {
    float x, y, z, u, v, w;
};

RS_DEV Member load_member(const Members& mb, int64_t g) {
    return Member{mb.x[g], mb.y[g], mb.z[g], mb.vx[g], mb.vy[g], mb.vz[g]};
}

RS_DEV float member_d2(const Member& p, const Member& q, bool nowrap, float fa, float fc,
                       const PhaseParams& pp) {
    return nowrap ? phase_d2<false>(p.x, p.y, p.z, p.u, p.v, p.w, q.x, q.y, q.z, q.u, q.v, q.w,
                                    fa, fc, pp.L, pp.h)
                  : phase_d2<true>(p.x, p.y, p.z, p.u, p.v, p.w, q.x, q.y, q.z, q.u, q.v, q.w,
                                   fa, fc, pp.L, pp.h);
}

// d^2 of every lane's member to those of the lanes in `mask`, one at a time
template <bool WRAP, class F>
RS_DEV void wave_pairs(uint64_t mask, const Member& p, float fa, float fc, const PhaseParams& pp,
                       F&& use) {
    while (mask) {
        const int j = __builtin_ctzll(mask);
        mask &= mask - 1;
        use(j, phase_d2<WRAP>(p.x, p.y, p.z, p.u, p.v, p.w, lane_f(p.x, j), lane_f(p.y, j),
                              lane_f(p.z, j), lane_f(p.u, j), lane_f(p.v, j), lane_f(p.w, j), fa,
                              fc, pp.L, pp.h));
    }
}

// The subtree of a node of at most 64 members, one per lane (those of
// `root`), by one wavefront with all lanes active.  Pending nodes are lane
// masks, entry t held by lane t; every node's children are disjoint, so 32
// entries are the most there can be.
template <bool FEAT>
RS_DEV void wave_subtree(uint64_t root, const Member& p, int32_t idx, int32_t slot0,
                         int32_t level0, const PhaseParams& pp, const NodeRec& nr,
                         int32_t* __restrict__ deepest) {
    const int lane = threadIdx.x & 63;
    uint64_t st_mask = lane == 0 ? root : 0;
    int32_t st_slot = slot0, st_level = level0;
    int sp = 1;
    while (sp > 0) {
        sp--;
        const uint64_t mask = (uint64_t)lane_i64((int64_t)st_mask, sp);
        const int slot = __builtin_amdgcn_readlane(st_slot, sp);
        const int level = __builtin_amdgcn_readlane(st_level, sp);
        const int sz = __builtin_popcountll(mask);
        const bool in = (mask >> lane) & 1;
        // exact moments about the member of smallest index
        const uint32_t mi = wave_min_u32(in ? (uint32_t)idx : 0xffffffffu);
        const int rl = __builtin_ctzll(__ballot(in && (uint32_t)idx == mi));
        unsigned long long acc[18];
        const float ps[3] = {p.x, p.y, p.z}, vs[3] = {p.u, p.v, p.w};
        bool nowrap = true;
#pragma unroll
        for (int ax = 0; ax < 3; ax++) {
            const int64_t q = quant_pos(ps[ax]);
            int64_t d = q - lane_i64(q, rl);
            if (2 * d > pp.LQ) d -= pp.LQ;
            else if (2 * d <= -pp.LQ) d += pp.LQ;
            const int64_t w = quant_vel(vs[ax]);
            const uint64_t d2 = in ? (uint64_t)(d * d) : 0, w2 = in ? (uint64_t)(w * w) : 0;
            acc[ax] = wave_sum_u64(in ? (uint64_t)d : 0);
            acc[3 + ax] = wave_sum_u64(in ? (uint64_t)w : 0);
            const u128 sd = wave_sum_u128(d2), sw = wave_sum_u128(w2);
            acc[6 + 2 * ax] = (uint64_t)sd;
            acc[7 + 2 * ax] = (uint64_t)(sd >> 64);
            acc[12 + 2 * ax] = (uint64_t)sw;
            acc[13 + 2 * ax] = (uint64_t)(sw >> 64);
            const uint32_t b = __float_as_uint(ps[ax]);
            const uint32_t lo = wave_min_u32(in ? b : 0xffffffffu);
            const uint32_t hi = ~wave_min_u32(in ? ~b : 0xffffffffu);
            nowrap = nowrap && (__uint_as_float(hi) - __uint_as_float(lo) <= pp.h);
        }
        const Norm nm = mom_finalize(acc, sz);
        const float fa = nm.a, fc = nm.c;
        if constexpr (FEAT) {
            const FeatFrame fr = feat_frame(acc, sz, lane_f(p.x, rl), lane_f(p.y, rl),
                                            lane_f(p.z, rl), nm.sx2, nm.sv2);
            int br, bv;
            feat_member_bins(fr, p.x, p.y, p.z, p.u, p.v, p.w, pp.L, pp.h, &br, &bv);
            int32_t hist[16];
#pragma unroll
            for (int b = 0; b < 8; b++) {
                hist[b] = __builtin_popcountll(__ballot(in && br == b));
                hist[8 + b] = __builtin_popcountll(__ballot(in && bv == 8 + b));
            }
            if (lane == 0) feat_write(nr.feat + (int64_t)slot * RS_NFEAT, acc, sz, level, hist);
        }
        // nearest neighbours
        float best = __builtin_huge_valf();
        auto nearest = [&](int j, float d) { best = lane != j && d < best ? d : best; };
        if (nowrap) wave_pairs<false>(mask, p, fa, fc, pp, nearest);
        else wave_pairs<true>(mask, p, fa, fc, pp, nearest);
        // k-th smallest, bit by bit (non-negative floats order like their bits)
        const uint32_t bits = __float_as_uint(best);
        uint64_t cand = mask;
        int kk = (int)select_rank(sz, pp.f_ppm);
        for (int b = 30; b >= 0; b--) {
            const uint64_t zero = cand & __ballot(((bits >> b) & 1u) == 0);
            const int c = __builtin_popcountll(zero);
            if (kk <= c) cand = zero;
            else {
                kk -= c;
                cand &= ~zero;
            }
        }
        const float l2 = lane_f(best, __builtin_ctzll(cand));
        if (lane == 0) {
            nr.a[slot] = fa;
            nr.c[slot] = fc;
            nr.sx2[slot] = nm.sx2;
            nr.sv2[slot] = nm.sv2;
            nr.l2[slot] = l2;
        }
        // links among the members with d_i^2 <= l^2, as one mask per lane
        const uint64_t act = __ballot(in && best <= l2);
        uint64_t adj = 0;
        auto link = [&](int j, float d) { adj |= d <= l2 ? 1ull << j : 0ull; };
        if (nowrap) wave_pairs<false>(act, p, fa, fc, pp, link);
        else wave_pairs<true>(act, p, fa, fc, pp, link);
        if (!((act >> lane) & 1)) adj = 0;
        // components; lane sp + c takes child c
        int nch = 0, mychild = -1;
        int32_t ch_size = 0, ch_min = 0;
        uint64_t left = act;
        while (left) {
            uint64_t comp = left & (0 - left), grown = comp;
            do {
                comp = grown;
                grown = comp | __ballot((adj & comp) != 0);
            } while (grown != comp);
            left &= ~comp;
            const int cs = __builtin_popcountll(comp);
            if (cs < pp.min_sub || cs >= sz) continue;
            const bool mine = (comp >> lane) & 1;
            const uint32_t cm = wave_min_u32(mine ? (uint32_t)idx : 0xffffffffu);
            if (mine) mychild = nch;
            if (lane == sp + nch) {
                st_mask = comp;
                ch_size = cs;
                ch_min = (int32_t)cm;
            }
            nch++;
        }
        if (nch == 0) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(nr.count, nch);
        base = __builtin_amdgcn_readfirstlane(base);
        if (base + nch > nr.cap) {
            if (lane == 0) atomicOr(nr.overflow, 1);
            continue;
        }
        if (lane >= sp && lane < sp + nch) {
            const int cs = base + lane - sp;
            st_slot = cs;
            st_level = level + 1;
            nr.level[cs] = level + 1;
            nr.minidx[cs] = ch_min;
            nr.parent[cs] = slot;
            nr.size[cs] = ch_size;
        }
        if (mychild >= 0) deepest[idx] = base + mychild;
        sp += nch;
    }
}

// nodes of at most 64 members: one wavefront each
template <bool FEAT>
__global__ void __launch_bounds__(256)
k_wave_subtree(const SmallItem* __restrict__ items, int n_items, Members mb, NodeRec nr,
               PhaseParams pp, int32_t* __restrict__ deepest) {
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (w >= n_items) return;
    const SmallItem it = items[w];
    const int n = __builtin_amdgcn_readfirstlane(it.size);
    const int64_t g = it.off + (lane < n ? lane : 0);
    wave_subtree<FEAT>(n >= 64 ? ~0ull : (1ull << n) - 1, load_member(mb, g), mb.idx[g],
                       __builtin_amdgcn_readfirstlane(it.slot),
                       __builtin_amdgcn_readfirstlane(it.level), pp, nr, deepest);
}

// v, unknown to the compiler: what the exact evaluation derives from it is not
// kept in registers through the rest of the kernel (8 to 10 fewer spilled)
RS_DEV int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

template <int MAXN, int NT, bool FEAT>
__global__ void __launch_bounds__(NT, 4)
k_small_subtree(const SmallItem* __restrict__ items, int n_items, Members mb, NodeRec nr,
                PhaseParams pp, int32_t* __restrict__ deepest) {
    static_assert(MAXN % 64 == 0 && MAXN <= 2048, "row numbers take 9 bits of a key");
    constexpr int NS = n_stride(MAXN);
    extern __shared__ __align__(16) char smem[];
    float* N = reinterpret_cast<float*>(smem);                    // [N_ROWS][NS]
    float* d2 = N + N_ROWS * NS;                                  // [MAXN], later:
    int32_t* par = reinterpret_cast<int32_t*>(d2);                // union-find parents
    uint16_t* perm = reinterpret_cast<uint16_t*>(d2 + MAXN);
    uint16_t* tmp = perm + MAXN;
    const int capn = MAXN / pp.min_sub + 1;
    StackEntry* stk = reinterpret_cast<StackEntry*>(tmp + MAXN);  // [capn]
    uint32_t* queue = reinterpret_cast<uint32_t*>(stk + capn) + QCAP * (threadIdx.x >> 6);
    // step 6, over the rows: per member a packed (index, member) minimum and
    // a count, then the child table
    unsigned long long* mpk = reinterpret_cast<unsigned long long*>(smem);   // [MAXN]
    int32_t* cnt = reinterpret_cast<int32_t*>(mpk + MAXN);                   // [MAXN]
    int32_t* ch = cnt + MAXN;                                                // [capn][5]
    static_assert(N_ROWS * NS * 4 >= MAXN * 12 + (MAXN / 2 + 1) * 20, "child table room");
    __shared__ unsigned long long acc[18];
    __shared__ uint32_t ext[12];
    // the 256-bin histogram of the select lives in the member list `tmp` where
    // that is large enough: the two are never live together
    constexpr bool HIST_IN_TMP = MAXN >= 512;
    __shared__ int32_t hist_own[HIST_IN_TMP ? 16 : 256];
    int32_t* hist = HIST_IN_TMP ? reinterpret_cast<int32_t*>(tmp) : hist_own;
    __shared__ int32_t sh[SH_N];
    __shared__ float shf[10];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 15, lk = lane >> 4;   // tile column (or row), k offset
    // where every pair is evaluated, the rows' space holds the coordinates
    constexpr int R = (MAXN + NT - 1) / NT;     // members per thread
    float4* PA = reinterpret_cast<float4*>(smem);                 // [MAXN] x y z u
    float2* PB = reinterpret_cast<float2*>(PA + MAXN);            // [MAXN] v w
    auto exact_member = [&](int m) {
        const float4 a = PA[m];
        const float2 b = PB[m];
        return Member{a.x, a.y, a.z, a.w, b.x, b.y};
    };

    for (int w = blockIdx.x; w < n_items; w += gridDim.x) {
        const SmallItem it = items[w];
        const int n = it.size;
        if (tid == 0) {
            stk[0] = StackEntry{it.slot, 0, (uint16_t)n, 0, 0};
            sh[SH_SP] = 1;
            sh[SH_NSMALL] = 0;
        }
        __syncthreads();
        for (int m = tid; m < n; m += NT) {
            perm[m] = (uint16_t)m;
            if (mb.idx[it.off + m] == it.refidx) stk[0].ref = (uint16_t)m;   // exactly one
        }
        __syncthreads();

        // Nodes of more than 64 members, last pushed first: the stack grows
        // from the front, the list of smaller nodes from the back.
        for (;;) {
            const int sp = sh[SH_SP];
            if (sp == 0) break;
            const StackEntry e = stk[sp - 1];
            const int s0 = e.s0, sz = e.size, slot = e.slot, level = it.level + e.depth;
            __syncthreads();                 // every thread has read the stack
            if (tid == 0) {
                sh[SH_SP] = sp - 1;
                sh[SH_NC] = 0;
                sh[SH_NCH] = 0;
                sh[SH_NEXT] = 0;
                sh[SH_NQ] = 0;
            }
            if (tid < 18) acc[tid] = 0;
            if (tid < 12) ext[tid] = tid < 6 ? 0xffffffffu : 0u;
            __syncthreads();
            const Member ref = load_member(mb, it.off + e.ref);

            // ---- 1. moments and extents ----
            {
                const int64_t qref[3] = {quant_pos(ref.x), quant_pos(ref.y), quant_pos(ref.z)};
                Moments mo;
                mom_zero(mo);
                uint32_t mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[3] = {0u, 0u, 0u};
                for (int m = tid; m < sz; m += NT) {
                    const Member p = load_member(mb, it.off + perm[s0 + m]);
                    mom_add(mo, p.x, p.y, p.z, p.u, p.v, p.w, qref, pp.LQ);
                    const uint32_t b[3] = {__float_as_uint(p.x), __float_as_uint(p.y),
                                           __float_as_uint(p.z)};
#pragma unroll
                    for (int ax = 0; ax < 3; ax++) {
                        mn[ax] = b[ax] < mn[ax] ? b[ax] : mn[ax];
                        mx[ax] = b[ax] > mx[ax] ? b[ax] : mx[ax];
                    }
                }
                if (wave * 64 < sz) {
#pragma unroll
                    for (int q = 0; q < 6; q++) {
                        mo.s1[q] = wave_sum_u64(mo.s1[q]);
                        mo.s2[q] = wave_sum_u128(mo.s2[q]);
                    }
#pragma unroll
                    for (int ax = 0; ax < 3; ax++) {
                        mn[ax] = wave_min_u32(mn[ax]);
                        mx[ax] = ~wave_min_u32(~mx[ax]);
                    }
                    if (lane == 0) {
                        mom_accumulate(acc, mo);
#pragma unroll
                        for (int ax = 0; ax < 3; ax++) {
                            atomicMin(ext + ax, mn[ax]);
                            atomicMax(ext + 6 + ax, mx[ax]);
                        }
                    }
                }
            }
            __syncthreads();
            if (tid == 0) {
                const Norm nm = mom_finalize(acc, sz);
                const float r[3] = {ref.x, ref.y, ref.z};
                shf[0] = nm.a;
                shf[1] = nm.c;
                shf[2] = nm.sx2;
                shf[3] = nm.sv2;
                bool nowrap = true;
#pragma unroll
                for (int ax = 0; ax < 3; ax++) {
                    const float d = __uint_as_float(ext[6 + ax]) - __uint_as_float(ext[ax]);
                    nowrap = nowrap && (d <= pp.h);
                    double c = (double)r[ax] + nm.mean[ax];   // centre, moved into the box
                    if (c < 0.0) c += (double)pp.L;
                    else if (c >= (double)pp.L) c -= (double)pp.L;
                    shf[4 + ax] = (float)c;
                    shf[7 + ax] = (float)nm.mean[3 + ax];
                }
                sh[SH_NOWRAP] = nowrap ? 1 : 0;
                nr.a[slot] = nm.a;
                nr.c[slot] = nm.c;
                nr.sx2[slot] = nm.sx2;
                nr.sv2[slot] = nm.sv2;
            }
            __syncthreads();
            const float fa = shf[0], fc = shf[1];
            const bool nowrap = sh[SH_NOWRAP] != 0;

            // ---- proposer features (only when requested) ----
            if (FEAT) {
                if (tid < 16) hist[tid] = 0;
                __syncthreads();
                const FeatFrame fr = feat_frame(acc, sz, ref.x, ref.y, ref.z, shf[2], shf[3]);
                for (int m = tid; m < sz; m += NT) {
                    const Member p = load_member(mb, it.off + perm[s0 + m]);
                    int br, bv;
                    feat_member_bins(fr, p.x, p.y, p.z, p.u, p.v, p.w, pp.L, pp.h, &br, &bv);
                    atomicAdd(hist + br, 1);
                    atomicAdd(hist + bv, 1);
                }
                __syncthreads();
                if (tid == 0) feat_write(nr.feat + (int64_t)slot * RS_NFEAT, acc, sz, level, hist);
                __syncthreads();
            }

            // ---- 2. normalised rows, padded to whole groups of 64 ----
            const int ng = (sz + 63) >> 6;
            {
                const float sa = sqrtf(fa), sc = sqrtf(fc);
                const float cx[3] = {shf[4], shf[5], shf[6]}, cv[3] = {shf[7], shf[8], shf[9]};
                float mn[3], mx[3];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) {
                    mn[ax] = __builtin_huge_valf();
                    mx[ax] = -__builtin_huge_valf();
                }
                for (int m = tid; m < 64 * ng; m += NT) {
                    float norm = NORM_PAD;
                    float X[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                    if (m < sz) {
                        const Member p = load_member(mb, it.off + perm[s0 + m]);
                        float d[3] = {p.x - cx[0], p.y - cx[1], p.z - cx[2]};
                        if (!nowrap) {
#pragma unroll
                            for (int ax = 0; ax < 3; ax++) {
                                d[ax] = min_image(d[ax], pp.L, pp.h);
                                mn[ax] = fminf(mn[ax], d[ax]);
                                mx[ax] = fmaxf(mx[ax], d[ax]);
                            }
                        }
                        X[0] = sa * d[0]; X[1] = sa * d[1]; X[2] = sa * d[2];
                        X[3] = sc * (p.u - cv[0]); X[4] = sc * (p.v - cv[1]);
                        X[5] = sc * (p.w - cv[2]);
                        norm = X[0] * X[0];
#pragma unroll
                        for (int k = 1; k < 6; k++) norm = fmaf(X[k], X[k], norm);
                        norm *= 1.0f - LB_EPS;
                    }
#pragma unroll
                    for (int k = 0; k < 6; k++) N[k * NS + m] = X[k];
                    N[6 * NS + m] = norm;
                }
                if (!nowrap) {
                    // extents in [-L, L], offset to order as unsigned bits
#pragma unroll
                    for (int ax = 0; ax < 3; ax++) {
                        if (mn[ax] <= mx[ax]) {
                            atomicMin(ext + 3 + ax, __float_as_uint(fmaxf(mn[ax] + pp.L, 0.0f)));
                            atomicMax(ext + 9 + ax, __float_as_uint(fmaxf(mx[ax] + pp.L, 0.0f)));
                        }
                    }
                }
            }
            __syncthreads();
            // Pair differences of X are those of the nearest images as long as
            // the node spans less than half the box; a wider one (it
            // percolates) has every pair evaluated.
            bool wide = false;
            const float tiny = lb_abs(fa, fc);
            float lb_k = 0.0f, lb_add = 0.0f;
            if (!nowrap) {
#pragma unroll
                for (int ax = 0; ax < 3; ax++)
                    wide = wide || __uint_as_float(ext[9 + ax]) - __uint_as_float(ext[3 + ax]) >=
                                       0.999f * pp.h;
                const float eta = sqrtf(fa) * box_slack(pp.L);
                lb_k = LB_WRAP;
                lb_add = (1.0f + 1.0f / LB_WRAP) * eta * eta * 1.001f;
            }

            // ---- 3. nearest-neighbour distances ----
            // A wavefront takes 64 members as columns (four tiles, in
            // registers) against all rows.  A key is the pair's bound with the
            // row's number within its lane group in the low nine bits.  Members
            // left undecided (ties, near ties) are listed in tmp; too many of
            // them end the screening.
            const int most = sz / EXACT_PART;
            if (!wide) {
                for (;;) {
                    int g = 0;
                    if (lane == 0)
                        g = __hip_atomic_load(sh + SH_NQ, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP) > most
                                ? ng : atomicAdd(sh + SH_NEXT, 1);
                    g = __builtin_amdgcn_readfirstlane(g);
                    if (g >= ng) break;
                    const int q = 64 * g + lane;
                    const Member pq = load_member(mb, it.off + perm[s0 + (q < sz ? q : 0)]);
                    float b0[4], b1[4];
                    int32_t k1[4], k2[4];
#pragma unroll
                    for (int cb = 0; cb < 4; cb++) {
                        const int c = 64 * g + 16 * cb + lm;
                        const float hi = N[(lk < 3 ? 4 + lk : 6) * NS + c];
                        b0[cb] = -2.0f * N[lk * NS + c];
                        b1[cb] = lk < 2 ? -2.0f * hi : lk == 2 ? 1.0f : hi;
                        if (lk == 3) b1[cb] = N[6 * NS + c];
                        k1[cb] = k2[cb] = 0x7fffffff;
                    }
                    const int nrb = 4 * ng;
                    const int32_t kmask = key_mask();
                    const float* n0 = N + lk * NS + lm;
                    const float* n1 = N + (lk < 3 ? 4 + lk : 6) * NS + lm;
                    float a0 = n0[0], a1 = n1[0];
                    for (int rb = 0; rb < nrb; rb++) {
                        if (lk == 3) a1 = 1.0f;
                        const int nx = 16 * min(rb + 1, nrb - 1);   // the next block's operands
                        const float p0 = n0[nx], p1 = n1[nx];
                        f32x4 o[4];
#pragma unroll
                        for (int cb = 0; cb < 4; cb++) {
                            const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                            o[cb] = mfma_16x16x4(a0, b0[cb], zero);
                        }
#pragma unroll
                        for (int cb = 0; cb < 4; cb++) o[cb] = mfma_16x16x4(a1, b1[cb], o[cb]);
                        if ((rb >> 2) == g) {   // a member is not its own neighbour
#pragma unroll
                            for (int cb = 0; cb < 4; cb++)
#pragma unroll
                                for (int r = 0; r < 4; r++)
                                    if ((rb & 3) == cb && 4 * lk + r == lm) o[cb][r] = NORM_PAD;
                        }
#pragma unroll
                        for (int cb = 0; cb < 4; cb++)
#pragma unroll
                            for (int r = 0; r < 4; r++)
                                key_take(k1[cb], k2[cb], key_of(o[cb][r], rb << 2 | r, kmask));
                        a0 = p0;
                        a1 = p1;
                    }
                    // the four lanes of a column agree on its two smallest keys
                    int row = 0;
                    float bound = 0.0f;
#pragma unroll
                    for (int cb = 0; cb < 4; cb++) {
                        int r1 = (key_row(k1[cb]) >> 2) * 16 + 4 * lk + (k1[cb] & 3);
#pragma unroll
                        for (int o = 16; o <= 32; o <<= 1) {
                            const int32_t f1 = __shfl_xor(k1[cb], o, 64);
                            const int32_t f2 = __shfl_xor(k2[cb], o, 64);
                            const int fr = __shfl_xor(r1, o, 64);
                            k2[cb] = min(max(k1[cb], f1), min(k2[cb], f2));
                            r1 = f1 < k1[cb] ? fr : r1;
                            k1[cb] = min(k1[cb], f1);
                        }
                        if (lk == cb) {   // this lane's own member
                            row = r1;
                            bound = key_value(k2[cb]);
                        }
                    }
                    row = row < sz ? row : 0;
                    const Member pr = load_member(mb, it.off + perm[s0 + row]);
                    const float d = member_d2(pq, pr, nowrap, fa, fc, pp);
                    const bool ok = q < sz && row != q &&
                                    d <= (bound - lb_add) * (1.0f - lb_k) - tiny;
                    if (ok) d2[q] = d;
                    const uint64_t open = __ballot(q < sz && !ok);
                    if (open) {
                        int at = 0;
                        if (lane == 0) at = atomicAdd(sh + SH_NQ, __builtin_popcountll(open));
                        at = __builtin_amdgcn_readfirstlane(at);
                        if (q < sz && !ok)
                            tmp[at + __builtin_popcountll(open & lanemask_lt())] = (uint16_t)q;
                    }
                }
                __syncthreads();
            }
            const int nq = sh[SH_NQ];
            const bool exact = wide || nq > most;
            if (!exact) {   // each listed member against all others
                for (int t = wave; t < nq; t += NT / 64) {
                    const int qm = tmp[t];
                    const Member pm = load_member(mb, it.off + perm[s0 + qm]);
                    float best = __builtin_huge_valf();
                    for (int m = lane; m < sz; m += 64) {
                        const Member pr = load_member(mb, it.off + perm[s0 + m]);
                        const float d = member_d2(pm, pr, nowrap, fa, fc, pp);
                        best = m != qm && d < best ? d : best;
                    }
                    const uint32_t mn = wave_min_u32(__float_as_uint(best));
                    if (lane == 0) d2[qm] = __uint_as_float(mn);
                }
            } else {
                // Every pair once, the coordinates over the rows, by the thread
                // that holds its earlier member (d^2 is symmetric bit for bit:
                // the differences only change sign).  The later member's minimum
                // is gathered over the wavefront; a wavefront skips a member
                // that none of its row precedes.
                const int et = opaque(tid);                            // this thread,
                const int ew = __builtin_amdgcn_readfirstlane(et & ~63);   // its wavefront's first
                for (int m = et; m < sz; m += NT) {
                    const Member p = load_member(mb, it.off + perm[s0 + m]);
                    PA[m] = make_float4(p.x, p.y, p.z, p.u);
                    PB[m] = make_float2(p.v, p.w);
                    d2[m] = __builtin_huge_valf();
                }
                __syncthreads();
                Member pi[R];
                float best[R];
#pragma unroll
                for (int r = 0; r < R; r++) {
                    pi[r] = exact_member(et + r * NT < sz ? et + r * NT : 0);
                    best[r] = __builtin_huge_valf();
                }
                auto scan = [&](auto wrap) {
                    constexpr bool WRAP = decltype(wrap)::value;
                    for (int j = ew + 1; j < sz; j++) {
                        const Member p = exact_member(j);
                        float rev = __builtin_huge_valf();
#pragma unroll
                        for (int r = 0; r < R; r++) {
                            if (j > r * NT + ew) {   // uniform over the wavefront
                                const float d = phase_d2<WRAP>(
                                    pi[r].x, pi[r].y, pi[r].z, pi[r].u, pi[r].v, pi[r].w, p.x, p.y,
                                    p.z, p.u, p.v, p.w, fa, fc, pp.L, pp.h);
                                const bool ok = et + r * NT < j;
                                best[r] = ok && d < best[r] ? d : best[r];
                                rev = ok ? fminf(rev, d) : rev;
                            }
                        }
                        const uint32_t mn = wave_min_u32(__float_as_uint(rev));
                        if (lane == 0) atomicMin(reinterpret_cast<uint32_t*>(d2) + j, mn);
                    }
                };
                if (nowrap) scan(std::false_type{});
                else scan(std::true_type{});
#pragma unroll
                for (int r = 0; r < R; r++)
                    if (et + r * NT < sz)
                        atomicMin(reinterpret_cast<uint32_t*>(d2) + et + r * NT,
                                  __float_as_uint(best[r]));
            }
            __syncthreads();

            // ---- 4. k-th smallest nearest-neighbour distance ----
            uint32_t prefix = 0, pmask = 0;
            {
                int kk = (int)select_rank(sz, pp.f_ppm);
                for (int pass = 0; pass < 4; pass++) {
                    const int shift = 24 - 8 * pass;
                    for (int b = tid; b < 256; b += NT) hist[b] = 0;
                    __syncthreads();
                    for (int m = tid; m < sz; m += NT) {
                        uint32_t u = __float_as_uint(d2[m]);
                        if ((u & pmask) == prefix) atomicAdd(hist + ((u >> shift) & 255u), 1);
                    }
                    __syncthreads();
                    if (wave == 0) {
                        int h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2],
                            h3 = hist[4 * lane + 3];
                        int tot = h0 + h1 + h2 + h3, inc = tot;
#pragma unroll
                        for (int o = 1; o < 64; o <<= 1) {
                            int t = __shfl_up(inc, o, 64);
                            if (lane >= o) inc += t;
                        }
                        int before = inc - tot;
                        if (before < kk && kk <= inc) {
                            int k2 = kk - before, b = 4 * lane;
                            if (k2 > h0) { k2 -= h0; b++;
                                if (k2 > h1) { k2 -= h1; b++;
                                    if (k2 > h2) { k2 -= h2; b++; } } }
                            sh[SH_BUCKET] = b;
                            sh[SH_KK] = k2;
                        }
                    }
                    __syncthreads();
                    prefix |= (uint32_t)sh[SH_BUCKET] << shift;
                    pmask |= 255u << shift;
                    kk = sh[SH_KK];
                }
            }
            const float l2 = __uint_as_float(prefix);
            __syncthreads();                 // the histogram (in tmp) is done with

            // ---- 5. links within l ----
            if (tid == 0) {
                nr.l2[slot] = l2;
                sh[SH_NEXT] = 0;
            }
            for (int m = tid; m < sz; m += NT)
                if (d2[m] <= l2) tmp[atomicAdd(sh + SH_NC, 1)] = (uint16_t)m;
            __syncthreads();
            for (int m = tid; m < sz; m += NT) par[m] = m;   // over d2
            __syncthreads();
            if (exact) {   // as the nearest neighbours: each pair of active members once
                const int nc = sh[SH_NC], et = opaque(tid);
                const int ew = __builtin_amdgcn_readfirstlane(et & ~63);
                Member pi[R];
                int si[R];
#pragma unroll
                for (int r = 0; r < R; r++) {
                    si[r] = et + r * NT < nc ? tmp[et + r * NT] : -1;
                    pi[r] = exact_member(max(si[r], 0));
                }
                for (int q = ew + 1; q < nc; q++) {
                    const int j = tmp[q];
                    const Member p = exact_member(j);
#pragma unroll
                    for (int r = 0; r < R; r++)
                        if (si[r] >= 0 && q > et + r * NT &&
                            member_d2(pi[r], p, nowrap, fa, fc, pp) <= l2)
                            lds_unite(par, si[r], j);
                }
            } else {
                const int nc = sh[SH_NC], ngl = (nc + 63) >> 6;
                const float thr =
                    (l2 * (1.0f + lb_k) + lb_add) * (nowrap ? 1.0f : 1.00001f) + tiny;
                int qn = 0;   // queued pairs (uniform)
                auto drain = [&](int count) {
                    __builtin_amdgcn_wave_barrier();
                    if (lane < count) {
                        const uint32_t pr = queue[lane];
                        const int i = tmp[pr & 0xffffu], j = tmp[pr >> 16];
                        const Member pi = load_member(mb, it.off + perm[s0 + i]);
                        const Member pj = load_member(mb, it.off + perm[s0 + j]);
                        if (member_d2(pi, pj, nowrap, fa, fc, pp) <= l2) lds_unite(par, i, j);
                    }
                    __builtin_amdgcn_wave_barrier();
                };
                for (;;) {
                    int t = 0;
                    if (lane == 0) t = atomicAdd(sh + SH_NEXT, 1);
                    t = __builtin_amdgcn_readfirstlane(t);
                    if (t >= ngl) break;
                    const int g = ngl - 1 - t;   // the longest columns first
                    float b0[4], b1[4];
#pragma unroll
                    for (int cb = 0; cb < 4; cb++) {
                        const int c = 64 * g + 16 * cb + lm;
                        const int mc = c < nc ? tmp[c] : 0;
                        const float hi = N[(lk < 3 ? 4 + lk : 6) * NS + mc];
                        b0[cb] = -2.0f * N[lk * NS + mc];
                        b1[cb] = lk < 2 ? -2.0f * hi : lk == 2 ? 1.0f : c < nc ? hi : NORM_PAD;
                    }
                    const int nrb = min(4 * g + 4, (nc + 15) >> 4);
                    for (int rb = 0; rb < nrb; rb++) {
                        const int ri = 16 * rb + lm;
                        const int mr = ri < nc ? tmp[ri] : 0;
                        const float a0 = N[lk * NS + mr];
                        float a1 = N[(lk < 3 ? 4 + lk : 6) * NS + mr];
                        if (lk == 3) a1 = 1.0f;
                        if (lk == 2 && ri >= nc) a1 = NORM_PAD;
                        f32x4 o[4];
#pragma unroll
                        for (int cb = 0; cb < 4; cb++) {
                            const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                            o[cb] = mfma_16x16x4(a0, b0[cb], zero);
                        }
#pragma unroll
                        for (int cb = 0; cb < 4; cb++) o[cb] = mfma_16x16x4(a1, b1[cb], o[cb]);
                        if ((rb >> 2) == g) {   // each pair once: row before column
#pragma unroll
                            for (int cb = 0; cb < 4; cb++)
#pragma unroll
                                for (int r = 0; r < 4; r++)
                                    if (16 * (rb & 3) + 4 * lk + r >= 16 * cb + lm)
                                        o[cb][r] = NORM_PAD;
                        }
#pragma unroll
                        for (int cb = 0; cb < 4; cb++)
#pragma unroll
                            for (int r = 0; r < 4; r++) {
                                const bool hit = o[cb][r] <= thr;
                                const uint64_t bal = __ballot(hit);
                                if (bal) {
                                    if (hit)
                                        queue[qn + __builtin_popcountll(bal & lanemask_lt())] =
                                            (uint32_t)(16 * rb + 4 * lk + r) |
                                            (uint32_t)(64 * g + 16 * cb + lm) << 16;
                                    qn += __builtin_popcountll(bal);
                                    if (qn >= 64) {
                                        drain(64);
                                        qn -= 64;
                                        uint32_t moved = 0;
                                        if (lane < qn) moved = queue[64 + lane];
                                        __builtin_amdgcn_wave_barrier();
                                        if (lane < qn) queue[lane] = moved;
                                    }
                                }
                            }
                    }
                }
                if (qn > 0) drain(qn);
            }
            __syncthreads();

            // ---- 6. components and children ----
            for (int m = tid; m < sz; m += NT) {
                par[m] = lds_root(par, m);
                cnt[m] = 0;
                mpk[m] = ~0ull;
            }
            __syncthreads();
            for (int m = tid; m < sz; m += NT) {
                const int r = par[m];
                atomicAdd(cnt + r, 1);
                atomicMin(mpk + r, ((unsigned long long)(uint32_t)mb.idx[it.off + perm[s0 + m]]
                                    << 16) | (unsigned)m);
            }
            __syncthreads();
            for (int m = tid; m < sz; m += NT) {
                const int cs = cnt[m];
                if (par[m] == m && cs >= pp.min_sub && cs < sz) {
                    int c = atomicAdd(sh + SH_NCH, 1);
                    ch[5 * c + 0] = m;
                    ch[5 * c + 1] = cs;
                    ch[5 * c + 2] = (int)(mpk[m] >> 16);
                    ch[5 * c + 3] = perm[s0 + (int)(mpk[m] & 0xffffull)];
                }
            }
            __syncthreads();
            const int nch = sh[SH_NCH];
            if (nch > 0) {
                if (tid == 0) {
                    int base = atomicAdd(nr.count, nch);
                    bool ok = base + nch <= nr.cap;
                    if (!ok) atomicOr(nr.overflow, 1);
                    sh[SH_OK] = ok ? 1 : 0;
                    sh[SH_BASE] = base;
                    int off = 0;
                    for (int c = 0; c < nch; c++) {
                        ch[5 * c + 4] = off;
                        off += ch[5 * c + 1];
                    }
                    sh[SH_TOT] = off;
                }
                __syncthreads();
                if (sh[SH_OK]) {
                    const int base = sh[SH_BASE];
                    for (int c = tid; c < nch; c += NT) {
                        const int cs = base + c, size = ch[5 * c + 1];
                        nr.level[cs] = level + 1;
                        nr.minidx[cs] = ch[5 * c + 2];
                        nr.parent[cs] = slot;
                        nr.size[cs] = size;
                        cnt[ch[5 * c + 0]] = -(c + 1);
                        const StackEntry ce = {cs, (uint16_t)(s0 + ch[5 * c + 4]), (uint16_t)size,
                                               (uint16_t)ch[5 * c + 3], (uint16_t)(e.depth + 1)};
                        if (size > WAVE_MAX) stk[atomicAdd(sh + SH_SP, 1)] = ce;
                        else stk[capn - 1 - atomicAdd(sh + SH_NSMALL, 1)] = ce;
                    }
                    __syncthreads();
                    for (int m = tid; m < sz; m += NT) {
                        const int cv = cnt[par[m]];
                        if (cv < 0) {
                            const int c = -cv - 1, s = perm[s0 + m];
                            const int pos = atomicAdd(ch + 5 * c + 4, 1);
                            tmp[pos] = (uint16_t)s;
                            deepest[mb.idx[it.off + s]] = base + c;
                        }
                    }
                    __syncthreads();
                    const int tot = sh[SH_TOT];
                    for (int m = tid; m < tot; m += NT) perm[s0 + m] = tmp[m];
                }
            }
            __syncthreads();
        }

        // ---- nodes of at most 64 members, one wavefront each ----
        __syncthreads();
        if (tid == 0) sh[SH_NEXT] = 0;
        __syncthreads();
        const int nsmall = sh[SH_NSMALL];
        for (;;) {
            int t = 0;
            if (lane == 0) t = atomicAdd(sh + SH_NEXT, 1);
            t = __builtin_amdgcn_readfirstlane(t);
            if (t >= nsmall) break;
            const StackEntry e = stk[capn - 1 - t];
            const int sz = __builtin_amdgcn_readfirstlane((int)e.size);
            const int64_t g = it.off + perm[e.s0 + (lane < sz ? lane : 0)];
            wave_subtree<FEAT>(sz >= 64 ? ~0ull : (1ull << sz) - 1, load_member(mb, g), mb.idx[g],
                               __builtin_amdgcn_readfirstlane(e.slot),
                               __builtin_amdgcn_readfirstlane(it.level + (int)e.depth), pp, nr,
                               deepest);
        }
        __syncthreads();
    }
}

template <int MAXN, int NT>
static int launch_small(const SmallItem* items, int n_items, const Members& mb,
                        const NodeRec& nr, const PhaseParams& pp, int32_t* deepest,
                        hipStream_t st, const char* timer) {
    if (n_items <= 0) return RS_OK;
    size_t lds = small_lds_bytes(MAXN, NT, pp.min_sub);
    auto kern = pp.want_feat ? k_small_subtree<MAXN, NT, true> : k_small_subtree<MAXN, NT, false>;
    RS_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    unsigned grid = (unsigned)(n_items < (1 << 20) ? n_items : (1 << 20));
    prof_begin(timer, st);
    kern<<<grid, NT, lds, st>>>(items, n_items, mb, nr, pp, deepest);
    RS_HIP(hipGetLastError());
    prof_end(timer, st, 0.0);
    return RS_OK;
}

static int launch_wave(const SmallItem* items, int n_items, const Members& mb, const NodeRec& nr,
                       const PhaseParams& pp, int32_t* deepest, hipStream_t st,
                       const char* timer) {
    if (n_items <= 0) return RS_OK;
    auto kern = pp.want_feat ? k_wave_subtree<true> : k_wave_subtree<false>;
    prof_begin(timer, st);
    kern<<<(unsigned)((n_items + 3) / 4), 256, 0, st>>>(items, n_items, mb, nr, pp, deepest);
    RS_HIP(hipGetLastError());
    prof_end(timer, st, 0.0);
    return RS_OK;
}

// bucket b: 0 -> <= 64 members, 1 -> <= 256, 2 -> <= 1024, 3 -> <= 2048
int small_bucket_of(int size) { return size <= 64 ? 0 : size <= 256 ? 1 : size <= 1024 ? 2 : 3; }

// Threads per workgroup of buckets 1..3, from the tuning table (each value is
// one of the compiled shapes; results do not depend on the choice).
int run_small_bucket(int b, const SmallItem* items, int n_items, const Members& mb,
                     const NodeRec& nr, const PhaseParams& pp, int32_t* deepest,
                     hipStream_t st, const char* timer) {
    switch (b) {
        case 0: return launch_wave(items, n_items, mb, nr, pp, deepest, st, timer);
        case 1:
            if (tune_get(TUNE_SMALL_NT_256) == 128)
                return launch_small<256, 128>(items, n_items, mb, nr, pp, deepest, st, timer);
            return launch_small<256, 256>(items, n_items, mb, nr, pp, deepest, st, timer);
        case 2:
            if (tune_get(TUNE_SMALL_NT_1024) == 256)
                return launch_small<1024, 256>(items, n_items, mb, nr, pp, deepest, st, timer);
            if (tune_get(TUNE_SMALL_NT_1024) == 1024)
                return launch_small<1024, 1024>(items, n_items, mb, nr, pp, deepest, st, timer);
            return launch_small<1024, 512>(items, n_items, mb, nr, pp, deepest, st, timer);
        default:
            if (tune_get(TUNE_SMALL_NT_2048) == 512)
                return launch_small<SMALL_MAX, 512>(items, n_items, mb, nr, pp, deepest, st, timer);
            return launch_small<SMALL_MAX, 1024>(items, n_items, mb, nr, pp, deepest, st, timer);
    }
}

int run_small_buckets(const SmallItem* buckets, int64_t stride, const int32_t* counts,
                      const Members& mb, const NodeRec& nr, const PhaseParams& pp,
                      int32_t* deepest, hipStream_t st, const SmallFork& fork,
                      const char* timer) {
    const bool split =
        fork.stream && counts[3] > 0 && (counts[0] > 0 || counts[1] > 0 || counts[2] > 0);
    hipStream_t low = split ? fork.stream : st;
    if (split) {
        RS_HIP(hipEventRecord(fork.ready, st));
        RS_HIP(hipStreamWaitEvent(low, fork.ready, 0));
    }
    int rc = RS_OK;
    for (int b = 3; b >= 0 && rc == RS_OK; b--)
        rc = run_small_bucket(b, buckets + b * stride, counts[b], mb, nr, pp, deepest,
                              b == 3 ? st : low, timer);
    if (split) {
        // also after a failure: what has been launched ends before `st` goes on
        RS_HIP(hipEventRecord(fork.done, low));
        RS_HIP(hipStreamWaitEvent(st, fork.done, 0));
    }
    return rc;
}

}  // namespace rs
