// phase_tile.hip -- tile-cooperative searches over the 6D tree: the links
// within the linking length, and the nearest-neighbour distances.
//
// One wavefront owns a tile of 64 consecutive members (one query per lane).
// It walks the tree ONCE with the bounding box of its queries, collecting
// every leaf that any query could need into an LDS list (up to four stack
// entries per pass: cells average about ten children).  Up to 64 listed
// leaves at a time, one per lane, are then bounded against every query; each
// admitted leaf is read once and screened by matrix products against the
// queries that admit it (see k_tile_search), and the pairs that the screening
// cannot exclude are evaluated exactly, 64 at a time, and united or taken for
// the minima.
//
// What bounds it: vector instructions (four fifths of the issue slots in the
// nearest-neighbour search), and in the linking also the union-find's
// dependent reads.  All levels of one step, before this kernel and with it:
//   linking          512^3 199 -> 117 ms, deeply nested 9.1M particles
//                    34.2 -> 14.3 ms, 256^3 15.0 -> 8.1 ms
//   nearest (bracketed search) 512^3 237 -> 135 ms, deeply nested 29.7 -> 26.7
//   nearest (exact) 256^3 36.4 -> 13.1 + 1.1 ms (left to k_tree_nn),
//                    1M particles 6.5 -> 3.3 + 0.4 ms
// Loading the next leaf's operands ahead measured the same, as did five to
// eight wavefronts per SIMD.
#include "phase_common.h"

namespace rs {

// LDS per wavefront stays small enough for seven wavefronts per SIMD (the
// registers allow six): more of them hide more latency than larger buffers
// save
constexpr int TSTACK = 520;   // >= 64 internal children x 8 levels
constexpr int TLIST = 128;    // candidate leaves buffered (up to 63, and one pass)
constexpr int THITS = 64;     // linked pairs buffered before their unions (>= 64)
static_assert(TLIST >= 127 && THITS == 64, "one pass adds up to 64 leaves or pairs");
// A leaf that at most FEW queries admit is screened with one member per lane, a
// query at a time (some 20 vector instructions), instead of in a 16-wide tile
// that would be mostly empty columns (some 160 with its 8 products).  Two
// thirds of the leaves are such in 512^3 particles, nearly all of them with
// more than 32 members.  512^3, nearest and linking: none 193 + 140 ms, up to
// 2 queries 154 + 123, 4 146 + 118, 6 145 + 117, 9 144 + 117, 14 145 + 119.
constexpr int FEW = 6;
// The bounds exclude little where distances are tiny beside the node's extent
// (compact clumps far apart, below the resolution of the tree's cells), and
// evaluating most pairs from the queue costs several times what testing all of
// them does.  A tile is crowded when more than half of the pairs of the leaves
// so far with the queries had to be evaluated in the nearest-neighbour search,
// and CROWDED_MIN more: its queries are left to k_tree_nn then, and in the linking
// its leaves are replayed.  Two such clumps of 150000 members each: nearest 130
// -> 70 ms, linking 89 -> 30.  (Counting in the linking itself costs it 7 % where
// most of its time goes into true links.)
constexpr int CROWDED_MIN = 512;
constexpr int QS = 68;        // row stride of the queries' coordinates

struct TileRec {
    float lo[6], hi[6];
    int32_t start, end, cfirst, ccount;
};

RS_DEV TileRec trec_load(const float* __restrict__ erec, int32_t k) {
    const float4* p = reinterpret_cast<const float4*>(erec + 16 * (int64_t)k);
    float4 a = p[0], b = p[1], c = p[2], d = p[3];
    TileRec r;
    r.lo[0] = a.x; r.lo[1] = a.y; r.lo[2] = a.z; r.lo[3] = a.w; r.lo[4] = b.x; r.lo[5] = b.y;
    r.hi[0] = b.z; r.hi[1] = b.w; r.hi[2] = c.x; r.hi[3] = c.y; r.hi[4] = c.z; r.hi[5] = c.w;
    r.start = __float_as_int(d.x);
    r.end = __float_as_int(d.y);
    r.cfirst = __float_as_int(d.z);
    r.ccount = __float_as_int(d.w);
    return r;
}

// exact lower bound of the computed d^2 between a point (w: unwrapped
// position, u: velocity) or a box (wlo..whi, ulo..uhi) and a record's box;
// the record's position box is stored widened by the slack that covers the
// rounding of the coordinates relative to the reference member, of the pair
// difference and of the image shift; velocity gaps and the bound lose a
// relative margin
RS_DEV float box_box_lb(const float blo[6], const float bhi[6], const TileRec& r, float a,
                        float c) {
    float sp = 0.0f, sv = 0.0f;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const float g = fmaxf(fmaxf(r.lo[d] - bhi[d], blo[d] - r.hi[d]), 0.0f);
        sp += g * g;
        float h = fmaxf(fmaxf(r.lo[3 + d] - bhi[3 + d], blo[3 + d] - r.hi[3 + d]), 0.0f) *
                  0.99999905f;
        sv += h * h;
    }
    return (a * sp + c * sv) * 0.99999f;
}

RS_DEV float tw_min(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

RS_DEV float tw_max(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

struct TStackEnt {
    int32_t cfirst, ccount;
};

// A pushed cell in LDS.  In the compact form (below 2^26 child records) four
// bytes: the first child's record below the count of 1 to 63 children, or 0
// and the cell's own record, from which the range is read back.
template <bool COMPACT>
struct TSlot;
template <>
struct TSlot<true> {
    uint32_t v;
    static RS_DEV TSlot pack(int32_t rec, int32_t cfirst, int32_t ccount) {
        return ccount < 64 ? TSlot{(uint32_t)ccount << 26 | (uint32_t)cfirst} : TSlot{(uint32_t)rec};
    }
    RS_DEV TStackEnt unpack(const float* __restrict__ erec) const {
        const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
        TStackEnt e{(int32_t)(u & 0x3ffffffu), (int32_t)(u >> 26)};
        if (e.ccount == 0) {
            const int2 c = *reinterpret_cast<const int2*>(erec + 16 * (int64_t)e.cfirst + 14);
            e = TStackEnt{__builtin_amdgcn_readfirstlane(c.x), __builtin_amdgcn_readfirstlane(c.y)};
        }
        return e;
    }
};
template <>
struct TSlot<false> {
    int32_t cfirst, ccount;
    static RS_DEV TSlot pack(int32_t, int32_t cfirst, int32_t ccount) {
        return TSlot{cfirst, ccount};
    }
    RS_DEV TStackEnt unpack(const float* __restrict__) const { return TStackEnt{cfirst, ccount}; }
};

// sum over the 64 lanes, in every lane (counting build)
RS_DEV int32_t wave_sum_i32(int32_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// an element of the normalised rows (below 2^28 members a 32-bit byte offset)
template <bool O32>
RS_DEV float xload(const float* __restrict__ base, int64_t i, int off = 0) {
    if constexpr (O32)
        return (reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) +
                                               ((uint32_t)i << 2)))[off];
    else
        return base[i + off];
}

// exact d^2 of two members (the image shift changes nothing where a node has
// none)
template <bool O32>
RS_DEV float exact_d2(const Members& T, int64_t i, int64_t j, const LParam& P,
                      const PhaseParams& pp) {
    return phase_d2<true>(mload<O32>(T.x, i), mload<O32>(T.y, i), mload<O32>(T.z, i),
                          mload<O32>(T.vx, i), mload<O32>(T.vy, i), mload<O32>(T.vz, i),
                          mload<O32>(T.x, j), mload<O32>(T.y, j), mload<O32>(T.z, j),
                          mload<O32>(T.vx, j), mload<O32>(T.vy, j), mload<O32>(T.vz, j), P.a,
                          P.c, pp.L, pp.h);
}

// Unites the components of a and b, whose parents pa and pb have just been
// read.  Both walks advance together, and both ends are left pointing at the
// root they found (a non-root's parent is only ever replaced by an ancestor),
// so that most of the many pairs inside one component end at the comparison
// of their parents.
RS_DEV void unite_pair(int* par, int a, int b, int pa, int pb) {
    int ra = pa, rb = pb;
    for (;;) {
        const int na = uf_load(par, ra), nb = uf_load(par, rb);
        if (na != ra || nb != rb) {
            ra = na;
            rb = nb;
            if (ra != rb) continue;
        }
        if (ra == rb) break;
        const int lo = min(ra, rb), hi = max(ra, rb);
        const int old = atomicCAS(par + hi, hi, lo);
        ra = lo;
        rb = old == hi ? lo : old;
        if (ra == rb) break;
    }
    if (pa != ra && a != ra)
        __hip_atomic_store(par + a, ra, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (pb != ra && b != ra)
        __hip_atomic_store(par + b, ra, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// pair tests of the counting build (instrumentation level 2)
__device__ unsigned long long g_link_pairs[64], g_near_pairs[64];

// NN false: links within l among later members; the active queries are those
// with d_i^2 <= l^2, all with that threshold.
//
// NN true: nearest-neighbour d^2 of the tile's members in the modes of
// k_tree_nn (which explains them and their codes).  A query's threshold is
// its best d^2 so far, first the nearest in its own tile, and the search cap;
// it falls as candidates are evaluated, and a query whose best is within the
// early stop leaves the search.  Without a cap (modes 0 and 5) the tile
// searches up to the first guess that nine tenths of its queries stay below,
// as one far outlier would have the whole tile walk the tree; a query with
// nothing that near is left for k_tree_nn, marked by the negated bound it has
// (256^3, both kernels: three quarters 19.7 ms, half 25.8, nine tenths 17.7).
// Nodes that percolate are left to it altogether.
template <bool NN, bool O32, bool CNT>
__global__ void __launch_bounds__(64, 6)
k_tile_search(TArgs A, int ntiles, int chunk, float* __restrict__ d2,
              int32_t* __restrict__ par) {
    __shared__ TSlot<O32> stk[TSTACK];
    __shared__ int32_t list[TLIST];
    __shared__ int2 hits[THITS];
    __shared__ float qX[9 * QS];     // -2 X of the queries, 1, scaled norm less the threshold,
                                     // and the threshold of the box bounds
    __shared__ uint32_t bst[NN ? 64 : 1];   // best d^2 of the queries, as bits
    __shared__ float tbox[12];       // box of the active queries
    __shared__ int32_t col[16];      // query of each column
    const int lane = threadIdx.x;
    const int t = xcd_chunk_index(blockIdx.x, chunk);
    if (t >= ntiles) return;
    const TreeBuf& tb = A.tb;
    const int v = A.tile_node[t];
    const LNode nd = A.nodes[v];
    const int64_t ts = nd.t_off + 64ll * (t - nd.tile0);
    const int64_t te = min(ts + 64, nd.t_off + (int64_t)nd.size);
    const LParam P = A.prm[v];
    const Members& T = A.T;
    const PhaseParams& pp = A.pp;
    const bool cull = P.cull != 0;
    if (NN && lane == 0 && P.nnmode <= 1) A.crowded[t] = 0;   // a level's first search
    if (NN && (!cull || P.nnmode == 2)) return;
    const NNMode md = nn_mode(P);

    // this lane's query
    const int64_t mq = ts + lane;
    const bool valid = mq < te;
    const int64_t mm = valid ? mq : ts;
    const float l2 = P.l2;
    bool act = valid && (NN ? !md.refine || d2[mm] == md.redo : mload<O32>(d2, mm) <= l2);
    uint64_t amask = __ballot(act);
    if (!amask) return;
    const int lm = lane & 15, lk = lane >> 4, lkb = lk < 2 ? lk : 2;
    // A pair is a candidate when its bound does not exceed the threshold (with
    // the slack of image shifts where the node has them); the tiny constant
    // makes the difference negative for coinciding points at threshold 0, and
    // covers the denormal range.
    const float tiny = 1e-30f + lb_abs(P.a, P.c);
    const float eta = sqrtf(P.a) * box_slack(pp.L);
    auto slacked = [&](float r2) {
        return P.nowrap ? r2
                        : r2 * (1.0f + LB_WRAP) + (1.0f + 1.0f / LB_WRAP) * 1.001f * eta * eta;
    };
    const float norm = xload<O32>(A.X.b, 3 * mm + 2);
    auto set_threshold = [&](float r2) {
        const float thr = slacked(r2);
        qX[7 * QS + lane] = norm - (thr * 1.000001f + tiny);
        qX[8 * QS + lane] = 4.0f * (thr * 1.00001f + tiny);
    };
#pragma unroll
    for (int k = 0; k < 4; k++) qX[k * QS + lane] = -2.0f * xload<O32>(A.X.a, 4 * mm + k);
#pragma unroll
    for (int k = 0; k < 2; k++) qX[(4 + k) * QS + lane] = -2.0f * xload<O32>(A.X.b, 3 * mm + k);
    qX[6 * QS + lane] = 1.0f;
    qX[7 * QS + lane] = norm;
    if (lane < 8) qX[lane * QS + 64] = lane < 6 ? 0.0f : lane == 6 ? 1.0f : NORM_PAD;
    if (lane < 16) col[lane] = 0;
    __syncthreads();

    float best = 0.0f;      // NN: nearest d^2 found (or the cap)
    float r2 = l2;          // largest threshold of the active queries
    float limit = md.cap;   // NN: distances beyond it are not resolved here
    if constexpr (NN) {
        // the nearest in the tile: all its pairs' bounds, then the exact d^2 to
        // the best bounded (only a first threshold: the tile's leaves are
        // searched like all others)
        const int n = (int)(te - ts);
        const int32_t kmask = key_mask();
        int32_t k1[4];
#pragma unroll
        for (int cb = 0; cb < 4; cb++) k1[cb] = 0x7fffffff;
        for (int rb = 0; rb < 4; rb++) {
            const int64_t m = ts + 16 * rb + lm;
            const float a0 = xload<O32>(A.X.a, 4 * m + lk);
            float a1 = xload<O32>(A.X.b, 3 * m + lkb);
            if (lk == 3) a1 = 1.0f;
#pragma unroll
            for (int cb = 0; cb < 4; cb++) {
                f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
                o = mfma_16x16x4(a0, qX[lk * QS + 16 * cb + lm], o);
                o = mfma_16x16x4(a1, qX[(4 + lk) * QS + 16 * cb + lm], o);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int row = 16 * rb + 4 * lk + k;
                    const float b = row >= n || row == 16 * cb + lm ? NORM_PAD : o[k];
                    k1[cb] = min(k1[cb], key_of(b, rb << 2 | k, kmask));
                }
            }
        }
        int near = 0;
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            int row = (key_row(k1[cb]) >> 2) * 16 + 4 * lk + (k1[cb] & 3);
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const int32_t f = __shfl_xor(k1[cb], o, 64);
                const int fr = __shfl_xor(row, o, 64);
                row = f < k1[cb] ? fr : row;
                k1[cb] = min(k1[cb], f);
            }
            if (lk == cb) near = row;
        }
        best = md.cap;
        if (act && n > 1 && near < n && near != lane)
            best = fminf(best, exact_d2<O32>(T, mm, ts + near, P, pp));
        act = act && !(best <= md.stop);
        amask = __ballot(act);
        if (!(md.cap < __builtin_huge_valf())) {
            // the bound that nine tenths of the queries stay below
            const uint32_t bits = __float_as_uint(best);
            uint64_t cand = amask;
            int kk = (9 * __popcll(amask) + 9) / 10;
            for (int b = 30; b >= 0 && __popcll(cand) > 1; b--) {
                const uint64_t zero = cand & __ballot(((bits >> b) & 1u) == 0);
                const int c = __popcll(zero);
                if (kk <= c) cand = zero;
                else {
                    kk -= c;
                    cand &= ~zero;
                }
            }
            if (cand) limit = lane_f(best, __builtin_ctzll(cand));
            if (!(limit < __builtin_huge_valf())) {   // no guess at all (a lone member)
                limit = -1.0f;
                act = false;
                amask = 0;
            }
        }
        bst[lane] = __float_as_uint(best);
        set_threshold(fminf(best, limit));
        r2 = __uint_as_float(~wave_min_u32(act ? ~__float_as_uint(fminf(best, limit)) : ~0u));
    } else {
        set_threshold(l2);
    }
    // its place in the boxes' frame, loaded where it is needed (registers
    // decide how many wavefronts hide each other's latencies here)
    auto load_query = [&](float q[6]) {
        q[0] = min_image(mload<O32>(T.x, mm) - P.rx, pp.L, pp.h);
        q[1] = min_image(mload<O32>(T.y, mm) - P.ry, pp.L, pp.h);
        q[2] = min_image(mload<O32>(T.z, mm) - P.rz, pp.L, pp.h);
        q[3] = mload<O32>(T.vx, mm);
        q[4] = mload<O32>(T.vy, mm);
        q[5] = mload<O32>(T.vz, mm);
    };
    {
        float q[6];
        load_query(q);
#pragma unroll
        for (int d = 0; d < 6; d++) {
            const float lo = tw_min(act ? q[d] : __builtin_huge_valf());
            const float hi = tw_max(act ? q[d] : -__builtin_huge_valf());
            if (lane == 0) {
                tbox[d] = lo;
                tbox[6 + d] = hi;
            }
        }
    }
    const float reach = sqrtf(slacked(r2));
    const int64_t first_act =
        NN ? -1 : ts + __ffsll((unsigned long long)amask) - 1;   // later members only

    int nhit = 0;
    uint64_t adm = 0;       // of the leaves screened together those to come,
    int nadm = 0;           // their number in all,
    int nexact = 0;         // NN: candidates of theirs evaluated,
    // and whether these are too many; the linking takes over what the search found
    bool crowded = !NN && __builtin_amdgcn_readfirstlane(A.crowded[t]) != 0;
    unsigned long long npairs = 0;   // counting build only
    // the queued candidates, one per lane: linked, or taken for the minima
    auto drain = [&]() {
        __syncthreads();
        if (lane < nhit) {
            const int2 p = hits[lane];
            if constexpr (NN) {
                atomicMin(bst + (p.x - (int)ts),
                          __float_as_uint(exact_d2<O32>(T, p.x, p.y, P, pp)));
            } else {
                const int pa = uf_load(par, p.x), pb = uf_load(par, p.y);
                if (pa != pb && exact_d2<O32>(T, p.x, p.y, P, pp) <= l2)   // else one component
                    unite_pair(par, p.x, p.y, pa, pb);
            }
        }
        if constexpr (NN) {
            nexact += nhit;
            crowded = nexact > CROWDED_MIN + 32 * __popcll(amask) * (nadm - __popcll(adm));
        }
        nhit = 0;
        __syncthreads();
        if constexpr (NN) {
            const float b = __uint_as_float(bst[lane]);
            if (b < best) {
                best = b;
                set_threshold(fminf(best, limit));
                act = act && !(best <= md.stop);
            }
            amask = __ballot(act);
        }
    };

    // Nodes that percolate (no culling) and crowded tiles: per buffered leaf, every
    // active query is replayed against the members, on all lanes (a lane past the leaf's end
    // holds a valid member and is masked afterwards).
    auto replay = [&](int n) {
        const float qx = mload<O32>(T.x, mm), qy = mload<O32>(T.y, mm), qz = mload<O32>(T.z, mm);
        const float qu = mload<O32>(T.vx, mm), qv = mload<O32>(T.vy, mm),
                    qw = mload<O32>(T.vz, mm);
        for (int li = 0; li < n; li++) {
            const TileRec r = trec_load(tb.erec, list[li]);
            uint64_t mk = __ballot(act && r.end > mq + 1);
            if (!mk) continue;
            const int64_t mj = r.start + lane;
            const bool has = mj < r.end;
            const int64_t mjj = has ? mj : r.start;
            const float xj = mload<O32>(T.x, mjj), yj = mload<O32>(T.y, mjj),
                        zj = mload<O32>(T.z, mjj);
            const float uj = mload<O32>(T.vx, mjj), vj = mload<O32>(T.vy, mjj),
                        wj = mload<O32>(T.vz, mjj);
            // pairs are taken with later members only: for query ts + src the
            // lanes holding later members are those above src + ts - r.start
            const uint64_t hasm = __builtin_amdgcn_ballot_w64(has);
            const int32_t off = (int32_t)(ts + 1) - __builtin_amdgcn_readfirstlane(r.start);
            while (mk) {
                const int src = __ffsll((unsigned long long)mk) - 1;
                mk &= mk - 1;
                const float dd = phase_d2<true>(lane_f(qx, src), lane_f(qy, src), lane_f(qz, src),
                                                lane_f(qu, src), lane_f(qv, src), lane_f(qw, src),
                                                xj, yj, zj, uj, vj, wj, P.a, P.c, pp.L, pp.h);
                const int32_t k0 = off + src;
                const uint64_t later = k0 <= 0 ? hasm : (k0 >= 64 ? 0ull : hasm & (~0ull << k0));
                if (CNT) npairs += (unsigned long long)__popcll(later);
                const uint64_t hm = later & __builtin_amdgcn_ballot_w64(dd <= l2);
                if (hm) {
                    if (nhit + __popcll(hm) > THITS) drain();
                    if ((hm >> lane) & 1)
                        hits[nhit + __popcll(hm & lanemask_lt())] =
                            make_int2((int)(ts + src), (int)mj);
                    nhit += __popcll(hm);
                }
            }
        }
    };

    // Up to 64 buffered leaves at a time, one per lane: every active query is
    // broadcast and bounded against all of them, which leaves each lane the
    // mask of the queries that admit its leaf.  Per admitted leaf the queries
    // are gathered into the columns of 16-wide tiles, and lower bounds of d^2
    // less the threshold of all their pairs with the leaf's members come from
    // two matrix products per 16 members.  The sign bits of a lane's sixteen
    // results are its candidates; they are queued and evaluated exactly before
    // they are united.
    auto screen = [&](int n) {
        const bool in = lane < n;
        const TileRec r = trec_load(tb.erec, list[in ? lane : 0]);
        const int32_t rstart = r.start, rend = r.end;
        // the leaf's box in the frame of qX (-2 X), widened by what rounding
        // X can take from a difference (2 units of 2^-24 of either end's X,
        // and the shift from the reference member to the centre, at most two
        // of the eight units of L that the stored box is wider by)
        float lo[6], hi[6];
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const float s = k < 3 ? P.sa : P.sc;
            const float o = k == 0 ? P.rx - P.cx : k == 1 ? P.ry - P.cy : k == 2 ? P.rz - P.cz
                            : k == 3 ? -P.cu : k == 4 ? -P.cv : -P.cw;
            const float x0 = s * (r.lo[k] + o), x1 = s * (r.hi[k] + o);
            const float e = 2e-6f * (fmaxf(fabsf(x0), fabsf(x1)) + reach);
            lo[k] = -2.0f * (x1 + e);
            hi[k] = -2.0f * (x0 - e);
        }
        const float l2x4 = NN ? 0.0f : qX[8 * QS];
        // lane q: the leaves that query q admits.  A step bounds one query
        // against all leaves (some 23 vector instructions, coordinates
        // broadcast from LDS) or one leaf against all queries (some 33, box
        // broadcast from its lane), whichever set is cheaper to go through.
        uint32_t glo = 0, ghi = 0;
        adm = 0;
        if (23 * __popcll(amask) < 33 * n) {
            for (uint64_t left = amask; left; left &= left - 1) {
                const int q = __builtin_ctzll(left);
                float g2 = 0.0f;
#pragma unroll
                for (int k = 0; k < 6; k++) {
                    const float p = qX[k * QS + q];
                    const float g = p - __builtin_amdgcn_fmed3f(p, lo[k], hi[k]);
                    g2 = fmaf(g, g, g2);
                }
                const uint64_t m = __ballot(in && g2 <= (NN ? qX[8 * QS + q] : l2x4));
                adm |= m;
                if (lane == q) {
                    glo = (uint32_t)m;
                    ghi = (uint32_t)(m >> 32);
                }
            }
        } else {
            float p[6];
#pragma unroll
            for (int k = 0; k < 6; k++) p[k] = qX[k * QS + lane];
            for (int j = 0; j < n; j++) {
                float g2 = 0.0f;
#pragma unroll
                for (int k = 0; k < 6; k++) {
                    const float g =
                        p[k] - __builtin_amdgcn_fmed3f(p[k], lane_f(lo[k], j), lane_f(hi[k], j));
                    g2 = fmaf(g, g, g2);
                }
                const bool need = act && g2 <= (NN ? qX[8 * QS + lane] : l2x4);
                adm |= __ballot(need) ? 1ull << j : 0ull;
                if (j < 32) glo |= need ? 1u << j : 0u;
                else ghi |= need ? 1u << (j - 32) : 0u;
            }
        }
        // row operands: member start + 16 rb + lm, coordinates lk and 4 + lk
        nadm = __popcll(adm);
        nexact = 0;
        while (adm) {
            if (NN && crowded) return;
            const int src = __builtin_ctzll(adm);
            adm &= adm - 1;
            const int32_t start = __builtin_amdgcn_readlane(rstart, src);
            const int32_t len = __builtin_amdgcn_readlane(rend, src) - start;
            const uint64_t mk =
                __ballot(((src < 32 ? glo : ghi) >> (src & 31)) & 1u) & (NN ? amask : ~0ull);
            if (NN && !mk) continue;
            // members of this tile (or, linking, before it) among the leaf's
            const bool own = start < (int32_t)te && (!NN || start + len > (int32_t)ts);
            if (CNT) {
                const int32_t later = !((mk >> lane) & 1) ? 0
                    : NN ? len : max(start + len - (int32_t)max((int64_t)start, mq + 1), 0);
                npairs += (unsigned long long)wave_sum_i32(later);
            }
            const int nq = __popcll(mk);
            if (nq <= FEW) {
                // the same bound, summed in the vector unit
                const int64_t m = (int64_t)start + lane;
                float x[7];
#pragma unroll
                for (int k = 0; k < 4; k++) x[k] = xload<O32>(A.X.a, 4 * m + k);
#pragma unroll
                for (int k = 0; k < 3; k++) x[4 + k] = xload<O32>(A.X.b, 3 * m + k);
                const int32_t j = start + lane;
                for (uint64_t left = mk; left; left &= left - 1) {
                    const int q = __builtin_ctzll(left);
                    float s = qX[7 * QS + q] + x[6];
#pragma unroll
                    for (int k = 0; k < 6; k++) s = fmaf(x[k], qX[k * QS + q], s);
                    const int32_t i = (int32_t)ts + q;
                    const bool ok = lane < len && __float_as_int(s) < 0 &&
                                    (!own || (NN ? j != i : j > i));
                    const uint64_t hm = __ballot(ok);
                    if (!hm) continue;
                    if (nhit + __popcll(hm) > THITS) drain();
                    if (ok) hits[nhit + __popcll(hm & lanemask_lt())] = make_int2(i, j);
                    nhit += __popcll(hm);
                }
                continue;
            }
            // all four row blocks, whatever the leaf's length (rows past its end
            // are masked below): no branches between the products
            const int64_t m = (int64_t)start + lm;
            float a0[4], a1[4];
#pragma unroll
            for (int rb = 0; rb < 4; rb++) {
                a0[rb] = xload<O32>(A.X.a, 4 * m + lk, 64 * rb);
                a1[rb] = xload<O32>(A.X.b, 3 * m + lkb, 48 * rb);
            }
            // results 4 rb + t of a lane, the first in bit 15, are rows
            // 16 rb + 4 lk + t
            const uint32_t rows =
                (0xffff0000u >> (4 * (len >> 4) + min(max((len & 15) - 4 * lk, 0), 4))) & 0xffffu;
            const int rank0 = __popcll(mk & lanemask_lt());
#pragma unroll
            for (int rb = 0; rb < 4; rb++) a1[rb] = lk == 3 ? 1.0f : a1[rb];
            for (int c0 = 0; c0 < nq && !(NN && crowded); c0 += 16) {
                const uint32_t rank = (uint32_t)(rank0 - c0);
                if (((mk >> lane) & 1) && rank < 16u) col[rank] = lane;
                __builtin_amdgcn_wave_barrier();
                const int qc = col[lm];
                const int q = c0 + lm < nq ? qc : 64;   // column 64: no query
                __builtin_amdgcn_wave_barrier();
                const float b0 = qX[lk * QS + q], b1 = qX[(4 + lk) * QS + q];
                f32x4 o[4];
                const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int rb = 0; rb < 4; rb++) o[rb] = mfma_16x16x4(a0[rb], b0, zero);
#pragma unroll
                for (int rb = 0; rb < 4; rb++) o[rb] = mfma_16x16x4(a1[rb], b1, o[rb]);
                uint32_t bits = 0;
#pragma unroll
                for (int rb = 0; rb < 4; rb++)
#pragma unroll
                    for (int t = 0; t < 4; t++)
                        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(o[rb][t]), 31);
                bits &= rows;
                uint64_t any = __ballot(bits != 0);
                while (any) {
                    const int b = 16 - __ffs((int)bits);
                    const int32_t i = (int32_t)ts + q;
                    const int32_t j = start + 16 * (b >> 2) + 4 * lk + (b & 3);
                    const bool ok = bits != 0 && (!own || (NN ? j != i : j > i));
                    const uint64_t hm = __ballot(ok);
                    if (nhit + __popcll(hm) > THITS) drain();
                    if (ok) hits[nhit + __popcll(hm & lanemask_lt())] = make_int2(i, j);
                    nhit += __popcll(hm);
                    bits &= bits - 1;
                    any = __ballot(bits != 0);
                }
            }
        }
    };
    auto process = [&](int n) {
        if (n == 0) return;   // nothing listed: no entry to read
        __syncthreads();
        if constexpr (!NN) {
            if (cull && !crowded) screen(n);
            else replay(n);
        } else if (!crowded) {
            screen(n);
            if (nhit) drain();
            if (crowded) {
                if (lane == 0) A.crowded[t] = 1;
                limit = -1.0f;
                act = false;
                amask = 0;
            }
            r2 = __uint_as_float(
                ~wave_min_u32(act ? ~__float_as_uint(fminf(best, limit)) : ~0u));
        }
    };

    // walk the tree with the tile box; buffer leaves, flush when full
    int nlist = 0;
    // a root is not a record: it is walked directly before anything is popped
    TStackEnt se{tb.cfirst[A.root[v]], tb.ccount[A.root[v]]};
    int sp = 0;
    __syncthreads();
    while (!NN || amask) {
        // cells average about ten children: up to four entries whose
        // children fit in 64 lanes are scanned in one pass, each on its own
        // run of lanes (a pass pushes at most 64 entries, as one cell does)
        int32_t cf1 = 0, cf2 = 0, cf3 = 0, e1 = 64, e2 = 64, e3 = 64, tot = se.ccount;
        if (sp > 0 && tot < 64) {
            TStackEnt n1 = stk[sp - 1].unpack(tb.erec);
            if (tot + n1.ccount <= 64) {
                sp--;
                cf1 = n1.cfirst;
                e1 = tot;
                tot += n1.ccount;
                if (sp > 0 && tot < 64) {
                    n1 = stk[sp - 1].unpack(tb.erec);
                    if (tot + n1.ccount <= 64) {
                        sp--;
                        cf2 = n1.cfirst;
                        e2 = tot;
                        tot += n1.ccount;
                        if (sp > 0 && tot < 64) {
                            n1 = stk[sp - 1].unpack(tb.erec);
                            if (tot + n1.ccount <= 64) {
                                sp--;
                                cf3 = n1.cfirst;
                                e3 = tot;
                                tot += n1.ccount;
                            }
                        }
                    }
                }
            }
            // lanes [0, e1) scan the first entry, [e1, e2) the second, ...
            se.ccount = tot;
        }
        __syncthreads();
        for (int32_t b0 = 0; b0 < se.ccount; b0 += 64) {
            const int32_t k = lane >= e3   ? cf3 + lane - e3
                              : lane >= e2 ? cf2 + lane - e2
                              : lane >= e1 ? cf1 + lane - e1
                                           : se.cfirst + b0 + lane;
            bool need = false, leaf = false;
            TileRec r;
            r.cfirst = -1;
            r.ccount = 0;
            if (b0 + lane < se.ccount) {
                r = trec_load(tb.erec, k);
                leaf = r.cfirst < 0;
                float blo[6], bhi[6];
#pragma unroll
                for (int d = 0; d < 6; d++) {
                    blo[d] = tbox[d];
                    bhi[d] = tbox[6 + d];
                }
                need = r.end > first_act + 1 &&
                       (!cull || !(box_box_lb(blo, bhi, r, P.a, P.c) > r2));
            }
            const uint64_t imask = __ballot(need && !leaf);
            // nearest first: the cell that holds the tile goes on top, so that its
            // neighbourhood is searched before what is further up the tree (512^3
            // 143 -> 135 ms; boxes of the queries still active, taken anew, cost
            // more than they save)
            int at = sp + __popcll(imask & lanemask_lt());
            if constexpr (NN) {
                const bool top = need && !leaf && r.start <= (int32_t)ts && (int32_t)ts < r.end;
                const uint64_t tm = __ballot(top);
                if (tm) at = top ? sp + __popcll(imask) - 1 : at - (int)((tm & lanemask_lt()) != 0);
            }
            if (need && !leaf) stk[at] = TSlot<O32>::pack(k, r.cfirst, r.ccount);
            sp += __popcll(imask);
            const uint64_t lmask = __ballot(need && leaf);
            if (need && leaf) list[nlist + __popcll(lmask & lanemask_lt())] = k;
            nlist += __popcll(lmask);
            __syncthreads();
            if (nlist >= 64) {
                process(64);
                nlist -= 64;
                const int32_t rest = lane < nlist ? list[64 + lane] : 0;
                __syncthreads();
                if (lane < nlist) list[lane] = rest;
                __syncthreads();
            }
        }
        if (sp == 0) break;
        se = stk[--sp].unpack(tb.erec);
    }
    process(nlist);
    if constexpr (NN) {
        if (valid && (!md.refine || d2[mm] == md.redo))
            d2[mm] = best <= limit ? nn_code(md, P, best)
                     : md.cap < __builtin_huge_valf() && !crowded ? __builtin_huge_valf() : -best;
        if (CNT && lane == 0 && npairs) atomicAdd(&g_near_pairs[blockIdx.x & 63], npairs);
    } else {
        drain();
        if (CNT && lane == 0 && npairs) atomicAdd(&g_link_pairs[blockIdx.x & 63], npairs);
    }
}

// Runs one search over the level's tiles; the counting build clears its
// counters before and reads them back after (synchronous).
template <bool NN>
static int tile_search(const TArgs& A, int ntiles, float* d2, int32_t* par, hipStream_t st) {
    if (ntiles <= 0) return RS_OK;
    const int c = xcd_chunk(ntiles);
    // 32-bit offsets: four floats a member in the widest rows, and compact stack
    // entries
    const bool o32 = use_o32(4 * A.nmem) && A.tb.cap_entry < (1 << 26);
    const unsigned grid = xcd_chunk_grid(ntiles, c);
    if (!prof_count_pairs()) {
        if (o32) k_tile_search<NN, true, false><<<grid, 64, 0, st>>>(A, ntiles, c, d2, par);
        else k_tile_search<NN, false, false><<<grid, 64, 0, st>>>(A, ntiles, c, d2, par);
        RS_HIP(hipGetLastError());
        return RS_OK;
    }
    unsigned long long h[64] = {0};
    RS_HIP(hipStreamSynchronize(st));
    RS_HIP(NN ? hipMemcpyToSymbol(HIP_SYMBOL(g_near_pairs), h, sizeof(h))
              : hipMemcpyToSymbol(HIP_SYMBOL(g_link_pairs), h, sizeof(h)));
    if (o32) k_tile_search<NN, true, true><<<grid, 64, 0, st>>>(A, ntiles, c, d2, par);
    else k_tile_search<NN, false, true><<<grid, 64, 0, st>>>(A, ntiles, c, d2, par);
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(st));
    RS_HIP(NN ? hipMemcpyFromSymbol(h, HIP_SYMBOL(g_near_pairs), sizeof(h))
              : hipMemcpyFromSymbol(h, HIP_SYMBOL(g_link_pairs), sizeof(h)));
    double sum = 0.0;
    for (int i = 0; i < 64; i++) sum += (double)h[i];
    prof_add_count(NN ? "pairs_nn" : "pairs_link", sum);
    return RS_OK;
}

int tile_nn(const TArgs& A, int ntiles, float* d2, hipStream_t st) {
    return tile_search<true>(A, ntiles, d2, nullptr, st);
}

int tile_link(const TArgs& A, int ntiles, float* d2, int32_t* par, hipStream_t st) {
    return tile_search<false>(A, ntiles, d2, par, st);
}

}  // namespace rs
