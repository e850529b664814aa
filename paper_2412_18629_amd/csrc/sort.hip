// sort.hip -- stable LSD radix sort of (u64 or u32 key, i32 value) pairs over
// the low `bits` bits of the key, 8-bit digits, one pass per digit (the last
// pass narrower when `bits` is not a multiple of 8).
//
// Up to SB_MAX pairs one workgroup runs all passes in LDS (one launch).
// Above, each pass is three launches:
//   hist     per-tile digit counts, stored digit-major (cnt[d * ntiles + t])
//   scan     one workgroup per digit: exclusive scan of its counts over the
//            tiles in place, and the digit's total; tiles stay in input order
//            inside a digit, which makes the pass stable
//   scatter  each wavefront ranks a contiguous run of the tile's keys
//            (digit peers by ballots, running per-digit counts in its own LDS
//            row), the rows are combined into slots, the tile is laid out
//            in digit order in LDS and written back: keys of one digit from
//            one tile land in consecutive global slots, so the writes coalesce
// Passes alternate between the output and a scratch buffer so the last one
// lands in the output; the input is never written.
//
// What bounds it: memory traffic, 32 bytes a pair and pass of 64-bit keys, 20
// of 32-bit ones (keys read twice).  The
// scatter reaches the rate of a plain copy only when the lines that
// neighbouring tiles share are completed in one L2 (see the tile order
// below): 134M pairs, five passes, 9.03 -> 4.86 ms, its scatter 1.33 -> 0.70
// ms a pass (4.6 TB/s); with the tiles in launch order 8.3 ms.  12M pairs of
// 64-bit keys: 1.36 -> 0.77 ms.
#include <algorithm>

#include "common.h"

namespace rs {

constexpr int RB_T = 512;              // threads per block (8 wavefronts)
constexpr int RB_W = RB_T / 64;
constexpr int RB_D = 256;              // digits per pass
constexpr int RB_CHUNK = 256;          // consecutive tiles per XCD and round, at most
// Keys per thread: 16 make longer runs of a digit per tile (134M pairs, five
// passes: 4.86 ms against 5.76 with 8); below RB_LONG pairs 8 give the chip
// more tiles (12M pairs, eight passes: 0.77 ms against 0.79 with 16).
constexpr int64_t RB_LONG = (int64_t)1 << 24;

// peers of a lane's digit among the lanes with ok, and the rank of its key
// among the wavefront's keys so far (wc: the wavefront's running counts)
RS_DEV int rank_key(int d, bool ok, int32_t* wc) {
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; b++) {
        const bool bit = (d >> b) & 1;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    const int below = __popcll(peers & lanemask_lt());
    const int rk = ok ? wc[d] + below : -1;
    __builtin_amdgcn_wave_barrier();
    if (ok && below == 0) wc[d] += __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    return rk;
}

// exclusive scan of one value per thread of the first RB_D threads (four
// wavefronts); every thread of the block must call it
RS_DEV int32_t digit_scan(int32_t v, int32_t* part /* [4] */) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63 && w < 4) part[w] = inc;
    __syncthreads();
    int32_t before = 0;
#pragma unroll
    for (int q = 0; q < 3; q++) before += q < w ? part[q] : 0;
    __syncthreads();
    return before + inc - v;
}

// Tiles are dealt so that consecutive ones run on one XCD: their runs of one
// digit are neighbours in the output, and the lines they share are completed
// in one L2 instead of being written back in parts by several.
template <typename K, int RB_I>
__global__ void __launch_bounds__(RB_T)
k_rsort_hist(const K* __restrict__ keys, int64_t n, int shift, uint32_t dmask, int ntiles,
             int chunk, int32_t* __restrict__ cnt) {
    constexpr int RB_TILE = RB_T * RB_I;
    __shared__ int32_t h[RB_W][RB_D];
    const int tid = threadIdx.x, w = tid >> 6;
    const int t = xcd_chunk_index(blockIdx.x, chunk);
    if (t >= ntiles) return;
    for (int q = tid; q < RB_W * RB_D; q += RB_T) h[0][q] = 0;
    __syncthreads();
    const int64_t base = (int64_t)t * RB_TILE;
#pragma unroll
    for (int r = 0; r < RB_I; r++) {
        const int64_t i = base + r * RB_T + tid;
        if (i >= n) continue;
        const int d = (int)((keys[i] >> shift) & dmask);
        if constexpr (sizeof(K) == 4) {
            // 32-bit keys are labels and node indices, many of them equal: the lanes
            // with the first lane's digit count as one addition (16.7M members by
            // node, three passes 127 -> 77 us; 64-bit keys 0.18 -> 0.19 ms)
            const int d0 = __builtin_amdgcn_readfirstlane(d);
            const uint64_t same = __ballot(d == d0);
            if (d != d0) atomicAdd(&h[w][d], 1);
            else if ((same & lanemask_lt()) == 0) atomicAdd(&h[w][d], __popcll(same));
        } else {
            atomicAdd(&h[w][d], 1);
        }
    }
    __syncthreads();
    if (tid < RB_D) {
        int32_t s = 0;
#pragma unroll
        for (int q = 0; q < RB_W; q++) s += h[q][tid];
        cnt[(int64_t)tid * ntiles + t] = s;
    }
}

// one workgroup per digit: its counts over the tiles, scanned in place
constexpr int RS_T = 1024, RS_I = 4;

__global__ void __launch_bounds__(RS_T)
k_rsort_scan(int ntiles, int32_t* __restrict__ cnt, int32_t* __restrict__ total) {
    __shared__ int32_t part[RS_T / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int32_t* c = cnt + (int64_t)blockIdx.x * ntiles;
    int32_t carry = 0;
    for (int b = 0; b < ntiles; b += RS_T * RS_I) {
        int32_t v[RS_I], s = 0;
        const int i0 = b + tid * RS_I;
#pragma unroll
        for (int k = 0; k < RS_I; k++) {
            v[k] = i0 + k < ntiles ? c[i0 + k] : 0;
            s += v[k];
        }
        int32_t inc = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        if (lane == 63) part[w] = inc;
        __syncthreads();
        int32_t run = carry + inc - s;
#pragma unroll
        for (int q = 0; q < RS_T / 64; q++) {
            const int32_t p = part[q];
            if (q < w) run += p;
            carry += p;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RS_I; k++) {
            if (i0 + k < ntiles) c[i0 + k] = run;
            run += v[k];
        }
    }
    if (tid == 0) total[blockIdx.x] = carry;
}

template <typename K, int RB_I>
__global__ void __launch_bounds__(RB_T)
k_rsort_scatter(const K* __restrict__ kin, const int32_t* __restrict__ vin,
                K* __restrict__ kout, int32_t* __restrict__ vout, int64_t n, int shift,
                uint32_t dmask, int ntiles, int chunk, const int32_t* __restrict__ offs,
                const int32_t* __restrict__ total) {
    constexpr int RB_TILE = RB_T * RB_I;
    __shared__ K sk[RB_TILE];          // keys in digit order, then the values
    __shared__ int32_t wc[RB_W][RB_D]; // per wavefront: keys of each digit (then offsets)
    __shared__ int32_t gbase[RB_D];    // global slot of a digit's first key, less its tile slot
    __shared__ int32_t part[4];
    int32_t* sv = reinterpret_cast<int32_t*>(sk);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int t = xcd_chunk_index(blockIdx.x, chunk);
    if (t >= ntiles) return;
    const int64_t base = (int64_t)t * RB_TILE;
    const int nt = (int)min<int64_t>(RB_TILE, n - base);

    // each wavefront ranks its own contiguous run of RB_I * 64 keys in input
    // order: digit peers by ballots, running per-digit counts in its own LDS row
    K k[RB_I];
    int32_t v[RB_I];
    int rk[RB_I];
    const int64_t wbase = base + (int64_t)w * RB_I * 64;
#pragma unroll
    for (int r = 0; r < RB_I; r++) {
        const int64_t i = wbase + r * 64 + lane;
        k[r] = i < n ? kin[i] : 0;
        v[r] = i < n ? vin[i] : 0;
    }
    const int32_t dtot = tid < RB_D ? total[tid] : 0;
    const int32_t doff = tid < RB_D ? offs[(int64_t)tid * ntiles + t] : 0;
    for (int q = tid; q < RB_W * RB_D; q += RB_T) wc[0][q] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB_I; r++)
        rk[r] = rank_key((int)((k[r] >> shift) & dmask), wbase + r * 64 + lane < n, wc[w]);
    const int32_t dbase = digit_scan(dtot, part);
    // per digit: slots of wavefront w start after the lower wavefronts' keys
    int32_t c = 0;
    if (tid < RB_D)
#pragma unroll
        for (int q = 0; q < RB_W; q++) c += wc[q][tid];
    const int32_t dstart = digit_scan(c, part);
    if (tid < RB_D) {
        gbase[tid] = dbase + doff - dstart;
        int o = dstart;
#pragma unroll
        for (int q = 0; q < RB_W; q++) {
            const int cq = wc[q][tid];
            wc[q][tid] = o;
            o += cq;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB_I; r++) {
        if (rk[r] >= 0) {
            rk[r] += wc[w][(int)((k[r] >> shift) & dmask)];
            sk[rk[r]] = k[r];
        }
    }
    __syncthreads();
    int32_t g[RB_I];
#pragma unroll
    for (int r = 0; r < RB_I; r++) {
        const int j = r * RB_T + tid;
        if (j < nt) {
            const K kk = sk[j];
            g[r] = gbase[(int)((kk >> shift) & dmask)] + j;
            kout[g[r]] = kk;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB_I; r++)
        if (rk[r] >= 0) sv[rk[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB_I; r++) {
        const int j = r * RB_T + tid;
        if (j < nt) vout[g[r]] = sv[j];
    }
}

// All passes of at most SB_MAX pairs in one workgroup's LDS.  Three or more
// launches a pass cost more than the work of so few keys: 5000 pairs of 24
// bits 47 us in nine launches, 20 us in one.
constexpr int SB_T = 1024, SB_W = SB_T / 64, SB_I = 8, SB_MAX = SB_T * SB_I;

template <typename K>
__global__ void __launch_bounds__(SB_T)
k_rsort_block(const K* __restrict__ kin, const int32_t* __restrict__ vin, K* __restrict__ kout,
              int32_t* __restrict__ vout, int n, int bits) {
    extern __shared__ __align__(16) char smem[];
    K* sk = reinterpret_cast<K*>(smem);                            // [SB_MAX]
    int32_t* sv = reinterpret_cast<int32_t*>(sk + SB_MAX);         // [SB_MAX]
    int32_t* wc = sv + SB_MAX;                                     // [SB_W][RB_D]
    __shared__ int32_t part[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int rounds = (n + SB_T - 1) / SB_T;                      // keys per thread in use
    const int wbase = w * rounds * 64;
    K k[SB_I];
    int32_t v[SB_I];
    int rk[SB_I];
#pragma unroll
    for (int r = 0; r < SB_I; r++) {
        const int i = wbase + r * 64 + lane;
        const bool ok = r < rounds && i < n;
        k[r] = ok ? kin[i] : 0;
        v[r] = ok ? vin[i] : 0;
    }
    for (int shift = 0; shift < bits; shift += 8) {
        const uint32_t dmask = bits - shift < 8 ? (1u << (bits - shift)) - 1u : 255u;
        for (int q = tid; q < SB_W * RB_D; q += SB_T) wc[q] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < SB_I; r++)
            if (r < rounds)
                rk[r] = rank_key((int)((k[r] >> shift) & dmask), wbase + r * 64 + lane < n,
                                 wc + w * RB_D);
        __syncthreads();
        int32_t c = 0;
        if (tid < RB_D)
            for (int q = 0; q < SB_W; q++) c += wc[q * RB_D + tid];
        int32_t o = digit_scan(c, part);
        if (tid < RB_D)
            for (int q = 0; q < SB_W; q++) {
                const int cq = wc[q * RB_D + tid];
                wc[q * RB_D + tid] = o;
                o += cq;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < SB_I; r++)
            if (r < rounds && rk[r] >= 0) {
                const int pos = wc[w * RB_D + (int)((k[r] >> shift) & dmask)] + rk[r];
                sk[pos] = k[r];
                sv[pos] = v[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < SB_I; r++) {
            const int i = wbase + r * 64 + lane;
            if (r < rounds && i < n) {
                k[r] = sk[i];
                v[r] = sv[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < SB_I; r++) {
        const int i = wbase + r * 64 + lane;
        if (r < rounds && i < n) {
            kout[i] = k[r];
            vout[i] = v[r];
        }
    }
}

// Work space: a scratch pair of arrays, and at least the digit counts and
// totals.  Sized for 2048-key tiles and a second table as well, which the
// callers' limits (the work space of fixed size) are documented for.
size_t sort_temp_bytes(int64_t n, size_t key_bytes) {
    if (n < 1) n = 1;
    const int64_t nc = RB_D * ((n + 2047) / 2048);
    return arena_round((size_t)n * key_bytes) + arena_round((size_t)n * 4) +
           2 * arena_round((size_t)nc * 4) + arena_round(scan_temp_bytes(nc));
}

template <typename K, int I>
static int sort_passes(const K* kin, K* kout, const int32_t* vin, int32_t* vout, int64_t n,
                       int bits, void* temp, hipStream_t st) {
    const int passes = (bits + 7) / 8;
    const int64_t ntiles = (n + RB_T * I - 1) / (RB_T * I);
    char* p = static_cast<char*>(temp);
    K* kalt = reinterpret_cast<K*>(p);
    p += arena_round((size_t)n * sizeof(K));
    int32_t* valt = reinterpret_cast<int32_t*>(p);
    p += arena_round((size_t)n * 4);
    int32_t* cnt = reinterpret_cast<int32_t*>(p);
    p += arena_round((size_t)RB_D * ntiles * 4);
    int32_t* total = reinterpret_cast<int32_t*>(p);

    // chunks stay short enough for every XCD to get several
    const int64_t per = ntiles / (16 * XCDS);
    const int chunk = per < 1 ? 1 : per > RB_CHUNK ? RB_CHUNK : (int)per;
    const unsigned grid = (unsigned)xcd_chunk_grid((int)ntiles, chunk);
    const K* sk = kin;
    const int32_t* svv = vin;
    for (int pass = 0; pass < passes; pass++) {
        const bool to_out = ((passes - 1 - pass) % 2) == 0;
        K* dk = to_out ? kout : kalt;
        int32_t* dv = to_out ? vout : valt;
        const int shift = 8 * pass;
        const int db = bits - shift < 8 ? bits - shift : 8;   // digit width of this pass
        const uint32_t dmask = (1u << db) - 1u;
        k_rsort_hist<K, I><<<grid, RB_T, 0, st>>>(sk, n, shift, dmask, (int)ntiles, chunk, cnt);
        k_rsort_scan<<<RB_D, RS_T, 0, st>>>((int)ntiles, cnt, total);
        k_rsort_scatter<K, I><<<grid, RB_T, 0, st>>>(sk, svv, dk, dv, n, shift, dmask,
                                                     (int)ntiles, chunk, cnt, total);
        RS_HIP(hipGetLastError());
        sk = dk;
        svv = dv;
    }
    return RS_OK;
}

template <typename K>
static int sort_pairs(const K* kin, K* kout, const int32_t* vin, int32_t* vout, int64_t n,
                      int bits, void* temp, size_t temp_bytes, hipStream_t st) {
    if (n <= 0) return RS_OK;
    if (n >= ((int64_t)1 << 31)) return RS_EINVAL;
    if (temp_bytes < sort_temp_bytes(n, sizeof(K)) || !temp) return RS_EINTERNAL;
    bits = std::max(1, std::min(bits, (int)(8 * sizeof(K))));
    if (n <= SB_MAX) {
        const size_t lds = (size_t)SB_MAX * (sizeof(K) + 4) + (size_t)SB_W * RB_D * 4;
        RS_HIP(hipFuncSetAttribute((const void*)k_rsort_block<K>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        k_rsort_block<K><<<1, SB_T, lds, st>>>(kin, vin, kout, vout, (int)n, bits);
        RS_HIP(hipGetLastError());
        return RS_OK;
    }
    return n < RB_LONG ? sort_passes<K, 8>(kin, kout, vin, vout, n, bits, temp, st)
                       : sort_passes<K, 16>(kin, kout, vin, vout, n, bits, temp, st);
}

int sort_pairs_u64_i32(const uint64_t* kin, uint64_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, int bits, void* temp, size_t temp_bytes,
                       hipStream_t st) {
    return sort_pairs(kin, kout, vin, vout, n, bits, temp, temp_bytes, st);
}

int sort_pairs_u32_i32(const uint32_t* kin, uint32_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, int bits, void* temp, size_t temp_bytes,
                       hipStream_t st) {
    return sort_pairs(kin, kout, vin, vout, n, bits, temp, temp_bytes, st);
}

}  // namespace rs
