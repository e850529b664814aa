// common.h -- shared device helpers and host plumbing of librsfof.
//
// Pair arithmetic follows the fixed fp32 recipe of rsfof.h: one periodic
// shift per axis, squares summed as ((x^2 + y^2) + z^2), no contraction.
// The library is compiled with -ffp-contract=off; the helpers below keep
// every rounding step as a separate statement so no fusion can occur.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <mutex>

#include "../../include/rsfof.h"

#define RS_DEV __device__ __forceinline__

namespace rs {

// ---------------------------------------------------------------------------
// fp32 pair arithmetic
// ---------------------------------------------------------------------------

RS_DEV float min_image(float d, float L, float h) {
    // one periodic image shift; identical for (i,j) and (j,i) up to sign
    return d > h ? d - L : (d < -h ? d + L : d);
}

RS_DEV float sum_sq3(float dx, float dy, float dz) {
    float sx = dx * dx;
    float sy = dy * dy;
    float sz = dz * dz;
    float t = sx + sy;
    return t + sz;
}

RS_DEV float pos_d2_wrap(float xi, float yi, float zi, float xj, float yj, float zj,
                         float L, float h) {
    return sum_sq3(min_image(xi - xj, L, h), min_image(yi - yj, L, h),
                   min_image(zi - zj, L, h));
}

RS_DEV float pos_d2_nowrap(float xi, float yi, float zi, float xj, float yj, float zj) {
    return sum_sq3(xi - xj, yi - yj, zi - zj);
}

RS_DEV float metric(float a, float Dx, float c, float Dv) {
    float u = a * Dx;
    float w = c * Dv;
    return u + w;
}

// ---------------------------------------------------------------------------
// lock-free union-find over an int32 parent array.
// Invariant: parent[v] <= v, roots satisfy parent[r] == r.  Hooks always put
// the larger root under the smaller one (CAS on the root), so no cycle can
// form; path halving stores only ancestors, which is benign under races.
//
// Reads are relaxed at workgroup scope, so they are served by the XCD's own
// L2 and may return an older value written from another XCD.  An older value
// of parent[v] is still an ancestor of v (links are never undone and every
// store writes an ancestor), so a walk still ends at a former root, two walks
// ending at the same node still prove one component, and a stale answer only
// costs a redundant test.  Hooking is a CAS at agent scope on the root itself:
// it fails on a stale root and returns the current parent, which is smaller,
// so the retry loop makes progress.  Path-halving stores stay at agent scope.
// ---------------------------------------------------------------------------

RS_DEV int uf_load(const int* p, int v) {
    return __hip_atomic_load(p + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

RS_DEV int uf_find(int* par, int v) {
    int cur = uf_load(par, v);
    if (cur == v) return v;
    int prev = v, next;
    while (cur > (next = uf_load(par, cur))) {
        __hip_atomic_store(par + prev, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        prev = cur;
        cur = next;
    }
    return cur;
}

// read-only root walk used when flattening: it stores nothing, so parallel
// flatteners cannot overwrite a finished entry with an intermediate ancestor
RS_DEV int uf_root(const int* par, int v) {
    int cur = uf_load(par, v);
    while (cur != v) {
        v = cur;
        cur = uf_load(par, v);
    }
    return v;
}

RS_DEV void uf_unite(int* par, int a, int b) {
    int ra = uf_find(par, a), rb = uf_find(par, b);
    while (ra != rb) {
        if (ra > rb) { int t = ra; ra = rb; rb = t; }
        int old = atomicCAS(par + rb, rb, ra);
        if (old == rb) return;
        rb = uf_find(par, old);
        ra = uf_find(par, ra);
    }
}

// ---------------------------------------------------------------------------
// wave-level aggregation of atomics on clustered keys: lanes holding the same
// key elect a leader, so a run of equal keys costs one atomic, not one per
// lane.  Every lane of the wavefront must call these (ballots).
// ---------------------------------------------------------------------------

RS_DEV uint64_t lanemask_lt() { return (1ull << (threadIdx.x & 63)) - 1ull; }

RS_DEV unsigned long long wave_min_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, o, 64);
        unsigned hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), o, 64);
        unsigned long long w = ((unsigned long long)hi << 32) | lo;
        v = w < v ? w : v;
    }
    return v;
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Blocks are remapped so that every XCD runs consecutive chunks of C
// tiles: neighbouring tiles, which read mostly the same candidate data, then
// share one L2.  The grid is rounded up to whole rounds of 8*C blocks; the
// mapping is a bijection on the rounded range, and blocks whose tile index
// is past the end exit.
constexpr int XCDS = 8;
RS_DEV int xcd_chunk_index(int b, int C) {
    const int x = b % XCDS, r = b / XCDS;
    return ((r / C) * XCDS + x) * C + r % C;
}
inline int xcd_chunk_grid(int n, int C) {
    const int g = XCDS * C;
    return (n + g - 1) / g * g;
}

// value of lane l (uniform) in every lane
RS_DEV float lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// minimum over the 64 lanes, uniform: row steps by DPP, then two row
// broadcasts carry it to lane 63.  All 64 lanes must be active.  Rows a
// broadcast skips read the identity (all ones), so each step is one DPP
// minimum.
RS_DEV uint32_t wave_min_u32(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0xB1, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x4E, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x124, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x128, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xa, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// ---------------------------------------------------------------------------
// Lower bounds of many pairs' d^2 by fp32 matrix products.  With norms and
// products of normalised coordinates, |Xi|^2 + |Xj|^2 - 2 Xi.Xj of 256 pairs
// takes two 16x16x4 products.  A lane holds operand element (row or column
// lane % 16, k = lane / 16) and the results of column lane % 16, rows
// 4 (lane / 16) + r.
//
// Squared norms are scaled by 1 - 2^-18, which lowers a pair's value by
// 64 * 2^-24 (|Xi|^2 + |Xj|^2): more than the rounding of X (2 units each,
// so at most 8 in the sum), of the norms (8), of the products and their
// summation (at most 24) and of the exact d^2 itself (8 units of d^2, which
// is at most 2 (|Xi|^2 + |Xj|^2)).
//
// In the denormal range roundings are no longer relative: a squared norm or
// coordinate sum may be off by a few units of 2^-149 (2^-126 each, should the
// products flush), and d^2 = a Dx + c Dv by that times a and c.  lb_abs() is
// above all of it together, and far below any d^2 of the normal range.
// ---------------------------------------------------------------------------

constexpr float LB_EPS = 3.814697265625e-06f;
RS_DEV float lb_abs(float a, float c) { return 1e-36f * (1.0f + a + c); }
constexpr float NORM_PAD = 1e30f;   // value of absent rows and columns
// Across a periodic face X also carries the absolute rounding of the image
// shift, at most eta = sqrt(a) box_slack(L) per pair of positions, and
// (D + eta)^2 <= (1 + k) D^2 + (1 + 1/k) eta^2.
constexpr float LB_WRAP = 0.0078125f;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Keys that order like non-negative floats (low KEY_BITS bits dropped, which
// only lowers them) and carry a row number there.  The mask comes from
// key_mask(), opaque to the compiler, so that a key is one bit-select.
constexpr int KEY_BITS = 9;

RS_DEV int32_t key_mask() {
    int32_t m = (1 << KEY_BITS) - 1;
    asm volatile("" : "+v"(m));
    return m;
}

RS_DEV int32_t key_of(float v, int32_t row, int32_t mask) {
    return (mask & row) | (~mask & __float_as_int(v));
}

RS_DEV float key_value(int32_t k) { return __int_as_float(k & ~((1 << KEY_BITS) - 1)); }
RS_DEV int32_t key_row(int32_t k) { return k & ((1 << KEY_BITS) - 1); }

// the two smallest keys, k1 <= k2
RS_DEV void key_take(int32_t& k1, int32_t& k2, int32_t key) {
    k2 = max(min(k1, k2), min(max(k1, k2), key));   // the median
    k1 = min(k1, key);
}

RS_DEV f32x4 mfma_16x16x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// exact 128-bit helpers
// ---------------------------------------------------------------------------

typedef __int128 i128;
typedef unsigned __int128 u128;

// Round-to-nearest-even conversion of a signed 128-bit integer to fp64.
RS_DEV double i128_to_f64(i128 v) {
    bool neg = v < 0;
    u128 u = neg ? (u128)0 - (u128)v : (u128)v;
    if (u == 0) return 0.0;
    uint64_t hi = (uint64_t)(u >> 64), lo = (uint64_t)u;
    int nbits = hi ? 128 - __builtin_clzll(hi) : 64 - __builtin_clzll(lo);
    double r;
    if (nbits <= 53) {
        r = (double)lo;                       // exact
    } else {
        int shift = nbits - 53;
        u128 m = u >> shift;
        u128 rem = u & (((u128)1 << shift) - 1);
        u128 half = (u128)1 << (shift - 1);
        if (rem > half || (rem == half && (m & 1))) m += 1;
        if (m == ((u128)1 << 53)) { m >>= 1; shift += 1; }
        r = __builtin_ldexp((double)(uint64_t)m, shift);
    }
    return neg ? -r : r;
}

}  // namespace rs

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

#define RS_HIP(expr)                                                        \
    do {                                                                    \
        hipError_t e_ = (expr);                                             \
        if (e_ != hipSuccess) return rs::hip_status(e_);                    \
    } while (0)

#define RS_TRY(expr)                                                        \
    do {                                                                    \
        int s_ = (expr);                                                    \
        if (s_ != RS_OK) return s_;                                         \
    } while (0)

namespace rs {

inline int hip_status(hipError_t e) {
    return e == hipErrorOutOfMemory ? RS_ENOMEM : RS_EDEVICE;
}

// Grow-only per-device workspaces with a bump allocator.  A call reserves
// the footprint of one phase once, then carves sub-buffers (256-byte
// aligned).  AR_BASE holds either the 3D pass's work space or the 6D pass's
// level-0 tables: both entry points synchronise their stream before they
// return, so the two are never live together and share one allocation (at
// 1024^3 each is about 100 GiB; two would not fit beside the large-node work
// space, and re-allocating them on every call costs seconds).  AR_LARGE and
// AR_TREE are the 6D pass's level pipeline, AR_MLP the proposer network,
// AR_SORT the standalone sort.
struct Arena {
    char* base = nullptr;
    size_t cap = 0;
    size_t off = 0;
};

constexpr int N_ARENAS = 5;
constexpr int AR_BASE = 0, AR_LARGE = 1, AR_MLP = 2, AR_SORT = 3, AR_TREE = 4;
// The arenas an API call uses; when a reservation cannot be met, the
// device's other arenas (left by earlier calls of other phases) are
// released and the allocation is tried again.
int arena_call_begin(uint32_t keep_mask);
// Serialises the library's calls on the current device (its workspaces are
// per device): every entry point that uses them holds this lock.
int call_lock(std::unique_lock<std::mutex>* lk);
// device bytes the current call could obtain: free memory plus the arenas it
// does not hold plus those in replace_mask (about to be re-reserved)
int device_budget(uint32_t replace_mask, size_t* bytes);
int arena_release(int which);
int arena_reserve(int which, size_t bytes, Arena** out);   // resets the bump pointer
void* arena_take(Arena* a, size_t bytes);       // NULL if the reservation is exceeded
size_t arena_round(size_t bytes);

template <class T>
inline T* take(Arena* a, size_t count) {
    return static_cast<T*>(arena_take(a, count * sizeof(T)));
}

// small pinned host scratch for reading back counters
int host_scratch(void** out, size_t bytes);

inline unsigned grid_for(int64_t n, int block, int64_t cap = 1 << 20) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// Optional per-kernel timing with HIP events recorded on the launching
// stream around instrumented launches (off unless enabled by the caller).
// `units` counts the work items a launch processed (members, particles).
void prof_begin(const char* name, hipStream_t st);
void prof_end(const char* name, hipStream_t st, double units);
// Level 2 of the instrumentation also counts the pair tests of the searches
// (kernels built with counters, slower; for measurement runs only).  After a
// counted launch the caller adds its count with prof_add_count (synchronous).
bool prof_count_pairs();
void prof_add_count(const char* name, double count);

// Tuning table: launch shapes chosen per size bucket by the autotuner.  Every
// value is one of a small compiled set; results are the same for all of them.
enum TuneKnob { TUNE_SMALL_NT_256, TUNE_SMALL_NT_1024, TUNE_SMALL_NT_2048, TUNE_XCD_CHUNK,
                TUNE_N };
int tune_get(TuneKnob k);

// device-wide primitives (prims.hip)
size_t scan_temp_bytes(int64_t n);
int scan_exclusive_i32(const int32_t* in, int32_t* out, int64_t n, void* temp,
                       int32_t* total_dev, hipStream_t st);
size_t sort_temp_bytes(int64_t n, size_t key_bytes = 8);
int sort_pairs_u32_i32(const uint32_t* kin, uint32_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, int bits, void* temp, size_t temp_bytes,
                       hipStream_t st);
int sort_pairs_u64_i32(const uint64_t* kin, uint64_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, int bits, void* temp, size_t temp_bytes,
                       hipStream_t st);
int fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st);

}  // namespace rs
