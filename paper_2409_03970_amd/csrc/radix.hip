// Plain sorts by stable digit passes (least significant digit first): the
// library's own choice where the caller asks for no merge shape (the sizes stand at
// radix_route in abi.hip).
//
// A merge sort of 2^28 keys makes seven four-way trips through HBM with two
// LDS merge levels in each; four passes over 8-bit digits read the keys twice
// and write them once each, whatever their distribution, and need no co-rank
// search.  Elements are compared by their mapped words: the key map of the
// sort turned into unsigned order, applied by the first pass as it reads and
// undone by the last as it writes.
//
// One pass is three launches:
//   count    digit histogram of every chunk of tiles (one workgroup each; LDS
//            atomics on 8 interleaved copies, so that equal digits in a wave
//            meet 8 counters), and before each tile the chunk's counts so far;
//   scan     exclusive prefix of every digit's counts over the chunks, and
//            the digits' totals;
//   scatter  a wave ranks 64 keys at a time: eight ballots give each lane the
//            mask of lanes with its digit, a counter per wave and digit
//            carries the rank on.  The tile is brought into digit order in
//            LDS and written out in runs.
// No workgroup waits for another.
//
// What bounds a pass (2^28 uniform keys): the count reads 1.07 GB in 0.20 ms
// (5.5 TB/s; 0.27 with loads that fill the memory-side cache on their way).
// The scatter takes 0.61 ms (0.58 in the first pass, see `spread`) for
// 2.15 GB: with its ranks left out and its writes made linear it would take
// 0.39, with the writes alone linear 0.52, so both the partial cache lines at
// the ends of the runs (8 % more bytes written than the keys have) and the 60
// VALU operations per key (32 of them the ballots; 28 in the first pass; 0.41 ms
// at the rate of all SIMDs) show.  Run ends are why the tile is as large as two workgroups
// per CU allow (16,384 keys, runs of 64: 0.665 against 0.79 ms at 8,192),
// and why the tiles are dealt so that an XCD's workgroups walk one contiguous
// range together: the line that two tiles' runs share is completed in that
// XCD's L2 by a neighbouring workgroup (0.61 against 0.665 ms with a
// contiguous range per workgroup).  Writing complete lines only, with the
// rest of each run held back in LDS for the next tile, was no faster (0.685:
// the branch per key and a third barrier cost what the lines saved), nor was
// loading the next tile's keys ahead (registers spill at 128).
//
// The first count also finds which bits vary and whether the input is
// already in order (or in reverse order).  From that one workgroup of the
// first scan launch makes the plan of the sort: passes over constant digits
// are skipped and presorted input is copied (sorted 2^28 keys 0.67 ms, of which
// the copy 0.44; 1.01 with one key to a thread in flight in both).  A
// pair sort whose values ascend in the input skips its value digits, since
// stable passes over the key alone then give the lexicographic order.
// Skipped launches return at once; nothing is read back by the host.
#include "common.h"
#include "hvms_internal.h"
#include "radix_plan.h"

namespace hvms {

namespace {

constexpr int RADIX = 256;
constexpr int COUNT_NT = 512;
constexpr int MAX_CHUNKS = 512;
constexpr int FEW_TILES = 32;
constexpr int SAMPLE_RUNS_MAX = 64;
constexpr int64_t SAMPLE_MIN = (int64_t)1 << 24;  // elements from which a sample is taken
constexpr int COPIES = 8;  // interleaved histogram copies of the count kernel

// The step of a pass, in scalar registers.
__device__ __forceinline__ Step step_of(const Ctl *ctl, int round, int pass)
{
    const uint32_t *q = (const uint32_t *)&ctl->step[round][pass];
    Step s;
    s.mode = round == 0 || ctl->again ? q[0] : (uint32_t)STEP_SKIP;
    s.mode = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.mode);
    s.src = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[1]);
    s.dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[2]);
    s.first = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[3]);
    s.last = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[4]);
    return s;
}
__device__ __forceinline__ Step step_of(const RadixArgs &a, int pass)
{
    return step_of((const Ctl *)a.ctl, a.round, pass);
}

// What one chunk's count found; flags as of the plan.
// near0, near1: the smallest difference (xor, minus 1) between an element and the
// one after it, over those that differ in the low word only, and in the high word.
struct ChunkInfo {
    uint32_t and0, or0, and1, or1, flags, near0, near1, pad;
};
constexpr ChunkInfo NOTHING_FOUND{~0u, 0u, ~0u, 0u, 0u, ~0u, ~0u, 0u};

__device__ __forceinline__ uint32_t map_key(uint32_t v, RadixMap m)
{
    return v ^ ((uint32_t)((int32_t)v >> 31) & m.f) ^ m.x;
}
__device__ __forceinline__ uint32_t unmap_key(uint32_t u, RadixMap m)
{
    const uint32_t v = u ^ m.x;
    return v ^ ((uint32_t)((int32_t)v >> 31) & m.f);
}

// An element: hi is the key (or the high word of a 64-bit key), lo the value
// (or the low word); keys alone leave lo unused.
struct Elem {
    uint32_t hi, lo;
};

template <int KIND> __device__ __forceinline__ Elem map_elem2(Elem e, const RadixArgs &a)
{
    Elem r = e;
    if constexpr (KIND == RADIX_KEYS64) {
        const uint32_t s = (uint32_t)((int32_t)e.hi >> 31);
        r.hi = e.hi ^ (s & a.map.f) ^ a.map.x;
        r.lo = e.lo ^ (s & a.fl);
    } else {
        r.hi = map_key(e.hi, a.map);
        if constexpr (KIND == RADIX_PAIRS)
            r.lo = e.lo ^ 0x80000000u;
    }
    return r;
}
template <int KIND> __device__ __forceinline__ Elem unmap_elem2(Elem e, const RadixArgs &a)
{
    Elem r = e;
    if constexpr (KIND == RADIX_KEYS64) {
        const uint32_t v = e.hi ^ a.map.x;
        const uint32_t s = (uint32_t)((int32_t)v >> 31);
        r.hi = v ^ (s & a.map.f);
        r.lo = e.lo ^ (s & a.fl);
    } else {
        r.hi = unmap_key(e.hi, a.map);
        if constexpr (KIND == RADIX_PAIRS)
            r.lo = e.lo ^ 0x80000000u;
    }
    return r;
}

// Element i of buffer b as stored (the 64-bit kind's caller arrays are
// packed; its intermediate buffers are two word arrays).
template <int KIND> __device__ __forceinline__ Elem load_raw(const RadixArgs &a, int b, int64_t i)
{
    Elem e{0, 0};
    if constexpr (KIND == RADIX_KEYS64) {
        if (b == B_IN || b == B_OUT) {
            const uint64_t q = ((const uint64_t *)a.k[b])[i];
            e.lo = (uint32_t)q;
            e.hi = (uint32_t)(q >> 32);
            return e;
        }
    }
    e.hi = a.k[b][i];
    if constexpr (KIND == RADIX_PAIRS || KIND == RADIX_KEYS64)
        e.lo = a.v[b][i];
    return e;
}
template <int KIND>
__device__ __forceinline__ void store_raw(const RadixArgs &a, int b, int64_t i, Elem e)
{
    if constexpr (KIND == RADIX_KEYS64) {
        if (b == B_IN || b == B_OUT) {
            ((uint2 *)a.k[b])[i] = make_uint2(e.lo, e.hi);
            return;
        }
    }
    a.k[b][i] = e.hi;
    if constexpr (KIND == RADIX_PAIRS || KIND == RADIX_KEYS64)
        a.v[b][i] = e.lo;
}

// ------------------------------------------------------------------- count

__device__ __forceinline__ uint32_t wave_and(uint32_t x)
{
#pragma unroll
    for (int d = 1; d < 64; d *= 2)
        x &= (uint32_t)__shfl_xor((int)x, d);
    return x;
}
__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
#pragma unroll
    for (int d = 1; d < 64; d *= 2)
        x |= (uint32_t)__shfl_xor((int)x, d);
    return x;
}

__device__ __forceinline__ uint32_t wave_min(uint32_t x)
{
#pragma unroll
    for (int d = 1; d < 64; d *= 2)
        x = min(x, (uint32_t)__shfl_xor((int)x, d));
    return x;
}
// (Keys alone have no low word, and no digits to leave out.)
__device__ __forceinline__ ChunkInfo wave_info(ChunkInfo f, bool two)
{
    f.and1 = wave_and(f.and1);
    f.or1 = wave_or(f.or1);
    f.flags = wave_or(f.flags);
    if (two) {
        f.and0 = wave_and(f.and0);
        f.or0 = wave_or(f.or0);
        f.near0 = wave_min(f.near0);
        f.near1 = wave_min(f.near1);
    }
    return f;
}
__device__ __forceinline__ void add_info(ChunkInfo &f, const ChunkInfo &g)
{
    f.and0 &= g.and0;
    f.or0 |= g.or0;
    f.and1 &= g.and1;
    f.or1 |= g.or1;
    f.flags |= g.flags;
    f.near0 = min(f.near0, g.near0);
    f.near1 = min(f.near1, g.near1);
}

// Digit d of the workgroup's histogram so far (d < 256).
__device__ __forceinline__ uint32_t hist_sum(const uint32_t *hist, int d)
{
    uint32_t s = 0;
    const uint4 *q = (const uint4 *)(hist + d * COPIES);
#pragma unroll
    for (int c = 0; c < COPIES / 4; ++c)
        s += q[c].x + q[c].y + q[c].z + q[c].w;
    return s;
}

typedef uint32_t Words __attribute__((ext_vector_type(4)));

// A whole tile from element i0 on for the first count; the caller's arrays are
// 16-byte aligned, and `more` if an element follows the tile.  A lane takes the
// consecutive elements of one load, so that all but one of their comparisons
// with the element after need no other lane: the first count reads 2^28 keys
// in 0.21 ms, as the others do (0.27 with one key to a lane and load).
template <int KIND, int T>
__device__ __forceinline__ void count_first_tile(const RadixArgs &a, int64_t i0, bool more,
                                                 ChunkInfo &f, uint32_t *hist)
{
    constexpr bool TWO = KIND == RADIX_PAIRS || KIND == RADIX_KEYS64;
    constexpr bool STREAM = KIND == RADIX_KEYS && T >= 16384;
    constexpr int NE = KIND == RADIX_KEYS64 ? 2 : 4;  // elements of a load
    constexpr int LOADS = T / (NE * COUNT_NT);
    constexpr int UN = LOADS < (KIND == RADIX_PAIRS ? 4 : 8) ? LOADS : KIND == RADIX_PAIRS ? 4 : 8;
    const int lane = lane_id(), copy = lane & (COPIES - 1);
    const uint32_t *pk = a.k[B_IN] + (KIND == RADIX_KEYS64 ? 2 : 1) * i0;
    const uint32_t *pv = KIND == RADIX_PAIRS ? a.v[B_IN] + i0 : nullptr;
    bool gt = false, lt = false, vgt = false;
#pragma unroll 1
    for (int u0 = 0; u0 < LOADS; u0 += UN) {
        Words q[UN], v[UN];
        Elem after[UN];  // the element after the wave's
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int at = (u0 + u) * COUNT_NT + threadIdx.x;
            const Words *w = (const Words *)pk + at;
            q[u] = STREAM ? __builtin_nontemporal_load(w) : *w;
            if constexpr (KIND == RADIX_PAIRS)
                v[u] = ((const Words *)pv)[at];
            const int e = NE * ((u0 + u) * COUNT_NT + (int)(threadIdx.x & ~63u) + 64);
            after[u] = load_raw<KIND>(a, B_IN, i0 + (e < T || more ? e : T - 1));
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            Elem k[NE + 1];
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                if constexpr (KIND == RADIX_KEYS64)
                    k[j] = Elem{q[u][2 * j + 1], q[u][2 * j]};
                else if constexpr (KIND == RADIX_PAIRS)
                    k[j] = Elem{q[u][j], v[u][j]};
                else
                    k[j] = Elem{q[u][j], 0};
                k[j] = map_elem2<KIND>(k[j], a);
            }
            after[u] = map_elem2<KIND>(after[u], a);
            k[NE].hi = (uint32_t)__shfl_down((int)k[0].hi, 1);
            k[NE].hi = lane == 63 ? after[u].hi : k[NE].hi;
            if constexpr (TWO) {
                k[NE].lo = (uint32_t)__shfl_down((int)k[0].lo, 1);
                k[NE].lo = lane == 63 ? after[u].lo : k[NE].lo;
            }
            // the array's last element has none after it
            const bool end = !more && u0 + u == LOADS - 1 && threadIdx.x == COUNT_NT - 1;
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                bool g = k[j].hi > k[j + 1].hi;
                // a stable sort may reverse only where no two keys are equal
                bool l = KIND == RADIX_BY_KEY ? k[j].hi <= k[j + 1].hi : k[j].hi < k[j + 1].hi;
                if constexpr (TWO) {
                    // (one compare each: by words the flags are kept in vector registers)
                    const uint64_t x = (uint64_t)k[j].hi << 32 | k[j].lo;
                    const uint64_t y = (uint64_t)k[j + 1].hi << 32 | k[j + 1].lo;
                    g = x > y;
                    l = x < y;
                    const bool eq = k[j].hi == k[j + 1].hi;
                    f.near0 = min(f.near0, eq ? (k[j].lo ^ k[j + 1].lo) - 1 : ~0u);
                    f.near1 = min(f.near1, (k[j].hi ^ k[j + 1].hi) - 1);
                    if constexpr (KIND == RADIX_PAIRS)
                        vgt = vgt || k[j].lo > k[j + 1].lo;
                    f.and0 &= k[j].lo;
                    f.or0 |= k[j].lo;
                }
                gt = gt || g;
                lt = lt || (l && !(j == NE - 1 && end));
                f.and1 &= k[j].hi;
                f.or1 |= k[j].hi;
                const uint32_t w = TWO ? k[j].lo : k[j].hi;
                atomicAdd(&hist[(w & 255) * COPIES + copy], 1u);
            }
        }
    }
    f.flags |= (gt ? NOT_ASCENDING : 0) | (lt ? NOT_DESCENDING : 0) |
               (vgt ? VALUES_NOT_ASCENDING : 0);
}

// Pass 0: the histogram of digit 0 and what the plan needs to know.
template <int KIND, int T>
__global__ __launch_bounds__(COUNT_NT) void radix_count_first(RadixArgs a)
{
    __shared__ __align__(16) uint32_t hist[RADIX * COPIES];
    __shared__ ChunkInfo part[COUNT_NT / 64];
    for (int i = threadIdx.x; i < RADIX * COPIES; i += COUNT_NT)
        hist[i] = 0;
    const int lane = lane_id();
    ChunkInfo f = NOTHING_FOUND;
    // rows of 64 x UN consecutive elements per wave; lane l of row r holds
    // element 64 r + l, and the next element comes from the next lane
    constexpr int UN = KIND == RADIX_KEYS ? 8 : 4;
    constexpr int STEP = COUNT_NT * UN;
    const bool wide = (((uintptr_t)a.k[B_IN] | (KIND == RADIX_PAIRS ? (uintptr_t)a.v[B_IN] : 0)) &
                       15) == 0;
    const int64_t t0 = (int64_t)blockIdx.x << a.per_log2;
    const int64_t t1 = min(t0 + ((int64_t)1 << a.per_log2), a.tiles);
    for (int64_t tile = t0; tile < t1; ++tile) {
        __syncthreads();
        if (threadIdx.x < RADIX)
            a.rows[tile * RADIX + threadIdx.x] = hist_sum(hist, threadIdx.x);
        __syncthreads();
        const int64_t hi = (tile + 1) * T < a.n ? (tile + 1) * T : a.n;
        if (wide && hi - tile * T == T) {
            count_first_tile<KIND, T>(a, tile * T, hi < a.n, f, hist);
            continue;
        }
        for (int64_t base = tile * T + (int64_t)(threadIdx.x / 64) * (64 * UN); base < hi;
             base += STEP) {
            Elem e[UN + 1];
#pragma unroll
            for (int r = 0; r <= UN; ++r) {
                const int64_t i = base + r * 64 + (r < UN ? lane : 0);
                e[r] = load_raw<KIND>(a, B_IN, i < a.n ? i : a.n - 1);
            }
#pragma unroll
            for (int r = 0; r <= UN; ++r)
                e[r] = map_elem2<KIND>(e[r], a);
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const int64_t i = base + r * 64 + lane;
                // the element after this one: the next lane's, or the next row's first
                Elem nx;
                nx.hi = (uint32_t)__shfl_down((int)e[r].hi, 1);
                const uint32_t nh = (uint32_t)__builtin_amdgcn_readfirstlane((int)e[r + 1].hi);
                nx.hi = lane == 63 ? nh : nx.hi;
                bool gt = e[r].hi > nx.hi, lt = e[r].hi < nx.hi;
                if constexpr (KIND == RADIX_PAIRS || KIND == RADIX_KEYS64) {
                    nx.lo = (uint32_t)__shfl_down((int)e[r].lo, 1);
                    const uint32_t nl = (uint32_t)__builtin_amdgcn_readfirstlane((int)e[r + 1].lo);
                    nx.lo = lane == 63 ? nl : nx.lo;
                    const bool eq = e[r].hi == nx.hi;
                    gt = gt || (eq && e[r].lo > nx.lo);
                    lt = lt || (eq && e[r].lo < nx.lo);
                    // past the array's end an element meets itself
                    f.near0 = min(f.near0, eq ? (e[r].lo ^ nx.lo) - 1 : ~0u);
                    f.near1 = min(f.near1, (e[r].hi ^ nx.hi) - 1);
                    if (KIND == RADIX_PAIRS && i + 1 < a.n && e[r].lo > nx.lo)
                        f.flags |= VALUES_NOT_ASCENDING;
                }
                // a stable sort may reverse only where no two keys are equal
                if constexpr (KIND == RADIX_BY_KEY)
                    lt = e[r].hi <= nx.hi;
                if (i + 1 < a.n)
                    f.flags |= (gt ? NOT_ASCENDING : 0) | (lt ? NOT_DESCENDING : 0);
                if (i < hi) {
                    f.and1 &= e[r].hi;
                    f.or1 |= e[r].hi;
                    if constexpr (KIND == RADIX_PAIRS || KIND == RADIX_KEYS64) {
                        f.and0 &= e[r].lo;
                        f.or0 |= e[r].lo;
                    }
                    const uint32_t w =
                        (KIND == RADIX_PAIRS || KIND == RADIX_KEYS64) ? e[r].lo : e[r].hi;
                    atomicAdd(&hist[(w & 255) * COPIES + (lane & (COPIES - 1))], 1u);
                }
            }
        }
    }
    f = wave_info(f, KIND == RADIX_PAIRS || KIND == RADIX_KEYS64);
    if (lane == 0)
        part[threadIdx.x / 64] = f;
    __syncthreads();
    if (threadIdx.x < RADIX)
        a.counts[(int64_t)blockIdx.x * RADIX + threadIdx.x] = hist_sum(hist, threadIdx.x);
    if (threadIdx.x == 0) {
        for (int w = 1; w < COUNT_NT / 64; ++w)
            add_info(f, part[w]);
        ((ChunkInfo *)a.info)[blockIdx.x] = f;
    }
}

// Later passes: the histogram of one digit of one word array.
template <int KIND, int T>
__global__ __launch_bounds__(COUNT_NT) void radix_count(RadixArgs a, int pass)
{
    const Step st = step_of(a, pass);
    if (st.mode != STEP_SCATTER)
        return;
    __shared__ __align__(16) uint32_t hist[RADIX * COPIES];
    for (int i = threadIdx.x; i < RADIX * COPIES; i += COUNT_NT)
        hist[i] = 0;
    const int copy = threadIdx.x & (COPIES - 1);
    constexpr bool TWO = KIND == RADIX_PAIRS || KIND == RADIX_KEYS64;
    // The tiles of keys alone are this large from 2^27 keys, where reading past
    // the memory-side cache pays (2^27 keys 1.71 -> 1.54 ms, 2^28 3.40 -> 3.21;
    // 2^25 keys 0.397 -> 0.413, and two-word elements do not care).
    constexpr bool STREAM = KIND == RADIX_KEYS && T >= 16384;
    const bool low = TWO && pass < 4;
    const int shift = 8 * (pass & 3);
    const uint32_t *p = low ? a.v[st.src] : a.k[st.src];
    // st.first: the caller's array, unmapped (the passes before were skipped)
    const bool packed = KIND == RADIX_KEYS64 && st.first;
    const bool wide = ((uintptr_t)(packed ? a.k[st.src] : p) & 15) == 0;
    auto add = [&](uint32_t w) { atomicAdd(&hist[((w >> shift) & 255) * COPIES + copy], 1u); };
    const int64_t t0 = (int64_t)blockIdx.x << a.per_log2;
    const int64_t t1 = min(t0 + ((int64_t)1 << a.per_log2), a.tiles);
    for (int64_t tile = t0; tile < t1; ++tile) {
        const int64_t lo = tile * T, hi = lo + T < a.n ? lo + T : a.n;
        constexpr int UN = T / (4 * COUNT_NT);
        Words q[UN];
        const bool full = wide && hi - lo == T;
        const Words *w = (const Words *)(packed ? a.k[st.src] + 2 * lo : p + lo) + threadIdx.x;
        if (full) {
#pragma unroll
            for (int u = 0; u < UN; ++u)
                q[u] = STREAM ? __builtin_nontemporal_load(w + u * COUNT_NT) : w[u * COUNT_NT];
        }
        __syncthreads();
        if (threadIdx.x < RADIX)
            a.rows[tile * RADIX + threadIdx.x] = hist_sum(hist, threadIdx.x);
        __syncthreads();
        if (full && !st.first) {
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    add(q[u][j]);
        } else if (full && !packed) {
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    add(KIND == RADIX_PAIRS && low ? q[u][j] ^ 0x80000000u
                                                   : map_key(q[u][j], a.map));
        } else if (full) {
            // two elements to a load: the tile's second half follows
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    if (h)
                        q[u] = w[(UN + u) * COUNT_NT];
                }
#pragma unroll
                for (int u = 0; u < UN; ++u)
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        const Elem e = map_elem2<KIND>(Elem{q[u][j + 1], q[u][j]}, a);
                        add(low ? e.lo : e.hi);
                    }
            }
        } else {
            for (int64_t i = lo + threadIdx.x; i < hi; i += COUNT_NT) {
                uint32_t x;
                if (st.first) {
                    const Elem e = map_elem2<KIND>(load_raw<KIND>(a, st.src, i), a);
                    x = low ? e.lo : e.hi;
                } else {
                    x = p[i];
                }
                add(x);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < RADIX)
        a.counts[(int64_t)blockIdx.x * RADIX + threadIdx.x] = hist_sum(hist, threadIdx.x);
}

// Orders one wave's LDS operations before those after, also where they go through
// other types: the hardware completes them in order, so only the compiler has to
// keep them so.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// -------------------------------------------------------------------- scan

// Inclusive prefix sum over the lanes of a wave (row shifts, then the row
// sums broadcast to the following rows).
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false); // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false); // row_bcast:31
    return x;
}

// The steps of the sort from what the chunks found, by one workgroup of at
// most 512 threads (ctl: where they go, in LDS or memory).
__device__ void make_plan(const RadixArgs &a, int passes, bool two, bool keys64, bool inplace,
                          Ctl *ctl)
{
    __shared__ ChunkInfo part[8];
    __shared__ uint32_t same[8];
    ChunkInfo f = NOTHING_FOUND;
    const ChunkInfo *info = (const ChunkInfo *)a.info;
    for (int c = threadIdx.x; c < a.chunks; c += blockDim.x)
        add_info(f, info[c]);
    f = wave_info(f, two);
    if (lane_id() == 0)
        part[threadIdx.x / 64] = f;
    if (threadIdx.x < 8) {  // sum of the runs' counts
        uint32_t c = 0;
        if (a.sample_pairs)
            for (int r = 0; r < a.sample_runs; ++r)
                c += a.sample_pairs[r * 8 + threadIdx.x];
        same[threadIdx.x] = c;
    }
    __syncthreads();
    if (threadIdx.x != 0)
        return;
    for (int w = 1; w < (int)blockDim.x / 64; ++w)
        add_info(f, part[w]);
    plan_sort(Found{f.flags, f.and0 ^ f.or0, f.and1 ^ f.or1, f.near0, f.near1, same,
                    a.sample_pairs ? a.sample_runs : 0, a.n},
              passes, two, keys64, inplace, ctl);
}

// Workgroup g: the exclusive prefixes of the counts of digits 16 g .. 16 g +
// 15 over the chunks, in place, and the digits' totals; thread t walks digit
// t mod 16 over the (t / 16)th part of the chunks.  In pass 0 one more
// workgroup makes the plan.
__global__ __launch_bounds__(512) void radix_scan(RadixArgs a, int pass, int passes, int two,
                                                  int keys64, int inplace)
{
    if (blockIdx.x == RADIX / 16) {
        make_plan(a, passes, two != 0, keys64 != 0, inplace != 0, (Ctl *)a.ctl);
        return;
    }
    if ((pass > 0 || a.round) && step_of(a, pass).mode != STEP_SCATTER)
        return;
    __shared__ uint32_t sum[32][16];
    const int d = threadIdx.x & 15, q = threadIdx.x >> 4;
    constexpr int PER = MAX_CHUNKS / 32;
    uint32_t *col = a.counts + blockIdx.x * 16 + d;
    uint32_t v[PER], s = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = q * PER + i;
        v[i] = c < a.chunks ? col[c * RADIX] : 0;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        s += v[i];
    sum[q][d] = s;
    __syncthreads();
    uint32_t ex = 0, all = 0;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        ex += i < q ? sum[i][d] : 0;
        all += sum[i][d];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = q * PER + i;
        if (c < a.chunks)
            col[c * RADIX] = ex;
        ex += v[i];
    }
    if (q == 0)
        a.totals[blockIdx.x * 16 + d] = all;
}

// ---------------------------------------------- top digits and the finish
//
// Elements of two words rarely need all their eight digits: once the top ones
// tell nearly all of them apart, the few that are left alike stand next to
// each other and are ordered where they are.  How many digits that takes is
// estimated from a sample sorted in runs:
// neighbours that are equal in the top digits and different below are what a
// shorter key would leave alike.  The finish checks its own work, so the
// estimate only costs time where it is wrong: the second round then makes
// every pass that is needed.  Pairs of 2^26 uniform keys and random values take
// four passes and the finish, 1.80 ms, for eight passes 2.48 and the merge sort
// 2.62; 5e7 doubles five and 1.61 ms for 2.19 by the merge sort.

// Sample element j comes from position SplitMix64(j) * n / 2^64.  (From the
// j-th of equal parts of the input it would not do: in presorted input the
// elements that are alike stand side by side and would never meet.)
//
// A workgroup draws a run, sorts it and counts its neighbours by the highest
// digit in which they differ (equal neighbours are no pair to be told apart; the
// top digit is never left out, and its count gives way to that of the elements
// that equal the one after next).
// It runs after the first count, whose flags say whether the plan will ask:
// 2^24 pairs with index values 341 -> 304 us, 2^26 1184 -> 1130.  Drawn by a
// launch over the whole chip, sorted by the block sort and counted by a third
// launch, it took 15 us more for 5e7 doubles, 6 us less for 2^24 pairs with
// random values.
template <int KIND> __global__ __launch_bounds__(SAMPLE_LEN / 8) void radix_sample(RadixArgs a)
{
    constexpr int R = 8, NT = SAMPLE_LEN / R;
    __shared__ __attribute__((aligned(16))) int64_t S[LdsSkew<int64_t>::size(R * NT)];
    __shared__ uint32_t c[8], flags;
    const LdsSkew<int64_t> Z{S, 0};
    if (threadIdx.x < 8)
        c[threadIdx.x] = 0;
    if (threadIdx.x == 8)
        flags = 0;
    __syncthreads();
    uint32_t f = 0;
    for (int i = threadIdx.x; i < a.chunks; i += NT)
        f |= ((const ChunkInfo *)a.info)[i].flags;
    if (f)
        atomicOr(&flags, f);
    __syncthreads();
    if (!sample_matters(flags, KIND == RADIX_KEYS64))
        return;
    int64_t v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        uint64_t z = ((uint64_t)blockIdx.x * SAMPLE_LEN + NT * j + threadIdx.x + 1) *
                     0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        const int64_t i = (int64_t)__umul64hi(z ^ (z >> 31), (uint64_t)a.n);
        const Elem e = map_elem2<KIND>(load_raw<KIND>(a, B_IN, i), a);
        // signed order, as the block sort compares
        v[j] = (int64_t)(((uint64_t)(e.hi ^ 0x80000000u) << 32) | e.lo);
    }
    sort_tile_core<R, NT, int64_t, 0>(S, v, threadIdx.x, 6, 4);
    uint32_t count[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = threadIdx.x + NT * j;
        const uint64_t d = i + 1 < SAMPLE_LEN ? (uint64_t)(Z[i] ^ Z[i + 1]) : 0;
        const int t = d ? (63 - __clzll((long long)d)) >> 3 : 8;
        const bool third = i + 2 < SAMPLE_LEN && Z[i] == Z[i + 2];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            count[q] += __popcll(__builtin_amdgcn_ballot_w64(q == 7 ? third : t == q));
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (lane_id() == q)
            atomicAdd(&c[q], count[q]);
    __syncthreads();
    if (threadIdx.x < 8)
        a.sample_pairs[blockIdx.x * 8 + threadIdx.x] = c[threadIdx.x];
}

// Orders the groups that the first round left alike, in the output.  A wave
// looks at windows of 64 consecutive elements, 32 apart; a group belongs to the
// window in whose first half it starts.  The groups that end inside their
// window (all of up to 33 elements) are sorted in the lanes, all at once, by
// odd-even transposition, and every lane stores its own element.  A longer
// group is read through and, if it is out of order, put on a list for
// radix_groups; past GROUP_MAX elements, or past the end of the list, the
// sort goes to the second round.  What others look at while an element moves,
// the common digits of its group, does not change.  Bound by its instructions
// (5e7 doubles 0.22 ms: 122 VALU and 20 LDS operations an element, for a read of
// 0.09 ms; 2^28 uniform pairs, 12 % of them alike: 2.5 ms when the first lane of
// each group read it through in memory, now 1.0).
constexpr int GROUP_MAX = 16384;    // elements of a listed group: the LDS of one workgroup
constexpr int GROUPS_MAX = 131072;  // listed groups

template <int KIND> __device__ __forceinline__ uint64_t finish_elem(const RadixArgs &a, int64_t i)
{
    const Elem e = map_elem2<KIND>(load_raw<KIND>(a, B_OUT, i), a);
    return ((uint64_t)e.hi << 32) | e.lo;
}
template <int KIND>
__device__ __forceinline__ void finish_store(const RadixArgs &a, int64_t i, uint64_t x)
{
    store_raw<KIND>(a, B_OUT, i,
                    unmap_elem2<KIND>(Elem{(uint32_t)(x >> 32), (uint32_t)x}, a));
}

template <int KIND> __global__ __launch_bounds__(256) void radix_finish(RadixArgs a)
{
    Ctl *ctl = (Ctl *)a.ctl;
    const int shift = 8 * (int)ctl->drop;
    if (shift == 0)
        return;
    const int lane = lane_id();
    constexpr int ROWS = 8;  // of 64 elements, to a wave
    const int64_t w0 = ((int64_t)blockIdx.x * 4 + threadIdx.x / 64) * (64 * ROWS);
    if (w0 >= a.n)
        return;
    const auto at = [&](int64_t i) {
        return finish_elem<KIND>(a, i < 0 ? 0 : i < a.n ? i : a.n - 1);
    };
    uint64_t prior = at(w0 - 64 + lane), cur = at(w0 + lane), then = at(w0 + 64 + lane);
    // lane h: the group that window h lists (one at most), none at length 0
    int64_t list_at = 0;
    int list_len = 0;
#pragma unroll 1
    for (int h = 0; h < 2 * ROWS; ++h) {
        const int64_t b = w0 + 32 * h, i = b + lane;
        if (b >= a.n)
            break;
        // the window: row `cur`, or its second half and the next row's first
        uint64_t x = cur, prev, next;
        if (h & 1) {
            const uint64_t m = lane < 32 ? then : cur;  // what lane ^ 32 asks for
            x = __shfl_xor((unsigned long long)m, 32);
            prev = __shfl((unsigned long long)cur, 31);
            next = __shfl((unsigned long long)then, 32);
            prior = cur;
            cur = then;
            then = at(b + 96 + lane);
        } else {
            prev = __shfl((unsigned long long)prior, 63);
            next = __shfl((unsigned long long)then, 0);
        }
        const uint64_t up = __shfl_up((unsigned long long)x, 1);
        const uint64_t down = __shfl_down((unsigned long long)x, 1);
        prev = lane == 0 ? prev : up;
        next = lane == 63 ? next : down;
        const bool eqn = i + 1 < a.n && (x >> shift) == (next >> shift);
        const bool eqp = i > 0 && i < a.n && (x >> shift) == (prev >> shift);
        const bool wrong = eqn && x > next;
        const uint64_t link = __ballot(eqn), before = __ballot(eqp);
        // in order, and no group runs on past the window (where it may not be)
        if (__ballot(wrong) == 0 && !(link >> 63))
            continue;
        // this lane's group inside the window: lanes start .. last
        const uint64_t heads = ~(link << 1) | 1;  // no link from the lane below
        const int start = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
        const uint64_t ends = ~(link >> lane);    // zero: links to the last lane and on
        const int end = ends ? lane + __ffsll((unsigned long long)ends) - 1 : 64;
        const int last = end < 63 ? end : 63;
        const bool enters = start == 0 && (before & 1), leaves = last == 63 && (link >> 63);
        const bool own = start < 32 && !enters;
        const bool inside = own && !leaves && last > start;
        const uint64_t x0 = x;
        for (int round = 0;; ++round) {
            const bool low = ((lane - start + round) & 1) == 0;  // lower lane of its pair
            const int other = low ? lane + 1 : lane - 1;
            const uint64_t y = __shfl((unsigned long long)x, other & 63);
            if (inside && other >= start && other <= last && (low ? y < x : x < y))
                x = y;
            const uint64_t above = __shfl_down((unsigned long long)x, 1);
            if (__ballot(inside && lane < last && x > above) == 0)
                break;
        }
        if (inside && x != x0)
            finish_store<KIND>(a, i, x);

        const uint64_t leaving = __ballot(own && leaves);
        if (leaving) {  // one group at most: read it through
            const int s0 = __ffsll((unsigned long long)leaving) - 1;
            const uint64_t digits = (uint64_t)__shfl((unsigned long long)x0, 63) >> shift;
            bool order = __ballot(wrong && lane >= s0) == 0;
            int64_t pos = b + 64;
            uint64_t tail = __shfl((unsigned long long)x0, 63);
            int more = 64;
            // some way past GROUP_MAX, where the windows below see for themselves
            while (more == 64 && pos - (b + s0) <= GROUP_MAX + 256) {
                const uint64_t y = at(pos + lane);
                const uint64_t in = __ballot(pos + lane < a.n && (y >> shift) == digits);
                more = ~in ? __ffsll((unsigned long long)~in) - 1 : 64;
                const uint64_t under = __shfl_up((unsigned long long)y, 1);
                order = order && __ballot(lane < more && (lane == 0 ? tail : under) > y) == 0;
                tail = __shfl((unsigned long long)y, 63);
                pos += more;
            }
            const int64_t len = pos - (b + s0);
            if (!order) {
                if (more == 64 || len > GROUP_MAX) {
                    if (lane == 0)
                        atomicOr(&ctl->again, 1u);
                } else if (lane == h) {
                    list_at = b + s0;
                    list_len = (int)len;
                }
            }
        }
        // out of order in a group that started before: its own window's
        // reader has seen it, unless it started too far back
        if (__ballot(enters && wrong && lane < 32) && !ctl->again) {
            const uint64_t digits = (uint64_t)__shfl((unsigned long long)x0, 0) >> shift;
            int64_t pos = b - 1;
            while (pos >= 0 && b - pos <= GROUP_MAX &&
                   __ballot(pos - lane < 0 || (at(pos - lane) >> shift) != digits) == 0)
                pos -= 64;
            if (b - pos > GROUP_MAX && lane == 0)
                atomicOr(&ctl->again, 1u);
        }
    }
    // one place in the list for all the wave's groups: an atomic for each, all on
    // one counter, took 1.6 of 2.8 ms with 58,000 groups
    const uint64_t listed = __ballot(list_len != 0);
    if (listed == 0)
        return;
    uint32_t g = 0;
    if (lane == 0)
        g = atomicAdd(&ctl->groups, (uint32_t)__popcll(listed));
    g = (uint32_t)__builtin_amdgcn_readfirstlane((int)g) +
        (uint32_t)__popcll(listed & ((1ull << lane) - 1));
    if (list_len != 0) {
        if (g < GROUPS_MAX)
            a.groups[g] = make_longlong2(list_at, list_len);
        else
            atomicOr(&ctl->again, 1u);
    }
}

// A listed group of at most 64 ROWS elements, by one wave: every element's
// position is the number of elements before it, counted against each in turn.
template <int KIND, int ROWS>
__device__ __forceinline__ void wave_group(const RadixArgs &a, int64_t i0, int len)
{
    const int lane = lane_id();
    uint64_t x[ROWS];
    int at[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = 64 * r + lane;
        x[r] = finish_elem<KIND>(a, i0 + (i < len ? i : 0));
        at[r] = 0;
    }
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
        const int m = len - 64 * q < 64 ? len - 64 * q : 64;
        for (int j = 0; j < m; ++j) {  // element 64 q + j; equal ones keep their order
            const uint64_t y =
                (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x[q] >> 32), j) << 32 |
                (uint32_t)__builtin_amdgcn_readlane((int)x[q], j);
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
                at[r] += r < q ? y < x[r] : r > q ? y <= x[r] : lane > j ? y <= x[r] : y < x[r];
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (64 * r + lane < len)
            finish_store<KIND>(a, i0 + at[r], x[r]);
}

// Part of a listed group, at most one padded tile of the block sort.
constexpr int GROUP_TILE = GROUP_MAX / 2;
template <int KIND>
__device__ __forceinline__ void tile_group(const RadixArgs &a, int64_t *S, int64_t i0, int len)
{
    constexpr int NT = 1024, R = GROUP_TILE / NT;
    const LdsSkew<int64_t> Z{S, 0};
    int64_t v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = (threadIdx.x >> 6) * (64 * R) + 64 * j + (threadIdx.x & 63);
        // unsigned order to signed; pads sort last
        v[j] = i < len ? (int64_t)(finish_elem<KIND>(a, i0 + i) ^ (1ull << 63))
                       : Traits<int64_t>::kMax;
    }
    sort_tile_core<R, NT, int64_t, 0>(S, v, threadIdx.x, 6, 4);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = threadIdx.x + NT * j;
        if (i < len)
            finish_store<KIND>(a, i0 + i, (uint64_t)Z[i] ^ (1ull << 63));
    }
    __syncthreads();
}

// A group of two sorted parts: every element's position is its own in its part
// and its rank in the other.
template <int KIND>
__device__ __forceinline__ void merge_group(const RadixArgs &a, uint64_t *S, int64_t i0, int len)
{
    for (int i = threadIdx.x; i < len; i += 1024)
        S[i] = finish_elem<KIND>(a, i0 + i);
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += 1024) {
        const bool first = i < GROUP_TILE;
        const uint64_t x = S[i];
        int lo = first ? GROUP_TILE : 0, hi = first ? len : GROUP_TILE;
        while (lo < hi) {  // equal elements of the first part come first
            const int mid = (lo + hi) >> 1;
            const bool before = first ? S[mid] < x : S[mid] <= x;
            lo = before ? mid + 1 : lo;
            hi = before ? hi : mid;
        }
        finish_store<KIND>(a, i0 + i + lo - GROUP_TILE, x);
    }
    __syncthreads();
}

// Sorts the listed groups: a wave each those of up to WAVE_GROUP elements, then
// a workgroup each the others.  What the finish lists is mostly little more than
// half a window: 9,232 groups of about 40 pairs (2^27 pairs of mixture keys and
// random values, without two digits) took 810 us as padded tiles, now 26.
constexpr int WAVE_GROUP = 256;
template <int KIND> __global__ __launch_bounds__(1024) void radix_groups(RadixArgs a)
{
    const Ctl *ctl = (const Ctl *)a.ctl;
    if (ctl->drop == 0 || ctl->again)
        return;
    __shared__ __attribute__((aligned(16))) int64_t S[GROUP_MAX];
    static_assert(LdsSkew<int64_t>::size(GROUP_TILE) <= GROUP_MAX, "a tile fits");
    const uint32_t count = ctl->groups < GROUPS_MAX ? ctl->groups : GROUPS_MAX;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    for (uint32_t g = blockIdx.x * 16 + wave; g < count; g += gridDim.x * 16) {
        const int64_t i0 = a.groups[g].x;
        const int len = __builtin_amdgcn_readfirstlane((int)a.groups[g].y);
        if (len <= 64)
            wave_group<KIND, 1>(a, i0, len);
        else if (len <= WAVE_GROUP)
            wave_group<KIND, WAVE_GROUP / 64>(a, i0, len);
    }
    for (uint32_t g = blockIdx.x; g < count; g += gridDim.x) {
        const int64_t i0 = a.groups[g].x;
        const int len = (int)a.groups[g].y;
        if (len <= WAVE_GROUP)
            continue;
        for (int i = 0; i < len; i += GROUP_TILE)
            tile_group<KIND>(a, S, i0 + i, len - i < GROUP_TILE ? len - i : GROUP_TILE);
        if (len > GROUP_TILE)
            merge_group<KIND>(a, (uint64_t *)S, i0, len);
    }
}

// ----------------------------------------------------------------- scatter

// Mask of the lanes whose digit (8 bits at `shift`) equals this lane's.
__device__ __forceinline__ void match_digit(uint32_t d, uint32_t &lo, uint32_t &hi)
{
    lo = ~0u;
    hi = ~0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        // all ones where the bit is set; hidden from the optimizer, which
        // would otherwise compute the sign a second time by a shift
        int32_t t = __builtin_amdgcn_sbfe((int)d, b, 1);
        asm("" : "+v"(t));
        const uint64_t set = __builtin_amdgcn_ballot_w64(t != 0);
        // mask & ~(set ^ t): lanes whose bit equals this lane's
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)set, (uint32_t)t, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(set >> 32), (uint32_t)t, 0x90);
    }
}

// Copies the input (or reverses it); UN elements to a thread in flight, since
// the scatter's LDS leaves few waves on a CU.
template <int NT, int KIND, int UN>
__device__ __forceinline__ void copy_step(const RadixArgs &a, const Step &st)
{
    for (int64_t i0 = (int64_t)blockIdx.x * (NT * UN); i0 < a.n;
         i0 += (int64_t)gridDim.x * (NT * UN)) {
        Elem e[UN];
        uint64_t pay[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t i = i0 + u * NT + threadIdx.x;
            const int64_t c = i < a.n ? i : a.n - 1;
            e[u] = load_raw<KIND>(a, st.src, c);
            if constexpr (KIND == RADIX_BY_KEY)
                pay[u] = a.p[st.src][c];
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t i = i0 + u * NT + threadIdx.x;
            const int64_t o = st.mode == STEP_REVERSE ? a.n - 1 - i : i;
            if (st.first)
                e[u] = map_elem2<KIND>(e[u], a);
            if (st.last)
                e[u] = unmap_elem2<KIND>(e[u], a);
            if (i < a.n) {
                store_raw<KIND>(a, st.dst, o, e[u]);
                if constexpr (KIND == RADIX_BY_KEY)
                    a.p[st.dst][o] = pay[u];
            }
        }
    }
}

// Where a scatter's output positions come from.  OF_SCAN: the scan launch.
// OF_TILES (one workgroup to a tile, at most FEW_TILES tiles): every workgroup
// adds up the tiles' counts itself, and in the first pass makes the plan.
// OF_CHUNKS: the chunks' counts likewise, 512 KB for a workgroup, more than the
// scan launch costs; the second round's passes do so, which hardly ever run,
// since a launch that returns at once still takes 1.5 us (2^24 pairs with index
// values 352 -> 341 us, 2^26 1197 -> 1184).
enum { OF_SCAN = 0, OF_TILES = 1, OF_CHUNKS = 2 };
template <int NT, int K, int KIND, int WAVES, int SUMS>
__global__ __launch_bounds__(NT, WAVES) void radix_scatter(RadixArgs a, int pass, int inplace)
{
    constexpr bool FEW = SUMS == OF_TILES;
    constexpr int T = NT * K;
    constexpr int NW = NT / 64;
    constexpr int B = 8;  // positions written out at a time
    constexpr bool TWO = KIND == RADIX_PAIRS || KIND == RADIX_KEYS64;
    // 64-bit payloads are exchanged as such, 32-bit words one after the other
    constexpr int XB = KIND == RADIX_BY_KEY ? 8 : 4;
    static_assert(T <= 65536 && K % B == 0, "16-bit tile positions");
    __shared__ __align__(16) unsigned char xraw[T * XB];
    __shared__ __align__(16) uint16_t cnt[NW][RADIX];  // keys of each digit per wave
    __shared__ __align__(16) uint16_t off[NW][RADIX];  // tile position of a wave's first such key
    __shared__ __align__(16) uint32_t gbase[RADIX];    // output index minus tile position
    __shared__ __align__(16) uint32_t gpre[RADIX];     // output index of the tile's first such key
    uint32_t *xch = (uint32_t *)xraw;

    Step st;
    if (FEW && pass == 0) {
        __shared__ Ctl plan;
        make_plan(a, 4, false, false, inplace != 0, &plan);
        __syncthreads();
        st = step_of(&plan, 0, 0);
        if (blockIdx.x == 0) {
            for (int i = threadIdx.x; i < (int)(sizeof(Ctl) / 4); i += NT)
                ((uint32_t *)a.ctl)[i] = ((const uint32_t *)&plan)[i];
        }
    } else {
        st = step_of(a, pass);
    }
    if (st.mode == STEP_SKIP)
        return;
    if (st.mode != STEP_SCATTER) {
        copy_step<NT, KIND, (K >= 32 ? 8 : 4)>(a, st);
        return;
    }
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int shift = 8 * (pass & 3);
    const bool low = TWO && pass < 4;  // the digit's word
    const bool packed_in = KIND == RADIX_KEYS64 && st.src == B_IN;
    const bool packed_out = KIND == RADIX_KEYS64 && st.dst == B_OUT;
    // w: the array of the word that holds the digit, s: the other word's
    const uint32_t *wsrc = low && !packed_in ? a.v[st.src] : a.k[st.src];
    const uint32_t *ssrc = low || packed_in ? a.k[st.src] : a.v[st.src];
    uint32_t *wdst = low ? a.v[st.dst] : a.k[st.dst];
    uint32_t *sdst = low ? a.k[st.dst] : a.v[st.dst];

    // An XCD's workgroups (every eighth one) walk one contiguous range of
    // tiles together, so that the lines two neighbouring tiles share are
    // completed in that XCD's L2.
    const int slots = FEW ? (int)a.tiles : (int)gridDim.x >> 3;
    const int64_t xcd = blockIdx.x & 7;
    const int64_t tile1 = FEW ? a.tiles : (xcd + 1) * a.tiles >> 3;
    int64_t tile = FEW ? (int64_t)blockIdx.x : (xcd * a.tiles >> 3) + (blockIdx.x >> 3);

    // thread t < 256: where digit t's region of the output starts (FEW: this
    // tile's part of it)
    uint32_t region = 0;
    // Keys alone may leave the first pass in any order within a digit: there
    // an LDS atomic per key takes the place of the ballots (2^28 keys 3.18 ->
    // 3.11 ms, 2^25 0.391 -> 0.374).  Lanes of one digit queue at its counter:
    // with half the keys in one digit the sort took 3.10 against 2.90 ms, with a
    // third of them it gained, so the line is at three eighths of the keys.
    // A ragged tile is ranked in order, which puts its pads last.
    __shared__ int spread;
    int chunk = FEW ? (int)tile : (int)(tile >> a.per_log2);  // the last one region counts to
    if constexpr (SUMS != OF_SCAN) {
        // thread d + 256 h: digit d over every (NT / 256)th tile (or chunk) from h
        constexpr int H = NT / RADIX, U = 16;
        const int rows = FEW ? (int)a.tiles : a.chunks;
        uint32_t *sums = xch;  // [h][digit]: all tiles', then the ones before
        uint32_t all = 0, mine = 0;
        for (int c0 = tid / RADIX; c0 < rows; c0 += U * H) {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[u] = c0 + u * H < rows
                           ? a.counts[(c0 + u * H) * RADIX + (tid & (RADIX - 1))]
                           : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                all += v[u];
                mine += c0 + u * H < chunk ? v[u] : 0;
            }
        }
        sums[tid] = all;
        sums[NT + tid] = mine;
        __syncthreads();
        if (tid < RADIX) {
            all = 0;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                all += sums[h * RADIX + tid];
                region += sums[NT + h * RADIX + tid];
            }
            gbase[tid] = all;
        }
        __syncthreads();
    }
    if (wave == 0) {
        const uint4 t = *(const uint4 *)((SUMS != OF_SCAN ? gbase : a.totals) + 4 * lane);
        const uint32_t s = t.x + t.y + t.z + t.w;
        const uint32_t ex = wave_inclusive(s) - s;
        *(uint4 *)&gpre[4 * lane] =
            make_uint4(ex, ex + t.x, ex + t.x + t.y, ex + t.x + t.y + t.z);
        if constexpr (KIND == RADIX_KEYS) {
            const uint32_t most = max(max(t.x, t.y), max(t.z, t.w));
            const bool heavy = __builtin_amdgcn_ballot_w64(most > 3 * (uint32_t)(a.n >> 3)) != 0;
            if (lane == 0)
                spread = st.first && !heavy;
        }
    }
    __syncthreads();
    if (tid < RADIX)
        region += gpre[tid];
    const bool loose = KIND == RADIX_KEYS && __builtin_amdgcn_readfirstlane(spread) != 0;

    // Loads of a tile's words through buffer resources: they end at the
    // array's last element (zeros past it) and take one lane offset and
    // constant row offsets.  hi: which word of a packed array.
    const auto load_words = [&](const uint32_t *p, bool packed, bool hi, int64_t base, int e0,
                                uint32_t(&x)[K]) {
        const uint32_t valid = a.n - base < T ? (uint32_t)(a.n - base) : (uint32_t)T;
        if (packed) {
            const __amdgpu_buffer_rsrc_t r = raw_rsrc(p + 2 * base, 8u * valid);
            const int h = hi ? 4 : 0;
#pragma unroll
            for (int k = 0; k < K; ++k)
                x[k] = __builtin_amdgcn_raw_buffer_load_b32(r, 8 * e0 + 8 * 64 * k, h, 0);
        } else {
            // streamed (nt): the L2 is for the lines being written
            const __amdgpu_buffer_rsrc_t r = raw_rsrc(p + base, 4u * valid);
#pragma unroll
            for (int k = 0; k < K; ++k)
                x[k] = __builtin_amdgcn_raw_buffer_load_b32(r, 4 * e0 + 4 * 64 * k, 0, 2);
        }
    };
    uint32_t w[K];
    for (; tile < tile1; tile += slots) {
        const int64_t base = tile * T;
        const int cnt_valid = a.n - base < T ? (int)(a.n - base) : T;
        if constexpr (SUMS == OF_CHUNKS) {
            for (; chunk < (int)(tile >> a.per_log2); ++chunk)
                if (tid < RADIX)
                    region += a.counts[chunk * RADIX + tid];
        }
        uint32_t first = region;
        if (SUMS == OF_CHUNKS && tid < RADIX)
            first += a.rows[tile * RADIX + tid];
        if (SUMS == OF_SCAN && tid < RADIX)
            first += a.rows[tile * RADIX + tid] + a.counts[(tile >> a.per_log2) * RADIX + tid];
        int t0 = tid;
        asm("" : "+v"(t0));  // keeps the row offsets out of registers held across tiles
        const int e0 = wave * (64 * K) + (t0 & 63);
        load_words(wsrc, packed_in, !low, base, e0, w);
        if (st.first) {
            if (KIND == RADIX_KEYS64 && low) {  // the low word's map follows the sign
                uint32_t h[K];
                load_words(ssrc, packed_in, true, base, e0, h);
#pragma unroll
                for (int k = 0; k < K; ++k)
                    w[k] = map_elem2<KIND>(Elem{h[k], w[k]}, a).lo;
            } else {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const Elem e = map_elem2<KIND>(Elem{w[k], w[k]}, a);
                    w[k] = low ? e.lo : e.hi;
                }
            }
        }
        // pads take the last positions of the tile: the largest digit,
        // after every real element in tile order
        if (cnt_valid != T) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (e0 + k * 64 >= cnt_valid)
                    w[k] = ~0u;
        }

        // ranks among the wave's keys of the same digit, two to a register
        *(uint2 *)&cnt[wave][4 * lane] = make_uint2(0, 0);
        wave_lds_fence();
        uint32_t pos[K / 2];
        if (loose && cnt_valid == T) {
            // an LDS atomic per key, in no order among a row's lanes
            uint32_t *c2 = (uint32_t *)cnt[wave];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t d = (w[k] >> shift) & 255, sh = (d & 1) * 16;
                const uint32_t two = __hip_atomic_fetch_add(
                    c2 + (d >> 1), 1u << sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                const uint32_t c = (two >> sh) & 0xffff;
                if (k & 1)
                    pos[k / 2] |= c << 16;
                else
                    pos[k / 2] = c;
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t d = (w[k] >> shift) & 255;
                uint32_t mlo, mhi;
                match_digit(d, mlo, mhi);
                const uint32_t before =
                    __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0));
                const uint32_t all = __popc(mlo) + __popc(mhi);
                const uint32_t c = cnt[wave][d];
                if (k & 1)
                    pos[k / 2] |= (c + before) << 16;
                else
                    pos[k / 2] = c + before;
                if (before == 0)
                    cnt[wave][d] = (uint16_t)(c + all);
                // the next row's reads follow this row's writes of other lanes
                wave_lds_fence();
                __builtin_amdgcn_sched_barrier(0);  // one row's masks at a time
            }
        }
        if (tid < RADIX)
            gpre[tid] = first;
        __syncthreads();

        // every wave adds up the waves' counts itself: 4 digits per lane
        {
            uint32_t t[4] = {0, 0, 0, 0}, mine[4] = {0, 0, 0, 0};
#pragma unroll 4
            for (int v = 0; v < NW; ++v) {
                const uint2 q = *(const uint2 *)&cnt[v][4 * lane];
                if (v == wave) {
                    mine[0] = t[0];
                    mine[1] = t[1];
                    mine[2] = t[2];
                    mine[3] = t[3];
                }
                t[0] += q.x & 0xffff;
                t[1] += q.x >> 16;
                t[2] += q.y & 0xffff;
                t[3] += q.y >> 16;
            }
            const uint32_t sum = t[0] + t[1] + t[2] + t[3];
            uint32_t ex = wave_inclusive(sum) - sum;
            if (wave == 0) {
                uint4 g = *(const uint4 *)&gpre[4 * lane];
                g.x -= ex;
                g.y -= ex + t[0];
                g.z -= ex + t[0] + t[1];
                g.w -= ex + t[0] + t[1] + t[2];
                *(uint4 *)&gbase[4 * lane] = g;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mine[j] += ex;
                ex += t[j];
            }
            *(uint2 *)&off[wave][4 * lane] =
                make_uint2(mine[0] | (mine[1] << 16), mine[2] | (mine[3] << 16));
            wave_lds_fence();
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            asm("" : "+v"(w[k]));  // the digit is cheaper taken again than kept
            const uint32_t o = off[wave][(w[k] >> shift) & 255];
            pos[k / 2] += k & 1 ? o << 16 : o;
            xch[k & 1 ? pos[k / 2] >> 16 : (pos[k / 2] & 0xffff)] = w[k];
        }
        // the other words travel while the first are written out
        uint32_t s[TWO ? K : 1];
        uint64_t q[KIND == RADIX_BY_KEY ? K : 1];
        if constexpr (TWO)
            load_words(ssrc, packed_in, low, base, e0, s);
        if constexpr (KIND == RADIX_BY_KEY) {
            const __amdgpu_buffer_rsrc_t rp =
                raw_rsrc(a.p[st.src] + base, 8u * (uint32_t)cnt_valid);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rp, 8 * e0 + 8 * 64 * k, 0, 2);
                q[k] = ((uint64_t)(uint32_t)v[1] << 32) | (uint32_t)v[0];
            }
        }
        __syncthreads();
        // out in digit order; o: each position's output index
        const bool full = cnt_valid == T;
        uint32_t o[K];
#pragma unroll
        for (int i0 = 0; i0 < K; i0 += B) {
#pragma unroll
            for (int i = i0; i < i0 + B; ++i)
                w[i] = xch[t0 + i * NT];
#pragma unroll
            for (int i = i0; i < i0 + B; ++i) {
                o[i] = gbase[(w[i] >> shift) & 255] + (uint32_t)(t0 + i * NT);
                if (!packed_out) {
                    uint32_t v = w[i];
                    if (st.last) {
                        const Elem e = unmap_elem2<KIND>(Elem{v, v}, a);
                        v = low ? e.lo : e.hi;
                    }
                    if (full || t0 + i * NT < cnt_valid)
                        wdst[o[i]] = v;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (TWO) {
            // a 64-bit key's low word is mapped by the sign: below, beside it
            const bool pair_map = KIND == RADIX_KEYS64 && !low && st.first;
            if (st.first && !pair_map) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const Elem e = map_elem2<KIND>(Elem{s[k], s[k]}, a);
                    s[k] = low ? e.hi : e.lo;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k)
                xch[k & 1 ? pos[k / 2] >> 16 : (pos[k / 2] & 0xffff)] = s[k];
            __syncthreads();
#pragma unroll
            for (int i0 = 0; i0 < K; i0 += B) {
#pragma unroll
                for (int i = i0; i < i0 + B; ++i)
                    s[i] = xch[t0 + i * NT];
#pragma unroll
                for (int i = i0; i < i0 + B; ++i) {
                    if (!(full || t0 + i * NT < cnt_valid))
                        continue;
                    if (pair_map)
                        s[i] = map_elem2<KIND>(
                                   Elem{unmap_elem2<KIND>(Elem{w[i], 0}, a).hi, s[i]}, a)
                                   .lo;
                    if (packed_out) {
                        const Elem e =
                            unmap_elem2<KIND>(Elem{low ? s[i] : w[i], low ? w[i] : s[i]}, a);
                        ((uint2 *)a.k[B_OUT])[o[i]] = make_uint2(e.lo, e.hi);
                    } else {
                        uint32_t v = s[i];
                        if (st.last) {
                            const Elem e = unmap_elem2<KIND>(Elem{v, v}, a);
                            v = low ? e.hi : e.lo;
                        }
                        sdst[o[i]] = v;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (KIND == RADIX_BY_KEY) {
            uint64_t *pdst = a.p[st.dst];
            uint64_t *x8 = (uint64_t *)xraw;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k)
                x8[k & 1 ? pos[k / 2] >> 16 : (pos[k / 2] & 0xffff)] = q[k];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (full || t0 + i * NT < cnt_valid)
                    pdst[o[i]] = x8[t0 + i * NT];
        }
    }
}

constexpr int64_t align256(int64_t b) { return (b + 255) & ~(int64_t)255; }


// Workgroup shapes of the scatter kernel; the layout of the workspace and the
// launches both follow from shape_of, so they cannot disagree on the tile.
struct Shape {
    int nt, k;
};
constexpr Shape SHAPES[] = {{256, 8}, {512, 16}, {512, 32}, {1024, 16}, {512, 8}};

// Small sorts take small tiles (more workgroups than 8,192-key tiles give:
// 2^20 keys 66 against 71 us, 2^22 keys 96 and 97), up to 2^17 keys such that
// there are at most FEW_TILES (32) of them, whose sums cost a workgroup less
// than the scan launch (2^16 keys 51 -> 42 us, 100,003 keys 53 -> 43; 64 tiles
// of 2,048 keys 52 -> 50, 128 52 -> 64); keys alone large ones once
// the runs go to HBM (2^25 keys 0.40 against 0.43 ms, 2^26 0.77 with either tile,
// 2^27 1.74 -> 1.51, 2^28 3.72 -> 3.10).  Two words a key at K = 32 would spill; they take 16,384 with 1024
// threads from 5 * 2^23 on (4e7 doubles 1.35 ms with either tile, 5e7 1.70 ->
// 1.65, 5e7 pairs with random values 1.92 -> 1.80), keys with payloads from 2^25
// (0.96 -> 0.88 ms; 3e7 zipf keys 0.557 against 0.583, 2^26 keys 2.14 -> 1.87).
// small_counts: 8,192-key tiles below 2^22 keys too, for a scratch that does not
// hold the counts of four times as many tiles (3,850,241 to 4,194,303 keys 94-105
// us, 92-94 with 2,048-key tiles, 215 by merge passes).
int shape_of(int kind, int64_t n, bool small_counts)
{
    if (n < ((int64_t)1 << 22) && !small_counts)
        return n > ((int64_t)1 << 16) && n <= ((int64_t)1 << 17) ? 4 : 0;
    if (kind == RADIX_KEYS)
        return n >= ((int64_t)1 << 27) ? 2 : 1;
    return n >= (int64_t)(kind == RADIX_BY_KEY ? 4 : 5) << 23 ? 3 : 1;
}
int tile_of(int kind, int64_t n, bool small_counts)
{
    const Shape s = SHAPES[shape_of(kind, n, small_counts)];
    return s.nt * s.k;
}

// log2 of the tiles per chunk: at most MAX_CHUNKS chunks, half as many where
// there are few tiles (whose counts then fit the fixed scratch of the
// allocation-free sort beside 2^22 keys, see small_counts).
int chunk_log2(int64_t tiles)
{
    const int64_t most = tiles > 2 * MAX_CHUNKS ? MAX_CHUNKS : MAX_CHUNKS / 2;
    int l = 0;
    while ((tiles + ((int64_t)1 << l) - 1) >> l > most)
        ++l;
    return l;
}

}  // namespace

// Runs of the sample, sorted a run to a CU: 2^18 or 2^19 elements.
static int sample_runs(int64_t n)
{
    const int64_t r = n >> 19;
    return (int)(r < SAMPLE_RUNS_MAX ? r : SAMPLE_RUNS_MAX);
}

RadixLayout radix_layout(int kind, int64_t n, bool small_counts)
{
    RadixLayout w{};
    int64_t off = 0;
    w.a_k = off;
    off += align256(n * 4);
    if (kind == RADIX_PAIRS || kind == RADIX_KEYS64) {
        w.a_v = off;
        off += align256(n * 4);
    }
    if (kind == RADIX_KEYS64) {
        w.b_k = off;
        off += align256(n * 4);
        w.b_v = off;
        off += align256(n * 4);
    }
    if (kind == RADIX_BY_KEY) {
        w.a_p = off;
        off += align256(n * 8);
    }
    const int tile = tile_of(kind, n, small_counts);
    const int64_t tiles = (n + tile - 1) / tile;
    const int l = chunk_log2(tiles);
    const int64_t chunks = (tiles + ((int64_t)1 << l) - 1) >> l;
    w.ctl = off;
    off += align256(sizeof(Ctl));
    w.totals = off;
    off += align256(RADIX * 4);
    w.info = off;
    off += align256(chunks * (int64_t)sizeof(ChunkInfo));
    w.counts = off;
    off += align256(chunks * RADIX * 4);
    w.rows = off;
    off += align256(tiles * RADIX * 4);
    if ((kind == RADIX_PAIRS || kind == RADIX_KEYS64) && n >= SAMPLE_MIN) {
        w.sample_pairs = off;
        off += sample_runs(n) * 8 * 4;
        w.groups = off;
        off += GROUPS_MAX * (int64_t)sizeof(longlong2);
    }
    w.total = off;
    return w;
}

// One launch of a sort.  Each reads what the ones before wrote (positions from
// counts), so after one that failed nothing more is enqueued.
template <typename... P, typename... Args>
static void launch(hipError_t &e, void (*kernel)(P...), dim3 grid, int threads, hipStream_t s,
                   Args... args)
{
    if (e != hipSuccess)
        return;
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, s, args...);
    e = hipGetLastError();
}

// WAVES: waves per SIMD the registers are kept to; WGS: workgroups per CU.
template <int KIND, int SHAPE, int WAVES, int WGS>
static hipError_t run_radix(RadixArgs a, bool inplace, hipStream_t s)
{
    constexpr int NT = SHAPES[SHAPE].nt, K = SHAPES[SHAPE].k, T = NT * K;
    constexpr bool two = KIND == RADIX_PAIRS || KIND == RADIX_KEYS64;
    constexpr bool keys64 = KIND == RADIX_KEYS64;
    constexpr int passes = two ? 8 : 4;
    hipError_t e = hipSuccess;
    a.tiles = (a.n + T - 1) / T;
    a.per_log2 = chunk_log2(a.tiles);
    a.chunks = (int)((a.tiles + ((int64_t)1 << a.per_log2) - 1) >> a.per_log2);
    if constexpr (SHAPE == 0 || SHAPE == 4) {
        if (a.tiles <= FEW_TILES) {
            const dim3 grid((unsigned)a.tiles);
            for (int p = 0; p < passes; ++p) {
                if (p == 0)
                    launch(e, radix_count_first<KIND, T>, grid, COUNT_NT, s, a);
                else
                    launch(e, radix_count<KIND, T>, grid, COUNT_NT, s, a, p);
                launch(e, radix_scatter<NT, K, KIND, WAVES, OF_TILES>, grid, NT, s, a, p,
                       (int)inplace);
            }
            return e;
        }
    }
    const int64_t fit = (int64_t)device_cus() * WGS;
    int64_t wg = a.tiles < fit ? a.tiles : fit;
    wg = (wg + 7) & ~(int64_t)7;
    const dim3 cgrid((unsigned)a.chunks), sgrid((unsigned)wg);
    for (int p = 0; p < passes; ++p) {
        if (p == 0)
            launch(e, radix_count_first<KIND, T>, cgrid, COUNT_NT, s, a);
        else
            launch(e, radix_count<KIND, T>, cgrid, COUNT_NT, s, a, p);
        if constexpr (two) {
            if (p == 0 && a.sample_pairs)
                launch(e, radix_sample<KIND>, dim3(a.sample_runs), SAMPLE_LEN / 8, s, a);
        }
        launch(e, radix_scan, dim3(RADIX / 16 + (p == 0)), 512, s, a, p, passes, (int)two,
               (int)keys64, (int)inplace);
        launch(e, radix_scatter<NT, K, KIND, WAVES, OF_SCAN>, sgrid, NT, s, a, p, (int)inplace);
    }
    if constexpr (two) {
        if (a.sample_pairs) {
            launch(e, radix_finish<KIND>, dim3((unsigned)((a.n + 2047) / 2048)), 256, s, a);
            launch(e, radix_groups<KIND>, dim3(device_cus()), 1024, s, a);
            a.round = 1;  // the second round sorts the output, in place
            a.k[B_IN] = a.k[B_OUT];
            a.v[B_IN] = a.v[B_OUT];
            for (int p = 0; p < passes; ++p) {
                launch(e, radix_count<KIND, T>, cgrid, COUNT_NT, s, a, p);
                launch(e, radix_scatter<NT, K, KIND, WAVES, OF_CHUNKS>, sgrid, NT, s, a, p, 1);
            }
        }
    }
    return e;
}

hipError_t launch_radix(int kind, const RadixIO &io, int64_t n, void *ws, KeyMap km,
                        hipStream_t s, bool small_counts)
{
    const RadixLayout w = radix_layout(kind, n, small_counts);
    char *base = (char *)ws;
    RadixArgs a{};
    a.n = n;
    a.k[B_IN] = (uint32_t *)io.kin;
    a.v[B_IN] = (uint32_t *)io.vin;
    a.p[B_IN] = (uint64_t *)io.pin;
    a.k[B_OUT] = (uint32_t *)io.kout;
    a.v[B_OUT] = (uint32_t *)io.vout;
    a.p[B_OUT] = io.pout;
    a.k[B_A] = (uint32_t *)(base + w.a_k);
    a.v[B_A] = (uint32_t *)(base + w.a_v);
    a.p[B_A] = (uint64_t *)(base + w.a_p);
    a.k[B_B] = (uint32_t *)(base + w.b_k);
    a.v[B_B] = (uint32_t *)(base + w.b_v);
    a.ctl = base + w.ctl;
    a.totals = (uint32_t *)(base + w.totals);
    a.info = base + w.info;
    a.counts = (uint32_t *)(base + w.counts);
    a.rows = (uint32_t *)(base + w.rows);
    if (w.sample_pairs) {
        a.sample_runs = sample_runs(n);
        a.sample_pairs = (uint32_t *)(base + w.sample_pairs);
        a.groups = (longlong2 *)(base + w.groups);
    }
    // signed order (after the key map) to unsigned order of the words
    a.map.f = (uint32_t)km.fm;
    a.map.x = (uint32_t)km.um ^ 0x80000000u;
    a.fl = (uint32_t)km.fl;
    const bool inplace = io.kin == io.kout || (io.vin && io.vin == io.vout);
    const int shape = shape_of(kind, n, small_counts);
    switch (kind) {
    case RADIX_KEYS:
        return shape == 0   ? run_radix<RADIX_KEYS, 0, 6, 6>(a, inplace, s)
               : shape == 4 ? run_radix<RADIX_KEYS, 4, 6, 3>(a, inplace, s)
               : shape == 1 ? run_radix<RADIX_KEYS, 1, 6, 3>(a, inplace, s)
                            : run_radix<RADIX_KEYS, 2, 4, 2>(a, inplace, s);
    case RADIX_PAIRS:
        if (shape == 0 || shape == 4)
            break;
        return shape == 3 ? run_radix<RADIX_PAIRS, 3, 4, 1>(a, inplace, s)
                          : run_radix<RADIX_PAIRS, 1, 4, 2>(a, inplace, s);
    case RADIX_KEYS64:
        if (shape == 0 || shape == 4)
            break;
        return shape == 3 ? run_radix<RADIX_KEYS64, 3, 4, 1>(a, inplace, s)
                          : run_radix<RADIX_KEYS64, 1, 4, 2>(a, inplace, s);
    case RADIX_BY_KEY:
        return shape == 0   ? run_radix<RADIX_BY_KEY, 0, 4, 4>(a, inplace, s)
               : shape == 4 ? run_radix<RADIX_BY_KEY, 4, 4, 2>(a, inplace, s)
               : shape == 1 ? run_radix<RADIX_BY_KEY, 1, 4, 2>(a, inplace, s)
                            : run_radix<RADIX_BY_KEY, 3, 4, 1>(a, inplace, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace hvms
