// Kernels of the two-step HBP SpMV (Fig. 1, Algorithm 3, Section 3.3) and of the in-repo CSR
// baselines (Algorithm 1), as templates over the value type, with their launchers.  Included by
// one translation unit per value type (hbp_spmv.hip: fp32, hbp_spmv_f64.hip: fp64) so that the two
// sets of instantiations compile side by side.
#pragma once

#include "hbp_internal.h"

#include <atomic>
#include <type_traits>

namespace hbp {
namespace {

__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Wave-uniform read of a layout array that no kernel writes while an SpMV runs.  Going through
// the constant address space lets the compiler use a scalar load, whose result lands in an
// SGPR without a wait at the point of issue: this is what keeps the prefetch of the next
// groups' metadata off the critical path.
__device__ __forceinline__ int32_t uniform_load(const int32_t *p, int32_t i)
{
    typedef const int32_t __attribute__((address_space(4))) *const_ptr;
    return ((const_ptr)(uintptr_t)p)[i];
}

// One group, one wavefront.  Lane q owns slot q and has n nonzeros.  Rounds are taken U at a
// time ("a batch"): the U ballots give each round's live lanes, a lane's element in a round
// sits at the round's base plus the number of live lanes below it, all 2U loads are issued,
// then the products are accumulated through the staged vector segment.
// T is the value type, float or double.
template <int U, typename T>
struct Batch {
    uint32_t c[U];
    T v[U];
    int rounds;  // rounds of the batch in which some lane has a nonzero (they are the leading ones)
};

// a * b + c in one instruction (a lane without an element in the round drops the whole sum: a zero in place
// of the value alone would make NaN of an infinity in x that belongs to another row)
__device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Issues the loads of rounds k .. k+U-1 and advances base past them.  No load is predicated: a
// lane without an element in a round reads a neighbour's (or the position just behind the
// round: inside the group, or inside the padding behind the last group) and drops the product.
template <int U, typename T>
__device__ __forceinline__ void issue_batch(Batch<U, T> &b, const uint16_t *__restrict__ col_local,
                                            const T *__restrict__ data, uint32_t &base, int32_t n, int32_t k)
{
    b.rounds = 0;
#pragma unroll
    for (int u = 0; u < U; u++) {
        const uint64_t live = __ballot(k + u < n);
        b.c[u] = 0;
        b.v[u] = T(0);
        if (live) {  // wave-uniform: rounds past every row's end issue nothing
            // the round's base stays in the scalar part of the address, the lane's rank among the
            // live lanes is the 32-bit vector part: no 64-bit vector arithmetic per load
            const uint32_t rank = (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
            const char *round_col = reinterpret_cast<const char *>(col_local) + ((uint64_t)base << 1);
            const char *round_val = reinterpret_cast<const char *>(data) + (uint64_t)base * sizeof(T);
            b.c[u] = __builtin_nontemporal_load(reinterpret_cast<const uint16_t *>(round_col + (rank << 1)));
            b.v[u] = __builtin_nontemporal_load(reinterpret_cast<const T *>(round_val + rank * (uint32_t)sizeof(T)));
            base += (uint32_t)__popcll(live);
            b.rounds = u + 1;
        }
    }
}

// Products of the batch, summed per lane.  QUARTERS: the batch is taken in four quarters and a
// quarter without a nonzero is skipped (deep batches behind a group's first one are mostly
// empty when the rows are only a little longer than the first batch).
template <int U, bool QUARTERS = false, typename T>
__device__ __forceinline__ T consume_batch(const Batch<U, T> &b, const T *xs, int32_t n, int32_t k)
{
    T acc = T(0);
    if constexpr (QUARTERS) {
        constexpr int Q = U / 4;
#pragma unroll
        for (int q0 = 0; q0 < U; q0 += Q) {
            if (q0 < b.rounds) {  // wave-uniform
                T xv[Q];
#pragma unroll
                for (int u = 0; u < Q; u++) xv[u] = xs[b.c[q0 + u]];
#pragma unroll
                for (int u = 0; u < Q; u++) {
                    const T more = fma_of(b.v[q0 + u], xv[u], acc);
                    acc = k + q0 + u < n ? more : acc;
                }
            }
        }
    } else {
        T xv[U];
#pragma unroll
        for (int u = 0; u < U; u++) xv[u] = xs[b.c[u]];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const T more = fma_of(b.v[u], xv[u], acc);
            acc = k + u < n ? more : acc;
        }
    }
    return acc;
}

// Fast path for a full group whose 64 rows all have the same length n0 >= 4: its nonzeros are
// one contiguous run of 64 n0 elements in which element o belongs to the row of lane o mod 64.
// The run is read in 256-element chunks aligned to 1 KB (fp32 data) / 512 B (columns), four
// consecutive elements per lane with one 16-byte and one 8-byte load.  With d = distance from
// the first chunk's start to the run, lane l's j-th element of every chunk belongs to the row
// of lane (4 l + j - d) mod 64, so a lane keeps four running sums and no shuffle is needed
// until the end, when the four lanes l, l^16, l^32, l^48 that serve the same rows are added.
// Lanes whose four elements lie outside the run load nothing; elements outside the run that
// share a 16-byte quad with it are read but contribute nothing.  Used by the fp32 kernels only:
// with fp64 values the round-by-round walk measured 5 % faster on the 27-point stencil.
template <typename T>
struct Vec4 {
    typedef T type __attribute__((ext_vector_type(4)));
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int CH, typename T>
struct WideBatch {
    typename Vec4<T>::type v[CH];
    u32x2 c[CH];
};

// FIRST: the chunks start at the run's first chunk; only that one can hold elements in front of
// the run, so the other chunks are tested against the run's end alone.
template <int CH, bool FIRST = true, typename T>
__device__ __forceinline__ void issue_wide(WideBatch<CH, T> &b, const uint16_t *__restrict__ col_local,
                                           const T *__restrict__ data, uint32_t chunk0, uint32_t i0, uint32_t run_begin,
                                           uint32_t run_end, int lane)
{
#pragma unroll
    for (int u = 0; u < CH; u++) {
        const uint32_t p = chunk0 + 256u * (i0 + u) + 4u * (uint32_t)lane;
        b.v[u] = typename Vec4<T>::type{T(0), T(0), T(0), T(0)};
        b.c[u] = u32x2{0u, 0u};
        if ((!(FIRST && u == 0) || p + 3u >= run_begin) && p < run_end) {  // lanes whose four elements miss the run load nothing
            b.v[u] = __builtin_nontemporal_load(reinterpret_cast<const typename Vec4<T>::type *>(data + p));
            b.c[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(col_local + p));
        }
    }
}

template <int CH, bool FIRST = true, typename T>
__device__ __forceinline__ void consume_wide(const WideBatch<CH, T> &b, const T *xs, uint32_t chunk0, uint32_t i0,
                                             uint32_t run_begin, uint32_t run_end, int lane, T (&acc)[4])
{
    uint32_t c[CH][4];
    bool ok[CH][4];
    T xv[CH][4];
#pragma unroll
    for (int u = 0; u < CH; u++) {
        const uint32_t p = chunk0 + 256u * (i0 + u) + 4u * (uint32_t)lane;
        const uint32_t lo = b.c[u].x, hi = b.c[u].y;
        c[u][0] = lo & 0xffffu; c[u][1] = lo >> 16; c[u][2] = hi & 0xffffu; c[u][3] = hi >> 16;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            ok[u][j] = (!(FIRST && u == 0) || p + j >= run_begin) && p + j < run_end;
            c[u][j] = ok[u][j] ? c[u][j] : 0u;  // never index the segment with a foreign column
        }
    }
#pragma unroll
    for (int u = 0; u < CH; u++)
#pragma unroll
        for (int j = 0; j < 4; j++) xv[u][j] = xs[c[u][j]];
#pragma unroll
    for (int u = 0; u < CH; u++) {
        const T v[4] = {b.v[u].x, b.v[u].y, b.v[u].z, b.v[u].w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const T prod = v[j] * xv[u][j];
            acc[j] += ok[u][j] ? prod : T(0);
        }
    }
}

// Buffer resources: wave-uniform base and length in scalar registers, a lane's offset in one vector register.  Lanes at or
// behind the length read zero or store nothing, so that no load or store of a pack stands behind a branch and the
// compiler's counts of what is in flight stay exact.
typedef __amdgpu_buffer_rsrc_t Window;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Window window_of(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00027000);
}
constexpr int kNonTemporal = 2;
__device__ __forceinline__ uint32_t rank_from(uint64_t mask, uint32_t first)  // first + number of set lanes below this one
{
    return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, first));
}
// block-local columns of a lane's 16 bytes of fp32 values
__device__ __forceinline__ u32x2 load_columns(Window w, int lane) { return __builtin_amdgcn_raw_buffer_load_b64(w, lane * 8, 0, kNonTemporal); }
__device__ __forceinline__ void unpack_columns(u32x2 c, uint32_t (&out)[4])
{
    out[0] = c.x & 0xffffu; out[1] = c.x >> 16; out[2] = c.y & 0xffffu; out[3] = c.y >> 16;
}

// An element on its way to the lane of its row.
template <typename T>
struct alignas(2 * sizeof(T)) Routed {
    T v, x;
};

// Where to cut a group so that `target` of its nonzeros lie in front: the smallest round k with at
// least that many nonzeros in the rounds 0 .. k-1, and their number.  lens: the 64 rows' lengths, in LDS.
__device__ __forceinline__ void cut_rounds(const int32_t *lens, uint32_t target, int lane, int32_t &cut_k, uint32_t &cut_pos)
{
    // nonzeros of the group in rounds 0 .. k-1; every lane may ask for another k
    auto before = [&](int32_t k) __attribute__((always_inline)) {
        uint32_t sum = 0;
#pragma unroll 16
        for (int t = 0; t < 64; t++) sum += (uint32_t)min(lens[t], k);
        return sum;
    };
    cut_k = 0;
    cut_pos = 0;
    if (target == 0) return;  // wave-uniform
    // three 64-way splits of (0, 65536]: a segment has fewer than 65536 nonzeros, so all of the
    // group's lie in front of round 65536
    int32_t lo = 0;
    auto split = [&](int32_t step) __attribute__((always_inline)) {
        // candidates lo + step, lo + 2 step, ...: the last one is known to reach the target
        const uint32_t got = before(lo + (lane + 1) * step);
        const int first = __builtin_ctzll(__ballot(got >= target));
        lo += first * step;
        return (uint32_t)__shfl(got, first);
    };
    split(1024);
    split(16);
    cut_pos = split(1);
    cut_k = lo + 1;
}

template <int THREADS, int U, int GP, bool HEAVY, bool STEPS, typename T>
// (second launch bound: four wavefronts per SIMD, i.e. at most 128 vector registers per lane
// whatever the workgroup size; with more, two 512-thread workers no longer fit a CU together)
__global__ __launch_bounds__(THREADS, 4) void k_spmv_part(Layout L,
                                                       const T *__restrict__ x, T *__restrict__ partial,
                                                       T *__restrict__ y, uint32_t *__restrict__ col_ticket)
{
    const T *__restrict__ const data = static_cast<const T *>(L.data);
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    T *const xs = reinterpret_cast<T *>(dyn_lds);  // the staged vector segment, C values
    __shared__ int32_t sh_next;  // whose range to compete for next, broadcast to the worker
    __shared__ unsigned long long sh_rng;  // groups of the worker still to draw: end << 32 | next
    __shared__ int32_t sh_dry;   // nothing more to claim from the current competitive part
    __shared__ int32_t sh_lock;  // end of the last range reported as used up
    __shared__ int32_t sh_col[3];  // whose competitive part is being claimed, its first group, its end
    // per wavefront: elements (value, x) on their way to the lanes of their rows, or 64 sums
    // (With 224 and 112 for the packs, too, R-MAT 2^20 takes 90.2 us a product against 90.1, fp64 110.1 against 109.8.)
    constexpr int kRoute = STEPS ? kStepElements : sizeof(T) == 4 ? 192 : 96;
    // STEPS: fp32 groups are taken in steps instead of packs, where lists come last (see run_range)
    static_assert(!STEPS || sizeof(T) == 4, "a step's loads are of fp32 values");
    constexpr int E = 4, kWindow = 64 * E;  // elements of a step per lane and in all
    constexpr int kChunk = 8, kDepth = 3;  // groups of a draw at most, steps in flight (two to five measured within 3 % of each other)
    __shared__ __align__(16) Routed<T> sh_route[THREADS / 64 * kRoute + 1];
    constexpr int kHeavyCap = 64;
    __shared__ int32_t sh_heavy[kHeavyCap];  // heavy groups of the current range, each left to several wavefronts
    constexpr int kLongCap = 256;
    __shared__ int32_t sh_long[kLongCap];  // long groups of the current range, each left to the next free wavefront
    // the same for the groups the range begins with, as offsets from its first group: known before it is walked
    constexpr int kFirstHeavyCap = 64, kFirstLongCap = 1024;
    static_assert(THREADS / 64 <= 2 * kMaxOutweighing, "more groups could outweigh the others than have a place");
    __shared__ uint16_t sh_first_heavy[kFirstHeavyCap + kMaxOutweighing], sh_first_long[kFirstLongCap];  // (the last heavy places: those that outweigh the others)
    __shared__ __align__(16) T sh_nowhere[16 / sizeof(T)];
    __shared__ int32_t sh_heavy_n[2], sh_long_n[2], sh_long_next[2];  // 0: known before, 1: found among the claimed groups
    __shared__ int32_t sh_outweighing_n;
    static_assert(sizeof sh_route + sizeof sh_heavy + sizeof sh_long + sizeof sh_first_heavy + sizeof sh_first_long +
                      128 <= part_static_lds(THREADS), "part_static_lds is out of date");
    constexpr int kWaves = THREADS / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int staged_bn = -1;
    // Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Workers with
    // neighbouring ranges share block columns, hence slices of x: runs of four consecutive
    // workers are placed on one XCD (a slice is then fetched into that L2 once and re-staged from
    // there), successive runs on successive XCDs so that no XCD gets one contiguous part of the
    // matrix.
    const int32_t n_workers = (int32_t)gridDim.x;
    int32_t worker = (int32_t)blockIdx.x;
    if ((n_workers & 31) == 0) {
        const int32_t xcd = worker & 7, i = worker >> 3;
        worker = (((i >> 2) << 3) + xcd) * 4 + (i & 3);
    }

    // Starts the copy of the vector segment of block column bn into LDS: 16-byte loads that write LDS
    // themselves (no registers, nothing to wait for here) when the slice is 16-byte aligned.
    // The caller waits (wait_slice) and orders it with barriers.  (Against loads into registers and
    // stores to LDS, us per product: 27-point grid of 67^3 28.3 -> 27.8, lognormal 150001 x 400009 38.5 -> 36.9, 27-point grid of 128^3
    // 84.3 -> 83.6, R-MAT 2^22 and lognormal 4M x 1M as they were.)
    auto copy_slice = [&](int32_t bn) __attribute__((always_inline)) {
        const int64_t c0 = (int64_t)bn * L.C;
        const int32_t width = (int32_t)min((int64_t)L.C, L.n_cols - c0);
        constexpr int32_t kPer = 16 / (int32_t)sizeof(T);
        const T *src = x + c0;
        const int32_t n4 = (reinterpret_cast<uintptr_t>(src) & 15u) == 0 ? width / kPer : 0;
        typedef __attribute__((address_space(1))) const uint32_t *global_ptr;
        typedef __attribute__((address_space(3))) uint32_t *lds_ptr;
        for (int32_t i0 = wave * 64; i0 < n4; i0 += THREADS) {  // a wavefront's 64 quads land side by side
            const int32_t i = i0 + lane;
            if (i < n4)
                __builtin_amdgcn_global_load_lds((global_ptr)(uintptr_t)(src + kPer * i), (lds_ptr)(uint32_t)(uintptr_t)(xs + kPer * i0), 16, 0, 0);
        }
        for (int32_t i = kPer * n4 + threadIdx.x; i < width; i += THREADS) xs[i] = src[i];
    };
    auto wait_slice = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0x0F70); };  // vmcnt(0)

    // The wavefronts of the worker share out the groups [*, g_end) of the current range by
    // drawing packs of GP consecutive groups from an LDS counter (wavefronts do not progress at
    // the same speed, so a static deal would leave the slow ones behind).  Each wavefront keeps
    // three draws in hand and runs them as a two-deep software pipeline: while a pack is
    // walked, the lane lengths of the next one and the slot ranges / first positions of the one
    // after it are already on their way, and the partial sums of the previous one are stored
    // behind the current pack's loads.  GP > 1 is for matrices whose groups hold few nonzeros:
    // the first batches of all GP groups are issued before any is consumed.  A group index at
    // or beyond g_end gives an idle lane set (n = 0, position 0).
    //
    // Draws.  sh_rng holds the worker's current range of groups; a draw takes GP groups off its
    // front with one LDS atomic (draw_issue) whose result is looked at an iteration later
    // (draw_resolve), so that its latency is never waited for.  A draw that finds the range
    // used up, in a worker that competes for some worker's range (Section 3.3), leads to a claim:
    // the first wavefront to report the range that ended at `end` as used up (atomic max on
    // sh_lock; the ends of successive ranges grow) takes that range's next `claim` competitive
    // groups from its counter in global memory and publishes them as the new range;
    // the other wavefronts wait for the range to move (a bounded wait: a wavefront that gives
    // up just stops drawing, the claimed groups are walked by those that go on).  So the
    // wavefronts of a worker pass from fixed to competitive groups and from claim to claim
    // without a barrier.  Once the competitive part has nothing left (or in a worker that does not
    // compete) a used-up range makes the draw, and every later draw of the wavefront in this
    // range, return kNone.
    constexpr int32_t kNone = 0x7fffffff;
    constexpr int kSpinLimit = 1 << 16;
    bool stop = false;  // this wavefront draws no more in the current range
    int32_t per_draw = GP;  // groups of the next draw
    // does group g + q of the pack (g, its end e) exist?
    auto in_pack = [&](int32_t g, int32_t e, int q) __attribute__((always_inline)) {
        return GP == 1 ? g != kNone : q < e - g;
    };
    // In steps: fewer groups a draw towards the end of a range, so that the wavefronts are done with it together.
    auto draw_of = [&](int32_t left) __attribute__((always_inline)) { return max(min(left / (2 * kWaves), kChunk), 2); };
    auto draw_issue = [&]() __attribute__((always_inline)) {
        unsigned long long old = 0;  // reads as a used-up range
        if (lane == 0 && !stop) old = atomicAdd(&sh_rng, (unsigned long long)per_draw);
        return old;
    };
    auto draw_resolve = [&](unsigned long long old, int32_t &pack_end) __attribute__((always_inline)) {
        int32_t v = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)old);
        int32_t end = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(old >> 32));
        int spins = 0;
        while (v >= end) {
            if (stop || __hip_atomic_load(&sh_dry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                stop = true;
                pack_end = 0;
                return kNone;
            }
            int32_t reported = 0;
            if (lane == 0) reported = atomicMax(&sh_lock, end);
            reported = __builtin_amdgcn_readfirstlane(reported);
            if (reported < end) {
                // first to report this range as used up: claim the next competitive groups
                // (their owner's numbers sit in LDS: this path is rare, registers are not)
                const int32_t claim = L.claim, col_end = sh_col[2];
                uint32_t t = 0;
                if (lane == 0) t = atomicAdd(&col_ticket[sh_col[0]], (uint32_t)claim);
                t = __builtin_amdgcn_readfirstlane(t);
                const int64_t c0 = (int64_t)sh_col[1] + t;
                if (c0 >= col_end) {
                    if (lane == 0) __hip_atomic_store(&sh_dry, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    continue;  // leaves through the test above
                }
                const unsigned long long c1 = (unsigned long long)min(c0 + claim, (int64_t)col_end);
                if (lane == 0) atomicExch(&sh_rng, (c1 << 32) | (unsigned long long)c0);
            } else {
                // another wavefront claims: wait until the range's end moves or the column is dry
                bool moved = false;
                while (spins < kSpinLimit) {
                    const unsigned long long now = __hip_atomic_load(&sh_rng, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const int dry = __hip_atomic_load(&sh_dry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    spins++;
                    if ((int32_t)(uint32_t)(now >> 32) != end || dry) { moved = true; break; }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (!moved) stop = true;  // gave up: leaves through the test above
            }
            if (stop) continue;
            unsigned long long again = 0;
            if (lane == 0) again = atomicAdd(&sh_rng, (unsigned long long)per_draw);
            v = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)again);
            end = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(again >> 32));
        }
        pack_end = GP == 1 ? v + 1 : min(v + per_draw, end);
        if constexpr (STEPS) per_draw = draw_of(end - pack_end);
        return v;
    };
    // The rest of a group, rounds from k on, `count` <= kRoute elements from `base` on: the wavefront reads them
    // side by side and every lane picks the elements of its row out of LDS, round by round.  (A group of short rows
    // with one or a few longer ones has most of its lanes idle after a few rounds: of the 8 % of the groups of the 4M x 1M
    // lognormal matrix with more than 16 rounds 18 % of the lanes are alive.  Round by round they waited for memory
    // every 16 rounds, two loads a round; product 295 -> 285 us.)
    auto route = [&](uint32_t base, uint32_t count, int32_t n, int32_t k, T &acc) __attribute__((always_inline)) {
        constexpr int E = (kRoute + 63) / 64;
        Routed<T> *const way = sh_route + wave * kRoute;
        uint32_t c[E];
        T v[E];
#pragma unroll
        for (int u = 0; u < E; u++) {
            c[u] = 0;
            v[u] = T(0);
            if (64u * u < count) {  // wave-uniform
                const uint32_t o = base + min(64u * u + (uint32_t)lane, count - 1u);
                c[u] = __builtin_nontemporal_load(L.col_local + o);
                v[u] = __builtin_nontemporal_load(data + o);
            }
        }
#pragma unroll
        for (int u = 0; u < E; u++)
            if (64u * u + (uint32_t)lane < count) way[64 * u + lane] = {v[u], xs[c[u]]};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t off = 0;
        for (; __ballot(k < n); k += 4) {
            Routed<T> e[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const uint64_t live = __ballot(k + t < n);
                e[t] = way[off + (uint32_t)lanes_below(live)];  // (a lane without one: some entry, or the one behind the last)
                off += (uint32_t)__popcll(live);
            }
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const T more = fma_of(e[t].v, e[t].x, acc);
                acc = k + t < n ? more : acc;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // Rounds k, k+1, ... of one group until no lane has a nonzero left (lane q has n; `base` is
    // the position of round k, `end` the one behind the last element), added into acc.
    auto walk_rounds = [&](uint32_t &base, uint32_t end, int32_t n, int32_t k, T &acc) __attribute__((always_inline)) {
        for (;;) {
            if (end - base <= (uint32_t)kRoute) {
                if (end != base) route(base, end - base, n, k, acc);
                break;
            }
            const uint64_t live = __ballot(k < n);
            if (!live) break;
            const int32_t m = __popcll(live);
            constexpr int UL = 16;
            // (The folded batches below are compiled into the variant for matrices with very long
            // rows only: in the other variants, whose groups rarely get there, their code cost the
            // main path 4-10 % through registers and instruction cache.)
            const bool few = HEAVY ? m <= 32 : (m <= 32 && __ballot(k + 2 * U < n) == live);
            if (!few) {
                // many rows still going: a deep batch of rounds
                Batch<UL, T> deep;
                issue_batch<UL>(deep, L.col_local, data, base, n, k);
                acc += consume_batch<UL, true>(deep, xs, n, k);
                k += UL;
                continue;
            }
            if (HEAVY && __ballot(k + 2 * U < n) != live) {
                // Few rows left and one of them ends soon.  A batch would use m of 64 lanes, so the
                // wavefront is folded: with mm the power of two that holds the m live rows and
                // f = 64 / mm, lane j * mm + c serves the c-th live row in the rounds k + j, k + j + f,
                // k + j + 2f, ...  In that lane order (round, then row) the elements of f consecutive
                // rounds are exactly what one step of a batch reads, so the batch code runs
                // unchanged on the folded lanes' own counts and covers UL * f rounds.
                const int sh = m > 16 ? 5 : m > 8 ? 4 : m > 4 ? 3 : m > 2 ? 2 : m > 1 ? 1 : 0;  // mm = 2^sh
                int32_t *left = reinterpret_cast<int32_t *>(sh_route + wave * kRoute);
                left[lane] = 0;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (k < n) left[lanes_below(live)] = n - k;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int32_t mine = left[lane & ((1 << sh) - 1)], j = lane >> sh;  // rounds left in the row this lane serves
                const int32_t steps = mine > j ? (mine - j + (64 >> sh) - 1) >> (6 - sh) : 0;
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                Batch<UL, T> deep;
                issue_batch<UL>(deep, L.col_local, data, base, steps, 0);
                T *hand = reinterpret_cast<T *>(sh_route + wave * kRoute);
                hand[lane] = consume_batch<UL, true>(deep, xs, steps, 0);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (k < n)
                    for (int32_t t = lanes_below(live); t < 64; t += 1 << sh) acc += hand[t];
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                k += UL << (6 - sh);
                continue;
            }
            // Few rows left, all of them with at least 2U more rounds.  Until the shortest of
            // them ends, the live set is constant and the rounds k .. k_end-1 form one contiguous
            // span in which element o belongs to the (o mod m)-th live row.  The whole wavefront
            // reads the span: lanes 0 .. S-1 (S = largest multiple of m up to 64) take elements
            // lane, lane + S, ..., all for one row each, and the per-lane sums are handed to the
            // owning lanes through LDS.
            int32_t k_end = k < n ? n : 0x7fffffff;
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) k_end = min(k_end, __shfl_xor(k_end, d));
            const uint32_t span = (uint32_t)m * (uint32_t)(k_end - k);
            const uint32_t S = (64u / (uint32_t)m) * (uint32_t)m;
            T sum = T(0);
            if ((uint32_t)lane < S) {
                uint32_t o = (uint32_t)lane;
                for (; o + 3u * S < span; o += 4u * S) {
                    uint32_t c4[4];
                    T v4[4];
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        c4[u] = __builtin_nontemporal_load(L.col_local + base + o + u * S);
                        v4[u] = __builtin_nontemporal_load(data + base + o + u * S);
                    }
#pragma unroll
                    for (int u = 0; u < 4; u++) sum += v4[u] * xs[c4[u]];
                }
                for (; o < span; o += S) sum += data[base + o] * xs[L.col_local[base + o]];
            }
            T *hand = reinterpret_cast<T *>(sh_route + wave * kRoute);
            hand[lane] = sum;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (k < n)
                for (uint32_t t = (uint32_t)lanes_below(live); t < S; t += (uint32_t)m) acc += hand[t];
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            base += span;
            k = k_end;
        }
    };
    // Runs the groups [g_begin, g_end) of block column bn with all wavefronts of the worker; where it
    // competes, the groups claimed afterwards come from worker `owner`'s [c_lo, c_end).
    auto run_range = [&](int32_t bn, int32_t g_begin, int32_t g_end, bool compete, int32_t owner, int32_t c_lo, int32_t c_end) __attribute__((always_inline)) {
        __syncthreads();  // every wavefront has left the previous range (and its slice of x)
        if (threadIdx.x == 0) {
            sh_rng = ((unsigned long long)(uint32_t)g_end << 32) | (uint32_t)g_begin;
            sh_dry = compete ? 0 : 1;
            sh_lock = -1;
            sh_heavy_n[0] = sh_heavy_n[1] = 0;
            sh_outweighing_n = 0;
            sh_long_n[0] = sh_long_n[1] = 0;
            sh_long_next[0] = sh_long_next[1] = 0;
            sh_col[0] = owner;  // whose competitive groups are claimed from here on
            sh_col[1] = c_lo;
            sh_col[2] = c_end;
        }
        stop = false;
        __syncthreads();
        bool first_heavy = false, first_long = false;  // are the range's own heavy and long groups on the lists?
        if (HEAVY && bn != staged_bn) copy_slice(bn);
        if (HEAVY && !STEPS && L.lists_first) {
            const uint32_t in_range = (uint32_t)uniform_load(L.group_ptr, g_end) - (uint32_t)uniform_load(L.group_ptr, g_begin);
            for (int32_t i = g_begin + (int32_t)threadIdx.x; i < g_end; i += THREADS) {
                const int32_t longest = L.group_rounds[i + 1] - L.group_rounds[i];
                if (longest > L.long_rounds) {
                    const uint16_t offset = (uint16_t)(i - g_begin);
                    const int32_t in_group = L.group_ptr[i + 1] - L.group_ptr[i];
                    if (longest > L.heavy_rounds) {
                        const int32_t idx = atomicAdd(&sh_heavy_n[0], 1);
                        if (idx < kFirstHeavyCap) sh_first_heavy[idx] = offset;
                    } else if (in_group > L.heavy_elements && outweighs((uint32_t)in_group, in_range, kWaves)) {
                        sh_first_heavy[kFirstHeavyCap + atomicAdd(&sh_outweighing_n, 1)] = offset;
                    } else {
                        const int32_t idx = atomicAdd(&sh_long_n[0], 1);
                        if (idx < kFirstLongCap) sh_first_long[idx] = offset;
                    }
                }
            }
            wait_slice();
            __syncthreads();
            staged_bn = bn;
            first_heavy = sh_heavy_n[0] <= kFirstHeavyCap && g_end - g_begin <= 65536;
            first_long = sh_long_n[0] <= kFirstLongCap && g_end - g_begin <= 65536;  // (those that outweigh the others with them)
        }
        // (HEAVY: the listed groups, the others, what was listed meanwhile)
        for (int pass = 0;; pass++) {
        if constexpr (HEAVY) {
            // Heavy groups: the wavefronts of the worker walk up to four of them at a time, `share` wavefronts each.  The w-th of
            // these takes the rounds [k_w, k_{w+1}), where k_w is the first round that has w / share of the group's nonzeros
            // before it, and their per-lane sums are added in LDS in wavefront order.
            // (Bound by memory round trips, a few for the group's numbers and one for every 1024 nonzeros of a wavefront.  All wavefronts on
            // one group after the other: 15 us a group, however few nonzeros were left to each; R-MAT 2^22 has nine such groups in the
            // first worker's range, which took 247 us where the average worker took 160.  Product 296 -> 267 us.)
            const int32_t n_by_row = pass ? min(sh_heavy_n[1], kHeavyCap) : first_heavy ? sh_heavy_n[0] : 0;
            const int32_t n_heavy = n_by_row + (!pass && first_long ? sh_outweighing_n : 0);
            // Where the range competes, how many of them a worker has claimed differs from call to call, and how a group is cut, hence the last
            // bits of its sums, must not: there it is two at a time, whatever has been claimed.  (With a share given, us per product, one at
            // a time / two / four: R-MAT 2^22 317 / 254 / 256, 2^20 124 / 118 / 113, fp64 137 / 136 / 143, 2^19 81 / 80 / 80.)
            const int log_at_once = pass && compete ? 1 : n_heavy >= 4 ? 2 : n_heavy >= 2 ? 1 : 0, share = kWaves >> log_at_once;
            for (int32_t i0 = 0; i0 < n_heavy; i0 += 1 << log_at_once) {
                const int32_t i = i0 + wave / share, part = wave % share;
                T *const sums = reinterpret_cast<T *>(sh_route + wave * kRoute);  // the wavefront's place: lengths, what the walk holds there, its sums
                int32_t hs0 = 0, hs1 = 0;
                if (i < n_heavy) {
                    const int32_t gh = __builtin_amdgcn_readfirstlane(
                        pass ? sh_heavy[i] : g_begin + (int32_t)sh_first_heavy[i < n_by_row ? i : kFirstHeavyCap + i - n_by_row]);
                    hs0 = uniform_load(L.group_slot, gh);
                    hs1 = uniform_load(L.group_slot, gh + 1);
                    const uint32_t b0 = (uint32_t)uniform_load(L.group_ptr, gh);
                    const uint32_t total = (uint32_t)uniform_load(L.group_ptr, gh + 1) - b0;
                    const int32_t len = hs0 + lane < hs1 ? (int32_t)L.seg_len[hs0 + lane] : 0;
                    int32_t *lens = reinterpret_cast<int32_t *>(sums);
                    lens[lane] = len;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    int32_t k_lo, k_hi = 1 << 16;
                    uint32_t lo, hi = total;
                    cut_rounds(lens, (uint32_t)(((uint64_t)total * (uint32_t)part) / (uint32_t)share), lane, k_lo, lo);
                    if (part + 1 < share) cut_rounds(lens, (uint32_t)(((uint64_t)total * (uint32_t)(part + 1)) / (uint32_t)share), lane, k_hi, hi);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    uint32_t pos = b0 + lo;
                    T sum = T(0);
                    walk_rounds(pos, b0 + hi, min(len, k_hi), k_lo, sum);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    sums[lane] = sum;
                }
                __syncthreads();
                if (part == 0 && hs0 + lane < hs1) {
                    T total_sum = sums[lane];
                    for (int w = 1; w < share; w++) total_sum += reinterpret_cast<const T *>(sh_route + (wave + w) * kRoute)[lane];
                    partial[hs0 + lane] = total_sum;
                }
                __syncthreads();  // the places are used again
            }
            // Long groups: one wavefront each, whoever is free next.
            const int32_t n_long = pass ? min(sh_long_n[1], kLongCap) : first_long ? sh_long_n[0] : 0;
            while (n_long > 0) {
                int32_t i = 0;
                if (lane == 0) i = atomicAdd(&sh_long_next[pass], 1);
                i = __builtin_amdgcn_readfirstlane(i);
                if (i >= n_long) break;
                const int32_t gl = __builtin_amdgcn_readfirstlane(pass ? sh_long[i] : g_begin + (int32_t)sh_first_long[i]);
                const int32_t ls0 = uniform_load(L.group_slot, gl), ls1 = uniform_load(L.group_slot, gl + 1);
                uint32_t pos = (uint32_t)uniform_load(L.group_ptr, gl);
                const int32_t len = ls0 + lane < ls1 ? (int32_t)L.seg_len[ls0 + lane] : 0;
                T sum = T(0);
                walk_rounds(pos, (uint32_t)uniform_load(L.group_ptr, gl + 1), len, 0, sum);
                if (ls0 + lane < ls1) partial[ls0 + lane] = sum;
            }
            if (pass == 1) break;
        }
        if constexpr (STEPS) {
            // In steps.  A step is a run of up to E groups whose rows all have one nonzero, or one other group.  Its elements lie
            // side by side, so every lane loads E of them with one 16-byte and one 2E-byte load; where they begin and end follows
            // from group_ptr alone, so the loads of kDepth steps are in flight, whatever the rows' lengths.  In a run of rows
            // of one nonzero the products are the sums: no lengths are read, and E sums per lane are stored together.
            // Otherwise values and gathered x go through LDS, and every lane picks the elements of its row there round by round.
            // What does not fit there is walked after the others of a turn, as in the packs, with nothing of its own in flight.
            // (Bound by HBM where segments are short: 340 MB at 5.4 TB/s on 2^20 rows of 32 from templates, a quarter of it stores; half of the
            // groups there and of 4M x 1M lognormal rows have rows of one nonzero.  Products: walk_in_steps.)
            int32_t e = 0, e1 = 0;  // ends of the chunks g and g1 of groups
            per_draw = draw_of(g_end - g_begin);
            int32_t g = draw_resolve(draw_issue(), e), g1 = draw_resolve(draw_issue(), e1);
            // Lane l: first slot and first element of the chunk's group l; from the chunk's end on the ends of its last group.
            // (Of no chunk: those of group 0, so that it is empty.)
            uint32_t chunk_slot, chunk_pos, chunk_slot_n, chunk_pos_n;  // of the chunks g and g1
            auto chunk_at = [&](int32_t first, int32_t end) __attribute__((always_inline)) {
                return (uint32_t)((first == kNone ? 0 : first) + min(lane, first == kNone ? 0 : end - first));
            };
            // Bit i: a step begins with the chunk's group i; the highest bit: behind the last group.
            uint32_t starts = 0;
            auto open_chunk = [&]() __attribute__((always_inline)) {
                const int32_t count = g == kNone ? 0 : e - g;
                const uint32_t slots = (uint32_t)__shfl_down((int)chunk_slot, 1) - chunk_slot;
                const uint32_t elements = (uint32_t)__shfl_down((int)chunk_pos, 1) - chunk_pos;
                const uint32_t ones = (uint32_t)__ballot(lane < count && slots == elements);
                uint32_t run = ones;  // bit i: groups i - E .. i are all of such rows
#pragma unroll
                for (int t = 1; t <= E; t++) run &= ones << t;
                starts = ~(ones & ones << 1);
#pragma unroll
                for (int t = E; t < kChunk; t += E) starts |= starts << E & run;
                starts = (starts & ((1u << count) - 1u)) | 1u << count;
            };
            u32x4 v[kDepth];
            u32x2 c[kDepth];
            uint32_t len[kDepth];
            int32_t at[kDepth], slot[kDepth];   // the step's first group and slot
            uint32_t pos[kDepth], slots[kDepth], count[kDepth];  // its first element, its slots and elements
            // Does a step's group fit the wavefront's place in LDS: all of it, or what is left once its first two rounds are done?
            // (Asked about in `fetch`, too, it costs bands of 2 nonzeros per row 4 %: groups of so few rows are loaded and then walked.)
            auto fits = [&](uint32_t elements, uint32_t rows) __attribute__((always_inline)) {
                return elements <= (uint32_t)kRoute || (elements <= (uint32_t)kWindow && rows >= (uint32_t)(kWindow - kRoute) + E);
            };
            auto fetch = [&](int d) __attribute__((always_inline)) {
                const int i = __builtin_ctz(starts);
                const uint32_t rest = starts & (starts - 1u);
                const int j = rest ? __builtin_ctz(rest) : i;  // (nothing left: an empty step)
                starts = rest ? rest : starts;
                at[d] = g + i;
                slot[d] = (int32_t)__builtin_amdgcn_readlane(chunk_slot, i);
                pos[d] = (uint32_t)__builtin_amdgcn_readlane(chunk_pos, i);
                slots[d] = (uint32_t)__builtin_amdgcn_readlane(chunk_slot, j) - (uint32_t)slot[d];
                count[d] = (uint32_t)__builtin_amdgcn_readlane(chunk_pos, j) - pos[d];
                const uint32_t n = count[d] <= (uint32_t)kWindow ? count[d] : 0u;
                v[d] = __builtin_amdgcn_raw_buffer_load_b128(window_of(data + pos[d], n * (uint32_t)sizeof(T)), lane * 16, 0, kNonTemporal);
                c[d] = load_columns(window_of(L.col_local + pos[d], ((n + 3u) & ~3u) * 2u), lane);  // (whole words; the arrays are padded)
                len[d] = __builtin_amdgcn_raw_buffer_load_b16(window_of(L.seg_len + slot[d], count[d] == slots[d] ? 0u : slots[d] * 2u), lane * 2, 0, 0);
            };
            uint32_t next_at = chunk_at(g, e);
            chunk_slot = (uint32_t)L.group_slot[next_at];
            chunk_pos = (uint32_t)L.group_ptr[next_at];
            next_at = chunk_at(g1, e1);
            chunk_slot_n = (uint32_t)L.group_slot[next_at];
            chunk_pos_n = (uint32_t)L.group_ptr[next_at];
            open_chunk();
            if (bn != staged_bn && !HEAVY) copy_slice(bn);
#pragma unroll
            for (int d = 0; d < kDepth; d++) fetch(d);
            if (bn != staged_bn) {
                wait_slice();
                __syncthreads();
                staged_bn = bn;
            }
            // (nothing in flight on any way into the loop: the compiler does not see that the copy to LDS, which counts as a load and as
            // an LDS access, has always been waited for, and would wait for everything throughout)
            __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
            // the wavefront's elements on their way to the lanes of their rows: kRoute values, then their x; where a lane's E go
            // (lanes whose elements never count write where nothing is read)
            T *const way_v = reinterpret_cast<T *>(sh_route + wave * kRoute), *const way_x = way_v + kRoute;
            const bool counts = lane < kRoute / E;
            T *const write_v = counts ? way_v + E * lane : sh_nowhere, *const write_x = counts ? way_x + E * lane : sh_nowhere;
            uint32_t long_step = 0;  // lanes 4 d .. 4 d + 3: first slot, slots, first element and elements of a group to be walked
            for (;;) {
                const bool used_up = (starts & (starts - 1u)) == 0;
                if (used_up && g != kNone) {
                    // the next chunk; its numbers were asked for when this one was begun
                    chunk_slot = chunk_slot_n;
                    chunk_pos = chunk_pos_n;
                    g = g1;
                    e = e1;
                    g1 = draw_resolve(draw_issue(), e1);
                    asm volatile("" : "+v"(chunk_slot), "+v"(chunk_pos));
                    next_at = chunk_at(g1, e1);
                    open_chunk();
                }
                // (in every turn, although they change with the chunk only: loaded in the branch they would be copied to where the
                // other way leaves them, and waited for right there)
                chunk_slot_n = (uint32_t)L.group_slot[next_at];
                chunk_pos_n = (uint32_t)L.group_ptr[next_at];
                const bool last = g == kNone;  // (a wavefront that has drawn nothing draws nothing more)
                uint32_t walked = 0;  // bit d: the group of step d is too long for its window
                int32_t rest[kDepth];
#pragma unroll
                for (int d = 0; d < kDepth; d++) {
                    T vv[E];
                    __builtin_memcpy(vv, &v[d], 16);
                    uint32_t cc[E];
                    unpack_columns(c[d], cc);
                    rest[d] = (int32_t)len[d];
                    asm volatile("" : "+v"(rest[d]));  // (the value from here on: a copy made elsewhere would wait for loads just issued)
                    const Window out = window_of(partial + slot[d], slots[d] * (uint32_t)sizeof(T));
                    if (count[d] == slots[d]) {
                        // rows of one nonzero: the products are the sums
                        T xv[E], sum[E];
#pragma unroll
                        for (int t = 0; t < E; t++) xv[t] = xs[cc[t]];
#pragma unroll
                        for (int t = 0; t < E; t++) sum[t] = fma_of(vv[t], xv[t], T(0));
                        u32x4 bits;
                        __builtin_memcpy(&bits, sum, 16);
                        __builtin_amdgcn_raw_buffer_store_b128(bits, out, lane * 16, 0, 0);
                    } else {
                        int32_t n = rest[d];
                        T acc = T(0);
                        const bool walk = !fits(count[d], slots[d]);
                        bool stored = !walk;
                        if constexpr (HEAVY) {
                            // (see below: what the lists hold looks empty here)
                            if (__ballot(n > L.long_rounds)) {
                                const bool heavy = __ballot(n > L.heavy_rounds) != 0;
                                int32_t idx = 0;
                                if (lane == 0) idx = atomicAdd(heavy ? &sh_heavy_n[1] : &sh_long_n[1], 1);
                                idx = __builtin_amdgcn_readfirstlane(idx);
                                if (idx < (heavy ? kHeavyCap : kLongCap)) {
                                    if (lane == 0) (heavy ? sh_heavy : sh_long)[idx] = at[d];
                                    n = 0;
                                    rest[d] = 0;
                                    stored = false;
                                }
                            }
                        }
                        if (walk) {
                            walked |= 1u << d;
                            const int l = lane - 4 * d;
                            long_step = l == 0 ? (uint32_t)slot[d] : l == 1 ? slots[d] : l == 2 ? pos[d] : l == 3 ? count[d] : long_step;
                        } else {
                            T xv[E];
#pragma unroll
                            for (int t = 0; t < E; t++) xv[t] = xs[cc[t]];
                            __builtin_memcpy(write_v, vv, 16);
                            __builtin_memcpy(write_x, xv, 16);
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                            __builtin_amdgcn_wave_barrier();
                            // round 0 has every row, so a lane's element there is the lane-th
                            uint32_t off = slots[d];
                            uint64_t live = __ballot(n > 1);
                            const uint32_t i1 = rank_from(live, off);
                            const T v0 = way_v[lane], x0 = way_x[lane], v1 = way_v[i1], x1 = way_x[i1];
                            off += (uint32_t)__popcll(live);
                            acc = fma_of(v0, x0, T(0));
                            const T two = fma_of(v1, x1, acc);
                            acc = n > 1 ? two : acc;
                            for (int32_t k = 2; (live = __ballot(k < n)) != 0; k += 2) {
                                if (k == 2 && count[d] > (uint32_t)kRoute) {
                                    // the elements of these rounds take the place of the first two rounds'
                                    const uint32_t done = off & ~(uint32_t)(E - 1), place = (uint32_t)(E * lane) - done;
                                    off -= done;
                                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                                    __builtin_amdgcn_wave_barrier();
                                    const bool left = place < (uint32_t)kRoute;  // (in front of `done`: wrapped around)
                                    __builtin_memcpy(left ? way_v + place : sh_nowhere, vv, 16);
                                    __builtin_memcpy(left ? way_x + place : sh_nowhere, xv, 16);
                                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                                    __builtin_amdgcn_wave_barrier();
                                }
                                const uint32_t ia = rank_from(live, off);
                                off += (uint32_t)__popcll(live);
                                live = __ballot(k + 1 < n);
                                const uint32_t ib = rank_from(live, off);
                                off += (uint32_t)__popcll(live);
                                const T va = way_v[ia], xa = way_x[ia], vb = way_v[ib], xb = way_x[ib];
                                const T ma = fma_of(va, xa, acc);
                                acc = k < n ? ma : acc;
                                const T mb = fma_of(vb, xb, acc);
                                acc = k + 1 < n ? mb : acc;
                            }
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                            __builtin_amdgcn_wave_barrier();
                        }
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, acc), window_of(partial + slot[d], stored ? slots[d] * 4u : 0u), lane * 4, 0, 0);
                    }
                    fetch(d);
                }
                asm volatile("" : "+v"(chunk_slot_n), "+v"(chunk_pos_n));  // (waited for here, in front of whatever the walks load)
                for (; walked; walked &= walked - 1) {
                    const int d = __builtin_ctz(walked);
                    int32_t n = rest[0];
#pragma unroll
                    for (int t = 1; t < kDepth; t++) n = d == t ? rest[t] : n;
                    const int32_t s0 = (int32_t)__builtin_amdgcn_readlane(long_step, 4 * d), rows = (int32_t)__builtin_amdgcn_readlane(long_step, 4 * d + 1);
                    uint32_t base = (uint32_t)__builtin_amdgcn_readlane(long_step, 4 * d + 2);
                    const uint32_t end = base + (uint32_t)__builtin_amdgcn_readlane(long_step, 4 * d + 3);
                    T acc = T(0);
                    if (__ballot(n != 0)) {  // (else it is on a list)
                        walk_rounds(base, end, n, 0, acc);
                        if (lane < rows) partial[s0 + lane] = acc;
                    }
                }
                if (last) break;
            }
        } else {
        int32_t e = 0, e1 = 0, e2 = 0;  // ends of the packs g, g1, g2: group g + q exists if it is below e
        int32_t g = draw_resolve(draw_issue(), e), g1 = draw_resolve(draw_issue(), e1), g2 = kNone;
        unsigned long long raw2 = draw_issue();
        int32_t s0[GP], s1[GP], n[GP], done_slot[GP];
        // The slot ranges and first positions of a pack's groups travel in one vector register per
        // pack: lane l <= GP holds group_slot[first + l], lane 32 + l holds
        // group_ptr[first + l], zero where the pack has no such group; they are read out into
        // scalars where they are used.  (Loaded as scalars and carried three packs deep they did
        // not fit the scalar registers: the spills cost some fifty instructions per pack and made
        // the wavefront wait for each scalar load right where it was issued.)
        auto load_meta = [&](int32_t first, int32_t end) __attribute__((always_inline)) {
            uint32_t m = 0;
            const int32_t l = lane & 31;
            const bool position = lane >= 32;
            if (first != kNone && l <= GP && l <= end - first)
                m = (uint32_t)(position ? L.group_ptr : L.group_slot)[first + l];
            return m;
        };
        auto meta_slots = [&](uint32_t m, int32_t first, int32_t end, int q, int32_t &from, int32_t &to) __attribute__((always_inline)) {
            const bool there = in_pack(first, end, q);
            from = there ? (int32_t)__builtin_amdgcn_readlane(m, q) : 0;
            to = there ? (int32_t)__builtin_amdgcn_readlane(m, q + 1) : 0;
        };
        auto meta_base = [&](uint32_t m, int32_t first, int32_t end, int q) __attribute__((always_inline)) {
            return q == 0 || in_pack(first, end, q - 1) ? (uint32_t)__builtin_amdgcn_readlane(m, 32 + q) : 0u;
        };
        uint32_t meta = load_meta(g, e), meta_n = load_meta(g1, e1);  // of the packs g and g1
        // Packs of short rows have a path of their own in the fp64 kernels.  (In fp32 it measured
        // 2-3 % slower than the general path: the kernel is bound by the latency of a pack's
        // loads, not by its instructions, and the extra code costs registers.)
        constexpr bool kShortPacks = GP > 1 && sizeof(T) == 8;
        // longest row of the packs g and g1 (wave-uniform; only looked at where kShortPacks)
        int32_t pack_longest = 0, pack_longestn = 0;
        auto longest_in_pack = [&](int32_t first, int32_t end) __attribute__((always_inline)) {
            int32_t most = 0;
            if constexpr (kShortPacks) {
#pragma unroll
                for (int q = 0; q < GP; q++)
                    if (in_pack(first, end, q))
                        most = max(most, uniform_load(L.group_rounds, first + q + 1) - uniform_load(L.group_rounds, first + q));
            }
            return most;
        };
        uint32_t base[GP];  // positions stay 32-bit: nnz < 2^31
        T done_acc[GP];
#pragma unroll
        for (int q = 0; q < GP; q++) {
            done_slot[q] = -1;
            done_acc[q] = T(0);
            meta_slots(meta, g, e, q, s0[q], s1[q]);
            n[q] = s0[q] + lane < s1[q] ? L.seg_len[s0[q] + lane] : 0;
        }
        pack_longest = longest_in_pack(g, e);
        pack_longestn = longest_in_pack(g1, e1);
        // (without lists the slice starts here, behind the first packs' lengths: loads return in order, and in front of
        // them it would delay them; 27-point grid of 67^3 29.6 against 28.6 us)
        if (bn != staged_bn) {
            if (!HEAVY) copy_slice(bn);
            wait_slice();
            __syncthreads();
            staged_bn = bn;
        }
        for (;;) {
            g2 = draw_resolve(raw2, e2);  // drawn an iteration ago
            if (g == kNone && g1 == kNone && g2 == kNone) break;  // and this wavefront has stopped drawing
            raw2 = draw_issue();
#pragma unroll
            for (int q = 0; q < GP; q++) {
                meta_slots(meta, g, e, q, s0[q], s1[q]);
                base[q] = meta_base(meta, g, e, q);
            }
            // A group with a row of more than heavy_rounds nonzeros would keep this wavefront busy long
            // after the rest of the worker has run dry, and groups with rows of more than long_rounds come
            // in runs (the last groups of a block), of which a pack hands several to one wavefront to walk
            // one after the other.  Those that the range began with have been walked before (unless they
            // did not fit the lists) and look empty here; among the claimed ones the heavy ones go on the
            // worker's heavy list, the long ones on the long list (unless it is full), which are walked
            // when the range's other groups are done.
            if (HEAVY && (!kShortPacks || pack_longest > L.long_rounds)) {
#pragma unroll
                for (int q = 0; q < GP; q++) {
                    if (__ballot(n[q] > L.long_rounds)) {
                        const bool heavy = __ballot(n[q] > L.heavy_rounds) != 0;
                        bool listed = heavy ? first_heavy : first_long;
                        if (g + q >= g_end || !L.lists_first) {
                            int32_t idx = 0;
                            if (lane == 0) idx = atomicAdd(heavy ? &sh_heavy_n[1] : &sh_long_n[1], 1);
                            idx = __builtin_amdgcn_readfirstlane(idx);
                            listed = idx < (heavy ? kHeavyCap : kLongCap);
                            if (listed && lane == 0) (heavy ? sh_heavy : sh_long)[idx] = g + q;
                        }
                        if (listed) {
                            n[q] = 0;
                            s1[q] = s0[q];
                        }
                    }
                }
            }
            int32_t nn[GP], slot[GP];
            const int32_t pack_longestnn = longest_in_pack(g2, e2);
            const uint32_t meta_nn = load_meta(g2, e2);
            T acc[GP];
            // lane lengths of group q of the pack g1
            auto next_lengths = [&](int q) __attribute__((always_inline)) {
                int32_t from, to;
                meta_slots(meta_n, g1, e1, q, from, to);
                return from + lane < to ? (int32_t)L.seg_len[from + lane] : 0;
            };
            bool wide = false;
            if constexpr (GP == 1 && sizeof(T) == 4) {
                const int32_t n0 = __builtin_amdgcn_readfirstlane(n[0]);
                wide = s1[0] - s0[0] == 64 && n0 >= 4 && __ballot(n[0] != n0) == 0;
                if (wide) {
                    // full group, equal rows: aligned wide loads
                    constexpr int CH = 4;
                    const uint32_t chunk0 = base[0] & ~255u, run_end = base[0] + 64u * (uint32_t)n0;
                    const uint32_t n_chunks = (run_end - chunk0 + 255u) >> 8;
                    T a4[4] = {T(0), T(0), T(0), T(0)};
                    WideBatch<CH, T> wb;
                    issue_wide<CH>(wb, L.col_local, data, chunk0, 0, base[0], run_end, lane);
                    if (done_slot[0] >= 0) partial[done_slot[0]] = done_acc[0];
                    nn[0] = next_lengths(0);
                    consume_wide<CH>(wb, xs, chunk0, 0, base[0], run_end, lane, a4);
                    for (uint32_t i0 = CH; i0 < n_chunks; i0 += CH) {
                        issue_wide<CH, false>(wb, L.col_local, data, chunk0, i0, base[0], run_end, lane);
                        consume_wide<CH, false>(wb, xs, chunk0, i0, base[0], run_end, lane, a4);
                    }
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        a4[j] += __shfl_xor(a4[j], 16);
                        a4[j] += __shfl_xor(a4[j], 32);
                    }
                    const int m = lane >> 4;  // this lane reports the m-th of its four rows
                    acc[0] = m == 0 ? a4[0] : m == 1 ? a4[1] : m == 2 ? a4[2] : a4[3];
                    slot[0] = s0[0] + (int32_t)((4u * (uint32_t)(lane & 15) + (uint32_t)m + 256u - (base[0] - chunk0)) & 63u);
                }
            }
            if (kShortPacks && pack_longest <= 2) {
                // Packs of groups whose rows have one or two nonzeros (wave-uniform, known from the
                // groups' longest rows): round 0 of a group is its slots in order, so lane q's first
                // element sits at base + q and no ballot is needed; round 1 holds the second
                // elements of the rows that have one.  Lanes without a slot or a second element read
                // a position inside the group or the padding behind it and drop the product.
                uint32_t c0[GP], c1[GP];
                T v0[GP], v1[GP];
#pragma unroll
                for (int q = 0; q < GP; q++) {
                    c0[q] = __builtin_nontemporal_load(L.col_local + base[q] + lane);
                    v0[q] = __builtin_nontemporal_load(data + base[q] + lane);
                }
                if (pack_longest == 2) {
#pragma unroll
                    for (int q = 0; q < GP; q++) {
                        const uint64_t live = __ballot(n[q] > 1);
                        const uint32_t j = (uint32_t)__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, base[q] + (uint32_t)(s1[q] - s0[q])));
                        c1[q] = __builtin_nontemporal_load(L.col_local + j);
                        v1[q] = __builtin_nontemporal_load(data + j);
                    }
                }
#pragma unroll
                for (int q = 0; q < GP; q++) {
                    if (done_slot[q] >= 0) partial[done_slot[q]] = done_acc[q];
                    nn[q] = next_lengths(q);
                }
                if (pack_longest == 2) {
                    T x0[GP], x1[GP];
#pragma unroll
                    for (int q = 0; q < GP; q++) { x0[q] = xs[c0[q]]; x1[q] = xs[c1[q]]; }
#pragma unroll
                    for (int q = 0; q < GP; q++) {
                        const T p1 = v1[q] * x1[q];
                        acc[q] = v0[q] * x0[q] + (n[q] > 1 ? p1 : T(0));
                    }
                } else {
                    T x0[GP];
#pragma unroll
                    for (int q = 0; q < GP; q++) x0[q] = xs[c0[q]];
#pragma unroll
                    for (int q = 0; q < GP; q++) acc[q] = v0[q] * x0[q];
                }
#pragma unroll
                for (int q = 0; q < GP; q++) slot[q] = s0[q] + lane < s1[q] ? s0[q] + lane : -1;
            } else if (!wide) {
                // general groups: round by round, U rounds per batch
                Batch<U, T> bt[GP];
#pragma unroll
                for (int q = 0; q < GP; q++) issue_batch<U>(bt[q], L.col_local, data, base[q], n[q], 0);
#pragma unroll
                for (int q = 0; q < GP; q++) {
                    if (done_slot[q] >= 0) partial[done_slot[q]] = done_acc[q];
                    nn[q] = next_lengths(q);
                }
#pragma unroll
                for (int q = 0; q < GP; q++) acc[q] = consume_batch<U>(bt[q], xs, n[q], 0);
#pragma unroll
                for (int q = 0; q < GP; q++) {  // rows longer than U, one group at a time
                    // (the test keeps what the compiler hoists out of the walk's loops, a dozen
                    // values per group, off the path of the groups without such rows)
                    if (__ballot(U < n[q])) walk_rounds(base[q], meta_base(meta, g, e, q + 1), n[q], U, acc[q]);
                    slot[q] = s0[q] + lane < s1[q] ? s0[q] + lane : -1;
                }
            }
#pragma unroll
            for (int q = 0; q < GP; q++) {
                done_acc[q] = acc[q];
                done_slot[q] = slot[q];
                n[q] = nn[q];
            }
            meta = meta_n;
            meta_n = meta_nn;
            g = g1; g1 = g2;
            e = e1; e1 = e2;
            pack_longest = pack_longestn; pack_longestn = pack_longestnn;
        }
#pragma unroll
        for (int q = 0; q < GP; q++)
            if (done_slot[q] >= 0) partial[done_slot[q]] = done_acc[q];

        }
        if constexpr (!HEAVY) break;
        __syncthreads();
        }
    };

    // The worker's ranges, one after the other (run_range is expanded once, here):
    //   phase 0, fixed part (Section 3.3): the group list is cut into P contiguous ranges of
    //     equal weight; worker w runs, column by column, the groups of its range below comp_lo[w].
    //     The groups from comp_lo[w] on, all in the last column of the range, are its competitive
    //     part: the worker goes on, without a break, to claim them piece by piece from the range's
    //     counter (the segment of x is staged already), and so may others;
    //   phase 2, competitive part: the counter of a range holds how many of its competitive groups
    //     have been claimed; a worker that has run out of work moves to the range with the most
    //     weight left (and stages the segment of x of that range's last column), until no range
    //     has enough left to be worth entering.  So a range that takes longer than its weight said is finished by the workers
    //     that were faster than theirs;
    //   phase 3 instead of 2, the paper's schedule: one ticket counter over the blocks that were not pre-assigned.
    const bool competitive = L.competitive != 0 && uniform_load(L.any_open, 0) != 0;
    int32_t col = uniform_load(L.fixed_col, worker);
    int32_t g_next = uniform_load(L.fixed_start, worker);
    const int32_t g_stop = uniform_load(L.fixed_start, worker + 1);
    const int32_t own_lo = uniform_load(L.ticket_b0 >= 0 ? L.comp_lo : L.own_end, worker);
    for (int phase = 0;;) {
        int32_t r_bn = 0, r_g0 = 0, r_g1 = 0, r_owner = worker, r_lo = own_lo, r_end = g_stop;
        bool r_compete = true;
        if (phase == 0) {
            bool found = false;
            while (g_next < g_stop && !found) {
                const int32_t c_end = uniform_load(L.col_group_ptr, col + 1);
                if (g_next >= c_end) { col++; continue; }  // columns without groups
                const int32_t ge = min(g_stop, c_end), fe = max(g_next, min(ge, own_lo));
                const bool last = ge == g_stop;
                if (g_next < fe || (last && competitive && own_lo < g_stop)) {
                    r_bn = col;
                    // (an empty fixed part is handed over as [0, 0): the ends of a worker's
                    // successive ranges must grow, and claimed ranges start at comp_lo)
                    r_g0 = g_next < fe ? g_next : 0;
                    r_g1 = g_next < fe ? fe : 0;
                    r_compete = last && competitive && own_lo < g_stop;
                    found = true;
                }
                g_next = ge;
            }
            if (!found) {
                if (L.ticket_b0 >= 0) { phase = 3; continue; }
                if (!competitive) break;
                phase = 2;
                continue;
            }
        } else if (phase == 3) {
            // The paper's own competitive part (Section 3.3, when the handle was built for it): the
            // blocks behind the pre-assigned ones are claimed one at a time through a single ticket
            // counter; whoever holds a ticket fetches that block's segment of x and walks the block.
            if (threadIdx.x == 0) sh_next = (int32_t)atomicAdd(&col_ticket[0], 1u);
            __syncthreads();
            const int64_t b = (int64_t)L.ticket_b0 + (uint32_t)sh_next;
            __syncthreads();  // sh_next is rewritten in the next turn
            if (b >= L.B) break;
            r_bn = L.blk_bn[b];
            r_g0 = L.blk_group_ptr[b];
            r_g1 = L.blk_group_ptr[b + 1];
            r_compete = false;
        } else {
            if (wave == 0) {
                int32_t best = -1;
                uint32_t best_left = 0;
                for (int32_t v0 = 0; v0 < L.P; v0 += 64) {
                    int32_t v = v0 + lane;
                    uint32_t left = 0;
                    if (v < L.P) {
                        // weight of the competitive groups of range v that nobody has claimed; a range
                        // with less left than entering it costs (staging its segment of x, about two
                        // block columns' weight counting the pipeline restart) is left to those who
                        // are there already
                        const int32_t end = L.fixed_start[v + 1];
                        const int64_t total = end - L.comp_lo[v];
                        const int64_t used = (int64_t)__hip_atomic_load(&col_ticket[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (used < total) {
                            const int32_t g = L.comp_lo[v] + (int32_t)used;
                            auto before = [&](int32_t i) {
                                return (int64_t)L.group_ptr[i] + (int64_t)L.SW * L.group_slot[i] + (int64_t)L.RW * L.group_rounds[i] +
                                       (int64_t)L.GW * i;
                            };
                            const int64_t w_left = before(end) - before(g);
                            left = w_left < L.steal_min ? 0u : w_left > 0xffffffffll ? 0xffffffffu : (uint32_t)w_left;
                        }
                    }
#pragma unroll
                    for (int d = 32; d > 0; d >>= 1) {
                        const uint32_t o_left = __shfl_xor(left, d);
                        const int32_t o_v = __shfl_xor(v, d);
                        if (o_left > left || (o_left == left && o_v < v)) { left = o_left; v = o_v; }
                    }
                    if (left > best_left) { best_left = left; best = v; }
                }
                if (lane == 0) sh_next = best;
            }
            __syncthreads();
            r_owner = sh_next;
            __syncthreads();  // sh_next is rewritten in the next turn
            if (r_owner < 0) break;
            r_bn = L.comp_col[r_owner];
            r_lo = L.comp_lo[r_owner];
            r_end = L.fixed_start[r_owner + 1];
        }
        run_range(r_bn, r_g0, r_g1, r_compete, r_owner, r_lo, r_end);
    }
    // Row blocks that the combine part cuts into several units are summed into y with atomic
    // adds: their rows of y start at zero.  (Done last: in front of the first range it delays
    // every worker's start.)
    for (int32_t ms = (int32_t)blockIdx.x; ms < L.NM; ms += n_workers) {
        const int64_t r0 = (int64_t)L.multi_stripes[ms] * L.R;
        const int32_t rows = (int32_t)min((int64_t)L.R, L.n_rows - r0);
        for (int32_t r = threadIdx.x; r < rows; r += THREADS) y[r0 + r] = T(0);
    }
}

// SpMV part of a small matrix (flat_wavefronts says which): one group after the other across the grid, no
// workers, no schedule, x read straight from L2.  Bound by latency: a group's chain is metadata -> lane
// lengths -> columns and values -> x, four dependent loads, and every group of the matrix is in flight at
// once.  (5-point grid of 64 x 64: 16 us for k_spmv_part and 6.6 us for the combine part -> 3.8 us for this
// kernel, which then writes y itself.)
// Workgroups of 16 wavefronts.  The first n_long take one of the matrix's long groups (is_long_group) each,
// cut at rounds into 16 pieces of equal nonzeros: one wavefront walks such a group at U rounds per memory
// round trip (R-MAT of 2^16 rows: 722 us without, 40 us with them).  The others take 16 / WPG groups, WPG
// wavefronts per group, wavefront w of them the rounds U w .. U w + U - 1, then those U WPG further on, ...;
// round k starts at the group's first position plus the sum over its rows of min(length, k).  The sums of a
// group's wavefronts meet in LDS, in wavefront order.
// DIRECT: the matrix has one block column, so a row has one slot at most and the slot's sum is y's
// value: it is stored there too and no combine part follows.  The last NBR workgroups of the grid
// (only launched where rows are empty) then write the zeros of the rows without a slot.
template <int WPG, int U, bool DIRECT, typename T>
__global__ __launch_bounds__(1024) void k_spmv_flat(Layout L, const T *__restrict__ x, T *__restrict__ partial, T *__restrict__ y,
                                                    int32_t n_long, int32_t group_wgs)
{
    constexpr int kThreads = 1024, kWaves = 16, kGroups = kWaves / WPG;
    __shared__ T sh_sum[kThreads];
    __shared__ int32_t sh_left[kThreads];  // per wavefront: rounds left in the rows it is folded onto
    __shared__ int32_t sh_len[64];
    __shared__ int32_t sh_cut_k[kWaves + 1];
    const T *__restrict__ const data = static_cast<const T *>(L.data);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t wg = (int32_t)blockIdx.x - n_long;
    if (DIRECT && wg >= group_wgs) {
        uint32_t *present = reinterpret_cast<uint32_t *>(sh_left);  // a bit per row of the row block
        const int32_t bm = wg - group_wgs;
        const int64_t r0 = (int64_t)bm * L.R;
        const int32_t rows = (int32_t)min((int64_t)L.R, L.n_rows - r0);
        for (int32_t i = threadIdx.x; i < kMaxR / 32; i += kThreads) present[i] = 0u;
        __syncthreads();
        for (int32_t k = L.stripe_ptr[bm]; k < L.stripe_ptr[bm + 1]; k++) {
            const int32_t b = L.stripe_blk[k];
            for (int32_t s = L.slot_ptr[b] + (int32_t)threadIdx.x; s < L.slot_ptr[b + 1]; s += kThreads) {
                const uint32_t r = L.row_local[s];
                atomicOr(&present[r >> 5], 1u << (r & 31u));
            }
        }
        __syncthreads();
        for (int32_t i = threadIdx.x; i < rows; i += kThreads)
            if (!((present[i >> 5] >> (i & 31)) & 1u)) y[r0 + i] = T(0);
        return;
    }
    // rows of y that the combine part adds into with atomics start at zero (see k_spmv_part)
    if constexpr (!DIRECT)
        for (int32_t ms = (int32_t)blockIdx.x; ms < L.NM; ms += (int32_t)gridDim.x) {
            const int64_t r0 = (int64_t)L.multi_stripes[ms] * L.R;
            const int32_t rows = (int32_t)min((int64_t)L.R, L.n_rows - r0);
            for (int32_t r = threadIdx.x; r < rows; r += kThreads) y[r0 + r] = T(0);
        }
    const bool is_long = wg < 0;
    const int part = is_long ? wave : wave % WPG;
    int32_t g = is_long ? uniform_load(L.long_groups, (int32_t)blockIdx.x) : wg * kGroups + wave / WPG;
    int32_t s0 = 0, s1 = 0, bn = 0, bm = 0;
    uint32_t first = 0;
    if (!is_long && (g >= L.G || is_long_group(uniform_load(L.group_ptr, g + 1) - uniform_load(L.group_ptr, g),
                                              uniform_load(L.group_rounds, g + 1) - uniform_load(L.group_rounds, g), WPG))) {
        if (WPG == 1) return;  // no barrier below
    } else {
        s0 = uniform_load(L.group_slot, g);
        s1 = uniform_load(L.group_slot, g + 1);
        first = (uint32_t)uniform_load(L.group_ptr, g);
        const int32_t b = uniform_load(L.group_blk, g);
        bn = uniform_load(L.blk_bn, b);
        if (DIRECT) bm = uniform_load(L.blk_bm, b);
    }
    const bool mine = s0 + lane < s1;
    const int32_t n = mine ? (int32_t)L.seg_len[s0 + lane] : 0;
    uint32_t row = 0;
    if (DIRECT && part == 0 && mine) row = L.row_local[s0 + lane];
    const T *const xs = x + (int64_t)bn * L.C;
    // U steps of the lanes' rows from step k on; `base` is the position of step k and advances past them
    auto add_steps = [&](uint32_t &base, int32_t steps, int32_t k) __attribute__((always_inline)) {
        Batch<U, T> bt;
        issue_batch<U>(bt, L.col_local, data, base, steps, k);
        T xv[U], sum = T(0);
#pragma unroll
        for (int u = 0; u < U; u++) xv[u] = xs[k + u < steps ? bt.c[u] : 0u];  // never index x with a foreign column
#pragma unroll
        for (int u = 0; u < U; u++) {
            const T more = fma_of(bt.v[u], xv[u], sum);
            sum = k + u < steps ? more : sum;
        }
        return sum;
    };
    T acc = T(0);
    // rounds k, k + 1, ... of the group until no lane has any left (up to end); `base` is the position of round k
    auto walk = [&](uint32_t base, int32_t end, int32_t k) __attribute__((always_inline)) {
        int32_t *left = sh_left + wave * 64;
        T *hand = sh_sum + wave * 64;
        for (;;) {
            const uint64_t live = __ballot(k < end);
            if (!live) break;
            const int32_t m = __popcll(live);
            if (m > 32 || !__ballot(k + U < end)) {
                acc += add_steps(base, end, k);
                k += U;
                continue;
            }
            // few rows left, one of them for a while: the wavefront is folded, lane j * mm + c serving the c-th live row in the
            // rounds k + j, k + j + 64 / mm, ... (see walk_rounds in k_spmv_part)
            const int sh = m > 16 ? 5 : m > 8 ? 4 : m > 4 ? 3 : m > 2 ? 2 : m > 1 ? 1 : 0;  // mm = 2^sh
            left[lane] = 0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (k < end) left[lanes_below(live)] = end - k;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int32_t rest = left[lane & ((1 << sh) - 1)], j = lane >> sh;
            const int32_t steps = rest > j ? (rest - j + (64 >> sh) - 1) >> (6 - sh) : 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            hand[lane] = add_steps(base, steps, 0);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (k < end)
                for (int32_t t = lanes_below(live); t < 64; t += 1 << sh) acc += hand[t];
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            k += U << (6 - sh);
        }
    };
    if (is_long) {
        const uint32_t total = (uint32_t)uniform_load(L.group_ptr, g + 1) - first;
        if (wave == 0) sh_len[lane] = n;
        __syncthreads();
        int32_t k;
        uint32_t base;
        cut_rounds(sh_len, (uint32_t)(((uint64_t)total * (uint32_t)wave) / kWaves), lane, k, base);
        base += first;
        if (lane == 0) sh_cut_k[wave] = k;
        if (threadIdx.x == 0) sh_cut_k[kWaves] = 0x10000;
        __syncthreads();
        walk(base, min(n, sh_cut_k[wave + 1]), k);
    } else if constexpr (WPG == 1) {
        walk(first, n, 0);
    } else {
        uint32_t base = first;
        for (int32_t k = U * part; __ballot(k < n); k += U * WPG) {
            if (WPG > 1 && k > 0) {  // position of round k
                uint32_t before = (uint32_t)min(n, k);
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) before += __shfl_xor(before, d);
                base = first + before;
            }
            acc += add_steps(base, n, k);
        }
    }
    if (WPG > 1 || is_long) {
        const int count = is_long ? kWaves : WPG;
        sh_sum[threadIdx.x] = acc;
        __syncthreads();
        if (part != 0) return;
        for (int w = 1; w < count; w++) acc += sh_sum[(wave + w) * 64 + lane];
    }
    if (mine) {
        partial[s0 + lane] = acc;
        if constexpr (DIRECT) y[(int64_t)bm * L.R + row] = acc;
    }
}

// Combine part (Fig. 1): one workgroup per row block adds the partial sums of that row block's
// blocks into LDS copies of its y slice and writes the slice out, zeros included.  The slot
// ranges of up to kPass blocks are fetched in parallel first; then wavefronts take blocks
// round-robin and lanes stride over a block's slots.  With kRing > 0 a wavefront keeps a ring of
// kRing chunks of 64 kChunk slots in flight across its blocks (the kernel is bound by the bytes
// it has in flight); with kRing = 0 it walks block by block, four loads per lane at a time, and
// loads the small blocks of a pass together.
// Every wavefront accumulates into its own copy of the slice with plain LDS read-add-write:
// a block holds a row at most once, so the lanes of one instruction never collide, and a
// wavefront's LDS accesses complete in order.  (LDS float atomics would allow one shared copy
// but run an order of magnitude slower on this hardware.)  The copies are summed on the way out.
// Also re-arms the per-column ticket counters for the next call (the SpMV part of this call
// has finished: same stream).
template <int THREADS, typename T, int kRing, int kChunk>
__global__ __launch_bounds__(THREADS) void k_combine(Layout L, const T *__restrict__ partial, T *__restrict__ y,
                                                     uint32_t *__restrict__ ticket)
{
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    T *const ys_all = reinterpret_cast<T *>(dyn_lds);  // kWaves copies of R values
    constexpr int kPass = 128, kWaves = THREADS / 64;
    __shared__ int32_t range[2 * kPass];
    static_assert(kRing == 0 || sizeof(range) == kCombineStaticLds, "what combine_units_by_lds counts for it");
    // One workgroup per combine unit: entries [unit_k[j], unit_k[j + 1]) of stripe_blk, all of row
    // block bm.  A row block with a single unit is stored; the units of a split row block add
    // their sums into y, which the SpMV part has zeroed.
    const int32_t unit = blockIdx.x;
    const int32_t bm = L.unit_stripe[unit];
    const bool split = L.unit_ptr[bm + 1] - L.unit_ptr[bm] > 1;
    for (int64_t i = (int64_t)unit * THREADS + threadIdx.x; i < L.P; i += (int64_t)gridDim.x * THREADS) ticket[i] = 0u;
    const int64_t r0 = (int64_t)bm * L.R;
    const int32_t rows = (int32_t)min((int64_t)L.R, L.n_rows - r0);
    for (int32_t i = threadIdx.x; i < kWaves * L.R; i += THREADS) ys_all[i] = T(0);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    T *ys = ys_all + wave * L.R;
    const int32_t k1 = L.unit_k[unit + 1];
    for (int32_t k0 = L.unit_k[unit]; k0 < k1; k0 += kPass) {
        const int32_t nb = min(kPass, k1 - k0);
        __syncthreads();  // slices zeroed / previous pass done with range[]
        constexpr int kTogether = 4, kFirst = 4;
        int small = 0;  // does the pass hold a block with few slots?
        for (int32_t t = threadIdx.x; t < nb; t += THREADS) {
            const int32_t b = L.stripe_blk[k0 + t];
            const int32_t first = L.slot_ptr[b], end = L.slot_ptr[b + 1];
            range[2 * t] = first;
            range[2 * t + 1] = end;
            small |= end - first <= 64 * kFirst;
        }
        if constexpr (kRing > 0) {
            __syncthreads();
            // A ring of kRing chunks of up to 64 kChunk consecutive slots of one block is kept in
            // flight per wavefront: the chunks of a wavefront's blocks follow each other whatever
            // the blocks' sizes, and a chunk is added (read all, then write all: its slots are
            // distinct rows) while the loads of the next kRing - 1 are on their way.
            int32_t next_block = wave, cur = 0, cur_end = 0;
            int32_t c0[kRing], c1[kRing];
            uint32_t r[kRing][kChunk];
            T p[kRing][kChunk];
            auto issue = [&](int d) __attribute__((always_inline)) {
                while (cur >= cur_end && next_block < nb) {
                    cur = __builtin_amdgcn_readfirstlane(range[2 * next_block]);
                    cur_end = __builtin_amdgcn_readfirstlane(range[2 * next_block + 1]);
                    next_block += kWaves;
                }
                c0[d] = cur;
                c1[d] = min(cur + 64 * kChunk, cur_end);
                cur = c1[d];
#pragma unroll
                for (int u = 0; u < kChunk; u++) {
                    r[d][u] = 0;
                    p[d][u] = T(0);
                    if (c0[d] + 64 * u < c1[d]) {  // wave-uniform; clamped: always a slot of this chunk
                        const int32_t idx = min(c0[d] + lane + 64 * u, c1[d] - 1);
                        r[d][u] = L.row_local[idx];
                        p[d][u] = partial[idx];
                    }
                }
            };
#pragma unroll
            for (int d = 0; d < kRing; d++) issue(d);
            while (c1[0] > c0[0]) {  // chunks are issued in order: when this one is empty, all are
#pragma unroll
                for (int d = 0; d < kRing; d++) {
                    if (c1[d] > c0[d]) {
                        T o[kChunk];
#pragma unroll
                        for (int u = 0; u < kChunk; u++) o[u] = ys[r[d][u]];
#pragma unroll
                        for (int u = 0; u < kChunk; u++)
                            if (c0[d] + lane + 64 * u < c1[d]) ys[r[d][u]] = o[u] + p[d][u];
                    }
                    issue(d);
                }
            }
            continue;
        }
        if (!__syncthreads_or(small)) {
            // only blocks with many slots: wavefronts take them one by one, KU slots per lane in
            // flight (the kernel is bound by the bytes it has in flight); the slots of a step are
            // distinct rows of one block: read all, then write all
            for (int32_t i = wave; i < nb; i += kWaves) {
                const int32_t s0 = range[2 * i], s1 = range[2 * i + 1];
                auto add_block = [&](auto ku) __attribute__((always_inline)) {
                    constexpr int KU = decltype(ku)::value;
                    for (int32_t s = s0 + lane; s < s1; s += 64 * KU) {
                        uint32_t r[KU];
                        T p[KU], o[KU];
#pragma unroll
                        for (int u = 0; u < KU; u++) {
                            const int32_t idx = min(s + 64 * u, s1 - 1);  // clamped: always a slot of this block
                            r[u] = L.row_local[idx];
                            p[u] = partial[idx];
                        }
#pragma unroll
                        for (int u = 0; u < KU; u++) o[u] = ys[r[u]];
#pragma unroll
                        for (int u = 0; u < KU; u++)
                            if (s + 64 * u < s1) ys[r[u]] = o[u] + p[u];
                    }
                };
                add_block(std::integral_constant<int, 4>{});
            }
            continue;
        }
        // A wavefront takes kTogether blocks at a time.  Blocks with few slots are one load deep:
        // taken one by one, a wavefront would sit through a memory latency per block.  So the
        // slots of those of the kTogether blocks that have at most 64 kFirst of them are loaded
        // first; then the blocks are added one after the other (a row occurs once per block but
        // may occur in several blocks), a larger block with KU slots per lane in flight (the
        // kernel is bound by the bytes it has in flight).
        for (int32_t i0 = wave; i0 < nb; i0 += kWaves * kTogether) {
            int32_t b0[kTogether], b1[kTogether];
            uint32_t rf[kTogether][kFirst];
            T pf[kTogether][kFirst];
#pragma unroll
            for (int j = 0; j < kTogether; j++) {
                const int32_t i = i0 + j * kWaves;
                b0[j] = b1[j] = 0;
                if (i < nb) { b0[j] = range[2 * i]; b1[j] = range[2 * i + 1]; }
                const int32_t slots = b1[j] - b0[j];  // 0 for a block that does not exist
#pragma unroll
                for (int u = 0; u < kFirst; u++) {
                    rf[j][u] = 0;
                    pf[j][u] = T(0);
                    if (slots > 64 * u && slots <= 64 * kFirst) {  // wave-uniform; clamped: always a slot of this block
                        const int32_t idx = min(b0[j] + lane + 64 * u, b1[j] - 1);
                        rf[j][u] = L.row_local[idx];
                        pf[j][u] = partial[idx];
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kTogether; j++) {
                const int32_t s0 = b0[j], s1 = b1[j], slots = s1 - s0;
                if (slots <= 64 * kFirst) {  // wave-uniform
                    if (slots <= 0) continue;
                    // the slots of a step are distinct rows of one block: read all, then write all
                    T o[kFirst];
#pragma unroll
                    for (int u = 0; u < kFirst; u++) o[u] = ys[rf[j][u]];
#pragma unroll
                    for (int u = 0; u < kFirst; u++)
                        if (s0 + lane + 64 * u < s1) ys[rf[j][u]] = o[u] + pf[j][u];
                    continue;
                }
                auto add_block = [&](auto ku) __attribute__((always_inline)) {
                    constexpr int KU = decltype(ku)::value;
                    for (int32_t s = s0 + lane; s < s1; s += 64 * KU) {
                        uint32_t r[KU];
                        T p[KU], o[KU];
#pragma unroll
                        for (int u = 0; u < KU; u++) {
                            const int32_t idx = min(s + 64 * u, s1 - 1);  // clamped: always a slot of this block
                            r[u] = L.row_local[idx];
                            p[u] = partial[idx];
                        }
#pragma unroll
                        for (int u = 0; u < KU; u++) o[u] = ys[r[u]];
#pragma unroll
                        for (int u = 0; u < KU; u++)
                            if (s + 64 * u < s1) ys[r[u]] = o[u] + p[u];
                    }
                };
                add_block(std::integral_constant<int, 4>{});
            }
        }
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < rows; i += THREADS) {
        T sum = ys_all[i];
#pragma unroll
        for (int w = 1; w < kWaves; w++) sum += ys_all[w * L.R + i];
        if (split) atomicAdd(&y[r0 + i], sum);
        else y[r0 + i] = sum;
    }
}

// ------------------------------------------------------------------ CSR baselines (Algorithm 1)

template <typename T>
__global__ __launch_bounds__(256) void k_csr_scalar(const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                                    const T *__restrict__ val, const T *__restrict__ x,
                                                    T *__restrict__ y, int64_t n_rows)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_rows) return;
    T sum = T(0);
    for (int32_t j = ptr[i]; j < ptr[i + 1]; j++) sum += val[j] * x[col[j]];
    y[i] = sum;
}

// LPR lanes per row (a power of two below 64): the mapping between one thread and one wavefront per
// row, for matrices whose rows hold a few to a few dozen nonzeros.
template <int LPR, typename T>
__global__ __launch_bounds__(256) void k_csr_sub(const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                                 const T *__restrict__ val, const T *__restrict__ x,
                                                 T *__restrict__ y, int64_t n_rows)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t i = t / LPR;
    const int sub = (int)(t % LPR);
    T sum = T(0);
    if (i < n_rows)
        for (int32_t j = ptr[i] + sub; j < ptr[i + 1]; j += LPR) sum += val[j] * x[col[j]];
#pragma unroll
    for (int d = LPR / 2; d > 0; d >>= 1) sum += __shfl_xor(sum, d);  // stays inside the row's LPR lanes
    if (i < n_rows && sub == 0) y[i] = sum;
}

template <typename T>
__global__ __launch_bounds__(256) void k_csr_vector(const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                                    const T *__restrict__ val, const T *__restrict__ x,
                                                    T *__restrict__ y, int64_t n_rows)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_rows) return;
    T sum = T(0);
    for (int32_t j = ptr[i] + lane; j < ptr[i + 1]; j += 64) sum += val[j] * x[col[j]];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if (lane == 0) y[i] = sum;
}

}  // namespace

// Raises a kernel's dynamic-LDS cap on `device` (the attribute is per device).  `done` has a bit
// per device and is only a fast path: the call is idempotent, so two threads that both find the
// bit clear may both make it.
template <typename K>
static int raise_lds_cap(std::atomic<uint64_t> &done, int device, K kernel, int bytes)
{
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return HBP_OK;
    HBP_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    if (bit) done.fetch_or(bit, std::memory_order_release);
    return HBP_OK;
}

template <int THREADS, int U, int GP, bool HEAVY, bool STEPS, typename T>
static int launch_part(const hbp_handle_s *h, const Layout &L, const T *x, T *y, hipStream_t st, SpmvScratch sc)
{
    const size_t lds = (size_t)h->C * sizeof(T);
    static std::atomic<uint64_t> configured{0};  // per instantiation
    const int rc = raise_lds_cap(configured, h->device, k_spmv_part<THREADS, U, GP, HEAVY, STEPS, T>,
                                 kMaxC * (int)sizeof(float));  // 128 KB: kMaxC floats or kMaxC64 doubles
    if (rc != HBP_OK) return rc;
    k_spmv_part<THREADS, U, GP, HEAVY, STEPS, T><<<dim3((unsigned)h->P), THREADS, lds, st>>>(L, x, static_cast<T *>(sc.partial), y, sc.ticket);
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

template <int THREADS, bool HEAVY, typename T>
static int launch_part_u(const hbp_handle_s *h, const Layout &L, const T *x, T *y, hipStream_t st, SpmvScratch sc)
{
    // fp64: half as many groups at once, or the batches spill (128 registers per lane whatever the workgroup size).
    // (256 and 512 threads with all eight or four: 64 to 196 registers spilled; 3M rows of 1 to 5 nonzeros over 7900 columns 96 against
    // 58 us, 1M lognormal rows in blocks of 7900 columns 472 against 155.)
    constexpr int kHalf = sizeof(T) == 8 ? 2 : 1;
    if constexpr (sizeof(T) == 4)
        if (walk_in_steps(h->unroll, L.lists_first, h->nnz, h->G)) return launch_part<THREADS, 4, 4, HEAVY, true, T>(h, L, x, y, st, sc);
    switch (h->unroll) {  // rounds per batch; short batches walk several groups at once
    case 2: return launch_part<THREADS, 2, 4 / kHalf, HEAVY, false, T>(h, L, x, y, st, sc);  // (eight: up to 45 registers spilled, 119 against 80 us)
    case 4: return launch_part<THREADS, 4, 4 / kHalf, HEAVY, false, T>(h, L, x, y, st, sc);
    case 9: return launch_part<THREADS, 9, 1, HEAVY, false, T>(h, L, x, y, st, sc);
    case 16: return launch_part<THREADS, 16, 1, HEAVY, false, T>(h, L, x, y, st, sc);
    default: return launch_part<THREADS, 8, 1, HEAVY, false, T>(h, L, x, y, st, sc);
    }
}

template <typename T>
static int launch_flat(const hbp_handle_s *h, const Layout &L, const T *x, T *y, hipStream_t st, SpmvScratch sc)
{
    const bool direct = h->NBC == 1;
    auto go = [&](auto wpg) {
        constexpr int WPG = decltype(wpg)::value, U = 8, kGroups = 16 / WPG;
        const int32_t group_wgs = (int32_t)((h->G + kGroups - 1) / kGroups), n_long = h->n_long;
        if (direct) {
            const int64_t wgs = (int64_t)n_long + group_wgs + (h->S < h->n_rows ? h->NBR : 0);
            k_spmv_flat<WPG, U, true, T><<<dim3((unsigned)wgs), 1024, 0, st>>>(L, x, static_cast<T *>(sc.partial), y, n_long, group_wgs);
        } else {
            k_spmv_flat<WPG, U, false, T><<<dim3((unsigned)(n_long + group_wgs)), 1024, 0, st>>>(L, x, static_cast<T *>(sc.partial), y, n_long, group_wgs);
        }
    };
    if (h->flat_wpg == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 4>{});
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

template <typename T>
static int launch_part_t(const hbp_handle_s *h, const T *x, T *y, hipStream_t st, SpmvScratch sc)
{
    const Layout L = hbp_view(h);
    if (h->flat_wpg) return launch_flat<T>(h, L, x, y, st, sc);
    // the kernel that can share heavy groups among a worker's wavefronts only where the matrix has one
    if (h->longest_segment > L.long_rounds) {
        if (h->threads == 1024) return launch_part_u<1024, true, T>(h, L, x, y, st, sc);
        if (h->threads == 512) return launch_part_u<512, true, T>(h, L, x, y, st, sc);
        return launch_part_u<256, true, T>(h, L, x, y, st, sc);
    }
    if (h->threads == 1024) return launch_part_u<1024, false, T>(h, L, x, y, st, sc);
    if (h->threads == 512) return launch_part_u<512, false, T>(h, L, x, y, st, sc);
    return launch_part_u<256, false, T>(h, L, x, y, st, sc);
}

template <typename T>
static int launch_combine_t(const hbp_handle_s *h, T *y, hipStream_t st, SpmvScratch sc)
{
    const Layout L = hbp_view(h);
    const T *partial = static_cast<const T *>(sc.partial);
    if (h->flat_wpg && h->NBC == 1) return HBP_OK;  // k_spmv_flat has written y
    if (h->R <= 1024) {
        // two copies of a short slice: enough workgroups per CU for the plain block-by-block walk
        k_combine<128, T, 0, 0><<<dim3((unsigned)h->U), 128, 2 * (size_t)h->R * sizeof(T), st>>>(L, partial, y, sc.ticket);
    } else {
        // a copy per wavefront (up to 128 KB in all: kMaxR floats or kMaxR64 doubles for four of them); a ring
        // of chunks in flight, shorter chunks and more of them where the blocks hold few slots on average
        auto go = [&](auto kt, auto kr, auto kc) {
            constexpr int KT = decltype(kt)::value, KR = decltype(kr)::value, KC = decltype(kc)::value;
            static std::atomic<uint64_t> configured{0};  // per instantiation
            const int rc = raise_lds_cap(configured, h->device, k_combine<KT, T, KR, KC>, kCombineLds);
            if (rc != HBP_OK) return rc;
            k_combine<KT, T, KR, KC><<<dim3((unsigned)h->U), KT, KT / 64 * (size_t)h->R * sizeof(T), st>>>(L, partial, y, sc.ticket);
            return (int)HBP_OK;
        };
        auto pick = [&](auto kt) {
            return h->S < 128 * h->B ? go(kt, std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{})
                                     : go(kt, std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
        };
        int rc = HBP_OK;
        switch (combine_wavefronts(h->cus, h->U, h->R, (int32_t)sizeof(T))) {
        case 16: rc = pick(std::integral_constant<int, 1024>{}); break;
        case 8: rc = pick(std::integral_constant<int, 512>{}); break;
        case 3: rc = pick(std::integral_constant<int, 192>{}); break;
        default: rc = pick(std::integral_constant<int, 256>{}); break;
        }
        if (rc != HBP_OK) return rc;
    }
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

template <typename T>
static int launch_csr_t(int kind, const int32_t *ptr, const int32_t *col, const T *val, const T *x, T *y, int64_t n_rows,
                        hipStream_t st)
{
    auto sub = [&](auto lanes) {
        constexpr int LPR = decltype(lanes)::value;
        k_csr_sub<LPR, T><<<dim3((unsigned)((n_rows * LPR + 255) / 256)), 256, 0, st>>>(ptr, col, val, x, y, n_rows);
    };
    switch (kind) {
    case 0: k_csr_scalar<T><<<dim3((unsigned)((n_rows + 255) / 256)), 256, 0, st>>>(ptr, col, val, x, y, n_rows); break;
    case 1: k_csr_vector<T><<<dim3((unsigned)((n_rows + 3) / 4)), 256, 0, st>>>(ptr, col, val, x, y, n_rows); break;
    case 2: sub(std::integral_constant<int, 2>{}); break;
    case 4: sub(std::integral_constant<int, 4>{}); break;
    case 8: sub(std::integral_constant<int, 8>{}); break;
    case 16: sub(std::integral_constant<int, 16>{}); break;
    case 32: sub(std::integral_constant<int, 32>{}); break;
    default: return HBP_ERR_INVALID_ARGUMENT;
    }
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

}  // namespace hbp
