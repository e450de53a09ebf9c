// HBP preprocessing on the GPU: CSR -> compact HBP layout (Sections 3.1-3.3 of the paper).
//
// The paper's Algorithm 2 walks one matrix row per thread and inserts rows into a per-block
// hash table with atomics.  Here the same quantities are produced with coalesced passes
// over the CSR arrays and a deterministic placement:
//   1-3. segments, counted the row pointers are checked; a nonzero starts a segment when it starts a row or its column
//                          block differs from its left neighbour's (Algorithm 2's inner
//                          while loop, evaluated for all nonzeros at once); segments per
//                          (column block, row block), and a list of the segments
//   4. block table         scans give each non-empty block its slot range, group range and
//                          list position
//   5. segments, placed    every segment drops (length, local row, first nonzero) into its
//                          block's slot range through an atomic cursor
//   6. block ordering      each block's range is ordered by (key, local row) in LDS; the
//                          pair is unique inside a block, so the result does not depend on
//                          the order in which step 5's atomics were served.  This is the
//                          deterministic limit of the paper's atomic hash-table insertion.
//   7. fill                one wavefront per group writes col/data round by round
//                          (column-major inside the group, Section 3.2 last paragraph)
// Where row segments are short, steps 5 to 7 are done by row blocks as a whole instead (k_panel_slots, k_panel_fill), with the same result.
#include "hbp_internal.h"

#include <chrono>
#include <mutex>
#include <type_traits>
#include <vector>

namespace hbp {
namespace {

constexpr int32_t kErrPtr = 1, kErrCol = 2;  // bits of the device-side error word

__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Element i of an array whose address is the same in all lanes: an access by the array's address in scalar registers and a 32-bit offset in a
// vector register (an index added to a pointer costs 64-bit vector arithmetic per access), but for stores in loops, whose vector address
// the compiler steps on.  By way of bytes, not of an integer: an address that has been an integer may be LDS for all the compiler knows,
// and a flat access has no scalar address and waits with the LDS ones (k_order_block, 13 of its accesses flat / none: lognormal 4M x 1M 365 / 360
// us, R-MAT 2^20 in fp64 126 / 124.5, 27-point grid of 128^3 35.9 / 35.4).  sizeof(T) i < 2^32.
template <typename T>
__device__ __forceinline__ T &lane_at(T *uniform, uint32_t i)
{
    using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *reinterpret_cast<T *>(reinterpret_cast<Byte *>(uniform) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// Inclusive sum over the lanes; sum and maximum over the wavefront, the same in all lanes (row shifts and broadcasts inside the vector ALU: six instructions each, no
// LDS).  All lanes have to be active.
template <int kControl, int kRows>
__device__ __forceinline__ uint32_t lanes_moved(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kControl, kRows, 0xf, false); }
__device__ __forceinline__ uint32_t sum_up_to_lane(uint32_t v)
{
    v += lanes_moved<0x111, 0xf>(v);  // from 1, 2, 4, 8 lanes below in the row of 16 (0 where there is none)
    v += lanes_moved<0x112, 0xf>(v);
    v += lanes_moved<0x114, 0xf>(v);
    v += lanes_moved<0x118, 0xf>(v);
    v += lanes_moved<0x142, 0xa>(v);  // lane 15 of a row to the next row: rows 1 and 3
    return v + lanes_moved<0x143, 0xc>(v);  // lane 31 to rows 2 and 3
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)sum_up_to_lane(v), 63); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max(v, lanes_moved<0x111, 0xf>(v));
    v = max(v, lanes_moved<0x112, 0xf>(v));
    v = max(v, lanes_moved<0x114, 0xf>(v));
    v = max(v, lanes_moved<0x118, 0xf>(v));
    v = max(v, lanes_moved<0x142, 0xa>(v));
    v = max(v, lanes_moved<0x143, 0xc>(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Exclusive scan of one value per thread over a 256-thread workgroup; *total is the
// workgroup sum.  sh needs 4 entries.
__device__ __forceinline__ uint32_t block_excl_scan_256(uint32_t v, uint32_t *total, uint32_t *sh)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(inc, d);
        if (lane >= d) inc += t;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    uint32_t woff = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        uint32_t s = sh[i];
        if (i < w) woff += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return woff + inc - v;
}

// ------------------------------------------------------------------ device-wide exclusive scans
//
// Up to five scans of arrays of one length go through the same launches: the arrays are short (tens of
// thousands of entries), so a scan costs its launches, some 5 us each, whatever it does.

enum { kOpIdentity = 0, kOpCeilDivW = 1, kOpNonZero = 2, kOpUnits = 3, kOpSplit = 4 };  // (the last two: combine units of W slots, see k_stripe_fill)
__device__ __forceinline__ uint32_t scan_input(int32_t op, uint32_t v, uint32_t W)
{
    return op == kOpCeilDivW ? (v + W - 1) / W : op == kOpNonZero ? (v ? 1u : 0u) : op == kOpUnits ? max(1u, (v + W - 1) / W) : op == kOpSplit ? (v > W ? 1u : 0u) : v;
}

constexpr int kScanTile = 2048;  // 256 threads x 8 consecutive items

// out[0..n) = exclusive scan of op(in), out[n] = total.  `in` and `out` may alias where only one scan reads `in`.
struct Scans {
    const uint32_t *in[5];
    uint32_t *out[5];
    int32_t op[5];
};

__global__ __launch_bounds__(256) void k_scan_reduce(Scans s, int64_t n, uint32_t W, int64_t n_tiles, uint32_t *__restrict__ tile_sum)
{
    __shared__ uint32_t sh[4];
    const int a = blockIdx.y;
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 8; i++)
        if (base + i < n) sum += scan_input(s.op[a], s.in[a][base + i], W);
    uint32_t total;
    block_excl_scan_256(sum, &total, sh);
    if (threadIdx.x == 0) tile_sum[a * n_tiles + blockIdx.x] = total;
}

// One workgroup per scan turns the tile sums into prefix sums in place (for more tiles than every
// workgroup of k_scan_down would want to add up by itself).
__global__ __launch_bounds__(256) void k_scan_tiles(uint32_t *__restrict__ tile_sum, int64_t n_tiles)
{
    __shared__ uint32_t sh[4];
    uint32_t *sums = tile_sum + blockIdx.x * n_tiles;
    uint32_t carry = 0;
    for (int64_t base = 0; base < n_tiles; base += 256) {
        int64_t i = base + threadIdx.x;
        uint32_t v = i < n_tiles ? sums[i] : 0u, total;
        uint32_t ex = block_excl_scan_256(v, &total, sh);
        if (i < n_tiles) sums[i] = carry + ex;
        carry += total;
    }
}

__global__ __launch_bounds__(256) void k_scan_down(Scans s, int64_t n, uint32_t W, int64_t n_tiles, int32_t prefixed,
                                                   const uint32_t *__restrict__ tile_sum)
{
    __shared__ uint32_t sh[4];
    const int a = blockIdx.y;
    const uint32_t *sums = tile_sum + a * n_tiles;
    uint32_t before = 0;
    if (prefixed) {
        before = sums[blockIdx.x];
    } else if (blockIdx.x > 0) {
        uint32_t part = 0;
        for (int64_t i = threadIdx.x; i < blockIdx.x; i += 256) part += sums[i];
        block_excl_scan_256(part, &before, sh);
    }
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
    uint32_t v[8], sum = 0;
#pragma unroll
    for (int i = 0; i < 8; i++) {
        v[i] = base + i < n ? scan_input(s.op[a], s.in[a][base + i], W) : 0u;
        sum += v[i];
    }
    uint32_t total;
    uint32_t run = before + block_excl_scan_256(sum, &total, sh);
#pragma unroll
    for (int i = 0; i < 8; i++) {
        if (base + i < n) s.out[a][base + i] = run;
        run += v[i];
    }
    if (blockIdx.x == n_tiles - 1 && threadIdx.x == 0) s.out[a][n] = before + total;
}

// Short scans in one launch in place of two: a workgroup per scan, 8192 items at a time.  4 to 6 us in place of 4.5 to 5 each for
// k_scan_reduce and k_scan_down; two of a build's five scans are as short on R-MAT 2^20 and the 4M x 1M lognormal matrix, three on the 27-point
// grid of 128^3, all of them on small matrices.
constexpr int64_t kScanAlone = 16384;
__global__ __launch_bounds__(1024) void k_scan_alone(Scans s, int64_t n, uint32_t W)
{
    __shared__ uint32_t sh[16];
    const int a = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t carry = 0;
    for (int64_t base0 = 0; base0 < n; base0 += 1024 * 8) {
        const int64_t base = base0 + (int64_t)threadIdx.x * 8;
        uint32_t v[8], sum = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            v[i] = base + i < n ? scan_input(s.op[a], s.in[a][base + i], W) : 0u;
            sum += v[i];
        }
        const uint32_t incl = sum_up_to_lane(sum);
        if (lane == 63) sh[wave] = incl;
        __syncthreads();
        uint32_t run = carry + incl - sum;
#pragma unroll
        for (int w = 0; w < 16; w++) {
            const uint32_t t = sh[w];
            if (w < wave) run += t;
            carry += t;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if (base + i < n) s.out[a][base + i] = run;
            run += v[i];
        }
    }
    if (threadIdx.x == 0) s.out[a][n] = carry;
}

// tile_tmp must hold `count` * ceil(n / 2048) entries.
int exclusive_scans(const Scans &s, int count, int64_t n, uint32_t W, uint32_t *tile_tmp, hipStream_t st)
{
    if (n <= 0) {
        for (int a = 0; a < count; a++) HBP_HIP(hipMemsetAsync(s.out[a], 0, sizeof(uint32_t), st));
        return HBP_OK;
    }
    if (n <= kScanAlone) {
        k_scan_alone<<<dim3(1, (unsigned)count), 1024, 0, st>>>(s, n, W);
        HBP_HIP(hipGetLastError());
        return HBP_OK;
    }
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    const dim3 grid((unsigned)tiles, (unsigned)count);
    const bool prefixed = tiles > 4096;
    k_scan_reduce<<<grid, 256, 0, st>>>(s, n, W, tiles, tile_tmp);
    if (prefixed) k_scan_tiles<<<dim3((unsigned)count), 256, 0, st>>>(tile_tmp, tiles);
    k_scan_down<<<grid, 256, 0, st>>>(s, n, W, tiles, prefixed ? 1 : 0, tile_tmp);
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

// ------------------------------------------------------------------ Section 3.2: hash

// key(n) = min(min(n >> a, 8) * b + (((n mod 2^a) * d) >> a), R - 1) with b = d = max(1, R / 9):
// aggregation (shift, rows beyond class 8 count as 8), dispersion (class bands of width b),
// linear mapping (position inside the band).
__device__ __forceinline__ uint32_t hash_key(uint32_t n, uint32_t a, uint32_t b, uint32_t R)
{
    uint32_t agg = n >> a;
    agg = agg > 8u ? 8u : agg;
    uint32_t lin = ((n & ((1u << a) - 1u)) * b) >> a;
    uint32_t key = agg * b + lin;
    return key > R - 1u ? R - 1u : key;
}

// Sampling of the shift a: histogram, over the segments of up to 4096 evenly spaced rows, of
// the smallest a in 0..12 with n < 9 * 2^a.  One wavefront walks one sampled row.  hist[14] also
// counts the sampled segments with at least kLongSegment nonzeros (block sizes are chosen by it).  hist: kHistCopies copies, kHistStride words
// apart (one copy, to which 1024 workgroups add: 16.2 against 5.0 us on the 27-point grid of 128^3, 19.8 against 14.2 on 4M x 1M lognormal rows).
// row_stats: kStatsCopies copies that add up to the statistics of all rows, where they matter (and the grid has the workgroups).
// (Every wavefront of the sampling workgroups counting its share of the rows into 16 copies: 15 to 20 us more per build.)
constexpr int kLongSegment = 6;
constexpr int kStatsCopies = 64;  // so that the workgroups do not queue up for one address
constexpr int kStatsGroups = 1024;
constexpr int kHistCopies = 16, kHistStride = 32;
__global__ __launch_bounds__(256) void k_sample_hist(const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                                     int64_t n_rows, int32_t C, int32_t S, uint32_t *__restrict__ hist,
                                                     RowStats *__restrict__ row_stats)
{
    // Pointers that do not start at 0 (a row slice of a larger matrix) are refused when the host has them; until then
    // csr_col is not read through them: every row counts as empty.  (Both words are read before either is looked at.)
    const int32_t first = ptr[0], last = ptr[n_rows];
    const int64_t nnz = first == 0 ? last : 0;
    __shared__ uint32_t sh_hist[15];  // [14]: sampled segments with kLongSegment or more nonzeros
    if (threadIdx.x < 15) sh_hist[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int32_t sampling = (S + 3) / 4;  // workgroups; kStatsGroups more look at all rows (beside them: they wait for loads too)
    if ((int32_t)blockIdx.x >= sampling) {
        if (!rows_matter(nnz, n_rows)) return;
        const int64_t per = (n_rows + kStatsGroups - 1) / kStatsGroups, r0 = (int64_t)(blockIdx.x - sampling) * per, r1 = min(n_rows, r0 + per);
        const int64_t cap = max((int64_t)1, 64 * nnz / n_rows);
        uint32_t rows = 0;
        unsigned long long skew = 0;
#pragma unroll 4
        for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
            const int64_t n = (int64_t)ptr[r + 1] - ptr[r];
            rows += n > 0 ? 1u : 0u;
            skew += n > 0 ? (unsigned long long)(n * min(n, cap)) : 0ull;
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            rows += __shfl_xor(rows, d);
            skew += __shfl_xor(skew, d);
        }
        __shared__ RowStats sh_stats[4];
        if (lane == 0) sh_stats[threadIdx.x >> 6] = {rows, skew};
        __syncthreads();
        if (threadIdx.x == 0) {
            RowStats *const mine = row_stats + blockIdx.x % kStatsCopies;
            atomicAdd(&mine->rows, sh_stats[0].rows + sh_stats[1].rows + sh_stats[2].rows + sh_stats[3].rows);
            atomicAdd(&mine->skew, sh_stats[0].skew + sh_stats[1].skew + sh_stats[2].skew + sh_stats[3].skew);
        }
        return;
    }
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    auto tally = [&](int n) {
        int a = 0;
        while (a < 13 && n >= (9 << a)) a++;
        atomicAdd(&sh_hist[a], 1u);
        if (n >= kLongSegment) atomicAdd(&sh_hist[14], 1u);
    };
    if (k < S) {
        const int64_t r = ((int64_t)k * n_rows) / S;
        int64_t j0 = ptr[r], j1 = ptr[r + 1];
        if (j0 < 0 || j1 > nnz || j1 < j0) j1 = j0;  // malformed ptr is reported by k_check_ptr
        int64_t open = -1;                            // start of the segment whose end is not yet seen
        int bn_left = -1;                             // column block of the nonzero left of this chunk
        // A long row that spans few column blocks (R-MAT has rows of 10^5 nonzeros; walking one
        // chunk by chunk took 0.36 ms): its columns ascend, so its segment in column block bn is
        // [first column >= bn C, first column >= (bn + 1) C), two binary searches per lane.
        if (j1 - j0 > 4096) {
            const int64_t bn_first = col[j0] / C, bn_last = col[j1 - 1] / C;
            if (col[j0] >= 0 && bn_last >= bn_first && bn_last - bn_first < 4096) {
                auto lower_bound = [&](int64_t target) {  // first j in [j0, j1] with col[j] >= target
                    int64_t lo = j0, hi = j1;
                    while (lo < hi) {
                        const int64_t mid = lo + ((hi - lo) >> 1);
                        if ((int64_t)col[mid] >= target) hi = mid; else lo = mid + 1;
                    }
                    return lo;
                };
                for (int64_t bn = bn_first + lane; bn <= bn_last; bn += 64) {
                    const int64_t n = lower_bound((bn + 1) * C) - lower_bound(bn * C);
                    if (n > 0) tally((int)n);
                }
                j1 = j0;  // done: the walk below finds nothing
            }
        }
        // eight chunks of 64 columns are fetched at a time
        constexpr int kAhead = 8;
        for (int64_t base0 = j0; base0 < j1; base0 += 64 * kAhead) {
            int32_t cols[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; u++) {
                const int64_t j = base0 + 64 * u + lane;
                cols[u] = j < j1 ? col[j] : -1;
            }
#pragma unroll
            for (int u = 0; u < kAhead; u++) {
            const int64_t base = base0 + 64 * u;
            if (base >= j1) break;
            const int64_t j = base + lane;
            const bool valid = j < j1;
            const int bn = valid ? cols[u] / C : -2;
            int bn_prev = __shfl_up(bn, 1);
            if (lane == 0) bn_prev = bn_left;
            const bool start = valid && bn != bn_prev;
            const uint64_t mask = __ballot(start);
            if (mask) {
                const int first = __ffsll((long long)mask) - 1;
                if (open >= 0 && lane == 0) tally((int)(base + first - open));
                if (start) {
                    const uint64_t above = mask & ~((2ull << lane) - 1ull);
                    if (above) tally(__ffsll((long long)above) - 1 - lane);
                }
                open = base + (63 - __clzll((long long)mask));
            }
            bn_left = __shfl(bn, 63);
            }
        }
        if (open >= 0 && lane == 0) tally((int)(j1 - open));
    }
    __syncthreads();
    if (threadIdx.x < 15 && sh_hist[threadIdx.x]) atomicAdd(&hist[kHistStride * (blockIdx.x % kHistCopies) + threadIdx.x], sh_hist[threadIdx.x]);
}

// a = smallest shift for which at least 15/16 of the sampled segments aggregate into 0..8.  host: pinned words for what the build's parameters are
// chosen by, or null.
__global__ __launch_bounds__(64) void k_pick_shift(const uint32_t *__restrict__ hist, int32_t *__restrict__ a_out, const RowStats *__restrict__ row_stats,
                                                   const int32_t *__restrict__ ptr, int64_t n_rows, uint32_t *__restrict__ host)
{
    const int i = threadIdx.x;
    uint32_t here = 0;  // lane i: segments in bin i
    if (i < 15)
        for (int c = 0; c < kHistCopies; c++) here += hist[kHistStride * c + i];
    const uint32_t counted = i < 14 ? here : 0u;
    const uint64_t upto = sum_up_to_lane(counted);  // (fewer than 2^31 nonzeros in all)
    const uint64_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    const uint64_t enough = __ballot(i <= 12 && 16 * upto >= 15 * total);
    const int a = total == 0 ? 0 : enough ? __builtin_ctzll(enough) : 12;
    if (i == 0) *a_out = a;
    if (!host) return;
    RowStats all = row_stats[i];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        all.rows += __shfl_xor(all.rows, d);
        all.skew += __shfl_xor(all.skew, d);
    }
    if (i < 16) host[i] = here;
    if (i == 0) {
        host[16] = (uint32_t)a;
        host[17] = (uint32_t)ptr[0];
        host[18] = (uint32_t)ptr[n_rows];
        host[19] = all.rows;
        host[20] = (uint32_t)all.skew;
        host[21] = (uint32_t)(all.skew >> 32);
    }
}

// What a build begins with: zeros in two ranges of words, and the shift where it is given.
__global__ __launch_bounds__(256) void k_begin(uint32_t *__restrict__ first, int64_t n_first, uint32_t *__restrict__ second, int64_t n_second,
                                               int32_t *__restrict__ a_out, int32_t a)
{
    const int64_t threads = (int64_t)gridDim.x * 256, t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = t; i < n_first; i += threads) first[i] = 0u;
    for (int64_t i = t; i < n_second; i += threads) second[i] = 0u;
    if (t == 0 && a >= 0) *a_out = a;
}

// Empty matrix: one empty combine unit per row block (it writes the zeros of y).
__global__ __launch_bounds__(256) void k_iota_units(int32_t *unit_ptr, int32_t *unit_stripe, int32_t *unit_k, int32_t NBR)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > NBR) return;
    unit_ptr[i] = (int32_t)i;
    unit_k[i] = 0;
    if (i < NBR) unit_stripe[i] = (int32_t)i;
}

// ------------------------------------------------------------------ steps 1-3: segments

constexpr int kTile = 4096, kTileThreads = 512, kTileWords = kTile / 64, kWordsPerWave = kTileWords / (kTileThreads / 64);
constexpr int kTileCounters = 4096;  // 16 KB of LDS
// A tile with as many rows and more between its first and its last has its nonzeros look for their rows instead of walking
// them all.  Whole builds, us, walked / looked for, rows per tile: 16 K 514 / 540, 41 K 411 / 400, 64 K 481 / 500, 128 K 731 / 714.
constexpr int kTileRowsWalked = 64 * kTileThreads;

// Rounds of a group that one wavefront fills where the groups are cut (step 7).  A wavefront copies 8 to 32 rounds per memory round trip:
// left to one, the longest row segment of R-MAT 2^20 (fp64) is on its way for 320 us.
constexpr int kFillRounds = 128;

constexpr int kLongRow = 4 * kFillRounds;

// What k_check_ptr and k_segments find out, zeros to begin with: what is wrong; the longest row, where it has more than kLongRow
// nonzeros; whether a tile shows a long segment.  The last two in copies apart from each other (one word for all: 101 us for k_check_ptr in
// place of 10 where one row in 40 has to be told), and all behind one pointer (another argument, two more scalar registers, and
// a compute unit holds three tiles of k_segments instead of four: 98 -> 114 us on the 27-point grid of 128^3).
struct Findings {
    int32_t err;
    uint32_t most_slots, most_nonzeros;  // of a row block
    uint32_t dealt[9];                   // shares of row blocks for the eight XCDs, row blocks that hold something (see deal_row_blocks)
    int32_t apart[4];
    struct { uint32_t longest_row, long_segment, apart[14]; } copy[64];
};
__device__ __forceinline__ auto &findings_of_workgroup(Findings *found) { return found->copy[blockIdx.x % 64]; }

// kTile consecutive nonzeros: the row that holds the first of them, and the segments that start there.
struct Tile {
    int32_t row, first, count, unused;  // first: where the first segment starts; -1: none does
};

// Checks csr_ptr and notes every tile's row (where the pointers are valid).
__global__ __launch_bounds__(256) void k_check_ptr(const int32_t *__restrict__ ptr, int64_t n_rows, int64_t nnz, Tile *__restrict__ tiles,
                                                   Findings *__restrict__ found)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t length = 0;
    if (r < n_rows) {
        const int64_t p0 = ptr[r], p1 = ptr[r + 1];
        if (p0 < 0 || p1 < p0 || p1 > nnz) {
            atomicOr(&found->err, kErrPtr);
        } else {
            for (int64_t t = (p0 + kTile - 1) / kTile; t * kTile < p1; t++) tiles[t].row = (int32_t)r;
            length = (uint32_t)(p1 - p0);
        }
    }
    const uint32_t longest = wave_max(length);
    if (longest > (uint32_t)kLongRow && (threadIdx.x & 63) == 0) atomicMax(&findings_of_workgroup(found).longest_row, longest);
}

// Wave-aggregated fetch-add: lanes of the wavefront that target the same counter are served by
// one atomic (neighbouring segments mostly fall into the same block, and same-address atomics
// serialise).  Returns, for an active lane, the value its own atomicAdd(&counters[key], 1) would
// have returned in some serial order.  After a few distinct keys the rest go one by one.
__device__ __forceinline__ uint32_t aggregated_add(uint32_t *counters, int64_t key, bool active)
{
    const int lane = threadIdx.x & 63;
    uint64_t todo = __ballot(active);
    uint32_t result = 0;
    for (int it = 0; todo && it < 8; it++) {
        const int leader = __ffsll((long long)todo) - 1;
        const int64_t k = __shfl(key, leader);
        const uint64_t same = __ballot(active && key == k) & todo;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&counters[k], (uint32_t)__popcll(same));
        base = __shfl(base, leader);
        if ((same >> lane) & 1ull) result = base + (uint32_t)lanes_below(same);
        todo &= ~same;
    }
    if ((todo >> lane) & 1ull) result = atomicAdd(&counters[key], 1u);
    return result;
}

// Smallest i in [lo, hi] for which reached(i) holds, given that reached(hi) does: the lanes of a wavefront ask
// for 64 candidates at once, so that a million entries take four dependent steps instead of twenty.
template <typename F>
__device__ __forceinline__ int32_t first_reached(int32_t lo, int32_t hi, F reached)
{
    const int lane = threadIdx.x & 63;
    while (lo < hi) {  // wave-uniform
        const int32_t step = (int32_t)(((int64_t)hi - lo + 63) / 64);
        const int32_t i = (int32_t)min((int64_t)hi, lo + (int64_t)lane * step);
        const uint64_t yes = __ballot(reached(i));
        if (yes & 1) return lo;
        if (yes == 0) {  // behind the last candidate below hi
            lo = (int32_t)min((int64_t)hi, lo + 63 * (int64_t)step + 1);
        } else {
            const int f = __builtin_ctzll(yes);
            hi = (int32_t)min((int64_t)hi, lo + (int64_t)f * step);
            lo = (int32_t)(lo + (int64_t)(f - 1) * step + 1);
        }
    }
    return lo;
}

// The same for two questions at once, 32 candidates each: reached(i) answers a lane's own, that of the lower or the upper half of the
// wavefront.  Returns the answers in the halves' lanes.
template <typename F>
__device__ __forceinline__ int32_t first_reached_by_halves(int32_t lo, int32_t hi, F reached)
{
    const int lane = threadIdx.x & 63, half = lane & 32;
    while (__ballot(lo < hi)) {  // wave-uniform
        const int32_t step = (int32_t)(((int64_t)hi - lo + 31) / 32);
        const int32_t i = (int32_t)min((int64_t)hi, lo + (int64_t)(lane & 31) * step);
        const uint32_t yes = (uint32_t)(__ballot(reached(i)) >> half);
        if (yes == 0) {  // behind the last candidate below hi
            lo = (int32_t)min((int64_t)hi, lo + 31 * (int64_t)step + 1);
        } else if (yes & 1) {
            hi = lo;
        } else {
            const int f = __builtin_ctz(yes);
            hi = (int32_t)min((int64_t)hi, lo + (int64_t)f * step);
            lo = (int32_t)(lo + (int64_t)(f - 1) * step + 1);
        }
    }
    return lo;
}

// inclusive maximum over the lanes up to this one, of values from -1 up (all lanes active; six vector instructions)
template <int kControl, int kRows>
__device__ __forceinline__ int32_t highest_moved(int32_t v) { return max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, kControl, kRows, 0xf, false)); }
__device__ __forceinline__ int32_t highest_up_to_lane(int32_t v)
{
    v = highest_moved<0x111, 0xf>(v);
    v = highest_moved<0x112, 0xf>(v);
    v = highest_moved<0x114, 0xf>(v);
    v = highest_moved<0x118, 0xf>(v);
    v = highest_moved<0x142, 0xa>(v);
    return highest_moved<0x143, 0xc>(v);
}
// v with `value` (the same in all lanes) in place of what lane `l` (a constant) holds
__device__ __forceinline__ int32_t with_lane(int32_t value, int32_t l, int32_t v)
{
    // (a vector instruction that reads a scalar register which another has written, as a ballot does, has to stay two wait states behind it; the
    // compiler sees to that, but does not look into assembly)
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(value), "i"(l));
    return v;
}
// the value of the lane below; lane 0 gets `first`
__device__ __forceinline__ int32_t lane_below(int32_t v, int32_t first) { return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xf, 0xf, false); }

enum class Pass { kCount, kCountAndList, kCountListAndWords, kEmit };
constexpr int kPlaceBits = 12;  // of a list's entry: the segment's first nonzero, counted from its tile's
static_assert(kTile == 1 << kPlaceBits, "a place in a tile");
constexpr uint32_t kNoSegment = 0xffffffffu;  // no entry whose place is still zero

// 64 consecutive nonzeros: which of them start a segment, and how many segments start in the words of the tile before.
struct SegmentWords {
    uint64_t *starts;
    uint16_t *at;
};

// The segments of kTile consecutive nonzeros per workgroup: a nonzero starts one when it starts a row or
// its block column differs from its left neighbour's.  The rows that start inside the tile are read from
// csr_ptr (empty rows own no position) into an LDS table by position, or looked for from the nonzeros where most
// rows are empty; a segment's row is the last one that starts at or before it.  The matrix's columns are read once, 4 bytes per nonzero:
//   kCountAndList  counts the segments of every block (cursor: the block table), notes every tile's first segment start and whether a tile
//                  shows a long segment, and leaves the tile's segments in a list, a word each: block column, row in its
//                  block, place in the tile.  After the scans over the block table k_place reads the list, 4 bytes per segment.
//   kCountListAndWords  the same, and which nonzeros start a segment, for k_panel_fill.
//   kCount, kEmit  where an entry takes more than a word (R = 2048: over 512 block columns): the same without a list, and a second pass that
//                  finds the segments again and drops (length << 16 | local row, first nonzero) of every one into its block's
//                  slot range (cursor: the blocks' next free slots), in no particular order: k_order_block sorts them.
// A tile's rows are neighbours, so it touches the blocks of a few row blocks only: (bm_hi - bm_lo + 1) * NBC
// counters.  When those fit in LDS the tile counts there (LDS integer atomics are two orders of magnitude
// faster than scattered global ones) and goes to global memory once per counter it has touched;
// otherwise every segment goes to global memory with wave-aggregated atomics.
// (Before: row-start bits by global atomics, segment flags, a scan, segment records with a binary search per
// segment, a counting pass and a bucket pass over the records, 20 bytes per segment written and read twice: 1239 us
// on the 4M x 1M lognormal matrix, 535 in two passes; 300 and 288 on the 27-point grid of 128^3, 181 and 186 on R-MAT 2^20.  A
// tile is a chain of dependent loads of some 8 us, four tiles to a CU at a time.  With a nonzero's row found by a maximum over the lanes up to
// it in place of a bit search and an LDS read, and the scans over a tile's words without LDS, 517, 227 and 118: first pass 197 -> 182 us on the
// lognormal matrix and 115 -> 98 us on the grid, second pass 160 -> 129 us on the grid by the scans alone (65 -> 62 registers: all four tiles of
// a CU).  Issuing vector instructions takes 77 and 88 % of the passes' time on the grid, 73 and 59 % on the lognormal matrix.  With the list in
// place of the second reading 100 + 133 -> 106 + 28 us on the grid, 183 + 337 -> 186 + 300 on the lognormal matrix, 52 + 65 -> 51 + 46 on R-MAT
// 2^20 in fp64 (the first pass with the list, but before the shifts, masks and stores by words below: 123, 216, 56; with more than 80 scalar
// registers a compute unit holds three tiles in place of four: 139, 247, 60).
// Rows that hold a nonzero far apart, 40M rows, build in us, one in 200 / one in 1000: 440 / 410; walked 512 at a time with a
// jump over the gaps 3260 / 20900.)
template <Pass PASS, bool POW2>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_num_sgpr(80)))
void k_segments(const int32_t *__restrict__ ptr, const int32_t *__restrict__ col, int64_t n_rows,
                                                           int64_t nnz, int64_t n_cols, int32_t R, int32_t shift_r, int32_t C, int32_t shift_c,
                                                           int32_t NBR, int32_t NBC, int validate, Tile *__restrict__ tiles,
                                                           uint32_t *__restrict__ cursor, uint2 *__restrict__ bucket,
                                                           uint32_t *__restrict__ list, int32_t row_bits, SegmentWords words, Findings *found)
{
    constexpr bool EMIT = PASS == Pass::kEmit, WORDS = PASS == Pass::kCountListAndWords, LIST = PASS == Pass::kCountAndList || WORDS;
    __shared__ uint32_t cnt[kTileCounters];
    __shared__ __align__(16) int32_t row_at[kTile];  // row that starts at a position, counted from the tile's first row; -1: none
    __shared__ int32_t word_last[kTileWords], word_first[kTileWords];  // last row start, first segment start of a word; -1, kTile: none
    __shared__ uint32_t word_starts[kTileWords];  // LIST: segments that start in a word
    __shared__ int32_t sh_next;
    if (found->err & kErrPtr) return;  // k_check_ptr's finding: the rows below would not ascend
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j0 = (int64_t)blockIdx.x * kTile;
    const int32_t count = (int32_t)min((int64_t)kTile, nnz - j0);
    const int32_t first_word = wave * kWordsPerWave;
    int32_t c[kWordsPerWave], before = -1;  // before: the nonzero in front of this wavefront's first
#pragma unroll
    for (int u = 0; u < kWordsPerWave; u++) {
        const int32_t i = (first_word + u) * 64 + lane;
        c[u] = i < count ? lane_at(col + j0, i) : 0;
    }
    if (lane == 0 && j0 + first_word * 64 > 0 && first_word * 64 < count) before = col[j0 + first_word * 64 - 1];
    for (int i = threadIdx.x; i < kTile / 4; i += kTileThreads) reinterpret_cast<int4 *>(row_at)[i] = int4{-1, -1, -1, -1};
    if (EMIT && wave == 0) {  // where the segment that is open at the tile's end ends: a segment has fewer than 2^16 nonzeros, 16 tiles
        const int64_t n_tiles = (nnz + kTile - 1) / kTile, t = (int64_t)blockIdx.x + 1 + lane;
        const int32_t f = t < n_tiles ? tiles[t].first : (int32_t)nnz;
        const uint64_t there = __ballot(f >= 0);
        const int32_t next = there ? __shfl(f, __builtin_ctzll(there)) : (int32_t)nnz;
        if (lane == 0) sh_next = next;
    }
    __syncthreads();
    // the rows that can start in the tile: from the one that holds its first nonzero to the one that holds the next tile's
    const int32_t row_lo = tiles[blockIdx.x].row;
    const int32_t row_hi = j0 + count < nnz ? tiles[blockIdx.x + 1].row : (int32_t)(n_rows - 1);
    if (row_hi - row_lo < kTileRowsWalked) {
        const int32_t *const first = ptr + row_lo;
        for (int32_t r = threadIdx.x; r <= row_hi - row_lo; r += kTileThreads) {
            const uint32_t p0 = (uint32_t)lane_at(first, r), p1 = (uint32_t)lane_at(first + 1, r), place = p0 - (uint32_t)j0;
            if (p1 > p0 && place < (uint32_t)count) row_at[place] = r;
        }
    } else {
        // Empty rows by the thousand: every nonzero looks for its row, the last one that starts at or before it, a lane's
        // kAtOnce searches side by side (all eight would take the registers of the whole kernel from 66 to 100).
        constexpr int kAtOnce = 4;
#pragma unroll 1
        for (int u0 = 0; u0 < kWordsPerWave; u0 += kAtOnce) {
            int32_t r[kAtOnce];
            uint32_t p[kAtOnce];
#pragma unroll
            for (int u = 0; u < kAtOnce; u++) r[u] = row_lo;
            const int32_t i0 = (first_word + u0) * 64 + lane;
            const uint32_t j = (uint32_t)(j0 + i0);  // (behind the last nonzero: beyond 2^31, not beyond 2^32)
#pragma unroll 1
            for (int32_t step = 1 << (31 - __clz(row_hi - row_lo)); step > 0; step >>= 1) {
#pragma unroll
                for (int u = 0; u < kAtOnce; u++) p[u] = step <= row_hi - r[u] ? (uint32_t)ptr[r[u] + step] : 0xffffffffu;
#pragma unroll
                for (int u = 0; u < kAtOnce; u++)
                    if (p[u] <= j + 64 * u) r[u] += step;
            }
#pragma unroll
            for (int u = 0; u < kAtOnce; u++) p[u] = (uint32_t)ptr[r[u]];
#pragma unroll
            for (int u = 0; u < kAtOnce; u++)
                if (i0 + 64 * u < count && p[u] == j + 64 * u) row_at[i0 + 64 * u] = r[u] - row_lo;
        }
    }
    __syncthreads();
    uint64_t rows_here[kWordsPerWave];
    int32_t latest[kWordsPerWave];  // the last row that starts in the word, up to this lane; -1: none
    int32_t of_word = 0;            // lane u: something about the wavefront's word u, on its way to LDS
#pragma unroll
    for (int u = 0; u < kWordsPerWave; u++) {
        const int32_t w = first_word + u, r = row_at[w * 64 + lane];
        rows_here[u] = __builtin_amdgcn_ballot_w64(r >= 0);
        latest[u] = highest_up_to_lane(r);
        of_word = with_lane(__builtin_amdgcn_readlane(latest[u], 63), u, of_word);
    }
    if (lane < kWordsPerWave) word_last[first_word + lane] = of_word;
    __syncthreads();
    // lane w: the last row that starts in the words 0 .. w (rows ascend)
    const int32_t last_row = highest_up_to_lane(max(0, word_last[lane]));
    // POW2: both block sizes are powers of two (or there is one block column, and shift_c 31)
    auto row_block = [&](int32_t row) { return POW2 ? row >> shift_r : row / R; };
    auto row_in_block = [&](int32_t row) { return (uint32_t)(POW2 ? row & (R - 1) : row - row / R * R); };
    auto block_column = [&](int32_t column) { return POW2 ? column >> shift_c : column / C; };
    const int32_t bm_lo = row_block(row_lo), bm_hi = row_block(row_lo + __builtin_amdgcn_readlane(last_row, 63));
    const int64_t counters = (int64_t)(bm_hi - bm_lo + 1) * NBC;
    const bool in_lds = counters <= kTileCounters;
    if (in_lds) {
        for (int i = threadIdx.x; i < (int)counters; i += kTileThreads) cnt[i] = 0u;
        __syncthreads();
    }
    int32_t row[kWordsPerWave], local[kWordsPerWave];
    uint32_t rank[kWordsPerWave];  // LIST: the segment's entry but for its place
    uint64_t starts[kWordsPerWave];
    const uint32_t cols = (uint32_t)n_cols;  // below 2^31
    int32_t last_bn = 0;  // block column of the last nonzero of the word before
    int32_t n_of_word = 0, lo_of_word = 0, hi_of_word = 0;
#pragma unroll
    for (int u = 0; u < kWordsPerWave; u++) {
        const int32_t w = first_word + u, i = w * 64 + lane;
        const bool valid = i < count;
        const int32_t carried = w > 0 ? __builtin_amdgcn_readlane(last_row, w > 0 ? w - 1 : 0) : 0;
        row[u] = row_lo + max(latest[u], carried);  // (rows ascend)
        const bool row_start = (rows_here[u] >> lane) & 1ull;
        const int32_t c_prev = lane_below(c[u], u > 0 ? __builtin_amdgcn_readlane(c[u > 0 ? u - 1 : 0], 63) : __builtin_amdgcn_readfirstlane(before));
        const bool in_range = (uint32_t)c[u] < cols;
        if (!EMIT && valid && (!in_range || (validate && !row_start && c[u] <= c_prev))) atomicOr(&found->err, kErrCol);
        const int32_t bn = block_column(c[u]);
        const int32_t bn_prev = lane_below(bn, u > 0 ? last_bn : block_column(__builtin_amdgcn_readfirstlane(before)));
        last_bn = __builtin_amdgcn_readlane(bn, 63);
        const bool start = valid && (row_start || bn != bn_prev);
        starts[u] = __builtin_amdgcn_ballot_w64(start);
        of_word = with_lane(starts[u] ? w * 64 + __builtin_ctzll(starts[u]) : kTile, u, of_word);
        if (LIST) n_of_word = with_lane(__popcll(starts[u]), u, n_of_word);
        if (WORDS) {
            lo_of_word = with_lane((int32_t)(uint32_t)starts[u], u, lo_of_word);
            hi_of_word = with_lane((int32_t)(starts[u] >> 32), u, hi_of_word);
        }
        local[u] = -1;
        rank[u] = 0;
        if (LIST) rank[u] = start ? ((uint32_t)bn << row_bits | row_in_block(row[u])) << kPlaceBits : kNoSegment;
        const bool mine = start && in_range;  // (a column out of range has been reported; never index with it)
        if (in_lds) {
            if (mine) {
                local[u] = (int32_t)__umul24((uint32_t)(row_block(row[u]) - bm_lo), (uint32_t)NBC) + bn;  // (below kTileCounters)
                const uint32_t before_me = atomicAdd(&cnt[local[u]], 1u);
                if (EMIT) rank[u] = before_me;
            }
        } else {
            const uint32_t before_me = aggregated_add(cursor, mine ? (int64_t)bn * NBR + row_block(row[u]) : 0, mine);
            if (EMIT) rank[u] = before_me;
            if (mine) local[u] = 0;
        }
    }
    if (lane < kWordsPerWave) {
        word_first[first_word + lane] = of_word;
        if (LIST) word_starts[first_word + lane] = (uint32_t)n_of_word;
    }
    __syncthreads();
    if (in_lds) {
        for (int i = threadIdx.x; i < (int)counters; i += kTileThreads) {
            const uint32_t n = cnt[i];
            if (n) {
                const uint32_t at = atomicAdd(&cursor[(int64_t)(i % NBC) * NBR + bm_lo + i / NBC], n);
                if (EMIT) cnt[i] = at;
            }
        }
    }
    if constexpr (!EMIT) {
        if (wave == 0) {
            const int32_t f = word_first[lane];
            const uint64_t there = __ballot(f < kTile);
            const int32_t first = there ? __shfl(f, __builtin_ctzll(there)) : -1;
            if (lane == 0) tiles[blockIdx.x].first = first < 0 ? -1 : (int32_t)(j0 + first);
            if (lane == 0 && shows_long_segment(there, count))  // (several workgroups may write it, side by side)
                __hip_atomic_store(&findings_of_workgroup(found).long_segment, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if constexpr (LIST) {
            const uint32_t upto = sum_up_to_lane(word_starts[lane]);  // lane w: segments that start in the words 0 .. w
            if (wave == 0 && lane == 63) tiles[blockIdx.x].count = (int32_t)upto;
            if constexpr (WORDS) {
                const int64_t word0 = (int64_t)blockIdx.x * kTileWords;
                if (lane < kWordsPerWave) words.starts[word0 + first_word + lane] = (uint64_t)(uint32_t)hi_of_word << 32 | (uint32_t)lo_of_word;
                if (wave == 0) words.at[word0 + lane] = (uint16_t)(upto - word_starts[lane]);
            }
            uint32_t *const mine = list + j0;  // (as many entries as nonzeros: where a tile's begin does not depend on the others)
#pragma unroll
            for (int u = 0; u < kWordsPerWave; u++) {
                const int32_t w = first_word + u;
                const uint32_t at = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto, w > 0 ? w - 1 : 0) : 0u;
                const uint64_t there = __builtin_amdgcn_ballot_w64(rank[u] != kNoSegment);  // (`starts` kept until here would take 14 more scalar registers)
                if (rank[u] != kNoSegment) lane_at(mine + at, (uint32_t)lanes_below(there)) = rank[u] | (uint32_t)(w * 64 + lane);
            }
        }
    } else {
        __syncthreads();
        // lane 63 - w: the first segment start in the words w .. 63, counted back from the tile's end (0: none)
        const int32_t next_start = highest_up_to_lane(kTile - word_first[63 - lane]);
#pragma unroll
        for (int u = 0; u < kWordsPerWave; u++) {
            const int32_t w = first_word + u, i = w * 64 + lane;
            const uint64_t above = starts[u] & ~((2ull << lane) - 1ull);
            const int32_t later = w < kTileWords - 1 ? kTile - __builtin_amdgcn_readlane(next_start, w < kTileWords - 1 ? kTileWords - 2 - w : 0) : kTile;
            const int32_t j = (int32_t)(j0 + i);
            const int32_t end = above ? (int32_t)(j0 + w * 64) + __builtin_ctzll(above) : later < kTile ? (int32_t)(j0 + later) : sh_next;
            if (local[u] < 0) continue;
            const uint32_t pos = rank[u] + (in_lds ? cnt[local[u]] : 0u);
            bucket[pos] = {((uint32_t)(end - j) << 16) | row_in_block(row[u]), (uint32_t)j};  // length <= C <= 32768
        }
    }
}

// Drops the segments of the list into their blocks' slot ranges: `parts` wavefronts to a tile (ALL: all of the workgroup), a lane per segment.  A segment's row block is
// the last one that begins at or before its first nonzero.
// (Bound by the stores, 8 bytes to a line of their own for most lanes, where segments are short; by a tile's chain of loads where they are long,
// hence several tiles to a workgroup there.)
template <bool ALL>
__global__ __launch_bounds__(kTileThreads) void k_place(const int32_t *__restrict__ ptr, int64_t n_rows, int64_t nnz, int32_t R, int32_t shift_r,
                                                        int32_t NBR, int32_t NBC, int32_t n_tiles, int32_t parts, const Tile *__restrict__ tiles,
                                                        const uint32_t *__restrict__ list, int32_t row_bits, uint32_t *__restrict__ cursor,
                                                        uint2 *__restrict__ bucket)
{
    constexpr int kWaves = kTileThreads / 64;
    __shared__ uint32_t cnt[kTileCounters];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (ALL) parts = kWaves;
    const int32_t here = kWaves / parts, t0 = (int32_t)blockIdx.x * here, t = t0 + wave / parts, part = wave % parts;
    auto row_block = [&](int32_t row) { return shift_r >= 0 ? row >> shift_r : row / R; };
    // the row block that holds the first nonzero of tile i, or the last one behind the last tile
    auto first_block = [&](int32_t i) { return i < n_tiles ? row_block(tiles[i].row) : NBR - 1; };
    auto begin_of = [&](int32_t bm) { return ptr[min((int64_t)bm * R, n_rows)]; };  // (of row block NBR: the end)
    const int32_t bm_lo = first_block(t0), bm_hi = first_block(min(t0 + here, n_tiles));
    const int64_t counters = (int64_t)(bm_hi - bm_lo + 1) * NBC;
    const bool in_lds = counters <= kTileCounters;
    if (in_lds) {
        for (int i = threadIdx.x; i < (int)counters; i += kTileThreads) cnt[i] = 0u;
        __syncthreads();
    }
    const int32_t count = t < n_tiles ? tiles[t].count : 0;
    const int32_t tile_lo = t < n_tiles ? row_block(tiles[t].row) : 0, tile_hi = t < n_tiles ? first_block(t + 1) : 0;
    const uint32_t *const mine = list + (int64_t)t * kTile;
    const uint32_t j0 = (uint32_t)t * kTile, second = tile_hi > tile_lo ? (uint32_t)begin_of(tile_lo + 1) : 0xffffffffu;
    const int32_t row_mask = (1 << row_bits) - 1;
    auto block_of = [&](uint32_t j) {
        int32_t lo = tile_lo, hi = tile_hi;
        if (hi - lo <= 1) return j >= second ? hi : lo;  // wave-uniform
        while (lo < hi) {
            const int32_t mid = lo + ((hi - lo + 1) >> 1);
            if ((uint32_t)begin_of(mid) <= j) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    auto counter_of = [&](uint32_t e, int32_t bm) { return (int32_t)__umul24((uint32_t)(bm - bm_lo), (uint32_t)NBC) + (int32_t)(e >> kPlaceBits >> row_bits); };
    // ALL: a lane's segments stay in registers between the two passes, with their ranks in the tile
    constexpr int kPer = ALL ? kTile / kTileThreads : 1;
    uint32_t kept[kPer];
    int32_t kept_at[kPer];  // counter << 12 | rank
    if (in_lds) {
        if constexpr (ALL) {
#pragma unroll
            for (int u = 0; u < kPer; u++) {
                const int32_t i = kTileThreads * u + (int32_t)threadIdx.x;
                kept[u] = i < count ? lane_at(mine, i) : 0u;
            }
#pragma unroll
            for (int u = 0; u < kPer; u++) {
                const int32_t i = kTileThreads * u + (int32_t)threadIdx.x;
                kept_at[u] = 0;
                if (i < count) {
                    const int32_t at = counter_of(kept[u], block_of(j0 + (kept[u] & (kTile - 1))));
                    kept_at[u] = at << 12 | (int32_t)atomicAdd(&cnt[at], 1u);  // (fewer than 4096 in front of the last)
                }
            }
        } else {
            for (int32_t i = part * 64 + lane; i < count; i += 64 * parts) {
                const uint32_t e = mine[i];
                atomicAdd(&cnt[counter_of(e, block_of(j0 + (e & (kTile - 1))))], 1u);
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < (int)counters; i += kTileThreads) {
            const uint32_t n = cnt[i];
            if (n) cnt[i] = atomicAdd(&cursor[(int64_t)(i % NBC) * NBR + bm_lo + i / NBC], n);
        }
        __syncthreads();
    }
    // where the segment that is open at the tile's end ends: a segment has fewer than 2^16 nonzeros, 16 tiles
    const int32_t next_tile = t + 1 + lane;
    const int32_t f = next_tile < n_tiles ? tiles[next_tile].first : (int32_t)nnz;
    const uint64_t there = __ballot(f >= 0);
    const uint32_t next = there ? (uint32_t)__builtin_amdgcn_readlane(f, __builtin_ctzll(there)) : (uint32_t)nnz;
    if constexpr (ALL) {
        if (in_lds) {
#pragma unroll
            for (int u = 0; u < kPer; u++) {
                const int32_t i = kTileThreads * u + (int32_t)threadIdx.x;
                if (i >= count) break;
                const uint32_t e = kept[u], j = j0 + (e & (kTile - 1));
                const uint32_t end = i + 1 < count ? j0 + (lane_at(mine, i + 1) & (kTile - 1)) : next;
                bucket[cnt[kept_at[u] >> 12] + (uint32_t)(kept_at[u] & 4095)] = {(end - j) << 16 | (e >> kPlaceBits & (uint32_t)row_mask), j};
            }
            return;
        }
    }
    for (int32_t i0 = part * 64; i0 < count; i0 += 64 * parts) {  // wave-uniform
        const int32_t i = i0 + lane;
        const bool valid = i < count;
        const uint32_t e = valid ? mine[i] : 0u, j = j0 + (e & (kTile - 1));
        const uint32_t end = i + 1 < count ? j0 + (mine[i + 1] & (kTile - 1)) : next;
        const int32_t bm = valid ? block_of(j) : tile_lo, bn = (int32_t)(e >> kPlaceBits >> row_bits);
        uint32_t pos = 0;
        if (in_lds) {
            if (valid) pos = atomicAdd(&cnt[counter_of(e, bm)], 1u);
        } else {
            pos = aggregated_add(cursor, valid ? (int64_t)bn * NBR + bm : 0, valid);
        }
        if (valid) bucket[pos] = {(end - j) << 16 | (e >> kPlaceBits & (uint32_t)row_mask), j};
    }
}

// ------------------------------------------------------------------ step 4: block table

// Non-empty blocks get their coordinates and ranges; thread d also fills col_blk_ptr[d] and col_group_ptr[d].  And what else can be written once the
// totals are known: the padding behind the layout's last group, which is read (and its products dropped) by lanes without an element, the
// end of the last group, zeros in the counters.
__global__ __launch_bounds__(256) void k_compact_blocks(const uint32_t *__restrict__ dense_cnt, const uint32_t *__restrict__ slot_off,
                                                        const uint32_t *__restrict__ group_off, const uint32_t *__restrict__ blk_id,
                                                        int64_t D, int32_t NBR, int32_t NBC, int32_t *__restrict__ blk_bm,
                                                        int32_t *__restrict__ blk_bn, int32_t *__restrict__ slot_ptr,
                                                        int32_t *__restrict__ blk_group_ptr, int32_t *__restrict__ col_blk_ptr,
                                                        int32_t *__restrict__ col_group_ptr, uint16_t *__restrict__ col_padding,
                                                        uint32_t *__restrict__ data_padding, int32_t padding_words, int32_t *__restrict__ last_group_end,
                                                        uint32_t *__restrict__ counters)
{
    const int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0) {
        col_padding[threadIdx.x] = 0;
        for (int32_t i = threadIdx.x; i < padding_words; i += 256) data_padding[i] = 0u;
        if (threadIdx.x < 3) counters[threadIdx.x] = 0u;
    }
    if (d <= NBC) {
        col_blk_ptr[d] = (int32_t)blk_id[d * NBR];   // blk_id[D] = B closes the last column
        col_group_ptr[d] = (int32_t)group_off[d * NBR];
    }
    if (d > D) return;
    if (d == D) {
        const uint32_t B = blk_id[D];
        slot_ptr[B] = (int32_t)slot_off[D];
        blk_group_ptr[B] = (int32_t)group_off[D];
        *last_group_end = (int32_t)slot_off[D];
        return;
    }
    if (!dense_cnt[d]) return;
    const uint32_t b = blk_id[d];
    blk_bn[b] = (int32_t)(d / NBR);
    blk_bm[b] = (int32_t)(d % NBR);
    slot_ptr[b] = (int32_t)slot_off[d];
    blk_group_ptr[b] = (int32_t)group_off[d];
}

constexpr int kShareBits = 2;  // of an entry of the list of shares: which of its row block

// Combine index.  A workgroup takes 64 row blocks (a wavefront reads 64 neighbouring entries of a row of the block
// table) and deals the block columns out to its 16 wavefronts in contiguous slices.  (One thread per row
// block walking all block columns: 15 + 33 us for 512 x 64 blocks in 2 workgroups.)
constexpr int kStripeSlices = 16;

__device__ __forceinline__ uint32_t stripe_slice_count(const uint32_t *__restrict__ dense_cnt, int64_t bm, int32_t NBR, int32_t NBC,
                                                       uint32_t W, int32_t &bn0, int32_t &bn1, uint32_t &slots, uint32_t &groups)
{
    const int32_t slice = threadIdx.x >> 6;
    bn0 = (int32_t)(((int64_t)NBC * slice) / kStripeSlices);
    bn1 = (int32_t)(((int64_t)NBC * (slice + 1)) / kStripeSlices);
    uint32_t n = 0;
    slots = groups = 0;
    if (bm < NBR) {
#pragma unroll 8
        for (int64_t bn = bn0; bn < bn1; bn++) {
            const uint32_t here = dense_cnt[bn * NBR + bm];
            n += here ? 1u : 0u;
            slots += here;
            groups += (here + W - 1) / W;
        }
    }
    return n;
}

// Where row blocks are taken as a whole: the lists of those that hold something, and of their shares (k_panel_fill's workgroups).  A wavefront deals the
// ones of 64 row blocks out to the eight XCDs, a row block's shares all to one of them; a lane returns what becomes of one of them (or of none: no shares).
// (Before, the grids had a workgroup for every row block and for every share that the fullest row block needs; one without work waits for a compute unit's
// whole LDS, 5 us of the unit's time.  Builds, us, with them / without: fp64, 2000 row blocks of 5100 nonzeros and one of them of 60,000 531 / 401, none of them 394 /
// 396; 20,000 row blocks, all but 300 empty, 357 / 299, all but 1000 413 / 327; lognormal 4M x 1M, 2.05 shares on average and 3 at most, 1465 / 1456.)
struct Dealt {
    int64_t bm;
    uint32_t rank;          // of these row blocks
    uint32_t shares, upto;  // upto: of this XCD in front of the row block's
    uint32_t total;         // lanes 0 .. 7: shares of the XCD; lane 8: row blocks
};

__device__ __forceinline__ Dealt deal_row_blocks(int64_t bm, uint32_t nonzeros, uint32_t room)
{
    __shared__ uint32_t sh_shares[64], sh_row_block[64];
    const int lane = threadIdx.x & 63;
    const uint64_t some = __ballot(nonzeros > 0);
    // (the first of them to the XCD of its number, so that neighbours that go on over several wavefronts' 64 are spread evenly)
    const int count = __popcll(some), first = some ? __builtin_ctzll(some) & 7 : 0;
    if (nonzeros) {
        const int i = first + lanes_below(some);  // (below 64)
        sh_shares[i] = (nonzeros + room - 1) / room;
        sh_row_block[i] = (uint32_t)bm;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool there = lane >= first && lane < first + count;
    Dealt d;
    d.shares = there ? sh_shares[lane] : 0u;
    d.bm = there ? (int64_t)sh_row_block[lane] : 0;
    d.rank = (uint32_t)(lane - first);
    uint32_t upto = d.shares;
    for (int i = 8; i < 64; i <<= 1) {
        const uint32_t t = __shfl_up(upto, i);
        if (lane >= i) upto += t;
    }
    d.upto = upto - d.shares;
    const uint32_t of_xcd = __shfl(upto, 56 + (lane & 7));
    d.total = lane < 8 ? of_xcd : lane == 8 ? (uint32_t)count : 0u;
    return d;
}

__global__ __launch_bounds__(1024) void k_stripe_count(const uint32_t *__restrict__ dense_cnt, int32_t NBR, int32_t NBC, const int32_t *__restrict__ ptr,
                                                       int64_t n_rows, int32_t R, uint32_t W, uint32_t *__restrict__ stripe_cnt,
                                                       uint32_t *__restrict__ stripe_slots, uint32_t *__restrict__ stripe_groups,
                                                       uint32_t room, uint32_t *__restrict__ dealt, Findings *__restrict__ found)
{
    __shared__ uint32_t sh[kStripeSlices * 64], sh_slots[kStripeSlices * 64], sh_groups[kStripeSlices * 64];
    const int64_t bm = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    int32_t bn0, bn1;
    uint32_t slots, groups_in_slice;
    sh[threadIdx.x] = stripe_slice_count(dense_cnt, bm, NBR, NBC, W, bn0, bn1, slots, groups_in_slice);
    sh_slots[threadIdx.x] = slots;
    sh_groups[threadIdx.x] = groups_in_slice;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    uint32_t n = 0;
    uint32_t groups = 0;
    slots = 0;
#pragma unroll
    for (int i = 0; i < kStripeSlices; i++) {
        n += sh[i * 64 + threadIdx.x];
        groups += sh_groups[i * 64 + threadIdx.x];
        slots += sh_slots[i * 64 + threadIdx.x];
    }
    uint32_t nonzeros = 0;
    if (bm < NBR) {
        stripe_cnt[bm] = n;
        stripe_slots[bm] = slots;
        stripe_groups[bm] = groups;
        nonzeros = (uint32_t)(ptr[min((bm + 1) * R, n_rows)] - ptr[bm * R]);
    }
    if (!room) return;  // (what follows is for row blocks as a whole)
    const uint32_t total = deal_row_blocks(bm, nonzeros, room).total;
    if (threadIdx.x < 9) {
        dealt[threadIdx.x * gridDim.x + blockIdx.x] = total;
        if (total) atomicAdd(&found->dealt[threadIdx.x], total);
    }
    slots = wave_max(slots);
    nonzeros = wave_max(nonzeros);
    if (threadIdx.x == 0) {
        // (many look first: atomics on one address queue up, 4.4 -> 10.5 us for the kernel where 20,000 row blocks are told)
        auto raise = [](uint32_t *most, uint32_t v) {
            if (gridDim.x < 64 || v > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(most, v);
        };
        raise(&found->most_slots, slots);
        raise(&found->most_nonzeros, nonzeros);
    }
}

// The combine index and the combine work units.  A row block with many slots is cut into u = ceil(slots / unit_slots) units of consecutive
// stripe_blk entries, so that no workgroup of the combine part gets much more than unit_slots slots; unit i starts at the first entry whose
// preceding slots, times u, reach i times the row block's slots.
// blk_turn: the groups that come before the block's where groups are taken row block by row block.
// row_blocks, shares: the lists (where they are needed) of row blocks that hold something and of their shares, each XCD's at every eighth place.  dealt: prefix
// sums over the XCDs' totals of k_stripe_count's workgroups, one XCD after the other, and the row blocks'.
__global__ __launch_bounds__(1024) void k_stripe_fill(const uint32_t *__restrict__ dense_cnt, const uint32_t *__restrict__ blk_id,
                                                      const int32_t *__restrict__ stripe_ptr, const uint32_t *__restrict__ stripe_slots,
                                                      const int32_t *__restrict__ unit_ptr, const uint32_t *__restrict__ multi_idx,
                                                      const uint32_t *__restrict__ stripe_turn, uint32_t W, int32_t NBR, int32_t NBC, int32_t B,
                                                      int32_t *__restrict__ stripe_blk, uint32_t *__restrict__ blk_turn, int32_t *__restrict__ unit_stripe,
                                                      int32_t *__restrict__ unit_k, int32_t *__restrict__ multi_stripes, const int32_t *__restrict__ ptr,
                                                      int64_t n_rows, int32_t R, uint32_t room, const uint32_t *__restrict__ dealt,
                                                      int32_t *__restrict__ row_blocks, uint32_t *__restrict__ shares)
{
    __shared__ uint32_t sh[kStripeSlices * 64], sh_slots[kStripeSlices * 64], sh_groups[kStripeSlices * 64];
    const int64_t bm = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    int32_t bn0, bn1;
    uint32_t slots, groups_in_slice;
    sh[threadIdx.x] = stripe_slice_count(dense_cnt, bm, NBR, NBC, W, bn0, bn1, slots, groups_in_slice);
    sh_slots[threadIdx.x] = slots;
    sh_groups[threadIdx.x] = groups_in_slice;
    if (shares && threadIdx.x < 64) {
        const Dealt d = deal_row_blocks(bm, bm < NBR ? (uint32_t)(ptr[min((bm + 1) * R, n_rows)] - ptr[bm * R]) : 0u, room);
        const uint32_t xcd = threadIdx.x & 7u, at = dealt[xcd * gridDim.x + blockIdx.x] - dealt[xcd * gridDim.x] + d.upto;
        if (row_blocks && d.shares) row_blocks[dealt[8 * gridDim.x + blockIdx.x] - dealt[8 * gridDim.x] + d.rank] = (int32_t)d.bm;
        for (uint32_t i = 0; i < d.shares; i++) shares[8u * (at + i) + xcd] = (uint32_t)d.bm << kShareBits | i;
    }
    __syncthreads();
    if (bm >= NBR) return;
    int32_t k = stripe_ptr[bm];
    const int32_t u0 = unit_ptr[bm], u = unit_ptr[bm + 1] - u0;
    const int64_t all = stripe_slots[bm];
    int64_t before = 0;
    uint32_t turn = stripe_turn[bm];
    if (threadIdx.x < 64) {
        unit_stripe[u0] = (int32_t)bm;
        unit_k[u0] = k;
        if (u > 1) multi_stripes[multi_idx[bm]] = (int32_t)bm;
        if (bm == NBR - 1) unit_k[u0 + u] = B;
    }
    for (uint32_t i = threadIdx.x & 63; i < threadIdx.x; i += 64) {
        k += (int32_t)sh[i];
        before += sh_slots[i];
        turn += sh_groups[i];
    }
#pragma unroll 8
    for (int64_t bn = bn0; bn < bn1; bn++) {
        const int64_t d = bn * NBR + bm;
        const int32_t id = (int32_t)blk_id[d];
        const uint32_t here = dense_cnt[d];
        if (!here) continue;
        stripe_blk[k++] = id;
        blk_turn[id] = turn;
        turn += (here + W - 1) / W;
        if (u > 1) {  // the units that start behind this entry
            const int64_t next = (before + here) * u / all;
            for (int64_t i = before * u / all + 1; i <= next && i < u; i++) {
                unit_stripe[u0 + i] = (int32_t)bm;
                unit_k[u0 + i] = k;
            }
        }
        before += here;
    }
}

// ------------------------------------------------------------------ steps 5-6: hash + placement

// Which blocks a workgroup of k_fill takes.  The kernel gathers from arrays in CSR order (columns,
// values), where the pieces that the blocks of one row block need lie side by side in the same
// 128-byte lines.  Taken in the layout's column-major order every block fetches those lines anew
// (16 times the bytes on a matrix with short row segments).  Here the blocks are taken row block
// by row block (the order of stripe_blk), `parts` workgroups per row block, each taking every
// parts-th block of it; and since consecutive workgroups are dealt round-robin to the 8 XCDs,
// each with its own L2, the workgroups of a row block are numbered so that all of them land on
// one XCD: an XCD runs a few dozen workgroups at a time, which then share the lines of one or a
// few row blocks.
struct StripeWalk {
    int32_t k, k_end, step;  // entries k, k + step, ... below k_end of stripe_blk
};

__device__ __forceinline__ StripeWalk stripe_walk(const int32_t *__restrict__ stripe_ptr, int32_t NBR, int32_t parts)
{
    const int32_t q = (int32_t)(blockIdx.x >> 3), x = (int32_t)(blockIdx.x & 7u);
    const int32_t octet = q / parts, p = q % parts;
    // Which of the octet's eight row blocks goes to XCD x: x xor-ed with every 3-bit field of the
    // octet's number, a bijection inside the octet.  (With bm mod 8 itself a matrix whose density
    // follows the bits of the row index, as R-MAT's does, put 44 % of the work on one XCD.)
    int32_t fold = 0;
    for (int32_t t = octet; t; t >>= 3) fold ^= t & 7;
    const int32_t bm = octet * 8 + (x ^ fold);
    if (bm >= NBR) return {0, 0, 1};
    return {stripe_ptr[bm] + p, stripe_ptr[bm + 1], parts};
}

// Exclusive prefix sums of a[0 .. n) in LDS, in place, by the 256 threads of a workgroup.
// sh_wave: four words of LDS.  Ends with a barrier.
__device__ __forceinline__ void scan_in_lds(uint32_t *a, int n, uint32_t *sh_wave)
{
    const int chunk = (n + 255) / 256, lo = min(n, (int)threadIdx.x * chunk), hi = min(n, lo + chunk);
    uint32_t sum = 0;
    for (int i = lo; i < hi; i++) sum += a[i];
    uint32_t incl = sum;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
    }
    if (lane == 63) sh_wave[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int w = 0; w < (int)(threadIdx.x >> 6); w++) run += sh_wave[w];
    for (int i = lo; i < hi; i++) {
        const uint32_t t = a[i];
        a[i] = run;
        run += t;
    }
    __syncthreads();
}

// One workgroup per non-empty block: compute the keys of its segments, order its slots by (key,
// local row), then write the slot arrays and the nonzero count of each group.
// reorder 0: no key (plain 2D partition), 1: the hash with the matrix's shift, 2: the length
// itself, 3: the hash with a shift of the block's own (Section 3.2: denser blocks call for a
// larger a; a = smallest shift for which at least 15/16 of the block's rows aggregate into 0..8).
// Blocks of more than kSmallBlock slots: the local rows of a block are distinct, so the order by
// row costs nothing: entry (key << 16 | position in the block's bucket) is stored at index `row`
// of an LDS array, which leaves holes for the rows without a segment.  Stable counting passes
// over 4 bits of the key at a time, lowest first, then put the entries in key order and keep the
// row order inside a key; the first pass also closes the holes.  In a pass a wavefront takes 64
// consecutive entries at a time; the lanes that hold the same digit find each other with four
// ballots, which gives an entry its rank among them and the tile its count per digit; a prefix
// sum over (digit, tile) turns the counts into positions.  As many passes as the block's largest
// key has hex digits.  Smaller blocks (the passes would still walk all R rows): a bitonic network
// over (key, row, length, position) words.
// (second launch bound: all eight workgroups of small blocks to a CU, which 105 scalar registers had made seven; with a
// barrier less at the end, 1.9M blocks of 9 slots 4725 -> 3450 us, 3880 before long rows were counted per block;
// 4M x 1M lognormal matrix 529 -> 475.)
// Bound by its vector instructions: 253M of them per launch there, 4 cycles each on 1024 SIMDs, were nine tenths of 467 us.  With the wavefront's
// number and most of the arrays' addresses in scalar registers, sums over a wavefront without LDS and the lanes of a digit found by two
// instructions per half and bit: 188M (86 % of the time), 360 us; 27-point grid of 128^3 54 -> 35 us, R-MAT 2^20 146 -> 124 us.
__global__ __launch_bounds__(256, 8) void k_order_block(const uint2 *__restrict__ bucket,
                                                     const int32_t *__restrict__ slot_ptr, const int32_t *__restrict__ blk_group_ptr,
                                                     int32_t W, uint16_t *__restrict__ row_local, uint16_t *__restrict__ seg_len,
                                                     int32_t *__restrict__ slot_j, uint32_t *__restrict__ group_nnz, uint32_t *__restrict__ group_longest,
                                                     int32_t *__restrict__ group_slot, int32_t *__restrict__ group_blk, uint32_t heavy_rounds,
                                                     uint32_t *__restrict__ longest_all, uint32_t *__restrict__ n_long,
                                                     int32_t *__restrict__ long_groups, int32_t flat_wpg, int32_t reorder, uint32_t R,
                                                     const int32_t *__restrict__ a_ptr, int32_t *__restrict__ blk_shift,
                                                     uint32_t *__restrict__ slot_key)
{
    extern __shared__ __align__(8) uint32_t order_lds[];  // two arrays of cap entries, then 16 counters per tile of 64
    __shared__ uint32_t sh_hist[14];
    __shared__ int32_t sh_shift;
    __shared__ uint32_t sh_max_key, sh_wave[4], sh_long_n, sh_long_at;
    constexpr uint32_t kHole = 0xffffffffu;
    constexpr int kSmallBlock = 256;  // slots: one entry per thread
    const int cap = (int)((R + 63u) & ~63u);
    uint32_t *from = order_lds, *to = order_lds + cap, *cnt = order_lds + 2 * cap;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x;
    const int s0 = slot_ptr[b], m = slot_ptr[b + 1] - s0;
    const bool small = m <= kSmallBlock;
    const uint2 *const mine = bucket + s0;
    uint16_t *const out_row = row_local + s0, *const out_len = seg_len + s0;
    int32_t *const out_j = slot_j + s0;
    uint32_t *const out_key = slot_key ? slot_key + s0 : nullptr;
    if (!small)
        for (int i = threadIdx.x; i < cap; i += 256) from[i] = kHole;
    if (threadIdx.x < 14) sh_hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        sh_max_key = 0u;
        sh_long_n = 0u;
        sh_shift = *a_ptr;
    }
    __syncthreads();
    if (reorder == 3) {
        for (int i = threadIdx.x; i < m; i += 256) {
            const uint32_t n = lane_at(mine, i).x >> 16;
            int a = 0;
            while (a < 13 && n >= (9u << a)) a++;
            atomicAdd(&sh_hist[a], 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t below = 0;
            int a = 12;
            for (int i = 0; i <= 12; i++) {
                below += sh_hist[i];
                if (16ull * below >= 15ull * (uint32_t)m) { a = i; break; }
            }
            sh_shift = a;
        }
        __syncthreads();
    }
    const uint32_t shift_a = (uint32_t)sh_shift, band = R / 9u ? R / 9u : 1u;
    auto key_of = [&](uint32_t n) __attribute__((always_inline)) {
        return reorder == 0 ? 0u : reorder == 2 ? n : hash_key(n, shift_a, band, R);
    };
    // What the slots are sorted by.  The hash is b = d bands of class (n >> a, 8 at most) and inside them ascends with n
    // mod 2^a; where a band is wide enough to keep all 2^a remainders apart, class and remainder put side by
    // side give the same order and the same ties in 4 + a bits instead of the key's 11 (R = 2048): one pass over
    // the block instead of three at a = 0 (4M x 1M lognormal matrix 732 -> 529 us).
    const bool compact = (reorder == 1 || reorder == 3) && R >= 9u && band >= (1u << shift_a);
    auto sort_key = [&](uint32_t n) __attribute__((always_inline)) {
        return compact ? (min(n >> shift_a, 8u) << shift_a) | (n & ((1u << shift_a) - 1u)) : key_of(n);
    };
    if (threadIdx.x == 0) blk_shift[b] = (int32_t)shift_a;
    if (small) {
        uint64_t *wide = reinterpret_cast<uint64_t *>(order_lds);  // 2 cap words: room for cap >= m entries
        int n2 = 1;
        while (n2 < m) n2 <<= 1;
        for (int i = threadIdx.x; i < n2; i += 256) {
            uint64_t e = ~0ull;
            if (i < m) {
                const uint32_t lr = lane_at(mine, i).x;
                e = ((uint64_t)sort_key(lr >> 16) << 48) | ((uint64_t)(lr & 0xffffu) << 32) | (lr & 0xffff0000u) | (uint32_t)i;
            }
            wide[i] = e;
        }
        __syncthreads();
        for (int k = 2; k <= n2; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int t = threadIdx.x; t < n2 / 2; t += 256) {  // pair t: i has bit j clear, its partner has it set
                    const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), p = i | j;
                    const uint64_t x = wide[i], y = wide[p];
                    if ((x > y) == ((i & k) == 0)) { wide[i] = y; wide[p] = x; }
                }
                __syncthreads();
            }
        const int i = threadIdx.x;  // m <= 256: one entry per thread
        uint64_t e = 0;
        if (i < m) e = wide[i];
        __syncthreads();  // `to` may overlap `wide`
        if (i < m) {
            const uint32_t n = (uint32_t)(e >> 16) & 0xffffu;
            lane_at(out_row, i) = (uint16_t)((e >> 32) & 0xffffu);
            lane_at(out_len, i) = (uint16_t)n;
            if (out_key) lane_at(out_key, i) = key_of(n);
            lane_at(out_j, i) = (int32_t)lane_at(mine, (uint32_t)(e & 0xffffu)).y;  // a gather inside the block's own range
            to[i] = n;
        }
    } else {
        uint32_t most = 0;
        for (int i = threadIdx.x; i < m; i += 256) {
            const uint32_t lr = lane_at(mine, i).x;
            const uint32_t key = sort_key(lr >> 16);
            from[lr & 0xffffu] = (key << 16) | (uint32_t)i;
            most = max(most, key);
        }
        most = wave_max(most);
        if (most && lane == 0) atomicMax(&sh_max_key, most);
        __syncthreads();
        const uint32_t max_key = sh_max_key;
        const int passes = max_key ? (35 - __clz(max_key)) / 4 : 1;  // hex digits of the largest key; one pass at least: it closes the holes
        int len = cap;  // entries of `from` (with holes in the first pass)
        for (int pass = 0; pass < passes; pass++) {
            const int tiles = (len + 63) / 64, shift = 16 + 4 * pass;
            for (int i = threadIdx.x; i < 16 * tiles; i += 256) cnt[i] = 0u;
            __syncthreads();
            // the lanes of a tile with the same digit as this lane (its rank among them: the lanes below it)
            auto classify = [&](int tile, uint32_t &e, uint32_t &digit, uint64_t &same) __attribute__((always_inline)) {
                const int i = tile * 64 + lane;
                e = i < len ? from[i] : kHole;
                const bool valid = e != kHole;
                digit = (e >> shift) & 15u;
                const uint64_t there = __ballot(valid);
                uint32_t same_lo = (uint32_t)there, same_hi = (uint32_t)(there >> 32);
#pragma unroll
                for (int bit = 0; bit < 4; bit++) {
                    // (holes may count as whatever they hold: they are not in `same` to begin with)
                    const uint32_t set = (uint32_t)((int32_t)(digit << (31 - bit)) >> 31);  // all ones or zero
                    const uint64_t with = __ballot(set != 0u);
                    same_lo &= ~((uint32_t)with ^ set);
                    same_hi &= ~((uint32_t)(with >> 32) ^ set);
                }
                same = (uint64_t)same_hi << 32 | same_lo;
                return valid;
            };
            // the first kKeep tiles of a wavefront (all of them up to R = 2048) keep their entry,
            // counter and rank in registers for the scatter; tiles beyond are classified again
            constexpr int kKeep = 8;
            uint32_t kept_e[kKeep], kept_at[kKeep];  // kept_at: counter index << 6 | rank
#pragma unroll
            for (int t = 0; t < kKeep; t++) {
                const int tile = wave + 4 * t;
                kept_e[t] = kHole;
                kept_at[t] = 0u;
                if (tile < tiles) {
                    uint32_t digit;
                    uint64_t same;
                    const bool valid = classify(tile, kept_e[t], digit, same);
                    const uint32_t rank = (uint32_t)lanes_below(same), at = __umul24(digit, (uint32_t)tiles) + (uint32_t)tile;
                    if (valid && rank == 0) cnt[at] = (uint32_t)__popcll(same);
                    kept_at[t] = (at << 6) | rank;
                }
            }
            for (int tile = wave + 4 * kKeep; tile < tiles; tile += 4) {
                uint32_t e, digit;
                uint64_t same;
                const bool valid = classify(tile, e, digit, same);
                if (valid && lanes_below(same) == 0) cnt[digit * tiles + tile] = (uint32_t)__popcll(same);
            }
            __syncthreads();
            scan_in_lds(cnt, 16 * tiles, sh_wave);
#pragma unroll
            for (int t = 0; t < kKeep; t++)
                if (kept_e[t] != kHole) to[cnt[kept_at[t] >> 6] + (kept_at[t] & 63u)] = kept_e[t];
            for (int tile = wave + 4 * kKeep; tile < tiles; tile += 4) {
                uint32_t e, digit;
                uint64_t same;
                const bool valid = classify(tile, e, digit, same);
                if (valid) to[cnt[digit * tiles + tile] + (uint32_t)lanes_below(same)] = e;
            }
            __syncthreads();
            uint32_t *t = from; from = to; to = t;
            len = m;
        }
        // `from` holds the m entries in (key, local row) order; `to` is free: the lengths go there
        for (int i = threadIdx.x; i < m; i += 256) {
            const uint32_t e = from[i];
            const uint2 entry = lane_at(mine, e & 0xffffu);  // the segment's place in the block's bucket (gathers inside the block's own range)
            const uint32_t lr = entry.x;
            lane_at(out_row, i) = (uint16_t)(lr & 0xffffu);
            lane_at(out_len, i) = (uint16_t)(lr >> 16);
            if (out_key) lane_at(out_key, i) = key_of(lr >> 16);
            lane_at(out_j, i) = (int32_t)entry.y;
            to[i] = lr >> 16;
        }
    }
    __syncthreads();
    // a wavefront per group (W <= 64 slots): nonzeros and longest row by a reduction over the lanes
    const int g0 = blk_group_ptr[b], ng = (m + W - 1) / W;
    int32_t *listed = reinterpret_cast<int32_t *>(from);  // the block's long groups (as many as groups at most)
    for (int gi = wave; gi < ng; gi += 4) {
        const int i = gi * W + lane;
        const uint32_t n = lane < W && i < m ? to[i] : 0u, sum = wave_sum(n), longest = wave_max(n);
        if (lane == 0) {
            group_nnz[g0 + gi] = sum;
            group_longest[g0 + gi] = longest;
            // only that long rows matter to the caller; one that has been beaten already need not queue up for the counter
            if (longest > heavy_rounds && longest > __hip_atomic_load(longest_all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(longest_all, longest);
            group_slot[g0 + gi] = s0 + gi * W;
            group_blk[g0 + gi] = b;
            if (long_groups && is_long_group((int32_t)sum, (int32_t)longest, flat_wpg)) listed[atomicAdd(&sh_long_n, 1u)] = g0 + gi;
        }
    }
    if (!long_groups) return;
    __syncthreads();
    const uint32_t found = sh_long_n;
    if (found == 0) return;
    if (threadIdx.x == 0) sh_long_at = atomicAdd(n_long, found);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < found; i += 256) long_groups[sh_long_at + i] = listed[i];
}

// ------------------------------------------------------------------ step 7: fill

// One group, one wavefront.  Round k stores the k-th nonzero of every lane that still has one,
// lanes in slot order; rows keep their CSR (ascending column) order.  col0 is the first column of
// the group's block column.  CUT: the rounds k0 .. k0 + kFillRounds - 1 alone.
template <bool CUT, typename T>
__device__ __forceinline__ void fill_group(int32_t g, int32_t k0, int32_t col0, int lane, int64_t nnz, const int32_t *__restrict__ csr_col,
                                           const T *__restrict__ csr_val, const int32_t *__restrict__ group_ptr,
                                           const int32_t *__restrict__ group_slot, const uint16_t *__restrict__ seg_len,
                                           const int32_t *__restrict__ slot_j, uint16_t *__restrict__ col_local, T *__restrict__ data)
{
    const int s0 = group_slot[g], cnt = group_slot[g + 1] - s0;
    const int len = lane < cnt ? seg_len[s0 + lane] : 0, n = CUT ? min(len, k0 + kFillRounds) : len;
    const int64_t j = lane < cnt ? slot_j[s0 + lane] : 0;
    uint32_t base = (uint32_t)group_ptr[g];
    if (CUT && k0 > 0) base += wave_sum((uint32_t)min(len, k0));
    // Where the element of a lane goes in a round that begins at `at`: in rounds that look for their live lanes the round's place is the
    // scalar part of the address and the lane's rank among them its vector part; where the lanes stay the same over several rounds the compiler
    // keeps base and rank in a 64-bit vector address and adds the round to it.  (With 64-bit vector addresses everywhere and every round of a
    // batch gone through, k_fill took 1027 us on the 4M x 1M lognormal matrix, k_fill_flat 247 on the 27-point grid of 128^3 and 350 on
    // R-MAT 2^20 in fp64; now 877, 225 and 322, or 267 where the groups are cut.  What bounds k_fill since is the latency of L2: a
    // 128-byte line per segment and array, 103M of them, 300 cycles each, 59 on their way per compute unit, L1 held up by pending ones in 78 % of
    // its cycles; their 15 TB/s are not what L2 could deliver.  k_fill_flat on the grid streams 780 MB at 3.5 TB/s.)
    auto put = [&](uint32_t at, uint32_t rank, int32_t c, T v) __attribute__((always_inline)) {
        char *const round_col = reinterpret_cast<char *>(col_local) + ((uint64_t)at << 1);
        char *const round_val = reinterpret_cast<char *>(data) + (uint64_t)at * sizeof(T);
        *reinterpret_cast<uint16_t *>(round_col + (rank << 1)) = (uint16_t)(c - col0);
        *reinterpret_cast<T *>(round_val + rank * (uint32_t)sizeof(T)) = v;
    };
    // eight rounds at a time: the sixteen loads are independent of each other and of the stores
    constexpr int kRounds = 8, kLongRounds = 32;
    for (int k = CUT ? k0 : 0; __ballot(k < n); k += kRounds) {
        // Few rows left, each with at least kLongRounds more nonzeros: the set of live lanes does
        // not change over these rounds, so round k + u of a live lane lands at base + u * m + its
        // rank, and a lane copies kLongRounds of its row at a time.  (Eight rounds per memory
        // round trip made the longest row of the matrix the critical path of the whole kernel.)
        for (;;) {
            const uint64_t live = __ballot(k < n);
            const int m = __popcll(live);
            if (m == 0 || m > 16 || __ballot(k + kLongRounds <= n) != live) break;
            if (k < n) {
                const uint32_t rank = (uint32_t)lanes_below(live);
                int32_t cl[kLongRounds];
                T vl[kLongRounds];
                __builtin_memcpy(cl, csr_col + j + k, sizeof cl);  // unaligned 16-byte loads
                __builtin_memcpy(vl, csr_val + j + k, sizeof vl);
#pragma unroll
                for (int u = 0; u < kLongRounds; u++) put(base + (uint32_t)(u * m), rank, cl[u], vl[u]);
            }
            base += (uint32_t)(kLongRounds * m);
            k += kLongRounds;
        }
        if (!__ballot(k < n)) break;
        int32_t c[kRounds];
        T v[kRounds];
        if (k + kRounds <= n) {
            // a full batch: 16-byte loads (the row starts at any multiple of 4 bytes; the copies
            // below are unaligned vector loads).  Lanes read different rows, so a 4-byte load
            // would cost a whole sector of L2 traffic per element.
            __builtin_memcpy(c, csr_col + j + k, sizeof c);
            __builtin_memcpy(v, csr_val + j + k, sizeof v);
        } else {
            // The end of a row: its elements are read four at a time all the same, as long as the
            // four lie inside the arrays (what is read past the row's end is not stored).  Lanes
            // read different rows: an instruction costs a line per lane whatever its width.
#pragma unroll
            for (int u = 0; u < kRounds; u++) {
                c[u] = 0;
                v[u] = T(0);
            }
#pragma unroll
            for (int q = 0; q < kRounds; q += 4) {
                if (k + q < n) {
                    if (j + k + q + 4 <= nnz) {
                        __builtin_memcpy(c + q, csr_col + j + k + q, 4 * sizeof(int32_t));
                        __builtin_memcpy(v + q, csr_val + j + k + q, 4 * sizeof(T));
                    } else {
#pragma unroll
                        for (int u = q; u < q + 4; u++)
                            if (k + u < n) {
                                c[u] = csr_col[j + k + u];
                                v[u] = csr_val[j + k + u];
                            }
                    }
                }
            }
        }
        const uint64_t first = __ballot(k < n);
        if (__ballot(k + kRounds <= n) == first) {  // no row ends in the batch: the same lanes in every round
            const uint32_t m = (uint32_t)__popcll(first);
            if (k < n) {
                const uint32_t rank = (uint32_t)lanes_below(first);
#pragma unroll
                for (int u = 0; u < kRounds; u++) put(base + (uint32_t)u * m, rank, c[u], v[u]);
            }
            base += kRounds * m;
            continue;
        }
#pragma unroll
        for (int u = 0; u < kRounds; u++) {
            const uint64_t live = __ballot(k + u < n);
            if (!live) break;  // wave-uniform: rounds past every row's end
            if (k + u < n) put(base, (uint32_t)lanes_below(live), c[u], v[u]);
            base += (uint32_t)__popcll(live);
        }
    }
}

// Workgroups take blocks as stripe_walk says, the wavefronts of one taking a block's groups in turn.
template <typename T>
__global__ __launch_bounds__(256) void k_fill(const int32_t *__restrict__ stripe_ptr, const int32_t *__restrict__ stripe_blk,
                                              int32_t NBR, int32_t B, int32_t parts,
                                              const int32_t *__restrict__ csr_col, const T *__restrict__ csr_val,
                                              const int32_t *__restrict__ group_ptr, const int32_t *__restrict__ group_slot,
                                              const int32_t *__restrict__ blk_group_ptr, const int32_t *__restrict__ blk_bn,
                                              const uint16_t *__restrict__ seg_len, const int32_t *__restrict__ slot_j,
                                              int32_t C, int64_t nnz, uint16_t *__restrict__ col_local, T *__restrict__ data)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const StripeWalk walk = stripe_walk(stripe_ptr, NBR, parts);
    for (int32_t entry = walk.k; entry < walk.k_end; entry += walk.step) {
        const int32_t b = stripe_blk[entry];
        const int32_t col0 = blk_bn[b] * C;
        const int32_t g_end = blk_group_ptr[b + 1];
        for (int32_t g = blk_group_ptr[b] + wave; g < g_end; g += 4)
            fill_group<false, T>(g, 0, col0, lane, nnz, csr_col, csr_val, group_ptr, group_slot, seg_len, slot_j, col_local, data);
    }
}

// fill_order: the groups row block by row block.
__global__ __launch_bounds__(256) void k_group_turns(const int32_t *__restrict__ group_blk, const int32_t *__restrict__ blk_group_ptr,
                                                    const uint32_t *__restrict__ blk_turn, int32_t G, int32_t *__restrict__ fill_order)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= G) return;
    const int32_t b = group_blk[g];
    fill_order[blk_turn[b] + (uint32_t)((int32_t)g - blk_group_ptr[b])] = (int32_t)g;
}

// The same with one wavefront per group, in the layout's own order, or in that of `fill_order`: then kFillChunk workgroups' groups in a row on one XCD, as
// the blocks of a row block share the lines of the CSR arrays (32 of them: R-MAT 2^20 in fp64 195 against 200 us, the 27-point grid of 128^3
// 243 against 220; 256: 208 and 220).  CUT: the first kFillRounds rounds of a group alone.
constexpr int kFillChunk = 128;
template <bool CUT, typename T>
__global__ __launch_bounds__(256) void k_fill_flat(const int32_t *__restrict__ fill_order, const int32_t *__restrict__ csr_col,
                                                   const T *__restrict__ csr_val, const int32_t *__restrict__ group_ptr,
                                                   const int32_t *__restrict__ group_slot, const int32_t *__restrict__ group_blk,
                                                   const int32_t *__restrict__ blk_bn, const uint16_t *__restrict__ seg_len,
                                                   const int32_t *__restrict__ slot_j, int32_t G, int32_t C, int64_t nnz,
                                                   uint16_t *__restrict__ col_local, T *__restrict__ data)
{
    const uint32_t x = blockIdx.x & 7u, q = blockIdx.x >> 3;
    const int64_t turn = ((int64_t)(8u * (q / kFillChunk) + x) * kFillChunk + q % kFillChunk) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t at = fill_order ? turn : (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (at >= G) return;
    const int32_t g = fill_order ? fill_order[at] : (int32_t)at;
    fill_group<CUT, T>(g, 0, blk_bn[group_blk[g]] * C, (int)(threadIdx.x & 63), nnz, csr_col, csr_val, group_ptr, group_slot, seg_len, slot_j, col_local, data);
}

// The rest of groups that are cut, entries (group, first round) of a list.  A workgroup of k_list_rest looks at 1024 groups and goes to
// the list's counter once: same-address atomics serialise at some 30 ns (listed by k_order_block, block by block: 66 us on R-MAT 2^20).
__global__ __launch_bounds__(256) void k_list_rest(const uint32_t *__restrict__ group_longest, int32_t G, int2 *__restrict__ rest,
                                                   uint32_t *__restrict__ n_rest)
{
    constexpr int kPer = 4;
    __shared__ uint32_t sh[4], sh_at;
    uint32_t more[kPer], mine = 0, total;
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const int64_t g = (int64_t)blockIdx.x * (256 * kPer) + 256 * u + threadIdx.x;
        const uint32_t longest = g < G ? group_longest[g] : 0u;
        more[u] = longest ? (longest - 1u) / kFillRounds : 0u;
        mine += more[u];
    }
    uint32_t at = block_excl_scan_256(mine, &total, sh);
    if (total == 0) return;
    if (threadIdx.x == 0) sh_at = atomicAdd(n_rest, total);
    __syncthreads();
    at += sh_at;
#pragma unroll
    for (int u = 0; u < kPer; u++)
        for (uint32_t t = 0; t < more[u]; t++)
            rest[at++] = {(int32_t)(blockIdx.x * (256 * kPer) + 256 * u + threadIdx.x), (int32_t)((t + 1u) * kFillRounds)};
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill_rest(const int2 *__restrict__ rest, const uint32_t *__restrict__ n_rest,
                                                   const int32_t *__restrict__ csr_col, const T *__restrict__ csr_val,
                                                   const int32_t *__restrict__ group_ptr, const int32_t *__restrict__ group_slot,
                                                   const int32_t *__restrict__ group_blk, const int32_t *__restrict__ blk_bn,
                                                   const uint16_t *__restrict__ seg_len, const int32_t *__restrict__ slot_j,
                                                   int32_t C, int64_t nnz, uint16_t *__restrict__ col_local, T *__restrict__ data)
{
    const uint32_t n = *n_rest;
    for (uint32_t i = blockIdx.x * 4u + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); i < n; i += gridDim.x * 4u) {
        const int32_t g = rest[i].x, k0 = rest[i].y;
        fill_group<true, T>(g, k0, blk_bn[group_blk[g]] * C, (int)(threadIdx.x & 63), nnz, csr_col, csr_val, group_ptr, group_slot, seg_len, slot_j,
                            col_local, data);
    }
}

// ------------------------------------------------------------------ steps 5-7 by row blocks
//
// Where row segments are short, steps 5 to 7 above are scattered accesses of a few bytes: the segments' way to their blocks, and the fill's gather,
// a 128-byte line per segment and array.  In CSR order a row block's segments and nonzeros lie side by side, and a workgroup holds
// all of a row block's segments (k_panel_slots) or a good part of its nonzeros (k_panel_fill) in registers and LDS: everything is then read and
// written in runs, and sorted on the chip.

constexpr int kPanelThreads = 1024, kPanelWaves = kPanelThreads / 64;
// A segment in two registers: length - 1, block column, row (15, 6, 11 bits); first nonzero counted from the row block's, rank in its block (18, 11).
constexpr int kPanelRows = 2048, kPanelColumns = 64;
constexpr int kPanelPer = 32, kPanelSlots = kPanelPer * kPanelThreads;  // segments of a row block at most
constexpr int kPanelNonzeros = 1 << 16;                                 // its nonzeros at most: places of 16 bits, and in 64 tiles
constexpr int kPanelLds = 148 * 1024;                                   // dynamic LDS of k_panel_slots at most (its own arrays: below 12 KB)
// Rounds in its list of tails at most: what a workgroup asks for of the LDS.  Builds, us, with 0 / 4096 / 12288, rows of 8 in 300 row blocks and long rows: forty of
// 5000 231 / 232 / 213, forty of 2000 214 / 204 / 206, ten of 1200 in one row block 235 / 225 / 204, 30 row blocks with 300 of 100 each 258 / 211 / 217.
constexpr int kPanelTails = 12288;
constexpr int kPanelShift = 2;                                          // a at most: a band of 64 rows and more keeps 4 remainders apart
// Row blocks, at least.  With 128 of them half of the device is idle; builds, us, block by block / by row blocks: templates of 262K rows (128 row blocks) 335 /
// 318, of 300K (147) 314 / 269, 524K (256) 428 / 333; lognormal 300K x 300K (147) 269 / 261, in fp64 280 / 285, 500K x 200K (245) in fp64 380 / 332.
constexpr int kPanelLeast = 128;
// Segments and 8-byte words of the CSR arrays, at least, for every 256 row blocks that hold something, a turn of the compute units with one row block to each: a turn's
// phases and barriers take some 15 us whatever the row blocks hold, and block by block a million segments take some 9 us more than by row blocks, a million
// words 2.  Where row blocks are empty fewer will do in proportion: the older kernels deal their workgroups out to all of them.  Builds, us, block by block / by row
// blocks, rows of Poisson lengths over 300,000 columns, by row blocks and millions a turn: 256: 3.8 149 / 143, 4.6 155 / 147, 6.6 168 / 154; 300: 2.7 164 / 182, 5.0 198 / 205,
// 7.0 235 / 227; 400: 3.6 179 / 187, 5.2 204 / 200, 6.6 227 / 217; 600: 3.6 216 / 228, 5.2 238 / 244, 6.6 295 / 276; 1000: 2.4 224 / 244, 3.7 260 / 268, 4.5 294 / 288, 6.5
// 373 / 316; 1500: 2.4 282 / 320, 3.7 339 / 339, 4.5 401 / 374; 2000: 2.4 338 / 382, 4.5 500 / 454; fp64 300: 3.5 170 / 181, 6.5 214 / 219, 9.2 265 / 251; 600: 4.7 232 / 238, 6.7 296 /
// 265; 1000: 3.0 245 / 254, 4.7 304 / 278; 100,000 columns, 1000: 3.8 246 / 271, 5.3 318 / 292, 6.7 379 / 330; 128 of 2000 row blocks 4.9 228 / 176, fp64, 60 of 2000 3.3 236 /
// 178, 300 of 2000 2.2 236 / 200.  (The first turn: a million less, as not going by row blocks has by then cost the marks of where segments start, some 4 us.)
// Where a long row lies in long segments, block by block all wait for the wavefront that fills its group, and row blocks pay whatever they hold: rows of 8 and one of
// 600 / 2000 / 5000 / 10,000 / 20,000 / 32,000 in 300 row blocks 194 / 192, 220 / 192, 288 / 191, 397 / 197, 638 / 302, 997 / 383 (with forty of them 206 / 202, 246 / 200, 339 / 210,
// 500 / 229, 842 / 336, 1179 / 419; fewer than that gain: ten of 3000 in one row block 261 / 291, 30 row blocks with fifteen of 2000 277 / 293).
constexpr int kPanelTurn = 256;
constexpr int64_t kPanelMost = ((int64_t(1) << 32) - 1) / kPanelThreads;  // workgroups: a grid has fewer than 2^32 threads (the lists never name more than there would be without)
constexpr double kPanelWork = 4.5e6, kPanelWorkOnce = 1e6;
constexpr int kPanelLongRow = 1024;

// Words of 64 rows; an odd number of them, so that neighbouring segments, which differ in their block columns, lie in different banks.
__host__ __device__ inline uint32_t panel_row_words(int32_t R) { return (((uint32_t)R + 63u) / 64u) | 1u; }

// Bytes of a group's row in k_panel_slots' table, 8 * 2^a entries (an odd number of words: neighbouring groups' entries for a round lie in different banks).
__host__ __device__ inline uint32_t panel_table_row(uint32_t a) { return 2u * ((8u << a) + 2u); }

// The part of the list that holds the segments of a row block that has some.
struct Panel {
    uint32_t p0, p1;    // its nonzeros
    int32_t t0;         // tile of the first of them
    uint32_t skip;      // segments of that tile that belong to the row block before
    uint32_t upto;      // lane l: the row block's segments in the tiles t0 .. t0 + l
};

__device__ __forceinline__ Panel panel_of(int32_t bm, const int32_t *__restrict__ ptr, int64_t n_rows, int32_t R, const Tile *__restrict__ tiles,
                                          const uint64_t *__restrict__ word_starts, const uint16_t *__restrict__ word_at)
{
    const int lane = threadIdx.x & 63;
    Panel p;
    p.p0 = (uint32_t)ptr[(int64_t)bm * R];
    p.p1 = (uint32_t)ptr[min(((int64_t)bm + 1) * R, n_rows)];
    p.t0 = (int32_t)(p.p0 / kTile);
    const uint32_t last = p.p1 - 1;
    const int32_t t1 = (int32_t)(last / kTile), t = p.t0 + lane;
    p.skip = word_at[p.p0 / 64] + (uint32_t)__popcll(word_starts[p.p0 / 64] & ((1ull << (p.p0 & 63u)) - 1ull));
    const uint32_t up_to_last = word_at[last / 64] + (uint32_t)__popcll(word_starts[last / 64] & ((2ull << (last & 63u)) - 1ull));
    uint32_t n = t < t1 ? (uint32_t)tiles[t].count : t == t1 ? up_to_last : 0u;
    if (lane == 0) n -= p.skip;
    p.upto = sum_up_to_lane(n);
    return p;
}

// One workgroup per row block: the segments of all its blocks are put in order of (key, row), which gives every segment its slot, and every
// nonzero its place in the layout, counted in the row block's nonzeros: `places`, in the order of the CSR arrays.
// Compact sort codes only (see k_order_block): `codes` of them, (9 << a) - 1.  A bit per row, code and block column; the bits in front of a
// segment's own, counted, are its rank in the block, whatever order the bits were set in.
// In a group the rows of fewer than 8 * 2^a (`head`) nonzeros are in the order of their lengths and the others come behind, so in each of the first `head`
// rounds the lanes from some lane on have a nonzero: lane q's is the q-th behind table[group][round].  The places of the rounds behind these, which
// few groups have, come from a list of their lanes, or, where there is no room for them in it, are written group by group.
// The LDS holds in turn where the segments start, the bits with their counts, the slots with the table behind them, and in place of the slots, in CSR order,
// a segment's group and lane (10 and 6 bits) and the last 16 bits of where it starts.
// Bound by its instructions and by the waits between its phases, since the LDS has room for one workgroup on a CU: lognormal 4M x 1M, 1954 row blocks of 24,500
// segments, 461 us, in place of 301 + 368 for k_place and k_order_block.  Of 140,000 cycles a row block 21,000 pass until the segments are there, 52,000 with bits,
// ranks and slots (with an even number of words per code 64 neighbouring segments met in two banks: 495 against 343 us for the kernel as it was then),
// 29,000 with table and tails (the table by ballots, group by group: 50,000), 33,000 with the places.
__global__ __launch_bounds__(kPanelThreads) void k_panel_slots(const int32_t *__restrict__ row_blocks, const int32_t *__restrict__ ptr, int64_t n_rows, int32_t R, int32_t NBR, int32_t NBC,
                                                               const Tile *__restrict__ tiles, const uint64_t *__restrict__ word_starts,
                                                               const uint16_t *__restrict__ word_at, const uint32_t *__restrict__ list, int32_t row_bits,
                                                               const uint32_t *__restrict__ slot_off, const uint32_t *__restrict__ group_off,
                                                               const uint32_t *__restrict__ blk_id, uint32_t a, uint32_t heavy_rounds,
                                                               uint32_t *__restrict__ longest_all, uint16_t *__restrict__ row_local,
                                                               uint16_t *__restrict__ seg_len, uint32_t *__restrict__ slot_key,
                                                               uint32_t *__restrict__ group_nnz, uint32_t *__restrict__ group_longest,
                                                               int32_t *__restrict__ group_slot, int32_t *__restrict__ group_blk,
                                                               int32_t *__restrict__ blk_shift, uint16_t *__restrict__ places,
                                                               int32_t *__restrict__ slot_j, uint32_t most_tails)
{
    extern __shared__ __align__(8) uint32_t panel_lds[];
    __shared__ uint32_t sh_slot[kPanelColumns + 1], sh_group[kPanelColumns + 1];  // slots and groups of the row block in front of a block column
    __shared__ uint32_t sh_first[kPanelColumns];                                  // the block's first slot
    constexpr int kGroups = kPanelSlots / 64 + kPanelColumns;
    __shared__ uint32_t sh_sum[kGroups];    // nonzeros of a group; nonzeros in front of it
    __shared__ uint16_t sh_longest[kGroups];
    __shared__ uint16_t sh_shorter[kPanelColumns << (3 + kPanelShift)];  // of a block, for each k below `head`: rows of up to k nonzeros
    __shared__ uint32_t sh_tail_rounds, sh_tails_n, sh_uneven_n;
    __shared__ uint16_t sh_uneven[kGroups];  // groups with rows of `head` nonzeros and more
    __shared__ uint16_t sh_tails[kGroups];  // groups with more rounds than the table and the list of tails hold
    const int32_t bm = row_blocks ? row_blocks[blockIdx.x] : (int32_t)blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (ptr[(int64_t)bm * R] == ptr[min(((int64_t)bm + 1) * R, n_rows)]) return;  // (few of them, or the list would leave them out)
    const Panel p = panel_of(bm, ptr, n_rows, R, tiles, word_starts, word_at);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)p.upto, 63);
    // lane bn: the block's first slot and group, slots and groups in front of it
    const int64_t d = (int64_t)min(lane, NBC - 1) * NBR + bm;
    const uint32_t s0 = slot_off[d], slots = lane < NBC ? slot_off[d + 1] - s0 : 0u, g0 = group_off[d], groups = (slots + 63) / 64, id = blk_id[d];
    const uint32_t slots_upto = sum_up_to_lane(slots), groups_upto = sum_up_to_lane(groups);
    if (wave == 0) {
        sh_slot[lane + 1] = slots_upto;
        sh_group[lane + 1] = groups_upto;
        if (lane == 0) sh_slot[0] = sh_group[0] = sh_tail_rounds = sh_tails_n = sh_uneven_n = 0u;
        sh_first[lane] = s0;
        if (slots) blk_shift[id] = (int32_t)a;
    }
    // the segments: a wavefront takes `turns` times 64 neighbouring ones
    uint32_t x[kPanelPer], y[kPanelPer];
    const uint32_t turns = (total + kPanelThreads - 1) / kPanelThreads;
    const uint32_t first0 = 64u * turns * (uint32_t)wave;
    uint32_t i0 = first0 + (uint32_t)lane;  // the u-th: i0 + 64 u
    // (between the phases: what one has computed of x and y is not kept in registers for the next)
    auto forget = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kPanelPer; u++) asm volatile("" : "+v"(x[u]), "+v"(y[u]));
        asm volatile("" : "+v"(i0));
    };
    auto there = [&](int u) { return (uint32_t)u < turns && i0 + 64u * u < total; };
    const uint32_t *const here = list + (int64_t)p.t0 * kTile;
    int32_t tile = min(__popcll(__ballot(p.upto <= first0)), 63);
    uint32_t begin = tile > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)p.upto, tile > 0 ? tile - 1 : 0) : 0u;
    uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)p.upto, tile);
#pragma unroll
    for (int u = 0; u < kPanelPer; u++) {  // where in the list
        const uint32_t first = first0 + 64u * u, i = i0 + 64u * u;
        y[u] = p.skip;
        if ((uint32_t)u >= turns || first >= total) continue;
        uint32_t at = (uint32_t)tile * kTile - begin + i;
        while (end < min(first + 64u, total)) {  // wave-uniform
            tile++;
            begin = end;
            end = (uint32_t)__builtin_amdgcn_readlane((int)p.upto, tile);
            if (i >= begin) at = (uint32_t)tile * kTile - begin + i;
        }
        if (at < (uint32_t)kTile) at += p.skip;
        if (i < total) y[u] = at;
    }
#pragma unroll
    for (int u = 0; u < kPanelPer; u++) {
        x[u] = 0u;
        if ((uint32_t)u < turns) x[u] = lane_at(here, y[u]);
    }
    forget();  // (all loads are on their way at once)
#pragma unroll
    for (int u = 0; u < kPanelPer; u++) {
        const uint32_t e = x[u], bn = e >> kPlaceBits >> row_bits, row = e >> kPlaceBits & ((1u << row_bits) - 1u);
        y[u] = (uint32_t)p.t0 * kTile + (y[u] & ~(uint32_t)(kTile - 1)) + (e & (kTile - 1)) - p.p0;
        x[u] = bn << 11 | row;
        if (there(u)) panel_lds[i0 + 64u * u] = y[u];
    }
    __syncthreads();
    forget();
    const uint32_t row_words = panel_row_words(R), codes = (9u << a) - 1u, words = row_words * codes;
    auto word_of = [&](uint32_t v) {  // of the segment in v
        const uint32_t n = (v >> 17) + 1u, code = ((min(n >> a, 8u) << a) | (n & ((1u << a) - 1u))) - 1u;
        return __umul24(__umul24(v >> 11 & 63u, codes) + code, row_words) + ((v & 2047u) >> 6);
    };
#pragma unroll
    for (int u = 0; u < kPanelPer; u++) {
        const uint32_t i = i0 + 64u * u;
        if (there(u)) x[u] |= ((i + 1 < total ? panel_lds[i + 1] : p.p1 - p.p0) - y[u] - 1u) << 17;
        y[u] |= word_of(x[u]) << 18;  // (below 2^14: ten bytes each fit the LDS)
    }
    __syncthreads();
    forget();
    uint64_t *const bits = reinterpret_cast<uint64_t *>(panel_lds);
    uint16_t *const before = reinterpret_cast<uint16_t *>(bits + (uint32_t)NBC * words);
    for (uint32_t i = threadIdx.x; i < (uint32_t)NBC * words; i += kPanelThreads) bits[i] = 0ull;
    __syncthreads();
    forget();
#pragma unroll
    for (int u = 0; u < kPanelPer; u++)
        if (there(u)) (void)atomicOr(panel_lds + 2 * (y[u] >> 18) + (x[u] >> 5 & 1u), 1u << (x[u] & 31u));
    __syncthreads();
    forget();
    const uint32_t per = (words + 63) / 64;
    for (int bn = wave; bn < NBC; bn += kPanelWaves) {
        const uint32_t lo = min((uint32_t)lane * per, words), hi = min(lo + per, words);
        const uint64_t *const mine = bits + (uint32_t)bn * words;
        uint32_t n = 0;
        for (uint32_t i = lo; i < hi; i++) n += (uint32_t)__popcll(mine[i]);
        uint32_t run = sum_up_to_lane(n) - n;
        for (uint32_t i = lo; i < hi; i++) {
            before[(uint32_t)bn * words + i] = (uint16_t)run;
            run += (uint32_t)__popcll(mine[i]);
        }
    }
    __syncthreads();
    forget();
    const int32_t head = 8 << a;
    for (uint32_t i = threadIdx.x; i < (uint32_t)NBC * (uint32_t)head; i += kPanelThreads)
        sh_shorter[i] = before[(i >> (3u + a)) * words + (i & (uint32_t)(head - 1)) * row_words];
#pragma unroll
    for (int u = 0; u < kPanelPer; u++)
        if (there(u)) {
            const uint32_t w = y[u] >> 18;
            y[u] = (y[u] & 0x3ffffu) | (before[w] + (uint32_t)__popcll(bits[w] & ((1ull << (x[u] & 63u)) - 1ull))) << 18;
        }
    __syncthreads();
    forget();
#pragma unroll
    for (int u = 0; u < kPanelPer; u++)
        if (there(u)) panel_lds[sh_slot[x[u] >> 11 & 63u] + (y[u] >> 18)] = (x[u] & 2047u) << 16 | ((x[u] >> 17) + 1u);
    __syncthreads();
    forget();
    const uint32_t all_groups = (uint32_t)__builtin_amdgcn_readlane((int)groups_upto, 63);
    const uint32_t stride = panel_table_row(a) / 2u;
    // behind the slots, or what takes their place: lanes and places of the rounds behind the first `head`; the table
    uint64_t *const tail_lanes = reinterpret_cast<uint64_t *>(panel_lds + ((total + 1u) & ~1u));
    uint16_t *const tail_places = reinterpret_cast<uint16_t *>(tail_lanes + most_tails), *const table = tail_places + most_tails;
    auto block_of = [&](uint32_t gi) __attribute__((always_inline)) {
        int bn = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
            if (sh_group[bn + step] <= gi) bn += step;
        return bn;
    };
    // the slots' arrays, a wavefront per group
    for (uint32_t gi = wave; gi < all_groups; gi += kPanelWaves) {
        const int bn = __popcll(__ballot(groups_upto <= gi));
        const uint32_t q0 = 64u * (gi - (uint32_t)__builtin_amdgcn_readlane((int)(groups_upto - groups), bn));  // the group's first slot in its block
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)(slots_upto - slots), bn) + q0;             // and in the row block
        const uint32_t slot = (uint32_t)__builtin_amdgcn_readlane((int)s0, bn) + q0;
        if ((uint32_t)lane < (uint32_t)__builtin_amdgcn_readlane((int)slots, bn) - q0) {
            const uint32_t v = panel_lds[at + lane];
            lane_at(row_local + slot, lane) = (uint16_t)(v >> 16);
            lane_at(seg_len + slot, lane) = (uint16_t)v;
            if (slot_key) lane_at(slot_key + slot, lane) = hash_key(v & 0xffffu, a, (uint32_t)R / 9u, (uint32_t)R);
        }
    }
    // The table, an entry per lane, 64 / head groups at a time: from the group's first nonzero on, the round's place less the lanes that have none.
    for (uint32_t i0 = 64u * (uint32_t)wave; i0 < all_groups * (uint32_t)head; i0 += kPanelThreads) {
        const uint32_t i = i0 + (uint32_t)lane, gi = min(i >> (3u + a), all_groups - 1u), k = i & (uint32_t)(head - 1);
        const int bn = block_of(gi);
        const int32_t q0 = 64 * (int32_t)(gi - sh_group[bn]), count = min((int32_t)(sh_slot[bn + 1] - sh_slot[bn]) - q0, 64);
        const int32_t shorter = (int32_t)sh_shorter[((uint32_t)bn << (3u + a)) + k] - q0, none = min(max(shorter, 0), count);
        int32_t upto = count - none;  // nonzeros of the rounds up to this one
        for (int32_t d = 1; d < head; d <<= 1) {
            const int32_t t = __shfl_up(upto, d);
            if ((int32_t)k >= d) upto += t;
        }
        const uint64_t longer = __ballot(shorter < count);  // a row has more than k nonzeros
        const uint32_t longest = (uint32_t)__popcll(longer >> (lane & ~(head - 1)) & ((1ull << head) - 1ull));
        if (i < all_groups * (uint32_t)head) {
            table[gi * stride + k] = (uint16_t)(upto - (count - none) - none);
            if (k == (uint32_t)head - 1u) {
                sh_sum[gi] = (uint32_t)upto;
                sh_longest[gi] = (uint16_t)longest;
                if (longest == (uint32_t)head) sh_uneven[atomicAdd(&sh_uneven_n, 1u)] = (uint16_t)gi;
            }
        }
    }
    __syncthreads();
    // groups with rows of `head` nonzeros and more: their longest row and place in the list of tails
    auto lengths_of = [&](uint32_t gi) __attribute__((always_inline)) {  // gi the same in all lanes
        const int bn = __popcll(__ballot(groups_upto <= gi));
        const uint32_t q0 = 64u * (gi - (uint32_t)__builtin_amdgcn_readlane((int)(groups_upto - groups), bn));
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)(slots_upto - slots), bn) + q0;
        return (int32_t)((uint32_t)lane < (uint32_t)__builtin_amdgcn_readlane((int)slots, bn) - q0 ? panel_lds[at + lane] & 0xffffu : 0u);
    };
    const uint32_t uneven = sh_uneven_n;
    for (uint32_t i = wave; i < uneven; i += kPanelWaves) {
        const uint32_t gi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_uneven[i]);
        const uint32_t n = (uint32_t)lengths_of(gi), longest = wave_max(n), rounds = longest - (uint32_t)head, sum = wave_sum(n);
        if (lane == 0) {
            sh_sum[gi] = sum;
            sh_longest[gi] = (uint16_t)longest;
            const uint32_t tail = rounds ? atomicAdd(&sh_tail_rounds, rounds) : 0u;
            const bool room = tail + rounds <= most_tails;
            table[gi * stride + (uint32_t)head] = room ? (uint16_t)tail : (uint16_t)0xffffu;
            if (!room) sh_tails[atomicAdd(&sh_tails_n, 1u)] = (uint16_t)gi;
        }
    }
    __syncthreads();
    forget();
    // the list of tails, the wavefronts taking 64 rounds of a group in turn
    for (uint32_t b0 = 0; b0 < uneven; b0 += 64) {
        const uint32_t mine = sh_uneven[min(b0 + (uint32_t)lane, uneven - 1u)], tail_of = table[mine * stride + (uint32_t)head];
        const uint32_t rounds_of = b0 + (uint32_t)lane < uneven && tail_of != 0xffffu ? sh_longest[mine] - (uint32_t)head : 0u;
        const uint32_t pieces = (rounds_of + 63u) / 64u, pieces_upto = sum_up_to_lane(pieces), all = (uint32_t)__builtin_amdgcn_readlane((int)pieces_upto, 63);
        for (uint32_t piece = wave; piece < all; piece += kPanelWaves) {
            const int l = __popcll(__ballot(pieces_upto <= piece));
            const uint32_t r0 = 64u * (piece - (uint32_t)__builtin_amdgcn_readlane((int)(pieces_upto - pieces), l));
            const uint32_t r1 = min((uint32_t)__builtin_amdgcn_readlane((int)rounds_of, l), r0 + 64u), tail = (uint32_t)__builtin_amdgcn_readlane((int)tail_of, l);
            const int32_t n = lengths_of((uint32_t)__builtin_amdgcn_readlane((int)mine, l));
            uint32_t at = wave_sum((uint32_t)min(n, head + (int32_t)r0));
            for (uint32_t r = r0; r < r1; r += 8) {
                int32_t lanes_lo = 0, lanes_hi = 0, begin = 0;
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    const uint64_t live = __builtin_amdgcn_ballot_w64(n > head + (int32_t)r + t);
                    lanes_lo = with_lane((int32_t)(uint32_t)live, t, lanes_lo);
                    lanes_hi = with_lane((int32_t)(live >> 32), t, lanes_hi);
                    begin = with_lane((int32_t)at, t, begin);
                    at += (uint32_t)__popcll(live);
                }
                if (lane < 8 && r + (uint32_t)lane < r1) {
                    tail_lanes[tail + r + (uint32_t)lane] = (uint64_t)(uint32_t)lanes_hi << 32 | (uint32_t)lanes_lo;
                    tail_places[tail + r + (uint32_t)lane] = (uint16_t)begin;
                }
            }
        }
    }
    // the groups' numbers, 64 groups at a time
    for (uint32_t b0 = 64u * (uint32_t)wave; b0 < all_groups; b0 += kPanelThreads) {
        const uint32_t gi = min(b0 + (uint32_t)lane, all_groups - 1u), longest = sh_longest[gi];
        const int bn = block_of(gi);
        const uint32_t in_block = gi - sh_group[bn], g = (uint32_t)__shfl((int)g0, bn) + in_block;
        const int32_t block = __shfl((int)id, bn);
        if (b0 + (uint32_t)lane < all_groups) {
            group_nnz[g] = sh_sum[gi];
            group_longest[g] = longest;
            group_slot[g] = (int32_t)(sh_first[bn] + 64u * in_block);
            group_blk[g] = block;
        }
        const uint32_t most = wave_max(longest);  // only that long rows matter to the caller
        if (lane == 0 && most > heavy_rounds && most > __hip_atomic_load(longest_all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(longest_all, most);
    }
    __syncthreads();
    forget();
    if (wave == 0) {
        uint32_t run = 0;
        for (uint32_t i0 = 0; i0 < all_groups; i0 += 64) {
            const uint32_t n = i0 + lane < all_groups ? sh_sum[i0 + lane] : 0u, upto = sum_up_to_lane(n);
            if (i0 + lane < all_groups) sh_sum[i0 + lane] = run + upto - n;
            run += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        }
    }
#pragma unroll
    for (int u = 0; u < kPanelPer; u++) {
        const uint32_t bn = x[u] >> 11 & 63u, q = y[u] >> 18, j = y[u] & 0x3ffffu;
        if (there(u)) {
            panel_lds[i0 + 64u * u] = (64u * sh_group[bn] + q) << 16 | (j & 0xffffu);
            if ((x[u] >> 17) >= (uint32_t)head) slot_j[sh_first[bn] + q] = (int32_t)(p.p0 + j);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < all_groups * (uint32_t)head; i += kPanelThreads) {
        const uint32_t gi = i >> (3u + a);
        table[gi * stride + (i & (uint32_t)(head - 1))] += (uint16_t)sh_sum[gi];
    }
    __syncthreads();
    // the rounds for which there was no room: the first 64 of a group by a wavefront, the rest by all, 32 rounds at a time
    const uint32_t n_tails = sh_tails_n;
    auto place_rounds = [&](uint32_t gi, int32_t k0, int32_t most, int32_t step) __attribute__((always_inline)) {  // k0 .. k0 + most - 1, and so on every `step`
        const int bn = __popcll(__ballot(groups_upto <= gi));
        const uint32_t q0 = 64u * (gi - (uint32_t)__builtin_amdgcn_readlane((int)(groups_upto - groups), bn));
        const uint32_t slot = (uint32_t)__builtin_amdgcn_readlane((int)s0, bn) + q0;
        const int32_t n = (uint32_t)lane < (uint32_t)__builtin_amdgcn_readlane((int)slots, bn) - q0 ? (int32_t)lane_at(seg_len + slot, lane) : 0;
        uint16_t *const mine = n > head ? places + lane_at(slot_j + slot, lane) : places;
        for (; __ballot(n > k0); k0 += step) {
            uint32_t at = sh_sum[gi] + wave_sum((uint32_t)min(n, k0));
            for (int32_t k = k0; k < k0 + most; k++) {
                const uint64_t live = __ballot(n > k);
                if (!live) break;
                if (n > k) mine[k] = (uint16_t)(at + (uint32_t)lanes_below(live));
                at += (uint32_t)__popcll(live);
            }
            if (step == 0) return (bool)__ballot(n > k0 + most);
        }
        return false;
    };
    for (uint32_t i = wave; i < n_tails; i += kPanelWaves) {
        const uint32_t gi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_tails[i]);
        if (place_rounds(gi, head, 64, 0) && lane == 0) sh_tails[i] = (uint16_t)(gi | 0x8000u);
    }
    // The other nonzeros, 64 neighbouring ones at a time (a word of word_starts), the wavefront's l-th word in lane l, 64 words at a time.  A nonzero's
    // segment is the last one that starts at or before it.
    auto round_of = [&](uint32_t j, uint32_t f) { return (j - f) & 0xffffu; };  // j: in the row block
    auto entry_of = [&](uint32_t j, uint32_t f) { return (uint32_t)table[__umul24(f >> 22, stride) + min(round_of(j, f), (uint32_t)head - 1u)] + (f >> 16 & 63u); };
    auto place_tail = [&](uint32_t j, uint32_t f) __attribute__((always_inline)) {
        const uint32_t k = round_of(j, f), gi = f >> 22;
        if (k < (uint32_t)head) return;
        const uint32_t tail = table[__umul24(gi, stride) + (uint32_t)head];
        if (tail == 0xffffu) return;
        const uint32_t i = tail + k - (uint32_t)head;
        lane_at(places + p.p0, j) = (uint16_t)(sh_sum[gi] + tail_places[i] + (uint32_t)__popcll(tail_lanes[i] & ((1ull << (f >> 16 & 63u)) - 1ull)));
    };
    const uint32_t w0 = (p.p0 + 63u) / 64u, w1 = p.p1 / 64u;  // whole words
    for (uint32_t b0 = w0 + wave; b0 < w1; b0 += 64u * kPanelWaves) {
        const uint32_t w = min(b0 + (uint32_t)(kPanelWaves * lane), w1 - 1u);
        const uint64_t starts = word_starts[w];
        const int32_t t = (int32_t)(w / kTileWords) - p.t0;
        const uint32_t in_tiles = (uint32_t)__shfl((int)p.upto, t > 0 ? t - 1 : 0);
        const uint32_t base = (t > 0 ? in_tiles : 0u - p.skip) + word_at[w] + ((uint32_t)starts & 1u) - 1u;  // the segment of the word's first nonzero
        const uint32_t behind_lo = (uint32_t)(starts >> 1), behind_hi = (uint32_t)(starts >> 33);
        const int n_words = (int)min(64u, (w1 - b0 + kPanelWaves - 1) / kPanelWaves);
        constexpr int kAtOnce = 8;
        for (int l0 = 0; l0 < n_words; l0 += kAtOnce) {
            uint32_t f[kAtOnce], entry[kAtOnce];
            const uint32_t j = 64u * (b0 + (uint32_t)(kPanelWaves * l0)) - p.p0 + (uint32_t)lane;
#pragma unroll
            for (int u = 0; u < kAtOnce; u++) {
                const int l = min(l0 + u, n_words - 1);
                f[u] = panel_lds[__builtin_amdgcn_mbcnt_hi((uint32_t)__builtin_amdgcn_readlane((int)behind_hi, l),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)__builtin_amdgcn_readlane((int)behind_lo, l),
                                                                                     (uint32_t)__builtin_amdgcn_readlane((int)base, l)))];
            }
#pragma unroll
            for (int u = 0; u < kAtOnce; u++) entry[u] = entry_of(j + 64u * kPanelWaves * u, f[u]);
            bool tails = false;
#pragma unroll
            for (int u = 0; u < kAtOnce; u++) {
                const bool in_head = round_of(j + 64u * kPanelWaves * u, f[u]) < (uint32_t)head;
                tails |= !in_head;
                if (l0 + u < n_words && in_head) lane_at(places + 64ull * (b0 + (uint32_t)(kPanelWaves * (l0 + u))), lane) = (uint16_t)entry[u];
            }
            if (!__ballot(tails)) continue;
#pragma unroll
            for (int u = 0; u < kAtOnce; u++)
                if (l0 + u < n_words) place_tail(j + 64u * kPanelWaves * u, f[u]);
        }
    }
    if (wave < 2) {  // the words that hold the row block's first and last nonzero, and others'
        const uint32_t w = wave == 0 ? p.p0 / 64u : w1, j = 64u * w + (uint32_t)lane;
        if ((wave == 0 ? w < w0 : w * 64u < p.p1 && w >= w0) && j >= p.p0 && j < p.p1) {
            const int32_t t = (int32_t)(w / kTileWords) - p.t0;
            const uint32_t in_front = t > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)p.upto, t > 0 ? t - 1 : 0) : 0u - p.skip;
            const uint32_t f = panel_lds[in_front + word_at[w] + (uint32_t)__popcll(word_starts[w] & ((2ull << lane) - 1ull)) - 1u];
            if (round_of(j - p.p0, f) < (uint32_t)head) places[j] = (uint16_t)entry_of(j - p.p0, f);
            place_tail(j - p.p0, f);
        }
    }
    __syncthreads();
    for (uint32_t i = 0; i < n_tails; i++) {
        const uint32_t gi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_tails[i]);
        if (gi & 0x8000u) (void)place_rounds(gi & 0x7fffu, head + 64 + 32 * wave, 32, 32 * kPanelWaves);
    }
}

// The fill: a workgroup takes a share of a row block's nonzeros in the layout's order, `room` at most, and puts them in place in LDS; they come from the CSR arrays
// in their order, and what it writes are whole runs.  The shares of one row block run on one XCD, whose L2 then holds what all of them read.
// Bound by what it reads, 10 bytes a nonzero and share at 8 TB/s, and by its stores, one after the other as the LDS has room for one workgroup on a CU: lognormal
// 4M x 1M in 2.05 shares a row block 398 us, in place of 880 for k_fill.  (Two workgroups of 80 KB to a CU, so four shares: 488; of 512 threads 471.)
template <typename T>
__global__ __launch_bounds__(kPanelThreads) void k_panel_fill(const uint32_t *__restrict__ shares, const Findings *__restrict__ found,
                                                              const int32_t *__restrict__ ptr, int64_t n_rows, int32_t R, int32_t NBR, int32_t NBC, int32_t C,
                                                              uint32_t most_parts, uint32_t room, const uint16_t *__restrict__ places,
                                                              const int32_t *__restrict__ csr_col, const T *__restrict__ csr_val,
                                                              const uint32_t *__restrict__ group_off, const int32_t *__restrict__ group_ptr,
                                                              uint16_t *__restrict__ col_local, T *__restrict__ data)
{
    extern __shared__ __align__(8) uint32_t panel_lds[];
    T *const vals = reinterpret_cast<T *>(panel_lds);
    uint16_t *const cols = reinterpret_cast<uint16_t *>(vals + room);
    const uint32_t turn = blockIdx.x >> 3, xcd = blockIdx.x & 7u;
    const uint32_t entry = shares ? shares[blockIdx.x] : (8u * (turn / most_parts) + xcd) << kShareBits | turn % most_parts;
    const uint32_t share = entry & ((1u << kShareBits) - 1u);
    const int32_t bm = (int32_t)(entry >> kShareBits);
    if (shares ? turn >= found->dealt[xcd] : bm >= NBR) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t p0 = (uint32_t)ptr[(int64_t)bm * R], p1 = (uint32_t)ptr[min(((int64_t)bm + 1) * R, n_rows)];
    const int64_t d = (int64_t)min(lane, NBC - 1) * NBR + bm;
    const uint32_t g0 = group_off[d], g1 = lane < NBC ? group_off[d + 1] : g0;
    const uint32_t nonzeros = p1 - p0, parts = (nonzeros + room - 1) / room;
    if (share >= parts) return;
    const uint32_t each = (nonzeros + parts - 1) / parts, lo = each * share, hi = min(nonzeros, lo + each), size = hi - lo;
    auto put = [&](uint32_t place, int32_t column, T value) __attribute__((always_inline)) {
        const uint32_t at = place - lo;
        if (at < size) {
            vals[at] = value;
            cols[at] = (uint16_t)column;
        }
    };
    // whole runs of 256 nonzeros, four to a lane, and what lies in front of and behind them, one to a thread
    const uint32_t run0 = (p0 + 255u) / 256u, run1 = p1 / 256u;
    constexpr int kAtOnce = sizeof(T) == 4 ? 4 : 3;
    for (uint32_t run = run0 + wave; run < run1; run += kAtOnce * kPanelWaves) {
        uint16_t at[kAtOnce][4];
        int32_t c[kAtOnce][4];
        T v[kAtOnce][4];
#pragma unroll
        for (int u = 0; u < kAtOnce; u++) {
            const uint64_t j = 256ull * min(run + (uint32_t)(kPanelWaves * u), run1 - 1u);
            __builtin_memcpy(at[u], reinterpret_cast<const char *>(places + j) + 8u * (uint32_t)lane, sizeof at[u]);
            __builtin_memcpy(c[u], reinterpret_cast<const char *>(csr_col + j) + 16u * (uint32_t)lane, sizeof c[u]);  // (at any multiple of 4 bytes)
            __builtin_memcpy(v[u], reinterpret_cast<const char *>(csr_val + j) + 4u * (uint32_t)sizeof(T) * (uint32_t)lane, sizeof v[u]);
        }
#pragma unroll
        for (int u = 0; u < kAtOnce; u++) {
            if (run + (uint32_t)(kPanelWaves * u) >= run1) break;
#pragma unroll
            for (int i = 0; i < 4; i++) put(at[u][i], c[u][i], v[u][i]);
        }
    }
    const uint32_t in_front = run0 < run1 ? 256u * run0 : p1, behind = run0 < run1 ? 256u * run1 : p1;
    for (uint32_t j = p0 + threadIdx.x; j < in_front; j += kPanelThreads) put(places[j], csr_col[j], csr_val[j]);
    for (uint32_t j = behind + threadIdx.x; j < p1; j += kPanelThreads) put(places[j], csr_col[j], csr_val[j]);
    // lane bn: the block's place in the layout, its nonzeros, those in front of it
    const uint32_t e0 = (uint32_t)group_ptr[g0], elements = (uint32_t)group_ptr[g1] - e0, elements_upto = sum_up_to_lane(elements);
    const uint32_t to_layout = e0 + lo - (elements_upto - elements);  // a place in the share and this: the place in the layout
    const int bn_first = __popcll(__ballot(elements_upto <= lo)), bn_last = __popcll(__ballot(elements_upto < hi));
    __syncthreads();
    uint32_t next = (uint32_t)wave;  // 256 nonzeros of a block at a time
    for (int bn = bn_first; bn <= bn_last; bn++) {
        const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)elements_upto, bn);
        const uint32_t a = max((uint32_t)__builtin_amdgcn_readlane((int)(elements_upto - elements), bn), lo) - lo, b = min(upto, hi) - lo, col0 = (uint32_t)bn * (uint32_t)C;
        const uint32_t turns = b > a ? (b - a + 255u) / 256u : 0u, shift = (uint32_t)__builtin_amdgcn_readlane((int)to_layout, bn);
        for (; next < turns; next += kPanelWaves) {
            const uint32_t i0 = a + 256u * next;
            uint16_t *const to_col = col_local + (i0 + shift);
            T *const to_val = data + (i0 + shift);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const uint32_t i = i0 + 64u * u + (uint32_t)lane;
                if (i < b) {
                    lane_at(to_col, 64u * u + (uint32_t)lane) = (uint16_t)(cols[i] - col0);
                    lane_at(to_val, 64u * u + (uint32_t)lane) = vals[i];
                }
            }
        }
        next -= turns;
    }
}

// add_sign derived from seg_len (Section 3.2: distance to the row's next nonzero = nonzeros
// after it in this round + nonzeros before it in the next round + 1; -1 at the row's end).
__global__ __launch_bounds__(256) void k_add_sign(const int32_t *__restrict__ group_ptr, const int32_t *__restrict__ group_slot,
                                                  const uint16_t *__restrict__ seg_len, int32_t G, int32_t *__restrict__ add_sign)
{
    const int lane = threadIdx.x & 63;
    const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= G) return;
    const int s0 = group_slot[g], cnt = group_slot[g + 1] - s0;
    const int n = lane < cnt ? seg_len[s0 + lane] : 0;
    int64_t base = group_ptr[g];
    const uint64_t above_me = ~((2ull << lane) - 1ull);
    for (int k = 0;; k++) {
        const uint64_t live = __ballot(k < n);
        if (!live) break;
        const uint64_t next = __ballot(k + 1 < n);
        if (k < n) {
            const int64_t dst = base + lanes_below(live);
            add_sign[dst] = k + 1 < n ? __popcll(live & above_me) + lanes_below(next) + 1 : -1;
        }
        base += __popcll(live);
    }
}

// ------------------------------------------------------------------ Section 3.3: schedule
//
// Weight of a group = GW + its nonzeros + SW times its slots + RW times its rounds (GW =
// group_weight, SW = slot_weight, RW = round_weight: the costs of a group as such, of a row and
// of a round of a group, measured in nonzeros; a group has as many rounds as its longest row
// has nonzeros);
// Wt(g) = group_ptr[g] + SW * group_slot[g] + RW * group_rounds[g] + GW * g is the weight of all
// groups before g.
struct Weights {
    const int32_t *group_ptr, *group_slot, *group_rounds;
    int64_t SW, RW, GW;
    __device__ __forceinline__ int64_t before(int32_t g) const
    {
        return (int64_t)group_ptr[g] + SW * group_slot[g] + RW * group_rounds[g] + GW * g;
    }
};

// A few words that kernels write for the host: one synchronisation instead of a blocking copy per word.
constexpr int kReadback = 32;
struct Words { const void *at[kReadback]; };

constexpr int kColumnsKept = 2048;  // block columns whose first groups and ranks k_schedule keeps in LDS

// For more of them, col_rank[c], c in 0..NBC: block columns before c that hold a group (col_group_ptr[c]: first group of block column c).  One workgroup: every thread counts a contiguous piece, the pieces' counts are scanned, every
// thread writes its piece.
__global__ __launch_bounds__(256) void k_col_ranks(const int32_t *__restrict__ col_group_ptr, int32_t NBC, int32_t *__restrict__ col_rank)
{
    __shared__ uint32_t sh[4];
    const int32_t per = (NBC + 255) / 256, c0 = min(NBC, (int32_t)threadIdx.x * per), c1 = min(NBC, c0 + per);
    uint32_t mine = 0, total;
    for (int32_t c = c0; c < c1; c++) mine += col_group_ptr[c + 1] > col_group_ptr[c];
    uint32_t run = block_excl_scan_256(mine, &total, sh);
    for (int32_t c = c0; c < c1; c++) {
        col_rank[c] = (int32_t)run;
        run += col_group_ptr[c + 1] > col_group_ptr[c];
    }
    if (threadIdx.x == 0) col_rank[NBC] = (int32_t)total;
}

// One wavefront per worker w.
// fixed_start[w]: first g with Wc(g) * P >= w * Wc(G) (P contiguous ranges of equal weight), where
// Wc(g) = Wt(g) + CW * (block columns with a group that start before g): entering a block column
// costs a worker the fetch of its vector segment, charged to the column's first group;
// fixed_col[w]: the last block column that starts at or before that group.
// comp_lo[w]: first group of worker w's range left to competition: the first g in the range whose
// preceding weight inside the range reaches fixed_q8/256 of the range's weight, but not before
// the first group of the block column that holds the range's last group (comp_col[w]), so that
// the competitive groups of a range need one segment of the vector.
__global__ __launch_bounds__(256) void k_schedule(const int32_t *__restrict__ col_group_ptr, Weights wt,
                                                  const int32_t *__restrict__ col_rank, int64_t CW, int32_t NBC, int32_t G, int32_t P,
                                                  int32_t fixed_q8, int32_t *__restrict__ fixed_start, int32_t *__restrict__ fixed_col,
                                                  int32_t *__restrict__ comp_lo, int32_t *__restrict__ comp_col,
                                                  int64_t least_open, int32_t *__restrict__ own_end, int32_t *__restrict__ any_open,
                                                  Words words, int32_t n_words, uint32_t *__restrict__ host)
{
    // (for the host, words that are final since the kernels before)
    if (blockIdx.x == 0 && (int32_t)threadIdx.x < n_words) host[threadIdx.x] = *static_cast<const uint32_t *>(words.at[threadIdx.x]);
    __shared__ int32_t sh_first[kColumnsKept + 1];
    __shared__ uint16_t sh_rank[kColumnsKept + 1];  // block columns that hold a group before each
    __shared__ uint32_t sh[4];
    const bool kept = NBC <= kColumnsKept;
    if (kept) {
        for (int32_t c = threadIdx.x; c <= NBC; c += 256) sh_first[c] = col_group_ptr[c];
        __syncthreads();
        const int32_t per = (NBC + 255) / 256, c0 = min(NBC, (int32_t)threadIdx.x * per), c1 = min(NBC, c0 + per);
        uint32_t mine = 0, total;
        for (int32_t c = c0; c < c1; c++) mine += sh_first[c + 1] > sh_first[c];
        uint32_t run = block_excl_scan_256(mine, &total, sh);
        for (int32_t c = c0; c < c1; c++) {
            sh_rank[c] = (uint16_t)run;
            run += sh_first[c + 1] > sh_first[c];
        }
        if (threadIdx.x == 0) sh_rank[NBC] = (uint16_t)total;
    }
    __syncthreads();
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w > P) return;
    auto first_group = [&](int32_t c) { return kept ? sh_first[c] : col_group_ptr[c]; };
    auto before = [&](int32_t g) {
        int64_t v = wt.before(g);
        if (CW) {
            int32_t c_lo = 0, c_hi = NBC;  // first c in 0..NBC with col_group_ptr[c] >= g (col_group_ptr[NBC] = G)
            while (c_lo < c_hi) {
                const int32_t mid = c_lo + ((c_hi - c_lo) >> 1);
                if (first_group(mid) >= g) c_hi = mid; else c_lo = mid + 1;
            }
            v += CW * (kept ? (int32_t)sh_rank[c_lo] : col_rank[c_lo]);
        }
        return v;
    };
    auto column_of = [&](int32_t g) {  // largest c with col_group_ptr[c] <= g
        int32_t c_lo = 0, c_hi = NBC - 1;
        while (c_lo < c_hi) {
            const int32_t mid = c_lo + ((c_hi - c_lo + 1) >> 1);
            if (first_group(mid) <= g) c_lo = mid; else c_hi = mid - 1;
        }
        return c_lo;
    };
    const int64_t all = before(G);
    // (one search after the other: the kernel 12.4 us on the 27-point grid of 128^3, both at once 11.2; lognormal 4M x 1M 16.2 and 12.8)
    const int64_t target = (w + ((threadIdx.x & 32) >> 5)) * all;  // of this worker and of the next
    const int32_t starts = first_reached_by_halves(0, G, [&](int32_t g) { return before(g) * P >= target; });
    const int32_t g0 = __builtin_amdgcn_readlane(starts, 0);
    const bool writes = (threadIdx.x & 63) == 0;
    if (writes) fixed_start[w] = g0;
    if (w == P) return;
    const int32_t g1 = __builtin_amdgcn_readlane(starts, 32), col0 = column_of(g0);
    const int64_t w0 = wt.before(g0), need = (wt.before(g1) - w0) * fixed_q8;
    int32_t lo = first_reached(g0, g1, [&](int32_t g) { return (wt.before(g) - w0) * 256 >= need; });
    int32_t c = col0;
    if (g1 > g0) {
        c = column_of(g1 - 1);
        lo = max(lo, first_group(c));
    }
    if (writes) {
        fixed_col[w] = col0;
        comp_lo[w] = lo;
        comp_col[w] = c;
        // Competitive groups of less weight than `least_open` are the worker's own all the same: it runs them like its fixed
        // part, and where all ranges are like that nobody looks for one to enter.
        const bool open = lo < g1 && wt.before(g1) - wt.before(lo) >= least_open;
        own_end[w] = open ? lo : g1;
        if (open) *any_open = 1;
    }
}

// The paper's schedule (Section 3.3 read literally): worker w is pre-assigned the F blocks
// [w F, (w + 1) F) of the column-major block list; handed over as group ranges (the unit the
// kernels walk).  Nothing inside a range is competitive: the blocks from P F on are claimed one at
// a time through a single ticket counter.
__global__ __launch_bounds__(256) void k_paper_schedule(const int32_t *__restrict__ blk_group_ptr, const int32_t *__restrict__ blk_bn,
                                                        int64_t F, int32_t B, int32_t NBC, int32_t P, int32_t *__restrict__ fixed_start,
                                                        int32_t *__restrict__ fixed_col, int32_t *__restrict__ comp_lo,
                                                        int32_t *__restrict__ comp_col)
{
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w > P) return;
    const int64_t b = w * F;  // <= P F <= B
    fixed_start[w] = blk_group_ptr[b];
    if (w == P) return;
    const int32_t first_col = b < B ? blk_bn[b] : NBC - 1;
    fixed_col[w] = first_col;
    comp_lo[w] = blk_group_ptr[b + F];
    comp_col[w] = F > 0 ? blk_bn[b + F - 1] : first_col;
}

__global__ __launch_bounds__(256) void k_hash_keys(const uint32_t *__restrict__ n, int64_t count, uint32_t a, uint32_t R,
                                                   uint32_t *__restrict__ keys)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) keys[i] = hash_key(n[i], a, R / 9u ? R / 9u : 1u, R);
}

#define HBP_TRY(expr) do { int rc_ = (expr); if (rc_ != HBP_OK) return rc_; } while (0)

constexpr int kWorkspaceDevices = 64;  // devices whose memory is kept

// Allocations of freed handles, kept for the next ones: a program that rebuilds its matrix (time stepping,
// Newton) otherwise pays milliseconds per build for hipMalloc and hipFree of hundreds of megabytes
// (mapping and unmapping; stencil 128^3: 4.0 of 5.2 ms).  Bounded per device by kCacheBytes and
// kCacheBlocks, given back by hbp_release_workspace() and when an allocation fails.  A block comes here only
// after a wait for everything that used it has succeeded, so whatever stream gets it next finds it idle.
constexpr size_t kCacheBytes = size_t(4) << 30;
constexpr size_t kCacheBlocks = 16;
struct CachedBlock { void *base; size_t bytes; };
struct BlockCache {
    CachedBlock at[kCacheBlocks];  // oldest first
    size_t count = 0, bytes = 0;
    CachedBlock take(size_t i)
    {
        const CachedBlock c = at[i];
        for (size_t j = i + 1; j < count; j++) at[j - 1] = at[j];
        count--;
        bytes -= c.bytes;
        return c;
    }
};
BlockCache g_cache[kWorkspaceDevices];
std::mutex g_cache_mutex[kWorkspaceDevices];

int drop_cached_blocks(int device)
{
    int rc = HBP_OK;
    std::lock_guard<std::mutex> lock(g_cache_mutex[device]);
    BlockCache &cache = g_cache[device];
    while (cache.count > 0)
        if (hipFree(cache.take(0).base) != hipSuccess) rc = HBP_ERR_HIP;
    return rc;
}

}  // namespace

int device_alloc(int device, size_t bytes, void **out)
{
    hipError_t e = hipMalloc(out, bytes);
    if (e == hipErrorOutOfMemory && device >= 0 && device < kWorkspaceDevices) {
        (void)hipGetLastError();
        (void)drop_cached_blocks(device);
        e = hipMalloc(out, bytes);
    }
    HBP_HIP(e);
    return HBP_OK;
}

namespace {

// Scratch memory of the build, kept between builds: freeing a few hundred megabytes costs a
// quarter of a millisecond per allocation, a good part of a build.  Two slots per device (a
// build has two scratch arenas alive at a time), grown when a build needs more, given back by
// hbp_release_workspace().  The device's lock is held for the whole of build_layout: the builds
// of one process on one device are serialised; builds on different devices are not.
constexpr int kWorkspaceSlots = 2;
struct Workspace { void *base = nullptr; size_t bytes = 0; };
Workspace g_workspace[kWorkspaceDevices][kWorkspaceSlots];
std::mutex g_workspace_mutex[kWorkspaceDevices];

std::mutex &workspace_mutex(int device) { return g_workspace_mutex[device >= 0 && device < kWorkspaceDevices ? device : 0]; }

int workspace_get(int device, int slot, size_t bytes, void **out)
{
    if (device < 0 || device >= kWorkspaceDevices) return HBP_ERR_INTERNAL;
    Workspace &w = g_workspace[device][slot];
    if (w.bytes < bytes) {
        if (w.base) (void)hipFree(w.base);
        w.base = nullptr;
        w.bytes = 0;
        const size_t want = bytes + bytes / 8;  // some room, so that similar matrices do not reallocate
        HBP_TRY(device_alloc(device, want, &w.base));
        w.bytes = want;
    }
    *out = w.base;
    return HBP_OK;
}

// The smallest kept block that is large enough and not more than an eighth larger (the latest of several), or a new one of just
// the size.
int block_get(int device, size_t bytes, void **out, size_t *got)
{
    if (device >= 0 && device < kWorkspaceDevices) {
        std::lock_guard<std::mutex> lock(g_cache_mutex[device]);
        BlockCache &cache = g_cache[device];
        size_t best = cache.count;
        for (size_t i = 0; i < cache.count; i++)
            if (cache.at[i].bytes >= bytes && cache.at[i].bytes <= bytes + bytes / 8 && (best == cache.count || cache.at[i].bytes <= cache.at[best].bytes))
                best = i;
        if (best < cache.count) {
            const CachedBlock block = cache.take(best);
            *out = block.base;
            *got = block.bytes;
            return HBP_OK;
        }
    }
    *got = bytes;
    return device_alloc(device, bytes, out);
}

uint32_t *g_readback[kWorkspaceDevices];  // pinned; guarded by the device's workspace lock

int readback_get(int device, uint32_t **out)
{
    if (device < 0 || device >= kWorkspaceDevices) return HBP_ERR_INTERNAL;
    if (!g_readback[device]) HBP_HIP(hipHostMalloc((void **)&g_readback[device], kReadback * sizeof(uint32_t), hipHostMallocDefault));
    *out = g_readback[device];
    return HBP_OK;
}

// found: the largest of the copies, and the rest, go behind the words
__global__ __launch_bounds__(64) void k_publish(Words words, int32_t count, uint32_t *__restrict__ host, const Findings *__restrict__ found)
{
    const int i = threadIdx.x;
    if (i < count) host[i] = *static_cast<const uint32_t *>(words.at[i]);
    if (!found) return;
    const uint32_t longest = wave_max(found->copy[i].longest_row), segment = wave_max(found->copy[i].long_segment);
    const uint32_t dealt = i < 8 ? found->dealt[i] : 0u, most_shares = wave_max(dealt), shares = wave_sum(dealt);
    if (i == 0) {
        host[count] = longest;
        host[count + 1] = segment;
        host[count + 2] = found->most_slots;
        host[count + 3] = found->most_nonzeros;
        host[count + 4] = found->dealt[8];
        host[count + 5] = most_shares;
        host[count + 6] = shares;
    }
}

// One device allocation carved into 256-byte aligned arrays: reserve() every array first,
// commit() allocates once and hands out the pointers.  hipMalloc/hipFree calls are a large part
// of the preprocessing time otherwise (each hipFree synchronises the device).  An arena is
// either handed to the caller (the handle's arrays) or lives in a workspace slot.
class Arena {
public:
    explicit Arena(bool owned_by_caller, int device = -1, int workspace_slot = -1)
        : keep_(owned_by_caller), device_(device), slot_(workspace_slot) {}
    ~Arena() { if (free_at_end_ && base_) (void)hipFree(base_); }
    template <typename T>
    void reserve(T **out, int64_t count)
    {
        reserve_bytes((void **)out, (int64_t)sizeof(T) * (count > 0 ? count : 1));
    }
    void reserve_bytes(void **out, int64_t n_bytes)
    {
        const size_t bytes = ((size_t)(n_bytes > 0 ? n_bytes : 1) + 255) & ~(size_t)255;
        slots_.push_back({out, total_});
        total_ += bytes;
    }
    int commit()
    {
        if (keep_) {
            const int rc = block_get(device_, total_ ? total_ : 256, &base_, &bytes_);
            if (rc != HBP_OK) return rc;
        } else if (device_ < 0 || device_ >= kWorkspaceDevices || slot_ < 0 || slot_ >= kWorkspaceSlots) {
            HBP_TRY(device_alloc(device_, total_ ? total_ : 256, &base_));  // no workspace slot for it: freed when the build ends
            free_at_end_ = true;
        } else {
            const int rc = workspace_get(device_, slot_, total_ ? total_ : 256, &base_);
            if (rc != HBP_OK) return rc;
        }
        for (auto &s : slots_) *s.out = (char *)base_ + s.offset;
        return HBP_OK;
    }
    void *base() const { return base_; }
    size_t bytes() const { return bytes_; }
    size_t total() const { return total_; }

private:
    struct Slot { void **out; size_t offset; };
    std::vector<Slot> slots_;
    size_t total_ = 0, bytes_ = 0;  // bytes_: of the block, where the caller keeps it
    void *base_ = nullptr;
    bool keep_, free_at_end_ = false;
    int device_, slot_;
};

inline unsigned blocks_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

}  // namespace

// Parameters left at "choose for me" (Section 3.1 derives its 512 x 4096 from the shared memory of
// the paper's GPUs; here they follow the matrix and the 160 KB of LDS of a gfx950 compute unit):
//   C     the widest segment of x that fits the LDS budget of a worker (32768 fp32 / 16384 fp64
//         values), or the whole vector when it is shorter: every column block less means one
//         partial sum less per row, and the partial sums are the traffic the method adds;
//   R, rounds per batch
//         from the nonzeros the sampled rows have inside one column block (the sampling pass of
//         Section 3.2, which also yields the shift a): when at least half of the sampled segments
//         hold 6 or more nonzeros, the paper's R = 512 and deep batches (8 rounds, one group at a
//         time); otherwise R = 2048 (four times fewer, fuller blocks for the same slots) and 4
//         rounds with four groups in flight.  Both thresholds are measured on MI355X.
// The sampled shift is written back into p.hash_shift, so that the build does not sample again.
int choose_block_parameters(const int32_t *csr_ptr, const int32_t *csr_col, int64_t n_rows, int64_t n_cols, int32_t value_bytes,
                            hbp_params_t &p, int64_t *nnz_out, RowStats *rows_out, hipStream_t st)
{
    const int32_t max_c = value_bytes == 8 ? kMaxC64 : kMaxC;
    if (p.cols_per_block == 0) p.cols_per_block = (int32_t)std::min<int64_t>(max_c, n_cols);
    const bool need_stats = p.rows_per_block == 0 || p.rounds_per_batch == 0;
    if (!need_stats) return HBP_OK;
    if (p.cols_per_block < 1 || p.cols_per_block > max_c) return HBP_ERR_INVALID_ARGUMENT;
    int device = 0;
    HBP_HIP(hipGetDevice(&device));
    std::lock_guard<std::mutex> workspace_lock(workspace_mutex(device));
    uint32_t *host = nullptr;
    HBP_TRY(readback_get(device, &host));
    void *buf = nullptr;
    constexpr size_t kHistWords = kHistCopies * kHistStride;
    HBP_TRY(workspace_get(device, 1, sizeof(uint32_t) * (kHistWords + 1) + kStatsCopies * sizeof(RowStats), &buf));
    RowStats *row_stats = static_cast<RowStats *>(buf);
    uint32_t *hist = reinterpret_cast<uint32_t *>(row_stats + kStatsCopies);
    int32_t *d_a = reinterpret_cast<int32_t *>(hist + kHistWords);
    HBP_HIP(hipMemsetAsync(buf, 0, sizeof(uint32_t) * kHistWords + kStatsCopies * sizeof(RowStats), st));
    const int32_t S_rows = (int32_t)std::min<int64_t>(n_rows, 4096);
    k_sample_hist<<<blocks_for(S_rows, 4) + kStatsGroups, 256, 0, st>>>(csr_ptr, csr_col, n_rows, p.cols_per_block, S_rows, hist, row_stats);
    k_pick_shift<<<1, 64, 0, st>>>(hist, d_a, row_stats, csr_ptr, n_rows, host);
    HBP_HIP(hipGetLastError());
    HBP_HIP(hipStreamSynchronize(st));
    const int32_t a = (int32_t)host[16], first = (int32_t)host[17];
    *nnz_out = (int32_t)host[18];
    rows_out->rows = host[19];
    rows_out->skew = host[20] | (unsigned long long)host[21] << 32;
    if (first != 0 || *nnz_out < 0) return HBP_ERR_BAD_CSR_PTR;
    const int64_t nnz = *nnz_out;
    uint64_t segments = 0;
    for (int i = 0; i < 14; i++) segments += host[i];
    const bool long_segments = segments > 0 && 2 * (uint64_t)host[14] >= segments;
    if (p.rows_per_block == 0) p.rows_per_block = long_segments ? 512 : 2048;
    if (p.rounds_per_batch == 0) p.rounds_per_batch = long_segments ? 8 : 4;
    if (p.hash_shift < 0 && nnz > 0) p.hash_shift = a;
    return HBP_OK;
}

// Schedule weights, in units of one nonzero, where the caller left them open.  They are costs of
// the SpMV-part kernel on MI355X, not properties of a matrix: measured over workers with very
// different mixes, a group costs a wavefront 18 ns, a round 3 ns, a slot 0.6 ns and entering a
// block column costs the worker 19 us, next to 0.03 ns per nonzero while the wavefront waits for
// its loads anyway (groups of a few hundred nonzeros).  Groups of 512 nonzeros and more are
// streamed at the worker's share of the memory bandwidth instead (0.3 ns per nonzero): the same
// costs are a tenth as many nonzeros there.  And the device default of the workers: no more than
// the groups can keep busy, one group per wavefront.
static void choose_schedule(hbp_handle_s *h, const hbp_params_t &p)
{
    const bool streamed = h->G > 0 && h->nnz >= 512 * h->G;
    h->slot_weight = p.slot_weight >= 0 ? p.slot_weight : streamed ? 2 : 20;
    h->group_weight = p.group_weight >= 0 ? p.group_weight : streamed ? 60 : 600;
    h->round_weight = p.round_weight >= 0 ? p.round_weight : streamed ? 10 : 100;
    h->column_weight = p.column_weight >= 0 ? p.column_weight : streamed ? 60000 : 600000;
    if (p.num_workers == 0) {
        const int64_t waves = h->threads / kWave;
        const int64_t useful = std::max<int64_t>(1, (h->G + waves - 1) / waves);
        if (useful < h->P) h->P = (int32_t)useful;
    }
}

// Section 3.3: which groups are pre-assigned to which worker and which are left to competition.
static int launch_schedule(hbp_handle_s *h, hipStream_t st, const Words &words, int32_t n_words, uint32_t *host)  // and reads `words` back
{
    const int32_t NBC = (int32_t)h->NBC;
    if (NBC > kColumnsKept && !(h->flags & HBP_FLAG_PAPER_SCHEDULE)) k_col_ranks<<<1, 256, 0, st>>>(h->col_group_ptr, NBC, h->col_rank);
    if (h->flags & HBP_FLAG_PAPER_SCHEDULE) {
        const int64_t F = (h->B * (int64_t)h->fixed_q8) / (256 * (int64_t)h->P);
        h->first_ticket_block = F * h->P;
        k_paper_schedule<<<blocks_for((int64_t)h->P + 1, 256), 256, 0, st>>>(h->blk_group_ptr, h->blk_bn, F, (int32_t)h->B, NBC, h->P,
                                                                             h->fixed_start, h->fixed_col, h->comp_lo, h->comp_col);
        k_publish<<<1, 64, 0, st>>>(words, n_words, host, nullptr);
    } else {
        const Weights wt{h->group_ptr, h->group_slot, h->group_rounds, (int64_t)h->slot_weight, (int64_t)h->round_weight,
                         (int64_t)h->group_weight};
        // Where the share is the library's choice, groups that nobody would enter the range for are not left to competition: claims from
        // a counter that one worker alone adds to, and the search for another range at the end, gain nothing.  Products,
        // us, with / without: 27-point grid of 67^3 24.5 / 20.6, of 128^3 83.6 / 81.1, lognormal 150001 x 400009 36.1 / 31.7, 4M x 1M 281 /
        // 277, fp64 1.2M x 300K 129.4 / 124.0, R-MAT 2^22 258 / 255, 2^18 51.7 / 50.8.
        const int64_t least_open = h->share_chosen ? steal_weight(h->column_weight) : 0;
        k_schedule<<<blocks_for((int64_t)h->P + 1, 4), 256, 0, st>>>(h->col_group_ptr, wt, h->col_rank, (int64_t)h->column_weight, NBC,
                                                                     (int32_t)h->G, h->P, h->fixed_q8, h->fixed_start, h->fixed_col,
                                                                     h->comp_lo, h->comp_col, least_open, h->own_end, h->any_open, words, n_words, host);
    }
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

static int build_layout_locked(hbp_handle_s *h, const int32_t *csr_ptr, const int32_t *csr_col, const void *csr_val,
                               const hbp_params_t &p, hipStream_t st);

int build_layout(hbp_handle_s *h, const int32_t *csr_ptr, const int32_t *csr_col, const void *csr_val,
                 const hbp_params_t &p, hipStream_t st)
{
    std::lock_guard<std::mutex> workspace_lock(workspace_mutex(h->device));
    const int rc = build_layout_locked(h, csr_ptr, csr_col, csr_val, p, st);
    // A build that gives up may have kernels in flight that still use the shared workspace: they
    // have to finish before the lock is released and the next build takes the workspace over.
    if (rc != HBP_OK) (void)hipStreamSynchronize(st);
    return rc;
}

static int build_layout_locked(hbp_handle_s *h, const int32_t *csr_ptr, const int32_t *csr_col, const void *csr_val,
                               const hbp_params_t &p, hipStream_t st)
{
    const int64_t n_rows = h->n_rows, n_cols = h->n_cols;
    const int32_t R = h->R, C = h->C, W = h->W;
    const int64_t NBR = h->NBR, NBC = h->NBC, D = NBR * NBC;

    uint32_t *host = nullptr;
    HBP_TRY(readback_get(h->device, &host));
    // nnz and csr_ptr[0] are needed on the host before anything can be sized
    if (h->nnz < 0) {
        k_publish<<<1, 64, 0, st>>>(Words{{csr_ptr, csr_ptr + n_rows}}, 2, host, nullptr);
        HBP_HIP(hipGetLastError());
        HBP_HIP(hipStreamSynchronize(st));
        if (host[0] != 0 || (int32_t)host[1] < 0) return HBP_ERR_BAD_CSR_PTR;
        h->nnz = host[1];
    }
    const int64_t nnz = h->nnz;
    if (nnz >= (int64_t(1) << 31) - 64) return HBP_ERR_TOO_LARGE;

    // arrays whose size does not depend on the matrix content
    Arena own0(true, h->device);
    own0.reserve(&h->col_blk_ptr, NBC + 1);
    own0.reserve(&h->stripe_ptr, NBR + 1);
    own0.reserve(&h->ticket, (int64_t)h->P);
    own0.reserve(&h->comp_lo, (int64_t)h->P);
    own0.reserve(&h->comp_col, (int64_t)h->P);
    own0.reserve(&h->own_end, (int64_t)h->P);
    own0.reserve(&h->any_open, 1);
    own0.reserve(&h->col_group_ptr, NBC + 1);
    own0.reserve(&h->fixed_start, (int64_t)h->P + 1);
    own0.reserve(&h->fixed_col, (int64_t)h->P);
    own0.reserve(&h->unit_ptr, NBR + 1);
    own0.reserve(&h->col_rank, NBC + 1);
    const size_t own0_zeros = own0.total();
    if (nnz > 0) {  // 256 elements of padding: the SpMV part reads whole aligned 256-element chunks
        own0.reserve(&h->col_local, nnz + 256);
        own0.reserve_bytes(&h->data, (nnz + 256) * h->value_bytes);
    }
    HBP_TRY(own0.commit());
    h->arena[0] = own0.base(); h->arena_bytes[0] = own0.bytes();

    if (nnz == 0) {  // empty matrix: no blocks; the combine part alone writes y = 0
        HBP_HIP(hipMemsetAsync(own0.base(), 0, own0_zeros, st));
        h->B = h->S = h->G = 0;
        h->a = p.hash_shift >= 0 ? p.hash_shift : 0;
        Arena own1(true, h->device);
        own1.reserve(&h->blk_bm, 1); own1.reserve(&h->blk_bn, 1); own1.reserve(&h->slot_ptr, 1);
        own1.reserve(&h->blk_group_ptr, 1); own1.reserve(&h->stripe_blk, 1); own1.reserve(&h->group_ptr, 1);
        own1.reserve(&h->group_slot, 1); own1.reserve(&h->group_rounds, 1); own1.reserve(&h->group_blk, 1);
        own1.reserve(&h->row_local, 1); own1.reserve(&h->seg_len, 1); own1.reserve(&h->blk_shift, 1);
        own1.reserve(&h->col_local, 1); own1.reserve_bytes(&h->data, 8); own1.reserve_bytes(&h->partial, 8);
        own1.reserve(&h->unit_stripe, NBR + 1); own1.reserve(&h->unit_k, NBR + 2); own1.reserve(&h->multi_stripes, 1);
        HBP_TRY(own1.commit());
        h->arena[1] = own1.base(); h->arena_bytes[1] = own1.bytes();
        h->U = NBR; h->NM = 0;
        if (h->unit_slots == 0) h->unit_slots = 16384;
        k_iota_units<<<blocks_for(NBR + 1, 256), 256, 0, st>>>(h->unit_ptr, h->unit_stripe, h->unit_k, (int32_t)NBR);
        HBP_HIP(hipMemsetAsync(h->slot_ptr, 0, 4, st)); HBP_HIP(hipMemsetAsync(h->blk_group_ptr, 0, 4, st));
        HBP_HIP(hipMemsetAsync(h->group_ptr, 0, 4, st)); HBP_HIP(hipMemsetAsync(h->group_slot, 0, 4, st));
        HBP_HIP(hipMemsetAsync(h->group_rounds, 0, 4, st));
        choose_schedule(h, p);
        HBP_HIP(hipStreamSynchronize(st));
        return HBP_OK;
    }

    Arena tmp(false, h->device, 0);
    const int64_t n_tiles = (nnz + kTile - 1) / kTile;
    const int64_t scan_n = std::max<int64_t>(D, std::max<int64_t>(NBR, nnz / W + D)) + 1;
    Findings *found;
    uint32_t *dense_cnt, *slot_off, *group_off, *blk_id, *scan_tmp, *hist, *stripe_cnt, *stripe_slots, *stripe_groups, *dealt;
    int32_t *d_a;
    Tile *tiles;
    // The first pass leaves a list of the segments, one word each (block column, row, place in the tile), where these fit a word.  A tile's part of
    // it begins where the tile does, so it takes the room of as many words as there are nonzeros: that of the layout's values, which are written last.
    auto bits_for = [](int64_t values) { int32_t b = 0; while ((int64_t(1) << b) < values) b++; return b; };
    const int32_t row_bits = bits_for(R);
    const bool listed = kPlaceBits + row_bits + bits_for(NBC) <= 32;
    const int32_t reorder = (p.flags & HBP_FLAG_NO_REORDER) ? 0 : (p.flags & HBP_FLAG_KEY_LENGTH) ? 2 : (p.flags & HBP_FLAG_BLOCK_SHIFT) ? 3 : 1;
    uint32_t *const list = static_cast<uint32_t *>(h->data);
    // could steps 5 to 7 go by row blocks? (see below)  Which nonzeros start a segment is kept where the layout's columns come to be, ten bytes for
    // 64 nonzeros (only a matrix of a few hundred nonzeros has not the room).
    const bool short_rows = listed && n_tiles * kTileWords * 10 <= 2 * nnz && h->unroll <= 4 && reorder == 1 && W == 64 && R >= 64 && R <= kPanelRows && NBC <= kPanelColumns && NBR >= kPanelLeast &&
                            10 * 8 * NBC * panel_row_words(R) <= kPanelLds;  // (the bits at a = 0)
    const uint32_t room = (uint32_t)(kLdsPerCu / (h->value_bytes + (int32_t)sizeof(uint16_t)));  // nonzeros that a workgroup of k_panel_fill puts in place
    const SegmentWords words{reinterpret_cast<uint64_t *>(h->col_local), h->col_local + 4 * n_tiles * kTileWords};
    static_assert(sizeof(*words.starts) == 4 * sizeof(*h->col_local) && sizeof(*words.at) == sizeof(*h->col_local), "where the second array begins");
    // the arrays that start at zero side by side: one fill
    tmp.reserve(&dense_cnt, D);
    tmp.reserve(&hist, kHistCopies * kHistStride);
    tmp.reserve(&found, 1);
    tmp.reserve(&dealt, short_rows ? NBR + 1 : 1);  // nine entries for 64 row blocks
    static_assert(9 * ((kPanelLeast + 63) / 64) <= kPanelLeast, "as long as the arrays that are scanned beside it");
    tmp.reserve(&tiles, n_tiles);
    tmp.reserve(&slot_off, D + 1);
    tmp.reserve(&group_off, D + 1);
    tmp.reserve(&blk_id, D + 1);
    tmp.reserve(&stripe_cnt, NBR);
    tmp.reserve(&stripe_slots, NBR);
    tmp.reserve(&stripe_groups, NBR);
    tmp.reserve(&scan_tmp, 5 * (scan_n / kScanTile + 2));
    tmp.reserve(&d_a, 1);
    HBP_TRY(tmp.commit());
    const int64_t first_words = (int64_t)(own0_zeros / sizeof(uint32_t)), second_words = ((char *)tiles - (char *)dense_cnt) / (int64_t)sizeof(uint32_t);
    k_begin<<<(unsigned)std::min<int64_t>(1024, (first_words + second_words + 1023) / 1024), 256, 0, st>>>(
        static_cast<uint32_t *>(own0.base()), first_words, dense_cnt, second_words, d_a, p.hash_shift);

    // Section 3.2: shift a, sampled or given
    if (p.hash_shift < 0) {
        const int32_t S_rows = (int32_t)std::min<int64_t>(n_rows, 4096);
        k_sample_hist<<<blocks_for(S_rows, 4), 256, 0, st>>>(csr_ptr, csr_col, n_rows, C, S_rows, hist, nullptr);
        k_pick_shift<<<1, 64, 0, st>>>(hist, d_a, nullptr, csr_ptr, n_rows, nullptr);
    }

    // steps 1-3
    int32_t shift_c = -1, shift_r = -1;  // C = 2^shift_c (or one block column, 31), R = 2^shift_r, or -1
    for (int32_t b = 0; b < 31; b++) {
        if (C == (int32_t(1) << b)) shift_c = b;
        if (R == (int32_t(1) << b)) shift_r = b;
    }
    if (NBC == 1) shift_c = 31;
    const bool pow2 = shift_c >= 0 && shift_r >= 0;
    k_check_ptr<<<blocks_for(n_rows, 256), 256, 0, st>>>(csr_ptr, n_rows, nnz, tiles, found);
    const auto first_pass = short_rows ? (pow2 ? k_segments<Pass::kCountListAndWords, true> : k_segments<Pass::kCountListAndWords, false>)
                            : listed ? (pow2 ? k_segments<Pass::kCountAndList, true> : k_segments<Pass::kCountAndList, false>)
                                   : (pow2 ? k_segments<Pass::kCount, true> : k_segments<Pass::kCount, false>);
    first_pass<<<dim3((unsigned)n_tiles), kTileThreads, 0, st>>>(csr_ptr, csr_col, n_rows, nnz, n_cols, R, shift_r, C, shift_c, (int32_t)NBR,
                                                                 (int32_t)NBC, (p.flags & HBP_FLAG_VALIDATE) ? 1 : 0, tiles,
                                                                 dense_cnt, nullptr, list, row_bits, words, found);
    // step 4: scans over the block table
    HBP_TRY(exclusive_scans(Scans{{dense_cnt, dense_cnt, dense_cnt}, {slot_off, group_off, blk_id}, {kOpIdentity, kOpCeilDivW, kOpNonZero}}, 3,
                            D, (uint32_t)W, scan_tmp, st));
    k_stripe_count<<<blocks_for(NBR, 64), 1024, 0, st>>>(dense_cnt, (int32_t)NBR, (int32_t)NBC, csr_ptr, n_rows, R, (uint32_t)W, stripe_cnt, stripe_slots,
                                                      stripe_groups, short_rows ? room : 0u, dealt, found);
    HBP_HIP(hipGetLastError());

    // a host round trip: totals (and the error word)
    k_publish<<<1, 64, 0, st>>>(Words{{slot_off + D, group_off + D, blk_id + D, &found->err, d_a}}, 5, host, found);
    HBP_HIP(hipGetLastError());
    HBP_HIP(hipStreamSynchronize(st));
    const int32_t err = (int32_t)host[3], a = (int32_t)host[4];
    if (err & kErrPtr) return HBP_ERR_BAD_CSR_PTR;
    if (err & kErrCol) return HBP_ERR_BAD_CSR_COL;
    const int64_t S = host[0], G = host[1], B = host[2], longest_row = host[5];
    const bool long_segments = host[6] != 0;
    const int64_t most_slots = host[7], most_nonzeros = host[8];
    const int64_t n_row_blocks = host[9], most_shares = host[10], n_shares = host[11];  // (see deal_row_blocks; most_shares: of an XCD)
    h->S = S; h->G = G; h->B = B; h->a = a;

    Arena own1(true, h->device);
    own1.reserve(&h->blk_bm, B + 1); own1.reserve(&h->blk_bn, B + 1);
    own1.reserve(&h->slot_ptr, B + 1); own1.reserve(&h->blk_group_ptr, B + 1);
    own1.reserve(&h->stripe_blk, B + 1);
    own1.reserve(&h->group_ptr, G + 1); own1.reserve(&h->group_slot, G + 1); own1.reserve(&h->group_rounds, G + 1);
    own1.reserve(&h->group_blk, G + 1);
    h->flat_wpg = h->scheduled ? 0 : flat_wavefronts(nnz, S, NBC, h->value_bytes, h->rows);
    if (h->flat_wpg) own1.reserve(&h->long_groups, G + 1);
    own1.reserve(&h->row_local, S + 1); own1.reserve(&h->seg_len, S + 1);
    own1.reserve(&h->blk_shift, B + 1);
    if (p.flags & HBP_FLAG_KEEP_KEYS) own1.reserve(&h->slot_key, S + 1);
    own1.reserve_bytes(&h->partial, (S + 1) * h->value_bytes);
    if (h->unit_slots == 0) {
        // default: only row blocks with more than twice the average number of slots are cut
        const int64_t twice_mean = 2 * ((S + NBR - 1) / NBR);
        h->unit_slots = (int32_t)std::min<int64_t>(std::max<int64_t>(16384, twice_mean), INT32_MAX);
    }
    const int64_t max_units = NBR + S / h->unit_slots + 2;
    own1.reserve(&h->unit_stripe, max_units); own1.reserve(&h->unit_k, max_units + 1);
    own1.reserve(&h->multi_stripes, NBR);
    HBP_TRY(own1.commit());
    h->arena[1] = own1.base(); h->arena_bytes[1] = own1.bytes();
    // The order in which k_fill takes the blocks (see stripe_walk).  Row block by
    // row block pays where a row segment is a small part of the 128-byte lines it is gathered from
    // (fewer than 4 nonzeros on average) and the blocks are large enough to keep a workgroup busy
    // (256 slots on average); measured: k_fill 2.30 -> 1.10 ms on the 4M x 1M matrix with 2 nonzeros
    // per segment, 0.79 -> 0.37 ms on the 2^20 one with 1.6; with 13 nonzeros per segment (27-point
    // stencil) or 86 slots per block (R-MAT, whose dense row blocks then also wait for a few
    // workgroups) it is slower than the layout's own order with a wavefront per group.
    const bool by_row_block = NBR >= 64 && nnz < 4 * S && S >= 256 * B;
    // Steps 5 to 7 by row blocks as a whole under the same rule, where a row block fits the registers and the LDS of a workgroup (a, the row blocks' slots
    // and nonzeros, the bits).  Builds, us, block by block / by row blocks: templates of 400K rows 359 / 295; lognormal 1M x 1M 615 / 483, 4M x 1M
    // 1946 / 1253; fp64 1.2M x 300K 734 / 629, 2M x 500K 1251 / 905. (Rows may be of any length: see kPanelLongRow.)
    const size_t panel_words = (size_t)NBC * ((9u << a) - 1u) * panel_row_words(R);
    const size_t slots_table = sizeof(uint32_t) * (size_t)most_slots + (size_t)(most_slots / 64 + NBC) * panel_table_row((uint32_t)(a & 15)) + 8;
    const size_t slots_lds = std::max<size_t>(slots_table, panel_words * (sizeof(uint64_t) + sizeof(uint16_t)));
    const double panel_work = (double)S + (double)nnz * (double)(4 + h->value_bytes) / 8, panel_turns = (double)((n_row_blocks + kPanelTurn - 1) / kPanelTurn);
    const bool worth_panels = (long_segments && longest_row > kPanelLongRow) || panel_work * (double)NBR >= (kPanelWork * panel_turns - kPanelWorkOnce) * (double)n_row_blocks;
    const int64_t most_parts = (most_nonzeros + room - 1) / room, all_parts = 8 * ((NBR + 7) / 8) * most_parts;
    const bool by_panel = short_rows && by_row_block && worth_panels && !h->flat_wpg && a <= kPanelShift && most_slots <= kPanelSlots && most_nonzeros <= kPanelNonzeros &&
                          slots_lds <= (size_t)kPanelLds && all_parts <= kPanelMost;
    const int32_t parts = !by_row_block ? 0 : (int32_t)std::min<int64_t>(32, std::max<int64_t>(1, (B + NBR - 1) / NBR));
    // Rows much longer than the others: their groups are cut, or the longest is what the kernel waits for.  512 rounds are less than 60 us
    // for a wavefront; without such a row the two more launches are not worth their 10 us (27-point grid of 128^3 224 -> 234 us), nor
    // where the long rows lie in short segments over many block columns (20 rows of 4000 over 123 and 31 of them: 27.0 -> 36.5 and 55.2 -> 63.8);
    // where all rows are long nothing waits.  Fill kernels, us, whole / cut: R-MAT 2^20 (fp64) 322 / 267; 50 rows of 30000 beside rows of 40 506 /
    // 108; 250 of 600 beside rows of 70 211 / 214; one row in 40 held, of 400, 50 of 2500 93 / 51; one in 10, of 100, 50 of 700 61 / 57; one in
    // 100, of 600 44.5 / 51.5 (the average counts empty rows: groups so few that the device is not full gain by being cut as a rule).  Not
    // for k_fill, whose short segments have few such groups: the 4M x 1M lognormal matrix lost 60 us.
    const bool cut = parts == 0 && long_segments && longest_row > kLongRow && longest_row > 8 * (nnz / n_rows);
    Arena tmp2(false, h->device, 1);
    uint32_t *multi_idx, *stripe_turn, *blk_turn;
    tmp2.reserve(&multi_idx, NBR + 1); tmp2.reserve(&stripe_turn, NBR + 1); tmp2.reserve(&blk_turn, B);
    // k_fill_flat takes the groups row block by row block, too, where segments are short and there are several block columns.  Fill kernels, us, in the
    // layout's order / row block by row block: R-MAT 2^22 827 / 574, 2^20 (fp64) 223 / 200, 2^18 51 / 43; 13 nonzeros per segment (27-point
    // grid of 128^3) 226 / 220, 4.4 (5-point grid of 1500^2) 33.2 / 31.7, which the 4 us of k_group_turns are not worth.  Nor are they where the CSR arrays are little
    // more than the 4 MB of an XCD's L2, which then holds the lines anyway.  Builds, us, in the layout's order / row block by row block, by the MB of columns and values: 0.4
    // 107 / 110, 1.6 111 / 115, 2.4 112 / 116, 3.2 116 / 120, 4.8 123 / 123, 6.4 129 / 127, 9.6 (fp64) 147 / 142, 12 161 / 159, 28 200 / 169.
    const bool by_turns = parts == 0 && nnz < 4 * S && NBC > 1 && nnz * (4 + h->value_bytes) >= (6 << 20);
    uint2 *bucket = nullptr;
    uint32_t *group_nnz, *group_longest, *longest_all, *d_n_long;
    int32_t *slot_j;
    uint16_t *places = nullptr;
    // Where few of them would find nothing to do, all row blocks get a workgroup, and as many for their shares as the fullest needs: one that is told what to do by a list
    // begins with the wait for its entry (2000 row blocks of 15,400 nonzeros, fp64, 575 -> 584 us; 1500 of 41,000, two shares each, 730 -> 740).
    const bool listed_row_blocks = by_panel && 8 * (NBR - n_row_blocks) > NBR, listed_shares = by_panel && (listed_row_blocks || 8 * (all_parts - n_shares) > all_parts);
    int32_t *row_blocks = nullptr;
    uint32_t *shares = nullptr;
    if (by_panel) {
        tmp2.reserve(&places, n_tiles * kTile);
        if (listed_row_blocks) tmp2.reserve(&row_blocks, n_row_blocks);
        if (listed_shares) tmp2.reserve(&shares, 8 * most_shares);
    } else {
        tmp2.reserve(&bucket, S);
    }
    tmp2.reserve(&slot_j, S); tmp2.reserve(&group_nnz, G + 1); tmp2.reserve(&group_longest, G + 1); tmp2.reserve(&longest_all, 3);
    int2 *rest = nullptr;  // an entry per kFillRounds nonzeros of a group's longest row at most
    if (cut) tmp2.reserve(&rest, nnz / kFillRounds + 1);
    HBP_TRY(tmp2.commit());
    int32_t *const fill_order = by_turns ? reinterpret_cast<int32_t *>(bucket) : nullptr;  // (k_order_block has read the buckets by then; G <= S)
    d_n_long = longest_all + 1;
    uint32_t *const d_n_rest = longest_all + 2;

    k_compact_blocks<<<blocks_for(std::max<int64_t>(D, NBC) + 1, 256), 256, 0, st>>>(
        dense_cnt, slot_off, group_off, blk_id, D, (int32_t)NBR, (int32_t)NBC, h->blk_bm, h->blk_bn, h->slot_ptr,
        h->blk_group_ptr, h->col_blk_ptr, h->col_group_ptr, h->col_local + nnz, reinterpret_cast<uint32_t *>((char *)h->data + (size_t)nnz * h->value_bytes),
        256 * h->value_bytes / 4, h->group_slot + G, longest_all);
    HBP_TRY(exclusive_scans(Scans{{stripe_cnt, stripe_slots, stripe_slots, stripe_groups, dealt}, {(uint32_t *)h->stripe_ptr, (uint32_t *)h->unit_ptr, multi_idx, stripe_turn, dealt},
                                  {kOpIdentity, kOpUnits, kOpSplit, kOpIdentity, kOpIdentity}}, shares ? 5 : 4, NBR, (uint32_t)h->unit_slots, scan_tmp, st));
    k_stripe_fill<<<blocks_for(NBR, 64), 1024, 0, st>>>(dense_cnt, blk_id, h->stripe_ptr, stripe_slots, h->unit_ptr, multi_idx, stripe_turn, (uint32_t)W,
                                                       (int32_t)NBR, (int32_t)NBC, (int32_t)B, h->stripe_blk, blk_turn, h->unit_stripe, h->unit_k, h->multi_stripes,
                                                       csr_ptr, n_rows, R, room, dealt, row_blocks, shares);
    const dim3 stripe_grid((unsigned)(8 * ((NBR + 7) / 8) * std::max(parts, 1)));
    // steps 5-6 (slot_off doubles as the per-block cursor from here on, but for row blocks as a whole)
    if (by_panel) {
        HBP_HIP(hipFuncSetAttribute((const void *)k_panel_slots, hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
        // rounds behind the table's, ten bytes each, as many as there is room for
        const uint32_t most_tails = (uint32_t)std::min<size_t>(kPanelTails, ((size_t)kPanelLds - slots_table) / 10) & ~3u;
        k_panel_slots<<<dim3((unsigned)(row_blocks ? n_row_blocks : NBR)), kPanelThreads, std::max(slots_lds, slots_table + 10 * (size_t)most_tails), st>>>(
            row_blocks, csr_ptr, n_rows, R, (int32_t)NBR, (int32_t)NBC, tiles, words.starts, words.at, list, row_bits, slot_off, group_off, blk_id, (uint32_t)a,
            (uint32_t)long_rounds_of(h->heavy_rounds, true), longest_all, h->row_local, h->seg_len, h->slot_key, group_nnz, group_longest,
            h->group_slot, h->group_blk, h->blk_shift, places, slot_j, most_tails);
    } else {
        if (listed) {
            // a wavefront per tile where it holds few segments, up to eight where it holds many
            int32_t wavefronts = 1;
            while (wavefronts < kTileThreads / 64 && S > 256 * wavefronts * n_tiles) wavefronts *= 2;
            const auto place = wavefronts == kTileThreads / 64 ? k_place<true> : k_place<false>;
            place<<<blocks_for(n_tiles * wavefronts, kTileThreads / 64), kTileThreads, 0, st>>>(
                csr_ptr, n_rows, nnz, R, shift_r, (int32_t)NBR, (int32_t)NBC, (int32_t)n_tiles, wavefronts, tiles, list, row_bits, slot_off, bucket);
        } else {
            const auto second_pass = pow2 ? k_segments<Pass::kEmit, true> : k_segments<Pass::kEmit, false>;
            second_pass<<<dim3((unsigned)n_tiles), kTileThreads, 0, st>>>(csr_ptr, csr_col, n_rows, nnz, n_cols, R, shift_r, C, shift_c, (int32_t)NBR,
                                                                          (int32_t)NBC, 0, tiles, slot_off, bucket, nullptr, row_bits, SegmentWords{nullptr, nullptr}, found);
        }
        const size_t order_cap = ((size_t)R + 63) & ~(size_t)63;
        size_t small_n2 = 1;  // the bitonic network of a small block: 8-byte words, the next power of two above min(R, 256) slots
        while (small_n2 < (size_t)std::min(R, 256)) small_n2 <<= 1;
        const size_t order_lds = std::max(sizeof(uint32_t) * (2 * order_cap + 16 * (order_cap / 64)),  // two entry arrays, 16 counters per tile
                                          sizeof(uint64_t) * small_n2);
        HBP_HIP(hipFuncSetAttribute((const void *)k_order_block, hipFuncAttributeMaxDynamicSharedMemorySize, (int)order_lds));
        k_order_block<<<dim3((unsigned)B), 256, order_lds, st>>>(bucket, h->slot_ptr, h->blk_group_ptr, W,
                                                                h->row_local, h->seg_len, slot_j, group_nnz, group_longest, h->group_slot,
                                                                h->group_blk, (uint32_t)long_rounds_of(h->heavy_rounds, true), longest_all,
                                                                d_n_long, h->long_groups, h->flat_wpg, reorder, (uint32_t)R, d_a, h->blk_shift, h->slot_key);
    }
    HBP_TRY(exclusive_scans(Scans{{group_nnz, group_longest}, {(uint32_t *)h->group_ptr, (uint32_t *)h->group_rounds}, {kOpIdentity, kOpIdentity}}, 2,
                            G, 1, scan_tmp, st));
    // step 7
    auto fill = [&](const auto *val, auto *data) {
        using T = std::remove_reference_t<decltype(*data)>;
        if (by_panel) {
            constexpr uint32_t kRoom = kLdsPerCu / (sizeof(T) + sizeof(uint16_t));
            static_assert((kPanelNonzeros + kRoom - 1) / kRoom <= 1u << kShareBits, "the shares of a row block");
            (void)hipFuncSetAttribute((const void *)k_panel_fill<T>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
            k_panel_fill<T><<<dim3((unsigned)(shares ? 8 * most_shares : all_parts)), kPanelThreads, room * (sizeof(T) + sizeof(uint16_t)), st>>>(
                shares, found, csr_ptr, n_rows, R, (int32_t)NBR, (int32_t)NBC, C, (uint32_t)most_parts, room, places, csr_col, val, group_off, h->group_ptr, h->col_local, data);
            return;
        }
        if (parts > 0) {
            k_fill<T><<<stripe_grid, 256, 0, st>>>(h->stripe_ptr, h->stripe_blk, (int32_t)NBR, (int32_t)B, parts, csr_col, val, h->group_ptr,
                                                   h->group_slot, h->blk_group_ptr, h->blk_bn, h->seg_len, slot_j, C, nnz, h->col_local, data);
            return;
        }
        if (fill_order) k_group_turns<<<blocks_for(G, 256), 256, 0, st>>>(h->group_blk, h->blk_group_ptr, blk_turn, (int32_t)G, fill_order);
        const auto flat = cut ? k_fill_flat<true, T> : k_fill_flat<false, T>;
        flat<<<fill_order ? 8 * kFillChunk * blocks_for(G, 32 * kFillChunk) : blocks_for(G, 4), 256, 0, st>>>(fill_order, csr_col, val, h->group_ptr, h->group_slot, h->group_blk, h->blk_bn, h->seg_len, slot_j, (int32_t)G, C,
                                               nnz, h->col_local, data);
        if (!cut) return;
        k_list_rest<<<blocks_for(G, 1024), 256, 0, st>>>(group_longest, (int32_t)G, rest, d_n_rest);
        k_fill_rest<T><<<dim3(2048), 256, 0, st>>>(rest, d_n_rest, csr_col, val, h->group_ptr, h->group_slot, h->group_blk, h->blk_bn, h->seg_len,
                                                   slot_j, C, nnz, h->col_local, data);
    };
    if (h->value_bytes == 8) fill(static_cast<const double *>(csr_val), static_cast<double *>(h->data));
    else fill(static_cast<const float *>(csr_val), static_cast<float *>(h->data));
    HBP_HIP(hipGetLastError());
    choose_schedule(h, p);
    HBP_TRY(launch_schedule(h, st, Words{{h->unit_ptr + NBR, multi_idx + NBR, longest_all, d_n_long}}, 4, host));
    HBP_HIP(hipGetLastError());
    HBP_HIP(hipStreamSynchronize(st));
    h->U = host[0]; h->NM = host[1];
    h->longest_segment = (int32_t)host[2];  // 0 unless it makes a group long
    h->n_long = (int32_t)host[3];
    return HBP_OK;
}

// Memory that may still be in use goes back to the driver, which does not hand it out before its users are done.
void release_block(int device, void *base, size_t bytes, bool idle)
{
    if (!base) return;
    if (!idle || device < 0 || device >= kWorkspaceDevices || bytes > kCacheBytes) {
        (void)hipFree(base);
        return;
    }
    std::lock_guard<std::mutex> lock(g_cache_mutex[device]);
    BlockCache &cache = g_cache[device];
    while (cache.count == kCacheBlocks || cache.bytes + bytes > kCacheBytes) (void)hipFree(cache.take(0).base);
    cache.at[cache.count++] = {base, bytes};
    cache.bytes += bytes;
}

int release_workspace()
{
    int rc = HBP_OK;
    for (int device = 0; device < kWorkspaceDevices; device++) {
        std::lock_guard<std::mutex> workspace_lock(workspace_mutex(device));
        for (auto &w : g_workspace[device]) {
            if (w.base && hipFree(w.base) != hipSuccess) rc = HBP_ERR_HIP;
            w.base = nullptr;
            w.bytes = 0;
        }
        if (g_readback[device] && hipHostFree(g_readback[device]) != hipSuccess) rc = HBP_ERR_HIP;
        g_readback[device] = nullptr;
        if (drop_cached_blocks(device) != HBP_OK) rc = HBP_ERR_HIP;
    }
    return rc;
}

int hash_keys(const uint32_t *n, int64_t count, int32_t a, int32_t R, uint32_t *keys, hipStream_t st)
{
    if (count > 0) k_hash_keys<<<blocks_for(count, 256), 256, 0, st>>>(n, count, (uint32_t)a, (uint32_t)R, keys);
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

int derive_add_sign(const hbp_handle_s *h, int32_t *d_out, hipStream_t st)
{
    if (h->G > 0)
        k_add_sign<<<blocks_for(h->G, 4), 256, 0, st>>>(h->group_ptr, h->group_slot, h->seg_len, (int32_t)h->G, d_out);
    HBP_HIP(hipGetLastError());
    return HBP_OK;
}

}  // namespace hbp
