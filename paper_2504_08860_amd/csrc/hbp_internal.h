// Internal declarations shared by the translation units of libhbp (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbp.h"

namespace hbp {

constexpr int kWave = 64;            // gfx950 wavefront width
constexpr int kMaxR = 8192;          // rows per block: one block's slots are ordered in 64 KB of LDS
constexpr int kMaxC = 32768;         // columns per block: fp32 vector segment of 128 KB in LDS
constexpr int kMaxC64 = 16384;       // the same 128 KB with fp64 values
constexpr int kMaxR64 = 4096;        // fp64: the combine part keeps four copies of a y slice in LDS
// LDS of a k_spmv_part workgroup next to its slice of x, at most (the kernel checks its arrays against it)
constexpr int kLdsPerCu = 160 * 1024;
constexpr int part_static_lds(int threads) { return 28 * threads + threads / 8 + 3648; }
static_assert(kMaxC * 4 + part_static_lds(1024) <= kLdsPerCu && kMaxC64 * 8 == kMaxC * 4, "the largest slice has to fit beside the kernel's own arrays");
constexpr int64_t kMaxDense = int64_t(1) << 27;  // NBR * NBC table entries
// Rows longer than long_rounds_of (and up to heavy_group_rounds) make their group a "long" one.  Where a worker has
// few groups they are walked first, so that the others fill up the wavefronts that are done with theirs; the worker's
// start then waits for its slice of x (2 us), and where it has many groups the long ones are lost among them.
// Measured, us per product, after the others from 256 rounds on / first from 32 rounds on (groups per worker): lognormal rows
// 400K x 100K (72) 70 / 46, fp64 (120) 66 / 57, 1.2M x 300K (473) 103 / 92, 4M x 1M (3037) 285 / 297; R-MAT 2^20 (241)
// 120 / 114, fp64 (340) 119.6 / 121.5, 2^22 (1785) 299 / 309.  (For heavy_group_rounds given as 64, 1M x 1M lognormal rows: first from 1 round on
// 118, from 8 on, an eighth of it, 92.)
inline bool walk_long_first(int64_t G, int64_t P) { return G < 1024 * P; }
inline int32_t long_rounds_of(int32_t heavy_rounds, bool long_first)
{
    const int32_t eighth = heavy_rounds / 8, few = eighth < 32 ? eighth : 32;
    const int32_t rounds = !long_first ? eighth : heavy_rounds / 64 > few ? heavy_rounds / 64 : few;
    return rounds > 0 ? rounds : 1;
}

// Where the long groups go first, one of more nonzeros than this is heavy, however they are spread over its rows, if it outweighs the
// other groups of its range: one wavefront takes 2.5 us for every 1024 of them while the rest of its worker runs dry.  Shared by several
// wavefronts it costs the worker about 5 us, which fewer nonzeros are not worth.  Products, us, by rows alone / from 32768
// nonzeros on / 16384 / 8192 / 4096: R-MAT 2^20 119 / 118 / 92 / 90 / 94, fp64 117 / 117 / 115 / 109 / 105.  (Where they go last, with 1024 groups
// per worker and more, it gains nothing: 2^22 253 / 253 / 253 / 278 / 320.)
inline int32_t heavy_elements_of(bool heavy_chosen) { return heavy_chosen ? 8192 : 0x7fffffff; }  // (a given heavy_group_rounds alone counts)

// Does it?  Where the other wavefronts have as much to do, nobody waits for the one that walks it, and sharing it costs more.
// Fewer than half as many groups as wavefronts can have more than twice a wavefront's share of the range's nonzeros.
// Products, us, by rows alone / shared without this / from one wavefront's share on / two / four: rows of 150 and of 20 nonzeros in equal
// parts, 300K 38.5 / 57.9 / 58.1 / 43.0 / 38.6, 1M 98 / 126 / 98 / 98 / 98, fp64 160 / 178 / 161 / 161 / 162; R-MAT, five of each, 2^19 81 / 62 / 62 / 64 /
// 75, 2^20 116 / 91 / 91 / 94 / 115, fp64 115 / 112 / 112 / 104 / 115, 2^21 134 / 139 / 133 / 133 / 134.
constexpr int kMaxOutweighing = 8;
__host__ __device__ inline bool outweighs(uint32_t elements, uint32_t range_elements, int wavefronts)
{
    return (uint64_t)elements * (uint32_t)wavefronts > 2 * (uint64_t)range_elements;
}

// Long is only what is longer than the others: a listed group is walked without the next one's loads on their way, which
// costs more than the order brings where all groups are of about one length (`mean` rounds on average).  Up to three
// times the mean, or 96 rounds, or a quarter more than the mean, is not; where the caller gives heavy_group_rounds, that alone
// counts.  Measured, SpMV part in us, from 32 rounds on / with this line / never below 256 rounds: bands of 48 nonzeros per row 68 / 60 /
// 64, of 200 69 / 61 / 61 (fp64 93 / 79 / 82); rows of 60 random nonzeros 48 / 42 / 42, of 1 to 79 44 / 36 / 36, of 1 to 299 64 /
// 61 / 85; lognormal rows of 111 on average 154 / 152 / 180 (fp64, 55 per column block: 168 / 170 / 163).
inline int32_t long_rounds_beside(int64_t mean)
{
    const int64_t rounds = mean + mean / 4 > 96 ? mean + mean / 4 : 3 * mean < 96 ? 3 * mean : 96;
    return rounds < (1 << 16) ? (int32_t)rounds : 1 << 16;
}

// What choose_block_parameters finds out about the rows of a matrix that flat_wavefronts may ask for (zeros: not looked at).
struct RowStats {
    uint32_t rows;            // with a nonzero
    unsigned long long skew;  // sum over the rows of length * min(length, 64 * mean length)
};
constexpr int64_t kFlatLeast = 1000000, kFlatMost = 12000000;  // nonzeros: flat whatever the rows are like, never flat
__host__ __device__ inline bool rows_matter(int64_t nnz, int64_t n_rows) { return nnz > kFlatLeast && nnz <= kFlatMost && n_rows <= 4 * nnz; }

// Matrices small enough for k_spmv_flat (one group after the other across the grid, x read from L2) in
// place of k_spmv_part (persistent workers with x staged in LDS): the wavefronts it gives a group, or 0.
// The workers spend 5-7 us before the first product and have at most a pack or two per wavefront here;
// against that x comes out of L2 at some 100 G random elements/s for the whole chip.  Not held up by that are rows that each
// stay in a block column or two of several (a grid operator's, which read neighbouring elements), and less so rows of
// very uneven length (a graph's, whose columns are as uneven: an average nonzero lies in a row of 8 times the average
// length and more, rows of over 64 times the average counted as that; lognormal rows 4, R-MAT 12 to 14), which the workers in turn
// wait for.  The rest is the sooner too large the more block columns and bytes of x there are; over four block columns and more
// the workers cope better with uneven rows than with even ones.
// Measured, us per product, workers / flat, fp32 (fp64):
//   5-point grid     1M 27 / 13 (27 / 15)    4M 33 / 22 (38 / 27)    12M 59 / 50 (80 / 69)    20M 77 / 70 (110 / 116)
//   27-point grid    2M 20 / 13 (23 / 16)    2.9M 21 / 14 (25 / 20)  3.9M 22 / 20 (27 / 24)   5.6M 23 / 24 (29 / 31)
//   R-MAT            1M 67 / 43 (62 / 43)    2M 62 / 55 (78 / 46)    3.9M 67 / 57 (88 / 62)   8M 80 / 79 (92 / 96)
//   random columns, one block column: rows of 20    3M 19 / 17 (21 / 19)   4M 20 / 22 (22 / 25); lognormal rows 3M 42 / 28, 4M -
//     two or three: lognormal rows 2M 38 / 30 (36 / 32)   2.5M (36 / 40)   4M 40 / 48 (44 / 52); rows of 32 2M 20 / 19   3M 23 / 32
//     more: rows of 4 1M 23 / 16 (27 / 22)   2M 28 / 28 (33 / 36)   3M 34 / 39 (41 / 50)
//           lognormal rows 1M 34 / 35 (34 / 36)   1.5M 32 / 37 (39 / 38)   2M 33 / 40 (39 / 40)
//           10 in every third row 1M 22 / 14 (24 / 20)   2M 24 / 21 (32 / 33)   3M 27 / 28 (35 / 43)   10M 45 / 80
// Segments of 8 nonzeros and more on average get four wavefronts per group, shorter ones would leave three idle:
// 27-point grid 0.75M 17.9 (one) / 7.3 (four); 5-point grid 5M 25 / 51.
inline int flat_wavefronts(int64_t nnz, int64_t S, int64_t NBC, int32_t value_bytes, RowStats rows)
{
    const bool short_segments = nnz < 8 * S;
    const bool local = 2 * S <= (NBC < 4 ? NBC : 4) * (int64_t)rows.rows && nnz >= 2 * S;
    const double uneven = (double)rows.skew * (double)rows.rows / ((double)nnz * (double)nnz);
    const int64_t most = local && short_segments ? kFlatMost
                         : local || uneven >= 8  ? 4000000
                         : NBC == 1              ? 3000000
                         : NBC <= 3              ? 2250000
                         : value_bytes == 4 && uneven < 2 ? 2000000
                                                          : kFlatLeast;
    return nnz > most ? 0 : short_segments ? 1 : 4;
}
// whether k_spmv_flat with `wpg` wavefronts per group gives a group a workgroup of its own: one wavefront
// takes 8 rounds, up to 512 nonzeros, per memory round trip
__host__ __device__ inline bool is_long_group(int32_t nnz, int32_t longest, int wpg) { return nnz > 2048 || (wpg > 1 && longest > 64); }

// The build cuts groups with long segments where it can.  Whether a tile of 64 words of 64 nonzeros (`count` of them there) shows that a
// segment has more than 192 nonzeros: three words in a row without a start of one (bit w: one starts in word w).  More than 512
// nonzeros show in one of their tiles, wherever they begin: at least 256 in a row behind the start lie in one.
__host__ __device__ inline bool shows_long_segment(uint64_t words_with_start, int32_t count)
{
    const int32_t full = count >> 6;
    const uint64_t without = ~words_with_start & (full < 64 ? (1ull << full) - 1ull : ~0ull);
    return (without & without >> 1 & without >> 2) != 0;
}

// Combine part, blocks of more than 1024 rows: wavefronts of a workgroup, each with its own copy of the unit's slice of y in LDS.
constexpr int kCombineLds = 4 * kMaxR * (int)sizeof(float);  // all copies, at most
constexpr int kCombineStaticLds = 1024;                       // the kernel's own array (checked there)
constexpr int kLdsStep = 1280, kWavesPerCu = 32;              // LDS is given out in these units; wavefronts on a compute unit (the kernel keeps to 64 registers)
inline int64_t combine_units_by_lds(int64_t copy_bytes, int wavefronts)  // on a compute unit at a time
{
    return kLdsPerCu / ((wavefronts * copy_bytes + kCombineStaticLds + kLdsStep - 1) / kLdsStep * kLdsStep);
}
// Few units: more wavefronts for each, as many as the copies' LDS lets one workgroup (up to a unit per compute unit, 256 units) or two of
// them (up to 512) have on a CU.  Whole products, us, four wavefronts per unit / now: 3.6M nonzeros in 74 units 51.6 / 47.0, 12.8M in 196
// units 56.3 / 50.2; fp64 3.7M in 74 units 50.8 / 47.3.  (One workgroup of eight per CU for 489 fp64 units: combine part 12.1 / 17.7,
// hence the second bound.)
// Three wavefronts where four would leave some units for a second round and three do not (a unit's time is that of its wavefronts'
// loads, so a nearly empty second round doubles the kernel).  Whole products, us, four / three, R = 2048: fp64 (513 to 768 units) lognormal
// rows 1.2M 137.5 / 128.9, 1.5M 186.7 / 172.5, 1.1M 108.3 / 102.5, R-MAT 2^20 136.9 / 132.5; fp32 (1025 to 1536 units) 2.5M 175.9 /
// 168.6, 2.2M 132.4 / 129.7, R-MAT 2^21 166.1 / 157.5.  Whether they do counts the wavefronts a compute unit holds, too; where these alone keep
// four from one round, three wait for as long.  Combine part, us, four / three, fp32: R = 1025 (LDS for 9 and 11 units, wavefronts for 8 and
// 10) 2100 units 26.8 / 27.1, 2250 27.8 / 28.2, 2600 29.7 / 33.3, 2900 32.3 / 34.2; R = 1200 (LDS for 8 and 9) 2320 units 30.9 / 34.3.
inline int combine_wavefronts(int64_t cus, int64_t units, int64_t R, int32_t value_bytes)
{
    const int64_t copy = R * value_bytes;
    if (units <= cus && 16 * copy <= kCombineLds) return 16;
    if ((units <= cus && 8 * copy <= kCombineLds) || (units <= 2 * cus && 16 * copy <= kCombineLds)) return 8;
    const int64_t by_lds = combine_units_by_lds(copy, 3), by_waves = kWavesPerCu / 3;
    return units > cus * combine_units_by_lds(copy, 4) && units <= cus * (by_lds < by_waves ? by_lds : by_waves) ? 3 : 4;
}

// Short batches of fp32 values are walked in steps where a worker has many groups and the average one fits a wavefront's place in LDS:
// a group that does not is walked with nothing of its own in flight.  Products, us, packs / steps: 20M rows along the
// diagonal of 1 nonzero and, one in 11, 20 (175 elements a group) 224 / 209, of 1 and 10, three to one (208) 239 / 233, of 1 and
// 4 (160) 196 / 192, two to one (128) 186 / 177, of 1 to 5 (192) 226 / 230, of 2 (128) 154 / 159, of 3 (192) 169 / 176, of 4 (256) 191 / 199,
// of 5 (320) 237 / 252; 5-point grid of 4300^2 (253) 276 / 274; 2^20 rows from templates (98) 98.7 / 96.5; lognormal 4M x 1M (126) 275 / 260,
// x 400K (203) 249 / 244, 5M x 200K (318) 287 / 289; R-MAT 2^22 (143) 254 / 252.
// (With few groups, 71 a worker on lognormal 150001 x 400009, the packs' four groups at once start sooner: 36.0 against 38.3.  fp64 windows
// hold half as many elements, so half of the groups would be walked on their own: lognormal 1.2M x 300K 128 against 139.)
constexpr int kStepElements = 224;
inline bool walk_in_steps(int32_t rounds_per_batch, bool long_first, int64_t nnz, int64_t G)
{
    return rounds_per_batch <= 4 && !long_first && nnz <= kStepElements * G;
}

// Weight that another worker's range must have left for a worker to enter it: what entering a block column costs (the fetch of
// its slice of x), twice, counting the restart of the pipeline.
__host__ __device__ inline int32_t steal_weight(int32_t column_weight) { return 2 * column_weight; }

// Device-side view of the layout, passed by value to kernels.
struct Layout {
    int32_t R, C, W;
    int32_t B, S, G;
    int32_t NBR, NBC, P;
    int32_t competitive;  // 0 when every group is fixed (nothing to compete for)
    int32_t ticket_b0;    // the paper's schedule: first block behind the single ticket counter; -1: not in use
    int64_t n_rows, n_cols;
    const int32_t *blk_bm, *blk_bn, *slot_ptr, *blk_group_ptr, *col_blk_ptr, *stripe_ptr, *stripe_blk;
    const int32_t *group_ptr, *group_slot, *group_rounds, *group_blk, *long_groups;
    const int32_t *col_group_ptr, *comp_lo, *comp_col, *fixed_start, *fixed_col;  // schedule (Section 3.3)
    const int32_t *own_end, *any_open;
    const int32_t *unit_ptr, *unit_stripe, *unit_k, *multi_stripes;               // combine work units
    int32_t NM;                                                        // row blocks with several units
    int32_t claim;  // competitive groups a worker claims from a range's counter at a time
    int32_t SW, RW, GW;  // schedule weights of a slot, a round, a group (a nonzero weighs 1)
    int32_t steal_min;   // weight a range's competitive part must have left for another worker to enter it
    int32_t heavy_rounds;  // a group with a longer row is walked by several wavefronts of a worker together
    int32_t heavy_elements;  // and so is, where lists_first, a long group of more nonzeros that outweighs the others of its range
    int32_t long_rounds;   // a group with a longer row (up to heavy_rounds) gets a wavefront of its own
    int32_t lists_first;   // and is walked, like the heavy ones, before the other groups of its range
    const uint16_t *row_local, *seg_len, *col_local;
    const void *data;  // float or double, by the handle's value type
};

}  // namespace hbp

struct hbp_handle_s {
    int device;
    int64_t n_rows, n_cols, nnz;
    int32_t R, C, W, a;
    int64_t NBR, NBC, B, S, G;
    int32_t P, fixed_q8, slot_weight, claim_chunk, threads;
    int32_t cus;         // compute units of the device
    int32_t unroll;      // rounds taken per batch by the SpMV-part kernel
    double build_ms;
    // device arrays (owned): views into two allocations, arena[0] sized before the matrix is
    // looked at, arena[1] after the segment, group and block counts are known
    void *arena[2];
    size_t arena_bytes[2];
    int32_t *blk_bm, *blk_bn, *slot_ptr, *blk_group_ptr, *col_blk_ptr, *stripe_ptr, *stripe_blk;
    int32_t *group_ptr, *group_slot;
    int32_t *col_group_ptr, *comp_lo, *comp_col, *fixed_start, *fixed_col;
    int32_t *own_end;                    // [P] end of the groups that are a worker's own: comp_lo, or the range's end where nobody would enter it
    int32_t *any_open;                   // is there a range that somebody would enter?
    int32_t *group_rounds;               // [G+1] prefix sums of the groups' longest rows
    int32_t *group_blk;                  // [G] block of each group
    int32_t *long_groups;                // [n_long] groups that k_spmv_flat gives a workgroup of their own
    int32_t n_long;
    int32_t flat_wpg;                    // wavefronts per group of k_spmv_flat; 0: k_spmv_part runs
    bool scheduled;                      // the caller chose something about the workers or their schedule
    hbp::RowStats rows;
    int32_t *unit_ptr, *unit_stripe, *unit_k, *multi_stripes;
    int64_t U, NM;       // combine work units, row blocks cut into several units
    int32_t unit_slots;  // target slots per combine unit
    bool share_chosen;     // fixed_q8, by the library
    int32_t heavy_rounds;  // groups with a longer row are shared by a worker's wavefronts
    bool heavy_chosen;     // by the library
    int32_t group_weight;  // schedule weight of a group as such
    int32_t longest_segment;  // longest row segment of the matrix (0 unless it makes a group long)
    int32_t round_weight;  // schedule weight of a group on top of its nonzeros and slots
    int32_t column_weight;  // schedule weight of entering a block column
    int32_t *col_rank;     // [NBC+1] non-empty block columns before each column
    uint16_t *row_local, *seg_len, *col_local;
    int32_t value_bytes; // 4: fp32 values (data, partial, x, y), 8: fp64
    void *data;
    void *partial;       // [S] per-slot partial sums of the SpMV part
    uint32_t *ticket;    // [P] competitive groups of every worker's range claimed so far, zero between calls
    uint32_t *slot_key;  // [S] key each slot was placed by, or null (HBP_FLAG_KEEP_KEYS)
    int32_t *blk_shift;  // [B] shift a of each block's keys
    int64_t first_ticket_block;  // the paper's schedule (HBP_FLAG_PAPER_SCHEDULE): P F; -1 otherwise
    uint32_t flags;      // HBP_FLAG_* the handle was built with
};

namespace hbp {

// error plumbing -----------------------------------------------------------------------
void set_last_hip_error(hipError_t e);
#define HBP_HIP(expr)                                  \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) {                        \
            hbp::set_last_hip_error(e_);               \
            return e_ == hipErrorOutOfMemory ? HBP_ERR_OUT_OF_MEMORY : HBP_ERR_HIP; \
        }                                              \
    } while (0)

// build (hbp_build.hip)
int build_layout(hbp_handle_s *h, const int32_t *csr_ptr, const int32_t *csr_col, const void *csr_val,
                 const hbp_params_t &p, hipStream_t stream);
// *nnz, *rows: unchanged where the matrix was not looked at
int choose_block_parameters(const int32_t *csr_ptr, const int32_t *csr_col, int64_t n_rows, int64_t n_cols, int32_t value_bytes,
                            hbp_params_t &p, int64_t *nnz, RowStats *rows, hipStream_t stream);
int derive_add_sign(const hbp_handle_s *h, int32_t *d_out, hipStream_t stream);
int hash_keys(const uint32_t *n, int64_t count, int32_t a, int32_t R, uint32_t *keys, hipStream_t stream);
int release_workspace();
int device_alloc(int device, size_t bytes, void **out);  // hipMalloc; where memory is short, after giving back what freed handles left
// takes back a handle's allocation; idle: nothing on the device uses it any more
void release_block(int device, void *base, size_t bytes, bool idle);

// spmv (hbp_spmv.hip)
Layout hbp_view(const hbp_handle_s *h);
int default_workers(int device, int32_t C, int32_t value_bytes, int32_t threads_wanted, int32_t *threads_out, int32_t *workers_out,
                    int32_t *cus_out);
// x, y (and val): arrays of the handle's value type (value_bytes for the CSR baselines)
// where one SpMV keeps its per-slot partial sums (S values of the handle's type) and its claim counters (P)
struct SpmvScratch {
    void *partial;
    uint32_t *ticket;
};
int launch_spmv_part(const hbp_handle_s *h, const void *x, void *y, hipStream_t stream, SpmvScratch scratch);
int launch_combine(const hbp_handle_s *h, void *y, hipStream_t stream, SpmvScratch scratch);  // nothing where k_spmv_flat has written y
int launch_csr(int kind, int value_bytes, const int32_t *ptr, const int32_t *col, const void *val, const void *x, void *y,
               int64_t n_rows, hipStream_t stream);

}  // namespace hbp
