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
// 120 / 114, fp64 (340) 119.6 / 121.5, 2^22 (1785) 299 / 309.
inline bool walk_long_first(int64_t G, int64_t P) { return G < 1024 * P; }
inline int32_t long_rounds_of(int32_t heavy_rounds, bool long_first)
{
    const int32_t rounds = heavy_rounds / (long_first ? 64 : 8);
    return rounds > 0 ? rounds : 1;
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

// Matrices small enough for k_spmv_flat (one group after the other across the grid, x read from L2) in
// place of k_spmv_part (persistent workers with x staged in LDS): the wavefronts it gives a group, or 0.
// The workers spend 5-7 us before the first product and have at most a pack or two per wavefront here;
// against that x comes out of L2 at some 100 G random elements/s for the whole chip (rows that each stay in a block
// column or two of several, as a grid operator's, read neighbouring elements and are not held up by that).
// Measured, us per product, workers / flat: 20K nonzeros in one block column 20.5 / 3.8; random columns 1.2M
// 43 / 19, 2.4M (fp64) 45 / 47, 4.2M 26.6 / 32, 9.7M 70 / 91; R-MAT 3.9M 89 / 59; 5-point grid 5M 37 / 25, 11M
// 56 / 46; 27-point grid 2.4M 22 / 13.6, 7.9M 27.8 / 30.
// Segments of 8 nonzeros and more on average get four wavefronts per group, shorter ones would leave three idle:
// 27-point grid 0.75M 17.9 (one) / 7.3 (four); 5-point grid 5M 25 / 51.
inline int flat_wavefronts(int64_t nnz, int64_t S, int64_t n_rows, int64_t NBC)
{
    const bool short_segments = nnz < 8 * S;
    const bool local = NBC >= 4 && S <= 2 * n_rows && nnz >= 2 * S;
    const int64_t most = !local ? 3000000 : short_segments ? 12000000 : 4000000;
    return nnz > most ? 0 : short_segments ? 1 : 4;
}
// whether k_spmv_flat with `wpg` wavefronts per group gives a group a workgroup of its own: one wavefront
// takes 8 rounds, up to 512 nonzeros, per memory round trip
__host__ __device__ inline bool is_long_group(int32_t nnz, int32_t longest, int wpg) { return nnz > 2048 || (wpg > 1 && longest > 64); }

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
    const int32_t *unit_ptr, *unit_stripe, *unit_k, *multi_stripes;               // combine work units
    int32_t NM;                                                        // row blocks with several units
    int32_t claim;  // competitive groups a worker claims from a range's counter at a time
    int32_t SW, RW, GW;  // schedule weights of a slot, a round, a group (a nonzero weighs 1)
    int32_t steal_min;   // weight a range's competitive part must have left for another worker to enter it
    int32_t heavy_rounds;  // a group with a longer row is walked by all wavefronts of a worker together
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
    int32_t unroll;      // rounds taken per batch by the SpMV-part kernel
    double build_ms;
    // device arrays (owned): views into two allocations, arena[0] sized before the matrix is
    // looked at, arena[1] after the segment, group and block counts are known
    void *arena[2];
    size_t arena_bytes[2];
    int32_t *blk_bm, *blk_bn, *slot_ptr, *blk_group_ptr, *col_blk_ptr, *stripe_ptr, *stripe_blk;
    int32_t *group_ptr, *group_slot;
    int32_t *col_group_ptr, *comp_lo, *comp_col, *fixed_start, *fixed_col;
    int32_t *group_rounds;               // [G+1] prefix sums of the groups' longest rows
    int32_t *group_blk;                  // [G] block of each group
    int32_t *long_groups;                // [n_long] groups that k_spmv_flat gives a workgroup of their own
    int32_t n_long;
    int32_t flat_wpg;                    // wavefronts per group of k_spmv_flat; 0: k_spmv_part runs
    bool scheduled;                      // the caller chose something about the workers or their schedule
    int32_t *unit_ptr, *unit_stripe, *unit_k, *multi_stripes;
    int64_t U, NM;       // combine work units, row blocks cut into several units
    int32_t unit_slots;  // target slots per combine unit
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
int choose_block_parameters(const int32_t *csr_ptr, const int32_t *csr_col, int64_t n_rows, int64_t n_cols, int32_t value_bytes,
                            hbp_params_t &p, int64_t *nnz, hipStream_t stream);  // *nnz: unchanged where the matrix was not looked at
int derive_add_sign(const hbp_handle_s *h, int32_t *d_out, hipStream_t stream);
int hash_keys(const uint32_t *n, int64_t count, int32_t a, int32_t R, uint32_t *keys, hipStream_t stream);
int release_workspace();
int device_alloc(int device, size_t bytes, void **out);  // hipMalloc; where memory is short, after giving back what freed handles left
// takes back a handle's allocation; idle: nothing on the device uses it any more
void release_block(int device, void *base, size_t bytes, bool idle);

// spmv (hbp_spmv.hip)
Layout hbp_view(const hbp_handle_s *h);
int default_workers(int device, int32_t C, int32_t value_bytes, int32_t threads_wanted, int32_t *threads_out, int32_t *workers_out);
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
