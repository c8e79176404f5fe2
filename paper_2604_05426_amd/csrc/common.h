// Internal declarations shared by the translation units of libmultilora (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <memory>
#include <vector>

#include "multi_lora.h"

namespace mlora {

// ---- tiling constants (reported through multi_lora_plan_geometry) ------------------
constexpr int kBlockRows = 64;       // rows per LoRA block of the shrink kernels
constexpr int kBlockRowsWide = 128;  // the same for adapters of the wide rank class (their adapter tiles are the larger operand)
constexpr int kGemmBandTiles = 8;    // row tiles per band of the fused GEMM's tile order
constexpr int kGemmTileRows = 256;   // fused GEMM macro tile
constexpr int kGemmTileCols = 256;
constexpr int kWgradMinChunkRows = 512;  // smallest token chunk one weight-gradient work item reduces
constexpr int kNarrowMaxRank = 64;       // ranks above it form the wide rank class (their own kernel builds)
constexpr int kMaxSortedChunks = 16384;  // larger weight-gradient tables keep the canonical order
constexpr int kWgradPanelCols = 128;     // columns of X / dY one weight-gradient work item covers

// Tiled shrink kernels.  A contraction of 32 steps (64 elements each) or more is summed in 8 pieces whoever does it (see
// shrink_tiled_body): below, even the split launches would gain no more than 1 us, and the pieces cost the others 0.5-1 us.
constexpr int kMaxShrinkSplits = 8;
constexpr int shrink_log_pieces(int steps) { return steps < 32 ? 0 : 3; }

// Bytes of one work group's share (fp32 accumulators) where the largest rank of the block's class is `rank`: as many 16-wide rank blocks
// as that takes, of 64 rows (ranks up to 64) or 128.
constexpr int shrink_share_bytes(int rank) { return (rank + 15) / 16 * (rank > kNarrowMaxRank ? 8192 : 4096); }
// Allocations that hold a plan's shares, and the bytes of one (see mlora_plan::split_blocks).
constexpr int kSplitChunks = 3, kSplitChunkBytes = (2 << 20) - (128 << 10);

// Work groups that share one row block's contraction (`wide`: some block belongs to the wide rank class): the most that find room
// on the CUs, where the steps they save are more than the handing-over (stores and loads that bypass the L2, one counter round trip, and
// the last one reads all shares; four times the bytes in the wide class).  Measured on both sides of each line, us, blocks x contraction:
//   8 ways rather than 4: 19 x 3072  12.2 / 12.2, x 4096  12.8 / 13.3, x 14336  17.2 / 23.0; of few blocks always: 4 x 2048  10.6 / 11.6
//   4 ways rather than 1: 64 x 1792  12.8 / 13.2, x 2048  13.0 / 14.3, x 4096  17.0 / 22.4; wide: 32 x 2048  29.2 / 30.5,
//     64 x 2048  33.9 / 31.0, x 3072  37.1 / 41.7
//   2 ways rather than 1: 66 x 2560  14.7 / 15.9, x 3072  15.6 / 18.0; 128 x 2560  17.9 / 17.0, x 3072  19.0 / 19.2; wide: 128 x 4096
//     52.3 / 54.5 forward, 58.5 / 53.0 backward, x 5120  58.4 / 66.4 and 60.2 / 65.4
// `halves`: undivided, such a launch is divided by rows (shrink_halves_kernel), which hands nothing over, and the shares that it saves are
// large (a rank above 32; the lines above hold for smaller ones).  us, split / halves, the decoupled forward of 256 columns (shrink and expand-add), warm:
//   4 ways, 57 to 64 blocks, from 44 steps: 64 blocks, rank 64 at 32, 44, 52 steps split 1.11, 1.07, 1.04 times the halves' time, ranks 8 .. 64
//     1.04, 1.00, 0.98, one adapter of rank 64 among seven of 8 and 16 1.04, 0.97, 0.93; 33 to 56 blocks, from 36: 56 blocks, rank 64 at 32, 36, 44
//     1.02, 0.99, 0.97, ranks 8 .. 64 1.01, 1.00, 0.94, rank 48 0.98, 0.97, 0.92; 40 blocks, rank 64 at 48, 63 0.90, 0.86
//   2 ways, 65 to 128 blocks, from 80: 128 blocks, rank 64 at 48, 79 steps 1.15, 1.10, one of 64 among seven 1.09, 1.10; 96 blocks 1.09, 1.05 and
//     1.07, 1.03
// Blocks of 32 rows or fewer have no second half: neither form is faster for them within these lines (48 segments of 20 tokens at 32 .. 48 steps
// 0.97 .. 1.02, 64 of 31 0.98 .. 1.01, 100 of 30 at 48 .. 79 0.98 .. 1.01).
inline int shrink_splits(int64_t blocks, int64_t contraction, int num_cus, bool wide, bool halves = false) {
    const int64_t steps = contraction / 64;
    if (blocks <= 0 || shrink_log_pieces((int)steps) == 0) return 1;
    if (8 * blocks <= num_cus && (steps >= 64 || blocks <= 8)) return 8;
    if (4 * blocks <= num_cus) return steps >= (blocks <= 32 ? 32 : halves ? (blocks > 56 ? 44 : 36) : wide ? 48 : 32) ? 4 : 1;
    if (2 * blocks <= num_cus) return steps >= (wide || halves ? 80 : 48) ? 2 : 1;
    return 1;
}

// One entry of any plan table: 4 x int32 (meaning depends on the table).
struct Entry4 {
    int32_t a, b, c, d;
};

// Per-adapter pointers, refreshed by every fwd/bwd call (device resident).
struct AdapterPtrs {
    const void* A;
    const void* B;
    void* dA;
    void* dB;
};

// Owner of one hipMalloc'd block.
struct DeviceBlock {
    void* ptr = nullptr;
    ~DeviceBlock() {
        if (ptr) (void)hipFree(ptr);
    }
};

// Device-resident view of a plan, passed by value to kernels.
struct PlanView {
    int32_t N;
    int64_t T, k, n;
    const int32_t* off;     // [N+1] segment offsets (rows)
    const int32_t* rank;    // [N]
    const float* scale;     // [N]
    const int64_t* soff;    // [N+1] element offsets of S_i / dS_i in the ragged buffers
    const AdapterPtrs* ptrs; // [N]
    const Entry4* row_blocks;  int32_t n_row_blocks;      // canonical order (adapter, block)
    const Entry4* class_blocks; int32_t n_class_blocks;   // the same blocks, wide rank class first: what the kernels walk
    const Entry4* gemm_tiles;  int32_t n_gemm_tiles;
    const Entry4* band_order;  int32_t n_bands;           // launch order of the fused GEMM's row bands
    const Entry4* wgrad_chunks; int32_t n_wgrad_chunks;
    const int32_t* wgrad_chunk_start; // [N+1] canonical prefix: adapter i has start[i+1] - start[i] chunks
    const int64_t* part_off;   // [N] float offset of adapter i's partial weight-gradient block (adapters with > 1 chunk)
};

// What the device-side scheduler chose and counted; read back once by plan creation (sizes of the chunk table and of
// the workspace, launch grids).
struct DevGeo {
    int32_t chunk_rows, chunk_rows_wide;      // token chunk of the weight-gradient items per rank class
    int32_t n_chunks, n_chunks_wide;          // entries of the chunk table; the first n_chunks_wide are the wide class
    int32_t max_chunks_per_adapter, n_reduce; // n_reduce adapters have their tokens split over several chunks
    int64_t partial_floats;                   // fp32 partial sums those adapters need
    int64_t R1;                               // cross-checks of the sizes the host derived from the same offsets
    int32_t n_row_blocks, n_blocks_wide;
};

}  // namespace mlora

struct mlora_plan {
    int dtype = 0;
    int64_t T = 0, k = 0, n = 0;
    int32_t N = 0;
    std::vector<int32_t> ranks;
    std::vector<float> scales;
    std::vector<int64_t> off;
    std::vector<int32_t> off32;      // N+1, upload source
    int64_t R1 = 0;
    bool use_mfma = false;
    int32_t n_row_blocks = 0, n_gemm_tiles = 0, n_bands = 0;
    int32_t max_rank = 0;
    // Row blocks by rank class (<= 64 / wider): the class table puts the wide class first (its blocks run longest); plans
    // that mix narrow and wide ranks run each class through the kernel build made for it.
    int32_t n_blocks_narrow = 0, n_blocks_wide = 0;
    // Weight-gradient items: chosen, counted and ordered on the device (DevGeo).  Plans that mix ranks <= 64 and wider
    // ones launch the items of the two classes as two launches over their own parts of the table, each through the
    // kernel build - and so at the workgroups per CU - its class allows, and chunk the tokens per class.
    mlora::DevGeo geo{};
    int32_t max_rank_narrow = 0, max_rank_wide = 0;      // largest rank <= 64 and largest rank above it among adapters with tokens
    bool ranks_mult8 = true;          // every rank of an adapter with tokens is a multiple of 8
    // Device allocations: the plan's own blocks, and every block of other plans its view points into (a plan made by
    // multi_lora_plan_create_like uses the segmentation tables of its base in place - and through it those of the
    // base's base -, so plans may be destroyed in any order).
    std::vector<std::shared_ptr<mlora::DeviceBlock>> blocks;
    std::vector<std::shared_ptr<mlora::DeviceBlock>> shared_blocks;
    bool shares_tables = false;
    mlora::PlanView view{};
    mlora::AdapterPtrs* d_ptrs = nullptr;
    // host mirror of the device pointer table: a call whose pointers match what the same stream uploaded last skips the
    // upload.  Once an upload has been recorded into a captured graph the mirror is never trusted again: a replay
    // rewrites the table behind the host's back.
    std::vector<mlora::AdapterPtrs> ptr_mirror;
    bool ptr_mirror_valid = false;
    bool ptr_upload_captured = false;
    hipStream_t ptr_mirror_stream = nullptr;
    bool grads_over_A = false;        // a gradient of the mirror lies over an A_i of it (see upload_ptrs)
    // Shares of split shrink contractions.  Up to kSplitChunks allocations of less than 2 MB, each for as many whole row blocks as
    // fit at `split_slot` bytes a share (both rank classes alike): those come from memory the runtime keeps at hand (1 us for an
    // allocation and its release, 24 us from 2 MB on, which a plan made for every step would pay every step; more than three of them
    // cost 100 us).  What does not fit is one allocation with shares of each class's own size (split_slot 0).
    std::vector<std::shared_ptr<mlora::DeviceBlock>> split_blocks;
    int32_t split_slot = 0, split_chunk_shares = 0;      // shares in every allocation but the last
    uint32_t* d_arrived = nullptr;    // arrival counters of the split contractions (two per block)
    int32_t* d_reduce_list = nullptr; // adapters whose tokens are split over several weight-gradient chunks
    bool has_empty_ranked = false;    // some adapter has a rank but no tokens (its dA, dB are zero-filled)
    size_t ws_ds_bytes = 0;           // workspace: dS
    size_t ws_partial_bytes = 0;      // workspace: fp32 partial weight gradients
    hipStream_t build_stream = nullptr;
    int num_cus = 256;
    // per-kernel event timing (multi_lora_profile_begin / _end)
    bool prof_on = false;
    int32_t prof_used = 0;
    std::vector<int32_t> prof_kernel;
    std::vector<hipEvent_t> prof_start, prof_stop;
};

namespace mlora {

// Whether the plan's tiled shrink (fwd) or gradient shrink deals undivided row blocks out by halves, and into how many shares it divides their
// contraction: what the launches do and what plan creation holds memory for.
inline bool shrink_by_halves(const mlora_plan* p, bool fwd) {
    return p->n_blocks_wide == 0 && 2 * p->n_blocks_narrow <= p->num_cus && !(fwd && !p->ranks_mult8) && (fwd ? p->k : p->n) >= 256;
}
inline int shrink_splits(const mlora_plan* p, bool fwd) {
    return shrink_splits((int64_t)p->n_blocks_wide + p->n_blocks_narrow, fwd ? p->k : p->n, p->num_cus, p->n_blocks_wide != 0,
                         shrink_by_halves(p, fwd) && p->max_rank_narrow > 32);
}

void set_error(const std::string& msg);
int hip_fail(hipError_t e, const char* what);

#define MLORA_HIP_TRY(expr)                                   \
    do {                                                      \
        hipError_t e__ = (expr);                              \
        if (e__ != hipSuccess) return ::mlora::hip_fail(e__, #expr); \
    } while (0)

// Brackets one kernel launch with events while profiling is on (no-op otherwise).
struct ProfScope {
    mlora_plan* p;
    hipStream_t st;
    int32_t idx = -1;
    ProfScope(mlora_plan* plan, int kernel, hipStream_t stream) : p(plan), st(stream) {
        if (p->prof_on && p->prof_used < (int32_t)p->prof_start.size()) {
            idx = p->prof_used++;
            p->prof_kernel[idx] = kernel;
            (void)hipEventRecord(p->prof_start[idx], st);
        }
    }
    ~ProfScope() {
        if (idx >= 0) (void)hipEventRecord(p->prof_stop[idx], st);
    }
};

// api.hip : looks up the static workspace of multi_lora_bwd_static on the current device (idempotent)
void prepare_static_workspace();

// plan.hip
int upload_ptrs(mlora_plan* p, const void* const* A, const void* const* B, void* const* dA,
                void* const* dB, hipStream_t st);

// general.hip : fp32, and bf16 whose k or n is not a multiple of 8
int general_forward(mlora_plan* p, const void* X, const void* W, void* Y, void* S, uint32_t flags,
                    hipStream_t st);
int general_backward(mlora_plan* p, const void* dY, const void* X, const void* W, const void* S,
                     void* dX, void* dS, uint32_t flags, hipStream_t st);

// mfma_*.hip : bf16 MFMA kernels
int mfma_forward(mlora_plan* p, const void* X, const void* W, void* Y, void* S, uint32_t flags,
                 hipStream_t st);
int mfma_backward(mlora_plan* p, const void* dY, const void* X, const void* W, const void* S,
                  void* dX, void* dS, float* partials, uint32_t flags, hipStream_t st);

}  // namespace mlora
