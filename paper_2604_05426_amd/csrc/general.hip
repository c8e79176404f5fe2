// The general kernels: fp32 plans, and bf16 plans whose k or n is not a multiple of 8 (rows that start at any element).
// Every step of the layer (paper Sec. 5.1) is one grouped launch on the matrix units, with fp32 accumulation:
//   S_i = X_i A_i, dS_i = s_i dY_i B_i^T               general_shrink_kernel
//   Y = X W + s_i S_i B_i, dX = dY W^T + dS_i A_i^T    general_gemm_kernel, whole_tile_kernel in bf16 (also either term alone); fp32: f32_gemm.hip
//   dA_i = X_i^T dS_i, dB_i = s_i S_i^T dY_i           general_wgrad_kernel
// No operand needs an alignment beyond its element: 16-byte pieces are loaded from wherever they start (global memory takes any
// alignment), pieces that cross an edge element by element.
//
// Everything here is bound by latency (short segments, few tiles): the contractions of shrink and weight gradients are split over the
// wavefronts of a work group and summed in a fixed order in LDS, and loads run ahead of the MFMAs in registers.  Edges cost nothing in the main
// loops: the last tile of rows or columns starts early enough to be whole, and only the last step of a contraction takes a mask (with a
// condition on every load, the edge tiles alone made the bf16 products of 1500 x 1001 outputs 52 us instead of 27).
//
// Order of the sums: it follows from the contraction alone, not from the tile or the build that a batch is given, so that an adapter's rows
// of S, Y, dS and dX have the same bits whatever its neighbours' tokens and ranks are.
//
// One step forward and backward, before (a scalar-FMA grouped product whose descriptors took a launch each) and now: fp32, 4 x 64
// tokens, 256 x 256: 171 -> 21 us; fp32, 2048 tokens, 2048 x 2048: 1590 -> 255 us; bf16, 1500 tokens, 2048 x 1001: 1105 -> 62 us.
#include <type_traits>

#include "general_wgrad.h"

namespace mlora {

namespace {

// ---- shrink ------------------------------------------------------------------------------------------------------------------
// Work group = 16 rows of one adapter x 16 NB of its ranks (see `shrink`); its eight wavefronts deal the contraction among themselves
// two neighbouring pieces at a time (whole 128-byte lines of a row), straight from memory into MFMA operands (X / dY rows are read
// once; the adapter matrix comes from the caches), with the operands of the next load in flight.  In fp32 a wavefront's pairs of
// pieces take turns on two accumulator sets (less rounding error than one chain) and a contraction of up to eight pieces is dealt
// singly; the wavefronts' sums are added in LDS in wavefront order.
template <typename T> struct GenShrinkArgs {
    const T* src; int64_t ld;     // X (ld k) or dY (ld n); the contraction has ld elements
    T* out;                       // ragged S or dS
    int32_t rank_items;           // work groups along the ranks, 16 NB each
    int32_t order;                // 0: these side by side, 1: one after the other, 2: side by side, all blocks' first 16 rows before the others
    PlanView pv;
};

template <typename T, bool FWD, int NB>
__global__ __launch_bounds__(512) void general_shrink_kernel(GenShrinkArgs<T> g) {
    constexpr int NW = 8;
    constexpr int RLD = NB * 16 + 4;
    __shared__ float red[NW * 16 * RLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int64_t item = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, groups = (int64_t)g.pv.n_row_blocks * 4;
    if (item >= groups * g.rank_items) return;
    auto quotient = [](int64_t a, int64_t b) { return ((a | b) >> 32) == 0 ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b; };     // (64-bit ones cost 0.2 us a launch)
    const int64_t over = quotient(item, g.order == 1 ? groups : g.rank_items);
    const int64_t wg = g.order == 1 ? item - over * groups : over;
    const int64_t rank_item = g.order == 1 ? over : item - over * g.rank_items;
    const int64_t place = g.order == 2 ? quotient(wg, g.pv.n_row_blocks) : wg & 3;
    const Entry4 e = g.pv.row_blocks[g.order == 2 ? wg - place * g.pv.n_row_blocks : wg >> 2];
    const int sub = (int)place * 16, rows = min(16, e.d - sub);
    if (rows <= 0) return;
    const int i = e.a, row0 = e.c + sub;
    const int r = g.pv.rank[i], rho0 = (int)rank_item * (16 * NB), rl = min(r - rho0, 16 * NB);      // this work group's ranks
    if (rl <= 0) return;
    const float s = FWD ? 1.0f : g.pv.scale[i];
    const T* F = global_ptr<const T>(FWD ? g.pv.ptrs[i].A : g.pv.ptrs[i].B) + (FWD ? (int64_t)rho0 : rho0 * g.ld);
    const int K = (int)g.ld;
    const T* xrow = g.src + (int64_t)(row0 + min(l16, rows - 1)) * g.ld;    // rows past the block repeat its last one: not stored
    // Ranks of block b, from rho0 on: 16 b + l16, or, where four blocks share one 64-rank row piece of A_i, quad(b / 4) + b % 4: four adjacent
    // ranks per lane.  The lane that would cross r_i takes the last four ranks instead (what it repeats comes out the same, bit for
    // bit, from the lane before), so that any rank from 4 on is read in whole quads.
    constexpr bool QUAD = FWD && NB >= 4;
    constexpr bool TWO = sizeof(T) == 4;                 // two chains a wavefront; in bf16, rounded to 16 bits, one does: fewer registers
    f32x4 acc[NB], other[TWO ? NB : 1];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (TWO) {
#pragma unroll
        for (int b = 0; b < NB; ++b) other[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int U = NB >= 8 ? 1 : 2;                   // pieces a wavefront loads at a time (two would spill)
    constexpr int NQ = QUAD ? NB / 4 : 1, NF = QUAD ? 1 : NB;
    uint4 xa[2][U], fb[2][U][NF];
    quad_t<T> fq[2][U][NQ][kQuadRows<T>];
    // Ranks past r_i repeat valid ones (their sums are not stored); only the end of the contraction has to read as zero, in both
    // operands.  The plain loads of a whole unit stand in one branch: a condition per load would make each wait for itself.
    const bool quads = rl >= 4;
    auto quad = [&](int q) { return min(64 * q + 4 * l16, rl - 4); };
    auto load = [&](int unit, int set) {
        const int k0 = unit * U * kBlockK<T> + g4 * kEpc<T>;
        if ((unit + 1) * U * kBlockK<T> <= K && (quads || !QUAD)) {     // uniform over the wavefront
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * kBlockK<T>;
                __builtin_memcpy(&xa[set][u], xrow + k, 16);
                if constexpr (QUAD) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
#pragma unroll
                        for (int e = 0; e < kQuadRows<T>; ++e)
                            __builtin_memcpy(&fq[set][u][q][e], F + (int64_t)(k + e) * r + quad(q), sizeof(quad_t<T>));
                } else {
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const int rho = min(16 * b + l16, rl - 1);
                        if constexpr (FWD) {
                            T* o = reinterpret_cast<T*>(&fb[set][u][b]);
#pragma unroll
                            for (int e = 0; e < kEpc<T>; ++e) o[e] = F[(int64_t)(k + e) * r + rho];
                        } else {
                            __builtin_memcpy(&fb[set][u][b], F + (int64_t)rho * g.ld + k, 16);
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * kBlockK<T>, valid = K - k;
                xa[set][u] = load16<T>(xrow + k, valid);
                if constexpr (QUAD) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int rho = quads ? quad(q) : min(4 * l16, rl - 1);
#pragma unroll
                        for (int e = 0; e < kQuadRows<T>; ++e) {
                            fq[set][u][q][e] = (quad_t<T>)(0u);
                            if (e < valid) fq[set][u][q][e] = load_quad<T>(F + (int64_t)(k + e) * r + rho, quads, rl - rho);
                        }
                    }
                } else {
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const int rho = min(16 * b + l16, rl - 1);
                        if (FWD) fb[set][u][b] = gather16<T>(F + (int64_t)k * r + rho, r, valid);
                        else     fb[set][u][b] = load16<T>(F + (int64_t)rho * g.ld + k, valid);
                    }
                }
            }
        }
    };
    auto compute_piece = [&](int set, int u, f32x4 (&to)[NB]) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if constexpr (QUAD) {
                if (64 * (b / 4) < rl) to[b] = block_mma<T>(xa[set][u], quad_column<T>(fq[set][u][b / 4], b % 4), to[b]);
            } else {
                if (16 * b < rl) to[b] = block_mma<T>(xa[set][u], fb[set][u][b], to[b]);
            }
        }
    };
    auto compute = [&](int set, f32x4 (&to)[NB]) {
#pragma unroll
        for (int u = 0; u < U; ++u) compute_piece(set, u, to);
    };
    const int units = (K + U * kBlockK<T> - 1) / (U * kBlockK<T>);
    // wavefront w takes the pairs of pieces w, w + 8, w + 16, ..., in fp32 in turn into acc and other
    if (TWO && K <= NW * kBlockK<T>) {
        // up to 128 elements of fp32, one piece a wavefront: S is off by 0.8 of what it is with pairs (1.07e-7 -> 8.4e-8 relative at 64
        // elements), in the same time
        if (wave / U < units) {
            load(wave / U, 0);
            if (U == 1 || wave % 2 == 0) compute_piece(0, 0, acc);
            else                         compute_piece(0, U - 1, acc);
        }
    } else if constexpr (U == 2) {
        if (wave < units) load(wave, 0);
        for (int p = wave; p < units; p += 2 * NW) {
            if (p + NW < units) load(p + NW, 1);
            compute(0, acc);
            if (p + 2 * NW < units) load(p + 2 * NW, 0);
            if constexpr (TWO) { if (p + NW < units) compute(1, other); }
            else               { if (p + NW < units) compute(1, acc); }
        }
    } else {
        // the same sums, all of one chain first: both sets in one loop spill
        constexpr int NEXT = (TWO ? 4 : 2) * NW;         // from one pair of a chain to its next
#pragma unroll 1
        for (int turn = 0; turn < (TWO ? 2 : 1); ++turn) {
            const int first = 2 * (wave + NW * turn);
            if constexpr (TWO) {
#pragma unroll
                for (int b = 0; b < NB; ++b) { other[b] = acc[b]; acc[b] = f32x4{0.f, 0.f, 0.f, 0.f}; }
            }
            if (first < units) load(first, 0);
            for (int p = first; p < units; p += NEXT) {
                if (p + 1 < units) load(p + 1, 1);
                compute(0, acc);
                if (p + NEXT < units) load(p + NEXT, 0);
                if (p + 1 < units) compute(1, acc);
            }
        }
    }
    if constexpr (TWO) {
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] += other[b];
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rho = !QUAD ? 16 * b + l16 : quads ? quad(b / 4) + b % 4 : 4 * l16 + b;
            if (!QUAD || (64 * (b / 4) < rl && rho < rl)) red[(wave * 16 + 4 * g4 + q) * RLD + rho] = acc[b][q];
        }
    __syncthreads();
    T* out = g.out + g.pv.soff[i] + (int64_t)(row0 - g.pv.off[i]) * r + rho0;
    for (int idx = tid; idx < rows * rl; idx += 64 * NW) {
        const int row = idx / rl, col = idx - row * rl;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[(w * 16 + row) * RLD + col];
        out[(int64_t)row * r + col] = from_f32<T>(s * v);
    }
}

// ---- bf16 products with the frozen weight, and the rank extension (fp32: f32_gemm.hip) -------------------------------------------
struct GenGemmArgs {
    typedef u16 T;
    const T* A; const T* W;       // X (fwd) or dY (bwd); W [k][n]
    T* C;                         // Y or dX
    const T* E;                   // ragged S or dS
    int64_t lda, ldw, ldc;
    int64_t M, N, K;
    int64_t tiles_n;
    int64_t R1;                   // elements of E
    int32_t base, lora;           // which terms; without the base term C += LoRA term
    int32_t xcd_run;              // whole tiles: consecutive tiles per XCD
    PlanView pv;
};

// ---- whole 64 x 64 tiles ---------------------------------------------------------------------------------------------------------
// For products of at least 128 rows, 64 columns and a contraction of 64 that fill half of the chip with such tiles (see the launch): four wavefronts
// load and four multiply.  The loads of four steps are on their way in the loading wavefronts' registers (rows start at any element, so they cannot go to
// LDS directly), which hand a step over in one of two LDS stages per barrier; the multiplying ones (2 x 2 sub-tiles) read a step's fragments while the
// one before it is multiplied.  With wavefronts that did both (KC = 1 below, which other sizes and the LoRA term alone still take) a step took
// 1500 cycles, the time of its loads, LDS stores, fragment reads and products after one another.  us, before / now: 1500 x 1001 outputs, contraction 2048, 22.2 /
// 17.5; 1000 x 1001 15.1 / 11.0; 1500 x 2048, contraction 1001, backward 22.4 / 20.2.
// Sums in the order of the other tiles (see below).  The operands of the first rank-extension pass are staged while the contraction ends.
// BM x 64, BM 64 or 128.
template <int BM> constexpr int kWholeStage = (BM + 64) * 128;       // bytes of a step's operand tiles [BM][64] and [64][64]
template <bool FWD, int BM>
__device__ __forceinline__ void whole_tile_body(const GenGemmArgs& g, unsigned char* const lds, const uint32_t wg) {
    constexpr int STAGE = kWholeStage<BM>, AT = BM * 128, NA = BM / 32, MB = BM / 32;      // pieces of A per lane and step; row blocks of a wavefront
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave >= 4;
    const int wm = (wave >> 1) & 1, wn = wave & 1, l16 = lane & 15, g4 = lane >> 4;
    const int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (int)g.tiles_n;
    const uint32_t slot_x = wg / 8, L = ((slot_x / g.xcd_run) * 8 + wg % 8) * g.xcd_run + slot_x % g.xcd_run;
    if (L >= (uint32_t)tiles_m * (uint32_t)tiles_n) return;         // (a launch of two dimensions holds more)
    const int band = (int)(L / (8u * tiles_n)), in_band = (int)(L - (uint32_t)band * 8u * tiles_n), band_rows = min(8, tiles_m - band * 8);
    // The last tile of rows / columns starts early enough to be whole; what it shares with the tile before is not stored.
    const int64_t m_own = (int64_t)(band * 8 + in_band % band_rows) * BM, n_own = (int64_t)(in_band / band_rows) * 64;
    const int64_t m0 = min(m_own, g.M - BM), n0 = min(n_own, g.N - 64);
    const int lo_t = (int)m0, hi_t = lo_t + BM;

    // lane l holds the metadata of candidate adapter first + l
    int first = 0, cand_end = g.lora ? g.pv.N : 0;
    if (cand_end > 64) {
        first = g.pv.gemm_tiles[m0 / kGemmTileRows].c;
        cand_end = g.pv.gemm_tiles[(m0 + BM - 1) / kGemmTileRows].d;
    }
    int c_rank = 0, c_off = 0, c_end = 0;
    int64_t c_so = 0;
    uint64_t c_f = 0;
    float c_sc = 1.0f;
    auto candidates = [&]() {
        const int cand = min(first + lane, cand_end - 1);
        c_rank = g.pv.rank[cand]; c_off = g.pv.off[cand]; c_end = g.pv.off[cand + 1];
        c_so = g.pv.soff[cand];
        c_f = reinterpret_cast<uint64_t>(FWD ? g.pv.ptrs[cand].B : g.pv.ptrs[cand].A);
        if (FWD) c_sc = g.pv.scale[cand];
    };
    auto mine = [&]() { return __ballot(first + lane < cand_end && c_rank > 0 && max(c_off, lo_t) < min(c_end, hi_t)); };
    auto barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // where 16-byte piece (row, c) of a tile whose contraction is contiguous goes, and (contraction row k, 8 columns c) of a W / B_i tile
    auto place = [](int row, int c) { return row * 128 + ((c ^ (row & 7)) << 4); };
    auto key = [](int k) { return ((k >> 1) & 1) | (((k >> 3) & 1) << 1); };
    auto place_w = [&](int k, int c) { return k * 128 + (((c >> 1) ^ key(k)) << 5) + ((c & 1) << 4); };
    const int whole = (int)(g.K / 64), left = (int)(g.K - (int64_t)whole * 64), steps = whole + (left > 0);
    unsigned char* const pass = lds + 2 * STAGE;

    if (loader) {
        // each wavefront takes a quarter of the rows of both tiles, eight at a time, lane l piece (l / 8, l % 8) of these
        const int arow = (wave - 4) * (BM / 4) + (lane >> 3), row = (wave - 4) * 16 + (lane >> 3), ch = lane & 7;
        const u16* const pa = g.A + (m0 + arow) * g.lda + ch * 8;
        const u16* const pb = FWD ? g.W + (int64_t)row * g.ldw + n0 + ch * 8 : g.W + (n0 + row) * g.ldw + ch * 8;
        const int64_t a8 = 8 * g.lda, b8 = 8 * g.ldw, bstep = FWD ? 64 * g.ldw : 64;
        constexpr int D = 4;                             // steps on their way
        auto as_vec = [](uint4 v) { return u32x4v{v.x, v.y, v.z, v.w}; };
        auto as_uint4 = [](u32x4v v) { return make_uint4(v[0], v[1], v[2], v[3]); };
        u32x4v ra[D + 2][NA], rb[D + 2][2];              // the last two: what is left of the contraction, a pass of the rank extension
        auto load = [&](int d, int t) __attribute__((always_inline)) {
            const u16* const a = pa + (int64_t)t * 64;
            const u16* const b = pb + t * bstep;
#pragma unroll
            for (int j = 0; j < NA; ++j) __builtin_memcpy(&ra[d][j], a + j * a8, 16);
            __builtin_memcpy(&rb[d][0], b, 16);
            __builtin_memcpy(&rb[d][1], b + b8, 16);
        };
        auto store = [&](unsigned char* to, int d) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NA; ++j) *reinterpret_cast<u32x4v*>(to + place(arow + 8 * j, ch)) = ra[d][j];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                *reinterpret_cast<u32x4v*>(to + AT + (FWD ? place_w(row + 8 * j, ch) : place(row + 8 * j, ch))) = rb[d][j];
            }
        };
        // What is left of a contraction that is no multiple of 64: pieces that would reach past their row are loaded from where they still fit and
        // shifted, contraction rows past the end (forward: of W) repeat the last one and are taken as zero.
        auto load_rest = [&]() __attribute__((always_inline)) {
            const int64_t k0 = (int64_t)whole * 64;
            const int64_t at = min(k0 + ch * 8, g.K - 8) - ch * 8;
#pragma unroll
            for (int j = 0; j < NA; ++j) __builtin_memcpy(&ra[D][j], pa + at + j * a8, 16);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const u16* const b = FWD ? g.W + min(k0 + row + 8 * j, g.K - 1) * g.ldw + n0 + ch * 8 : pb + j * b8 + at;
                __builtin_memcpy(&rb[D][j], b, 16);
            }
        };
        // Passes of the rank extension: 64 ranks of an adapter each; the first one's operands are asked for before the contraction's.  Elements
        // r0 + 8 ch .. of rows of rk that start anywhere: a piece that would reach past its row is loaded from where it still fits and shifted.
        uint64_t todo = 0;
        int r0 = 0, by = 0, ranks = 0, rank = 0;         // ranks of the lowest adapter in todo asked for; of the pass asked for last: shift, ranks, its adapter's
        bool fetched = false;
        auto fetch = [&]() __attribute__((always_inline)) {
            fetched = todo != 0;
            if (!fetched) return;
            const int l = (int)__builtin_ctzll(todo);
            auto lane64 = [&](uint64_t x) __attribute__((always_inline)) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)x, l);
            };
            const int rk = __builtin_amdgcn_readlane(c_rank, l), seg0 = __builtin_amdgcn_readlane(c_off, l), seg1 = __builtin_amdgcn_readlane(c_end, l);
            const u16* const F = global_ptr<const u16>(reinterpret_cast<const void*>(lane64(c_f)));
            const u16* const E = g.E + (int64_t)lane64((uint64_t)c_so);
            auto e_row = [&](int j) { return E + (int64_t)(min(max(lo_t + arow + 8 * j, seg0), seg1 - 1) - seg0) * rk; };      // (rows of others: dropped)
            auto f_row = [&](int j) { return F + (n0 + row + 8 * j) * rk; };
            const int at = r0 + ch * 8;
            ranks = min(64, rk - r0);
            rank = rk;
            if (rk >= 8) {
                const int from = min(at, rk - 8);
                by = at - from;
#pragma unroll
                for (int j = 0; j < NA; ++j) __builtin_memcpy(&ra[D + 1][j], e_row(j) + from, 16);
                if (!FWD) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) __builtin_memcpy(&rb[D + 1][j], f_row(j) + from, 16);
                }
            } else {         // less than a piece: one that starts with the row, or early enough to end with the buffer
                by = 0;
                auto few = [&](u32x4v& v, const u16* row_, const u16* end, int j) __attribute__((always_inline)) {
                    const u16* const from = min(row_, end - 8);
                    by |= (int)(row_ - from) << 4 * j;
                    __builtin_memcpy(&v, from, 16);
                };
#pragma unroll
                for (int j = 0; j < NA; ++j) few(ra[D + 1][j], e_row(j), g.E + g.R1, j);
                if (!FWD) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) few(rb[D + 1][j], f_row(j), F + g.N * rk, NA + j);
                }
            }
            if (FWD) {
#pragma unroll
                for (int j = 0; j < 2; ++j) __builtin_memcpy(&rb[D + 1][j], F + (int64_t)min(r0 + row + 8 * j, rk - 1) * g.N + n0 + ch * 8, 16);
            }
            if (r0 + 64 < rk) r0 += 64;
            else { todo &= todo - 1; r0 = 0; }
        };
        auto shift = [&]() __attribute__((always_inline)) {      // zeros past the ranks
            auto each = [&](auto piece) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NA; ++j) ra[D + 1][j] = as_vec(piece(as_uint4(ra[D + 1][j]), j));
                if (!FWD) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) rb[D + 1][j] = as_vec(piece(as_uint4(rb[D + 1][j]), NA + j));
                }
            };
            if ((rank & 7) == 0) each([&](uint4 v, int) { return by == 0 ? v : zero4(); });      // (a pass takes longer by what stands here)
            else if (rank > 8)   each([&](uint4 v, int) { return drop_front(v, by); });
            else                 each([&](uint4 v, int j) { return keep_front(drop_front(v, by >> 4 * j & 15), ch == 0 ? rank : 0); });
            if (FWD) {
#pragma unroll
                for (int j = 0; j < 2; ++j) rb[D + 1][j] = as_vec(row + 8 * j < ranks ? as_uint4(rb[D + 1][j]) : zero4());
            }
        };
        // (Oldest first and in the loop's own order: the waits in the loop are for the worse of what comes in from here and from its end.)
        if (first < cand_end) { candidates(); todo = mine(); fetch(); }
        if (left > 0) load_rest();
        __builtin_amdgcn_sched_barrier(0);
        load(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(1, min(1, whole - 1));
        __builtin_amdgcn_sched_barrier(0);
        load(2, min(2, whole - 1));
        __builtin_amdgcn_sched_barrier(0);
        load(3, min(3, whole - 1));
        __builtin_amdgcn_sched_barrier(0);
        int t = 0;
        auto one_step = [&](auto d_) __attribute__((always_inline)) {        // (D is even: step t + d is of the parity of d)
            constexpr int d = decltype(d_)::value;
            store(lds + (d & 1) * STAGE, d);
            load(d, min(t + d + D, whole - 1));
            __builtin_amdgcn_sched_barrier(0);
            barrier();
        };
        for (; t + D <= whole; t += D) {
            one_step(std::integral_constant<int, 0>{});
            one_step(std::integral_constant<int, 1>{});
            one_step(std::integral_constant<int, 2>{});
            one_step(std::integral_constant<int, 3>{});
        }
        static_assert(D == 4, "what is left of the steps");
        if (t < whole) { store(lds, 0); barrier(); }
        if (t + 1 < whole) { store(lds + STAGE, 1); barrier(); }
        if (t + 2 < whole) { store(lds, 2); barrier(); }
        if (left > 0) {
            const int sh = max(0, ch * 8 + 8 - left);
#pragma unroll
            for (int j = 0; j < NA; ++j) ra[D][j] = as_vec(drop_front(as_uint4(ra[D][j]), sh));
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                rb[D][j] = as_vec(FWD ? (row + 8 * j < left ? as_uint4(rb[D][j]) : zero4()) : drop_front(as_uint4(rb[D][j]), sh));
            }
            store(lds + (whole & 1) * STAGE, D);
            barrier();
        }
        // ---- passes of the rank extension ----
        while (first < cand_end) {
            while (fetched) {
                shift();
                store(pass, D + 1);
                barrier();                               // staged
                fetch();
                barrier();                               // used
            }
            first += 64;
            if (first < cand_end) { candidates(); todo = mine(); fetch(); }
        }
    }

    f32x4 acc[MB][2];
    if (!loader) {
        if (first < cand_end) candidates();
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
        bf16x8 fa[2][2][MB], fb[2][2][2];                // [set][32-wide half][block]
        auto read = [&](auto set, const unsigned char* from) __attribute__((always_inline)) {
            constexpr int S = decltype(set)::value;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int x = 0; x < MB; ++x) fa[S][h][x] = lds_read_frag(reinterpret_cast<const u16*>(from + place(wm * (BM / 2) + x * 16 + l16, h * 4 + g4)));
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    if (FWD) {
                        const int k = h * 32 + 8 * g4 + (l16 >> 2);
                        const unsigned char* p = from + AT + k * 128 + (((wn * 2 + x) ^ key(k)) << 5) + (l16 & 3) * 8;      // (rows k and k + 4 share their key)
                        fb[S][h][x] = lds_read_frag_tr(reinterpret_cast<const u16*>(p), reinterpret_cast<const u16*>(p + 4 * 128));
                    } else {
                        fb[S][h][x] = lds_read_frag(reinterpret_cast<const u16*>(from + AT + place(wn * 32 + x * 16 + l16, h * 4 + g4)));
                    }
                }
            }
        };
        // operands swapped: a lane holds one output row and 4 consecutive columns of each block
        auto multiply = [&](f32x4 (&c)[MB][2], auto set) __attribute__((always_inline)) {
            constexpr int S = decltype(set)::value;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < MB; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) c[x][y] = mfma16(fb[S][h][y], fa[S][h][x], c[x][y]);
        };
        const std::integral_constant<int, 0> f0{};
        const std::integral_constant<int, 1> f1{};
        barrier();
        read(f0, lds);
        int t = 0;
        for (; t + 2 < steps; t += 2) {
            barrier();
            read(f1, lds + STAGE);
            multiply(acc, f0);
            barrier();
            read(f0, lds);
            multiply(acc, f1);
        }
        if (t + 1 < steps) {
            barrier();
            read(f1, lds + STAGE);
            multiply(acc, f0);
            multiply(acc, f1);
        } else {
            multiply(acc, f0);
        }
        // rank extension, adapter by adapter into a second accumulator set, of which the adapter's own rows are added: another adapter's
        // operands never touch a row, whatever they hold
        while (first < cand_end) {
            uint64_t todo = mine();
            while (todo) {
                const int l = (int)__builtin_ctzll(todo);
                todo &= todo - 1;
                const int rk = __builtin_amdgcn_readlane(c_rank, l);
                const int lo = max(__builtin_amdgcn_readlane(c_off, l), lo_t), hi = min(__builtin_amdgcn_readlane(c_end, l), hi_t);
                const float s = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c_sc), l));
                f32x4 ext[MB][2];
#pragma unroll
                for (int x = 0; x < MB; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) ext[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int r0 = 0; r0 < rk; r0 += 64) {
                    barrier();                           // staged
                    read(f0, pass);
                    multiply(ext, f0);
                    barrier();                           // used
                }
#pragma unroll
                for (int x = 0; x < MB; ++x) {
                    const int row = lo_t + wm * (BM / 2) + x * 16 + l16;
                    const bool own = row >= lo && row < hi;
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[x][y][q] = own ? acc[x][y][q] + s * ext[x][y][q] : acc[x][y][q];
                }
            }
            first += 64;
            if (first < cand_end) candidates();
        }
    }

    // the tile goes through LDS, whole rows of it to memory
    barrier();
    constexpr int E_LD = 64 + 8;
    u16* const Es = reinterpret_cast<u16*>(lds);
    if (!loader) {
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                uint2 v;
                v.x = pack2(acc[x][y][0], acc[x][y][1]);
                v.y = pack2(acc[x][y][2], acc[x][y][3]);
                *reinterpret_cast<uint2*>(Es + (wm * (BM / 2) + x * 16 + l16) * E_LD + wn * 32 + y * 16 + g4 * 4) = v;
            }
    }
    barrier();
    const int c = (tid & 7) * 8;
    const int64_t col = n0 + c;
#pragma unroll
    for (int it = 0; it < BM / 64; ++it) {
        const int rr = (tid >> 3) + 64 * it;
        const int64_t row = m0 + rr;
        if (row < m_own) continue;
        const uint4 v = *reinterpret_cast<const uint4*>(Es + rr * E_LD + c);
        u16* const out = g.C + row * g.ldc + col;
        if (col >= n_own) {
            __builtin_memcpy(out, &v, 16);
        } else {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (col + e >= n_own) out[e] = (u16)(w[e >> 1] >> (16 * (e & 1)));
        }
    }
}

template <bool FWD, int BM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(BM == 64 ? 4 : 2))) void whole_tile_kernel(GenGemmArgs g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[3 * kWholeStage<BM>];      // two steps and a pass
    whole_tile_body<FWD, BM>(g, lds, blockIdx.y * gridDim.x + blockIdx.x);
}

// Tile: KC = 1: 64 x 64, KC = 4: 32 x 32; four wavefronts 2 x 2, each 2 x 2 blocks or one.
// A step is KC chunks of 128 bytes per row (64 elements).  LDS rows of operands whose contraction is contiguous are padded to 144 bytes
// (16-byte reads of 16 rows then touch every bank once); a W / B_i tile [contraction][column] is XOR-swizzled in 32-byte units for the
// transposing read.
// Forward: B operand (W, B_i) has its columns contiguous; backward (W, A_i transposed): its contraction.
// Order of the sum, in both tiles and both loops below (the tile follows from the number of tokens, and a row's bits must not): one chain of
// MFMAs over groups of 32 elements that start at multiples of that, zero-filled at the end, in ascending order, then each adapter's term.
template <bool FWD, int KC> constexpr int kGenGemmLds = 2 * KC * (KC == 1 ? 64 : 32) * (144 + (FWD ? 128 : 144));      // bytes of LDS
template <bool FWD, int KC>
__device__ __forceinline__ void general_gemm_body(const GenGemmArgs& g, unsigned char* const lds, const uint32_t wg) {
    typedef u16 T;
    constexpr int BT = KC == 1 ? 64 : 32;                    // tile edge
    if (wg >= (uint32_t)((g.M + BT - 1) / BT * g.tiles_n)) return;      // (a launch of two dimensions holds more)
    constexpr int NB = BT / 32;                              // blocks of a wavefront, each way
    constexpr int KW = 128 / (int)sizeof(T), KT = KW * KC;   // contraction per chunk and per step
    constexpr int EPC = kEpc<T>;
    constexpr int CPK = 8 * KC;                              // 16-byte pieces of a contraction row
    constexpr int NCH = BT * CPK / 256;                      // pieces per thread and operand
    constexpr int CPN = BT / EPC;                            // pieces of a column row (fwd W tile)
    constexpr int A_TILE = KC * BT * 144;
    constexpr int NC_PITCH = BT * 2;
    constexpr int B_TILE = FWD ? KT * NC_PITCH : A_TILE;
    constexpr int STAGE = A_TILE + B_TILE;
    static_assert(2 * STAGE == kGenGemmLds<FWD, KC>);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, g4 = lane >> 4;
    // The last tile of rows / columns starts early enough to be whole (its loads then need no conditions); what it shares with
    // the tile before is not stored.
    const int64_t m_own = (int64_t)(wg / g.tiles_n) * BT, n_own = (int64_t)(wg % g.tiles_n) * BT;
    const int64_t m0 = max((int64_t)0, min(m_own, g.M - BT)), n0 = max((int64_t)0, min(n_own, g.N - BT));
    auto unit = [](int k, int u) {      // swizzled 32-byte unit of a bf16 W row
        return BT == 64 ? u ^ (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) : u ^ ((k >> 3) & 1);
    };

    auto lds_off = [&](int idx) {        // where piece idx of an operand whose contraction is contiguous goes
        const int row = idx / CPK, cc = idx % CPK;
        return ((cc >> 3) * BT + row) * 144 + (cc & 7) * 16;
    };
    auto store_piece = [&](int stage, int idx, uint4 a, uint4 b) {
        unsigned char* As = lds + stage * STAGE;
        unsigned char* Bs = As + A_TILE;
        *reinterpret_cast<uint4*>(As + lds_off(idx)) = a;
        if (FWD) {
            const int kr = idx / CPN, cn = idx % CPN;
            *reinterpret_cast<uint4*>(Bs + kr * NC_PITCH + ((unit(kr, cn >> 1) << 5) | ((cn & 1) << 4))) = b;
        } else {
            *reinterpret_cast<uint4*>(Bs + lds_off(idx)) = b;
        }
    };
    struct Frags { uint4 a[2][NB], b[2][NB]; };          // [64-byte half of the chunk][block]
    auto read_frags = [&](Frags (&fr)[KC], int stage) {
        const unsigned char* As = lds + stage * STAGE;
        const unsigned char* Bs = As + A_TILE;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    Frags& f = fr[kc];
                    f.a[h][x] = *reinterpret_cast<const uint4*>(As + (kc * BT + (wm * NB + x) * 16 + l16) * 144 + h * 64 + g4 * 16);
                    if (!FWD) {
                        f.b[h][x] = *reinterpret_cast<const uint4*>(Bs + (kc * BT + (wn * NB + x) * 16 + l16) * 144 + h * 64 + g4 * 16);
                    } else {
                        const int k = kc * KW + h * 32 + 8 * g4 + (l16 >> 2);
                        const unsigned char* p = Bs + k * NC_PITCH + (unit(k, wn * NB + x) << 5) + (l16 & 3) * 8;
                        f.b[h][x] = __builtin_bit_cast(uint4, lds_read_frag_tr(reinterpret_cast<const u16*>(p), reinterpret_cast<const u16*>(p + 4 * NC_PITCH)));
                    }
                }
    };
    // operands swapped: a lane holds one output row and 4 consecutive columns of each block
    using Acc = f32x4[NB][NB];
    auto clear = [&](Acc& acc) {
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto multiply = [&](Acc& acc, const Frags (&fr)[KC]) {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < NB; ++x)
#pragma unroll
                    for (int y = 0; y < NB; ++y) acc[x][y] = block_mma<T>(fr[kc].b[h][y], fr[kc].a[h][x], acc[x][y]);
    };

    // acc += A B over a contraction of K.  Element (row m0 + i, c) of A at a[i * lda + c], rows [row_lo, row_hi) exist; column
    // n0 + j, element c of B at b[c * ldb + j] (fwd) or b[j * ldb + c] (bwd).  Any sizes, one step at a time: for short contractions.
    auto contract_any = [&](Acc& acc, const T* a, int64_t lda, int64_t row_lo, int64_t row_hi, const T* b, int64_t ldb, int64_t K) {
        for (int64_t k0 = 0; k0 < K; k0 += KT) {
            const int left = (int)min((int64_t)KT, K - k0);
            uint4 ra[NCH], rb[NCH];
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const int idx = tid + 256 * c, row = idx / CPK, k = (idx % CPK) * EPC;
                ra[c] = load16<T>(a + row * lda + k0 + k, m0 + row >= row_lo && m0 + row < row_hi ? min(EPC, left - k) : 0);
                if (FWD) {
                    const int kr = idx / CPN, col = (idx % CPN) * EPC;
                    rb[c] = load16<T>(b + (k0 + kr) * ldb + col, kr < left ? (int)max((int64_t)0, min((int64_t)EPC, g.N - n0 - col)) : 0);
                } else {
                    rb[c] = load16<T>(b + row * ldb + k0 + k, n0 + row < g.N ? min(EPC, left - k) : 0);
                }
            }
            __syncthreads();                             // whoever read the stage before is done
#pragma unroll
            for (int c = 0; c < NCH; ++c) store_piece(0, tid + 256 * c, ra[c], rb[c]);
            __syncthreads();
            Frags f[KC];
            read_frags(f, 0);
            multiply(acc, f);
        }
    };

    // The same for whole tiles and at least one whole step: every load is inside its rows and takes no condition.  Step t travels
    // in register set t & 1 and LDS stage t & 1 (loads past the last step fetch it again); products may
    // be scheduled across the barrier.  What is left of a contraction that is not a multiple of the step is one more, zero-filled step: a piece that
    // reaches past the end is loaded from where it still fits into its row and shifted into place.
    auto contract_whole = [&](Acc& acc, const T* a, int64_t lda, const T* b, int64_t ldb, int64_t K) {
        uint4 ra[2][NCH], rb[2][NCH];
        const T *pa[NCH], *pb[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int idx = tid + 256 * c, row = idx / CPK, k = (idx % CPK) * EPC;
            pa[c] = a + row * lda + k;
            pb[c] = FWD ? b + (idx / CPN) * ldb + (idx % CPN) * EPC : b + row * ldb + k;
        }
        const int64_t nt = K / KT;
        auto load_step = [&](int64_t step, int set) {
            const int64_t k0 = min(step, nt - 1) * KT;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                __builtin_memcpy(&ra[set][c], pa[c] + k0, 16);
                __builtin_memcpy(&rb[set][c], pb[c] + (FWD ? k0 * ldb : k0), 16);
            }
        };
        auto store = [&](int stage, const uint4 (&va)[NCH], const uint4 (&vb)[NCH]) {
#pragma unroll
            for (int c = 0; c < NCH; ++c) store_piece(stage, tid + 256 * c, va[c], vb[c]);
        };
        Frags f[KC];
        load_step(0, 0);
        load_step(1, 1);
        store(0, ra[0], rb[0]);
        load_step(2, 0);
        __syncthreads();
        int64_t t = 0;
        auto two_steps = [&]() {
            store(1, ra[1], rb[1]);
            load_step(t + 3, 1);
            read_frags(f, 0);
            __builtin_amdgcn_sched_barrier(0);           // all reads are on their way before the first product
            multiply(acc, f);
            __syncthreads();
            store(0, ra[0], rb[0]);
            load_step(t + 4, 0);
            read_frags(f, 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(acc, f);
            __syncthreads();
            t += 2;
        };
        while (t + 1 < nt) two_steps();
        if (t < nt) {
            read_frags(f, 0);
            multiply(acc, f);
        }
        const int left = (int)(K - nt * KT);
        if (left > 0) {
            int miss[NCH];                               // elements by which a piece of this step reaches past the end
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const int idx = tid + 256 * c, k = (idx % CPK) * EPC, kr = idx / CPN;
                miss[c] = max(0, k + EPC - left);
                __builtin_memcpy(&ra[0][c], pa[c] + nt * KT - miss[c], 16);
                if (FWD) __builtin_memcpy(&rb[0][c], pb[c] + (nt * KT - max(0, kr + 1 - left)) * ldb, 16);
                else     __builtin_memcpy(&rb[0][c], pb[c] + nt * KT - miss[c], 16);
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                ra[0][c] = drop_front(ra[0][c], miss[c]);
                rb[0][c] = FWD ? ((tid + 256 * c) / CPN < left ? rb[0][c] : zero4()) : drop_front(rb[0][c], miss[c]);
            }
            __syncthreads();                             // the fragments of stage 0 have been read
            store(0, ra[0], rb[0]);
            __syncthreads();
            read_frags(f, 0);
            multiply(acc, f);
        }
    };

    Acc acc;
    bool owned[NB] = {};
    clear(acc);
    // lane l holds the metadata of candidate adapter first + l of this row tile; fetched ahead of the contraction that hides it
    Entry4 tile{0, 0, 0, 0};
    if (g.lora) {
        tile = g.pv.gemm_tiles[m0 / kGemmTileRows];
        tile.d = g.pv.gemm_tiles[(min(g.M, m0 + BT) - 1) / kGemmTileRows].d;      // an early last tile may reach into the next
    }
    int first = tile.c;
    int c_rank = 0, c_off = 0, c_end = 0;
    int64_t c_so = 0;
    uint64_t c_f = 0;
    float c_sc = 1.0f;
    auto candidates = [&]() {
        const int cand = min(first + lane, tile.d - 1);
        c_rank = g.pv.rank[cand]; c_off = g.pv.off[cand]; c_end = g.pv.off[cand + 1];
        c_so = g.pv.soff[cand];
        c_f = reinterpret_cast<uint64_t>(FWD ? g.pv.ptrs[cand].B : g.pv.ptrs[cand].A);
        if (FWD) c_sc = g.pv.scale[cand];
    };
    if (first < tile.d) candidates();

    if (g.base) {
        const T* w = FWD ? g.W + n0 : g.W + n0 * g.ldw;
        if (g.M >= BT && g.N >= BT && g.K >= KT) contract_whole(acc, g.A + m0 * g.lda, g.lda, w, g.ldw, g.K);
        else contract_any(acc, g.A + m0 * g.lda, g.lda, m0, g.M, w, g.ldw, g.K);
    }

    // rank extension, adapter by adapter into a second accumulator set, of which the adapter's own rows are added: another
    // adapter's operands never touch a row, whatever they hold
    const int lo_t = (int)m0, hi_t = (int)min(g.M, m0 + BT);
    while (first < tile.d) {
        uint64_t todo = __ballot(first + lane < tile.d && c_rank > 0 && max(c_off, lo_t) < min(c_end, hi_t));
        while (todo) {
            const int l = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            auto lane64 = [&](uint64_t v) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)v, l);
            };
            const int r = __builtin_amdgcn_readlane(c_rank, l), seg0 = __builtin_amdgcn_readlane(c_off, l);
            const int lo = max(seg0, lo_t), hi = min(__builtin_amdgcn_readlane(c_end, l), hi_t);
            const T* F = global_ptr<const T>(reinterpret_cast<const void*>(lane64(c_f)));
            const float s = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c_sc), l));
            Acc ext;
            clear(ext);
            contract_any(ext, g.E + (int64_t)lane64((uint64_t)c_so) + (int64_t)(lo_t - seg0) * r, r, lo, hi, FWD ? F + n0 : F + n0 * r,
                     FWD ? g.N : r, r);
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                const int row = lo_t + (wm * NB + x) * 16 + l16;
                const bool own = row >= lo && row < hi;
                owned[x] = owned[x] || own;
#pragma unroll
                for (int y = 0; y < NB; ++y)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[x][y][q] = own ? acc[x][y][q] + s * ext[x][y][q] : acc[x][y][q];
            }
        }
        first += 64;
        if (first < tile.d) candidates();
    }

#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) {
            const f32x4 v = acc[x][y];
            const int64_t row = m0 + (wm * NB + x) * 16 + l16, col = n0 + (wn * NB + y) * 16 + 4 * g4;
            if (row >= g.M || row < m_own || (!g.base && !owned[x])) continue;
            T* c = g.C + row * g.ldc + col;
            T o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = (g.base || col + q >= g.N) ? from_f32<T>(v[q]) : from_f32<T>(v[q] + to_f32<T>(c[q]));
            if (col >= n_own && col + 4 <= g.N) __builtin_memcpy(c, o, sizeof(o));
            else
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (col + q >= n_own && col + q < g.N) c[q] = o[q];
        }
}

template <bool FWD, int KC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KC == 1 ? 3 : 2))) void general_gemm_kernel(GenGemmArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kGenGemmLds<FWD, KC>];
    general_gemm_body<FWD, KC>(g, lds, blockIdx.y * gridDim.x + blockIdx.x);
}

// The backward product and the weight gradients of a small batch: both need dS alone.  The first `gemm_groups` work groups take the
// tiles of dX, the others a weight-gradient item of 16 ranks each (32 would leave the product fewer work groups a CU).
template <int KC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KC == 1 ? 3 : 2)))
void general_bwd_kernel(GenGemmArgs g, GenWgradArgs<u16> w, uint32_t gemm_groups) {
    static_assert(kGenWgradFloats<1> * 4 <= kGenGemmLds<false, KC>);
    __shared__ __attribute__((aligned(16))) unsigned char lds[kGenGemmLds<false, KC>];
    const uint32_t wg = blockIdx.x;
    if (wg < gemm_groups) {
        general_gemm_body<false, KC>(g, lds, wg);
        return;
    }
    const int item = (int)(wg - gemm_groups), i = item / w.panels % w.pv.N;
    general_wgrad_body<u16, 1, true, 4>(w, reinterpret_cast<float*>(lds), item % w.panels, i, item / w.panels / w.pv.N);
}

// ---- weight gradients --------------------------------------------------------------------------------------------------------------
template <typename T, int NB, bool WHOLE>
__global__ __launch_bounds__(512) void general_wgrad_kernel(GenWgradArgs<T> g) {
    __shared__ float red[kGenWgradFloats<NB>];
    general_wgrad_body<T, NB, WHOLE>(g, red, (int)(blockIdx.z / g.rank_items * gridDim.x + blockIdx.x), blockIdx.y, (int)(blockIdx.z % g.rank_items));
}

// ---- launches --------------------------------------------------------------------------------------------------------------------

// Work groups along x (a multiple of the 8 XCDs where there are more); a dimension of a launch holds fewer than 2^32 work items (2^23 work groups of
// 512), the rest goes along y.  Kernels drop the groups by which the last row of the grid is too long.
constexpr int64_t kGridX = 1 << 20;
dim3 two_dims(int64_t groups) { return dim3((unsigned)(groups < kGridX ? groups : kGridX), (unsigned)((groups + kGridX - 1) / kGridX)); }

template <typename T, bool FWD>
int shrink(mlora_plan* p, const void* src, void* out, hipStream_t st) {
    if (p->n_row_blocks == 0) return MLORA_OK;
    GenShrinkArgs<T> a{};
    a.src = (const T*)src; a.ld = FWD ? p->k : p->n; a.out = (T*)out; a.pv = p->view;
    ProfScope prof(p, FWD ? MLORA_K_SHRINK : MLORA_K_DSHRINK, st);
    const int64_t groups = (int64_t)p->n_row_blocks * 4;
    // Ranks per work group: 16, 64 or all.  With all of them a few row blocks of wide ranks keep a few CUs busy with the whole adapter matrix
    // each; with 16 the rows are read once per 16 ranks (from the caches).  The lines are limits on the work groups in CUs that 295 drawn shapes
    // give (64 .. 8000 tokens, contractions 64 .. 4095; each type and direction): with them a launch takes 3.4 % more than the best of the three
    // on average (by the widest rank alone: 38 %), and at most 1.24 times as long as by the widest rank alone.  us, 16 / 64 / all: forward, bf16
    // 2197 tokens, contraction 769, ranks to 100 - / 13.2 / 10.6, 414, 3076, 24 adapters to 64 15.1 / 12.1 / -, fp32 2814, 3415, rank 128 78 / 55
    // / 49, 333, 4000, rank 128 18.5 / - / 68.6; backward, bf16 1500, 2048, ranks to 33 8.4 / 13.0 / -, fp32 7383, 963, rank 64 28.0 / 26.1 / -.
    auto items = [&](int nb) { return (p->max_rank + 16 * nb - 1) / (16 * nb); };
    const bool wide = p->max_rank > 64;
    const int eighths = sizeof(T) == 4 ? (FWD ? (wide ? 32 : 28) : 48) : (FWD ? (wide ? 16 : 11) : (wide ? 28 : 16));      // of the CUs
    const int one = eighths * p->num_cus / 8;
    const int four = p->num_cus * (FWD ? 2 : 3) / 2;
    const int nb = p->max_rank <= 16 || groups * items(1) <= one ? 1 : !wide || groups * items(4) <= four ? 4 : 8;
    a.rank_items = items(nb);
    // The rank items of 16 rows stand side by side, so that the rows come from the caches, or one after the other.  Work group number modulo 8 is the XCD: with
    // an even number of items the higher ones, empty for most adapters, would all be on the same ones; with ranks that fill them a number of neighbours on an
    // XCD want the same slice of the adapter's matrix, which is worth more as long as the rows' second reading comes from the L2s (32 MB in all).  Side by side's
    // time over apart's in 396 shapes (256 .. 8000 tokens, contractions 520 .. 4095, both directions), fp32 and bf16: even, more than half of the items empty
    // 1.11, 1.07 (8 items to 1.65); even and full 1.02, 1.01 (64 MB, ranks 64 0.91; backward, where a slice is whole lines of B_i, fp32
    // to 12 MB 1.02, 24 to 50 MB 0.98: 2880 tokens, 32 adapters of rank 64, 1320 -> 3952 the step 565 / 571 us); odd and full 1.03, 1.02 (ranks 100, 8 MB 1.14;
    // ranks 33, 33 and 65 MB 0.95, 0.93 of a call); odd, more than half empty 0.98, 0.96 (three items from 0.66).  The rule takes 0.5 % longer than the better of the two, 14 % at worst.
    // Short segments fill the first of a block's four places alone: every fourth work group has rows.  (Turning the places so that these are on all XCDs gained nothing.)
    // With no more than half of the places filled the first ones of all blocks stand together, from ten blocks on.  us a call, side by side / apart / so: fp32 forward
    // 160 tokens, 32 adapters of ranks 16 to 128, contraction 909 27.2 / 28.6 / 21.8, 576, 24, 4 to 33, 2677 23.4 / 23.4 / 17.0; bf16 backward 480, 32, 64, 3279
    // 82.1 / 82.9 / 67.3; not 104, 8, 32, 524 11.7 / 11.8 / 12.3.  495 such calls, over the best of the three: by the rule above fp32 1.04, bf16 1.02, now
    // 1.004 and 1.006, 1.05 and 1.06 at worst.
    int64_t places = 0, all = 0, full = 0;
    for (int32_t i = 0; i < p->N; ++i) {
        const int64_t rows = p->ranks[i] > 0 ? p->off[i + 1] - p->off[i] : 0;
        places += (rows + 15) / 16;
        all += rows * a.rank_items;
        full += rows * ((p->ranks[i] + 16 * nb - 1) / (16 * nb));
    }
    const bool mostly_full = 5 * full >= 3 * all;
    const int64_t bytes = p->T * a.ld * (int64_t)sizeof(T);
    const bool apart = (a.rank_items & 1) == 0 ? bytes < (FWD ? 50000000 : 20000000) || !mostly_full : bytes < 30000000 && mostly_full;
    a.order = a.rank_items > 1 && 2 * places <= groups ? (p->n_row_blocks >= 10 ? 2 : 0) : apart ? 1 : 0;
    const dim3 grid = two_dims(groups * a.rank_items);
    if (nb == 1)      hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 1>), grid, dim3(512), 0, st, a);
    else if (nb == 4) hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 4>), grid, dim3(512), 0, st, a);
    else              hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 8>), grid, dim3(512), 0, st, a);
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

// Whether the weight gradients go with the backward product (one launch less).  A work group of four wavefronts takes twice as long for an item as
// the eight of a launch of its own, so the longest adapter decides: its tokens times the work groups of both in CUs, or a contraction of
// the product twice its tokens.  us a backward call, apart / together, tokens x k x n (longest adapter, work groups of both in CUs): 1500 x 2048 x 1001
// (534, 6.4) 40.0 / 35.3, 256 x 257 x 256 (105, 0.4) 15.2 / 12.0, 1600 x 2048 x 1001 (1600, 3.5) 47.0 / 41.9, 2000 x 100 x 333 (2000, 1.0) 23.0 / 19.2;
// not: 2000 x 1001 x 300 (2000, 2.1) 25.9 / 27.9, 3200 x 300 x 777 (1600, 1.1) 27.4 / 29.5, 6000 x 1001 x 2048 (1617, 10.4) 79.6 / 83.2, 6000 x 1001 x 300
// (1617, 6.4) 39.0 / 42.2, 6000 x 100 x 333 (4241, 0.9) 36.5 / 42.9, 8000 x 1001 x 300 (6444, 8.9) 66.5 / 82.8.  Over 398 shapes a
// call takes 4.0 % more than the better of the two on average (always apart 14.4 %), and at most 4.1 % more than apart; what the limit of ten work groups a CU
// leaves apart would take up to a third less together (127 x 1232 x 553, 24 adapters 45.0 / 29.6).
bool beside_product(const mlora_plan* p, const GenWgradArgs<u16>& w, int64_t groups, int64_t K) {
    const int64_t all = groups + (int64_t)w.panels * p->N * ((p->max_rank + 15) / 16);
    if (all > 10 * p->num_cus) return false;
    int64_t longest = 0;
    for (int32_t i = 0; i < p->N; ++i)
        if (p->ranks[i] > 0) longest = std::max(longest, p->off[i + 1] - p->off[i]);
    return longest <= (p->T <= 2048 ? 2000 : 1500) && (longest * all <= 4000 * p->num_cus || 2 * longest <= K);
}

template <bool FWD>
int gemm(mlora_plan* p, const void* A, const void* W, void* C, const void* E, uint32_t flags, const GenWgradArgs<u16>* w, bool* with_w,
         hipStream_t st) {
    GenGemmArgs a{};
    a.A = (const u16*)A; a.W = (const u16*)W; a.C = (u16*)C; a.E = (const u16*)E;
    a.M = p->T; a.K = FWD ? p->k : p->n; a.N = FWD ? p->n : p->k;
    a.lda = a.K; a.ldw = p->n; a.ldc = a.N; a.R1 = p->R1;
    a.base = (flags & MLORA_FLAG_LORA_ONLY) ? 0 : 1;
    a.lora = ((flags & MLORA_FLAG_BASE_ONLY) || p->n_row_blocks == 0) ? 0 : 1;
    a.pv = p->view;
    if (a.M == 0 || (!a.base && !a.lora)) return MLORA_OK;
    auto tiles = [&](int64_t edge) { return ((a.M + edge - 1) / edge) * ((a.N + edge - 1) / edge); };
    // 32 x 32 tiles where 64 x 64 ones would leave half the chip idle.  us, 32 x 32 / 64 x 64, by the number of 64 x 64 tiles: 20 (256 x 257,
    // contraction 256) 8.4 / 9.6, 72 (500 x 513, 1000) 14.2 / 14.1, 128 (512 x 1024, 1024) 20 / 14, 136 (500 x 1025, 4096) 44 / 31, 176
    // (700 x 1001, 1001) 23 / 15.  The results are the same bit for bit.
    const bool split = tiles(64) <= p->num_cus / 2;
    a.tiles_n = (a.N + (split ? 31 : 63)) / (split ? 32 : 64);
    const int64_t groups = tiles(split ? 32 : 64);
    const bool beside = !FWD && w && beside_product(p, *w, groups, a.K);
    ProfScope prof(p, FWD ? MLORA_K_GEMM_FWD : beside ? MLORA_K_GEMM_BWD_WGRAD : MLORA_K_GEMM_BWD, st);
    if constexpr (!FWD) {
        if (beside) {
            GenWgradArgs<u16> b = *w;
            b.rank_items = (uint32_t)((p->max_rank + 15) / 16);
            const dim3 grid((unsigned)(groups + (int64_t)b.panels * p->N * b.rank_items));
            if (split) hipLaunchKernelGGL((general_bwd_kernel<4>), grid, dim3(256), 0, st, a, b, (uint32_t)groups);
            else       hipLaunchKernelGGL((general_bwd_kernel<1>), grid, dim3(256), 0, st, a, b, (uint32_t)groups);
            *with_w = true;
            MLORA_HIP_TRY(hipGetLastError());
            return MLORA_OK;
        }
    }
    // Whole tiles of 128 rows, 64 columns and a contraction of 64 or more where that makes one round, two work groups a CU, or the contraction has two steps
    // and as many as its tiles have passes of the rank extension: of the others' work groups three or four share a CU and hide each other's beginnings and passes.
    // us, others / whole, tokens x outputs x contraction (rounds; passes a tile): forward 1500 x 1001 x 300 (0.8; 1.2) 17.4 / 15.8, 600 x 2001 x 130 (0.6; 4.8)
    // 22.9 / 18.6, 8000 x 2048 x 65 (7.8; 1.1) 0.93 of whole's time, 2000 x 2048 x 129 (2; 1.2) 1.10, 2000 x 2048 x 129 and 193 (2; 3.1) 0.98, 333 1.10.
    const double steps = (double)a.K / 64;
    auto passes = [&](int log_rows) {                    // of the rank extension, a tile of that many rows on average
        int64_t sum = 0;
        for (int32_t i = 0; a.lora && i < p->N; ++i)
            if (p->off[i + 1] > p->off[i]) sum += (((p->off[i + 1] - 1) >> log_rows) - (p->off[i] >> log_rows) + 1) * ((p->ranks[i] + 63) >> 6);
        return (double)sum / (double)(((a.M - 1) >> log_rows) + 1);
    };
    const bool pieces = !a.lora || a.R1 >= 8;            // (what a tile reads of E at least)
    if (!split && a.base && a.M >= 128 && a.N >= 64 && a.K >= 64 && pieces && (groups <= 2 * p->num_cus || (steps >= 2 && steps >= passes(6)))) {
        // 128 x 64 tiles (forward) by what both take in us: a work group of 128 x 64, alone on its CU, waits for every pass with nothing else to run.  us, 64 x 64 /
        // 128 x 64, tokens x outputs x contraction (passes a tile of 64, 128 rows): 1500 x 1001 x 2048 (1.2, 1.4) 28.9 / 25.4, 4000 x 1001 x 2048 (1.5,
        // 2.0) 52.5 / 49.8, 2000 x 1001 x 700 (3.8, 6.3) 38.0 / 41.2, 2000 x 2001 x 130 (3.1, 5.3) 32.6 / 45.8, 4000 x 1001 x 700 (3.7, 6.4) 55.4 / 65.3;
        // without extension 1500 x 1001 x 300 8.6 / 7.5, 4611 x 4018 x 729 77 / 99, 8000 x 1001 x 700 35.4 / 38.7.  Over 478 forward calls the choice takes
        // 0.5 % longer on average than the best of these and the others (by rounds and steps alone 4.8).  Backward (both operands from rows that start
        // anywhere) 1500 x 2048 x 1001 20.6 / 25.1, 4000 x 2048 x 1001 46.9 / 48.4.
        const int64_t tall = (a.M + 127) / 128 * a.tiles_n;
        auto rounds = [&](int64_t n) { return (double)((n + p->num_cus - 1) / p->num_cus); };
        const bool wide = FWD && rounds(tall) * (3.5 + 0.45 * steps + 0.8 * passes(7)) < 2.5 + rounds(groups) * (0.5 + 0.28 * steps + 0.3 * passes(6));
        const int64_t n = wide ? tall : groups;
        a.xcd_run = n >= 256 ? 32 : (int32_t)((n + 7) / 8);
        const dim3 grid = two_dims((n + 8 * a.xcd_run - 1) / (8 * a.xcd_run) * (8 * a.xcd_run));
        if (wide) hipLaunchKernelGGL((whole_tile_kernel<FWD, FWD ? 128 : 64>), grid, dim3(512), 0, st, a);
        else      hipLaunchKernelGGL((whole_tile_kernel<FWD, 64>), grid, dim3(512), 0, st, a);
    } else if (split) hipLaunchKernelGGL((general_gemm_kernel<FWD, 4>), two_dims(groups), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((general_gemm_kernel<FWD, 1>), two_dims(groups), dim3(256), 0, st, a);
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

// The weight gradients of a batch: the arguments, and the build (16-wide rank blocks per work item; whole panels).
template <typename T> struct GenWgrad { GenWgradArgs<T> args; int nb; bool whole; };
template <typename T>
GenWgrad<T> wgrad_of(mlora_plan* p, const void* dY, const void* X, const void* S, const void* dS, uint32_t flags) {
    GenWgrad<T> w{};
    GenWgradArgs<T>& a = w.args;
    a.X = (const T*)X; a.dY = (const T*)dY; a.S = (const T*)S; a.dS = (const T*)dS;
    a.panels_k = (int32_t)((p->k + 63) / 64);
    a.panels = (int32_t)(a.panels_k + (p->n + 63) / 64);
    a.accumulate = (flags & MLORA_FLAG_ACCUM_GRADS) ? 1 : 0;
    a.pv = p->view;
    // ranks per work item: as many as the plan needs; bf16 keeps each rank element of a lane's eight tokens in a register of its own
    // and would spill with 64, panels that are not whole with more than 16
    w.whole = p->k >= 64 && p->n >= 64;
    w.nb = p->max_rank <= 16 || !w.whole ? 1 : p->max_rank <= 32 || sizeof(T) == 2 ? 2 : 4;
    a.rank_items = (uint32_t)((p->max_rank + 16 * w.nb - 1) / (16 * w.nb));
    return w;
}

template <typename T>
int launch_wgrad(mlora_plan* p, const GenWgrad<T>& w, hipStream_t st) {
    ProfScope prof(p, MLORA_K_WGRAD, st);
    const GenWgradArgs<T>& a = w.args;
    const dim3 xy = two_dims(a.panels), grid(xy.x, (unsigned)p->N, xy.y * a.rank_items), block(512);
    if (!w.whole)       hipLaunchKernelGGL((general_wgrad_kernel<T, 1, false>), grid, block, 0, st, a);
    else if (w.nb == 1) hipLaunchKernelGGL((general_wgrad_kernel<T, 1, true>), grid, block, 0, st, a);
    else if (w.nb == 2) hipLaunchKernelGGL((general_wgrad_kernel<T, 2, true>), grid, block, 0, st, a);
    else if constexpr (sizeof(T) == 4) hipLaunchKernelGGL((general_wgrad_kernel<T, 4, true>), grid, block, 0, st, a);
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

template <typename T>
int fwd_t(mlora_plan* p, const void* X, const void* W, void* Y, void* S, uint32_t flags, hipStream_t st) {
    if (!(flags & MLORA_FLAG_BASE_ONLY)) {
        const int rc = shrink<T, true>(p, X, S, st);
        if (rc != MLORA_OK) return rc;
    }
    if constexpr (sizeof(T) == 4) return f32_gemm(p, true, X, W, Y, S, flags, nullptr, 0, false, nullptr, st);
    else                          return gemm<true>(p, X, W, Y, S, flags, nullptr, nullptr, st);
}

template <typename T>
int bwd_t(mlora_plan* p, const void* dY, const void* X, const void* W, const void* S, void* dX, void* dS, uint32_t flags, hipStream_t st) {
    int rc;
    const bool lora = !(flags & MLORA_FLAG_BASE_ONLY), grads = lora && p->N > 0 && p->max_rank > 0;
    if (lora && (rc = shrink<T, false>(p, dY, dS, st)) != MLORA_OK) return rc;
    const GenWgrad<T> w = wgrad_of<T>(p, dY, X, S, dS, flags);
    bool joined = false;
    const bool may_join = grads && !p->grads_over_A;
    if constexpr (sizeof(T) == 4) rc = f32_gemm(p, false, dY, W, dX, dS, flags, may_join ? &w.args : nullptr, w.nb, w.whole, &joined, st);
    else                          rc = gemm<false>(p, dY, W, dX, dS, flags, may_join && w.whole ? &w.args : nullptr, &joined, st);
    if (rc != MLORA_OK || !grads || joined) return rc;
    return launch_wgrad<T>(p, w, st);
}

}  // namespace

int general_forward(mlora_plan* p, const void* X, const void* W, void* Y, void* S, uint32_t flags, hipStream_t st) {
    return p->dtype == MLORA_F32 ? fwd_t<float>(p, X, W, Y, S, flags, st) : fwd_t<u16>(p, X, W, Y, S, flags, st);
}

int general_backward(mlora_plan* p, const void* dY, const void* X, const void* W, const void* S, void* dX, void* dS, uint32_t flags,
                     hipStream_t st) {
    return p->dtype == MLORA_F32 ? bwd_t<float>(p, dY, X, W, S, dX, dS, flags, st) : bwd_t<u16>(p, dY, X, W, S, dX, dS, flags, st);
}

}  // namespace mlora
