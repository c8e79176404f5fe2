// The general kernels: fp32 plans, and bf16 plans whose k or n is not a multiple of 8 (rows that start at any element).
// Every step of the layer (paper Sec. 5.1) is one grouped launch on the matrix units, with fp32 accumulation:
//   S_i = X_i A_i, dS_i = s_i dY_i B_i^T               general_shrink_kernel
//   Y = X W + s_i S_i B_i, dX = dY W^T + dS_i A_i^T    general_gemm_kernel in bf16 (also either term alone); fp32: f32_gemm.hip
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
// tokens, 256 x 256: 171 -> 21 us; fp32, 2048 tokens, 2048 x 2048: 1590 -> 265 us; bf16, 1500 tokens, 2048 x 1001: 1105 -> 67 us.
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
    PlanView pv;
};

template <typename T, bool FWD, int NB>
__global__ __launch_bounds__(512) void general_shrink_kernel(GenShrinkArgs<T> g) {
    constexpr int NW = 8;
    constexpr int RLD = NB * 16 + 4;
    __shared__ float red[NW * 16 * RLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    // The rank items of 16 rows stand side by side, so that the rows come from the caches; but not where there are 2, 4 or 8 of them: work group
    // number modulo 8 is the XCD, and the higher items, empty for most adapters, would all be on the same ones.  us, fp32, 2048 tokens, contraction
    // 2048, ranks 8 to 64 (4 items): side by side 19.0 forward, 23.5 backward, one item after the other 14.0, 18.4; in turned order 19.8, 24.7.  bf16, 1500
    // tokens, contraction 2048, ranks to 33 (3 items): 6.0 and 7.7, 8.1 and 8.2.
    const int64_t item = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, groups = (int64_t)g.pv.n_row_blocks * 4;
    if (item >= groups * g.rank_items) return;
    const bool apart = (g.rank_items & 1) == 0;
    const int64_t wg = apart ? item % groups : item / g.rank_items;
    const Entry4 e = g.pv.row_blocks[wg >> 2];
    const int sub = (wg & 3) * 16, rows = min(16, e.d - sub);
    if (rows <= 0) return;
    const int i = e.a, row0 = e.c + sub;
    const int r = g.pv.rank[i], rho0 = (int)(apart ? item / groups : item % g.rank_items) * (16 * NB), rl = min(r - rho0, 16 * NB);      // this work group's ranks
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
    int32_t base, lora;           // which terms; without the base term C += LoRA term
    PlanView pv;
};

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
            auto drop = [&](uint4 v, int d) {            // the piece without its first d elements, zeros behind it
                uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
                const int sh = min(d * (int)sizeof(T) * 8, 128);
                const uint64_t up = sh == 0 ? lo : sh < 64 ? (lo >> sh) | (hi << (64 - sh)) : sh < 128 ? hi >> (sh - 64) : 0;
                hi = sh < 64 ? hi >> sh : 0;
                return make_uint4((uint32_t)up, (uint32_t)(up >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
            };
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
                ra[0][c] = drop(ra[0][c], miss[c]);
                rb[0][c] = FWD ? ((tid + 256 * c) / CPN < left ? rb[0][c] : zero4()) : drop(rb[0][c], miss[c]);
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
    general_gemm_body<FWD, KC>(g, lds, blockIdx.x);
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

// Work groups along x; a dimension of a launch holds fewer than 2^32 work items (2^23 work groups of 512), the rest goes along y.
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
    const dim3 grid = two_dims(groups * a.rank_items);
    if (nb == 1)      hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 1>), grid, dim3(512), 0, st, a);
    else if (nb == 4) hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 4>), grid, dim3(512), 0, st, a);
    else              hipLaunchKernelGGL((general_shrink_kernel<T, FWD, 8>), grid, dim3(512), 0, st, a);
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

// Whether the weight gradients go with the backward product (one launch less).  A work group of four wavefronts takes twice as long for an item as
// the eight of a launch of its own, so the longest adapter decides: its tokens times the work groups of both in CUs, or a contraction of
// the product twice its tokens.  us a step, apart / together, tokens x k x n (longest adapter, work groups of both in CUs): 1500 x 2048 x 1001
// (about 400, 6.4) 74.2 / 67.3, 256 x 257 x 256 (100, 0.4) 27.8 / 24.1, 1024 x 1001 x 3000 (60, 8.9) 79 / 70.6, 6000 x 1001 x 2048 (1000, 7.4) 154.5 /
// 149.7, 6000 x 300 x 777 (1000, 2.7) 77.3 / 74.0, 2000 x 100 x 333 (2000, 1.0) 35.9 / 30.6; not: 2000 x 1001 x 300 (2000, 2.1) 45.9 / 46.9,
// 6000 x 1001 x 300 (1000, 6.9) 73.1 / 77.4, 6000 x 100 x 333 (3000, 1.0) 56.0 / 60.1, 8000 x 1001 x 300 (4000, 8.5) 98.9 / 120.5.  Over 150 drawn
// shapes a backward call takes 2.8 % more than the better of the two on average (always apart 18.3 %), and at most 2.8 % more than apart.
bool beside_product(const mlora_plan* p, const GenWgradArgs<u16>& w, int64_t groups, int64_t K) {
    const int64_t all = groups + (int64_t)w.panels * p->N * ((p->max_rank + 15) / 16);
    if (all > 10 * p->num_cus) return false;
    int64_t longest = 0;
    for (int32_t i = 0; i < p->N; ++i)
        if (p->ranks[i] > 0) longest = std::max(longest, p->off[i + 1] - p->off[i]);
    return longest <= 2000 && (longest * all <= 4000 * p->num_cus || 2 * longest <= K);
}

template <bool FWD>
int gemm(mlora_plan* p, const void* A, const void* W, void* C, const void* E, uint32_t flags, const GenWgradArgs<u16>* w, bool* with_w,
         hipStream_t st) {
    GenGemmArgs a{};
    a.A = (const u16*)A; a.W = (const u16*)W; a.C = (u16*)C; a.E = (const u16*)E;
    a.M = p->T; a.K = FWD ? p->k : p->n; a.N = FWD ? p->n : p->k;
    a.lda = a.K; a.ldw = p->n; a.ldc = a.N;
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
    if (split) hipLaunchKernelGGL((general_gemm_kernel<FWD, 4>), dim3((unsigned)groups), dim3(256), 0, st, a);
    else       hipLaunchKernelGGL((general_gemm_kernel<FWD, 1>), dim3((unsigned)groups), dim3(256), 0, st, a);
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
