// Fused frozen-weight GEMM + LoRA expand for shapes that give the 256 x 256 kernel too few tiles to fill the chip
// (short batches, narrow projections): Y = X W + s_i S_i B_i and dX = dY W^T + dS_i A_i^T (paper Sec. 5.1 / App. A.1),
// one store of the output, like the large-tile kernel.
//
// With one 256 x 256 tile per CU a layer of 1024 x 4096 outputs keeps 64 of 256 CUs busy for the whole contraction; 128 x 128
// tiles keep all of them busy.  What bounds a CU then is the operand stream: 32 KB per 64-wide step at the 47-51 B/clk its load path takes are
// 640-690 cycles, against 512 of MFMA.  Four wavefronts load (direct global -> LDS loads into rings that fill the LDS, one barrier per step)
// and four multiply, one of each per SIMD: sub-tiles of a quarter of the tile need a third fewer LDS reads than eighths, no MFMA waits behind
// the issue of a load, and the fragments of the next step (128 x 128: half step) are read while one is multiplied.  Cycles per step, eight
// wavefronts that do both / now: 128 x 128 forward 847 / 697, backward 805 / 660; 64 x 128 632 / 500 and 519 / 515; 64 x 64 460 / 343 and 430 / 355
// (without direct loads 128 x 128 takes 690-750: both halves of the work group are near their own limit).  Half as many wavefronts issue a step's loads:
// a contraction of up to eight steps takes 0.2-0.35 us longer (64 x 256, contraction 64 2.7 / 3.0 us, 256 3.1 / 3.45; 300 x 3072, 768 the same).
//
// Order of the sum: every output element is one chain of MFMAs - rank extension, contraction in ascending order, tail - exactly as in
// the 256 x 256 kernel, so that a row has the same bits whichever tile its batch is given: the tile follows from the number of tokens
// of the whole batch, and a job's results must not change when a neighbour joins or leaves it.  That is why the wavefronts (2 x 2 sub-tiles of
// the output) do not share a step's contraction among themselves.
//
// Rank extension: adapter by adapter into the accumulators, of which only the adapter's own rows take the result over (scaled
// in fp32).  Rows of other adapters never reach the result, so no operand has to be masked and a diverged neighbour's Inf / NaN
// stays out of it.  What bounds it is a pass's own chain - operands, fragments, products, selects - since nothing else runs on the CU (three passes
// in flight instead of two were 10 % slower).  us, eight wavefronts / four that waited for fragments per row block / now: 64 x 256, contraction 256, 16
// adapters of rank 64 forward 15.7 / 19.3 / 15.7, backward 16.6 / 14.8 / 13.8, of rank 8 13.7 / 15.2 / 13.8, 14.0 / 12.5 / 12.2; 48 adapters of rank 33 in 300
// x 256 forward 18.8 / 19.4 / 19.1, backward with the weight gradients 26.7 / 25.4 / 18.4; 128 x 128 tiles of 2000 x 2048, contraction 512, 64 adapters of
// rank 33 22.0 / 22.0 / 23.0, 16 of rank 128 15.2 / 16.5 / 15.9.
//
// us, 256 x 256 tiles / eight wavefronts that load and multiply / now: 1024 x 14336 x 4096 forward - / 112 / 102, its weight from HBM 133 / 121; 1024 x
// 4096 x 4096 forward with eight adapters, with its shrink, - / 46.0 / 43.5; 200 x 512, k = 2048: 67 / 9.2 / 8.1.
#include <type_traits>

#include "mfma_wgrad.h"

namespace mlora {

namespace {

constexpr int SG_THREADS = 512;
constexpr int SG_LDS = 163840;

template <int N> __device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Stages of the two rings, operand tiles of 64-wide steps: the rows (X / dY, which the shrink has just read) and the weight, which comes from further away
template <int BM, int BN> constexpr int kStagesA = BN == 64 ? 5 : BM == 64 ? 4 : 3;
template <int BM, int BN> constexpr int kStagesB = (SG_LDS - kStagesA<BM, BN> * BM * 128) / (BN * 128);
template <int BM, int BN> constexpr int kRing = kStagesA<BM, BN> * BM * 128 + kStagesB<BM, BN> * BN * 128;      // bytes of LDS

// The weight gradients of a batch that fills the chip with neither go with the backward product: both need dS alone and run side by side, the
// first `gemm_groups` work groups on the tiles of dX, the others on two weight-gradient items each (four wavefronts an item).
template <int MAXNB> struct Beside { WgradArgs w; int32_t gemm_groups, items; };
template <> struct Beside<0> {};
template <int MAXNB> constexpr int kItem = 2 * (WX_TILE + WT * MAXNB * 32);      // elements of LDS an item takes
template <int MAXNB>
__device__ __forceinline__ void two_items(const Beside<MAXNB>& b, unsigned char* lds) {
    const WgradArgs& w = b.w;
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int panels = w.panels_k + w.panels_n;
    const int item = 2 * (int)(blockIdx.x - b.gemm_groups) + half, other = item ^ 1;
    const Entry4 none{0, 0, 0, 0};
    const Entry4 e = item < b.items ? w.pv.wgrad_chunks[w.chunk_base + item / panels] : none;
    const Entry4 o = other < b.items ? w.pv.wgrad_chunks[w.chunk_base + other / panels] : none;
    const int steps = max(wgrad_steps(e), wgrad_steps(o));           // both halves pass the same barriers
    if (item >= b.items) {
        for (int t = 0; t <= steps; ++t) __syncthreads();
        return;
    }
    u16* mine = reinterpret_cast<u16*>(lds) + half * kItem<MAXNB>;
    const int panel = item % panels, tid = threadIdx.x & 255;
    if (panel < w.panels_k) wgrad_body<MAXNB, true, 4, true>(w, mine, tid, e, panel, steps);
    else                    wgrad_body<MAXNB, false, 4, true>(w, mine, tid, e, panel - w.panels_k, steps);
}

// MAXNB > 0: with weight gradients, built for that many 32-wide rank blocks.  (The product stands in the kernel itself: as a function that two kernels
// call it took 1-3 % longer, 149 x 256 x 12288 backward 73.9 -> 75.8 us.)
template <bool NN, int BM, int BN, int MAXNB = 0>
__global__ __launch_bounds__(SG_THREADS) void small_gemm_kernel(GemmArgs g, Beside<MAXNB> beside) {
    constexpr int LDS = MAXNB > 0 && 4 * kItem<MAXNB> > kRing<BM, BN> ? 4 * kItem<MAXNB> : kRing<BM, BN>;
    static_assert(LDS <= SG_LDS, "two items fit");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS];
    if constexpr (MAXNB > 0) {
        if ((int)blockIdx.x >= beside.gemm_groups) {
            two_items(beside, lds);
            return;
        }
    }
    constexpr int AT = BM * 128, BT = BN * 128;                    // bytes: operand tiles of one 64-wide step
    constexpr int NSA = kStagesA<BM, BN>, NSB = kStagesB<BM, BN>;  // ring stages
    constexpr int B0 = NSA * AT;                                   // where the weight's ring starts
    constexpr int HELD = 2 + (2 * AT + BT - 1) / BT;               // weight stages that the passes of the rank extension use first: two of each operand
    auto pass_a = [](int slot) { return B0 + (NSB - 2) * BT - (slot + 1) * AT; };
    auto pass_b = [](int slot) { return B0 + (NSB - 1 - slot) * BT; };
    constexpr int NA = BM / 32, NB_ = BN / 32;                     // direct loads per multiplying wavefront and pass (rank extension, tail)
    constexpr int WTM = BM / 2, WTN = BN / 2;                      // sub-tile of a multiplying wavefront
    constexpr int MB = WTM / 16, NB = WTN / 16;
    constexpr int BROW = BN * 2;                                   // NN: bytes per contraction row of the weight tile
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave >= 4;       // wavefronts 4 .. 7 load (4, 5 the rows, 6, 7 the weight), 0 .. 3 multiply
    const int wm = (wave >> 1) & 1, wn = wave & 1;
    const int l16 = lane & 15, g4 = lane >> 4;

    // Tile order: bands of 8 row tiles x all column tiles, numbered down the rows first; every XCD (blockIdx % 8) takes runs of
    // `xcd_run` consecutive tiles, which share operand panels in its L2.  At most 32 (its CUs), fewer if that is what spreads a
    // launch of less than 256 tiles over all eight.
    const int total = g.tiles_m * g.tiles_n;
    const int xcd = blockIdx.x % 8, slot_x = blockIdx.x / 8;
    const int L = ((slot_x / g.xcd_run) * 8 + xcd) * g.xcd_run + slot_x % g.xcd_run;
    if (L >= total) return;
    const int per_band = 8 * g.tiles_n;
    const int band = L / per_band, in_band = L - band * per_band;
    const int band_rows = min(8, g.tiles_m - band * 8);
    const int tm = band * 8 + in_band % band_rows, tn = in_band / band_rows;
    const int m0 = tm * BM, n0 = tn * BN;

    // swizzle key of contraction row k of the NN weight tile
    auto fkey = [](int k) { return BN == 128 ? nn_swz(k) : (((k >> 1) & 1) | (((k >> 3) & 1) << 1)); };

    // ---- direct loads ---------------------------------------------------------------------------
    const int nk = g.Kdim / 64;
    const unsigned lds0 = (unsigned)(uintptr_t)lds;
    constexpr int LPR = BROW / 16;       // NN: lanes of a contraction row
    constexpr int CA = BM / 8, CB = BN / 8;          // pieces of 1 KB, a load each, of a step's tiles

    // ---- fragments and MFMAs ----------------------------------------------------------------------
    f32x4 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Register sets: what is multiplied and what is read meanwhile, U 32-wide halves of a step each (128 x 128: one, or they would spill)
    constexpr int U = MB * NB < 16 ? 2 : 1;
    static_assert(U == 2 || MB == NB, "a row block and a column block with each group of products");
    bf16x8 fa[2][U][MB], fb[2][U][NB];
    const int a_off = (wm * WTM + l16) * 128, bnt_off = (wn * WTN + l16) * 128;
    const int vq = fkey(8 * g4 + (l16 >> 2));
    const int bnn_off = (8 * g4 + (l16 >> 2)) * BROW + (l16 & 3) * 8;
    auto frag_a = [&](int at, int h, int a) {
        return lds_read_frag(reinterpret_cast<const u16*>(lds + at + a_off + (((h * 4 + g4) ^ (l16 & 7)) << 4) + a * 2048));
    };
    auto frag_b = [&](int at, int h, int b) {
        const unsigned char* Bs = lds + at;
        if (NN) {
            const unsigned char* p = Bs + bnn_off + h * 32 * BROW + (((wn * NB + b) ^ vq) << 5);
            return lds_read_frag_tr(reinterpret_cast<const u16*>(p), reinterpret_cast<const u16*>(p + 4 * BROW));
        }
        return lds_read_frag(reinterpret_cast<const u16*>(Bs + bnt_off + (((h * 4 + g4) ^ (l16 & 7)) << 4) + b * 2048));
    };
    // fragment i of a set that starts with half h0 of the step in slots slot_a, slot_b, in the order the products want them
    constexpr int NF = U * (MB + NB);
    auto read_frag = [&](int slot_a, int slot_b, int h0, int set, int i) {
        const int u = i / (MB + NB), j = i % (MB + NB);
        if (j < NB) fb[set][u][j] = frag_b(B0 + slot_b * BT, h0 + u, j);
        else        fa[set][u][j - NB] = frag_a(slot_a * AT, h0 + u, j - NB);
    };
    int sa = 0, sb = 0;                  // slots of the step that is read
    auto read_set = [&](int h0, int set) {
#pragma unroll
        for (int f = 0; f < NF; ++f) read_frag(sa, sb, h0, set, f);
    };
    // The products of register set `set`; with `read` the next set's fragments are read meanwhile, most of them early.  Operands swapped: a
    // lane ends with one output row and 4 consecutive columns of each 16 x 16 block.
    auto multiply = [&](auto set_, bool read, int h0) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value;
#pragma unroll
        for (int i = 0; i < U * MB; ++i) {
            const int u = i / MB, a = i % MB;
            constexpr int G = U * MB > 4 ? U * MB - 2 : U * MB - 1;            // U = 2: groups of products that the reads go with
            __builtin_amdgcn_sched_barrier(0);
            if (read && U == 1) {                        // a row block and a column block with each group
                read_frag(sa, sb, h0, set ^ 1, NB + a);
                read_frag(sa, sb, h0, set ^ 1, a);
            } else if (read) {
#pragma unroll
                for (int f = i * NF / G; f < (i + 1) * NF / G && f < NF; ++f) read_frag(sa, sb, h0, set ^ 1, f);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b] = mfma16(fb[set][u][b], fa[set][u][a], acc[a][b]);
            if (read) {
                for (int x = 0; x < NB; ++x) {
                    if (U == 1) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, (NN ? 2 : 1) * (MB == 2 && NB == 2 ? 2 : 1), 0);
                    if (U == 2) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    const std::integral_constant<int, 0> zero{};
    const std::integral_constant<int, 1> one{};
    // ---- passes: at most 64 contraction elements that are not a whole step (rank extension, tail) ----
    // Pieces of rows outside [lo, hi) alone and chunks past kc are not loaded: what stands there is dropped or taken as zero (take_pass); the other
    // rows outside repeat the first or last one inside and columns past the edge the last ones.  Element (row t, c) of the row operand at a[(t - lo) a_ld + c],
    // of the weight's at b[c b_ld + col] (NN) or b[(col - n0) b_ld + c].
    auto dma_pass = [&](int slot, const void* a, int64_t a_ld, int lo, int hi, const void* b, int64_t b_ld, int kc) {
        const char* ab = uniform_ptr(a);
        const char* bb = uniform_ptr(b);
        const unsigned dst_a = lds0 + pass_a(slot), dst_b = lds0 + pass_b(slot);
#pragma unroll
        for (int c = 0; c < NB_; ++c) {                  // (first: of many lines)
            const int kb = wave * NB_ + c;
            unsigned v;
            if (NN) {
                if (kb * (64 / LPR) >= kc) continue;             // (uniform; kc is a multiple of 8: a piece is there or not)
                const int k = kb * (64 / LPR) + lane / LPR, pos = lane % LPR;
                const int chunk = (((pos >> 1) ^ fkey(k)) << 1) | (pos & 1);
                v = (unsigned)((int64_t)k * b_ld + min(n0 + chunk * 8, g.Ncols - 8)) * 2u;
                dma16(v, bb, dst_b + kb * 1024);
            } else {
                const int row = kb * 8 + (lane >> 3), ch = (lane & 7) ^ (lane >> 3);
                v = (unsigned)((int64_t)(min(n0 + row, g.Ncols - 1) - n0) * b_ld + ch * 8) * 2u;
                if (ch * 8 < kc) dma16(v, bb, dst_b + kb * 1024);
            }
        }
#pragma unroll
        for (int c = 0; c < NA; ++c) {
            const int row0 = m0 + (wave * NA + c) * 8, ch = (lane & 7) ^ (lane >> 3);
            if (row0 >= hi || row0 + 8 <= lo) continue;          // (uniform)
            const unsigned v = (unsigned)((int64_t)(min(max(row0 + (lane >> 3), lo), hi - 1) - lo) * a_ld + ch * 8) * 2u;
            if (ch * 8 < kc) dma16(v, ab, dst_a + (wave * NA + c) * 1024);
        }
    };
    // The same for rows of r elements that start anywhere (ranks that are no multiples of 8): elements r0 .. r0 + kc - 1 of each, through registers, loaded while
    // the pass before is multiplied.  A piece that would reach past its row is loaded from where it still fits (ranks below 8: past its buffer, which then
    // has a piece; else element by element) and shifted.
    constexpr int PT = SG_THREADS / 2;                   // the multiplying wavefronts' threads
    uint4 pa[NA], pb[NB_];
    int ea[NA], eb[NB_];                                 // elements to drop in front
    auto any_piece = [&](const u16* row, int r, int at, const u16* end, bool whole, int& drop) {
        uint4 v;
        if (whole) {
            const u16* const from = r >= 8 ? row + min(at, r - 8) : min(row, end - 8);
            drop = (int)(r >= 8 ? row + at - from : row - from);
            __builtin_memcpy(&v, from, 16);
        } else {
            drop = 0;
            v = load_chunk(row, r, false);
        }
        return v;
    };
    auto load_pass = [&](const u16* e, int lo, int hi, const u16* F, int r, int r0, int kc) {
        const bool whole = r >= 8 || g.R1 >= 8;
#pragma unroll
        for (int c = 0; c < NA; ++c) {
            const int idx = tid + PT * c, t = min(max(m0 + (idx & (BM - 1)), lo), hi - 1), cc = idx / BM;
            if (c >= NA / 2 && kc <= 32) continue;
            pa[c] = any_piece(e + (int64_t)(t - lo) * r, r, r0 + cc * 8, g.E + g.R1, whole, ea[c]);
        }
#pragma unroll
        for (int c = 0; c < NB_; ++c) {
            const int idx = tid + PT * c;
            if (c >= NB_ / 2 && kc <= 32) continue;
            if (NN) {
                const int k = idx / (BN / 8), gcol = min(n0 + (idx % (BN / 8)) * 8, g.Ncols - 8);
                pb[c] = *reinterpret_cast<const uint4*>(F + (int64_t)(r0 + min(k, kc - 1)) * g.Ncols + gcol);
            } else {
                pb[c] = any_piece(F + (int64_t)min(n0 + (idx & (BN - 1)), g.Ncols - 1) * r, r, r0 + idx / BN * 8, F + (int64_t)g.Ncols * r, true, eb[c]);
            }
        }
    };
    auto store_pass = [&](int slot, int r, int r0, int kc) {
        unsigned char* const Pa = lds + pass_a(slot);
        unsigned char* const Pb = lds + pass_b(slot);
        auto store = [&](auto in_place) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < NA; ++c) {
                const int idx = tid + PT * c, row = idx & (BM - 1), cc = idx / BM;
                if (c >= NA / 2 && kc <= 32) continue;
                *reinterpret_cast<uint4*>(Pa + row * 128 + ((cc ^ (row & 7)) << 4)) = in_place(pa[c], ea[c], r0 + cc * 8);
            }
#pragma unroll
            for (int c = 0; c < NB_; ++c) {
                const int idx = tid + PT * c;
                if (c >= NB_ / 2 && kc <= 32) continue;
                if (NN) {
                    const int k = idx / (BN / 8), nc = idx % (BN / 8);
                    *reinterpret_cast<uint4*>(Pb + k * BROW + ((((nc >> 1) ^ fkey(k)) << 5) | ((nc & 1) << 4))) = k < kc ? pb[c] : zero4();
                } else {
                    const int row = idx & (BN - 1), cc = idx / BN;
                    *reinterpret_cast<uint4*>(Pb + row * 128 + ((cc ^ (row & 7)) << 4)) = in_place(pb[c], eb[c], r0 + cc * 8);
                }
            }
        };
        if (r >= 8) store([](uint4 v, int drop, int) { return drop_front(v, drop); });
        else        store([&](uint4 v, int drop, int at) { return keep_front(drop_front(v, drop), r - at); });
    };
    // rows [lo, hi) of the accumulators take the products of the pass in `slot`, then times f.  A half's fragments (128 x 128; else both halves') are read
    // before its first product and there are no branches: with a wait per row block a pass took 1000 cycles more, and 300 more with the number of halves
    // decided behind the first one's reads.
    auto take_pass = [&](int slot, int kc, int lo, int hi, float f) {
        const bf16x8 z = __builtin_bit_cast(bf16x8, zero4());
        auto halves = [&](auto count, int h0, float times) __attribute__((always_inline)) {
            constexpr int H = decltype(count)::value;
#pragma unroll
            for (int h = 0; h < H; ++h) {
#pragma unroll
                for (int b = 0; b < NB; ++b) fb[h][0][b] = frag_b(pass_b(slot), h0 + h, b);
#pragma unroll
                for (int a = 0; a < MB; ++a) fa[h][0][a] = frag_a(pass_a(slot), h0 + h, a);
            }
            const bool in = (h0 + H - 1) * 32 + 8 * g4 < kc;     // (the first of two halves is whole)
#pragma unroll
            for (int b = 0; b < NB; ++b) fb[H - 1][0][b] = in ? fb[H - 1][0][b] : z;
#pragma unroll
            for (int a = 0; a < MB; ++a) fa[H - 1][0][a] = in ? fa[H - 1][0][a] : z;
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                const int row0 = m0 + wm * WTM + a * 16, row = row0 + l16;
                if (MB == 4 && (row0 >= hi || row0 + 16 <= lo)) continue;        // (uniform; a pass of few rows has most of its time in the selects below)
                const bool own = row >= lo && row < hi;
                f32x4 t[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) t[b] = mfma16(fb[0][0][b], fa[0][0][a], acc[a][b]);
                if (H == 2) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) t[b] = mfma16(fb[H - 1][0][b], fa[H - 1][0][a], t[b]);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[a][b][q] = own ? times * t[b][q] : acc[a][b][q];
            }
        };
        const std::integral_constant<int, 1> single{};
        if constexpr (MB * NB == 16) {                   // (registers for one half)
            for (int h = 0; h * 32 < kc; ++h) halves(single, h, h * 32 + 32 >= kc ? f : 1.0f);
        } else {
            if (kc > 32) halves(std::integral_constant<int, 2>{}, 0, f);
            else         halves(single, 0, f);
        }
    };

    int first = 0, cand_end = g.pv.N;    // candidate adapters of the tile
    // (up to 64 adapters are all candidates: one round trip less than by way of the row-tile table)
    if (!g.skip_lora && cand_end > 64) {
        const Entry4 tile = g.pv.gemm_tiles[m0 / kGemmTileRows];
        first = tile.c; cand_end = tile.d;
    }
    uint32_t* const count = reinterpret_cast<uint32_t*>(lds + pass_a(1));     // free until the second pass is asked for

    // ---- the loading wavefronts ---------------------------------------------------------------------
    // Wavefronts 4 and 5 load the rows.  The weight's lines are the same for the row tiles of a band, on one XCD: asked for by all of them at once, a
    // line that is not in its L2 yet is fetched for each.  So each of 8, 4 or 2 row tiles asks for its share of the lines early (wavefront 6)
    // and for the others' when they are there (wavefront 7).  One copy of the loads for filling the rings and for the steady state: what a
    // launch of few steps executes is short.
    if (loader) {
        constexpr int D_REST = (NSB + 1) / 2;        // steps ahead
        const bool rows = wave < 6;
        // piece kb at byte min(kb stride + at, last) of the step's tile (at0 or at1 by its swizzle); rows past the edge repeat the last one
        const int64_t ld = rows ? g.lda : g.ldb;
        unsigned at0, at1, last, stride;
        if (rows || !NN) {
            const unsigned ch = ((lane & 7) ^ (lane >> 3)) * 16;
            stride = (unsigned)ld * 16u;
            at0 = at1 = (unsigned)(lane >> 3) * (unsigned)ld * 2u + ch;
            last = (unsigned)((rows ? min(g.M - m0, BM) - 1 : min(g.Ncols - n0, BN) - 1) * ld * 2) + ch;
        } else {
            const int k = lane / LPR, pos = lane % LPR;
            stride = (unsigned)(64 / LPR * ld * 2);
            auto column = [&](int key) { return min(n0 + ((((pos >> 1) ^ key) << 1) | (pos & 1)) * 8, g.Ncols - 8); };
            at0 = (unsigned)(k * ld + column(fkey(k))) * 2u;
            at1 = (unsigned)(k * ld + column(fkey(k + 8))) * 2u;
            last = ~0u;
        }
        const char* base = uniform_ptr(rows ? g.Aop + (int64_t)m0 * g.lda : NN ? g.Bop : g.Bop + (int64_t)n0 * g.ldb);
        const int64_t lstep = !rows && NN ? (int64_t)64 * g.ldb * 2 : 128;
        // NUM loads a step, piece(c) the c-th; D steps ahead in a ring of NS, FREE of them before the rank extension is through
        auto run = [&](auto num, auto ahead, auto stages, auto held, auto piece) __attribute__((always_inline)) {
            constexpr int NUM = decltype(num)::value, D = decltype(ahead)::value, NS = decltype(stages)::value, FREE = NS - decltype(held)::value;
            static_assert(NUM * D < 64 && D <= NS && D <= 16 && D > 1, "vmcnt holds 6 bits; drain steps");
            int slot = 0;
            bool extended = g.skip_lora != 0;
            auto extension = [&]() __attribute__((always_inline)) {      // passes the barriers of the multiplying wavefronts' passes
                extended = true;
                for (int f = first; f < cand_end; f += 64) {
                    lds_barrier();
                    const int passes = __builtin_amdgcn_readfirstlane((int)*count);
                    for (int q = 0; q <= passes; ++q) lds_barrier();
                }
            };
            for (int t = 0; t < nk; ++t) {
                if (t == FREE && !extended) extension();
                if (t >= D) {
                    if (!extended) extension();
                    wait_loads_and_barrier<NUM * (D - 2)>();             // step t - D + 1 has landed, step t - D has been read
                    if (t == D) lds_barrier();
                }
                const unsigned dst = lds0 + (rows ? slot * AT : B0 + slot * BT);
#pragma unroll
                for (int c = 0; c < NUM; ++c) {
                    const int kb = piece(c);
                    const bool odd = NN && !rows && (BN == 128 ? (kb >> 1) & 1 : kb & 1);
                    dma16(min((unsigned)kb * stride + (odd ? at1 : at0), last), base, dst + kb * 1024);
                }
                base += lstep;
                slot = slot == NS - 1 ? 0 : slot + 1;
            }
            if (!extended) extension();
            // the last steps, or all of a short contraction: nothing left to load
            if (nk == D) wait_loads_and_barrier<NUM * (D - 1)>();
#define SG_DRAIN(J) if (J + 1 < D && J + 1 + nk >= D) wait_loads_and_barrier<(D - 2 - J > 0 ? D - 2 - J : 0) * NUM>();
            SG_DRAIN(0) SG_DRAIN(1) SG_DRAIN(2) SG_DRAIN(3) SG_DRAIN(4) SG_DRAIN(5) SG_DRAIN(6) SG_DRAIN(7)
            SG_DRAIN(8) SG_DRAIN(9) SG_DRAIN(10) SG_DRAIN(11) SG_DRAIN(12) SG_DRAIN(13) SG_DRAIN(14)
#undef SG_DRAIN
        };
        const int tm_in = in_band % band_rows;
        auto share = [&](auto p) __attribute__((always_inline)) {
            constexpr int P = decltype(p)::value, OWN = CB / P, REST = CB - OWN;
            const int own = tm_in & (P - 1);
            const std::integral_constant<int, NSB> ring{};
            const std::integral_constant<int, HELD> held{};
            if (wave == 6) run(std::integral_constant<int, OWN>{}, std::integral_constant<int, (NSB * OWN < 64 ? NSB : 63 / OWN)>{}, ring, held, [=](int c) { return c * P + own; });
            else           run(std::integral_constant<int, REST>{}, std::integral_constant<int, D_REST>{}, ring, held, [=](int c) { return c / (P - 1) * P + ((own + 1 + c % (P - 1)) & (P - 1)); });
        };
        if (nk == 0) {
            for (int f = first; f < cand_end && !g.skip_lora; f += 64) {
                lds_barrier();
                const int passes = __builtin_amdgcn_readfirstlane((int)*count);
                for (int q = 0; q <= passes; ++q) lds_barrier();
            }
        } else if (rows) {
            run(std::integral_constant<int, CA / 2>{}, std::integral_constant<int, NSA>{}, std::integral_constant<int, NSA>{}, std::integral_constant<int, 0>{}, [=](int c) { return (wave & 1) * (CA / 2) + c; });
        } else if (band_rows >= 8) {
            share(std::integral_constant<int, 8>{});
        } else if (band_rows >= 4) {
            share(std::integral_constant<int, 4>{});
        } else {
            share(std::integral_constant<int, 2>{});
        }
    }

    // ---- rank extension -----------------------------------------------------------------------------
    // Lane l holds the metadata of candidate adapter first + l, so that walking the adapters of a tile costs no memory round trips; the operands of
    // the next pass are on their way while one is multiplied.  An adapter's own rows hold zero before its passes and nothing but its
    // term after them; what its operands give in other rows is dropped, whatever they hold.
    if (!g.skip_lora && !loader) {
        const int m_end = min(g.M, m0 + BM);
        for (; first < cand_end; first += 64) {
            const int cand = min(first + lane, cand_end - 1);
            const int v_rank = g.pv.rank[cand], v_off = g.pv.off[cand], v_end = g.pv.off[cand + 1];
            const int64_t v_so = g.pv.soff[cand];
            const uint64_t v_f = reinterpret_cast<uint64_t>(NN ? g.pv.ptrs[cand].B : g.pv.ptrs[cand].A);
            const float v_sc = NN ? g.pv.scale[cand] : 1.0f;
            const bool mine = first + lane < cand_end && v_rank > 0 && max(v_off, m0) < min(v_end, m_end);
            uint64_t todo = __ballot(mine);
            const int passes = __popcll(todo) + __popcll(__ballot(mine && v_rank > 64));
            auto lane64 = [](uint64_t v, int l) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)v, l);
            };
            int r0 = 0;                            // ranks of the lowest adapter in todo that have been asked for
            int lo = 0, hi = 0, kc = 0, pr = 0, pr0 = 0;         // of the pass asked for last; rank of its adapter and first of its ranks
            bool staged = false;                   // it comes through registers
            float f = 1.0f;
            auto request = [&](int slot) {
                const int l = (int)__builtin_ctzll(todo);
                const int r = __builtin_amdgcn_readlane(v_rank, l), seg0 = __builtin_amdgcn_readlane(v_off, l);
                lo = max(seg0, m0);
                hi = min(__builtin_amdgcn_readlane(v_end, l), m_end);
                kc = min(64, r - r0);
                const int64_t so = (int64_t)lane64((uint64_t)v_so, l);
                const u16* F = global_ptr<const u16>(reinterpret_cast<const void*>(lane64(v_f, l)));
                const u16* e = g.E + so + (int64_t)(lo - seg0) * r;
                pr = r; pr0 = r0;
                staged = (r & 7) != 0 || (so & 7) != 0;
                if (staged) load_pass(e, lo, hi, F, r, r0, kc);
                else        dma_pass(slot, e + r0, r, lo, hi, NN ? F + (int64_t)r0 * g.Ncols : F + (int64_t)n0 * r + r0, NN ? g.Ncols : r, kc);
                const bool last = r0 + 64 >= r;
                f = last ? __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v_sc), l)) : 1.0f;
                if (last) { todo &= todo - 1; r0 = 0; }
                else r0 += 64;
            };
            if (todo) request(0);
            if (passes > 0 && staged) store_pass(0, pr, pr0, kc);
            if (tid == 0) *count = (uint32_t)passes;
            lds_barrier();                         // the loading wavefronts read it
            for (int q = 0; q < passes; ++q) {
                const int slot = q & 1, p_lo = lo, p_hi = hi, p_kc = kc;
                const float p_f = f;
                wait_loads_and_barrier<0>();       // pass q is here, everybody is done with pass q - 1
                if (todo) request(slot ^ 1);
                if (MB * NB == 16 && q + 1 < passes && staged) store_pass(slot ^ 1, pr, pr0, kc);      // (not enough registers to multiply meanwhile)
                take_pass(slot, p_kc, p_lo, p_hi, p_f);
                if (MB * NB < 16 && q + 1 < passes && staged) store_pass(slot ^ 1, pr, pr0, kc);
            }
            lds_barrier();                         // the passes have been read
        }
    }

    // ---- contraction over the frozen weight -----------------------------------------------------------
    // Step t starts with the fragments of its first half in registers: the second half's are read while the first is multiplied.  Then
    // stage t + 1 has landed and everybody has read stage t (its slots are free); the first half of t + 1 is
    // read while the second of t is multiplied.
    if (nk > 0 && !loader) {
        lds_barrier();
        read_set(0, 0);
        auto next = [&]() __attribute__((always_inline)) {      // stage t + 1 has landed, everybody has read stage t
            lds_barrier();
            sa = sa == NSA - 1 ? 0 : sa + 1;
            sb = sb == NSB - 1 ? 0 : sb + 1;
        };
        if constexpr (U == 2) {
            int t = 0;
            for (; t + 2 < nk; t += 2) {
                next();
                multiply(zero, true, 0);
                next();
                multiply(one, true, 0);
            }
            if (t + 1 < nk) {
                next();
                multiply(zero, true, 0);
                multiply(one, false, 0);
            } else {
                multiply(zero, false, 0);
            }
        } else {
            for (int t = 0; t < nk - 1; ++t) {
                multiply(zero, true, 1);
                next();
                multiply(one, true, 0);
            }
            multiply(zero, true, 1);
            multiply(one, false, 0);
        }
    }

    // ---- tail of a contraction that is not a multiple of 64 (it is one of 8) -----------------------------
    if ((g.Kdim & 63) != 0) {
        const int k0 = nk * 64;
        lds_barrier();
        if (!loader) dma_pass(0, g.Aop + (int64_t)m0 * g.lda + k0, g.lda, m0, min(g.M, m0 + BM), NN ? g.Bop + (int64_t)k0 * g.ldb : g.Bop + (int64_t)n0 * g.ldb + k0,
                              g.ldb, g.Kdim - k0);
        wait_loads_and_barrier<0>();
        if (!loader) take_pass(0, g.Kdim - k0, m0, g.M, 1.0f);
    }

    // ---- the tile goes through LDS, whole rows of it to memory ----------------------------------------
    lds_barrier();
    constexpr int E_LD = BN + 8;
    static_assert(BM * E_LD * 2 <= kRing<BM, BN>, "epilogue staging fits the ring");
    u16* Es = reinterpret_cast<u16*>(lds);
    if (!loader) {
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                uint2 v;
                v.x = pack2hw(acc[a][b][0], acc[a][b][1]);
                v.y = pack2hw(acc[a][b][2], acc[a][b][3]);
                *reinterpret_cast<uint2*>(Es + (wm * WTM + a * 16 + l16) * E_LD + wn * WTN + b * 16 + g4 * 4) = v;
            }
    }
    lds_barrier();
    constexpr int CPR = BN / 8;
#pragma unroll
    for (int it = 0; it < BM * CPR / SG_THREADS; ++it) {
        const int idx = tid + SG_THREADS * it, rr = idx / CPR, c = idx % CPR;
        const int row = m0 + rr, col = n0 + c * 8;
        if (row >= g.M || col >= g.Ncols) continue;   // Ncols is a multiple of 8: chunks are all-in or all-out
        store_streaming(g.C + (int64_t)row * g.ldc + col, *reinterpret_cast<const uint4*>(Es + rr * E_LD + c * 8));
    }
}

}  // namespace

// `w` (backward only, may be null): the weight-gradient items that run beside the product, `items` of them, built for max_nb 32-wide rank blocks
template <int BM, int BN>
static void launch_small(GemmArgs g, bool fwd, const WgradArgs* w, int items, int max_nb, hipStream_t st) {
    g.tiles_m = (g.M + BM - 1) / BM;
    g.tiles_n = (g.Ncols + BN - 1) / BN;
    const int total = g.tiles_m * g.tiles_n;
    g.xcd_run = total >= 256 ? 32 : (total + 7) / 8;
    const int per = 8 * g.xcd_run, grid = (total + per - 1) / per * per;
    if (w) {
        const dim3 both(grid + (items + 1) / 2);
        if (max_nb == 1) hipLaunchKernelGGL((small_gemm_kernel<false, BM, BN, 1>), both, dim3(SG_THREADS), 0, st, g, (Beside<1>{*w, grid, items}));
        else             hipLaunchKernelGGL((small_gemm_kernel<false, BM, BN, 2>), both, dim3(SG_THREADS), 0, st, g, (Beside<2>{*w, grid, items}));
    } else if (fwd) {
        hipLaunchKernelGGL((small_gemm_kernel<true, BM, BN>), dim3(grid), dim3(SG_THREADS), 0, st, g, Beside<0>{});
    } else {
        hipLaunchKernelGGL((small_gemm_kernel<false, BM, BN>), dim3(grid), dim3(SG_THREADS), 0, st, g, Beside<0>{});
    }
}

// Which kernel a product of M x N outputs over a contraction of K takes: -1 the 256 x 256 one, else an index of the table.
// Every kernel runs one work group per CU, so a launch takes  launch + rounds x (fill and epilogue + steps x step)  with
// rounds = tiles over CUs, rounded up.  The step times are what the kernels sustain with all CUs busy (64-wide step; the
// 256 x 256 kernel moves the fewest bytes per product and wins wherever its last round is not too empty).  They are those of the kernel before
// its wavefronts were divided: with what it sustains now (0.44, 0.275, 0.175) more products went to small tiles, which does not fit launches that
// leave CUs to the 256 x 256 kernel's clock (2249 x 3840 x 8448 206 -> 232 us, 2927 tokens through an 8B block 2.51 -> 2.83 ms).  Over 192 products of the
// present kernels (64 .. 16384 tokens, widths 512 .. 14336, both directions) the choice takes 0.4 % longer on average than the best of the four, 10 % at
// worst (8192 x 1000 x 1096 backward 34.2 / 37.8).  Measured (us, launches timed singly, about 5 of them the events': 256 x 256 / 128 x 128 / 64 x 128 / 64 x 64, tokens
// x outputs x contraction, forward): 1000 x 4096 x 4096  82 / 37 / 47 / 65;  1000 x 1024 x 4096  81 / 30 / 23 / 20;  200 x 512 x 2048  67 / 24 / 16 / 13.5;
// 4000 x 4096 x 4096  103 / 128 / 164 / 230.
int small_gemm_tile(int64_t M, int64_t N, int64_t K, int num_cus) {
    struct { int bm, bn; double launch, round, step; } const tab[4] = {
        {256, 256, 3.0, 4.5, 1.45}, {128, 128, 4.0, 2.5, 0.48}, {64, 128, 4.0, 2.0, 0.32}, {64, 64, 3.5, 2.0, 0.225}};
    int best = 0;
    double best_us = 0;
    for (int i = 0; i < 4; ++i) {
        const int64_t tiles = ((M + tab[i].bm - 1) / tab[i].bm) * ((N + tab[i].bn - 1) / tab[i].bn);
        const double us = tab[i].launch + (double)((tiles + num_cus - 1) / num_cus) * (tab[i].round + (double)((K + 63) / 64) * tab[i].step);
        if (i == 0 || us < best_us) { best = i; best_us = us; }
    }
    return best - 1;
}

void launch_small_gemm(int tile, const GemmArgs& g, bool fwd, const WgradArgs* w, int items, int max_nb, hipStream_t st) {
    if (tile == 0)      launch_small<128, 128>(g, fwd, w, items, max_nb, st);
    else if (tile == 1) launch_small<64, 128>(g, fwd, w, items, max_nb, st);
    else                launch_small<64, 64>(g, fwd, w, items, max_nb, st);
}

}  // namespace mlora
