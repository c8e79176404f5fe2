// Fused frozen-weight GEMM + LoRA expand for shapes that give the 256 x 256 kernel too few tiles to fill the chip
// (short batches, narrow projections): Y = X W + s_i S_i B_i and dX = dY W^T + dS_i A_i^T (paper Sec. 5.1 / App. A.1),
// one store of the output, like the large-tile kernel.
//
// With one 256 x 256 tile per CU a layer of 1024 x 4096 outputs keeps 64 of 256 CUs busy for the whole contraction; 128 x 128
// tiles keep all of them busy.  What bounds a CU then is the operand stream (32 KB per 64-wide step against 512 cycles of MFMA)
// and, before that, latency, so the tiles come by direct global -> LDS loads into a ring that fills the LDS (all but the
// current step in flight, one barrier per step) and the fragments of each 32-wide half step are read while the one before it is
// multiplied.
//
// Order of the sum: every output element is one chain of MFMAs - rank extension, contraction in ascending order, tail - exactly as in
// the 256 x 256 kernel, so that a row has the same bits whichever tile its batch is given: the tile follows from the number of tokens
// of the whole batch, and a job's results must not change when a neighbour joins or leaves it.  That is why the 8 wavefronts
// (2 x 4 sub-tiles of the output, two per SIMD) do not share a step's contraction among themselves; with 2 x 2 sub-tiles and the
// two halves of a step summed apart the LDS reads per MFMA were a third fewer; over 190 products the mean time moved by -2.5 %
// (128 x 128), 0 (64 x 128) and +5 % (64 x 64).
//
// Rank extension: adapter by adapter into a second accumulator set, of which the adapter's own rows are then taken over (scaled
// in fp32).  Rows of other adapters never reach the result, so no operand has to be masked and a diverged neighbour's Inf / NaN
// stays out of it.
//
// 1000 x 4096 outputs, k = 4096: 85 us with 256 x 256 tiles, 40 with 128 x 128; 200 x 512, k = 2048: 67 and, with 64 x 64, 14.  A
// 128 x 128 work group spends about 0.5 us per step with all CUs busy (32 KB of operands at the 45-50 B/clk a CU's load path takes
// are 0.3), where the MFMAs alone would take 0.21.
#include "mfma_wgrad.h"

namespace mlora {

namespace {

constexpr int SG_THREADS = 512;
constexpr int SG_LDS = 163840;

template <int N> __device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// bytes of LDS: ring stages of the operand tiles of one 64-wide step
template <int BM, int BN> constexpr int kStages = SG_LDS / ((BM + BN) * 128) < 8 ? SG_LDS / ((BM + BN) * 128) : 8;
template <int BM, int BN> constexpr int kRing = kStages<BM, BN> * (BM + BN) * 128;

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
    constexpr int AT = BM * 128, BT = BN * 128, STAGE = AT + BT;   // bytes: operand tiles of one 64-wide step
    constexpr int NST = kStages<BM, BN>;                           // ring stages
    constexpr int NA = BM / 64, NB_ = BN / 64, LPS = NA + NB_;     // direct loads per wavefront and step
    constexpr int WTM = BM / 2, WTN = BN / 4;                      // sub-tile of a wavefront
    constexpr int MB = WTM / 16, NB = WTN / 16;
    constexpr int BROW = BN * 2;                                   // NN: bytes per contraction row of the weight tile
    static_assert(LPS * (NST - 2) < 64, "vmcnt holds 6 bits");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
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
    unsigned oa[NA], ob[NB_];
#pragma unroll
    for (int c = 0; c < NA; ++c) {
        const int row = (wave * NA + c) * 8 + (lane >> 3), ch = (lane & 7) ^ (lane >> 3);
        oa[c] = (unsigned)((int64_t)(min(m0 + row, g.M - 1) - m0) * g.lda + ch * 8) * 2u;
    }
#pragma unroll
    for (int c = 0; c < NB_; ++c) {
        const int kb = wave * NB_ + c;
        if (NN) {
            constexpr int LPR = BROW / 16;
            const int k = kb * (64 / LPR) + lane / LPR, pos = lane % LPR;
            const int chunk = (((pos >> 1) ^ fkey(k)) << 1) | (pos & 1);
            ob[c] = (unsigned)((int64_t)k * g.ldb + min(n0 + chunk * 8, g.Ncols - 8)) * 2u;
        } else {
            const int row = kb * 8 + (lane >> 3), ch = (lane & 7) ^ (lane >> 3);
            ob[c] = (unsigned)((int64_t)(min(n0 + row, g.Ncols - 1) - n0) * g.ldb + ch * 8) * 2u;
        }
    }
    const char* baseA = uniform_ptr(g.Aop + (int64_t)m0 * g.lda);
    const char* baseB = NN ? uniform_ptr(g.Bop) : uniform_ptr(g.Bop + (int64_t)n0 * g.ldb);
    const int64_t bstep = NN ? (int64_t)64 * g.ldb * 2 : 128;
    const unsigned lds0 = (unsigned)(uintptr_t)lds;
    int slot_in = 0;
    auto issue1 = [&](int c) {           // load c (of LPS) of the next step's tiles into the next ring slot
        const unsigned dst = lds0 + slot_in * STAGE;
        if (c < NA) dma16(oa[c < NA ? c : 0], baseA, dst + (wave * NA + c) * 1024);
        else        dma16(ob[c < NA ? 0 : c - NA], baseB, dst + AT + (wave * NB_ + c - NA) * 1024);
        if (c == LPS - 1) {
            baseA += 128; baseB += bstep;
            slot_in = slot_in == NST - 1 ? 0 : slot_in + 1;
        }
    };
    auto issue = [&]() {
#pragma unroll
        for (int c = 0; c < LPS; ++c) issue1(c);
    };
    // all slots but the last, which the rank extension uses first
    const int early = min(nk, NST - 1);
    for (int t = 0; t < early; ++t) issue();

    // ---- fragments and MFMAs ----------------------------------------------------------------------
    f32x4 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 fa[2][MB], fb[2][NB];
    // a step is two 32-wide halves h; the fragments of one are read while the other is multiplied
    const int a_off = (wm * WTM + l16) * 128, bnt_off = (wn * WTN + l16) * 128;
    const int vq = fkey(8 * g4 + (l16 >> 2));
    const int bnn_off = (8 * g4 + (l16 >> 2)) * BROW + (l16 & 3) * 8;
    auto read_frag_a = [&](int slot, int h, int a) {
        fa[h][a] = lds_read_frag(reinterpret_cast<const u16*>(lds + slot * STAGE + a_off + (((h * 4 + g4) ^ (l16 & 7)) << 4) + a * 2048));
    };
    auto read_frag_b = [&](int slot, int h, int b) {
        const unsigned char* Bs = lds + slot * STAGE + AT;
        if (NN) {
            const unsigned char* p = Bs + bnn_off + h * 32 * BROW + (((wn * NB + b) ^ vq) << 5);
            fb[h][b] = lds_read_frag_tr(reinterpret_cast<const u16*>(p), reinterpret_cast<const u16*>(p + 4 * BROW));
        } else {
            fb[h][b] = lds_read_frag(reinterpret_cast<const u16*>(Bs + bnt_off + (((h * 4 + g4) ^ (l16 & 7)) << 4) + b * 2048));
        }
    };
    auto read_frags = [&](int slot, int h) {
#pragma unroll
        for (int a = 0; a < MB; ++a) read_frag_a(slot, h, a);
#pragma unroll
        for (int b = 0; b < NB; ++b) read_frag_b(slot, h, b);
    };
    // ask the scheduler to alternate a group's LDS reads with its MFMAs
    auto interleave = [&]() {
        for (int i = 0; i < NB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, NB == 1 ? 3 : 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // operands swapped: a lane ends with one output row and 4 consecutive columns of each 16 x 16 block
    auto mma = [&](f32x4 (&c)[MB][NB], int h) {
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) c[a][b] = mfma16(fb[h][b], fa[h][a], c[a][b]);
    };

    // Operands that are not whole aligned 64-wide steps (rank extension, tail of the contraction) go through registers into the
    // last slot, zero-filled up to a multiple of 32 in the contraction.
    unsigned char* const Ps = lds + (NST - 1) * STAGE;
    uint4 pa[NA], pb[NB_];
    auto pass_load = [&](const u16* a_src, int64_t a_ld, int a_lo, int a_hi, bool a_vec, const u16* b_src, int64_t b_ld, bool b_vec,
                         int kc) {                  // a_src: row a_lo
#pragma unroll
        for (int c = 0; c < NA; ++c) {
            const int idx = tid + SG_THREADS * c, t = m0 + (idx & (BM - 1)), cc = idx / BM;
            pa[c] = zero4();
            if (t >= a_lo && t < a_hi && cc * 8 < kc) pa[c] = load_chunk(a_src + (int64_t)(t - a_lo) * a_ld + cc * 8, min(8, kc - cc * 8), a_vec);
        }
#pragma unroll
        for (int c = 0; c < NB_; ++c) {
            const int idx = tid + SG_THREADS * c;
            pb[c] = zero4();
            if (NN) {
                const int k = idx / (BN / 8), gcol = n0 + (idx % (BN / 8)) * 8;
                if (k < kc && gcol < g.Ncols) pb[c] = *reinterpret_cast<const uint4*>(b_src + (int64_t)k * b_ld + gcol);
            } else {
                const int gcol = n0 + (idx & (BN - 1)), cc = idx / BN;
                if (gcol < g.Ncols && cc * 8 < kc) pb[c] = load_chunk(b_src + (int64_t)gcol * b_ld + cc * 8, min(8, kc - cc * 8), b_vec);
            }
        }
    };
    auto pass_store = [&](int kc) {
        const int kpad = (kc + 31) & ~31;
#pragma unroll
        for (int c = 0; c < NA; ++c) {
            const int idx = tid + SG_THREADS * c, row = idx & (BM - 1), cc = idx / BM;
            if (cc * 8 < kpad) *reinterpret_cast<uint4*>(Ps + row * 128 + ((cc ^ (row & 7)) << 4)) = pa[c];
        }
#pragma unroll
        for (int c = 0; c < NB_; ++c) {
            const int idx = tid + SG_THREADS * c;
            if (NN) {
                const int k = idx / (BN / 8), nc = idx % (BN / 8);
                if (k < kpad) *reinterpret_cast<uint4*>(Ps + AT + k * BROW + ((((nc >> 1) ^ fkey(k)) << 5) | ((nc & 1) << 4))) = pb[c];
            } else {
                const int row = idx & (BN - 1), cc = idx / BN;
                if (cc * 8 < kpad) *reinterpret_cast<uint4*>(Ps + AT + row * 128 + ((cc ^ (row & 7)) << 4)) = pb[c];
            }
        }
    };

    // ---- rank extension -----------------------------------------------------------------------------
    // Lane l holds the metadata of candidate adapter base + l, so that walking the adapters of a tile costs no memory round
    // trips; the operands of the next pass are in flight while one is multiplied.
    if (!g.skip_lora) {
        const Entry4 tile = g.pv.gemm_tiles[m0 / kGemmTileRows];
        const int m_end = min(g.M, m0 + BM);
        for (int base = tile.c; base < tile.d; base += 64) {
            const int cand = min(base + lane, tile.d - 1);
            const int v_rank = g.pv.rank[cand], v_off = g.pv.off[cand], v_end = g.pv.off[cand + 1];
            const int64_t v_so = g.pv.soff[cand];
            const uint64_t v_f = reinterpret_cast<uint64_t>(NN ? g.pv.ptrs[cand].B : g.pv.ptrs[cand].A);
            const float v_sc = NN ? g.pv.scale[cand] : 1.0f;
            uint64_t todo = __ballot(base + lane < tile.d && v_rank > 0 && max(v_off, m0) < min(v_end, m_end));
            if (todo == 0) continue;
            auto lane64 = [](uint64_t v, int l) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)v, l);
            };
            int l = 0, r = 0, lo = 0, hi = 0, r0 = 0;
            auto load_next = [&]() {               // operands of pass (adapter lane l, ranks from r0)
                const int seg0 = __builtin_amdgcn_readlane(v_off, l);
                r = __builtin_amdgcn_readlane(v_rank, l);
                lo = max(seg0, m0);
                hi = min(__builtin_amdgcn_readlane(v_end, l), m_end);
                const int64_t so = (int64_t)lane64((uint64_t)v_so, l);
                const u16* F = global_ptr<const u16>(reinterpret_cast<const void*>(lane64(v_f, l)));
                const u16* e = g.E + so + (int64_t)(lo - seg0) * r + r0;
                const bool vec = (r & 7) == 0, e_vec = vec && (so & 7) == 0;
                if (NN) pass_load(e, r, lo, hi, e_vec, F + (int64_t)r0 * g.Ncols, g.Ncols, true, min(64, r - r0));
                else    pass_load(e, r, lo, hi, e_vec, F + r0, r, vec, min(64, r - r0));
            };
            l = (int)__builtin_ctzll(todo);
            load_next();
            bool first = true;
            f32x4 ext[MB][NB];
            for (;;) {
                const int kc = min(64, r - r0), c_lo = lo, c_hi = hi;
                const float sc = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v_sc), l));
                if (r0 == 0) {
#pragma unroll
                    for (int a = 0; a < MB; ++a)
#pragma unroll
                        for (int b = 0; b < NB; ++b) ext[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                if (!first || base != tile.c) lds_barrier();      // the previous pass has been read
                first = false;
                pass_store(kc);
                const bool last_of_adapter = r0 + 64 >= r;
                if (last_of_adapter) { todo &= todo - 1; r0 = 0; if (todo) l = (int)__builtin_ctzll(todo); }
                else r0 += 64;
                if (todo) load_next();
                lds_barrier();
                read_frags(NST - 1, 0);
                mma(ext, 0);
                if (kc > 32) { read_frags(NST - 1, 1); mma(ext, 1); }
                if (last_of_adapter) {
#pragma unroll
                    for (int a = 0; a < MB; ++a) {
                        const int row = m0 + wm * WTM + a * 16 + l16;
                        const bool own = row >= c_lo && row < c_hi;
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int q = 0; q < 4; ++q) acc[a][b][q] = own ? sc * ext[a][b][q] : acc[a][b][q];
                    }
                }
                if (!todo) break;
            }
        }
    }

    // ---- contraction over the frozen weight -----------------------------------------------------------
    // Step t starts with the fragments of its first half in registers: the second half's are read while the first is multiplied.  Then
    // stage t + 1 has landed and everybody has read stage t (its slot is free for stage t + NST); the first half of t + 1 is
    // read while the second of t is multiplied.
    if (nk >= NST) {
        lds_barrier();                   // the pass slot has been read
        issue();                         // stage NST - 1
        wait_loads_and_barrier<LPS * (NST - 1)>();
        read_frags(0, 0);
        int cur = 0, nxt = 1;            // slots of stages t and t + 1
        auto half = [&](int h, int slot, bool load) {    // multiply half h, read the other half from `slot`
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                __builtin_amdgcn_sched_barrier(0);
                if (load) {
#pragma unroll
                    for (int c = 0; c < LPS; ++c)
                        if (c * MB / LPS == a) issue1(c);
                }
                __builtin_amdgcn_sched_barrier(0);
                read_frag_a(slot, h ^ 1, a);
#pragma unroll
                for (int b = a * NB / MB; b < (a + 1) * NB / MB; ++b) read_frag_b(slot, h ^ 1, b);
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = mfma16(fb[h][b], fa[h][a], acc[a][b]);
                interleave();
            }
        };
        auto advance = [&]() {
            cur = nxt;
            nxt = nxt == NST - 1 ? 0 : nxt + 1;
        };
        for (int t = 0; t < nk - NST; ++t) {
            half(0, cur, false);
            wait_loads_and_barrier<LPS * (NST - 2)>();
            half(1, nxt, true);
            advance();
        }
        // the last NST stages: nothing left to load
#define SG_DRAIN(J)                                                                             \
        if (J < NST) {                                                                          \
            half(0, cur, false);                                                                \
            if (J + 1 < NST) {                                                                  \
                wait_loads_and_barrier<(NST - 2 - J > 0 ? NST - 2 - J : 0) * LPS>();            \
                half(1, nxt, false);                                                            \
            } else {                                                                            \
                mma(acc, 1);                                                                    \
            }                                                                                   \
            advance();                                                                          \
        }
        SG_DRAIN(0) SG_DRAIN(1) SG_DRAIN(2) SG_DRAIN(3) SG_DRAIN(4) SG_DRAIN(5) SG_DRAIN(6) SG_DRAIN(7)
        static_assert(NST <= 8, "drain steps");
#undef SG_DRAIN
    } else if (nk > 0) {
        wait_loads_and_barrier<0>();
        for (int t = 0; t < nk; ++t) { read_frags(t, 0); read_frags(t, 1); mma(acc, 0); mma(acc, 1); }
    }

    // ---- tail of a contraction that is not a multiple of 64 -----------------------------------------
    if ((g.Kdim & 63) != 0) {
        const int k0 = nk * 64;
        lds_barrier();
        pass_load(g.Aop + (int64_t)m0 * g.lda + k0, g.lda, m0, min(g.M, m0 + BM), true, NN ? g.Bop + (int64_t)k0 * g.ldb : g.Bop + k0,
                  g.ldb, true, g.Kdim - k0);
        pass_store(g.Kdim - k0);
        lds_barrier();
        read_frags(NST - 1, 0);
        mma(acc, 0);
        if (g.Kdim - k0 > 32) { read_frags(NST - 1, 1); mma(acc, 1); }
    }

    // ---- the tile goes through LDS, whole rows of it to memory ----------------------------------------
    lds_barrier();
    constexpr int E_LD = BN + 8;
    static_assert(BM * E_LD * 2 <= NST * STAGE, "epilogue staging fits the ring");
    u16* Es = reinterpret_cast<u16*>(lds);
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            uint2 v;
            v.x = pack2hw(acc[a][b][0], acc[a][b][1]);
            v.y = pack2hw(acc[a][b][2], acc[a][b][3]);
            *reinterpret_cast<uint2*>(Es + (wm * WTM + a * 16 + l16) * E_LD + wn * WTN + b * 16 + g4 * 4) = v;
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
// 256 x 256 kernel moves the fewest bytes per product and wins wherever its last round is not too empty).  Over 192 products
// (64 .. 16384 tokens, widths 512 .. 14336, both directions) the choice takes 0.1 % longer in all than the best of the four, 11 % at worst.
// Measured (us, 256 x 256 / 128 x 128 / 64 x 128 / 64 x 64, tokens x outputs x contraction): 1000 x 4096 x 4096  86 / 41 / 56 / 81;
// 1000 x 1024 x 4096  81 / 34 / 28 / 23;  200 x 512 x 2048  67 / 25 / 18 / 14;  4000 x 4096 x 4096  110 / 157 / 220 / 300.
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
