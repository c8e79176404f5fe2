// Weight-gradient work items of the bf16 MFMA path: their own kernels in mfma_lora.hip, and beside the small tiles of the backward product in
// mfma_gemm_small.hip.
#pragma once

#include "mfma_common.h"

namespace mlora {

// =========================================================================================
// Weight gradients (token reductions):
//   dA_i[kappa][rho] = sum_t X[t][kappa] dS[t][rho]          out [k][r]
//   dB_i[rho][nu]    = s_i sum_t S[t][rho] dY[t][nu]         out [r][n]  (stored transposed)
// Work item = (token chunk of one adapter, 128-column panel of X or dY).  Both MFMA operands
// have the token index as the row index in memory, so both are read with transposing loads.
// A chunk that covers its whole segment stores the result directly; otherwise fp32 partials go
// to the workspace and a second kernel adds them in chunk order (no atomics, deterministic).
// The kernel is a stream of X / dY, and what it sustains depends on the bytes a CU keeps in flight, i.e. on how
// many workgroups fit a CU: it is built per rank class MAXNB (32-wide rank blocks: 1, 2 or 4, chosen per plan from
// the largest rank), which sizes the accumulators, the prefetch registers and the S / dS tile.  LDS tiles are
// unpadded and XOR-swizzled in 64-byte units so that the transposing reads (4 token rows x 64 bytes per half
// wavefront) are conflict free: the panel tile [64 tokens][128] and a 128-wide S tile keep unit u of token row t at
// u ^ (t & 3), a 64-wide S tile at u ^ ((t >> 1) & 1), a 32-wide one needs none.  Two stages: 40 / 48 / 64 KB.
// =========================================================================================
constexpr int WP = kWgradPanelCols;   // panel columns (128)
constexpr int WT = 64;           // tokens per step
constexpr int WX_TILE = WT * 128;     // panel tile (elements)

struct WgradArgs {
    const u16* X; const u16* dY; const u16* S; const u16* dS;
    float* partials;
    int32_t panels_k, panels_n;
    PlanView pv;
    int32_t accumulate;        // dA_i, dB_i += result (MLORA_FLAG_ACCUM_GRADS)
    int32_t chunk_base;        // first entry of the chunk table this launch covers (the table is ordered by rank class)
};

__device__ __forceinline__ int wgrad_steps(const Entry4& e) { return (e.d + WT - 1) / WT; }

// One work item; isA: a dA_i item (panel of X against dS_i), else a dB_i item (panel of dY against S_i).  The two forms
// are separate instantiations (the kernel branches once, uniformly): they use the MFMA operands the other way round.
// NW: wavefronts per work group: 4, or 8 for the wide build (64 columns x 32 ranks per wavefront: half the accumulators and half
// the prefetch registers per wavefront, 128 registers instead of 240, so twice the wavefronts per CU hide the latency of the
// same two work groups' loads; weight gradients of 4 x 2048 tokens at rank 128, 8192 + 28672 wide: 190 -> 173 us)
// tid: index within the item's 64 NW threads; SHARED: another item has the rest of the work group, which runs sync_steps steps (at least the
// item's own)
template <int MAXNB, bool isA, int NW = 4, bool SHARED = false>
__device__ __forceinline__ void wgrad_body(const WgradArgs& g, u16* lds, const int tid, const Entry4 e, const int panel, const int sync_steps = 0) {
    constexpr int NTHW = 64 * NW;
    static_assert(NW == 4 || (NW == 8 && MAXNB == 4), "8 wavefronts: wide build only");
    constexpr int SW = MAXNB * 32;                 // S / dS tile width (elements)
    constexpr int CPRS = SW / 8;                   // 16-byte chunks per S tile row
    constexpr int W_STAGE = WX_TILE + WT * SW;     // elements per stage
    // byte offset of element column c (multiple of 4) of token row t
    auto x_off = [](int t, int c) { return t * 256 + ((((c >> 5) ^ (t & 3)) << 6) | ((c & 31) << 1)); };
    auto s_off = [](int t, int c) {
        const int u = c >> 5;
        const int us = MAXNB == 4 ? (u ^ (t & 3)) : MAXNB == 2 ? (u ^ ((t >> 1) & 1)) : u;
        return t * (SW * 2) + ((us << 6) | ((c & 31) << 1));
    };
    const int lane = tid & 63, wave = tid >> 6;
    const int i = e.a, chunk = e.b, row0 = e.c, rows = e.d;
    const int r = g.pv.rank[i];
    const int rpad = (r + 31) & ~31;
    const int nblk = rpad / 32;
    const int64_t so = g.pv.soff[i];
    const int seg0 = g.pv.off[i];
    const int width = (int)(isA ? g.pv.k : g.pv.n);
    const u16* big = isA ? g.X : g.dY;
    const u16* small = (isA ? g.dS : g.S) + so + (int64_t)(row0 - seg0) * r;
    const int col0 = panel * WP;
    const bool s_vec = ((r & 7) == 0) && ((so & 7) == 0);
    // ranks that are multiples of 4 but not of 8: 8-byte halves of a chunk, loaded straight into the prefetch registers
    // (the element-wise path combines what it loads at once, which would make every step wait for its own loads)
    const bool s_v8 = !s_vec && ((r & 3) == 0) && ((so & 3) == 0) && ((reinterpret_cast<uintptr_t>(isA ? g.dS : g.S) & 7) == 0);

    // Accumulator blocks of a wavefront: NCB 32-column blocks x NRB 32-rank blocks.  Up to 64 ranks every wavefront takes
    // 32 panel columns against all ranks; the widest build splits the work group 2 x 4 (64 columns x 32 ranks per wavefront;
    // with four wavefronts it was 2 x 2 with 64 x 64 each),
    // which reads a fifth less from LDS for the same MFMAs - that build is bound by LDS bandwidth.
    constexpr int NCB = MAXNB == 4 ? 2 : 1;
    constexpr int NRB = MAXNB == 4 ? (NW == 8 ? 1 : 2) : MAXNB;
    const int cwave = MAXNB == 4 ? (wave & 1) * 64 : wave * 32;      // first panel column of this wavefront
    const int rb0 = MAXNB == 4 ? (wave >> 1) * NRB : 0;              // its first rank block
    f32x16 acc[NCB * NRB];
#pragma unroll
    for (int nb = 0; nb < NCB * NRB; ++nb)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[nb][q] = 0.f;

    const int nt = wgrad_steps(e);
    constexpr int NRA = 1024 / NTHW, NRS = MAXNB * 256 / NTHW;      // 16-byte chunks per thread: panel tile, S tile
    uint4 ra[2][NRA], rb[2][NRS];   // two register sets: tiles of even / odd index, two steps of loads in flight
    auto gload = [&](int tt, int set) {
        const int t0 = tt * WT;
#pragma unroll
        for (int jj = 0; jj < NRA; ++jj) {
            const int trow = (tid >> 4) + (NTHW / 16) * jj, cc = tid & 15;
            const int col = col0 + cc * 8;
            ra[set][jj] = (t0 + trow < rows && col < width)
                              ? load_streaming(big + (int64_t)(row0 + t0 + trow) * width + col) : zero4();
        }
#pragma unroll
        for (int jj = 0; jj < NRS; ++jj) {
            const int idx = tid + NTHW * jj, trow = idx / CPRS, cc = idx % CPRS;
            rb[set][jj] = zero4();
            if (t0 + trow < rows && cc * 8 < r) {
                const u16* ps = small + (int64_t)(t0 + trow) * r + cc * 8;
                if (s_v8) {
                    const uint2 lo = *reinterpret_cast<const uint2*>(ps);
                    rb[set][jj].x = lo.x; rb[set][jj].y = lo.y;
                    if (r - cc * 8 >= 8) {
                        const uint2 hi = *reinterpret_cast<const uint2*>(ps + 4);
                        rb[set][jj].z = hi.x; rb[set][jj].w = hi.y;
                    }
                } else {
                    rb[set][jj] = load_chunk(ps, min(8, r - cc * 8), s_vec);
                }
            }
        }
    };
    auto lstore = [&](int stage, int set) {
        unsigned char* Xs = reinterpret_cast<unsigned char*>(lds + stage * W_STAGE);
        unsigned char* Ss = Xs + WX_TILE * 2;
#pragma unroll
        for (int jj = 0; jj < NRA; ++jj) {
            const int trow = (tid >> 4) + (NTHW / 16) * jj, cc = tid & 15;
            *reinterpret_cast<uint4*>(Xs + x_off(trow, cc * 8)) = ra[set][jj];
        }
#pragma unroll
        for (int jj = 0; jj < NRS; ++jj) {
            const int idx = tid + NTHW * jj, trow = idx / CPRS, cc = idx % CPRS;
            *reinterpret_cast<uint4*>(Ss + s_off(trow, cc * 8)) = rb[set][jj];
        }
    };
    const int lm = lane & 31, h = lane >> 5, gq = lane >> 4, j = lane & 15;
    auto compute = [&](int stage) {
        const unsigned char* Xs = reinterpret_cast<const unsigned char*>(lds + stage * W_STAGE);
        const unsigned char* Ss = Xs + WX_TILE * 2;
#pragma unroll
        for (int ks = 0; ks < WT / 16; ++ks) {
            const int trow = ks * 16 + 8 * (gq >> 1) + (j >> 2);    // token rows trow and trow + 4 share their swizzle keys
            const int coff = 16 * (gq & 1) + 4 * (j & 3);
            bf16x8 a[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                const unsigned char* pa = Xs + x_off(trow, cwave + cb * 32 + coff);
                a[cb] = lds_read_frag_tr(reinterpret_cast<const u16*>(pa), reinterpret_cast<const u16*>(pa + 4 * 256));
            }
#pragma unroll
            for (int rbl = 0; rbl < NRB; ++rbl) {
                if (rb0 + rbl < nblk) {
                    const unsigned char* pb = Ss + s_off(trow, (rb0 + rbl) * 32 + coff);
                    const bf16x8 b = lds_read_frag_tr(reinterpret_cast<const u16*>(pb), reinterpret_cast<const u16*>(pb + 4 * SW * 2));
                    // dA_i items compute the transposed block (ranks down the accumulator rows), so that for both outputs a
                    // lane ends up with 4 consecutive elements of an output row
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
                        acc[cb * NRB + rbl] = isA ? mfma32(b, a[cb], acc[cb * NRB + rbl]) : mfma32(a[cb], b, acc[cb * NRB + rbl]);
                }
            }
        }
    };
    // Tile u travels in register set u & 1 and is computed from LDS stage u & 1.  At the top of step t
    // tile t+1 is written to the other stage (last read before the previous barrier) and the loads
    // of tile t+3 start, so every tile's loads have two whole steps to land.
    if (nt > 0) {
        gload(0, 0);
        if (nt > 1) gload(1, 1);
        lstore(0, 0);
        if (nt > 2) gload(2, 0);
    }
    __syncthreads();
    const int all = SHARED ? sync_steps : nt;
    for (int tt = 0; tt < all; tt += 2) {
        if (tt + 1 < nt) lstore(1, 1);
        if (tt + 3 < nt) gload(tt + 3, 1);
        if (tt < nt) compute(0);
        __syncthreads();
        if (tt + 1 < all) {
            if (tt + 2 < nt) lstore(0, 0);
            if (tt + 4 < nt) gload(tt + 4, 0);
            if (tt + 1 < nt) compute(1);
            __syncthreads();
        }
    }

    const int nchunks = g.pv.wgrad_chunk_start[i + 1] - g.pv.wgrad_chunk_start[i];
    const float s = isA ? 1.0f : g.pv.scale[i];
    const int64_t kk = g.pv.k, nn = g.pv.n;
    // Accumulator element q of lane (lm, h) of block nb is at (row 8 (q >> 2) + 4 h + (q & 3), column lm) of a 32 x 32 block.
    //   dB_i item: rows = panel columns, lane column = rank: out[rho][c], 4 consecutive c per (lane, q >> 2)
    //   dA_i item (transposed block): rows = ranks, lane column = panel column: out[c][rho], 4 consecutive rho
    // so every lane stores 8-byte (bf16) or 16-byte (fp32 partial) pieces; ranks that are not multiples of 4 and
    // the ragged edge go element by element.
    u16* out = global_ptr<u16>(isA ? g.pv.ptrs[i].dA : g.pv.ptrs[i].dB);
    float* part = nchunks == 1 ? nullptr
                               : g.partials + g.pv.part_off[i] + (int64_t)chunk * (kk + nn) * r + (isA ? 0 : kk * r);
    const bool vec = isA ? ((r & 3) == 0) : ((nn & 3) == 0);
    const bool part_vec = vec && ((reinterpret_cast<uintptr_t>(part) & 15) == 0);
#pragma unroll
    for (int ab = 0; ab < NCB * NRB; ++ab) {
        const int nb = rb0 + ab % NRB, cbase = cwave + (ab / NRB) * 32;
        if (nb >= nblk) continue;
#pragma unroll
        for (int qg = 0; qg < 4; ++qg) {
            const int inner = 8 * qg + 4 * h;
            const int c = col0 + cbase + (isA ? lm : inner);
            const int rho = nb * 32 + (isA ? inner : lm);
            if (c >= width || rho >= r) continue;
            const int64_t idx0 = isA ? ((int64_t)c * r + rho) : ((int64_t)rho * nn + c);
            const int nvalid = min(4, isA ? r - rho : width - c);
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = s * acc[ab][4 * qg + q];
            if (part) {
                if (part_vec && nvalid == 4) {
                    *reinterpret_cast<float4*>(part + idx0) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q < nvalid) part[idx0 + q] = v[q];
                }
            } else if (vec && nvalid == 4) {
                uint2* dst = reinterpret_cast<uint2*>(out + idx0);
                if (g.accumulate) {
                    const uint2 old = *dst;
                    v[0] += __uint_as_float(old.x << 16); v[1] += __uint_as_float(old.x & 0xffff0000u);
                    v[2] += __uint_as_float(old.y << 16); v[3] += __uint_as_float(old.y & 0xffff0000u);
                }
                *dst = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < nvalid) out[idx0 + q] = f2bf(g.accumulate ? v[q] + bf2f(out[idx0 + q]) : v[q]);
            }
        }
    }
}

// mfma_gemm_small.hip : the tile that the products of M x N outputs over a contraction of K take (-1: 256 x 256), and their launch
int small_gemm_tile(int64_t M, int64_t N, int64_t K, int num_cus);
void launch_small_gemm(int tile, const GemmArgs& g, bool fwd, const WgradArgs* w, int items, int max_nb, hipStream_t st);

// mfma_gemm.hip ; `w`, `items`, `max_nb`: the weight gradients, launched with the product where *with_w comes back true
int mfma_gemm_fwd(mlora_plan* p, const void* X, const void* W, void* Y, const void* S, uint32_t flags, hipStream_t st);
int mfma_gemm_bwd(mlora_plan* p, const void* dY, const void* W, void* dX, const void* dS, uint32_t flags, const WgradArgs* w, int items,
                  int max_nb, bool* with_w, hipStream_t st);

}  // namespace mlora
