// Weight-gradient work items of the general kernels (fp32, and bf16 with rows that start at any element): their own kernel in general.hip, and
// beside the fp32 backward product in f32_gemm.hip.
#pragma once

#include "general_common.h"

namespace mlora {

// ---- weight gradients ------------------------------------------------------------------------------------------------------------
// Work item = 64 columns of X (dA_i) or dY (dB_i) x 16 NB ranks of one adapter, over all its tokens; the eight wavefronts deal the
// tokens in pieces of 16 (fp32) / 32 (bf16).  The contraction (tokens) is the row index of both operands in memory, so a lane
// loads four adjacent columns 4 l16 .. 4 l16 + 3 of its tokens at once and those feed four different blocks (block x holds the
// columns 4 j + x); nothing goes through LDS but the final sum over the wavefronts.
template <typename T> struct GenWgradArgs {
    const T* X; const T* dY; const T* S; const T* dS;
    int32_t panels_k, panels;     // 64-column panels of X, and of X and dY
    uint32_t rank_items;          // work items along the ranks
    int32_t accumulate;
    PlanView pv;
};

// WHOLE: k and n are at least 64, so that every panel can be whole.  red: kGenWgradFloats<NB> floats of LDS.  NW: wavefronts of the work group, 8,
// or 4 that each do the part of two, one after the other (the same sums in the same order).
template <int NB> constexpr int kGenWgradFloats = 4 * 64 * (16 * NB + 1);
template <typename T, int NB, bool WHOLE, int NW = 8>
__device__ __forceinline__ void general_wgrad_body(const GenWgradArgs<T>& g, float* const red, const int panel, const int i, const int rank_item) {
    constexpr int RW = 16 * NB, RLD = RW + 1;
    constexpr int PT = kBlockK<T>;                       // tokens per piece
    constexpr int TPL = kQuadRows<T>;                    // tokens per lane and piece
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int r = g.pv.rank[i], rho0 = rank_item * RW;
    if (rho0 >= r || panel >= g.panels) return;
    const bool isA = panel < g.panels_k;
    const int64_t width = isA ? g.pv.k : g.pv.n;
    // the last panel starts early enough to be whole; what it shares with the one before is not stored
    const int64_t col_own = (int64_t)(isA ? panel : panel - g.panels_k) * 64, col0 = max((int64_t)0, min(col_own, width - 64));
    const int row0 = g.pv.off[i], rows = g.pv.off[i + 1] - row0;
    const int lcol = (int)min((int64_t)4 * l16, width - col0 - 1);      // (panels narrower than 64: lanes past the edge repeat its last column)
    const T* big = (isA ? g.X : g.dY) + (int64_t)row0 * width + col0 + lcol;
    const T* small = (isA ? g.dS : g.S) + g.pv.soff[i];
    const int cols = (int)min((int64_t)4, width - col0 - lcol);
    int rho[NB];                                         // ranks past r repeat the last one: not stored
#pragma unroll
    for (int b = 0; b < NB; ++b) rho[b] = min(rho0 + 16 * b + l16, r - 1);
    // a lane's tokens of a piece: T0, T0 + TE, ...
    constexpr int TE = sizeof(T) == 4 ? 4 : 1;
    const int T0 = sizeof(T) == 4 ? g4 : 8 * g4;

    f32x4 acc[4][NB];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[x][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int D = sizeof(T) == 4 ? 2 : 3;            // pieces on their way (fp32: its MFMAs take longer than its loads)
    quad_t<T> wide[D + 1][TPL];
    T narrow[D + 1][TPL][NB];
    auto compute = [&](int set) {
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (rho0 + 16 * b >= r) continue;
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        acc[x][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wide[set][e][x]), narrow[set][e][b], acc[x][b], 0, 0, 0);
                }
        } else {
            uint4 fw[4], fn[NB];
#pragma unroll
            for (int x = 0; x < 4; ++x) fw[x] = quad_column<T>(wide[set], x);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                uint32_t w[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) w[p] = (uint32_t)narrow[set][2 * p][b] | ((uint32_t)narrow[set][2 * p + 1][b] << 16);
                fn[b] = make_uint4(w[0], w[1], w[2], w[3]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[x][b] = block_mma<T>(fw[x], fn[b], acc[x][b]);
        }
    };
    // Wavefront w takes the pieces w, w + 8, ...  Whole ones are loaded without conditions, D ahead (past the last one it is loaded again): with a
    // condition per load, even one that always holds, the loop waited for all its loads in every turn.  us before / now, two adapters:
    // bf16 8000 tokens x (300 + 777) 42 / 30, 3000 x (1001 + 2048) 18 / 13; fp32 8000 x (128 + 128) 37 / 30, 3000 x (512 + 512) 17 / 14.
    const int whole = rows / PT;
#pragma nounroll
    for (int part = 0; part < 8 / NW; ++part) {
        const int w8 = wave + NW * part;                     // of eight
        const int mine = whole > w8 ? (whole - w8 + 7) / 8 : 0;
        const bool rest = rows % PT != 0 && whole % 8 == w8;
        if (rest) {                                          // what is left of the tokens, zero-filled; multiplied last
#pragma unroll
            for (int e = 0; e < TPL; ++e) {
                const int t = whole * PT + T0 + TE * e, tc = min(t, rows - 1);
                const quad_t<T> v = load_quad<T>(big + (int64_t)tc * width, WHOLE, cols);
                wide[D][e] = t < rows ? v : (quad_t<T>)(0u);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const T n = small[(int64_t)tc * r + rho[b]];
                    narrow[D][e][b] = t < rows ? n : (T)0;
                }
            }
        }
        if (mine > 0) {
            const T* pw = big + (int64_t)(w8 * PT + T0) * width;
            const T* pn = small + (int64_t)(w8 * PT + T0) * r;
            int next = 0;
            auto load = [&](int set) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < TPL; ++e) {
                    wide[set][e] = load_quad<T>(pw + (int64_t)(TE * e) * width, WHOLE, cols);
#pragma unroll
                    for (int b = 0; b < NB; ++b) narrow[set][e][b] = pn[(int64_t)(TE * e) * r + rho[b]];
                }
                const bool more = ++next < mine;
                pw += more ? (int64_t)(8 * PT) * width : 0;
                pn += more ? (int64_t)(8 * PT) * r : 0;
            };
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (d < mine) load(d);                       // (uniform)
            int p = 0;
            for (; p + D <= mine; p += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) { compute(d); load(d); }
            }
#pragma unroll
            for (int d = 0; d + 1 < D; ++d)
                if (p + d < mine) compute(d);
        }
        if (rest) compute(D);

        // wavefronts 0 .. 3 of the eight write, 4 .. 7 add theirs; the four sums are added in order.  Lane (l16, g4) holds rank 16 b + l16 of
        // the columns 4 (4 g4 + q) + x.
        for (int half = 0; half < 2; ++half) {
            if (w8 >> 2 == half) {
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            float* d = red + ((wave & 3) * 64 + 16 * g4 + 4 * q + x) * RLD + 16 * b + l16;
                            *d = half ? *d + acc[x][b][q] : acc[x][b][q];
                        }
                        if constexpr (NW == 4) acc[x][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
            if (NW == 8) __syncthreads();
        }
    }
    if (NW == 4) __syncthreads();
    const float s = isA ? 1.0f : g.pv.scale[i];
    T* out = global_ptr<T>(isA ? g.pv.ptrs[i].dA : g.pv.ptrs[i].dB);
    for (int idx = tid; idx < 64 * RW; idx += 64 * NW) {
        // consecutive threads, consecutive elements of the output: ranks of a dA_i row, columns of a dB_i row
        const int c = isA ? idx / RW : idx % 64, rho = isA ? idx % RW : idx / 64;
        if (col0 + c < col_own || col0 + c >= width || rho0 + rho >= r) continue;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += red[(w * 64 + c) * RLD + rho];
        v *= s;
        T* o = out + (isA ? (col0 + c) * r + rho0 + rho : (int64_t)(rho0 + rho) * width + col0 + c);
        *o = from_f32<T>(g.accumulate ? v + to_f32<T>(*o) : v);
    }
}

// f32_gemm.hip : Y = X W + s_i S_i B_i (fwd) or dX = dY W^T + dS_i A_i^T in fp32, or either term alone.  `w` (backward, may be null): weight
// gradients built for nb 16-wide rank blocks (`whole`: see above) that go with the product where *with_w comes back true.
int f32_gemm(mlora_plan* p, bool fwd, const void* A, const void* W, void* C, const void* E, uint32_t flags, const GenWgradArgs<float>* w, int nb,
             bool whole, bool* with_w, hipStream_t st);

}  // namespace mlora
