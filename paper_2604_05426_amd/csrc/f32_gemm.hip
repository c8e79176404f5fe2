// fp32 products with the frozen weight, and the rank extension: Y = X W + s_i S_i B_i, dX = dY W^T + dS_i A_i^T (paper Sec. 5.1), or either
// term alone.  No operand needs an alignment beyond its element.
//
// The fp32 matrix instructions of this chip run at 1/16 of the bf16 rate (154 TFLOP/s in a register-only loop), so the contraction over the
// frozen weight goes through the bf16 units: a fp32 value is the sum of three bf16 values, exactly (eight bits of its significand each; see
// Range), and of the nine products of parts the six that reach 2^-24 of the whole are summed in fp32, from the smallest up.  Relative error
// against 64 bits (standard normal operands): contraction 256 1.5e-7 -> 8.1e-8, 2048 1.8e-7 -> 1.3e-7, 4096 2.1e-7 -> 1.7e-7 (before:
// v_mfma_f32_16x16x4_f32).  Time: 2048 x 2048 x 2048 162 -> 106 us (106 -> 162 TFLOP/s), 8000 x 512 x 512 47 -> 34; small layers, where a
// work group's latency counts, are equal or a little faster (256 x 256 x 256 with its adapters 11.7 -> 9.8 us).  Slower are wide outputs of
// a contraction below about 150, forward: a work group takes 17000 cycles for a 64 x 64 tile whose products are a sixth of that, and is alone
// on its CU, where three of the fp32 instruction's were (1500 x 80 x 3000 28 -> 41 us, 4000 x 100 x 2500 52 -> 61, with six adapters of rank
// 128 76 -> 107).
//
// What bounds it: a 128 x 128 work group spends 2650 cycles per 32 elements of contraction whatever else runs (1536 of them are MFMAs; without
// the conversions 1950, without the MFMAs 1500: the two hardly overlap, although they alternate in the code), and the clock falls to 1.85
// GHz with all CUs busy.  Measured and not adopted: the differences of the conversion by the two-element dot product (a third fewer instructions, 8 %
// slower: its result is late), all fragments read behind the barrier (+-2 %), 8-byte stores of the parts (+3 %).
//
// Range: below 2^-110 a value's last parts fall under the smallest bf16, below 2^-134 all three do; close to the largest fp32 number the first part, or
// a product of first parts, rounds to Inf, and Inf itself has no parts.  The first kind is off by 2^-125 at most an element (also
// if the units dropped all that is denormal), times the other operand; the second leaves Inf or NaN.  So an output of K products is in doubt where it
// is not finite or below K 2^-96 max(1, largest of its row of X, largest of its column of W): any other is off by less than 2^-27 of itself beside
// the rounding of the sum.  Of those in doubt, rows (backward: and columns) of zeros and what a NaN in row or column has made NaN are right, and so
// are small sums of two halves (see Order) that are not small: one output in 10^8 of ordinary values is an exact zero by rounding alone, and to
// search its row and column takes the launch 104 -> 130 us at 2048 x 2048 x 2048.  Right are also small results of rows and columns that hold nothing
// below 2^-103 but zero and whose products are all zero or above 2^-90 (cancellation inside a half, zero columns of W); the others are computed again
// with fp32 MFMAs from memory.  All of this follows from the row and the column alone.  us, 2048 x 2048 x 2048 forward / backward (ordinary values
// 110 / 95): one Inf in X 175 / 152, an eighth of the rows with Inf 348 / 369, W zero 183 / 82, eight of its columns zero 145 / 94, -1, 0 and 1
// throughout 183 / 252; rows of zeros and NaN anywhere 106 / 97.
//
// Order of the sum, in all tiles (the tile follows from the number of tokens, and a row's bits must not): units of 32 elements that start at
// multiples of 32, zero-filled at the end; the even and the odd ones are summed apart, in ascending order, and added; then each adapter's
// term.  The rank extension stays with fp32 MFMAs: its operands are other adapters' neighbours, and whatever they hold stays out.
#include <type_traits>

#include "general_wgrad.h"

namespace mlora {

namespace {

struct F32GemmArgs {
    const float* A; const float* W;       // X (fwd) or dY (bwd); W [k][n]
    float* C;                     // Y or dX
    const float* E;               // ragged S or dS
    int64_t lda, ldw, ldc;
    int64_t M, N, K;
    int32_t tiles_m, tiles_n;
    int32_t xcd_run;              // consecutive tiles per XCD
    int32_t base, lora;           // which terms; without the base term C += LoRA term
    PlanView pv;
};

constexpr int FG_THREADS = 512;
typedef u32x4v piece_t;           // 16 bytes of a row
__device__ __forceinline__ piece_t as_piece(uint4 v) { return piece_t{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Two fp32 values as three pairs of bf16 that add up to them: eight bits of the significand each, rounded to nearest.
__device__ __forceinline__ void split2(float a, float b, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    p0 = pack2hw(a, b);
    a -= __uint_as_float(p0 << 16);
    b -= __uint_as_float(p0 & 0xffff0000u);
    p1 = pack2hw(a, b);
    a -= __uint_as_float(p1 << 16);
    b -= __uint_as_float(p1 & 0xffff0000u);
    p2 = pack2hw(a, b);
}

// Tile BT x BT, eight wavefronts: 2 x 2 sub-tiles times the two wavefront groups kg that share the contraction.
// EDGE: the forward of a layer narrower than the tile.
// lds: kF32Lds<BT> bytes; wg: the work group's number in the launch.
template <int BT> constexpr int kF32Ring = (BT == 128 ? 3 : 2) * (BT == 128 ? 1 : 2) * BT * 384;
template <int BT> constexpr int kF32Lds = kF32Ring<BT> + 2 * BT * 4;
template <bool FWD, int BT, bool EDGE>
__device__ __forceinline__ void f32_gemm_body(const F32GemmArgs& g, unsigned char* const lds, const int64_t wg) {
    constexpr int KU = 32;                                   // contraction of a unit: one 16x16x32 MFMA, 64 bytes of a row of parts
    constexpr int Q = BT == 128 ? 1 : 2;                     // units of a stage
    constexpr int KS = Q * KU;
    constexpr int RB = KU * 2;                               // bytes of a contraction row of parts
    constexpr int PLANE = BT * RB, OPER = 3 * PLANE, UNIT = 2 * OPER, STAGE = Q * UNIT;
    constexpr int SLOTS = BT == 128 ? 3 : 2;                 // stages in LDS
    constexpr int PE = 8;                                    // elements of a piece: two loads of 16 bytes, 16 bytes of every part
    constexpr int PP = 2 * BT * KS / PE / FG_THREADS;        // pieces per thread and stage, both operands
    constexpr int CPK = KS / PE, CPN = BT / PE;              // pieces of a contraction row, of a column row (fwd W tile)
    constexpr int D = 2;                                     // stages on their way in registers
    constexpr int MB = BT / 32, NB = BT / 32;                // 16 x 16 blocks of a wavefront
    constexpr int HB = MB > 1 ? MB / 2 : 1;                  // row blocks of a half
    constexpr int NT = 6;                                    // products of parts
    static_assert(SLOTS * STAGE == kF32Ring<BT>, "ring");
    uint32_t* const row_max = reinterpret_cast<uint32_t*>(lds + SLOTS * STAGE);
    uint32_t* const col_max = row_max + BT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l16 = lane & 15, g4 = lane >> 4;

    const int64_t total = (int64_t)g.tiles_m * g.tiles_n;
    const int64_t slot_x = wg / 8;
    const int64_t L = (slot_x / g.xcd_run * 8 + wg % 8) * g.xcd_run + slot_x % g.xcd_run;
    if (L >= total) return;
    const int64_t per_band = (int64_t)8 * g.tiles_n;
    const int64_t band = L / per_band, in_band = L - band * per_band;
    const int band_rows = (int)min((int64_t)8, g.tiles_m - band * 8);
    // The last tile of rows / columns starts early enough to be whole; what it shares with the tile before is not stored.
    const int64_t m_own = (band * 8 + in_band % band_rows) * BT, n_own = in_band / band_rows * BT;
    const int64_t m0 = max((int64_t)0, min(m_own, g.M - BT)), n0 = max((int64_t)0, min(n_own, g.N - BT));

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

    // ---- pieces ----------------------------------------------------------------------------------
    auto is_b = [&](int c) { return PP == 1 ? tid >= FG_THREADS / 2 : c >= PP / 2; };
    auto index = [&](int c) { return PP == 1 ? tid % (FG_THREADS / 2) : tid + FG_THREADS * (c % (PP > 1 ? PP / 2 : 1)); };      // within the operand
    // swizzle key of contraction row k of the fwd W tile (32-byte units)
    auto key = [](int k) {
        return BT == 128 ? nn_swz(k) : BT == 64 ? ((k >> 1) & 1) | (((k >> 3) & 1) << 1) : (k >> 3) & 1;
    };
    auto row_chunk = [](int row, int c) { return c ^ ((row >> 1) & 3); };     // where 16-byte chunk c of a row of parts goes
    int place[PP];                       // where the piece goes inside a stage
#pragma unroll
    for (int c = 0; c < PP; ++c) {
        const int idx = index(c);
        if (FWD && is_b(c)) {
            const int k = idx / CPN, kr = k % KU, at = idx % CPN * 16;      // byte inside the row of 16-bit values
            place[c] = k / KU * UNIT + OPER + kr * BT * 2 + (((at >> 5) ^ key(kr)) << 5) + (at & 16);
        } else {
            const int row = idx / CPK, ch = idx % CPK;
            place[c] = ch / (KU / 8) * UNIT + (is_b(c) ? OPER : 0) + row * RB + (row_chunk(row, ch % (KU / 8)) << 4);
        }
    }
    struct Piece { piece_t w[2]; };
    // largest magnitude of the piece's row, or of its columns (fwd W: the first parts' bits, two columns a register)
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr int PB_ = PP > 1 ? PP / 2 : 1;                 // pieces of the weight operand
    float row_big[PP];
    u16x2 col_big[FWD ? PB_ : 1][4];
#pragma unroll
    for (int c = 0; c < PP; ++c) row_big[c] = 0.f;
#pragma unroll
    for (int c = 0; c < (FWD ? PB_ : 1); ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) col_big[c][q] = u16x2{0, 0};
    uint32_t parts[3][4];                // the piece that is being split
    // two elements of a piece
    auto split_quarter = [&](int c, const Piece& v, int h) __attribute__((always_inline)) {
        const float a = __uint_as_float(v.w[h / 2][2 * (h & 1)]), b = __uint_as_float(v.w[h / 2][2 * (h & 1) + 1]);
        split2(a, b, parts[0][h], parts[1][h], parts[2][h]);
        if (FWD && (PP == 1 || c >= PP / 2))                 // (PP == 1: the operand is the wavefront's, so both are kept)
            col_big[c % PB_][h] = __builtin_elementwise_max(col_big[c % PB_][h], __builtin_bit_cast(u16x2, parts[0][h] & 0x7fff7fffu));
        if (!FWD || PP == 1 || c < PP / 2)
            row_big[c] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(row_big[c], fabsf(a)), fabsf(b));      // (NaN stays)
    };
    auto store_parts = [&](int slot, int c) __attribute__((always_inline)) {
        unsigned char* d = lds + slot * STAGE + place[c];
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<piece_t*>(d + p * PLANE) = piece_t{parts[p][0], parts[p][1], parts[p][2], parts[p][3]};
    };
    auto put = [&](int slot, const Piece (&v)[PP]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < PP; ++c) {
#pragma unroll
            for (int h = 0; h < 4; ++h) split_quarter(c, v[c], h);
            store_parts(slot, c);
        }
    };

    // ---- fragments and products ----------------------------------------------------------------------
    auto frag_a = [&](int unit, int x, int p) {              // part p; `unit`: byte where the unit starts
        return lds_read_frag(reinterpret_cast<const u16*>(lds + unit + p * PLANE + ((wm * MB + x) * 16 + l16) * RB + (row_chunk(l16, g4) << 4)));
    };
    auto frag_b = [&](int unit, int y, int p) {
        const unsigned char* Bs = lds + unit + OPER + p * PLANE;
        if (FWD) {
            const int k = 8 * g4 + (l16 >> 2);
            const unsigned char* at = Bs + k * BT * 2 + (((wn * NB + y) ^ key(k)) << 5) + (l16 & 3) * 8;
            return lds_read_frag_tr(reinterpret_cast<const u16*>(at), reinterpret_cast<const u16*>(at + 4 * BT * 2));
        }
        return lds_read_frag(reinterpret_cast<const u16*>(Bs + ((wn * NB + y) * 16 + l16) * RB + (row_chunk(l16, g4) << 4)));
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Six of the nine products of parts, small ones first (the three left out are below 2^-24 of the whole), summed from zero; the sum is added to
    // acc.  Operands swapped: a lane holds one output row and 4 consecutive columns of each block.
    constexpr int PA[NT] = {0, 1, 2, 0, 1, 0}, PB[NT] = {2, 1, 0, 1, 0, 0};
    auto term = [&](int t, const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x4& part) __attribute__((always_inline)) {
        part = mfma16(b[PB[t]], a[PA[t]], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : part);
    };
    // the products of the unit at byte `at`; `meanwhile` runs between the reads of its fragments and them
    auto unit = [&](int at, auto meanwhile) __attribute__((always_inline)) {
        bf16x8 fa[MB][3], fb[NB][3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int x = 0; x < MB; ++x) fa[x][p] = frag_a(at, x, p);
#pragma unroll
            for (int y = 0; y < NB; ++y) fb[y][p] = frag_b(at, y, p);
        }
        meanwhile();
        f32x4 part[MB][NB];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int x = 0; x < MB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y) term(t, fa[x], fb[y], part[x][y]);
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) acc[x][y] += part[x][y];
    };

    // ---- contraction over the frozen weight ------------------------------------------------------------
    if (BT != 128 && first < tile.d) candidates();       // (128: after the contraction, its registers are needed)
    if (g.base) {
        const int NS = (int)(g.K / KS);              // whole stages
        const float* src[PP];
        int64_t step[PP];
        int cols[PP];                                // EDGE: columns from the piece's first that exist
#pragma unroll
        for (int c = 0; c < PP; ++c) {
            const int idx = index(c);
            cols[c] = PE;
            if (!is_b(c)) {
                src[c] = g.A + min(m0 + idx / CPK, g.M - 1) * g.lda + idx % CPK * PE;
                step[c] = KS;
            } else if (FWD) {
                const int64_t col = n0 + idx % CPN * PE;
                src[c] = g.W + (int64_t)(idx / CPN) * g.ldw + col;
                step[c] = KS * g.ldw;
                if (EDGE) cols[c] = (int)min((int64_t)PE, g.N - col);
            } else {
                src[c] = g.W + min(n0 + idx / CPK, g.N - 1) * g.ldw + idx % CPK * PE;
                step[c] = KS;
            }
        }
        int fetched = 0;                         // the stage `src` points at
        bool more = true;
        auto fetch1 = [&](Piece& v, int c) __attribute__((always_inline)) {
            if (c == 0) more = ++fetched < NS;       // past the last stage: that one again
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                if (EDGE) v.w[w] = as_piece(load16(src[c] + 4 * w, cols[c] - 4 * w));
                else      __builtin_memcpy(&v.w[w], src[c] + 4 * w, 16);
            }
            src[c] += more ? step[c] : 0;
        };
        auto fetch = [&](Piece (&v)[PP]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < PP; ++c) fetch1(v[c], c);
        };
        const std::integral_constant<int, 0> zero{};
        const std::integral_constant<int, 1> one{};
        if (BT == 128 && NS > 0) {
            // Wavefront group kg multiplies every other stage, half of the row blocks per step, one step behind the other group.  A step writes stage
            // (step + 2) and, in a group's second half, reads the fragments of its next stage as those of the present one are used up:
            // no read of a fragment is waited for behind the barrier.
            bf16x8 fa[3][3], fb[NB][3];                      // row blocks take turns on fa
            f32x4 part[NB];
            Piece reg[D][PP];
            auto read_a = [&](int slot, int x, int ua) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < 3; ++p) fa[ua][p] = frag_a(slot * STAGE, x, p);
            };
            auto read_b = [&](int slot, int p) __attribute__((always_inline)) {
#pragma unroll
                for (int y = 0; y < NB; ++y) fb[y][p] = frag_b(slot * STAGE, y, p);
            };
            {
                Piece v0[PP], v1[PP];
                fetch(v0);
                fetch(v1);
#pragma unroll
                for (int d = 0; d < D; ++d) fetch(reg[d]);
                put(0, v0);
                put(1, v1);
            }
            lds_barrier();
            if (kg == 1) {
                put(2, reg[0]);
#pragma unroll
                for (int c = 0; c < PP; ++c) reg[0][c] = reg[1][c];
                fetch(reg[1]);
            }
            int cur = kg, in = kg == 1 ? 0 : 2;      // slots of this group's stage and of the one that is written next
            read_a(cur, 0, 0);
            read_a(cur, 1, 1);
#pragma unroll
            for (int p = 0; p < 3; ++p) read_b(cur, p);
            if (kg == 1) lds_barrier();
            auto step_of = [&](auto half, auto set_, bool mine) __attribute__((always_inline)) {
                constexpr int h = decltype(half)::value, set = decltype(set_)::value;
                constexpr int PREP = 5;              // groups of products that a piece's conversion is spread over
                const int next = cur == 0 ? 2 : cur - 1;
#pragma unroll
                for (int i = 0; i < HB * NT; ++i) {
                    // the second half takes its row blocks backwards: the buffer of the third is the last to be free
                    const int t = i % NT, x = h == 0 ? i / NT : MB - 1 - i / NT, ua = x == MB - 1 ? 0 : x;
                    if (mine) {
                        if (h == 0 && i == 0) { read_a(cur, 2, 2); read_b(cur, 0); }      // (used up last in the step before)
                        if (h == 0 && i == NT) read_a(cur, 3, 0);
                        if (h == 1 && i == 0) read_a(next, 1, 1);
                        if (h == 1 && i == NT) read_a(next, 0, 0);
                    }
                    const int c = i / PREP;
                    if (c < PP && i % PREP < PREP - 1) split_quarter(c, reg[set][c], i % PREP);
                    else if (c < PP) { store_parts(in, c); fetch1(reg[set][c], c); }
                    if (mine) {
#pragma unroll
                        for (int y = 0; y < NB; ++y) term(t, fa[ua], fb[y], part[y]);
                        if (t == NT - 1) {
#pragma unroll
                            for (int y = 0; y < NB; ++y) acc[x][y] += part[y];
                        }
                        if (h == 1 && i / NT == HB - 1) {
                            if (t == 0) read_b(next, 2);
                            if (t == 3) read_b(next, 1);
                        }
                    }
                    // conversions between the products
#pragma unroll
                    for (int y = 0; y < NB; ++y) { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x002, 3, 0); }
                    __builtin_amdgcn_sched_barrier(0);
                }
                lds_barrier();
                in = in == 2 ? 0 : in + 1;
                if (h == 1) cur = next;
            };
            for (int pairs = NS / 2; pairs > 0; --pairs) { step_of(zero, zero, true); step_of(one, one, true); }
            if (NS & 1) { step_of(zero, zero, kg == 0); step_of(one, one, kg == 0); }
            if (kg == 0) lds_barrier();
        } else if (NS > 0) {
            // All wavefronts on one stage, group kg on its unit kg; the next stage is written meanwhile
            Piece first_stage[PP], reg[D][PP];
            fetch(first_stage);
#pragma unroll
            for (int d = 0; d < D; ++d) fetch(reg[d]);
            put(0, first_stage);
            lds_barrier();
            auto step_of = [&](int slot, Piece (&r)[PP]) __attribute__((always_inline)) {
                unit(slot * STAGE + kg * UNIT, [&]() __attribute__((always_inline)) { put(slot ^ 1, r); fetch(r); });
                lds_barrier();
            };
            int t = 0;
            for (; t + 1 < NS; t += 2) { step_of(0, reg[0]); step_of(1, reg[1]); }
            if (t < NS) step_of(0, reg[0]);
        }
        const int left = (int)(g.K - (int64_t)NS * KS);
        if (left > 0) {                              // the rest of the contraction: one more stage, zero-filled
            Piece v[PP];
#pragma unroll
            for (int c = 0; c < PP; ++c)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const int idx = index(c), k = idx % CPK * PE + 4 * w;
                    if (!is_b(c)) {
                        v[c].w[w] = as_piece(load16(g.A + min(m0 + idx / CPK, g.M - 1) * g.lda + (int64_t)NS * KS + k, left - k));
                    } else if (FWD) {
                        const int kr = idx / CPN;
                        const int64_t col = n0 + idx % CPN * PE + 4 * w;
                        v[c].w[w] = as_piece(load16(g.W + ((int64_t)NS * KS + kr) * g.ldw + col,
                                                       kr < left ? (int)max((int64_t)0, min((int64_t)4, g.N - col)) : 0));
                    } else {
                        v[c].w[w] = as_piece(load16(g.W + min(n0 + idx / CPK, g.N - 1) * g.ldw + (int64_t)NS * KS + k, left - k));
                    }
                }
            put(0, v);                               // everybody has passed the barrier behind the last stage's products
            lds_barrier();
            if (Q == 1 ? kg == (NS & 1) : kg * KU < left) unit(Q == 1 ? 0 : kg * UNIT, []() {});
            lds_barrier();
        }
    }

    if (BT == 128 && first < tile.d) candidates();
    // ---- the two halves of the sum are added: wavefront group kg takes the row blocks kg * OB .. of its sub-tile -------------------
    constexpr int OB = HB;
    f32x4 out[OB][NB];
    {
        f32x4* mine = reinterpret_cast<f32x4*>(lds) + (wave * OB * NB) * 64 + lane;
        const f32x4* other = reinterpret_cast<const f32x4*>(lds) + ((wave ^ 4) * OB * NB) * 64 + lane;
#pragma unroll
        for (int x = 0; x < OB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) {
                const f32x4 lo = acc[x][y], hi = acc[MB - OB + x][y];
                mine[(x * NB + y) * 64] = kg ? lo : hi;
                out[x][y] = kg ? hi : lo;
            }
        if (tid < BT) { row_max[tid] = 0; col_max[tid] = 0; }
        lds_barrier();
#pragma unroll
        for (int x = 0; x < OB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) out[x][y] += other[(x * NB + y) * 64];
    }
    const bool owner = MB > 1 || kg == 0;            // (32 x 32: wavefronts 4 .. 7 have handed everything over)
    const int xb = wm * MB + (MB > 1 ? kg * OB : 0); // first row block of this wavefront inside the tile

    // ---- what the parts may have got wrong is computed again in fp32 (see Range above) -----------------------------------------------------
    if (g.base) {
#pragma unroll
        for (int c = 0; c < PP; ++c) {
            const int idx = index(c);
            if (FWD && is_b(c)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u16x2 m = col_big[c % PB_][q];
                    atomicMax(&col_max[idx % CPN * PE + 2 * q], (uint32_t)m[0] << 16);
                    atomicMax(&col_max[idx % CPN * PE + 2 * q + 1], (uint32_t)m[1] << 16);
                }
            } else {
                atomicMax(is_b(c) ? &col_max[idx / CPK] : &row_max[idx / CPK], __float_as_uint(row_big[c]) & 0x7fffffffu);
            }
        }
        lds_barrier();
        if (owner) {
            auto row_top = [&](int x) { return __uint_as_float(row_max[(xb + x) * 16 + l16]); };
            auto col_top = [&](int y, int q) { return __uint_as_float(col_max[(wn * NB + y) * 16 + 4 * g4 + q]); };
            const float least = (float)g.K * 0x1p-96f;
            uint32_t redo = 0;                               // bit 4 (x NB + y) + q: column q of block y, row block x
            bool small = false;
#pragma unroll
            for (int x = 0; x < OB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float rm = row_top(x), cm = col_top(y, q), v = fabsf(out[x][y][q]);
                        const bool finite = v < __builtin_inff(), held = finite && v >= least * fmaxf(fmaxf(rm, cm), 1.f);
                        const bool zero = v == 0.f && (rm == 0.f || (!FWD && cm == 0.f)), nan = rm != rm || cm != cm;
                        const bool doubt = !held && !zero && !nan;
                        redo |= (uint32_t)doubt << (4 * (x * NB + y) + q);
                        small = small || (doubt && finite);
                    }
            if (__ballot(redo != 0)) {
                constexpr int AT = BT == 128 ? 2 : 4;        // 16-wide steps of the contraction whose loads are in flight together
                // The blocks stand in LDS, lane by lane, so that the loops over them need not be unrolled: with the unrolled code here, the contraction
                // is allocated worse (ordinary values, 2048 x 2048 x 2048: 106.3 / 122.1 us forward / backward with weight gradients instead of 105.2 /
                // 120.5)
                f32x4* const held = reinterpret_cast<f32x4*>(lds) + ((8 + wave) * OB * NB) * 64 + lane;
                const f32x4* const half = reinterpret_cast<const f32x4*>(lds) + ((wave ^ 4) * OB * NB) * 64 + lane;      // (stays until the extension)
                static_assert(16 * OB * NB * 64 * 16 <= SLOTS * STAGE, "two blocks' exchange fits the ring");
#pragma unroll
                for (int b = 0; b < OB * NB; ++b) held[b * 64] = out[b / NB][b % NB];
                auto row_of = [&](int x) { return g.A + min(m0 + (xb + x) * 16 + l16, g.M - 1) * g.lda + 4 * g4; };
                auto col_of = [&](int y) {
                    const int64_t col = min(n0 + (wn * NB + y) * 16 + l16, g.N - 1);
                    return FWD ? g.W + 4 * g4 * g.ldw + col : g.W + col * g.ldw + 4 * g4;
                };
                auto load_w = [&](const float* w, int64_t k, int valid) { return FWD ? gather16(w + k * g.ldw, g.ldw, valid) : load16(w + k, valid); };
                auto valid_at = [&](int64_t k) { return (int)max((int64_t)0, min((int64_t)4, g.K - k - 4 * g4)); };
                if (__ballot(small)) {                       // halves that cancel: their sum is exact, so either one gives both
                    small = false;
#pragma nounroll
                    for (int b = 0; b < OB * NB; ++b) {
                        if (!__ballot((redo >> (4 * b) & 15) != 0)) continue;
                        const f32x4 v = held[b * 64], h = half[b * 64];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float top = least * fmaxf(fmaxf(row_top(b / NB), col_top(b % NB, q)), 1.f);
                            const uint32_t bit = 1u << (4 * b + q);
                            const bool finite = fabsf(v[q]) < __builtin_inff();
                            if (finite && fabsf(h[q]) >= 3.f * top && fmaxf(fabsf(h[q]), fabsf(v[q] - h[q])) >= 4.f * top) redo &= ~bit;
                            small = small || (finite && (redo & bit));
                        }
                    }
                }
                if (__ballot(small)) {                       // the smallest magnitudes but zero, as bits; small results of none that lose bits are right
                    uint32_t lo[OB + NB];
                    const float* src[OB + NB];
#pragma unroll
                    for (int i = 0; i < OB + NB; ++i) { lo[i] = ~0u; src[i] = i < OB ? row_of(i) : col_of(i - OB); }
                    auto take = [&](int i, uint4 v) { lo[i] = min(min(lo[i], min(2 * v.x - 1, 2 * v.y - 1)), min(2 * v.z - 1, 2 * v.w - 1)); };
                    int64_t k = 0;
                    for (; k + 16 * AT <= g.K; k += 16 * AT) {
                        uint4 v[AT][OB + NB];
#pragma unroll
                        for (int s = 0; s < AT; ++s)
#pragma unroll
                            for (int i = 0; i < OB + NB; ++i) v[s][i] = i < OB ? load16(src[i] + k + 16 * s, 4) : load_w(src[i], k + 16 * s, 4);
#pragma unroll
                        for (int s = 0; s < AT; ++s)
#pragma unroll
                            for (int i = 0; i < OB + NB; ++i) take(i, v[s][i]);
                    }
                    for (; k < g.K; k += 16)
#pragma unroll
                        for (int i = 0; i < OB + NB; ++i) take(i, i < OB ? load16(src[i] + k, valid_at(k)) : load_w(src[i], k, valid_at(k)));
                    auto value = [](uint32_t u) { return __uint_as_float(min(u >> 1, 0x7f7fffffu)); };
#pragma unroll
                    for (int i = 0; i < OB + NB; ++i) {
                        lo[i] = min(lo[i], (uint32_t)__shfl_xor((int)lo[i], 16));
                        lo[i] = min(lo[i], (uint32_t)__shfl_xor((int)lo[i], 32));
                    }
#pragma unroll
                    for (int y = 0; y < NB; ++y)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float c = value((uint32_t)__shfl((int)lo[OB + y], 4 * g4 + q));
#pragma unroll
                            for (int x = 0; x < OB; ++x) {
                                const float r = value(lo[x]);
                                const bool right = fabsf(held[(x * NB + y) * 64][q]) < __builtin_inff() && r >= 0x1p-103f && c >= 0x1p-103f && r * c >= 0x1p-90f;
                                redo &= ~((uint32_t)right << (4 * (x * NB + y) + q));
                            }
                        }
                }
                constexpr int YB = FWD && NB > 2 ? 2 : NB;   // blocks of a row block that are computed together (registers)
#pragma nounroll
                for (int b = 0; b < OB * NB; b += YB) {
                    const uint32_t mine = redo >> (4 * b) & (uint32_t)((1ull << (4 * YB)) - 1);
                    if (!__ballot(mine != 0)) continue;
                    const float* a = row_of(b / NB);
                    const float* w[YB];
                    f32x4 sum[YB], part[YB];
#pragma unroll
                    for (int y = 0; y < YB; ++y) { w[y] = col_of(b % NB + y); sum[y] = part[y] = f32x4{0.f, 0.f, 0.f, 0.f}; }
                    auto multiply = [&](uint4 av, const uint4 (&wv)[YB]) {
#pragma unroll
                        for (int y = 0; y < YB; ++y) part[y] = block_mma<float>(wv[y], av, part[y]);
                    };
                    auto add = [&]() {
#pragma unroll
                        for (int y = 0; y < YB; ++y) { sum[y] += part[y]; part[y] = f32x4{0.f, 0.f, 0.f, 0.f}; }
                    };
                    int64_t k = 0;
                    for (; k + 64 <= g.K; k += 64) {
                        uint4 av[4], wv[4][YB];              // all in flight together
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            av[s] = load16(a + k + 16 * s, 4);
#pragma unroll
                            for (int y = 0; y < YB; ++y) wv[s][y] = load_w(w[y], k + 16 * s, 4);
                        }
#pragma unroll
                        for (int s = 0; s < 4; ++s) multiply(av[s], wv[s]);
                        add();
                    }
                    for (; k < g.K; k += 16) {
                        uint4 wv[YB];
#pragma unroll
                        for (int y = 0; y < YB; ++y) wv[y] = load_w(w[y], k, valid_at(k));
                        multiply(load16(a + k, valid_at(k)), wv);
                    }
                    add();
#pragma unroll
                    for (int y = 0; y < YB; ++y) {
                        f32x4 v = held[(b + y) * 64];
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = mine >> (4 * y + q) & 1 ? sum[y][q] : v[q];
                        held[(b + y) * 64] = v;
                    }
                }
#pragma unroll
                for (int b = 0; b < OB * NB; ++b) out[b / NB][b % NB] = held[b * 64];
            }
        }
    }

    // ---- rank extension, adapter by adapter into an accumulator set of its own, of which the adapter's own rows are added: another
    // adapter's operands never touch a row, whatever they hold
    // All ranks of an adapter at once: one wait for its operands instead of one per 32 ranks, which nothing hides with one work group per CU; and no
    // products for 16-row blocks without a row of its.  us, 32 ranks at a time / all, and with v_mfma_f32_16x16x4_f32 for the frozen weight too (tiles of
    // 64 x 64 and three work groups per CU): 100 x 300 x 300 with 32 adapters of rank 128 47.8 / 38.8 / 36.9, 500 x 500 x 3000 with these 89.6 / 67.8 / 72.4,
    // 2000 x 2000 x 2000 with these 144 / 129 / 191, 4000 x 100 x 2500 with 6 of rank 128 113 / 107 / 76.
    constexpr int KX = EDGE ? 32 : MLORA_MAX_RANK;           // ranks whose loads are in flight together
    constexpr int XC = KX / 32;                              // in chunks of 32
    constexpr int XP = KX * 4 + 16, XN = (BT + 4) * 4;       // bytes of a row of the staged operands, of a column row
    constexpr int XB = BT * XP;                              // where the second operand starts
    static_assert(XB + (FWD ? KX * XN : BT * XP) <= SLOTS * STAGE, "the extension's operands fit the ring");
    constexpr int XW = BT / 32, XCPN = BT / 4;             // words per thread and chunk, both operands; words of a column row
    auto x_is_b = [&](int c) { return BT == 32 ? tid >= 256 : c >= XW / 2; };
    auto x_index = [&](int c) { return BT == 32 ? tid & 255 : tid + FG_THREADS * (c % (XW > 1 ? XW / 2 : 1)); };
    auto x_place = [&](int h, int c) {
        const int idx = x_index(c);
        if (FWD && x_is_b(c)) return XB + (32 * h + idx / XCPN) * XN + idx % XCPN * 16;
        return (x_is_b(c) ? XB : 0) + (idx >> 3) * XP + 128 * h + (idx & 7) * 16;
    };
    bool owned[OB] = {};
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
            const float* F = global_ptr<const float>(reinterpret_cast<const void*>(lane64(c_f)));
            const float* E = g.E + (int64_t)lane64((uint64_t)c_so) + (int64_t)(lo_t - seg0) * r;
            const float s = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c_sc), l));
            f32x4 ext[OB][NB];
#pragma unroll
            for (int x = 0; x < OB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y) ext[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int r0 = 0; r0 < r; r0 += KX) {
                const int left = min(KX, r - r0);
                piece_t v[XC][XW];
#pragma unroll
                for (int h = 0; h < XC; ++h) {
                    if (h > 0 && 32 * h >= left) break;      // (uniform)
#pragma unroll
                    for (int c = 0; c < XW; ++c) {
                        const int idx = x_index(c), row = idx >> 3, k = 32 * h + (idx & 7) * 4;
                        if (!x_is_b(c)) {
                            v[h][c] = as_piece(load16(E + (int64_t)row * r + r0 + k, lo_t + row >= lo && lo_t + row < hi ? left - k : 0));
                        } else if (FWD) {
                            const int kr = 32 * h + idx / XCPN;
                            const int64_t col = n0 + (idx % XCPN) * 4;
                            v[h][c] = as_piece(load16(F + (int64_t)(r0 + kr) * g.N + col, kr < left ? (int)max((int64_t)0, min((int64_t)4, g.N - col)) : 0));
                        } else {
                            v[h][c] = as_piece(load16(F + (n0 + row) * r + r0 + k, n0 + row < g.N ? left - k : 0));
                        }
                    }
                }
                lds_barrier();                       // whoever read the stage before is done
#pragma unroll
                for (int h = 0; h < XC; ++h) {
                    if (h > 0 && 32 * h >= left) break;
#pragma unroll
                    for (int c = 0; c < XW; ++c) *reinterpret_cast<piece_t*>(lds + x_place(h, c)) = v[h][c];
                }
                lds_barrier();
                if (owner) {
#pragma unroll
                    for (int k = 0; k < KX; k += 32) {       // 32 ranks are summed by themselves
                        if (k >= left) break;
                        f32x4 part[OB][NB];
#pragma unroll
                        for (int x = 0; x < OB; ++x)
#pragma unroll
                            for (int y = 0; y < NB; ++y) part[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int h = k / 16; h < k / 16 + 2; ++h) {
                            if (h * 16 >= left) continue;
                            uint4 ea[OB], eb[NB];
#pragma unroll
                            for (int x = 0; x < OB; ++x) {
                                ea[x] = *reinterpret_cast<const uint4*>(lds + ((xb + x) * 16 + l16) * XP + h * 64 + g4 * 16);
                            }
#pragma unroll
                            for (int y = 0; y < NB; ++y) {
                                const int col = (wn * NB + y) * 16 + l16;
                                if (FWD) {
                                    const uint32_t* p = reinterpret_cast<const uint32_t*>(lds + XB + (h * 16 + 4 * g4) * XN) + col;
                                    eb[y] = make_uint4(p[0], p[XN / 4], p[2 * (XN / 4)], p[3 * (XN / 4)]);
                                } else {
                                    eb[y] = *reinterpret_cast<const uint4*>(lds + XB + col * XP + h * 64 + g4 * 16);
                                }
                            }
#pragma unroll
                            for (int x = 0; x < OB; ++x) {
                                const int row0 = lo_t + (xb + x) * 16;
                                if (row0 + 16 <= lo || row0 >= hi) continue;      // (uniform: none of the adapter's rows)
#pragma unroll
                                for (int y = 0; y < NB; ++y) part[x][y] = block_mma<float>(eb[y], ea[x], part[x][y]);
                            }
                        }
#pragma unroll
                        for (int x = 0; x < OB; ++x)
#pragma unroll
                            for (int y = 0; y < NB; ++y) ext[x][y] += part[x][y];
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < OB; ++x) {
                const int row = lo_t + (xb + x) * 16 + l16;
                const bool own = row >= lo && row < hi;
                owned[x] = owned[x] || own;
#pragma unroll
                for (int y = 0; y < NB; ++y)
#pragma unroll
                    for (int q = 0; q < 4; ++q) out[x][y][q] = own ? out[x][y][q] + s * ext[x][y][q] : out[x][y][q];
            }
        }
        first += 64;
        if (first < tile.d) candidates();
    }

    if (!owner) return;
#pragma unroll
    for (int x = 0; x < OB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) {
            const f32x4 v = out[x][y];
            const int64_t row = m0 + (xb + x) * 16 + l16, col = n0 + (wn * NB + y) * 16 + 4 * g4;
            if (row >= g.M || row < m_own || (!g.base && !owned[x])) continue;
            float* c = g.C + row * g.ldc + col;
            f32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = (g.base || col + q >= g.N) ? v[q] : v[q] + c[q];
            if (col >= n_own && col + 4 <= g.N) __builtin_memcpy(c, &o, sizeof(o));
            else
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (col + q >= n_own && col + q < g.N) c[q] = o[q];
        }
}

template <bool FWD, int BT, bool EDGE>
__global__ __launch_bounds__(FG_THREADS) __attribute__((amdgpu_waves_per_eu(BT == 32 ? 4 : 2))) void f32_gemm_kernel(F32GemmArgs g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kF32Lds<BT>];
    f32_gemm_body<FWD, BT, EDGE>(g, lds, (int64_t)blockIdx.y * gridDim.x + blockIdx.x);
}

// The backward product and the weight gradients of a small batch: both need dS alone.  The first `gemm_groups` work groups take the
// tiles of dX, the others a weight-gradient item each.
template <int BT, int NB, bool WHOLE>
__global__ __launch_bounds__(FG_THREADS) __attribute__((amdgpu_waves_per_eu(BT == 32 ? 4 : 2)))
void f32_bwd_kernel(F32GemmArgs g, GenWgradArgs<float> w, int gemm_groups) {
    constexpr int BYTES = kF32Lds<BT> > kGenWgradFloats<NB> * 4 ? kF32Lds<BT> : kGenWgradFloats<NB> * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[BYTES];
    const int wg = blockIdx.x;
    if (wg < gemm_groups) {
        f32_gemm_body<false, BT, false>(g, lds, wg);
        return;
    }
    const int item = wg - gemm_groups, i = item / w.panels % w.pv.N;
    general_wgrad_body<float, NB, WHOLE>(w, reinterpret_cast<float*>(lds), item % w.panels, i, item / w.panels / w.pv.N);
}

template <int BT> int64_t set_tiles(F32GemmArgs& a) {        // work groups
    a.tiles_m = (int32_t)((a.M + BT - 1) / BT);
    a.tiles_n = (int32_t)((a.N + BT - 1) / BT);
    const int64_t total = (int64_t)a.tiles_m * a.tiles_n;
    a.xcd_run = total >= 256 ? 32 : (int32_t)((total + 7) / 8);
    const int64_t per = 8 * a.xcd_run;
    return (total + per - 1) / per * per;
}

template <bool FWD, int BT, bool EDGE = false>
void launch(F32GemmArgs a, hipStream_t st) {
    const int64_t groups = set_tiles<BT>(a);
    constexpr int64_t GX = 1 << 20;      // (a dimension of a launch holds fewer than 2^32 work items)
    hipLaunchKernelGGL((f32_gemm_kernel<FWD, BT, EDGE>), dim3((unsigned)(groups < GX ? groups : GX), (unsigned)((groups + GX - 1) / GX)),
                       dim3(FG_THREADS), 0, st, a);
}

// Weight gradients beside the product: up to eight rounds of work groups (beyond, equal within 1 %), and not where they need more registers than
// the two work groups a CU of the 32 x 32 tile leave (ranks above 32).  us a step, apart / together, tokens x k x n (work groups of both in
// CUs): 4 x 64 tokens, 256 x 256 (0.4) 25.1 / 21.3, 600 x 512 x 512 (2.3) 37.4 / 33.6, 1000 x 300 x 700 (3.3) 46.5 / 42.1, 4000 x 128 x 256 (4)
// 40.1 / 37.4, 2048 x 2048 x 2048 (3) 278 / 267, 8000 x 512 x 512 (2.5) 104.5 / 101.9; 32 x 32 tiles and ranks of 64, 500 x 1024 x 512 (2.2)
// 54.9 / 57.7.  Over 150 drawn shapes (64 .. 8000 tokens) a backward call takes 0.2 % more than the better of the two on average, at worst 7 %
// more than apart (350 x 3888 x 64, 16 adapters of rank 16: 28.6 / 30.5); always apart it is 10.6 %.
template <int BT> bool side_by_side(const F32GemmArgs& g, const GenWgradArgs<float>& w, int nb, int num_cus) {
    F32GemmArgs a = g;
    return set_tiles<BT>(a) + (int64_t)w.panels * w.pv.N * w.rank_items <= 8 * num_cus && !(BT == 32 && nb == 4);
}
template <int BT>
void launch_with_wgrad(F32GemmArgs a, const GenWgradArgs<float>& w, int nb, bool whole, hipStream_t st) {
    const int64_t groups = set_tiles<BT>(a), items = (int64_t)w.panels * w.pv.N * w.rank_items;
    const dim3 grid((unsigned)(groups + items)), block(FG_THREADS);
    if (!whole)       hipLaunchKernelGGL((f32_bwd_kernel<BT, 1, false>), grid, block, 0, st, a, w, (int)groups);
    else if (nb == 1) hipLaunchKernelGGL((f32_bwd_kernel<BT, 1, true>), grid, block, 0, st, a, w, (int)groups);
    else if (nb == 2) hipLaunchKernelGGL((f32_bwd_kernel<BT, 2, true>), grid, block, 0, st, a, w, (int)groups);
    else if constexpr (BT != 32) hipLaunchKernelGGL((f32_bwd_kernel<BT, 4, true>), grid, block, 0, st, a, w, (int)groups);
}

// Tile edge for M x N outputs over a contraction of K, the one that the times measured give the least for:
//   launch 4 us + rounds x (fill and epilogue + 64-wide steps x step)
// 128 x 128 and 64 x 64 run one work group per CU, 32 x 32 two (and a step then takes 0.88 us instead of 0.52).
// Measured (us, 32 / 64 / 128, tokens x outputs x contraction):  200 x 2048 x 2048  30 / 33 / 82;  500 x 2048 x 2048  58 / 38 / 84;
// 2048 x 2048 x 2048  270 / 147 / 106;  3000 x 512 x 512  27 / 24 / 29;  8000 x 512 x 512  68 / 48 / 34;  256 x 256 x 256  6 / 9 / 19.
// Over 85 shapes the forward product takes 0.6 % more than with the best tile on average, at worst 15 % (1500 x 3000 x 80).
int tile_edge(int64_t M, int64_t N, int64_t K, int num_cus) {
    auto per_cu = [&](int64_t e) { return (double)(((M + e - 1) / e * ((N + e - 1) / e) + num_cus - 1) / num_cus); };
    const double steps = (double)((K + 63) / 64);
    const double c32 = per_cu(32), r32 = c32 > 1 ? (double)(int64_t)((c32 + 1) / 2) : 1;
    const double fill = (double)((M + 127) / 128 * ((N + 127) / 128)) / num_cus;
    const double t32 = r32 * (1.75 + steps * (c32 > 1 ? 0.88 : 0.52)), t64 = per_cu(64) * (2.0 + steps * 1.07);
    const double t128 = per_cu(128) * (5.0 + steps * (2.5 + 0.7 * (fill < 1 ? fill : 1)));
    return t128 < t64 && t128 < t32 ? 128 : t64 < t32 ? 64 : 32;
}

void forward(const F32GemmArgs& a, int edge, hipStream_t st) {
    if (a.N < 32)                       launch<true, 32, true>(a, st);
    else if (edge == 128 && a.N >= 128) launch<true, 128>(a, st);
    else if (edge == 64 && a.N >= 64)   launch<true, 64>(a, st);
    else                                launch<true, 32>(a, st);
}
// whether the weight gradients `w` (may be null) went with it
template <int BT>
bool backward(mlora_plan* p, const F32GemmArgs& a, const GenWgradArgs<float>* w, int nb, bool whole, hipStream_t st) {
    const bool beside = w && side_by_side<BT>(a, *w, nb, p->num_cus);
    ProfScope prof(p, beside ? MLORA_K_GEMM_BWD_WGRAD : MLORA_K_GEMM_BWD, st);
    if (beside) launch_with_wgrad<BT>(a, *w, nb, whole, st);
    else        launch<false, BT>(a, st);
    return beside;
}

}  // namespace

int f32_gemm(mlora_plan* p, bool fwd, const void* A, const void* W, void* C, const void* E, uint32_t flags, const GenWgradArgs<float>* w, int nb,
             bool whole, bool* with_w, hipStream_t st) {
    F32GemmArgs a{};
    a.A = (const float*)A; a.W = (const float*)W; a.C = (float*)C; a.E = (const float*)E;
    a.M = p->T; a.K = fwd ? p->k : p->n; a.N = fwd ? p->n : p->k;
    a.lda = a.K; a.ldw = p->n; a.ldc = a.N;
    a.base = (flags & MLORA_FLAG_LORA_ONLY) ? 0 : 1;
    a.lora = ((flags & MLORA_FLAG_BASE_ONLY) || p->n_row_blocks == 0) ? 0 : 1;
    a.pv = p->view;
    if (a.M == 0 || (!a.base && !a.lora)) return MLORA_OK;
    const int edge = tile_edge(a.M, a.N, a.K, p->num_cus);
    if (fwd) {
        ProfScope prof(p, MLORA_K_GEMM_FWD, st);
        forward(a, edge, st);
    } else {
        const bool joined = edge == 128  ? backward<128>(p, a, w, nb, whole, st)
                            : edge == 64 ? backward<64>(p, a, w, nb, whole, st)
                                         : backward<32>(p, a, w, nb, whole, st);
        if (w) *with_w = joined;
    }
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

}  // namespace mlora
