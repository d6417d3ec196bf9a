// stree_linear_ssd: the ordinary causal scan of a long token sequence (the lower-triangular case of
// the tree mask: the paper's remark in Sec. 3 that a chain reduces the method to Mamba2 with an
// initial state).  This is the prefix pass in front of tree decoding: y for every prefix token and
// the state after the last one, which then seeds stree_tree_ssd.
//
// The sequence is walked in chunks of 32 tokens.  With s_i the inclusive cumulative log-decay inside
// the chunk and h the state before it,
//
//   y_i   = exp(s_i) h C_i + sum_{j <= i} exp(s_i - s_j) dt_j <C_i, B_j> x_j + D x_i
//   h_new = exp(s_last) h + sum_j dt_j exp(s_last - s_j) x_j (outer) B_j
//
// A wave owns 32 of the P columns of one (sequence, head), with the state h^T[s][p] (S x 32, fp32) in its MFMA
// accumulators for a whole run of chunks; what a chunk needs beyond that flows through registers and LDS tiles.
//
// The three products are chained through registers by choosing which state column or token each
// accumulator row stands for.  A 32x32 accumulator holds, in lane l, column l%32 and rows
// 8(r/4) + 4(l/32) + r%4; a 32x32x16 operand wants, in lane l, row l%32 and eight k's at 8(l/32).
// The k order of a product is free as long as both operands agree, so registers 8kk .. 8kk+7 of an
// accumulator ARE an operand whose k slot e of half lh stands for row 16kk + 8(e/4) + 4lh + e%4:
//   * Gt[j][i] = B C^T is turned (decay, causal select, bf16) into the M operand of M x in place;
//   * h^T becomes the state operand of C h in place (rounded to bf16), its rows standing for the
//     state columns s so that slot e is column 16kk + 8lh + e: C rows are then read in 16-byte pieces;
//   * x^T and B^T (tokens along k) come from row-major LDS tiles through the transposing LDS read
//     (ds_read_b64_tr_b16), which takes the rows in exactly that order.
//
// Precision: the weights w_j = dt_j exp(s_last - s_j) are fp32 and the state must stay fp32 accurate
// over thousands of tokens, so w_j x_j enters as two bf16 terms (value and rounding remainder): each
// product is then exact to about 2^-17.  Only h and M as operands of the y product are bf16.
//
// What bounds it: the length of one chunk's dependent chain (LDS round trips, eight products into one accumulator,
// the transcendental functions of the decay), not a pipe -- on 8 x 4096 tokens x 80 heads vector units, matrix
// units and LDS are busy about 30 % of the time each.  So the work is laid out in as many waves as the registers
// admit, in the form that suits how many columns there are:
//   * TEAMS (enough heads for every CU): per head one wave for 32 columns each and two more that bring the tiles to
//     LDS and form M, which the columns share, one chunk ahead;
//   * SEGMENTS (a few sequences): a workgroup's eight waves are pieces of one sequence for the same 32 columns.  Each
//     forms the state of its piece alone, the pieces are chained through LDS (h <- exp(sum s) h + local, each wave
//     an eighth of the elements), and each wave then runs its piece again, with y, from its true initial state.  The waves
//     share nothing in the loop: no barrier.  State only (no y): the first half is all there is;
//   * STATE ONLY, long or with many columns: segments whose states are added up, by waves of one or two column groups.
// Measured (80 heads x 64, S = 128, bf16), before = four waves per head, 64-token chunks, four barriers a chunk:
// 8 x 4096 tokens 515 -> 302 us, 4 x 3000 235 -> 153 us, 1 x 4096 242 -> 84 us, 1 x 1013 65 -> 28 us.
#include "common.hpp"
#include "launch.hpp"
#include "tiles.hpp"
#include <type_traits>

namespace stree {

namespace {

constexpr int kQ = 32;             // tokens per chunk
constexpr int kCols = 32;          // columns of P per wave
constexpr int kCUs = 256;

// The LDS of an independent wave, in bytes from its start: the chunk's B rows, with y its C rows, its x rows (32
// columns), then per token of two chunks exp(s), s - log dt, the state's weight, s.
template <int S, bool WY>
struct WaveLds {
    static constexpr int c = kQ * S * 2, x = c + (WY ? kQ * S * 2 : 0), e = x + kQ * kCols * 2;
    static constexpr int u = e + 8 * kQ, w = u + 8 * kQ, s2 = w + 8 * kQ;
    static constexpr int size = s2 + 8 * kQ;          // a multiple of a row: addresses inside the tile can be flipped
    static_assert(size % 512 == 0, "");
};

// B rows keep their 16-byte pieces permuted: the 64-byte block of a row by the row's low bits (the
// transposing read takes one block of four consecutive rows: all 64 banks once), the piece inside
// the block by the next two (a row-parallel 16-byte store then touches every bank once as well).
template <int S>
__device__ __forceinline__ int b_piece_at(int row, int piece) {
    const int blk = S == 64 ? (row >> 1) & 1 : row & 3;
    return row * (S * 2) + ((piece ^ (blk << 2) ^ ((row >> 2) & 3)) << 4);
}

// One chunk of rows (B or C), whole rows to consecutive lanes, from a buffer that ends with the sequence's last
// row: rows past it read as zeros.  The row goes into the vector offset, which is the one that the buffer's range is
// checked against: a scalar offset is not part of it, or is subtracted from a range that may be smaller, and rows
// past the end would then come from whatever lies there (a weight of 0 does not undo a NaN).
// (WIDE: token strides for which 64 rows outgrow a 32-bit offset; rows past
// the sequence are then copies of the last one -- their step size is 0 and their y is not stored.)
template <int S, bool WIDE>
__device__ __forceinline__ void load_rows(u32x4 (&r)[S / 16], const bf16_t *base, long sn, int t0, int T, int lane) {
    constexpr int NK = S / 16, kPieces = S / 8, kRowsAt = kQ / NK;
    const int row0 = lane / kPieces, piece0 = lane % kPieces;
    if constexpr (WIDE) {
#pragma unroll
        for (int q = 0; q < NK; ++q)
            r[q] = *reinterpret_cast<const u32x4 *>(base + (size_t)min(t0 + q * kRowsAt + row0, T - 1) * sn + piece0 * 8);
    } else {
        const int rows = min(kQ, T - t0);
        const auto buf = make_buffer(base + (size_t)t0 * sn, rows > 0 ? (size_t)((rows - 1) * (uint32_t)sn + S) * 2 : 0);
        const uint32_t off = fresh((uint32_t)row0 * (uint32_t)sn * 2 + piece0 * 16);
#pragma unroll
        for (int q = 0; q < NK; ++q)
            r[q] = __builtin_amdgcn_raw_buffer_load_b128(buf, off + q * kRowsAt * (uint32_t)sn * 2, 0, 0);
    }
}
// x: 32 columns of two chunks, four lanes a row
template <bool WIDE>
__device__ __forceinline__ void load_x_rows(u32x4 (&r)[4], const bf16_t *base, long sn, int t0, int T, int lane) {
    if constexpr (WIDE) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            r[q] = *reinterpret_cast<const u32x4 *>(base + (size_t)min(t0 + q * 16 + (lane >> 2), T - 1) * sn + (lane & 3) * 8);
    } else {
        const int rows = min(2 * kQ, T - t0);
        const auto buf = make_buffer(base + (size_t)t0 * sn, rows > 0 ? (size_t)((rows - 1) * (uint32_t)sn + kCols) * 2 : 0);
        const uint32_t off = fresh((uint32_t)(lane >> 2) * (uint32_t)sn * 2 + (lane & 3) * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            r[q] = __builtin_amdgcn_raw_buffer_load_b128(buf, off + q * 16 * (uint32_t)sn * 2, 0, 0);
    }
}
template <int S>
__device__ __forceinline__ void stage_rows(const u32x4 (&r)[S / 16], uint32_t tile, int lane) {
    constexpr int NK = S / 16, kRowsAt = kQ / NK;
    const uint32_t at = fresh(tile + b_piece_at<S>(lane / (S / 8), lane % (S / 8)));
#pragma unroll
    for (int q = 0; q < NK; ++q)                      // row q kRowsAt + row0: what that adds to b_piece_at
        lds_at<u32x4>((at ^ (b_piece_at<S>(q * kRowsAt, 0) & (S * 2 - 1))) + q * kRowsAt * S * 2) = r[q];
}
// Row operand of k step kk (lane = row, eight state columns) from base tile + b_piece_at(lane % 32, lane / 32).
__device__ __forceinline__ bf16x8 row_operand(uint32_t at, int kk) { return lds_at<bf16x8>(at ^ (kk << 5)); }

// The addresses of a lane in the transposing reads of an x tile and of a row tile.
template <int S>
struct TransposedAt {
    uint32_t x, b0, b1;
    __device__ __forceinline__ TransposedAt(uint32_t x_tile, uint32_t row_tile, int lane) {
        const int row = 4 * (lane >> 5) + ((lane & 15) >> 2), quad = lane & 3, blk = (lane >> 4) & 1;
        x = x_tile + row * (kCols * 2) + blk * 32 + quad * 8;
        // B^T: lane row m of a state tile stands for state column 16(m/16) + 8(m/4%2) + 4(m/8%2) + m%4, i.e. column
        // quads 1 and 2 of each 16 change places: that makes the accumulator an operand (see above)
        const int bq = ((quad & 1) << 1) | (quad >> 1);
        b0 = row_tile + b_piece_at<S>(row, blk * 2 + (bq >> 1)) + (bq & 1) * 8;
        b1 = row_tile + b_piece_at<S>(row + 8, blk * 2 + (bq >> 1)) + (bq & 1) * 8;
    }
};
// x^T operand of tokens 16kk .. 16kk+15: lane = column, slot e = token 16kk + 8(e/4) + 4lh + e%4
__device__ __forceinline__ bf16x8 x_operand(uint32_t at, int kk) {
    const uint32_t a = at + 16 * kk * (kCols * 2);
    return join(read_transposed(a), read_transposed(a + 8 * kCols * 2));
}
template <int S>
__device__ __forceinline__ bf16x8 b_operand(uint32_t at0, uint32_t at1, int st, int kk) {
    return join(read_transposed((at0 ^ (st << 6)) + 16 * kk * S * 2), read_transposed((at1 ^ (st << 6)) + 16 * kk * S * 2));
}
__device__ __forceinline__ void widen(const bf16x8 v, float (&f)[8]) {
    const u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) { f[2 * e] = bf16_lo(u[e]); f[2 * e + 1] = bf16_hi(u[e]); }
}

// Log-decays of two chunks, lane = token: s = inclusive prefix sum inside the token's chunk, behind = the sum of
// the steps BEHIND it, sum = each chunk's total.  The state's weights dt_j exp(s_last - s_j) take `behind`, a sum
// of its own: its rounding error is relative to that sum -- small wherever the weight is not negligible -- while
// s_last - s_j as a difference of prefix sums carries the error of |s_last|.
__device__ __forceinline__ void chunk_scan(float a, int lane, float &s, float &behind, float (&sum)[2]) {
    s = a;                                            // row_shr / row_shl 1, 2, 4, 8 in rows of 16, no LDS round trips
    s += dpp_move<0x111, 0xf, true>(s);
    s += dpp_move<0x112, 0xf, true>(s);
    s += dpp_move<0x114, 0xf, true>(s);
    s += dpp_move<0x118, 0xf, true>(s);
    s += dpp_move<0x142, 0xa, false>(s);              // row 0 into row 1, row 2 into row 3
    float t = a;
    t += dpp_move<0x101, 0xf, true>(t);
    t += dpp_move<0x102, 0xf, true>(t);
    t += dpp_move<0x104, 0xf, true>(t);
    t += dpp_move<0x108, 0xf, true>(t);
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 16));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 48));
    t += (lane & 16) ? 0.f : (lane & 32) ? r3 : r1;
    behind = dpp_move<0x130, 0xf, true>(t);           // wave_shl:1
    if ((lane & 31) == 31) behind = 0.f;
    sum[0] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
    sum[1] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 32));
}

// M[i][j] = Gt exp(s_i - s_j) dt_j for j <= i, as the operand of k step kk: lane = i, slot e = token
// 16kk + 8(e/4) + 4lh + e%4, which is Gt's register 8kk + e.  u_at: this half's first quad of s_j - log2 dt_j.
__device__ __forceinline__ bf16x8 decay_operand(const floatx16 &gt, int kk, float s2_i, uint32_t u_at, int l32, int lh) {
    u_at = fresh(u_at);
    const f32x4 u0 = lds_at<f32x4>(u_at + 16 * kk * 4), u1 = lds_at<f32x4>(u_at + (16 * kk + 8) * 4);
    const float uv[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
    u32x4 m;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        // select, never 0 * inf: an overflowed weight above the diagonal is dropped
        const int j = 16 * kk + 8 * (e >> 2) + 4 * lh + (e & 3);
        const float a = gt[8 * kk + e] * __builtin_amdgcn_exp2f(s2_i - uv[e]);
        const float b = gt[8 * kk + e + 1] * __builtin_amdgcn_exp2f(s2_i - uv[e + 1]);
        m[e / 2] = pack2(j <= l32 ? a : 0.f, j + 1 <= l32 ? b : 0.f);
    }
    return __builtin_bit_cast(bf16x8, m);
}

// h^T <- decay h^T + B^T (w x), the weighted x as two bf16 terms.  w_at: this half's first quad of the weights.
template <int S>
__device__ __forceinline__ void update_state(floatx16 (&hacc)[S / 32], float decay, const float (&xf)[2][8], uint32_t w_at,
                                             uint32_t b0, uint32_t b1) {
    const uint32_t at0 = fresh(b0), at1 = fresh(b1);
    w_at = fresh(w_at);
#pragma unroll
    for (int st = 0; st < S / 32; ++st)
#pragma unroll
        for (int e = 0; e < 16; ++e) hacc[st][e] *= decay;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const f32x4 w0 = lds_at<f32x4>(w_at + 16 * kk * 4), w1 = lds_at<f32x4>(w_at + (16 * kk + 8) * 4);
        const float wv[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
        u32x4 v0, v1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = wv[2 * e] * xf[kk][2 * e], b = wv[2 * e + 1] * xf[kk][2 * e + 1];
            v0[e] = pack2(a, b);
            v1[e] = pack2(a - bf16_lo(v0[e]), b - bf16_hi(v0[e]));
        }
        const bf16x8 t0 = __builtin_bit_cast(bf16x8, v0), t1 = __builtin_bit_cast(bf16x8, v1);
#pragma unroll
        for (int st = 0; st < S / 32; ++st) {
            const bf16x8 bt = b_operand<S>(at0, at1, st, kk);
            hacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bt, t0, hacc[st], 0, 0, 0);
            hacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bt, t1, hacc[st], 0, 0, 0);
        }
    }
}
// the state tile as the operand of k step kk of C h, rounded to bf16
template <int ST>
__device__ __forceinline__ bf16x8 state_operand(const floatx16 (&hacc)[ST], int kk) {
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = pack2(hacc[kk / 2][8 * (kk & 1) + 2 * e], hacc[kk / 2][8 * (kk & 1) + 2 * e + 1]);
    return __builtin_bit_cast(bf16x8, v);
}

// The chunk's y, turned around in LDS (where its x rows were), to memory in 16-byte pieces of rows; rows past the
// sequence are dropped.  (The row goes into the vector offset of the store and the scalar offset stays 0: with a
// scalar register there the compiler sees no hazard in overwriting the data registers right behind the store, but
// it was seen here -- the first dword of the last lanes came from the next instruction.)
__device__ __forceinline__ void store_y_rows(uint32_t y_tile, bf16_t *y0, int y_row, int rows, int lane) {
    const auto yr = make_store_rsrc(y0, rows > 0 ? (uint32_t)((rows - 1) * y_row + kCols * 2) : 0u);
#pragma unroll
    for (int q = 0; q < 2; ++q)
        __builtin_amdgcn_raw_buffer_store_b128(lds_at<u32x4>(y_tile + q * 1024 + lane * 16), yr,
                                               ((lane >> 2) + q * 16) * y_row + (lane & 3) * 16, 0, 0);
}
// One chunk for the wave's 32 columns: y into the LDS tile `ys` (where the chunk's x rows were, which are dead by
// then), the state advanced.  at_c, at_b0, at_b1, x_at: this lane's addresses in the C, B and x tiles; e_at, w_at:
// this half's first quad of exp(s) and of the weights; m_operand(kk): the decay-weighted Gt; mid(): called between
// C h and the rest.
// AHEAD: the next state tile's B^T operands are read before this tile's are done with (eight registers more).
// The issue order is set by hand (a wave's matrix instructions run beside the vector instructions behind them, as
// long as those do not wait for them): first the k steps of C h, each with its share of the weighting of x; then
// the state tiles, each tile's four products between the scaling of the next tile and the parts of y.
template <int S, bool AHEAD, typename Mid, typename MOperand>
__device__ __forceinline__ void chunk_columns(floatx16 (&hacc)[S / 32], uint32_t at_c, uint32_t at_b0, uint32_t at_b1,
                                              uint32_t x_at, uint32_t ys, uint32_t e_at, uint32_t w_at, float decay,
                                              float D_h, int lane, Mid &&mid, MOperand &&m_operand) {
    constexpr int NK = S / 16, ST = S / 32;
    const int l32 = lane & 31, lh = lane >> 5;
    x_at = fresh(x_at), e_at = fresh(e_at), w_at = fresh(w_at);
    const uint32_t y_at = fresh(ys + 4 * lh * (kCols * 2) + l32 * 2);
    bf16x8 xt[2], c_op[2];
    f32x4 wv[2];                                      // weights of slots 4q .. 4q+3, one quad ahead
    c_op[0] = row_operand(at_c, 0);
    c_op[1] = row_operand(at_c, 1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) xt[kk] = x_operand(x_at, kk);
    wv[0] = lds_at<f32x4>(w_at);
    __builtin_amdgcn_sched_barrier(0);
    floatx16 yt;
#pragma unroll
    for (int e = 0; e < 16; ++e) yt[e] = 0.f;
    u32x4 t0[2], t1[2];                   // w x as two bf16 terms
    auto weigh = [&](int i) {             // slots 2i, 2i + 1
        const uint32_t xw = __builtin_bit_cast(u32x4, xt[i / 4])[i % 4];
        if ((i & 1) == 0 && i < 6) wv[(i / 2 + 1) & 1] = lds_at<f32x4>(w_at + 8 * (i / 2 + 1) * 4);
        const f32x4 w4 = wv[(i / 2) & 1];
        const float a = w4[2 * (i & 1)] * bf16_lo(xw), b2 = w4[2 * (i & 1) + 1] * bf16_hi(xw);
        const uint32_t hi = pack2(a, b2);
        t0[i / 4][i % 4] = hi;
        t1[i / 4][i % 4] = pack2(a - bf16_lo(hi), b2 - bf16_hi(hi));
    };
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
        yt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c_op[kk & 1], state_operand(hacc, kk), yt, 0, 0, 0);
        if (kk + 2 < NK) c_op[kk & 1] = row_operand(at_c, kk + 2);
#pragma unroll
        for (int i = kk * 8 / NK; i < (kk + 1) * 8 / NK; ++i) weigh(i);
        __builtin_amdgcn_sched_barrier(0);
    }
    mid();
    auto scale = [&](int st, int q) {
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e) hacc[st][e] *= decay;
    };
    bf16x8 bt[2], m[2];
    f32x4 ev = lds_at<f32x4>(e_at);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) bt[kk] = b_operand<S>(at_b0, at_b1, 0, kk);
#pragma unroll
    for (int q = 0; q < 4; ++q) scale(0, q);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < ST; ++st) {
        bf16x8 bn[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            hacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                bt[q >> 1], __builtin_bit_cast(bf16x8, (q & 1) ? t1[q >> 1] : t0[q >> 1]), hacc[st], 0, 0, 0);
            if (st + 1 < ST) {
                if (AHEAD && (q & 1) == 0) bn[q >> 1] = b_operand<S>(at_b0, at_b1, st + 1, q >> 1);
                if (!AHEAD && (q & 1) == 1) bt[q >> 1] = b_operand<S>(at_b0, at_b1, st + 1, q >> 1);
                scale(st + 1, q);
            }
            if (st == 0) {                // rows of C h by exp(s_i), then M x
#pragma unroll
                for (int e = 0; e < 4; ++e) yt[4 * q + e] *= ev[e];
                if (q < 3) ev = lds_at<f32x4>(e_at + 8 * (q + 1) * 4);
                if (q >= 2) m[q - 2] = m_operand(q - 2);
            }
            if (st == ST - 1) {           // y = yt + D x (register r of yt and slot r of x are the same token)
#pragma unroll
                for (int r = 4 * q; r < 4 * q + 4; r += 2) {
                    const uint32_t xw = __builtin_bit_cast(u32x4, xt[r / 8])[(r % 8) / 2];
                    const uint32_t v = pack2(fmaf(D_h, bf16_lo(xw), yt[r]), fmaf(D_h, bf16_hi(xw), yt[r + 1]));
                    const uint32_t at = y_at + (8 * (r >> 2) + (r & 3)) * (kCols * 2);
                    lds_at<unsigned short>(at) = (unsigned short)v;
                    lds_at<unsigned short>(at + kCols * 2) = (unsigned short)(v >> 16);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (st == 0) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) yt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(m[kk], xt[kk], yt, 0, 0, 0);
        }
#pragma unroll
        for (int kk = 0; kk < 2 && AHEAD; ++kk) bt[kk] = bn[kk];
    }
}

// The state between memory and the accumulators: register r of tile st is h[p = l%32][s = st*32 + 16(r/8) + 8lh + r%8],
// so a lane's pieces of 16 bytes lie 32 bytes apart, in 32 different rows.  Moved like that a state was read and written
// at 2.6 TB/s, and prompts of a few tokens are little else; so it goes through LDS, 128 bytes of every row at a time
// (a block: 32 fp32 columns or 64 bf16 ones, 4 KB), and memory sees eight whole lines an instruction.  Each 16-byte
// piece of a block's row lies at piece ^ (row % 8), which keeps both sides free of bank conflicts.  32 sequences x 80
// heads x 64, one token, fp32 state, y / state only: S = 128 65 / 64 -> 38 / 31 us, S = 64 38 / 39 -> 22 / 18 us (the
// four waves per head of the kernel before these forms: 50 / 45 and 32 / 23 us); S = 128, 64 tokens, state only, bf16
// state 44 -> 24 us.
constexpr int kStateBlock = 32 * 128;
template <typename HT>
struct StateBlock {
    static constexpr int cols = 128 / (int)sizeof(HT), tiles = cols / 32;
};
template <int ST>
__device__ __forceinline__ void zero_state(floatx16 (&hacc)[ST]) {
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int e = 0; e < 16; ++e) hacc[st][e] = 0.f;
}
__device__ __forceinline__ f32x4 quad(const floatx16 &v, int q) { return f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}; }
// Requests the 32 rows at `rows` (sr elements apart); they arrive as they lie in memory, in the registers of each
// block's first tile, and spread_state brings them where they belong.
template <int ST, typename HT>
__device__ __forceinline__ void request_state(floatx16 (&hacc)[ST], const HT *rows, int sr, int lane) {
    using Blk = StateBlock<HT>;
    lane = (int)fresh(lane);
#pragma unroll
    for (int st = 0; st < ST; st += Blk::tiles)
#pragma unroll
        for (int q = 0; q < 4; ++q) {                 // rows 8q .. 8q+7, eight lanes each
            const uint4 v = load_stream16(rows + (8 * q + (lane >> 3)) * sr + st * 32 + (lane & 7) * (Blk::cols / 8));
            hacc[st][4 * q] = __uint_as_float(v.x); hacc[st][4 * q + 1] = __uint_as_float(v.y);
            hacc[st][4 * q + 2] = __uint_as_float(v.z); hacc[st][4 * q + 3] = __uint_as_float(v.w);
        }
}
// the place of a lane's row-wise pieces in a block (+ 1024 for every eight rows), and of its pieces as a column
__device__ __forceinline__ uint32_t block_row_at(uint32_t block, int lane) { return block + (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) << 4); }
__device__ __forceinline__ uint32_t block_piece_at(uint32_t block, int piece, int lane) { return block + (lane & 31) * 128 + ((piece ^ (lane & 7)) << 4); }

// ROOM = blocks that the LDS at `room` holds: so many make the trip together.
template <int ROOM, int ST, typename HT>
__device__ __forceinline__ void spread_state(floatx16 (&hacc)[ST], uint32_t room, int lane) {
    using Blk = StateBlock<HT>;
    lane = (int)fresh(lane);
    const int lh = lane >> 5;
#pragma unroll
    for (int st0 = 0; st0 < ST; st0 += ROOM * Blk::tiles) {
#pragma unroll
        for (int i = 0; i < ROOM * 4; ++i) {
            const int st = st0 + i / 4 * Blk::tiles, q = i % 4;
            if (st < ST) lds_at<f32x4>(block_row_at(room + i / 4 * kStateBlock, lane) + q * 1024) = quad(hacc[st], q);
        }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < ROOM * 4; ++i) {
            const int st = st0 + i / 4 * Blk::tiles, q = i % 4;
            const uint32_t block = room + i / 4 * kStateBlock;
            if (st >= ST) continue;
            if constexpr (sizeof(HT) == 4) {          // columns 16(q/2) + 8lh + 4(q%2)
                const f32x4 v = lds_at<f32x4>(block_piece_at(block, 4 * (q >> 1) + 2 * lh + (q & 1), lane));
#pragma unroll
                for (int e = 0; e < 4; ++e) hacc[st][4 * q + e] = v[e];
            } else {                                  // tile q/2, columns 16(q%2) + 8lh
                const u32x4 v = lds_at<u32x4>(block_piece_at(block, 2 * q + lh, lane));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hacc[st + (q >> 1)][8 * (q & 1) + 2 * e] = bf16_lo(v[e]);
                    hacc[st + (q >> 1)][8 * (q & 1) + 2 * e + 1] = bf16_hi(v[e]);
                }
            }
        }
        wave_lds_fence();
    }
}
// The way back, ROOM blocks from tile st0 on: value(st, q) are registers 4q .. 4q+3 of tile st.
template <int ROOM, int ST, typename HT, typename Value>
__device__ __forceinline__ void gather_state(Value &&value, int st0, uint32_t room, int lane) {
    using Blk = StateBlock<HT>;
    lane = (int)fresh(lane);
    const int lh = lane >> 5;
#pragma unroll
    for (int i = 0; i < ROOM * 4; ++i) {
        const int st = st0 + i / 4 * Blk::tiles, q = i % 4;
        const uint32_t block = room + i / 4 * kStateBlock;
        if (st >= ST) continue;
        if constexpr (sizeof(HT) == 4) {
            lds_at<f32x4>(block_piece_at(block, 4 * (q >> 1) + 2 * lh + (q & 1), lane)) = value(st, q);
        } else {
            const f32x4 a = value(st + (q >> 1), 2 * (q & 1)), b = value(st + (q >> 1), 2 * (q & 1) + 1);
            const u32x4 v = {pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3])};
            lds_at<u32x4>(block_piece_at(block, 2 * q + lh, lane)) = v;
        }
    }
    wave_lds_fence();
}
template <int ROOM, int ST, typename HT>
__device__ __forceinline__ void write_state(HT *rows, int sr, int st0, uint32_t room, int lane) {
    using Blk = StateBlock<HT>;
    lane = (int)fresh(lane);
    u32x4 v[ROOM * 4];
#pragma unroll
    for (int i = 0; i < ROOM * 4; ++i)
        if (st0 + i / 4 * Blk::tiles < ST) v[i] = lds_at<u32x4>(block_row_at(room + i / 4 * kStateBlock, lane) + i % 4 * 1024);
#pragma unroll
    for (int i = 0; i < ROOM * 4; ++i) {
        const int st = st0 + i / 4 * Blk::tiles, q = i % 4;
        if (st < ST)
            store_stream16(rows + (8 * q + (lane >> 3)) * sr + st * 32 + (lane & 7) * (Blk::cols / 8),
                           make_uint4(v[i].x, v[i].y, v[i].z, v[i].w));
    }
    wave_lds_fence();
}
template <int ROOM, int ST, typename HT, typename Value>
__device__ __forceinline__ void store_state(Value &&value, HT *rows, int sr, uint32_t room, int lane) {
#pragma unroll
    for (int st0 = 0; st0 < ST; st0 += ROOM * StateBlock<HT>::tiles) {
        gather_state<ROOM, ST, HT>(value, st0, room, lane);
        write_state<ROOM, ST>(rows, sr, st0, room, lane);
    }
}

// ---- independent waves --------------------------------------------------------------------------------------
// WY: y wanted.  NSEG segments x NP column groups of 32 = the waves of a workgroup.  `SR`: the state's row length;
// without y nothing couples the state's columns, and S = 256 runs as two parts of S = 128.  (h_out may be h0: no
// __restrict__ on either.)
template <int S, bool WY, int NSEG, int NP, bool WIDE, typename HT>
__global__ __launch_bounds__(64 * NSEG * NP, (S == 256 ? 1 : 2)) void linear_ssd_kernel(
    int T, int H, int G, int P, int SR, int units, const bf16_t *__restrict__ x, long x_sn, const float *__restrict__ dt,
    const float *__restrict__ dt_bias, const float *__restrict__ A, const bf16_t *__restrict__ Bm, long b_sn,
    const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D, const HT *h0,
    bf16_t *__restrict__ y, HT *h_out) {
    constexpr int NK = S / 16;                        // k steps of a product over the state index
    constexpr int ST = S / 32;                        // state tiles h^T[32 s][32 p]
    constexpr size_t kStage = (size_t)WaveLds<S, WY>::size * NSEG * NP;
    constexpr size_t kChain = NSEG > 1 ? (size_t)NSEG * S * kCols * 4 : 0;   // overlays the wave tiles
    [[maybe_unused]] __shared__ float sums[NSEG];
    __shared__ __align__(512) char lds[kStage > kChain ? kStage : kChain];

    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
    const int seg = wave / NP;
    const int pgs = P / (kCols * NP), parts = WY ? 1 : SR / S;   // workgroups per head: column groups x parts
    const int bh = unit / (pgs * parts), b = bh / H, h = bh % H, g = h / (H / G);
    const int p0 = ((unit % pgs) * NP + wave % NP) * kCols, s0 = WY ? 0 : unit / pgs % parts * S;
    using L = WaveLds<S, WY>;
    const uint32_t tile = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds + wave * L::size;

    const float A2 = A[h] * 1.44269504088896340736f;  // log2 domain
    const float bias_h = dt_bias ? dt_bias[h] : 0.f;
    const float D_h = D ? D[h] : 0.f;
    const bf16_t *xb = x + (size_t)b * T * x_sn + (size_t)h * P + p0;
    const bf16_t *Bb = Bm + (size_t)b * T * b_sn + (size_t)g * SR + s0;
    const bf16_t *Cb = Cm + (size_t)b * T * c_sn + (size_t)g * S;
    const float *dtb = dt + (size_t)b * T * H + h;
    const size_t state_at = ((size_t)bh * P + p0) * SR + s0;
    constexpr int kRoom = L::size / kStateBlock;      // blocks of the state that a wave's tile has room for
    static_assert(kRoom >= 1, "");
    bf16_t *yb = WY ? y + (size_t)b * T * H * P + (size_t)h * P + p0 : nullptr;

    // pairs of chunks [pair0, pair1) of this wave's segment
    const int pairs = (T + 2 * kQ - 1) / (2 * kQ);
    const int pair0 = (int)((long)pairs * seg / NSEG), pair1 = (int)((long)pairs * (seg + 1) / NSEG);

    floatx16 hacc[ST];
    u32x4 rb[NK], rx[4];
    [[maybe_unused]] u32x4 rc[NK];
    float rdt = 0.f;
    auto load_x = [&](int t0) {
        load_x_rows<WIDE>(rx, xb, x_sn, t0, T, lane);
        rdt = dtb[(size_t)min(t0 + lane, T - 1) * H];
    };
    const TransposedAt<S> tr(tile + L::x, tile, lane);
    const uint32_t row_read = tile + b_piece_at<S>(l32, lh);
    const uint32_t quads = tile + 16 * lh;            // tokens 4 lh .. 4 lh + 3 of a per-token array

    // per-token scalars (lane = token) of two chunks to LDS; the sum of each chunk's log2 decays
    auto stage_scalars = [&](int t0, float (&sum)[2]) {
        float d_ = rdt;
        if (dt_bias) d_ = softplus_step(d_ + bias_h);
        if (t0 + lane >= T) d_ = 0.f;
        float s, behind;
        chunk_scan(d_ * A2, lane, s, behind, sum);
        const uint32_t at = fresh(tile + lane * 4);
        if constexpr (WY) {
            lds_at<float>(at + L::e) = __builtin_amdgcn_exp2f(s);
            lds_at<float>(at + L::s2) = s;
            lds_at<float>(at + L::u) = s - __log2f(d_);   // dt = 0 -> +inf -> weight 0
        }
        lds_at<float>(at + L::w) = d_ * __builtin_amdgcn_exp2f(behind);
    };
    auto stage_x = [&](int c) {                       // the x rows of one of the two chunks
        const uint32_t at = fresh(tile + lane * 16);
#pragma unroll
        for (int q = 0; q < 2; ++q) lds_at<u32x4>(at + L::x + q * 1024) = rx[2 * c + q];
    };
    auto first_loads = [&]() {
        // The wait before a use is the least that holds on every way into a loop: the loads ahead of it are
        // issued in the loop's own order, or every iteration would wait for loads that are meant to stay in flight.
        load_x(pair0 * 2 * kQ);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WY) load_rows<S, WIDE>(rc, Cb, c_sn, pair0 * 2 * kQ, T, lane);
        __builtin_amdgcn_sched_barrier(0);
        load_rows<S, WIDE>(rb, Bb, b_sn, pair0 * 2 * kQ, T, lane);
        __builtin_amdgcn_sched_barrier(0);
    };
    const bool from_h0 = (NSEG == 1 || seg == 0) && h0;
    if (from_h0) request_state(hacc, h0 + state_at, SR, lane);
    __builtin_amdgcn_sched_barrier(0);
    first_loads();
    if (from_h0)
        spread_state<kRoom, ST, HT>(hacc, tile, lane);
    else
        zero_state(hacc);

    // ---- the state at the end of the segment: of the first one from h0, of the others from a zero state -------
    if constexpr (NSEG > 1 || !WY) {
        float sum2 = 0.f;
#pragma unroll 1
        for (int pr = pair0; pr < pair1; ++pr) {
            const int t0 = pr * 2 * kQ;
            float sum[2];
            stage_scalars(t0, sum);
            sum2 += sum[0] + sum[1];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                stage_x(c);
                if (c == 1) load_x(t0 + 2 * kQ);      // (past the end: an empty buffer)
                __builtin_amdgcn_sched_barrier(0);
                stage_rows<S>(rb, tile, lane);
                load_rows<S, WIDE>(rb, Bb, b_sn, t0 + (c + 1) * kQ, T, lane);
                wave_lds_fence();
                float xf[2][8];
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) widen(x_operand(tr.x, kk), xf[kk]);
                update_state<S>(hacc, __builtin_amdgcn_exp2f(sum[c]), xf, quads + L::w + c * kQ * 4, tr.b0, tr.b1);
                wave_lds_fence();
            }
        }
        if constexpr (NSEG > 1) {
            if constexpr (WY) first_loads();          // of the second pass: in flight through the chain
            // The segments' states to LDS; each wave chains its share of the elements through all of them, h <- exp(sum s) h +
            // local (the k-th state <- what segment k's y starts from, the first one <- the end of them all).  One wave after the
            // other with a whole state each, the same sums, took (S = 128, 160 column groups, HBM cold): 1013 tokens with y 31.4
            // us, now 30.4; state only 2000 tokens 24.9 -> 22.4; 256 groups x 900 18.1 -> 15.6 and, with y, 35.3 -> 33.8.
            constexpr int kQuads = ST * 4, kShare = kQuads / NSEG;
            static_assert(NP == 1 && kQuads % NSEG == 0, "");
            f32x4 *states = reinterpret_cast<f32x4 *>(lds) + lane;
            if (lane == 0) sums[seg] = sum2;
            __syncthreads();                          // the tiles are dead
#pragma unroll
            for (int i = 0; i < kQuads; ++i) states[(seg * kQuads + i) * 64] = quad(hacc[i / 4], i % 4);
            if constexpr (WY) {
                if (from_h0) request_state(hacc, h0 + state_at, SR, lane);
            }
            __syncthreads();
            f32x4 v[kShare];
#pragma unroll
            for (int k = 0; k < NSEG; ++k) {
                const float whole = __builtin_amdgcn_exp2f(sums[k]);
#pragma unroll
                for (int j = 0; j < kShare; ++j) {
                    f32x4 *at = states + (k * kQuads + seg * kShare + j) * 64;
                    f32x4 l = *at;
                    if (k > 0) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) l[e] = fmaf(whole, v[j][e], l[e]);
                        if constexpr (WY) *at = v[j];
                    }
                    v[j] = l;
                }
            }
#pragma unroll
            for (int j = 0; j < kShare; ++j) states[(seg * kShare + j) * 64] = v[j];
            auto end = [&](int st, int q) { return states[(st * 4 + q) * 64]; };
            if constexpr (WY) {
                // h0, read again for the first segment's y, has arrived ahead of a barrier behind which another wave writes
                // h_out, which may be h0 (by way of the last wave's tile, which lies behind the states)
                static_assert(kChain <= (size_t)L::size * (NSEG - 1), "");
                if (from_h0)
                    spread_state<kRoom, ST, HT>(hacc, tile + (NSEG - 1) * L::size, lane);
                else if (seg == 0)
                    zero_state(hacc);
                __syncthreads();
                if (seg > 0) {
#pragma unroll
                    for (int i = 0; i < kQuads; ++i) {
                        const f32x4 s = states[(seg * kQuads + i) * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e) hacc[i / 4][4 * (i % 4) + e] = s[e];
                    }
                }
                static_assert(kRoom * StateBlock<HT>::tiles >= ST, "");
                if (seg == NSEG - 1) gather_state<kRoom, ST, HT>(end, 0, tile, lane);
                __syncthreads();                      // the states are the wave tiles' again
                if (seg == NSEG - 1) write_state<kRoom, ST>(h_out + state_at, SR, 0, tile, lane);
            } else {
                __syncthreads();
                if (seg == NSEG - 1) store_state<kRoom, ST>(end, h_out + state_at, SR, tile, lane);
            }
        }
    }

    // ---- y ---------------------------------------------------------------------------------------
    if constexpr (WY) {
        const int y_row = H * P * 2;                  // bytes (32 rows: below 2^31, see the envelope)
#pragma unroll 1
        for (int pr = pair0; pr < pair1; ++pr) {
            const int t0 = pr * 2 * kQ;
            float sum[2];
            stage_scalars(t0, sum);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int tc = t0 + c * kQ;
                stage_x(c);
                if (c == 1) load_x(t0 + 2 * kQ);
                __builtin_amdgcn_sched_barrier(0);
                stage_rows<S>(rc, tile + L::c, lane);
                load_rows<S, WIDE>(rc, Cb, c_sn, tc + kQ, T, lane);
                __builtin_amdgcn_sched_barrier(0);
                stage_rows<S>(rb, tile, lane);
                load_rows<S, WIDE>(rb, Bb, b_sn, tc + kQ, T, lane);
                __builtin_amdgcn_sched_barrier(0);
                wave_lds_fence();
                // Gt = B C^T (column = token i, rows = tokens j), decay-weighted: the M operand
                const uint32_t at_b = fresh(row_read), at_c = fresh(row_read + L::c);
                floatx16 gt;
#pragma unroll
                for (int e = 0; e < 16; ++e) gt[e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < NK; ++kk)
                    gt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(at_b, kk), row_operand(at_c, kk), gt, 0, 0, 0);
                const float s2_i = lds_at<float>(tile + L::s2 + (c * kQ + l32) * 4);
                bf16x8 m[2];
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) m[kk] = decay_operand(gt, kk, s2_i, quads + L::u + c * kQ * 4, l32, lh);
                __builtin_amdgcn_sched_barrier(0);
                chunk_columns<S, false>(hacc, at_c, fresh(tr.b0), fresh(tr.b1), tr.x, tile + L::x, quads + L::e + c * kQ * 4,
                                 quads + L::w + c * kQ * 4, __builtin_amdgcn_exp2f(sum[c]), D_h, lane, [] {},
                                 [&](int kk) { return m[kk]; });
                wave_lds_fence();
                store_y_rows(tile + L::x, yb + (size_t)tc * H * P, y_row, min(kQ, T - tc), lane);
                wave_lds_fence();
            }
        }
    }
    if constexpr (NSEG == 1) store_state<kRoom, ST>([&](int st, int q) { return quad(hacc[st], q); }, h_out + state_at, SR, tile, lane);
}

// ---- state only -----------------------------------------------------------------------------------------------
// Without y nothing couples the state's columns along S (S = 256 runs as two parts of S = 128) and a chunk is one product,
// h^T <- decay h^T + B^T (w x): NC column groups of 32 to a wave share the B tile, its transposed operands and the steps.
// `SR`: the state's row length.  (h_out may be h0: no __restrict__ on either.)
//
// What bounds it: the rows' way from memory and L2 into LDS, not the products (S = 64, 480 groups x 2050 tokens, of 33 us
// with 32 columns a wave: without x from memory 23, without B's rows 28, without half of the products 32; every second
// request more for the same rows costs 5 %).  So a wave takes 64 columns, whole 128-byte lines of x, where enough of them are
// left; and the segments' states, which one wave after the other took up before (1 to 2 us a segment), are
// scaled to the end of them all and added up in pairs.  Before (32 columns, chained) -> now, HBM cold: S = 64, 480 x 2050,
// bf16 state 33 -> 24 us, 1280 x 4000 121 -> 103; S = 128, 320 x 2000 37 -> 29, 1280 x 4000 161 -> 136, 160 x 600 14.6 -> 10.9,
// 1280 x 250 20.7 -> 18.8.
template <int S, int NC>
struct StateLds {
    static constexpr int x = kQ * S * 2, w = x + NC * kQ * kCols * 2, size = w + 512;   // (a multiple of a row, see WaveLds)
    static_assert(size % 512 == 0 && 2 * kQ * 4 <= 512, "");
};
template <int S, int NSEG, int NC, typename HT>
__global__ __launch_bounds__(64 * NSEG, 2) void linear_state_kernel(
    int T, int H, int G, int P, int SR, int units, const bf16_t *__restrict__ x, long x_sn, const float *__restrict__ dt,
    const float *__restrict__ dt_bias, const float *__restrict__ A, const bf16_t *__restrict__ Bm, long b_sn,
    const HT *h0, HT *h_out) {
    constexpr int NK = S / 16, ST = S / 32, XR = 2 * NC, kRow = 4 * NC;     // 16-byte pieces: of x a lane holds, of an x row
    using L = StateLds<S, NC>;
    constexpr size_t kStage = (size_t)L::size * NSEG, kChain = (size_t)(NSEG / 2) * NC * S * kCols * 4;   // overlays the tiles
    __shared__ float sums[NSEG];
    __shared__ __align__(512) char lds[kStage > kChain ? kStage : kChain];

    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const int seg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lh = lane >> 5;
    const int pgs = P / (kCols * NC), parts = SR / S;              // workgroups per head: column groups x parts
    const int bh = unit / (pgs * parts), b = bh / H, h = bh % H, g = h / (H / G);
    const int p0 = unit % pgs * NC * kCols, s0 = unit / pgs % parts * S;
    const uint32_t tile = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds + seg * L::size;
    const float A2 = A[h] * 1.44269504088896340736f;  // log2 domain
    const float bias_h = dt_bias ? dt_bias[h] : 0.f;
    const bf16_t *xb = x + (size_t)b * T * x_sn + (size_t)h * P + p0;
    const bf16_t *Bb = Bm + (size_t)b * T * b_sn + (size_t)g * SR + s0;
    const float *dtb = dt + (size_t)b * T * H + h;
    const size_t state_at = ((size_t)bh * P + p0) * SR + s0;
    constexpr int kRoom = L::size / kStateBlock;      // blocks of the state that a wave's tile has room for
    static_assert(kRoom >= 1, "");

    // pairs of chunks [pair0, pair1) of this wave's segment
    const int pairs = (T + 2 * kQ - 1) / (2 * kQ);
    const int pair0 = (int)((long)pairs * seg / NSEG), pair1 = (int)((long)pairs * (seg + 1) / NSEG);

    floatx16 hacc[NC][ST];
    u32x4 rb[NK], rx[XR];
    float rdt = 0.f;
    auto load_dt = [&](int t0) { rdt = dtb[(size_t)min(t0 + lane, T - 1) * H]; };
    auto load_x = [&](int t0) {                       // a chunk's rows (past the end: an empty buffer)
        const int n = min(kQ, T - t0);
        const auto buf = make_buffer(xb + (size_t)t0 * x_sn, n > 0 ? (size_t)((n - 1) * (uint32_t)x_sn + NC * kCols) * 2 : 0);
        const uint32_t off = fresh((uint32_t)(lane / kRow) * (uint32_t)x_sn * 2 + (lane % kRow) * 16);
#pragma unroll
        for (int q = 0; q < XR; ++q)
            rx[q] = __builtin_amdgcn_raw_buffer_load_b128(buf, off + q * (64 / kRow) * (uint32_t)x_sn * 2, 0, 0);
    };
    const TransposedAt<S> tr(tile + L::x, tile, lane);
    const uint32_t quads = tile + L::w + 16 * lh;     // this half's first quad of the weights

    const bool from_h0 = seg == 0 && h0;
#pragma unroll
    for (int n = 0; n < NC; ++n)
        if (from_h0) request_state(hacc[n], h0 + state_at + (size_t)n * kCols * SR, SR, lane);
    __builtin_amdgcn_sched_barrier(0);
    // (in the loop's own order: the wait before a use is the least that holds on every way into a loop)
    load_dt(pair0 * 2 * kQ);
    load_x(pair0 * 2 * kQ);
    __builtin_amdgcn_sched_barrier(0);
    load_rows<S, false>(rb, Bb, b_sn, pair0 * 2 * kQ, T, lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        if (from_h0) spread_state<kRoom, ST, HT>(hacc[n], tile, lane);
        else zero_state(hacc[n]);
    }

    // the state at the end of the segment: of the first one from h0, of the others from a zero state
    float sum2 = 0.f;
#pragma unroll 1
    for (int pr = pair0; pr < pair1; ++pr) {
        const int t0 = pr * 2 * kQ;
        float d_ = rdt, s, behind, sum[2];
        if (dt_bias) d_ = softplus_step(d_ + bias_h);
        if (t0 + lane >= T) d_ = 0.f;
        chunk_scan(d_ * A2, lane, s, behind, sum);
        lds_at<float>(fresh(tile + L::w + lane * 4)) = d_ * __builtin_amdgcn_exp2f(behind);   // (lane = token)
        sum2 += sum[0] + sum[1];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t at_x = fresh(tile + L::x + (lane % kRow) / 4 * (kQ * kCols * 2) + (lane / kRow) * (kCols * 2) + (lane & 3) * 16);
#pragma unroll
            for (int q = 0; q < XR; ++q) lds_at<u32x4>(at_x + q * (64 / kRow) * (kCols * 2)) = rx[q];
            if (c == 1) load_dt(t0 + 2 * kQ);
            load_x(t0 + (c + 1) * kQ);
            __builtin_amdgcn_sched_barrier(0);
            stage_rows<S>(rb, tile, lane);
            load_rows<S, false>(rb, Bb, b_sn, t0 + (c + 1) * kQ, T, lane);
            wave_lds_fence();
            const uint32_t at0 = fresh(tr.b0), at1 = fresh(tr.b1), x_at = fresh(tr.x), w_at = fresh(quads + c * kQ * 4);
            const float decay = __builtin_amdgcn_exp2f(sum[c]);
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int e = 0; e < 16; ++e) hacc[n][st][e] *= decay;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const f32x4 w0 = lds_at<f32x4>(w_at + 16 * kk * 4), w1 = lds_at<f32x4>(w_at + (16 * kk + 8) * 4);
                const float wv[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                bf16x8 term[NC][2];                   // w x as two bf16 terms
#pragma unroll
                for (int n = 0; n < NC; ++n) {
                    float xf[8];
                    widen(x_operand(x_at + n * (kQ * kCols * 2), kk), xf);
                    u32x4 v0, v1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float a = wv[2 * e] * xf[2 * e], b2 = wv[2 * e + 1] * xf[2 * e + 1];
                        v0[e] = pack2(a, b2);
                        v1[e] = pack2(a - bf16_lo(v0[e]), b2 - bf16_hi(v0[e]));
                    }
                    term[n][0] = __builtin_bit_cast(bf16x8, v0), term[n][1] = __builtin_bit_cast(bf16x8, v1);
                }
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    const bf16x8 bt = b_operand<S>(at0, at1, st, kk);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int n = 0; n < NC; ++n)
                            hacc[n][st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bt, term[n][i], hacc[n][st], 0, 0, 0);
                }
            }
            wave_lds_fence();
        }
    }
    // Each segment's share of the state at the end of them all, added up in pairs, then pairs of pairs.  A wave hands its
    // sum on in the slot that it took the first one from (nobody else reads that).
    if constexpr (NSEG > 1) {
        if (lane == 0) sums[seg] = sum2;
        __syncthreads();                              // (and the tiles are dead)
        float later = 0.f;
        for (int k = seg + 1; k < NSEG; ++k) later += sums[k];
        // (in one factor; where steps grow the state so much that it is infinite, in one a segment: a state of zeros stays one)
        const float share = __builtin_amdgcn_exp2f(later);
        const bool beyond = share > 3.4e38f;
#pragma unroll 1
        for (int k = beyond ? seg + 1 : NSEG - 1; k < NSEG; ++k) {
            const float factor = beyond ? __builtin_amdgcn_exp2f(sums[k]) : share;
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int e = 0; e < 16; ++e) hacc[n][st][e] *= factor;
        }
        constexpr int kSlot = NC * ST * 4 * 64;
        f32x4 *slots = reinterpret_cast<f32x4 *>(lds) + lane;
#pragma unroll 1
        for (int step = 1; step < NSEG; step *= 2) {
            const bool gives = (seg & (2 * step - 1)) == step, takes = (seg & (2 * step - 1)) == 0;
            if (gives) {
#pragma unroll
                for (int i = 0; i < NC * ST * 4; ++i) slots[(seg >> 1) * kSlot + i * 64] = quad(hacc[i / 4 / ST][i / 4 % ST], i % 4);
            }
            __syncthreads();
            if (takes) {
#pragma unroll
                for (int i = 0; i < NC * ST * 4; ++i) {
                    const f32x4 v = slots[((seg + step) >> 1) * kSlot + i * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) hacc[i / 4 / ST][i / 4 % ST][4 * (i % 4) + e] += v[e];
                }
            }
        }
        if (seg > 0) return;
    }
#pragma unroll
    for (int n = 0; n < NC; ++n)
        store_state<kRoom, ST>([&](int st, int q) { return quad(hacc[n][st], q); }, h_out + state_at + (size_t)n * kCols * SR, SR, tile, lane);
}

// ---- teams ------------------------------------------------------------------------------------------------
// One workgroup per (sequence, head): NM = P/32 waves that own 32 columns each, and two helpers that work a chunk ahead
// of them: they bring the rows to LDS (one C and x, the other B and the per-token scalars), and behind a barrier
// form Gt and from it the M operand (which do not depend on the columns), half of M each.  The tiles are double
// buffered: two barriers per chunk, which the others meet between C h and the state.  (One helper that does it all
// is the slowest wave of the team: 1.2 us a chunk with one team on the CU against 1.05 us; with three teams on it,
// where the issue slots count, it is 5 to 12 % ahead: 297 and 304 us for 8 x 4096 tokens, 144 and 153 for 4 x 3000.)
// What bounds a team is the chunk after chunk of its head beside the others of its CU, with no unit of its own full:
// without the x loads 8 x 4096 tokens (640 heads) take 272 of 291 us, without the y stores 267, without the MFMAs of
// C h 275, with neither memory nor MFMAs 157.  So a launch lasts as long as the CU with the most teams, and the heads
// left over from a multiple of the CUs are split where that evens it out: into halves, a team of one column wave each
// (the rows and Gt are made twice).
template <int S>
constexpr int kTeams = S == 256 ? 2 : 3;              // of a CU
// The unit of a workgroup behind those of the whole heads (its XCD's share in a row, as unit_of_block); -1: none.
__device__ __forceinline__ int half_of_block(int whole, int units) {
    const int n = units - whole, at = (int)blockIdx.x - 8 * ((whole + 7) / 8), per = (n + 7) / 8;
    const int slot = at >> 3, i = (at & 7) * per + slot;
    return slot < per && i < n ? whole + i : -1;
}
template <int S, int NM>
struct TeamLds {
    static constexpr int rows = kQ * S * 2;           // bytes of one tile
    static constexpr int c = 0, b = 2 * rows, x = b + 2 * rows, m = x + NM * 2 * kQ * kCols * 2, e = m + 2 * 2048;
    static constexpr int w = e + 2 * 2 * kQ * 4, u = w + 2 * 2 * kQ * 4, s2 = u + 2 * kQ * 4, sum = s2 + 2 * kQ * 4, size = sum + 32;
};
template <int S, int NM, bool HALVES, typename HT>
__global__ __launch_bounds__(64 * (NM + 2), kTeams<S>) void linear_ssd_team_kernel(
    int T, int H, int G, int units, int whole, const bf16_t *__restrict__ x, long x_sn, const float *__restrict__ dt,
    const float *__restrict__ dt_bias, const float *__restrict__ A, const bf16_t *__restrict__ Bm, long b_sn,
    const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D, const HT *h0,
    bf16_t *__restrict__ y, HT *h_out) {
    constexpr int NK = S / 16, ST = S / 32, P = NM * kCols;
    using L = TeamLds<S, NM>;
    __shared__ __align__(512) char lds[L::size];
    // HALVES: the first `whole` units are heads, the others halves of heads, whose second column wave has nothing to do.
    const int unit = !HALVES || (int)blockIdx.x < 8 * ((whole + 7) / 8) ? unit_of_block(whole) : half_of_block(whole, units);
    if (unit < 0) return;
    const bool half = HALVES && unit >= whole;
    // The waves of a workgroup go to the four SIMDs in turn: every other workgroup of a CU (32 CUs to an XCD) swaps
    // the roles around, so that the column waves of all of them do not share two SIMDs.
    const int hw_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = NM == 2 && ((blockIdx.x >> 8) & 1) ? hw_wave ^ 2 : hw_wave;
    const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
    const int bh = half ? whole + ((unit - whole) >> 1) : unit, b = bh / H, h = bh % H, g = h / (H / G);
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int pairs = (T + 2 * kQ - 1) / (2 * kQ);

    if (wave >= NM) {
        const bool second = wave > NM;                // brings B and the scalars; the first one brings C and x
        const float A2 = A[h] * 1.44269504088896340736f;
        const float bias_h = dt_bias ? dt_bias[h] : 0.f;
        const bf16_t *rows = second ? Bm + (size_t)b * T * b_sn + (size_t)g * S : Cm + (size_t)b * T * c_sn + (size_t)g * S;
        const long sn = second ? b_sn : c_sn;
        const float *dtb = dt + (size_t)b * T * H + h;
        const bf16_t *xb = x + (size_t)b * T * x_sn + (size_t)h * P;
        // x comes from memory, not from L2 like the others: two chunks ahead
        constexpr int XR = NM * kCols / 16;
        u32x4 rr[NK], rx[2][XR];
        float rdt = 0.f;
        auto load_x = [&](u32x4 (&r)[XR], int t0) {
            const int n = min(kQ, T - t0);
            const auto buf = make_buffer(xb + (size_t)t0 * x_sn, n > 0 ? (size_t)((n - 1) * (uint32_t)x_sn + P) * 2 : 0);
            const uint32_t off = fresh((uint32_t)(lane / (P / 8)) * (uint32_t)x_sn * 2 + (lane % (P / 8)) * 16);
#pragma unroll
            for (int q = 0; q < XR; ++q)
                r[q] = __builtin_amdgcn_raw_buffer_load_b128(buf, off + q * (512 / P) * (uint32_t)x_sn * 2, 0, 0);
        };
        // column tiles of [32 tokens][32 columns]
        const uint32_t x_store = base + L::x + (lane % (P / 8)) / 4 * (2 * kQ * kCols * 2) + (lane / (P / 8)) * (kCols * 2) + (lane & 3) * 16;
        const uint32_t tile = base + (second ? L::b : L::c), row_read = base + b_piece_at<S>(l32, lh);
        auto prepare = [&](auto role) {
            constexpr bool kB = decltype(role)::value;
            if constexpr (kB) {
                rdt = dtb[(size_t)min(lane, T - 1) * H];
            } else {
                load_x(rx[0], 0);
                __builtin_amdgcn_sched_barrier(0);
                load_x(rx[1], kQ);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_rows<S, false>(rr, rows, sn, 0, T, lane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
            for (int pr = 0; pr < pairs; ++pr) {
                const int t0 = pr * 2 * kQ;
                if constexpr (kB) {
                    float d_ = rdt, s, behind, sum[2];
                    if (dt_bias) d_ = softplus_step(d_ + bias_h);
                    if (t0 + lane >= T) d_ = 0.f;
                    chunk_scan(d_ * A2, lane, s, behind, sum);
                    const uint32_t at = base + lane * 4, slot = (pr & 1) * 2 * kQ * 4;     // (read by the others up to a pair later)
                    lds_at<float>(at + L::e + slot) = __builtin_amdgcn_exp2f(s);
                    lds_at<float>(at + L::w + slot) = d_ * __builtin_amdgcn_exp2f(behind);
                    lds_at<float>(at + L::s2) = s;
                    lds_at<float>(at + L::u) = s - __log2f(d_);   // dt = 0 -> +inf -> weight 0
                    if (lane < 2) lds_at<float>(at + L::sum + (pr & 1) * 8) = __builtin_amdgcn_exp2f(lane ? sum[1] : sum[0]);
                    rdt = dtb[(size_t)min(t0 + 2 * kQ + lane, T - 1) * H];
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int tn = t0 + (c + 1) * kQ;
                    if constexpr (!kB) {
#pragma unroll
                        for (int q = 0; q < XR; ++q) lds_at<u32x4>(x_store + c * (kQ * kCols * 2) + q * (512 / P) * (kCols * 2)) = rx[c][q];
                        load_x(rx[c], tn + kQ);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    stage_rows<S>(rr, tile + c * L::rows, lane);
                    load_rows<S, false>(rr, rows, sn, tn, T, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    __syncthreads();
                    // both: Gt, and half of M each
                    const uint32_t at_c = fresh(row_read + L::c + c * L::rows), at_b = fresh(row_read + L::b + c * L::rows);
                    floatx16 gt;
#pragma unroll
                    for (int e = 0; e < 16; ++e) gt[e] = 0.f;
#pragma unroll
                    for (int kk = 0; kk < NK; ++kk)
                        gt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(at_b, kk), row_operand(at_c, kk), gt, 0, 0, 0);
                    const float s2_i = lds_at<float>(base + L::s2 + (c * kQ + l32) * 4);
                    constexpr int kk = kB;
                    lds_at<bf16x8>(base + L::m + c * 2048 + kk * 1024 + lane * 16) =
                        decay_operand(gt, kk, s2_i, base + 16 * lh + L::u + c * kQ * 4, l32, lh);
                    __syncthreads();
                }
            }
            __syncthreads();                          // (the last chunk is still being worked on)
            __syncthreads();
        };
        if (second)
            prepare(std::true_type{});
        else
            prepare(std::false_type{});
    } else {
        if (half && wave > 0) {                       // the others' barriers
            for (int c = 0; c < 4 * pairs + 2; ++c) __syncthreads();
            return;
        }
        const int column = half ? (unit - whole) & 1 : wave, p0 = column * kCols;
        const float D_h = D ? D[h] : 0.f;
        bf16_t *yb = y + (size_t)b * T * H * P + (size_t)h * P + p0;
        const size_t state_at = ((size_t)bh * P + p0) * S;
        const uint32_t x_tile = base + L::x + column * (2 * kQ * kCols * 2);
        const int y_row = H * P * 2;
        floatx16 hacc[ST];
        if (h0)
            request_state(hacc, h0 + state_at, S, lane);
        else
            zero_state(hacc);
        const TransposedAt<S> tr(x_tile, base + L::b, lane);
        const uint32_t row_read = base + L::c + b_piece_at<S>(l32, lh);
        __syncthreads();                              // the first chunk is being prepared
        // (through the second chunk's B and C tiles, which the helpers write behind the next barrier)
        static_assert((NM / 2) * kStateBlock <= L::rows, "");
        if (h0) spread_state<1, ST, HT>(hacc, base + (wave & 1 ? L::b : L::c) + L::rows + (wave >> 1) * kStateBlock, lane);
        __syncthreads();
#pragma unroll 1
        for (int pr = 0; pr < pairs; ++pr) {
            const int t0 = pr * 2 * kQ;
            const uint32_t slot = (pr & 1) * 2 * kQ * 4;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int tc = t0 + c * kQ;
                const uint32_t quads = base + 16 * lh + slot + c * kQ * 4, x_at = tr.x + c * kQ * kCols * 2;
                chunk_columns<S, true>(
                    hacc, fresh(row_read + c * L::rows), fresh(tr.b0 + c * L::rows), fresh(tr.b1 + c * L::rows), x_at,
                    x_tile + c * (kQ * kCols * 2), quads + L::e, quads + L::w,
                    lds_at<float>(base + L::sum + (pr & 1) * 8 + c * 4), D_h, lane, [] { __syncthreads(); },
                    [&](int kk) { return lds_at<bf16x8>(base + L::m + c * 2048 + kk * 1024 + lane * 16); });
                wave_lds_fence();
                store_y_rows(x_tile + c * (kQ * kCols * 2), yb + (size_t)tc * H * P, y_row, min(kQ, T - tc), lane);
                __syncthreads();
            }
        }
        static_assert(kStateBlock <= 2 * kQ * kCols * 2, "");
        store_state<1, ST>([&](int st, int q) { return quad(hacc[st], q); }, h_out + state_at, S, x_tile, lane);
    }
}

template <int S, int NM, typename HT>
hipError_t launch_team(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *Cm,
                       const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    // Halves where every CU has a team and at most half of them would get one more, and all are there at once: S = 128,
    // 640 heads x 4096 tokens 305 -> 291 us, 320 x 2000 104 -> 95, 288 x 1500 77 -> 71; S = 64, 640 x 1500 92 -> 84;
    // S = 256, 288 x 1000 80 -> 71.  Where they are not, the order evens itself out (S = 128, 880 heads 90.2 and 89.8
    // us, 1920 heads 78.9 and 79.6; S = 256, 640 heads 187 and 189), and with fewer than 256 heads a CU's one team
    // pays for a second (160 heads 96.3 and 99.9 us).
    const long heads = (long)d.batch * d.nheads, rest = heads % kCUs;
    const bool split = NM == 2 && rest > 0 && heads > kCUs && 2 * rest <= kCUs && heads + rest <= kTeams<S> * kCUs;
    const int whole = (int)(split ? heads - rest : heads), units = (int)(split ? heads + rest : heads);
    // (Without halves a kernel of its own: the arithmetic of halves costs a launch that has none 2 to 5 %; S = 128, 160 heads x
    // 1013 tokens 37.7 and 36.7 us, 240 x 2050 72.5 and 68.6, 24 x 700 25.8 and 25.3.)
    const auto kernel = split ? linear_ssd_team_kernel<S, NM, NM == 2, HT> : linear_ssd_team_kernel<S, NM, false, HT>;
    hipLaunchKernelGGL(kernel, dim3(8 * ((whole + 7) / 8 + (units - whole + 7) / 8)), dim3(64 * (NM + 2)), 0, st, d.nnodes,
                       d.nheads, d.ngroups, units, whole,
                       (const bf16_t *)x, (long)d.x_stride_n, dt, step_bias(d), A,
                       (const bf16_t *)Bm, (long)d.b_stride_n, (const bf16_t *)Cm, (long)d.c_stride_n, D, (const HT *)h0,
                       (bf16_t *)y, (HT *)h_out);
    return hipGetLastError();
}

template <int S, bool WY, int NSEG, int NP, bool WIDE, typename HT>
hipError_t launch_n(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *Cm,
                    const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    const int units = d.batch * d.nheads * (d.headdim / (kCols * NP)) * (WY ? 1 : d.dstate / S);
    hipLaunchKernelGGL((linear_ssd_kernel<S, WY, NSEG, NP, WIDE, HT>), dim3(8 * ((units + 7) / 8)), dim3(64 * NSEG * NP), 0, st,
                       d.nnodes, d.nheads, d.ngroups, d.headdim, d.dstate, units, (const bf16_t *)x, (long)d.x_stride_n, dt,
                       step_bias(d), A, (const bf16_t *)Bm, (long)d.b_stride_n, (const bf16_t *)Cm, (long)d.c_stride_n,
                       D, (const HT *)h0, (bf16_t *)y, (HT *)h_out);
    return hipGetLastError();
}

template <int S, int NSEG, int NC, typename HT>
hipError_t launch_s(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *h0, void *h_out,
                    hipStream_t st) {
    const int units = d.batch * d.nheads * (d.headdim / (kCols * NC)) * (d.dstate / S);
    hipLaunchKernelGGL((linear_state_kernel<S, NSEG, NC, HT>), dim3(8 * ((units + 7) / 8)), dim3(64 * NSEG), 0, st, d.nnodes,
                       d.nheads, d.ngroups, d.headdim, d.dstate, units, (const bf16_t *)x, (long)d.x_stride_n, dt, step_bias(d), A,
                       (const bf16_t *)Bm, (long)d.b_stride_n, (const HT *)h0, (HT *)h_out);
    return hipGetLastError();
}

// 64 rows beyond a 32-bit byte offset: never met in earnest, one form of the kernel takes them all
bool wide_strides(const stree_dims &d) {
    return d.x_stride_n >= (1L << 25) || d.b_stride_n >= (1L << 25) || d.c_stride_n >= (1L << 25);
}

// With y: eight segments of a sequence where their waves still fit the chip at two a SIMD and each has a chunk pair and a
// half (80 heads x 64, S = 128: 84 us against the team's 126 us for 4096 tokens; 28 against 36 for 1013; at 700 tokens they
// meet).  S = 256: the segments' registers do not fit.
bool y_in_segments(const stree_dims &d) {
    const long waves = (long)d.batch * d.nheads * (d.headdim / kCols);
    return d.dstate != 256 && (d.nnodes + 2 * kQ - 1) / (2 * kQ) >= 12 && waves * 8 <= 2048;
}

// State only, from 8 chunk pairs on: where four segments of 64 columns a wave (whole lines of x, half as many workgroups) are
// ahead of 32 columns, as the pairs from which they are, by the column groups (of 32, with S = 256 two parts each).  A group
// of 64 columns is worth it where the CUs that get one more of them are many, or the prompt is long.  In us, 64 / 32 columns
// (the better of two and four segments):
//   up to 2 groups a CU: S = 64, 400 x 460 10.0 / 11.3, 320 x 2050 22.5 / 25.0; S = 128, 400 x 700 16.3 / 16.4, 460 14.1 / 13.6,
//     4096 50.8 / 65.5, 264 x 1100 21.1 / 20.2, 4096 49.5 / 50.9; S = 256, 400 x 1100 21.4 / 20.9, 4096 51.4 / 54.5
//   up to 3: S = 64, 520 x 2050 36.4 / 33.9, 640 x 4096 66.6 / 74.9; S = 128, 640 x 700 23.6 / 20.8, 4096 88.6 / 95.9, 520 x 4096
//     80.5 / 77.4; S = 256, 640 x 1500 37.1 / 34.7
//   up to 4: S = 64, 800 x 900 21.1 / 25.3; S = 128, 800 x 700 24.6 / 25.2, 2050 55.0 / 65.2; S = 256, 800 x 900 28.1 / 28.4
//   up to 5: S = 64, 1280 x 4096 104 / 129; S = 128, 1280 x 700 35.7 / 31.9, 1500 61.4 / 68.1; S = 256, 1280 x 700 34.7 / 31.0
//   above: S = 128, 1800 x 1000 56.5 / 65.6; S = 256, 1800 x 1200 61.7 / 65.9, 700 40.0 / 38.8.
int pairs_for_64_columns(int dstate, long groups) {
    constexpr int kNever = 1 << 30;
    const int k = dstate == 64 ? 0 : dstate == 128 ? 1 : 2;
    if (groups <= kCUs) return kNever;
    if (groups <= 2 * kCUs) {
        const int from[] = {8, groups >= 272 ? 11 : 20, 24};
        return from[k];
    }
    const int from[4][3] = {{20, 28, kNever}, {10, 11, 11}, {10, 16, 33}, {10, 12, 16}};
    if (groups < 528) return kNever;
    if (groups <= 3 * kCUs) return from[0][k];
    if (groups <= 4 * kCUs) return from[1][k];
    if (groups < 1312) return from[2][k];
    if (groups < 1792) return from[3][k];
    return k == 2 ? 12 : 10;
}

// State only: segments NSEG and 32-column groups NC a wave.  Below 8 pairs the state is formed chunk after chunk, and where
// y would take segments in those: the two give the same bits.  Else the segments' states are added up:
//   * four segments of 64 columns (see above);
//   * up to two groups a CU four segments of 32 columns (160 x 600, S = 128 10.9 us, two 12.5, eight 12.5), but long prompts of
//     few groups with S = 256 eight, chained (64 x 4096 30.4 and 33.0 us, 200 x 2050 21.2 and 22.2; at 1500 tokens they meet);
//   * beyond, two of 32 columns (S = 128, 640 x 520 18.9 us, four 20.8; 520 x 700 20.0 and 20.7; 1280 x 700 31.9 and 34.0), four
//     for long prompts up to three a CU (520 x 1500 33.1 us, two 35.6; S = 256, 640 x 900 25.0 and 25.3);
//   * none with many groups and fewer than 10 pairs (1280 x 520, S = 64 23.4 us, two 24.5).
// One segment: workgroups of one wave; where they are few, or a wave has one pair only, of two waves that ask for a
// pair's x at once (S = 64, 320 x 400: 11.8 and, one wave, 13.1 us; S = 128 15.5 and 15.9 us; 1280 x 60 11.0 and 11.5 us;
// but 1280 x 400 29.2 and 26.4 us; S = 64 20.9 and 19.6 us, 1280 x 60 7.9 and 7.4 us).
template <int S, typename HT>
hipError_t launch_state(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *Cm,
                        const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    if (wide_strides(d)) return launch_n<S, false, 1, 2, true, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    const long groups = (long)d.batch * d.nheads * (d.headdim / kCols) * (d.dstate / S);
    const int pairs = (d.nnodes + 2 * kQ - 1) / (2 * kQ);
    if (pairs < 8 && (groups < 2 * kCUs || (S == 128 && pairs < 2)))
        return launch_n<S, false, 1, 2, false, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    if (pairs < 8 || (pairs < 10 && groups >= 4 * kCUs)) return launch_s<S, 1, 1, HT>(d, x, dt, A, Bm, h0, h_out, st);
    if (y_in_segments(d)) return launch_n<S, false, 8, 1, false, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    if (groups <= kCUs && d.dstate == 256 && pairs >= 28)
        return launch_n<S, false, 8, 1, false, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    if (pairs >= pairs_for_64_columns(d.dstate, groups)) return launch_s<S, 4, 2, HT>(d, x, dt, A, Bm, h0, h_out, st);
    if (groups <= 2 * kCUs || (groups <= 3 * kCUs && S != 64 && pairs >= (d.dstate == 256 ? 12 : 20)))
        return launch_s<S, 4, 1, HT>(d, x, dt, A, Bm, h0, h_out, st);
    return launch_s<S, 2, 1, HT>(d, x, dt, A, Bm, h0, h_out, st);
}

// With y: segments (see above) or teams (160 heads, 1500 tokens: 52 us, two segments each 67 us; 640 heads, 4096 tokens: 300
// us, independent waves without segments 410 us).
template <int S, typename HT>
hipError_t launch_y(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *Cm,
                    const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    if (wide_strides(d)) return launch_n<S, true, 1, 2, true, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    if constexpr (S != 256) {
        if (y_in_segments(d)) return launch_n<S, true, 8, 1, false, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    }
    if constexpr (S == 128) {
        if (d.headdim == 128) return launch_team<S, 4, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    }
    return launch_team<S, 2, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
}

template <typename HT>
hipError_t launch_h(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm, const void *Cm,
                    const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    if (!y) return d.dstate == 64 ? launch_state<64, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st)
                                  : launch_state<128, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    switch (d.dstate) {
        case 64: return launch_y<64, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
        case 128: return launch_y<128, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
        case 256: return launch_y<256, HT>(d, x, dt, A, Bm, Cm, D, h0, y, h_out, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool linear_ssd_supported(const stree_dims &d, const void *x, const void *Bm, const void *Cm, const void *y,
                          const void *h0, const void *h_out) {
    if (d.io_dtype != STREE_BF16) return false;
    const int P = d.headdim, S = d.dstate;
    if (!((P == 64 && (S == 128 || S == 64 || S == 256)) || (P == 128 && S == 128))) return false;
    if ((d.x_stride_n | d.b_stride_n | d.c_stride_n) % 8 != 0) return false;
    // (the state is read and written 16 bytes at a time, like the rows)
    return (((uintptr_t)x | (uintptr_t)Bm | (uintptr_t)Cm | (uintptr_t)y | (uintptr_t)h0 | (uintptr_t)h_out) % 16) == 0;
}

hipError_t launch_linear_ssd(const stree_dims &d, const void *x, const float *dt, const float *A, const void *Bm,
                             const void *Cm, const float *D, const void *h0, void *y, void *h_out, hipStream_t st) {
    // A grid dimension holds 2^32 work items; a head takes at most four workgroups of 512 lanes.  More heads than 2^20
    // go as several launches, whole sequences each.
    const int64_t T = d.nnodes, es = d.state_dtype == STREE_BF16 ? 2 : 4;
    const int per = (1 << 20) / d.nheads;
    auto at = [](auto *p, int64_t bytes) {
        typedef typename std::conditional<std::is_const<typename std::remove_pointer<decltype(p)>::type>::value, const char, char>::type byte;
        return p ? (decltype(p))((byte *)p + bytes) : p;
    };
    for (int b = 0; b < d.batch; b += per) {
        stree_dims s = d;
        s.batch = d.batch - b < per ? d.batch - b : per;
        const int64_t state = (int64_t)b * d.nheads * d.headdim * d.dstate * es;
        const void *xs = at(x, b * T * d.x_stride_n * 2), *Bs = at(Bm, b * T * d.b_stride_n * 2);
        const void *Cs = at(Cm, b * T * d.c_stride_n * 2), *hs = at(h0, state);
        const float *ds = at(dt, b * T * d.nheads * 4);
        void *ys = at(y, b * T * d.nheads * d.headdim * 2), *ho = at(h_out, state);
        const hipError_t e = d.state_dtype == STREE_BF16 ? launch_h<bf16_t>(s, xs, ds, A, Bs, Cs, D, hs, ys, ho, st)
                                                         : launch_h<float>(s, xs, ds, A, Bs, Cs, D, hs, ys, ho, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace stree
