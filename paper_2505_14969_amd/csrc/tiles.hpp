// LDS tiles and matrix operands shared by the kernels whose products are chained through registers.
#pragma once
#include "common.hpp"

namespace stree {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// LDS by byte address: a tile's accesses differ by a few flipped address bits, which is then one
// instruction (through pointers it is a flip and an addition).
template <typename V>
__device__ __forceinline__ __attribute__((address_space(3))) V &lds_at(uint32_t addr) {
    return *(__attribute__((address_space(3))) V *)(uintptr_t)addr;
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {      // bf16 pair, round to nearest even
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// 16-bit transposing read: the 16 lanes of a group each pass the address of 4 elements (lane i: row
// i/4, column quad i%4 of a 4 x 16 block) and lane i receives column i of the block's four rows.
__device__ __forceinline__ s16x4 read_transposed(uint32_t addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(&lds_at<s16x4>(addr));
}
__device__ __forceinline__ bf16x8 join(s16x4 a, s16x4 b) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// LDS written by some lanes of this wave is about to be read by others: the LDS pipe serves a wave
// in order, so this only keeps the compiler from moving accesses across.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS addresses differ from a lane's base address by flipped bits or a constant.  This hides the base from the
// compiler, which would otherwise keep every one of them in a register across the chunk loop (and, having computed
// it there, not see that the constant fits the instruction).
__device__ __forceinline__ uint32_t fresh(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// ---- tree scans whose waves own blocks of 32 nodes ------------------------------------------------------------------
constexpr int kRB = 32;            // nodes per row (and column) block
constexpr int kPC = 64;            // columns of a head that a workgroup takes
// Where no |s2| of a head's tree reaches this, exp(s_i - s_j) dt_j is the product of a factor per row and one per
// column instead of an exponential per pair (16 of a lane's some 100 instructions a tile, each four times as long).
constexpr float kNarrow = 64.f;

// Rows of S bf16 in LDS: the 16-byte pieces of a row are permuted by the row, so that 16 rows' reads of one piece touch
// every bank once.
template <int S>
__device__ __forceinline__ uint32_t piece_at(int row, int piece) {
    return row * (S * 2) + ((piece ^ (S == 64 ? (row >> 1) & 7 : row & 15)) << 4);
}

// bit `b` of w as a mask (the compiler would compare and select, an instruction more)
__device__ __forceinline__ uint32_t bit_as_mask(uint32_t w, int b) {
    uint32_t m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(w), "i"(b));
    return m;
}
// x as tiles of 32 columns, 64 bytes a row: its four pieces permuted by the row's quad, for the lanes that read one
// piece of 32 rows (the transposing read takes whole quads of rows).
__device__ __forceinline__ uint32_t x_piece_at(int row, int piece) { return row * 64 + ((piece ^ ((row >> 2) & 3)) << 4); }

// The previous iteration's tree and cached activations (replay).
struct ReplayArgs {
    const int32_t *parent, *accepted;   // [B, pn], [B]
    const bf16_t *x, *Bm;               // [B, pn, H, P], [B, pn, G, S] with token strides x_sn, b_sn
    const float *dt;                    // [B, pn, H]
    long x_sn, b_sn;
    int pn;
    void *h_out;                        // [B, H, P, S]: the replayed state, in the type the state is kept in
    int32_t *status;                    // [B] or null
};

// The state of a replay in a workgroup's registers: the accumulators of the fp32 matrix instructions that advance it (16 x
// 16 x 4, accumulator row = state row p, column = state column s).  A wave owns 16 rows, lane l the rows 4 (l >> 4) + i of those
// and kCW consecutive columns kCW (l & 15) + t -- column t of each lane makes up tile t, so that a lane's columns are 16-byte
// pieces in memory (8 bytes for a bf16 state of 64 columns).
template <int S, typename HT>
struct StateTiles {
    static constexpr int kCW = (sizeof(HT) == 2 && S % 128 == 0) ? 8 : 4, kCols = S / (16 * kCW);   // columns per piece; column blocks
    static constexpr int kBytes = kCW * (int)sizeof(HT), kPieces = 4 * kCols;
    typedef floatx4 Values[kCols][kCW];               // [column block][tile]

    // piece q of a thread whose rows are row0 + 0 .. 3 and whose first column is col0: row q % 4, column block q / 4
    static __device__ __forceinline__ void request(u32x4 (&r)[kPieces], __amdgpu_buffer_rsrc_t state, int row0, int lane16) {
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const int at = ((row0 + q % 4) * S + (q / 4 * 16 + lane16) * kCW) * (int)sizeof(HT);
            if constexpr (kBytes == 16) {
                r[q] = __builtin_amdgcn_raw_buffer_load_b128(state, at, 0, 2);     // nt
            } else {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(state, at, 0, 2);
                r[q].x = v.x;
                r[q].y = v.y;
            }
        }
    }
    static __device__ __forceinline__ void widen(Values &hv, const u32x4 (&r)[kPieces], float scale) {
#pragma unroll
        for (int q = 0; q < kPieces; ++q)
#pragma unroll
            for (int e = 0; e < kCW; ++e)
                hv[q / 4][e][q % 4] = scale * (sizeof(HT) == 4 ? __uint_as_float(r[q][e % 4])
                                               : (e & 1) ? bf16_hi(r[q][e / 2]) : bf16_lo(r[q][e / 2]));
    }
    // Four path nodes a turn: lane group kj holds node j of them, its weight (0 past the end of the path), its x at row l of
    // the wave's rows (operand A) and weight * B at the lane's columns (operand B).  `rows`: nl nodes' x rows, then the B rows
    // of all `room` nodes; `weights`: theirs.
    // (STEPWISE: one column block's operands at a time, where registers are short.)
    template <bool STEPWISE>
    static __device__ __forceinline__ void advance(Values &hv, uint32_t rows, int room, uint32_t weights, int nl, int prow, int l, int kj) {
        for (int j0 = 0; j0 < nl; j0 += 4) {
            const bool on = j0 + kj < nl;
            const int j = min(j0 + kj, nl - 1);
            const float cf_j = lds_at<float>(weights + j * 4);
            const uint32_t xw = lds_at<unsigned short>(rows + (j * kPC + prow + l) * 2);
            const float av = on ? __uint_as_float(xw << 16) : 0.f;
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                uint32_t bw[kCW / 2];
#pragma unroll
                for (int w = 0; w < kCW / 2; w += 2) {
                    const u32x2 v = lds_at<u32x2>(rows + (room * kPC + j * S + (c * 16 + l) * kCW + 2 * w) * 2);
                    bw[w] = v.x;
                    bw[w + 1] = v.y;
                }
#pragma unroll
                for (int e = 0; e < kCW; ++e) {
                    const float bv = on ? cf_j * ((e & 1) ? bf16_hi(bw[e / 2]) : bf16_lo(bw[e / 2])) : 0.f;
                    hv[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, hv[c][e], 0, 0, 0);
                }
                if constexpr (STEPWISE) __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // The replayed state, written once (never read again by this kernel), to memory and as bf16 to the tile; a bf16 state is
    // rounded once: the value written back is the operand.
    static __device__ __forceinline__ void store(const Values &hv, __amdgpu_buffer_rsrc_t state, uint32_t tile, uint32_t row0, uint32_t lane16) {
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const uint32_t row = row0 + q % 4, col = (q / 4 * 16 + lane16) * kCW;
            uint32_t w[kCW / 2];
#pragma unroll
            for (int e = 0; e < kCW; e += 2) w[e / 2] = pack2(hv[q / 4][e][q % 4], hv[q / 4][e + 1][q % 4]);
            const uint32_t dst = (uint32_t)(row * S + col) * (uint32_t)sizeof(HT);
            const uint32_t op = tile + piece_at<S>(row, col / 8);
            if constexpr (sizeof(HT) == 4)
                buffer_store_through16(state, dst, make_uint4(__float_as_uint(hv[q / 4][0][q % 4]), __float_as_uint(hv[q / 4][1][q % 4]),
                                                              __float_as_uint(hv[q / 4][2][q % 4]), __float_as_uint(hv[q / 4][3][q % 4])));
            if constexpr (kCW == 8) {
                buffer_store_through16(state, dst, make_uint4(w[0], w[1], w[2], w[3]));
                lds_at<u32x4>(op) = u32x4{w[0], w[1], w[2], w[3]};
            } else {
                if constexpr (sizeof(HT) == 2)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, state, (int)dst, 0, 1 | 2 | 16);
                lds_at<u32x2>(op + (col & 4) * 2) = u32x2{w[0], w[1]};
            }
        }
    }
};

// A state that is not replayed: whole rows in consecutive threads' registers (piece q: the T threads' q-th 16 bytes each), to
// the tile as bf16.
template <int S, int T, typename HT, int N>
__device__ __forceinline__ void stage_state(const u32x4 (&r)[N], uint32_t tile, uint32_t t) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        if constexpr (sizeof(HT) == 4) {
            const uint32_t e = (q * T + t) * 4;
            lds_at<u32x2>(tile + piece_at<S>(e / S, e % S / 8) + (e & 4) * 2) =
                u32x2{pack2(__uint_as_float(r[q].x), __uint_as_float(r[q].y)), pack2(__uint_as_float(r[q].z), __uint_as_float(r[q].w))};
        } else {                                      // a bf16 state is the operand as it comes
            const uint32_t e = (q * T + t) * 8;
            lds_at<u32x4>(tile + piece_at<S>(e / S, e % S / 8)) = r[q];
        }
    }
}

// The rows of `room` nodes of the previous tree's path, by the T threads of a workgroup: 16-byte pieces of each node's x
// row (this workgroup's kPC columns), then of its B row.  CLAMPED: threads past the end write the last piece again (a branch
// costs the scan of at most 64 nodes up to 3 %, the writes the larger one 1 %).
template <int S, int T, int room, bool CLAMPED>
struct PathRows {
    static constexpr int PX = kPC / 8, PR = PX + S / 8, kPieces = (room * PR + T - 1) / T;
    // `nodes`: the path's nodes from the first of these on, `left` of them (clamped: the last piece again past the end)
    static __device__ __forceinline__ void request(u32x4 (&r)[kPieces], const ReplayArgs &R, const char *x, const char *B, uint32_t nodes, int left, uint32_t t) {
        const int total = min(left, room) * PR;
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const uint32_t idx = min(q * T + t, (uint32_t)total - 1), c = idx % PR, node = lds_at<unsigned char>(nodes + idx / PR);
            r[q] = *reinterpret_cast<const u32x4 *>(c < PX ? x + (uint32_t)(node * (int)R.x_sn + c * 8) * 2u
                                                           : B + (uint32_t)(node * (int)R.b_sn + (c - PX) * 8) * 2u);
        }
    }
    static __device__ __forceinline__ void stage(const u32x4 (&r)[kPieces], uint32_t rows, int left, uint32_t t) {
        const int total = min(left, room) * PR;
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const uint32_t idx = CLAMPED ? min(q * T + t, (uint32_t)total - 1) : q * T + t, c = idx % PR, at = idx / PR;
            if (CLAMPED || idx < (uint32_t)total) lds_at<u32x4>(rows + (c < PX ? at * kPC + c * 8 : room * kPC + at * S + (c - PX) * 8) * 2) = r[q];
        }
    }
};

// Gt -> the operand of Yt += X^T M, in place: times exp(s_i - s_j) dt_j, cleared where j is not on node i's path (bit
// 8(r/4) + r%4 of `word` <-> Gt's register r), as bf16.  u_at: this half's first quad of u; `wide`: see kNarrow.
__device__ __forceinline__ void weigh(u32x4 (&m)[2], const floatx16 &gt, uint32_t word, uint32_t u_at, float s2_i, float e_i, int wide) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 u = lds_at<f32x4>(u_at + 8 * q * 4);
        float v[4];
        f32x4 f;
        if (wide) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = __builtin_amdgcn_exp2f(s2_i - u[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = e_i * u[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)                   // bitwise select: an overflow under a cleared mask bit never reaches M
            v[e] = __uint_as_float(__float_as_uint(gt[4 * q + e] * f[e]) & bit_as_mask(word, 8 * q + e));
        m[q / 2][2 * (q % 2)] = pack2(v[0], v[1]);
        m[q / 2][2 * (q % 2) + 1] = pack2(v[2], v[3]);
        // (formed here: the compiler would put all of this off to the end, behind the branches, and keep f until then)
        asm volatile("" : "+v"(m[q / 2][2 * (q % 2)]), "+v"(m[q / 2][2 * (q % 2) + 1]));
    }
}

}  // namespace

}  // namespace stree
