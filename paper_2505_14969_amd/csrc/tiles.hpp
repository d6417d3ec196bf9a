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

}  // namespace

}  // namespace stree
