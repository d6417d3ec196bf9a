// Tree scan for trees of 65 .. 256 nodes: a workgroup per (sequence, head), whose waves own blocks of 32 nodes.
//
//   y_i = exp(s_i) h0 C_i + sum_{j on path(i)} exp(s_i - s_j) dt_j <C_i, B_j> x_j + D x_i
//
// All products are formed transposed, so that a lane owns one node i in every accumulator, and they are chained
// through registers (the k order of a product is free as long as both operands agree):
//   for each block J <= I of 32 columns:
//     Gt[j][i] = B_J C_I^T                           B rows from LDS, C rows in registers (through LDS once)
//     M = L ? Gt exp(s_i - s_j) dt_j : 0 -> bf16     in place: registers 8kk .. 8kk+7 of the 32 x 32 accumulator ARE
//                                                    the operand whose k slot e of half lh is node 16kk + 8(e/4) + 4lh + e%4
//     Yt += X_J^T M                                  x from row-major LDS through the transposing LDS read
//   y = exp(s_i) h0b C^T + Yt + D x, in the place of x in LDS, stored as whole rows
// A wave meets the others while the tree's index is built, when B and x are in LDS, at every fourth column block (new B
// rows) and when the state is in LDS; in between it runs its row block alone, with no tile of its own to stage.
//
// What bounds it: the chain of a workgroup -- requests, index, products, state, stores -- of which two or three are
// resident on a CU.  The state, half of all bytes, is requested last and used last: it streams in while the products are
// formed, and nothing small waits behind it.  Operands read from memory as a product wants them (a lane its own row, 32
// bytes of 32 rows an instruction) cost an L1 look-up a row: 27 us for 4 x 256 nodes where whole rows through LDS take 24.
// Before, persistent workgroups of alternating roles with two barriers per pair of 64-node blocks (fp32 state, cold):
// 8 x 128 nodes x 80 heads 19.8 -> 14.7 us, 16 x 128 30.7 -> 23.3, 16 x 81 29.9 -> 20.0, 4 x 256 x 128 heads 33.6 -> 23.7,
// 16 x 256 x 80 68.7 -> 50.4; 16 x 128 x 40 heads of 128 42.0 -> 23.3; 16 x 128 x 32 heads, S = 256, 24.1 -> 18.0.
#include "common.hpp"
#include "launch.hpp"
#include "tiles.hpp"
#include <type_traits>

namespace stree {

namespace {

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

// LDS of a workgroup for NR node blocks, in bytes: the rows of B for one phase (behind the last one the state tile),
// x, which y takes the place of, and the tree.  C passes through the B and x tiles on its way in.
template <int S, int NR>
struct RowsLds {
    static constexpr int kNodes = NR * kRB;
    static constexpr int kCB = S == 256 ? 2 : 4;                                 // column blocks per phase
    static constexpr int bm = 0, x = bm + kCB * kRB * S * 2, s2 = x + kNodes * kPC * 2;
    static constexpr int u = s2 + kNodes * 4, mask = u + kNodes * 4, bad = mask + NR * kNodes * 4, size = bad + 32;
    static constexpr int c_cols = S >= 128 && NR * kRB * 256 <= s2 ? 128 : 64;   // columns of C per trip
    static_assert(kCB * kRB >= kPC && NR * kRB * c_cols * 2 <= s2, "");
    static constexpr int per_cu = 160 * 1024 / size;
};

template <int S, int NR, int WPE, typename HT>
__global__ __launch_bounds__(64 * NR) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void tree_ssd_rows_kernel(
    const int32_t *__restrict__ parent, int n, int units, int H, int G, int P, const bf16_t *__restrict__ x, long x_sn,
    const float *__restrict__ dt, const float *__restrict__ dt_bias, const float *__restrict__ A,
    const bf16_t *__restrict__ Bm, long b_sn, const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D,
    const HT *__restrict__ h0, bf16_t *__restrict__ y, int32_t *__restrict__ status) {
    using L = RowsLds<S, NR>;
    constexpr int T = 64 * NR, NK = S / 16, kPieces = S / 8, kNodes = L::kNodes;
    constexpr int NH = kPC * S * (int)sizeof(HT) / 16 / T;      // 16-byte pieces of the state per thread
    constexpr int kCB = L::kCB, NB = kCB * kRB * kPieces / T;                   // of the B rows of a phase
    constexpr int kRowsX = T / 8, NX = kNodes / kRowsX;         // rows of x per round; rounds
    constexpr int kAhead = NR == 8 ? 2 : 4;
    constexpr int kSlots = NR / 2;                              // groups of 64 nodes, a wave each for the index
    static_assert(NH >= 1 && NB >= 1 && NX == 4, "");
    __shared__ __align__(512) char lds[L::size];

    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int halves = P / kPC, bh = unit / halves, p0 = unit % halves * kPC;
    const int b = bh / H, h = bh % H, g = h / (H / G);
    const int nblk = (n + kRB - 1) / kRB, phases = (nblk + kCB - 1) / kCB;
    // The row block of this wave.  The waves of a workgroup go to the four SIMDs in turn and block I has I + 1 column
    // blocks: of eight, a long and a short one share a SIMD; of four, every other workgroup turns the order around.
    const int I = NR == 8 ? (wave < 4 ? wave : 11 - wave) : (blockIdx.x >> 8) & 1 ? NR - 1 - wave : wave;
    const int last = I < nblk ? I : -1;               // its last column block

    // ---- requests, in the order in which they are waited for -------------------------------------------------
    // (rows past the tree: copies of the last one -- as columns they have no ancestor bit and weight 0, as rows they
    // are not stored)
    int par = -1;
    float d_ = 0.f;
    if (wave < kSlots) {
        const uint32_t at = (uint32_t)(b * n + min(tid, n - 1));
        par = parent[at];
        d_ = dt[at * (uint32_t)H + (uint32_t)h];
    }
    __builtin_amdgcn_sched_barrier(0);
    const char *const Cb = reinterpret_cast<const char *>(Cm + (size_t)b * n * c_sn + (size_t)g * S);
    const char *const Bb = reinterpret_cast<const char *>(Bm + (size_t)b * n * b_sn + (size_t)g * S);
    uint4 cr[NK], xr[NX];
    u32x4 br[NB];
#pragma unroll
    for (int q = 0; q < NK; ++q)                      // whole rows to consecutive lanes
        cr[q] = *reinterpret_cast<const uint4 *>(
            Cb + (uint32_t)(min(I * kRB + q * (64 / kPieces) + lane / kPieces, n - 1) * (int)c_sn + lane % kPieces * 8) * 2u);
    __builtin_amdgcn_sched_barrier(0);
    auto request_b = [&](int phase) {
        const int t = (int)fresh(tid);
#pragma unroll
        for (int q = 0; q < NB; ++q)
            br[q] = *reinterpret_cast<const u32x4 *>(
                Bb + (uint32_t)(min(phase * kCB * kRB + q * (T / kPieces) + t / kPieces, n - 1) * (int)b_sn + t % kPieces * 8) * 2u);
    };
    request_b(0);
    {
        const char *xb = reinterpret_cast<const char *>(x + (size_t)b * n * x_sn + (size_t)h * P + p0);
#pragma unroll
        for (int q = 0; q < NX; ++q)
            xr[q] = *reinterpret_cast<const uint4 *>(
                xb + (uint32_t)(min(q * kRowsX + tid / 8, n - 1) * (int)x_sn + tid % 8 * 8) * 2u);
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- the tree's index (Sec. 3: depth-ordered packing, Eq. a_tree), in log2 units ---------------------------
    //   s2[i] = log2(e) s_i      u[j] = s2[j] - log2(dt_j)      exp(s_i - s_j) dt_j = exp2(s2[i] - u[j])
    // A wave owns 64 nodes: pointer doubling among those in registers, then one merge with the first ancestor in a
    // lower wave's nodes, whose own aggregate is complete by then.  Ancestor bits: [word][node].
    const float A2 = A[h] * 1.44269504088896340736f;
    float s = 0.f;
    int j = -1;
    if (wave < kSlots) {
        if (dt_bias) d_ = softplus_step(d_ + dt_bias[h]);        // raw projection -> step size
        if (tid >= n) d_ = 0.f;
        const int node0 = wave * 64;
        const bool ok = tid >= n || ((tid == 0) ? (par == -1) : (par >= 0 && par < tid));
        const unsigned long long bm = __ballot(!ok);
        if (lane == 0) lds_at<int>(base + L::bad + wave * 4) = bm ? node0 + (int)__ffsll((long long)bm) : 0x7fffffff;
        j = (tid < n && ok) ? par : -1;
        s = d_ * A2;
        uint32_t mlo = (tid < n && lane < 32) ? 1u << lane : 0u, mhi = (tid < n && lane >= 32) ? 1u << (lane - 32) : 0u;
        for (int round = 0; round < 6; ++round) {                // chains of at most 64 nodes
            const bool in = j >= node0;
            if (!__any(in)) break;
            const int q = in ? j - node0 : lane;
            const float rs = wave_read(s, q);
            const int rj = wave_read(j, q);
            const uint32_t rlo = wave_read(mlo, q), rhi = wave_read(mhi, q);
            if (in) {
                s += rs;
                mlo |= rlo;
                mhi |= rhi;
                j = rj;
            }
        }
        lds_at<float>(base + L::s2 + tid * 4) = s;
#pragma unroll
        for (int w = 0; w < NR; ++w)
            lds_at<uint32_t>(base + L::mask + (w * kNodes + tid) * 4) = w == 2 * wave ? mlo : w == 2 * wave + 1 ? mhi : 0u;
    }
    // the lane's place in the transposing reads of an x tile (x_operand of the prefix scan, with the permuted pieces)
    const uint32_t x_lane = base + L::x + x_piece_at(4 * lh + ((lane & 15) >> 2), ((lane >> 4) & 1) * 2 + ((lane & 2) >> 1)) + (lane & 1) * 8;
    // C: from rows as they lie in memory to the lane's own row, through this wave's part of the x and B tiles
    bf16x8 cf[NK];
    {
        constexpr int kC = L::c_cols, kTrips = S / kC;
        const uint32_t c_at = base + wave * (kRB * kC * 2);
#pragma unroll
        for (int t = 0; t < kTrips; ++t) {
            if (lane % kPieces / (kC / 8) == t) {
#pragma unroll
                for (int q = 0; q < NK; ++q)
                    lds_at<u32x4>(c_at + piece_at<kC>(q * (64 / kPieces) + lane / kPieces, lane % (kC / 8))) =
                        u32x4{cr[q].x, cr[q].y, cr[q].z, cr[q].w};
            }
            wave_lds_fence();
#pragma unroll
            for (int kk = 0; kk < kC / 16; ++kk) cf[t * (kC / 16) + kk] = lds_at<bf16x8>(c_at + piece_at<kC>(l32, 2 * kk + lh));
            wave_lds_fence();
        }
    }
    __syncthreads();
    int bad = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < kSlots; ++w) bad = min(bad, lds_at<int>(base + L::bad + w * 4));
    bad = bad == 0x7fffffff ? 0 : bad;
    if (status && h == 0 && p0 == 0 && tid == 0) status[b] = bad;
    if (bad) {                                                   // (uniform) the sequence's outputs are zeros
        bf16_t *yb = y + (size_t)b * n * H * P + (size_t)h * P + p0;
        for (int i = tid / 8; i < n; i += kRowsX)
            *reinterpret_cast<uint4 *>(yb + (size_t)i * H * P + tid % 8 * 8) = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
#pragma unroll
    for (int k = 1; k < kSlots; ++k) {
        if (64 * k >= n) break;
        if (wave == k && j >= 0) {
            s += lds_at<float>(base + L::s2 + j * 4);
            lds_at<float>(base + L::s2 + tid * 4) = s;
#pragma unroll
            for (int w = 0; w < 2 * k; ++w)
                lds_at<uint32_t>(base + L::mask + (w * kNodes + tid) * 4) = lds_at<uint32_t>(base + L::mask + (w * kNodes + j) * 4);
        }
        if (k + 1 < kSlots) __syncthreads();
    }
    if (wave < kSlots) {
        const bool wide = __any(!(fabsf(s) < kNarrow));
        if (lane == 0) lds_at<int>(base + L::bad + 16 + wave * 4) = wide;
    }

    // ---- B and x to LDS ----------------------------------------------------------------------------------------
    auto stage_b = [&]() {
        const int t = (int)fresh(tid);
#pragma unroll
        for (int q = 0; q < NB; ++q)
            lds_at<u32x4>(base + L::bm + piece_at<S>(q * (T / kPieces) + t / kPieces, t % kPieces)) = br[q];
    };
    stage_b();
#pragma unroll
    for (int q = 0; q < NX; ++q)
        lds_at<u32x4>(base + L::x + (tid % 8) / 4 * (kNodes * 64) + x_piece_at(q * kRowsX + tid / 8, tid & 3)) =
            u32x4{xr[q].x, xr[q].y, xr[q].z, xr[q].w};
    __syncthreads();
    int wide = 0;
#pragma unroll
    for (int w = 0; w < kSlots; ++w) wide |= lds_at<int>(base + L::bad + 16 + w * 4);
    wide = __builtin_amdgcn_readfirstlane(wide);
    if (wave < kSlots)                                // dt = 0 (and nodes past the tree): weight 0
        lds_at<float>(base + L::u + tid * 4) = wide ? s - __log2f(d_) : d_ * __builtin_amdgcn_exp2f(-s);
    __syncthreads();

    // The state, used behind the last phase: it streams in while the products are formed.
    u32x4 hr[NH];
    {   // (a buffer, empty without a state: no branch that the registers would have to agree behind)
        const auto hbuf = make_buffer(h0 + ((size_t)bh * P + p0) * S, h0 ? (size_t)kPC * S * sizeof(HT) : 0);
#pragma unroll
        for (int q = 0; q < NH; ++q) hr[q] = __builtin_amdgcn_raw_buffer_load_b128(hbuf, (q * T + tid) * 16, 0, 2);   // nt
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- row block I, kCB column blocks a phase --------------------------------------------------------------
    const int i = I * kRB + l32;
    const float s2_i = lds_at<float>(base + L::s2 + i * 4);
    const float e_i = __builtin_amdgcn_exp2f(s2_i);
    const uint32_t mask_at = base + L::mask + i * 4;
    // the lane's row of a tile of rows: k step kk lies at ^ (kk << 5)
    const uint32_t row_at = base + L::bm + piece_at<S>(l32, lh);
    floatx16 acc[2];
#pragma unroll
    for (int pt = 0; pt < 2; ++pt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[pt][e] = 0.f;
#pragma unroll 1
    for (int phase = 0; phase < phases; ++phase) {
        if (phase > 0) {
            request_b(phase);
            __syncthreads();                          // the B rows of the phase before are dead
            stage_b();
            __syncthreads();                          // this phase's are there
        }
#pragma unroll 1
        for (int J = kCB * phase; J < kCB * (phase + 1) && J <= last; ++J) {
            const uint32_t b_at = fresh(row_at + (J & (kCB - 1)) * (kRB * S * 2));
            floatx16 gt;
#pragma unroll
            for (int e = 0; e < 16; ++e) gt[e] = 0.f;
            // (operands a few k steps ahead, not all at once: register budget)
            bf16x8 bo[kAhead];
#pragma unroll
            for (int kk = 0; kk < kAhead; ++kk) bo[kk] = lds_at<bf16x8>(b_at ^ (kk << 5));
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                gt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bo[kk % kAhead], cf[kk], gt, 0, 0, 0);
                if (kk + kAhead < NK) bo[kk % kAhead] = lds_at<bf16x8>(b_at ^ ((kk + kAhead) << 5));
                __builtin_amdgcn_sched_barrier(0);
            }
            // bit 8(r/4) + r%4 of `word` <-> Gt's register r
            const uint32_t word = lds_at<uint32_t>(mask_at + J * (kNodes * 4)) >> (4 * lh), u_at = fresh(base + L::u + 16 * lh + J * (kRB * 4));
            u32x4 m[2];
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
                for (int e = 0; e < 4; ++e)           // bitwise select: an overflow under a cleared mask bit never reaches M
                    v[e] = __uint_as_float(__float_as_uint(gt[4 * q + e] * f[e]) & bit_as_mask(word, 8 * q + e));
                m[q / 2][2 * (q % 2)] = pack2(v[0], v[1]);
                m[q / 2][2 * (q % 2) + 1] = pack2(v[2], v[3]);
                if constexpr (NR == 8) __builtin_amdgcn_sched_barrier(0);     // (register budget)
            }
            const uint32_t x_at = fresh(x_lane + J * (kRB * 64));
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int pt = 0; pt < 2; ++pt) {
                    const uint32_t at = x_at + pt * (kNodes * 64) + kk * (16 * 64);
                    acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join(read_transposed(at), read_transposed((at ^ 32) + 8 * 64)),
                                                                      __builtin_bit_cast(bf16x8, m[kk]), acc[pt], 0, 0, 0);
                    if constexpr (NR == 8) __builtin_amdgcn_sched_barrier(0);
                }
        }
    }
    __syncthreads();                                  // all products with B and x are done
    const int ft = (int)fresh(tid);
#pragma unroll
    for (int q = 0; q < NH; ++q) {
        if constexpr (sizeof(HT) == 4) {
            const int e = (q * T + ft) * 4;
            lds_at<u32x2>(base + L::bm + piece_at<S>(e / S, e % S / 8) + (e & 4) * 2) =
                u32x2{pack2(__uint_as_float(hr[q].x), __uint_as_float(hr[q].y)), pack2(__uint_as_float(hr[q].z), __uint_as_float(hr[q].w))};
        } else {                                      // a bf16 state is the operand as it comes
            const int e = (q * T + ft) * 8;
            lds_at<u32x4>(base + L::bm + piece_at<S>(e / S, e % S / 8)) = hr[q];
        }
    }
    __syncthreads();
    if (last < 0) return;
    const int ln = (int)fresh(lane);
    // y = exp(s_i) h0 C + Yt + D x: a lane has 4 consecutive columns of one node, which take the place of x
    const float D_h = D ? D[h] : 0.f;
#pragma unroll
    for (int pt = 0; pt < 2; ++pt) {
        floatx16 ch;
#pragma unroll
        for (int e = 0; e < 16; ++e) ch[e] = 0.f;
        if (h0) {
            const uint32_t h_at = fresh(row_at + pt * 32 * S * 2);
#pragma unroll
            for (int kk = 0; kk < NK; ++kk)
                ch = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    lds_at<bf16x8>(h_at ^ (kk << 5)), cf[kk], ch, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t at = base + L::x + pt * (kNodes * 64) + x_piece_at(I * kRB + (ln & 31), q) + (ln >> 5) * 8;
            const u32x2 xv = lds_at<u32x2>(at);
            const float xf[4] = {bf16_lo(xv.x), bf16_hi(xv.x), bf16_lo(xv.y), bf16_hi(xv.y)};
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(D_h, xf[e], fmaf(e_i, ch[4 * q + e], acc[pt][4 * q + e]));
            lds_at<u32x2>(at) = u32x2{pack2(v[0], v[1]), pack2(v[2], v[3])};
        }
    }
    wave_lds_fence();
    const __amdgpu_buffer_rsrc_t yr = make_store_rsrc(y + (size_t)b * n * H * P + (size_t)h * P + p0, (uint32_t)(n * H * P - h * P - p0) * 2u);
#pragma unroll
    for (int r0 = 0; r0 < kRB; r0 += 8) {             // whole rows of 128 bytes
        const int row = I * kRB + r0 + ln / 8;
        const u32x4 v = lds_at<u32x4>(base + L::x + (ln & 4) / 4 * (kNodes * 64) + x_piece_at(row, ln & 3));
        if (row < n) buffer_store_through16(yr, (uint32_t)(row * H * P + ln % 8 * 8) * 2u, make_uint4(v.x, v.y, v.z, v.w));
    }
}

template <int S, int NR>
hipError_t launch_rows_s(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                         const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                         hipStream_t st) {
    using L = RowsLds<S, NR>;
    constexpr int kFit = L::per_cu * NR / 4, kMost = S == 256 ? 2 : NR == 8 ? 4 : 3, WPE = kFit < kMost ? kFit : kMost;   // waves per SIMD
    const int units = d.batch * d.nheads * (d.headdim / kPC);
#define STREE_LAUNCH_ROWS(HT)                                                                                       \
    hipLaunchKernelGGL((tree_ssd_rows_kernel<S, NR, WPE, HT>), dim3(8 * ((units + 7) / 8)), dim3(64 * NR), 0, st,   \
                       parent, d.nnodes, units, d.nheads, d.ngroups, d.headdim, (const bf16_t *)x,                  \
                       (long)d.x_stride_n, dt, step_bias(d), A, (const bf16_t *)Bm, (long)d.b_stride_n,             \
                       (const bf16_t *)Cm, (long)d.c_stride_n, D, (const HT *)h0, (bf16_t *)y, status)
    if (d.state_dtype == STREE_BF16) STREE_LAUNCH_ROWS(bf16_t);
    else STREE_LAUNCH_ROWS(float);
#undef STREE_LAUNCH_ROWS
    return hipGetLastError();
}

}  // namespace

bool tree_ssd_rows_supported(const stree_dims &d) {
    if (d.nnodes <= 64 || d.nnodes > 256) return false;
    return (d.headdim == 64 && (d.dstate == 128 || d.dstate == 64 || d.dstate == 256)) ||
           (d.headdim == 128 && d.dstate == 128);
}

hipError_t launch_tree_ssd_rows(const stree_dims &d, const int32_t *parent, const void *x, const float *dt,
                                const float *A, const void *Bm, const void *Cm, const float *D, const void *h0,
                                void *y, int32_t *status, hipStream_t st) {
    const bool small = d.nnodes <= 128;
    if (d.dstate == 128)
        return small ? launch_rows_s<128, 4>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st)
                     : launch_rows_s<128, 8>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
    if (d.dstate == 256)
        return small ? launch_rows_s<256, 4>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st)
                     : launch_rows_s<256, 8>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
    return small ? launch_rows_s<64, 4>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st)
                 : launch_rows_s<64, 8>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
}

}  // namespace stree
