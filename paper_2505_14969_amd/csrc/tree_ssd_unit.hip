// Tree scan for trees of at most 64 nodes, the shape of a speculative-decoding step: a workgroup of four waves per
// (sequence, head), small enough that five of them share a CU.
//
//   y_i = exp(s_i) h0 C_i + sum_{j on path(i)} exp(s_i - s_j) dt_j <C_i, B_j> x_j + D x_i
//
// Products and operand layouts are those of tree_ssd_rows.hip; a wave owns 32 nodes x 32 columns.  One tile of LDS holds
// one after the other what the products need: C on its way to the registers, the state, B.
//
//   requests: tree, previous tree (RP), C, x, state
//   wave 0: the tree's index     wave 3 (RP): the previous tree's path and its weights     all: C to LDS
//   -- C to registers; RP: the path's x and B rows to LDS -- state (RP: advanced along the path in the registers it came
//   in, written back once) to LDS as bf16 -- Yt = exp(s_i) h0b C^T -- B to LDS -- per column block Gt = B C^T, weighted and
//   masked in place, Yt += X^T M -- y = Yt + D x in the place of x, stored as pieces of rows
//
// RP folds the commit of the previous tree (Alg. 1: replay at the start of the next iteration) into the state as it passes
// through the registers:  h* = exp(s_k) h0 + sum_{j on path(k)} dt_j exp(s_k - s_j) x_j (outer) B_j.
//
// What bounds it: few heads -- the chain of dependent steps, some 1800 instructions of a wave; many -- issue slots and
// memory together (bf16 state, 64 x 49 nodes: 4.3 TB/s; fp32, 64 x 64: 5.2).  So: registers for five waves a SIMD (the
// state is advanced and done with before B is requested; five workgroups where four take 59 us for 64 x 49 nodes, 57);
// two chains, of the tree and of the path, on two waves at once; divisions by arguments as multiplications.
// Before, persistent workgroups of eight waves with alternating roles, replay + scan, 80 heads, S = 128: 1 x 15 nodes
// 7.8 -> 6.7 us, 4 x 29 11.0 -> 8.9, 16 x 16 21.5 -> 20.3, 64 x 64 86 -> 78, 64 chains of 64 158 -> 93; bf16 state, 64 x
// 49 nodes 66 -> 51; 40 heads of 128, 16 x 40 26.7 -> 22.8; scan alone, 1 x 15 nodes 5.6 -> 4.5.
#include "common.hpp"
#include "launch.hpp"
#include "tiles.hpp"
#include <type_traits>

namespace stree {

namespace {

template <int S, bool RP>
struct UnitLds {
    static constexpr int tile = 0, x = tile + kPC * S * 2, s2 = x + 64 * kPC * 2, u = s2 + 256, mask = u + 256;
    static constexpr int flags = mask + 512, tree_end = flags + 32;              // bad, wide, previous bad, path length, exp(s_k)
    static constexpr int kPath = 15;                                             // path rows held at a time
    static constexpr int weight = tree_end, node = weight + 256, rows = RP ? node + 64 : tree_end;
    static constexpr int row_bytes = RP ? kPath * (kPC + S) * 2 : 0;             // (y of the lower nodes is turned around there, too)
    static constexpr int size = rows + (row_bytes > 4096 ? row_bytes : 4096);
    static constexpr int per_cu = 128 / ((size + 1279) / 1280);                  // LDS is handed out in 1280 bytes
};

// LATE: the state is requested behind C, x and the path's rows instead of ahead of them.
template <int S, int WPE, bool RP, bool LATE, typename HT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void tree_ssd_unit_kernel(
    const int32_t *__restrict__ parent, int n, int units, Divisor H, Divisor per_group, int P, const bf16_t *__restrict__ x, long x_sn,
    const float *__restrict__ dt, const float *__restrict__ dt_bias, const float *__restrict__ A,
    const bf16_t *__restrict__ Bm, long b_sn, const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D,
    const HT *h0, bf16_t *__restrict__ y, int32_t *__restrict__ status, ReplayArgs R) {
    using L = UnitLds<S, RP>;
    constexpr int NK = S / 16, kPieces = S / 8;
    constexpr int NR = 64 * kPieces / 256, kStep = 256 / kPieces;      // pieces of 64 rows per thread; rows between them
    constexpr int NH = kPC * S * (int)sizeof(HT) / 16 / 256;           // of the state
    constexpr int kAhead = 4;                                          // operands in flight ahead of a product's k step
    __shared__ __align__(512) char lds[L::size];
    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int halves = P / kPC, bh = halves == 2 ? unit >> 1 : unit, p0 = halves == 2 ? (unit & 1) * kPC : 0;
    const int b = H.quotient(bh), h = bh - b * H.d, g = per_group.quotient(h);
    // nodes 32 I .. 32 I + 31 and columns 32 pt .. of this wave; the waves of a workgroup go to the four SIMDs in turn and
    // the upper nodes have the more to do, so every other workgroup of a CU turns the order around
    const int I = (wave ^ (int)(blockIdx.x >> 8)) & 1, pt = wave >> 1;

    // ---- requests, in the order in which they are waited for -------------------------------------------------
    int par = -1;
    float d_ = 0.f;
    if (wave == 0) {
        const uint32_t at = (uint32_t)(b * n + min(lane, n - 1));
        par = parent[at];
        d_ = dt[at * (uint32_t)H.d + (uint32_t)h];
    } else if (RP && wave == 3) {
        const uint32_t at = (uint32_t)(b * R.pn + min(lane, R.pn - 1));
        par = R.parent[at];
        d_ = R.dt[at * (uint32_t)H.d + (uint32_t)h];
    }
    __builtin_amdgcn_sched_barrier(0);
    // (buffers that end with the sequence's last row: rows past the tree read as zeros)
    const auto rows_of = [&](const bf16_t *first, long sn, int width) {
        return make_buffer(first + (uint64_t)(uint32_t)(b * n) * (uint32_t)sn, (size_t)((uint32_t)((n - 1) * (int)sn + width) * 2u));
    };
    auto request = [&](auto &r, __amdgpu_buffer_rsrc_t rows, int sn, uint32_t row, uint32_t at, int step) {    // row, row + step, ...
        uint32_t off = (uint32_t)(row * sn + at * 8) * 2u;
#pragma unroll
        for (auto &v : r) {
            v = __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, 0);
            off += (uint32_t)(step * sn) * 2u;
        }
    };
    u32x4 rr[NR], xr[2];               // C rows, later B rows; x rows
    const uint32_t t_row = tid / kPieces, t_piece = tid % kPieces;
    request(rr, rows_of(Cm + (size_t)g * S, c_sn, S), (int)c_sn, t_row, t_piece, kStep);      // whole rows to consecutive lanes
    request(xr, rows_of(x + (size_t)h * P + p0, x_sn, kPC), (int)x_sn, tid / 8, tid % 8, 32);
    __builtin_amdgcn_sched_barrier(0);
    // The state: with the replay as the tiles that advance it, else as whole rows.
    using Tiles = StateTiles<S, HT>;
    constexpr int NHR = RP ? Tiles::kPieces : NH;
    u32x4 hr[NHR];
    auto request_state = [&]() {   // (a buffer, empty without a state: no branch that the registers would have to agree behind)
        const auto hbuf = make_buffer(h0 + (uint64_t)(uint32_t)bh * (uint32_t)(P * S) + (uint32_t)(p0 * S), h0 ? (size_t)kPC * S * sizeof(HT) : 0);
        if constexpr (RP) {
            Tiles::request(hr, hbuf, wave * 16 + (lane >> 4) * 4, lane & 15);
        } else {
#pragma unroll
            for (int q = 0; q < NHR; ++q) hr[q] = __builtin_amdgcn_raw_buffer_load_b128(hbuf, (q * 256 + tid) * 16, 0, 2);   // nt
        }
    };
    if constexpr (!LATE) request_state();
    __builtin_amdgcn_sched_barrier(0);

    // ---- the tree's index (Sec. 3: depth-ordered packing, Eq. a_tree), in log2 units: lane = node ------------------
    //   s2[i] = log2(e) s_i      u[j] = s2[j] - log2(dt_j)      exp(s_i - s_j) dt_j = exp2(s2[i] - u[j])
    // or, where no |s2| is large, u[j] = exp2(-s2[j]) dt_j: a factor of its own
    const float A_h = A[h], bias_h = dt_bias ? dt_bias[h] : 0.f;
    if (wave == 0) {
        if (dt_bias) d_ = softplus_step(d_ + bias_h);            // raw projection -> step size
        if (lane >= n) d_ = 0.f;
        const bool ok = lane >= n || ((lane == 0) ? (par == -1) : (par >= 0 && par < lane));
        const unsigned long long bm = __ballot(!ok);
        int j = (lane < n && ok) ? par : -1;
        float s = d_ * A_h * 1.44269504088896340736f;
        uint32_t mlo = (lane < n && lane < 32) ? 1u << lane : 0u, mhi = (lane < n && lane >= 32) ? 1u << (lane - 32) : 0u;
        for (int round = 0; round < 6; ++round) {                // pointer doubling, in registers
            const bool in = j >= 0;
            if (!__any(in)) break;
            const int q = in ? j : lane;
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
        const bool any_wide = __any(!(fabsf(s) < kNarrow));
        lds_at<float>(base + L::s2 + lane * 4) = s;
        lds_at<float>(base + L::u + lane * 4) = any_wide ? s - __log2f(d_) : d_ * __builtin_amdgcn_exp2f(-s);   // dt = 0: weight 0
        lds_at<uint32_t>(base + L::mask + lane * 4) = mlo;
        lds_at<uint32_t>(base + L::mask + 256 + lane * 4) = mhi;
        if (lane == 0) {
            const int bad = bm ? (int)__ffsll((long long)bm) : 0;
            lds_at<int>(base + L::flags) = bad;
            lds_at<int>(base + L::flags + 4) = any_wide;
            if (status && h == 0 && p0 == 0) status[b] = bad;
        }
    } else if (RP && wave == 3) {
        // The previous tree's path: ancestor bits by pointer doubling, then the weights along it.  exp(s_k - s_j) is the
        // exponential of the sum over the nodes BEHIND j, summed along the path itself (ancestors have smaller labels:
        // lanes in ascending order are the path root first): its rounding error is relative to that sum, which is small
        // wherever the weight is not negligible.
        const int k = R.accepted[b], pn = R.pn;
        const bool k_bad = k < -1 || k >= pn;
        if (dt_bias) d_ = softplus_step(d_ + bias_h);
        const bool ok = lane >= pn || ((lane == 0) ? (par == -1) : (par >= 0 && par < lane));
        const unsigned long long bm = __ballot(!ok);
        const int bad = bm ? (int)__ffsll((long long)bm) : 0;
        int len = 0;
        float whole = 0.f;
        if (!bad && k >= 0 && !k_bad) {                          // (else the state passes through)
            int j = lane < pn ? par : -1;
            uint32_t mlo = lane < 32 ? 1u << lane : 0u, mhi = lane >= 32 ? 1u << (lane - 32) : 0u;
            for (int round = 0; round < 6; ++round) {
                const bool in = j >= 0;
                if (!__any(in)) break;
                const int q = in ? j : lane;
                const int rj = wave_read(j, q);
                const uint32_t rlo = wave_read(mlo, q), rhi = wave_read(mhi, q);
                if (in) {
                    mlo |= rlo;
                    mhi |= rhi;
                    j = rj;
                }
            }
            const int ku = __builtin_amdgcn_readfirstlane(k);
            const unsigned long long path = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)mhi, ku) << 32) |
                                            (uint32_t)__builtin_amdgcn_readlane((int)mlo, ku);
            len = __popcll(path);
            const bool on = (path >> lane) & 1ull;
            float t = on ? d_ * A_h : 0.f;                       // suffix sums: inside rows of 16 lanes, then the rows behind
            t += dpp_move<0x101, 0xf, true>(t);
            t += dpp_move<0x102, 0xf, true>(t);
            t += dpp_move<0x104, 0xf, true>(t);
            t += dpp_move<0x108, 0xf, true>(t);
            const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 16));
            const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 32));
            const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 48));
            t += lane < 16 ? r1 + (r2 + r3) : lane < 32 ? r2 + r3 : lane < 48 ? r3 : 0.f;
            whole = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
            float behind = dpp_move<0x130, 0xf, true>(t);        // wave_shl:1
            if (lane == 63) behind = 0.f;
            if (on) {
                const int pos = __popcll(path & ((1ull << lane) - 1ull));
                lds_at<unsigned char>(base + L::node + pos) = (unsigned char)lane;
                lds_at<float>(base + L::weight + pos * 4) = d_ * __expf(behind);
            }
        }
        if (lane == 0) {
            lds_at<int>(base + L::flags + 12) = len;
            lds_at<float>(base + L::flags + 16) = __expf(whole); // (no path: 1)
            if (R.status && h == 0 && p0 == 0) R.status[b] = bad ? bad : (k_bad ? -1 : 0);
        }
    }
    // ---- C and x to LDS ------------------------------------------------------------------------------------------
    auto stage_rows = [&]() {
        const uint32_t t = fresh(tid), r = t / kPieces, c = t % kPieces;
#pragma unroll
        for (int q = 0; q < NR; ++q) lds_at<u32x4>(base + L::tile + piece_at<S>(q * kStep + r, c)) = rr[q];
    };
    stage_rows();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        lds_at<u32x4>(base + L::x + (tid & 4) / 4 * 4096 + x_piece_at(q * 32 + tid / 8, tid & 3)) = xr[q];
    __syncthreads();

    // ---- C to registers; the path's rows ---------------------------------------------------------------------------
    // the lane's row of a tile of rows: k step kk lies at ^ (kk << 5)
    const uint32_t row_at = base + L::tile + piece_at<S>(l32, lh);
    bf16x8 cf[NK];
    {
        const uint32_t c_at = fresh(row_at + I * (kRB * S * 2));
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) cf[kk] = lds_at<bf16x8>(c_at ^ (kk << 5));
    }
    const int bad = __builtin_amdgcn_readfirstlane(lds_at<int>(base + L::flags));
    using Path = PathRows<S, 256, L::kPath, true>;
    [[maybe_unused]] int plen = 0;
    u32x4 pr[Path::kPieces];
    [[maybe_unused]] auto request_path = [&](int first) {
        const char *xb = reinterpret_cast<const char *>(R.x + (uint64_t)(uint32_t)(b * R.pn) * (uint32_t)R.x_sn + (size_t)h * P + p0);
        const char *Bp = reinterpret_cast<const char *>(R.Bm + (uint64_t)(uint32_t)(b * R.pn) * (uint32_t)R.b_sn + (size_t)g * S);
        Path::request(pr, R, xb, Bp, base + L::node + first, plen - first, fresh(tid));
    };
    [[maybe_unused]] auto stage_path = [&](int first) { Path::stage(pr, base + L::rows, plen - first, fresh(tid)); };
    if constexpr (RP) {
        plen = __builtin_amdgcn_readfirstlane(lds_at<int>(base + L::flags + 12));
        if (plen > 0) request_path(0);
    } else if (bad) {                                            // (uniform) the sequence's outputs are zeros
        bf16_t *yb = y + (uint64_t)(uint32_t)(b * n) * (uint32_t)(H.d * P) + (uint32_t)(h * P + p0);
        for (int i = (int)tid / 8; i < n; i += 32)
            *reinterpret_cast<uint4 *>(yb + (size_t)i * H.d * P + tid % 8 * 8) = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LATE) request_state();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (RP) {
        if (plen > 0) stage_path(0);
    }
    __syncthreads();                                  // the C tile is dead, the path's rows are there

    // ---- the state to LDS ------------------------------------------------------------------------------------------
    if constexpr (RP) {
        const uint32_t ft = fresh(tid), l = ft & 15, kj = (ft & 63) >> 4, prow = (ft >> 6) * 16;
        const float dec = lds_at<float>(base + L::flags + 16);
        typename Tiles::Values hv;
        Tiles::widen(hv, hr, dec);
        for (int first = 0; first < plen; first += L::kPath) {
            if (first > 0) {                          // longer paths: the next rows, a round trip for fifteen
                request_path(first);
                __syncthreads();
                stage_path(first);
                __syncthreads();
            }
            Tiles::template advance<true>(hv, base + L::rows, L::kPath, base + L::weight + first * 4, min(plen - first, L::kPath), prow, l, kj);
        }
        const auto ho = make_store_rsrc(reinterpret_cast<HT *>(R.h_out) + (uint64_t)(uint32_t)bh * (uint32_t)(P * S) + (uint32_t)(p0 * S), (uint32_t)(kPC * S * sizeof(HT)));
        const uint32_t wt = fresh(tid);
        Tiles::store(hv, ho, base + L::tile, (wt >> 6) * 16 + ((wt & 63) >> 4) * 4, wt & 15);
        if (bad) {                                    // (uniform) the state is replayed, the outputs are zeros
            bf16_t *yb = y + (uint64_t)(uint32_t)(b * n) * (uint32_t)(H.d * P) + (uint32_t)(h * P + p0);
            for (int i = (int)tid / 8; i < n; i += 32)
                *reinterpret_cast<uint4 *>(yb + (size_t)i * H.d * P + tid % 8 * 8) = make_uint4(0u, 0u, 0u, 0u);
            return;
        }
    } else {
        stage_state<S, 256, HT>(hr, base + L::tile, fresh(tid));
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        const uint32_t t = fresh(tid);
        request(rr, rows_of(Bm + (size_t)g * S, b_sn, S), (int)b_sn, t / kPieces, t % kPieces, kStep);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();

    // ---- Yt = exp(s_i) h0b C^T -------------------------------------------------------------------------------------
    const int i = I * kRB + l32;
    const float s2_i = lds_at<float>(base + L::s2 + i * 4), e_i = __builtin_amdgcn_exp2f(s2_i);
    floatx16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    if (RP || h0) {
        const uint32_t h_at = fresh(row_at + pt * (kRB * S * 2));
        bf16x8 ho[kAhead];
#pragma unroll
        for (int kk = 0; kk < kAhead; ++kk) ho[kk] = lds_at<bf16x8>(h_at ^ (kk << 5));
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ho[kk % kAhead], cf[kk], acc, 0, 0, 0);
            if (kk + kAhead < NK) ho[kk % kAhead] = lds_at<bf16x8>(h_at ^ ((kk + kAhead) << 5));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();                                  // the state tile is dead
    stage_rows();                                     // B
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] *= e_i;

    // ---- column blocks ---------------------------------------------------------------------------------------------
    const int wide = __builtin_amdgcn_readfirstlane(lds_at<int>(base + L::flags + 4));
    const uint32_t x_tile = base + L::x + pt * 4096;
    // the lane's place in the transposing reads of an x tile
    const uint32_t x_lane = x_tile + x_piece_at(4 * lh + ((lane & 15) >> 2), ((lane >> 4) & 1) * 2 + ((lane & 2) >> 1)) + (lane & 1) * 8;
    if (I * kRB >= n) return;
#pragma unroll 1
    for (int J = 0; J <= I; ++J) {
        const uint32_t b_at = fresh(row_at + J * (kRB * S * 2));
        floatx16 gt;
#pragma unroll
        for (int e = 0; e < 16; ++e) gt[e] = 0.f;
        bf16x8 bo[kAhead];                            // (operands a few k steps ahead, not all at once: register budget)
#pragma unroll
        for (int kk = 0; kk < kAhead; ++kk) bo[kk] = lds_at<bf16x8>(b_at ^ (kk << 5));
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            gt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bo[kk % kAhead], cf[kk], gt, 0, 0, 0);
            if (kk + kAhead < NK) bo[kk % kAhead] = lds_at<bf16x8>(b_at ^ ((kk + kAhead) << 5));
            __builtin_amdgcn_sched_barrier(0);
        }
        const uint32_t word = lds_at<uint32_t>(base + L::mask + J * 256 + i * 4) >> (4 * lh), u_at = fresh(base + L::u + 16 * lh + J * (kRB * 4));
        u32x4 m[2];
        weigh(m, gt, word, u_at, s2_i, e_i, wide);
        const uint32_t x_at = fresh(x_lane + J * (kRB * 64));
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const uint32_t at = x_at + kk * (16 * 64);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join(read_transposed(at), read_transposed((at ^ 32) + 8 * 64)),
                                                          __builtin_bit_cast(bf16x8, m[kk]), acc, 0, 0, 0);
        }
    }
    // ---- y = Yt + D x: a lane has 4 consecutive columns of one node; turned around in LDS.  The upper nodes' y takes the
    // place of their x, which no other wave reads; the lower nodes' x belongs to the upper nodes' products as well.
    const float D_h = D ? D[h] : 0.f;
    const int ln = (int)fresh(lane);
    const uint32_t x_own = x_tile + I * 2048, y_tile = I ? x_own : base + L::rows + pt * 2048;
    u32x2 out[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const u32x2 xv = lds_at<u32x2>(x_own + x_piece_at(ln & 31, q) + (ln >> 5) * 8);
        out[q] = u32x2{pack2(fmaf(D_h, bf16_lo(xv.x), acc[4 * q]), fmaf(D_h, bf16_hi(xv.x), acc[4 * q + 1])),
                       pack2(fmaf(D_h, bf16_lo(xv.y), acc[4 * q + 2]), fmaf(D_h, bf16_hi(xv.y), acc[4 * q + 3]))};
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) lds_at<u32x2>(y_tile + x_piece_at(ln & 31, q) + (ln >> 5) * 8) = out[q];
    wave_lds_fence();
    const __amdgpu_buffer_rsrc_t yr = make_store_rsrc(y + (uint64_t)(uint32_t)(b * n) * (uint32_t)(H.d * P) + (uint32_t)(h * P + p0), (uint32_t)(n * H.d * P - h * P - p0) * 2u);
#pragma unroll
    for (int r0 = 0; r0 < kRB; r0 += 16) {
        const int row = r0 + ln / 4;
        const u32x4 v = lds_at<u32x4>(y_tile + x_piece_at(row, ln & 3));
        if (I * kRB + row < n)
            buffer_store_through16(yr, (uint32_t)((I * kRB + row) * H.d * P + pt * 32 + ln % 4 * 8) * 2u, make_uint4(v.x, v.y, v.z, v.w));
    }
}

template <int S, bool RP>
hipError_t launch_unit_s(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                         const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                         const ReplayArgs &R, hipStream_t st) {
    using L = UnitLds<S, RP>;
    constexpr int kMost = S == 256 ? 3 : 5, WPE = L::per_cu < kMost ? L::per_cu : kMost;   // waves per SIMD
    const int units = d.batch * d.nheads * (d.headdim / kPC);
    // More heads than are resident at once (five a CU, 1280) and two blocks of nodes: the workgroups of a CU are then at
    // different places of their chains, and the small requests of one need not stand behind the state of another.  Early /
    // late, us, fp32 state, S = 128: 64 nodes x 5120 heads 81.6 / 79.0 (bf16 56.9 / 55.3), 40 x 1440 26.7 / 25.8, 1280 22.9 / 23.3;
    // one block waits for the state alone: 16 x 1440 23.3 / 23.7, S = 64 14.2 / 15.8, bf16, S = 128, 16 x 1600 17.0 / 18.6; few heads
    // do at any size (4 x 29 nodes x 80 heads 8.9 / 10.0).  S = 256, where three are resident: even from 1280 to 2560 heads.
    const bool late = RP && units > 1408 && d.nnodes > kRB;
#define STREE_LAUNCH_UNIT(LATE, HT)                                                                                       \
    hipLaunchKernelGGL((tree_ssd_unit_kernel<S, WPE, RP, RP && LATE, HT>), dim3(8 * ((units + 7) / 8)), dim3(256), 0, st,       \
                       parent, d.nnodes, units, Divisor(d.nheads), Divisor(d.nheads / d.ngroups), d.headdim,        \
                       (const bf16_t *)x, (long)d.x_stride_n, dt, step_bias(d), A, (const bf16_t *)Bm,              \
                       (long)d.b_stride_n, (const bf16_t *)Cm, (long)d.c_stride_n, D, (const HT *)h0, (bf16_t *)y, status, R)
    if (d.state_dtype == STREE_BF16) {
        if (late) STREE_LAUNCH_UNIT(true, bf16_t);
        else STREE_LAUNCH_UNIT(false, bf16_t);
    } else {
        if (late) STREE_LAUNCH_UNIT(true, float);
        else STREE_LAUNCH_UNIT(false, float);
    }
#undef STREE_LAUNCH_UNIT
    return hipGetLastError();
}

template <bool RP>
hipError_t launch_unit(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                       const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                       const ReplayArgs &R, hipStream_t st) {
    return launch_in_parts(d, [&](const stree_dims &s, int b) {
        const int64_t nodes = (int64_t)b * s.nnodes, d_inner = (int64_t)s.nheads * s.headdim, es = s.state_dtype == STREE_BF16 ? 2 : 4;
        const int64_t state = b * d_inner * s.dstate * es;
        ReplayArgs r = R;
        if (RP) {
            const int64_t pnodes = (int64_t)b * r.pn;
            r.parent += pnodes, r.accepted += b, r.x += pnodes * r.x_sn, r.Bm += pnodes * r.b_sn, r.dt += pnodes * s.nheads;
            r.h_out = advance(r.h_out, state), r.status = advance(r.status, b);
        }
        const auto launch = s.dstate == 64 ? launch_unit_s<64, RP> : s.dstate == 128 ? launch_unit_s<128, RP> : launch_unit_s<256, RP>;
        return launch(s, parent + nodes, advance(x, nodes * s.x_stride_n * 2), dt + nodes * s.nheads, A,
                      advance(Bm, nodes * s.b_stride_n * 2), advance(Cm, nodes * s.c_stride_n * 2), D, advance(h0, state),
                      advance(y, nodes * d_inner * 2), advance(status, b), r, st);
    });
}

}  // namespace

hipError_t launch_tree_ssd_unit(const stree_dims &d, const int32_t *parent, const void *x, const float *dt,
                                const float *A, const void *Bm, const void *Cm, const float *D, const void *h0,
                                void *y, int32_t *status, hipStream_t st) {
    return launch_unit<false>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, ReplayArgs{}, st);
}

hipError_t launch_tree_ssd_replay_unit(const stree_dims &d, const stree_dims &dp, const int32_t *pparent,
                                       const int32_t *paccepted, const void *px, const float *pdt, const void *pB,
                                       const int32_t *parent, const void *x, const float *dt, const float *A,
                                       const void *Bm, const void *Cm, const float *D, const void *h0,
                                       void *h_out, void *y, int32_t *status, int32_t *rstatus, hipStream_t st) {
    const ReplayArgs R = {pparent, paccepted, (const bf16_t *)px, (const bf16_t *)pB, pdt,
                          (long)dp.x_stride_n, (long)dp.b_stride_n, dp.nnodes, h_out, rstatus};
    return launch_unit<true>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, R, st);
}

}  // namespace stree
