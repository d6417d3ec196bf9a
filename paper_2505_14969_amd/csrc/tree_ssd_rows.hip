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
// bytes of 32 rows an instruction) cost an L1 look-up a row: 27 us for 4 x 256 nodes where whole rows through LDS took 24.
// Before, persistent workgroups of alternating roles with two barriers per pair of 64-node blocks (fp32 state, rotating inputs):
// 8 x 128 nodes x 80 heads 19.4 -> 13.7 us, 16 x 128 29.0 -> 21.9, 16 x 81 27.2 -> 18.1, 4 x 256 x 128 heads 32 -> 18.6,
// 16 x 256 x 80 70 -> 41; 16 x 128 x 40 heads of 128 41 -> 22; 16 x 128 x 32 heads, S = 256, 24 -> 17.
//
// RP: the commit of the previous tree (Alg. 1: replay at the start of the next iteration) on the state while it passes
// through the registers, for trees of at most 128 nodes; the path is worked out beside the tree's index, its rows are
// fetched ahead of the state.  As a kernel of its own in front of the scan the commit read and wrote the state once more
// than needed: replay + scan of 16 x 81 nodes x 80 heads 46.4 -> 26.8 us, 1 x 81 19.6 -> 10.1, 32 x 100 90 -> 49 us.
#include "common.hpp"
#include "launch.hpp"
#include "tiles.hpp"
#include <type_traits>

namespace stree {

namespace {

// LDS of a workgroup for NR node blocks, in bytes: the rows of B for one phase (behind the last one the state tile),
// x, which y takes the place of, and the tree.  C passes through the B and x tiles on its way in.
template <int S, int NR, bool RP>
struct RowsLds {
    static constexpr int kNodes = NR * kRB;
    static constexpr int kCB = S == 256 ? 2 : 4;                                 // column blocks per phase
    static constexpr int bm = 0, x = bm + kCB * kRB * S * 2, s2 = x + kNodes * kPC * 2;
    static constexpr int u = s2 + kNodes * 4, mask = u + kNodes * 4, bad = mask + NR * kNodes * 4, tree_end = bad + 32;
    // replay: the previous tree's groups of nodes (where x comes later), the path (node; step size, then weight), its
    // first bad node per group and exp(s_k), the x and B rows of kPath nodes of it (in the B tile where the state leaves room)
    static constexpr int kPath = 16, row_bytes = kPath * (kPC + S) * 2;
    static constexpr int weight = tree_end, pbad = weight + kMaxNodes * 4, node = pbad + 32;
    static constexpr bool kRowsInB = kCB * kRB * S * 2 >= kPC * S * 2 + row_bytes;
    static constexpr int rows = kRowsInB ? bm + kPC * S * 2 : node + kMaxNodes;
    static constexpr int groups = kRowsInB ? x : rows;           // (free at that time)
    static constexpr int size = !RP ? tree_end : kRowsInB ? node + kMaxNodes : rows + row_bytes;
    static_assert(!RP || (kRowsInB ? kNodes * kPC * 2 : row_bytes) >= kMaxNodes * 16, "");
    static constexpr int c_cols = S >= 128 && NR * kRB * 256 <= (RP ? x : s2) ? 128 : 64;   // columns of C per trip
    static_assert(kCB * kRB >= kPC && NR * kRB * c_cols * 2 <= (RP ? x : s2), "");
    static constexpr int per_cu = 160 * 1024 / size;
};

template <int S, int NR, int WPE, bool RP, typename HT>
__global__ __launch_bounds__(64 * NR) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void tree_ssd_rows_kernel(
    const int32_t *__restrict__ parent, int n, int units, Divisor H, Divisor per_group, int P, const bf16_t *__restrict__ x, long x_sn,
    const float *__restrict__ dt, const float *__restrict__ dt_bias, const float *__restrict__ A,
    const bf16_t *__restrict__ Bm, long b_sn, const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D,
    const HT *h0, bf16_t *__restrict__ y, int32_t *__restrict__ status, ReplayArgs R) {
    using L = RowsLds<S, NR, RP>;
    constexpr int T = 64 * NR, NK = S / 16, kPieces = S / 8, kNodes = L::kNodes;
    constexpr int NH = kPC * S * (int)sizeof(HT) / 16 / T;      // 16-byte pieces of the state per thread
    constexpr int kCB = L::kCB, NB = kCB * kRB * kPieces / T;                   // of the B rows of a phase
    constexpr int kRowsX = T / 8, NX = kNodes / kRowsX;         // rows of x per round; rounds
    constexpr bool kTight = NR == 8;                            // little room in the registers
    constexpr int kAhead = kTight ? 3 : 4;
    constexpr int kSlots = NR / 2;                              // groups of 64 nodes, a wave each for the index
    static_assert(NH >= 1 && NB >= 1 && NX == 4 && (!RP || NR == 4), "");
    __shared__ __align__(512) char lds[L::size];

    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int halves = P / kPC, bh = halves == 2 ? unit >> 1 : unit, p0 = halves == 2 ? (unit & 1) * kPC : 0;
    const int b = H.quotient(bh), h = bh - b * H.d, g = per_group.quotient(h);
    const int nblk = (n + kRB - 1) / kRB, phases = NR <= kCB ? 1 : (nblk + kCB - 1) / kCB;
    // The row block of this wave.  The waves of a workgroup go to the four SIMDs in turn and block I has I + 1 column
    // blocks: of eight, a long and a short one share a SIMD; of four, every other workgroup turns the order around.
    const int I = NR == 8 ? (wave < 4 ? wave : 11 - wave) : (blockIdx.x >> 8) & 1 ? NR - 1 - wave : wave;
    const int last = I < nblk ? I : -1;               // its last column block

    // ---- requests, in the order in which they are waited for -------------------------------------------------
    int par = -1;
    float d_ = 0.f;
    if (wave < kSlots) {
        const uint32_t at = (uint32_t)(b * n + min(tid, n - 1));
        par = parent[at];
        d_ = dt[at * (uint32_t)H.d + (uint32_t)h];
    }
    int ppar = -1, k_prev = -1;
    float pd = 0.f;
    bool k_bad = false;
    // the previous tree: 64 nodes a wave, the first ones to the last wave (the first has the tree's index to build)
    [[maybe_unused]] const int pslot = NR - 1 - wave, pnode = pslot * 64 + lane;
    if constexpr (RP) {
        const uint32_t at = (uint32_t)(b * R.pn + min(pnode, R.pn - 1));
        ppar = R.parent[at];
        pd = R.dt[at * (uint32_t)H.d + (uint32_t)h];
        k_prev = R.accepted[b];
        k_bad = k_prev < -1 || k_prev >= R.pn;
    }
    __builtin_amdgcn_sched_barrier(0);
    // (buffers that end with the sequence's last row: rows past the tree read as zeros)
    const auto rows_of = [&](const bf16_t *first, long sn, int width) {
        return make_buffer(first + (size_t)b * n * sn, (size_t)((uint32_t)((n - 1) * (int)sn + width) * 2u));
    };
    const auto Cb = rows_of(Cm + (size_t)g * S, c_sn, S), Bb = rows_of(Bm + (size_t)g * S, b_sn, S);
    const auto xb = rows_of(x + (size_t)h * P + p0, x_sn, kPC);
    u32x4 cr[NK], br[NB], xr[NX];
    auto request = [&](auto &r, __amdgpu_buffer_rsrc_t rows, int sn, int row, int at, int step) {    // row, row + step, ...
        uint32_t off = (uint32_t)(row * sn + at * 8) * 2u;
#pragma unroll
        for (auto &v : r) {
            v = __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, 0);
            off += (uint32_t)(step * sn) * 2u;
        }
    };
    request(cr, Cb, (int)c_sn, I * kRB + lane / kPieces, lane % kPieces, 64 / kPieces);     // whole rows to consecutive lanes
    __builtin_amdgcn_sched_barrier(0);
    auto request_b = [&](int phase) {
        const int t = (int)fresh(tid);
        request(br, Bb, (int)b_sn, phase * kCB * kRB + t / kPieces, t % kPieces, T / kPieces);
    };
    request_b(0);
    request(xr, xb, (int)x_sn, tid / 8, tid % 8, kRowsX);
    __builtin_amdgcn_sched_barrier(0);
    // The state, used behind the last phase: it streams in while the products are formed.  With the replay it lies in
    // the registers as the tiles that advance it, else as whole rows.
    using Tiles = StateTiles<S, HT>;
    constexpr int NHR = RP ? Tiles::kPieces : NH;
    u32x4 hr[NHR];
    auto request_state = [&]() {   // (a buffer, empty without a state: no branch that the registers would have to agree behind)
        const auto hbuf = make_buffer(h0 + ((size_t)bh * P + p0) * S, h0 ? (size_t)kPC * S * sizeof(HT) : 0);
        const int t = (int)fresh(tid);
        if constexpr (RP) {
            Tiles::request(hr, hbuf, (t >> 6) * 16 + ((t & 63) >> 4) * 4, t & 15);
        } else {
#pragma unroll
            for (int q = 0; q < NHR; ++q) hr[q] = __builtin_amdgcn_raw_buffer_load_b128(hbuf, (q * T + t) * 16, 0, 2);   // nt
        }
    };
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
    if constexpr (RP) {
        // The previous tree's path: a wave finds, for each of its 64 nodes, the ancestors among those and the first one
        // below them; the path of the accepted node is then at most four hops from one wave's nodes to a lower one's.
        const int node0 = pslot * 64;
        const bool ok = pnode >= R.pn || ((pnode == 0) ? (ppar == -1) : (ppar >= 0 && ppar < pnode));
        const unsigned long long bm = __ballot(!ok);
        if (lane == 0) lds_at<int>(base + L::pbad + wave * 4) = bm ? node0 + (int)__ffsll((long long)bm) : 0x7fffffff;
        int pj = (pnode < R.pn && ok) ? ppar : -1;
        unsigned long long m = pnode < R.pn ? 1ull << lane : 0ull;
        for (int round = 0; round < 6; ++round) {
            const bool in = pj >= node0;
            if (!__any(in)) break;
            const int q = in ? pj - node0 : lane;
            const int rj = wave_read(pj, q);
            const unsigned long long rm = wave_read(m, q);
            if (in) {
                m |= rm;
                pj = rj;
            }
        }
        lds_at<u32x4>(base + L::groups + pnode * 16) = u32x4{(uint32_t)m, (uint32_t)(m >> 32), (uint32_t)pj, 0u};
        if (dt_bias) pd = softplus_step(pd + dt_bias[h]);
    }
    // C: from rows as they lie in memory to the lane's own row, through this wave's part of the B and x tiles
    bf16x8 cf[NK];
    {
        constexpr int kC = L::c_cols, kTrips = S / kC;
        const uint32_t c_at = base + wave * (kRB * kC * 2);
#pragma unroll
        for (int t = 0; t < kTrips; ++t) {
            if (lane % kPieces / (kC / 8) == t) {
#pragma unroll
                for (int q = 0; q < NK; ++q)
                    lds_at<u32x4>(c_at + piece_at<kC>(q * (64 / kPieces) + lane / kPieces, lane % (kC / 8))) = cr[q];
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
    auto zero_y = [&]() {                             // a bad tree: the sequence's outputs are zeros
        bf16_t *yb = y + (size_t)b * n * H.d * P + (size_t)h * P + p0;
        for (int i = tid / 8; i < n; i += kRowsX)
            *reinterpret_cast<uint4 *>(yb + (size_t)i * H.d * P + tid % 8 * 8) = make_uint4(0u, 0u, 0u, 0u);
    };
    if (!RP && bad) {                                 // (uniform; with the replay the state comes first)
        zero_y();
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
    [[maybe_unused]] int plen = 0;                    // nodes of the path to replay
    if constexpr (RP) {
        int pbad = 0x7fffffff;
#pragma unroll
        for (int w = 0; w < NR; ++w) pbad = min(pbad, lds_at<int>(base + L::pbad + w * 4));
        pbad = pbad == 0x7fffffff ? 0 : pbad;
        if (R.status && h == 0 && p0 == 0 && tid == 0) R.status[b] = pbad ? pbad : (k_bad ? -1 : 0);
        if (!pbad && k_prev >= 0 && !k_bad) {         // (else the state passes through)
            unsigned long long mine = 0;
            int before = 0;                           // path nodes in the waves below this one
            for (int cur = k_prev; cur >= 0;) {       // (a jump goes to a lower wave's node: at most four)
                const u32x4 v = lds_at<u32x4>(base + L::groups + cur * 16);
                const unsigned long long m = ((unsigned long long)v.y << 32) | v.x;
                const int cnt = __popcll(m);
                plen += cnt;
                if ((cur >> 6) < pslot) before += cnt;
                if ((cur >> 6) == pslot) mine = m;
                cur = (int)v.z;
            }
            plen = __builtin_amdgcn_readfirstlane(plen);
            if ((mine >> lane) & 1ull) {              // (ancestors have smaller labels: ascending label = root first)
                const int pos = before + __popcll(mine & ((1ull << lane) - 1ull));
                lds_at<unsigned char>(base + L::node + pos) = (unsigned char)pnode;
                lds_at<float>(base + L::weight + pos * 4) = pd;         // the step size for now
            }
        }
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
    __syncthreads();                                  // (with the replay: the groups lie where x comes)
    int wide = 0;
#pragma unroll
    for (int w = 0; w < kSlots; ++w) wide |= lds_at<int>(base + L::bad + 16 + w * 4);
    wide = __builtin_amdgcn_readfirstlane(wide);
    if (wave < kSlots)                                // dt = 0 (and nodes past the tree): weight 0
        lds_at<float>(base + L::u + tid * 4) = wide ? s - __log2f(d_) : d_ * __builtin_amdgcn_exp2f(-s);
#pragma unroll
    for (int q = 0; q < NX; ++q)
        lds_at<u32x4>(base + L::x + (tid % 8) / 4 * (kNodes * 64) + x_piece_at(q * kRowsX + tid / 8, tid & 3)) = xr[q];
    __syncthreads();

    // ---- replay: the first rows of the path --------------------------------------------------------------------
    using Path = PathRows<S, T, L::kPath, false>;
    u32x4 pr[Path::kPieces];
    [[maybe_unused]] auto request_path = [&](int first) {
        const char *xb = reinterpret_cast<const char *>(R.x + (size_t)b * R.pn * R.x_sn + (size_t)h * P + p0);
        const char *Bp = reinterpret_cast<const char *>(R.Bm + (size_t)b * R.pn * R.b_sn + (size_t)g * S);
        Path::request(pr, R, xb, Bp, base + L::node + first, plen - first, fresh(tid));
    };
    [[maybe_unused]] auto stage_path = [&](int first) { Path::stage(pr, base + L::rows, plen - first, fresh(tid)); };
    if constexpr (RP) {
        if (plen > 0) request_path(0);
    }
    __builtin_amdgcn_sched_barrier(0);

    request_state();
    __builtin_amdgcn_sched_barrier(0);
    // replay: the weights along the path,
    //   h* = exp(s_k) h0 + sum_{j on path(k)} dt_j exp(s_k - s_j) x_j (outer) B_j
    // exp(s_k - s_j) is the exponential of the sum over the nodes BEHIND j, summed along the path itself: its rounding
    // error is relative to that sum, which is small wherever the weight is not negligible.
    [[maybe_unused]] float weight = 0.f, dec = 1.f;
    [[maybe_unused]] const int chunks = (plen + 63) >> 6;
    if constexpr (RP) {
        if (wave < chunks) {                          // lane = position on the path, a wave 64 of them
            const float A_h = A[h];
            float behind = 0.f;
            for (int c = chunks - 1; c >= wave; --c) {
                const float own = c * 64 + lane < plen ? lds_at<float>(base + L::weight + (c * 64 + lane) * 4) : 0.f;
                float suf = own * A_h;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const float v = __shfl_down(suf, off);
                    if (lane + off < 64) suf += v;
                }
                float next = __shfl_down(suf, 1);
                if (lane == 63) next = 0.f;
                weight = own * __expf(behind + next); // (the last turn's, this wave's own positions, is the one kept)
                behind += __shfl(suf, 0);
            }
            if (tid == 0) lds_at<float>(base + L::pbad + 16) = __expf(behind);
        }
        if (chunks > 1) __syncthreads();              // (the steps are read by several waves)
        if (wave < chunks) lds_at<float>(base + L::weight + tid * 4) = weight;
    }

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
            const uint32_t word = lds_at<uint32_t>(mask_at + J * (kNodes * 4)) >> (4 * lh), u_at = fresh(base + L::u + 16 * lh + J * (kRB * 4));
            u32x4 m[2];
            weigh(m, gt, word, u_at, s2_i, e_i, wide);
            const uint32_t x_at = fresh(x_lane + J * (kRB * 64));
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int pt = 0; pt < 2; ++pt) {
                    const uint32_t at = x_at + pt * (kNodes * 64) + kk * (16 * 64);
                    acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join(read_transposed(at), read_transposed((at ^ 32) + 8 * 64)),
                                                                      __builtin_bit_cast(bf16x8, m[kk]), acc[pt], 0, 0, 0);
                }
        }
    }
    if constexpr (RP) {
        if (L::kRowsInB) __syncthreads();
        if (plen > 0) stage_path(0);
    }
    __syncthreads();                                  // all products with B and x are done
    const int ft = (int)fresh(tid);
    if constexpr (RP) {
        const int l = ft & 15, kj = (ft & 63) >> 4, prow = (ft >> 6) * 16;
        if (plen > 0) dec = lds_at<float>(base + L::pbad + 16);
        typename Tiles::Values hv;
        Tiles::widen(hv, hr, dec);
        for (int first = 0; first < plen; first += L::kPath) {
            if (first > 0) {                          // longer paths: the next rows, one round trip for sixteen
                request_path(first);
                __syncthreads();
                stage_path(first);
                __syncthreads();
            }
            Tiles::template advance<false>(hv, base + L::rows, L::kPath, base + L::weight + first * 4, min(plen - first, L::kPath), prow, l, kj);
        }
        const auto ho = make_store_rsrc(reinterpret_cast<HT *>(R.h_out) + ((size_t)bh * P + p0) * S, (uint32_t)(kPC * S * sizeof(HT)));
        Tiles::store(hv, ho, base + L::bm, prow + kj * 4, l);
    } else {
        stage_state<S, T, HT>(hr, base + L::bm, ft);
    }
    __syncthreads();
    if (RP && bad) {
        zero_y();
        return;
    }
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
            for (int e = 0; e < 4; ++e) {
                v[e] = fmaf(D_h, xf[e], fmaf(e_i, ch[4 * q + e], acc[pt][4 * q + e]));
            }
            lds_at<u32x2>(at) = u32x2{pack2(v[0], v[1]), pack2(v[2], v[3])};
        }
    }
    wave_lds_fence();
    const __amdgpu_buffer_rsrc_t yr = make_store_rsrc(y + (size_t)b * n * H.d * P + (size_t)h * P + p0, (uint32_t)(n * H.d * P - h * P - p0) * 2u);
#pragma unroll
    for (int r0 = 0; r0 < kRB; r0 += 8) {             // whole rows of 128 bytes
        const int row = I * kRB + r0 + ln / 8, pc = ln % 8;
        const u32x4 v = lds_at<u32x4>(base + L::x + pc / 4 * (kNodes * 64) + x_piece_at(row, pc & 3));
        if (row < n) buffer_store_through16(yr, (uint32_t)(row * H.d * P + pc * 8) * 2u, make_uint4(v.x, v.y, v.z, v.w));
    }
}

template <int S, int NR, bool RP>
hipError_t launch_rows_s(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                         const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                         const ReplayArgs &R, hipStream_t st) {
    using L = RowsLds<S, NR, RP>;
    constexpr int kFit = L::per_cu * NR / 4, kMost = S == 256 ? 2 : NR == 8 ? 4 : 3, WPE = kFit < kMost ? kFit : kMost;   // waves per SIMD
    const int units = d.batch * d.nheads * (d.headdim / kPC);
#define STREE_LAUNCH_ROWS(HT)                                                                                       \
    hipLaunchKernelGGL((tree_ssd_rows_kernel<S, NR, WPE, RP, HT>), dim3(8 * ((units + 7) / 8)), dim3(64 * NR), 0, st, \
                       parent, d.nnodes, units, Divisor(d.nheads), Divisor(d.nheads / d.ngroups), d.headdim, (const bf16_t *)x,                  \
                       (long)d.x_stride_n, dt, step_bias(d), A, (const bf16_t *)Bm, (long)d.b_stride_n,             \
                       (const bf16_t *)Cm, (long)d.c_stride_n, D, (const HT *)h0, (bf16_t *)y, status, R)
    if (d.state_dtype == STREE_BF16) STREE_LAUNCH_ROWS(bf16_t);
    else STREE_LAUNCH_ROWS(float);
#undef STREE_LAUNCH_ROWS
    return hipGetLastError();
}

template <int NR, bool RP>
hipError_t launch_rows(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
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
        const auto launch = s.dstate == 64 ? launch_rows_s<64, NR, RP> : s.dstate == 128 ? launch_rows_s<128, NR, RP> : launch_rows_s<256, NR, RP>;
        return launch(s, parent + nodes, advance(x, nodes * s.x_stride_n * 2), dt + nodes * s.nheads, A,
                      advance(Bm, nodes * s.b_stride_n * 2), advance(Cm, nodes * s.c_stride_n * 2), D, advance(h0, state),
                      advance(y, nodes * d_inner * 2), advance(status, b), r, st);
    });
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
    const ReplayArgs none = {};
    if (d.nnodes <= 128) return launch_rows<4, false>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, none, st);
    return launch_rows<8, false>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, none, st);
}

// (above 128 nodes the state would not fit the registers beside the products: commit, then scan)
bool tree_ssd_replay_rows_supported(const stree_dims &d, const stree_dims &dp, const void *px, const void *pB,
                                     const void *x, const void *Bm, const void *Cm, const void *y, const void *h0,
                                     const void *h_out) {
    if (d.io_dtype != STREE_BF16 || !tree_ssd_rows_supported(d) || d.nnodes > 128 || (d.flags & STREE_FLAG_GENERAL_MFMA))
        return false;
    if ((d.x_stride_n | d.b_stride_n | d.c_stride_n | dp.x_stride_n | dp.b_stride_n) % 8 != 0) return false;
    const uintptr_t bits = (uintptr_t)x | (uintptr_t)Bm | (uintptr_t)Cm | (uintptr_t)y | (uintptr_t)px | (uintptr_t)pB |
                           (uintptr_t)h0 | (uintptr_t)h_out;   // (the state is read and written 16 bytes at a time)
    return bits % 16 == 0;
}

hipError_t launch_tree_ssd_replay_rows(const stree_dims &d, const stree_dims &dp, const int32_t *pparent,
                                        const int32_t *paccepted, const void *px, const float *pdt, const void *pB,
                                        const int32_t *parent, const void *x, const float *dt, const float *A,
                                        const void *Bm, const void *Cm, const float *D, const void *h0,
                                        void *h_out, void *y, int32_t *status, int32_t *rstatus, hipStream_t st) {
    const ReplayArgs R = {pparent, paccepted, (const bf16_t *)px, (const bf16_t *)pB, pdt,
                          (long)dp.x_stride_n, (long)dp.b_stride_n, dp.nnodes, h_out, rstatus};
    return launch_rows<4, true>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, R, st);
}

}  // namespace stree
