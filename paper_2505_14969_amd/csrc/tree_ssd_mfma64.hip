// Tree scan for trees of at most 64 nodes, most of them with two to six heads a CU, the bands in
// which it is ahead of the workgroup per head of tree_ssd_unit.hip (see unit_is_slower): persistent, software-pipelined,
// wave-specialised (products and accumulator layouts as in tree_ssd_mfma.hip).
//
// A workgroup of 8 waves walks a list of (batch, head) units.  Units are dealt
// out so that all heads of one sequence land on the same XCD (workgroup id % 8),
// whose L2 then serves the B / C rows that the heads of a group share.
//
//   Y waves 0-3   own the four 32x32 tiles of Yt[p][i]; carry the h0 prefetch of even units
//   G waves 4,5,7 own the three live tiles of Gt[j][i]; carry the x prefetch and, with the
//   T wave  6     (its Gt tile has j > i everywhere; builds the tree index), the h0 prefetch
//                 of odd units: the h0 tiles of two future units are always in flight
//
// A workgroup's units are consecutive, so mostly heads of one sequence and
// group: C, B and Gt = B C^T are staged / computed once per run of such heads
// (CB^T once per group), only the decay weighting is redone per head.
//
// Steady state for unit k, with the registers already holding unit k+1:
//   barrier 1
//     Y: phase 1  Yt = h0b C^T, *= exp(s_i)
//     G: phase 2  (Gt = B C^T if the tiles are new) M = L ? Gt exp(s_i - s_j) dt_j : 0 -> LDS
//   barrier 2   (h0b tile and the tree arrays are dead from here on)
//     Y: phase 3  Yt += Xt M^T; y = Yt + D x -> bf16, turned around per wave in LDS, stored as row pieces
//     Y or G (whoever carries unit k+1): h0(k+1) regs -> LDS as bf16; issue h0(k+3) loads
//     G: new C tile if unit k+1 starts another sequence or group
//     T: tree index of unit k+1, issue parent/dt (k+2) loads
//     G: x(k+1) regs -> the other X^T tile in LDS, issue x(k+2) loads
// so the big global loads (h0, x) are in flight for a whole unit period.
//
// Template flag RP folds the commit of the previous tree into the state as it is loaded
// (Alg. 1: replay at the start of the next iteration).
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "tiles.hpp"

namespace stree {

namespace {

constexpr int kB64 = 64;
constexpr int kNP64 = kB64 + 8;
constexpr int kT64 = 512;   // 8 waves: 4 Y waves, 3 G waves, 1 tree wave

constexpr int kYStage = 4 * 2048;   // bytes at the start of the B tile's LDS that the Y waves turn y around in

// static LDS of the kernel below (C, B, h0b tiles, two X^T tiles, M, tree arrays; with replay the path arrays)
template <int P, int S>
struct Lds64 {
    static constexpr int SP = S + 8;
    static constexpr size_t row_bytes = (size_t)(P + S) * 2;                      // x row and B row of a path node
    static constexpr size_t b_bytes = (size_t)kB64 * SP * 2, m_bytes = (size_t)kB64 * kNP64 * 2;
    // path nodes whose rows LDS has room for: behind the y staging area of the B tile and (first pass) in the M tile
    static constexpr size_t room_b = (b_bytes > kYStage ? b_bytes - kYStage : 0) / row_bytes, room_m = m_bytes / row_bytes;
    static constexpr int kRows = (int)(room_b < room_m ? room_b : room_m);
    static constexpr size_t total = (size_t)2 * kB64 * SP * 2 + (size_t)P * SP * 2 + (size_t)2 * P * kNP64 * 2 +
                                    (size_t)kB64 * kNP64 * 2 + 1040;
    static constexpr size_t total_replay = total + 336;
};

// Wave-level tree index for n <= 64: lane i owns node i; pointer doubling with
// cross-lane reads (ds_bpermute), no barriers.  Returns the status (uniform).
// Outputs are in log2 units so that the decay is one v_exp_f32 per element:
//   s2[i] = log2(e) * s_i          u[j] = s2[j] - log2(dt_j)
//   exp(s_i - s_j) * dt_j = exp2(s2[i] - u[j])      (dt_j = 0 -> u = +inf -> 0)
__device__ __forceinline__ int wave_tree_index(int lane, int n, int parent_i, float dt_i, float A_h, float *s2_out,
                                               float *u_out, uint32_t *mask_out) {
    int p = -1;
    bool ok = true;
    if (lane < n) {
        p = parent_i;
        ok = (lane == 0) ? (p == -1) : (p >= 0 && p < lane);
        if (!ok) p = -1;
    }
    const unsigned long long badmask = __ballot(!ok);
    if (badmask) return __ffsll((long long)badmask);  // first bad lane + 1
    float s = lane < n ? dt_i * A_h : 0.f;
    uint32_t mlo = (lane < 32) ? (1u << lane) : 0u, mhi = (lane >= 32) ? (1u << (lane - 32)) : 0u;
    if (lane >= n) mlo = mhi = 0u;
    for (int round = 0; round < 6; ++round) {
        if (!__any(p >= 0)) break;
        const int q = p >= 0 ? p : lane;
        const float rs = wave_read(s, q);
        const int rp = wave_read(p, q);
        const uint32_t rlo = wave_read(mlo, q), rhi = wave_read(mhi, q);
        if (p >= 0) {
            s += rs;
            mlo |= rlo;
            mhi |= rhi;
            p = rp;
        }
    }
    const float s2 = s * 1.44269504088896340736f;
    s2_out[lane] = s2;
    u_out[lane] = s2 - __log2f(lane < n ? dt_i : 0.f);
    mask_out[lane * 2] = mlo;
    mask_out[lane * 2 + 1] = mhi;
    return 0;
}

// WPE = waves per SIMD the register budget is sized for: 4 when two workgroups fit a CU's LDS.
//
// RP = fused activation replay (Alg. 1): the state loaded for a unit is first advanced along the
// accepted path of the previous tree,
//   h* = exp(s_k) h0 + sum_{j on path(k)} dt_j exp(s_k - s_j) x_j (outer) B_j,
// in the fp32 registers it arrives in, written back once to h_out, and only then rounded to the
// bf16 MFMA operand.  The tree wave works the path of the next unit out in the scan half, in which
// it has nothing else to do (same pointer doubling as the tree index, on the previous tree).  The x / B
// rows of the path's first kRows nodes are fetched by the three G waves, which have nothing to do between
// barrier 2 and barrier (c): all requested at once, put into LDS, one round trip behind phase 3 whatever the
// length of the path.  (Rows read one by one behind the eighth cost beams of 3 tokens over 16 layers at batch
// 64 x 80 heads with a bf16 state 104.8 against 92.5 us.  Rows requested by the tree wave a half earlier, into its copy of the
// accumulator, were in flight for longer, but the compiler does not know the roles: it made every wave's
// products wait for those registers, i.e. for all of its own prefetches.  Without them: 73.5 -> 69.5 us for trees
// of depth 4 to 8, 82 -> 78 us for the beams.)  Paths of more than kRows nodes read what is left from
// global memory, four nodes at a time.  The update itself runs on the fp32 matrix units (16 x 16 x 4: four path
// nodes an instruction, the fp32 FMAs of the recurrence in the same precision): as vector FMAs it cost the four
// waves that carry a unit some 56 instructions per path node, while the other four waited (the beams above:
// 92.5 -> 82.4 us, chains of up to 49 nodes 195 -> 134 us, trees of depth 4 to 8 75.9 -> 72.9 us).
// HT = type the state is kept in: fp32, or bf16 (then h0 is the MFMA operand as it comes, and the replayed
// state is rounded once, to the value that is both written back and scanned from).
template <int P, int S, int WPE, bool RP, bool SPL, typename HT>
__global__ __launch_bounds__(kT64) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void tree_ssd_mfma64_kernel(
    const int32_t *__restrict__ parent, int n, int nbatch, int H, int G, const bf16_t *__restrict__ x, long x_sn,
    const float *__restrict__ dt, const float *__restrict__ dt_bias, const float *__restrict__ A,
    const bf16_t *__restrict__ Bm, long b_sn,
    const bf16_t *__restrict__ Cm, long c_sn, const float *__restrict__ D, const HT *__restrict__ h0,
    bf16_t *__restrict__ y, int32_t *__restrict__ status, ReplayArgs R) {
    using L = Lds64<P, S>;
    constexpr int SP = L::SP;
    constexpr int kHalf = kT64 / 2;                 // threads per role group
    constexpr int NC = kB64 * (S / 8) / kHalf;      // 16-byte chunks of C (and of B) per G thread
    constexpr int NX = kB64 * (P / 8) / kHalf;      // of x per G thread; of y per Y thread
    constexpr int NH = P * S / 4 / kHalf;           // float4 chunks of h0 per Y thread
    constexpr int YT = (P / 32) * 2, YQ = YT / 4;   // Yt tiles, tiles per Y wave
    constexpr int kRowsC = kHalf / (S / 8), kRowsX = kHalf / (P / 8);
    static_assert(NC >= 1 && NX >= 1 && NH >= 1 && YQ >= 1, "tile too small for this thread count");
    // separate LDS objects (not slices of one array), so that the compiler knows that a write to
    // one tile cannot alias a read of another and does not serialise them
    __shared__ __align__(16) bf16_t sC[kB64 * SP];
    __shared__ __align__(16) bf16_t sB[kB64 * SP];
    __shared__ __align__(16) bf16_t sH[P * SP];
    __shared__ __align__(16) unsigned short sXT2[2][P * kNP64];   // X^T of units k and k+1
    __shared__ __align__(16) bf16_t sM[kB64 * kNP64];
    __shared__ __align__(16) float sS2[kB64];
    __shared__ __align__(16) float sU[kB64];
    __shared__ uint32_t sMask[kB64 * 2];
    __shared__ int sBad[1];
    __shared__ float sDh[1];
    // replay: path of the accepted node (position -> node, weight), its length and exp(s_k)
    __shared__ float sRcoef[RP ? kB64 : 1];
    __shared__ unsigned char sRnode[RP ? kB64 : 4];
    __shared__ int sRlen[1];
    __shared__ float sRdec[1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = tid >> 6;
    constexpr int kTreeWave = 6;
    const bool isY = wave < 4;
    const int rt = tid & (kHalf - 1);    // thread index within its role group
    const int n_units = nbatch * H;
    const int per_xcd = (n_units + 7) >> 3;
    const int xcd = blockIdx.x & 7;
    const int wg = blockIdx.x >> 3, nwg = gridDim.x >> 3;   // this workgroup among its XCD's
    const int hpg = H / G;
    // XCD x owns the contiguous unit range [x*per_xcd, ...); its workgroups split that range
    // into contiguous runs, so a workgroup mostly sees consecutive heads of one sequence and
    // group: their C, B tiles, the tree mask and Gt = B C^T are then reused, not redone.
    const int cnt = max(0, min(per_xcd, n_units - xcd * per_xcd));
    // the first cnt % nwg workgroups take one unit more.  (Workgroups are placed one per CU first and
    // the second one per CU later: a CU then holds workgroup w and w + nwg/2, a long and a short run.)
    const int ubase = cnt / nwg, urem = cnt % nwg;
    const int u0 = xcd * per_xcd + wg * ubase + min(wg, urem);
    const int nU = ubase + (wg < urem ? 1 : 0);
    // (b, h) of unit k by stepping from unit 0 (k is 0, 1 or 2 units ahead of a known one):
    // scalar adds and compares only, no division inside the unit loop
    const int ub0 = __builtin_amdgcn_readfirstlane(u0 / H), uh0 = __builtin_amdgcn_readfirstlane(u0 % H);
    auto step = [&](int &b, int &h) {
        if (++h == H) {
            h = 0;
            ++b;
        }
    };
    // a unit needs new C/B tiles when it is the first one or starts another sequence or group
    auto fresh_at = [&](int k, int h) -> bool { return k == 0 || h % hpg == 0; };

    // ---- prefetch registers and their loaders ---------------------------------------------------
    // per-thread chunk offsets never change from unit to unit; the unit's base pointer is uniform.
    // Rows >= n are read from row n-1 (valid memory) and zeroed when staged: no branches.
    // one register array serves both roles (a thread is either Y or G for its whole life):
    //   pre[0..NH)  h0 chunks (fp32 bits) of a future unit: the Y threads carry the even units
    //               of the run, the G threads the odd ones, so two units' h0 are in flight
    //   pre[NH..)   x chunks of the next unit (G threads)
    constexpr int NPRE = NH + NX;
    uint4 pre[NPRE];
    int rpar = -1;
    float rdt = 0.f;
    // The chunk coordinates of a thread are loop invariants; keeping them all in registers
    // across the unit loop would cost more registers than the budget of 128 allows, so every
    // helper below re-derives them from an opaque copy of the thread index (a few VALU ops).
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    // the node half of the tiles a wave owns.  With the replay the register budget has no room for
    // it (nor for anything else the compiler would hoist out of the unit loop): kept live it is
    // spilled, and a reload waits for every load in flight, so there it is re-derived where used
    // from a copy of the wave index that the compiler cannot see through.
    const int it0 = wave & 1;

    float rD = 0.f;                  // D[h] of the unit whose h0 is in pre[]
    // The state tile in a thread's registers.  Without replay chunk q is element (t + q*kHalf)*4 of the P x S tile.
    // With replay it is the accumulator of the fp32 matrix instructions that advance it (16 x 16 x 4, accumulator
    // row = state row p, column = state column s): a wave owns 16 rows of every 64, lane l the rows 4 (l >> 4) + i of
    // those and kCW consecutive columns kCW (l & 15) + t -- column t of each lane makes up tile t, so that a lane's columns
    // are 16-byte pieces in memory all the same.
    constexpr uint32_t HB = sizeof(HT);
    constexpr int kCW = 16 / HB, kCB = S / (16 * kCW), kPG = P / 64; // columns per chunk; column blocks; 64-row groups
    static_assert(kCB >= 1 && NH % 2 == 0, "a state is moved 16 bytes at a time");
    auto load_H = [&](int b, int h) {       // the role group that carries this unit
        // the lane-dependent zero keeps this a vector load: it then sits in the same in-order
        // queue as the h0 chunks instead of forcing a scalar-cache wait in the hot window
        if (D) rD = D[h + (opaque(lane) & 0)];
        const char *hb = reinterpret_cast<const char *>(h0 + ((size_t)b * H + h) * P * S);
        if constexpr (RP) {
            const int t = opaque(rt), row0 = (t >> 6) * 16 + ((t & 63) >> 4) * 4, col0 = (t & 15) * kCW;
            const uint32_t off = (uint32_t)(row0 * S + col0) * HB;
#pragma unroll
            for (int q = 0; q < kPG * kCB * 4; ++q)   // q = (row group, column block, row)
                pre[q] = load_stream16(hb + off + ((q / (4 * kCB) * 64 + q % 4) * S + q / 4 % kCB * 16 * kCW) * HB);
        } else {
            const uint32_t off = (uint32_t)opaque(rt) * 16u;
#pragma unroll
            for (int q = 0; q < NH * (int)HB / 4; ++q) pre[q] = load_stream16(hb + q * (kHalf * 16) + off);
        }
    };
    // C and B tiles of a unit: global -> registers -> LDS in one go (G threads).  Runs only when
    // the (sequence, group) changes, i.e. about once per workgroup.
    auto restage_CB = [&](int b, int h) {
        const int g = h / hpg;
        const char *Cb = reinterpret_cast<const char *>(Cm + (size_t)b * n * c_sn + (size_t)g * S);
        const char *Bb = reinterpret_cast<const char *>(Bm + (size_t)b * n * b_sn + (size_t)g * S);
        const int t = opaque(rt), rc0 = t / (S / 8), cc0 = t % (S / 8);
        uint4 c[NC], bq[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int rr = min(rc0 + q * kRowsC, n - 1);
            c[q] = *reinterpret_cast<const uint4 *>(Cb + (uint32_t)(rr * (int)c_sn + cc0 * 8) * 2u);
            bq[q] = *reinterpret_cast<const uint4 *>(Bb + (uint32_t)(rr * (int)b_sn + cc0 * 8) * 2u);
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int rr = rc0 + q * kRowsC;
            const uint32_t keep = rr < n ? 0xffffffffu : 0u;   // zero the rows beyond the tree
            *reinterpret_cast<uint4 *>(&sC[rr * SP + cc0 * 8]) =
                make_uint4(c[q].x & keep, c[q].y & keep, c[q].z & keep, c[q].w & keep);
            *reinterpret_cast<uint4 *>(&sB[rr * SP + cc0 * 8]) =
                make_uint4(bq[q].x & keep, bq[q].y & keep, bq[q].z & keep, bq[q].w & keep);
        }
    };
    auto load_X = [&](int b, int h) {       // G threads
        const char *xb = reinterpret_cast<const char *>(x + (size_t)b * n * x_sn + (size_t)h * P);
        const int t = opaque(rt), rx0 = t / (P / 8), cx0 = t % (P / 8);
#pragma unroll
        for (int q = 0; q < NX; ++q)
            pre[NH + q] = *reinterpret_cast<const uint4 *>(
                xb + (uint32_t)(min(rx0 + q * kRowsX, n - 1) * (int)x_sn + cx0 * 8) * 2u);
    };
    // an array element that is the same for the whole wave, by a scalar load: a vector load would be the newest one in
    // flight, and waiting for it would be waiting for the whole state prefetch
    auto uniform_load = [](auto *a, int i) {
        typedef __attribute__((address_space(4))) const typename std::remove_const<typename std::remove_pointer<decltype(a)>::type>::type *ptr_t;
        return ((ptr_t)(uintptr_t)a)[__builtin_amdgcn_readfirstlane(i)];
    };
    auto load_T = [&](int b, int h) {       // tree wave
        const int node = min(opaque(lane), n - 1);
        rpar = parent[(uint32_t)(b * n + node)];
        rdt = dt[(uint32_t)((b * n + node) * H + h)];
    };
    // ---- registers -> LDS -------------------------------------------------------------------------
    // rbuf: the LDS rows of the replayed path (x rows [kRows][P], then B rows [kRows][S]); b, h: the unit
    constexpr int kRows = L::kRows;
    auto stage_H = [&]([[maybe_unused]] const char *rbuf, [[maybe_unused]] int b, [[maybe_unused]] int h) {
        const int t = opaque(rt);
        if constexpr (RP) {
            const int l = t & 15, kj = (t & 63) >> 4, prow = (t >> 6) * 16;
            const int len = *sRlen;
            const float dec = *sRdec;
            floatx4 hv[kPG * kCB][kCW];                    // [row group, column block][tile]
#pragma unroll
            for (int q = 0; q < kPG * kCB * 4; ++q) {
                const uint32_t w4[4] = {pre[q].x, pre[q].y, pre[q].z, pre[q].w};
#pragma unroll
                for (int e = 0; e < kCW; ++e)
                    hv[q / 4][e][q % 4] = dec * (HB == 4 ? __uint_as_float(w4[e % 4]) : (e & 1) ? bf16_hi(w4[e / 2]) : bf16_lo(w4[e / 2]));
            }
            // four path nodes: lane group kj holds node j of them, its weight cf (0 past the end of the path),
            // its x at row (t & 15) of the wave's rows (operand A) and cf * B at the lane's columns (operand B)
            auto rank4 = [&](bool on, float cf, const char *xr, const char *br) {
                float av[kPG];
#pragma unroll
                for (int g = 0; g < kPG; ++g) {
                    const uint32_t xw = *reinterpret_cast<const unsigned short *>(xr + (prow + l + g * 64) * 2);
                    av[g] = on ? __uint_as_float(xw << 16) : 0.f;
                }
#pragma unroll
                for (int c = 0; c < kCB; ++c) {
                    const char *at = br + (c * 16 + l) * kCW * 2;
                    float bf[kCW];
#pragma unroll
                    for (int e = 0; e < kCW; e += 4) {
                        const uint2 bw = *reinterpret_cast<const uint2 *>(at + e * 2);
                        bf[e] = bf16_lo(bw.x), bf[e + 1] = bf16_hi(bw.x), bf[e + 2] = bf16_lo(bw.y), bf[e + 3] = bf16_hi(bw.y);
                    }
#pragma unroll
                    for (int e = 0; e < kCW; ++e)
#pragma unroll
                        for (int g = 0; g < kPG; ++g)
                            hv[g * kCB + c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[g], on ? cf * bf[e] : 0.f, hv[g * kCB + c][e], 0, 0, 0);
                }
            };
            const int nl = min(len, kRows);
            for (int j0 = 0; j0 < nl; j0 += 4) {
                const int j = min(j0 + kj, nl - 1);
                rank4(j0 + kj < nl, sRcoef[j], rbuf + j * P * 2, rbuf + (kRows * P + j * S) * 2);
            }
            if (len > kRows) {   // the rest of a very long path: rows straight from global memory
                const int g = h / hpg;
                const char *xb = reinterpret_cast<const char *>(R.x + (size_t)b * R.pn * R.x_sn + (size_t)h * P);
                const char *Bb = reinterpret_cast<const char *>(R.Bm + (size_t)b * R.pn * R.b_sn + (size_t)g * S);
                for (int j0 = kRows; j0 < len; j0 += 4) {
                    const int j = min(j0 + kj, len - 1), node = sRnode[j];
                    rank4(j0 + kj < len, sRcoef[j], xb + (size_t)node * R.x_sn * 2, Bb + (size_t)node * R.b_sn * 2);
                }
            }
            // the replayed state, written once, through L2 (never read again by this kernel)
            char *ob = reinterpret_cast<char *>(reinterpret_cast<HT *>(R.h_out) + ((size_t)b * H + h) * P * S);
#pragma unroll
            for (int q = 0; q < kPG * kCB * 4; ++q) {
                const int at_row = prow + kj * 4 + q / (4 * kCB) * 64 + q % 4, at_col = (q / 4 % kCB * 16 + l) * kCW;
                float v[kCW];
#pragma unroll
                for (int e = 0; e < kCW; ++e) v[e] = hv[q / 4][e][q % 4];
                char *dst = ob + (uint32_t)(at_row * S + at_col) * HB;
                bf16_t *op = &sH[at_row * SP + at_col];
                if constexpr (HB == 4) {
                    store_through16(dst, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])));
                    *reinterpret_cast<uint2 *>(op) = pack_bf16x4(v[0], v[1], v[2], v[3]);
                } else {
                    const uint2 lo = pack_bf16x4(v[0], v[1], v[2], v[3]), hi = pack_bf16x4(v[kCW - 4], v[kCW - 3], v[kCW - 2], v[kCW - 1]);
                    store_through16(dst, make_uint4(lo.x, lo.y, hi.x, hi.y));
                    *reinterpret_cast<uint4 *>(op) = make_uint4(lo.x, lo.y, hi.x, hi.y);
                }
            }
        } else if constexpr (HB == 4) {
#pragma unroll
            for (int q = 0; q < NH; ++q) {
                const int e = (t + q * kHalf) * 4, p = e / S, sidx = e % S;
                bf16x4 o;
                o[0] = (bf16_t)__uint_as_float(pre[q].x); o[1] = (bf16_t)__uint_as_float(pre[q].y);
                o[2] = (bf16_t)__uint_as_float(pre[q].z); o[3] = (bf16_t)__uint_as_float(pre[q].w);
                *reinterpret_cast<bf16x4 *>(&sH[p * SP + sidx]) = o;
            }
        } else {                                   // already the MFMA operand: copied as it came
#pragma unroll
            for (int q = 0; q < NH / 2; ++q) {
                const int e = (t + q * kHalf) * 8, p = e / S, sidx = e % S;
                *reinterpret_cast<uint4 *>(&sH[p * SP + sidx]) = pre[q];
            }
        }
        if (rt == 0) *sDh = rD;      // D of that unit, for the Y waves
    };
    auto stage_X = [&](int buf) {
        unsigned short *sXT = sXT2[buf];
        const int t = opaque(rt), rx0 = t / (P / 8), cx0 = t % (P / 8);
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int rr = rx0 + q * kRowsX;
            const uint32_t keep = rr < n ? 0xffffffffu : 0u;
            const uint4 xq = pre[NH + q];
            store_transposed_pair<P / 8>(sXT, kNP64, rr, cx0 * 8,
                                         make_uint4(xq.x & keep, xq.y & keep, xq.z & keep, xq.w & keep), opaque(lane));
        }
    };
    auto stage_T = [&](int h) {
        const int ln = opaque(lane);   // LDS addresses re-derived here, not carried across the loop
        float dt_i = rdt;
        float A_h;
        if constexpr (RP) {
            A_h = uniform_load(A, h);
            if constexpr (SPL) dt_i = softplus_step(rdt + uniform_load(dt_bias, h));   // raw projection -> step size
        } else {
            A_h = A[h];
            if constexpr (SPL) dt_i = softplus_step(rdt + dt_bias[h]);
        }
        const int bad = wave_tree_index(ln, n, rpar, dt_i, A_h, sS2, sU, sMask);
        if (ln == 0) *sBad = bad;
    };

    // ---- replay (tree wave): previous tree's path one unit ahead ----------------------------------
    constexpr int PX = P / 8, PB = S / 8;                     // 16-byte pieces per x row, per B row
    int rpp = -1;
    float rpdt = 0.f;
    auto load_R = [&](int b, int h) {
        const int node = min(opaque(lane), R.pn - 1);
        rpp = R.parent[(uint32_t)(b * R.pn + node)];
        rpdt = R.dt[(uint32_t)((b * R.pn + node) * H + h)];
    };
    auto path_R = [&](int b, int h) {
        const int ln = opaque(lane);
        const int pn = R.pn;
        // uniform values by scalar loads (a vector load here would be the newest one in flight, and
        // waiting for it would wait for the whole h0 prefetch)
        const int rk = uniform_load(R.accepted, b);
        const float rRA = uniform_load(A, h);
        float pdt_i = rpdt;
        if constexpr (SPL) pdt_i = softplus_step(rpdt + uniform_load(dt_bias, h));
        const bool kbad = rk < -1 || rk >= pn;
        int pos = -1, len = 0;
        float cf = 0.f, dc = 1.f;
        const int st = wave_path(ln, pn, (rk >= 0 && !kbad) ? rk : 0, rpp, pdt_i, rRA, pos, cf, len, dc);
        if (st != 0 || rk < 0 || kbad) {   // nothing to replay: the state passes through
            pos = -1;
            len = 0;
            cf = 0.f;
            dc = 1.f;
        }
        if (R.status && h == 0 && ln == 0) R.status[b] = st ? st : (kbad ? -1 : 0);
        // (the arrays are read in the staging half only)
        if (pos >= 0) {
            sRnode[pos] = (unsigned char)ln;
            sRcoef[pos] = cf;
        }
        if (ln == 0) {
            *sRlen = len;
            *sRdec = dc;
        }
    };
    // x / B rows of its first kRows nodes (the three G waves, between barrier 2 and barrier (c))
    auto fetch_R = [&](char *rbuf, int b, int h) {
        constexpr int PR = PX + PB, NT = 192, NQ = (kRows * PR + NT - 1) / NT;
        const int total = min(*sRlen, kRows) * PR;
        if (total <= 0) return;
        const int t0 = opaque(tid) - kHalf, t = t0 < 128 ? t0 : t0 - 64;     // waves 4, 5, 7
        const int g = h / hpg;
        const char *xb = reinterpret_cast<const char *>(R.x + (size_t)b * R.pn * R.x_sn + (size_t)h * P);
        const char *Bb = reinterpret_cast<const char *>(R.Bm + (size_t)b * R.pn * R.b_sn + (size_t)g * S);
        static_assert(NQ <= 3, "pieces of the path rows per thread");
        auto fetch = [&](int q) {                      // (clamped: the last piece again past the end)
            const int idx = min(t + q * NT, total - 1), c = idx % PR, node = sRnode[idx / PR];
            const char *src = c < PX ? xb + (uint32_t)(node * (int)R.x_sn + c * 8) * 2u
                                     : Bb + (uint32_t)(node * (int)R.b_sn + (c - PX) * 8) * 2u;
            return *reinterpret_cast<const uint4 *>(src);
        };
        auto put = [&](int q, uint4 v) {
            const int idx = min(t + q * NT, total - 1), c = idx % PR, j = idx / PR;
            *reinterpret_cast<uint4 *>(rbuf + (c < PX ? j * P + c * 8 : kRows * P + j * S + (c - PX) * 8) * 2) = v;
        };
        // (the second and third piece only where the path asks for them: most have at most eight nodes)
        const uint4 v0 = fetch(0);
        if (total > NT) {
            const uint4 v1 = fetch(1), v2 = fetch(2);
            put(1, v1);
            put(2, v2);
        }
        put(0, v0);
    };
    // LDS rows of the replayed path: behind the y staging area of the idle B tile
    char *const rrows = reinterpret_cast<char *>(sB) + kYStage;

    if (nU <= 0) return;
    // (b, h) of the current unit and of the next three.  The loop starts one unit early (k = -1):
    // that pass has no unit to compute and only runs the staging half, which brings unit 0 into
    // LDS and issues the loads of units 1 and 2 -- the same code as in the steady state, so the
    // instruction cache sees each part of the loop body once.
    int cb = ub0, ch = uh0, b1 = ub0, h1 = uh0;
    int b2 = b1, h2 = h1;
    step(b2, h2);
    int b3 = b2, h3 = h2;
    step(b3, h3);
    // One accumulator set serves both roles: the Y waves' Yt tiles of the current unit, or
    // (acc[0]) the G waves' Gt tile of the current (sequence, group), kept across its heads.
    floatx16 acc[YQ];

    // the first loads of every role, before anything is waited for.  With the replay the first state
    // tile is the exception (kLateH0): it is asked for once the tree wave knows the path of unit 0.
    // The replay of unit 0 is two dependent round trips (the previous tree's parents and step sizes,
    // then the rows of the path), and behind 16 KB of state per thread group and workgroup each of
    // them takes several times as long, while the first scan waits for them all the same.  The state
    // of unit 1 (G threads) goes out while the path is worked out and nothing else uses the memory
    // system: asked for behind the rows of that path it is what a workgroup of two or three units
    // waits for (48 heads in 8 groups, 34 nodes, fp32 state: batch 16 15.8 against 12.6 us, batch 33
    // 30.8 against 27.5 us; 80 heads, 64 nodes, batch 16: 22.9 against 22.0 us).
    constexpr bool kLateH0 = RP;
    if constexpr (kLateH0) {
#pragma unroll
        for (int q = 0; q < YQ; ++q)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
        if (!isY) {
            load_X(b1, h1);
            if (wave == kTreeWave) {
                load_T(b1, h1);
                load_R(b1, h1);
            }
        }
        if (wave == kTreeWave) path_R(b1, h1);
        if (!isY && h0 && nU > 1) load_H(b2, h2);
        __syncthreads();                                      // the path of unit 0 is in LDS
        if (isY) {
            if (h0) load_H(b1, h1);
        }
    } else {
        if (isY) {
            if (h0) load_H(b1, h1);
        } else {
            load_X(b1, h1);
            if (wave == kTreeWave) load_T(b1, h1);
        }
#pragma unroll
        for (int q = 0; q < YQ; ++q)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    }

    for (int k = -1; k < nU; ++k) {
        const bool live = k >= 0;                             // false in the staging-only first pass
        int bad = 0;
        float D_h = 0.f;
        if (live) {
            __syncthreads();                                  // barrier 1: unit k is staged
            bad = *sBad;
            D_h = *sDh;
            if (status && ch == 0 && tid == 0) status[cb] = bad;
        }
        const unsigned short *sXT = sXT2[k & 1];

        if (!live) {
        } else if (isY) {
#pragma unroll
            for (int q = 0; q < YQ; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
            // ---- phase 1: Yt = h0b C^T, then *= exp(s_i) -------------------------------------------
            if (h0 && !bad) {
                const int lnp = opaque(lane), l32 = lnp & 31, lh = lnp >> 5, it = RP ? (opaque(wave) & 1) : it0, il = it * 32 + l32;   // re-derived per phase
                const bf16_t *cp = &sC[il * SP + 8 * lh];
#pragma unroll
                for (int kb = 0; kb < S; kb += S / 2) {   // fragments of half the state index per batch
                    bf16x8 cf[S / 32], hf[YQ][S / 32];
#pragma unroll
                    for (int j = 0; j < S / 32; ++j) {
                        cf[j] = *reinterpret_cast<const bf16x8 *>(cp + kb + 16 * j);
#pragma unroll
                        for (int q = 0; q < YQ; ++q)
                            hf[q][j] = *reinterpret_cast<const bf16x8 *>(
                                &sH[(((wave + 4 * q) >> 1) * 32 + l32) * SP + 8 * lh + kb + 16 * j]);
                    }
#pragma unroll
                    for (int j = 0; j < S / 32; ++j)
#pragma unroll
                        for (int q = 0; q < YQ; ++q)
                            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hf[q][j], cf[j], acc[q], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);   // keep the batches apart: register budget
                }
                const float e = __builtin_amdgcn_exp2f(sS2[il]);
#pragma unroll
                for (int q = 0; q < YQ; ++q)
#pragma unroll
                    for (int rg = 0; rg < 16; ++rg) acc[q][rg] *= e;
            }
        } else if (wave != kTreeWave && !bad) {
            // ---- phase 2: Gt = B C^T (only when the C/B tiles are new), mask and decay -> M ----------
            const int jt = ((RP ? opaque(wave) : wave) - 4) >> 1;   // (see it0)
            const int lnp = opaque(lane), l32 = lnp & 31, lh = lnp >> 5, it = RP ? (opaque(wave) & 1) : it0, il = it * 32 + l32;   // re-derived per phase
            floatx16 &gt = acc[0];
            if (fresh_at(k, ch)) {
#pragma unroll
                for (int e = 0; e < 16; ++e) gt[e] = 0.f;
                const bf16_t *cp = &sC[il * SP + 8 * lh];
                const bf16_t *bp = &sB[(jt * 32 + l32) * SP + 8 * lh];
#pragma unroll
                for (int kb = 0; kb < S; kb += S / 2) {
                    bf16x8 cf[S / 32], bf[S / 32];
#pragma unroll
                    for (int j = 0; j < S / 32; ++j) {
                        cf[j] = *reinterpret_cast<const bf16x8 *>(cp + kb + 16 * j);
                        bf[j] = *reinterpret_cast<const bf16x8 *>(bp + kb + 16 * j);
                    }
#pragma unroll
                    for (int j = 0; j < S / 32; ++j)
                        gt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[j], cf[j], gt, 0, 0, 0);
                }
            }
            const float s2_i = sS2[il];
            const uint32_t mrow = sMask[il * 2 + jt] >> (4 * lh);   // bit 8*rg + e <-> j = jl + e
            float4 uj[4];
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) uj[rg] = *reinterpret_cast<const float4 *>(&sU[jt * 32 + 8 * rg + 4 * lh]);
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int jl = jt * 32 + 8 * rg + 4 * lh;
                const float ujv[4] = {uj[rg].x, uj[rg].y, uj[rg].z, uj[rg].w};
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // bitwise select: an overflowed exp2 under a cleared mask bit never reaches M
                    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)mrow, 8 * rg + e, 1);
                    const float v = gt[4 * rg + e] * __builtin_amdgcn_exp2f(s2_i - ujv[e]);
                    o[e] = (bf16_t)__uint_as_float(__float_as_uint(v) & keep);
                }
                *reinterpret_cast<bf16x4 *>(&sM[il * kNP64 + jl]) = o;
            }
        } else if (RP && wave == kTreeWave) {
            // ---- replay: path of unit k+1 on the previous tree and the loads of its x / B rows, in the
            //      half in which this wave has nothing else to do; they are written to LDS at the start
            //      of the staging half.  Then the parent / dt loads for the path of unit k+2.
            if (k + 1 < nU) {
                path_R(b1, h1);
                if (k + 2 < nU) load_R(b2, h2);
            }
        }
        if (live) __syncthreads();                            // barrier 2: M is ready; h0b, C and the tree arrays are dead

        const bool more = k + 1 < nU, more2 = k + 2 < nU, more3 = k + 3 < nU;
        const bool y_stages = (k & 1) != 0;    // unit k+1 is even: its h0 sits in the Y threads
        // new C / B tiles for unit k+1 overwrite the B tile's LDS, which this half uses as scratch
        // (y staging, replayed path rows): they wait for one more barrier (a).  Not in the first
        // pass, which has no such use and wants the tiles early.
        const bool fresh_next = more && fresh_at(k + 1, h1);
        const bool late_tiles = live && fresh_next;
        // replayed path rows of unit k+1: in the first pass the M tile's LDS (the B tile is being
        // written), later the B tile's
        [[maybe_unused]] char *rbuf = !live ? reinterpret_cast<char *>(sM) : rrows;
        if (isY) {
            // ---- phase 3: Yt += Xt M^T over j <= i only (nodes i < 32 have no ancestor j >= 32:
            //      that quadrant of M is never written or read); y = Yt + D x ---------------------------
            bf16x4 yreg[YQ][4];
            const int lnp = opaque(lane), l32 = lnp & 31, lh = lnp >> 5, it = RP ? (opaque(wave) & 1) : it0, il = it * 32 + l32;   // re-derived per phase
#pragma unroll
            for (int q = 0; q < YQ; ++q) {
                if (!live) break;
                const int pt = ((RP ? opaque(wave) : wave) + 4 * q) >> 1;   // (see it0)
                float xv[16];   // x[i][p] of this lane's node for the 16 p of its accumulator
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        xv[4 * rg + e] =
                            __uint_as_float((uint32_t)sXT[(pt * 32 + 8 * rg + 4 * lh + e) * kNP64 + il] << 16);
                if (!bad) {
                    const bf16_t *ap = reinterpret_cast<const bf16_t *>(sXT) + (pt * 32 + l32) * kNP64 + 8 * lh;
                    const bf16_t *bp = &sM[il * kNP64 + 8 * lh];
                    if (it) {
                        bf16x8 a[4], bb[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            a[j] = *reinterpret_cast<const bf16x8 *>(ap + 16 * j);
                            bb[j] = *reinterpret_cast<const bf16x8 *>(bp + 16 * j);
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j], bb[j], acc[q], 0, 0, 0);
                    } else {
                        bf16x8 a[2], bb[2];
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            a[j] = *reinterpret_cast<const bf16x8 *>(ap + 16 * j);
                            bb[j] = *reinterpret_cast<const bf16x8 *>(bp + 16 * j);
                        }
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j], bb[j], acc[q], 0, 0, 0);
                    }
                }
                // y = Yt + D x; kept in registers as bf16 until the stores further down
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[e] = bad ? (bf16_t)0.f : (bf16_t)fmaf(D_h, xv[4 * rg + e], acc[q][4 * rg + e]);
                    yreg[q][rg] = o;
                }
            }
            // first pass: the Y threads have nothing to scan and stage the first C / B tiles (later
            // tiles come from the G threads, after barrier (a))
            if (!live && fresh_next) restage_CB(b1, h1);
            if (RP && more) __syncthreads();                  // barrier (c): path rows of unit k+1 are in LDS
            // next unit's state tile (its loads have been in flight for a whole unit period), and behind it the
            // request for the state of unit k+3.  Unit 2 is the exception: asked for in the first pass it would
            // sit in the memory queues in front of the small x / parent / dt loads of units 1 and 2 and make the
            // last scan wait for them; asked for one pass later, the state of the last unit of a short run is the
            // last thing to arrive.  (With the replay ahead of the y stores: the compiler cannot tell that these registers'
            // last loads have been waited for and waits for everything in front of the next ones, stores included.  Without
            // it the stores go first: 40 heads x 128, 64 nodes at batch 16: 17.2 against 18.2 us.)
            if (more) {
                if (h0) {
                    if (y_stages) stage_H(rbuf, b1, h1);
                } else if (rt == 0) {
                    *sDh = D ? D[h1] : 0.f;
                }
            }
            auto later_states = [&]() {
                if (h0 && more3 && y_stages && live) load_H(b3, h3);
                if (h0 && more2 && k == 0) load_H(b2, h2);
            };
            if constexpr (RP) later_states();
            // y leaves as 64-byte row pieces: the accumulators give a lane 4 consecutive p of one
            // node, which as direct stores would be 16-byte pieces of 32 different lines per
            // instruction.  Each wave therefore turns its 32x32 tile around in a private 2 KB of LDS
            // (a wave's LDS operations complete in order: no barrier) and stores 16 bytes per lane,
            // four lanes to a row.  The LDS used is the B tile's, which is idle in this half.
            // The stores go out after the wait for the h0 loads above and are long complete at
            // the next such wait: on gfx9 loads and stores share one counter and complete out of
            // order with respect to each other, so a store in flight would turn that wait into a
            // wait for everything.
            if (live) {
                char *yb = reinterpret_cast<char *>(y + (size_t)cb * n * H * P + (size_t)ch * P);
                char *ys = reinterpret_cast<char *>(sB) + opaque(wave) * 2048;
                const int ln = opaque(lane), wr = ln & 31, wh = ln >> 5;
                const int rr = ln >> 2, rc = ln & 3;
#pragma unroll
                for (int q = 0; q < YQ; ++q) {
                    const int pt = (wave + 4 * q) >> 1;
                    // row r keeps its 16-byte chunk c at slot c ^ ((r >> 2) & 3)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg)
                        *reinterpret_cast<bf16x4 *>(ys + wr * 64 + ((rg ^ ((wr >> 2) & 3)) * 16) + wh * 8) =
                            yreg[q][rg];
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int row = half * 16 + rr;
                        const uint4 v =
                            *reinterpret_cast<const uint4 *>(ys + row * 64 + ((rc ^ ((row >> 2) & 3)) * 16));
                        const int node = (RP ? (opaque(wave) & 1) : it0) * 32 + row;
                        if (node < n)
                            store_through16(yb + (uint32_t)(node * H * P + pt * 32 + rc * 8) * 2u, v);
                    }
                }
            }
            if constexpr (!RP) later_states();
            if (late_tiles) __syncthreads();                  // barrier (a): scratch use of the B tile is over
        } else if (more) {
            if constexpr (RP) {
                if (wave == kTreeWave) {
                    if (!live && more2) load_R(b2, h2);
                } else {
                    fetch_R(rbuf, b1, h1);
                }
                __syncthreads();                           // barrier (c)
            }
            if (wave == kTreeWave) {
                stage_T(h1);
                // (the path inputs of unit k+2 are waited for here, with the others, and not at the start of the next
                // scan half, where the state tile requested below would be waited for with them)
                if constexpr (RP) asm volatile("" : "+v"(rpp), "+v"(rpdt));
            }
            stage_X((k + 1) & 1);                          // the other X^T tile: unit k still reads its own
            // the registers just staged are free: x and parent / dt of unit k+2 go out at once (a
            // pass is short when HBM is idle, and they are needed at this point of the next one)
            if (more2) {
                load_X(b2, h2);
                if (wave == kTreeWave) load_T(b2, h2);
            }
            if (h0 && !y_stages) {
                stage_H(rbuf, b1, h1);
                if (more3) load_H(b3, h3);
            }
            if (!RP && more2 && !live && h0) load_H(b2, h2);   // unit 1: the first odd unit (with the replay: before the loop)
            if (late_tiles) {
                __syncthreads();                           // barrier (a)
                restage_CB(b1, h1);
            }
        }
        cb = b1; ch = h1;
        b1 = b2; h1 = h2;
        b2 = b3; h2 = h3;
        step(b3, h3);
    }
}

template <int P, int S, bool RP, typename HT>
hipError_t launch64(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                    const void *Bm, const void *Cm, const float *D, const void *h0, void *y,
                    int32_t *status, const ReplayArgs &R, hipStream_t st) {
    constexpr size_t lds = RP ? Lds64<P, S>::total_replay : Lds64<P, S>::total;   // static LDS (upper bound)
    constexpr int kPerCU = 2 * (lds + 64) <= 160 * 1024 ? 2 : 1;                  // workgroups
    const int n_units = d.batch * d.nheads;
    const int grid = n_units > 256 * kPerCU ? 256 * kPerCU : (n_units + 7) / 8 * 8;
    // (the in-kernel softplus is a variant of its own: compiled into the common one, even unused, it costs time)
#define STREE_LAUNCH64(SPL)                                                                                         \
    hipLaunchKernelGGL((tree_ssd_mfma64_kernel<P, S, 2 * kPerCU, RP, SPL, HT>), dim3(grid), dim3(kT64), 0, st, parent,          \
                       d.nnodes, d.batch, d.nheads, d.ngroups, (const bf16_t *)x, (long)d.x_stride_n, dt,           \
                       step_bias(d), A, (const bf16_t *)Bm, (long)d.b_stride_n, (const bf16_t *)Cm,                 \
                       (long)d.c_stride_n, D, (const HT *)h0, (bf16_t *)y, status, R)
    if (step_bias(d)) STREE_LAUNCH64(true);
    else STREE_LAUNCH64(false);
#undef STREE_LAUNCH64
    return hipGetLastError();
}

// The bands in which the persistent kernel is ahead of a workgroup per head: so many heads that (nearly) all of them enter
// the workgroup-per-head kernel at once and read their C and B rows at once, where a persistent workgroup reads them once
// for the two or three heads it walks; the more nodes, the more so, and most where its workgroups (two a CU) have the same
// number of heads each.  80 heads, S = 128, us, persistent / per head, fp32 state:
//   replay + scan   batch 8, 64 nodes 14.8 / 15.5, 50 nodes 14.8 / 14.5; 9, 58 nodes 14.9 / 15.4, 48 nodes 15.3 / 14.6; 11, 44
//                   nodes 18.5 / 19.7; 12, 64 19.6 / 20.8; 15, 48 22.6 / 23.7; 16, 64 23.3 / 24.9; 18 27.9 / 27.5; 19, 54 27.0 / 27.6
//   scan            batch 10, 64 nodes 12.7 / 13.1; 14, 64 14.0 / 15.8, 44 13.4 / 13.8, 36 13.2 / 13.0; 19, 48 16.6 / 16.9; 21, 64
//                   19.0 / 20.0; 24 22.6 / 22.0; S = 64, batch 14, 64 11.5 / 11.8, 16 11.8 / 12.3
// and with a state in bf16, half the bytes:
//   replay + scan   batch 14, 64 nodes 17.9 / 18.3; 15, 44 17.3 / 17.5; 16, 64 18.2 / 18.4, 48 17.3 / 17.0
//   scan            batch 14, 54 nodes 11.9 / 12.3; 16, 58 12.0 / 12.8; 18, 64 14.4 / 15.1, 58 14.3 / 14.5; 64, 64 36.7 / 38.0
// Headdim 128 (one persistent workgroup a CU), replay + scan, fp32 state: 440 heads, 64 nodes 18.8 / 20.9, 40 nodes 18.6 / 19.5;
// 380 heads 18.4 / 15.6, 520 heads 27.6 / 22.9.  Elsewhere the workgroup per head is ahead by 2 to 30 %.
bool unit_is_slower(const stree_dims &d, bool replay) {
    const int heads = d.batch * d.nheads, n = d.nnodes;
    const bool f32 = d.state_dtype == STREE_F32;
    if (d.headdim == 128) return replay && f32 && heads > 384 && heads <= 512 && n > 36;
    if (d.dstate == 64) return !replay && f32 && heads > 1088 && heads <= 1280 && n > 56;
    if (d.dstate != 128) return false;
    int from = 65;                                    // nodes from which it is
    if (!f32 && replay) from = heads <= 1024 ? 65 : heads <= 1216 ? 41 : heads <= 1280 ? 61 : 65;
    else if (!f32) from = heads <= 1024 ? 65 : heads <= 1280 ? 53 : 59;
    else if (replay) from = heads <= 512 ? 65 : heads <= 640 ? 55 : heads <= 768 ? 53 : heads <= 1408 ? 33 : heads <= 1472 ? 65 : heads <= 1536 ? 49 : 65;
    else from = heads <= 768 ? 65 : heads <= 1024 ? 57 : heads <= 1280 ? 41 : heads <= 1700 ? 45 : 65;
    return n >= from;
}

}  // namespace

// (Rows past a small tree are addressed as well, with 32-bit byte offsets that have to lie behind its last row: token strides
// for which 64 rows outgrow those, never met in earnest, go to the kernel for every head shape.)
bool tree_ssd_mfma64_supported(const stree_dims &d) {
    if (d.nnodes > kB64) return false;
    if (d.x_stride_n >= (1L << 25) || d.b_stride_n >= (1L << 25) || d.c_stride_n >= (1L << 25)) return false;
    const int P = d.headdim, S = d.dstate;
    return (P == 64 && (S == 128 || S == 64 || S == 256)) || (P == 128 && S == 128);
}

bool tree_ssd_replay_fused_supported(const stree_dims &d, const stree_dims &dp, const void *px, const void *pB,
                                     const void *x, const void *Bm, const void *Cm, const void *y, const void *h0,
                                     const void *h_out) {
    if (d.nnodes > kB64) return tree_ssd_replay_rows_supported(d, dp, px, pB, x, Bm, Cm, y, h0, h_out);
    if (d.io_dtype != STREE_BF16 || !tree_ssd_mfma64_supported(d) || dp.nnodes > kB64) return false;
    if ((d.x_stride_n | d.b_stride_n | d.c_stride_n | dp.x_stride_n | dp.b_stride_n) % 8 != 0) return false;
    const uintptr_t bits = (uintptr_t)x | (uintptr_t)Bm | (uintptr_t)Cm | (uintptr_t)y | (uintptr_t)px | (uintptr_t)pB |
                           (uintptr_t)h0 | (uintptr_t)h_out;   // (the state is read and written 16 bytes at a time)
    return bits % 16 == 0;
}

hipError_t launch_tree_ssd_replay_fused(const stree_dims &d, const stree_dims &dp, const int32_t *pparent,
                                        const int32_t *paccepted, const void *px, const float *pdt, const void *pB,
                                        const int32_t *parent, const void *x, const float *dt, const float *A,
                                        const void *Bm, const void *Cm, const float *D, const void *h0,
                                        void *h_out, void *y, int32_t *status, int32_t *rstatus, hipStream_t st) {
    if (d.nnodes > kB64)
        return launch_tree_ssd_replay_rows(d, dp, pparent, paccepted, px, pdt, pB, parent, x, dt, A, Bm, Cm, D, h0, h_out, y,
                                           status, rstatus, st);
    if (!unit_is_slower(d, true))
        return launch_tree_ssd_replay_unit(d, dp, pparent, paccepted, px, pdt, pB, parent, x, dt, A, Bm, Cm, D, h0, h_out, y,
                                           status, rstatus, st);
    const ReplayArgs R = {pparent, paccepted, (const bf16_t *)px, (const bf16_t *)pB, pdt,
                          (long)dp.x_stride_n, (long)dp.b_stride_n, dp.nnodes, h_out, rstatus};
    const auto launch = d.headdim == 128 ? launch64<128, 128, true, float>
                        : d.state_dtype == STREE_F32 ? launch64<64, 128, true, float> : launch64<64, 128, true, bf16_t>;
    return launch(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, R, st);
}

hipError_t launch_tree_ssd_mfma64(const stree_dims &d, const int32_t *parent, const void *x, const float *dt,
                                  const float *A, const void *Bm, const void *Cm, const float *D,
                                  const void *h0, void *y, int32_t *status, hipStream_t st) {
    if (!unit_is_slower(d, false)) return launch_tree_ssd_unit(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
    const auto launch = d.dstate == 64 ? launch64<64, 64, false, float>
                        : d.state_dtype == STREE_F32 ? launch64<64, 128, false, float> : launch64<64, 128, false, bf16_t>;
    return launch(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, ReplayArgs{}, st);
}

}  // namespace stree
