// Tree scan in fp32 for trees of at most 64 nodes on the fp32 matrix units (dstate 64, 128 or 256, rows on 16-byte
// boundaries); tree_ssd_fma.hip keeps every other fp32 shape.
//
// One wave per (sequence, head, 32 nodes, 32 columns of P), no LDS tiles and no barriers: the layer in fp32 is a small
// problem (a state of 32 KB per head), and what it costs is the length of the chain from the first request to the
// last store.  A wave asks for its C, B and state rows at once, straight into the operand registers, works the tree
// index out meanwhile (lane = node, pointer doubling across lanes), and then only computes:
//   Gt[j][i] = <B_j, C_i>,  M = L ? Gt exp(s_i - s_j) dt_j : 0,  Y[i][p] = exp(s_i) <C_i, h0_p> + sum_j M_ij x_jp + D x_ip
//
// v_mfma_f32_32x32x2_f32 takes, in lane l, row l%32 of an operand and one k per half wave; four steps' worth of k are
// the four floats of one 16-byte piece (the order of k is free as long as both operands agree: step t of a group of
// eight stands for columns 4(l/32) + t).  The accumulator Gt holds, in lane l, column i = l%32 and rows
// j = 8(r/4) + 4(l/32) + r%4, which makes its registers, weighted in place, the M operand of sixteen steps whose x rows
// are read from memory as they lie; D x uses the same x registers.
//
// A matrix instruction multiplies the weight 0 of a node that is no ancestor with that node's x, and 0 times an infinity
// or NaN would spread one bad node over every row of the tile.  So values of x that are not finite enter the matrix
// instructions as 0, and a wave that met one adds them to the rows that have a weight for them, one by one: the FMA
// kernel's results, at the price of two vector instructions per x register otherwise.
//
// What bounds it is that chain: the loads (about 2 us), 64 + 64 dependent steps of 64 cycles (S = 128), 16 more per
// column tile, launch and store.  Measured, against the FMA kernel (one workgroup per head, 16 rows at a time through
// LDS): batch 4 x 31 nodes x 80 heads, S = 128: 101 -> 13.5 us; 15 nodes x 4 heads, S = 64: 25.2 -> 8.2 us.
#include "common.hpp"
#include "launch.hpp"

namespace stree {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int S>
__global__ __launch_bounds__(64, 1) void tree_ssd_f32_kernel(
    const int32_t *__restrict__ parent, int n, int H, int P, int G, int units, const float *__restrict__ x, long x_sn,
    const float *__restrict__ dt, const float *__restrict__ dt_bias, const float *__restrict__ A,
    const float *__restrict__ Bm, long b_sn, const float *__restrict__ Cm, long c_sn, const float *__restrict__ D,
    const float *__restrict__ h0, float *__restrict__ y, int32_t *__restrict__ status) {
    constexpr int KC = S < 128 ? S : 128;             // state columns in registers at a time
    constexpr int NG = KC / 8;                        // groups of eight: one 16-byte piece per lane, four steps
    __shared__ __align__(16) float sS[64], sDt[64];
    __shared__ float sM[32 * 33], sX[32 * 33];        // weights [j][i] and x [j][p] of a tile whose x is not finite throughout
    const int unit = unit_of_block(units);
    if (unit < 0) return;
    const int lane = threadIdx.x, l32 = lane & 31, lh = lane >> 5;
    const int pts = (P + 31) / 32, its = (n + 31) / 32;
    const int it = its - 1 - unit % its;              // (the longer row block first)
    const int pt = unit / its % pts, bh = unit / (its * pts), b = bh / H, h = bh % H, g = h / (H / G);
    const int p = pt * 32 + l32, pc = min(p, P - 1), i = it * 32 + l32;
    const float *crow = Cm + ((size_t)b * n + min(i, n - 1)) * c_sn + (size_t)g * S + 4 * lh;
    const float *hrow = h0 ? h0 + ((size_t)bh * P + pc) * S + 4 * lh : nullptr;
    const float *bbase = Bm + (size_t)b * n * b_sn + (size_t)g * S + 4 * lh;
    const float *xbase = x + (size_t)b * n * x_sn + (size_t)h * P + pc;

    // the tree index' inputs first: everything else is only needed behind it
    const int par = lane < n ? parent[(size_t)b * n + lane] : -1;
    const float raw = lane < n ? dt[((size_t)b * n + lane) * H + h] : 0.f;
    f32x4 c[NG], k[NG];                               // k: state rows, then B rows
#pragma unroll
    for (int q = 0; q < NG; ++q) c[q] = *reinterpret_cast<const f32x4 *>(crow + 8 * q);
    if (hrow) {
#pragma unroll
        for (int q = 0; q < NG; ++q) k[q] = *reinterpret_cast<const f32x4 *>(hrow + 8 * q);
    }
    f32x4 bv[NG];
    const float *brow = bbase + (size_t)min(l32, n - 1) * b_sn;
#pragma unroll
    for (int q = 0; q < NG; ++q) bv[q] = *reinterpret_cast<const f32x4 *>(brow + 8 * q);

    // depth sums and ancestor bits, lane = node
    int pj = par;
    const bool ok = lane >= n || (lane == 0 ? pj == -1 : pj >= 0 && pj < lane);
    const unsigned long long badmask = __ballot(!ok);
    const float A_h = A[h], D_h = D ? D[h] : 0.f;
    const int bad = badmask ? __ffsll((long long)badmask) : 0;
    if (status && h == 0 && pt == 0 && it == its - 1 && lane == 0) status[b] = bad;
    float *yrow = y + ((size_t)b * n + it * 32) * H * P + (size_t)h * P + p;
    if (bad) {
        for (int r = lh; r < 32; r += 2)
            if (it * 32 + r < n && p < P) yrow[(size_t)r * H * P] = 0.f;
        return;
    }
    const float dt_j = lane < n ? (dt_bias ? softplus_step(raw + dt_bias[h]) : raw) : 0.f;
    float s = dt_j * A_h;
    unsigned long long m = 1ull << lane;
    for (int round = 0; round < 6; ++round) {
        if (!__any(pj >= 0)) break;
        const int q = pj >= 0 ? pj : lane;
        const float rs = wave_read(s, q);
        const int rp = wave_read(pj, q);
        const unsigned long long rm = wave_read(m, q);
        if (pj >= 0) {
            s += rs;
            m |= rm;
            pj = rp;
        }
    }
    sS[lane] = s;                                     // (one wave: no barrier)
    sDt[lane] = dt_j;
    const float s_i = wave_read(s, min(i, 63));
    const unsigned long long m_i = wave_read(m, min(i, 63));

    auto steps = [](floatx16 &acc, const f32x4 (&a)[NG], const f32x4 (&b_)[NG]) {
#pragma unroll
        for (int q = 0; q < NG; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][t], b_[q][t], acc, 0, 0, 0);
    };
    floatx16 acc, gt;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = gt[e] = 0.f;
    if (hrow) steps(acc, c, k);
    steps(gt, bv, c);
    if constexpr (S > KC) {                           // the second half of the state columns
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            c[q] = *reinterpret_cast<const f32x4 *>(crow + KC + 8 * q);
            bv[q] = *reinterpret_cast<const f32x4 *>(brow + KC + 8 * q);
            if (hrow) k[q] = *reinterpret_cast<const f32x4 *>(hrow + KC + 8 * q);
        }
        if (hrow) steps(acc, c, k);
        steps(gt, bv, c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {                     // rows of C h0 by exp(s_i) (no state: 0 by 1, whatever s_i is)
        const f32x4 sv = *reinterpret_cast<const f32x4 *>(&sS[it * 32 + 8 * q + 4 * lh]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * q + e] *= expf(hrow ? sv[e] : 0.f);
    }
    float xv[16];
    auto column_tile = [&](int jt) {                  // += M x over the nodes 32 jt ..
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int j = jt * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
            xv[r] = xbase[(size_t)min(j, n - 1) * x_sn];
        }
        // weights of nodes j0 + e, j0 = jt * 32 + 8 q + 4 lh, for row i (a select: a non-ancestor's weight may overflow)
        auto weights = [&](int q) {
            const int j0 = jt * 32 + 8 * q + 4 * lh;
            const f32x4 sv = *reinterpret_cast<const f32x4 *>(&sS[j0]), dv = *reinterpret_cast<const f32x4 *>(&sDt[j0]);
            f32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = gt[4 * q + e] * expf(s_i - sv[e]) * dv[e];
                w[e] = (m_i >> (j0 + e)) & 1ull ? v : 0.f;
            }
            return w;
        };
        bool spoiled = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 w = weights(q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool fin = __builtin_isfinite(xv[4 * q + e]);
                spoiled |= !fin;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], fin ? xv[4 * q + e] : 0.f, acc, 0, 0, 0);
            }
        }
        if (__any(spoiled)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 w = weights(q);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sM[(8 * q + 4 * lh + e) * 33 + l32] = w[e];
                    sX[(8 * q + 4 * lh + e) * 33 + l32] = xv[4 * q + e];
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int j = 0; j < 32; ++j) {
                const float xj = sX[j * 33 + l32];
                if (__builtin_isfinite(xj)) continue;
#pragma unroll
                for (int r = 0; r < 16; ++r) {        // accumulator rows
                    const float w = sM[j * 33 + 8 * (r >> 2) + 4 * lh + (r & 3)];
                    if (w != 0.f) acc[r] = fmaf(w, xj, acc[r]);
                }
            }
            __syncthreads();
        }
    };
    column_tile(0);
    if (it > 0) {                                     // (n > 32) Gt of the other column tile, then the rest of the sum
        const float *row = bbase + (size_t)min(32 + l32, n - 1) * b_sn;
#pragma unroll
        for (int e = 0; e < 16; ++e) gt[e] = 0.f;
#pragma unroll
        for (int s0 = S - KC; s0 >= 0; s0 -= KC) {
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                bv[q] = *reinterpret_cast<const f32x4 *>(row + s0 + 8 * q);
                if (S > KC) c[q] = *reinterpret_cast<const f32x4 *>(crow + s0 + 8 * q);
            }
            steps(gt, bv, c);
        }
        column_tile(1);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {                    // xv: the x rows of this row block (its own column tile came last)
        const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
        if (it * 32 + row < n && p < P) yrow[(size_t)row * H * P] = fmaf(D_h, xv[r], acc[r]);
    }
}

}  // namespace

static int64_t units_of(const stree_dims &d) {
    return (int64_t)d.batch * d.nheads * ((d.headdim + 31) / 32) * ((d.nnodes + 31) / 32);
}

// Trees of at most 64 nodes, dstate a tile of the kernel, rows of B, C and the state on 16-byte boundaries, and no more
// waves than one grid dimension takes (2^32 work items; the FMA kernel's grid has two).  Without a state, a few nodes
// of a wide head stay with the FMA kernel too: every 32 columns have a wave of their own here, which forms <B, C> for 32
// rows again.  64 sequences, S = 128: 40 heads of 128 columns, one node 47.9 us, FMA kernel 38.8 us, two 48.8 and 42.0 us,
// four 50.3 and 50.9 us; 20 heads of 192, four nodes 38.5 and 32.1 us, five 40.6 and 37.9 us; 80 heads of 64, one node 47.8
// and 52.6 us.  S = 64, 40 heads of 96, two nodes 28.3 and 24.0 us.
bool tree_ssd_f32_supported(const stree_dims &d, const void *Bm, const void *Cm, const void *h0) {
    if (d.io_dtype != STREE_F32 || d.nnodes > 64) return false;
    if (d.dstate != 64 && d.dstate != 128 && d.dstate != 256) return false;
    const int tiles = (d.headdim + 31) / 32;
    if (!h0 && d.nnodes <= (tiles < 3 ? 0 : tiles < 5 ? 2 : 4)) return false;
    if ((d.b_stride_n | d.c_stride_n) % 4 != 0 || units_of(d) > (1L << 25)) return false;
    return (((uintptr_t)Bm | (uintptr_t)Cm | (uintptr_t)h0) % 16) == 0;
}

template <int S>
static hipError_t launch_f32_s(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                               const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                               hipStream_t st) {
    const int units = (int)units_of(d);
    hipLaunchKernelGGL((tree_ssd_f32_kernel<S>), dim3(8 * ((units + 7) / 8)), dim3(64), 0, st, parent, d.nnodes, d.nheads,
                       d.headdim, d.ngroups, units, (const float *)x, (long)d.x_stride_n, dt, step_bias(d), A,
                       (const float *)Bm, (long)d.b_stride_n, (const float *)Cm, (long)d.c_stride_n, D,
                       (const float *)h0, (float *)y, status);
    return hipGetLastError();
}

hipError_t launch_tree_ssd_f32(const stree_dims &d, const int32_t *parent, const void *x, const float *dt, const float *A,
                               const void *Bm, const void *Cm, const float *D, const void *h0, void *y, int32_t *status,
                               hipStream_t st) {
    switch (d.dstate) {
        case 64: return launch_f32_s<64>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
        case 128: return launch_f32_s<128>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
        case 256: return launch_f32_s<256>(d, parent, x, dt, A, Bm, Cm, D, h0, y, status, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace stree
