// stree_gate_norm: output gate and grouped RMS norm of the Mamba2 block behind the tree scan,
//   v   = y * silu(z)
//   out = v / sqrt(mean over the channel group of v^2 + eps) * w
// per node, the H*P channels split into `ngroups` runs of consecutive channels.
//
// Streaming kernel: y and z are read once, out is written once.  A norm group spans the heads of a
// group (all heads when ngroups = 1), i.e. many (batch, head) units of the scan kernels, so the
// step cannot ride on a unit's y store; fused there it would move the z read into the scan and save
// no byte.  Some lanes of a wave or one workgroup per (node, group) segment, by its size; the gated
// values stay in registers between the sum of squares and the scaling.
#include "common.hpp"
#include "launch.hpp"

namespace stree {

namespace {

template <typename T>
struct Pack16;
template <>
struct Pack16<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void unpack(const uint4 &v, float (&o)[4]) {
        o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ uint4 pack(const float (&o)[4]) {
        return make_uint4(__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3]));
    }
};
template <>
struct Pack16<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void unpack(const uint4 &v, float (&o)[8]) {
        o[0] = bf16_lo(v.x); o[1] = bf16_hi(v.x); o[2] = bf16_lo(v.y); o[3] = bf16_hi(v.y);
        o[4] = bf16_lo(v.z); o[5] = bf16_hi(v.z); o[6] = bf16_lo(v.w); o[7] = bf16_hi(v.w);
    }
    static __device__ __forceinline__ uint4 pack(const float (&o)[8]) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (bf16_t)o[e];
        return __builtin_bit_cast(uint4, v);
    }
};

__device__ __forceinline__ float gate(float y, float z) { return y * z * __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

// sum over the workgroup (whole waves: WAVES of them, or up to 16 where that is 0); every thread gets the result
template <int WAVES>
__device__ __forceinline__ float block_sum(float v) {
    __shared__ float part[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < (WAVES ? WAVES : (int)blockDim.x / 64); ++w) s += part[w];
    return s;
}

// TEAM threads per segment: 16, 32 or 64 lanes of a wave (a workgroup of 256 threads then takes 256 / TEAM segments
// and needs no barrier), 256 = that workgroup, or 0 = a workgroup whose size follows the segment's.  CPT = 16-byte
// chunks of a segment per thread.
//
// HBM-bound, and what keeps many segments from the memory's rate is idle lanes: with one workgroup of 256 threads per
// segment the 80 chunks of a group of 640 bf16 channels used 80 of 256 threads and one barrier for 2.5 KB of loads.
// (Figures: the rule in launch_t.)
template <typename T, int CPT, int TEAM>
__global__ __launch_bounds__(TEAM ? kThreads : 1024) void gate_norm_kernel(const T *__restrict__ y,
                                                                           const T *__restrict__ z, long z_sn,
                                                                           const T *__restrict__ w, T *out, int d, int G,
                                                                           int gs, float eps, int segs) {
    constexpr int EPV = Pack16<T>::N;
    const int team = TEAM ? TEAM : (int)blockDim.x;
    const int t = TEAM ? (int)threadIdx.x & (team - 1) : (int)threadIdx.x;
    constexpr bool kWhole = TEAM == kThreads || TEAM == 0;     // a workgroup per segment
    const unsigned own = kWhole ? blockIdx.x : blockIdx.x * (kThreads / (TEAM ? TEAM : 1)) + threadIdx.x / team;
    // (lanes past the last segment follow along and store nothing)
    const unsigned seg = kWhole ? own : min(own, (unsigned)segs - 1u);
    const int row = seg / G, g = seg % G;
    const size_t oy = (size_t)row * d + (size_t)g * gs, oz = (size_t)row * z_sn + (size_t)g * gs;
    const int chunks = gs / EPV;
    float v[CPT][EPV];
    uint4 ry[CPT], rz[CPT];
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        const int c = min(q * team + t, chunks - 1);
        ry[q] = load_stream16(y + oy + (size_t)c * EPV);
        rz[q] = load_stream16(z + oz + (size_t)c * EPV);
    }
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        float fy[EPV], fz[EPV];
        Pack16<T>::unpack(ry[q], fy);
        Pack16<T>::unpack(rz[q], fz);
        const bool live = q * team + t < chunks;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            v[q][e] = live ? gate(fy[e], fz[e]) : 0.f;
            ss = fmaf(v[q][e], v[q][e], ss);
        }
    }
    if constexpr (kWhole) {
        ss = block_sum<TEAM / 64>(ss);
    } else {
#pragma unroll
        for (int o = TEAM / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    }
    const float scale = rsqrtf(ss / (float)gs + eps);
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        const int c = q * team + t;
        if (c < chunks && (kWhole || own < (unsigned)segs)) {
            float fw[EPV], o[EPV];
            Pack16<T>::unpack(*reinterpret_cast<const uint4 *>(w + (size_t)g * gs + (size_t)c * EPV), fw);
#pragma unroll
            for (int e = 0; e < EPV; ++e) o[e] = v[q][e] * scale * fw[e];
            store_stream16(out + oy + (size_t)c * EPV, Pack16<T>::pack(o));
        }
    }
}

// any group size, any alignment: two passes over the segment, one element at a time
template <typename T>
__global__ __launch_bounds__(kThreads) void gate_norm_plain_kernel(const T *__restrict__ y, const T *__restrict__ z,
                                                                   long z_sn, const T *__restrict__ w, T *out, int d,
                                                                   int G, int gs, float eps) {
    const int row = blockIdx.x / G, g = blockIdx.x % G;
    const size_t oy = (size_t)row * d + (size_t)g * gs, oz = (size_t)row * z_sn + (size_t)g * gs;
    float ss = 0.f;
    for (int c = threadIdx.x; c < gs; c += kThreads) {
        const float v = gate(to_f32(y[oy + c]), to_f32(z[oz + c]));
        ss = fmaf(v, v, ss);
    }
    const float scale = rsqrtf(block_sum<kThreads / 64>(ss) / (float)gs + eps);
    for (int c = threadIdx.x; c < gs; c += kThreads) {
        const float v = gate(to_f32(y[oy + c]), to_f32(z[oz + c]));
        T o;
        from_f32(v * scale * to_f32(w[(size_t)g * gs + c]), o);
        out[oy + c] = o;
    }
}

template <typename T>
hipError_t launch_t(const stree_dims &d, const void *y, const void *z, long z_sn, const void *w, float eps, void *out,
                    hipStream_t st) {
    constexpr int EPV = Pack16<T>::N;
    const int dd = d.nheads * d.headdim, G = d.ngroups, gs = dd / G;
    const long segs = (long)d.batch * d.nnodes * G;
    const bool vec = gs % EPV == 0 && z_sn % EPV == 0 &&
                     (((uintptr_t)y | (uintptr_t)z | (uintptr_t)w | (uintptr_t)out) % 16) == 0;
    const int chunks = vec ? gs / EPV : 0;
#define STREE_GN_VEC(CPT, TEAM, GRID, THREADS)                                                                       \
    hipLaunchKernelGGL((gate_norm_kernel<T, CPT, TEAM>), dim3((unsigned)(GRID)), dim3(THREADS), 0, st, (const T *)y,  \
                       (const T *)z, z_sn, (const T *)w, (T *)out, dd, G, gs, eps, (int)segs)
#define STREE_GN_TEAM(TEAM)                                                                                          \
    do {                                                                                                             \
        const long grid = (segs + kThreads / TEAM - 1) / (kThreads / TEAM);                                          \
        const int cpt = (chunks + TEAM - 1) / TEAM;                                                                  \
        if (cpt == 1) STREE_GN_VEC(1, TEAM, grid, kThreads);                                                         \
        else if (cpt == 2) STREE_GN_VEC(2, TEAM, grid, kThreads);                                                    \
        else if (cpt == 3) STREE_GN_VEC(3, TEAM, grid, kThreads);                                                    \
        else if (cpt == 4) STREE_GN_VEC(4, TEAM, grid, kThreads);                                                    \
        else STREE_GN_VEC(5, TEAM, grid, kThreads);                                                                  \
    } while (0)
    // Many segments: lanes of one wave for each, as few as hold it in five chunks a lane, which fills the chip.  25088
    // segments of 80 chunks 30.0 us with a workgroup each, 19.6 us with 16 lanes each (4.9 TB/s, the rate of a plain
    // copy); 8192 of 128 chunks 12.6 -> 9.3 us with 32 lanes; 4096 of 256 chunks 10.2 -> 9.4 us with 64; 2048 of 128
    // chunks 4.5 -> 4.3 us.  Above 256 chunks a wave's loads are more than keeps enough waves on a CU once memory is the
    // bound: 4096 segments of 320 chunks 12.6 -> 10.7 us, but 16384 of them 40.9 -> 43.1 us.
    // Few segments are a matter of latency, and every chunk more a lane is more of it, so they get a workgroup: 64
    // segments of 192 chunks 3.5 us so, 4.2 us with a wave; 500 of 256 chunks 4.2 and 5.5 us, 2048 of them 5.3 and 6.3 us.
    // With one chunk a lane a wave waits no longer: 2000 segments of 16 chunks 3.7 us with a workgroup, 3.0 us with a wave,
    // 250 of 32 or 64 the same, 120 of 16 2.7 and 2.9 us.
    // Larger segments take a workgroup: 256 threads up to four chunks a thread (1024 rows of 640 chunks in a decoding
    // step: 320 threads of two chunks cost 0.5 us more), then as many as four chunks a thread ask for.  124 rows of
    // 1280 fp32 chunks took 12.9 us in the two-pass kernel, 4.7 us so.
    const int wave_chunks = segs < 256 ? 0 : segs < 2048 ? 64 : segs < 4096 ? 128 : segs < 8192 ? 320 : 256;
    const bool many = segs >= 4096;
    if (chunks == 0 || chunks > 4096)
        hipLaunchKernelGGL((gate_norm_plain_kernel<T>), dim3((unsigned)segs), dim3(kThreads), 0, st, (const T *)y,
                           (const T *)z, z_sn, (const T *)w, (T *)out, dd, G, gs, eps);
    else if (many && chunks <= 16 * 5) STREE_GN_TEAM(16);
    else if (many && chunks <= 32 * 5) STREE_GN_TEAM(32);
    else if (chunks <= wave_chunks) STREE_GN_TEAM(64);
    else if (chunks <= kThreads) STREE_GN_VEC(1, kThreads, segs, kThreads);
    else if (chunks <= 2 * kThreads) STREE_GN_VEC(2, kThreads, segs, kThreads);
    else if (chunks <= 3 * kThreads) STREE_GN_VEC(3, kThreads, segs, kThreads);
    else if (chunks <= 4 * kThreads) STREE_GN_VEC(4, kThreads, segs, kThreads);
    else STREE_GN_VEC(4, 0, segs, (chunks + 255) / 256 * 64);
#undef STREE_GN_TEAM
#undef STREE_GN_VEC
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gate_norm(const stree_dims &d, const void *y, const void *z, long z_sn, const void *w, float eps,
                            void *out, hipStream_t st) {
    if (d.io_dtype == STREE_BF16) return launch_t<bf16_t>(d, y, z, z_sn, w, eps, out, st);
    return launch_t<float>(d, y, z, z_sn, w, eps, out, st);
}

}  // namespace stree
