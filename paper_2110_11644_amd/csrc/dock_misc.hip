// Small kernels (grid conversion, counter reset) and the dispatch of the dock
// launches over texel storage types.
#include <math.h>

#include <algorithm>

#include "exs_internal.h"
#include "rank_poses.inc"
#include "rescore2.inc"
#include "unfold.inc"

namespace exs {

hipError_t launch_dock_f32(const DockArgs& a, int lanes, dim3 grid, dim3 block, size_t lds, hipStream_t st);
hipError_t launch_dock_bf16(const DockArgs& a, int lanes, dim3 grid, dim3 block, size_t lds, hipStream_t st);
hipError_t launch_dock_f16(const DockArgs& a, int lanes, dim3 grid, dim3 block, size_t lds, hipStream_t st);
const void* dock_kernel_fn_f32(int S, int lanes);
const void* dock_kernel_fn_bf16(int S, int lanes);
const void* dock_kernel_fn_f16(int S, int lanes);
hipError_t upload_trig_f32(const float* t32, const double* t64);
hipError_t upload_trig_bf16(const float* t32, const double* t64);
hipError_t upload_trig_f16(const float* t32, const double* t64);
hipError_t launch_gather_probe_f32(const GridDesc* gd, int nb, int64_t blocks, int per_lane,
                                   float half, float walk, uint32_t seed, float* out, hipStream_t st);
hipError_t launch_gather_probe_bf16(const GridDesc* gd, int nb, int64_t blocks, int per_lane,
                                   float half, float walk, uint32_t seed, float* out, hipStream_t st);
hipError_t launch_gather_probe_f16(const GridDesc* gd, int nb, int64_t blocks, int per_lane,
                                   float half, float walk, uint32_t seed, float* out, hipStream_t st);



// FP32 -> 16-bit texel bits, round to nearest even.
__device__ __forceinline__ uint32_t to16(float v, int storage) {
    if (storage == 1) {                       // BF16
        uint32_t u = __builtin_bit_cast(uint32_t, v);
        u += 0x7fffu + ((u >> 16) & 1u);
        return u >> 16;
    }
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v);   // FP16
}

// Expand the FP32 master [C][nz][ny][nx] (x fastest) into the gather layout, one entry per thread:
// entry (x, y, z) holds the texels of the y-z square of the node, V(y, z), V(y+1, z), V(y, z+1),
// V(y+1, z+1) at x, as four floats (storage 0) or as four 16-bit values (1 BF16, 2 FP16, rounded to
// nearest even).  The padding is neither written nor read.
__global__ void expand_grid_kernel(const float* __restrict__ src, void* __restrict__ dst, int nx, int ny,
                                   int nz, int64_t count, int storage, GatherLayout g) {
    const int64_t nxy = (int64_t)nx * ny, chan = g.bytes / (storage == 0 ? 16 : 8);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        int64_t e = i;
        const int64_t x = e % nx;
        e /= nx;
        const int64_t y = e % (ny - 1);
        e /= ny - 1;
        const int64_t z = e % (nz - 1), c = e / (nz - 1);
        const float* q = src + (c * nz + z) * nxy + y * nx + x;
        const float v0 = q[0], v1 = q[nx], v2 = q[nxy], v3 = q[nxy + nx];
        const int64_t at = c * chan + z * g.slice + y * g.row + x;
        if (storage == 0)
            static_cast<float4*>(dst)[at] = make_float4(v0, v1, v2, v3);
        else
            static_cast<uint2*>(dst)[at] = make_uint2(to16(v0, storage) | (to16(v1, storage) << 16),
                                                      to16(v2, storage) | (to16(v3, storage) << 16));
    }
}

// Zero a small int array with a kernel (safe inside a captured graph).
__global__ void zero_ints_kernel(int* p, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_dock(const DockArgs& a, int storage, const DockShape& sh, int n_blocks, hipStream_t st) {
    const dim3 grid(n_blocks), block(sh.waves * kWave);
    const size_t lds = (size_t)sh.lds.total;
    switch (storage) {
        case 0: return launch_dock_f32(a, sh.pair ? 2 * sh.lanes : sh.lanes, grid, block, lds, st);
        case 1: return launch_dock_bf16(a, sh.pair ? 2 * sh.lanes : sh.lanes, grid, block, lds, st);
        case 2: return launch_dock_f16(a, sh.pair ? 2 * sh.lanes : sh.lanes, grid, block, lds, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gather_probe(const GridDesc* gd, int storage, int nb, int64_t blocks, int per_lane,
                               float half, float walk, uint32_t seed, float* out, hipStream_t st) {
    switch (storage) {
        case 0: return launch_gather_probe_f32(gd, nb, blocks, per_lane, half, walk, seed, out, st);
        case 1: return launch_gather_probe_bf16(gd, nb, blocks, per_lane, half, walk, seed, out, st);
        case 2: return launch_gather_probe_f16(gd, nb, blocks, per_lane, half, walk, seed, out, st);
        default: return hipErrorInvalidValue;
    }
}

const void* dock_kernel_fn(int storage, int S, int lanes) {
    switch (storage) {
        case 0: return dock_kernel_fn_f32(S, lanes);
        case 1: return dock_kernel_fn_bf16(S, lanes);
        case 2: return dock_kernel_fn_f16(S, lanes);
        default: return nullptr;
    }
}

hipError_t launch_expand_grid(const float* src, void* dst, int nx, int ny, int nz, int channels,
                              int storage, const GatherLayout& g, hipStream_t st) {
    const int64_t count = (int64_t)nx * (ny - 1) * (nz - 1) * channels;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(expand_grid_kernel, dim3((unsigned)blocks), dim3(256), 0, st, src,
                       dst, nx, ny, nz, count, storage, g);
    return hipGetLastError();
}

hipError_t launch_rank(const DockArgs& a, int n_lig, int64_t n_atoms, const int32_t* order, hipStream_t st) {
    if (n_lig <= 0) return hipSuccess;
    const int waves = rank_waves(n_lig, n_atoms, a.K);
    hipLaunchKernelGGL(rank_kernel, dim3(n_lig), dim3(waves * kWave),
                       (size_t)rank_lds_words(a.K, a.n_max) * sizeof(int), st, a, n_lig, order);
    return hipGetLastError();
}

hipError_t launch_rescore2(const DockArgs& a, int n_lig, const int32_t* order, hipStream_t st) {
    if (n_lig <= 0) return hipSuccess;
    const int waves = rescore2_waves(n_lig, a.rank_keep);
    hipLaunchKernelGGL(rescore2_kernel, dim3(n_lig), dim3(waves * kWave), rescore2_lds_bytes(waves), st, a, n_lig, order);
    return hipGetLastError();
}

hipError_t launch_unfold(const LigInfo* info, float4* ref, double* ref64, const uint32_t* rot_uv,
                         const uint4* rot_mask, int32_t* turns, const int32_t* order, int n_lig, int R,
                         int S, int passes, hipStream_t st) {
    if (n_lig <= 0) return hipSuccess;
    UnfoldArgs a{info, ref, ref64, rot_uv, rot_mask, turns, order, n_lig, R, passes, 0};
    switch (S) {
        case 8: hipLaunchKernelGGL((unfold_kernel<8, 4>), dim3(n_lig), dim3(64), 0, st, a); break;
        case 16: hipLaunchKernelGGL((unfold_kernel<16, 4>), dim3(n_lig), dim3(128), 0, st, a); break;
        case 32:
            if (n_lig >= kUnfoldMany) hipLaunchKernelGGL((unfold_kernel<32, 1>), dim3(n_lig), dim3(64), 0, st, a);
            else hipLaunchKernelGGL((unfold_kernel<32, 4>), dim3(n_lig), dim3(256), 0, st, a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// flag |= 1 for a non-finite texel, |= 2 for a finite texel that rounds to infinity in the
// 16-bit storage (RNE thresholds: FP16 |v| >= 65520, BF16 |v| >= 0x7f7f8000).
__global__ void check_texels_kernel(const float* __restrict__ v, int64_t count, int storage,
                                    int* flag) {
    int bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t a = __builtin_bit_cast(uint32_t, v[i]) & 0x7fffffffu;
        if (a >= 0x7f800000u) bad |= 1;
        else if ((storage == 2 && a >= 0x477ff000u) || (storage == 1 && a >= 0x7f7f8000u)) bad |= 2;
    }
    if (bad) atomicOr(flag, bad);
}

hipError_t launch_check_texels(const float* v, int64_t count, int storage, int* flag, hipStream_t st) {
    int64_t blocks = (count + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(check_texels_kernel, dim3((unsigned)blocks), dim3(256), 0, st, v, count,
                       storage, flag);
    return hipGetLastError();
}

hipError_t launch_zero_ints(int* p, int n, hipStream_t st) {
    hipLaunchKernelGGL(zero_ints_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

__global__ void stage_ints_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int n,
                                  int* __restrict__ zero, int nz, int lig, int n_lig,
                                  int32_t* __restrict__ slot) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = t; i < nz; i += gridDim.x * blockDim.x) zero[i] = 0;   // queues, and a count per split ligand
    for (int i = t; i < n; i += gridDim.x * blockDim.x) dst[i] = src[i];
    for (int j = t; j < n_lig; j += gridDim.x * blockDim.x) slot[src[lig + j]] = j;
}

hipError_t launch_stage_ints(const int32_t* src, int32_t* dst, int n, int* zero, int nz, int lig,
                             int n_lig, int32_t* slot, hipStream_t st) {
    const int blocks = std::max(1, std::min(256, (std::max(n, nz) + 255) / 256));
    hipLaunchKernelGGL(stage_ints_kernel, dim3(blocks), dim3(256), 0, st, src, dst, n, zero, nz, lig,
                       n_lig, slot);
    return hipGetLastError();
}

// Fibonacci-sphere orientations R_k = Rz(phi_k) Ry(beta_k): z_k = 1 - (2k+1)/K, beta_k = acos z_k,
// phi_k = k * golden angle, rows of the product in FP64 and rounded to FP32.  Computed on the
// device so that every launch path (and a path that cannot allocate or copy from the host)
// reads the same table bit for bit.
__host__ __device__ inline int orientation_bands(int K) {
    int b = 1;   // round(sqrt(K) / 7): a wave's patch about as high as it is wide
    while ((2 * b + 1) * (2 * b + 1) * 49 <= 4 * K) ++b;
    return b;
}
__global__ void orientation_table_kernel(int K, float* __restrict__ r32, double* __restrict__ r64,
                                         int32_t* __restrict__ order_k, int32_t* __restrict__ zero, int n_zero) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    for (int t = k; t < n_zero; t += gridDim.x * blockDim.x) zero[t] = 0;
    if (k >= K) return;
    const double golden = 3.14159265358979323846 * (3.0 - sqrt(5.0));
    const double zk = 1.0 - (2.0 * k + 1.0) / (double)K;
    const double beta = acos(zk), phi = (double)k * golden;
    const double cb = cos(beta), sb = sin(beta), cp = cos(phi), sp = sin(phi);
    const double m[9] = {cp * cb, -sp, cp * sb, sp * cb, cp, sp * sb, -sb, 0.0, cb};
    for (int t = 0; t < 9; ++t) {
        if (r64) r64[(size_t)k * 9 + t] = m[t];
        r32[(size_t)k * 9 + t] = (float)m[t];
    }
    // Order of the chunks: bands of consecutive k (consecutive z), by azimuth within a band, so
    // that the orientations of a wave are neighbours and its lookups share lines.  The azimuth in
    // turns as a 32-bit fraction (integer arithmetic: every thread sees the same order).
    const int bands = orientation_bands(K);
    const int b = (int)((int64_t)k * bands / K);
    const int k0 = (int)(((int64_t)b * K + bands - 1) / bands), k1 = (int)(((int64_t)(b + 1) * K + bands - 1) / bands);
    constexpr uint32_t kGoldenTurn = 1640531527u;   // round((3 - sqrt 5) / 2 * 2^32)
    const uint32_t mine = (uint32_t)k * kGoldenTurn;
    int at = k0;
    for (int j = k0; j < k1; ++j) {
        const uint32_t p = (uint32_t)j * kGoldenTurn;
        at += p < mine || (p == mine && j < k) ? 1 : 0;
    }
    order_k[at] = k;
}

hipError_t launch_orientation_table(int K, float* r32, double* r64, int32_t* order_k, int32_t* zero, int n_zero,
                                    hipStream_t st) {
    hipLaunchKernelGGL(orientation_table_kernel, dim3((K + 63) / 64), dim3(64), 0, st, K, r32, r64, order_k, zero,
                       n_zero);
    return hipGetLastError();
}

// Fill the turn tables of the current device: FP32 from the quarter-period literals (the
// same values the unrolled kernels use), checked against FP64 cos / sin rounded to FP32;
// FP64 from the host's cos / sin.
template <int S>
static bool fill_trig(float* t32, double* t64) {
    const int off = trig_offset(S);
    bool ok = true;
    for (int s = 0; s < S; ++s) {
        double a = 2.0 * 3.14159265358979323846 * (double)s / (double)S;
        double c = (4 * s == S || 4 * s == 3 * S) ? 0.0 : (s == 0 ? 1.0 : cos(a));
        double sn = (s == 0 || 2 * s == S) ? 0.0 : (4 * s == S ? 1.0 : (4 * s == 3 * S ? -1.0 : sin(a)));
        t64[off + s] = c;
        t64[off + S + s] = sn;
        t32[off + s] = kcos<S>(s);
        t32[off + S + s] = ksin<S>(s);
        ok = ok && t32[off + s] == (float)c && t32[off + S + s] == (float)sn;
    }
    return ok;
}

hipError_t upload_trig_tables() {
    float t32[kTrigEntries];
    double t64[kTrigEntries];
    if (!fill_trig<8>(t32, t64) || !fill_trig<16>(t32, t64) || !fill_trig<32>(t32, t64))
        return hipErrorInvalidValue;   // a literal of the quarter-period table is wrong
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_trig64), t64, sizeof(double) * kTrigEntries);
    if (e == hipSuccess) e = upload_trig_f32(t32, t64);
    if (e == hipSuccess) e = upload_trig_bf16(t32, t64);
    if (e == hipSuccess) e = upload_trig_f16(t32, t64);
    return e;
}

}  // namespace exs
