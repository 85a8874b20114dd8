// Instantiates the dock kernel for FP32 texels.
#include "dock_kernels.inc"
#include "gather_probe.inc"

namespace exs {

hipError_t launch_dock_f32(const DockArgs& a, int lanes, dim3 grid, dim3 block, size_t lds,
                           hipStream_t st) {
#define EXS_LAUNCH(SS, GG) \
    if (a.S == SS && lanes == GG) { \
        hipLaunchKernelGGL((dock_kernel<SS, (GG < SS ? GG : SS), TexF32, (GG > SS)>), grid, block, lds, st, a); \
        return hipGetLastError(); \
    }
    EXS_LAUNCH(8, 4) EXS_LAUNCH(8, 8) EXS_LAUNCH(16, 4) EXS_LAUNCH(16, 8) EXS_LAUNCH(16, 16)
    EXS_LAUNCH(32, 4) EXS_LAUNCH(32, 8) EXS_LAUNCH(32, 16) EXS_LAUNCH(32, 32)
    EXS_LAUNCH(8, 16) EXS_LAUNCH(16, 32) EXS_LAUNCH(32, 64)
#undef EXS_LAUNCH
    return hipErrorInvalidValue;
}

const void* dock_kernel_fn_f32(int S, int lanes) {
#define EXS_FN(SS, GG) \
    if (S == SS && lanes == GG) return reinterpret_cast<const void*>(&dock_kernel<SS, (GG < SS ? GG : SS), TexF32, (GG > SS)>);
    EXS_FN(8, 4) EXS_FN(8, 8) EXS_FN(16, 4) EXS_FN(16, 8) EXS_FN(16, 16)
    EXS_FN(32, 4) EXS_FN(32, 8) EXS_FN(32, 16) EXS_FN(32, 32)
    EXS_FN(8, 16) EXS_FN(16, 32) EXS_FN(32, 64)
#undef EXS_FN
    return nullptr;
}

hipError_t launch_gather_probe_f32(const GridDesc* gd, int nb, int64_t blocks, int per_lane,
                                float half, float walk, uint32_t seed, float* out, hipStream_t st) {
    const dim3 grid((unsigned)blocks), block(256);
    switch (nb) {
        case 8: hipLaunchKernelGGL((gather_probe_kernel<TexF32, 8>), grid, block, 0, st, gd, per_lane, half, walk, seed, out); break;
        case 16: hipLaunchKernelGGL((gather_probe_kernel<TexF32, 16>), grid, block, 0, st, gd, per_lane, half, walk, seed, out); break;
        case 32: hipLaunchKernelGGL((gather_probe_kernel<TexF32, 32>), grid, block, 0, st, gd, per_lane, half, walk, seed, out); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t upload_trig_f32(const float* t32, const double* t64) {
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_trig32), t32, sizeof(float) * kTrigEntries);
    if (e != hipSuccess) return e;
    return hipMemcpyToSymbol(HIP_SYMBOL(c_trig64), t64, sizeof(double) * kTrigEntries);
}

}  // namespace exs
