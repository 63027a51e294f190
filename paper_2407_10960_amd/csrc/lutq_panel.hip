// Instantiates panel_kernel for one (bit width, dtype) pair; group size, blocks of 32 activation rows and panel height
// are dispatched at run time.
#include "lutq_launch.hpp"

#ifndef LUTQ_INST_BITS
#error "compile with -DLUTQ_INST_BITS=2|3|4 -DLUTQ_INST_DT=F16|BF16"
#endif

#define LUTQ_CAT3(a, b, c) a##b##_##c
#define LUTQ_NAME(prefix, b, dt) LUTQ_CAT3(prefix, b, dt)

namespace lutq {

namespace {

template <int GROUP, int MB, int RP, bool SCH>
hipError_t launch_panel_sch(const PanelParams& p, hipStream_t stream) {
    auto kernel = panel_kernel<LUTQ_INST_BITS, GROUP, MB, LUTQ_INST_DT, RP, SCH>;
    constexpr int lds_bytes = panel_lds_bytes<LUTQ_INST_BITS>(MB);
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kernel, dim3((unsigned)p.G), dim3(64 * kPanelWaves), lds_bytes, stream, p);
    return hipGetLastError();
}

template <int GROUP, int MB, int RP>
hipError_t launch_panel_one(const PanelParams& p, hipStream_t stream) {
    if constexpr (!panel_instance_exists(LUTQ_INST_BITS, MB, RP)) return hipErrorInvalidValue;
    else return p.SG2 % 16 == 0 ? launch_panel_sch<GROUP, MB, RP, true>(p, stream) : launch_panel_sch<GROUP, MB, RP, false>(p, stream);
}

template <int GROUP>
hipError_t launch_panel_group(int mb, int rp, const PanelParams& p, hipStream_t stream) {
    if (rp == 1) {
        if (mb == 1) return launch_panel_one<GROUP, 1, 1>(p, stream);
        if (mb == 2) return launch_panel_one<GROUP, 2, 1>(p, stream);
        if (mb == 3) return launch_panel_one<GROUP, 3, 1>(p, stream);
        if (mb == 4) return launch_panel_one<GROUP, 4, 1>(p, stream);
    } else if (rp == 2) {
        if (mb == 1) return launch_panel_one<GROUP, 1, 2>(p, stream);
        if (mb == 2) return launch_panel_one<GROUP, 2, 2>(p, stream);
        if (mb == 3) return launch_panel_one<GROUP, 3, 2>(p, stream);
        if (mb == 4) return launch_panel_one<GROUP, 4, 2>(p, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t LUTQ_NAME(launch_panel_b, LUTQ_INST_BITS, LUTQ_INST_DT)(int group, int mb, int rp, const PanelParams& p,
                                                                   hipStream_t stream) {
    switch (group) {
        case 32: return launch_panel_group<32>(mb, rp, p, stream);
        case 64: return launch_panel_group<64>(mb, rp, p, stream);
        case 128: return launch_panel_group<128>(mb, rp, p, stream);
        case 256: return launch_panel_group<256>(mb, rp, p, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace lutq
