// amsim_tab.hip -- the table kernels of one operation, AMSIM_TAB_OP (0 GEMM, 1 forward,
// 2 backward data, 3 backward weight), on rows of 128 entries (AMSIM_TAB_WIDE = 0) or of 256 and more
// (1), with their launch and attribute set-up.  The build sets both and compiles this file once for
// each, so that the eight instantiation sets build in parallel.
#include "amsim_tab.h"

#ifndef AMSIM_TAB_OP
#error "AMSIM_TAB_OP must name the operation (0..3)"
#endif
#ifndef AMSIM_TAB_WIDE
#error "AMSIM_TAB_WIDE must choose the row lengths (0, 1)"
#endif

namespace amsim_detail __attribute__((visibility("hidden"))) {

namespace {

// Raises the kernel's dynamic LDS limit, and checks that it has no static LDS: the bf16 path
// addresses its slabs as LDS addresses starting at 0.  Keeps the first error in err.
template <typename K>
void allow_lds(K kernel, size_t bytes, hipError_t &err)
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    hipFuncAttributes fa{};
    if (e == hipSuccess) e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kernel));
    if (e == hipSuccess && fa.sharedSizeBytes != 0) e = hipErrorInvalidKernelFile;
    if (err == hipSuccess) err = e;
}

template <typename F>
void dispatch_tab_tile(const Tile &t, int rl, F &&f)
{
#define X(TM, TN, WR, NW, RL)                                                             \
    if constexpr ((RL > 7) == (AMSIM_TAB_WIDE != 0)) {                                    \
        if (t.tm == TM && t.tn == TN && t.wr == WR && t.nw == NW && rl == RL) {           \
            f(std::integral_constant<int, TM>{}, std::integral_constant<int, TN>{},       \
              std::integral_constant<int, WR>{}, std::integral_constant<int, NW>{},       \
              std::integral_constant<int, RL>{});                                         \
            return;                                                                       \
        }                                                                                 \
    }
    AMSIM_FOR_TAB_TILES(X)
#undef X
}

}  // namespace

template <int OP, int WIDE>
hipError_t tab_attributes_of()
{
    hipError_t err = hipSuccess;
#define X(TM, TN, WR, NW, RL)                                                                              \
    if constexpr ((RL > 7) == (WIDE != 0))                                                                  \
        allow_lds(tab_kernel<OP, TM, TN, WR, NW, RL, kTabApprox>, tab_lds_bytes(TN, WR, NW, RL), err);      \
    if constexpr (RL == 7 && WIDE == 0) {                                                                   \
        allow_lds(tab_kernel<OP, TM, TN, WR, NW, 7, kTabNative>, tab_native_lds_bytes(TN, WR, NW), err);    \
        allow_lds(tab_kernel<OP, TM, TN, WR, NW, 7, kTabApproxSelf>, tab_lds_bytes(TN, WR, NW, 7), err);    \
    }
    AMSIM_FOR_TAB_TILES(X)
#undef X
    if constexpr (WIDE != 0) {
        allow_lds(own_kernel<OP, 8, kOwnWide>, own_lds_bytes(8, kOwnWide), err);
        allow_lds(own_kernel<OP, 4, kOwnWide>, own_lds_bytes(4, kOwnWide), err);
    } else {
        allow_lds(own_kernel<OP, 8, kOwnTab>, own_lds_bytes(8, kOwnTab), err);
        allow_lds(own_kernel<OP, 4, kOwnTab>, own_lds_bytes(4, kOwnTab), err);
        allow_lds(own_kernel<OP, 8, kOwnNative>, own_lds_bytes(8, kOwnNative), err);
        allow_lds(own_kernel<OP, 4, kOwnNative>, own_lds_bytes(4, kOwnNative), err);
    }
    return err;
}

template <int OP, int WIDE>
hipError_t own_launch_of(int nw, int cls, unsigned blocks, const TabArgs &a, const OwnPrep &p, hipStream_t st)
{
    bool launched = false;
    auto run = [&](auto nw_c, auto cls_c) {
        constexpr int NW = decltype(nw_c)::value, CLS = decltype(cls_c)::value;
        if constexpr ((CLS == kOwnWide) == (WIDE != 0)) {
            if (nw == NW && cls == CLS) {
                hipLaunchKernelGGL((own_kernel<OP, NW, CLS>), dim3(blocks), dim3(64 * NW), own_lds_bytes(NW, CLS), st, a, p);
                launched = true;
            }
        }
    };
    auto both = [&](auto cls_c) {
        run(std::integral_constant<int, 8>{}, cls_c);
        run(std::integral_constant<int, 4>{}, cls_c);
    };
    both(std::integral_constant<int, kOwnTab>{});
    both(std::integral_constant<int, kOwnWide>{});
    both(std::integral_constant<int, kOwnNative>{});
    return launched ? hipGetLastError() : hipErrorInvalidConfiguration;
}

template <int OP, int WIDE>
hipError_t tab_launch_of(const Tile &t, int rl, int var, const TabArgs &a, dim3 grid, hipStream_t st)
{
    bool launched = false;
    auto run = [&](auto tm, auto tn, auto wr, auto nw, auto rl_c) {
        constexpr int TM = decltype(tm)::value, TN = decltype(tn)::value, WR = decltype(wr)::value;
        constexpr int NW = decltype(nw)::value, RL = decltype(rl_c)::value;
        if (var == kTabNative) {
            if constexpr (RL == 7) {
                hipLaunchKernelGGL((tab_kernel<OP, TM, TN, WR, NW, 7, kTabNative>), grid, dim3(64 * NW),
                                   tab_native_lds_bytes(TN, WR, NW), st, a);
                launched = true;
            }
            return;
        }
        if (var == kTabApproxSelf) {  // rows of 128 entries only
            if constexpr (RL == 7) {
                hipLaunchKernelGGL((tab_kernel<OP, TM, TN, WR, NW, 7, kTabApproxSelf>), grid, dim3(64 * NW),
                                   tab_lds_bytes(TN, WR, NW, 7), st, a);
                launched = true;
            }
            return;
        }
        hipLaunchKernelGGL((tab_kernel<OP, TM, TN, WR, NW, RL, kTabApprox>), grid, dim3(64 * NW),
                           tab_lds_bytes(TN, WR, NW, RL), st, a);
        launched = true;
    };
    dispatch_tab_tile(t, rl, run);
    return launched ? hipGetLastError() : hipErrorInvalidConfiguration;
}

template hipError_t tab_attributes_of<AMSIM_TAB_OP, AMSIM_TAB_WIDE>();
template hipError_t tab_launch_of<AMSIM_TAB_OP, AMSIM_TAB_WIDE>(const Tile &, int, int, const TabArgs &, dim3, hipStream_t);
template hipError_t own_launch_of<AMSIM_TAB_OP, AMSIM_TAB_WIDE>(int, int, unsigned, const TabArgs &, const OwnPrep &,
                                                                hipStream_t);

}  // namespace amsim_detail
