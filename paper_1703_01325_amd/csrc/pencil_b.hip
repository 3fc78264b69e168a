// Pencil sweep launchers for one block size, BILU_B (set by the build, 1..8).
#include <hip/hip_runtime.h>

#include "bilu.h"
#include "launch.h"
#include "pencil_kernels.h"

#ifndef BILU_B
#error "BILU_B (the block size of this translation unit) must be defined"
#endif

namespace bilu {
namespace launch {

namespace {

template <int B, typename T, int K, int CB>
void pencil_k(bool fuse, int blocks, size_t lds, hipStream_t s, const dev::PencilArgs& a)
{
    if (fuse) hipLaunchKernelGGL((dev::k_sweep_pencil<B, T, K, CB, true>), dim3(blocks), dim3(256), lds, s, a);
    else hipLaunchKernelGGL((dev::k_sweep_pencil<B, T, K, CB, false>), dim3(blocks), dim3(256), lds, s, a);
}

template <int B, typename T, int CB>
bool pencil_t(int width, bool fuse, int blocks, size_t lds, hipStream_t s, const dev::PencilArgs& a)
{
    switch (width) {
    case 3: pencil_k<B, T, 3, CB>(fuse, blocks, lds, s, a); return true;
    case 6: pencil_k<B, T, 6, CB>(fuse, blocks, lds, s, a); return true;
    case 11:
        if constexpr (CB == 1 || kPencilPairWidth >= 11) {
            pencil_k<B, T, 11, CB>(fuse, blocks, lds, s, a);
            return true;
        }
        return false;
    case 21:
        if constexpr (pencil_width(B, 21) == 21 && (CB == 1 || kPencilPairWidth >= 21)) {
            pencil_k<B, T, 21, CB>(fuse, blocks, lds, s, a);
            return true;
        }
        return false;
    }
    return false;
}

template <int B, typename T>
bool pencil_c(int width, int cb, bool fuse, int blocks, size_t lds, hipStream_t s, const dev::PencilArgs& a)
{
    switch (cb) {
    case 1: return pencil_t<B, T, 1>(width, fuse, blocks, lds, s, a);
    case 2: return pencil_t<B, T, 2>(width, fuse, blocks, lds, s, a);
    }
    return false;
}

}  // namespace

template <int B>
bool pencil(int width, int cb, int prec, bool fuse, int blocks, size_t lds, hipStream_t s, const dev::PencilArgs& a)
{
    if (prec == BILU_FACTORS_FP32) return pencil_c<B, float>(width, cb, fuse, blocks, lds, s, a);
    return pencil_c<B, double>(width, cb, fuse, blocks, lds, s, a);
}

template bool pencil<BILU_B>(int, int, int, bool, int, size_t, hipStream_t, const dev::PencilArgs&);

}  // namespace launch
}  // namespace bilu
