// Which products the kernels of mm_staged.hpp take, and the per-type entry points (a translation unit each).
#include "common.hpp"
#include "launch.hpp"

namespace sp24 {

sp24_status staged_f16(const MmArgs& a, hipStream_t st);
sp24_status staged_bf16(const MmArgs& a, hipStream_t st);
sp24_status staged_i8(const MmArgs& a, hipStream_t st);
sp24_status staged_f8(const MmArgs& a, hipStream_t st);

sp24_status launch_mm_staged(const MmArgs& a, hipStream_t st, bool* handled)
{
    *handled = false;
    if (!a.sparse || a.k_slices > 1) return SP24_OK;
    if (a.M > ((int64_t)1 << 30) || a.N > ((int64_t)1 << 30) || ((a.M + 31) / 32) * ((a.N + 127) / 128) >= ((int64_t)1 << 30) ||
        a.K > ((int64_t)1 << 30))
        return SP24_OK;
    *handled = true;
    if (a.in == SP24_I8) return staged_i8(a, st);
    if (a.in == SP24_F8) return staged_f8(a, st);
    if (a.in == SP24_F16) return staged_f16(a, st);
    return staged_bf16(a, st);
}

} // namespace sp24
