// Products whose second operand passes through registers (mm_staged.hpp), bf16 inputs.
#include "mm_staged.hpp"

namespace sp24 {

sp24_status staged_bf16(const MmArgs& a, hipStream_t st) { return run_staged<SP24_BF16>(a, st); }

} // namespace sp24
