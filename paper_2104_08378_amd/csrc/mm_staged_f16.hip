// Products whose second operand passes through registers (mm_staged.hpp), f16 inputs.
#include "mm_staged.hpp"

namespace sp24 {

sp24_status staged_f16(const MmArgs& a, hipStream_t st) { return run_staged<SP24_F16>(a, st); }

} // namespace sp24
