// Products whose second operand passes through registers (mm_staged.hpp), i8 inputs.
#include "mm_staged.hpp"

namespace sp24 {

sp24_status staged_i8(const MmArgs& a, hipStream_t st) { return run_staged<SP24_I8>(a, st); }

} // namespace sp24
