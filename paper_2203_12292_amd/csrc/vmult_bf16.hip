#include "vmult.hpp"

namespace mfmg {

void vmult_bf16(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  vmult_s<bf16>(c, nv, dst, src, f, s);
}

}  // namespace mfmg
