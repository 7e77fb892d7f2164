#include "vmult.hpp"

namespace mfmg {

void vmult_f32(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  vmult_s<float>(c, nv, dst, src, f, s);
}

}  // namespace mfmg
