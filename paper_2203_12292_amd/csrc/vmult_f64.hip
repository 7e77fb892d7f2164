#include "vmult.hpp"

namespace mfmg {

void vmult_f64(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  vmult_s<double>(c, nv, dst, src, f, s);
}

}  // namespace mfmg
