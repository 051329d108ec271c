// FP32 instantiations of the matrix-core recurrence: sampling and evaluation.
#include "recur_mm.hpp"

namespace minsr {

bool rec_f32_fits(const minsr_model* m) { return rec_fits<float>(m); }

int launch_rec_f32(minsr_model* m, int mode, const RecCall& c, hipStream_t s) {
  return rec_forward<float>(m, m->wf, mode, c, s);
}

}  // namespace minsr
