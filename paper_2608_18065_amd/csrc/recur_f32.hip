// FP32 instantiations of the matrix-core recurrence: sampling and evaluation.
#include "recur_mm.hpp"

namespace minsr {

bool rec_f32_fits(const minsr_model* m) { return rec_fits<float>(m); }

int launch_rec_f32(minsr_model* m, int mode, const RecCall& c, hipStream_t s) {
  return rec_forward<float>(m, m->wf, mode, c, s);
}

int launch_rec_eloc_f32(minsr_model* m, const minsr_hamiltonian* H, int Ns, const uint8_t* sigma,
                        const void* states, const double* site, int M, hipStream_t s) {
  return rec_eloc<float>(m, m->wf, H, Ns, sigma, states, site, M, s);
}

}  // namespace minsr
