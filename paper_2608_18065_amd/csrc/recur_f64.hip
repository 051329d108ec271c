// FP64 instantiations of the matrix-core recurrence: sampling, evaluation and
// local energies.
#include "recur_mm.hpp"

namespace minsr {

bool rec_f64_fits(const minsr_model* m) { return rec_fits<double>(m); }

int launch_rec_f64(minsr_model* m, int mode, const RecCall& c, hipStream_t s) {
  return rec_forward<double>(m, m->wd, mode, c, s);
}

int launch_rec_eloc_f64(minsr_model* m, const minsr_hamiltonian* H, int Ns, const uint8_t* sigma,
                        const void* states, const double* site, int M, hipStream_t s) {
  return rec_eloc<double>(m, m->wd, H, Ns, sigma, states, site, M, s);
}

}  // namespace minsr
