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
  RecArgs<double> a = rec_args<double>(m, m->wd, Ns);
  a.sigma_in = sigma; a.states_in = (const double*)states; a.site_in = site;
  a.bonds = m->bonds; a.n_nn = m->n_nn; a.ham_kind = H->kind; a.M = M;
  a.hx = H->h; a.J1 = H->J; a.J2 = H->J2; a.contrib = m->contrib;
  a.nchunks = (Ns + 15) / 16;
  unsigned grid = (unsigned)(a.nchunks * M);
  if (H->kind == MINSR_HAM_J1J2) {
    const int rc = launch_eloc_lists(m, Ns, sigma, M, s);
    if (rc) return rc;
    a.list = m->elist; a.count = m->ecount; a.items = m->eitems;
    grid = 2u * (unsigned)((Ns + 31) / 32) * (unsigned)M;   // at most; the rest leave at once
  }
  return rec_dispatch<double, RM_ELOC>(m, a, grid, s);
}

}  // namespace minsr
