// FP64 instantiations of the matrix-core Jacobian: chains and 2D models.
#include "jac_mm.hpp"

namespace minsr {

bool jac_mm_f64_fits(const minsr_model* m) {
  if (!rec_f64_fits(m)) return false;
  const int d = m->dim, Lx = m->d.Lx;
  return m->H == 8    ? jm_rev_smem<double, 8, 1>(d, Lx) <= MM_LDS
         : m->H == 16 ? jm_rev_smem<double, 16, 1>(d, Lx) <= MM_LDS
         : m->H == 32 ? jm_rev_smem<double, 32, 1>(d, Lx) <= MM_LDS
                      : m->H == 64 && jm_rev_smem<double, 64, 1>(d, Lx) <= MM_LDS;
}

int launch_jac_mm_f64(minsr_model* m, int Ns, const uint8_t* sigma, const void* states, void* O,
                      bool have_tape, hipStream_t s) {
  auto run = [&](const JmArgs<double>& a) {
    const bool two = m->dim == 2;
    switch (m->H) {
      case 8: return two ? jm_chunk<double, 8, 2, 1>(a, s) : jm_chunk<double, 8, 1, 1>(a, s);
      case 16: return two ? jm_chunk<double, 16, 2, 1>(a, s) : jm_chunk<double, 16, 1, 1>(a, s);
      case 32: return two ? jm_chunk<double, 32, 2, 1>(a, s) : jm_chunk<double, 32, 1, 1>(a, s);
      case 64: return two ? jm_chunk<double, 64, 2, 1>(a, s) : jm_chunk<double, 64, 1, 1>(a, s);
    }
    return fail(MINSR_E_UNSUPPORTED, "matrix-core Jacobian: hidden width");
  };
  return jm_run<double>(m, jm_args<double>(m, m->wd, Ns, sigma, states, O), have_tape,
                        launch_rec_f64, run, s);
}

size_t jac_mm_site_elems(const minsr_model* m) { return jm_site_elems(m->dim, m->H, m->cplx); }

}  // namespace minsr
