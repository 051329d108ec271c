// FP32 instantiations of the matrix-core Jacobian: 2D models.  The parts of
// the reverse product are k_jacobian's built-in choice for the width.
#include "jac_mm.hpp"

namespace minsr {

bool jac_mm_f32_fits(const minsr_model* m) {
  if (m->dim != 2 || !rec_f32_fits(m)) return false;
  const int Lx = m->d.Lx;
  return m->H == 32   ? jm_rev_smem<float, 32, 1>(2, Lx) <= MM_LDS
         : m->H == 64 ? jm_rev_smem<float, 64, 4>(2, Lx) <= MM_LDS
                      : m->H == 128 && jm_rev_smem<float, 128, 2>(2, Lx) <= MM_LDS;
}

int launch_jac_mm_f32(minsr_model* m, int Ns, const uint8_t* sigma, const void* states, void* O,
                      bool have_tape, hipStream_t s) {
  auto run = [&](const JmArgs<float>& a) {
    switch (m->H) {
      case 32: return jm_chunk<float, 32, 2, 1>(a, s);
      case 64: return jm_chunk<float, 64, 2, 4>(a, s);
      case 128: return jm_chunk<float, 128, 2, 2>(a, s);
    }
    return fail(MINSR_E_UNSUPPORTED, "matrix-core Jacobian: hidden width");
  };
  return jm_run<float>(m, jm_args<float>(m, m->wf, Ns, sigma, states, O), have_tape,
                       launch_rec_f32, run, s);
}

}  // namespace minsr
