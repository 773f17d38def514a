// Time-line kernels instantiated for double2 spinor storage (see k_line_impl.h).
#define TP_LINE_S double2
#define TP_LINE_SUFFIX f64
#include "k_line_impl.h"

void line_canon_f64(tp_op op, int mode, const double2* src, double2* dst) {
  switch (mode) {
    case LM_CL: line_canon_t<LM_CL>(op, src, dst); break;
    case LM_CR: line_canon_t<LM_CR>(op, src, dst); break;
    case LM_TINV: line_canon_t<LM_TINV>(op, src, dst); break;
    case LM_TDINV: line_canon_t<LM_TDINV>(op, src, dst); break;
    default: TP_THROW(TP_EINVAL, "line mode");
  }
}
