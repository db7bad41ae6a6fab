// D2Q9 passes of four steps.
#include "lbm_d2q9_pass.h"

namespace lbm {

template hipError_t launch_steps_t<4>(const Geo&, const Rates&, const double*, double*,
                                      hipStream_t, int, int);

}  // namespace lbm
