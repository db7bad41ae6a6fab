// D2Q9 passes of eight steps from FORM_TWIN.
#include "lbm_d2q9_pass.h"

namespace lbm {

template hipError_t launch_steps_from<8, FORM_TWIN>(const Geo&, const Rates&, const double*,
                                                  double*, hipStream_t, int);

}  // namespace lbm
