// Kinds of the middle-row kernel (mid_kernel.h), split over files that compile in parallel.
#include "mid_kernel.h"

namespace fn {

template hipError_t launch_mid_epi<EPI_LN>(const PrefillArgs&, int);
template hipError_t launch_mid_epi<EPI_NONE>(const PrefillArgs&, int);

}  // namespace fn
