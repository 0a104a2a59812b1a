// Kinds of the middle-row kernel (mid_kernel.h), split over files that compile in parallel.
#include "mid_kernel.h"

namespace fn {

template hipError_t launch_mid_epi<EPI_REGLU>(const PrefillArgs&, int);
template hipError_t launch_mid_epi<EPI_BILINEAR>(const PrefillArgs&, int);

}  // namespace fn
