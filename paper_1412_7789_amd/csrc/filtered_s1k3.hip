// Filtered-scan kernels of stride 1 and prefix length 3 (see filtered.hpp).
#include "filtered.hpp"

namespace pfac {

dev::FilteredFn pick_filtered_s1k3(int kind, int segs) { return dev::pick_filter<3, 1, false>(kind, segs); }

}  // namespace pfac
