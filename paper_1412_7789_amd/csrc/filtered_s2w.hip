// Filtered-scan kernels of stride 2 with the window table (see filtered.hpp).
#include "filtered.hpp"

namespace pfac {

dev::FilteredFn pick_filtered_s2w(int kind, int segs) { return dev::pick_filter<3, 2, true>(kind, segs); }

}  // namespace pfac
