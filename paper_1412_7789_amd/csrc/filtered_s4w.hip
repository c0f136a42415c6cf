// Filtered-scan kernels of stride 4 with the window table (see filtered.hpp).
#include "filtered.hpp"

namespace pfac {

dev::FilteredFn pick_filtered_s4w(int kind, int segs) { return dev::pick_filter<3, 4, true>(kind, segs); }

}  // namespace pfac
