// Register-engine ring kernels in FP32 (one translation unit per precision, compiled in parallel).
#include "akra_ring16.h"

namespace akra {
template void ring16_launch<float, 0>(Plan &, const RingSet &, const RingArgs &, int, bool);
template void ring16_launch<float, 1>(Plan &, const RingSet &, const RingArgs &, int, bool);
template void ring16_launch<float, 2>(Plan &, const RingSet &, const RingArgs &, int, bool);
void launch_bhat_reorder_f32(Plan &P, int logm, const int64_t *src_ofs, const int64_t *dst_ofs, int n)
{
    bhat_reorder<float>(P, logm, src_ofs, dst_ofs, n);
}
}  // namespace akra
