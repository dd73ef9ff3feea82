// The marching sweep on bfloat16 storage (a unit of its own: its kernels, one per
// step count, take as long to compile as all others of the storage type).
#include "lbm_march.h"
#include "lbm_offset.h"

namespace lbm {

template <>
hipError_t launch_march<bf16>(const SweepArgs<bf16> &a, const MarchPlan &p, bool check,
                             hipStream_t s) {
    return sweep::launch_march<BF16Cell>(a, p, check, s);
}

}  // namespace lbm
