// bis_f64.hip -- instantiations of the second-order directional kernels (double).
#include <hip/hip_runtime.h>

#include "bis_kernels.hpp"

namespace dirac {

#define BISL(N, DIR, L, CPT, FROM)                                                                      \
    BisEntry{0, N, DIR, L, bis_threads(N, L, CPT), FROM,                                               \
             {reinterpret_cast<const void*>(&bis_stage_kernel<double, N, L, CPT, DIR == 1, 1>),                \
              reinterpret_cast<const void*>(&bis_stage_kernel<double, N, L, CPT, DIR == 1, 2>)}}
#define BIS(N, DIR) BISL(N, DIR, bis_lines(N), bis_cpt(N), 0)

const BisEntry* bis_entries_f64(int* count) {
    static const BisEntry e[] = {BIS(16, 0),  BIS(32, 0),  BIS(64, 0),  BIS(128, 0), BIS(256, 0),  BIS(512, 0),
                                 BIS(1024, 0), BIS(2048, 0), BIS(16, 1), BIS(32, 1),  BIS(64, 1),   BIS(128, 1),
                                 BIS(256, 1), BISL(512, 1, 2, 1, 0), BISL(512, 1, 2, 2, 1024), BIS(1024, 1),
                                 BIS(2048, 1)};
    *count = (int)(sizeof e / sizeof e[0]);
    return e;
}

}  // namespace dirac
