// Direction-y (columns) kernel schedules, FP64, n = 512..4096: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T double
#define DIRAC_PREC 0
#define DIRAC_COLS true
#define DIRAC_DIR 1
REGOD(512, 8, 2, 1, 256, 256, 256)
REG(512, 4, 2, 2)
REG(512, 8, 2, 2)
REG(512, 8, 4, 2)
REG(512, 8, 4, 1)
REGD(512, 8, 1, 1, 0, 0, 0)
REGOD(1024, 8, 4, 2, -1, 1024, -1)
REGD(1024, 8, 4, 1, 1024, -1, -1)
REGD(1024, 8, 2, 2, 2048, 2048, 1024)
REGD(1024, 8, 2, 1, 0, 0, 0)
REGO(2048, 8, 2, 2)
REGD(2048, 8, 1, 2, 0, 0, 0)
REGD(2048, 8, 2, 1, 256, -1, -1)
REGD(2048, 16, 2, 2, 1024, 512, 512)
REGO(4096, 8, 1, 2)
REGD(4096, 8, 1, 1, 0, 0, 0)
REG(4096, 8, 2, 2)
REGD(4096, 16, 2, 2, 512, 512, 512)
