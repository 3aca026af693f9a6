// Direction-x (rows) kernel schedules, FP64, n = 512..4096: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T double
#define DIRAC_PREC 0
#define DIRAC_COLS false
#define DIRAC_DIR 0
REGO(512, 4, 1, 2)
REGD(512, 8, 2, 1, 1024, 1024, 1024)
REGD(512, 4, 1, 1, -1, 0, 0)
REG(512, 8, 1, 2)
REGD(512, 8, 1, 1, 0, -1, -1)
REGOD(1024, 8, 1, 1, 0, 0, 0)
REGD(1024, 8, 1, 2, -1, -1, 1024)
REG(1024, 4, 1, 1)
REG(1024, 8, 2, 2)
REGOD(2048, 8, 1, 2, -1, 512, 0)
REGD(2048, 8, 1, 1, 0, 0, -1)
REG(2048, 4, 1, 1)
REG(2048, 16, 2, 2)
REGOD(4096, 8, 1, 2, -1, -1, 0)
REGD(4096, 8, 1, 1, 0, 0, -1)
REGD(4096, 16, 1, 2, 512, -1, -1)
