// Direction-y (columns) kernel schedules, FP64, n = 16..256: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T double
#define DIRAC_PREC 0
#define DIRAC_COLS true
#define DIRAC_DIR 1
REGO(16, 4, 16, 2)
REGD(16, 4, 8, 1, 0, 0, 0)
REG(16, 4, 16, 1)
REGO(32, 4, 8, 2)
REGD(32, 4, 4, 1, 0, 0, 0)
REG(32, 4, 8, 1)
REGO(64, 4, 8, 2)
REGD(64, 4, 4, 1, 1024, 1024, 1024)
REG(64, 8, 8, 2)
REGD(64, 4, 2, 1, 0, 0, 0)
REGO(128, 4, 4, 1)
REG(128, 4, 4, 2)
REG(128, 8, 4, 2)
REG(128, 8, 4, 1)
REGD(128, 4, 1, 1, 0, 0, 0)
REGD(128, 4, 2, 1, 1024, 1024, 1024)
REGO(256, 4, 4, 1)
REG(256, 8, 4, 2)
REG(256, 8, 4, 1)
REG(256, 8, 8, 2)
REGD(256, 4, 2, 1, 512, 512, 512)
REGD(256, 4, 1, 1, 0, 0, 0)
