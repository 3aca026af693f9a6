// Direction-x (rows) kernel schedules, FP32, n = 16..256: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T float
#define DIRAC_PREC 1
#define DIRAC_COLS false
#define DIRAC_DIR 0
REGO(16, 4, 16, 2)
REGD(16, 4, 8, 1, 0, 0, 0)
REG(16, 16, 64, 2)
REGO(32, 4, 8, 2)
REGD(32, 4, 4, 1, 0, 0, 0)
REG(32, 4, 8, 1)
REGO(64, 4, 4, 2)
REGD(64, 4, 2, 1, 0, 0, 0)
REG(64, 8, 8, 2)
REGO(128, 4, 2, 2)
REGD(128, 4, 1, 1, 0, 0, 0)
REG(128, 8, 4, 2)
REG(128, 8, 2, 1)
REGOD(256, 4, 1, 1, 0, 0, 0)
REG(256, 8, 2, 2)
REG(256, 8, 1, 1)
REG(256, 16, 4, 2)
