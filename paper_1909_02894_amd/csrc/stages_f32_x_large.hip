// Direction-x (rows) kernel schedules, FP32, n = 512..8192: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T float
#define DIRAC_PREC 1
#define DIRAC_COLS false
#define DIRAC_DIR 0
REGOD(512, 4, 1, 1, -1, 0, 0)
REGD(512, 8, 1, 2, -1, 4096, 4096)
REGD(512, 8, 1, 1, 0, -1, -1)
REGD(512, 8, 2, 2, 4096, -1, -1)
REGOD(1024, 8, 2, 2, 4096, -1, -1)
REG(1024, 8, 1, 1)
REG(1024, 8, 1, 2)
REG(1024, 16, 1, 2)
REGD(1024, 4, 1, 1, 0, 0, 0)
REGOD(2048, 8, 1, 2, 1024, 1024, 1024)
REG(2048, 16, 1, 2)
REGD(2048, 8, 1, 1, 0, 0, 0)
REG(2048, 16, 1, 1)
REG(2048, 16, 2, 2)
REGOD(4096, 16, 1, 2, 512, 512, 512)
REGD(4096, 8, 1, 2, 0, 0, 0)
REG(4096, 16, 2, 1)
REGOD(8192, 16, 1, 2, 0, 0, 0)
REG(8192, 16, 1, 1)
