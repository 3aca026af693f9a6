// Direction-y (columns) kernel schedules, FP32, n = 512..8192: REG(n, radix,
// lines per workgroup, spinor components per thread; D: default from so many lines,
// flat, with a layer, curved; O: carries the observable kernel).
#include "stage_kernels.hpp"
#include "registry.hpp"
#define DIRAC_T float
#define DIRAC_PREC 1
#define DIRAC_COLS true
#define DIRAC_DIR 1
REGOD(512, 8, 4, 2, 2048, 2048, 2048)
REG(512, 8, 4, 1)
REGD(512, 8, 2, 1, 0, 0, 0)
REG(512, 8, 8, 2)
REG(512, 16, 8, 2)
REG(512, 4, 2, 1)
REGOD(1024, 8, 4, 1, 0, 0, 0)
REG(1024, 8, 4, 2)
REGD(1024, 16, 4, 2, 2048, 2048, 2048)
REGD(2048, 16, 2, 2, 512, 512, 512)
REGOD(2048, 8, 2, 2, 0, 0, 0)
REG(2048, 16, 4, 1)
REGD(2048, 16, 4, 2, -1, 2048, 2048)
REGOD(4096, 16, 2, 2, 0, 0, 0)
REG(4096, 16, 2, 1)
REG(4096, 8, 2, 2)
// 8192 points: two lines per workgroup (1024 threads, one workgroup per compute unit) pay
// for their wider row pieces only on many lines.  us per step, one line / two: 64 lines flat
// 37.3 / 54.6, layer 45.7 / 67.1, curved 47.8 / 93.1; 256 curved 86.9 / 118; 512 128 / 132
// (layer), 198 / 181 (curved); 2048 393 / 429, 603 / 653, 982 / 798; 4096 932 / 887, 1195 / 1167,
// 1464 / 1419.
REGOD(8192, 16, 1, 2, 0, 0, 0)
REG(8192, 16, 1, 1)
REGD(8192, 16, 2, 2, 4096, 4096, 512)
