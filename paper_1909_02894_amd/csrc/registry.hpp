// registry.hpp -- compiled kernel variants of the direction and observable
// kernels, registered per (precision, n, direction, schedule) by the
// translation units that instantiate them.
#pragma once
#include <vector>

namespace dirac {

struct KernelEntry {
    int prec;       // 0 = FP64, 1 = FP32
    int n;          // transform length
    int dir;        // 0 = x (rows), 1 = y (columns)
    int radix;      // values per thread per component
    int lines;      // lines per workgroup
    int cpt;        // spinor components per thread (1 or 2)
    int nthreads;   // workgroup size
    const void* stage_fn[3];   // by mode: 0 flat, 1 flat + layer, 2 curved
    const void* stream_fn[3];  // by mode: the kernel of grids with stream_from_tiles(mode) tiles, or null
    const void* obs_fn;
    int from_lines[3];         // by mode: default schedule from this many lines (negative: never)
};

std::vector<KernelEntry>& kernel_registry();

struct Registrar {
    Registrar(const KernelEntry& e) { kernel_registry().push_back(e); }
};

}  // namespace dirac

// REG(N, R, L, CPT) inside a translation unit that defines DIRAC_T (double /
// float), DIRAC_PREC (0/1), DIRAC_COLS (false/true), DIRAC_DIR (0/1).
#define DIRAC_CAT2(a, b) a##b
#define DIRAC_CAT(a, b) DIRAC_CAT2(a, b)
#define DIRAC_STREAM(N, R, L, MODE, CPT) ::dirac::stream_fn<DIRAC_T, N, R, L, DIRAC_COLS, MODE, CPT>()
#define DIRAC_REG_IMPL(N, R, L, CPT, OBS, FLAT, LAYER, CURVED)                                        \
    static ::dirac::Registrar DIRAC_CAT(reg_, __LINE__)(::dirac::KernelEntry{                        \
        DIRAC_PREC, N, DIRAC_DIR, R, L, CPT,                                                          \
        ::dirac::LineFFT<DIRAC_T, N, R, L, DIRAC_COLS, CPT>::NT,                                       \
        {reinterpret_cast<const void*>(&::dirac::stage_kernel<DIRAC_T, N, R, L, DIRAC_COLS, 0, CPT>), \
         reinterpret_cast<const void*>(&::dirac::stage_kernel<DIRAC_T, N, R, L, DIRAC_COLS, 1, CPT>), \
         reinterpret_cast<const void*>(&::dirac::stage_kernel<DIRAC_T, N, R, L, DIRAC_COLS, 2, CPT>)},\
        {DIRAC_STREAM(N, R, L, 0, CPT), DIRAC_STREAM(N, R, L, 1, CPT), DIRAC_STREAM(N, R, L, 2, CPT)},\
        OBS, {FLAT, LAYER, CURVED}});
// REG: a direction-kernel schedule.  REGD: one that is the default of grids with at
// least so many lines, up to the next threshold (a negative number: never), per
// mode: flat, flat with a layer, curved.  REGO / REGOD:
// the same plus the observable kernel with that schedule (one per precision, n
// and direction).
#define REG(N, R, L, CPT) DIRAC_REG_IMPL(N, R, L, CPT, nullptr, -1, -1, -1)
#define REGD(N, R, L, CPT, FLAT, LAYER, CURVED) DIRAC_REG_IMPL(N, R, L, CPT, nullptr, FLAT, LAYER, CURVED)
#define DIRAC_OBS(N, R, L, CPT) reinterpret_cast<const void*>(&::dirac::obs_kernel<DIRAC_T, N, R, L, DIRAC_COLS, CPT>)
#define REGO(N, R, L, CPT) DIRAC_REG_IMPL(N, R, L, CPT, DIRAC_OBS(N, R, L, CPT), -1, -1, -1)
#define REGOD(N, R, L, CPT, FLAT, LAYER, CURVED) \
    DIRAC_REG_IMPL(N, R, L, CPT, DIRAC_OBS(N, R, L, CPT), FLAT, LAYER, CURVED)
