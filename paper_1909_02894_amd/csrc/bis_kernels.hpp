// bis_kernels.hpp -- direction kernels of the second-order directional step
// (Sec. 5.2, eq. (step2bis), corrected reading).  Per line, after the forward
// transform psi_hat = F_i psi:
//   psi* = b Xi + (1 - b) psi
//          + ((c dt)^2 / 2) (b (1 - b) F^-1[xi^2 psi_hat] + b b' F^-1[i xi psi_hat]),
//   Xi = F^-1[K_i psi_hat],  b = a / S^i,  b' = (d_i a) / S^i,
// i.e. the blend of eq. (second_scheme) plus the difference between the exact
// transport d_t psi = -c b sigma_i d_i psi and the blend at second order in dt.
// Three inverse transforms share the forward one; Step 1 / Step 5 are fused as
// in the plain direction kernel.  One schedule per size, radix 4 (bis_cpt,
// bis_lines), up to n = 2048.
#pragma once
#include "stage_kernels.hpp"

namespace dirac {

template <typename T>
struct BisParams {
    StageParams<T> s;
    const T* da;       // (d_x a, d_y a) per point (curved), or null
    const T* D;        // xi / n along the line direction
    T hh;              // (c dt)^2 / 2
    T n;               // transform length, so xi^2 / n = n D^2
};

struct BisEntry {
    int prec, n, dir, lines, nthreads;
    int from_lines;        // for this many lines and more
    const void* fn[2];     // [0] flat with layer, [1] curved
};

// Shape of the kernel of n-point lines.  Up to 512 points one spinor component per
// lane (twice the waves of the two-component form, whose single wave per SIMD was
// bound by its own chain) and as few lines per workgroup as whole waves allow, two
// of 512-point columns; the inverse transforms run side by side, sharing barriers
// and twiddle reads.  Curved 512^2: FP64 35.4 -> 26.1 us per step, FP32 22.6 -> 18.5.
// Longer lines, and 1024 and more columns of 512 points: both components per
// thread, the inverse transforms one after the other (three exchange buffers do
// not fit, or leave one workgroup per compute unit: FP64 2048 x 512 111 against 121).
constexpr int kBisRadix = 4;
__host__ __device__ constexpr int bis_cpt(int n) { return n <= 512 ? 1 : 2; }
__host__ __device__ constexpr int bis_lines(int n) { return n / kBisRadix < 32 ? 32 / (n / kBisRadix) : 1; }
__host__ __device__ constexpr int bis_threads(int n, int lines, int cpt) {
    return (n / kBisRadix) * lines * (cpt == 1 ? 2 : 1);
}

const BisEntry* bis_entry(int prec, int n, int dir, int nlines);

// MODE 1: flat with layer (b = 1/S, b' = 0, uniform diagonal E); MODE 2: curved.
template <typename T, int N, int L, int CPT, bool COLS, int MODE>
__global__ void __launch_bounds__(bis_threads(N, L, CPT)) bis_stage_kernel(BisParams<T> bp) {
    constexpr int R = kBisRadix;
    using F = LineFFT<T, N, R, L, COLS, CPT, kSeqLoose>;
    using TS = TwStage<T, N>;
    constexpr int P = F::P;
    constexpr int dir = COLS ? 1 : 0;
    constexpr int NV = MODE == 2 ? 3 : 2;              // inverse transforms
    constexpr bool BATCH = CPT == 1;
    __shared__ cpx<T> lds[(BATCH ? NV : 1) * F::LDS_ELEMS];
    __shared__ cpx<T> twl[TS::ELEMS];
    const StageParams<T>& p = bp.s;
    const typename F::Coord c = F::coord(threadIdx.x);
    const int line = xcd_tile(blockIdx.x, gridDim.x) * L + c.l;
    const bool valid = line < p.nlines;
    const int lline = valid ? line : p.nlines - 1;     // loads: clamped, branch-free
    const uint32_t n1 = (uint32_t)p.n1;
    auto gidx = [&](int ln, int pos) -> uint32_t {
        return COLS ? (uint32_t)pos * n1 + ln : (uint32_t)ln * n1 + pos;
    };

    // t[cc][r] <- f(own, other, component, r) of a, for every carried component
    auto mix = [&](const cpx<T> (*a)[R], cpx<T> (*t)[R], auto&& f) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (CPT == 1) {
                t[0][r] = f(a[0][r], partner(a[0][r]), c.comp, r);
            } else {
                const cpx<T> a0 = a[0][r], a1 = a[1][r];
                t[0][r] = f(a0, a1, 0, r);
                t[1][r] = f(a1, a0, 1, r);
            }
        }
    };
    // point r of this thread: a lane part (line, c.j) plus a wave-uniform part r step
    const uint32_t ln = gidx(lline, c.j), step = COLS ? P * n1 : P;
    const PointAt<T, sizeof(T) == 8 && CPT == 2> pt(ln);
    static_assert(L <= 16, "every line of a tile exists (grids of at least 16 lines): whole waves store");
    // every global load of the tile goes out before the first wait
    cpx<T> v[CPT][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T* q = upt(p.psi, 4 * (r * step));
        if constexpr (CPT == 1) v[0][r] = load_comp(q, ln, c.comp);
        else pt.load(q, v[0][r], v[1][r]);
    }
    // Step 1 / Step 5: row comp of E = [[e0, e1], [conj e1, conj e0]];
    // direction-x launches always open with Step 1 and load E up front
    constexpr bool PRELOAD_E = MODE == 2 && !COLS;
    cpx<T> e0[MODE == 2 ? R : 1], e1[MODE == 2 ? R : 1];
    auto loadE = [&]() {
        if constexpr (MODE == 2) {
#pragma unroll
            for (int r = 0; r < R; ++r) pt.load(upt(p.E, 4 * (r * step)), e0[r], e1[r]);
        }
    };
    if constexpr (PRELOAD_E) loadE();
    const cpx<T>* tw = p.tw;
    cpx<T> twv[TS::ON ? F::TW_ITER : 1];
    if constexpr (TS::ON) F::template tw_load<false>(twv, p.tw, threadIdx.x);
    T b[R], k2[R], k1[R], dsym[R];
    cpx<T> ksym[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int pos = c.j + r * P;
        const T s = gld(p.inv_s + pos);            // ones without a layer
        T a = T(1), da = T(0);
        if constexpr (MODE == 2) {
            a = ld_at(p.a + r * P, (uint32_t)lline * N + c.j);   // a along this direction's lines
            da = ld_at(upt(bp.da, 2 * (r * step)), 2 * ln + dir);
        }
        b[r] = a * s;
        k2[r] = bp.hh * (b[r] * (T(1) - b[r]));
        k1[r] = bp.hh * (b[r] * (da * s));
        dsym[r] = gld(bp.D + pos);
        ksym[r] = gld(p.K + pos);
    }
    if constexpr (TS::ON) {
        F::tw_store(twv, twl, threadIdx.x);
        tw = twl;
    }
    auto applyE = [&](int times) {
        for (int t = 0; t < times; ++t)
            mix(v, v, [&](cpx<T> own, cpx<T> other, int comp, int r) {
                const T sg = comp ? T(-1) : T(1);
                if constexpr (MODE == 2)
                    return cmul(cpx<T>{e0[r].re, sg * e0[r].im}, own) + cmul(cpx<T>{e1[r].re, sg * e1[r].im}, other);
                else                               // uniform diag(e0u, conj e0u)
                    return cmul(cpx<T>{p.e0u.re, sg * p.e0u.im}, own);
            });
    };
    if constexpr (PRELOAD_E) {
        applyE(1);                             // e_pre is 1 or 2 here
        if (p.e_pre > 1) applyE(1);
    } else if (p.e_pre > 0) {
        loadE();
        applyE(p.e_pre);
    }
    cpx<T> old[CPT][R];
#pragma unroll
    for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
        for (int r = 0; r < R; ++r) old[cc][r] = v[cc][r];

    F::template fft<false, true>(v, lds, c, tw);
    // the spectra of the inverse transforms: K psi_hat, xi^2 psi_hat, i xi psi_hat
    auto symK = [&](cpx<T> (*t)[R]) {
        mix(v, t, [&](cpx<T> own, cpx<T> other, int comp, int s) {
            const cpx<T> k = ksym[s];
            if constexpr (!COLS) return scal(k.re, own) + mul_mi(scal(k.im, other));  // K_x = cos I - i sin sigma_x
            else return scal(k.re, own) - scal(comp ? -k.im : k.im, other);           // K_y = [[cos, -sin], [sin, cos]]
        });
    };
    auto sym2 = [&](cpx<T> (*t)[R]) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int s = 0; s < R; ++s) t[cc][s] = scal(bp.n * dsym[s] * dsym[s], v[cc][s]);
    };
    auto sym1 = [&](cpx<T> (*t)[R]) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int s = 0; s < R; ++s) t[cc][s] = mul_i(scal(dsym[s], v[cc][s]));
    };
    cpx<T> acc[CPT][R];
    // (c dt)^2 / 2 (b (1 - b) F^-1[xi^2 psi_hat] + b b' F^-1[i xi psi_hat])
    auto add2 = [&](const cpx<T> (*t)[R]) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[cc][r] = scal(k2[r], t[cc][r]);
    };
    auto add1 = [&](const cpx<T> (*t)[R]) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[cc][r] = acc[cc][r] + scal(k1[r], t[cc][r]);
    };
    if constexpr (BATCH) {
        cpx<T> t[NV * CPT][R];
        symK(t);
        sym2(t + CPT);
        if constexpr (MODE == 2) sym1(t + 2 * CPT);
        F::template fft<true, true, 1, 0, NV>(t, lds, c, tw);
        add2(t + CPT);
        if constexpr (MODE == 2) add1(t + 2 * CPT);
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int r = 0; r < R; ++r) v[cc][r] = t[cc][r];
    } else {
        cpx<T> t[CPT][R];
        sym2(t);
        F::template fft<true, true>(t, lds, c, tw);
        add2(t);
        if constexpr (MODE == 2) {
            sym1(t);
            F::template fft<true, true>(t, lds, c, tw);
            add1(t);
        }
        symK(v);
        F::template fft<true, true>(v, lds, c, tw);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
            v[cc][r] = scal(b[r], v[cc][r]) + scal(T(1) - b[r], old[cc][r]) + acc[cc][r];
    }
    if (p.e_post) {
        loadE();
        applyE(1);
    }
    if (!valid) return;
    const bool wt = (!COLS || N <= kStoreWtMaxColN) && p.wt;       // write-through (as in stage_tile)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if constexpr (CPT == 1) {
            if (wt) store_comp<T, true>(p.psi, ln, c.comp, v[0][r], r * step);
            else store_comp(p.psi, ln, c.comp, v[0][r], r * step);
        } else {
            if (wt) pt.template store<true>(p.psi, v[0][r], v[1][r], r * step);
            else pt.template store<false>(p.psi, v[0][r], v[1][r], r * step);
        }
    }
}

}  // namespace dirac
