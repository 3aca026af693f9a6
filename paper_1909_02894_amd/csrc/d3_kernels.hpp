// d3_kernels.hpp -- direction kernels of the 3-D, 4-spinor step (Scheme II with
// three directions, Sec. 5.2; Dirac representation beta = diag(1, 1, -1, -1),
// alpha^i = [[0, sigma_i], [sigma_i, 0]]).
//
// State: [n3][n2][n1] points, each 4 complex components (u0, u1, w0, w1), i.e.
// 8 T per point.  A line of direction x is a row (stride 1); of direction y a
// column of one z plane (stride n1, lines ordered x-fastest); of direction z a
// column through the planes (stride n1 n2, lines ordered x-fastest), so the L
// lines of a tile are neighbours in memory for y and z.  Per line:
//   [Step 1 (and Step 5 of the previous step): psi <- E psi]
//   psi <- b F^-1[K_i F psi] + (1 - b) psi,  K_i = cos I - i sin alpha^i
//   [Step 5 after the last step]
// E = [[e0 I, D g.sigma], [D g.sigma, conj(e0) I]] with e0 = C - i D w, stored per
// point as (C, -D w, D g_x, D g_y, D g_z) (curved), or diag(e0u, e0u, conj, conj) (flat).
#pragma once
#include "stage_kernels.hpp"

namespace dirac {

template <typename T>
struct D3Params {
    T* psi;                 // 8 T per point
    const T* a;             // a(x) per point, or null (flat)
    const T* E;             // exponential record per point (D3_EREC T), or null (flat)
    const T* inv_s;         // 1/S along the line direction (ones without a layer)
    const cpx<T>* K;        // (cos, sin)(c dt xi) / n
    const cpx<T>* tw;       // exp(-2 pi i m / n) in the per-pass layout of radix d3_radix(n)
    int n1, n2;
    int nlines;
    int e_pre, e_post;
    cpx<T> e0u;             // flat: e^{-i dt m c^2 / 2}
};

template <typename T>
__host__ __device__ constexpr int d3_erec() { return sizeof(T) == 8 ? 6 : 8; }
template <typename T>
__host__ __device__ constexpr int d3_radix(int n) { return (sizeof(T) == 8 || n <= 64) ? 4 : 8; }
// Lines per workgroup: 256 threads (the lines' two half-waves each), one line from
// 128 threads per pair on.
template <typename T>
__host__ __device__ constexpr int d3_lines(int n) {
    return (n / d3_radix<T>(n)) >= 128 ? 1 : 128 / (n / d3_radix<T>(n));
}
template <typename T>
__host__ __device__ constexpr int d3_threads(int n) { return 2 * (n / d3_radix<T>(n)) * d3_lines<T>(n); }

struct D3Entry {
    int prec, n, dir, lines, nthreads;
    const void* fn[3];      // flat, flat + layer, curved
};
const D3Entry* d3_entry(int prec, int n, int dir);

// (C, -D w, D g_x, D g_y, D g_z)
template <typename T>
__device__ __forceinline__ void load_erec(const T* E, uint32_t idx, T (&e)[5]) {
    const char* b = reinterpret_cast<const char*>(E) + idx * (uint32_t)(d3_erec<T>() * sizeof(T));
    if constexpr (sizeof(T) == 8) {
        const double2* q = reinterpret_cast<const double2*>(b);
        const double2 A = q[0], B = q[1], C = q[2];
        e[0] = A.x; e[1] = A.y; e[2] = B.x; e[3] = B.y; e[4] = C.x;
    } else {
        const float4* q = reinterpret_cast<const float4*>(b);
        const float4 A = q[0], B = q[1];
        e[0] = A.x; e[1] = A.y; e[2] = A.z; e[3] = A.w; e[4] = B.x;
    }
}

// DIR 0: x (rows), 1: y, 2: z.  MODE 0 flat, 1 flat + layer, 2 curved.
//
// The two component pairs sit in the two halves of a wave: lanes 0..31 carry (u0,
// u1) and lanes 32..63 (w0, w1) of the same 32 logical threads, and E and K take the
// other pair from the partner lane.  Against all four components in one thread
// (pairs transformed one after the other through one buffer): half the registers
// (226 -> 152 VGPRs for curved FP64 128-point columns, 2 -> 3 waves per SIMD), half the
// barriers, and every load of the tile issued before the first wait.  Bound by
// memory: us per step, before / now: 128^3 FP64 curved 264 / 175 (956 MB, 5.5 TB/s),
// FP32 125 / 95, 64^3 FP64 54 / 39, 256 x 256 x 128 FP32 flat 285 / 247.
template <typename T, int N, int DIR, int MODE>
__global__ void __launch_bounds__(d3_threads<T>(N)) d3_stage_kernel(D3Params<T> p) {
    constexpr int R = d3_radix<T>(N), L = d3_lines<T>(N);
    constexpr bool COLS = DIR != 0, BLEND = MODE != 0, PRELOAD_E = MODE == 2 && DIR == 0;
    using F = LineFFT<T, N, R, L, COLS, 2, kSeqLoose>;
    using TS = TwStage<T, N>;
    static_assert(F::NT % 32 == 0 && !F::SEQ, "whole half-waves, both components exchanged at once");
    constexpr int P = F::P;
    __shared__ cpx<T> lds[2 * F::LDS_ELEMS];
    __shared__ cpx<T> twl[TS::ELEMS];
    const int pair = (threadIdx.x >> 5) & 1, th = ((threadIdx.x >> 6) << 5) | (threadIdx.x & 31);
    const typename F::Coord c = F::coord(th);
    cpx<T>* buf = lds + pair * F::LDS_ELEMS;
    const int line = xcd_tile(blockIdx.x, gridDim.x) * L + c.l;
    const bool valid = line < p.nlines;
    const uint32_t ln = (uint32_t)(valid ? line : p.nlines - 1);     // loads: clamped, branch-free
    const uint32_t n1 = (uint32_t)p.n1, plane = (uint32_t)p.n1 * (uint32_t)p.n2;
    // point r of this thread: a lane part plus a wave-uniform part r step
    uint32_t q0, stride;
    if constexpr (DIR == 0) { q0 = ln * n1; stride = 1; }
    else if constexpr (DIR == 1) { q0 = (ln / n1) * plane + ln % n1; stride = n1; }
    else { q0 = ln; stride = plane; }
    q0 += (uint32_t)c.j * stride;
    const uint32_t step = P * stride;
    const uint32_t h0 = 2 * q0 + pair;                               // this thread's half of the point (4 T)

    cpx<T> v[2][R];
#pragma unroll
    for (int r = 0; r < R; ++r) load_point(upt(p.psi, 8 * (r * step)), h0, v[0][r], v[1][r]);
    T e[MODE == 2 ? R : 1][5];
    auto loadE = [&]() {
        if constexpr (MODE == 2) {
#pragma unroll
            for (int r = 0; r < R; ++r) load_erec(upt(p.E, d3_erec<T>() * (r * step)), q0, e[r]);
        }
    };
    if constexpr (PRELOAD_E) loadE();
    const cpx<T>* tw = p.tw;
    cpx<T> twv[TS::ON ? F::TW_ITER : 1];
    if constexpr (TS::ON) F::template tw_load<false>(twv, p.tw, th);
    T b[BLEND ? R : 1];
    if constexpr (BLEND) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b[r] = ld_at(p.inv_s + r * P, (uint32_t)c.j);            // ones without a layer
            if constexpr (MODE == 2) b[r] = ld_at(upt(p.a, r * step), q0) * b[r];
        }
    }
    cpx<T> kk[R];
#pragma unroll
    for (int s = 0; s < R; ++s) kk[s] = ld_at(p.K + s * P, (uint32_t)c.j);
    if constexpr (TS::ON) {
        if (pair == 0) F::tw_store(twv, twl, th);
        tw = twl;
    }
    // E of the record (C, -D w, D g): the diagonal e0 for u, conj e0 for w; D g.sigma
    // couples to the other pair
    auto applyE = [&](int times) {
        for (int t = 0; t < times; ++t) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (MODE == 2) {
                    const cpx<T> e0{e[r][0], pair ? -e[r][1] : e[r][1]};
                    const cpx<T> pxy{e[r][2], -e[r][3]}, mxy{e[r][2], e[r][3]};
                    const cpx<T> a0 = v[0][r], a1 = v[1][r], b0 = partner(a0), b1 = partner(a1);
                    v[0][r] = cmul(e0, a0) + scal(e[r][4], b0) + cmul(pxy, b1);
                    v[1][r] = cmul(e0, a1) + cmul(mxy, b0) - scal(e[r][4], b1);
                } else {
                    const cpx<T> e0{p.e0u.re, pair ? -p.e0u.im : p.e0u.im};
                    v[0][r] = cmul(e0, v[0][r]);
                    v[1][r] = cmul(e0, v[1][r]);
                }
            }
        }
    };
    if constexpr (PRELOAD_E) {
        applyE(p.e_pre);                                             // 1 or 2
    } else if constexpr (DIR == 0) {                                 // only x launches open with Step 1
        if (p.e_pre > 0) applyE(p.e_pre);
    }
    cpx<T> old[BLEND ? 2 : 1][BLEND ? R : 1];
    if constexpr (BLEND) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            old[0][r] = v[0][r];
            old[1][r] = v[1][r];
        }
    }
    F::template fft<false, true>(v, buf, c, tw);
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const T cs = kk[s].re, sn = kk[s].im;
        const cpx<T> a0 = v[0][s], a1 = v[1][s], b0 = partner(a0), b1 = partner(a1);
        if constexpr (DIR == 0) {                                    // -i sin sigma_x
            v[0][s] = scal(cs, a0) + mul_mi(scal(sn, b1));
            v[1][s] = scal(cs, a1) + mul_mi(scal(sn, b0));
        } else if constexpr (DIR == 1) {                             // -i sin sigma_y = sin (-v1, v0)
            v[0][s] = scal(cs, a0) - scal(sn, b1);
            v[1][s] = scal(cs, a1) + scal(sn, b0);
        } else {                                                     // -i sin sigma_z
            v[0][s] = scal(cs, a0) + mul_mi(scal(sn, b0));
            v[1][s] = scal(cs, a1) + mul_i(scal(sn, b1));
        }
    }
    F::template fft<true, true>(v, buf, c, tw);
    if constexpr (BLEND) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T ob = T(1) - b[r];
            v[0][r] = scal(b[r], v[0][r]) + scal(ob, old[0][r]);
            v[1][r] = scal(b[r], v[1][r]) + scal(ob, old[1][r]);
        }
    }
    if (p.e_post) {
        loadE();
        applyE(1);
    }
    if (!valid) return;
#pragma unroll
    for (int r = 0; r < R; ++r) store_point(p.psi, h0, v[0][r], v[1][r], 2 * (r * step));
}

}  // namespace dirac
