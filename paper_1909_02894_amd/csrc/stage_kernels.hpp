// stage_kernels.hpp -- fused direction kernels of one time step, and the fused
// spectral-derivative / reduction kernels of the observables.
//
// Direction kernel (one launch per direction per step), for each line:
//   [Step 1: psi <- E psi, once or twice (Step 5 of the previous step, then
//    Step 1 of this one)]                      (Scheme II Steps 1 and 5)
//   old <- psi
//   psi_hat <- F_i psi (both components)        (Sec. 5 partial DFT)
//   psi_hat <- (K_i(xi) / n) psi_hat, K_x = cos I - i sin sigma_x,
//              K_y = cos I - i sin sigma_y, angle c dt xi   (eq. (second_scheme))
//   Xi <- unnormalised inverse transform of psi_hat
//   psi <- b Xi + (1 - b) old, b = a(x) / S^i(x^i)          (eq. (second_scheme) with PML)
//   [Step 5 after the last step: psi <- E psi]
// The state is an AoS array of points (component 0, component 1), each a
// complex (re, im), so one grid point is 4 reals: rows are contiguous (x
// direction), columns are read as coalesced row segments of L points.
#pragma once
#include "fft_line.hpp"

namespace dirac {

template <typename T>
struct StageParams {
    T* psi;                      // state, 4 T per point, row pitch `pitch` points
    const T* a;                  // a(x) per point along this direction's lines (row-major for x,
                                 // the transposed table for y: a[line * n + pos]), or null (a = 1)
    const T* E;                  // half-step exponential per point (e0 re, im, e1 re, im), or null
    const T* inv_s;              // 1/S along the line direction (n entries; ones without a layer)
    const cpx<T>* K;             // symbol per mode, already scaled by 1/n
    const cpx<T>* tw;            // exp(-2 pi i m / n) in the per-pass layout of the kernel's radix
    int n1;                      // points per row (pitch of the E table)
    int pitch;                   // points from one state row to the next (>= n1)
    int nlines;                  // lines of this direction
    int e_pre;                   // Step-1 exponentials applied before the transform: 1 or 2 in
                                 // direction-x launches (which load E up front; 0 in the flat
                                 // ones behind a potentials pass); direction-y kernels ignore it
    int e_post;                  // Step-5 exponential applied after the blend (0, 1)
    cpx<T> e0u;                  // uniform e0 when E is null (flat: e^{-i dt m c^2 / 2})
    int wt;                      // 1: write-through state stores (rows; columns of n <= 1024)
};

struct ObsParams {
    const void* psi;             // state (T)
    const double* w;             // observable weight planes, each n1*n2 doubles:
    const double* ca;            //   w = e^{chi - Phi + Psi}, ca = c a,
    const double* gx;            //   gx = c a chi_x / 2, gy = c a chi_y / 2,
    const double* gy;            //   V = e^Phi m c^2
    const double* V;
    const double* ax;            // potentials, or null: e c a A_x, e c a A_y, e V planes
    const double* ay;
    const double* v0;
    double fA, fV;               //   and their envelopes at the observation time
    const void* D;               // derivative symbol xi_p / n (T), n entries
    const void* tw;              // twiddles (cpx<T>)
    double* partials;            // 8 doubles per workgroup
    int n1, n2;
    int pitch;                   // points from one state row to the next
    int nlines;
    double a1, a2, h1, h2;
};

// Point access with 32-bit byte offsets (every supported state is < 2 GiB), so
// addresses are formed as a scalar base plus a 32-bit vector offset.
template <typename T>
__device__ __forceinline__ T ld_at(const T* base, uint32_t elem) {
    return gld(reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + elem * (uint32_t)sizeof(T)));
}
template <typename T>
__device__ __forceinline__ T ld_nt(const T* p) {
    return __builtin_nontemporal_load((const __attribute__((address_space(1))) T*)p);
}
// base advanced by a wave-uniform number of elements: a scalar addition, so that
// the R accesses of a thread share one vector offset (its lane part) instead of
// holding R of them (n = 4096 FP32 columns: 22 VGPRs fewer).
template <typename T>
__device__ __forceinline__ T* upt(T* base, uint32_t elems) { return base + (size_t)elems; }

// One spinor component of a point (component c at byte offset c * 2 sizeof(T)).
template <typename T>
__device__ __forceinline__ cpx<T> load_comp(const T* p, uint32_t idx, int c) {
    const char* b = reinterpret_cast<const char*>(p) + idx * (uint32_t)(4 * sizeof(T)) + c * (uint32_t)(2 * sizeof(T));
    return gld(reinterpret_cast<const cpx<T>*>(b));
}
// Both components of a point in one access (16 B for FP32) or two (FP64).
template <typename T>
__device__ __forceinline__ void load_point(const T* p, uint32_t idx, cpx<T>& u, cpx<T>& v) {
    const char* b = reinterpret_cast<const char*>(p) + idx * (uint32_t)(4 * sizeof(T));
    if constexpr (sizeof(T) == 8) {
        const d2v A = gld(reinterpret_cast<const d2v*>(b)), B = gld(reinterpret_cast<const d2v*>(b) + 1);
        u = {(T)A.x, (T)A.y};
        v = {(T)B.x, (T)B.y};
    } else {
        const f4v A = gld(reinterpret_cast<const f4v*>(b));
        u = {(T)A.x, (T)A.y};
        v = {(T)A.z, (T)A.w};
    }
}
// FP64 points in accesses that cover whole cache lines.  A thread that holds both
// components reads its 32-byte point as two 16-byte pieces, and each of the wave's
// two accesses touches half of every line.  Instead the half-waves share: access A
// reads the points of lanes 0..31 (component 0 in those lanes, component 1 in their
// partners lane xor 32), access B those of lanes 32..63, and one half-wave swap
// per word puts each point into its own lane (stores: the swap first).  us per
// launch, plain / shared: FP64 2048 rows radix 8 flat 79 / 70, curved 100 / 95,
// columns 99 / 90 and 113 / 104; 4096 curved rows 610 / 423, columns 585 / 495;
// 1024 curved columns radix 8 x 2 lines 34 / 26.
struct PairOffsets { uint32_t a, b; };         // byte offsets of a lane's part of accesses A and B
__device__ __forceinline__ PairOffsets pair_offsets(uint32_t idx) {
    const uint32_t other = partner_u32(idx);
    return (threadIdx.x & 32) ? PairOffsets{other * 32 + 16, idx * 32 + 16} : PairOffsets{idx * 32, other * 32};
}
// upper half of A <-> lower half of B
__device__ __forceinline__ void swap_halves(d2v& A, d2v& B) {
    u32x4 a = __builtin_bit_cast(u32x4, A), b = __builtin_bit_cast(u32x4, B);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(a[k], b[k], false, false);
        a[k] = r[0];
        b[k] = r[1];
    }
    A = __builtin_bit_cast(d2v, a);
    B = __builtin_bit_cast(d2v, b);
}
__device__ __forceinline__ void load_points(const double* p, PairOffsets o, cpx<double>& u, cpx<double>& v) {
    const char* c = reinterpret_cast<const char*>(p);
    d2v A = gld(reinterpret_cast<const d2v*>(c + o.a)), B = gld(reinterpret_cast<const d2v*>(c + o.b));
    swap_halves(A, B);
    u = {A.x, A.y};
    v = {B.x, B.y};
}
template <bool WT = false>
__device__ __forceinline__ void store_points(double* p, PairOffsets o, cpx<double> u, cpx<double> v, uint32_t uidx = 0) {
    d2v A{u.re, u.im}, B{v.re, v.im};
    swap_halves(A, B);
    p = upt(p, 4 * uidx);
    if constexpr (WT) {
        gst_wt16(p, o.a, __builtin_bit_cast(u32x4, A));
        gst_wt16(p, o.b, __builtin_bit_cast(u32x4, B));
    } else {
        char* c = reinterpret_cast<char*>(p);
        gst(reinterpret_cast<d2v*>(c + o.a), A);
        gst(reinterpret_cast<d2v*>(c + o.b), B);
    }
}
// A point (idx + a wave-uniform part in the base or uidx) by either way: plain
// accesses, or (PAIRED, FP64) those above, which need every lane of the wave.
template <typename T, bool PAIRED>
struct PointAt {
    uint32_t idx;
    __device__ __forceinline__ explicit PointAt(uint32_t i) : idx(i) {}
    __device__ __forceinline__ void load(const T* p, cpx<T>& u, cpx<T>& v) const { load_point(p, idx, u, v); }
    template <bool WT>
    __device__ __forceinline__ void store(T* p, cpx<T> u, cpx<T> v, uint32_t uidx) const {
        store_point<T, WT>(p, idx, u, v, uidx);
    }
};
template <>
struct PointAt<double, true> {
    PairOffsets o;
    __device__ __forceinline__ explicit PointAt(uint32_t i) : o(pair_offsets(i)) {}
    __device__ __forceinline__ void load(const double* p, cpx<double>& u, cpx<double>& v) const { load_points(p, o, u, v); }
    template <bool WT>
    __device__ __forceinline__ void store(double* p, cpx<double> u, cpx<double> v, uint32_t uidx) const {
        store_points<WT>(p, o, u, v, uidx);
    }
};

// Longest column line whose kernel carries the write-through store path.
constexpr int kStoreWtMaxColN = 1024;

// WT: device-scope write-through stores (gst_wt16 / gst_wt8) instead of
// ordinary ones; p must be wave-uniform then (the kernel's state pointer).
// The point is idx + uidx (uidx wave-uniform).
template <typename T, bool WT = false>
__device__ __forceinline__ void store_point(T* p, uint32_t idx, cpx<T> u, cpx<T> v, uint32_t uidx = 0) {
    const uint32_t off = idx * (uint32_t)(4 * sizeof(T));
    p = upt(p, 4 * uidx);
    char* b = reinterpret_cast<char*>(p) + off;
    if constexpr (sizeof(T) == 8) {
        const d2v a{u.re, u.im}, c{v.re, v.im};
        if constexpr (WT) {
            gst_wt16(p, off, __builtin_bit_cast(u32x4, a));
            gst_wt16(p, off + 16, __builtin_bit_cast(u32x4, c));
        } else {
            gst(reinterpret_cast<d2v*>(b), a);
            gst(reinterpret_cast<d2v*>(b) + 1, c);
        }
    } else {
        const f4v a{u.re, u.im, v.re, v.im};
        if constexpr (WT) gst_wt16(p, off, __builtin_bit_cast(u32x4, a));
        else gst(reinterpret_cast<f4v*>(b), a);
    }
}
template <typename T, bool WT = false>
__device__ __forceinline__ void store_comp(T* p, uint32_t idx, int c, cpx<T> v, uint32_t uidx = 0) {
    const uint32_t off = idx * (uint32_t)(4 * sizeof(T)) + c * (uint32_t)(2 * sizeof(T));
    p = upt(p, 4 * uidx);
    char* b = reinterpret_cast<char*>(p) + off;
    if constexpr (sizeof(T) == 8) {
        const d2v a{v.re, v.im};
        if constexpr (WT) gst_wt16(p, off, __builtin_bit_cast(u32x4, a));
        else gst(reinterpret_cast<d2v*>(b), a);
    } else {
        const f2v a{v.re, v.im};
        if constexpr (WT) gst_wt8(p, off, __builtin_bit_cast(u32x2, a));
        else gst(reinterpret_cast<f2v*>(b), a);
    }
}

// Workgroup -> tile map that keeps neighbouring tiles on one XCD.  Workgroups
// are dispatched round-robin over the 8 XCDs, each with its own L2; tiles that
// share cache lines (adjacent column tiles, adjacent rows of the per-point
// tables) are given to consecutive workgroups of the same XCD.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
    const int x = b & 7, k = b >> 3;
    const int q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + k;
}

// Small twiddle tables are staged in LDS at kernel start (one coalesced read)
// so the per-pass twiddle reads do not sit on the critical path.
template <typename T, int N>
struct TwStage {
    static constexpr bool ON = N * sizeof(cpx<T>) <= kTwStageMax;
    static constexpr int ELEMS = ON ? N : 1;
};

// Exchange buffers of a single solve's direction kernel: two (one barrier per
// exchange instead of two) for the tiles of one component per lane, whose solves
// are small and bound by latency, where at least three workgroups still fit a
// compute unit.  us per step, one buffer / two: curved FP64 512^2 17.6 / 17.0,
// FP32 12.9 / 12.5; FP64 128^2 9.0 / 8.6.
template <typename T, int N, int R, int L, bool COLS, int CPT>
constexpr int stage_buffers() {
    using F = LineFFT<T, N, R, L, COLS, CPT>;
    return CPT == 1 && F::NPASS > 1 && 3 * (2 * F::LDS_ELEMS + TwStage<T, N>::ELEMS) * sizeof(cpx<T>) <= kLdsMax ? 2 : 1;
}

// MODE 0: flat, no absorbing layer (b = 1: psi <- Xi; E uniform diagonal)
// MODE 1: flat with layer (b = 1/S along the line; E uniform diagonal)
// MODE 2: curved (b = a(x) [/S]; E from the per-point table)
// One tile (L lines) of a direction stage, executed by F::NT threads.  lds and
// twl are the workgroup's NB exchange buffers (F::LDS_ELEMS each) and twiddle stage
// (TwStage::ELEMS).  Every per-line operation depends on (T, N, R, MODE) only:
// the 2x2 mixes are written per output component as (own, other) expressions
// that are the same whether the other component sits in the same thread
// (CPT = 2) or in the partner lane (CPT = 1), so results do not depend on L or CPT.
template <typename T, int N, int R, int L, bool COLS, int MODE, int CPT, int NB = 1, int RULE = kSeqTight>
__device__ __forceinline__ void stage_tile(const StageParams<T>& p, int tile, cpx<T>* lds, cpx<T>* twl) {
    using F = LineFFT<T, N, R, L, COLS, CPT, RULE>;
    using TS = TwStage<T, N>;
    constexpr int P = F::P;
    constexpr bool BLEND = MODE != 0;
    // prefetch symbols and blend weights before the transform when registers allow
    constexpr bool PF = sizeof(T) * R * CPT <= 64 && F::NT <= 512;
    const typename F::Coord c = F::coord(threadIdx.x);
    const int line = tile * L + c.l;
    const bool valid = line < p.nlines;
    // loads read a clamped line (always in bounds, results unused past the
    // last line) so that they carry no branches; stores are guarded
    const int lline = valid ? line : p.nlines - 1;
    const uint32_t pitch = (uint32_t)p.pitch, n1 = (uint32_t)p.n1;
    // Point r of this thread sits at position c.j + r P of its line: a lane part
    // (line, c.j) plus a wave-uniform part r P, which goes into the scalar base.
    const uint32_t sln = COLS ? (uint32_t)c.j * pitch + lline : (uint32_t)lline * pitch + c.j;   // state
    const uint32_t eln = COLS ? (uint32_t)c.j * n1 + lline : (uint32_t)lline * n1 + c.j;         // E table
    // the a table is laid out along this direction's lines (transposed for columns)
    const uint32_t aln = (uint32_t)lline * N + c.j;
    const uint32_t sstep = COLS ? P * pitch : P, estep = COLS ? P * n1 : P;
    // FP64 points by shared accesses; not in the flat radix-16 tiles of up to 256
    // threads, which hold two waves per SIMD with no register to spare (2048 columns
    // 77 / 93 us, 4096 rows 280 / 533).  Grids are powers of two from 16 points, so a
    // tile of up to 16 lines is never cut and all its lanes reach the stores.
    constexpr bool PAIRED = sizeof(T) == 8 && CPT == 2 && L <= 16 && !(R == 16 && MODE != 2 && F::NT <= 256);
    const PointAt<T, PAIRED> spt(sln), ept(eln);
    // v[cc][r] <- f(own, other, component, r) for every carried component
    auto mix = [&](cpx<T> (&a)[CPT][R], auto&& f) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (CPT == 1) {
                const cpx<T> o = a[0][r];
                a[0][r] = f(o, partner(o), c.comp, r);
            } else {
                const cpx<T> a0 = a[0][r], a1 = a[1][r];
                a[0][r] = f(a0, a1, 0, r);
                a[1][r] = f(a1, a0, 1, r);
            }
        }
    };

    // Every global load of the tile is issued in one branch-free block before
    // the first use of any of them, so the tile pays one memory latency:
    // state, Step-1 exponential, twiddles, symbols and blend weights.
    cpx<T> v[CPT][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T* q = upt(p.psi, 4 * (r * sstep));
        if constexpr (CPT == 1) v[0][r] = load_comp(q, sln, c.comp);
        else spt.load(q, v[0][r], v[1][r]);
    }
    // Step 1 (and Step 5 of the previous step): row `comp` of
    // E = [[e0, e1], [conj e1, conj e0]]: A own + B other with A = e0, B = e1 for
    // component 0 and their conjugates for component 1.  Direction-x launches
    // always open with Step 1 (e_pre is 1 or 2), so they load E up front and
    // apply it once unconditionally.
    constexpr bool PRELOAD_E = MODE == 2 && !COLS;
    cpx<T> e0[MODE == 2 ? R : 1], e1[MODE == 2 ? R : 1];
    auto loadE = [&]() {
        if constexpr (MODE == 2) {
#pragma unroll
            for (int r = 0; r < R; ++r) ept.load(upt(p.E, 4 * (r * estep)), e0[r], e1[r]);
        }
    };
    auto applyE = [&](int times) {
        if constexpr (MODE == 2) {
            for (int t = 0; t < times; ++t)
                mix(v, [&](cpx<T> own, cpx<T> other, int comp, int r) {
                    const T sg = comp ? T(-1) : T(1);
                    return cmul(cpx<T>{e0[r].re, sg * e0[r].im}, own) + cmul(cpx<T>{e1[r].re, sg * e1[r].im}, other);
                });
        } else {
            for (int t = 0; t < times; ++t)
                mix(v, [&](cpx<T> own, cpx<T>, int comp, int) {
                    return cmul(cpx<T>{p.e0u.re, comp ? -p.e0u.im : p.e0u.im}, own);
                });
        }
    };
    if constexpr (PRELOAD_E) loadE();
    const cpx<T>* tw = p.tw;
    cpx<T> twv[TS::ON ? F::TW_ITER : 1];
    if constexpr (TS::ON) F::template tw_load<false>(twv, p.tw, threadIdx.x);
    // blend weight b = a(x) / S(x^i) (MODE 2) or 1 / S(x^i) (MODE 1); the 1/S
    // table is always present in blended modes (ones without a layer)
    cpx<T> kk[PF ? R : 1];
    T bb[BLEND ? R : 1];
    auto blend_weights = [&]() {
        if constexpr (BLEND) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T sv = ld_at(p.inv_s + r * P, (uint32_t)c.j);
                // columns of 4096+ points (states beyond the Infinity Cache) read a with
                // a streaming load, which keeps it from evicting the partly written row
                // segments of neighbouring column tiles; shorter lines keep it cached
                // (curved FP64 2048² columns: 113 us cached, 133 us streamed)
                if constexpr (MODE == 2 && COLS && N >= 4096) bb[r] = ld_nt(p.a + r * P + aln) * sv;
                else bb[r] = MODE == 2 ? ld_at(p.a + r * P, aln) * sv : sv;
            }
        }
    };
    if constexpr (PF) {
#pragma unroll
        for (int s = 0; s < R; ++s) kk[s] = ld_at(p.K + s * P, (uint32_t)c.j);
        blend_weights();
    }
    if constexpr (TS::ON) {
        F::tw_store(twv, twl, threadIdx.x);
        tw = twl;
    }
    if constexpr (PRELOAD_E) {
        applyE(1);                                 // e_pre is 1 or 2 here
        if (p.e_pre > 1) applyE(1);
    } else if constexpr (!COLS) {                  // column launches never open with Step 1
        if (p.e_pre > 0) {
            loadE();
            applyE(p.e_pre);
        }
    }
    // The blend needs the state before the transform.  Long column tiles, whose
    // registers are the tightest, read it again from memory at the blend
    // instead of holding it through both transforms (no other workgroup writes
    // these points, and this one stores them only after the blend, and column
    // launches apply no E before the transform, so the values are the same).
    constexpr bool REREAD = BLEND && COLS && N * sizeof(cpx<T>) >= 32768;
    cpx<T> old[BLEND ? CPT : 1][BLEND ? R : 1];
    if constexpr (BLEND && !REREAD) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
            for (int r = 0; r < R; ++r) old[cc][r] = v[cc][r];
    }

    F::template fft<false, true, NB>(v, lds, c, tw);
    mix(v, [&](cpx<T> own, cpx<T> other, int comp, int s) {
        cpx<T> k;
        if constexpr (PF) k = kk[s];
        else k = ld_at(p.K + s * P, (uint32_t)c.j);    // (cos, sin) / n
        if constexpr (!COLS) {                         // K_x = cos I - i sin sigma_x
            return scal(k.re, own) + mul_mi(scal(k.im, other));
        } else {                                       // K_y = [[cos, -sin], [sin, cos]]
            return scal(k.re, own) - scal(comp ? -k.im : k.im, other);
        }
    });
    F::template fft<true, true, NB, (F::NPASS - 1) % 2>(v, lds, c, tw);

    if constexpr (BLEND) {
        if constexpr (REREAD) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T* q = upt(p.psi, 4 * (r * sstep));
                if constexpr (CPT == 1) old[0][r] = load_comp(q, sln, c.comp);
                else spt.load(q, old[0][r], old[1][r]);
            }
        }
        if constexpr (!PF) blend_weights();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T b = bb[r];
#pragma unroll
            for (int cc = 0; cc < CPT; ++cc) v[cc][r] = scal(b, v[cc][r]) + scal(T(1) - b, old[cc][r]);
        }
    }
    if (p.e_post) {
        loadE();
        applyE(1);
    }
    if (!valid) return;
    // write-through stores exist in every row kernel and in the column kernels
    // of n <= 1024: the extra store path perturbs the long column kernels
    // (the 4096-point one ran 16% slower with it, executed or not)
    if ((!COLS || N <= kStoreWtMaxColN) && p.wt) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (CPT == 1) store_comp<T, true>(p.psi, sln, c.comp, v[0][r], r * sstep);
            else spt.template store<true>(p.psi, v[0][r], v[1][r], r * sstep);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (CPT == 1) store_comp(p.psi, sln, c.comp, v[0][r], r * sstep);
            else spt.template store<false>(p.psi, v[0][r], v[1][r], r * sstep);
        }
    }
}

// Streamed column tiles.  A radix-16 tile of 64 KB per component pair leaves room for
// one workgroup per compute unit (its registers hold 64 KB twice over), so its loads,
// transforms and stores follow one another with nothing beside them: curved FP32 4096
// columns ran at 1.8 TB/s with the vector units 31% and the LDS 10% busy.  One
// workgroup per compute unit that takes several tiles in turn (stage_stream_kernel) has
// them overlap.  Grids with fewer tiles than that, and the flat FP64 tiles (two
// workgroups still fit: 4096 x 2048 276 us per step, streamed 300), keep a workgroup per
// tile.  us per step, a workgroup per tile / streamed: FP32 4096^2 flat 326 / 300, layer
// 355 / 303, curved 465 / 408; 512 x 4096 curved 60 / 55, flat 47.1 / 48.0; 256 x 4096
// curved 41.6 / 42.5; FP32 4096 x 2048 (4 lines) curved 226 / 186; FP64 2048^2 layer
// 176 / 159, curved 226 / 198.
template <typename T, int N, int R, int L, bool COLS, int MODE, int CPT>
constexpr bool stage_streams() {
    return COLS && CPT == 2 && R == 16 && N * sizeof(cpx<T>) <= 32768 && N >= 2048 &&
           N * L * sizeof(cpx<T>) == 65536 && (MODE != 0 || sizeof(T) == 4);
}
constexpr int kStreamGroups = 256;             // compute units
// Least number of tiles for a streamed launch: one per compute unit, where the staged
// tables already pay in the blended modes; more than that in the flat one.
constexpr int stream_from_tiles(int mode) { return mode == 0 ? kStreamGroups + 1 : kStreamGroups; }

// One workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ...: the loads of
// the next tile's state are issued before this tile's transforms and arrive behind
// them, its stores drain behind the next tile's.  Twiddles, symbols and 1/S are
// staged in LDS once, so that no short load waits behind the long ones (loads
// return in order); only a(x), issued first, and the call's last E are read per tile.
// Results are bitwise those of stage_tile: every operation on a line is the same.
template <typename T, int N, int R, int L, int MODE>
__global__ void __launch_bounds__((N / R) * L) stage_stream_kernel(StageParams<T> p) {
    using F = LineFFT<T, N, R, L, true, 2, kSeqAlways>;
    constexpr int P = F::P;
    constexpr bool BLEND = MODE != 0, WIDE = sizeof(T) == 8;
    using raw = std::conditional_t<WIDE, d2v, f4v>;
    constexpr int RW = WIDE ? 2 : 1;
    __shared__ cpx<T> lds[F::LDS_ELEMS];
    __shared__ cpx<T> twl[F::TW_ENTRIES], kl[N];
    __shared__ T sl[BLEND ? N : 1];
    const typename F::Coord c = F::coord(threadIdx.x);
    const uint32_t pitch = (uint32_t)p.pitch, n1 = (uint32_t)p.n1;
    const uint32_t sln = (uint32_t)c.j * pitch + c.l, eln = (uint32_t)c.j * n1 + c.l, aln = (uint32_t)c.l * N + c.j;
    const uint32_t sstep = P * pitch, estep = P * n1;
    const PointAt<T, WIDE> spt(sln), ept(eln);
    const int ntiles = p.nlines / L;           // grids are powers of two from 16 points
    // curved tiles have no registers for the last LATE points of the next tile until
    // this one's old values are used up (FP32 4096^2 with all 16 early: 20 registers
    // spilled, 452 us per step, with 12: 417)
    constexpr int LATE = MODE == 2 ? (L == 4 ? 6 : 4) : 0;
    raw nx[R][RW];
    auto load = [&](int tile, uint32_t sstep, int ra, int rb) {
        const T* base = upt(p.psi, 4 * (uint32_t)tile * L);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r < ra || r >= rb) continue;
            const char* q = reinterpret_cast<const char*>(upt(base, 4 * (r * sstep)));
            if constexpr (WIDE) {
                nx[r][0] = gld(reinterpret_cast<const d2v*>(q + spt.o.a));
                nx[r][1] = gld(reinterpret_cast<const d2v*>(q + spt.o.b));
            } else {
                nx[r][0] = gld(reinterpret_cast<const f4v*>(q + spt.idx * (uint32_t)(4 * sizeof(T))));
            }
        }
    };
    int t = blockIdx.x;
    load(xcd_tile(t, ntiles), sstep, 0, R);
    for (int e = threadIdx.x; e < F::TW_ENTRIES; e += F::NT) twl[e] = gld(p.tw + e);
    for (int e = threadIdx.x; e < N; e += F::NT) {
        kl[e] = gld(p.K + e);
        if constexpr (BLEND) sl[e] = gld(p.inv_s + e);
    }
    while (t < ntiles) {
        const int tile = xcd_tile(t, ntiles);
        cpx<T> v[2][R], old[BLEND ? 2 : 1][BLEND ? R : 1];
        T bb[MODE == 2 ? R : 1];
        if constexpr (MODE == 2) {
            const T* a = upt(p.a, (uint32_t)tile * L * N);
#pragma unroll
            for (int r = 0; r < R; ++r) bb[r] = N >= 4096 ? ld_nt(a + r * P + aln) : ld_at(a + r * P, aln);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (WIDE) {
                swap_halves(nx[r][0], nx[r][1]);
                v[0][r] = {nx[r][0].x, nx[r][0].y};
                v[1][r] = {nx[r][1].x, nx[r][1].y};
            } else {
                v[0][r] = {nx[r][0].x, nx[r][0].y};
                v[1][r] = {nx[r][0].z, nx[r][0].w};
            }
            if constexpr (BLEND) {
                old[0][r] = v[0][r];
                old[1][r] = v[1][r];
            }
        }
        t += gridDim.x;
        // past the last tile the loads go on, to one row of the tile in hand: a branch
        // around them costs registers on both of its sides
        const bool more = t < ntiles;
        const int next = more ? xcd_tile(t, ntiles) : tile;
        const uint32_t nstep = more ? sstep : 0;
        load(next, nstep, 0, R - LATE);
        F::template fft<false, true>(v, lds, c, twl);
#pragma unroll
        for (int s = 0; s < R; ++s) {          // K_y = [[cos, -sin], [sin, cos]]
            if (s % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            const cpx<T> k = kl[c.j + s * P], u = v[0][s], w = v[1][s];
            v[0][s] = scal(k.re, u) - scal(k.im, w);
            v[1][s] = scal(k.re, w) - scal(-k.im, u);
        }
        F::template fft<true, true>(v, lds, c, twl);
        if constexpr (BLEND) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                const T sv = sl[c.j + r * P], b = MODE == 2 ? bb[r] * sv : sv;
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) v[cc][r] = scal(b, v[cc][r]) + scal(T(1) - b, old[cc][r]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (LATE > 0) load(next, nstep, R - LATE, R);
        T* out = upt(p.psi, 4 * (uint32_t)tile * L);
        if (p.e_post) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r % 2 == 0) __builtin_amdgcn_sched_barrier(0);
                const cpx<T> u = v[0][r], w = v[1][r];
                if constexpr (MODE == 2) {
                    cpx<T> e0, e1;
                    ept.load(upt(upt(p.E, 4 * (uint32_t)tile * L), 4 * (r * estep)), e0, e1);
                    v[0][r] = cmul(cpx<T>{e0.re, T(1) * e0.im}, u) + cmul(cpx<T>{e1.re, T(1) * e1.im}, w);
                    v[1][r] = cmul(cpx<T>{e0.re, T(-1) * e0.im}, w) + cmul(cpx<T>{e1.re, T(-1) * e1.im}, u);
                } else {
                    v[0][r] = cmul(p.e0u, u);
                    v[1][r] = cmul(cpx<T>{p.e0u.re, -p.e0u.im}, w);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) spt.template store<false>(out, v[0][r], v[1][r], r * sstep);
    }
}

template <typename T, int N, int R, int L, bool COLS, int MODE, int CPT>
__global__ void __launch_bounds__((CPT == 1 ? 2 : 1) * (N / R) * L)
stage_kernel(StageParams<T> p) {
    constexpr int NB = stage_buffers<T, N, R, L, COLS, CPT>();
    __shared__ cpx<T> lds[NB * LineFFT<T, N, R, L, COLS, CPT>::LDS_ELEMS];
    __shared__ cpx<T> twl[TwStage<T, N>::ELEMS];
    stage_tile<T, N, R, L, COLS, MODE, CPT, NB>(p, xcd_tile(blockIdx.x, gridDim.x), lds, twl);
}

// The streamed kernel of a schedule and mode, or null.
template <typename T, int N, int R, int L, bool COLS, int MODE, int CPT>
const void* stream_fn() {
    if constexpr (stage_streams<T, N, R, L, COLS, MODE, CPT>())
        return reinterpret_cast<const void*>(&stage_stream_kernel<T, N, R, L, MODE>);
    else
        return nullptr;
}

// Deterministic workgroup sum of NV doubles per thread into out[0..NV).
template <int NT, int NV>
__device__ __forceinline__ void block_sum(double (&acc)[NV], double* out) {
    __shared__ double red[NT > 64 ? NT / 64 : 1][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double x = acc[k];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        acc[k] = x;
    }
    if (NT <= 64) {
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) out[k] = acc[k];
        }
        return;
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) red[wave][k] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double x = 0.0;
            for (int w = 0; w < NT / 64; ++w) x += red[w][k];
            out[k] = x;
        }
    }
}

// Observable pass along one direction: Dpsi = F_i^{-1}[i xi F_i psi] / n in
// registers, then FP64 partial sums per workgroup.  Direction x (rows) also
// accumulates the density moments and the pointwise Hamiltonian terms.
// partial layout: [sum|psi|^2, sum w|psi|^2, sum x|psi|^2, sum y|psi|^2,
//                  energy re, energy im, non-finite count, 0]
template <typename T, int N, int R, int L, bool COLS, int CPT>
__global__ void __launch_bounds__((CPT == 1 ? 2 : 1) * (N / R) * L)
obs_kernel(ObsParams p) {
    using F = LineFFT<T, N, R, L, COLS, CPT>;
    static_assert(F::NT % 64 == 0, "observable kernels reduce whole waves");
    constexpr int P = F::P;
    __shared__ cpx<T> lds[F::LDS_ELEMS];
    const typename F::Coord c = F::coord(threadIdx.x);
    const int line = xcd_tile(blockIdx.x, gridDim.x) * L + c.l;
    const bool valid = line < p.nlines;
    const T* psi = static_cast<const T*>(p.psi);
    const T* D = static_cast<const T*>(p.D);
    const cpx<T>* tw = static_cast<const cpx<T>*>(p.tw);

    cpx<T> v[CPT][R], old[CPT][R];
    uint32_t idx[R];                                       // of the observable planes
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int pos = c.j + r * P;
        idx[r] = COLS ? (uint32_t)pos * (uint32_t)p.n1 + line : (uint32_t)line * (uint32_t)p.n1 + pos;
        const uint32_t q = COLS ? (uint32_t)pos * (uint32_t)p.pitch + line : (uint32_t)line * (uint32_t)p.pitch + pos;
        if constexpr (CPT == 1) {
            v[0][r] = valid ? load_comp(psi, q, c.comp) : cpx<T>{0, 0};
        } else {
            v[0][r] = v[1][r] = cpx<T>{0, 0};
            if (valid) load_point(psi, q, v[0][r], v[1][r]);
        }
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) old[cc][r] = v[cc][r];
    }
    F::template fft<false>(v, lds, c, tw);
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) v[cc][s] = mul_i(scal(D[c.j + s * P], v[cc][s]));
    F::template fft<true>(v, lds, c, tw);

    // Each carried component adds its share of the sums; the other component
    // (same thread, or the partner lane) enters where the Hamiltonian mixes them.
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            cpx<T> dother, pother;
            if constexpr (CPT == 1) {
                dother = partner(v[0][r]);
                pother = partner(old[0][r]);
            } else {
                dother = v[1 - cc][r];
                pother = old[1 - cc][r];
            }
            const int comp = CPT == 1 ? c.comp : cc;
            if (!valid) continue;
            const double sgn = comp ? -1.0 : 1.0;
            const uint32_t q = idx[r];
            const double pr = old[cc][r].re, pi = old[cc][r].im;   // own component
            const double orr = pother.re, oi = pother.im;          // other component
            const double dr = dother.re, di = dother.im;           // derivative of the other component
            const double w = p.w[q], ca = p.ca[q];
            // conj(own) * D(other)
            const double sr = pr * dr + pi * di, si = pr * di - pi * dr;
            double er, ei;
            if constexpr (!COLS) {
                // -i ca (conj(p0) d1 + conj(p1) d0): this component's term -i ca conj(own) D(other)
                er = ca * si;
                ei = -ca * sr;
                // conj(own) [coef other] with coef = -i (gx - i gy) for component 0 and
                // -i (gx + i gy) for component 1, plus +-V |own|^2
                const double gx = p.gx[q], gy = p.gy[q];
                double V = sgn * p.V[q];
                double ar = -sgn * gy, ai = -gx;
                if (p.ax) {
                    // - e c a fA (A_x sigma_x + A_y sigma_y) - e A0: the other component's
                    // coefficient gains -fA (ax -+ i ay), the diagonal -fV v0
                    ar -= p.fA * p.ax[q];
                    ai += sgn * p.fA * p.ay[q];
                    V -= p.fV * p.v0[q];
                }
                const double tr = ar * orr - ai * oi, ti = ar * oi + ai * orr;
                er += pr * tr + pi * ti;
                ei += pr * ti - pi * tr;
                const double dens = pr * pr + pi * pi;
                er += V * dens;
                const int ix = COLS ? line : c.j + r * P;
                const int iy = COLS ? c.j + r * P : line;
                const double x = -p.a1 + ix * p.h1, y = -p.a2 + iy * p.h2;
                acc[0] += dens;
                acc[1] += w * dens;
                acc[2] += x * dens;
                acc[3] += y * dens;
                acc[6] += (isfinite(pr) && isfinite(pi)) ? 0.0 : 1.0;
            } else {
                // ca (-conj(p0) d1 + conj(p1) d0): this component's term -sgn ca conj(own) D(other)
                er = -sgn * ca * sr;
                ei = -sgn * ca * si;
            }
            acc[4] += w * er;
            acc[5] += w * ei;
        }
    }
    block_sum<F::NT, 8>(acc, p.partials + 8 * (size_t)blockIdx.x);
}

}  // namespace dirac
