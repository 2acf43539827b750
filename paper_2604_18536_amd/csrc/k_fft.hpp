// Device side of the FFT passes: small DFTs, twiddles, Stockham stages on batches of
// lines in LDS (see k_fft.hip).
//
// A field's bits do not depend on its batch. How many lines a workgroup takes, which
// instance runs and (2D) whether the row kernels do is chosen with the batch in view, and
// the compiler contracts a product and a sum of different statements into an FMA in one
// instance and not in another, or in one copy of an unrolled loop. So wherever a product
// meets a sum here and in k_fft.hip the FMA is written out, and the 2D kernels
// (k_rows2d, k_stencil, k_vjp) contract within an expression only. Cost: the inverse
// strided pass 54.4 -> 56.3 us at 256^3 (its other passes unchanged or 1 % faster, a step
// 2912 -> 2911 us), the 64^2 step 61.7 -> 62.9, ten 256^2 steps and their gradient 4045 -> 4085.
// (With the other product of cmulc in the FMA the inverse strided pass takes 57.0 us.)
#pragma once

#include "k_common.hpp"

namespace ins {

#define INS_INLINE __attribute__((always_inline))

// LDS layout of a batch of `nl` lines of length N: element j of line l lives at
// lds[j * ls + l] with the line stride ls = nl + pad. The plan pads (pad = 1,
// an odd stride, so neighbouring elements of one line fall in different banks)
// whenever the padded batch still fits the LDS budget.

// cos(2 pi j / R), sin(2 pi j / R), correctly rounded.
__device__ __forceinline__ constexpr double kcos(int R, int j) {
    return R == 3 ? (j == 0 ? 1.0 : -0.5)
         : R == 5 ? (j == 0 ? 1.0 : (j == 1 || j == 4) ? 0.30901699437494745 : -0.8090169943749475)
         : /*7*/ (j == 0 ? 1.0 : (j == 1 || j == 6) ? 0.6234898018587335
                            : (j == 2 || j == 5) ? -0.2225209339563144 : -0.9009688679024191);
}
__device__ __forceinline__ constexpr double ksin(int R, int j) {
    return R == 3 ? (j == 0 ? 0.0 : j == 1 ? 0.8660254037844386 : -0.8660254037844386)
         : R == 5 ? (j == 0 ? 0.0 : j == 1 ? 0.9510565162951535 : j == 2 ? 0.5877852522924731
                   : j == 3 ? -0.5877852522924731 : -0.9510565162951535)
         : (j == 0 ? 0.0 : j == 1 ? 0.7818314824680298 : j == 2 ? 0.9749279121818236
            : j == 3 ? 0.4338837391175581 : j == 4 ? -0.4338837391175581
            : j == 5 ? -0.9749279121818236 : -0.7818314824680298);
}

// i * z * sgn
template <int SIGN, class C>
__device__ __forceinline__ C rot(C z) {
    return SIGN < 0 ? C{z.y, -z.x} : C{-z.y, z.x};
}

// Small DFTs X[m] = sum_q x[q] exp(SIGN 2 pi i q m / R), in place.
template <int SIGN, class C>
__device__ __forceinline__ void dft2(C* v) {
    const C a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <int SIGN, class C>
__device__ __forceinline__ void dft4(C& x0, C& x1, C& x2, C& x3) {
    const C s02 = cadd(x0, x2), d02 = csub(x0, x2);
    const C s13 = cadd(x1, x3), d13 = rot<SIGN>(csub(x1, x3));
    x0 = cadd(s02, s13);
    x2 = csub(s02, s13);
    x1 = cadd(d02, d13);
    x3 = csub(d02, d13);
}

template <int SIGN, class C>
__device__ __forceinline__ void dft8(C* v) {
    using F = real_of<C>;
    C e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    C o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<SIGN>(e0, e1, e2, e3);
    dft4<SIGN>(o0, o1, o2, o3);
    constexpr F r = F(0.7071067811865476);
    // w^1 = (1 + SIGN i)/sqrt2, w^2 = SIGN i, w^3 = (-1 + SIGN i)/sqrt2
    const C t1 = {o1.x - SIGN * o1.y, o1.y + SIGN * o1.x};
    const C t2 = rot<SIGN>(o2);
    const C t3 = {-o3.x - SIGN * o3.y, -o3.y + SIGN * o3.x};
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = C{fma(r, t1.x, e1.x), fma(r, t1.y, e1.y)};
    v[5] = C{fma(-r, t1.x, e1.x), fma(-r, t1.y, e1.y)};
    v[2] = cadd(e2, t2);
    v[6] = csub(e2, t2);
    v[3] = C{fma(r, t3.x, e3.x), fma(r, t3.y, e3.y)};
    v[7] = C{fma(-r, t3.x, e3.x), fma(-r, t3.y, e3.y)};
}

// Odd R: pair x[q] with x[R-q]; X[m] = A_m + SIGN i B_m, X[R-m] = A_m - SIGN i B_m with
// A_m = x0 + sum_q (x_q + x_{R-q}) cos(2 pi q m / R), B_m = sum_q (x_q - x_{R-q}) sin(2 pi q m / R).
template <int R, int SIGN, class C>
__device__ __forceinline__ void dft_odd(C* v) {
    using F = real_of<C>;
    constexpr int H = (R - 1) / 2;
    C s[H], d[H];
#pragma unroll
    for (int q = 1; q <= H; ++q) {
        s[q - 1] = cadd(v[q], v[R - q]);
        d[q - 1] = csub(v[q], v[R - q]);
    }
    const C x0 = v[0];
    C sum = x0;
#pragma unroll
    for (int q = 0; q < H; ++q) sum = cadd(sum, s[q]);
    v[0] = sum;
#pragma unroll
    for (int m = 1; m <= H; ++m) {
        C A = x0, B = {F(0), F(0)};
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            const int j = (q * m) % R;
            A.x = fma(s[q - 1].x, F(kcos(R, j)), A.x);
            A.y = fma(s[q - 1].y, F(kcos(R, j)), A.y);
            B.x = fma(d[q - 1].x, F(ksin(R, j)), B.x);
            B.y = fma(d[q - 1].y, F(ksin(R, j)), B.y);
        }
        const C iB = rot<SIGN>(B);
        v[m] = cadd(A, iB);
        v[R - m] = csub(A, iB);
    }
}

template <int R, int SIGN, class C>
__device__ __forceinline__ void dft(C* v) {
    if constexpr (R == 2) dft2<SIGN>(v);
    else if constexpr (R == 4) dft4<SIGN>(v[0], v[1], v[2], v[3]);
    else if constexpr (R == 8) dft8<SIGN>(v);
    else dft_odd<R, SIGN>(v);
}

// q = n / d and r = n % d for 0 <= n < 2^21 and d >= 1, given rd ~ 1/d in float
// to within 2 ulp: the float quotient is then within one unit of the true one,
// and one correction each way makes it exact.
__device__ __forceinline__ int fdivmod(int n, int d, float rd, int& r) {
    int q = static_cast<int>(static_cast<float>(n) * rd);
    r = n - q * d;
    if (r < 0) {
        --q;
        r += d;
    }
    if (r >= d) {
        ++q;
        r -= d;
    }
    return q;
}

// The twiddles of every stage are powers of W_N = exp(-2 pi i / N): stage
// (p, R) multiplies element q of butterfly k by W_N^(q k N / (p R)). Each
// strided-pass workgroup copies the roots W_N^j into LDS once (j < N/2 for
// even N, using W_N^(j + N/2) = -W_N^j; all N for odd N), so no stage issues
// a global load for them. The host tabulates the roots in the precision of C from an exact
// integer angle reduction.
template <class C>
struct Roots {
    const C* t;  // LDS (or the global table, with half = N)
    int half;    // number of stored roots
    __device__ __forceinline__ C operator()(int j) const {
        const C w = t[j < half ? j : j - half];
        return j < half ? w : C{-w.x, -w.y};
    }
    // the twiddles W_N^(q k sN), q = 1 .. R-1, of butterfly k
    struct Cursor {
        const C* t;
        int half, j, ks;
        __device__ __forceinline__ C next() {
            j += ks;
            const C w = t[j < half ? j : j - half];
            return j < half ? w : C{-w.x, -w.y};
        }
    };
    __device__ __forceinline__ Cursor at(int, int k, int, int sN) const { return Cursor{t, half, 0, k * sN}; }
};

// Per-stage twiddle tables in global memory (the x passes, whose element-fast
// stages would read LDS roots with bank conflicts): stage s keeps
// exp(-2 pi i q k / (p R)) at tw[off[s] + k (R - 1) + q - 1].
template <class C>
struct TabTw {
    const C* tw;
    const int* off;
    struct Cursor {
        const C* p;
        __device__ __forceinline__ C next() { return *++p; }
    };
    __device__ __forceinline__ Cursor at(int s, int k, int R, int) const {
        return Cursor{tw + off[s] + k * (R - 1) - 1};
    }
};

// Number of roots a plan of length n keeps in LDS.
__host__ __device__ __forceinline__ int roots_count(int n) { return (n & 1) ? n : n / 2; }

// How the butterflies t = 0 .. S*nl-1 of a stage map to (line l, index i):
// line-fast keeps neighbouring threads on neighbouring lines (contiguous in LDS
// and, for a strided axis, in memory); element-fast keeps them on neighbouring
// elements of one line (contiguous in memory along x).
enum : int { kLineFast = 0, kElemFast = 1 };

template <int MAP>
__device__ __forceinline__ void slot_of(int t, int lnl, int S, float rS, int& l, int& i) {
    if constexpr (MAP == kLineFast) {
        l = t & ((1 << lnl) - 1);
        i = t >> lnl;
    } else {
        l = fdivmod(t, S, rS, i);
    }
}

// One Stockham stage of radix R over the nl lines of length N, p = product of
// the earlier radices. Butterfly (l, i) takes elements i + q S (S = N / R) of
// line l, multiplies element q by exp(SIGN 2 pi i q k / (p R)) with k = i mod p,
// applies DFT_R and produces elements (i - k) R + k + q p. A thread runs
// butterflies t = threadIdx.x + b NTH (NTH threads per workgroup), b < VM / R, in registers.
//   IN  0: inputs from load(l, e) (global memory);  1: from LDS.
//   OUT 0: outputs to LDS, then a barrier;
//       1: outputs handed to sink(l, e, z) (last stage: element i + q S);
//       2: pivot of a forward solve along this axis: every output z of the
//          last forward stage is replaced by divf(l, e, z), and the first stage
//          of the inverse (the same radix, p = 1, so the same butterflies) is
//          applied at once; its outputs i R + q go to LDS when the inverse has
//          more stages (`more`), else to sink.
// The LDS reads of an IN 1 stage that writes LDS are followed by a barrier.
template <int R, int SIGN, int VM, int NTH, int IN, int OUT, int MAP, class C, class TW, class Load, class Sink,
          class Div>
__device__ __forceinline__ void fft_stage(C* __restrict__ lds, int lnl, int ls, int N, int p, int s, const TW& tw,
                                          const Load& load, const Sink& sink, const Div& divf, bool more) {
    constexpr int BMAX = VM / R > 0 ? VM / R : 1;
    const int S = N / R;
    const int sN = S / p;  // exp(2 pi i q k / (p R)) = W_N^(q k sN)
    const int nb = S << lnl;
    const float rS = __builtin_amdgcn_rcpf(static_cast<float>(S));
    const float rp = __builtin_amdgcn_rcpf(static_cast<float>(p));
    C w[BMAX * R];
#pragma unroll
    for (int b = 0; b < BMAX; ++b) {
        const int t = threadIdx.x + b * NTH;
        if (t < nb) {
            int l, i;
            slot_of<MAP>(t, lnl, S, rS, l, i);
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if constexpr (IN == 0) w[b * R + q] = load(l, i + q * S);
                else w[b * R + q] = lds[(i + q * S) * ls + l];
            }
        }
    }
    if constexpr (IN == 1 && OUT != 1) __syncthreads();
#pragma unroll
    for (int b = 0; b < BMAX; ++b) {
        const int t = threadIdx.x + b * NTH;
        if (t < nb) {
            int l, i;
            slot_of<MAP>(t, lnl, S, rS, l, i);
            int k;
            fdivmod(i, p, rp, k);
            C* x = w + b * R;
            if (k != 0) {
                auto cur = tw.at(s, k, R, sN);
#pragma unroll
                for (int q = 1; q < R; ++q) {
                    const C w = cur.next();
                    x[q] = SIGN < 0 ? cmul(x[q], w) : cmulc(x[q], w);
                }
            }
            dft<R, SIGN>(x);
            if constexpr (OUT == 0) {
                const int base = (i - k) * R + k;
#pragma unroll
                for (int q = 0; q < R; ++q) lds[(base + q * p) * ls + l] = x[q];
            } else if constexpr (OUT == 1) {
#pragma unroll
                for (int q = 0; q < R; ++q) sink(l, i + q * S, x[q]);
            } else {
#pragma unroll
                for (int q = 0; q < R; ++q) x[q] = divf(l, i + q * S, x[q]);
                dft<R, -SIGN>(x);
                if (more) {
#pragma unroll
                    for (int q = 0; q < R; ++q) lds[(i * R + q) * ls + l] = x[q];
                } else {
#pragma unroll
                    for (int q = 0; q < R; ++q) sink(l, i * R + q, x[q]);
                }
            }
        }
    }
    if constexpr (OUT == 0 || OUT == 2) {
        if (OUT == 0 || more) __syncthreads();
    }
}

template <int SIGN, int VM, int NTH, int IN, int OUT, int MAP, class C, class TW, class Load, class Sink, class Div>
__device__ __forceinline__ void fft_stage_r(int R, C* lds, int lnl, int ls, int N, int p, int s, const TW& tw,
                                            const Load& load, const Sink& sink, const Div& divf, bool more) {
    switch (R) {
        case 8: fft_stage<8, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
        case 7: fft_stage<7, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
        case 5: fft_stage<5, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
        case 4: fft_stage<4, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
        case 3: fft_stage<3, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
        default: fft_stage<2, SIGN, VM, NTH, IN, OUT, MAP>(lds, lnl, ls, N, p, s, tw, load, sink, divf, more); break;
    }
}

struct NoOp {
    template <class C>
    __device__ C operator()(int, int, C z) const { return z; }
};

// The plan's twiddle table in the precision of C.
__device__ __forceinline__ const cd* plan_tw(const FftPlan& P, cd) { return P.tw; }
__device__ __forceinline__ const cf* plan_tw(const FftPlan& P, cf) { return P.twf; }

// The solve's eigenvalue tables and 1 / #cells in the precision of C.
__device__ __forceinline__ const double* const* solve_lam(const SolveTab& st, cd) { return st.lam; }
__device__ __forceinline__ const float* const* solve_lam(const SolveTab& st, cf) { return st.lamf; }
__device__ __forceinline__ double solve_inv_ncell(const SolveTab& st, cd) { return st.inv_ncell; }
__device__ __forceinline__ float solve_inv_ncell(const SolveTab& st, cf) { return st.inv_ncellf; }

// Every stage of plan P on nl = 2^lnl lines (LDS line stride ls); LDS must be
// free on entry. The first stage reads through `load` with mapping MAP0 (IN0 0)
// or from LDS (IN0 1); stages in between go LDS to LDS, line-fast; the last
// stage, with mapping MAPL (a single stage uses MAP0), writes per OUTL: 0 to
// LDS (element e of line l at lds[e ls + l], synchronised), 1 to sink, 2 as the
// pivot of a solve whose inverse plan is Q (then call fft_inverse_rest).
// The first and last stages are peeled off the loop so that the address
// arithmetic of the memory-facing stages is not kept live across the others.
template <int SIGN, int VM, int NTH, int IN0, int OUTL, int MAP0, int MAPL, class C, class TW, class Load, class Sink,
          class Div>
__device__ __forceinline__ void fft_run(C* lds, int lnl, int ls, const FftPlan& P, const TW& tw, const Load& load,
                                        const Sink& sink, const Div& divf, const FftPlan* Q) {
    const int ns = P.nst;
    const bool more = OUTL == 2 && Q->nst > 1;
    if (ns == 1) {
        fft_stage_r<SIGN, VM, NTH, IN0, OUTL, MAP0>(P.rad[0], lds, lnl, ls, P.n, 1, 0, tw, load, sink, divf, more);
        return;
    }
    fft_stage_r<SIGN, VM, NTH, IN0, 0, MAP0>(P.rad[0], lds, lnl, ls, P.n, 1, 0, tw, load, sink, divf, false);
    int p = P.rad[0];
    for (int st = 1; st < ns - 1; ++st) {
        fft_stage_r<SIGN, VM, NTH, 1, 0, kLineFast>(P.rad[st], lds, lnl, ls, P.n, p, st, tw, load, sink, divf, false);
        p *= P.rad[st];
    }
    fft_stage_r<SIGN, VM, NTH, 1, OUTL, MAPL>(P.rad[ns - 1], lds, lnl, ls, P.n, p, ns - 1, tw, load, sink, divf, more);
}

// The stages of inverse plan Q after a pivot consumed its first one (nothing
// when Q has a single stage): LDS to LDS, the last one to sink (mapping MAPL).
template <int SIGN, int VM, int NTH, int MAPL, class C, class TW, class Sink>
__device__ __forceinline__ void fft_inverse_rest(C* lds, int lnl, int ls, const FftPlan& Q, const TW& tw,
                                                 const Sink& sink) {
    const int ns = Q.nst;
    if (ns == 1) return;
    const NoOp nop;
    int p = Q.rad[0];
    for (int st = 1; st < ns - 1; ++st) {
        fft_stage_r<SIGN, VM, NTH, 1, 0, kLineFast>(Q.rad[st], lds, lnl, ls, Q.n, p, st, tw, nop, sink, nop, false);
        p *= Q.rad[st];
    }
    fft_stage_r<SIGN, VM, NTH, 1, 1, MAPL>(Q.rad[ns - 1], lds, lnl, ls, Q.n, p, ns - 1, tw, nop, sink, nop, false);
}

// Plan P's per-stage twiddle tables in global memory.
template <class C>
__device__ __forceinline__ TabTw<C> plan_tab(const FftPlan& P) {
    return TabTw<C>{plan_tw(P, C{}), P.tw_off};
}

// Copy plan P's roots into LDS at `dst` (synchronised by the caller's next barrier).
template <int NTH, class C>
__device__ __forceinline__ Roots<C> load_roots(C* dst, const FftPlan& P) {
    const C* src = plan_tw(P, C{}) + P.rt_off;
    const int ne = roots_count(P.n);
    for (int j = threadIdx.x; j < ne; j += NTH) dst[j] = src[j];
    return Roots<C>{dst, ne};
}

// Copy the nl lines into LDS element-major (lds[e ls + l]) with element-fast
// threads, so the global reads run along the rows and the LDS writes (odd
// stride ls) are conflict-free; then synchronise. (Along x a first stage that
// read memory directly would write its butterfly outputs i R + q from
// neighbouring threads R elements apart: bank conflicts.)
template <int NTH, class C, class Load>
__device__ __forceinline__ void stage_rows(C* __restrict__ lds, int lnl, int ls, int N, const Load& load) {
    const int nl = 1 << lnl;
    const float rN = __builtin_amdgcn_rcpf(static_cast<float>(N));
    for (int t = threadIdx.x; t < nl * N; t += NTH) {
        int e;
        const int l = fdivmod(t, N, rN, e);
        lds[e * ls + l] = load(l, e);
    }
    __syncthreads();
}

}  // namespace ins
