// RK stages and their pullbacks on 2D periodic grids, fused with the x passes of
// the pressure solves around them: a workgroup takes a block of rows and does, in
// LDS, what x_inv + stage + x_fwd (or x_inv + reverse stage + x_fwd) did in three
// launches:
//   inverse x FFT of the solved spectrum on the rows of the block and two more on
//   either side -> p; u = w - G p; F(u) on the block and one row before it; the new
//   stage sum; its divergence; forward x FFT -> the spectrum of the next solve.
// Between two of these kernels only the y pass (transform, divide, transform back)
// is left, so a step is 9 launches instead of 17 and a step's pullback 16 instead of
// 29. What bounds it: the launches (4.3 us each on the host) and, in each, one chain of
// LDS phases (load, 2-4 FFT stages, stencil, 2-4 FFT stages, store: 6 us at 64^2,
// about 12 at 256^2) on 16-64 of the 256 CUs; the data is 0.1-4 MB. The rows
// recomputed here (two inverse transforms per row instead of one, 5/4 of the stencil)
// cost less than the launches they replace. 64^2 step 75 -> 63 us, ten 256^2 steps and
// their gradient 4291 -> 4085 us.
//
// The solved spectrum is read with its neighbours' rows while the next one is
// written, so the spectra alternate between two buffers, and so do the fields a
// kernel reads with neighbours and writes. Arithmetic as in the separate kernels
// (divergence and projection in float64).
// Contraction within an expression only: the same bits in every kernel (see k_fft.hpp).
#pragma clang fp contract(on)
#include "k_fft.hpp"

namespace ins {

namespace {

constexpr int kRB = 4;             // rows of a block
constexpr int kRP = kRB + 4;       // rows of p: y0 - 2 .. y0 + kRB + 1 (8 lines: a full power of two)
constexpr int kRU = kRB + 3;       // rows of u: y0 - 2 .. y0 + kRB
constexpr int kRV = kRB + 1;       // rows of the stage sum: y0 - 1 .. y0 + kRB - 1
constexpr int kRNT = 512;           // 256 threads: 256^2 step 107 us, 512: 95, 1024 (spills): 107
constexpr int kRowsMaxNx = 256, kRowsMaxBlocks = 256;
constexpr int kLnlInv = 3, kLsInv = kRP + 1;  // line batches of the two x FFTs and their (odd) strides
constexpr int kLnlFwd = 2, kLsFwd = kRB + 1;

__device__ __forceinline__ int rmod(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// LDS: the FFT lines; p (later the stage sum); u; (reverse stage) the cotangent.
template <typename T>
struct RowsLds {
    cd* line;
    double* p;
    T* v;
    T* u;
    T* f;
    __device__ __forceinline__ explicit RowsLds(unsigned char* mem, int nx) {
        line = reinterpret_cast<cd*>(mem);
        p = reinterpret_cast<double*>(line + (nx / 2) * kLsInv);
        v = reinterpret_cast<T*>(p);  // p is not read any more once v is written
        const size_t pv = max(kRP * sizeof(double), 2 * kRV * sizeof(T)) * nx;
        u = reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(p) + pv);
        f = u + 2 * kRU * nx;
    }
};
template <typename T>
constexpr size_t rows_lds(int nx, bool reverse) {
    const size_t pv = std::max(kRP * sizeof(double), 2 * kRV * sizeof(T));
    return (size_t(kLsInv) * sizeof(cd) / 2 + pv + (reverse ? 4 : 2) * kRU * sizeof(T)) * nx;
}
static_assert(rows_lds<double>(kRowsMaxNx, true) == 94 * 1024, "LDS of the largest row block");

// Inverse x FFT of rows y0 - 2 .. of one field's spectrum into p[row][x]; synchronises.
__device__ __forceinline__ void inverse_rows(const Grid& g, const cd* __restrict__ spec, const FftPlan& X,
                                             const cd* __restrict__ post, cd* line, double* p, int y0) {
    const int M = X.n, nx = g.nx;
    const float rM = __builtin_amdgcn_rcpf(static_cast<float>(M));
    const int total = kRP * M;
    for (int t0 = 0; t0 < total; t0 += 4 * kRNT) {
        cd xk[4], xm[4], wk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = min(t0 + j * kRNT + static_cast<int>(threadIdx.x), total - 1);
            int k;
            const int l = fdivmod(t, M, rM, k);
            const cd* sr = spec + int64_t(rmod(y0 - 2 + l, g.ny)) * g.sx;
            xk[j] = sr[k];
            xm[j] = sr[M - k];
            wk[j] = post[k];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = t0 + j * kRNT + static_cast<int>(threadIdx.x);
            if (t < total) {
                int k;
                const int l = fdivmod(t, M, rM, k);
                const cd xc = cconj(xm[j]);
                const cd e = cadd(xk[j], xc);
                const cd d = csub(xk[j], xc);
                line[k * kLsInv + l] = cmadd(cd{-d.y, d.x}, cconj(wk[j]), e);
            }
        }
    }
    __syncthreads();
    const NoOp nop;
    auto sink = [&](int l, int m, cd z) INS_INLINE { reinterpret_cast<cd*>(p + l * nx)[m] = z; };
    fft_run<1, 8, kRNT, 1, 1, kLineFast, kElemFast>(line, kLnlInv, kLsInv, X, plan_tab<cd>(X), nop, sink, nop, nullptr);
    __syncthreads();
}

// Divergence of v (rows y0 - 1 ..; x component not needed on the first) on the
// block's rows, forward x FFT, half spectrum of the rows that exist.
template <typename T>
__device__ __forceinline__ void forward_rows(const Grid& g, const T* v, const FftPlan& X, const cd* __restrict__ post,
                                             cd* line, cd* __restrict__ spec, int y0) {
    const int M = X.n, nx = g.nx;
    const float rM = __builtin_amdgcn_rcpf(static_cast<float>(M)), rM1 = __builtin_amdgcn_rcpf(static_cast<float>(M + 1));
    for (int t = threadIdx.x; t < kRB * M; t += kRNT) {
        int m;
        const int l = fdivmod(t, M, rM, m);
        const int x0 = 2 * m, xm = x0 == 0 ? nx - 1 : x0 - 1;
        const T* vx = v + (l + 1) * nx;
        const T* vy = v + (kRV + l + 1) * nx;
        const double ux0 = vx[x0], ux1 = vx[x0 + 1];
        double r0 = (ux0 - double(vx[xm])) * g.ih[0];
        double r1 = (ux1 - ux0) * g.ih[0];
        r0 += (double(vy[x0]) - double(vy[x0 - nx])) * g.ih[1];
        r1 += (double(vy[x0 + 1]) - double(vy[x0 + 1 - nx])) * g.ih[1];
        line[m * kLsFwd + l] = cd{r0, r1};
    }
    __syncthreads();
    const NoOp nop;
    fft_run<-1, 8, kRNT, 1, 0, kLineFast, kLineFast>(line, kLnlFwd, kLsFwd, X, plan_tab<cd>(X), nop, nop, nop, nullptr);
    for (int t = threadIdx.x; t < kRB * (M + 1); t += kRNT) {
        int k;
        const int l = fdivmod(t, M + 1, rM1, k);
        if (y0 + l >= g.ny) continue;
        const cd zk = line[(k == M ? 0 : k) * kLsFwd + l];
        const cd zc = cconj(line[(k == 0 ? 0 : M - k) * kLsFwd + l]);
        const cd e = cscale(cadd(zk, zc), 0.5);
        const cd dd = csub(zk, zc);
        const cd o = {0.5 * dd.y, -0.5 * dd.x};
        spec[int64_t(y0 + l) * g.sx + k] = cmadd(post[k], o, e);
    }
}

// Velocity rows in LDS, [component][row][x]; this cell's row and x offsets.
template <typename T>
struct RowSrc {
    const T* u;
    int nx, row;
    int xo[3];
    __device__ __forceinline__ T operator()(int c, const Nb&, int dx, int dy, int) const {
        return u[(c * kRU + row + dy) * nx + xo[dx + 1]];
    }
};

struct RowBlock {
    int b, y0;
    int64_t voff, soff;  // this field's velocity and scalar offsets
    int64_t spoff;       // and spectrum offset
    __device__ __forceinline__ explicit RowBlock(const Grid& g) {
        const int nblk = (g.ny + kRB - 1) / kRB;
        const int id = xcd_logical(blockIdx.x, gridDim.x);
        b = id / nblk;
        y0 = (id - b * nblk) * kRB;
        voff = int64_t(b) * 2 * g.ncell;
        soff = int64_t(b) * g.ncell;
        spoff = int64_t(b) * g.ny * g.sx;
    }
};

}  // namespace

// Stage: u = w - G p (PROJ; p from spec_in) or w; F = F(u);
// yout = (yin ? yin : base) + cy F and wout = base + cw F where given; the spectrum
// of the divergence of wout (yout if there is no wout) -> spec_out. pout, if given,
// receives p. yout may be yin when wout is given (a neighbour's row is then not read).
template <typename T, bool PROJ>
__global__ __launch_bounds__(kRNT) void k_rows_stage(Grid g, FftPlan X, const cd* __restrict__ post,
                                                      const cd* __restrict__ spec_in, cd* __restrict__ spec_out,
                                                      const T* __restrict__ w, const T* __restrict__ base, const T* yin,
                                                      T* yout, T cy, T* __restrict__ wout, T cw, double* __restrict__ pout) {
    extern __shared__ __align__(16) unsigned char rows_smem[];
    const int nx = g.nx, ny = g.ny, nc = int(g.ncell);
    const RowsLds<T> L(rows_smem, nx);
    const RowBlock B(g);
    const float rnx = __builtin_amdgcn_rcpf(static_cast<float>(nx));
    if constexpr (PROJ) inverse_rows(g, spec_in + B.spoff, X, post, L.line, L.p, B.y0);
    for (int t = threadIdx.x; t < kRU * nx; t += kRNT) {
        int x;
        const int r = fdivmod(t, nx, rnx, x);
        const int64_t k = B.voff + int64_t(rmod(B.y0 - 2 + r, ny)) * nx + x;
        const T wx = w[k], wy = w[k + nc];
        if constexpr (PROJ) {
            const double pc = L.p[t];
            L.u[t] = T(double(wx) - (L.p[x + 1 == nx ? t + 1 - nx : t + 1] - pc) * g.ih[0]);
            L.u[kRU * nx + t] = T(double(wy) - (L.p[t + nx] - pc) * g.ih[1]);
            const int y = B.y0 - 2 + r;
            if (pout && r >= 2 && r < 2 + kRB && y < ny) pout[B.soff + int64_t(y) * nx + x] = pc;
        } else {
            L.u[t] = wx;
            L.u[kRU * nx + t] = wy;
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRV * nx; t += kRNT) {
        int x;
        const int r = fdivmod(t, nx, rnx, x);
        const RowSrc<T> U{L.u, nx, r + 1, {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1}};
        T F[2];
        rhs_cell<T, 2>(g, U, Nb{}, F);
        const int y = B.y0 - 1 + r;
        const bool own = r > 0 && y < ny;
        const int64_t k0 = B.voff + int64_t(rmod(y, ny)) * nx + x;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int64_t k = k0 + int64_t(a) * nc;
            const T b0 = base ? base[k] : T(0);
            T v = T(0);
            if (yout && (own || !wout)) {
                v = (yin ? yin[k] : b0) + cy * F[a];
                if (own) yout[k] = v;
            }
            if (wout) {
                v = b0 + cw * F[a];
                if (own) wout[k] = v;
            }
            L.v[(a * kRV + r) * nx + x] = v;
        }
    }
    __syncthreads();
    forward_rows<T>(g, L.v, X, post, L.line, spec_out + B.spoff, B.y0);
}

// u_out = w - G p with p from spec_in (u_out null: only p -> pout).
template <typename T>
__global__ __launch_bounds__(kRNT) void k_rows_project(Grid g, FftPlan X, const cd* __restrict__ post,
                                                        const cd* __restrict__ spec_in, const T* w, T* u_out,
                                                        double* __restrict__ pout) {
    extern __shared__ __align__(16) unsigned char rows_smem[];
    const int nx = g.nx, ny = g.ny, nc = int(g.ncell);
    const RowsLds<T> L(rows_smem, nx);
    const RowBlock B(g);
    const float rnx = __builtin_amdgcn_rcpf(static_cast<float>(nx));
    inverse_rows(g, spec_in + B.spoff, X, post, L.line, L.p, B.y0);
    for (int t = threadIdx.x; t < kRB * nx; t += kRNT) {
        int x;
        const int r = fdivmod(t, nx, rnx, x);
        const int y = B.y0 + r;
        if (y >= ny) continue;
        const int q = t + 2 * nx;
        const double pc = L.p[q];
        if (pout) pout[B.soff + int64_t(y) * nx + x] = pc;
        if (u_out) {
            const int64_t k = B.voff + int64_t(y) * nx + x;
            u_out[k] = T(double(w[k]) - (L.p[x + 1 == nx ? q + 1 - nx : q + 1] - pc) * g.ih[0]);
            u_out[k + nc] = T(double(w[k + nc]) - (L.p[q + nx] - pc) * g.ih[1]);
        }
    }
}

// Reverse stage: q from spec_in, un' = un - G q; the cotangent of F is
// Fbar = cb ybar + cw un' (FIRST: ybar = un', stored to yb_out); u_i = w - G p (p
// null: w); out = J_F(u_i)^T Fbar. u0bar, if given,
//   = (mode 0 or 3 ? ybar : u0bar) + (FIRST ? 0 : un') + (mode 2 or 3 ? out : 0).
// DIV: out -> ubar_out and the spectrum of its divergence -> spec_out.
template <typename T, bool FIRST, bool DIV>
__global__ __launch_bounds__(kRNT) void k_rows_vjp(Grid g, FftPlan X, const cd* __restrict__ post,
                                                    const cd* __restrict__ spec_in, cd* __restrict__ spec_out,
                                                    const T* __restrict__ w, const double* __restrict__ p, const T* ybar,
                                                    const T* __restrict__ un, T cb, T cw, T* u0bar, int mode,
                                                    T* __restrict__ ubar_out, T* __restrict__ yb_out) {
    extern __shared__ __align__(16) unsigned char rows_smem[];
    const int nx = g.nx, ny = g.ny, nc = int(g.ncell);
    const RowsLds<T> L(rows_smem, nx);
    const RowBlock B(g);
    const float rnx = __builtin_amdgcn_rcpf(static_cast<float>(nx));
    inverse_rows(g, spec_in + B.spoff, X, post, L.line, L.p, B.y0);
    for (int t = threadIdx.x; t < kRU * nx; t += kRNT) {
        int x;
        const int r = fdivmod(t, nx, rnx, x);
        const int yr = rmod(B.y0 - 2 + r, ny);
        const int xp = x + 1 == nx ? 0 : x + 1;
        const int64_t k = B.voff + int64_t(yr) * nx + x;
        const double qc = L.p[t];
        const T ux = T(double(un[k]) - (L.p[t - x + xp] - qc) * g.ih[0]);
        const T uy = T(double(un[k + nc]) - (L.p[t + nx] - qc) * g.ih[1]);
        T fx, fy;
        if constexpr (FIRST) {
            fx = cb * ux;
            fy = cb * uy;
        } else {
            fx = cb * ybar[k];
            fy = cb * ybar[k + nc];
            fx += cw * ux;
            fy += cw * uy;
        }
        L.f[t] = fx;
        L.f[kRU * nx + t] = fy;
        T vx = w[k], vy = w[k + nc];
        if (p) {
            const double* pr = p + B.soff + int64_t(yr) * nx;
            const double pc = pr[x];
            vx = T(double(vx) - (pr[xp] - pc) * g.ih[0]);
            vy = T(double(vy) - (pr[x + (yr + 1 == ny ? -(int64_t(ny) - 1) * nx : nx)] - pc) * g.ih[1]);
        }
        L.u[t] = vx;
        L.u[kRU * nx + t] = vy;
        // the projected cotangent at the block's own cells
        const int y = B.y0 - 2 + r;
        if (r >= 2 && r < 2 + kRB && y < ny) {
            if constexpr (FIRST) {
                yb_out[k] = ux;
                yb_out[k + nc] = uy;
            }
            if (u0bar && mode < 2) {
                u0bar[k] = FIRST ? ux : (mode == 0 ? ybar[k] : u0bar[k]) + ux;
                u0bar[k + nc] = FIRST ? uy : (mode == 0 ? ybar[k + nc] : u0bar[k + nc]) + uy;
            }
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRV * nx; t += kRNT) {
        int x;
        const int r = fdivmod(t, nx, rnx, x);
        const int y = B.y0 - 1 + r;
        const bool own = r > 0 && y < ny;
        if (!DIV && !own) continue;
        const RowSrc<T> U{L.u, nx, r + 1, {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1}};
        const RowSrc<T> Fb{L.f, nx, r + 1, {U.xo[0], U.xo[1], U.xo[2]}};
        T out[2];
        rhs_vjp_cell<T, 2>(g, U, Fb, Nb{}, out);
        const int64_t k0 = B.voff + int64_t(y) * nx + x;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if constexpr (DIV) {
                // after the last read of q (the loop above): v shares its space
                L.v[(a * kRV + r) * nx + x] = out[a];
                if (own) ubar_out[k0 + int64_t(a) * nc] = out[a];
            } else {
                const int64_t k = k0 + int64_t(a) * nc;
                // un' again from q, as stored for no one: the last stage only
                const int q = (r + 1) * nx + x;
                const double qn = a == 0 ? L.p[q - x + U.xo[2]] : L.p[q + nx];
                const T up = T(double(un[k]) - (qn - L.p[q]) * g.ih[a]);
                u0bar[k] = (mode == 3 ? ybar[k] : u0bar[k]) + up + out[a];
            }
        }
    }
    if constexpr (DIV) {
        __syncthreads();
        forward_rows<T>(g, L.v, X, post, L.line, spec_out + B.spoff, B.y0);
    }
}

namespace {
int rows_blocks(const Grid& g) { return (g.ny + kRB - 1) / kRB * g.batch; }
}  // namespace

// Whether the row kernels take this field. Its workgroups have to be resident at once,
// one per CU (a second round costs what the launches saved), and its rows short (one
// workgroup's phases grow with them, the separate kernels spread them over the chip).
// Step / pullback in us here against the separate kernels:
//   float64  64^2 63 / 111 vs 75 / 137, 128^2 78 / 138 vs 85 / 150,
//            16 x 64^2 66 / 115 vs 81 / 137, 256^2 98 / 173 vs 99 / 174,
//            256 x 1024 (256 groups) 131 / 251 vs 140 / 263;
//   beyond:  16 x 128^2 (512 groups) 112 / 211 vs 106 / 196, 16 x 256^2 305 / 529 vs
//            236 / 457, 400 x 300 115 / 201 vs 108 / 197, float32 512^2 123 / 235 vs
//            116 / 209.
// At the limit the LDS is 94 KiB and no FFT stage holds more than 8 values per thread.
bool rows2d_ok(const Grid& g) { return g.dim == 2 && g.nx <= kRowsMaxNx && rows_blocks(g) <= kRowsMaxBlocks; }

template <typename T>
hipError_t launch_rows_stage(const Grid& g, const FftPlan& X, const cd* post, const cd* spec_in, cd* spec_out, bool proj,
                             const T* w, const T* base, const T* yin, T* yout, double cy, T* wout, double cw, double* pout,
                             hipStream_t s) {
    const size_t lds = rows_lds<T>(g.nx, false);
    if (proj)
        hipLaunchKernelGGL((k_rows_stage<T, true>), dim3(rows_blocks(g)), dim3(kRNT), lds, s, g, X, post, spec_in, spec_out,
                           w, base, yin, yout, T(cy), wout, T(cw), pout);
    else
        hipLaunchKernelGGL((k_rows_stage<T, false>), dim3(rows_blocks(g)), dim3(kRNT), lds, s, g, X, post, spec_in, spec_out,
                           w, base, yin, yout, T(cy), wout, T(cw), pout);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rows_project(const Grid& g, const FftPlan& X, const cd* post, const cd* spec_in, const T* w, T* u_out,
                               double* pout, hipStream_t s) {
    hipLaunchKernelGGL((k_rows_project<T>), dim3(rows_blocks(g)), dim3(kRNT), rows_lds<T>(g.nx, false), s, g, X, post,
                       spec_in, w, u_out, pout);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rows_vjp(const Grid& g, const FftPlan& X, const cd* post, const cd* spec_in, cd* spec_out, const T* w,
                           const double* p, const T* ybar, const T* un, double cb, double cw, T* u0bar, int mode,
                           T* ubar_out, T* yb_out, hipStream_t s) {
    const size_t lds = rows_lds<T>(g.nx, true);
#define INS_ROWS_VJP(FIRST, DIV)                                                                                       \
    hipLaunchKernelGGL((k_rows_vjp<T, FIRST, DIV>), dim3(rows_blocks(g)), dim3(kRNT), lds, s, g, X, post, spec_in,     \
                       spec_out, w, p, ybar, un, T(cb), T(cw), u0bar, mode, ubar_out, yb_out)
    if (yb_out)
        INS_ROWS_VJP(true, true);
    else if (spec_out)
        INS_ROWS_VJP(false, true);
    else
        INS_ROWS_VJP(false, false);
#undef INS_ROWS_VJP
    return hipGetLastError();
}

#define INS_ROWS(T)                                                                                                      \
    template hipError_t launch_rows_stage<T>(const Grid&, const FftPlan&, const cd*, const cd*, cd*, bool, const T*,     \
                                             const T*, const T*, T*, double, T*, double, double*, hipStream_t);          \
    template hipError_t launch_rows_project<T>(const Grid&, const FftPlan&, const cd*, const cd*, const T*, T*, double*, \
                                               hipStream_t);                                                             \
    template hipError_t launch_rows_vjp<T>(const Grid&, const FftPlan&, const cd*, const cd*, cd*, const T*,             \
                                           const double*, const T*, const T*, double, double, T*, int, T*, T*,           \
                                           hipStream_t);
INS_ROWS(double)
INS_ROWS(float)

}  // namespace ins
