// Spectral pressure solve of Sec. 2.6.1 on gfx950: p = DFT^-1 L^-1 DFT r with
// the exact discrete transfer function, as a real-to-complex FFT along x
// followed by complex FFTs along y (and z), all hand-written.
//
// Each workgroup moves a batch of whole lines into LDS, runs a Stockham
// autosort FFT of mixed radix (8, 7, 5, 4, 3, 2) on them there (every
// butterfly's inputs are read into registers, a barrier, then its outputs are
// written, so one LDS buffer suffices), and writes the lines back.
//   x pass   : rows of n_x reals, packed as n_x/2 complex values; the
//              divergence of the stage velocity is formed on the fly while
//              loading, so r is never stored.
//   y/z pass : lines of a strided axis; a workgroup takes `lines` adjacent kx
//              so each global access is a contiguous run of `lines` values.
//   last axis: forward FFT, multiply by 1/(L(k) #cells), inverse FFT in the
//              same launch (the spectrum of that axis never leaves LDS).
// The spectral arithmetic runs in the precision of the complex type C: cd
// (float64, every mode but one) or cf (float32, the all-float32 comparison
// mode), with twiddles and eigenvalues tabulated in that precision.
#include "k_fft.hpp"

namespace ins {

// One spectrum value loaded / stored non-temporally (the strided passes over a
// spectrum much larger than the MALL, where no pass can find the previous
// pass's output in it anyway: their short strided runs then stream better).
template <class C>
__device__ __forceinline__ C ld_stream_c(const C* p) {
    return C{__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y)};
}
template <class C>
__device__ __forceinline__ void st_stream_c(C* p, C z) {
    __builtin_nontemporal_store(z.x, &p->x);
    __builtin_nontemporal_store(z.y, &p->y);
}

// Two consecutive values of a row (x even), as one load.
template <class F>
__device__ __forceinline__ void ld_pair(const double* p, F& a, F& b) {
    const double2 t = *reinterpret_cast<const double2*>(p);
    a = F(t.x);
    b = F(t.y);
}
template <class F>
__device__ __forceinline__ void ld_pair(const float* p, F& a, F& b) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    a = t.x;
    b = t.y;
}

// Row staging of the periodic divergence (the x pass's SRC 0): the offsets of
// the rows a batch row reads (u_x; u_y at y and y-1; u_z at z and z-1) are
// formed once per row in LDS, then each thread issues the loads of kXBatch
// values back to back (clamped, branch-free addresses) before it uses any, so
// it waits for memory once per kXBatch values instead of twice per value
// (x forward pass: 0.143 -> 0.125 ms at 256^3, 5.5 -> 4.9 ms at 840^3 with 256
// instead of 1024 threads per workgroup). Writes r[2m] + i r[2m+1] of
// row l to lds[m ls + l] (rows past nrows: 0) and synchronises; at most 16
// rows (the plan's batch limit). Same arithmetic as the per-value load.
constexpr int kXBatch = 4;
struct DivRows {
    int64_t ux, uy, vy, uz, vz;
};
template <typename T, int DIM, int NTH, class C>
__device__ __forceinline__ void stage_div_rows(const Grid& g, const T* __restrict__ vel, C* __restrict__ lds, int lnl,
                                               int ls, int M, int row0, int nrows) {
    using F = real_of<C>;
    __shared__ DivRows rows[16];
    const int nl = 1 << lnl;
    if (static_cast<int>(threadIdx.x) < nl) {
        const int row = min(row0 + static_cast<int>(threadIdx.x), nrows - 1);
        const int yy = row % g.ny, zb = row / g.ny, zz = zb % g.nz, b = zb / g.nz;
        const int64_t base = int64_t(b) * DIM * g.ncell;
        const int ym = yy == 0 ? g.ny - 1 : yy - 1;
        const int zm = zz == 0 ? g.nz - 1 : zz - 1;
        const int64_t r = int64_t(zz * g.ny + yy) * g.nx;
        DivRows d;
        d.ux = base + r;
        d.uy = base + g.ncell + r;
        d.vy = base + g.ncell + int64_t(zz * g.ny + ym) * g.nx;
        d.uz = DIM == 3 ? base + 2 * g.ncell + r : 0;
        d.vz = DIM == 3 ? base + 2 * g.ncell + int64_t(zm * g.ny + yy) * g.nx : 0;
        rows[threadIdx.x] = d;
    }
    __syncthreads();
    const int total = nl * M;
    const float rM = __builtin_amdgcn_rcpf(static_cast<float>(M));
    const F ihx = F(g.ih[0]), ihy = F(g.ih[1]), ihz = F(g.ih[2]);
    for (int t0 = 0; t0 < total; t0 += kXBatch * NTH) {
        F ux0[kXBatch], ux1[kXBatch], uxm[kXBatch], uy0[kXBatch], uy1[kXBatch], vy0[kXBatch], vy1[kXBatch];
        F uz0[kXBatch], uz1[kXBatch], vz0[kXBatch], vz1[kXBatch];
#pragma unroll
        for (int j = 0; j < kXBatch; ++j) {
            const int t = min(t0 + j * NTH + static_cast<int>(threadIdx.x), total - 1);
            int m;
            const int l = fdivmod(t, M, rM, m);
            const DivRows d = rows[l];
            const int x0 = 2 * m, xm = x0 == 0 ? g.nx - 1 : x0 - 1;
            ld_pair(vel + d.ux + x0, ux0[j], ux1[j]);
            uxm[j] = vel[d.ux + xm];
            ld_pair(vel + d.uy + x0, uy0[j], uy1[j]);
            ld_pair(vel + d.vy + x0, vy0[j], vy1[j]);
            if constexpr (DIM == 3) {
                ld_pair(vel + d.uz + x0, uz0[j], uz1[j]);
                ld_pair(vel + d.vz + x0, vz0[j], vz1[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < kXBatch; ++j) {
            const int t = t0 + j * NTH + static_cast<int>(threadIdx.x);
            if (t < total) {
                int m;
                const int l = fdivmod(t, M, rM, m);
                F r0 = (ux0[j] - uxm[j]) * ihx;
                F r1 = (ux1[j] - ux0[j]) * ihx;
                r0 = fma(uy0[j] - vy0[j], ihy, r0);
                r1 = fma(uy1[j] - vy1[j], ihy, r1);
                if constexpr (DIM == 3) {
                    r0 = fma(uz0[j] - vz0[j], ihz, r0);
                    r1 = fma(uz1[j] - vz1[j], ihz, r1);
                }
                lds[m * ls + l] = row0 + l < nrows ? C{r0, r1} : C{F(0), F(0)};
            }
        }
    }
    __syncthreads();
}

// ----------------------------------------------------------------------------
// x pass, forward: real rows (n_x = 2M) -> half spectrum X[0..M].
// Packing: z[m] = x[2m] + i x[2m+1]; Z = FFT_M(z);
// X[k] = (Z[k] + conj Z[M-k]) / 2 + W^k (Z[k] - conj Z[M-k]) / (2i), W = exp(-2 pi i / n_x).
// ----------------------------------------------------------------------------
// SRC 0: rows are the divergence of the velocity field `vel`;
// SRC 1: rows of the float64 scalar field r; SRC 2: rows of component `comp` of vel;
// SRC 3: the channel divergence D u (both wall faces of u^y read as 0, row
// widths from Grid::ym); SRC 4: the channel's D Omega_u^{-1} u (u^y / d_j,
// tangential components / w_j), the right-hand side inside the transposed
// projection.
// The rows are staged in LDS first (see stage_rows); the untangling needs Z[k]
// and Z[M-k] together, so the last stage writes to LDS as well.
template <typename T, int DIM, int SRC, int VM, int NTH, class C = cd>
__global__ __launch_bounds__(NTH) void k_fft_x_fwd(Grid g, const T* __restrict__ vel,
                                                        const real_of<C>* __restrict__ r, C* __restrict__ spec,
                                                        FftPlan P, const C* __restrict__ post, int lnl, int comp) {
    using F = real_of<C>;
    extern __shared__ __align__(16) unsigned char fft_smem[];
    C* lds = reinterpret_cast<C*>(fft_smem);
    const int nl = 1 << lnl;
    const int ls = nl + P.pad;
    const int M = P.n;
    const int nrows = g.batch * g.nz * g.ny;
    const int row0 = xcd_logical(blockIdx.x, gridDim.x) * nl;
    // (y, z, batch) of the first row; row0 + l follows by carrying (l < nl <= 16)
    const int yy0 = row0 % g.ny, zb0 = row0 / g.ny, zz0 = zb0 % g.nz, b0 = zb0 / g.nz;
    auto load = [&](int l, int m) INS_INLINE -> C {
        const int row = row0 + l;
        if (row >= nrows) return C{F(0), F(0)};
        if constexpr (SRC == 1) {
            return reinterpret_cast<const C*>(r + int64_t(row) * g.nx)[m];
        } else {
            int yy = yy0 + l, zz = zz0, b = b0;
            while (yy >= g.ny) {
                yy -= g.ny;
                if (++zz == g.nz) {
                    zz = 0;
                    ++b;
                }
            }
            const int rowoff = (zz * g.ny + yy) * g.nx;
            const int x0 = 2 * m;
            if constexpr (SRC == 2) {
                F a0, a1;
                ld_pair(vel + (int64_t(b) * DIM + comp) * g.ncell + rowoff + x0, a0, a1);
                return C{a0, a1};
            } else if constexpr (SRC >= 3) {
                const T* wb = vel + int64_t(b) * DIM * g.ncell;
                const int S = g.ny + 2;
                const double sp = SRC == 4 ? g.ym[3 * S + yy] : 1.0;  // w_j
                const int xm = x0 == 0 ? g.nx - 1 : x0 - 1;
                double ux0, ux1;
                ld_pair(wb + rowoff + x0, ux0, ux1);
                const double uxm = wb[rowoff + xm];
                double r0 = (ux0 - uxm) * g.ih[0];
                double r1 = (ux1 - ux0) * g.ih[0];
                if constexpr (DIM == 3) {
                    const int zm = zz == 0 ? g.nz - 1 : zz - 1;
                    const T* wz = wb + 2 * g.ncell;
                    double uz0, uz1, vz0, vz1;
                    ld_pair(wz + rowoff + x0, uz0, uz1);
                    ld_pair(wz + (zm * g.ny + yy) * g.nx + x0, vz0, vz1);
                    r0 = fma(uz0 - vz0, g.ih[2], r0);
                    r1 = fma(uz1 - vz1, g.ih[2], r1);
                }
                if constexpr (SRC == 4) {
                    r0 /= sp;
                    r1 /= sp;
                }
                const T* wy = wb + g.ncell;
                double uy0 = 0.0, uy1 = 0.0, vy0 = 0.0, vy1 = 0.0;
                if (yy < g.ny - 1) ld_pair(wy + rowoff + x0, uy0, uy1);
                if (yy > 0) ld_pair(wy + rowoff - g.nx + x0, vy0, vy1);
                double dy0 = uy0 - vy0, dy1 = uy1 - vy1;
                if constexpr (SRC == 4) {
                    const double iu = g.ym[S + yy + 1], id = g.ym[S + yy];  // 1 / d_j, 1 / d_{j-1}
                    dy0 = fma(uy0, iu, -(vy0 * id));
                    dy1 = fma(uy1, iu, -(vy1 * id));
                }
                const double iw = g.ym[yy];
                r0 = fma(dy0, iw, r0);
                r1 = fma(dy1, iw, r1);
                return C{F(r0), F(r1)};
            } else {
                const T* wb = vel + int64_t(b) * DIM * g.ncell;
                const int xm = x0 == 0 ? g.nx - 1 : x0 - 1;
                F ux0, ux1;
                ld_pair(wb + rowoff + x0, ux0, ux1);
                const F uxm = wb[rowoff + xm];
                F r0 = (ux0 - uxm) * F(g.ih[0]);
                F r1 = (ux1 - ux0) * F(g.ih[0]);
                const int ym = yy == 0 ? g.ny - 1 : yy - 1;
                const T* wy = wb + g.ncell;
                F uy0, uy1, vy0, vy1;
                ld_pair(wy + rowoff + x0, uy0, uy1);
                ld_pair(wy + (zz * g.ny + ym) * g.nx + x0, vy0, vy1);
                r0 += (uy0 - vy0) * F(g.ih[1]);
                r1 += (uy1 - vy1) * F(g.ih[1]);
                if constexpr (DIM == 3) {
                    const int zm = zz == 0 ? g.nz - 1 : zz - 1;
                    const T* wz = wb + 2 * g.ncell;
                    F uz0, uz1, vz0, vz1;
                    ld_pair(wz + rowoff + x0, uz0, uz1);
                    ld_pair(wz + (zm * g.ny + yy) * g.nx + x0, vz0, vz1);
                    r0 += (uz0 - vz0) * F(g.ih[2]);
                    r1 += (uz1 - vz1) * F(g.ih[2]);
                }
                return C{r0, r1};
            }
        }
    };
    const NoOp nop;
    const TabTw<C> rt = plan_tab<C>(P);
    if constexpr (SRC == 0)
        stage_div_rows<T, DIM, NTH>(g, vel, lds, lnl, ls, M, row0, nrows);
    else
        stage_rows<NTH>(lds, lnl, ls, M, load);
    fft_run<-1, VM, NTH, 1, 0, kLineFast, kLineFast>(lds, lnl, ls, P, rt, load, nop, nop, nullptr);
    const int M1 = M + 1;
    const float rM1 = __builtin_amdgcn_rcpf(static_cast<float>(M1));
    for (int t = threadIdx.x; t < nl * M1; t += NTH) {
        int k;
        const int l = fdivmod(t, M1, rM1, k);
        const int row = row0 + l;
        if (row >= nrows) continue;
        const C zk = lds[(k == M ? 0 : k) * ls + l];
        const C zc = cconj(lds[(k == 0 ? 0 : M - k) * ls + l]);
        const C e = cscale(cadd(zk, zc), F(0.5));
        const C dd = csub(zk, zc);
        const C o = {F(0.5) * dd.y, F(-0.5) * dd.x};
        spec[int64_t(row) * g.sx + k] = cmadd(post[k], o, e);
    }
}

// Row staging of the inverse x pass, batched like stage_div_rows: the three
// loads of kXBatch values (X[k], X[M-k], W^k) go out back to back, then the
// tangled values Z[k] are formed and written to lds[k ls + l] (rows past
// nrows: 0); synchronises. Same arithmetic as the per-value load.
template <int NTH, class C>
__device__ __forceinline__ void stage_tangled_rows(const Grid& g, const C* __restrict__ spec, const C* __restrict__ post,
                                                   C* __restrict__ lds, int lnl, int ls, int M, int row0, int nrows) {
    const int total = (1 << lnl) * M;
    const float rM = __builtin_amdgcn_rcpf(static_cast<float>(M));
    for (int t0 = 0; t0 < total; t0 += kXBatch * NTH) {
        C xk[kXBatch], xm[kXBatch], wk[kXBatch];
#pragma unroll
        for (int j = 0; j < kXBatch; ++j) {
            const int t = min(t0 + j * NTH + static_cast<int>(threadIdx.x), total - 1);
            int k;
            const int l = fdivmod(t, M, rM, k);
            const C* sr = spec + int64_t(min(row0 + l, nrows - 1)) * g.sx;
            xk[j] = sr[k];
            xm[j] = sr[M - k];
            wk[j] = post[k];
        }
#pragma unroll
        for (int j = 0; j < kXBatch; ++j) {
            const int t = t0 + j * NTH + static_cast<int>(threadIdx.x);
            if (t < total) {
                int k;
                const int l = fdivmod(t, M, rM, k);
                const C xc = cconj(xm[j]);
                const C e = cadd(xk[j], xc);
                // e + i (X[k] - conj X[M-k]) conj(W^k)
                const C d = csub(xk[j], xc);
                const C z = cmadd(C{-d.y, d.x}, cconj(wk[j]), e);
                lds[k * ls + l] = row0 + l < nrows ? z : C{real_of<C>(0), real_of<C>(0)};
            }
        }
    }
    __syncthreads();
}

// x pass, inverse: half spectrum -> real rows, scaled by n_x (unnormalised).
// Z[k] = (X[k] + conj X[M-k]) + i (X[k] - conj X[M-k]) conj(W^k), z = IFFT_M(Z),
// x[2m] = Re z[m], x[2m+1] = Im z[m]. The tangled rows are staged in LDS; the
// last stage writes the real rows directly (element-fast).
template <int VM, int NTH, class C = cd>
__global__ __launch_bounds__(NTH) void k_fft_x_inv(Grid g, const C* __restrict__ spec, real_of<C>* __restrict__ p,
                                                        FftPlan P, const C* __restrict__ post, int lnl) {
    extern __shared__ __align__(16) unsigned char fft_smem[];
    C* lds = reinterpret_cast<C*>(fft_smem);
    const int nl = 1 << lnl;
    const int ls = nl + P.pad;
    const int M = P.n;
    const int nrows = g.batch * g.nz * g.ny;
    const int row0 = xcd_logical(blockIdx.x, gridDim.x) * nl;
    auto sink = [&](int l, int m, C z) INS_INLINE {
        const int row = row0 + l;
        if (row < nrows) reinterpret_cast<C*>(p + int64_t(row) * g.nx)[m] = z;
    };
    const NoOp nop;
    const TabTw<C> rt = plan_tab<C>(P);
    stage_tangled_rows<NTH>(g, spec, post, lds, lnl, ls, M, row0, nrows);
    fft_run<1, VM, NTH, 1, 1, kLineFast, kElemFast>(lds, lnl, ls, P, rt, nop, sink, nop, nullptr);
}

// Strided complex pass along y (axis 1) or z (axis 2) of the half spectrum
// [batch][n_z][n_y][sx] (columns 0 .. n_x/2 in use). MODE 0 forward, 1 inverse, 2 forward + divide +
// inverse. Columns kx < n_x/2 go in chunks of nl adjacent kx per batch (each
// access a contiguous run of nl values); the Nyquist column kx = n_x/2 is taken
// by extra batches, nl lines of it (adjacent values of the other non-x index)
// each, so no batch transforms a chunk that is mostly padding. Either way line
// l of a batch starts at lb0 + l*lstep, has wavenumbers (kx0 + l*kxstep,
// fk0 + l*fkstep) and exists for l < nvalid.
struct LineBatch {
    int64_t lb0, lstep;
    int kx0, kxstep, fk0, fkstep, nvalid;
};

__device__ __forceinline__ LineBatch line_batch(const Grid& g, int axis, int lnl, int w) {
    const int M = g.nx / 2;
    const int nchunk = (M + (1 << lnl) - 1) >> lnl;
    const int nfix = axis == 1 ? g.nz : g.ny;  // the other non-x index
    const int nouter = g.batch * nfix;
    const int64_t plane = int64_t(g.nz) * g.ny * g.sx;                          // one batch entry
    const int64_t fstride = axis == 1 ? int64_t(g.sx) * g.ny : int64_t(g.sx);  // along the other index
    LineBatch B;
    if (w < nchunk * nouter) {
        const int outer = w / nchunk;
        const int b = outer / nfix, f = outer - b * nfix;
        B.kx0 = (w - outer * nchunk) << lnl;
        B.kxstep = 1;
        B.fk0 = f;
        B.fkstep = 0;
        B.lb0 = b * plane + f * fstride + B.kx0;
        B.lstep = 1;
        B.nvalid = M - B.kx0;
    } else {
        const int nfc = (nfix + (1 << lnl) - 1) >> lnl;
        const int j = w - nchunk * nouter;
        const int b = j / nfc;
        const int f0 = (j - b * nfc) << lnl;
        B.kx0 = M;
        B.kxstep = 0;
        B.fk0 = f0;
        B.fkstep = 1;
        B.lb0 = b * plane + f0 * fstride + M;
        B.lstep = fstride;
        B.nvalid = nfix - f0;
    }
    return B;
}

// Number of batches of a strided pass.
__host__ __device__ __forceinline__ int strided_batches(const Grid& g, int axis, int lnl) {
    const int nchunk = (g.nx / 2 + (1 << lnl) - 1) >> lnl;
    const int nfix = axis == 1 ? g.nz : g.ny;
    return nchunk * g.batch * nfix + g.batch * ((nfix + (1 << lnl) - 1) >> lnl);
}

// 1 / a to working precision: the hardware estimate refined by Newton's
// iteration r <- r + r (1 - a r) (each step squares the relative error).
__device__ __forceinline__ double recip(double a) {
    double r = __builtin_amdgcn_rcp(a);
    r = fma(r, fma(-a, r, 1.0), r);
    r = fma(r, fma(-a, r, 1.0), r);
    return fma(r, fma(-a, r, 1.0), r);
}
__device__ __forceinline__ float recip(float a) {
    const float r = __builtin_amdgcn_rcpf(a);
    return fmaf(r, fmaf(-a, r, 1.0f), r);
}

// The eigenvalue sum of the directions other than the line's, for this
// thread's line of batch B (line-fast mapping: a thread's butterflies all lie
// on line threadIdx.x mod nl), and whether those wavenumbers are all zero.
template <class F>
struct LineLam {
    F other;
    bool zero;
};
template <class C>
__device__ __forceinline__ LineLam<real_of<C>> line_lam(const SolveTab& st, const LineBatch& B, int axis, int lnl) {
    const auto* const* lt = solve_lam(st, C{});
    const int l = min(static_cast<int>(threadIdx.x) & ((1 << lnl) - 1), B.nvalid - 1);
    const int kx = B.kx0 + l * B.kxstep, fk = B.fk0 + l * B.fkstep;
    if (axis == 2) return {lt[0][kx] + lt[1][fk], kx == 0 && fk == 0};
    return {lt[0][kx], kx == 0};
}

// One batch of a strided pass per workgroup (NT: non-temporal spectrum access).
template <int MODE, int VM, int NTH, bool NT, class C>
__device__ __forceinline__ void strided_batch(const Grid& g, C* __restrict__ spec, const FftPlan& P, const FftPlan& Q,
                                              int axis, int lnl, const SolveTab& st, int w, C* lds,
                                              const Roots<C>& rt, const real_of<C>* lam_line) {
    using F = real_of<C>;
    const int ls = (1 << lnl) + P.pad;
    const int64_t stride = axis == 1 ? int64_t(g.sx) : int64_t(g.sx) * g.ny;  // along the line
    const LineBatch B = line_batch(g, axis, lnl, w);
    auto load = [&](int l, int e) INS_INLINE -> C {
        if (l >= B.nvalid) return C{F(0), F(0)};
        const C* q = spec + B.lb0 + l * B.lstep + e * stride;
        if constexpr (NT) return ld_stream_c(q);
        else return *q;
    };
    auto store = [&](int l, int e, C z) INS_INLINE {
        if (l >= B.nvalid) return;
        C* q = spec + B.lb0 + l * B.lstep + e * stride;
        if constexpr (NT) st_stream_c(q, z);
        else *q = z;
    };
    const NoOp nop;
    if constexpr (MODE == 1) {
        fft_run<1, VM, NTH, 0, 1, kLineFast, kLineFast>(lds, lnl, ls, P, rt, load, store, nop, nullptr);
    } else if constexpr (MODE == 0) {
        fft_run<-1, VM, NTH, 0, 1, kLineFast, kLineFast>(lds, lnl, ls, P, rt, load, store, nop, nullptr);
    } else {
        // divide by L(k) * #cells; L(0) := 1.
        const LineLam<F> lam = line_lam<C>(st, B, axis, lnl);
        const F inv_ncell = solve_inv_ncell(st, C{});
        auto divide = [&](int l, int e, C z) INS_INLINE -> C {
            if (l >= B.nvalid) return z;
            const F sc = (lam.zero && e == 0) ? inv_ncell : -inv_ncell * recip(lam.other + lam_line[e]);
            C v = cscale(z, sc);
            asm("" : "+v"(v.x), "+v"(v.y));  // a product on its own in every instance
            return v;
        };
        fft_run<-1, VM, NTH, 0, 2, kLineFast, kLineFast>(lds, lnl, ls, P, rt, load, store, divide, &Q);
        fft_inverse_rest<1, VM, NTH, kLineFast>(lds, lnl, ls, Q, rt, store);
    }
}

// First and last stages touch memory directly; in MODE 2 the forward run leaves
// its outputs in registers, they are divided there, and the inverse runs the
// stages in reverse radix order (plan Q, whose first radix is P's last) from
// those same registers. LDS: the line batch, then the roots, then (MODE 2) the
// eigenvalues of the line axis.
template <int MODE, int VM, int NTH, bool NT, class C = cd>
__global__ __launch_bounds__(NTH) void k_fft_strided(Grid g, C* __restrict__ spec, FftPlan P, FftPlan Q, int axis,
                                                          int lnl, SolveTab st) {
    using F = real_of<C>;
    extern __shared__ __align__(16) unsigned char fft_smem[];
    C* lds = reinterpret_cast<C*>(fft_smem);
    const int ls = (1 << lnl) + P.pad;
    const Roots<C> rt = load_roots<NTH>(lds + ls * P.n, P);
    F* lam_line = nullptr;
    if constexpr (MODE == 2) {
        lam_line = reinterpret_cast<F*>(lds + ls * P.n + roots_count(P.n));
        const F* src = solve_lam(st, C{})[axis];
        for (int j = threadIdx.x; j < P.n; j += NTH) lam_line[j] = src[j];
    }
    __syncthreads();  // roots and eigenvalues in LDS before any stage
    strided_batch<MODE, VM, NTH, NT>(g, spec, P, Q, axis, lnl, st, xcd_logical(blockIdx.x, gridDim.x), lds, rt,
                                     lam_line);
}

// ----------------------------------------------------------------------------
// Launchers
// ----------------------------------------------------------------------------
namespace {

template <typename T, class C>
hipError_t fft_x_fwd(const Grid& g, const T* vel, const real_of<C>* r, C* spec, const FftPlan& px, const C* post,
                     int lnl, hipStream_t s, int comp) {
    const int nl = 1 << lnl;
    const int nrows = g.batch * g.nz * g.ny;
    const int nblk = (nrows + nl - 1) / nl;
    const size_t shm = size_t(nl + px.pad) * px.n * sizeof(C);
#define INS_XF(D, SRC, VM, NTH)                                                                                \
    hipLaunchKernelGGL((k_fft_x_fwd<T, D, SRC, VM, NTH, C>), dim3(nblk), dim3(NTH), shm, s, g, vel, r, spec, px, post, \
                       lnl, comp)
#define INS_XF_VM(D, SRC)                                    \
    do {                                                     \
        if (px.nth == 512) INS_XF(D, SRC, 10, 512);          \
        else if (px.vm == 8) INS_XF(D, SRC, 8, 256);         \
        else INS_XF(D, SRC, 16, 256);                        \
    } while (0)
    if (vel && comp < 0) {
        if (g.dim == 3) INS_XF_VM(3, 0); else INS_XF_VM(2, 0);
    } else if (vel) {
        if (g.dim == 3) INS_XF_VM(3, 2); else INS_XF_VM(2, 2);
    } else {
        INS_XF_VM(3, 1);
    }
#undef INS_XF_VM
#undef INS_XF
    return hipGetLastError();
}

template <class C>
hipError_t fft_x_inv(const Grid& g, const C* spec, real_of<C>* p, const FftPlan& px, const C* post, int lnl,
                     hipStream_t s) {
    const int nl = 1 << lnl;
    const int nrows = g.batch * g.nz * g.ny;
    const int nblk = (nrows + nl - 1) / nl;
    const size_t shm = size_t(nl + px.pad) * px.n * sizeof(C);
    if (px.nth == 512)
        hipLaunchKernelGGL((k_fft_x_inv<10, 512, C>), dim3(nblk), dim3(512), shm, s, g, spec, p, px, post, lnl);
    else if (px.vm == 8)
        hipLaunchKernelGGL((k_fft_x_inv<8, 256, C>), dim3(nblk), dim3(256), shm, s, g, spec, p, px, post, lnl);
    else
        hipLaunchKernelGGL((k_fft_x_inv<16, 256, C>), dim3(nblk), dim3(256), shm, s, g, spec, p, px, post, lnl);
    return hipGetLastError();
}

template <class C>
hipError_t fft_strided(const Grid& g, C* spec, const FftPlan& pl, const FftPlan& rev, int axis, int mode, int lnl,
                       const SolveTab& st, hipStream_t s) {
    const int nl = 1 << lnl;
    const int nwork = strided_batches(g, axis, lnl);
    const size_t shm = (size_t(nl + pl.pad) * pl.n + roots_count(pl.n)) * sizeof(C) +
                       (mode == 2 ? size_t(pl.n) * sizeof(real_of<C>) : 0);
    // non-temporal access once the spectrum is well beyond the 256 MB MALL and the
    // batches give 128-byte runs (512^3: y passes 7-10% faster; with the 64-byte
    // runs of 840 lines it changed nothing)
    const bool nt = nl >= 8 && size_t(g.batch) * g.nz * g.ny * g.sx * sizeof(C) > (size_t(512) << 20);
#define INS_ST2(MODE, VM, NTH, NT)                                                                                   \
    hipLaunchKernelGGL((k_fft_strided<MODE, VM, NTH, NT, C>), dim3(nwork), dim3(NTH), shm, s, g, spec, pl, rev, axis, \
                       lnl, st)
#define INS_ST(MODE, VM, NTH)                                            \
    do {                                                                 \
        if (nt) INS_ST2(MODE, VM, NTH, true);                            \
        else INS_ST2(MODE, VM, NTH, false);                              \
    } while (0)
#define INS_ST_VM(MODE)                                                  \
    do {                                                                 \
        if (pl.nth == 512) INS_ST(MODE, 8, 512);                         \
        else if (pl.vm == 8) INS_ST(MODE, 8, 256);                       \
        else INS_ST(MODE, 16, 256);                                      \
    } while (0)
    if (mode == 0)
        INS_ST_VM(0);
    else if (mode == 1)
        INS_ST_VM(1);
    else
        INS_ST_VM(2);
#undef INS_ST_VM
#undef INS_ST
#undef INS_ST2
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_fft_x_fwd(const Grid& g, const T* vel, const double* r, cd* spec, const FftPlan& px, const cd* post,
                            int lnl, hipStream_t s, int comp) {
    return fft_x_fwd<T, cd>(g, vel, r, spec, px, post, lnl, s, comp);
}

hipError_t launch_fft_x_inv(const Grid& g, const cd* spec, double* p, const FftPlan& px, const cd* post, int lnl,
                            hipStream_t s) {
    return fft_x_inv<cd>(g, spec, p, px, post, lnl, s);
}

hipError_t launch_fft_strided(const Grid& g, cd* spec, const FftPlan& pl, const FftPlan& rev, int axis, int mode,
                              int lnl, const SolveTab& st, hipStream_t s) {
    return fft_strided<cd>(g, spec, pl, rev, axis, mode, lnl, st, s);
}

hipError_t launch_fft_x_fwd_f32(const Grid& g, const float* vel, const float* r, cf* spec, const FftPlan& px,
                                const cf* post, int lnl, hipStream_t s) {
    return fft_x_fwd<float, cf>(g, vel, r, spec, px, post, lnl, s, -1);
}

hipError_t launch_fft_x_inv_f32(const Grid& g, const cf* spec, float* p, const FftPlan& px, const cf* post, int lnl,
                                hipStream_t s) {
    return fft_x_inv<cf>(g, spec, p, px, post, lnl, s);
}

hipError_t launch_fft_strided_f32(const Grid& g, cf* spec, const FftPlan& pl, const FftPlan& rev, int axis, int mode,
                                  int lnl, const SolveTab& st, hipStream_t s) {
    return fft_strided<cf>(g, spec, pl, rev, axis, mode, lnl, st, s);
}

template <typename T>
hipError_t launch_fft_x_fwd_wall(const Grid& g, const T* vel, bool scaled, cd* spec, const FftPlan& px, const cd* post,
                                 int lnl, hipStream_t s) {
    const int nl = 1 << lnl;
    const int nrows = g.batch * g.nz * g.ny;
    const int nblk = (nrows + nl - 1) / nl;
    const size_t shm = size_t(nl + px.pad) * px.n * sizeof(cd);
#define INS_XF(D, SRC, VM, NTH)                                                                                \
    hipLaunchKernelGGL((k_fft_x_fwd<T, D, SRC, VM, NTH>), dim3(nblk), dim3(NTH), shm, s, g, vel, nullptr, spec, px, \
                       post, lnl, 0)
#define INS_XF_VM(D, SRC)                                    \
    do {                                                     \
        if (px.nth == 512) INS_XF(D, SRC, 10, 512);          \
        else if (px.vm == 8) INS_XF(D, SRC, 8, 256);         \
        else INS_XF(D, SRC, 16, 256);                        \
    } while (0)
    if (g.dim == 3) {
        if (scaled) INS_XF_VM(3, 4); else INS_XF_VM(3, 3);
    } else {
        if (scaled) INS_XF_VM(2, 4); else INS_XF_VM(2, 3);
    }
#undef INS_XF_VM
#undef INS_XF
    return hipGetLastError();
}

template hipError_t launch_fft_x_fwd_wall<double>(const Grid&, const double*, bool, cd*, const FftPlan&, const cd*,
                                                  int, hipStream_t);
template hipError_t launch_fft_x_fwd_wall<float>(const Grid&, const float*, bool, cd*, const FftPlan&, const cd*, int,
                                                 hipStream_t);
template hipError_t launch_fft_x_fwd<double>(const Grid&, const double*, const double*, cd*, const FftPlan&, const cd*,
                                             int, hipStream_t, int);
template hipError_t launch_fft_x_fwd<float>(const Grid&, const float*, const double*, cd*, const FftPlan&, const cd*,
                                            int, hipStream_t, int);

}  // namespace ins
