// Smagorinsky eddy-viscosity closure (appendix on eddy-viscosity models:
// general framework, eq. smagorinsky) on the uniform periodic staggered grid,
// and its pullback. Every kernel is a gather stencil (one thread per cell, no
// atomics); arithmetic in float64, fields in the context type.
//
// Locations: D_a = delta_a u^a at the pressure point I; G_ab = delta_b u^a on
// the (a, b) edge J + e_a/2 + e_b/2; the velocity gradient at I takes G_ab as
// the mean of the four edges around I; nu_t = (C_s Delta)^2 sqrt(2 S:S) at I;
// nu_t on an edge is the mean of its four pressure points. The term added to
// the a-momentum right-hand side on the a-face I is
//   M^a = (T_aa[I + e_a] - T_aa[I]) / h_a + sum_{b != a} (T_ab[I] - T_ab[I - e_b]) / h_b,
//   T_aa = 2 nu_t D_a (pressure points), T_ab = 2 nu_e (G_ab + G_ba) / 2 (edges),
// i.e. +sum_b delta_b (2 nu_t S_ab): the appendix's sub-grid stress with the
// sign that makes it dissipate energy.
#include "k_common.hpp"
#include "k_zmarch.hpp"

namespace ins {

namespace {

// Velocity component c at the neighbour (dx, dy, dz) (each in -1..1).
template <typename T>
struct Vel {
    const T* __restrict__ u;
    int ncell;
    const Nb& nb;
    __device__ __forceinline__ double operator()(int c, int dx, int dy, int dz) const {
        return double(u[c * ncell + nb.at(dx, dy, dz)]);
    }
};

template <int DIM>
__device__ __forceinline__ void unit(int a, int& x, int& y, int& z) {
    x = a == 0;
    y = a == 1;
    z = (DIM == 3) && a == 2;
}

// delta_a u^a at the pressure point shifted by o.
template <typename V>
__device__ __forceinline__ double diag_at(const V& U, const Grid& g, int a, int ox, int oy, int oz) {
    const int ax = a == 0, ay = a == 1, az = a == 2;
    return (U(a, ox, oy, oz) - U(a, ox - ax, oy - ay, oz - az)) * g.ih[a];
}

// S_ab = (G_ab + G_ba) / 2 on the (a, b) edge J = I + o.
template <typename V>
__device__ __forceinline__ double edge_strain(const V& U, const Grid& g, int a, int b, int ox, int oy, int oz) {
    const int ax = a == 0, ay = a == 1, az = a == 2;
    const int bx = b == 0, by = b == 1, bz = b == 2;
    const double gab = (U(a, ox + bx, oy + by, oz + bz) - U(a, ox, oy, oz)) * g.ih[b];
    const double gba = (U(b, ox + ax, oy + ay, oz + az) - U(b, ox, oy, oz)) * g.ih[a];
    return 0.5 * (gab + gba);
}

// Symmetric strain S at the pressure point I + o (S[a][b], a, b < DIM) and sqrt(2 S:S).
template <int DIM, typename V>
__device__ __forceinline__ double centre_strain(const V& U, const Grid& g, int ox, int oy, int oz, double S[3][3]) {
    double ss = 0.0;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        S[a][a] = diag_at(U, g, a, ox, oy, oz);
        ss += S[a][a] * S[a][a];
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
#pragma unroll
        for (int b = a + 1; b < DIM; ++b) {
            // A_ab at I: mean over the 4 edges = (u^a[I+e_b] - u^a[I-e_b] + u^a[I-e_a+e_b] - u^a[I-e_a-e_b]) / (4 h_b)
            const int ax = a == 0, ay = a == 1, az = a == 2;
            const int bx = b == 0, by = b == 1, bz = b == 2;
            const double aab = 0.25 * g.ih[b] *
                               (U(a, ox + bx, oy + by, oz + bz) - U(a, ox - bx, oy - by, oz - bz) +
                                U(a, ox - ax + bx, oy - ay + by, oz - az + bz) - U(a, ox - ax - bx, oy - ay - by, oz - az - bz));
            const double aba = 0.25 * g.ih[a] *
                               (U(b, ox + ax, oy + ay, oz + az) - U(b, ox - ax, oy - ay, oz - az) +
                                U(b, ox - bx + ax, oy - by + ay, oz - bz + az) - U(b, ox - bx - ax, oy - by - ay, oz - bz - az));
            const double s = 0.5 * (aab + aba);
            S[a][b] = S[b][a] = s;
            ss += 2.0 * s * s;
        }
    }
    return sqrt(2.0 * ss);
}

}  // namespace

// nu[b][I] = c2 sqrt(2 S:S).
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_eddy_nu(Grid g, const T* __restrict__ u, T* __restrict__ nu, double c2) {
    const TileIdx t = tile_of(g);
    if (!t.valid) return;
    const Nb nb = make_nb<DIM>(g, t.x, t.y, t.z);
    const Vel<T> U{u + int64_t(t.b) * DIM * g.ncell, int(g.ncell), nb};
    double S[3][3];
    const double root = centre_strain<DIM>(U, g, 0, 0, 0, S);
    nu[int64_t(t.b) * g.ncell + nb.at(0, 0, 0)] = T(c2 * root);
}

// m = M(u) (overwritten).
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_eddy_term(Grid g, const T* __restrict__ u, const T* __restrict__ nu,
                                                        T* __restrict__ m) {
    const TileIdx t = tile_of(g);
    if (!t.valid) return;
    const Nb nb = make_nb<DIM>(g, t.x, t.y, t.z);
    const int64_t boff = int64_t(t.b) * DIM * g.ncell;
    const Vel<T> U{u + boff, int(g.ncell), nb};
    const T* nub = nu + int64_t(t.b) * g.ncell;
    auto N = [&](int dx, int dy, int dz) { return double(nub[nb.at(dx, dy, dz)]); };
    const int c0 = nb.at(0, 0, 0);
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        int ax, ay, az;
        unit<DIM>(a, ax, ay, az);
        double acc = (2.0 * N(ax, ay, az) * diag_at(U, g, a, ax, ay, az) - 2.0 * N(0, 0, 0) * diag_at(U, g, a, 0, 0, 0)) *
                     g.ih[a];
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            if (b == a) continue;
            int bx, by, bz;
            unit<DIM>(b, bx, by, bz);
            // edges J = I and J = I - e_b
            const double nu0 = 0.25 * (N(0, 0, 0) + N(ax, ay, az) + N(bx, by, bz) + N(ax + bx, ay + by, az + bz));
            const double nu1 = 0.25 * (N(-bx, -by, -bz) + N(ax - bx, ay - by, az - bz) + N(0, 0, 0) + N(ax, ay, az));
            const double t0 = 2.0 * nu0 * edge_strain(U, g, a, b, 0, 0, 0);
            const double t1 = 2.0 * nu1 * edge_strain(U, g, a, b, -bx, -by, -bz);
            acc += (t0 - t1) * g.ih[b];
        }
        m[boff + a * g.ncell + c0] = T(acc);
    }
}

// RK stage with the eddy-viscosity term on 3D grids, one z-march: the stage velocity
// u = w - G p (PROJ; float64 projection) is formed once per plane on the tile plus two
// cells in an LDS ring, nu_t of plane z + 1 once on the tile plus one cell, and plane z
// then takes F(u) + M(u) from LDS only. Streams (PT, YW) and update as in k_stage_zm:
//   y = (yinit ? u0 : y, or with YW u0 + ry (wprev - u0) + rw (w - u0)) + cy (F + M),
//   wout = u0 + cw (F + M), each where given.
// The stress on the z edges below a plane and T_zz are carried from the plane before.
// The projection, nu_t, M and stage kernels it replaces moved 1.3 GB per stage of
// 4 x 128^3 float32 cells through memory (382 us), this one 0.57-0.67 GB (160-179 us,
// 3.7 TB/s): about 230 float64 operations per cell (50 us at the card's rate) and two
// barriers per plane at 16 waves per CU are not fully overlapped with the loads. A step
// 2631 -> 1840 us, float64 at 128^3 982 -> 564 us.
// All loads of the plane loop are unconditional, as in k_stage_zm.
template <typename T, int HX, int HP>
struct EddyRing {
    const T *zm, *z0, *zp;  // ring slots of the planes below, at and above
    int centre;
    __device__ __forceinline__ double operator()(int c, int dx, int dy, int dz) const {
        return double((dz < 0 ? zm : (dz > 0 ? zp : z0))[c * HP + centre + dy * HX + dx]);
    }
    __device__ __forceinline__ T operator()(int c, const Nb&, int dx, int dy, int dz) const {
        return (dz < 0 ? zm : (dz > 0 ? zp : z0))[c * HP + centre + dy * HX + dx];
    }
};

template <typename T, bool PROJ, int TX, int TY, bool YW, int PT>
__global__ __launch_bounds__(TX * TY) void k_eddy_stage_zm(Grid g, const T* __restrict__ w, const double* __restrict__ p,
                                                             const T* __restrict__ u0, T* __restrict__ y, int yinit, T cy,
                                                             T* wout, T cw, int zc, double c2, const T* wprev, T ry, T rw) {
    constexpr int NT = TX * TY, HX = TX + 4, HP = HX * (TY + 4), NX = TX + 2, NP = NX * (TY + 2), NR = 5;
    constexpr int NS = (HP + NT - 1) / NT, NN = (NP + NT - 1) / NT;
    constexpr bool LB = (PT & 1) != 0, LY = (PT & 2) != 0;
    __shared__ T ring[NR][3 * HP];
    __shared__ T nu[2][NP];
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY, nzc = (nz + zc - 1) / zc;
    int L = xcd_logical(blockIdx.x, gridDim.x);
    const int tx = L % ntx;
    L /= ntx;
    const int ty = L % nty;
    L /= nty;
    const int zci = L % nzc;
    const int b = L / nzc;
    const int x0 = tx * TX, y0 = ty * TY, z0 = zci * zc;
    const int z1 = min(z0 + zc, nz);
    const int64_t boff = int64_t(b) * 3 * g.ncell;
    const T* wb = w + boff;
    const double* pb = PROJ ? p + int64_t(b) * g.ncell : nullptr;
    const int nc = int(g.ncell);
    const int plane = nx * ny;

    // halo-plane positions loaded by this thread (slots past the halo load the
    // first position and are not parked)
    int hxy[NS], hxp[NS], hyp[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int q = threadIdx.x + s * NT;
        const int qq = q < HP ? q : 0;
        const int gx = pmod(x0 - 2 + qq % HX, nx);
        const int gy = pmod(y0 - 2 + qq / HX, ny);
        hxy[s] = gy * nx + gx;
        hxp[s] = gy * nx + (gx + 1 == nx ? 0 : gx + 1);
        hyp[s] = (gy + 1 == ny ? 0 : gy + 1) * nx + gx;
    }
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int cxg = x0 + lx, cyg = y0 + ly;
    const bool valid = cxg < nx && cyg < ny;
    const int cxy = min(cyg, ny - 1) * nx + min(cxg, nx - 1);
    const int centre = (ly + 2) * HX + (lx + 2);
    const int ncen = (ly + 1) * NX + (lx + 1);

    T vw[NS][3];
    double vp[NS][4];
    auto fetch = [&](int zz) {
        const int zoff = zz * plane;
        const int zpo = (zz + 1 == nz ? 0 : zz + 1) * plane;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int j = zoff + hxy[s];
            vw[s][0] = wb[j];
            vw[s][1] = wb[nc + j];
            vw[s][2] = wb[2 * nc + j];
            if constexpr (PROJ) {
                vp[s][0] = pb[j];
                vp[s][1] = pb[zoff + hxp[s]];
                vp[s][2] = pb[zoff + hyp[s]];
                vp[s][3] = pb[zpo + hxy[s]];
            }
        }
    };
    auto park = [&](T* slot) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int q = threadIdx.x + s * NT;
            if (q < HP) {
                if constexpr (PROJ) {
                    const double pc = vp[s][0];
                    slot[q] = T(double(vw[s][0]) - (vp[s][1] - pc) * g.ih[0]);
                    slot[HP + q] = T(double(vw[s][1]) - (vp[s][2] - pc) * g.ih[1]);
                    slot[2 * HP + q] = T(double(vw[s][2]) - (vp[s][3] - pc) * g.ih[2]);
                } else {
                    slot[q] = vw[s][0];
                    slot[HP + q] = vw[s][1];
                    slot[2 * HP + q] = vw[s][2];
                }
            }
        }
    };
    auto viscosity = [&](const T* zm, const T* zc0, const T* zp, T* out) {
#pragma unroll 1
        for (int s = 0; s < NN; ++s) {
            const int q = threadIdx.x + s * NT;
            if (q < NP) {
                const int qy = q / NX;
                const EddyRing<T, HX, HP> U{zm, zc0, zp, (qy + 1) * HX + (q - qy * NX) + 1};
                double S[3][3];
                out[q] = T(c2 * centre_strain<3>(U, g, 0, 0, 0, S));
            }
        }
    };
    constexpr bool WPT = YW;
    T pbase[3] = {T(0), T(0), T(0)}, pyv[3] = {T(0), T(0), T(0)}, pwc[3] = {T(0), T(0), T(0)};
    const T* ysrc = YW ? wprev : y;
    auto fetch_point = [&](int z) {
        const int c0 = z * plane + cxy;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int64_t kk = boff + int64_t(a) * nc + c0;
            if constexpr (LB) pbase[a] = ld_stream(u0 + kk);
            if constexpr (LY) pyv[a] = ld_stream(ysrc + kk);
            if constexpr (WPT) pwc[a] = wb[int64_t(a) * nc + c0];
        }
    };

    // planes z0 - 2 .. z0 + 1 parked, nu_t of z0 - 1; then plane z0 - 1 runs through the
    // loop without output (the stresses it leaves are carried into z0)
    T *s0 = ring[0], *s1 = ring[1], *s2 = ring[2], *s3 = ring[3], *s4 = ring[4];  // planes z - 1 .. z + 3
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
        fetch(pmod(z0 - 2 + k, nz));
        park(ring[k]);
    }
    T *n0 = nu[0], *n1 = nu[1];
    __syncthreads();
    viscosity(s0, s1, s2, n0);
    double txz_m = 0.0, tyz_m = 0.0, tzz0 = 0.0;
    for (int z = z0 - 1; z < z1; ++z) {
        fetch(pmod(min(z + 3, z1 + 1), nz));
        viscosity(s1, s2, s3, n1);
        __syncthreads();  // nu_t of z + 1 is read below
        const EddyRing<T, HX, HP> U{s0, s1, s2, centre};
        auto N = [&](int dx, int dy, int dz) { return double((dz ? n1 : n0)[ncen + dy * NX + dx]); };
        // 4 T_ab on the (a, b) edge I + o (the factors 2 nu_e and S_ab hold powers of two)
        auto edge = [&](int a, int b2, int ox, int oy, int oz) {
            const int ax = a == 0, ay = a == 1, az = a == 2;
            const int bx = b2 == 0, by = b2 == 1, bz = b2 == 2;
            const double gab = (U(a, ox + bx, oy + by, oz + bz) - U(a, ox, oy, oz)) * g.ih[b2];
            const double gba = (U(b2, ox + ax, oy + ay, oz + az) - U(b2, ox, oy, oz)) * g.ih[a];
            return (N(ox, oy, oz) + N(ox + ax, oy + ay, oz + az) + N(ox + bx, oy + by, oz + bz) +
                    N(ox + ax + bx, oy + ay + by, oz + az + bz)) *
                   (gab + gba);
        };
        // T_aa / 2 at the pressure point I + e_a or I
        auto diag = [&](int a, int o) {
            const int ax = a == 0, ay = a == 1, az = a == 2;
            return N(o * ax, o * ay, o * az) * diag_at(U, g, a, o * ax, o * ay, o * az);
        };
        const double txz = edge(0, 2, 0, 0, 0), tyz = edge(1, 2, 0, 0, 0), tzz1 = diag(2, 1);
        if (z >= z0) {
            const double txy = edge(0, 1, 0, 0, 0);
            double M[3];
            M[0] = 2.0 * (diag(0, 1) - diag(0, 0)) * g.ih[0] + 0.25 * (txy - edge(0, 1, 0, -1, 0)) * g.ih[1] +
                   0.25 * (txz - txz_m) * g.ih[2];
            M[1] = 2.0 * (diag(1, 1) - diag(1, 0)) * g.ih[1] + 0.25 * (txy - edge(0, 1, -1, 0, 0)) * g.ih[0] +
                   0.25 * (tyz - tyz_m) * g.ih[2];
            M[2] = 2.0 * (tzz1 - tzz0) * g.ih[2] + 0.25 * (txz - edge(0, 2, -1, 0, 0)) * g.ih[0] +
                   0.25 * (tyz - edge(1, 2, 0, -1, 0)) * g.ih[1];
            T F[3];
            rhs_cell<T, 3>(g, U, Nb{}, F);
            if (valid) {
                const int c0 = z * plane + cyg * nx + cxg;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int64_t kk = boff + int64_t(a) * nc + c0;
                    const T base = LB ? pbase[a] : T(0);
                    T yv;
                    if constexpr (YW) yv = base + ry * (pyv[a] - base) + rw * (pwc[a] - base);
                    else if constexpr (LY) yv = pyv[a];
                    else yv = base;
                    F[a] += T(M[a]);
                    if (y) st_stream(yv + cy * F[a], y + kk);
                    if (wout) st_stream(base + cw * F[a], wout + kk);
                }
            }
        }
        txz_m = txz;
        tyz_m = tyz;
        tzz0 = tzz1;
        fetch_point(min(z + 1, z1 - 1));
        park(s4);
        T* sf = s0;
        s0 = s1;
        s1 = s2;
        s2 = s3;
        s3 = s4;
        s4 = sf;
        T* nf = n0;
        n0 = n1;
        n1 = nf;
        __syncthreads();
    }
}

// Pullback, first pass (pressure points): with tbar_aa = (mbar^a[I - e_a] - mbar^a[I]) / h_a
// and, on each (a, b) edge J, tbar_ab = (mbar^a[J] - mbar^a[J + e_b]) / h_b,
//   nubar[I] = sum_a 2 tbar_aa D_a + sum_{a<b} 1/4 sum_{4 edges J around I} 2 S_ab[J] (tbar_ab + tbar_ba)[J],
//   g = c2 nubar / sqrt(2 S:S) (0 where S = 0), P_ab[I] = 2 g S_ab[I] (symmetric, a <= b),
// the cotangent of the centre velocity gradient. P is stored as DIM (DIM + 1) / 2
// planar fields per batch entry, ordered (0,0), (1,1), [(2,2),] (0,1), [(0,2), (1,2)].
template <int DIM>
__device__ __forceinline__ int pidx(int a, int b) {
    if (a == b) return a;
    if (a > b) {
        const int t = a;
        a = b;
        b = t;
    }
    return DIM == 2 ? 2 : (a == 0 ? (b == 1 ? 3 : 4) : 5);
}

template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_eddy_vjp_centre(Grid g, const T* __restrict__ u, const T* __restrict__ mbar,
                                                              T* __restrict__ P, double c2) {
    const TileIdx t = tile_of(g);
    if (!t.valid) return;
    constexpr int NP = DIM * (DIM + 1) / 2;
    const Nb nb = make_nb<DIM>(g, t.x, t.y, t.z);
    const int64_t boff = int64_t(t.b) * DIM * g.ncell;
    const Vel<T> U{u + boff, int(g.ncell), nb};
    const Vel<T> MB{mbar + boff, int(g.ncell), nb};
    double S[3][3];
    const double root = centre_strain<DIM>(U, g, 0, 0, 0, S);
    double nubar = 0.0;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        int ax, ay, az;
        unit<DIM>(a, ax, ay, az);
        const double tbar = (MB(a, -ax, -ay, -az) - MB(a, 0, 0, 0)) * g.ih[a];
        nubar += 2.0 * tbar * S[a][a];
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
#pragma unroll
        for (int b = a + 1; b < DIM; ++b) {
            int ax, ay, az, bx, by, bz;
            unit<DIM>(a, ax, ay, az);
            unit<DIM>(b, bx, by, bz);
            double e = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {  // edges J = I - (k & 1) e_a - (k >> 1) e_b
                const int ox = -(k & 1) * ax - (k >> 1) * bx;
                const int oy = -(k & 1) * ay - (k >> 1) * by;
                const int oz = -(k & 1) * az - (k >> 1) * bz;
                const double tab = (MB(a, ox, oy, oz) - MB(a, ox + bx, oy + by, oz + bz)) * g.ih[b];
                const double tba = (MB(b, ox, oy, oz) - MB(b, ox + ax, oy + ay, oz + az)) * g.ih[a];
                e += edge_strain(U, g, a, b, ox, oy, oz) * (tab + tba);
            }
            nubar += 0.5 * e;  // 1/4 * 2
        }
    }
    const double gg = root > 0.0 ? c2 * nubar / root : 0.0;
    const int c0 = nb.at(0, 0, 0);
    T* pb = P + int64_t(t.b) * NP * g.ncell;
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int b = a; b < DIM; ++b) pb[pidx<DIM>(a, b) * g.ncell + c0] = T(2.0 * gg * S[a][b]);
}

// Pullback, second pass (faces): ubar^a[I] += (Dbar_a[I] - Dbar_a[I + e_a]) / h_a
//   + sum_{b != a} (Gbar_ab[I - e_b] - Gbar_ab[I]) / h_b, with
//   Dbar_a[K] = 2 tbar_aa[K] nu[K] + P_aa[K],
//   Gbar_ab[J] = nu_e[J] (tbar_ab + tbar_ba)[J] + 1/4 sum_{4 pressure points around J} P_ab.
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_eddy_vjp_face(Grid g, const T* __restrict__ nu, const T* __restrict__ mbar,
                                                            const T* __restrict__ P, T* __restrict__ ubar) {
    const TileIdx t = tile_of(g);
    if (!t.valid) return;
    constexpr int NP = DIM * (DIM + 1) / 2;
    const Nb nb = make_nb<DIM>(g, t.x, t.y, t.z);
    const int64_t boff = int64_t(t.b) * DIM * g.ncell;
    const Vel<T> MB{mbar + boff, int(g.ncell), nb};
    const T* nub = nu + int64_t(t.b) * g.ncell;
    const T* pb = P + int64_t(t.b) * NP * g.ncell;
    auto N = [&](int dx, int dy, int dz) { return double(nub[nb.at(dx, dy, dz)]); };
    auto PP = [&](int k, int dx, int dy, int dz) { return double(pb[k * g.ncell + nb.at(dx, dy, dz)]); };
    const int c0 = nb.at(0, 0, 0);
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        int ax, ay, az;
        unit<DIM>(a, ax, ay, az);
        auto dbar = [&](int ox, int oy, int oz) {
            const double tbar = (MB(a, ox - ax, oy - ay, oz - az) - MB(a, ox, oy, oz)) * g.ih[a];
            return 2.0 * tbar * N(ox, oy, oz) + PP(a, ox, oy, oz);
        };
        double acc = (dbar(0, 0, 0) - dbar(ax, ay, az)) * g.ih[a];
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            if (b == a) continue;
            int bx, by, bz;
            unit<DIM>(b, bx, by, bz);
            const int k = pidx<DIM>(a, b);
            auto gbar = [&](int ox, int oy, int oz) {  // on the (a, b) edge J = I + o
                const double nue = 0.25 * (N(ox, oy, oz) + N(ox + ax, oy + ay, oz + az) + N(ox + bx, oy + by, oz + bz) +
                                           N(ox + ax + bx, oy + ay + by, oz + az + bz));
                const double tab = (MB(a, ox, oy, oz) - MB(a, ox + bx, oy + by, oz + bz)) * g.ih[b];
                const double tba = (MB(b, ox, oy, oz) - MB(b, ox + ax, oy + ay, oz + az)) * g.ih[a];
                const double pav = 0.25 * (PP(k, ox, oy, oz) + PP(k, ox + ax, oy + ay, oz + az) +
                                           PP(k, ox + bx, oy + by, oz + bz) + PP(k, ox + ax + bx, oy + ay + by, oz + az + bz));
                return nue * (tab + tba) + pav;
            };
            acc += (gbar(-bx, -by, -bz) - gbar(0, 0, 0)) * g.ih[b];
        }
        T* dst = ubar + boff + a * g.ncell + c0;
        *dst = T(double(*dst) + acc);
    }
}

#define INS_EDDY_DISPATCH(g, KER, ...)                                                     \
    do {                                                                                   \
        const int nblk = stencil_blocks(g);                                                \
        if ((g).dim == 3)                                                                  \
            hipLaunchKernelGGL((KER<T, 3>), dim3(nblk), dim3(kBlock), 0, s, __VA_ARGS__);  \
        else                                                                               \
            hipLaunchKernelGGL((KER<T, 2>), dim3(nblk), dim3(kBlock), 0, s, __VA_ARGS__);  \
    } while (0)

template <typename T>
hipError_t launch_eddy_forward(const Grid& g, const T* u, T* nu, T* m, double c2, hipStream_t s) {
    INS_EDDY_DISPATCH(g, k_eddy_nu, g, u, nu, c2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    INS_EDDY_DISPATCH(g, k_eddy_term, g, u, nu, m);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_eddy_backward(const Grid& g, const T* u, const T* nu, const T* mbar, T* P, T* ubar, double c2,
                                hipStream_t s) {
    INS_EDDY_DISPATCH(g, k_eddy_vjp_centre, g, u, mbar, P, c2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    INS_EDDY_DISPATCH(g, k_eddy_vjp_face, g, nu, mbar, P, ubar);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_eddy_viscosity(const Grid& g, const T* u, T* nu, double c2, hipStream_t s) {
    INS_EDDY_DISPATCH(g, k_eddy_nu, g, u, nu, c2);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_eddy_stage_zm(const Grid& g, const T* w, const double* p, bool proj, const T* u0, T* y, bool yinit,
                                double cy, T* wout, double cw, double c2, const T* wprev, double ry, double rw,
                                hipStream_t s) {
    // 54 KB (64 x 8 float32) and 57 KB (32 x 8 float64) of LDS: two workgroups per CU and
    // more; 64 x 8 in float64 would hold one.
    constexpr int TX = sizeof(T) == 8 ? 32 : 64, TY = 8;
    const int pt = ((wout || yinit) ? 1 : 0) | ((y && !yinit) ? 2 : 0);
#define INS_ESZM(PR, YWI, PTI)                                                                                       \
    do {                                                                                                             \
        constexpr auto kern = &k_eddy_stage_zm<T, PR, TX, TY, YWI, PTI>;                                             \
        const int zc = zm_chunk(g, TX, TY, resident_groups<kern, TX * TY>(), 64);                                    \
        const int nblk = ((g.nx + TX - 1) / TX) * ((g.ny + TY - 1) / TY) * ((g.nz + zc - 1) / zc) * g.batch;         \
        hipLaunchKernelGGL((k_eddy_stage_zm<T, PR, TX, TY, YWI, PTI>), dim3(nblk), dim3(TX * TY), 0, s, g, w, p, u0, \
                           y, yinit ? 1 : 0, T(cy), wout, T(cw), zc, c2, wprev, T(ry), T(rw));                       \
    } while (0)
    if (wprev)
        INS_ESZM(true, true, 3);
    else if (pt == 3)
        return hipErrorInvalidValue;  // no schedule reads both u0 and y otherwise
    else if (!proj)
        INS_ESZM(false, false, 1);
    else if (pt == 2)
        INS_ESZM(true, false, 2);
    else
        INS_ESZM(true, false, 1);
#undef INS_ESZM
    return hipGetLastError();
}

#undef INS_EDDY_DISPATCH

template hipError_t launch_eddy_forward<double>(const Grid&, const double*, double*, double*, double, hipStream_t);
template hipError_t launch_eddy_forward<float>(const Grid&, const float*, float*, float*, double, hipStream_t);
template hipError_t launch_eddy_backward<double>(const Grid&, const double*, const double*, const double*, double*,
                                                 double*, double, hipStream_t);
template hipError_t launch_eddy_backward<float>(const Grid&, const float*, const float*, const float*, float*, float*,
                                                double, hipStream_t);

#define INS_EDDY_STAGE(T)                                                                                                \
    template hipError_t launch_eddy_viscosity<T>(const Grid&, const T*, T*, double, hipStream_t);                        \
    template hipError_t launch_eddy_stage_zm<T>(const Grid&, const T*, const double*, bool, const T*, T*, bool, double,  \
                                                T*, double, double, const T*, double, double, hipStream_t);
INS_EDDY_STAGE(double)
INS_EDDY_STAGE(float)
#undef INS_EDDY_STAGE

}  // namespace ins
