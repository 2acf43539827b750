// Conjugate-gradient solve of one field in one launch (channel and stretched
// grids whose field fits on the chip): the residual, the solution, A p and the
// operator's coefficients of a workgroup's block of cells live in registers, the
// search direction with a one-cell halo in LDS, for all iterations.
//
// Why: a 4096-cell field took two launches of 5-6 us per iteration, a 238k-cell
// field 13 + 10 us, for 0.1-6 MB of data: launch, fill and drain, and every
// workgroup's re-reduction of the partial sums. What bounds it here is latency:
// that of the sums, and of the stencil's LDS reads at 2 waves per SIMD. Per iteration
// (two kernels -> one launch): 64^2 11.5 -> 1.6 us, 128^2 12 -> 2.7, 33 x 32 x 32 13.3 ->
// 3.0, 70 x 63 x 54 23 -> 5.65, the channel 66 x 81 x 48 24 -> 6.0, 79^3 26 -> 10 us.
//
// One workgroup (fields of at most 4096 cells): the recurrence, stop test and sums
// of k_cg.hpp, two sums per iteration. Several workgroups: one exchange per
// iteration instead of two. p.q, r.q, q.q and r.r are summed together and the
// boundary of q = A p travels with them (the halo's r and p follow the recurrence
// locally); beta needs rr_{k+1} before it is summed and takes
// |r - alpha q|^2 = rr_k - 2 alpha r.q + alpha^2 q.q, while alpha and the stop test
// use the summed r.r, one exchange later. The split depends on the field's sizes
// alone, so a field of a batch gives bitwise what it gives alone.
//
// Between workgroups. Every value that crosses workgroups (a partial sum, a
// boundary value of A p) is one double sent as two 64-bit words {half, tag},
// written and polled with device scope: a reader that sees the tag of the
// iteration it waits for has the half that came with it, so no fence,
// cache write-back or barrier counter is needed (a device-scope fence writes back
// an XCD's L2). Tags count up within a launch, from slots zeroed by the launch
// before. Even and odd iterations have slots of their own: those of iteration k
// are rewritten in iteration k + 2, after the sums of iteration k + 1, which every
// reader of the old values has entered by then.
//
// The fields of a batch run side by side, as many per launch as the chip holds
// (128^2, us per iteration for 1 / 16 / 256 fields: 2.7 / 3.5 / 55; one field after
// another 2.75 / 44 / 705; the two-kernel iteration 12 / 14 / 93).
//
// The workgroups of a field have to be resident together. The launch is cooperative,
// which sees to that. One recorded into a graph replays as a plain one: there
// workgroups take their field and block in the order in which they start (`ordered`).
// Those that run then form whole fields, and a launch has at most one field that waits
// for workgroups still to start, with at most kCgMaxGroups - 1 = 63 of them on the chip:
// launches on four hardware queues keep 252 workgroups waiting, fewer than there are
// CUs, so the next one to start always finds room. (The order of start places
// neighbouring blocks worse: 8 fields of 41 x 40 x 40 9.5 us per iteration instead of
// 9.0, 64 of 128^2 15.7 instead of 13.7.) Neither says anything of other processes on the
// same GPU, so every wait is bounded: past the bound a workgroup marks its field
// (CgScal::failed) and leaves, the others follow, and k_cg_alone, launched behind every
// such solve, solves a marked field again from r_0 with one workgroup, which waits for
// nobody. The caller gets a solved field either way.
#include <algorithm>

#include "k_cg.hpp"

namespace ins {

#define INS_AINLINE __attribute__((always_inline))

namespace {

using u64 = unsigned long long;

// Halo cells per thread of an instance.
constexpr int cg_halo(int c) { return c > 12 ? 6 : 4; }

typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

// Device-scope buffer access (sc1: past the XCD's L2): what a relaxed device-scope
// atomic is, 16 bytes at once. The empty asm in the polling loops keeps their loads
// from being moved or merged (the volatile bit would make them system scope).
constexpr int kDeviceScope = 16;

__device__ __forceinline__ void post(Rsrc b, unsigned slot, unsigned tag, double v) {
    const u64 u = static_cast<u64>(__double_as_longlong(v));
    __builtin_amdgcn_raw_buffer_store_b128(v4u{unsigned(u >> 32), tag, unsigned(u), tag}, b, slot * 8u, 0, kDeviceScope);
}
__device__ __forceinline__ v4u peek(Rsrc b, unsigned slot) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, slot * 8u, 0, kDeviceScope);
}
__device__ __forceinline__ double value_of(v4u w) {
    return __longlong_as_double(static_cast<long long>((u64(w.x) << 32) | w.z));
}

// Wait for this thread's N slots; all loads of a round go out together (no branch
// between them). False: gave up after `spin` polls.
template <int N>
__device__ __forceinline__ bool collect(Rsrc base, const unsigned (&slot)[N], unsigned off, unsigned tag, double (&v)[N],
                                        unsigned spin) {
    for (unsigned n = 0; n < spin; ++n) {
        v4u w[N];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = peek(base, slot[i] + off);
        bool all = true;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            all = all && w[i].y == tag && w[i].w == tag;
            v[i] = value_of(w[i]);
        }
        if (all) return true;
    }
    return false;
}

// Lane l of the first wave waits for sum l & 3 of the workgroups l >> 2,
// (l >> 2) + 16, ... (four slots of two words per workgroup) and adds them.
__device__ __forceinline__ bool collect_sum(Rsrc base, unsigned off, int groups, unsigned tag, double& sum,
                                            unsigned spin) {
    constexpr int NP = kCgMaxGroups / 16;
    const unsigned w0 = threadIdx.x >> 2;
    const unsigned slot0 = off + 8 * min(w0, unsigned(groups) - 1u) + 2 * (threadIdx.x & 3);
    sum = 0.0;
    for (unsigned n = 0; n < spin; ++n) {
        v4u w[NP];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < NP; ++i)
            w[i] = peek(base, int(w0) + 16 * i < groups ? slot0 + 128 * i : slot0);
        bool all = true;
        sum = 0.0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            all = all && w[i].y == tag && w[i].w == tag;
            sum += int(w0) + 16 * i < groups ? value_of(w[i]) : 0.0;
        }
        if (all) return true;
    }
    return false;
}

// Sum over a wave, uniform: DPP adds within rows of 16, then across rows (the xor
// shuffles of k_cg.hpp go through the LDS unit, six dependent trips per sum).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const u64 b = static_cast<u64>(__double_as_longlong(v));
    const unsigned lo = __builtin_amdgcn_update_dpp(0, int(unsigned(b)), CTRL, ROWS, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, int(unsigned(b >> 32)), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double(static_cast<long long>((u64(hi) << 32) | lo));
}
__device__ __forceinline__ double wave_total(double v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row holds its sum
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3: lane 63 holds the total
    const u64 b = static_cast<u64>(__double_as_longlong(v));
    const unsigned lo = __builtin_amdgcn_readlane(int(unsigned(b)), 63);
    const unsigned hi = __builtin_amdgcn_readlane(int(unsigned(b >> 32)), 63);
    return __longlong_as_double(static_cast<long long>((u64(hi) << 32) | lo));
}

// Width w^a_i and 1 / d^a_i of direction a (i = -1 .. n - 1): a stretched grid's
// metrics, the channel's y metrics, or the uniform spacing in the channel's
// scaling (A = -w_y D G there: w = 1 and 1 / h^2 along x and z).
__device__ __forceinline__ double met_w(const Grid& g, int a, int n, int i) {
    if (g.gm[0]) return g.gm[a][3 * (n + 2) + i + 1];
    return a == 1 ? g.ym[3 * (n + 2) + i] : 1.0;
}
__device__ __forceinline__ double met_id(const Grid& g, int a, int n, int i) {
    if (g.gm[0]) return g.gm[a][(n + 2) + i + 1];
    return a == 1 ? g.ym[(n + 2) + i + 1] : g.ih2[a];
}

// What a solve leaves for ins_cg_info.
__device__ __forceinline__ void cg_report(CgScal& s, double rr, double rr0, int k) {
    s.rr = rr;
    s.rr0 = rr0;
    s.relres = rr0 > 0.0 ? sqrt(rr / rr0) : 0.0;
    s.it = k;
    s.done = 1;
}

}  // namespace

// NT threads, C consecutive cells each along the last direction (z; y in 2D):
// their neighbours along it are mostly in the thread's own registers, the lateral
// coefficients are constants of the thread, those of the last direction come from
// an LDS table. MULTI: several workgroups per field.
template <int NT, int C, int DIM, bool MULTI>
__global__ __launch_bounds__(NT, 2) void k_cg_solve(Grid g, CgPlan P, const double* __restrict__ r0,
                                                  double* __restrict__ x, const double* __restrict__ rb0,
                                                  CgScal* __restrict__ st, u64* __restrict__ ex, int field0,
                                                  double rtol2, int maxiter, unsigned spin, int ordered) {
    // p on the block plus halo, the table of the last direction, (MULTI) q on the block
    extern __shared__ double pl[];
    __shared__ double sh[NT / 64][4], tot[4];
    __shared__ int lost;
    constexpr int NW = NT / 64, HALO = cg_halo(C);
    constexpr int M = DIM - 1;  // the last direction
    const int tid = threadIdx.x;
    int id = blockIdx.x;
    if constexpr (MULTI)
        if (ordered) {  // by order of start; ex[0]: workgroups of this launch that have started
            __shared__ unsigned started;
            if (tid == 0) started = atomicAdd(reinterpret_cast<unsigned*>(ex), 1u);
            __syncthreads();
            id = __builtin_amdgcn_readfirstlane(started);
        }
    const int fs = id / P.G;  // field of this launch
    const int f = field0 + fs;
    const int wg = id - fs * P.G;
    const int n[3] = {g.nx, g.ny, g.nz};
    const int bc[3] = {wg % P.nb[0], (wg / P.nb[0]) % P.nb[1], wg / (P.nb[0] * P.nb[1])};
    int o[3], e[3];  // origin and extent of the block
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = bc[a] * P.b[a];
        e[a] = min(P.b[a], n[a] - o[a]);
    }
    const int sy = P.b[0] + 2, sz = sy * (P.b[1] + 2);
    const int st3[3] = {1, sy, sz};
    const int sm = st3[M];
    const int npl = sz * (DIM == 3 ? P.b[2] + 2 : 1);
    const bool wally = g.ywalls || !g.gm[0];  // no faces beyond the first and last row
    for (int i = tid; i < npl; i += NT) pl[i] = 0.0;
    double* tw = pl + npl;        // w of the last direction's cells
    double* td = tw + P.b[M];     // 1 / d of their lower faces, then of the last upper one (0 at a wall)
    double* ql = td + P.b[M] + 1;
    for (int i = tid; i <= e[M]; i += NT) {
        if (i < e[M]) tw[i] = met_w(g, M, n[M], o[M] + i);
        const bool wall = M == 1 && wally && (o[M] + i == 0 || o[M] + i == n[M]);
        td[i] = wall ? 0.0 : met_id(g, M, n[M], o[M] + i - 1);
    }
    // (a workgroup that starts after another has given up need not wait its own bound out)
    if constexpr (MULTI)
        if (tid == 0) lost = __hip_atomic_load(&st[f].failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // words of this field, for even and odd iterations: P.G * 2 * DIM outboxes of
    // P.face slots, then the four partial sums of each workgroup
    const Rsrc fx = __builtin_amdgcn_make_buffer_rsrc(ex + kCgHeadWords + size_t(fs) * P.words(), 0, int(P.words() * sizeof(u64)), 0x00027000);
    const unsigned red = P.G * 2 * DIM * P.face * 2;
    const unsigned half = unsigned(P.words() / 2);
    auto outbox = [&](int w, int face) { return unsigned((w * 2 * DIM + face) * P.face * 2); };

    // this thread's column: lateral cell (lx, ly) and the run c0 .. c0 + C - 1 of the last direction
    const int lx = tid % e[0];
    const int ly = DIM == 3 ? (tid / e[0]) % e[1] : 0;
    // (a thread without cells reads, and never writes, the block's first ones)
    int c0 = (DIM == 3 ? tid / (e[0] * e[1]) : tid / e[0]) * C;
    const bool idle = c0 >= e[M];
    if (idle) c0 = 0;
    const int nc = idle ? 0 : min(C, e[M] - c0);  // cells of this thread
    const int nl = max(nc - 1, 0);
    const int gx = o[0] + lx, gy = o[1] + ly;
    const int cell0 = (lx + 1) + (DIM == 3 ? (ly + 1) * sy : 0) + (c0 + 1) * sm;
    const int rm = DIM == 3 ? P.b[0] * P.b[1] : P.b[0];
    const int ql0 = lx + (DIM == 3 ? ly * P.b[0] : 0) + c0 * rm;
    // lateral neighbours: a direction of one block wraps inside it (beyond a wall: the halo row, always 0)
    const int xm = (P.nb[0] == 1 && lx == 0) ? e[0] - 1 : -1, xp = (P.nb[0] == 1 && lx == e[0] - 1) ? 1 - e[0] : 1;
    const bool ywrap = DIM == 3 && P.nb[1] == 1 && !wally;
    const int ym = (ywrap && ly == 0) ? (e[1] - 1) * sy : -sy, yp = (ywrap && ly == e[1] - 1) ? (1 - e[1]) * sy : sy;
    const bool mwrap = P.nb[M] == 1 && !(M == 1 && wally);
    const int mlo = (mwrap && c0 == 0) ? (e[M] - 1) * sm : -sm;
    const int mhi = (mwrap && c0 + nl == e[M] - 1) ? (1 - e[M]) * sm : sm;  // of the run's last cell
    const double wx = met_w(g, 0, n[0], gx), wy = DIM == 3 ? met_w(g, 1, n[1], gy) : 1.0;
    const double axm = wy * met_id(g, 0, n[0], gx - 1), axp = wy * met_id(g, 0, n[0], gx);
    double aym = 0.0, ayp = 0.0;
    if constexpr (DIM == 3) {
        if (!(wally && gy == 0)) aym = wx * met_id(g, 1, n[1], gy - 1);
        if (!(wally && gy == g.ny - 1)) ayp = wx * met_id(g, 1, n[1], gy);
    }
    const double am = wx * wy;
    const int64_t foff = int64_t(f) * g.ncell;
    const int64_t gm = DIM == 3 ? int64_t(g.ny) * g.nx : g.nx;  // stride of the last direction
    const int64_t g0 = foff + gx + (DIM == 3 ? int64_t(gy) * g.nx : 0) + (o[M] + c0) * gm;
    double r[C], xs[C], p[C], q[MULTI ? 1 : C];  // MULTI: q, whose boundary is sent on, lives in LDS
#pragma unroll
    for (int j = 0; j < C; ++j) {
        r[j] = j < nc ? r0[g0 + j * gm] : 0.0;
        xs[j] = 0.0;
        p[j] = r[j];
    }

    // the table's entries of this thread's cells, where the registers allow it
    // (0 past the thread's run, so that its cells' loads and sums need no branch; the
    // longest runs keep the branch and the LDS table: they spill otherwise)
    constexpr bool TREG = C <= 12;
    double twr[TREG ? C : 1], tdr[TREG ? C + 1 : 1];
    auto tw_of = [&](int j) { return TREG ? twr[TREG ? j : 0] : tw[c0 + j]; };
    auto td_of = [&](int j) { return TREG ? tdr[TREG ? j : 0] : td[c0 + j]; };

    // halo cells of this thread: their LDS index, the slot they come from, and (the
    // same face seen from inside) the boundary cell to send and its slot
    int hl[HALO], hb[HALO];
    unsigned hs[HALO], ho[HALO];
    double hr[HALO];  // r there
    if constexpr (MULTI) {
#pragma unroll
        for (int h = 0; h < HALO; ++h) {
            hl[h] = -1;
            hb[h] = 0;
            hs[h] = ho[h] = red + 8 * wg;  // none: its own sum, there in any case
            hr[h] = 0.0;
            int k = (NT - 1 - tid) + h * NT;  // the first wave, which collects the sums, last
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                if (P.nb[a] == 1) continue;
                const int a1 = a == 0 ? 1 : 0, a2 = a == 2 ? 1 : 2;
                const int size = e[a1] * e[a2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    if (a == 1 && wally && bc[1] == (s ? P.nb[1] - 1 : 0)) continue;
                    if (k >= 0 && k < size) {
                        const int i1 = k % e[a1], i2 = k / e[a1];
                        int nbr[3] = {bc[0], bc[1], bc[2]};
                        nbr[a] = s ? (bc[a] + 1 == P.nb[a] ? 0 : bc[a] + 1) : (bc[a] == 0 ? P.nb[a] - 1 : bc[a] - 1);
                        const int w2 = (nbr[2] * P.nb[1] + nbr[1]) * P.nb[0] + nbr[0];
                        hl[h] = (s ? e[a] + 1 : 0) * st3[a] + (i1 + 1) * st3[a1] + (DIM == 3 ? (i2 + 1) * st3[a2] : 0);
                        hs[h] = outbox(w2, 2 * a + (1 - s)) + 2 * k;
                        ho[h] = outbox(wg, 2 * a + s) + 2 * k;
                        const int c[3] = {a == 0 ? (s ? e[0] - 1 : 0) : i1, a == 1 ? (s ? e[1] - 1 : 0) : (a == 0 ? i1 : i2),
                                          a == 2 ? (s ? e[2] - 1 : 0) : i2};
                        hb[h] = (c[2] * P.b[1] + c[1]) * P.b[0] + c[0];
                        // r_0 comes from memory
                        int c3[3];
                        c3[a] = s ? o[a] + e[a] : o[a] - 1;
                        c3[a] = c3[a] < 0 ? c3[a] + n[a] : (c3[a] >= n[a] ? c3[a] - n[a] : c3[a]);
                        c3[a1] = o[a1] + i1;
                        c3[a2] = o[a2] + i2;
                        hr[h] = r0[foff + (int64_t(c3[2]) * g.ny + c3[1]) * g.nx + c3[0]];
                    }
                    k -= size;
                }
            }
        }
    }

    // Sum over the workgroup, in every thread (the only one of its field); which: p.q or r.r
    auto wg_sum = [&](double v, int which) {
        v = wave_total(v);
        if ((tid & 63) == 0) sh[tid >> 6][which] = v;
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NW; ++i) s += sh[i][which];
        return s;
    };

    // rr_0 from the partial sums of the kernel that formed r_0
    double rr0;
    {
        const int np = cg_blocks_of(g);
        double s = 0.0;
        for (int i = tid; i < np; i += NT) s += rb0[int64_t(f) * np + i];
        rr0 = block_sum<NT>(s, &sh[0][0]);  // synchronises: pl, the table and lost are set
    }
    if constexpr (TREG) {
#pragma unroll
        for (int j = 0; j < C; ++j) twr[j] = j < nc ? tw[c0 + j] : 0.0;
#pragma unroll
        for (int j = 0; j <= C; ++j) tdr[j] = j <= nc && nc > 0 ? td[c0 + j] : 0.0;
    }
    double rr = rr0;
    int k = 0;
    if (!(MULTI && lost) && !cg_stopped(rr0, rr0, 0, rtol2, maxiter)) {
#pragma unroll
        for (int j = 0; j < C; ++j)
            if (j < nc) pl[cell0 + j * sm] = p[j];
        if constexpr (MULTI) {
#pragma unroll
            for (int h = 0; h < HALO; ++h)
                if (hl[h] >= 0) pl[hl[h]] = hr[h];
        }
        for (;;) {
            const unsigned tag = unsigned(k) + 1u;
            const unsigned bx = (k & 1) ? half : 0u;
            // keep the addresses below out of registers held across iterations
            int cell = cell0, qb = ql0;
            asm volatile("" : "+v"(cell), "+v"(qb));
            __syncthreads();
            // q = A p
            double s4[4] = {0.0, 0.0, 0.0, 0.0};
            const double pfirst = pl[cell + mlo], plast = pl[cell + nl * sm + mhi];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                auto cell_ap = [&]() INS_AINLINE {
                    const int c = cell + (TREG ? min(j, nl) : j) * sm;
                    const double pc = p[j];
                    // along the last direction: registers but at the run's ends
                    const double pm = j == 0 ? pfirst : p[j > 0 ? j - 1 : 0];
                    const double pp = j == nl || j == C - 1 ? plast : p[j < C - 1 ? j + 1 : j];
                    double lat = (pc - pl[c + xp]) * axp + (pc - pl[c + xm]) * axm;
                    if constexpr (DIM == 3) lat += (pc - pl[c + yp]) * ayp + (pc - pl[c + ym]) * aym;
                    const double v = tw_of(j) * lat + am * ((pc - pp) * td_of(j + 1) + (pc - pm) * td_of(j));
                    s4[0] += pc * v;
                    if constexpr (MULTI) {
                        if (j < nc) ql[qb + j * rm] = v;
                        s4[1] += r[j] * v;
                        s4[2] += j < nc ? v * v : 0.0;
                        s4[3] += r[j] * r[j];
                    } else {
                        q[j] = j < nc ? v : 0.0;
                    }
                };
                if constexpr (TREG) cell_ap();
                else if (j < nc) cell_ap();
            }
            if constexpr (!MULTI) {
                const double pq = wg_sum(s4[0], 0);
                if (!(pq > 0.0)) {  // no component outside the constants: ends without an update
                    rr = 0.0;
                    break;
                }
                const double alpha = rr / pq;
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    xs[j] += alpha * p[j];
                    r[j] -= alpha * q[j];
                    acc += r[j] * r[j];
                }
                const double rrm = rr;
                rr = wg_sum(acc, 1);
                ++k;
                if (cg_stopped(rr, rr0, k, rtol2, maxiter)) break;
                const double beta = rr / rrm;
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    p[j] = r[j] + beta * p[j];
                    if (j < nc) pl[cell + j * sm] = p[j];
                }
            } else {
                // totals over the field of p.q, r.q, q.q and r.r, in every thread; q at the halo
#pragma unroll
                for (int i = 0; i < 4; ++i) s4[i] = wave_total(s4[i]);
                if ((tid & 63) == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) sh[tid >> 6][i] = s4[i];
                }
                __syncthreads();
                if (tid < 64) {
                    if (tid < 4) {
                        double s = 0.0;
#pragma unroll
                        for (int i = 0; i < NW; ++i) s += sh[i][tid];
                        post(fx, bx + red + 8 * wg + 2 * tid, tag, s);
                    }
                    // lane l collects sum l & 3 of the workgroups l >> 2, (l >> 2) + 16, ...
                    double t;
                    if (!collect_sum(fx, bx + red, P.G, tag, t, spin)) lost = 1;
#pragma unroll
                    for (int o = 4; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
                    if (tid < 4) tot[tid] = t;
                }
                double hq[HALO];
#pragma unroll
                for (int h = 0; h < HALO; ++h) {
                    hq[h] = 0.0;
                    if (hl[h] >= 0) post(fx, bx + ho[h], tag, ql[hb[h]]);
                }
                if (!collect<HALO>(fx, hs, bx, tag, hq, spin)) lost = 1;
                __syncthreads();
                if (lost) {  // x and st are then k_cg_alone's
                    if (tid == 0) __hip_atomic_store(&st[f].failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                rr = tot[3];
                if (cg_stopped(rr, rr0, k, rtol2, maxiter)) break;
                const double pq = tot[0];
                if (!(pq > 0.0)) {
                    rr = 0.0;
                    break;
                }
                const double alpha = rr / pq;
                // rr_{k+1} = |r - alpha q|^2, for beta alone: the next sums bring it as summed
                const double beta = fmax(rr - alpha * (2.0 * tot[1] - alpha * tot[2]), 0.0) / rr;
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    auto cell_up = [&]() INS_AINLINE {
                        const double v = ql[qb + (TREG ? min(j, nl) : j) * rm];
                        xs[j] += alpha * p[j];
                        if (j < nc) r[j] -= alpha * v;
                        p[j] = r[j] + beta * p[j];
                        if (j < nc) pl[cell + j * sm] = p[j];
                    };
                    if constexpr (TREG) cell_up();
                    else if (j < nc) cell_up();
                }
#pragma unroll
                for (int h = 0; h < HALO; ++h) {
                    if (hl[h] >= 0) {
                        hr[h] -= alpha * hq[h];
                        pl[hl[h]] = hr[h] + beta * pl[hl[h]];
                    }
                }
                ++k;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < C; ++j)
        if (j < nc) x[g0 + j * gm] = xs[j];
    if (wg == 0 && tid == 0) cg_report(st[f], rr, rr0, k);
}

// The fields that k_cg_solve gave up, each by one workgroup through memory: r = r_0 and
// the scratch fields p, q (r_0 is not needed afterwards); the same operator, recurrence
// and stop test as a field of one workgroup. A field that was solved costs one read.
constexpr int kCgAloneNT = 1024;
template <int DIM>
__global__ __launch_bounds__(kCgAloneNT) void k_cg_alone(Grid g, double* r, double* x, double* p, double* q,
                                                         const double* __restrict__ rb0, CgScal* st, double rtol2,
                                                         int maxiter) {
    __shared__ double sh[kCgAloneNT / 64];
    const int f = blockIdx.x;
    if (!st[f].failed) return;
    const int nx = g.nx, ny = g.ny, nz = DIM == 3 ? g.nz : 1, plane = nx * ny, n = int(g.ncell);
    const bool wally = g.ywalls || !g.gm[0];
    const int64_t foff = int64_t(f) * g.ncell;
    r += foff;
    x += foff;
    p += foff;
    q += foff;
    // sum over the two neighbours of direction a of (p - p_neighbour) / d
    auto pair = [&](int a, int len, int i, int stride, int c) {
        const bool wall = a == 1 && wally;
        const double pc = p[c];
        double s = 0.0;
        if (!(wall && i == 0)) s += (pc - p[i == 0 ? c + (len - 1) * stride : c - stride]) * met_id(g, a, len, i - 1);
        if (!(wall && i == len - 1)) s += (pc - p[i == len - 1 ? c - (len - 1) * stride : c + stride]) * met_id(g, a, len, i);
        return s;
    };
    auto apply = [&](int c) {
        const int z = c / plane, y = c / nx - z * ny, cx = c % nx;
        const double wx = met_w(g, 0, nx, cx), wy = met_w(g, 1, ny, y), wz = DIM == 3 ? met_w(g, 2, nz, z) : 1.0;
        double v = wy * wz * pair(0, nx, cx, 1, c) + wx * wz * pair(1, ny, y, nx, c);
        if constexpr (DIM == 3) v += wx * wy * pair(2, nz, z, plane, c);
        return v;
    };
    double rr0 = 0.0;
    const int np = cg_blocks_of(g);
    for (int i = threadIdx.x; i < np; i += kCgAloneNT) rr0 += rb0[int64_t(f) * np + i];
    rr0 = block_sum<kCgAloneNT>(rr0, sh);
    for (int c = threadIdx.x; c < n; c += kCgAloneNT) {
        x[c] = 0.0;
        p[c] = r[c];
    }
    double rr = rr0;
    int k = 0;
    while (!cg_stopped(rr, rr0, k, rtol2, maxiter)) {
        __syncthreads();  // p is read at neighbouring cells
        double s = 0.0;
        for (int c = threadIdx.x; c < n; c += kCgAloneNT) {
            const double v = apply(c);
            q[c] = v;
            s += p[c] * v;
        }
        const double pq = block_sum<kCgAloneNT>(s, sh);
        if (!(pq > 0.0)) {
            rr = 0.0;
            break;
        }
        const double alpha = rr / pq;
        s = 0.0;
        for (int c = threadIdx.x; c < n; c += kCgAloneNT) {
            x[c] += alpha * p[c];
            const double v = r[c] - alpha * q[c];
            r[c] = v;
            s += v * v;
        }
        const double rrm = rr;
        rr = block_sum<kCgAloneNT>(s, sh);
        ++k;
        const double beta = rr / rrm;
        for (int c = threadIdx.x; c < n; c += kCgAloneNT) p[c] = r[c] + beta * p[c];
    }
    if (threadIdx.x == 0) cg_report(st[f], rr, rr0, k);
}

__global__ __launch_bounds__(kBlock) void k_cg_clear(u64* p, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = 0;
}

namespace {

template <int NT, int C, int DIM, bool MULTI>
const void* kernel_of() {
    return reinterpret_cast<const void*>(&k_cg_solve<NT, C, DIM, MULTI>);
}

// The instance of a plan: threads and cells per thread.
const void* cg_kernel(const Grid& g, const CgPlan& P) {
#define INS_CGK(NT, C, MULTI) (g.dim == 3 ? kernel_of<NT, C, 3, MULTI>() : kernel_of<NT, C, 2, MULTI>())
    if (P.G == 1) return P.nt == 256 ? INS_CGK(256, 4, false) : INS_CGK(512, 8, false);
    switch (P.c) {
        case 2: return INS_CGK(512, 2, true);
        case 4: return INS_CGK(512, 4, true);
        case 6: return INS_CGK(512, 6, true);
        case 8: return INS_CGK(512, 8, true);
        case 10: return INS_CGK(512, 10, true);
        case 12: return INS_CGK(512, 12, true);
        case 16: return INS_CGK(512, 16, true);
        default: return INS_CGK(512, 20, true);
    }
#undef INS_CGK
}

size_t cg_lds(const Grid& g, const CgPlan& P) {
    return (size_t(P.b[0] + 2) * (P.b[1] + 2) * (g.dim == 3 ? P.b[2] + 2 : 1) + 2 * P.b[g.dim - 1] + 1 +
            (P.G > 1 ? size_t(P.b[0]) * P.b[1] * P.b[2] : 0)) *
           sizeof(double);
}

// Threads a block of the plan needs: lateral cells times runs of c cells.
int64_t cg_threads(const CgPlan& P) {
    const int m = P.dim - 1;
    return int64_t(P.b[0]) * (P.dim == 3 ? P.b[1] : 1) * ((P.b[m] + P.c - 1) / P.c);
}

}  // namespace

// Plan of a field: G = 0 when it does not fit (the two-kernel iteration runs it).
CgPlan cg_plan(const Grid& g, int cus) {
    CgPlan P{};
    P.dim = g.dim;
    const int n[3] = {g.nx, g.ny, g.nz};
    // one workgroup while a thread has at most 4 cells
    P.G = 1;
    for (int a = 0; a < 3; ++a) {
        P.nb[a] = 1;
        P.b[a] = n[a];
    }
    for (int nt : {256, 512}) {
        P.nt = nt;
        P.c = nt == 256 ? 4 : 8;
        if (cg_threads(P) <= nt && cg_lds(g, P) <= kCgLdsMax) return P;
    }
    // several: the fewest cells per thread that a quarter of the chip's room allows
    // (an iteration costs its two sums and C steps of the stencil): an even number up to 12,
    // where the table still fits the registers, then 16 and 20 with the table in LDS, which
    // holds no more (p with its halo and q of 512 x 24 cells are 200 KB). us per
    // iteration 2.7 (2 cells) 4.0 (4) 4.7 (6) 5.6 (8) 6.0 (10) 6.9 (12) 7.7 (16) 10 (20).
    // Among the splits with that many cells the one with the smallest halo, but at least kCgMinCells cells per workgroup (the
    // smallest halo alone took 54 workgroups for 17^3 and 64 for 128^2, no faster alone
    // than 9 and 32: 2.9 / 2.8 and 2.75 / 2.75 us per iteration; 256 fields of 128^2
    // then took 117 us on the whole chip instead of 55, the two-kernel iteration 93)
    for (int c : {2, 4, 6, 8, 10, 12, 16, 20}) {
        CgPlan B{};
        int64_t best = 0;
        P.nt = 512;
        P.c = c;
        P.G = 2;
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cg_kernel(g, P), P.nt, kCgLdsMulti) != hipSuccess) {
            (void)hipGetLastError();
            break;
        }
        const int gmax = std::max(2, int(std::min<int64_t>(std::min(kCgMaxGroups, per_cu * cus / 4), g.ncell / kCgMinCells)));
        for (int i = 1; i <= std::min(n[0], gmax); ++i) {
            P.b[0] = (n[0] + i - 1) / i;
            if ((n[0] + P.b[0] - 1) / P.b[0] != i) continue;
            for (int j = 1; j <= n[1] && i * j <= gmax; ++j) {
                P.b[1] = (n[1] + j - 1) / j;
                if ((n[1] + P.b[1] - 1) / P.b[1] != j) continue;
                for (int l = 1; l <= n[2] && i * j * l <= gmax; ++l) {
                    P.b[2] = (n[2] + l - 1) / l;
                    if ((n[2] + P.b[2] - 1) / P.b[2] != l) continue;
                    if (cg_threads(P) > P.nt || cg_lds(g, P) > kCgLdsMulti) continue;
                    int64_t halo = 0, face = 1;
                    const int64_t area[3] = {int64_t(P.b[1]) * P.b[2], int64_t(P.b[0]) * P.b[2], int64_t(P.b[0]) * P.b[1]};
                    const int nb[3] = {i, j, l};
                    for (int a = 0; a < 3; ++a) {
                        if (nb[a] == 1) continue;
                        halo += 2 * area[a];
                        face = std::max(face, area[a]);
                    }
                    if (i * j * l == 1 || halo > cg_halo(c) * P.nt || (B.G != 0 && halo >= best)) continue;
                    best = halo;
                    B = P;
                    B.G = i * j * l;
                    for (int a = 0; a < 3; ++a) B.nb[a] = nb[a];
                    B.face = int(face);
                }
            }
        }
        if (B.G) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cg_kernel(g, B), B.nt, cg_lds(g, B)) != hipSuccess) {
                (void)hipGetLastError();
                break;
            }
            B.fields = std::max(1, std::min(g.batch, per_cu * cus / B.G));
            return B;
        }
    }
    return CgPlan{};
}

hipError_t launch_cg_solve(const Grid& g, const CgPlan& P, double* r, double* x, double* p, double* q, const double* rb0,
                           CgScal* st, void* exch, double rtol2, int maxiter, unsigned spin, hipStream_t s) {
    Grid ga = g;
    CgPlan pa = P;
    u64* ex = static_cast<u64*>(exch);
    const void* kern = cg_kernel(g, P);
    const size_t lds = cg_lds(g, P);
    const int step = P.G == 1 ? g.batch : P.fields;
    // a launch of one field needs no order; an error here is that of a stream which must
    // not be used while another one records, and the launch below reports it
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (P.fields > 1 && hipStreamIsCapturing(s, &capture) != hipSuccess) (void)hipGetLastError();
    int ordered = capture != hipStreamCaptureStatusNone;
    for (int f0 = 0; f0 < g.batch; f0 += step) {
        const int nf = std::min(step, g.batch - f0);
        void* args[] = {&ga, &pa, &r, &x, &rb0, &st, &ex, &f0, &rtol2, &maxiter, &spin, &ordered};
        hipError_t e;
        if (P.G == 1) {
            e = hipLaunchKernel(kern, dim3(nf), dim3(P.nt), args, lds, s);
        } else {
            const int64_t words = kCgHeadWords + int64_t(P.words()) * nf;
            hipLaunchKernelGGL(k_cg_clear, dim3(int((words + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, ex, words);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            e = hipLaunchCooperativeKernel(kern, dim3(nf * P.G), dim3(P.nt), args, unsigned(lds), s);
        }
        if (e != hipSuccess) return e;
    }
    if (P.G == 1) return hipSuccess;
    if (g.dim == 3)
        hipLaunchKernelGGL((k_cg_alone<3>), dim3(g.batch), dim3(kCgAloneNT), 0, s, g, r, x, p, q, rb0, st, rtol2, maxiter);
    else
        hipLaunchKernelGGL((k_cg_alone<2>), dim3(g.batch), dim3(kCgAloneNT), 0, s, g, r, x, p, q, rb0, st, rtol2, maxiter);
    return hipGetLastError();
}

}  // namespace ins
