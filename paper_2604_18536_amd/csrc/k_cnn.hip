// Learned closure m_theta(u) (Sec. 4 of the paper: a neural closure embedded in
// the solver and trained through it) as hand-written bfloat16 MFMA kernels for
// gfx950: a 3D CNN 3 -> 32 -> 32 -> 3 channels, 3x3x3 kernels, circular
// padding, exact GELU, FP32 accumulation.
//
// Activations are channels-last bfloat16 ([cell][C], C = 8 for the packed
// 3-channel input, 32 for hidden layers). A convolution is an implicit GEMM
// D[cell][n] = sum_k A[cell][k] B[k][n] with k = (tap, channel), executed as
// v_mfma_f32_16x16x32_bf16 tiles (lane l holds A[m = l%16][k = 8(l/16)+j],
// B[k = 8(l/16)+j][n = l%16], D[m = 4(l/16)+i][n = l%16]). A K tile of 32 is
// one tap x 32 channels (C = 32) or four taps x 8 channels (C = 8); every lane
// fetches its 8 bfloat16 operands with one 16-byte load. A workgroup stages
// its input block (with the periodic halo) in LDS once and reads all 27 taps'
// A operands from there; weights are packed per K tile ([kt][n][32]) and read
// from global memory, where they stay cache-resident. The input gradient
// (dgrad) is the same kernel with flipped taps and transposed weights; the
// weight gradient (wgrad) reduces over cells with operands transposed through
// LDS and per-workgroup partial sums.
#include <hip/hip_bf16.h>

#include "k_common.hpp"

namespace ins {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16;

constexpr int kTaps = 27;

__device__ __forceinline__ u16 bf16_bits(float v) {
    const __bf16 b = __bf16(v);  // round to nearest even
    return __builtin_bit_cast(u16, b);
}
__device__ __forceinline__ float bf16_val(u16 bits) { return float(__builtin_bit_cast(__bf16, bits)); }

// Exact GELU z Phi(z) and its derivative Phi(z) + z phi(z) of N values per lane, after
// erff and expf: two fits of their own (weighted least squares towards the minimax error).
//   |z| < 1.4 (derivative: 1): z/2 + z^2 K(z^2) and 1/2 + z P(z^2), absolute error 2e-9;
//   beyond, where any lane of the wave needs it: the upper tail
//     Q(t) = 1 - Phi(t) = exp(-t^2/2) s (c1 + ... + c7 s^6),  s = 1 / (1 + 0.45 t),
//   the form of Abramowitz & Stegun 7.1.26 (3e-9), and max(z, 0) - |z| Q(|z|), which does
//   not cancel. Q is 0 beyond 20.
// An epilogue evaluates one per output, 268 M at 4 x 128^3, on the same issue slots as
// the matrix products: erff and expf were 60-70 % of the 8 -> 32 layers' vector work.
// Those went from 398 (forward) and 520 us (pullback) to 364 and 423, the 32 -> 32 ones
// from 705 and 800 to 660 and 734. Largest / rms error against float64 on [-7, 7]:
// GELU 2.4e-7 / 5.5e-8 (erff 4.5e-7 / 7.3e-8), derivative 1.32e-7 / 2.72e-8 (1.42e-7 /
// 2.74e-8); on a unit normal 2.4e-7 / 1.8e-8 (4.2e-7 / 2.5e-8) and 1.40e-7 / 2.59e-8
// (1.43e-7 / 2.70e-8).
constexpr float kGeluCentre = 1.4f, kGradCentre = 1.0f;

// A constant in a scalar register: as literals half of the polynomials' constants were
// moved to vector registers before each use.
template <unsigned BITS>
__device__ __forceinline__ float sconst() {
    float r;
    asm("s_mov_b32 %0, %1" : "=s"(r) : "i"(BITS));
    return r;
}
#define INS_SC(v) sconst<__builtin_bit_cast(unsigned, v)>()

template <int N>
__device__ __forceinline__ bool gelu_far(const float (&z)[N], float centre) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) m = fmaxf(m, fabsf(z[i]));
    return __builtin_amdgcn_ballot_w64(m >= centre) != 0;
}
// e = exp(-z^2 / 2) and Q(min(|z|, 20)).
__device__ __forceinline__ float gelu_tail(float z, float t, float& e) {
    e = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);
    const float d = fmaf(t, INS_SC(0.45f), 1.0f);
    float s = __builtin_amdgcn_rcpf(d);
    s = fmaf(s, fmaf(-d, s, 1.0f), s);
    float p = fmaf(s, INS_SC(-0.0377919599f), INS_SC(0.217211068f));
    p = fmaf(s, p, INS_SC(-0.473691344f));
    p = fmaf(s, p, INS_SC(0.39339155f));
    p = fmaf(s, p, INS_SC(0.0182143468f));
    p = fmaf(s, p, INS_SC(0.205396548f));
    p = fmaf(s, p, INS_SC(0.177269787f));
    return p * (s * e);
}
template <int N>
__device__ __forceinline__ void gelu_n(const float (&z)[N], float (&a)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float q = z[i] * z[i];
        float k = fmaf(q, INS_SC(3.60695452e-07f), INS_SC(-8.32990918e-06f));
        k = fmaf(q, k, INS_SC(0.000113203139f));
        k = fmaf(q, k, INS_SC(-0.00118481647f));
        k = fmaf(q, k, INS_SC(0.00997202843f));
        k = fmaf(q, k, INS_SC(-0.0664899349f));
        k = fmaf(q, k, INS_SC(0.398942232f));
        a[i] = fmaf(q, k, 0.5f * z[i]);
    }
    if (gelu_far(z, kGeluCentre)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float e;
            const float t = fminf(fabsf(z[i]), 20.0f), tail = gelu_tail(z[i], t, e);
            if (t >= kGeluCentre) a[i] = fmaf(z[i] > 0.0f ? -t : z[i], tail, fmaxf(z[i], 0.0f));
        }
    }
}
template <int N>
__device__ __forceinline__ void gelu_grad_n(const float (&z)[N], float (&d)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float q = z[i] * z[i];
        float c = fmaf(q, INS_SC(-3.40459962e-07f), INS_SC(8.06192656e-06f));
        c = fmaf(q, c, INS_SC(-0.000110526133f));
        c = fmaf(q, c, INS_SC(0.00115069456f));
        c = fmaf(q, c, INS_SC(-0.00949590001f));
        c = fmaf(q, c, INS_SC(0.0598402545f));
        c = fmaf(q, c, INS_SC(-0.265961319f));
        c = fmaf(q, c, INS_SC(0.797884524f));
        d[i] = fmaf(z[i], c, 0.5f);
    }
    if (gelu_far(z, kGradCentre)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float e;
            const float t = fminf(fabsf(z[i]), 20.0f), tail = gelu_tail(z[i], t, e);
            const float far = fmaf(z[i] * 0.39894228040143268f, e, 0.5f + copysignf(0.5f - tail, z[i]));
            if (t >= kGradCentre) d[i] = far;
        }
    }
}

__device__ __forceinline__ int wrapi(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }
// Output channel of column lm of tile nt: with two tiles (32 channels) a lane holds two
// neighbouring channels, which it stores (and reads, z) as one value.
template <int NT>
__host__ __device__ __forceinline__ constexpr int out_chan(int nt, int lm) { return NT == 2 ? 2 * lm + nt : nt * 16 + lm; }

// K tile kt, lane group gq: which tap and which first channel the lane's 8 operands hold.
template <int CIN>
__device__ __forceinline__ void ktile_tap(int kt, int gq, int& tap, int& c0) {
    if constexpr (CIN == 32) {
        tap = kt;
        c0 = 8 * gq;
    } else {
        tap = 4 * kt + gq;
        c0 = 0;
    }
}

enum { EPI_HIDDEN = 0, EPI_OUT = 1, EPI_DGRAD_HIDDEN = 2, EPI_DGRAD_INPUT = 3 };

// Implicit-GEMM 3x3x3 convolution over all cells of the batch.
//   in   : [cells][CIN] bfloat16
//   wpk  : [NKT][NT*16][32] bfloat16 packed weights (zero where k or n is padding; column
//          nt * 16 + lm holds output channel out_chan(nt, lm))
//   EPI_HIDDEN      : z = acc + bias -> zout [cells][32] fp32 (unless null), a = bf16(gelu(z)) -> aout [cells][32]
//   EPI_OUT         : m[b][n][cell] = acc + bias (n < nout), field type T (planar velocity layout)
//   EPI_DGRAD_HIDDEN: zbar = acc * gelu'(zin[cell][n]) -> aout [cells][32] bf16
//   EPI_DGRAD_INPUT : ubar[b][n][cell] += acc (n < nout), field type T
// The input block is staged in LDS. A workgroup owns a
// 32 x 4 x BZ block of output cells (x, y, z); it copies the 34 x 6 x (BZ + 2)
// input block (periodic halo included) into LDS once, so the 27 taps read their
// A operands from LDS instead of re-fetching them from memory. B operands
// (packed weights) come from global memory (every wave of every workgroup reads
// the same few KB per tap; they stay cache-resident). Wave w computes the
// output row y = w of every z plane of the block (M tiles mt: plane mt / 2,
// x half mt % 2). With 32 input channels the K loop runs over the nine (ty, tx)
// tap columns and, inside, over the BZ + 2 halo planes: each A operand fetched
// from LDS serves every output plane it is a tap of (tz = hz - z), and each
// weight operand fetched for a tap column serves 2 BZ M tiles. Hidden
// layer outputs are staged through LDS so that every global store is a full
// 16-byte chunk of one cell. In LDS the input block is split by 8-channel
// chunk, xs[chunk][cell][8]: the 16 lanes of an operand fetch read 16
// consecutive 16-byte cells (no bank conflicts, every access 16-byte aligned).
constexpr int kCbX = 32, kCbY = 4, kCbZ = 2, kCbCells = kCbX * kCbY * kCbZ;
constexpr int kChX = kCbX + 2, kChY = kCbY + 2, kChZ = kCbZ + 2, kChCells = kChX * kChY * kChZ;

// Block row (y + 4 z) of M tile mt of wave w: row y = w of plane mt / 2.
__device__ __forceinline__ int conv_row(int wave, int mt) { return (mt >> 1) * kCbY + wave; }

// The convolution kernel's output block is 32 x 4 x BZ cells: BZ = 4 for 32 -> 32
// channels (every weight operand a wave fetches then feeds 8 MFMAs instead of 4: 579 us
// against 675 with BZ = 2, pullback 647 against 667), else 2.
//
// What bounds it at 4 x 128^3 (us, before -> now): two or three workgroups per CU (LDS)
// run load, products and epilogue one after the other, so every serial wait counts. All
// loads of the input block are in flight together (before: one round trip of 4 per
// thread after the other), as are the z or cotangent values the epilogue reads (before:
// round trips through LDS or one at a time after the products); the 3-channel outputs
// are written as whole rows. 32 -> 32 676 -> 575 (464 GFLOP: 0.8 PFLOP/s) and pullback
// 861 -> 650, 8 -> 32 401 -> 341 and pullback 705 -> 385, 32 -> 3 469 -> 279 and
// pullback 537 -> 280. (The staging arrays are native vectors: as arrays of uint4 they
// were kept in scratch memory and everything took 1.5-2 times as long.)
template <int BZ>
constexpr int conv_halo_cells() { return kChX * kChY * (BZ + 2); }

// Cells from one 8-channel chunk of the input block in LDS to the next: a multiple of
// 16, all the banks, so that lanes of different chunks conflict only if their cells do.
template <int CIN, int BZ>
constexpr int conv_chunk_cells() { return CIN == 32 ? (conv_halo_cells<BZ>() + 15) / 16 * 16 : conv_halo_cells<BZ>(); }
constexpr int kAtRow = 40;  // bfloat16 output cell in LDS: 32 channels padded (conflict-free stores)

template <int CIN, int BZ>
constexpr size_t conv_t_lds_bytes(bool hidden) {
    const size_t halo = size_t(conv_chunk_cells<CIN, BZ>()) * CIN * 2;
    const size_t epi = size_t(kCbX * kCbY * BZ) * (hidden ? kAtRow * 2 : 3 * 4);
    return halo > epi ? halo : epi;
}

// The layers with one tile of outputs (32 -> 3 channels) hold all their weights in
// registers and walk over the blocks, the next block's loads in flight through a block's
// work: 356 -> 279 us, pullback 366 -> 282. The others would need more registers than two
// waves per SIMD have (the 32 -> 32 layers spilled 160-260 of them and took 1.4 ms).
template <int CIN, int NT>
constexpr bool conv_walks() { return CIN == 32 && NT == 1; }
constexpr int kWalkGroups = 512;  // two per CU, by registers

// v in [-1, n + 4] into [0, n), n >= 2.
__device__ __forceinline__ int wrap_near(int v, int n) {
    v = v < 0 ? v + n : v;
    v = v >= n ? v - n : v;
    return v >= n ? v - n : v;
}

template <typename T, int CIN, int NT, int EPI, int BZ>
__global__ __launch_bounds__(kBlock) void k_conv_t(Grid g, const u16* __restrict__ in, const u16* __restrict__ wpk,
                                                     const float* __restrict__ bias, const float* __restrict__ zin,
                                                     float* __restrict__ zout, u16* __restrict__ aout,
                                                     T* __restrict__ fout, int nout) {
    constexpr int NKT = (kTaps * CIN + 31) / 32;
    constexpr int MT = 2 * BZ;  // M tiles per wave: BZ planes x 2 halves of x
    constexpr int HZ = BZ + 2, HCELLS = conv_halo_cells<BZ>(), HC = conv_chunk_cells<CIN, BZ>();
    constexpr int CH = CIN / 8;  // 16-byte chunks per cell
    constexpr int NROW = kChY * HZ;
    extern __shared__ __attribute__((aligned(16))) u16 xs[];
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int nbx = nx / kCbX, nby = (ny + kCbY - 1) / kCbY, nbz = (nz + BZ - 1) / BZ;
    constexpr bool WALK = conv_walks<CIN, NT>();
    const int nblocks = nbx * nby * nbz * g.batch;
    const int64_t vol = int64_t(nx) * ny * nz;
    int b, x0, y0, z0;
    int64_t bcell;
    auto place = [&](int blk) {
        int L = blk;
        x0 = L % nbx * kCbX;
        L /= nbx;
        y0 = L % nby * kCbY;
        L /= nby;
        z0 = L % nbz * BZ;
        b = L / nbz;
        bcell = b * vol;
    };
    int blk = xcd_logical(blockIdx.x, gridDim.x);
    place(blk);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, gq = lane >> 4;
    // 1. input block with periodic halo -> LDS. A wave takes whole halo rows, 64 / CH cells a
    // load with the lanes of a chunk together: the row's address is scalar and a lane's
    // place in it the same for every row. The last two cells of every row follow. Every load of a
    // thread is in flight before the first is stored.
    auto row_base = [&](int row) {
        const int hz = row / kChY, hy = row - hz * kChY;
        return in + (bcell + int64_t(wrap_near(z0 - 1 + hz, nz) * ny + wrap_near(y0 - 1 + hy, ny)) * nx) * CIN;
    };
    constexpr int RW = CH == 4 ? 1 : 2, RPW = NROW / (4 * RW);  // rows a load covers, loads per 32 cells of a wave's rows
    constexpr int NE = NROW * 2 * CH, KE = (NE + kBlock - 1) / kBlock;
    static_assert(NROW % (4 * RW) == 0, "whole rows per wave");
    const int sch = CH == 4 ? gq : 0, sx = CH == 4 ? lm : lane & 31, srow = CH == 4 ? 0 : lane >> 5;
    u32x4 va[RPW], vb[RPW], ve[KE];
    auto fetch_in = [&]() __attribute__((always_inline)) {
        const int xo0 = wrapi(x0 - 1 + sx, nx) * CIN + sch * 8, xo1 = (x0 + 15 + sx) * CIN + sch * 8;
#pragma unroll
        for (int k = 0; k < RPW; ++k) {
            const int row = (wave * RPW + k) * RW;
            const u16* base = row_base(row);
            if constexpr (RW == 2) {
                const u16* next = row_base(row + 1);
                base = srow ? next : base;
            }
            va[k] = *reinterpret_cast<const u32x4*>(base + xo0);
            if constexpr (CH == 4) vb[k] = *reinterpret_cast<const u32x4*>(base + xo1);
        }
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            const int e = min(k * kBlock + tid, NE - 1), row = e / (2 * CH);
            ve[k] = *reinterpret_cast<const u32x4*>(row_base(row) + wrapi(x0 + 31 + (e / CH & 1), nx) * CIN + e % CH * 8);
        }
    };
    // block cell q = r * 32 + x of block row r; its grid cell
    auto block_cell = [&](int q, int64_t& c) -> bool {
        const int r = q >> 5, xx = q & 31;
        const int yy = y0 + r % kCbY, zz = z0 + r / kCbY;
        c = bcell + (int64_t(zz) * ny + yy) * nx + x0 + xx;
        return yy < ny && zz < nz;
    };
    // what the epilogue reads, in flight through the GEMM: z at this lane's accumulators,
    // or the input cotangent so far at cell tid
    constexpr int ZM = EPI == EPI_DGRAD_HIDDEN ? MT : 1;
    float zr[ZM][4][NT];
    T old[3];
    auto fetch_epi = [&]() __attribute__((always_inline)) {
        if constexpr (EPI == EPI_DGRAD_HIDDEN) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int r = conv_row(wave, mt);
                const int yy = min(y0 + r % kCbY, ny - 1), zz = min(z0 + r / kCbY, nz - 1);
                const float* zp = zin + (bcell + (int64_t(zz) * ny + yy) * nx + x0 + (mt & 1) * 16 + 4 * gq) * 32 + 2 * lm;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f32x2 z2 = *reinterpret_cast<const f32x2*>(zp + i * 32);
                    zr[mt][i][0] = z2[0];
                    zr[mt][i][NT - 1] = z2[1];
                }
            }
        }
        if constexpr (EPI == EPI_DGRAD_INPUT) {
            int64_t c;
            const bool ok = block_cell(tid, c);
#pragma unroll
            for (int n = 0; n < 3; ++n) old[n] = fout[(int64_t(b) * 3 + n) * vol + (ok ? c - bcell : 0)];
        }
    };
    // the weight operands of tap column tyx (tz = 0, 1, 2; 32 input channels), fetched one
    // column ahead; with one tile of outputs all of them, once per workgroup
    constexpr int PF = NT == 1 ? 9 : 1;
    bf16x8 bn[PF][3][NT];
    auto fetch_w = [&](int tyx) __attribute__((always_inline)) {
#pragma unroll
        for (int tz = 0; tz < 3; ++tz)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                bn[tyx % PF][tz][nt] =
                    *reinterpret_cast<const bf16x8*>(wpk + (((tz * 9 + tyx) * NT * 16 + nt * 16 + lm) * 32 + 8 * gq));
    };
    fetch_in();
    if constexpr (!WALK) fetch_epi();
    if constexpr (WALK) {
#pragma unroll
        for (int k = 0; k < PF; ++k) fetch_w(k);
    }
    do {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WALK) __syncthreads();  // the previous block's outputs are no longer read
        {
            u16* dst = xs + (sch * HC + (wave * RPW * RW + srow) * kChX + sx) * 8;
#pragma unroll
            for (int k = 0; k < RPW; ++k) {
                *reinterpret_cast<u32x4*>(dst + k * RW * kChX * 8) = va[k];
                if constexpr (CH == 4) *reinterpret_cast<u32x4*>(dst + (k * RW * kChX + 16) * 8) = vb[k];
            }
#pragma unroll
            for (int k = 0; k < KE; ++k) {
                const int e = k * kBlock + tid;
                if (e < NE)
                    *reinterpret_cast<u32x4*>(xs + (e % CH * HC + e / (2 * CH) * kChX + 32 + (e / CH & 1)) * 8) = ve[k];
            }
        }
        if constexpr (WALK) {
            fetch_epi();
            const int next = blk + int(gridDim.x);
            place(next < nblocks ? next : blk);
            fetch_in();
            place(blk);
            __builtin_amdgcn_sched_barrier(0);
        }
        // 2. implicit GEMM from LDS
        f32x4 acc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        int hbase[MT];  // halo cell of (tap offset 0, 0, 0) for this lane's row of each M tile
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int r = conv_row(wave, mt);
            const int yy = r % kCbY, zz = r / kCbY;
            hbase[mt] = (zz * kChY + yy) * kChX + (mt & 1) * 16 + lm;
        }
        if constexpr (CIN == 32) {
            const u16* xq = xs + (gq * HC) * 8;  // this lane's 8-channel chunk
            if constexpr (!WALK) {
#pragma unroll
                for (int k = 0; k < PF; ++k) fetch_w(k);
            }
            __syncthreads();
#pragma unroll
            for (int tyx = 0; tyx < 9; ++tyx) {
                const int ty = tyx / 3, tx = tyx % 3;
                bf16x8 bv[3][NT];
#pragma unroll
                for (int tz = 0; tz < 3; ++tz)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) bv[tz][nt] = bn[tyx % PF][tz][nt];
                if (!WALK && tyx + PF < 9) fetch_w(tyx + PF);
                __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of this column's work
#pragma unroll
                for (int hz = 0; hz < HZ; ++hz) {
#pragma unroll
                    for (int xh = 0; xh < 2; ++xh) {
                        // halo cell of source plane hz for output row (y = wave) and x half xh
                        const int cell = (hz * kChY + wave + ty) * kChX + xh * 16 + lm + tx;
                        const bf16x8 av = *reinterpret_cast<const bf16x8*>(xq + cell * 8);
#pragma unroll
                        for (int zz = 0; zz < BZ; ++zz) {
                            const int tz = hz - zz;
                            if (tz < 0 || tz > 2) continue;
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
                                acc[zz * 2 + xh][nt] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[tz][nt], acc[zz * 2 + xh][nt], 0, 0, 0);
                        }
                    }
                }
            }
        } else {
            // the weight operands of K tile kt, fetched one tile ahead
            bf16x8 kn[NT];
            auto fetch_k = [&](int kt) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    kn[nt] = *reinterpret_cast<const bf16x8*>(wpk + ((kt * NT * 16 + nt * 16 + lm) * 32 + 8 * gq));
            };
            fetch_k(0);
            __syncthreads();
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
                int tap, c0;
                ktile_tap<CIN>(kt, gq, tap, c0);
                const bool tap_ok = tap < kTaps;
                const int t = tap_ok ? tap : 0;
                const int toff = ((t / 9) * kChY + (t / 3) % 3) * kChX + t % 3;
                bf16x8 bv[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) bv[nt] = kn[nt];
                if (kt + 1 < NKT) fetch_k(kt + 1);
                __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of this tile's work
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    bf16x8 av;
                    if (tap_ok) {
                        av = *reinterpret_cast<const bf16x8*>(xs + (hbase[mt] + toff) * 8);
                    } else {
#pragma unroll
                        for (int j = 0; j < 8; ++j) av[j] = __bf16(0.0f);
                    }
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[nt], acc[mt][nt], 0, 0, 0);
                }
            }
        }
        // 3. epilogue: lane holds D[m = 4 gq + i][n = nt*16 + lm] of M tile mt, i.e. block
        // cell q = r * 32 + (mt & 1) * 16 + 4 gq + i with r = conv_row(wave, mt)
        constexpr int NCELL = kCbX * kCbY * BZ;
        __syncthreads();  // every wave is done reading the input block
        if constexpr (EPI == EPI_HIDDEN || EPI == EPI_DGRAD_HIDDEN) {
            // z (if kept) from the registers, a cell's 128 bytes at once; the bfloat16 output
            // through LDS
            u16* at = xs;
            float bv[NT];
            if constexpr (EPI == EPI_HIDDEN)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) bv[nt] = bias[out_chan<NT>(nt, lm)];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int qb = conv_row(wave, mt) * 32 + (mt & 1) * 16 + 4 * gq;  // four cells of a row
                int64_t c;
                const bool ok = block_cell(qb, c);
                float z[4 * NT], o[4 * NT];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if constexpr (EPI == EPI_HIDDEN) z[i * NT + nt] = acc[mt][nt][i] + bv[nt];
                        else z[i * NT + nt] = zr[mt][i][nt];
                    }
                if constexpr (EPI == EPI_HIDDEN) {
                    if (zout && ok) {
                        float* zp = zout + c * 32 + 2 * lm;
#pragma unroll
                        for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x2*>(zp + i * 32) = f32x2{z[i * NT], z[i * NT + 1]};
                    }
                    gelu_n(z, o);
                } else {
                    gelu_grad_n(z, o);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f32x2 v = {o[i * NT], o[i * NT + 1]};
                    if constexpr (EPI == EPI_DGRAD_HIDDEN) v = f32x2{acc[mt][0][i] * v[0], acc[mt][1][i] * v[1]};
                    *reinterpret_cast<bf16x2*>(at + (qb + i) * kAtRow + 2 * lm) = __builtin_convertvector(v, bf16x2);
                }
            }
            __syncthreads();
#pragma unroll
            for (int e = tid; e < NCELL * 4; e += kBlock) {  // 4 chunks per cell
                const int q = e >> 2, ch = e & 3;
                int64_t c;
                if (block_cell(q, c))
                    *reinterpret_cast<uint4*>(aout + c * 32 + ch * 8) =
                        *reinterpret_cast<const uint4*>(at + q * kAtRow + ch * 8);
            }
        } else {
            static_assert(NCELL == kBlock, "one cell per thread");
            float* ot = reinterpret_cast<float*>(xs);  // [3][cell]
            if (lm < nout) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int qb = conv_row(wave, mt) * 32 + (mt & 1) * 16 + 4 * gq;
                    *reinterpret_cast<f32x4*>(ot + lm * NCELL + qb) = acc[mt][0];
                }
            }
            __syncthreads();
            int64_t c;
            if (block_cell(tid, c)) {
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    T* dst = fout + (int64_t(b) * 3 + n) * vol + (c - bcell);
                    const float v = ot[n * NCELL + tid];
                    if constexpr (EPI == EPI_OUT)
                        *dst = T(v + bias[n]);
                    else
                        *dst = T(double(old[n]) + double(v));
                }
            }
        }
        if constexpr (!WALK) break;
        blk += gridDim.x;
        place(blk);
    } while (blk < nblocks);
}

// Planar velocity u = w - G p (PROJ: float64 projection rounded to T; else w) ->
// channels-last bfloat16 [cell][8] (channels 3..7 zero). Bound by its bytes: 300 MB at
// 4 x 128^3 float32; projecting in a launch of its own wrote u and read it again (97 us
// for the two, 54 us here).
template <typename T, bool PROJ>
__global__ __launch_bounds__(kBlock) void k_pack_input(Grid g, const T* __restrict__ w, const double* __restrict__ p,
                                                         u16* __restrict__ x0) {
    const int64_t c = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t vol = g.ncell;
    if (c >= vol * g.batch) return;
    const int64_t b = c / vol;
    const int r = int(c - b * vol);
    T u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] = w[(b * 3 + a) * vol + r];
    if constexpr (PROJ) {
        const int row = r / g.nx, x = r - row * g.nx, z = row / g.ny, y = row - z * g.ny;
        const double* pb = p + b * vol;
        const double pc = pb[r];
        const double dp[3] = {pb[x + 1 == g.nx ? r + 1 - g.nx : r + 1] - pc, pb[y + 1 == g.ny ? r + g.nx - g.nx * g.ny : r + g.nx] - pc,
                              pb[z + 1 == g.nz ? row % g.ny * g.nx + x : r + g.nx * g.ny] - pc};
#pragma unroll
        for (int a = 0; a < 3; ++a) u[a] = T(double(u[a]) - dp[a] * g.ih[a]);
    }
    u16 v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = bf16_bits(float(u[a]));
    uint4 out;
    out.x = v[0] | (unsigned(v[1]) << 16);
    out.y = v[2] | (unsigned(v[3]) << 16);
    out.z = v[4] | (unsigned(v[5]) << 16);
    out.w = v[6] | (unsigned(v[7]) << 16);
    reinterpret_cast<uint4*>(x0)[c] = out;
}

// FP32 parameters -> packed bfloat16 forward and dgrad weights.
// Forward layer (cin, cout): wf[kt][column][32] (out_chan gives the column's n), K tile kt covering (tap, channel) as in ktile_tap<CINP>.
// Dgrad of the layer: a convolution from cout channels to cin channels with
// W'[n = i][k = (t', o)] = W[o][i][26 - t'].
__global__ void k_pack_weights(const float* __restrict__ w, int cin, int cout, int cinp, int ntf, u16* __restrict__ wf,
                               int coutp, int ntd, u16* __restrict__ wd) {
    const int nktf = (kTaps * cinp + 31) / 32;
    const int nktd = (kTaps * coutp + 31) / 32;
    const int totf = nktf * ntf * 16 * 32;
    const int totd = nktd * ntd * 16 * 32;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < totf) {
        const int kk = i & 31, col = (i >> 5) % (ntf * 16), kt = i / (32 * ntf * 16);
        const int n = ntf == 2 ? out_chan<2>(col >> 4, col & 15) : col;
        const int gq = kk >> 3, j = kk & 7;
        int tap, c;
        if (cinp == 32) {
            tap = kt;
            c = 8 * gq + j;
        } else {
            tap = 4 * kt + gq;
            c = j;
        }
        float v = 0.f;
        if (tap < kTaps && c < cin && n < cout) v = w[(n * cin + c) * kTaps + tap];
        wf[i] = bf16_bits(v);
    } else if (i < totf + totd) {
        const int e = i - totf;
        const int kk = e & 31, col = (e >> 5) % (ntd * 16), kt = e / (32 * ntd * 16);
        const int n = ntd == 2 ? out_chan<2>(col >> 4, col & 15) : col;
        const int gq = kk >> 3, j = kk & 7;
        int tap, o;
        if (coutp == 32) {
            tap = kt;
            o = 8 * gq + j;
        } else {
            tap = 4 * kt + gq;
            o = j;
        }
        float v = 0.f;
        if (tap < kTaps && o < cout && n < cin) v = w[(o * cin + n) * kTaps + (kTaps - 1 - tap)];
        wd[e] = bf16_bits(v);
    }
}

// Weight gradient on 32 x 4 x 2 cell blocks:
// W'[n][tap][c] = sum_p g[p][n] x[p + off(tap)][c], bias'[n] = sum_p g[p][n].
// A workgroup stages, transposed to channel-major in LDS, the cotangent g of
// its block (gT[n][p]) and the input x of the block's halo (xT[c][z][y][x]);
// the K dimension of each MFMA is 32 cells of one block row. The work of a row is
// split in 18 units over the waves: a tap column (dz, dy) with its three dx, and one
// half of the 32 channels (of x, or of g where x has 8). A unit reads its B operand
// once, 16 + 4 bytes per lane: the three dx start 0, 2 or 4 bytes past a 16-byte
// boundary, and a byte-align selects each. (With taps dealt out singly every tap read
// 32 bytes per lane: 27 x 2 x 2 LDS reads per row.) The loads of the next block are in flight through a
// block's products. Cells outside the grid (partial blocks in y or z) stage g = 0.
// Workgroups loop over a contiguous range of blocks and write per-workgroup partial
// sums (reduced in order by k_wgrad_reduce). At 4 x 128^3: 32 x 32 channels 858 -> 750 us
// (0.6 PFLOP/s), 3 (as 8) x 32 739 -> 409, 32 x 3 462 -> 332; what is left is 2 waves per
// SIMD sharing MFMA (27 %), transposing and selecting (32 %) and LDS (40 %, half of it
// conflicts of the 16- and 4-byte reads).
constexpr int kGtStride = kCbCells + 8;  // gT row: 256 cells + pad (conflict-free A reads)
constexpr int kXtRow = 40;               // xT halo row: 34 cells padded to 40
constexpr int kXtStride = kChZ * kChY * kXtRow + 8;

// LDS row of channel 8 ch + i, and the channel of a row. With 32 channels a wave stores
// 4 chunks of 16 cell pairs at once; 4 rows between the chunks are 16 banks (the strides
// are 4 times an odd number of dwords), so its stores do not conflict (chunk after chunk
// they did, 8 cycles a store).
template <int C>
__device__ __forceinline__ constexpr int chan_row(int ch, int i) { return C == 32 ? (i & 3) + 4 * ch + 16 * (i >> 2) : i; }
template <int C>
__device__ __forceinline__ constexpr int row_chan(int r) { return C == 32 ? 8 * ((r >> 2) & 3) + (r & 3) + 4 * (r >> 4) : r; }

template <int CIN, int COUTP>
__global__ __launch_bounds__(kBlock, 2) void k_wgrad_t(Grid g, const u16* __restrict__ gin, const u16* __restrict__ xin,
                                                         float* __restrict__ partial) {
    constexpr int MT = COUTP == 32 ? 2 : 1;      // tiles of output channels n
    constexpr int NT = CIN == 32 ? 2 : 1;        // tiles of input channels c
    constexpr int MU = CIN == 32 ? MT : 1;       // tiles of n in a unit
    constexpr int NU = 5;                        // units per wave (18 over 4 waves)
    constexpr int NCOL = 9;
    extern __shared__ __attribute__((aligned(16))) u16 ws[];
    u16* gT = ws;                                // [MT*16][kGtStride]
    u16* xT = ws + MT * 16 * kGtStride;          // [NT*16][kXtStride]
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, gq = lane >> 4;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    // padding channels stay zero
    if constexpr (MT * 16 > COUTP)
        for (int e = tid; e < (MT * 16 - COUTP) * kGtStride; e += kBlock) gT[COUTP * kGtStride + e] = 0;
    if constexpr (NT * 16 > CIN)
        for (int e = tid; e < (NT * 16 - CIN) * kXtStride; e += kBlock) xT[CIN * kXtStride + e] = 0;
    f32x4 acc[NU][3][MU];
#pragma unroll
    for (int j = 0; j < NU; ++j)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int mt = 0; mt < MU; ++mt) acc[j][dx][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bacc = 0.f;
    const int nbx = nx / kCbX, nby = (ny + kCbY - 1) / kCbY, nbz = (nz + kCbZ - 1) / kCbZ;
    const int nblocks = nbx * nby * nbz * g.batch;
    // each workgroup takes a contiguous range of blocks, z fastest: consecutive
    // blocks share two of their four halo planes, which are still in cache
    const int per = (nblocks + gridDim.x - 1) / gridDim.x;
    const int blk0 = blockIdx.x * per, blk1 = min(nblocks, blk0 + per);
    // items of 8 channels of a cell pair along x: g of the block, x of the halo block
    constexpr int G8 = COUTP / 8, NG = (kCbCells / 2) * G8, KG = (NG + kBlock - 1) / kBlock;
    constexpr int C8 = CIN / 8, NX = kChZ * kChY * (kChX / 2) * C8, KX = (NX + kBlock - 1) / kBlock;
    u32x4 g0[KG], g1[KG], h0[KX], h1[KX];
    auto fetch = [&](int blk) {
        int L = blk;
        const int bz = L % nbz;
        L /= nbz;
        const int bx = L % nbx;
        L /= nbx;
        const int by = L % nby;
        const int b = L / nby;
        const int x0 = bx * kCbX, y0 = by * kCbY, z0 = bz * kCbZ;
        const int64_t bcell = int64_t(b) * nz * ny * nx;
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const int e = min(k * kBlock + tid, NG - 1);
            const int ch = e % G8, q = 2 * (e / G8), r = q >> 5;
            const int yy = y0 + r % kCbY, zz = z0 + r / kCbY;
            const bool ok = yy < ny && zz < nz;
            const u16* src = gin + (bcell + (int64_t(ok ? zz : z0) * ny + (ok ? yy : y0)) * nx + x0 + (q & 31)) * COUTP + ch * 8;
            g0[k] = *reinterpret_cast<const u32x4*>(src);
            g1[k] = *reinterpret_cast<const u32x4*>(src + COUTP);
            if (!ok) g0[k] = g1[k] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int k = 0; k < KX; ++k) {
            const int e = min(k * kBlock + tid, NX - 1);
            const int ch = e % C8, pr = e / C8;
            const int hrow = pr / (kChX / 2), hx = 2 * (pr - hrow * (kChX / 2));
            const int hz = hrow / kChY, hy = hrow - hz * kChY;
            const int64_t rowc = bcell + (int64_t(wrap_near(z0 - 1 + hz, nz)) * ny + wrap_near(y0 - 1 + hy, ny)) * nx;
            h0[k] = *reinterpret_cast<const u32x4*>(xin + (rowc + wrapi(x0 - 1 + hx, nx)) * CIN + ch * 8);
            h1[k] = *reinterpret_cast<const u32x4*>(xin + (rowc + wrapi(x0 + hx, nx)) * CIN + ch * 8);
        }
    };
    // 8 channels of a cell pair -> 8 rows of dst, one 32-bit store each
    auto spread = [&](auto chans, const u32x4& lo, const u32x4& hi, u16* dst, int stride) {
        constexpr int C = decltype(chans)::value;
        const unsigned a[4] = {lo.x, lo.y, lo.z, lo.w}, c[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *reinterpret_cast<unsigned*>(dst + chan_row<C>(0, 2 * i) * stride) = __builtin_amdgcn_perm(c[i], a[i], 0x05040100u);
            *reinterpret_cast<unsigned*>(dst + chan_row<C>(0, 2 * i + 1) * stride) = __builtin_amdgcn_perm(c[i], a[i], 0x07060302u);
        }
    };
    // offsets of this wave's units in xT (B operand) and gT (A operand)
    int xo[NU], go[NU];
#pragma unroll
    for (int j = 0; j < NU; ++j) {
        const int u = min(wave + 4 * j, 2 * NCOL - 1), half = u / NCOL, col = u - half * NCOL;
        xo[j] = ((col / 3) * kChY + col % 3) * kXtRow + (CIN == 32 ? half * 16 * kXtStride : 0);
        go[j] = CIN == 32 ? 0 : half * 16 * kGtStride;
    }
    if (blk0 < blk1) fetch(blk0);
    for (int blk = blk0; blk < blk1; ++blk) {
        __syncthreads();  // the previous block's operands are no longer read
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const int e = k * kBlock + tid;
            if (e < NG) spread(std::integral_constant<int, COUTP>{}, g0[k], g1[k], gT + (e % G8) * 4 * kGtStride + 2 * (e / G8), kGtStride);
        }
#pragma unroll
        for (int k = 0; k < KX; ++k) {
            const int e = k * kBlock + tid;
            const int pr = e / C8, hrow = pr / (kChX / 2);
            if (e < NX)
                spread(std::integral_constant<int, CIN>{}, h0[k], h1[k],
                       xT + (e % C8) * 4 * kXtStride + hrow * kXtRow + 2 * (pr - hrow * (kChX / 2)), kXtStride);
        }
        __syncthreads();
        fetch(min(blk + 1, blk1 - 1));
        // bias: thread (row tid mod 32, part = tid / 32) sums cells part*32 .. +31 of its channel
        if ((tid & 31) < COUTP) {
            const u16* row = gT + (tid & 31) * kGtStride + (tid >> 5) * 32;
#pragma unroll
            for (int q = 0; q < 32; q += 8) {
                const uint4 v = *reinterpret_cast<const uint4*>(row + q);
                const unsigned w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) bacc += bf16_val(u16((w4[i >> 1] >> ((i & 1) * 16)) & 0xffffu));
            }
        }
#pragma unroll 1
        for (int r = 0; r < kCbY * kCbZ; ++r) {
            const int yy = r % kCbY, zz = r / kCbY;
            const u16* gr = gT + lm * kGtStride + r * 32 + 8 * gq;
            const u16* xr = xT + lm * kXtStride + (zz * kChY + yy) * kXtRow + 8 * gq;
            bf16x8 av[MU];
            if constexpr (CIN == 32)
#pragma unroll
                for (int mt = 0; mt < MU; ++mt) av[mt] = *reinterpret_cast<const bf16x8*>(gr + mt * 16 * kGtStride);
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                if (wave + 4 * j >= 2 * NCOL) continue;
                if constexpr (CIN != 32) av[0] = *reinterpret_cast<const bf16x8*>(gr + go[j]);
                const uint4 c = *reinterpret_cast<const uint4*>(xr + xo[j]);
                const unsigned d[5] = {c.x, c.y, c.z, c.w, *reinterpret_cast<const unsigned*>(xr + xo[j] + 8)};
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    unsigned o[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        o[i] = dx == 1 ? __builtin_amdgcn_alignbyte(d[i + 1], d[i], 2u) : d[i + dx / 2];
                    const bf16x8 bv = __builtin_bit_cast(bf16x8, (uint4{o[0], o[1], o[2], o[3]}));
#pragma unroll
                    for (int mt = 0; mt < MU; ++mt)
                        acc[j][dx][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[mt], bv, acc[j][dx][mt], 0, 0, 0);
                }
            }
        }
    }
    // partial layout per workgroup: [n (COUTP)][tap][c (CIN)] then bias [COUTP]
    float* out = partial + int64_t(blockIdx.x) * (COUTP * kTaps * CIN + COUTP);
#pragma unroll
    for (int j = 0; j < NU; ++j) {
        const int u = wave + 4 * j, half = u / NCOL, col = u - half * NCOL;
        if (u >= 2 * NCOL) continue;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int mt = 0; mt < MU; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int n = (CIN == 32 ? mt : half) * 16 + 4 * gq + i, c = (CIN == 32 ? half : 0) * 16 + lm;
                    if (n < COUTP && c < CIN)
                        out[(row_chan<COUTP>(n) * kTaps + col * 3 + dx) * CIN + row_chan<CIN>(c)] = acc[j][dx][mt][i];
                }
    }
    // the eight partial bias sums of each channel, added in part order
    __syncthreads();
    float* red = reinterpret_cast<float*>(ws);
    red[tid] = bacc;
    __syncthreads();
    if (tid < COUTP) {
        float sum = 0.f;
#pragma unroll
        for (int part = 0; part < kBlock / 32; ++part) sum += red[part * 32 + tid];
        out[COUTP * kTaps * CIN + row_chan<COUTP>(tid)] = sum;
    }
}

template <int CIN, int COUTP>
constexpr size_t wgrad_t_lds_bytes() {
    return (size_t((COUTP == 32 ? 2 : 1) * 16) * kGtStride + size_t((CIN == 32 ? 2 : 1) * 16) * kXtStride) * 2;
}

// theta_bar += sum over workgroups of the partials, in a fixed order (deterministic).
// Partial layout [n < coutp][tap][c < cinp] then bias [coutp]; only the real
// channels (n < cout, c < cin) map to W[o = n][i = c][tap] and b[o].
// A workgroup takes 64 values; its 16 groups of 64 threads each add every 16th
// partial row, then the groups' sums are added in order. Bound by one read of the
// partials (512 rows, 57 MB for the 32 -> 32 layer): one thread per value walking
// all rows took 126 us per layer (4 x 128^3), 1.5 of a training step's 40.5 ms.
constexpr int kReduceRows = 16;
__global__ __launch_bounds__(64 * kReduceRows) void k_wgrad_reduce(const float* __restrict__ partial, int nwg, int cinp,
                                                                   int coutp, int cin, int cout,
                                                                   float* __restrict__ wbar, float* __restrict__ bbar) {
    __shared__ double sh[kReduceRows][64];
    const int per = coutp * kTaps * cinp + coutp;
    const int l = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + l;
    double s = 0.0;
    if (e < per) {
#pragma unroll 4
        for (int w = q; w < nwg; w += kReduceRows) s += partial[int64_t(w) * per + e];
    }
    sh[q][l] = s;
    __syncthreads();
    if (q != 0 || e >= per) return;
    s = 0.0;
#pragma unroll
    for (int i = 0; i < kReduceRows; ++i) s += sh[i][l];
    if (e < coutp * kTaps * cinp) {
        const int c = e % cinp, tap = (e / cinp) % kTaps, n = e / (cinp * kTaps);
        if (n < cout && c < cin) wbar[(n * cin + c) * kTaps + tap] += float(s);
    } else {
        const int n = e - coutp * kTaps * cinp;
        if (n < cout) bbar[n] += float(s);
    }
}

// ----------------------------------------------------------------------------
// Launchers
// ----------------------------------------------------------------------------
template <typename T>
hipError_t launch_closure_pack_input(const Grid& g, const T* w, const double* p, u16* x0, hipStream_t s) {
    const dim3 grid(int((g.ncell * g.batch + kBlock - 1) / kBlock));
    if (p)
        hipLaunchKernelGGL((k_pack_input<T, true>), grid, dim3(kBlock), 0, s, g, w, p, x0);
    else
        hipLaunchKernelGGL((k_pack_input<T, false>), grid, dim3(kBlock), 0, s, g, w, p, x0);
    return hipGetLastError();
}

hipError_t launch_closure_pack_weights(const float* w, int cin, int cout, int cinp, int ntf, u16* wf, int coutp, int ntd,
                                       u16* wd, hipStream_t s) {
    const int tot = ((kTaps * cinp + 31) / 32) * ntf * 512 + ((kTaps * coutp + 31) / 32) * ntd * 512;
    hipLaunchKernelGGL(k_pack_weights, dim3((tot + 255) / 256), dim3(256), 0, s, w, cin, cout, cinp, ntf, wf, coutp, ntd, wd);
    return hipGetLastError();
}

// layer: 0 = 8 -> 32 hidden, 1 = 32 -> 32 hidden, 2 = 32 -> 3 output;
// dgrad: 10 = 8 -> 32 (cotangent of m into the last hidden layer), 11 = 32 -> 32,
// 12 = 32 -> 3 input gradient.
template <typename T>
hipError_t launch_closure_conv(const Grid& g, int which, const u16* in, const u16* wpk, const float* bias,
                               const float* zin, float* zout, u16* aout, T* fout, hipStream_t s) {
#define INS_CONV(CIN, NT, EPI, NOUT)                                                                                \
    do {                                                                                                            \
        constexpr int BZ = CIN == 32 && NT == 2 ? 4 : 2;                                                  \
        const int nblk = (g.nx / kCbX) * ((g.ny + kCbY - 1) / kCbY) * ((g.nz + BZ - 1) / BZ) * g.batch;            \
        const int grid = conv_walks<CIN, NT>() && nblk > kWalkGroups ? kWalkGroups : nblk;                          \
        const size_t shm = conv_t_lds_bytes<CIN, BZ>(EPI == EPI_HIDDEN || EPI == EPI_DGRAD_HIDDEN);                         \
        hipLaunchKernelGGL((k_conv_t<T, CIN, NT, EPI, BZ>), dim3(grid), dim3(kBlock), shm, s, g, in, wpk, bias, zin, \
                           zout, aout, fout, NOUT);                                                                 \
    } while (0)
    switch (which) {
        case 0: INS_CONV(8, 2, EPI_HIDDEN, 32); break;
        case 1: INS_CONV(32, 2, EPI_HIDDEN, 32); break;
        case 2: INS_CONV(32, 1, EPI_OUT, 3); break;
        case 10: INS_CONV(8, 2, EPI_DGRAD_HIDDEN, 32); break;
        case 11: INS_CONV(32, 2, EPI_DGRAD_HIDDEN, 32); break;
        default: INS_CONV(32, 1, EPI_DGRAD_INPUT, 3); break;
    }
#undef INS_CONV
    return hipGetLastError();
}

int wgrad_grid(int64_t ncells) {
    const int64_t nstrip = ncells / 32;
    return int(nstrip < 512 ? nstrip : 512);
}

// which: 0 = layer 1 (g: 32 ch, x: 8 packed ch of which 3 real), 1 = layer 2 (32, 32),
// 2 = layer 3 (g: 8 packed ch of which 3 real, x: 32 ch). wbar/bbar point at the
// layer's weights and bias inside the flat parameter gradient.
hipError_t launch_closure_wgrad(const Grid& g, int which, const u16* gin, const u16* xin, float* partial, float* wbar,
                                float* bbar, hipStream_t s) {
    const int64_t n = int64_t(g.nx) * g.ny * g.nz * g.batch;
    const int grid = wgrad_grid(n);
    int cinp, coutp, cin, cout;
    constexpr size_t shm0 = wgrad_t_lds_bytes<8, 32>(), shm1 = wgrad_t_lds_bytes<32, 32>(),
                     shm2 = wgrad_t_lds_bytes<32, 8>();
    if (which == 0) {
        hipLaunchKernelGGL((k_wgrad_t<8, 32>), dim3(grid), dim3(kBlock), shm0, s, g, gin, xin, partial);
        cinp = 8, coutp = 32, cin = 3, cout = 32;
    } else if (which == 1) {
        hipLaunchKernelGGL((k_wgrad_t<32, 32>), dim3(grid), dim3(kBlock), shm1, s, g, gin, xin, partial);
        cinp = 32, coutp = 32, cin = 32, cout = 32;
    } else {
        hipLaunchKernelGGL((k_wgrad_t<32, 8>), dim3(grid), dim3(kBlock), shm2, s, g, gin, xin, partial);
        cinp = 32, coutp = 8, cin = 32, cout = 3;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int per = coutp * kTaps * cinp + coutp;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((per + 63) / 64), dim3(64 * kReduceRows), 0, s, partial, grid, cinp, coutp,
                       cin, cout, wbar, bbar);
    return hipGetLastError();
}

// Partial-sum floats needed by launch_closure_wgrad for a grid of n cells.
size_t closure_wgrad_partial_floats(int64_t ncells) {
    return size_t(wgrad_grid(ncells)) * (32 * kTaps * 32 + 32);
}

template hipError_t launch_closure_pack_input<double>(const Grid&, const double*, const double*, u16*, hipStream_t);
template hipError_t launch_closure_pack_input<float>(const Grid&, const float*, const double*, u16*, hipStream_t);
template hipError_t launch_closure_conv<double>(const Grid&, int, const u16*, const u16*, const float*, const float*,
                                                float*, u16*, double*, hipStream_t);
template hipError_t launch_closure_conv<float>(const Grid&, int, const u16*, const u16*, const float*, const float*,
                                               float*, u16*, float*, hipStream_t);

}  // namespace ins
