// Work split and access helpers of the z-marching 3D stencils (stages and reverse stages).
#pragma once

#include "k_common.hpp"

namespace ins {

// Workgroups of NT threads of kernel K that the device holds at once (a constant
// of the kernel and the device; asked once).
template <auto K, int NT>
int resident_groups() {
    static const int n = [] {
        int dev = 0, cus = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(K), NT, 0) != hipSuccess) {
            (void)hipGetLastError();
            return 512;
        }
        return per * cus > 0 ? per * cus : 512;
    }();
    return n;
}

// z planes per workgroup of a z-march over tx x ty tiles, `slots` workgroups
// resident at once. A workgroup of zc planes takes about zc + 2 halo planes + 3
// for its unoverlapped start, and ceil(workgroups / slots) of them run one after
// the other: the split with the least product, at most zmax planes. (A rule that
// halved the chunk until there were `slots` workgroups gave a 2 x 150 x 126 x 98
// field 672 workgroups on 512 slots, a second round a third full: its stages
// 98 -> 80 us, a step 743 -> 677 us; 192 x 160 x 144 973 -> 903 us; powers of
// two keep their split.) A reverse stage takes at most 32 planes (64: 3 % slower
// at 256^3).
inline int zm_chunk(const Grid& g, int tx, int ty, int slots, int zmax) {
    const int64_t tiles = int64_t((g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty) * g.batch;
    int best = 1;
    int64_t cost = -1;
    for (int m = (g.nz + zmax - 1) / zmax; m <= g.nz; ++m) {
        const int zc = (g.nz + m - 1) / m;
        if (zc < 2 && cost >= 0) break;
        const int64_t groups = tiles * ((g.nz + zc - 1) / zc);
        const int64_t c = (groups + slots - 1) / slots * (zc + 5);
        if (cost < 0 || c < cost) {
            cost = c;
            best = zc;
        }
    }
    return best;
}

__device__ __forceinline__ int pmod(int v, int n) {
    const int r = v % n;
    return r < 0 ? r + n : r;
}

// Streams touched exactly once per step (u0, y, the new stage register) bypass
// the caches' normal allocation.
template <typename T>
__device__ __forceinline__ T ld_stream(const T* p) {
    return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void st_stream(T v, T* p) {
    __builtin_nontemporal_store(v, p);
}

}  // namespace ins
