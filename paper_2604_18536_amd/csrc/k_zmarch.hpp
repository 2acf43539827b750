// Work split and access helpers of the z-marching 3D stencils (stages and reverse stages).
#pragma once

#include "k_common.hpp"

namespace ins {

// Workgroups of NT threads and LDS dynamic bytes of kernel K that the device holds at once (a constant
// of the kernel and the device; asked once).
template <auto K, int NT, int LDS = 0>
int resident_groups() {
    static const int n = [] {
        int dev = 0, cus = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(K), NT, LDS) != hipSuccess) {
            (void)hipGetLastError();
            return 512;
        }
        return per * cus > 0 ? per * cus : 512;
    }();
    return n;
}

// z planes per workgroup of a z-march over tx x ty tiles, `slots` workgroups
// resident at once. A workgroup of zc planes takes about zc + 2 halo planes + 3
// for its unoverlapped start; workgroups beyond `slots` run in further rounds, and a
// workgroup that shares its CU with k - 1 others takes 1 + 0.6 (k - 1) times as long
// (64^3 x 2, float64: 4 planes in 256 workgroups 13.3 us, 2 planes in 512 16.8; tiles of
// 256 threads half that: a reverse step there 397 us with 4 planes, 411 with 8). The
// split with the least product, at most zmax planes. Measured against other splits
// (a float64 step, us): 64^3 x 2 213 (2 planes 224, 8 planes 235), 128^3 8 or 16 planes
// 480 (4: 505, 32: 565), 126 x 150 x 98 8 planes 513 (16: 598), 192 x 160 x 144 903 (a
// rule that halved the chunk until there were `slots` workgroups, 973), 2 x 150 x 126 x
// 98 20 planes 677 (14, a second round a third full: 743). A reverse stage takes at most
// 32 planes (64: 3 % slower at 256^3).
inline int zm_chunk(const Grid& g, int tx, int ty, int slots, int zmax) {
    constexpr int kCus = 256;
    const int64_t tiles = int64_t((g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty) * g.batch;
    // relative time of a round of n workgroups
    const int share = tx * ty > 256 ? 6 : 3;
    auto round = [&](int64_t n) { return n > 0 ? 10 + share * ((n + kCus - 1) / kCus - 1) : 0; };
    int best = 1;
    int64_t cost = -1;
    for (int m = (g.nz + zmax - 1) / zmax; m <= g.nz; ++m) {
        const int zc = (g.nz + m - 1) / m;
        if (zc < 2 && cost >= 0) break;
        const int64_t groups = tiles * ((g.nz + zc - 1) / zc);
        const int64_t c = (groups / slots * round(slots) + round(groups % slots)) * (zc + 5);
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
