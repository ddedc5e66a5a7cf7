// Host emulation of the HIP device-code subset used by grid.hip, for checking
// its indexing on the CPU: a workgroup runs as blockDim.x host threads that
// meet at a std::barrier in __syncthreads(); workgroups run one after
// another; dynamic LDS is one host array whose bytes beyond the launch's
// request are poisoned for AddressSanitizer.  Test use only.
#pragma once
#include <algorithm>
#include <barrier>
#include <cstddef>
#include <thread>
#include <vector>

#include <sanitizer/asan_interface.h>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(x)
#define __shared__
#define __restrict__
#define __align__(n) __attribute__((aligned(n)))

typedef struct mockgrid_stream *hipStream_t;
struct int2 {
    int x, y;
};
struct int4 {
    int x, y, z, w;
};
struct dim3 {
    unsigned x = 1, y = 1, z = 1;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct mockgrid_idx {
    unsigned x = 0, y = 0, z = 0;
};
inline thread_local mockgrid_idx threadIdx, blockIdx;
inline dim3 gridDim, blockDim;
inline std::barrier<> *mockgrid_barrier = nullptr;
inline void __syncthreads() { mockgrid_barrier->arrive_and_wait(); }
using std::max;
using std::min;

constexpr size_t kMockLds = size_t(160) << 10;
namespace hhgr {
extern unsigned char grid_lds[];
}
inline unsigned char *mockgrid_lds() { return hhgr::grid_lds; }

template <typename K, typename... A>
void mockgrid_launch(K kernel, dim3 grid, dim3 block, size_t lds, A... args) {
    unsigned char *l = mockgrid_lds();
    ASAN_UNPOISON_MEMORY_REGION(l, kMockLds);
    for (size_t q = 0; q < kMockLds; q++) l[q] = 0xff;  // NaN: unwritten LDS must not reach a result
    ASAN_POISON_MEMORY_REGION(l + lds, kMockLds - lds);
    gridDim = grid;
    blockDim = block;
    std::barrier<> bar((std::ptrdiff_t)block.x);
    mockgrid_barrier = &bar;
    std::vector<std::thread> th;
    for (unsigned tx = 0; tx < block.x; tx++)
        th.emplace_back([&, tx]() {
            threadIdx.x = tx;
            for (unsigned q = 0; q < grid.x * grid.y * grid.z; q++) {
                blockIdx.x = q % grid.x;
                blockIdx.y = (q / grid.x) % grid.y;
                blockIdx.z = q / (grid.x * grid.y);
                kernel(args...);
                bar.arrive_and_wait();
            }
        });
    for (auto &t : th) t.join();
    ASAN_UNPOISON_MEMORY_REGION(l, kMockLds);
}
#define hipLaunchKernelGGL(K, G, B, L, S, ...) mockgrid_launch(K, G, B, L, __VA_ARGS__)
