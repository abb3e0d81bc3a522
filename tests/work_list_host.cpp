// The work list of the expert FFN kernels (ffn_plan.h) on the CPU: the block's 256 threads are threads of this process.  Standard input: cases of
// "e_count tile_m total_rows max_tiles offsets[0..e_count]"; output per case: the number of tiles and their four numbers each.
#include <hip/hip_runtime.h>
#include <pthread.h>

#include <algorithm>
#include <cstdio>
#include <thread>
#include <vector>

using std::max;
using std::min;
struct Index { int x; };
static thread_local Index threadIdx;
static const Index blockDim{256};
static pthread_barrier_t barrier, wave_barrier[4];
static void __syncthreads() { pthread_barrier_wait(&barrier); }
static int __shfl_up(int v, int off) {          // all 64 threads of a wave call it
    static int values[256];
    const int t = threadIdx.x;
    values[t] = v;
    pthread_barrier_wait(&wave_barrier[t / 64]);
    const int got = t % 64 >= off ? values[t - off] : v;
    pthread_barrier_wait(&wave_barrier[t / 64]);
    return got;
}
static unsigned long long __ballot(int) { return 0; }      // (named by a function of common.h that is not called here)

#include "ffn_plan.h"

int main() {
    pthread_barrier_init(&barrier, nullptr, 256);
    for (auto& b : wave_barrier) pthread_barrier_init(&b, nullptr, 64);
    int e_count, tile_m, total_rows, max_tiles;
    while (std::scanf("%d %d %d %d", &e_count, &tile_m, &total_rows, &max_tiles) == 4) {
        std::vector<int> offsets(e_count + 1), plan(moe::kPlanHeader + 4 * static_cast<size_t>(max_tiles), -1);
        for (int& v : offsets)
            if (std::scanf("%d", &v) != 1) return 1;
        alignas(16) static int scratch[moe::kPlanScratch][256];
        std::vector<std::thread> block;
        for (int t = 0; t < 256; ++t)
            block.emplace_back([&, t] {
                threadIdx.x = t;
                moe::ffn_plan_block(offsets.data(), 0, e_count, tile_m, plan.data(), total_rows, max_tiles, scratch, 0);
            });
        for (auto& th : block) th.join();
        std::printf("%d", plan[16]);
        for (int i = 0; i < 4 * plan[16]; ++i) std::printf(" %d", plan[moe::kPlanHeader + i]);
        std::printf("\n");
    }
}
