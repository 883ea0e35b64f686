// The tile staging of split_device.h by a workgroup of several waves, as the
// evaluator uses it: the tile as bytes, and, where a demand is past a byte,
// the same LDS staged again as int16, half of the scenarios at a time.  Each
// lane is a thread, so a thread sanitizer sees every pair of accesses to the
// rows or the flag word that no barrier orders.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <thread>
#include <vector>

#include "split_device.h"

thread_local Index3 threadIdx, blockIdx, blockDim, gridDim;
thread_local HostWave *host_wave;
pthread_barrier_t host_group;

#define EXPECT(c)                                                                                \
    do {                                                                                         \
        if (!(c)) {                                                                              \
            fprintf(stderr, "line %d, wave %u: %s\n", __LINE__, threadIdx.x / 64, #c);            \
            abort();                                                                             \
        }                                                                                        \
    } while (0)

using namespace splitk;

struct Tile {
    int N, rows;
    std::vector<int16_t> demands;
    bool byte_ok, half_ok[2];
};

static void lane_main(const Tile &t, int tid, int waves, HostWave *wave, uint8_t *lds, int &flag)
{
    threadIdx = {(unsigned)tid, 0, 0};
    blockDim = {64u * waves, 1, 1};
    host_wave = wave;
    const int threads = 64 * waves;
    const bool ok = stage_tile_u8(t.demands.data(), lds, (int64_t)t.rows * t.N, tid, threads, flag);
    (void)ballot(true); // the lanes of a wave leave the call together; waves do not
    EXPECT(ok == t.byte_ok);
    if (ok) {
        for (int i = tid; i < t.rows * t.N; i += threads)
            EXPECT(lds[i] == t.demands[i]);
        return;
    }
    for (int h = 0; h < 2; ++h) {
        const int rh = t.rows - 32 * h < 0 ? 0 : t.rows - 32 * h > 32 ? 32 : t.rows - 32 * h;
        const int16_t *src = t.demands.data() + (rh ? 32 * h * t.N : 0);
        const bool clean = stage_rows_i16(src, lds, (int64_t)rh * t.N, tid, threads, flag);
        (void)ballot(true);
        EXPECT(clean == t.half_ok[h]);
        const int16_t *row = reinterpret_cast<const int16_t *>(lds);
        for (int i = tid; i < rh * t.N; i += threads)
            EXPECT(row[i] == src[i]);
        __syncthreads();
    }
}

static void run(const Tile &t, int waves)
{
    std::vector<HostWave> w(waves);
    for (HostWave &x : w)
        pthread_barrier_init(&x.barrier, nullptr, 64);
    pthread_barrier_init(&host_group, nullptr, 64 * waves);
    std::vector<uint64_t> lds(((size_t)64 * t.N + 15) / 16 * 2 + 2);
    int flag = 0;
    std::vector<std::thread> lanes;
    for (int i = 0; i < 64 * waves; ++i)
        lanes.emplace_back([&, i] {
            lane_main(t, i, waves, &w[i / 64], reinterpret_cast<uint8_t *>(lds.data()), flag);
        });
    for (std::thread &l : lanes)
        l.join();
    pthread_barrier_destroy(&host_group);
    for (HostWave &x : w)
        pthread_barrier_destroy(&x.barrier);
}

int main()
{
    for (int waves : {2, 4, 1})
        for (int rows : {64, 33, 7}) {
            Tile t;
            t.N = 37;
            t.rows = rows;
            t.demands.resize((size_t)rows * t.N);
            for (size_t i = 0; i < t.demands.size(); ++i)
                t.demands[i] = (int16_t)(i % 251);
            t.byte_ok = t.half_ok[0] = t.half_ok[1] = true;
            run(t, waves);
            t.demands[5] = 256; // past a byte
            t.byte_ok = false;
            run(t, waves);
            t.demands[t.demands.size() - 2] = -1;
            t.half_ok[rows > 32] = false;
            run(t, waves);
        }
    puts("all expectations met");
    return 0;
}
