// split_values.hip -- the full value table of one giant tour over every
// scenario: V_s(j) for j = 1..n (paper Sec. 2.3 recursion; the batched DP
// of App. A returns the value array over positions and scenarios, not only
// V_s(n)).
//
// One wave per tile of 64 scenarios, one scenario per lane: the evaluator's
// pruned-stack recursion over the tile staged in LDS (bytes, or int16 half a
// tile at a time), which writes V_s(j) = m_j + b_j as it goes.  The output is
// position-major (V[(j-1)*S + s]), so a wave writes one coalesced row per
// position.  What bounds it: the evaluator's recursion plus the stores (the
// table is written once and never read).  The definition walked per cell
// (values_exact_column) reads one demand and one value per cell through
// memory: n = 100, S = 1e5 took 690 us (25 us now; its bytes take 12.6),
// n = 200, S = 1e6 51 ms.
//
// Tiles whose windows leave the ring or that hold a negative demand are
// recomputed from the definition (listed for a kernel of their own where the
// call has more tiles than the chip holds at once), as are calls whose tile does
// not fit in LDS or whose demands are not 16-byte aligned.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "split_device.h"
#include "split_stack.h"
#include "split_eval.h"
#include "split_internal.h"
#include "split_values.h"

namespace splitk {

namespace {

// V of one scenario from the definition: for each position j the lane walks
// its predecessors p = j-1, j-2, ... while the route load stays within Q,
// reading V_s(p) back from its own column of the output.
__device__ __forceinline__ void values_exact_column(const int16_t *__restrict__ demands, int32_t N,
                                                    int64_t S, int32_t Q, const Workspace &ws,
                                                    int32_t *__restrict__ V,
                                                    int32_t *__restrict__ status, int64_t s)
{
    const TourRec rec = ws.rec[0];
    const int n = rec.n;
    if (s >= S)
        return;
    if (rec.status != ST_OK) {
        for (int j = 1; j <= n; ++j)
            V[(int64_t)(j - 1) * S + s] = SPLIT_INF;
        return;
    }
    // (scalar loads, which plain pointers would lose after the stores of the
    // tile's first attempt: n = 200, S = 5e4, windows of 80: 9.6 ms)
    CInt *tab = (CInt *)ws.tab; // {customer index, c_j}, entry j = position j
    CInt *ab = (CInt *)ws.ab;   // {a_k, b_k}, entry k-1 = position k
    const int16_t *__restrict__ row = demands + s * N;
    bool neg = false;
    for (int j = 1; j <= n; ++j) {
        const int bj = tab_at(ab, j - 1).y;
        int best = SPLIT_INF;
        int load = 0;
        for (int p = j - 1; p >= 0; --p) {
            const int q = row[tab_at(tab, p + 1).x];
            neg = neg || q < 0;
            load += q;
            if (load > Q) // demands are non-negative: every longer route is too heavy
                break;
            const int vp = p == 0 ? 0 : V[(int64_t)(p - 1) * S + s];
            if (vp != SPLIT_INF)
                best = min(best, vp + tab_at(ab, p).x + bj); // V(p) + W(p, j)
        }
        V[(int64_t)(j - 1) * S + s] = best;
    }
    if (neg) {
        for (int j = 1; j <= n; ++j)
            V[(int64_t)(j - 1) * S + s] = SPLIT_INF;
        atomicOr(status, 1);
    }
}

__global__ __launch_bounds__(kWave) void values_exact_kernel(const int16_t *__restrict__ demands,
                                                             int32_t N, int64_t S, int32_t Q,
                                                             Workspace ws,
                                                             int32_t *__restrict__ V,
                                                             int32_t *__restrict__ status)
{
    values_exact_column(demands, N, S, Q, ws, V, status,
                        (int64_t)blockIdx.x * kWave + threadIdx.x);
}

__global__ __launch_bounds__(kWave) void values_listed_kernel(const int16_t *__restrict__ demands,
                                                              int32_t N, int64_t S, int32_t Q,
                                                              Workspace ws,
                                                              int32_t *__restrict__ V,
                                                              int32_t *__restrict__ status)
{
    const int count = *ws.list_count;
    for (int li = blockIdx.x; li < count; li += gridDim.x)
        values_exact_column(demands, N, S, Q, ws, V, status,
                            (int64_t)ws.list[li] * kWave + threadIdx.x);
}

// The last row, and SPLIT_INF from the first position whose demand alone
// exceeds Q (every later prefix is infeasible too) for a lane with no split.
template <class T>
__device__ __forceinline__ void finish_column(const T *row, CInt *tab, int n, int Q, int v,
                                              int32_t *col, int64_t S)
{
    if (v < kInf) {
        col[(int64_t)(n - 1) * S] = v;
        return;
    }
    int j = 1;
    while (j < n && (int)row[tab_at(tab, j).x] <= Q)
        ++j;
    for (; j <= n; ++j)
        col[(int64_t)(j - 1) * S] = SPLIT_INF;
}

// grid = tiles, one wave each; LDS: 64 x N demand bytes, or (pitch > 0) the
// tour's demands gathered, 64 x pitch bytes.  Tiles to be redone are listed, or
// (alone) recomputed here.
template <int R>
__global__ __launch_bounds__(kWave) void values_tile_kernel(const int16_t *__restrict__ demands,
                                                            int32_t N, int64_t S, int32_t Q,
                                                            int32_t pitch,
                                                            const int2 *__restrict__ pos,
                                                            int32_t alone, Workspace ws,
                                                            int32_t *__restrict__ V,
                                                            int32_t *__restrict__ status)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int64_t k = blockIdx.x;
    const int lane = threadIdx.x;
    const int64_t s0 = k * kWave;
    const int rows = (int)min<int64_t>(kWave, S - s0);
    const TourRec rec = ws.rec[0];
    const int n = rec.n;
    const int stride = pitch ? pitch : N;
    int unused = 0; // (one wave stages: no flag word)
    const bool ok =
        pitch ? stage_gather<uint8_t, true>(demands + s0 * N, N, rows, ws.tab, n, pitch, lds, lane,
                                            kWave, unused)
              : stage_tile_u8<kStageBatch, true>(demands + s0 * N, lds, (int64_t)rows * N, lane,
                                                 kWave, unused);
    if (rec.status != ST_OK) {
        if (lane < rows)
            for (int j = 1; j <= n; ++j)
                V[(int64_t)(j - 1) * S + s0 + lane] = SPLIT_INF;
        return;
    }
    CInt *tab = (CInt *)(pitch ? pos : ws.tab);
    const StackTable table{V + s0, (uint64_t)S * sizeof(int32_t), 4u * (uint32_t)lane, ws.ab};
    int32_t *col = V + s0 + lane;
    const uint32_t base = (uint32_t)(uintptr_t)(const LdsByte *)lds;
    bool redo = false;
    if (ok) {
        bool ovf = false;
        if (lane < rows) {
            const int v = stack_lane_values<R, false>(base + (uint32_t)(lane * stride), tab, n, rec.f0,
                                                      byte_capacity(Q, n), table, ovf) +
                          rec.bn;
            if (!ovf)
                finish_column(lds + (int64_t)lane * stride, tab, n, Q, v, col, S);
        }
        redo = ballot(ovf) != 0;
    } else {
        redo = n > kWideMaxLen;
        for (int h = 0; h < 2 && !redo; ++h) {
            const int rh = min(max(rows - 32 * h, 0), 32);
            if (rh == 0)
                break;
            const int16_t *src = demands + (s0 + 32 * h) * N;
            const bool clean =
                pitch ? stage_gather<int16_t, true>(src, N, rh, ws.tab, n, pitch,
                                                    reinterpret_cast<int16_t *>(lds), lane, kWave,
                                                    unused)
                      : stage_rows_i16<kStageBatch, true>(src, lds, (int64_t)rh * N, lane, kWave,
                                                          unused);
            if (!clean) {
                redo = true; // a negative demand
                break;
            }
            bool ovf = false;
            if ((lane >> 5) == h && (lane & 31) < rh) {
                const uint32_t off = (uint32_t)((lane & 31) * stride * 2);
                const int v = stack_lane_values<32, true>(base + off, tab, n, rec.f0,
                                                          wide_capacity(Q, n), table, ovf) +
                              rec.bn;
                if (!ovf)
                    finish_column(reinterpret_cast<const int16_t *>(lds + off), tab, n, Q, v, col,
                                  S);
            }
            redo = ballot(ovf) != 0;
        }
    }
    if (redo && alone)
        values_exact_column(demands, N, S, Q, ws, V, status, s0 + lane);
    else if (redo && lane == 0) {
        const int slot = atomicAdd(ws.list_count, 1);
        ws.list[slot] = (int)k;
    }
}

size_t values_lds_bytes(int32_t N, int32_t pitch)
{
    return ((size_t)kTile * (size_t)(pitch ? pitch : N) + 15) & ~(size_t)15;
}

template <int R>
hipError_t launch_values_tiles(const int16_t *demands, int32_t N, int64_t S, int32_t Q,
                               int32_t pitch, const int2 *pos, int32_t alone, const Workspace &ws,
                               int32_t *V, int32_t *status, hipStream_t stream)
{
    static std::mutex mu;
    static uint64_t ready = 0; // devices whose limit is set
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (dev >= 64 || !(ready >> dev & 1)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&values_tile_kernel<R>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
            if (e != hipSuccess)
                return e;
            if (dev < 64)
                ready |= 1ull << dev;
        }
    }
    hipLaunchKernelGGL(values_tile_kernel<R>, dim3((unsigned)num_tiles(S)), dim3(kWave),
                       values_lds_bytes(N, pitch), stream, demands, N, S, Q, pitch, pos,
                       alone, ws, V, status);
    return hipGetLastError();
}

// The tour's demands are gathered, a line of the row for a few of them, where
// whole rows would be many times as much: us rows / gathered, S = 6e7 / N (at
// most 1e5), Q = 60: n = 5, N = 400 24 / 18, N = 2000 54 / 16; n = 20, N = 200
// 16.0 / 19.3, N = 400 27 / 24, N = 2000 57 / 19; n = 100, N = 400 45.6 / 43.3,
// N = 2000 76 / 47; n = 200, N = 1000 85 / 88; n = 400, N = 1000 132 / 165,
// N = 2500 158 / 139.
bool gather_values(int32_t n, int32_t N) { return N > 256 && 6 * (int64_t)n <= N; }

constexpr int kWavesPerUnit = 12; // three per SIMD, by the kernel's registers

// Waves that share the listed tiles: as many one-wave workgroups as the chip
// holds, so that a call whose every tile is listed keeps the whole chip busy.
constexpr int kValuesListBlocks = kComputeUnits * 32;

} // namespace

hipError_t launch_values(const int32_t *tour, int32_t n, const int32_t *dist, int32_t N,
                         const int16_t *demands, int64_t S, int32_t Q, int32_t *V,
                         int32_t *status, const Workspace &ws, hipStream_t stream)
{
    // the table by position takes the fallback's value history, not used here
    int2 *pos = reinterpret_cast<int2 *>(ws.vscratch);
    const int32_t pitch = gather_values(n, N) ? n + 1 : 0;
    hipError_t e =
        launch_prep(tour, nullptr, 1, n, dist, N, ws, stream, pitch ? pos : nullptr, status);
    if (e != hipSuccess || n == 0)
        return e;
    const int64_t tiles = num_tiles(S);
    if (values_lds_bytes(N, 0) > (size_t)kLdsLimit || reinterpret_cast<uintptr_t>(demands) % 16) {
        hipLaunchKernelGGL(values_exact_kernel, dim3((unsigned)tiles), dim3(kWave), 0, stream,
                           demands, N, S, Q, ws, V, status);
        return hipGetLastError();
    }
    // where every tile is on the chip at once, a tile to be redone keeps its
    // wave, and the call one launch less (about 2 us)
    const int64_t per_cu = std::min<int64_t>(kLdsLimit / values_lds_bytes(N, pitch), kWavesPerUnit);
    const int32_t alone = tiles <= per_cu * kComputeUnits ? 1 : 0;
    e = Q > 200
            ? launch_values_tiles<64>(demands, N, S, Q, pitch, pos, alone, ws, V, status, stream)
            : launch_values_tiles<32>(demands, N, S, Q, pitch, pos, alone, ws, V, status, stream);
    if (e != hipSuccess || alone)
        return e;
    hipLaunchKernelGGL(values_listed_kernel,
                       dim3((unsigned)(tiles < kValuesListBlocks ? tiles : kValuesListBlocks)),
                       dim3(kWave), 0, stream, demands, N, S, Q, ws, V, status);
    return hipGetLastError();
}

} // namespace splitk
