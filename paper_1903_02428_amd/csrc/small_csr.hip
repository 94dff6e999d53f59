// The target-sorted CSR of a small edge list in one launch.
//
// A mini-batch of small graphs is a new edge list in every step, and its sort
// is all latency: two radix passes are eight dependent launches (35 us of
// kernels for 14,000 edges) around a few microseconds of work. Here workgroup
// b owns the 64 targets from 64 b on and does the whole job for them: it reads
// every target of the list (108 KB, from L2), keeps the edges of its own in
// edge order, counts those below its targets (the row bound it starts at),
// ranks its own stably by target and writes their slots. Reading the list
// once per workgroup is why the route ends at 16,384 nodes and 24,576 edges
// (256 workgroups, 5 bytes of LDS per edge should all of them meet one
// workgroup). Measured for 3,200 nodes and
// 14,080 edges: 35 us of kernels before, 11 us now (the mini-batch's whole step,
// with its fewer launches and less host work, 76 -> 41 us).
#include "common.hpp"

namespace pyg {
namespace {

constexpr int kOwn = 64;         // targets per workgroup: one per lane of a wavefront
constexpr int kThreads = 1024;
constexpr int kWavesS = kThreads / kWave;
constexpr int64_t kMaxEdges = 24576, kMaxNodes = 16384;

// LDS: edge masks [groups], ids and sorted ids [E] of 2 bytes, targets [E] of 1 byte
size_t small_lds(int64_t E) { return static_cast<size_t>((E + kWave - 1) / kWave * 8 + E * 5 + 16); }

__global__ __launch_bounds__(kThreads) void k_small_csr(const int64_t *__restrict__ src, const int64_t *__restrict__ dst,
                                                        int E, int64_t N, const float *__restrict__ w,
                                                        int64_t *__restrict__ rowptr, int32_t *__restrict__ col,
                                                        int64_t *__restrict__ perm, float *__restrict__ w_out) {
    extern __shared__ uint64_t lds64[];
    const int G = (E + kWave - 1) / kWave;  // groups of 64 edges
    uint64_t *mask = lds64;
    uint16_t *id = reinterpret_cast<uint16_t *>(mask + G);
    uint16_t *sorted = id + E;
    uint8_t *tgt = reinterpret_cast<uint8_t *>(sorted + E);
    __shared__ int s_cnt[kWavesS], s_less[kWavesS], cur[kOwn];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t t0 = (int64_t)blockIdx.x * kOwn;
    const int nt = static_cast<int>((N - t0) < kOwn ? (N - t0) : kOwn);
    if (threadIdx.x < kOwn) cur[threadIdx.x] = 0;

    // this wavefront's contiguous groups: which edges are the workgroup's own,
    // how many lie below its targets
    const int g0 = G * wave / kWavesS, g1 = G * (wave + 1) / kWavesS;
    constexpr int U = 8;
    int mine = 0, less = 0;
    for (int g = g0; g < g1; g += U) {
        int64_t d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = (g + u) * kWave + lane;
            d[u] = (g + u < g1 && e < E) ? dst[e] - t0 : int64_t(kOwn);  // no edge: beyond the targets
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g + u >= g1) break;
            const uint64_t m = __ballot(d[u] >= 0 && d[u] < nt);
            mask[g + u] = m;  // every lane the same value
            mine += __popcll(m);
            less += __popcll(__ballot(d[u] < 0));
        }
    }
    s_cnt[wave] = mine;
    s_less[wave] = less;
    __syncthreads();
    int base = 0, n = 0, first = 0;
    for (int v = 0; v < kWavesS; ++v) {
        if (v < wave) base += s_cnt[v];
        n += s_cnt[v];
        first += s_less[v];
    }
    // the own edges in edge order (ids and targets), counted by target
    for (int g = g0; g < g1; ++g) {
        const uint64_t m = mask[g];
        if (m == 0) continue;
        if ((m >> lane) & 1) {
            const int at = base + __popcll(m & ((uint64_t(1) << lane) - 1));
            const int e = g * kWave + lane;
            const int t = static_cast<int>(dst[e] - t0);
            id[at] = static_cast<uint16_t>(e);
            tgt[at] = static_cast<uint8_t>(t);
            atomicAdd(&cur[t], 1);
        }
        base += __popcll(m);
    }
    __syncthreads();
    if (wave == 0) {
        // row bounds, then every edge's place: 64 edges at a time in order,
        // equal targets matched by ballots over the six target bits
        const int c = cur[lane];
        int incl = c;
        for (int off = 1; off < kWave; off <<= 1) {
            const int y = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += y;
        }
        if (lane < nt) rowptr[t0 + lane] = first + incl - c;
        if (lane == 0 && t0 + kOwn >= N) rowptr[N] = E;
        cur[lane] = incl - c;
        __builtin_amdgcn_wave_barrier();
        for (int k = 0; k < n; k += kWave) {
            const bool on = k + lane < n;
            const int t = on ? tgt[k + lane] : 0;
            uint64_t m = __ballot(on);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const uint64_t bb = __ballot((t >> b) & 1);
                m &= ((t >> b) & 1) ? bb : ~bb;
            }
            const int rank = __popcll(m & ((uint64_t(1) << lane) - 1));
            const int at = on ? cur[t] : 0;
            __builtin_amdgcn_wave_barrier();  // every lane has read the counter before its group's first lane moves it
            if (on) {
                sorted[at + rank] = id[k + lane];
                if (rank == 0) cur[t] = at + __popcll(m);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kThreads) {
        const int e = sorted[i];
        const int64_t slot = (int64_t)first + i;
        perm[slot] = e;
        col[slot] = static_cast<int32_t>(src[e]);
        if (w) w_out[slot] = w[e];
    }
}

}  // namespace

bool small_csr_ok(int64_t E, int64_t N) { return E > 0 && E <= kMaxEdges && N > 0 && N <= kMaxNodes; }

int small_csr(const int64_t *src, const int64_t *dst, int64_t E, int64_t N, const float *w, int64_t *rowptr,
              int32_t *col, int64_t *perm, float *w_out, hipStream_t s) {
    const size_t lds = small_lds(E);
    if (lds > 60 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(k_small_csr), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(small_lds(kMaxEdges))) != hipSuccess)
        return PYG_ERR_HIP;
    k_small_csr<<<static_cast<unsigned>((N + kOwn - 1) / kOwn), kThreads, lds, s>>>(src, dst, static_cast<int>(E), N, w,
                                                                                   rowptr, col, perm, w_out);
    PYG_LAUNCH_CHECK();
    return PYG_OK;
}

}  // namespace pyg
