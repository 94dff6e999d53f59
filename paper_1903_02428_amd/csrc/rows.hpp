// The walk of one wavefront over its chunk of CSR slots, shared by the fused
// attention kernels and the fused gradient kernel: the same work split as the
// segment kernel (equal chunks of slots per wavefront, a row of at most
// `chunk` slots reduced whole by the chunk that holds its first slot, a longer
// row cut at chunk boundaries into pieces that are folded afterwards).
#pragma once

#include "lanes.hpp"

namespace pyg {

// Sum over the 2^lg lanes that share a head (aligned groups), every lane
// ending with the sum. The first four steps are cross-lane moves inside a
// 16-lane row (quad permutes, then mirrors: after the quads agree, the mirror
// image of a lane lies in the other half), one VALU instruction each instead
// of an LDS permute; the order is fixed.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true);
    return v + __int_as_float(o);
}
template <int U>
__device__ __forceinline__ void group_sum(float (&d)[U], int lg) {
    if (lg >= 1)
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = dpp_add<0xB1>(d[u]);  // quad_perm [1,0,3,2]
    if (lg >= 2)
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = dpp_add<0x4E>(d[u]);  // quad_perm [2,3,0,1]
    if (lg >= 3)
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = dpp_add<0x141>(d[u]);  // row_half_mirror
    if (lg >= 4)
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = dpp_add<0x140>(d[u]);  // row_mirror
    for (int off = 16; off < (1 << lg); off <<= 1)
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] += __shfl_xor(d[u], off, kWave);
}

struct RowWalk {
    const int64_t *rowptr;
    int64_t N;  // rows
    int64_t E;
    int64_t chunk;
    int64_t light_row;  // light rows: slots up to which a sub-group takes a row
    int64_t nchunks;
    int32_t *head_row;  // [nchunks]: the long row that starts in the chunk, or -1
};

constexpr int kRowFull = 0, kRowPiece = 1;

// Heavy rows: op.run(r, s, t, kind, slot) with wave-uniform arguments, once
// per non-empty row (kRowFull) or piece (kRowPiece, slot of its partial).
// Empty rows are not visited.
template <class OP>
__device__ __forceinline__ void walk_heavy(const RowWalk &p, int64_t c, int lane, OP &op) {
    const int64_t e0 = c * p.chunk;
    const int64_t e1 = (e0 + p.chunk) < p.E ? (e0 + p.chunk) : p.E;
    const int64_t rA = uniform64(wave_lower_bound(p.rowptr, p.N + 1, e0, lane));
    const int64_t rpA = uniform64(p.rowptr[rA]);
    // a long row that started in an earlier chunk has a piece here
    bool cont = false;
    if (rA > 0 && rpA > e0) cont = rpA - uniform64(p.rowptr[rA - 1]) > p.chunk;
    int32_t head = -1;
    int64_t r = rA, rb = rA - kWave, rp = 0;
    while (true) {
        int64_t rr = r, s = e0, t = rpA < e1 ? rpA : e1, slot = 2 * c;
        int kind = kRowPiece;
        if (cont) {
            rr = rA - 1;
        } else {
            if (r >= p.N) break;
            if (r + 1 - rb >= kWave) {  // the next 64 row bounds, past a run of empty rows
                rb = r;
                rp = p.rowptr[(rb + lane) < p.N ? (rb + lane) : p.N];
                const int64_t s0 = lane_value64(rp, 0);
                if (s0 >= e1) break;
                if (rb + kWave - 1 <= p.N && lane_value64(rp, kWave - 1) == s0) {
                    r = uniform_lower_bound(p.rowptr, p.N + 1, s0 + 1) - 1;
                    rr = r;
                    rb = r;
                    rp = p.rowptr[(rb + lane) < p.N ? (rb + lane) : p.N];
                }
            }
            s = lane_value64(rp, static_cast<int>(r - rb));
            t = lane_value64(rp, static_cast<int>(r + 1 - rb));
            if (s >= e1) break;
            if (t == s) {
                ++r;
                continue;
            }
            kind = kRowFull;
            if (t - s > p.chunk) {
                kind = kRowPiece;
                slot = 2 * c + 1;
                t = e1;
                head = static_cast<int32_t>(r);
            }
        }
        op.run(rr, s, t, kind, slot);
        if (head >= 0) break;
        if (cont) cont = false;
        else ++r;
    }
    p.head_row[c] = head;  // uniform: every lane stores the same value
}

// Light rows: each of the 64 >> lg sub-groups takes a row of its own of up to
// light_row slots, op.light(r, s, t, mine); longer rows and pieces of long
// ones go to the whole wavefront (op.run).
template <class OP>
__device__ __forceinline__ void walk_light(const RowWalk &p, int64_t c, int lane, int lg, OP &op) {
    const int64_t e0 = c * p.chunk;
    const int64_t e1 = (e0 + p.chunk) < p.E ? (e0 + p.chunk) : p.E;
    const int64_t rA = uniform64(wave_lower_bound(p.rowptr, p.N + 1, e0, lane));
    const int64_t rpA = uniform64(p.rowptr[rA]);
    bool cont = rA > 0 && rpA > e0 && rpA - uniform64(p.rowptr[rA - 1]) > p.chunk;
    const int S = kWave >> lg, sg = lane >> lg;
    int32_t head = -1;
    int64_t rb = rA;
    while (true) {
        const int64_t rp = p.rowptr[(rb + lane) < p.N ? (rb + lane) : p.N];
        // rows rb .. rb + cnt - 1 start in the chunk; lane i + 1 holds the end of row rb + i
        const bool in = lane < kWave - 1 && rb + lane < p.N && rp < e1;
        const int cnt = __popcll(__ballot(in));
        const int64_t s_first = lane_value64(rp, 0);
        if (cnt == kWave - 1 && lane_value64(rp, kWave - 1) == s_first) {
            rb = uniform_lower_bound(p.rowptr, p.N + 1, s_first + 1) - 1;  // a run of empty rows
            continue;
        }
        for (int i0 = 0; i0 < cnt; i0 += S) {
            const int i = i0 + sg;
            const int ii = i < cnt ? i : cnt - 1;
            const int64_t s = __shfl(rp, ii, kWave), t = __shfl(rp, ii + 1, kWave);
            op.light(rb + i, s, t, i < cnt && t > s && t - s <= p.light_row);
        }
        // the whole wavefront's: rows above light_row slots, the first piece of
        // a long row (only the chunk's last row can be one), the piece that came in
        const int64_t len = __shfl_down(rp, 1, kWave) - rp;
        uint64_t jobs = __ballot(lane < cnt && len > p.light_row);
        while (cont || jobs) {
            int64_t r = rA - 1, s = e0, t = rpA < e1 ? rpA : e1, slot = 2 * c;
            int kind = kRowPiece;
            if (!cont) {
                const int k = __ffsll(static_cast<unsigned long long>(jobs)) - 1;
                jobs &= jobs - 1;
                r = rb + k;
                s = lane_value64(rp, k);
                t = lane_value64(rp, k + 1);
                kind = kRowFull;
                if (t - s > p.chunk) {
                    kind = kRowPiece;
                    slot = 2 * c + 1;
                    t = e1;
                    head = static_cast<int32_t>(r);
                }
            }
            cont = false;
            op.run(r, s, t, kind, slot);
        }
        if (cnt < kWave - 1) break;  // the chunk's rows end in this batch
        rb += cnt;
    }
    p.head_row[c] = head;
}

// Empty rows r of the z-th group of `per` rows (a multiple of 64): f(row).
template <class FN>
__device__ __forceinline__ void each_empty_row(const int64_t *rowptr, int64_t N, int64_t z, int64_t per, int lane, FN f) {
    const int64_t end = (z + 1) * per < N ? (z + 1) * per : N;
    for (int64_t r0 = z * per; r0 < end; r0 += kWave) {
        const int64_t r = r0 + lane;
        const bool in = r < end;
        const int64_t a = in ? rowptr[r] : 0, b = in ? rowptr[r + 1] : 1;
        uint64_t m = __ballot(in && a == b);
        while (m) {
            const int k = __ffsll(static_cast<unsigned long long>(m)) - 1;
            m &= m - 1;
            f(r0 + k);
        }
    }
}

// The slot of piece m of the long row whose head chunk is c.
__device__ __forceinline__ int64_t piece_of(int64_t c, int64_t m) { return m == 0 ? 2 * c + 1 : 2 * (c + m); }

}  // namespace pyg
