// GAT's attention aggregation fused into one gather pass per direction
// (coefficients alpha = softmax over each target's incoming edges of
// LeakyReLU(a_src[j] + a_dst[i]) per head, then out_i = sum alpha x_j).
//
// What bounds it: on the large power-law graph (114.8M edges, 8 heads of 16)
// everything but the gathers of feature rows was stream traffic over [E, H]
// arrays: the coefficients written once and read four times, their gradients
// and the score gradients written and read, and a second gather pass for the
// dot products. None of these arrays is needed:
//   forward   an online softmax (running maximum, rescaled sums) computes the
//             scores from a_src[j] beside the row gather of x_j; per node and
//             head it keeps (a_dst, maximum, 1 / sum, A+) for the gradient,
//             and the fp32 sums P = sum alpha x_j and
//             P+ = sum over v >= 0 of alpha x_j, A+ = sum over v >= 0 of alpha
//             (v = a_src[j] + a_dst[i], the argument of LeakyReLU);
//   backward  with g = dL/d out and t_i = sum_k alpha_k <g_i, x_k> = <g_i, P_i>
//             the softmax gradient of edge j -> i is
//               dv = alpha (<g_i, x_j> - t_i) (v >= 0 ? 1 : slope),
//             and since the alpha (<g_i, x_k> - t_i) of a target sum to zero,
//               grad a_dst[i] = sum_k dv_k = (1 - slope) (<g_i, P+_i> - t_i A+_i):
//             per-node work only. One pass over the reversed graph gathers g_i
//             and the node's (a_dst, maximum, 1 / sum, t) and forms
//             grad x_j = sum alpha g_i, <g_i, x_j> with x_j held in registers,
//             and grad a_src[j] = sum dv.
// Measured there (fp32, forward and backward): 35.0 ms by the separate kernels,
// 17.0 ms by these (8.0 ms forward, 8.9 ms reversed pass), both bound by the
// rate of cache lines past L2 (five lines gathered per slot and direction; 2,
// 4 or 8 slots in flight per lane take the same time). Windows of 8 or 16
// lanes per slot lose (22.0 and 18.9 ms: the scores and the table are gathered
// again for every window), the non-temporal hint for rows that are no hubs
// gains (18.0 to 17.3 ms). A 108k-edge graph (8 heads of 8): 16 launches and
// 214 us of kernels become 5 and 58 us.
// All sums run in fixed orders: deterministic. Heads never straddle a lane's
// 16-byte vector; other shapes take the separate softmax and sum kernels.
#include "rows.hpp"

#include <cmath>

namespace pyg {
namespace {

__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
// exp(v - m), 0 for a masked score (-inf), whatever m is
__device__ __forceinline__ float pexp(float v, float m) { return v == -INFINITY ? 0.f : fexp(v - m); }
__device__ __forceinline__ float leaky(float v, float slope) { return v >= 0.f ? v : slope * v; }

struct GatParams {
    RowWalk walk;
    int64_t zero_items, zero_rows;
    int64_t nwin;  // windows of whole heads, window-major
    int lg;        // log2 of the lanes per slot and window
    int lgc;       // log2 of the lanes per head
    int64_t F, H;
    float slope;
    const int32_t *col;
    const uint8_t *node_class;  // cache hint: rows of classes below *hot are gathered non-temporally
    const int32_t *hot;         // NULL: no hint
    const float *a_src;
    const void *x;       // forward: x; backward: the rows' own x
    // forward
    const float *a_dst;
    void *out;
    float *all, *plus;   // [N, F] P and P+ (GRAD)
    float4 *stat;        // [N, H] (a_dst, max, 1 / sum, A+) (GRAD)
    float4 *part_st;     // [2 * nchunks, H] (max, sum, sum over v >= 0, -)
    // backward
    const void *g;
    const float4 *tab;   // [N, H] (a_dst, max, 1 / sum, t)
    void *grad_x;
    float *grad_src;
    float *part_gs;      // [2 * nchunks, H]
    // both: [2 * nchunks, F] (and a second such array for P+)
    float *part, *part_plus;
};

// Column of slot e, bit 31 marking a cold source row.
__device__ __forceinline__ int column(const GatParams &p, int64_t e, int hot) {
    int c = __builtin_nontemporal_load(p.col + e);
    if (hot > 0 && p.node_class[c] < hot) c |= static_cast<int>(0x80000000u);
    return c;
}
__device__ __forceinline__ int hot_level(const GatParams &p) {
    return p.hot ? __builtin_amdgcn_readfirstlane(*p.hot) : 0;
}
template <class LN, class T>
__device__ __forceinline__ typename LN::R load_row(const T *x, int j, int64_t F, int64_t f0) {
    const T *src = x + (int64_t)(j & 0x7FFFFFFF) * F + f0;
    return j < 0 ? LN::load_nt(src) : LN::load(src);
}

// ------------------------------------------------------------------ forward
template <typename T, int U, bool GRAD, bool WIDE>
struct GatForward {
    using LN = Lane<T, true>;
    using R = typename LN::R;
    static constexpr int EP = LN::N;
    const GatParams &p;
    int lane, L, S, q, sg;
    int64_t f0, h;
    int hot;
    bool act, owner;  // owner: the lane that stores its head's per-row state
    // state of the row under way
    float m, z, zp, ad;
    float all[EP], plus[EP];

    __device__ GatForward(const GatParams &pp, int ln, int64_t win) : p(pp), lane(ln) {
        L = 1 << p.lg, S = kWave >> p.lg;
        hot = hot_level(p);
        q = lane & (L - 1), sg = lane >> p.lg;
        f0 = ((win << p.lg) + q) * EP;
        act = f0 < p.F;
        h = act ? ((win << p.lg) + q) >> p.lgc : 0;
        owner = act && (q & ((1 << p.lgc) - 1)) == 0;
    }
    __device__ __forceinline__ void begin(int64_t r) {
        m = -INFINITY, z = 0.f, zp = 0.f;
        ad = act ? p.a_dst[r * p.H + h] : 0.f;
#pragma unroll
        for (int e = 0; e < EP; ++e) all[e] = 0.f, plus[e] = 0.f;
    }
    // U slots of this sub-group: sources jj (valid where ok)
    __device__ __forceinline__ void take(const int (&jj)[U], const bool (&ok)[U]) {
        float sc[U];
        R v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) sc[u] = (ok[u] && act) ? p.a_src[(int64_t)(jj[u] & 0x7FFFFFFF) * p.H + h] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            v[u] = (ok[u] && act) ? load_row<LN>(static_cast<const T *>(p.x), jj[u], p.F, f0) : LN::zero();
        bool pos[U];
        float mx = m;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float s = sc[u] + ad;
            pos[u] = s >= 0.f;
            sc[u] = ok[u] ? leaky(s, p.slope) : -INFINITY;
            mx = fmaxf(mx, sc[u]);
        }
        const float k = pexp(m, mx);
        m = mx;
        // the batch is summed by itself first: shorter rounding chains
        float bz = 0.f, bzp = 0.f, ba[EP], bp[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) ba[e] = bp[e] = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {  // no slot: score -inf, weight 0, row 0
            const float w = pexp(sc[u], mx), wp = pos[u] ? w : 0.f;
            bz += w, bzp += wp;
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                const float xv = LN::get(v[u], e);
                ba[e] = fmaf(w, xv, ba[e]);
                if constexpr (GRAD) bp[e] = fmaf(wp, xv, bp[e]);
            }
        }
        z = fmaf(z, k, bz), zp = fmaf(zp, k, bzp);
#pragma unroll
        for (int e = 0; e < EP; ++e) {
            all[e] = fmaf(all[e], k, ba[e]);
            if constexpr (GRAD) plus[e] = fmaf(plus[e], k, bp[e]);
        }
    }
    __device__ __forceinline__ void store(int64_t r) {
        const float inv = 1.f / z;
        float o[EP], o2[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) o[e] = all[e] * inv, o2[e] = plus[e] * inv;
        LN::store(static_cast<T *>(p.out) + r * p.F + f0, o);
        if constexpr (GRAD) {
            store_out<T, true, true>(p.all, r * p.F + f0, o);
            store_out<T, true, true>(p.plus, r * p.F + f0, o2);
            if (owner) p.stat[r * p.H + h] = make_float4(ad, m, inv, zp / z);
        }
    }
    __device__ __forceinline__ void run(int64_t r, int64_t s, int64_t t, int kind, int64_t slot) {
        begin(r);
        // WIDE (64 lanes a slot, one sub-group): 32 slots are summed by themselves
        // before they join the row, whose chain would be a quarter of its slots
        // (rows of 800 slots, 8 heads of 32, grad a_dst from 64 bits: 7.5e-7 by
        // the separate kernels, 1.1e-6 in one chain, 5.8e-7 so, at the same
        // time). Two and more sub-groups are not further off than the separate
        // kernels, and would lose 1 to 3 % by it.
        constexpr int NB = WIDE ? EP : 1;
        float tm = -INFINITY, tz = 0.f, tzp = 0.f, ta[NB], tp[NB];
#pragma unroll
        for (int e = 0; e < NB; ++e) ta[e] = tp[e] = 0.f;
        int nx = (s + lane < t) ? column(p, s + lane, hot) : 0;
        for (int64_t base = s; base < t; base += kWave) {
            const int n = static_cast<int>(uniform64((t - base) < kWave ? (t - base) : kWave));
            const int my = nx;
            if (base + kWave + lane < t) nx = column(p, base + kWave + lane, hot);
            for (int st = 0; st < n; st += S * U) {
                int jj[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int idx = st + u * S + sg;
                    ok[u] = idx < n;
                    jj[u] = __shfl(my, idx & (kWave - 1), kWave);
                }
                take(jj, ok);
                if constexpr (WIDE) {
                    if (((st + S * U) & 31) != 0 && st + S * U < n) continue;
                    const float k = pexp(tm, m);
                    tm = m;
                    tz = fmaf(tz, k, z), z = 0.f;
                    tzp = fmaf(tzp, k, zp), zp = 0.f;
#pragma unroll
                    for (int e = 0; e < EP; ++e) {
                        ta[e] = fmaf(ta[e], k, all[e]), all[e] = 0.f;
                        if constexpr (GRAD) tp[e] = fmaf(tp[e], k, plus[e]), plus[e] = 0.f;
                    }
                }
            }
        }
        if constexpr (WIDE) {
            z = tz, zp = tzp;
#pragma unroll
            for (int e = 0; e < EP; ++e) all[e] = ta[e], plus[e] = tp[e];
        }
        if (L < kWave) {  // the sub-groups' states: common maximum, then sums
            float mt = m;
            for (int off = L; off < kWave; off <<= 1) mt = fmaxf(mt, __shfl_xor(mt, off, kWave));
            const float k = pexp(m, mt);
            m = mt;
            z *= k, zp *= k;
#pragma unroll
            for (int e = 0; e < EP; ++e) all[e] *= k, plus[e] *= k;
            for (int off = L; off < kWave; off <<= 1) {
                z += __shfl_xor(z, off, kWave);
                if constexpr (GRAD) zp += __shfl_xor(zp, off, kWave);
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    all[e] += __shfl_xor(all[e], off, kWave);
                    if constexpr (GRAD) plus[e] += __shfl_xor(plus[e], off, kWave);
                }
            }
        }
        if (sg != 0 || !act) return;
        if (kind == kRowFull) {
            store(r);
            return;
        }
        store_out<T, true, true>(p.part, slot * p.F + f0, all);
        if constexpr (GRAD) store_out<T, true, true>(p.part_plus, slot * p.F + f0, plus);
        if (owner) p.part_st[slot * p.H + h] = make_float4(m, z, zp, 0.f);
    }
    __device__ __forceinline__ void light(int64_t r, int64_t s, int64_t t, bool mine) {
        if (!mine) return;
        begin(r);
        for (int64_t b = s; b < t; b += U) {
            int jj[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = b + u < t;
                jj[u] = ok[u] ? p.col[b + u] : 0;
            }
            take(jj, ok);
        }
        if (act) store(r);
    }
};

template <typename T, int U, bool GRAD, bool LIGHT, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_gat_forward(GatParams p) {
    const int lane = threadIdx.x & (kWave - 1);
    int64_t c = uniform64((int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave);
    if (c < p.zero_items) {
        each_empty_row(p.walk.rowptr, p.walk.N, c, p.zero_rows, lane, [&](int64_t r) {
            for (int64_t f = lane; f < p.F; f += kWave) {
                static_cast<T *>(p.out)[r * p.F + f] = T(0);
                if constexpr (GRAD) p.all[r * p.F + f] = 0.f, p.plus[r * p.F + f] = 0.f;
            }
            if constexpr (GRAD)
                for (int64_t h = lane; h < p.H; h += kWave) p.stat[r * p.H + h] = make_float4(0.f, 0.f, 0.f, 0.f);
        });
        return;
    }
    c -= p.zero_items;
    const int64_t win = c / p.walk.nchunks;
    if (win >= p.nwin) return;
    c -= win * p.walk.nchunks;
    GatForward<T, U, GRAD, WIDE> op(p, lane, win);
    if constexpr (LIGHT) walk_light(p.walk, c, lane, p.lg, op);
    else walk_heavy(p.walk, c, lane, op);
}

// Where wavefront w's quarter of n pieces begins.
__device__ __forceinline__ int first_piece(int n, int w) { return static_cast<int>(static_cast<int64_t>(n) * w / (kBlock / kWave)); }

// Pieces m0 .. m1 - 1 of a long row (head chunk c), one feature per lane: sums
// rescaled to the largest maximum so far, four pieces in flight; LONG: each 16
// pieces are summed by themselves before they join the rest.
struct GatState {
    float m, z, zp, a, b;
    __device__ __forceinline__ void rescale(float mx) {
        const float k = pexp(m, mx);
        z *= k, zp *= k, a *= k, b *= k;
        m = mx;
    }
    __device__ __forceinline__ void add(float k, const GatState &o) {
        z = fmaf(k, o.z, z), zp = fmaf(k, o.zp, zp), a = fmaf(k, o.a, a), b = fmaf(k, o.b, b);
    }
};
template <bool GRAD, bool LONG>
__device__ __forceinline__ GatState fold_pieces(const GatParams &p, int64_t c, int m0, int m1, int64_t f, int64_t h) {
    constexpr int U = 4;
    GatState some{-INFINITY, 0.f, 0.f, 0.f, 0.f}, all = some;  // one maximum for both: some.m
    for (int i0 = m0; i0 < m1; i0 += U) {
        GatState t[U];
        float mx = some.m;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = i0 + u < m1;
            const int64_t sl = piece_of(c, i0 + u);
            const float4 st = on ? p.part_st[sl * p.H + h] : make_float4(-INFINITY, 0.f, 0.f, 0.f);
            t[u] = {st.x, st.y, st.z, on ? p.part[sl * p.F + f] : 0.f, GRAD && on ? p.part_plus[sl * p.F + f] : 0.f};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) mx = fmaxf(mx, t[u].m);
        if constexpr (LONG) all.m = some.m, all.rescale(mx);
        some.rescale(mx);
#pragma unroll
        for (int u = 0; u < U; ++u) some.add(pexp(t[u].m, mx), t[u]);
        if (LONG && ((i0 - m0) & 12) == 12) all.add(1.f, some), some = {mx, 0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (LONG) some.add(1.f, all);
    return some;
}

// Per long row and feature the sums over its pieces. A wavefront looks at
// `per` chunks and folds the long rows that start in them; rows of more than
// kFoldWave pieces are left to the workgroup, whose wavefronts take a quarter
// of the pieces each (a hub of 500,000 of 2M edges, 8 heads of 32: 4.8 ms in one
// wavefront, 0.4 ms so). A workgroup has a
// group of 64 features of its long rows. The short ones are split like that
// (`split`) only while there are too few chunks to fill the chip; else the
// first group's workgroup takes whole rows (20,000 rows of 150 slots in two
// pieces, 8 heads of 32: 34 us, 50 split, as every part finds the rows again).
inline bool fold_split(int64_t nchunks) { return nchunks < 8192; }

template <typename T, bool GRAD>
__global__ __launch_bounds__(kBlock) void k_gat_fold(GatParams p, FoldGrid grid, bool split) {
    constexpr int kW = kBlock / kWave;
    __shared__ GatState part[kW][kWave];
    __shared__ int32_t big_row[kW * kFoldPerMax];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const FoldPlace at(grid);
    const int per = at.per;
    const int64_t c0 = uniform64(at.first + wave * per), f_first = at.group * kWave, step = at.groups * kWave;
    int32_t row = -1, K = 0;
    if (lane < per && c0 + lane < p.walk.nchunks) {
        row = p.walk.head_row[c0 + lane];
        if (row >= 0) K = pieces_of(p.walk.rowptr[row + 1], p.walk.chunk, c0 + lane);
    }
    const bool big = K > kFoldWave;
    if (lane < per) big_row[wave * per + lane] = big ? row : -1;
    uint64_t hit = __ballot(row >= 0 && !big && (split || f_first == 0));
    const int64_t C = p.F / p.H;
    auto store = [&](int64_t r, int64_t f, int64_t h, const GatState &s) {
        const float inv = 1.f / s.z;
        if constexpr (sizeof(T) == 2) static_cast<T *>(p.out)[r * p.F + f] = f32_to_bf16_rne(s.a * inv);
        else static_cast<T *>(p.out)[r * p.F + f] = s.a * inv;
        if constexpr (GRAD) {
            p.all[r * p.F + f] = s.a * inv;
            p.plus[r * p.F + f] = s.b * inv;
            if (f == h * C) p.stat[r * p.H + h] = make_float4(p.a_dst[r * p.H + h], s.m, inv, s.zp / s.z);
        }
    };
    while (hit) {
        const int k = __ffsll(static_cast<unsigned long long>(hit)) - 1;
        hit &= hit - 1;
        const int64_t r = __builtin_amdgcn_readlane(row, k);
        const int n = __builtin_amdgcn_readlane(K, k);
        for (int64_t f = (split ? f_first : 0) + lane; f < p.F; f += split ? step : kWave)
            store(r, f, f / C, fold_pieces<GRAD, false>(p, c0 + k, 0, n, f, f / C));
    }
    __syncthreads();
    // the workgroup's long rows (kW * per is at most a wavefront): uniform over it
    hit = __ballot(lane < kW * per && big_row[lane] >= 0);
    while (hit) {
        const int k = __ffsll(static_cast<unsigned long long>(hit)) - 1;
        hit &= hit - 1;
        const int64_t r = big_row[k], c = at.first + k;
        const int n = pieces_of(p.walk.rowptr[r + 1], p.walk.chunk, c);
        for (int64_t fg = f_first; fg < p.F; fg += step) {
            const int64_t f = fg + lane, h = f < p.F ? f / C : 0;
            if (f < p.F) part[wave][lane] = fold_pieces<GRAD, true>(p, c, first_piece(n, wave), first_piece(n, wave + 1), f, h);
            __syncthreads();
            if (wave == 0 && f < p.F) {
                GatState s = part[0][lane];
                for (int w = 1; w < kW; ++w) {
                    const GatState o = part[w][lane];
                    s.rescale(fmaxf(s.m, o.m));
                    s.add(pexp(o.m, s.m), o);
                }
                store(r, f, h, s);
            }
            __syncthreads();
        }
    }
}

// ----------------------------------------------------------------- backward
// Per node and head: t = <g, P>, grad a_dst = (1 - slope)(<g, P+> - t A+), and
// the table (a_dst, max, 1 / sum, t) that the reversed pass gathers.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gat_node(const T *__restrict__ g, const float *__restrict__ all,
                                                     const float *__restrict__ plus, const float4 *__restrict__ stat,
                                                     int64_t nvec, int lgc, float slope,
                                                     float4 *__restrict__ tab, float *__restrict__ grad_dst) {
    using LN = Lane<T, true>;
    constexpr int EP = LN::N;
    // whole groups of 2^lgc lanes share a head; nvec is a multiple of it
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < nvec; k += (int64_t)gridDim.x * kBlock) {
        const auto gv = LN::load(g + k * EP);
        float d[2] = {0.f, 0.f};
#pragma unroll
        for (int e = 0; e < EP; e += 4) {
            const float4 a = *reinterpret_cast<const float4 *>(all + k * EP + e);
            const float4 b = *reinterpret_cast<const float4 *>(plus + k * EP + e);
            const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                d[0] = fmaf(LN::get(gv, e + i), av[i], d[0]);
                d[1] = fmaf(LN::get(gv, e + i), bv[i], d[1]);
            }
        }
        group_sum(d, lgc);
        if ((k & ((int64_t(1) << lgc) - 1)) == 0) {
            const int64_t nh = k >> lgc;  // node * H + head
            const float4 st = stat[nh];
            tab[nh] = make_float4(st.x, st.y, st.z, d[0]);
            // no incoming edges (1 / sum is 0 there alone): an empty sum, whatever g holds
            grad_dst[nh] = st.z == 0.f ? 0.f : (1.f - slope) * (d[1] - d[0] * st.w);
        }
    }
}

template <typename T, int U>
struct GatBackward {
    using LN = Lane<T, true>;
    using R = typename LN::R;
    static constexpr int EP = LN::N;
    const GatParams &p;
    int lane, L, S, q, sg;
    int64_t f0, h;
    int hot;
    bool act, owner;
    float as, gs;
    float xo[EP], acc[EP];

    __device__ GatBackward(const GatParams &pp, int ln, int64_t win) : p(pp), lane(ln) {
        L = 1 << p.lg, S = kWave >> p.lg;
        hot = hot_level(p);
        q = lane & (L - 1), sg = lane >> p.lg;
        f0 = ((win << p.lg) + q) * EP;
        act = f0 < p.F;
        h = act ? ((win << p.lg) + q) >> p.lgc : 0;
        owner = act && (q & ((1 << p.lgc) - 1)) == 0;
    }
    __device__ __forceinline__ void begin(int64_t r) {
        gs = 0.f;
        as = act ? p.a_src[r * p.H + h] : 0.f;
        const R xr = act ? LN::load(static_cast<const T *>(p.x) + r * p.F + f0) : LN::zero();
#pragma unroll
        for (int e = 0; e < EP; ++e) xo[e] = LN::get(xr, e), acc[e] = 0.f;
    }
    __device__ __forceinline__ float4 load_tab(int j) const {
        const float *t = reinterpret_cast<const float *>(p.tab + (int64_t)(j & 0x7FFFFFFF) * p.H + h);
        return j < 0 ? Lane<float, true>::load_nt(t) : Lane<float, true>::load(t);
    }
    __device__ __forceinline__ void take(const int (&jj)[U], const bool (&ok)[U]) {
        float4 tb[U];
        R v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            tb[u] = (ok[u] && act) ? load_tab(jj[u]) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < U; ++u)
            v[u] = (ok[u] && act) ? load_row<LN>(static_cast<const T *>(p.g), jj[u], p.F, f0) : LN::zero();
        float d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            d[u] = 0.f;
#pragma unroll
            for (int e = 0; e < EP; ++e) d[u] = fmaf(LN::get(v[u], e), xo[e], d[u]);
        }
        group_sum(d, p.lgc);
        float bg = 0.f, ba[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) ba[e] = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float s = as + tb[u].x;
            const float al = ok[u] ? pexp(leaky(s, p.slope), tb[u].y) * tb[u].z : 0.f;
            const float ds = al * (d[u] - tb[u].w);
            bg += s >= 0.f ? ds : p.slope * ds;
#pragma unroll
            for (int e = 0; e < EP; ++e) ba[e] = fmaf(al, LN::get(v[u], e), ba[e]);
        }
        gs += bg;
#pragma unroll
        for (int e = 0; e < EP; ++e) acc[e] += ba[e];
    }
    __device__ __forceinline__ void run(int64_t r, int64_t s, int64_t t, int kind, int64_t slot) {
        begin(r);
        float total = 0.f;
        int nx = (s + lane < t) ? column(p, s + lane, hot) : 0;
        for (int64_t base = s; base < t; base += kWave) {
            const int n = static_cast<int>(uniform64((t - base) < kWave ? (t - base) : kWave));
            const int my = nx;
            if (base + kWave + lane < t) nx = column(p, base + kWave + lane, hot);
            for (int st = 0; st < n; st += S * U) {
                int jj[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int idx = st + u * S + sg;
                    ok[u] = idx < n;
                    jj[u] = __shfl(my, idx & (kWave - 1), kWave);
                }
                take(jj, ok);
            }
            total += gs, gs = 0.f;  // per batch: shorter rounding chains
        }
        gs = total;
        for (int off = L; off < kWave; off <<= 1) {
            gs += __shfl_xor(gs, off, kWave);
#pragma unroll
            for (int e = 0; e < EP; ++e) acc[e] += __shfl_xor(acc[e], off, kWave);
        }
        if (sg != 0 || !act) return;
        if (kind == kRowFull) {
            LN::store(static_cast<T *>(p.grad_x) + r * p.F + f0, acc);
            if (owner) p.grad_src[r * p.H + h] = gs;
        } else {
            store_out<T, true, true>(p.part, slot * p.F + f0, acc);
            if (owner) p.part_gs[slot * p.H + h] = gs;
        }
    }
    __device__ __forceinline__ void light(int64_t r, int64_t s, int64_t t, bool mine) {
        if (!mine) return;
        begin(r);
        for (int64_t b = s; b < t; b += U) {
            int jj[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = b + u < t;
                jj[u] = ok[u] ? p.col[b + u] : 0;
            }
            take(jj, ok);
        }
        if (!act) return;
        LN::store(static_cast<T *>(p.grad_x) + r * p.F + f0, acc);
        if (owner) p.grad_src[r * p.H + h] = gs;
    }
};

template <typename T, int U, bool LIGHT>
__global__ __launch_bounds__(kBlock) void k_gat_backward(GatParams p) {
    const int lane = threadIdx.x & (kWave - 1);
    int64_t c = uniform64((int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave);
    if (c < p.zero_items) {
        each_empty_row(p.walk.rowptr, p.walk.N, c, p.zero_rows, lane, [&](int64_t r) {
            for (int64_t f = lane; f < p.F; f += kWave) static_cast<T *>(p.grad_x)[r * p.F + f] = T(0);
            for (int64_t h = lane; h < p.H; h += kWave) p.grad_src[r * p.H + h] = 0.f;
        });
        return;
    }
    c -= p.zero_items;
    const int64_t win = c / p.walk.nchunks;
    if (win >= p.nwin) return;
    c -= win * p.walk.nchunks;
    GatBackward<T, U> op(p, lane, win);
    if constexpr (LIGHT) walk_light(p.walk, c, lane, p.lg, op);
    else walk_heavy(p.walk, c, lane, op);
}

// The pieces of every long row: the F features, then the H sums of dv, split
// as in k_gat_fold. (One wavefront and one chain for a row of whatever length:
// the output of a hub of 150,000 edges was 9e-7 from 64 bits, below 3e-7 split.)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gat_backward_fold(GatParams p, FoldGrid grid, bool split) {
    constexpr int kW = kBlock / kWave;
    __shared__ float part[kW][kWave];
    __shared__ int32_t big_row[kW * kFoldPerMax];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const FoldPlace at(grid);
    const int per = at.per;
    const int64_t c0 = uniform64(at.first + wave * per), f_first = at.group * kWave, step = at.groups * kWave;
    int32_t row = -1, K = 0;
    if (lane < per && c0 + lane < p.walk.nchunks) {
        row = p.walk.head_row[c0 + lane];
        if (row >= 0) K = pieces_of(p.walk.rowptr[row + 1], p.walk.chunk, c0 + lane);
    }
    const bool big = K > kFoldWave;
    if (lane < per) big_row[wave * per + lane] = big ? row : -1;
    uint64_t hit = __ballot(row >= 0 && !big && (split || f_first == 0));
    const int64_t cols = p.F + p.H;
    // pieces m0 .. m1 - 1, each 16 summed by themselves
    auto fold = [&](int64_t c, int m0, int m1, int64_t f) {
        constexpr int U = 8;
        const float *src = f < p.F ? p.part + f : p.part_gs + (f - p.F);
        const int64_t stride = f < p.F ? p.F : p.H;
        float all = 0.f, some = 0.f;
        for (int i0 = m0; i0 < m1; i0 += U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = i0 + u < m1 ? src[piece_of(c, i0 + u) * stride] : 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) some += v[u];
            if ((i0 - m0) & U) all += some, some = 0.f;
        }
        return all + some;
    };
    auto store = [&](int64_t r, int64_t f, float v) {
        if (f >= p.F) p.grad_src[r * p.H + f - p.F] = v;
        else if constexpr (sizeof(T) == 2) static_cast<T *>(p.grad_x)[r * p.F + f] = f32_to_bf16_rne(v);
        else static_cast<T *>(p.grad_x)[r * p.F + f] = v;
    };
    while (hit) {
        const int k = __ffsll(static_cast<unsigned long long>(hit)) - 1;
        hit &= hit - 1;
        const int64_t r = __builtin_amdgcn_readlane(row, k);
        const int n = __builtin_amdgcn_readlane(K, k);
        for (int64_t f = (split ? f_first : 0) + lane; f < cols; f += split ? step : kWave)
            store(r, f, fold(c0 + k, 0, n, f));
    }
    __syncthreads();
    // the workgroup's long rows (kW * per is at most a wavefront): uniform over it
    hit = __ballot(lane < kW * per && big_row[lane] >= 0);
    while (hit) {
        const int k = __ffsll(static_cast<unsigned long long>(hit)) - 1;
        hit &= hit - 1;
        const int64_t r = big_row[k], c = at.first + k;
        const int n = pieces_of(p.walk.rowptr[r + 1], p.walk.chunk, c);
        for (int64_t fg = f_first; fg < cols; fg += step) {
            const int64_t f = fg + lane;
            if (f < cols) part[wave][lane] = fold(c, first_piece(n, wave), first_piece(n, wave + 1), f);
            __syncthreads();
            if (wave == 0 && f < cols) {
                float v = part[0][lane];
                for (int w = 1; w < kW; ++w) v += part[w][lane];
                store(r, f, v);
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------- launching
struct GatWs {
    float *part, *part_plus, *part_gs;
    float4 *part_st, *tab;
    int32_t *head_row;
    uint8_t *node_class;
    int32_t *hist, *hot;
    size_t bytes;
};

GatWs carve_gat(void *base, int64_t N, int64_t H, int64_t F, int64_t E, int64_t chunk, bool backward) {
    const int64_t nchunks = E > 0 ? (E + chunk - 1) / chunk : 0;
    Carver c(base);
    GatWs w{};
    w.part = c.take<float>(2 * nchunks * F);
    w.head_row = c.take<int32_t>(nchunks);
    w.node_class = c.take<uint8_t>(N);
    w.hist = c.take<int32_t>(kHotClasses);
    w.hot = c.take<int32_t>(1);
    if (backward) {
        w.part_gs = c.take<float>(2 * nchunks * H);
        w.tab = c.take<float4>(N * H);
    } else {
        w.part_plus = c.take<float>(2 * nchunks * F);
        w.part_st = c.take<float4>(2 * nchunks * H);
    }
    w.bytes = c.used + 256;
    return w;
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// Shapes of the fused kernels: heads of a power-of-two count of whole 16-byte
// lane vectors, at most one wavefront (64 of them) per head.
bool gat_shape_ok(int64_t sz, int64_t C) {
    const int64_t EP = 16 / sz;
    if (C <= 0 || C % EP != 0) return false;
    const int64_t lh = C / EP;
    return lh <= kWave && (lh & (lh - 1)) == 0;
}

// Lanes per window: whole heads, at most max_lanes.
void set_windows(GatParams &p, int64_t sz, int64_t C, int max_lanes) {
    const int64_t EP = 16 / sz, nvec = p.F / EP, lh = C / EP;
    p.lgc = 0;
    while ((int64_t(1) << p.lgc) < lh) ++p.lgc;
    p.lg = p.lgc;
    while ((int64_t(1) << p.lg) < nvec && (2 << p.lg) <= max_lanes) ++p.lg;
    p.nwin = (nvec + (int64_t(1) << p.lg) - 1) >> p.lg;
}

void set_walk(GatParams &p, const pyg_csr *csr, int64_t chunk, int32_t *head_row) {
    p.walk = {csr->rowptr, csr->N, csr->E, chunk, light_row_slots(csr->E, csr->N, chunk), (csr->E + chunk - 1) / chunk, head_row};
    int64_t per = (csr->N + 1023) / 1024;
    per = (per + kWave - 1) / kWave * kWave;
    p.zero_rows = per > kWave ? per : kWave;
    p.zero_items = (csr->N + p.zero_rows - 1) / p.zero_rows;
    p.col = csr->col;
}

// The hub-row hint, where the gathered rows are large (whole rows only).
int set_hint(GatParams &p, const GatWs &w, int64_t sz, hipStream_t s) {
    const int64_t row_bytes = p.F * sz;
    if (p.nwin > 1 || !hint_pays(p.walk.N, row_bytes)) return PYG_OK;
    PYG_TRY(hot_rows(p.walk.rowptr, p.walk.N, row_bytes, w.hist, w.node_class, w.hot, s));
    p.node_class = w.node_class;
    p.hot = w.hot;
    return PYG_OK;
}

template <typename T, bool GRAD>
int launch_forward(const GatParams &p, hipStream_t s) {
    constexpr int U = 4;
    const int64_t items = p.zero_items + p.walk.nchunks * p.nwin;
    const unsigned grid = static_cast<unsigned>((items + 3) / 4);
    const bool light = p.lg < 6 && p.walk.E <= kLightMaxDegree * p.walk.N;
    if (light) k_gat_forward<T, U, GRAD, true, false><<<grid, kBlock, 0, s>>>(p);
    else if (p.lg < 6) k_gat_forward<T, U, GRAD, false, false><<<grid, kBlock, 0, s>>>(p);
    else k_gat_forward<T, U, GRAD, false, true><<<grid, kBlock, 0, s>>>(p);
    PYG_LAUNCH_CHECK();
    if (p.walk.nchunks > 1) {
        const FoldGrid g(p.walk.nchunks, p.F, !fold_split(p.walk.nchunks));
        k_gat_fold<T, GRAD><<<g.grid, kBlock, 0, s>>>(p, g, fold_split(p.walk.nchunks));
        PYG_LAUNCH_CHECK();
    }
    return PYG_OK;
}

template <typename T>
int launch_backward(const GatParams &p, const float *all, const float *plus, const float4 *stat, float4 *tab,
                    float *grad_dst, hipStream_t s) {
    constexpr int U = 4, EP = 16 / sizeof(T);
    const int64_t nvec = p.walk.N * p.F / EP;
    k_gat_node<T><<<grid_for(nvec, kBlock * 2), kBlock, 0, s>>>(static_cast<const T *>(p.g), all, plus, stat, nvec,
                                                                p.lgc, p.slope, tab, grad_dst);
    PYG_LAUNCH_CHECK();
    const int64_t items = p.zero_items + p.walk.nchunks * p.nwin;
    const unsigned grid = static_cast<unsigned>((items + 3) / 4);
    const bool light = p.lg < 6 && p.walk.E <= kLightMaxDegree * p.walk.N;
    if (light) k_gat_backward<T, U, true><<<grid, kBlock, 0, s>>>(p);
    else k_gat_backward<T, U, false><<<grid, kBlock, 0, s>>>(p);
    PYG_LAUNCH_CHECK();
    if (p.walk.nchunks > 1) {
        const FoldGrid g(p.walk.nchunks, p.F + p.H, !fold_split(p.walk.nchunks));
        k_gat_backward_fold<T><<<g.grid, kBlock, 0, s>>>(p, g, fold_split(p.walk.nchunks));
        PYG_LAUNCH_CHECK();
    }
    return PYG_OK;
}

int gat_check(int dtype, int64_t H, int64_t C, float slope, const pyg_csr *c) {
    if ((dtype != PYG_F32 && dtype != PYG_BF16) || H <= 0 || C < 0 || !std::isfinite(slope)) return PYG_ERR_INVALID_ARG;
    if (!c || c->N < 0 || c->E < 0 || c->chunk < 0 || !c->rowptr || (c->E > 0 && !c->col)) return PYG_ERR_INVALID_ARG;
    const int64_t lim = int64_t(1) << 31;
    if (c->N >= lim || c->E >= lim || H * C >= lim) return PYG_ERR_UNSUPPORTED;
    if (c->E == 0 || !gat_shape_ok(dtype == PYG_BF16 ? 2 : 4, C)) return PYG_ERR_UNSUPPORTED;
    return PYG_OK;
}

}  // namespace
}  // namespace pyg

using namespace pyg;

extern "C" int pyg_gat_forward_workspace(int64_t N, int64_t H, int64_t C, int64_t E, int64_t chunk, size_t *bytes) {
    if (!bytes || N < 0 || H < 0 || C < 0 || E < 0 || chunk < 0) return PYG_ERR_INVALID_ARG;
    const int64_t lim = int64_t(1) << 31;
    if (N >= lim || E >= lim || H * C >= lim) return PYG_ERR_UNSUPPORTED;
    *bytes = carve_gat(nullptr, N, H, H * C, E, segment_chunk(E, N, chunk), false).bytes;
    return PYG_OK;
}

extern "C" int pyg_gat_forward(const void *x, int dtype, int64_t H, int64_t C, const float *a_src, const float *a_dst,
                               float negative_slope, const pyg_csr *csr, void *out, float *all, float *plus, float *stat,
                               void *ws, size_t ws_bytes, void *stream) {
    PYG_TRY(gat_check(dtype, H, C, negative_slope, csr));
    const int64_t N = csr->N, E = csr->E, F = H * C;
    if (!x || !a_src || !a_dst || !out || x == out) return PYG_ERR_INVALID_ARG;
    const bool grad = all || plus || stat;
    if (grad && (!all || !plus || !stat)) return PYG_ERR_INVALID_ARG;
    if (!aligned16(x) || !aligned16(out) || !aligned16(all) || !aligned16(plus) || !aligned16(stat))
        return PYG_ERR_UNSUPPORTED;
    const int64_t chunk = segment_chunk(E, N, csr->chunk);
    const GatWs w = carve_gat(ws, N, H, F, E, chunk, false);
    if (!ws || ws_bytes < w.bytes) return PYG_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    GatParams p{};
    p.F = F, p.H = H, p.slope = negative_slope;
    p.a_src = a_src, p.a_dst = a_dst, p.x = x, p.out = out;
    p.all = all, p.plus = plus, p.stat = reinterpret_cast<float4 *>(stat);
    p.part = w.part, p.part_plus = w.part_plus, p.part_st = w.part_st;
    set_walk(p, csr, chunk, w.head_row);
    const int64_t sz = dtype == PYG_BF16 ? 2 : 4;
    set_windows(p, sz, C, kWave);
    PYG_TRY(set_hint(p, w, sz, s));
    if (dtype == PYG_BF16)
        return grad ? launch_forward<uint16_t, true>(p, s) : launch_forward<uint16_t, false>(p, s);
    return grad ? launch_forward<float, true>(p, s) : launch_forward<float, false>(p, s);
}

extern "C" int pyg_gat_backward_workspace(int64_t N, int64_t H, int64_t C, int64_t E, int64_t chunk_t, size_t *bytes) {
    if (!bytes || N < 0 || H < 0 || C < 0 || E < 0 || chunk_t < 0) return PYG_ERR_INVALID_ARG;
    const int64_t lim = int64_t(1) << 31;
    if (N >= lim || E >= lim || H * C >= lim) return PYG_ERR_UNSUPPORTED;
    *bytes = carve_gat(nullptr, N, H, H * C, E, segment_chunk(E, N, chunk_t), true).bytes;
    return PYG_OK;
}

extern "C" int pyg_gat_backward(const void *grad_out, const void *x, int dtype, int64_t H, int64_t C, const float *a_src,
                                float negative_slope, const float *all, const float *plus, const float *stat,
                                const pyg_csr *csr_t, void *grad_x, float *grad_a_src, float *grad_a_dst, void *ws,
                                size_t ws_bytes, void *stream) {
    PYG_TRY(gat_check(dtype, H, C, negative_slope, csr_t));
    const int64_t N = csr_t->N, E = csr_t->E, F = H * C;
    if (!grad_out || !x || !a_src || !all || !plus || !stat || !grad_x || !grad_a_src || !grad_a_dst ||
        grad_x == grad_out || grad_x == x)
        return PYG_ERR_INVALID_ARG;
    if (!aligned16(grad_out) || !aligned16(x) || !aligned16(grad_x) || !aligned16(all) || !aligned16(plus) ||
        !aligned16(stat))
        return PYG_ERR_UNSUPPORTED;
    const int64_t chunk = segment_chunk(E, N, csr_t->chunk);
    const GatWs w = carve_gat(ws, N, H, F, E, chunk, true);
    if (!ws || ws_bytes < w.bytes) return PYG_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    GatParams p{};
    p.F = F, p.H = H, p.slope = negative_slope;
    p.a_src = a_src, p.x = x, p.g = grad_out, p.tab = w.tab;
    p.grad_x = grad_x, p.grad_src = grad_a_src;
    p.part = w.part, p.part_gs = w.part_gs;
    set_walk(p, csr_t, chunk, w.head_row);
    const int64_t sz = dtype == PYG_BF16 ? 2 : 4;
    set_windows(p, sz, C, kWave);
    PYG_TRY(set_hint(p, w, sz, s));
    const float4 *st = reinterpret_cast<const float4 *>(stat);
    if (dtype == PYG_BF16) return launch_backward<uint16_t>(p, all, plus, st, w.tab, grad_a_dst, s);
    return launch_backward<float>(p, all, plus, st, w.tab, grad_a_dst, s);
}
