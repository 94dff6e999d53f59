// Both gradients of a propagate whose edges carry values (scalar weights, or
// F-dimensional edge features), in one pass over the reversed graph.
//
// grad x_j sums over the edges j -> i what the upstream row g_i passes back,
// and the edge's own gradient is made of the same row g_i and of x_j:
//   w x_j           grad x_j += w g_i          grad w = <g_i, x_j>
//   x_j + e         grad x_j += g_i            grad e = g_i
//   max(x_j + e, 0) both times [x_j + e > 0]
//   x_j e           grad x_j += e g_i          grad e = g_i x_j
// (g scaled by 1 / deg_i under mean; scalar weights divide here). Over the rows
// of the reversed CSR x_j stays in registers, so one gather of g_i serves both;
// a second pass over the CSR gathered x_j again and, for edge features, read
// every e again. The per-edge arrays are reached through perm (the edge ids),
// loaded with the columns one batch of 64 slots ahead. Deterministic: one writer
// per edge, and the segment kernel's order for the sums, hence its bits, but
// for rows that it sums in windows of 128 bytes.
//
// Measured on a power-law graph of 100,000 nodes and 2M edges: both gradients
// of the weighted sum (fp32, F = 100) 657 us in two passes, 180 us in one; of
// max(x_j + e, 0) (bf16, F = 64) 709 and 175 us. What is left is latency (rows
// of 20 slots) rather than bytes (100 and 550 MB): fewer slots in flight per
// lane and more wavefronts are faster (weights 8, 4, 2 slots: 199, 175, 195 us;
// edge features 8, 4, 2: 294, 200, 167 us).
#include "rows.hpp"

namespace pyg {
namespace {

constexpr int kWeight = 0, kAdd = 1, kRelu = 2, kMul = 3;
// kWeight under mean: g is the upstream row itself. grad x_j takes g_i / deg_i
// as the scaling pass rounds it; grad w is the dot product of the unscaled rows
// over deg_i, so that its terms carry no rounding of their own (the dot product of
// rows scaled beforehand was 1.2 times as far from 64 bits).
constexpr int kWeightMean = 4;

// n / d from inv = 1 / d, correctly rounded where the quotient is a normal
// number (a subnormal one may miss a tie): one correction of n * inv by its exact
// remainder (Markstein's step); the fix-up settles infinities and NaN.
__device__ __forceinline__ float div_by(float n, float d, float inv) {
    const float q = n * inv;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-d, q, n), inv, q), d, n);
}

struct FusedParams {
    RowWalk walk;
    int64_t zero_items, zero_rows;
    int lg;  // log2 of the lanes per slot
    int64_t F;
    const int32_t *col;
    const int64_t *perm;  // edge id of every slot
    const float *w;       // kWeight, kWeightMean: slot order
    const int64_t *deg_ptr;  // kWeightMean: the targets' row bounds [N + 1]
    const uint8_t *node_class;
    const int32_t *hot;
    const void *g;        // [N, F] of TG
    const void *x;        // [N, F] of T (not read by kAdd)
    const void *ea;       // [E, F] of T, edge ids (kRelu, kMul)
    void *grad_x;         // [N, F] of T
    float *grad_w;        // [E], edge ids
    void *grad_e;         // [E, F] of T, edge ids
    float *part;          // [2 * nchunks, F]
};

template <typename TG, typename T, int KIND, int U, bool BATCHED>
struct FusedBackward {
    using LN = Lane<TG, true>;
    using R = typename LN::R;
    static constexpr int EP = LN::N;
    static constexpr bool MEAN = KIND == kWeightMean, WEIGHT = KIND == kWeight || MEAN, EDGE = !WEIGHT;
    template <typename TE> using Share = typename std::conditional<sizeof(TE) == 4 || EP == 8, uint4, uint2>::type;
    template <typename TE>
    __device__ static __forceinline__ float share_get(const Share<TE> &r, int e) {
        const uint32_t *w = reinterpret_cast<const uint32_t *>(&r);
        if constexpr (sizeof(TE) == 4) return __uint_as_float(w[e]);
        else return __uint_as_float((e & 1) ? w[e >> 1] & 0xFFFF0000u : w[e >> 1] << 16);
    }
    const FusedParams &p;
    int lane, L, S, q, sg, hot;
    int64_t f0;
    bool act;
    float xo[EP], acc[EP];

    __device__ FusedBackward(const FusedParams &pp, int ln) : p(pp), lane(ln) {
        L = 1 << p.lg, S = kWave >> p.lg;
        q = lane & (L - 1), sg = lane >> p.lg;
        f0 = (int64_t)q * EP;
        act = f0 < p.F;
        hot = p.hot ? __builtin_amdgcn_readfirstlane(*p.hot) : 0;
    }
    __device__ __forceinline__ void begin(int64_t r) {
#pragma unroll
        for (int e = 0; e < EP; ++e) xo[e] = 0.f, acc[e] = 0.f;
        if (KIND != kAdd && act) ldv<T, EP>(static_cast<const T *>(p.x) + r * p.F + f0, xo);
    }
    __device__ __forceinline__ void take(const int (&jj)[U], const bool (&ok)[U], const float (&ww)[U],
                                         const int (&ee)[U], const float (&dd)[U]) {
        R v[U];
        Share<T> ev[EDGE ? U : 1];  // raw: a lane's share of the edge row
        if constexpr (KIND == kRelu || KIND == kMul) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const T *e = static_cast<const T *>(p.ea) + (int64_t)ee[u] * p.F + f0;
                if (ok[u] && act) ev[u] = *reinterpret_cast<const Share<T> *>(e);
                else ev[u] = Share<T>{};
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const TG *src = static_cast<const TG *>(p.g) + (int64_t)(jj[u] & 0x7FFFFFFF) * p.F + f0;
            if (!(ok[u] && act)) v[u] = LN::zero();
            else if (jj[u] < 0) v[u] = LN::load_nt(src);
            else v[u] = LN::load(src);
        }
        if constexpr (WEIGHT) {
            float d[U], inv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d[u] = 0.f;
                inv[u] = MEAN ? 1.f / dd[u] : 1.f;
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    const float gv = LN::get(v[u], e);
                    d[u] = fmaf(gv, xo[e], d[u]);
                    acc[e] = fmaf(ok[u] ? ww[u] : 0.f, MEAN ? div_by(gv, dd[u], inv[u]) : gv, acc[e]);
                }
            }
            group_sum(d, p.lg);
            if constexpr (MEAN)
#pragma unroll
                for (int u = 0; u < U; ++u) d[u] *= inv[u];
            // lane q of a sub-group stores the dot product of its q-th slot
            for (int u0 = 0; u0 < U; u0 += L) {
                float val = d[0];
                int id = ee[0];
                bool on = ok[0] && u0 + q == 0;
#pragma unroll
                for (int u = 1; u < U; ++u)
                    if (u0 + q == u) val = d[u], id = ee[u], on = ok[u];
                if (on) p.grad_w[id] = val;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float o[EP];
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    const float gv = LN::get(v[u], e);
                    float c = gv;  // what grad x_j receives (0 where there is no slot: v is 0)
                    if constexpr (KIND == kRelu) c = xo[e] + share_get<T>(ev[u], e) > 0.f ? gv : 0.f;
                    if constexpr (KIND == kMul) {
                        o[e] = gv * xo[e];
                        acc[e] = fmaf(gv, share_get<T>(ev[u], e), acc[e]);
                    } else {
                        o[e] = c;
                        acc[e] += c;
                    }
                }
                if (ok[u] && act) stv<T, EP>(static_cast<T *>(p.grad_e) + (int64_t)ee[u] * p.F + f0, o);
            }
        }
    }
    // incoming edges of node j
    __device__ __forceinline__ float degree(int j) const {
        return MEAN ? static_cast<float>(p.deg_ptr[j + 1] - p.deg_ptr[j]) : 1.f;
    }
    // column (bit 31: cold), weight, edge id and degree of slot e
    __device__ __forceinline__ void fetch(int64_t e, int &c, float &w, int &id, float &d) const {
        c = __builtin_nontemporal_load(p.col + e);
        d = degree(c);
        if (hot > 0 && p.node_class[c] < hot) c |= static_cast<int>(0x80000000u);
        if constexpr (WEIGHT) w = __builtin_nontemporal_load(p.w + e);
        id = static_cast<int>(__builtin_nontemporal_load(p.perm + e));
    }
    __device__ __forceinline__ void run(int64_t r, int64_t s, int64_t t, int kind, int64_t slot) {
        begin(r);
        // Where the segment kernel sums in narrow windows, a row's chains there
        // are an eighth of its slots; over whole rows of 64 lanes they would be
        // all of them (20,000 rows of 150 slots, F = 256: 1.8e-7 against 8.8e-8
        // from 64 bits). There (BATCHED) the slots in flight, then 32 slots, are
        // summed by themselves before they join the row (8.8e-8; 9.4e-8 with the 64 of a
        // batch). Registers: a flag read at run time took two wavefronts per SIMD
        // from the kernels that are never batched.
        constexpr int NB = BATCHED ? EP : 1;
        float in_batch[NB], in_row[NB];
#pragma unroll
        for (int e = 0; e < NB; ++e) in_batch[e] = in_row[e] = 0.f;
        int nc = 0, ni = 0;
        float nw = 0.f, nd = 1.f;
        if (s + lane < t) fetch(s + lane, nc, nw, ni, nd);
        for (int64_t base = s; base < t; base += kWave) {
            const int n = static_cast<int>(uniform64((t - base) < kWave ? (t - base) : kWave));
            const int mc = nc, mi = ni;
            const float mw = nw, md = nd;
            if (base + kWave + lane < t) fetch(base + kWave + lane, nc, nw, ni, nd);
            for (int st = 0; st < n; st += S * U) {
                int jj[U], ee[U];
                float ww[U], dd[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int idx = st + u * S + sg;
                    ok[u] = idx < n;
                    jj[u] = __shfl(mc, idx & (kWave - 1), kWave);
                    ee[u] = __shfl(mi, idx & (kWave - 1), kWave);
                    if constexpr (WEIGHT) ww[u] = __shfl(mw, idx & (kWave - 1), kWave);
                    else ww[u] = 0.f;
                    dd[u] = 1.f;
                    if constexpr (MEAN) dd[u] = __shfl(md, idx & (kWave - 1), kWave);
                }
                take(jj, ok, ww, ee, dd);
                if constexpr (BATCHED) {
                    const bool flush = ((st + S * U) & 31) == 0 || st + S * U >= n;
#pragma unroll
                    for (int e = 0; e < EP; ++e) {
                        in_batch[e] += acc[e], acc[e] = 0.f;
                        if (flush) in_row[e] += in_batch[e], in_batch[e] = 0.f;
                    }
                }
            }
        }
        if constexpr (BATCHED)
#pragma unroll
            for (int e = 0; e < EP; ++e) acc[e] = in_row[e];
        for (int off = L; off < kWave; off <<= 1)
#pragma unroll
            for (int e = 0; e < EP; ++e) acc[e] += __shfl_xor(acc[e], off, kWave);
        if (sg != 0 || !act) return;
        if (kind == kRowFull) stv<T, EP>(static_cast<T *>(p.grad_x) + r * p.F + f0, acc);
        else stv<float, EP>(p.part + slot * p.F + f0, acc);
    }
    __device__ __forceinline__ void light(int64_t r, int64_t s, int64_t t, bool mine) {
        if (!mine) return;
        begin(r);
        for (int64_t b = s; b < t; b += U) {
            int jj[U], ee[U];
            float ww[U], dd[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = b + u < t;
                jj[u] = ok[u] ? p.col[b + u] : 0;
                ee[u] = ok[u] ? static_cast<int>(p.perm[b + u]) : 0;
                ww[u] = (WEIGHT && ok[u]) ? p.w[b + u] : 0.f;
                dd[u] = ok[u] ? degree(jj[u]) : 1.f;
            }
            take(jj, ok, ww, ee, dd);
        }
        if (act) stv<T, EP>(static_cast<T *>(p.grad_x) + r * p.F + f0, acc);
    }
};

template <typename TG, typename T, int KIND, int U, bool LIGHT, bool BATCHED>
__global__ __launch_bounds__(kBlock) void k_fused_backward(FusedParams p) {
    const int lane = threadIdx.x & (kWave - 1);
    int64_t c = uniform64((int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave);
    if (c < p.zero_items) {
        each_empty_row(p.walk.rowptr, p.walk.N, c, p.zero_rows, lane, [&](int64_t r) {
            for (int64_t f = lane; f < p.F; f += kWave) static_cast<T *>(p.grad_x)[r * p.F + f] = T(0);
        });
        return;
    }
    c -= p.zero_items;
    if (c >= p.walk.nchunks) return;
    FusedBackward<TG, T, KIND, U, BATCHED> op(p, lane);
    if constexpr (LIGHT) walk_light(p.walk, c, lane, p.lg, op);
    else walk_heavy(p.walk, c, lane, op);
}

struct FusedWs {
    float *part;
    int32_t *head_row, *hist, *hot;
    uint8_t *node_class;
    size_t bytes;
};

FusedWs carve_fused(void *base, int64_t N, int64_t F, int64_t E, int64_t chunk) {
    const int64_t nchunks = E > 0 ? (E + chunk - 1) / chunk : 0;
    Carver c(base);
    FusedWs w{};
    w.part = c.take<float>(2 * nchunks * F);
    w.head_row = c.take<int32_t>(nchunks);
    w.hist = c.take<int32_t>(kHotClasses);
    w.hot = c.take<int32_t>(1);
    w.node_class = c.take<uint8_t>(N);
    w.bytes = c.used + 256;
    return w;
}

template <typename TG, typename T, int KIND>
int launch_fused(const FusedParams &p, bool batched, hipStream_t s) {
    // slots in flight per lane: registers, and with them wavefronts, count for more
    constexpr int U = KIND == kWeight || KIND == kWeightMean ? 4 : 2;
    const unsigned grid = static_cast<unsigned>((p.zero_items + p.walk.nchunks + 3) / 4);
    const bool light = p.lg < 6 && p.walk.E <= kLightMaxDegree * p.walk.N;
    if constexpr (KIND != kRelu && KIND != kMul) {  // the segment kernel's windows take no other
        if (batched) {
            if (light) k_fused_backward<TG, T, KIND, U, true, true><<<grid, kBlock, 0, s>>>(p);
            else k_fused_backward<TG, T, KIND, U, false, true><<<grid, kBlock, 0, s>>>(p);
            PYG_LAUNCH_CHECK();
            return PYG_OK;
        }
    }
    if (light) k_fused_backward<TG, T, KIND, U, true, false><<<grid, kBlock, 0, s>>>(p);
    else k_fused_backward<TG, T, KIND, U, false, false><<<grid, kBlock, 0, s>>>(p);
    PYG_LAUNCH_CHECK();
    return PYG_OK;
}

template <typename TG, typename T>
int launch_kind(const FusedParams &p, int kind, bool batched, hipStream_t s) {
    if constexpr (sizeof(TG) == sizeof(T)) {
        if (kind == kWeight) return launch_fused<TG, T, kWeight>(p, batched, s);
        if constexpr (sizeof(T) == 4)
            if (kind == kWeightMean) return launch_fused<TG, T, kWeightMean>(p, batched, s);
    }
    if (kind == kAdd) return launch_fused<TG, T, kAdd>(p, batched, s);
    if (kind == kRelu) return launch_fused<TG, T, kRelu>(p, batched, s);
    return launch_fused<TG, T, kMul>(p, batched, s);
}

}  // namespace

size_t fused_backward_workspace(int64_t N, int64_t F, int64_t E, int64_t chunk) {
    return carve_fused(nullptr, N, F, E, segment_chunk(E, N, chunk)).bytes;
}

// Rows of whole 16-byte vectors of the gathered type, at most a wavefront of
// them, every array aligned to its share of a vector.
bool fused_backward_ok(const FusedBackwardArgs &a) {
    const int64_t ep = a.g_dtype == PYG_BF16 ? 8 : 4;
    const int64_t sz = a.dtype == PYG_BF16 ? 2 : 4;
    auto al = [](const void *q, int64_t b) { return reinterpret_cast<uintptr_t>(q) % b == 0; };
    // (weights: g in the type of x, as the dot products of the pass over the CSR
    // take it; a bf16 mean sums fp32 rows, 4 features a lane: the separate kernels)
    if (a.deg_ptr && a.dtype != PYG_F32) return false;
    return a.E > 0 && a.F > 0 && (a.msg != PYG_MSG_SRC || a.g_dtype == a.dtype) && a.F % ep == 0 &&
           a.F / ep <= kWave && a.perm && al(a.g, 16) && al(a.x, ep * sz) && al(a.edge_attr, ep * sz) &&
           al(a.grad_x, ep * sz) && al(a.grad_e, ep * sz);
}

int fused_backward(const FusedBackwardArgs &a, void *ws, size_t ws_bytes, hipStream_t s) {
    const int64_t chunk = segment_chunk(a.E, a.N, a.chunk);
    const FusedWs w = carve_fused(ws, a.N, a.F, a.E, chunk);
    if (!ws || ws_bytes < w.bytes) return PYG_ERR_WORKSPACE;
    FusedParams p{};
    // below 64-slot chunks the segment kernel leaves no light row to the whole
    // wavefront: nor here, for its bits
    const int64_t light_row = chunk < kMixedChunk ? chunk : light_row_slots(a.E, a.N, chunk);
    p.walk = {a.rowptr, a.N, a.E, chunk, light_row, (a.E + chunk - 1) / chunk, w.head_row};
    int64_t per = ((a.N + 1023) / 1024 + kWave - 1) / kWave * kWave;
    p.zero_rows = per > kWave ? per : kWave;
    p.zero_items = (a.N + p.zero_rows - 1) / p.zero_rows;
    const int64_t ep = a.g_dtype == PYG_BF16 ? 8 : 4, row_bytes = a.F * (16 / ep);
    while ((int64_t(1) << p.lg) < a.F / ep) ++p.lg;
    const bool batched = (a.msg == PYG_MSG_SRC || a.msg == PYG_MSG_EDGE_ADD) && segment_windows(a.N, row_bytes);
    p.F = a.F;
    p.col = a.col, p.perm = a.perm, p.w = a.weight;
    p.g = a.g, p.x = a.x, p.ea = a.edge_attr;
    p.grad_x = a.grad_x, p.grad_w = a.grad_w, p.grad_e = a.grad_e;
    p.part = w.part;
    if (hint_pays(a.N, row_bytes)) {
        PYG_TRY(hot_rows(a.rowptr, a.N, row_bytes, w.hist, w.node_class, w.hot, s));
        p.node_class = w.node_class;
        p.hot = w.hot;
    }
    const int kind = a.msg == PYG_MSG_EDGE_ADD ? kAdd : a.msg == PYG_MSG_EDGE_RELU ? kRelu
                     : a.msg == PYG_MSG_EDGE_MUL ? kMul : a.deg_ptr ? kWeightMean : kWeight;
    p.deg_ptr = a.deg_ptr;
    if (a.g_dtype == PYG_BF16) PYG_TRY((launch_kind<uint16_t, uint16_t>(p, kind, batched, s)));
    else if (a.dtype == PYG_BF16) PYG_TRY((launch_kind<float, uint16_t>(p, kind, batched, s)));
    else PYG_TRY((launch_kind<float, float>(p, kind, batched, s)));
    return segment_fold_pieces(a.rowptr, a.N, a.E, a.F, chunk, w.head_row, w.part, a.grad_x, a.dtype, s);
}

}  // namespace pyg
