// Sampled decoding (temperature > 0): token draws and the speculative-sampling verification.
//
// Section 1 cites the speculative-sampling rule for sampled decoding (temperatures 0.2 and 0.6 in the
// experiments) without printing it; this is that published rule.  A draft token x ~ q is kept with
// probability min(1, p(x)/q(x)); the first rejected draft is replaced by a draw from the normalised
// residual max(0, p - q); when every draft is kept one more token is drawn from the full model's next
// distribution.  q and p are softmax(logits / T) of the draft and the full model.
//
// Uniforms are counter based, so a run is reproducible and independent of how cycles fall:
//   U(e, c) = (mix64(stream + (3e + c + 1) * GOLD) >> 11) * 2^-53 for output index e and purpose c
//   (0 draft draw, 1 accept test, 2 replacement / extra / plain draw).
// Each draw is one workgroup of SAMPLE_THREADS threads; every reduction has a fixed order, decisions are taken in double on
// fp32 weights.
//
// What bounds a draw is latency: 128 KB of logits through one compute unit and a chain of reductions.  A wave holds a
// contiguous run of a row as 256-value tiles, four values per lane and tile, so that its loads are whole lines all in flight
// at once (a thread-contiguous split touched 64 lines per load); sums go through shuffles and one LDS exchange of the 16
// waves' totals instead of a halving tree with a barrier per level; only the one wave that the drawn point falls into
// walks its tiles again.  The softmax statistics of a verification pass's rows are a launch of their own, one
// workgroup per row, instead of one workgroup walking row after row.  7B vocabulary (32000): draft draw 33 -> 13 us, acceptance of four
// drafts 92 -> 7 + 15 us.
#pragma once
#include "asd_common.h"
#include "asd_misc.h"

#define SAMPLE_THREADS 1024

struct SampleArgs {
    const float* logits;     // [rows][V] logits of the pass just finished
    float* qlogits;          // [draft steps][V] draft-model logits kept until the verification
    double* qstat;           // [draft steps][2] their softmax statistics (maximum, Z), left by the draft draws
    double* pstat;           // [rows][2] the statistics of the verification pass's rows
    int32_t V;
    float inv_T;
    uint64_t stream;         // key of the sampling stream (from the seed)
    DevState* st;
    int32_t* tokbuf;
    int32_t* out;
};

__device__ __forceinline__ double sample_uniform(uint64_t stream, int64_t index, int purpose) {
    const uint64_t G = 0x9E3779B97F4A7C15ULL;
    const uint64_t c = (uint64_t)(3 * index + purpose);
    return (double)(mix64(stream + (c + 1) * G) >> 11) * (1.0 / 9007199254740992.0);
}

#define SAMPLE_WAVES (SAMPLE_THREADS / 64)
// reductions over a wave (every lane gets the result; the butterfly adds the same pairs in every lane)
__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
// the waves' values side by side in LDS, visible to every thread on return
template <class V> __device__ __forceinline__ void share_waves(V v, V* red) {
    __syncthreads();                      // the last exchange has been read
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
}
__device__ __forceinline__ float blk_max(float v, double* red) {
    share_waves((float)wave_max(v), (float*)red);
    float r = ((float*)red)[0];
#pragma unroll
    for (int i = 1; i < SAMPLE_WAVES; ++i) r = fmaxf(r, ((float*)red)[i]);
    return r;
}
__device__ __forceinline__ double blk_sum(double v, double* red) {
    share_waves(wave_sum(v), red);
    double r = red[0];
#pragma unroll
    for (int i = 1; i < SAMPLE_WAVES; ++i) r += red[i];
    return r;
}

// A wave's share of a row of V values (a multiple of 4): tiles tile0 .. tile0 + n - 1 of 256 values, value 4 lane + j of a
// tile in lane's component j.  TILES > 0: held in registers (V <= TILES * 256 * SAMPLE_WAVES), values past the row are -inf.
// TILES = 0: read from memory at every use (any V).  Both run the same arithmetic in the same order.
#define SAMPLE_TILES 8
#define SAMPLE_REG_MAX (SAMPLE_TILES * 256 * SAMPLE_WAVES)

template <int TILES>
struct RowTiles {
    const float* row;
    int V, n, first;                      // first: index of this lane's first value
    float4 v[TILES > 0 ? TILES : 1];
    __device__ __forceinline__ int index(int k) const { return first + 256 * k; }
    __device__ __forceinline__ void load(const float* r, int V_) {
        const int tiles = (V_ + 255) / 256;
        row = r; V = V_; n = (tiles + SAMPLE_WAVES - 1) / SAMPLE_WAVES;
        first = (int)(threadIdx.x >> 6) * n * 256 + 4 * (int)(threadIdx.x & 63);
        if constexpr (TILES > 0) {
#pragma unroll
            for (int k = 0; k < TILES; ++k) v[k] = k < n ? at(k) : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        }
    }
    __device__ __forceinline__ float4 at(int k) const {
        const int i = index(k);
        return i < V ? *(const float4*)(row + i) : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    // f(k, values) for the wave's tiles in ascending order; the register variant also visits tiles n .. TILES-1 (all -inf)
    template <class F> __device__ __forceinline__ void each(F f) const {
        if constexpr (TILES > 0) {
#pragma unroll
            for (int k = 0; k < TILES; ++k) f(k, v[k]);
        } else {
            for (int k = 0; k < n; ++k) f(k, at(k));
        }
    }
    __device__ __forceinline__ float4 tile(int k) const {                 // k the same in every lane of the wave
        if constexpr (TILES > 0) {
            float4 x = v[0];
#pragma unroll
            for (int i = 1; i < TILES; ++i) if (k == i) x = v[i];
            return x;
        } else {
            return at(k);
        }
    }
};

__device__ __forceinline__ float4 softmax_weights(const float4& x, float mx, float inv_T) {
    return float4{expf((x.x - mx) * inv_T), expf((x.y - mx) * inv_T), expf((x.z - mx) * inv_T), expf((x.w - mx) * inv_T)};
}

__device__ __forceinline__ double lane_sum(const float4& x) { return ((double)x.x + (double)x.y) + ((double)x.z + (double)x.w); }

// A lane's sums of the weights w(index, values) of its tiles: one by one (register variant) and altogether
template <int TILES> struct TileSums { double tile[TILES > 0 ? TILES : 1], all; };
template <int TILES, class F>
__device__ __forceinline__ void tile_sums(const RowTiles<TILES>& r, F w, TileSums<TILES>& s) {
    s.all = 0.0;
    r.each([&](int k, float4 x) {
        const double v = lane_sum(w(r.index(k), x));
        if constexpr (TILES > 0) s.tile[k] = v;
        s.all += v;
    });
}

// softmax statistics of a logit row at temperature 1/inv_T: the maximum, and Z = sum exp((l - max) * inv_T) of whose terms
// the sums are left in s
template <int TILES>
__device__ __forceinline__ void row_stats(const RowTiles<TILES>& r, float inv_T, float* mx, double* Z, TileSums<TILES>& s, double* red, DevState* st) {
    float m = -INFINITY;
    r.each([&](int, float4 x) { m = fmaxf(fmaxf(m, fmaxf(x.x, x.y)), fmaxf(x.z, x.w)); });
    const float mxv = blk_max(m, red);
    // a row without a maximum (every logit NaN or -inf) is reported as the greedy pass reports it
    if (mxv == -INFINITY && threadIdx.x == 0) __hip_atomic_fetch_or(&st->err, (int)DEV_ERR_LOGITS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tile_sums(r, [&](int, const float4& x) { return softmax_weights(x, mxv, inv_T); }, s);
    *mx = mxv;
    *Z = blk_sum(s.all, red);
}

// ---- where a point of a running sum falls (plain functions: the CPU tests compile and run them too)
#define SAMPLE_HD __host__ __device__ __forceinline__
// Intervals laid end to end from `run`, visited in order: the first whose end exceeds t, and the running sum before it.  Where
// rounding leaves none (a level's sums are added in another order than the level above added them), the last interval
// with a positive sum, and a running sum that stays below every t: all levels inside it then take their last one as well.
struct IntervalSearch {
    double t, run, before;
    int hit, last;
    SAMPLE_HD IntervalSearch(double t_, double run_) : t(t_), run(run_), before(-(double)INFINITY), hit(-1), last(0) {}
    SAMPLE_HD void visit(int i, double sum) {
        if (hit < 0 && t < run + sum) { hit = i; before = run; }
        if (sum > 0.0) last = i;
        run += sum;
    }
    SAMPLE_HD int index() const { return hit >= 0 ? hit : last; }
};
// The lane of a tile: over: lanes whose inclusive running sum exceeds t; some: lanes with a positive sum.  The scan adds in
// a different order for every lane, so `over` may begin at a lane without any weight: only lanes with some are asked.
SAMPLE_HD int sample_lane(uint64_t over, uint64_t some) {
    over &= some;
    return over ? __builtin_ctzll(over) : some ? 63 - __builtin_clzll(some) : 0;
}
// The value of a lane's four, z = running sum before them: the first that carries it past t, else the last positive one
SAMPLE_HD int sample_of_four(const float (&e)[4], double z, double t) {
    int pick = -1, pos = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        z += (double)e[j];
        if (pick < 0 && e[j] > 0.f && z > t) pick = j;
        if (e[j] > 0.f) pos = j;
    }
    return pick >= 0 ? pick : pos;
}

// The last index with a positive weight, or -1 (every thread).  Off the usual path: the row is read anew, because keeping the caller's tiles for
// it spilled registers of the usual path (draft draw 13.1 -> 14.3 us).
template <class F>
__device__ __forceinline__ int blk_last_positive(const float* row, int V, F w, double* red) {
    RowTiles<0> r;
    r.load(row, V);
    int best = -1;
#pragma unroll 1
    for (int k = 0; k < r.n; ++k) {
        const float4 q = w(r.index(k), r.at(k));
        const int i = r.index(k), j = q.w > 0.f ? 3 : q.z > 0.f ? 2 : q.y > 0.f ? 1 : q.x > 0.f ? 0 : -1;
        if (j >= 0) best = i + j;
    }
    for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o));
    share_waves(best, (int*)red);
#pragma unroll
    for (int i = 0; i < SAMPLE_WAVES; ++i) best = max(best, ((int*)red)[i]);
    return best;
}

// Inverse-CDF draw from the non-negative weights w(index, values) of a row's tiles, whose sums are in s: an index whose interval of
// the running sum holds u * total (the smallest index whose running sum exceeds it, sums taken tile by tile); where
// rounding leaves none at some level (wave, tile, lane, value), the last positive one of that level.  The drawn index never has
// weight zero.  A row with a NaN among its weights has no running sum: its last index with a positive weight.  Every thread
// returns the drawn index, or -1 if no weight is positive.
template <int TILES, class F>
__device__ __forceinline__ int blk_sample(const RowTiles<TILES>& r, F w, const TileSums<TILES>& s, double u, double* red, int* ired) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    share_waves(wave_sum(s.all), red);
    double total = 0.0;
#pragma unroll
    for (int i = 0; i < SAMPLE_WAVES; ++i) total += red[i];
    if (total == 0.0) return -1;
    if (__builtin_expect(!(total > 0.0), 0)) return blk_last_positive(r.row, r.V, w, red);
    const double t = u * total;
    IntervalSearch waves(t, 0.0);
#pragma unroll
    for (int i = 0; i < SAMPLE_WAVES; ++i) waves.visit(i, red[i]);
    if (wave == waves.index()) {
        IntervalSearch tiles(t, waves.before);
        if constexpr (TILES > 0) {
            double sum[TILES];
#pragma unroll
            for (int k = 0; k < TILES; ++k) sum[k] = wave_sum(s.tile[k]);
#pragma unroll
            for (int k = 0; k < TILES; ++k) tiles.visit(k, sum[k]);
        } else {
            for (int k = 0; k < r.n; ++k) tiles.visit(k, wave_sum(lane_sum(w(r.index(k), r.at(k)))));
        }
        const int kt = tiles.index();
        const float4 q = w(r.index(kt), r.tile(kt));
        const double sl = lane_sum(q);
        double incl = sl;                                             // running sum over the lanes
        for (int o = 1; o < 64; o <<= 1) { const double up = __shfl_up(incl, o); if (lane >= o) incl += up; }
        const double before = __shfl_up(incl, 1);
        const int hit = sample_lane(__ballot(t < tiles.before + incl), __ballot(sl > 0.0));
        if (lane == hit) {
            const float e[4] = {q.x, q.y, q.z, q.w};
            ired[0] = r.index(kt) + sample_of_four(e, tiles.before + (lane ? before : 0.0), t);
        }
    }
    __syncthreads();
    return ired[0];
}

// After a draft step: keep its logits for the verification and draw the draft token of output index
// index_base + emitted + j into row j+1 of the coming verification pass (keep: this workgroup writes them).  Every thread returns the token.
template <int TILES>
__device__ __forceinline__ int draft_draw(const SampleArgs& a, const int j, const bool keep, double* red, int* ired) {
    float* kept = a.qlogits + (size_t)j * a.V;
    const int64_t index = (int64_t)a.st->index_base + a.st->emitted + j;
    RowTiles<TILES> r;
    r.load(a.logits, a.V);
    if (keep) r.each([&](int k, float4 x) { if (r.index(k) < a.V && k < r.n) *(float4*)(kept + r.index(k)) = x; });
    float mx; double Z;
    const float inv_T = a.inv_T;
    TileSums<TILES> s;
    row_stats(r, inv_T, &mx, &Z, s, red, a.st);
    const int tok = max(0, blk_sample(r, [&](int, const float4& x) { return softmax_weights(x, mx, inv_T); }, s, sample_uniform(a.stream, index, 0), red, ired));
    if (keep && threadIdx.x == 0) { a.tokbuf[j + 1] = tok; a.qstat[2 * j] = (double)mx; a.qstat[2 * j + 1] = Z; }
    return tok;
}
template <int TILES>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_draft_kernel(const SampleArgs a, int j) {
    __shared__ double red[SAMPLE_WAVES];
    __shared__ int ired[1];
    draft_draw<TILES>(a, j, true, red, ired);
}
// Between two draft steps: the draw and the embedding of the token, in one launch of EMBED_SPLIT workgroups, each of which draws for itself (the draw is one workgroup's latency,
// and the logits come to eight nearly as fast as to one; see finish_embed_kernel).  Vocabulary 32000, 4096 features: 13.0 + 4.6 us and the gap between them -> 15.2 us.  Calls
// that sample 24 tokens with four or eight drafts (7B, 13B and 512-feature fp32 widths, one to four layers, vocabularies of 1024 to 128256), four processes of each build in turn: 1.001 to
// 1.008x, runs of one build within 0.7 % (13B width, 8 drafts: 5126 -> 5099 us; 512 features: 2846 -> 2824; vocabulary 128256, re-read by every workgroup: 8713 -> 8701).
template <class T, int TILES>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_draft_embed_kernel(const SampleArgs a, int j, const typename T::elem* E, int d, const float* g_first,
                                                                            float* xres, void* xb, size_t xb_plane, float* part) {
    __shared__ double red[SAMPLE_WAVES];
    __shared__ int ired[1];
    __shared__ float sums[EMBED_THREADS];
    const int tok = draft_draw<TILES>(a, j, blockIdx.x == 0, red, ired);
    embed_block<T>(E, nullptr, d, a.V, a.st, g_first, xres, xb, xb_plane, 1, part, blockIdx.x, 0, sums, tok);
}

// A plain draw (purpose 2) of output index `index` from logits row `row` into tokbuf[0]: the prompt pass's token.
template <int TILES>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_plain_kernel(const SampleArgs a, int row, int64_t index) {
    __shared__ double red[SAMPLE_WAVES];
    __shared__ int ired[1];
    RowTiles<TILES> r;
    r.load(a.logits + (size_t)row * a.V, a.V);
    float mx; double Z;
    const float inv_T = a.inv_T;
    TileSums<TILES> s;
    row_stats(r, inv_T, &mx, &Z, s, red, a.st);
    const int tok = max(0, blk_sample(r, [&](int, const float4& x) { return softmax_weights(x, mx, inv_T); }, s, sample_uniform(a.stream, index, 2), red, ired));
    if (threadIdx.x == 0) a.tokbuf[0] = tok;
}

// grid = rows: the softmax statistics of the verification pass's rows, for sample_accept_kernel
template <int TILES>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_stats_kernel(const SampleArgs a) {
    __shared__ double red[SAMPLE_WAVES];
    RowTiles<TILES> r;
    r.load(a.logits + (size_t)blockIdx.x * a.V, a.V);
    float mx; double Z;
    TileSums<TILES> s;
    row_stats(r, a.inv_T, &mx, &Z, s, red, a.st);
    if (threadIdx.x == 0) { a.pstat[2 * blockIdx.x] = (double)mx; a.pstat[2 * blockIdx.x + 1] = Z; }
}

// After a verification pass over rows [last, d_1 .. d_kk] and sample_stats_kernel on its rows: speculative-sampling accept /
// replace, then the same bookkeeping as the greedy accept step (emit, advance the cache length by a + 1, next first row).
template <int TILES>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_accept_kernel(const SampleArgs a, int kk) {
    __shared__ double red[SAMPLE_WAVES];
    __shared__ int ired[1];
    const int V = a.V, lane = threadIdx.x & 63;
    const float inv_T = a.inv_T;
    const int64_t e0 = (int64_t)a.st->index_base + a.st->emitted;
    // draft i's decision in lane i of every wave (kk < 64)
    bool kept = true;
    if (lane < kk) {
        const float* ql = a.qlogits + (size_t)lane * V;
        const float* pl = a.logits + (size_t)lane * V;
        const int x = a.tokbuf[lane + 1];
        // (both rows' statistics: the same arithmetic on the same values as where they were taken)
        const float mq = (float)a.qstat[2 * lane], mp = (float)a.pstat[2 * lane];
        const double Zq = a.qstat[2 * lane + 1], Zp = a.pstat[2 * lane + 1];
        const double q = (double)expf((ql[x] - mq) * inv_T) / Zq, p = (double)expf((pl[x] - mp) * inv_T) / Zp;
        kept = sample_uniform(a.stream, e0 + lane, 1) * q < p;
    }
    const unsigned long long rejected = __ballot(!kept);
    const int acc = rejected ? __ffsll((long long)rejected) - 1 : kk;      // the same in every wave
    // the token after the kept drafts: a draw from the normalised residual of the first rejected one's row, from p should the
    // residual vanish; with all kept, from the last row's p
    const float mp = (float)a.pstat[2 * acc];
    const double u = sample_uniform(a.stream, e0 + acc, 2);
    RowTiles<TILES> rp;
    rp.load(a.logits + (size_t)acc * V, V);
    TileSums<TILES> s;
    int next = -1;
    if (acc < kk) {
        const float* ql = a.qlogits + (size_t)acc * V;
        const float mq = (float)a.qstat[2 * acc];
        const float iZq = (float)(1.0 / a.qstat[2 * acc + 1]), iZp = (float)(1.0 / a.pstat[2 * acc + 1]);
        auto resid = [&](int i, const float4& x) {
            const float4 y = i < V ? *(const float4*)(ql + i) : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            const float4 p = softmax_weights(x, mp, inv_T), q = softmax_weights(y, mq, inv_T);
            return float4{fmaxf(0.f, p.x * iZp - q.x * iZq), fmaxf(0.f, p.y * iZp - q.y * iZq), fmaxf(0.f, p.z * iZp - q.z * iZq), fmaxf(0.f, p.w * iZp - q.w * iZq)};
        };
        tile_sums(rp, resid, s);
        next = blk_sample(rp, resid, s, u, red, ired);
    }
    if (next < 0) {
        auto from_p = [&](int, const float4& x) { return softmax_weights(x, mp, inv_T); };
        tile_sums(rp, from_p, s);
        next = max(0, blk_sample(rp, from_p, s, u, red, ired));
    }
    if (threadIdx.x != 0) return;
    DevState* st = a.st;
    int e = st->emitted;
    for (int q = 1; q <= acc && e < st->target; ++q) a.out[e++] = a.tokbuf[q];
    if (e < st->target) a.out[e++] = next;
    st->emitted = e;
    st->pos += acc + 1;
    st->cycles += 1; st->drafted += kk; st->accepted += acc;
    a.tokbuf[0] = next;
}
