// Decode passes of small fp32 models: one launch per sublayer instead of five per layer.
//
// A pass of such a model is a chain of launches of 3 to 6 us each that hardly compute: 256 features, 4 layers: 22 launches, 99 us.
// Here a sublayer is one launch of SM_SLICES workgroups, one per K slice of its residual projection (the slices that the
// eight waves of gemm_kernel<EPI_RES> take): the workgroup computes everything that its slice of the projection needs, so nothing
// is exchanged inside the launch:
//   sm_attn_kernel  its slice is HS = q_dim / 8 dims of one head: that head's q and K rows and HS rows of V (q and K again in
//                   the other workgroups of the head), rotary, the head's attention, HS output dims, their share of the O-projection;
//   sm_mlp_kernel   its slice is every eighth hidden tile: the gate and up rows of those, SiLU, their share of the down-projection;
//   sm_lm_kernel    64 logits per workgroup.
// Each begins with what the sublayer before left open: it adds the eight slices to the residual stream and takes the norm
// (or embeds its tokens), in every workgroup alike; workgroup 0 writes the stream and finishes the cosine.  The stream and
// the slices alternate between two buffers, because a launch reads the old ones while its workgroup 0 writes the new.
//
// The bits are those of the launches this replaces.  A 16x16x4 fp32 matrix instruction adds its four products to the
// accumulator as a chain of fused multiply-adds in ascending k (measured: 4M outputs, magnitudes down to subnormal, no
// difference), so an output of gemm_kernel is one chain per wave over its k-blocks (within a k-block component j of the four lane
// groups' fragments, j = 0..3) and the waves' sums in order.  Here a lane runs that chain for its weight row: with v_fma for one row, with
// 4x4x1 matrix instructions (64 weight rows x 4 activation rows, one k per instruction: the same chain) for more.
//
// What bounds a launch is latency.  One row, 256 features, 64 head dims, context 45, ns from a workgroup's first instruction: input whole 1150 (the arguments, then the slices from
// other XCDs' L2s), q/K/V rows 2700, rotated 3100, attention 4800, merged 5300, done 5700; the MLP 1750, 3100, 3500, 4300.  A pass (4 layers) 99 -> 55 us for one row, 101 -> 78 for five.
#pragma once
#include "asd_attn.h"
#include "asd_gemm.h"
#include "asd_misc.h"

#define SM_SLICES 8
#define SM_NW 12                    // waves per workgroup: three on a SIMD, 168 registers each
#define SM_NT (SM_NW * 64)
#define SM_D 256                    // most features
#define SM_Q 256                    // most query dims (heads x head_dim)
#define SM_FFN_TILES 6              // most hidden tiles per slice (d_ffn <= 768)
#define SM_CHUNKS SM_NW             // most 64-key chunks of the context: one per wave
#define SM_ROWS 8                   // most rows of a pass (the caller's rule)
#define SM_LM_NW 8

struct SmallIn {                    // a sublayer's input
    const float* xin;               // [M][d] residual stream before the open projection
    const float* part;              // [SM_SLICES][M][d] the open projection's slices
    float* xout;                    // [M][d] the stream with it (NULL: nobody reads it)
    const float* gain;              // gain of this sublayer's norm
    float* ssq;                     // [16] ||x||^2 of the stream before
    float* fin_cos_rows;            // as GemmArgs
    double* fin_cos_acc;
    int32_t d, M;
    float inv_d, eps;
    int32_t embed;                  // the input is the embedding of the tokens (xin and part are read ahead all the same, and dropped)
    // embedding: ids from BeginArgs (n_tok > 0) or tokens; cand: the last row's is the greedy token of these candidates, draft number `draft`
    const float* E;
    const int32_t* tokens;
    const AmaxCand* cand;
    int32_t* argmax;
    int32_t* tokbuf;
    DevState* st;
    int32_t vocab, P, draft;
    int32_t has_begin;              // the call starts here: its state is set up as well (BeginArgs, an argument of its own: what is indexed must not be copied)
};
struct SmallAttn {
    const float* Wo;
    float* part_out;
    float* kv;                      // this layer's cache pages
    const int32_t* page_table;
    int32_t pos_off, page_tokens, nc;
    float scale;
};
// ---- chains
// Rows of a pass a kernel instance takes: 4 RM in matrix instructions, RV (0 or 1) more by v_fma beside them (one row alone, and the fifth of a
// verification of four drafts, would leave three of four columns empty)
template <int RM, int RV> struct SmAcc { f32x4 v[RM ? RM : 1]; float s; };
template <int RM, int RV> __device__ __forceinline__ void sm_zero(SmAcc<RM, RV>& a) {
    a.s = 0.f;
#pragma unroll
    for (int c = 0; c < RM; ++c) a.v[c] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// this lane's weight row r (0..15 of a tile) of one k-block: the four lane groups' 16-byte pieces
__device__ __forceinline__ void sm_load(f32x4 (&w)[4], const float* frag, int r) {
#pragma unroll
    for (int g = 0; g < 4; ++g) w[g] = *(const f32x4*)(frag + (g * 16 + r) * 4);
}
__device__ __forceinline__ void sm_hold(float& x) { asm volatile("" : "+v"(x)); }
// activations of one k-block: rows c * 4 + (lane & 3) of RM groups, and the row after them (the same address in every lane)
template <int RM, int RV> struct SmX { f32x4 b[RM ? RM : 1][4], s[4]; };
template <int RM, int RV> __device__ __forceinline__ void sm_read(SmX<RM, RV>& b, const float* x, int xs, int lane) {
    const float* xl = x + (lane & 3) * xs;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int c = 0; c < RM; ++c) b.b[c][g] = *(const f32x4*)(xl + c * 4 * xs + 4 * g);
        if constexpr (RV != 0) b.s[g] = *(const f32x4*)(x + RM * 4 * xs + 4 * g);
    }
}
// The chain over n (at least 1) of N k-blocks; x = row 0 of the first one's 16 values in LDS, xs floats to the next row, xk to the next k-block's; seen(b) is called with the
// activations of each.  The next k-block's are read beside this one's products where registers allow; the scheduler is held to that (left alone it reads
// all of them first, and spills), the sums that are plain arithmetic by empty statements that take them as an operand.
template <int RM, int RV, int N, class F>
__device__ __forceinline__ void sm_chain(SmAcc<RM, RV>& a, const f32x4 (&w)[N][4], int n, const float* x, int xk, int xs, int lane, F seen) {
    constexpr bool AHEAD = RM + RV <= 1;
    SmX<RM, RV> b[AHEAD ? 2 : 1];
    sm_read(b[0], x, xs, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i >= n) break;
        SmX<RM, RV>& u = b[AHEAD ? i & 1 : 0];
        if constexpr (AHEAD) {
            if (i + 1 < N) sm_read(b[(i + 1) & 1], x + (i + 1 < n ? i + 1 : 0) * xk, xs, lane);
        } else if (i > 0) sm_read(u, x + i * xk, xs, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
#pragma unroll
                for (int c = 0; c < RM; ++c) a.v[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[i][g][j], u.b[c][g][j], a.v[c], 0, 0, 0);
                if constexpr (RV != 0) a.s = __builtin_fmaf(w[i][g][j], u.s[g][j], a.s);
            }
        if constexpr (RV != 0) sm_hold(a.s);
        seen(u);
        __builtin_amdgcn_sched_barrier(0);
    }
}
template <int RM, int RV, int N>
__device__ __forceinline__ void sm_chain(SmAcc<RM, RV>& a, const f32x4 (&w)[N][4], int n, const float* x, int xk, int xs, int lane) {
    sm_chain(a, w, n, x, xk, xs, lane, [](const auto&) {});
}
// a wave's 64 weight rows x activation rows to out[row m][64 values], os floats between the rows; the first n values
template <int RM, int RV> __device__ __forceinline__ void sm_put(const SmAcc<RM, RV>& a, float* out, int os, int lane, int n = 64) {
#pragma unroll
    for (int c = 0; c < RM; ++c)
        if ((lane & ~3) < n) *(f32x4*)(out + (size_t)(c * 4 + (lane & 3)) * os + (lane & ~3)) = a.v[c];
    if (RV != 0 && lane < n) out[(size_t)RM * 4 * os + lane] = a.s;
}
// the same to a global array [M][d] from feature n0 on, of which n (a multiple of 16) exist
template <int RM, int RV> __device__ __forceinline__ void sm_put_global(const SmAcc<RM, RV>& a, float* out, int d, int n0, int n, int M, int lane) {
#pragma unroll
    for (int c = 0; c < RM; ++c) {
        const int m = c * 4 + (lane & 3);
        if (m < M && (lane & ~3) < n) *(f32x4*)(out + m * d + n0 + (lane & ~3)) = a.v[c];
    }
    if (RV != 0 && RM * 4 < M && lane < n) out[RM * 4 * d + n0 + lane] = a.s;
}
// maximum over the lanes that share lane & 3 (ALL: over all lanes), in every lane, without a trip through LDS
template <bool ALL> __device__ __forceinline__ float sm_max(float v) {
    auto dpp = [](float x, auto ctrl) { return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, false)); };
    if constexpr (ALL) {
        v = fmaxf(v, dpp(v, std::integral_constant<int, 0xb1>{}));       // quad_perm: lane ^ 1
        v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4e>{}));       // quad_perm: lane ^ 2
    }
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x124>{}));          // row_ror:4
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x128>{}));          // row_ror:8
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// ---- input stage
#define SM_XS (SM_D + 4)            // row stride of x in LDS: rows four banks apart
template <int NR> struct SmInLds {
    float x[NR][SM_XS];               // normed input before the row scale: y * gain
    float pyy[NR][SM_D + 4], pxy[NR][SM_D + 4];
    float tyy[NR][16], txy[NR][16];
    float yy[16], xy[16];
    int tok[16];
};
// Wave m takes row m, lane l its features 4 l .. 4 l + 3.  The loads are requested before the weights' (loads return in order).  What bounds the stage is the issue of loads: a
// compute unit takes one of 1 KiB in about 16 cycles, its oldest waves' first, and a wave gets to its input when all its own are issued.  Hence 16 bytes per lane, the
// oldest waves, and only the first of a wave's weights before it (a feature per thread and all weights before it: the input was whole at 2250 ns instead of 1150, in the MLP at 2700
// instead of 1750; a pass 60 -> 55 us for one row, 77 -> 69 for four, 87 -> 78 for five).
struct SmFirst { f32x4 x, g, p[SM_SLICES]; };
__device__ __forceinline__ void sm_request(const SmallIn& a, SmFirst& f, int w, int lane) {
    if (w >= a.M) return;                                         // (the same for a whole wave)
    const int n = min(4 * lane, a.d - 4);
#pragma unroll
    for (int s = 0; s < SM_SLICES; ++s) f.p[s] = *(const f32x4*)(a.part + (s * a.M + w) * a.d + n);
    f.x = *(const f32x4*)(a.xin + w * a.d + n);
    f.g = *(const f32x4*)(a.gain + n);
}
// y = x + the eight slices in order, into LDS as y * gain with the products of the cosine's sums; x is whole after the next barrier
template <int NT, int NR> __device__ __forceinline__ void sm_input(const SmallIn& a, const BeginArgs& begin, const SmFirst& f, SmInLds<NR>& l, int tid, int w, int lane) {
#pragma clang fp contract(off)
    static_assert(NT / 64 >= SM_ROWS, "a wave per row");
    if (!a.embed) {
        const int n = 4 * lane;
        if (w >= a.M) return;
        f32x4 y, xg, yy, xy;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = 0.f;
#pragma unroll
            for (int s = 0; s < SM_SLICES; ++s) v += f.p[s][i];
            y[i] = f.x[i] + v;
            xg[i] = y[i] * f.g[i];
            yy[i] = y[i] * y[i];
            xy[i] = f.x[i] * y[i];
        }
        if (n < a.d) {
            *(f32x4*)&l.x[w][n] = xg;
            *(f32x4*)&l.pyy[w][n] = yy;
            *(f32x4*)&l.pxy[w][n] = xy;
            if (blockIdx.x == 0 && a.xout) *(f32x4*)(a.xout + w * a.d + n) = y;
        }
        return;
    }
    const int n = tid % SM_D;
    // the tokens of the pass
    if (tid < 64) {
        float conf;
        int tok = 0;
        if (tid < a.M) tok = a.has_begin && begin.n_tok ? begin.tok[tid & 15] : a.tokens[tid];
        if (a.cand) {
            const bool writer = blockIdx.x == 0;
            const int idx = row_winner(a.cand, a.P, a.vocab, a.st, writer, writer ? &conf : nullptr);
            if (tid == a.M - 1) {
                tok = idx;
                if (writer) { a.argmax[0] = idx; a.tokbuf[a.draft + 1] = idx; a.st->conf = conf; }
            }
        }
        // (an id that is no row of the table must not become an address: row 0, and the state's error bit)
        const bool bad = (unsigned)tok >= (unsigned)a.vocab;
        const int err = __any(bad) ? DEV_ERR_TOKEN : 0;
        if (tid < a.M) l.tok[tid] = bad ? 0 : tok;
        if (blockIdx.x == 0) {
            if (a.has_begin) begin_state(begin, tid, 64, err);
            else if (err && tid == 0) __hip_atomic_fetch_or(&a.st->err, (int)DEV_ERR_TOKEN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (n >= a.d) return;
    const float g = a.gain[n];
    for (int m = tid / SM_D; m < a.M; m += NT / SM_D) {
        const float x = a.E[(size_t)l.tok[m] * a.d + n];
        l.x[m][n] = x * g;
        l.pyy[m][n] = x * x;
        if (blockIdx.x == 0 && a.xout) a.xout[m * a.d + n] = x;
    }
}
// The rows' scales (for everybody after the next barrier) and, in workgroup 0, the cosine of the sublayer before: waves of 64 threads from thread 0 on, four rows each, 16
// threads per row.  Sums as the launches this replaces take them: 16 features in order, then these in order; the embedding's in
// EMBED_SPLIT parts, each a halving tree.
template <int NR> __device__ __forceinline__ void sm_norms(const SmallIn& a, SmInLds<NR>& l, int tid) {
#pragma clang fp contract(off)
    const int m = tid >> 4, q = tid & 15;
    if ((tid & ~63) >= a.M * 16) return;                          // (whole waves)
    const bool on = m < a.M, writer = blockIdx.x == 0;
    float yy = 0.f, xy = 0.f;
    if (!a.embed) {
        if (on && q < a.d / 16) {
            f32x4 p[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = *(const f32x4*)&l.pyy[m][q * 16 + 4 * i];
#pragma unroll
            for (int i = 0; i < 16; ++i) yy += p[i >> 2][i & 3];
            if (writer) {
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = *(const f32x4*)&l.pxy[m][q * 16 + 4 * i];
#pragma unroll
                for (int i = 0; i < 16; ++i) xy += p[i >> 2][i & 3];
            }
        }
    } else if (on && q < EMBED_SPLIT) {
        // (d <= 256: at most 32 of the tree's leaves are not zero)
        const int per = a.d / EMBED_SPLIT;
        auto leaf = [&](int i) { return i < per ? l.pyy[m][q * per + i] : 0.f; };
        auto quad = [&](int i) { return (leaf(i) + leaf(i + 16)) + (leaf(i + 8) + leaf(i + 24)); };       // levels 16, 8
        auto oct = [&](int i) { return quad(i) + quad(i + 4); };                                          // level 4
        yy = (oct(0) + oct(2)) + (oct(1) + oct(3));                                                       // levels 2, 1
    }
    if (on) { l.tyy[m][q] = yy; l.txy[m][q] = xy; }               // (zero where there is no part: the sums below run over all 16)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (on && q == 0) {
        f32x4 p[4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { p[i] = *(const f32x4*)&l.tyy[m][4 * i]; r[i] = *(const f32x4*)&l.txy[m][4 * i]; }
        yy = 0.f; xy = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) { yy += p[i >> 2][i & 3]; xy += r[i >> 2][i & 3]; }
        l.yy[m] = yy; l.xy[m] = xy;
    }
}
__device__ __forceinline__ float sm_scale(float yy, float inv_d, float eps) { return rsqrtf(yy * inv_d + eps); }
// Workgroup 0, one wave that has nothing else to do at the end, long after the sums became visible: cosines and ||x||^2 as gemm_block leaves them
template <int NR> __device__ __forceinline__ void sm_finish(const SmallIn& a, SmInLds<NR>& l, int lane) {
    double acc = 0.0;
    if (a.fin_cos_rows) acc = *a.fin_cos_acc;
    if (lane < a.M) {
        const float yy = l.yy[lane], xy = l.xy[lane];
        if (a.fin_cos_rows) {
            const float xx = a.ssq[lane];
            float c = xy * rsqrtf(fmaxf(xx, 1e-16f) * fmaxf(yy, 1e-16f));
            c = fminf(1.f, fmaxf(-1.f, c));
            a.fin_cos_rows[lane] = c;
            l.xy[lane] = c;
        }
        a.ssq[lane] = yy;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane == 0 && a.fin_cos_rows) {
        double sum = 0.0;
        for (int r = 0; r < a.M; ++r) sum += (double)l.xy[r];
        *a.fin_cos_acc = acc + sum;
    }
}
// What a wave needs for its first requests comes as leading scalar parameters, preloaded into SGPRs (the structures come from memory, which takes
// 0.4 us at the head of a launch).  dims = d | M << 16.
#define SM_IN_PARAMS const float* part, const float* xin, const float* gain, int32_t dims
#define SM_IN_ARGS(in, in0)                                                              \
    SmallIn in = in0;                                                                    \
    in.part = part; in.xin = xin; in.gain = gain; in.d = dims & 0xffff; in.M = dims >> 16;

// ---- attention sublayer
template <int H, int NR> struct SmAttnLds {
    static constexpr int NG = (2 * H + SM_Q / SM_SLICES + 63) / 64,      // groups of 64 rows (fewer dims per slice need as many)
                          RS = NG * 64 + 4, QS = H + 4, VS = SM_Q / SM_SLICES + 4, PS = 64 + 4;
    SmInLds<NR> in;
    union {
        float red[4][NR][RS];                                     // the four K splits' sums of the q, K and V rows
        struct { float p[SM_CHUNKS][NR][PS], o[SM_CHUNKS][NR][VS]; } att;    // a chunk's probabilities, its output
    };
    float ml[SM_CHUNKS][NR][2];                                   // its maximum and sum
    float q[NR][QS], k[NR][QS], v[NR][VS], ao[NR][VS];
};

// heads = n_h | (log2 slices per head) << 8 | (log2 dims per slice) << 16
template <int H, int RM, int RV>
__global__ __launch_bounds__(SM_NT) void sm_attn_kernel(SM_IN_PARAMS, int32_t heads, const float* Wqkv, const DevState* st, const float* rope, const SmallIn in0, const BeginArgs begin, const SmallAttn a) {
    constexpr int NR = 4 * RM + RV, HB = H / 16, PB = HB < 4 ? HB : 4;              // k-blocks of a head, of which PB are requested ahead
    using L = SmAttnLds<H, NR>;
    using Acc = SmAcc<RM, RV>;
    __shared__ L l;
    SM_IN_ARGS(in, in0)
    const int n_h = heads & 255, s_log = (heads >> 8) & 255, hs_log = heads >> 16, qkv_tiles = 3 * n_h * HB;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = blockIdx.x, head = slice >> s_log, sv = slice & ((1 << s_log) - 1), HS = 1 << hs_log;
    const int KB = in.d / 16, M = in.M;
    const int st_pos = st->pos;

    SmFirst first;
    sm_request(in, first, w, lane);

    // weight row of local row lr: the head's H query rows, its H key rows (tile row order), then HS value dims
    auto row_of = [&](int lr, int* tile, int* r) {
        if (lr >= 2 * H + HS) lr = 0;
        if (lr < 2 * H) { *tile = (lr < H ? head * HB : (n_h + head) * HB - HB) + lr / 16; *r = lr & 15; }
        else {
            const int dim = sv * HS + lr - 2 * H, i = dim % (H / 2);
            *tile = (2 * n_h + head) * HB + i / 8; *r = (i & 7) + (dim >= H / 2 ? 8 : 0);
        }
    };
    // task t: rows of group t >> 2, K split t & 3 (k-blocks split, split + 4, ...); the first task's requests go out in two parts (see sm_request)
    f32x4 wq[4][4], kf[PB][4];
    int tile, r;
    row_of((w >> 2) * 64 + lane, &tile, &r);
    auto load_q = [&](int i) { sm_load(wq[i], Wqkv + (min((w & 3) + 4 * i, KB - 1) * qkv_tiles + tile) * 256, r); };
    load_q(0);
    constexpr int np = H / 2;
    const int rp = min(tid, M * np - 1), pos0 = (in.has_begin ? begin.pos : st_pos) + a.pos_off;

    sm_input<SM_NT>(in, begin, first, l.in, tid, w, lane);
    // this wave's 64-key chunk of the cache.  Its K rows are requested once the weights are used, its V^T rows with them where registers allow, else one step later.
    constexpr bool EARLY = RM == 0 && HB <= PB;
    const int PT = a.page_tokens;
    const float* chunk = a.kv;
    const bool have = w < a.nc;
    if (have) chunk += ((size_t)a.page_table[(w * 64) / PT] * n_h + head) * 2 * PT * H + kv_chunk_off<F32>((w * 64) % PT / 64, H);
    const int vd = sv * HS + (lane & (HS - 1));
    auto load_k = [&](int h0) {
#pragma unroll
        for (int hs = 0; hs < PB; ++hs) sm_load(kf[hs], chunk + kv_k_frag_off<F32>(lane >> 4, h0 + hs, H), lane & 15);
    };
    auto load_v = [&](f32x4 (&vf)[4][4]) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) sm_load(vf[ks], chunk + kv_v_frag_off<F32>(vd >> 4, ks, H), vd & 15);
    };
    __syncthreads();
#pragma unroll
    for (int i = 1; i < 4; ++i) load_q(i);
    // rotary factors of this thread's first pair
    const float2 rot = *(const float2*)(rope + ((size_t)(pos0 + rp / np) * np + rp % np) * 2);
    sm_norms(in, l.in, tid);
#pragma unroll
    for (int t0 = 0; t0 < L::NG * 4; t0 += SM_NW) {
        const int t = t0 + w;
        if (t >= L::NG * 4) break;
        Acc acc;
        sm_zero(acc);
        if (t0) {
            row_of((t >> 2) * 64 + lane, &tile, &r);
#pragma unroll
            for (int i = 0; i < 4; ++i) sm_load(wq[i], Wqkv + (min((t & 3) + 4 * i, KB - 1) * qkv_tiles + tile) * 256, r);
        }
        if ((t & 3) < KB) sm_chain(acc, wq, (KB - (t & 3) + 3) / 4, &l.in.x[0][(t & 3) * 16], 64, SM_XS, lane);
        sm_put(acc, &l.red[t & 3][0][(t >> 2) * 64], L::RS, lane);
    }
    f32x4 vf[4][4];
    if (have) {
        load_k(0);
        if constexpr (EARLY) load_v(vf);
    }
    __syncthreads();

    // ---- rotary embedding; q, and the new positions' K and V, into LDS
    auto sum4 = [&](int m, int lr) {
        float v = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s) v += l.red[s][m][lr];
        return v;
    };
    // (the rotation contracted as the compiler contracts gemm_kernel's)
    for (int e = tid; e < M * np; e += SM_NT) {
        const int m = e / np, i = e % np, lr = i / 8 * 16 + (i & 7);
        const float rs = sm_scale(l.in.yy[m], in.inv_d, in.eps);
        float c = rot.x, sn = rot.y;
        if (e != tid) { const size_t o = ((size_t)(pos0 + m) * np + i) * 2; c = rope[o]; sn = rope[o + 1]; }
        {
            const float v0 = sum4(m, lr) * rs, v1 = sum4(m, lr + 8) * rs;
            const float o0 = __builtin_fmaf(v0, c, -(v1 * sn)), o1 = __builtin_fmaf(v1, c, v0 * sn);
            l.q[m][i] = o0; l.q[m][i + np] = o1;
        }
        const float v0 = sum4(m, H + lr) * rs, v1 = sum4(m, H + lr + 8) * rs;
        const float o0 = __builtin_fmaf(v0, c, -(v1 * sn)), o1 = __builtin_fmaf(v1, c, v0 * sn);
        l.k[m][i] = o0; l.k[m][i + np] = o1;
    }
    for (int e = SM_NT - 1 - tid; e < M * HS; e += SM_NT) {
        const int m = e >> hs_log, i = e & (HS - 1);
        l.v[m][i] = sum4(m, 2 * H + i) * sm_scale(l.in.yy[m], in.inv_d, in.eps);
    }
    __syncthreads();

    // ---- V, and in the head's first workgroup K, into the cache: from the last wave on, which has the least else to do
    for (int e = SM_NT - 1 - tid; e < M * (sv == 0 ? HS + H : HS); e += SM_NT) {
        const bool isv = e < M * HS;
        const int m = isv ? e >> hs_log : (e - M * HS) / H, i = isv ? e & (HS - 1) : (e - M * HS) % H, pos = pos0 + m, slot = pos % PT;
        float* base = a.kv + ((size_t)a.page_table[pos / PT] * n_h + head) * 2 * PT * H;
        if (isv) base[kv_v_off<F32>(slot, sv * HS + i, H)] = l.v[m][i];
        else base[kv_k_off<F32>(slot, i, H)] = l.k[m][i];
    }

    // ---- this wave's chunk: scores, probabilities, output
    const int last = pos0 + M - 1, c = w, key0 = c * 64;
    const bool active = have && key0 <= last;
    const bool fresh = active && key0 + 63 >= pos0;                // the chunk holds positions of this pass: their K and V from LDS
    const int n_og = (in.d + 63) / 64, OB = HS / 16;              // 64-row groups of the O-projection, k-blocks of the slice
    if (active) {
        Acc s;
        sm_zero(s);
        const int nk = key0 + lane - pos0;                        // this lane's key among the new positions
#pragma unroll
        for (int h0 = 0; h0 < HB; h0 += PB) {
#pragma unroll
            for (int hs = 0; hs < PB; ++hs) {
                if (fresh && nk >= 0 && nk < M) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) kf[hs][g] = *(const f32x4*)&l.k[nk][(h0 + hs) * 16 + g * 4];
                }
            }
            sm_chain(s, kf, PB, &l.q[0][h0 * 16], 16, L::QS, lane);
            if (h0 + PB < HB) load_k(h0 + PB);
        }
        if constexpr (!EARLY) load_v(vf);
#pragma unroll
        for (int cg = 0; cg < RM; ++cg) {
            const int m = cg * 4 + (lane & 3);
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s.v[cg][i] = (key0 + (lane & ~3) + i <= pos0 + m) ? s.v[cg][i] * a.scale : -INFINITY;
                mx = fmaxf(mx, s.v[cg][i]);
            }
            mx = sm_max<false>(mx);
            f32x4 p;
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = (s.v[cg][i] == -INFINITY) ? 0.f : __expf(s.v[cg][i] - mx);
            *(f32x4*)&l.att.p[c][m][lane & ~3] = p;
            if (lane < 4) l.ml[c][m][0] = mx;
        }
        if constexpr (RV != 0) {
            constexpr int m = 4 * RM;
            const float v = (key0 + lane <= pos0 + m) ? s.s * a.scale : -INFINITY, mx = sm_max<true>(v);
            l.att.p[c][m][lane] = (v == -INFINITY) ? 0.f : __expf(v - mx);
            if (lane == 0) l.ml[c][m][0] = mx;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (fresh) {                                              // the new positions' V, four keys a piece
            const int n0 = key0 - pos0;                           // row of the chunk's first key
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (n0 + 4 * q + 3 >= 0 && n0 + 4 * q < M) {      // (the same in every lane)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int n = n0 + 4 * q + i;
                        const float v = l.v[min(max(n, 0), M - 1)][lane & (HS - 1)];
                        vf[q >> 2][q & 3][i] = n >= 0 && n < M ? v : vf[q >> 2][q & 3][i];
                    }
                }
        }
        // the output, and beside it the chunk's sums of probabilities: lane group g's keys 16 ks + 4 g + j in order, then the groups in pairs
        Acc o;
        sm_zero(o);
        float lv[RM ? RM : 1][4], ls[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            ls[g] = 0.f;
#pragma unroll
            for (int cg = 0; cg < RM; ++cg) lv[cg][g] = 0.f;
        }
        sm_chain(o, vf, 4, &l.att.p[c][0][0], 16, L::PS, lane, [&](const SmX<RM, RV>& b) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if constexpr (RV != 0) ls[g] += b.s[g][j];
#pragma unroll
                    for (int cg = 0; cg < RM; ++cg) lv[cg][g] += b.b[cg][g][j];
                }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if constexpr (RV != 0) sm_hold(ls[g]);
#pragma unroll
                for (int cg = 0; cg < RM; ++cg) sm_hold(lv[cg][g]);
            }
        });
#pragma unroll
        for (int cg = 0; cg < RM; ++cg)
            if (lane < 4) l.ml[c][cg * 4 + lane][1] = (lv[cg][0] + lv[cg][1]) + (lv[cg][2] + lv[cg][3]);
        if constexpr (RV != 0) { if (lane == 0) l.ml[c][4 * RM][1] = (ls[0] + ls[1]) + (ls[2] + ls[3]); }
        sm_put(o, &l.att.o[c][0][0], L::VS, lane, HS);
    }
    f32x4 wo[2][4];                                               // the O-projection's weights, on their way while the chunks are merged
    if (w < n_og) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i < OB) sm_load(wo[i], a.Wo + ((size_t)min(w * 4 + (lane >> 4), in.d / 16 - 1) * (n_h * HB) + slice * OB + i) * 256, lane & 15);
    }
    __syncthreads();

    // ---- merge: a group's four chunks, then (more than 256 positions) the groups
    for (int e = tid; e < M * HS; e += SM_NT) {
        const int m = e >> hs_log, i = e & (HS - 1);
        const int n_groups = last / ATT_GROUP + 1, nc_row = (pos0 + m) / ATT_GROUP + 1, n_c = last / 64 + 1;
        float gm[SM_CHUNKS / ATT_GW], gl[SM_CHUNKS / ATT_GW], ga[SM_CHUNKS / ATT_GW];
        float acc0 = 0.f, Ls = 1.f;
#pragma unroll
        for (int gr = 0; gr < SM_CHUNKS / ATT_GW; ++gr) {
            gm[gr] = -INFINITY; gl[gr] = ga[gr] = 0.f;
            if (gr >= n_groups) continue;
            // (read without a condition, so that the reads are on their way together: a chunk past the context is left out by its maximum)
            float gmax = -INFINITY, mx[ATT_GW], ml[ATT_GW], v[ATT_GW];
#pragma unroll
            for (int ww = 0; ww < ATT_GW; ++ww) {
                const int ch = gr * ATT_GW + ww;
                mx[ww] = l.ml[ch][m][0]; ml[ww] = l.ml[ch][m][1]; v[ww] = l.att.o[ch][m][i];
            }
#pragma unroll
            for (int ww = 0; ww < ATT_GW; ++ww) {
                const bool on = gr * ATT_GW + ww < n_c;
                mx[ww] = on ? mx[ww] : -INFINITY; ml[ww] = on ? ml[ww] : 0.f; v[ww] = on ? v[ww] : 0.f;
                gmax = fmaxf(gmax, mx[ww]);
            }
            float Lg = 0.f, acc = 0.f;
            if (gmax != -INFINITY) {
#pragma unroll
                for (int ww = 0; ww < ATT_GW; ++ww) {
                    const float wgt = __expf(mx[ww] - gmax);
                    Lg += ml[ww] * wgt;
                    acc += v[ww] * wgt;
                }
            }
            gm[gr] = gmax; gl[gr] = Lg; ga[gr] = acc;
        }
        if (n_groups == 1) { acc0 = ga[0]; Ls = gl[0]; }
        else {
            float gmax = -INFINITY, wq_[4] = {0.f, 0.f, 0.f, 0.f}, ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int gr = 0; gr < SM_CHUNKS / ATT_GW; ++gr) if (gr < nc_row) gmax = fmaxf(gmax, gm[gr]);
#pragma unroll
            for (int gr = 0; gr < SM_CHUNKS / ATT_GW; ++gr)
                if (gr < nc_row) { wq_[gr] = __expf(gm[gr] - gmax); ls[gr] += gl[gr] * wq_[gr]; }
            Ls = (ls[0] + ls[2]) + (ls[1] + ls[3]);                // (the butterfly over one group per lane)
#pragma unroll
            for (int gr = 0; gr < SM_CHUNKS / ATT_GW; ++gr) if (gr < nc_row) acc0 += ga[gr] * wq_[gr];
        }
        l.ao[m][i] = acc0 / Ls;
    }
    __syncthreads();

    // ---- the slice of the O-projection
    for (int gr = w; gr < n_og; gr += SM_NW) {
        Acc o;
        sm_zero(o);
        sm_chain(o, wo, OB, &l.ao[0][0], 16, L::VS, lane);
        sm_put_global(o, a.part_out + slice * M * in.d, in.d, gr * 64, in.d - gr * 64, M, lane);
    }
    if (w == SM_NW - 1 && slice == 0) sm_finish(in, l.in, lane);
}

// ---- MLP sublayer
template <int NR> struct SmMlpLds {
    static constexpr int RS = 2 * SM_FFN_TILES * 16 + 4, HS = SM_FFN_TILES * 16 + 4;
    SmInLds<NR> in;
    float red[8][NR][RS];
    float hid[NR][HS];
};
template <int RM, int RV>
__global__ __launch_bounds__(SM_NT) void sm_mlp_kernel(SM_IN_PARAMS, int32_t n_hid, const float* Wg, const float* Wu, const float* Wd, const SmallIn in0, const BeginArgs begin, float* part_out) {
    constexpr int NR = 4 * RM + RV;
    constexpr int GW = 8;                                         // waves of the gate and up rows; the others have the down-projection's weights in flight
    constexpr int PT_ = 3;                                        // a wave's tasks, all requested ahead
    using L = SmMlpLds<NR>;
    using Acc = SmAcc<RM, RV>;
    __shared__ L l;
    SM_IN_ARGS(in, in0)
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = blockIdx.x, KB = in.d / 16, M = in.M;
    const int n_t = (n_hid - slice + SM_SLICES - 1) / SM_SLICES;           // hidden tiles slice, slice + 8, ...
    const int n_rg = (2 * n_t + 3) / 4, n_og = (in.d + 63) / 64;           // 64-row groups
    SmFirst first;
    sm_request(in, first, w, lane);
    // wave w < 8: K slice w (as gemm_kernel's wave w) of the row groups; waves 8 ..: row groups of the down-projection
    const int kb0 = w * KB / 8, nk = (w + 1) * KB / 8 - kb0;               // at most two k-blocks (d <= 256)
    // (indexes past the end are clamped, not skipped: the compiler's wait counts are exact only without conditions)
    auto gate_frag = [&](int gr, int kb) {
        const int ti = min(gr * 4 + (lane >> 4), 2 * n_t - 1), hid = slice + SM_SLICES * (ti < n_t ? ti : ti - n_t);
        return (ti < n_t ? Wg : Wu) + (hid * KB + kb) * 256;
    };
    auto down_frag = [&](int gr, int i) {
        return Wd + ((slice + SM_SLICES * i) * (in.d / 16) + min(gr * 4 + (lane >> 4), in.d / 16 - 1)) * 256;
    };
    f32x4 wt[SM_FFN_TILES][4];                                    // (two k-blocks x three tasks, or a down row group's six k-blocks)
    static_assert(SM_FFN_TILES == 2 * PT_, "one register set for both roles");
    auto load_gate = [&](int t) {
#pragma unroll
        for (int i = 0; i < 2; ++i) sm_load(wt[t * 2 + i], gate_frag(t, min(kb0 + i, KB - 1)), lane & 15);
    };
    if (w < GW) load_gate(0);
    sm_input<SM_NT>(in, begin, first, l.in, tid, w, lane);
    if (w < GW) {
#pragma unroll
        for (int t = 1; t < PT_; ++t) load_gate(t);
    }
    __syncthreads();
    // (the norms' sums in the waves without a product to wait for; their weights, needed last, are requested behind the others')
    if (w >= GW) {
#pragma unroll
        for (int i = 0; i < SM_FFN_TILES; ++i)
            sm_load(wt[i], down_frag(w - GW, min(i, n_t - 1)), lane & 15);
        sm_norms(in, l.in, tid - GW * 64);
    }
    if (w < GW) {
#pragma unroll
        for (int t = 0; t < PT_; ++t) {
            if (t < n_rg) {
                Acc acc;
                sm_zero(acc);
                if (nk > 0) sm_chain(acc, *(const f32x4 (*)[2][4])&wt[t * 2], nk, &l.in.x[0][kb0 * 16], 16, SM_XS, lane);
                sm_put(acc, &l.red[w][0][t * 64], L::RS, lane);
            }
        }
    }
    __syncthreads();
    for (int m = tid >> 7; m < M; m += SM_NT >> 7) {
        const int i = tid & 127;                                  // (at most 96 hidden features)
        if (i >= n_t * 16) break;
        float g = 0.f, u = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) { g += l.red[s][m][i]; u += l.red[s][m][n_t * 16 + i]; }
        const float rs = sm_scale(l.in.yy[m], in.inv_d, in.eps);
        g = g * rs; u = u * rs;
        l.hid[m][i] = g / (1.f + __expf(-g)) * u;
    }
    __syncthreads();
    if (w >= GW && w - GW < n_og) {
        Acc o;
        sm_zero(o);
        sm_chain(o, wt, n_t, &l.hid[0][0], 16, L::HS, lane);
        sm_put_global(o, part_out + slice * M * in.d, in.d, (w - GW) * 64, in.d - (w - GW) * 64, M, lane);
    }
    if (w == 0 && slice == 0) sm_finish(in, l.in, lane);
}

// ---- final norm and LM head: 64 logits per workgroup, candidates per 32 as gemm_kernel<EPI_LM> with two tiles leaves them
template <int NR> struct SmLmLds {
    static constexpr int RS = 64 + 4;
    SmInLds<NR> in;
    float red[SM_LM_NW][NR][RS];
    float lg[NR][RS];
};
template <int RM, int RV>
__global__ __launch_bounds__(SM_LM_NW * 64) void sm_lm_kernel(SM_IN_PARAMS, int32_t V, const float* W, const SmallIn in0, const BeginArgs begin, float* logits, AmaxPart* amax) {
    constexpr int NR = 4 * RM + RV, NT = SM_LM_NW * 64;
    using L = SmLmLds<NR>;
    __shared__ L l;
    SM_IN_ARGS(in, in0)
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = in.d / 16, M = in.M, tiles = V / 16, n0 = blockIdx.x * 64;
    SmFirst first;
    sm_request(in, first, w, lane);
    f32x4 wt[2][4];                                               // k-blocks w, w + 8 (d <= 256)
    const int tile = min((int)blockIdx.x * 4 + (lane >> 4), tiles - 1);
#pragma unroll
    for (int i = 0; i < 2; ++i)
        sm_load(wt[i], W + ((size_t)min(w + 8 * i, KB - 1) * tiles + tile) * 256, lane & 15);
    sm_input<NT>(in, begin, first, l.in, tid, w, lane);
    __syncthreads();
    sm_norms(in, l.in, tid);
    {
        SmAcc<RM, RV> acc;
        sm_zero(acc);
        if (w < KB) sm_chain(acc, wt, (KB - w + 7) / 8, &l.in.x[0][w * 16], 128, SM_XS, lane);
        sm_put(acc, &l.red[w][0][0], L::RS, lane);
    }
    __syncthreads();
    for (int e = tid; e < M * 64; e += NT) {
        const int m = e >> 6, i = e & 63;
        float v = 0.f;
#pragma unroll
        for (int s = 0; s < SM_LM_NW; ++s) v += l.red[s][m][i];
        v = v * sm_scale(l.in.yy[m], in.inv_d, in.eps);
        const bool ok = n0 + i < V;
        if (ok) logits[(size_t)m * V + n0 + i] = v;
        l.lg[m][i] = ok ? v : -INFINITY;
    }
    __syncthreads();
    if (w == SM_LM_NW - 1 && blockIdx.x == 0) sm_finish(in, l.in, lane);
    if (tid < 2 * M) {
        const int m = tid >> 1, half = tid & 1;
        if (n0 + half * 32 >= V) return;
        AmaxPart best{-INFINITY, 0x7fffffff, 0.f, 0.f};
        for (int i = 0; i < 32; ++i) {
            const float v = l.lg[m][half * 32 + i];
            if (v > best.v) { best.v = v; best.i = n0 + half * 32 + i; }
        }
        float se = 0.f;
        if (best.v != -INFINITY)
            for (int i = 0; i < 32; ++i) se += __expf(l.lg[m][half * 32 + i] - best.v);
        best.s = se;
        amax[(size_t)(blockIdx.x * 2 + half) * 16 + m] = best;
    }
}
