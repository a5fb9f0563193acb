// Prompt processing as large-M contractions: the pass that fills the KV cache and measures the prompt's
// average cosine similarity per sublayer (Section 3.2, the definition of C_l) before the draft / verify loop starts.
//
// The prompt is processed in blocks of up to 2048 rows, layer by layer, so every weight is read once per
// block instead of once per 16 rows.  Activations of a block are kept as 16-row chunks, each chunk in the same
// tiled layout the decode kernels use with a row stride of 16 ([K/KE][16][KE], hi and lo planes for bf16):
// one (chunk, k-block) fragment is one contiguous KiB that a wave loads with one instruction, and the prompt attention kernels
// use the decode kernel's fragments.
//
// pf_ring_kernel: a tile of weight tiles x chunks per workgroup (3 x 2 to 24 x 8 and 16 x 16), both operands brought
// into an LDS ring by direct-to-LDS loads; see its own comment.  The kernel and tile of a launch are the ones with the
// smallest estimated time.
// pf_gemm_kernel (at some lengths between whole rounds of the ring's larger tiles): a workgroup of NW waves owns NW*NA weight tiles (16 output features each) x NC chunks of
// rows and, with a K split, one slice of K.  Per k-block the waves stage the NC chunks' activation fragments
// in LDS (double buffered, one barrier per k-block); each wave streams its own NA weight fragments from
// global memory and feeds NA*NC accumulators.  Workgroups that share weights (same features, other rows)
// and those that share activations run at the same time on the same XCD, so both are served by its L2.
//   PF_QKV  RMSNorm scale, rotary embedding, q -> chunked q buffer, k/v -> paged cache
//   PF_GU   RMSNorm scale, silu(gate) * up -> chunked activation
//   PF_RAW  the slice's partial sums -> raw[k slice][row][feature]; pf_resid_kernel then adds the slices to
//           the residual stream in slice order, writes the normed copy for the next sublayer and finishes the
//           cosine tap of every row.
#pragma once
#include <type_traits>
#include "asd_gemm.h"
#include "asd_misc.h"

// A block holds up to 512, 1024 or 2048 rows, whatever the engine's workspace has room for (PF_MIN_ROWS always fits);
// the raw partial sums of a block take slices x rows <= PF_RAW_ROWS rows of d_model.
#define PF_MIN_ROWS 512
#define PF_MAX_ROWS 2048
#define PF_MAX_KSPLIT 8
#define PF_RAW_ROWS (PF_MAX_KSPLIT * PF_MIN_ROWS)

enum { PF_QKV = 0, PF_RAW = 1, PF_GU = 2 };

struct PfArgs {
    const u32x4 *W, *W2, *X;
    int64_t x_plane, x_chunk;        // fragment strides of X: between planes, between 16-row chunks
    int32_t n_tiles, KB;
    int64_t w_tile_stride, w_kb_stride;
    int32_t n_fb, n_rb, ksplit;      // feature blocks (NW*NA tiles each), row blocks (NC chunks each), K slices
    int32_t rows;                    // valid rows of this prompt block
    int32_t raw_rows;                // row stride between the K slices of raw
    const float* rscale;             // [rows] RMSNorm scale of each row (PF_QKV, PF_GU)
    float* raw;                      // PF_RAW: [ksplit][raw_rows][16 * n_tiles]
    // PF_QKV
    int32_t pos0;                    // cache position of row 0
    const float* rope;
    void* q; int64_t q_plane, q_chunk;         // element strides
    void* kv; const int32_t* page_table;
    int32_t n_h, n_kv, h, page_tokens;
    // PF_GU
    void* hmid; int64_t hmid_plane, hmid_chunk;
};

// four consecutive single-plane elements (cache rows)
template <class T> __device__ __forceinline__ void store_elem4(typename T::elem* p, const float (&v)[4]) {
    if constexpr (sizeof(typename T::elem) == 2) {
        const uint32_t a = T::from_f32(v[0]), b = T::from_f32(v[1]), c = T::from_f32(v[2]), d = T::from_f32(v[3]);
        *(uint2*)p = uint2{a | (b << 16), c | (d << 16)};
    } else {
        *(float4*)p = float4{v[0], v[1], v[2], v[3]};
    }
}

// the value of the lane 32 away
__device__ __forceinline__ float other_half(float x, int lane) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);     // {lower, lower}, {upper, upper}
    return __uint_as_float(lane < 32 ? r[1] : r[0]);
}
// v[j] of lane i of a quad <-> v[i] of lane j (q = the lane's place in its quad)
__device__ __forceinline__ void quad_transpose(float (&v)[4], const int q) {
    auto swapped = [](float x, auto ctrl) { return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    using X1 = std::integral_constant<int, 0xb1>;          // lanes 1, 0, 3, 2
    using X2 = std::integral_constant<int, 0x4e>;          // lanes 2, 3, 0, 1
#pragma unroll
    for (int p = 0; p < 4; p += 2) {                       // 2 x 2 blocks: v[p + 1] of the even lane <-> v[p] of the odd one
        const float got = swapped((q & 1) ? v[p] : v[p + 1], X1{});
        if (q & 1) v[p] = got; else v[p + 1] = got;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {                          // v[p + 2] of the lower pair <-> v[p] of the upper one
        const float got = swapped((q & 2) ? v[p] : v[p + 2], X2{});
        if (q & 2) v[p] = got; else v[p + 2] = got;
    }
}
// Epilogues of the prompt GEMMs, straight from the accumulators: lane 16g + m holds features 4g..4g+3 of each tile for
// row m of each chunk.  PF_GU: acc[0 .. NA-1] gate, acc[NA .. 2NA-1] up.  RD: PF_QKV's (tile, chunk) pairs whose rotary factors are held.
template <class T, int EPI, int RD, int NA, int NAT, int NC>
__device__ __forceinline__ void pf_epilogue(const PfArgs& a, const f32x4 (&acc)[NAT][NC], const int (&tile)[NA], const bool (&tval)[NA],
                                            const int chunk0, const int ks, const int lane) {
    using E = typename T::elem;
    const int g = lane >> 4, m = lane & 15;
    int row[NC];
    bool rv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) { row[c] = (chunk0 + c) * 16 + m; rv[c] = row[c] < a.rows; }

    if constexpr (EPI == PF_RAW) {
        const int N = a.n_tiles * 16;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (!rv[c]) continue;
            float* dst = a.raw + ((size_t)ks * a.raw_rows + row[c]) * N + 4 * g;
#pragma unroll
            for (int s = 0; s < NA; ++s)
                if (tval[s]) *(f32x4*)(dst + tile[s] * 16) = acc[s][c];
        }
    }

    if constexpr (EPI == PF_GU) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (!rv[c]) continue;
            const float rs = a.rscale[row[c]];
#pragma unroll
            for (int s = 0; s < NA; ++s) {
                if (!tval[s]) continue;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float gt = acc[s][c][j] * rs, up = acc[NA + s][c][j] * rs;
                    v[j] = gt / (1.f + __expf(-gt)) * up;
                }
                store_act4<T>(a.hmid, a.hmid_plane, (int64_t)(chunk0 + c) * a.hmid_chunk, tile[s] * 16 + 4 * g, m, v);
            }
        }
    }

    if constexpr (EPI == PF_QKV) {
        // tile j of a head: rows 0..7 = head dims 8j..8j+7, rows 8..15 = the same dims + h/2 (rotary partners):
        // lane groups 0,1 hold the first halves, groups 2,3 their partners, 32 lanes away.
        // A workgroup of the ring kernel has its compute unit to itself, so what this waits for nobody hides: the rotary factors are requested RD - 1 (tile, chunk)
        // pairs ahead (read between the stores they cost a memory round trip per pair), the rows' pages and scales once.
        // 7B, 2048 rows, the ring kernel's launch: 350 -> 332 us, with V^T's 2-byte stores, one per row and dim, made 8-byte ones below.  The four-wave kernel shares its
        // unit and hides these waits: with eight chunks, which fill its registers, it asks for a pair as it needs it (three ahead spilled 57 registers).
        const int hpt = a.h / 16, hh = a.h / 2, PT = a.page_tokens;
        float rs[NC];
        int page[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            rs[c] = rv[c] ? a.rscale[row[c]] : 0.f;
            page[c] = a.page_table[(a.pos0 + min(row[c], a.rows - 1)) / PT];      // (a quad's lanes beyond the last row store for those before it)
        }
        f32x4 rope[RD][2];                                // (cos, sin) of four dims
        auto rotary = [&](const int i) {
            const int s = i / NC, c = i % NC, head = tile[s] / hpt;
            if (!tval[s] || head >= a.n_h + a.n_kv) return;
            const float* rp = a.rope + ((size_t)(a.pos0 + min(row[c], a.rows - 1)) * hh + tile[s] % hpt * 8 + 4 * (g & 1)) * 2;
            rope[i % RD][0] = *(const f32x4*)rp;
            rope[i % RD][1] = *(const f32x4*)(rp + 4);
        };
#pragma unroll
        for (int i = 0; i < RD - 1 && i < NA * NC; ++i) rotary(i);
#pragma unroll
        for (int s = 0; s < NA; ++s) {
            const int head = tile[s] / hpt, jt = tile[s] % hpt;
            const int i0 = jt * 8 + 4 * (g & 1), dim = i0 + (g >= 2 ? hh : 0);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (s * NC + c + RD - 1 < NA * NC) rotary(s * NC + c + RD - 1);
                if (!tval[s]) continue;               // wave-uniform
                const int slot = (a.pos0 + row[c]) % PT;
                E* kvp = (E*)a.kv + (size_t)page[c] * a.n_kv * 2 * PT * a.h;
                float own[4], v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) own[j] = acc[s][c][j] * rs[c];
                if (head < a.n_h + a.n_kv) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float oth = other_half(own[j], lane), cs = rope[(s * NC + c) % RD][j >> 1][2 * (j & 1)], sn = rope[(s * NC + c) % RD][j >> 1][2 * (j & 1) + 1];
                        v[j] = g < 2 ? own[j] * cs - oth * sn : own[j] * cs + oth * sn;
                    }
                    if (!rv[c]) continue;
                    if (head < a.n_h) store_act4<T>(a.q, a.q_plane, (int64_t)(chunk0 + c) * a.q_chunk, head * a.h + dim, m, v);
                    else store_elem4<T>(kvp + (size_t)(head - a.n_h) * 2 * PT * a.h + kv_k_off<T>(slot, dim, a.h), v);      // dim is a multiple of 4: the four values stay inside one lane's KE elements
                } else {
                    // V^T: the keys of a dim follow each other, so four rows' values of one dim are one store: a 4 x 4 transpose over the
                    // four lanes of a quad (rows m & ~3 .. m | 3; a block starts at a multiple of 16, so they are neighbours in a fragment)
                    E* base = kvp + (size_t)(head - a.n_h - a.n_kv) * 2 * PT * a.h;
                    quad_transpose(own, m & 3);
                    int rows = a.rows;                        // (compared anew for every tile: the masks of all chunks held side by side spilled 50 scalar registers)
                    asm("" : "+s"(rows));
                    if ((row[c] | 3) < rows) {
                        store_elem4<T>(base + kv_v_off<T>(slot & ~3, dim + (m & 3), a.h), own);
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if ((row[c] & ~3) + k < rows) base[kv_v_off<T>((slot & ~3) + k, dim + (m & 3), a.h)] = T::from_f32(own[k]);
                    }
                }
            }
        }
    }
}

template <class T, int EPI, int NA, int NC, int NW, int PD>
__global__ __launch_bounds__(NW * 64, PD >= 2 ? 2 : 1) void pf_gemm_kernel(const PfArgs a) {
    constexpr int NP = T::NP;
    constexpr int NAT = (EPI == PF_GU) ? 2 * NA : NA;
    constexpr int XF = NC * NP;                       // activation fragments per k-block of this row block
    constexpr int XW = (XF + NW - 1) / NW;            // ... staged by each wave
    __shared__ u32x4 xs[2][XF][64];

    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup -> (feature block, row block, K slice): consecutive workgroup ids go to the 8 XCDs in turn, so the
    // XCD is the low 3 bits; on one XCD the row blocks and K slices of a feature block follow each other.
    const int L = blockIdx.x, inner = a.n_rb * a.ksplit;
    const int fb = ((L >> 3) / inner) * 8 + (L & 7), in = (L >> 3) % inner, rb = in % a.n_rb, ks = in / a.n_rb;
    if (fb >= a.n_fb) return;
    const int chunk0 = rb * NC;

    int tile[NA];
    bool tval[NA];
#pragma unroll
    for (int s = 0; s < NA; ++s) { tile[s] = (fb * NW + w) * NA + s; tval[s] = tile[s] < a.n_tiles; }
    const u32x4* A[NAT];
#pragma unroll
    for (int s = 0; s < NAT; ++s) {
        const u32x4* base = (EPI == PF_GU && s >= NA) ? a.W2 : a.W;
        A[s] = base + (size_t)(tval[s % NA] ? tile[s % NA] : 0) * a.w_tile_stride * ASD_WAVE + lane;
    }
    const int kb0 = (int)((long)ks * a.KB / a.ksplit), kb1 = (int)((long)(ks + 1) * a.KB / a.ksplit);
    const u32x4* Xp[XW];
#pragma unroll
    for (int i = 0; i < XW; ++i) {
        const int f = w + NW * i, c = (f < XF ? f : 0) / NP, pl = (f < XF ? f : 0) % NP;
        Xp[i] = a.X + (size_t)pl * a.x_plane + (size_t)(chunk0 + c) * a.x_chunk + lane;
    }

    f32x4 acc[NAT][NC];
#pragma unroll
    for (int s = 0; s < NAT; ++s)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[s][c] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Weight and activation fragments are requested PD k-blocks ahead of their use (register ring).  Every trip of
    // the main loop issues the same loads whatever the k-block (past the end of the range the last k-block is asked
    // for again and never used): the wait counts the compiler derives are exact only when no path skips a load, and
    // one conditional request is enough to turn every wait into a full drain, which undoes the prefetch.
    u32x4 an[PD][NAT], xg[PD][XW];
    auto issue = [&](int slot, int kb) {
#pragma unroll
        for (int i = 0; i < XW; ++i)
            if (XF % NW == 0 || w + NW * i < XF) xg[slot][i] = Xp[i][(size_t)kb * ASD_WAVE];
#pragma unroll
        for (int s = 0; s < NAT; ++s) an[slot][s] = A[s][(size_t)kb * a.w_kb_stride * ASD_WAVE];
    };
    // One k-block from ring slot p.  The slot's next request goes out only after its products (straight into the
    // same registers): asked for any earlier, the old values would have to be copied aside and the new ones copied
    // back at the loop's end, which the compiler can only do after waiting for them, every trip.
    auto k_block = [&](const int p, const int kb, auto prefetch) {
        const int buf = (kb - kb0) & 1;
#pragma unroll
        for (int i = 0; i < XW; ++i)
            if (XF % NW == 0 || w + NW * i < XF) xs[buf][w + NW * i][lane] = xg[p][i];
        __syncthreads();
        // all LDS reads of the k-block are requested before its first MFMA: one LDS latency per k-block, not one per pair
        u32x4 b[NC][NP];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl) b[c][pl] = xs[buf][c * NP + pl][lane];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
#pragma unroll
                for (int s = 0; s < NAT; ++s) mma16<T>(acc[s][c], an[p][s], b[c][pl]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(prefetch)::value) issue(p, kb + PD < kb1 ? kb + PD : kb1 - 1);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p) issue(p, kb0 + p < kb1 ? kb0 + p : kb1 - 1);
    const int n_full = (kb1 - kb0) / PD * PD;
    for (int kbb = kb0; kbb < kb0 + n_full; kbb += PD) {
#pragma unroll
        for (int p = 0; p < PD; ++p) k_block(p, kbb + p, std::true_type{});
    }
#pragma unroll
    for (int p = 0; p + 1 < PD; ++p)                    // the last, partial round: nothing further to request
        if (kb0 + n_full + p < kb1) k_block(p, kb0 + n_full + p, std::false_type{});

    pf_epilogue<T, EPI, NC == 8 ? 1 : 4, NA, NAT, NC>(a, acc, tile, tval, chunk0, ks, lane);
}

// ---- the LDS ring kernel of the prompt GEMMs
// Both operands are read once per workgroup into LDS (no fragment passes through a register on its way there) and every wave
// takes its fragments from there: a wave's tile (NT weight tiles x NC chunks, both planes) reads NT + 2 NC fragments for
// 2 NT NC products.  FW x RW waves share a k-block, FW over the weight tiles, RW over the chunks.  An output is one wave's sum
// over its K slice in k-block order, hi plane before lo plane, as in pf_gemm_kernel: the tile shape does not enter a result.
//
// What bounds it goes by the length of the block.  Long blocks: the clock the card keeps under the products (a loop of them on random operands in registers,
// nothing else, runs at 2.06 GHz and 2.1 PFLOP/s) and the cycles in which none issues; the tile is as large as LDS and registers allow.
// Short ones: what a compute unit takes in.  With all units busy a fragment from HBM costs it 1/23 us (non-temporal 1/25) and one from L2 about 1/110 us
// (one weight fragment and 0, 1, 2, 4 shared ones: 44, 48, 58, 80 ns): few chunks per tile while the weights weigh more, row blocks that share them otherwise.  In between: how
// evenly the tiles fill the 256 units, hence the number of shapes.
//
// Requests.  A direct-to-LDS load holds its wave up for 55 cycles, for 78 while one wave on each SIMD asks and 114 while two do, and the product waves of a
// workgroup, in step behind their barrier, all did, without a product meanwhile (7B QKV at 144 rows 60 us).  So NL waves of their own ask
// for the fragments and do nothing else (47 us), and the product waves hold only accumulators and fragments.  The largest tile leaves them no
// registers: there, and in fp32, the product waves request (NL = 0), spread between the products.
//
// A stage is one k-block; S stages form a ring.  Per stage one barrier, before which the requesting waves wait until their share of the stage to come has arrived and
// the product waves until their reads of the slot that is refilled next have.  PF: the next stage's fragments are read into a second
// set of registers during this stage's products (all tiles but the three largest, whose accumulators leave no room).
// Products run with one weight fragment held over NC chunks in alternating direction (2 % less time than the other
// order).
template <int NP, int NT, int NC, int FW, int RW, int NL> struct PfRing {
    static constexpr int W = FW * RW, WAVES = W + NL;               // product waves, waves
    static constexpr int ASK = NL ? NL : W;                         // waves that request
    static constexpr int FT = FW * NT, RC = RW * NC;                // weight tiles and chunks per workgroup
    static constexpr int NF = FT + NP * RC;                         // fragments per k-block
    // requests per wave and stage, the same number from every wave (the wait counts depend on it): where they do not come
    // out even, some waves' last request reads nothing (into a spare KiB)
    static constexpr int L = (NF + ASK - 1) / ASK, SPARE = NF % ASK ? 1 : 0;
    static constexpr int FIT = (160 - SPARE) / NF;                  // stages the LDS holds; an even number of them, except three where four do not fit
    static constexpr int S = FIT == 3 ? 3 : FIT > 16 ? 16 : FIT / 2 * 2;
    static_assert(S >= 3 && (S - 1) * L < 64, "a ring, and what the request counter can hold");
};
// One wave's requests of a stage: fragments j, j + ASK, ... of the stage's FT weight and NP RC chunk fragments.  A tile
// beyond the last re-reads the last one, a chunk beyond the block's last re-reads that one (the buffers end with it where
// the block is full and RC does not divide it): their products are never looked at.
// A wave keeps one address per request and nothing else of its own: places in LDS follow from j, weights share one step and chunks another, and
// only the last request can be one that reads nothing.  (With step, place and length kept per request and the first stages unrolled the compiler spilled up
// to 293 scalar registers, and the first request of a workgroup waited for 160 to 420 instructions.)
template <class T, class SH, int EPI, int NT> struct PfRequests {
    static constexpr int NP = T::NP, NA = EPI == PF_GU ? NT / 2 : NT, L = SH::L, NF = SH::NF, FT = SH::FT;
    const char* src[L];
    int64_t w_step;                                                 // to a weight tile's next k-block (a chunk's: 1 KiB)
    int x_step, j;
    int last;                                                       // the last request's fragment of slot 0
    uint32_t last_bytes;
    int left;                                                       // stages still to ask for; past the last one it is asked for again
    __device__ __forceinline__ PfRequests(const PfArgs& a, int fb, int rb, int kb0, int n, int j) : w_step(a.w_kb_stride * 1024), x_step(1024), j(j), left(n) {
        const bool real = j + SH::ASK * (L - 1) < NF;
        last = real ? j + SH::ASK * (L - 1) : SH::S * NF;
        last_bytes = real ? 0xffffffffu : 0u;
        const int wt = (int)a.w_tile_stride, xc = (int)a.x_chunk;       // fragments: a tensor of 2^31 of them would be 2 TiB
        const char* const X = (const char*)a.X + (int64_t)kb0 * 1024;
        const int64_t w0 = kb0 * a.w_kb_stride;
        const int last_chunk = (a.rows + 15) / 16 - 1;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const int f = min(j + SH::ASK * i, NF - 1), s = f % NT, x = f - FT;
            if (is_weight(i, f)) {
                const bool up = EPI == PF_GU && s >= NA;
                const int t = min((fb * (FT / NT) + f / NT) * NA + (up ? s - NA : s), a.n_tiles - 1);
                src[i] = (const char*)(up ? a.W2 : a.W) + ((int64_t)t * wt + w0) * 1024;
            } else {
                src[i] = X + ((x % NP ? a.x_plane : 0) + (int64_t)min(rb * SH::RC + x / NP, last_chunk) * xc) * 16;
            }
        }
    }
    // fragment f, the wave's i-th request (which of the two it is is known when compiling for all i but one)
    static __device__ __forceinline__ bool is_weight(const int i, const int f) { return SH::ASK * (i + 1) <= FT || (SH::ASK * i < FT && f < FT); }
    // Called once per trip of a loop whose slots are known when compiling: keeps the compiler from holding every slot's places in registers.
    __device__ __forceinline__ void next_trip() { asm volatile("" : "+s"(j), "+s"(last)); }
    // ONCE: no other workgroup reads the weights (where a request is a weight's for every wave)
    template <bool ONCE> __device__ __forceinline__ void issue(u32x4* sm, const int slot, const int lane) {
        u32x4* const to = sm + (slot * NF + j) * 64;
        --left;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const bool odd = SH::SPARE && i == L - 1;
            const uint32_t bytes = odd ? last_bytes : 0xffffffffu;
            u32x4* const at = odd ? &sm[(last + (slot * NF & (int)last_bytes)) * 64] : to + SH::ASK * i * 64;
            if (ONCE && SH::ASK * (i + 1) <= FT) frag_to_lds<true>(src[i], bytes, at, lane);
            else frag_to_lds(src[i], bytes, at, lane);
            src[i] += left <= 0 ? 0 : is_weight(i, j + SH::ASK * i) ? w_step : x_step;
        }
    }
};
template <class T, int EPI, int NT, int NC, int FW, int RW, int NL, bool PF>
__global__ __launch_bounds__((FW * RW + NL) * 64, (FW * RW + NL + 3) / 4) void pf_ring_kernel(const PfArgs a) {
    constexpr int NP = T::NP;
    using SH = PfRing<NP, NT, NC, FW, RW, NL>;
    constexpr int W = SH::W, FT = SH::FT, RC = SH::RC, NF = SH::NF, L = SH::L, S = SH::S;
    constexpr int NA = EPI == PF_GU ? NT / 2 : NT;                  // output tiles per wave
    constexpr int AHEAD = PF ? S : S - 1;                           // stages asked for before the first product
    static_assert(!PF || S % 2 == 0, "two register sets: stages in pairs");
    __shared__ u32x4 sm[(S * NF + SH::SPARE) * 64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup -> (feature block, row block, K slice), XCD-first as in pf_gemm_kernel (a mapping that balances the bytes of
    // weights and activations an XCD's running workgroups share, 8 row blocks x 4 feature blocks instead of 16 x 2, measured the same)
    const int Lb = blockIdx.x, inner = a.n_rb * a.ksplit;
    const int fb = ((Lb >> 3) / inner) * 8 + (Lb & 7), in = (Lb >> 3) % inner, rb = in % a.n_rb, ks = in / a.n_rb;
    if (fb >= a.n_fb) return;
    const int kb0 = ks * a.KB / a.ksplit, n = (ks + 1) * a.KB / a.ksplit - kb0;      // (at most eight slices: far inside 32 bits)

    if constexpr (NL > 0) {
        if (w >= W) {                                               // a requesting wave
            PfRequests<T, SH, EPI, NT> q(a, fb, rb, kb0, n, w - W);
            auto feed = [&](auto once) {
                constexpr bool ONCE = decltype(once)::value;
#pragma unroll 1
                for (int b = 0; b < AHEAD; ++b) q.template issue<ONCE>(sm, b, lane);
                if constexpr (PF) {
                    wait_vm<(S - 1) * L, false>();
                    __builtin_amdgcn_s_barrier();
                }
                int slot = AHEAD % S;
                for (int i = 0; i < n; ++i) {
                    wait_vm<(S - 2) * L, false>();
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    q.template issue<ONCE>(sm, slot, lane);
                    slot = slot + 1 == S ? 0 : slot + 1;
                }
            };
            // weights that no other row block reads: non-temporal (45 rows: down 70B 92 -> 83 us, QKV 7B 27 -> 26 us); with several row blocks they should stay in L2
            if (a.n_rb == 1) feed(std::true_type{}); else feed(std::false_type{});
            wait_vm<0, true>();                                     // no request may outlive the workgroup's LDS
            return;
        }
    }
    const int fw = w % FW, rw = w / FW;
    f32x4 acc[NT][NC];
#pragma unroll
    for (int s = 0; s < NT; ++s)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[s][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 fa[PF ? 2 : 1][NT], fx[PF ? 2 : 1][NP * NC];
    auto read = [&](const int slot, const int r) {
        const u32x4* p = &sm[slot * NF * 64 + lane];
#pragma unroll
        for (int b = 0; b < NP * NC; ++b) fx[r][b] = p[(FT + rw * NP * NC + b) * 64];
#pragma unroll
        for (int s = 0; s < NT; ++s) fa[r][s] = p[(fw * NT + s) * 64];
    };
    auto products = [&](const int r) {
#pragma unroll
        for (int s = 0; s < NT; ++s)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
#pragma unroll
                for (int cc = 0; cc < NC; ++cc) {
                    const int c = ((NP * s + pl) & 1) ? NC - 1 - cc : cc;
                    mma16<T>(acc[s][c], fa[r][s], fx[r][NP * c + pl]);
                }
    };
    constexpr int NM = NP * NT * NC * (sizeof(typename T::elem) == 4 ? 4 : 1), ND = NT + NP * NC, TAIL = NM > 16 ? 6 : 0;     // products and fragment reads per stage
    // issue: the requests of a later stage, where this wave makes them
    auto stage = [&](const int slot, const int r, auto issue) {
        wait_vm<NL ? 63 : (S - 2) * L, true>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PF) {
            if constexpr (NL == 0) issue(slot);                     // its fragments are in registers since the last stage
            read((slot + 1) % S, r ^ 1);
            products(r);
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                if (j < NM - TAIL && (j * ND) / (NM - TAIL) != ((j - 1) * ND + NM - TAIL) / (NM - TAIL) - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (NL == 0 && (j * L) / NM != ((j - 1) * L + NM) / NM - 1) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            }
        } else {
            read(slot, 0);
            if constexpr (NL == 0) {
                __builtin_amdgcn_sched_barrier(0);
                issue((slot + S - 1) % S);
            }
            products(0);
            if constexpr (NL == 0) {
#pragma unroll
                for (int j = 0; j < NM; ++j) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    if ((j * L) / NM != ((j - 1) * L + NM) / NM - 1) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    auto stages = [&](auto issue, auto next_trip) {
        if constexpr (PF) {
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            read(0, 0);
        }
        int i = 0;
        for (; i + S <= n; i += S) {
            next_trip();
#pragma unroll
            for (int u = 0; u < S; ++u) stage(u, PF ? u & 1 : 0, issue);
        }
#pragma unroll
        for (int u = 0; u + 1 < S; ++u)
            if (i + u < n) stage(u, PF ? u & 1 : 0, issue);
    };
    if constexpr (NL > 0) {
        stages([](int) {}, [] {});
    } else {
        PfRequests<T, SH, EPI, NT> q(a, fb, rb, kb0, n, w);
#pragma unroll
        for (int b = 0; b < AHEAD; ++b) q.template issue<false>(sm, b, lane);
        if constexpr (PF) wait_vm<(S - 1) * L, false>();
        stages([&](const int slot) { q.template issue<false>(sm, slot, lane); }, [&] { q.next_trip(); });
        wait_vm<0, true>();                                         // no request may outlive the workgroup's LDS
    }

    int tile[NA];
    bool tval[NA];
#pragma unroll
    for (int s = 0; s < NA; ++s) { tile[s] = (fb * FW + fw) * NA + s; tval[s] = tile[s] < a.n_tiles; }
    pf_epilogue<T, EPI, 4, NA, NT, NC>(a, acc, tile, tval, rb * RC + rw * NC, ks, lane);
}

// ---- fp32, short K ranges: a wave on its own
// A wave takes one weight tile (gate/up: a pair) and one chunk, and asks for the fragments of PF_DIRECT_KB k-blocks at once, straight into registers: no ring to fill, no
// barrier.  A few k-blocks in fp32 last as long as one wave's products (32 cycles each, two chunks in a wave of the smallest ring tile): here a wave has half
// as many, and there are waves for all compute units.  Every wave reads its own fragments, which L2 serves.  256 features, 17 to 200 rows (to 100 for O and
// down), ring / this, us between events: QKV 8.3 / 7.2, gate/up 10.3 / 8.5, O 6.3 / 6.2, down 6.8 / 6.3; 512 features: 10.4 / 9.3, 14.2 / 12.3, 6.5 / 6.2, 8.3 / 7.9.  Two chunks per wave: 9.2 and 10.5
// us for the first two.  An output is one wave's sum over its K slice in k-block order, as everywhere.
#define PF_DIRECT_KB 16
template <class T, int EPI>
__global__ __launch_bounds__(256) void pf_direct_kernel(const PfArgs a) {
    static_assert(T::NP == 1, "one plane");
    constexpr int NAT = EPI == PF_GU ? 2 : 1, B = PF_DIRECT_KB;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int Lb = blockIdx.x, inner = a.n_rb * a.ksplit;          // as in pf_gemm_kernel
    const int fb = ((Lb >> 3) / inner) * 8 + (Lb & 7), in = (Lb >> 3) % inner, rb = in % a.n_rb, ks = in / a.n_rb;
    const int tile[1] = {fb * 4 + w};
    if (tile[0] >= a.n_tiles) return;
    const int kb0 = ks * a.KB / a.ksplit, n = (ks + 1) * a.KB / a.ksplit - kb0;
    const u32x4* A[NAT];
#pragma unroll
    for (int s = 0; s < NAT; ++s) A[s] = (s ? a.W2 : a.W) + (tile[0] * a.w_tile_stride + kb0 * a.w_kb_stride) * ASD_WAVE;
    const u32x4* const X = a.X + (size_t)rb * a.x_chunk + (size_t)kb0 * ASD_WAVE;
    f32x4 acc[NAT][1];
#pragma unroll
    for (int s = 0; s < NAT; ++s) acc[s][0] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int b = 0; b < n; b += B) {
        u32x4 wf[B][NAT], xf[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {                              // (past the end the last k-block again: the wait counts are exact only without conditions)
            const int kb = min(b + i, n - 1);
            xf[i] = X[(size_t)kb * ASD_WAVE + lane];
#pragma unroll
            for (int s = 0; s < NAT; ++s) wf[i][s] = A[s][kb * a.w_kb_stride * ASD_WAVE + lane];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < B; ++i)
            if (b + i < n) {
#pragma unroll
                for (int s = 0; s < NAT; ++s) mma16<T>(acc[s][0], wf[i][s], xf[i]);
            }
    }
    const bool tval[1] = {true};
    pf_epilogue<T, EPI, 1, 1, NAT, 1>(a, acc, tile, tval, rb, ks, lane);
}

// The bf16 shapes, X(number, weight tiles per wave, chunks per wave, waves over the tiles, waves over the chunks, requesting waves,
// second register set): for QKV and the raw sums, and for gate/up, whose tiles come in pairs.  Of some 40 shapes measured on the 7B, 13B and 70B matrices at 20 to
// 2048 rows, the sixteen of each list that left the least time on the table (under 1 % over all lengths).  Over 1500 configurations of other widths the estimate takes each of them somewhere.
#define PF_RING_SHAPES(X)                                                                                                \
    X(0, 4, 4, 4, 2, 4, false) X(1, 6, 4, 2, 2, 4, true) X(2, 8, 4, 2, 4, 0, false) X(3, 1, 2, 4, 1, 4, true)            \
    X(4, 1, 3, 3, 1, 3, true) X(5, 1, 4, 4, 1, 4, true) X(6, 2, 3, 4, 1, 4, true) X(7, 2, 4, 4, 1, 4, true)              \
    X(8, 2, 4, 3, 1, 3, true) X(9, 4, 3, 2, 2, 4, true) X(10, 4, 4, 2, 2, 4, true) X(11, 4, 5, 2, 2, 4, true)            \
    X(12, 5, 4, 2, 2, 4, true) X(13, 5, 5, 2, 2, 4, true) X(14, 6, 3, 2, 2, 4, true) X(15, 8, 3, 2, 2, 4, true)
#define PF_RING_PAIR_SHAPES(X)                                                                                           \
    X(0, 4, 4, 4, 2, 4, false) X(1, 6, 4, 4, 2, 4, false) X(2, 8, 4, 2, 4, 0, false) X(3, 2, 5, 4, 1, 4, true)           \
    X(4, 2, 3, 3, 1, 3, true) X(5, 2, 4, 3, 1, 3, true) X(6, 2, 2, 4, 1, 4, true) X(7, 2, 4, 4, 1, 4, true)              \
    X(8, 4, 4, 4, 1, 4, true) X(9, 4, 3, 2, 2, 4, true) X(10, 4, 4, 2, 2, 4, true) X(11, 4, 5, 2, 2, 4, true)            \
    X(12, 6, 3, 2, 2, 4, true) X(13, 6, 4, 2, 2, 4, true) X(14, 4, 5, 4, 1, 4, true) X(15, 8, 3, 2, 2, 4, true)
// In fp32 a product takes eight times as long (128 cycles of a SIMD per fragment pair): the requests hide behind the products, and
// a prompt pass of a small model, a few k-blocks per launch, pays for every wave more (256 k values, 4 layers, 30 rows: 168 us like this, 203 with
// requesting waves).  N weight tiles per wave: one, two for gate/up.  D(number): pf_direct_kernel.  The estimate takes 3 and 10 on no width tried (1500 configurations): a tuning string reaches them.
#define PF_RING_F32_SHAPES(X, D, N)                                                                                      \
    X(0, 6, 2, 2, 4, 0, true) X(1, 4, 4, 4, 2, 0, true) D(2) X(3, 8, 4, 2, 4, 0, false)                                  \
    X(4, N, 2, 3, 1, 0, true) X(5, N, 3, 3, 1, 0, true) X(6, N, 4, 3, 1, 0, true) X(7, N, 2, 4, 1, 0, true)              \
    X(8, N, 3, 4, 1, 0, true) X(9, N, 4, 4, 1, 0, true) X(10, N, 6, 4, 1, 0, true) X(11, N, 8, 4, 1, 0, true)            \
    X(12, N, 2, 8, 1, 0, true) X(13, N, 3, 8, 1, 0, true) X(14, N, 4, 8, 1, 0, true) X(15, N, 8, 8, 1, 0, true)

// ---------------------------------------------------------------- rows of a block: embedding, residual add + cosine tap
// What bounds these kernels is memory (per row and sublayer the K slices, the residual row both ways and its normed copy), and two
// things kept them from its rate: a normed copy leaves a row as 16-byte pieces 256 bytes apart, so the rows of one
// chunk share every cache line; and each row's sums went through LDS level by level.  So the 16 rows of a chunk go to
// workgroups of one XCD that follow each other (consecutive workgroup ids go to the 8 XCDs in turn), whose L2 puts the
// lines together, all requests of a row are made before the first use, and the two sums take one pass through LDS
// and shuffles, in the order the level-by-level sum had.  7B: residual add 15.4 -> 12.1 us at 512 rows (four slices, 4.8 TB/s), 45 -> 33 us at 2048 rows;
// embedding 18.6 -> 8.4 us and 66 -> 32 us.
__device__ __forceinline__ int pf_row_of_block(int b) { return ((b >> 7) * 8 + (b & 7)) * 16 + ((b >> 3) & 15); }
inline unsigned pf_row_grid(int n_chunks) { return (unsigned)((n_chunks + 7) / 8 * 128); }

// sums of one value pair per thread of a 256-thread workgroup, each in the order of a halving tree (t, t + 128), (t, t + 64),
// ...; valid in thread 0
__device__ __forceinline__ void pf_block_sum2(float& u, float& v, float2* red) {
    const int tid = threadIdx.x;
    red[tid] = float2{u, v};
    __syncthreads();
    if (tid < 64) {
        const float2 a = red[tid], b = red[tid + 128], c = red[tid + 64], d = red[tid + 192];
        u = (a.x + b.x) + (c.x + d.x);
        v = (a.y + b.y) + (c.y + d.y);
        for (int s = 32; s > 0; s >>= 1) { u += __shfl_down(u, s); v += __shfl_down(v, s); }
    }
}

// grid = pf_row_grid; rows of the last chunk at or beyond `rows` are zero-filled.  begin: what a call sets up first (st NULL: a later block)
template <class T>
__global__ __launch_bounds__(256) void pf_embed_kernel(const typename T::elem* E, const int32_t* tokens, int rows, int n_chunks, int d, const float* g_first,
                                                       float* xres, void* xb, int64_t xb_plane, int64_t xb_chunk, float* ssq, float* rscale,
                                                       float inv_d, float eps, const BeginArgs begin) {
    using El = typename T::elem;
    __shared__ float2 red[256];
    const int r = pf_row_of_block(blockIdx.x), tid = threadIdx.x;
    if (begin.st && blockIdx.x == 0) begin_state(begin, tid, 256, 0);
    if (r >= n_chunks * 16) return;
    const bool valid = r < rows;
    const El* src = E + (size_t)(valid ? tokens[r] : 0) * d;
    float ss = 0.f, none = 0.f;
    constexpr int PB = 4;
    struct alignas(4 * sizeof(El)) Four { El e[4]; };
    for (int base = tid * 4; base < d; base += PB * 1024) {
        Four e4[PB];
        float4 g4[PB];
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int n0 = base + q * 1024;
            if (n0 < d) { e4[q] = *(const Four*)(src + n0); g4[q] = *(const float4*)&g_first[n0]; }
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int n0 = base + q * 1024;
            if (n0 < d) {
                const float gg[4] = {g4[q].x, g4[q].y, g4[q].z, g4[q].w};
                float x[4], v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[j] = valid ? T::to_f32(e4[q].e[j]) : 0.f;
                    v[j] = x[j] * gg[j];
                    ss += x[j] * x[j];
                }
                *(float4*)&xres[(size_t)r * d + n0] = float4{x[0], x[1], x[2], x[3]};
                store_act4<T>(xb, xb_plane, (int64_t)(r / 16) * xb_chunk, n0, r % 16, v);
            }
        }
    }
    pf_block_sum2(ss, none, red);
    if (tid == 0) { ssq[r] = ss; rscale[r] = rsqrtf(ss * inv_d + eps); }
}

// grid = pf_row_grid: y = x + sum of the K slices (slice order), residual stream, normed copy for the next sublayer,
// the row's cosine(x, y) (the summand of C_l, Section 3.2) and the statistics of y.  KS = number of K slices.  out: row out.row is the prompt's last and goes to the LM
// head as row 0 of a one-row pass: its normed copy, and ||y||^2 as the one partial that the LM head sums (out.row < 0: none).
struct PfLastRow { int32_t row; void* xb; int64_t xb_plane; float* part; };
template <class T, int KS>
__global__ __launch_bounds__(256) void pf_resid_kernel(const float* raw, int raw_rows, int rows, int d, float* xres, void* xb, int64_t xb_plane,
                                                       int64_t xb_chunk, const float* g_next, float* ssq, float* rscale, float* cos_row,
                                                       float inv_d, float eps, const PfLastRow out) {
    __shared__ float2 red[256];
    const int r = pf_row_of_block(blockIdx.x), tid = threadIdx.x;
    if (r >= rows) return;
    float sxy = 0.f, syy = 0.f;
    constexpr int PB = 4;
    for (int base = tid * 4; base < d; base += PB * 1024) {
        float4 x4[PB], gn[PB], t4[PB][KS];
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int n0 = base + q * 1024;
            if (n0 < d) {
                x4[q] = *(const float4*)&xres[(size_t)r * d + n0];
                gn[q] = *(const float4*)&g_next[n0];
#pragma unroll
                for (int k = 0; k < KS; ++k) t4[q][k] = *(const float4*)&raw[((size_t)k * raw_rows + r) * d + n0];
            }
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int n0 = base + q * 1024;
            if (n0 < d) {
                float4 s4 = t4[q][0];
#pragma unroll
                for (int k = 1; k < KS; ++k) { s4.x += t4[q][k].x; s4.y += t4[q][k].y; s4.z += t4[q][k].z; s4.w += t4[q][k].w; }
                const float x[4] = {x4[q].x, x4[q].y, x4[q].z, x4[q].w}, sv[4] = {s4.x, s4.y, s4.z, s4.w};
                const float gg[4] = {gn[q].x, gn[q].y, gn[q].z, gn[q].w};
                float y[4], v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) { y[j] = x[j] + sv[j]; v[j] = y[j] * gg[j]; sxy += x[j] * y[j]; syy += y[j] * y[j]; }
                *(float4*)&xres[(size_t)r * d + n0] = float4{y[0], y[1], y[2], y[3]};
                store_act4<T>(xb, xb_plane, (int64_t)(r / 16) * xb_chunk, n0, r % 16, v);
                if (r == out.row) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) store_act<T>(out.xb, (size_t)out.xb_plane, 1, n0 + j, 0, v[j]);
                }
            }
        }
    }
    pf_block_sum2(sxy, syy, red);
    if (tid == 0) {
        const float xx = ssq[r];
        float c = sxy * rsqrtf(fmaxf(xx, 1e-16f) * fmaxf(syy, 1e-16f));
        c = fminf(1.f, fmaxf(-1.f, c));
        cos_row[r] = c;
        ssq[r] = syy;
        rscale[r] = rsqrtf(syy * inv_d + eps);
        if (r == out.row) { out.part[0] = 0.f; out.part[1] = syy; }
    }
}

// one sublayer's row cosines of a block (fixed order, double) added to the running sum of C_l (Section 3.2); 256 threads
__device__ __forceinline__ void pf_cos_sum(const float* row, int rows, double* acc, double* red) {
    const int tid = threadIdx.x;
    double s = 0.0;
    for (int r = tid; r < rows; r += 256) s += (double)row[r];
    red[tid] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) *acc += red[0];
}
// grid = sublayers
__global__ __launch_bounds__(256) void pf_cos_sum_kernel(const float* cos_rows /* [sublayers][stride] */, int stride, int rows, double* cos_acc) {
    __shared__ double red[256];
    pf_cos_sum(cos_rows + (size_t)blockIdx.x * stride, rows, cos_acc + blockIdx.x, red);
}

// What follows the LM head of a prompt, in one launch: grid = sublayers + 1 + workgroups that copy.  The last block's cosine sums, the greedy token of the last row, and what the
// call hands back (state, token, cosine sums, the last row's logits where asked for) written straight into pinned host memory (host.st NULL: nothing).  None of them waits for another, and
// a dependent launch costs as much as any of the three: 2 layers of 4096 features, 45 rows, cosine sums with the row's
// hand-over, token and copies in a launch each 5.0 + 4.6 + 4.9 us, this 5.0.  Whole prompts, us,
// four processes of each build in turn: 7B width, 2 layers, 45 rows 307.2 -> 304.4, 1 layer, 130 rows 252.0 -> 247.2; 13B width, 300 rows 467.6 -> 461.9; 70B width, 60 rows 467.0 -> 463.0.
struct PfHost { DevState* st; int32_t* argmax; double* cos; float* logits; };
__global__ __launch_bounds__(256) void pf_finish_kernel(const float* cos_rows, int stride, int rows, double* cos_acc, int sublayers, const AmaxCand* cand, int P, int V,
                                                        int32_t* argmax, DevState* st, const float* logits, const PfHost host) {
    __shared__ double red[256];
    const int b = (int)blockIdx.x, tid = threadIdx.x;
    if (b < sublayers) {
        pf_cos_sum(cos_rows + (size_t)b * stride, rows, cos_acc + b, red);
        if (tid == 0 && host.cos) host.cos[b] = cos_acc[b];
        return;
    }
    if (b == sublayers) {
        if (tid >= 64) return;
        const int idx = row_winner(cand, P, V, st, true, nullptr);
        if (tid == 0) { argmax[0] = idx; if (host.argmax) host.argmax[0] = idx; }
        __builtin_amdgcn_s_waitcnt(0);                            // (an error that row_winner reported is in the state)
        constexpr int N = sizeof(DevState) / 4;
        if (host.st && tid < N) ((uint32_t*)host.st)[tid] = __hip_atomic_load((uint32_t*)st + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (!host.logits) return;
    const int step = ((int)gridDim.x - sublayers - 1) * 256;
    for (int i = (b - sublayers - 1) * 256 + tid; i < V; i += step) host.logits[i] = logits[i];
}
