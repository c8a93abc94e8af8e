// Per-image variable-length attention over the patch batch.
//
// Self-attention needs every token of the OWN image as key/value ("Patch-based
// Self-Attention Module").  The paper rebuilds full images and batches them by resolution;
// because attention carries no positional term inside the block, the token order within an
// image does not matter, so the patch-major token matrix is used as it is: the keys of a
// query token are the contiguous token range cu_seqlens[s] .. cu_seqlens[s+1] of its request
// slot s (RequestOffset of the CSP format times the tokens per patch).  Cross-attention
// ("pixel-wise" operator) attends to the request's own text tokens.
//
// Softmax runs in base 2 on logits pre-multiplied by log2(e)/sqrt(d) (done by the Q projection).
#include "kernels.h"
#include <type_traits>

namespace pserve {

// ---- plain reference kernel: one wavefront per (query token, head), keys spread over lanes ------
template <typename T, int DMAX>
__global__ void __launch_bounds__(256)
attn_simple_kernel(AttnArgs a) {
    __shared__ float sQ[4][DMAX];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t item = (int64_t)blockIdx.x * 4 + wave;
    const int ri = (int)(item / a.heads), h = (int)(item - (int64_t)ri * a.heads);
    const int S = a.geom.S;
    int64_t rows = (int64_t)a.geom.P * S;
    if (a.act.active) rows = (int64_t)(*a.act.count) * S;
    const bool live = ri < rows;            // wave-uniform
    int64_t tok = 0;
    int p = 0;
    if (live) {
        const int pi = ri / S;
        p = a.act.active ? a.act.active[pi] : pi;
        tok = (int64_t)p * S + (ri - pi * S);
    }
    const int d = a.d;
    const T* Q = (const T*)a.Q;
    const T* K = (const T*)a.K;
    const T* V = (const T*)a.V;
    if (live)
        for (int c = lane; c < d; c += 64) sQ[wave][c] = ld_f<T>(Q + tok * a.C + h * d + c);
    __syncthreads();
    if (!live) return;
    const int s = a.owner[p];
    int64_t k0, nk;
    if (a.cross_len) { k0 = (int64_t)a.perm[s] * a.cross_ld; nk = a.cross_len; }
    else { k0 = a.cu_seqlens[s]; nk = a.seq_len ? a.seq_len[s] : a.cu_seqlens[s + 1] - k0; }

    float m = -INFINITY, l = 0.f;
    float acc[DMAX];
#pragma unroll
    for (int c = 0; c < DMAX; ++c) acc[c] = 0.f;
    for (int64_t j = lane; j < nk; j += 64) {
        const int64_t kr = k0 + j;
        const T* kp = K + kr * a.C + h * d;
        float sc = 0.f;
#pragma unroll
        for (int c = 0; c < DMAX; ++c)
            if (c < d) sc = fmaf(sQ[wave][c], ld_f<T>(kp + c), sc);
        const float mn = fmaxf(m, sc);
        const float corr = exp2f(m - mn), pr = exp2f(sc - mn);
        l = l * corr + pr;
        m = mn;
#pragma unroll
        for (int c = 0; c < DMAX; ++c)
            if (c < d) {
                const float v = a.v_transposed ? ld_f<T>(V + (int64_t)(h * d + c) * a.ldv + kr)
                                               : ld_f<T>(V + kr * a.ldv + h * d + c);
                acc[c] = fmaf(pr, v, acc[c] * corr);
            }
    }
    float mall = m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mall = fmaxf(mall, __shfl_xor(mall, off, 64));
    const float sc = (m == -INFINITY) ? 0.f : exp2f(m - mall);
    float lall = l * sc;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lall += __shfl_xor(lall, off, 64);
    const float inv = 1.f / lall;
    T* O = (T*)a.O;
#pragma unroll
    for (int c = 0; c < DMAX; ++c) {
        float v = acc[c] * sc;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (c < d && lane == (c & 63)) st_f<T>(O + tok * a.C + h * d + c, v * inv);
    }
}

// ---- the same on the fp32 matrix cores --------------------------------------------------------------
// For fp32, and for the bf16 shapes the bf16 matrix kernels do not take (widened while they are staged).  A block is 32
// queries of one (request, head); its four wavefronts take every fourth tile of 32 keys each, with a softmax state of
// their own, and meet once at the end: many blocks for few queries, no barrier in the loop, and the long and short
// requests of a batch spread evenly over the CUs.  S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x2_f32: a lane owns
// one query column, and its 16 scores are exactly the B operands of the 16 steps of the second product (key 8 (e / 4) +
// 4 h + e % 4 for lane half h), so the probabilities stay in their registers.  Bound by the matrix pipe (a tile is
// 2 x D / 2 MFMAs of 64 clocks against ~150 vector instructions of softmax and staging): the next tile's rows travel in
// registers while the current one, in LDS private to the wavefront, is computed.  Measured against the plain kernel
// above (5 heads of 64, requests of 4,096 and 3,072 tokens): 62.0 -> 0.41 ms (81 TFLOP/s); 2 heads of 32, 256 and 576 tokens: 136 -> 13 us.
typedef __attribute__((ext_vector_type(16))) float at_f32x16;

typedef __attribute__((ext_vector_type(4))) float at_f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t at_u32x2;

// four elements as loaded (converted where they are used: a load that is converted at once is waited for at once)
template <typename T> struct AtRaw;
template <> struct AtRaw<float> {
    at_f32x4 r;
    __device__ __forceinline__ void load(const float* p) { r = *reinterpret_cast<const at_f32x4*>(p); }
    __device__ __forceinline__ at_f32x4 get() const { return r; }
};
template <> struct AtRaw<uint16_t> {
    at_u32x2 r;
    __device__ __forceinline__ void load(const uint16_t* p) { r = *reinterpret_cast<const at_u32x2*>(p); }
    __device__ __forceinline__ at_f32x4 get() const {
        return at_f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xFFFF0000u), __uint_as_float(r[1] << 16),
                        __uint_as_float(r[1] & 0xFFFF0000u)};
    }
};

// D: head dim rounded up to 32, 64 or 128 (FULL: it is that; else channels past d are zero).  VT: V is [C][ldv] instead of
// [rows][ldv].
template <typename T, int D, bool VT, bool FULL>
__global__ void __launch_bounds__(256, D == 128 ? 1 : 2)
attn_f32mma_kernel(AttnArgs a, int group) {
    constexpr int KT = 32;                              // keys per tile
    constexpr int LK = D + 4;                           // LDS row of a key (16-byte fragment reads: odd number of units)
    constexpr int LV = VT ? KT + 4 : D + 8;             // VT: row of a channel; else row of a key (4 LV = 32 mod 64 banks)
    constexpr int NV = VT ? D : KT;
    constexpr int WAVE = KT * LK + NV * LV;             // floats of LDS per wavefront
    constexpr int NQ = D / 8;                           // 16-byte fragments of a query / key row per lane half
    constexpr int NL = KT * D / 256;                    // vectors of four per lane and operand of a tile
    static_assert(WAVE >= 32 * LK + 64, "the partial results reuse the tiles");
    extern __shared__ __attribute__((aligned(16))) float at_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    float* sK = at_smem + wave * WAVE;
    float* sV = sK + KT * LK;

    // groups of `group` consecutive items (query tiles of one head) are dealt to the XCDs in turn
    const int nsub = 4 * a.qt;                          // 32-query tiles per tile of the call's tables
    const int64_t seq = blockIdx.x >> 3;
    const int64_t it = ((seq / group) * 8 + (blockIdx.x & 7)) * group + seq % group;
    int s, h, tile;
    if (!attn_item_at(a, it / nsub, s, h, tile)) return;
    const int S = a.geom.S;
    const int rows_s = (a.act_off[s + 1] - a.act_off[s]) * S;
    const int r0 = (tile * nsub + (int)(it % nsub)) * 32;
    if (r0 >= rows_s) return;
    int64_t k0;
    int nk;
    if (a.cross_len) { k0 = (int64_t)a.perm[s] * a.cross_ld; nk = a.cross_len; }
    else { k0 = a.cu_seqlens[s]; nk = a.seq_len ? a.seq_len[s] : a.cu_seqlens[s + 1] - (int)k0; }
    const int d = a.d, C = a.C;
    auto token = [&](int r) -> int64_t {                // compact row of the request -> token
        const int pi = a.act_off[s] + r / S;
        const int p = a.act.active ? a.act.active[pi] : pi;
        return (int64_t)p * S + (r - (r / S) * S);
    };
    const at_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    at_f32x4 q[NQ];
    {
        const T* qp = (const T*)a.Q + token(min(r0 + fr, rows_s - 1)) * C + h * d;
        AtRaw<T> raw[NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) raw[j].load(qp + (FULL ? 8 * j + 4 * fh : min(8 * j + 4 * fh, d - 4)));
#pragma unroll
        for (int j = 0; j < NQ; ++j) q[j] = FULL || 8 * j + 4 * fh < d ? raw[j].get() : zero;
    }
    const T* Kp = (const T*)a.K + k0 * C + h * d;
    const T* Vp = VT ? (const T*)a.V + (int64_t)h * d * a.ldv + k0 : (const T*)a.V + k0 * a.ldv + h * d;
    // staging: vector v of a lane is row (v * 64 + lane) / (D / 4) of the tile; rows past the last key are clamped to it
    // (their scores are masked, their probabilities zero) and their values staged as zeros (zero times a last value that is
    // not finite would be NaN).  VT: channel row, four keys a vector.
    constexpr int VR = D / 4, VK = KT / 4;
    const int ch = (lane % VR) * 4, chc = FULL ? ch : min(ch, d - 4);        // the lane's channels (64 is a multiple of VR)
    AtRaw<T> rk[NL], rv[VT ? 1 : NL];
    at_f32x4 rvt[VT ? NL : 1];
    auto load = [&](int t) {
        const int last = nk - 1 - t * KT;               // last row of the tile that exists
        const T* kt = Kp + (int64_t)t * KT * C;
        const T* vt = VT ? Vp + t * KT : Vp + (int64_t)t * KT * a.ldv;
#pragma unroll
        for (int v = 0; v < NL; ++v) {
            const int row = min((v * 64 + lane) / VR, last);
            rk[v].load(kt + row * C + chc);
            if constexpr (!VT) rv[v].load(vt + row * (int)a.ldv + chc);
        }
        if constexpr (VT) {
#pragma unroll
            for (int v = 0; v < NL; ++v) {
                const int i = v * 64 + lane, kk = (i % VK) * 4;
                const T* vp = vt + (int64_t)(i / VK) * a.ldv;
#pragma unroll
                for (int u = 0; u < 4; ++u) rvt[v][u] = ld_f<T>(vp + min(kk + u, last));
            }
        }
    };
    float m = -INFINITY, l = 0.f;                       // of the lane's query, over the keys of this wavefront
    at_f32x16 o[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    const int tiles = (nk + KT - 1) / KT;
    if (wave < tiles) load(wave);
    for (int t = wave; t < tiles; t += 4) {
        // LDS of the wavefront alone: its accesses execute in order, only the compiler has to keep that order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int v = 0; v < NL; ++v) {
            const int i = v * 64 + lane;
            const bool in = FULL || ch < d;
            *reinterpret_cast<at_f32x4*>(sK + (i / VR) * LK + ch) = in ? rk[v].get() : zero;
            if constexpr (VT) *reinterpret_cast<at_f32x4*>(sV + (i / VK) * LV + (i % VK) * 4) = rvt[v];
            else *reinterpret_cast<at_f32x4*>(sV + (i / VR) * LV + ch) = in ? rv[v].get() : zero;
        }
        if (const int left = nk - t * KT; left < KT) {  // ragged last tile
#pragma unroll 1
            for (int i = lane; i < KT * D; i += 64)
                if ((VT ? i % KT : i / D) >= left) sV[VT ? (i / KT) * LV + i % KT : (i / D) * LV + i % D] = 0.f;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (t + 4 < tiles) load(t + 4);
        at_f32x16 sc[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[0][e] = sc[1][e] = 0.f;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const at_f32x4 kf = *reinterpret_cast<const at_f32x4*>(sK + fr * LK + 8 * j + 4 * fh);
            sc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.x, q[j].x, sc[0], 0, 0, 0);
            sc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.y, q[j].y, sc[1], 0, 0, 0);
            sc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.z, q[j].z, sc[0], 0, 0, 0);
            sc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.w, q[j].w, sc[1], 0, 0, 0);
        }
        float p[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) p[e] = sc[0][e] + sc[1][e];
        if ((t + 1) * KT > nk) {                        // ragged last tile
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (t * KT + 8 * (e >> 2) + 4 * fh + (e & 3) >= nk) p[e] = -INFINITY;
        }
        float mn = m;
#pragma unroll
        for (int e = 0; e < 16; ++e) mn = fmaxf(mn, p[e]);
        mn = fmaxf(mn, __shfl_xor(mn, 32, 64));
        const float corr = exp2f(m - mn);
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            p[e] = exp2f(p[e] - mn);
            sum += p[e];
        }
        l = l * corr + sum;
        m = mn;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] *= corr;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (VT) {
                at_f32x4 vf[D / 32];
#pragma unroll
                for (int dt = 0; dt < D / 32; ++dt)
                    vf[dt] = *reinterpret_cast<const at_f32x4*>(sV + (32 * dt + fr) * LV + 8 * g + 4 * fh);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int dt = 0; dt < D / 32; ++dt)
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[dt][i], p[4 * g + i], o[dt], 0, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int dt = 0; dt < D / 32; ++dt)
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(sV[(8 * g + 4 * fh + i) * LV + 32 * dt + fr], p[4 * g + i],
                                                                     o[dt], 0, 0, 0);
            }
        }
    }
    l += __shfl_xor(l, 32, 64);
    // ---- the four wavefronts' results: common maximum, then the sums in a fixed order
    __syncthreads();                                    // all tiles of LDS are free
    float* sO = sK;                                     // [32 queries][LK], then the row sums and maxima
    float* sL = sK + 32 * LK;
    if (fh == 0) { sL[fr] = m; sL[32 + fr] = l; }
    __syncthreads();
    float mall = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mall = fmaxf(mall, at_smem[w * WAVE + 32 * LK + fr]);
    const float f = m == -INFINITY ? 0.f : exp2f(m - mall);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<at_f32x4*>(sO + fr * LK + 32 * dt + 8 * g + 4 * fh) =
                at_f32x4{o[dt][4 * g] * f, o[dt][4 * g + 1] * f, o[dt][4 * g + 2] * f, o[dt][4 * g + 3] * f};
    __syncthreads();
    const int qr = tid >> 3;                            // eight threads per query
    if (r0 + qr >= rows_s) return;
    float mq = -INFINITY, lq = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) mq = fmaxf(mq, at_smem[w * WAVE + 32 * LK + qr]);
    float fw[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float mw = at_smem[w * WAVE + 32 * LK + qr];
        fw[w] = mw == -INFINITY ? 0.f : exp2f(mw - mq);
        lq += at_smem[w * WAVE + 32 * LK + 32 + qr] * fw[w];
    }
    const float inv = 1.f / lq;
    T* op = (T*)a.O + token(r0 + qr) * C + h * d;
#pragma unroll
    for (int c = (tid & 7) * 4; c < D; c += 32) {
        if (c >= d) break;
        at_f32x4 v = zero;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const at_f32x4*>(at_smem + w * WAVE + qr * LK + c);
        if constexpr (sizeof(T) == 2)
            *reinterpret_cast<uint2*>(op + c) = make_uint2(pack_bf16x2(v.x * inv, v.y * inv), pack_bf16x2(v.z * inv, v.w * inv));
        else if (a.out_pieces) {
            store_pieces4((uint16_t*)a.O + token(r0 + qr) * 3 * C + piece_index(h * d + c), v.x * inv, v.y * inv, v.z * inv, v.w * inv);
        } else
            *reinterpret_cast<at_f32x4*>(op + c) = v * inv;
    }
}

template <typename T, int D, bool VT, bool FULL>
static int attn_f32mma_launch(const AttnArgs& a, hipStream_t st) {
    const int64_t items = (int64_t)a.max_tiles * 4 * a.qt * a.heads;
    // eight groups per XCD: its share of the long and short items, and consecutive query tiles of a head on one L2
    const int group = (int)std::min<int64_t>(64, cdiv(items, 64));
    const unsigned grid = (unsigned)(8 * group * cdiv(items, 8 * group));
    constexpr int lds = 4 * (32 * (D + 4) + (VT ? D * 36 : 32 * (D + 8))) * 4;
    PS_SET_LDS_ONCE((attn_f32mma_kernel<T, D, VT, FULL>), lds);
    attn_f32mma_kernel<T, D, VT, FULL><<<grid, 256, lds, st>>>(a, group);
    return check_launch("attn_f32mma_kernel");
}

template <typename T>
static int attn_f32mma(const AttnArgs& a, hipStream_t st) {
    if constexpr (sizeof(T) == 2)                       // the transposed layout: bf16, 64 channels a head, rows of 2^25 values and more
        if (a.v_transposed) return attn_f32mma_launch<T, 64, true, true>(a, st);
#define PS_AF(DD) (a.d == DD ? attn_f32mma_launch<T, DD, false, true>(a, st) : attn_f32mma_launch<T, DD, false, false>(a, st))
    return a.d <= 32 ? PS_AF(32) : a.d <= 64 ? PS_AF(64) : PS_AF(128);
#undef PS_AF
}

// For tests (no part of the ABI): self-attention of all tokens of a plan with the transposed bf16 layout on the fp32 matrix
// cores, which a forward call takes from 2^25 tokens on.  Q pre-scaled, V [C][ldv]; tables: device, 2 (n + 1) int32.
extern "C" int pserve_test_attn_transposed(const pserve_plan_t* plan, const void* Q, const void* K, const void* V, int64_t ldv, void* O,
                                           int32_t C, int32_t* tables, void* stream) {
    PS_REQUIRE(plan && Q && K && V && O && tables && C % 64 == 0 && ldv >= plan->T && plan->text_len == 0, "pserve_test_attn_transposed");
    AttnArgs a{};
    a.Q = Q; a.K = K; a.V = V; a.O = O; a.C = C; a.heads = C / 64; a.d = 64; a.v_transposed = true; a.ldv = ldv; a.n = plan->n;
    a.geom = PatchGeom{plan->P, plan->S, plan->ph, plan->pw, plan->pw + 2, (plan->ph + 2) * (plan->pw + 2)};
    a.act = ActiveList{nullptr, nullptr};
    a.owner = plan->d_tab[PSERVE_TAB_PATCH_OWNER]; a.perm = plan->d_tab[PSERVE_TAB_PERM]; a.cu_seqlens = plan->d_tab[PSERVE_TAB_CU_SEQLENS];
    a.act_off = tables; a.tile_off = tables + plan->n + 1; a.qt = 1; a.max_tiles = attention_max_tiles(plan, 1);
    a.max_rows = plan->max_tokens_per_image;
    PS_TRY(attention_tiles(plan->d_tab[PSERVE_TAB_REQUEST_OFFSET], nullptr, plan->n, plan->S, 1, tables, tables + plan->n + 1, (hipStream_t)stream));
    return attn_f32mma<uint16_t>(a, (hipStream_t)stream);
}

// ---- fp32 self-attention on the bf16 matrix cores ---------------------------------------------------------
// As the fp32 layers: every operand in three bf16 pieces (cut3x2), six products of which all terms are exact in the fp32
// accumulators.  attn_cut_kernel lays the keys and values of a request out in tiles of 32 keys and one head, K rows of
// [3][D] and V^T rows of [3][32], in the very order (swizzle included) in which a tile lies in LDS: a tile is one linear copy.
// attn_split_kernel: a block is 128 queries of one (request, head), four wavefronts of 32; K and V^T fragments and P stay as in
// the bf16 kernel (a lane owns a query column, its eight scores of a 16-key step are consecutive keys), Q is cut once, P in
// registers.  Two blocks a CU.  A step forms the scores of the NEXT tile while the softmax of this one runs (24 MFMAs beside
// most of its ~270 vector instructions), then the output products; keys and values have rings of three stages of their own,
// filled two steps ahead.  The softmax reference moves only when a score passes it by 8 (a factor of 256 costs fp32 nothing).
// Requests of 4,096 and 3,072 tokens, 5 heads of 64 (280 items of 128 and 96 tiles): 360 (fp32 kernel) -> 234 us, a block an item ->
// 173 + 15 us, 512 shares and no spilled register in the loop (143 -> 178 TFLOP/s of fp32).  Bound by the issue of MFMAs (1,536 of 2,770 clocks a tile) and vector
// instructions, with every CU busy by the clock (2.15 GHz with 160 CUs busy, 1.8 with all).
constexpr int ASP_NS = 3;
constexpr float AT_LOWEST = -3.402823466e38f;       // the softmax reference in front of the first key
constexpr int AT_SHARES = 512;       // shares of a call (a multiple of 8)
// Units of a share at least.  us of an LSATTN layer, no such bound / 8 / 12 / 16: 4,096 tokens, 4 heads of 64, a fiftieth computed 216 / 107 / 106 / 108, a
// twentieth 160 / 109 / 109 / 110; all of 1,024 + 12 x 256 88 / 79 / 75 / 82, 1,600 + 20 x 256 117 / 114 / 116 / 121.
constexpr int AT_SHORTEST = 12;
static_assert(AT_SHORTEST > AT_START, "a share without keys");
template <int D> struct AttnSplitCfg {
    static constexpr int KV = 3 * 32 * D / 8, TILE_V = 2 * KV;       // 16-byte slots of the keys, of a tile
    static constexpr int LPT = TILE_V / 256;                         // direct loads of a wavefront and tile
    static constexpr size_t LDS = (size_t)ASP_NS * TILE_V * 16;
    static constexpr int PART = (D / 2 + 2) * 256;                   // floats of a partial result: 256 lanes' outputs, references, sums
};
typedef __attribute__((ext_vector_type(8))) __bf16 at_bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t at_u32x4;
typedef __attribute__((address_space(3))) void at_lds_void;
template <int D> __device__ __forceinline__ int at_swz(int row) { return D == 64 ? (row >> 1) & 7 : (row >> 2) & 3; }
// first tile of request slot s: room for the tiles of all slots before it
__device__ __forceinline__ int64_t at_tile0(const int32_t* cu_seqlens, int s) { return cu_seqlens[s] / 32 + s; }
// three pieces of eight values
template <bool PLAIN = false>
__device__ __forceinline__ void at_cut(const float (&x)[8], at_u32x4 (&o)[3]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t u[3];
        if constexpr (PLAIN) cut3x2_plain(x[2 * q], x[2 * q + 1], u);
        else cut3x2(x[2 * q], x[2 * q + 1], u);
#pragma unroll
        for (int p = 0; p < 3; ++p) o[p][q] = u[p];
    }
}

// Block = (tile of the grid's upper bound, head); tiles that no request has are left alone.
template <int D>
__global__ void __launch_bounds__(4 * D)
attn_cut_kernel(const float* __restrict__ K, const float* __restrict__ V, const int32_t* __restrict__ cu_seqlens,
                const int32_t* __restrict__ seq_len, int32_t n, int32_t C, at_u32x4* __restrict__ out) {
    using Cfg = AttnSplitCfg<D>;
    const int64_t tile = blockIdx.x;
    const int h = blockIdx.y, tid = threadIdx.x;
    int lo = 0, hi = n;                                 // largest s with tile0(s) <= tile
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (at_tile0(cu_seqlens, mid) <= tile) lo = mid; else hi = mid;
    }
    const int64_t k0 = cu_seqlens[lo];
    const int nk = seq_len ? seq_len[lo] : cu_seqlens[lo + 1] - (int)k0, key0 = (int)(tile - at_tile0(cu_seqlens, lo)) * 32;
    if (key0 >= nk) return;
    at_u32x4* dst = out + (tile * gridDim.y + h) * Cfg::TILE_V;
    const float* Kh = K + k0 * C + h * D;
    const float* Vh = V + k0 * C + h * D;
    float x[8];
    at_u32x4 o[3];
    {                                                   // eight channels of a key
        const int r = tid / (D / 8), c = tid % (D / 8), key = key0 + r;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const at_f32x4 w = *reinterpret_cast<const at_f32x4*>(Kh + (int64_t)min(key, nk - 1) * C + 8 * c + 4 * q);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * q + i] = key < nk ? w[i] : 0.f;
        }
        at_cut(x, o);
#pragma unroll
        for (int p = 0; p < 3; ++p) dst[r * (3 * D / 8) + p * (D / 8) + (c ^ at_swz<D>(r))] = o[p];
    }
    {                                                   // eight keys of a channel
        const int ch = tid % D, c = tid / D;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int key = key0 + 8 * c + i;
            const float w = Vh[(int64_t)min(key, nk - 1) * C + ch];
            x[i] = key < nk ? w : 0.f;
        }
        at_cut(x, o);
#pragma unroll
        for (int p = 0; p < 3; ++p) dst[Cfg::KV + ch * 12 + p * 4 + (c ^ at_swz<32>(ch))] = o[p];
    }
}

// O of a lane's query (column fr of the output tiles), scaled
template <int D>
__device__ __forceinline__ void at_store(const AttnArgs& a, const at_f32x16 (&ot)[D / 32], float inv, bool mine, int64_t tok, int h, int fh) {
    constexpr int DT = D / 32;
    const int C = a.C;
    if (mine) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = h * D + 32 * dt + 8 * g + 4 * fh;
                const at_f32x4 v = {ot[dt][4 * g] * inv, ot[dt][4 * g + 1] * inv, ot[dt][4 * g + 2] * inv, ot[dt][4 * g + 3] * inv};
                if (a.out_pieces) store_pieces4((uint16_t*)a.O + tok * 3 * C + piece_index(c), v.x, v.y, v.z, v.w);
                else *reinterpret_cast<at_f32x4*>((float*)a.O + tok * C + c) = v;
            }
    }
}

// The work of a call is a row of units: slot by slot, head by head, 128 queries by 128 queries, an item of AT_START units for its start and end
// and one for each 32 keys.  It is cut into equal shares, one a block; a cut that falls into an item's start lies in front of its first key.
// Items that a cut goes through leave partial results, which attn_join_kernel puts together.
// slot, head, query tile of nq, keys, tile of keys k of steps that a share with this unit starts at; the item's first unit
struct AttnUnit { int s, h, tile, nq, nk, steps, k; int64_t first; };
__host__ __device__ __forceinline__ AttnUnit at_unit(const AttnArgs& a, int64_t u) {
    AttnUnit r;
    int lo = 0, hi = a.n;                               // largest s with unit_off[s] <= u
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.unit_off[mid] <= u) lo = mid; else hi = mid;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    lo = __builtin_amdgcn_readfirstlane(lo);
#endif
    r.s = lo;
    r.nk = a.seq_len ? a.seq_len[r.s] : a.cu_seqlens[r.s + 1] - a.cu_seqlens[r.s];
    r.steps = (r.nk + 31) / 32;
    r.nq = ((a.act_off[r.s + 1] - a.act_off[r.s]) * a.geom.S + 127) / 128;
    const int64_t in = u - a.unit_off[r.s], item = in / (r.steps + AT_START);
    const int at = (int)(in - item * (r.steps + AT_START));
    r.k = at < AT_START ? 0 : at - AT_START;
    r.h = (int)(item / r.nq);
    r.tile = (int)(item - (int64_t)r.h * r.nq);
    r.first = u - at;
    return r;
}
// tiles of keys of an item that lie in front of unit u
__host__ __device__ __forceinline__ int at_tiles(const AttnUnit& w, int64_t u) {
    const int64_t t = u - w.first - AT_START;
    return t >= w.steps ? w.steps : t < 0 ? 0 : (int)t;
}
// Shares of a call for which the plan allows `blocks`: a mask may leave few units.  None is shorter than AT_SHORTEST, so none has no keys: the join
// reads a part of every share that an item lies in.
__host__ __device__ __forceinline__ int at_shares(int64_t units, int blocks) {
    const int64_t most = units / AT_SHORTEST;
    return units == 0 ? 0 : most < 1 ? 1 : most < blocks ? (int)most : blocks;
}
__host__ __device__ __forceinline__ int64_t at_share(int64_t units, int b, int shares) { return units * b / shares; }
// share of a block, -1: none.  An XCD's blocks take neighbouring shares: they stream the keys of the same few heads through its L2.
__host__ __device__ __forceinline__ int at_share_of(int block, int shares) {
    const int xcd = block & 7, b = xcd * shares / 8 + (block >> 3);
    return b < (xcd + 1) * shares / 8 ? b : -1;
}
// place of the part that share b leaves of an item: 2 b of the item that it starts in, 2 b + 1 of its last, whose head it has
__host__ __device__ __forceinline__ int64_t at_place(int b, bool head) { return 2 * (int64_t)b + head; }
// block j of the join: whether an item's first cut is that behind share j, the item, and the share that it ends in
__host__ __device__ __forceinline__ bool at_join_of(const AttnArgs& a, int j, int blocks, AttnUnit* w, int* last) {
    const int64_t units = a.unit_off[a.n];
    const int shares = at_shares(units, blocks);
    if (j + 1 >= shares) return false;
    *w = at_unit(a, at_share(units, j + 1, shares));
    if (w->k == 0 || at_tiles(*w, at_share(units, j, shares)) > 0) return false;       // between two items; or not the item's first cut
    *last = j + 1;
    while (at_tiles(*w, at_share(units, *last + 1, shares)) < w->steps) ++*last;
    return true;
}

// SHARED: a block takes a share of the units; else an item, longest first.
template <int D, bool SHARED>
__global__ void __launch_bounds__(256, 2)
attn_split_kernel(AttnArgs a, const at_u32x4* __restrict__ tiles_kv, float* __restrict__ parts) {
    using Cfg = AttnSplitCfg<D>;
    constexpr int KS = D / 16, DT = D / 32, LPT = Cfg::LPT, TILE_V = Cfg::TILE_V, KV = Cfg::KV;
    extern __shared__ __attribute__((aligned(16))) float at_smem[];
    at_u32x4* ring = reinterpret_cast<at_u32x4*>(at_smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int S = a.geom.S, C = a.C;
    int b = 0;
    int64_t u = 0, u1 = 1;
    if constexpr (SHARED) {
        const int64_t units = a.unit_off[a.n];
        const int shares = at_shares(units, gridDim.x);
        b = at_share_of(blockIdx.x, shares);
        if (b < 0) return;
        u = at_share(units, b, shares);
        u1 = at_share(units, b + 1, shares);
    }
#pragma unroll 1
    while (u < u1) {
    AttnUnit w{};
    int steps;                                          // tiles of this share, and below the keys from its first on
    if constexpr (SHARED) {
        w = at_unit(a, u);
        steps = at_tiles(w, u1) - w.k;
        u = w.first + AT_START + w.steps;
        if (steps == 0) return;                         // (the share ends in this item's start)
    } else {
        const int seq = blockIdx.x >> 3, grp = seq / a.group, it = (grp * 8 + (blockIdx.x & 7)) * a.group + (seq - grp * a.group);
        if (!attn_item_at(a, it / a.qt, w.s, w.h, w.tile)) return;
        w.tile = w.tile * a.qt + it % a.qt;
        w.nk = a.seq_len ? a.seq_len[w.s] : a.cu_seqlens[w.s + 1] - a.cu_seqlens[w.s];
        steps = w.steps = (w.nk + 31) / 32;
    }
    const int s = w.s, h = w.h, r0 = w.tile * 128, rows_s = (a.act_off[s + 1] - a.act_off[s]) * S;
    if (!SHARED && r0 >= rows_s) return;
    const int nk = w.nk - w.k * 32;
    const bool whole = !SHARED || steps == w.steps;
    const at_u32x4* src = tiles_kv + ((at_tile0(a.cu_seqlens, s) + w.k) * a.heads + h) * TILE_V;
    const int64_t src_step = (int64_t)a.heads * TILE_V;
    // Keys of tile tk and values of tile tv into stages of their own (past the end: the last tile again, never read).  Buffer
    // loads: behind flat ones the compiler waits for all LDS reads in flight instead of counting them.
    auto issue = [&](int tk, int tv, bool values) {
#if defined(__HIP_DEVICE_COMPILE__)
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(src + min(tk, steps - 1) * src_step), 0, TILE_V * 16, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(src + min(tv, steps - 1) * src_step), 0, TILE_V * 16, 0x00020000);
        at_u32x4* dk = ring + tk % ASP_NS * KV;
        at_u32x4* dv = ring + (ASP_NS - 1 + tv % ASP_NS) * KV;         // (index i counts on behind the keys of a tile)
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int idx = wave + 4 * i;
            if (idx < KV / 64) __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (at_lds_void*)(dk + idx * 64), 16, tid * 16, i * 4096, 0, 0);
            else if (values) __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (at_lds_void*)(dv + idx * 64), 16, tid * 16, i * 4096, 0, 0);
        }
#endif
    };
    issue(0, 0, false);
    issue(1, 0, true);
    issue(2, 1, true);
    auto token = [&](int r) -> int64_t {                // compact row of the request -> token
        const int pi = a.act_off[s] + r / S;
        const int p = a.act.active ? a.act.active[pi] : pi;
        return (int64_t)p * S + (r - (r / S) * S);
    };
    const int my_row = r0 + wave * 32 + fr;
    const int64_t tok = token(min(my_row, rows_s - 1));
    at_bf16x8 q[3][KS];
    {
        const float* qp = (const float*)a.Q + tok * C + h * D + 8 * fh;
        float x[KS][8];
        bool plain = true;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const at_f32x4 w0 = *reinterpret_cast<const at_f32x4*>(qp + 16 * ks), w1 = *reinterpret_cast<const at_f32x4*>(qp + 16 * ks + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[ks][i] = w0[i]; x[ks][4 + i] = w1[i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i) plain = plain && cut_is_plain(x[ks][2 * i], x[ks][2 * i + 1]);
        }
        // one branch for all values (one a pair costs 6,000 clocks a share; the loop over 32 keys 2,770)
        auto cut_all = [&](auto plain_c) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                at_u32x4 o[3];
                at_cut<decltype(plain_c)::value>(x[ks], o);
#pragma unroll
                for (int p = 0; p < 3; ++p) q[p][ks] = __builtin_bit_cast(at_bf16x8, o[p]);
            }
        };
        if (__all(plain)) cut_all(std::true_type{});
        else cut_all(std::false_type{});
    }
    const int krow = (fr & ~12) | ((fr & 4) << 1) | ((fr & 8) >> 1);         // key of MFMA row fr (bits 2 and 3 swapped)
    const at_u32x4* pK = ring + krow * (3 * D / 8);
    const at_u32x4* pV = ring + ASP_NS * KV + fr * 12;
    const int ksw = at_swz<D>(krow), vsw = at_swz<32>(fr);
    at_f32x16 sc[2];                                    // scores of a tile: products of the large pieces, the others
    // Fragments of 16 channels (keys) / of 16 keys x 32 channels (values).  Product n takes pieces pa[n] and pb[n] (n = 1 the large
    // ones): piece 0 is read two products into the set before into registers of its own, piece 1 behind the last product of the
    // set before that reads it (n = 3), piece 2 at the head of its set, five products ahead.
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {1, 0, 0, 1, 2, 0};
    at_bf16x8 kf[4], vf[4];                             // pieces 0 (two sets), 1, 2
    auto at_piece = [](int set, int pl) constexpr { return pl == 0 ? set & 1 : 1 + pl; };
    auto read_k = [&](int st, int ks, int pl) {
        kf[at_piece(ks, pl)] = __builtin_bit_cast(at_bf16x8, pK[st * KV + pl * (D / 8) + ((2 * ks + fh) ^ ksw)]);
    };
    auto read_v = [&](int st, int f, int pl) {          // f: 16-key step f / DT, channels 32 (f % DT) ..
        vf[at_piece(f, pl)] = __builtin_bit_cast(at_bf16x8, pV[st * KV + (f % DT) * 384 + pl * 4 + ((2 * (f / DT) + fh) ^ vsw)]);
    };
    const at_f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto score = [&](int ks, int n) {
        at_f32x16& c = sc[n != 1];
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[at_piece(ks, pa[n])], q[pb[n]][ks], ks == 0 && n < 2 ? zero16 : c, 0, 0, 0);
    };
    // Output: products of the large pieces, the others (beside a large sum the matrix unit cuts small products off), and the
    // total they are added to every ATT_FLUSH tiles (the rounding errors of a long chain).
    constexpr int ATT_FLUSH = 8;
    at_f32x16 o[DT], ol[DT], ot[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = ol[dt][e] = ot[dt][e] = 0.f;
    // (the reference is never -infinity, so that scores of -infinity have probabilities of zero until there is another)
    float m = AT_LOWEST, l = 0.f, p[16], mx;
    // the scores of tile t are summed (p, their maximum in mx): those behind the last key are masked, the lane halves meet
    auto finish = [&](int t) {
        if ((t + 1) * 32 > nk) {
            mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (t * 32 + 16 * (e >> 3) + 8 * fh + (e & 7) >= nk) p[e] = -INFINITY;
                mx = fmaxf(mx, p[e]);
            }
        }
        const uint32_t u = __float_as_uint(mx);
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        mx = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    };
    auto add_scores = [&](int e) {
        p[e] = sc[0][e] + sc[1][e];
        mx = e == 0 ? p[0] : fmaxf(mx, p[e]);
    };
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * LPT) : "memory");     // the keys of tile 0 have landed
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) read_k(0, ks, pl);
#pragma unroll
        for (int n = 0; n < 6; ++n) score(ks, n);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) add_scores(e);
    finish(0);
    int st = 0;
#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
        const int nst = st + 1 == ASP_NS ? 0 : st + 1;
        // The keys of tile t + 1 and the values of tile t have landed (the next ones are on their way); everybody has left
        // iteration t - 1, which read the keys of tile t and the values of tile t - 1.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPT) : "memory");
        read_k(nst, 0, 0);
        read_k(nst, 0, 1);
        issue(t + 3, t + 2, true);
        const bool flush = t % ATT_FLUSH == 0;
        if (flush || __any(mx > m + 8.f)) {             // (a row sum that is not a number stays one)
            const float mn = mx > m + 8.f ? mx : m, corr = exp2_square(0.5f * (m - mn));
            m = mn;
            l *= corr;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    ot[dt][e] = (ot[dt][e] + (o[dt][e] + ol[dt][e])) * corr;
                    o[dt][e] = ol[dt][e] = 0.f;
                }
        }
        const float hm = -0.5f * m;
        // The next tile's scores, and behind each MFMA up to five of this tile's vector instructions (about four are free, and none
        // where there is no MFMA: as two phases a tile took 3,360 clocks of which 1,536 are MFMAs) and a fragment read for six MFMAs
        // later: the probabilities in pairs, in four (D = 32: two) steps each; those that the first output products do not need
        // behind these; then the sums of the next scores.  (Past the end: scores never used.)
        constexpr int PS = D == 64 ? 6 : 8, SL = 6 * KS, PST = D == 64 ? 4 : 1;      // pairs beside the scores; slots a pair
        at_u32x4 pp[2][3];
        float sum = 0.f, x0 = 0.f, x1 = 0.f;
        auto pair = [&](int g, int step) {              // step 0 .. 3 of pair g
            if (step == 0) {
                x0 = exp2_square(fmaf(p[2 * g], 0.5f, hm));
                x1 = exp2_square(fmaf(p[2 * g + 1], 0.5f, hm));
                return;
            }
            if (step == 1) sum += x0 + x1;
            const uint32_t u = near_bf16x2(x0, x1);                 // (cut3x2 of values of at most 2^8; a NaN stays one in x0)
            pp[g >> 2][step - 1][g & 3] = u;
            if (step < 3) {
                x0 -= lo_bf16(u);
                x1 -= hi_bf16(u);
            }
        };
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int ks = i / 6, n = i % 6;
            score(ks, n);
            if (n == 0) read_k(nst, ks, 2);
            if (n == 2) { if (ks + 1 < KS) read_k(nst, ks + 1, 0); else read_v(st, 0, 0); }
            if (n == 4) { if (ks + 1 < KS) read_k(nst, ks + 1, 1); else read_v(st, 0, 1); }
            if (D == 64) pair(i / PST, i % PST);
            else {                                      // 32 steps over 12 slots
#pragma unroll
                for (int z = i * 32 / SL; z < (i + 1) * 32 / SL; ++z) pair(z / 4, z % 4);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < 12 * DT; ++i) {
            const int f = i / 6, n = i % 6;
            at_f32x16& acc = n == 1 ? o[f % DT] : ol[f % DT];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[at_piece(f, pa[n])], __builtin_bit_cast(at_bf16x8, pp[f / DT][pb[n]]), acc, 0, 0, 0);
            if (n == 0) read_v(st, f, 2);
            if (n == 2 && f + 1 < 2 * DT) read_v(st, f + 1, 0);
            if (n == 4 && f + 1 < 2 * DT) read_v(st, f + 1, 1);
            if (D == 64) {
                if (i < 8) pair(PS + i / 4, i % 4);
                else add_scores(i - 8);
            } else if (i >= 4) {
                add_scores(2 * (i - 4));
                add_scores(2 * (i - 4) + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        l += sum;
        finish(t + 1);
        st = nst;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) ot[dt][e] += o[dt][e] + ol[dt][e];
    // no load may still target LDS, and nobody may still read it, when the next share of an item starts
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    l += __shfl_xor(l, 32, 64);
    if (!whole) {
        float* dst = parts + at_place(b, w.k == 0) * Cfg::PART + tid;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) dst[(16 * dt + e) * 256] = ot[dt][e];
        dst[16 * DT * 256] = m;
        dst[(16 * DT + 1) * 256] = l;
        continue;
    }
    at_store<D>(a, ot, 1.f / l, my_row < rows_s, tok, h, fh);
    if constexpr (!SHARED) return;
    }
}

// Puts the items together that a cut between two shares goes through: block j those whose first cut is that behind share j.  The
// parts come in a fixed order, each scaled to the common reference.
template <int D>
__global__ void __launch_bounds__(256)
attn_join_kernel(AttnArgs a, const float* __restrict__ parts, int nb) {
    using Cfg = AttnSplitCfg<D>;
    constexpr int DT = D / 32;
    const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, fr = lane & 31, fh = lane >> 5;
    AttnUnit w;
    int last;
    if (!at_join_of(a, j, nb, &w, &last)) return;
    const int rows_s = (a.act_off[w.s + 1] - a.act_off[w.s]) * a.geom.S;
    const int my_row = w.tile * 128 + (tid >> 6) * 32 + fr, row = min(my_row, rows_s - 1), S = a.geom.S;
    const int pi = a.act_off[w.s] + row / S;
    const int64_t tok = (int64_t)(a.act.active ? a.act.active[pi] : pi) * S + row % S;
    auto part = [&](int b) { return parts + at_place(b, b == j) * Cfg::PART + tid; };
    float m = AT_LOWEST, l = 0.f;
    for (int b = j; b <= last; ++b) m = fmaxf(m, part(b)[16 * DT * 256]);
    at_f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    for (int b = j; b <= last; ++b) {
        const float* src = part(b);
        const float mb = src[16 * DT * 256], f = exp2_square(0.5f * (mb - m));
        l = fmaf(src[(16 * DT + 1) * 256], f, l);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] = fmaf(src[(16 * dt + e) * 256], f, o[dt][e]);
    }
    at_store<D>(a, o, 1.f / l, my_row < rows_s, tok, w.h, fh);
}

template <int D>
static int attn_split(const AttnArgs& a, hipStream_t st) {
    using Cfg = AttnSplitCfg<D>;
    const int64_t tiles = (int64_t)a.geom.P * a.geom.S / 32 + a.n;
    attn_cut_kernel<D><<<dim3((unsigned)tiles, (unsigned)a.heads), 4 * D, 0, st>>>((const float*)a.K, (const float*)a.V, a.cu_seqlens,
        a.seq_len, a.n, a.C, (at_u32x4*)a.cut);
    PS_TRY(check_launch("attn_cut_kernel"));
    if (a.shares) {
        float* parts = (float*)((at_u32x4*)a.cut + tiles * a.heads * Cfg::TILE_V);
        PS_SET_LDS_ONCE((attn_split_kernel<D, true>), Cfg::LDS);
        attn_split_kernel<D, true><<<(unsigned)a.shares, 256, Cfg::LDS, st>>>(a, (const at_u32x4*)a.cut, parts);
        PS_TRY(check_launch("attn_split_kernel"));
        attn_join_kernel<D><<<(unsigned)a.shares - 1, 256, 0, st>>>(a, parts, a.shares);
        return check_launch("attn_join_kernel");
    }
    AttnArgs b = a;
    const int64_t items = (int64_t)a.max_tiles * a.qt * a.heads;
    b.group = (int)std::min<int64_t>(8, cdiv(items, 8));
    PS_SET_LDS_ONCE((attn_split_kernel<D, false>), Cfg::LDS);
    attn_split_kernel<D, false><<<(unsigned)(8 * b.group * cdiv(items, 8 * b.group)), 256, Cfg::LDS, st>>>(b, (const at_u32x4*)a.cut, nullptr);
    return check_launch("attn_split_kernel");
}

// From 128 blocks of 128 queries on, where a request has 1,024 keys: below, the fp32 kernel's blocks of 32 queries with the keys
// shared out to four wavefronts spread better.  With heads of 32 channels from 129 on: at 128 the fp32 kernel's 512 blocks run all at once
// (4,096 tokens, 4 of 32 121 / 138, 16,384, 1 of 32 390 / 448, 4 x 1,024, 4 of 32 52 / 60; 4,096, 5 of 32 (160) 164 / 140; 136 blocks 159 / 135;
// of 64 channels, 128 blocks: 212 / 207, 682 / 629, 89 / 90).  us of an LSATTN layer, fp32 kernel / this: 4,096 + 3,072 tokens, 5 heads of 64
// (280 blocks) 460 / 309; 2 x 2,304, 5 of 32 (180) 117 / 102; 4,608, 10 of 32 (360) 391 / 282; 2,304, 5 of 64 (90) 138 / 133;
// 4 x 576, 5 of 64 (100) 68 / 70; 4,096, 2 of 64 (64) 124 / 181; 16 x 256, 5 of 64 (160) 72 / 73.  Error of a layer
// against 64 bits: 4,096 tokens 4.8e-8 / 3.4e-8, 4 x 1,024 4.7e-8 / 3.4e-8, 4,608 (10 heads) 4.9e-8 / 3.4e-8, 2 x 2,304 4.2e-8 / 3.5e-8.
size_t attention_cut_bytes(const pserve_plan_t* plan, int32_t C, int32_t heads, int dtype, int mode) {
    if (dtype != PSERVE_F32 || mode != 0 || C % heads != 0 || (C / heads != 32 && C / heads != 64)) return 0;
    if ((int64_t)attention_max_tiles(plan, 1) * heads < (C / heads == 32 ? 129 : 128) || plan->max_tokens_per_image < 1024) return 0;
    const size_t part = (C / heads == 32 ? AttnSplitCfg<32>::PART : AttnSplitCfg<64>::PART) * sizeof(float);
    return (size_t)(plan->T / 32 + plan->n) * C * 32 * 12 + 2 * attention_shares(plan, C, heads) * part;
}

// Blocks that share out the units of such a call equally, 0: a block an item.  Both in tiles of one CU (1.25 us with 64 channels a head, 0.76 with
// 32): items go, the longest first, to the CU with the least work, the last one of an odd number alone, which costs a fifth of it more; shares
// take their mean, and cutting and joining.  185 batches (1,024 to 16,384 tokens, up to 100 small requests beside a large one): the slower
// form by 2.3 % at most.  us of an LSATTN layer, items / shares: 64 channels, 5 heads: 4,096 tokens 220 / 181, 2 x 4,096 373 / 331, 4,096 + 3,072
// 316 / 277, 4 x 4,096 653 / 628, 8 x 4,096 1,161 / 1,192, 5 x 2,304 309 / 332, 16,384 1,980 / 1,813, 1,024 + 24 x 64 90 / 84, 4,096 + 60 x 64 274 / 237;
// 32 channels, 5 heads: 4,096 140 / 107, 9,216 443 / 375, 3 x 4,096 256 / 260, 5 x 1,024 70 / 75.
int attention_shares(const pserve_plan_t* plan, int32_t C, int32_t heads) {
    struct Len { int64_t cost, items; };
    std::vector<Len> len;
    int64_t items = 0, units = 0;
    const int32_t *ro = plan->h_tab[PSERVE_TAB_REQUEST_OFFSET], *sl = plan->h_tab[PSERVE_TAB_SEQ_LEN];
    for (int s = 0; s < plan->n; ++s) {
        const int64_t rows = (int64_t)(ro[s + 1] - ro[s]) * plan->S;
        len.push_back({AT_START + cdiv(sl[s], 32), cdiv(rows, 128) * heads});
        items += len.back().items;
        units += len.back().items * len.back().cost;
    }
    const int shares = (int)std::min<int64_t>(AT_SHARES, units / AT_SHORTEST / 8 * 8);
    if (shares == 0 || items > 32 * 256) return 0;      // (so many items come out even)
    std::sort(len.begin(), len.end(), [](const Len& x, const Len& y) { return x.cost > y.cost; });
    struct Cu { int64_t load, last; bool odd; };
    auto more = [](const Cu& x, const Cu& y) { return x.load > y.load; };
    std::vector<Cu> cu(256, Cu{0, 0, false});           // a heap, the least load in front
    for (const Len& l : len)
        for (int64_t i = 0; i < l.items; ++i) {
            std::pop_heap(cu.begin(), cu.end(), more);
            cu.back() = Cu{cu.back().load + l.cost, l.cost, !cu.back().odd};
            std::push_heap(cu.begin(), cu.end(), more);
        }
    double by_item = 0.0;
    for (const Cu& c : cu) by_item = std::max(by_item, c.load + (c.odd ? 0.2 * c.last : 0.0));
    return 1.04 * units / 256 + 27 < by_item ? shares : 0;
}

// For tests (host only, no part of the ABI): whether the fp32 self-attention of a plan goes to the bf16 matrix cores
extern "C" int pserve_test_attn_cut(const pserve_plan_t* plan, int32_t C, int32_t heads) {
    return attention_cut_bytes(plan, C, heads, PSERVE_F32, 0) != 0;
}
// ... and in how many shares (0: a block an item)
extern "C" int pserve_test_attn_shares(const pserve_plan_t* plan, int32_t C, int32_t heads) { return attention_shares(plan, C, heads); }
// Both kernels' walk over the units of a call, on the host: n requests of rows[s] computed rows (a patch each) and keys[s] keys.  0 if every
// unit is taken once and the join reads the parts that are written, each once; else the number of the check that fails.
extern "C" int pserve_test_attn_walk(const int32_t* rows, const int32_t* keys, int32_t n, int32_t heads) {
    PS_REQUIRE(rows && keys && n > 0 && heads > 0, "pserve_test_attn_walk");
    return guarded("pserve_test_attn_walk", [&]() -> int {
        std::vector<int32_t> act(n + 1, 0), cu(n + 1, 0);
        std::vector<int64_t> off(n + 1, 0);
        for (int s = 0; s < n; ++s) {
            act[s + 1] = act[s] + rows[s];
            cu[s + 1] = cu[s] + keys[s];
            off[s + 1] = off[s] + cdiv(rows[s], 128) * heads * (AT_START + cdiv(keys[s], 32));
        }
        AttnArgs a{};
        a.n = n; a.heads = heads; a.geom.S = 1; a.act_off = act.data(); a.cu_seqlens = cu.data(); a.unit_off = off.data();
        const int64_t units = off[n];
        const int shares = at_shares(units, AT_SHARES);
        std::vector<int> taken(units, 0), part(2 * AT_SHARES, -1);      // part: the first unit of the item it is of
        for (int block = 0; block < AT_SHARES; ++block) {
            const int b = at_share_of(block, shares);
            if (b < 0) continue;
            int64_t u = at_share(units, b, shares);
            const int64_t u1 = at_share(units, b + 1, shares);
            while (u < u1) {
                const AttnUnit w = at_unit(a, u);
                const int steps = at_tiles(w, u1) - w.k;
                if (steps < 0) return 5;
                for (int i = 0; i < steps; ++i) ++taken[w.first + AT_START + w.k + i];
                if (steps != 0 && steps != w.steps) {
                    if (part[at_place(b, w.k == 0)] >= 0) return 1;
                    part[at_place(b, w.k == 0)] = (int)w.first;
                }
                u = w.first + AT_START + w.steps;
                if (steps == 0) break;
            }
        }
        for (int s = 0; s < n; ++s)                     // (nobody takes the units of an item's start)
            for (int64_t u = off[s]; u < off[s + 1]; u += cdiv(keys[s], 32) + AT_START)
                for (int i = 0; i < AT_START; ++i) ++taken[u + i];
        for (int t : taken) if (t != 1) return 2;
        for (int j = 0; j < AT_SHARES - 1; ++j) {
            AttnUnit w;
            int last;
            if (!at_join_of(a, j, AT_SHARES, &w, &last)) continue;
            for (int b = j; b <= last; ++b) {
                int& p = part[at_place(b, b == j)];
                if (p != w.first) return 3;
                p = -1;
            }
        }
        for (int p : part) if (p >= 0) return 4;
        return 0;
    });
}

int attention_mfma_bf16(const AttnArgs& a, hipStream_t st, bool* handled);     // attn_mfma.hip

int attention(const AttnArgs& a, int dtype, int mode, hipStream_t st) {
    PS_REQUIRE(a.d > 0 && a.d <= 128, "attention: head dim %d not supported (max 128)", a.d);
    if (mode == 0 && dtype == PSERVE_BF16) {
        bool handled = false;
        PS_TRY(attention_mfma_bf16(a, st, &handled));
        if (handled) return PSERVE_OK;
    }
    if (mode == 0 && dtype == PSERVE_F32 && a.cut && !a.cross_len && a.tile_off && a.act_off)
        return a.d == 64 ? attn_split<64>(a, st) : attn_split<32>(a, st);
    // four channels a load (the queries, keys and values are the library's own buffers: rows start 16-byte aligned when C
    // and d are multiples of four)
    if (mode == 0 && a.d % 4 == 0 && a.C % 4 == 0 && (a.v_transposed ? a.d == 64 && dtype == PSERVE_BF16 : a.ldv % 4 == 0) &&
        a.tile_off && a.act_off)
        return dtype == PSERVE_BF16 ? attn_f32mma<uint16_t>(a, st) : attn_f32mma<float>(a, st);
    const int64_t items = (int64_t)a.geom.P * a.geom.S * a.heads;
    const unsigned grid = (unsigned)cdiv(items, 4);
#define PS_ATTN(TT, DM) attn_simple_kernel<TT, DM><<<grid, 256, 0, st>>>(a)
    if (dtype == PSERVE_BF16) {
        if (a.d <= 32) PS_ATTN(uint16_t, 32); else if (a.d <= 64) PS_ATTN(uint16_t, 64); else PS_ATTN(uint16_t, 128);
    } else {
        if (a.d <= 32) PS_ATTN(float, 32); else if (a.d <= 64) PS_ATTN(float, 64); else PS_ATTN(float, 128);
    }
#undef PS_ATTN
    return check_launch("attn_simple_kernel");
}

}  // namespace pserve
