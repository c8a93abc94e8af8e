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
            uint16_t* o16 = (uint16_t*)a.O + token(r0 + qr) * 3 * C + piece_index(h * d + c);
            v *= inv;
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                uint32_t u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { u[e] = __float_as_uint(v[e]); v[e] -= __uint_as_float(u[e] & 0xFFFF0000u); }
                *reinterpret_cast<uint2*>(o16 + 32 * pl) =
                    make_uint2(__builtin_amdgcn_perm(u[1], u[0], 0x07060302), __builtin_amdgcn_perm(u[3], u[2], 0x07060302));
            }
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
    if constexpr (sizeof(T) == 2)                       // the transposed layout: bf16, 64 channels a head, rows past 32-bit offsets
        if (a.v_transposed) return attn_f32mma_launch<T, 64, true, true>(a, st);
#define PS_AF(DD) (a.d == DD ? attn_f32mma_launch<T, DD, false, true>(a, st) : attn_f32mma_launch<T, DD, false, false>(a, st))
    return a.d <= 32 ? PS_AF(32) : a.d <= 64 ? PS_AF(64) : PS_AF(128);
#undef PS_AF
}

int attention_mfma_bf16(const AttnArgs& a, hipStream_t st, bool* handled);     // attn_mfma.hip

int attention(const AttnArgs& a, int dtype, int mode, hipStream_t st) {
    PS_REQUIRE(a.d > 0 && a.d <= 128, "attention: head dim %d not supported (max 128)", a.d);
    if (mode == 0 && dtype == PSERVE_BF16) {
        bool handled = false;
        PS_TRY(attention_mfma_bf16(a, st, &handled));
        if (handled) return PSERVE_OK;
    }
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
