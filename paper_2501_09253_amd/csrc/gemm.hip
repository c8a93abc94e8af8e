// GEMM / implicit-GEMM 3x3 convolution over the patch batch, and weight packing.
//
// out[t][co] = bias[co] + sum_{tap, ci} a[nbr(t, tap)][ci] * W[co][ci][tap]  (+ residual)
// The 3x3 convolution reads the padded patch buffer [P][ph+2][pw+2][C] whose one-pixel ring
// was filled from same-image neighbours (zeros at image edges), so every patch is a
// self-contained tile and the nine taps are nine shifted views of it (patch-based
// convolution, "Patch-Tailored Diffusion Operators").  Pixel-wise operators (linear layers,
// feed-forward, attention projections) are the one-tap case and run on the patch batch
// unchanged.
//
// Packed weights: B[tap][n][k], k contiguous (conv W[co][ci][ky][kx] -> tap = ky*3+kx;
// linear W[k][n] -> transposed).  Accumulation is fp32.
#include "kernels.h"
#include <type_traits>

namespace pserve {

// ---- row / column addressing shared by the kernels ------------------------------------------------
struct RowInfo {
    int64_t tok;       // input row id
    int64_t out_row;   // row id used for output / residual addressing
    int64_t a_off;     // element offset of the row's first A element (tap 0)
    bool valid;
};

__device__ __forceinline__ RowInfo row_info(const GemmArgs& a, int ri) {
    RowInfo r;
    int64_t tok = ri;
    bool valid;
    if (a.tokens_are_rows && a.act.active) {
        const int cnt = *a.act.count;
        const int pi = ri / a.geom.S;
        valid = pi < cnt;
        tok = valid ? (int64_t)a.act.active[pi] * a.geom.S + (ri - pi * a.geom.S) : 0;
    } else {
        valid = ri < a.M;
        if (!valid) tok = 0;
    }
    r.out_row = (!a.tokens_are_rows && a.row_group > 0) ? (tok / a.row_group) * a.row_group_pad + tok % a.row_group : tok;
    r.tok = tok;
    r.valid = valid;
    if (a.conv) {
        const int p = (int)(tok / a.geom.S), q = (int)(tok - (int64_t)p * a.geom.S);
        const int y = q / a.geom.pw, x = q - y * a.geom.pw;
        const int am = a.a_mul ? a.a_mul : 1;
        r.a_off = ((int64_t)p * a.geom.pS + (am * y + a.a_dy) * a.geom.ppw + am * x + a.a_dx) * a.lda;
        if (a.o_mul) r.out_row = (int64_t)p * a.o_S + (a.o_mul * y + a.o_dy) * a.o_pw + a.o_mul * x + a.o_dx;
    } else {
        r.a_off = tok * a.lda;
    }
    return r;
}

// tanh form: v/2 (1 + tanh(sqrt(2/pi) (v + 0.044715 v^3)))
__device__ __forceinline__ float gelu_tanh_f(float v) {
    return 0.5f * v * (1.f + tanhf(0.7978845608028654f * (v + 0.044715f * v * v * v)));
}
__device__ __forceinline__ float gelu_f(float v) { return 0.5f * v * (1.f + erff(v * 0.70710678118654752f)); }

template <typename T>
__device__ __forceinline__ void route_store(const GemmArgs& a, int64_t tok, int col, float v) {
    const int sg = col / a.seg_cols, c = col - sg * a.seg_cols;
    const GemmSeg& s = a.seg[sg];
    v *= s.scale;
    T* o = (T*)s.ptr;
    if (s.transposed) st_f<T>(o + (int64_t)c * s.ld + tok, v);
    else st_f<T>(o + tok * s.ld + c, v);
}

// ---- plain reference kernel: 64x64 tile, fp32 FMA, any shape --------------------------------------
template <typename T, bool GEGLU>
__global__ void __launch_bounds__(256)
gemm_simple_kernel(GemmArgs a) {
    constexpr int BM = 64, BN = 64, BK = 16;
    constexpr int NB = GEGLU ? 2 : 1;                 // B tiles per block (value + gate)
    __shared__ float sA[BK][BM + 1];
    __shared__ float sB[NB][BK][BN + 1];
    __shared__ int64_t s_aoff[BM];
    __shared__ int64_t s_tok[BM];
    __shared__ int s_valid[BM];
    const int tid = threadIdx.x;
    const int m0 = blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;                   // output column (GEGLU: in F space)
    if (a.tokens_are_rows && a.act.active && m0 >= *a.act.count * a.geom.S) return;
    if (tid < BM) {
        const RowInfo r = row_info(a, m0 + tid);
        s_aoff[tid] = r.a_off;
        s_tok[tid] = r.out_row;
        s_valid[tid] = r.valid;
    }
    __syncthreads();
    const T* A = (const T*)a.A;
    const T* B = (const T*)a.B;
    const int tx = tid & 15, ty = tid >> 4;
    float acc[NB][4][4] = {};
    for (int tap = 0; tap < a.taps; ++tap) {
        const int tw = a.tap_w ? a.tap_w : 3;
        const int64_t tap_off = a.conv ? ((int64_t)(tap / tw) * a.geom.ppw + (tap % tw)) * a.lda : 0;
        for (int k0 = 0; k0 < a.K; k0 += BK) {
            for (int i = tid; i < BM * BK; i += 256) {
                const int m = i / BK, k = i - m * BK;
                float v = 0.f;
                if (s_valid[m] && k0 + k < a.K) v = ld_f<T>(A + s_aoff[m] + tap_off + k0 + k);
                sA[k][m] = v;
            }
            for (int h = 0; h < NB; ++h)
                for (int i = tid; i < BN * BK; i += 256) {
                    const int n = i / BK, k = i - n * BK;
                    // GEGLU: packed columns hold [GROUP values | GROUP gates] per group
                    int col = n0 + n;
                    bool ok = col < (GEGLU ? a.N / 2 : a.N);
                    if (GEGLU) col = (col / GEGLU_GROUP) * 2 * GEGLU_GROUP + h * GEGLU_GROUP + col % GEGLU_GROUP;
                    float v = 0.f;
                    if (ok && k0 + k < a.K) v = ld_f<T>(B + ((int64_t)tap * a.N + col) * a.K + k0 + k);
                    sB[h][k][n] = v;
                }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < BK; ++k) {
                float av[4], bv[NB][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) av[i] = sA[k][ty * 4 + i];
#pragma unroll
                for (int h = 0; h < NB; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) bv[h][j] = sB[h][k][tx * 4 + j];
#pragma unroll
                for (int h = 0; h < NB; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[h][i][j] = fmaf(av[i], bv[h][j], acc[h][i][j]);
            }
            __syncthreads();
        }
    }
    const int ncols = GEGLU ? a.N / 2 : a.N;
    for (int i = 0; i < 4; ++i) {
        const int m = ty * 4 + i;
        if (!s_valid[m]) continue;
        const int64_t tok = s_tok[m];
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + tx * 4 + j;
            if (col >= ncols) continue;
            float v;
            if (GEGLU) {
                const int pc = (col / GEGLU_GROUP) * 2 * GEGLU_GROUP + col % GEGLU_GROUP;
                const float val = acc[0][i][j] + (a.bias ? a.bias[pc] : 0.f);
                const float gate = acc[NB - 1][i][j] + (a.bias ? a.bias[pc + GEGLU_GROUP] : 0.f);
                v = val * gelu_f(gate);
                st_f<T>((T*)a.seg[0].ptr + tok * a.seg[0].ld + col, v);
            } else {
                v = acc[0][i][j] + (a.bias ? a.bias[col] : 0.f);
                if (a.rowbias) v += a.rowbias[(int64_t)a.row_owner[tok / a.geom.S] * a.N + col];
                if (a.act_gelu) v = gelu_tanh_f(v);
                if (a.rowscale) v *= a.rowscale[(int64_t)a.row_owner[tok / a.geom.S] * a.rowscale_ld + col];
                if (a.res) v += ld_f<T>((const T*)a.res + tok * a.ldr + col);
                route_store<T>(a, tok, col, v);
            }
        }
    }
}

// ---- the same on the fp32 matrix cores ------------------------------------------------------------
// v_mfma_f32_32x32x2_f32: full fp32 products and sums, 256 flops per clock and CU.  Bound by the matrix pipe: a tile of
// 32 x 32 per wavefront needs two 16-byte LDS reads per four MFMAs (256 clocks), so nothing of the bf16 kernels'
// staging effort is called for and small tiles cost little.  A fragment read of 16 bytes serves four MFMAs: lane half h
// holds k = 8j + 4h + i for MFMA i of step j, the same for both operands.  Tiles are staged through registers (the next
// step's loads travel while this step is computed) into a double-buffered LDS tile, one barrier per step; LDS rows are
// padded by 16 bytes (an odd number of 16-byte units: conflict free).  The taps of a convolution run inside a channel
// chunk, so the nine reads of a pixel's chunk come from the cache.  WK wavefronts share a tile's K range (summed through
// LDS at the end), which keeps small problems on many CUs.  bf16 operands (the shapes the bf16 matrix kernels do not
// take) are widened while they are staged.  Measured against the plain kernel above: two 3x3 convolutions, q/k/v and out
// projection of 7,168 tokens x 320 channels 1,288 -> 430 us together (a convolution 173 us = 76 TFLOP/s); one convolution,
// q/k/v and out projection of 832 tokens x 64 channels 126 -> 21 us.
typedef __attribute__((ext_vector_type(16))) float gm_f32x16;

typedef __attribute__((ext_vector_type(4))) float gm_f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t gm_u32x2;
// four elements as loaded (converted when they go to LDS: a load that is converted at once is waited for at once)
template <typename T> struct GmRaw;
template <> struct GmRaw<float> {
    gm_f32x4 r;
    __device__ __forceinline__ void load(const float* p) { r = *reinterpret_cast<const gm_f32x4*>(p); }
    __device__ __forceinline__ gm_f32x4 get() const { return r; }
};
template <> struct GmRaw<uint16_t> {
    gm_u32x2 r;
    __device__ __forceinline__ void load(const uint16_t* p) { r = *reinterpret_cast<const gm_u32x2*>(p); }
    __device__ __forceinline__ gm_f32x4 get() const {
        return gm_f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xFFFF0000u), __uint_as_float(r[1] << 16),
                        __uint_as_float(r[1] & 0xFFFF0000u)};
    }
};

template <typename T, int BM, int BN, bool GEGLU>
__global__ void __launch_bounds__(256)
gemm_f32mma_kernel(GemmArgs a) {
    constexpr int WM = BM / 32, WN = BN / 32, WK = 4 / (WM * WN);    // wavefronts along M, N and K
    constexpr int NB = GEGLU ? 2 : 1;                                // B tiles per block (value + gate)
    constexpr int BK = WK == 4 ? 64 : 32, LD = BK + 4;
    constexpr int VA = BM * BK / 1024, VB = NB * BN * BK / 1024;     // 16-byte vectors per thread and step
    constexpr int VPR = BK / 4;                                      // vectors per row
    constexpr int STAGE = (BM + NB * BN) * LD;
    static_assert(2 * STAGE >= WK * WM * WN * NB * 1024, "the partial tiles of the K groups reuse the staging buffers");
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
    __shared__ int64_t s_aoff[BM];
    __shared__ int64_t s_tok[BM];
    __shared__ int s_valid[BM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;            // n0: output column (GEGLU: in F space)
    if (a.tokens_are_rows && a.act.active && m0 >= *a.act.count * a.geom.S) return;
    if (tid < BM) {
        const RowInfo r = row_info(a, m0 + tid);
        s_aoff[tid] = r.a_off;
        s_tok[tid] = r.out_row;
        s_valid[tid] = r.valid;
    }
    __syncthreads();
    const int ncols = GEGLU ? a.N / 2 : a.N;
    // what this thread stages: rows of A and packed weight rows of B, always the same columns of the step
    const T* pa[VA];
    const T* pb[VB];
#pragma unroll
    for (int v = 0; v < VA; ++v) {
        const int row = (tid + v * 256) / VPR;
        pa[v] = (const T*)a.A + s_aoff[s_valid[row] ? row : 0];        // rows past the end: any that exists (not stored)
    }
#pragma unroll
    for (int v = 0; v < VB; ++v) {
        const int row = (tid + v * 256) / VPR, h = row / BN;
        int col = min(n0 + row - h * BN, ncols - 1);
        if (GEGLU) col = (col / GEGLU_GROUP) * 2 * GEGLU_GROUP + h * GEGLU_GROUP + col % GEGLU_GROUP;
        pb[v] = (const T*)a.B + (int64_t)col * a.K;
    }
    const int kv = (tid % VPR) * 4;                                  // 256 is a multiple of VPR: the same for every v
    const int tw = a.tap_w ? a.tap_w : 3;
    const int64_t tap_b = (int64_t)a.N * a.K;
    const int steps = a.taps * ((a.K + BK - 1) / BK);
    GmRaw<T> ra[VA], rb[VB];
    bool in = true;                                                  // the loaded k exist (K is a multiple of 4, not of BK)
    int tap = 0, k0 = 0;                                             // of the step loaded next
    auto load = [&]() {
        const int k = min(k0 + kv, a.K - 4);
        in = k0 + kv < a.K;
        const int64_t ao = (a.conv ? ((int64_t)(tap / tw) * a.geom.ppw + (tap % tw)) * a.lda : 0) + k;
        const int64_t bo = tap * tap_b + k;
#pragma unroll
        for (int v = 0; v < VA; ++v) ra[v].load(pa[v] + ao);
#pragma unroll
        for (int v = 0; v < VB; ++v) rb[v].load(pb[v] + bo);
        if (++tap == a.taps) { tap = 0; k0 += BK; }
    };
    // two accumulators per tile (even and odd k): shorter chains of dependent MFMAs, shorter sums
    gm_f32x16 acc[NB][2];
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[h][0][e] = acc[h][1][e] = 0.f;
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / (WK * WN);
    const int a_rd = (wm * 32 + fr) * LD + 4 * fh, b_rd = (BM + wn * 32 + fr) * LD + 4 * fh;
    load();
    for (int s = 0; s < steps; ++s) {
        float* st = smem + (s & 1) * STAGE;
#pragma unroll
        for (int v = 0; v < VA; ++v)
            *reinterpret_cast<gm_f32x4*>(st + ((tid + v * 256) / VPR) * LD + kv) = in ? ra[v].get() : gm_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < VB; ++v)
            *reinterpret_cast<gm_f32x4*>(st + (BM + (tid + v * 256) / VPR) * LD + kv) = in ? rb[v].get() : gm_f32x4{0.f, 0.f, 0.f, 0.f};
        if (s + 1 < steps) load();
        // one barrier a step: the buffer written above was last read in step s - 2, before the barrier of step s - 1
        __syncthreads();
#pragma unroll
        for (int j = 0; j < BK / 8 / WK; ++j) {
            const int k8 = (wk * (BK / 8 / WK) + j) * 8;
            const gm_f32x4 av = *reinterpret_cast<const gm_f32x4*>(st + a_rd + k8);
#pragma unroll
            for (int h = 0; h < NB; ++h) {
                const gm_f32x4 bv = *reinterpret_cast<const gm_f32x4*>(st + b_rd + h * BN * LD + k8);
                acc[h][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv.x, acc[h][0], 0, 0, 0);
                acc[h][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv.y, acc[h][1], 0, 0, 0);
                acc[h][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv.z, acc[h][0], 0, 0, 0);
                acc[h][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv.w, acc[h][1], 0, 0, 0);
            }
        }
    }
    // element e of a lane: row 8 (e / 4) + 4 fh + e % 4, column fr of the wavefront's 32 x 32 tile.  The K groups of a
    // tile share its rows out: group wk finishes the elements e / (16 / WK) == wk.
    constexpr int EW = 16 / WK;
    float out[NB][EW];
    if constexpr (WK == 1) {
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
            for (int e = 0; e < 16; ++e) out[h][e] = acc[h][0][e] + acc[h][1][e];
    } else {
        __syncthreads();
        float* part = smem + (wm * WN + wn) * WK * NB * 1024 + lane;
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
            for (int e = 0; e < 16; ++e) part[((wk * NB + h) * 16 + e) * 64] = acc[h][0][e] + acc[h][1][e];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                float v = 0.f;
#pragma unroll
                for (int g = 0; g < WK; ++g) v += part[((g * NB + h) * 16 + wk * EW + e) * 64];
                out[h][e] = v;
            }
    }
    const int col = n0 + wn * 32 + fr;
    if (col >= ncols) return;
    const int pc = GEGLU ? (col / GEGLU_GROUP) * 2 * GEGLU_GROUP + col % GEGLU_GROUP : col;
    const float b0 = a.bias ? a.bias[pc] : 0.f, b1 = GEGLU && a.bias ? a.bias[pc + GEGLU_GROUP] : 0.f;
    const int sg = GEGLU ? 0 : col / a.seg_cols;
    const GemmSeg seg = a.seg[sg];
    T* op = (T*)seg.ptr + (int64_t)(col - sg * a.seg_cols) * (seg.transposed ? seg.ld : 1);
    const int64_t o_ld = seg.transposed ? 1 : seg.ld;
#pragma unroll
    for (int e = 0; e < EW; ++e) {
        const int ee = wk * EW + e;
        const int m = wm * 32 + 8 * (ee >> 2) + 4 * fh + (ee & 3);
        if (!s_valid[m]) continue;
        const int64_t tok = s_tok[m];
        float v = out[0][e] + b0;
        if (GEGLU) {
            v *= gelu_f(out[NB - 1][e] + b1);
        } else {
            if (a.rowbias) v += a.rowbias[(int64_t)a.row_owner[tok / a.geom.S] * a.N + col];
            if (a.act_gelu) v = gelu_tanh_f(v);
            if (a.rowscale) v *= a.rowscale[(int64_t)a.row_owner[tok / a.geom.S] * a.rowscale_ld + col];
            if (a.res) v += ld_f<T>((const T*)a.res + tok * a.ldr + col);
            v *= seg.scale;
        }
        st_f<T>(op + tok * o_ld, v);
    }
}

// Time of a launch of gemm_f32mma_kernel in 64 x 64 tiles on the fullest CU (a tile: 32 clocks a k), and its tile: 32 x 32
// (bm = bn = 32), 64 x 32 or 64 x 64.  The smaller tiles fetch more per MFMA and pay the K reduction, so they must win by
// their share.
static double f32mma_tiles(int64_t M, int64_t ncols, int* bm, int* bn) {
    const double c64 = (double)cdiv(cdiv(M, 64) * cdiv(ncols, 64), 256), cmn = 0.5 * 1.05 * cdiv(cdiv(M, 64) * cdiv(ncols, 32), 256),
                 c32 = 0.25 * 1.15 * cdiv(cdiv(M, 32) * cdiv(ncols, 32), 256);
    *bm = c32 < c64 && c32 < cmn ? 32 : 64;
    *bn = *bm == 64 && c64 <= cmn ? 64 : 32;
    return std::min(c64, std::min(cmn, c32));
}

template <typename T>
static bool gemm_f32mma(const GemmArgs& a, hipStream_t st) {
    // 16-byte (bf16: 8-byte) loads of four k
    if (a.K % 4 != 0 || a.lda % 4 != 0 || ((uintptr_t)a.A | (uintptr_t)a.B) % (4 * sizeof(T)) != 0) return false;
    const bool geglu = a.epi == EPI_GEGLU;
    const int ncols = geglu ? a.N / 2 : a.N;
    int bm, bn;
    f32mma_tiles(a.M, ncols, &bm, &bn);
    const dim3 grid((unsigned)cdiv(a.M, bm), (unsigned)cdiv(ncols, bn));
#define PS_F32MMA(BM_, BN_)                                                            \
    do {                                                                               \
        if (geglu) gemm_f32mma_kernel<T, BM_, BN_, true><<<grid, 256, 0, st>>>(a);     \
        else gemm_f32mma_kernel<T, BM_, BN_, false><<<grid, 256, 0, st>>>(a);          \
    } while (0)
    if (bm == 32) PS_F32MMA(32, 32);
    else if (bn == 32) PS_F32MMA(64, 32);
    else PS_F32MMA(64, 64);
#undef PS_F32MMA
    return true;
}

// ---- fp32 on the bf16 matrix cores ----------------------------------------------------------------
// The bf16 MFMA does 16 times the work of the fp32 one, so an fp32 value is cut into three bf16 pieces
// (cut3x2: x = x0 + x1 + x2) and a product is x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0), every term exact in
// the fp32 accumulators; what is left out is at most 2^-23.9 of a product, of either sign, and a sum has an eighth as many
// roundings.  The large terms and the others have accumulators of their own.  Both operands come in pieces, rows of [K / 32][3][32]: the weights
// are cut when they are packed (split_packed), the activations by the kernel that produces them (cutting them here, once a tile
// and step, took as long as the MFMAs).  A step's 32 k of a row are 192 contiguous bytes: as three runs of 64 the loads into LDS,
// which bound the kernel, took twice as long.
//   Tile 64 x 32 TN, four wavefronts: two along M, two sharing a step's 32 k (summed through LDS at the end).  A wavefront reads
// 3 (1 + TN) fragments for 6 TN MFMAs, so LDS and matrix pipe are about level at TN = 5.  Both operands are staged by direct
// loads into a ring of three stages (two blocks a CU at TN = 2); behind the barrier of a step its stage is refilled and the NEXT step's fragments are read
// between the MFMAs of this one.  LDS rows are 192 bytes, chunk c of a piece at c ^ ((row >> 2) & 3): conflict free.
//   Two convolutions of 7,168 tokens x 320 channels: 162 -> 78 us each (170 TFLOP/s of fp32); bound by the bf16 matrix pipe at the clock it
// gets (1.0 PFLOP/s) and, for few tiles, by a tile's start and end (7 us).  Error of a block of two convolutions and an attention
// against 64 bits 2.6e-7 -> 1.9e-7.
typedef __attribute__((ext_vector_type(8))) __bf16 gs_bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t gs_u32x4;
typedef __attribute__((address_space(3))) void gs_lds_void;

// f(integral_constant 0), f(1), .. f(N - 1)
template <int I, int N, class F> __device__ __forceinline__ void gs_for_from(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); gs_for_from<I + 1, N>(f); }
}
template <int N, class F> __device__ __forceinline__ void gs_for(F&& f) { gs_for_from<0, N>(f); }

template <int TN> struct SplitCfg {
    static constexpr int BM = 64, BN = 32 * TN, NS = 3;
    static constexpr int STAGE_V = 3 * (BM + BN) * 4;                  // 16-byte slots: rows of A, then of B, [3][4] each
    static constexpr int LD = (STAGE_V / 64 + 3) / 4;                  // direct loads of a wavefront and step: three of A, then B
    static constexpr size_t LDS = (size_t)NS * STAGE_V * 16;
    static_assert(LDS >= (size_t)4 * TN * 4096 && LDS + BM * 16 <= 160 * 1024, "tile");
};

template <int TN, bool GEGLU>
__global__ void __launch_bounds__(256, (SplitCfg<TN>::LDS <= 79 * 1024 ? 2 : 1))
gemm_split_kernel(GemmArgs a, const uint16_t* __restrict__ Bs) {
    using Cfg = SplitCfg<TN>;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, NS = Cfg::NS, STAGE_V = Cfg::STAGE_V, LD = Cfg::LD, NINS = STAGE_V / 64;
    static_assert(!GEGLU || TN % 2 == 0, "GEGLU: as many values as gates");
    extern __shared__ __attribute__((aligned(16))) uint8_t gs_smem[];
    gs_u32x4* ring = reinterpret_cast<gs_u32x4*>(gs_smem);
    __shared__ int64_t s_tok[BM];                                      // -1: the row does not exist
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * (GEGLU ? BN / 2 : BN);       // n0: output column
    if (a.tokens_are_rows && a.act.active && m0 >= *a.act.count * a.geom.S) return;
    const int ncols = GEGLU ? a.N / 2 : a.N;
    // packed column of output column f (GEGLU: its value or gate)
    auto packed = [&](int f, int gate) { return GEGLU ? (f / GEGLU_GROUP) * 2 * GEGLU_GROUP + gate * GEGLU_GROUP + f % GEGLU_GROUP : f; };
    const int K = a.K, tw = a.tap_w ? a.tap_w : 3;
    const int steps = a.taps * (K / 32);
    // staging: a load fills 64 slots.  Load l of a wavefront: slots of A for l < 3, else of B; row slot / 12, chunk slot % 12
    int a_lane[3], b_lane[LD - 3];
#pragma unroll
    for (int l = 0; l < LD; ++l) {
        const int slot = min(wave + 4 * l, NINS - 1) * 64 + lane - (l < 3 ? 0 : 12 * BM), row = slot / 12, c = slot - row * 12;
        const int chunk = c ^ ((row >> 2) & 3);             // the two low bits: the place inside the piece
        if (l < 3) {
            const RowInfo r = row_info(a, m0 + row);
            if (c == 0) s_tok[row] = r.valid ? r.out_row : -1;
            a_lane[l < 3 ? l : 0] = (int)((r.a_off * 3 + chunk * 8) * 2);
        } else {
            const int h = GEGLU && row >= BN / 2, col = packed(min(n0 + row - h * (BN / 2), ncols - 1), h);
            b_lane[l >= 3 ? l - 3 : 0] = (int)(((int64_t)col * 3 * K + chunk * 8) * 2);
        }
    }
    int tap = 0, k0 = 0, left = steps, istage = 0;      // of the step loaded next; past the last one it is loaded again (never read)
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t ga = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t gb = __builtin_amdgcn_make_buffer_rsrc((void*)Bs, 0, 0x7fffffff, 0x00020000);
#define PS_LOAD(l_)                                                                                                     \
    {                                                                                                                   \
        gs_u32x4* d_ = ring + istage * STAGE_V + min(wave + 4 * (l_), NINS - 1) * 64;                                   \
        if ((l_) < 3) __builtin_amdgcn_raw_ptr_buffer_load_lds(ga, (gs_lds_void*)d_, 16, a_lane[(l_) < 3 ? (l_) : 0], a_s, 0, 0);       \
        else if ((l_) < LD) __builtin_amdgcn_raw_ptr_buffer_load_lds(gb, (gs_lds_void*)d_, 16, b_lane[(l_) >= 3 && (l_) < LD ? (l_) - 3 : 0], b_s, 0, 0); \
    }
#else       // the host pass only needs the kernel's stub
#define PS_LOAD(l_) (void)0
#endif
    // scalar byte offsets of the step loaded next; then the one after it
#define PS_OFFSETS()                                                                                                    \
    const int a_s = (int)(((a.conv ? ((int64_t)(tap / tw) * a.geom.ppw + (tap % tw)) * a.lda : 0) + k0) * 6);            \
    const int b_s = (int)(((int64_t)tap * a.N * K + k0) * 6);
#define PS_ADVANCE()                                                                                                    \
    {                                                                                                                   \
        if (--left > 0) { if (++tap == a.taps) { tap = 0; k0 += 32; } }                                                 \
        istage = istage + 1 == NS ? 0 : istage + 1;                                                                     \
    }
#pragma unroll
    for (int d = 0; d < NS; ++d) {
        PS_OFFSETS();
#pragma unroll
        for (int l = 0; l < LD; ++l) PS_LOAD(l);
        PS_ADVANCE();
    }
    gm_f32x16 acc[TN][2];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][0][e] = acc[j][1][e] = 0.f;
    const int wk = wave & 1, wm = wave >> 1;
    const int arow = wm * 32 + fr, kc = 2 * wk + fh;
    const gs_u32x4* pA = ring + arow * 12 + (kc ^ ((arow >> 2) & 3));
    const gs_u32x4* pB = ring + (BM + fr) * 12 + (kc ^ ((fr >> 2) & 3));           // 32 rows further: the same swizzle
    gs_bf16x8 fa[2][3], fb[2][TN][3];
    // fragment read r of a step: pieces of A and of the columns, in the order in which the products need them
#define PS_READ(set_, st_, r_)                                                                                          \
    {                                                                                                                   \
        constexpr int g_ = (r_) / (TN + 1), i_ = (r_) % (TN + 1);                                                       \
        if constexpr (g_ < 3) {                                                                                         \
            if constexpr (i_ == 0) fa[set_][g_] = __builtin_bit_cast(gs_bf16x8, pA[(st_) * STAGE_V + g_ * 4]);          \
            else fb[set_][i_ > 0 ? i_ - 1 : 0][g_] = __builtin_bit_cast(gs_bf16x8, pB[(st_) * STAGE_V + (i_ > 0 ? i_ - 1 : 0) * 384 + g_ * 4]); \
        }                                                                                                               \
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * LD) : "memory");
    gs_for<3 * (TN + 1)>([&](auto r) { PS_READ(0, 0, decltype(r)::value); });
    int st = 0;
    auto step = [&](auto set_c) {
        constexpr int set = decltype(set_c)::value;
        const int nst = st + 1 == NS ? 0 : st + 1;
        // this step's fragments are all read (its stage is free), the next step has landed
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 2) * LD) : "memory");
        PS_OFFSETS();
        gs_for<6 * TN>([&](auto q_c) {
            constexpr int q = decltype(q_c)::value, p = q / TN, j = q % TN;
            constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
            acc[j][p > 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][pa[p]], fb[set][j][pb[p]], acc[j][p > 0], 0, 0, 0);
            PS_READ(set ^ 1, nst, q);
            if constexpr (q % 2 == 1) PS_LOAD(q / 2);
            __builtin_amdgcn_sched_barrier(0);
        });
        static_assert(LD <= 3 * TN, "a load behind every other MFMA");
        PS_ADVANCE();
        st = nst;
    };
#pragma unroll 1
    for (int s = 0; s + 2 <= steps; s += 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    if (steps & 1) step(std::integral_constant<int, 0>{});      // (inside the loop the compiler moved all accumulators twice a round)
#undef PS_READ
#undef PS_LOAD
#undef PS_OFFSETS
#undef PS_ADVANCE
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // element e of a lane: row 8 (e / 4) + 4 fh + e % 4, column fr of a 32 x 32 tile.  The two K groups of a wavefront tile share
    // its rows out: group wk finishes the elements 8 wk .. 8 wk + 7, a column tile at a time (a loop: unrolled over the column tiles
    // this was 25 KB of code that runs once a tile, 20 us of instruction fetches).
    float* part = reinterpret_cast<float*>(gs_smem) + wm * 2 * TN * 1024 + lane;
    auto at = [&](int g, int j, int e) -> float& { return part[((g * TN + j) * 16 + e) * 64]; };
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) at(wk, j, e) = acc[j][0][e] + acc[j][1][e];
    __syncthreads();
    const int row0 = wm * 32 + 16 * wk + 4 * fh;        // row of element e: row0 + 8 (e / 4) + e % 4
    auto sums = [&](int j, float (&v)[8]) {             // of column tile j
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = at(0, j, 8 * wk + e) + at(1, j, 8 * wk + e);
    };
    int64_t tok[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) tok[e] = s_tok[row0 + 8 * (e >> 2) + (e & 3)];
    // residual of the next column tile
    float rn[8];
    auto res_load = [&](int j) {
        const float* rp = (const float*)a.res + min(n0 + 32 * j + fr, ncols - 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) rn[e] = rp[max(tok[e], (int64_t)0) * a.ldr];
    };
    if (!GEGLU && a.res) res_load(0);
#pragma unroll 1
    for (int j = 0; j < (GEGLU ? TN / 2 : TN); ++j) {
        float v[8], gate[GEGLU ? 8 : 1], r[8];
        if (!GEGLU && a.res) {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = rn[e];
            if (j + 1 < TN) res_load(j + 1);
        }
        sums(j, v);
        if constexpr (GEGLU) sums(j + TN / 2, gate);
        const int col = n0 + 32 * j + fr;
        if (col >= ncols) break;
        const int pc = packed(col, 0);
        const float b0 = a.bias ? a.bias[pc] : 0.f, b1 = GEGLU && a.bias ? a.bias[pc + GEGLU_GROUP] : 0.f;
        const int sg = GEGLU ? 0 : col / a.seg_cols;
        const GemmSeg seg = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
        const int sc = col - sg * a.seg_cols;
        if constexpr (GEGLU) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (v[e] + b0) * gelu_f(gate[e] + b1);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += b0;
            if (a.rowbias || a.rowscale) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int own = a.row_owner[max(tok[e], (int64_t)0) / a.geom.S];
                    if (a.rowbias) v[e] += a.rowbias[(int64_t)own * a.N + col];
                    if (a.act_gelu) v[e] = gelu_tanh_f(v[e]);
                    if (a.rowscale) v[e] *= a.rowscale[(int64_t)own * a.rowscale_ld + col];
                }
            } else if (a.act_gelu) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = gelu_tanh_f(v[e]);
            }
            if (a.res) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += r[e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= seg.scale;
        }
        if (a.out_pieces) {
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                uint32_t u[3];
                cut3x2(v[e], v[e + 1], u);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (tok[e + q] < 0) continue;
                    uint16_t* op = (uint16_t*)seg.ptr + tok[e + q] * 3 * seg.ld + piece_index(sc);
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) op[32 * pl] = (uint16_t)(u[pl] >> 16 * q);
                }
            }
        } else {
            const int64_t rs = seg.transposed ? 1 : seg.ld;
            float* op = (float*)seg.ptr + (int64_t)sc * (seg.transposed ? seg.ld : 1);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tok[e] >= 0) op[tok[e] * rs] = v[e];
        }
    }
}

// Packed fp32 weights [rows][K] are followed, on the next 256-byte boundary, by their pieces (K a multiple of 32).
static size_t split_offset(int64_t rows, int K) { return (rows * K * sizeof(float) + 255) / 256 * 256; }
size_t packed_weight_bytes(int64_t rows, int32_t K, int dtype) {
    if (dtype == PSERVE_BF16) return (size_t)rows * K * 2;
    const bool pieces = K % 32 == 0 && rows * K * 6 < (int64_t)1 << 31;          // (as split_select: else nothing reads them)
    return pieces ? split_offset(rows, K) + (size_t)rows * 3 * K * 2 : (size_t)rows * K * 4;
}
__global__ void split_packed_kernel(const float* __restrict__ w, uint16_t* __restrict__ dst, int64_t rows, int32_t K) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * K) return;
    const int64_t r = i / K;
    uint32_t u[3];
    cut3x2(w[i], 0.f, u);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) dst[r * 3 * K + piece_index((int)(i - r * K)) + 32 * pl] = (uint16_t)u[pl];
}
int split_packed(void* packed, int64_t rows, int32_t K, int dtype, hipStream_t st) {
    if (packed_weight_bytes(rows, K, dtype) == dtype_size(dtype) * rows * K) return PSERVE_OK;
    split_packed_kernel<<<(unsigned)cdiv(rows * K, 256), 256, 0, st>>>((const float*)packed, (uint16_t*)((char*)packed + split_offset(rows, K)), rows, K);
    return check_launch("split_packed_kernel");
}

template <int TN, bool GEGLU>
static int launch_split(const GemmArgs& a, const uint16_t* Bs, hipStream_t st) {
    using Cfg = SplitCfg<TN>;
    PS_SET_LDS_ONCE((gemm_split_kernel<TN, GEGLU>), Cfg::LDS);
    const dim3 grid((unsigned)cdiv(a.M, Cfg::BM), (unsigned)cdiv(a.N, Cfg::BN));         // (GEGLU: a.N packed columns)
    gemm_split_kernel<TN, GEGLU><<<grid, 256, Cfg::LDS, st>>>(a, Bs);
    return check_launch("gemm_split_kernel");
}

// Column tiles of 32 the split kernel takes a problem with (whose A would come in pieces), 0: not at all.  The modelled times
// in us are within 15 % of what was measured at 576 .. 7,168 rows, 64 .. 320 columns, K = 64 .. 2,880: two tiles wide two blocks
// run on a CU (0.33 us a step alone, 0.65 together), five tiles wide one (0.62 us a step on an idle chip, 0.80 on a full one).
// Convolutions, fp32 kernel / two / five tiles wide: 7,168 x 320 162 / 100 / 78, 1,024 x 320 52 / 35 / 62, 2,304 x 256 50 / 30 / 53,
// 4,096 x 96 19.5 / 16.1 / 25, 576 x 128 14.3 / 17.7 / 30.  Three and four tiles wide were between or behind in all of them.
static int split_select(const GemmArgs& a) {
    if (a.K % 32 != 0 || a.lda != a.K || a.classes) return 0;
    if (gemm_a_rows(a) * a.lda * 6 >= (int64_t)1 << 31 || (int64_t)a.taps * a.N * a.K * 6 >= (int64_t)1 << 31) return 0;
    if (((uintptr_t)a.A | (uintptr_t)a.B) & 15) return 0;
    const bool geglu = a.epi == EPI_GEGLU;
    const int64_t steps = (int64_t)a.taps * (a.K / 32), mt = cdiv(a.M, 64), t2 = mt * cdiv(a.N, 64), t5 = mt * cdiv(a.N, 160);
    const int64_t r2 = t2 % 512, r5 = t5 % 256;
    const double c2 = t2 / 512 * (steps * 0.65 + 4.0) + (r2 == 0 ? 0.0 : r2 <= 256 ? steps * 0.33 + 6.0 : steps * 0.65 + 6.0);
    const double c5 = geglu || a.N % 160 != 0 ? 1e30 : t5 / 256 * (steps * 0.80 + 7.0) + (r5 == 0 ? 0.0 : steps * (0.62 + 0.18 * r5 / 256) + 7.0);
    int bm, bn;
    const double tiles = f32mma_tiles(a.M, geglu ? a.N / 2 : a.N, &bm, &bn) * (geglu ? 2 : 1);
    const double plain = 4.5 + tiles * a.taps * a.K * (tiles < 0.6 ? 0.0304 : 0.0224);
    return std::min(c2, c5) > 0.95 * plain ? 0 : c5 < c2 ? 5 : 2;
}
bool gemm_takes_pieces(const GemmArgs& a, int dtype, int mode) { return dtype == PSERVE_F32 && mode == 0 && split_select(a) != 0; }

static int gemm_split(const GemmArgs& a, hipStream_t st) {
    const uint16_t* Bs = (const uint16_t*)((const char*)a.B + split_offset((int64_t)a.taps * a.N, a.K));
    const int tn = split_select(a);
    PS_REQUIRE(tn, "gemm: activations in pieces for a layer that does not take them");
    if (a.epi == EPI_GEGLU) return launch_split<2, true>(a, Bs, st);
    return tn == 5 ? launch_split<5, false>(a, Bs, st) : launch_split<2, false>(a, Bs, st);
}

// For tests (host only, no part of the ABI): what split_select says of an fp32 layer of M rows (taps = 9: a 3x3 convolution).
extern "C" int pserve_test_split_tiles(int32_t M, int32_t N, int32_t K, int32_t taps, int32_t geglu) {
    GemmArgs a{};
    a.M = M; a.N = N; a.K = a.lda = K; a.taps = taps; a.epi = geglu ? EPI_GEGLU : EPI_ROUTE;
    return split_select(a);
}

// ---- packing kernels -----------------------------------------------------------------------------------
template <typename T>
__global__ void pack_conv_kernel(const T* __restrict__ w, T* __restrict__ dst, int32_t Cout, int32_t Cin) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;       // over dst [9][Cout][Cin]
    if (i >= (int64_t)9 * Cout * Cin) return;
    const int ci = (int)(i % Cin);
    const int co = (int)((i / Cin) % Cout);
    const int tap = (int)(i / ((int64_t)Cin * Cout));
    dst[i] = w[((int64_t)co * Cin + ci) * 9 + tap];
}

// four parity classes x four taps of the nearest-up convolution (see pack_conv_up2 in kernels.h)
template <typename T>
__global__ void pack_conv_up2_kernel(const T* __restrict__ w, T* __restrict__ dst, int32_t Cout, int32_t Cin) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;       // over dst [4][4][Cout][Cin]
    if (i >= (int64_t)16 * Cout * Cin) return;
    const int ci = (int)(i % Cin);
    const int co = (int)((i / Cin) % Cout);
    const int t = (int)(i / ((int64_t)Cin * Cout));
    const int cls = t >> 2, a = cls >> 1, b = cls & 1, j = (t >> 1) & 1, ii = t & 1;
    // 3x3 rows merged into 2x2 row j: a = 0: {0}, {1, 2};  a = 1: {0, 1}, {2}
    const int y0 = a == 0 ? (j == 0 ? 0 : 1) : (j == 0 ? 0 : 2), y1 = a == 0 ? (j == 0 ? 0 : 2) : (j == 0 ? 1 : 2);
    const int x0 = b == 0 ? (ii == 0 ? 0 : 1) : (ii == 0 ? 0 : 2), x1 = b == 0 ? (ii == 0 ? 0 : 2) : (ii == 0 ? 1 : 2);
    float acc = 0.f;
    for (int ty = y0; ty <= y1; ++ty)
        for (int tx = x0; tx <= x1; ++tx) acc += ld_f<T>(w + ((int64_t)co * Cin + ci) * 9 + ty * 3 + tx);
    st_f<T>(dst + i, acc);
}

// dst row (row0 + perm(n)) = column n of w[K][Ncols]; geglu_F > 0 applies the value/gate interleave
template <typename T>
__global__ void pack_linear_kernel(const T* __restrict__ w, T* __restrict__ dst, int32_t K, int32_t Ncols, int32_t row0,
                                   int32_t geglu_F) {
    __shared__ T tile[32][33];
    const int k0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;      // 256 threads: ty 0..7
    for (int r = ty; r < 32; r += 8)
        if (k0 + r < K && n0 + tx < Ncols) tile[r][tx] = w[(int64_t)(k0 + r) * Ncols + n0 + tx];
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int n = n0 + r, k = k0 + tx;
        if (n < Ncols && k < K) {
            int row = n;
            if (geglu_F > 0) {
                const int half = n >= geglu_F, c = half ? n - geglu_F : n;
                row = (c / GEGLU_GROUP) * 2 * GEGLU_GROUP + half * GEGLU_GROUP + c % GEGLU_GROUP;
            }
            dst[(int64_t)(row0 + row) * K + k] = tile[tx][r];
        }
    }
}

template <typename T>
__global__ void pack_bias_kernel(const T* __restrict__ b, float* __restrict__ dst, int32_t N, int32_t geglu_F) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    int row = n;
    if (geglu_F > 0) {
        const int half = n >= geglu_F, c = half ? n - geglu_F : n;
        row = (c / GEGLU_GROUP) * 2 * GEGLU_GROUP + half * GEGLU_GROUP + c % GEGLU_GROUP;
    }
    dst[row] = ld_f<T>(b + n);
}

int pack_conv(const void* w, void* dst, int32_t Cout, int32_t Cin, int dtype, hipStream_t st) {
    const int64_t total = (int64_t)9 * Cout * Cin;
    const unsigned grid = (unsigned)cdiv(total, 256);
    if (dtype == PSERVE_BF16) pack_conv_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)w, (uint16_t*)dst, Cout, Cin);
    else pack_conv_kernel<float><<<grid, 256, 0, st>>>((const float*)w, (float*)dst, Cout, Cin);
    return check_launch("pack_conv_kernel");
}

int pack_conv_up2(const void* w, void* dst, int32_t Cout, int32_t Cin, int dtype, hipStream_t st) {
    const unsigned grid = (unsigned)cdiv((int64_t)16 * Cout * Cin, 256);
    if (dtype == PSERVE_BF16) pack_conv_up2_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)w, (uint16_t*)dst, Cout, Cin);
    else pack_conv_up2_kernel<float><<<grid, 256, 0, st>>>((const float*)w, (float*)dst, Cout, Cin);
    return check_launch("pack_conv_up2_kernel");
}

static int pack_linear_impl(const void* w, void* dst, int32_t K, int32_t Ncols, int32_t row0, int32_t gF, int dtype,
                            hipStream_t st) {
    dim3 grid((unsigned)cdiv(K, 32), (unsigned)cdiv(Ncols, 32));
    if (dtype == PSERVE_BF16)
        pack_linear_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)w, (uint16_t*)dst, K, Ncols, row0, gF);
    else
        pack_linear_kernel<float><<<grid, 256, 0, st>>>((const float*)w, (float*)dst, K, Ncols, row0, gF);
    return check_launch("pack_linear_kernel");
}

int pack_linear(const void* w, void* dst, int32_t K, int32_t Ncols, int32_t row0, int dtype, hipStream_t st) {
    return pack_linear_impl(w, dst, K, Ncols, row0, 0, dtype, st);
}

static int pack_bias_impl(const void* b, float* dst, int32_t N, int32_t gF, int dtype, hipStream_t st) {
    const unsigned grid = (unsigned)cdiv(N, 256);
    if (dtype == PSERVE_BF16) pack_bias_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)b, dst, N, gF);
    else pack_bias_kernel<float><<<grid, 256, 0, st>>>((const float*)b, dst, N, gF);
    return check_launch("pack_bias_kernel");
}

int pack_bias(const void* b, float* dst, int32_t N, int dtype, hipStream_t st) { return pack_bias_impl(b, dst, N, 0, dtype, st); }

int pack_geglu(const void* w1, const void* b1, void* dst, float* bias_dst, int32_t K, int32_t F, int dtype, hipStream_t st) {
    PS_REQUIRE(F % GEGLU_GROUP == 0, "FFN: hidden width %d must be a multiple of %d", F, GEGLU_GROUP);
    PS_TRY(pack_linear_impl(w1, dst, K, 2 * F, 0, F, dtype, st));
    return pack_bias_impl(b1, bias_dst, 2 * F, F, dtype, st);
}

// ---- dispatch -------------------------------------------------------------------------------------------
int gemm_mfma_bf16(const GemmArgs& a, hipStream_t st, bool* handled);     // gemm_mfma.hip

bool gemm_few_f32(const GemmArgs& a, hipStream_t st);       // gemm_few.hip
int gemm(const GemmArgs& a, int dtype, int mode, hipStream_t st) {
    PS_REQUIRE(a.M > 0 && a.N > 0 && a.K > 0, "gemm: empty problem");
    if (a.a_pieces) return gemm_split(a, st);
    if (mode == 0 && dtype == PSERVE_BF16) {
        bool handled = false;
        PS_TRY(gemm_mfma_bf16(a, st, &handled));
        if (handled) return PSERVE_OK;
    }
    PS_REQUIRE(!a.B2, "gemm: no kernel takes the second problem of this shape");
    if (a.classes) {                                    // the kernels below take one class at a time
        for (int c = 0; c < a.classes; ++c) {
            GemmArgs g = a;
            g.classes = 0;
            g.a_dy = g.o_dy = c >> 1;
            g.a_dx = g.o_dx = c & 1;
            g.B = (const char*)a.B + (size_t)c * a.taps * a.N * a.K * dtype_size(dtype);
            PS_TRY(gemm(g, dtype, mode, st));
        }
        return PSERVE_OK;
    }
    if (mode == 0 && dtype == PSERVE_F32 && gemm_few_f32(a, st)) return check_launch("gemm_few_kernel");
    if (mode == 0 && (dtype == PSERVE_BF16 ? gemm_f32mma<uint16_t>(a, st) : gemm_f32mma<float>(a, st)))
        return check_launch("gemm_f32mma_kernel");
    const bool geglu = a.epi == EPI_GEGLU;
    const int ncols = geglu ? a.N / 2 : a.N;
    dim3 grid((unsigned)cdiv(a.M, 64), (unsigned)cdiv(ncols, 64));
    if (dtype == PSERVE_BF16) {
        if (geglu) gemm_simple_kernel<uint16_t, true><<<grid, 256, 0, st>>>(a);
        else gemm_simple_kernel<uint16_t, false><<<grid, 256, 0, st>>>(a);
    } else {
        if (geglu) gemm_simple_kernel<float, true><<<grid, 256, 0, st>>>(a);
        else gemm_simple_kernel<float, false><<<grid, 256, 0, st>>>(a);
    }
    return check_launch("gemm_simple_kernel");
}

}  // namespace pserve
