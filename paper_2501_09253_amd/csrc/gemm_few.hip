// bf16 GEMM / implicit-GEMM convolution of few tiles for gfx950: linear layers and convolutions whose 128-row tiles would leave
// much of the chip idle, so that one round of small tiles does (few_pick).
//
// Such a launch is a chain: a block walks its K steps one behind the other, and the time of a step is what a CU fetches into
// LDS (90 GB/s a CU, whatever the number of CUs) or the latency of a load, not the matrix cores.  So the tiles are small (more
// CUs fetch), and the wavefronts of a block share K and not the tile: wavefront w computes the whole tile over the 64-wide K
// steps w, w + 4, ... from a ring of two steps of its own.  Nothing in the loop waits for another wavefront (no barrier, only
// the count of the own loads), eight steps are in flight, and a fragment read from LDS is read once.  The partial sums meet in
// LDS at the end, where each thread finishes eight outputs with whatever bias and residual it asked for at the start.
// us of one launch, 128 x 64 (GEGLU: 256 x 128) tiles / here: 216 x 128, K = 1,152 10.7 / 5.3; 1,024 x 640, K = 640 8.7 / 6.5,
// K = 5,120 30.2 / 17.2; 1,024 x 1,280, K = 1,280 12.4 / 11.2, K = 5,120 31.7 / 23.8; 231 text rows x 640, K = 2,048 16.6 / 7.0;
// 464 x 1,920 value-gate pairs, K = 960 19.5 / 7.7; 3x3 convolutions against tiles shared between blocks: 1,024 x 320 23.9 / 9.9,
// 4,096 x 320 34.5 / 15.5, 1,024 x 640 31.4 / 18.9.
// Tried: fragments loaded straight into registers, no LDS (twice the time: 64-byte pieces of 16 rows a load); rings of three and
// four steps, eight wavefronts (no gain in one round, and one block a CU instead of two); two rounds (no gain but for GEGLU).
#include "mfma_util.h"
#include <type_traits>

namespace pserve {

// Block tile BM x BN, W wavefronts.  Partial tiles: rows of RED_LD floats, 16-byte chunk c of row r at c ^ ((r >> 3) & 7), so that
// both ways of reading them (eight columns of a row, eight rows of a column) spread over the banks.
template <int BM, int BN, int W> struct FewCfg {
    static constexpr int STAGE = (BM + BN) * 128;                   // bytes of one K step of the tile
    static constexpr int RED_LD = (BN + 31) / 32 * 32 + 4;          // floats per row of a partial tile
    static constexpr int PART = 2 * STAGE;                          // bytes of a wavefront's ring, later its partial tile
    static constexpr size_t LDS = (size_t)W * PART + 3 * BM * sizeof(int32_t);
    static_assert(LDS <= 160 * 1024 && BM * RED_LD * 4 <= PART, "LDS");
};

// TWO: a second problem (GemmArgs::B2: another patch list, weights, bias and gate of its own) continues the row tiles of the first.
// HALO: a convolution that reads the unpadded batch (GemmArgs::halo_src), its A rows' offsets in a table of taps x BM.
// F32: fp32 operands and outputs.  A K step is then 32 wide (the same 128 bytes a row), and a lane's 16-byte chunks, four k of a row,
// feed four MFMAs of 16 x 16 x 4; no GELU and no transposed segments.
enum : int { FEW_TWO = 1, FEW_HALO = 2 };
template <int BM, int BN, int W, bool GEGLU, int FORM, bool F32 = false>
__global__ void __launch_bounds__(64 * W)
gemm_few_kernel(std::conditional_t<FORM != 0, GemmArgs, GemmCore> a, int pads, int m_first) {
    constexpr bool TWO = FORM == FEW_TWO, HALO = FORM == FEW_HALO;
    constexpr int ES = F32 ? 4 : 2, KW = 128 / ES;                              // bytes of a value, K of a step
    static_assert(!F32 || (!GEGLU && FORM == 0 && BM == 16 && BN == 16), "fp32 form");
    using Cfg = FewCfg<BM, BN, W>;
    constexpr int TM = BM / 16, TN = BN / 16, AL = BM / 8, BL = BN / 8, LD = AL + BL;
    static_assert(!GEGLU || BN == 64, "a tile of value-gate pairs is 32 values and their 32 gates");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int32_t* s_tok = reinterpret_cast<int32_t*>(smem + W * Cfg::PART);          // [BM] output row, -1: none
    int32_t* s_off = s_tok + BM;                                                // [BM] byte offset of the A row
    int32_t* s_own = s_off + BM;                                                // [BM] request slot (rowbias / rowscale)
    int32_t* s_src = s_own + BM;                                                // HALO: [taps][BM]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Tiles: XCD x (block id mod 8) takes the x-th eighth of the tile numbers, rows or columns fastest (m_first), so that its L2
    // fetches an eighth of the larger operand.
    const bool masked = a.tokens_are_rows && a.act.active;
    // (the counts decide which tile a block has and so what its loads' scalar offsets and descriptors are: scalars)
    const int act_count = masked ? __builtin_amdgcn_readfirstlane(*a.act.count) : 0;
    int m_limit = masked ? act_count * a.geom.S : pads ? a.M / a.row_group * a.row_group_pad : a.M;
    const int mt1 = (m_limit + BM - 1) / BM;
    int m_tiles = mt1, m_limit2 = 0;
    if constexpr (TWO) {
        m_limit2 = __builtin_amdgcn_readfirstlane(*a.act2.count) * a.geom.S;
        m_tiles += (m_limit2 + BM - 1) / BM;
    }
    const int n_in = a.N / BN, n_tiles = n_in * (a.classes ? a.classes : 1);
    const int total = n_tiles * m_tiles, xcd = blockIdx.x & 7;
    const int t = (int)((int64_t)total * xcd / 8) + (int)(blockIdx.x >> 3);
    if (t >= (int)((int64_t)total * (xcd + 1) / 8)) return;
    const int mt = m_first ? t % m_tiles : t / n_tiles, nt = m_first ? t / m_tiles : t - (t / n_tiles) * n_tiles;
    const int cls = a.classes ? nt / n_in : 0;
    const int ntile = nt - cls * n_in;
    int m0 = mt * BM;
    // what differs between the problems (locals: writing to the arguments would move all of them to memory)
    const void* B = a.B;
    const float *bias_v = a.bias, *rowscale = a.rowscale;
    const int32_t* active = a.act.active;
    if constexpr (TWO) {
        if (mt >= mt1) {
            m0 -= mt1 * BM;
            m_limit = m_limit2;
            B = a.B2; bias_v = a.bias2; rowscale = a.rowscale2; active = a.act2.active;
        }
    }
    // packed column of column c of the tile (value-gate pairs: 32 values, then their gates, 64 further in groups of 128)
    auto bcol = [&](int c) { return GEGLU ? (ntile >> 1) * (2 * GEGLU_GROUP) + (ntile & 1) * 32 + (c >> 5) * GEGLU_GROUP + (c & 31) : ntile * BN + c; };

    const int kchunks = a.K / KW, KT = a.taps * kchunks;
    const int mine = wave < KT ? (KT - wave + W - 1) / W : 0;       // K steps of this wavefront
    const int tap_w = a.tap_w ? a.tap_w : 3;
    const int fr = lane & 15, kq = lane >> 4;                       // fragment row / column, quarter of a 32-wide K piece
#if defined(__HIP_DEVICE_COMPILE__)
    int a_bytes = 0x7fffffff;
    if constexpr (HALO) a_bytes = halo_bytes(a);
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, 0x7fffffff, 0x00020000);
#define PS_LOAD(rsrc_, dst_, lane_off_, off_) \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_, (lds_void*)(dst_), 16, lane_off_, off_, 0, 0)
#else       // the host pass only needs the kernel's stub
#define PS_LOAD(rsrc_, dst_, lane_off_, off_) (void)0
#endif
    // (tap, chunk) of a K step: a wavefront's next one is W chunks further
    auto advance = [&](int& tap, int& kc) { for (kc += W; kc >= kchunks; kc -= kchunks) ++tap; };
    int tap0 = 0, kc0 = wave;
    for (; kc0 >= kchunks; kc0 -= kchunks) ++tap0;
    auto b_base = [&](int tap, int kc) { return (int)(((int64_t)(cls * a.taps + tap) * a.N * a.K + kc * KW) * ES); };
    auto a_base = [&](int tap, int kc) {
        const int ty = tap == 0 ? 0 : tap / tap_w, tx = tap - ty * tap_w;
        return (int)(((a.conv && !HALO ? (int64_t)(ty * a.geom.ppw + tx) * a.lda : 0) + kc * KW) * ES);
    };

    // staging: lane -> (row lane / 8 of a load's eight, 16-byte position lane % 8); chunk c of row r at c ^ ((r >> 1) & 7)
    const int lrow = lane >> 3, lc = lane & 7, sw = lane >> 4;
    const int gc0 = (lc ^ sw) * 16, gc1 = (lc ^ (sw + 4)) * 16;     // byte offset of the chunk, even / odd load
    typedef __attribute__((address_space(3))) uint8_t lds_u8;
    lds_u8* ring = (lds_u8*)(smem + wave * Cfg::PART);
    const int b_lane0 = lrow * a.K * ES + gc0, b_lane1 = lrow * a.K * ES + gc1;
    auto load_b = [&](int tap, int kc, int st) {
        const int base = b_base(tap, kc);
#pragma unroll
        for (int i = 0; i < BL; ++i)
            PS_LOAD(b_rsrc, ring + st * Cfg::STAGE + BM * 128 + i * 1024, i & 1 ? b_lane1 : b_lane0, base + bcol(8 * i) * a.K * ES);
    };
    int tap1 = tap0, kc1 = kc0;
    constexpr int NSRC = HALO ? (9 * BM + 64 * W - 1) / (64 * W) : 1;
    int src[NSRC];
    if constexpr (HALO) {           // (asked for first: a wait for a load waits for all before it)
        const int tok = min(m0 + tid % BM, m_limit - 1);
        const int p = tok / a.geom.S, q = tok - p * a.geom.S, y = q / a.geom.pw, x = q - y * a.geom.pw, am = a.a_mul ? a.a_mul : 1;
#pragma unroll
        for (int u = 0; u < NSRC; ++u) {
            const int k = tid / BM + u * (64 * W / BM);
            if (k < a.taps) src[u] = halo_token(a, p, am * y + (cls >> 1) + k / tap_w, am * x + (cls & 1) + k % tap_w);
        }
        asm volatile("" ::: "memory");
    }
    // the weights need no table: they travel while it is built
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (s < mine) load_b(tap1, kc1, s);
        advance(tap1, kc1);
    }
    if (tid < BM) {
        int tok = m0 + tid;
        bool valid = tok < m_limit;
        if (masked) {
            const int pi = tok / a.geom.S;
            tok = valid ? active[pi] * a.geom.S + (tok - pi * a.geom.S) : 0;
        } else {
            if (pads && valid) {
                const int g = tok / a.row_group_pad, j = tok - g * a.row_group_pad;
                valid = j < a.row_group;
                tok = g * a.row_group + j;
            }
            if (!valid) tok = 0;
        }
        int orow = tok;
        int64_t off;
        if (a.conv) {
            const int p = tok / a.geom.S, q = tok - p * a.geom.S, y = q / a.geom.pw, x = q - y * a.geom.pw;
            const int am = a.a_mul ? a.a_mul : 1;
            const int ady = a.classes ? cls >> 1 : a.a_dy, adx = a.classes ? cls & 1 : a.a_dx;
            off = ((int64_t)p * a.geom.pS + (am * y + ady) * a.geom.ppw + am * x + adx) * a.lda;
            if (a.o_mul) {
                const int ody = a.classes ? cls >> 1 : a.o_dy, odx = a.classes ? cls & 1 : a.o_dx;
                orow = p * a.o_S + (a.o_mul * y + ody) * a.o_pw + a.o_mul * x + odx;
            }
        } else {
            off = (int64_t)tok * a.lda;
        }
        if (!a.tokens_are_rows && a.row_group > 0) orow = tok / a.row_group * a.row_group_pad + tok % a.row_group;
        s_tok[tid] = valid ? orow : -1;
        s_off[tid] = (int)(off * ES);
        if (a.rowbias || rowscale) s_own[tid] = a.row_owner[tok / a.geom.S];
    }
    if constexpr (HALO) {
#pragma unroll
        for (int u = 0; u < NSRC; ++u) {
            const int k = tid / BM + u * (64 * W / BM);
            if (k < a.taps) s_src[k * BM + tid % BM] = halo_offset(a, src[u]);
        }
    }
    // the table is written; the loads stay in flight (__syncthreads() would wait for them)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    const int pcol0 = bcol(0), sg = GEGLU ? 0 : pcol0 / a.seg_cols;
    const GemmSeg seg = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
    const int ocol0 = GEGLU ? ntile * 32 : pcol0 - sg * a.seg_cols;
    const bool tr = !GEGLU && !F32 && seg.transposed;
    // what the end of the tile needs of memory, asked for in front of the activations
    constexpr int CV = (GEGLU ? 32 : BN) / 8, ITEMS = BM * CV, NIT = (ITEMS + 64 * W - 1) / (64 * W);
    u32x4 res[NIT][F32 ? 2 : 1];
    float bias[NIT][GEGLU ? 16 : 8];
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
        const int it = tid + u * (64 * W);
#pragma unroll
        for (int q = 0; q < (F32 ? 2 : 1); ++q) res[u][q] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < (GEGLU ? 16 : 8); ++q) bias[u][q] = 0.f;
        if (it >= ITEMS) continue;
        if (tr) {
            if (bias_v) bias[u][0] = bias_v[pcol0 + it / (BM / 8)];
            continue;
        }
        const int row = it / CV, ch = it % CV * 8, tok = s_tok[row];
        if (bias_v) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                bias[u][q] = bias_v[pcol0 + ch + q];
                if (GEGLU) bias[u][8 + q] = bias_v[pcol0 + GEGLU_GROUP + ch + q];
            }
        }
        if (!GEGLU && a.res && tok >= 0) {
#pragma unroll
            for (int q = 0; q < (F32 ? 2 : 1); ++q)
                res[u][q] = *reinterpret_cast<const u32x4*>((const uint8_t*)a.res + ((int64_t)tok * a.ldr + pcol0 + ch) * ES + 16 * q);
        }
    }
    asm volatile("" ::: "memory");                                  // (no load sinks below the next ones)

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int a_lane[AL];
#pragma unroll
    for (int i = 0; i < AL; ++i) a_lane[i] = s_off[8 * i + lrow] + (i & 1 ? gc1 : gc0);
    auto load_a = [&](int tap, int kc, int st) {
        const int base = a_base(tap, kc);
        if constexpr (HALO) {
#pragma unroll
            for (int i = 0; i < AL; ++i) a_lane[i] = s_src[tap * BM + 8 * i + lrow] + (i & 1 ? gc1 : gc0);
        }
#pragma unroll
        for (int i = 0; i < AL; ++i) PS_LOAD(a_rsrc, ring + st * Cfg::STAGE + i * 1024, a_lane[i], base);
    };
    {
        int tap = tap0, kc = kc0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (s < mine) load_a(tap, kc, s);
            advance(tap, kc);
        }
    }
    f32x4 sum[F32 ? 8 : 1];                 // fp32: eight sums of an eighth of the products each, so that rounding does not grow with K
#pragma unroll
    for (int e = 0; e < (F32 ? 8 : 1); ++e) sum[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int fsw = (fr >> 1) & 7;
    for (int s = 0; s < mine; ++s) {
        // the own loads of step s have landed (in flight behind them: those of step s + 1, at first only its A rows)
        if (s + 1 >= mine) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (s == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AL) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LD) : "memory");
        typedef const __attribute__((address_space(3))) u32x4* frag_ptr;
        const lds_u8* st = ring + (s & 1) * Cfg::STAGE;
        typedef std::conditional_t<F32, f32x4, bf16x8> Frag;
        Frag fa[2][TM], fb[2][TN];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int pos = ((4 * h + kq) ^ fsw) * 16;
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[h][i] = __builtin_bit_cast(Frag, *(frag_ptr)(st + (i * 16 + fr) * 128 + pos));
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[h][j] = __builtin_bit_cast(Frag, *(frag_ptr)(st + (BM + j * 16 + fr) * 128 + pos));
        }
        if (s + 2 < mine) {                                        // all fragments are read: the stage is free
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            load_b(tap1, kc1, s & 1);
            load_a(tap1, kc1, s & 1);
            advance(tap1, kc1);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (F32) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[4 * h + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[h][i][e], fb[h][j][e], sum[4 * h + e], 0, 0, 0);
                    } else {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
                    }
                }
    }
#undef PS_LOAD
    if constexpr (F32) acc[0][0] = ((sum[0] + sum[1]) + (sum[2] + sum[3])) + ((sum[4] + sum[5]) + (sum[6] + sum[7]));

    // ---- partial sums, each in its wavefront's own ring (nobody else reads that before the barrier)
    float* red = reinterpret_cast<float*>(smem);
    constexpr int PART = Cfg::PART / 4, RLD = Cfg::RED_LD;
    if (mine > 0) {
        float* own = red + wave * PART + (fr & 3);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    own[(16 * i + 4 * kq + e) * RLD + (((4 * j + (fr >> 2)) ^ ((2 * i + (kq >> 1)) & 7)) << 2)] = acc[i][j][e];
    }
    __syncthreads();
    const int parts = min(W, KT);
    uint16_t* out = (uint16_t*)seg.ptr;
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
        const int it = tid + u * (64 * W);
        if (it >= ITEMS) break;
        if (tr) {                                                   // one column, eight rows: out[col][token]
            const int c = it / (BM / 8), r0 = it % (BM / 8) * 8;
            const float* src = red + r0 * RLD + (((c >> 2) ^ ((r0 >> 3) & 7)) << 2) + (c & 3);
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = bias[u][0];
            for (int w = 0; w < parts; ++w)
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] += src[w * PART + q * RLD];
            const int t0 = s_tok[r0], t3 = s_tok[r0 + 3], t4 = s_tok[r0 + 4], t7 = s_tok[r0 + 7];
            uint16_t* dst = out + (int64_t)(ocol0 + c) * seg.ld;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (a.rowbias) v[q] += a.rowbias[(int64_t)s_own[r0 + q] * a.N + pcol0 + c];
                if (a.act_gelu) v[q] = gelu_tanh(v[q]);
                if (rowscale) v[q] *= rowscale[(int64_t)s_own[r0 + q] * a.rowscale_ld + pcol0 + c];
                v[q] *= seg.scale;
            }
            if (t0 >= 0 && t7 == t0 + 7 && t3 == t0 + 3 && t4 == t0 + 4 && (t0 & 7) == 0 && (seg.ld & 7) == 0) {
                *reinterpret_cast<u32x4*>(dst + t0) = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                            pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int tk = s_tok[r0 + q];
                    if (tk >= 0) dst[tk] = float_to_bf16_bits(v[q]);
                }
            }
            continue;
        }
        const int row = it / CV, ch = it % CV * 8, tok = s_tok[row], rsw = (row >> 3) & 7;
        if (tok < 0) continue;
        float v[8], g[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[q] = bias[u][q];
            if (GEGLU) g[q] = bias[u][(GEGLU ? 8 : 0) + q];
        }
        const float* src = red + row * RLD;
        for (int w = 0; w < parts; ++w) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(src + w * PART + ((((ch >> 2) + h) ^ rsw) << 2));
#pragma unroll
                for (int q = 0; q < 4; ++q) v[4 * h + q] += x[q];
                if (GEGLU) {
                    const f32x4 y = *reinterpret_cast<const f32x4*>(src + w * PART + ((((ch >> 2) + 8 + h) ^ rsw) << 2));
#pragma unroll
                    for (int q = 0; q < 4; ++q) g[4 * h + q] += y[q];
                }
            }
        }
        if (GEGLU) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] *= gelu_erf(g[q]);
        } else {
            if (a.rowbias) {
                const float* rb_ = a.rowbias + (int64_t)s_own[row] * a.N + pcol0 + ch;
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] += rb_[q];
            }
            if (a.act_gelu) {
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = gelu_tanh(v[q]);
            }
            if (rowscale) {
                const float* rs = rowscale + (int64_t)s_own[row] * a.rowscale_ld + pcol0 + ch;
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] *= rs[q];
            }
            if (a.res) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (F32) {
                        v[q] += __uint_as_float(res[u][0][q]);
                        v[4 + q] += __uint_as_float(res[u][1][q]);
                    } else {
                        v[2 * q] += __uint_as_float(res[u][0][q] << 16);
                        v[2 * q + 1] += __uint_as_float(res[u][0][q] & 0xFFFF0000u);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] *= seg.scale;
        }
        if constexpr (F32) {
            f32x4* dst = reinterpret_cast<f32x4*>((float*)seg.ptr + (int64_t)tok * seg.ld + ocol0 + ch);
            dst[0] = f32x4{v[0], v[1], v[2], v[3]};
            dst[1] = f32x4{v[4], v[5], v[6], v[7]};
            continue;
        }
        *reinterpret_cast<u32x4*>(out + (int64_t)tok * seg.ld + ocol0 + ch) =
            u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
    }
}

static int64_t few_tiles(const GemmArgs& a, int bm, int bn) {
    return (cdiv(gemm_rows(a), bm) + (a.B2 ? cdiv(a.M2, bm) : 0)) * (a.N / bn) * std::max(1, a.classes);
}
template <int BM, int BN, bool GEGLU, int FORM>
static int launch_few_as(const GemmArgs& a, hipStream_t st) {
    constexpr int W = 4;
    constexpr size_t lds = FewCfg<BM, BN, W>::LDS + (FORM == FEW_HALO ? 9 * BM * sizeof(int32_t) : 0);
    PS_SET_LDS_ONCE((gemm_few_kernel<BM, BN, W, GEGLU, FORM>), lds);
    const bool pads = gemm_pads_rows(a);
    const int m_first = (int64_t)a.M <= (int64_t)a.N * a.taps * std::max(1, a.classes);
    gemm_few_kernel<BM, BN, W, GEGLU, FORM><<<(unsigned)(8 * cdiv(few_tiles(a, BM, BN), 8)), 64 * W, lds, st>>>(a, pads, m_first);
    return check_launch("gemm_few_kernel");
}
template <int BM, int BN, bool GEGLU>
static int launch_few(const GemmArgs& a, hipStream_t st) {
    if constexpr (!GEGLU) {
        if (a.B2) return launch_few_as<BM, BN, GEGLU, FEW_TWO>(a, st);
        if (a.halo_src) return launch_few_as<BM, BN, GEGLU, FEW_HALO>(a, st);
    }
    return launch_few_as<BM, BN, GEGLU, 0>(a, st);
}

// Which tile a problem would take here (0: none) and how long it would run, in us: a round of 256 tiles (32 x 32: 512, two
// blocks a CU, each then slower) is a fixed time, of which 4 are launch, tables and end, and a time per K step, fitted to 160
// measured sizes (within 10 %).  Linear layers and convolutions that conv_mfma_kernel takes too only where it is one round: with two, the 128-row tiles win (1,280 x
// 1,280, K = 1,280 13.4 against 17.7; RES2 of 4,096 x 512 93 against 102, 4,608 x 320 64.5 against 66.7); value-gate pairs with two (768 x 2,560, K = 960
// 12.9 against 19.9, K = 320 8.9 against 12.2; three rounds 18.0 against 20.2 and 12.5 against 12.4).
static const struct { int bm, bn; double fixed, step; } FEW[] = {{0, 0, 0, 0},        {32, 32, 4.0, 0.083}, {32, 64, 4.4, 0.125},
                                                                 {32, 80, 5.0, 0.145}, {64, 64, 4.9, 0.18},  {64, 80, 5.8, 0.205}};
int few_pick(const GemmArgs& a, int most_rounds, double* us) {
    const bool geglu = a.epi == EPI_GEGLU;
    int best = 0;
    *us = 1e30;
    if (geglu && a.N % 128 != 0) return 0;
    if (a.B2 && !gemm_two_eligible(a)) return 0;
    for (int v = 1; v <= 5; ++v) {
        const int bm = FEW[v].bm, bn = FEW[v].bn;
        if (geglu ? bn != 64 : a.N % bn != 0 || a.seg_cols % bn != 0) continue;
        const int64_t tiles = few_tiles(a, bm, bn);
        const int64_t steps = (int64_t)a.taps * (a.K / 64), rounds = cdiv(tiles, 256);
        if (v == 1 ? tiles > 512 : rounds > most_rounds) continue;
        double t = v == 1 && tiles > 256 ? 4.3 + 0.17 * steps : rounds * (FEW[v].fixed + FEW[v].step * steps);
        if (geglu) t = rounds * (3.4 + 0.2 * steps);
        if (t < *us) { *us = t; best = v; }
    }
    return best;
}

int gemm_few_bf16(const GemmArgs& a, int tile, hipStream_t st) {
    if (a.epi == EPI_GEGLU) return tile == 2 ? launch_few<32, 64, true>(a, st) : launch_few<64, 64, true>(a, st);
    switch (tile) {
    case 1: return launch_few<32, 32, false>(a, st);
    case 2: return launch_few<32, 64, false>(a, st);
    case 3: return launch_few<32, 80, false>(a, st);
    case 4: return launch_few<64, 64, false>(a, st);
    default: return launch_few<64, 80, false>(a, st);
    }
}

// fp32 (false: not for this kernel): up to 1,024 tiles of 16 x 16, four blocks a CU.  gemm_f32mma_kernel's smallest tile, 32 x 32, is four
// wavefronts that each walk all of K at 32 clocks per four k; here they share it, on four times the blocks.  us, 32 x 32 / here:
// convolutions 832 x 64 10.0 / 5.7, 576 x 96 14.5 / 6.1, 576 x 192 19.5 / 10.4, 1,152 x 160 19.1 / 11.4, 576 x 320 30.6 / 17.8, 1,728 x 128
// (864 tiles) 15.3 / 12.6; linear layers 144 x 256, K = 1,024 12.4 / 5.8, 576 x 320, K = 320 7.8 / 5.6, 576 x 96, K = 96 4.8 / 4.1, but 576 x 384,
// K = 128 (864 tiles) 5.6 / 5.9 and K = 64 alike (a launch's 4 us).  Pieces, where gemm_takes_pieces says so, come first.
bool gemm_few_f32(const GemmArgs& a, hipStream_t st) {
    const int64_t tiles = cdiv(a.M, 16) * (a.N / 16) * std::max(1, a.classes), k = (int64_t)a.taps * a.K;
    if (tiles > 1024 || k < (tiles > 768 ? 256 : 96) || a.N % 16 != 0 || a.seg_cols % 16 != 0 || a.K % 32 != 0 || a.lda % 4 != 0 || a.epi != EPI_ROUTE || a.B2 ||
        a.halo_src || a.a_pieces || a.out_pieces || a.act_gelu || a.stats || gemm_pads_rows(a) ||
        (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.res) & 15) || (a.res && a.ldr % 4 != 0) ||
        gemm_a_rows(a) * a.lda >= (int64_t)1 << 29 || k * a.N * std::max(1, a.classes) >= (int64_t)1 << 29) return false;
    for (int s = 0; s < cdiv(a.N, a.seg_cols); ++s)
        if (a.seg[s].transposed || ((uintptr_t)a.seg[s].ptr & 15) || a.seg[s].ld % 4 != 0) return false;
    constexpr int W = 4;
    const int m_first = (int64_t)a.M <= (int64_t)a.N * a.taps * std::max(1, a.classes);
    gemm_few_kernel<16, 16, W, false, 0, true><<<(unsigned)(8 * cdiv(tiles, 8)), 64 * W, FewCfg<16, 16, W>::LDS, st>>>(a, 0, m_first);
    return true;
}

}  // namespace pserve
