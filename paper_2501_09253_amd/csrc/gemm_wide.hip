// bf16 linear layers on 256 x 256 tiles, gfx950.
//
// Eight wavefronts (two per SIMD), each 64 rows x 128 columns of the tile: 0.75 LDS fragment reads per MFMA, K in steps
// of 64, both operands staged by direct global -> LDS loads into a ring of two stages (128 KB).  What a tile costs
// besides its main loop decides at these sizes (K = 640 .. 6144: 10 .. 96 steps), so the end of a tile is kept short:
//   * the bias is what the accumulators start from;
//   * the MFMA operands are ordered so that a lane holds CONSECUTIVE elements of an output row: of a token's columns for
//     a plain segment, of a channel's tokens for a transposed one (operands swapped; decided per wavefront).  The rows
//     of the first operand are assigned through kperm, so that they come in pieces of eight: an output tile is rounded
//     in registers and passes LDS as 16-byte bf16 pieces (4 + 4 LDS accesses per 32 x 64 elements and wavefront instead
//     of 32 + 8 with fp32 values one by one), and leaves in stores of 128 contiguous bytes per row;
//   * the residual is fetched in that same layout, a piece of 32 x 64 ahead;
//   * the first step of the next tile is in flight while the current one is finished.
#include "mfma_util.h"
#include <type_traits>

namespace pserve {

// MFMA tile row r holds element kperm(r) (bits 2 and 3 swapped): the 16 elements of a lane are two runs of eight
__device__ __forceinline__ int gw_kperm(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

template <int WGM, int WGN, int TM, int TN>
struct WideCfg {
    static constexpr int NW = WGM * WGN, WM = 32 * TM, WN = 32 * TN, BM = WGM * WM, BN = WGN * WN;
    static constexpr int STAGE = (BM + BN) * 128;                    // bytes: rows of 64 bf16
    static constexpr size_t LDS = 2 * STAGE + 2 * BM * sizeof(int32_t);     // ring, token tables
    static_assert(LDS <= 160 * 1024, "ring does not fit the LDS");
    static_assert(STAGE >= NW * 4096, "the output staging (4 KB a wavefront) reuses the second stage");
};

// What the end of a tile does, besides the bias (compiled in: a skipped path in straight-line code that runs once a tile
// costs instruction fetches).  GW_PLAIN also takes the segment's scale and transposed segments.
enum { GW_PLAIN = 0, GW_RES = 1, GW_GATE_RES = 2, GW_GELU = 3, GW_GEGLU = 4 };

template <int WGM, int WGN, int TM, int TN, int END>
__global__ void __launch_bounds__(64 * WGM * WGN, 2)
gemm_wide_kernel(GemmArgs a) {
    using Cfg = WideCfg<WGM, WGN, TM, TN>;
    constexpr bool GEGLU = END == GW_GEGLU;
    constexpr int NW = Cfg::NW, WM = Cfg::WM, WN = Cfg::WN, BM = Cfg::BM, BN = Cfg::BN;
    constexpr int RP = 8 * NW, A_LD = BM / RP, B_LD = BN / RP, LD = A_LD + B_LD;     // rows per load, loads per step
    constexpr int STAGE_V = Cfg::STAGE / 16;
    constexpr int NM = TM * TN, NR = TM + TN;
    constexpr int LSP = 2;                              // slots between two loads of a refill
    constexpr int GM = 6;                               // M tiles of a group (see below)
    // With more A tiles than B tiles the A fragments have one register set: tile i is refilled behind the last MFMA of the
    // sub-step that reads it (acc of 160 registers and two full sets would not fit 256).
    constexpr bool SA = TM > TN;
    constexpr int QB = 2;                               // MFMAs of a step's last sub-step in front of the barrier
    static_assert(TN % 2 == 0 && NR + QB <= NM + (SA ? 1 : 0) && BM % RP == 0 && BN % RP == 0 && (!SA || TN == 2), "tile shape");
    static_assert(!GEGLU || WN == 2 * GEGLU_GROUP, "GEGLU needs a wavefront tile of [GROUP values | GROUP gates]");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    u32x4* ring = reinterpret_cast<u32x4*>(smem);                        // [2][STAGE_V]: A rows, then B rows
    int32_t* s_tok2 = reinterpret_cast<int32_t*>(ring + 2 * STAGE_V);    // [2][BM] output row of each tile row, -1 = none

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;         // the two wavefronts of a SIMD share their rows
    const int fr = lane & 31, fh = lane >> 5;

    // Tile order.  Tiles are numbered in groups of GM M tiles, M fastest inside a group; XCD x (block id mod 8) takes the
    // x-th eighth of the numbers: the ~32 blocks of an XCD run on about GM x 32 / GM neighbouring tiles whose A and B
    // panels they stream at the same time, and every XCD has the same share whatever the number of M tiles is.
    // A second problem (a.B2: another patch list, weights of its own) continues the M tiles of the first.
    const bool masked = a.tokens_are_rows && a.act.active;
    const int cnt1 = masked ? *a.act.count : 0, cnt2 = a.B2 ? *a.act2.count : 0;                // computed patches
    const int mt1 = ((masked ? cnt1 * a.geom.S : a.M) + BM - 1) / BM;
    const int n_tiles = (a.N + BN - 1) / BN, m_tiles = mt1 + (cnt2 * a.geom.S + BM - 1) / BM;
    const int total = n_tiles * m_tiles, xcd = blockIdx.x & 7;
    const int t_end = (int)((int64_t)total * (xcd + 1) / 8), t_step = gridDim.x >> 3;
    int t = (int)((int64_t)total * xcd / 8) + (blockIdx.x >> 3);
    if (t >= t_end) return;
    auto decode = [&](int tt, int& m0, int& n0, bool& second) {
        const int grp = tt / (GM * n_tiles), r = tt - grp * (GM * n_tiles);
        const int gm = min(GM, m_tiles - grp * GM);
        const int nt = r / gm;
        const int mt = grp * GM + r - nt * gm;
        second = mt >= mt1;
        m0 = (second ? mt - mt1 : mt) * BM;
        n0 = nt * BN;
    };
    int m0, n0;
    bool second;
    decode(t, m0, n0, second);

    // staging: a load of a wavefront fills 8 rows x 8 chunks; the lane at (row, position) fetches chunk
    // position ^ ((row >> 1) & 7), so the bank swizzle is free.  Rows lr + RP * l of both operands.
    const int lc = lane & 7, lr = 8 * wave + (lane >> 3);
    const int gc = lc ^ ((lr >> 1) & 7);
    int a_lane[A_LD], b_lane[B_LD];                     // byte offsets from the tensors' bases
    const void* b_cur = second ? a.B2 : a.B;            // weights of the tile being loaded
    const int KT = a.K / 64;
    auto setup = [&](int tm0, int tn0, bool sec, int32_t* tok_tab) {
        int tok[A_LD], orow[A_LD];                      // input row (0 where there is none), output row
        if (masked) {
            const int32_t* active = sec ? a.act2.active : a.act.active;
            const int act_count = sec ? cnt2 : cnt1;
            int p[A_LD];
#pragma unroll
            for (int l = 0; l < A_LD; ++l) p[l] = active[min((tm0 + lr + l * RP) / a.geom.S, act_count - 1)];
#pragma unroll
            for (int l = 0; l < A_LD; ++l) {
                const int ri = tm0 + lr + l * RP, pi = ri / a.geom.S;
                tok[l] = p[l] * a.geom.S + ri - pi * a.geom.S;
                orow[l] = pi < act_count ? tok[l] : -1;
            }
        } else {
#pragma unroll
            for (int l = 0; l < A_LD; ++l) {
                const int ri = tm0 + lr + l * RP;
                tok[l] = min(ri, a.M - 1);
                orow[l] = ri < a.M ? ri : -1;
            }
            if (!a.tokens_are_rows && a.row_group > 0) {
#pragma unroll
                for (int l = 0; l < A_LD; ++l)
                    if (orow[l] >= 0) orow[l] = (orow[l] / a.row_group) * a.row_group_pad + orow[l] % a.row_group;
            }
        }
#pragma unroll
        for (int l = 0; l < A_LD; ++l) {
            a_lane[l] = (tok[l] * (int)a.lda + gc * 8) * 2;
            if (lc == 0) tok_tab[lr + l * RP] = orow[l];
        }
        // columns past the last one (N is a multiple of 64, not of BN) re-read the last row and are not stored
#pragma unroll
        for (int l = 0; l < B_LD; ++l) b_lane[l] = (min(tn0 + lr + l * RP, a.N - 1) * a.K + gc * 8) * 2;
    };
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t ga_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, 0x7fffffff, 0x00020000);
#define PS_LOAD(dst_, koff_, l_)                                                                                       \
    {                                                                                                                  \
        if ((l_) < A_LD)                                                                                               \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ga_rsrc, (lds_void*)((dst_) + (l_) * (64 * NW)), 16,              \
                                                     a_lane[(l_) < A_LD ? (l_) : 0], (koff_), 0, 0);                   \
        else if ((l_) < LD)                                                                                            \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)b_cur, 0, 0x7fffffff, 0x00020000), \
                                                     (lds_void*)((dst_) + BM * 8 + ((l_) - A_LD) * (64 * NW)), 16, \
                                                     b_lane[(l_) >= A_LD && (l_) < LD ? (l_) - A_LD : 0], (koff_), 0, 0); \
    }
#else       // the host pass only needs the kernel's stub
#define PS_LOAD(dst_, koff_, l_) (void)0
#endif
    auto load_stage = [&](int kt, int st) {
        u32x4* dst = ring + st * STAGE_V + wave * 64;
#pragma unroll
        for (int l = 0; l < LD; ++l) PS_LOAD(dst, kt * 128, l);
    };

    f32x16 acc[TM][TN];
    bf16x8 fa[SA ? 1 : 2][TM], fb[2][TN];
    int buf = 0;
    setup(m0, n0, second, s_tok2);
    load_stage(0, 0);
    if (KT > 1) load_stage(1, 1);

    // one tile of this wavefront: main loop and output.  TR: the wavefront's columns belong to a transposed segment.
    auto tile = [&](auto tr_c, int nt, int nm0, int nn0, bool nsec) {
        constexpr bool TR = decltype(tr_c)::value;
        const int rowA = wm * WM + (TR ? gw_kperm(fr) : fr), rowB = wn * WN + (TR ? fr : gw_kperm(fr));
        const int swA = (rowA >> 1) & 7, swB = (rowB >> 1) & 7;
        const u32x4* pA = ring + rowA * 8;
        const u32x4* pB = ring + BM * 8 + rowB * 8;
        const int wcol = n0 + wn * WN;                  // first packed column of the wavefront
    // one fragment read of sub-step ks_ of stage st_: r_ < TN: B tile r_, else A tile r_ - TN
#define PS_READ(set_, st_, ks_, r_)                                                                                    \
    {                                                                                                                  \
        const int c_ = 2 * (ks_) + fh;                                                                                 \
        const int jb_ = (r_) < TN ? (r_) : 0, ia_ = (r_) >= TN && (r_) < NR ? (r_) - TN : 0;                           \
        if ((r_) < TN) fb[set_][jb_] = __builtin_bit_cast(bf16x8, pB[(st_) * STAGE_V + jb_ * 256 + (c_ ^ swB)]);       \
        else if ((r_) < NR) fa[SA ? 0 : (set_)][ia_] = __builtin_bit_cast(bf16x8, pA[(st_) * STAGE_V + ia_ * 256 + (c_ ^ swA)]); \
    }
        // what is read behind MFMA q of a sub-step (-1: nothing); `late`: the sub-step with the barrier, nothing before QB
        auto read_at = [](int q, bool late) constexpr -> int {
            if constexpr (SA) {                         // A tile i is free behind MFMA 2 i + 1
                if (!late) return q % 2 ? TN + q / 2 : (q / 2 < TN ? q / 2 : -1);
                constexpr int seq[10] = {-1, -1, TN, TN + 1, 0, TN + 2, 1, TN + 3, -1, TN + 4};
                return q < 10 ? seq[q] : -1;
            } else {
                const int k = late ? q - QB : q;        // A tile 0, the B tiles, the other A tiles
                return k < 0 || k >= NR ? -1 : k == 0 ? TN : k <= TN ? k - 1 : k;
            }
        };
        // accumulators start at the bias (of columns that exist)
        const float* bias = second ? a.bias2 : a.bias;
        if (bias) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const float* bp = bias + min(wcol + 32 * j, a.N - 32);
                if constexpr (TR) {
                    const float b = bp[fr];
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[0][j][e] = b;
                } else {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 b = *reinterpret_cast<const f32x4*>(bp + 16 * (g >> 1) + 8 * fh + 4 * (g & 1));
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[0][j][4 * g + e] = b[e];
                    }
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[0][j][e] = 0.f;
        }
#pragma unroll
        for (int i = 1; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = acc[0][j];
        if (KT > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LD) : "memory");       // the first step has landed
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < NR; ++r) PS_READ(0, 0, 0, r);
#pragma unroll 1
        for (int kt = 0; kt < KT; ++kt) {
            const int cur = kt & 1, nxt = cur ^ 1;
            const bool refill = kt + 2 < KT;
            u32x4* dst = ring + cur * STAGE_V + wave * 64;
            const int koff = (kt + 2) * 128;
            // loads of the previous step's refill that are still to be issued: into the other stage, step kt + 1
            const bool late = kt > 0 && kt + 1 < KT;
            u32x4* dst_p = ring + nxt * STAGE_V + wave * 64;
            const int koff_p = (kt + 1) * 128;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
                for (int q = 0; q < NM; ++q) {
                    const int i = q / TN, j = q % TN, f = SA ? 0 : ks & 1;
                    // The fragments of this step are all read (its stage is free), the next step has landed.  A few MFMAs
                    // into the sub-step: at its head a wavefront would wait out its last fragment reads.
                    if (ks == 3 && q == QB) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
                    if constexpr (TR) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[f][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
                    else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][j], fa[f][i], acc[i][j], 0, 0, 0);
                    const int r = read_at(q, ks == 3);
                    if (r >= 0) {
                        if (ks < 3) { PS_READ((ks + 1) & 1, cur, ks + 1, r); }
                        else { PS_READ(0, nxt, 0, r); }
                    }
                    // The stage freed by the barrier is refilled over the slots that follow it, into the next step (ring
                    // position of the slots after the barrier: 0 ..): the eight wavefronts' loads in one burst would queue up
                    // at the address unit and hold the MFMAs behind them.
                    const int sl = ks == 3 ? q - QB : NM - QB + ks * NM + q;
                    if (ks == 3 && q >= QB && refill) {
#pragma unroll
                        for (int l = 0; l < LD; ++l) if (l * LSP == sl) PS_LOAD(dst, koff, l);
                    }
                    if (ks < 3 && late) {
#pragma unroll
                        for (int l = 0; l < LD; ++l) if (l * LSP == sl) PS_LOAD(dst_p, koff_p, l);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
#undef PS_READ
        // ---- output, in pieces of 32 rows (tokens; TR: channels) x 64 elements
        const int32_t* w_tok = s_tok2 + buf * BM + wm * WM;
        u32x4* ep = ring + STAGE_V + wave * 256;        // [32 rows][8 chunks], chunk ^ ((row >> 1) & 7)
        const int er = lane >> 3, ec = lane & 7;        // row (+ 8 k) and chunk this lane stores
        constexpr int NP = GEGLU ? 1 : TN / 2, RD = 3;  // pieces per 32 rows; pieces of the residual in flight
        constexpr bool has_res = END == GW_RES || END == GW_GATE_RES;
        u32x4 rres[has_res ? RD : 1][4];
        auto res_load = [&](int p) {                    // the lane's residual of piece p, in the accumulators' layout
            const int tok = max(w_tok[32 * (p / NP) + fr], 0);
            const uint16_t* rp = (const uint16_t*)a.res + (int64_t)tok * a.ldr + min(wcol + 64 * (p % NP), a.N - 64) + 8 * fh;
#pragma unroll
            for (int c = 0; c < 4; ++c) rres[has_res ? p % RD : 0][c] = *reinterpret_cast<const u32x4*>(rp + 16 * c);
        };
        if constexpr (has_res) {
#pragma unroll
            for (int p = 0; p < RD - 1; ++p) res_load(p);
        }
        asm volatile("" ::: "memory");                  // ahead of the next tile's loads: those would be waited for too
        // every wavefront has read its last fragments (a bare barrier: __syncthreads() would wait for the residual)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (nt < t_end) {                               // first step of the next tile beside the end of this one
            b_cur = nsec ? a.B2 : a.B;
            setup(nm0, nn0, nsec, s_tok2 + (buf ^ 1) * BM);
            load_stage(0, 0);
        }
        if (wcol >= a.N) return;
        if constexpr (TR) {
            const int sg = wcol / a.seg_cols;
            const GemmSeg seg = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
#pragma unroll
            for (int p = 0; p < TN * ((TM + 1) / 2); ++p) {
                const int j = p % TN, i0 = 2 * (p / TN), nv = TM - i0 < 2 ? TM - i0 : 2;     // channels 32 j.., tokens 32 i0..
                if (wcol + 32 * j >= a.N) continue;
#pragma unroll
                for (int ii = 0; ii < nv; ++ii)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int i = i0 + ii;
                        u32x4 o;
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            o[q] = pack_bf16x2(acc[i][j][8 * c + 2 * q] * seg.scale, acc[i][j][8 * c + 2 * q + 1] * seg.scale);
                        ep[fr * 8 + ((4 * ii + 2 * c + fh) ^ ((fr >> 1) & 7))] = o;
                    }
                __builtin_amdgcn_wave_barrier();
                const int trow = 32 * i0 + 8 * (ec & (4 * nv - 1));
                const int t0 = w_tok[trow], t7 = w_tok[trow + 7];
                uint16_t* col0 = (uint16_t*)seg.ptr + (int64_t)(wcol + 32 * j - sg * a.seg_cols + er) * seg.ld;
                if (__all(t0 >= 0 && t7 == t0 + 7 && (t0 & 7) == 0)) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int row = 8 * k + er;
                        const u32x4 o = ep[row * 8 + (ec ^ ((row >> 1) & 7))];
                        if (ec < 4 * nv) *reinterpret_cast<u32x4*>(col0 + 8 * k * seg.ld + t0) = o;
                    }
                } else {                                // ends of requests or of the rows inside a run of eight tokens
#pragma unroll 1
                    for (int k = 0; k < 4; ++k) {
                        const int row = 8 * k + er;
                        const uint16_t* o = reinterpret_cast<const uint16_t*>(ep + row * 8 + (ec ^ ((row >> 1) & 7)));
                        if (ec < 4 * nv)
#pragma unroll 1
                            for (int q = 0; q < 8; ++q) {
                                const int tq = w_tok[trow + q];
                                if (tq >= 0) col0[8 * k * seg.ld + tq] = o[q];
                            }
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        } else {
#pragma unroll
            for (int p = 0; p < TM * NP; ++p) {
                const int i = p / NP, jp = p % NP;
                const int pcol = GEGLU ? wcol / 2 : wcol + 64 * jp;
                if constexpr (has_res) if (p + RD - 1 < TM * NP) res_load(p + RD - 1);
                if (!GEGLU && pcol >= a.N) continue;
                const int sg = GEGLU ? 0 : pcol / a.seg_cols;
                const GemmSeg seg = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
                const float* gate = nullptr;
                if constexpr (END == GW_GATE_RES)
                    gate = (second ? a.rowscale2 : a.rowscale) + (int64_t)a.row_owner[max(w_tok[32 * i + fr], 0) / a.geom.S] * a.rowscale_ld + pcol + 8 * fh;
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int j = GEGLU ? jj : 2 * jp + jj;
                        float v[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            v[q] = acc[i][j][8 * c + q];
                            if constexpr (GEGLU) v[q] *= gelu_erf(acc[i][j + 2][8 * c + q]);
                        }
                        if constexpr (END == GW_GELU) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] = gelu_tanh(v[q]);
                        }
                        if constexpr (END == GW_GATE_RES) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] *= gate[32 * jj + 16 * c + q];
                        }
                        if constexpr (has_res) {
                            const u32x4 r = rres[p % RD][2 * jj + c];
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                v[2 * q] += __uint_as_float(r[q] << 16);
                                v[2 * q + 1] += __uint_as_float(r[q] & 0xFFFF0000u);
                            }
                        }
                        if constexpr (END == GW_PLAIN) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] *= seg.scale;
                        }
                        u32x4 o;
#pragma unroll
                        for (int q = 0; q < 4; ++q) o[q] = pack_bf16x2(v[2 * q], v[2 * q + 1]);
                        ep[fr * 8 + ((4 * jj + 2 * c + fh) ^ ((fr >> 1) & 7))] = o;
                    }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int row = 8 * k + er, tok = w_tok[32 * i + row];
                    const u32x4 o = ep[row * 8 + (ec ^ ((row >> 1) & 7))];
                    if (tok >= 0) *reinterpret_cast<u32x4*>((uint16_t*)seg.ptr + (int64_t)tok * seg.ld + pcol - sg * a.seg_cols + 8 * ec) = o;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    };

#pragma unroll 1
    for (;;) {
        const int nt = t + t_step;
        int nm0 = 0, nn0 = 0;
        bool nsec = false;
        if (nt < t_end) decode(nt, nm0, nn0, nsec);
        bool tr = false;
        if constexpr (END == GW_PLAIN) {
            const int sg = min(n0 + wn * WN, a.N - 1) / a.seg_cols;
            tr = (sg == 0 ? a.seg[0].transposed : (sg == 1 ? a.seg[1].transposed : a.seg[2].transposed)) != 0;
            if (tr) tile(std::true_type{}, nt, nm0, nn0, nsec);
        }
        if (!tr) tile(std::false_type{}, nt, nm0, nn0, nsec);
        if (nt >= t_end) break;
        // the output staging is done with the second stage (a bare barrier: the stores are not waited for)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (KT > 1) load_stage(1, 1);
        t = nt; m0 = nm0; n0 = nn0; second = nsec; buf ^= 1;
    }
#undef PS_LOAD
}

template <int WGM, int WGN, int TM, int TN, int END>
static int launch_wide_end(const GemmArgs& a, hipStream_t st) {
    using Cfg = WideCfg<WGM, WGN, TM, TN>;
    PS_SET_LDS_ONCE((gemm_wide_kernel<WGM, WGN, TM, TN, END>), Cfg::LDS);
    const int64_t tiles = (cdiv(a.M, Cfg::BM) + cdiv(a.B2 ? a.M2 : 0, Cfg::BM)) * cdiv(a.N, Cfg::BN);
    const unsigned grid = (unsigned)std::min<int64_t>(256, 8 * cdiv(tiles, 8));
    gemm_wide_kernel<WGM, WGN, TM, TN, END><<<grid, 64 * Cfg::NW, Cfg::LDS, st>>>(a);
    return check_launch("gemm_wide_kernel");
}

// the end of a tile a problem needs, -1: none of those compiled
static int wide_end(const GemmArgs& a) {
    if (a.epi == EPI_GEGLU) return GW_GEGLU;
    bool plain_segs = true;                             // neither scaled nor transposed
    for (int s = 0; s * a.seg_cols < a.N; ++s) plain_segs = plain_segs && a.seg[s].scale == 1.f && !a.seg[s].transposed;
    if (!a.act_gelu && !a.rowscale && !a.res) return GW_PLAIN;
    if (!plain_segs) return -1;
    if (a.act_gelu) return a.rowscale || a.res ? -1 : GW_GELU;
    return !a.res ? -1 : a.rowscale ? GW_GATE_RES : GW_RES;
}

template <int WGM, int WGN, int TM, int TN>
static int launch_wide(const GemmArgs& a, hipStream_t st) {
    switch (wide_end(a)) {
    case GW_PLAIN: return launch_wide_end<WGM, WGN, TM, TN, GW_PLAIN>(a, st);
    case GW_RES: return launch_wide_end<WGM, WGN, TM, TN, GW_RES>(a, st);
    case GW_GATE_RES: return launch_wide_end<WGM, WGN, TM, TN, GW_GATE_RES>(a, st);
    case GW_GELU: return launch_wide_end<WGM, WGN, TM, TN, GW_GELU>(a, st);
    default:
        if constexpr (32 * TN == 2 * GEGLU_GROUP) return launch_wide_end<WGM, WGN, TM, TN, GW_GEGLU>(a, st);
        set_error("gemm_wide: no such tile");
        return PSERVE_EINVAL;
    }
}

// what the kernel can do at all; wave_cols: columns of a wavefront
static bool wide_eligible(const GemmArgs& a, int wave_cols) {
    if (a.conv || a.taps != 1 || a.rowbias || a.stats || a.K % 64 != 0 || a.lda % 8 != 0 || wide_end(a) < 0) return false;
    if (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.bias | (uintptr_t)a.res) & 15) return false;
    if (!gemm_fits32(a)) return false;
    if (a.epi == EPI_GEGLU)
        return wave_cols == 2 * GEGLU_GROUP && a.N % 128 == 0 && !((uintptr_t)a.seg[0].ptr & 15) && a.seg[0].ld % 8 == 0;
    if (a.N % 64 != 0 || a.seg_cols % 64 != 0 || (a.res && a.ldr % 8 != 0)) return false;
    if (a.rowscale && !a.tokens_are_rows) return false;
    if (a.B2 && (!a.tokens_are_rows || !a.act.active || !a.act2.active || (((uintptr_t)a.B2 | (uintptr_t)a.bias2) & 15) ||
                 !a.bias != !a.bias2 || !a.rowscale != !a.rowscale2)) return false;
    for (int s = 0; s * a.seg_cols < a.N; ++s) {
        if (((uintptr_t)a.seg[s].ptr & 15) || a.seg[s].ld % 8 != 0) return false;
        // a wavefront's columns take one operand order
        if (a.seg[s].transposed && a.seg_cols % wave_cols != 0) return false;
    }
    return true;
}

// Time of a launch in microseconds as measured on full rounds of 256 tiles (one block per CU) and on partly filled ones:
// a step of 64 columns takes s0 on an otherwise idle chip and s1 with every CU busy (the clock drops with the power
// drawn), a tile's start and end take o, the first start 2 us more.
static double wide_cost(int64_t tiles, int64_t steps, double s0, double s1, double o) {
    const double f = (double)(tiles % 256) / 256;
    return 2.0 + (double)(tiles / 256) * (steps * s1 + o) + (f > 0 ? steps * (s0 + (s1 - s0) * f) + o : 0.0);
}

// The linear layers these tiles take.  Against 128-row tiles with two blocks per CU (the other kernel): 12,544 x 1536
// tokens q/k/v 222 -> 168 us, out 74 -> 58, 1536 -> 6144 291 -> 228, 6144 -> 1536 270 -> 207; 13,312 x 1280 q/k/v 150 -> 136,
// out 61 -> 48; 13,312 x 640 q/k/v 47.6 -> 41.7, GEGLU 115 -> 108.  They lose where their rounds come out badly (13,312 x
// 640 x 640: 156 tiles for 256 CUs, 25 against 22 us) and to smaller tiles on few rows, so the launch compares the
// modelled times of both; the model is within 10 % of the measured shapes (K = 640 .. 6144).
// Returns the rows of the tile to use, 0: the other kernel.
static int wide_select(const GemmArgs& a) {
    const int64_t steps = a.K / 64;
    auto m_tiles = [&](int bm) { return cdiv(a.M, bm) + cdiv(a.B2 ? a.M2 : 0, bm); };
    int64_t t256 = m_tiles(256) * cdiv(a.N, 256), t320 = m_tiles(320) * cdiv(a.N, 256);
    if (!wide_eligible(a, 128)) t256 = 0;
    if (!wide_eligible(a, 64)) t320 = 0;
    if (std::max(t256, t320) < 128) return 0;                   // half the chip idle: smaller tiles
    const double c256 = t256 >= 128 ? wide_cost(t256, steps, 0.97, 1.62, 8.0) : 1e30;
    const double c320 = t320 >= 128 ? wide_cost(t320, steps, 1.20, 2.05, 9.0) : 1e30;
    // the other kernel's tiles: 512 blocks at a time, a last round at most half full leaves one block per CU
    const bool geglu = a.epi == EPI_GEGLU, n160 = !geglu && a.N % 160 == 0;
    const int64_t t128 = m_tiles(128) * cdiv(a.N, n160 ? 160 : 128), full = t128 / 512, rest = t128 % 512;
    const double per = n160 ? 0.95 * steps + 9.0 : geglu ? 0.80 * steps + 5.5 : 0.97 * steps + 6.0;
    const double last = n160 ? 1.05 * steps + 11.8 : 1.1 * per;
    const double c128 = full * per + (rest == 0 ? 0.0 : rest <= 256 ? 0.75 * last : last);
    return c128 <= std::min(c256, c320) ? 0 : c256 <= c320 ? 256 : 320;
}

// Two problems (a.B2) whose rows are too few for wide_select, or whose tiles come out badly: whichever is modelled fastest of these
// tiles all the same, 128 x 64 or 128 x 128 (gemm_two_bf16), and the small ones of gemm_few.hip in up to four rounds.  As two launches
// on two streams, the text stream's kernel waits for CUs that the image stream's holds, and every fork and join costs ~10 us.
// us of a step, two streams / one launch a layer: 576 + 864 rows x 768 166 / 128, 3,072 + 1,280 283 / 211, 6,400 + 600 408 / 327; 3,072 +
// 1,024 x 1,536 552 / 440, 2,304 + 288 377 / 355; 26 sizes 1.15x in the mean, none slower.
// Returns the rows of the tile here, 128: gemm_two_bf16 with *tile columns, -1: gemm_few.hip's tile *tile, 0: none takes the problem.
int few_pick(const GemmArgs& a, int most_rounds, double* us);
int gemm_few_bf16(const GemmArgs& a, int tile, hipStream_t st);
int gemm_two_cols(const GemmArgs& a, double* us);
int gemm_two_bf16(const GemmArgs& a, int cols, hipStream_t st);
static int two_select(const GemmArgs& a, int* tile) {
    auto t = [&](int bm) { return (cdiv(a.M, bm) + cdiv(a.M2, bm)) * cdiv(a.N, 256); };
    if (!gemm_two_eligible(a)) return 0;
    double us[4];
    const int few = few_pick(a, 4, &us[0]), cols = gemm_two_cols(a, &us[1]);
    us[2] = wide_eligible(a, 128) ? 1.1 * wide_cost(t(256), a.K / 64, 0.97, 1.62, 8.0) : 1e30;
    us[3] = wide_eligible(a, 64) ? 1.1 * wide_cost(t(320), a.K / 64, 1.20, 2.05, 9.0) : 1e30;
    static const int rows[4] = {-1, 128, 256, 320};
    const int64_t best = std::min_element(us, us + 4) - us;
    *tile = best ? cols : few;
    return us[best] < 1e30 ? rows[best] : 0;
}

bool gemm_takes_two(const GemmArgs& a, int dtype, int mode) {
    int tile;
    return dtype == PSERVE_BF16 && mode == 0 && a.B2 && gemm_mfma_eligible(a) && (wide_select(a) != 0 || two_select(a, &tile) != 0);
}

int gemm_wide_bf16(const GemmArgs& a, hipStream_t st, bool* handled) {
    int tile = 0, rows = wide_select(a);
    if (!rows && a.B2) rows = two_select(a, &tile);
    *handled = rows != 0;
    if (rows < 0) return gemm_few_bf16(a, tile, st);
    if (rows == 128) return gemm_two_bf16(a, tile, st);
    if (rows == 256) return launch_wide<4, 2, 2, 4>(a, st);
    if (rows == 320) return launch_wide<2, 4, 5, 2>(a, st);
    return PSERVE_OK;
}

// For tests (host only, no part of the ABI): the rows of the tile such a layer takes here, 0: another kernel's.  P patches of
// S tokens; rows: those of the layer's patch list, rows2: of a second problem's, 0: none.  flags: 1 last segment transposed,
// 2 residual, 4 gate, 8 GELU, 16 value-gate pairs, 32 rows without a patch list, 64 a mask,
// 128 beside another stream's kernels.
static GemmArgs test_args(int32_t P, int32_t S, int32_t rows, int32_t rows2, int32_t N, int32_t K, int32_t seg_cols, int32_t flags) {
    GemmArgs a{};
    void* some = reinterpret_cast<void*>(64);           // tested for alignment, never read
    static const int32_t list = 0;
    a.A = a.B = some; a.lda = a.K = K; a.N = N; a.M = rows; a.taps = 1; a.seg_cols = seg_cols; a.ldr = N;
    a.geom.P = P; a.geom.S = S; a.tokens_are_rows = !(flags & 32);
    for (int s = 0; s < 3; ++s) { a.seg[s].ptr = some; a.seg[s].ld = 8; a.seg[s].scale = 1.f; }
    if (flags & 1) a.seg[N / seg_cols - 1].transposed = 1;
    if (flags & 2) a.res = some;
    if (flags & 4) a.rowscale = a.rowscale2 = static_cast<float*>(some);
    a.act_gelu = (flags & 8) != 0;
    a.epi = flags & 16 ? EPI_GEGLU : EPI_ROUTE;
    if (flags & 64) a.act.active = a.act.count = &list;
    a.beside = (flags & 128) != 0;
    if (rows2) { a.B2 = some; a.M2 = rows2; a.act.active = a.act.count = a.act2.active = a.act2.count = &list; }
    return a;
}
extern "C" int pserve_test_linear_tile(int32_t P, int32_t S, int32_t rows, int32_t rows2, int32_t N, int32_t K, int32_t seg_cols,
                                       int32_t flags) {
    return wide_select(test_args(P, S, rows, rows2, N, K, seg_cols, flags));
}
// The kernel of such a layer: -1 .. -5 a small tile (gemm_few.hip), 256 or 320 rows of a tile here, 10 x columns + stages of a 128-row one.
// owner_rows: GemmArgs.  flags & 256: a 2x upsampling of K channels.
int gemm_tile_code(const GemmArgs& a);
extern "C" int pserve_test_linear_kernel(int32_t P, int32_t S, int32_t rows, int32_t N, int32_t K, int32_t seg_cols, int32_t flags, int32_t owner_rows) {
    GemmArgs a = test_args(P, S, rows, 0, N, K, seg_cols, flags);
    a.owner_rows = owner_rows;
    if (flags & 256) {
        a.conv = 1; a.taps = a.classes = 4;
        return gemm_tile_code(a);
    }
    double us;
    const int few = a.beside ? 0 : few_pick(a, a.epi == EPI_GEGLU ? 2 : 1, &us);
    if (few) return -few;
    if (const int r = wide_select(a)) return r;
    return a.epi == EPI_GEGLU ? (N % 128 == 0 ? 1282 : 0) : gemm_tile_code(a);
}
// The tile that two problems in one launch take where that one is 0: rows of a tile here, 64 or 128: columns of a 128-row one, -1 .. -5:
// a small one (gemm_few.hip), 0: none.
extern "C" int pserve_test_two_tile(int32_t P, int32_t S, int32_t rows, int32_t rows2, int32_t N, int32_t K, int32_t seg_cols, int32_t flags) {
    int tile;
    const int r = two_select(test_args(P, S, rows, rows2, N, K, seg_cols, flags), &tile);
    return r == 128 ? tile : r < 0 ? -tile : r;
}

}  // namespace pserve
