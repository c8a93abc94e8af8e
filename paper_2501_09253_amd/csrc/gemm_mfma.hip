// bf16 MFMA GEMM / implicit-GEMM 3x3 convolution for gfx950.
//
// Two kernels share one epilogue:
//   gemm_mfma_kernel  block tile 128 x 160 / 128 x 128 (GEGLU) with four wavefronts stacked along M or 128 x 128 / 128 x 64 (2 x 2), K in
//                     steps of 64, A and B tiles staged by direct global -> LDS loads into a ring of two, three or four stages (one
//                     barrier per step); the linear layers that neither gemm_few.hip nor gemm_wide.hip (asked first) takes, and
//                     convolutions (taps re-load A): level changes, patches the other kernel does not take, and all others where
//                     its rounds fit better (conv_choose).  The tiles with two stages run two blocks per CU.
//   conv_mfma_kernel  3x3 convolution with the haloed activation tile kept in LDS across the nine taps;
//                     preferred tile 256 x 160 with four wavefronts stacked along M, each doubled by a second
//                     wavefront that takes the other half of every K step (two wavefronts per SIMD).
// In both, every LDS fragment read and every global load is issued behind an MFMA (a wavefront issues in order,
// and with one block per CU and four wavefronts there is no other wavefront on the SIMD to fill a bubble).
// MFMA shape v_mfma_f32_32x32x16_bf16, fp32 accumulation.  LDS rows are 128 bytes (8 chunks of 16 bytes); chunk c of
// row r sits at position c ^ ((r >> 1) & 7), which keeps the fragment reads (32 rows at one chunk position)
// bank-conflict free; the swizzle is applied by choosing which global chunk each lane of a load fetches.
#include "mfma_util.h"
#include <type_traits>

namespace pserve {

// ---- epilogue shared by the kernels.  A lane holds column (lane % 32) of each 32x32 tile and rows
// 8*(e/4) + 4*(lane/32) + e%4.  One tile column (WM rows x 32 columns) at a time is finished in registers (bias,
// scale, GEGLU), staged as fp32 in this wavefront's private LDS region and read back row-wise, so that residual
// loads and output stores are 16 bytes per lane and 64 contiguous bytes per row.  Residual loads of the next tile
// column are issued before the current one is staged.  `smem` must be free (all staged operands consumed).
// bias_pre: the lane's bias of each of its TN tile columns, loaded by the caller (a kernel that has other loads in
// flight reads it before issuing those: a wait for a later load waits for all earlier ones).
// FEAT: which of the rarely taken paths are compiled in.  The epilogue is straight-line code that a block runs once per
// tile, fully unrolled over the tile columns: every path that is present but skipped costs a jump to an instruction
// line that is not in the cache (per-column timestamps showed 2 us per column, about five such jumps each, whatever
// the memory traffic), so a kernel that can rule a path out by its launch conditions leaves it out.
enum : int {
    EPF_TRANS = 1,      // transposed output segments
    EPF_GELU = 2,       // tanh GELU on the result
    EPF_GATE = 4,       // per-request gate (rowscale)
    EPF_MIXED = 8,      // rows of several requests in one wavefront tile: per-element look-ups of rowbias / rowscale
    EPF_SCALE = 16,     // output segments with a scale other than 1 (the pre-multiplied Q)
    EPF_ALL = 31,
    EPF_PADS = 32,      // tiles walk the padded rows of the requests (gemm_pads_rows)
    EPF_TWO = 64,       // a second problem (GemmArgs::B2) continues the row tiles; one tile a block
    EPF_HALO = 128,     // a convolution that reads the unpadded batch (GemmArgs::halo_src)
    EPF_STAT = 256      // moments of the output (GemmCore::stats)
};
template <int BM, int BN, bool GEGLU, int WGM = 2, int WGN = 2, bool MAY_STAT = true, int FEAT = EPF_ALL>
__device__ __forceinline__ void gemm_epilogue(const GemmCore& a, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32], uint8_t* smem,
                                              const int32_t* s_tok, int n0, const float* bias_pre, const float* rowscale) {
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;     // WGM x WGN wavefront grid
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int fr = lane & 31, fh = lane >> 5;
    constexpr int EP_LD = 36;                                       // floats per staged row (16-byte aligned, skewed banks)
    float* ep = reinterpret_cast<float*>(smem) + wave * (WM * EP_LD);
    const int32_t* w_tok = s_tok + wm * WM;
    constexpr int TNO = GEGLU ? TN / 2 : TN;                        // output tile columns per wavefront
    static_assert(!GEGLU || (WN == 2 * GEGLU_GROUP), "GEGLU needs a wavefront tile of [GROUP values | GROUP gates]");
    // residual rows of this lane's read-back items (row = item / 4, 8-column chunk = item % 4)
    constexpr int NIT = WM * 4 / 64;
    const bool HAS_RES = !GEGLU && a.res != nullptr;
    const uint16_t* res_row[NIT];
    // residual of the lane's items: with a small wavefront tile all tile columns are fetched at once (every column
    // otherwise waits out a memory round trip of its own, with one column of work to cover it), else one column ahead
    constexpr bool RES_ALL = TNO * NIT <= 12;
    constexpr int RSETS = RES_ALL ? TNO : 2;
    u32x4 rres[RSETS][NIT];
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
        const int item = t * 64 + lane;
        const int tok = w_tok[item >> 2];
        res_row[t] = (const uint16_t*)a.res + (int64_t)(tok < 0 ? 0 : tok) * a.ldr + (item & 3) * 8;
    }
    if (HAS_RES) {
#pragma unroll
        for (int jj = 0; jj < (RES_ALL ? TNO : 1); ++jj)
#pragma unroll
            for (int t = 0; t < NIT; ++t) rres[jj][t] = *reinterpret_cast<const u32x4*>(res_row[t] + n0 + wn * WN + jj * 32);
    }
    // per-request bias (time embedding): one value per column when all rows of the wavefront's tile belong to one
    // request (rows are ordered by request, so first == last decides), else looked up per element
    bool rb_uniform = false;
    int rb_slot = 0;
    if (!GEGLU && (a.rowbias || ((FEAT & EPF_GATE) && rowscale))) {
        const int t_first = w_tok[0], t_last = w_tok[WM - 1];
        if (t_first >= 0 && t_last >= 0) {
            rb_slot = a.row_owner[t_first / a.geom.S];
            rb_uniform = rb_slot == a.row_owner[t_last / a.geom.S];
        }
    }
    // GroupNorm partial sums of the output (optional): column moments over this wavefront's WM rows (32 or 64), which lie in one patch
    const bool STATS = MAY_STAT && !GEGLU && a.stats != nullptr;     // only convolutions leave them behind
    float* colsum = reinterpret_cast<float*>(smem) + WGM * WGN * (WM * EP_LD) + wave * (2 * WN + 2);    // [WN][2] + row count
    uint32_t row_ok[TM];                                            // bit e: row 8*(e/4) + 4*fh + e%4 of tile i exists
    const bool all_rows = STATS && w_tok[WM - 1] >= 0;              // existing rows are a prefix of the tile
    if (STATS && !all_rows) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            row_ok[i] = 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) row_ok[i] |= (w_tok[i * 32 + 8 * (e >> 2) + 4 * fh + (e & 3)] >= 0 ? 1u : 0u) << e;
        }
    }
#pragma unroll
    for (int j = 0; j < TNO; ++j) {
        const int pcol = n0 + wn * WN + j * 32;                     // first packed column of the tile
        int ocol0;                                                  // first output column within its segment
        GemmSeg sgm;
        float vals[TM][16];
        if (GEGLU) {
            const float bv = bias_pre ? bias_pre[j] : (a.bias ? a.bias[pcol + fr] : 0.f);
            const float bg = bias_pre ? bias_pre[j + TN / 2] : (a.bias ? a.bias[pcol + fr + GEGLU_GROUP] : 0.f);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) vals[i][e] = (acc[i][j][e] + bv) * gelu_erf(acc[i][j + TN / 2][e] + bg);
            sgm = a.seg[0];
            ocol0 = (n0 + wn * WN) / 2 + j * 32;
        } else {
            const int sg = pcol / a.seg_cols;
            sgm = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
            ocol0 = pcol - sg * a.seg_cols;
            float bias = bias_pre ? bias_pre[j] : (a.bias ? a.bias[pcol + fr] : 0.f);
            if (rb_uniform && a.rowbias) bias += a.rowbias[(int64_t)rb_slot * a.N + pcol + fr];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) vals[i][e] = acc[i][j][e] + bias;
            if ((FEAT & EPF_MIXED) && a.rowbias && !rb_uniform) {   // rows of several requests in this wavefront's tile
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int tok = w_tok[i * 32 + 8 * (e >> 2) + 4 * fh + (e & 3)];
                        if (tok >= 0) vals[i][e] += a.rowbias[(int64_t)a.row_owner[tok / a.geom.S] * a.N + pcol + fr];
                    }
            }
            if ((FEAT & EPF_GELU) && a.act_gelu) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) vals[i][e] = gelu_tanh(vals[i][e]);
            }
            if ((FEAT & EPF_GATE) && rowscale) {              // gate of the request, before the residual is added
                if (rb_uniform || !(FEAT & EPF_MIXED)) {
                    const float gate = rowscale[(int64_t)rb_slot * a.rowscale_ld + pcol + fr];
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int e = 0; e < 16; ++e) vals[i][e] *= gate;
                } else {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int tok = w_tok[i * 32 + 8 * (e >> 2) + 4 * fh + (e & 3)];
                            if (tok >= 0) vals[i][e] *= rowscale[(int64_t)a.row_owner[tok / a.geom.S] * a.rowscale_ld + pcol + fr];
                        }
                }
            }
            if (STATS) {
                // column moments over the wavefront's WM rows, around the value of the column's first row (shifted sums:
                // nothing is lost when the mean is far from zero); stored as (mean, M2) of the column
                const float own0 = vals[0][0], oth0 = other_half_f(own0);
                const float kc = fh == 0 ? own0 : oth0;             // both lane halves of a column use the lower half's value
                float s1 = 0.f, s2 = 0.f, nr = 0.f;
                if (all_rows) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int e = 0; e < 16; ++e) { const float d = vals[i][e] - kc; s1 += d; s2 = fmaf(d, d, s2); }
                    nr = (float)(TM * 16);
                } else {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const bool ok = (row_ok[i] >> e) & 1u;
                            const float d = ok ? vals[i][e] - kc : 0.f;
                            s1 += d;
                            s2 = fmaf(d, d, s2);
                            nr += ok ? 1.f : 0.f;
                        }
                }
                s1 += other_half_f(s1);
                s2 += other_half_f(s2);
                nr += other_half_f(nr);
                if (fh == 0) {
                    const float inv = nr > 0.f ? 1.f / nr : 0.f;
                    colsum[2 * (j * 32 + fr)] = kc + s1 * inv;
                    colsum[2 * (j * 32 + fr) + 1] = fmaxf(s2 - s1 * s1 * inv, 0.f);
                    if (j == 0 && fr == 0) colsum[2 * WN] = nr;     // rows of this wavefront's tile that exist
                }
            }
        }
        uint16_t* out = (uint16_t*)sgm.ptr;
        if ((FEAT & EPF_TRANS) && sgm.transposed) {
            // out[col][token]: the four rows e%4 of a lane are consecutive tokens -> one 8-byte store
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int eg = 0; eg < 4; ++eg) {
                    const int row = i * 32 + 8 * eg + 4 * fh;
                    const int t0 = w_tok[row], t3 = w_tok[row + 3];
                    uint16_t* dst = out + (int64_t)(ocol0 + fr) * sgm.ld;
                    if (t0 >= 0 && t3 == t0 + 3 && (t0 & 3) == 0 && (sgm.ld & 3) == 0) {
                        const uint32_t lo = pack_bf16x2(vals[i][4 * eg] * sgm.scale, vals[i][4 * eg + 1] * sgm.scale);
                        const uint32_t hi = pack_bf16x2(vals[i][4 * eg + 2] * sgm.scale, vals[i][4 * eg + 3] * sgm.scale);
                        *reinterpret_cast<uint2*>(dst + t0) = make_uint2(lo, hi);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int t = w_tok[row + q];
                            if (t >= 0) dst[t] = float_to_bf16_bits(vals[i][4 * eg + q] * sgm.scale);
                        }
                    }
                }
            continue;
        }
        // stage the tile column: ep[row][col]
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) ep[(i * 32 + 8 * (e >> 2) + 4 * fh + (e & 3)) * EP_LD + fr] = vals[i][e];
        __builtin_amdgcn_wave_barrier();
        // prefetch the residual of the next tile column while this one is finished
        if (HAS_RES && !RES_ALL && j + 1 < TNO) {
#pragma unroll
            for (int t = 0; t < NIT; ++t) rres[(j + 1) & 1][t] = *reinterpret_cast<const u32x4*>(res_row[t] + pcol + 32);
        }
#pragma unroll
        for (int t = 0; t < NIT; ++t) {
            const int item = t * 64 + lane;
            const int row = item >> 2, ch = item & 3;
            const int tok = w_tok[row];
            const f32x4 lo = *reinterpret_cast<const f32x4*>(ep + row * EP_LD + ch * 8);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(ep + row * EP_LD + ch * 8 + 4);
            const int64_t tk = tok < 0 ? 0 : tok;                   // rows past the end read row 0 and store nothing
            float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            if (HAS_RES) {
                const u32x4 r = rres[RES_ALL ? j : (j & 1)][t];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[2 * q] += __uint_as_float(r[q] << 16);
                    v[2 * q + 1] += __uint_as_float(r[q] & 0xFFFF0000u);
                }
            }
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                o[q] = (FEAT & EPF_SCALE) ? pack_bf16x2(v[2 * q] * sgm.scale, v[2 * q + 1] * sgm.scale) : pack_bf16x2(v[2 * q], v[2 * q + 1]);
            if (tok >= 0) *reinterpret_cast<u32x4*>(out + tk * sgm.ld + ocol0 + ch * 8) = o;
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (STATS) {
        __builtin_amdgcn_wave_barrier();
        const int cg = a.N / a.stats_G;                             // channels per group (divides WN, see gemm_stats_rows)
        const int tok0 = w_tok[0];
        if (lane < WN / cg && tok0 >= 0) {
            // the group's columns cover the same rows: mean of the column means, M2 by the merge formula
            const float nr = colsum[2 * WN];
            float m = 0.f;
            for (int c = lane * cg; c < (lane + 1) * cg; ++c) m += colsum[2 * c];
            m /= (float)cg;
            float m2 = 0.f;
            for (int c = lane * cg; c < (lane + 1) * cg; ++c) { const float d = colsum[2 * c] - m; m2 += colsum[2 * c + 1] + nr * d * d; }
            const int p = tok0 / a.geom.S, slot = (tok0 - p * a.geom.S) / WM;
            float* dst = a.stats + (((int64_t)p * a.stats_slots + slot) * a.stats_G + (n0 + wn * WN) / cg + lane) * 2;
            dst[0] = m;
            dst[1] = m2;
        }
    }
}

// LDS bytes of one kernel instance: NS stages of (BM + BN) rows x 128 bytes, two row -> token tables and, with
// OVERLAP, a staging region of the epilogue of its own (otherwise the epilogue stages in the drained ring)
template <int BM, int BN, int NS, bool OVERLAP> struct GemmCfg {
    static constexpr int STAGE = (BM + BN) * 128;
    static constexpr int EPI = 4 * (BM / 4 >= 64 ? BM / 4 : 64) * 36 * 4;      // >= 4 wavefronts x WM rows x 36 floats
    static constexpr size_t LDS = (size_t)NS * STAGE + 2 * BM * sizeof(int32_t) + (OVERLAP ? EPI : 0);
    static_assert(LDS <= 160 * 1024, "ring does not fit the LDS");
    static_assert(OVERLAP || NS * STAGE >= EPI, "epilogue staging does not fit the ring");
};

// Block tile BM x BN, WGM x WGN wavefront grid (four wavefronts), ring of NS stages.
// Step = 64 columns of K: 4 sub-steps of TM*TN MFMAs.  Every memory instruction rides behind an MFMA: during sub-steps
// 0..2 the fragment reads of the next sub-step, during sub-step 3 the first fragments of the NEXT step and the refill
// of this step's stage with step + NS.  The block barrier sits before sub-step 3: by then every wavefront has read all
// of this step's fragments (its stage is free) and has seen its own loads of the next step land, NS - 2 further steps
// still being in flight.
// A block walks over tiles (grid = the blocks that fit the chip at once).  With OVERLAP the first NS steps of the next
// tile are issued BEFORE the epilogue of the current one, so that the load latency of a tile start and the vector work
// and stores of a tile end (about 4 us and 6 us of a 19 us tile at K = 640) run beside each other.
template <int BM, int BN, bool GEGLU, int WGM, int WGN, int NS, bool OVERLAP, int FEAT>
__global__ void __launch_bounds__(256, (GemmCfg<BM, BN, NS, OVERLAP>::LDS <= 80 * 1024 ? 2 : 1))
gemm_mfma_kernel(GemmArgs a) {
    constexpr int BK = 64;
    constexpr int CH = BK / 8;                      // 16-byte chunks per row
    constexpr int WM = BM / WGM, WN = BN / WGN;     // wavefront tile
    constexpr int TM = WM / 32, TN = WN / 32;       // 32x32 MFMA tiles per wavefront
    constexpr int A_LD = BM * CH / 256;             // 16-byte loads per thread and K step
    constexpr int B_LD = BN * CH / 256;
    constexpr int LD = A_LD + B_LD;
    constexpr int STAGE_V = (BM + BN) * CH;         // 16-byte slots per stage: A rows then B rows
    static_assert(WGM * WGN == 4 && WM % 32 == 0 && WN % 32 == 0 && (BM * CH) % 256 == 0 && (BN * CH) % 256 == 0 &&
                  NS >= 2 && (NS - 1) * LD <= 63, "tile shape");
    static_assert(4 * WM * 36 * 4 <= GemmCfg<BM, BN, NS, OVERLAP>::EPI, "epilogue staging size");
    // Without a staging region of its own the epilogue stages in the drained ring.  Where the stages behind the first
    // hold that staging (4 wavefronts x WM rows x 36 floats), the first step of the next tile is loaded into stage 0
    // BEFORE the epilogue and the remaining stages after it: the load latency of a tile start (the long part of the
    // ~4 us a tile start costs at K = 640) passes beside the epilogue's vector work and stores.
    constexpr bool HALF = !OVERLAP && (NS - 1) * (BM + BN) * 128 >= 4 * WM * 36 * 4;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    u32x4* ring = reinterpret_cast<u32x4*>(smem);                     // [NS][STAGE_V]
    int32_t* s_tok2 = reinterpret_cast<int32_t*>(ring + NS * STAGE_V); // [2][BM] output row of each tile row, -1 = none
    constexpr bool HALO = (FEAT & EPF_HALO) != 0;
    int32_t* s_src = s_tok2 + 2 * BM;                                  // HALO: [taps][BM] byte offset of the pixel a tap reads
    uint8_t* ep_smem = OVERLAP ? reinterpret_cast<uint8_t*>(s_src + (HALO ? 9 * BM : 0)) : smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // scalar: LDS destinations of the loads are SGPR math
    const int wm = wave / WGN, wn = wave % WGN;
    // Tile order.  Tiles are numbered in groups of gm M tiles, M fastest inside a group, and XCD x (block id mod 8; each has
    // its own L2) takes the x-th eighth of the numbers: the blocks in flight on an XCD (64 at most) cover about gm x 64 / gm
    // neighbouring tiles, so gm is chosen for the fewest bytes of A and B panels, and few rows with many columns end up
    // shared out by columns.  (An eighth of the M tiles per XCD instead: with 8 M tiles every XCD read all weights, 115 MB
    // for 13 MB of them at K = 5120.)
    int act_count = (a.tokens_are_rows && a.act.active) ? *a.act.count : 0;                    // computed patches
    if (FEAT & EPF_TWO) act_count = __builtin_amdgcn_readfirstlane(act_count);      // (decides which problem's pointers a block takes)
    constexpr bool PADS = (FEAT & EPF_PADS) != 0, TWO = (FEAT & EPF_TWO) != 0;
    int m_limit = (a.tokens_are_rows && a.act.active) ? act_count * a.geom.S : PADS ? gemm_rows(a) : a.M;      // rows that exist
    const int n_tiles = a.N / BN * (a.classes ? a.classes : 1), mt1 = (m_limit + BM - 1) / BM;
    const int cnt2 = TWO ? __builtin_amdgcn_readfirstlane(*a.act2.count) : 0, m_tiles = TWO ? mt1 + (cnt2 * a.geom.S + BM - 1) / BM : mt1;
    const int total = n_tiles * m_tiles, slot_step = gridDim.x >> 3;
    const int slots = (int)((int64_t)total * ((blockIdx.x & 7) + 1) / 8);      // end of this XCD's tiles
    const int gm = min(max((int)(sqrtf((float)min((total + 7) / 8, 64) * BN / BM) + 0.5f), 1), max(m_tiles, 1));
    auto decode = [&](int slot, int& m0, int& n0) {
        const int grp = slot / (gm * n_tiles), r_in = slot - grp * (gm * n_tiles);
        const int gm_here = min(gm, m_tiles - grp * gm);    // the last group may be short
        const int n_tile = r_in / gm_here;
        m0 = (grp * gm + r_in - n_tile * gm_here) * BM;
        n0 = n_tile * BN;
    };
    int m0 = 0, n0 = 0;
    int slot = (int)((int64_t)total * (blockIdx.x & 7) / 8) + (blockIdx.x >> 3);
    if (slot >= slots) return;
    decode(slot, m0, n0);
    // what differs between the problems (locals: writing to the arguments would move all of them to memory)
    const void* B = a.B;
    const float *bias_v = a.bias, *rowscale = a.rowscale;
    const int32_t* active = a.act.active;
    if constexpr (TWO) {
        if (m0 >= mt1 * BM) {
            m0 -= mt1 * BM;
            act_count = cnt2;
            m_limit = cnt2 * a.geom.S;
            B = a.B2; bias_v = a.bias2; rowscale = a.rowscale2; active = a.act2.active;
        }
    }

    // Staging by direct global -> LDS loads.  One wavefront instruction fills 64 consecutive 16-byte slots
    // (8 rows x 8 chunk positions); the lane at (row, position pos) fetches global chunk pos ^ f(row),
    // f(row) = (row >> 1) & 7, so the swizzle costs nothing.  Thread rows: lr + 32*i, position lc.
    const int lc = lane & 7, lr = 8 * wave + (lane >> 3);
    const int gc = lc ^ ((lr >> 1) & 7);            // global chunk this lane fetches (same for every i)
    int a_lane[A_LD], b_lane;                       // byte offsets of this lane's rows from the tensors' bases
    const int64_t b_row32 = (int64_t)32 * a.K;
    const int kchunks = a.K / BK;
    const int KT = a.taps * kchunks;
    const int64_t b_tap_stride = (int64_t)a.N * a.K;
    const int tap_w = a.tap_w ? a.tap_w : 3;
    int tap, kc, issued;                            // K step that is issued next (stays at the last one past the end:
                                                    // it is fetched again into a free stage and never read)

    // operand pointers and the row -> token table `tok_tab` of tile (tm0, tn0)
#define PS_SETUP(tm0, tn0, tok_tab)                                                                               \
    {                                                                                                             \
        const int cls_ = a.classes ? (tn0) / a.N : 0, nl_ = (tn0) - cls_ * a.N;      /* class, column inside it */             \
        const int ady_ = a.classes ? cls_ >> 1 : a.a_dy, adx_ = a.classes ? cls_ & 1 : a.a_dx;                    \
        const int ody_ = a.classes ? cls_ >> 1 : a.o_dy, odx_ = a.classes ? cls_ & 1 : a.o_dx;                    \
        /* the patch ids of all rows first (one memory round trip for the tile, not one per row) */              \
        int act_p[A_LD];                                                                                          \
        if (a.tokens_are_rows && a.act.active) {                                                                  \
            _Pragma("unroll") for (int i = 0; i < A_LD; ++i) {                                                    \
                const int pi = ((tm0) + lr + i * 32) / a.geom.S;                                                  \
                act_p[i] = pi < act_count ? active[pi] : -1;                                                \
            }                                                                                                     \
        }                                                                                                         \
        _Pragma("unroll") for (int i = 0; i < A_LD; ++i) {                                                        \
            const int row = lr + i * 32;                                                                          \
            int64_t tok = (tm0) + row;                                                                            \
            bool valid;                                                                                           \
            if (a.tokens_are_rows && a.act.active) {                                                              \
                const int pi = (int)tok / a.geom.S;                                                               \
                valid = act_p[i] >= 0;                                                                            \
                tok = valid ? (int64_t)act_p[i] * a.geom.S + ((int)tok - pi * a.geom.S) : 0;                      \
            } else {                                                                                              \
                valid = tok < m_limit;                                                                            \
                if (PADS && valid) {                                                                              \
                    const int g_ = (int)tok / a.row_group_pad, j_ = (int)tok - g_ * a.row_group_pad;              \
                    valid = j_ < a.row_group;                                                                     \
                    tok = g_ * a.row_group + j_;                                                                  \
                }                                                                                                 \
                if (!valid) tok = 0;                                                                              \
            }                                                                                                     \
            int64_t off, orow = tok;                                                                              \
            if (a.conv) {                                                                                         \
                const int p = (int)(tok / a.geom.S), q = (int)(tok - (int64_t)p * a.geom.S);                      \
                const int y = q / a.geom.pw, x = q - y * a.geom.pw;                                               \
                const int am = a.a_mul ? a.a_mul : 1;                                                             \
                off = ((int64_t)p * a.geom.pS + (am * y + ady_) * a.geom.ppw + am * x + adx_) * a.lda;        \
                if (a.o_mul) orow = (int64_t)p * a.o_S + (a.o_mul * y + ody_) * a.o_pw + a.o_mul * x + odx_;  \
            } else {                                                                                              \
                off = tok * a.lda;                                                                                \
            }                                                                                                     \
            a_lane[i] = (int)((off + gc * 8) * 2);                                                                \
            if (lc == 0) {                                                                                        \
                if (!a.tokens_are_rows && a.row_group > 0)                                                        \
                    orow = (tok / a.row_group) * a.row_group_pad + tok % a.row_group;                             \
                (tok_tab)[row] = valid ? (int32_t)orow : -1;                                                      \
            }                                                                                                     \
        }                                                                                                         \
        b_lane = (int)((((int64_t)cls_ * a.taps * a.N + nl_ + lr) * a.K + gc * 8) * 2);                                               \
        if constexpr (HALO) {                                                                                     \
            const int row = tid % BM, tok = min((tm0) + row, m_limit - 1);                                        \
            const int p = tok / a.geom.S, q = tok - p * a.geom.S, y = q / a.geom.pw, x = q - y * a.geom.pw;       \
            const int am = a.a_mul ? a.a_mul : 1;                                                                 \
            for (int t = tid / BM; t < a.taps; t += 256 / BM)                                                     \
                s_src[t * BM + row] = halo_offset(a, halo_token(a, p, am * y + ady_ + t / tap_w, am * x + adx_ + t % tap_w)); \
            /* the table is written; loads stay in flight */                                                      \
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");                                       \
        }                                                                                                         \
    }
#define PS_HALO_ROWS(tap_)                                                                                        \
    {                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < A_LD; ++i) a_lane[i] = s_src[(tap_) * BM + lr + i * 32] + gc * 16;  \
    }
    // one direct global->LDS load (64 lanes x 16 bytes): l < A_LD an A row group, else a B row group
    // (buffer loads rather than global loads into LDS: behind a flat-class load the compiler turns every wait for one
    // fragment into a wait for all LDS reads in flight; 2-4 % on every linear layer)
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t ga_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, HALO ? halo_bytes(a) : 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t gb_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, 0x7fffffff, 0x00020000);
#define PS_LOAD(dst_, a_off_, b_off_, l_)                                                                         \
    {                                                                                                             \
        if ((l_) < A_LD)                                                                                          \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ga_rsrc, (lds_void*)((dst_) + (l_) * 256), 16,               \
                                                     a_lane[(l_) < A_LD ? (l_) : 0], (int)((a_off_) * 2), 0, 0);  \
        else if ((l_) < LD)                                                                                       \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(gb_rsrc, (lds_void*)((dst_) + BM * CH + ((l_) - A_LD) * 256), 16, \
                                                     b_lane, (int)((((l_) - A_LD) * b_row32 + (b_off_)) * 2), 0, 0); \
    }
#else       // the host pass only needs the kernel's stub
#define PS_LOAD(dst_, a_off_, b_off_, l_) (void)0
#endif
    // global offsets of K step (tap, kc)
#define PS_OFFSETS(tap_, kc_)                                                                                     \
    const int ty_ = (tap_) / tap_w, tx_ = (tap_) - ty_ * tap_w;                                                   \
    const int64_t a_off = (a.conv && !HALO ? ((int64_t)ty_ * a.geom.ppw + tx_) * a.lda : 0) + (kc_) * BK;                  \
    const int64_t b_off = (tap_) * b_tap_stride + (kc_) * BK;
    // the first NS steps of a tile: all stages in flight
#define PS_PROLOGUE_STAGES(st0_, st1_)                                                                            \
    {                                                                                                             \
        if ((st0_) == 0) { tap = 0; kc = 0; issued = 0; }                                                         \
        _Pragma("unroll") for (int st = (st0_); st < (st1_); ++st) {                                              \
            PS_OFFSETS(tap, kc);                                                                                  \
            if constexpr (HALO) PS_HALO_ROWS(tap);                                                                \
            u32x4* dst = ring + st * STAGE_V + wave * 64;                                                         \
            _Pragma("unroll") for (int l = 0; l < LD; ++l) PS_LOAD(dst, a_off, b_off, l);                         \
            if (++issued < KT) { if (++kc == kchunks) { kc = 0; ++tap; } } else { issued = KT - 1; }              \
        }                                                                                                         \
    }
#define PS_PROLOGUE() PS_PROLOGUE_STAGES(0, NS)

    const int fr = lane & 31, fh = lane >> 5;       // fragment row within a 32-row tile, k half
    // LDS fragment slots of this lane: row*CH + ((2*ks + fh) ^ f(row))
    int fa_base[TM], fa_sw[TM], fb_base[TN], fb_sw[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) { const int r = wm * WM + i * 32 + fr; fa_base[i] = r * CH; fa_sw[i] = (r >> 1) & 7; }
#pragma unroll
    for (int j = 0; j < TN; ++j) { const int r = wn * WN + j * 32 + fr; fb_base[j] = BM * CH + r * CH; fb_sw[j] = (r >> 1) & 7; }

    bf16x8 fa[2][TM], fb[2][TN];                    // register double buffer of the MFMA fragments
    // one fragment read (16 bytes per lane) of K sub-step ks_ into register set dst; r_ = 0: A tile 0, 1 .. TN: B tiles,
    // TN+1 ..: the remaining A tiles (the order in which the MFMAs of a sub-step first need them)
#define PS_READ_ONE(dst, stage_, ks_, r_)                                                                         \
    {                                                                                                             \
        const int c_ = (ks_) * 2 + fh;                                                                            \
        const int jb_ = ((r_) >= 1 && (r_) <= TN) ? (r_) - 1 : 0;                                             \
        const int ia_ = ((r_) > TN && (r_) < TM + TN) ? (r_) - TN : 0;                                        \
        if ((r_) == 0) fa[dst][0] = __builtin_bit_cast(bf16x8, (stage_)[fa_base[0] + (c_ ^ fa_sw[0])]);           \
        else if ((r_) <= TN) fb[dst][jb_] = __builtin_bit_cast(bf16x8, (stage_)[fb_base[jb_] + (c_ ^ fb_sw[jb_])]); \
        else if ((r_) < TM + TN) fa[dst][ia_] = __builtin_bit_cast(bf16x8, (stage_)[fa_base[ia_] + (c_ ^ fa_sw[ia_])]); \
    }
    constexpr int NM = TM * TN;                     // MFMAs per 16-wide sub-step
    constexpr int NR = TM + TN;                     // fragment reads per sub-step
    constexpr int R_PER = (NR + NM - 1) / NM;       // fragment reads slipped in behind one MFMA
    constexpr int L_PER = (LD + NM - 1) / NM;       // loads slipped in behind one MFMA of sub-step 3
    constexpr bool SKIP_TAIL = NS == 2;

    int buf = 0;                                    // token table of the current tile
    PS_SETUP(m0, n0, s_tok2);
    PS_PROLOGUE();
#pragma unroll 1
    for (;;) {
        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        // stage 0 has landed when at most the NS - 1 later stages (and nothing issued after them) are in flight
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * LD) : "memory");
        __syncthreads();                            // step 0 and the token table visible to everyone
#pragma unroll
        for (int r = 0; r < NR; ++r) PS_READ_ONE(0, ring, 0, r);

        int rd = 0;                                 // ring stage of the current step
#pragma unroll 1
        for (int kt = 0; kt < KT; ++kt) {
            const u32x4* cur = ring + rd * STAGE_V;
            const int nst = rd + 1 == NS ? 0 : rd + 1;
            const u32x4* nxt = ring + nst * STAGE_V;
            PS_OFFSETS(tap, kc);                    // step kt + NS goes into this step's stage
            if constexpr (HALO) {
                if (kc == 0) PS_HALO_ROWS(tap);
            }
            if (++issued < KT) { if (++kc == kchunks) { kc = 0; ++tap; } } else { issued = KT - 1; }
            u32x4* dst = ring + rd * STAGE_V + wave * 64;
            // With two stages the barrier waits for ALL loads in flight (vmcnt(0)), so the last steps of a tile need not
            // keep the count up with loads of steps that do not exist: they issue none, and nothing is in flight when
            // the tile's epilogue starts (it used to wait out a memory round trip for them).
            const bool refill = kt + NS < KT;
#pragma unroll
            for (int ks = 0; ks < BK / 16; ++ks) {
                if (ks == BK / 16 - 1) {
                    // own fragment reads of this step are complete; own loads of the next step have landed.  A bare
                    // s_barrier: __syncthreads() carries a fence that waits for ALL loads in flight (vmcnt(0)), which
                    // would cut the ring down to one step ahead whatever its depth.
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 2) * LD) : "memory");
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks & 1][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
                        const int q = i * TN + j;
#pragma unroll
                        for (int u = 0; u < R_PER; ++u) {
                            if (ks < BK / 16 - 1) { PS_READ_ONE((ks + 1) & 1, cur, ks + 1, q * R_PER + u); }
                            else { PS_READ_ONE(0, nxt, 0, q * R_PER + u); }
                        }
                        if (ks == BK / 16 - 1 && (!SKIP_TAIL || refill)) {
#pragma unroll
                            for (int u = 0; u < L_PER; ++u) PS_LOAD(dst, a_off, b_off, q * L_PER + u);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
            rd = nst;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                            // ring drained: free for the next tile (or the epilogue's staging)
        int nm0 = 0, nn0 = 0;
        const int nslot = slot + slot_step;
        if (nslot < slots) decode(nslot, nm0, nn0);
        const int32_t* tok_cur = s_tok2 + buf * BM;
        const int n0_cur = a.classes ? n0 % a.N : n0;
        // the bias is read before the next tile's loads are issued: a wait for a load waits for all loads issued
        // before it, so a bias load behind them would stall the epilogue until the whole next tile start has landed
        float bias_t[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) bias_t[j] = bias_v ? bias_v[n0_cur + wn * WN + j * 32 + fr] : 0.f;
        asm volatile("" ::: "memory");              // keeps the compiler from sinking these loads below the next ones
        if (OVERLAP && nslot < slots) {             // next tile's first steps in flight during this tile's epilogue
            PS_SETUP(nm0, nn0, s_tok2 + (buf ^ 1) * BM);
            PS_PROLOGUE();
        } else if (HALF && nslot < slots) {         // its first step only: the epilogue stages in the stages behind it
            PS_SETUP(nm0, nn0, s_tok2 + (buf ^ 1) * BM);
            PS_PROLOGUE_STAGES(0, 1);
        }
        gemm_epilogue<BM, BN, GEGLU, WGM, WGN, (FEAT & EPF_STAT) != 0, FEAT>(a, acc, HALF ? smem + STAGE_V * 16 : ep_smem, tok_cur, n0_cur, bias_t, rowscale);
        if (nslot >= slots) break;
        if (!OVERLAP) {
            __syncthreads();                        // every wavefront is done with its staging region in the ring
            if (HALF) {
                PS_PROLOGUE_STAGES(1, NS);
            } else {
                PS_SETUP(nm0, nn0, s_tok2 + (buf ^ 1) * BM);
                PS_PROLOGUE();
            }
        }
        slot = nslot; m0 = nm0; n0 = nn0; buf ^= 1;
    }
#undef PS_READ_ONE
#undef PS_PROLOGUE
#undef PS_PROLOGUE_STAGES
#undef PS_OFFSETS
#undef PS_LOAD
#undef PS_HALO_ROWS
#undef PS_SETUP
}

// ---- 3x3 convolution with the A operand kept in LDS across the nine taps -------------------------------------
// The M tile is a set of segments, each `seg_rows` whole pixel rows of one patch.  For every 64-channel chunk
// the haloed pixels of the segments ((seg_rows+2) x (pw+2) per segment, taken from the padded patch buffer) are
// loaded into LDS ONCE and the nine taps read them as nine shifted views, so the activation traffic from L2 /
// MALL is ~5x lower than re-loading a 128-row tile per tap.  Only the weights stream per (tap, chunk) step.
// LDS: [2 weight stages][2 halo stages of CONV_APIX pixel slots][row -> token table].
struct ConvTile {
    int32_t seg_rows, seg_tokens, nseg, seg_pix;    // seg_tokens = seg_rows*pw, seg_pix = (seg_rows+2)*(pw+2)
    // ceil(2^32 / d) for d = seg_pix, pw + 2, seg_tokens, pw: x / d == __umulhi(x, m) for the small x of the set-up
    // (x * d < 2^32; a true integer division is ~40 instructions, and 28 of them sat in front of the first halo load)
    uint32_t m_seg_pix, m_hw, m_seg_tokens, m_pw;
};
struct SharedConvTile : ConvTile {
    float* ws;                                      // GemmArgs::split_ws
    int32_t splits;                                 // blocks that share a tile's channel chunks
};
__device__ __forceinline__ int div_small(int x, uint32_t m, int d) { return d == 1 ? x : (int)__umulhi((uint32_t)x, m); }

// Template: block tile BM x BN, WGM x WGN wavefront grid (4 wavefronts), APIX halo pixel slots per stage
// (multiple of 32), NSB weight stages.
// KS = 2: eight wavefronts, two per SIMD.  Wavefronts w and w + 4 own the same output rows and split every 64-wide
// K step (sub-steps 0, 1 / 2, 3); the first four fetch the weights, the last four the halo; the partial sums meet in
// LDS before the epilogue, which the first four run.
// SPLIT: the tile's channel chunks are shared by ct.splits blocks, which leave fp32 partial sums behind (compiled apart: the
// few values it keeps across the loop cost the other form 5 %).
template <int BM, int BN, int WGM, int WGN, int APIX, int NSB, int KS, bool SPLIT>
__global__ void __launch_bounds__(256 * KS)
conv_mfma_kernel(GemmCore a, std::conditional_t<SPLIT, SharedConvTile, ConvTile> ct) {
    constexpr int BK = 64, CH = 8;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int B_LD = BN * CH / 256, A_LD = APIX * CH / 256;
    constexpr int BSTAGE = BN * CH, ASTAGE = APIX * CH;            // 16-byte slots
    static_assert(WGM * WGN == 4 && (BN * CH) % 256 == 0 && (APIX * CH) % 256 == 0 && (NSB == 2 || NSB == 3), "conv tile");
    static_assert(KS == 1 || KS == 2, "K split");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    u32x4* sB = reinterpret_cast<u32x4*>(smem);                    // [NSB][BSTAGE]
    u32x4* sA = sB + NSB * BSTAGE;                                 // [2][ASTAGE]
    int32_t* s_tok = reinterpret_cast<int32_t*>(sA + 2 * ASTAGE);  // [BM]
    int32_t* s_seg = s_tok + BM;                                   // [nseg] padded-pixel index of each segment's halo origin

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: LDS destinations of the loads are SGPR math
    const int wave = wave_all & 3, kg = KS == 1 ? 0 : wave_all >> 2;    // place in the wavefront grid, K group
    const bool pro_b = kg == 0, pro_a = kg == KS - 1;            // who issues the first weight stages / the first halo
    const int wm = wave / WGN, wn = wave % WGN;
    // XCD-aware tile order: block ids are dealt round-robin to the 8 XCDs, so all N tiles of one M tile get ids of
    // the same residue mod 8 and consecutive slots: they run on one XCD back to back and share the A tile in its L2
    const int n_tiles = a.N / BN, m_tiles = (a.M + BM - 1) / BM;
    const int slot = blockIdx.x >> 3;
    int m_tile = (slot / n_tiles) * 8 + (blockIdx.x & 7), n_tile = slot % n_tiles, part = 0;
    if constexpr (SPLIT) {
        // shared tiles: an XCD takes all M tiles of a (column tile, share of the chunks), whose weights it then fetches once
        const int unit = (slot / m_tiles) * 8 + (blockIdx.x & 7);
        if (unit >= n_tiles * ct.splits) return;
        m_tile = slot % m_tiles;
        n_tile = unit % n_tiles;
        part = unit / n_tiles;
    }
    if (m_tile >= m_tiles) return;
    const int m0 = m_tile * BM, n0 = n_tile * BN;
    if (a.act.active && m0 >= *a.act.count * a.geom.S) return;
    const int S = a.geom.S, pw = a.geom.pw, hw = pw + 2;

    // one direct global->LDS load (64 lanes x 16 bytes) of the weight / halo stage
    // Buffer loads into LDS rather than global loads into LDS: behind a flat-class load the compiler takes the LDS
    // counter for out of order and turns every wait for ONE fragment into a wait for all reads in flight
    // (lgkmcnt(0)), the read issued an instruction earlier included; behind buffer loads it counts (lgkmcnt(4..0)
    // down a row of MFMAs): 498 -> 487 us at C = 640 on 79 k rows, 374 -> 358 us at C = 1280.  Offsets are 32-bit
    // byte offsets from the tensor's base (the launch checks that both tensors stay below 2^31 bytes).
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.B, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, 0x7fffffff, 0x00020000);
#define PS_LOAD_B(dstB_, off_, i_) \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, (lds_void*)((dstB_) + (i_) * 256), 16, b_lane, (int)(((i_) * b_row32 + (off_)) * 2), 0, 0)
#define PS_LOAD_A(dstA_, off_, i_) \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void*)((dstA_) + (i_) * 256), 16, a_pos[i_], (int)((off_) * 2), 0, 0)
#else       // the host pass only needs the kernel's stub
#define PS_LOAD_B(dstB_, off_, i_) (void)0
#define PS_LOAD_A(dstA_, off_, i_) (void)0
#endif

    // The weights of the first NSB steps go first: they need no table, and the index arithmetic below runs while
    // they are in flight.  Thread rows lr + 32*i, chunk position lc; the lane fetches global chunk lc ^ f(row).
    const int lc = lane & 7, lr = 8 * wave + (lane >> 3);
    const int gc = lc ^ ((lr >> 1) & 7);
    const int b_lane = (int)(((int64_t)(n0 + lr) * a.K + gc * 8) * 2);   // byte offset of this lane's first weight row
    const int64_t b_row32 = (int64_t)32 * a.K;
    const int64_t b_tap_stride = (int64_t)a.N * a.K;
    int kbase = 0, kchunks = a.K / BK;              // first channel chunk of this block, and their number
    if constexpr (SPLIT) {
        kbase = a.K / BK * part / ct.splits;
        kchunks = a.K / BK * (part + 1) / ct.splits - kbase;
    }
    int itap = 0, ikc = 0;                          // (tap, chunk) of the next weight stage to issue; clamps at the last step
#pragma unroll
    for (int t = 0; t < NSB; ++t) {
        u32x4* dB = sB + t * BSTAGE + wave * 64;
        const int64_t off = itap * b_tap_stride + (kbase + ikc) * BK;
        if (pro_b) {
#pragma unroll
            for (int i = 0; i < B_LD; ++i) PS_LOAD_B(dB, off, i);
        }
        if (!(itap == 8 && ikc == kchunks - 1)) { if (++itap == 9) { itap = 0; ++ikc; } }
    }

    // row -> token table and segment origins
    if (tid < BM) {
        const int ri = m0 + tid;
        int64_t tok;
        bool valid;
        if (a.act.active) {
            const int pi = ri / S;
            valid = pi < *a.act.count;
            tok = valid ? (int64_t)a.act.active[pi] * S + (ri - pi * S) : 0;
        } else {
            valid = ri < a.M;
            tok = valid ? ri : 0;
        }
        s_tok[tid] = valid ? (int32_t)tok : -1;
        if (tid % ct.seg_tokens == 0) {
            const int p = (int)(tok / S), q = (int)(tok - (int64_t)p * S);
            s_seg[tid / ct.seg_tokens] = p * a.geom.pS + (q / pw) * a.geom.ppw;    // padded pixel of halo (0, 0)
        }
    }
    __syncthreads();

    const uint16_t* A = (const uint16_t*)a.A;
    int32_t a_pos[A_LD];                            // byte offsets (the launch checks that the padded buffer stays below 2^31 bytes)
    const int apix = ct.nseg * ct.seg_pix;
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        int sl = lr + 32 * i;
        if (sl >= apix) sl = 0;                                    // unused slots re-read a valid pixel
        const int g = div_small(sl, ct.m_seg_pix, ct.seg_pix), l = sl - g * ct.seg_pix;
        const int ly = div_small(l, ct.m_hw, hw), lx = l - ly * hw;
        a_pos[i] = ((s_seg[g] + ly * a.geom.ppw + lx) * (int32_t)a.lda + gc * 8) * 2;
    }
    if (pro_a) {                                    // halo of chunk 0: in flight during the rest of the set-up
        u32x4* dA = sA + wave * 64;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) PS_LOAD_A(dA, kbase * BK, i);
    }
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;


    const int fr = lane & 31, fh = lane >> 5;
    // halo slot of each fragment row for tap (0, 0)
    int fa_slot[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = wm * WM + i * 32 + fr;
        const int g = div_small(r, ct.m_seg_tokens, ct.seg_tokens), rr = r - g * ct.seg_tokens;
        const int ry = div_small(rr, ct.m_pw, pw), rx = rr - ry * pw;
        fa_slot[i] = g * ct.seg_pix + ry * hw + rx;
    }
    // weight fragment j: row wn*WN + 32*j + fr; the chunk swizzle (row >> 1) & 7 is the same for every j
    const int fb_base0 = (wn * WN + fr) * CH, fb_sw0 = ((wn * WN + fr) >> 1) & 7;

    // fragment registers: two sets, filled one sub-step ahead.  With the K split (256 registers per wavefront) the
    // weight fragments have one set: fb[j] is refilled right behind the last MFMA of the sub-step that reads it.
    constexpr int FBS = KS == 1 ? 2 : 1;
    bf16x8 fa[2][TM], fb[FBS][TN];
    // one fragment read (16 bytes per lane) of K sub-step ks_ into register set dst; r_ = 0: A tile 0, 1 .. TN: B tiles,
    // TN+1 ..: the remaining A tiles (the order in which the MFMAs of a sub-step first need them)
#define PS_READ_ONE(dst, stA_, stB_, cur_, sw_, ks_, r_)                                                          \
    {                                                                                                             \
        const int c_ = ((ks_) + koff) * 2 + fh;                                                                   \
        const int jb_ = ((r_) >= 1 && (r_) <= TN) ? (r_) - 1 : 0;                                             \
        const int ia_ = ((r_) > TN && (r_) < TM + TN) ? (r_) - TN : 0;                                        \
        if ((r_) == 0) fa[dst][0] = __builtin_bit_cast(bf16x8, (stA_)[cur_[0] * CH + (c_ ^ sw_[0])]);             \
        else if ((r_) <= TN) fb[(dst) & (FBS - 1)][jb_] = __builtin_bit_cast(bf16x8, (stB_)[fb_base0 + jb_ * 32 * CH + (c_ ^ fb_sw0)]); \
        else if ((r_) < TM + TN) fa[dst][ia_] = __builtin_bit_cast(bf16x8, (stA_)[cur_[ia_] * CH + (c_ ^ sw_[ia_])]); \
    }

    constexpr int NM = TM * TN;                     // MFMAs per 16-wide sub-step
    constexpr int NR = TM + TN;                     // fragment reads per sub-step
    constexpr int R_PER = (NR + NM - 1) / NM;       // fragment reads slipped in behind one MFMA
    constexpr int SUB = BK / 16 / KS;               // sub-steps of a step one wavefront computes
    constexpr int A_PER = (A_LD + (SUB - 1) * NM - 1) / ((SUB - 1) * NM);   // halo loads slipped in per MFMA before the last sub-step
    static_assert(B_LD <= NM, "weight loads are interleaved one per MFMA");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // The loop comes in three forms, chosen per wavefront: 0 = no K split (all sub-steps, both kinds of loads),
    // 1 = first half of every step + the weight loads, 2 = second half + the halo loads.
    auto main_loop = [&](auto role_c) {
        constexpr int ROLE = decltype(role_c)::value;
        constexpr bool issue_b = ROLE != 2, issue_a = ROLE != 1;
        constexpr int koff = ROLE == 2 ? SUB : 0;       // first sub-step of this wavefront
        // MFMAs of a step's last sub-step that a wavefront issues IN FRONT of the block barrier (K split only).  With the
        // barrier at the head of the sub-step a wavefront reaches it right behind its last fragment reads and waits out
        // their LDS latency there.  A few MFMAs later the reads have landed: those MFMAs take fragments read a
        // sub-step earlier, and everything that must follow the barrier (the next step's first fragments, the refill
        // of this step's weight stage) moves behind the remaining MFMAs.  Different slots for the two K groups keep the
        // two wavefronts of a SIMD from reaching their sub-step boundaries together.  Worth 3 % while every wait for a
        // fragment was a wait for all reads in flight (see the loads above), about 1 % since.
        constexpr int QB = KS == 1 ? 0 : (ROLE == 1 ? 2 : 5);
        static_assert(QB + B_LD <= NM && QB + TM <= NM && QB <= NM - TN, "barrier slot");
        int fa_cur[TM], fa_sw[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) { fa_cur[i] = fa_slot[i]; fa_sw[i] = (fa_cur[i] >> 1) & 7; }
#pragma unroll
        for (int r = 0; r < NR; ++r) PS_READ_ONE(0, sA, sB, fa_cur, fa_sw, 0, r);

        // Step = (chunk kc, tap): 4 sub-steps of NM MFMAs.  Every memory instruction rides behind an MFMA: during
        // sub-steps 0..2 the fragment reads of the next sub-step (and, in tap 0, the halo of the next chunk), during
        // sub-step 3 the first fragments of the NEXT step and the refill of this step's weight stage.  The block barrier
        // sits in sub-step 3 (at its head, or QB MFMAs into it): by then every wavefront has read all of this step's
        // fragments (its stage is free) and has seen its own loads of the next step's weights land.
        int bst = 0;                                    // weight stage of the current step
        // The two wavefronts of a SIMD compete for the matrix pipe, and the older one (the first K group) wins every
        // time both have an MFMA ready: it runs ahead to the barrier and waits there a third of the loop's time
        // (timestamps of a work build) while the second group finishes the step on its own.  With the second group
        // at the higher priority the first one fills the gaps instead: 1-2 % (347 -> 339 us at C = 1280).
        if (ROLE == 2) asm volatile("s_setprio 2" ::: "memory");
        for (int kc = 0; kc < kchunks; ++kc) {
            const u32x4* curA = sA + (kc & 1) * ASTAGE;
            const int nkc_a = kc + 1 < kchunks ? kc + 1 : kc;   // halo chunk fetched during tap 0 (last: itself, never read)
            u32x4* dA = sA + ((kc & 1) ^ 1) * ASTAGE + wave * 64;
            const int a_off = (kbase + nkc_a) * BK;
#pragma unroll 1
            for (int tap = 0; tap < 9; ++tap) {
                const u32x4* curB = sB + bst * BSTAGE;
                const int nst = bst + 1 == NSB ? 0 : bst + 1;
                const u32x4* nxtB = sB + nst * BSTAGE;
                const int ntap = tap == 8 ? 0 : tap + 1;
                const u32x4* nxtA = tap == 8 ? sA + ((kc & 1) ^ 1) * ASTAGE : curA;
                const int nty = ntap / 3, ntx = ntap - nty * 3;
                int nfa_cur[TM], nfa_sw[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i) { nfa_cur[i] = fa_slot[i] + nty * hw + ntx; nfa_sw[i] = (nfa_cur[i] >> 1) & 7; }
                const int64_t b_off = itap * b_tap_stride + (kbase + ikc) * BK;
                if (!(itap == 8 && ikc == kchunks - 1)) { if (++itap == 9) { itap = 0; ++ikc; } }
                u32x4* dB = sB + bst * BSTAGE + wave * 64;
#pragma unroll
                for (int ks = 0; ks < SUB; ++ks) {
                    auto step_barrier = [&] {
                        // own fragment reads of this step are complete; own loads of the next step's weights have landed.
                        // Still allowed in flight: the NSB-2 later weight stages and a halo issued in this or a recent tap 0.
                        // A bare s_barrier: __syncthreads() carries a fence that waits for ALL loads in flight (vmcnt(0)),
                        // which would cut the weight ring down to one step ahead whatever its depth.
                        // With the K split a wavefront waits for the kind it fetches: weights as above, or the halo (needed
                        // from tap 8 on, issued in tap 0).
                        if (KS == 1 ? tap < NSB - 1 : (!issue_b && tap == 0))
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((KS == 1 ? (NSB - 2) * B_LD : 0) + A_LD) : "memory");
                        else if (KS == 1 || issue_b)
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NSB - 2) * B_LD) : "memory");
                        else
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
                    };
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const int q = i * TN + j;
                            if (ks == SUB - 1 && q == QB) step_barrier();
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks & 1][i], fb[ks & (FBS - 1)][j], acc[i][j], 0, 0, 0);
                            if (KS == 1) {
#pragma unroll
                                for (int u = 0; u < R_PER; ++u) {
                                    if (ks < SUB - 1) { PS_READ_ONE((ks + 1) & 1, curA, curB, fa_cur, fa_sw, ks + 1, q * R_PER + u); }
                                    else { PS_READ_ONE(0, nxtA, nxtB, nfa_cur, nfa_sw, 0, q * R_PER + u); }
                                }
                            } else {
                                // A fragments of the next sub-step behind the first TM MFMAs (other register set), B fragment j
                                // behind the last MFMA that reads the current one (i == TM - 1)
                                const int r = q < TM ? (q == 0 ? 0 : TN + q) : (i == TM - 1 ? 1 + j : NR);
                                if (ks < SUB - 1) { PS_READ_ONE((ks + 1) & 1, curA, curB, fa_cur, fa_sw, ks + 1, r); }
                                else {
                                    // behind the barrier only: the A fragments from slot QB on, B fragment j where it was
                                    const int qa = q - QB;
                                    const int ra = (qa >= 0 && qa < TM) ? (qa == 0 ? 0 : TN + qa) : NR;
                                    const int rb = i == TM - 1 ? 1 + j : NR;
                                    PS_READ_ONE(0, nxtA, nxtB, nfa_cur, nfa_sw, 0, ra);
                                    PS_READ_ONE(0, nxtA, nxtB, nfa_cur, nfa_sw, 0, rb);
                                }
                            }
                            if (ks == SUB - 1) {
                                if (q >= QB && q < QB + B_LD && issue_b) PS_LOAD_B(dB, b_off, q - QB);
                            } else {
#pragma unroll
                                for (int u = 0; u < A_PER; ++u) {
                                    const int qa = (ks * NM + q) * A_PER + u;
                                    if (qa < A_LD && tap == 0 && issue_a) PS_LOAD_A(dA, a_off, qa);
                                }
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                }
#pragma unroll
                for (int i = 0; i < TM; ++i) { fa_cur[i] = nfa_cur[i]; fa_sw[i] = nfa_sw[i]; }
                bst = nst;
            }
        }
    };
    if (KS == 1) main_loop(std::integral_constant<int, 0>{});
    else if (kg == 0) main_loop(std::integral_constant<int, 1>{});
    else main_loop(std::integral_constant<int, 2>{});
#undef PS_READ_ONE
#undef PS_LOAD_A
#undef PS_LOAD_B
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // The lane's bias of each tile column, loaded here in one batch: inside the epilogue the load of a column sits
    // behind the staging of the previous one (a memory round trip per column); here it hides behind the exchange
    // (1.5 us of a 60 us kernel).
    float bias_t[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bias_t[j] = a.bias ? a.bias[n0 + wn * WN + j * 32 + fr] : 0.f;
    if (KS == 2) {
        // the partial sums of wavefront w + 4 go to wavefront w through the drained ring, half the tile columns at a
        // time; the first four wavefronts then run the epilogue
        constexpr int JH = (TN + 1) / 2;
        static_assert(KS == 1 || 4 * JH * TM * 16 * 64 * 4 <= (NSB * BSTAGE + 2 * ASTAGE) * 16, "exchange does not fit the ring");
        f32x4* xch = reinterpret_cast<f32x4*>(smem) + wave * (JH * TM * 4 * 64) + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j0 = h * JH, j1 = h ? TN : JH;
            if (kg == 1) {
#pragma unroll
                for (int j = j0; j < j1; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                            xch[(((j - j0) * TM + i) * 4 + q) * 64] = v;
                        }
            }
            __syncthreads();
            if (kg == 0) {
#pragma unroll
                for (int j = j0; j < j1; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 v = xch[(((j - j0) * TM + i) * 4 + q) * 64];
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
                        }
            }
            __syncthreads();
        }
        if (kg == 1) return;
    }
    if constexpr (SPLIT) {
        // fp32 partial sums [share][row of the tile grid][N]: 128 contiguous bytes per row and store
        float* dst = ct.ws + ((int64_t)part * (m_tiles * BM) + m0 + wm * WM + 4 * fh) * a.N + n0 + wn * WN + fr;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float* row = dst + (int64_t)(i * 32 + 8 * (e >> 2) + (e & 3)) * a.N;
#pragma unroll
                for (int j = 0; j < TN; ++j) row[j * 32] = acc[i][j][e];
            }
        return;
    }
    // the launch conditions of these kernels rule the other paths out (conv_select)
    gemm_epilogue<BM, BN, false, WGM, WGN, true, 0>(a, acc, smem, s_tok, n0, bias_t, nullptr);
}

// Second half of a convolution whose tiles were shared: sums the partial tiles in a fixed order, adds the bias (and the
// request's), leaves the next norm's moments behind (column sums of 64 rows, exact two-pass form) and adds the residual.
// A block is 64 rows x W columns (whole groups of the norm): 16 row lanes x W / 8 column vectors, four rows a thread.
// Memory bound: (4 x splits + 2 (+ 2 with a residual)) bytes per output.
constexpr int SPLIT_RL = 16;
__global__ void __launch_bounds__(256)
split_reduce_kernel(GemmArgs a, int splits, int m_pad, int W) {
    const int cvs = W / 8, tid = threadIdx.x, cv = tid % cvs, rl = tid / cvs;
    const int n0 = blockIdx.y * W, col = n0 + cv * 8, m0 = blockIdx.x * 64;
    __shared__ float s_part[SPLIT_RL][128];
    __shared__ float s_grp[64];
    const int cnt = a.act.active ? *a.act.count * a.geom.S : a.M;
    if (m0 >= cnt) return;
    const bool in = col < a.N;                      // (the last slab may be narrower; the threads stay for the barriers)
    const int colc = in ? col : 0;
    float v[4][8];
    int64_t tok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = m0 + rl + SPLIT_RL * r;
        tok[r] = -1;
        if (row < cnt) {
            tok[r] = row;
            if (a.act.active) { const int pi = row / a.geom.S; tok[r] = (int64_t)a.act.active[pi] * a.geom.S + (row - pi * a.geom.S); }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) v[r][q] = 0.f;
    }
    const float* src = a.split_ws + (int64_t)(m0 + rl) * a.N + colc;     // rows up to the next multiple of 64 exist in the scratch
    for (int z = 0; z < splits; ++z) {
        f32x4 lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* p = src + ((int64_t)z * m_pad + SPLIT_RL * r) * a.N;
            lo[r] = *reinterpret_cast<const f32x4*>(p);
            hi[r] = *reinterpret_cast<const f32x4*>(p + 4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) { v[r][q] += lo[r][q]; v[r][4 + q] += hi[r][q]; }
    }
    float bias[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) bias[q] = a.bias ? a.bias[colc + q] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float* rb = a.rowbias && tok[r] >= 0 ? a.rowbias + (int64_t)a.row_owner[tok[r] / a.geom.S] * a.N + colc : nullptr;
#pragma unroll
        for (int q = 0; q < 8; ++q) v[r][q] += bias[q] + (rb ? rb[q] : 0.f);
    }
    if (a.stats) {                                  // all 64 rows exist and lie in one patch (gemm_stats_rows)
        const int cg = a.N / a.stats_G, groups = W / cg;
        float mean[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) mean[q] = 0.f;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {      // sums, then squared deviations from the group's mean
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float s = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) { const float d = v[r][q] - mean[q]; s += pass ? d * d : d; }
                s_part[rl][cv * 8 + q] = s;
            }
            __syncthreads();
            if (tid < W) {                          // column sums over the row lanes
                float s = 0.f;
#pragma unroll
                for (int r = 0; r < SPLIT_RL; ++r) s += s_part[r][tid];
                s_part[0][tid] = s;
            }
            __syncthreads();
            if (tid < groups) {
                float s = 0.f;
                for (int c = 0; c < cg; ++c) s += s_part[0][tid * cg + c];
                if (!pass) s_grp[tid] = s / (64.f * cg);
                else if (n0 + tid * cg < a.N) {
                    const int p = m0 / a.geom.S, slot = (m0 - p * a.geom.S) / 64;
                    float* dst = a.stats + (((int64_t)p * a.stats_slots + slot) * a.stats_G + n0 / cg + tid) * 2;
                    dst[0] = s_grp[tid];
                    dst[1] = s;
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 8; ++q) mean[q] = s_grp[(cv * 8 + q) / cg];
        }
    }
    if (!in) return;
    const int sg = col / a.seg_cols;
    const GemmSeg seg = sg == 0 ? a.seg[0] : (sg == 1 ? a.seg[1] : a.seg[2]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (tok[r] < 0) continue;
        if (a.res) {
            const u32x4 x = *reinterpret_cast<const u32x4*>((const uint16_t*)a.res + tok[r] * a.ldr + col);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[r][2 * q] += __uint_as_float(x[q] << 16);
                v[r][2 * q + 1] += __uint_as_float(x[q] & 0xFFFF0000u);
            }
        }
        u32x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = pack_bf16x2(v[r][2 * q], v[r][2 * q + 1]);
        *reinterpret_cast<u32x4*>((uint16_t*)seg.ptr + tok[r] * seg.ld + col - sg * a.seg_cols) = o;
    }
}

// Columns of a block of split_reduce_kernel: whole groups of cg channels and whole vectors of 8, about 64, at most 128.
static int split_slab(int cg) {
    int unit = 8;
    while (unit % cg != 0 && unit <= 128) unit += 8;
    return unit > 128 ? 0 : unit >= 64 ? unit : unit * ((63 + unit) / unit);
}

// Blocks that share a tile: as many as the chip has CUs for, in equal shares of the channel chunks; only where less than
// half of the CUs would have a tile (each share writes and reads back 4 bytes per output: at half the chip the second
// pass would cost what the split saves).
static int conv_splits(int64_t tiles, int64_t kchunks) {
    if (tiles * 2 > 256 || kchunks < 2) return 1;
    const int64_t z = std::min<int64_t>(256 / tiles, kchunks), share = cdiv(kchunks, z);
    // the second pass is a launch of ~5 us; a chunk is nine steps of ~0.6 us
    return kchunks - share < 2 ? 1 : (int)cdiv(kchunks, share);
}

template <int BM, int BN, int WGM, int WGN, int APIX, int NSB, int KS = 1>
static int launch_conv(const GemmArgs& a, const ConvTile& ct, int splits, hipStream_t st) {
    constexpr size_t lds = (size_t)(NSB * BN + 2 * APIX) * 128 + BM * sizeof(int32_t) + 64 * sizeof(int32_t);
    static_assert(lds <= 160 * 1024, "conv LDS budget");
    const int64_t mt = cdiv(a.M, BM), nt = a.N / BN;
    const int slab = split_slab(a.stats ? a.N / a.stats_G : 8);
    if (splits == 1 || !a.split_ws || a.split_ws_bytes < sizeof(float) * splits * mt * BM * a.N || slab == 0) {
        PS_SET_LDS_ONCE((conv_mfma_kernel<BM, BN, WGM, WGN, APIX, NSB, KS, false>), lds);
        conv_mfma_kernel<BM, BN, WGM, WGN, APIX, NSB, KS, false><<<(unsigned)(8 * cdiv(mt, 8) * nt), 256 * KS, lds, st>>>(a, ct);
        return check_launch("conv_mfma_kernel");
    }
    PS_SET_LDS_ONCE((conv_mfma_kernel<BM, BN, WGM, WGN, APIX, NSB, KS, true>), lds);
    conv_mfma_kernel<BM, BN, WGM, WGN, APIX, NSB, KS, true><<<(unsigned)(8 * cdiv(nt * splits, 8) * mt), 256 * KS, lds, st>>>(
        a, SharedConvTile{ct, a.split_ws, splits});
    PS_TRY(check_launch("conv_mfma_kernel"));
    split_reduce_kernel<<<dim3((unsigned)cdiv(a.M, 64), (unsigned)cdiv(a.N, slab)), SPLIT_RL * slab / 8, 0, st>>>(
        a, splits, (int)(mt * BM), slab);
    return check_launch("split_reduce_kernel");
}

// Tile geometry of the halo-in-LDS convolution; false if the patch shape does not fit it.
static bool conv_tile(const GemmArgs& a, int BM, int apix_max, ConvTile* ct) {
    const int pw = a.geom.pw, ph = a.geom.ph;
    if (!a.conv || !a.tokens_are_rows || a.taps != 9 || BM % pw != 0) return false;
    int R = BM / pw;
    if (R > ph) R = ph;
    if (ph % R != 0 || BM % (R * pw) != 0) return false;
    ct->seg_rows = R;
    ct->seg_tokens = R * pw;
    ct->nseg = BM / ct->seg_tokens;
    ct->seg_pix = (R + 2) * (pw + 2);
    auto magic = [](int d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };      // d == 1 is handled apart
    ct->m_seg_pix = magic(ct->seg_pix);
    ct->m_hw = magic(pw + 2);
    ct->m_seg_tokens = magic(ct->seg_tokens);
    ct->m_pw = magic(pw);
    return ct->nseg * ct->seg_pix <= apix_max && ct->nseg <= 64;
}

template <int BM, int BN, bool GEGLU, int WGM, int WGN, int NS, bool OVERLAP, int FEAT>
static int launch_feat(const GemmArgs& a, hipStream_t st) {
    constexpr size_t sums = FEAT & EPF_STAT ? 4 * (2 * (BN / WGN) + 2) * sizeof(float) : 0;         // behind the epilogue's staging
    constexpr size_t lds = GemmCfg<BM, BN, NS, OVERLAP>::LDS + (FEAT & EPF_HALO ? 9 * BM * sizeof(int32_t) : 0) + (OVERLAP ? sums : 0);
    static_assert(OVERLAP || NS * GemmCfg<BM, BN, NS, OVERLAP>::STAGE - GemmCfg<BM, BN, NS, OVERLAP>::STAGE * ((NS - 1) * (BM + BN) * 128 >= 4 * (BM / WGM) * 144) >=
                  4 * (BM / WGM) * 144 + sums, "epilogue staging and sums do not fit the stages they lie in");
    static_assert(lds <= 160 * 1024, "LDS");
    PS_SET_LDS_ONCE((gemm_mfma_kernel<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, FEAT>), lds);
    // all tiles, or as many blocks as run at once (256 CUs x the blocks of this LDS size per CU): each block then
    // walks over several tiles
    const int64_t m_tiles = cdiv(FEAT & EPF_PADS ? gemm_rows(a) : a.M, BM) + (FEAT & EPF_TWO ? cdiv(a.M2, BM) : 0);
    const int64_t all = 8 * cdiv(m_tiles * (a.N / BN) * std::max(1, a.classes), 8);
    const int64_t resident = FEAT & EPF_TWO ? all : 256 * (int64_t)std::max<size_t>(1, std::min<size_t>(2, (160 * 1024) / lds));
    const unsigned grid = (unsigned)std::min(all, resident);
    gemm_mfma_kernel<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, FEAT><<<grid, 256, lds, st>>>(a);
    return check_launch("gemm_mfma_kernel");
}

// The end of a tile without the paths that this problem does not take, against all of them: 22.7 -> 21.7 us (13,312 x 640 x
// 640), 112 -> 107 us (78,848 x 640 x 640) on 128 x 160 tiles, 345 -> 312 (78,848 x 1,920 x 640, 256 x 128), 39.4 -> 34.8
// (13,312 x 640 x 640, 256 x 128).  Not for 128 x 64 tiles, which get slower by it (1,024 x 1,280, plain / all paths: with
// residual K = 1,280 14.0 / 12.3 and 14.9 / 12.3, K = 5,120 31.1 / 30.5; scaled queries 12.7 / 11.6; q, k and v 20.5 / 19.6).
// GEGLU has the one segment, neither transposed nor scaled.
template <int BM, int BN, bool GEGLU, int WGM, int WGN, int NS, bool OVERLAP>
static int launch(const GemmArgs& a, hipStream_t st) {
    bool seg = false;
    for (const GemmSeg& s : a.seg) seg |= s.transposed || s.scale != 1.f;
    if constexpr (GEGLU) {
        PS_REQUIRE(!seg, "gemm: GEGLU has no transposed or scaled output");
        return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, 0>(a, st);
    } else {
        if (gemm_pads_rows(a)) return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, EPF_TRANS | EPF_SCALE | EPF_PADS>(a, st);
        if (a.halo_src) return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, EPF_HALO>(a, st);
        if (a.stats) return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, EPF_STAT>(a, st);       // (gemm_stats_rows)
        if constexpr (BN != 64) {
            // (a request's bias needs no look-up per row where a wavefront's rows lie in one patch)
            if ((!a.rowbias || (a.tokens_are_rows && a.geom.S % (BM / WGM) == 0)) && !a.rowscale && !a.act_gelu) {
                if (seg) return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, EPF_TRANS | EPF_SCALE>(a, st);
                return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, 0>(a, st);
            }
        }
        return launch_feat<BM, BN, GEGLU, WGM, WGN, NS, OVERLAP, EPF_ALL>(a, st);
    }
}

// Which halo-in-LDS convolution kernel a problem takes (0: none).
// Preferred: 256 x 160 tiles, four wavefronts stacked along M (each 64 x 160), three weight stages: half the weight
// bytes per MFMA of the 128 x 320 tile at the same accumulator shape.  That tile runs with the K split (eight
// wavefronts): 66 instead of 70 us at C = 320 / 29,696 tokens, 541 instead of 576 us at C = 640 / about 79,000 tokens.
static int conv_select(const GemmArgs& a, ConvTile* ct) {
    int sel = 0;
    const bool plain3x3 = a.taps == 9 && (a.tap_w == 0 || a.tap_w == 3) && a.a_mul <= 1 && !a.a_dy && !a.a_dx && !a.o_mul;
    // no gate, no GELU, no transposed segment; a per-request bias only where a wavefront's 64 rows lie in one patch (the
    // kernels compile the epilogue without those paths)
    const bool lean = a.seg[0].scale == 1.f && !a.rowscale && !a.act_gelu && (!a.rowbias || (a.geom.S % 64 == 0 && a.geom.pw <= 64 && 64 % a.geom.pw == 0));
    if (plain3x3 && gemm_fits32(a) && lean && a.epi == EPI_ROUTE && a.seg_cols % 32 == 0 && a.seg_cols == a.N && !a.seg[0].transposed) {
        if (a.N % 160 == 0 && conv_tile(a, 256, 384, ct)) sel = 1;
        // small patches (8 x 8: four segments of 10 x 10 pixels per 256 rows) need more halo slots than that tile's LDS
        // has beside three weight stages; with two weight stages 416 slots fit
        else if (a.N % 160 == 0 && conv_tile(a, 256, 416, ct)) sel = 6;
        else if (conv_tile(a, 128, 256, ct)) {
            if (a.N % 320 == 0) sel = 2;
            else if (a.N % 256 == 0) sel = 3;
            else if (a.N % 128 == 0) sel = 4;
            else if (a.N % 64 == 0) sel = 5;
        }
    }
    return sel;
}

int few_pick(const GemmArgs& a, int most_rounds, double* us);            // gemm_few.hip
int gemm_few_bf16(const GemmArgs& a, int tile, hipStream_t st);

static constexpr int CONV_BM[7] = {0, 256, 128, 128, 128, 128, 256}, CONV_BN[7] = {1, 160, 320, 256, 128, 64, 160};

// How long the halo-in-LDS kernel `sel` takes, in us (a step is a tap of a 64-channel chunk, slower the more of the chip is at it; a
// shared tile's sums are written and read back), and in how many shares of the channel chunks it does.  Fitted to 150 measured sizes
// (within a tenth).
static double conv_time(const GemmArgs& a, int sel, int* splits) {
    static const double step[7] = {0, 0.95, 0.95, 0.93, 0.6, 0.49, 0.95};
    const int64_t tiles = cdiv(a.M, CONV_BM[sel]) * (a.N / CONV_BN[sel]), chunks = a.K / 64, rounds = cdiv(tiles, 256);
    const int z = conv_splits(tiles, chunks);
    // (a shared tile's blocks go to the XCDs by column tile and share, all row tiles of one to the same 32 CUs: 3,072 x 640, 48 tiles x 5
    // 48.7 + 11.7 us, 4,096 x 640, 64 x 4 39.6 + 12)
    const int64_t xcd_rounds = cdiv(cdiv(a.N / CONV_BN[sel] * z, 8) * cdiv(a.M, CONV_BM[sel]), 32);
    const double whole = CONV_BM[sel] == 256 ? rounds * 12.0 + 9 * chunks * (0.6 * rounds + 0.42 * tiles / 256) : rounds * (5.0 + 9 * chunks * step[sel]);
    const double shared = 11.0 + 9 * cdiv(chunks, z) * step[sel] * xcd_rounds + 1.5e-6 * z * (double)a.M * a.N;
    *splits = z > 1 && shared < whole ? z : 1;
    return *splits > 1 ? shared : whole;
}

// 128 x 128 tiles with three stages, one block a CU, in place of t64 tiles of 128 x 64 that have CUs with two: where the chain of steps is long.
// us, 128 x 64 / these, narrow tiles 264 / 342 / 408 / 504:
//   linear layers  K = 2,048 22.1 / 21.6, 23.2 / 22.3, 23.5 / 22.9, 25.8 / 24.7;  K = 2,560 28.1 / 25.5, 30.0 / 25.9, 29.7 / 26.6, 32.0 / 28.8;
//     K = 4,608 42.9 / 38.7, 45.3 / 39.2, 45.2 / 40.6, 49.2 / 44.2;  K = 6,144 58.5 / 49.4, 61.3 / 49.7, 61.7 / 51.0, 66.3 / 55.3.
//     With a gate, or a transposed segment, K = 2,048 is a tie (300 tiles 23.1 / 23.6, 22.1 / 22.3); 2,176 26.2 / 24.4, 25.9 / 24.0.
//   rows of several requests in a wavefront (64 x 64 values a look-up each, not 64 x 32): 342 tiles, patches of 20 x 20, K = 2,048 29.0 / 35.3,
//     4,608 50.5 / 52.1 (in a block 51.6 / 57.1), 6,144 66.2 / 62.7.
//   3x3 convolutions  256 channels 25.7 / 26.5, 26.6 / 27.0, 27.1 / 27.3 (400), 29.4 / 28.7;  384 34.2 / 34.9, 35.2 / 35.5, 36.4 / 35.9, 40.2 / 38.0;
//     512 42.4 / 43.2, 43.9 / 43.8, 45.8 / 44.2, 50.5 / 47.1;  640 53.6 / 51.5, 56.9 / 52.2, 56.1 / 52.7, 62.3 / 57.2.
//   2x upsampling (four taps), the level around it, 280 / 320 narrow tiles: 640 channels 47.7 / 46.3, 48.9 / 47.3;  768, 288 / 336 56.3 / 54.2,
//     55.8 / 54.3.
//   With a mask t64 is only a bound: a linear layer, 360 narrow tiles, a third of the patches computed, K = 2,560 20.7 / 27.4; a 3x3
//     convolution of 768 channels, 492, seven tenths 55.5 / 62.2 (all 77.0 / 72.5).
static bool three_stages(const GemmArgs& a, int64_t t64) {
    const int64_t steps = (int64_t)a.taps * (a.K / 64);
    if (a.act.active || a.beside || ((a.rowscale || a.rowbias) && a.owner_rows < 64)) return false;
    if (a.conv && a.taps == 9) return steps >= 80 || (steps >= 32 && t64 >= 400);
    return steps > 32 || (steps == 32 && !a.rowscale && !a.rowbias && !a.seg[0].transposed && !a.seg[1].transposed && !a.seg[2].transposed);
}

// gemm_mfma_kernel's tile for a problem: its columns (0: none) and the stages of its ring.  Two stages run two blocks a CU, as do three of the
// 128 x 64 tile.
static int tile_pick(const GemmArgs& a, int* stages) {
    // Two blocks of 128 rows a CU (one block's prologue and epilogue run beside the other's main loop).
    const int64_t m128 = cdiv(a.M, 128), classes = std::max(1, a.classes);
    const int64_t t160 = a.N % 160 == 0 ? m128 * (a.N / 160) * classes : 0, t128 = a.N % 128 == 0 ? m128 * (a.N / 128) * classes : 0;
    *stages = 2;
    if (a.seg_cols % 32 != 0) return 0;             // a 32-column tile must not straddle output segments
    // N a multiple of 160: 128 x 160 tiles (wavefront tile 32 x 160).  Against a 256 x 160 tile
    // the rounds were the same: 34 -> 28 us (13,312 x 640 x 640), 68 -> 63 us (K = 2560), 80 -> 72 us
    // (13.4 k x 1280 x 1280), 165 -> 137 us (79 k x 640 x 640).
    // From 208 tiles on: the 128 x 64 tiles, 2.5 times as many, run 512 at a time, so up to 204 of these they take one round
    // and then two.  us, 128 x 160 / 128 x 64: 200 tiles K = 320 16.8 / 13.1, 640 20.1 / 15.8, 1280 26.6 / 22.8, 2560 40.3 / 33.8,
    // 5120 69.3 / 59.5; 204 tiles K = 640 18.9 / 16.8; 208 tiles 17.0 / 17.4, 20.2 / 21.0, 27.0 / 30.0, 42.7 / 46.3, 69.3 / 82.6.
    // But where 128 x 128 tiles still run in one round and these have CUs with two: 9,000 x 640, K = 640 20.3 / 128 x 128 18.4; 6,000 x
    // 1,280, K = 1,280 32.5 / 30.2; 1,536 x 3,840 29.2 / 26.6 (4,096 x 1,280, K = 5,120, 256 tiles: 67.8 / 74.2).
    const bool one_round = t128 > 256 && t128 <= 512;
    if (t160 >= 208 && !(one_round && t160 > 256)) {
        // One block a CU: the LDS that a second one would take holds two more stages.  us, two / four: text keys and values of 22 x 77
        // tokens x 2,560, K = 2,048 38.7 / 32.6 (and 183.4 / 189.9 for the cross-attention around them); residual blocks of one
        // convolution, 4,400 tokens x 960 112 / 98, 4,000 x 1280 146 / 135, 8,000 x 640 85.5 / 83.5.  (Three: the same to 1 us; the
        // 128 x 64 tiles with six instead of three 29.6 / 30.7, 47.5 / 48.1.)
        if (t160 <= 256 && !a.beside) *stages = 4;
        return 160;
    }
    // 128 x 128 tiles from where they do not fit one block a CU.  us, these / 256 x 128 (one block a CU) / 128 x 64: 306 tiles K = 384
    // 14.6 / 19.4 / 16.5, 480 K = 768 22.6 / 26.2 / 28.3, 576 K = 1,536 48.9 / 56.9 / 50.5, 816 K = 512 31.2 / 36.4 / 37.3, 1,278 K = 768
    // 49.6 / 60.5 / 60.3.  With fewer, 128 x 64 (204 tiles K = 128 8.5 / 11.9 / 8.9, 120 K = 1,536 22.3 / - / 15.4), unless three_stages.
    if (t128 > 256) return 128;
    const int64_t t64 = a.N % 64 == 0 ? m128 * (a.N / 64) * classes : 0;
    if (!t64) return 0;
    *stages = 3;
    return t128 && t64 > 256 && three_stages(a, t64) ? 128 : 64;
}
// How long that takes for a convolution without a mask, in us; fitted to 83 measured sizes (within a tenth).  (Calls with a mask take the same
// kernel: the scratch of shared tiles is there or not.)
static double tile_time(const GemmArgs& args) {
    int stages;
    GemmArgs a = args;
    a.act.active = nullptr;
    const int bn = tile_pick(a, &stages);
    if (!bn) return 1e30;
    const int64_t t = cdiv(a.M, 128) * (a.N / bn) * std::max(1, a.classes), full = (t - 1) / 512, rest = t - 512 * full;
    const double s = (double)a.taps * (a.K / 64), one = std::min<int64_t>(t, 256) / 256.0, over = std::max<int64_t>(rest - 256, 0) / 256.0;
    if (bn == 128 && stages == 3) return 8.0 + s * (0.47 + 0.09 * one);
    if (bn == 64) {
        const double k = (double)cdiv(t, 256);
        return t <= 256 ? 7.0 + 0.385 * s : t <= 512 ? 9.0 + s * (0.46 + 0.12 * over) : 4.0 * k + s * (0.04 + 0.28 * k);
    }
    if (bn == 160) {
        if (!full) return t <= 256 ? 9.5 + 0.67 * s : 8.0 + s * (0.96 + 0.37 * over);
        return full * (6.0 + 1.33 * s) + (rest <= 256 ? 4.0 + s * (0.33 + 0.28 * rest / 256) : 6.0 + s * (0.93 + 0.37 * over));
    }
    if (!full) return 8.0 + s * (0.84 + 0.26 * over);
    return full * (6.0 + 1.09 * s) + (rest <= 256 ? 4.0 + s * (0.28 + 0.19 * rest / 256) : 6.0 + s * (0.8 + 0.25 * over));
}

// The kernel a convolution takes: the small tiles of gemm_few.hip (few: which), the halo in LDS (sel, its tile, its shares) or, with
// neither, gemm_mfma_kernel.  The first are ahead while one round of them does; the second with many channels, where the nine
// reads of a pixel are long; the last has two blocks a CU and a round of 512 tiles, so it wastes less of one.  By the three models,
// the last only where it is clearly ahead.  us of one 3x3 convolution, 16 x 16 patches, few or halo / gemm_mfma_kernel:
//   1,024 tokens x 320 channels 9.9 / 23.9;  4,096 x 640 51.5 / 54.2;  9,216 x 256 31.6 / 26.9, 16,384 38.9 / 29.6, 36,864 79.5 / 61.7;
//   36,864 x 64 17.3 / 13.4, x 128 33.9 / 25.1, x 192 65.3 / 43.7, x 384 153 / 123, x 512 215 / 202, x 768 422 / 408;
//   12,288 x 320 44.4 / 35.0, 16,384 48.5 / 41.6, 24,576 53.1 / 59.3, 36,864 100 / 90; 16,384 x 640 107 / 129, 36,864 283 / 287;
//   6,144 x 960 122 / 144; 2,048 x 1280 71 / 101, 12,288 345 / 356.  Patches the halo does not take, two layers with their norms:
//   2,304 x 960 154 / 185.
// Small tiles up to 1,024 channels where the halo is the other choice: above, the weights (more than 29 MB) come from HBM in a whole
// network, and the longer chain waits for them (1,024 x 1,280 41 / 46, with cold weights 52 / 48).
// With a mask the rows are a bound: more than one round of small tiles then (4,096 x 512, three fifths reused, RES2 + SATTN 145 / 172 us with
// the 128-row tiles).
// Moments of the output that one of the two leaves behind are worth moments_us: 9,216 tokens x 64 channels, two layers, few / halo 43.6 / 41.2 us
// (few for the second alone: 38).
struct ConvChoice {
    int sel, few, splits;
    ConvTile ct;
};
// rows of a partial sum that the halo kernel (sel) or gemm_mfma_kernel (0) leaves behind, 0: none
static int moment_rows(const GemmArgs& a, int sel) {
    if (a.stats_G <= 0 || a.act.active || a.N % a.stats_G != 0) return 0;
    // a wavefront's rows must lie in one patch, and its columns must hold whole groups
    static constexpr int cols[7] = {0, 160, 160, 128, 64, 32, 160};
    int stages;
    const int bn = sel ? 0 : tile_pick(a, &stages);
    if (!sel && !bn) return 0;
    const int rows = sel || bn != 160 ? 64 : 32, wc = sel ? cols[sel] : bn == 160 ? 160 : bn / 2;
    return a.geom.S % rows == 0 && wc % (a.N / a.stats_G) == 0 ? rows : 0;
}
static ConvChoice conv_choose(const GemmArgs& a) {
    ConvChoice c{0, 0, 1, {}};
    double few = 1e30;
    // (gemm_mfma_kernel's end is longer for it: 36.0 -> 39.4 us at 3,456 x 512, 91.8 -> 95.7 at 36,864 x 320)
    auto spared = [&](int sel) { return a.moments_us > 0 && moment_rows(a, sel) ? (sel ? 1.0 : 0.7) * a.moments_us : 0.0; };
    c.sel = conv_select(a, &c.ct);
    c.few = few_pick(a, 1, &few);
    const double tile = tile_time(a) - spared(0);
    const bool mask = a.act.active != nullptr;
    if (mask && c.sel && !c.few && a.K <= 1024) c.few = few_pick(a, 4, &few);
    if (!c.sel) {           // more than one round only for plain convolutions
        if (!c.few && a.K <= 1024 && a.taps == 9 && a.a_mul <= 1) {
            c.few = few_pick(a, 4, &few);
            if (few > 0.95 * tile) c.few = 0;
        }
        if (spared(0) > 0 && few > tile) c.few = 0;
        return c;
    }
    const double halo = conv_time(a, c.sel, &c.splits) - spared(c.sel);
    if (a.K > 1024 || few >= halo) c.few = 0;
    if (tile < (c.few ? (mask ? 0.9 : 0.95) * few : c.sel == 4 || c.sel == 5 ? halo : 0.95 * halo)) c.few = c.sel = 0;
    if (c.few) c.sel = 0;
    return c;
}

int gemm_stats_rows(const GemmArgs& a, int dtype, int mode) {
    if (mode != 0 || dtype != PSERVE_BF16 || !a.conv || a.epi != EPI_ROUTE || a.taps != 9 || a.stats_G <= 0 || !gemm_mfma_eligible(a)) return 0;
    const ConvChoice c = conv_choose(a);
    return c.few || (!c.sel && a.moments_us <= 0) ? 0 : moment_rows(a, c.sel);       // (gn_direct_kernel costs less than moments from there)
}

static GemmArgs conv_args(const PatchGeom& g, int32_t M, int32_t N, int32_t K) {
    GemmArgs a{};
    a.conv = 1; a.tokens_are_rows = 1; a.taps = 9; a.geom = g; a.M = M; a.N = a.seg_cols = N; a.K = a.lda = K;
    for (auto& s : a.seg) s.scale = 1.f;
    return a;
}
size_t conv_split_bytes(const PatchGeom& g, int32_t M, int32_t N, int32_t K, int32_t G, int dtype, int mode) {
    if (dtype != PSERVE_BF16 || mode != 0 || K % 64 != 0) return 0;
    GemmArgs a = conv_args(g, M, N, K);
    a.stats_G = G;
    size_t most = 0;
    for (const float us : {0.f, MOMENTS_US}) {          // whether somebody reads the output's moments or not
        a.moments_us = us;
        const ConvChoice c = conv_choose(a);
        if (c.sel && c.splits > 1) most = std::max(most, sizeof(float) * c.splits * cdiv(M, CONV_BM[c.sel]) * CONV_BM[c.sel] * (size_t)N);
    }
    return most;
}

// For tests (host only, no part of the ABI): 1 if the 3x3 convolutions of such a batch (bf16, C to C channels) have few enough
// tiles to share them, where no other kernel takes them.
extern "C" int pserve_test_conv_shares(int32_t P, int32_t ph, int32_t pw, int32_t C) {
    ConvTile ct;
    const int sel = conv_select(conv_args(PatchGeom{P, ph * pw, ph, pw, pw + 2, (ph + 2) * (pw + 2)}, P * ph * pw, C, C), &ct);
    return sel && conv_splits(cdiv((int64_t)P * ph * pw, CONV_BM[sel]) * (C / CONV_BN[sel]), C / 64) > 1;
}
// How such a convolution runs where somebody reads its output's moments (32 groups): 0 the small tiles, 1 the halo in LDS, 2 the linear
// layers' tiles; + 10 x the rows of the moments.
extern "C" int pserve_test_conv_kernel(int32_t P, int32_t ph, int32_t pw, int32_t C) {
    GemmArgs a = conv_args(PatchGeom{P, ph * pw, ph, pw, pw + 2, (ph + 2) * (pw + 2)}, P * ph * pw, C, C);
    a.stats_G = 32;
    a.moments_us = MOMENTS_US;
    const ConvChoice c = conv_choose(a);
    return (c.few ? 0 : c.sel ? 1 : 2) + 10 * gemm_stats_rows(a, PSERVE_BF16, 0);
}
// 10 x columns + stages of the last
int gemm_tile_code(const GemmArgs& a);
extern "C" int pserve_test_conv_tile(int32_t P, int32_t ph, int32_t pw, int32_t C) {
    GemmArgs a = conv_args(PatchGeom{P, ph * pw, ph, pw, pw + 2, (ph + 2) * (pw + 2)}, P * ph * pw, C, C);
    a.stats_G = 32;
    a.moments_us = MOMENTS_US;
    const ConvChoice c = conv_choose(a);
    return c.few || c.sel ? 0 : gemm_tile_code(a);
}
// The tile of gemm_few.hip that such a convolution, without moments, takes (1 .. 5: 32 x 32, 32 x 64, 32 x 80, 64 x 64, 64 x 80), 0: none; linear:
// that of a linear layer of P * ph * pw rows, K = C, N columns in segments of seg_cols (value-gate pairs: seg_cols = 0).
extern "C" int pserve_test_few_tile(int32_t P, int32_t ph, int32_t pw, int32_t C, int32_t linear, int32_t N, int32_t seg_cols) {
    GemmArgs a = conv_args(PatchGeom{P, ph * pw, ph, pw, pw + 2, (ph + 2) * (pw + 2)}, P * ph * pw, C, C);
    if (!linear) return conv_choose(a).few;
    a.taps = 1; a.conv = 0; a.N = N;
    a.epi = !seg_cols ? EPI_GEGLU : EPI_ROUTE;
    a.seg_cols = seg_cols ? seg_cols : N;
    double us;
    return few_pick(a, a.epi == EPI_GEGLU ? 2 : 1, &us);
}

// For tests: tile_pick of a linear layer, 10 x columns + stages
int gemm_tile_code(const GemmArgs& a) {
    int stages;
    const int bn = tile_pick(a, &stages);
    return bn ? 10 * bn + stages : 0;
}

int gemm_wide_bf16(const GemmArgs& a, hipStream_t st, bool* handled);     // gemm_wide.hip

// Two problems in one launch (two_select in gemm_wide.hip): columns of the tile modelled faster, and its time in us, fitted to 70
// sizes (within a fifth: the time of a gate depends on how many requests a wavefront's rows belong to).  Both run two blocks a CU.
int gemm_two_cols(const GemmArgs& a, double* us) {
    const int64_t mt = cdiv(a.M, 128) + cdiv(a.M2, 128), steps = a.K / 64;
    double t64 = 1e30, t128 = 1e30;
    if (a.N % 64 == 0 && a.seg_cols % 32 == 0) {
        const int64_t t = mt * (a.N / 64);
        const double k = (double)cdiv(t, 256);      // rounds of 256 blocks: each slows the steps of those beside it
        t64 = t <= 256 ? 5.6 + 0.31 * steps : t <= 512 ? 8.0 + steps * (0.52 + 0.1 * (t - 256) / 256) : 4.0 * k + steps * (0.04 + 0.28 * k);
    }
    if (a.N % 128 == 0 && a.seg_cols % 32 == 0) {
        const int64_t t = mt * (a.N / 128), full = t / 512, rest = t % 512;
        const double first = full ? 5.0 + 0.55 * steps : 7.2 + 0.61 * steps;
        t128 = full * (9.0 + 1.05 * steps) + (rest == 0 ? 0.0 : rest <= 256 ? first : 9.0 + steps * (0.75 + 0.3 * (rest - 256) / 256));
    }
    *us = std::min(t64, t128);
    return *us >= 1e30 ? 0 : t64 <= t128 ? 64 : 128;
}
int gemm_two_bf16(const GemmArgs& a, int cols, hipStream_t st) {
    if (cols == 64) return launch_feat<128, 64, false, 2, 2, 3, false, EPF_ALL | EPF_TWO>(a, st);
    return launch_feat<128, 128, false, 2, 2, 2, false, EPF_ALL | EPF_TWO>(a, st);
}

// What gemm_mfma_bf16 sends to gemm_few_kernel or gemm_mfma_kernel, whose HALO forms look up where each row's pixels lie once a tile.
bool gemm_takes_halo(const GemmArgs& a, int dtype, int mode) {
    if (dtype != PSERVE_BF16 || mode != 0 || !gemm_mfma_eligible(a) || !a.conv || a.epi != EPI_ROUTE || !a.tokens_are_rows || a.act.active || a.B2 ||
        a.taps > 9 || a.rowbias || a.rowscale || a.act_gelu || a.seg[0].transposed || a.seg[0].scale != 1.f || a.seg_cols != a.N) return false;
    const ConvChoice c = conv_choose(a);
    int stages;
    return !c.sel && (c.few || tile_pick(a, &stages));
}

int gemm_mfma_bf16(const GemmArgs& a, hipStream_t st, bool* handled) {
    *handled = false;
    if (!gemm_mfma_eligible(a)) return PSERVE_OK;
    double us;
    const bool conv = a.conv && a.epi == EPI_ROUTE;
    const ConvChoice c = conv ? conv_choose(a) : ConvChoice{0, 0, 1, {}};
    const int few = a.B2 || a.beside ? 0 : conv ? c.few : few_pick(a, a.epi == EPI_GEGLU ? 2 : 1, &us);
    if (few) {
        *handled = true;
        return gemm_few_bf16(a, few, st);
    }
    if (!a.conv) {
        PS_TRY(gemm_wide_bf16(a, st, handled));
        if (*handled || a.B2) return PSERVE_OK;
    }
    if (a.epi == EPI_GEGLU) {
        if (a.N % 128 != 0) return PSERVE_OK;
        *handled = true;
        // The epilogue (GELU of every gate) is as long as the main loop at K = 640: two blocks of 128 rows a CU, so that one
        // block's epilogue runs beside the other's main loop, and with fewer tiles on one block a CU.  The wavefront tile is 32 x
        // 128 = [64 values | 64 gates].  us, 256 x 128 tiles (one block a CU, before) / these: 512 x 7,680, K = 960 20.4 / 15.7; 512 x 10,240,
        // K = 1,280 25.8 / 22.3; 1,024 x 5,120, K = 640 18.8 / 16.0; 13,312 x 5,120, K = 640 163 / 142.
        return launch<128, 128, true, 4, 1, 2, false>(a, st);
    }
    *handled = true;
    switch (c.sel) {
    case 1: return launch_conv<256, 160, 4, 1, 384, 3, 2>(a, c.ct, c.splits, st);
    case 2: return launch_conv<128, 320, 2, 2, 256, 2>(a, c.ct, c.splits, st);
    case 3: return launch_conv<128, 256, 2, 2, 256, 2>(a, c.ct, c.splits, st);
    case 4: return launch_conv<128, 128, 2, 2, 256, 2>(a, c.ct, c.splits, st);
    case 5: return launch_conv<128, 64, 2, 2, 256, 2>(a, c.ct, c.splits, st);
    case 6: return launch_conv<256, 160, 4, 1, 416, 2, 2>(a, c.ct, c.splits, st);
    default: break;
    }
    int stages;
    switch (tile_pick(a, &stages)) {
    case 160: return stages == 4 ? launch<128, 160, false, 4, 1, 4, false>(a, st) : launch<128, 160, false, 4, 1, 2, false>(a, st);
    case 128: return stages == 3 ? launch<128, 128, false, 2, 2, 3, true>(a, st) : launch<128, 128, false, 2, 2, 2, false>(a, st);
    case 64: return launch<128, 64, false, 2, 2, 3, false>(a, st);
    default: break;
    }
    *handled = false;
    return PSERVE_OK;
}

}  // namespace pserve
