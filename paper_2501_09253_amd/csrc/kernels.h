// Internal launch interface between the block executor and the kernel files.
#pragma once

#include "common.h"

namespace pserve {

// ---- element access helpers (device) ------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {       // round to nearest even (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}
// two floats -> packed bf16 pair (lo in bits 0..15), one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
template <typename T> __device__ __forceinline__ float ld_f(const T* p);
template <> __device__ __forceinline__ float ld_f<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld_f<uint16_t>(const uint16_t* p) { return bf16_bits_to_float(*p); }
template <typename T> __device__ __forceinline__ void st_f(T* p, float v);
template <> __device__ __forceinline__ void st_f<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st_f<uint16_t>(uint16_t* p, float v) { *p = float_to_bf16_bits(v); }

// fp32 rows as bf16 pieces: rows of [C / 32][3][32], three pieces of every value.  Index of the first piece of value c; the
// others follow 32 and 64 further.
__host__ __device__ __forceinline__ int piece_index(int c) { return (c >> 5) * 96 + (c & 31); }
// bf16 numbers nearest to two values (ties to even), the first in the lower half; a half as a float
typedef __attribute__((ext_vector_type(2))) float ps_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 ps_bf16x2;
__device__ __forceinline__ uint32_t near_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(ps_f32x2{a, b}, ps_bf16x2));
}
__device__ __forceinline__ float lo_bf16(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
// The pieces x0, x1, x2 of two values, u[piece]: each the nearest bf16 number to what the ones before it leave, so |x1| <= 2^-8
// |x|, |x2| <= 2^-17 |x|, their signs are as likely one as the other, and they sum to x exactly; below 2^-110, where the last
// piece leaves the range of bf16, to within 2^-134.  The product of two values takes six of the nine products of pieces; x1 y2, x2 y1
// and x2 y2 are at most 2^-23.9 of it and zero in the mean (four million pairs: 2^-24.2, 1e-12).  Pieces cut off instead of
// rounded lose up to 2^-21.0, always towards zero (2^-21.2, 4e-8).
// A value that is not finite is (2^-126, 0, x) with x's sign: of the six products only those with the other factor's x0 then hold it,
// which is zero or has the factor's sign, so infinities and NaN come out as those of the plain product.  (A finite product within
// 1 % of the largest number may come out infinite: x0 y0 may be that much larger.)
constexpr float PIECE_TINY = 1.17549435e-38f, PIECE_MAX = 3.38953139e38f;       // smallest normal, largest bf16 number
__device__ __forceinline__ bool cut_is_plain(float a, float b) { return fabsf(a) + fabsf(b) <= PIECE_MAX; }
__device__ __forceinline__ void cut3x2_plain(float a, float b, uint32_t (&u)[3]) {     // where cut_is_plain
    u[0] = near_bf16x2(a, b);
    const float ra = a - lo_bf16(u[0]), rb = b - hi_bf16(u[0]);
    u[1] = near_bf16x2(ra, rb);
    u[2] = near_bf16x2(ra - lo_bf16(u[1]), rb - hi_bf16(u[1]));
}
__device__ __forceinline__ void cut3x2(float a, float b, uint32_t (&u)[3]) {
    if (cut_is_plain(a, b)) {
        cut3x2_plain(a, b, u);
        return;
    }
    // not finite, or large (the largest values would round to infinity)
    const bool fa = fabsf(a) < INFINITY, fb = fabsf(b) < INFINITY;
    u[0] = near_bf16x2(fa ? fminf(fmaxf(a, -PIECE_MAX), PIECE_MAX) : copysignf(PIECE_TINY, a),
                       fb ? fminf(fmaxf(b, -PIECE_MAX), PIECE_MAX) : copysignf(PIECE_TINY, b));
    const float ra = fa ? a - lo_bf16(u[0]) : 0.f, rb = fb ? b - hi_bf16(u[0]) : 0.f;
    u[1] = near_bf16x2(ra, rb);
    u[2] = near_bf16x2(fa ? ra - lo_bf16(u[1]) : a, fb ? rb - hi_bf16(u[1]) : b);
}
// 2^(2 h).  The instruction returns zero below 2^-126; the square of its result goes down to the smallest subnormal, as exp2f,
// at a multiplication instead of exp2f's five instructions.
__device__ __forceinline__ float exp2_square(float h) { const float e = __builtin_amdgcn_exp2f(h); return e * e; }
// pieces of four neighbouring values (a multiple of four in front of them), the first at dst
__device__ __forceinline__ void store_pieces4(uint16_t* dst, float a, float b, float c, float d) {
    uint32_t u[2][3];
    cut3x2(a, b, u[0]);
    cut3x2(c, d, u[1]);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(dst + 32 * p) = make_uint2(u[0][p], u[1][p]);
}

// Patch geometry shared by the kernels that walk tokens.
struct PatchGeom {
    int32_t P, S, ph, pw;      // patches, tokens per patch, patch height / width
    int32_t ppw, pS;           // padded patch width (pw+2) and padded pixels per patch ((ph+2)*(pw+2))
};

// Optional compaction of the patches that are computed (reuse mask == 0).  active == nullptr means
// "all patches, identity order".
struct ActiveList {
    const int32_t* active;     // [P] patch ids, first *count entries valid
    const int32_t* count;      // device scalar
};

// ---- GroupNorm (norm.hip) -------------------------------------------------------------------
struct GroupNormArgs {
    const void* x;             // [T][C]
    const void* gamma;         // [C] block dtype
    const void* beta;          // [C]
    int32_t C, G, n;
    float eps;
    int32_t max_tokens;        // tokens of the largest request
    int32_t nsplit;            // token chunks per patch used for the partial sums
    float* partial;            // [P][nsplit][G][2] (sum, sum of squares)
    float* scale_shift;        // [n][C][2]: y = x*scale + shift for sorted slot s
    const int32_t* request_offset;   // [n+1]
    const int32_t* owner;      // [P]
    const int32_t* neighbour;  // [P][8] (stitching only)
    const uint8_t* rim_only = nullptr;   // [P] or nullptr; apply pass into the padded layout: only the border tokens of these patches
};
int gn_stats(const GroupNormArgs& a, const PatchGeom& g, int dtype, hipStream_t st);
// true if that is one launch, about as long as gn_finalize alone
bool gn_takes_direct(const GroupNormArgs& a, const PatchGeom& g, int dtype);
// statistics and application of a small batch (gn_takes_whole) in one launch: conv: SiLU into the padded buffer with the rims,
// else plain rows; all patches, no pieces
bool gn_takes_whole(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool conv);
int gn_whole(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool conv, void* out, hipStream_t st);
// second half of gn_stats alone: a.partial already holds [P][slots][G][2] partial sums (filled by a convolution)
int gn_finalize(const GroupNormArgs& a, const PatchGeom& g, int dtype, int32_t slots, hipStream_t st, bool per_channel = false);
// bf16 split that also leaves per-channel moments stats[P][nch][C][2] behind (plan.hip); *done = false where its
// fast path does not apply (nothing is written then)
int split_with_stats(const pserve_plan_t* plan, const void* const* images, int32_t C, void* x, float* stats, int32_t nch,
                     hipStream_t st, bool* done);
// y = x*scale+shift (then SiLU if silu).  padded: write into the interior of the padded patch buffer
// [P][ph+2][pw+2][C]; else plain [T][C].  Only patches of `act` are written.  stitch (padded, all patches):
// border tokens also fill the neighbours' ring slots / zero the own ring at image edges (no halo_gather needed).
// pieces (fp32): every value as three bf16 pieces (piece_index).
int gn_apply(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool silu, bool padded, bool stitch, void* out,
             ActiveList act, hipStream_t st, bool pieces = false);
// Per-token LayerNorm over the C channels (biased variance) of the patches of `act`; out [T][C] at the same token
// positions.  Affine part: gamma / beta [C] of the block dtype, or (gamma == nullptr) the adaptive form
// xhat * (1 + scale) + shift with shift = mod[slot * mod_ld + c], scale = mod[slot * mod_ld + C + c], slot = owner[patch].
// mod_txt (with patch_rc [P][2]): the table of the text patches (patch_rc[2p] < 0), mod being that of the image patches.
int layer_norm(const void* x, const void* gamma, const void* beta, const float* mod, int64_t mod_ld, const int32_t* owner,
               int32_t C, float eps, const PatchGeom& g, int dtype, void* out, ActiveList act, hipStream_t st,
               const float* mod_txt = nullptr, const int32_t* patch_rc = nullptr, bool pieces = false);
// Fill the one-pixel ring of every active padded patch from the interiors of its neighbours (zeros outside the image).
int halo_gather(void* apad, const int32_t* halo_src, const PatchGeom& g, int32_t C, int32_t ring, int dtype,
                ActiveList act, hipStream_t st);

// ---- GEMM / implicit-GEMM convolution (gemm.hip) -----------------------------------------------
struct GemmSeg {
    void* ptr;                 // output of this column segment
    int64_t ld;                // row stride (elements); for transposed: stride between channels
    int32_t transposed;        // 1: out[col][row] instead of out[row][col]
    float scale;               // multiplies the result (after bias)
};
enum { EPI_ROUTE = 0, EPI_GEGLU = 1 };
// What every kernel takes.  A convolution whose tiles are not shared takes this alone: with the fields of GemmArgs among its
// arguments it waited for more of them before its first loads (two convolutions of 29,696 tokens x 320 channels with their
// norms, split and reassembly, mean over ten placements of the buffers: 164.2 against 163.7 us).  Arguments are fetched in
// pieces of up to 32 bytes by dependent reads, so their offsets count in short kernels: `geom` at a multiple of eight bytes,
// 10.9 / 5.0 / 4.4 -> 10.6 / 4.8 / 4.2 us for three fp32 products of 832 rows.
struct GemmCore {
    const void* A;             // linear: [rows][lda]; conv: padded patch buffer
    int64_t lda;
    int32_t conv;              // 1: rows are tokens read through the padded layout with `taps` taps
    // conv only (0 = the defaults 3 / 1 / identity): taps are laid out tap_w per pixel row; row token (p, y, x) reads
    // the padded pixels (a_mul*y + a_dy + ty, a_mul*x + a_dx + tx) of patch p (a_mul = 2: stride-2 convolution whose
    // rows are OUTPUT tokens of the half-size patch geometry in `geom.S / geom.pw`, while geom.ppw / geom.pS stay those
    // of the input); with o_mul = 2 the result of row (p, y, x) goes to token p*o_S + (2y + o_dy)*o_pw + 2x + o_dx
    // (one parity class of a nearest-up convolution, whose rows are INPUT tokens)
    int32_t tap_w, a_mul, a_dy, a_dx;
    int32_t o_mul, o_dy, o_dx, o_S, o_pw;
    // 4: the four parity classes (2a + b) of a nearest-up convolution in one call: a_dy = o_dy = a, a_dx = o_dx = b, and
    // the weights are [class][taps][N][K].  0: one problem as described by the fields above.
    int32_t classes;
    PatchGeom geom;
    ActiveList act;            // row compaction by patch (rows are tokens)
    int32_t tokens_are_rows;   // 1: row ids are token ids (act applies); 0: plain row ids (M rows)
    int32_t M;                 // number of rows (upper bound when act is used: P*S)
    int32_t row_group, row_group_pad;   // plain rows only: output row = (r / row_group) * row_group_pad + r % row_group (0 = identity)
    int32_t N, K;              // N packed output columns, K reduction length per tap
    int32_t taps;              // 1 or 9
    const void* B;             // packed weights [taps][N][K]
    const float* bias;         // [N] packed order, or nullptr
    const float* rowbias;      // optional [n][N]: row r also gets rowbias[row_owner[token / S]][col] (rows are tokens)
    const int32_t* row_owner;  // [P] request slot of each patch (with rowbias / rowscale)
    const float* rowscale;     // optional: (acc + bias [+ rowbias]) is multiplied by rowscale[slot * rowscale_ld + col]
    int64_t rowscale_ld;       //           before the residual is added (gated residual of an adaLN sub-layer)
    int32_t act_gelu;          // 1: tanh-form GELU of (acc + bias) (EPI_ROUTE only)
    const void* res;           // residual [rows][ldr] or nullptr (added after bias)
    int64_t ldr;
    int32_t epi;               // EPI_ROUTE: columns go to segment col / seg_cols; EPI_GEGLU: value*GELU(gate) pairs
    int32_t seg_cols;
    GemmSeg seg[3];
    // Optional GroupNorm partial sums of the OUTPUT (bias included, before the residual), in the layout gn_finalize
    // reads: stats[P][stats_slots][stats_G][2] = (mean, sum of squared deviations) of S / stats_slots consecutive tokens of a patch
    // and one group.  Only the kernels gemm_stats_rows() accepts fill it (plain stores).
    float* stats;
    int32_t stats_G, stats_slots;
};
struct GemmArgs : GemmCore {
    // Optional scratch for partial sums (fp32): a convolution with too few tiles for the chip shares the K range of a tile
    // between blocks (conv_split_bytes says how much it needs).  Not shared with a call that may run at the same time.
    float* split_ws;
    size_t split_ws_bytes;
    // Optional second problem in the same launch: the rows of another patch list (act2, at most M2 of them) with weights,
    // bias and gate of their own, everything else alike.  Only where gemm_takes_two() says so.
    const void* B2;
    const float* bias2;
    const float* rowscale2;
    ActiveList act2;
    int32_t M2;
    // conv: A is the unpadded batch [tokens of the input][lda], and the pixels around a patch are looked up here ([P][ring] source tokens, -1: zeros).
    // Only where gemm_takes_halo() says so, without a patch list.
    const int32_t* halo_src;
    // fp32: A is in bf16 pieces (gemm_takes_pieces) / the output is written in pieces
    int32_t a_pieces, out_pieces;
    int32_t owner_rows;        // with rowbias / rowscale: the rows of every request start at a multiple of this (1, 2, .. 64; 0: not known)
    int32_t beside;            // runs beside kernels of another stream that fill the chip: no kernel whose blocks want a CU's LDS for themselves
    float moments_us;          // conv with stats_G: what the output's moments spare its norm (0: nothing)
};
// Rows of A a problem can address: where rows are tokens, any token of the batch, however few patches its list has (the two
// lists of a joint batch lie interleaved in one token matrix).
inline int64_t gemm_a_rows(const GemmArgs& a) {
    return a.conv ? (int64_t)a.geom.P * a.geom.pS : a.tokens_are_rows ? (int64_t)a.geom.P * a.geom.S : (int64_t)a.M;
}
// The bf16 matrix kernels stage both operands by buffer loads with 32-bit byte offsets below 2^31 from the tensors' bases.
inline bool gemm_fits32(const GemmArgs& a) {
    return gemm_a_rows(a) * a.lda < ((int64_t)1 << 30) &&
           (int64_t)a.taps * a.N * a.K * std::max(1, a.classes) < ((int64_t)1 << 30);
}
// true if gemm(a, ...) with its second problem will take a kernel that runs both in one launch
bool gemm_takes_two(const GemmArgs& a, int dtype, int mode);
// true if gemm(a, ...) will take a kernel that reads the unpadded batch through a.halo_src
bool gemm_takes_halo(const GemmArgs& a, int dtype, int mode);
// true if gemm(a, ...) is faster with its activations in bf16 pieces (a.a_pieces, which the caller then sets)
bool gemm_takes_pieces(const GemmArgs& a, int dtype, int mode);
// scratch a 3x3 convolution of M rows, N output and K input channels over this patch geometry can use (0: none)
constexpr float MOMENTS_US = 6.f;      // gn_partial_kernel, 4.5 us at 9,216 tokens x 64 to 8 at 4,096 x 640
size_t conv_split_bytes(const PatchGeom& g, int32_t M, int32_t N, int32_t K, int32_t G, int dtype, int mode);
// tokens a partial sum of a.stats covers where gemm(a, ...), with a.stats_G groups, takes a kernel that fills it, else 0 (the caller then
// runs gn_stats on the output)
int gemm_stats_rows(const GemmArgs& a, int dtype, int mode);
int gemm(const GemmArgs& a, int dtype, int mode, hipStream_t st);

// Weight packing into [taps][N][K] (K contiguous); all on device.  fp32 weights (rows = taps x N) of a layer that may take its
// activations in pieces are followed by their own: packed_weight_bytes is the size of both (of the weights alone where no kernel
// reads pieces of them), split_packed fills in the pieces once all rows are packed.
size_t packed_weight_bytes(int64_t rows, int32_t K, int dtype);
int split_packed(void* packed, int64_t rows, int32_t K, int dtype, hipStream_t st);
int pack_conv(const void* w, void* dst, int32_t Cout, int32_t Cin, int dtype, hipStream_t st);
// linear W[K][Ncols] -> rows [row0, row0+Ncols) of dst[Ntotal][K]
int pack_linear(const void* w, void* dst, int32_t K, int32_t Ncols, int32_t row0, int dtype, hipStream_t st);
// GEGLU: W1[K][2F] -> dst[2F][K] with value / gate columns interleaved in groups of GEGLU_GROUP
int pack_geglu(const void* w1, const void* b1, void* dst, float* bias_dst, int32_t K, int32_t F, int dtype, hipStream_t st);
int pack_bias(const void* b, float* dst, int32_t N, int dtype, hipStream_t st);
// Nearest-up 2x followed by a 3x3 convolution = four 2x2-tap convolutions on the input, one per output parity (a, b):
// dst[(2a+b)][2j+i][Cout][Cin] = sum of the 3x3 taps (ty, tx) that fall on input pixel (y - 1 + a + j, x - 1 + b + i),
// i.e. rows {0 | 1,2} for a = 0 and {0,1 | 2} for a = 1 (same for columns); summed in fp32, rounded once.
int pack_conv_up2(const void* w, void* dst, int32_t Cout, int32_t Cin, int dtype, hipStream_t st);
constexpr int GEGLU_GROUP = 64;

// ---- attention (attn.hip) -------------------------------------------------------------------------
constexpr int AT_START = 4;          // fp32 attention in pieces: an item's start and end, in tiles of 32 keys (us, shares of equal numbers of tiles, 0, and of
                                     // these units, 2 / 4 / 6 / 9: 4,096 + 8 x 64 tokens, 5 heads of 64 281 / 202 / 188 / 190 / 190 us, 2,304 + 60 x 64
                                     // 177 / 137 / 134 / 139 / 143)
struct AttnArgs {
    const void* Q;             // [T][C], already multiplied by log2(e)/sqrt(d)
    const void* K;             // self: [T][C]; cross: [n*L][C]
    const void* V;             // [rows][C], or transposed [C][ldv] when v_transposed
    int64_t ldv;
    int32_t v_transposed;
    void* O;                   // [T][C]
    int32_t C, heads, d;
    PatchGeom geom;
    ActiveList act;
    const int32_t* owner;      // [P] sorted slot of a patch
    const int32_t* cu_seqlens; // self: [n+1] token range of slot s
    const int32_t* seq_len;    // self: [n] valid tokens of slot s (keys cu_seqlens[s] .. + seq_len[s]); nullptr: the whole range
    const int32_t* perm;       // cross: caller index of slot s
    int32_t cross_len;         // 0 = self-attention; else keys of slot s are rows perm[s]*cross_len .. +cross_len
    int32_t cross_ld;          // cross: padded key rows per request (>= cross_len)
    // query tiling of the MFMA kernel (attention_tiles fills the two prefix tables)
    const int32_t* act_off;    // [n+1] computed patches before slot s (== RequestOffset without a mask)
    const int32_t* tile_off;   // [n+1] query tiles before slot s
    const int64_t* unit_off;   // [n+1] fp32 attention in pieces: units (at_unit) before slot s
    int32_t n;                 // request slots
    int32_t max_tiles;         // host upper bound of tile_off[n]
    int32_t qt;                // 1 or 2: the tables were built for query tiles of 128 * qt rows
    int32_t max_rows;          // host upper bound of the query rows of one request (its tokens)
    int32_t group;             // consecutive work items dealt to an XCD at a time (filled in by the launch)
    int32_t shares;            // fp32 attention in pieces: attention_shares, with unit_off
    int32_t out_pieces;        // fp32: O is written as bf16 pieces
    void* cut;                 // fp32 self-attention: scratch of attention_cut_bytes, nullptr: the fp32 kernel
};
// Item k of the work list of a call, longest first: request slots from the last (the plan sorts requests by size,
// largest last) to the first, head-major inside a slot, so that consecutive items are consecutive query tiles of one head.
__device__ __forceinline__ bool attn_item_at(const AttnArgs& a, int64_t k, int& s, int& head, int& tile_in_s) {
    const int total_tiles = a.tile_off[a.n];
    const int64_t items = (int64_t)total_tiles * a.heads;
    if (k >= items) return false;
    const int64_t q = items - 1 - k;                 // position in ascending slot order
    const int qt = (int)(q / a.heads);
    int lo = 0, hi = a.n;                            // largest s with tile_off[s] <= qt
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.tile_off[mid] <= qt) lo = mid; else hi = mid;
    }
    s = lo;
    const int tiles_s = a.tile_off[s + 1] - a.tile_off[s];
    const int r = tiles_s * a.heads - 1 - (int)(q - (int64_t)a.tile_off[s] * a.heads);
    head = r / tiles_s;
    tile_in_s = r - head * tiles_s;
    return true;
}
// unit_off (optional, with the tables it takes): see AttnArgs
int attention_tiles(const int32_t* request_offset, const uint8_t* mask, int32_t n, int32_t S, int32_t qt, int32_t* act_off,
                    int32_t* tile_off, hipStream_t st, int64_t* unit_off = nullptr, const int32_t* cu_seqlens = nullptr,
                    const int32_t* seq_len = nullptr, int32_t heads = 0);
int attention_max_tiles(const pserve_plan_t* plan, int32_t qt);
// scratch (keys and values in bf16 pieces) of an fp32 self-attention over this plan, 0: it takes the fp32 kernel
size_t attention_cut_bytes(const pserve_plan_t* plan, int32_t C, int32_t heads, int dtype, int mode);
// blocks that such an attention's work is shared out to (0: one an item)
int attention_shares(const pserve_plan_t* plan, int32_t C, int32_t heads);
int attention(const AttnArgs& a, int dtype, int mode, hipStream_t st);

// ---- reuse (block.hip) -------------------------------------------------------------------------------

}  // namespace pserve
