// Segmented GroupNorm over the patch batch and the 3x3 halo gather.
//
// GroupNorm statistics of a patch batch must be those of the whole image: mean and
// variance of a group are reduced over ALL patches of the owning request (the patches of
// request s are RequestOffset[s] .. RequestOffset[s+1], "Compressed Sparse Patch Format").
// The halo gather is the pull form of the paper's edge stitching ("Patch Edge Stitcher"):
// border pixels of same-image neighbour patches, zeros where the neighbour is absent
// ("Patch-Tailored Diffusion Operators").
//
// Kernels of the norm:
//   gn_partial_kernel   per (patch, token chunk): per-group mean and sum of squared deviations
//                       (fp32, shifted sums), 16-byte loads, per-thread channel accumulators,
//                       LDS tree to groups
//   gn_finalize_kernel  per (request, group): the partial moments merged in fp64 (shuffles +
//                       LDS) -> mean, rstd -> per (request, channel) scale and shift
//   gn_direct_kernel    both of these in one launch, for small requests
//   gn_whole_kernel     all three in one launch, for small batches
//   gn_apply_kernel     y = x*scale + shift (+SiLU), written plain or into the interior of
//                       the padded patch buffer the convolution reads
// Reductions are deterministic (no float atomics).
#include "kernels.h"

namespace pserve {

template <typename T> struct Vec;
template <> struct Vec<float> { static constexpr int N = 4; };
template <> struct Vec<uint16_t> { static constexpr int N = 8; };

template <typename T>
__device__ __forceinline__ void load_vec(const T* p, float (&v)[Vec<T>::N]);
template <>
__device__ __forceinline__ void load_vec<float>(const float* p, float (&v)[4]) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
template <>
__device__ __forceinline__ void load_vec<uint16_t>(const uint16_t* p, float (&v)[8]) {
    const uint4 q = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}
template <typename T>
__device__ __forceinline__ void store_vec(T* p, const float (&v)[Vec<T>::N]);
template <>
__device__ __forceinline__ void store_vec<float>(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <>
__device__ __forceinline__ void store_vec<uint16_t>(uint16_t* p, const float (&v)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// Output rows of the apply passes: the type's own values, or (fp32, PIECES) three bf16 pieces of each value (cut3x2,
// piece_index).  row: first element of the row, c: the vector's first channel.
template <typename T, int V> struct __attribute__((aligned(V * sizeof(T)))) GnChunk { T e[V]; };
template <typename T, bool PIECES, int N>
__device__ __forceinline__ void store_out(T* out, int64_t row, int c, const float (&v)[N]) {
    if constexpr (N != Vec<T>::N) {                 // part of a vector
        GnChunk<T, N> o;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            if constexpr (sizeof(T) == 4) o.e[e] = v[e];
            else o.e[e] = float_to_bf16_bits(v[e]);
        }
        *reinterpret_cast<GnChunk<T, N>*>(out + row + c) = o;
    } else if constexpr (!PIECES) {
        store_vec<T>(out + row + c, v);
    } else {
        store_pieces4((uint16_t*)out + row + piece_index(c), v[0], v[1], v[2], v[3]);
    }
}

// 16 raw bytes of a row now, floats later: lets a kernel issue its row loads before loads it would otherwise wait for
template <typename T>
__device__ __forceinline__ void unpack_vec(const uint4& q, float (&v)[Vec<T>::N]);
template <>
__device__ __forceinline__ void unpack_vec<float>(const uint4& q, float (&v)[4]) {
    v[0] = __uint_as_float(q.x); v[1] = __uint_as_float(q.y); v[2] = __uint_as_float(q.z); v[3] = __uint_as_float(q.w);
}
template <>
__device__ __forceinline__ void unpack_vec<uint16_t>(const uint4& q, float (&v)[8]) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}

constexpr int GN_U = 8;     // token rows a thread keeps in flight

// thread (tl, cv): cv = channel vector (fixed channels for the whole kernel), tl = token lane.
// Moments that can be merged (Chan, Golub, LeVeque: combining the moments of two samples): a block leaves, per group,
// the mean and the sum of squared deviations M2 of its n = (tokens of the chunk) x (channels per group) elements.  The
// sums run over x - K with K = the channel's value in the chunk's first token, so that nothing is lost when the mean
// is far from zero (sum of squares minus square of the sum would lose the variance at |mean| >> deviation).
template <typename T>
__global__ void gn_partial_kernel(const T* __restrict__ x, int32_t C, int32_t G, int32_t S, int32_t nsplit,
                                  int32_t TL, float* __restrict__ partial) {
    constexpr int VN = Vec<T>::N;
    extern __shared__ float red[];             // [2][TL][C]
    const int CV = C / VN;
    const int cv = threadIdx.x % CV, tl = threadIdx.x / CV;
    const int p = blockIdx.x, sp = blockIdx.y;
    const int chunk = (S + nsplit - 1) / nsplit;
    const int t0 = sp * chunk, t1 = min(S, t0 + chunk);
    float s1[VN], s2[VN], k0[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) { s1[e] = 0.f; s2[e] = 0.f; }
    const T* base = x + ((int64_t)p * S) * C + cv * VN;
    load_vec<T>(base + (int64_t)min(t0, S - 1) * C, k0);       // the shift: this channel vector in the chunk's first token
    // up to GN_U independent 16-byte loads in flight per thread; rows past the chunk re-read its last row and are skipped
    for (int tb = t0 + tl; tb < t1; tb += GN_U * TL) {
        float v[GN_U][VN];
#pragma unroll
        for (int u = 0; u < GN_U; ++u) load_vec<T>(base + (int64_t)min(tb + u * TL, t1 - 1) * C, v[u]);
#pragma unroll
        for (int u = 0; u < GN_U; ++u) {
            if (tb + u * TL < t1) {
#pragma unroll
                for (int e = 0; e < VN; ++e) { const float d = v[u][e] - k0[e]; s1[e] += d; s2[e] = fmaf(d, d, s2[e]); }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < VN; ++e) {
        red[tl * C + cv * VN + e] = s1[e];
        red[(TL + tl) * C + cv * VN + e] = s2[e];
    }
    __syncthreads();
    // two short phases instead of one long serial loop per group: first the token lanes of every channel (plain sums:
    // one shift per channel), which leave the channel's mean and M2 over the chunk ...
    const float nt = (float)max(t1 - t0, 0);
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
        float a = 0.f, b = 0.f;
        for (int l = 0; l < TL; ++l) { a += red[l * C + c]; b += red[(TL + l) * C + c]; }
        const float kc = ld_f<T>(x + ((int64_t)p * S + min(t0, S - 1)) * C + c);
        const float inv = nt > 0.f ? 1.f / nt : 0.f;
        red[c] = kc + a * inv;                          // mean of the channel over the chunk
        red[TL * C + c] = fmaxf(b - a * a * inv, 0.f);  // M2 around it
    }
    __syncthreads();
    // ... then the channels of every group (equal counts: mean of the means, M2 by the merge formula; fixed order)
    const int cg = C / G;
    for (int g = threadIdx.x; g < G; g += blockDim.x) {
        float m = 0.f;
        for (int c = g * cg; c < (g + 1) * cg; ++c) m += red[c];
        m /= (float)cg;
        float m2 = 0.f;
        for (int c = g * cg; c < (g + 1) * cg; ++c) { const float d = red[c] - m; m2 += red[TL * C + c] + nt * d * d; }
        float* dst = partial + (((int64_t)p * nsplit + sp) * G + g) * 2;
        dst[0] = m;
        dst[1] = m2;
    }
}

constexpr int GN_FIN_THREADS = 256;

// block = four wavefronts per (request slot s, group g): merges the moments of all partials of the request in fp64.
// Partial i of a patch covers rows(i) = the tokens of chunk i (S split into `nsplit` chunks) times C/G channels;
// sum n_i mean_i and sum (M2_i + n_i mean_i^2) in fp64 give the mean and the M2 of the whole request (the fp64 sums
// carry 16 digits against the eight or so that |mean| / deviation can cost).
// epg = entries per group in a partial row: 1 (moments of whole groups) or C/G (moments of single channels, as the
// split pass leaves them: partial[p][chunk][C][2]).
template <typename T, int THREADS>
__global__ void __launch_bounds__(THREADS)
gn_finalize_kernel(const float* __restrict__ partial, const int32_t* __restrict__ request_offset,
                                   const T* __restrict__ gamma, const T* __restrict__ beta, int32_t C, int32_t G,
                                   int32_t S, int32_t nsplit, int32_t epg, float eps, float* __restrict__ scale_shift) {
    const int s = blockIdx.x, g = blockIdx.y;
    const int p0 = request_offset[s], p1 = request_offset[s + 1];
    const int items = (p1 - p0) * nsplit * epg;
    const int cg = C / G;
    const int chunk = (S + nsplit - 1) / nsplit;
    double a = 0.0, b = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < items; i += THREADS) {      // independent loads: several in flight per thread
        const int row = i / epg, e = i - row * epg;
        const float* src = partial + (((int64_t)p0 * nsplit + row) * G * epg + g * epg + e) * 2;
        const int sp = row % nsplit;
        const double n = (double)max(min(S, (sp + 1) * chunk) - sp * chunk, 0) * (cg / epg);
        const double m = (double)src[0];
        a += n * m;
        b += (double)src[1] + n * m * m;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    __shared__ double red[THREADS / 64][2];
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6][0] = a; red[threadIdx.x >> 6][1] = b; }
    __syncthreads();
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) { a += red[w][0]; b += red[w][1]; }    // fixed order: deterministic
    const double cnt = (double)(p1 - p0) * S * cg;
    const double mean = a / cnt;
    double var = b / cnt - mean * mean;
    var = var > 0.0 ? var : 0.0;
    const double rstd = 1.0 / sqrt(var + (double)eps);
    for (int c = g * cg + threadIdx.x; c < (g + 1) * cg; c += THREADS) {
        const double sc = rstd * (double)ld_f<T>(gamma + c);
        float* dst = scale_shift + ((int64_t)s * C + c) * 2;
        dst[0] = (float)sc;
        dst[1] = (float)((double)ld_f<T>(beta + c) - mean * sc);
    }
}

// Statistics of small requests in one launch: a block is one (request slot, group) and reads the group's channels of all
// the request's tokens (V channels a load).  Two launches of ~5 us each otherwise, of which the second waits for the first
// (1,024 tokens x 1280 channels in bf16: 12.1 -> 5.0 us back to back, 24 requests of it 19.8 -> 13.1).  A thread keeps mean
// and sum of squared deviations, the U * V elements of an iteration around their own mean and merged into it (Chan, Golub,
// LeVeque: all terms positive), so one far-off value costs no digits of the others; threads are merged in fp64.  (Sums of
// x - K with one K for the block took the same time and lost 3 digits of the variance when K was 1,000 deviations out.)
constexpr int GN_DIRECT_THREADS = 512;
// Mean and 1 / deviation of a block's elements: `items` chunks of V channels, `per` of them a token, rows of C from `base`
template <typename T, int V>
__device__ __forceinline__ void gn_moments(const T* __restrict__ base, int items, int per, int C, float eps, double& mu, double& rstd) {
    using Chunk = GnChunk<T, V>;
    float n = 0.f, mean = 0.f, m2 = 0.f;                        // moments of x - k0 over the n elements read so far
    float k0 = 0.f;                                             // fp32: the thread's first element (8 bits of bf16 need none)
    constexpr int U = 4;                                        // loads in flight
    for (int i = threadIdx.x; i < items; i += U * GN_DIRECT_THREADS) {
        Chunk v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(i + u * GN_DIRECT_THREADS, items - 1), t = j / per;
            v[u] = *reinterpret_cast<const Chunk*>(base + (int64_t)t * C + (j - t * per) * V);
        }
        if (sizeof(T) == 4 && n == 0.f) k0 = ld_f<T>(&v[0].e[0]);
        auto value = [&](int u, int e) { const float f = ld_f<T>(&v[u].e[e]); return sizeof(T) == 4 ? f - k0 : f; };
        float sum[U], dev[U], cnt = 0.f;                        // a chain of sums for every load
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = i + u * GN_DIRECT_THREADS < items;
            cnt += in ? (float)V : 0.f;
            sum[u] = 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) sum[u] += value(u, e);
            sum[u] = in ? sum[u] : 0.f;
        }
        // (a mean that is an ulp off shifts nothing: the deviations are taken from the value used)
        const float local = ((sum[0] + sum[1]) + (sum[2] + sum[3])) * __builtin_amdgcn_rcpf(cnt);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            dev[u] = 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) { const float d = value(u, e) - local; dev[u] = fmaf(d, d, dev[u]); }
            dev[u] = i + u * GN_DIRECT_THREADS < items ? dev[u] : 0.f;
        }
        const float delta = local - mean, share = cnt * __builtin_amdgcn_rcpf(n + cnt);
        mean = fmaf(delta, share, mean);
        m2 += ((dev[0] + dev[1]) + (dev[2] + dev[3])) + delta * delta * n * share;
        n += cnt;
    }
    const double at = (double)k0 + (double)mean;
    double a = (double)n * at, b = (double)m2 + a * at;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    __shared__ double red[GN_DIRECT_THREADS / 64][2];
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6][0] = a; red[threadIdx.x >> 6][1] = b; }
    __syncthreads();
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int w = 0; w < GN_DIRECT_THREADS / 64; ++w) { a += red[w][0]; b += red[w][1]; }    // fixed order: deterministic
    const double total = (double)items * V;
    mu = a / total;
    double var = b / total - mu * mu;
    var = var > 0.0 ? var : 0.0;
    rstd = 1.0 / sqrt(var + (double)eps);
}

template <typename T, int V>
__global__ void __launch_bounds__(GN_DIRECT_THREADS)
gn_direct_kernel(const T* __restrict__ x, const int32_t* __restrict__ request_offset, const T* __restrict__ gamma,
                 const T* __restrict__ beta, int32_t C, int32_t G, int32_t S, float eps, float* __restrict__ scale_shift) {
    const int s = blockIdx.x, g = blockIdx.y, cg = C / G, per = cg / V;
    const int p0 = request_offset[s], items = (request_offset[s + 1] - p0) * S * per;
    double mu, rstd;
    gn_moments<T, V>(x + (int64_t)p0 * S * C + g * cg, items, per, C, eps, mu, rstd);
    for (int c = g * cg + threadIdx.x; c < (g + 1) * cg; c += GN_DIRECT_THREADS) {
        const double sc = rstd * (double)ld_f<T>(gamma + c);
        float* dst = scale_shift + ((int64_t)s * C + c) * 2;
        dst[0] = (float)sc;
        dst[1] = (float)((double)ld_f<T>(beta + c) - mu * sc);
    }
}

template <typename T>
static int gn_direct(const GroupNormArgs& a, const PatchGeom& g, hipStream_t st) {
    const int cg = a.C / a.G;
#define PS_GND(V) gn_direct_kernel<T, V><<<dim3(a.n, a.G), GN_DIRECT_THREADS, 0, st>>>((const T*)a.x, a.request_offset, \
        (const T*)a.gamma, (const T*)a.beta, a.C, a.G, g.S, a.eps, a.scale_shift)
    if (sizeof(T) == 2 && cg % 8 == 0) PS_GND(16 / sizeof(T));
    else if (cg % 4 == 0) PS_GND(4);
    else if (cg % 2 == 0) PS_GND(2);
    else PS_GND(1);
#undef PS_GND
    return check_launch("gn_direct_kernel");
}

// v * sigmoid(v) with the hardware reciprocal (1 ulp): a true division expands to ten instructions per element
__device__ __forceinline__ float silu_f(float v) { return v * __builtin_amdgcn_rcpf(1.f + __expf(-v)); }

// Edge stitching fused into the normalisation (the push form of the paper's "Patch Edge Stitcher"): a border
// token's normalised value is also written into the ring slot of every same-image neighbour patch that needs
// it; where that neighbour is absent (image edge) the token zero-fills the matching ring slot of its OWN patch.
// Every ring slot of every patch is written by exactly one thread, so there is no race and no extra pass.
template <typename T, bool PIECES, int N>
__device__ __forceinline__ void stitch_store(T* __restrict__ out, const int32_t (&nb)[8], const PatchGeom& gm,
                                             int p, int y, int x, int C, int coff, const float (&v)[N]) {
    if (y != 0 && y != gm.ph - 1 && x != 0 && x != gm.pw - 1) return;
    const int CW = PIECES ? 3 * C : C;
    float z[N];
#pragma unroll
    for (int e = 0; e < N; ++e) z[e] = 0.f;
    int k = 0;
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
            if (dy == 0 && dx == 0) continue;
            const bool on = (dy == 0 || (dy < 0 ? y == 0 : y == gm.ph - 1)) && (dx == 0 || (dx < 0 ? x == 0 : x == gm.pw - 1));
            if (on) {
                const int q = nb[k];
                if (q >= 0)
                    store_out<T, PIECES>(out, ((int64_t)q * gm.pS + (y - dy * gm.ph + 1) * gm.ppw + (x - dx * gm.pw + 1)) * CW, coff, v);
                else
                    store_out<T, PIECES>(out, ((int64_t)p * gm.pS + (y + dy + 1) * gm.ppw + (x + dx + 1)) * CW, coff, z);
            }
            ++k;
        }
}

// Statistics and application in one launch, for small batches, where a launch costs what its kernel does.  A block is one
// (request, group) and one of gridDim.z shares of its elements: every share reads them all for the moments (the same value
// in each: fixed order), then its own once more, out of the caches.  Bound by latency.  CONV: SiLU, padded, stitched.
constexpr int GN_WHOLE_CG = 256;        // channels of a group at most
template <typename T, int V, bool CONV>
__global__ void __launch_bounds__(GN_DIRECT_THREADS)
gn_whole_kernel(const T* __restrict__ x, const int32_t* __restrict__ request_offset, const int32_t* __restrict__ neighbour,
                const T* __restrict__ gamma, const T* __restrict__ beta, PatchGeom gm, int32_t C, int32_t G, float eps, T* __restrict__ out) {
    using Chunk = GnChunk<T, V>;
    const int s = blockIdx.x, g = blockIdx.y, cg = C / G, per = cg / V;
    const int p0 = request_offset[s], items = (request_offset[s + 1] - p0) * gm.S * per;
    const T* base = x + (int64_t)p0 * gm.S * C + g * cg;
    __shared__ float l_sc[GN_WHOLE_CG], l_sh[GN_WHOLE_CG];
    double mu, rstd;
    gn_moments<T, V>(base, items, per, C, eps, mu, rstd);
    for (int c = threadIdx.x; c < cg; c += GN_DIRECT_THREADS) {
        const double sc = rstd * (double)ld_f<T>(gamma + g * cg + c);
        l_sc[c] = (float)sc;
        l_sh[c] = (float)((double)ld_f<T>(beta + g * cg + c) - mu * sc);
    }
    __syncthreads();
    const int share = (items + (int)gridDim.z - 1) / (int)gridDim.z, end = min(items, ((int)blockIdx.z + 1) * share);
    constexpr int U = 4;                        // loads in flight
    for (int i = blockIdx.z * share + threadIdx.x; i < end; i += U * GN_DIRECT_THREADS) {
        Chunk raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(i + u * GN_DIRECT_THREADS, end - 1), t = j / per;
            raw[u] = *reinterpret_cast<const Chunk*>(base + (int64_t)t * C + (j - t * per) * V);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = i + u * GN_DIRECT_THREADS, t = j / per, ch = (j - t * per) * V;
            if (j >= end) break;
            float v[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                v[e] = fmaf(ld_f<T>(&raw[u].e[e]), l_sc[ch + e], l_sh[ch + e]);
                if (CONV) v[e] = silu_f(v[e]);
            }
            const int pl = t / gm.S, q = t - pl * gm.S, p = p0 + pl;
            if constexpr (CONV) {
                const int py = q / gm.pw, px = q - py * gm.pw;
                store_out<T, false>(out, ((int64_t)p * gm.pS + (py + 1) * gm.ppw + px + 1) * C, g * cg + ch, v);
                if (py == 0 || py == gm.ph - 1 || px == 0 || px == gm.pw - 1) {
                    int32_t nb[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) nb[k] = neighbour[8 * p + k];
                    stitch_store<T, false>(out, nb, gm, p, py, px, C, g * cg + ch, v);
                }
            } else {
                store_out<T, false>(out, ((int64_t)p * gm.S + q) * C, g * cg + ch, v);
            }
        }
    }
}

// rim_only (padded output): patches with rim_only[p] != 0 are not convolved themselves (their result is reused); only
// their border tokens are normalised, because the neighbours' rings need them.
template <typename T, bool SILU, bool PADDED, bool STITCH, bool PIECES>
__global__ void gn_apply_kernel(const T* __restrict__ x, const float* __restrict__ scale_shift,
                                const int32_t* __restrict__ owner, const int32_t* __restrict__ neighbour, PatchGeom gm,
                                int32_t C, int32_t nsplit, int32_t TL, ActiveList act, const uint8_t* __restrict__ rim_only,
                                T* __restrict__ out) {
    constexpr int VN = Vec<T>::N;
    const int CW = PIECES ? 3 * C : C;          // elements of an output row
    int p = blockIdx.x;
    if (act.active) {
        if (p >= *act.count) return;
        p = act.active[p];
    }
    if (PADDED && rim_only && rim_only[p]) {
        // border token b of the patch: top row, bottom row, then left / right column of the rows between
        const int CVb = C / VN, cvb = threadIdx.x % CVb;
        const int nb_tok = gm.ph > 1 ? 2 * gm.pw + 2 * (gm.ph - 2) : gm.pw;
        // a few blocks with about four border tokens per thread row (as for whole patches); the others leave at once
        const int per = max((nb_tok + nsplit - 1) / nsplit, 4 * TL);
        const int b0 = blockIdx.y * per, b1 = min(nb_tok, b0 + per);
        if (b0 >= b1) return;
        float sc[VN], sh[VN];
        const float* ss = scale_shift + ((int64_t)owner[p] * C + cvb * VN) * 2;
#pragma unroll
        for (int e = 0; e < VN; ++e) { sc[e] = scale_shift ? ss[2 * e] : 1.f; sh[e] = scale_shift ? ss[2 * e + 1] : 0.f; }
        int32_t nbr[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) nbr[k] = STITCH ? neighbour[8 * p + k] : -1;
        for (int b = b0 + (int)threadIdx.x / CVb; b < b1; b += TL) {
            int y, xx;
            if (b < gm.pw) { y = 0; xx = b; }
            else if (b < 2 * gm.pw) { y = gm.ph - 1; xx = b - gm.pw; }
            else { const int r = b - 2 * gm.pw; y = 1 + (r >> 1); xx = (r & 1) ? gm.pw - 1 : 0; }
            float v[VN];
            load_vec<T>(x + ((int64_t)p * gm.S + y * gm.pw + xx) * C + cvb * VN, v);
#pragma unroll
            for (int e = 0; e < VN; ++e) {
                v[e] = fmaf(v[e], sc[e], sh[e]);
                if (SILU) v[e] = silu_f(v[e]);
            }
            store_out<T, PIECES>(out, ((int64_t)p * gm.pS + (y + 1) * gm.ppw + xx + 1) * CW, cvb * VN, v);
            if (STITCH) stitch_store<T, PIECES>(out, nbr, gm, p, y, xx, C, cvb * VN, v);
        }
        return;
    }
    const int CV = C / VN;
    const int cv = threadIdx.x % CV, tl = threadIdx.x / CV;
    const int sp = blockIdx.y;
    const int chunk = (gm.S + nsplit - 1) / nsplit;
    const int t0 = sp * chunk, t1 = min(gm.S, t0 + chunk);
    // Rows of this thread: t0 + tl + k*TL.  Their pixel coordinates and offsets advance by additions (a division and
    // 64-bit multiplications per row were a third of the kernel's vector instructions).
    const int pw = gm.pw;
    const int dyy = TL / pw, dxx = TL - dyy * pw;                       // one row step in pixel rows / columns
    const int step_in = TL * C;
    const int step_out = PADDED ? (dyy * gm.ppw + dxx) * CW : TL * CW;
    const int wrap_out = PADDED ? (gm.ppw - pw) * CW : 0;                // extra when the column wraps into the next pixel row
    int tb = t0 + tl;
    int py = tb / pw, px = tb - py * pw;
    const T* xin = x + ((int64_t)p * gm.S) * C + cv * VN;
    const int64_t po = ((int64_t)p * (PADDED ? gm.pS : gm.S)) * CW;
    int in_off = tb * C;
    int out_off = (PADDED ? (py + 1) * gm.ppw + px + 1 : tb) * CW;
    const int last_in = (t1 - 1) * C;
    // The row loads of the first batch go first: they depend on the patch only, while scale / shift hang on the
    // owner table (two dependent loads).  Up to GN_U independent 16-byte loads in flight per thread; rows past the
    // chunk re-read its last row and are skipped.
    uint4 raw[GN_U];
    if (tb < t1) {
#pragma unroll
        for (int u = 0; u < GN_U; ++u) raw[u] = *reinterpret_cast<const uint4*>(xin + min(in_off + u * step_in, last_in));
    }
    float sc[VN], sh[VN];
    if (scale_shift) {
        const int s = owner[p];
        const float* ss = scale_shift + ((int64_t)s * C + cv * VN) * 2;
#pragma unroll
        for (int e = 0; e < VN; ++e) { sc[e] = ss[2 * e]; sh[e] = ss[2 * e + 1]; }
    } else {                                    // no table: plain copy into the padded layout (with the rims)
#pragma unroll
        for (int e = 0; e < VN; ++e) { sc[e] = 1.f; sh[e] = 0.f; }
    }
    int32_t nb[8];                              // neighbour patches, read once (no dependent loads behind the stores)
#pragma unroll
    for (int k = 0; k < 8; ++k) nb[k] = (PADDED && STITCH) ? neighbour[8 * p + k] : -1;
    for (; tb < t1; tb += GN_U * TL) {
        float v[GN_U][VN];
#pragma unroll
        for (int u = 0; u < GN_U; ++u) unpack_vec<T>(raw[u], v[u]);
        in_off += GN_U * step_in;
        if (tb + GN_U * TL < t1) {              // next batch in flight while this one is finished
#pragma unroll
            for (int u = 0; u < GN_U; ++u) raw[u] = *reinterpret_cast<const uint4*>(xin + min(in_off + u * step_in, last_in));
        }
#pragma unroll
        for (int u = 0; u < GN_U; ++u) {
            if (tb + u * TL < t1) {
#pragma unroll
                for (int e = 0; e < VN; ++e) {
                    v[u][e] = fmaf(v[u][e], sc[e], sh[e]);
                    if (SILU) v[u][e] = silu_f(v[u][e]);
                }
                store_out<T, PIECES>(out, po + out_off, cv * VN, v[u]);
                if (PADDED && STITCH) stitch_store<T, PIECES>(out, nb, gm, p, py, px, C, cv * VN, v[u]);
            }
            // next row of this thread
            px += dxx;
            py += dyy;
            out_off += step_out;
            if (px >= pw) { px -= pw; ++py; out_off += wrap_out; }
        }
    }
}

// ---- per-token LayerNorm over the channels -------------------------------------------------------------------
// LPT lanes (a power of two) share a token; lane `sub` holds the 16-byte vectors sub, sub + LPT, ... (VPL of them) of
// the row in registers.  Mean, then variance around it (two passes over the registers), each reduced by a butterfly
// over the LPT lanes; fp32 throughout.  One 16-byte load and one 16-byte store per vector: 2*b*C bytes per token.
// A wavefront has few tokens, so what it waits for decides: everything it needs besides the row is asked for beside it, the
// next token's row before the current one is reduced, and the butterfly stays in the vector unit where it can (bf16:
// 14,272 tokens x 1280 channels 22.2 -> 14.4 us, 13,312 x 640 12.3 -> 8.5, 1,024 x 1280 7.1 -> 5.1, adaptive 12,288 x 1536 23.5 -> 18.5).
__device__ __forceinline__ float lane_sum(float v, int lpt) {
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    // quads, then mirrors (the halves of a mirrored row hold one value each: the same sums as with lane ^ 4 and ^ 8)
    if (lpt > 1) v += dpp(v, std::integral_constant<int, 0xB1>{});           // lane ^ 1
    if (lpt > 2) v += dpp(v, std::integral_constant<int, 0x4E>{});           // lane ^ 2
    if (lpt > 4) v += dpp(v, std::integral_constant<int, 0x141>{});          // 7 - lane in eights
    if (lpt > 8) v += dpp(v, std::integral_constant<int, 0x140>{});          // 15 - lane in sixteens
    if (lpt > 16) v += __shfl_xor(v, 16, 64);
    if (lpt > 32) v += __shfl_xor(v, 32, 64);
    return v;
}

template <typename T, int VPL, bool MOD, bool PIECES>
__global__ void __launch_bounds__(256)
layer_norm_kernel(const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
                  const float* __restrict__ mod, int64_t mod_ld, const int32_t* __restrict__ owner,
                  const float* __restrict__ mod_txt, const int32_t* __restrict__ patch_rc, int32_t C, int32_t S,
                  int32_t LPT, float eps, ActiveList act, T* __restrict__ out) {
    constexpr int VN = Vec<T>::N;
    int p = blockIdx.x;
    if (act.active) {
        if (p >= *act.count) return;                            // the list may be no longer than its count
        p = act.active[p];
    }
    const int CV = C / VN;
    const int sub = threadIdx.x % LPT, tl = threadIdx.x / LPT, tpb = blockDim.x / LPT;
    int t = blockIdx.y * tpb + tl;
    uint4 raw[VPL];
    auto load = [&](int tt) {
        const T* px = x + ((int64_t)p * S + min(tt, S - 1)) * C;
#pragma unroll
        for (int k = 0; k < VPL; ++k) raw[k] = *reinterpret_cast<const uint4*>(px + min(sub + k * LPT, CV - 1) * VN);
    };
    load(t);
    // adaptive form (MOD): [shift | scale] of the request, of the patch's stream where there are two
    constexpr int MV = MOD ? VPL : 1, RV = MOD ? 1 : VPL;
    uint4 graw[RV], braw[RV];
    float gm[MV][VN], bm[MV][VN];
    if constexpr (MOD) {
        const int own = owner[p], side = mod_txt ? patch_rc[2 * p] : 0;
        const float* mrow = (side < 0 ? mod_txt : mod) + (int64_t)own * mod_ld;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int c = min(sub + k * LPT, CV - 1) * VN;
#pragma unroll
            for (int e = 0; e < VN; ++e) { bm[k][e] = mrow[c + e]; gm[k][e] = mrow[C + c + e]; }
        }
    } else {
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int cv = min(sub + k * LPT, CV - 1);
            graw[k] = *reinterpret_cast<const uint4*>(gamma + cv * VN);
            braw[k] = *reinterpret_cast<const uint4*>(beta + cv * VN);
        }
    }
    const float inv_c = 1.f / (float)C;
    const bool tail = sub + (VPL - 1) * LPT < CV;               // the lane's last vector exists (all others do)
    const int step = gridDim.y * tpb;
    // kept as loaded and unpacked where they are used: fp32 copies would cost wavefronts in flight
    auto as_loaded = [](uint4& q) { asm volatile("" : "+v"(q.x), "+v"(q.y), "+v"(q.z), "+v"(q.w)); };
    for (; t < S; t += step) {
        uint4 cur[VPL];
#pragma unroll
        for (int k = 0; k < VPL; ++k) { cur[k] = raw[k]; as_loaded(cur[k]); }
        if (t + step < S) load(t + step);
        float v[VN], s1 = 0.f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            if (k < VPL - 1 || tail) {
                unpack_vec<T>(cur[k], v);
#pragma unroll
                for (int e = 0; e < VN; ++e) s1 += v[e];
            }
        }
        const float mean = lane_sum(s1, LPT) * inv_c;
        float s2 = 0.f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            as_loaded(cur[k]);
            if (k < VPL - 1 || tail) {
                unpack_vec<T>(cur[k], v);
#pragma unroll
                for (int e = 0; e < VN; ++e) { v[e] -= mean; s2 = fmaf(v[e], v[e], s2); }
            }
        }
        const float rstd = 1.f / sqrtf(lane_sum(s2, LPT) * inv_c + eps);
        const int64_t po = ((int64_t)p * S + t) * (PIECES ? 3 * C : C);
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            as_loaded(cur[k]);
            if (k < VPL - 1 || tail) {
                float g[VN], b[VN];
                if constexpr (MOD) {
#pragma unroll
                    for (int e = 0; e < VN; ++e) { b[e] = bm[k][e]; g[e] = 1.f + gm[k][e]; }
                } else {
                    as_loaded(graw[k]);
                    as_loaded(braw[k]);
                    unpack_vec<T>(graw[k], g);
                    unpack_vec<T>(braw[k], b);
                }
                unpack_vec<T>(cur[k], v);
#pragma unroll
                for (int e = 0; e < VN; ++e) v[e] = fmaf((v[e] - mean) * rstd, g[e], b[e]);
                store_out<T, PIECES>(out, po, (sub + k * LPT) * VN, v);
            }
        }
    }
}

// one thread per (ring entry, channel vector) of an active patch
template <typename T>
__global__ void halo_gather_kernel(T* __restrict__ apad, const int32_t* __restrict__ halo_src, PatchGeom gm,
                                   int32_t C, int32_t ring, ActiveList act) {
    constexpr int VN = Vec<T>::N;
    int p = blockIdx.x;
    if (act.active) {
        if (p >= *act.count) return;
        p = act.active[p];
    }
    const int CV = C / VN;
    const int items = ring * CV;
    for (int i = blockIdx.y * blockDim.x + threadIdx.x; i < items; i += gridDim.y * blockDim.x) {
        const int k = i / CV, cv = i - k * CV;
        int y, x;                          // ring pixel relative to the patch origin
        if (k < gm.pw + 2) { y = -1; x = k - 1; }
        else if (k < 2 * (gm.pw + 2)) { y = gm.ph; x = k - (gm.pw + 2) - 1; }
        else if (k < 2 * (gm.pw + 2) + gm.ph) { y = k - 2 * (gm.pw + 2); x = -1; }
        else { y = k - 2 * (gm.pw + 2) - gm.ph; x = gm.pw; }
        const int tok = halo_src[(int64_t)p * ring + k];
        uint4 v = make_uint4(0, 0, 0, 0);
        if (tok >= 0) {
            const int q = tok / gm.S, r = tok - q * gm.S;
            const int ys = r / gm.pw, xs = r - ys * gm.pw;
            v = *reinterpret_cast<const uint4*>(apad + ((int64_t)q * gm.pS + (ys + 1) * gm.ppw + xs + 1) * C + cv * VN);
        }
        *reinterpret_cast<uint4*>(apad + ((int64_t)p * gm.pS + (y + 1) * gm.ppw + x + 1) * C + cv * VN) = v;
    }
}

// ---- host side ---------------------------------------------------------------------------------
static int norm_layout(int32_t C, int dtype, int* CV, int* TL) {
    const int vn = dtype == PSERVE_BF16 ? 8 : 4;
    PS_REQUIRE(C % vn == 0, "GroupNorm: C=%d must be a multiple of %d for this dtype", C, vn);
    *CV = C / vn;
    PS_REQUIRE(*CV <= 1024, "GroupNorm: C=%d too wide", C);
    int tl = (256 + *CV / 2) / *CV;
    if (tl < 1) tl = 1;
    while (tl * *CV > 1024) --tl;
    *TL = tl;
    return PSERVE_OK;
}

bool gn_takes_direct(const GroupNormArgs& a, const PatchGeom& g, int dtype) {
    // One launch for small requests: a block reads its request's tokens in pieces of C / G channels, so its time grows with
    // its elements and, past an L2's 4 MB, with the lines shared between groups.  us, two launches -> one:
    // G = 32 at 1,024 tokens, 1 .. 24 requests of 64 .. 1280 channels: 6.2 .. 27 -> 3.4 .. 20, always faster; at 2,048, 6
    // requests of C = 320: bf16 9.6 -> 6.0, fp32 (16 MB) 9.5 -> 12.0; bf16 C = 640: 3 requests 10.0 -> 8.3, 6 (16 MB) 10.2 -> 12.1.
    // Few wide groups up to 1,024 tokens: always faster too (fp32, G = 1: C = 320 35.9 -> 8.3 at 256, 37.0 -> 25.6 at 1,024).  At
    // 2,048 the block's elements decide in fp32 (163,840: 14.5 -> 14.3; 655,360: 37.3 -> 48.7; bf16 35.8 -> 33.8), and more than
    // 32 groups share too many lines (G = 64, 3 requests: fp32 C = 320 7.4 -> 11.3, bf16 C = 640 9.1 -> 11.4).
    const int64_t bytes = (int64_t)g.P * g.S * a.C * dtype_size(dtype), block = (int64_t)a.max_tokens * (a.C / a.G);
    return a.max_tokens <= 1024 ||
           (a.max_tokens <= 2048 && bytes <= (8 << 20) && a.G <= 32 && (dtype == PSERVE_BF16 || block <= 200000));
}

template <typename T>
static int gn_whole(const GroupNormArgs& a, const PatchGeom& g, bool conv, void* out, hipStream_t st) {
    const int cg = a.C / a.G;
    const int z = (int)std::max<int64_t>(1, std::min<int64_t>(256 / ((int64_t)a.n * a.G), 4));
#define PS_GNW(V)                                                                                                        \
    {                                                                                                                    \
        if (conv) gn_whole_kernel<T, V, true><<<dim3(a.n, a.G, z), GN_DIRECT_THREADS, 0, st>>>((const T*)a.x, a.request_offset, a.neighbour, \
            (const T*)a.gamma, (const T*)a.beta, g, a.C, a.G, a.eps, (T*)out);                                           \
        else gn_whole_kernel<T, V, false><<<dim3(a.n, a.G, z), GN_DIRECT_THREADS, 0, st>>>((const T*)a.x, a.request_offset, a.neighbour, \
            (const T*)a.gamma, (const T*)a.beta, g, a.C, a.G, a.eps, (T*)out);                                           \
    }
    if (sizeof(T) == 2 && cg % 8 == 0) PS_GNW(16 / sizeof(T))
    else if (cg % 4 == 0) PS_GNW(4)
    else if (cg % 2 == 0) PS_GNW(2)
    else PS_GNW(1)
#undef PS_GNW
    return check_launch("gn_whole_kernel");
}

bool gn_takes_whole(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool conv) {
    // us, two launches -> one, bf16: 64 tokens 7 .. 10.5 -> 5.0 .. 5.6 into the padded buffer, 6.2 .. 9 -> 3.6 .. 5 plain (C = 64 .. 1280,
    // G = 32); 1,024 tokens 8.7 .. 12.8 -> 5.8 .. 9.9, 7.1 .. 11.4 -> 4.2 .. 8.1; 2,048 tokens 8.9 .. 14.9 -> 6.0 .. 12.4.  Past
    // that the pieces of C / G channels in which a block writes cost more than the launch, at rows of ten channels first:
    // 4,096 tokens C = 320 11.2 -> 13.2, C = 1280 17.9 -> 18.4, 12,288 15.5 -> 26.8; plain 10.1 -> 8.4, 13.6 -> 12.2, 13.0 -> 15.0.
    // A block of many elements reads them alone: G = 1, C = 128: 256 tokens (32,768) 10.6 -> 9.8, 512 11.2 -> 12.1, 1,024 13.6 -> 17.9.
    return gn_takes_direct(a, g, dtype) && a.C / a.G <= GN_WHOLE_CG && (int64_t)a.max_tokens * (a.C / a.G) <= 40960 &&
           (int64_t)g.P * g.S <= (conv ? 2048 : 4096);
}
int gn_whole(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool conv, void* out, hipStream_t st) {
    int CV, TL;
    PS_TRY(norm_layout(a.C, dtype, &CV, &TL));
    PS_REQUIRE(a.C % a.G == 0, "GroupNorm: C %% G != 0");
    return dtype == PSERVE_BF16 ? gn_whole<uint16_t>(a, g, conv, out, st) : gn_whole<float>(a, g, conv, out, st);
}

int gn_stats(const GroupNormArgs& a, const PatchGeom& g, int dtype, hipStream_t st) {
    int CV, TL;
    PS_TRY(norm_layout(a.C, dtype, &CV, &TL));
    PS_REQUIRE(a.C % a.G == 0, "GroupNorm: C %% G != 0");
    const size_t lds = sizeof(float) * 2 * TL * a.C;
    PS_REQUIRE(lds <= 64 * 1024, "GroupNorm: C=%d too wide for the reduction buffer", a.C);
    if (gn_takes_direct(a, g, dtype)) return dtype == PSERVE_BF16 ? gn_direct<uint16_t>(a, g, st) : gn_direct<float>(a, g, st);
    dim3 grid(g.P, a.nsplit);
    if (dtype == PSERVE_BF16)
        gn_partial_kernel<uint16_t><<<grid, TL * CV, lds, st>>>((const uint16_t*)a.x, a.C, a.G, g.S, a.nsplit, TL, a.partial);
    else
        gn_partial_kernel<float><<<grid, TL * CV, lds, st>>>((const float*)a.x, a.C, a.G, g.S, a.nsplit, TL, a.partial);
    PS_TRY(check_launch("gn_partial_kernel"));
    return gn_finalize(a, g, dtype, a.nsplit, st, false);
}

int gn_finalize(const GroupNormArgs& a, const PatchGeom& g, int dtype, int32_t slots, hipStream_t st, bool per_channel) {
    dim3 fgrid(a.n, a.G);
    const int epg = per_channel ? a.C / a.G : 1;
    // per-channel entries: C / G times as many per (request, group): 1,024 threads (a 256^2 latent in 32 x 32 patches
    // has 10,240 of them; with 256 threads that block alone took 27 us)
#define PS_FIN(T, TH)                                                                                              \
    gn_finalize_kernel<T, TH><<<fgrid, TH, 0, st>>>(a.partial, a.request_offset, (const T*)a.gamma, (const T*)a.beta, a.C, \
                                                    a.G, g.S, slots, epg, a.eps, a.scale_shift)
    if (dtype == PSERVE_BF16) { if (per_channel) PS_FIN(uint16_t, 1024); else PS_FIN(uint16_t, GN_FIN_THREADS); }
    else { if (per_channel) PS_FIN(float, 1024); else PS_FIN(float, GN_FIN_THREADS); }
#undef PS_FIN
    return check_launch("gn_finalize_kernel");
}

constexpr int APPLY_ROWS = 4;        // rows per thread of the apply pass (measured: 1-2 too many blocks, 6-8 too few)

template <typename T>
static void launch_apply(const GroupNormArgs& a, const PatchGeom& g, bool silu, bool padded, bool stitch, void* out,
                         ActiveList act, int CV, int TL, bool pieces, hipStream_t st) {
    // Own chunking (independent of the statistics pass): about APPLY_ROWS rows per thread.  Many short blocks are
    // dispatched over time, so some load while others compute or store; with few long blocks every wavefront of
    // the chip is in the same phase at once.
    const int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(cdiv(g.S, (int64_t)APPLY_ROWS * TL), 65535));
    dim3 grid(g.P, nsplit);
    const int nt = TL * CV;
#define PS_APPLY_(SI, PA, ST, PI)                                                                                     \
    gn_apply_kernel<T, SI, PA, ST, PI><<<grid, nt, 0, st>>>((const T*)a.x, a.scale_shift, a.owner, a.neighbour, g, a.C, \
                                                            nsplit, TL, act, a.rim_only, (T*)out)
#define PS_APPLY(SI, PA, ST) PS_APPLY_(SI, PA, ST, false)
    if constexpr (sizeof(T) == 4) {
        if (pieces) {                       // what feeds a layer: the stitched form of a convolution, the plain one of an attention
            if (padded) PS_APPLY_(true, true, true, true);
            else PS_APPLY_(false, false, false, true);
            return;
        }
    }
    if (silu && padded && stitch) PS_APPLY(true, true, true);
    else if (padded && stitch) PS_APPLY(false, true, true);
    else if (silu && padded) PS_APPLY(true, true, false);
    else if (silu) PS_APPLY(true, false, false);
    else if (padded) PS_APPLY(false, true, false);
    else PS_APPLY(false, false, false);
#undef PS_APPLY
#undef PS_APPLY_
}

int gn_apply(const GroupNormArgs& a, const PatchGeom& g, int dtype, bool silu, bool padded, bool stitch, void* out,
             ActiveList act, hipStream_t st, bool pieces) {
    int CV, TL;
    PS_TRY(norm_layout(a.C, dtype, &CV, &TL));
    PS_REQUIRE(!pieces || (dtype == PSERVE_F32 && silu == padded && stitch == padded), "gn_apply: no such form in pieces");
    PS_REQUIRE(!stitch || (padded && a.neighbour && !act.active), "gn_apply: stitching needs the padded layout and all patches");
    if (dtype == PSERVE_BF16) launch_apply<uint16_t>(a, g, silu, padded, stitch, out, act, CV, TL, false, st);
    else launch_apply<float>(a, g, silu, padded, stitch, out, act, CV, TL, pieces, st);
    return check_launch("gn_apply_kernel");
}

template <typename T>
static void launch_layer_norm(const void* x, const void* gamma, const void* beta, const float* mod, int64_t mod_ld,
                              const int32_t* owner, const float* mod_txt, const int32_t* patch_rc, int32_t C, float eps,
                              const PatchGeom& g, void* out, ActiveList act, int LPT, int VPL, bool pieces, hipStream_t st) {
    const int tpb = 256 / LPT;
    // one token per lane group while that gives at most ~16 blocks per CU, else more tokens per group
    int64_t per = 1;
    while (per < 8 && g.P * cdiv(g.S, tpb * per) > 4096) per *= 2;
    dim3 grid(g.P, (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(g.S, tpb * per), 65535)));
    constexpr bool F32 = sizeof(T) == 4;
#define PS_LNP(V, M, PI) layer_norm_kernel<T, V, M, PI><<<grid, 256, 0, st>>>((const T*)x, (const T*)gamma, (const T*)beta, mod, mod_ld, owner, mod_txt, patch_rc, C, g.S, LPT, eps, act, (T*)out)
#define PS_LNK(V, M) do { if (F32 && pieces) PS_LNP(V, M, F32); else PS_LNP(V, M, false); } while (0)
#define PS_LN(V) case V: if (mod) PS_LNK(V, true); else PS_LNK(V, false); break
    switch (VPL) { PS_LN(1); PS_LN(2); PS_LN(3); PS_LN(4); PS_LN(5); PS_LN(6); PS_LN(7); PS_LN(8); }
#undef PS_LN
#undef PS_LNK
#undef PS_LNP
}

int layer_norm(const void* x, const void* gamma, const void* beta, const float* mod, int64_t mod_ld, const int32_t* owner,
               int32_t C, float eps, const PatchGeom& g, int dtype, void* out, ActiveList act, hipStream_t st,
               const float* mod_txt, const int32_t* patch_rc, bool pieces) {
    PS_REQUIRE(!pieces || dtype == PSERVE_F32, "LayerNorm: pieces are those of fp32 values");
    PS_REQUIRE((gamma && beta) || (mod && owner), "LayerNorm: neither gamma / beta nor a modulation table");
    if (gamma) mod = nullptr;
    const int vn = dtype == PSERVE_BF16 ? 8 : 4;
    PS_REQUIRE(C % vn == 0, "LayerNorm: C=%d must be a multiple of %d for this dtype", C, vn);
    const int CV = C / vn;
    PS_REQUIRE(CV <= 512, "LayerNorm: C=%d too wide", C);
    // lanes per token: the power of two that wastes the fewest vector slots (ties: more lanes)
    int LPT = 64, VPL = (int)cdiv(CV, 64), waste = VPL * 64 - CV;
    for (int l = 32; l >= 1; l >>= 1) {
        const int v = (int)cdiv(CV, l);
        if (v <= 8 && v * l - CV < waste) { LPT = l; VPL = v; waste = v * l - CV; }
    }
    if (dtype == PSERVE_BF16) launch_layer_norm<uint16_t>(x, gamma, beta, mod, mod_ld, owner, mod_txt, patch_rc, C, eps, g, out, act, LPT, VPL, false, st);
    else launch_layer_norm<float>(x, gamma, beta, mod, mod_ld, owner, mod_txt, patch_rc, C, eps, g, out, act, LPT, VPL, pieces, st);
    return check_launch("layer_norm_kernel");
}

int halo_gather(void* apad, const int32_t* halo_src, const PatchGeom& g, int32_t C, int32_t ring, int dtype,
                ActiveList act, hipStream_t st) {
    int CV, TL;
    PS_TRY(norm_layout(C, dtype, &CV, &TL));
    const int items = ring * CV;
    dim3 grid(g.P, (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(items, 256 * 4), 64)));
    if (dtype == PSERVE_BF16)
        halo_gather_kernel<uint16_t><<<grid, 256, 0, st>>>((uint16_t*)apad, halo_src, g, C, ring, act);
    else
        halo_gather_kernel<float><<<grid, 256, 0, st>>>((float*)apad, halo_src, g, C, ring, act);
    return check_launch("halo_gather_kernel");
}

}  // namespace pserve
