// Patch planner (Compressed Sparse Patch tables + neighbour / halo metadata) and the
// split / reassembly copies between per-image NCHW latents and the patch-major token matrix.
//
// Paper: section "Compressed Sparse Patch Format" (requests reordered by resolution,
// RequestOffset, per-patch request index, resolution offsets) and section
// "Patch-Tailored Diffusion Operators" (neighbours recorded at split time, absent
// neighbour = zero fill).
#include "common.h"

#include <algorithm>
#include <mutex>
#include <numeric>
#include <string.h>

namespace pserve {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

// ---- kernels ----------------------------------------------------------------------------

// Where the tables of one plan lie: offsets in int32 into an arena that the device and the host hold alike, each a multiple of
// 64 (PSERVE_TAB_* index; the sorted sizes stand at 0, the per-request tables behind them, then the four per-patch ones).
struct PlanLayout {
    int64_t request_offset, owner, rc, neighbour, halo_src, total;
};

// Requests whose sizes and offsets a block keeps in LDS, and the largest arena written to host memory as well
constexpr int PLAN_REQ = 256;
constexpr size_t PLAN_STAGE_BYTES = 1 << 20;

// One thread per entry of the arena, so that every store is one of 64 in a row: over the host link a scattered four-byte
// store costs as much as a whole line.  The patch's owner comes by binary search in RequestOffset (a serving batch has few
// requests).  HALO_SRC: global token id of the pixel one step outside the patch.  Text patches: local index >= gh * gw;
// grid position (-1, k), no neighbours.
// STAGED: the per-request tables are read from host memory (one trip per block, into LDS) and copied to the device arena,
// and the per-patch entries go to both arenas.  Else the device arena already holds the per-request part.
// Bound by latency: 24 requests with 40,000 entries take 14 us, an empty launch and the wait for it 12.
template <bool STAGED>
__global__ void __launch_bounds__(256)
plan_patches_kernel(int32_t* __restrict__ dev, int32_t* __restrict__ host, PlanLayout at, int32_t n, int32_t P, int32_t ph,
                    int32_t pw, int32_t ring) {
    __shared__ int32_t l_hw[STAGED ? 2 * PLAN_REQ : 1], l_ro[STAGED ? PLAN_REQ + 1 : 1];
    if (STAGED) {
        for (int k = threadIdx.x; k < 2 * n; k += 256) l_hw[k] = host[k];
        for (int k = threadIdx.x; k <= n; k += 256) l_ro[k] = host[at.request_offset + k];
        __syncthreads();
    }
    const int32_t* sorted_hw = STAGED ? l_hw : dev;
    const int32_t* request_offset = STAGED ? l_ro : dev + at.request_offset;
    for (int64_t e = (STAGED ? 0 : at.owner) + (int64_t)blockIdx.x * 256 + threadIdx.x; e < at.total; e += (int64_t)gridDim.x * 256) {
        if (STAGED && e < at.owner) {
            dev[e] = host[e];
            continue;
        }
        int p, k, kind;                           // entry k of patch p
        if (e < at.rc) { kind = 0; p = (int)(e - at.owner); k = 0; }
        else if (e < at.neighbour) { kind = 1; k = (int)(e - at.rc); p = k >> 1; k &= 1; }
        else if (e < at.halo_src) { kind = 2; k = (int)(e - at.neighbour); p = k >> 3; k &= 7; }
        else { kind = 3; k = (int)(e - at.halo_src); p = k / ring; k -= p * ring; }
        if (p >= P) continue;                     // between two tables
        int lo = 0, hi = n;                       // largest s with request_offset[s] <= p
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (request_offset[mid] <= p) lo = mid; else hi = mid;
        }
        const int s = lo, first = request_offset[s];
        const int H = sorted_hw[2 * s], W = sorted_hw[2 * s + 1], gh = H / ph, gw = W / pw;
        const int local = p - first;
        const bool image = local < gh * gw;
        const int r = image ? local / gw : -1, c = image ? local - r * gw : local - gh * gw;
        int32_t v = -1;
        if (kind == 0) v = s;
        else if (kind == 1) v = k ? c : r;
        else if (kind == 2) {
            const int j = k < 4 ? k : k + 1;      // the eight neighbours row by row, the patch itself left out
            const int rr = r + j / 3 - 1, cc = c + j % 3 - 1;
            if (image && rr >= 0 && rr < gh && cc >= 0 && cc < gw) v = first + rr * gw + cc;
        } else {
            int y, x;                             // ring pixel relative to the patch origin
            if (k < pw + 2) { y = -1; x = k - 1; }
            else if (k < 2 * (pw + 2)) { y = ph; x = k - (pw + 2) - 1; }
            else if (k < 2 * (pw + 2) + ph) { y = k - 2 * (pw + 2); x = -1; }
            else { y = k - 2 * (pw + 2) - ph; x = pw; }
            const int Y = r * ph + y, X = c * pw + x;                      // absolute pixel in the image
            if (image && Y >= 0 && Y < H && X >= 0 && X < W) {
                const int q = first + (Y / ph) * gw + (X / pw);
                v = q * ph * pw + (Y % ph) * pw + (X % pw);
            }
        }
        dev[e] = v;
        if (STAGED) host[e] = v;
    }
}

// Pinned host buffers that plans' tables pass through (allocating one takes longer than a whole pserve_plan call).  A buffer is in
// use only inside one call, which waits for its kernel before it returns, and serves any thread: as many as plan at once, four at most
// (a fifth call copies); when the last plan is freed all but one are given back.  Coherent memory: the kernel's reads and
// writes go to the host and not to a cache, so a buffer that the next call fills anew is never stale; what the kernel
// wrote is there when the wait for it returns.
constexpr int PLAN_STAGES = 4;
static struct {
    std::mutex m;
    int32_t* idle[PLAN_STAGES];
    int n_idle, total, plans;
} g_stages;
struct PlanStage {
    int32_t* p = nullptr;
    bool done = false;                          // the call's kernel has ended: another call may have the buffer
    void get() {
        {
            std::lock_guard<std::mutex> lock(g_stages.m);
            if (g_stages.n_idle) { p = g_stages.idle[--g_stages.n_idle]; return; }
            if (g_stages.total == PLAN_STAGES) return;
            ++g_stages.total;
        }
        if (hipHostMalloc((void**)&p, PLAN_STAGE_BYTES, hipHostMallocPortable | hipHostMallocCoherent) == hipSuccess) return;
        (void)hipGetLastError();
        p = nullptr;
        std::lock_guard<std::mutex> lock(g_stages.m);
        --g_stages.total;
    }
    ~PlanStage() {
        if (!p) return;
        if (done) {
            std::lock_guard<std::mutex> lock(g_stages.m);
            g_stages.idle[g_stages.n_idle++] = p;
            return;
        }
        (void)hipHostFree(p);
        std::lock_guard<std::mutex> lock(g_stages.m);
        --g_stages.total;
    }
};
static void plans_changed(int by) {
    int32_t* back[PLAN_STAGES];
    int n = 0;
    {
        std::lock_guard<std::mutex> lock(g_stages.m);
        g_stages.plans += by;
        if (g_stages.plans == 0)
            while (g_stages.n_idle > 1) { back[n++] = g_stages.idle[--g_stages.n_idle]; --g_stages.total; }
    }
    while (n) (void)hipHostFree(back[--n]);
}
// For tests (host only, no part of the ABI): pinned buffers that exist.
extern "C" int pserve_test_plan_stages() {
    std::lock_guard<std::mutex> lock(g_stages.m);
    return g_stages.total;
}

// ---- split / reassemble -------------------------------------------------------------------
constexpr int IMG_CHUNK = 32;
struct ImagePtrs {
    void* p[IMG_CHUNK];       // image of sorted slot slot0 + k
};

// Block = one patch row (patch p, row y) x 64 channels; 32-pixel chunks are transposed through LDS.
// TO_PATCH: NCHW image -> x[T][C]; else the reverse.
template <typename T, bool TO_PATCH>
__global__ void __launch_bounds__(256)
split_kernel(ImagePtrs imgs, int slot0, int patch0, const int32_t* __restrict__ sorted_hw,
             const int32_t* __restrict__ owner, const int32_t* __restrict__ rc, int32_t ph, int32_t pw, int32_t C,
             T* __restrict__ x) {
    __shared__ T tile[64][33];
    const int p = patch0 + blockIdx.x / ph;
    const int y = blockIdx.x % ph;
    const int c0 = blockIdx.y * 64;
    if (rc[2 * p] < 0) return;                  // a text patch: not part of any image
    const int s = owner[p];
    const int H = sorted_hw[2 * s], W = sorted_hw[2 * s + 1];
    T* img = (T*)imgs.p[s - slot0];
    const int Y = rc[2 * p] * ph + y, X0 = rc[2 * p + 1] * pw;
    const int64_t tok0 = (int64_t)p * ph * pw + (int64_t)y * pw;
    const int tid = threadIdx.x;
    for (int xc = 0; xc < pw; xc += 32) {
        if (TO_PATCH) {
            for (int i = tid; i < 64 * 32; i += 256) {
                const int px = i & 31, ch = i >> 5;
                if (xc + px < pw && c0 + ch < C)
                    tile[ch][px] = img[((int64_t)(c0 + ch) * H + Y) * W + X0 + xc + px];
            }
            __syncthreads();
            for (int i = tid; i < 64 * 32; i += 256) {
                const int ch = i & 63, px = i >> 6;
                if (xc + px < pw && c0 + ch < C) x[(tok0 + xc + px) * C + c0 + ch] = tile[ch][px];
            }
        } else {
            for (int i = tid; i < 64 * 32; i += 256) {
                const int ch = i & 63, px = i >> 6;
                if (xc + px < pw && c0 + ch < C) tile[ch][px] = x[(tok0 + xc + px) * C + c0 + ch];
            }
            __syncthreads();
            for (int i = tid; i < 64 * 32; i += 256) {
                const int px = i & 31, ch = i >> 5;
                if (xc + px < pw && c0 + ch < C)
                    img[((int64_t)(c0 + ch) * H + Y) * W + X0 + xc + px] = tile[ch][px];
            }
        }
        __syncthreads();
    }
}

// Any patch shape (C a multiple of 64): a channel's plane of an image is one run of H * W values, whatever the patches are, so a block
// takes 128 bytes of it (64 bf16 pixels, 32 fp32) in 64 channels, VEC pixels an access, and the 128 or 256 bytes of 64 channels of each of
// these pixels' tokens.  Transposed in LDS; 16-byte piece c of a pixel's row lies at c ^ (pixel / 16 bytes), so that neither side's accesses
// meet in a bank.  us, rows of patches with two-byte accesses (split_kernel) / here:
// 19,008 tokens x 512 in 12 x 12 patches 28.6 / 8.9 and back 22.2 / 7.3 (39 MB: 4.4 and 5.3 TB/s), 7,600 x 512 in 20 x 20 11.4 / 6.0 and 10.2 / 5.5,
// fp32 7,168 x 320 in 16 x 16 12.5 / 7.1 and 8.6 / 5.6, 832 x 64 4.5 / 3.0 and 3.9 / 2.9.  Against 16-byte accesses along the rows of bf16
// patches (back): 13,312 x 1280 in 8 x 8 26.0 / 12.2, 19,008 x 640 in 24 x 24 16.0 / 9.2, 20,480 x 512 in 16 x 32 8.8 / 8.1.
struct PlaneTiles {
    int32_t end[IMG_CHUNK];   // tiles of the launch's requests up to and with this one
};
template <typename T, int VEC, bool TO_PATCH>
__global__ void __launch_bounds__(256)
split_plane_kernel(ImagePtrs imgs, PlaneTiles at, int slot0, const int32_t* __restrict__ sorted_hw,
                   const int32_t* __restrict__ request_offset, int32_t ph, int32_t pw, int32_t C, T* __restrict__ x) {
    constexpr int PX = 128 / sizeof(T), E = 16 / sizeof(T), LOADS = 64 * PX / VEC / 256, STORES = PX * 64 / E / 256;
    struct alignas(VEC * sizeof(T)) Vec { T v[VEC]; };
    struct alignas(16) Row { T v[E]; };
    __shared__ __attribute__((aligned(16))) T tile[PX * 64];
    __shared__ int32_t s_tok[PX];
    const int tid = threadIdx.x, c0 = blockIdx.y * 64;
    int k = 0;
    while ((int)blockIdx.x >= at.end[k]) ++k;
    const int q0 = ((int)blockIdx.x - (k ? at.end[k - 1] : 0)) * PX, s = slot0 + k;
    const int H = sorted_hw[2 * s], W = sorted_hw[2 * s + 1], N = H * W;
    T* img = (T*)imgs.p[k];
    auto place = [&](int px, int ch) { return px * 64 + (((ch / E) ^ ((px / E) & 7)) * E) + ch % E; };
    auto plane = [&](int i) { return img + (int64_t)(c0 + i / (PX / VEC)) * N + q0 + i % (PX / VEC) * VEC; };
    Vec in[LOADS];
    if (TO_PATCH) {
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            const int i = tid + 256 * l;
            if (q0 + i % (PX / VEC) * VEC < N) in[l] = *reinterpret_cast<const Vec*>(plane(i));
        }
    }
    if (tid < PX) {
        const int q = min(q0 + tid, N - 1), Y = q / W, X = q - Y * W, r = Y / ph, c = X / pw;
        s_tok[tid] = (request_offset[s] + r * (W / pw) + c) * (ph * pw) + (Y - r * ph) * pw + X - c * pw;
    }
    if (TO_PATCH) {
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            const int i = tid + 256 * l;
#pragma unroll
            for (int v = 0; v < VEC; ++v) tile[place(i % (PX / VEC) * VEC + v, i / (PX / VEC))] = in[l].v[v];
        }
        __syncthreads();
#pragma unroll
        for (int l = 0; l < STORES; ++l) {
            const int i = tid + 256 * l, px = i / (64 / E), ch = i % (64 / E) * E;
            if (q0 + px < N) *reinterpret_cast<Row*>(x + (int64_t)s_tok[px] * C + c0 + ch) = *reinterpret_cast<const Row*>(tile + place(px, ch));
        }
    } else {
        __syncthreads();
#pragma unroll
        for (int l = 0; l < STORES; ++l) {
            const int i = tid + 256 * l, px = i / (64 / E), ch = i % (64 / E) * E;
            *reinterpret_cast<Row*>(tile + place(px, ch)) = *reinterpret_cast<const Row*>(x + (int64_t)s_tok[px] * C + c0 + ch);
        }
        __syncthreads();
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            const int i = tid + 256 * l;
            Vec out;
#pragma unroll
            for (int v = 0; v < VEC; ++v) out.v[v] = tile[place(i % (PX / VEC) * VEC + v, i / (PX / VEC))];
            if (q0 + i % (PX / VEC) * VEC < N) *reinterpret_cast<Vec*>(plane(i)) = out;
        }
    }
}

// Blocks go to the eight XCDs in turn: numbers b of one XCD get consecutive places, so neighbouring patches, whose rows share cache
// lines of the image, are read through one L2 (patches narrower than 64 bytes: 13,312 tokens x 1280 in 8 x 8 patches 26.0 -> 18.1 us with
// the next tile's load ahead, 19,008 x 640 in 24 x 24 17.3 -> 12.9; wider ones gain nothing, 32 wide 10.5 -> 11.5 at 20,480 x 512).
__device__ __forceinline__ int xcd_run(int b, int n) {
    const int q = n / 8, r = n % 8, xcd = b % 8;
    return xcd * q + min(xcd, r) + b / 8;
}

// Split (bf16 fast path) that also leaves the moments of every channel behind, for a GroupNorm that reads x next:
// block = (patch, one of `nch` token chunks, 64 channels); it walks the chunk's tiles of 32 tokens, one 16-byte access
// a thread on each side (8 pixels of a channel's row, 8 channels of a token), transposed in LDS, the next tile's pixels
// already on their way, and keeps, per thread, the sums of (x - K) and (x - K)^2 of its eight channels (K = the channel's value in the
// chunk's first token: nothing is lost when the mean is far from zero).  Per (patch, chunk, channel) it stores the
// mean and the sum of squared deviations M2 of the chunk's tokens: stats[((p * nch + chunk) * C + c) * 2 + {0, 1}],
// which the GroupNorm finalize merges (fixed order, no atomics).
__global__ void __launch_bounds__(256)
split_stats_kernel(ImagePtrs imgs, int slot0, int patch0, const int32_t* __restrict__ sorted_hw,
                   const int32_t* __restrict__ owner, const int32_t* __restrict__ rc, int32_t ph, int32_t pw, int32_t C,
                   int32_t nch, uint16_t* __restrict__ x, float* __restrict__ stats) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[32][72];      // [token][channel], rows padded to 144 bytes
    __shared__ float red[2][32][65];
    __shared__ float kk[64];
    const int S = ph * pw, tiles = S / 32, tpc = tiles / nch;
    const int bx = pw % 32 ? xcd_run(blockIdx.x, gridDim.x) : blockIdx.x;
    const int p = patch0 + bx / nch, tc = bx % nch;
    const int c0 = blockIdx.y * 64;
    if (rc[2 * p] < 0) return;                  // a text patch: not part of any image
    const int s = owner[p];
    const int H = sorted_hw[2 * s], W = sorted_hw[2 * s + 1];
    const uint16_t* img = (const uint16_t*)imgs.p[s - slot0];
    const int tid = threadIdx.x;
    const int ich = tid >> 2, iq = tid & 3;     // image side: channel ich, 8 pixels starting at token t0 + 8*iq
    const int ptk = tid >> 3, pq = tid & 7;     // patch side: token t0 + ptk, channels 8*pq .. +8
    const uint16_t* ibase = img + ((int64_t)(c0 + ich) * H + rc[2 * p] * ph) * W + rc[2 * p + 1] * pw;
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    float s1[8], s2[8], k0[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { s1[e] = 0.f; s2[e] = 0.f; k0[e] = 0.f; }
    auto load = [&](int ti) {
        const int it = (tc * tpc + ti) * 32 + 8 * iq, iy = it / pw, ix = it - iy * pw;
        return *reinterpret_cast<const u32x4*>(ibase + (int64_t)iy * W + ix);
    };
    u32x4 next = load(0);
    for (int ti = 0; ti < tpc; ++ti) {
        const int t0 = (tc * tpc + ti) * 32;
        const u32x4 v = next;
        if (ti + 1 < tpc) next = load(ti + 1);
        if (ti) __syncthreads();                // the previous tile has been read
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            tile[8 * iq + 2 * k][ich] = (uint16_t)(v[k] & 0xFFFFu);
            tile[8 * iq + 2 * k + 1][ich] = (uint16_t)(v[k] >> 16);
        }
        __syncthreads();
        const u32x4 o = *reinterpret_cast<const u32x4*>(&tile[ptk][8 * pq]);
        if (ti == 0) {
            const u32x4 f = *reinterpret_cast<const u32x4*>(&tile[0][8 * pq]);
#pragma unroll
            for (int k = 0; k < 4; ++k) { k0[2 * k] = __uint_as_float(f[k] << 16); k0[2 * k + 1] = __uint_as_float(f[k] & 0xFFFF0000u); }
        }
        *reinterpret_cast<u32x4*>(x + ((int64_t)p * S + t0 + ptk) * C + c0 + 8 * pq) = o;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float lo = __uint_as_float(o[k] << 16) - k0[2 * k], hi = __uint_as_float(o[k] & 0xFFFF0000u) - k0[2 * k + 1];
            s1[2 * k] += lo; s2[2 * k] = fmaf(lo, lo, s2[2 * k]);
            s1[2 * k + 1] += hi; s2[2 * k + 1] = fmaf(hi, hi, s2[2 * k + 1]);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) { red[0][ptk][8 * pq + e] = s1[e]; red[1][ptk][8 * pq + e] = s2[e]; }
    if (ptk == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) kk[8 * pq + e] = k0[e];
    }
    __syncthreads();
    if (tid < 64) {
        float a = 0.f, b = 0.f;
        for (int l = 0; l < 32; ++l) { a += red[0][l][tid]; b += red[1][l][tid]; }      // fixed order
        const float nt = (float)(tpc * 32), inv = 1.f / nt;
        float* dst = stats + (((int64_t)p * nch + tc) * C + c0 + tid) * 2;
        dst[0] = kk[tid] + a * inv;
        dst[1] = fmaxf(b - a * a * inv, 0.f);
    }
}

// Text tokens of every request <-> the text patches of the joint token matrix.  One thread per (slot, text row
// incl. padding, 16-byte vector).  TO_PATCH: text [n][L][C] (caller order) -> x, padding rows zeroed; else x -> text.
template <bool TO_PATCH>
__global__ void text_rows_kernel(uint4* __restrict__ x, uint4* __restrict__ text, const int32_t* __restrict__ perm,
                                 const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ seq_len, int32_t n,
                                 int32_t L, int32_t rows_pad, int32_t CV) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n * rows_pad * CV) return;
    const int cv = (int)(i % CV);
    const int r = (int)((i / CV) % rows_pad);
    const int s = (int)(i / ((int64_t)CV * rows_pad));
    const int64_t xrow = (int64_t)cu_seqlens[s] + seq_len[s] - L + r;         // first text row sits behind the image tokens
    if (TO_PATCH) x[xrow * CV + cv] = r < L ? text[((int64_t)perm[s] * L + r) * CV + cv] : make_uint4(0, 0, 0, 0);
    else if (r < L) text[((int64_t)perm[s] * L + r) * CV + cv] = x[xrow * CV + cv];
}

template <bool TO_PATCH>
static int run_text(const pserve_plan_t* plan, void* x, void* text, int32_t C, int dtype, hipStream_t st) {
    PS_REQUIRE(plan && x && text, "text scatter/gather: NULL argument");
    PS_REQUIRE(plan->text_len > 0, "text scatter/gather: the plan has no text patches (pserve_plan_text)");
    PS_REQUIRE(dtype == PSERVE_F32 || dtype == PSERVE_BF16, "text scatter/gather: unknown dtype %d", dtype);
    const int vn = dtype == PSERVE_BF16 ? 8 : 4;
    PS_REQUIRE(C > 0 && C % vn == 0, "text scatter/gather: C=%d must be a multiple of 16 bytes", C);
    const int rows_pad = plan->text_patches * plan->S, CV = C / vn;
    const int64_t items = (int64_t)plan->n * rows_pad * CV;
    text_rows_kernel<TO_PATCH><<<(unsigned)cdiv(items, 256), 256, 0, st>>>((uint4*)x, (uint4*)text, plan->d_tab[PSERVE_TAB_PERM],
        plan->d_tab[PSERVE_TAB_CU_SEQLENS], plan->d_tab[PSERVE_TAB_SEQ_LEN], plan->n, plan->text_len, rows_pad, CV);
    return check_launch("text_rows_kernel");
}

template <bool TO_PATCH>
static int run_split(const pserve_plan_t* plan, void* const* images, int32_t C, int dtype, void* x, hipStream_t st) {
    PS_REQUIRE(plan && images && x, "split/reassemble: NULL argument");
    PS_REQUIRE(C > 0, "split/reassemble: C must be positive");
    PS_REQUIRE(dtype == PSERVE_F32 || dtype == PSERVE_BF16, "split/reassemble: unknown dtype %d", dtype);
    const auto& ro = plan->h_tab[PSERVE_TAB_REQUEST_OFFSET];
    const auto& perm = plan->h_tab[PSERVE_TAB_PERM];
    for (int i = 0; i < plan->n; ++i) PS_REQUIRE(images[i], "split/reassemble: image %d is NULL", i);
    for (int s0 = 0; s0 < plan->n; s0 += IMG_CHUNK) {
        const int s1 = std::min(plan->n, s0 + IMG_CHUNK);
        ImagePtrs ip;
        memset(&ip, 0, sizeof(ip));
        for (int s = s0; s < s1; ++s) ip.p[s - s0] = images[perm[s]];
        const int patch0 = ro[s0], npatch = ro[s1] - ro[s0];
        // pixels an access of split_plane_kernel takes: all planes start at a multiple of as many
        const int es = (int)dtype_size(dtype);
        int px = C % 64 == 0 && ((uintptr_t)x & 15) == 0 ? 16 / es : 0;
        PlaneTiles at{};
        for (int s = s0, end = 0; s < s1; ++s) {
            const int64_t N = (int64_t)plan->h_sorted_hw[2 * s] * plan->h_sorted_hw[2 * s + 1];
            while (px > 1 && (N % px != 0 || ((uintptr_t)ip.p[s - s0] & (px * es - 1)))) px /= 2;
            at.end[s - s0] = end += (int)cdiv(N, 128 / es);
        }
        if (px > 1) {
            const dim3 pgrid((unsigned)at.end[s1 - s0 - 1], (unsigned)(C / 64));
#define PS_PLANE(T_, V_) split_plane_kernel<T_, V_, TO_PATCH><<<pgrid, 256, 0, st>>>(ip, at, s0, plan->d_sorted_hw, \
                             plan->d_tab[PSERVE_TAB_REQUEST_OFFSET], plan->ph, plan->pw, C, (T_*)x)
            if (dtype == PSERVE_BF16) { if (px == 8) PS_PLANE(uint16_t, 8); else if (px == 4) PS_PLANE(uint16_t, 4); else PS_PLANE(uint16_t, 2); }
            else { if (px == 4) PS_PLANE(float, 4); else PS_PLANE(float, 2); }
#undef PS_PLANE
            PS_TRY(check_launch("split_plane_kernel"));
            continue;
        }
        dim3 grid(npatch * plan->ph, (unsigned)cdiv(C, 64));
        if (dtype == PSERVE_BF16)
            split_kernel<uint16_t, TO_PATCH><<<grid, 256, 0, st>>>(ip, s0, patch0, plan->d_sorted_hw,
                plan->d_tab[PSERVE_TAB_PATCH_OWNER], plan->d_tab[PSERVE_TAB_PATCH_RC], plan->ph, plan->pw, C, (uint16_t*)x);
        else
            split_kernel<float, TO_PATCH><<<grid, 256, 0, st>>>(ip, s0, patch0, plan->d_sorted_hw,
                plan->d_tab[PSERVE_TAB_PATCH_OWNER], plan->d_tab[PSERVE_TAB_PATCH_RC], plan->ph, plan->pw, C, (float*)x);
        PS_TRY(check_launch("split_kernel"));
    }
    return PSERVE_OK;
}


// pserve_split (bf16 fast path only) that also writes the per-channel moments of x; *done = false (and nothing is
// written) where the fast path does not apply
int split_with_stats(const pserve_plan_t* plan, const void* const* images, int32_t C, void* x, float* stats, int32_t nch,
                     hipStream_t st, bool* done) {
    *done = false;
    const auto& ro = plan->h_tab[PSERVE_TAB_REQUEST_OFFSET];
    const auto& perm = plan->h_tab[PSERVE_TAB_PERM];
    bool vec = plan->pw % 8 == 0 && plan->S % 32 == 0 && C % 64 == 0 && ((uintptr_t)x & 15) == 0 && nch >= 1 &&
               (plan->S / 32) % nch == 0 && plan->text_len == 0;
    for (int i = 0; i < plan->n && vec; ++i)
        vec = images[i] && plan->h_sorted_hw[2 * i + 1] % 8 == 0 && ((uintptr_t)images[i] & 15) == 0;
    if (!vec) return PSERVE_OK;
    for (int s0 = 0; s0 < plan->n; s0 += IMG_CHUNK) {
        const int s1 = std::min(plan->n, s0 + IMG_CHUNK);
        ImagePtrs ip;
        memset(&ip, 0, sizeof(ip));
        for (int s = s0; s < s1; ++s) ip.p[s - s0] = (void*)images[perm[s]];
        const int patch0 = ro[s0], npatch = ro[s1] - ro[s0];
        dim3 grid(npatch * nch, (unsigned)(C / 64));
        split_stats_kernel<<<grid, 256, 0, st>>>(ip, s0, patch0, plan->d_sorted_hw, plan->d_tab[PSERVE_TAB_PATCH_OWNER],
                                                 plan->d_tab[PSERVE_TAB_PATCH_RC], plan->ph, plan->pw, C, nch, (uint16_t*)x, stats);
        PS_TRY(check_launch("split_stats_kernel"));
    }
    *done = true;
    return PSERVE_OK;
}
}  // namespace pserve

using namespace pserve;

extern "C" {

const char* pserve_last_error(void) { return g_err; }

int pserve_plan(const int32_t* res, int32_t n, int32_t ph, int32_t pw, void* stream, pserve_plan_t** out) {
    return pserve_plan_text(res, n, ph, pw, 0, stream, out);
}

int pserve_text_scatter(const pserve_plan_t* plan, const void* text, int32_t C, int dtype, void* x, void* stream) {
    return run_text<true>(plan, x, const_cast<void*>(text), C, dtype, (hipStream_t)stream);
}

int pserve_text_gather(const pserve_plan_t* plan, const void* x, int32_t C, int dtype, void* text, void* stream) {
    return run_text<false>(plan, const_cast<void*>(x), text, C, dtype, (hipStream_t)stream);
}

static int plan_text_impl(const int32_t* res, int32_t n, int32_t ph, int32_t pw, int32_t text_len, void* stream,
                     pserve_plan_t** out) {
    PS_REQUIRE(out, "pserve_plan: out is NULL");
    PS_REQUIRE(text_len >= 0, "pserve_plan: negative text_len");
    *out = nullptr;
    PS_REQUIRE(res && n > 0, "pserve_plan: need n > 0 resolutions");
    PS_REQUIRE((ph == 0) == (pw == 0) && ph >= 0 && pw >= 0, "pserve_plan: patch must be (0,0) or both positive");
    for (int i = 0; i < n; ++i)
        PS_REQUIRE(res[2 * i] > 0 && res[2 * i + 1] > 0, "pserve_plan: request %d has a non-positive size", i);
    if (ph == 0) {                                            // patch-size rule: gcd per dimension
        for (int i = 0; i < n; ++i) { ph = std::gcd(ph, res[2 * i]); pw = std::gcd(pw, res[2 * i + 1]); }
    }
    int64_t P = 0, max_tok = 0;
    for (int i = 0; i < n; ++i) {
        PS_REQUIRE(res[2 * i] % ph == 0 && res[2 * i + 1] % pw == 0,
                   "pserve_plan: request %d (%dx%d) is not a multiple of the patch %dx%d", i, res[2 * i], res[2 * i + 1], ph, pw);
        P += (int64_t)(res[2 * i] / ph) * (res[2 * i + 1] / pw);
        max_tok = std::max<int64_t>(max_tok, (int64_t)res[2 * i] * res[2 * i + 1]);
    }
    const int32_t tp = (int32_t)cdiv(text_len, (int64_t)ph * pw);     // text patches per request
    P += (int64_t)n * tp;
    max_tok += (int64_t)tp * ph * pw;
    const int64_t T = P * ph * pw;
    const int32_t ring = 2 * (pw + 2) + 2 * ph;
    PS_REQUIRE(T < (int64_t)1 << 31 && P * ring < (int64_t)1 << 31, "pserve_plan: batch too large (%lld tokens)", (long long)T);

    pserve_plan_t* pl = new (std::nothrow) pserve_plan_t();
    if (!pl) { set_error("pserve_plan: out of host memory"); return PSERVE_ENOMEM; }
    struct Guard { pserve_plan_t* p; ~Guard() { delete p; } } guard{pl};

    // reorder requests by resolution: ascending (H, W), stable in arrival order
    std::vector<int32_t> perm(n);
    std::iota(perm.begin(), perm.end(), 0);
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) {
        if (res[2 * a] != res[2 * b]) return res[2 * a] < res[2 * b];
        return res[2 * a + 1] < res[2 * b + 1];
    });
    auto new_run = [&](int s) {               // sorted slot s is the first of its resolution
        return s == 0 || res[2 * perm[s]] != res[2 * perm[s - 1]] || res[2 * perm[s] + 1] != res[2 * perm[s - 1] + 1];
    };
    int R = 0;
    for (int s = 0; s < n; ++s) R += new_run(s);
    pl->n = n; pl->R = R; pl->P = (int32_t)P; pl->ph = ph; pl->pw = pw; pl->ring = ring; pl->T = T; pl->S = ph * pw;
    pl->max_tokens_per_image = (int32_t)max_tok;
    pl->text_len = text_len; pl->text_patches = tp;

    int64_t* cnt = pl->tab_count;
    cnt[PSERVE_TAB_PERM] = n;
    cnt[PSERVE_TAB_REQUEST_OFFSET] = n + 1;
    cnt[PSERVE_TAB_RES_OFFSET] = R + 1;
    cnt[PSERVE_TAB_RES_HW] = 2 * R;
    cnt[PSERVE_TAB_PATCH_OWNER] = P;
    cnt[PSERVE_TAB_PATCH_RC] = 2 * P;
    cnt[PSERVE_TAB_NEIGHBOUR] = 8 * P;
    cnt[PSERVE_TAB_HALO_SRC] = P * ring;
    cnt[PSERVE_TAB_CU_SEQLENS] = n + 1;
    cnt[PSERVE_TAB_SEQ_LEN] = n;
    // One allocation and one launch.  The per-request tables, a few numbers per request, are filled in on the host; one
    // kernel builds the per-patch tables.  Up to PLAN_STAGE_BYTES and PLAN_REQ requests (nearly every batch that is served)
    // the kernel itself moves both ways through pinned host memory: for 24 requests launch and wait take 14 us, with a copy
    // from and one to ordinary host memory around them 32 us.  Larger plans, where the tables' size decides, and any that
    // find no pinned memory are copied.  Every table starts on a 256-byte boundary.
    static const int order[PSERVE_TAB_COUNT] = {PSERVE_TAB_PERM, PSERVE_TAB_REQUEST_OFFSET, PSERVE_TAB_RES_OFFSET, PSERVE_TAB_RES_HW,
                                                PSERVE_TAB_CU_SEQLENS, PSERVE_TAB_SEQ_LEN, PSERVE_TAB_PATCH_OWNER,
                                                PSERVE_TAB_PATCH_RC, PSERVE_TAB_NEIGHBOUR, PSERVE_TAB_HALO_SRC};
    auto pad = [](int64_t v) { return (v + 63) / 64 * 64; };
    int64_t at[PSERVE_TAB_COUNT], total = pad(2 * n), per_request = 0;
    for (int t : order) {
        if (t == PSERVE_TAB_PATCH_OWNER) per_request = total;
        at[t] = total;
        total += pad(cnt[t]);
    }
    int32_t* dev = nullptr;
    PS_TRY(pl->pool.alloc_t(&dev, (size_t)(total + P * 16)));
    pl->h_arena.reset(new int32_t[(size_t)total]);
    int32_t* h[PSERVE_TAB_COUNT];
    for (int t : order) { h[t] = pl->h_arena.get() + at[t]; pl->h_tab[t] = h[t]; pl->d_tab[t] = dev + at[t]; }
    int32_t* hw = pl->h_arena.get();
    pl->h_sorted_hw = hw;
    pl->d_sorted_hw = dev;
    pl->mse_partial = reinterpret_cast<float*>(dev + total);
    int32_t run = 0, off = 0;
    for (int s = 0; s < n; ++s) {
        const int32_t H = res[2 * perm[s]], W = res[2 * perm[s] + 1];
        hw[2 * s] = H;
        hw[2 * s + 1] = W;
        h[PSERVE_TAB_PERM][s] = perm[s];
        h[PSERVE_TAB_REQUEST_OFFSET][s] = off;
        h[PSERVE_TAB_CU_SEQLENS][s] = off * ph * pw;
        h[PSERVE_TAB_SEQ_LEN][s] = H * W + text_len;          // valid tokens (padding of the last text patch excluded)
        if (new_run(s)) {
            h[PSERVE_TAB_RES_OFFSET][run] = s;
            h[PSERVE_TAB_RES_HW][2 * run] = H;
            h[PSERVE_TAB_RES_HW][2 * run + 1] = W;
            ++run;
        }
        off += (H / ph) * (W / pw) + tp;                      // tp text patches ride behind the image patches
    }
    h[PSERVE_TAB_REQUEST_OFFSET][n] = off;
    h[PSERVE_TAB_CU_SEQLENS][n] = off * ph * pw;
    h[PSERVE_TAB_RES_OFFSET][run] = n;

    const PlanLayout lay = {at[PSERVE_TAB_REQUEST_OFFSET], at[PSERVE_TAB_PATCH_OWNER], at[PSERVE_TAB_PATCH_RC],
                            at[PSERVE_TAB_NEIGHBOUR], at[PSERVE_TAB_HALO_SRC], total};
    hipStream_t st = (hipStream_t)stream;
    PlanStage ps;
    if (n <= PLAN_REQ && total * sizeof(int32_t) <= PLAN_STAGE_BYTES) ps.get();
    if (int32_t* stage = ps.p) {
        memcpy(stage, hw, sizeof(int32_t) * per_request);
        plan_patches_kernel<true><<<(unsigned)cdiv(total, 256), 256, 0, st>>>(dev, stage, lay, n, (int32_t)P, ph, pw, ring);
        PS_TRY(check_launch("plan_patches_kernel"));
        PS_CHECK_HIP(hipStreamSynchronize(st));
        ps.done = true;
        memcpy(hw + per_request, stage + per_request, sizeof(int32_t) * (total - per_request));
    } else {
        PS_CHECK_HIP(hipMemcpyAsync(dev, hw, sizeof(int32_t) * per_request, hipMemcpyHostToDevice, st));
        const unsigned blocks = (unsigned)std::min<int64_t>(cdiv(total - per_request, 256), 1 << 22);
        plan_patches_kernel<false><<<blocks, 256, 0, st>>>(dev, nullptr, lay, n, (int32_t)P, ph, pw, ring);
        PS_TRY(check_launch("plan_patches_kernel"));
        PS_CHECK_HIP(hipMemcpyAsync(hw + per_request, dev + per_request, sizeof(int32_t) * (total - per_request),
                                    hipMemcpyDeviceToHost, st));
        PS_CHECK_HIP(hipStreamSynchronize(st));
    }
    guard.p = nullptr;
    *out = pl;
    plans_changed(1);
    return PSERVE_OK;
}

int pserve_plan_text(const int32_t* res, int32_t n, int32_t ph, int32_t pw, int32_t text_len, void* stream,
                     pserve_plan_t** out) {
    return guarded("pserve_plan_text", [&] { return plan_text_impl(res, n, ph, pw, text_len, stream, out); });
}

void pserve_plan_free(pserve_plan_t* plan) {
    if (!plan) return;
    delete plan;
    plans_changed(-1);
}

int pserve_plan_info(const pserve_plan_t* plan, pserve_plan_info_t* out) {
    PS_REQUIRE(plan && out, "pserve_plan_info: NULL argument");
    out->n = plan->n; out->R = plan->R; out->P = plan->P; out->ph = plan->ph; out->pw = plan->pw;
    out->ring = plan->ring; out->T = plan->T;
    out->text_len = plan->text_len; out->text_patches = plan->text_patches;
    return PSERVE_OK;
}

int pserve_plan_table(const pserve_plan_t* plan, int which, int on_device, const int32_t** ptr, int64_t* count) {
    PS_REQUIRE(plan && ptr && count, "pserve_plan_table: NULL argument");
    PS_REQUIRE(which >= 0 && which < PSERVE_TAB_COUNT, "pserve_plan_table: unknown table %d", which);
    *ptr = on_device ? plan->d_tab[which] : plan->h_tab[which];
    *count = plan->tab_count[which];
    return PSERVE_OK;
}

int pserve_split(const pserve_plan_t* plan, const void* const* images, int32_t C, int dtype, void* x, void* stream) {
    return run_split<true>(plan, (void* const*)images, C, dtype, x, (hipStream_t)stream);
}

int pserve_reassemble(const pserve_plan_t* plan, const void* y, int32_t C, int dtype, void* const* images, void* stream) {
    return run_split<false>(plan, images, C, dtype, (void*)y, (hipStream_t)stream);
}

}  // extern "C"
