// decoder.hip -- what lies between the weight products of a decode pass
// (splice_decoder.h).  The rows of a pass are few and short, so a launch costs
// more than its bytes: each kernel here takes the place of a chain of
// elementwise operations over the same rows, rounding exactly where the chain
// rounds (floating-point contraction is off).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decoder_head.hpp"
#include "splice_decoder.h"

#pragma clang fp contract(off)

namespace {

using namespace splice_dev;

typedef __bf16 bf16x8v_t __attribute__((ext_vector_type(8)));
typedef float f32x8v_t __attribute__((ext_vector_type(8)));

constexpr int kDecThreads = 256;

__device__ __forceinline__ f32x8v_t load_f32x8(const float *p) { return *reinterpret_cast<const f32x8v_t *>(p); }
__device__ __forceinline__ f32x8v_t load_bf16x8(const __bf16 *p) {
    return __builtin_convertvector(*reinterpret_cast<const bf16x8v_t *>(p), f32x8v_t);
}
__device__ __forceinline__ void store_bf16x8(__bf16 *p, f32x8v_t v) {
    *reinterpret_cast<bf16x8v_t *>(p) = __builtin_convertvector(v, bf16x8v_t);
}

__global__ __launch_bounds__(kDecThreads) void residual_kernel(float *x, const __bf16 *delta, float *sq, int64_t units,
                                                               int assign) {
    const int64_t u = (int64_t)blockIdx.x * kDecThreads + threadIdx.x;
    if (u >= units) return;
    f32x8v_t v = load_bf16x8(delta + 8 * u);
    if (!assign) v = load_f32x8(x + 8 * u) + v;
    *reinterpret_cast<f32x8v_t *>(x + 8 * u) = v;
    *reinterpret_cast<f32x8v_t *>(sq + 8 * u) = v * v;
}

// Where value c of a normed row goes: packed is the head's tile order
// [d / 32][ceil(rows / 16)][16][32].
__device__ __forceinline__ int64_t norm_at(int row, int c, int rows, int d, int packed) {
    return packed ? ((int64_t)(c >> 5) * ((rows + 15) / 16) + (row >> 4)) * 512 + (row & 15) * 32 + (c & 31)
                  : (int64_t)row * d + c;
}

__global__ __launch_bounds__(kDecThreads) void norm_kernel(const float *x, const float *mean_sq, const __bf16 *gain,
                                                           __bf16 *h, int rows, int d, float eps, int packed) {
    const int per = d / 8;
    const int64_t u = (int64_t)blockIdx.x * kDecThreads + threadIdx.x;
    if (u >= (int64_t)rows * per) return;
    const int row = (int)(u / per), c = 8 * (int)(u % per);
    const float r = (float)(1.0 / sqrt((double)(mean_sq[row] + eps)));   // correctly rounded, as the operation's
    store_bf16x8(h + norm_at(row, c, rows, d, packed), load_f32x8(x + 8 * u) * r * load_bf16x8(gain + c));
}

// residual_kernel, the mean of the squares and norm_kernel in one launch, a
// work group per row: launches and one round of loads bound the three.  The
// squares are added as the mean operation adds a row of this length: 64 lanes,
// each four interleaved sums over units of four values, the four in order, then
// neighbouring lanes; times 1 / d.  At 8 rows of 2560 values 4.2 us a
// norm, before 13.0 (4.0 + 5.8 + 3.2); at 128 of 4096 5.2, before 17.8.
__global__ __launch_bounds__(kDecThreads) void add_norm_kernel(float *x, const __bf16 *delta, const __bf16 *gain,
                                                               __bf16 *h, __bf16 *hp, int rows, int d, float inv_d,
                                                               float eps, int assign) {
    constexpr int U = SPLICE_ADD_NORM_MAX_D / (8 * kDecThreads);   // units of eight values a thread
    __shared__ f32x4_t s_sq[SPLICE_ADD_NORM_MAX_D / 4];
    __shared__ float s_mean;
    const int row = blockIdx.x, tid = threadIdx.x, n = d / 8;
    float *xr = x + (size_t)row * d;
    const __bf16 *dr = delta + (size_t)row * d;
    f32x8v_t v[U], g[U];
    static_for<0, U>([&](auto i) {
        const int u = tid + (int)i * kDecThreads;
        if (u < n) {
            v[i] = load_bf16x8(dr + 8 * u);
            if (!assign) v[i] = load_f32x8(xr + 8 * u) + v[i];
            g[i] = load_bf16x8(gain + 8 * u);
        }
    });
    static_for<0, U>([&](auto i) {
        const int u = tid + (int)i * kDecThreads;
        if (u < n) {
            const f32x8v_t sq = v[i] * v[i];
            s_sq[2 * u] = f32x4_t{sq[0], sq[1], sq[2], sq[3]};
            s_sq[2 * u + 1] = f32x4_t{sq[4], sq[5], sq[6], sq[7]};
            *reinterpret_cast<f32x8v_t *>(xr + 8 * u) = v[i];
        }
    });
    __syncthreads();
    if (tid < 64) {
        f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int e = tid; e < 2 * n; e += 64) a += s_sq[e];
        float t = ((a.x + a.y) + a.z) + a.w;
        for (int o = 1; o < 64; o <<= 1) t += __shfl_xor(t, o);
        if (tid == 0) s_mean = t * inv_d;
    }
    __syncthreads();
    const float r = (float)(1.0 / sqrt((double)(s_mean + eps)));   // correctly rounded, as the operation's
    static_for<0, U>([&](auto i) {
        const int u = tid + (int)i * kDecThreads;
        if (u < n) {
            const f32x8v_t y = v[i] * r * g[i];
            if (h) store_bf16x8(h + norm_at(row, 8 * u, rows, d, 0), y);
            if (hp) store_bf16x8(hp + norm_at(row, 8 * u, rows, d, 1), y);
        }
    });
}

struct RopeSteps {
    int32_t step[SPLICE_MAX_CELLS];
};
__global__ __launch_bounds__(kDecThreads) void rope_table_kernel(float2 *tab, const double *pos, RopeSteps st,
                                                                 int prompt_len, int rows, int half, double theta) {
    const int e = blockIdx.x * kDecThreads + threadIdx.x;
    if (e >= rows * half) return;
    const int row = e / half, i = e % half;
    const double p = pos ? pos[row] : (double)(prompt_len + max(st.step[row], 0));
    const float ang = (float)(p * pow(theta, -(double)i * 2.0 / (double)(2 * half)));
    tab[e] = make_float2(cosf(ang), sinf(ang));
}

// A unit is four pairs (i, i + D / 2) of one (row, head).
__global__ __launch_bounds__(kDecThreads) void rope_kernel(__bf16 *q, __bf16 *k, const float2 *tab, int rows, int Hq,
                                                           int Hkv, int D) {
    const int half = D / 2, per = half / 4, heads = Hq + Hkv;
    const int u = blockIdx.x * kDecThreads + threadIdx.x;
    if (u >= rows * heads * per) return;
    const int i = 4 * (u % per), item = u / per, row = item / heads, hd = item % heads;
    __bf16 *p = (hd < Hq ? q + ((size_t)row * Hq + hd) * D : k + ((size_t)row * Hkv + hd - Hq) * D) + i;
    const f32x4_t x1 = __builtin_convertvector(*reinterpret_cast<const bf16x4_t *>(p), f32x4_t);
    const f32x4_t x2 = __builtin_convertvector(*reinterpret_cast<const bf16x4_t *>(p + half), f32x4_t);
    f32x4_t y1, y2;
    static_for<0, 4>([&](auto j) {
        const float2 cs = tab[row * half + i + (int)j];
        const float a = x1[(int)j], b = x2[(int)j];
        y1[(int)j] = a * cs.x - b * cs.y;
        y2[(int)j] = b * cs.x + a * cs.y;
    });
    *reinterpret_cast<bf16x4_t *>(p) = __builtin_convertvector(y1, bf16x4_t);
    *reinterpret_cast<bf16x4_t *>(p + half) = __builtin_convertvector(y2, bf16x4_t);
}

// Where unit u (eight values) of [rows][d] goes.
__device__ __forceinline__ int64_t unit_at(int64_t u, int rows, int d, int packed) {
    return packed ? norm_at((int)(u / (d / 8)), 8 * (int)(u % (d / 8)), rows, d, 1) : 8 * u;
}

__global__ __launch_bounds__(kDecThreads) void round_kernel(const float *src, __bf16 *dst, int64_t units, int rows, int d,
                                                            int packed) {
    const int64_t u = (int64_t)blockIdx.x * kDecThreads + threadIdx.x;
    if (u < units) store_bf16x8(dst + unit_at(u, rows, d, packed), load_f32x8(src + 8 * u));
}

__global__ __launch_bounds__(kDecThreads) void silu_kernel(const __bf16 *gate, const __bf16 *up, __bf16 *act,
                                                           int64_t units, int rows, int d, int packed) {
    const int64_t u = (int64_t)blockIdx.x * kDecThreads + threadIdx.x;
    if (u >= units) return;
    const f32x8v_t g = load_bf16x8(gate + 8 * u), w = load_bf16x8(up + 8 * u);
    f32x8v_t o;
    static_for<0, 8>([&](auto i) {
        const float x = g[(int)i];
        o[(int)i] = (float)(__bf16)(x / (1.f + expf(-x))) * w[(int)i];
    });
    store_bf16x8(act + unit_at(u, rows, d, packed), o);
}

// ---------------------------------------------------------------- argmax

// Orders floats as unsigned words, NaN above everything, -0 as 0; the low word
// makes the lower index the larger key.
__device__ __forceinline__ uint64_t max_key(float x, int i) {
    uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
    u = x != x ? 0xffffffffu : ((u >> 31) ? ~u : u | 0x80000000u);
    return ((uint64_t)u << 32) | (uint32_t)~i;
}

__device__ __forceinline__ uint64_t block_max(uint64_t k) {
    __shared__ uint64_t s_k[kDecThreads / 64];
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t y = __shfl_xor((unsigned long long)k, o);
        k = y > k ? y : k;
    }
    if ((threadIdx.x & 63) == 0) s_k[threadIdx.x >> 6] = k;
    __syncthreads();
    for (int w = 0; w < kDecThreads / 64; ++w) k = s_k[w] > k ? s_k[w] : k;
    return k;
}

__global__ __launch_bounds__(kDecThreads) void argmax_part_kernel(const float *logits, int vocab, uint64_t *keys) {
    const int row = blockIdx.y, parts = gridDim.x;
    const int per = (vocab + parts - 1) / parts, b = blockIdx.x * per, e = min(b + per, vocab);
    const float *r = logits + (size_t)row * vocab;
    uint64_t k = 0;
    for (int i = b + threadIdx.x; i < e; i += 4 * kDecThreads) {
        float x[4];
        static_for<0, 4>([&](auto j) { x[(int)j] = r[min(i + (int)j * kDecThreads, e - 1)]; });
        static_for<0, 4>([&](auto j) {
            const uint64_t y = max_key(x[(int)j], min(i + (int)j * kDecThreads, e - 1));
            k = y > k ? y : k;
        });
    }
    k = block_max(k);
    if (threadIdx.x == 0) keys[(size_t)row * parts + blockIdx.x] = k;
}

__global__ __launch_bounds__(kDecThreads) void argmax_kernel(const uint64_t *keys, int parts, int64_t *tokens) {
    const uint64_t k = block_max((int)threadIdx.x < parts ? keys[(size_t)blockIdx.x * parts + threadIdx.x] : 0);
    if (threadIdx.x == 0) tokens[blockIdx.x] = (int64_t)(uint32_t)~(uint32_t)k;
}

// ---------------------------------------------------------------- host side

unsigned blocks_of(int64_t units) { return (unsigned)((units + kDecThreads - 1) / kDecThreads); }

constexpr int64_t kMostValues = (int64_t)1 << 38;   // the grid of eight values a thread stays below 2^31 blocks

bool good(std::initializer_list<const void *> ptrs) {
    for (const void *p : ptrs)
        if (!p || !splice::aligned(p, 16)) return false;
    return true;
}

// [rows][d] as units of eight values, packed in steps of 32.
bool good_rows(int32_t rows, int32_t d, int32_t packed) {
    return rows >= 1 && d >= 8 && d % 8 == 0 && !(packed && d % 32) && (int64_t)rows * d <= kMostValues;
}

// How the columns of a head are spread: `n_full` whole tiles, the rest split
// over K.  Tiles run in rounds of as many work groups as the GPU holds; a last
// round that is at most half full takes as long as a full one, so its tiles
// are cut over K until they fill it.
struct HeadPlan {
    int n_full, split, rest;   // rest: columns that are split
};

int compute_units() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

HeadPlan head_plan(int tiles, int cols, int resident, int M, int K, int N) {
    HeadPlan p{tiles, 1, 0};
    if (resident < 1 || tiles <= resident || M > 128) return p;
    const int last = tiles % resident;
    int split = last > 0 ? resident / last : 1;
    if (split > K / 512) split = K / 512;   // at least 16 steps each
    if (split > 8) split = 8;
    if (split < 2) return p;
    p.n_full = tiles - last;
    p.split = split;
    p.rest = N - p.n_full * cols;
    return p;
}

// Up to 16 rows X is a small part of what a work group reads: 128 columns and
// two work groups a compute unit (8 rows, 151936 columns: 214 us against 220 of
// 256 columns and one); above, 256 columns (32 rows, 131072 columns: 165 us
// against 186).
constexpr int kHeadNarrowRows = 16;
constexpr int kHeadWide = 256;

template <int MB, int NS, int NB, int WN, int WM>
void launch_head(HeadArgs a, const HeadPlan &p, float *part, hipStream_t stream) {
    using X = Head<MB, NS, NB, WN, WM>;
    a.n_full = p.n_full;
    a.split = p.split;
    a.part = part;
    const int tiles = (a.N + X::COLS - 1) / X::COLS;
    const dim3 grid((unsigned)(p.n_full + (tiles - p.n_full) * p.split), (unsigned)((a.M + 16 * MB - 1) / (16 * MB)));
    hipLaunchKernelGGL((head_kernel<MB, NS, NB, WN, WM, 1, false>), grid, dim3(64 * WN * WM), 0, stream, a);
    if (p.rest > 0)
        hipLaunchKernelGGL(head_sum_kernel, dim3((unsigned)(((int64_t)a.M * p.rest / 4 + 255) / 256)), dim3(256), 0, stream,
                           part, a.y, a.M, a.N, a.N - p.rest, p.split);
}

HeadPlan plan_of(int rows, int d, int vocab) {
    if (rows <= kHeadNarrowRows) return HeadPlan{(vocab + 127) / 128, 1, 0};
    return head_plan((vocab + kHeadWide - 1) / kHeadWide, kHeadWide, compute_units(), rows, d, vocab);
}

int32_t launched() { return hipGetLastError() == hipSuccess ? SPLICE_OK : SPLICE_EHIP; }

}  // namespace

extern "C" {

int32_t splice_decoder_residual(float *x, const void *delta, float *sq, int64_t n, int32_t assign, void *stream) {
    if (!good({x, delta, sq})) return SPLICE_EINVAL;
    if (n < 8 || n % 8 || n > kMostValues) return SPLICE_EUNSUPPORTED;
    hipLaunchKernelGGL(residual_kernel, dim3(blocks_of(n / 8)), dim3(kDecThreads), 0, (hipStream_t)stream, x,
                       (const __bf16 *)delta, sq, n / 8, assign);
    return launched();
}

int32_t splice_decoder_norm(const float *x, const float *mean_sq, const void *gain, void *h, int32_t rows, int32_t d,
                            float eps, int32_t packed, void *stream) {
    if (!good({x, gain, h}) || !mean_sq || !splice::aligned(mean_sq, 4)) return SPLICE_EINVAL;
    if (!good_rows(rows, d, packed)) return SPLICE_EUNSUPPORTED;
    hipLaunchKernelGGL(norm_kernel, dim3(blocks_of((int64_t)rows * (d / 8))), dim3(kDecThreads), 0, (hipStream_t)stream,
                       x, mean_sq, (const __bf16 *)gain, (__bf16 *)h, rows, d, eps, packed);
    return launched();
}

int32_t splice_decoder_add_norm(float *x, const void *delta, const void *gain, void *h, void *h_packed, int32_t rows,
                                int32_t d, float eps, int32_t assign, void *stream) {
    if (!good({x, delta, gain, h ? h : h_packed, h_packed ? h_packed : h})) return SPLICE_EINVAL;
    if (rows < 1 || d < 8 || d % 8 || d > SPLICE_ADD_NORM_MAX_D || (h_packed && d % 32)) return SPLICE_EUNSUPPORTED;
    hipLaunchKernelGGL(add_norm_kernel, dim3((unsigned)rows), dim3(kDecThreads), 0, (hipStream_t)stream, x,
                       (const __bf16 *)delta, (const __bf16 *)gain, (__bf16 *)h, (__bf16 *)h_packed, rows, d,
                       (float)(1.0 / d), eps, assign);
    return launched();
}

int32_t splice_decoder_rope_table(float *tab, const double *pos, const int32_t *cell_step, int32_t rows,
                                  int32_t head_dim, int32_t prompt_len, double theta, void *stream) {
    if (!good({tab}) || (!pos && !cell_step) || (pos && !splice::aligned(pos, 8))) return SPLICE_EINVAL;
    if (rows < 1 || rows > SPLICE_MAX_CELLS || head_dim < 2 || head_dim % 2 || head_dim > 1024)
        return SPLICE_EUNSUPPORTED;
    RopeSteps st;
    for (int c = 0; c < SPLICE_MAX_CELLS; ++c) st.step[c] = !pos && c < rows ? cell_step[c] : 0;
    hipLaunchKernelGGL(rope_table_kernel, dim3(blocks_of((int64_t)rows * (head_dim / 2))), dim3(kDecThreads), 0,
                       (hipStream_t)stream, (float2 *)tab, pos, st, prompt_len, rows, head_dim / 2, theta);
    return launched();
}

int32_t splice_decoder_rope(void *q, void *k, const float *tab, int32_t rows, int32_t n_q, int32_t n_kv,
                            int32_t head_dim, void *stream) {
    if (!good({q, k, tab})) return SPLICE_EINVAL;
    if (rows < 1 || n_q < 1 || n_kv < 1 || head_dim < 8 || head_dim % 8 ||
        (int64_t)rows * ((int64_t)n_q + n_kv) * head_dim > INT32_MAX)
        return SPLICE_EUNSUPPORTED;
    hipLaunchKernelGGL(rope_kernel, dim3(blocks_of((int64_t)rows * (n_q + n_kv) * (head_dim / 8))), dim3(kDecThreads), 0,
                       (hipStream_t)stream, (__bf16 *)q, (__bf16 *)k, (const float2 *)tab, rows, n_q, n_kv, head_dim);
    return launched();
}

int32_t splice_decoder_round(const float *src, void *dst, int32_t rows, int32_t d, int32_t packed, void *stream) {
    if (!good({src, dst})) return SPLICE_EINVAL;
    if (!good_rows(rows, d, packed)) return SPLICE_EUNSUPPORTED;
    const int64_t units = (int64_t)rows * (d / 8);
    hipLaunchKernelGGL(round_kernel, dim3(blocks_of(units)), dim3(kDecThreads), 0, (hipStream_t)stream, src, (__bf16 *)dst,
                       units, rows, d, packed);
    return launched();
}

int32_t splice_decoder_silu(const void *gate, const void *up, void *act, int32_t rows, int32_t d, int32_t packed,
                            void *stream) {
    if (!good({gate, up, act}) || (packed && (act == gate || act == up))) return SPLICE_EINVAL;
    if (!good_rows(rows, d, packed)) return SPLICE_EUNSUPPORTED;
    const int64_t units = (int64_t)rows * (d / 8);
    hipLaunchKernelGGL(silu_kernel, dim3(blocks_of(units)), dim3(kDecThreads), 0, (hipStream_t)stream,
                       (const __bf16 *)gate, (const __bf16 *)up, (__bf16 *)act, units, rows, d, packed);
    return launched();
}

// A layer's product in one round of small tiles. Each work group sums all of K
// in order, as the library's kernels for 64 and 128 rows do (the same bits: no
// split over K), so a product takes the time of one chain over K. The library
// takes 64 or 128 rows at once there and leaves most compute units idle; tiles
// of 32 rows and 64 columns fill the GPU (us, library against this, 128 rows:
// K = 4096, 4096 columns 39.2 / 22.6, 2560 columns 40.9 / 23.2, K = 12288, 4096
// columns 106.5 / 59.5; a barrier every 32 of K instead of every 128: 27.2,
// 26.5, 70.0).  The rule names 64 and 128 rows because at just these the
// library takes slower kernels than beside them (K = 12288, 4096 columns,
// library / this: 63 rows 42 / 56 and other bits, 64 rows 65 / 57, 65 rows
// 50 / 57, 127 rows 49 / 57, 128 rows 82 / 58).  More than one round of tiles
// loses (K = 4096, 12288 columns: 42.6 / 68.4).  Where the library splits K the
// sums differ and its time is as good: 2048 columns at 128 rows (K = 8192:
// 34 / 39), and every width from K = 17920 on (K = 18944, 64 rows, 3072
// columns: 74 / 86).  Up to K = 16384 and at the other widths the bits were the
// same at all of 1500 random sizes.
using Product = Head<2, 1, 5, 4, 1, 4, true>;
constexpr int kProductCols = 2048;     // fewer: left to the library
constexpr int kProductMaxK = 16384;

int32_t splice_decoder_product_takes(int32_t rows, int32_t k, int32_t n) {
    return (rows == 64 || rows == 128) && k >= 128 && k % 128 == 0 && k <= kProductMaxK && n >= kProductCols &&
           !(rows == 128 && n == kProductCols) && n % 8 == 0 &&
           (int64_t)(rows / 32) * ((n + Product::COLS - 1) / Product::COLS) <= compute_units();
}

int32_t splice_decoder_product(const void *x, const void *w, void *y, int32_t rows, int32_t k, int32_t n, void *stream) {
    if (!good({x, w, y})) return SPLICE_EINVAL;
    if (rows < 1 || rows > SPLICE_MAX_CELLS || k < 128 || k % 128 || k > 1 << 20 || n < 8 || n % 8 || n > 1 << 24)
        return SPLICE_EUNSUPPORTED;
    const int tiles = (n + Product::COLS - 1) / Product::COLS;
    const HeadArgs a{(const char *)x, (const char *)w, (float *)y, rows, k, n, tiles, 1, nullptr};
    hipLaunchKernelGGL((head_kernel<2, 1, 5, 4, 1, 4, true>), dim3((unsigned)tiles, (unsigned)((rows + 31) / 32)), dim3(256),
                       0, (hipStream_t)stream, a);
    return launched();
}

// The own head where it is the faster one (us, the library's product with its
// conversion / this, some 25 of the former the host's): columns for three
// quarters of the compute units (K = 4096, 128 rows: 49152 columns 96 / 81, but
// 32000 62 / 73, 16384 43 / 69) and at most 128 rows, more read the weights again
// (K = 4096, 151936 columns, 128 rows 313 / 240, 129 rows 333 / 444); with fewer
// columns a work group's chain over K is what it takes, so K short for the rows
// (16384 columns: 16 rows K = 4096 30 / 29, 5120 33 / 36; 64 rows K = 2048 28 / 29,
// 2560 28 / 35; 128 rows K = 1024 27 / 23, 2048 29 / 39).
int32_t splice_decoder_head_takes(int32_t rows, int32_t d, int32_t vocab) {
    if (rows < 1 || rows > SPLICE_MAX_CELLS || d < 32 || d % 32 || d > 1 << 20 || vocab < 8 || vocab % 8 || vocab > 1 << 24)
        return 0;
    const int tiles = rows <= kHeadNarrowRows ? (vocab + 127) / 128 : (vocab + kHeadWide - 1) / kHeadWide;
    if (4 * tiles >= 3 * compute_units()) return rows <= 128;
    return d <= (rows <= kHeadNarrowRows ? 4096 : (rows <= 64 ? 2048 : 1024));
}

int64_t splice_decoder_head_bytes(int32_t rows, int32_t d, int32_t vocab) {
    if (rows < 1 || rows > SPLICE_MAX_CELLS || d < 32 || d % 32 || d > 1 << 20 || vocab < 8 || vocab % 8 ||
        vocab > 1 << 24)
        return SPLICE_EUNSUPPORTED;
    const HeadPlan p = plan_of(rows, d, vocab);
    return p.rest > 0 ? (int64_t)p.split * rows * p.rest * 4 : 0;
}

int32_t splice_decoder_head(const void *h, const void *w, float *logits, int32_t rows, int32_t d, int32_t vocab,
                            void *scratch, size_t scratch_bytes, void *stream) {
    const int64_t need = splice_decoder_head_bytes(rows, d, vocab);
    if (need < 0) return (int32_t)need;
    if (!good({h, w, logits})) return SPLICE_EINVAL;
    if (need > 0 && (!scratch || !splice::aligned(scratch, 16) || scratch_bytes < (size_t)need)) return SPLICE_EWORKSPACE;
    const HeadPlan p = plan_of(rows, d, vocab);
    const HeadArgs a{(const char *)h, (const char *)w, logits, rows, d, vocab, 0, 1, nullptr};
    hipStream_t st = (hipStream_t)stream;
    float *part = (float *)scratch;
    // as many row blocks as there are rows, at most 128 rows a work group (then
    // the weights are read again)
    if (rows <= 16) launch_head<1, 2, 8, 4, 1>(a, p, part, st);
    else if (rows <= 32) launch_head<2, 4, 8, 8, 1>(a, p, part, st);
    else if (rows <= 64) launch_head<4, 4, 7, 4, 2>(a, p, part, st);
    else launch_head<8, 4, 6, 4, 2>(a, p, part, st);
    return launched();
}

int32_t splice_decoder_argmax(const float *logits, int32_t rows, int32_t vocab, int64_t *tokens, void *scratch,
                              void *stream) {
    if (!logits || !tokens || !scratch || !splice::aligned(logits, 4) || !splice::aligned(tokens, 8) ||
        !splice::aligned(scratch, 8))
        return SPLICE_EINVAL;
    if (rows < 1 || rows > 65535 || vocab < 1 || vocab > 1 << 24) return SPLICE_EUNSUPPORTED;
    // about eight work groups a compute unit, each with a thousand values or more
    int parts = (2048 + rows - 1) / rows;
    const int most = (vocab + 1023) / 1024;
    parts = parts < most ? parts : most;
    parts = parts < SPLICE_ARGMAX_PARTS ? parts : SPLICE_ARGMAX_PARTS;
    hipLaunchKernelGGL(argmax_part_kernel, dim3((unsigned)parts, (unsigned)rows), dim3(kDecThreads), 0,
                       (hipStream_t)stream, logits, vocab, (uint64_t *)scratch);
    hipLaunchKernelGGL(argmax_kernel, dim3((unsigned)rows), dim3(kDecThreads), 0, (hipStream_t)stream,
                       (const uint64_t *)scratch, parts, tokens);
    return launched();
}

}  // extern "C"
