// decoder_head.hpp -- rows times a large bf16 weight matrix, the weights
// streamed once: Y[M][N] = X[M][K] W[K][N], for the few rows (one per sweep
// cell) of a decode pass and the many columns of a language-model head.
//
// Bound by reading W.  A work group owns 64 NS output columns and up to 16 MB
// rows and walks K in steps of 32: the step's W rows (4 NS KB) and X columns
// (MB KB) go from memory straight into an LDS ring, so what is in flight holds
// no registers.  Per step a wave computes Y^T += W^T X^T on
// v_mfma_f32_16x16x32_bf16: the W^T operand (16 columns x 32 k) comes out of
// the row-major tile through transposing LDS reads, the X operand is 16
// contiguous bytes a lane.
//
// What mattered (K = 4096, 151936 columns, 128 rows unless named; the library
// product with its conversion to fp32 takes 305 us, 246 at 8 rows):
//   * X in the order it is read ([K / 32][rows / 16][16][32]): rows 8 KB apart
//     fall on one L2 channel, 319 us against 274;
//   * W non-temporal (it is read once): 8 rows 211 -> 187 us (6.7 TB/s), 128
//     rows 267 -> 256; X, which every work group reads, stays cached (the same
//     hint on both: 313 us);
//   * 256 columns a work group, alone on its compute unit, halve the reads of
//     X: 131072 columns 239 -> 202 us, at 32 rows 201 -> 180;
//   * the columns of a last round that is less than half full split over K:
//     267 -> 256 us, at 32 rows 222 -> 208.
#pragma once

#include "prompt_wide.hpp"

namespace splice_dev {

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));

struct HeadArgs {
    const char *x;   // [K / 32][ceil(M / 16)][16][32] bf16: a step's rows are contiguous
    const char *w;   // [K][N] bf16
    float *y;        // [M][N] (bf16 if OUT16)
    int M, K, N;
    // the column tiles from n_full on are split over K: `split` work groups
    // each write a partial [split][M][N - n_full COLS] that head_sum_kernel adds
    int n_full, split;
    float *part;
};

// MB: 16-row blocks of a work group; NS: blocks of 64 columns; NB: ring
// buffers; WN x WM: waves over the columns and over the rows; KS: steps of 32
// between two barriers (K a multiple of 32 KS); OUT16: Y is bf16.
template <int MB, int NS, int NB, int WN, int WM, int KS = 1, bool OUT16 = false>
struct Head {
    static constexpr int BK = 32;
    static constexpr int COLS = 64 * NS;
    static constexpr int NW = WN * WM;
    static constexpr int SUB = BK * 128;                 // one block of 64 columns
    static constexpr int STEP = NS * SUB + MB * 1024;
    static constexpr int STAGE = KS * STEP;
    static constexpr int LDS = NB * STAGE;
    static constexpr int RB = MB / WM;                    // row blocks per wave
    static constexpr int T = 4 * NS / WN;                 // 16-column tiles per wave
    static constexpr int WI = 4 * NS / NW;                // W load instructions per wave and step
    static constexpr int XI = (MB + NW - 1) / NW;         // X load instructions (waves below MB)
    static_assert(MB % WM == 0 && 4 * NS % WN == 0 && 4 * NS % NW == 0, "whole tiles and loads per wave");
};

// Chunk-slot swizzles of the tiles (XOR on the 16-byte chunk of a row), so
// that one operand read touches every bank once.  W rows are 128 bytes (two
// share a bank line) and a half-wave of transposing reads names rows
// 4 h .. + 3 and 8 + 4 h .. + 3, two adjacent chunks each; X rows are 64
// bytes and 16 lanes read one chunk of 16 rows.
__device__ __forceinline__ int swz_w(int r) { return (((r >> 1) & 1) | (((r >> 3) & 1) << 1)) << 1; }
__device__ __forceinline__ int swz_x(int r) { return (r >> 2) & 3; }

template <int MB, int NS, int NB, int WN, int WM, int KS, bool OUT16>
__global__ __launch_bounds__(64 * WN * WM) void head_kernel(HeadArgs a) {
    using X = Head<MB, NS, NB, WN, WM, KS, OUT16>;
    constexpr int NW = X::NW, WI = X::WI, XI = X::XI, T = X::T, RB = X::RB;
    __shared__ __attribute__((aligned(16))) char lds[X::LDS];
    const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rest = (int)blockIdx.x - a.n_full;
    const bool whole = rest < 0;
    const int sp = whole ? 0 : rest % a.split;
    const int n0 = (whole ? (int)blockIdx.x : a.n_full + rest / a.split) * X::COLS;
    const int m0 = blockIdx.y * 16 * MB, rows = min(a.M - m0, 16 * MB);
    const int all = a.K / (X::BK * KS);
    const int s0 = whole ? 0 : all * sp / a.split, steps = whole ? all : all * (sp + 1) / a.split;   // [s0, steps)

    // this lane's sources within a step: W instruction q = WI wave + i fills
    // rows 8 (q mod 4) .. + 7 of column block q / 4; X instruction i fills row
    // block wave + NW i
    int woff[WI], nb[WI];
    const int wr = lane >> 3, wc = lane & 7;
    static_for<0, WI>([&](auto i) {
        const int q = WI * wave + (int)i, r = 8 * (q & 3) + wr;
        woff[i] = r * a.N * 2 + (wc ^ swz_w(r)) * 16;
        nb[i] = n0 + 64 * (q >> 2);
    });
    const int xr = lane >> 2;
    const int xoff = xr * 64 + ((lane & 3) ^ swz_x(xr)) * 16;
    const int n_rb = (a.M + 15) / 16;
    const bool has_x = wave < MB;
    const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_offset(lds));

    // Rows past M and columns past the end of W read as zero; columns past N
    // within W are other rows' values, in columns that are not stored.
    auto issue = [&](int s, uint32_t base) {
        const bool live = s < steps;   // past the end: an empty range, so that every stage issues as many loads
        static_for<0, KS>([&](auto ks) {
            const int k = (s * KS + (int)ks) * X::BK;
            const uint32_t to = base + (uint32_t)ks * X::STEP;
            static_for<0, WI>([&](auto i) {
                const int64_t left = ((int64_t)(a.K - k) * a.N - nb[i]) * 2;
                const int wbytes = live && nb[i] < a.N ? (int)min(left, (int64_t)64 * a.N) : 0;   // at most 32 rows
                lds_dma16<!OUT16>(rows_desc(a.w + ((int64_t)k * a.N + nb[i]) * 2, wbytes),
                                  to + (uint32_t)(WI * wave + (int)i) * 1024u, woff[i]);
            });
            if (has_x) {
                static_for<0, XI>([&](auto i) {
                    const int b = wave + NW * (int)i;
                    const int xrows = live ? min(max(rows - 16 * b, 0), 16) : 0;
                    const u32x4_t rx =
                        rows_desc(a.x + ((int64_t)(s * KS + (int)ks) * n_rb + m0 / 16 + b) * 1024, xrows * 64);
                    lds_dma16(rx, to + (uint32_t)(NS * X::SUB) + (uint32_t)b * 1024u, xoff);
                });
            }
        });
    };

    const int wn = wave % WN, wm = wave / WN;
    f32x4_t acc[T][RB];
    static_for<0, T>([&](auto t) { static_for<0, RB>([&](auto rb) { acc[t][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });

    static_for<0, NB - 1>([&](auto i) { issue(s0 + (int)i, lds0 + (uint32_t)i * X::STAGE); });
    for (int base = s0; base < steps; base += NB) {
        static_for<0, NB>([&](auto j) {
            constexpr int jj = decltype(j)::value;
            constexpr int jn = (jj + NB - 1) % NB;   // the buffer of step s - 1, free after the barrier
            const int s = base + jj;
            if (s < steps) {   // uniform
                if (has_x) wait_vmcnt<KS * (WI + XI) * (NB - 2)>();   // this wave's loads of stage s are done
                else wait_vmcnt<KS * WI * (NB - 2)>();
                __syncthreads();
                issue(s + NB - 1, lds0 + (uint32_t)jn * X::STAGE);
                static_for<0, KS>([&](auto ks) {
                    const char *buf = lds + jj * X::STAGE + (int)ks * X::STEP;
                    bf16x8_t xf[RB];
                    static_for<0, RB>([&](auto rb) {
                        xf[rb] = *reinterpret_cast<const bf16x8_t *>(buf + NS * X::SUB + (wm * RB + rb) * 1024 + col * 64 +
                                                                     (quad ^ swz_x(col)) * 16);
                    });
                    // lane (quad, col) names k 8 quad + 4 h + col / 4, columns
                    // 4 (col mod 4) .. + 3, and receives k 8 quad + 4 h .. + 3 of column col
                    i16x4_t wf[T][2];
                    static_for<0, T>([&](auto t) {
                        const int tile = wn * T + (int)t;
                        const int c = 2 * (tile & 3) + ((col & 3) >> 1);
                        static_for<0, 2>([&](auto h) {
                            const int r = 8 * quad + 4 * h + (col >> 2);
                            wf[t][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                (lds_i16x4_t *)(buf + (tile >> 2) * X::SUB + r * 128 + (c ^ swz_w(r)) * 16 + (col & 1) * 8));
                        });
                    });
                    static_for<0, T>([&](auto t) {
                        const u32x2_t v0 = __builtin_bit_cast(u32x2_t, wf[t][0]), v1 = __builtin_bit_cast(u32x2_t, wf[t][1]);
                        const bf16x8_t w8 = __builtin_bit_cast(bf16x8_t, u32x4_t{v0.x, v0.y, v1.x, v1.y});
                        static_for<0, RB>([&](auto rb) {
                            acc[t][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w8, xf[rb], acc[t][rb], 0, 0, 0);
                        });
                    });
                });
            }
        });
    }
    wait_vmcnt<0>();   // the empty loads past the end are done with the ring
    // lane (quad, col): columns 16 t + 4 quad .. + 3 of row col of each row block
    static_for<0, RB>([&](auto rb) {
        const int row = 16 * (wm * RB + rb) + col;
        if (row < rows) {
            const int ld = whole ? a.N : a.N - a.n_full * X::COLS;
            float *y = whole ? a.y + (size_t)(m0 + row) * a.N
                             : a.part + ((size_t)sp * a.M + m0 + row) * ld - a.n_full * X::COLS;
            static_for<0, T>([&](auto t) {
                const int n = n0 + 16 * (wn * T + (int)t) + 4 * quad;
                if (n < a.N) {
                    f32x4_t o = acc[t][rb];
                    if constexpr (OUT16) {
                        *reinterpret_cast<bf16x4_t *>(reinterpret_cast<__bf16 *>(a.y) + (size_t)(m0 + row) * a.N + n) =
                            __builtin_convertvector(o, bf16x4_t);
                    } else {
                        if (whole) static_for<0, 4>([&](auto i) { o[(int)i] = (float)(__bf16)o[(int)i]; });
                        *reinterpret_cast<f32x4_t *>(y + n) = o;
                    }
                }
            });
        }
    });
}

// The columns from n1 on: the partials added in order, rounded to bf16.
__global__ __launch_bounds__(256) void head_sum_kernel(const float *part, float *y, int M, int N, int n1, int split) {
    const int per = (N - n1) / 4;
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= M * per) return;
    const int row = u / per, c = 4 * (u % per);
    const size_t stride = (size_t)M * 4 * per;
    const float *p = part + (size_t)row * 4 * per + c;
    f32x4_t v = *reinterpret_cast<const f32x4_t *>(p);
    for (int s = 1; s < split; ++s) v += *reinterpret_cast<const f32x4_t *>(p + s * stride);
    static_for<0, 4>([&](auto i) { v[(int)i] = (float)(__bf16)v[(int)i]; });
    *reinterpret_cast<f32x4_t *>(y + (size_t)row * N + n1 + c) = v;
}

}  // namespace splice_dev
