// wide_f32.hpp -- float32 calls over a shared prompt: the prompt contraction
// for many (cell, q head) rows at once on the fp32 matrix cores.
//
// One launch of two kinds of work group, as in the bf16 kernel:
//   prompt items, four waves that own 64 rows of one KV head (rows of unspliced
//     and of spliced cells apart) and one prompt chunk: each tile of K and V is
//     read once for all 64 rows, straight into an LDS ring.  Per wave and 16
//     keys, with v_mfma_f32_16x16x4_f32 (fp32 products and sums):
//       S = K Q^T: lane (quad, col) holds four consecutive d of key col and of
//         row col, 16 bytes each, and four products take them one d at a time;
//       O^T += V^T P: product i takes key 4 quad + i, whose weight this lane
//         holds already; 16 bytes of V row 4 quad + i give the lane
//         d 64 u + 4 col + j of product (u, j).
//   generated-row items, one per (cell, KV head), on the vector ALUs.
// A second launch merges the partials.
//
// The vector-ALU kernels read the prompt again for every cell, which at many
// cells is what bounds them (64 cells, 1024 keys: 0.5 GB of L2 reads a call);
// here the fp32 products bound the prompt items (12 us a 1024 keys at 64 cells,
// 8 KV heads, G = 4, D = 128; the products' peak allows 8.5) and run beside the
// generated rows' reads.  Measured there, 129 generated rows: 1024 keys 75.0 ->
// 38.1 us a call, 2048 keys 113.9 -> 51.3; 16 cells and 1024 keys 32.1 -> 21.2.
// The second launch costs less than counting arrivals and merging in the last
// item to finish (1024 keys: 41 us against 56), and all partials are stored
// plainly.  Sums are kept in short chains (see WideF), so that the error against
// 64 bits is below that of the vector-ALU kernels: over 200 random shapes by D
// and G 0.55 to 0.95 of it at D <= 128 (prompts of 200 to 40000 keys), 0.43 to
// 0.77 at D = 256 (0.15 to 0.51 from 6144 keys on, where theirs are longer
// still).  With one chain per chunk above the 16 keys, one
// chain over the slots in the merge and eight accumulators at D = 256 it was up
// to 1.09 of it on average and 2.8 at prompts of 30000 keys; the short chains
// cost 2% of a call (D = 256: 4.5%).
//
// Part of attn_kernels.hpp, included there after what it builds on.
#pragma once

#include "prompt_wide.hpp"

namespace splice_dev {

template <int D>
struct WideF {
    static constexpr int NW = 4;
    static constexpr int ROWS = 16 * NW;
    static constexpr int TK = D <= 64 ? 32 : 16;     // keys per tile
    static constexpr int ROW = D * 4;
    static constexpr int CH = ROW / 16;              // 16-byte chunks per row
    static constexpr int TILE = TK * ROW;
    static constexpr int BUF = 2 * TILE;             // K tile, then V tile
    static constexpr int NB = D <= 128 ? 3 : 2;      // at D <= 128 LDS for three work groups a compute unit
    static constexpr int LDS = NB * BUF;
    static constexpr int PER = TK * CH / 64 / NW;    // load instructions per wave and operand
    static constexpr int KH = TK / 16, NG = D / 16, NU = D / 64;
    // Roundings of a chain add up, so chains are short: NS accumulators a score;
    // for the outputs a product chain per 16 keys (D = 256: two), then chains of
    // RAISE tiles, then those (D = 256 has no registers for these)
    static constexpr int NS = D <= 128 ? 8 : 16;
    static constexpr int NT = D <= 128 ? 1 : 2;
    static constexpr int RAISE = D <= 128 ? 64 / TK : 0;
};

template <int D, int G>
struct WideFLds {
    static constexpr int GEN = kWaves * 4 * G * (D + 1) * 4 + kWaves * G * 4;   // valu_merge
    static constexpr int BYTES = cmax(WideF<D>::LDS, GEN);
};

template <int D, int G>
__device__ __forceinline__ void wide_prompt_item(const AttnArgs &a, int item, char *lds) {
    using X = WideF<D>;
    constexpr int X8 = splice::kXcds, NB = X::NB;
    // the layout of the blocks is that of fused_prompt_item
    const int rg = (item / X8) % a.n_rb;
    const int unit = (item / X8 / a.n_rb) * X8 + item % X8;
    if (unit >= a.n_p * a.Hkv) return;
    const int g = unit / a.n_p, pk = unit % a.n_p;
    const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool clean_group = rg < a.n_rg_clean;
    const int first_cell = clean_group ? 0 : a.n_clean, end_cell = clean_group ? a.n_clean : a.n_active;
    const int grp = clean_group ? rg : rg - a.n_rg_clean;
    const int R = grp * X::ROWS + wave * 16 + col;
    const int cidx = first_cell + R / G, hh = R % G;
    const bool ok = cidx < end_cell;
    const int cell = ok ? a.order[cidx] : 0;

    const int k0 = a.jp0 + pk * a.p_len, k1 = min(k0 + a.p_len, a.Tp);
    const size_t head = (size_t)g * a.Tp * X::ROW;
    const char *ck = a.ck + head, *cv = a.cv + head;
    const int pre1 = min(k1, a.sa), sp0 = max(k0, a.sa), sp1 = min(k1, a.sb), post0 = max(k0, a.sb);
    KeyList L;
    list_init(L);
    list_add<X::TK>(L, ck + (size_t)k0 * X::ROW, cv + (size_t)k0 * X::ROW, pre1 - k0);
    if (clean_group) {
        list_add<X::TK>(L, ck + (size_t)sp0 * X::ROW, cv + (size_t)sp0 * X::ROW, sp1 - sp0);
    } else if (!a.zero_donor) {
        list_add<X::TK>(L, a.dk + head + (size_t)sp0 * X::ROW, a.dv + head + (size_t)sp0 * X::ROW, sp1 - sp0);
    }
    list_add<X::TK>(L, ck + (size_t)post0 * X::ROW, cv + (size_t)post0 * X::ROW, k1 - post0);
    const int n_tiles = list_tiles(L);

    f32x4_t o[X::NU][4], oh[X::RAISE ? X::NU : 1][4];   // oh, lh: the finished chains
    static_for<0, X::NU>([&](auto u) { static_for<0, 4>([&](auto j) { o[u][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });
    if constexpr (X::RAISE)
        static_for<0, X::NU>([&](auto u) { static_for<0, 4>([&](auto j) { oh[u][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });
    float m = -INFINITY, lsum = 0.f, lh = 0.f;
    if (n_tiles > 0) {
        // this lane's sources within a tile; chunk c of K row r sits at slot
        // c ^ (r mod 16), so that the 16 rows of a quarter-wave read touch every bank
        int koff[X::PER], voff[X::PER];
        static_for<0, X::PER>([&](auto i) {
            const int q = ((int)i * X::NW + wave) * 64 + lane;
            const int r = q / X::CH, sl = q % X::CH;
            koff[i] = r * X::ROW + (sl ^ (r & 15)) * 16;
            voff[i] = r * X::ROW + sl * 16;
        });
        const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_offset(lds));
        auto issue = [&](const TileRef &t, uint32_t base) {
            const u32x4_t rk = rows_desc(t.k, t.n * X::ROW), rv = rows_desc(t.v, t.n * X::ROW);
            static_for<0, X::PER>([&](auto i) {
                const uint32_t slot = (uint32_t)(((int)i * X::NW + wave) * 1024);
                lds_dma16(rk, base + slot, koff[i]);
                lds_dma16(rv, base + X::TILE + slot, voff[i]);
            });
        };
        TileIter it;
        it.k = L.k[0];
        it.v = L.v[0];
        it.key0 = 0;
        it.seg = 0;
        iter_seg(L, it);
        TileRef ref[NB];
        static_for<0, NB - 1>([&](auto i) {
            ref[i] = iter_next<X::TK>(L, it, X::ROW);
            issue(ref[i], lds0 + (uint32_t)i * X::BUF);
        });
        f32x4_t qf[X::NG];
        const char *qrow = a.q + ((size_t)cell * a.Hq + (size_t)g * G + hh) * X::ROW;
        static_for<0, X::NG>([&](auto n) {
            qf[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (ok) qf[n] = *reinterpret_cast<const f32x4_t *>(qrow + (16 * n + 4 * quad) * 4);
        });
        wait_vmcnt<0>();
        for (int base = 0; base < n_tiles; base += NB) {
            static_for<0, NB>([&](auto jb) {
                constexpr int jj = decltype(jb)::value, jn = (jj + NB - 1) % NB;
                if (base + jj < n_tiles) {   // uniform
                    wait_vmcnt<2 * X::PER *(NB - 2)>();   // this wave's loads of the tile are done
                    __syncthreads();
                    ref[jn] = iter_next<X::TK>(L, it, X::ROW);
                    issue(ref[jn], lds0 + (uint32_t)jn * X::BUF);
                    const char *sK = lds + jj * X::BUF, *sV = sK + X::TILE;
                    const int n_valid = ref[jj].n;
                    // NS sums of D / NS products, added at the end
                    f32x4_t s[X::KH], sn[X::KH][X::NS];
                    static_for<0, X::KH>([&](auto kh) {
                        static_for<0, X::NS>([&](auto j) { sn[kh][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
                    });
                    static_for<0, X::NG>([&](auto n) {
                        static_for<0, X::KH>([&](auto kh) {
                            const int r = 16 * kh + col;
                            const f32x4_t kf =
                                *reinterpret_cast<const f32x4_t *>(sK + r * X::ROW + ((4 * n + quad) ^ (r & 15)) * 16);
                            static_for<0, 4>([&](auto j) {
                                constexpr int sj = 4 * (decltype(n)::value % (X::NS / 4)) + decltype(j)::value;
                                sn[kh][sj] =
                                    __builtin_amdgcn_mfma_f32_16x16x4f32(kf[(int)j], qf[n][(int)j], sn[kh][sj], 0, 0, 0);
                            });
                        });
                    });
                    static_for<0, X::KH>([&](auto kh) {
                        if constexpr (X::NS == 16) static_for<0, 8>([&](auto j) { sn[kh][j] += sn[kh][j + 8]; });
                        s[kh] = ((sn[kh][0] + sn[kh][1]) + (sn[kh][2] + sn[kh][3])) +
                                ((sn[kh][4] + sn[kh][5]) + (sn[kh][6] + sn[kh][7]));
                    });
                    float mt = -INFINITY;
                    static_for<0, X::KH>([&](auto kh) {
                        static_for<0, 4>([&](auto i) {
                            if (16 * kh + 4 * quad + i >= n_valid) s[kh][(int)i] = -INFINITY;
                            mt = fmaxf(mt, s[kh][(int)i]);
                        });
                    });
                    mt *= a.qk_scale;
                    if (__any(mt > m + kSlack)) {   // as direct_compute
                        mt = fmaxf(mt, __shfl_xor(mt, 16));
                        mt = fmaxf(mt, __shfl_xor(mt, 32));
                        const bool need = mt > m + kSlack;
                        const float mn = need ? fmaxf(m, mt) : m;
                        const float al = need ? fast_exp2(m - (mn == -INFINITY ? 0.f : mn)) : 1.f;
                        lsum *= al;
                        lh *= al;
                        static_for<0, X::NU>([&](auto u) { static_for<0, 4>([&](auto j) { o[u][j] *= al; }); });
                        if constexpr (X::RAISE)
                            static_for<0, X::NU>([&](auto u) { static_for<0, 4>([&](auto j) { oh[u][j] *= al; }); });
                        m = mn;
                    }
                    const float ms = m == -INFINITY ? 0.f : m;
                    static_for<0, X::KH>([&](auto kh) {
                        float p[4];
                        static_for<0, 4>(
                            [&](auto i) { p[(int)i] = fast_exp2(fmaf(s[kh][(int)i], a.qk_scale, -ms)); });
                        lsum += (p[0] + p[1]) + (p[2] + p[3]);
                        static_for<0, X::NU>([&](auto u) {
                            f32x4_t t[X::NT][4];
                            static_for<0, X::NT>([&](auto k) {
                                static_for<0, 4>([&](auto j) { t[k][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
                            });
                            static_for<0, 4>([&](auto i) {
                                const f32x4_t vf = *reinterpret_cast<const f32x4_t *>(
                                    sV + (16 * kh + 4 * quad + i) * X::ROW + col * 16 + 256 * u);
                                constexpr int k = decltype(i)::value * X::NT / 4;
                                static_for<0, 4>([&](auto j) {
                                    t[k][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[(int)j], p[(int)i], t[k][j], 0, 0, 0);
                                });
                            });
                            static_for<0, 4>([&](auto j) { o[u][j] += X::NT > 1 ? t[0][j] + t[X::NT - 1][j] : t[0][j]; });
                        });
                    });
                    if constexpr (X::RAISE) {
                        if ((base + jj) % X::RAISE == X::RAISE - 1) {   // uniform
                            lh += lsum;
                            lsum = 0.f;
                            static_for<0, X::NU>([&](auto u) {
                                static_for<0, 4>([&](auto j) {
                                    oh[u][j] += o[u][j];
                                    o[u][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                                });
                            });
                        }
                    }
                }
            });
        }
        wait_vmcnt<0>();
    }
    lsum += lh;
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
    if constexpr (X::RAISE)
        static_for<0, X::NU>([&](auto u) { static_for<0, 4>([&](auto j) { o[u][j] += oh[u][j]; }); });
    if (ok) {   // o[u][j][i] is d 64 u + 16 quad + 4 i + j
        using SL = Slot<D, G, false>;
        char *slot = reinterpret_cast<char *>(a.part) + pslot_off(a, cell, g, pk);
        static_for<0, X::NU>([&](auto u) {
            static_for<0, 4>([&](auto i) {
                *reinterpret_cast<f32x4_t *>(slot + SL::o(hh, 64 * u + 16 * quad + 4 * i)) =
                    f32x4_t{o[u][0][(int)i], o[u][1][(int)i], o[u][2][(int)i], o[u][3][(int)i]};
            });
        });
        if (quad == 0) {
            *reinterpret_cast<float *>(slot + SL::m(hh)) = m;
            *reinterpret_cast<float *>(slot + SL::l(hh)) = lsum;
        }
    }
}

// The generated rows of (cell c, KV head g) as one more partial result.
template <int D, int G>
__device__ __forceinline__ void wide_gen_item(const AttnArgs &a, int c, int g, char *lds) {
    using V = Valu<D, G, false>;
    using SL = Slot<D, G, false>;
    uint32_t qr[G][V::QW];
    load_q<D, G, false>(a, c, g, qr);
    const size_t off = (((size_t)c * a.Hkv + g) * (size_t)a.cap + a.i0) * V::ROW;
    const char *kb = a.gk + off, *vb = a.gv + off;
    float m[G], l[G], o[G][V::EL];
    valu_stream<D, G, false, 1>(qr, 0, a.n_gen, a.qk_scale,
                             [&](int key, const char *&kp, const char *&vp) {
                                 kp = kb + (size_t)key * V::ROW;
                                 vp = vb + (size_t)key * V::ROW;
                                 return true;
                             },
                             m, l, o);
    char *slot = reinterpret_cast<char *>(a.part) + gslot_off(a, c, g, 0);
    valu_merge<D, G, false>(m, l, o, lds, [&](int h, int d, float M, float L, f32x4_t O) {
        *reinterpret_cast<f32x4_t *>(slot + SL::o(h, d)) = O;
        if (d == 0) {
            *reinterpret_cast<float *>(slot + SL::m(h)) = M;
            *reinterpret_cast<float *>(slot + SL::l(h)) = L;
        }
    });
}

template <int D, int G>
__global__ __launch_bounds__(kThreads) void wide_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[WideFLds<D, G>::BYTES];
    const int item = (int)blockIdx.x - a.n_prompt_items;
    if (item < 0) wide_prompt_item<D, G>(a, blockIdx.x, lds);
    else wide_gen_item<D, G>(a, item / a.Hkv, item % a.Hkv, lds);
}

// Launched after wide_kernel, so the partials are simply in memory: a thread
// per (cell, q head, four outputs) folds them in the fixed order.
template <int D, int G>
__global__ __launch_bounds__(kThreads) void wide_merge_kernel(AttnArgs a) {
    using SL = Slot<D, G, false>;
    const int u = blockIdx.x * kThreads + threadIdx.x, per = D / 4;
    if (u >= a.C * a.Hq * per) return;
    const int d = 4 * (u % per), c = u / per / a.Hq, hq = u / per % a.Hq, g = hq / G, h = hq % G;
    const char *part = reinterpret_cast<const char *>(a.part);
    const char *ps = part + pslot_off(a, c, g, 0), *gs = part + gslot_off(a, c, g, 0);
    constexpr int B = splice::kWideF32MaxChunks + 1;
    float mk[B], lk[B];
    f32x4_t ok[B];
    static_for<0, B>([&](auto k) {   // every slot's loads in one round; the generated rows' slot comes last
        if (k <= a.n_p) {
            const char *s = k < a.n_p ? ps + (size_t)k * a.p_slot_bytes : gs;
            mk[k] = *reinterpret_cast<const float *>(s + SL::m(h));
            lk[k] = *reinterpret_cast<const float *>(s + SL::l(h));
            ok[k] = *reinterpret_cast<const f32x4_t *>(s + SL::o(h, d));
        }
    });
    const int nz = zero_slots(a, c);
    float M = nz > 0 ? 0.f : -INFINITY;
    static_for<0, B>([&](auto k) {
        if (k <= a.n_p) M = fmaxf(M, mk[k]);
    });
    // four chains of slots: every addition to an output that one key dominates rounds it
    float Lc[4] = {nz > 0 ? (float)nz * fast_exp2(-M) : 0.f, 0.f, 0.f, 0.f};
    f32x4_t Oc[4];
    static_for<0, 4>([&](auto c4) { Oc[c4] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
    static_for<0, B>([&](auto k) {
        if (k <= a.n_p) fold_slot(mk[k], lk[k], ok[k], M, Lc[k % 4], Oc[k % 4]);
    });
    const float L = (Lc[0] + Lc[1]) + (Lc[2] + Lc[3]);
    const f32x4_t O = (Oc[0] + Oc[1]) + (Oc[2] + Oc[3]);
    const size_t row = (size_t)c * a.Hq + hq;
    *reinterpret_cast<f32x4_t *>(a.out + row * D + d) = O * (1.f / L);
    if (d == 0) a.lse[row] = (M + log2f(L)) * kLn2;
}

}  // namespace splice_dev
