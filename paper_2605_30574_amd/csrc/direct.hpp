// direct.hpp -- bf16 calls over short key lists: one work group per (cell, KV
// head) streams the cell's whole visible list (its prompt slots by pointer,
// then its generated rows), NW waves taking tiles in turn, and writes out and
// lse itself.
//
// Such a call is a chain of latencies.  The shared-prompt kernel's chain is
// first tiles, partial stores written through, arrival counters, polls, slot
// loads; here it is first tiles, then a merge of the waves in LDS.  The prompt
// tiles that the cells share are read again for each, from L2.
//
// Part of attn_kernels.hpp, included there after what it builds on.
#pragma once

#include "wave_mfma.hpp"

namespace splice_dev {

template <int D>
struct DirectWaves {
    static constexpr int NW = 4;
    static constexpr int DEPTH = D <= 128 ? 2 : 1;   // tiles in flight per wave
    static constexpr int NT = 64 * NW;
};

template <int D, int G>
__global__ __launch_bounds__(DirectWaves<D>::NT) void direct_kernel(AttnArgs a) {
    using W = WaveMfma<D>;
    constexpr int NW = DirectWaves<D>::NW, NT = DirectWaves<D>::NT, NSEG = 5;
    __shared__ __attribute__((aligned(16))) char lds[cmax(NW * W::LDS, NW * G * (D + 2) * 4)];
    const int g = blockIdx.x % a.Hkv, c = a.gorder[blockIdx.x / a.Hkv];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = threadIdx.x & 15;
    bf16x8_t qb[W::NDS];
    load_q_cols<D>(a.q + ((size_t)c * a.Hq + (size_t)g * G + col % G) * W::ROW, qb);
    // the segments are the same for spliced and unspliced cells, so a splice
    // moves no tile boundary
    const CellGeo geo = cell_geo(a, c);
    const bool spl = bit_set(a.spliced, c);
    KeyListN<NSEG> L;
    list_init(L);
    const size_t head = (size_t)g * a.Tp * W::ROW;
    const char *ck = a.ck + head, *cv = a.cv + head;
    auto at = [](const char *p, int row) { return p + (size_t)row * W::ROW; };
    list_add<kTileKeys, NSEG>(L, at(ck, geo.jp0), at(cv, geo.jp0), geo.sa - geo.jp0);
    if (!spl) list_add<kTileKeys, NSEG>(L, at(ck, geo.sa), at(cv, geo.sa), geo.sb - geo.sa);
    else if (!a.zero_donor)
        list_add<kTileKeys, NSEG>(L, at(a.dk + head, geo.sa), at(a.dv + head, geo.sa), geo.sb - geo.sa);
    list_add<kTileKeys, NSEG>(L, at(ck, geo.sb), at(cv, geo.sb), a.Tp - geo.sb);
    const int i1 = geo.i0 + geo.n_gen;
    const bool fork = a.trunk >= 0 && c != a.trunk;   // rows below the fork step are the trunk's
    const int wf = fork ? min(max(a.wfork[c], geo.i0), i1) : geo.i0;
    if (fork) {
        const size_t off = ((size_t)a.trunk * a.Hkv + g) * (size_t)a.cap * W::ROW;
        list_add<kTileKeys, NSEG>(L, at(a.gk + off, geo.i0), at(a.gv + off, geo.i0), wf - geo.i0);
    }
    const size_t off = ((size_t)c * a.Hkv + g) * (size_t)a.cap * W::ROW;
    list_add<kTileKeys, NSEG>(L, at(a.gk + off, wf), at(a.gv + off, wf), i1 - wf);

    WaveState<D> S;
    state_init(S);
    const ColMask cm{true, true, true};
    wave_stream<D, DirectWaves<D>::DEPTH, kAuxNormal, kAuxNormal, NSEG>(L, wave, NW, cm, qb, a.qk_scale,
                                                                         lds + wave * W::LDS, S);
    state_finish(S);
    const int nz = zero_slots(a, c);
    waves_merge<D, G, NW>(S, lds, NW, 1, [&](int, int h, int d, float M, float Ls, f32x4_t O) {
        if (nz > 0) {   // nz keys of score 0 and value 0
            const float Mz = fmaxf(M, 0.f), f = fast_exp2(M - Mz);
            Ls = Ls * f + (float)nz * fast_exp2(-Mz);
            O *= f;
            M = Mz;
        }
        write_row(a, c, g * G + h, d, D, M, Ls, O);
    });
    if (c == a.trunk && a.n_dormant > 0) {   // uniform
        __syncthreads();
        dormant_copy<D, G, NT>(a, g, lds);
    }
}

}  // namespace splice_dev
