// Attention of a long block of ONE sequence (a prompt chunk of up to some hundred rows; paper Eq. 2: the target
// model's forward over given tokens).  The decode kernel (sj_attn.h) keeps the block's own K / V rows in LDS and
// is limited to 64 of them; here the rows go to the cache first and every query row then reads the cache:
//
//  prefill_rotary_kernel  sums the QKV split-K partials of 16 positions x one kv head, rotates Q and K, appends
//                         K and (through LDS, transposed) V to the cache and writes the query rows as MFMA fragments;
//  prefill_attn_kernel    one wave = MQ tiles of 16 query columns over the cached keys they can see.
//
// Query columns of a kv head are ordered position-major (column = position * G + head of the group), so a tile of 16
// covers 16 / G neighbouring positions and a wave stops at the last key its positions see: half of the score matrix is
// never formed.  Products, key permutation and running softmax are those of the decode kernel, so a row's result does
// not depend on which of the two computed it beyond the order of the sums.
//
// What bounds it: little at the sizes of a prompt.  A layer of the 8B shape over 509 rows is 4 GFLOP here against 440
// GFLOP (two operand planes) of projections.  What it buys is the length of a chunk: 509 tokens through 4 layers and the
// scoring of a block took 36.7 ms in 85 blocks of 6 rows, and take 3.1 ms in one chunk.
#pragma once
#include "sj_attn.h"

namespace sj {

constexpr int PF_POS = 16;         // positions per workgroup of the rotary kernel (= G whole query tiles)

// Query fragments: qbuf[kv head][query tile][head-dim step][plane][64 lanes] of 16 bytes; tiles of a kv head = G * ceil(rps / 16).
template <typename T, int HD, int SPL>
__global__ __launch_bounds__(256) void prefill_rotary_kernel(const StepParams* __restrict__ sp, ModelDims md,
                                                             const float* __restrict__ part, int nparts, int R,
                                                             const float* __restrict__ cs, KvView<T> kv, int layer,
                                                             u32x4* __restrict__ qbuf) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP, KK = HD / KSTEP, HALF = HD / 2;
    __shared__ T vt[HD][PF_POS + 2];
    const int rps = sp->rps, b = sp->seq_base, L = kv.len[b], cap = kv.cap[b];
    const int p0 = blockIdx.x * PF_POS, kvh = blockIdx.y, tid = threadIdx.x;
    const int Nq = md.Hq * HD, Nk = md.Hkv * HD, N = Nq + 2 * Nk;
    const int ntiles = md.G * gridDim.x;
    T* Kb = kv.K + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * cap * HD;
    T* Vb = kv.V + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * HD * cap;
    // sum of the partials of four neighbouring columns of one row, in slice order
    auto sum4 = [&](int row, int col) {
        f32x4 v = *reinterpret_cast<const f32x4*>(part + (size_t)row * N + col);
        for (int s = 1; s < nparts; ++s) v += *reinterpret_cast<const f32x4*>(part + ((size_t)s * R + row) * N + col);
        return v;
    };

    // queries: item = (column pair of fragments kk, kk + KK/2; lane group; column of the workgroup's 16 * G)
    const int nq = PF_POS * md.G * 4 * (KK / 2);
    for (int it = tid; it < nq; it += 256) {
        const int r = it & 15, g = (it >> 4) & 3, rest = it >> 6;
        const int kk = rest % (KK / 2), tt = rest / (KK / 2);
        const int col = tt * 16 + r, j = small_div(col, md.G), gi = col - j * md.G;
        const int row = min(p0 + j, rps - 1);          // columns past the block: valid memory, never used
        const int i0 = kk * KSTEP + g * KF, c0 = (kvh * md.G + gi) * HD + i0;
        Frag f0[SPL], f1[SPL];
#pragma unroll
        for (int e4 = 0; e4 < KF; e4 += 4) {
            const f32x4 lo = sum4(row, c0 + e4), hi = sum4(row, c0 + HALF + e4);
            const float* csr = cs + ((size_t)row * HALF + i0 + e4) * 2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = csr[2 * e], s = csr[2 * e + 1];
                Traits<T>::template pack_split<SPL>(f0, e4 + e, lo[e] * c - hi[e] * s);
                Traits<T>::template pack_split<SPL>(f1, e4 + e, hi[e] * c + lo[e] * s);
            }
        }
        u32x4* q = qbuf + (((size_t)kvh * ntiles + (size_t)blockIdx.x * md.G + tt) * KK) * SPL * 64 + 16 * g + r;
#pragma unroll
        for (int pl = 0; pl < SPL; ++pl) {
            q[(kk * SPL + pl) * 64] = f0[pl].u;
            q[((kk + KK / 2) * SPL + pl) * 64] = f1[pl].u;
        }
    }
    // keys: four neighbouring columns of the lower and of the upper half of one position
    for (int it = tid; it < PF_POS * (HALF / 4); it += 256) {
        const int j = it / (HALF / 4), i = (it % (HALF / 4)) * 4, row = p0 + j;
        if (row < rps && L + row < cap) {
            const f32x4 lo = sum4(row, Nq + kvh * HD + i), hi = sum4(row, Nq + kvh * HD + HALF + i);
            const float* csr = cs + ((size_t)row * HALF + i) * 2;
            T* k = Kb + (size_t)(L + row) * HD + i;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = csr[2 * e], s = csr[2 * e + 1];
                Traits<T>::store(k + e, lo[e] * c - hi[e] * s);
                Traits<T>::store(k + HALF + e, hi[e] * c + lo[e] * s);
            }
        }
    }
    // values: transposed through LDS, then 16 consecutive positions per row of the cache
    for (int it = tid; it < PF_POS * (HD / 4); it += 256) {
        const int j = it / (HD / 4), i = (it % (HD / 4)) * 4, row = min(p0 + j, rps - 1);
        const f32x4 v = sum4(row, Nq + Nk + kvh * HD + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) Traits<T>::store(&vt[i + e][j], v[e]);
    }
    __syncthreads();
    for (int it = tid; it < PF_POS * HD; it += 256) {
        const int j = it % PF_POS, i = it / PF_POS, pos = L + p0 + j;
        if (p0 + j < rps && pos < cap) Vb[(size_t)i * cap + pos] = vt[i][j];
    }
}

template <typename T, int HD, int MQ, int SPL>
__global__ __launch_bounds__(256) void prefill_attn_kernel(const StepParams* __restrict__ sp, ModelDims md, KvView<T> kv, int layer,
                                                           const u32x4* __restrict__ qbuf, int ntiles, T* __restrict__ attn_out,
                                                           size_t aplane, int otks) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP, NS = KF / 4, KK = HD / KSTEP, HT = HD / 16;
    const int rps = sp->rps, b = sp->seq_base, L = kv.len[b], cap = kv.cap[b], kvh = blockIdx.y;
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    // the tiles with the most keys first: the launch ends with its shortest waves
    const int t0 = __builtin_amdgcn_readfirstlane((((int)(gridDim.x - 1 - blockIdx.x)) * 4 + (int)(threadIdx.x >> 6)) * MQ);
    if (t0 >= ntiles) return;                          // no barrier in this kernel
    const T* Kb = kv.K + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * cap * HD;
    const T* Vb = kv.V + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * HD * cap;

    // column of tile t: position (t / G) * 16 + c / G, head c % G, c = (t % G) * 16 + r
    Frag qf[MQ][KK][SPL];
    int jrow[MQ], girow[MQ], jmax = 0;
    bool rowvalid[MQ];
#pragma unroll
    for (int mq = 0; mq < MQ; ++mq) {
        const int t = min(t0 + mq, ntiles - 1), blk = small_div(t, md.G), c = (t - blk * md.G) * 16 + r;
        const int j = small_div(c, md.G);
        jrow[mq] = blk * PF_POS + j;
        girow[mq] = c - j * md.G;
        rowvalid[mq] = t0 + mq < ntiles && jrow[mq] < rps;
        jmax = max(jmax, blk * PF_POS + small_div((t - blk * md.G) * 16 + 15, md.G));
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int pl = 0; pl < SPL; ++pl)
                qf[mq][kk][pl].u = qbuf[((((size_t)kvh * ntiles + t) * KK + kk) * SPL + pl) * 64 + lane];
    }
    const int key_hi = min(L + min(jmax, rps - 1) + 1, cap);   // keys this wave's rows can see

    Frag kf[2][NS][KK], vf[2][HT];
    auto load_keys = [&](int set, int key) {           // key < cap: capacities are multiples of 64
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            const int krow = key + KF * (r >> 2) + 4 * t + (r & 3);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kf[set][t][kk].u = *reinterpret_cast<const u32x4*>(Kb + (size_t)krow * HD + kk * KSTEP + g * KF);
        }
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) vf[set][ht].u = *reinterpret_cast<const u32x4*>(Vb + (size_t)(ht * 16 + r) * cap + key + g * KF);
    };

    f32x4 o[HT][MQ];
    float m_run[MQ], l_run[MQ];
#pragma unroll
    for (int mq = 0; mq < MQ; ++mq) {
        m_run[mq] = -INFINITY;
        l_run[mq] = 0.f;
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) o[ht][mq] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto step = [&](int set, int key0) {
        if (key0 + KSTEP > L + rps) {                  // V past the block holds whatever the cache had: 0 * value stays 0
#pragma unroll
            for (int ht = 0; ht < HT; ++ht)
#pragma unroll
                for (int e = 0; e < KF; ++e)
                    if (key0 + g * KF + e >= L + rps) {
                        if constexpr (sizeof(T) == 2) vf[set][ht].s[e] = 0; else vf[set][ht].f[e] = 0.f;
                    }
        }
        f32x4 s[NS][MQ];
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) {
                s[t][mq] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                    for (int pl = 0; pl < SPL; ++pl) Traits<T>::mma(kf[set][t][kk], qf[mq][kk][pl], s[t][mq]);
            }
        Frag pf[MQ][SPL];
#pragma unroll
        for (int mq = 0; mq < MQ; ++mq) {
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = rowvalid[mq] && key0 + KF * g + 4 * t + i <= L + jrow[mq] ? s[t][mq][i] * md.scale : -INFINITY;
                    s[t][mq][i] = v;
                    mx = fmaxf(mx, v);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_new = fmaxf(m_run[mq], mx);
            const bool dead = (m_new == -INFINITY);
            const float alpha = dead ? 1.f : __expf(m_run[mq] - m_new);
            float psum = 0.f;
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float p = dead ? 0.f : __expf(s[t][mq][i] - m_new);
                    psum += p;
                    Traits<T>::template pack_split<SPL>(pf[mq], 4 * t + i, p);
                }
            l_run[mq] = l_run[mq] * alpha + psum;
            m_run[mq] = m_new;
#pragma unroll
            for (int ht = 0; ht < HT; ++ht) o[ht][mq] *= alpha;
        }
#pragma unroll
        for (int ht = 0; ht < HT; ++ht)
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq)
#pragma unroll
                for (int pl = 0; pl < SPL; ++pl) Traits<T>::mma(vf[set][ht], pf[mq][pl], o[ht][mq]);
    };
    load_keys(0, 0);
    int key0 = 0;
    while (key0 + KSTEP < key_hi) {                    // the next step is requested before the current one is used
        load_keys(1, key0 + KSTEP);
        step(0, key0);
        load_keys(0, min(key0 + 2 * KSTEP, cap - KSTEP));       // may lie past this wave's keys: in bounds, unused then
        step(1, key0 + KSTEP);
        key0 += 2 * KSTEP;
    }
    if (key0 < key_hi) step(0, key0);

#pragma unroll
    for (int mq = 0; mq < MQ; ++mq) {
        float l = l_run[mq];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (rowvalid[mq]) {
            const float inv = 1.f / l;
#pragma unroll
            for (int ht = 0; ht < HT; ++ht) {
                const float v[4] = {o[ht][mq][0] * inv, o[ht][mq][1] * inv, o[ht][mq][2] * inv, o[ht][mq][3] * inv};
                Traits<T>::template store_split4<SPL>(attn_out + opnd_off<T>(jrow[mq], (kvh * md.G + girow[mq]) * HD + ht * 16 + 4 * g, md.Hq * HD, otks), aplane, v);
            }
        }
    }
}

}  // namespace sj
