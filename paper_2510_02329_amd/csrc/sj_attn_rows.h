// Attention over many query rows (a prompt chunk of one sequence, or the blocks of a large batch; paper Eq. 2: the target
// model's forward over given tokens), in two launches.  The decode kernel (sj_attn.h) is one launch whose workgroups each sum and
// rotate the query rows they need and keep the block's own K / V rows in LDS; with many rows that work is repeated for every key
// range.  Here it is done once:
//
//  rows_rotary_kernel  (a workgroup each for queries, keys and values) sums the QKV split-K partials of 16 positions x one kv
//                      head, rotates Q and K, appends K and (through LDS, transposed) V to the cache and writes the query rows as
//                      MFMA fragments;
//  rows_attn_kernel    reads the cache only: a workgroup of eight waves takes 8 / KW tiles of 16 query columns, KW waves share a
//                      tile's keys (every KW-th step of 32) and meet in LDS.
//
// Query columns of a kv head are ordered position-major (column = position * G + head of the group), so a tile of 16
// covers 16 / G neighbouring positions and its waves stop at the last key its positions see.  Products, key permutation and
// running softmax are those of the decode kernel, so a row's result does not depend on which of the two computed it beyond the
// order of the sums.
//
// What bounds it: per step of 32 keys and tile, 32 MFMAs (two operand planes) and about 150 vector instructions, which
// two waves of a SIMD overlap (one tile a wave: about 200 registers; the decode kernel's three tiles a wave take 478 and leave one).
// Measured (8B shape, two planes): 6 blocks of 21 rows over 60 - 700 keys: 83 us in one launch, 13 + 13 us in two; a prompt chunk of
// 509 rows: 19 + 11 us; 16 blocks of 9 rows over 512 - 4096 keys: 66 + 15 us against 69 in one launch, whose key ranges fill the
// chip better - the rule at many_rows_attention keeps it there.
#pragma once
#include "sj_attn.h"

namespace sj {

constexpr int ROT_POS = 16;        // positions per workgroup of the rotary kernel (= G whole query tiles)

// Query fragments: qbuf[sequence][kv head][query tile][head-dim step][plane][64 lanes] of 16 bytes; ntiles = ceil(rps * G / 16).
// q0: positions before it want no attention output (a prompt's last layer; 0: all do).  Their keys and values are appended like the others';
// their query tiles are not formed, and the output rows begin with position q0.
template <typename T, int HD, int SPL, int PB>
__global__ __launch_bounds__(256) void rows_rotary_kernel(const StepParams* __restrict__ sp, ModelDims md,
                                                             const float* __restrict__ part, int nparts, int R,
                                                             const float* __restrict__ cs, KvView<T> kv, int layer,
                                                             u32x4* __restrict__ qbuf, int ntiles, int q0) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP, KK = HD / KSTEP, HALF = HD / 2;
    __shared__ T vt[HD][ROT_POS + 2];
    const int rps = sp->rps, bi = blockIdx.z, b = sp->seq_base + bi, L = kv.len[b], cap = kv.cap[b];
    const int p0 = blockIdx.x * ROT_POS, kvh = blockIdx.y % md.Hkv, tid = threadIdx.x, r0 = bi * rps;   // r0: the sequence's first row
    const int Nq = md.Hq * HD, Nk = md.Hkv * HD, N = Nq + 2 * Nk;
    T* Kb = kv.K + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * cap * HD;
    T* Vb = kv.V + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * HD * cap;
    // sums of the partials of four neighbouring columns of one row (at each of n places), in slice order; PB slices of
    // independent loads at a time (index clamped, surplus ignored)
    auto sums = [&](auto& v, int row, auto col_of) {
        constexpr int n = sizeof(v) / sizeof(v[0]);
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < nparts; s0 += PB) {
            f32x4 t[PB][n];
#pragma unroll
            for (int u = 0; u < PB; ++u)
#pragma unroll
                for (int i = 0; i < n; ++i)
                    t[u][i] = *reinterpret_cast<const f32x4*>(part + ((size_t)min(s0 + u, nparts - 1) * R + row) * N + col_of(i));
#pragma unroll
            for (int u = 0; u < PB; ++u)
#pragma unroll
                for (int i = 0; i < n; ++i)
                    if (s0 + u < nparts) v[i] += t[u][i];
        }
    };
    const int role = blockIdx.y / md.Hkv;                // 0: queries, 1: keys, 2: values

    // queries: item = (column pair of fragments kk, kk + KK/2; lane group; column of the workgroup's 16 * G)
    const int nq = role != 0 || p0 + ROT_POS <= q0 ? 0 : min(md.G, ntiles - (int)blockIdx.x * md.G) * 16 * 4 * (KK / 2);
    for (int it = tid; it < nq; it += 256) {
        const int r = it & 15, g = (it >> 4) & 3, rest = it >> 6;
        const int kk = rest % (KK / 2), tt = rest / (KK / 2);
        const int col = tt * 16 + r, j = small_div(col, md.G), gi = col - j * md.G;
        const int row = r0 + min(p0 + j, rps - 1);     // columns past the block: valid memory, never used
        const int i0 = kk * KSTEP + g * KF, c0 = (kvh * md.G + gi) * HD + i0;
        Frag f0[SPL], f1[SPL];
        f32x4 v[KF / 2];                               // KF / 4 places of the lower half, then of the upper
        sums(v, row, [&](int i) { return c0 + (i % (KF / 4)) * 4 + (i / (KF / 4)) * HALF; });
#pragma unroll
        for (int e4 = 0; e4 < KF; e4 += 4) {
            const f32x4 lo = v[e4 / 4], hi = v[KF / 4 + e4 / 4];
            const float* csr = cs + ((size_t)row * HALF + i0 + e4) * 2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = csr[2 * e], s = csr[2 * e + 1];
                Traits<T>::template pack_split<SPL>(f0, e4 + e, lo[e] * c - hi[e] * s);
                Traits<T>::template pack_split<SPL>(f1, e4 + e, hi[e] * c + lo[e] * s);
            }
        }
        u32x4* q = qbuf + ((((size_t)bi * md.Hkv + kvh) * ntiles + (size_t)blockIdx.x * md.G + tt) * KK) * SPL * 64 + 16 * g + r;
#pragma unroll
        for (int pl = 0; pl < SPL; ++pl) {
            q[(kk * SPL + pl) * 64] = f0[pl].u;
            q[((kk + KK / 2) * SPL + pl) * 64] = f1[pl].u;
        }
    }
    // keys: four neighbouring columns of the lower and of the upper half of one position
    for (int it = role == 1 ? tid : ROT_POS * HALF; it < ROT_POS * (HALF / 4); it += 256) {
        const int j = it / (HALF / 4), i = (it % (HALF / 4)) * 4, row = p0 + j;
        if (row < rps && L + row < cap) {
            f32x4 v[2];
            sums(v, r0 + row, [&](int k) { return Nq + kvh * HD + k * HALF + i; });
            const f32x4 lo = v[0], hi = v[1];
            const float* csr = cs + ((size_t)(r0 + row) * HALF + i) * 2;
            T *k0 = Kb + kv_k_off<T>(L + row, i, HD), *k1 = Kb + kv_k_off<T>(L + row, HALF + i, HD);   // four neighbours each
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = csr[2 * e], s = csr[2 * e + 1];
                Traits<T>::store(k0 + e, lo[e] * c - hi[e] * s);
                Traits<T>::store(k1 + e, hi[e] * c + lo[e] * s);
            }
        }
    }
    // values: transposed through LDS, then into the cache's fragments (16 positions of a column are two runs of 16 bytes)
    if (role != 2) return;                               // uniform for the workgroup
    for (int it = tid; it < ROT_POS * (HD / 4); it += 256) {
        const int j = it / (HD / 4), i = (it % (HD / 4)) * 4, row = min(p0 + j, rps - 1);
        f32x4 v[1];
        sums(v, r0 + row, [&](int) { return Nq + Nk + kvh * HD + i; });
#pragma unroll
        for (int e = 0; e < 4; ++e) Traits<T>::store(&vt[i + e][j], v[0][e]);
    }
    __syncthreads();
    for (int it = tid; it < ROT_POS * HD; it += 256) {
        const int j = it % ROT_POS, i = it / ROT_POS, pos = L + p0 + j;
        if (p0 + j < rps && pos < cap) Vb[kv_v_off<T>(pos, i, HD)] = vt[i][j];
    }
}

constexpr int ROWS_WAVES = 8;

template <typename T, int HD, int KW, int SPL>
__global__ __launch_bounds__(ROWS_WAVES * 64) void rows_attn_kernel(const StepParams* __restrict__ sp, ModelDims md, KvView<T> kv, int layer,
                                                                    const u32x4* __restrict__ qbuf, int ntiles, int q0, T* __restrict__ attn_out,
                                                                    size_t aplane, int rm) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP, NS = KF / 4, KK = HD / KSTEP, HT = HD / 16;
    static_assert(KW == 2 || KW == 4 || KW == 8, "waves per tile");
    __shared__ f32x4 mo[ROWS_WAVES][HT][64];
    __shared__ float mm[ROWS_WAVES][64], ml[ROWS_WAVES][64];
    // Workgroups are handed to the 8 XCDs (each with an L2 of its own) round robin: those of one (sequence, kv head) are 8
    // apart, so its keys and values come from HBM once.  Among them a prompt chunk's last tiles, which see the most keys, go first.
    const int tile0 = q0 * md.G / 16;                  // the first tile with a position that is wanted
    const int groups = ((ntiles - tile0) * KW + ROWS_WAVES - 1) / ROWS_WAVES, at = blockIdx.x >> 3;
    const int pair = at / groups * 8 + (blockIdx.x & 7), grp = groups - 1 - at % groups;
    if (pair >= sp->nseq * md.Hkv) return;             // padding of the grid to whole XCD rounds (uniform)
    const int rps = sp->rps, bi = pair / md.Hkv, b = sp->seq_base + bi, L = kv.len[b], cap = kv.cap[b], kvh = pair - bi * md.Hkv;
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), ks = w % KW;
    const int tile = tile0 + grp * (ROWS_WAVES / KW) + w / KW;
    const bool live = tile < ntiles;                   // waves of a tile past the end only take part in the barrier
    const T* Kb = kv.K + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * cap * HD;
    const T* Vb = kv.V + (size_t)layer * kv.layer_stride + kv.seq_off[b] + (size_t)kvh * HD * cap;

    // column of the tile: position m / G, head m % G, m = tile * 16 + r
    const int m = min(tile, ntiles - 1) * 16 + r, jrow = small_div(m, md.G), girow = m - jrow * md.G;
    const bool rowvalid = live && jrow < rps && jrow >= q0;
    const int jmax = min(small_div(min(tile, ntiles - 1) * 16 + 15, md.G), rps - 1);
    const int key_hi = live ? min(L + jmax + 1, cap) : 0;      // keys this tile's rows can see
    Frag qf[KK][SPL];
    {
        const u32x4* q = qbuf + (((size_t)bi * md.Hkv + kvh) * ntiles + min(tile, ntiles - 1)) * KK * SPL * 64 + lane;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int pl = 0; pl < SPL; ++pl) qf[kk][pl].u = q[(kk * SPL + pl) * 64];
    }

    Frag kf[2][NS][KK], vf[2][HT];
    auto load_keys = [&](int set, int key) {           // any whole step: clamped to the cache
        key = min(key, cap - KSTEP);
        const T *kb = Kb + (size_t)key * HD + lane * KF, *vb = Vb + (size_t)key * HD + lane * KF;
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kf[set][t][kk].u = *reinterpret_cast<const u32x4*>(kb + (t * KK + kk) * 64 * KF);
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) vf[set][ht].u = *reinterpret_cast<const u32x4*>(vb + ht * 64 * KF);
    };

    f32x4 o[HT];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int ht = 0; ht < HT; ++ht) o[ht] = f32x4{0.f, 0.f, 0.f, 0.f};
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
        f32x4 s[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int pl = 0; pl < SPL; ++pl) Traits<T>::mma(kf[set][t][kk], qf[kk][pl], s[t]);
        }
        Frag pf[SPL];
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = rowvalid && key0 + KF * g + 4 * t + i <= L + jrow ? s[t][i] * md.scale : -INFINITY;
                s[t][i] = v;
                mx = fmaxf(mx, v);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const bool dead = (m_new == -INFINITY);
        const float alpha = dead ? 1.f : __expf(m_run - m_new);
        float psum = 0.f;
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = dead ? 0.f : __expf(s[t][i] - m_new);
                psum += p;
                Traits<T>::template pack_split<SPL>(pf, 4 * t + i, p);
            }
        l_run = l_run * alpha + psum;
        m_run = m_new;
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) {
            o[ht] *= alpha;
#pragma unroll
            for (int pl = 0; pl < SPL; ++pl) Traits<T>::mma(vf[set][ht], pf[pl], o[ht]);
        }
    };
    // this wave's steps: ks, ks + KW, ..; the next one is requested before the current one is used
    constexpr int STRIDE = KW * KSTEP;
    int key0 = ks * KSTEP;
    load_keys(0, key0);
    while (key0 + STRIDE < key_hi) {
        load_keys(1, key0 + STRIDE);
        step(0, key0);
        load_keys(0, key0 + 2 * STRIDE);               // may lie past this tile's keys: in bounds, unused then
        step(1, key0 + STRIDE);
        key0 += 2 * STRIDE;
    }
    if (key0 < key_hi) step(0, key0);

    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    // merge of the KW waves of a tile, in wave order; wave ks of them finishes head tiles ks, ks + KW, ..
#pragma unroll
    for (int ht = 0; ht < HT; ++ht) mo[w][ht][lane] = o[ht];
    mm[w][lane] = m_run;
    ml[w][lane] = l_run;
    __syncthreads();
    const int w0 = w - ks;
    float mn = -INFINITY, l = 0.f, f[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) mn = fmaxf(mn, mm[w0 + k][lane]);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        const float mk = mm[w0 + k][lane];
        f[k] = (mk == -INFINITY) ? 0.f : __expf(mk - mn);
        l += f[k] * ml[w0 + k][lane];
    }
    if (!rowvalid) return;
    const float inv = 1.f / l;
#pragma unroll
    for (int h = 0; h < HT; h += KW) {
        const int ht = h + ks;
        if (ht >= HT) break;                           // uniform
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KW; ++k) acc += mo[w0 + k][ht][lane] * f[k];
        const float v[4] = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
        Traits<T>::template store_split4<SPL>(attn_out + opnd_off<T>(bi * (rps - q0) + jrow - q0, (kvh * md.G + girow) * HD + ht * 16 + 4 * g, md.Hq * HD, rm), aplane, v);
    }
}

}  // namespace sj
