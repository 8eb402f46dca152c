// Gate / up projection of many rows on large tiles (bf16, two operand planes): silu(gate) * up of X[R][K] * W[N][K]^T with W in the
// re-tiled layout.  Paper reference: the MLP of the target forward, Eq. 2 / Eq. 4.
//
// What bounds the loader-wave kernel (sj_gemm_rows.h) with several row groups: its 128 rows x 7 or 8 n-tiles fetch 23 - 24 KB a k-step for
// 128 products of a SIMD - L2 and LDS traffic above what either delivers beside the matrix cores - and its tiles come in four rounds
// with a prologue and an epilogue each.  Here a workgroup owns up to 256 rows x 16 n-tiles: both planes of a row tile meet in one
// accumulator, so 48 KB a k-step feed 512 products of a SIMD, and a 509-row chunk of the 8B shape is one round of the chip.
//  * Eight waves, two to a SIMD; a wave owns half of the row tiles x 4 n-tiles (4 waves of twice that: 264 us where this form takes 238).
//    No loader waves: every wave requests its share of a stage (one k-step, weights and operand) straight into LDS, NS stages deep.
//  * A row tile's fragments are read from LDS two row tiles ahead of their products, and the stage's barrier falls between its last read
//    and the products of its last two row tiles; sched_barrier keeps the compiler from moving the reads next to their use, where
//    every one is waited for (297 -> 259 us; two ahead instead of one 245 -> 238).
//  * A workgroup takes every TILE_WGS-th tile; its requests run over the end of a tile into the next one.
// Measured (8B shape, N = 28672, K = 4096, 509 rows, back to back): 298 -> 238 us = 1.0 PFLOP/s; other sizes at tile_rows.  The chip then
// runs at 1.7 GHz instead of 2.4 (power: with zeros for an operand the same launch takes 207 us at 2.0 GHz), 71 % of those cycles
// are products.  32x32x16 products instead of 16x16x32: 259 us, at a lower clock still.
#pragma once
#include "sj_gemm_rows.h"

namespace sj {

constexpr int TILE_WAVES = 8;

// RT row tiles to a row group, NS stages of RT * SPL + 16 KB in LDS (up to 160 KB)
// (EPI_LOGITS: a statistic per row and wave, that is per TILE_STAT n-tiles, in a.stats [R][ntiles / TILE_STAT])
template <typename T, int EPI, int SPL, int RT, int NS>
__global__ __launch_bounds__(TILE_WAVES * 64) void gemm_tile_kernel(GemmArgs a) {
    static_assert(RT >= 4 && std::is_same<T, bf16_t>::value, "two halves of at least two row tiles");
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP, NT = TILE_NT, WAVES = TILE_WAVES;
    constexpr int WR = 2, WN = WAVES / WR, NTW = NT / WN;
    static_assert(NTW == TILE_STAT, "n-tiles of a wave");
    constexpr int NX = RT * SPL, NF = NX + NT, PER = (NF + WAVES - 1) / WAVES;      // fragments of a stage, requests of a wave
    static_assert(NS >= 3 && NS * PER < 64, "the load counter holds 63");
    __shared__ u32x4 st[NS][NF][64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.K / KSTEP, ntiles = a.N / 16, ngroups = (ntiles + NT - 1) / NT, rtiles = (a.R + 15) / 16;
    // Workgroups are handed to the 8 XCDs round robin by index.  An XCD takes every eighth n-tile group, its workgroups the row groups
    // of one n-tile group, then the next: the weights come from HBM once and are found in that XCD's L2 by the others.
    const int xcd = blockIdx.x & 7, slots = gridDim.x >> 3;
    const int half = w / WN, m0 = half * ((RT + 1) / 2), t0 = w % WN * NTW;      // an odd number of row tiles: the first half has one more
    auto group_of = [&](int j) { return j / a.rgroups * 8 + xcd; };

    // what is requested next: k-step lk of tile lj; past the last tile its k-steps again (in bounds, never used)
    int lj = blockIdx.x >> 3, lk = 0;
    if (group_of(lj) >= ngroups) return;               // uniform
    const char* src[PER];
    auto aim = [&](int j) {
        const int nt0 = group_of(j) * NT, rt0 = j % a.rgroups * RT;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int f = min(w + WAVES * q, NF - 1);
            if (f < NX) {                              // tiles past the rows repeat the last one: multiplied, never stored
                const T* plane = reinterpret_cast<const T*>(a.X) + (size_t)(f % SPL) * a.xplane;
                src[q] = reinterpret_cast<const char*>(plane + ((size_t)min(rt0 + f / SPL, rtiles - 1) * KS * 64 + lane) * KF);
            } else {
                src[q] = reinterpret_cast<const char*>(a.Wt) + ((size_t)min(nt0 + f - NX, ntiles - 1) * KS * 64 + lane) * 16;
            }
        }
    };
    aim(lj);
    auto issue = [&](int buf) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[q] + (size_t)lk * 1024),
                                             (__attribute__((address_space(3))) void*)&st[buf][min(w + WAVES * q, NF - 1)][0], 16, 0, 0);
        if (++lk == KS) {
            lk = 0;
            if (group_of(lj + slots) < ngroups) { lj += slots; aim(lj); }
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) issue(s);

    // everything behind the first requests, for a wave with RTW row tiles
    auto work = [&](auto rtw_tag) {
        constexpr int RTW = decltype(rtw_tag)::value;
        f32x4 acc[RTW][NTW];
        Frag wf[2][NTW], bq[3][SPL];
        auto fetch_w = [&](Frag& f, int buf, int t) { f.u = st[buf][NX + t0 + t][lane]; };
        auto fetch_x = [&](Frag (&f)[SPL], int buf, int i) {
#pragma unroll
            for (int p = 0; p < SPL; ++p) f[p].u = st[buf][(m0 + i) * SPL + p][lane];
        };
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 1) * PER));            // stage 0 has landed
        lds_barrier();
#pragma unroll
        for (int t = 0; t < NTW; ++t) fetch_w(wf[0][t], 0, t);
        fetch_x(bq[0], 0, 0);
        fetch_x(bq[1], 0, 1);
        int buf = 0;
        // One k-step.  At its barrier every wave has read the whole stage (its buffer takes the requests of NS stages on) and the next
        // stage has landed: at most NS - 2 stages of this wave's requests are still in flight.
        auto step = [&](auto par_tag) {
            constexpr int PAR = decltype(par_tag)::value;
            const int nbuf = buf + 1 == NS ? 0 : buf + 1;
#pragma unroll
            for (int i = 0; i < RTW; ++i) {
                if (i + 2 < RTW) fetch_x(bq[(i + 2) % 3], buf, i + 2);
                else if (i + 2 == RTW) {
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * PER));
                    lds_barrier();
                    fetch_x(bq[(i + 2) % 3], nbuf, 0);
#pragma unroll
                    for (int t = 0; t < NTW / 2; ++t) fetch_w(wf[PAR ^ 1][t], nbuf, t);
                } else {
                    fetch_x(bq[(i + 2) % 3], nbuf, 1);
#pragma unroll
                    for (int t = NTW / 2; t < NTW; ++t) fetch_w(wf[PAR ^ 1][t], nbuf, t);
                    issue(buf);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < NTW; ++t)
#pragma unroll
                    for (int p = 0; p < SPL; ++p) Traits<T>::mma(wf[PAR][t], bq[i % 3][p], acc[i][t]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (RTW % 3 != 0) {                  // the next stage's first two row tiles to where it starts
                Frag n0[SPL], n1[SPL];
#pragma unroll
                for (int p = 0; p < SPL; ++p) { n0[p] = bq[RTW % 3][p]; n1[p] = bq[(RTW + 1) % 3][p]; }
#pragma unroll
                for (int p = 0; p < SPL; ++p) { bq[0][p] = n0[p]; bq[1][p] = n1[p]; }
            }
            buf = nbuf;
        };
        for (int j = blockIdx.x >> 3; group_of(j) < ngroups; j += slots) {              // uniform
#pragma unroll
            for (int i = 0; i < RTW; ++i)
#pragma unroll
                for (int t = 0; t < NTW; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int s = 0; s < KS; s += 2) {              // K is a multiple of 64: whole pairs of k-steps
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
            }
            const int nt0 = group_of(j) * NT + t0, rt0 = j % a.rgroups * RT + m0;
            if constexpr (EPI == EPI_LOGITS) {
                const int nv = min(NTW, ntiles - nt0);       // n-tiles of this wave that exist
#pragma unroll
                for (int i = 0; i < RTW; ++i) {
                    const int row = (rt0 + i) * 16 + r;
                    if (nv <= 0 || m0 + i >= RT || rt0 + i >= rtiles) continue;        // uniform
                    float4 stat = rows_softmax_stat<NTW>(acc[i], nt0, nv, a.inv_temp, g);
                    if (!(stat.y > 0.f)) stat.y = 0.f;       // (columns that are all infinite leave no sum, as with the loader waves)
                    if (row >= a.R) continue;
                    if (g == 0) a.stats[(size_t)row * (ntiles / TILE_STAT) + nt0 / TILE_STAT] = stat;
#pragma unroll
                    for (int t = 0; t < NTW; ++t)
                        if (t < nv) *reinterpret_cast<f32x4*>(a.out + (size_t)row * a.N + (size_t)(nt0 + t) * 16 + 4 * g) = acc[i][t];
                }
            } else {
#pragma unroll
                for (int t = 0; t < NTW; ++t)
#pragma unroll
                    for (int i = 0; i < RTW; ++i)
                        if (nt0 + t < ntiles && rt0 + i < rtiles) rows_epilogue_tile<T, EPI, SPL>(a, acc[i][t], rt0 + i, nt0 + t, r, g);
            }
        }
    };
    if constexpr (RT % 2 == 0) work(std::integral_constant<int, RT / 2>{});
    else if (half == 0) work(std::integral_constant<int, (RT + 1) / 2>{});       // (the two halves meet at the same barriers: one a k-step)
    else work(std::integral_constant<int, RT / 2>{});
    wait_vm0();                                        // the requests past the last tile
}

}  // namespace sj
