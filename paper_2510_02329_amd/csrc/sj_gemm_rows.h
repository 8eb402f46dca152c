// Weight-streaming GEMM for more than two row tiles (batched verification, scoring, prompt chunks: more than 32 rows, in row groups of
// 64 - 288): Y[R][N] = X[R][K] * W[N][K]^T with W in the re-tiled layout.
// Paper reference: the projections of the target forward, Eq. 2 / Eq. 4.
//
// With many rows the few-row kernel's scheme (every wave fetches the operand fragments of all rows
// for its own K-slice) makes the operand the dominant traffic, and every weight byte should still be
// read once.  Measured facts that shaped this kernel:
//  * a wave's loads return in order, so a wave that requests weights (HBM, ~2 us) and operand
//    (L2, < 1 us) can never consume the operand before the weights requested ahead of it arrive -
//    mixing the two streams in one wave ties the short latency to the long one;
//  * a barrier that also waits for global loads keeps all waves in lock step with the slowest weight load;
//  * compute waves that load operand fragments themselves run at the sum of weight stream and MFMA time, without those loads at their
//    maximum, and a row-major operand fragment touches 16 cache lines of which it uses half.
// So LOADER waves move weight tiles and operand fragments straight from global memory into LDS rings, from planes that the
// producing kernels wrote as fragments (opnd_off: 1 KB of consecutive memory each), and COMPUTE waves issue no global loads at all.
// No cross-wave reduction is needed: the epilogue runs straight from the accumulators.  Split-K across workgroups (gridDim.y slices,
// partials summed by the consumer in slice order) keeps the short projections on all CUs.
//
// MFMA convention as in the few-row kernel: A = weight fragment (rows = n), B = operand fragment
// (rows = m), lane 16g + r then holds D[n = 4g + i][m = r].
#pragma once
#include <type_traits>

#include "sj_kernels.h"
#include "sj_plan.h"

namespace sj {

constexpr int ROWS_NT = 8;         // n-tiles per workgroup

// Softmax partial (max, sum exp((l - max)/T), lowest arg-max) of a row over `n` <= NTILES neighbouring n-tiles from nt on: the row's four
// lanes hold four columns of each tile; all of them get the result.
template <int NTILES>
__device__ __forceinline__ float4 rows_softmax_stat(const f32x4* v, int nt, int n, float inv_temp, int g) {
    float mx = v[0][0];
    int arg = nt * 16 + 4 * g;
#pragma unroll
    for (int t = 0; t < NTILES; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (t < n && v[t][e] > mx) { mx = v[t][e]; arg = (nt + t) * 16 + 4 * g + e; }
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
        const float omx = __shfl_xor(mx, o, 64);
        const int oarg = __shfl_xor(arg, o, 64);
        if (omx > mx || (omx == mx && oarg < arg)) { mx = omx; arg = oarg; }
    }
    float se = 0.f;
    if (inv_temp > 0.f) {
#pragma unroll
        for (int t = 0; t < NTILES; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) se += t < n ? expf((v[t][e] - mx) * inv_temp) : 0.f;
        se += __shfl_xor(se, 16, 64);
        se += __shfl_xor(se, 32, 64);
    }
    return float4{mx, se, __int_as_float(arg), 0.f};
}

// Epilogue of partial sums and SwiGLU for ONE accumulator tile (row tile m, n-tile nt): the lane holds columns
// nt*16 + 4g .. +3 of row m*16 + r.  Uniform per wave; rows >= R take part in the shuffles and store nothing.
template <typename T, int EPI, int SPL>
__device__ __forceinline__ void rows_epilogue_tile(const GemmArgs& a, const f32x4& v, int m, int nt, int r, int g) {
    const int row = m * 16 + r;
    const bool valid = row < a.R;
    if constexpr (EPI == EPI_PARTIAL) {
        if (valid)
            *reinterpret_cast<f32x4*>(a.out + ((size_t)blockIdx.y * a.slice_rows + row) * a.N + (size_t)nt * 16 + 4 * g) = v;
    } else if constexpr (EPI == EPI_SWIGLU) {
        // tile rows 0-7 are gate of FFN columns 8*nt .. 8*nt+7, rows 8-15 their up projections:
        // the up value of this lane's gate sits two lane groups further
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float up = __shfl_down(v[e], 32, 64);
            const float gate = v[e];
            y[e] = gate / (1.0f + expf(-gate)) * up;
        }
        if (valid && g < 2)
            Traits<T>::template store_split4<SPL>(reinterpret_cast<T*>(a.act) + opnd_off<T>(row, nt * 8 + 4 * g, a.N / 2), a.actplane, y);
    }
}

// ---------------------------------------------------------------------------------------------
// A stage is ONE k-step; a wave's loads come back in the order it issued them, so weights (HBM: 8 stages of 8 KB) and operand (an L2
// hit: 5 stages of RT x SPL KB) are fetched by different loader waves with rings of their own; one barrier per k-step;
// the compute waves read the fragments of step s + 1 from LDS while they multiply step s.  An
// operand fragment in LDS has the layout the lanes read it in (lane l: 16 bytes at l * 16), which is
// also how a direct global->LDS load of 16 bytes per lane deposits it.
constexpr int R4_NSW = 8;          // weight stages (k-steps) in LDS: HBM latency to cover
constexpr int R4_NSX = 5;          // operand stages: an L2 hit away
constexpr int R4_LW = 4;           // loader waves: two for the weights, two for the operand

// NT = n-tiles per workgroup: 8, or 7 where that makes the number of workgroups a multiple of the CU count
// (gate/up projection of the 8B shape: 1792 n-tiles = 256 x 7).
// Several row groups in ONE launch (a.rgroups > 1): the weights should come from HBM once for all of them, so the
// workgroups that share an n-tile group must run at the same time on compute units that share a cache.  Workgroups
// are handed to the 8 XCDs (each with an L2 of its own) round robin by index, so workgroup i works for XCD i % 8;
// within an XCD consecutive workgroups take the row groups of one n-tile group, then the next n-tile group: the first
// of them pulls a weight tile from HBM, the others find it in their L2 a moment later.
//
// EIGHT compute waves with an even split of the 9 x NT accumulator tiles: wave w = (a = w % 4, b = w / 4) owns row tiles
// a and a + 4 for the n-tiles of half b, and n-tile w of row tile 8: 9 tiles each for NT = 8 (8 / 8 / 8 / 8 / 7 / 7 / 7 / 6
// for NT = 7), 36 accumulator registers, two compute waves per SIMD.  An earlier form with four compute waves (row tiles
// w, w + 4, w + 8: one wave with three) measured the same on two-plane operands, where the L2 traffic of the operand sets
// the pace, and 12 % slower on the one-plane LM head of the verify-head workload (909 -> 799 us).
constexpr int R8_CW = 8;

// RT = row tiles of a row group: up to 9 (144 rows) with two operand planes or fp32, 6 with three, 18 with a single bf16 plane (288
// rows: the same 18 operand fragments per k-step in LDS, half as many workgroups re-reading every weight tile through L2).  A wave owns RT / 4
// whole row tiles for its half of the n-tiles and n-tile w of each of the RT % 4 tiles left over.  Every tile of the group is
// fetched and multiplied whether it has rows or not, so the group is chosen to fit the rows (row_tiles in sj_plan.h).
template <typename T, int EPI, int SPL, int NT = ROWS_NT, int RT = ROWS_MT>
__global__ __launch_bounds__((R8_CW + R4_LW) * 64) void gemm_rows8_kernel(GemmArgs a, int mt) {
    static_assert(NT == 7 || NT == 8, "n-tile halves are 4 + 4 or 4 + 3");
    static_assert(RT * SPL <= 2 * ROWS_MT, "the operand stages in LDS hold 18 fragments");
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP;
    constexpr int NX = RT * SPL;                       // operand fragments per stage
    constexpr int NFULL = RT / 4, NREM = RT % 4;       // whole row tiles per wave; tiles shared out by n-tile
    __shared__ u32x4 Wst[R4_NSW][NT][64];
    __shared__ u32x4 Xst[R4_NSX][NX][64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.K / KSTEP, ntiles = a.N / 16;
    int bx = blockIdx.x;
    if (a.rgroups > 1) {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
        const int rg = j % a.rgroups;
        bx = (j / a.rgroups) * 8 + xcd;
        if (bx * NT >= ntiles) return;                 // padding of the grid to whole XCD rounds (uniform)
        const int row0 = rg * (RT * 16), nr = min(RT * 16, a.R - row0);
        a.X = reinterpret_cast<const char*>(a.X) + (size_t)row0 * a.K * sizeof(T);
        if (EPI == EPI_SWIGLU) a.act = reinterpret_cast<char*>(a.act) + (size_t)row0 * (a.N / 2) * sizeof(T);
        else a.out += (size_t)row0 * a.N;
        if (EPI == EPI_LOGITS) a.stats += (size_t)row0 * ((ntiles + NT - 1) / NT);
        a.R = nr;
        mt = (nr + 15) / 16;
    }
    const int nt0 = bx * NT;
    const int ks0 = (int)((long long)blockIdx.y * KS / gridDim.y), ks1 = (int)((long long)(blockIdx.y + 1) * KS / gridDim.y);
    const int nks = ks1 - ks0;
    if (nks <= 0) return;                              // uniform for the workgroup

    if (w >= R8_CW) {
        // ---------------- loader waves ----------------
        // A wave's loads come back in the order it issued them, so the weights (HBM, deep ring) and the operand (L2, shallow
        // ring) are fetched by different waves.  Stage = k-step of the slice (clamped: a stage past the end re-reads the last
        // one into its own buffer).  The compute waves read stage s + 1 while they multiply stage s, so stage s + 2 has to be
        // in LDS when iteration s ends: NS - 3 stages of a loader wave's loads may still be in flight.
        const int lw = w - R8_CW;
        auto run = [&](auto nl_tag, auto ns_tag, auto aux_tag, auto make_src, auto dst_of) {
            constexpr int NL = decltype(nl_tag)::value, NS = decltype(ns_tag)::value, AUX = decltype(aux_tag)::value;
            const char* src[NL];
            size_t step[NL];
#pragma unroll
            for (int j = 0; j < NL; ++j) make_src(j, src[j], step[j]);
            auto issue = [&](int s) {
                const size_t k = (size_t)min(s, nks - 1);
#pragma unroll
                for (int j = 0; j < NL; ++j)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + k * step[j]),
                                                     (__attribute__((address_space(3))) void*)dst_of(s % NS, j), 16, 0, AUX);
            };
            constexpr int BEHIND = (NS - 3) * NL;
            static_assert((NS - 1) * NL < 64, "the load counter holds 63");
#pragma unroll
            for (int s = 0; s < NS - 1; ++s) issue(s);
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(BEHIND));            // stages 0 and 1 have landed
            lds_barrier();
            for (int s = 0; s < nks; ++s) {
                issue(s + NS - 1);
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(BEHIND));        // stage s + 2 has landed
                lds_barrier();
            }
            wait_vm0();
            if constexpr (EPI == EPI_LOGITS) { lds_barrier(); lds_barrier(); }   // the statistics' barriers
        };
        if (lw < 2) {
            auto make_src = [&](int j, const char*& sp, size_t& st) {
                const size_t tile = (size_t)min(nt0 + min(lw + 2 * j, NT - 1), ntiles - 1);
                sp = reinterpret_cast<const char*>(a.Wt) + ((tile * KS + ks0) * 64 + lane) * 16;
                st = 1024;
            };
            auto dst_of = [&](int buf, int j) { return &Wst[buf][min(lw + 2 * j, NT - 1)][0]; };
            if (a.rgroups > 1)
                run(std::integral_constant<int, (NT + 1) / 2>{}, std::integral_constant<int, R4_NSW>{}, std::integral_constant<int, 0>{}, make_src, dst_of);
            else
                run(std::integral_constant<int, (NT + 1) / 2>{}, std::integral_constant<int, R4_NSW>{}, std::integral_constant<int, 2>{}, make_src, dst_of);
        } else {
            const int x = lw - 2;
            auto make_src = [&](int j, const char*& sp, size_t& st) {
                const int it = min(x + 2 * j, NX - 1);
                const int m = it / SPL, p = it % SPL;
                const T* plane = reinterpret_cast<const T*>(a.X) + (size_t)p * a.xplane;
                const size_t mt_ok = m * 16 < a.R ? m : 0;
                sp = reinterpret_cast<const char*>(plane + ((mt_ok * KS + ks0) * 64 + lane) * KF);
                st = 1024;
            };
            auto dst_of = [&](int buf, int j) { return &Xst[buf][min(x + 2 * j, NX - 1)][0]; };
            run(std::integral_constant<int, (NX + 1) / 2>{}, std::integral_constant<int, R4_NSX>{}, std::integral_constant<int, 0>{}, make_src, dst_of);
        }
        return;
    }

    // ---------------- compute waves ----------------
    const int ra = w & 3, nb = w >> 2;                 // row tiles ra, ra + 4; n-tiles of half nb; n-tile w of row tile 8
    constexpr int NH = 4;                              // n-tiles of half 0 (half 1 has NT - 4)
    const int t0 = nb * NH, nh = nb == 0 ? NH : NT - NH;
    f32x4 acc[NFULL][NH], acc8[NREM ? NREM : 1];
#pragma unroll
    for (int i = 0; i < NFULL; ++i)
#pragma unroll
        for (int t = 0; t < NH; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NREM; ++j) acc8[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Where the products are exact to 24 bits, the rounding of the running sums is the error: the accumulators are added to totals of
    // their own every FOLD k-steps, so that a sum is a chain of short chains, as it is in the few-row kernels, whose waves share K
    // (fp32, K = 1024 / 8192: rms error against 64 bits 3.7e-7 / 2.9e-6 in one chain, 1.0e-7 / 4.6e-7 folded, 1.9e-7 / 1.5e-6 in the
    // few-row kernels; three planes, K = 4096: of 1.1 M stored K / V elements 560 round away from the 64-bit value's neighbour in one
    // chain, 304 folded, 281 in the few-row kernels).  It takes 1 - 2 % of a step of 33 - 144 rows.  With one or two bf16 planes the
    // operand's rounding (2^-9, 2^-18) is above that of the sums.
    constexpr int FOLD = std::is_same<T, float>::value ? 4 : SPL == 3 ? 8 : 0;
    f32x4 tot[FOLD ? NFULL : 1][NH], tot8[FOLD && NREM ? NREM : 1];
    auto fold = [&](bool first) {
#pragma unroll
        for (int i = 0; i < NFULL; ++i)
#pragma unroll
            for (int t = 0; t < NH; ++t) {
                tot[i][t] = first ? acc[i][t] : tot[i][t] + acc[i][t];
                acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
        for (int j = 0; j < NREM; ++j) {
            tot8[j] = first ? acc8[j] : tot8[j] + acc8[j];
            acc8[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    if constexpr (FOLD > 0) fold(true);

    // The k-steps of a wave with NHW n-tiles in its half.  No predicate in the k-step: a row tile past the rows (tile 0 again) is multiplied into an
    // accumulator that the epilogue never stores.  The second half of seven n-tiles has a loop of its own: its waves multiplied a fourth
    // tile for nothing, and these kernels run at the clock that their products and fetches leave (1.5 - 2.3 of 2.4 GHz).
    auto k_steps = [&](auto nhw_tag) {
        constexpr int NHW = decltype(nhw_tag)::value;
        struct Frags { Frag wf[NHW]; Frag w8; Frag bq[NFULL + NREM][SPL]; };
        Frags fA, fB;
        auto fetch = [&](Frags& f, int s) {
            const u32x4* Xs = &Xst[s % R4_NSX][0][0];
            const u32x4* Ws = &Wst[s % R4_NSW][0][0];
#pragma unroll
            for (int sp = 0; sp < SPL; ++sp) {
#pragma unroll
                for (int i = 0; i < NFULL; ++i) f.bq[i][sp].u = Xs[((ra + 4 * i) * SPL + sp) * 64 + lane];
#pragma unroll
                for (int j = 0; j < NREM; ++j) f.bq[NFULL + j][sp].u = Xs[((4 * NFULL + j) * SPL + sp) * 64 + lane];
            }
#pragma unroll
            for (int t = 0; t < NHW; ++t) f.wf[t].u = Ws[(t0 + t) * 64 + lane];
            f.w8.u = Ws[min(w, NT - 1) * 64 + lane];
        };
        auto multiply = [&](const Frags& f) {
#pragma unroll
            for (int sp = 0; sp < SPL; ++sp) {
#pragma unroll
                for (int t = 0; t < NHW; ++t)
#pragma unroll
                    for (int i = 0; i < NFULL; ++i) Traits<T>::mma(f.wf[t], f.bq[i][sp], acc[i][t]);
#pragma unroll
                for (int j = 0; j < NREM; ++j) Traits<T>::mma(f.w8, f.bq[NFULL + j][sp], acc8[j]);
            }
        };
        lds_barrier();                                     // stages 0 and 1 are in LDS
        fetch(fA, 0);
        for (int s = 0; s < nks; s += 2) {
            fetch(fB, s + 1);
            multiply(fA);
            lds_barrier();                                 // stage s + 2 has landed
            if (s + 1 < nks) {                             // uniform
                fetch(fA, s + 2);
                multiply(fB);
                lds_barrier();                             // stage s + 3 has landed
            }
            if constexpr (FOLD > 0) {
                if ((s + 2) % FOLD == 0) fold(false);      // uniform
            }
        }
    };
    if constexpr (NT == 2 * NH) k_steps(std::integral_constant<int, NH>{});
    else if (nb == 0) k_steps(std::integral_constant<int, NH>{});
    else k_steps(std::integral_constant<int, NT - NH>{});
    if constexpr (FOLD > 0) {
#pragma unroll
        for (int i = 0; i < NFULL; ++i)
#pragma unroll
            for (int t = 0; t < NH; ++t) acc[i][t] += tot[i][t];
#pragma unroll
        for (int j = 0; j < NREM; ++j) acc8[j] += tot8[j];
    }
    if constexpr (EPI == EPI_LOGITS) {
        // Logits, and ONE softmax partial per row and workgroup: a partial per n-tile (16 bytes for 64 bytes of logits) was 74 MB
        // to write and to read again for the 576 rows of a 64-sequence batch (merge launch 41 us, now a tenth of the bytes).
        // A wave reduces its n-tiles of a row in registers; the waves' partials meet in the ring's memory.
        static_assert(NT == 8, "two halves of four n-tiles");
        constexpr int HALVES = 2;
        float4* st_full = reinterpret_cast<float4*>(&Wst[0][0][0]);      // [4 * NFULL row tiles][half][16 rows]
        float4* st_rem = st_full + 4 * NFULL * HALVES * 16;              // [NREM][8 waves][16 rows]
        static_assert((4 * NFULL * HALVES + NREM * R8_CW) * 16 * sizeof(float4) <= sizeof(Wst), "fits the weight ring");
        lds_barrier();                                 // the loaders' last requests have landed, every fragment has been read
        const int nv = min(nh, ntiles - (nt0 + t0));   // n-tiles of this wave's half that exist
#pragma unroll
        for (int i = 0; i < NFULL; ++i) {
            const int m = ra + 4 * i, row = m * 16 + r;
            if (m >= mt) continue;                     // uniform
            float4 st = float4{-INFINITY, 0.f, __int_as_float(0x7fffffff), 0.f};
            if (nv > 0) st = rows_softmax_stat<NH>(acc[i], nt0 + t0, nv, a.inv_temp, g);
            if (g == 0) st_full[(m * HALVES + nb) * 16 + r] = st;
            if (row < a.R)
#pragma unroll
                for (int t = 0; t < NH; ++t)
                    if (t < nv) *reinterpret_cast<f32x4*>(a.out + (size_t)row * a.N + (size_t)(nt0 + t0 + t) * 16 + 4 * g) = acc[i][t];
        }
#pragma unroll
        for (int j = 0; j < NREM; ++j) {
            const int m = 4 * NFULL + j, row = m * 16 + r;
            if (m >= mt) continue;
            float4 st = float4{-INFINITY, 0.f, __int_as_float(0x7fffffff), 0.f};
            if (nt0 + w < ntiles) {
                st = rows_softmax_stat<1>(&acc8[j], nt0 + w, 1, a.inv_temp, g);
                if (row < a.R) *reinterpret_cast<f32x4*>(a.out + (size_t)row * a.N + (size_t)(nt0 + w) * 16 + 4 * g) = acc8[j];
            }
            if (g == 0) st_rem[(j * R8_CW + w) * 16 + r] = st;
        }
        lds_barrier();
        for (int row = tid; row < a.R; row += R8_CW * 64) {
            const int m = row >> 4, rr = row & 15;
            const bool full = m < 4 * NFULL;
            const float4* p = full ? st_full + m * HALVES * 16 + rr : st_rem + (m - 4 * NFULL) * R8_CW * 16 + rr;
            const int n = full ? HALVES : R8_CW;
            float4 s = p[0];
            for (int k = 1; k < n; ++k) {              // ascending columns: an equal maximum keeps the lower index
                const float4 o = p[k * 16];
                if (o.x > s.x) { s.x = o.x; s.z = o.z; }
            }
            float se = 0.f;
            if (a.inv_temp > 0.f)
                for (int k = 0; k < n; ++k) {
                    const float4 o = p[k * 16];
                    if (o.y > 0.f) se += o.y * expf((o.x - s.x) * a.inv_temp);
                }
            a.stats[(size_t)row * ((ntiles + NT - 1) / NT) + bx] = float4{s.x, se, s.z, 0.f};
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < NH; ++t) {
        if (t >= nh || nt0 + t0 + t >= ntiles) continue;   // uniform
#pragma unroll
        for (int i = 0; i < NFULL; ++i)
            if (ra + 4 * i < mt) rows_epilogue_tile<T, EPI, SPL>(a, acc[i][t], ra + 4 * i, nt0 + t0 + t, r, g);
    }
    if (w < NT && nt0 + w < ntiles) {
#pragma unroll
        for (int j = 0; j < NREM; ++j)
            if (4 * NFULL + j < mt) rows_epilogue_tile<T, EPI, SPL>(a, acc8[j], 4 * NFULL + j, nt0 + w, r, g);
    }
}

}  // namespace sj
