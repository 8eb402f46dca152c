// Few-row weight-streaming GEMM with the weights delivered through LDS, every wave keeping a ring of its own: Y[R][N] = X[R][K] * W[N][K]^T,
// R <= 16 MT (MT = 1 or 2 row tiles), W in the re-tiled layout (paper: the projections of the target forward, Eq. 2 / Eq. 4).  Same
// arguments, grid meaning (x: groups of NT n-tiles, y: K-slices) and epilogues as gemm_skinny_kernel, whose loads go to registers.
//
// Eight waves interleave K: wave w multiplies k-steps ks0 + 8 kb + w of the slice, so the workgroup pulls 8 KB of consecutive memory per tile
// and k-block.  Everything a wave multiplies - NT weight fragments and the operand fragments (one packed, or MT x planes) of its k-step - comes
// by direct global->LDS loads into DEPTH fragments of 1 KB of LDS that no other wave touches: a k-block that the wave has read into registers
// makes room at once for the fragments DEPTH places on, and the only wait is the wave's own count of loads.  No barrier before the reduction,
// no loader waves.  The 8 waves' accumulators meet in LDS (the rings' memory, free by then) and are added in wave order: deterministic, and the
// same sums for every NT and DEPTH.
//
// What bounds it: the stream, and the 3 - 4 us that a launch spends before its first fragment and after its last.  us a launch, back to back on
// rotating weights, before (two loader waves feeding a workgroup-wide ring of 8 KB stages, one barrier a stage; above 8 rows the
// register-ring kernel) and now: 8B shape, 6 rows: gate / up 39.2 -> 37.4 (6.3 TB/s), QKV 10.6 -> 10.2, O 8.9 -> 8.5, down 22.0 -> 22.0,
// LM head 172 -> 164 (6.4); 20 rows: gate / up 43.0 -> 39.0, QKV 12.8 -> 11.4, down 23.5 -> 21.6, LM head 201 -> 191; 1B, 1 row: gate / up
// 14.1 -> 13.0, QKV 5.6 -> 4.9, O 5.2 -> 4.7, LM head 82.5 -> 76.7; 12 rows: gate / up 15.0 -> 13.8, down 9.6 -> 8.6, QKV 6.1 -> 5.2, LM head
// 104 -> 92; 70B, 24 rows: gate / up 154 -> 147, down 78 -> 72, QKV 31.4 -> 28.8, O 26.3 -> 24.8.
// DEPTH: 9 leaves room for two workgroups a CU, 18 for one.  More is not better: 1B gate / up, four n-tiles, 6 / 12 / 18 fragments: 14.8 / 16.6 /
// 18.1 us; two n-tiles, 4 / 9 / 12: 13.2 / 13.0 / 14.7.  Every workgroup starting at another k-block changed nothing.
//
// Closing a sub-layer from 9 rows on (`tickets`): O and down need K-slices there (one n-tile a workgroup, all of K: down of the 1B shape at 12 rows
// 15.7 us against 8.6), so the slices of a group of n-tiles draw tickets and the last to finish adds them, in slice order, to the residual
// stream and leaves what EPI_RESID leaves, 1/rms to be applied by the consumer.  The norm launch it replaces takes 4.6 - 6.7 us, store, ticket and
// reading back 2 - 3: 1B, 12 rows, in the order of a draft block, O 7.1 and down 11.4 (QKV, which has no tickets, 6.1).
//
// PACK (two operand planes, at most 8 rows): MFMA row r < 8 of the B operand carries plane 0 of row r, row r + 8 plane 1 of the same row, so ONE
// product per weight fragment yields both planes' contributions in output columns r and r + 8, which the reduction adds (hi first).
// Without PACK one product per plane.  The operand of such a block is stored that way, too (packed planes: one plane whose rows
// 8 - 15 are plane 1).
#pragma once
#include "sj_kernels.h"
#include "sj_plan.h"

namespace sj {

// N fragments at 32-bit LDS addresses, waited for in the same block: as ordinary reads they would wait for every direct load of the wave,
// since the compiler cannot tell which of them the data came with.
template <int N> __device__ __forceinline__ void lds_frags(u32x4 (&v)[N], const unsigned (&at)[N]);
#define SJ_LDS_FRAGS_OUT1 "=&v"(v[0])
#define SJ_LDS_FRAGS_OUT2 SJ_LDS_FRAGS_OUT1, "=&v"(v[1])
#define SJ_LDS_FRAGS_OUT3 SJ_LDS_FRAGS_OUT2, "=&v"(v[2])
#define SJ_LDS_FRAGS_OUT4 SJ_LDS_FRAGS_OUT3, "=&v"(v[3])
#define SJ_LDS_FRAGS_OUT5 SJ_LDS_FRAGS_OUT4, "=&v"(v[4])
#define SJ_LDS_FRAGS_OUT6 SJ_LDS_FRAGS_OUT5, "=&v"(v[5])
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[1], const unsigned (&at)[1]) {
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : SJ_LDS_FRAGS_OUT1 : "v"(at[0]) : "memory");
}
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[2], const unsigned (&at)[2]) {
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)" : SJ_LDS_FRAGS_OUT2 : "v"(at[0]), "v"(at[1]) : "memory");
}
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[3], const unsigned (&at)[3]) {
    asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %4\n\tds_read_b128 %2, %5\n\ts_waitcnt lgkmcnt(0)"
                 : SJ_LDS_FRAGS_OUT3 : "v"(at[0]), "v"(at[1]), "v"(at[2]) : "memory");
}
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[4], const unsigned (&at)[4]) {
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                 : SJ_LDS_FRAGS_OUT4 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]) : "memory");
}
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[5], const unsigned (&at)[5]) {
    asm volatile("ds_read_b128 %0, %5\n\tds_read_b128 %1, %6\n\tds_read_b128 %2, %7\n\tds_read_b128 %3, %8\n\tds_read_b128 %4, %9\n\ts_waitcnt lgkmcnt(0)"
                 : SJ_LDS_FRAGS_OUT5 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]) : "memory");
}
template <> __device__ __forceinline__ void lds_frags(u32x4 (&v)[6], const unsigned (&at)[6]) {
    asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %7\n\tds_read_b128 %2, %8\n\tds_read_b128 %3, %9\n\tds_read_b128 %4, %10\n\tds_read_b128 %5, %11\n\t"
                 "s_waitcnt lgkmcnt(0)" : SJ_LDS_FRAGS_OUT6 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]) : "memory");
}

template <typename F, int... Q> __device__ __forceinline__ void each_const(std::integer_sequence<int, Q...>, F f) { (f(std::integral_constant<int, Q>{}), ...); }

// KB of LDS a wave has a use for: its ring, then its accumulators
constexpr int ring_lds(int depth, int nt, int mt, int nb) { return depth > nt + nb ? (depth > nt * mt ? depth : nt * mt) : (nt + nb > nt * mt ? nt + nb : nt * mt); }

template <typename T, int NT, int MT, int EPI, int SPL, bool PACK, int DEPTH>
__global__ __launch_bounds__(RING_CW * 64, ring_lds(DEPTH, NT, MT, ring_operand(PACK, SPL, MT)) <= RING_TWO ? 4 : 2) void gemm_ring_kernel(GemmArgs a) {
    static_assert(!PACK || (SPL == 2 && MT == 1), "packing is for two planes of one row tile");
    constexpr int KSTEP = Traits<T>::KSTEP;
    constexpr int NB = ring_operand(PACK, SPL, MT), PER = NB + NT; // fragments of a k-block, the operand's first
    constexpr int D = DEPTH < PER ? PER : DEPTH;                  // fragments of a wave's ring: a k-block at least
    constexpr int CH = (PER + 5) / 6, CF = (PER + CH - 1) / CH;   // read in CH chunks of CF
    constexpr int TAIL = (D + PER - 1) / PER;                     // last k-blocks, behind which some of a k-block's places have no successor
    static_assert(D < 64, "the load counter holds 63");
    __shared__ u32x4 lds[RING_CW * ring_lds(DEPTH, NT, MT, NB) * 64];
    __shared__ float inv_rms[MT * 16];
    __shared__ int last;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.K / KSTEP, nt0 = blockIdx.x * NT;
    const int nkb = KS / RING_CW / (int)gridDim.y, ks0 = blockIdx.y * nkb * RING_CW;     // whole k-blocks, at least TAIL (ring_fits)

    // what the end needs from memory, in front of the stream (loads are counted in order): the residual stream and gain of the tiles that this
    // wave finishes, and the shares of the rows' sums of squares (packed: at most 8 rows, else MT x 16)
    constexpr int FIN = (NT * MT + RING_CW - 1) / RING_CW;        // (tile, row tile) pairs a wave finishes: w, w + 8, ..
    f32x4 res_x[FIN];
    float res_g[FIN][4];
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int f = 0; f < FIN; ++f) {
            const int p = min(w + f * RING_CW, NT * MT - 1), row = min(p / NT * 16 + (lane >> 2), a.R - 1), col = (nt0 + p % NT) * 16 + (lane & 3) * 4;
            res_x[f] = *reinterpret_cast<const f32x4*>(a.x + (size_t)row * a.N + col);
#pragma unroll
            for (int i = 0; i < 4; ++i) res_g[f][i] = Traits<T>::load(reinterpret_cast<const T*>(a.gain) + col + i);
        }
    }
    constexpr bool SS = EPI == EPI_PARTIAL || EPI == EPI_SWIGLU;  // the products that follow a residual epilogue
    constexpr int SSR = PACK ? 1 : MT * 16 / RING_CW;             // rows whose 1/rms a wave finds: w, w + 8, ..
    const int nss = a.K / 16;                                     // a multiple of 4
    float4 ssv[SSR][2];                                           // of a row of up to 8192 columns
    if constexpr (SS) {
#pragma unroll
        for (int q = 0; q < SSR; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                ssv[q][i] = *reinterpret_cast<const float4*>(a.ss_in ? a.ss_in + (size_t)min(w + q * RING_CW, a.R - 1) * nss + min(lane * 4 + i * 256, nss - 4)
                                                                     : reinterpret_cast<const float*>(a.X));   // (any valid address: no load under a branch)
    }
    asm volatile("" ::: "memory");                                // (not behind the stream's requests)

    // place i = kb * PER + j of the stream: j < NB operand fragment j of the k-block, else weight fragment j - NB
    u32x4* mine = lds + w * D * 64;
    const char* wsrc = reinterpret_cast<const char*>(a.Wt) + (((size_t)nt0 * KS + ks0 + w) * 64 + lane) * 16;
    const char* xsrc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = m * 16 + (PACK ? r & 7 : r), xr = (PACK ? r & 8 : 0) + (row < a.R ? (PACK ? r & 7 : r) : 0);   // lanes of rows past R repeat the first of the tile
        xsrc[m] = reinterpret_cast<const char*>(a.X) + (((size_t)m * KS + ks0 + w) * 64 + (a.rm ? xr * 4 + g : g * 16 + xr)) * 16;
    }
    const size_t tile_step = (size_t)KS * 1024;
    auto request = [&](auto jc, int kb, int slot) {
        constexpr int j = decltype(jc)::value;
        const size_t at = (size_t)kb * (RING_CW * 1024);
        auto dst = (__attribute__((address_space(3))) void*)(mine + slot * 64);
        if constexpr (j < NB)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xsrc[j / (PACK ? 1 : SPL)] + (j % (PACK ? 1 : SPL)) * a.xplane * sizeof(T) + at), dst, 16, 0, 0);
        else
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(wsrc + (j - NB) * tile_step + at), dst, 16, 0, 2);
    };
    each_const(std::make_integer_sequence<int, D>{}, [&](auto ic) { request(std::integral_constant<int, decltype(ic)::value % PER>{}, decltype(ic)::value / PER, decltype(ic)::value); });

    if constexpr (SS) {
        if (a.ss_in) {                                            // uniform
#pragma unroll
            for (int q = 0; q < SSR; ++q) {
                const int row = w + q * RING_CW;
                if (row >= a.R) break;                            // uniform
                float s = lane * 4 < nss ? (ssv[q][0].x + ssv[q][0].y) + (ssv[q][0].z + ssv[q][0].w) : 0.f;
                if (lane * 4 + 256 < nss) s += (ssv[q][1].x + ssv[q][1].y) + (ssv[q][1].z + ssv[q][1].w);
                for (int e = lane * 4 + 512; e < nss; e += 256) {
                    const float4 v = *reinterpret_cast<const float4*>(a.ss_in + (size_t)row * nss + e);
                    s += (v.x + v.y) + (v.z + v.w);
                }
                s = wave_sum(s);
                if (lane == 0) inv_rms[row] = 1.0f / sqrtf(s / (float)a.K + a.eps);
            }
        }
    }

    f32x4 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned base = (unsigned)(unsigned long long)(const __attribute__((address_space(3))) void*)mine + lane * 16;
    int slot0 = 0;                                                // place of the k-block's first fragment
    // one k-block; LEFT = k-blocks from here to the end (TAIL + 1: more)
    auto step = [&](auto left_c, int kb) {
        constexpr int LEFT = decltype(left_c)::value;
        constexpr int END = LEFT > TAIL ? 1 << 20 : LEFT * PER;   // places of the stream that are left, from this k-block's first
        Frag f[PER];
        each_const(std::make_integer_sequence<int, CH>{}, [&](auto cc) {
            constexpr int c0 = decltype(cc)::value * CF, n = c0 + CF < PER ? CF : PER - c0;
            // requested so far: up to place c0 + D, where there are so many; this chunk ends at c0 + n
            constexpr int out = (c0 + D < END ? c0 + D : END) - (c0 + n);
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(out));
            unsigned at[n];
            u32x4 v[n];
            int slot[n];
#pragma unroll
            for (int i = 0; i < n; ++i) {
                const int s = slot0 + c0 + i;                     // < 2 D: PER <= D
                slot[i] = s >= D ? s - D : s;
                at[i] = base + slot[i] * 1024;
            }
            lds_frags(v, at);
#pragma unroll
            for (int i = 0; i < n; ++i) f[c0 + i].u = v[i];
            each_const(std::make_integer_sequence<int, n>{}, [&](auto ic) {
                constexpr int i = decltype(ic)::value, next = c0 + i + D;
                if constexpr (next < END) request(std::integral_constant<int, next % PER>{}, kb + next / PER, slot[i]);
            });
#pragma unroll
            for (int i = 0; i < n; ++i)
                if (c0 + i >= NB) {
#pragma unroll
                    for (int m = 0; m < MT; ++m)
#pragma unroll
                        for (int sp = 0; sp < NB / MT; ++sp) Traits<T>::mma(f[c0 + i], f[m * (NB / MT) + sp], acc[c0 + i - NB][m]);
                }
        });
        slot0 += PER;
        if (slot0 >= D) slot0 -= D;
    };
    int kb = 0;
    for (; kb < nkb - TAIL; ++kb) step(std::integral_constant<int, TAIL + 1>{}, kb);
    each_const(std::make_integer_sequence<int, TAIL>{}, [&](auto qc) { step(std::integral_constant<int, TAIL - decltype(qc)::value>{}, kb + decltype(qc)::value); });

    __syncthreads();                                              // every wave is done with its ring
    float* red = reinterpret_cast<float*>(lds);                   // [wave][tile][row tile][row * 16 + n], D[n = 4g + i][row = r] in lane 16g + r
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m) *reinterpret_cast<f32x4*>(red + ((w * MT + m) * NT + t) * 256 + r * 16 + 4 * g) = acc[t][m];
    __syncthreads();
    if constexpr (EPI != EPI_LOGITS) {
        // one wave per tile, four neighbouring columns of a row per lane (lane l: row l / 4, columns 4 (l % 4) ..)
        const int n0 = (lane & 3) * 4;
        // a finished piece of the residual stream: the stream, the next operand without its 1/rms, the tile's share of the row's sum of squares
        auto close = [&](const f32x4& xv, const float (&gn)[4], int t, int row) {
            const int col = (nt0 + t) * 16 + n0;
            float ss = 0.f;
            if (row < a.R) {
                *reinterpret_cast<f32x4*>(a.x + (size_t)row * a.N + col) = xv;
                float y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { y[i] = xv[i] * gn[i]; ss += xv[i] * xv[i]; }
                Traits<T>::template store_split4<SPL>(reinterpret_cast<T*>(a.act) + opnd_off<T>(row, col, a.N, a.rm), a.actplane, y);
            }
            ss += __shfl_xor(ss, 1, 64);
            ss += __shfl_xor(ss, 2, 64);
            if (row < a.R && (lane & 3) == 0) a.ss_out[(size_t)row * (a.N / 16) + nt0 + t] = ss;
        };
#pragma unroll
        for (int f = 0; f < FIN; ++f) {
            const int p = w + f * RING_CW;
            if (p >= NT * MT) break;                              // uniform
            const int t = p % NT, row = p / NT * 16 + (lane >> 2);
            auto sum_at = [&](int pos) {
                f32x4 sum = *reinterpret_cast<const f32x4*>(red + p * 256 + pos);
#pragma unroll
                for (int ww = 1; ww < RING_CW; ++ww) sum += *reinterpret_cast<const f32x4*>(red + (ww * NT * MT + p) * 256 + pos);
                return sum;
            };
            f32x4 v = sum_at(lane * 4);
            if constexpr (PACK) v += sum_at(((lane + 32) & 63) * 4);   // the second plane's products sit 8 rows further on
            if constexpr (SS) {
                if (a.ss_in && row < a.R) v *= inv_rms[row];
            }
            if constexpr (EPI == EPI_RESID) close(res_x[f] + v, res_g[f], t, row);
            else if constexpr (EPI == EPI_PARTIAL) {
                float* at = a.out + ((size_t)blockIdx.y * a.slice_rows + row) * a.N + (size_t)(nt0 + t) * 16 + n0;
                if (row < a.R) {
                    if (a.tickets) {                              // uniform; write-through: another XCD's workgroup may read it in this launch
                        st_coh(reinterpret_cast<unsigned long long*>(at), __builtin_bit_cast(unsigned long long, float2{v[0], v[1]}));
                        st_coh(reinterpret_cast<unsigned long long*>(at) + 1, __builtin_bit_cast(unsigned long long, float2{v[2], v[3]}));
                    } else *reinterpret_cast<f32x4*>(at) = v;
                }
            } else {
                // tile column n < 8 is gate of FFN column 8 * tile + n, column n + 8 its up projection: two lanes further on
                f32x4 up;
#pragma unroll
                for (int i = 0; i < 4; ++i) up[i] = __shfl_down(v[i], 2, 64);
                if (row < a.R && n0 < 8) {
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = v[i] / (1.0f + expf(-v[i])) * up[i];
                    Traits<T>::template store_split4<SPL>(reinterpret_cast<T*>(a.act) + opnd_off<T>(row, (nt0 + t) * 8 + n0, a.N / 2, a.rm), a.actplane, y);
                }
            }
        }
        if constexpr (EPI == EPI_PARTIAL) {
            if (!a.tickets) return;                               // uniform
            wait_vm0();                                           // this wave's write-through stores are acknowledged ..
            __syncthreads();                                      // .. and so are the other waves', before the ticket is drawn
            if (threadIdx.x == 0)
                last = __hip_atomic_fetch_add(&a.tickets[blockIdx.x], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.y - 1;
            __syncthreads();
            if (!last) return;                                    // uniform for the workgroup
            constexpr int SB = 4;                                 // slices asked for at once (clamped, surplus ignored), added in order as the norm kernel does
#pragma unroll
            for (int f = 0; f < FIN; ++f) {
                const int p = w + f * RING_CW;
                if (p >= NT * MT) break;                          // uniform
                const int t = p % NT, row = p / NT * 16 + (lane >> 2), rd = min(row, a.R - 1), col = (nt0 + t) * 16 + n0;
                f32x4 xv = *reinterpret_cast<const f32x4*>(a.x + (size_t)rd * a.N + col);
                float gn[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) gn[i] = Traits<T>::load(reinterpret_cast<const T*>(a.gain) + col + i);
                for (int s0 = 0; s0 < (int)gridDim.y; s0 += SB) {
                    unsigned long long q[SB][2];
#pragma unroll
                    for (int u = 0; u < SB; ++u) {
                        const auto* at = reinterpret_cast<const unsigned long long*>(a.out + ((size_t)min(s0 + u, (int)gridDim.y - 1) * a.slice_rows + rd) * a.N + col);
                        q[u][0] = ld_coh(at);
                        q[u][1] = ld_coh(at + 1);
                    }
#pragma unroll
                    for (int u = 0; u < SB; ++u)
                        if (s0 + u < (int)gridDim.y) {
                            const float2 lo = __builtin_bit_cast(float2, q[u][0]), hi = __builtin_bit_cast(float2, q[u][1]);
                            xv += f32x4{lo.x, lo.y, hi.x, hi.y};
                        }
                }
                close(xv, gn, t, row);
            }
            if (threadIdx.x == 0) st_coh(&a.tickets[blockIdx.x], 0u);   // ready for the next launch
        }
        return;
    }
    if (threadIdx.x >= 256) return;
    const int tid = threadIdx.x;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            auto sum_at = [&](int pos) {
                float sum = red[(m * NT + t) * 256 + pos];
#pragma unroll
                for (int ww = 1; ww < RING_CW; ++ww) sum += red[((ww * MT + m) * NT + t) * 256 + pos];
                return sum;
            };
            v[t] = sum_at(tid);
            if constexpr (PACK) v[t] += sum_at((tid + 128) & 255);
        }
        few_epilogue<T, NT, EPI, SPL>(a, v, m * 16 + (tid >> 4), tid & 15, nt0);
    }
}

}  // namespace sj
