// HIP kernels of the verification step.  Each kernel cites the part of the method it carries out
// (paper "Method": Eq. 2 / Eq. 4 target forward, Eq. 3 ratio test, Eq. 5 judge, Sec. 3.1 scan and
// extra token, Sec. 2.2 residual resampling).  Workgroups are 256 threads unless noted.
#pragma once
#include "sj_types.h"

#include <type_traits>

namespace sj {

// ---------------------------------------------------------------------------------------------
// Weight re-tiling (model load).  Row-major W[N][K] -> tiles [N/16][K/KSTEP][64 lanes][16 bytes]
// in MFMA A-operand order, so that one wave-wide 16-byte load reads 1 KB of contiguous memory.
// interleave = 1 (stacked [gate; up] source, N = 2F): destination tile t holds gate rows
// 8t..8t+7 in its rows 0-7 and up rows 8t..8t+7 in its rows 8-15, so every tile carries both
// projections of 8 FFN columns and SwiGLU can be applied inside the tile's own epilogue.
template <typename T>
__global__ void retile_kernel(const T* __restrict__ src, T* __restrict__ dst, int N, int K, int interleave) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP;
    const int KS = K / KSTEP;
    const size_t total = (size_t)(N / 16) * KS * 64;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(idx & 63);
        const size_t tile = idx >> 6;
        const int ks = (int)(tile % KS);
        const int nt = (int)(tile / KS);
        const int r = lane & 15, g = lane >> 4;
        const int srow = interleave ? ((r >> 3) * (N / 2) + nt * 8 + (r & 7)) : nt * 16 + r;
        const u32x4* s = reinterpret_cast<const u32x4*>(src + (size_t)srow * K + ks * KSTEP + g * KF);
        reinterpret_cast<u32x4*>(dst)[idx] = *s;
    }
}

// K/V upload of one (seq, layer): host layout [Hkv][len][hd] -> fragments (kv_k_off, kv_v_off).
template <typename T>
__global__ void kv_scatter_kernel(const T* __restrict__ ksrc, const T* __restrict__ vsrc, T* __restrict__ K,
                                  T* __restrict__ V, int Hkv, int len, int cap, int hd) {
    const size_t total = (size_t)Hkv * len * hd;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int dcol = (int)(idx % hd);
        const int pos = (int)((idx / hd) % len);
        const int h = (int)(idx / ((size_t)hd * len));
        K[(size_t)h * cap * hd + kv_k_off<T>(pos, dcol, hd)] = ksrc[idx];
        V[(size_t)h * cap * hd + kv_v_off<T>(pos, dcol, hd)] = vsrc[idx];
    }
}

template <typename T>
__global__ void kv_gather_kernel(T* __restrict__ kdst, T* __restrict__ vdst, const T* __restrict__ K,
                                 const T* __restrict__ V, int Hkv, int pos0, int n, int cap, int hd) {
    const size_t total = (size_t)Hkv * n * hd;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int dcol = (int)(idx % hd);
        const int pos = pos0 + (int)((idx / hd) % n);
        const int h = (int)(idx / ((size_t)hd * n));
        kdst[idx] = K[(size_t)h * cap * hd + kv_k_off<T>(pos, dcol, hd)];
        vdst[idx] = V[(size_t)h * cap * hd + kv_v_off<T>(pos, dcol, hd)];
    }
}

// Caller-supplied hidden states [R][d] (storage dtype) -> operand plane 0 in the layout the LM-head kernel
// reads (opnd_off), and their fp32 copy for the judge.  One thread per 4 consecutive columns.
template <typename T>
__global__ __launch_bounds__(256) void hidden_in_kernel(const T* __restrict__ src, T* __restrict__ xn, float* __restrict__ hn32,
                                                        int R, int d) {
    const size_t n4 = (size_t)R * d / 4;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (size_t)gridDim.x * blockDim.x) {
        const int row = (int)(i / (d / 4)), k = (int)(i % (d / 4)) * 4;
        T* out = xn + opnd_off<T>(row, k, d);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const T v = src[(size_t)row * d + k + e];
            out[e] = v;
            hn32[(size_t)row * d + k + e] = Traits<T>::load(&v);
        }
    }
}

__global__ void set_params_kernel(StepParams p, StepParams* dst) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst = p;
}

__global__ void set_state_kernel(int32_t* len, int32_t* pending, int seq, int l, int p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) { len[seq] = l; pending[seq] = p; }
}

// lengths and pending tokens of a small batch, given with the launch
constexpr int REWIND_SEQS = 64;
struct RewindArgs { int32_t len[REWIND_SEQS], pending[REWIND_SEQS]; };
__global__ __launch_bounds__(REWIND_SEQS) void rewind_kernel(RewindArgs a, int batch, int32_t* __restrict__ len, int32_t* __restrict__ pending) {
    const int b = threadIdx.x;
    if (b < batch) { len[b] = a.len[b]; pending[b] = a.pending[b]; }
}

// ---------------------------------------------------------------------------------------------
// Step start (Eq. 2 input): one workgroup of 1024 threads per query row.  Resolves the row's token and position,
// gathers its embedding into the fp32 residual stream, writes the first layer's normed operand planes (RMSNorm as in
// add_rmsnorm_kernel) and the row's rotary cos/sin table
// (angle = pos * base^(-2i/hd), evaluated in double so the table is correctly rounded fp32).
template <typename T, int SPL>
__global__ __launch_bounds__(1024) void step_begin_kernel(StepParams* __restrict__ sp, ModelDims md,
                                                          const T* __restrict__ embed, const int32_t* __restrict__ len,
                                                          const int32_t* __restrict__ pending, float* __restrict__ x,
                                                          float* __restrict__ cs, int32_t* __restrict__ row_tok,
                                                          double log_base, const T* __restrict__ gain, T* __restrict__ xn,
                                                          size_t xplane, int rm) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    const int rps = sp->rps;
    const int bi = r / rps, j = r % rps;
    const int b = sp->seq_base + bi;
    int tok;
    if (sp->tok_mode == 1) tok = sp->prefill_tokens[j];
    else if (sp->tok_mode == 2) tok = sp->draft_tokens[bi * rps + j];
    else tok = (j == 0) ? pending[b] : sp->draft_tokens[bi * sp->gamma + (j - 1)];
    tok = min(max(tok, 0), md.V - 1);
    const int pos = len[b] + j;
    if (threadIdx.x == 0) row_tok[r] = tok;
    if (r == 0 && threadIdx.x == 0) ++sp->step;        // read by the step's last kernels only
    const T* e = embed + (size_t)tok * md.d;
    constexpr int MAXP = 4;                            // d <= 16384 (host-checked), a multiple of 64
    float v[MAXP][4], ss = 0.f;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        const int c = (p * 1024 + threadIdx.x) * 4;
        if (c < md.d) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[p][i] = Traits<T>::load(e + c + i);
                ss += v[p][i] * v[p][i];
            }
            *reinterpret_cast<f32x4*>(x + (size_t)r * md.d + c) = f32x4{v[p][0], v[p][1], v[p][2], v[p][3]};
        }
    }
    const int half = md.hd >> 1;
    for (int i = threadIdx.x; i < half; i += 1024) {
        const double inv_freq = exp(-2.0 * (double)i / (double)md.hd * log_base);
        double s, c;
        sincos((double)pos * inv_freq, &s, &c);
        cs[((size_t)r * half + i) * 2 + 0] = (float)c;
        cs[((size_t)r * half + i) * 2 + 1] = (float)s;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += red[w];
    const float inv = 1.0f / sqrtf(tot / (float)md.d + md.eps);
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        const int c = (p * 1024 + threadIdx.x) * 4;
        if (c < md.d) {
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = v[p][i] * inv * Traits<T>::load(gain + c + i);
            Traits<T>::template store_split4<SPL>(xn + opnd_off<T>(r, c, md.d, rm), xplane, y);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Residual add + RMSNorm.  x[r] += sum_s part[s][r] (fixed order), then
// xn[r] = x[r] * gain / sqrt(mean(x[r]^2) + eps) as the next GEMM's operand (SPL planes in bf16),
// optionally also in fp32 (final hidden state for the judge, Eq. 4).
template <typename T, int PB, int SPL>
__global__ __launch_bounds__(1024) void add_rmsnorm_kernel(int R, int d, float eps, float* __restrict__ x,
                                                           const float* __restrict__ part, int nparts,
                                                           const T* __restrict__ gain, T* __restrict__ xn,
                                                           size_t xplane, float* __restrict__ xn32, int rm) {
    // one workgroup of 1024 threads per row, 4 columns per thread and pass; all loads of a pass are
    // independent.  Rows wider than 16384 columns are not supported (host-checked).
    constexpr int MAXP = 4;
    __shared__ float red[16];
    const int r = blockIdx.x;
    float* xr = x + (size_t)r * d;
    f32x4 v[MAXP];
    T gn[MAXP][4];                                     // the gain, on its way while the row is summed (asked for after the barrier, 12 rows of 2048: 4.7 us, so 4.5)
    float ss = 0.f;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        const int c = (p * 1024 + threadIdx.x) * 4;
        v[p] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (c < d) {
            v[p] = *reinterpret_cast<const f32x4*>(xr + c);
#pragma unroll
            for (int i = 0; i < 4; ++i) gn[p][i] = gain[c + i];
            // partials in batches of PB independent loads (index clamped, surplus ignored), added in order
            for (int s0 = 0; s0 < nparts; s0 += PB) {
                f32x4 t[PB];
#pragma unroll
                for (int u = 0; u < PB; ++u)
                    t[u] = *reinterpret_cast<const f32x4*>(part + ((size_t)min(s0 + u, nparts - 1) * R + r) * d + c);
#pragma unroll
                for (int u = 0; u < PB; ++u)
                    if (s0 + u < nparts) v[p] += t[u];
            }
            if (nparts) *reinterpret_cast<f32x4*>(xr + c) = v[p];
            ss += v[p][0] * v[p][0] + v[p][1] * v[p][1] + v[p][2] * v[p][2] + v[p][3] * v[p][3];
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += red[w];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        const int c = (p * 1024 + threadIdx.x) * 4;
        if (c < d) {
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = v[p][i] * inv * Traits<T>::load(&gn[p][i]);
            Traits<T>::template store_split4<SPL>(xn + opnd_off<T>(r, c, d, rm), xplane, y);
            if (xn32) *reinterpret_cast<f32x4*>(xn32 + (size_t)r * d + c) = f32x4{y[0], y[1], y[2], y[3]};
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Weight-streaming skinny GEMM: Y[R][N] = X[R][K] * W[N][K]^T with W in the re-tiled layout.
// Every byte of W is read exactly once; X (a few rows) is re-read from cache.
// Workgroup (bx, by): n-tiles [bx*NT, bx*NT+NT), K-slice by of gridDim.y; its 4 waves split that
// slice again and are summed through LDS in wave order (deterministic).
// EPI_RESID closes a sub-layer without a norm launch: the workgroup holds finished output columns (no K-slices), adds them to
// the fp32 residual stream, writes the next product's operand planes WITHOUT the 1/rms factor - (x + y) * gain - and each
// tile's share of every row's sum of squares.  The consumer (QKV or gate / up: EPI_PARTIAL or EPI_SWIGLU, few rows, `ss_in` set) sums
// the shares and multiplies its finished sums by 1/rms: a factor of the row commutes with the product.
enum { EPI_PARTIAL = 0, EPI_SWIGLU = 1, EPI_LOGITS = 2, EPI_RESID = 3 };

struct GemmArgs {
    const void* Wt;     // tiled weights
    const void* X;      // [SPL planes] of fragments (opnd_off), storage dtype; rows >= R are padding
    size_t xplane;      // elements between consecutive planes of X
    size_t actplane;    // same for act
    int32_t K, N, R;
    int32_t rm;         // few-row kernels: operand and result planes have rows side by side in a block (opnd_off)
    int32_t slice_rows; // EPI_PARTIAL: rows between consecutive K-slices of out (>= R)
    float* out;         // EPI_PARTIAL: [gridDim.y][slice_rows][N] fp32;  EPI_LOGITS: [R][N] fp32
    void* act;          // EPI_SWIGLU: planes of rows of width N/2 (opnd_off), storage dtype = silu(gate) * up
    float4* stats;      // EPI_LOGITS: [R][gridDim.x] (max, sum exp((l-max)/T), argmax as float bits, 0)
    float inv_temp;     // 1/T, 0 when T = 0
    int32_t rgroups;    // many-row kernel: row groups of one launch (0 or 1: the launch is one group of R rows); with
                        // more, R is the total row count and every workgroup derives its group's rows and pointers
    const float* ss_in; // EPI_PARTIAL, EPI_SWIGLU, few rows: null, or [R][K / 16] shares of the rows' sums of squares: the operand lacks 1/rms
    float eps;
    float* x;           // EPI_RESID: [R][N] residual stream, updated in place
    const void* gain;   // EPI_RESID: [N] norm gain of the next product, storage dtype
    float* ss_out;      // EPI_RESID: [R][N / 16]; the operand planes go to act / actplane ([R][N])
    unsigned* tickets;  // EPI_PARTIAL of the LDS-ring kernel: null, or one word per workgroup of the grid's x, zero between launches: the last
                        // K-slice of a group of n-tiles adds all of them in slice order and closes the sub-layer as EPI_RESID does
};

// 1/rms of row r from the shares of its sum of squares, by one wave (fixed order); K = width of the row, a multiple of 64
__device__ __forceinline__ float row_inv_rms(const GemmArgs& a, int r, int lane) {
    const int n = a.K / 16;
    float s = 0.f;
    for (int i = lane * 4; i < n; i += 256) {
        const float4 v = *reinterpret_cast<const float4*>(a.ss_in + (size_t)r * n + i);
        s += (v.x + v.y) + (v.z + v.w);
    }
    s = wave_sum(s);
    return 1.0f / sqrtf(s / (float)a.K + a.eps);
}

// Epilogue of the few-row kernels for one (row, column en of every tile) position: v[t] is the finished sum of tile
// nt0 + t.  Every thread of the first 256 of the workgroup calls it (16 consecutive lanes share a row; rows >= R
// take part in the shuffles and store nothing).
template <typename T, int NT, int EPI, int SPL>
__device__ __forceinline__ void few_epilogue(const GemmArgs& a, const float (&v)[NT], int row, int en, int nt0) {
    if constexpr (EPI == EPI_PARTIAL) {
        if (row < a.R) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                a.out[((size_t)blockIdx.y * a.slice_rows + row) * a.N + (size_t)(nt0 + t) * 16 + en] = v[t];
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        // tile column en < 8 is gate of FFN column 8*tile + en, column en + 8 its up projection
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float up = __shfl_down(v[t], 8, 64);
            if (row < a.R && en < 8) {
                const float gate = v[t];
                const float y = gate / (1.0f + expf(-gate)) * up;
                Traits<T>::template store_split<SPL>(reinterpret_cast<T*>(a.act) + opnd_off<T>(row, (nt0 + t) * 8 + en, a.N / 2, a.rm),
                                                     a.actplane, y);
            }
        }
    } else {
        // logits + this workgroup's softmax partial for the row (16 lanes share a row)
        float mx = v[0];
        int arg = nt0 * 16 + en;
#pragma unroll
        for (int t = 1; t < NT; ++t)
            if (v[t] > mx) { mx = v[t]; arg = (nt0 + t) * 16 + en; }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const float omx = __shfl_xor(mx, o, 64);
            const int oarg = __shfl_xor(arg, o, 64);
            if (omx > mx || (omx == mx && oarg < arg)) { mx = omx; arg = oarg; }
        }
        float se = 0.f;
        if (a.inv_temp > 0.f) {
#pragma unroll
            for (int t = 0; t < NT; ++t) se += expf((v[t] - mx) * a.inv_temp);
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) se += __shfl_xor(se, o, 64);
        }
        if (row < a.R) {
#pragma unroll
            for (int t = 0; t < NT; ++t) a.out[(size_t)row * a.N + (size_t)(nt0 + t) * 16 + en] = v[t];
            if (en == 0) a.stats[(size_t)row * gridDim.x + blockIdx.x] = float4{mx, se, __int_as_float(arg), 0.f};
        }
    }
}

#ifdef SJ_GEMM_PROF
__device__ unsigned long long gemm_prof[8192 * 8];
#define GEMM_STAMP(k) do { if ((threadIdx.x & 63) == 0) gemm_prof[(((blockIdx.y * gridDim.x + blockIdx.x) * WAVES + (threadIdx.x >> 6)) & 8191) * 8 + (k)] = wall_clock64(); } while (0)
#else
#define GEMM_STAMP(k) do { } while (0)
#endif

template <typename T, int NT, int MT, int EPI, int SPL, int WAVES, int D = 2>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(GemmArgs a) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP;
    __shared__ float red[WAVES][NT * MT][256];
    __shared__ float inv_rms[MT * 16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.K / KSTEP;
    const int nt0 = blockIdx.x * NT;
    const int parts = gridDim.y * WAVES, part = blockIdx.y * WAVES + w;
    const int ks0 = (int)((long long)part * KS / parts), ks1 = (int)((long long)(part + 1) * KS / parts);
    const u32x4* Wt = reinterpret_cast<const u32x4*>(a.Wt) + ((size_t)nt0 * KS + ks0) * 64 + lane;
    // padding rows (>= R) feed columns of D that are never stored: their lanes repeat row 0 of the tile
    const T* Xr[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int xr = m * 16 + r < a.R ? r : 0;
        Xr[m] = reinterpret_cast<const T*>(a.X) + (((size_t)m * KS + ks0) * 64 + (a.rm ? xr * 4 + g : g * 16 + xr)) * KF;
    }

    f32x4 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Without K-slices a wave of the residual epilogue sums an eighth of K, up to eight times as much as with them.  fp32 operands are
    // exact, the sums are the error: they are folded into totals every FOLD k-steps (fp32, d 3072, FFN 8192, 6 rows: error of the
    // hidden states against 64 bits 1.69e-6 with slices, 1.96e-6 in one chain, 1.66e-6 folded).
    constexpr int FOLD = EPI == EPI_RESID && std::is_same<T, float>::value ? 8 : 0;
    static_assert(FOLD % D == 0, "whole turns of the ring");
    f32x4 tot[FOLD ? NT : 1][MT];
    if constexpr (FOLD > 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int m = 0; m < MT; ++m) tot[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto fold = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                tot[t][m] += acc[t][m];
                acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };

    // Ring of D single-k-step register buffers.  The load of step i + D - 1 is always issued (index
    // clamped to the last step) before step i is consumed, so the loop body is branch-free around the
    // loads - a load under a branch makes the compiler wait for everything outstanding - and the wave
    // keeps D - 1 k-steps of weight tiles in flight, waited for one step at a time.
    Frag fa[D][NT], fb[D][MT][SPL];
    auto load = [&](int buf, int ks) {
#pragma unroll
        for (int t = 0; t < NT; ++t) fa[buf][t].u = __builtin_nontemporal_load(Wt + ((size_t)t * KS + ks) * 64);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int sp = 0; sp < SPL; ++sp)
                fb[buf][m][sp].u = *reinterpret_cast<const u32x4*>(Xr[m] + sp * a.xplane + (size_t)ks * (16 * KSTEP));
    };
    auto compute = [&](int buf) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int sp = 0; sp < SPL; ++sp) Traits<T>::mma(fa[buf][t], fb[buf][m][sp], acc[t][m]);
    };
    const int nks = ks1 - ks0;
    GEMM_STAMP(0);
    if (nks > 0) {
#pragma unroll
        for (int j = 0; j < D - 1; ++j) load(j, min(j, nks - 1));
    }
    // What the end needs from memory, asked for behind the first weights (in front of them, or at the end, it was a memory trip of its
    // own: 1 us of a launch of 5): the shares of the rows' sums of squares (at most 8 rows where there are any), and the residual
    // stream and gain of this thread's columns.  Without them any valid address: no load under a branch.
    constexpr bool SS = MT == 1 && (EPI == EPI_PARTIAL || EPI == EPI_SWIGLU);     // the products that follow a residual epilogue
    constexpr int SSR = SS ? (8 + WAVES - 1) / WAVES : 1;
    float4 ssv[SSR];
    const int nss = a.K / 16;                            // a multiple of 4
#pragma unroll
    for (int i = 0; SS && i < SSR; ++i)
        ssv[i] = *reinterpret_cast<const float4*>(a.ss_in ? a.ss_in + (size_t)min(w + i * WAVES, a.R - 1) * nss + min(lane * 4, nss - 4)
                                                          : reinterpret_cast<const float*>(a.X));
    float res_x[NT], res_g[NT];
    if constexpr (EPI == EPI_RESID) {
        const int row = min((int)(threadIdx.x >> 4) & 15, a.R - 1);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = (nt0 + t) * 16 + (threadIdx.x & 15);
            res_x[t] = a.x[(size_t)row * a.N + col];
            res_g[t] = Traits<T>::load(reinterpret_cast<const T*>(a.gain) + col);
        }
    }
    GEMM_STAMP(1);
    if (nks > 0) {
        for (int c = 0; c < nks; c += D) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                load((j + D - 1) % D, min(c + j + D - 1, nks - 1));
                if (c + j < nks) compute(j);
            }
            if constexpr (FOLD > 0) {
                if ((c + D) % FOLD == 0) fold();       // uniform
            }
        }
        if constexpr (FOLD > 0) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[t][m] += tot[t][m];
        }
    }

    if (SS && a.ss_in) {                                 // uniform; read after the reduction's barrier
#pragma unroll
        for (int i = 0; i < SSR; ++i) {
            const int row = w + i * WAVES;
            if (row >= a.R) break;                       // uniform
            float ss = lane * 4 < nss ? (ssv[i].x + ssv[i].y) + (ssv[i].z + ssv[i].w) : 0.f;
            for (int e = lane * 4 + 256; e < nss; e += 256) {
                const float4 v = *reinterpret_cast<const float4*>(a.ss_in + (size_t)row * nss + e);
                ss += (v.x + v.y) + (v.z + v.w);
            }
            ss = wave_sum(ss);
            if (lane == 0) inv_rms[row] = 1.0f / sqrtf(ss / (float)a.K + a.eps);
        }
    }
    GEMM_STAMP(2);
    // D[n = 4g+i][row = r]  ->  red[w][tile][row*16 + n]
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[w][t * MT + m][r * 16 + 4 * g + i] = acc[t][m][i];
    __syncthreads();

    GEMM_STAMP(3);
    // the first 256 threads own one (row, column) position of every tile; partial sums are added in
    // wave order
    if (threadIdx.x >= 256) return;
    const int tid = threadIdx.x;
    const int er = tid >> 4, en = tid & 15;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = m * 16 + er;
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float sum = red[0][t * MT + m][tid];
#pragma unroll
            for (int ww = 1; ww < WAVES; ++ww) sum += red[ww][t * MT + m][tid];
            v[t] = SS && a.ss_in && row < a.R ? sum * inv_rms[row] : sum;
        }
        if constexpr (EPI == EPI_RESID) {                // at most 8 rows: one row tile
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int col = (nt0 + t) * 16 + en;
                float xv = 0.f;
                if (row < a.R) {
                    xv = res_x[t] + v[t];
                    a.x[(size_t)row * a.N + col] = xv;
                    Traits<T>::template store_split<SPL>(reinterpret_cast<T*>(a.act) + opnd_off<T>(row, col, a.N, a.rm), a.actplane, xv * res_g[t]);
                }
                float ss = xv * xv;
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
                if (row < a.R && en == 0) a.ss_out[(size_t)row * (a.N / 16) + nt0 + t] = ss;
            }
        } else few_epilogue<T, NT, EPI, SPL>(a, v, row, en, nt0);
    }
}

// ---------------------------------------------------------------------------------------------
// Vocabulary softmax statistics of each row from the LM-head workgroups' partials:
// row max, Z = sum exp((l - max)/T), lowest-index arg-max.  One workgroup per row.
// Bound by the latency of its loads, and from some hundred rows on by their bytes: a thread requests its first KEEP statistics together and keeps
// them for the sum; KEEP is the least of 1, 4, 8 and 16 that holds the row.  us with 4 up to 1024 statistics, else 16 (the rest of a thread's
// loads repeat the last one) / as it is: 128 statistics 3.16 / 2.96, 2004 of 126 rows 6.0 / 5.4, of 576 rows with 512 judge scores 13.5 / 13.1.
template <int KEEP>
__device__ __forceinline__ void softmax_merge_keep(int r, const float4* __restrict__ stats, int nblk, float inv_temp,
                                                   float4* __restrict__ rowstat) {
    __shared__ float smx[4];
    __shared__ int sarg[4];
    __shared__ float red[4];
    const float4* s = stats + (size_t)r * nblk;
    const int i0 = threadIdx.x;
    float4 keep[KEEP];
#pragma unroll
    for (int k = 0; k < KEEP; ++k) keep[k] = s[min(i0 + k * 256, nblk - 1)];       // past the end the last one again: no new maximum, not summed
    float mx = -INFINITY;
    int arg = 0x7fffffff;
    auto take = [&](const float4& v) {
        const int a = __float_as_int(v.z);
        if (v.x > mx || (v.x == mx && a < arg)) { mx = v.x; arg = a; }
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k) take(keep[k]);
    for (int i = i0 + KEEP * 256; i < nblk; i += 256) take(s[i]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float omx = __shfl_xor(mx, o, 64);
        const int oarg = __shfl_xor(arg, o, 64);
        if (omx > mx || (omx == mx && oarg < arg)) { mx = omx; arg = oarg; }
    }
    if ((threadIdx.x & 63) == 0) { smx[threadIdx.x >> 6] = mx; sarg[threadIdx.x >> 6] = arg; }
    __syncthreads();
    mx = smx[0]; arg = sarg[0];
    for (int w = 1; w < 4; ++w)
        if (smx[w] > mx || (smx[w] == mx && sarg[w] < arg)) { mx = smx[w]; arg = sarg[w]; }
    float z = 0.f;
    if (inv_temp > 0.f) {
#pragma unroll
        for (int k = 0; k < KEEP; ++k)
            if (i0 + k * 256 < nblk) z += keep[k].y * expf((keep[k].x - mx) * inv_temp);
        for (int i = i0 + KEEP * 256; i < nblk; i += 256) {
            const float4 v = s[i];
            z += v.y * expf((v.x - mx) * inv_temp);
        }
    }
    z = block_sum_256(z, red);
    if (threadIdx.x == 0) rowstat[r] = float4{mx, z, __int_as_float(arg), 0.f};
}

__device__ __forceinline__ void softmax_merge_row(int r, const float4* __restrict__ stats, int nblk, float inv_temp, float4* __restrict__ rowstat) {
    if (nblk <= 256) softmax_merge_keep<1>(r, stats, nblk, inv_temp, rowstat);                              // uniform
    else if (nblk <= 1024) softmax_merge_keep<4>(r, stats, nblk, inv_temp, rowstat);
    else if (nblk <= 2048) softmax_merge_keep<8>(r, stats, nblk, inv_temp, rowstat);
    else softmax_merge_keep<16>(r, stats, nblk, inv_temp, rowstat);
}

__global__ __launch_bounds__(256) void softmax_merge_kernel(const float4* __restrict__ stats, int nblk, float inv_temp,
                                                            float4* __restrict__ rowstat) {
    softmax_merge_row(blockIdx.x, stats, nblk, inv_temp, rowstat);
}

// ---------------------------------------------------------------------------------------------
// Judge verifier (Eq. 5): score = sigmoid(w . h + b) on the final, normed hidden state of the row
// whose input is the draft token.  One workgroup per (sequence, draft position); entry j scores
// d_{j+1}, i.e. block row j + 1.
// In the top-k mode (the relaxed baseline of Sec. 4.1) the workgroup also ranks d_{j+1} in the target's
// row j: the number of vocabulary entries with a larger logit, or an equal one at a lower index.
template <typename T>
__device__ __forceinline__ void judge_token(int blk, const StepParams* __restrict__ sp, int d,
                                            const float* __restrict__ hn32, const float* __restrict__ row_scale,
                                            const T* __restrict__ w, const T* __restrict__ bias,
                                            float* __restrict__ scores, int V, const float* __restrict__ logits,
                                            int32_t* __restrict__ ranks) {
    __shared__ float red[4];
    const int gamma = sp->gamma;
    const int bi = blk / gamma, j = blk % gamma;
    const int row = bi * (gamma + 1) + j + 1;
    if (sp->mode == 3) {                                   // uniform for the launch
        const float* l = logits + (size_t)(row - 1) * V;
        const int tok = min(max(sp->draft_tokens[bi * gamma + j], 0), V - 1);
        const float ref = l[tok];
        int cnt = 0;
        for (int c = threadIdx.x * 4; c < V; c += 1024) {  // V is a multiple of 128
            const float4 v = *reinterpret_cast<const float4*>(l + c);
            cnt += (v.x > ref || (v.x == ref && c < tok)) + (v.y > ref || (v.y == ref && c + 1 < tok)) +
                   (v.z > ref || (v.z == ref && c + 2 < tok)) + (v.w > ref || (v.w == ref && c + 3 < tok));
        }
        const float total = block_sum_256((float)cnt, red);   // exact: counts stay below 2^24
        if (threadIdx.x == 0) ranks[blk] = (int)total;
        __syncthreads();
    }
    const float* h = hn32 + (size_t)row * d;
    float acc = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) acc += h[c] * Traits<T>::load(w + c);
    acc = block_sum_256(acc, red);
    if (threadIdx.x == 0) {
        // row_scale: the hidden state was stored without its 1/rms factor (applied here)
        const float z = acc * (row_scale ? row_scale[row] : 1.0f) + Traits<T>::load(bias);
        scores[blk] = 1.0f / (1.0f + expf(-z));
    }
}

template <typename T>
__global__ __launch_bounds__(256) void judge_kernel(const StepParams* __restrict__ sp, int d,
                                                    const float* __restrict__ hn32, const float* __restrict__ row_scale,
                                                    const T* __restrict__ w, const T* __restrict__ bias,
                                                    float* __restrict__ scores, int V, const float* __restrict__ logits,
                                                    int32_t* __restrict__ ranks) {
    judge_token<T>(blockIdx.x, sp, d, hn32, row_scale, w, bias, scores, V, logits, ranks);
}

// The two of them in one launch (they do not depend on each other: the judge reads hidden states, and in the top-k
// mode raw logits): workgroups [0, R) merge the softmax statistics of a row, the others score one draft token each.
template <typename T>
__global__ __launch_bounds__(256) void merge_judge_kernel(int R, const float4* __restrict__ stats, int nblk, float inv_temp,
                                                          float4* __restrict__ rowstat, const StepParams* __restrict__ sp, int d,
                                                          const float* __restrict__ hn32, const T* __restrict__ w,
                                                          const T* __restrict__ bias, float* __restrict__ scores, int V,
                                                          const float* __restrict__ logits, int32_t* __restrict__ ranks) {
    if ((int)blockIdx.x < R) softmax_merge_row(blockIdx.x, stats, nblk, inv_temp, rowstat);
    else judge_token<T>(blockIdx.x - R, sp, d, hn32, nullptr, w, bias, scores, V, logits, ranks);
}

// ---------------------------------------------------------------------------------------------
// Ratio test (Eq. 3), OR with the judge (Sec. 3.2), first-rejection scan (Sec. 3.1): one wave per
// sequence, lane j handles draft d_{j+1}:  accept iff u*q(d) < p(d)  with p(d) read from block row j,
// or score > theta.  accepted_len = number of leading accepted lanes (ballot + count trailing ones).
// One wave, lane j; returns accepted_len to every lane; `write` says whether this wave stores the results.
__device__ __forceinline__ int accept_scan_seq(int bi, int j, bool write, const StepParams* __restrict__ sp, int V, float inv_temp,
                                               const float* __restrict__ logits, const float4* __restrict__ rowstat,
                                               const float* __restrict__ scores, float* __restrict__ p_at_d,
                                               int32_t* __restrict__ bits, int32_t* __restrict__ nacc,
                                               const int32_t* __restrict__ ranks) {
    const int gamma = sp->gamma;
    bool ok = false;
    if (j < gamma) {
        const int row = bi * (gamma + 1) + j;
        int tok = sp->draft_tokens[bi * gamma + j];
        tok = min(max(tok, 0), V - 1);
        const float4 st = rowstat[row];
        float p;
        if (inv_temp > 0.f) p = expf((logits[(size_t)row * V + tok] - st.x) * inv_temp) / st.y;
        else p = (tok == __float_as_int(st.z)) ? 1.f : 0.f;
        const float q = sp->draft_probs[((size_t)bi * gamma + j) * V + tok];
        const float u = sp->uniforms[bi * (gamma + 1) + j];
        const bool a = (u * q < p);
        const bool jd = scores[bi * gamma + j] > sp->theta;
        const bool tk = (sp->mode == 3) && ranks[bi * gamma + j] < sp->topk;
        ok = (sp->mode == 1) ? a : (sp->mode == 2) ? jd : (sp->mode == 3) ? tk : (a || jd);
        if (write) {
            p_at_d[bi * gamma + j] = p;
            bits[bi * gamma + j] = (a ? 1 : 0) | (jd ? 2 : 0) | (tk ? 4 : 0);
        }
    }
    const unsigned long long mask = __ballot(ok);
    const int n = __builtin_ctzll(~mask);          // lanes >= gamma vote false, so n <= gamma
    if (write && j == 0) {
        nacc[bi] = n;
        sp->accepted_len[bi] = n;
    }
    return n;
}

__global__ __launch_bounds__(64) void accept_scan_kernel(const StepParams* __restrict__ sp, int V, float inv_temp,
                                                         const float* __restrict__ logits,
                                                         const float4* __restrict__ rowstat,
                                                         const float* __restrict__ scores,
                                                         float* __restrict__ p_at_d, int32_t* __restrict__ bits,
                                                         int32_t* __restrict__ nacc, const int32_t* __restrict__ ranks) {
    accept_scan_seq(blockIdx.x, threadIdx.x, true, sp, V, inv_temp, logits, rowstat, scores, p_at_d, bits, nacc, ranks);
}

// ---------------------------------------------------------------------------------------------
// Extra token (Sec. 3.1 bonus / Sec. 2.2 residual), inverse CDF in vocabulary order with one
// uniform.  Weights are formed in double from the fp32 logits so that the draw is reproducible
// from those logits to ~1e-15:  e_k = exp((l_k - max)/T),  Z = sum e_k,
//   all accepted:  w_k = e_k          else:  w_k = max(0, e_k - Z * q_k)   (q = draft law of the
// first rejected token);  if sum w = 0 fall back to w = e.
// Element k belongs to slab k / slab_len; slab s is owned by thread s % 256 of workgroup s / 256.
//   pass 1 (resample_e):    per-slab and per-workgroup sums of e -> epart, eblk
//   pass 2 (resample_w):    Z from eblk, the same sums of w      -> wpart, wblk
//   pass 3 (resample_pick): scan the workgroup sums, then the slab sums of the workgroup that holds the target, then that
//                           slab's weights; commit the sequence state.
// The passes are chains of dependent memory round trips over little data, so the search goes down three levels with one round
// trip each; scanning all slab sums of a 128256-entry vocabulary (8192) in every workgroup that needs Z took 64 KB of reads
// each (64 sequences: pass 2 29 us, pick 23 us).
struct ResampleArgs {
    int32_t V, nslab, slab_len;   // nslab = 256 * gridDim.x of passes 1, 2
    float inv_temp;
    const float* logits;
    const float4* rowstat;
    const int32_t* nacc;
    double* epart;    // [nseq][nslab]
    double* wpart;    // [nseq][nslab]
    double* eblk;     // [nseq][nslab / 256]
    double* wblk;     // [nseq][nslab / 256]
};

__device__ __forceinline__ double e_of(float logit, float mx, float inv_temp) {
    return exp(((double)logit - (double)mx) * (double)inv_temp);
}

// pass 1 of the draw for the row after `n` accepted tokens; q_out (a plain decode step of a draft block): the row's law as fp32
// probabilities
__device__ __forceinline__ void resample_e_slab(const StepParams* __restrict__ sp, const ResampleArgs& a, int n, float* __restrict__ q_out) {
    __shared__ double red[4];
    const int bi = blockIdx.y, slab = blockIdx.x * 256 + threadIdx.x;
    const int gamma = sp->gamma;
    const int row = bi * (gamma + 1) + n;
    const float4 st = a.rowstat[row];
    const float mx = st.x, invz = 1.0f / st.y;
    const float* l = a.logits + (size_t)row * a.V;
    const int k0 = slab * a.slab_len, k1 = min(a.V, k0 + a.slab_len);
    double s = 0.0;
    if (((a.slab_len | a.V) & 3) == 0) {               // 16-byte loads; same summation order
        for (int k = k0; k < k1; k += 4) {
            const float4 v = *reinterpret_cast<const float4*>(l + k);
            s += e_of(v.x, mx, a.inv_temp);
            s += e_of(v.y, mx, a.inv_temp);
            s += e_of(v.z, mx, a.inv_temp);
            s += e_of(v.w, mx, a.inv_temp);
        }
    } else {
        for (int k = k0; k < k1; ++k) s += e_of(l[k], mx, a.inv_temp);
    }
    a.epart[(size_t)bi * a.nslab + slab] = s;
    s = block_sum_256(s, red);
    if (threadIdx.x == 0) a.eblk[(size_t)bi * (a.nslab / 256) + blockIdx.x] = s;
    if (q_out) {                                       // uniform; consecutive entries per thread, whatever the slabs are
        const int lo = blockIdx.x * 256 * a.slab_len, hi = min(a.V, lo + 256 * a.slab_len);
        for (int k = lo + threadIdx.x; k < hi; k += 256) q_out[k] = expf((l[k] - mx) * a.inv_temp) * invz;
    }
}

// Scan and pass 1 in one launch: pass 1 only needs accepted_len to know its row, and the scan is a handful of loads,
// so the first wave of EVERY workgroup repeats it for the workgroup's sequence (same inputs, same arithmetic, same
// result) and the workgroups with blockIdx.x == 0 store it.
__global__ __launch_bounds__(256) void scan_resample_e_kernel(const StepParams* __restrict__ sp, ResampleArgs a,
                                                              const float* __restrict__ scores, float* __restrict__ p_at_d,
                                                              int32_t* __restrict__ bits, int32_t* __restrict__ nacc,
                                                              const int32_t* __restrict__ ranks) {
    __shared__ int n_sh;
    if (threadIdx.x < 64) {
        const int n = accept_scan_seq(blockIdx.y, threadIdx.x, blockIdx.x == 0, sp, a.V, a.inv_temp, a.logits, a.rowstat, scores,
                                      p_at_d, bits, nacc, ranks);
        if (threadIdx.x == 0) n_sh = n;
    }
    __syncthreads();
    resample_e_slab(sp, a, n_sh, sp->emit_probs ? sp->emit_probs + ((size_t)blockIdx.y * sp->emit_gamma + sp->step) * a.V : nullptr);
}

// sum of n workgroup sums by one wave; fixed order, every lane gets the result
__device__ __forceinline__ double total_of(const double* part, int n) {
    double s = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64) s += part[i];
    return wave_sum(s);
}

// pass 2: the same sums of w (nothing is drawn from them when every draft token was accepted)
__device__ __forceinline__ void resample_w_slab(const StepParams* __restrict__ sp, const ResampleArgs& a, int n) {
    __shared__ double red[4];
    const int bi = blockIdx.y, slab = blockIdx.x * 256 + threadIdx.x, nblk = a.nslab / 256;
    const int gamma = sp->gamma;
    double s = 0.0;
    if (n < gamma) {                                   // uniform for the workgroup
        const double Z = total_of(a.eblk + (size_t)bi * nblk, nblk);
        const int row = bi * (gamma + 1) + n;
        const float mx = a.rowstat[row].x;
        const float* l = a.logits + (size_t)row * a.V;
        const int k0 = slab * a.slab_len, k1 = min(a.V, k0 + a.slab_len);
        const float* q = sp->draft_probs + ((size_t)bi * gamma + n) * a.V;
        if (((a.slab_len | a.V) & 3) == 0 && (reinterpret_cast<uintptr_t>(q) & 15) == 0) {   // 16-byte loads; same order
            for (int k = k0; k < k1; k += 4) {
                const float4 v = *reinterpret_cast<const float4*>(l + k);
                const float4 u = *reinterpret_cast<const float4*>(q + k);
                s += fmax(0.0, e_of(v.x, mx, a.inv_temp) - Z * (double)u.x);
                s += fmax(0.0, e_of(v.y, mx, a.inv_temp) - Z * (double)u.y);
                s += fmax(0.0, e_of(v.z, mx, a.inv_temp) - Z * (double)u.z);
                s += fmax(0.0, e_of(v.w, mx, a.inv_temp) - Z * (double)u.w);
            }
        } else {
            for (int k = k0; k < k1; ++k) s += fmax(0.0, e_of(l[k], mx, a.inv_temp) - Z * (double)q[k]);
        }
    }
    a.wpart[(size_t)bi * a.nslab + slab] = s;
    s = block_sum_256(s, red);
    if (threadIdx.x == 0) a.wblk[(size_t)bi * nblk + blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void resample_w_kernel(const StepParams* __restrict__ sp, ResampleArgs a) {
    resample_w_slab(sp, a, a.nacc[blockIdx.y]);
}

// pass 3 for sequence bi, after n accepted tokens
__device__ __forceinline__ void resample_pick(const StepParams* __restrict__ sp, const ResampleArgs& a, int bi, int n, int32_t* len,
                                              int32_t* pending, const float* scores, const float* p_at_d, const int32_t* bits) {
    __shared__ double wave_tot[4];
    __shared__ double slab_w[256];
    __shared__ int hit_slab, last_slab;
    __shared__ double hit_before, last_before;
    const int tid = threadIdx.x, lane = tid & 63;
    const int b = sp->seq_base + bi;
    const int gamma = sp->gamma, nblk = a.nslab / 256;
    const int row = bi * (gamma + 1) + n;
    const float4 st = a.rowstat[row];
    if (sp->mirror && tid < gamma) {                 // gamma <= 63; written through, done when the launch is
        const int k = bi * gamma + tid;
        sp->mirror[k] = scores[k];
        sp->mirror[sp->mirror_stride + k] = p_at_d[k];
        sp->mirror[2 * sp->mirror_stride + k] = __int_as_float(bits[k]);
    }
    int next = -1;
    if (!(a.inv_temp > 0.f)) {
        next = __float_as_int(st.z);                 // one-hot target: residual and bonus are the arg-max
    } else {
        const double Z = total_of(a.eblk + (size_t)bi * nblk, nblk);
        double W = (n < gamma) ? total_of(a.wblk + (size_t)bi * nblk, nblk) : 0.0;
        const bool use_e = (n == gamma) || !(W > 0.0);
        const double* part = (use_e ? a.epart : a.wpart) + (size_t)bi * a.nslab;
        const double* blk = (use_e ? a.eblk : a.wblk) + (size_t)bi * nblk;
        if (use_e) W = Z;
        const double target = (double)sp->uniforms[(size_t)sp->step * sp->nseq + bi * (gamma + 1) + gamma] * W;
        if (tid == 0) { hit_slab = 0x7fffffff; last_slab = -1; }
        // level 1, every wave alike: the first workgroup sum whose range of the cumulative sum holds the target
        int owner = -1;
        double base = 0.0, carry = 0.0;
        for (int i0 = 0; i0 < nblk && owner < 0; i0 += 64) {
            const double mine = i0 + lane < nblk ? blk[i0 + lane] : 0.0;
            double incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const double t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            incl += carry;
            const double up = __shfl_up(incl, 1, 64);      // every lane takes part in the exchange
            const double excl = lane ? up : carry;
            const unsigned long long hit = __ballot(mine > 0.0 && target < incl);
            // the last range with weight takes what rounding leaves above the total
            const unsigned long long any = __ballot(mine > 0.0);
            if (hit) {
                owner = i0 + __builtin_ctzll(hit);
                base = __shfl(excl, __builtin_ctzll(hit), 64);
            } else if (i0 + 64 >= nblk && any && target == target) {
                const int l = 63 - __builtin_clzll(any);
                owner = i0 + l;
                base = __shfl(excl, l, 64);
            }
            carry = __shfl(incl, 63, 64);
        }
        __syncthreads();
        // level 2: the slab sums of that workgroup, scanned in slab order
        if (owner >= 0) {                                // uniform
            const double mine = part[owner * 256 + tid];
            double incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const double t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            if (lane == 63) wave_tot[tid >> 6] = incl;
            __syncthreads();
            double before = base;
            for (int w = 0; w < (tid >> 6); ++w) before += wave_tot[w];
            incl += before;
            const double up = __shfl_up(incl, 1, 64);
            const double excl = lane ? up : before;
            // one lane a wave speaks for it: 256 atomics on one LDS word took 3 us (the launch: 9.5 -> 6.0 us)
            const unsigned long long hit = __ballot(mine > 0.0 && target < incl), any = __ballot(mine > 0.0);
            if (lane == 0) {
                if (hit) atomicMin(&hit_slab, tid + __builtin_ctzll(hit));
                if (any) atomicMax(&last_slab, tid + 63 - __builtin_clzll(any));
            }
            __syncthreads();
            if (tid == hit_slab) hit_before = excl;
            if (tid == last_slab) last_before = excl;
            __syncthreads();
        }
        const bool have_slab = owner >= 0 && last_slab >= 0;
        const bool in_range = hit_slab != 0x7fffffff;
        const float mx = st.x;
        const float* l = a.logits + (size_t)row * a.V;
        const float* q = (n < gamma) ? sp->draft_probs + ((size_t)bi * gamma + n) * a.V : nullptr;
        auto weight = [&](int k) {
            const double e = e_of(l[k], mx, a.inv_temp);
            return use_e ? e : fmax(0.0, e - Z * (double)q[k]);
        };
        // level 3: the weights of the slab that holds the target, one per thread (slabs of up to 256 entries),
        // then scanned in vocabulary order by one thread
        const int hs = owner * 256 + (in_range ? hit_slab : last_slab);
        const int hk0 = have_slab ? hs * a.slab_len : 0, hk1 = have_slab ? min(a.V, hk0 + a.slab_len) : 0;
        const bool staged = have_slab && a.slab_len <= 256;
        if (staged && hk0 + tid < hk1) slab_w[tid] = weight(hk0 + tid);
        __syncthreads();
        if (tid == 0) {
            if (have_slab) {
                double c = in_range ? hit_before : last_before;
                int last_pos = -1;
                for (int k = hk0; k < hk1; ++k) {
                    const double v = staged ? slab_w[k - hk0] : weight(k);
                    if (v > 0.0) last_pos = k;
                    c += v;
                    if (c > target) { next = k; break; }
                }
                if (next < 0) next = last_pos;
            }
            if (next < 0) {            // no weight anywhere the sums say: last token with weight, else the arg-max
                for (int k = a.V - 1; k >= 0; --k)
                    if (weight(k) > 0.0) { next = k; break; }
                if (next < 0) next = __float_as_int(st.z);
            }
        }
    }
    if (tid == 0) {
        sp->next_token[bi] = next;
        len[b] += 1 + n;           // commit: rows beyond the new length are dead
        pending[b] = next;
        if (sp->emit_tokens) sp->emit_tokens[(size_t)bi * sp->emit_gamma + sp->step] = next;
    }
}

__global__ __launch_bounds__(256) void resample_pick_kernel(const StepParams* __restrict__ sp, ResampleArgs a,
                                                            int32_t* __restrict__ len, int32_t* __restrict__ pending,
                                                            const float* __restrict__ scores, const float* __restrict__ p_at_d,
                                                            const int32_t* __restrict__ bits) {
    resample_pick(sp, a, blockIdx.x, a.nacc[blockIdx.x], len, pending, scores, p_at_d, bits);
}

// Scan and all three passes in one launch (grid: 1 x sequences) where one workgroup holds the whole vocabulary (up to 4096 entries): what
// the passes leave for each other is the workgroup's own, and a barrier stands where a launch did (tiny model: 7.2 - 7.9 us, 13.2 in three
// launches and a gap).
__global__ __launch_bounds__(256) void scan_draw_kernel(const StepParams* __restrict__ sp, ResampleArgs a, const float* scores, float* p_at_d,
                                                        int32_t* bits, int32_t* nacc, const int32_t* ranks, int32_t* len, int32_t* pending) {
    __shared__ int n_sh;
    const int bi = blockIdx.y;
    if (threadIdx.x < 64) {
        const int n = accept_scan_seq(bi, threadIdx.x, true, sp, a.V, a.inv_temp, a.logits, a.rowstat, scores, p_at_d, bits, nacc, ranks);
        if (threadIdx.x == 0) n_sh = n;
    }
    __syncthreads();
    const int n = n_sh;
    resample_e_slab(sp, a, n, sp->emit_probs ? sp->emit_probs + ((size_t)bi * sp->emit_gamma + sp->step) * a.V : nullptr);
    __syncthreads();                                   // its sums are in memory
    if (n < sp->gamma) {                               // uniform
        resample_w_slab(sp, a, n);
        __syncthreads();
    }
    resample_pick(sp, a, bi, n, len, pending, scores, p_at_d, bits);
}

// Draft proposal (Eq. 1) at T = 0: the row's next-token law, one-hot at the arg-max, into column `step` of draft_probs
// [nseq][gamma][V].  (T > 0: pass 1 of the draw writes it; the token is written with the state in either case.)
__global__ __launch_bounds__(256) void draft_onehot_kernel(const StepParams* __restrict__ sp, int V, const float4* __restrict__ rowstat) {
    const int bi = blockIdx.y;
    float* q = sp->emit_probs;
    if (!q) return;
    q += ((size_t)bi * sp->emit_gamma + sp->step) * V;
    const int arg = __float_as_int(rowstat[bi].z);
    for (int k = blockIdx.x * 256 + threadIdx.x; k < V; k += gridDim.x * 256) q[k] = k == arg ? 1.f : 0.f;
}

// Teacher-forced scoring (Sec. 3.3, the terms of Eq. 7): log-probability of a given next token under every
// row's distribution, logp[r] = (l[r][t] - max) / T - log Z from the row's softmax statistics; T = 0: 0 for
// the arg-max, -inf otherwise.  Optionally copies the normed hidden state of row `hrow` of every sequence
// (the judge's feature of the token fed there, Eq. 4).
__global__ __launch_bounds__(256) void score_gather_kernel(int nseq, int rps, int V, int d, float inv_temp,
                                                           const float* __restrict__ logits, const float4* __restrict__ rowstat,
                                                           const int32_t* __restrict__ targets, float* __restrict__ logp,
                                                           const float* __restrict__ hn32, int hrow, float* __restrict__ hidden_out) {
    const int R = nseq * rps;
    for (int r = blockIdx.x * 256 + threadIdx.x; r < R; r += gridDim.x * 256) {
        const int t = min(max(targets[r], 0), V - 1);
        const float4 st = rowstat[r];
        logp[r] = (inv_temp > 0.f) ? (logits[(size_t)r * V + t] - st.x) * inv_temp - logf(st.y)
                                   : (t == __float_as_int(st.z) ? 0.f : -INFINITY);
    }
    if (hidden_out)
        for (int i = blockIdx.x * 256 + threadIdx.x; i < nseq * d; i += gridDim.x * 256)
            hidden_out[i] = hn32[((size_t)(i / d) * rps + hrow) * d + i % d];
}

// the cache rows of this call are kept: advance every sequence's length by rps
__global__ void advance_len_kernel(const StepParams* __restrict__ sp, int32_t* __restrict__ len) {
    const int bi = blockIdx.x * blockDim.x + threadIdx.x;
    if (bi < sp->nseq) len[sp->seq_base + bi] += sp->rps;
}

// Prefill bookkeeping: advance the length by the chunk; after the last chunk the pending token is the
// arg-max continuation of the last prompt token (the last of the head_rows rows that the LM head ran over).
__global__ void prefill_commit_kernel(const StepParams* __restrict__ sp, const float4* __restrict__ rowstat,
                                      int32_t* __restrict__ len, int32_t* __restrict__ pending, int last, int head_rows) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const int b = sp->seq_base;
        len[b] += sp->rps;
        if (last) pending[b] = __float_as_int(rowstat[head_rows - 1].z);
    }
}

}  // namespace sj
