// Training of the judge verifier on the device (paper Sec. 3.4 "Verifier Training" and appendix
// "Training Logistic Regressor"): L2-regularised logistic regression on (hidden state, label) pairs
// for every C of a grid, model selection by validation ROC-AUC, thresholds with the best F1 and the
// best recall.
//
//   f(w, b) = 1/2 |w|^2 + C sum_i log(1 + exp(-t_i (w.h_i + b))),  t_i = 2 y_i - 1   (bias unpenalised)
//
// f is strictly convex, so any solver reaches the same optimum; this one is a truncated Newton
// method: conjugate gradients on the Newton system, every gradient and every Hessian-vector product
// being ONE pass over the feature matrix (the only large object: n x d floats, HBM-bound):
//   per row i:  z_i = h_i . x + x_b;   c_i = sigmoid(z_i) - y_i   (gradient at x)
//                                   or c_i = D_i z_i,  D_i = s_i (1 - s_i)   (Hessian times x)
//   out += c_i h_i,  out_b += c_i
// The values of C are independent problems over the same matrix, so a pass serves several of them: up to
// four SLOTS each hold one problem and the vector it needs next (its point, its trial point or its search
// direction), and a pass multiplies every row with all of them.  What a problem does between passes - the
// conjugate-gradient update, the line search, the convergence tests, taking the next C - is decided on the
// device by a workgroup per slot, so a round is three launches (pass, sum of the partials, advance) without
// the host: it keeps rounds queued and looks at the number of finished problems every few of them.
// All arithmetic is fp64 on the fp32 features.  Sums are taken in a fixed order (rows of a workgroup, lanes,
// waves, workgroups) that does not depend on the slot, so a run is bit-reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <utility>
#include <vector>

#include "../../include/sj.h"

__attribute__((visibility("hidden"))) int sj_set_error(int code, const char* msg);   // defined next to sj_last_error

namespace {

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return sj_set_error(code, buf);
}

#define HIPCHK(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(SJ_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)
#define LAUNCHCHK(name)                                                                          \
    do {                                                                                         \
        hipError_t e_ = hipGetLastError();                                                       \
        if (e_ != hipSuccess) return fail(SJ_EHIP, "launch of %s failed: %s", name, hipGetErrorString(e_)); \
    } while (0)

// Workgroup barrier that waits for this wave's LDS traffic only: __syncthreads() would also wait for the
// next rows' loads, which are meant to stay in flight across the barriers of the current rows.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int PASS_WG = 256;        // workgroups of a pass: one per compute unit
constexpr int PASS_WAVES = 8;
constexpr int MAX_SLOTS = 4;
enum { PH_IDLE = 0, PH_START = 1, PH_HESS = 2, PH_TRIAL = 3 };   // what the slot's next pass is: -, gradient at 0, Hessian product, gradient at the trial point
enum { V_X = 0, V_G = 2, V_S = 4, V_R = 5, V_P = 6, V_COUNT = 7 };   // a slot's vectors: two points, two gradients, step, residual, direction

struct Slot {
    int phase, prob, flip;          // flip: which of the two point / gradient vectors is the current one
    int it, k, ls, passes;          // Newton iterations, conjugate-gradient steps, line-search trials, passes so far
    double C, tol, f, g0, gnorm, eta, rr, alpha, gs;
};
struct Fit { int converged, passes; };

struct TrainArgs {
    const float* H;                 // [n][d]
    const int32_t* y;               // [n]
    long long n;
    int d, n_C;
    Slot* slots;                    // [slots]
    double* vecs;                   // [slots][V_COUNT][vstride]
    long long vstride;
    double* D;                      // [slots][n] s (1 - s): written by a gradient pass, read by the Hessian passes
    double* partial;                // [rows][slots][d + 2]: sum c h, sum c, sum of losses
    double* raw;                    // [slots][d + 2]
    int nrows;                      // rows of `partial`
    const double* C_list;           // [n_C]
    const int32_t* order;           // problems in the order they are taken
    int32_t* queue;                 // next entry of `order`, and [1]: problems finished
    double* x_all;                  // [n_C][d + 1]
    Fit* fits;                      // [n_C]
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// the vector a slot's next pass multiplies the rows with
__device__ __forceinline__ int pass_vector(int phase, int flip) { return phase == PH_HESS ? V_P : V_X + (phase == PH_TRIAL ? 1 - flip : flip); }

// x summed over lane pairs O = 32 or 16 apart in the lanes below, y in the lanes above, by the swap of lane halves (of rows of 16
// lanes) that gfx950 does in one instruction a word; a shuffle takes two selects a word and a trip through the LDS unit.
template <int O>
__device__ __forceinline__ double swap_add(double x, double y) {
    const uint2 xu = __builtin_bit_cast(uint2, x), yu = __builtin_bit_cast(uint2, y);
    auto swap = [](unsigned p, unsigned q) {
        if constexpr (O == 32) return __builtin_amdgcn_permlane32_swap(p, q, false, false);
        else return __builtin_amdgcn_permlane16_swap(p, q, false, false);
    };
    const auto lo = swap(xu.x, yu.x), hi = swap(xu.y, yu.y);
    return __builtin_bit_cast(double, uint2{lo[0], hi[0]}) + __builtin_bit_cast(double, uint2{lo[1], hi[1]});
}

// Sums of Q values per lane over the wave, Q a power of two: every step halves the number of values a lane keeps and adds
// the other half's from the lane across, so Q sums cost Q - 1 + log2(64 / Q) exchanges instead of 6 Q.  The sum of value q
// ends in the lanes with lane / (64 / Q) == q.
template <int M, int Q>
__device__ __forceinline__ void halve_sums(double (&v)[Q], int lane) {
    if constexpr (M >= 1) {
        constexpr int o = 32 / (Q / 2 / M);
        const bool up = lane & o;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            if constexpr (o >= 16) v[q] = swap_add<o>(v[q], v[q + M]);
            else {
                const double send = up ? v[q] : v[q + M], keep = up ? v[q + M] : v[q];
                v[q] = keep + __shfl_xor(send, o, 64);
            }
        }
        halve_sums<M / 2, Q>(v, lane);
    }
}
template <int Q>
__device__ __forceinline__ double wave_sums(double (&v)[Q], int lane) {
    halve_sums<Q / 2, Q>(v, lane);
    double r = v[0];
#pragma unroll
    for (int o = 32 / Q; o > 0; o /= 2) r += __shfl_xor(r, o, 64);
    return r;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One pass over the matrix for A slots.  A workgroup of eight waves: CW of them share a group of RB rows, wave c of the CW
// owning the columns [c * NJ * 256, (c + 1) * NJ * 256) (lane l: elements 4l .. 4l + 3 of each of its NJ 256-column pieces, so
// every load instruction of a wave covers 1 KB of consecutive memory); the 8 / CW teams take neighbouring row groups.  A wave's
// slices of the A accumulators stay in registers, those of the vectors in LDS (d = 4096, A = 4: 64 registers and 128 KB; both
// in registers, next to two row buffers of 32, spilled and ran 99 us).  Per group: partial dot products of RB rows x A
// slots -> LDS -> one barrier -> every wave finishes all RB x A coefficients itself (lane q / Q; sigmoid only where a slot is in
// a gradient phase) and updates its columns.  The next group's loads (64 KB a CU) are issued before the current group is used.  Columns at
// or past d are loaded from a clamped address and meet x = 0; their accumulators are never stored.  An idle slot rides along
// with a zero vector and zero coefficients.
// Bound: reads of the matrix (284 MB of 17358 x 4096 in 50 us) and, above them, the chain of a group - dot products, wave
// sums, barrier, coefficients, update - which the two waves of a SIMD cross together.  Measured at that size with four slots:
// 79 us a pass = 20 us a problem, + 9 us for the sum of the partials and 8 us for the slots' updates; with one problem at a
// time a pass took 53 us, its vector kernels and the host's look at the result 65 us more.  A grid of ten C: 86 ms -> 26 ms.
// Converting a row once for dot product and update (32 registers more) measured the same.
// The exchanges across 32 and 16 lanes as swaps (swap_add): 74 -> 71 us a pass, ten C 26.4 -> 25.4 ms.  Groups of two rows with three
// buffers, so that the next group's dot products cover a group's exchange and barrier: 30.5 ms (the vectors are read from LDS for
// half as many rows).
constexpr int pass_rows(int nj) { return nj > 2 ? 2 : 4; }          // rows per group: at most 32 registers a buffer

template <int NJ, int A, int CW>
__global__ __launch_bounds__(PASS_WAVES * 64) void lr_pass_kernel(TrainArgs a) {
    constexpr int RB = pass_rows(NJ), TEAMS = PASS_WAVES / CW, Q = RB * A;
    __shared__ double2 xs[CW][NJ * 2 * A][64];           // the vectors: entry (4 j + k) A + s of a lane, in pairs
    __shared__ double part[2][TEAMS][CW][Q];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int team = w / CW, cw = w % CW;

    int ph[A];
    bool any = false;
    const double* xv[A];
#pragma unroll
    for (int s = 0; s < A; ++s) {
        ph[s] = a.slots[s].phase;
        any = any || ph[s] != PH_IDLE;
        xv[s] = a.vecs + ((long long)s * V_COUNT + pass_vector(ph[s], a.slots[s].flip)) * a.vstride;
    }
    if (!any) return;                                    // every problem is done (uniform for the launch)

    int off[NJ];
    double acc[NJ][4][A];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int e = (cw * NJ + j) * 256 + lane * 4;
        off[j] = min(e, a.d - 4);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int s = 0; s < A; ++s) {
                const int at = (4 * j + k) * A + s;
                reinterpret_cast<double*>(&xs[cw][at / 2][lane])[at % 2] = ph[s] != PH_IDLE && e + k < a.d ? xv[s][e + k] : 0.0;
                acc[j][k][s] = 0.0;
            }
    }
    // this lane's coefficient: row rb of the group, slot sl
    const int ql = lane / (64 / Q), sl = ql % A, rb_l = ql / A;
    int ph_l = PH_IDLE;
    double xb = 0.0;
#pragma unroll
    for (int s = 0; s < A; ++s)
        if (s == sl) { ph_l = ph[s]; xb = ph[s] != PH_IDLE ? xv[s][a.d] : 0.0; }
    double* Dl = a.D + (long long)sl * a.n;
    double accb = 0.0, loss = 0.0;

    const long long ngroups = (a.n + RB - 1) / RB;
    float4 bufA[RB][NJ], bufB[RB][NJ];
    double auxA = 0.0, auxB = 0.0;                       // label or D of this lane's row
    auto load = [&](float4 (&buf)[RB][NJ], double& aux, long long grp) {
        const long long g = grp < ngroups ? grp : ngroups - 1;   // groups past the end re-read the last (not used)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const long long i = g * RB + rb;
            const float* row = a.H + (i < a.n ? i : a.n - 1) * a.d;
#pragma unroll
            for (int j = 0; j < NJ; ++j) buf[rb][j] = *reinterpret_cast<const float4*>(row + off[j]);
        }
        const long long il = g * RB + rb_l < a.n ? g * RB + rb_l : a.n - 1;
        aux = ph_l == PH_HESS ? Dl[il] : (double)a.y[il];
    };
    auto process = [&](float4 (&buf)[RB][NJ], double aux, long long grp, int par) {
        double dot[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) dot[q] = 0.0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int k = 0; k < 4; k += 2) {             // two columns: 2 A doubles of x
                double x2[2 * A];
#pragma unroll
                for (int t = 0; t < A; ++t) {
                    const double2 v = xs[cw][(4 * j + k) * A / 2 + t][lane];
                    x2[2 * t] = v.x;
                    x2[2 * t + 1] = v.y;
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const double h0 = k ? buf[rb][j].z : buf[rb][j].x, h1 = k ? buf[rb][j].w : buf[rb][j].y;
#pragma unroll
                    for (int s = 0; s < A; ++s) dot[rb * A + s] += h0 * x2[s];
#pragma unroll
                    for (int s = 0; s < A; ++s) dot[rb * A + s] += h1 * x2[A + s];
                }
            }
        const double dq = wave_sums<Q>(dot, lane);
        if (lane % (64 / Q) == 0) part[par][team][cw][ql] = dq;
        lds_barrier();
        const long long i = grp * RB + rb_l;
        double z = part[par][team][0][ql];
#pragma unroll
        for (int c = 1; c < CW; ++c) z += part[par][team][c][ql];
        z += xb;
        double c = 0.0;
        if (i < a.n) {
            if (ph_l == PH_HESS) c = aux * z;
            else if (ph_l != PH_IDLE) {
                const double sg = 1.0 / (1.0 + exp(-z));
                c = sg - aux;
                if (cw == 0) {
                    const double m = aux > 0.5 ? -z : z; // -t z
                    loss += fmax(m, 0.0) + log1p(exp(-fabs(m)));
                    if (lane % (64 / Q) == 0) Dl[i] = sg * (1.0 - sg);
                }
            }
        }
        accb += c;
        // the update converts the row again: kept from the dot products, its doubles would be 16 registers a row and piece
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                asm volatile("" : "+v"(buf[rb][j].x), "+v"(buf[rb][j].y), "+v"(buf[rb][j].z), "+v"(buf[rb][j].w));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int s = 0; s < A; ++s) {
                const double cs = lane_value(c, (rb * A + s) * (64 / Q));
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    acc[j][0][s] += cs * (double)buf[rb][j].x;
                    acc[j][1][s] += cs * (double)buf[rb][j].y;
                    acc[j][2][s] += cs * (double)buf[rb][j].z;
                    acc[j][3][s] += cs * (double)buf[rb][j].w;
                }
            }
    };

    // group numbers of this team: blockIdx.x * TEAMS + team, + gridDim.x * TEAMS, ...; the number of turns is the workgroup's
    // (barriers inside): a team past the last group works on rows that do not count.  A slot of `part` is written again two
    // turns later, after a barrier every wave passes only once all its reads of the earlier turn are done.
    const long long G = (long long)gridDim.x * TEAMS;
    const long long g0 = (long long)blockIdx.x * TEAMS;
    load(bufA, auxA, g0 + team);
    __syncthreads();                                     // the vectors are in LDS
    for (long long grp = g0; grp < ngroups; grp += 2 * G) {
        load(bufB, auxB, grp + team + G);
        process(bufA, auxA, grp + team, 0);
        load(bufA, auxA, grp + team + 2 * G);
        if (grp + G < ngroups) process(bufB, auxB, grp + team + G, 1);   // uniform for the workgroup
    }

    double* out = a.partial + ((long long)blockIdx.x * TEAMS + team) * A * (a.d + 2);
#pragma unroll
    for (int s = 0; s < A; ++s)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int e = (cw * NJ + j) * 256 + lane * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (e + k < a.d) out[(long long)s * (a.d + 2) + e + k] = acc[j][k][s];
        }
    if (cw == 0) {                                       // sums over the rows of a group, in row order
        double sb = 0.0, sls = 0.0;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            sb += __shfl(accb, (rb * A + sl) * (64 / Q), 64);
            sls += __shfl(loss, (rb * A + sl) * (64 / Q), 64);
        }
        if (rb_l == 0 && lane % (64 / Q) == 0) {
            out[(long long)sl * (a.d + 2) + a.d] = sb;
            out[(long long)sl * (a.d + 2) + a.d + 1] = sls;
        }
    }
}

// raw[s][e] = sum over the rows of `partial` (e <= d + 1), in a fixed order: thread (slice q, column c) adds the rows of slice q
// of 16 in order, the 16 slice sums are then added in slice order.
__global__ __launch_bounds__(1024) void lr_reduce_kernel(TrainArgs a, int A) {
    __shared__ double sl[16][64];
    const int s = blockIdx.y;
    if (a.slots[s].phase == PH_IDLE) return;             // uniform
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + c, nv = a.d + 2;
    const double* p = a.partial + (long long)s * nv + (e < nv ? e : nv - 1);
    const int lo = q * a.nrows / 16, hi = (q + 1) * a.nrows / 16;
    double t = 0.0;
    for (int i0 = lo; i0 < hi; i0 += 16) {               // 16 independent loads (index clamped, surplus ignored)
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = p[(long long)min(i0 + i, hi - 1) * A * nv];
#pragma unroll
        for (int i = 0; i < 16; ++i) t += i0 + i < hi ? v[i] : 0.0;
    }
    sl[q][c] = t;
    __syncthreads();
    if (q == 0 && e < nv) {
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) r += sl[i][c];
        a.raw[(long long)s * nv + e] = r;
    }
}

__device__ __forceinline__ double block_sum_1024(double v, double* red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i];
    return t;
}
__device__ __forceinline__ double block_max_1024(double v, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) t = fmax(t, red[i]);
    return t;
}

// a slot takes the next problem of the queue: x = 0, gradient pass.  The whole workgroup calls it.
__device__ __forceinline__ void take_problem(const TrainArgs& a, Slot& S, double* vecs, int32_t* sh) {
    __syncthreads();
    if (threadIdx.x == 0) *sh = atomicAdd(&a.queue[0], 1);
    __syncthreads();
    const int q = *sh;
    S.phase = PH_IDLE;
    if (q < a.n_C) {
        S.phase = PH_START;
        S.prob = a.order[q];
        S.C = a.C_list[S.prob];
        S.tol = 1e-11 * fmax(1.0, S.C * (double)a.n);    // converged: max |g| <= tol
        S.flip = S.it = S.k = S.ls = S.passes = 0;
        S.f = S.g0 = S.gnorm = S.eta = S.rr = S.alpha = S.gs = 0.0;
        for (int e = threadIdx.x; e <= a.d; e += 1024) vecs[V_X * a.vstride + e] = 0.0;
    }
}

__global__ __launch_bounds__(1024) void lr_start_kernel(TrainArgs a) {
    __shared__ int32_t sh;
    Slot S{};
    take_problem(a, S, a.vecs + (long long)blockIdx.x * V_COUNT * a.vstride, &sh);
    if (threadIdx.x == 0) a.slots[blockIdx.x] = S;
}

// What a slot does with the result of its pass (one workgroup per slot; a thread owns EPT of the d + 1 unknowns, all loads are
// requested at once):
//   gradient:  g = (x_w, 0) + C raw, f = 1/2 |x_w|^2 + C loss.  At a trial point: the step is taken if f fell enough (near the
//              optimum the decrease is below the rounding of f: the step is taken), else it is halved.  At an accepted point:
//              converged, or conjugate gradients start on  Hess s = -g:  s = 0, r = p = -g.
//   Hessian:   q = (p_w, 0) + C raw;  alpha = rr / p.q;  s += alpha p;  r -= alpha q;  p = r + (r.r / rr) p.  Inexact Newton: the
//              system is solved to a tolerance that tightens with the gradient; then the first trial point x + s.
template <int EPT>
__global__ __launch_bounds__(1024) void lr_advance_kernel(TrainArgs a) {
    __shared__ double red[16];
    __shared__ int32_t sh;
    const int d = a.d, slot = blockIdx.x, tid = threadIdx.x;
    Slot S = a.slots[slot];
    if (S.phase == PH_IDLE) return;
    double* V = a.vecs + (long long)slot * V_COUNT * a.vstride;
    const double* raw = a.raw + (long long)slot * (d + 2);
    auto vec = [&](int k) { return V + (long long)k * a.vstride; };
    const double C = S.C;
    bool done = false, converged = false;
    double* x = vec(V_X + S.flip);                       // the current point

    if (S.phase == PH_HESS) {
        double *sv = vec(V_S), *rv = vec(V_R), *pv = vec(V_P);
        const double* gv = vec(V_G + S.flip);
        double pe[EPT], qe[EPT], re[EPT], se[EPT], pq = 0.0;
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = min(tid + 1024 * k, d);
            pe[k] = pv[e]; re[k] = rv[e]; se[k] = sv[e];
            qe[k] = raw[e];
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = tid + 1024 * k;
            qe[k] = (e < d ? pe[k] : 0.0) + C * qe[k];
            if (e <= d) pq += pe[k] * qe[k];
        }
        pq = block_sum_1024(pq, red);
        const double al = pq > 0.0 ? S.rr / pq : 0.0;
        double rn = 0.0;
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            se[k] += al * pe[k];
            re[k] -= al * qe[k];
            if (tid + 1024 * k <= d) rn += re[k] * re[k];
        }
        rn = block_sum_1024(rn, red);
        const double beta = S.rr > 0.0 ? rn / S.rr : 0.0;
        S.rr = rn;
        ++S.k;
        ++S.passes;
        if (!(sqrt(rn) <= S.eta * S.gnorm || pq <= 0.0 || S.k >= 4 * (d + 1) + 50)) {
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                const int e = tid + 1024 * k;
                if (e <= d) { sv[e] = se[k]; rv[e] = re[k]; pv[e] = re[k] + beta * pe[k]; }
            }
        } else {
            double gs = 0.0;
            double* xt = vec(V_X + 1 - S.flip);
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                const int e = tid + 1024 * k;
                if (e <= d) {
                    sv[e] = se[k];
                    gs += gv[e] * se[k];
                    xt[e] = x[e] + se[k];
                }
            }
            S.gs = block_sum_1024(gs, red);
            S.alpha = 1.0;
            S.ls = 0;
            S.phase = PH_TRIAL;
        }
    } else {
        const bool trial = S.phase == PH_TRIAL;
        const int at = trial ? 1 - S.flip : S.flip;
        const double* pt = vec(V_X + at);
        double* g = vec(V_G + at);
        double xe[EPT], ge[EPT], ww = 0.0, gg = 0.0, gm = 0.0;
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = min(tid + 1024 * k, d);
            xe[k] = e < d ? pt[e] : 0.0;
            ge[k] = raw[e];
        }
        const double lossv = raw[d + 1];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = tid + 1024 * k;
            ge[k] = xe[k] + C * ge[k];
            if (e <= d) {
                g[e] = ge[k];
                ww += xe[k] * xe[k];
                gg += ge[k] * ge[k];
                gm = fmax(gm, fabs(ge[k]));
            }
        }
        ww = block_sum_1024(ww, red);
        gg = block_sum_1024(gg, red);
        gm = block_max_1024(gm, red);
        const double f = 0.5 * ww + C * lossv;
        bool accepted = true;
        if (trial) {
            ++S.passes;
            accepted = f <= S.f + 1e-4 * S.alpha * S.gs || fabs(S.gs) <= 1e-9 * fabs(S.f);
            if (accepted) {
                S.flip ^= 1;
                x = vec(V_X + S.flip);
                ++S.it;
            }
        } else
            S.g0 = sqrt(gg);
        if (accepted) {
            if (S.it >= 100 || !isfinite(gg) || !isfinite(f)) done = true;   // a NaN gradient has no maximum: gm would be 0
            else if (gm <= S.tol) done = converged = true;
            else {
                S.f = f;
                S.gnorm = sqrt(gg);
                S.eta = fmin(0.1, sqrt(S.gnorm / fmax(S.g0, 1e-300)));
                S.rr = gg;
                S.k = 0;
                S.phase = PH_HESS;
                double *sv = vec(V_S), *rv = vec(V_R), *pv = vec(V_P);
#pragma unroll
                for (int k = 0; k < EPT; ++k) {
                    const int e = tid + 1024 * k;
                    if (e <= d) { sv[e] = 0.0; rv[e] = -ge[k]; pv[e] = -ge[k]; }
                }
            }
        } else if (++S.ls == 40) {
            done = true;                                 // no descent within rounding: the point is kept
        } else {
            S.alpha *= 0.5;
            const double* sv = vec(V_S);
            double* xt = vec(V_X + 1 - S.flip);
            for (int e = tid; e <= d; e += 1024) xt[e] = x[e] + S.alpha * sv[e];
        }
    }
    if (done) {                                          // uniform
        for (int e = tid; e <= d; e += 1024) a.x_all[(long long)S.prob * (d + 1) + e] = x[e];
        if (tid == 0) {
            a.fits[S.prob] = Fit{converged ? 1 : 0, S.passes};
            atomicAdd(&a.queue[1], 1);
        }
        take_problem(a, S, V, &sh);
    }
    __syncthreads();                                     // every thread has read the slot
    if (tid == 0) a.slots[slot] = S;
}

// ---- validation: ROC-AUC by its pair definition, F1 of every candidate threshold --------------------
// score[m][i] = sigmoid(h_i . w_m + b_m): one wave per row, the model in LDS (at most 64 KB)
__global__ __launch_bounds__(256) void val_scores_kernel(const float* __restrict__ H, long long n, int d, const double* __restrict__ x_all,
                                                         double* __restrict__ score) {
    extern __shared__ double xs[];
    const double* x = x_all + (long long)blockIdx.y * (d + 1);
    for (int e = threadIdx.x; e < d; e += 256) xs[e] = x[e];
    const double xb = x[d];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += 4LL * gridDim.x) {
        const float* row = H + i * d;
        double z = 0.0;
        for (int e = lane * 4; e < d; e += 256) {
            const float4 h = *reinterpret_cast<const float4*>(row + e);
            z += (double)h.x * xs[e] + (double)h.y * xs[e + 1] + (double)h.z * xs[e + 2] + (double)h.w * xs[e + 3];
        }
        z = wave_sum(z) + xb;
        if (lane == 0) score[(long long)blockIdx.y * n + i] = 1.0 / (1.0 + exp(-z));
    }
}

// Model m = blockIdx.z of the launch (counting) or blockIdx.x (selection).  Candidate i < n is theta = score_i, candidate n is theta = 0.  For each candidate:
//   tp = #{acceptable j: score_j > theta},  fp = #{unacceptable j: score_j > theta};
// for an acceptable sample i also  below2 = 2 #{unacceptable j: score_j < score_i} + #{... == score_i}.
__global__ __launch_bounds__(256) void val_count_kernel(long long n, const double* __restrict__ score, const int32_t* __restrict__ y,
                                                        int want_f1, int32_t* __restrict__ tp, int32_t* __restrict__ fp,
                                                        long long* __restrict__ below2) {
    __shared__ double ss[256];
    __shared__ int32_t ys[256];
    score += blockIdx.z * n;
    below2 += blockIdx.z * n;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const double si = i < n ? score[i] : 0.0;              // candidate n: theta = 0
    const bool pos_i = i < n && y[i] != 0;
    int ctp = 0, cfp = 0;
    long long b2 = 0;
    // blockIdx.y takes every gridDim.y-th tile of j; the counts are integers, so the order of the atomic
    // additions does not matter
    for (long long j0 = (long long)blockIdx.y * 256; j0 < n; j0 += 256LL * gridDim.y) {
        __syncthreads();
        const long long j = j0 + threadIdx.x;
        ss[threadIdx.x] = j < n ? score[j] : -1.0;         // scores are in [0, 1]: -1 never counts
        ys[threadIdx.x] = j < n ? y[j] : -1;
        __syncthreads();
        const int m = (int)((n - j0) < 256 ? (n - j0) : 256);
        for (int k = 0; k < m; ++k) {
            const double sj = ss[k];
            const bool pj = ys[k] != 0;
            if (want_f1) { ctp += (pj && sj > si); cfp += (!pj && sj > si); }
            if (!pj) b2 += (sj < si) ? 2 : (sj == si ? 1 : 0);
        }
    }
    if (i <= n && want_f1) { atomicAdd(&tp[i], ctp); atomicAdd(&fp[i], cfp); }
    if (i < n && pos_i) atomicAdd(reinterpret_cast<unsigned long long*>(&below2[i]), (unsigned long long)b2);
}

struct ValResult {
    unsigned long long auc2;      // 2 * (pairs ordered correctly) + ties
    long long n_pos, n_neg;
    double f1, theta_f1, theta_recall;
};

__global__ __launch_bounds__(1024) void val_select_kernel(long long n, const double* __restrict__ score, const int32_t* __restrict__ y,
                                                          int want_f1, const int32_t* __restrict__ tp, const int32_t* __restrict__ fp,
                                                          const long long* __restrict__ below2, ValResult* __restrict__ out) {
    __shared__ unsigned long long s_auc[1024];
    __shared__ long long s_pos[1024];
    __shared__ double s_f1[1024], s_th[1024], s_neg[1024];
    score += blockIdx.x * n;
    below2 += blockIdx.x * n;
    out += blockIdx.x;
    unsigned long long auc2 = 0;
    long long npos = 0;
    double negmax = 0.0;
    for (long long i = threadIdx.x; i < n; i += 1024) {
        auc2 += (unsigned long long)below2[i];
        npos += y[i] != 0;
        if (y[i] == 0) negmax = fmax(negmax, score[i]);
    }
    s_auc[threadIdx.x] = auc2; s_pos[threadIdx.x] = npos; s_neg[threadIdx.x] = negmax;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            s_auc[threadIdx.x] += s_auc[threadIdx.x + o];
            s_pos[threadIdx.x] += s_pos[threadIdx.x + o];
            s_neg[threadIdx.x] = fmax(s_neg[threadIdx.x], s_neg[threadIdx.x + o]);
        }
        __syncthreads();
    }
    const long long total_pos = s_pos[0];
    // best F1, the smallest threshold among equals: F1 = 2 tp / (2 tp + fp + fn), fn = n_pos - tp
    double bf = -1.0, bt = 0.0;
    if (want_f1)
        for (long long i = threadIdx.x; i <= n; i += 1024) {
            const double t = (double)tp[i];
            const double f1 = tp[i] == 0 ? 0.0 : 2.0 * t / (2.0 * t + (double)fp[i] + (double)(total_pos - tp[i]));
            const double th = i < n ? score[i] : 0.0;
            if (f1 > bf || (f1 == bf && th < bt)) { bf = f1; bt = th; }
        }
    s_f1[threadIdx.x] = bf; s_th[threadIdx.x] = bt;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            const double f1 = s_f1[threadIdx.x + o], th = s_th[threadIdx.x + o];
            if (f1 > s_f1[threadIdx.x] || (f1 == s_f1[threadIdx.x] && th < s_th[threadIdx.x])) { s_f1[threadIdx.x] = f1; s_th[threadIdx.x] = th; }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out->auc2 = s_auc[0];
        out->n_pos = total_pos;
        out->n_neg = n - total_pos;
        out->f1 = s_f1[0];
        out->theta_f1 = s_th[0];
        out->theta_recall = s_neg[0];
    }
}

// ---- host side -----------------------------------------------------------------------------------------
// Device memory of one call: one allocation, carved up after all pieces are known.
struct Arena {
    char* base = nullptr;
    size_t used = 0;
    std::vector<std::pair<void**, size_t>> pieces;
    hipStream_t st = nullptr;
    int32_t* done_host = nullptr;                        // pinned: finished problems as of two batches of rounds
    hipEvent_t ev[2] = {nullptr, nullptr};
    ~Arena() {
        if (base || done_host) (void)hipStreamSynchronize(st);
        if (base) (void)hipFree(base);
        if (done_host) (void)hipHostFree(done_host);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
    template <typename T> void want(T*& p, size_t count) {
        pieces.emplace_back(reinterpret_cast<void**>(&p), used);
        used = (used + count * sizeof(T) + 255) / 256 * 256;
    }
    int get() {
        hipError_t e = hipMalloc(reinterpret_cast<void**>(&base), used);
        if (e != hipSuccess) return fail(e == hipErrorOutOfMemory ? SJ_ENOMEM : SJ_EHIP, "hipMalloc(%zu) failed: %s", used, hipGetErrorString(e));
        for (auto& p : pieces) *p.first = base + p.second;
        HIPCHK(hipHostMalloc(reinterpret_cast<void**>(&done_host), 2 * sizeof(int32_t), hipHostMallocDefault));
        for (hipEvent_t& e2 : ev) HIPCHK(hipEventCreateWithFlags(&e2, hipEventDisableTiming));
        return SJ_OK;
    }
};

// Columns of a row are spread over as many waves as 256-column pieces ask for (all eight from d > 1024 on, with up to four
// pieces each); narrow rows leave waves over, which take further rows.
struct PassShape { int nj, cw; };
PassShape pass_shape(int d) {
    const int pieces = (d + 255) / 256;
    if (pieces <= 1) return {1, 1};
    if (pieces <= 2) return {1, 2};
    if (pieces <= 4) return {1, 4};
    return {(pieces + 7) / 8, 8};
}
// Slots of a pass: as many problems as the registers allow (four up to d = 4096, two above), and no more than there are.
int pass_slots(int d, int n_C) {
    const int most = pass_shape(d).nj <= 2 ? MAX_SLOTS : 2;
    return n_C >= 3 ? most : n_C == 2 ? 2 : 1;
}

int launch_pass(const TrainArgs& a, int A, int grid, hipStream_t st) {
    const PassShape p = pass_shape(a.d);
#define SJ_PASS(NJ, CW, AA)                                                                           \
    if (p.nj == NJ && p.cw == CW && A == AA) {                                                        \
        lr_pass_kernel<NJ, AA, CW><<<grid, PASS_WAVES * 64, 0, st>>>(a);                              \
        LAUNCHCHK("lr_pass");                                                                         \
        return SJ_OK;                                                                                 \
    }
#define SJ_PASS3(NJ, CW) SJ_PASS(NJ, CW, 1) SJ_PASS(NJ, CW, 2) SJ_PASS(NJ, CW, 4)
    SJ_PASS3(1, 1) SJ_PASS3(1, 2) SJ_PASS3(1, 4) SJ_PASS3(1, 8) SJ_PASS3(2, 8)
    SJ_PASS(3, 8, 1) SJ_PASS(3, 8, 2) SJ_PASS(4, 8, 1) SJ_PASS(4, 8, 2)
#undef SJ_PASS3
#undef SJ_PASS
    return fail(SJ_EINVAL, "d = %d above 8192 is not supported", a.d);
}

int launch_advance(const TrainArgs& a, int A, hipStream_t st) {
    const int ept = (a.d + 1 + 1023) / 1024;
    if (ept <= 1) lr_advance_kernel<1><<<A, 1024, 0, st>>>(a);
    else if (ept <= 3) lr_advance_kernel<3><<<A, 1024, 0, st>>>(a);
    else if (ept <= 5) lr_advance_kernel<5><<<A, 1024, 0, st>>>(a);
    else lr_advance_kernel<9><<<A, 1024, 0, st>>>(a);
    LAUNCHCHK("lr_advance");
    return SJ_OK;
}

}  // namespace

extern "C" int sj_judge_train(const float* H_train, const int32_t* y_train, int64_t n_train, const float* H_val,
                              const int32_t* y_val, int64_t n_val, int32_t d, const double* C_grid, int32_t n_C,
                              double* w_all, double* auc, int32_t* passes, int32_t* best_index, double* w_best,
                              double* theta_f1, double* theta_recall, void* stream) {
    if (!H_train || !y_train || !H_val || !y_val || !C_grid || !auc || !best_index || !w_best || !theta_f1 || !theta_recall)
        return fail(SJ_EINVAL, "null argument");
    if (n_train < 2 || n_val < 2 || n_C < 1) return fail(SJ_EINVAL, "need at least two samples per set and one C");
    if (n_val > (1 << 24)) return fail(SJ_EINVAL, "validation set above 2^24 samples is not supported");
    if (d < 4 || d % 4 || d > 8192) return fail(SJ_EINVAL, "d must be a multiple of 4 in 4 .. 8192");
    if (((uintptr_t)H_train | (uintptr_t)H_val) & 15) return fail(SJ_EINVAL, "feature matrices must be 16-byte aligned");
    for (int c = 0; c < n_C; ++c)
        if (!(C_grid[c] > 0.0) || !std::isfinite(C_grid[c])) return fail(SJ_EINVAL, "C[%d] must be positive and finite", c);
    hipStream_t st = (hipStream_t)stream;

    // labels: 0 / 1, both classes in both sets (the optimum does not exist otherwise)
    std::vector<int32_t> lab((size_t)(n_train > n_val ? n_train : n_val));
    for (int pass = 0; pass < 2; ++pass) {
        const int64_t n = pass ? n_val : n_train;
        HIPCHK(hipMemcpyAsync(lab.data(), pass ? y_val : y_train, (size_t)n * 4, hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        int64_t ones = 0;
        for (int64_t i = 0; i < n; ++i) {
            if (lab[i] != 0 && lab[i] != 1) return fail(SJ_EINVAL, "label %lld of the %s set is %d (must be 0 or 1)", (long long)i, pass ? "validation" : "training", lab[i]);
            ones += lab[i];
        }
        if (ones == 0 || ones == n) return fail(SJ_EINVAL, "the %s set holds one class only", pass ? "validation" : "training");
    }

    // the largest C first: they take the most passes, and the slots run dry together at the end
    std::vector<int32_t> order((size_t)n_C);
    for (int c = 0; c < n_C; ++c) order[c] = c;
    std::stable_sort(order.begin(), order.end(), [&](int32_t p, int32_t q) { return C_grid[p] > C_grid[q]; });

    const int A = pass_slots(d, n_C);
    const int teams = PASS_WAVES / pass_shape(d).cw, rb = pass_rows(pass_shape(d).nj);
    const int64_t turns = (n_train + (int64_t)rb * teams - 1) / ((int64_t)rb * teams);
    const int grid = (int)std::min<int64_t>(PASS_WG, turns);
    // validation runs over as many models at a time as 64 MB of scores and counts allow
    const int vm = (int)std::max<int64_t>(1, std::min<int64_t>(n_C, (int64_t)(64 << 20) / (16 * n_val)));

    Arena ar;
    ar.st = st;
    TrainArgs a{};
    a.H = H_train; a.y = y_train; a.n = n_train; a.d = d; a.n_C = n_C;
    a.vstride = d + 2;
    a.nrows = grid * teams;
    double *C_dev, *score;
    int32_t *order_dev, *tp, *fp;
    long long* below2;
    ValResult* vres;
    ar.want(a.slots, (size_t)A);
    ar.want(a.vecs, (size_t)A * V_COUNT * a.vstride);
    ar.want(a.D, (size_t)A * n_train);
    ar.want(a.partial, (size_t)a.nrows * A * (d + 2));
    ar.want(a.raw, (size_t)A * (d + 2));
    ar.want(C_dev, (size_t)n_C);
    ar.want(order_dev, (size_t)n_C);
    ar.want(a.queue, 2);
    ar.want(a.x_all, (size_t)n_C * (d + 1));
    ar.want(a.fits, (size_t)n_C);
    ar.want(score, (size_t)vm * n_val);
    ar.want(below2, (size_t)vm * n_val);
    ar.want(tp, 2 * ((size_t)n_val + 1));
    ar.want(vres, (size_t)vm);
    int rc;
    if ((rc = ar.get())) return rc;
    fp = tp + n_val + 1;
    a.C_list = C_dev;
    a.order = order_dev;
    HIPCHK(hipMemcpyAsync(C_dev, C_grid, (size_t)n_C * sizeof(double), hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(order_dev, order.data(), (size_t)n_C * sizeof(int32_t), hipMemcpyHostToDevice, st));
    HIPCHK(hipMemsetAsync(a.queue, 0, 2 * sizeof(int32_t), st));
    lr_start_kernel<<<A, 1024, 0, st>>>(a);
    LAUNCHCHK("lr_start");

    // Rounds are queued in batches; the host waits for the batch before the last, so the device always has one to work on.
    // Every problem ends after at most 100 iterations of at most 4 (d + 1) + 50 + 40 passes; rounds after the last one return at once.
    constexpr int BATCH = 8;
    for (int64_t batch = 0;; ++batch) {
        for (int r = 0; r < BATCH; ++r) {
            if ((rc = launch_pass(a, A, grid, st))) return rc;
            lr_reduce_kernel<<<dim3((d + 2 + 63) / 64, A), 1024, 0, st>>>(a, A);
            LAUNCHCHK("lr_reduce");
            if ((rc = launch_advance(a, A, st))) return rc;
        }
        HIPCHK(hipMemcpyAsync(ar.done_host + (batch & 1), a.queue + 1, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIPCHK(hipEventRecord(ar.ev[batch & 1], st));
        if (batch == 0) continue;
        HIPCHK(hipEventSynchronize(ar.ev[(batch - 1) & 1]));
        if (ar.done_host[(batch - 1) & 1] == n_C) break;
    }
    std::vector<Fit> fits((size_t)n_C);
    HIPCHK(hipMemcpyAsync(fits.data(), a.fits, (size_t)n_C * sizeof(Fit), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    int good = 0;                                        // the models before the first that did not converge
    while (good < n_C && fits[good].converged) ++good;
    for (int c = 0; c < good && passes; ++c) passes[c] = fits[c].passes;
    if (w_all && good) HIPCHK(hipMemcpyAsync(w_all, a.x_all, (size_t)good * (d + 1) * sizeof(double), hipMemcpyDeviceToHost, st));

    // validation of `count` models from c0 on (their scores, and the counts of the requested kind) into host_res
    const unsigned xb = (unsigned)((n_val + 1 + 255) / 256), yb = xb >= 1024 ? 1 : (1024 + xb - 1) / xb;   // about 1024 workgroups a model
    auto validate = [&](int c0, int count, int want_f1, ValResult* host_res) -> int {
        // about 1024 workgroups in all (four to a CU at d = 4096, by the model's LDS): one model over 120000 rows of 4096 features
        // takes 0.36 ms = 5.5 TB/s, with 64 workgroups it took 3.5 ms
        const unsigned sb = (unsigned)std::min<int64_t>(std::max(64, (1024 + count - 1) / count), (n_val + 3) / 4);
        val_scores_kernel<<<dim3(sb, count), 256, (size_t)d * sizeof(double), st>>>(H_val, n_val, d, a.x_all + (size_t)c0 * (d + 1), score);
        LAUNCHCHK("val_scores");
        HIPCHK(hipMemsetAsync(below2, 0, (size_t)count * n_val * sizeof(long long), st));
        if (want_f1) HIPCHK(hipMemsetAsync(tp, 0, 2 * ((size_t)n_val + 1) * sizeof(int32_t), st));
        val_count_kernel<<<dim3(xb, std::max(1u, yb / (unsigned)count), count), 256, 0, st>>>(n_val, score, y_val, want_f1, tp, fp, below2);
        LAUNCHCHK("val_count");
        val_select_kernel<<<count, 1024, 0, st>>>(n_val, score, y_val, want_f1, tp, fp, below2, vres);
        LAUNCHCHK("val_select");
        HIPCHK(hipMemcpyAsync(host_res, vres, count * sizeof(ValResult), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        return SJ_OK;
    };
    std::vector<ValResult> vr((size_t)std::max(good, 1));
    int best = -1;
    for (int c0 = 0; c0 < good; c0 += vm)
        if ((rc = validate(c0, std::min(vm, good - c0), 0, vr.data() + c0))) return rc;
    for (int c = 0; c < good; ++c) {
        auc[c] = (double)vr[c].auc2 / (2.0 * (double)vr[c].n_pos * (double)vr[c].n_neg);
        if (best < 0 || vr[c].auc2 > vr[best].auc2) best = c;   // equal AUC keeps the earlier C
    }
    if (good < n_C) return fail(SJ_EHIP, "the solver did not converge for C[%d] = %g", good, C_grid[good]);
    if ((rc = validate(best, 1, 1, vr.data()))) return rc;
    HIPCHK(hipMemcpyAsync(w_best, a.x_all + (size_t)best * (d + 1), (size_t)(d + 1) * sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    *best_index = best;
    *theta_f1 = vr[0].theta_f1;
    *theta_recall = vr[0].theta_recall;
    return SJ_OK;
}
