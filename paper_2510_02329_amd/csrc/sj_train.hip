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
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/sj.h"
#include "sj_device.h"

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

using sj::f32x4;
using sj::lds_barrier;      // (__syncthreads() would also wait for the next rows' loads, which stay in flight across the barriers of the current ones)
using sj::vmcnt_imm;

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
    double* partial;                // [rows][slots][pcols + 2]: sum c h, sum c, sum of losses
    double* raw;                    // [slots][d + 2]
    int nslots;
    int nrows, pcols;               // rows of `partial`; its columns of a slot besides the two sums (d, or whole waves' slices in lane order: partial_col)
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

// v of this lane + v of the lane O behind it in its row of 16 (rotating)
template <int O>
__device__ __forceinline__ double block_sum(double v) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    const uint2 r{(unsigned)__builtin_amdgcn_update_dpp(0, (int)u.x, 0x120 + O, 0xf, 0xf, false), (unsigned)__builtin_amdgcn_update_dpp(0, (int)u.y, 0x120 + O, 0xf, 0xf, false)};
    return v + __builtin_bit_cast(double, r);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One pass over the matrix for the slots.  The eight waves of a workgroup share a group of RB rows, wave c owning the columns
// [c * NJ * 256, (c + 1) * NJ * 256).  Rows come through LDS by direct loads, each wave its own columns (1 KB of consecutive memory an
// instruction) into 16 KB of its own, so no wave waits for another's: the group that a wave has read into registers makes room at once for the
// one 16 KB later.  A wave's slices of the slots' vectors and
// accumulators are registers.  Per group: partial dot products of RB rows x slots -> LDS -> one barrier -> every wave finishes all
// coefficients itself (sigmoid only where a slot is in a gradient phase) and updates its columns.  Columns at or past d are loaded from a
// clamped address and meet x = 0; their accumulators are never used.  An idle slot rides along with a zero vector and zero coefficients.
// Bound: reads of the matrix (284 MB of 17358 x 4096: 41 us at 6.9 TB/s), the partial sums (34 MB written, 10 us), and 9 us of launch, first loads
// and end.  Launched back to back at that size, four slots, Hessian products: 84.5 us with the vectors in LDS, read there for every row, rows in two
// sets of registers, and the prologue's 32 loads each waited for in a branch of its own; 81.6 with rows through LDS and the prologue's loads
// together; 66 with the products on the matrix cores (below).  A grid of ten C at that size is 280 rounds of, in its trace, 59 us on average for this
// pass (the last rounds have idle slots), 8.6 for the sum of the partials and 7.8 for the slots' updates; vector units / matrix cores: 25.1 / 22.1 ms, one card
// in turn.
// This form, products on the vector units, is the one of d > 4096, where two slots' vectors and accumulators are all that fits (8000 x 8192:
// 68.1 -> 59.8 us a pass; 8000 x 5120: 40.1 -> 37.9).
constexpr int PASS_ROWS_MFMA = 4, PASS_ROWS_VALU = 2;                // rows of a group: a matrix block; at most 32 registers a buffer

__device__ __forceinline__ unsigned lds_addr(const void* p) { return (unsigned)(unsigned long long)(const __attribute__((address_space(3))) void*)p; }

// N pieces of 16 bytes a lane, STEP bytes apart in LDS, waited for in the same block.  As ordinary reads they would wait for every direct
// global->LDS load of the wave, since the compiler cannot tell which of them the data came with.
template <int STEP, int N> __device__ __forceinline__ void lds_read(f32x4 (&v)[N], unsigned at) {
    static_assert(N == 4 || N == 6 || N == 8, "pieces");
    if constexpr (N == 4)
        asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%5\n\tds_read_b128 %2, %4 offset:%6\n\tds_read_b128 %3, %4 offset:%7\n\t"
                     "s_waitcnt lgkmcnt(0)" : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP) : "memory");
    else if constexpr (N == 6)
        asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %6 offset:%7\n\tds_read_b128 %2, %6 offset:%8\n\tds_read_b128 %3, %6 offset:%9\n\t"
                     "ds_read_b128 %4, %6 offset:%10\n\tds_read_b128 %5, %6 offset:%11\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5])
                     : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP), "n"(4 * STEP), "n"(5 * STEP) : "memory");
    else
        asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:%9\n\tds_read_b128 %2, %8 offset:%10\n\tds_read_b128 %3, %8 offset:%11\n\t"
                     "ds_read_b128 %4, %8 offset:%12\n\tds_read_b128 %5, %8 offset:%13\n\tds_read_b128 %6, %8 offset:%14\n\t"
                     "ds_read_b128 %7, %8 offset:%15\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP), "n"(4 * STEP), "n"(5 * STEP), "n"(6 * STEP), "n"(7 * STEP) : "memory");
}

// The same for what the waves leave one another: a value written, and N values STEP bytes apart read.
__device__ __forceinline__ void lds_put(unsigned at, double v) { asm volatile("ds_write_b64 %0, %1" :: "v"(at), "v"(v) : "memory"); }
template <int STEP, int N> __device__ __forceinline__ void lds_get(double (&v)[N], unsigned at) {
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "waves that share a row");
    if constexpr (N == 1) asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v[0]) : "v"(at) : "memory");
    else if constexpr (N == 2)
        asm volatile("ds_read_b64 %0, %2\n\tds_read_b64 %1, %2 offset:%3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v[0]), "=&v"(v[1]) : "v"(at), "n"(STEP) : "memory");
    else if constexpr (N == 4)
        asm volatile("ds_read_b64 %0, %4\n\tds_read_b64 %1, %4 offset:%5\n\tds_read_b64 %2, %4 offset:%6\n\tds_read_b64 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP) : "memory");
    else
        asm volatile("ds_read_b64 %0, %8\n\tds_read_b64 %1, %8 offset:%9\n\tds_read_b64 %2, %8 offset:%10\n\tds_read_b64 %3, %8 offset:%11\n\t"
                     "ds_read_b64 %4, %8 offset:%12\n\tds_read_b64 %5, %8 offset:%13\n\tds_read_b64 %6, %8 offset:%14\n\tds_read_b64 %7, %8 offset:%15\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP), "n"(4 * STEP), "n"(5 * STEP), "n"(6 * STEP), "n"(7 * STEP) : "memory");
}

template <int NJ, int A>
__global__ __launch_bounds__(PASS_WAVES * 64) void lr_pass_kernel(TrainArgs a) {
    constexpr int RB = PASS_ROWS_VALU, CW = PASS_WAVES, Q = RB * A;
    constexpr int PIECES = RB * NJ, DEPTH = 16 / PIECES; // 1 KB pieces of a row group; groups that a wave's 16 KB of LDS hold
    __shared__ f32x4 ring[PASS_WAVES][DEPTH][PIECES][64];
    __shared__ double part[2][CW][Q];
    static_assert(DEPTH % 2 == 0, "the slots of `part` take turns");
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);

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
#pragma unroll
    for (int j = 0; j < NJ; ++j) off[j] = min((w * NJ + j) * 256 + lane * 4, a.d - 4);
    // the wave's slices of the vectors, all asked for at once (an idle slot's memory is there, too)
    double2 x2[NJ][A][2];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int s = 0; s < A; ++s) {
            x2[j][s][0] = *reinterpret_cast<const double2*>(xv[s] + off[j]);
            x2[j][s][1] = *reinterpret_cast<const double2*>(xv[s] + off[j] + 2);
        }
    // this lane's coefficient: row rb of the group, slot sl
    const int ql = lane / (64 / Q), sl = ql % A, rb_l = ql / A;
    int ph_l = PH_IDLE;
#pragma unroll
    for (int s = 0; s < A; ++s)
        if (s == sl) ph_l = ph[s];
    double xb_l = 0.0;                                   // its intercept
#pragma unroll
    for (int s = 0; s < A; ++s)
        if (s == sl) xb_l = ph[s] != PH_IDLE ? xv[s][a.d] : 0.0;
    double* Dl = a.D + (long long)sl * a.n;
    double accb = 0.0, loss = 0.0;

    const long long ngroups = (a.n + RB - 1) / RB;
    // D or the label of this lane's row, by two word loads (the label twice) that no branch and no conversion waits for
    const int32_t* aux_at = ph_l == PH_HESS ? reinterpret_cast<const int32_t*>(Dl) : a.y;
    const int wide = ph_l == PH_HESS ? 1 : 0;
    int alo[DEPTH], ahi[DEPTH];
    auto load = [&](int u, long long grp) {
        const long long g = grp < ngroups ? grp : ngroups - 1;   // groups past the end re-read the last (not used)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const long long i = g * RB + rb;
            const float* row = a.H + (i < a.n ? i : a.n - 1) * a.d;
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + off[j]),
                                                 (__attribute__((address_space(3))) void*)&ring[w][u][rb * NJ + j][0], 16, 0, 0);
        }
        const long long il = g * RB + rb_l < a.n ? g * RB + rb_l : a.n - 1;
        alo[u] = aux_at[il << wide];
        ahi[u] = aux_at[(il << wide) + wide];
    };
    // group numbers: blockIdx.x, + gridDim.x, ...  A slot of `part` is written again two turns later, after a barrier every wave passes only
    // once all its reads of the earlier turn are done.
    const long long G = gridDim.x, g0 = blockIdx.x;
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        load(u, g0 + u * G);
        asm volatile("" ::: "memory");                   // (the waits count a group's requests: they stay in front of the next group's)
    }
    double x[NJ][4][A], acc[NJ][4][A];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int s = 0; s < A; ++s) {
            asm volatile("" : "+v"(x2[j][s][0].x), "+v"(x2[j][s][0].y), "+v"(x2[j][s][1].x), "+v"(x2[j][s][1].y));   // (a load that only a branch uses would wait there)
            const bool in = ph[s] != PH_IDLE && (w * NJ + j) * 256 + lane * 4 < a.d;
            x[j][0][s] = in ? x2[j][s][0].x : 0.0;
            x[j][1][s] = in ? x2[j][s][0].y : 0.0;
            x[j][2][s] = in ? x2[j][s][1].x : 0.0;
            x[j][3][s] = in ? x2[j][s][1].y : 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[j][k][s] = 0.0;
        }
    auto process = [&](int u, long long grp) {
        f32x4 h[PIECES];
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((DEPTH - 1) * (PIECES + 2)));   // this group has landed (what else the wave asked for since only waits longer)
        lds_read<1024>(h, lds_addr(&ring[w][u][0][0]) + lane * 16);
        const int lo = alo[u], hi = ahi[u];
        load(u, grp + DEPTH * G);                        // the group's place is free
        double dot[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) dot[q] = 0.0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const double hd = h[rb * NJ + j][k];
#pragma unroll
                    for (int s = 0; s < A; ++s) dot[rb * A + s] += hd * x[j][k][s];
                }
        const double dq = wave_sums<Q>(dot, lane);
        const unsigned pt = lds_addr(&part[u & 1][0][ql]);
        if (lane % (64 / Q) == 0) lds_put(pt + w * (Q * 8), dq);
        lds_barrier();
        const long long i = grp * RB + rb_l;
        double zs[CW];
        lds_get<Q * 8>(zs, pt);
        double z = zs[0];
#pragma unroll
        for (int c = 1; c < CW; ++c) z += zs[c];
        z += xb_l;
        double c = 0.0;
        if (i < a.n) {
            if (ph_l == PH_HESS) c = __hiloint2double(hi, lo) * z;
            else if (ph_l != PH_IDLE) {
                const double aux = lo;
                const double sg = 1.0 / (1.0 + exp(-z));
                c = sg - aux;
                if (w == 0) {
                    const double m = aux > 0.5 ? -z : z; // -t z
                    loss += fmax(m, 0.0) + log1p(exp(-fabs(m)));
                    if (lane % (64 / Q) == 0) Dl[i] = sg * (1.0 - sg);
                }
            }
        }
        accb += c;
        // the update converts the row again: kept from the dot products, its doubles would be 16 registers a row and piece
#pragma unroll
        for (int p = 0; p < PIECES; ++p) asm volatile("" : "+v"(h[p]));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int s = 0; s < A; ++s) {
                const double cs = lane_value(c, (rb * A + s) * (64 / Q));
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc[j][k][s] += cs * (double)h[rb * NJ + j][k];
            }
    };
    for (long long grp = g0; grp < ngroups; grp += DEPTH * G)
#pragma unroll
        for (int u = 0; u < DEPTH; ++u)
            if (grp + u * G < ngroups) process(u, grp + u * G);   // uniform for the workgroup

    double* out = a.partial + (long long)blockIdx.x * A * (a.d + 2);
#pragma unroll
    for (int s = 0; s < A; ++s)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int e = (w * NJ + j) * 256 + lane * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (e + k < a.d) out[(long long)s * (a.d + 2) + e + k] = acc[j][k][s];
        }
    if (w == 0) {                                       // sums over the rows of a group, in row order
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

// The same pass with the products on the matrix cores, up to d = 4096: CW waves share a group of rows, wave c of them with NJ 256-column pieces, and
// the 8 / CW teams take neighbouring groups.  On the vector units a turn of four rows x four slots is 650 instructions
// a wave: 16 dot products to be summed over the lanes, 32 read-lanes of coefficients.  Here it is 200: four rows x four slots are one 4x4x4 block
// (four blocks an instruction, 256 multiply-adds in 8 ns a SIMD where 64 of the vector units' take 2.7), a dot product is one register pair a lane
//   dot:     D[row][slot] += A[row][column] B[column][slot]     (h, x)
//   update:  D[column][slot] += A[column][row] B[row][slot]     (h, c)
// Lane maps of v_mfma_f64_4x4x4_4b: A: i + 4 block + 16 k, B: j + 4 block + 16 k, D: j + 4 block + 16 i.  The dot's result, summed over the
// four blocks, is a lane's coefficient (slot lane % 4, row lane / 16) and then, as it stands, the update's B operand.  A lane holds a row's
// columns for the dot and a column's rows for the update: h is read from LDS once in either order, rows 64 bytes apart from a multiple of 256
// so that no bank is hit twice.  Column of MFMA (m, k) of a wave: m * 64 + 4 * (lane / 4) + k for the dot and x, m * 64 + 4 * (lane % 16) + k for the
// update's operand, m * 64 + 4 * (lane / 16 + 4 (lane / 4 % 4)) + k for the accumulators.
template <int NJ, int CW>
__global__ __launch_bounds__(PASS_WAVES * 64) void lr_pass_mfma_kernel(TrainArgs a) {
    constexpr int RB = PASS_ROWS_MFMA, A = 4, TEAMS = PASS_WAVES / CW, NM = NJ * 4;
    constexpr int DEPTH = 4 / NJ, ROW = NJ * 1024 + 64, GROUP = RB * ROW;    // groups in LDS; bytes of a row's slice, of a group's
    __shared__ __align__(16) unsigned char ring[PASS_WAVES * DEPTH * GROUP];
    __shared__ double part[2][TEAMS][CW][RB * A];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = w / CW, cw = w % CW;
    const int sl = lane & 3, rb_l = lane >> 4;           // this lane's coefficient: slot, row of the group
    bool any = false, gradient = false;
    for (int s = 0; s < a.nslots; ++s) {
        const int ph = a.slots[s].phase;
        any = any || ph != PH_IDLE;
        gradient = gradient || (ph != PH_IDLE && ph != PH_HESS);
    }
    if (!any) return;                                    // every problem is done (uniform for the launch)
    const int slot = min(sl, a.nslots - 1);
    const int ph_l = sl < a.nslots ? a.slots[slot].phase : PH_IDLE;
    const double* xv = a.vecs + ((long long)slot * V_COUNT + pass_vector(ph_l, a.slots[slot].flip)) * a.vstride;
    double* Dl = a.D + (long long)slot * a.n;

    double2 x2[NM][2];                                   // all asked for at once (an idle slot's memory is there, too)
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const double* at = xv + min(cw * NJ * 256 + m * 64 + (lane >> 2) * 4, a.d - 4);
        x2[m][0] = *reinterpret_cast<const double2*>(at);
        x2[m][1] = *reinterpret_cast<const double2*>(at + 2);
    }
    const double xb_l = xv[a.d];
    asm volatile("" ::: "memory");                       // (not behind the rows' requests)
    int off[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) off[j] = min((cw * NJ + j) * 256 + lane * 4, a.d - 4);
    double accb = 0.0, loss = 0.0;

    const long long ngroups = (a.n + RB - 1) / RB;
    // D or the label of this lane's row, by two word loads (the label twice) that no branch and no conversion waits for
    const int32_t* aux_at = ph_l == PH_HESS ? reinterpret_cast<const int32_t*>(Dl) : a.y;
    const int wide = ph_l == PH_HESS ? 1 : 0;
    int alo[DEPTH], ahi[DEPTH];
    unsigned char* mine = ring + w * DEPTH * GROUP;
    auto load = [&](int u, long long grp) {
        const long long g = grp < ngroups ? grp : ngroups - 1;   // groups past the end re-read the last (not used)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const long long i = g * RB + rb;
            const float* row = a.H + (i < a.n ? i : a.n - 1) * a.d;
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + off[j]),
                                                 (__attribute__((address_space(3))) void*)(mine + u * GROUP + rb * ROW + j * 1024), 16, 0, 0);
        }
        const long long il = g * RB + rb_l < a.n ? g * RB + rb_l : a.n - 1;
        alo[u] = aux_at[il << wide];
        ahi[u] = aux_at[(il << wide) + wide];
    };
    // group numbers of this team: blockIdx.x * TEAMS + team, + gridDim.x * TEAMS, ...; the number of turns is the workgroup's
    // (barriers inside): a team past the last group works on rows that do not count.  A slot of `part` is written again two
    // turns later, after a barrier every wave passes only once all its reads of the earlier turn are done.
    const long long G = (long long)gridDim.x * TEAMS;
    const long long g0 = (long long)blockIdx.x * TEAMS;
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        load(u, g0 + team + u * G);
        asm volatile("" ::: "memory");                   // (the waits count a group's requests: they stay in front of the next group's)
    }
    double x[NM][4], acc[NM][4];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        asm volatile("" : "+v"(x2[m][0].x), "+v"(x2[m][0].y), "+v"(x2[m][1].x), "+v"(x2[m][1].y));   // (a load that only a branch uses would wait there)
        const bool in = ph_l != PH_IDLE && cw * NJ * 256 + m * 64 + (lane >> 2) * 4 < a.d;
        x[m][0] = in ? x2[m][0].x : 0.0;
        x[m][1] = in ? x2[m][0].y : 0.0;
        x[m][2] = in ? x2[m][1].x : 0.0;
        x[m][3] = in ? x2[m][1].y : 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[m][k] = 0.0;
    }
    const double xb = ph_l != PH_IDLE ? xb_l : 0.0;

    auto process = [&](auto grad, int u, long long grp) {
        f32x4 h[NM], ht[NM];
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((DEPTH - 1) * (RB * NJ + 2)));   // this group has landed (what else the wave asked for since only waits longer)
        const unsigned at = lds_addr(mine + u * GROUP);
        lds_read<256>(h, at + sl * ROW + (lane >> 2) * 16);
        const int lo = alo[u], hi = ahi[u];
        auto free_place = [&]() {                        // the group's second order, and the next group into its place
            lds_read<256>(ht, at + rb_l * ROW + (lane & 15) * 16);
            load(u, grp + DEPTH * G);
        };
        if constexpr (!decltype(grad)::value) free_place();
        double dot[4] = {0.0, 0.0, 0.0, 0.0};            // four chains: a product waits for the one before it in its chain
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k) dot[k] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)h[m][k], x[m][k], dot[k], 0, 0, 0);
        double dq = (dot[0] + dot[1]) + (dot[2] + dot[3]);
        dq = block_sum<8>(dq);                           // over the four blocks
        dq = block_sum<4>(dq);
        const unsigned pt = lds_addr(&part[u & 1][team][0][rb_l * A + sl]);
        if ((lane & 12) == 0) lds_put(pt + cw * (RB * A * 8), dq);
        lds_barrier();
        const long long i = grp * RB + rb_l;
        double zs[CW];
        lds_get<RB * A * 8>(zs, pt);
        double z = zs[0];
#pragma unroll
        for (int c = 1; c < CW; ++c) z += zs[c];
        z += xb;
        double c = 0.0;
        if (i < a.n) {
            if (ph_l == PH_HESS) c = __hiloint2double(hi, lo) * z;
            else if (decltype(grad)::value && ph_l != PH_IDLE) {
                const double aux = lo;
                const double t = exp(-fabs(z)), inv = 1.0 / (1.0 + t), sg = z < 0.0 ? t * inv : inv;   // one exp for the sigmoid and the loss
                c = sg - aux;
                if (cw == 0) {
                    loss += fmax(aux > 0.5 ? -z : z, 0.0) + log1p(t);
                    if ((lane & 12) == 0) Dl[i] = sg * (1.0 - sg);
                }
            }
        }
        accb += c;
        if constexpr (decltype(grad)::value) {
            free_place();                                // (held since before exp and log1p, the 32 registers would have others spilled)
            asm volatile("" ::: "memory");               // (as above; in the other order the exchange is between this group's requests and the next wait)
        }
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[m][k] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)ht[m][k], c, acc[m][k], 0, 0, 0);
    };
    // a loop of its own for rounds of Hessian products only: the constants of exp and log1p are registers it does not have
    auto run = [&](auto grad) {
        for (long long grp = g0; grp < ngroups; grp += DEPTH * G)
#pragma unroll
            for (int u = 0; u < DEPTH; ++u)
                if (grp + u * G < ngroups) process(grad, u, grp + team + u * G);   // uniform for the workgroup
    };
    if (gradient) run(std::true_type{}); else run(std::false_type{});

    if (ph_l == PH_IDLE) return;
    // 256 bytes of a slot side by side in each store (in column order a lane's neighbours are 32 bytes apart: 6 us more a pass of 17358 x 4096)
    double* out = a.partial + (((long long)blockIdx.x * TEAMS + team) * a.nslots + sl) * (a.pcols + 2);
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int half = 0; half < 2; ++half)
            *reinterpret_cast<double2*>(out + ((cw * NM + m) * 2 + half) * 32 + (lane >> 2) * 2) = double2{acc[m][2 * half], acc[m][2 * half + 1]};
    if (cw == 0) {                                       // sums over the rows of a group, in row order
        double sb = 0.0, sls = 0.0;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            sb += __shfl(accb, rb * 16 + sl, 64);
            sls += __shfl(loss, rb * 16 + sl, 64);
        }
        if (lane < 4) {
            out[a.pcols] = sb;
            out[a.pcols + 1] = sls;
        }
    }
}
// column of position e of a slot's partial sums
__device__ __forceinline__ int partial_col(int e) {
    const int u = e % 32 / 2;
    return e / 64 * 64 + (u / 4 + u % 4 * 4) * 4 + e % 64 / 32 * 2 + e % 2;
}

// raw[s][column] = sum over the rows of `partial` (and the two sums behind the columns), in a fixed order: thread (slice q, position c) adds
// the rows of slice q of 16 in order, the 16 slice sums are then added in slice order.
template <bool LANES>
__global__ __launch_bounds__(1024) void lr_reduce_kernel(TrainArgs a) {
    __shared__ double sl[16][64];
    const int s = blockIdx.y;
    if (a.slots[s].phase == PH_IDLE) return;             // uniform
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + c, nv = a.pcols + 2;
    const double* p = a.partial + (long long)s * nv + (e < nv ? e : nv - 1);
    const int lo = q * a.nrows / 16, hi = (q + 1) * a.nrows / 16;
    double t = 0.0;
    for (int i0 = lo; i0 < hi; i0 += 16) {               // 16 independent loads (index clamped, surplus ignored)
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = p[(long long)min(i0 + i, hi - 1) * a.nslots * nv];
#pragma unroll
        for (int i = 0; i < 16; ++i) t += i0 + i < hi ? v[i] : 0.0;
    }
    sl[q][c] = t;
    __syncthreads();
    if (q == 0 && e < nv) {
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) r += sl[i][c];
        const int col = e >= a.pcols ? a.d + (e - a.pcols) : LANES ? partial_col(e) : e;
        if (e >= a.pcols || col < a.d) a.raw[(long long)s * (a.d + 2) + col] = r;
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
bool pass_mfma(int d) { return pass_shape(d).nj <= 2; }      // d <= 4096: the accumulators and vectors of four slots fit the registers
// Slots of a pass: as many problems as the registers allow (four up to d = 4096, two above), and no more than there are.
int pass_slots(int d, int n_C) {
    const int most = pass_mfma(d) ? MAX_SLOTS : 2;
    return n_C >= 3 ? most : n_C == 2 ? 2 : 1;
}

int launch_pass(const TrainArgs& a, int A, int grid, hipStream_t st) {
    const PassShape p = pass_shape(a.d);
#define SJ_PASS_MFMA(NJ, CW)                                                                          \
    if (p.nj == NJ && p.cw == CW) {                                                                   \
        lr_pass_mfma_kernel<NJ, CW><<<grid, PASS_WAVES * 64, 0, st>>>(a);                             \
        LAUNCHCHK("lr_pass_mfma");                                                                    \
        return SJ_OK;                                                                                 \
    }
    SJ_PASS_MFMA(1, 1) SJ_PASS_MFMA(1, 2) SJ_PASS_MFMA(1, 4) SJ_PASS_MFMA(1, 8) SJ_PASS_MFMA(2, 8)
#undef SJ_PASS_MFMA
#define SJ_PASS(NJ, AA)                                                                               \
    if (p.nj == NJ && A == AA) {                                                                      \
        lr_pass_kernel<NJ, AA><<<grid, PASS_WAVES * 64, 0, st>>>(a);                                  \
        LAUNCHCHK("lr_pass");                                                                         \
        return SJ_OK;                                                                                 \
    }
    SJ_PASS(3, 1) SJ_PASS(3, 2) SJ_PASS(4, 1) SJ_PASS(4, 2)
#undef SJ_PASS
    return fail(SJ_EINVAL, "d = %d above 8192 is not supported", a.d);
}

int launch_reduce(const TrainArgs& a, hipStream_t st) {
    const dim3 grid((a.pcols + 2 + 63) / 64, a.nslots);
    if (pass_mfma(a.d)) lr_reduce_kernel<true><<<grid, 1024, 0, st>>>(a);
    else lr_reduce_kernel<false><<<grid, 1024, 0, st>>>(a);
    LAUNCHCHK("lr_reduce");
    return SJ_OK;
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
    const int teams = PASS_WAVES / pass_shape(d).cw, rb = pass_mfma(d) ? PASS_ROWS_MFMA : PASS_ROWS_VALU;
    const int64_t turns = (n_train + (int64_t)rb * teams - 1) / ((int64_t)rb * teams);
    const int grid = (int)std::min<int64_t>(PASS_WG, turns);
    // validation runs over as many models at a time as 64 MB of scores and counts allow
    const int vm = (int)std::max<int64_t>(1, std::min<int64_t>(n_C, (int64_t)(64 << 20) / (16 * n_val)));

    Arena ar;
    ar.st = st;
    TrainArgs a{};
    a.H = H_train; a.y = y_train; a.n = n_train; a.d = d; a.n_C = n_C;
    a.vstride = d + 2;
    a.nslots = A;
    a.pcols = pass_mfma(d) ? pass_shape(d).cw * pass_shape(d).nj * 256 : d;
    a.nrows = grid * teams;
    double *C_dev, *score;
    int32_t *order_dev, *tp, *fp;
    long long* below2;
    ValResult* vres;
    ar.want(a.slots, (size_t)A);
    ar.want(a.vecs, (size_t)A * V_COUNT * a.vstride);
    ar.want(a.D, (size_t)A * n_train);
    ar.want(a.partial, (size_t)a.nrows * A * (a.pcols + 2));
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
            if ((rc = launch_reduce(a, st))) return rc;
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
