// Plain structs shared by the kernels and the host code: per-call parameters, model dimensions, cache view.
#pragma once
#include "sj_device.h"

namespace sj {

// Per-call parameters, kept in device memory so that a captured launch graph can be replayed with
// new caller pointers: only this struct is rewritten between replays.
struct StepParams {
    int32_t nseq;        // sequences processed by this call
    int32_t seq_base;    // first sequence index (prefill of one sequence: its index)
    int32_t rps;         // query rows per sequence (verify: gamma + 1; prefill: chunk length)
    int32_t gamma;       // draft length (verify only)
    int32_t tok_mode;    // 0: row 0 = pending token, rows 1.. = draft tokens; 1: rows = prefill tokens;
                         // 2: every row's token is given: draft_tokens [nseq, rps]
    int32_t mode;        // SJ_MODE_*
    float theta;         // judge threshold
    int32_t topk;        // k of the top-k mode
    const int32_t* draft_tokens;   // [nseq, gamma]
    const float* draft_probs;      // [nseq, gamma, V]
    const float* uniforms;         // [nseq, gamma + 1]
    int32_t* accepted_len;         // [nseq]
    int32_t* next_token;           // [nseq]
    const int32_t* prefill_tokens; // [rps] (tok_mode 1)
    int32_t step = -1;             // forwards since the parameters were set, counted by a forward's first kernel (a head-only
                                   // call has none: 0)
    int32_t emit_gamma;            // draft block: columns of emit_tokens / emit_probs
    int32_t* emit_tokens;          // draft block: [nseq, emit_gamma], column `step`
    float* emit_probs;             // draft block: [nseq, emit_gamma, V]
    float* mirror;                 // null, or host memory for the judge scores, p(draft) and accept bits, mirror_stride words each
    int32_t mirror_stride;
};

struct ModelDims {
    int32_t d, Hq, Hkv, hd, F, V, G;   // G = Hq / Hkv
    float eps, inv_temp, temperature, scale;   // scale = 1/sqrt(hd)
};

// KV cache view.  K and V of (layer, seq, kv head): `cap` positions in blocks of KSTEP (capacities are multiples of 64), each block
// the MFMA fragments that attention multiplies, in lane order (16 bytes a lane, 1 KB a fragment): a wave's load is consecutive
// memory.  (With rows of head-dim elements, and V as rows of positions, every lane's 16 bytes were a look-up of their own in the
// vector cache: 62 a load.)  K fragments [t][head-dim step]: row r of fragment t is key KF * (r / 4) + 4 t + r % 4 of the block,
// the order in which the accumulators of K . Q^T are the second product's operand; V fragments [16 head-dim columns]: rows are
// columns, the contraction runs over the block's keys.  seq_off[b] = element offset of sequence b inside one layer; layer_stride =
// elements per layer.
template <typename T>
__host__ __device__ __forceinline__ size_t kv_k_off(int pos, int c, int hd) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP;
    const int i = pos % KSTEP, r = i / KF * 4 + i % 4, t = i % KF / 4;
    return (size_t)(pos / KSTEP) * KSTEP * hd + (size_t)(((t * (hd / KSTEP) + c / KSTEP) * 4 + c % KSTEP / KF) * 16 + r) * KF + c % KF;
}
template <typename T>
__host__ __device__ __forceinline__ size_t kv_v_off(int pos, int c, int hd) {
    constexpr int KF = Traits<T>::KF, KSTEP = Traits<T>::KSTEP;
    const int i = pos % KSTEP;
    return (size_t)(pos / KSTEP) * KSTEP * hd + (size_t)((c / 16 * 4 + i / KF) * 16 + c % 16) * KF + i % KF;
}
template <typename T> struct KvView {
    T* K;
    T* V;
    const int64_t* seq_off;
    const int32_t* cap;
    int32_t* len;
    int32_t* pending;
    int64_t layer_stride;
};

}  // namespace sj
