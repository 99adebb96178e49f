// Attention tile for token generation (Fig. 2b with cached keys and values, one new token per
// sequence): one workgroup per (head, sequence).  There is a single query row, so the work is
// streaming the sequence's cached K and V rows once; the matrix cores have nothing to do here.
//
// The four waves split the keys: in every step a wave takes 16 consecutive keys, eight lanes
// per key and two keys per lane (each lane owns 16 of the 128 head dimensions, in two runs of 8, so that the eight read a
// 128-byte line of a row together; 16 + 16 values of state per lane leave the registers that the GeMM tile it shares
// a kernel with has for two steps of K and V rows).  Every lane keeps an
// online softmax of its own keys: running maximum m, sum l and 16 un-normalised output values.  At the end the lanes of
// a wave are brought to the wave's maximum and summed through LDS, then the four waves are
// combined the same way, the result is normalised, rounded and stored.  Key order: the cached
// tokens, then the new token's own key (which the QKV GeMM has just produced, like the query).
//
// A handful of (head, sequence) pairs cannot fill 256 CUs, and one workgroup walking thousands
// of keys is a chain of memory round trips, so the keys of a pair are split over `ksplit`
// workgroups (the stage's split, as for the GeMM tiles): each leaves its un-normalised result,
// maximum and sum in the scratch buffer and counts itself in, and the last to arrive combines
// the parts in key order, normalises, stores and posts.
#pragma once
#include <hip/hip_runtime.h>

#include "attn_tile.hpp"
#include "chain_args.h"
#include "sync_device.hpp"

namespace depsync {

constexpr int DEC_LDS_BYTES = 4 * 64 * 17 * 4 + 4 * 130 * 4;   // per-wave transposition areas + the waves' partial results
static_assert(DEC_LDS_BYTES <= ATT_LDS_BYTES, "the generation tile fits the LDS of the attention tile");

template <typename T, bool SYNC, class DR>
__device__ __forceinline__ void attn_decode_tile(const ChainArgs& args, const StageDesc& s, uint32_t head, uint32_t tyz,
                                                 uint32_t rel_ticket, char* lds, uint64_t t_enter, DR& dr) {
    typedef T T8 __attribute__((ext_vector_type(8)));
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = uni(tid >> 6);
    const uint32_t oct = lane & 7u, slot = lane >> 3;            // runs of the head dimensions, key slots (slot, slot + 8) in the step
    const uint32_t heads = uni(s.heads), E = heads * ATT_D;
    const uint32_t ld = uni(s.lda), ldt = uni(s.ldc);
    const uint32_t cached = uni(s.cached), ldkv = uni(s.ld_cache);
    const T* QKV = (const T*)uni_ptr(s.A);
    const T* Kc = (const T*)uni_ptr(s.kcache);
    const T* Vc = (const T*)uni_ptr(s.vcache);
    T* Tout = (T*)uni_ptr(s.C);
    const uint32_t KS = uni(s.ksplit);
    const uint32_t b = tyz / KS, ks = tyz % KS;                  // sequence, part of its keys
    const uint32_t row = b;                                      // seq = 1: the sequence's only new row

    const uint32_t n = cached + 1;                               // keys: the cache, then the new token
    const uint32_t chunk = ((n + KS - 1) / KS + 63u) & ~63u;     // keys per part, whole steps of 64
    const uint32_t k_begin = ks * chunk, k_end = min(n, k_begin + chunk);

    // Cached keys and values of a step, requested two steps before they are multiplied: with one step in flight a CU took in
    // 32 KB per round trip, and a part of 410 keys 10 to 22 us (7 to 16 so).  The first two are requested before the wait
    // (unless the caller wants no operand requested before its wait): nothing in the chain writes them.  Buffer loads, whose 32-bit offsets serve both operands: with 64-bit addresses the
    // three-per-CU kernels spilled 43 registers and lost more than the steps gained (25 chains of 1 to 16 sequences 1.4 %
    // slower than with one step in flight; so 6.3 % faster: four of 2048 tokens 67.8 -> 62.0 us, eleven of 1787 65.0 -> 55.5).
    // (The buffers end with the part's last key, so positions past it are zeros: their probability is zero, and zero times an
    // infinite value would not be.  A cache within a step of 4 GiB aside, whose last offsets wrap to its start.)
    const uint32_t pitch = ldkv * 2u, kc_end = min(k_end, cached);
    const uint32_t seq_off = b * cached * pitch + (head * ATT_D + oct * 8) * 2u;
    const uint32_t part_end = uni((b * cached + kc_end) * pitch);  // (caches are below 4 GiB: checked on the host)
    const OperandBuf bufK((const char*)Kc, part_end), bufV((const char*)Vc, part_end);
    struct Rows { T8 k[2][2], v[2][2]; };
    auto fetch = [&](uint32_t k0) __attribute__((always_inline)) {
        Rows x;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t off = seq_off + (k0 + slot + 8 * i) * pitch;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                x.k[i][c] = __builtin_bit_cast(T8, bufK.load16(off, c * 128));
                x.v[i][c] = __builtin_bit_cast(T8, bufV.load16(off, c * 128));
            }
        }
        return x;
    };
    WaitCtx wctx{&args, rel_ticket, true};
    const bool tracing = SYNC && (args.flags & DS_FLAG_TRACE) && args.trace != nullptr && rel_ticket < args.trace_cap;
    uint64_t t_start = 0, t_ready = 0;
    if (tracing) t_start = now_ticks();
    const uint32_t w_begin = k_begin + wave * 16;
    const bool reorder = !(args.flags & DS_FLAG_NO_REORDER);
    if (!reorder) attn_wait_qkv<SYNC>(wctx, s, head, row, row);
    Rows x0, x1;
    if (w_begin < kc_end) x0 = fetch(w_begin);
    if (w_begin + 64 < kc_end) x1 = fetch(w_begin + 64);
    if (reorder) attn_wait_qkv<SYNC>(wctx, s, head, row, row);
    if (tracing) t_ready = now_ticks();

    // this lane's part of the query, scaled to the base-2 softmax: 16 values
    const float sc = 0.08838834764831845f * 1.4426950408889634f;   // 1/sqrt(128) * log2(e)
    float q[16];
    {
        const T* qp = QKV + (size_t)row * ld + head * ATT_D + oct * 8;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const T8 v = *(const T8*)(qp + c * 64);
#pragma unroll
            for (int e = 0; e < 8; ++e) q[c * 8 + e] = (float)v[e] * sc;
        }
    }
    float o[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) o[j] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;
    auto step = [&](const Rows& x, uint32_t k0, uint32_t end) __attribute__((always_inline)) {
        float sv[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float dot = 0.0f;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e) dot = __builtin_fmaf(q[c * 8 + e], (float)x.k[i][c][e], dot);
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) dot += __shfl_xor(dot, d);   // the whole score, in all eight lanes
            sv[i] = k0 + slot + 8 * i < end ? dot : -INFINITY;
        }
        const float m_new = fmaxf(m_run, fmaxf(sv[0], sv[1]));
        const float m_use = (m_new == -INFINITY) ? 0.0f : m_new;  // no live key yet: keep the exponentials finite
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
        const float p0 = __builtin_amdgcn_exp2f(sv[0] - m_use), p1 = __builtin_amdgcn_exp2f(sv[1] - m_use);
        l_run = l_run * alpha + (p0 + p1);
        m_run = m_new;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float t = __builtin_fmaf(p0, (float)x.v[0][c][e], o[c * 8 + e] * alpha);
                o[c * 8 + e] = __builtin_fmaf(p1, (float)x.v[1][c][e], t);
            }
    };
    for (uint32_t k0 = w_begin; k0 < kc_end; k0 += 128) {        // (bounds that a wave's lanes share)
        step(x0, k0, kc_end);
        if (k0 + 128 < kc_end) x0 = fetch(k0 + 128);
        if (k0 + 64 >= kc_end) break;
        step(x1, k0 + 64, kc_end);
        if (k0 + 192 < kc_end) x1 = fetch(k0 + 192);
    }
    if (k_begin < n && k_end == n && wave == 0) {                // the new token's own key comes last
        const OperandBuf own(uni_ptr(QKV + (size_t)row * ld + E + head * ATT_D), uni((E + ATT_D) * 2u));
        const uint32_t off = slot == 0 ? oct * 16u : 0x7fffff00u;   // (the other slots: zeros)
        const T8 zero = {};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            x0.k[0][c] = __builtin_bit_cast(T8, own.load16(off, c * 128)); x0.k[1][c] = zero;
            x0.v[0][c] = __builtin_bit_cast(T8, own.load16(off, E * 2u + c * 128)); x0.v[1][c] = zero;
        }
        step(x0, 0, 1);
    }

    // ---- the wave's lanes to the wave's maximum, summed through LDS ----
    float m_w = m_run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) m_w = fmaxf(m_w, __shfl_xor(m_w, d));
    const float m_wu = (m_w == -INFINITY) ? 0.0f : m_w;
    const float f = __builtin_amdgcn_exp2f(m_run - m_wu);         // 0 for lanes that saw no live key
    float l_w = (oct == 0) ? l_run * f : 0.0f;                    // the eight lanes of a key hold the same l
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) l_w += __shfl_xor(l_w, d);
    float* const tr = reinterpret_cast<float*>(lds) + wave * (64 * 17);
    float* const part = reinterpret_cast<float*>(lds) + 4 * (64 * 17) + wave * 130;   // [128 values, m, l]
    __syncthreads();                                              // (uniform) the LDS is free: the last tile is done with it
#pragma unroll
    for (int j = 0; j < 16; ++j) tr[lane * 17 + j] = o[j] * f;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // this wave's writes are in LDS
    __builtin_amdgcn_wave_barrier();
    // each lane sums two of the 128 dimensions over the 8 key slots: dimension c * 64 + q * 8 + j lives in
    // the lanes 8 * slot + q, at position c * 8 + j
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t dim = 2 * lane + e, qd = (dim >> 3) & 7u, jj = (dim >> 6) * 8u + (dim & 7u);
        float acc = 0.0f;
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) acc += tr[(8 * sl + qd) * 17 + jj];
        part[dim] = acc;
    }
    if (lane == 0) { part[128] = m_w; part[129] = l_w; }
    dr.peek();
    __syncthreads();

    // ---- the four waves combined: thread t < 64 owns dimensions 2t, 2t+1 ----
    const float* const all = reinterpret_cast<const float*>(lds) + 4 * (64 * 17);
    float M = -INFINITY, L = 0.0f, r0 = 0.0f, r1 = 0.0f;
    if (tid < 64) {
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, all[w * 130 + 128]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = all[w * 130 + 128];
            const float g = (mw == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mw - M);
            L += all[w * 130 + 129] * g;
            r0 += all[w * 130 + 2 * tid] * g;
            r1 += all[w * 130 + 2 * tid + 1] * g;
        }
    }
    // ---- keys split over several workgroups: leave the part, carry on only as the last to arrive ----
    bool finish = true;
    if (KS > 1) {
        const uint32_t pair = b * heads + head;
        float* const parts = s.partials + (size_t)pair * KS * 130;
        if (tid < 64) {   // written through to memory, so that the count below can follow
            float* dst = parts + ks * 130;
            __hip_atomic_store(dst + 2 * tid, r0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(dst + 2 * tid + 1, r1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) {
                __hip_atomic_store(dst + 128, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(dst + 129, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        uint32_t* flag = reinterpret_cast<uint32_t*>(lds);        // the transposition areas are done with
        if (tid == 0) {
            const uint32_t old = __hip_atomic_fetch_add(s.arrive + pair * SYNC_WORD_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag[0] = old;
        }
        __syncthreads();
        finish = __builtin_amdgcn_readfirstlane(flag[0]) == KS - 1;
        __syncthreads();
        if (finish) {
            // every part is in memory (each counted after its stores had completed); combine in key order
            if (tid == 0) __hip_atomic_store(s.arrive + pair * SYNC_WORD_STRIDE, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid < 64) {
                M = -INFINITY;
                for (uint32_t z = 0; z < KS; ++z)
                    M = fmaxf(M, __hip_atomic_load(parts + z * 130 + 128, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                L = 0.0f; r0 = 0.0f; r1 = 0.0f;
                for (uint32_t z = 0; z < KS; ++z) {
                    const float* pz = parts + z * 130;
                    const float mz = __hip_atomic_load(pz + 128, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const float g = (mz == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mz - M);
                    L += __hip_atomic_load(pz + 129, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * g;
                    r0 += __hip_atomic_load(pz + 2 * tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * g;
                    r1 += __hip_atomic_load(pz + 2 * tid + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * g;
                }
            }
        }
    }
    // ---- normalised, rounded and stored ----
    if (finish && tid < 64 && wctx.ok) {
        const float inv = 1.0f / L;
        typedef T T2 __attribute__((ext_vector_type(2)));
        T2 pk;
        pk[0] = (T)(r0 * inv); pk[1] = (T)(r1 * inv);
        T* out = Tout + (size_t)row * ldt + head * ATT_D + 2 * tid;
        if constexpr (SYNC) {   // written through to memory, like every tile that posts
            uint32_t bits;
            __builtin_memcpy(&bits, &pk, 4);
            __hip_atomic_store(reinterpret_cast<uint32_t*>(out), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            *(T2*)out = pk;
        }
    }
    dr.grab();
    if (SYNC && finish) post_tile<true>(args, s, b * heads + head, head, b);
    if (tracing && tid == 0) {
        TraceRec r;
        r.rel = rel_ticket; r.where = hw_where(2u); r.tx = head; r.ty = tyz;
        r.t_enter = t_enter; r.t_start = t_start; r.t_ready = t_ready; r.t_end = now_ticks();
        args.trace[rel_ticket] = r;
    }
}

}  // namespace depsync
