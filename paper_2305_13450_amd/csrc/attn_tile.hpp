// Middle stage of the attention chain (Fig. 2b of the paper, prompt phase: no cached keys or
// values, dropout is the identity): one tile computes, for one head and one block of 128 query
// rows of one sequence,  T = softmax(Q K^T / sqrt(d) + causal mask) V  with d = 128,
// flash-attention style (keys/values streamed in blocks of 64, running maximum and sum).
//
// MFMA formulation.  Everything is computed transposed so that a lane owns ONE query:
//   S^T[key][q] = K[key][:] . Q[q][:]      A operand = K block (LDS), B operand = Q (registers)
//   O^T[d][q]  += V^T[d][key] P^T[key][q]   A operand = V^T block (LDS), B operand = P^T, which
// is exactly what the S^T accumulators hold: for v_mfma_f32_32x32x16 a lane owns column
// (lane % 32) and rows 8*(v/4) + 4*(lane/32) + v%4, so the 8 accumulator values v0..v0+7 of a
// lane are 8 keys of its query, and since the order of the 16 K-slots of an MFMA is free as
// long as both operands agree, they can be fed straight back as the B operand while V^T is
// read with the same key permutation: runs of 4 keys of one d, which the transposing LDS read
// (ds_read_b64_tr_b16) gathers from rows of V as they lie in memory.  Row maxima and sums are in-lane
// reductions plus one exchange between the two half-waves.
//
// Dependencies: the tile reads the Q columns of its own rows and the K and V columns of all
// rows of its sequence up to its last row, from the QKV GeMM before it; it posts like any
// producer tile (grid: x = head, y = query block) for the output GeMM after it.
#pragma once
#include <hip/hip_runtime.h>

#include "chain_args.h"
#include "gemm_tile.hpp"
#include "sync_device.hpp"

namespace depsync {

constexpr int ATT_BLK_BYTES = ATT_BK * ATT_D * 2;       // one block of K or V rows (16 KB)
constexpr int ATT_LDS_BYTES = 4 * ATT_BLK_BYTES;        // rings of at least two K and two V blocks

// Position of the 16-byte chunk of row `key` of V in its LDS row.  A transposing read takes, per group of
// 16 lanes, 32 bytes of each of 4 consecutive keys (64 bytes with the neighbouring group): the low
// bits of the key choose the 64-byte window, so that those 4 keys lie in different banks.
__device__ __forceinline__ uint32_t att_vswz(uint32_t key) { return ((key & 3u) << 2) | ((key >> 2) & 3u); }

// Four 16-bit elements per lane, transposed: the 16 lanes of a group address a 4 x 16 tile (lane i: row
// i / 4, elements 4 * (i % 4) ..), and lane i receives column i.
template <typename T> struct TrRead;
template <> struct TrRead<__bf16> {
    typedef __bf16 T4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ T4 read(const char* p) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) T4*)(p));
    }
};
template <> struct TrRead<_Float16> {
    typedef _Float16 T4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ T4 read(const char* p) {
        typedef __fp16 H4 __attribute__((ext_vector_type(4)));
        return __builtin_bit_cast(T4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((__attribute__((address_space(3))) H4*)(p)));
    }
};

// Wait for everything an attention tile reads from the QKV GeMM: rows row_first .. row_last, in this
// head's Q, K and V columns.
template <bool SYNC>
__device__ __forceinline__ void attn_wait_qkv(WaitCtx& w, const StageDesc& s, uint32_t head, uint32_t row_first,
                                              uint32_t row_last) {
    if (!SYNC || s.dep_kind == DEP_NONE) return;
    const uint32_t target = s.sem_target_base + s.sem_value;
    attn_for_each_wait(s, head, row_first, row_last, [&](uint32_t x, uint32_t y) __attribute__((always_inline)) {
        const uint32_t* sem = s.sems + policy_sem(s.dep_kind, x, y, s.prod_grid_y, s.stride) * SYNC_WORD_STRIDE;
        const uint32_t v = sem_load(sem);
        const bool polled = !sem_reached(v, target);
        if (polled) sem_wait(w, sem, target, v);
        count_wait(*w.args, polled);
    });
}

// Floats one part of a tile split along the keys leaves in the scratch buffer: the un-normalised
// O^T accumulators of the 256 lanes (64 each), then every lane's running maximum and sum.
constexpr uint32_t ATT_PART_FLOATS = 256 * 64 + 2 * 256;

// What bounds it: the longest tiles of a causal stage are one serial chain of key blocks, walked by one
// wave per SIMD: per block 32 MFMAs (0.5 us), 32 scores per lane through exp2 and conversion (as
// much again), and all four waves reading the whole block from LDS.  So V is transposed by the read
// (writing V^T back to LDS element by element took longer than everything else together), a block has
// one barrier, half of the next block's scores are multiplied beside the exponentials, and the
// operands' offsets fit few registers (with more, the loop reloaded them from scratch memory and waited
// for the DMA in flight each time).  12 heads, 2048 tokens, bf16: the longest tile (32 blocks) 185 -> 76 to
// 84 us (two boards), of which about 20 are waits for K and V; the whole chain 438 -> 372 us by this.
// NBUF: blocks in the LDS rings of K and V: 4 where the tile has the CU to itself, 2 where two workgroups
// share it (and cover each other's waits).
template <typename T, bool SYNC, int NBUF, class DR>
__device__ __forceinline__ void attn_tile(const ChainArgs& args, const StageDesc& s, uint32_t head, uint32_t tyz,
                                          uint32_t rel_ticket, char* lds, uint64_t t_enter, DR& dr) {
    using M = Mma<T>;
    using V8 = typename M::V8;
    typedef T T4 __attribute__((ext_vector_type(4)));

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = uni(tid >> 6);
    const uint32_t h2 = lane >> 5, lq = lane & 31u;
    const uint32_t seq = uni(s.seq), heads = uni(s.heads);
    const uint32_t E = heads * ATT_D;
    const uint32_t ld = uni(s.lda), ldt = uni(s.ldc);
    // A long causal tile is one dependent chain of key blocks, so the stage may split every tile's
    // keys over KS workgroups (the stage's split, as for the GeMM tiles): part z takes a run of
    // whole key blocks, leaves un-normalised results, maxima and sums in the scratch buffer and
    // counts itself in; the last part to arrive combines the parts in key order, normalises,
    // stores and posts.  Tiles of few key blocks use fewer parts (the rest find nothing to do).
    const uint32_t KS = uni(s.ksplit);
    // cached keys and values of this sequence come first in key order
    const uint32_t cached = uni(s.cached), ldkv = uni(s.ld_cache);
    const AttnSpan span = attn_span(tyz, KS, seq, cached);
    const uint32_t qblk = span.qblk, part = span.part, nparts = span.nparts;
    const uint32_t seq_row0 = span.seq_row0, b = seq_row0 / seq;  // first row of the sequence, sequence
    const uint32_t q0 = span.q0, q_last = span.q_last;            // first and last query (inside the sequence)
    const uint32_t kb_begin = span.kb_begin, kb_end = span.kb_end;
    const T* QKV = (const T*)uni_ptr(s.A);
    T* Tout = (T*)uni_ptr(s.C);
    const T* Kc = (const T*)uni_ptr(s.kcache);
    const T* Vc = (const T*)uni_ptr(s.vcache);

    WaitCtx wctx{&args, rel_ticket, true};
    const bool tracing = SYNC && (args.flags & DS_FLAG_TRACE) && args.trace != nullptr && rel_ticket < args.trace_cap;
    uint64_t t_start = 0, t_ready = 0;
    if (tracing) t_start = now_ticks();

    if (part >= nparts) {                                          // nothing for this part: the tile is short
        if (tracing && tid == 0) {
            TraceRec r;
            r.rel = rel_ticket; r.where = hw_where(2u); r.tx = head; r.ty = tyz;
            r.t_enter = t_enter; r.t_start = t_start; r.t_ready = t_start; r.t_end = now_ticks();
            args.trace[rel_ticket] = r;
        }
        return;
    }

    attn_wait_qkv<SYNC>(wctx, s, head, seq_row0, seq_row0 + q_last);
    if (tracing) t_ready = now_ticks();

    // ---- this lane's query row as the B operand of S^T = K Q^T: 8 fragments of 8 d values ----
    const uint32_t qi = q0 + wave * 32 + lq;                      // query index inside the sequence
    const uint32_t qrow = seq_row0 + min(qi, seq - 1);
    V8 qf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
        qf[kk] = *(const V8*)(QKV + (size_t)qrow * ld + head * ATT_D + kk * 16 + h2 * 8);

    f32x16 o[4];                                                   // O^T: 4 blocks of 32 d x this lane's query
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;                         // reference value and sum of this query's weights
    const float sc = 0.08838834764831845f * 1.4426950408889634f;   // 1/sqrt(128) * log2(e)

    // LDS: NBUF blocks of K rows and NBUF of V rows ([64 keys][128 d], 16-byte chunks swizzled), DMA'd
    // from global memory.  Step kb multiplies the scores of block kb+1 and the values of block kb, so
    // it requests K of block kb+NBUF and V of block kb+NBUF-1 into the slots the step before has left.
    // The compiler waits for every DMA in flight before a transposing read, so with slots to spare
    // the requests go out behind the step's last such read and have a whole step to land.
    constexpr bool LATE = NBUF > 2;
    const uint32_t wave_q_first = min(q0 + wave * 32, seq - 1);
    const uint32_t wave_q_last = min(q0 + wave * 32 + 31, seq - 1);
    char* const ldsK = lds;
    char* const ldsV = lds + NBUF * ATT_BLK_BYTES;
    // a lane's 16 bytes of rows tid/16, tid/16 + 16, .. of a block (both swizzles repeat every 16 rows)
    const uint32_t frow = tid >> 4;
    const uint32_t fck = ((tid & 15u) ^ frow) * 16u, fcv = ((tid & 15u) ^ att_vswz(frow)) * 16u;
    const OperandBuf bufN((const char*)QKV), bufC((const char*)(cached ? Kc : QKV)), bufCV((const char*)(cached ? Vc : QKV));
    auto fetch = [&](uint32_t kb, bool v) __attribute__((always_inline)) {
        char* dst = (v ? ldsV : ldsK) + (kb % NBUF) * ATT_BLK_BYTES + wave * 1024;
        const uint32_t k0 = kb * ATT_BK, fc = v ? fcv : fck;      // position in key order: cache first
        const uint32_t colN = ((v ? 2 * E : E) + head * ATT_D) * 2u, colC = head * ATT_D * 2u;
        if (attn_block_in_one_run(k0, cached, q_last)) {
            const bool in_cache = k0 < cached;
            const uint32_t pitch = 2u * (in_cache ? ldkv : ld), off = frow * pitch + fc;
            const uint32_t first = in_cache ? (b * cached + k0) * pitch + colC : (seq_row0 + k0 - cached) * pitch + colN;
            if (in_cache) {
#pragma unroll
                for (int i = 0; i < 4; ++i) (v ? bufCV : bufC).dma16(off, first + (uint32_t)i * 16u * pitch, dst + i * 4096);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) bufN.dma16(off, first + (uint32_t)i * 16u * pitch, dst + i * 4096);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t key = k0 + i * 16 + frow;
                if (key < cached) (v ? bufCV : bufC).dma16((b * cached + key) * (2u * ldkv) + colC + fc, 0, dst + i * 4096);
                else bufN.dma16((seq_row0 + attn_key_row(key, cached, q_last)) * (2u * ld) + colN + fc, 0, dst + i * 4096);
            }
        }
    };
    // Per-lane LDS offsets.  K fragments are rows lq (and 32 + lq), chunk 2 * kk + h2; V fragments are
    // transposed reads of 4 keys x 16 d per 16 lanes (key 4 * h2 + .., and 8 further on; 32 d further on
    // per block of d).  The swizzles are exclusive-ors, so one offset serves all fragments of an operand.
    const uint32_t koff = lq * 256u + ((h2 ^ (lq & 15u)) << 4);
    const uint32_t vkey = 4u * h2 + ((lane & 15u) >> 2);
    const uint32_t voff = vkey * 256u + (((((lane >> 4) & 1u) * 2u + ((lane & 3u) >> 1)) ^ att_vswz(vkey)) << 4) + (lane & 1u) * 8u;
    // S^T of one 32-key half of block kb, with `between(kk)` after the MFMA of each 16-wide slice kk of d.
    // Fragments are read two slices ahead and the order is pinned: left alone the compiler reads each
    // fragment right before the wait for it.
    auto scores = [&](uint32_t kb, int kh, auto&& between) __attribute__((always_inline)) {
        const uint32_t k = (kb % NBUF) * ATT_BLK_BYTES + koff;
        V8 kf[3];
        auto rd = [&](int kk) __attribute__((always_inline)) { kf[kk % 3] = *(const V8*)(ldsK + (k ^ (kk * 32u)) + kh * (32 * 256)); };
        rd(0); rd(1);
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            __builtin_amdgcn_sched_barrier(0);
            if (kk + 2 < 8) rd(kk + 2);
            acc = M::mma(kf[kk % 3], qf[kk], acc);
            between(kk);
        }
        __builtin_amdgcn_sched_barrier(0);
        return acc;
    };
    auto request = [&](uint32_t kb) __attribute__((always_inline)) {   // what step kb requests
        if (kb + NBUF < kb_end) fetch(kb + NBUF, false);
        if (kb + NBUF - 1 < kb_end) fetch(kb + NBUF - 1, true);
    };
    // Everything step kb reads has landed for every wave, and every wave is done with the slots its
    // requests go into.
    auto arrive = [&](uint32_t kb) __attribute__((always_inline)) {
        if (LATE && kb + NBUF - 1 < kb_end) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * (NBUF - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

#pragma unroll
    for (int p = 0; p < NBUF; ++p) {                               // in the order the steps before kb_begin would have requested them
        if (p > 0 && kb_begin + p - 1 < kb_end) fetch(kb_begin + p - 1, true);
        if (p == 0 || kb_begin + p < kb_end) fetch(kb_begin + p, false);
    }
    // the scores of the first block: its K rows are the oldest request
    if (kb_begin + NBUF - 1 < kb_end) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * (NBUF - 1)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x16 st[2];
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) st[kh] = scores(kb_begin, kh, [](int) {});

    // Blocks above a wave's diagonal contribute nothing to it: it only keeps the others company.
    const uint32_t kb_live = min(kb_end, (cached + wave_q_last) / ATT_BK + 1);
    uint32_t kb = kb_begin;
    for (; kb < kb_live; ++kb) {
        const uint32_t k0 = kb * ATT_BK;
        arrive(kb);
        if (!LATE) request(kb);
        // ---- causal mask (blocks on the diagonal and at the end only), running maximum ----
        if (k0 + ATT_BK - 1 > cached + wave_q_first) {
#pragma unroll
            for (int kh = 0; kh < 2; ++kh)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t key = k0 + kh * 32 + 8 * (v / 4) + 4 * h2 + (v % 4);
                    if (key > cached + qi || key >= cached + seq) st[kh][v] = -INFINITY;
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, st[kh][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * sc;
        const float m_new = fmaxf(m_run, mx);
        // a query beyond the sequence end or with no visible key yet keeps m = -inf: guard the exps
        const float m_use = (m_new == -INFINITY) ? 0.0f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);   // arguments are <= 0 or -inf: v_exp_f32 as is
        m_run = m_new;
        // ---- weights of this block, relative to the largest seen (which 16 bits then hold exactly: a reference
        // that lags behind the maximum, to save the rescaling of O, left errors 1 % larger), summed in 32 bits
        // before they are rounded for the product with V.  The first half's registers then take the next
        // block's scores, whose MFMAs run beside the exponentials of the second half and the rescaling of O (past the
        // wave's last block they multiply whatever the slot holds, and nothing reads the result) ----
        V8 pf[4];
        float psum = 0.0f;
        auto weight = [&](int kh, int v) __attribute__((always_inline)) {
#pragma clang fp contract(off)
            const float p = __builtin_amdgcn_exp2f(st[kh][v] * sc - m_use);   // the largest score gives exactly 1
            psum += p;
            pf[kh * 2 + (v >> 3)][v & 7] = (T)p;
        };
#pragma unroll
        for (int v = 0; v < 16; ++v) weight(0, v);
        st[0] = scores(kb + 1, 0, [&](int kk) __attribute__((always_inline)) { weight(1, 2 * kk); weight(1, 2 * kk + 1); });
        psum += __shfl_xor(psum, 32);
        l_run = l_run * alpha + psum;
        st[1] = scores(kb + 1, 1, [&](int kk) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 8; ++v) o[kk >> 1][(kk & 1) * 8 + v] *= alpha;
        });
        // ---- O^T += V^T P^T : 4 steps of 16 keys, fragments of a step read while the one before is multiplied ----
        const uint32_t vb = (kb % NBUF) * ATT_BLK_BYTES + voff;
        T4 vf[2][4][2];
        auto rdv = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
            for (int db = 0; db < 4; ++db)                         // keys 16*ks + 4*h2 ..+3 and 16*ks + 8 + 4*h2 ..+3 of 32 d
#pragma unroll
                for (int c = 0; c < 2; ++c) vf[ks & 1][db][c] = TrRead<T>::read(ldsV + (vb ^ (db * 64u + c * 32u)) + (ks * 16 + c * 8) * 256);
        };
        rdv(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            if (ks < 3) rdv(ks + 1);
#pragma unroll
            for (int db = 0; db < 4; ++db)
                o[db] = M::mma(__builtin_shufflevector(vf[ks & 1][db][0], vf[ks & 1][db][1], 0, 1, 2, 3, 4, 5, 6, 7), pf[ks], o[db]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (LATE) request(kb);
    }
    for (; kb < kb_end; ++kb) {
        arrive(kb);
        request(kb);
    }

    dr.peek();   // the look at the dispatch queues for the next tile travels while the result is stored
    // ---- keys split over several workgroups: leave the part, carry on only as the last to arrive ----
    bool finish = true;
    if (nparts > 1) {
        const uint32_t tile_lin = qblk * heads + head;
        float* const parts = s.partials + (size_t)tile_lin * KS * ATT_PART_FLOATS;
        float* const mine = parts + (size_t)part * ATT_PART_FLOATS;
        // fragment order, 16 bytes per lane next to its neighbours', written through to memory so
        // that the count below can follow
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                const f32x2 v2 = {o[i][2 * q], o[i][2 * q + 1]};
                uint64_t bits;
                __builtin_memcpy(&bits, &v2, 8);
                __hip_atomic_store(reinterpret_cast<uint64_t*>(mine + (((i * 8 + q) * 256 + tid) << 1)), bits, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        __hip_atomic_store(mine + 256 * 64 + 2 * tid, m_run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(mine + 256 * 64 + 2 * tid + 1, l_run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                                           // every wave's part is in memory; the K and V buffers are done with
        uint32_t* flag = reinterpret_cast<uint32_t*>(lds);
        if (tid == 0) {
            const uint32_t old = __hip_atomic_fetch_add(s.arrive + tile_lin * SYNC_WORD_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag[0] = old;
        }
        __syncthreads();
        finish = __builtin_amdgcn_readfirstlane(flag[0]) == nparts - 1;
        __syncthreads();
        if (finish) {
            // every part is in memory (each counted after its stores had completed): combine in key
            // order, whoever came last, so that the result does not depend on the arrival order
            if (tid == 0) __hip_atomic_store(s.arrive + tile_lin * SYNC_WORD_STRIDE, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            float m_all = -INFINITY;
            for (uint32_t z = 0; z < nparts; ++z)
                m_all = fmaxf(m_all, __hip_atomic_load(parts + (size_t)z * ATT_PART_FLOATS + 256 * 64 + 2 * tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            const float m_use = (m_all == -INFINITY) ? 0.0f : m_all;
            l_run = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[i][v] = 0.0f;
            for (uint32_t z = 0; z < nparts; ++z) {
                const float* pz = parts + (size_t)z * ATT_PART_FLOATS;
                const float mz = __hip_atomic_load(pz + 256 * 64 + 2 * tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const float lz = __hip_atomic_load(pz + 256 * 64 + 2 * tid + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const float g = (mz == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mz - m_use);
                l_run += lz * g;
                uint64_t t2[32];                                   // agent-scope loads: what the parts wrote through, not a cached line
#pragma unroll
                for (int j = 0; j < 32; ++j)
                    t2[j] = __hip_atomic_load(reinterpret_cast<const uint64_t*>(pz + ((j * 256 + tid) << 1)), __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        typedef float f32x2 __attribute__((ext_vector_type(2)));
                        f32x2 v2;
                        __builtin_memcpy(&v2, &t2[i * 8 + q], 8);
                        o[i][2 * q] += v2[0] * g;
                        o[i][2 * q + 1] += v2[1] * g;
                    }
            }
        }
    }
    // ---- normalise and store: lane owns query qi, d = 32*db + 8*(v/4) + 4*h2 + v%4 ----
    if (finish && wctx.ok && qi < seq) {
        const float inv = 1.0f / l_run;
        T* out = Tout + (size_t)(seq_row0 + qi) * ldt + head * ATT_D;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                T4 pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) pk[j] = (T)(o[db][g * 4 + j] * inv);
                if constexpr (SYNC) {   // written through to memory, like the GeMM tile's output
                    uint64_t bits;
                    __builtin_memcpy(&bits, &pk, 8);
                    __hip_atomic_store(reinterpret_cast<uint64_t*>(out + db * 32 + g * 8 + h2 * 4), bits, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    *(T4*)(out + db * 32 + g * 8 + h2 * 4) = pk;
                }
            }
    }

    dr.grab();   // the increment for the next tile travels while the stores drain
    if (SYNC && finish) post_tile<true>(args, s, qblk * heads + head, head, qblk);
    if (tracing && tid == 0) {
        TraceRec r;
        r.rel = rel_ticket; r.where = hw_where(2u); r.tx = head; r.ty = tyz;
        r.t_enter = t_enter; r.t_start = t_start; r.t_ready = t_ready; r.t_end = now_ticks();
        args.trace[rel_ticket] = r;
    }
}

}  // namespace depsync
