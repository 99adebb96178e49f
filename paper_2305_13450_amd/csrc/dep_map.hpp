// Index arithmetic of the dependencies between the tiles of two consecutive stages: which
// semaphore a producer tile posts to under each policy (Fig. 4b of the paper), at which K steps
// of a consumer tile a new group of producer tiles has to be waited for, and which producer
// tiles those are.  Plain integer functions, compiled for the device (the tiles call them) and
// for the host (the planner checks with them that every slice a consumer tile loads is covered
// by a wait issued no later than that slice's K step).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "chain_args.h"

namespace depsync {

__host__ __device__ __forceinline__ uint32_t dm_min(uint32_t a, uint32_t b) { return a < b ? a : b; }
__host__ __device__ __forceinline__ int dm_imin(int a, int b) { return a < b ? a : b; }
__host__ __device__ __forceinline__ int dm_imax(int a, int b) { return a > b ? a : b; }

// Semaphore a producer tile (x,y) posts to / a consumer looks at, per policy (Fig. 4b):
//   row:     sem = y                      value = grid_x
//   tile:    sem = x*grid_y + y           value = 1
//   strided: sem = y*stride + x % stride  value = grid_x / stride
__host__ __device__ __forceinline__ uint32_t policy_sem(uint32_t kind, uint32_t x, uint32_t y, uint32_t grid_y, uint32_t stride) {
    switch (kind) {
        case DEP_TILE:
        case DEP_CONV_TILE:
            return x * grid_y + y;
        case DEP_STRIDED:
        case DEP_ATTN_QKV:
            return y * stride + (x % stride);
        default:
            return y;
    }
}

// Range of producer row tiles and the producer column tile a K step depends on.
struct DepRange {
    bool any;          // there is something to wait for
    uint32_t y0, y1;   // inclusive producer row-tile range
    uint32_t x;        // producer column tile (TILE / STRIDED kinds)
};

// Dependency segments of a consumer tile start at multiples of this many K steps of 64 elements
// (0: only at the first step of the tile's K range).
__host__ __device__ __forceinline__ uint32_t dep_seg_steps(const StageDesc& s) {
    switch (s.dep_kind) {
        case DEP_TILE: case DEP_STRIDED: return s.prod_tn / 64;
        case DEP_CONV_TAPROW: return 3 * s.Cin / 64;
        case DEP_CONV_TILE: {   // starts of filter rows and of producer channel tiles inside them
            uint32_t a = 3 * s.Cin / 64, b = s.prod_tn / 64;
            while (b != 0) { const uint32_t r = a % b; a = b; b = r; }
            return a;
        }
        default: return 0;
    }
}

// K steps of part kz of a stage split along K: parts start on multiples of part_seg steps, the first part_extra of them
// are one such piece longer than the others, the last one also takes what is left of the K steps.
struct KRange { uint32_t kb, ke; };
__host__ __device__ __forceinline__ KRange k_part(const StageDesc& s, uint32_t kz, uint32_t k_steps) {
    KRange r;
    r.kb = kz * s.part_steps + dm_min(kz, s.part_extra) * s.part_seg;
    r.ke = kz + 1 == s.ksplit ? k_steps : (kz + 1) * s.part_steps + dm_min(kz + 1, s.part_extra) * s.part_seg;
    return r;
}

// Does the A slice of K step kt start a new dependency segment, and on what?
// kb: first K step of this workgroup's K range (0 unless the stage is split along K).
// (Returned by value: filled in through a reference the range lived in scratch memory on the device, and each look at it on a
// consumer tile's way to its first request waited for the weights in flight: one token of 12288 x 6144 x 12288 73.6 -> 68.8
// us, 17 attention chains 1.1 % and 36 GeMM chains 1.2 % faster.)
__host__ __device__ __forceinline__ DepRange dep_segment(const StageDesc& s, uint32_t m0, uint32_t tm, uint32_t kt, uint32_t kb) {
    const DepRange none = {false, 0, 0, 0};
    const uint32_t m_last = dm_min(m0 + tm, s.M) - 1;
    switch (s.dep_kind) {
        case DEP_ROW:
            if (kt != kb) return none;
            return {true, m0 / s.prod_tm, m_last / s.prod_tm, 0};
        case DEP_TILE:
        case DEP_STRIDED: {
            const uint32_t k0 = kt * 64;
            if (k0 % s.prod_tn != 0) return none;
            const uint32_t x = k0 / s.prod_tn;
            // same semaphore as x - stride, which this workgroup has already waited for if that
            // segment lies inside its K range
            if (s.dep_kind == DEP_STRIDED && x >= s.stride && (x - s.stride) * (s.prod_tn / 64) >= kb) return none;
            return {true, m0 / s.prod_tm, m_last / s.prod_tm, x};
        }
        case DEP_CONV_ROW: {
            if (kt != kb) return none;
            const int lo = (int)m0 - (int)s.W - 1, hi = (int)m_last + (int)s.W + 1;
            return {true, (uint32_t)dm_imax(lo, 0) / s.prod_tm, (uint32_t)dm_imin(hi, (int)s.M - 1) / s.prod_tm, 0};
        }
        case DEP_CONV_TAPROW:
        case DEP_CONV_TILE: {
            // K runs filter-row major: k = ((fr*3 + fs) * Cin + c).  A new segment starts with
            // every filter row (TAPROW) or every producer channel tile of a filter row's first tap (TILE).
            const uint32_t k0 = kt * 64;
            const uint32_t tap = k0 / s.Cin, c0 = k0 % s.Cin;
            const uint32_t fr = tap / 3, fs = tap % 3;
            uint32_t x = 0;
            if (fs != 0) return none;
            if (s.dep_kind == DEP_CONV_TAPROW) { if (c0 != 0) return none; }
            else { if (c0 % s.prod_tn != 0) return none; x = c0 / s.prod_tn; }
            const int sh = ((int)fr - 1) * (int)s.W;
            const int lo = (int)m0 + sh - 1, hi = (int)m_last + sh + 1;
            if (hi < 0 || lo > (int)s.M - 1) return none;      // whole filter row is padding
            return {true, (uint32_t)dm_imax(lo, 0) / s.prod_tm, (uint32_t)dm_imin(hi, (int)s.M - 1) / s.prod_tm, x};
        }
        default:
            return none;
    }
}

// ---- the prompt-phase attention tile: which rows it covers, waits for and reads -------------------

constexpr int ATT_BQ = 128;      // query rows per tile (32 per wave)
constexpr int ATT_BK = 64;       // keys per block
constexpr int ATT_D = 128;       // head dimension
// Key blocks per part when a tile's keys are split over workgroups (at least this many: a part
// re-reads the queries and leaves 65 KB of partial results).
constexpr uint32_t ATT_MIN_PART_BLOCKS = 4;

// Dispatch row tyz of the stage: part `part` of the keys of query block q0 .. q_last (positions inside
// the sequence, whose rows of the QKV tensor start at seq_row0).  Its key blocks are kb_begin .. kb_end - 1, in
// key order: the cached keys first, then the new tokens.
struct AttnSpan {
    uint32_t qblk, part, nparts;
    uint32_t seq_row0, q0, q_last;
    uint32_t kb_begin, kb_end;
};
__host__ __device__ __forceinline__ AttnSpan attn_span(uint32_t tyz, uint32_t ksplit, uint32_t seq, uint32_t cached) {
    AttnSpan t;
    t.qblk = tyz / ksplit; t.part = tyz % ksplit;
    const uint32_t qblocks = (seq + ATT_BQ - 1) / ATT_BQ;
    t.seq_row0 = t.qblk / qblocks * seq;
    t.q0 = t.qblk % qblocks * ATT_BQ;
    t.q_last = dm_min(t.q0 + ATT_BQ, seq) - 1;
    const uint32_t nblk = (cached + t.q_last) / ATT_BK + 1;                // key blocks the query block sees
    uint32_t chunk = (nblk + ksplit - 1) / ksplit;                         // key blocks per part
    if (chunk < ATT_MIN_PART_BLOCKS) chunk = ATT_MIN_PART_BLOCKS;
    t.nparts = (nblk + chunk - 1) / chunk;                                 // parts that have any (<= ksplit)
    t.kb_begin = t.part * chunk;
    t.kb_end = dm_min(nblk, t.kb_begin + chunk);
    return t;
}

// Producer tiles (x, y) of the QKV GeMM a tile waits for: row tiles y of the sequence's rows up to its last query,
// and in each the column tiles with this head's Q, K and V columns (x = 0 where a whole row shares a semaphore).
template <class F>
__host__ __device__ __forceinline__ void attn_for_each_wait(const StageDesc& s, uint32_t head, uint32_t row_first, uint32_t row_last, F&& f) {
    const uint32_t E = s.heads * ATT_D;
    for (uint32_t y = row_first / s.prod_tm; y <= row_last / s.prod_tm; ++y) {
        if (s.dep_kind == DEP_ROW) { f(0u, y); continue; }
        const uint32_t nblk = (s.dep_kind == DEP_STRIDED) ? 1u : 3u;       // strided: Q, K, V share a semaphore
        for (uint32_t b = 0; b < nblk; ++b) {
            const uint32_t c0 = b * E + head * ATT_D;
            for (uint32_t x = c0 / s.prod_tn; x <= (c0 + ATT_D - 1) / s.prod_tn; ++x) f(x, y);
        }
    }
}

// A key block is read whole, also where it runs past the tile's last query (a cache whose length is no
// multiple of 64 shifts the blocks against the rows).  What lies past that query is masked, and its rows belong to
// producer tiles nobody has waited for: the weight 0 does not make up for whatever they hold (0 x NaN), and a line
// read before its producer has posted would stay in this XCD's L2 for the tiles that read it later.  So those
// positions read the last query's row again.
// All 64 positions from k0 on are rows of one source, in a run:
__host__ __device__ __forceinline__ bool attn_block_in_one_run(uint32_t k0, uint32_t cached, uint32_t q_last) {
    return k0 + ATT_BK <= cached || (k0 >= cached && k0 + ATT_BK <= cached + q_last + 1);
}
// Row, inside the sequence, of the new token read for position key >= cached:
__host__ __device__ __forceinline__ uint32_t attn_key_row(uint32_t key, uint32_t cached, uint32_t q_last) {
    return dm_min(key - cached, q_last);
}

}  // namespace depsync
