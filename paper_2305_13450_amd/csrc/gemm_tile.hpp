// One output macro-tile of a GeMM or implicit-GeMM 3x3 convolution on CDNA4 (gfx950):
//   C[m0:m0+TM, n0:n0+TN] = act( A[m0:m0+TM, :] * B[n0:n0+TN, :]^T ),   A, B contiguous along K.
// 256 threads = 4 wave64s in a WM x WN grid; each wave owns a (TM/WM) x (TN/WN) sub-tile built
// from 32x32 accumulator blocks of v_mfma_f32_32x32x16 (bf16 or f16 in, fp32 accumulate).
// Operand tiles of 64 K-elements (128-byte rows) are DMA'd from global memory straight into
// LDS (buffer_load_dwordx4 lds), two to eight stages deep (a ring per operand), with the 16-byte
// chunks of every row XOR swizzled so that the 128-bit fragment reads are free of bank conflicts.
//
// The tile is the unit the synchronisation subsystem works on (Fig. 4a of the paper): a
// consumer tile waits before loading the slice of A that an earlier stage produces, and a
// producer tile posts after its stores.  The independent operand B (weights) is requested
// before the wait (the load/wait reordering of Section IV-C).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "chain_args.h"
#include "dep_map.hpp"
#include "sync_device.hpp"

namespace depsync {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// WK: waves that share a sub-tile, each with 1 / WK of a step's K slices; the first adds up what they have at the end.
template <int TM_, int TN_, int WM_, int WN_, int MINB_, int NSTAGE_, int NSTB_ = 0, int WK_ = 1>
struct TileCfg {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, MINB = MINB_;
    static constexpr int BK = 64;                     // K elements per pipeline step
    static constexpr int ROWB = BK * 2;               // bytes per LDS row: one 128-byte line of the operand
    static constexpr int WK = WK_;
    static constexpr int KK = BK / 16 / WK;           // 16-wide K slices (one MFMA deep) per step and wave
    static constexpr int RPD = 1024 / ROWB;           // operand rows one 1 KB DMA instruction fills
    static constexpr int LPR = ROWB / 16;             // lanes (16-byte chunks) per row
    static constexpr int NSTAGE = NSTAGE_;               // LDS stages of the A operand: NSTAGE-1 K steps in flight
    static constexpr int NSTB = NSTB_ ? NSTB_ : NSTAGE_; // LDS stages of the B operand (no more than A's)
    static constexpr int WTM = TM / WM, WTN = TN / WN;  // wave sub-tile
    static constexpr int FM = WTM / 32, FN = WTN / 32;  // 32x32 blocks per wave
    static constexpr int NIA = TM / (4 * RPD), NIB = TN / (4 * RPD);  // 1 KB DMA instructions per wave per step
    static constexpr int A_BYTES = TM * ROWB, B_BYTES = TN * ROWB;
    static constexpr int B_BASE = NSTAGE * A_BYTES;      // the B stages follow the A stages
    static constexpr int LDS_BYTES = NSTAGE * A_BYTES + NSTB * B_BYTES;
    static_assert(WM * WN * WK == 4, "four waves per workgroup");
    static_assert(NSTB >= 2 && NSTAGE >= NSTB && MINB * LDS_BYTES <= 160 * 1024, "stages must fit the 160 KB LDS");
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile is made of 32x32 blocks");
    static_assert(TM % (4 * RPD) == 0 && TN % (4 * RPD) == 0, "each wave issues whole DMA groups");
};

template <typename T> struct Mma;
template <> struct Mma<__bf16> {
    using V8 = bf16x8;
    static __device__ __forceinline__ f32x16 mma(V8 a, V8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mma<_Float16> {
    using V8 = f16x8;
    static __device__ __forceinline__ f32x16 mma(V8 a, V8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};

// Position swizzle of the 16-byte chunks of LDS row r (128-byte rows).  Any 8 consecutive rows
// get 8 distinct positions (32 banks), and any 16 consecutive rows get 16 distinct (position, row
// parity) pairs (64 banks).  The pattern repeats every 16 rows, so fragment blocks 32 rows apart
// share one per-lane offset.
__device__ __forceinline__ uint32_t swz(uint32_t r) { return (r & 7u) ^ ((r >> 3) & 1u); }

typedef __attribute__((address_space(3))) void* lptr_t;

// Operand reads, `off` (per lane) and `uniform_off` bytes from a wave-uniform base, 16 bytes per lane straight to LDS at
// l + 16 * lane.  A buffer instruction rather than global_load_lds: no address arithmetic per lane, and the compiler
// counts it exactly.  global_load_lds is a FLAT instruction that touches LDS; with one in flight every wait for an
// LDS read became a wait for all of them (2048 tokens of the 12288 x 6144 x 12288 chain 507 -> 499 us, one token of
// 1024 x 1024 x 1024 14.1 -> 13.1).  (An operand is smaller than 4 GiB; `bytes` is where it ends: reads at
// and past that offset, 0xfffffff0 at the latest, give zeros.)
struct OperandBuf {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ explicit OperandBuf(const char* uniform_base, uint32_t bytes = 0xffffffffu)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc((void*)uniform_base, (short)0, (int)bytes, 0x00027000)) {}
    __device__ __forceinline__ void dma16(uint32_t off, uint32_t uniform_off, char* l) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)l, 16, off, uniform_off, 0, 0);
    }
    __device__ __forceinline__ u32x4 load16(uint32_t off, uint32_t uniform_off) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, uniform_off, 0);
    }
};
// Store one 16-bit output element.  With the synchronisation hooks compiled in, the store is an
// agent-scope store: it is written through this XCD's L2 to memory, so that the post needs no
// write-back of the whole L2 before the semaphore moves.
template <bool THROUGH, typename T>
__device__ __forceinline__ void store_out(T* p, T v) {
    if constexpr (THROUGH) {
        uint16_t bits;
        __builtin_memcpy(&bits, &v, 2);
        __hip_atomic_store(reinterpret_cast<uint16_t*>(p), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        *p = v;
    }
}
// GeLU x * Phi(x) with Phi written through erfc: Phi(x) = erfc(-x / sqrt 2) / 2, and for z >= 0
// erfc(z) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-z^2), t = 1 / (1 + p z), to 1.5e-7
// absolute (Abramowitz and Stegun 7.1.26).  Working from erfc on the negative side keeps the
// small values of the left tail free of the cancellation in 1 + erf; the whole thing is two
// transcendental and a dozen plain instructions, less than half of a library erff, which
// matters where the epilogue is not hidden (the workgroup that finishes a tile split along K).
__device__ __forceinline__ float gelu_erf(float x) {
    const float z = fabsf(x) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, z, 1.0f));
    float h = __builtin_fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);   // coefficients of erfc / 2
    h = __builtin_fmaf(t, h, 0.5f * 1.421413741f);
    h = __builtin_fmaf(t, h, 0.5f * -0.284496736f);
    h = __builtin_fmaf(t, h, 0.5f * 0.254829592f);
    h = h * t * __builtin_amdgcn_exp2f(z * z * -1.4426950408889634f);          // erfc(z) / 2 = Phi(-|x|)
    return x * (x >= 0.0f ? 1.0f - h : h);
}
__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }

// ---- dependency bookkeeping of a consumer tile -------------------------------------------

// Wait for the semaphores of one dependency segment.  Acquire ordering without a cache
// invalidate: the semaphore reads are agent-scope atomic loads whose values this wave branches
// on before it issues the dependent operand's loads.  Those loads cannot hit a stale line in
// this XCD's L2: caches are invalidated when a kernel starts, nothing reads a line of the
// intermediate before the tile that produces it has posted, and the host requires the
// intermediate's rows to be 128-byte aligned, so a cache line never mixes the outputs of two
// producer tiles.
__device__ __forceinline__ void dep_wait(WaitCtx& w, const StageDesc& s, const DepRange& r) {
    const uint32_t target = s.sem_target_base + s.sem_value;
    for (uint32_t y = r.y0; y <= r.y1; ++y) {
        const uint32_t* sem = s.sems + policy_sem(s.dep_kind, r.x, y, s.prod_grid_y, s.stride) * SYNC_WORD_STRIDE;
        const uint32_t v = sem_load(sem);
        if (!sem_reached(v, target)) sem_wait(w, sem, target, v);
    }
}

// ---- the tile ------------------------------------------------------------------------------

// DEP != 0: this tile's A operand is produced by the previous stage of the chain (the tile waits
// on semaphores before it requests a slice of A).  DEP == 1: everything it depends on is waited
// for before its first slice (RowSync, and the convolution's whole-halo wait), so the K loop is
// the one of a tile without dependencies; DEP == 2: new dependency segments start inside the K
// loop (TileSync, StridedSync, the convolution's per-filter-row waits).
// THROUGH: the tile's output is waited for by a later stage and is stored write-through.
template <class Cfg, typename T, bool SYNC, uint32_t AMODE, int DEP, bool THROUGH, class DR>
__device__ __forceinline__ void gemm_tile(const ChainArgs& args, const StageDesc& s, uint32_t tx, uint32_t tyz,
                                          uint32_t rel_ticket, char* lds, uint64_t t_enter, DR& dr) {
    using M = Mma<T>;
    using V8 = typename M::V8;
    constexpr int TM = Cfg::TM, TN = Cfg::TN, FM = Cfg::FM, FN = Cfg::FN;
    constexpr int NIA = Cfg::NIA, NIB = Cfg::NIB;
    static_assert(!DEP || SYNC, "dependencies exist only with the synchronisation hooks compiled in");
    // A tile whose output a later stage waits for stores it write-through, so that the post needs
    // no write-back of the L2: a chain's first stage, and the middle stages of a chain of three or
    // four convolutions.  The last stage stores normally.  (A posting tile instantiated without
    // THROUGH still works: post_tile then writes the L2 back for it.)
    static_assert(!THROUGH || SYNC, "write-through stores belong to the synchronised kernels");

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = uni(tid >> 6);
    constexpr uint32_t NW = Cfg::WM * Cfg::WN;             // sub-tiles; wave w and, where waves share them, w + NW work on the same
    const uint32_t kw = wave / NW, wm = wave % NW / Cfg::WN, wn = wave % Cfg::WN;
    const bool holds = Cfg::WK == 1 || kw == 0;            // this wave holds a sub-tile after the K loop
    const uint32_t sM = uni(s.M), sN = uni(s.N);
    const bool gate_up = AMODE != A_CONV3X3 && s.bmode == B_GATE_UP;
    const uint32_t tn_out = gate_up ? TN / 2 : TN;       // output columns this tile owns
    const uint32_t S = uni(s.ksplit);                      // workgroups per output tile (split along K)
    // (No division by a runtime value where it can be helped: each is some forty dependent instructions, and the tiles
    // of short chains have nothing to hide them behind.)
    uint32_t ty = tyz, kz = 0;
    if (S > 1) { ty = uni(tyz / S); kz = tyz - ty * S; }
    const uint32_t m0 = ty * TM, n0 = tx * tn_out;
    constexpr uint32_t BK = Cfg::BK, ROWB = Cfg::ROWB;
    const uint32_t KT = uni(s.K / BK);
    uint32_t kb = 0, ke = KT;                              // this workgroup's K steps
    if (S > 1) { const KRange r = k_part(s, kz, KT); kb = uni(r.kb); ke = uni(r.ke); }
    const OperandBuf bufA(uni_ptr(s.A), AMODE == A_CONV3X3 ? uni(s.M * s.lda * 2u) : 0xffffffffu), bufB(uni_ptr(s.B));
    const uint32_t bkstep = uni(s.b_kstep_bytes);
    // conv geometry (unused otherwise)
    const uint32_t cH = uni(s.H), cW = uni(s.W), cCin = uni(s.Cin);

    WaitCtx wctx{&args, rel_ticket, true};
    const bool tracing = SYNC && (args.flags & DS_FLAG_TRACE) && args.trace != nullptr && rel_ticket < args.trace_cap;
    uint64_t t_start = 0, t_ready = 0;
    if (tracing) t_start = now_ticks();

    // ---- per-lane DMA source offsets (bytes from the operand base, K step 0) ----
    const uint32_t lrow = lane / Cfg::LPR, lpos = lane % Cfg::LPR;
    uint32_t offA[NIA], offB[NIB];
    uint32_t pixyx[AMODE == A_CONV3X3 ? NIA : 1];   // conv: (y << 16) | x of the output pixel of each DMA row
    // conv: pixel of the first row by division, the others RPD pixels on (rows past the end of the matrix are never
    // stored: any coordinates inside the image do)
    uint32_t px = 0, py = 0;
    if constexpr (AMODE == A_CONV3X3) {
        const uint32_t rem = min(m0 + wave * NIA * Cfg::RPD + lrow, sM - 1) % (cH * cW);
        py = rem / cW; px = rem - py * cW;
    }
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
        const uint32_t r = (wave * NIA + i) * Cfg::RPD + lrow;
        const uint32_t c = lpos ^ swz(r);
        const uint32_t m = min(m0 + r, sM - 1);
        offA[i] = m * s.lda * 2u + c * 16u;
        if constexpr (AMODE == A_CONV3X3) {
            pixyx[i] = (py << 16) | px;
            px += Cfg::RPD;
            while (px >= cW) { px -= cW; py = py + 1 == cH ? 0 : py + 1; }
        }
    }
#pragma unroll
    for (int i = 0; i < NIB; ++i) {
        const uint32_t q = (wave * NIB + i) * Cfg::RPD + lrow;
        const uint32_t c = lpos ^ swz(q);
        uint32_t row;
        if (gate_up) {
            const uint32_t blk = q >> 5, within = q & 31u;
            const uint32_t col = min(n0 + (blk >> 1) * 32 + within, sN - 1);
            row = (blk & 1u) * sN + col;
        } else {
            row = min(n0 + q, sN - 1);
        }
        offB[i] = row * s.b_row_bytes + c * 16u;
    }

    // Source of the K step that is being requested ("next" step): a byte offset for B and the
    // dense A, and for the conv the filter tap (fr, fs in -1..1) and the byte shift of that tap.
    struct NextStep {
        uint32_t kbytes;     // byte offset of the K step in a row of A
        uint32_t kbytes_b;   // byte offset of the K step in B
        uint32_t c0;         // conv: first input channel of the step
        int fr, fs;          // and its filter tap (-1..1 each)
        uint32_t shift;      // (of 32 bits, like the offsets it is added to)
    } nx;
    // (A and B may be requested a different number of steps ahead, so each has its own "next")
    auto set_next_A = [&](uint32_t kt) __attribute__((always_inline)) {
        nx.kbytes = kt * ROWB;
        if constexpr (AMODE == A_CONV3X3) {
            uint32_t tap = 0;
            nx.c0 = 0;
            if (kt != 0) { tap = kt * BK / cCin; nx.c0 = kt * BK - tap * cCin; }
            nx.fr = (int)(tap / 3) - 1; nx.fs = (int)(tap % 3) - 1;
            nx.shift = (uint32_t)((nx.fr * (int)cW + nx.fs) * (int)cCin + (int)nx.c0) * 2u;
        }
    };
    // conv: the K step after the one set last.  (A step on is BK channels on in memory, over the end of a tap too; from
    // the last tap of a filter row to the next row it is a row of pixels less three.)
    const uint32_t row_jump = AMODE == A_CONV3X3 ? uni((cW - 3) * cCin * 2u) : 0u;
    auto step_next_A = [&]() __attribute__((always_inline)) {
        nx.shift += ROWB;
        nx.c0 += BK;
        const bool tap_end = nx.c0 == cCin;
        nx.c0 = tap_end ? 0u : nx.c0;
        nx.fs += tap_end ? 1 : 0;
        const bool row_end = nx.fs == 2;
        nx.fs = row_end ? -1 : nx.fs;
        nx.fr += row_end ? 1 : 0;
        nx.shift += row_end ? row_jump : 0u;
    };
    auto set_next_B = [&](uint32_t kt) __attribute__((always_inline)) {
        nx.kbytes_b = kt * bkstep;
    };
    // One 1 KB DMA instruction of the B (weights) or A operand of the next K step into `stage`.
    auto dma_B = [&](uint32_t stage, int i) __attribute__((always_inline)) {
        char* l = lds + Cfg::B_BASE + stage * Cfg::B_BYTES + wave * (NIB * 1024);
        bufB.dma16(offB[i], nx.kbytes_b, l + i * 1024);
    };
    auto dma_A = [&](uint32_t stage, int i) __attribute__((always_inline)) {
        char* l = lds + stage * Cfg::A_BYTES + wave * (NIA * 1024);
        if constexpr (AMODE == A_CONV3X3) {
            // a tap outside the image reads past the end of the tensor, which the buffer's range check turns into zeros
            // (every lane takes part in every request: the waits count instructions)
            const uint32_t y = (pixyx[i] >> 16) + (uint32_t)nx.fr, x = (pixyx[i] & 0xffffu) + (uint32_t)nx.fs;   // (-1: a large number)
            const bool valid = y < cH && x < cW;
            bufA.dma16(valid ? offA[i] + nx.shift : 0xfffffff0u, 0, l + i * 1024);
        } else {
            bufA.dma16(offA[i], nx.kbytes, l + i * 1024);
        }
    };
    auto issue_B = [&](uint32_t stage) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NIB; ++i) dma_B(stage, i);
    };
    auto issue_A = [&](uint32_t stage) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NIA; ++i) dma_A(stage, i);
    };

    // ---- per-lane fragment read offsets (bytes inside the A / B part of a stage) ----
    constexpr int KK = Cfg::KK;
    uint32_t aoff[KK], boff[KK];
    {
        const uint32_t ra = wm * Cfg::WTM + (lane & 31u), rb = wn * Cfg::WTN + (lane & 31u);
        const uint32_t h = lane >> 5;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const uint32_t c = (kw * KK + (uint32_t)kk) * 2u + h;
            aoff[kk] = ra * ROWB + ((c ^ swz(ra)) << 4);
            boff[kk] = rb * ROWB + ((c ^ swz(rb)) << 4);
        }
    }

    // How the parts of a tile split along K are put together.  SLICED: every part finishes a slice of the tile's rows.
    // Else the last part to arrive finishes the whole tile: a part of a 64 x 64 tile is 16 KB, which one workgroup
    // reads back in the round trip that a slice would take too (64 x 4096 x 1536 x 4096 20.2 us, by slices 22.8), two
    // workgroups on a CU cover each other's exchange, and the largest tiles, hardly ever split, have no registers to
    // spare for the code (256 x 192: 93 spilled around the tile loop, the 2048-token chain 500 -> 510 us).
    constexpr bool SLICED = Cfg::MINB == 1 && FM * FN > 1 && FM * FN <= 9;
    // this part of a tile split along K has been started (see the exchange below)
    if (SLICED && S > 1 && tid == 0)
        __hip_atomic_fetch_add(s.arrive + (ty * s.grid_x + tx) * SYNC_WORD_STRIDE, SPLIT_STARTED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const bool reorder = !(args.flags & DS_FLAG_NO_REORDER);

    // Dependency segments start at multiples of seg_steps K steps (0: only at step 0).
    uint32_t seg_steps = 0, seg_next = kb;   // the host makes K ranges start on segment boundaries
    if constexpr (DEP == 2) seg_steps = uni(dep_seg_steps(s));
    // Called before the A slice of K step k (< KT) is requested into `stage`: if a dependency
    // segment starts there, make sure its producer tiles have posted.  The semaphores are looked
    // at 64 segments at a time (lane l tests the segment l places ahead, one load instruction
    // for the wave), so a tile whose producers are long done pays one round trip for its whole
    // K loop instead of one per segment.  When the segment at hand has not been posted, the
    // weights of the step are requested first (the load/wait reordering) and then the wave
    // really waits; the caller requests the slice (and, harmlessly, the weights again) afterwards.
    uint32_t ready_until = 0;      // every segment that starts before this K step is known to be posted
    auto dep_before_request = [&](uint32_t k, uint32_t stage, bool b_due) __attribute__((always_inline)) {
        if constexpr (DEP) {
            // (rare: the K loop's common path must stay one straight run of code; with the check's
            // branches laid out between the hand-over and the slices, the three taken jumps per step
            // cost the dependent tiles 7 % on a 256x192 tile)
            if (__builtin_expect(k == seg_next, 0)) {
                seg_next = seg_steps ? seg_next + seg_steps : 0xffffffffu;
                const DepRange dr = dep_segment(s, m0, TM, k, kb);
                if (!dr.any) return;
                bool polled = false;
                if (k >= ready_until) {
                    const uint32_t ka = k + lane * seg_steps;          // lane's segment start
                    bool ok = true;
                    if (ka < ke && (lane == 0 || seg_steps != 0)) {
                        const DepRange la = dep_segment(s, m0, TM, ka, kb);
                        const uint32_t target = s.sem_target_base + s.sem_value;
                        for (uint32_t y = la.y0; la.any && y <= la.y1; ++y) {
                            const uint32_t* sem = s.sems + policy_sem(s.dep_kind, la.x, y, s.prod_grid_y, s.stride) * SYNC_WORD_STRIDE;
                            ok = ok && sem_reached(__hip_atomic_load(sem, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), target);
                        }
                    }
                    const uint64_t mask = __ballot(ok);
                    // the requests for the dependent slice stay behind the look at its semaphores:
                    // a compiler fence (the loads are relaxed atomics, which the compiler may
                    // otherwise reorder with ordinary memory operations); the hardware returns
                    // loads in issue order, and the wave acts on the values only after they arrived
                    __atomic_signal_fence(__ATOMIC_ACQUIRE);
                    const uint32_t n_ready = (~mask == 0) ? 64u : (uint32_t)__builtin_ctzll(~mask);
                    if (n_ready == 0) {
                        if (reorder && b_due) issue_B(stage);
                        dep_wait(wctx, s, dr);
                        polled = true;
                        ready_until = k + 1;
                    } else {
                        ready_until = seg_steps ? k + n_ready * seg_steps : 0xffffffffu;
                        // the segments seen posted need no further look: the next check is due where
                        // they end (unless every wait is being counted)
                        if (!(args.flags & DS_FLAG_COUNT)) seg_next = ready_until;
                    }
                }
                if (args.flags & DS_FLAG_COUNT) {
                    for (uint32_t y = dr.y0; y <= dr.y1; ++y) count_wait(args, polled);
                }
            }
        }
    };

    // ---- prologue ----
    // A is requested NSA-1 steps ahead into a ring of NSA stages, B NSB-1 steps ahead into a ring
    // of NSB <= NSA stages (a tile too large for three stages of both keeps three of A and two of B:
    // then only B's requests of a step, issued first, have to land within the step, and A's
    // are spread over the rest of it with a step more to land).
    constexpr int NSA = Cfg::NSTAGE, NSB = Cfg::NSTB;
    constexpr int NG = KK * FM;           // MFMA groups per step
    constexpr int ND = NIA + NIB;         // DMA instructions per step
    // groups the DMA instructions are spread over: with two stages the step's requests must
    // have landed by the end of the same step, so they go out at its start (measured on the
    // GPT-3 chain at M = 2048: 128x192 601 -> 581 us, 128x128 727 -> 669 us with all of them in
    // the first group; the 256-row tiles, with twice the requests per wave, do best with a
    // quarter of the groups: 256x192 714 -> 684 us)
    constexpr int NGD = (NSA > 2) ? NG : (FM <= 2 ? 1 : NG / 4);
    // Tiles that have a CU to themselves (one wave per SIMD) read all fragments of the next
    // 16-wide K slice together, a whole slice of MFMAs before their first use, with the order
    // pinned: left to itself the compiler issues each read right before the wait for it (while
    // LDS DMA is in flight it only ever waits for lgkmcnt(0)), and with no second workgroup on
    // the CU nothing fills that round trip.  Measured on the GPT-3 chain at M = 2048: 256x128
    // 609 -> 585 us, 256x192 621 -> 612 us; with two workgroups per CU it gains nothing.
    constexpr bool S2 = (Cfg::MINB == 1);
    // At the top of step k the requests of A(k) and B(k) must have landed.  Requests complete in
    // issue order, and a step issues B's before A's, so what may still be outstanding is what was
    // issued after B(k): the A requests of that same step when A runs further ahead than B, and
    // the NSB-2 whole steps after it.
    constexpr int OUTSTANDING = (NSA > NSB ? NIA : 0) + (NSB - 2) * ND;
    static_assert(OUTSTANDING <= 48, "outstanding DMA instructions must fit the vmcnt counter");
    // the steps before the loop, in the order the loop itself would have issued them
#pragma unroll
    for (int p = 0; p < NSA - 1; ++p) {
        const int pb = p - (NSA - NSB);    // B's step issued alongside A's step p
        if (AMODE != A_CONV3X3 || p == 0) set_next_A(min(kb + (uint32_t)p, ke - 1));
        else if (kb + (uint32_t)p < ke) step_next_A();
        if (pb >= 0) set_next_B(min(kb + (uint32_t)pb, ke - 1));
        // the weights of the step go out before the look at the semaphores (the load/wait reordering
        // of Section IV-C), so the poll's round trip is not added to their latency
        if (reorder && pb >= 0) issue_B(pb);
        if (kb + (uint32_t)p < ke) dep_before_request(kb + p, pb >= 0 ? pb : 0, false);
        if (p == 0 && tracing) t_ready = now_ticks();
        if (!reorder && pb >= 0) issue_B(pb);
        issue_A(p);
    }

    // The K loop, as one stream of 16-wide K slices (KK per step, each KK*... FM groups of FN MFMAs
    // per wave).  While a slice's MFMAs run, the fragments of the next slice are read from LDS
    // into the other fragment buffer.  The workgroup barrier that hands over a step's stage sits
    // before the LAST slice of the step before it: at that point every wave has read (not yet
    // multiplied) its last fragments of the current stage, so the stage is free for new requests,
    // and the next step's first fragments travel from LDS while the last slice's MFMAs run; no
    // fragment read is exposed at a step boundary.  The DMA instructions a barrier releases (the
    // steps NSB-1 / NSA-1 ahead, weights first) are spread over the first NGD of the NG groups
    // that follow it.  Past the end of K the last step is simply requested again into an idle
    // stage, so the body is free of branches.
    V8 af[2][FM], bf[2][FN];
    auto load_frags = [&](int buf, const char* la, const char* lb, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i) af[buf][i] = *(const V8*)(la + aoff[kk] + i * (32 * ROWB));
#pragma unroll
        for (int j = 0; j < FN; ++j) bf[buf][j] = *(const V8*)(lb + boff[kk] + j * (32 * ROWB));
    };
    uint32_t reqA = NSA - 1, reqB = NSB - 1;                 // stages the next requests go into
    // DMA instructions of group g (counted from the barrier that released them)
    auto dma_group = [&](int g) __attribute__((always_inline)) {
        if (g < NGD) {
#pragma unroll
            for (int d = (g * ND) / NGD; d < ((g + 1) * ND) / NGD; ++d) {
                if (d < NIB) dma_B(reqB, d);
                else dma_A(reqA, d - NIB);
            }
        }
    };
    // One slice: MFMAs on fragment buffer `buf`; meanwhile read the fragments of slice nkk of the
    // stage at (nla, nlb) into the other buffer (nkk < 0: none) and issue the DMA groups g0 .. g0+FM-1
    // (g0 < 0: none).
    auto slice = [&](int buf, const char* nla, const char* nlb, int nkk, int g0) __attribute__((always_inline)) {
        const int n = buf ^ 1;
        if constexpr (S2) {
            // One wave per SIMD: nothing else fills the matrix unit while this wave issues other
            // instructions, and a run of fragment reads takes longer to issue than one MFMA to
            // execute.  So the order is pinned: after each MFMA at most one fragment read of the
            // next slice (the fragments the next slice needs first go first), DMA instructions at
            // the start of a group.  The empty asm that reads the current slice's fragments is where
            // the compiler's wait for them lands, before anything of this slice is issued.
#pragma unroll
            for (int i = 0; i < FM; ++i) asm volatile("" ::"v"(__builtin_bit_cast(u32x4, af[buf][i])));
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" ::"v"(__builtin_bit_cast(u32x4, bf[buf][j])));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                if (g0 >= 0) dma_group(g0 + i);
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    acc[i][j] = M::mma(af[buf][i], bf[buf][j], acc[i][j]);
                    // fragment read number m of the next slice (A0, B0 .. B(FN-1), A1 ..) follows MFMA
                    // number m; a wave tile of fewer MFMAs than fragments reads the rest after the last
                    constexpr int NF = FM + FN, NM = FM * FN;
                    const int m0 = i * FN + j, m1 = (m0 == NM - 1 && NM < NF) ? NF : m0 + 1;
                    if (nkk >= 0) {
#pragma unroll
                        for (int m = m0; m < m1; ++m) {
                            if (m == 0) af[n][0] = *(const V8*)(nla + aoff[nkk]);
                            else if (m <= FN) bf[n][m - 1] = *(const V8*)(nlb + boff[nkk] + (m - 1) * (32 * ROWB));
                            else if (m < NF) af[n][m - FN] = *(const V8*)(nla + aoff[nkk] + (m - FN) * (32 * ROWB));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if (nkk >= 0) {
                af[n][i] = *(const V8*)(nla + aoff[nkk] + i * (32 * ROWB));
#pragma unroll
                for (int j = (i * FN) / FM; j < ((i + 1) * FN) / FM; ++j)
                    bf[n][j] = *(const V8*)(nlb + boff[nkk] + j * (32 * ROWB));
            }
            if (g0 >= 0) dma_group(g0 + i);
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = M::mma(af[buf][i], bf[buf][j], acc[i][j]);
            // A wave with a single block has one MFMA per slice, each waiting for the one before: left to itself the compiler
            // collects them behind the step's requests in some kernels, and a step of the dependent 64x64 convolution tile took
            // 16 ns more (four 14x14x512 convolutions 48.0 us, 46.8 with the order pinned; 256 x 1024 x 4096 x 1024 level).
            if constexpr (FM * FN == 1) __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Hand-over of step k's stage: its requests have landed for every wave (requests complete in
    // issue order; a bare s_barrier, since __syncthreads() would also wait for the younger ones),
    // and every wave has finished reading the stage of step k-1.  Then point the requests at the
    // steps ahead of k (after waiting for what the A slice depends on, if a dependency segment starts).
    auto hand_over = [&](uint32_t k) __attribute__((always_inline)) {
        // The sources of the requests this hand-over releases and the test for a dependency
        // segment are scalar arithmetic: done BEFORE the wait and the barrier, where the wave
        // would idle anyway, and passed through the asm statement as operands so that the
        // compiler cannot sink them into the gap between the barrier and the first MFMA behind
        // it (with a branch in that gap it did: the dependent tiles' steps were 7 % slower than
        // the same steps of a tile without dependencies).
        const uint32_t kreq = k + (NSA - 1);
        if constexpr (AMODE == A_CONV3X3) { if (kreq < ke) step_next_A(); }   // (past the end the last step again)
        else set_next_A(min(kreq, ke - 1));
        set_next_B(min(k + (NSB - 1), ke - 1));
        uint32_t seg = 0;
        if constexpr (DEP == 2) seg = uni((kreq < ke && kreq == seg_next) ? 1u : 0u);
        nx.kbytes_b = uni(nx.kbytes_b);
        if constexpr (AMODE == A_CONV3X3) {
            nx.shift = uni(nx.shift);
            uint32_t fr = uni((uint32_t)nx.fr), fs = uni((uint32_t)nx.fs);
            asm volatile("s_waitcnt vmcnt(%5) lgkmcnt(0)\n\ts_barrier"
                         : "+s"(nx.shift), "+s"(fr), "+s"(fs), "+s"(nx.kbytes_b), "+s"(seg) : "n"(OUTSTANDING) : "memory");
            nx.fr = (int)fr; nx.fs = (int)fs;
        } else {
            nx.kbytes = uni(nx.kbytes);
            asm volatile("s_waitcnt vmcnt(%3) lgkmcnt(0)\n\ts_barrier"
                         : "+s"(nx.kbytes), "+s"(nx.kbytes_b), "+s"(seg) : "n"(OUTSTANDING) : "memory");
        }
        if constexpr (DEP == 2) {
            if (__builtin_expect(seg != 0, 0)) dep_before_request(kreq, reqB, true);
        }
    };
    auto advance = [&](uint32_t& st, uint32_t n) __attribute__((always_inline)) { st = (st + 1 == n) ? 0 : st + 1; };
    static_assert(KK % 2 == 0, "fragment buffers alternate with the slices");

    // head: step kb's stage is handed over, its requests go out with slices 0 .. KK-2 (the groups
    // that the missing slice before them would have carried are issued at once)
    uint32_t curA = 0, curB = 0;
    hand_over(kb);
    const char* la = lds;
    const char* lb = lds + Cfg::B_BASE;
    load_frags(0, la, lb, 0);
#pragma unroll
    for (int g = 0; g < FM; ++g) dma_group(g);
#pragma unroll
    for (int kk = 0; kk < KK - 1; ++kk) slice(kk & 1, la, lb, kk + 1, (kk + 1) * FM);
    advance(reqA, NSA); advance(reqB, NSB);
    for (uint32_t kt = kb + 1; kt < ke; ++kt) {
        // the last fragments of step kt-1 are in registers: hand over step kt's stage, multiply
        // them while step kt's first fragments are read, then step kt's slices 0 .. KK-2
        hand_over(kt);
        advance(curA, NSA); advance(curB, NSB);
        la = lds + curA * Cfg::A_BYTES;
        lb = lds + Cfg::B_BASE + curB * Cfg::B_BYTES;
        slice((KK - 1) & 1, la, lb, 0, 0);
#pragma unroll
        for (int kk = 0; kk < KK - 1; ++kk) slice(kk & 1, la, lb, kk + 1, (kk + 1) * FM);
        advance(reqA, NSA); advance(reqB, NSB);
    }
    slice((KK - 1) & 1, nullptr, nullptr, -1, -1);   // tail: the last slice of the last step
    // every DMA into LDS has landed before the staging area is given up
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    dr.peek();   // the look at the dispatch queues for this workgroup's next tile travels during the epilogue

    if constexpr (Cfg::WK > 1) {   // the waves of a sub-tile add up
        static_assert(Cfg::WK == 2 && FM * FN == 1 && Cfg::MINB > 1, "two waves, one block each");
        float* const half = reinterpret_cast<float*>(lds) + (wave % NW) * 1024 + lane;
        __syncthreads();   // every wave has read its last operand fragments
        if (!holds) {
#pragma unroll
            for (int v = 0; v < 16; ++v) half[v * 64] = acc[0][0][v];
        }
        __syncthreads();
        if (holds) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[0][0][v] += half[v * 64];
        }
    }
    constexpr uint32_t NT = 64 * NW;   // threads that hold values of the tile

    // ---- split-K: leave the partial tile, and carry on only as the last part to arrive ----
    bool finish = !SLICED || S == 1;
    if (!SLICED && S > 1) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const uint32_t tile_lin = ty * s.grid_x + tx;
        const float* const part = s.partials + (size_t)tile_lin * S * (TM * TN);
        // fragment order: each lane stores 16 bytes next to its neighbours' (1 KB per instruction),
        // written through to memory so that the count below can follow without a write-back
        // of this XCD's whole L2
        const ThroughBuf mine(uni_ptr(part + (size_t)kz * (TM * TN)));
        if (holds) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v4 = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                        mine.store16(tid * 16u, ((i * FN + j) * 4 + q) * NT * 16u, __builtin_bit_cast(u32x4, v4));
                    }
        }
        // the partial is in memory before the count moves (every wave's stores, then the barrier)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        uint32_t* slot = reinterpret_cast<uint32_t*>(lds);
        if (tid == 0) {
            const uint32_t old = __hip_atomic_fetch_add(s.arrive + tile_lin * SYNC_WORD_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            slot[0] = old;
        }
        __syncthreads();
        finish = __builtin_amdgcn_readfirstlane(slot[0]) == S - 1;
        __syncthreads();
        if (finish) {
            // Every part's partial is in memory (each counted after its stores had completed) and none of
            // these lines has been read on this XCD since the kernel started.  Sum in K order,
            // whoever came last, so that the result does not depend on the arrival order.
            if (tid == 0) __hip_atomic_store(s.arrive + tile_lin * SYNC_WORD_STRIDE, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // The sum is p0 + p1 + p2 + ... from the left.  A finisher that holds part 0 or
            // part 1 starts from its registers (p1 + p0 and p0 + p1 are the same number) and
            // skips reading its own partial back; any other starts from zero and reads them all.
            const bool own = kz <= 1;
            if (!own) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
            }
            // The partials were written on other XCDs and come from memory: a read costs a round
            // trip of a couple of microseconds whatever its size, and a skinny chain's tile has
            // little else left to do.  So the loads of as many whole parts as the registers
            // beside the accumulators hold (PARTS_IN_FLIGHT) are issued before the first of them
            // is added; the adds stay in K order.
            constexpr int ACCF = FM * FN * 16;                                   // accumulator floats per lane
            constexpr int ROOM = Cfg::MINB == 1 ? (472 - ACCF < 192 ? 472 - ACCF : 192) : (Cfg::MINB == 2 ? 216 : 112) - ACCF;
            constexpr int PARTS_IN_FLIGHT = ROOM / ACCF > 8 ? 8 : ROOM / ACCF;
            const uint32_t at = holds ? tid << 2 : 0u;   // (a wave that holds nothing adds up what nobody reads)
            if constexpr (PARTS_IN_FLIGHT >= 1) {
                constexpr int NV = FM * FN * 4;                                  // 16-byte loads per lane and part
                for (uint32_t z0 = 0; z0 < S; z0 += PARTS_IN_FLIGHT) {
                    f32x4 t4[PARTS_IN_FLIGHT][NV];
                    // (parts past the end read the last part again and are not added: the loads stay
                    // unconditional, so that all of a batch are in flight together)
#pragma unroll
                    for (int d = 0; d < PARTS_IN_FLIGHT; ++d) {
                        const uint32_t z = min(z0 + d, S - 1);
                        const float* src = part + (size_t)z * (TM * TN) + at;
#pragma unroll
                        for (int u = 0; u < NV; ++u) t4[d][u] = *(const f32x4*)(src + u * NT * 4);
                    }
#pragma unroll
                    for (int d = 0; d < PARTS_IN_FLIGHT; ++d) {
                        const uint32_t z = z0 + d;
                        if (z < S && !(own && z == kz)) {
#pragma unroll
                            for (int i = 0; i < FM; ++i)
#pragma unroll
                                for (int j = 0; j < FN; ++j)
#pragma unroll
                                    for (int q = 0; q < 4; ++q)
#pragma unroll
                                        for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += t4[d][(i * FN + j) * 4 + q][e];
                        }
                    }
                }
            } else {
                // no room for a whole part: one row of blocks of one part at a time
                for (uint32_t z = 0; z < S; ++z) {
                    if (own && z == kz) continue;
                    const float* src = part + (size_t)z * (TM * TN) + at;
#pragma unroll
                    for (int i = 0; i < FM; ++i) {
                        f32x4 t4[FN][4];
#pragma unroll
                        for (int j = 0; j < FN; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) t4[j][q] = *(const f32x4*)(src + ((i * FN + j) * 4 + q) * NT * 4);
#pragma unroll
                        for (int j = 0; j < FN; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += t4[j][q][e];
                    }
                }
            }
        }
    }

    // ---- epilogue: activation, round to 16 bits, store ----
    // Accumulator layout of the 32x32 block: lane holds column (lane % 32) and rows
    // 8*(v/4) + 4*(lane/32) + v%4 for v = 0..15, i.e. a lane's values run DOWN a column.  Each
    // wave therefore transposes its sub-tile, 32 or 64 rows at a time (BR) and in fp32, through its own piece of the
    // (now idle) operand staging area, and a loop over 16-byte row segments applies the activation,
    // rounds and stores: whole lines instead of 2-byte pieces for the write-through stores.  The loop is
    // what keeps the code short: with the activation unrolled over the accumulators a kernel was 70 to 290
    // KB of straight code, executed once per tile and fetched from memory each time a chain's weights
    // had swept it out of the L2.  (A convolution has ReLU or nothing: its kernels hold no code for the others, which
    // takes 2-4 % off the chains of short tiles: four of 9x59x59x64 in fp16 68.4 -> 66.2 us.)
    constexpr int PITCH = Cfg::WTN * 4 + 16;                    // bytes per row of a wave's piece of the staging area
    constexpr int BR = FM >= 3 ? 2 : 1;                         // block rows transposed at a time
    constexpr int WROWS = BR * 32;                              // rows of a piece (a slice of a split tile, at most half of the wave's rows, fits too)
    static_assert(WROWS >= FM * 16, "half of the wave's rows");
    constexpr int SLOT = Cfg::LDS_BYTES - 64;                   // word of the staging area behind all four pieces
    static_assert(4 * WROWS * PITCH <= SLOT, "the pieces of every wave fit the staging area");
    char* const reg = lds + wave * (WROWS * PITCH);
    const uint32_t act = s.act;
    T* const Cp = (T*)s.C;
    const uint32_t wtn_out = gate_up ? Cfg::WTN / 2 : Cfg::WTN;  // output columns of this wave
    const uint32_t cpr = wtn_out / 8;                            // 16-byte chunks per row
    const uint32_t col0 = n0 + wn * wtn_out;
    constexpr uint32_t CPR = Cfg::WTN / 8, CPR_GU = Cfg::WTN / 16;
    const uint32_t r_first = gate_up ? lane / CPR_GU : lane / CPR, ch_first = lane - r_first * cpr;
    const uint32_t r_step = gate_up ? 64 / CPR_GU : 64 / CPR, ch_step = gate_up ? 64 % CPR_GU : 64 % CPR;
    uint32_t ldc = uni(s.ldc);
    asm volatile("" : "+s"(ldc));                                // (kept: the loop would read the kernel argument again per segment)
    const ThroughBuf out(uni_ptr(Cp));                           // (an output is smaller than 4 GiB)
    // Rows 0 .. rows-1 of the wave's piece are rows row0 .. of the output: activation, rounding, store.
    auto store_rows = [&](uint32_t row0, uint32_t rows) __attribute__((always_inline)) {
        uint32_t r = r_first, ch = ch_first;
#pragma unroll 1
        for (; r < rows; r += r_step, ch += ch_step) {
            if (ch >= cpr) { ch -= cpr; if (++r >= rows) break; }
            const uint32_t col = col0 + ch * 8;
            if (col >= sN) continue;
            float x[8];
            // gate and up columns alternate in blocks of 32
            const char* src = reg + r * PITCH + (gate_up ? (ch >> 2) * 256 + (ch & 3u) * 32 : ch * 32);
            __builtin_memcpy(x, __builtin_assume_aligned(src, 16), 32);
            if (gate_up) {
                float u[8];
                __builtin_memcpy(u, __builtin_assume_aligned(src + 128, 16), 32);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = silu_f(x[e]) * u[e];
            } else if (AMODE != A_CONV3X3 && act == ACT_GELU) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = gelu_erf(x[e]);
            } else if (act == ACT_RELU) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = fmaxf(x[e], 0.0f);
            }
            V8 val;
#pragma unroll
            for (int e = 0; e < 8; ++e) val[e] = (T)x[e];
            const uint32_t at = (row0 + r) * ldc + col;
            T* dst = Cp + at;
            if (col + 8 <= sN) {
                if constexpr (THROUGH) out.store16(at * 2u, 0, __builtin_bit_cast(u32x4, val));
                else *(V8*)dst = val;
            } else {
                for (uint32_t e = 0; e < sN - col; ++e) store_out<THROUGH>(dst + e, (T)val[e]);
            }
        }
    };
    if (!SLICED || S == 1) {
        __syncthreads();   // every wave has read its last operand fragments
        if (wctx.ok && finish && holds) {
#pragma unroll
            for (int i0 = 0; i0 < FM; i0 += BR) {
                // the region is private to the wave: its own LDS writes are ordered before its reads
                char* const w = reg + ((lane >> 5) * 4u) * PITCH + (lane & 31u) * 4u;
#pragma unroll
                for (int i = i0; i < FM && i < i0 + BR; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) *(float*)(w + ((i - i0) * 32 + 8 * (v / 4) + (v % 4)) * PITCH + j * 128) = acc[i][j][v];
                if (i0 == 0) dr.grab();   // the counters read by peek() have arrived by now: start the next tile's draw
                const uint32_t row0 = m0 + wm * Cfg::WTM + i0 * 32;
                constexpr uint32_t most = BR * 32;
                store_rows(row0, row0 < sM ? min(sM - row0, FM - i0 < BR ? (uint32_t)(FM - i0) * 32u : most) : 0u);
            }
        }
    } else {
        // ---- split along K: the parts exchange partial tiles, and each finishes a slice of the rows ----
        // The wave's rows come in groups of 4 (what one half of a wave holds of a column in 4 accumulator registers:
        // group 2 * (4 * i + q) + h, registers 4 * q .. 4 * q + 3 of block row i, lanes of half h).  Slice z, the groups
        // slice_lo(z) .. slice_lo(z + 1) - 1 of those that have rows of the matrix, is finished by part z: it leaves
        // everything but that slice in the scratch buffer, waits for the other parts to have done the same, adds
        // their partials to its own in K order (the same bits whoever comes last), and stores the slice.
        // With one part finishing the whole tile, the last to arrive, that workgroup alone read S - 1 partial tiles
        // back at one CU's rate behind a write-through of its own (64 x 192 tiles split in eight: 13 us).
        //
        // A part waits only if every part of its tile has been started: those are held by resident workgroups that
        // end without its help.  If one has not been (the chip is shared with other work), the part leaves its own
        // slice in the buffer as well, says so and goes on; the last part to publish finishes such slices.
        // Consumers see one post per tile, as without the split, by the last part to leave.
        // (What is done with the tile's word, in order: split_word.hpp.)
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const uint32_t tile_lin = ty * s.grid_x + tx;
        const float* const part = s.partials + (size_t)tile_lin * S * (TM * TN);
        auto sem_waits = [&]() __attribute__((always_inline)) {   // (segments of a part, row tiles of the producer at each)
            if constexpr (DEP == 0) return 0u;
            else return (seg_steps ? (ke - kb) / seg_steps + 1u : 1u) * ((TM + (AMODE == A_CONV3X3 ? 2 * (cW + 1) : 0u)) / s.prod_tm + 2);
        };
        PartsWord<decltype(sem_waits)> word{s.arrive + tile_lin * SYNC_WORD_STRIDE, wctx, sem_waits};
        volatile uint32_t* const slot = reinterpret_cast<uint32_t*>(lds + SLOT);
        const uint32_t tile_rows = min(sM - m0, (uint32_t)TM);
        const uint32_t wave_row0 = wm * Cfg::WTM;
        const uint32_t groups = (min(tile_rows, (uint32_t)Cfg::WTM) + 3) / 4;          // with rows of the matrix, first row of waves
        const uint32_t my_groups = tile_rows > wave_row0 ? (min(tile_rows - wave_row0, (uint32_t)Cfg::WTM) + 3) / 4 : 0;
        auto slice_lo = [&](uint32_t z) __attribute__((always_inline)) { return (z * groups + S - 1) / S; };
        const uint32_t h = lane >> 5;
        const uint32_t own_lo = slice_lo(kz), own_hi = slice_lo(kz + 1);

        uint32_t seen = 0;
        if (tid == 0) seen = word.load();   // in flight beside the stores
        // The own slice goes to LDS, transposed.  The rest goes to the buffer in fragment order: each lane stores 16 bytes
        // next to its neighbours' (1 KB per instruction), written through to memory so that the count can follow
        // without a write-back of this XCD's whole L2.
        const ThroughBuf mine(uni_ptr(part + (size_t)kz * (TM * TN)));
        char* const w = reg + (lane & 31u) * 4u;
        __syncthreads();   // every wave has read its last operand fragments
#pragma unroll
        for (int u = 0; u < FM * 4; ++u) {
            const uint32_t g = 2 * u + h;
            if (2 * u < my_groups) {
                if (g >= own_lo && g < own_hi) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) *(float*)(w + (4 * (g - own_lo) + e) * PITCH + j * 128) = acc[u / 4][j][4 * (u % 4) + e];
                } else if (g < my_groups) {
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        const f32x16& c = acc[u / 4][j];
                        const f32x4 v4 = {c[4 * (u % 4)], c[4 * (u % 4) + 1], c[4 * (u % 4) + 2], c[4 * (u % 4) + 3]};
                        mine.store16(tid * 16u, (((u / 4) * FN + j) * 4 + u % 4) * 4096, __builtin_bit_cast(u32x4, v4));
                    }
                }
            }
        }
        // the partial is in memory before the count moves (every wave's stores, then the barrier)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) *slot = split_publish(word, S, kz, own_lo != own_hi, split_all_started(seen, S));
        __syncthreads();
        uint32_t todo = uni(*slot);
        dr.grab();   // the counters read by peek() have arrived by now: start the next tile's draw
        if (todo == SPLIT_AGAIN) {
#pragma unroll 1
            for (uint32_t u = own_lo / 2; u < (min(own_hi, my_groups) + 1) / 2; ++u) {
                const uint32_t g = 2 * u + h;
                if (g < own_lo || g >= min(own_hi, my_groups)) continue;
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    f32x4 v4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v4[e] = *(const float*)(w + (4 * (g - own_lo) + e) * PITCH + j * 128);
                    mine.store16(tid * 16u + (((u >> 2) * FN + j) * 4 + (u & 3u)) * 4096u, 0, __builtin_bit_cast(u32x4, v4));
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();                                     // (and everyone has read the slot)
            if (tid == 0) *slot = split_publish_whole(word, S, kz);
            __syncthreads();
            todo = uni(*slot);
        }
        // Sum of the S <= Z parts of a slice (groups lo .. hi - 1) in K order, in fragment order, to its place in LDS.  The
        // partials were written on other CUs and a read costs a round trip of a microsecond or two whatever its size: the
        // loads of all parts of NB pieces (8 rows x 32 columns per wave) are in flight together.
        auto sum_slice = [&](uint32_t lo, uint32_t hi, bool own, auto zc, auto nbc) __attribute__((always_inline)) {
            constexpr int Z = decltype(zc)::value, NB = decltype(nbc)::value;
            const uint32_t n_end = (hi + 1) / 2 * FN;
#pragma unroll 1
            for (uint32_t n0 = lo / 2 * FN; n0 < n_end; n0 += NB) {
                f32x4 t[NB][Z];
#pragma unroll
                for (int z = 0; z < Z; ++z) {
                    if ((uint32_t)z >= S || (own && (uint32_t)z == kz)) continue;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const uint32_t n = min(n0 + b, n_end - 1), u = n / FN, j = n % FN;
                        t[b][z] = *(const f32x4*)(part + (size_t)z * (TM * TN) + (((u >> 2) * FN + j) * 4 + (u & 3u)) * 1024 + tid * 4);
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const uint32_t n = n0 + b, u = n / FN, j = n % FN, g = 2 * u + h;
                    if (n >= n_end || g < lo || g >= hi) continue;
                    char* const p = w + (4 * (g - lo)) * PITCH + j * 128;
                    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int z = 0; z < Z; ++z) {
                        if ((uint32_t)z >= S) continue;
                        if (own && (uint32_t)z == kz) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) sum[e] += *(const float*)(p + e * PITCH);
                        } else {
                            sum += t[b][z];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) *(float*)(p + e * PITCH) = sum[e];
                }
            }
        };
#pragma unroll 1
        for (uint32_t i = 0; i < S; ++i) {                       // the own slice first: it lies in LDS
            const uint32_t z0 = kz + i < S ? kz + i : kz + i - S;
            if (!((todo >> z0) & 1u)) continue;
            const uint32_t lo = slice_lo(z0), hi = min(slice_lo(z0 + 1), my_groups);
            if (lo < hi) {
                if (S <= 3) sum_slice(lo, hi, i == 0, std::integral_constant<int, 3>(), std::integral_constant<int, 6>());
                else sum_slice(lo, hi, i == 0, std::integral_constant<int, 8>(), std::integral_constant<int, 2>());
                const uint32_t row0 = m0 + wave_row0 + 4 * lo;
                if (wctx.ok) store_rows(row0, min(4 * (hi - lo), sM - row0));
            }
        }
        // (the part's slices are in memory before it leaves)
        if (SYNC && s.post_kind != DEP_NONE) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        if (tid == 0) {
            if (SYNC && !THROUGH && s.post_kind != DEP_NONE) write_back_l2();
            split_leave(word, S, SYNC && args.draw_cas != 0, [&]() __attribute__((always_inline)) {
                if (SYNC && s.post_kind != DEP_NONE) post_sem(args, s, tile_lin, tx, ty);
            });
        }
    }

    if (SYNC && finish) post_tile<THROUGH>(args, s, ty * s.grid_x + tx, tx, ty);
    if (tracing && tid == 0) {
        TraceRec r;
        r.rel = rel_ticket; r.where = hw_where(DEP ? 1u : 0u); r.tx = tx; r.ty = tyz;
        r.t_enter = t_enter; r.t_start = t_start; r.t_ready = t_ready; r.t_end = now_ticks();
        args.trace[rel_ticket] = r;
    }
}

}  // namespace depsync
