// Matrix-core attention over the assembled cache with the unit's TOKENS split over the waves,
// bf16, head_dim 128: the decode step (paper Section V-A "decode time": the newest token of
// each instance over every chunk key and the whole tail), alone or fused with the projection of
// that token's K/V (Section III-B steps 2-3), and - as the fallback of the row-parallel kernel in
// attn_prefill.hip - the question prefill (rows i of the question over every chunk key and
// question keys j <= i).
//
// The M dimension of the tiles is the flattened (question row, query head of one KV head)
// index, so the G query heads that share a KV head ride in the same matrix-core operation.
// Per wave and per block of 32 token rows:
//   S^T = K Q^T     mfma 16x16x32: A = K rows straight from HBM in operand layout (16 tokens x
//                   8 consecutive dims per lane), B = Q held in registers for the whole unit
//   softmax         per lane on its own column (one (row, head)) with a running maximum that
//                   the four 16-lane groups agree on through register swaps
//   O^T += V^T P^T  A = V transposed on the fly: V rows land in a private LDS strip as loaded
//                   (coalesced 16-byte loads) and come back through the transposing LDS read,
//                   B = P rounded to bf16, already sitting in operand layout
// Waves of a workgroup split the unit's tokens; workgroups split the cache; merging is the
// same as in the plain-ALU kernel.
#include <type_traits>

#include "attn_common.h"
#include "gemv_common.h"

namespace matkv {
namespace {

using namespace attn;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int D = 128;
constexpr int BLK = 32;             // token rows per wave step
constexpr int VSTR = D + 16;        // bf16 elements per LDS row of the V strip (bank spread)
constexpr int ACCS = D + 4;         // floats per LDS row of the merge buffer

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& r) { return __builtin_bit_cast(bf16x8, r); }

// Transposing LDS read: the 16 lanes of a group each name 8 bytes (4 bf16); lane i of the group
// receives element i of the group's four 16-element rows.
__device__ __forceinline__ s16x4 lds_read_tr(const uint16_t* p) {
    typedef s16x4 __attribute__((address_space(3))) * lptr;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(uintptr_t)p);
}

// What a fused decode step adds to the attention launch (paper Section III-B steps 2-3 for the
// newest token of every instance, then Section V-A's decode attention over everything).
struct StepArgs {
    const void* hidden;         // [batch][Hd]
    const void* w_k;            // [Hkv * D][Hd]
    const void* w_v;
    const RopeEntry* rope;
    int32_t Hd, batch;
    int32_t workgroups;         // per KV head
};

// The NS waves' states of a decode tile's rows (accumulators WS floats apart) to the workgroup's partials, with agent-scope
// stores.  A wave takes RB rows at a time, lane l the dims 2l, 2l + 1: where a row goes is then the same for all lanes, and everything it
// needs of LDS is read at once.  (By columns over all threads, as the fallback prefill does it, it took 1 us of a step.)
template <int NWV, int NS, int ROWS, int WS, int RB, typename MapFn>
__device__ __forceinline__ void publish_rows(const KernelArgs& a, const float* sm_acc, const float* sm_m, const float* sm_l, int n_rows,
                                             MapFn map, int wave, int lane) {
    lds_barrier();                                      // (global stores may still be on their way)
    for (int i0 = wave; i0 < n_rows; i0 += NWV * RB) {
        float m[RB][NS], l[RB][NS];
        float2 v[RB][NS];
        float* prow[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = min(i0 + NWV * r, n_rows - 1);
#pragma unroll
            for (int w = 0; w < NS; ++w) {
                m[r][w] = sm_m[w * ROWS + i];
                l[r][w] = sm_l[w * ROWS + i];
                v[r][w] = *reinterpret_cast<const float2*>(sm_acc + w * WS + i * ACCS + 2 * lane);
            }
            const RowMap rm = map(i);
            prow[r] = a.partials + ((size_t)(rm.unit_slot >= 0 ? rm.unit_slot : (int)blockIdx.x) * a.Hq + rm.head) * kPartialStride(D);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            float mn = m[r][0];
#pragma unroll
            for (int w = 1; w < NS; ++w) mn = fmaxf(mn, m[r][w]);
            float ax = 0.f, ay = 0.f, lv = 0.f;
#pragma unroll
            for (int w = 0; w < NS; ++w) {
                const float c = fast_exp2(m[r][w] - mn);
                ax = fmaf(v[r][w].x, c, ax);
                ay = fmaf(v[r][w].y, c, ay);
                lv = fmaf(l[r][w], c, lv);
            }
            if (RB > 1 && i0 + NWV * r >= n_rows) break;
            st_agent2(prow[r] + 2 * lane, ax, ay);
            if (lane == 0) st_agent2(prow[r] + D, mn, lv);
        }
    }
}

// Folding the partials of a decode launch.  A wave takes RB output rows (an instance's newest token, one
// query head) at a time; its lower half takes the even units, its upper half the odd ones, lane l of a half the dims
// 4l .. 4l + 3.  Per pass of UPC units lane k fetches the (maximum, sum) of unit k of every row, and all loads of the pass are
// requested before anything is consumed: one memory round trip for UPC units of RB rows, in 16-byte loads (loads past the L2s
// leave one after the other: 32 units of a row 1.6 us in 8-byte ones).  The wave agrees on the maximum, every lane has the
// weight of its unit and hands it to the half that needs it.
// src[i]: partial of row i's first unit; n[i]: its units (0: row not taken); ustride: floats between units.
// meanwhile(): done while the first pass's loads are on their way.
template <int RB, int UPC, typename F>
__device__ __forceinline__ void fold_partials(const float* const (&src)[RB], const int (&n)[RB], uint32_t ustride, int lane,
                                              float (&M)[RB], float (&L)[RB], float4 (&o)[RB], F meanwhile) {
    static_assert(UPC <= 64 && UPC % 2 == 0, "a lane per unit, two units a load");
    const int half = lane >> 5, l32 = lane & 31;
    int nmax = 0;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        nmax = max(nmax, n[i]);
        M[i] = kNegBig; L[i] = 0.f; o[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int u0 = 0; u0 < nmax; u0 += UPC) {
        float4 av[RB][UPC / 2];
        float2 ml[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) ml[i] = ld_agent2(src[i] + (size_t)min(u0 + lane, max(n[i], 1) - 1) * ustride + D);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const uint32_t top = (uint32_t)(max(n[i], 1) - 1) * ustride * 4;        // (past a row's units: its last one again)
            uint32_t off = (uint32_t)(u0 + half) * ustride * 4;
#pragma unroll
            for (int k = 0; k < UPC / 2; ++k, off += 8 * ustride) av[i][k] = dev::ld_agent4(src[i], min(off, top) + 16 * l32);
        }
        if (u0 == 0) meanwhile();
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const bool own = lane < UPC && u0 + lane < n[i];
            const float mn = fmaxf(M[i], gemv::wave_max(own ? ml[i].x : kNegBig, lane));
            const float w = own ? fast_exp2(ml[i].x - mn) : 0.f;
            const float cold = fast_exp2(M[i] - mn);
            L[i] = fmaf(L[i], cold, gemv::wave_sum(w * ml[i].y, lane));
            o[i].x *= cold; o[i].y *= cold; o[i].z *= cold; o[i].w *= cold;
            M[i] = mn;
            const int wi = __float_as_int(w);
#pragma unroll
            for (int k = 0; k < UPC / 2; ++k) {
                const float c = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (2 * k + half), wi));
                o[i].x = fmaf(av[i][k].x, c, o[i].x); o[i].y = fmaf(av[i][k].y, c, o[i].y);
                o[i].z = fmaf(av[i][k].z, c, o[i].z); o[i].w = fmaf(av[i][k].w, c, o[i].w);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {                      // the halves' sums together, in either
        o[i].x += lane_xor(o[i].x, 32, lane); o[i].y += lane_xor(o[i].y, 32, lane);
        o[i].z += lane_xor(o[i].z, 32, lane); o[i].w += lane_xor(o[i].w, 32, lane);
    }
}
// One row out, from the lower half of a wave.
__device__ __forceinline__ void store_row(const KernelArgs& a, size_t row, int lane, const float4& o, float inv) {
    if (lane < 32) store_out4(a.out, a.out_f32, row * D + 4 * lane, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
}

// Last arrival at (instance, KV head) of a plain decode launch: NWV waves fold the G rows.
template <int G, int NWV, int UPC>
__device__ __forceinline__ void merge_decode(const KernelArgs& a, const Unit& unit, int kvh, int wave, int lane) {
    constexpr int PSTRIDE = kPartialStride(D), RB = (G + NWV - 1) / NWV;
    const float* src[RB];
    int n[RB];
    float M[RB], L[RB];
    float4 o[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int g = wave + NWV * i;
        n[i] = g < G ? unit.n_units_inst : 0;
        src[i] = a.partials + ((size_t)unit.unit0_inst * a.Hq + kvh * G + min(g, G - 1)) * PSTRIDE;
    }
    fold_partials<RB, UPC>(src, n, (uint32_t)a.Hq * PSTRIDE, lane, M, L, o, []() {});
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        if (n[i] == 0) continue;
        store_row(a, (size_t)unit.inst * a.Hq + kvh * G + wave + NWV * i, lane, o[i], 1.0f / L[i]);
    }
}

// Last arrivals of a fused decode step at KV head kvh: folds, for every instance at whose counter the
// workgroup arrived last, the units' partials and the newest token into the G output rows - all such
// instances at once.  The newest token's K/V row is read back from the tail cache, where the projection
// waves left it with agent-scope stores; its score is a 64-lane dot product, and it enters as one more
// contribution of weight 1.  What a wave's rows are is looked up before the workgroup arrives.
template <int G, int NWV, int RB>
struct StepRows {
    const float* src[RB];
    int n[RB], b[RB];
    uint32_t qw[RB];
    size_t toff[RB], row[RB];
    __device__ __forceinline__ StepRows(const KernelArgs& a, const InstanceInfo* __restrict__ insts, int batch, int kvh, int wave, int lane) {
        const int rows = batch * G;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int r = min(wave + NWV * i, rows - 1), head = kvh * G + r % G;
            b[i] = r / G;
            const InstanceInfo inst = insts[b[i]];
            n[i] = wave + NWV * i < rows ? inst.n_dunits : 0;
            src[i] = a.partials + ((size_t)inst.dunit0 * a.Hq + head) * kPartialStride(D);
            toff[i] = (((size_t)b[i] * a.Hkv + kvh) * (size_t)a.max_tail + (size_t)max(inst.tail_len - 1, 0)) * D;
            row[i] = (size_t)b[i] * a.Hq + head;
            qw[i] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint16_t*>(a.q) + row[i] * D + 2 * lane);
        }
    }
};
template <int G, int NWV, int RB, int UPC>
__device__ __forceinline__ void merge_decode_step(const KernelArgs& a, const StepRows<G, NWV, RB>& rows, const int* lastv, int lane) {
    typedef uint16_t T;
    int n[RB], any = 0;
#pragma unroll
    for (int i = 0; i < RB; ++i) { n[i] = __builtin_amdgcn_readfirstlane(lastv[rows.b[i]]) ? rows.n[i] : 0; any |= n[i]; }
    if (any == 0) return;
    uint32_t kw[RB];
    uint64_t vw[RB];
    float M[RB], L[RB], sx[RB];
    float4 o[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        kw[i] = __hip_atomic_load(reinterpret_cast<const uint32_t*>(reinterpret_cast<const T*>(a.tail_k) + rows.toff[i] + 2 * lane),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        vw[i] = __hip_atomic_load(reinterpret_cast<const uint64_t*>(reinterpret_cast<const T*>(a.tail_v) + rows.toff[i] + 4 * (lane & 31)),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    fold_partials<RB, UPC>(rows.src, n, (uint32_t)a.Hq * kPartialStride(D), lane, M, L, o, [&]() {
#pragma unroll
        for (int i = 0; i < RB; ++i) sx[i] = gemv::wave_sum(gemv::dot2(rows.qw[i], kw[i], 0.f), lane) * a.scale_log2e;
    });
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        if (n[i] == 0) continue;
        const float mn = fmaxf(M[i], sx[i]);
        const float cold = fast_exp2(M[i] - mn), cx = fast_exp2(sx[i] - mn);
        const float l = fmaf(L[i], cold, cx);
        const uint32_t v01 = (uint32_t)vw[i], v23 = (uint32_t)(vw[i] >> 32);
        o[i].x = fmaf(o[i].x, cold, __uint_as_float(v01 << 16) * cx);
        o[i].y = fmaf(o[i].y, cold, __uint_as_float(v01 & 0xffff0000u) * cx);
        o[i].z = fmaf(o[i].z, cold, __uint_as_float(v23 << 16) * cx);
        o[i].w = fmaf(o[i].w, cold, __uint_as_float(v23 & 0xffff0000u) * cx);
        store_row(a, rows.row[i], lane, o[i], 1.0f / l);
    }
}

// A projection wave of a fused decode step: one task = one rotary pair of K or of V of KV head
// kvh for a group of FR instances; the pair is stored (bf16, agent scope) at the newest tail
// row of each instance.  The n_waves projection waves of this KV head share the tasks round-robin.
template <int FR, bool AHEAD>
__device__ __forceinline__ void projection_tasks(const KernelArgs& a, const StepArgs& f, const InstanceInfo* __restrict__ insts,
                                                 int kvh, int wave_id, int n_waves, int lane) {
    typedef uint16_t T;
    const int groups = (f.batch + FR - 1) / FR;
    for (int task = wave_id; task < groups * D; task += n_waves) {
        const int b0 = (task / D) * FR;
        const int kv = (task % D) / (D / 2), j = task % (D / 2);
        const T* w = reinterpret_cast<const T*>(kv == 0 ? f.w_k : f.w_v);
        const T* w0 = w + ((size_t)kvh * D + j) * f.Hd;
        const T* w1 = w0 + (size_t)(D / 2) * f.Hd;
        const T* x = reinterpret_cast<const T*>(f.hidden) + (size_t)b0 * f.Hd;
        // AHEAD (several instances): where the pair goes and how far it is turned is asked for ahead of the weights instead of behind the sums (us per pass of eight
        // layers, three 3B users of a few hundred tokens 1368 -> 1318, four 8B users of 3000 1189 -> 1161).  For one these are scalar loads, which the weights would wait
        // for (8B, 10 000 tokens 988 -> 1022); behind the weights it gives less (1372, 1182; 989).  Which launches do, see launch_step_v.
        struct Place { int row; int64_t pos_base; RopeEntry turn; } at;
        auto look_up = [&](int b) { at.row = insts[b].tail_len - 1; at.pos_base = insts[b].pos_base; at.turn = f.rope[j]; };
        if (AHEAD) look_up(min(b0 + lane % FR, f.batch - 1));
        float acc0[FR], acc1[FR];
        if (f.Hd % 4096 == 0) gemv::pair_dots<FR, 8>(w0, w1, x, (size_t)f.Hd, f.batch - b0, f.Hd, lane, acc0, acc1);
        else                  gemv::pair_dots<FR, 6>(w0, w1, x, (size_t)f.Hd, f.batch - b0, f.Hd, lane, acc0, acc1);   // multiples of 3072
        if (lane < FR && b0 + lane < f.batch) {
            float r0 = 0.f, r1 = 0.f;
#pragma unroll
            for (int r = 0; r < FR; ++r) if (lane == r) { r0 = acc0[r]; r1 = acc1[r]; }
            const int b = b0 + lane;
            const int row = AHEAD ? at.row : insts[b].tail_len - 1;
            if (row >= 0 && row < a.max_tail) {
                if (kv == 0) {
                    if (!AHEAD) look_up(b);
                    gemv::rotate_pair(at.turn, (float)(at.pos_base + row), r0, r1);
                }
                T* out = reinterpret_cast<T*>(const_cast<void*>(kv == 0 ? a.tail_k : a.tail_v)) +
                         (((size_t)b * a.Hkv + kvh) * (size_t)a.max_tail + (size_t)row) * D + j;
                __hip_atomic_store(out, f32_to_bf16_rne(r0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(out + D / 2, f32_to_bf16_rne(r1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// Shared decode units: fold, for every user of this unit at whose counter the workgroup arrived
// last (the first n_live entries of live), that instance's partial slots into its G output rows - all such users at once.
// users[u] = {instance, this unit's slot, first slot, slots}.
template <int G, int NWV, int RB, int UPC>
__device__ __forceinline__ void merge_shared(const KernelArgs& a, const int4* users, const int* live, int n_live, int kvh, int wave, int lane) {
    constexpr int PSTRIDE = kPartialStride(D);
    const int rows = n_live * G;
    for (int r0 = wave; r0 < rows; r0 += NWV * RB) {
        const float* src[RB];
        int n[RB];
        size_t row[RB];
        float M[RB], L[RB];
        float4 o[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int r = min(r0 + NWV * i, rows - 1), head = kvh * G + r % G;
            const int4 us = users[live[r / G]];
            n[i] = r0 + NWV * i < rows ? __builtin_amdgcn_readfirstlane(us.w) : 0;
            src[i] = a.partials + ((size_t)__builtin_amdgcn_readfirstlane(us.z) * a.Hq + head) * PSTRIDE;           // decode: one row per slot
            row[i] = (size_t)us.x * a.Hq + head;
        }
        fold_partials<RB, UPC>(src, n, (uint32_t)a.Hq * PSTRIDE, lane, M, L, o, []() {});
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (n[i] == 0) continue;
            store_row(a, row[i], lane, o[i], 1.0f / L[i]);
        }
    }
}

// (Second launch bound: two waves per SIMD, i.e. at most 256 registers, wherever the decode
// tile fits them - a few registers more would halve the workgroups resident per compute unit.)
// FR = 0: attention only, NW waves.  FR > 0: fused decode step - the workgroup has NW more
// waves, which project the newest token's K/V (FR instances per task) while the first NW walk
// the cache; every compute unit then holds both kinds of work side by side.  In that form each
// workgroup of a KV head arrives at the counter of EVERY instance of the batch once all its
// work is out, so the last arrival at an instance's counter knows that instance's partials and
// its newest K/V row are complete, whichever workgroups produced them.
// The table's addresses and the number of walking workgroups (n_units, per KV head; those beyond only project) come first among the
// arguments: the build asks for the leading ones in registers when a workgroup starts, so that its unit's record is requested without
// waiting for the argument buffer (0.3 us for the slowest of 256 workgroups).
// F8: the pages hold E4M3 codes with per-head power-of-two scales; a block's codes are widened
// to bf16 in registers (exact), the K scale multiplies the block's scores and the V scale its
// weights on their way to bf16 (exact too: powers of two), the row sums stay unscaled.
// SH: decode over the shared partition - `units` are SUnit records: one piece of a page (or one
// instance's tail) and up to 16 / G instances whose newest tokens attend to it; the rows of the
// tile are (user, query head) pairs, the piece is streamed once for all of them, every user gets
// its own partial, and the workgroup arrives at every user's counter: the last arrival at an
// instance's counter folds that instance's partial slots.
// NT: the cache's rows are not left in the last-level cache.
// STEP: instances per projection task of a fused step (0: attention alone); negative: the same, their places looked up behind the sums.
template <int G, int NW, int MS, int PF, int STEP, bool F8, bool SH = false, bool NT = false>
__global__ __launch_bounds__((STEP != 0 ? 2 : 1) * NW * 64, (STEP != 0 || (MS == 1 && PF <= 2)) ? 2 : 1) void attn_mfma_kernel(
        const Unit* __restrict__ units, const InstanceInfo* __restrict__ insts, const Item* __restrict__ items, int n_units,
        KernelArgs a, StepArgs f) {
    constexpr int FR = STEP < 0 ? -STEP : STEP;
    constexpr int ROWS = 16 * MS;                       // (row, head) pairs per workgroup
    constexpr int NTH = (FR > 0 ? 2 : 1) * NW * 64;     // threads of the workgroup
    typedef uint16_t T;
    static_assert(!SH || (FR == 0 && MS == 1), "shared units: decode tiles only");
    __shared__ int sm_last, sm_lastv[SH ? kMaxSharedUsers : (FR > 0 ? kFusedMaxBatch : 1)];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    const int kvh = blockIdx.y, tile = blockIdx.z;
    const int m0 = tile * ROWS;

    const SUnit* const su = reinterpret_cast<const SUnit*>(units) + blockIdx.x;     // SH only
    // fused step: workgroups beyond the units of the cache have projection waves only
    const bool walks = FR == 0 || (int)blockIdx.x < n_units;
    const Unit unit = SH ? table_record(&su->u) : table_record(units + (FR > 0 ? min((int)blockIdx.x, n_units - 1) : (int)blockIdx.x));

    if (SH && su->n_users == 0) return;                 // (the even partition's last runs may be empty)

    // The other arguments are wanted here, together with the record: fetched where they are first used, each group of them
    // would be waited for by itself (3B shape, three short instances: 1428 -> 1385 us per pass of 128 steps and layers).
    asm volatile("" :: "s"(a.q), "s"(a.out), "s"(a.tail_k), "s"(a.tail_v), "s"(a.partials), "s"(a.counters), "s"(a.layer), "s"(a.Hq), "s"(a.Hkv),
                       "s"(a.max_tail), "s"(a.prefill), "s"(a.cstride), "s"(a.out_f32), "s"(a.scale_log2e));
    if (FR > 0) asm volatile("" :: "s"(f.hidden), "s"(f.w_k), "s"(f.w_v), "s"(f.rope), "s"(f.Hd), "s"(f.batch), "s"(f.workgroups));

    int n_m, q_row0, tail_len = 0, tail_visible;
    if (SH) {
        n_m = su->n_users * G;
        q_row0 = 0;
        if (unit.has_tail) tail_len = insts[unit.inst].tail_len;
        tail_visible = tail_len;
    } else if (a.prefill) {
        const InstanceInfo inst = insts[unit.inst];
        n_m = inst.q_len * G;
        if (m0 >= n_m) return;                          // whole workgroup leaves together
        q_row0 = inst.cu_q;
        const int r_last = (min(m0 + ROWS, n_m) - 1) / G;
        tail_visible = r_last + 1;                      // the most any row of this tile may see
    } else {
        n_m = G;
        q_row0 = unit.inst;
        if (unit.has_tail) tail_len = insts[unit.inst].tail_len - (FR > 0 ? 1 : 0);   // fused: the newest row is not in the cache yet
        tail_visible = tail_len;
    }

    f32x4 ot[MS][8];                                    // O^T: dims 16s + 4*g4 + i of row 16j + c16
    float mrow[MS], lrow[MS];
#pragma unroll
    for (int j = 0; j < MS; ++j) {
        mrow[j] = kNegBig; lrow[j] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) ot[j][s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // LDS: per-wave V strips during the walk, the waves' finished states afterwards, each over its own wave's strip.
    constexpr int V_BYTES = BLK * VSTR * 2, ACC_BYTES = ROWS * ACCS * 4;
    constexpr int WAVE_BYTES = V_BYTES > ACC_BYTES ? V_BYTES : ACC_BYTES, WS = WAVE_BYTES / 4;
    __shared__ __attribute__((aligned(16))) char smem[NW * WAVE_BYTES];
    __shared__ float sm_m[NW * ROWS], sm_l[NW * ROWS];

    // shared unit: its users with their slot ranges, for the publishing and folding at the end
    __shared__ int4 sm_users[SH ? kMaxSharedUsers : 1];
    if (SH && tid < su->n_users) {
        const int inst = su->users[tid].inst;
        sm_users[tid] = make_int4(inst, su->users[tid].slot, insts[inst].sslot0, insts[inst].n_sslots);
    }

    if (FR > 0 && (wave >= NW || !walks)) {
        if constexpr (FR > 0) {
            // the waves of the projection-only workgroups come first: they have nothing else to do
            const int extra = (f.workgroups - n_units) * 2 * NW;
            const int id = walks ? extra + (int)blockIdx.x * NW + (wave - NW) : ((int)blockIdx.x - n_units) * 2 * NW + wave;
            projection_tasks<FR, (STEP > 1)>(a, f, insts, kvh, id, extra + n_units * NW, lane);
        }
    } else {
    // Q in operand layout: lane (c16, g4) holds, for sub-tile j and chunk c of the head
    // dimension, the 8 dims dim0(c) .. +8 of row m0 + 16j + c16: 32c + 8*g4 for plain pages; with
    // compressed pages 16*g4 + 8*(c%2) + 64*(c/2), so that the two chunks of a pair are the 16
    // codes of one 16-byte load.  Padding rows repeat the last real row.
    auto dim0 = [&](int c) { return F8 ? 16 * g4 + 8 * (c & 1) + 64 * (c >> 1) : 32 * c + 8 * g4; };
    bf16x8 bq[MS][4];
    int vis[MS];                                        // tail rows this lane's row may see
    int row_user[MS];                                   // shared units: index of the row's user in the unit's list
#pragma unroll
    for (int j = 0; j < MS; ++j) {
        const int m = min(m0 + 16 * j + c16, n_m - 1);
        const int r = m / G, g = m % G;
        row_user[j] = r;
        int q_row = a.prefill ? q_row0 + r : q_row0;
        if (SH) {           // the record's user list comes through scalar loads; pick this lane's
#pragma unroll
            for (int k = 0; k < kMaxSharedUsers; ++k) {
                const int v = su->users[k].inst;
                q_row = (r == k) ? v : q_row;
            }
        }
        const T* qp = reinterpret_cast<const T*>(a.q) + ((size_t)q_row * a.Hq + (size_t)kvh * G + g) * D;
#pragma unroll
        for (int c = 0; c < 4; ++c) bq[j][c] = as_bf16x8(ldg16(qp + dim0(c)));
        vis[j] = (a.prefill && !SH) ? r + 1 : tail_len;
    }

    uint16_t* const vstrip = reinterpret_cast<uint16_t*>(smem + wave * WAVE_BYTES);

    // One block's loads in registers.  Plain rows: lane (c16, g4) holds, per 16-token half, the
    // 8 dims of each of the 4 chunks of its token row, and 8 V rows' worth of 8 dims.  Code rows
    // (one byte per element): 16 dims per load, so half as many loads carry the same tokens.
    struct PlainBuf { uint4 k[2][4], v[8]; };
    struct CodeBuf { uint4 k[2][2], v[4]; };

    // Rows past the block's end are clamped to its last row and masked in the softmax.
    auto issue_plain = [&](const BlockRef<T>& r, PlainBuf& b) {
        const T* const kp = r.k + (size_t)r.t0 * D;
        const T* const vp = r.v + (size_t)r.t0 * D;
        const int n = r.tok_end - r.t0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t row = min(16 * h + c16, n - 1) * (2 * D);
#pragma unroll
            for (int c = 0; c < 4; ++c) b.k[h][c] = dev::ld16_at<NT>(kp, row + 2 * dim0(c));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) b.v[u] = dev::ld16_at<NT>(vp, min(4 * u + g4, n - 1) * (2 * D) + 16 * c16);
    };
    // K: the two 16-byte pieces of the lane's token row that hold its dims (chunks 0-1, 2-3);
    // V: lane l takes 16 dims (l % 8) of token row 8u + l / 8.
    auto issue_codes = [&](const BlockRef<T>& r, CodeBuf& b) {
        const uint8_t* const kp = reinterpret_cast<const uint8_t*>(r.k) + (size_t)r.t0 * D;
        const uint8_t* const vp = reinterpret_cast<const uint8_t*>(r.v) + (size_t)r.t0 * D;
        const int n = r.tok_end - r.t0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t row = min(16 * h + c16, n - 1) * D + 16 * g4;
            b.k[h][0] = dev::ld16_at<NT>(kp, row);
            b.k[h][1] = dev::ld16_at<NT>(kp, row + 64);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) b.v[u] = dev::ld16_at<NT>(vp, min(8 * u + (lane >> 3), n - 1) * D + 16 * (lane & 7));
    };

    // Scores, online softmax and P V of one block whose K operands are in ak and whose V rows
    // are in this wave's strip.  sc_blk: score scale of the block; pv_scale: factor of its
    // weights on their way to bf16 (both carry a compressed page's power-of-two scales).
    auto attend = [&](const BlockRef<T>& r, const uint4 (*ak)[4], float sc_blk, float pv_scale) {
        bf16x8 pb[MS];
#pragma unroll
        for (int j = 0; j < MS; ++j) {
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ak[0][c]), bq[j][c], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ak[1][c]), bq[j][c], s1, 0, 0, 0);
            }
            // lane holds tokens t0 + 4*g4 + i (s0) and t0 + 16 + 4*g4 + i (s1) of its row
            // (shared units: a row whose user does not use this piece sees none of it)
            const int limit = (SH && !((r.umask >> row_user[j]) & 1)) ? 0 : (r.is_tail ? min(r.tok_end, vis[j]) : r.tok_end);
            const int tb = r.t0 + 4 * g4;
            float sv[8];
            bool ok[8];
            float mx = kNegBig;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ok[i] = tb + i < limit;
                ok[4 + i] = tb + 16 + i < limit;
                sv[i] = ok[i] ? s0[i] * sc_blk : kNegBig;
                sv[4 + i] = ok[4 + i] ? s1[i] * sc_blk : kNegBig;
                mx = fmaxf(mx, fmaxf(sv[i], sv[4 + i]));
            }
            mx = fmaxf(mx, lane_xor(mx, 16, lane));
            mx = fmaxf(mx, lane_xor(mx, 32, lane));
            const float mn = fmaxf(mrow[j], mx);
            const float alpha = fast_exp2(mrow[j] - mn);
            mrow[j] = mn;
            float psum = 0.f;
            float p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                p[i] = ok[i] ? fast_exp2(sv[i] - mn) : 0.f;
                psum += p[i];
            }
            lrow[j] = lrow[j] * alpha + psum;
#pragma unroll
            for (int i = 0; i < 8; ++i) pb[j][i] = (__bf16)(p[i] * pv_scale);
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {   // wave-uniform: some row's maximum moved
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    ot[j][s][0] *= alpha; ot[j][s][1] *= alpha; ot[j][s][2] *= alpha; ot[j][s][3] *= alpha;
                }
            }
        }

        __builtin_amdgcn_wave_barrier();                // strip writes stay ahead of the reads below
        // lane (c16, g4) names 4 dims (4*(c16%4) ..) of token 4*g4 + c16/4 (+16 for the second
        // half) and receives dim 16s + c16 of tokens 4*g4 .. 4*g4+3: the k order of P above
        const uint16_t* vp = vstrip + (4 * g4 + (c16 >> 2)) * VSTR + 4 * (c16 & 3);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const s16x4 lo = lds_read_tr(vp + 16 * s);
            const s16x4 hi = lds_read_tr(vp + 16 * VSTR + 16 * s);
            const bf16x8 av = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int j = 0; j < MS; ++j)
                ot[j][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb[j], ot[j][s], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();                // and the next block's writes behind them
    };

    auto consume_plain = [&](const BlockRef<T>& r, const PlainBuf& b) {
        // V rows into this wave's strip, as loaded
#pragma unroll
        for (int u = 0; u < 8; ++u)
            *reinterpret_cast<uint4*>(vstrip + (4 * u + g4) * VSTR + 8 * c16) = b.v[u];
        attend(r, b.k, a.scale_log2e, 1.0f);
    };
    auto consume_codes = [&](const BlockRef<T>& r, const CodeBuf& b) {
        uint4 ak[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            ak[h][0] = e4m3x8_to_bf16x8(make_uint2(b.k[h][0].x, b.k[h][0].y));
            ak[h][1] = e4m3x8_to_bf16x8(make_uint2(b.k[h][0].z, b.k[h][0].w));
            ak[h][2] = e4m3x8_to_bf16x8(make_uint2(b.k[h][1].x, b.k[h][1].y));
            ak[h][3] = e4m3x8_to_bf16x8(make_uint2(b.k[h][1].z, b.k[h][1].w));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint16_t* dst = vstrip + (8 * u + (lane >> 3)) * VSTR + 16 * (lane & 7);
            *reinterpret_cast<uint4*>(dst) = e4m3x8_to_bf16x8(make_uint2(b.v[u].x, b.v[u].y));
            *reinterpret_cast<uint4*>(dst + 8) = e4m3x8_to_bf16x8(make_uint2(b.v[u].z, b.v[u].w));
        }
        attend(r, ak, a.scale_log2e * r.sk, r.sv);
    };

    // PF blocks of loads stay in flight: block i + PF is issued right after block i is consumed.
    // The loads are issued without a branch (past the end of the wave's share they all fall on
    // one row) and the loop has one exit: only then can the compiler count the loads in flight
    // exactly, instead of waiting for all of them before each block.
    auto stream = [&](auto& walk, auto buf_tag, auto issue, auto consume) {
        decltype(buf_tag) b[PF];
        BlockRef<T> rb[PF];
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            rb[i] = walk.next_safe();
            issue(rb[i], b[i]);
        }
        do {
#pragma unroll
            for (int i = 0; i < PF; ++i) {
                if (rb[i].valid) consume(rb[i], b[i]);
                rb[i] = walk.next_safe();
                issue(rb[i], b[i]);
            }
        } while (rb[0].valid);
    };
    if constexpr (!F8) {
        Walker<T, D, NW, BLK, 8> walk(a, unit, items, kvh, tail_visible, wave);
        stream(walk, PlainBuf{}, issue_plain, consume_plain);
    } else {
        // Compressed pages first, then the (plain) tail, each in a loop of its own: one loop
        // over both kinds would put the two load patterns under a branch.
        {
            Walker<T, D, NW, BLK, 8, true> walk(a, unit, items, kvh, 0, wave);
            stream(walk, CodeBuf{}, issue_codes, consume_codes);
        }
        if (unit.has_tail && tail_visible > 0) {
            Unit tu = unit;                             // the unit's last item, alone
            tu.item0 = unit.item0 + unit.n_items - 1; tu.n_items = 1; tu.page_tokens = 0;
            tu.first.base = 0; tu.first.page_tokens = a.max_tail; tu.first.tok0 = 0; tu.first.ntok = a.max_tail;
            tu.first.fmt = 0; tu.first.scales16 = 0;
            if (SH) tu.first.umask = items[tu.item0].umask;     // the users that see it (its owner)
            Walker<T, D, NW, BLK, 8> walk(a, tu, items, kvh, tail_visible, wave);
            stream(walk, PlainBuf{}, issue_plain, consume_plain);
        }
    }

#pragma unroll
    for (int j = 0; j < MS; ++j) {
        lrow[j] += lane_xor(lrow[j], 16, lane);
        lrow[j] += lane_xor(lrow[j], 32, lane);
    }
    }   // attention waves

    // ---- per-wave states to LDS (the wave's strip is dead now), then the common merge ----
    float* const sm_acc = reinterpret_cast<float*>(smem);
    if (wave < NW && walks) {
#pragma unroll
        for (int j = 0; j < MS; ++j) {
            float* dst = sm_acc + wave * WS + (16 * j + c16) * ACCS + 4 * g4;
#pragma unroll
            for (int s = 0; s < 8; ++s)
                *reinterpret_cast<float4*>(dst + 16 * s) = make_float4(ot[j][s][0], ot[j][s][1], ot[j][s][2], ot[j][s][3]);
            if (g4 == 0) { sm_m[wave * ROWS + 16 * j + c16] = mrow[j]; sm_l[wave * ROWS + 16 * j + c16] = lrow[j]; }
        }
    }
    const int prefill = a.prefill;
    auto map = [&](int i) {
        RowMap rm;
        const int m = m0 + i;
        const int r = m / G, g = m % G;
        rm.slot_row = (prefill && !SH) ? r : 0;
        rm.head = kvh * G + g;
        rm.q_row = prefill ? q_row0 + r : q_row0;
        if (SH) { const int4 us = sm_users[r]; rm.q_row = us.x; rm.unit_slot = __builtin_amdgcn_readfirstlane(us.y); }      // (a wave has one row)
        return rm;
    };
    if constexpr (SH) {
        publish_rows<NW, NW, ROWS, WS, 2>(a, sm_acc, sm_m, sm_l, n_m, map, wave, lane);
        // arrival at the counter of every user of this unit
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        const int n_users = n_m / G;
        if (tid < n_users) {
            const int4 us = sm_users[tid];
            const int prev = __hip_atomic_fetch_add(&a.counters[counter_index(a, us.x, kvh, 0)], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool last = prev == us.w - 1;
            if (last)                                   // ready for the next launch
                __hip_atomic_store(&a.counters[counter_index(a, us.x, kvh, 0)], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t who = __builtin_amdgcn_ballot_w64(last);       // (n_users <= 16: all in the first wave)
            if (last) sm_lastv[__popcll(who & ((1ull << tid) - 1))] = tid;
            const bool many = __builtin_amdgcn_ballot_w64(last && us.w > 8) != 0;
            if (tid == 0) sm_last = 2 * __popcll(who) + many;
        }
        __syncthreads();
        // Which instances a workgroup is the last of is a matter of timing, the order of an instance's sums is not: 16 partials a pass where
        // one of them has more than 8 (up to 8, passes of 8 and of 16 do the same sums).
        const int n_live = __builtin_amdgcn_readfirstlane(sm_last) >> 1;
        const bool many = __builtin_amdgcn_readfirstlane(sm_last) & 1;
        if (n_live * G <= NW) merge_shared<G, NW, 1, 16>(a, sm_users, sm_lastv, n_live, kvh, wave, lane);
        else if (many)        merge_shared<G, NW, 2, 16>(a, sm_users, sm_lastv, n_live, kvh, wave, lane);
        else                  merge_shared<G, NW, 4, 8>(a, sm_users, sm_lastv, n_live, kvh, wave, lane);
    } else if constexpr (FR == 0) {
        if constexpr (MS > 1) {                         // (prefill tiles)
            finish_unit<T, D, NW, NW, ROWS, ACCS, WS>(a, unit, kvh, tile, sm_acc, sm_m, sm_l, &sm_last, min(ROWS, n_m - m0), map);
        } else {
            const int cidx = counter_index(a, unit.inst, kvh, 0);
            publish_rows<NW, NW, ROWS, WS, (G + NW - 1) / NW>(a, sm_acc, sm_m, sm_l, G, map, wave, lane);
            if (!arrive(a, cidx, unit.n_units_inst, &sm_last)) return;
            if (unit.n_units_inst <= 8)       merge_decode<G, NW, 8>(a, unit, kvh, wave, lane);
            else if (unit.n_units_inst <= 16) merge_decode<G, NW, 16>(a, unit, kvh, wave, lane);
            else                              merge_decode<G, NW, (G + NW - 1) / NW <= 2 ? 32 : 16>(a, unit, kvh, wave, lane);   // (four rows x 32 units would not fit the registers)
            reset_counter(a, cidx);
        }
    } else {
        if (walks) publish_rows<NTH / 64, NW, ROWS, WS, (G + NTH / 64 - 1) / (NTH / 64)>(a, sm_acc, sm_m, sm_l, G, map, wave, lane);      // (uniform)
        // arrival at every instance's counter of this KV head, then the fold, in
        // one round trip where it fits: one row per wave, or two where the batch has more rows than the
        // workgroup has waves; units requested per row: the smallest of 8, 16, 32 that covers the partition
        // (an even cut: the batch's instances have at most n_units - batch + 1 units each)
        constexpr int NWV = NTH / 64;
        auto arrive_and_fold = [&](auto rb, auto fold) {
            const StepRows<G, NWV, decltype(rb)::value> rows(a, insts, f.batch, kvh, wave, lane);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid < f.batch) {
                const int prev = __hip_atomic_fetch_add(&a.counters[counter_index(a, tid, kvh, 0)], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sm_lastv[tid] = (prev == f.workgroups - 1);
            }
            __syncthreads();
            fold(rows);
        };
        if (FR == 1 || f.batch * G <= NWV) {            // (FR = 1: one instance)
            arrive_and_fold(std::integral_constant<int, 1>{}, [&](const auto& rows) {
                if (n_units <= 8)       merge_decode_step<G, NWV, 1, 8>(a, rows, sm_lastv, lane);
                else if (n_units <= 16) merge_decode_step<G, NWV, 1, 16>(a, rows, sm_lastv, lane);
                else                      merge_decode_step<G, NWV, 1, 32>(a, rows, sm_lastv, lane);
            });
        } else {
            arrive_and_fold(std::integral_constant<int, 2>{}, [&](const auto& rows) {
                if (n_units <= 8 * f.batch) merge_decode_step<G, NWV, 2, 8>(a, rows, sm_lastv, lane);
                else                          merge_decode_step<G, NWV, 2, 16>(a, rows, sm_lastv, lane);
            });
        }
        if (tid < f.batch && sm_lastv[tid])             // ready for the next launch
            __hip_atomic_store(&a.counters[counter_index(a, tid, kvh, 0)], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int G, int NW, int MS, int PF, bool F8 = false, bool NT = false>
hipError_t launch_v(const AttnArgs& a, int tiles, hipStream_t s) {
    const KernelArgs k = make_kernel_args(a);
    dim3 grid(a.n_units, a.Hkv, tiles), block(NW * 64);
    hipLaunchKernelGGL((attn_mfma_kernel<G, NW, MS, PF, 0, F8, false, NT>), grid, block, 0, s,
                       reinterpret_cast<const Unit*>(a.table + a.off_units), reinterpret_cast<const InstanceInfo*>(a.table + a.off_inst),
                       reinterpret_cast<const Item*>(a.table + a.off_items), a.n_units, k, StepArgs{});
    return hipGetLastError();
}

template <int G, int NW, int FR>
hipError_t launch_step_v(const AttnArgs& a, const MaterializeArgs& m, hipStream_t s) {
    const KernelArgs k = make_kernel_args(a);
    StepArgs f;
    f.hidden = m.hidden; f.w_k = m.w_k; f.w_v = m.w_v; f.rope = m.rope;
    f.Hd = m.Hd; f.batch = a.batch;
    // A short cache is cut into few units, and their projection waves alone would each have several of
    // a KV head's 128 rotary pairs (of K and of V) to do one after the other: workgroups that only project
    // are added until every pair has a wave or every compute unit a workgroup (3B shape, three instances
    // of 300 to 800 tokens, 14 units: 20.7 -> 11 us per layer).
    const int tasks = (a.batch + FR - 1) / FR * D;
    const int lacking = tasks - a.n_units * NW;
    const int extra = std::max(0, std::min((lacking + 2 * NW - 1) / (2 * NW), 256 / a.Hkv - a.n_units));
    f.workgroups = a.n_units + extra;
    dim3 grid(f.workgroups, a.Hkv, 1), block(2 * NW * 64);
    const bool f8 = a.kv_fmt == MATKV_PAGE_E4M3;
    // Several instances' places are looked up ahead over plain pages (298 seeded steps of two to four users take 1/1.025 of the time in the mean), and over compressed
    // ones where a unit with a tail has been spared tokens.  302 such steps, against neither: both throughout 1/1.011 of the time and up to 1.05 (3B, four users of 3 x 158 tokens
    // 10.4 -> 11.0 us a layer), spared with the places behind 1/1.004 and up to 1.10, ahead and not spared 1.002 and up to 1.06, both where spared and neither elsewhere 1/1.012
    // and up to 1.045 (two 8B users of 5000 906 -> 867 a pass).
    auto kern = a.past_llc ? (f8 ? attn_mfma_kernel<G, NW, 1, 2, FR, true, false, true> : attn_mfma_kernel<G, NW, 1, 2, FR, false, false, true>)
                           : (f8 ? attn_mfma_kernel<G, NW, 1, 2, FR, true> : attn_mfma_kernel<G, NW, 1, 2, FR, false>);
    if constexpr (FR > 1) {
        if (f8 && !a.tail_spared) kern = a.past_llc ? attn_mfma_kernel<G, NW, 1, 2, -FR, true, false, true> : attn_mfma_kernel<G, NW, 1, 2, -FR, true>;
    }
    hipLaunchKernelGGL(kern, grid, block, 0, s,
                       reinterpret_cast<const Unit*>(a.table + a.off_units), reinterpret_cast<const InstanceInfo*>(a.table + a.off_inst),
                       reinterpret_cast<const Item*>(a.table + a.off_items), a.n_units, k, f);
    return hipGetLastError();
}

template <int G>
hipError_t launch_step_g(const AttnArgs& a, const MaterializeArgs& m, hipStream_t s) {
    if constexpr (G <= 4) return a.batch == 1 ? launch_step_v<G, 4, 1>(a, m, s) : launch_step_v<G, 4, 4>(a, m, s);
    return hipErrorInvalidValue;
}

// past_llc: the cache's rows are not left in the last-level cache (rows_pass_llc, where the table is assembled, says when).  us per pass of
// 8 steps, left there -> not: decode of sixteen 8B users over 5000 tokens 1925 -> 1762, of four 70B users over 20 000 2250 -> 2073, of
// one 8B user over 10 000 1052 -> 990.  The weights stay on the ordinary path: what is left of the cache then holds them.
template <int G>
hipError_t launch_g(const AttnArgs& a, hipStream_t s) {
    const bool f8 = a.kv_fmt == MATKV_PAGE_E4M3;        // compressed pages: the default shapes only
    if (a.prefill) {
        const int tiles = (a.rows * G + 31) / 32;
        return f8 ? launch_v<G, 4, 2, 2, true>(a, tiles, s) : launch_v<G, 4, 2, 2>(a, tiles, s);
    }
    if (a.shared) {
        const KernelArgs k = make_kernel_args(a);
        auto kern = a.past_llc ? (f8 ? attn_mfma_kernel<G, 4, 1, 2, 0, true, true, true> : attn_mfma_kernel<G, 4, 1, 2, 0, false, true, true>)
                               : (f8 ? attn_mfma_kernel<G, 4, 1, 2, 0, true, true> : attn_mfma_kernel<G, 4, 1, 2, 0, false, true>);
        hipLaunchKernelGGL(kern, dim3(a.n_units, a.Hkv, 1), dim3(4 * 64), 0, s,
                           reinterpret_cast<const Unit*>(a.table + a.off_units), reinterpret_cast<const InstanceInfo*>(a.table + a.off_inst),
                           reinterpret_cast<const Item*>(a.table + a.off_items), a.n_units, k, StepArgs{});
        return hipGetLastError();
    }
    if (f8) return a.past_llc ? launch_v<G, 4, 1, 2, true, true>(a, 1, s) : launch_v<G, 4, 1, 2, true>(a, 1, s);
    // decode: variant 9000 + 10 * (blocks in flight) + waves
    switch (a.variant % 100) {
        case 24: return launch_v<G, 4, 1, 2>(a, 1, s);
        case 34: return launch_v<G, 4, 1, 3>(a, 1, s);
        case 28: return launch_v<G, 8, 1, 2>(a, 1, s);
        case 22: return launch_v<G, 2, 1, 2>(a, 1, s);
        default: break;
    }
    // measured: four waves are ahead for every group size (config 4, G = 8: 62.7 us against
    // 65.1 us with eight)
    return a.past_llc ? launch_v<G, 4, 1, 2, false, true>(a, 1, s) : launch_v<G, 4, 1, 2>(a, 1, s);
}

}  // namespace

bool attn_mfma_supported(const AttnArgs& a, int dtype) {
    const int g = a.Hq / a.Hkv;
    return dtype == MATKV_BF16 && a.D == 128 && group_size_built(g);
}

hipError_t launch_attn_mfma(const AttnArgs& a, int dtype, hipStream_t s) {
    if (a.n_units <= 0) return hipSuccess;
    if (!attn_mfma_supported(a, dtype)) return hipErrorInvalidValue;
    switch (a.Hq / a.Hkv) {
        case 1: return launch_g<1>(a, s);
        case 2: return launch_g<2>(a, s);
        case 3: return launch_g<3>(a, s);
        case 4: return launch_g<4>(a, s);
        case 8: return launch_g<8>(a, s);
    }
    return hipErrorInvalidValue;
}


// Fused decode step: K/V projection of every instance's newest token and the decode attention
// in one launch (default kernel shape only).
bool decode_step_supported(const AttnArgs& a, const MaterializeArgs& m, int dtype) {
    // Measured: the single launch wins while every projection wave has one task (up to four
    // instances) at the 8B shape; at group size 8 with hidden 8192 (config 4) it is 3 % behind
    // the two launches (it halves the attention waves per compute unit), so it stops at group
    // size 4.  Projection workgroups of their own beside the attention workgroups (for larger
    // batches) lose outright: the decode kernel wants exactly one attention workgroup per
    // compute unit - a second resident workgroup of any kind on a compute unit stretches the
    // launch by a third (batch 16: 57 us with 256 workgroups, 83 us with 264).
    return !a.prefill && !a.shared && a.variant == 0 && fused_step_shape(dtype, a.D, a.Hq / a.Hkv, m.Hd, a.batch);
}

hipError_t launch_decode_step(const AttnArgs& a, const MaterializeArgs& m, int dtype, hipStream_t s) {
    if (a.n_units <= 0 || !decode_step_supported(a, m, dtype)) return hipErrorInvalidValue;
    switch (a.Hq / a.Hkv) {
        case 1: return launch_step_g<1>(a, m, s);
        case 2: return launch_step_g<2>(a, m, s);
        case 3: return launch_step_g<3>(a, m, s);
        case 4: return launch_step_g<4>(a, m, s);
        case 8: return launch_step_g<8>(a, m, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace matkv
