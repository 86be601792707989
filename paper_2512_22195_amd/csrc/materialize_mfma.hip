// K/V materialization of one layer as a matrix-core GEMM with the rotary embedding in the
// epilogue (paper Section III-B steps 2-3, cut to the K/V projection):
//   [T, Hd] x [2*Hkv*D, Hd]^T  ->  K = RoPE(X Wk^T, pos), V = X Wv^T,   bf16, D = 128.
// Both operands are contiguous along the contraction (hidden) axis, which is what the
// matrix-core operand layout wants: a lane's 8 consecutive bf16 of one row.
//
// Three forms by row count: the tiled GEMM (below), a skinny form for too few rows to fill the chip with tiles (a
// question) and one for a handful (a decode step of a batch), whose eight waves split the hidden axis.  In all of
// them the two features of a rotary pair sit in the same lane, so the rotation is lane-local on the fp32 accumulators,
// and values are rounded to bf16 once, on store.
#include <type_traits>

#include "device_util.h"

namespace matkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 128, BK = 64;             // BK: hidden columns per step of the tiled GEMM

using dev::ldg16;
using dev::f32_to_bf16_rne;

struct RowDest {
    float pos;          // rotary position (exact in fp32: below 2^24)
    size_t elem_off;    // element offset of [head 0][row][0] in the destination
    bool valid;
};

__device__ __forceinline__ RowDest resolve_row(const MaterializeArgs& a, int r) {
    RowDest d;
    d.valid = false; d.pos = 0.f; d.elem_off = 0;
    if (a.table == nullptr) {
        if (r < a.n_tokens) { d.valid = true; d.pos = (float)(a.pos0 + r); d.elem_off = (size_t)r * D; }
        return d;
    }
    const InstanceInfo* insts = reinterpret_cast<const InstanceInfo*>(a.table + a.off_inst);
    int b = -1, j = 0;
    int64_t base = 0;
    if (a.rows_per_instance > 0) {
        if (r < a.batch * a.rows_per_instance) {
            b = r / a.rows_per_instance;
            j = insts[b].tail_len - a.rows_per_instance + (r % a.rows_per_instance);
            base = insts[b].pos_base;
        }
    } else {
        // every lane walks all instances through the constant address space (no kernel of the launch
        // writes the table): scalar loads, several of them in flight, which do not wait for copies on their way
        // (as a walk of dependent loads ahead of the first copy it cost 1.3 us of a launch's 38 at 16 instances)
        typedef const __attribute__((address_space(4))) InstanceInfo* cptr;
        const cptr t = (cptr)(uintptr_t)insts;
#pragma unroll 4
        for (int i = 0; i < a.batch; ++i) {
            const int c0 = t[i].cu_q, n = t[i].q_len;
            const int64_t p = t[i].pos_base;
            if (r >= c0 && r < c0 + n) { b = i; j = r - c0; base = p; }
        }
    }
    if (b < 0 || j < 0 || j >= a.token_stride) return d;
    d.valid = true;
    d.pos = (float)(base + j);
    d.elem_off = ((size_t)b * a.Hkv * a.token_stride + (size_t)j) * D;
    return d;
}

// cos / sin of pos * theta_j with the angle kept in turns: hi/lo split product, whole turns
// dropped exactly, then the hardware sine / cosine (which take turns).
__device__ __forceinline__ void rope_cs(float turns_hi, float turns_lo, float p, float& c, float& s) {
    // no contraction here: were p * turns_hi - rint(t) fused into one multiply-add, the product
    // would enter exactly and the rounding error of t, added back below, would count twice
    // (half an ulp of t: 1e-4 turns at position 20 000)
#pragma clang fp contract(off)
    const float t = p * turns_hi;
    const float err = fmaf(p, turns_hi, -t);
    float fr = t - rintf(t);
    fr += fmaf(p, turns_lo, err);
    c = __builtin_amdgcn_cosf(fr);
    s = __builtin_amdgcn_sinf(fr);
}
__device__ __forceinline__ void rope_cs(const RopeEntry& e, float p, float& c, float& s) { rope_cs(e.turns_hi, e.turns_lo, p, c, s); }

// ---- tiled GEMM ----------------------------------------------------------------------------------
// A workgroup of eight waves owns 32 MI token rows x one head of K or of V (128 features: both halves
// of every rotary pair), over the whole hidden axis or (SK = 2) over half of it.  What bounds it is
// the path from L2 into a compute unit: a read of L2-resident memory peaks at 110 GB/s per compute
// unit with the chip full (46 bytes a cycle, whether the bytes go to registers or to LDS), and a step
// of 64 hidden columns brings 16 KB of weights whatever the tile's height.  So a launch takes as long
// as one workgroup's operands take to arrive, and the choices follow from that:
//  - operands go from global memory straight into LDS (dma16): no registers, no LDS write
//    instructions, as many steps in flight as LDS holds (six of 24 KB at MI = 2, three of 48 KB at
//    MI = 8), one barrier per step.  The form this replaced moved operands through registers with
//    four of its eight waves and reached 17 bytes a cycle.
//  - LDS rows are unpadded 128 bytes (the copy writes 1 KB runs); the eight 16-byte pieces of row r
//    are permuted by (r >> 1) & 7 instead - the copy picks its global addresses accordingly - which
//    spreads an operand read of sixteen rows over all banks.
//  - half a step is multiplied while the operands of the next half are on their way from LDS and copies are
//    requested, instruction by instruction: all waves' copies at once hold up their matrix instructions.
//  - behind the loop every wave is on its own: results leave registers as 8 or 16 bytes of a row (its four or two
//    waves along the features fill 256 bytes), rotated with entries fetched at the start.
// Two workgroups that share a tile (SK = 2) each hold half of every sum, wave by wave.  Up to 96 rows each wave leaves its fp32 partial in the
// workspace (agent-scope stores) and arrives at a counter of its own, and of a pair the second to arrive adds the other's and finishes; from 128 rows on (and hidden above 512) one of
// the pair leaves its half and the other waits for it (below).  Either way the two workgroups share that work too.
// Measured, us per launch with every layer's weights from HBM, 8 KV heads, when results went through LDS and whole workgroups arrived -> wave by wave, before
// skewed starts (`first`) and draws:
//   hidden 4096:  1000 rows 26.3 -> 24.0, 1206 rows 30.9 -> 29.2, 3501 rows 66.9 -> 60.6
//   hidden 8192:  512 rows 36.3 -> 34.5, 1000 rows 49.7 -> 46.5, 1206 rows 62 -> 50, 2000 rows 73 -> 67
// At 1000 rows of hidden 4096 that launch took 37 800 cycles: 3800 for its first operands, 740 for each of 32 steps (44
// bytes a cycle), then 1900 until its partials had left, 2700 to arrive, 3600 to fetch the other's and 1300 for the results (6500,
// 3500 and 7400 for the last three before).  From the last-level cache 512 rows of hidden 8192 would take 24.7 us.
// Tried and left out: an extra wave that touches the weight rows
// some steps ahead (-12 % at 512 rows of hidden 8192, +20 % at 64 rows, nothing at 1000), workgroups that share an operand touching it
// some steps ahead in turn (-10 % there, +8 to 13 % at 1000 rows and more).
// (The operands' addresses and sizes come first among the arguments of these kernels: they arrive in registers, and the first operands are
// asked for without waiting for the argument buffer.)
template <int MI> struct TileShape {
    static constexpr int BM = 32 * MI;                              // token rows of a workgroup
    static constexpr int ROWS = BM + D;                             // LDS rows of a step: tokens, then weight rows
    static constexpr int STEP_BYTES = ROWS * BK * 2;
    static constexpr int NBUF = 158 * 1024 / STEP_BYTES;            // steps that fit in LDS
};

// WN: waves along the features; the other 8 / WN split the rows.  Few waves along the features read
// fewer LDS bytes per product from MI = 6 on, as many at MI = 4, and store 16 bytes of a row instead of 8.
template <int MI, int WN, int SK, bool DRAWN>
__global__ __launch_bounds__(512) void materialize_tile_kernel(
        const void* __restrict__ hidden, const void* __restrict__ w_k, const void* __restrict__ w_v, int Hd, int Hkv, int total_rows, int row_tiles, MaterializeArgs a) {
    typedef TileShape<MI> S;
    constexpr int WM = 8 / WN, XB = 2 * MI / WM, PB = 4 / WN;       // waves along the rows; row blocks and pair blocks of a wave
    constexpr int BM = S::BM, NBUF = S::NBUF;
    __shared__ __attribute__((aligned(16))) char smem[NBUF * S::STEP_BYTES];
    __shared__ RowDest sm_dest[BM];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    // Workgroup -> (half of the hidden axis, column tile, row tile).  Workgroups go to the eight XCDs in
    // turn; an XCD's L2 should see few distinct operands: with SK = 2 an XCD holds one half of the hidden
    // axis and every fourth column tile, with SK = 1 every fourth column tile and every second row tile.
    const int nct = 2 * Hkv;
    int part = 0, ct, rt;
    if (SK == 2) {
        part = blockIdx.x & 1;
        ct = (blockIdx.x >> 1) % nct; rt = (blockIdx.x >> 1) / nct;
    } else if (nct % 4 == 0) {                                      // (the grid has an even number of row tiles)
        const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
        ct = (x & 3) + 4 * (q % (nct / 4)); rt = 2 * (q / (nct / 4)) + (x >> 2);
        if (rt >= row_tiles) return;
    } else {
        ct = blockIdx.x % nct; rt = blockIdx.x / nct;
    }
    const int kv = ct >= Hkv, head = ct - kv * Hkv;
    const int row0 = rt * BM;
    const int nk = Hd / (BK * SK);
    // The step of the hidden axis at which this workgroup starts; it goes round from there.  A compute unit has 64 KB on their way at the
    // most, which come at 50 GB/s from HBM and at 108 out of an L2, and workgroups of an XCD that share weight rows and ask
    // for them at the same step all wait for HBM.  A few steps apart, one of them does and the others find them in the L2 (further
    // apart they have left it: 256 rows of hidden 8192 27.6 -> 25.6 with 4 steps, 33.5 with 6).  The other XCDs start at other quarters, so that not all ask the
    // same channels.  us per launch, all at step 0 -> this (weights from HBM, 8 KV heads): hidden 3072 150 rows 13.5 -> 11.3, 3000 38.5 -> 35.6;
    // 4096 150 15.7 -> 14.2, 512 19.7 -> 17.6, 1000 25.4 -> 23.8, 3501 56.0 -> 51.2; 8192 512 33.8 -> 30.4, 1000 43.6 -> 40.6, 3501 105 -> 97.
    // Steps from one row tile to the next: 1, 2, 3 and 4 measured, 4096 300 rows (tiles of 64) 17.4, 16.9, 16.7, 16.3, 512 18.3, 18.4, 18.1, 18.7,
    // 1000 (128) 23.8, 24.5, 25.1, 25.7; 8192 1000 42.2, 40.4, 40.7, 41.6.
    // Where the few layers of a small program stay in the last-level cache the wait is shorter and 4 a little too many: chunk passes of the 3B shape, 224
    // tokens, all at step 0 / 1 / 2 / 4: four layers (50 MB) 79.3 / 78.6 / 79.9 / 80.7, eight (three such programs in turn) 183 / 177 / 174 / 170.
    // Distances are counted in the row tiles that share weight rows on an XCD: all of them where the column tiles are a multiple of four, else every second (SK = 1: every
    // second, every fourth).  Counted in all of them an odd number of KV heads lay 4 to 8 steps apart: hidden 8192, 3 KV heads, all at step 0 / counted in all / this, 512
    // rows 22.4 / 32.6 / 19.8, 1300 27.7 / 47.5 / 26.2, 4000 51.5 / 71.7 / 50.0; 5, 300 22.8 / 32.6 / 21.6, 724 27.9 / 41.8 / 26.7; 7, 224 23.5 / 30.3 / 23.1, 1050 37.1 / 40.9 / 38.1 (the
    // worst); hidden 4096, 5, 724 16.9 / 19.1 / 16.1.  Quarters by column tile instead of by XCD are the same for multiples of four and else 2 to 3 % behind in the mean.
    const int xcd = blockIdx.x & 7;
    const int neighbour = SK == 2 ? (nct % 4 == 0 ? rt : rt >> 1) : (nct % 4 == 0 ? rt >> 1 : rt >> 2);
    const int first = (SK == 2 ? neighbour * (MI == 1 ? 4 : MI == 2 ? 3 : nk >= 40 ? 2 : 1) + (xcd >> 1) * (nk / 4)
                               : neighbour + (xcd & 3) * nk / 4) % nk;

    // LDS row r of the weights -> feature.  Sixteen rows are one operand of a matrix instruction, whose results
    // land in lanes by fours of these rows: the order makes a lane's results of its PB low (and of its PB high) operands features in a row.
    auto feature = [](int r) {
        const int b = (r & 63) >> 4, c = r & 15;
        return (r & 64) + 16 * PB * (b / PB) + 4 * PB * (c >> 2) + 4 * (b % PB) + (c & 3);
    };
    // Copies of a step: 8 rows x 128 bytes per instruction; token rows are instructions 0 .. 4 MI - 1,
    // wave w takes w, w + 8, ...; of the 16 weight instructions every wave takes two.  LDS row r holds
    // its eight 16-byte pieces permuted: piece g sits at place g ^ ((r >> 1) & 7).
    constexpr int XI = 4 * MI, XW = (XI + 7) / 8;
    const int n_x = (XI - wave + 7) / 8;                            // token copies of this wave per step (XW or XW - 1)
    const int lrow = lane >> 3, place = lane & 7;
    const size_t row_bytes = (size_t)Hd * 2;
    const char* X = reinterpret_cast<const char*>(hidden) + (size_t)row0 * row_bytes + (size_t)part * nk * (BK * 2);
    const char* W = reinterpret_cast<const char*>(kv == 0 ? w_k : w_v) + (size_t)head * D * row_bytes + (size_t)part * nk * (BK * 2);
    uint32_t xoff[XW], woff[2];
#pragma unroll
    for (int i = 0; i < XW; ++i) {
        const int r = (wave + 8 * i) * 8 + lrow;
        xoff[i] = (uint32_t)(min(r, total_rows - 1 - row0) * row_bytes) + 16 * (place ^ ((r >> 1) & 7));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (wave + 8 * i) * 8 + lrow;
        woff[i] = (uint32_t)(feature(r) * row_bytes) + 16 * (place ^ ((r >> 1) & 7));
    }
    const uint32_t lds0 = dev::lds_address(smem);
    constexpr int NC = 2 + XW;                                      // copies of a wave per step
    auto copy_one = [&](int ks, int buf, int i) {
        const uint32_t base = lds0 + buf * S::STEP_BYTES + wave * 1024;
        const int at = ks + first;
        const size_t k = (size_t)(at >= nk ? at - nk : at) * (BK * 2);
        if (i < 2)                                    dev::dma16(W + k, woff[i], base + BM * BK * 2 + i * 8192);
        else if (XI % 8 == 0 || i - 2 < n_x)          dev::dma16(X + k, xoff[i - 2], base + (i - 2) * 8192);
    };
    auto copy_step = [&](int ks, int buf) {
#pragma unroll
        for (int i = 0; i < NC; ++i) copy_one(ks, buf, i);
    };

    const int wm = wave / WN, wn = wave % WN;
    f32x4 acc[XB][2 * PB];                                          // [row block][low pair blocks, then their partners]
#pragma unroll
    for (int mi = 0; mi < XB; ++mi)
#pragma unroll
        for (int p = 0; p < 2 * PB; ++p) acc[mi][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags { bf16x8 b[2 * PB], x[XB]; };                      // operands of half a step: 32 hidden columns
    const int sw = (c16 >> 1) & 7;                                  // (the rows a lane reads differ by multiples of 16)
    const char* const At = smem + (16 * XB * wm + c16) * 128;
    const char* const Bt = smem + (BM + 16 * PB * wn + c16) * 128;
    constexpr int NF = 2 * PB + XB, NM = XB * 2 * PB;               // operands and matrix instructions of half a step
    auto read_one = [&](Frags& f, int buf, int k2, int i) {
        const int off = buf * S::STEP_BYTES + 16 * ((4 * k2 + g4) ^ sw);
        if (i < 2 * PB) f.b[i] = *reinterpret_cast<const bf16x8*>(Bt + (i < PB ? i * 2048 : 64 * 128 + (i - PB) * 2048) + off);
        else            f.x[i - 2 * PB] = *reinterpret_cast<const bf16x8*>(At + (i - 2 * PB) * 2048 + off);
    };
    auto read = [&](Frags& f, int buf, int k2) {
#pragma unroll
        for (int i = 0; i < NF; ++i) read_one(f, buf, k2, i);
    };
    // (keeps the instructions of a half step in the order written)
    auto pin = [](auto& v) { asm volatile("" : "+v"(v)); };
    // Half a step: f multiplied, the operands g of the next half read (block k2 of buffer rbuf) and copies c0 .. c1 of step ks into buffer
    // cbuf requested, all in turn: copies of all waves at once would hold up their matrix instructions for as long as
    // the address path takes them, 16 cycles each.
    auto half_step = [&](const Frags& f, Frags& g, int rbuf, int k2, int ks, int cbuf, auto c0, auto c1) {
        constexpr int C0 = decltype(c0)::value, CN = decltype(c1)::value - C0;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            f32x4& c = acc[m / (2 * PB)][m % (2 * PB)];
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[m % (2 * PB)], f.x[m / (2 * PB)], c, 0, 0, 0);
            pin(c);
#pragma unroll
            for (int i = m * NF / NM; i < (m + 1) * NF / NM; ++i) read_one(g, rbuf, k2, i);
#pragma unroll
            for (int i = m * CN / NM; i < (m + 1) * CN / NM; ++i) copy_one(ks, cbuf, C0 + i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // all but the youngest `steps` steps of this wave's copies have landed
    auto wait_steps = [&](auto steps_tag) {
        constexpr int K = decltype(steps_tag)::value;
        if (XI % 8 == 0 || n_x == XW) dev::dma_wait<K * (2 + XW)>();
        else                          dev::dma_wait<K * (1 + XW)>();
    };
    // Half a step is multiplied while the operands of the next half are on their way from LDS.  Behind
    // the barrier every wave has its operands of step ks in registers, so step ks + NBUF is copied over it.
    const int ahead = min(NBUF, nk);
    for (int i = 0; i < ahead; ++i) copy_step(i, i);
    // (while they are on their way) where the rows go, and this lane's rotary entries
    if (tid < BM) sm_dest[tid] = resolve_row(a, row0 + tid);
    const int j0 = 16 * PB * wn + 4 * PB * g4;                      // first of the lane's features (and of their partners, 64 further)
    float2 turns[4 * PB];
    if (kv == 0) {
#pragma unroll
        for (int i = 0; i < 4 * PB; ++i) turns[i] = *reinterpret_cast<const float2*>(&a.rope[j0 + i].turns_hi);
    }
    if (ahead == NBUF) wait_steps(std::integral_constant<int, NBUF - 1>{}); else dev::dma_wait<0>();
    lds_barrier();
    Frags f0, f1;
    read(f0, 0, 0);
    int buf = 0, ks = 0;
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, NC / 2> CH;
    typedef std::integral_constant<int, NC> CN;
    // (copies of step ks + NBUF: the first half behind step ks's barrier, the rest in the step after)
    int last = 0;                                                   // buffer of the step before
    if (nk > NBUF) {
        half_step(f0, f1, 0, 1, 0, 0, C0{}, C0{});
        for (;;) {
            wait_steps(std::integral_constant<int, NBUF - 2>{});
            lds_barrier();
            const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
            half_step(f1, f0, nbuf, 0, ks + NBUF, buf, C0{}, CH{});
            last = buf; buf = nbuf;
            ++ks;
            half_step(f0, f1, buf, 1, ks + NBUF - 1, last, CH{}, CN{});
            if (ks >= nk - NBUF) break;
        }
    } else {
        half_step(f0, f1, 0, 1, 0, 0, C0{}, C0{});
    }
    // Nothing more to ask for.  Where halves are drawn for, the last steps are multiplied as they arrive; elsewhere all of them are waited for at first, in shorter code.  us
    // per launch, all waited for -> as they arrive (median of three runs, 8 KV heads): drawn, hidden 4096 1300 rows 27.96 -> 27.80, 1500 29.41 -> 29.20, hidden 8192 1500 49.8 -> 49.5,
    // 2048 61.6 -> 61.4 (1050 42.6 -> 43.0); not drawn, hidden 512 150 rows 5.8 -> 6.1, hidden 3072 150 11.5 -> 11.9, hidden 4096 224 13.5 -> 13.8, 3501 (one workgroup per tile) 54.0 -> 54.1.
    int drawn = 0;
    int32_t* const counter = a.ws_counters + (size_t)(rt * nct + ct) * kDecodeCounterStride + wave;
    if (DRAWN) {                                                    // (see below)
        // On an address that all lanes share the compiler makes of it a sum over the wave, whose result it asks for at once: the last steps' copies and the
        // trip would be waited for before any of them is multiplied.  us per launch, so -> as it is: hidden 4096 1000 rows 24.0 -> 23.9, hidden 3072 1300 24.2 -> 23.8,
        // hidden 8192 1000 40.5 -> 39.9, 1500 50.9 -> 50.1, 2048 63.0 -> 62.7.
        uint32_t at = 0;
        asm volatile("" : "+v"(at));
        if (lane == 0) drawn = __hip_atomic_fetch_add(counter + at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    auto wait_left = [&](auto self, int left, auto steps_tag) -> void {
        constexpr int K = decltype(steps_tag)::value;
        if (left >= K || K == 0) wait_steps(steps_tag);         // (what was drawn counts as one more copy: waited for a little early)
        else if constexpr (K > 0) self(self, left, std::integral_constant<int, K - 1>{});
    };
    for (;; ++ks) {
        if constexpr (DRAWN) wait_left(wait_left, nk - 2 - ks, std::integral_constant<int, NBUF - 2>{});
        else                 dev::dma_wait<0>();
        lds_barrier();
        buf = buf + 1 == NBUF ? 0 : buf + 1;
        half_step(f1, f0, buf, 0, 0, 0, C0{}, C0{});                // (past the end: not used)
        if (ks == nk - 1) break;
        half_step(f0, f1, buf, 1, 0, 0, C0{}, C0{});
    }
    // From here on a wave is on its own.
    if constexpr (SK == 2) {
        // One of the two waves that hold a sum's halves leaves its half in the workspace, past the L2s, which are not coherent, 16 bytes a lane,
        // and the other goes on with both.  Tiles of up to 96 rows: both leave theirs, and the one that arrives second goes on.  Taller ones: the one that
        // drew first, some steps ago, leaves its half, raises the counter once more and is done; the other waits for that.  It waits
        // for a wave that has started and waits for nobody, so the wait ends whatever else the chip does.  That spares it its own stores and a trip
        // to the counter, and the memory half of the writes, for a trip more where both end at once: us per launch, both leave theirs -> one does, hidden
        // 4096 150 rows (tiles of 32) 14.2 -> 15.0, 300 (64) 15.9 -> 16.4, 512 (64) 17.9 -> 18.2, 700 (96) 21.6 -> 21.6, 1000 (128) 24.2 -> 23.9; hidden 3072 150 rows 11.7 ->
        // 12.4, 700 (96) 18.3 -> 18.2; hidden 8192 700 (96) 34.3 -> 34.6, 1000 rows 40.6 -> 39.2, 1500 (192) 52.0 -> 50.0, 2048 (256) 64.2 -> 61.8 (the last three with the draw waited for);
        // hidden 768 900 rows (128) 12.2 -> 11.2, 1024 12.6 -> 11.7, 2048 15.4 -> 15.2, 3072 18.9 -> 18.6; hidden 512, where a wave draws at its end, 11.1 -> 11.6: not there.  (In 8-byte pieces chunk passes of 1000 tokens took 397 us for 393, 311 for 309 at hidden 8192.)
        constexpr int NP = XB * 2 * PB;
        const int tile = rt * nct + ct;
        float* const halves = a.ws_partials + (size_t)tile * (DRAWN ? 1 : 2) * 8 * (BM * 16);
        auto leave = [&](float* to) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const f32x4& v = acc[i / (2 * PB)][i % (2 * PB)];
                dev::st_agent4(to, i * 1024 + lane * 16, __builtin_bit_cast(uint4, v));
            }
        };
        int from = part ^ 1;
        if constexpr (DRAWN) {
            from = 0;
            if (__builtin_amdgcn_readfirstlane(drawn) == 0) {
                leave(halves + (size_t)wave * (BM * 16));
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_s_waitcnt(0);                      // (acknowledged)
                if (lane == 0) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < 3) __builtin_amdgcn_s_sleep(1);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            leave(halves + (size_t)(part * 8 + wave) * (BM * 16));
            if (!dev::wave_arrives_last(counter, SK)) return;
        }
        const float* const theirs = halves + (size_t)(from * 8 + wave) * (BM * 16);
        float4 o[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) o[i] = dev::ld_agent4(theirs, i * 1024 + lane * 16);
        if (DRAWN && lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);     // (ready for the next launch)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            f32x4& v = acc[i / (2 * PB)][i % (2 * PB)];
            v[0] += o[i].x; v[1] += o[i].y; v[2] += o[i].z; v[3] += o[i].w;
        }
    }

    // lane: token 16 (XB wm + mi) + c16, features j0 .. j0 + 4 PB - 1 and 64 further, 4 PB in a row each.  A chunk's rows leave through
    // the L2s (agent scope): what lies there when a launch ends is written back before the next one starts (390 -> 385 us).
    char* const chunk_out = reinterpret_cast<char*>(kv == 0 ? a.k_out : a.v_out) + ((size_t)head * a.token_stride + row0) * (2 * D);
    uint16_t* const out = reinterpret_cast<uint16_t*>(kv == 0 ? a.k_out : a.v_out) + (size_t)head * a.token_stride * D + j0;
#pragma unroll
    for (int mi = 0; mi < XB; ++mi) {
        const RowDest d = sm_dest[16 * (XB * wm + mi) + c16];
        uint32_t lo[2 * PB], hi[2 * PB];
#pragma unroll
        for (int p = 0; p < PB; ++p)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                float l[2], h[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    l[k] = acc[mi][p][i + k]; h[k] = acc[mi][PB + p][i + k];
                    if (kv == 0) {
                        float c, s;
                        rope_cs(turns[4 * p + i + k].x, turns[4 * p + i + k].y, d.pos, c, s);
                        const float k0 = l[k] * c - h[k] * s;
                        const float k1 = l[k] * s + h[k] * c;
                        l[k] = k0; h[k] = k1;
                    }
                }
                lo[2 * p + i / 2] = dev::pack_bf16(l[0], l[1]);
                hi[2 * p + i / 2] = dev::pack_bf16(h[0], h[1]);
            }
        if (!d.valid) continue;
        uint16_t* const o = out + d.elem_off;
        if constexpr (PB == 1) {
            *reinterpret_cast<uint2*>(o) = make_uint2(lo[0], lo[1]);
            *reinterpret_cast<uint2*>(o + 64) = make_uint2(hi[0], hi[1]);
        } else if (a.table == nullptr) {                            // a chunk's rows lie one behind the other
            const uint32_t at = (16 * (XB * wm + mi) + c16) * (2 * D) + 2 * j0;
            dev::st_agent4(chunk_out, at, make_uint4(lo[0], lo[1], lo[2], lo[3]));
            dev::st_agent4(chunk_out, at + D, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        } else {
            *reinterpret_cast<uint4*>(o) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<uint4*>(o + 64) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        }
    }
}

template <int MI, int WN, int SK, bool DRAWN = SK == 2 && split_drawn(MI, 4096)>
hipError_t launch_tile(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    const int row_tiles = (total_rows + 32 * MI - 1) / (32 * MI), nct = 2 * a.Hkv;
    const int grid_tiles = SK == 1 && nct % 4 == 0 ? (row_tiles + 1) / 2 * 2 : row_tiles;
    hipLaunchKernelGGL((materialize_tile_kernel<MI, WN, SK, DRAWN>), dim3(nct * grid_tiles * SK), dim3(512), 0, s,
                       a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, row_tiles, a);
    return hipGetLastError();
}

// Tile height.  One workgroup fills a compute unit's LDS, a launch is as long as its slowest
// compute unit, and a workgroup's time grows slower than its height: so the smallest height that gives no compute unit two
// workgroups, hidden axis halved while that holds.  Up to 128 rows two workgroups per tile are ahead at every width; taller
// tiles leave the chip fewer bytes to fetch, but more partials to exchange, and pay from some hidden size on (us, one workgroup per tile
// of fewer rows -> two per taller tile, before only one of the two left its half; 160 and 192 rows: hidden 2048 1050 rows 18.6 -> 19.5, 1500 18.7 -> 20.6, hidden 2560
// 1206 23.4 -> 22.3, hidden 3072 1050 26.4 -> 23.1, hidden 4096 1050 32.4 -> 29.1, 1500 31.7 -> 30.3, hidden 5120 1206 41.6 -> 33.9, hidden 6144 1500 47.4 -> 41.3; since then
// a chunk pass of 1050 tokens (8B, four layers) 207 -> 191, of 1300 219 -> 212; 256 rows: hidden 4096 1700
// 31.7 -> 34.8, hidden 5120 1800 41.9 -> 44.4, 2048 48.0 -> 45.6, hidden 6144 2000 52.4 -> 52.0, hidden 8192 2000 71.0 -> 66.7 when it was drawn).  Behind the attention of a question pass, which
// streams the cache over the partials, the taller split costs more than it gives below hidden 8192: passes of four layers, sixteen 8B users 657 -> 674, twelve 3B users of
// 100 rows 421 -> 438 (one card of several: 419 -> 408); 70B, split against not, sixteen of 100 rows 1046 against 1088.  Beyond one full round the
// height with the smallest rounds x (4 + MI), which is what the times follow (hidden 4096, tiles of 128 / 160 / 192 / 256 rows: 2500 rows 72 / 47 / 49 / 56 us, 3501
// rows 76 / 86 / 94 / 58).
hipError_t launch_tiled(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    const int nct = 2 * a.Hkv;
    auto groups = [&](int mi) { return nct * ((total_rows + 32 * mi - 1) / (32 * mi)); };
    auto halved = [&](int mi) {
        const int64_t tiles = groups(mi);
        return (a.Hd % (2 * BK)) == 0 && tiles * 2 <= 256 && 32 * mi <= most_split_rows(a.Hd, a.table != nullptr) && a.ws_partials &&
               tiles * split_partials(mi, a.Hd) * (32 * mi) * D <= a.ws_partial_floats && tiles * kDecodeCounterStride <= a.ws_n_counters;
    };
    if (halved(1)) return launch_tile<1, 4, 2>(a, total_rows, s);
    if (halved(2)) return launch_tile<2, 4, 2>(a, total_rows, s);
    if (halved(3)) return launch_tile<3, 4, 2>(a, total_rows, s);
    if (halved(4)) return split_drawn(4, a.Hd) ? launch_tile<4, 2, 2>(a, total_rows, s) : launch_tile<4, 2, 2, false>(a, total_rows, s);
    if (halved(5)) return launch_tile<5, 4, 2>(a, total_rows, s);
    if (halved(6)) return launch_tile<6, 2, 2>(a, total_rows, s);
    if (halved(8)) return launch_tile<8, 2, 2>(a, total_rows, s);
    int best = 3;
    long best_cost = -1;
    for (int mi : {3, 4, 5, 6, 8}) {
        const long cost = (long)((groups(mi) + 255) / 256) * (4 + mi);
        if (best_cost < 0 || cost < best_cost) { best = mi; best_cost = cost; }
    }
    switch (best) {
        case 3: return launch_tile<3, 4, 1>(a, total_rows, s);
        case 4: return launch_tile<4, 2, 1>(a, total_rows, s);
        case 5: return launch_tile<5, 4, 1>(a, total_rows, s);
        case 6: return launch_tile<6, 2, 1>(a, total_rows, s);
        default: return launch_tile<8, 2, 1>(a, total_rows, s);
    }
}

// ---- skinny form: a few hundred token rows at most, hidden a multiple of 1024 ------------------
// Too few rows for the tiled GEMM to fill the chip.  Here a workgroup owns 16 or 32 rows x 16 rotary
// pairs (features 16g .. 16g+15 and their partners 64 further) of one head of K or of V, and its eight
// waves split the HIDDEN axis.  Loading operands straight into matrix-core layout was bound by the
// vector cache's request rate - consecutive lanes sit on sixteen different rows, every lane's 16 bytes
// is a request of its own (64 rows, hidden 4096: 98 MB in 17 us) - so a wave loads its slice of the
// hidden axis row-wise: sixteen consecutive lanes take 256 consecutive bytes of one row; it parks the rows in a private LDS region (272-byte rows: sixteen
// lanes write one whole row, sixteen lanes read 16 bytes of sixteen different rows, both without a
// bank conflict) and reads them back in operand layout.  The region belongs to one wave: no
// workgroup barrier in the loop.  The eight partial tiles meet in LDS, and the rotation and the single
// rounding to bf16 follow.
template <int MI, int NB>
__global__ __launch_bounds__(512) void materialize_skinny_staged_kernel(
        const void* __restrict__ hidden, const void* __restrict__ w_k, const void* __restrict__ w_v, int Hd, int Hkv, int total_rows, MaterializeArgs a) {
    constexpr int NWV = 8, SC = 128;                    // waves; hidden columns per wave and round
    constexpr int TM = 16 * MI;
    constexpr int NR = 32 + TM;                         // rows staged per round: 16 + 16 weight rows, TM token rows
    constexpr int NL = NR / 4;                          // 16-byte loads per lane and round (a load covers 4 rows)
    constexpr int RS = SC + 8;                          // bf16 per staged row
    constexpr int STAGE_BYTES = NWV * NR * RS * 2, RED_BYTES = NWV * TM * 33 * 4;
    __shared__ __attribute__((aligned(16))) char smem[STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    const int pg = blockIdx.x & 3, kv = (int)(blockIdx.x >> 2) >= Hkv, head = (int)(blockIdx.x >> 2) - kv * Hkv;
    const int row0 = blockIdx.y * TM;
    const int kslice = Hd / NWV;                      // a multiple of SC (checked by the launcher)
    const int n_rounds = kslice / SC;

    // the epilogue's row and rotary entry of this thread are fixed: asked for now, not after the sums
    static_assert(TM * 16 <= NWV * 64, "one output pair per thread");
    const int et = tid >> 4, ep = tid & 15;
    const RopeEntry rope_e = a.rope[16 * pg + ep];
    RowDest edest = resolve_row(a, row0 + min(et, TM - 1));
    if (et >= TM) edest.valid = false;

    // load i of a round: row 4 i + lane / 16 of the staged rows, 16 bytes at column 8 (lane % 16)
    const int lr = lane >> 4, lc = 8 * (lane & 15);
    const size_t col0 = (size_t)wave * kslice + lc;
    const uint16_t* wbase = reinterpret_cast<const uint16_t*>(kv == 0 ? w_k : w_v) + ((size_t)head * D + 16 * pg + lr) * Hd + col0;
    const uint16_t* xp[MI * 4];
#pragma unroll
    for (int i = 0; i < MI * 4; ++i)
        xp[i] = reinterpret_cast<const uint16_t*>(hidden) + (size_t)min(row0 + 4 * i + lr, total_rows - 1) * Hd + col0;
    auto load = [&](uint4 (&b)[NL], int r) {
        const int off = min(r, n_rounds - 1) * SC;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b[i] = ldg16(wbase + (size_t)(4 * i) * Hd + off);
            b[4 + i] = ldg16(wbase + (size_t)(D / 2 + 4 * i) * Hd + off);
        }
#pragma unroll
        for (int i = 0; i < MI * 4; ++i) b[8 + i] = ldg16(xp[i] + off);
    };

    uint16_t* const st = reinterpret_cast<uint16_t*>(smem) + (size_t)wave * NR * RS;
    f32x4 acc[MI][2];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) { acc[mi][0] = f32x4{0.f, 0.f, 0.f, 0.f}; acc[mi][1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    auto process = [&](const uint4 (&b)[NL]) {
        __builtin_amdgcn_wave_barrier();                // the last round's reads stay ahead of these writes
#pragma unroll
        for (int i = 0; i < NL; ++i) *reinterpret_cast<uint4*>(st + (4 * i + lr) * RS + lc) = b[i];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < SC / 32; ++j) {
            const bf16x8 wl = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(st + c16 * RS + 32 * j + 8 * g4));
            const bf16x8 wh = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(st + (16 + c16) * RS + 32 * j + 8 * g4));
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const bf16x8 xa = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(st + (32 + 16 * mi + c16) * RS + 32 * j + 8 * g4));
                acc[mi][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, wl, acc[mi][0], 0, 0, 0);
                acc[mi][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, wh, acc[mi][1], 0, 0, 0);
            }
        }
    };
    // NB rounds of loads in flight; no load under a branch (the launcher sees to it that the rounds
    // are a multiple of NB), the last NB rounds are consumed without asking for more
    {
        uint4 b[NB][NL];
#pragma unroll
        for (int i = 0; i < NB; ++i) load(b[i], i);
        for (int r = NB; r < n_rounds; r += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                process(b[i]);
                load(b[i], r + i);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) process(b[i]);
    }

    // the eight partial tiles meet in LDS (over the staging rows, once every wave is done with its own)
    __syncthreads();
    float (*red)[TM][33] = reinterpret_cast<float (*)[TM][33]>(smem);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[wave][16 * mi + 4 * g4 + i][16 * h + c16] = acc[mi][h][i];
    __syncthreads();

    uint16_t* out = reinterpret_cast<uint16_t*>(kv == 0 ? a.k_out : a.v_out) + (size_t)head * a.token_stride * D;
    if (edest.valid) {
        const RowDest d = edest;
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) { lo += red[w][et][ep]; hi += red[w][et][16 + ep]; }
        const int j = 16 * pg + ep;
        if (kv == 0) {
            float c, s;
            rope_cs(rope_e, d.pos, c, s);
            const float k0 = lo * c - hi * s;
            const float k1 = lo * s + hi * c;
            lo = k0; hi = k1;
        }
        out[d.elem_off + j] = f32_to_bf16_rne(lo);
        out[d.elem_off + j + 64] = f32_to_bf16_rne(hi);
    }
}


// ---- a handful of rows (a decode step) on the staged form ---------------------------------------
// The same scheme cut finer, so that a launch with 1 .. 16 token rows still has 256 workgroups: a
// workgroup owns NP rotary pairs (2 NP weight rows: NP "low" features and their partners) and TMR
// token rows, which together fill part of one 16 x 16 matrix tile - lanes beyond repeat a row and
// their results are dropped.  Eight waves split the hidden axis as above; only the TMR real token
// rows are staged.
template <int NP, int TMR, int NB>
__global__ __launch_bounds__(512) void materialize_fewrows_kernel(
        const void* __restrict__ hidden, const void* __restrict__ w_k, const void* __restrict__ w_v, int Hd, int Hkv, int total_rows, MaterializeArgs a) {
    constexpr int NWV = 8, SC = 128;                    // waves; hidden columns per wave and round
    constexpr int NR = 2 * NP + TMR;                    // rows staged per round
    static_assert(NP % 4 == 0 && TMR % 4 == 0 && 2 * NP <= 16 && TMR <= 16, "whole loads of four rows; one matrix tile");
    constexpr int NL = NR / 4;                          // 16-byte loads per lane and round
    constexpr int RS = SC + 8;                          // bf16 per staged row
    constexpr int STAGE_BYTES = NWV * NR * RS * 2, RED_BYTES = NWV * TMR * (2 * NP + 1) * 4;
    __shared__ __attribute__((aligned(16))) char smem[STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    constexpr int GPH = (D / 2) / NP;                   // pair groups per head
    const int pg = blockIdx.x % GPH, kv = (int)(blockIdx.x / GPH) >= Hkv, head = (int)(blockIdx.x / GPH) - kv * Hkv;
    const int row0 = blockIdx.y * TMR;
    const int kslice = Hd / NWV;                      // a multiple of SC (checked by the launcher)
    const int n_rounds = kslice / SC;

    // the epilogue's row and rotary entry of this thread are fixed: asked for now, not after the sums
    const int et = tid / NP, ep = tid % NP;
    const RopeEntry rope_e = a.rope[NP * pg + ep];
    RowDest edest = resolve_row(a, row0 + min(et, TMR - 1));
    if (et >= TMR) edest.valid = false;

    // load i of a round: staged row 4 i + lane / 16, 16 bytes at column 8 (lane % 16)
    const int lr = lane >> 4, lc = 8 * (lane & 15);
    const size_t col0 = (size_t)wave * kslice + lc;
    const uint16_t* wbase = reinterpret_cast<const uint16_t*>(kv == 0 ? w_k : w_v) + ((size_t)head * D + NP * pg + lr) * Hd + col0;
    const uint16_t* xp[TMR / 4];
#pragma unroll
    for (int i = 0; i < TMR / 4; ++i)
        xp[i] = reinterpret_cast<const uint16_t*>(hidden) + (size_t)min(row0 + 4 * i + lr, total_rows - 1) * Hd + col0;
    auto load = [&](uint4 (&b)[NL], int r) {
        const int off = min(r, n_rounds - 1) * SC;
#pragma unroll
        for (int i = 0; i < NP / 4; ++i) {
            b[i] = ldg16(wbase + (size_t)(4 * i) * Hd + off);
            b[NP / 4 + i] = ldg16(wbase + (size_t)(D / 2 + 4 * i) * Hd + off);
        }
#pragma unroll
        for (int i = 0; i < TMR / 4; ++i) b[NP / 2 + i] = ldg16(xp[i] + off);
    };

    uint16_t* const st = reinterpret_cast<uint16_t*>(smem) + (size_t)wave * NR * RS;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int brow = c16 < 2 * NP ? c16 : 0;            // weight row of this lane's column (columns beyond: dropped)
    const int arow = 2 * NP + min(c16, TMR - 1);        // token row of this lane's operand row
    auto process = [&](const uint4 (&b)[NL]) {
        __builtin_amdgcn_wave_barrier();                // the last round's reads stay ahead of these writes
#pragma unroll
        for (int i = 0; i < NL; ++i) *reinterpret_cast<uint4*>(st + (4 * i + lr) * RS + lc) = b[i];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < SC / 32; ++j) {
            const bf16x8 wv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(st + brow * RS + 32 * j + 8 * g4));
            const bf16x8 xa = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(st + arow * RS + 32 * j + 8 * g4));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, wv, acc, 0, 0, 0);
        }
    };
    {
        uint4 b[NB][NL];
#pragma unroll
        for (int i = 0; i < NB; ++i) load(b[i], i);
        for (int r = NB; r < n_rounds; r += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                process(b[i]);
                load(b[i], r + i);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) process(b[i]);
    }

    // the eight partial tiles meet in LDS (over the staging rows, once every wave is done with its own)
    __syncthreads();
    float (*red)[TMR][2 * NP + 1] = reinterpret_cast<float (*)[TMR][2 * NP + 1]>(smem);
    // lane holds tokens 4 g4 + i, column c16
    if (c16 < 2 * NP)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * g4 + i < TMR) red[wave][4 * g4 + i][c16] = acc[i];
    __syncthreads();

    if (edest.valid) {
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) { lo += red[w][et][ep]; hi += red[w][et][NP + ep]; }
        const int j = NP * pg + ep;
        if (kv == 0) {
            float c, s;
            rope_cs(rope_e, edest.pos, c, s);
            const float k0 = lo * c - hi * s;
            const float k1 = lo * s + hi * c;
            lo = k0; hi = k1;
        }
        uint16_t* out = reinterpret_cast<uint16_t*>(kv == 0 ? a.k_out : a.v_out) + (size_t)head * a.token_stride * D;
        out[edest.elem_off + j] = f32_to_bf16_rne(lo);
        out[edest.elem_off + j + 64] = f32_to_bf16_rne(hi);
    }
}

template <int TMR>
hipError_t launch_fewrows_t(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    constexpr int NP = 4;
    const dim3 grid(2 * a.Hkv * (64 / NP), (total_rows + TMR - 1) / TMR), block(512);
    const int rounds = a.Hd / 1024;
    if (rounds % 4 == 0) hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 4>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
    else if (rounds % 2 == 0) hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 2>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
    else hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 1>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_materialize_fewrows(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    if (total_rows <= 4) return launch_fewrows_t<4>(a, total_rows, s);
    if (total_rows <= 8) return launch_fewrows_t<8>(a, total_rows, s);
    return launch_fewrows_t<16>(a, total_rows, s);
}

hipError_t launch_materialize_tiles(const MaterializeArgs& a, int total_rows, hipStream_t s) { return launch_tiled(a, total_rows, s); }

hipError_t launch_materialize_staged(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    // rows staged through LDS: 16-row tiles up to 64 rows (64 x 4 workgroups fill the chip),
    // 32-row tiles beyond (half the workgroups, the weights re-read half as often)
    const int rounds = a.Hd / 1024;             // per wave: an eighth of the hidden axis, 128 columns a round
    const bool mi2 = total_rows > 64;
    const dim3 grid(2 * a.Hkv * 4, mi2 ? (total_rows + 31) / 32 : (total_rows + 15) / 16), block(512);
    if (rounds % 2 == 0) {
        if (mi2) hipLaunchKernelGGL((materialize_skinny_staged_kernel<2, 2>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
        else     hipLaunchKernelGGL((materialize_skinny_staged_kernel<1, 2>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
    } else {
        if (mi2) hipLaunchKernelGGL((materialize_skinny_staged_kernel<2, 1>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
        else     hipLaunchKernelGGL((materialize_skinny_staged_kernel<1, 1>), grid, block, 0, s, a.hidden, a.w_k, a.w_v, a.Hd, a.Hkv, total_rows, a);
    }
    return hipGetLastError();
}

}  // namespace matkv
