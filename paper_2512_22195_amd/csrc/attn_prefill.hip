// Question prefill attention on the matrix cores, bf16, head_dim 128 (paper Section V-A "prefill
// time": row i of the question attends to every chunk key and to question keys j <= i).
//
// The M dimension is the flattened (question row, query head of one KV head) index.  A
// workgroup of eight waves owns a tile of 256 or 128 such rows and one work unit of the cache; a wave
// owns 32 rows and walks the unit's tokens in blocks:
//   S^T = K Q^T     32x32x16; A = K rows from LDS, B = Q held in registers
//   softmax         online, per lane on its own column; the two half waves agree on the running
//                   maximum through a register swap
//   O^T += V^T P^T  A = V through the transposing LDS read, B = P rounded to bf16
// 256-row tiles: all waves walk the same 64-token blocks.  128-row tiles: waves 0 to 3 and 4 to 7 own
// the same rows and take every second block; at the end each finishes half of the dims for both.
//
// What bounds it.  A step of 64 tokens needs of a SIMD 2 x 32 matrix instructions and 2 x 8 small ones (2200 cycles), of its
// vector ALU about 1300 cycles (an exponential takes 8), and of the compute unit's LDS 2 x 8 x 16 KB at 256 bytes a cycle (1024
// cycles) and the copies' 256.  On long walks the chip's power limit sets the pace: at 3290 cycles a step (3170 by now) the clock is
// 1.68 GHz (matrix instructions alone on such data would run at 1.7), and a large library GEMM reaches 1385 TFLOP/s here.  Hence:
//  - K and V go from global memory straight into LDS (dma16), into unpadded rows whose 16-byte pieces
//    are permuted so that operand reads and transposing reads meet no bank conflict; up to three blocks
//    are on their way while another is in use.
//  - matrix and vector work of a wave alternate instruction by instruction (see "the walk").  The two waves of a SIMD half a step
//    apart with a barrier behind each phase - one multiplies while the other is in its softmax - took 3550
//    cycles a step: every phase had its own chain of dependent maxima, reads and scalar work with nothing beside it.
//  - 32x32x16 rather than 16x16x32: one row per lane halves the work per row.
//  - the fixed part of a workgroup, 10 us around a 1000-token chunk's longest walk of 13, is kept short: it starts when Q and K of its first
//    block have landed and copies the rest beside the first scores, and token groups are folded in registers (3.2 -> 1.9 us).
// Measured, us per pass, that form -> this one without the last point: chunk passes of 1000 tokens (8B, 8 layers) 418 -> 404, (70B, 4 layers) 320 -> 314,
// of 3501 674 -> 664; question passes (4 or 8 layers) of sixteen 8B users over 5000 tokens 705 -> 686, of four 70B users over
// 20 000 1475 -> 1440 (a step 2.03 -> 1.95 us), of one over 10 000 316 -> 312.  Left out of a step of 1.95 us, for the measurement
// only: every LDS read 1.94, the exponentials 1.90, the copies 1.80.  Tried: the weights formed beside the scores' matrix
// instructions only 3870 cycles, all copies of a step at once 3900, the waves of a SIMD taking turns at the higher priority
// 3360 against 3390, scalar work ahead of the first matrix instructions instead of between the periods 3390 against 3250.
// Of a step's 3275 cycles between two periods' matrix instructions 180 went to the maxima, 190 to the row sums, 130 to the copies, 130 to
// finding the next block and 60 to whether it is ragged (each left out in turn).  What is rare stands out of line, whether a block is ragged is
// found with the block and the maxima take three instructions less: 3170, and 0.3 to 0.7 % per chunk and question pass, nothing where the power
// limit sets the pace (70B, 20 000 tokens: 1.87 -> 1.76 GHz).  Tried: the maxima, the operands' addresses and the search for the next block among
// the matrix instructions (3190 to 3230; 128-row tiles 3430 -> 3590), K copied a step earlier (no change), whole blocks on a path of their own (3270).
// The last point: chunk passes 407 -> 385, 319 -> 301, 654 -> 637, question passes 687 -> 681, 1439 -> 1445, 318 -> 313.
//
// An instance whose cache is one unit gets its output rows directly; otherwise every unit leaves an
// unnormalised partial (accumulator, running maximum, sum) per row and a second, chip-wide
// launch folds the units of each row together (the last-arrival merge of the decode kernels
// would leave that work to a handful of compute units here: the partials of a question are
// megabytes, not kilobytes).
#include <type_traits>

#include "attn_common.h"

namespace matkv {
namespace {

using namespace attn;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int D = 128;
constexpr int NW = 8;                 // waves of a workgroup
constexpr int WR = 32;                // rows of a wave
constexpr int TB = 64;                // tokens of a block
constexpr int kPageT0 = -(1 << 30);   // "position" of a page block: every row sees all of it
constexpr float kLazyLog2 = 8.0f;     // slack of the running reference exponent, in powers of two

__device__ __forceinline__ s16x4 lds_read_tr(const char* p) {
    typedef s16x4 __attribute__((address_space(3))) * lptr;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(uintptr_t)p);
}

// One block as the multiplying side sees it (wave-uniform).
struct BlockDesc {
    int n;              // token rows; 0: none that a row of this wave may see, -1: no group of the workgroup has a block in this step
    int t0;             // tail row of the block's first token; far below every row for a page
    bool ragged;        // fewer than a whole block, or past what the wave's first row may see
    float sk, sv;       // scales of a compressed page's codes
};

// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);      // one, two, four, eight lanes to the right within 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // lane 15 of a row to the next, of the first and third
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // lane 31 to the upper half
    return v;
}

// A launch has units x KV heads x the longest question's tiles workgroups, and a shorter question has no work for
// the last of them.  Left where they fall, those idle ones lie between the others, and since workgroups go to the XCDs, and
// there to the engines, in turn, some compute units are given two working ones while others have none (70B shape,
// questions of 64, 50 and 21 rows over 12 900 tokens: 142 us per layer, 75 without them).  So the tiles beyond the first of every
// unit are dealt to the workgroups behind the first ones without a gap, instance after instance.
// k-th such tile -> instance, unit and tile; false: there is none.
__device__ __forceinline__ bool find_further_tile(const InstanceInfo* __restrict__ insts, int batch, int k, int G, int rt, int& b, int& unit, int& tile) {
    const int lane = threadIdx.x & 63;
    for (int b0 = 0; b0 < batch; b0 += 64) {            // a lane per instance
        const InstanceInfo* in = insts + min(b0 + lane, batch - 1);
        const int further = (in->q_len * G - 1) / rt, unit0 = in->punit0;
        const int n = b0 + lane < batch ? in->n_punits * further : 0, upto = wave_scan(n);
        const uint64_t past = __builtin_amdgcn_ballot_w64(upto > k);
        if (past) {
            const int l = __builtin_ctzll(past), t = __builtin_amdgcn_readlane(further, l);
            const int r = k - __builtin_amdgcn_readlane(upto - n, l);
            b = b0 + l;
            unit = r / t; tile = 1 + r - unit * t;
            unit += __builtin_amdgcn_readlane(unit0, l);
            return true;
        }
        k -= __builtin_amdgcn_readlane(upto, 63);
    }
    return false;
}

// units .. chunk (a chunk's own attention) arrive in registers, so that the unit's record is asked for without waiting for the other arguments.
// batch: given where the tiles beyond the first are dealt out by find_further_tile, and left out elsewhere: one
// argument more moves the implicit ones into another line of the argument buffer, which costs every launch 0.3 us.
template <int RW, bool F8, typename... Batch>
__global__ __launch_bounds__(NW * 64, 2) void attn_prefill_kernel(
        const Unit* __restrict__ units, const InstanceInfo* __restrict__ insts, const Item* __restrict__ items, int chunk,
        KernelArgs a, Batch... batch) {
    constexpr bool DEAL = sizeof...(Batch) > 0;
    constexpr int TS = NW / RW;                         // token groups
    constexpr int RT = RW * WR;                         // rows per workgroup
    constexpr int TILE = TB * D * 2;                    // bytes of a K or a V tile
    constexpr int GROUP = TS == 1 ? 8 * TILE : 5 * TILE;    // LDS of a token group (see "the walk")
    constexpr int NI = TB / (4 * RW);                   // copies of four rows per wave, of K and of V
    typedef uint16_t T;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % RW, tg = wave / RW;           // row wave, token group
    const int lane = tid & 63;
    const int c32 = lane & 31, g2 = lane >> 5;
    const int G = a.Hq / a.Hkv;                         // 1, 2, 3, 4 or 8
    auto div_g = [&](int m) { return (int)__umulhi((unsigned)m << 3, a.g_mul); };     // m / G, m < 2^28
    // a chunk's own attention: tile t walks (t + 1) * RT / G keys, so the longest go first
    int kvh = blockIdx.y, tile = chunk ? gridDim.z - 1 - blockIdx.z : blockIdx.z, unit_i = blockIdx.x, b = -1;
    if constexpr (DEAL) {
        if (blockIdx.z > 0) {
            const int further = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * (blockIdx.z - 1)), k = further / a.Hkv;
            if (!find_further_tile(insts, batch..., k, G, RT, b, unit_i, tile)) return;
            kvh = further - k * a.Hkv;
        }
    }

    Unit unit;
    InstanceInfo inst;
    if (chunk) {                               // the chunk: one instance without pages, its tail the one item
        unit = Unit{};
        unit.n_items = 1; unit.n_units_inst = 1; unit.has_tail = 1; unit.first.ntok = a.rows;
        inst = InstanceInfo{};
        inst.q_len = a.rows;
    } else {
        unit = table_record(units + unit_i);
        inst = table_record(insts + (DEAL && b >= 0 ? b : unit.inst));
    }
    const int m0 = tile * RT;
    const int n_m = inst.q_len * G;
    if (m0 >= n_m) return;                              // whole workgroup leaves together
    const int r_last = div_g(min(m0 + RT, n_m) - 1);
    const int wm0 = m0 + WR * rw;
    const bool wave_live = wm0 < n_m;                   // this wave has at least one real row
    const int vis_min = div_g(wm0) + 1;                    // tail rows every row of this wave may see
    const int vis_max = div_g(max(min(wm0 + WR, n_m) - 1, 0)) + 1;

    // K and V tiles of the token groups; the finished rows and their (maximum, sum) once those are dead
    __shared__ __attribute__((aligned(1024))) char smem[TS * GROUP + (TS == 1 ? 2 * NW * WR * 4 : 0)];

    // Every group walks the same blocks - the unit's items end to end (the tail clipped to the rows
    // this tile may see), TB token rows at a time, never across two items - and takes every TS-th.
    // All of it is wave-uniform.
    struct { const char* k; const char* v; int left, t0, item_i, row_bytes; float sk, sv; } wk;
    const int tail_visible = min(r_last + 1, a.max_tail);
    // the item's next block: K and V at k and v, tail row t0 (a page: far below every row); rows left from there on
    auto set_item = [&](uint64_t base, int page_tokens, int tok0, int ntok) {
        wk.left = base ? ntok : min(ntok, tail_visible);
        wk.t0 = base ? kPageT0 : tok0;
        wk.row_bytes = F8 && base ? D : 2 * D;
        if (base) {
            const size_t row = F8 ? D : 2 * D, head = (size_t)page_tokens * row;
            wk.k = reinterpret_cast<const char*>(base) + ((size_t)a.layer * 2 * a.Hkv + kvh) * head + (size_t)tok0 * row;
            wk.v = wk.k + (size_t)a.Hkv * head;
        } else {
            const size_t off = (((size_t)unit.inst * a.Hkv + kvh) * (size_t)a.max_tail + tok0) * (2 * D);
            wk.k = reinterpret_cast<const char*>(a.tail_k) + off;
            wk.v = reinterpret_cast<const char*>(a.tail_v) + off;
        }
    };
    // The next item's record is fetched (scalar loads) when its predecessor is taken up, so that taking
    // it up waits for nothing.
    struct { Item it; float sk, sv; } ahead;
    auto fetch_item = [&](int i) {
        ahead.it = table_record(items + unit.item0 + min(i, unit.n_items - 1));
        ahead.sk = 1.f; ahead.sv = 1.f;
        if (F8 && ahead.it.base) page_scales(ahead.it, a.layer, a.Hkv, kvh, ahead.sk, ahead.sv);
    };
    wk.item_i = 0;
    wk.sk = 1.f; wk.sv = 1.f;
    set_item(unit.first.base, unit.first.page_tokens, unit.first.tok0, unit.first.ntok);
    if (F8 && unit.first.base) page_scales(unit.first, a.layer, a.Hkv, kvh, wk.sk, wk.sv);
    fetch_item(1);
    // where a block's rows lie: K and V of its first row, row stride 2 D bytes (codes: D bytes).  Past the
    // unit's end the last block's first row is copied instead (a branch around the copies there cost 3 %); over compressed
    // pages (n = 0) nothing is: two blocks fetched and widened for nothing are a large part of a walk of three steps.
    struct Source { const char* k; const char* v; int n; bool codes; };
    Source src;
    src.k = wk.k; src.v = wk.v; src.n = 1; src.codes = F8 && wk.row_bytes == D;
    auto next_step = [&](BlockDesc& d) {
        d.n = -1; d.t0 = kPageT0; d.sk = 1.f; d.sv = 1.f; d.ragged = true;
        src.n = F8 ? 0 : 1;
        if (F8) src.codes = false;
#pragma unroll
        for (int g = 0; g < TS; ++g) {
            while (__builtin_expect(wk.left <= 0 && wk.item_i + 1 < unit.n_items, 0)) {
                ++wk.item_i;
                set_item(ahead.it.base, ahead.it.page_tokens, ahead.it.tok0, ahead.it.ntok);
                if (F8) { wk.sk = ahead.sk; wk.sv = ahead.sv; }
                fetch_item(wk.item_i + 1);
            }
            const int n = min(TB, wk.left);
            if (n <= 0) return;
            if (g == 0) d.n = 0;
            if (g == tg) {
                src.k = wk.k; src.v = wk.v; src.n = n; src.codes = F8 && wk.row_bytes == D;
                d.n = wave_live && wk.t0 < vis_max ? n : 0;
                d.t0 = wk.t0;
                d.ragged = n != TB || d.t0 + n > vis_min;
                if (F8) {
                    d.sk = wk.sk; d.sv = wk.sv;
                    if (TS == 2) asm volatile("" : "+v"(d.sk), "+v"(d.sv));      // (in vector registers: the scalar ones are all taken)
                }
            }
            wk.left -= n;
            wk.t0 += n;
            wk.k += n * wk.row_bytes; wk.v += n * wk.row_bytes;
        }
    };

    // A tile's rows are 256 bytes, sixteen 16-byte pieces.  Piece p of K row r sits at place
    // p ^ (r & 15), of V row r at p ^ 4 (r & 3); rows past the block's end repeat its last one.
    char* const group_lds = smem + tg * GROUP;
    const uint32_t lds0 = dev::lds_address(smem) + tg * GROUP;
    // Tiles of block i + d.  One group: four blocks of K and V.  Two groups: two tiles of K, three of V.
    int i4 = 0, i3 = 0;                                 // i mod 4, i mod 3
    auto k_at = [&](int d) { return TS == 1 ? ((i4 + d) & 3) * 2 * TILE : ((i4 + d) & 1) * TILE; };
    auto v_at = [&](int d) {
        if (TS == 1) return ((i4 + d) & 3) * 2 * TILE + TILE;
        const int j = i3 + d;
        return (2 + (j >= 3 ? j - 3 : j)) * TILE;
    };
    const int lrow = lane >> 4, place = lane & 15;
    auto copy_k1 = [&](const Source& s, int d, int i) {
        const int r = 4 * (rw + RW * i) + lrow;
        dev::dma16(s.k, (uint32_t)min(r, s.n - 1) * (2 * D) + 16 * (place ^ (r & 15)), lds0 + k_at(d) + rw * 1024 + i * RW * 1024);
    };
    auto copy_v1 = [&](const Source& s, int d, int i) {
        const int r = 4 * (rw + RW * i) + lrow;
        dev::dma16(s.v, (uint32_t)min(r, s.n - 1) * (2 * D) + 16 * (place ^ (4 * (r & 3))), lds0 + v_at(d) + rw * 1024 + i * RW * 1024);
    };
    auto copy_k = [&](const Source& s, int d) {
#pragma unroll
        for (int i = 0; i < NI; ++i) copy_k1(s, d, i);
    };
    auto copy_v = [&](const Source& s, int d) {
#pragma unroll
        for (int i = 0; i < NI; ++i) copy_v1(s, d, i);
    };
    // Compressed pages: codes go through registers (one step ahead of the copy they replace) and are
    // widened to bf16 on their way into the tile.  A lane moves 16 codes of a row: two pieces.
    // As with plain pages, the first scores wait for Q and K of the first block only, and V and the second block are widened beside
    // them.  us per layer, one user, the form with a barrier behind each phase / both blocks waited for and two more
    // widened past the end / now: 8B shape, 10 000 tokens and 4 rows 17.2 / 18.4 / 17.0, 64 rows 29.4 / 29.7 / 28.7, 1200 tokens and 32 rows 16.2 / 17.3 / 16.4,
    // 333 tokens and 100 rows 16.0 / 16.8 / 16.0; 70B shape, 10 000 tokens and 4 rows 18.0 / 19.6 / 17.9.
    // Tried: the codes of a step widened between its matrix instructions, K's half a step after they were asked for (+3 to 17 %).
    constexpr int NC = TB * D / (RW * 64 * 16);         // 16-byte loads per lane, of K and of V
    struct Codes { uint4 w[NC]; } kc, vc;
    const int ct = rw * 64 + lane;
    auto load_codes = [&](Codes& c, const char* from, int n) {
#pragma unroll
        for (int i = 0; i < NC; ++i) c.w[i] = ldg16(from + (uint32_t)min((ct >> 3) + RW * 8 * i, n - 1) * D + 16 * (ct & 7));
    };
    auto store_codes1 = [&](const Codes& c, int at, bool v, int i) {
        const int r = (ct >> 3) + RW * 8 * i, p = 2 * (ct & 7), turn = v ? 4 * (r & 3) : r & 15;
        char* const row = group_lds + at + r * (2 * D);
        *reinterpret_cast<uint4*>(row + 16 * (p ^ turn)) = e4m3x8_to_bf16x8(make_uint2(c.w[i].x, c.w[i].y));
        *reinterpret_cast<uint4*>(row + 16 * ((p + 1) ^ turn)) = e4m3x8_to_bf16x8(make_uint2(c.w[i].z, c.w[i].w));
    };
    auto store_codes = [&](const Codes& c, int at, bool v) {
#pragma unroll
        for (int i = 0; i < NC; ++i) store_codes1(c, at, v, i);
    };

    f32x16 ot[4];                     // O^T: dims 32 t + 8 (i / 4) + 4 g2 + i % 4 of the lane's row
    f32x4 ol = f32x4{0.f, 0.f, 0.f, 0.f};   // sum of this lane's weights (every element the same; [0] is kept right)
    float mrow = kNegBig;             // reference score of the lane's row, unscaled
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) ot[t][i] = 0.f;

    // Scores stay unscaled until the exponent: 2^((s - m) c) is one multiply-add and one
    // exponential per element, with m the row's reference score (unscaled too).
    const int koff = c32 * 256 + 16 * (g2 ^ (c32 & 15));
    const int e16 = lane & 15;
    const int voff = (4 * g2 + (e16 >> 2)) * 256 + 64 * (e16 >> 2) + 32 * ((lane >> 4) & 1) + 8 * (e16 & 3);
    // ---- the walk ----
    // A block is taken in halves of 32 tokens.  A period of a wave multiplies the scores of half t + 1 (eight matrix
    // instructions), then the output of half t - 1 (eight more), and between these, evenly, forms the weights of half t and finds the
    // maximum of half t + 1: the vector work of a SIMD's two waves then stands beside their matrix work.  (Counters, four
    // 70B users over 20 000 tokens: matrix cores at work 60 % of the launch, 54 with a barrier behind each phase, the vector ALU beside them in 45 % of that.)
    // Step i reads K of block i + 1 and V of block i and has one barrier.  It copies block i + AHEAD, K first, and ends when that K has
    // landed and all V before it: all but the youngest NI copies (compressed pages: all that was widened).  One token group
    // (256 rows): tiles of four blocks.  Of plain pages AHEAD = 3 and the copy goes over block i - 1; since K of block i + 2 is there
    // when step i begins, its first operands are read within step i.  Two groups (128 rows; all of LDS): two tiles of K, three of V.  These,
    // and compressed pages: AHEAD = 2, and the first operands of K of block i + 2 are read behind step i's barrier.
    constexpr bool RING4 = TS == 1 && !F8;
    constexpr int AHEAD = RING4 ? 3 : 2;
    BlockDesc q[AHEAD + 1];           // descriptors of blocks i .. i + AHEAD
    Codes k0, v0, k1, v1;             // (compressed pages: of blocks 0 and 1)
    next_step(q[0]);
    const Source src0 = src;
    if (F8 && src0.codes)         load_codes(k0, src0.k, src0.n);
    else if (!F8 || src0.n > 0)   copy_k(src0, 0);
    // Q comes through LDS as well - over tiles that nothing else needs yet - so
    // that whole rows are fetched; padding rows repeat the last real row.  Placed like K rows, and read like them: B operand, lane's row c32.
    // (Two groups: rows 0 to 63 in the third V tile of the first, the rest in that of the second.)
    const auto q_row = [&](int row) { return TS == 1 ? 4 * TILE + row * (2 * D) : (row >> 6) * GROUP + 4 * TILE + (row & 63) * (2 * D); };
    static_assert(RT * 2 * D <= (TS == 1 ? 4 : TS) * TILE, "Q fits");
    {
        const int r0 = div_g(m0);               // (offsets from the tile's first row: they are 32 bits)
        const T* qb = reinterpret_cast<const T*>(a.q) + ((size_t)(inst.cu_q + r0) * a.Hq + (size_t)kvh * G) * D;
        const uint32_t q0 = dev::lds_address(smem);
#pragma unroll
        for (int i = 0; i < RT / (4 * NW); ++i) {
            const int row = 4 * (wave + NW * i) + lrow, m = min(m0 + row, n_m - 1);
            if (m0 + (4 * (wave + NW * i) & ~(WR - 1)) >= n_m) continue;        // rows of a wave that has none
            const int r = div_g(m), g = m - r * G;
            dev::dma16(qb, (uint32_t)(((r - r0) * a.Hq + g) * (2 * D)) + 16 * (place ^ (row & 15)), q0 + q_row(4 * (wave + NW * i)));
        }
    }
    next_step(q[1]);
    const Source src1 = src;
    const bool both = F8 && TS == 2 && src0.codes && src1.codes;
    if (both) {                                 // (one straight piece, so that K is waited for without the loads behind it; 256-row tiles got 1 to 2 % slower by it)
        load_codes(v0, src0.v, src0.n);
        load_codes(k1, src1.k, src1.n); load_codes(v1, src1.v, src1.n);
        store_codes(k0, k_at(0), false);
    } else if (F8) {
        if (src0.codes)         { load_codes(v0, src0.v, src0.n); store_codes(k0, k_at(0), false); }
        else if (src0.n > 0)    copy_v(src0, 0);
#pragma unroll
        for (int i = 0; i < NC; ++i)            // (K has arrived here too: otherwise all is waited for where the branches meet)
            asm volatile("" :: "v"(k0.w[i].x), "v"(k0.w[i].y), "v"(k0.w[i].z), "v"(k0.w[i].w));
        if (src1.codes)         { load_codes(k1, src1.k, src1.n); load_codes(v1, src1.v, src1.n); }
        else if (src1.n > 0)    { copy_k(src1, 1); copy_v(src1, 1); }
    }
    next_step(q[2]);
    const Source src2 = src;
    // Q and K of block 0 are there (of compressed pages the 3 NC loads behind them may still be on their way)
    if (both) dev::dma_wait<3 * NC>(); else dev::dma_wait<0>();
    lds_barrier();
    bf16x8 bq[8];                     // dims 16 c + 8 g2 ..
    const int vis = div_g(min(wm0 + c32, n_m - 1)) + 1;    // tail rows this lane's row may see
#pragma unroll
    for (int c = 0; c < 8; ++c) bq[c] = *reinterpret_cast<const bf16x8*>(smem + q_row(WR * rw) + (koff ^ (32 * c)));
    if (RING4) { lds_barrier(); next_step(q[AHEAD]); }       // (block 2 comes over Q)
    Source next_src = src;            // where block i + AHEAD lies (compressed pages: its codes wait in registers)
    if (F8 && next_src.codes) { load_codes(kc, next_src.k, next_src.n); load_codes(vc, next_src.v, next_src.n); }

    auto barrier_plain = [&]() {      // every LDS read before it is consumed before the next one
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    const float sc = a.scale_log2e;
    const float lazy_raw = kLazyLog2 / sc;
    // weight = 2^(score scb + nmc): scb the score scale (compressed page: with sk), nmc minus the reference score in its
    // units (compressed page: plus log2 sv)
    float scb = sc, nmc = 0.f, ones_v = 1.0f;       // (ones_v: 1 / sv, so that the factor sv of the weights cancels in their sum)
    // Half h of block d's scores.  masked: the block is ragged, or lies in the tail and reaches past what the wave's first
    // row may see (per-row causal limit); otherwise all rows see all of it
    auto mask = [&](f32x16& st, const BlockDesc& d, int h) {
        if (__builtin_expect(d.ragged, 0)) {            // wave-uniform
            const int limit = min(d.n, vis - d.t0) - 4 * g2 - 32 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i) st[i] = 8 * (i / 4) + i % 4 < limit ? st[i] : kNegBig;
        }
    };
    // The reference score of a row moves only when the maximum of a half exceeds it by
    // more than kLazyLog2 powers of two: weights stay below 2^kLazyLog2, and the
    // accumulators are rescaled on few blocks instead of on most - once the half before, whose weights are
    // formed against the old reference, has been added to them.
    float alpha = 1.f;
    bool moved = false;               // (wave-uniform)
    auto max2 = [](float x, float y) { float m; asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(x), "v"(y)); return m; };     // (fmaxf makes both quiet first)
    float mlim = kNegBig + lazy_raw;  // scores above it move the reference
    auto take_max = [&](float mx, const BlockDesc& d) {
        const u32x2 both = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false));
        mx = max2(__uint_as_float(both.x), __uint_as_float(both.y));
        if (F8) mx = mx > 0.5f * kNegBig ? mx * d.sk : kNegBig;     // into the units of the reference
        const bool moves = mx > mlim;
        moved = __builtin_amdgcn_ballot_w64(moves) != 0;
        if (__builtin_expect(moved, 0)) {
            alpha = moves ? fast_exp2((mrow - mx) * sc) : 1.0f;
            if (moves) { mrow = mx; mlim = mx + lazy_raw; }
            // a row that has seen no key yet keeps the floor as its reference; its masked
            // scores must still come out as weight 0, not 2^0
            if (!F8) nmc = mrow > 0.5f * kNegBig ? -mrow * sc : 0.f;
        }
        if (F8) nmc = (mrow > 0.5f * kNegBig ? -mrow * sc : 0.f) + (__builtin_amdgcn_frexp_expf(d.sv) - 1.0f);
    };
    auto rescale = [&]() {
        if (__builtin_expect(moved, 0)) {
            ol[0] *= alpha;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) ot[t][i] *= alpha;
        }
    };
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    auto pack2 = [&](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2)); };
    // (keeps what is computed here here, among instructions that the compiler would reorder)
    auto pin = [](auto& x) { asm volatile("" : "+v"(x)); };
    constexpr int PD = 4;             // LDS reads ahead of the matrix instructions
    // operand addresses of a step: K of a block by 16 dims, V by 32
    auto read_k1 = [&](int o) { return *reinterpret_cast<const bf16x8*>(smem + o); };
    auto read_v1 = [&](int o) {                 // 16 tokens
        const s16x4 lo = lds_read_tr(smem + o), hi = lds_read_tr(smem + o + 8 * 256);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    const f32x16 zero = {};
    // The row sums come from the matrix cores as well: they add the weights exactly as the output uses
    // them (rounded to bf16).  A column of the 4x4x4 instruction's sixteen blocks is a lane's own four
    // values, so with ones as A each lane gets the sum of its own weights (and a row that is not a number
    // reaches no other).
    auto row_sums = [&](const uint32_t (&pw)[8], float ones_v) {
        const short one = __builtin_bit_cast(short, (__bf16)(F8 ? ones_v : 1.0f));
        const s16x4 ones = {one, one, one, one};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            ol = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, u32x2{pw[2 * u], pw[2 * u + 1]}), ol, 0, 0, 0);
    };

    f32x16 s0, s1;                    // S^T of a block's halves: tokens 8 (i / 4) + 4 g2 + i % 4, + 32
    uint32_t p0[8], p1[8];            // their weights, two to a register
    auto weight_pair = [&](const uint32_t (&p)[8], int u) { return __builtin_bit_cast(bf16x8, u32x4{p[4 * u], p[4 * u + 1], p[4 * u + 2], p[4 * u + 3]}); };
    // The matrix instructions find their first four operands in f, and those of the next eight are left there.
    bf16x8 f[PD];
    // st: scores at hand, sn: next scores (half h of block dn, K at ka), pt: weights at hand, pp: weights before (half h of V at va);
    // K at kn comes next.  between(j): what else is to be done behind the j-th matrix instruction.
    auto period = [&](const f32x16& st, f32x16& sn, uint32_t (&pt)[8], const uint32_t (&pp)[8], const int (&ka)[8], const int (&va)[4],
                      const int (&kn)[8], int kn_off, const BlockDesc& dn, int h, float ones_pp, auto between) {
        bf16x8 g[8 - PD];
        float x = fmaf(st[0], scb, nmc), e[2];
        auto vector_work = [&](int j) {     // one weight; those of the step before are packed
            if (j > 0 && j % 2 == 0) { pt[j / 2 - 1] = pack2(e[0], e[1]); pin(pt[j / 2 - 1]); }
            e[j & 1] = fast_exp2(x); pin(e[j & 1]);
            if (j < 15) { x = fmaf(st[j + 1], scb, nmc); pin(x); }
        };
        auto v_operand = [&](int j) { return read_v1(va[j & 3] + 8192 * h + 4096 * (j >> 2)); };
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j < PD ? f[j] : g[j - PD], bq[j], j ? sn : zero, 0, 0, 0);
            pin(sn);
            if (j < 8 - PD) g[j] = read_k1(ka[j + PD] + 8192 * h); else f[j - (8 - PD)] = v_operand(j - (8 - PD));
            between(j);
            vector_work(j);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(sn, dn, h);
        __builtin_amdgcn_sched_barrier(0);
        float mx = sn[0];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            ot[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j < PD ? f[j] : g[j - PD], weight_pair(pp, j >> 2), ot[j & 3], 0, 0, 0);
            pin(ot[j & 3]);
            if (j < 8 - PD) g[j] = v_operand(j + PD); else f[j - (8 - PD)] = read_k1(kn[j - (8 - PD)] + kn_off);
            between(8 + j);
            mx = j ? fmaxf(fmaxf(mx, sn[2 * j]), sn[2 * j + 1]) : fmaxf(mx, sn[1]);
            pin(mx);
            vector_work(8 + j);
            __builtin_amdgcn_sched_barrier(0);
        }
        pt[7] = pack2(e[0], e[1]);
        row_sums(pp, ones_pp);
        rescale();
        return mx;
    };
    auto weights = [&](const f32x16& st, uint32_t (&p)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) p[j] = pack2(fast_exp2(fmaf(st[2 * j], scb, nmc)), fast_exp2(fmaf(st[2 * j + 1], scb, nmc)));
    };
    auto half_max = [&](const f32x16& st) {
        float mx = st[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, st[i]);
        return mx;
    };
    const int kb = koff + tg * GROUP, vb = voff + tg * GROUP;
    auto k_operands = [&](int (&ka)[8], int d) {
#pragma unroll
        for (int c = 0; c < 8; ++c) { ka[c] = (kb + k_at(d)) ^ (32 * c); pin(ka[c]); }
    };
    auto v_operands = [&](int (&va)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) { va[t] = (vb + v_at(0)) ^ (64 * t); pin(va[t]); }
    };
    // Block 0's scores, first weights and maxima; what else step 0 finds in LDS is copied meanwhile, in the order in which it
    // is needed (the copies ahead of them would hold up the waves for 1.5 us).
    auto first_copies = [&](int i) {
        if (F8) {                                   // (codes: widened beside the second half's scores)
            const int k = i - 8;
            if (k < 0)                               return;
            if (k < NC)                              { if (src0.codes) store_codes1(v0, v_at(0), true, k); }
            else if (k < 2 * NC)                     { if (src1.codes) store_codes1(k1, k_at(1), false, k - NC); }
            else if (k < 3 * NC)                     { if (src1.codes) store_codes1(v1, v_at(1), true, k - 2 * NC); }
            return;
        }
        if (i < NI)                      copy_v1(src0, 0, i);
        else if (i < 2 * NI)             copy_k1(src1, 1, i - NI);
        else if (i < 3 * NI)             copy_v1(src1, 1, i - 2 * NI);
        else if (RING4 && i < 4 * NI)    copy_k1(src2, 2, i - 3 * NI);
        else if (RING4 && i < 5 * NI)    copy_v1(src2, 2, i - 4 * NI);
    };
    static_assert((RING4 ? 5 : 3) * NI <= 16 && 3 * NC <= 8, "a copy behind every matrix instruction at most");
    if (q[0].n > 0) {
        int ka[8];
        k_operands(ka, 0);
        if (F8) { scb = sc * q[0].sk; ones_v = 1.0f / q[0].sv; }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k1(ka[c]), bq[c], c ? s0 : zero, 0, 0, 0);
            pin(s0);
            first_copies(c);
        }
        mask(s0, q[0], 0);
        float mx = s0[0];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k1(ka[c] + 8192), bq[c], c ? s1 : zero, 0, 0, 0);
            pin(s1);
            first_copies(8 + c);
            mx = c ? fmaxf(fmaxf(mx, s0[2 * c]), s0[2 * c + 1]) : fmaxf(mx, s0[1]);
            pin(mx);
        }
        // One reference for the whole block: its weight is exact in bf16, and the largest of 64 is worth more than that of 32
        // (distance from float64 on a 1000-token chunk 2.022e-3 of the norm with one per half, 2.000e-3 so).
        mask(s1, q[0], 1);
        take_max(fmaxf(mx, half_max(s1)), q[0]);
        moved = false;                          // (nothing summed yet)
        weights(s0, p0);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) first_copies(i);
    }
    // all but the youngest block's V is there (compressed pages: and all that was widened), and K of block 0 read by every wave
    if (F8) lds_barrier(); else { dev::dma_wait<NI>(); barrier_plain(); }
    // Step i: descriptors and sources move on by one block
    bool copied = false;
    Source now;
    BlockDesc d, dn;
    auto begin_step = [&]() {
        d = q[0]; dn = q[1];
        copied = false;
        if (F8) {
            if (next_src.codes)         { store_codes(kc, k_at(2), false); store_codes(vc, v_at(2), true); }
            else if (next_src.n > 0)    { copy_k(next_src, 2); copy_v(next_src, 2); copied = true; }
        }
        now = next_src;
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) q[k] = q[k + 1];
        next_step(q[AHEAD]);
        next_src = src;
        if (F8 && next_src.codes) { load_codes(kc, next_src.k, next_src.n); load_codes(vc, next_src.v, next_src.n); }
    };
    auto end_step = [&]() {
        i4 = (i4 + 1) & 3;
        i3 = i3 == 2 ? 0 : i3 + 1;
        if (F8) {
            if (copied) dev::dma_wait<0>();
            lds_barrier();                          // (the widened codes are written)
        } else {
            dev::dma_wait<NI>();
            barrier_plain();
        }
    };
    auto first_operands = [&]() {
#pragma unroll
        for (int c = 0; c < PD; ++c) f[c] = read_k1((kb + k_at(1)) ^ (32 * c));
    };
    first_operands();
    while (q[0].n > 0 && q[1].n > 0) {
        d = q[0]; dn = q[1];
        int ka[8], kn[8], va[4];
        k_operands(ka, 1);
        v_operands(va);
        // (The copies go among the matrix instructions: all at once they would hold up the waves.  Two token groups wait at the
        // end of this very step for the K copied in it, so it goes behind the first ones.  Spread out -> so, us per layer: 1000-token
        // chunks 19.6 -> 19.2 (8B), 27.5 -> 26.9 (70B), twenty-four 16-row questions over 2000 tokens 41.9 -> 40.9.)
        now = next_src;
        auto copies_k = [&](int j) {
            if (F8) return;
            if (TS == 2) { if (j < NI) copy_k1(now, AHEAD, j); }
            else if (j % (16 / NI) == 1) copy_k1(now, AHEAD, j / (16 / NI));
        };
        auto copies_v = [&](int j) { if (!F8 && j % (16 / NI) == 1) copy_v1(now, AHEAD, j / (16 / NI)); };
        const float ones_now = ones_v;
        float mx = period(s1, s0, p1, p0, ka, va, ka, 8192, dn, 0, ones_now, copies_k);
        if (F8) { scb = sc * dn.sk; ones_v = 1.0f / dn.sv; }
        take_max(mx, dn);
        begin_step();
        if (RING4) k_operands(kn, 2);               // (it has landed)
        mx = period(s0, s1, p0, p1, ka, va, RING4 ? kn : ka, 0, dn, 1, ones_now, copies_v);
        take_max(mx, dn);
        end_step();
        if (!RING4) first_operands();
    }
    if (q[0].n > 0) {                               // the wave's last block
        begin_step();
        int va[4];
        v_operands(va);
        bf16x8 g[16];
#pragma unroll
        for (int j = 0; j < PD; ++j) g[j] = read_v1(va[j]);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            ot[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[j], weight_pair(j < 8 ? p0 : p1, (j >> 2) & 1), ot[j & 3], 0, 0, 0);
            pin(ot[j & 3]);
            if (j + PD < 16) g[j + PD] = read_v1(va[j & 3] + 4096 * ((j + PD) >> 2));
            if (j < 8) { p1[j] = pack2(fast_exp2(fmaf(s1[2 * j], scb, nmc)), fast_exp2(fmaf(s1[2 * j + 1], scb, nmc))); pin(p1[j]); }
            __builtin_amdgcn_sched_barrier(0);
            if (j == 7) { row_sums(p0, ones_v); rescale(); }
        }
        row_sums(p1, ones_v);
        if (!F8) { copy_k(now, AHEAD); copy_v(now, AHEAD); }
        end_step();
    }
    while (q[0].n >= 0) {                           // blocks that other waves see
        begin_step();
        if (!F8) { copy_k(now, AHEAD); copy_v(now, AHEAD); }
        end_step();
    }
    dev::dma_wait<0>();                                  // (copies past the end)
    __syncthreads();

    // ---- out ----
    // Of two waves with the same rows (two token groups) each finishes half of the dims: it hands the other half's accumulators, as
    // they lie in its registers, to its partner.  Finished rows - normalised and rounded by the lane that holds them, or as partials -
    // go through LDS, so that they leave as whole rows.  (Folded and divided row by row on their way out they took 3.2 us.)
    constexpr int NT = 4 / TS;                           // 32-dim tiles that a wave finishes
    constexpr int ROWS_AT = TS == 1 ? 0 : NW * 8192 + NW * 256, ML_AT = ROWS_AT + RT * D * 4;
    static_assert(ML_AT + RT * 8 <= sizeof(smem), "rows fit beside what the waves exchange");
    f32x16 o[NT];
    float M = mrow * sc, L = ol[0] + lane_xor(ol[0], 32, lane);
    if constexpr (TS == 1) {
#pragma unroll
        for (int t = 0; t < NT; ++t) o[t] = ot[t];
    } else {
        f32x16 other[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) { o[t] = tg == 0 ? ot[t] : ot[2 + t]; other[t] = tg == 0 ? ot[2 + t] : ot[t]; }
        float2* const ml = reinterpret_cast<float2*>(smem + NW * 8192);
        if (wave_live) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                *reinterpret_cast<f32x4*>(smem + wave * 8192 + (j * 64 + lane) * 16) =
                    f32x4{other[j / 4][4 * (j & 3)], other[j / 4][4 * (j & 3) + 1], other[j / 4][4 * (j & 3) + 2], other[j / 4][4 * (j & 3) + 3]};
            if (g2 == 0) ml[wave * WR + c32] = make_float2(M, L);
        }
        lds_barrier();
        if (wave_live) {
            const int partner = wave ^ (NW / 2);
            const float2 mlp = ml[partner * WR + c32];
            const float mm = fmaxf(M, mlp.x), f0 = fast_exp2(M - mm), f1 = fast_exp2(mlp.x - mm);
            M = mm;
            L = fmaf(f1, mlp.y, L * f0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(smem + partner * 8192 + (j * 64 + lane) * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i) o[j / 4][4 * (j & 3) + i] = fmaf(f1, v[i], o[j / 4][4 * (j & 3) + i] * f0);
            }
        }
    }
    const bool single = unit.n_units_inst == 1, bf16_out = single && !a.out_f32;
    const int rows_here = min(RT, n_m - m0);
    if (wave_live) {
        const int row = WR * rw + c32;
        if (single) {
            const float inv = 1.0f / L;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[t][i] *= inv;
        } else if (g2 == 0 && tg == 0) {
            *reinterpret_cast<float2*>(smem + ML_AT + row * 8) = make_float2(M, L);
        }
        // 16-byte piece p of row r at place p ^ r (bf16 rows of 16 pieces: whose halves change places in rows 16 to 31 of 32)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int tt = TS == 1 ? t : 2 * tg + t;
                if (bf16_out)
                    *reinterpret_cast<uint2*>(smem + ROWS_AT + row * (D * 2) + 16 * ((4 * tt + j) ^ (c32 & 15)) + 8 * (g2 ^ (c32 >> 4))) =
                        make_uint2(pack2(o[t][4 * j], o[t][4 * j + 1]), pack2(o[t][4 * j + 2], o[t][4 * j + 3]));
                else
                    *reinterpret_cast<float4*>(smem + ROWS_AT + row * (D * 4) + 16 * ((8 * tt + 2 * j + g2) ^ c32)) =
                        make_float4(o[t][4 * j], o[t][4 * j + 1], o[t][4 * j + 2], o[t][4 * j + 3]);
            }
    }
    lds_barrier();
    if (bf16_out) {                                      // sixteen lanes take a row
        // Through the L2s: what lies there when the launch ends is written back before the next one starts (chunk passes 394 -> 390 us,
        // 309 -> 306).  Partials, which the fold reads next, stay in them (through: 323 -> 334 us per question pass of one 8B user).
        const int r0 = div_g(m0);                        // (offsets from the tile's first row: they are 32 bits)
        T* const tile_out = reinterpret_cast<T*>(a.out) + (size_t)(inst.cu_q + r0) * a.Hq * D;
        uint4 v[RT / 32];
#pragma unroll
        for (int i = 0; i < RT / 32; ++i) {
            const int row = (tid >> 4) + 32 * i;
            v[i] = *reinterpret_cast<const uint4*>(smem + ROWS_AT + row * (D * 2) + 16 * ((tid ^ row) & 15));
        }
#pragma unroll
        for (int i = 0; i < RT / 32; ++i) {
            const int row = (tid >> 4) + 32 * i, m = m0 + row, r = div_g(m), head = kvh * G + m - r * G;
            if (row >= rows_here) break;
            dev::st_agent4(tile_out, (uint32_t)((r - r0) * a.Hq + head) * (2 * D) + 16 * (tid & 15),
                           row & 16 ? make_uint4(v[i].z, v[i].w, v[i].x, v[i].y) : v[i]);
        }
    } else {                                             // half a wave takes a row
#pragma unroll
        for (int i0 = 0; i0 < RT / 16; i0 += 4) {
            float4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = (tid >> 5) + 16 * (i0 + i);
                v[i] = *reinterpret_cast<const float4*>(smem + ROWS_AT + row * (D * 4) + 16 * ((tid ^ row) & 31));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = (tid >> 5) + 16 * (i0 + i), m = m0 + row, r = div_g(m), head = kvh * G + m - r * G;
                if (row >= rows_here) break;
                if (single) {
                    *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.out) + ((size_t)(inst.cu_q + r) * a.Hq + head) * D + 4 * c32) = v[i];
                } else {
                    float* const prow = a.partials + (((size_t)unit_i * a.rows + r) * a.Hq + head) * kPartialStride(D);
                    *reinterpret_cast<float4*>(prow + 4 * c32) = v[i];
                    if (c32 == 0) *reinterpret_cast<float2*>(prow + D) = *reinterpret_cast<const float2*>(smem + ML_AT + row * 8);
                }
            }
        }
    }
}

// ---- questions of up to 64 (question row, query head) rows per KV head, chunks of up to 512 tokens ----
// A short question's launch is bound by fetching the cache, and the 128-row form above serves it
// badly: its waves compute 32 rows whether they are there or not, its first blocks are a quarter of a unit of a
// few hundred tokens, and a compute unit holds one workgroup.  Here a workgroup of four waves owns 64 rows, 16 per
// wave (16x16x32), all waves walk the same 64-token blocks out of double-buffered LDS tiles, and two workgroups
// share a compute unit.  The next block's loads are in flight in registers meanwhile.  8B shape, one row,
// us per layer with the fold, 128-row form -> this one: four over 3000 tokens 19.0 -> 17.0 (49 MB), one over 10 000
// 18.0 -> 16.6 (41 MB); compressed pages: sixteen 70B users of 4 000 tokens 62.6 -> 55.8, twenty-three 8B users of 4 400 87 -> 73.
// A short chunk's own attention walks few blocks, and the four waves start sooner than eight: 64 tokens 8.0 -> 4.9.
//   S^T = K Q^T     A = K rows from the LDS tile, B = Q held in registers
//   softmax         online, per lane on its own column; the four 16-lane groups agree on the maximum
//   O^T += V^T P^T  A = V through the transposing LDS read, B = P rounded to bf16
// Row strides of the tiles: the ones on which the 16-byte operand reads (K) and the transposing reads (V)
// measured fastest (K 288 bytes 5.4 cycles per instruction against 8.8 at 272; V 304 bytes 6.2 against 6.7 at 288).
constexpr int KSTR = D + 16, VSTR = D + 24;             // bf16 per LDS row of the K and of the V tile

template <bool F8>
__global__ __launch_bounds__(256, 2) void attn_prefill_short_kernel(
        const Unit* __restrict__ units, const InstanceInfo* __restrict__ insts, const Item* __restrict__ items, int chunk,
        KernelArgs a) {
    constexpr int NWV = 4, RT = 16 * NWV, SR = TB / (4 * NWV);
    constexpr int TILE_ELEMS = TB * KSTR + TB * VSTR;   // one K tile + one V tile
    typedef uint16_t T;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    const int G = a.Hq / a.Hkv;
    auto div_g = [&](int m) { return (int)__umulhi((unsigned)m << 3, a.g_mul); };
    const int kvh = blockIdx.y;

    Unit unit;
    InstanceInfo inst;
    int tile = blockIdx.z;
    if (chunk) {                               // the chunk, as above; the longest tiles go first
        unit = Unit{};
        unit.n_items = 1; unit.n_units_inst = 1; unit.has_tail = 1; unit.first.ntok = a.rows;
        inst = InstanceInfo{};
        inst.q_len = a.rows;
        tile = (a.rows * G - 1) / RT - tile;
    } else {
        unit = table_record(units + blockIdx.x);
        inst = table_record(insts + unit.inst);
    }
    const int m0 = tile * RT;
    const int n_m = inst.q_len * G;
    if (m0 >= n_m) return;                              // whole workgroup leaves together
    const bool wave_live = m0 + 16 * wave < n_m;        // this wave has at least one real row
    const int vis_min = div_g(m0 + 16 * wave) + 1;      // tail rows every row of this wave may see

    // Q in operand layout; padding rows repeat the last real row
    bf16x8 bq[4];
    const int mq = min(m0 + 16 * wave + c16, n_m - 1), rq = div_g(mq);
    const int vis = rq + 1;                             // tail rows this lane's row may see
    {
        const T* qp = reinterpret_cast<const T*>(a.q) + ((size_t)(inst.cu_q + rq) * a.Hq + (size_t)kvh * G + (mq - rq * G)) * D + 8 * g4;
#pragma unroll
        for (int c = 0; c < 4; ++c) bq[c] = __builtin_bit_cast(bf16x8, ldg16(qp + 32 * c));
    }

    f32x4 ot[8], ol = f32x4{0.f, 0.f, 0.f, 0.f};        // O^T accumulators; row sum (every element of a lane the same)
    float mrow = kNegBig;                               // reference score of the lane's row, unscaled
#pragma unroll
    for (int s = 0; s < 8; ++s) ot[s] = f32x4{0.f, 0.f, 0.f, 0.f};

    __shared__ __attribute__((aligned(16))) uint16_t tiles[2 * TILE_ELEMS];
    // the unit's item list sits in LDS: a fetch inside the loop would also drain the block loads in flight
    __shared__ __attribute__((aligned(16))) Item sm_items[kMaxPrefillItemsPerUnit];
    __shared__ float sm_scale[F8 ? kMaxPrefillItemsPerUnit : 1][2];      // K and V scale of every item
    if (!chunk)
        for (int i = tid; i < unit.n_items * 2; i += NWV * 64)
            reinterpret_cast<uint4*>(sm_items)[i] = reinterpret_cast<const uint4*>(items + unit.item0)[i];
    if (F8 && tid < unit.n_items) {
        const Item it = items[unit.item0 + tid];
        float sk = 1.f, sv = 1.f;
        if (it.base) page_scales(it, a.layer, a.Hkv, kvh, sk, sv);
        sm_scale[tid][0] = sk; sm_scale[tid][1] = sv;
    }
    __syncthreads();

    // Every wave walks the same blocks: the unit's items end to end (the tail clipped to the rows this tile
    // may see), TB token rows at a time, never across two items.  Past the unit's end the last block comes
    // back marked invalid: still safe to load, so that the loop's loads are unconditional.
    struct { Item item; int item_i, rows, left; } wk;   // current item, its visible rows, rows not yet handed out
    const int tail_visible = min(div_g(min(m0 + RT, n_m) - 1) + 1, a.max_tail);
    auto rows_of = [&](const Item& it) { return it.base ? it.ntok : min(it.ntok, tail_visible); };
    wk.item = unit.first; wk.item_i = 0; wk.rows = rows_of(wk.item); wk.left = wk.rows;
    BlockRef<T> last_block{};
    auto next_block = [&]() {
        BlockRef<T> r = last_block;
        r.valid = false;
        while (wk.left <= 0) {
            if (++wk.item_i >= unit.n_items) return r;
            wk.item = sm_items[wk.item_i];
            wk.rows = rows_of(wk.item);
            wk.left = wk.rows;
        }
        r.is_tail = wk.item.base == 0;
        if (!r.is_tail) {
            const size_t head = (size_t)wk.item.page_tokens * (F8 ? D / 2 : D);     // in units of T
            r.k = reinterpret_cast<const T*>(wk.item.base) + ((size_t)a.layer * 2 * a.Hkv + kvh) * head;
            r.v = r.k + (size_t)a.Hkv * head;
            if (F8) { r.sk = sm_scale[wk.item_i][0]; r.sv = sm_scale[wk.item_i][1]; }
        } else {
            const size_t off = ((size_t)unit.inst * a.Hkv + kvh) * (size_t)a.max_tail * D;
            r.k = reinterpret_cast<const T*>(a.tail_k) + off;
            r.v = reinterpret_cast<const T*>(a.tail_v) + off;
            if (F8) { r.sk = 1.f; r.sv = 1.f; }
        }
        const int n = min(TB, wk.left);
        r.t0 = wk.item.tok0 + (wk.rows - wk.left);
        r.tok_end = r.t0 + n;
        r.valid = true;
        wk.left -= n;
        last_block = r;
        return r;
    };

    // cooperative staging: thread t moves rows t / 16 + 16 i, columns 8 (t % 16), of K and of V; rows past the
    // block's end repeat its last one
    const int st_row = tid >> 4, st_col = (tid & 15) * 8;
    struct Stage { uint4 k[SR], v[SR]; };
    auto load_global = [&](const BlockRef<T>& r, Stage& g) {
        if (F8 && !r.is_tail) {         // codes: the same number of loads, half as wide
#pragma unroll
            for (int i = 0; i < SR; ++i) {
                const size_t off = (size_t)min(r.t0 + st_row + 4 * NWV * i, r.tok_end - 1) * D + st_col;
                const uint2 kw = ldg8(reinterpret_cast<const uint8_t*>(r.k) + off), vw = ldg8(reinterpret_cast<const uint8_t*>(r.v) + off);
                g.k[i] = make_uint4(kw.x, kw.y, 0u, 0u);
                g.v[i] = make_uint4(vw.x, vw.y, 0u, 0u);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            const size_t off = (size_t)min(r.t0 + st_row + 4 * NWV * i, r.tok_end - 1) * D + st_col;
            g.k[i] = ldg16(r.k + off);
            g.v[i] = ldg16(r.v + off);
        }
    };
    auto store_lds = [&](int buf, const Stage& g, bool codes) {
        uint16_t* kt = tiles + buf * TILE_ELEMS;
        uint16_t* vt = kt + TB * KSTR;
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            *reinterpret_cast<uint4*>(kt + (st_row + 4 * NWV * i) * KSTR + st_col) =
                F8 && codes ? e4m3x8_to_bf16x8(make_uint2(g.k[i].x, g.k[i].y)) : g.k[i];
            *reinterpret_cast<uint4*>(vt + (st_row + 4 * NWV * i) * VSTR + st_col) =
                F8 && codes ? e4m3x8_to_bf16x8(make_uint2(g.v[i].x, g.v[i].y)) : g.v[i];
        }
    };

    // Scores, reference scores, masks and the scales of compressed pages as in the kernel above.
    const float sc = a.scale_log2e;
    const float lazy_raw = kLazyLog2 / sc;
    auto compute = [&](const BlockRef<T>& r, int buf) {
        const bool masked = r.tok_end - r.t0 != TB || (r.is_tail && r.tok_end > vis_min);
        const uint16_t* kt = tiles + buf * TILE_ELEMS;
        const uint16_t* vt = kt + TB * KSTR;
        bf16x8 ones;
#pragma unroll
        for (int i = 0; i < 8; ++i) ones[i] = (__bf16)(F8 ? 1.0f / r.sv : 1.0f);
        // S^T in 16-token quarters q: lane holds tokens t0 + 16 q + 4 g4 + i of its row
        f32x4 st[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 ak[2][4];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    ak[hh][c] = *reinterpret_cast<const bf16x8*>(kt + (32 * h + 16 * hh + c16) * KSTR + 32 * c + 8 * g4);
            st[2 * h] = f32x4{0.f, 0.f, 0.f, 0.f};
            st[2 * h + 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
                    st[2 * h + hh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak[hh][c], bq[c], st[2 * h + hh], 0, 0, 0);
        }
        if (masked) {               // wave-uniform
            const int limit = (r.is_tail ? min(r.tok_end, vis) : r.tok_end) - r.t0 - 4 * g4;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) st[q][i] = 16 * q + i < limit ? st[q][i] : kNegBig;
        }
        float mx = st[0][0];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = fmaxf(mx, st[q][i]);
        mx = fmaxf(mx, lane_xor(mx, 16, lane));
        mx = fmaxf(mx, lane_xor(mx, 32, lane));
        if (F8) mx = mx > 0.5f * kNegBig ? mx * r.sk : kNegBig;
        const float scb = F8 ? sc * r.sk : sc;
        const float mn = mx > mrow + lazy_raw ? mx : mrow;
        const float alpha = fast_exp2((mrow - mn) * sc);
        mrow = mn;
        const float nmc = (mn > 0.5f * kNegBig ? -mn * sc : 0.f) + (F8 ? __builtin_amdgcn_frexp_expf(r.sv) - 1.0f : 0.f);
        bf16x8 pb[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 8; ++i) pb[h][i] = (__bf16)fast_exp2(fmaf(st[2 * h + i / 4][i % 4], scb, nmc));
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {           // wave-uniform: some row's reference moved
            ol[0] *= alpha;
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i) ot[s][i] *= alpha;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) ol = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[h], ol, 0, 0, 0);
        // lane (c16, g4) names 4 dims (4 (c16 % 4) ..) of token 4 g4 + c16 / 4 (+ 16 for the second quarter)
        // of a half and receives dim 16 s + c16 of tokens 4 g4 .. 4 g4 + 3: the k order of P
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const char* vp = reinterpret_cast<const char*>(vt + (32 * h + 4 * g4 + (c16 >> 2)) * VSTR + 4 * (c16 & 3));
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const s16x4 lo = lds_read_tr(vp + 32 * s);
                const s16x4 hi = lds_read_tr(vp + 32 * VSTR + 32 * s);
                const bf16x8 av = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                ot[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb[h], ot[s], 0, 0, 0);
            }
        }
    };

    // Loads and LDS stores carry no branch and the loop has one exit at the bottom, so the compiler counts the
    // loads in flight; every load before the loop (Q above all) is waited for once, ahead of it: otherwise each
    // use of Q inside is guarded with a wait that would also drain the block just requested.
    BlockRef<T> r0 = next_block();
    if (r0.valid) {
        Stage g;
        load_global(r0, g);
        store_lds(0, g, !r0.is_tail);
        __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0) only
        lds_barrier();
        int buf = 0;
        do {
            const BlockRef<T> r1 = next_block();
            load_global(r1, g);
            if (wave_live) compute(r0, buf);
            store_lds(buf ^ 1, g, !r1.is_tail);
            lds_barrier();
            r0 = r1;
            buf ^= 1;
        } while (r0.valid);
    }

    // a wave owns its rows: lane (c16, g4) holds dims 16 s + 4 g4 .. + 3 of row c16
    const int m = m0 + 16 * wave + c16;
    if (m >= n_m) return;
    const int r = div_g(m), head = kvh * G + m - r * G;
    if (unit.n_units_inst == 1) {
        const float inv = 1.0f / ol[0];
        const size_t oidx = ((size_t)(inst.cu_q + r) * a.Hq + head) * D + 4 * g4;
#pragma unroll
        for (int s = 0; s < 8; ++s)
            store_out4(a.out, a.out_f32, oidx + 16 * s, make_float4(ot[s][0] * inv, ot[s][1] * inv, ot[s][2] * inv, ot[s][3] * inv));
    } else {
        float* prow = a.partials + (((size_t)blockIdx.x * a.rows + r) * a.Hq + head) * kPartialStride(D);
#pragma unroll
        for (int s = 0; s < 8; ++s)
            *reinterpret_cast<float4*>(prow + 16 * s + 4 * g4) = make_float4(ot[s][0], ot[s][1], ot[s][2], ot[s][3]);
        if (g4 == 0) *reinterpret_cast<float2*>(prow + D) = make_float2(mrow * sc, ol[0]);
    }
}

// Folds the units' partials of every (question row, query head) of instances cut into several
// units: out = sum_u 2^(m_u - M) acc_u / sum_u 2^(m_u - M) l_u,  M = max_u m_u.
// Half a wave owns one row: lane k first fetches (m, l) of unit k, the half wave agrees on M
// and on every unit's weight, then each lane accumulates its 4 dims over the units.
// NU: units requested per round (the smallest of 2, 4, 8, 16 that covers the launch's largest
// instance: rounds beyond an instance's units would only re-read its last partial).
template <int NU>
__global__ __launch_bounds__(256) void prefill_merge_kernel(
        KernelArgs a, const InstanceInfo* __restrict__ insts, int batch, int total_pairs) {
    constexpr int PS = kPartialStride(D);
    const int lane = threadIdx.x & 63, hl = lane & 31;
    const int pair = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 2 + (lane >> 5);
    const bool in_range = pair < total_pairs;
    const int q_row = in_range ? pair / a.Hq : 0, head = in_range ? pair % a.Hq : 0;
    int b = 0;
    for (int i = 1; i < batch; ++i) if (q_row >= insts[i].cu_q) b = i;
    const InstanceInfo inst = insts[b];
    const int n_units = (in_range && inst.n_punits > 1) ? inst.n_punits : 0;     // 0: nothing to do
    const float* base = a.partials + (((size_t)inst.punit0 * a.rows + (q_row - inst.cu_q)) * a.Hq + head) * PS;
    const size_t ustride = (size_t)a.rows * a.Hq * PS;

    // the first NU units' accumulators are requested together with the (m, l) pairs, before
    // anything is consumed: one memory round trip for up to NU units, two for up to 2 NU
    auto load16 = [&](int u0, float4 (&v)[NU]) {
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const int u = min(u0 + k, max(n_units, 1) - 1);
            v[k] = *reinterpret_cast<const float4*>(base + (size_t)u * ustride + 4 * hl);
        }
    };
    float2 ml = make_float2(kNegBig, 0.f);
    if (hl < n_units) ml = *reinterpret_cast<const float2*>(base + (size_t)hl * ustride + D);
    float4 v[NU];
    load16(0, v);
    float M = ml.x;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float w = hl < n_units ? fast_exp2(ml.x - M) : 0.f;
    float L = w * ml.y;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) L += __shfl_xor(L, off);

    // both halves of the wave run the same number of steps (shuffles need every lane)
    const int steps = max(n_units, __shfl_xor(n_units, 32));
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int u0 = 0; u0 < steps; u0 += NU) {
        if (u0 > 0) load16(u0, v);
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const float c = __shfl(w, (lane & 32) + ((u0 + k) & 31));
            const float cc = (u0 + k < n_units) ? c : 0.f;
            acc.x = fmaf(v[k].x, cc, acc.x); acc.y = fmaf(v[k].y, cc, acc.y);
            acc.z = fmaf(v[k].z, cc, acc.z); acc.w = fmaf(v[k].w, cc, acc.w);
        }
    }
    if (n_units == 0) return;
    const float inv = 1.0f / L;
    const size_t oidx = ((size_t)q_row * a.Hq + head) * D + 4 * hl;
    store_out4(a.out, a.out_f32, oidx, make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv));
}

template <bool F8>
hipError_t launch_f(const AttnArgs& a, hipStream_t s) {
    const KernelArgs k = make_kernel_args(a);
    const int tiles = (a.rows * (a.Hq / a.Hkv) + a.tile_rows - 1) / a.tile_rows;
    const dim3 grid(a.n_units, a.Hkv, tiles), block(a.tile_rows <= 64 ? 256 : NW * 64);
    const InstanceInfo* insts = reinterpret_cast<const InstanceInfo*>(a.table + a.off_inst);
    const Item* items = reinterpret_cast<const Item*>(a.table + a.off_items);
    const Unit* units = reinterpret_cast<const Unit*>(a.table + a.off_units);
    const int chunk = a.prefill == 2;
    if (a.tile_rows <= 64)       hipLaunchKernelGGL(attn_prefill_short_kernel<F8>, grid, block, 0, s, units, insts, items, chunk, k);
    else if (a.deal_tiles) {
        if (a.tile_rows <= 128)  hipLaunchKernelGGL((attn_prefill_kernel<4, F8, int>), grid, block, 0, s, units, insts, items, chunk, k, a.batch);
        else                     hipLaunchKernelGGL((attn_prefill_kernel<8, F8, int>), grid, block, 0, s, units, insts, items, chunk, k, a.batch);
    }
    else if (a.tile_rows <= 128) hipLaunchKernelGGL((attn_prefill_kernel<4, F8>), grid, block, 0, s, units, insts, items, chunk, k);
    else                         hipLaunchKernelGGL((attn_prefill_kernel<8, F8>), grid, block, 0, s, units, insts, items, chunk, k);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.max_units_inst <= 1) return e;
    const int total_pairs = a.total_q * a.Hq;
    const dim3 mgrid((total_pairs + 7) / 8), mblock(256);
    if (a.max_units_inst <= 2)      hipLaunchKernelGGL(prefill_merge_kernel<2>, mgrid, mblock, 0, s, k, insts, a.batch, total_pairs);
    else if (a.max_units_inst <= 4) hipLaunchKernelGGL(prefill_merge_kernel<4>, mgrid, mblock, 0, s, k, insts, a.batch, total_pairs);
    else if (a.max_units_inst <= 8) hipLaunchKernelGGL(prefill_merge_kernel<8>, mgrid, mblock, 0, s, k, insts, a.batch, total_pairs);
    else                            hipLaunchKernelGGL(prefill_merge_kernel<16>, mgrid, mblock, 0, s, k, insts, a.batch, total_pairs);
    return hipGetLastError();
}

}  // namespace

bool attn_prefill_supported(const AttnArgs& a, int dtype) {
    const int g = a.Hq / a.Hkv;
    return a.prefill && dtype == MATKV_BF16 && a.D == 128 && group_size_built(g) && a.row_tiles;
}

hipError_t launch_attn_prefill(const AttnArgs& a, int dtype, hipStream_t s) {
    if (a.n_units <= 0) return hipSuccess;
    if (!attn_prefill_supported(a, dtype)) return hipErrorInvalidValue;
    return a.kv_fmt == MATKV_PAGE_E4M3 ? launch_f<true>(a, s) : launch_f<false>(a, s);
}

}  // namespace matkv
