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
__device__ __forceinline__ void rope_cs(const RopeEntry& e, float p, float& c, float& s) {
    // no contraction here: were p * turns_hi - rint(t) fused into one multiply-add, the product
    // would enter exactly and the rounding error of t, added back below, would count twice
    // (half an ulp of t: 1e-4 turns at position 20 000)
#pragma clang fp contract(off)
    const float t = p * e.turns_hi;
    const float err = fmaf(p, e.turns_hi, -t);
    float fr = t - rintf(t);
    fr += fmaf(p, e.turns_lo, err);
    c = __builtin_amdgcn_cosf(fr);
    s = __builtin_amdgcn_sinf(fr);
}

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
//  - half a step is multiplied while the operands of the next half are on their way from LDS.
//  - finished tiles leave through LDS as whole 256-byte rows.
// Two workgroups that share a tile (SK = 2) leave their fp32 partials in the workspace (agent-scope
// stores), arrive at the tile's counter, and the second to arrive adds the other's and finishes.
// Measured, us per launch with every layer's weights from HBM, 8 KV heads, before -> now:
//   hidden 4096:  256 rows 21.9 -> 17.3, 512 rows 32.3 -> 21.4, 1000 rows 34.5 -> 28.5, 1206 rows
//                 45.6 -> 33.5, 2048 rows 48.5 -> 42.3, 3501 rows 83 -> 62, 8192 rows 168 -> 133
//   hidden 8192:  512 rows 62.6 -> 36.3, 1000 rows 53 -> 48, 2048 rows 83 -> 72, 4096 rows 156 -> 121
// Tried and left out: starting every workgroup at another hidden column (no channel of the L2s is
// favoured by the power-of-two row strides: no change), an extra wave that touches the weight rows
// some steps ahead (-12 % at 512 rows of hidden 8192, +20 % at 64 rows, nothing at 1000).
template <int MI> struct TileShape {
    static constexpr int BM = 32 * MI;                              // token rows of a workgroup
    static constexpr int ROWS = BM + D;                             // LDS rows of a step: tokens, then weight rows
    static constexpr int STEP_BYTES = ROWS * BK * 2;
    static constexpr int NBUF = 158 * 1024 / STEP_BYTES;            // steps that fit in LDS
};

// WN: waves along the features; the other 8 / WN split the rows.  Few waves along the features read
// fewer LDS bytes per product from MI = 8 on (68 -> 64 us at 3501 rows), where LDS becomes the limit.
template <int MI, int WN, int SK>
__global__ __launch_bounds__(512) void materialize_tile_kernel(MaterializeArgs a, int total_rows, int row_tiles) {
    typedef TileShape<MI> S;
    constexpr int WM = 8 / WN, XB = 2 * MI / WM, PB = 4 / WN;       // waves along the rows; row blocks and pair blocks of a wave
    constexpr int BM = S::BM, NBUF = S::NBUF, OSTR = D + 8;         // OSTR: bf16 per LDS row of the finished tile
    static_assert(BM * OSTR * 2 + BM * (int)sizeof(RowDest) <= NBUF * S::STEP_BYTES, "epilogue fits over the dead buffers");
    __shared__ __attribute__((aligned(16))) char smem[NBUF * S::STEP_BYTES];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c16 = lane & 15, g4 = lane >> 4;
    // Workgroup -> (half of the hidden axis, column tile, row tile).  Workgroups go to the eight XCDs in
    // turn; an XCD's L2 should see few distinct operands: with SK = 2 an XCD holds one half of the hidden
    // axis and every fourth column tile, with SK = 1 every fourth column tile and every second row tile.
    const int nct = 2 * a.Hkv;
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
    const int kv = ct / a.Hkv, head = ct % a.Hkv;
    const int row0 = rt * BM;
    const int nk = a.Hd / (BK * SK);

    // Copies of a step: 8 rows x 128 bytes per instruction; token rows are instructions 0 .. 4 MI - 1,
    // wave w takes w, w + 8, ...; of the 16 weight instructions every wave takes two.  LDS row r holds
    // its eight 16-byte pieces permuted: piece g sits at place g ^ ((r >> 1) & 7).
    constexpr int XI = 4 * MI, XW = (XI + 7) / 8;
    const int n_x = (XI - wave + 7) / 8;                            // token copies of this wave per step (XW or XW - 1)
    const int lrow = lane >> 3, place = lane & 7;
    const size_t row_bytes = (size_t)a.Hd * 2;
    const char* X = reinterpret_cast<const char*>(a.hidden) + (size_t)row0 * row_bytes + (size_t)part * nk * (BK * 2);
    const char* W = reinterpret_cast<const char*>(kv == 0 ? a.w_k : a.w_v) + (size_t)head * D * row_bytes + (size_t)part * nk * (BK * 2);
    uint32_t xoff[XW], woff[2];
#pragma unroll
    for (int i = 0; i < XW; ++i) {
        const int r = (wave + 8 * i) * 8 + lrow;
        xoff[i] = (uint32_t)(min(r, total_rows - 1 - row0) * row_bytes) + 16 * (place ^ ((r >> 1) & 7));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (wave + 8 * i) * 8 + lrow;
        woff[i] = (uint32_t)(r * row_bytes) + 16 * (place ^ ((r >> 1) & 7));
    }
    const uint32_t lds0 = dev::lds_address(smem);
    auto copy_step = [&](int ks, int buf) {
        const uint32_t base = lds0 + buf * S::STEP_BYTES + wave * 1024;
        const size_t k = (size_t)ks * (BK * 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) dev::dma16(W + k, woff[i], base + BM * BK * 2 + i * 8192);
#pragma unroll
        for (int i = 0; i < XW; ++i) if (XI % 8 == 0 || i < n_x) dev::dma16(X + k, xoff[i], base + i * 8192);
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
    auto read = [&](Frags& f, int buf, int k2) {
        const int off = buf * S::STEP_BYTES + 16 * ((4 * k2 + g4) ^ sw);
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            f.b[p] = *reinterpret_cast<const bf16x8*>(Bt + p * 2048 + off);
            f.b[PB + p] = *reinterpret_cast<const bf16x8*>(Bt + 64 * 128 + p * 2048 + off);
        }
#pragma unroll
        for (int mi = 0; mi < XB; ++mi) f.x[mi] = *reinterpret_cast<const bf16x8*>(At + mi * 2048 + off);
    };
    auto multiply = [&](const Frags& f) {
#pragma unroll
        for (int mi = 0; mi < XB; ++mi)
#pragma unroll
            for (int p = 0; p < 2 * PB; ++p)
                acc[mi][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.x[mi], f.b[p], acc[mi][p], 0, 0, 0);
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
    const RowDest my_dest = resolve_row(a, row0 + min(tid, BM - 1));      // (while they are on their way)
    if (ahead == NBUF) wait_steps(std::integral_constant<int, NBUF - 1>{}); else dev::dma_wait<0>();
    lds_barrier();
    Frags f0, f1;
    read(f0, 0, 0);
    int buf = 0, ks = 0;
    for (; ks < nk - NBUF; ++ks) {
        read(f1, buf, 1);
        multiply(f0);
        wait_steps(std::integral_constant<int, NBUF - 2>{});
        lds_barrier();
        const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
        read(f0, nbuf, 0);
        copy_step(ks + NBUF, buf);
        multiply(f1);
        buf = nbuf;
    }
    for (; ks < nk; ++ks) {                                         // nothing more to ask for
        read(f1, buf, 1);
        multiply(f0);
        dev::dma_wait<0>();
        lds_barrier();
        buf = buf + 1 == NBUF ? 0 : buf + 1;
        read(f0, buf, 0);                                           // (past the end: not used)
        multiply(f1);
    }
    __syncthreads();                                                // the buffers are dead

    if constexpr (SK == 2) {
        const int tile = rt * nct + ct;
        int* const sm_last = reinterpret_cast<int*>(smem);
        // a tile's accumulators as runs of 512 bytes: 8 bytes per lane and store
        constexpr int NP2 = XB * 4 * PB;
        float* mine = a.ws_partials + ((size_t)(tile * SK + part) * 8 + wave) * (BM * 16) + lane * 2;
#pragma unroll
        for (int i = 0; i < NP2; ++i) {
            const f32x4& v = acc[i / (4 * PB)][i / 2 % (2 * PB)];
            dev::st_agent2(mine + i * 128, v[2 * (i & 1)], v[2 * (i & 1) + 1]);
        }
        int32_t* counter = a.ws_counters + (size_t)tile * kDecodeCounterStride;
        if (!dev::arrive_at(counter, SK, sm_last)) return;
        dev::reset_counter_at(counter);
        const float* theirs = a.ws_partials + ((size_t)(tile * SK + (part ^ 1)) * 8 + wave) * (BM * 16) + lane * 2;
        float2 o[NP2];
#pragma unroll
        for (int i = 0; i < NP2; ++i) o[i] = dev::ld_agent2(theirs + i * 128);
#pragma unroll
        for (int i = 0; i < NP2; ++i) {
            f32x4& v = acc[i / (4 * PB)][i / 2 % (2 * PB)];
            v[2 * (i & 1)] += o[i].x; v[2 * (i & 1) + 1] += o[i].y;
        }
        __syncthreads();
    }

    // epilogue: lane holds tokens 16 (XB wm + mi) + 4 g4 + i, features 16 (PB wn + p) + c16 and 64 further
    uint16_t* const ot = reinterpret_cast<uint16_t*>(smem);
    RowDest* const sm_dest = reinterpret_cast<RowDest*>(smem + BM * OSTR * 2);
    if (tid < BM) sm_dest[tid] = my_dest;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int j = 16 * (PB * wn + p) + c16;
        const RopeEntry re = a.rope[j];
#pragma unroll
        for (int mi = 0; mi < XB; ++mi)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * (XB * wm + mi) + 4 * g4 + i;
                float lo = acc[mi][p][i], hi = acc[mi][PB + p][i];
                if (kv == 0) {
                    float c, s;
                    rope_cs(re, sm_dest[r].pos, c, s);
                    const float k0 = lo * c - hi * s;
                    const float k1 = lo * s + hi * c;
                    lo = k0; hi = k1;
                }
                ot[r * OSTR + j] = f32_to_bf16_rne(lo);
                ot[r * OSTR + j + 64] = f32_to_bf16_rne(hi);
            }
    }
    __syncthreads();
    // whole rows out: sixteen lanes write one row of 256 bytes
    uint16_t* out = reinterpret_cast<uint16_t*>(kv == 0 ? a.k_out : a.v_out) + (size_t)head * a.token_stride * D;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int r = 32 * i + (tid >> 4), c = 8 * (tid & 15);
        const RowDest d = sm_dest[r];
        if (d.valid) *reinterpret_cast<uint4*>(out + d.elem_off + c) = *reinterpret_cast<const uint4*>(ot + r * OSTR + c);
    }
}

template <int MI, int WN, int SK>
hipError_t launch_tile(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    const int row_tiles = (total_rows + 32 * MI - 1) / (32 * MI), nct = 2 * a.Hkv;
    const int grid_tiles = SK == 1 && nct % 4 == 0 ? (row_tiles + 1) / 2 * 2 : row_tiles;
    hipLaunchKernelGGL((materialize_tile_kernel<MI, WN, SK>), dim3(nct * grid_tiles * SK), dim3(512), 0, s, a, total_rows, row_tiles);
    return hipGetLastError();
}

// Tile height.  One workgroup fills a compute unit's LDS, a launch is as long as its slowest
// compute unit, and a workgroup's time grows slower than its height (hidden 4096, us: two workgroups
// per tile of 32 / 64 / 96 / 128 rows 17 / 21 / 24 / 28, one per tile of 96 / 128 / 192 / 256 rows
// 33 / 38 / 47 / 57): so the smallest height that gives no compute unit two workgroups, hidden axis
// halved while that holds; beyond one full round the height with the smallest rounds x (4 + MI), which
// is what those times follow (6000 rows: 192-row tiles 103 us, 128 rows 119, 256 rows 117).
hipError_t launch_tiled(const MaterializeArgs& a, int total_rows, hipStream_t s) {
    const int nct = 2 * a.Hkv;
    auto groups = [&](int mi) { return nct * ((total_rows + 32 * mi - 1) / (32 * mi)); };
    auto halved = [&](int mi) {
        const int64_t tiles = groups(mi);
        return (a.Hd % (2 * BK)) == 0 && tiles * 2 <= 256 && a.ws_partials && tiles * 2 * (32 * mi) * D <= a.ws_partial_floats &&
               tiles * kDecodeCounterStride <= a.ws_n_counters;
    };
    if (halved(1)) return launch_tile<1, 4, 2>(a, total_rows, s);
    if (halved(2)) return launch_tile<2, 4, 2>(a, total_rows, s);
    if (halved(3)) return launch_tile<3, 4, 2>(a, total_rows, s);
    if (halved(4)) return launch_tile<4, 4, 2>(a, total_rows, s);
    int best = 3;
    long best_cost = -1;
    for (int mi : {3, 4, 6, 8}) {
        const long cost = (long)((groups(mi) + 255) / 256) * (4 + mi);
        if (best_cost < 0 || cost < best_cost) { best = mi; best_cost = cost; }
    }
    switch (best) {
        case 3: return launch_tile<3, 4, 1>(a, total_rows, s);
        case 4: return launch_tile<4, 4, 1>(a, total_rows, s);
        case 6: return launch_tile<6, 4, 1>(a, total_rows, s);
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
__global__ __launch_bounds__(512) void materialize_skinny_staged_kernel(MaterializeArgs a, int total_rows) {
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
    const int pg = blockIdx.x & 3, head = (blockIdx.x >> 2) % a.Hkv, kv = (blockIdx.x >> 2) / a.Hkv;
    const int row0 = blockIdx.y * TM;
    const int kslice = a.Hd / NWV;                      // a multiple of SC (checked by the launcher)
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
    const uint16_t* wbase = reinterpret_cast<const uint16_t*>(kv == 0 ? a.w_k : a.w_v) + ((size_t)head * D + 16 * pg + lr) * a.Hd + col0;
    const uint16_t* xp[MI * 4];
#pragma unroll
    for (int i = 0; i < MI * 4; ++i)
        xp[i] = reinterpret_cast<const uint16_t*>(a.hidden) + (size_t)min(row0 + 4 * i + lr, total_rows - 1) * a.Hd + col0;
    auto load = [&](uint4 (&b)[NL], int r) {
        const int off = min(r, n_rounds - 1) * SC;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b[i] = ldg16(wbase + (size_t)(4 * i) * a.Hd + off);
            b[4 + i] = ldg16(wbase + (size_t)(D / 2 + 4 * i) * a.Hd + off);
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
__global__ __launch_bounds__(512) void materialize_fewrows_kernel(MaterializeArgs a, int total_rows) {
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
    const int pg = blockIdx.x % GPH, head = (blockIdx.x / GPH) % a.Hkv, kv = (blockIdx.x / GPH) / a.Hkv;
    const int row0 = blockIdx.y * TMR;
    const int kslice = a.Hd / NWV;                      // a multiple of SC (checked by the launcher)
    const int n_rounds = kslice / SC;

    // the epilogue's row and rotary entry of this thread are fixed: asked for now, not after the sums
    const int et = tid / NP, ep = tid % NP;
    const RopeEntry rope_e = a.rope[NP * pg + ep];
    RowDest edest = resolve_row(a, row0 + min(et, TMR - 1));
    if (et >= TMR) edest.valid = false;

    // load i of a round: staged row 4 i + lane / 16, 16 bytes at column 8 (lane % 16)
    const int lr = lane >> 4, lc = 8 * (lane & 15);
    const size_t col0 = (size_t)wave * kslice + lc;
    const uint16_t* wbase = reinterpret_cast<const uint16_t*>(kv == 0 ? a.w_k : a.w_v) + ((size_t)head * D + NP * pg + lr) * a.Hd + col0;
    const uint16_t* xp[TMR / 4];
#pragma unroll
    for (int i = 0; i < TMR / 4; ++i)
        xp[i] = reinterpret_cast<const uint16_t*>(a.hidden) + (size_t)min(row0 + 4 * i + lr, total_rows - 1) * a.Hd + col0;
    auto load = [&](uint4 (&b)[NL], int r) {
        const int off = min(r, n_rounds - 1) * SC;
#pragma unroll
        for (int i = 0; i < NP / 4; ++i) {
            b[i] = ldg16(wbase + (size_t)(4 * i) * a.Hd + off);
            b[NP / 4 + i] = ldg16(wbase + (size_t)(D / 2 + 4 * i) * a.Hd + off);
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
    if (rounds % 4 == 0) hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 4>), grid, block, 0, s, a, total_rows);
    else if (rounds % 2 == 0) hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 2>), grid, block, 0, s, a, total_rows);
    else hipLaunchKernelGGL((materialize_fewrows_kernel<NP, TMR, 1>), grid, block, 0, s, a, total_rows);
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
        if (mi2) hipLaunchKernelGGL((materialize_skinny_staged_kernel<2, 2>), grid, block, 0, s, a, total_rows);
        else     hipLaunchKernelGGL((materialize_skinny_staged_kernel<1, 2>), grid, block, 0, s, a, total_rows);
    } else {
        if (mi2) hipLaunchKernelGGL((materialize_skinny_staged_kernel<2, 1>), grid, block, 0, s, a, total_rows);
        else     hipLaunchKernelGGL((materialize_skinny_staged_kernel<1, 1>), grid, block, 0, s, a, total_rows);
    }
    return hipGetLastError();
}

}  // namespace matkv
