// C-ABI of libmatkv: argument validation, host bookkeeping (tickets, slot states, cache
// tables, captured graphs) and the enqueue of copies and kernels.  See include/matkv.h for
// the contract of every entry point.
#include <dlfcn.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <errno.h>
#include <unistd.h>

#include <algorithm>
#include <climits>
#include <atomic>
#include <condition_variable>
#include <functional>
#include <list>
#include <mutex>
#include <exception>
#include <new>
#include <numeric>
#include <queue>
#include <thread>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "matkv_internal.h"

using namespace matkv;

namespace {

constexpr int kTicketRing = 4096;
constexpr int kStagingRing = 4;
constexpr int kReleaseRing = 8;                // events marking "work on a table's old contents is enqueued"
constexpr int kBounceRing = 6;                 // pinned pieces between a file and the load stream
constexpr size_t kBounceBytes = 8u << 20;

struct Ticket {
    hipEvent_t ev = nullptr;
    uint64_t id = 0;          // 0 = never used
    void* slot = nullptr;
    bool done = true;         // observed complete
    // loads from a file: the event is recorded by a reader thread once the last piece's copy is on
    // the load stream.  Guarded by the context's io mutex.
    bool queued = false;      // pieces still to be read or enqueued: the event is not recorded yet
    bool failed = false;      // a read failed (the reason is in io_err)
};

struct SlotState {
    uint64_t pending = 0;     // ticket id of the last load into the slot (0 = none)
    bool waited = true;       // compute stream has been ordered after that load
    int refs = 0;             // live cache tables that point into it
    hipEvent_t release = nullptr;   // recorded on the compute stream when its last table let go of it
};

// How the question prefill of a table is laid out.
struct PrefillLayout {
    int tile_rows = 0;        // rows of a workgroup's tile: 64, 128 or 256
    bool deal_tiles = false;  // workgroups without work (questions of fewer tiles than the longest) are left to the launch's end
    bool row_tiles = true;    // the prefill runs on the row-tile kernels (where the shape has them)
    int n_units = 0, max_units_inst = 0, max_unit_items = 0;    // units; most of any one instance, most items of any one unit
};

struct TableHost {
    int batch = 0, n_items = 0, n_dunits = 0, total_q = 0, max_q = 0;
    PrefillLayout prefill;
    int kv_fmt = 0;           // matkv_page_format of its pages
    int n_sunits = 0;         // units of the shared decode partition; 0 = the batch shares no page
    bool even = false;        // decode launches take the even partition, whose units lie behind the others in the table
    uint64_t sig_decode = 0, sig_prefill = 0;   // of what a recorded decode / prefill launch bakes in
    int max_tail_len = 0;     // largest tail_len of any instance (host mirror)
    int min_tail_len = 0;
    int n_decode_slots = 0;   // partial slots a decode launch writes (units, or (unit, user) pairs when shared)
    bool step_by_instance = false;      // a fused decode step reads every instance's cache for itself, beside a shared partition
    bool tail_spared = false; // compressed pages: some unit by instance that has a tail has fewer page tokens than the others
    bool past_llc = false, step_past_llc = false;   // decode launches, fused steps leave the cache's rows out of the last-level cache (rows_pass_llc)
    std::vector<const void*> slots;   // distinct slots its pages point into
};

struct Staging {
    char* host = nullptr;     // pinned
    char* host_on_device = nullptr;     // where kernels see it
    hipEvent_t ev = nullptr;
    bool used = false;
};

}  // namespace

// Scratch of matkv_decode_attn_static (the decode attention for callers that cannot allocate or
// pass a workspace): arrival counters, 128 bytes apart, then the units' partial results.  Every
// device the library runs on holds its own copy until the process ends.
constexpr size_t kStaticCounterBytes = 1u << 20;    // 8192 (instance, KV head) pairs
constexpr size_t kStaticPartialBytes = 7u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticCounterBytes + kStaticPartialBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device`, which must be the current device.  In host code the
// array's name is only a handle; the address comes from the runtime, once per device.
hipError_t scratch_address(int device, char** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = static_cast<char*>(p);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

// A table's filled sections: byte offsets and sizes, multiples of 16.
constexpr int kTableSections = 5;
struct TableSections { size_t off[kTableSections], bytes[kTableSections]; };
static_assert(sizeof(TableHeader) % 16 == 0 && sizeof(InstanceInfo) % 16 == 0 && sizeof(Item) % 16 == 0 && sizeof(Unit) % 16 == 0 &&
              sizeof(SUnit) % 16 == 0, "sections of whole 16-byte pieces");

// The sections from pinned host memory to the device table in one launch.  Copied one by one, each of the four or five ran as a launch
// of its own of about 4 us, with a gap behind it.  us per pass before -> after: question of one 8B user 320 -> 315, of sixteen 706 -> 700, the others 3 to 5 less.
// System scope: the staging buffer is written again by the host, nothing of it may be found in a cache.
__global__ __launch_bounds__(256) void table_copy_kernel(const char* src, char* dst, TableSections sec) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kTableSections; ++k) {
        const size_t n = sec.bytes[k] / 16;
        if (i < n) {
            const uint64_t* from = reinterpret_cast<const uint64_t*>(src + sec.off[k]) + 2 * i;
            uint64_t* to = reinterpret_cast<uint64_t*>(dst + sec.off[k]) + 2 * i;
            const uint64_t a = __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            const uint64_t b = __hip_atomic_load(from + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            to[0] = a; to[1] = b;
            return;
        }
        i -= n;
    }
}

__global__ void zero_ints_kernel(int32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

struct matkv_graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    std::vector<std::pair<void*, int>> advances;   // (table, n) recorded during capture
    struct TableUse { const void* table; bool decode, prefill; uint64_t sig_decode, sig_prefill; };
    std::vector<TableUse> tables;                  // every table the recording reads, with its partition signatures
    std::vector<hipKernelNodeParams> chain;        // the recording as kernel launches in order (empty: replayed as a graph)
};

struct matkv_ctx {
    matkv_config cfg;
    int device = 0;
    hipStream_t compute = nullptr, load = nullptr;
    char* workspace = nullptr;
    char* static_scratch = nullptr;           // this device's copy of `scratch`
    WorkspaceLayout wl;
    TableLayout tl;
    float scale_log2e = 0.f;
    char err[512];
    bool sticky_hip = false;
    uint64_t next_ticket = 1;
    std::vector<Ticket> tickets;
    std::unordered_map<const void*, SlotState> slots;
    std::unordered_map<const void*, TableHost> tables;
    Staging staging[kStagingRing];
    int staging_next = 0;
    Staging bounce[kBounceRing];              // allocated at the first matkv_load_file / matkv_store_file
    int bounce_next = 0;
    char* plain_buf = nullptr;                // matkv_store_file: direct writes that cannot come from pinned memory
    std::atomic<bool> read_via_plain{false};  // direct I/O cannot target the pinned buffers on this system
    // file loads: requests wait in a queue, reader threads take them piece by piece
    struct FileReq {
        int fd; uint64_t offset; size_t bytes; char* dst; Ticket* ticket;
        size_t n_pieces, next_piece, pieces_done;
    };
    std::mutex io_mu;
    std::condition_variable io_work, io_done;
    std::list<FileReq> io_queue;              // front = the oldest request (a list: readers keep pointers into it)
    std::vector<std::thread> io_readers;
    bool io_stop = false;
    char io_err[256] = {0};                   // reason of the last failed read
    hipEvent_t fence_ev = nullptr;
    hipEvent_t release_ev[kReleaseRing] = {};
    int release_next = 0;
    bool capturing = false;
    int chunk_table_tokens = -1;   // chunk length the workspace's one-instance table was last written for (-1: unknown)
    matkv_graph* cap = nullptr;
    std::vector<matkv_graph*> graphs;
};

namespace {

matkv_status fail(matkv_ctx* c, matkv_status s, const char* fmt, ...) {
    if (c) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(c->err, sizeof(c->err), fmt, ap);
        va_end(ap);
    }
    return s;
}

matkv_status hip_fail(matkv_ctx* c, hipError_t e, const char* what) {
    (void)hipGetLastError();
    if (c) {
        c->sticky_hip = true;
        snprintf(c->err, sizeof(c->err), "%s: %s", what, hipGetErrorString(e));
    }
    return MATKV_EHIP;
}

#define HIP_TRY(ctx, call)                                     \
    do {                                                       \
        hipError_t e_ = (call);                                \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #call); \
    } while (0)

// No C++ exception crosses the boundary: host containers and std::thread can throw
// (allocation failure, no thread to be had); every entry point that reaches them runs between
// these two and turns the exception into a status.
#define MATKV_TRY try {
#define MATKV_CATCH(ctx, name)                                                                     \
    } catch (const std::bad_alloc&) {                                                              \
        return fail(ctx, MATKV_ENOMEM, "%s: out of host memory", name);                            \
    } catch (const std::exception& ex_) {                                                          \
        return fail(ctx, MATKV_ENOMEM, "%s: %s", name, ex_.what());                                \
    } catch (...) {                                                                                \
        return fail(ctx, MATKV_ENOMEM, "%s: unexpected C++ exception", name);                      \
    }
#define MATKV_CATCH_INT                                                                            \
    } catch (...) {                                                                                \
        return -1;                                                                                 \
    }

int elem_bytes(const matkv_config& c) { return c.dtype == MATKV_F32 ? 4 : 2; }

matkv_status check_config(const matkv_config* c, const char** why) {
    static const char* ok = "";
    *why = ok;
    if (!c) { *why = "config is null"; return MATKV_EINVAL; }
    if (c->n_layers < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->hidden < 1 ||
        c->max_batch < 1 || c->max_pages < 0 || c->max_tail_tokens < 1) {
        *why = "sizes must be positive"; return MATKV_EINVAL;
    }
    if (c->dtype != MATKV_F32 && c->dtype != MATKV_BF16) { *why = "unknown dtype"; return MATKV_EINVAL; }
    if (c->n_q_heads % c->n_kv_heads) { *why = "n_q_heads not a multiple of n_kv_heads"; return MATKV_EINVAL; }
    if (!(c->rope_base > 1.0f)) { *why = "rope_base must exceed 1"; return MATKV_EINVAL; }
    if (c->softmax_scale < 0.f || isnan(c->softmax_scale)) { *why = "softmax_scale negative"; return MATKV_EINVAL; }
    if (c->hidden % 64) { *why = "hidden must be a multiple of 64"; return MATKV_EINVAL; }
    if (c->max_tail_tokens % 8) { *why = "max_tail_tokens must be a multiple of 8"; return MATKV_EINVAL; }
    if (c->decode_units < 0 || c->decode_units > kMaxDecodeUnitsPerInstance) { *why = "decode_units outside 0..256"; return MATKV_EINVAL; }
    if (c->decode_variant < 0) { *why = "decode_variant negative"; return MATKV_EINVAL; }
    if (c->out_f32 != 0 && c->out_f32 != 1) { *why = "out_f32 must be 0 or 1"; return MATKV_EINVAL; }
    if (c->max_batch > 1024 || c->max_pages > 4096) { *why = "max_batch <= 1024, max_pages <= 4096"; return MATKV_EINVAL; }
    if (c->head_dim != 64 && c->head_dim != 128) { *why = "head_dim must be 64 or 128"; return MATKV_EUNSUPPORTED; }
    const int g = c->n_q_heads / c->n_kv_heads;
    if (!group_size_built(g)) { *why = "group size must be 1, 2, 3, 4 or 8"; return MATKV_EUNSUPPORTED; }
    return MATKV_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Decode workgroups per (instance, KV head) when the configuration does not fix it: one
// workgroup per compute unit over the whole batch and never more than there are compute units
// (a compute unit that holds two runs a third longer, and the launch ends with it: batch 3,
// 8 KV heads: 240 workgroups 19.7 us, 264 workgroups 24.9 us), each with at least 128 tokens.
int choose_decode_units(const matkv_config& c, int batch, long inst_tokens) {
    int u = c.decode_units;
    if (u <= 0) {
        const int per_head = batch * c.n_kv_heads;
        u = 256 / per_head;
        const long cap = inst_tokens / 128;
        if (u > cap) u = (int)cap;
    }
    if (u < 1) u = 1;
    if (u > kMaxDecodeUnitsPerInstance) u = kMaxDecodeUnitsPerInstance;
    return u;
}

// Units one instance's cache is cut into for the question prefill.  The matrix-core kernel runs
// one workgroup per (unit, KV head, row tile), one workgroup per compute unit (its LDS); every extra
// unit costs a partial per question row and a share of the fold launch.  So: as many units as
// leave every workgroup a compute unit of its own and no more - one workgroup too many and the launch
// takes twice as long - none shorter than 256 tokens.  128-row tiles, whose workgroups take a
// step of 128 tokens: 128, unless the batch alone nearly fills the chip (more than 85 workgroups uncut): then a cut in
// two saves a step or two and costs the partials of many rows (8B shape, sixteen users of 300 tokens, us per layer
// in two units -> uncut: questions of 32 rows 25.1 -> 15.9, of 16 rows 20.5 -> 14.2) - and unless short pages make the walk longer
// than its tokens (a step takes two pieces at most: sixteen users over 120 pages of 4 tokens uncut 185, in two
// units 105).  The other kernels launch a workgroup per question row and want few units.
int choose_prefill_units(const matkv_config& cfg, long tiles_in_batch, long tile_rows, long tokens, long pieces) {
    const int g = cfg.n_q_heads / cfg.n_kv_heads;
    const bool mfma = cfg.dtype == MATKV_BF16 && cfg.head_dim == 128 && group_size_built(g);
    long pu = tokens / 1024;
    if (mfma) {
        const long wgs_per_unit = std::max<long>(1, tiles_in_batch * cfg.n_kv_heads);
        const long most = 256 / wgs_per_unit;
        pu = tokens / (tile_rows > 128 || most <= 2 ? 256 : 128);
        if (tile_rows <= 128 && most <= 2) pu = std::max(pu, std::min(tokens / 128, pieces / 4));
        pu = std::min(most, pu);
    }
    return (int)std::max<long>(1, std::min<long>(pu, kMaxPrefillUnitsPerInstance));
}

// Rows of a prefill workgroup's tile.  The cheaper estimate wins: 1.9 us a step of 64 tokens of a 256-row tile, 2.2 of 128
// of a 128-row tile (two groups of waves with 64 each), and about 3 us of every 128 rows for the partials of an instance that
// is cut.  Measured over plain pages, us per layer 128 against 256 rows.  128 taken: 8B shape, one 64-row question over 10 000 tokens
// 27.0 against 31.8, two 38.2 against 41.5, one of 100 rows over 3000 21.1 against 25.2.  256 taken: 8B, sixteen of
// 100 rows over 5000 188.8 against 158.4, 70B, sixteen of 64 rows over 5000 201.8 against 172.5, four of 128 over 20 000 335.7 against 330.0.
// Where the two are near it takes 256 rows too early by now (a step of 128 takes 1.75 to 2.1 us): 8B, four of 64 rows over 10 000 61.6 against
// 65.2, sixteen over 5000 102.5 against 113.6, 70B, one of 128 rows over 10 000 54.2 against 57.2; over compressed pages by less (8B 62.9
// against 63.8, 105.1 against 111.7, 70B 58.8 against 60.1).
int choose_prefill_tile(const matkv_config& cfg, long tiles128, long tiles256, long most_tokens, long most_pieces) {
    auto cost = [&](long tiles, long rows) {
        const long units = choose_prefill_units(cfg, tiles, rows, most_tokens, most_pieces), step = rows > 128 ? 64 : 128;
        const long rounds = (tiles * cfg.n_kv_heads * units + 255) / 256;
        const double steps = (double)(((most_tokens + units - 1) / units + step - 1) / step);
        return (double)rounds * (steps * (rows > 128 ? 1.9 : 2.2) + (units > 1 ? 3.0 * rows / 128 : 0.0));
    };
    return cost(tiles128, 128) <= cost(tiles256, 256) ? 128 : 256;
}

// Estimated time (us) of one layer's row-tile prefill attention without its fold: a start, then as
// many steps as the longest walk has (a step takes one block of 64 tokens, with 128-row tiles two, none across two
// pieces; two 64-row workgroups share a compute unit and take 1.23 times as long) or the reading of the
// cache, whichever is longer - near one another they add up, hence the fourth root; the reading takes longer where
// the compute units hold unequal numbers of workgroups.  The constants are fitted to measurements at the 3B, 8B and
// 70B layer shapes (1 to 24 instances of 64 to 30 000 tokens in 1 to 32 units, questions of up to 64 (row, head)
// rows).  They give the kernels as they are, fold included, within 12 % over plain pages (a launch of 64 tokens 17 %), and the 128-row
// form over compressed ones up to 26 % too slow, where its reading bounds it: so 64-row tiles are taken for twenty-four questions of 4 rows
// over 2000 compressed tokens, 41.9 us a layer against 39.8 (70B shape 45.9 against 40.0).  (A step of 128-row tiles over plain
// pieces that do not fill their blocks takes longer, 2.6 to 3 us: it looks each of them up.)
// walk_tokens, walk_pieces: of the longest unit (compressed pages: its blocks for its pieces); tile_mb: K and V bytes that the tiles read, in MB.
double prefill_form_time(int tile_rows, bool codes, long workgroups, long walk_tokens, long walk_pieces, double tile_mb) {
    const long blocks = std::max((walk_tokens + 63) / 64, walk_pieces), per_round = tile_rows == 64 ? 512 : 256;
    const long steps = tile_rows == 128 ? (blocks + 1) / 2 : blocks;
    double rounds = (double)((workgroups + per_round - 1) / per_round);
    if (tile_rows == 64) rounds = (rounds - 1) * 1.23 + ((workgroups - 1) % per_round >= 256 ? 1.23 : 1.0);
    double start = 7.0, step = 1.9, mb_time = 0.17;
    if (tile_rows == 64) {
        start = codes ? 5.8 : 5.28; step = codes ? 1.6 : 1.22;
        if (codes) mb_time = 0.185;
    } else if (tile_rows == 128) {
        start = codes ? 5.8 : 6.86; step = codes ? 2.25 : walk_pieces * 64 > walk_tokens + 63 ? 2.6 : 1.73;
        if (codes) mb_time = 0.32;
    }
    const double uneven = workgroups >= 96 ? (double)((workgroups + 255) / 256 * 256) / (double)workgroups : 256.0 / 96.0;
    const double walk = rounds * (double)steps * step, read = mb_time * tile_mb * pow(uneven, 0.147);
    return start + pow(pow(walk, 4) + pow(read, 4), 0.25);
}

// Another form and cut of a question prefill than the two rules above choose, where an estimate has it ahead by more than a tie: 128- or
// 256-row tiles, every cache in up to 32 units.  What the rules miss: a cut of a cache of a few hundred tokens costs more in partials and their
// fold than it saves, several rounds of workgroups want another number of them, and the line between the heights moves with how the tiles fill.
// A workgroup takes a start and its steps, a step of a 256-row tile with at most 128 rows less; the compute units of a KV head take them in launch
// order; beside the walk the tiles' K and V are read (near one another they add up, hence the fourth root), and partials are written, read
// and folded.  Constants fitted to 9700 timings of 2500 seeded tables (3B, 8B and 70B shape, 1 to 24 users of 32 to 50 000 tokens, 1- to 260-row questions), 7
// to 9 % apart from them.  Taken where it has a launch ahead by 6 % and 1.5 us, for questions of more than 64 (row, head) rows over 640 tokens and
// more.  Of 1200 other tables of those shapes 10 % are laid out another way, which takes 1/1.11 of the time over plain pages, 1/1.08 compressed, and
// of 2000 tables with 1 to 16 KV heads and 1 to 8 query heads to each 8 %, 1/1.11 and 1/1.08; six of those 158 were slower by 3 to 8 %, all of 12 to 23 us, when
// 6 % were enough.  us a layer: 8B shape, two users of 145 rows over 631 tokens 22.4 -> 16.3, compressed, eleven of up to 83 rows over 10 800 345 -> 286;
// 70B, eleven of 22 rows over 762 26.0 -> 19.3; 3B, compressed, nineteen of up to 42 rows over 27 000 501 -> 410.
// Shorter caches stay with the rules because their layouts are pinned as interface (tests hold matkv_plan_prefill's answers for them), not because the rules are
// ahead there: 8B shape, 32 rows, in units -> uncut, sixteen users of 500 tokens 28.4 -> 17.5, one of 300 13.4 -> 11.8.
// Of 6000 tables of those kinds and of 1 to 16 KV heads 268 are laid out another way than by the rules; 220 of them timed take 1/1.10 of the time in the mean, nine are more
// than 2 % slower: 2 to 7 %, and one 22 % (fifteen users with 16 KV heads, compressed, 85 -> 104).
struct PrefillShape {           // of an instance
    long rows, tokens, pieces;  // (question row, query head of one KV head) rows; cache and question; pages and tail
};
class PrefillTiles {
public:
    PrefillTiles(const std::vector<PrefillShape>& shapes, int Hkv, bool codes, int tile_rows)
        : shapes_(shapes), tile_rows_(tile_rows), Hkv_(Hkv), slots_(std::max(1, std::min(256, 256 / Hkv))) {
        static const Constants kForms[2][2] = {{{3.2, 3.1, 1.55, 1.55, 0.08, 0.126, 0.46, 3.6}, {2.2, 3.6, 1.46, 1.06, 0.02, 0.20, 0.39, 4.5}},
                                               {{3.0, 3.3, 2.0, 2.0, 0.10, 0.20, 0.40, 4.3}, {2.9, 2.7, 1.75, 1.30, 0.02, 0.32, 0.38, 4.9}}};
        k_ = kForms[codes][tile_rows > 128];
        const double row_mb = Hkv * (codes ? 256e-6 : 512e-6);
        double read = 0, whole = 0;
        for (const PrefillShape& s : shapes) {
            const Tiles t = tiles(s);
            read += row_mb * s.tokens * (k_.mb_once + k_.mb_tile * (t.full + t.half));
            whole += (t.full * k_.step + t.half * k_.half_step) * s.tokens * (tile_rows > 128 ? 1.0 / 64 : 1.0 / 128);
            n_tiles_ += t.full + t.half;
            rows_ += s.rows;
            least_tokens_ = std::min(least_tokens_, s.tokens);
        }
        read4_ = read * read * read * read;
        walk_ = (whole + k_.workgroup * n_tiles_) / slots_;
    }
    // Every cache in up to `units` units: no launch takes less than floor(), which grows with them, nor less than what bounds() finds with a look at
    // every instance, nor more than its second; time() deals the workgroups out.
    double floor(int units) const {
        const long u = std::min<long>(units, least_tokens_ / 64);           // of every instance at least
        return launch(walk_, k_.start + (u > 1 ? k_.fold + partials_us((double)rows_ * u) : 0.0));
    }
    std::pair<double, double> bounds(int units) {
        total_ = 0; longest_ = 0; n_jobs_ = 0;
        double partials = 0, shortest = 1e30;
        bool cut = false;
        for (const PrefillShape& s : shapes_) {
            const Job j = job(s, units);
            const Tiles t = tiles(s);
            shortest = std::min(shortest, t.half ? j.half_us : j.us);
            total_ += (t.full * j.us + t.half * j.half_us) * j.n;
            longest_ = std::max(longest_, t.full ? j.us : j.half_us);
            n_jobs_ += (t.full + t.half) * j.n;
            if (j.n > 1) { cut = true; partials += (double)s.rows * j.n; }
        }
        other_ = k_.start + (cut ? k_.fold + partials_us(partials) : 0.0);
        const double mean = total_ / slots_, rounds = (double)((n_jobs_ + slots_ - 1) / slots_);
        return {launch(std::max({longest_, mean, rounds * shortest}), other_), n_jobs_ <= slots_ ? launch(longest_, other_) : launch(mean + longest_, other_)};
    }
    double time(int units) {
        const double least_us = bounds(units).first;
        if (n_jobs_ <= slots_) return least_us;
        std::priority_queue<double, std::vector<double>, std::greater<double>> busy(std::greater<double>(), std::vector<double>(slots_, 0.0));
        double end = 0;
        for (long dealt = 0, tile = 0; dealt < n_tiles_; ++tile)            // launch order: the first tiles of all, then the second
            for (const PrefillShape& s : shapes_) {
                const Tiles t = tiles(s);
                if (tile >= t.full + t.half) continue;
                const Job j = job(s, units);
                for (long i = 0; i < j.n; ++i) {
                    const double us = busy.top() + (tile < t.full ? j.us : j.half_us);
                    busy.pop(); busy.push(us);
                    end = std::max(end, us);
                }
                ++dealt;
            }
        return launch(end, other_);
    }
private:
    struct Constants { double start, workgroup, step, half_step, mb_once, mb_tile, mb_partial, fold; };
    struct Tiles { long full, half; };          // of an instance; half: its last tile of 256, with at most 128 rows
    struct Job { double us, half_us; long n; }; // workgroups of an instance's tile, and how long each takes
    Tiles tiles(const PrefillShape& s) const {
        const long n = (s.rows + tile_rows_ - 1) / tile_rows_, half = tile_rows_ > 128 && s.rows - (n - 1) * tile_rows_ <= 128;
        return {n - half, half};
    }
    Job job(const PrefillShape& s, int units) const {
        const long u = std::max<long>(1, std::min<long>(units, s.tokens / 64));
        const double pieces = (double)s.pieces / u + 1.0 - 1.0 / u, blocks = std::max((double)s.tokens / u / 64 + 0.5 * pieces, pieces);
        const double steps = ceil(tile_rows_ > 128 ? blocks : 0.5 * blocks);
        return {k_.workgroup + steps * k_.step, k_.workgroup + steps * k_.half_step, u};
    }
    double partials_us(double rows) const { return rows * Hkv_ * 528e-6 * k_.mb_partial; }
    // (walk and reading near one another add up)
    double launch(double walk, double other) const { return other + sqrt(sqrt(walk * walk * walk * walk + read4_)); }

    const std::vector<PrefillShape>& shapes_;
    const int tile_rows_, Hkv_, slots_;
    Constants k_;
    long n_tiles_ = 0, rows_ = 0, least_tokens_ = LONG_MAX, n_jobs_ = 0;
    double read4_ = 0, walk_ = 0, total_ = 0, longest_ = 0, other_ = 0;
};

// Cuts one instance's cache (its pages in order, then its tail) into n_units runs of nearly
// equal token counts, in 8-token granules.  A run is a list of items (page pieces); the tail
// is one item and belongs to the last run.  Appends to items / units; returns the number of
// units made (runs that would hold no tokens are dropped).
template <typename ScalesOff>
int build_units(const matkv_page* pages, int n_pages, int inst, int n_units, int tail_estimate,
                int max_tail, Item* items, int* n_items, Unit* units, int* n_units_out, ScalesOff scales_off) {
    long page_gran = 0;
    for (int p = 0; p < n_pages; ++p) page_gran += (pages[p].n_tokens + 7) / 8;
    const long tail_gran = (tail_estimate + 7) / 8;
    const long total = page_gran + tail_gran;
    int made = 0;
    int p = 0;            // current page
    long p_g0 = 0;        // first granule (in the instance's page stream) of page p
    for (int u = 0; u < n_units; ++u) {
        long g0 = total * u / n_units, g1 = total * (u + 1) / n_units;
        const bool last = (u == n_units - 1);
        if (g0 > page_gran) g0 = page_gran;
        if (g1 > page_gran || last) g1 = page_gran;
        if (g1 <= g0 && !last) continue;
        Unit un;
        memset(&un, 0, sizeof(un));
        un.inst = inst; un.item0 = *n_items; un.idx_in_inst = made;
        long g = g0;
        while (g < g1) {
            long pg = (pages[p].n_tokens + 7) / 8;
            while (g >= p_g0 + pg) { p_g0 += pg; ++p; pg = (pages[p].n_tokens + 7) / 8; }
            const long e = (g1 < p_g0 + pg) ? g1 : p_g0 + pg;
            Item it;
            memset(&it, 0, sizeof(it));
            it.base = reinterpret_cast<uint64_t>(pages[p].slot);
            it.page_tokens = pages[p].n_tokens;
            it.tok0 = (int)((g - p_g0) * 8);
            const int t1 = (int)((e - p_g0) * 8);
            it.ntok = (t1 < pages[p].n_tokens ? t1 : pages[p].n_tokens) - it.tok0;
            it.fmt = pages[p].format;
            it.scales16 = (int32_t)(scales_off(pages[p].n_tokens) / 16);
            un.page_tokens += it.ntok;
            items[(*n_items)++] = it;
            g = e;
        }
        if (last) {
            Item it;
            memset(&it, 0, sizeof(it));
            it.base = 0; it.page_tokens = max_tail; it.tok0 = 0; it.ntok = max_tail;
            items[(*n_items)++] = it;
        }
        un.n_items = *n_items - un.item0;
        un.has_tail = last ? 1 : 0;
        un.first = items[un.item0];
        units[(*n_units_out)++] = un;
        ++made;
    }
    for (int k = 0; k < made; ++k) {
        Unit& un = units[*n_units_out - made + k];
        un.n_units_inst = made;
        un.unit0_inst = *n_units_out - made;
    }
    return made;
}

// Question prefill of a batch: tile height, units and their items (punit0 / n_punits of every instance), given the
// batch's pages [batch][max_pages].
template <typename ScalesOff>
PrefillLayout lay_out_prefill(const matkv_config& cfg, const matkv_page* pages, const int32_t* n_pages, const int32_t* q_len, int batch,
                              bool codes, InstanceInfo* insts, Item* items, int* n_items, Unit* units, ScalesOff scales_off) {
    PrefillLayout L;
    const int g = cfg.n_q_heads / cfg.n_kv_heads;
    long most_tokens = 0, most_rows = 0, most_pieces = 0, total_rows = 0;
    std::vector<long> tokens(batch);
    for (int b = 0; b < batch; ++b) {
        total_rows += q_len[b];
        tokens[b] = q_len[b];
        for (int p = 0; p < n_pages[b]; ++p) tokens[b] += pages[(size_t)b * cfg.max_pages + p].n_tokens;
        most_tokens = std::max(most_tokens, tokens[b]);
        most_pieces = std::max<long>(most_pieces, n_pages[b] + 1);
        most_rows = std::max(most_rows, (long)q_len[b] * g);
    }
    // (short questions over very many short pages are better off uncut, on the kernel for units of many pieces)
    const bool cut_pieces = most_rows > 64 || most_pieces <= kMaxPrefillItemsPerUnit;
    auto tiles = [&](long tile_rows) {                  // of (question row, query head of one KV head) over the batch
        long n = 0;
        for (int b = 0; b < batch; ++b) n += ((long)q_len[b] * g + tile_rows - 1) / tile_rows;
        return n;
    };
    L.tile_rows = choose_prefill_tile(cfg, tiles(128), tiles(256), most_tokens, cut_pieces ? most_pieces : 0);
    const long n_tiles = tiles(L.tile_rows);
    const int tall = L.tile_rows, items0 = *n_items;
    int other_units = 0;                                // of every cache at most, where the rules' form and cut are not taken
    if (cfg.dtype == MATKV_BF16 && cfg.head_dim == 128 && group_size_built(g) && most_rows > 64 && most_tokens >= 640 && most_pieces <= kMaxPrefillItemsPerUnit && tiles(128) <= 330) {
        std::vector<PrefillShape> shapes(batch);
        int rule_units = 1;
        for (int b = 0; b < batch; ++b) {
            shapes[b] = {(long)q_len[b] * g, tokens[b], (long)n_pages[b] + 1};
            rule_units = std::max(rule_units, choose_prefill_units(cfg, n_tiles, tall, tokens[b], n_pages[b] + 1));
        }
        PrefillTiles forms[2] = {{shapes, cfg.n_kv_heads, codes, 128}, {shapes, cfg.n_kv_heads, codes, 256}};
        // The rules' own launch is dealt out only where another form's floor is below what it can take at most, and another one only where its bounds are
        // below the best.  Host us of a layout, without the estimate / every candidate dealt out / this: one 8B user of 10 000 tokens 2.1 / 5.1 / 2.9, sixteen of
        // 5000 9.5 / 16.5 / 10.5, four over 17 chunks 4.1 / 10.0 / 4.7, four 70B users of 20 000 4.0 / 9.5 / 4.5 (the same layouts for 60 000 seeded tables).
        auto worth = [](double us) { return std::min(0.94 * us, us - 1.5); };       // another form has to stay below this
        PrefillTiles& by_rule = forms[tall > 128];
        if (std::min(forms[0].floor(1), forms[1].floor(1)) < worth(by_rule.bounds(rule_units).second)) {
            double best = worth(by_rule.time(rule_units));
            for (int f = 0; f < 2; ++f) {
                const long tiles_in_batch = tiles(f ? 256 : 128), one_round = 256 / std::max<long>(1, tiles_in_batch * cfg.n_kv_heads);
                long before = 0;
                // (up to 330 workgroups a KV head, which bounds the host's time: ten rounds at eight KV heads and little more than one at one, where more were not compared)
                for (long u : {1l, 2l, 3l, 4l, 5l, 6l, 8l, 10l, 12l, 16l, 20l, 24l, 32l, std::min<long>(one_round, kMaxPrefillUnitsPerInstance)}) {
                    if (u < 1 || (u > 1 && u > most_tokens / 64) || u == before || tiles_in_batch * u > 330) continue;
                    before = u;
                    if (forms[f].floor((int)u) >= best || forms[f].bounds((int)u).first >= best) continue;
                    const double us = forms[f].time((int)u);
                    if (us < best) { best = us; L.tile_rows = f ? 256 : 128; other_units = (int)u; }
                }
            }
        }
    }
    long walk_tokens = 0, walk_blocks = 0;              // of the longest unit; blocks of 64 tokens, none across two items
    auto cut = [&](auto units_of) {                     // units_of(b): units of instance b
        *n_items = items0;
        L.n_units = 0; L.max_units_inst = 0; L.max_unit_items = 0; walk_tokens = 0; walk_blocks = 0;
        for (int b = 0; b < batch; ++b) {
            insts[b].punit0 = L.n_units;
            insts[b].n_punits = build_units(pages ? pages + (size_t)b * cfg.max_pages : nullptr, n_pages[b], b, units_of(b), q_len[b],
                                            cfg.max_tail_tokens, items, n_items, units, &L.n_units, scales_off);
            L.max_units_inst = std::max(L.max_units_inst, insts[b].n_punits);
            for (int u = insts[b].punit0; u < L.n_units; ++u) {
                L.max_unit_items = std::max(L.max_unit_items, units[u].n_items);
                walk_tokens = std::max(walk_tokens, (long)units[u].page_tokens + (units[u].has_tail ? q_len[b] : 0));
                long blocks = 0;
                for (int i = units[u].item0; i < units[u].item0 + units[u].n_items; ++i)
                    blocks += ((items[i].base ? items[i].ntok : std::min(items[i].ntok, q_len[b])) + 63) / 64;
                walk_blocks = std::max(walk_blocks, blocks);
            }
        }
    };
    auto units_of = [&](int b) {
        if (other_units) return (int)std::max<long>(1, std::min<long>(other_units, tokens[b] / 64));
        return choose_prefill_units(cfg, n_tiles, tall, tokens[b], cut_pieces ? n_pages[b] + 1 : 0);
    };
    cut(units_of);
    // Questions of at most 64 (row, head) rows: 64-row tiles over the same units where they are estimated to be faster
    // by more than a tie.  8B shape, us per layer with 128-row tiles -> 64-row tiles: four 1-row questions over 3000
    // tokens 19.0 -> 17.0, one over 10 000 18.0 -> 16.6, one 16-row question over 64 tokens 7.5 -> 6.6; not: 24 over 2000
    // tokens 39.9 -> 49.8.
    if (cfg.dtype == MATKV_BF16 && cfg.head_dim == 128 && most_rows <= 64 && L.max_unit_items <= kMaxPrefillItemsPerUnit) {
        const double mb = (double)batch * cfg.n_kv_heads * (double)most_tokens * (codes ? 256e-6 : 512e-6);
        auto time = [&](int tile_rows) {                // (the fold included: units may differ)
            const double fold = L.max_units_inst > 1 ? 2.2 + 3.2e-4 * (double)total_rows * cfg.n_q_heads * L.max_units_inst : 0.0;
            return prefill_form_time(tile_rows, codes, (long)L.n_units * cfg.n_kv_heads, walk_tokens, codes ? walk_blocks : L.max_unit_items, mb) + fold;
        };
        const double t128 = time(tall), t64 = time(64);
        if (t64 < 0.98 * t128) L.tile_rows = 64;
        // Two of them share a compute unit, so up to 512 of them are one round: more units, none below 96 tokens, where the
        // estimate says so.  Compressed pages, us per layer with 128-row tiles -> 64-row tiles: twenty-three users of
        // 4 400 tokens in 1 -> 2 units 87 -> 73 (8B), sixteen of 4 000 in 2 -> 4 62.6 -> 55.8 (70B).
        const long most_units = std::min<long>(512 / std::max(1, batch * cfg.n_kv_heads), kMaxPrefillUnitsPerInstance);
        if (std::min(most_units, most_tokens / 96) > L.max_units_inst) {
            cut([&](int b) { return (int)std::max<long>(1, std::min(most_units, tokens[b] / 96)); });
            if (L.max_unit_items <= kMaxPrefillItemsPerUnit && time(64) < 0.96 * (L.tile_rows == 64 ? t64 : t128)) L.tile_rows = 64;
            else                                                                                             cut(units_of);
        }
    }
    // A question of fewer tiles than the longest has no work for the last of them.  Those idle workgroups are moved to the
    // launch's end where they make one more round of 256: 70B shape, questions of 64, 50 and 21 rows over 12 900 tokens 140 -> 94 us
    // per layer, two of 54 and 19 over 19 000 (3B) 84 -> 49.  Otherwise finding its work costs a workgroup about 1 us (nine
    // of 72 and fewer over 490 tokens 21.0 -> 23.1), as it does in several rounds of few tokens each (70B, 21 of 126 and fewer over
    // 218 75 -> 78.5).
    if (L.tile_rows > 64) {
        long live = 0;
        for (int b = 0; b < batch; ++b) live += insts[b].n_punits * (((long)q_len[b] * g + L.tile_rows - 1) / L.tile_rows) * cfg.n_kv_heads;
        const long all = (long)L.n_units * ((most_rows + L.tile_rows - 1) / L.tile_rows) * cfg.n_kv_heads;
        L.deal_tiles = (all + 255) / 256 > (live + 255) / 256 && (live <= 256 || walk_tokens >= 512);
    }
    // Units of more pieces than that (many pages, or short ones): the tile kernels take a piece, or two, a step however short it
    // is, and the kernel whose waves walk the tokens separately is ahead of them only where their workgroups are few or
    // mostly padding.  8B shape, us per layer on the tiles against the other kernel: twelve 64-row questions over 150
    // pages of 40 tokens 184 against 425, over 100 of 4 tokens 154 against 170; one over 90 of 4 tokens (16 workgroups) 135
    // against 55; 24 questions of 4 rows over 70 pages of 8 tokens 104 against 44.
    const long workgroups = (long)L.n_units * cfg.n_kv_heads * ((most_rows + L.tile_rows - 1) / L.tile_rows);
    L.row_tiles = L.max_unit_items <= kMaxPrefillItemsPerUnit || (most_rows > 64 && workgroups >= 96);
    return L;
}

// Even decode partition: the batch's caches end to end (an instance's pages, then its tail), cut into runs of nearly equal length
// without regard to where an instance ends, one workgroup per KV head each, in the records of the shared partition (below).  A run holds
// one tail at the most, so two instances, and each (run, instance) pair has a partial slot.  Always 256 / KV heads runs, empty ones at
// the end: a recorded step has that launch shape whatever the lengths.  By instance, a batch of 17 leaves half of the chip idle, and a
// ragged one waits for its longest cache.
// Items: at most one per run, page and tail, 256 / KV heads + pages + batch of them, for which the table has room behind the two
// partitions by instance (units + pages + batch each) in the 128 per instance that are the shared partition's.
// Returns whether launches take it.  Its kernel looks up whose rows are whose and costs 2 to 4 us more, so only where a run has 400 tokens fewer
// (500 of compressed pages) than the longest unit by instance, as that is cut, its tail whole - and where the longest run, whose tail is not cut either, is
// shorter than that unit.  us per layer step, by instance -> even: 8B shape, 17 users of 3600 tokens 56.3 -> 47.0, of 1000 19.0 -> 17.8, 24 of up to 2000 with 300-row
// questions 36.2 -> 31.5; 70B shape, 17 of 3600 56.6 -> 48.7.  Beyond the line: 9 of 3600 28.8 -> 29.4, 24 of 400 23.9 -> 25.5; 70B, five with 982-row questions
// over 3577 tokens 25.8 -> 33.7, seven with 1488 over 510 19.3 -> 25.6.  Mean gain over 5384 seeded steps (2 to 31 users of 100 to 8000 tokens, questions
// of up to 1600 rows, even and ragged; 3B, 8B, 70B; 4 to 28 layers) by how many tokens fewer: 200 to 300 -1 %, 300 to 400 +2 %, 400 to 500 +3 %, 500 to
// 1000 +8 %, more +17 %; compressed 300 to 400 -3 %, 400 to 500 -2 %, 500 to 700 +2 %, more +12 %.  The better of the two is taken but for 0.2 % of the
// time; by the runs' nominal length and a unit's mean alone, as the line once was, it was 1.1 %, and of 1312 steps over runs 470 were slower for it.
constexpr long kEvenMinGranules = 16;           // 128 tokens
bool build_even_units(const matkv_config& cfg, const matkv_page* pages, const int32_t* n_pages, int batch, InstanceInfo* insts, Item* items,
                      int* n_items, const Unit* dunits, int n_dunits, SUnit* sunits, int kv_fmt) {
    const int n_units = 256 / cfg.n_kv_heads;
    auto tail_gran = [&](int b) { return (long)(insts[b].q_len + (cfg.max_tail_tokens - insts[b].q_len) / 2 + 7) / 8; };
    long total = 0, by_inst = 0;                    // by_inst: tokens of the longest unit by instance
    for (int b = 0; b < batch; ++b) {
        total += tail_gran(b);
        for (int p = 0; p < n_pages[b]; ++p) total += (pages[(size_t)b * cfg.max_pages + p].n_tokens + 7) / 8;
    }
    for (int u = 0; u < n_dunits; ++u)
        by_inst = std::max(by_inst, dunits[u].page_tokens + (dunits[u].has_tail ? 8 * tail_gran(dunits[u].inst) : 0));
    long longest = 0;                               // granules of the longest run of the last cut
    // runs of `per` granules of eight tokens, and of what a tail in their last one has beyond that; emit = false only counts them
    auto cut = [&](long per, bool emit) {
        int n = 0;                                              // runs opened
        long room = 0;
        longest = 0;
        bool has_tail = true;                                   // (of the open run: nothing fits any more)
        SUnit* su = nullptr;
        Item* it = items + *n_items;
        for (int b = 0; b < batch; ++b) {
            if (emit) insts[b].n_sslots = 0;
            bool joined = false;                                // the open run has this instance among its users
            auto open = [&]() {
                if (emit) {
                    su = sunits + n;
                    memset(su, 0, sizeof(*su));
                    su->u.item0 = (int)(it - items);
                    su->u.idx_in_inst = n;
                }
                ++n;
                room = per; has_tail = false; joined = false;
            };
            auto add = [&](const Item& piece) {
                if (!joined) {
                    su->users[su->n_users].inst = b;
                    su->users[su->n_users++].slot = insts[b].n_sslots++;        // (of the instance; its first slot is added below)
                    joined = true;
                }
                *it = piece;
                it->umask = 1 << (su->n_users - 1);
                ++it; ++su->u.n_items;
            };
            for (int p = 0; p < n_pages[b]; ++p) {
                const matkv_page& pg = pages[(size_t)b * cfg.max_pages + p];
                const long gran = (pg.n_tokens + 7) / 8;
                for (long g = 0; g < gran;) {
                    if (room <= 0) open();
                    const long take = std::min(gran - g, room);
                    if (emit) {
                        Item piece;
                        memset(&piece, 0, sizeof(piece));
                        piece.base = reinterpret_cast<uint64_t>(pg.slot);
                        piece.page_tokens = pg.n_tokens;
                        piece.tok0 = (int)(g * 8);
                        piece.ntok = (int)std::min<long>(pg.n_tokens, (g + take) * 8) - piece.tok0;
                        piece.fmt = kv_fmt;
                        piece.scales16 = kv_fmt == MATKV_PAGE_E4M3 ? (int32_t)(compressed_codes_bytes(cfg, pg.n_tokens) / 16) : 0;
                        su->u.page_tokens += piece.ntok;
                        add(piece);
                    }
                    g += take; room -= take;
                    longest = std::max(longest, per - room);
                }
            }
            if (room <= 0 || has_tail) open();                  // a tail is not cut
            if (emit) {
                Item piece;
                memset(&piece, 0, sizeof(piece));
                piece.page_tokens = cfg.max_tail_tokens; piece.ntok = cfg.max_tail_tokens;
                su->u.has_tail = 1; su->u.inst = b;
                add(piece);
            }
            has_tail = true;
            room -= tail_gran(b);
            longest = std::max(longest, per - room);
        }
        if (emit) *n_items = (int)(it - items);
        return n;
    };
    // the shortest runs of which there are no more than workgroups (one per instance is always few enough)
    long per = std::max(kEvenMinGranules, (total + n_units - 1) / n_units);
    while (cut(per, false) > n_units) per += std::max<long>(1, per / 32);
    const int n = cut(per, true);
    if (n < n_units) memset(static_cast<void*>(sunits + n), 0, sizeof(SUnit) * (n_units - n));
    int slot0 = 0;
    for (int b = 0; b < batch; ++b) { insts[b].sslot0 = slot0; slot0 += insts[b].n_sslots; }
    for (int u = 0; u < n; ++u) {
        Unit& un = sunits[u].u;
        // the tail goes last (compressed pages: the kernel walks the code pages and then the plain tail)
        for (int i = un.item0; i + 1 < un.item0 + un.n_items; ++i)
            if (items[i].base == 0) std::rotate(items + i, items + i + 1, items + un.item0 + un.n_items);
        un.first = items[un.item0];
        for (int k = 0; k < sunits[u].n_users; ++k) sunits[u].users[k].slot += insts[sunits[u].users[k].inst].sslot0;
    }
    return by_inst - 8 * per > (kv_fmt == MATKV_PAGE_E4M3 ? 500 : 400) && by_inst > 8 * longest;
}

// Shared decode partition (instances of a batch that retrieved the same chunk read it once).
// The batch's DISTINCT pages and its tails form one stream of token rows - per instance its
// private pages, then the shared pages it uses first, then its tail - which is cut into equal
// runs, one workgroup (per KV head) each, never more workgroups than compute units.  A run is a
// list of pieces like any decode unit; every piece carries the set of the unit's users that
// may see it (Item::umask), the unit lists its users (at most 16 / G: the rows of its matrix
// tile are (user, query head) pairs) and each (unit, user) pair gets one of that user's
// consecutive partial slots.  A run ends early where one more piece would bring a user too many
// or a second tail.  tokens_out (may be null): [unit][kMaxSharedUsers] page tokens each user sees.
// Returns the number of units, 0 if the batch shares no page worth the trouble or the
// partition does not fit the table (then the per-instance partition is used).
int build_shared_units(const matkv_config& cfg, const matkv_page* pages, const int32_t* n_pages, int batch,
                       int max_sunits, int max_items, InstanceInfo* insts, Item* items, int* n_items, SUnit* sunits,
                       int kv_fmt, int32_t* tokens_out = nullptr) {
    struct PageUse { const void* slot; int n_tokens; std::vector<int> users; };
    std::vector<PageUse> distinct;
    std::unordered_map<const void*, std::vector<int>> by_slot;   // slot -> indices into distinct
    for (int b = 0; b < batch; ++b)
        for (int p = 0; p < n_pages[b]; ++p) {
            const matkv_page& pg = pages[(size_t)b * cfg.max_pages + p];
            // (an instance that lists one page twice attends to it twice: the second occurrence is a
            // page of its own)
            int found = -1;
            for (int i : by_slot[pg.slot])
                if (distinct[i].n_tokens == pg.n_tokens &&
                    std::find(distinct[i].users.begin(), distinct[i].users.end(), b) == distinct[i].users.end()) { found = i; break; }
            if (found < 0) {
                found = (int)distinct.size();
                distinct.push_back(PageUse{pg.slot, pg.n_tokens, {}});
                by_slot[pg.slot].push_back(found);
            }
            distinct[found].users.push_back(b);
        }
    // Worth it when the distinct pages are at least a twentieth fewer tokens than all uses together
    // (measured at batch 16, five 1000-token chunks each, per layer, per-instance against shared
    // partition: 81 % of the page tokens distinct 58.3 against 54.8 us, 41 % 43.4 against 35.5,
    // 6 % 33.5 against 18.3).
    long all_tokens = 0, distinct_tokens = 0;
    for (const PageUse& pu : distinct) {
        distinct_tokens += pu.n_tokens;
        all_tokens += (long)pu.n_tokens * (long)pu.users.size();
    }
    if (distinct_tokens * 20 > all_tokens * 19) return 0;

    const int G = cfg.n_q_heads / cfg.n_kv_heads;
    const int cap_users = kMaxSharedUsers / G;
    // a page with more users than a tile has rows for is streamed once per group of them: each
    // group becomes a page of its own from here on
    {
        std::vector<PageUse> split;
        for (const PageUse& pu : distinct)
            for (size_t u0 = 0; u0 < pu.users.size(); u0 += cap_users)
                split.push_back(PageUse{pu.slot, pu.n_tokens,
                                        std::vector<int>(pu.users.begin() + u0, pu.users.begin() + std::min(pu.users.size(), u0 + cap_users))});
        distinct.swap(split);
    }
    // the stream: per instance the pages it is the first user of (private ones first), then its
    // tail; an instance that is the first user of no page gets its tail behind a page it uses (one
    // tail per page at most), so that tails stay apart: a unit holds at most one
    struct Piece { int page; int inst; long gran; std::vector<int> users; };    // page < 0: the tail of inst
    std::vector<Piece> stream;
    std::vector<char> tail_placed(batch, 0), owns(batch, 0);
    for (const PageUse& pu : distinct) owns[pu.users[0]] = 1;
    long total_gran = 0;
    auto push_tail = [&](int b) {
        const int tail_est = insts[b].q_len + (cfg.max_tail_tokens - insts[b].q_len) / 2;
        stream.push_back(Piece{-1, b, (tail_est + 7) / 8, {b}});
        total_gran += stream.back().gran;
        tail_placed[b] = 1;
    };
    for (int b = 0; b < batch; ++b) {
        for (int pass = 0; pass < 2; ++pass)                     // private pages first
            for (size_t di = 0; di < distinct.size(); ++di) {
                const PageUse& pu = distinct[di];
                if (pu.users[0] != b || (pass == 0) != (pu.users.size() == 1)) continue;
                stream.push_back(Piece{(int)di, b, (pu.n_tokens + 7) / 8, pu.users});
                total_gran += stream.back().gran;
                for (int u : pu.users)
                    if (!tail_placed[u] && !owns[u]) { push_tail(u); break; }
            }
        if (owns[b]) push_tail(b);
    }
    for (int b = 0; b < batch; ++b)
        if (!tail_placed[b]) push_tail(b);
    int n_target = 256 / cfg.n_kv_heads;
    if (n_target > total_gran * 8 / 128) n_target = (int)(total_gran * 8 / 128);
    if (n_target < 1) n_target = 1;

    // Cuts the stream into units of `per` granules; returns the number of units, or -1 if they do
    // not fit.  emit = false only counts.
    std::vector<std::vector<int>> slot_of;                       // [unit][user index] -> partial slot (second pass)
    auto cut = [&](long per, bool emit, int first_item) -> int {
        int n = 0, n_it = first_item;
        long room = 0;                                           // granules the open unit may still take
        std::vector<int> users;                                  // of the open unit
        bool open = false, has_tail = false;
        SUnit* su = nullptr;
        auto close_unit = [&]() {
            if (!open) return;
            if (emit) {
                su->u.n_items = n_it - su->u.item0;
                // the unit's tail, if it has one, goes last (compressed pages: the kernel walks the
                // code pages and then the plain tail)
                for (int i = su->u.item0; i + 1 < n_it; ++i)
                    if (items[i].base == 0) std::rotate(items + i, items + i + 1, items + n_it);
                su->u.first = items[su->u.item0];
                su->n_users = (int)users.size();
                for (size_t k = 0; k < users.size(); ++k) su->users[k].inst = users[k];
            }
            ++n; open = false;
        };
        auto open_unit = [&]() {
            if (emit) {
                su = &sunits[n];
                memset(su, 0, sizeof(*su));
                su->u.item0 = n_it;
            }
            users.clear(); room = per; open = true; has_tail = false;
        };
        for (const Piece& pc : stream) {
            const std::vector<int>& pusers = pc.users;
            long g = 0;
            while (g < pc.gran) {
                if (open) {
                    int fresh = 0;
                    for (int u : pusers) if (std::find(users.begin(), users.end(), u) == users.end()) ++fresh;
                    if ((int)users.size() + fresh > cap_users || (pc.page < 0 && has_tail) || room <= 0) close_unit();
                }
                if (!open) {
                    if (n >= max_sunits) return -1;
                    open_unit();
                }
                uint32_t mask = 0;
                for (int u : pusers) {
                    auto it = std::find(users.begin(), users.end(), u);
                    if (it == users.end()) { users.push_back(u); it = users.end() - 1; }
                    mask |= 1u << (int)(it - users.begin());
                }
                // a tail is never cut; a page piece takes what room there is
                const long take = pc.page < 0 ? pc.gran : std::min(pc.gran - g, room);
                if (emit) {
                    if (n_it >= max_items) return -1;
                    Item it;
                    memset(&it, 0, sizeof(it));
                    if (pc.page < 0) {
                        it.base = 0; it.page_tokens = cfg.max_tail_tokens; it.tok0 = 0; it.ntok = cfg.max_tail_tokens;
                        su->u.has_tail = 1; su->u.inst = pc.inst;
                    } else {
                        const PageUse& pu = distinct[pc.page];
                        it.base = reinterpret_cast<uint64_t>(pu.slot);
                        it.page_tokens = pu.n_tokens;
                        it.tok0 = (int)(g * 8);
                        it.ntok = (int)std::min<long>(pu.n_tokens, (g + take) * 8) - it.tok0;
                        it.fmt = kv_fmt;
                        it.scales16 = kv_fmt == MATKV_PAGE_E4M3 ? (int32_t)(compressed_codes_bytes(cfg, pu.n_tokens) / 16) : 0;
                        su->u.page_tokens += it.ntok;
                        if (tokens_out)
                            for (int k = 0; k < kMaxSharedUsers; ++k)
                                if (mask >> k & 1) tokens_out[(size_t)n * kMaxSharedUsers + k] += it.ntok;
                    }
                    it.umask = (int32_t)mask;
                    items[n_it] = it;
                }
                ++n_it;
                if (pc.page < 0) has_tail = true;
                g += take; room -= take;
            }
        }
        close_unit();
        if (emit) *n_items = n_it;
        return n;
    };
    // unit size: the smallest with which the launch has no more workgroups than compute units
    long per = std::max<long>(16, (total_gran + n_target - 1) / n_target);
    int n = cut(per, false, *n_items);
    for (int it = 0; it < 64 && (n < 0 || n * cfg.n_kv_heads > 256); ++it) {
        per += std::max<long>(1, per / 32);
        n = cut(per, false, *n_items);
    }
    if (n <= 0 || n > max_sunits || n * cfg.n_kv_heads > 256) return 0;
    if (tokens_out) memset(tokens_out, 0, sizeof(int32_t) * (size_t)n * kMaxSharedUsers);
    n = cut(per, true, *n_items);
    if (n <= 0) return 0;
    // partial slots: every (unit, user) pair one, an instance's slots consecutive
    std::vector<int> count(batch, 0), next(batch, 0);
    for (int u = 0; u < n; ++u)
        for (int k = 0; k < sunits[u].n_users; ++k) ++count[sunits[u].users[k].inst];
    int slot0 = 0;
    for (int b = 0; b < batch; ++b) {
        if (count[b] > kMaxDecodeUnitsPerInstance) return 0;
        insts[b].sslot0 = slot0; insts[b].n_sslots = count[b];
        next[b] = slot0;
        slot0 += count[b];
    }
    for (int u = 0; u < n; ++u) {
        sunits[u].u.idx_in_inst = u;
        for (int k = 0; k < sunits[u].n_users; ++k) sunits[u].users[k].slot = next[sunits[u].users[k].inst]++;
    }
    return n;
}

// Whether a batch without shared pages gets the even partition (build_even_units) beside the one by instance: one whose step is not
// the fused launch.  A step that was recorded over it replays over every table with the same batch and units by instance, and this says the
// same of all of them.  Its units follow the others in their section (and are copied with them).
bool even_partition(const matkv_config& cfg, int batch, int n_dunits) {
    const int g = cfg.n_q_heads / cfg.n_kv_heads, n_units = 256 / cfg.n_kv_heads;
    return cfg.decode_units == 0 && cfg.decode_variant == 0 && cfg.dtype == MATKV_BF16 && cfg.head_dim == 128 && group_size_built(g) &&
           batch >= 2 && (batch > 4 || g > 4) && batch <= n_units &&
           sizeof(Unit) * n_dunits + sizeof(SUnit) * n_units <= sizeof(Unit) * (size_t)table_layout(cfg).max_dunits;
}

// Whether decode launches leave the cache's rows out of the last-level cache.  streamed, tail_rows: the page tokens and tail rows that they walk of a
// layer, distinct: the page tokens among them that are not the same ones again; longest: tokens of the longest workgroup's walk.  A step reads the rows and the projection's weights of all layers, and the next step reads them again.
//  - All of it fits: it is found there again, rows are left there.  Past that by a sixteenth, weights fit: rows pass by and the weights stay.
//    us per layer step, rows left there / passing by: 8B shape, 8 layers and 265 MB 11.0 / 11.3, 12 layers and 300 MB 10.3 / 10.0, 15 layers and
//    313 MB 9.9 / 9.4; 70B, 7 layers and 264 MB 14.9 / 15.5, 292 MB 15.9 / 16.2, 349 MB 18.4 / 18.1; sixteen 8B users over 5000 tokens 70.0 / 63.0.
//  - The weights alone exceed it, as they do in a whole model: nothing is found again either way, and short steps are better off with the ordinary
//    loads.  8B, 32 layers, by the rows of a layer: 4 MB 10.1 / 10.7, 8 MB 10.8 / 11.2, 16 MB 12.1 / 12.3 (four users 14.6 / 14.7), 33 MB 14.8 / 14.7
//    (eight users 24.0 / 23.4), 66 MB 21.0 / 20.3, 335 MB 70.0 / 65.5; 70B, 20 layers, 16 MB 18.8 / 19.1, 33 MB 21.7 / 21.4, 66 MB 27.3 / 26.6; compressed, two
//    users of 8B, 3B and 70B with 4 MB 12.0 / 12.2, 10.4 / 10.4, 16.7 / 16.8, three with 6 MB 12.7 / 12.6, 11.5 / 11.3, 17.1 / 17.1, four with 8 MB 13.5 / 13.5,
//    12.0 / 11.8, 17.8 / 17.8, one of 8B with 33 MB 16.0 / 15.7.  So a layer's rows have to be 24 MB, or 7 MB of codes.  In between (17 layers, 285 MB
//    of weights) part of the weights is found: 8 MB 10.7 / 11.0, 16 MB 12.1 / 12.0, compressed 8 MB 10.9 / 10.5: the line falls to nothing where they just fit.
//  - A load that passes by takes longer, and a workgroup has two blocks on their way: it gains only with most of the chip walking to the end.
//    Time saved by passing by, mean over seeded steps of 1 to 31 users (3B, 8B, 70B; 4 to 28 layers, plain pages), by the workgroups that would
//    take as long if all walks were as long as the longest: weights fit, up to 64 -5 %, 64 to 128 -3.5 %, 128 to 160 -1 %, 160 to 192 +1 %, 192 to 224 +4 %, more
//    +7 %; they exceed it, up to 128 -5 %, 128 to 192 -3 %, 192 to 208 -1 %, 208 to 224 0, more +2 %.  Compressed pages alike.  So 160 and 208 of them.
//    Attention over 2000 tokens each, one unit per user, 16 layers: one user 22.3 / 30.9, eight 28.4 / 33.5, 17 32.3 / 36.3, 24 38.0 / 38.8.
//  - Pages that several units stream (more users than a tile has rows; units by instance over pages that are shared after all) are found again
//    within the launch if they are left there.  Time saved by passing by, mean over seeded steps of 2 to 32 users of shared pages where the rest speaks for it, by
//    tokens walked per distinct one: 1 +5 %, up to 1.06 +3 %, 1.125 +1 %, 1.2 0, 1.3 -1 %, 1.6 -3 %, 3 -6 %, more -10 %; compressed pages 1 +4 %, up to 1.125 +3 %,
//    1.3 +2 %, 1.6 0, 3 -2 %, more -5 %.  So 9/8.  us per layer, left there / passing by, 4 layers: sixteen 70B users of the same 5000 tokens 20.8 / 26.4, of 5 in 20
//    chunks 45.8 / 51.7, 24 of 5 in 60 74.1 / 80.1.  Over 18147 such steps the slower of the two is taken for 0.2 % of the time; with the tokens walked for
//    the distinct ones it was 1.9 %.
//    A fused step over shared pages (four users at most, each walks all of its own) is worth that only where the weights exceed the cache; where they fit, keeping
//    them there is worth more.  us per layer step, passing by / left there: 8B, 32 layers, two users, 5000 tokens in common and 1000 of their own 16.5 / 15.2, 4000
//    19.7 / 19.1, four with 3500 and 3000 24.3 / 22.4, compressed, two with 9000 and 4000 17.5 / 16.9; 3B, three with 3500 and 8000 33.8 / 29.5; of 17 seeded
//    batches 1.045 times as fast in the mean, 0.995 at least.  Weights that fit: 8B, 14 layers, two with 770 and 2000 compressed 11.0 / 12.7, 8 layers, two with
//    1200 and 2000 12.8 / 13.0, four with 3500 and 3000 23.5 / 22.5; of 53 batches 0.991 in the mean, 0.87 at least.
// Over 8196 steps without shared pages (plain and compressed) the better of the two is taken but for 0.2 % of the time; where all beyond 256 MB passed by it was 1.6 %.
constexpr size_t kStreamedLayerBytes = (size_t)24 << 20, kStreamedCodeBytes = (size_t)7 << 20;
constexpr int kStreamedWalks = 160, kStreamedWalksFar = 208;
bool rows_pass_llc(const matkv_config& cfg, size_t distinct, size_t streamed, size_t tail_rows, size_t longest, int kv_fmt, bool fused_step = false) {
    const size_t row = 2 * (size_t)cfg.n_kv_heads * cfg.head_dim, esz = cfg.dtype == MATKV_BF16 ? 2 : 4, llc = kLastLevelCacheBytes;
    const size_t layer = row * (distinct * (kv_fmt == MATKV_PAGE_E4M3 ? 1 : esz) + tail_rows * esz);
    const size_t weights = row * cfg.hidden * esz * cfg.n_layers;
    if (8 * streamed > 9 * distinct && (!fused_step || weights > llc)) return false;
    if (layer * cfg.n_layers + weights <= llc + llc / 16) return false;
    const double over = weights > llc ? std::min(1.0, (double)(weights - llc) / (double)(llc / 8)) : 0.0;      // 1: nothing of the weights is found again
    const double walks = (double)cfg.n_kv_heads * (double)(streamed + tail_rows) / (double)std::max<size_t>(longest, 1);
    return (double)layer > over * (double)(kv_fmt == MATKV_PAGE_E4M3 ? kStreamedCodeBytes : kStreamedLayerBytes) &&
           walks >= kStreamedWalks + over * (kStreamedWalksFar - kStreamedWalks);
}

// Page tokens of a batch: every use of a page counted, and every slot once.
std::pair<size_t, size_t> count_page_tokens(const matkv_config& cfg, const matkv_page* pages, const int32_t* n_pages, int batch) {
    std::vector<std::pair<const void*, int>> seen;
    for (int b = 0; pages && b < batch; ++b)
        for (int p = 0; p < n_pages[b]; ++p) seen.emplace_back(pages[(size_t)b * cfg.max_pages + p].slot, pages[(size_t)b * cfg.max_pages + p].n_tokens);
    std::sort(seen.begin(), seen.end());
    size_t uses = 0, distinct = 0;
    for (size_t i = 0; i < seen.size(); ++i) {
        uses += seen[i].second;
        if (i == 0 || seen[i].first != seen[i - 1].first) distinct += seen[i].second;
    }
    return {uses, distinct};
}

// Whether a decode step that can be the fused launch is it although the batch shares pages.  That launch reads every instance's cache for itself, but
// hides the projection and spares the shared kernel's fold: 5 us for two instances, 6 for four, less the time of the bytes that are read twice.  us per layer step,
// over the shared partition -> fused, by what a layer reads twice (8B shape): two users, 1 MB 15.8 -> 11.1, 20 18.4 -> 17.2, 41 21.4 -> 22.6, 49 22.3 -> 24.4;
// three, 39 22.0 -> 18.1 in four layers, 65 23.5 -> 26.1; four, 39 24.6 -> 22.2, 61 22.9 -> 22.1, 74 23.5 -> 24.1.  3B: two, 41 20.8 -> 21.1, four, 61 21.3 -> 21.0.  Of
// compressed pages (8B) two, 20 18.6 -> 13.3, 41 22.5 -> 23.0, four, 61 25.3 -> 23.8; (3B) four, 74 24.2 -> 25.2.  Long caches end it: with 5 to 25 % of the uses
// shared, four users of 82 MB 1.04 to 1.24 times as fast, 131 MB in all 1.05, 164 1.00 to 1.06, 184 1.02, 246 0.985.
// A ragged batch ends it too, since the launch waits for the longest unit by instance, and shared units are even.  605 seeded steps of two to four users within those lines,
// by how many tokens longer it is (of codes half as many): up to 100 1.45 times as fast in the mean and 1.10 at least, 100 to 200 1.19, 200 to 300 1.10, 300 to 400 1.06, more
// 1.005 and 0.951 at least (8B, four users of up to 12 000 tokens with 1895 in common 34.0 -> 35.8).
bool step_by_instance(const matkv_config& cfg, size_t uses, size_t distinct, int batch, int kv_fmt, long longest, long longest_shared) {
    if (longest - longest_shared > (kv_fmt == MATKV_PAGE_E4M3 ? 800 : 400)) return false;
    const size_t row = (size_t)2 * cfg.n_kv_heads * cfg.head_dim * (kv_fmt == MATKV_PAGE_E4M3 ? 1 : 2);
    return (uses - distinct) * row <= (size_t)batch * 12000000 && uses * row <= 192000000;
}

// How an instance's cache is cut into decode units, one workgroup per (unit, KV head).  Over compressed pages a unit walks its codes first and asks for
// the tail behind them, a round trip of its own, and the launch ends with it (8B shape, one user of 10 000 tokens: 8.4 us against 7.5 of the others): the
// unit that has the tail gets 128 tokens fewer, unless the tail fills it anyway (of 750 with a 200-row question, whatever the tail fills, 298 -> 325 us a pass).
// Units below 192 tokens over several pages stay even: a longer unit is a wave that starts or goes on behind one more page boundary, whose record it has
// to look up.  us per layer step, even -> spared: one 8B user of 3 x 214 tokens 8.3 -> 9.1, of 6 x 65 8.9 -> 9.5, one 3B user of 8 x 88 8.4 -> 9.1 (left even); of 1 x
// 436 8.8 -> 8.1, one 3B user of 1 x 532 9.1 -> 8.0, two 8B users of 10 x 522 14.1 -> 13.0, one of 40 x 371 15.1 -> 14.3, four of 21 x 80 12.8 -> 13.1 (the worst); one of 4 x 1295, left even, would gain (11.3 -> 10.4).  Of 209
// seeded steps (3B, 8B, 70B; 1 to 10 users of 130 to 15 000 tokens) the 136 that spare take 1/1.038 of the time in the mean; the 73 left even would have been between 0.916 and
// 1.15 times as fast.  (256 fewer: in the mean the same.  Plain pages, 32 or 64 fewer: 0.98 to 1.02.)
// Nor where units are below 128 tokens, as they can be where the configuration fixes their number: several would come to lie behind the pages' end and
// fall away, and a step recorded over one table would not fit the next.
struct DecodeCut { int units, tail_tokens; bool spares; };      // units; tokens that the tail counts for
DecodeCut decode_cut(const matkv_config& cfg, int batch, long page_tokens, int n_pages, int q_len, int kv_fmt) {
    const int tail = q_len + (cfg.max_tail_tokens - q_len) / 2, units = choose_decode_units(cfg, batch, page_tokens + tail);
    const bool spares = kv_fmt == MATKV_PAGE_E4M3 && (long)std::max(tail + 1, n_pages > 1 ? 192 : 128) * units <= page_tokens + tail;
    return {units, tail + (spares ? 128 : 0), spares && units > 1};
}

// Decode attention of a batch (insts: q_len is set): the units of every instance, and beside them the shared partition or
// the even one where they apply.  sunits: the table's section of the shared partition; the even one's records follow dunits.
struct DecodeLayout {
    int n_dunits = 0, n_sunits = 0;
    bool even_built = false, even = false, past_llc = false, tail_spared = false;
    bool step_by_instance = false, step_past_llc = false;       // of a decode step in one launch
};
template <typename ScalesOff>
DecodeLayout lay_out_decode(const matkv_config& cfg, const TableLayout& tl, const matkv_page* pages, const int32_t* n_pages, int batch, int kv_fmt,
                            InstanceInfo* insts, Item* items, int* n_items, Unit* dunits, SUnit* sunits, ScalesOff scales_off) {
    DecodeLayout L;
    for (int b = 0; b < batch; ++b) {
        const matkv_page* pg = pages ? pages + (size_t)b * cfg.max_pages : nullptr;
        long inst_tokens = 0;
        for (int p = 0; p < n_pages[b]; ++p) inst_tokens += pg[p].n_tokens;
        const DecodeCut c = decode_cut(cfg, batch, inst_tokens, n_pages[b], insts[b].q_len, kv_fmt);
        L.tail_spared |= c.spares;
        insts[b].dunit0 = L.n_dunits;
        insts[b].n_dunits = build_units(pg, n_pages[b], b, c.units, c.tail_tokens, cfg.max_tail_tokens, items, n_items, dunits, &L.n_dunits, scales_off);
    }
    // over shared pages: only where the default matrix-core decode kernel runs
    if (batch >= 2 && pages && cfg.decode_units == 0 && cfg.decode_variant == 0 &&
        cfg.dtype == MATKV_BF16 && cfg.head_dim == 128 && group_size_built(cfg.n_q_heads / cfg.n_kv_heads))
        L.n_sunits = build_shared_units(cfg, pages, n_pages, batch, tl.max_sunits, tl.max_items, insts, items, n_items, sunits, kv_fmt);
    SUnit* const runs = reinterpret_cast<SUnit*>(dunits + L.n_dunits);
    if (L.n_sunits == 0 && even_partition(cfg, batch, L.n_dunits)) {
        L.even_built = true;
        L.even = build_even_units(cfg, pages, n_pages, batch, insts, items, n_items, dunits, L.n_dunits, runs, kv_fmt);
    }
    size_t uses = 0, distinct = 0;                  // page tokens, counted when they are first asked for
    auto count = [&]() { if (uses == 0) std::tie(uses, distinct) = count_page_tokens(cfg, pages, n_pages, batch); };
    auto past_llc = [&](auto unit, int n_units, bool fused_step) {      // of a launch over n_units units, unit(u) one of them
        size_t streamed = 0, tail_rows = 0, longest = 0;
        for (int u = 0; u < n_units; ++u) {
            const Unit& un = unit(u);
            const size_t tail = un.has_tail ? insts[un.inst].q_len : 0;
            streamed += un.page_tokens; tail_rows += tail;
            longest = std::max(longest, un.page_tokens + tail);
        }
        if (!rows_pass_llc(cfg, streamed, streamed, tail_rows, longest, kv_fmt)) return false;      // (with fewer distinct ones it is no other)
        count();
        return rows_pass_llc(cfg, distinct, streamed, tail_rows, longest, kv_fmt, fused_step);
    };
    auto by_instance = [&](int u) -> const Unit& { return dunits[u]; };
    int n_runs = 0;
    while (L.even && n_runs < 256 / cfg.n_kv_heads && runs[n_runs].n_users > 0) ++n_runs;
    if (L.even)              L.past_llc = past_llc([&](int u) -> const Unit& { return runs[u].u; }, n_runs, false);
    else if (L.n_sunits > 0) L.past_llc = past_llc([&](int u) -> const Unit& { return sunits[u].u; }, L.n_sunits, false);
    else                     L.past_llc = past_llc(by_instance, L.n_dunits, false);
    L.step_past_llc = L.past_llc;
    // (a fused step over the units by instance walks a shared page once for each of its users: its own answer)
    if (L.n_sunits > 0 && fused_step_shape(cfg.dtype, cfg.head_dim, cfg.n_q_heads / cfg.n_kv_heads, cfg.hidden, batch)) {
        count();
        long longest = 0, longest_shared = 0;
        for (int u = 0; u < L.n_dunits; ++u) longest = std::max<long>(longest, dunits[u].page_tokens);
        for (int u = 0; u < L.n_sunits; ++u) longest_shared = std::max<long>(longest_shared, sunits[u].u.page_tokens);
        L.step_by_instance = step_by_instance(cfg, uses, distinct, batch, kv_fmt, longest, longest_shared);
        if (L.step_by_instance) L.step_past_llc = past_llc(by_instance, L.n_dunits, true);
    }
    return L;
}

TableHost* find_table(matkv_ctx* c, const void* t) {
    auto it = c->tables.find(t);
    return it == c->tables.end() ? nullptr : &it->second;
}

// Launch shapes are fixed when a call is recorded; they follow from these.  Kernel choices are fixed too and need not: whether a step is the fused launch, whether rows
// pass the last-level cache and whether places are looked up ahead may be other for a table that is assembled later, and each gives the right result over
// every table of equal signature (the units by instance, the shared and the even ones are all there wherever they were).
uint64_t fnv(std::initializer_list<int> f) {
    uint64_t h = 1469598103934665603ull;
    for (int v : f) { h ^= (uint64_t)(uint32_t)v; h *= 1099511628211ull; }
    return h;
}
void sign_partition(TableHost& th) {
    th.sig_decode = fnv({th.batch, th.n_dunits, th.n_sunits, th.kv_fmt});
    // (a recorded prefill launch also bakes in the tile height.  It is left out: every height gives the right result
    // on every partition, and a table that would now take another one is replayed as recorded.)
    th.sig_prefill = fnv({th.batch, th.prefill.n_units, th.total_q, th.max_q, th.prefill.max_units_inst, th.prefill.max_unit_items, th.kv_fmt});
}
// While a graph is being recorded: remember that it reads this table's decode or prefill side.
void note_table_use(matkv_ctx* c, const void* table, const TableHost& th, bool prefill) {
    if (!c->capturing || !c->cap) return;
    for (auto& e : c->cap->tables)
        if (e.table == table) { (prefill ? e.prefill : e.decode) = true; return; }
    c->cap->tables.push_back({table, !prefill, prefill, th.sig_decode, th.sig_prefill});
}

matkv_status precheck(matkv_ctx* c) {
    if (!c) return MATKV_EINVAL;
    if (c->sticky_hip) return MATKV_EHIP;
    return MATKV_OK;
}

}  // namespace

extern "C" {

const char* matkv_status_string(matkv_status s) {
    switch (s) {
        case MATKV_OK: return "MATKV_OK";
        case MATKV_EINVAL: return "MATKV_EINVAL";
        case MATKV_EUNSUPPORTED: return "MATKV_EUNSUPPORTED";
        case MATKV_ENOTREADY: return "MATKV_ENOTREADY";
        case MATKV_EBUSY: return "MATKV_EBUSY";
        case MATKV_EHIP: return "MATKV_EHIP";
        case MATKV_ENOMEM: return "MATKV_ENOMEM";
        case MATKV_EIO: return "MATKV_EIO";
    }
    return "MATKV_?";
}

matkv_status matkv_config_check(const matkv_config* cfg) {
    const char* why;
    return check_config(cfg, &why);
}

size_t matkv_blob_bytes(const matkv_config* cfg, int32_t n_tokens) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK || n_tokens < 0) return 0;
    return (size_t)cfg->n_layers * 2 * cfg->n_kv_heads * (size_t)n_tokens * cfg->head_dim * elem_bytes(*cfg);
}

size_t matkv_compressed_blob_bytes(const matkv_config* cfg, int32_t n_tokens) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK || n_tokens < 0) return 0;
    return compressed_codes_bytes(*cfg, n_tokens) + compressed_scales_bytes(*cfg);
}

size_t matkv_tail_bytes(const matkv_config* cfg) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return 0;
    return (size_t)cfg->max_batch * cfg->n_kv_heads * (size_t)cfg->max_tail_tokens * cfg->head_dim * elem_bytes(*cfg);
}

size_t matkv_workspace_bytes(const matkv_config* cfg) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return 0;
    return workspace_layout(*cfg).bytes;
}

size_t matkv_table_bytes(const matkv_config* cfg) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return 0;
    return table_layout(*cfg).bytes;
}

matkv_status matkv_create(const matkv_config* cfg, void* workspace, size_t workspace_bytes,
                          void* compute_stream, void* load_stream, matkv_ctx** out) {
    if (!out) return MATKV_EINVAL;
    *out = nullptr;
    const char* why;
    matkv_status st = check_config(cfg, &why);
    if (st != MATKV_OK) return st;
    const WorkspaceLayout wl = workspace_layout(*cfg);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return MATKV_EINVAL;
    if (workspace_bytes < wl.bytes) return MATKV_ENOMEM;

    matkv_ctx* c = new (std::nothrow) matkv_ctx();
    if (!c) return MATKV_ENOMEM;
    c->cfg = *cfg;
    c->err[0] = 0;
    c->compute = reinterpret_cast<hipStream_t>(compute_stream);
    c->load = reinterpret_cast<hipStream_t>(load_stream);
    c->workspace = reinterpret_cast<char*>(workspace);
    c->wl = wl;
    c->tl = table_layout(*cfg);
    const float scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : 1.0f / sqrtf((float)cfg->head_dim);
    c->scale_log2e = scale * 1.4426950408889634f;
    try {
        c->tickets.resize(kTicketRing);
    } catch (...) {
        delete c;
        return MATKV_ENOMEM;
    }

    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess) e = scratch_address(c->device, &c->static_scratch);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->fence_ev, hipEventDisableTiming);
    // rotary table: inv_freq in double, and inv_freq / 2pi split into two floats
    RopeEntry rope[64];
    const int half = cfg->head_dim / 2;
    for (int j = 0; j < half; ++j) {
        const double f = pow((double)cfg->rope_base, -2.0 * j / (double)cfg->head_dim);
        const double turns = f / 6.283185307179586476925286766559;
        rope[j].inv_freq = f;
        rope[j].turns_hi = (float)turns;
        rope[j].turns_lo = (float)(turns - (double)rope[j].turns_hi);
    }
    if (e == hipSuccess) e = hipMemcpy(c->workspace + wl.off_rope, rope, sizeof(RopeEntry) * half, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemsetAsync(c->workspace + wl.off_counters, 0, wl.off_partials - wl.off_counters, c->compute);
    for (int i = 0; i < kStagingRing && e == hipSuccess; ++i) {
        e = hipHostMalloc(reinterpret_cast<void**>(&c->staging[i].host), c->tl.bytes, hipHostMallocDefault);
        if (e == hipSuccess) e = hipHostGetDevicePointer(reinterpret_cast<void**>(&c->staging[i].host_on_device), c->staging[i].host, 0);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&c->staging[i].ev, hipEventDisableTiming);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        matkv_destroy(c);
        return MATKV_EHIP;
    }
    *out = c;
    return MATKV_OK;
}

matkv_status matkv_destroy(matkv_ctx* c) {
    if (!c) return MATKV_EINVAL;
    {
        std::lock_guard<std::mutex> lk(c->io_mu);
        c->io_stop = true;                   // requests still queued are dropped with the context
    }
    c->io_work.notify_all();
    for (std::thread& th : c->io_readers) th.join();
    (void)hipStreamSynchronize(c->load);
    (void)hipStreamSynchronize(c->compute);
    for (matkv_graph* g : c->graphs) {
        if (g->exec) (void)hipGraphExecDestroy(g->exec);
        if (g->graph) (void)hipGraphDestroy(g->graph);
        delete g;
    }
    for (Ticket& t : c->tickets)
        if (t.ev) (void)hipEventDestroy(t.ev);
    for (int i = 0; i < kStagingRing; ++i) {
        if (c->staging[i].ev) (void)hipEventDestroy(c->staging[i].ev);
        if (c->staging[i].host) (void)hipHostFree(c->staging[i].host);
    }
    for (int i = 0; i < kBounceRing; ++i) {
        if (c->bounce[i].ev) (void)hipEventDestroy(c->bounce[i].ev);
        if (c->bounce[i].host) (void)hipHostFree(c->bounce[i].host);
    }
    free(c->plain_buf);
    for (int i = 0; i < kReleaseRing; ++i)
        if (c->release_ev[i]) (void)hipEventDestroy(c->release_ev[i]);
    if (c->fence_ev) (void)hipEventDestroy(c->fence_ev);
    (void)hipGetLastError();
    delete c;
    return MATKV_OK;
}

const char* matkv_last_error(const matkv_ctx* c) { return c ? c->err : "context is null"; }

// ------------------------------------------------------------------------------------ M ----

// The workspace's partial and counter regions as scratch of a projection launch (every call runs
// on the compute stream, so it never overlaps an attention launch that uses them).
static void materialize_scratch(matkv_ctx* c, MaterializeArgs& a) {
    a.ws_partials = reinterpret_cast<float*>(c->workspace + c->wl.off_partials);
    a.ws_counters = reinterpret_cast<int32_t*>(c->workspace + c->wl.off_counters);
    a.ws_partial_floats = (int64_t)c->wl.partial_floats;
    a.ws_n_counters = (int32_t)std::min<size_t>(c->wl.n_counters, 1u << 30);
}

matkv_status matkv_materialize(matkv_ctx* c, const void* hidden, const void* w_k, const void* w_v,
                               int32_t n_tokens, int64_t pos0, void* k_out, void* v_out,
                               int64_t token_stride) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!hidden || !w_k || !w_v || !k_out || !v_out) return fail(c, MATKV_EINVAL, "materialize: null pointer");
    if (!aligned16(hidden) || !aligned16(w_k) || !aligned16(w_v) || !aligned16(k_out) || !aligned16(v_out))
        return fail(c, MATKV_EINVAL, "materialize: pointers must be 16-byte aligned");
    if (n_tokens < 0 || pos0 < 0 || token_stride < n_tokens)
        return fail(c, MATKV_EINVAL, "materialize: n_tokens=%d pos0=%lld token_stride=%lld", n_tokens,
                    (long long)pos0, (long long)token_stride);
    if (pos0 + n_tokens > (1ll << 24)) return fail(c, MATKV_EINVAL, "materialize: positions beyond 2^24");
    if (n_tokens == 0) return MATKV_OK;
    MaterializeArgs a{};
    a.hidden = hidden; a.w_k = w_k; a.w_v = w_v; a.k_out = k_out; a.v_out = v_out;
    a.rope = reinterpret_cast<const RopeEntry*>(c->workspace + c->wl.off_rope);
    a.table = nullptr; a.off_inst = 0;
    a.pos0 = pos0; a.token_stride = token_stride; a.n_tokens = n_tokens;
    a.rows_per_instance = 0; a.batch = 1;
    a.Hkv = c->cfg.n_kv_heads; a.D = c->cfg.head_dim; a.Hd = c->cfg.hidden;
    materialize_scratch(c, a);
    HIP_TRY(c, launch_materialize(a, c->cfg.dtype, c->compute));
    return MATKV_OK;
}

matkv_status matkv_compress(matkv_ctx* c, const void* blob, int32_t n_tokens, void* out) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!blob || !out) return fail(c, MATKV_EINVAL, "compress: null pointer");
    if (!aligned16(blob) || !aligned16(out)) return fail(c, MATKV_EINVAL, "compress: pointers must be 16-byte aligned");
    if (c->cfg.dtype != MATKV_BF16) return fail(c, MATKV_EUNSUPPORTED, "compress: bf16 configurations only");
    if (n_tokens < 1) return fail(c, MATKV_EINVAL, "compress: n_tokens=%d", n_tokens);
    const char* a = static_cast<const char*>(blob);
    const char* b = static_cast<const char*>(out);
    if (a < b + matkv_compressed_blob_bytes(&c->cfg, n_tokens) && b < a + matkv_blob_bytes(&c->cfg, n_tokens))
        return fail(c, MATKV_EINVAL, "compress: output overlaps the blob");
    HIP_TRY(c, launch_compress(blob, out, c->cfg.n_layers, c->cfg.n_kv_heads, n_tokens, c->cfg.head_dim,
                               reinterpret_cast<float*>(c->workspace + c->wl.off_partials), c->wl.partial_floats, c->compute));
    return MATKV_OK;
}

matkv_status matkv_materialize_tail(matkv_ctx* c, const void* hidden, const void* w_k, const void* w_v,
                                    const void* table, int32_t rows_per_instance, void* tail_k,
                                    void* tail_v) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    MATKV_TRY
    if (!hidden || !w_k || !w_v || !table || !tail_k || !tail_v)
        return fail(c, MATKV_EINVAL, "materialize_tail: null pointer");
    if (!aligned16(hidden) || !aligned16(w_k) || !aligned16(w_v) || !aligned16(tail_k) || !aligned16(tail_v))
        return fail(c, MATKV_EINVAL, "materialize_tail: pointers must be 16-byte aligned");
    TableHost* th = find_table(c, table);
    if (!th) return fail(c, MATKV_EINVAL, "materialize_tail: table was not built by matkv_assemble");
    if (rows_per_instance == 0) return fail(c, MATKV_EINVAL, "materialize_tail: rows_per_instance is 0");
    note_table_use(c, table, *th, rows_per_instance < 0);
    if (rows_per_instance > 0 && rows_per_instance > th->min_tail_len)
        return fail(c, MATKV_EINVAL, "materialize_tail: %d newest rows but a tail holds only %d",
                    rows_per_instance, th->min_tail_len);
    MaterializeArgs a{};
    a.hidden = hidden; a.w_k = w_k; a.w_v = w_v; a.k_out = tail_k; a.v_out = tail_v;
    a.rope = reinterpret_cast<const RopeEntry*>(c->workspace + c->wl.off_rope);
    a.table = reinterpret_cast<const char*>(table); a.off_inst = c->tl.off_inst;
    a.pos0 = 0; a.token_stride = c->cfg.max_tail_tokens;
    a.rows_per_instance = rows_per_instance; a.batch = th->batch;
    a.n_tokens = rows_per_instance > 0 ? th->batch * rows_per_instance : th->total_q;
    a.Hkv = c->cfg.n_kv_heads; a.D = c->cfg.head_dim; a.Hd = c->cfg.hidden;
    materialize_scratch(c, a);
    HIP_TRY(c, launch_materialize(a, c->cfg.dtype, c->compute));
    return MATKV_OK;
    MATKV_CATCH(c, "materialize_tail")
}

// ------------------------------------------------------------------------------------ L ----

// Where a file load stands: 0 = all its copies are on the load stream (or it is no file load),
// 1 = pieces still to be read, 2 = a read failed.  block: wait until it is not 1.
static int file_state(matkv_ctx* c, Ticket* t, bool block) {
    std::unique_lock<std::mutex> lk(c->io_mu);
    if (block) c->io_done.wait(lk, [&] { return !t->queued; });
    if (t->queued) return 1;
    return t->failed ? 2 : 0;
}
static matkv_status file_failed(matkv_ctx* c) {
    std::lock_guard<std::mutex> lk(c->io_mu);
    return fail(c, MATKV_EIO, "%s", c->io_err);
}

// Checks shared by both load entry points; on success *t_out is the ticket record to fill and
// the load stream has been ordered after compute work that may still read the slot.
static matkv_status load_prepare(matkv_ctx* c, const char* name, size_t bytes, int32_t n_tokens,
                                 void* device_slot, size_t slot_bytes, Ticket** t_out) {
    // a copy ordered behind the compute stream would pull the load stream and the ticket's event
    // into the recording
    if (c->capturing) return fail(c, MATKV_EBUSY, "%s: not allowed while a graph is being captured", name);
    if (n_tokens < 1) return fail(c, MATKV_EINVAL, "%s: n_tokens=%d", name, n_tokens);
    const size_t want = matkv_blob_bytes(&c->cfg, n_tokens), want_c = matkv_compressed_blob_bytes(&c->cfg, n_tokens);
    if (bytes != want && bytes != want_c)
        return fail(c, MATKV_EINVAL, "%s: %zu bytes given, a %d-token blob has %zu (compressed: %zu)", name, bytes, n_tokens, want, want_c);
    if (slot_bytes < bytes) return fail(c, MATKV_EINVAL, "%s: slot of %zu bytes cannot hold %zu", name, slot_bytes, bytes);
    if (!aligned16(device_slot)) return fail(c, MATKV_EINVAL, "%s: pointers must be 16-byte aligned", name);
    hipPointerAttribute_t attr;
    hipError_t pe = hipPointerGetAttributes(&attr, device_slot);
    if (pe != hipSuccess || attr.type != hipMemoryTypeDevice) {
        (void)hipGetLastError();
        return fail(c, MATKV_EINVAL, "%s: slot is not device memory", name);
    }
    Ticket& t = c->tickets[c->next_ticket % kTicketRing];
    if (t.id != 0 && !t.done) {
        if (file_state(c, &t, false) == 1) return fail(c, MATKV_EBUSY, "%s: %d tickets outstanding", name, kTicketRing);
        hipError_t q = hipEventQuery(t.ev);
        if (q == hipErrorNotReady) { (void)hipGetLastError(); return fail(c, MATKV_EBUSY, "%s: %d tickets outstanding", name, kTicketRing); }
        if (q != hipSuccess) return hip_fail(c, q, "hipEventQuery");
        t.done = true;
    }
    if (!t.ev) HIP_TRY(c, hipEventCreateWithFlags(&t.ev, hipEventDisableTiming));
    SlotState& s = c->slots[device_slot];
    if (s.pending) {
        // a file load into this slot whose pieces are still being read: a second load would mix
        // its copies with theirs on the load stream
        Ticket& prev = c->tickets[s.pending % kTicketRing];
        if (prev.id == s.pending && file_state(c, &prev, false) == 1)
            return fail(c, MATKV_EBUSY, "%s: a load from a file into this slot is still being read", name);
    }
    if (s.refs > 0) {
        // a live table still points into the slot: order the copy after all compute work so far
        HIP_TRY(c, hipEventRecord(c->fence_ev, c->compute));
        HIP_TRY(c, hipStreamWaitEvent(c->load, c->fence_ev, 0));
    } else if (s.release) {
        // its last table was re-assembled onto other slots: the copy waits for the work that was
        // enqueued up to that moment, not for what has been enqueued since
        HIP_TRY(c, hipStreamWaitEvent(c->load, s.release, 0));
    }
    s.release = nullptr;
    *t_out = &t;
    return MATKV_OK;
}

// The copies of a load are on the load stream: record the ticket's event behind them.
static matkv_status load_finish(matkv_ctx* c, Ticket* t, void* device_slot, matkv_ticket* out) {
    HIP_TRY(c, hipEventRecord(t->ev, c->load));
    t->id = c->next_ticket++;
    t->slot = device_slot;
    t->done = false; t->queued = false; t->failed = false;
    SlotState& s = c->slots[device_slot];
    s.pending = t->id;
    s.waited = false;
    out->id = t->id;
    return MATKV_OK;
}

matkv_status matkv_load(matkv_ctx* c, const void* host_blob, size_t bytes, int32_t n_tokens,
                        void* device_slot, size_t slot_bytes, matkv_ticket* out) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    MATKV_TRY
    if (!host_blob || !device_slot || !out) return fail(c, MATKV_EINVAL, "load: null pointer");
    if (!aligned16(host_blob)) return fail(c, MATKV_EINVAL, "load: pointers must be 16-byte aligned");
    hipPointerAttribute_t attr;
    hipError_t pe = hipPointerGetAttributes(&attr, host_blob);
    if (pe != hipSuccess) { (void)hipGetLastError(); return fail(c, MATKV_EINVAL, "load: host blob is not pinned memory"); }
    if (attr.type != hipMemoryTypeHost) return fail(c, MATKV_EINVAL, "load: host blob is not pinned host memory");
    Ticket* t;
    st = load_prepare(c, "load", bytes, n_tokens, device_slot, slot_bytes, &t);
    if (st != MATKV_OK) return st;
    HIP_TRY(c, hipMemcpyAsync(device_slot, host_blob, bytes, hipMemcpyHostToDevice, c->load));
    return load_finish(c, t, device_slot, out);
    MATKV_CATCH(c, "load")
}

// ---- loads from a file: reader threads owned by the context -------------------------------
// matkv_load_file queues a request and returns.  kIoReaders threads take the queued requests
// piece by piece (8 MiB, several preads in flight at different offsets), each into one of its own
// two pinned bounce buffers - through a plain page-aligned buffer of its own where direct I/O
// cannot target pinned memory - and enqueue the piece's copy on the load stream.  The thread
// that finishes a request's last piece records the ticket's event behind all its copies.
constexpr int kIoReaders = 3;
static_assert(kBounceRing >= 2 * kIoReaders, "two bounce buffers per reader");

static void io_reader_main(matkv_ctx* c, int reader) {
    (void)hipSetDevice(c->device);
    char* plain = nullptr;
    int flip = 0;
    std::unique_lock<std::mutex> lk(c->io_mu);
    for (;;) {
        matkv_ctx::FileReq* rq = nullptr;
        c->io_work.wait(lk, [&] {
            if (c->io_stop) return true;
            for (auto& r : c->io_queue) if (r.next_piece < r.n_pieces) { rq = &r; return true; }
            return false;
        });
        if (c->io_stop) break;
        const size_t k = rq->next_piece++;
        const bool skip = rq->ticket->failed;           // an earlier piece failed: nothing more is read
        lk.unlock();

        char why[200] = {0};
        if (!skip) {
            Staging& b = c->bounce[2 * reader + flip];
            flip ^= 1;
            hipError_t he = b.used ? hipEventSynchronize(b.ev) : hipSuccess;     // its last copy has left the buffer
            const size_t piece = std::min(kBounceBytes, rq->bytes - k * kBounceBytes);
            const uint64_t at = rq->offset + k * kBounceBytes;
            size_t got = 0;
            while (he == hipSuccess && !why[0] && got < piece) {
                const bool via_plain = c->read_via_plain.load();
                if (via_plain && !plain && posix_memalign(reinterpret_cast<void**>(&plain), 4096, kBounceBytes) != 0) {
                    plain = nullptr;
                    snprintf(why, sizeof(why), "out of host memory");
                    break;
                }
                char* dest = via_plain ? plain : b.host;
                const ssize_t r = pread(rq->fd, dest + got, piece - got, (off_t)(at + got));
                if (r < 0 && errno == EINTR) continue;
                if (r < 0 && errno == EFAULT && !via_plain) {
                    // direct I/O cannot pin the device-mapped bounce buffer on this system: from now
                    // on read into plain page-aligned memory and copy into the bounce buffer
                    c->read_via_plain.store(true);
                    got = 0;
                    continue;
                }
                if (r < 0) snprintf(why, sizeof(why), "pread at %llu: %s", (unsigned long long)(at + got), strerror(errno));
                else if (r == 0) snprintf(why, sizeof(why), "file ends %llu bytes short of the blob",
                                          (unsigned long long)(rq->offset + rq->bytes - (at + got)));
                else got += (size_t)r;
            }
            if (he == hipSuccess && !why[0]) {
                if (c->read_via_plain.load()) memcpy(b.host, plain, piece);
                he = hipMemcpyAsync(rq->dst + k * kBounceBytes, b.host, piece, hipMemcpyHostToDevice, c->load);
                if (he == hipSuccess) he = hipEventRecord(b.ev, c->load);
                b.used = true;
            }
            if (he != hipSuccess) {
                (void)hipGetLastError();
                snprintf(why, sizeof(why), "copy of a piece: %s", hipGetErrorString(he));
            }
        }

        lk.lock();
        if (why[0] && !rq->ticket->failed) {
            rq->ticket->failed = true;
            snprintf(c->io_err, sizeof(c->io_err), "load_file: %s", why);
        }
        if (++rq->pieces_done == rq->n_pieces) {
            // every copy of this request is on the load stream (or the request was given up)
            if (hipEventRecord(rq->ticket->ev, c->load) != hipSuccess) {
                (void)hipGetLastError();
                rq->ticket->failed = true;
            }
            rq->ticket->queued = false;
            for (auto it = c->io_queue.begin(); it != c->io_queue.end(); ++it)
                if (&*it == rq) { c->io_queue.erase(it); break; }
            c->io_done.notify_all();
        }
    }
    free(plain);
}

// Blocks until no file load is queued or being read (the store path and the destructor share
// the bounce buffers with the readers).
static void io_drain(matkv_ctx* c) {
    std::unique_lock<std::mutex> lk(c->io_mu);
    c->io_done.wait(lk, [&] { return c->io_queue.empty(); });
}

static matkv_status bounce_buffers(matkv_ctx* c) {
    for (int i = 0; i < kBounceRing; ++i) {
        if (c->bounce[i].host) continue;
        HIP_TRY(c, hipHostMalloc(reinterpret_cast<void**>(&c->bounce[i].host), kBounceBytes, hipHostMallocDefault));
        HIP_TRY(c, hipEventCreateWithFlags(&c->bounce[i].ev, hipEventDisableTiming));
    }
    return MATKV_OK;
}

matkv_status matkv_load_file(matkv_ctx* c, int fd, uint64_t offset, size_t bytes, int32_t n_tokens,
                             void* device_slot, size_t slot_bytes, matkv_ticket* out) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    MATKV_TRY
    if (fd < 0 || !device_slot || !out) return fail(c, MATKV_EINVAL, "load_file: bad descriptor or null pointer");
    Ticket* t;
    st = load_prepare(c, "load_file", bytes, n_tokens, device_slot, slot_bytes, &t);
    if (st != MATKV_OK) return st;
    st = bounce_buffers(c);
    if (st != MATKV_OK) return st;
    if (c->io_readers.empty()) {
        c->io_readers.reserve(kIoReaders);
        for (int r = 0; r < kIoReaders; ++r) c->io_readers.emplace_back(io_reader_main, c, r);
    }
    {
        std::lock_guard<std::mutex> lk(c->io_mu);
        t->id = c->next_ticket++;
        t->slot = device_slot;
        t->done = false; t->queued = true; t->failed = false;
        matkv_ctx::FileReq rq{};
        rq.fd = fd; rq.offset = offset; rq.bytes = bytes; rq.dst = static_cast<char*>(device_slot); rq.ticket = t;
        rq.n_pieces = (bytes + kBounceBytes - 1) / kBounceBytes; rq.next_piece = 0; rq.pieces_done = 0;
        c->io_queue.push_back(rq);
    }
    c->io_work.notify_all();
    SlotState& s = c->slots[device_slot];
    s.pending = t->id;
    s.waited = false;
    out->id = t->id;
    return MATKV_OK;
    MATKV_CATCH(c, "load_file")
}

matkv_status matkv_store_file(matkv_ctx* c, int fd, uint64_t offset, const void* device_blob, size_t bytes) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (fd < 0 || !device_blob || bytes == 0) return fail(c, MATKV_EINVAL, "store_file: bad descriptor, null pointer or no bytes");
    if (c->capturing) return fail(c, MATKV_EBUSY, "store_file: not allowed while a graph is being captured");
    hipPointerAttribute_t attr;
    hipError_t pe = hipPointerGetAttributes(&attr, device_blob);
    if (pe != hipSuccess || attr.type != hipMemoryTypeDevice) {
        (void)hipGetLastError();
        return fail(c, MATKV_EINVAL, "store_file: blob is not device memory");
    }
    st = bounce_buffers(c);
    if (st != MATKV_OK) return st;
    io_drain(c);                             // the reader threads use the same bounce buffers
    // the blob was produced on the compute stream: the copies out follow what is enqueued there
    HIP_TRY(c, hipEventRecord(c->fence_ev, c->compute));
    HIP_TRY(c, hipStreamWaitEvent(c->load, c->fence_ev, 0));
    // piece k is written to the file while the copy of piece k+1 is in flight
    const size_t n_pieces = (bytes + kBounceBytes - 1) / kBounceBytes;
    auto piece_bytes = [&](size_t k) { return std::min(kBounceBytes, bytes - k * kBounceBytes); };
    auto enqueue = [&](size_t k) -> hipError_t {
        Staging& b = c->bounce[k % kBounceRing];
        if (b.used) { hipError_t e = hipEventSynchronize(b.ev); if (e != hipSuccess) return e; }
        hipError_t e = hipMemcpyAsync(b.host, static_cast<const char*>(device_blob) + k * kBounceBytes, piece_bytes(k),
                                      hipMemcpyDeviceToHost, c->load);
        if (e == hipSuccess) e = hipEventRecord(b.ev, c->load);
        b.used = true;
        return e;
    };
    HIP_TRY(c, enqueue(0));
    for (size_t k = 0; k < n_pieces; ++k) {
        if (k + 1 < n_pieces) HIP_TRY(c, enqueue(k + 1));
        Staging& b = c->bounce[k % kBounceRing];
        HIP_TRY(c, hipEventSynchronize(b.ev));
        const char* src = b.host;
        const size_t piece = piece_bytes(k);
        if (c->read_via_plain.load()) {
            if (!c->plain_buf && posix_memalign(reinterpret_cast<void**>(&c->plain_buf), 4096, kBounceBytes) != 0) {
                c->plain_buf = nullptr;
                return fail(c, MATKV_ENOMEM, "store_file: out of host memory");
            }
            memcpy(c->plain_buf, b.host, piece);
            src = c->plain_buf;
        }
        size_t put = 0;
        while (put < piece) {
            ssize_t r = pwrite(fd, src + put, piece - put, (off_t)(offset + k * kBounceBytes + put));
            if (r < 0 && errno == EINTR) continue;
            if (r < 0 && errno == EFAULT && !c->read_via_plain.load()) {
                // direct I/O cannot pin the device-mapped bounce buffer on this system (see the reader threads)
                if (!c->plain_buf && posix_memalign(reinterpret_cast<void**>(&c->plain_buf), 4096, kBounceBytes) != 0) {
                    c->plain_buf = nullptr;
                    return fail(c, MATKV_ENOMEM, "store_file: out of host memory");
                }
                c->read_via_plain.store(true);
                memcpy(c->plain_buf, b.host, piece);
                src = c->plain_buf;
                continue;
            }
            if (r <= 0) return fail(c, MATKV_EIO, "store_file: pwrite at %llu: %s", (unsigned long long)(offset + k * kBounceBytes + put),
                                    r < 0 ? strerror(errno) : "no progress");
            put += (size_t)r;
        }
    }
    return MATKV_OK;
}

static matkv_status ticket_lookup(matkv_ctx* c, matkv_ticket tk, Ticket** out) {
    if (tk.id == 0 || tk.id >= c->next_ticket) return fail(c, MATKV_EINVAL, "ticket %llu was never issued", (unsigned long long)tk.id);
    Ticket& t = c->tickets[tk.id % kTicketRing];
    if (t.id != tk.id) { *out = nullptr; return MATKV_OK; }   // ring slot reused: that copy finished long ago
    *out = &t;
    return MATKV_OK;
}

matkv_status matkv_wait(matkv_ctx* c, matkv_ticket tk) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    Ticket* t;
    st = ticket_lookup(c, tk, &t);
    if (st != MATKV_OK || !t) return st;
    // a file load still being read: the event is not recorded yet, so the host waits here until
    // the last piece's copy is on the load stream (the copies themselves are not waited for)
    if (!t->done && file_state(c, t, true) == 2) return file_failed(c);
    if (!t->done) HIP_TRY(c, hipStreamWaitEvent(c->compute, t->ev, 0));
    auto it = c->slots.find(t->slot);
    if (it != c->slots.end() && it->second.pending == tk.id) it->second.waited = true;
    return MATKV_OK;
}

matkv_status matkv_query(matkv_ctx* c, matkv_ticket tk) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    Ticket* t;
    st = ticket_lookup(c, tk, &t);
    if (st != MATKV_OK || !t) return st;
    if (t->done) return MATKV_OK;
    const int fs = file_state(c, t, false);
    if (fs == 1) return MATKV_ENOTREADY;
    if (fs == 2) return file_failed(c);
    hipError_t q = hipEventQuery(t->ev);
    if (q == hipErrorNotReady) { (void)hipGetLastError(); return MATKV_ENOTREADY; }
    if (q != hipSuccess) return hip_fail(c, q, "hipEventQuery");
    t->done = true;
    return MATKV_OK;
}

matkv_status matkv_sync(matkv_ctx* c, matkv_ticket tk) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    Ticket* t;
    st = ticket_lookup(c, tk, &t);
    if (st != MATKV_OK || !t) return st;
    if (!t->done && file_state(c, t, true) == 2) {
        (void)hipEventSynchronize(t->ev);     // the pieces that did get enqueued
        return file_failed(c);
    }
    if (!t->done) { HIP_TRY(c, hipEventSynchronize(t->ev)); t->done = true; }
    return MATKV_OK;
}

// A slot that was the target of a load nobody has waited for: if the copy has finished, the
// compute stream is ordered behind it (while a graph is being recorded nothing is ordered: a
// finished copy needs no edge) and the slot counts as waited for; if not, MATKV_ENOTREADY.
static matkv_status slot_ready(matkv_ctx* c, const void* slot, const char* name) {
    auto it = c->slots.find(slot);
    if (it == c->slots.end() || !it->second.pending || it->second.waited) return MATKV_OK;
    Ticket& t = c->tickets[it->second.pending % kTicketRing];
    bool done = (t.id != it->second.pending) || t.done;
    if (!done) {
        const int fs = file_state(c, &t, false);
        if (fs == 1) return fail(c, MATKV_ENOTREADY, "%s: a page's load from a file is still being read", name);
        if (fs == 2) return fail(c, MATKV_EIO, "%s: a page's load from a file failed", name);
        hipError_t q = hipEventQuery(t.ev);
        if (q == hipSuccess) { t.done = true; done = true; }
        else if (q == hipErrorNotReady) (void)hipGetLastError();
        else return hip_fail(c, q, "hipEventQuery");
    }
    if (!done) return fail(c, MATKV_ENOTREADY, "%s: a page's load has neither finished nor been waited for", name);
    if (t.id == it->second.pending && !c->capturing) HIP_TRY(c, hipStreamWaitEvent(c->compute, t.ev, 0));
    it->second.waited = true;
    return MATKV_OK;
}

// Every slot a table points into, before work that reads the table is enqueued: a load into one
// of them after the table was assembled must not race with that work.
static matkv_status table_pages_ready(matkv_ctx* c, const TableHost& th, const char* name) {
    for (const void* sl : th.slots) {
        matkv_status st = slot_ready(c, sl, name);
        if (st != MATKV_OK) return st;
    }
    return MATKV_OK;
}

// ------------------------------------------------------------------------------------ A ----

matkv_status matkv_assemble(matkv_ctx* c, const matkv_page* pages, const int32_t* n_pages,
                            const int32_t* q_len, const int64_t* pos_base, int32_t batch, void* table) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (c->capturing) return fail(c, MATKV_EBUSY, "assemble: not allowed while a graph is being captured");
    MATKV_TRY
    if (!n_pages || !q_len || !table) return fail(c, MATKV_EINVAL, "assemble: null pointer");
    if (!aligned16(table)) return fail(c, MATKV_EINVAL, "assemble: table must be 16-byte aligned");
    if (batch < 1 || batch > c->cfg.max_batch) return fail(c, MATKV_EINVAL, "assemble: batch=%d, max_batch=%d", batch, c->cfg.max_batch);
    const matkv_config& cfg = c->cfg;
    long total_tokens = 0;
    int kv_fmt = -1;                   // format of the table's pages (-1: none seen yet)
    for (int b = 0; b < batch; ++b) {
        if (n_pages[b] < 0 || n_pages[b] > cfg.max_pages) return fail(c, MATKV_EINVAL, "assemble: instance %d has %d pages, max_pages=%d", b, n_pages[b], cfg.max_pages);
        if (n_pages[b] > 0 && !pages) return fail(c, MATKV_EINVAL, "assemble: pages is null");
        if (q_len[b] < 1 || q_len[b] > cfg.max_tail_tokens) return fail(c, MATKV_EINVAL, "assemble: instance %d question length %d outside 1..%d", b, q_len[b], cfg.max_tail_tokens);
        if (pos_base && (pos_base[b] < 0 || pos_base[b] + cfg.max_tail_tokens > (1ll << 24))) return fail(c, MATKV_EINVAL, "assemble: instance %d pos_base out of range", b);
        for (int p = 0; p < n_pages[b]; ++p) {
            const matkv_page& pg = pages[(size_t)b * cfg.max_pages + p];
            if (!pg.slot || !aligned16(pg.slot) || pg.n_tokens < 1)
                return fail(c, MATKV_EINVAL, "assemble: instance %d page %d is invalid", b, p);
            if (pg.format != MATKV_PAGE_PLAIN && pg.format != MATKV_PAGE_E4M3)
                return fail(c, MATKV_EINVAL, "assemble: instance %d page %d has unknown format %d", b, p, pg.format);
            if (kv_fmt < 0) kv_fmt = pg.format;
            if (pg.format != kv_fmt) return fail(c, MATKV_EUNSUPPORTED, "assemble: plain and compressed pages in one table");
            st = slot_ready(c, pg.slot, "assemble");
            if (st == MATKV_ENOTREADY) return fail(c, MATKV_ENOTREADY, "assemble: instance %d page %d: load neither finished nor waited for", b, p);
            if (st != MATKV_OK) return st;
            total_tokens += pg.n_tokens;
        }
    }

    (void)total_tokens;
    if (kv_fmt < 0) kv_fmt = MATKV_PAGE_PLAIN;
    if (kv_fmt == MATKV_PAGE_E4M3 && !(cfg.dtype == MATKV_BF16 && cfg.head_dim == 128))
        return fail(c, MATKV_EUNSUPPORTED, "assemble: compressed pages need bf16 and head_dim 128");
    auto scales_off = [&](int n_tokens) { return kv_fmt == MATKV_PAGE_E4M3 ? compressed_codes_bytes(cfg, n_tokens) : (size_t)0; };
    Staging& sg = c->staging[c->staging_next];
    c->staging_next = (c->staging_next + 1) % kStagingRing;
    if (sg.used) HIP_TRY(c, hipEventSynchronize(sg.ev));
    char* h = sg.host;
    TableHeader* hdr = reinterpret_cast<TableHeader*>(h);
    InstanceInfo* insts = reinterpret_cast<InstanceInfo*>(h + c->tl.off_inst);
    Item* items = reinterpret_cast<Item*>(h + c->tl.off_items);
    Unit* dunits = reinterpret_cast<Unit*>(h + c->tl.off_dunits);
    Unit* punits = reinterpret_cast<Unit*>(h + c->tl.off_punits);
    memset(hdr, 0, sizeof(*hdr));
    int n_items = 0, cu = 0, max_q = 0;
    TableHost th;
    th.min_tail_len = cfg.max_tail_tokens;
    for (int b = 0; b < batch; ++b) {
        InstanceInfo& in = insts[b];
        memset(&in, 0, sizeof(in));
        const matkv_page* pg = pages ? pages + (size_t)b * cfg.max_pages : nullptr;
        long inst_tokens = 0;
        for (int p = 0; p < n_pages[b]; ++p) {
            inst_tokens += pg[p].n_tokens;
        }
        in.pos_base = pos_base ? pos_base[b] : inst_tokens;
        if (in.pos_base + cfg.max_tail_tokens > (1ll << 24)) return fail(c, MATKV_EINVAL, "assemble: positions beyond 2^24");
        in.tail_len = q_len[b];
        in.q_len = q_len[b];
        in.cu_q = cu;
        cu += q_len[b];
        if (q_len[b] > max_q) max_q = q_len[b];
        if (q_len[b] > th.max_tail_len) th.max_tail_len = q_len[b];
        if (q_len[b] < th.min_tail_len) th.min_tail_len = q_len[b];
    }
    const DecodeLayout decode = lay_out_decode(cfg, c->tl, pages, n_pages, batch, kv_fmt, insts, items, &n_items, dunits,
                                               reinterpret_cast<SUnit*>(h + c->tl.off_sunits), scales_off);
    const int n_dunits = decode.n_dunits, n_sunits = decode.n_sunits;
    th.even = decode.even; th.past_llc = decode.past_llc; th.tail_spared = decode.tail_spared;
    th.step_by_instance = decode.step_by_instance; th.step_past_llc = decode.step_past_llc;
    // prefill: coarse partition (the question rows supply most of the parallelism)
    th.prefill = lay_out_prefill(cfg, pages, n_pages, q_len, batch, kv_fmt == MATKV_PAGE_E4M3, insts, items, &n_items, punits, scales_off);
    const size_t dunit_bytes = sizeof(Unit) * n_dunits + (decode.even_built ? sizeof(SUnit) * (256 / cfg.n_kv_heads) : 0);
    hdr->batch = batch; hdr->n_items = n_items; hdr->n_dunits = n_dunits; hdr->n_punits = th.prefill.n_units;
    hdr->total_q = cu; hdr->max_q = max_q;

    char* d = reinterpret_cast<char*>(table);
    const TableSections sec = {{0, c->tl.off_items, c->tl.off_dunits, c->tl.off_punits, c->tl.off_sunits},
                               {c->tl.off_inst + sizeof(InstanceInfo) * batch, sizeof(Item) * n_items, dunit_bytes, sizeof(Unit) * th.prefill.n_units,
                                sizeof(SUnit) * n_sunits}};
    size_t vecs = 0;
    for (size_t n : sec.bytes) vecs += n / 16;
    hipLaunchKernelGGL(table_copy_kernel, dim3((unsigned)((vecs + 255) / 256)), dim3(256), 0, c->compute, sg.host_on_device, d, sec);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipEventRecord(sg.ev, c->compute));
    sg.used = true;

    th.batch = batch; th.n_items = n_items; th.n_dunits = n_dunits;
    th.total_q = cu; th.max_q = max_q; th.kv_fmt = kv_fmt; th.n_sunits = n_sunits;
    th.n_decode_slots = n_dunits;
    if (n_sunits > 0 || th.even) {
        th.n_decode_slots = 0;
        for (int b = 0; b < batch; ++b) th.n_decode_slots = std::max(th.n_decode_slots, insts[b].sslot0 + insts[b].n_sslots);
    }
    sign_partition(th);
    // Slot bookkeeping: the table's old contents are dead from here on in stream order, so the
    // slots only they pointed into may be overwritten once the work enqueued so far is done.
    for (int b = 0; b < batch; ++b) {
        const matkv_page* pg = pages ? pages + (size_t)b * cfg.max_pages : nullptr;
        for (int p = 0; p < n_pages[b]; ++p)
            if (std::find(th.slots.begin(), th.slots.end(), pg[p].slot) == th.slots.end()) th.slots.push_back(pg[p].slot);
    }
    auto old = c->tables.find(table);
    if (old != c->tables.end() && !old->second.slots.empty()) {
        hipEvent_t& ev = c->release_ev[c->release_next];
        c->release_next = (c->release_next + 1) % kReleaseRing;
        if (!ev) HIP_TRY(c, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        HIP_TRY(c, hipEventRecord(ev, c->compute));
        for (const void* sl : old->second.slots) {
            SlotState& ss = c->slots[sl];
            if (ss.refs > 0) --ss.refs;
            if (ss.refs == 0) ss.release = ev;
        }
    }
    for (const void* sl : th.slots) ++c->slots[sl].refs;
    c->tables[table] = th;
    return MATKV_OK;
    MATKV_CATCH(c, "assemble")
}

int32_t matkv_plan_decode_units_of(const matkv_config* cfg, const int32_t* page_tokens, int32_t n_pages, int32_t batch, int32_t q_len,
                                   int32_t format, int32_t* unit_tokens_out, int32_t* unit_items_out, int32_t cap) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return -1;
    MATKV_TRY
    if (n_pages < 0 || n_pages > cfg->max_pages || (n_pages > 0 && !page_tokens) || batch < 1 ||
        batch > cfg->max_batch || q_len < 1 || q_len > cfg->max_tail_tokens || cap < 0)
        return -1;
    if ((format != MATKV_PAGE_PLAIN && format != MATKV_PAGE_E4M3) || (format == MATKV_PAGE_E4M3 && !(cfg->dtype == MATKV_BF16 && cfg->head_dim == 128))) return -1;
    std::vector<matkv_page> pages((size_t)(n_pages > 0 ? n_pages : 1));
    long inst_tokens = 0;
    for (int p = 0; p < n_pages; ++p) {
        if (page_tokens[p] < 1) return -1;
        pages[p].slot = reinterpret_cast<const void*>((uintptr_t)0x1000);   // never dereferenced
        pages[p].n_tokens = page_tokens[p];
        pages[p].format = format;
        inst_tokens += page_tokens[p];
    }
    const DecodeCut c = decode_cut(*cfg, batch, inst_tokens, n_pages, q_len, format);
    std::vector<Item> items((size_t)kMaxDecodeUnitsPerInstance + n_pages + 2);
    std::vector<Unit> units((size_t)kMaxDecodeUnitsPerInstance);
    int n_items = 0, n_units = 0;
    const int made = build_units(pages.data(), n_pages, 0, c.units, c.tail_tokens, cfg->max_tail_tokens, items.data(), &n_items, units.data(), &n_units,
                                 [](int) { return (size_t)0; });
    for (int u = 0; u < made && u < cap; ++u) {
        if (unit_tokens_out) unit_tokens_out[u] = units[u].page_tokens;
        if (unit_items_out) unit_items_out[u] = units[u].n_items - units[u].has_tail;
    }
    return made < cap ? made : cap;
    MATKV_CATCH_INT
}

int32_t matkv_plan_decode_units(const matkv_config* cfg, const int32_t* page_tokens, int32_t n_pages, int32_t batch, int32_t q_len,
                                int32_t* unit_tokens_out, int32_t* unit_items_out, int32_t cap) {
    return matkv_plan_decode_units_of(cfg, page_tokens, n_pages, batch, q_len, MATKV_PAGE_PLAIN, unit_tokens_out, unit_items_out, cap);
}

int32_t matkv_plan_projection(const matkv_config* cfg, int32_t n_rows) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK || n_rows < 1) return -1;
    return (int32_t)projection_form(cfg->hidden, cfg->n_kv_heads, cfg->head_dim, cfg->dtype, n_rows);
}

int32_t matkv_plan_prefill(const matkv_config* cfg, const int32_t* page_tokens, const int32_t* n_pages, const int32_t* q_len,
                           int32_t batch, int32_t format, int32_t* units_out) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return -1;
    if (!n_pages || !q_len || batch < 1 || batch > cfg->max_batch || (format != MATKV_PAGE_PLAIN && format != MATKV_PAGE_E4M3)) return -1;
    const bool row_tiles = cfg->dtype == MATKV_BF16 && cfg->head_dim == 128;
    if (format == MATKV_PAGE_E4M3 && !row_tiles) return -1;
    MATKV_TRY
    std::vector<matkv_page> pages((size_t)batch * std::max(cfg->max_pages, 1));
    std::vector<InstanceInfo> insts((size_t)batch);
    for (int b = 0; b < batch; ++b) {
        if (n_pages[b] < 0 || n_pages[b] > cfg->max_pages || q_len[b] < 1 || q_len[b] > cfg->max_tail_tokens) return -1;
        if (n_pages[b] > 0 && !page_tokens) return -1;
        for (int p = 0; p < n_pages[b]; ++p) {
            const size_t i = (size_t)b * cfg->max_pages + p;
            if (page_tokens[i] < 1) return -1;
            pages[i].slot = reinterpret_cast<const void*>((uintptr_t)0x1000);     // never dereferenced
            pages[i].n_tokens = page_tokens[i];
            pages[i].format = format;
        }
    }
    const TableLayout tl = table_layout(*cfg);
    std::vector<Item> items((size_t)tl.max_items);
    std::vector<Unit> units((size_t)tl.max_punits);
    int n_items = 0;
    const PrefillLayout L = lay_out_prefill(*cfg, pages.data(), n_pages, q_len, batch, format == MATKV_PAGE_E4M3, insts.data(), items.data(),
                                            &n_items, units.data(), [](int) { return (size_t)0; });
    if (units_out) for (int b = 0; b < batch; ++b) units_out[b] = insts[b].n_punits;
    return row_tiles && L.row_tiles ? L.tile_rows : 0;
    MATKV_CATCH_INT
}

// The pages and instances of a batch as a preview gets them; ids: equal ones mean the same slot.  False on a bad argument.
static bool preview_batch(const matkv_config& cfg, const int32_t* ids, const int32_t* tokens, const int32_t* n_pages, const int32_t* q_len,
                          int32_t batch, int32_t format, std::vector<matkv_page>& pages, std::vector<InstanceInfo>& insts) {
    pages.resize((size_t)batch * std::max(cfg.max_pages, 1));
    insts.resize((size_t)batch);
    for (int b = 0; b < batch; ++b) {
        if (n_pages[b] < 0 || n_pages[b] > cfg.max_pages || q_len[b] < 1 || q_len[b] > cfg.max_tail_tokens) return false;
        if (n_pages[b] > 0 && (!ids || !tokens)) return false;
        memset(&insts[b], 0, sizeof(InstanceInfo));
        insts[b].q_len = q_len[b];
        for (int p = 0; p < n_pages[b]; ++p) {
            const size_t i = (size_t)b * cfg.max_pages + p;
            if (ids[i] < 0 || tokens[i] < 1) return false;
            pages[i].slot = reinterpret_cast<const void*>(((uintptr_t)ids[i] + 1) * 4096);   // never dereferenced
            pages[i].n_tokens = tokens[i];
            pages[i].format = format;
        }
    }
    return true;
}

int32_t matkv_plan_shared_units(const matkv_config* cfg, const int32_t* page_ids, const int32_t* page_tokens,
                                const int32_t* n_pages, const int32_t* q_len, int32_t batch,
                                int32_t* units_out, int32_t cap, int32_t* slots_out) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return -1;
    if (!n_pages || !q_len || batch < 1 || batch > cfg->max_batch || cap < 0 || (cap > 0 && !units_out)) return -1;
    MATKV_TRY
    const int grp = cfg->n_q_heads / cfg->n_kv_heads;
    std::vector<matkv_page> pages;
    std::vector<InstanceInfo> insts;
    if (!preview_batch(*cfg, page_ids, page_tokens, n_pages, q_len, batch, MATKV_PAGE_PLAIN, pages, insts)) return -1;
    // the conditions of matkv_assemble
    if (batch < 2 || cfg->decode_units != 0 || cfg->decode_variant != 0 || cfg->dtype != MATKV_BF16 ||
        cfg->head_dim != 128 || !group_size_built(grp))
        return 0;
    const TableLayout tl = table_layout(*cfg);
    std::vector<Item> items((size_t)tl.max_items);
    std::vector<SUnit> sunits((size_t)tl.max_sunits);
    int n_items = 0;
    std::vector<int32_t> user_tokens((size_t)tl.max_sunits * kMaxSharedUsers);
    const int n = build_shared_units(*cfg, pages.data(), n_pages, batch, tl.max_sunits, tl.max_items, insts.data(),
                                     items.data(), &n_items, sunits.data(), MATKV_PAGE_PLAIN, user_tokens.data());
    for (int u = 0; u < n && u < cap; ++u) {
        const SUnit& su = sunits[u];
        int32_t* o = units_out + (size_t)u * (4 + 3 * kMaxSharedUsers);
        const uintptr_t base = (uintptr_t)su.u.first.base;
        o[0] = base ? (int32_t)(base / 4096 - 1) : -1;     // id of the unit's first page; -1: it starts with a tail
        o[1] = su.u.page_tokens;                            // page tokens the unit streams (all its pieces)
        o[2] = su.u.has_tail ? su.u.inst : -1;              // the instance whose tail it holds, or -1
        o[3] = su.n_users;
        for (int k = 0; k < kMaxSharedUsers; ++k) {
            o[4 + 3 * k] = k < su.n_users ? su.users[k].inst : -1;
            o[5 + 3 * k] = k < su.n_users ? su.users[k].slot : -1;
            o[6 + 3 * k] = k < su.n_users ? user_tokens[(size_t)u * kMaxSharedUsers + k] : 0;
        }
    }
    if (slots_out && n > 0)
        for (int b = 0; b < batch; ++b) { slots_out[2 * b] = insts[b].sslot0; slots_out[2 * b + 1] = insts[b].n_sslots; }
    return n < cap ? n : cap;
    MATKV_CATCH_INT
}

static int32_t plan_streams(const matkv_config* cfg, const int32_t* page_ids, const int32_t* page_tokens, const int32_t* n_pages,
                            const int32_t* q_len, int32_t batch, int32_t format, bool step) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return -1;
    if (!n_pages || !q_len || batch < 1 || batch > cfg->max_batch || (format != MATKV_PAGE_PLAIN && format != MATKV_PAGE_E4M3)) return -1;
    if (format == MATKV_PAGE_E4M3 && !(cfg->dtype == MATKV_BF16 && cfg->head_dim == 128)) return -1;
    MATKV_TRY
    std::vector<matkv_page> pages;
    std::vector<InstanceInfo> insts;
    if (!preview_batch(*cfg, page_ids, page_tokens, n_pages, q_len, batch, format, pages, insts)) return -1;
    const TableLayout tl = table_layout(*cfg);
    std::vector<Item> items((size_t)tl.max_items);
    std::vector<Unit> units((size_t)tl.max_dunits);
    std::vector<SUnit> sunits((size_t)tl.max_sunits);
    int n_items = 0;
    const DecodeLayout L = lay_out_decode(*cfg, tl, pages.data(), n_pages, batch, format, insts.data(), items.data(), &n_items, units.data(),
                                          sunits.data(), [](int) { return (size_t)0; });
    return step ? L.step_past_llc : L.past_llc;
    MATKV_CATCH_INT
}

int32_t matkv_plan_decode_streams(const matkv_config* cfg, const int32_t* page_ids, const int32_t* page_tokens, const int32_t* n_pages,
                                  const int32_t* q_len, int32_t batch, int32_t format) {
    return plan_streams(cfg, page_ids, page_tokens, n_pages, q_len, batch, format, false);
}

int32_t matkv_plan_step_streams(const matkv_config* cfg, const int32_t* page_ids, const int32_t* page_tokens, const int32_t* n_pages,
                                const int32_t* q_len, int32_t batch, int32_t format) {
    return plan_streams(cfg, page_ids, page_tokens, n_pages, q_len, batch, format, true);
}

int32_t matkv_plan_even_units(const matkv_config* cfg, const int32_t* page_tokens, const int32_t* n_pages, const int32_t* q_len, int32_t batch,
                              int32_t format, int32_t* units_out, int32_t cap, int32_t* slots_out, int32_t* taken_out) {
    const char* why;
    if (check_config(cfg, &why) != MATKV_OK) return -1;
    if (!n_pages || !q_len || batch < 1 || batch > cfg->max_batch || cap < 0 || (cap > 0 && !units_out)) return -1;
    if ((format != MATKV_PAGE_PLAIN && format != MATKV_PAGE_E4M3) || (format == MATKV_PAGE_E4M3 && !(cfg->dtype == MATKV_BF16 && cfg->head_dim == 128))) return -1;
    MATKV_TRY
    std::vector<matkv_page> pages;
    std::vector<InstanceInfo> insts;
    std::vector<int32_t> ids((size_t)batch * std::max(cfg->max_pages, 1));
    std::iota(ids.begin(), ids.end(), 0);
    if (!preview_batch(*cfg, ids.data(), page_tokens, n_pages, q_len, batch, format, pages, insts)) return -1;
    const TableLayout tl = table_layout(*cfg);
    std::vector<Item> items((size_t)tl.max_items);
    std::vector<Unit> units((size_t)tl.max_dunits);
    std::vector<SUnit> sunits((size_t)tl.max_sunits);
    int n_items = 0;
    const DecodeLayout L = lay_out_decode(*cfg, tl, pages.data(), n_pages, batch, format, insts.data(), items.data(), &n_items, units.data(),
                                          sunits.data(), [](int) { return (size_t)0; });
    if (!L.even_built) return 0;
    if (taken_out) *taken_out = L.even;
    const int n = 256 / cfg->n_kv_heads;
    for (int u = 0; u < n && u < cap; ++u) {
        const SUnit& su = reinterpret_cast<const SUnit*>(units.data() + L.n_dunits)[u];
        int32_t* o = units_out + (size_t)u * 8;
        int32_t seen[2] = {0, 0};
        for (int i = su.u.item0; i < su.u.item0 + su.u.n_items; ++i)
            for (int k = 0; k < 2; ++k) if (items[i].base && (items[i].umask >> k & 1)) seen[k] += items[i].ntok;
        o[0] = su.u.page_tokens;
        o[1] = su.u.has_tail ? su.u.inst : -1;
        for (int k = 0; k < 2; ++k) {
            o[2 + 3 * k] = k < su.n_users ? su.users[k].inst : -1;
            o[3 + 3 * k] = k < su.n_users ? su.users[k].slot : -1;
            o[4 + 3 * k] = k < su.n_users ? seen[k] : 0;
        }
    }
    if (slots_out)
        for (int b = 0; b < batch; ++b) { slots_out[2 * b] = insts[b].sslot0; slots_out[2 * b + 1] = insts[b].n_sslots; }
    return n < cap ? n : cap;
    MATKV_CATCH_INT
}

int32_t matkv_table_shared_units(matkv_ctx* c, const void* table) {
    if (!c) return -1;
    TableHost* th = find_table(c, table);
    return th ? th->n_sunits : -1;
}

matkv_status matkv_advance(matkv_ctx* c, void* table, int32_t n) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    TableHost* th = find_table(c, table);
    if (!th) return fail(c, MATKV_EINVAL, "advance: table was not built by matkv_assemble");
    if (n < 1) return fail(c, MATKV_EINVAL, "advance: n=%d", n);
    MATKV_TRY
    note_table_use(c, table, *th, false);
    if (c->capturing) {
        c->cap->advances.emplace_back(table, n);
    } else {
        if (th->max_tail_len + n > c->cfg.max_tail_tokens)
            return fail(c, MATKV_EINVAL, "advance: tail would hold %d tokens, max_tail_tokens=%d", th->max_tail_len + n, c->cfg.max_tail_tokens);
        th->max_tail_len += n; th->min_tail_len += n;
    }
    HIP_TRY(c, launch_advance(reinterpret_cast<char*>(table), c->tl.off_inst, th->batch, n, c->cfg.max_tail_tokens, c->compute));
    return MATKV_OK;
    MATKV_CATCH(c, "advance")
}

// -------------------------------------------------------------------------------- P / D ----

static matkv_status attn_args(matkv_ctx* c, const char* name, int prefill, int32_t layer, const void* q,
                              const void* table, const void* tail_k, const void* tail_v, void* out, AttnArgs* out_args) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!q || !table || !tail_k || !tail_v || !out) return fail(c, MATKV_EINVAL, "%s: null pointer", name);
    if (!aligned16(q) || !aligned16(tail_k) || !aligned16(tail_v) || !aligned16(out))
        return fail(c, MATKV_EINVAL, "%s: pointers must be 16-byte aligned", name);
    if (layer < 0 || layer >= c->cfg.n_layers) return fail(c, MATKV_EINVAL, "%s: layer %d outside 0..%d", name, layer, c->cfg.n_layers - 1);
    TableHost* th = find_table(c, table);
    if (!th) return fail(c, MATKV_EINVAL, "%s: table was not built by matkv_assemble", name);
    MATKV_TRY
    st = table_pages_ready(c, *th, name);
    if (st != MATKV_OK) return st;
    note_table_use(c, table, *th, prefill != 0);
    MATKV_CATCH(c, name)
    AttnArgs a{};
    a.q = q; a.out = out; a.tail_k = tail_k; a.tail_v = tail_v;
    a.table = reinterpret_cast<const char*>(table);
    a.partials = reinterpret_cast<float*>(c->workspace + c->wl.off_partials);
    a.variant = prefill ? 0 : c->cfg.decode_variant;
    a.counters = reinterpret_cast<int32_t*>(c->workspace + c->wl.off_counters);
    a.layer = layer; a.n_layers = c->cfg.n_layers;
    a.Hq = c->cfg.n_q_heads; a.Hkv = c->cfg.n_kv_heads; a.D = c->cfg.head_dim;
    a.max_tail = c->cfg.max_tail_tokens;
    a.prefill = prefill;
    a.rows = prefill ? th->max_q : 1;
    const bool even = !prefill && th->even;
    a.shared = !prefill && (th->n_sunits > 0 || even);
    a.past_llc = !prefill && th->past_llc;
    a.tail_spared = !prefill && th->tail_spared;
    a.n_units = prefill ? th->prefill.n_units : (even ? 256 / c->cfg.n_kv_heads : a.shared ? th->n_sunits : th->n_dunits);
    a.max_units_inst = prefill ? th->prefill.max_units_inst : 0;
    a.batch = th->batch; a.total_q = th->total_q; a.kv_fmt = th->kv_fmt;
    a.row_tiles = th->prefill.row_tiles;
    a.tile_rows = th->prefill.tile_rows;
    a.deal_tiles = th->prefill.deal_tiles;
    a.scale_log2e = c->scale_log2e;
    a.out_f32 = c->cfg.dtype == MATKV_BF16 && c->cfg.out_f32;
    a.off_inst = c->tl.off_inst; a.off_items = c->tl.off_items;
    a.off_units = prefill ? c->tl.off_punits : even ? c->tl.off_dunits + sizeof(Unit) * th->n_dunits : (a.shared ? c->tl.off_sunits : c->tl.off_dunits);
    *out_args = a;
    return MATKV_OK;
}

static matkv_status attn_common(matkv_ctx* c, const char* name, int prefill, int32_t layer, const void* q,
                                const void* table, const void* tail_k, const void* tail_v, void* out,
                                bool static_scratch = false) {
    AttnArgs a{};
    matkv_status st = attn_args(c, name, prefill, layer, q, table, tail_k, tail_v, out, &a);
    if (st != MATKV_OK) return st;
    if (static_scratch) {
        const TableHost* th = find_table(c, table);
        const size_t need_p = (size_t)th->n_decode_slots * a.Hq * (a.D + 4) * sizeof(float);
        const size_t need_c = (size_t)a.batch * a.Hkv * kDecodeCounterStride * sizeof(int32_t);
        if (need_p > kStaticPartialBytes || need_c > kStaticCounterBytes)
            return fail(c, MATKV_ENOMEM, "%s: this batch needs %zu bytes of partial results and %zu bytes of counters, the static scratch holds %zu and %zu",
                        name, need_p, need_c, kStaticPartialBytes, kStaticCounterBytes);
        a.counters = reinterpret_cast<int32_t*>(c->static_scratch);
        a.partials = reinterpret_cast<float*>(c->static_scratch + kStaticCounterBytes);
        // the array keeps whatever the last call on this device left: the counters start at zero
        // (a fill kernel, so that the call can be recorded into a graph)
        const int n_ints = (int)(need_c / sizeof(int32_t));
        hipLaunchKernelGGL(zero_ints_kernel, dim3((n_ints + 255) / 256), dim3(256), 0, c->compute, a.counters, n_ints);
        HIP_TRY(c, hipGetLastError());
    }
    const bool want_mfma = prefill || a.variant == 0 || a.variant >= 9000;
    if (attn_prefill_supported(a, c->cfg.dtype)) HIP_TRY(c, launch_attn_prefill(a, c->cfg.dtype, c->compute));
    else if (want_mfma && attn_mfma_supported(a, c->cfg.dtype)) HIP_TRY(c, launch_attn_mfma(a, c->cfg.dtype, c->compute));
    else if (a.kv_fmt != MATKV_PAGE_PLAIN) return fail(c, MATKV_EUNSUPPORTED, "%s: compressed pages need the matrix-core kernels (decode_variant 0 or 90xx)", name);
    else HIP_TRY(c, launch_attn_rows(a, c->cfg.dtype, c->compute));
    return MATKV_OK;
}

matkv_status matkv_prefill_attn(matkv_ctx* c, int32_t layer, const void* q, const void* table,
                                const void* tail_k, const void* tail_v, void* out) {
    return attn_common(c, "prefill_attn", 1, layer, q, table, tail_k, tail_v, out);
}

matkv_status matkv_decode_attn(matkv_ctx* c, int32_t layer, const void* q, const void* table,
                               const void* tail_k, const void* tail_v, void* out) {
    return attn_common(c, "decode_attn", 0, layer, q, table, tail_k, tail_v, out);
}

matkv_status matkv_decode_attn_static(matkv_ctx* c, int32_t layer, const void* q, const void* table,
                                      const void* tail_k, const void* tail_v, void* out) {
    return attn_common(c, "decode_attn_static", 0, layer, q, table, tail_k, tail_v, out, true);
}

matkv_status matkv_decode_step(matkv_ctx* c, int32_t layer, const void* hidden, const void* w_k, const void* w_v,
                               const void* q, const void* table, void* tail_k, void* tail_v, void* out) {
    if (c && (!hidden || !w_k || !w_v)) return fail(c, MATKV_EINVAL, "decode_step: null pointer");
    if (c && (!aligned16(hidden) || !aligned16(w_k) || !aligned16(w_v)))
        return fail(c, MATKV_EINVAL, "decode_step: pointers must be 16-byte aligned");
    AttnArgs a{};
    matkv_status st = attn_args(c, "decode_step", 0, layer, q, table, tail_k, tail_v, out, &a);
    if (st != MATKV_OK) return st;
    TableHost* th = find_table(c, table);
    if (th->min_tail_len < 1) return fail(c, MATKV_EINVAL, "decode_step: a tail holds no row for the new token");
    MaterializeArgs m{};
    m.hidden = hidden; m.w_k = w_k; m.w_v = w_v; m.k_out = tail_k; m.v_out = tail_v;
    m.rope = reinterpret_cast<const RopeEntry*>(c->workspace + c->wl.off_rope);
    m.table = reinterpret_cast<const char*>(table); m.off_inst = c->tl.off_inst;
    m.pos0 = 0; m.token_stride = c->cfg.max_tail_tokens;
    m.rows_per_instance = 1; m.batch = th->batch; m.n_tokens = th->batch;
    m.Hkv = c->cfg.n_kv_heads; m.D = c->cfg.head_dim; m.Hd = c->cfg.hidden;
    materialize_scratch(c, m);
    AttnArgs step = a;
    if (th->step_by_instance) {         // (every table has these units)
        step.shared = 0; step.past_llc = th->step_past_llc;
        step.n_units = th->n_dunits; step.off_units = c->tl.off_dunits;
    }
    if (decode_step_supported(step, m, c->cfg.dtype)) {
        HIP_TRY(c, launch_decode_step(step, m, c->cfg.dtype, c->compute));
        return MATKV_OK;
    }
    if (decode_step_rows_supported(a, m, c->cfg.dtype)) {
        HIP_TRY(c, launch_decode_step_rows(a, m, c->cfg.dtype, c->compute));
        return MATKV_OK;
    }
    // shapes the fused kernels do not cover: the two launches they stand for
    const bool want_mfma = a.variant == 0 || a.variant >= 9000;
    if (a.kv_fmt != MATKV_PAGE_PLAIN && !(want_mfma && attn_mfma_supported(a, c->cfg.dtype)))
        return fail(c, MATKV_EUNSUPPORTED, "decode_step: compressed pages need the matrix-core kernels (decode_variant 0 or 90xx)");
    HIP_TRY(c, launch_materialize(m, c->cfg.dtype, c->compute));
    if (want_mfma && attn_mfma_supported(a, c->cfg.dtype)) HIP_TRY(c, launch_attn_mfma(a, c->cfg.dtype, c->compute));
    else HIP_TRY(c, launch_attn_rows(a, c->cfg.dtype, c->compute));
    return MATKV_OK;
}

matkv_status matkv_chunk_attn(matkv_ctx* c, int32_t layer, const void* q, const void* blob, int32_t n_tokens, void* out) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!q || !blob || !out) return fail(c, MATKV_EINVAL, "chunk_attn: null pointer");
    if (!aligned16(q) || !aligned16(blob) || !aligned16(out)) return fail(c, MATKV_EINVAL, "chunk_attn: pointers must be 16-byte aligned");
    if (layer < 0 || layer >= c->cfg.n_layers) return fail(c, MATKV_EINVAL, "chunk_attn: layer %d outside 0..%d", layer, c->cfg.n_layers - 1);
    if (n_tokens < 0 || n_tokens > 65535) return fail(c, MATKV_EINVAL, "chunk_attn: n_tokens=%d outside 0..65535", n_tokens);
    if (n_tokens == 0) return MATKV_OK;
    const matkv_config& cfg = c->cfg;
    const size_t head_bytes = (size_t)n_tokens * cfg.head_dim * elem_bytes(cfg);
    const char* k_layer = static_cast<const char*>(blob) + (size_t)layer * 2 * cfg.n_kv_heads * head_bytes;
    AttnArgs a{};
    a.q = q; a.out = out;
    a.tail_k = k_layer; a.tail_v = k_layer + (size_t)cfg.n_kv_heads * head_bytes;
    a.table = c->workspace + c->wl.off_chunk;
    a.off_inst = kChunkOffInst; a.off_items = kChunkOffItem; a.off_units = kChunkOffUnit;
    a.partials = reinterpret_cast<float*>(c->workspace + c->wl.off_partials);
    a.counters = reinterpret_cast<int32_t*>(c->workspace + c->wl.off_counters);
    a.layer = 0; a.n_layers = cfg.n_layers;      // the layer is in the pointers: the kernels see a tail, not a blob
    a.Hq = cfg.n_q_heads; a.Hkv = cfg.n_kv_heads; a.D = cfg.head_dim;
    a.max_tail = n_tokens;
    a.prefill = 2; a.rows = n_tokens; a.n_units = 1; a.max_units_inst = 1;
    a.batch = 1; a.total_q = n_tokens; a.row_tiles = 1;
    // 64-row tiles for the shortest chunks while all of their workgroups are on the chip at once (two share a compute unit): a
    // launch's start is shorter.  Then 128-row tiles, and 256-row tiles (twice the longest walk) once they give more workgroups than there are
    // compute units - a good third more where the walks are long, beside which a workgroup's start is little.  us with 64 / 128 / 256 rows: 8B shape,
    // 192 tokens 7.8 / 8.5, 256 9.0 / 9.2, 280 10.3 / 9.7, 512 14.6 / 12.2 / 17.2, 1000 27.4 / 19.3 / 28.9, 2100 70 / 51.0 / 56.3, 2600 100 / 72.1 / 74.1, 3000
    // 127 / 89.2 / 87.9; 3B 256 9.1 / 9.1, 280 10.3 / 9.6, 512 14.3 / 12.1, 2800 92 / 63.8 / 73.9, 3501 129 / 92.4 / 96.2, 4000 167 / 114.2 / 114.8; 70B 192 8.1 / 8.5,
    // 200 9.2 / 8.6, 256 9.5 / 9.2, 512 17.1 / 13.7, 1024 43.8 / 29.4 / 33.0, 1060 43.9 / 35.4 / 33.7, 1300 58 / 44.6 / 41.2.
    // The first line, from 193 tokens on, by the 64-row workgroups, time of 64 over 128 rows at 224 / 257 / 288 tokens: 1 to 16 KV heads of 1 query head 0.89 / 0.97 / 0.98, of 4, 1 to 8 heads
    // 0.97 / 0.97 / 1.02, 16 heads (224 workgroups) 1.01 / 1.09 / 1.14; of 8, 1 to 4 heads 0.975 / 0.97 / 1.025, 8 heads (224) 1.01 / 1.09 / 1.135.
    const long chunk_rows = (long)n_tokens * (cfg.n_q_heads / cfg.n_kv_heads);
    auto workgroups = [&](long rows) { return (chunk_rows + rows - 1) / rows * cfg.n_kv_heads; };
    const bool shortest = n_tokens <= 192 || (n_tokens <= 272 && workgroups(64) <= 192);
    a.tile_rows = shortest && workgroups(64) <= 512 ? 64 : workgroups(256) <= (n_tokens >= 2000 ? 352 : 256) ? 128 : 256;
    a.scale_log2e = c->scale_log2e;
    a.out_f32 = cfg.dtype == MATKV_BF16 && cfg.out_f32;
    const bool tiles = attn_prefill_supported(a, cfg.dtype);
    if (!tiles) {
        // the row-per-workgroup kernel leaves a partial and a counter per (row, head) in the workspace
        const size_t need_f = (size_t)n_tokens * cfg.n_q_heads * (cfg.head_dim + 4);
        const size_t need_c = (size_t)n_tokens * cfg.n_kv_heads;
        if (need_f > c->wl.partial_floats || need_c > c->wl.n_counters)
            return fail(c, MATKV_ENOMEM, "chunk_attn: the workspace of this configuration holds the partial results of %zu rows, the chunk has %d",
                        std::min(c->wl.partial_floats / ((size_t)cfg.n_q_heads * (cfg.head_dim + 4)), c->wl.n_counters / cfg.n_kv_heads), n_tokens);
    }
    // (the tile kernel knows the one instance from its arguments.)  The one-instance table of the other
    // kernel depends on the chunk's length alone: written again only when that
    // changes (a launch of its own costs 4-5 us per layer), always inside a capture (a replay
    // must not depend on what ran before it), and after any replay
    if (!tiles && (c->capturing || c->chunk_table_tokens != n_tokens)) {
        HIP_TRY(c, launch_chunk_table(c->workspace + c->wl.off_chunk, n_tokens, c->compute));
        c->chunk_table_tokens = c->capturing ? -1 : n_tokens;
    }
    if (tiles) HIP_TRY(c, launch_attn_prefill(a, cfg.dtype, c->compute));
    else HIP_TRY(c, launch_attn_rows(a, cfg.dtype, c->compute));
    return MATKV_OK;
}

matkv_status matkv_probe_read(matkv_ctx* c, const void* src, size_t bytes) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!src || !aligned16(src) || bytes == 0 || (bytes % 16)) return fail(c, MATKV_EINVAL, "probe_read: src / bytes");
    // sink: the last word of the rotary-table page of the workspace (never read by any kernel)
    unsigned* sink = reinterpret_cast<unsigned*>(c->workspace + c->wl.off_rope + 4096 - 4);
    HIP_TRY(c, launch_probe_read(src, bytes, sink, c->compute));
    return MATKV_OK;
}

// -------------------------------------------------------------------------------- graphs ----

// A replay of a short recording is issued as its kernel launches instead of as a graph: between two
// graph launches on one stream the device stands still for about 8 us, between two kernels of a stream it waits for
// less than 0.1 where the host is ahead.  A launch costs the host 2.7 us (a graph 15 and 0.5 a kernel), so the saving is
// kept over any number of long kernels and eaten up by many short ones.  Us per replay, graph -> launches:
//   projection and attention of bf16 models, hidden 3072 and more (8 us a kernel and up): one user of 64 tokens, 4 layers
//   (5 kernels) 41.2 -> 33.4, 16 layers 135.3 -> 127.6, 60 layers 481.6 -> 473.5; sixteen of 1000, 31 layers (63) 816.6 -> 811.3
//   fp32 and small hidden sizes (3 to 4 us a kernel): 4 layers (9) 44.9 -> 39.8, 8 layers (17) 79.6 -> 78.1, 16 layers (33)
//   149.2 -> 153.9, 31 layers (63) 289 -> 298
// so long kernels are launched up to kChainMaxNodes of them - the saving is 2 % of the replay there, 1.5 % of a step
// through all layers of a 32-layer model, and an 80-layer one is a graph - and short ones up to kChainMaxShort.
constexpr size_t kChainMaxNodes = 64, kChainMaxShort = 20;

// Whether a kernel is this library's own.  Launches of the caller's between them may carry attributes
// (cooperative, priority) that a plain launch would drop, and may be short.
static bool own_kernel(const void* func) {
    Dl_info mine, other;
    return dladdr(reinterpret_cast<const void*>(&matkv_graph_launch), &mine) && dladdr(func, &other) && mine.dli_fbase == other.dli_fbase;
}

// The recording's kernel launches in order, if it is a single chain of at most max_nodes kernels of this
// library; empty otherwise.  The parameters belong to the graph's nodes and live as long as the graph.
static std::vector<hipKernelNodeParams> kernel_chain(hipGraph_t graph, size_t max_nodes) {
    std::vector<hipKernelNodeParams> chain;
    size_t n = 0, roots = 0;
    if (hipGraphGetNodes(graph, nullptr, &n) != hipSuccess || n == 0 || n > max_nodes) return {};
    if (hipGraphGetRootNodes(graph, nullptr, &roots) != hipSuccess || roots != 1) return {};
    hipGraphNode_t node = nullptr;
    if (hipGraphGetRootNodes(graph, &node, &roots) != hipSuccess) return {};
    while (true) {
        hipGraphNodeType type;
        hipKernelNodeParams p{};
        if (hipGraphNodeGetType(node, &type) != hipSuccess || type != hipGraphNodeTypeKernel ||
            hipGraphKernelNodeGetParams(node, &p) != hipSuccess || !p.func || !p.kernelParams || p.extra || !own_kernel(p.func)) {
            (void)hipGetLastError();                // (a query that failed is no error of the recording)
            return {};
        }
        chain.push_back(p);
        size_t next = 0;
        if (hipGraphNodeGetDependentNodes(node, nullptr, &next) != hipSuccess || next > 1) return {};
        if (next == 0) break;
        if (hipGraphNodeGetDependentNodes(node, &node, &next) != hipSuccess) return {};
    }
    if (chain.size() != n) chain.clear();
    return chain;
}

matkv_status matkv_graph_begin(matkv_ctx* c) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (c->capturing) return fail(c, MATKV_EBUSY, "graph_begin: a capture is already open");
    matkv_graph* g = new (std::nothrow) matkv_graph();
    if (!g) return fail(c, MATKV_ENOMEM, "graph_begin: out of host memory");
    hipError_t e = hipStreamBeginCapture(c->compute, hipStreamCaptureModeRelaxed);
    if (e != hipSuccess) { delete g; return hip_fail(c, e, "hipStreamBeginCapture"); }
    c->capturing = true;
    c->cap = g;
    return MATKV_OK;
}

matkv_status matkv_graph_end(matkv_ctx* c, matkv_graph** out) {
    if (!c || !out) return MATKV_EINVAL;
    if (!c->capturing) return fail(c, MATKV_EINVAL, "graph_end: no capture is open");
    matkv_graph* g = c->cap;
    c->capturing = false;
    c->cap = nullptr;
    hipError_t e = hipStreamEndCapture(c->compute, &g->graph);
    if (e == hipSuccess) e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        if (g->graph) (void)hipGraphDestroy(g->graph);
        delete g;
        return hip_fail(c, e, "graph_end");
    }
    try {
        const bool long_kernels = c->cfg.dtype == MATKV_BF16 && c->cfg.head_dim == 128 && c->cfg.hidden >= 3072;
        g->chain = kernel_chain(g->graph, long_kernels ? kChainMaxNodes : kChainMaxShort);
        c->graphs.push_back(g);
    } catch (...) {
        (void)hipGraphExecDestroy(g->exec);
        (void)hipGraphDestroy(g->graph);
        delete g;
        return fail(c, MATKV_ENOMEM, "graph_end: out of host memory");
    }
    *out = g;
    return MATKV_OK;
}

matkv_status matkv_graph_launch(matkv_ctx* c, matkv_graph* g) {
    matkv_status st = precheck(c);
    if (st != MATKV_OK) return st;
    if (!g || !g->exec) return fail(c, MATKV_EINVAL, "graph_launch: null graph");
    if (c->capturing) return fail(c, MATKV_EBUSY, "graph_launch: a capture is open");
    // the tables must still be cut the way they were when the calls were recorded
    for (auto& e : g->tables) {
        TableHost* th = find_table(c, e.table);
        if (!th) return fail(c, MATKV_EINVAL, "graph_launch: a recorded table no longer exists");
        if ((e.decode && th->sig_decode != e.sig_decode) || (e.prefill && th->sig_prefill != e.sig_prefill))
            return fail(c, MATKV_EINVAL, "graph_launch: a table has been re-assembled into a different partition since the recording");
        // a load into one of its slots since the recording: the replay must not race with the copy
        st = table_pages_ready(c, *th, "graph_launch");
        if (st != MATKV_OK) return st;
    }
    // the recorded tail advances must still fit
    for (auto& adv : g->advances) {
        TableHost* th = find_table(c, adv.first);
        if (!th) return fail(c, MATKV_EINVAL, "graph_launch: a recorded table no longer exists");
        if (th->max_tail_len + adv.second > c->cfg.max_tail_tokens)
            return fail(c, MATKV_EINVAL, "graph_launch: tail would hold %d tokens, max_tail_tokens=%d", th->max_tail_len + adv.second, c->cfg.max_tail_tokens);
    }
    for (auto& adv : g->advances) {
        TableHost* th = find_table(c, adv.first);
        th->max_tail_len += adv.second; th->min_tail_len += adv.second;
    }
    c->chunk_table_tokens = -1;                // the replay may hold a chunk attention of another length
    // (a stream that the caller is recording by other means takes the graph as before)
    hipStreamCaptureStatus recording = hipStreamCaptureStatusNone;
    if (!g->chain.empty() && hipStreamIsCapturing(c->compute, &recording) == hipSuccess && recording == hipStreamCaptureStatusNone) {
        for (const hipKernelNodeParams& p : g->chain)
            HIP_TRY(c, hipLaunchKernel(p.func, p.gridDim, p.blockDim, p.kernelParams, p.sharedMemBytes, c->compute));
        return MATKV_OK;
    }
    HIP_TRY(c, hipGraphLaunch(g->exec, c->compute));
    return MATKV_OK;
}

int32_t matkv_graph_kernel_launches(const matkv_graph* g) { return g ? (int32_t)g->chain.size() : -1; }

matkv_status matkv_graph_destroy(matkv_ctx* c, matkv_graph* g) {
    if (!c || !g) return MATKV_EINVAL;
    for (size_t i = 0; i < c->graphs.size(); ++i) {
        if (c->graphs[i] == g) {
            (void)hipStreamSynchronize(c->compute);
            if (g->exec) (void)hipGraphExecDestroy(g->exec);
            if (g->graph) (void)hipGraphDestroy(g->graph);
            delete g;
            c->graphs.erase(c->graphs.begin() + i);
            return MATKV_OK;
        }
    }
    return fail(c, MATKV_EINVAL, "graph_destroy: unknown graph");
}

}  // extern "C"
