// Host side of the LASGD update library: context, validation, state machine,
// lookup tables, launches.  The C ABI is declared in include/lasgd.h.
//
// Stream protocol (single-GPU image of "the All-Reduce runs while the node
// keeps computing", Sec. 4):
//   main stream:  local_step ... snapshot/merge --evA--> ...        wait evZ, merge
//   side stream:                          wait evA, average --evZ-->
// (a mean that is over before the events around it would be stays on the main stream, see mean_on_main)
// evA orders the side stream's reads of s after the main stream's writes;
// evZ orders the main stream's reads of z after the side stream's writes.
// The state machine refuses call orders in which s or z could be overwritten
// while the other stream may still read them.
#include "lasgd_kernels.hip.h"
#include "../../include/lasgd.h"

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

using namespace lasgd;

namespace {

constexpr int kMaxK = 64;
// Elements.  Every tensor starts on 1 KiB inside a replica's slab, so that each 256-element tile is one aligned
// KiB: tiles that start 256 or 512 bytes off such a boundary stream 3-5 % slower on MI355X.
constexpr uint64_t kArenaAlign = 256;
constexpr uint64_t kMaxNpad = (1ull << 31) - (1ull << 20); // tile offsets stay far inside 32-bit element counts

thread_local std::string g_create_error;

} // namespace

struct lasgd_ctx {
    int32_t K = 0, n_tensors = 0;
    lasgd_dtype storage = LASGD_F32;
    float mu = 0.f, wd_scalar = 0.f;
    int32_t nesterov = 0;
    std::vector<int64_t> numel;
    std::vector<float> wd;
    std::vector<uint64_t> aoff;      // arena offset of each tensor (elements)
    uint64_t packed = 0;             // elements of one replica's tensors, each rounded up to whole rows
    uint64_t npad = 0, ntotal = 0;   // npad: the same and, for some lengths, a row more (see padded)
    hipStream_t main = nullptr, side = nullptr;
    hipEvent_t evA = nullptr, evZ = nullptr;
    bool back = false;               // the last launch ran from its last item to its first, see backwards
    bool clearing = false;           // a clear of the gradients may be queued on a stream of the caller's
    bool clear_in_graph = false;     // one was recorded: from then on a replay of it may be queued at any time
    int device = 0;

    // device memory: v, s, z and x32 are one allocation, carved up
    char *arena = nullptr;
    float *v = nullptr, *s = nullptr, *z = nullptr, *x32 = nullptr;
    float *gbar = nullptr;           // mean gradient [npad] of an SGD All-Reduce step in two kernels, see reserve_mean_grad
    bool gbar_tried = false;         // asked for; without it the step always takes one kernel
    // one set of lookup tables per tile size ever used (vec = 1, 2, 4), kept until destroy: a graph captured
    // under one tile size still points at its tables after the tile size has been changed
    struct Tables {
        uint32_t *mem = nullptr;                 // the two arrays, one behind the other
        const uint32_t *blocks = nullptr, *tile0 = nullptr;
        uint32_t ntiles = 0;
    };
    Tables tables_by_vec[3];
    const Tables *tables = nullptr;              // those of the current tile size
    Record *records = nullptr;                   // device table [K*n_tensors]
    std::vector<void *> h_xptr;
    std::vector<char> bound;
    int32_t n_bound = 0;

    // bf16 storage: where each replica's model is (bit k = replica k), see place_models
    uint64_t at_s = 0;               // in s[k], which it has just re-sent, and nowhere else
    bool both_places = true;         // a global update that re-sends writes the master copy too: small models, and any of which
                                     // a call has been recorded into a graph
    bool settled = true;             // both_places: all models are back in the master copies, on the main stream
    uint64_t settle_mask = 0;        // those that were in s when a call was first recorded
    bool settle_recorded = false;          // into a graph,
    unsigned long long settle_graph = 0;   // last into this capture
    uint32_t *settle = nullptr;            // words behind the master copies, see settle_word

    // protocol state (bit k = replica k)
    bool master_ready = false;   // bf16: master copy initialised
    uint64_t all = 0;            // every replica
    uint64_t snap_mask = 0;      // s[k] holds a model that may be averaged next
    uint64_t pending_mask = 0;   // participants of the launched mean that have not merged yet
    bool avg_ever = false;
    bool avg_in_graph = false;   // the last mean was recorded into a graph, not executed: evZ says nothing about it
    bool z_on_main = false;      // the pending mean was enqueued on the main stream: stream order already puts it first
    bool center_valid = false;   // z has been computed at least once
    float alpha = 1.f, beta = 1.f;   // elastic coefficients (Sec. 3, Eq. 5-6); 1, 1 = Algorithm 1

    lasgd_tuning tune{};             // .nontemporal: 1..4 as the caller has set it, for every call; -1 = by call and size (hint_of)
    bool fused_cycle = false;        // the pending mean was made by lasgd_step_merge_average: the steps in between go by its rule
    std::string err;
};

namespace {

lasgd_status fail(lasgd_ctx *ctx, lasgd_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    try {
        if (ctx) ctx->err = buf;
        else g_create_error = buf;
    } catch (...) {       // the message is lost, the status is not
    }
    return st;
}

#define LASGD_HIP(ctx, call)                                                                   \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess) {                                                                \
            (void)hipGetLastError(); /* reported here; do not leave it for the next HIP user */ \
            return fail(ctx, e_ == hipErrorOutOfMemory ? LASGD_ERR_ALLOC : LASGD_ERR_HIP,      \
                        "%s failed: %s", #call, hipGetErrorString(e_));                        \
        }                                                                                      \
    } while (0)

uint64_t round_up(uint64_t a, uint64_t b) { return (a + b - 1) / b * b; }

bool is_pow2(uint32_t k) { return k && !(k & (k - 1)); }

// One array (x, v, s or the gradients) of all replicas.
uint64_t array_bytes(const lasgd_ctx *c) { return (uint64_t)c->K * c->npad * sizeof(float); }
constexpr uint64_t kBackFrom = 8ull << 20, kBackBelow = 64ull << 20;      // see backwards

// What fast_div expects for a divisor d in 1 .. 2^31.
FastDiv make_div(uint32_t d)
{
    const uint32_t l = d > 1u ? 32u - (uint32_t)__builtin_clz(d - 1u) : 0u;          // ceil(log2 d)
    FastDiv f;
    f.shift = 31u + l;
    f.m = (uint32_t)(is_pow2(d) ? 1ull << 31 : (1ull << f.shift) / d + 1ull);
    return f;
}

// Build (on the host) the lookup tables for 256*vec-element tiles and copy them to the device.
lasgd_status upload_tables(lasgd_ctx *c, int vec)
{
    lasgd_ctx::Tables &t = c->tables_by_vec[vec == 1 ? 0 : vec == 2 ? 1 : 2];
    if (!t.mem) {
        const uint64_t T = 256ull * vec;
        std::vector<uint32_t> tile0((size_t)c->n_tensors);
        uint64_t tiles = 0;
        for (size_t i = 0; i < tile0.size(); ++i) {
            tile0[i] = (uint32_t)tiles;
            tiles += ((uint64_t)c->numel[i] + T - 1) / T;
            if (tiles > 0x7fffffffull / kMaxK) return fail(c, LASGD_ERR_UNSUPPORTED, "too many tiles (more than %llu)", 0x7fffffffull / kMaxK);
        }
        std::vector<uint32_t> host;              // blocks, then tile0
        const size_t nblocks = (size_t)((tiles + (1u << kBlockShift) - 1) >> kBlockShift);
        size_t t0 = 0;
        for (size_t b = 0; b < nblocks; ++b) {
            const uint32_t first = (uint32_t)(b << kBlockShift), next = first + (1u << kBlockShift);
            while (t0 + 1 < tile0.size() && tile0[t0 + 1] <= first) ++t0;
            host.push_back((uint32_t)t0 | (t0 + 1 < tile0.size() && tile0[t0 + 1] < next ? kMoreInBlock : 0u));
        }
        host.insert(host.end(), tile0.begin(), tile0.end());
        host.insert(host.end(), kProbe, 0xffffffffu);
        const size_t bytes = host.size() * sizeof(uint32_t);
        uint32_t *d = nullptr;
        LASGD_HIP(c, hipMalloc((void **)&d, bytes));
        hipError_t e = hipMemcpy(d, host.data(), bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipFree(d);
            (void)hipGetLastError();
            return fail(c, LASGD_ERR_HIP, "table upload failed: %s", hipGetErrorString(e));
        }
        t.mem = d;
        t.blocks = d;
        t.tile0 = d + nblocks;
        t.ntiles = (uint32_t)tiles;
    }
    c->tables = &t;
    return LASGD_OK;
}

// Defaults from sweeps on MI355X over the five benchmark workloads: the finest
// tile (one 128-bit vector per lane), one wave per (tile, replica), a grid that
// covers all items in one-wave workgroups (the waves are independent, and
// single-wave groups dispatch and retire with the least friction), and the
// streaming hint on every access except z from the sizes of hint_of on.  A local step sweeps one replica after the other
// (the longest contiguous runs); merges take the tiles in chunks of 8192 (8 MB
// of z per chunk, 1 MB per XCD) so that the chunk's z is still in L2 when the
// next replica needs it.  The mean's replicas are split over four groups of waves from K = 12 on (256-thread workgroups
// with LDS): merge + mean, us at split 1 / 2 / 4: ResNet-50 list K = 12 982 / 975 / 963, K = 16
// 1296 / 1294 / 1277, and the same on two streams; MobileNetV2 K = 16 178 / 183 / 178.  From 8 to 11 two groups
// where the mean runs beside the steps on the other stream, one where it has the GPU to itself.  A cycle, us at split 1 / 2, two streams:
// ResNet-50 K = 8, m = 4 2851 / 2847, ResNet-18 K = 8 1291 / 1288, bf16 K = 10, m = 2 957 / 951, MobileNetV2 K = 8 235.4 / 234.5, 10^6 elements
// K = 8 79.4 / 79.1, K = 10 94.5 / 94.2; one stream: 2831 / 2832, 1295 / 1296, 943 / 945, 228.8 / 229.6, 75.0 / 75.3, 91.0 / 91.0, 2e6 K = 8 135.0 / 136.6
// (profiles/mean_launch_shape_sweep.txt).  The in-order mean of lasgd_step_merge_average
// takes split 1: its z is to be that of the one-kernel form to the bit.
//
// From which size of one array of all replicas (x, v, s or the gradients) on a call takes the streaming hint.  The 256 MB
// memory-side cache would hold three or four arrays of 64 MB, but only for a program that calls nothing else: us without / with
// the hint, in a loop over one state | over three states in turn | with 1 GiB of other work between the passes.
//   cycle, m = 2, K = 4, 16 MB an array    39 / 41    40 / 45    53 / 48       bf16, 24 MB   56 / 58    60 / 62    73 / 65
//                        24 MB             56 / 56    60 / 60    75 / 64             32 MB   73 / 74    82 / 79    89 / 82
//                        32 MB             73 / 73    81 / 77    92 / 80             72 MB  160 / 158  167 / 162  180 / 168
//                        53 MB            112 / 115  124 / 118  146 / 124     MobileNetV2 list, K = 8, 112 MB      268 / 228
//                       104 MB            234 / 218  246 / 219  259 / 227     ResNet-18 list, K = 2, 94 MB         231 / 198
//   sgd_ar_step, K = 4, 32 MB              26 / 27    28 / 29    41 / 32       K = 8, 112 MB  89 / 99   112 / 95   121 / 98
//                       53 MB              41 / 43    54 / 46    64 / 48       bf16 K = 5, 70 MB 55 / 62   72 / 63    77 / 66
//   step_merge_average, K = 4, 53 MB      201 / 223  210 / 226  226 / 232     K = 8, 112 MB  456 / 480   468 / 462  479 / 473
// bf16 with the model in one place, two fused updates, three in turn | other work between: K = 4, 72 MB 150 / 155    178 / 160; 96 MB 203 / 192    210 / 200;
// 112 MB 244 / 218    249 / 228; K = 16, 72 MB 144 / 155    170 / 159; 96 MB 196 / 192    208 / 196; with two steps between, 96 MB 539 / 541    554 / 548.
// Local steps between two fused updates go by the fused update's line (with the hint of a cycle's, K = 4, 53 MB, m = 2 208 / 218 us).
// Gradients just cleared are written to next, so zero_grads keeps them in the cache as long as they may fit.
enum Use { USE_CYCLE, USE_SGD_AR, USE_FUSED, USE_ZERO };
int hint_of(const lasgd_ctx *c, Use use)
{
    if (c->tune.nontemporal >= 0) return c->tune.nontemporal & 3;           // 4, no hint, is 0
    const uint64_t array = array_bytes(c);
    const uint64_t from = use == USE_CYCLE ? 28ull << 20 : use == USE_SGD_AR ? 40ull << 20 : use == USE_FUSED && !c->both_places ? 96ull << 20 : 128ull << 20;
    return array >= from ? 3 : 0;
}

// A mean on the side stream costs the host an event, a wait, an event and a wait, about 20 us, and both streams their waits.
// One that moves no more than 16 MiB is done in 3 to 6 us, so it stays on the main stream.  A cycle's us on two streams /
// on one: K = 3, m = 2, 5000 elements 31 / 11, 10^5 31 / 13, 4e5 (6.4 MB) 38 / 19, 10^6 (16 MB) 40 / 32; K = 8, m = 4, 4e5 (14 MB) 56 / 53;
// K = 32, m = 4, 10^5 (13 MB) 56 / 53.  Beyond: K = 8, m = 4, 10^6 (36 MB) 123 / 124.  With other work between the calls a longer mean is
// worth hiding behind it.  Exactly 16 MiB, two streams / one, m = 2: K = 3, 2^20 elements 41.9 / 31.5, K = 7, 2^19 44.8 / 34.3, K = 15, 2^18 47.0 / 36.1,
// K = 63, 2^16 48.3 / 36.9.  So the line goes by the tensors, not by the row more that just such lengths have in the arenas.
bool mean_on_main(uint32_t participants, uint64_t packed)
{
    return (participants + 1ull) * packed * sizeof(float) <= (16ull << 20);
}

// A replica's arrays must not lie a round number apart: the rows of a tile would meet in a few sets of the caches and channels.  us
// without / with one row more, 2^20 elements: two fused updates K = 4 54.0 / 46.1, a cycle K = 8, m = 2 79.4 / 76.9, SGD-AR K = 4 18.0 / 16.8;
// 2^19 elements, two fused updates K = 4 30.4 / 29.0, a cycle K = 8 39.5 / 38.3 (3, 8 or 33 rows are no better).
uint64_t padded(uint64_t packed) { return packed * sizeof(float) % 65536u == 0u ? packed + kArenaAlign : packed; }

lasgd_tuning default_tuning(const lasgd_ctx &c)
{
    lasgd_tuning t{};
    t.vec = 1;
    t.kper_step = 1;
    t.kper_merge = 1;
    t.max_blocks = -1;
    t.avg_split = c.K >= 12 ? 4 : c.K >= 8 && c.side != c.main && !mean_on_main((uint32_t)c.K, c.packed) ? 2 : 1;
    t.avg_max_blocks = -1;
    t.nontemporal = -1;
    t.waves_per_block = 1;
    t.chunk_step = -1;
    t.chunk_merge = 8192;
    t.race_probe = -1;
    t.group_r = -1;
    return t;
}

// How many waves a CU may hold at once in the streaming kernels, set through the LDS a workgroup asks for (and does
// not use): 160 KiB in granules of 1280 bytes.  The memory system is fastest with about 60 KiB of loads in flight per
// CU; with all 32 waves a CU the kernels reach it through L2 misses that evict each other.  us at 0 (32 waves), 5 (25),
// 6 (21), 7 (18), 8 (16), 10 (12) granules a wave, ResNet-50 list, K = 8 (profiles/waves_in_flight_sweep.txt, with others):
//   local step (3 KiB of loads a wave, and a word before them)   629  607  605  611  598  648     bf16 657  653  637  618  627  668
//   step + update (4 KiB, and z), with the mean                 1088 1087 1070 1039 1030 1021
//   global update (2 KiB, and z), with the mean                  672  660  653  657  683  754
//   snapshot (1 KiB)                                             251  276  279  299  331  396
//   step with the mean gradient (2 KiB, and it), with its mean     -   656  652  656  682    -       bf16   -  667  661  655  662    -
// fp32 local steps take 6 and not 8: beside the mean on a second stream 21 waves were the better count.
// Nothing is gained where the state stays in the memory-side cache (no streaming hint).
// A caller's kernel on another stream does not wait longer for a CU: a bf16 product of 4096^3 beside local steps took
// 643-697 us, and 650-712 when the steps held all 32 waves and no LDS.
constexpr uint32_t kLdsGranule = 1280;
constexpr size_t kCuLds = 163840;
constexpr size_t kOneGroupLds = (kCuLds / 2 / kLdsGranule + 1) * kLdsGranule;      // two workgroups with this do not fit a CU
constexpr size_t kMaxLds = 65536;      // what a workgroup may ask for without further ado: pacing stops there, but for kOneGroupLds (launch_flat_update)
// Step + update asks for a word of its model before its loads, as the fp32 local step always does, and then runs 16 waves a CU in
// place of 12, up to 1e8 replica-parameters.  A pass's us without / with, over three states in turn (and with other work between
// the passes): MobileNetV2 list K = 16, every step 285 / 280 (287 / 290), with m = 2 456 / 449 (460 / 455), partial rounds 411 / 402 (422 / 416);
// ResNet-18 K = 8 (9.4e7), adaptive rounds 826 / 818 (847 / 841), K = 4, m = 4 671 / 663; ResNet-50 K = 4 (1.0e8), m = 2 844 / 846 (863 / 862).
// Beyond, ResNet-18 K = 24, m = 3 3858 / 3882, ResNet-50 K = 8, m = 4 2868 / 2876.  Two or three words gain on the fp32 step in a loop of
// nothing but steps, from what the last step left in the memory-side cache, and lose 0.3-1.3 % with other work between.
// Where every model is in s (at_s), a wave has no more to load than for a bf16 local step, and goes by its rule.  An update every
// step, us at 10 granules / 10 and a word / 6 / 7 / 8 / 6 and a word: ResNet-18 list K = 12 585 / 609 / 542 / 537 / 534 / 542, ResNet-50
// K = 16 1684 / 1776 / 1574 / 1557 / 1563 / 1596, MobileNetV2 K = 16 (8 granules and a word 227) 238 / 248 / 219 / 218 / 221 / 219.
bool word_first(int op, uint64_t replica_params, bool at_s) { return op == OP_STEP_MERGE && !at_s && replica_params <= 100000000u; }
uint32_t pace_lds(int op, bool bf16, const ExtArgs *xa, int nt, uint32_t vec, uint32_t waves_per_block, bool at_s)
{
    if (!(nt & 3)) return 0;
    const uint32_t step_merge = at_s ? 7u : nt & 4 ? 8u : 10u;        // without s to load; with a word first, and without
    uint32_t granules = op == OP_STEP ? (bf16 ? 7u : 6u) : op == OP_MERGE ? 6u : op == OP_STEP_MERGE ? step_merge : op == OP_STEP_MEAN ? (bf16 ? 7u : 6u) : 0u;
    if (xa && op == OP_STEP_MERGE) {         // replicas that only step or only merge load less: the mean over the waves
        const uint32_t both = (uint32_t)__builtin_popcountll(xa->step_mask & xa->merge_mask);
        const uint32_t step = (uint32_t)__builtin_popcountll(xa->step_mask & ~xa->merge_mask);
        const uint32_t merge = (uint32_t)__builtin_popcountll(xa->merge_mask & ~xa->step_mask);
        granules = (step_merge * both + 7u * step + 6u * merge) / (both + step + merge);
    }
    const uint32_t bytes = granules * kLdsGranule * vec * waves_per_block;
    return bytes < kMaxLds ? bytes : (uint32_t)kMaxLds;
}

bool all_at_s(const ApplyArgs &a) { return !(a.place & LOOK) && a.at_s == (a.K == 64u ? ~0ull : (1ull << a.K) - 1ull); }

template <int VEC, int OP, bool BF16>
hipError_t launch_nt(const ApplyArgs &a, const ExtArgs *xa, dim3 grid, dim3 bs, hipStream_t st, int nt)
{
    const uint32_t lds = pace_lds(OP, BF16, xa, nt, VEC, bs.x / 64u, all_at_s(a));
    if (xa) {      // extended variants: hints all on or all off
        if constexpr (VEC == 1 && OP == OP_STEP_MERGE) {
            if (nt == 7) {
                hipLaunchKernelGGL((apply_ext_kernel<VEC, OP, BF16, 7>), grid, bs, lds, st, a, *xa);
                return hipGetLastError();
            }
        }
        if (nt & 3) hipLaunchKernelGGL((apply_ext_kernel<VEC, OP, BF16, 3>), grid, bs, lds, st, a, *xa);
        else hipLaunchKernelGGL((apply_ext_kernel<VEC, OP, BF16, 0>), grid, bs, lds, st, a, *xa);
        return hipGetLastError();
    }
    if constexpr (VEC == 1 && OP == OP_STEP_MERGE) {
        if (nt == 7) {
            hipLaunchKernelGGL((apply_kernel<VEC, OP, BF16, 7>), grid, bs, lds, st, a);
            return hipGetLastError();
        }
    }
    switch (nt & 3) {
    case 0: hipLaunchKernelGGL((apply_kernel<VEC, OP, BF16, 0>), grid, bs, lds, st, a); break;
    case 1: hipLaunchKernelGGL((apply_kernel<VEC, OP, BF16, 1>), grid, bs, lds, st, a); break;
    case 2: hipLaunchKernelGGL((apply_kernel<VEC, OP, BF16, 2>), grid, bs, lds, st, a); break;
    default: hipLaunchKernelGGL((apply_kernel<VEC, OP, BF16, 3>), grid, bs, lds, st, a); break;
    }
    return hipGetLastError();
}

// Streaming and in tiles of 256 elements only.
template <int OP, bool BF16>
hipError_t launch_one(const ApplyArgs &a, dim3 grid, dim3 bs, hipStream_t st)
{
    hipLaunchKernelGGL((apply_kernel<1, OP, BF16, 3>), grid, bs, pace_lds(OP, BF16, nullptr, 3, 1, bs.x / 64u, false), st, a);
    return hipGetLastError();
}

template <int OP, bool BF16>
hipError_t launch_vec(const ApplyArgs &a, const ExtArgs *xa, dim3 grid, dim3 bs, hipStream_t st, int vec, int nt)
{
    switch (vec) {
    case 1: return launch_nt<1, OP, BF16>(a, xa, grid, bs, st, nt);
    case 2: return launch_nt<2, OP, BF16>(a, xa, grid, bs, st, nt);
    default: return launch_nt<4, OP, BF16>(a, xa, grid, bs, st, nt);
    }
}

template <int OP>
hipError_t launch_op(const ApplyArgs &a, const ExtArgs *xa, dim3 grid, dim3 bs, hipStream_t st, int vec, int nt, bool bf16)
{
    return bf16 ? launch_vec<OP, true>(a, xa, grid, bs, st, vec, nt) : launch_vec<OP, false>(a, xa, grid, bs, st, vec, nt);
}

void fill_common(const lasgd_ctx *c, ApplyArgs &a)
{
    a.blocks = c->tables->blocks;
    a.tile0 = c->tables->tile0;
    a.records = c->records;
    a.tile_elems = 256u * (uint32_t)c->tune.vec;
    a.x32 = c->x32;
    a.v = c->v;
    a.s = c->s;
    a.z = c->z;
    a.npad = c->npad;
    a.ntiles = c->tables->ntiles;
    a.K = (uint32_t)c->K;
    a.n_tensors = (uint32_t)c->n_tensors;
    a.mu = c->mu;
    a.nesterov = c->nesterov;
    a.use_mul = is_pow2((uint32_t)c->K) ? 1 : 0;
    a.inv_k = 1.0 / (double)c->K;
    a.k_as_double = (double)c->K;
}

// A multi-tensor pass, planned (arguments, grid; everything that can be refused)
// and then launched on the main stream.  Callers plan before they enqueue any
// stream dependency, so that a refused call leaves both streams untouched.
struct ApplyPlan {
    ApplyArgs a{};
    int op = 0;
    dim3 grid{1}, bs{64};
    bool has_ext = false;
    ExtArgs ext{};
};

// xa == nullptr: every replica takes part, one step size, alpha = 1 (the plain kernels).
lasgd_status plan_apply(lasgd_ctx *c, ApplyPlan &p, int op, float lr, int resnap, const ExtArgs *xa = nullptr)
{
    if (op < OP_STEP || op > OP_STEP_MEAN) return fail(c, LASGD_ERR_INVALID, "unknown op %d", op);
    ApplyArgs &a = p.a;
    fill_common(c, a);
    int kper = (op == OP_MERGE || op == OP_STEP_MERGE || op == OP_STEP_MEAN) ? c->tune.kper_merge : c->tune.kper_step;
    const int taking = xa ? __builtin_popcountll(xa->step_mask | xa->merge_mask) : c->K;
    if (kper < 1) kper = 1;
    if (kper > taking) kper = taking;
    a.kcount = (uint32_t)taking;
    a.kper = (uint32_t)kper;
    a.kgroups = (uint32_t)((taking + kper - 1) / kper);
    a.neg_lr = -lr;
    a.resnap = resnap;
    const bool merging = op == OP_MERGE || op == OP_STEP_MERGE || op == OP_STEP_MEAN;       // or reads a shared row as they do
    int64_t chunk = merging ? c->tune.chunk_merge : c->tune.chunk_step;
    // Steps between two fused updates, which go tile by tile, leave the same tiles of all replicas in the L2s if they go by short
    // chunks.  bf16 only: an fp32 model is the caller's, and where its replicas lie a round number apart the rows of a tile get in
    // each other's way.  Two fused updates and two steps, us without / with: bf16 K = 4, 2^20 elements 67.7 / 65.7, K = 8, 2^19 68.3 / 65.3, K = 6,
    // 2^21 189.6 / 187.7; fp32 K = 4, 1,000,003 elements 67.2 / 64.6, but 2^20 73.7 / 75.8 and with four steps 92.0 / 93.9.
    if (chunk < 1 && op == OP_STEP && c->fused_cycle && c->storage == LASGD_BF16 && !(hint_of(c, USE_FUSED) & 3)) chunk = 64;
    if (chunk < 1 || chunk > (int64_t)a.ntiles) chunk = 0;                        // one chunk, handled as the tail
    a.chunk = chunk ? (uint32_t)chunk : 1u;
    const uint32_t nfull = chunk ? a.ntiles / a.chunk : 0u;
    a.full_items = nfull * a.chunk * a.kgroups;
    a.tail_first = nfull * a.chunk;
    const uint32_t tail = a.ntiles - a.tail_first;
    a.tail_chunk = tail ? tail : 1u;
    // passes over the shared z should start on the same XCD for every replica group: 8 XCDs x up to 4 waves
    // per workgroup.  A local step or snapshot reads no z, but where the L2s hold a good part of the state its tiles belong on the
    // XCDs that the other kernels have them on (see backwards).
    a.tail_stride = (uint32_t)round_up(a.tail_chunk, merging ? 32u : array_bytes(c) < kBackBelow ? 8u * (uint32_t)c->tune.waves_per_block : 1u);
    const uint64_t nitems = (uint64_t)a.full_items + (tail ? (uint64_t)a.tail_stride * a.kgroups : 0u);
    if (nitems == 0 || nitems > 0x7fffffffull) return fail(c, LASGD_ERR_UNSUPPORTED, "work-item count %llu out of range", (unsigned long long)nitems);
    a.nitems = (uint32_t)nitems;
    a.by_per = make_div(a.chunk * a.kgroups);
    a.by_chunk = make_div(a.chunk);
    a.by_stride = make_div(a.tail_stride);
    const uint32_t wpb = (uint32_t)c->tune.waves_per_block;
    uint64_t blocks = (nitems + wpb - 1) / wpb;
    if (c->tune.max_blocks > 0 && blocks > (uint64_t)c->tune.max_blocks) blocks = (uint64_t)c->tune.max_blocks;
    a.wpb = wpb;
    a.nwaves = (uint32_t)blocks * wpb;
    p.op = op;
    p.grid = dim3((uint32_t)blocks);
    p.bs = dim3(64u * wpb);
    p.has_ext = xa != nullptr;
    if (xa) p.ext = *xa;
    return LASGD_OK;
}

// Is this stream recording into a graph rather than executing?  id: which capture, one of its own for each.
bool is_capturing(hipStream_t st, unsigned long long *id = nullptr)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if ((id ? hipStreamGetCaptureInfo(st, &cs, id) : hipStreamIsCapturing(st, &cs)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return cs != hipStreamCaptureStatusNone;
}

// bf16 storage: before a call that reads or writes the models.  A global update that re-sends leaves the model in s alone
// (apply_tile), and c->at_s says where each call finds it.  A recorded call cannot go by that: it is replayed whenever the
// caller likes.  So once a call has been recorded, every update writes the master copy too, recorded or not, and models that
// are in s at that moment are brought back once, by the first graph that is replayed or the first call that runs: in a graph by its first
// kernel as it goes (settle_word), where that writes all of them, else by a kernel in front (settle_kernel).
//
// From 8 MiB an array on.  us, both places / s alone, an update every step, every third step, two fused ones, K = 4:
// 0.3 MB an array 10 / 10, 21 / 21, 16 / 16; 4 MB 13.7 / 13.1, 25.2 / 23.7, 20.3 / 18.5; 16 MB 27.8 / 22.4, 55.9 / 51.9,
// 52.6 / 45.3; 32 MB 54.0 / 44.6, 109.9 / 106.6, 98.9 / 79.0.
constexpr uint64_t kOneCopyFrom = 8ull << 20;
constexpr uint32_t kSettleBlocks = 256;

// Is a call on the models being recorded (while that matters)?  With the first one the rule above changes.
bool note_recording(lasgd_ctx *c, unsigned long long *id = nullptr)
{
    if (c->storage != LASGD_BF16 || (c->both_places && c->settled)) return false;
    unsigned long long any = 0;
    if (!is_capturing(c->main, id ? id : &any)) return false;
    if (!c->both_places) {
        c->both_places = true;
        c->settle_mask = c->at_s;
        c->settled = !c->settle_mask;
        c->at_s = 0;
    }
    return !c->settled;
}

// a: the call's arguments, told where the models are.  rewritten: the replicas whose master copies it writes from their models; reads:
// it only reads the models, and leaves bringing them back to the next call.
lasgd_status place_models(lasgd_ctx *c, ApplyArgs *a = nullptr, uint64_t rewritten = 0, bool reads = false)
{
    if (c->storage != LASGD_BF16) return LASGD_OK;
    unsigned long long id = 0;
    const bool recording = note_recording(c, &id);
    if (a) {
        a->at_s = c->at_s;
        a->place = c->both_places ? ALSO_X : 0u;
    }
    if (!c->both_places || c->settled || (recording && c->settle_recorded && c->settle_graph == id)) return LASGD_OK;
    const bool as_it_goes = recording && a && (reads || !(c->settle_mask & ~rewritten));
    if (as_it_goes) {
        a->at_s = c->settle_mask;
        a->place |= reads ? LOOK : LOOK | SETTLES;
        if (reads) return LASGD_OK;
    } else {
        hipLaunchKernelGGL(settle_kernel, dim3(kSettleBlocks), dim3(256), 0, c->main, c->x32, c->s, c->npad, c->settle_mask, c->settle);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    }
    if (recording) {
        c->settle_recorded = true;
        c->settle_graph = id;
    } else c->settled = true;
    return LASGD_OK;
}

// The launch that would have brought the models back has failed.
void not_settled(lasgd_ctx *c, const ApplyArgs &a)
{
    if (a.place & SETTLES) c->settle_recorded = false;
}

// The L2s of the eight XCDs hold 32 MiB between them and keep it from launch to launch.  A tile meets the same L2 in every kernel
// (workgroup i runs on XCD i mod 8, and rows of items are padded to that), so what a launch touched last is there for the next
// one to start with: every other launch takes its items from the last to the first.  A cycle's us, three states in turn, as before / on one XCD /
// and backwards in turn: K = 4, 2^20 elements m = 2 43.0 / 43.0 / 40.0, m = 4 70.1 / 70.1 / 60.5; 700,003 elements 30.5 / 30.3 / 28.7; 300,001
// 20.0 / 19.3 / 19.2; K = 8, 250,007 24.4 / 22.0 / 21.9, 100,003 18.8 / 17.0 / 16.9.  With the hint (K = 8, m = 4): 30 MB an array 125.7 / 125.7 /
// 123.9, 53 MB 206.1 / 206.3 / 204.7; K = 4, m = 2: 30 MB 74.9 / 74.9 / 74.8, 80 MB 176.6 / 176.7 / 177.9, 112 MB 243 / 243 / 245.5.  So below 64 MiB
// (kBackBelow); below 8 MiB an array the L2s hold all of it either way.
void backwards(lasgd_ctx *c, ApplyArgs &a, uint32_t waves_per_group)
{
    if (waves_per_group != 1u || a.nitems % 8u != 0u || array_bytes(c) < kBackFrom || array_bytes(c) >= kBackBelow) return;
    c->back = !c->back;
    a.back = c->back ? a.nitems - 8u : 0u;
    a.back_mask = c->back ? ~7u : 0u;
}

// Plans before it launches: after the last check of a call, and just before its launch.
lasgd_status launch_apply(lasgd_ctx *c, ApplyPlan &p)
{
    const bool bf16 = c->storage == LASGD_BF16;
    const uint64_t taking = p.has_ext ? p.ext.step_mask | p.ext.merge_mask : c->all;
    const bool writes = p.op != OP_SNAPSHOT && p.op != OP_INIT;
    const lasgd_status st = place_models(c, &p.a, writes ? taking : 0, p.op == OP_SNAPSHOT);
    if (st != LASGD_OK) return st;
    backwards(c, p.a, p.a.wpb);
    const int vec = c->tune.vec;
    int nt = hint_of(c, p.op == OP_STEP && c->fused_cycle ? USE_FUSED : USE_CYCLE);
    if (nt == 3 && vec == 1 && word_first(p.op, (uint64_t)c->K * c->npad, all_at_s(p.a))) nt |= 4;
    const ExtArgs *xa = p.has_ext ? &p.ext : nullptr;
    hipError_t e = hipSuccess;
    switch (p.op) {
    case OP_STEP: e = launch_op<OP_STEP>(p.a, xa, p.grid, p.bs, c->main, vec, nt, bf16); break;
    case OP_MERGE: e = launch_op<OP_MERGE>(p.a, xa, p.grid, p.bs, c->main, vec, nt, bf16); break;
    case OP_STEP_MERGE: e = launch_op<OP_STEP_MERGE>(p.a, xa, p.grid, p.bs, c->main, vec, nt, bf16); break;
    case OP_STEP_MEAN:
        if (bf16) e = launch_one<OP_STEP_MEAN, true>(p.a, p.grid, p.bs, c->main);
        else e = launch_one<OP_STEP_MEAN, false>(p.a, p.grid, p.bs, c->main);
        break;
    case OP_SNAPSHOT: e = launch_op<OP_SNAPSHOT>(p.a, xa, p.grid, p.bs, c->main, vec, nt, bf16); break;
    default: e = launch_vec<OP_INIT, true>(p.a, nullptr, p.grid, p.bs, c->main, vec, nt); break;
    }
    if (e != hipSuccess) {
        not_settled(c, p.a);
        return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    }
    if (bf16 && p.op != OP_SNAPSHOT) {
        const bool merging = p.op == OP_MERGE || p.op == OP_STEP_MERGE;
        const uint64_t stepped = p.op == OP_MERGE ? 0 : xa ? xa->step_mask : c->all, merged = !merging ? 0 : xa ? xa->merge_mask : c->all;
        c->at_s &= ~(stepped | merged);
        if (p.a.resnap && !c->both_places) c->at_s |= merged;
    }
    return LASGD_OK;
}

lasgd_status enqueue_apply(lasgd_ctx *c, int op, float lr, int resnap, const ExtArgs *xa = nullptr)
{
    ApplyPlan p;
    lasgd_status st = plan_apply(c, p, op, lr, resnap, xa);
    if (st != LASGD_OK) return st;
    return launch_apply(c, p);
}

constexpr uint64_t kWavesOnChip = 256u * 32u;     // 256 CUs hold at most 32 waves each
// Streaming, lasgd_step_merge_average holds up to this many replicas in one workgroup; beyond, it takes two kernels.
// Where the update writes s alone (bf16, place_models) it loses less to the shape: two kernels / one, an update every
// step, ResNet-18 list K = 14 1261 / 1137, 18 1612 / 1517, 22 1946 / 1880, 24 2131 / 2076, MobileNetV2 K = 13 359 / 335, 22 595 / 586,
// 24 648 / 639; every second step, ResNet-18 K = 13 2321 / 2201, 20 3586 / 3494; beyond 24, every step, K = 28 2501 / 2465, 32 2844 / 2846,
// MobileNetV2 K = 32 848 / 881, 40 1056 / 1136.
uint32_t one_kernel_max(const lasgd_ctx *c) { return c->both_places ? 12u : 24u; }

// The replica-group kernels: one workgroup per tile, W waves, R replicas per wave.
struct GroupShape {
    uint32_t R, W, passes;
    bool staged;         // a wave's loads in two groups, the second when the first has arrived
    dim3 grid, bs;
    size_t lds;
};

// Does the SGD All-Reduce step take two kernels, given the array for the mean gradient between them?  Streaming, the
// workgroups of the one kernel, which hold all replicas of a tile, cost more with every replica; the two move 8 bytes a
// parameter more and need a second launch.  us, one kernel / two (three states in turn): ResNet-18 list K = 4 150 / 158, 6 233 / 233,
// 8 310 / 303, 12 465 / 449, 16 622 / 591, bf16 K = 5 199 / 200, 8 312 / 303, 16 666 / 595; ResNet-50 K = 8 673 / 652, bf16 695 / 655;
// MobileNetV2 K = 24 308 / 269.  In turn | with other work between: 41 MB an array K = 12 40.5 / 39.8    42.4 / 42.7, bf16 42.5 / 41.6    44.0 / 46.3,
// K = 32 44.0 / 39.2    46.0 / 42.0; 56 MB K = 12 55.3 / 51.0    54.6 / 53.9, bf16 59.9 / 53.9    58.0 / 57.9; 80 MB K = 8 72.5 / 75.1, K = 12 74.2 / 70.9
//    75.1 / 73.2; 112 MB K = 8 110 / 102    105.6 / 104.3, bf16 K = 6 103 / 103    105 / 105.  In the memory-side cache the second launch costs more
// than it gives (10 MB, K = 24 12.4 / 14.6).
bool mean_grad_first(const lasgd_ctx *c)
{
    const uint64_t array = array_bytes(c);
    return c->K >= (array >= (112ull << 20) ? 8 : array >= (56ull << 20) ? 12 : 16) && hint_of(c, USE_SGD_AR) == 3 && c->tune.vec == 1 &&
           c->tune.group_r <= 0;
}

// The array for the mean gradient, 1/(2K + 1) of what a context holds already, for those alone that make the call it is for.  The
// first such call takes one kernel, and the array is asked for while that runs, so no call is longer for it (asked for before
// the launch it made a first call of the ResNet-50 list, K = 8, 778 us in place of 707).  A call that is being recorded has no
// kernel to wait beside: there it comes first.  Where there is no memory for it, the step stays in one kernel.
void reserve_mean_grad(lasgd_ctx *c)
{
    c->gbar_tried = true;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;        // allowed while a stream of this thread is being recorded, and not recorded
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (hipMalloc((void **)&c->gbar, c->npad * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        c->gbar = nullptr;
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
}

// kind 0: SGD All-Reduce step; kind 1: fused step + global update + next mean
GroupShape group_shape(const lasgd_ctx *c, int kind)
{
    const bool at_s = c->at_s == c->all;
    GroupShape g{};
    const uint32_t K = (uint32_t)c->K;
    const bool streaming = (hint_of(c, kind == 0 ? USE_SGD_AR : USE_FUSED) & 3) != 0;
    // Replicas a wave takes at a time, us on MI355X.
    // SGD-AR, streaming: one, with the models asked for when the gradients are there (staged), up to K = 12, and beyond where
    // two workgroups of such waves fill 30 of a CU's 32 slots or more (13 and 14 fill 26 and 28).  One / two a wave: ResNet-18 list K = 12
    // 466 / 481, 13 520 / 519, 16 630 / 698, bf16 480 / 487, 551 / 536, 662 / 695; ResNet-50 K = 13 1190 / 1170, bf16
    // 1320 / 1217.  All loads at once / staged: ResNet-18 bf16 K = 6 260 / 234, 8 320 / 311, fp32 K = 10 406 / 389, K = 16
    // 727 / 630.  Two against four: MobileNetV2 K = 24 304 / 318, K = 32 433 / 411.
    // SGD-AR in the memory-side cache: one a wave while all waves fit the chip at once (small ragged list bf16 K = 8 4.3 / 5.2),
    // else two from K = 4 on (2^20 elements bf16 K = 4 16.8 / 15.0, MobileNetV2 bf16 K = 6 82 / 69, fp32 K = 3 32.9 / 32.9).
    // Fused update (its sum is the last thing a workgroup does): one a wave up to K = 9, streaming see below; in the
    // memory-side cache one / two at 2^20 elements K = 8 44.1 / 43.3, K = 16 100 / 92; 300,000 elements K = 16 27.1 / 25.6.
    const bool paced = streaming && kind == 1 && K <= one_kernel_max(c) && c->tune.group_r <= 0;
    const bool once = !c->both_places;
    const bool at_once = (uint64_t)c->tables->ntiles * K <= kWavesOnChip;
    if (paced && once) g.R = K <= 6u ? 1u : 2u;
    else if (kind == 1) g.R = K <= 9u || (paced && K >= 12u) ? 1u : K <= 2u * kGroupWaves ? 2u : 4u;
    else if (streaming) g.R = K <= 12u || (2u * K >= 30u && K <= kGroupWaves) ? 1u : K <= 24u ? 2u : 4u;
    else g.R = K <= (at_once ? kGroupWaves : 3u) ? 1u : K <= 2u * kGroupWaves ? 2u : 4u;
    if (c->tune.group_r > 0) g.R = (uint32_t)c->tune.group_r;
    if (g.R > K) g.R = K >= 4 ? 4 : K >= 2 ? 2 : 1;
    g.W = (K + g.R - 1) / g.R;
    if (g.W > kGroupWaves) g.W = kGroupWaves;
    g.passes = (K + g.W * g.R - 1) / (g.W * g.R);
    uint64_t blocks = c->tables->ntiles;
    if (c->tune.max_blocks > 0 && blocks > (uint64_t)c->tune.max_blocks) blocks = (uint64_t)c->tune.max_blocks;
    g.grid = dim3((uint32_t)blocks);
    g.bs = dim3(64u * g.W);
    g.lds = (size_t)K * 256u * sizeof(float);
    g.staged = kind == 0 && streaming && g.R == 1u;
    if (paced) {
        // Paced like the other kernels (pace_lds): about 60 KiB of loads in flight per CU, in whole workgroups.  Up to
        // K = 9 a wave issues all the loads of its replica, 4 KiB, and the LDS a workgroup asks for leaves room for 16 to
        // 21 waves.  From K = 10 on one workgroup a CU is too few and two are too many (70 to 96 KiB), so a wave asks for
        // the gradients when the rest is there: two workgroups then start with 3 KiB a replica, 60 to 72 KiB.  Two
        // replicas a wave, unless two workgroups of one-replica waves fill three quarters of the CU's 32 slots (K = 12).  us, means
        // over eight placements in memory, one replica and everything at once / one, staged / two, staged: ResNet-18 list bf16
        // K = 9 527 / 555 / 528, 10 586 / 607 / 579, 11 643 / 657 / 638, 12 717 / 687 / 699, fp32 K = 12 710 / 688 / 688;
        // ResNet-50 bf16 K = 12 1540 / 1520 / 1530; MobileNetV2 bf16 K = 12 218 / 214 / 219 (bf16 with
        // the model in both places).  The SGD-AR kernel waits for its gradients in the middle, and holding its waves back costs it.
        g.staged = K > 9u;
        size_t pace = g.staged ? 43u * kLdsGranule : (size_t)6u * kLdsGranule * g.W;      // 43 granules: two a CU
        if (once && K > 6u) {
            // 2.5 KiB of loads a replica where every model is in s, 3.5 where a step came between: two replicas a wave, everything
            // at once, and whole workgroups that come to about 16 waves a CU, or 13.  From 19 replicas on two groups are too much,
            // and the gradients wait again.  us, two updates: the rule of fp32 / this, every model in s: ResNet-18 list K = 7 575 / 571,
            // 8 675 / 648, 9 761 / 725, 10 890 / 802, 12 984 / 981, ResNet-50 K = 7 1265 / 1230, 8 1466 / 1404, 10 1934 / 1759, 12 2212 /
            // 2172; at two, three, four, five groups a CU K = 7 - / 592 / 571 / 576, K = 9 737 (four) / 725 (three); a step between: ResNet-18
            // K = 8 1370 / 1340, 10 1741 / 1692, 12 2027 / 2012, MobileNetV2 K = 12 632 / 629.  At once / staged: K = 17 1442 / 1450,
            // 18 1517 / 1525, 20 1706 / 1705, 22 1886 / 1880, 24 2109 / 2076.
            g.staged = K > 18u;
            const uint32_t groups = ((at_s ? 16u : 13u) + g.W / 2u) / g.W;
            pace = kCuLds / (groups > 2u ? groups : 2u) / kLdsGranule * kLdsGranule;
        }
        g.lds = pace > g.lds ? (pace < kMaxLds ? pace : kMaxLds) : g.lds;
    }
    return g;
}

template <int KIND, bool BF16, int NT, bool ST>
hipError_t launch_group_r(const ApplyArgs &a, const GroupShape &g, hipStream_t st)
{
#define LASGD_GROUP_AT(RR, P)                                                                            \
    do {                                                                                                 \
        if constexpr (KIND == 0) hipLaunchKernelGGL((sgd_ar_kernel<RR, BF16, NT, ST, P>), g.grid, g.bs, g.lds, st, a, g.passes); \
        else hipLaunchKernelGGL((step_merge_mean_kernel<RR, BF16, NT, ST, P>), g.grid, g.bs, g.lds, st, a, g.passes); \
    } while (0)
#define LASGD_GROUP(RR)                                                                                  \
    do {                                                                                                 \
        if (BF16 && (a.place & SETTLES)) LASGD_GROUP_AT(RR, BF16 ? PLACE_SETTLE : PLACE_AT_S);                      \
        else if (BF16 && KIND == 1 && all_at_s(a)) LASGD_GROUP_AT(RR, BF16 && KIND == 1 ? PLACE_ALL_IN_S : PLACE_AT_S); \
        else LASGD_GROUP_AT(RR, PLACE_AT_S);                                                             \
    } while (0)
    if (g.R == 1) LASGD_GROUP(1);
    else if (g.R == 2) LASGD_GROUP(2);
    else LASGD_GROUP(4);
#undef LASGD_GROUP
#undef LASGD_GROUP_AT
    return hipGetLastError();
}

// kind 0: SGD All-Reduce step; kind 1: fused step + global update + next mean
hipError_t launch_group(lasgd_ctx *c, int kind, ApplyArgs &a, const GroupShape &g, int nt)
{
    const bool hint = (nt & 3) != 0, bf16 = c->storage == LASGD_BF16;
    const hipStream_t st = c->main;
    a.wpb = g.W;
    a.nwaves = g.grid.x;
    a.nitems = a.ntiles & ~7u;
    if (!hint) backwards(c, a, 1u);              // a tile a workgroup
#define LASGD_KIND(KIND, BF)                                                                              \
    (!hint ? launch_group_r<KIND, BF, 0, false>(a, g, st)                                                 \
           : g.staged ? launch_group_r<KIND, BF, 3, true>(a, g, st) : launch_group_r<KIND, BF, 3, false>(a, g, st))
    if (kind == 0) return bf16 ? LASGD_KIND(0, true) : LASGD_KIND(0, false);
    return bf16 ? LASGD_KIND(1, true) : LASGD_KIND(1, false);
#undef LASGD_KIND
}

template <bool EXT>
hipError_t launch_average(const AvgArgs &a, dim3 grid, hipStream_t st, int split, bool nt, uint32_t bs1)
{
    if (split == 1) {
        if (nt) hipLaunchKernelGGL((average_kernel<3, EXT>), grid, dim3(bs1), 0, st, a);
        else hipLaunchKernelGGL((average_kernel<0, EXT>), grid, dim3(bs1), 0, st, a);
    } else if (split == 2) {
        if (nt) hipLaunchKernelGGL((average_split_kernel<2, 3, EXT>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((average_split_kernel<2, 0, EXT>), grid, dim3(256), 0, st, a);
    } else {
        if (nt) hipLaunchKernelGGL((average_split_kernel<4, 3, EXT>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((average_split_kernel<4, 0, EXT>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

// Enqueue the mean of the replicas in `mask` on `stream`.
lasgd_status enqueue_average(lasgd_ctx *c, uint64_t mask, bool elastic, hipStream_t stream, int split)
{
    AvgArgs a{};
    a.s = c->s;
    a.z = c->z;
    a.npad = c->npad;
    a.nvec = c->npad / 4;
    uint32_t kp = 0;
    for (int k = 0; k < c->K; ++k)
        if ((mask >> k) & 1ull) a.idx[kp++] = (uint8_t)k;
    a.K = kp;
    a.use_mul = is_pow2(kp) ? 1 : 0;
    a.inv_k = 1.0 / (double)kp;
    a.k_as_double = (double)kp;
    a.elastic = elastic ? 1 : 0;
    a.beta = (double)c->beta;
    a.one_minus_beta = 1.0 - (double)c->beta;
    const uint32_t bs1 = 64u * (uint32_t)c->tune.waves_per_block;           // block size of the unsplit kernel
    const uint64_t cols = split == 1 ? bs1 : 256u / (uint32_t)split;
    uint64_t blocks = (a.nvec + cols - 1) / cols;
    if (c->tune.avg_max_blocks > 0 && blocks > (uint64_t)c->tune.avg_max_blocks) blocks = (uint64_t)c->tune.avg_max_blocks;
    if (blocks > 0x7fffffffull) blocks = 0x7fffffffull;
    a.blocks = (uint32_t)blocks;
    a.threads = split == 1 ? bs1 : 256u;
    const dim3 grid((uint32_t)blocks);
    const bool nt = (hint_of(c, USE_CYCLE) & 1) != 0;
    const bool ext = elastic || mask != c->all;
    hipError_t e = ext ? launch_average<true>(a, grid, stream, split, nt, bs1) : launch_average<false>(a, grid, stream, split, nt, bs1);
    if (e != hipSuccess) return fail(c, LASGD_ERR_HIP, "average launch failed: %s", hipGetErrorString(e));
    return LASGD_OK;
}

lasgd_status check_ready_to_step(lasgd_ctx *c, float lr)
{
    if (!std::isfinite(lr)) return fail(c, LASGD_ERR_INVALID, "learning rate is not finite");
    if (c->n_bound != c->K) return fail(c, LASGD_ERR_STATE, "%d of %d replicas are bound", c->n_bound, c->K);
    if (c->storage == LASGD_BF16 && !c->master_ready)
        return fail(c, LASGD_ERR_STATE, "bf16 storage: call lasgd_init_master first");
    return LASGD_OK;
}

// Until no queued clear of the gradients can still read the records.  Clears run on streams that the caller names and may
// since have destroyed, so this waits for the device: an event after each clear would do for the stream alone, but costs
// every clear 3.5 us on the device (MobileNetV2 list, K = 4, clear + accumulate + step twice 251 us without, 258 with).
lasgd_status wait_for_clears(lasgd_ctx *c)
{
    if (!c->clearing && !c->clear_in_graph) return LASGD_OK;
    LASGD_HIP(c, hipDeviceSynchronize());
    c->clearing = false;
    return LASGD_OK;
}

void release(lasgd_ctx *c)
{
    if (c->arena) (void)hipFree(c->arena);
    for (const lasgd_ctx::Tables &t : c->tables_by_vec)
        if (t.mem) (void)hipFree(t.mem);
    if (c->records) (void)hipFree(c->records);
    if (c->gbar) (void)hipFree(c->gbar);
    if (c->evA) (void)hipEventDestroy(c->evA);
    if (c->evZ) (void)hipEventDestroy(c->evZ);
    delete c;
}

} // namespace

static lasgd_status create_impl(const lasgd_config *cfg, lasgd_ctx **out)
{
    if (out) *out = nullptr;
    if (!cfg || !out) return fail(nullptr, LASGD_ERR_INVALID, "NULL argument");
    if (cfg->K < 1 || cfg->K > kMaxK) return fail(nullptr, LASGD_ERR_INVALID, "K = %d outside 1..%d", cfg->K, kMaxK);
    if (cfg->n_tensors < 1 || !cfg->numel) return fail(nullptr, LASGD_ERR_INVALID, "empty parameter list");
    if (cfg->storage != LASGD_F32 && cfg->storage != LASGD_BF16) return fail(nullptr, LASGD_ERR_INVALID, "unknown storage dtype");
    if (!std::isfinite(cfg->momentum) || cfg->momentum < 0.f) return fail(nullptr, LASGD_ERR_INVALID, "momentum must be finite and >= 0");
    if (!std::isfinite(cfg->wd_scalar) || cfg->wd_scalar < 0.f) return fail(nullptr, LASGD_ERR_INVALID, "weight decay must be finite and >= 0");
    lasgd_ctx *c = new (std::nothrow) lasgd_ctx;
    if (!c) return fail(nullptr, LASGD_ERR_ALLOC, "out of host memory");
    c->K = cfg->K;
    c->n_tensors = cfg->n_tensors;
    c->storage = cfg->storage;
    c->mu = cfg->momentum;
    c->nesterov = cfg->nesterov ? 1 : 0;
    c->wd_scalar = cfg->wd_scalar;
    c->main = (hipStream_t)cfg->main_stream;
    c->side = (hipStream_t)cfg->side_stream;
    uint64_t off = 0, total = 0;
    for (int32_t i = 0; i < cfg->n_tensors; ++i) {
        if (cfg->numel[i] < 1) { delete c; return fail(nullptr, LASGD_ERR_INVALID, "numel[%d] = %lld", i, (long long)cfg->numel[i]); }
        const float w = cfg->weight_decay ? cfg->weight_decay[i] : cfg->wd_scalar;
        if (!std::isfinite(w) || w < 0.f) { delete c; return fail(nullptr, LASGD_ERR_INVALID, "weight_decay[%d] must be finite and >= 0", i); }
        c->numel.push_back(cfg->numel[i]);
        c->wd.push_back(w);
        c->aoff.push_back(off);
        total += (uint64_t)cfg->numel[i];
        off += round_up((uint64_t)cfg->numel[i], kArenaAlign);
        if (off > kMaxNpad) { delete c; return fail(nullptr, LASGD_ERR_UNSUPPORTED, "more than %llu elements per replica", (unsigned long long)kMaxNpad); }
    }
    c->packed = off;
    c->npad = padded(off);
    c->all = c->K == 64 ? ~0ull : ((1ull << c->K) - 1ull);
    c->ntotal = total;
    c->bound.assign((size_t)c->K, 0);
    c->h_xptr.assign((size_t)c->K * c->n_tensors, nullptr);
    c->tune = default_tuning(*c);

#define CREATE_HIP(call)                                                                       \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess) {                                                                \
            (void)hipGetLastError();                                                           \
            lasgd_status st_ = fail(nullptr, e_ == hipErrorOutOfMemory ? LASGD_ERR_ALLOC : LASGD_ERR_HIP, \
                                    "%s failed: %s", #call, hipGetErrorString(e_));            \
            release(c);                                                                        \
            return st_;                                                                        \
        }                                                                                      \
    } while (0)

    CREATE_HIP(hipGetDevice(&c->device));
    const bool bf16 = c->storage == LASGD_BF16;
    const uint64_t per = c->npad * sizeof(float);
    c->both_places = !bf16 || c->K * per < kOneCopyFrom;
    const uint64_t n_arrays = (uint64_t)c->K * (bf16 ? 3 : 2) + 1;       // v, s (, x32), z
    const uint64_t bytes = n_arrays * per + (bf16 ? kSettleWords * sizeof(uint32_t) : 0u);
    CREATE_HIP(hipMalloc((void **)&c->arena, bytes));
    CREATE_HIP(hipMemsetAsync(c->arena, 0, bytes, c->main));
    c->v = (float *)c->arena;
    c->s = c->v + (uint64_t)c->K * c->npad;
    c->z = c->s + (uint64_t)c->K * c->npad;
    c->x32 = bf16 ? c->z + c->npad : nullptr;
    c->settle = bf16 ? (uint32_t *)(c->x32 + (uint64_t)c->K * c->npad) : nullptr;
    const size_t tab = (size_t)c->K * c->n_tensors * sizeof(Record);
    CREATE_HIP(hipMalloc((void **)&c->records, tab));
    CREATE_HIP(hipMemset(c->records, 0, tab));
    CREATE_HIP(hipEventCreateWithFlags(&c->evA, hipEventDisableTiming));
    CREATE_HIP(hipEventCreateWithFlags(&c->evZ, hipEventDisableTiming));
    lasgd_status st = upload_tables(c, c->tune.vec);
    if (st != LASGD_OK) {
        g_create_error = c->err;
        release(c);
        return st;
    }
    CREATE_HIP(hipStreamSynchronize(c->main));
#undef CREATE_HIP
    *out = c;
    return LASGD_OK;
}

extern "C" {

// Host containers may throw on exhaustion; nothing may leave through the C ABI.
lasgd_status lasgd_create(const lasgd_config *cfg, lasgd_ctx **out)
{
    try {
        return create_impl(cfg, out);
    } catch (...) {
        if (out) *out = nullptr;
        try { g_create_error = "out of host memory"; } catch (...) {}
        return LASGD_ERR_ALLOC;
    }
}

lasgd_status lasgd_bind(lasgd_ctx *c, int32_t k, void *const *params, void *const *grads)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!params || !grads) return fail(c, LASGD_ERR_INVALID, "NULL pointer array");
    if (k < 0 || k >= c->K) return fail(c, LASGD_ERR_INVALID, "replica %d outside 0..%d", k, c->K - 1);
    for (int32_t t = 0; t < c->n_tensors; ++t) {
        if (!params[t] || !grads[t]) return fail(c, LASGD_ERR_INVALID, "NULL buffer for tensor %d", t);
        if (((uintptr_t)params[t] | (uintptr_t)grads[t]) & 15u)
            return fail(c, LASGD_ERR_INVALID, "buffer of tensor %d is not 16-byte aligned", t);
    }
    std::vector<Record> recs;
    try {
        recs.resize((size_t)c->n_tensors);
    } catch (...) {
        return fail(c, LASGD_ERR_ALLOC, "out of host memory");
    }
    // every reader of the records: the kernels on the main stream, and clears on streams of the caller's
    LASGD_HIP(c, hipStreamSynchronize(c->main));
    const lasgd_status st = wait_for_clears(c);
    if (st != LASGD_OK) return st;
    const size_t base = (size_t)k * c->n_tensors;
    for (size_t t = 0; t < recs.size(); ++t)
        recs[t] = Record{(uint64_t)(uintptr_t)params[t], (uint64_t)(uintptr_t)grads[t], (uint32_t)(c->aoff[t] / kArenaAlign),
                         (uint32_t)c->numel[t], c->wd[t], 0u};
    LASGD_HIP(c, hipMemcpy(c->records + base, recs.data(), recs.size() * sizeof(Record), hipMemcpyHostToDevice));
    memcpy(&c->h_xptr[base], params, recs.size() * sizeof(void *));
    if (!c->bound[(size_t)k]) {
        c->bound[(size_t)k] = 1;
        ++c->n_bound;
    }
    return LASGD_OK;
}

lasgd_status lasgd_init_master(lasgd_ctx *c)
{
    if (!c) return LASGD_ERR_INVALID;
    if (c->storage != LASGD_BF16) return fail(c, LASGD_ERR_STATE, "storage is fp32: there is no master copy");
    if (c->n_bound != c->K) return fail(c, LASGD_ERR_STATE, "%d of %d replicas are bound", c->n_bound, c->K);
    if (c->pending_mask) return fail(c, LASGD_ERR_STATE, "an average is in flight");
    lasgd_status st = enqueue_apply(c, OP_INIT, 0.f, 0);
    if (st != LASGD_OK) return st;
    c->master_ready = true;
    c->snap_mask = 0;
    return LASGD_OK;
}

// ---- shared by the plain and the extended entry points -------------------
// The plain calls are the extended ones with every replica taking part, one
// step size and alpha = 1; they launch the lean kernels.

static lasgd_status check_mask(lasgd_ctx *c, uint64_t mask, bool may_be_empty, const char *what)
{
    if (mask & ~c->all) return fail(c, LASGD_ERR_INVALID, "%s names replicas beyond K = %d", what, c->K);
    if (!may_be_empty && !mask) return fail(c, LASGD_ERR_INVALID, "%s is empty", what);
    return LASGD_OK;
}

static lasgd_status check_lrs(lasgd_ctx *c, const float *lr, uint64_t mask)
{
    if (!lr) return fail(c, LASGD_ERR_INVALID, "NULL learning-rate array");
    for (int k = 0; k < c->K; ++k)
        if (((mask >> k) & 1ull) && !std::isfinite(lr[k])) return fail(c, LASGD_ERR_INVALID, "learning rate of replica %d is not finite", k);
    return LASGD_OK;
}

static bool fill_ext(const lasgd_ctx *c, ExtArgs &x, const float *lr, uint64_t step_mask, uint64_t merge_mask)
{
    x.step_mask = step_mask;
    x.merge_mask = merge_mask;
    x.alpha = c->alpha;
    bool uniform = true;
    float first = 0.f;
    bool have = false;
    for (int k = 0; k < c->K; ++k) {        // the entries beyond K stay zero, as the caller made them
        const bool in = ((step_mask >> k) & 1ull) && lr;
        x.neg_lr_k[k] = in ? -lr[k] : 0.f;
        if (in) {
            if (!have) { first = lr[k]; have = true; }
            else if (lr[k] != first) uniform = false;
        }
    }
    return uniform;
}

static lasgd_status do_local_step(lasgd_ctx *c, const float *lr_k, float lr, uint64_t mask)
{
    lasgd_status st = check_ready_to_step(c, lr_k ? 0.f : lr);
    if (st != LASGD_OK) return st;
    if (!lr_k && mask == c->all) return enqueue_apply(c, OP_STEP, lr, 0);
    if ((st = check_mask(c, mask, true, "mask")) != LASGD_OK) return st;
    if ((st = check_lrs(c, lr_k, mask)) != LASGD_OK) return st;
    if (!mask) return LASGD_OK;                        // nobody steps: nothing to enqueue
    ExtArgs x{};
    const bool uniform = fill_ext(c, x, lr_k, mask, 0);
    if (uniform && mask == c->all) return enqueue_apply(c, OP_STEP, lr_k[0], 0);
    return enqueue_apply(c, OP_STEP, 0.f, 0, &x);
}

static lasgd_status do_snapshot(lasgd_ctx *c, uint64_t mask)
{
    lasgd_status st = check_ready_to_step(c, 0.f);
    if (st != LASGD_OK) return st;
    if ((st = check_mask(c, mask, false, "mask")) != LASGD_OK) return st;
    if (mask & c->pending_mask)
        return fail(c, LASGD_ERR_STATE, "an average over some of these replicas is in flight and not merged: s may still be read");
    note_recording(c);
    const uint64_t copied = mask & ~c->at_s;           // a model that is in s only has been sent already
    if (copied == c->all) st = enqueue_apply(c, OP_SNAPSHOT, 0.f, 0);
    else if (copied) {
        ExtArgs x{};
        fill_ext(c, x, nullptr, copied, 0);
        st = enqueue_apply(c, OP_SNAPSHOT, 0.f, 0, &x);
    }
    if (st != LASGD_OK) return st;
    c->snap_mask |= mask;
    return LASGD_OK;
}

static lasgd_status do_average(lasgd_ctx *c, uint64_t mask)
{
    // every refusal comes before the first event or launch
    lasgd_status st = check_mask(c, mask, false, "mask");
    if (st != LASGD_OK) return st;
    if (c->pending_mask) return fail(c, LASGD_ERR_STATE, "the previous average has not been merged by all its participants");
    if (mask & ~c->snap_mask) return fail(c, LASGD_ERR_STATE, "no snapshot to average for some of these replicas");
    const bool captured = is_capturing(c->main);
    const bool on_main = c->side == c->main || mean_on_main((uint32_t)__builtin_popcountll(mask), c->packed);
    const hipStream_t stream = on_main ? c->main : c->side;
    if (!on_main) {
        LASGD_HIP(c, hipEventRecord(c->evA, c->main));
        LASGD_HIP(c, hipStreamWaitEvent(c->side, c->evA, 0));
    }
    // the first mean initialises the centre: there is no earlier z to blend with
    const bool elastic = c->beta != 1.f && c->center_valid;
    if (c->tune.race_probe > 0 && !elastic) {
        // debugging aid: z is poisoned on the mean's stream just before the mean rewrites it
        hipLaunchKernelGGL(poison_kernel, dim3(1024), dim3(256), 0, stream, c->z, c->npad);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(c, LASGD_ERR_HIP, "poison launch failed: %s", hipGetErrorString(e));
    }
    st = enqueue_average(c, mask, elastic, stream, c->tune.avg_split);
    if (st != LASGD_OK) return st;
    // from here on that stream reads s and writes z: the state says so even if the event below fails
    c->pending_mask = mask;
    c->avg_ever = true;
    c->center_valid = true;
    c->avg_in_graph = captured;
    c->fused_cycle = false;
    c->z_on_main = on_main;
    LASGD_HIP(c, hipEventRecord(c->evZ, stream));
    return LASGD_OK;
}

static lasgd_status do_merge(lasgd_ctx *c, int op, const float *lr_k, float lr, uint64_t step_mask,
                             uint64_t merge_mask, int32_t resnapshot)
{
    lasgd_status st = check_ready_to_step(c, lr_k ? 0.f : lr);
    if (st != LASGD_OK) return st;
    if ((st = check_mask(c, merge_mask, false, "merge mask")) != LASGD_OK) return st;
    if ((st = check_mask(c, step_mask, true, "step mask")) != LASGD_OK) return st;
    if (op == OP_STEP_MERGE && lr_k && (st = check_lrs(c, lr_k, step_mask)) != LASGD_OK) return st;
    if (!c->pending_mask) return fail(c, LASGD_ERR_STATE, "no average launched since the last merge");
    if (merge_mask & ~c->pending_mask)
        return fail(c, LASGD_ERR_STATE, "some of these replicas did not take part in the pending average or have merged already");
    ExtArgs x{};
    float same[64];
    for (int k = 0; k < 64; ++k) same[k] = lr;
    const bool uniform = fill_ext(c, x, lr_k ? lr_k : same, step_mask, merge_mask);
    const bool plain = merge_mask == c->all && c->alpha == 1.f &&
                       (op == OP_MERGE || (step_mask == c->all && uniform));
    ApplyPlan p;
    if (plain) st = plan_apply(c, p, op, lr_k ? lr_k[0] : lr, resnapshot ? 1 : 0);
    else st = plan_apply(c, p, op, 0.f, resnapshot ? 1 : 0, &x);
    if (st != LASGD_OK) return st;
    // nothing can be refused any more: now the main stream waits for z (unless z is made on this very stream)
    if (!c->z_on_main) LASGD_HIP(c, hipStreamWaitEvent(c->main, c->evZ, 0));
    st = launch_apply(c, p);
    if (st != LASGD_OK) return st;
    c->pending_mask &= ~merge_mask;
    if (resnapshot) c->snap_mask |= merge_mask;
    else c->snap_mask &= ~merge_mask;
    return LASGD_OK;
}

lasgd_status lasgd_local_step(lasgd_ctx *c, float lr)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_local_step(c, nullptr, lr, c->all);
}

lasgd_status lasgd_local_step_ex(lasgd_ctx *c, const float *lr, uint64_t mask)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!lr) return fail(c, LASGD_ERR_INVALID, "NULL learning-rate array");
    return do_local_step(c, lr, 0.f, mask);
}

lasgd_status lasgd_zero_grads(lasgd_ctx *c, void *stream)
{
    if (!c) return LASGD_ERR_INVALID;
    if (c->n_bound != c->K) return fail(c, LASGD_ERR_STATE, "%d of %d replicas are bound", c->n_bound, c->K);
    ApplyArgs a{};
    fill_common(c, a);
    a.chunk = a.ntiles;
    a.by_chunk = make_div(a.ntiles);
    a.nitems = a.ntiles * a.K;           // upload_tables refuses more than 2^31 / 64 tiles
    a.nwaves = c->tune.max_blocks > 0 && a.nitems > (uint32_t)c->tune.max_blocks ? (uint32_t)c->tune.max_blocks : a.nitems;
    const dim3 grid(a.nwaves), bs(64);
    const hipStream_t st = (hipStream_t)stream;
    const bool hint = (hint_of(c, USE_ZERO) & 2) != 0;
    if (c->storage == LASGD_BF16) {
        if (hint) hipLaunchKernelGGL((zero_grads_kernel<true, 2>), grid, bs, 0, st, a);
        else hipLaunchKernelGGL((zero_grads_kernel<true, 0>), grid, bs, 0, st, a);
    } else {
        if (hint) hipLaunchKernelGGL((zero_grads_kernel<false, 2>), grid, bs, 0, st, a);
        else hipLaunchKernelGGL((zero_grads_kernel<false, 0>), grid, bs, 0, st, a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    c->clearing = true;
    if (is_capturing(st)) c->clear_in_graph = true;
    return LASGD_OK;
}

lasgd_status lasgd_snapshot(lasgd_ctx *c)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_snapshot(c, c->all);
}

lasgd_status lasgd_snapshot_ex(lasgd_ctx *c, uint64_t mask)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_snapshot(c, mask);
}

lasgd_status lasgd_average(lasgd_ctx *c)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_average(c, c->all);
}

lasgd_status lasgd_average_ex(lasgd_ctx *c, uint64_t mask)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_average(c, mask);
}

lasgd_status lasgd_average_done(lasgd_ctx *c, int32_t *done)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!done) return fail(c, LASGD_ERR_INVALID, "NULL argument");
    if (!c->avg_ever) return fail(c, LASGD_ERR_STATE, "no average has been launched");
    if (c->avg_in_graph)
        return fail(c, LASGD_ERR_STATE, "the last average was recorded into a graph: its completion cannot be polled here");
    hipError_t e = hipEventQuery(c->evZ);
    if (e == hipSuccess) *done = 1;
    else if (e == hipErrorNotReady) *done = 0;
    else return fail(c, LASGD_ERR_HIP, "hipEventQuery failed: %s", hipGetErrorString(e));
    return LASGD_OK;
}

lasgd_status lasgd_merge(lasgd_ctx *c, int32_t resnapshot)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_merge(c, OP_MERGE, nullptr, 0.f, 0, c->all, resnapshot);
}

lasgd_status lasgd_merge_ex(lasgd_ctx *c, uint64_t mask, int32_t resnapshot)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_merge(c, OP_MERGE, nullptr, 0.f, 0, mask, resnapshot);
}

lasgd_status lasgd_step_merge(lasgd_ctx *c, float lr, int32_t resnapshot)
{
    if (!c) return LASGD_ERR_INVALID;
    return do_merge(c, OP_STEP_MERGE, nullptr, lr, c->all, c->all, resnapshot);
}

lasgd_status lasgd_step_merge_ex(lasgd_ctx *c, const float *lr, uint64_t step_mask, uint64_t merge_mask,
                                 int32_t resnapshot)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!lr) return fail(c, LASGD_ERR_INVALID, "NULL learning-rate array");
    return do_merge(c, OP_STEP_MERGE, lr, 0.f, step_mask, merge_mask, resnapshot);
}

lasgd_status lasgd_set_elastic(lasgd_ctx *c, float alpha, float beta)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!(alpha >= 0.f && alpha <= 1.f) || !(beta >= 0.f && beta <= 1.f))
        return fail(c, LASGD_ERR_INVALID, "alpha and beta must lie in [0, 1]");
    c->alpha = alpha;
    c->beta = beta;
    return LASGD_OK;
}

lasgd_status lasgd_sgd_ar_step(lasgd_ctx *c, float lr)
{
    if (!c) return LASGD_ERR_INVALID;
    lasgd_status st = check_ready_to_step(c, lr);
    if (st != LASGD_OK) return st;
    const bool two = mean_grad_first(c);
    if (two && !c->gbar_tried && is_capturing(c->main)) reserve_mean_grad(c);
    if (two && c->gbar) {
        ApplyPlan p;
        if ((st = plan_apply(c, p, OP_STEP_MEAN, lr, 0)) != LASGD_OK) return st;
        p.a.z = c->gbar;
        const dim3 grid(c->tune.max_blocks > 0 && p.a.ntiles > (uint32_t)c->tune.max_blocks ? (uint32_t)c->tune.max_blocks : p.a.ntiles);
        ApplyArgs a = p.a;
        a.nwaves = grid.x;
        if (c->storage == LASGD_BF16) hipLaunchKernelGGL((mean_grad_kernel<true, 3>), grid, dim3(64), 0, c->main, a);
        else hipLaunchKernelGGL((mean_grad_kernel<false, 3>), grid, dim3(64), 0, c->main, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
        return launch_apply(c, p);
    }
    ApplyArgs a{};
    fill_common(c, a);
    a.neg_lr = -lr;
    if ((st = place_models(c, &a, c->all)) != LASGD_OK) return st;
    const GroupShape g = group_shape(c, 0);
    hipError_t e = launch_group(c, 0, a, g, hint_of(c, USE_SGD_AR));
    if (e != hipSuccess) {
        not_settled(c, a);
        return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    }
    c->at_s = 0;
    if (two && !c->gbar_tried) reserve_mean_grad(c);
    return LASGD_OK;
}

lasgd_status lasgd_step_merge_average(lasgd_ctx *c, float lr)
{
    if (!c) return LASGD_ERR_INVALID;
    lasgd_status st = check_ready_to_step(c, lr);
    if (st != LASGD_OK) return st;
    if (!c->pending_mask) return fail(c, LASGD_ERR_STATE, "no average launched since the last merge");
    if (c->pending_mask != c->all)
        return fail(c, LASGD_ERR_STATE, "the pending average is partial or partly merged: use lasgd_step_merge_ex and lasgd_average_ex");
    if (c->alpha != 1.f || c->beta != 1.f)
        return fail(c, LASGD_ERR_STATE, "elastic coefficients are set: use lasgd_step_merge and lasgd_average");
    const bool captured = is_capturing(c->main);
    note_recording(c);
    if (c->K > (int32_t)one_kernel_max(c) && (hint_of(c, USE_FUSED) & 3) && c->tune.group_r <= 0) {
        // Streaming from 13 replicas on (25 where the update writes s alone), workgroups that hold all replicas of a tile lose more
        // to their shape than the second pass over s costs: update, then the in-order mean.  us, one kernel / two: K = 12 ResNet-18
        // 667 / 706, bf16 with the model in both places 697 / 716, ResNet-50 bf16 1542 / 1563, MobileNetV2 bf16 217 / 216; K = 13
        // 737 / 765, 768 / 776, 1709 / 1700, 236 / 233; K = 16 MobileNetV2 286 / 282, bf16 293 / 285, ResNet-50 bf16 2102 / 2077.
        ApplyPlan p;
        if ((st = plan_apply(c, p, OP_STEP_MERGE, lr, 1)) != LASGD_OK) return st;
        if (!c->z_on_main) LASGD_HIP(c, hipStreamWaitEvent(c->main, c->evZ, 0));
        if ((st = launch_apply(c, p)) != LASGD_OK) return st;
        c->snap_mask = c->all;
        c->pending_mask = 0;
        if ((st = enqueue_average(c, c->all, false, c->main, 1)) != LASGD_OK) return st;
    } else {
        ApplyArgs a{};
        fill_common(c, a);
        a.neg_lr = -lr;
        a.resnap = 1;
        if (!c->z_on_main) LASGD_HIP(c, hipStreamWaitEvent(c->main, c->evZ, 0));
        if ((st = place_models(c, &a, c->all)) != LASGD_OK) return st;
        const GroupShape g = group_shape(c, 1);
        hipError_t e = launch_group(c, 1, a, g, hint_of(c, USE_FUSED));
        if (e != hipSuccess) {
            not_settled(c, a);
            return fail(c, LASGD_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
        }
        if (!c->both_places) c->at_s = c->all;
    }
    // every replica has merged and re-sent, and the mean of the sent models is (being) written to z
    // on the main stream: the same state as after lasgd_step_merge(lr, 1) + lasgd_average
    c->snap_mask = c->all;
    c->pending_mask = c->all;
    c->avg_in_graph = captured;
    c->fused_cycle = true;
    c->z_on_main = true;
    LASGD_HIP(c, hipEventRecord(c->evZ, c->main));
    return LASGD_OK;
}

lasgd_status lasgd_sync(lasgd_ctx *c)
{
    if (!c) return LASGD_ERR_INVALID;
    LASGD_HIP(c, hipStreamSynchronize(c->main));
    if (c->side != c->main) LASGD_HIP(c, hipStreamSynchronize(c->side));
    return LASGD_OK;
}

lasgd_status lasgd_read_state(lasgd_ctx *c, int32_t which, int32_t k, int32_t tensor, float *dst, int64_t n)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!dst) return fail(c, LASGD_ERR_INVALID, "NULL destination");
    if (which < LASGD_STATE_X || which > LASGD_STATE_Z) return fail(c, LASGD_ERR_INVALID, "unknown state array %d", which);
    if (which == LASGD_STATE_Z) k = 0;
    if (k < 0 || k >= c->K) return fail(c, LASGD_ERR_INVALID, "replica %d outside 0..%d", k, c->K - 1);
    if (tensor < -1 || tensor >= c->n_tensors) return fail(c, LASGD_ERR_INVALID, "tensor %d outside -1..%d", tensor, c->n_tensors - 1);
    const int64_t want = tensor < 0 ? (int64_t)c->ntotal : c->numel[(size_t)tensor];
    if (n != want) return fail(c, LASGD_ERR_INVALID, "n = %lld, expected %lld", (long long)n, (long long)want);
    const bool user_x = which == LASGD_STATE_X && c->storage == LASGD_F32;
    if (user_x && !c->bound[(size_t)k]) return fail(c, LASGD_ERR_STATE, "replica %d is not bound", k);
    lasgd_status st = which == LASGD_STATE_X ? place_models(c) : LASGD_OK;
    if (st != LASGD_OK) return st;
    if ((st = lasgd_sync(c)) != LASGD_OK) return st;
    if (which == LASGD_STATE_X && ((c->at_s >> k) & 1ull)) which = LASGD_STATE_S;
    const float *base = which == LASGD_STATE_V ? c->v : which == LASGD_STATE_S ? c->s : which == LASGD_STATE_Z ? c->z : c->x32;
    const int32_t t0 = tensor < 0 ? 0 : tensor, t1 = tensor < 0 ? c->n_tensors : tensor + 1;
    float *out = dst;
    for (int32_t t = t0; t < t1; ++t) {
        const void *src = user_x ? c->h_xptr[(size_t)k * c->n_tensors + t]
                                 : (const void *)(base + (which == LASGD_STATE_Z ? 0 : (uint64_t)k * c->npad) + c->aoff[(size_t)t]);
        LASGD_HIP(c, hipMemcpy(out, src, (size_t)c->numel[(size_t)t] * sizeof(float), hipMemcpyDeviceToHost));
        out += c->numel[(size_t)t];
    }
    return LASGD_OK;
}

static lasgd_status set_tuning_impl(lasgd_ctx *c, const lasgd_tuning *t)
{
    if (!c) return LASGD_ERR_INVALID;
    if (!t) return fail(c, LASGD_ERR_INVALID, "NULL argument");
    lasgd_tuning n = c->tune;
    if (t->vec) {
        if (t->vec != 1 && t->vec != 2 && t->vec != 4) return fail(c, LASGD_ERR_INVALID, "vec must be 1, 2 or 4");
        n.vec = t->vec;
    }
    if (t->kper_step) {
        if (t->kper_step < 1 || t->kper_step > c->K) return fail(c, LASGD_ERR_INVALID, "kper_step outside 1..K");
        n.kper_step = t->kper_step;
    }
    if (t->kper_merge) {
        if (t->kper_merge < 1 || t->kper_merge > c->K) return fail(c, LASGD_ERR_INVALID, "kper_merge outside 1..K");
        n.kper_merge = t->kper_merge;
    }
    if (t->max_blocks) n.max_blocks = t->max_blocks;
    if (t->avg_split) {
        if (t->avg_split != 1 && t->avg_split != 2 && t->avg_split != 4) return fail(c, LASGD_ERR_INVALID, "avg_split must be 1, 2 or 4");
        n.avg_split = t->avg_split;
    }
    if (t->avg_max_blocks) n.avg_max_blocks = t->avg_max_blocks;
    if (t->nontemporal) {
        if (t->nontemporal > 4) return fail(c, LASGD_ERR_INVALID, "nontemporal must be 1, 2, 3 or 4 (or negative for the default)");
        n.nontemporal = t->nontemporal < 0 ? -1 : t->nontemporal;
    }
    if (t->waves_per_block) {
        if (t->waves_per_block != 1 && t->waves_per_block != 2 && t->waves_per_block != 4)
            return fail(c, LASGD_ERR_INVALID, "waves_per_block must be 1, 2 or 4");
        n.waves_per_block = t->waves_per_block;
    }
    if (t->chunk_step) n.chunk_step = t->chunk_step < 0 ? -1 : t->chunk_step;
    if (t->chunk_merge) n.chunk_merge = t->chunk_merge < 0 ? -1 : t->chunk_merge;
    if (t->race_probe) n.race_probe = t->race_probe > 0 ? 1 : -1;
    if (t->group_r) {
        if (t->group_r > 0 && t->group_r != 1 && t->group_r != 2 && t->group_r != 4)
            return fail(c, LASGD_ERR_INVALID, "group_r must be 1, 2 or 4 (or negative for the default)");
        n.group_r = t->group_r < 0 ? -1 : t->group_r;
    }
    lasgd_status st = lasgd_sync(c);
    if (st != LASGD_OK) return st;
    if (n.vec != c->tune.vec) {
        st = upload_tables(c, n.vec);
        if (st != LASGD_OK) return st;
    }
    c->tune = n;
    return LASGD_OK;
}

lasgd_status lasgd_set_tuning(lasgd_ctx *c, const lasgd_tuning *t)
{
    try {
        return set_tuning_impl(c, t);
    } catch (...) {
        return LASGD_ERR_ALLOC;
    }
}

lasgd_status lasgd_get_tuning(const lasgd_ctx *c, lasgd_tuning *out)
{
    if (!c || !out) return LASGD_ERR_INVALID;
    *out = c->tune;
    return LASGD_OK;
}

const char *lasgd_last_error(const lasgd_ctx *c)
{
    return c ? c->err.c_str() : g_create_error.c_str();
}

void lasgd_destroy(lasgd_ctx *c)
{
    if (!c) return;
    (void)hipStreamSynchronize(c->main);
    if (c->side != c->main) (void)hipStreamSynchronize(c->side);
    (void)wait_for_clears(c);
    release(c);
}

} // extern "C"

// ---- the allocation-free entry point ---------------------------------------
// The limit is part of the interface, which promises to refuse longer vectors; the kernel would take them (64-bit offsets,
// one workgroup per 256 elements).
constexpr int64_t kStaticMaxN = LASGD_STATIC_MAX_N;

namespace {

template <int NT> hipError_t launch_flat_update(FlatArgs &a, uint32_t blocks, hipStream_t st)
{
    size_t lds = (size_t)a.K * 256u * sizeof(float);
    uint32_t R;                 // replicas a wave
    if (NT != 0) {
        // Streaming.  The memory system is fastest with about 24 replicas' rows on a CU (24 KiB of s, then 24 KiB of x), as
        // whole workgroups: the LDS a workgroup asks for leaves room for 24 / K of them, two at least up to K = 19.  us over three
        // states in turn, one replica a wave, everything at once and no bound / staged and bounded with one, two, four a wave:
        // K = 2 131 / 125, 125; K = 3 193 / 188, 189; K = 4 267 / 252, 249, 250; K = 6 397 / 386, 382, 385; K = 8 557 / 536, 529, 529.
        // Two or four a wave from K = 12 on is a matter of 0.5 % either way (150 MB an array, K = 12: 107.8 / 110.2; 1100 MB 707.6 / 705.7).
        // One group more or fewer on a CU costs 1-2 or 3-20 %.  Other work between the calls changes none of this
        // (K = 8 555 / 533, 526).  Vectors of 150 to 1100 MB together, before / staged with this rule: K = 9 -2 to -3 %,
        // K = 10 -1 to -3.5, K = 12 +1 to -4, K = 16 0 to -2, K = 20 -1 to -3.6, K = 24 to 32 -0.3 to -0.8.
        // K = 20 to 32, two groups a CU / one: 2,000,003 elements K = 18 100.8 / 101.3, 19 106.8 / 106.1, 20 113.6 / 112.0, 22 127.5 / 124.2,
        // 24 139.1 / 135.3; 12,000,000 K = 18 609.7 / 589.0, 20 689.8 / 655.2, 22 773.2 / 747.1, 24 839.0 / 819.5; 450 MB K = 25 336 / 323,
        // K = 27 356 / 342, K = 29 337 / 330, K = 32 351 / 345; but K = 17 94.6 / 96.9 and, of 12,000,000 elements, 567.9 / 558.6.
        // So from 20 on one group is better at every length; at 17 and 18 it is for long vectors only, and they keep two.
        // Four replicas a wave, K > 32, have enough in flight to wait for s alone at no gain, and are bounded to two groups: at once
        // and no bound / staged / at once and bounded, K = 33, n = 3.5e6 329.0 / 327.3 / 322.8, K = 40, 4e6 423.6 / 426.1 / 422.4,
        // K = 48, 3e6 451.7 / 456.4 / 451.4, K = 64, 3e6 560.3 / 563.4 / 560.3.
        R = a.K <= kFlatOneMaxK ? 1u : a.K <= 2u * kGroupWaves ? 2u : 4u;
        size_t pace = kOneGroupLds;
        if (a.K < 20u || R == 4u) {
            pace = kCuLds / (a.K <= 12u ? 24u / a.K : 2u) / kLdsGranule * kLdsGranule;
            if (pace > kMaxLds) pace = kMaxLds;
        }
        if (pace > lds) lds = pace;
    } else {
        // In the memory-side cache.  One wave per replica while a workgroup can hold that many (16), then two or four replicas
        // a wave.  Two win for K = 4..8 where the waves are more than the chip holds
        // at once (8192): K = 8, n = 2^19 13.8 us against 16.1, n = 600,000 13.5 against 13.9, K = 4, n = 2^20 12.4 against 14.0;
        // below that the extra wave is free and shortens the call (K = 4, n = 300,000 4.5 against 4.9), and from K = 12 on one
        // a wave is ahead again (n = 1,000,003 31.6 against 34.2).
        R = a.K <= kGroupWaves ? 1u : a.K <= 2u * kGroupWaves ? 2u : 4u;
        if (a.K >= 4u && a.K <= 8u && (uint64_t)blocks * a.K > kWavesOnChip) R = 2u;
    }
    a.W = (a.K + R - 1u) / R;
    const dim3 bs(64u * a.W);
    if (R == 1u) hipLaunchKernelGGL((flat_update_kernel<1, NT>), dim3(blocks), bs, lds, st, a);
    else if (R == 2u) hipLaunchKernelGGL((flat_update_kernel<2, NT>), dim3(blocks), bs, lds, st, a);
    else hipLaunchKernelGGL((flat_update_kernel<4, NT>), dim3(blocks), bs, lds, st, a);
    return hipGetLastError();
}

} // namespace

extern "C" lasgd_status lasgd_global_update_static(int32_t K, int64_t n, float *const *x, float *const *sent,
                                                   int32_t resnapshot, void *stream)
{
    try {
        if (!x || !sent) return fail(nullptr, LASGD_ERR_INVALID, "NULL pointer array");
        if (K < 1 || K > kMaxK) return fail(nullptr, LASGD_ERR_INVALID, "K = %d outside 1..%d", K, kMaxK);
        if (n < 1) return fail(nullptr, LASGD_ERR_INVALID, "n = %lld: nothing to update", (long long)n);
        if (n > kStaticMaxN)
            return fail(nullptr, LASGD_ERR_UNSUPPORTED,
                        "n = %lld exceeds LASGD_STATIC_MAX_N = %lld elements; split the vector or use a context",
                        (long long)n, (long long)kStaticMaxN);
        FlatArgs a{};
        for (int32_t k = 0; k < K; ++k) {
            if (!x[k] || !sent[k]) return fail(nullptr, LASGD_ERR_INVALID, "NULL buffer for replica %d", k);
            if (((uintptr_t)x[k] | (uintptr_t)sent[k]) & 15u)
                return fail(nullptr, LASGD_ERR_INVALID, "buffer of replica %d is not 16-byte aligned", k);
            a.x[k] = x[k];
            a.s[k] = sent[k];
        }
        // the 2K buffers must not overlap: every one of them is written by one replica's waves only
        const uintptr_t bytes = (uintptr_t)n * sizeof(float);
        for (int32_t i = 0; i < 2 * K; ++i)
            for (int32_t j = 0; j < i; ++j) {
                const uintptr_t p = (uintptr_t)(i < K ? x[i] : sent[i - K]), q = (uintptr_t)(j < K ? x[j] : sent[j - K]);
                if (p < q + bytes && q < p + bytes)
                    return fail(nullptr, LASGD_ERR_INVALID, "%s of replica %d overlaps %s of replica %d",
                                i < K ? "x" : "sent", i < K ? i : i - K, j < K ? "x" : "sent", j < K ? j : j - K);
            }
        a.n = (uint64_t)n;
        a.K = (uint32_t)K;
        a.use_mul = is_pow2((uint32_t)K) ? 1 : 0;
        a.inv_k = 1.0 / (double)K;
        a.k_as_double = (double)K;
        a.resnap = resnapshot ? 1 : 0;
        // the streaming hint from the size on at which the vectors no longer fit the 256 MB memory-side cache
        const bool hint = (uint64_t)K * (uint64_t)n * sizeof(float) >= (128ull << 20);
        const uint32_t blocks = (uint32_t)(((uint64_t)n + 255u) / 256u);
        const hipError_t e = hint ? launch_flat_update<3>(a, blocks, (hipStream_t)stream) : launch_flat_update<0>(a, blocks, (hipStream_t)stream);
        if (e != hipSuccess) return fail(nullptr, LASGD_ERR_HIP, "global-update launch failed: %s", hipGetErrorString(e));
        return LASGD_OK;
    } catch (...) {
        return LASGD_ERR_ALLOC;
    }
}
