// Device code of the LASGD update library (gfx950 / CDNA4, wave64).
//
// Everything here is bandwidth-bound streaming: a handful of fp32 FMAs per
// 20-28 bytes moved, so there is no matrix-core work.  What matters is that
// every lane moves 128 bits per access, that a wave covers a contiguous
// kilobyte per instruction, that many independent loads are in flight before
// the first use, and that the mean z (shared by all K replicas) is fetched
// once per tile and kept in registers while the wave walks the replicas.
//
// Arithmetic is pinned: contraction is off for this file, so only the
// __builtin_fmaf calls below fuse.  Local update: Algorithm 1 steps 3 and 7
// with the optimizer of Sec. 5.2; global update: step 9a-b; mean: Sec. 3 Eq. 8.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lasgd {

// One tile = up to 256*VEC consecutive elements of ONE tensor, handled by one
// wave: lane l owns elements [4l, 4l+4) of each 256-element row of the tile.
struct Tile {
    uint64_t toff;     // first element, relative to the tensor's start
    uint64_t aoff;     // first element, relative to a replica's start in the library arenas
    uint32_t count;    // elements in this tile (<= 256*VEC; smaller only at a tensor's end)
    float wd;          // the tensor's weight decay
};

// What the kernels look up: one 32-byte record per (replica, tensor).  A tile's tensor is named by its block of 64 tiles; the top bit
// says that more tensors start inside the block, and then the tile is compared with
// the following tensors' first tiles, sixteen at a time.
//
// The tables are read through the scalar cache.  They are per block and per tensor
// and not per tile (161 tensors, 10^5 tiles: 6 KB of blocks, 5.2 KB of records of
// one replica), so a few hundred waves in a row find them there, and
// a scalar hit does not queue behind the streaming loads of other waves as a vector
// load does.  A record per tile, read through the vector path, made every wave wait twice
// for the loaded memory system before its first data load: at 24 waves a CU that cost
// 13 % of a local step, and kernels in the memory-side cache 4 % (flat list of 2^20
// elements, K = 4, update cycle 42.0 -> 40.5 us).  With the short wait fewer waves do,
// and then the kernels can be paced (pace_lds in the host code).
constexpr uint32_t kBlockShift = 6;
constexpr uint32_t kMoreInBlock = 0x80000000u;
constexpr uint32_t kProbe = 16;
struct Record {        // one per (replica, tensor): everything a wave needs, in one load
    uint64_t x, g;     // device addresses of the caller's parameters and gradient
    uint32_t arow;     // arena offset in units of 256 elements
    uint32_t numel;
    float wd;
    uint32_t pad_;
};
static_assert(sizeof(Record) == 32, "one 32-byte scalar load");

enum Op : int { OP_STEP = 0, OP_MERGE = 1, OP_STEP_MERGE = 2, OP_SNAPSHOT = 3, OP_INIT = 4, OP_STEP_MEAN = 5 };

enum : uint32_t { ALSO_X = 1, LOOK = 2, SETTLES = 4 };     // LOOK, and SETTLES with it: early in a recorded graph, see settle_word

// n / d for n < 2^31 by a multiplication (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994): with l = ceil(log2 d) and m = floor(2^(31+l) / d) + 1 (2^31 for a power of two),
// floor(n * m / 2^(31+l)) is exact, and m fits 32 bits.
struct FastDiv {
    uint32_t m, shift;
};
__device__ __forceinline__ uint32_t fast_div(uint32_t n, FastDiv d)
{
    return (uint32_t)(((uint64_t)n * d.m) >> d.shift);
}

struct ApplyArgs {
    const uint32_t *blocks; // [ceil(ntiles / 64)] tensor of each block's first tile, kMoreInBlock if others follow in it
    const uint32_t *tile0;  // [n_tensors + 16] the tensors' first tiles, then 0xffffffff, which no tile reaches
    const Record *records;  // [K * n_tensors]
    float *x32;             // bf16 storage only: fp32 master, [K][npad], and behind it the words of settle_word
    float *v;               // momentum,     [K][npad]
    float *s;               // sent models,  [K][npad]
    float *z;               // mean,         [npad] (written only by the fused step+update+mean kernel); OP_STEP_MEAN and
                            // mean_grad_kernel: the mean gradient
    uint64_t npad;          // elements per replica in the arenas
    uint32_t ntiles, K, n_tensors;
    uint32_t kcount;        // replicas that take part (K, or fewer in the extended calls)
    uint32_t kper;          // replicas a wave handles back to back
    uint32_t kgroups;       // ceil(kcount / kper)
    uint32_t nitems;        // full_items + tail_stride * kgroups if there is a tail: padding items among them (the replica-group
                            // kernels: ntiles rounded down to a multiple of eight)
    // 0, 0: items in order; nitems (a multiple of eight) - 8, ~7: from the last eight to the first.  They stand here because a wave
    // needs them as early as its neighbours: at the end of the arguments, another cache line, they cost a short call 0.3 us.
    uint32_t back, back_mask;
    float neg_lr, mu;
    int32_t nesterov, resnap;
    // bf16 storage: bit k of at_s says that replica k's model is s[k], which it has just re-sent, and that its master copy is out of
    // date.  A global update that re-sends leaves it that way unless ALSO_X, and the next step writes the master again.
    uint32_t place;         // ALSO_X, LOOK, SETTLES
    uint64_t at_s;          // LOOK: until the words behind the master copies say otherwise
    uint32_t tile_elems;    // 256 * VEC
    uint32_t wpb, nwaves;   // waves per workgroup, and in the grid (the replica-group kernels: workgroups in the grid)
    uint32_t chunk;         // item order, see apply_kernel
    uint32_t full_items;    // (ntiles / chunk) * chunk * kgroups
    uint32_t tail_first;    // first tile of the last, shorter chunk
    uint32_t tail_chunk;    // its length (>= 1 even when unused)
    uint32_t tail_stride;   // items per replica group in the last chunk: tail_chunk rounded up so that every
                            // group's pass starts on the same XCD; the items in between do nothing
    FastDiv by_per, by_chunk, by_stride;   // division by chunk * kgroups, chunk, tail_stride
    // the replica-group kernels finish a mean over all K replicas themselves
    int32_t use_mul;        // K is a power of two: multiply by the exact reciprocal
    double inv_k, k_as_double;
};

// What the extended entry points add: replicas that sit a call out, a step size
// per replica (eta is indexed by each node's own clock, Algorithm 1) and the
// elastic coefficient alpha of Sec. 3, Eq. 6.
struct ExtArgs {
    uint64_t step_mask;     // bit k: replica k takes the local update (or is snapshotted / initialised)
    uint64_t merge_mask;    // bit k: replica k takes the global update
    float alpha;            // 1 = step 9a of Algorithm 1 exactly
    float neg_lr_k[64];     // -eta per replica
};

// ---- 128-bit / 64-bit accesses, optionally with the streaming hint --------
// NT: 1 the hint on loads, 2 on stores; 4 belongs to the kernels that ask for a word of their model before their loads.
// Every pointer the kernels dereference is device (global) memory.  Pointers
// that come out of the tables are generic as far as the compiler can tell and
// would be accessed with FLAT instructions; casting to the global address
// space makes every access a GLOBAL load or store.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
#define LASGD_GLOBAL_AS __attribute__((address_space(1)))
template <class T> __device__ __forceinline__ const LASGD_GLOBAL_AS T *as_global(const void *p)
{
    return reinterpret_cast<const LASGD_GLOBAL_AS T *>(reinterpret_cast<uintptr_t>(p));
}
template <class T> __device__ __forceinline__ LASGD_GLOBAL_AS T *as_global(void *p)
{
    return reinterpret_cast<LASGD_GLOBAL_AS T *>(reinterpret_cast<uintptr_t>(p));
}

#define LASGD_CONST_AS __attribute__((address_space(4)))
template <class T> __device__ __forceinline__ const LASGD_CONST_AS T *as_const(const T *p)
{
    return reinterpret_cast<const LASGD_CONST_AS T *>(reinterpret_cast<uintptr_t>(p));
}

typedef uint32_t u32x16_t __attribute__((ext_vector_type(16), aligned(4)));

// The tensor that tile `tile` (wave-uniform) belongs to.
__device__ __forceinline__ uint32_t tensor_of(const ApplyArgs &a, uint32_t tile)
{
    uint32_t t = 0;
    if (a.n_tensors > 1u) {
        // one probe holds the whole list when no more than sixteen tensors follow the first
        t = a.n_tensors > kProbe + 1u ? as_const(a.blocks)[tile >> kBlockShift] : kMoreInBlock;
        if (t & kMoreInBlock) {
            t &= ~kMoreInBlock;
            uint32_t below;              // how many of the next sixteen tensors start at or before the tile
            do {
                const u32x16_t n = *reinterpret_cast<const LASGD_CONST_AS u32x16_t *>(as_const(a.tile0) + t + 1u);
                below = 0;
#define LASGD_BELOW(n) "s_cmp_le_u32 %" #n ", %1\n\ts_addc_u32 %0, %0, 0\n\t"
                asm(LASGD_BELOW(2) LASGD_BELOW(3) LASGD_BELOW(4) LASGD_BELOW(5) LASGD_BELOW(6) LASGD_BELOW(7)
                    LASGD_BELOW(8) LASGD_BELOW(9) LASGD_BELOW(10) LASGD_BELOW(11) LASGD_BELOW(12) LASGD_BELOW(13)
                    LASGD_BELOW(14) LASGD_BELOW(15) LASGD_BELOW(16) LASGD_BELOW(17)
                    : "+&s"(below)
                    : "s"(tile), "s"(n[0]), "s"(n[1]), "s"(n[2]), "s"(n[3]), "s"(n[4]), "s"(n[5]), "s"(n[6]), "s"(n[7]),
                      "s"(n[8]), "s"(n[9]), "s"(n[10]), "s"(n[11]), "s"(n[12]), "s"(n[13]), "s"(n[14]), "s"(n[15])
                    : "scc");
#undef LASGD_BELOW
                t += below;
            } while (below == kProbe);
        }
    }
    return t;
}
__device__ __forceinline__ Record load_record(const ApplyArgs &a, uint32_t k, uint32_t tensor)
{
    const LASGD_CONST_AS Record *r = as_const(a.records) + ((size_t)k * a.n_tensors + tensor);
    return Record{r->x, r->g, r->arow, r->numel, r->wd, 0u};
}
// Where the tile lies in its tensor and in the arenas.  Tiles of 256 elements are the arenas' rows.
__device__ __forceinline__ Tile locate(const ApplyArgs &a, const Record &rec, uint32_t tile, uint32_t tensor, uint32_t tile_elems)
{
    const uint32_t first = tile_elems == 256u ? rec.arow : as_const(a.tile0)[tensor];
    const uint32_t off = (tile - first) * tile_elems;
    const uint32_t left = rec.numel - off;
    Tile r;
    r.toff = off;
    r.aoff = (uint64_t)rec.arow * 256u + off;
    r.count = left < tile_elems ? left : tile_elems;
    r.wd = rec.wd;
    return r;
}

// The arguments that a wave needs before its first load, asked for together: left to the compiler, they come where each is first
// used, in three rounds of scalar loads that wait for one another.  us, three rounds / one, three states in turn: a cycle of 2^20 elements
// K = 4 39.2 / 38.6, 250,007 K = 8 22.1 / 21.6, 100,003 K = 16 20.6 / 20.2, 60 tensors m = 4 32.1 / 31.3.
__device__ __forceinline__ void load_together(const ApplyArgs &a)
{
    asm volatile("" ::"s"(a.blocks), "s"(a.tile0), "s"(a.records), "s"(a.v), "s"(a.npad), "s"(a.n_tensors), "s"(a.kcount), "s"(a.kper),
                 "s"(a.nitems), "s"(a.back), "s"(a.back_mask), "s"(a.nwaves), "s"(a.nesterov), "s"(a.full_items), "s"(a.tail_first),
                 "s"(a.tail_chunk), "s"(a.tail_stride), "s"(a.by_stride.m), "s"(a.by_stride.shift));
}

// bf16 storage, and a graph recorded while models were in s only.  It is replayed at any time, so nothing in it may depend on where the
// last call left a model: its first kernel finds the models of at_s in s on the first replay and in the master copies, which it
// writes, on all later ones, unless a call has run in between (settle_kernel).  A word in memory says which: kSettled, once every wave of
// the one that comes first has counted itself there.  No wave can find it so before its own share is done, and the next kernel
// begins when all are.  Waves count in parts that share no cache line, since
// a million of them on one word would take longer than the kernel; later replays only read the word, beside the replica's record, so that
// it costs no wait of its own.  us a replay with a kernel in front that does nothing from the second replay on / this / recorded with the models
// in the master copies, three states in turn: fused update K = 8, 8 MiB an array 21.5 / 17.1 / 17.0, 92 MiB 145.3 / 140.9 / 141.0; K = 4, 16 MiB
// 29.9 / 25.5 / 25.3; a cycle, m = 1, K = 8, 8 MiB 20.9 / 19.3 / 19.3, 92 MiB 129.2 / 127.9 / 127.7.  The words lie where x32 tells: one pointer more among
// the arguments cost every call on bf16 models 0.1 us.
constexpr uint32_t kSettled = 0x80000000u, kSettleParts = 256u, kSettleStride = 16u;       // stride: words
constexpr uint32_t kSettleWords = kSettleStride * (1u + kSettleParts);

__device__ __forceinline__ uint32_t *settle_words(const ApplyArgs &a) { return reinterpret_cast<uint32_t *>(a.x32 + (uint64_t)a.K * a.npad); }
__device__ __forceinline__ uint32_t settle_word(const ApplyArgs &a)
{
    const uint32_t *p = settle_words(a);
    asm volatile("" : "+s"(p));               // here, where other loads are under way, and not in front of the loop
    return *as_const(p);
}
__device__ __forceinline__ void count_settled(uint32_t *settle, uint32_t wave, uint32_t waves, uint32_t lane)
{
    if (lane != 0u) return;
    const uint32_t parts = waves < kSettleParts ? waves : kSettleParts, part = wave % kSettleParts;
    const uint32_t others = (waves - 1u - part) / kSettleParts;                            // in this part
    if (atomicAdd(settle + kSettleStride * (1u + part), 1u) != others) return;
    atomicAdd(settle, part == 0u ? kSettled - (parts - 1u) : 1u);                          // the parts' sum is kSettled
}

// Which item a workgroup takes when the launch runs backwards.  Eight items at a time, so that each stays on its XCD.
__device__ __forceinline__ uint32_t in_order(uint32_t item, const ApplyArgs &a)
{
    return item + a.back - 2u * (item & a.back_mask);
}

template <int NT> __device__ __forceinline__ float4 ld4(const float *p)
{
    f32x4_t r;
    if constexpr (NT & 1) r = __builtin_nontemporal_load(as_global<f32x4_t>(p));
    else r = *as_global<f32x4_t>(p);
    return make_float4(r.x, r.y, r.z, r.w);
}
template <int NT> __device__ __forceinline__ void st4(float *p, float4 a)
{
    f32x4_t r = {a.x, a.y, a.z, a.w};
    if constexpr (NT & 2) __builtin_nontemporal_store(r, as_global<f32x4_t>(p));
    else *as_global<f32x4_t>(p) = r;
}
template <int NT> __device__ __forceinline__ uint2 ld2(const uint16_t *p)
{
    u32x2_t r;
    if constexpr (NT & 1) r = __builtin_nontemporal_load(as_global<u32x2_t>(p));
    else r = *as_global<u32x2_t>(p);
    return make_uint2(r.x, r.y);
}
template <int NT> __device__ __forceinline__ void st2(uint16_t *p, uint2 a)
{
    u32x2_t r = {a.x, a.y};
    if constexpr (NT & 2) __builtin_nontemporal_store(r, as_global<u32x2_t>(p));
    else *as_global<u32x2_t>(p) = r;
}

// Every load written before it has arrived, none written after it is issued yet.
__device__ __forceinline__ void wait_for_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// How long the word at p takes to come says how busy the memory is.
__device__ __forceinline__ void wait_for_word(const float *p)
{
    const uint32_t word = *as_global<uint32_t>(p);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(word) : "memory");
}

// ---- bf16 <-> fp32 ----------------------------------------------------------
__device__ __forceinline__ float bf16_widen(uint32_t h) { return __uint_as_float(h << 16); }

// Round to nearest, ties to even, by adding 0x7fff plus the kept LSB and
// truncating; NaN is kept a quiet NaN.
__device__ __forceinline__ uint32_t bf16_round(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    uint32_t nan = (u >> 16) | 0x40u;
    return ((u & 0x7fffffffu) > 0x7f800000u) ? nan : r;
}
__device__ __forceinline__ float4 widen4(uint2 p)
{
    return make_float4(bf16_widen(p.x & 0xffffu), bf16_widen(p.x >> 16),
                       bf16_widen(p.y & 0xffffu), bf16_widen(p.y >> 16));
}
__device__ __forceinline__ uint2 round4(float4 a)
{
    return make_uint2(bf16_round(a.x) | (bf16_round(a.y) << 16),
                      bf16_round(a.z) | (bf16_round(a.w) << 16));
}

// ---- the arithmetic, one element -------------------------------------------
// Local update (Algorithm 1 step 7; Sec. 5.2): four fused multiply-adds.
__device__ __forceinline__ void step_elem(float &x, float &v, float g, float wd, float mu,
                                          float neg_lr, int nesterov)
{
    float g1 = __builtin_fmaf(wd, x, g);
    float vn = __builtin_fmaf(mu, v, g1);
    float d = nesterov ? __builtin_fmaf(mu, vn, g1) : vn;
    x = __builtin_fmaf(neg_lr, d, x);
    v = vn;
}
// Global update (step 9a): z + (x - s), parenthesised as printed.
__device__ __forceinline__ float merge_elem(float x, float s, float z)
{
    float progress = x - s;
    return z + progress;
}

// Elastic form (Eq. 6 in the asynchronous setting): the pull alpha*(z - s) is
// measured at the sent model and applied to the current one.  alpha == 1 keeps
// the printed form of step 9a, so both entry-point families agree bit for bit there.
__device__ __forceinline__ float merge_elem_elastic(float x, float s, float z, float alpha)
{
    float pulled = __builtin_fmaf(alpha, z - s, x);
    return alpha == 1.0f ? merge_elem(x, s, z) : pulled;
}

#define LASGD_FOR4(body)                                                                       \
    {                                                                                          \
        { constexpr int c = 0; body }                                                          \
        { constexpr int c = 1; body }                                                          \
        { constexpr int c = 2; body }                                                          \
        { constexpr int c = 3; body }                                                          \
    }
__device__ __forceinline__ float &comp(float4 &a, int c)
{
    return c == 0 ? a.x : c == 1 ? a.y : c == 2 ? a.z : a.w;
}
__device__ __forceinline__ float compv(const float4 &a, int c)
{
    return c == 0 ? a.x : c == 1 ? a.y : c == 2 ? a.z : a.w;
}

// How many of the four elements from e0 on a tile of `count` elements has.
template <bool FULL> __device__ __forceinline__ uint32_t lane_elems(uint32_t e0, uint32_t count)
{
    return FULL ? 4u : e0 >= count ? 0u : count - e0 < 4u ? count - e0 : 4u;
}

// Apply one operation to VEC rows of one replica's tile.  `count` bounds the ragged
// path.  x/g point at the tile's first element in the caller's buffers
// (storage dtype), xm/v/s at the tile's first element in the arenas.  bf16 storage: the model is read from xr, which is
// xm or, where it has just been re-sent (AT_S), s.
//
// A ragged tile (the last of a tensor) takes the same 128-bit accesses in the lanes
// that have all four elements, and only the one lane that a tensor's odd end leaves
// with one to three goes element by element: all its loads before its first store,
// as everywhere, so that the wave waits once for memory.
// ALONE: the operation is the whole kernel's, not one of several in a masked call.
//
// bf16 storage, where the fp32 model and s are both the library's: a global update that re-sends would write the same values
// twice, and the next pass would read them from either place.  So it writes s alone, and whoever needs the model next reads it
// there: 4 bytes a replica-parameter fewer per update, 8 where an update follows directly, which then reads s once.  us before /
// after, over three states in turn: ResNet-18 list K = 12, two fused updates in a row 1405 / 990; ResNet-50 K = 32, an update
// every eight steps 21617 / 21212.
template <int VEC, int OP, bool BF16, int NT, bool FULL, bool EXT, bool ALONE, bool AT_S>
__device__ __forceinline__ void apply_tile(const ApplyArgs &a, void *xu, const void *gu, const float *xr, float *xm,
                                           float *v, float *s, const float4 (&zt)[VEC], float wd,
                                           uint32_t count, uint32_t lane, float neg_lr, float alpha)
{
    constexpr bool NEED_G = (OP == OP_STEP || OP == OP_STEP_MERGE);
    constexpr bool STEPS = NEED_G || OP == OP_STEP_MEAN;       // with a gradient of its own, or the mean of all
    constexpr bool NEED_V = STEPS;
    constexpr bool NEED_X = (OP != OP_INIT);
    constexpr bool NEED_S = (OP == OP_MERGE || OP == OP_STEP_MERGE);
    constexpr bool WRITE_X = (OP != OP_SNAPSHOT);
    constexpr bool WRITE_V = NEED_V || OP == OP_INIT;
    const float *xf = BF16 ? xr : static_cast<const float *>(xu);          // where the fp32 model lives
    float *xw = BF16 ? xm : static_cast<float *>(xu);                      // and where it goes
    uint16_t *x16 = static_cast<uint16_t *>(xu);
    const float *gf = static_cast<const float *>(gu);
    const uint16_t *g16 = static_cast<const uint16_t *>(gu);
    constexpr bool LOAD_S = NEED_S && !AT_S;
    const bool write_s = (OP == OP_SNAPSHOT) || (NEED_S && a.resnap);
    const bool write_x = !BF16 || !NEED_S || !a.resnap || (a.place & ALSO_X);

    if constexpr (OP == OP_SNAPSHOT && !FULL) {          // a copy
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const uint32_t e = j * 256u + lane * 4u, n = lane_elems<FULL>(e, count);
            if (n == 4u) st4<NT>(s + e, ld4<NT>(xf + e));
            else
                for (uint32_t i = 0; i < n; ++i) *as_global<float>(s + e + i) = *as_global<float>(xf + e + i);
        }
        return;
    }
    float4 x[VEC], vv[VEC], g[VEC], ss[VEC];
    if constexpr (!FULL) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) x[j] = vv[j] = g[j] = ss[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // An fp32 local step that streams from HBM asks for one word of its model first and issues its loads when that has
    // come: the busier the memory, the later.  us, with 18 waves a CU (pace_lds) / with 21 and this word: ResNet-18 list
    // K = 8 283 / 273, ResNet-50 K = 8 621 / 594, K = 24 1901 / 1863, K = 32 2495 / 2493, MobileNetV2 K = 16 172 / 165.
    // bf16 gains below 3e8 replica-parameters (ResNet-50 K = 8 622 / 607) and loses beyond (ResNet-18 K = 32 1140 / 1156,
    // ResNet-50 K = 32 2478 / 2492), so it goes without.  Step + update, masked or not, asks where NT says so (word_first).
    if constexpr (FULL && ((ALONE && OP == OP_STEP && !BF16 && (NT & 3) != 0) || (NT & 4) != 0)) wait_for_word(xf);
    // all loads first: up to 4*VEC independent 128-bit loads in flight per lane
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const uint32_t e = j * 256u + lane * 4u;
        if (FULL || lane_elems<FULL>(e, count) == 4u) {
            if constexpr (NEED_G) g[j] = BF16 ? widen4(ld2<NT>(g16 + e)) : ld4<NT>(gf + e);
            if constexpr (NEED_X) x[j] = ld4<NT>(xf + e);
            if constexpr (OP == OP_INIT) x[j] = widen4(ld2<NT>(x16 + e));
            if constexpr (NEED_V) vv[j] = ld4<NT>(v + e);
            if constexpr (LOAD_S) ss[j] = ld4<NT>(s + e);
        }
    }
    if constexpr (!FULL) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const uint32_t e = j * 256u + lane * 4u, n = lane_elems<FULL>(e, count);
            if (n - 1u < 3u) {
                LASGD_FOR4(if (c < 3 && (uint32_t)c < n) {
                    if constexpr (NEED_G) comp(g[j], c) = BF16 ? bf16_widen(*as_global<uint16_t>(g16 + e + c)) : *as_global<float>(gf + e + c);
                    if constexpr (NEED_X) comp(x[j], c) = *as_global<float>(xf + e + c);
                    if constexpr (OP == OP_INIT) comp(x[j], c) = bf16_widen(*as_global<uint16_t>(x16 + e + c));
                    if constexpr (NEED_V) comp(vv[j], c) = *as_global<float>(v + e + c);
                    if constexpr (LOAD_S) comp(ss[j], c) = *as_global<float>(s + e + c);
                })
            }
        }
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const uint32_t e = j * 256u + lane * 4u, n = lane_elems<FULL>(e, count);
        if constexpr (AT_S) ss[j] = x[j];
        if constexpr (OP == OP_STEP_MEAN) g[j] = zt[j];
        if constexpr (STEPS)
            LASGD_FOR4(step_elem(comp(x[j], c), comp(vv[j], c), compv(g[j], c), wd, a.mu,
                                 neg_lr, a.nesterov);)
        if constexpr (NEED_S) {
            if constexpr (EXT)
                LASGD_FOR4(comp(x[j], c) = merge_elem_elastic(compv(x[j], c), compv(ss[j], c), compv(zt[j], c), alpha);)
            else
                LASGD_FOR4(comp(x[j], c) = merge_elem(compv(x[j], c), compv(ss[j], c), compv(zt[j], c));)
        }
        if constexpr (OP == OP_INIT) vv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (FULL || n == 4u) {
            if constexpr (WRITE_V) st4<NT>(v + e, vv[j]);
            if constexpr (WRITE_X) {
                if (write_x) st4<NT>(xw + e, x[j]);
                if constexpr (BF16 && OP != OP_INIT) st2<NT>(x16 + e, round4(x[j]));
            }
            if (write_s) st4<NT>(s + e, x[j]);
        }
        if constexpr (!FULL) {
            if (n - 1u < 3u) {
                LASGD_FOR4(if (c < 3 && (uint32_t)c < n) {
                    if constexpr (WRITE_V) *as_global<float>(v + e + c) = compv(vv[j], c);
                    if constexpr (WRITE_X) {
                        if (write_x) *as_global<float>(xw + e + c) = compv(x[j], c);
                        if constexpr (BF16 && OP != OP_INIT) *as_global<uint16_t>(x16 + e + c) = (uint16_t)bf16_round(compv(x[j], c));
                    }
                    if (write_s) *as_global<float>(s + e + c) = compv(x[j], c);
                })
            }
        }
    }
}

// Position of the n-th set bit (n = 0: the lowest) of a word that has more than n: halve the word six times.
__device__ __forceinline__ uint32_t nth_bit(uint64_t word, uint32_t n)
{
    uint32_t pos = 0;
#pragma unroll
    for (uint32_t width = 32u; width; width >>= 1) {
        const uint32_t below = (uint32_t)__popcll(word & ((1ull << width) - 1ull));
        const bool above = n >= below;
        n -= above ? below : 0u;
        pos += above ? width : 0u;
        word >>= above ? width : 0u;
    }
    return pos;
}

// The j-th replica that takes part: only those of either mask get work items (a replica that sits the call out used to
// get waves that looked it up and left).  Found in the masks, which are in registers, not in a list in the arguments:
// that would be one more load in front of all others and 64 bytes more for the host to hand over with each launch.
template <bool EXT> __device__ __forceinline__ uint32_t replica_at(const ApplyArgs &a, const ExtArgs *xa, uint32_t j)
{
    if constexpr (EXT) {
        if (a.kcount != a.K) return nth_bit(xa->step_mask | xa->merge_mask, j);
    }
    return j;
}

// Multi-tensor apply.  Work item = (tile, group of kper replicas); one wave
// per item, items strided over the grid.  All table reads are wave-uniform.
// The waves of a workgroup are independent (no LDS, no barrier), so the
// workgroup size (64, 128 or 256 threads) is purely a dispatch-granularity knob.
template <int VEC, int OP, bool BF16, int NT, bool EXT>
__device__ __forceinline__ void apply_body(const ApplyArgs &a, const ExtArgs *xa)
{
    constexpr bool NEED_Z = (OP == OP_MERGE || OP == OP_STEP_MERGE || OP == OP_STEP_MEAN);
    const uint32_t lane = threadIdx.x & 63u;
    // the shape travels in the arguments: reading it from the dispatch would be a vector load before everything else
    const uint32_t wave0 = __builtin_amdgcn_readfirstlane(blockIdx.x * a.wpb + (threadIdx.x >> 6));
    load_together(a);
    uint32_t word = 0;
    bool looked = false;
    for (uint32_t i0 = wave0; i0 < a.nitems; i0 += a.nwaves) {
        const uint32_t item = in_order(i0, a);
        // Item order: tiles are taken in chunks of a.chunk; inside a chunk the items run
        // replica group by replica group, so that each replica's arrays are swept in
        // contiguous runs of a.chunk tiles while the chunk's z tiles are reused K times
        // within a short window (chunk = 1: the replicas of one tile are adjacent;
        // chunk = ntiles: one replica after the other).  Workgroups go to the eight
        // XCDs round-robin, each with its own L2: when a chunk is a multiple of eight
        // workgroups long, tile j of every replica lands on the same XCD, so only the
        // first replica's request for a z tile misses that L2.  The last, shorter chunk is
        // padded with idle items to such a multiple for the same reason, and so are the sweeps of a local step: what one
        // launch leaves in an XCD's L2, the next finds there, and what it left in another's costs more than the memory-side cache.
        uint32_t tile, kg;
        if (item < a.full_items) {
            const uint32_t ch = fast_div(item, a.by_per);
            const uint32_t r = item - ch * (a.chunk * a.kgroups);
            kg = fast_div(r, a.by_chunk);
            tile = ch * a.chunk + (r - kg * a.chunk);
        } else {
            const uint32_t r = item - a.full_items;
            kg = fast_div(r, a.by_stride);
            const uint32_t i = r - kg * a.tail_stride;
            if (i >= a.tail_chunk) continue;                    // padding item
            tile = a.tail_first + i;
        }
        const uint32_t k0 = kg * a.kper;
        const uint32_t k1 = (k0 + a.kper < a.kcount) ? k0 + a.kper : a.kcount;
        const uint32_t tensor = tensor_of(a, tile);
        if constexpr (BF16 && OP != OP_INIT) {
            if (__builtin_expect((a.place & LOOK) != 0u, 0)) {
                word = settle_word(a);
                looked = true;
            }
        }
        Record rec = load_record(a, replica_at<EXT>(a, xa, k0), tensor);
        const uint64_t in_s = !BF16 || word >= kSettled ? 0ull : a.at_s;
        const Tile t = locate(a, rec, tile, tensor, 256u * VEC);
        const bool full = (t.count == 256u * VEC);
        float4 zt[VEC];
        if constexpr (NEED_Z) {
            // the arenas are padded to whole rows: a full row of z is there even where the tensor ends inside it
            const float *zp = a.z + t.aoff;
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const uint32_t e = j * 256u + lane * 4u;
                zt[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (j == 0 || j * 256u < t.count) zt[j] = ld4<0>(zp + e);
            }
        }
        for (uint32_t j = k0;;) {
            const uint32_t k = replica_at<EXT>(a, xa, j);
            const size_t esz = BF16 ? 2 : 4;
            char *xu = reinterpret_cast<char *>(rec.x) + t.toff * esz;
            const char *gu = nullptr;
            if constexpr (OP == OP_STEP || OP == OP_STEP_MERGE)
                gu = reinterpret_cast<const char *>(rec.g) + t.toff * esz;
            const size_t ao = (size_t)k * a.npad + t.aoff;
            float *xm = BF16 ? a.x32 + ao : nullptr;
            const bool at_s = BF16 && ((in_s >> k) & 1ull);
            const float *xr = at_s ? a.s + ao : xm;
#define LASGD_TILE_AT(OPX, NLR, AL, AT)                                                                      \
    do {                                                                                                     \
        if (__builtin_expect(full, 1)) apply_tile<VEC, OPX, BF16, NT, true, EXT, OPX == OP, AT>(a, xu, gu, xr, xm, a.v + ao, a.s + ao, zt, t.wd, t.count, lane, NLR, AL); \
        else apply_tile<VEC, OPX, BF16, NT, false, EXT, OPX == OP, AT>(a, xu, gu, xr, xm, a.v + ao, a.s + ao, zt, t.wd, t.count, lane, NLR, AL);     \
    } while (0)
#define LASGD_TILE(OPX, NLR, AL)                                                                             \
    do {                                                                                                     \
        constexpr bool MAY = BF16 && (OPX == OP_MERGE || OPX == OP_STEP_MERGE);                              \
        if (MAY && at_s) LASGD_TILE_AT(OPX, NLR, AL, MAY);                                                   \
        else LASGD_TILE_AT(OPX, NLR, AL, false);                                                             \
    } while (0)
            if constexpr (!EXT) {
                LASGD_TILE(OP, a.neg_lr, 1.0f);
            } else {
                // a replica may take the local update, the global update, both or neither
                const bool in_step = (xa->step_mask >> k) & 1ull;
                const bool in_merge = (xa->merge_mask >> k) & 1ull;
                const float nlr = xa->neg_lr_k[k];
                if constexpr (OP == OP_STEP_MERGE) {
                    if (in_step && in_merge) LASGD_TILE(OP_STEP_MERGE, nlr, xa->alpha);
                    else if (in_step) LASGD_TILE(OP_STEP, nlr, 1.0f);
                    else if (in_merge) LASGD_TILE(OP_MERGE, 0.0f, xa->alpha);
                } else if constexpr (OP == OP_MERGE) {
                    if (in_merge) LASGD_TILE(OP_MERGE, 0.0f, xa->alpha);
                } else {
                    if (in_step) LASGD_TILE(OP, nlr, 1.0f);
                }
            }
#undef LASGD_TILE
#undef LASGD_TILE_AT
            if (++j == k1) break;
            rec = load_record(a, replica_at<EXT>(a, xa, j), tensor);
        }
    }
    if constexpr (BF16 && (NEED_Z || OP == OP_STEP)) {         // they write the master copy from the model, wherever that is
        if (__builtin_expect((a.place & SETTLES) != 0u, 0)) {
            if (!looked) word = settle_word(a);
            if (word < kSettled) count_settled(settle_words(a), wave0, a.nwaves, lane);
        }
    }
}

template <int VEC, int OP, bool BF16, int NT>
__global__ __launch_bounds__(256) void apply_kernel(const ApplyArgs a)
{
    apply_body<VEC, OP, BF16, NT, false>(a, nullptr);
}

template <int VEC, int OP, bool BF16, int NT>
__global__ __launch_bounds__(256) void apply_ext_kernel(const ApplyArgs a, const ExtArgs xa)
{
    apply_body<VEC, OP, BF16, NT, true>(a, &xa);
}

// ---- the mean (Sec. 3, Eq. 8) -----------------------------------------------
// z[e] = (1/K) sum_k s[k][e], fp64 accumulation in replica order, one rounding.
// The arenas are contiguous and padded with zeros, so this is a flat pass.
// EXT variants: the mean runs over a list of participants (partial All-Reduce,
// Sec. 6; the divisor is their number) and may be blended into the previous
// centre, z = (1-beta) z + beta mean (Sec. 3, Eq. 5).
struct AvgArgs {
    const float *s;
    float *z;
    uint64_t npad;      // elements per replica, multiple of 4
    uint64_t nvec;      // npad / 4
    uint32_t K;         // replicas summed (participants in the EXT variants)
    int32_t use_mul;    // K is a power of two: multiply by the exact reciprocal
    double inv_k, k_as_double;
    int32_t elastic;    // EXT: blend with the previous centre
    double beta, one_minus_beta;
    uint32_t blocks, threads; // the grid: reading it from the dispatch would be a vector load before everything else
    uint8_t idx[64];    // EXT: the participants, ascending
};

template <bool EXT> __device__ __forceinline__ uint32_t replica_of(const AvgArgs &a, uint32_t j)
{
    if constexpr (EXT) return a.idx[j];
    else return j;
}

template <bool EXT> __device__ __forceinline__ float finish_mean(double acc, float z_old, const AvgArgs &a)
{
    const double mean = a.use_mul ? acc * a.inv_k : acc / a.k_as_double;
    if constexpr (EXT) {
        if (a.elastic) {
            const double keep = a.one_minus_beta * (double)z_old;
            const double pull = a.beta * mean;
            return (float)(keep + pull);
        }
    }
    return (float)mean;
}

#define LASGD_ACC4(r)                                                                          \
    do { a0 += (double)(r).x; a1 += (double)(r).y; a2 += (double)(r).z; a3 += (double)(r).w; } while (0)

// SPLIT == 1: every lane owns one 128-bit column and walks all K replicas,
// eight loads in flight at a time.  z is stored without the hint in every form: it then waits in the memory-side cache for
// the global update, which hinted steps in between do not push out.  A cycle's us with / without the hint on z: ResNet-18
// list bf16 K = 6, m = 4 1012 / 995, ResNet-50 K = 3, m = 2 635 / 631 (other work between the passes 660 / 646), K = 1, 3e7 elements 279 / 270.
template <int NT, bool EXT>
__global__ __launch_bounds__(256) void average_kernel(const AvgArgs a)
{
    const uint64_t stride = (uint64_t)a.blocks * a.threads;
    // In one round, see load_together.  Not where the participants come from a list: there it makes the compiler hold the rows of two
    // batches at once, 78 registers in place of 48.  us with / without, an elastic mean and its update, ResNet-18 list: two participants
    // 101.7 / 98.0, three 139.5 / 134.4, six of eight 239.5 / 237.6; the plain mean K = 2 89.5 / 89.6, K = 3 125.0 / 125.9, K = 7 269 / 269.
    if constexpr (!EXT) asm volatile("" ::"s"(a.s), "s"(a.z), "s"(a.npad), "s"(a.K), "s"(a.use_mul));
    for (uint64_t i = (uint64_t)blockIdx.x * a.threads + threadIdx.x; i < a.nvec; i += stride) {
        const float *p = a.s + i * 4u;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        uint32_t k = 0;
        for (; k + 8u <= a.K; k += 8u) {
            float4 r[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = ld4<NT>(p + (uint64_t)replica_of<EXT>(a, k + u) * a.npad);
#pragma unroll
            for (int u = 0; u < 8; ++u) LASGD_ACC4(r[u]);
        }
        if (k + 4u <= a.K) {
            float4 r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = ld4<NT>(p + (uint64_t)replica_of<EXT>(a, k + u) * a.npad);
#pragma unroll
            for (int u = 0; u < 4; ++u) LASGD_ACC4(r[u]);
            k += 4u;
        }
        for (; k < a.K; ++k) {
            float4 r = ld4<NT>(p + (uint64_t)replica_of<EXT>(a, k) * a.npad);
            LASGD_ACC4(r);
        }
        float4 zo = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (EXT) {
            if (a.elastic) zo = *reinterpret_cast<const float4 *>(a.z + i * 4u);
        }
        float4 out = make_float4(finish_mean<EXT>(a0, zo.x, a), finish_mean<EXT>(a1, zo.y, a),
                                 finish_mean<EXT>(a2, zo.z, a), finish_mean<EXT>(a3, zo.w, a));
        st4<0>(a.z + i * 4u, out);          // the global update reads it back, K times
    }
}

// SPLIT in {2, 4}: the K replicas of one 256/SPLIT-column tile are divided
// among SPLIT groups of waves; each group sums a contiguous range of replicas
// in fp64, the partial sums meet in LDS and are added in group order.  More
// independent load streams per column for large K; the result can differ from
// the in-order sum only by fp64 rounding, i.e. in fp32 only at double-rounding ties.
template <int SPLIT, int NT, bool EXT>
__global__ __launch_bounds__(256) void average_split_kernel(const AvgArgs a)
{
    constexpr uint32_t COLS = 256u / SPLIT;             // 128-bit columns per workgroup pass
    __shared__ double part[SPLIT][COLS][4];
    const uint32_t g = threadIdx.x / COLS;              // which replica range
    const uint32_t c = threadIdx.x % COLS;
    const uint32_t kb = (uint32_t)(((uint64_t)a.K * g) / SPLIT);
    const uint32_t ke = (uint32_t)(((uint64_t)a.K * (g + 1u)) / SPLIT);
    const uint64_t ntile = (a.nvec + COLS - 1u) / COLS;
    for (uint64_t tile = blockIdx.x; tile < ntile; tile += a.blocks) {
        const uint64_t i = tile * COLS + c;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        if (i < a.nvec) {
            const float *p = a.s + i * 4u;
            uint32_t k = kb;
            for (; k + 4u <= ke; k += 4u) {
                float4 r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = ld4<NT>(p + (uint64_t)replica_of<EXT>(a, k + u) * a.npad);
#pragma unroll
                for (int u = 0; u < 4; ++u) LASGD_ACC4(r[u]);
            }
            for (; k < ke; ++k) {
                float4 r = ld4<NT>(p + (uint64_t)replica_of<EXT>(a, k) * a.npad);
                LASGD_ACC4(r);
            }
        }
        part[g][c][0] = a0; part[g][c][1] = a1; part[g][c][2] = a2; part[g][c][3] = a3;
        __syncthreads();
        // 256 threads finish COLS*4 = 1024/SPLIT elements: 4/SPLIT each, consecutive
        constexpr uint32_t PER = 4u / SPLIT;             // 2 or 1
        const uint32_t e0 = threadIdx.x * PER;           // element within the tile
        const uint64_t ebase = tile * COLS * 4u + e0;
        const bool inside = ebase + PER <= a.npad;
        float outv[PER];
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t e = e0 + q;
            double acc = 0.0;
#pragma unroll
            for (int gg = 0; gg < SPLIT; ++gg) acc += part[gg][e >> 2][e & 3u];
            float zo = 0.f;
            if constexpr (EXT) {
                if (a.elastic && inside) zo = a.z[ebase + q];
            }
            outv[q] = finish_mean<EXT>(acc, zo, a);
        }
        if (inside) {
            if constexpr (PER == 2) *reinterpret_cast<float2 *>(a.z + ebase) = make_float2(outv[0], outv[PER - 1]);
            else a.z[ebase] = outv[0];
        }
        __syncthreads();
    }
}

// ---- replica-group kernels ----------------------------------------------------
// Two operations need all K replicas of an element at once: the mean gradient of
// the SGD All-Reduce comparator, and the next mean z when it is computed in the
// same pass as the global update.  Both use one workgroup per tile with one wave
// per replica (wave w owns replicas w, w + W, ... when K exceeds the W = 16 waves
// a workgroup can hold).  Every wave streams its own replica's arrays exactly as
// the one-wave-per-(tile, replica) kernels do, the K values of each element meet
// in LDS as fp32 (exact), and the sum runs in fp64 in replica order, so the result
// is bit-identical to the in-order mean.  The tile is processed in rows of 256
// elements; LDS holds one row per replica (K KiB).
constexpr uint32_t kGroupWaves = 16;

// Elements [e0, e0+4) of one row for this lane; n = how many of them exist.
template <int NT, bool FULL> __device__ __forceinline__ float4 row_ld(const float *p, uint32_t e0, uint32_t n)
{
    if (FULL || n == 4u) return ld4<NT>(p + e0);
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (n > 0u) r.x = p[e0];
    if (n > 1u) r.y = p[e0 + 1u];
    if (n > 2u) r.z = p[e0 + 2u];
    return r;
}
template <int NT, bool FULL> __device__ __forceinline__ void row_st(float *p, uint32_t e0, uint32_t n, float4 a)
{
    if (FULL || n == 4u) { st4<NT>(p + e0, a); return; }
    if (n > 0u) p[e0] = a.x;
    if (n > 1u) p[e0 + 1u] = a.y;
    if (n > 2u) p[e0 + 2u] = a.z;
}
template <int NT, bool FULL> __device__ __forceinline__ void row_st16(uint16_t *p, uint32_t e0, uint32_t n, float4 a)
{
    if (FULL || n == 4u) { st2<NT>(p + e0, round4(a)); return; }
    if (n > 0u) p[e0] = (uint16_t)bf16_round(a.x);
    if (n > 1u) p[e0 + 1u] = (uint16_t)bf16_round(a.y);
    if (n > 2u) p[e0 + 2u] = (uint16_t)bf16_round(a.z);
}

// The next N rows of the exchange buffer, added to four columns' fp64 sums in replica order.  The N reads are issued
// before the first addition: one dependent read after the other costs 130 cycles each.
template <int N> __device__ __forceinline__ void add_rows(const float *p, double &a0, double &a1, double &a2, double &a3)
{
    float4 q[N];
#pragma unroll
    for (int k = 0; k < N; ++k) q[k] = *reinterpret_cast<const float4 *>(p + k * 256);
#pragma unroll
    for (int k = 0; k < N; ++k) LASGD_ACC4(q[k]);
}

// The same for K rows, FROM <= K <= TO.
template <int FROM, int TO> __device__ __forceinline__ void add_rows_of(uint32_t K, const float *p, double &a0, double &a1, double &a2, double &a3)
{
    if constexpr (FROM < TO)
        if (K != (uint32_t)FROM) return add_rows_of<FROM + 1, TO>(K, p, a0, a1, a2, a3);
    add_rows<FROM>(p, a0, a1, a2, a3);
}

// The mean of one row over its K values per element, which lie in lds[K][256]; every wave gets its lanes' columns.
// Up to K = 8 every wave sums them itself, which saves a barrier; beyond, up to four waves finish one column per
// thread and turn: only that thread reads the column, so the mean may replace replica 0's value in it.  SGD-AR mix,
// bare probe, every wave / shared: K = 4 6.12 / 6.01 TB/s, K = 8 6.08 / 6.01, K = 12 6.02 / 6.09, K = 16 5.51 / 5.89.
// FROM .. TO, if not 0: the kernel's K up to eight, and all reads of the rows come before the first addition, where few waves
// are on a CU to hide them.  It takes 20 registers more, too many for two sixteen-wave workgroups a CU in the SGD-AR step.
template <int FROM, int TO, class MEAN>
__device__ __forceinline__ float4 row_mean(float *lds, uint32_t K, uint32_t W, uint32_t lane, MEAN mean_of)
{
    if (K <= 8u) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        if constexpr (TO > 0) {
            add_rows_of<FROM, TO>(K, lds + lane * 4u, a0, a1, a2, a3);
        } else {
            for (uint32_t k = 0; k < K; ++k) {
                const float4 q = *reinterpret_cast<const float4 *>(lds + (size_t)k * 256u + lane * 4u);
                LASGD_ACC4(q);
            }
        }
        return make_float4(mean_of(a0), mean_of(a1), mean_of(a2), mean_of(a3));
    }
    const uint32_t fin = (W < 4u ? W : 4u) * 64u;
    if (threadIdx.x < fin) {
        for (uint32_t c = threadIdx.x; c < 256u; c += fin) {
            double acc = 0.0;
            for (uint32_t k = 0; k < K; ++k) acc += (double)lds[(size_t)k * 256u + c];
            lds[c] = mean_of(acc);
        }
    }
    __syncthreads();
    return *reinterpret_cast<const float4 *>(lds + lane * 4u);
}

template <int N> struct Count { static constexpr int value = N; };

__device__ __forceinline__ float group_mean_of(double acc, const ApplyArgs &a)
{
    return (float)(a.use_mul ? acc * a.inv_k : acc / a.k_as_double);
}

// Where replica k keeps one tile: the fp32 model (the caller's buffer, or the master
// copy for bf16 storage), the caller's 16-bit parameters and gradient, v and s.
template <bool BF16> struct ReplicaTile {
    const float *xf;       // read here, written at xw: another place only where the model has just been re-sent (at_s)
    float *xw, *v, *s;
    uint16_t *x16;
    const void *g;
};
// Where a replica-group kernel finds the models: each as at_s says; all in s; at_s holds until settled, and it counts (the last two: bf16 only).
// By kind and not by a test at the start, which was a round of scalar loads more in front of all others: 2-3 % of a fused update
// (us, K = 8, bf16: 2,000,003 elements 98.8 with, 97.0 without; 3,000,003 144.6 / 141.1).
enum Place : int { PLACE_AT_S = 0, PLACE_ALL_IN_S = 1, PLACE_SETTLE = 2 };
template <bool BF16>
__device__ __forceinline__ ReplicaTile<BF16> replica_tile(const ApplyArgs &a, const Tile &t, const Record &rec, uint32_t k, uint64_t in_s)
{
    constexpr size_t ESZ = BF16 ? 2 : 4;
    const size_t ao = (size_t)k * a.npad + t.aoff;
    char *xu = reinterpret_cast<char *>(rec.x) + t.toff * ESZ;
    ReplicaTile<BF16> r;
    r.xw = BF16 ? a.x32 + ao : reinterpret_cast<float *>(xu);
    r.xf = BF16 && ((in_s >> k) & 1ull) ? a.s + ao : r.xw;
    r.x16 = reinterpret_cast<uint16_t *>(xu);
    r.v = a.v + ao;
    r.s = a.s + ao;
    r.g = reinterpret_cast<const char *>(rec.g) + t.toff * ESZ;
    return r;
}
template <bool BF16>
__device__ __forceinline__ ReplicaTile<BF16> replica_tile(const ApplyArgs &a, const Tile &t, uint32_t k, uint32_t tensor, uint64_t in_s)
{
    return replica_tile<BF16>(a, t, load_record(a, k, tensor), k, in_s);
}
// The loads of R replicas' gradients (G) and models (X) from the caller's buffers.  The last row of a tensor takes the
// same 128-bit accesses in the lanes that have four elements; only the one lane with one to three goes element by
// element.  All replicas' loads are issued before anything waits: array by array, every one of them waited for the last
// (flat list of 1000 elements, K = 64: fused update 16.3 -> 12.9 us, SGD-AR 10.2 -> 8.1).  The library's own arrays need none of this: they are
// padded to whole rows.
template <int R, bool BF16, int NT, bool FULL, bool G, bool X>
__device__ __forceinline__ void ld_caller(const ReplicaTile<BF16> (&q)[R], uint32_t e0, uint32_t n, float4 (&g)[R], float4 (&x)[R])
{
    if constexpr (!FULL) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (G) g[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (X && !BF16) x[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    if constexpr (X && BF16) {             // the master copy: whole rows
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = ld4<NT>(q[r].xf + e0);
    }
    if (FULL || n == 4u) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (G) g[r] = BF16 ? widen4(ld2<NT>(static_cast<const uint16_t *>(q[r].g) + e0)) : ld4<NT>(static_cast<const float *>(q[r].g) + e0);
            if constexpr (X && !BF16) x[r] = ld4<NT>(q[r].xf + e0);
        }
    }
    if constexpr (!FULL) {
        if (n - 1u < 3u) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                LASGD_FOR4(if (c < 3 && (uint32_t)c < n) {
                    if constexpr (G) comp(g[r], c) = BF16 ? bf16_widen(*as_global<uint16_t>(static_cast<const uint16_t *>(q[r].g) + e0 + c))
                                                          : *as_global<float>(static_cast<const float *>(q[r].g) + e0 + c);
                    if constexpr (X && !BF16) comp(x[r], c) = *as_global<float>(q[r].xf + e0 + c);
                })
        }
    }
}

// A wave owns replicas w + q*W, q = 0, 1, ...; it takes them R at a time ("pass").
// A wave whose pass runs past K re-reads replica K-1 and keeps nothing of it, so
// that the loads of a pass stay free of branches.

// SGD All-Reduce comparator (Sec. 2; "SGD-AR" of Table 1), one row of a tile:
// the K gradients are averaged (fp64 in replica order, one rounding to fp32) and
// every replica takes the local update with that mean gradient.  Same 20 bytes
// per replica-parameter as a local step.
// STAGED: the models are asked for when the gradients have arrived, and fly while these go round through LDS.
template <int R, bool BF16, int NT, bool FULL, bool STAGED>
__device__ __forceinline__ void sgd_ar_row(const ApplyArgs &a, const Tile &t, const Record &rec0, uint32_t tensor, float *lds, uint32_t row,
                                           uint32_t w, uint32_t W, uint32_t passes, uint32_t lane, uint64_t in_s)
{
    const uint32_t e0 = row * 256u + lane * 4u;
    const uint32_t n = FULL ? 4u : (e0 >= t.count) ? 0u : (t.count - e0 < 4u) ? t.count - e0 : 4u;
    // first pass: the model loads are issued ahead of the exchange
    float4 x[R], v[R];
    ReplicaTile<BF16> rt[R];
    bool mine[R];
    {
        float4 g[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t kw = w + (uint32_t)r * W;
            mine[r] = kw < a.K;
            rt[r] = r == 0 ? replica_tile<BF16>(a, t, rec0, kw, in_s) : replica_tile<BF16>(a, t, mine[r] ? kw : a.K - 1u, tensor, in_s);
        }
        ld_caller<R, BF16, NT, FULL, true, !STAGED>(rt, e0, n, g, x);
        if constexpr (STAGED) {
            wait_for_loads();
            ld_caller<R, BF16, NT, FULL, false, true>(rt, e0, n, g, x);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = ld4<NT>(rt[r].v + e0);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (mine[r]) *reinterpret_cast<float4 *>(lds + (size_t)(w + (uint32_t)r * W) * 256u + lane * 4u) = g[r];
    }
    for (uint32_t p = 1; p < passes; ++p) {
        ReplicaTile<BF16> q[R];
        float4 g[R];
        uint32_t kw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            kw[r] = w + (p * R + (uint32_t)r) * W;
            q[r] = replica_tile<BF16>(a, t, kw[r] < a.K ? kw[r] : a.K - 1u, tensor, in_s);
        }
        ld_caller<R, BF16, NT, FULL, true, false>(q, e0, n, g, g);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (kw[r] < a.K) *reinterpret_cast<float4 *>(lds + (size_t)kw[r] * 256u + lane * 4u) = g[r];
    }
    __syncthreads();
    const float4 gbar = row_mean<0, 0>(lds, a.K, W, lane, [&a](double acc) { return group_mean_of(acc, a); });
#pragma unroll
    for (int r = 0; r < R; ++r) {
        LASGD_FOR4(step_elem(comp(x[r], c), comp(v[r], c), compv(gbar, c), t.wd, a.mu, a.neg_lr, a.nesterov);)
        if (mine[r]) {
            row_st<NT, FULL>(rt[r].v, e0, n, v[r]);
            row_st<NT, FULL>(rt[r].xw, e0, n, x[r]);
            if constexpr (BF16) row_st16<NT, FULL>(rt[r].x16, e0, n, x[r]);
        }
    }
    for (uint32_t p = 1; p < passes; ++p) {
        ReplicaTile<BF16> q[R];
        float4 xx[R], vv[R];
        bool ok[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t kw = w + (p * R + (uint32_t)r) * W;
            ok[r] = kw < a.K;
            q[r] = replica_tile<BF16>(a, t, ok[r] ? kw : a.K - 1u, tensor, in_s);
        }
        ld_caller<R, BF16, NT, FULL, false, true>(q, e0, n, xx, xx);
#pragma unroll
        for (int r = 0; r < R; ++r) vv[r] = ld4<NT>(q[r].v + e0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            LASGD_FOR4(step_elem(comp(xx[r], c), comp(vv[r], c), compv(gbar, c), t.wd, a.mu, a.neg_lr, a.nesterov);)
            if (ok[r]) {
                row_st<NT, FULL>(q[r].v, e0, n, vv[r]);
                row_st<NT, FULL>(q[r].xw, e0, n, xx[r]);
                if constexpr (BF16) row_st16<NT, FULL>(q[r].x16, e0, n, xx[r]);
            }
        }
    }
}

template <int R, bool BF16, int NT, bool STAGED, int PLACE>
__global__ __launch_bounds__(1024) void sgd_ar_kernel(const ApplyArgs a, const uint32_t passes)
{
    extern __shared__ float lds[];                        // [K][256]
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t W = a.wpb;
    bool again = false;
    uint32_t word = 0;
    for (uint32_t i0 = blockIdx.x; i0 < a.ntiles; i0 += a.nwaves) {
        const uint32_t tile = i0 < a.nitems ? in_order(i0, a) : i0;      // the last, less than eight, keep their places
        if constexpr (PLACE == PLACE_SETTLE) word = settle_word(a);
        const uint32_t tensor = tensor_of(a, tile);
        const Record rec0 = load_record(a, w, tensor);       // of this wave's first replica: W <= K
        const uint64_t in_s = !BF16 || word >= kSettled ? 0ull : a.at_s;
        const Tile t = locate(a, rec0, tile, tensor, a.tile_elems);
        const uint32_t rows = (t.count + 255u) >> 8;
        for (uint32_t row = 0; row < rows; ++row) {
            if (again) __syncthreads();     // a further row reuses the LDS buffer; after the last one waves leave as they finish
            again = true;
            if (t.count - row * 256u >= 256u) sgd_ar_row<R, BF16, NT, true, STAGED>(a, t, rec0, tensor, lds, row, w, W, passes, lane, in_s);
            else sgd_ar_row<R, BF16, NT, false, STAGED>(a, t, rec0, tensor, lds, row, w, W, passes, lane, in_s);
        }
    }
    if constexpr (PLACE == PLACE_SETTLE) {
        if (word < kSettled) count_settled(settle_words(a), blockIdx.x * W + w, a.nwaves * W, lane);       // every workgroup has a tile
    }
}

// The same in two kernels: the mean gradient (here) into an arena of its own, then OP_STEP_MEAN, which reads it as an update
// reads z.  Bound by HBM like the mean of the sent models: one wave a tile, eight replicas' rows in flight, summed in replica
// order, so the result is that of the one kernel to the bit.  It moves 8 bytes a parameter more than the one kernel and gains
// from one-wave workgroups; mean_grad_first in the host code holds the line and both sides.
template <bool BF16, int NT, bool FULL>
__device__ __forceinline__ void mean_grad_tile(const ApplyArgs &a, const Tile &t, uint32_t tensor, uint32_t lane)
{
    constexpr uint32_t N = 8;
    const uint32_t e = lane * 4u, n = lane_elems<FULL>(e, t.count);
    const LASGD_CONST_AS Record *rec = as_const(a.records) + tensor;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    auto rows = [&](uint32_t k, auto count) {
        constexpr int M = decltype(count)::value;
        float4 g[M];
        const char *p[M];
#pragma unroll
        for (int u = 0; u < M; ++u) {
            p[u] = reinterpret_cast<const char *>(rec[(size_t)(k + u) * a.n_tensors].g) + t.toff * (BF16 ? 2 : 4);
            if constexpr (!FULL) g[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if (FULL || n == 4u) {
#pragma unroll
            for (int u = 0; u < M; ++u)
                g[u] = BF16 ? widen4(ld2<NT>(reinterpret_cast<const uint16_t *>(p[u]) + e)) : ld4<NT>(reinterpret_cast<const float *>(p[u]) + e);
        }
        if constexpr (!FULL) {         // the one lane that a tensor's odd end leaves with one to three
            if (n - 1u < 3u) {
#pragma unroll
                for (int u = 0; u < M; ++u)
                    LASGD_FOR4(if (c < 3 && (uint32_t)c < n) comp(g[u], c) = BF16 ? bf16_widen(as_global<uint16_t>(p[u])[e + c]) : as_global<float>(p[u])[e + c];)
            }
        }
#pragma unroll
        for (int u = 0; u < M; ++u) LASGD_ACC4(g[u]);
    };
    uint32_t k = 0;
    for (; k + N <= a.K; k += N) rows(k, Count<N>{});
    if (k + 4u <= a.K) { rows(k, Count<4>{}); k += 4u; }
    if (k + 2u <= a.K) { rows(k, Count<2>{}); k += 2u; }
    if (k < a.K) rows(k, Count<1>{});
    // a whole row: the arena is padded, and the step that reads it takes whole rows too
    st4<0>(a.z + t.aoff + e, make_float4(group_mean_of(a0, a), group_mean_of(a1, a), group_mean_of(a2, a), group_mean_of(a3, a)));
}

template <bool BF16, int NT>
__global__ __launch_bounds__(64) void mean_grad_kernel(const ApplyArgs a)          // tiles of 256 elements
{
    for (uint32_t tile = blockIdx.x; tile < a.ntiles; tile += a.nwaves) {
        const uint32_t tensor = tensor_of(a, tile);
        const Tile t = locate(a, load_record(a, 0, tensor), tile, tensor, 256u);
        if (t.count == 256u) mean_grad_tile<BF16, NT, true>(a, t, tensor, threadIdx.x);
        else mean_grad_tile<BF16, NT, false>(a, t, tensor, threadIdx.x);
    }
}

// Steps 7 and 9a-c of Algorithm 1 and the next All-Reduce (Sec. 3, Eq. 8) in one
// pass: every replica takes its local update, then the global update with the
// pending z, re-sends (s <- x), and the tile's next z -- the mean of the models
// just sent -- is written over the old one.  Only this workgroup touches the
// tile's z, and all its waves have used the old values before the barrier.
// Same roundings as step_merge followed by the in-order mean.
// STAGED: the gradients are asked for when everything else has arrived, so that a wave has
// three quarters of its loads in flight.
// AT_S: every replica's model is the one it sent last (see apply_tile), read once for both.
template <int R, bool BF16, int NT, bool FULL, bool STAGED, bool AT_S>
__device__ __forceinline__ void step_merge_mean_row(const ApplyArgs &a, const Tile &t, const Record &rec0, uint32_t tensor, float *lds, uint32_t row,
                                                    uint32_t w, uint32_t W, uint32_t passes, uint32_t lane, uint64_t in_s)
{
    const uint32_t e0 = row * 256u + lane * 4u;
    const uint32_t n = FULL ? 4u : (e0 >= t.count) ? 0u : (t.count - e0 < 4u) ? t.count - e0 : 4u;
    float4 z;                                                      // shared by the K waves: cacheable
    if constexpr (!STAGED) z = ld4<0>(a.z + t.aoff + e0);
    for (uint32_t p = 0; p < passes; ++p) {
        ReplicaTile<BF16> q[R];
        float4 x[R], v[R], g[R], ss[R];
        uint32_t kw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            kw[r] = w + (p * R + (uint32_t)r) * W;
            q[r] = r == 0 && p == 0u ? replica_tile<BF16>(a, t, rec0, kw[r], in_s) : replica_tile<BF16>(a, t, kw[r] < a.K ? kw[r] : a.K - 1u, tensor, in_s);
        }
        ld_caller<R, BF16, NT, FULL, !STAGED, true>(q, e0, n, g, x);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = ld4<NT>(q[r].v + e0);
            if constexpr (STAGED) {
                if (r == 0 && p == 0u) z = ld4<0>(a.z + t.aoff + e0);
            }
            if constexpr (!AT_S) ss[r] = ld4<NT>(q[r].s + e0);
        }
        if constexpr (STAGED) {
            wait_for_loads();
            ld_caller<R, BF16, NT, FULL, true, false>(q, e0, n, g, x);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (AT_S) ss[r] = x[r];
            LASGD_FOR4(step_elem(comp(x[r], c), comp(v[r], c), compv(g[r], c), t.wd, a.mu, a.neg_lr, a.nesterov);)
            LASGD_FOR4(comp(x[r], c) = merge_elem(compv(x[r], c), compv(ss[r], c), compv(z, c));)
            if (kw[r] < a.K) {
                row_st<NT, FULL>(q[r].v, e0, n, v[r]);
                if (!BF16 || (a.place & ALSO_X)) row_st<NT, FULL>(q[r].xw, e0, n, x[r]);
                if constexpr (BF16) row_st16<NT, FULL>(q[r].x16, e0, n, x[r]);
                row_st<NT, FULL>(q[r].s, e0, n, x[r]);
                *reinterpret_cast<float4 *>(lds + (size_t)kw[r] * 256u + lane * 4u) = x[r];
            }
        }
    }
    __syncthreads();
    // up to four waves finish the row's mean, one element per thread and turn
    const uint32_t fin = (W < 4u ? W : 4u) * 64u;
    if (threadIdx.x < fin) {
        for (uint32_t c = threadIdx.x; c < 256u; c += fin) {
            const uint32_t e = row * 256u + c;
            if (FULL || e < t.count) {
                double acc = 0.0;
                for (uint32_t k = 0; k < a.K; ++k) acc += (double)lds[(size_t)k * 256u + c];
                a.z[t.aoff + e] = group_mean_of(acc, a);
            }
        }
    }
}

template <int R, bool BF16, int NT, bool STAGED, int PLACE>
__global__ __launch_bounds__(1024) void step_merge_mean_kernel(const ApplyArgs a, const uint32_t passes)
{
    extern __shared__ float lds[];                        // [K][256]
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t W = a.wpb;
    bool again = false;
    uint32_t word = 0;
    for (uint32_t i0 = blockIdx.x; i0 < a.ntiles; i0 += a.nwaves) {
        const uint32_t tile = i0 < a.nitems ? in_order(i0, a) : i0;      // the last, less than eight, keep their places
        if constexpr (PLACE == PLACE_SETTLE) word = settle_word(a);
        const uint32_t tensor = tensor_of(a, tile);
        const Record rec0 = load_record(a, w, tensor);       // of this wave's first replica: W <= K
        const uint64_t in_s = !BF16 || word >= kSettled ? 0ull : a.at_s;
        const Tile t = locate(a, rec0, tile, tensor, a.tile_elems);
        const uint32_t rows = (t.count + 255u) >> 8;
        for (uint32_t row = 0; row < rows; ++row) {
            if (again) __syncthreads();     // a further row reuses the LDS buffer; after the last one waves leave as they finish
            again = true;
            if (t.count - row * 256u >= 256u) step_merge_mean_row<R, BF16, NT, true, STAGED, PLACE == PLACE_ALL_IN_S>(a, t, rec0, tensor, lds, row, w, W, passes, lane, in_s);
            else step_merge_mean_row<R, BF16, NT, false, STAGED, PLACE == PLACE_ALL_IN_S>(a, t, rec0, tensor, lds, row, w, W, passes, lane, in_s);
        }
    }
    if constexpr (PLACE == PLACE_SETTLE) {
        if (word < kSettled) count_settled(settle_words(a), blockIdx.x * W + w, a.nwaves * W, lane);       // every workgroup has a tile
    }
}

// Every bound gradient to zero.  Bound by the stores (and, for small lists, by its one launch); one wave per (tile, replica) in
// sweeps of whole replicas, found through the records as everywhere, so that one launch does what a fill per tensor or
// a list of pointers handed over with each launch did.  MobileNetV2 list, K = 4, 632 tensors, clear + accumulate + step twice:
// 397 us with eight launches over pointer lists and walks in Python, 250 with this and the native walk (grad_walk.cpp).
template <bool BF16, int NT>
__global__ __launch_bounds__(64) void zero_grads_kernel(const ApplyArgs a)
{
    const uint32_t lane = threadIdx.x;
    for (uint32_t item = blockIdx.x; item < a.nitems; item += a.nwaves) {
        const uint32_t k = fast_div(item, a.by_chunk), tile = item - k * a.chunk;
        const uint32_t tensor = tensor_of(a, tile);
        const Record rec = load_record(a, k, tensor);
        const Tile t = locate(a, rec, tile, tensor, a.tile_elems);
        char *g = reinterpret_cast<char *>(rec.g) + t.toff * (BF16 ? 2 : 4);
        for (uint32_t e = lane * 4u; e < t.count; e += 256u) {
            const uint32_t n = lane_elems<false>(e, t.count);
            if constexpr (BF16) {
                uint16_t *p = reinterpret_cast<uint16_t *>(g) + e;
                if (n == 4u) st2<NT>(p, make_uint2(0u, 0u));
                else
                    for (uint32_t i = 0; i < n; ++i) *as_global<uint16_t>(p + i) = 0;
            } else {
                float *p = reinterpret_cast<float *>(g) + e;
                if (n == 4u) st4<NT>(p, make_float4(0.f, 0.f, 0.f, 0.f));
                else
                    for (uint32_t i = 0; i < n; ++i) *as_global<float>(p + i) = 0.f;
            }
        }
    }
}

// The same as a kernel of its own: the models of `mask` from s back to the master copies, once.  For a call that runs before the
// first replay, and in a graph whose first kernel does not write all of them.
__global__ __launch_bounds__(256) void settle_kernel(float *x32, const float *s, uint64_t npad, uint64_t mask, uint32_t *settle)
{
    if (*as_global<uint32_t>(settle) >= kSettled) return;
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (; mask; mask &= mask - 1ull) {
        const uint64_t k = (uint64_t)__builtin_ctzll(mask);
        for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < npad / 4u; i += stride) st4<3>(x32 + k * npad + i * 4u, ld4<3>(s + k * npad + i * 4u));
    }
    __syncthreads();
    count_settled(settle, blockIdx.x, gridDim.x, threadIdx.x);
}

// Debugging aid for the two-stream protocol: fill z with NaN.
__global__ __launch_bounds__(256) void poison_kernel(float *z, uint64_t n)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) z[i] = __uint_as_float(0x7fc00000u);
}

// ---- context-free global update on flat fp32 vectors -------------------------
// For callers that hold no context and may not allocate: the mean (Sec. 3,
// Eq. 8) of K sent models and the global update (Algorithm 1 step 9a-c) in one
// pass.  Same arithmetic and rounding order as the kernels above; replica
// pointers travel in the kernel arguments.
//
// Bound by HBM.  One workgroup per 256 elements, R replicas a wave: s and x are read once, the K values of s meet in
// LDS, and z stays on the chip, so a replica-parameter moves 16 bytes where a
// mean kernel followed by an update kernel moves 20 and z on top.  Where the vectors stream (NT) and a wave has one replica or
// two, x is asked for when s has arrived, and flies while s goes round through LDS, so that a wave puts half of its 2 KiB a
// replica in flight at a time.  launch_flat_update holds the shape's rule and what it measured.
// n = 25,000,000, us over three states in turn (before: one replica a wave, both loads at once, as many groups as fit): K = 8 511
// = 6.3 TB/s (542), K = 4 248 (264), K = 12 787 (814).  n = 300,000, K = 8 8.3 (a mean kernel and an update kernel: 14.2).
// Pointers of x and s side by side, one 16-byte scalar load a replica, were 2-4 % slower in the cache (n = 10^6, K = 6 17.4 / 18.0).
struct FlatArgs {
    float *x[64];       // local models, n elements each
    float *s[64];       // sent models
    uint64_t n;
    uint32_t K, W;      // replicas; waves per workgroup
    int32_t use_mul;    // K is a power of two: multiply by the exact reciprocal
    double inv_k, k_as_double;
    int32_t resnap;
};

__device__ __forceinline__ float flat_mean_of(double acc, const FlatArgs &a)
{
    return (float)(a.use_mul ? acc * a.inv_k : acc / a.k_as_double);
}

constexpr uint32_t kFlatOneMaxK = 3;      // streaming: up to so many replicas one a wave, beyond two

template <int R, int NT, bool FULL>
__device__ __forceinline__ void flat_update_row(const FlatArgs &a, float *lds, uint64_t first, uint32_t count,
                                                uint32_t w, uint32_t W, uint32_t lane)
{
    constexpr bool STAGED = NT != 0 && R < 4;
    const uint32_t e0 = lane * 4u;
    const uint32_t n = FULL ? 4u : (e0 >= count) ? 0u : (count - e0 < 4u) ? count - e0 : 4u;
    float4 x[R], ss[R];
    float *xp[R], *sp[R];
    bool mine[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {        // a wave that runs past K re-reads replica K-1 and keeps nothing of it
        const uint32_t kw = w + (uint32_t)r * W;
        mine[r] = kw < a.K;
        sp[r] = a.s[mine[r] ? kw : a.K - 1u] + first;
        xp[r] = a.x[mine[r] ? kw : a.K - 1u] + first;
        ss[r] = row_ld<NT, FULL>(sp[r], e0, n);
        if constexpr (!STAGED) x[r] = row_ld<NT, FULL>(xp[r], e0, n);
    }
    if constexpr (STAGED) {
        wait_for_loads();
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = row_ld<NT, FULL>(xp[r], e0, n);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (mine[r]) *reinterpret_cast<float4 *>(lds + (size_t)(w + (uint32_t)r * W) * 256u + e0) = ss[r];
    __syncthreads();
    const float4 z = row_mean<!STAGED ? 0 : R == 1 ? 1 : (int)kFlatOneMaxK + 1, !STAGED ? 0 : R == 1 ? (int)kFlatOneMaxK : 8>(
        lds, a.K, W, lane, [&a](double acc) { return flat_mean_of(acc, a); });
#pragma unroll
    for (int r = 0; r < R; ++r) {
        LASGD_FOR4(comp(x[r], c) = merge_elem(compv(x[r], c), compv(ss[r], c), compv(z, c));)
        if (mine[r]) {
            row_st<NT, FULL>(xp[r], e0, n, x[r]);
            if (a.resnap) row_st<NT, FULL>(sp[r], e0, n, x[r]);
        }
    }
}

template <int R, int NT>
__global__ __launch_bounds__(1024) void flat_update_kernel(const FlatArgs a)
{
    extern __shared__ float lds[];                        // [K][256]
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t W = a.W;
    const uint64_t first = (uint64_t)blockIdx.x * 256u;
    if (a.n - first >= 256u) flat_update_row<R, NT, true>(a, lds, first, 256u, w, W, lane);
    else flat_update_row<R, NT, false>(a, lds, first, (uint32_t)(a.n - first), w, W, lane);
}

} // namespace lasgd
