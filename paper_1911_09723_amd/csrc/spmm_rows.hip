// Row kernels for fp32: a wavefront sums one output channel at a time over many
// columns.  The row's channels and weights are wavefront-uniform (scalar loads,
// an SGPR operand of the multiply-adds), so a stored weight costs one address
// and one read of X a lane and 4 (or 2) multiply-adds, nothing is padded to a
// neighbour's length, and a row is stored in pieces of whole 128-byte lines.
//
// rows_kernel, for runs of few columns: 256 columns a wavefront, X straight from
// L2.  Such a run is bound by latency: the other kernels copy X to LDS, wait for
// the copy, and walk rows of several lane groups in lockstep (512 -> 512 @ 14 x
// 14, one image: 13.7 us).  Here every output channel is a wavefront of its own,
// nothing is staged and nothing is shared, and 16 loads are in flight (6.3 us;
// 512 -> 1024 @ 7 x 7 18.1 -> 5.8; 1280 -> 320 @ 7 x 7 57.7 -> 10.0; 32 -> 64 @ 56 x
// 56 5.1 -> 3.3).  What bounds it on longer runs is the L1 rate, 4 bytes per
// multiply-add.
//
// strip_rows_kernel, for longer runs of up to 160 input channels: X of 64 (or
// 32) units in LDS, the next tile's on its way in registers.  What bounds it: on
// narrow layers the traffic (a version without the products takes 66 of 66 us on
// 32 -> 64 @ 112 x 112, batch 64, at 4.7 TB/s; 52 of 64 on 128 -> 128 @ 56 x 56),
// on denser ones issue: a SIMD issues a vector instruction every 4.6 cycles with
// 4 wavefronts and every 8.6 with one, scalar ones beside them as long as they
// are not more.  So 16 wavefronts a compute unit, groups of 4 weights with 8
// scalar instructions to 20 vector ones, one wait a group.  Against the kernels
// it replaces (us): 24 -> 144 @ 56 x 56 batch 128 63 -> 55, 144 -> 24 77 -> 67, 96 ->
// 576 @ 14 x 14 29 -> 26, 160 -> 960 @ 7 x 7 34 -> 24, 128 -> 256 @ 28 x 28 batch 64
// 35 -> 28, 128 -> 128 @ 56 x 56 batch 64 64.4 -> 61.7 (70% sparse 130 -> 92, 1 x 4
// 92 -> 65), 32 -> 64 @ 112 x 112 68.6 -> 66.9, 144 -> 24 @ 56 x 56 1 x 4 130 -> 39.
//
// Columns are taken in units of 4 neighbours of one plane; the last unit of a
// plane whose size is not a multiple of 4 starts early and repeats columns of
// the one before (the same sums, the same bits), so every load and store is
// whole.  Each output is summed in ascending input channel from zero with
// fused multiply-adds (a row that the strip plan splits as the sum of its two
// pieces), the bias last: the bits of the other kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>

#include "launch.hpp"

namespace spconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

using ConstI = __attribute__((address_space(4))) const int32_t;
using ConstF = __attribute__((address_space(4))) const float;
typedef uint32_t u16v __attribute__((ext_vector_type(16), aligned(4)));
using ConstU16 = __attribute__((address_space(4))) const u16v;

constexpr int32_t kOutOfRange = static_cast<int32_t>(0x80000000u);
constexpr int64_t kMaxRecords = 0x7ffffff0;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), static_cast<short>(0),
                                             static_cast<int>(bytes < kMaxRecords ? bytes : kMaxRecords), 0x00020000);
}

struct RArgs {
    const float *x;
    float *y;
    const float *bias;       // every output channel
    const int32_t *row_ptr;  // stored weights by output channel
    const uint32_t *ent;     // channel, fp32 weight bits
    int32_t cin, cout, hw;
    int32_t units, all;      // 4-column units of a plane, of the run
    int32_t blocks;          // wavefronts (64 units) per output channel
    float lo, hi;            // the activation as a clamp
};

constexpr int kRowWaves = 4;
constexpr int kRowDepth = 8;  // loads per batch; two batches in flight

// The sum over n stored weights of one row (ent: weight t's channel in word 2 t,
// its bits in 2 t + 1; a batch's in one scalar load) times X at xb; P = 2: of the
// even and of the odd ones apart, then both.
template <int P>
__device__ __forceinline__ f4 row_sum(const ConstI *ent, int32_t n, const float *xb, int32_t hw) {
    f4 acc[P] = {};
    constexpr int D = kRowDepth;
    auto load = [&](const u16v &r, f4(&v)[D]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D; ++i)
            __builtin_memcpy(&v[i], xb + static_cast<int64_t>(static_cast<int32_t>(r[2 * i])) * hw, 16);
    };
    auto sum = [&](const u16v &r, const f4(&v)[D]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[i % P][e] = __builtin_fmaf(__uint_as_float(r[2 * i + 1]), v[i][e], acc[i % P][e]);
    };
    const int32_t batches = n / D;
    f4 va[D], vb[D];
    if (batches > 0) {
        const ConstU16 *rec = reinterpret_cast<const ConstU16 *>(ent);
        u16v ra = rec[0];
        load(ra, va);
        int32_t b = 0;
        for (; b + 2 <= batches; b += 2) {
            const u16v rb = rec[b + 1];
            load(rb, vb);
            sum(ra, va);
            if (b + 2 < batches) {
                ra = rec[b + 2];
                load(ra, va);
            }
            sum(rb, vb);
        }
        if (b < batches)
            sum(ra, va);
    }
    // the rest, 1 .. D - 1 weights: their loads together, too
    const int32_t done = batches * D;
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (done + i < n)
            __builtin_memcpy(&vb[i], xb + static_cast<int64_t>(ent[2 * (done + i)]) * hw, 16);
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (done + i < n) {
            const float w = __int_as_float(ent[2 * (done + i) + 1]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[i % P][e] = __builtin_fmaf(w, vb[i][e], acc[i % P][e]);
        }
    if constexpr (P == 2)
        acc[0] += acc[1];
    return acc[0];
}

// SPLIT: the plan has rows in two pieces.
template <bool SPLIT>
__global__ void __launch_bounds__(64 * kRowWaves) rows_kernel(RArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t item = static_cast<int32_t>(blockIdx.x) * kRowWaves + wave;
    const int32_t row = item / a.blocks;
    if (row >= a.cout)
        return;
    const int32_t g = min((item - row * a.blocks) * 64 + lane, a.all - 1);  // lanes past the end repeat the last unit
    const int32_t im = g / a.units;
    const int32_t p = min(4 * (g - im * a.units), a.hw - 4);
    const float *xb = a.x + static_cast<int64_t>(im) * a.cin * a.hw + p;
    const ConstI *rp = reinterpret_cast<const ConstI *>(reinterpret_cast<uintptr_t>(a.row_ptr));
    const int32_t r0 = rp[row], t0 = SPLIT ? r0 & ~kRowSplit : r0;
    const int32_t n = (SPLIT ? rp[row + 1] & ~kRowSplit : rp[row + 1]) - t0;
    const ConstI *ent = reinterpret_cast<const ConstI *>(reinterpret_cast<uintptr_t>(a.ent)) + 2 * static_cast<int64_t>(t0);
    f4 acc;
    if (SPLIT && (r0 & kRowSplit))
        acc = row_sum<2>(ent, n, xb, a.hw);
    else
        acc = row_sum<1>(ent, n, xb, a.hw);
    const ConstF *bias = reinterpret_cast<const ConstF *>(reinterpret_cast<uintptr_t>(a.bias));
    f4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = fminf(fmaxf(acc[e] + bias[row], a.lo), a.hi);
    __builtin_memcpy(a.y + (static_cast<int64_t>(im) * a.cout + row) * a.hw + p, &v, 16);
}

// ---------------------------------------------------------------------------
// LDS row kernel
// ---------------------------------------------------------------------------

struct SArgs {
    const float *x;
    float *y;
    const uint32_t *ent, *desc;
    const int32_t *list;
    int32_t cin, cout, hw, images;
    int32_t units;           // 4-column units of a plane
    int32_t tunits;          // units of a tile, of one or more images
    int32_t rounds;          // whole tiles of every workgroup
    int32_t rest, parts;     // tiles left after them, and workgroups sharing the rows of each
    int32_t nxcd;            // the grid is a multiple of it
    int32_t row_bytes;       // bytes of an LDS row: 16 * tunits
    int64_t x_bytes, y_bytes;
    float lo, hi;            // the activation as a clamp
};

constexpr int kStage = kRowMaxCin / 16;  // 16-byte vectors of the next tile a thread holds

typedef uint32_t u4v __attribute__((ext_vector_type(4), aligned(4)));
using ConstU4 = __attribute__((address_space(4))) const u4v;
typedef unsigned int vu4 __attribute__((vector_size(16)));

// V columns a lane: 4 / V lanes a unit, tiles of up to 16 V units.  SPLIT: the
// plan has rows in two pieces (a variant of its own: the test at each row's end
// costs 128 -> 128 @ 56 x 56, batch 64, 2 us of 62).
template <int V, bool SPLIT>
__global__ void __launch_bounds__(1024) strip_rows_kernel(SArgs a) {
    constexpr int LPU = 4 / V;
    constexpr int TU = 64 / LPU;  // units of a row of lanes
    typedef float fv __attribute__((ext_vector_type(V)));
    typedef unsigned int vv __attribute__((vector_size(4 * V)));
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = static_cast<int>(blockDim.x) >> 6;
    // Workgroup b is number b / nxcd of its XCD and takes one tile a round,
    // neighbouring workgroups of an XCD neighbouring tiles (they share lines of
    // X and Y); then a part of the rows of one of the tiles left over, if any.
    const int32_t per = static_cast<int32_t>(gridDim.x) / a.nxcd;  // workgroups of an XCD
    const int32_t xcd = static_cast<int32_t>(blockIdx.x) % a.nxcd, local = static_cast<int32_t>(blockIdx.x) / a.nxcd;
    const int32_t slot = xcd * per + local;
    const int32_t items = a.rounds + (slot < a.rest * a.parts ? 1 : 0);
    if (items == 0)
        return;
    auto tile_of = [&](int32_t it) __attribute__((always_inline)) {
        return it < a.rounds ? (xcd * a.rounds + it) * per + local
                             : a.rounds * static_cast<int32_t>(gridDim.x) + slot / a.parts;
    };
    // the first column of unit u of an item's tile: its image (from the tile's
    // first, n0) and position; none past the last
    int32_t n0 = 0, im = 0, p = 0;
    auto unit = [&](int32_t it, int32_t u) __attribute__((always_inline)) {
        const int32_t g0 = tile_of(it) * a.tunits, g = g0 + u;
        n0 = g0 / a.units;
        const int32_t n = g / a.units;
        im = n - n0;
        p = min(4 * (g - n * a.units), a.hw - 4);
        return u < a.tunits && n < a.images;
    };
    // a tile's X: a wavefront takes LPU channels at a time, a lane one unit of
    // one of them
    const int su = lane % TU, sc = lane / TU;
    vu4 sv[kStage];
    auto fetch = [&](int32_t it) __attribute__((always_inline)) {
        const bool ok = unit(it, su);
        const int64_t xbase = static_cast<int64_t>(n0) * a.cin * a.hw;
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x + xbase, a.x_bytes - 4 * xbase);
        const int32_t at = 4 * ((im * a.cin + sc) * a.hw + p);
#pragma unroll
        for (int k = 0; k < kStage; ++k) {
            const int32_t c = LPU * (wave + k * waves);
            if (c < a.cin)
                sv[k] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok && c + sc < a.cin ? at : kOutOfRange, 4 * c * a.hw, 0);
        }
    };
    fetch(0);
    if (tid < a.tunits)  // the row of zeros that padding reads
        *reinterpret_cast<vu4 *>(lds + a.cin * a.row_bytes + 16 * tid) = vu4{0u, 0u, 0u, 0u};
    const ConstI *list = reinterpret_cast<const ConstI *>(reinterpret_cast<uintptr_t>(a.list));
    const uint32_t base = static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)lds)) +
                          4 * V * min(lane, a.tunits * LPU - 1);
    uint32_t row_bytes = static_cast<uint32_t>(a.row_bytes);
    asm("" : "+v"(row_bytes));  // a vector operand: one v_mad_u32_u24 per address, no scalar multiply
    constexpr int G = kGroupRecs;
    for (int32_t item = 0; item < items;) {
        __syncthreads();  // done with the tile before
        if (su < a.tunits) {
#pragma unroll
            for (int k = 0; k < kStage; ++k) {
                const int32_t c = LPU * (wave + k * waves) + sc;
                if (c < a.cin)
                    *reinterpret_cast<vu4 *>(lds + c * a.row_bytes + 16 * su) = sv[k];
            }
        }
        // this wavefront's lists of the item
        const int32_t parts = item < a.rounds ? 1 : a.parts;
        const int32_t mine = kRowLists / waves / parts;
        const int32_t l0 = wave * (kRowLists / waves) + slot % parts * mine;
        const int32_t g0 = list[2 * l0 + 1];
        int32_t rows = list[2 * (l0 + mine)] - list[2 * l0];
        // group g: 4 channels (words 8 g ..), 4 weights (8 g + 4 ..)
        const ConstU4 *ent = reinterpret_cast<const ConstU4 *>(reinterpret_cast<uintptr_t>(a.ent)) + 2 * g0;
        const ConstU4 *desc = reinterpret_cast<const ConstU4 *>(reinterpret_cast<uintptr_t>(a.desc)) + list[2 * l0];
        u4v oa = ent[0], wa = ent[1], ob = ent[2], wb;
        u4v d = desc[0];
        const bool ok = unit(item, lane / LPU);
        const int64_t ybase = static_cast<int64_t>(n0) * a.cout * a.hw;
        const __amdgpu_buffer_rsrc_t ry = make_rsrc(a.y + ybase, a.y_bytes - 4 * ybase);
        const int32_t yo = ok ? 4 * (im * a.cout * a.hw + p + lane % LPU * V) : kOutOfRange;
        __syncthreads();  // the tile is in LDS
        if (++item < items)
            fetch(item);
        if (rows > 0) {
            fv xa[G], xb[G];
            fv acc = {}, first = {};
            int32_t left = static_cast<int32_t>(d[1]);
            auto read = [&](const u4v &o, fv(&x)[G]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < G; ++j)
                    x[j] = *reinterpret_cast<const __attribute__((address_space(3))) fv *>(
                        static_cast<uintptr_t>(__umul24(o[j], row_bytes) + base));
            };
            read(oa, xa);
            // Scalar loads and LDS reads share one counter and scalar loads
            // return out of order, so every wait is for all of them: one wait
            // per group, after which the next group's X (its channels are
            // here), its weights and the channels of the group after it are
            // requested; the group's own products follow meanwhile.  Returns
            // whether the wavefront's last row is done.
            auto group = [&](const fv(&x)[G], const u4v &w, fv(&xn)[G], const u4v &on, u4v &wn, u4v &of,
                             int at) __attribute__((always_inline)) {
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
                __builtin_amdgcn_sched_barrier(0);
                read(on, xn);
                wn = ent[at + 3];
                of = ent[at + 4];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < G; ++j)
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        acc[e] = __builtin_fmaf(__uint_as_float(w[j]), x[j][e], acc[e]);
                if (--left == 0) {
                    if (SPLIT && d[3] == 1) {  // the even weights of a split row: its odd ones follow
                        first = acc;
                    } else {
                        if (SPLIT && d[3] == 2)
                            acc = first + acc;
                        const float bias = __uint_as_float(d[2]);
                        vv o;
#pragma unroll
                        for (int e = 0; e < V; ++e)
                            o[e] = __float_as_uint(__builtin_amdgcn_fmed3f(acc[e] + bias, a.lo, a.hi));
                        const int32_t so = static_cast<int32_t>(d[0]) * a.hw * 4;
                        if constexpr (V == 4)
                            __builtin_amdgcn_raw_buffer_store_b128(o, ry, yo, so, 0);
                        else
                            __builtin_amdgcn_raw_buffer_store_b64(o, ry, yo, so, 0);
                    }
                    acc = fv{};
                    ++desc;
                    d = *desc;
                    left = static_cast<int32_t>(d[1]);
                    return --rows == 0;
                }
                return false;
            };
            for (;;) {
                if (group(xa, wa, xb, ob, wb, oa, 0))
                    break;
                if (group(xb, wb, xa, oa, wa, ob, 2))
                    break;
                ent += 4;
            }
        }
    }
}

}  // namespace

// Both sides in microseconds, from a sweep of 1 to 32 images of 12 layers
// (cin 24 .. 1280, 70 .. 95% sparse, 1 x 1 and 1 x 4): this kernel takes 2.3 plus
// the longest row's chain of loads, or the wavefronts' work where that is more;
// the kernels that stage X in LDS take about 4 and grow with the channels they
// stage and the length of the rows that their wavefronts walk together (less
// with few rows), those for wide inputs 13.  512 -> 512 @ 14 x 14: one image 6.7
// against 13.7, four 8.5 against 14.4, eight 13.4 against 14.9; 32 -> 64 @ 56 x
// 56: one image 3.3 against 5.1, four 4.5 against 5.8, eight 6.2 against 6.2.
// Every output channel reads X again, from L2 while it fits there: past 6 MB of X
// a wavefront's reads take longer, up to 2.3 times from 14 MB (512 -> 64 @ 28 x
// 28, 11 images: 16.7 against 9.0), and past 4 MB the chain of the longest row up
// to 1.5 times (940 -> 128 @ 10 x 10, 16 images: 14.4 against 8.8).  Of 2500 random
// runs taken here 16 are slower than on the other kernel by more than 5%, up to 1.6
// times; without the two factors 35, up to 1.95.
bool rows_pay(const DevicePlan &p, int64_t images, int64_t hw) {
    if (!p.rows || hw < 4)
        return false;
    const int64_t units = images * ((hw + 3) / 4);
    if (units > (int64_t(1) << 20))
        return false;
    const double mean = static_cast<double>(p.nnz) / p.cout;
    const double waves = static_cast<double>((units + 63) / 64) * p.cout;
    const double x_mb = 16e-6 * static_cast<double>(units) * p.cin;
    const double read = 0.053 * std::min(2.3, std::max(1.0, x_mb / 6.0));
    const double chain = 0.062 * std::min(1.5, std::max(1.0, x_mb / 4.0));
    const double here = 2.3 + std::max(chain * p.max_row, waves * (0.5 + read * mean) * 1e-3);
    double there = p.k == 4 ? 4.0 + 0.008 * p.cin
                            : 4.0 + 0.009 * p.cin + 0.1 * mean * std::min(1.0, p.cout / 128.0);
    if (p.kernel == KERNEL_DIRECT)
        there = 13.0;
    return here < there;
}

namespace {

// How a run is cut into tiles (SArgs), on one of two forms: 64 units, 4 columns
// a lane, by two workgroups of 8 wavefronts a compute unit while two tiles fit
// in its LDS; past that 32 units, 2 columns a lane, by two of 8, or (wide) 64
// units, 4 columns a lane, by one of 16.
struct StripRows {
    int v;
    int32_t waves, tunits, slots, rounds, rest, parts;
    double us;  // estimated time
};

// The estimate: a wavefront's groups of 4 weights (at least the longest row's) at
// 0.148 us (0.211 by 16 wavefronts) per 100, times its tiles, plus staging and
// traffic.  Against 5000 random layers of 8 .. 160 channels, 8 .. 1280 outputs,
// 50 .. 98% sparse, on 256 .. 100000 units: within 10% (one sigma).
StripRows strip_rows_form(const DevicePlan &p, int64_t all, bool wide) {
    const int32_t cus = std::max(p.num_cus, 8);
    const int32_t half = static_cast<int32_t>(kMaxLdsBytes / 2 / (16 * (p.cin + 1)));
    StripRows s;
    s.v = half >= 64 || wide ? 4 : 2;
    s.waves = wide ? 16 : 8;
    s.tunits = wide ? 64 : std::min(16 * s.v, half);
    const int64_t round = 64 * static_cast<int64_t>(cus);  // units of one round of the largest tiles
    if (wide && all > 3 * round) {
        // few whole rounds: the same number of units to every workgroup (128 ->
        // 128 @ 56 x 56, batch 64: 64.2 us against 65.6 with a remainder)
        const int64_t n = (all + round - 1) / round * (cus / 8 * 8);
        s.tunits = static_cast<int32_t>(std::min<int64_t>(64, (all + n - 1) / n));
    }
    s.slots = (s.waves == 8 ? 2 : 1) * cus / 8 * 8;
    const int64_t tiles = (all + s.tunits - 1) / s.tunits;
    s.rounds = static_cast<int32_t>(tiles / s.slots);
    s.rest = static_cast<int32_t>(tiles - static_cast<int64_t>(s.rounds) * s.slots);
    s.parts = 1;
    while (2 * s.parts <= kRowLists / s.waves && static_cast<int64_t>(s.rest) * 2 * s.parts <= s.slots)
        s.parts *= 2;
    const double turns = s.rounds + (s.rest ? 1.0 / s.parts : 0.0);
    const double groups = std::max<double>(static_cast<double>(p.groups) / s.waves, p.max_row / 4.0);
    const double mb = 16e-6 * static_cast<double>(all) * (p.cin + p.cout);
    s.us = wide ? 4.8 + 0.211 * turns * groups + 0.02 * turns * p.cin + 0.08 * mb
                : 4.5 + 0.148 * turns * groups + (s.rounds ? 0.01 * turns * p.cin : 0.0) + 0.11 * mb;
    return s;
}

// The faster form.  Over 80 .. 159 channels the wide one wins with the tiles and
// the weights to spread over it (128 -> 256 @ 28 x 28, batch 64: 28 us against 33;
// 96 -> 576 @ 14 x 14, batch 128: 26 against 35; 144 -> 24 @ 56 x 56, batch 128: 80
// against 67, whose wavefronts wait for the longest row); the estimates pick the
// slower one by more than 5% on 5% of the layers above.
StripRows strip_rows_shape(const DevicePlan &p, int64_t all) {
    const StripRows a = strip_rows_form(p, all, false);
    if (a.v == 4 || p.cin >= 160)  // (the wide form's tile and its row of zeros fill the LDS up to 159 channels)
        return a;
    const StripRows b = strip_rows_form(p, all, true);
    return b.us < a.us ? b : a;
}

// The estimated time of the run on `other`, the kernel it takes otherwise, over
// the same layers: within 14 to 18% (one sigma), 24% on the element paths (hw not a
// multiple of 4) of blocked weights.
double other_us(const DevicePlan &p, int64_t images, int64_t hw, int32_t other) {
    const double units = static_cast<double>(images) * ((hw + 3) / 4);
    const double x = 4e-6 * images * hw * p.cin, y = 4e-6 * images * hw * p.cout;  // MB
    const bool vec = hw % 4 == 0;
    if (other == 3)  // register-indexed
        return 1.9 + 0.157e-6 * units * p.nnz + 0.339 * x + 0.155 * y + 0.28 * p.max_row;
    if (other == 4)  // lockstep, 1 x 4 blocks
        return vec ? 4.0 + 0.076e-6 * units * p.nnz + 0.594 * x + 0.128 * y + 0.0285 * p.max_row
                   : 7.2 + 0.0215e-6 * units * p.nnz + 1.69 * x + 0.258 * y + 0.0412 * p.max_row;
    // LDS strip: the longest wavefront's slots times the vectors of a lane, per
    // tile; tiles left after whole rounds are shared as its launch shares them
    const int64_t cus = std::max(p.num_cus, 8);
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(kMaxLdsBytes / std::max(p.lds_bytes, 1), 32 / p.waves));
    const int64_t tiles = (images * hw + p.tile_cols - 1) / p.tile_cols, slots = cus * per_cu;
    const int64_t rest = tiles % slots;
    int64_t parts = 1;
    while (rest && 2 * parts <= p.max_parts && 2 * parts <= slots / 8 / ((rest + 7) / 8))
        parts *= 2;
    const double turns = static_cast<double>(tiles / slots) + (rest ? 1.0 / parts : 0.0);
    const double work = turns * static_cast<double>(p.max_wave_cost) * 16 / p.group_lanes;
    if (p.k == 1)
        return vec ? 4.5 + 0.0593 * work + 0.161 * (x + y) + 0.0009 * p.cin
                   : 5.7 + 0.040 * work + 0.109 * x + 0.635 * y + 0.0116 * p.cin;
    return vec ? 4.6 + 0.0526 * work + 0.085 * x + 0.214 * y + 0.0059 * p.cin
               : 4.85 + 0.100 * work + 0.767 * y + 0.0212 * p.cin;
}

}  // namespace

// Taken where its estimate is below the other kernel's, by up to a fifth above on
// planes that are not a multiple of 4, which cost the others element accesses
// and this one nothing (100 -> 1000 @ 13 x 13, batch 8: 14.9 against 11.2; their
// estimate is the rougher one).  It needs tiles for the card: about 8192 units
// (96 -> 96 @ 20 x 20: 3200 units 6.2 against 6.9, 12800 units 20.7 against 13.8),
// fewer where many rows share a tile (48 -> 512 @ 7 x 7, batch 256: 27.6 against
// 11.9; 24 -> 144 @ 56 x 56, batch 8: 12.6 against 8.5).  Where the estimates turn it
// down: long rows, whose weights cost this kernel as much LDS bandwidth and more
// issue (144 -> 1024 @ 28 x 28, batch 24, 80% sparse: 40 against 62; 160 -> 768,
// 1 x 4, half dense, batch 12: 25 against 77).  Of 3500 random runs 2% are slower
// than on the other kernel by more than 5% (the worst 1.5 times); by a rule on
// sizes alone it was 7% (2.8 times), and half of those with 80 .. 160 channels,
// 256 or more outputs and 1024 .. 8192 units.
bool strip_rows_pay(const DevicePlan &p, int64_t images, int64_t hw, int64_t image_bytes, int32_t other) {
    if (p.groups == 0 || hw < 4)
        return false;
    const int64_t units = (hw + 3) / 4, all = images * units;
    // the images of a tile must span less than 2^31 bytes
    if ((63 / units + 2) * image_bytes >= (int64_t(1) << 31) - 16 || all > (int64_t(1) << 29))
        return false;
    const int64_t least = hw % 4 != 0                       ? 256
                          : p.cout >= 256                   ? 1024
                          : p.cin <= 64 && p.cout >= 128 ? 4096
                                                            : 8192;
    return all >= least &&
           strip_rows_shape(p, all).us < (hw % 4 != 0 ? 1.2 : 1.0) * other_us(p, images, hw, other);
}

hipError_t launch_rows(const DevicePlan &p, const float *x, float *y, int32_t m, int32_t hw, hipStream_t stream) {
    RArgs a;
    a.x = x;
    a.y = y;
    a.bias = p.tbias;
    a.row_ptr = p.trow_ptr;
    a.ent = p.tent;
    a.cin = p.cin;
    a.cout = p.cout;
    a.hw = hw;
    a.units = (hw + 3) / 4;
    a.all = m / hw * a.units;
    a.blocks = (a.all + 63) / 64;
    a.lo = p.act == 0 ? -__builtin_huge_valf() : 0.0f;
    a.hi = p.act == 2 ? 6.0f : __builtin_huge_valf();
    const int64_t items = static_cast<int64_t>(a.blocks) * p.cout;
    hipLaunchKernelGGL(p.splits ? rows_kernel<true> : rows_kernel<false>, dim3(static_cast<unsigned>((items + kRowWaves - 1) / kRowWaves)),
                       dim3(64 * kRowWaves), 0, stream, a);
    return hipGetLastError();
}

hipError_t prepare_strip_rows(const DevicePlan &) {
    static std::atomic<uint64_t> done{0};  // a bit a device: the attribute stays with the function
    int dev = 0;
    if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess)
        return e;
    const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
    if (done.load() & bit)
        return hipSuccess;
    for (const void *k : {reinterpret_cast<const void *>(strip_rows_kernel<2, false>),
                          reinterpret_cast<const void *>(strip_rows_kernel<4, false>),
                          reinterpret_cast<const void *>(strip_rows_kernel<2, true>),
                          reinterpret_cast<const void *>(strip_rows_kernel<4, true>)}) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
        if (e != hipSuccess)
            return e;
    }
    done.fetch_or(bit);
    return hipSuccess;
}

hipError_t launch_strip_rows(const DevicePlan &p, const float *x, float *y, int32_t m, int32_t hw, int64_t x_bytes,
                             int64_t y_bytes, hipStream_t stream) {
    SArgs a;
    a.x = x;
    a.y = y;
    a.ent = p.gent;
    a.desc = p.gdesc;
    a.list = p.glist;
    a.cin = p.cin;
    a.cout = p.cout;
    a.hw = hw;
    a.images = m / hw;
    a.units = (hw + 3) / 4;
    a.x_bytes = x_bytes;
    a.y_bytes = y_bytes;
    a.lo = p.act == 0 ? -__builtin_huge_valf() : 0.0f;
    a.hi = p.act == 2 ? 6.0f : __builtin_huge_valf();
    const StripRows s = strip_rows_shape(p, static_cast<int64_t>(a.images) * a.units);
    a.tunits = s.tunits;
    a.row_bytes = 16 * a.tunits;
    a.rounds = s.rounds;
    a.rest = s.rest;
    a.parts = s.parts;
    // (a pass of the workgroup stages 4 / v * waves channels)
    static_assert(kRowMaxCin <= 16 * kStage && kMaxLdsBytes / 2 / (16 * 64) - 1 <= 8 * kStage, "staged in kStage passes");
    a.nxcd = 8;
    const int64_t grid = a.rounds > 0 ? s.slots : (static_cast<int64_t>(a.rest) * a.parts + 7) / 8 * 8;
    const auto kernel = p.splits ? (s.v == 4 ? strip_rows_kernel<4, true> : strip_rows_kernel<2, true>)
                                 : (s.v == 4 ? strip_rows_kernel<4, false> : strip_rows_kernel<2, false>);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(grid)),
                       dim3(64 * s.waves), (p.cin + 1) * a.row_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace spconv
