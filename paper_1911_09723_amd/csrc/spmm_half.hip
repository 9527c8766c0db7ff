// Matrix-core kernel for fp16 storage: Y = act(W X + b) with X, Y and W in
// fp16 and fp32 accumulation, whole row groups of W as dense 16 x 32
// fragments (format in planner.hpp, "Half kernel").
//
// Why dense fragments.  A column costs (cin + cout) * 2 bytes of HBM traffic
// and, multiplied out, cin * cout multiply-adds.  The fp16 16x16x32
// instruction does 8192 of them in 7.6 ns per SIMD (1.1e15 a second on the card), so
// up to cin * cout / (cin + cout) = 360 even the dense product takes less
// time than the traffic at 6.2 TB/s; walking only the stored 10% of the
// weights costs an LDS read per 4 stored weights.
// Products of fp16 values are exact in fp32, and the instruction's sum of 32
// of them has a smaller error than a chain of 32 fused multiply-adds (4.1e-8
// against 8.9e-8 rms).
//
// Work layout.  A tile is whole image planes, or an even piece of one plane
// that is too long: what bounds these layers is writing Y, and the write rate
// depends on who writes a 128-byte line.  Written by tiles of 128 columns that
// run across image borders (14 x 14 planes: 256-byte pieces of a 392-byte
// row), 135 MB take 44.8 us; by whole planes, whose rows follow each other in
// memory, 30.5 us (7 x 7, 58 MB: 24.9 against 11.6 us).  Columns are taken in
// units of 4 neighbours of one plane (the last unit of a plane may be short),
// 16 units a part.  A workgroup stages X for its tile, all input channels, in
// LDS in the order the instruction reads it: a lane loads 8 channels x 4
// columns (8 bytes each), transposes them in registers (byte permutes) to 4
// columns x 8 channels and writes 4 vectors of 16 bytes.  Column j of unit v
// is column v of operand j, so the results of a part's 4 operands leave a
// lane with 4 neighbouring columns per row and one 8-byte store.  After the
// barrier each wavefront walks row tiles: per 32 input channels one weight
// fragment (16 bytes a lane, from L2) and 4 operands a part from LDS.
//
// Measured (kernel time over back-to-back launches, batch 512, 90% 1 x 4 blocks; the
// automatic choice before, the bytes at 6.2 TB/s): 112 -> 672 @ 14 x 14 82 -> 41 us
// (25), 320 -> 1280 @ 7 x 7 78 -> 46 (13), 192 -> 1152 @ 7 x 7 66 -> 32 (11), 80 ->
// 480 @ 14 x 14 63 -> 26 (18), 40 -> 240 @ 28 x 28 112 -> 54 (36).  What is left
// over the bytes: staging, products and stores of a workgroup follow each other,
// and a run has too few workgroups per compute unit to hide all of one behind the
// others.
//
// A dense product reads X where the sparse one does not, and 0 * inf is NaN.
// Staging therefore checks every value: a workgroup that saw an infinity or a
// NaN sums the columns that hold one again, over the stored weights only, in
// ascending channel, from the same LDS copy.  (Columns do not mix in the
// products: the others keep their bits, whatever shares their tile.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include "launch.hpp"

namespace spconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

using Rsrc = __amdgpu_buffer_rsrc_t;

// An offset past every buffer resource: loads return zeros, stores are dropped.
constexpr int32_t kOutOfRange = static_cast<int32_t>(0x80000000u);
constexpr int64_t kMaxRecords = 0x7ffffff0;
constexpr int32_t kXcds = 8;

__device__ __forceinline__ Rsrc make_rsrc(const void *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), static_cast<short>(0),
                                             static_cast<int>(bytes < kMaxRecords ? bytes : kMaxRecords), 0x00020000);
}

struct HArgs {
    const _Float16 *x;
    _Float16 *y;
    const u4 *frag;          // weight fragments, 64 lanes x 16 bytes each
    const float *bias;       // every output channel, padded to whole row groups
    const int32_t *row_ptr;  // stored weights by output channel (the non-finite path)
    const u2 *ent;           // channel, fp32 weight bits
    int32_t cin, cout, hw, images;
    int32_t kb, rgroups;     // blocks of 32 input channels, groups of RT row tiles (16 output channels each)
    int32_t units;           // 4-column units of a plane
    int32_t tunits, tiles;   // units of a tile; tiles
    int32_t ipt, tpi;        // images per tile (tpi = 1), or tiles per image (ipt = 1)
    int32_t parts;           // 16-unit parts of a tile (a multiple of those taken at a time)
    int32_t chunks;          // wavefronts that share a row tile, each with its own parts
    int32_t rsplit;          // workgroups sharing one tile's row groups
    int32_t nxcd;            // the grid is a multiple of it
    int64_t x_bytes, y_bytes;
    float lo, hi;            // the activation as a clamp
};

// A unit's columns: element offsets of the first one in channel 0 of X and of
// Y from the tile's first image, how many there are (0: none), and a bit for
// each that holds an infinity or a NaN (after the products, where there are any).
struct Unit {
    int32_t xo, yo, k, mask;
};

__device__ __forceinline__ uint64_t load8(const _Float16 *p) {
    uint64_t v;
    __builtin_memcpy(&v, p, 8);
    return v;
}

// LDS: the fragments of X (part p, block b, operand j at 1 KB * (4 (p * kb + b) + j)),
// the units, the non-finite flag.
// VEC: H*W is a multiple of 4 and x and y are 8-byte aligned, so units are whole and aligned.
// KB: the plan's blocks of 32 input channels, up to kHalfRing; 0: any number.
constexpr int kHalfRing = 10;

template <bool VEC, int NH, int RT, int KB>
__global__ void __launch_bounds__(1024) half_kernel(HArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = static_cast<int>(blockDim.x) >> 6;
    const int n = lane & 15, q = lane >> 4;
    // neighbouring work items on one XCD: they share 128-byte lines of X and Y,
    // and the workgroups of one tile share its X
    const int32_t per = static_cast<int32_t>(gridDim.x) / a.nxcd;
    const int32_t item = static_cast<int32_t>(blockIdx.x) % a.nxcd * per + static_cast<int32_t>(blockIdx.x) / a.nxcd;
    const int32_t ct = item / a.rsplit, rs = item - ct * a.rsplit;
    if (ct >= a.tiles)
        return;
    Unit *tab = reinterpret_cast<Unit *>(lds + a.parts * a.kb * 4096);
    int32_t *bad = reinterpret_cast<int32_t *>(tab + 16 * a.parts);
    const int32_t n0 = a.tpi > 1 ? ct / a.tpi : ct * a.ipt;
    for (int i = tid; i < 16 * a.parts; i += blockDim.x) {
        const int32_t im = a.tpi > 1 ? 0 : i / a.units;  // from n0
        const int32_t u = a.tpi > 1 ? (ct - n0 * a.tpi) * a.tunits + i : i - im * a.units;
        const bool ok = i < a.tunits && u < a.units && n0 + im < a.images;
        tab[i] = Unit{im * a.cin * a.hw + 4 * u, im * a.cout * a.hw + 4 * u, ok ? min(4, a.hw - 4 * u) : 0, 0};
    }
    if (tid == 0)
        *bad = 0;
    __syncthreads();

    const int32_t chunk = wave % a.chunks;
    const int32_t stride = waves / a.chunks * a.rsplit;
    int32_t rg = rs * (waves / a.chunks) + wave / a.chunks;
    // With KB known the fragments of a whole row group sit in registers; each
    // is loaded again for the next group as soon as its last part is done, so
    // no weight load follows the group's stores (the memory counter completes
    // in order: such a load would wait for the stores).  The first group's
    // are on their way while X is staged, where the registers allow it.
    const int32_t tstep = a.kb * 64;  // fragments of one 16-row tile
    const u4 *wp = a.frag + static_cast<int64_t>(RT * min(rg, a.rgroups - 1)) * tstep + lane;
    constexpr int AN = KB ? KB : 1;
    constexpr bool kEarly = NH == 1;
    u4 an[AN][RT];
    auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < AN; ++kb)
#pragma unroll
            for (int t = 0; t < RT; ++t)
                an[kb][t] = wp[kb * 64 + t * tstep];
    };
    if constexpr (kEarly)
        weights();

    // ---- stage X: a wavefront takes (part, block) pairs, kBatch of them in
    // flight at once (the latency of memory, not its rate, is what staging
    // waits for) ----
    const int64_t xbase = static_cast<int64_t>(n0) * a.cin * a.hw;
    {
        const _Float16 *xt = a.x + xbase;
        const Rsrc rx = make_rsrc(xt, a.x_bytes - 2 * xbase);
        constexpr int kBatch = VEC ? 4 : 3;
        us2 top = {0, 0};
        const int blocks = a.parts * a.kb;
        for (int i0 = wave; i0 < blocks; i0 += kBatch * waves) {
            uint32_t d[kBatch][8][2];
            int32_t k[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int it = min(i0 + b * waves, blocks - 1);
                const int part = it / a.kb, kb = it - part * a.kb;
                const Unit u = tab[16 * part + n];
                k[b] = u.k;
                const int32_t back = VEC || a.hw < 4 ? 0 : 4 - u.k;  // a short unit is read with the columns before it
                const int32_t at = u.xo + (32 * kb + 8 * q) * a.hw - back;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool in = u.k > 0 && 32 * kb + 8 * q + i < a.cin;
                    if constexpr (VEC) {
                        const auto t =
                            __builtin_amdgcn_raw_buffer_load_b64(rx, in ? 2 * (at + i * a.hw) : kOutOfRange, 0, 0);
                        d[b][i][0] = t[0];
                        d[b][i][1] = t[1];
                    } else {
                        uint64_t w = 0;
                        if (a.hw >= 4) {
                            // no branch around a load: what lies outside reads the tile's first elements
                            w = load8(xt + (in ? at + i * a.hw : 0));
                        } else if (in) {
                            for (int e = 0; e < u.k; ++e)
                                w |= static_cast<uint64_t>(__builtin_bit_cast(uint16_t, xt[at + i * a.hw + e])) << (16 * e);
                        }
                        d[b][i][0] = static_cast<uint32_t>(w);
                        d[b][i][1] = static_cast<uint32_t>(w >> 32);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int it = i0 + b * waves;
                if (it >= blocks)
                    break;
                const int part = it / a.kb, kb = it - part * a.kb;
                if constexpr (!VEC) {
                    const int32_t back = a.hw < 4 ? 0 : 4 - k[b];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bool in = k[b] > 0 && 32 * kb + 8 * q + i < a.cin;
                        const uint64_t w = (d[b][i][0] | static_cast<uint64_t>(d[b][i][1]) << 32) >> (16 * (back & 3));
                        d[b][i][0] = in ? static_cast<uint32_t>(w) : 0;
                        d[b][i][1] = in ? static_cast<uint32_t>(w >> 32) : 0;
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, d[b][i][0] & 0x7fff7fffu));
                    top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, d[b][i][1] & 0x7fff7fffu));
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u4 o;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        o[w] = __builtin_amdgcn_perm(d[b][2 * w + 1][j >> 1], d[b][2 * w][j >> 1],
                                                     j & 1 ? 0x07060302u : 0x05040100u);
                    *reinterpret_cast<u4 *>(lds + (4 * it + j) * 1024 + lane * 16) = o;
                }
            }
        }
        if (top.x >= 0x7c00 || top.y >= 0x7c00)
            *bad = 1;
    }
    __syncthreads();

    const int64_t ybase = static_cast<int64_t>(n0) * a.cout * a.hw;

    // ---- row groups ----
    const int32_t redo = __builtin_amdgcn_readfirstlane(*bad);
    if (rg >= a.rgroups && !redo)
        return;
    const Rsrc ry = make_rsrc(a.y + ybase, a.y_bytes - 2 * ybase);
    if constexpr (!kEarly)
        weights();
    for (; rg < a.rgroups; rg += stride) {
        const bool more = rg + stride < a.rgroups;
        const u4 *wn = wp + (more ? static_cast<int64_t>(RT * stride) * tstep : 0);  // the next group
        for (int pp = chunk * NH; pp < a.parts; pp += NH * a.chunks) {
            f4 acc[RT][4 * NH];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int j = 0; j < 4 * NH; ++j)
                    acc[t][j] = f4{0.f, 0.f, 0.f, 0.f};
            const unsigned char *bl = lds + pp * a.kb * 4096 + lane * 16;
            auto block = [&](int kb, const u4(&ac)[RT]) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    u4 b[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        b[j] = *reinterpret_cast<const u4 *>(bl + (h * a.kb + kb) * 4096 + j * 1024);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int t = 0; t < RT; ++t)
                            acc[t][4 * h + j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                __builtin_bit_cast(h8, ac[t]), __builtin_bit_cast(h8, b[j]), acc[t][4 * h + j], 0, 0, 0);
                }
            };
            const bool last = pp + NH * a.chunks >= a.parts;
            if constexpr (KB > 0) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    block(kb, an[kb]);
                    if (last) {
#pragma unroll
                        for (int t = 0; t < RT; ++t)
                            an[kb][t] = wn[kb * 64 + t * tstep];
                    }
                }
            } else {
                for (int kb = 0; kb < a.kb; ++kb) {
                    u4 ac[RT];
                    const u4 *ws = kb + 1 < a.kb ? wp + (kb + 1) * 64 : last ? wn : wp;  // the next step's
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        ac[t] = an[0][t];
                        an[0][t] = ws[t * tstep];
                    }
                    block(kb, ac);
                }
            }
            Unit u[NH];
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                u[h] = tab[16 * (pp + h) + n];
                u[h].yo += 4 * q * a.hw;
            }
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const int32_t row0 = 16 * (RT * rg + t);
                const f4 bz = *reinterpret_cast<const f4 *>(a.bias + row0 + 4 * q);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = row0 + 4 * q + r < a.cout;
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        uint32_t o[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const float v0 = __builtin_amdgcn_fmed3f(acc[t][4 * h + 2 * e][r] + bz[r], a.lo, a.hi);
                            const float v1 = __builtin_amdgcn_fmed3f(acc[t][4 * h + 2 * e + 1][r] + bz[r], a.lo, a.hi);
                            o[e] = __builtin_bit_cast(uint16_t, static_cast<_Float16>(v0)) |
                                   static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<_Float16>(v1))) << 16;
                        }
                        // (a row past the last is dropped by its lanes' offsets, which are
                        // checked against what the scalar offset leaves of the resource:
                        // that one stays inside it)
                        const int32_t so = 2 * min(row0 + r, a.cout - 1) * a.hw;
                        if constexpr (VEC) {
                            typedef unsigned int vu2 __attribute__((vector_size(8)));
                            __builtin_amdgcn_raw_buffer_store_b64(vu2{o[0], o[1]}, ry,
                                                                  in && u[h].k > 0 ? 2 * u[h].yo : kOutOfRange, so, 0);
                        } else if (in && u[h].k == 4) {
                            __builtin_memcpy(reinterpret_cast<char *>(a.y + ybase) + so + 2 * u[h].yo, o, 8);
                        } else if (in) {
#pragma unroll
                            for (int i = 0; i < 3; ++i)
                                if (i < u[h].k)
                                    a.y[ybase + u[h].yo + i + static_cast<int64_t>(row0 + r) * a.hw] = __builtin_bit_cast(
                                        _Float16, static_cast<uint16_t>(o[i >> 1] >> (16 * (i & 1))));
                        }
                    }
                }
            }
        }
        wp = wn;
    }

    if (!redo)
        return;
    // The columns with an infinity or a NaN once more, over the stored weights
    // only: neither may reach the rows that do not read its channel.
    const int32_t columns = 64 * a.parts;
    // (the lane and the shares anew: kept through the products they cost registers there)
    const int32_t l = static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
    int32_t wv = wave;
    asm("" : "+s"(wv));
    auto column = [&](int32_t c) { return lds + ((c >> 6) * a.kb * 4 + (c & 3)) * 1024 + ((c & 63) >> 2) * 16; };
    for (int32_t c = 64 * wv + l; c < columns; c += 64 * waves) {
        const unsigned char *src = column(c);
        bool finite = true;
        for (int32_t k = 0; k < 4 * a.kb; ++k) {  // 8 channels each
            const u4 v = *reinterpret_cast<const u4 *>(src + (k >> 2) * 4096 + (k & 3) * 256);
#pragma unroll
            for (int w = 0; w < 4; ++w)
                finite = finite && (v[w] & 0x7c00u) != 0x7c00u && (v[w] & 0x7c000000u) != 0x7c000000u;
        }
        if (!finite)
            atomicOr(&tab[c >> 2].mask, 1 << (c & 3));
    }
    __threadfence();  // the products' results are written before these
    __syncthreads();
    for (rg = rs * (waves / a.chunks) + wv / a.chunks; rg < a.rgroups; rg += stride)
        for (int32_t o = 64 * (wv % a.chunks) + l; o < 16 * RT * columns; o += 64 * a.chunks) {
            const int32_t row = 16 * RT * rg + o / columns, c = o % columns;
            const Unit u = tab[c >> 2];
            if (row >= a.cout || (c & 3) >= u.k || !(u.mask >> (c & 3) & 1))
                continue;
            const unsigned char *src = column(c);
            float s = 0.0f;
            for (int32_t t = a.row_ptr[row]; t < a.row_ptr[row + 1]; ++t) {
                const u2 en = a.ent[t];
                const int32_t ch = static_cast<int32_t>(en.x);
                const _Float16 xv =
                    *reinterpret_cast<const _Float16 *>(src + (ch >> 5) * 4096 + ((ch >> 3) & 3) * 256 + (ch & 7) * 2);
                s = __builtin_fmaf(__uint_as_float(en.y), static_cast<float>(xv), s);
            }
            a.y[ybase + u.yo + (c & 3) + static_cast<int64_t>(row) * a.hw] =
                static_cast<_Float16>(fminf(fmaxf(s + a.bias[row], a.lo), a.hi));
        }
}

typedef void (*HKernel)(HArgs);

// The kernel for nh parts at a time and kb blocks of input channels.  Up to
// kHalfRing blocks, one row tile at a time with its weights in registers
// (except the four parts of odd planes, whose units need the registers);
// past them two row tiles, the weights one step ahead.
template <bool VEC, int NH>
HKernel pick_kb(int kb) {
    switch (kb) {
    case 1: return half_kernel<VEC, NH, 1, 1>;
    case 2: return half_kernel<VEC, NH, 1, 2>;
    case 3: return half_kernel<VEC, NH, 1, 3>;
    case 4: return half_kernel<VEC, NH, 1, 4>;
    case 5: return half_kernel<VEC, NH, 1, 5>;
    case 6: return half_kernel<VEC, NH, 1, 6>;
    case 7: return half_kernel<VEC, NH, 1, 7>;
    case 8: return half_kernel<VEC, NH, 1, 8>;
    case 9: return half_kernel<VEC, NH, 1, 9>;
    default: return half_kernel<VEC, NH, 1, 10>;
    }
}

HKernel pick(bool vec, int nh, int kb) {
    if (kb > kHalfRing) {
        if (nh == 1)
            return vec ? half_kernel<true, 1, 2, 0> : half_kernel<false, 1, 2, 0>;
        return vec ? half_kernel<true, 2, 2, 0> : half_kernel<false, 2, 2, 0>;
    }
    if (nh == 1)
        return vec ? pick_kb<true, 1>(kb) : pick_kb<false, 1>(kb);
    if (nh == 4)
        return vec ? pick_kb<true, 4>(kb) : half_kernel<false, 4, 1, 0>;
    return vec ? pick_kb<true, 2>(kb) : pick_kb<false, 2>(kb);
}

int row_tiles(int kb) { return kb > kHalfRing ? 2 : 1; }

int32_t half_lds_bytes(int32_t kb, int32_t parts) { return parts * (kb * 4096 + 16 * 16) + 16; }

}  // namespace

hipError_t prepare_half(const DevicePlan &p) {
    for (int nh : {1, 2, 4})
        for (bool vec : {false, true}) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick(vec, nh, p.hkb)),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
            if (e != hipSuccess)
                return e;
        }
    return hipSuccess;
}

namespace {

// How a run is cut into tiles and workgroups.
struct HalfShape {
    int nh;                            // parts at a time
    int32_t units, chunks, ipt, tpi, tunits, parts, rgroups, rsplit, waves, lds;
    int64_t tiles;
    int64_t grid;
};

HalfShape half_shape(const DevicePlan &p, int64_t images, int64_t hw, int64_t image_bytes) {
    HalfShape s;
    const int32_t kb = p.hkb;
    s.units = static_cast<int32_t>((hw + 3) / 4);
    const int32_t cus = std::max(p.num_cus, 1);
    // Parts at a time and per tile.  Whole planes of up to 64 units are taken
    // four parts at a time, larger ones by 4 wavefronts with four parts each
    // where that fits in LDS (40 -> 240 @ 28 x 28, batch 512: 52 us against 70
    // in four pieces); two parts otherwise, one where LDS holds no more or the
    // run is too short to fill the card (few tiles, or few rows for a
    // workgroup's wavefronts to share).
    const int32_t row_tiles16 = (p.cout + 15) / 16;
    const int64_t units16 = images * ((s.units + 15) / 16);  // parts of the whole run
    s.nh = kb > 19 ? 1 : s.units > 32 && kb <= kHalfRing - 1 ? 4 : 2;
    if (row_tiles16 <= 4 && s.nh == 4 && kb > 1)
        s.nh = 2;
    if (units16 < 4 * cus && s.nh > 1)
        s.nh = units16 < cus ? 1 : 2;
    s.chunks = 1;
    if (s.nh == 4 && s.units > 64 && kb <= 2)
        s.chunks = s.units > 128 ? 4 : 2;
    const int32_t rt = row_tiles(kb);
    s.rgroups = (p.cout + 16 * rt - 1) / (16 * rt);
    const int32_t most = 16 * s.nh * s.chunks;  // units of a tile, at most
    if (s.units > most) {
        s.ipt = 1;
        s.tpi = (s.units + most - 1) / most;
        s.tunits = (s.units + s.tpi - 1) / s.tpi;
    } else {
        // (the images of a tile must span less than 2^31 bytes)
        s.tpi = 1;
        s.ipt = static_cast<int32_t>(std::min<int64_t>(most / s.units,
                                                       std::max<int64_t>(1, (int64_t(1) << 30) / image_bytes)));
        s.tunits = s.ipt * s.units;
    }
    s.parts = ((s.tunits + 15) / 16 + s.nh - 1) / s.nh * s.nh;
    s.tiles = s.tpi > 1 ? images * s.tpi : (images + s.ipt - 1) / s.ipt;
    s.lds = half_lds_bytes(kb, s.parts);
    // wavefronts: 16 a compute unit, in one workgroup where LDS or the number
    // of tiles leaves no second one (192 -> 1152 @ 7 x 7, batch 512, 256
    // tiles: 34 us against 44 with 8).  Short runs share each tile among
    // workgroups by row groups: of 8 wavefronts where a compute unit has at least
    // 4 row groups, else of 4 (with 2, the card is short of wavefronts: 155 ->
    // 1540 @ 1 x 1, 1931 images, 44 us against 24 with 8; over 2000 random runs of
    // fewer than 128 tiles 8% behind 4 and, by row groups, 4 to 85% behind 8; 16
    // are slower).  Fewer for few rows.
    s.waves = 2 * s.tiles < cus ? (s.lds > kMaxLdsBytes / 2 || s.tiles * s.rgroups >= 4 * cus ? 8 : 4)
              : s.lds > kMaxLdsBytes / 2 || s.tiles <= 3 * cus / 2 ? 16
                                                                   : 8;
    if (row_tiles16 <= 4 && kb > 1)
        s.waves = std::min(s.waves, 4);
    s.waves = std::max(s.waves, s.chunks);
    const int32_t rows = s.waves / s.chunks;  // row groups a workgroup works on at a time
    s.rsplit = static_cast<int32_t>(
        std::max<int64_t>(1, std::min<int64_t>((s.rgroups + rows - 1) / rows, 2 * cus / (2 * s.tiles))));
    s.grid = (s.tiles * s.rsplit + kXcds - 1) / kXcds * kXcds;
    return s;
}

}  // namespace

// Both sides from 5500 random runs (8 .. 1216 channels, 8 .. 1600 outputs, 50 .. 98%
// sparse, 1 to 2048 images), which are 2.5 times as fast here as on the others.
// The dense product and the staging cost the same however few weights are stored;
// the strip and direct-load kernels pay by the weight, little where they read
// whole 16-byte vectors (hw a multiple of 8).  There they win with fewer than 2
// stored weights an input channel (slower here in 35% of those runs, even on
// average), fewer than 4 past 320 channels (1077 -> 10 @ 56 x 56, 98% sparse, 26
// images: 98 us here against 9.7; 80% slower, by 1.8 times on average); elsewhere
// only past 640 channels with fewer than 0.7 (1002 -> 12 @ 7 x 7: 92
// against 49).  The lockstep kernel wins on planes of up to 4 columns, which fill
// a quarter of a unit or one operand of it, past 320 channels where the products
// count (477 -> 628 @ 2 x 2, 617 images: 16.8 against 9.0).  Of 5500 other runs 3%
// are slower here by more than 5%, up to 1.9 times (without this rule 5%, up to
// 10 times).
// The rule does not look at the number of images: the matrix instruction sums in
// another order, and an image's bits must not depend on its batch.
bool half_pays(const DevicePlan &p, int64_t hw, bool lockstep) {
    if (p.hkb == 0)
        return false;
    const double uses = static_cast<double>(p.nnz) / p.cin;
    if (lockstep)
        return hw > 4 || p.hkb <= 10 || static_cast<double>(p.cin) * p.cout < 90.0 * (p.cin + p.cout);
    return uses >= (hw % 8 == 0 ? (p.hkb > 10 ? 4.0 : 2.0) : p.hkb > 20 ? 0.7 : 0.0);
}

bool half_fits(const DevicePlan &p, int64_t images, int64_t hw, int64_t image_bytes) {
    const HalfShape s = half_shape(p, images, hw, image_bytes);
    return s.grid * 64 * s.waves < int64_t(1) << 32;
}

hipError_t launch_half(const DevicePlan &p, const void *x, void *y, int32_t m, int32_t hw, int32_t vec,
                       int64_t x_bytes, int64_t y_bytes, hipStream_t stream) {
    HArgs a;
    a.x = static_cast<const _Float16 *>(x);
    a.y = static_cast<_Float16 *>(y);
    a.frag = reinterpret_cast<const u4 *>(p.hfrag);
    a.bias = p.tbias;
    a.row_ptr = p.trow_ptr;
    a.ent = reinterpret_cast<const u2 *>(p.tent);
    a.cin = p.cin;
    a.cout = p.cout;
    a.hw = hw;
    a.images = m / hw;
    a.kb = p.hkb;
    a.x_bytes = x_bytes;
    a.y_bytes = y_bytes;
    a.lo = p.act == 0 ? -__builtin_huge_valf() : 0.0f;
    a.hi = p.act == 2 ? 6.0f : __builtin_huge_valf();
    const HalfShape s = half_shape(p, a.images, hw, std::max(x_bytes, y_bytes) / a.images);
    a.rgroups = s.rgroups;
    a.units = s.units;
    a.tunits = s.tunits;
    a.tiles = static_cast<int32_t>(s.tiles);
    a.ipt = s.ipt;
    a.tpi = s.tpi;
    a.parts = s.parts;
    a.chunks = s.chunks;
    a.rsplit = s.rsplit;
    a.nxcd = kXcds;
    hipLaunchKernelGGL(pick(vec != 0, s.nh, a.kb), dim3(static_cast<unsigned>(s.grid)), dim3(64 * s.waves), s.lds,
                       stream, a);
    return hipGetLastError();
}

}  // namespace spconv
