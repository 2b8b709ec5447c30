// Device helpers shared by the kernel sources of libhsgd (gfx950, wave64). Not installed.
#pragma once

#include <hip/hip_runtime.h>

#include "hsgd_internal.h"

namespace hsgd {
namespace {

// Two FP32 values -> BF16 bits (a in the low half), round to nearest even, a NaN kept as a
// quiet NaN: one v_cvt_pk_bf16_f32, checked over every FP32 bit pattern against the integer
// form (add 0x7fff and the bit above, shift, NaNs apart), whose compare and branch per value
// were a third of the instructions of a BF16 plane sweep (1008x756x32, 5 tilted views: 419 us
// a call with it, 367 us without at the time, 345 us since; the finest level transition of a 1920x1080x64 refine: 437
// and 353 us).
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return f32x2_to_bf16x2(f, 0.0f); }

// 64-bit masks by a bit index that differs by lane, in 32-bit halves. A 64-bit vector shift reads
// its amount as a register pair, and gives wrong bits where the amount is the last register of
// the wave's allocation: 8 to 17% of the results of v_lshlrev_b64, v_lshrrev_b64 and
// v_ashrrev_i64 (amount in v39 of 40 registers, v63 of 64, v95 of 96, v119 of 120, v127 of 128,
// v255 of 256; none in v125 of 128). The compiler does not avoid that register, so no kernel
// shifts 64 bits by a register; the build refuses one that does.
__device__ __forceinline__ uint64_t halves(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
// bit z (0..63)
__device__ __forceinline__ uint64_t lane_bit(unsigned z) {
    const uint32_t b = 1u << (z & 31u);
    return halves(z < 32u ? b : 0u, z < 32u ? 0u : b);
}
// the bits below z (0..64)
__device__ __forceinline__ uint64_t lane_bits_below(unsigned z) {
    const uint32_t b = (1u << (z & 31u)) - 1u;
    return halves(z < 32u ? b : ~0u, z < 32u ? 0u : z < 64u ? b : ~0u);
}
__device__ __forceinline__ bool has_lane_bit(uint64_t m, unsigned z) {
    uint32_t hi = (uint32_t)(m >> 32);
    asm("" : "+v"(hi));     // (the compiler makes a 64-bit shift of a choice of halves)
    return (((z < 32u ? (uint32_t)m : hi) >> (z & 31u)) & 1u) != 0u;
}

// What one lane wrote to LDS before this another lane of the wave reads after it (the LDS
// operations of a wave execute in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Raw (untyped, stride 0) buffer resource over one MPI row of n_bytes bytes: loads at
// offsets outside [0, n_bytes) return 0, which is the zero padding of a plane outside the
// image; n_bytes = 0 makes a whole row read as padding. Word 3 selects the 32-bit data
// format that untyped loads require on this architecture family.
constexpr int kBufWord3 = 4 << 15;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const char* row, int n_bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), (short)0, n_bytes, kBufWord3);
}

// ------------------------------------------------------------------------------------
// positions under a general homography, one row of pixels at a time
// ------------------------------------------------------------------------------------
// The homogeneous position of pixel x of a fixed row y: q_i = a_i x + b_i, the products of y
// taken once per row (the same FP64 operations in the same order as for a single pixel).
// A translation record is the map x + ix + fx, y + iy + fy.
struct RowMap {
    double a0, a1, a2, b0, b1, b2;
};
__device__ __forceinline__ RowMap row_map(const double* g, double yd) {
    return RowMap{g[0], g[3], g[6], __builtin_fma(g[1], yd, g[2]), __builtin_fma(g[4], yd, g[5]),
                  __builtin_fma(g[7], yd, g[8])};
}
__device__ __forceinline__ RowMap shift_row(const hsgd_warp& w, double yd) {
    return RowMap{1.0, 0.0, 0.0, (double)w.ix + (double)w.fx, yd + (double)w.iy + (double)w.fy, 1.0};
}

// A record read at once: behind the branch on its kind its parts would wait for memory twice.
__device__ __forceinline__ hsgd_warp read_record(const hsgd_warp* p) {
    hsgd_warp w = *p;
    for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(w.G[i]));
    asm volatile("" : "+v"(w.is_shift), "+v"(w.ix), "+v"(w.iy), "+v"(w.fx), "+v"(w.fy));
    return w;
}

// The map of a record as the kernels that tabulate maps use it: they compute positions without
// a check, so what these cannot be computed from is replaced here, once per plane, by a map
// that places every pixel where the numbers would. An entry of the first two rows that is no
// number or infinite (from 2^960 on it counts as that), a third row with such an entry that is
// not +inf, or one of no normal number, places none in front. A third row with a +inf has an
// infinite q2, that is the position (0, 0), except where the inf is multiplied by x = 0 or
// y = 0; two infs so multiplied place none. (A check of each position cost the gradient 1 to 3%.)
struct PlaneMap {
    double g[9];
};
__device__ __forceinline__ PlaneMap plane_map(const hsgd_warp& w) {
    PlaneMap m;
    if (w.is_shift) {
        const RowMap r = shift_row(w, 0.0);
        return PlaneMap{{1.0, 0.0, r.b0, 0.0, 1.0, r.b1, 0.0, 0.0, 1.0}};
    }
    constexpr int kHuge = 1023 + 960;
    int e[9], most = 0;                                     // biased exponents
    for (int i = 0; i < 9; ++i) {
        m.g[i] = w.G[i];
        e[i] = (int)((__builtin_bit_cast(uint64_t, m.g[i]) >> 52) & 0x7ffu);
        most = max(most, e[i]);
    }
    if (most >= kHuge || (e[6] | e[7] | e[8]) == 0) {
        constexpr double kFar = 0x1p900;
        const bool ix = e[6] >= kHuge, iy = e[7] >= kHuge;
        bool none = (ix && iy) || !(ix || iy || e[8] >= kHuge);
        for (int i = 0; i < 9; ++i) none = none || (e[i] >= kHuge && (i < 6 || !(m.g[i] > 0.0)));
        for (int i = 0; i < 6; ++i) m.g[i] = none ? 0.0 : m.g[i];
        m.g[6] = !none && ix ? kFar : 0.0;
        m.g[7] = !none && iy ? kFar : 0.0;
        m.g[8] = !none && !ix && !iy ? kFar : -1.0;
    }
    return m;
}

// 1 / q to FP64 accuracy: the hardware's estimate and two Newton steps (its ~24 correct bits
// become 48 and then the 53 of the format). An IEEE division costs three times as many
// instructions and its last-bit rounding moves a position by 1e-13 pixels.
__device__ __forceinline__ double rcp_f64(double q) {
    double r = __builtin_amdgcn_rcp(q);
    r = __builtin_fma(__builtin_fma(-q, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-q, r, 1.0), r, r);
}

// Position (floor and fraction, FP64 until the fraction is rounded) of pixel x of the row.
struct MapPos {
    double fu, fv;     // floor of the position; anything when the point is not in front
    float fx, fy;
    bool front;
};
// CHECK: of any map; otherwise of a plane_map.
template <bool CHECK>
__device__ __forceinline__ MapPos map_pos(const RowMap& m, double x) {
    const double q0 = __builtin_fma(m.a0, x, m.b0), q1 = __builtin_fma(m.a1, x, m.b1);
    const double q2 = __builtin_fma(m.a2, x, m.b2);
    double r = rcp_f64(q2);
    double u = q0 * r, v = q1 * r;
    MapPos p;
    p.front = q2 > 0.0;
    // No number: from such an entry, or a q2 that the Newton steps do not bear (infinite, or so
    // small that its reciprocal is). The division decides; what is no number then is outside.
    if (CHECK && __builtin_amdgcn_ballot_w64(__builtin_isunordered(u, v))) {
        r = 1.0 / q2;
        u = q0 * r;
        v = q1 * r;
        p.front = p.front && !__builtin_isunordered(u, v);
    }
    p.fu = floor(u);
    p.fv = floor(v);
    p.fx = (float)(u - p.fu);
    p.fy = (float)(v - p.fv);
    return p;
}

// Byte offsets of the four taps in a W x H plane of S-byte pixels, for loads through a buffer
// resource over the plane: a tap outside it gets an offset past the resource and reads 0, the
// zero padding. A wave whose lanes all have the four taps inside (nearly every wave) takes
// the short way: one address, the others at fixed distances. When no tap of a lane is inside,
// its fractions (which may be NaN there) become 0.
constexpr unsigned kOutside = 0xfffffff0u;
struct TapOffs {
    unsigned o00, o10, o01, o11;
};
// FP64 -> int32 in one instruction: out-of-range values saturate, NaN gives 0.
__device__ __forceinline__ int cvt_i32_f64(double d) {
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(d));
    return i;
}
// For a kernel that also scatters: the top-left tap's cell y0 W + x0 and which of the two tap
// columns (bits 0, 1) and rows (bits 2, 3) lie in the plane.
struct TapCell {
    int cell;
    unsigned in;
};
template <int S>
__device__ __forceinline__ TapOffs tap_offsets(MapPos& p, int W, int H, TapCell& c) {
    TapOffs t;
    int x0 = cvt_i32_f64(p.fu), y0 = cvt_i32_f64(p.fv);
    const uint64_t inner = __builtin_amdgcn_ballot_w64(p.front) &
                           __builtin_amdgcn_ballot_w64((unsigned)x0 < (unsigned)(W - 1)) &
                           __builtin_amdgcn_ballot_w64((unsigned)y0 < (unsigned)(H - 1));
    if (inner == __builtin_amdgcn_read_exec()) {
        c.cell = y0 * W + x0;
        c.in = 15u;
        t.o00 = (unsigned)c.cell * (unsigned)S;
        t.o10 = t.o00 + S;
        t.o01 = t.o00 + (unsigned)W * S;
        t.o11 = t.o01 + S;
    } else {
        const bool any = p.front & (x0 >= -1) & (x0 < W) & (y0 >= -1) & (y0 < H);
        x0 = any ? x0 : -2;
        y0 = any ? y0 : -2;
        const bool bx0 = (unsigned)x0 < (unsigned)W, bx1 = (unsigned)(x0 + 1) < (unsigned)W;
        const bool by0 = (unsigned)y0 < (unsigned)H, by1 = (unsigned)(y0 + 1) < (unsigned)H;
        c.cell = y0 * W + x0;
        c.in = (bx0 ? 1u : 0u) | (bx1 ? 2u : 0u) | (by0 ? 4u : 0u) | (by1 ? 8u : 0u);
        const unsigned o = (unsigned)c.cell * (unsigned)S;
        t.o00 = bx0 && by0 ? o : kOutside;
        t.o10 = bx1 && by0 ? o + S : kOutside;
        t.o01 = bx0 && by1 ? o + (unsigned)W * S : kOutside;
        t.o11 = bx1 && by1 ? o + (unsigned)W * S + S : kOutside;
        p.fx = any ? p.fx : 0.0f;
        p.fy = any ? p.fy : 0.0f;
    }
    return t;
}
template <int S>
__device__ __forceinline__ TapOffs tap_offsets(MapPos& p, int W, int H) {
    TapCell c;
    return tap_offsets<S>(p, W, H, c);
}

// A grid dimension holds fewer than 2^32 threads; of a longer one the runtime launches the low
// 32 bits, without an error. Longer grids therefore go on in y.
// The grid of `each` workgroups for every one of N views, the views split evenly over y where
// they do not fit x (`each` alone must).
inline dim3 split_grid(int64_t each, int N, int threads) {
    int rows = 1;
    while (rows < N && (N % rows || each * (N / rows) * threads > (int64_t)UINT32_MAX)) ++rows;
    return dim3((unsigned)(each * (N / rows)), (unsigned)rows);
}
// The grid of n workgroups, with up to rows - 1 too many, which return at once.
inline dim3 items_grid(int64_t n, int threads) {
    const int64_t rows = ceil_div(n * threads, (int64_t)UINT32_MAX - threads);
    return dim3((unsigned)ceil_div(n, rows), (unsigned)rows);
}
// Index of a workgroup in either grid, and the first's number of workgroups.
__device__ __forceinline__ int flat_block() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }
__device__ __forceinline__ int flat_blocks() { return (int)(gridDim.x * gridDim.y); }

// Block index -> tile index so that each XCD (workgroups are dealt round-robin to the 8
// XCDs) works on a contiguous run of tiles: the views of one tile and neighbouring tiles
// share MPI lines in that XCD's L2.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
    const int q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

}  // namespace
}  // namespace hsgd
