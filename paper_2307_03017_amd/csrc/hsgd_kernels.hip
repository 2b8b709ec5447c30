// HIP kernels of libhsgd for gfx950 (wave64).
//
//  k_select     scores A_z = a_z T_z of the un-warped MPI in exact FP32 order, top-k per
//               pixel -> uint64 plane mask; per-(plane, wave) ballot counts
//               (Sec. 3.3 Gradient Sparsification, Eq. gradient / Eq. overA)
//  k_scan_*     exclusive scan of those counts in plane-major order
//  k_compact    wavefront ballot/popcount compaction -> ascending linear ids (S)
//  k_render     warp + front-to-back over per view ray (Eq. render, Eq. over, Eq. homo);
//               k_render_shift and k_render_shift_rows for translations (one row of rays
//               per wave on small calls, four or eight on large ones)
//  k_grad       forward scan, residual, back-to-front adjoint scan, transposed bilinear
//               scatter restricted to S (Sec. 3.3; Eq. 4 gradient)
//  k_update     restore the sparse step onto S with clamp (the M_{n+1} update)
//  k_upsample   2x bilinear MPI upsampling between hierarchy levels; k_upsample_select(_blk)
//               fuse it with the new level's first selection (per output pixel on small
//               levels, per 2 x 2 output block from three source rows on large ones)
//  k_downsample 2x2 box mean of target images (the H/2^l pyramid, Sec. 3.2); k_pyramid
//               computes up to three such levels from one read of the finer images
#include <hip/hip_runtime.h>

#include <climits>

#include "hsgd_device.h"
#include "hsgd_internal.h"

namespace hsgd {
namespace {

// ------------------------------------------------------------------------------------
// storage: FP32 float4 or BF16 (4 x 16 bit, round to nearest even on store)
// ------------------------------------------------------------------------------------

template <int DT>
struct Vox;

template <>
struct Vox<HSGD_FP32> {
    static __device__ __forceinline__ float4 load(const void* base, int i) {
        return reinterpret_cast<const float4*>(base)[i];
    }
    static __device__ __forceinline__ float alpha(const void* base, int i) {
        return reinterpret_cast<const float*>(base)[4 * (size_t)i + 3];
    }
    static __device__ __forceinline__ void store(void* base, int i, float4 v) {
        reinterpret_cast<float4*>(base)[i] = v;
    }
    // voxels i and i + 1 (i even)
    static __device__ __forceinline__ void store2(void* base, int i, float4 a, float4 b) {
        reinterpret_cast<float4*>(base)[i] = a;
        reinterpret_cast<float4*>(base)[i + 1] = b;
    }
    // voxel `col` of the row starting at `row` (row uniform across the wave)
    static __device__ __forceinline__ float4 load_row(const char* row, unsigned col) {
        return *reinterpret_cast<const float4*>(row + (col << 4));
    }
    static __device__ __forceinline__ const char* row_ptr(const void* base, int i) {
        return reinterpret_cast<const char*>(base) + (size_t)(unsigned)i * 16;
    }
    // voxel at byte offset `off` of a buffer resource (0 outside the resource's range)
    static __device__ __forceinline__ float4 load_buf(__amdgpu_buffer_rsrc_t r, unsigned off) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]),
                           __uint_as_float(v[3]));
    }
    static constexpr int kBytes = 16;
    static __device__ __forceinline__ float4 stored(float4 v) { return v; }
    using Raw = float4;                                     // a voxel as stored
    static __device__ __forceinline__ Raw load_raw(__amdgpu_buffer_rsrc_t r, unsigned off) { return load_buf(r, off); }
    static __device__ __forceinline__ float4 decode(const Raw& v) { return v; }
};

template <>
struct Vox<HSGD_BF16> {
    static __device__ __forceinline__ float4 load(const void* base, int i) {
        uint2 r = reinterpret_cast<const uint2*>(base)[i];
        return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                           __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
    }
    static __device__ __forceinline__ float alpha(const void* base, int i) {
        return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(base)[4 * (size_t)i + 3] << 16);
    }
    static __device__ __forceinline__ void store(void* base, int i, float4 v) {
        reinterpret_cast<uint2*>(base)[i] = make_uint2(f32x2_to_bf16x2(v.x, v.y), f32x2_to_bf16x2(v.z, v.w));
    }
    // voxels i and i + 1 (i even: one 16-byte store)
    static __device__ __forceinline__ void store2(void* base, int i, float4 a, float4 b) {
        reinterpret_cast<uint4*>(base)[i >> 1] = make_uint4(f32x2_to_bf16x2(a.x, a.y), f32x2_to_bf16x2(a.z, a.w),
                                                            f32x2_to_bf16x2(b.x, b.y), f32x2_to_bf16x2(b.z, b.w));
    }
    static __device__ __forceinline__ float4 load_row(const char* row, unsigned col) {
        const uint2 r = *reinterpret_cast<const uint2*>(row + (col << 3));
        return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                           __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
    }
    static __device__ __forceinline__ const char* row_ptr(const void* base, int i) {
        return reinterpret_cast<const char*>(base) + (size_t)(unsigned)i * 8;
    }
    static __device__ __forceinline__ float4 load_buf(__amdgpu_buffer_rsrc_t r, unsigned off) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        return make_float4(__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xffff0000u),
                           __uint_as_float(v[1] << 16), __uint_as_float(v[1] & 0xffff0000u));
    }
    static constexpr int kBytes = 8;
    using Raw = uint2;                                      // a voxel as stored
    static __device__ __forceinline__ Raw load_raw(__amdgpu_buffer_rsrc_t r, unsigned off) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        return make_uint2(v[0], v[1]);
    }
    static __device__ __forceinline__ float4 decode(const Raw& v) {
        return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                           __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
    }
    // the value a store followed by a load returns (round to nearest even, NaN quieted)
    static __device__ __forceinline__ float4 stored(float4 v) {
        return decode(make_uint2(f32x2_to_bf16x2(v.x, v.y), f32x2_to_bf16x2(v.z, v.w)));
    }
};

// A sample of a general map: the four taps as stored and their bilinear blend (explicit FMAs:
// every scan that samples a plane gets the same bits).
template <int DT>
struct Tap4 {
    typename Vox<DT>::Raw a, b, c, d;
};
template <int DT>
__device__ __forceinline__ Tap4<DT> load_taps(__amdgpu_buffer_rsrc_t plane, const TapOffs& o) {
    return Tap4<DT>{Vox<DT>::load_raw(plane, o.o00), Vox<DT>::load_raw(plane, o.o10), Vox<DT>::load_raw(plane, o.o01),
                    Vox<DT>::load_raw(plane, o.o11)};
}
struct TapW {
    float w00, w10, w01, w11;
};
__device__ __forceinline__ TapW tap_weights(float fx, float fy) {
    const float gx = 1.0f - fx, gy = 1.0f - fy;
    return TapW{gx * gy, fx * gy, gx * fy, fx * fy};
}
template <int DT>
__device__ __forceinline__ float4 blend_taps(const TapW& t, const Tap4<DT>& r) {
    const float4 va = Vox<DT>::decode(r.a), vb = Vox<DT>::decode(r.b), vc = Vox<DT>::decode(r.c), vd = Vox<DT>::decode(r.d);
    auto f = [&](float a, float b, float c, float d) {
        return __builtin_fmaf(t.w11, d, __builtin_fmaf(t.w01, c, __builtin_fmaf(t.w10, b, t.w00 * a)));
    };
    return make_float4(f(va.x, vb.x, vc.x, vd.x), f(va.y, vb.y, vc.y, vd.y), f(va.z, vb.z, vc.z, vd.z),
                       f(va.w, vb.w, vc.w, vd.w));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum over a 256-thread block; the result is valid on thread 0.
__device__ __forceinline__ float block_sum(float v, float* sh) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = 0.0f;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) r += sh[i];
    return r;
}

// ------------------------------------------------------------------------------------
// select: scores, top-k, and the active-set structures
// ------------------------------------------------------------------------------------
// Per pixel p: A_z = fl(a_z T_z), T_{z+1} = fl(T_z fl(1 - a_z)) front to back on the
// un-warped MPI, then the k largest A_z (equal scores: the nearer plane), then the optional
// threshold. Returns the plane bitmask of p. FP32 contraction is off for this function.
// One front-to-back step of the score recursion for plane alpha a: A = fl(a T) (NaN ranks
// last), T <- fl(T fl(1 - a)).
__device__ __forceinline__ float score_step(float a, float& T) {
#pragma clang fp contract(off)
    const float s = a * T;
    T = T * (1.0f - a);
    return (s == s) ? s : -INFINITY;
}

// The plane mask of the selection rule on the scores A[0..D), then the optional threshold.
// Top-k: the k largest scores (equal scores: the nearer plane). MVS window: the largest
// score (equal: the nearer plane) with (k-1)/2 planes before it (rounded down) and the
// rest after, moved inside [0, D).
// Every pass below is branch-free: the conditions are combined with bitwise operators
// and the running best is kept by selects (with short-circuit operators the unrolled
// passes compiled to a branch per plane).
template <int MAXD>
__device__ __forceinline__ uint64_t topk_bits(const float (&A)[MAXD], int D, int k, float tau, int rule) {
    const uint64_t full = D == 64 ? ~0ull : ((1ull << D) - 1);
    const int kk = min(k, D);
    uint64_t sel = 0;
    if (kk == D) {
        sel = full;
    } else if (rule == HSGD_SELECT_MVS) {
        int best = 0;
        float bestA = A[0];
#pragma unroll
        for (int z = 1; z < MAXD; ++z) {
            const bool b = (z < D) & (A[z] > bestA);
            best = b ? z : best;
            bestA = b ? A[z] : bestA;
        }
        const int lo = min(max(best - (kk - 1) / 2, 0), D - kk);
        sel = lane_bits_below(lo + kk) & ~lane_bits_below(lo);
    } else if (2 * kk <= D) {
        // kk passes: the best remaining score, the nearer plane on equal scores
        for (int j = 0; j < kk; ++j) {
            int best = -1;
            float bestA = 0.0f;
#pragma unroll
            for (int z = 0; z < MAXD; ++z) {
                const bool b = (z < D) & (((sel >> z) & 1ull) == 0ull) & ((best < 0) | (A[z] > bestA));
                best = b ? z : best;
                bestA = b ? A[z] : bestA;
            }
            sel |= lane_bit(best);
        }
    } else {
        // D - kk passes removing the worst: the lowest score, the farther plane on ties
        uint64_t out = 0;
        for (int j = 0; j < D - kk; ++j) {
            int worst = -1;
            float worstA = 0.0f;
#pragma unroll
            for (int z = 0; z < MAXD; ++z) {
                const bool b = (z < D) & (((out >> z) & 1ull) == 0ull) & ((worst < 0) | (A[z] <= worstA));
                worst = b ? z : worst;
                worstA = b ? A[z] : worstA;
            }
            out |= lane_bit(worst);
        }
        sel = full & ~out;
    }
    if (tau >= 0.0f) {
#pragma unroll
        for (int z = 0; z < MAXD; ++z)
            sel &= ~((uint64_t)((z < D) & !(A[z] > tau)) << z);
    }
    return sel;
}

// All D alpha loads are issued before the first is used (plane index clamped, so the loads
// need no guard): one memory latency per pixel rather than one per plane.
template <int DT, int MAXD>
__device__ __forceinline__ uint64_t select_bits(const void* __restrict__ mpi, int D, int HW, int p,
                                                int k, float tau, int rule) {
    float a[MAXD];
#pragma unroll
    for (int z = 0; z < MAXD; ++z) a[z] = Vox<DT>::alpha(mpi, min(z, D - 1) * HW + p);
    float A[MAXD];
    float T = 1.0f;
#pragma unroll
    for (int z = 0; z < MAXD; ++z)
        if (z < D) A[z] = score_step(a[z], T);
    return topk_bits<MAXD>(A, D, k, tau, rule);
}

// The transposed view of a 64-pixel block's masks: for every plane the wave ballot (bit
// = pixel of the block) and its population count. Every lane of the wave must call it.
__device__ __forceinline__ void emit_ballots(uint64_t sel, int D, int64_t wblk, int64_t nblk,
                                             uint64_t* __restrict__ bal, int* __restrict__ cnt) {
    for (int z = 0; z < D; ++z) {
        const uint64_t b = __ballot((sel >> z) & 1);
        if ((threadIdx.x & 63) == 0 && wblk < nblk) {
            bal[z * nblk + wblk] = b;
            cnt[z * nblk + wblk] = __popcll(b);
        }
    }
}

template <int DT, int MAXD>
__global__ __launch_bounds__(256) void k_select(const void* __restrict__ mpi, int D, int HW, int k,
                                                float tau, int rule, uint64_t* __restrict__ mask,
                                                uint64_t* __restrict__ bal, int* __restrict__ cnt,
                                                int64_t nblk) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t sel = 0;
    if (p < HW) {
        sel = select_bits<DT, MAXD>(mpi, D, HW, p, k, tau, rule);
        if (mask) mask[p] = sel;
    }
    if (bal) emit_ballots(sel, D, (int64_t)p >> 6, nblk, bal, cnt);
}

// Active-set structures from a caller's mask (NULL: every voxel); bits of a pixel beyond
// its first kcap set bits are dropped.
__global__ __launch_bounds__(256) void k_mask_ballot(const uint64_t* __restrict__ mask, int D, int HW,
                                                     int kcap, uint64_t* __restrict__ bal,
                                                     int* __restrict__ cnt, int64_t nblk) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t full = D == 64 ? ~0ull : ((1ull << D) - 1);
    uint64_t sel = 0;
    if (p < HW) {
        sel = (mask ? mask[p] : full) & full;
        if (__popcll(sel) > kcap) {
            uint64_t kept = 0;
            for (int j = 0; j < kcap; ++j) {
                const uint64_t low = sel & (~sel + 1);
                kept |= low;
                sel &= sel - 1;
            }
            sel = kept;
        }
    }
    emit_ballots(sel, D, (int64_t)p >> 6, nblk, bal, cnt);
}

// Segmented exclusive scan of the counts (plane-major), phase 1: each workgroup scans
// kSeg consecutive entries in place and writes its total.
constexpr int kSeg = kScanSeg;
__global__ __launch_bounds__(256) void k_scan_seg(int* __restrict__ v, int64_t n,
                                                  int* __restrict__ seg_total) {
    __shared__ int sv[kSeg];
    __shared__ int ssum[256];
    const int64_t base = (int64_t)blockIdx.x * kSeg;
    for (int i = threadIdx.x; i < kSeg; i += 256) sv[i] = base + i < n ? v[base + i] : 0;
    __syncthreads();
    int s = 0;
    for (int j = 0; j < kSeg / 256; ++j) s += sv[threadIdx.x * (kSeg / 256) + j];
    ssum[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        int t = threadIdx.x >= o ? ssum[threadIdx.x - o] : 0;
        __syncthreads();
        ssum[threadIdx.x] += t;
        __syncthreads();
    }
    int run = ssum[threadIdx.x] - s;
    for (int j = 0; j < kSeg / 256; ++j) {
        int c = sv[threadIdx.x * (kSeg / 256) + j];
        sv[threadIdx.x * (kSeg / 256) + j] = run;
        run += c;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSeg; i += 256)
        if (base + i < n) v[base + i] = sv[i];
    if (threadIdx.x == 255) seg_total[blockIdx.x] = ssum[255];
}

// Phase 2 (one workgroup): exclusive scan of the segment totals; plane offsets and |S|.
__global__ __launch_bounds__(1024) void k_scan_top(const int* __restrict__ v, int64_t nblk, int D,
                                                   int* __restrict__ seg, int nseg,
                                                   int* __restrict__ plane_off,
                                                   int* __restrict__ n_active) {
    __shared__ int sh[1024];
    __shared__ int carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int b = 0; b < nseg; b += 1024) {
        const int i = b + threadIdx.x;
        const int x = i < nseg ? seg[i] : 0;
        sh[threadIdx.x] = x;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            int t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += t;
            __syncthreads();
        }
        if (i < nseg) seg[i] = carry + sh[threadIdx.x] - x;
        __syncthreads();
        if (threadIdx.x == 1023) carry += sh[1023];
        __syncthreads();
    }
    if (plane_off) {
        for (int z = threadIdx.x; z < D; z += 1024) {
            const int64_t e = (int64_t)z * nblk;
            plane_off[z] = v[e] + seg[e / kSeg];
        }
    }
    if (threadIdx.x == 0) {
        if (plane_off) plane_off[D] = carry;
        *n_active = carry;
    }
}

// Wavefront compaction: each wave owns one 64-pixel block; for every plane its ballot
// word gives the selected lanes and their rank (popcount below the lane), its scanned
// offset the position of the block in the plane-major list. Also turns the offsets into
// global positions in place, for the gradient kernels.
__global__ __launch_bounds__(256) void k_compact(const uint64_t* __restrict__ bal, int* __restrict__ off,
                                                 const int* __restrict__ seg, int D, int HW,
                                                 int64_t nblk, int* __restrict__ ids, int64_t cap) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t wblk = (int64_t)p >> 6;
    if (wblk >= nblk) return;   // whole waves only
    const int lane = threadIdx.x & 63;
    for (int z = 0; z < D; ++z) {
        const int64_t e = (int64_t)z * nblk + wblk;
        const uint64_t b = bal[e];
        const int base = off[e] + seg[e / kSeg];
        if (has_lane_bit(b, lane)) {
            const int64_t pos = (int64_t)base + __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32),
                                                                          __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
            if (pos < cap) ids[pos] = z * HW + p;
        }
        if (lane == 0) off[e] = base;
    }
}

// ------------------------------------------------------------------------------------
// render
// ------------------------------------------------------------------------------------
// General homographies: a wave takes 64 neighbouring rays of one row of one view. Positions
// are FP64 (~20 instructions a sample: the row's part of the map is tabulated in LDS, the
// division is a reciprocal estimate with two Newton steps), the taps come through a buffer
// resource over the plane, and the loads of one plane (BF16: two) are in flight while one is
// blended. Bound by its instructions (about 75 per sample, a quarter of them FP64); more planes
// in flight cost waves and gain nothing: 512x384x32, 8 views, FP32 120 us with three and 115 with
// one (108 and 72 registers), BF16 107.7, 107.9 with two, 107.6 with one, 954x625x32, one view,
// BF16 46.7, 47.2, 49.2. No plane past the last is fetched: 980x775x9, 18 views, FP32 410 us with
// such fetches, 327 without.
// FEW: of one or two planes. A table and a barrier for a row's one use of each map, and the tiles'
// order by XCD, cost such a call more than they give: 980x775x1, 18 views, FP32 72 us, without
// table 65, by view as well 60; 980x775x3 119 in the order by XCD, 126 by view.
constexpr int kRenderFew = 2;
template <int DT, bool FEW>
__global__ __launch_bounds__(kBlock) void k_render(const void* __restrict__ mpi, int D, int H, int W, int N,
                                                   const hsgd_warp* __restrict__ warps,
                                                   const float* __restrict__ images,
                                                   float* __restrict__ out_rgb,
                                                   float* __restrict__ partials, int ntx) {
    constexpr int S = Vox<DT>::kBytes;
    __shared__ RowMap s_map[kTileH][FEW ? 1 : kMaxD];
    __shared__ float sred[kBlock / 64];
    int tile, view, x0, y0;
    if constexpr (FEW) {
        view = blockIdx.z;
        x0 = blockIdx.x * kTileW, y0 = blockIdx.y * kTileH;
        tile = (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
    } else {
        tile = xcd_tile(flat_block(), flat_blocks());
        view = tile % N;
        const int t2 = tile / N;
        x0 = (t2 % ntx) * kTileW, y0 = (t2 / ntx) * kTileH;
    }
    for (int i = threadIdx.x; !FEW && i < kTileH * D; i += kBlock) {
        const int r = i / D, z = i - r * D;
        const hsgd_warp w = read_record(warps + (size_t)view * D + z);
        const double yd = (double)(y0 + r);
        s_map[r][z] = w.is_shift ? shift_row(w, yd) : row_map(plane_map(w).g, yd);
    }
    if (!FEW) __syncthreads();
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int x = x0 + (int)(threadIdx.x & 63), y = y0 + wv;
    const double xd = (double)x;
    const size_t plane_bytes = (size_t)H * W * S;
    struct Fetched {
        Tap4<DT> t;
        float fx, fy;
    };
    auto fetch = [&](int z) {
        MapPos p;
        if constexpr (FEW) {
            const hsgd_warp& w = warps[(size_t)view * D + z];
            p = map_pos<true>(w.is_shift ? shift_row(w, (double)y) : row_map(w.G, (double)y), xd);
        } else {
            p = map_pos<false>(s_map[wv][z], xd);
        }
        const TapOffs o = tap_offsets<S>(p, W, H);
        const auto rs = row_rsrc(reinterpret_cast<const char*>(mpi) + (size_t)z * plane_bytes, (int)plane_bytes);
        return Fetched{load_taps<DT>(rs, o), p.fx, p.fy};
    };
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    auto blend = [&](const Fetched& f) {
        const float4 s = blend_taps<DT>(tap_weights(f.fx, f.fy), f.t);
        const float wgt = T * s.w;
        c0 = __builtin_fmaf(wgt, s.x, c0);
        c1 = __builtin_fmaf(wgt, s.y, c1);
        c2 = __builtin_fmaf(wgt, s.z, c2);
        T *= 1.0f - s.w;
    };
    constexpr int kQ = DT == HSGD_BF16 ? 3 : 2;             // planes in flight: kQ - 1
    Fetched q[kQ];
#pragma unroll
    for (int j = 0; j + 1 < kQ; ++j)
        if (j < D) q[j] = fetch(j);
    for (int z = 0; z < D; z += kQ) {
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            if (z + j + kQ - 1 < D) q[(j + kQ - 1) % kQ] = fetch(z + j + kQ - 1);
            if (z + j < D) blend(q[j]);
        }
    }
    float sq = 0.0f;
    if (x < W && y < H) {
        const size_t pix = ((size_t)view * H + y) * W + x;
        if (out_rgb) {
            out_rgb[3 * pix + 0] = c0;
            out_rgb[3 * pix + 1] = c1;
            out_rgb[3 * pix + 2] = c2;
        }
        if (partials) {
            const float d0 = c0 - images[3 * pix + 0];
            const float d1 = c1 - images[3 * pix + 1];
            const float d2 = c2 - images[3 * pix + 2];
            sq = __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
        }
    }
    if (partials) {
        const float tot = block_sum(sq, sred);
        if (threadIdx.x == 0) partials[tile] = tot;
    }
}

// Deterministic final reduction of per-block partials (FP64 accumulation).
__global__ __launch_bounds__(256) void k_reduce(const float* __restrict__ partials, int64_t n,
                                                double scale, float* __restrict__ out) {
    __shared__ double sh[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)partials[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = (float)(sh[0] * scale);
}

// ------------------------------------------------------------------------------------
// Gradient slots. A selected voxel (z, p) whose pixel has r selected planes nearer than z
// ("rank" r, r < kcap) owns slot (r, p) of a rank-major slice [kcap][H*W] of float4; the
// gradient kernels write per-view slices [N][kcap][H*W] (or one slice for general warps)
// and the update kernel sums them.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ uint64_t plane_bits(int D) { return D == 64 ? ~0ull : ((1ull << D) - 1); }

// ------------------------------------------------------------------------------------
// gradient, general warps: per-ray scans, transposed-bilinear scatter with atomics
//
// A workgroup takes 64 x 8 rays of one view; lane 63 of each wave only receives what lane 62
// sends to its right (its ray belongs to the next tile). Both scans are rolled loops over
// pairs of planes, so any plane count runs its own planes only (an odd count one transparent
// plane more). The front-to-back scan leaves the transmittance in front of each pair in LDS;
// the back-to-front scan samples a pair again and recomputes the second transmittance with
// the same operation.
//
// Scatter. A ray touches four cells of a plane; neighbouring rays nearly always share them.
// The right column of lane i - 1 is added to the left column of lane i, and the lower row of
// a wave to the upper row of the next wave through LDS, where the cells are the same, so
// about 1.15 cells per ray remain. Those that are selected are staged in LDS, and 64 at a
// time added to the slots with four lanes per cell: the memory system takes about 22 G
// 64-byte atomic requests a second whatever they hold, and a float4 added by one lane is
// four requests instead of one. A wave none of whose cells is selected (about half of them
// with 4 of 32 planes kept) skips a plane's adjoint and scatter.
// Bound by the two scans, FP64 positions and four tap loads a sample (57% of the vector issue
// slots of the finest 512x384x32 launch) at 4 waves per SIMD, and in a dense gradient by the
// atomics. The form for more than 32 planes has 109 KB of LDS in place of 75, so one workgroup
// per CU and 2 waves per SIMD. 512x384x32, 4 tilted views, k = 4: 672 us with an IEEE
// division per position and one atomic per lane and channel, 289 us now; the dense gradient
// of 501x333x24, 2 tilted views: 693 and 198 us. Taps of the next pair in flight behind the
// scatter, at 3 waves per SIMD or with spills at 4, measured slower (311 and 399 us), and so
// did 4 rows per workgroup in the dense gradient (207 us).
// ------------------------------------------------------------------------------------
// Whole-wave lane shifts: lane i <- lane i-1 / lane i+1; a lane without a source gets `none`.
__device__ __forceinline__ int lane_prev_i(int v, int none) {
    return __builtin_amdgcn_update_dpp(none, v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ int lane_next_i(int v, int none) {
    return __builtin_amdgcn_update_dpp(none, v, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ float4 lane_prev_f4(float4 v) {
    auto f = [](float a) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x138, 0xF, 0xF, false)); };
    return make_float4(f(v.x), f(v.y), f(v.z), f(v.w));
}
__device__ __forceinline__ float4 only_if(bool c, const float4& a) {
    return make_float4(c ? a.x : 0.0f, c ? a.y : 0.0f, c ? a.z : 0.0f, c ? a.w : 0.0f);
}
__device__ __forceinline__ float4 add4(const float4& a, const float4& b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float4 scale4(float w, const float4& g) {
    return make_float4(w * g.x, w * g.y, w * g.z, w * g.w);
}

// Slot rank of plane z (it differs by lane) among the pixel's selected planes, or -1 (not
// selected, or ranked kcap and beyond).
__device__ __forceinline__ int slot_rank_lane(uint64_t m, unsigned z, int kcap) {
    const int r = __popcll(m & lane_bits_below(z));
    return has_lane_bit(m, z) && r < kcap ? r : -1;
}

// One wave's cells on their way to the slots: a ring of values and the cells they go to
// (cell | plane << 26: H W <= 2^26 and z < 64), emptied 64 at a time. Emptying reads a mask
// word per lane to find each cell's slot, so that a stray cell, whose word nobody loaded
// ahead, costs a 64th of a memory latency; then four lanes add one cell.
constexpr int kStage = 128;
struct GradStage {
    float4 v[kStage];
    unsigned to[kStage];
};
struct GradSink {
    GradStage* st;
    float4* slots;
    const uint64_t* mask;
    uint64_t full;
    int lane, HW, kcap;
    int head, count;                     // wave-uniform
    __device__ void flush(int n) {
        wave_lds_fence();
        if (lane < n) {
            const int i = (head + lane) & (kStage - 1);
            const unsigned to = st->to[i], cell = to & ((1u << 26) - 1);
            const int r = slot_rank_lane(mask ? mask[cell] : full, to >> 26, kcap);
            st->to[i] = r >= 0 ? (unsigned)r * (unsigned)HW + cell : ~0u;
        }
        wave_lds_fence();
        for (int e0 = 0; e0 < n; e0 += 16) {
            const int e = e0 + (lane >> 2);
            const int i = (head + e) & (kStage - 1);
            const unsigned slot = e < n ? st->to[i] : ~0u;
            if (slot != ~0u)
                atomicAdd(reinterpret_cast<float*>(reinterpret_cast<char*>(slots) + (slot * 16u + (lane & 3) * 4u)),
                          reinterpret_cast<const float*>(st->v)[4 * i + (lane & 3)]);
        }
        head = (head + n) & (kStage - 1);
        count -= n;
        wave_lds_fence();
    }
    // lanes with `on` add v to the cell of plane z (every lane of the wave calls it)
    __device__ void put(bool on, int z, int cell, const float4& v) {
        const uint64_t b = __builtin_amdgcn_ballot_w64(on);
        if (b == 0) return;
        const int r = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
        const int i = (head + count + r) & (kStage - 1);
        if (on) {
            st->v[i] = v;
            st->to[i] = (unsigned)cell | ((unsigned)z << 26);
        }
        count += __popcll(b);
        if (count >= 64) flush(64);
    }
};

constexpr int kGenOX = 63, kGenY = 8;
constexpr int kGenThreads = 64 * kGenY;
template <int DT, int MAXD>
__global__ __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_grad(
    const void* __restrict__ mpi, int D, int H, int W, int N, const hsgd_warp* __restrict__ warps,
    const float* __restrict__ images, const float* __restrict__ dimg, const uint64_t* __restrict__ mask, int kcap,
    float inv_n, float4* __restrict__ slots, float* __restrict__ partials, int ntx) {
    constexpr int S = Vox<DT>::kBytes;
    __shared__ double s_map[MAXD][10];                      // G of each plane (rows of three, padded)
    __shared__ float s_T[MAXD / 2][kGenThreads];            // transmittance in front of each pair of planes
    // by plane parity: every lane's left-column cell and what it holds for the row below
    __shared__ int s_key[2][kGenThreads];
    __shared__ float4 s_low[2][kGenThreads];
    __shared__ GradStage s_stage[kGenY];
    __shared__ float sred[kGenY];
    const int tile = xcd_tile(flat_block(), flat_blocks());
    const int view = tile % N, t2 = tile / N;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x = (t2 % ntx) * kGenOX + lane, y = (t2 / ntx) * kGenY + wv;
    const int HW = H * W, D2 = (D + 1) & ~1;
    for (int z = tid; z < D2; z += kGenThreads) {
        PlaneMap m{{0, 0, 0, 0, 0, 0, 0, 0, -1.0}};          // planes behind the last: nowhere in front
        if (z < D) m = plane_map(warps[(size_t)view * D + z]);
        for (int i = 0; i < 9; ++i) s_map[z][i] = m.g[i];
    }
    __syncthreads();
    // rays that contribute; the other lanes sample like the rest and add zeros
    const bool own = lane < kGenOX && x < W && y < H;
    const double xd = (double)x, yd = (double)y;
    const size_t plane_bytes = (size_t)HW * S;
    struct Fetched {
        Tap4<DT> t;
        float fx, fy;
    };
    auto fetch = [&](int z, TapOffs& o, TapCell& c) {
        MapPos p = map_pos<false>(row_map(s_map[z], yd), xd);
        o = tap_offsets<S>(p, W, H, c);
        return Fetched{load_taps<DT>(row_rsrc(reinterpret_cast<const char*>(mpi) + (size_t)min(z, D - 1) * plane_bytes,
                                              (int)plane_bytes), o), p.fx, p.fy};
    };
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    {
        constexpr int kA = DT == HSGD_BF16 ? 3 : 2;         // planes in flight behind the current one
        Fetched q[4];
        TapOffs o;
        TapCell c;
#pragma unroll
        for (int j = 0; j < kA; ++j) q[j] = fetch(min(j, D2 - 1), o, c);
        for (int z = 0; z < D2; z += 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                q[(j + kA) % 4] = fetch(min(z + j + kA, D2 - 1), o, c);
                if (z + j < D2) {
                    if (j % 2 == 0) s_T[(z + j) / 2][tid] = T;
                    const float4 s = blend_taps<DT>(tap_weights(q[j].fx, q[j].fy), q[j].t);
                    const float wgt = T * s.w;
                    c0 = __builtin_fmaf(wgt, s.x, c0);
                    c1 = __builtin_fmaf(wgt, s.y, c1);
                    c2 = __builtin_fmaf(wgt, s.z, c2);
                    T *= 1.0f - s.w;
                }
            }
        }
    }
    float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f, sq = 0.0f;
    if (own) {
        const size_t pix = ((size_t)view * H + y) * W + x;
        if (images) {
            const float d0 = c0 - images[3 * pix + 0];
            const float d1 = c1 - images[3 * pix + 1];
            const float d2 = c2 - images[3 * pix + 2];
            sq = __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
            g0 = d0 * inv_n;
            g1 = d1 * inv_n;
            g2 = d2 * inv_n;
        }
        if (dimg) {
            g0 = dimg[3 * pix + 0];
            g1 = dimg[3 * pix + 1];
            g2 = dimg[3 * pix + 2];
        }
    }
    const uint64_t full = plane_bits(D);
    const auto mask_rs = row_rsrc(reinterpret_cast<const char*>(mask), mask ? HW * 8 : 0);
    // the half of a cell's mask word that holds plane z, 0 (nothing selected) outside the plane;
    // o: the cell's byte offset in a plane
    auto mask_of = [&](unsigned o, int z) -> unsigned {
        if (!mask) return o < (unsigned)plane_bytes ? ~0u : 0u;
        return __builtin_amdgcn_raw_buffer_load_b32(mask_rs, o / (unsigned)(S / 8), z >= 32 ? 4 : 0, 0);
    };
    GradSink sink{&s_stage[wv], slots, mask, full, lane, HW, kcap, 0, 0};
    constexpr int kNone = INT_MIN;
    float b0 = 0.0f, b1 = 0.0f, b2 = 0.0f;   // composite behind plane z
    for (int zb = D2 - 2; zb >= 0; zb -= 2) {
        float4 sm[2];
        float fx[2], fy[2], Tz[2];
        TapCell cell[2];
        bool s00[2], s10[2], s01[2], s11[2];                // which of the four cells are selected
        {
            Fetched f[2];
            unsigned m[2][4];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                TapOffs o;
                f[j] = fetch(zb + j, o, cell[j]);
                m[j][0] = mask_of(o.o00, zb + j);
                m[j][1] = mask_of(o.o10, zb + j);
                m[j][2] = mask_of(o.o01, zb + j);
                m[j][3] = mask_of(o.o11, zb + j);
            }
            float t = s_T[zb / 2][tid];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                sm[j] = blend_taps<DT>(tap_weights(f[j].fx, f[j].fy), f[j].t);
                fx[j] = f[j].fx;
                fy[j] = f[j].fy;
                const unsigned bit = 1u << ((zb + j) & 31);
                s00[j] = (m[j][0] & bit) != 0u;
                s10[j] = (m[j][1] & bit) != 0u;
                s01[j] = (m[j][2] & bit) != 0u;
                s11[j] = (m[j][3] & bit) != 0u;
                Tz[j] = t;
                t *= 1.0f - sm[j].w;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 1; j >= 0; --j) {
            const int z = zb + j;
            const float4 s = sm[j];
            // (the buffers of the row merge alternate by plane: the next plane's writes go to
            // the other)
            int key = kNone;
            float4 v00, v01, v10, v11;
            int right = kNone;
            bool keep = false;
            // a wave none of whose cells is selected has nothing to add, nor to pass on
            const bool some = __builtin_amdgcn_ballot_w64(s00[j] | s10[j] | s01[j] | s11[j]) != 0;
            if (some) {
                // (without a ray the residual is zero, but zero times an infinite sample is not)
                const float ca = own ? s.w * Tz[j] : 0.0f;
                float4 gs;
                gs.x = g0 * ca;
                gs.y = g1 * ca;
                gs.z = g2 * ca;
                gs.w = own ? Tz[j] * (g0 * (s.x - b0) + g1 * (s.y - b1) + g2 * (s.z - b2)) : 0.0f;
                const TapW w = tap_weights(fx[j], fy[j]);
                const unsigned in = cell[j].in;
                key = (in & 1u) ? cell[j].cell : kNone;
                right = (in & 2u) && own && fx[j] != 0.0f ? cell[j].cell + 1 : kNone;
                v00 = scale4(w.w00, gs);
                v01 = scale4(w.w01, gs);
                v10 = scale4(w.w10, gs);
                v11 = scale4(w.w11, gs);
                // a tap of no weight takes nothing, whatever the adjoint
                if (__builtin_amdgcn_ballot_w64(fy[j] == 0.0f)) {
                    v01 = only_if(fy[j] != 0.0f, v01);
                    v11 = only_if(fy[j] != 0.0f, v11);
                }
                if (__builtin_amdgcn_ballot_w64(w.w00 == 0.0f)) {   // a fraction that rounded to 1
                    v00 = only_if(w.w00 != 0.0f, v00);
                    v10 = only_if(w.w10 != 0.0f, v10);
                    v01 = only_if(w.w01 != 0.0f, v01);
                }
                // lane i takes lane i-1's right column where it is its own left column; where it
                // is not, lane i-1 adds it to the cells by itself and sends zeros
                const bool sent = (lane_next_i(key, kNone) == right) & (right != kNone);
                keep = !sent & (right != kNone);
                float4 w10 = v10, w11 = v11;
                if (__builtin_amdgcn_ballot_w64(!sent) & (~0ull >> 1)) {
                    w10 = only_if(sent, v10);
                    w11 = only_if(sent, v11);
                }
                v00 = add4(v00, lane_prev_f4(w10));
                v01 = add4(v01, lane_prev_f4(w11));
                s_low[j][tid] = v01;
            }
            s_key[j][tid] = key;
            const float oa = 1.0f - s.w;
            b0 = s.w * s.x + oa * b0;
            b1 = s.w * s.y + oa * b1;
            b2 = s.w * s.z + oa * b2;
            __syncthreads();
            if (some) {
                if (wv > 0) {
                    const int above = s_key[j][tid - 64];
                    v00 = add4(v00, only_if((above != kNone) & (above + W == key), s_low[j][tid - 64]));
                }
                // what this wave adds: its upper left cells, a lower row that the row below does
                // not take, and right columns that were not sent
                const bool low = s01[j] & !(wv + 1 < kGenY && s_key[j][min(tid + 64, kGenThreads - 1)] == key + W);
                sink.put(s00[j], z, key, v00);
                sink.put(low, z, key + W, v01);
                sink.put(keep & s10[j], z, right, v10);
                sink.put(keep & s11[j], z, right + W, v11);
            }
        }
    }
    while (sink.count > 0) sink.flush(min(sink.count, 64));
    if (partials) {
        const float tot = block_sum(sq, sred);
        if (threadIdx.x == 0) partials[tile] = tot;
    }
}

// ------------------------------------------------------------------------------------
// gradient, pure-translation warps: owner-computes, no atomics, deterministic
//
// A workgroup takes a 64 x 8 block of view rays: lane 0 and wave 0 are a halo column and
// row, lane 63 only supplies the right-hand bilinear taps of lane 62, and the 62 x 7 rays
// in between are "owners". For plane z every owner (x, y) also owns the reference cell
// (x + ix_z, y + iy_z): with a translation, the four rays whose bilinear footprint covers
// that cell are the owner and its left, upper and upper-left neighbours, all in the block.
// Per-ray adjoints are combined across lanes with DPP and across waves through LDS, and
// each owner writes its cell's gradient once, into its view's slice of the slots.
// The front-to-back scan also fetches every owned cell's mask word and keeps one byte per
// plane (rank + 1, or 0 if the cell is not selected), so the back-to-front scan needs no
// memory access besides LDS, and skips the adjoint of planes no cell of the rows needs.
// ------------------------------------------------------------------------------------
constexpr int kSX = 64, kSY = kShiftOY + 1;
constexpr int kOX = kShiftOX, kOY = kShiftOY;
static_assert(kOX == kSX - 2, "lanes: halo, owners, tap supplier");

// DPP wave shifts (bound_ctrl: a lane without a source reads 0)
// Lane i <- lane i+1 (lane 63 <- 0) and lane i <- lane i-1 (lane 0 <- 0), written so that
// the shift folds into the consuming add or multiply as a DPP operand.
__device__ __forceinline__ float lane_from_next(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_from_prev(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, false));
}

__device__ __forceinline__ int rl(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float rlf(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Bilinear sample of a translation warp, one channel: this lane holds its column of the
// two tap rows (a0 above, a1 below), the next lane the column to the right. Vertical lerp
// of the own column, then the horizontal lerp with the next lane's (4 instructions, the
// lane shift folded into a multiply). wt = (upper row weight, lower row weight, 1 - fx,
// fx), a row outside the plane weighted 0.
template <typename W>
__device__ __forceinline__ float lerp_taps(float a0, float a1, const W& wt) {
    const float v = __builtin_fmaf(a1, wt.y, a0 * wt.x);
    return __builtin_fmaf(v, wt.z, lane_from_next(v) * wt.w);
}

using f32x4 = float __attribute__((ext_vector_type(4)));
using lds_f32x4 = __attribute__((address_space(3))) f32x4;

// One 64 x 8 tile of one view (tile = view + N * (tx + ntx * ty)); every thread of the
// workgroup calls it.
// The tile's forms by plane-count class: the planes whose front-to-back samples it keeps in
// registers for its back-to-front scan (keep), the leading planes whose transmittance lives
// in LDS instead of registers (tl), and the waves per SIMD it is compiled for. Small classes
// (and BF16 at 32 planes) keep nothing and are compiled for 6 waves per SIMD (3 workgroups per
// CU, within 80 registers and 53 KB; 8 and 16 planes need no more than 62 registers and 38 KB,
// so 4 workgroups are resident); the others keep as many samples as the registers of 4 waves per
// SIMD hold without spills once 2 workgroups' 160 KB of LDS are filled with transmittances.
// The forms are within a few percent of each other (BF16, 24 planes, 512 x 384, 4 views:
// 85 us against 88 at 6 waves; 48 planes: 172 us against 179 without kept samples). No one
// limit holds the kernel: its finest launch fills 53% of the vector and 40% of the scalar issue
// slots at 512 x 384 x 32 in FP32 (26% of the waves' time waiting) and 68% and 46% at 1920 x
// 1080 x 64 in BF16 (34% waiting). Of what the code spends it is the planes run and the vector
// instructions per plane that could be cut (105 per wave, plane and pair of scans in BF16, 62 of
// them the interpolation, the compositing and the adjoint), so it runs no more planes than the
// MPI has (see maxd_class). With separate weight tables for every row, the shift's fractions beside them and LDS
// addresses rebuilt per plane it was 119: FP32, 512 x 384 x 32, 4 views 119 us, now 108 (46 and
// 23 us one and two levels below, from 51 and 26); BF16, 1920 x 1080 x 64, 8 views 4442 us, now
// 4343.
template <int DT, int MAXD>
constexpr int grad_shift_keep() {
    if (MAXD <= 16 || (DT == HSGD_BF16 && MAXD == 32)) return 0;
    if (MAXD <= 32) return 16;
    if (MAXD == 40) return 12;
    if (MAXD == 48) return DT == HSGD_FP32 ? 8 : 10;
    return DT == HSGD_FP32 ? 4 : 6;
}
template <int DT, int MAXD>
constexpr int grad_shift_waves() {
    return grad_shift_keep<DT, MAXD>() > 0 ? 4 : 6;
}
template <int DT, int MAXD>
constexpr int grad_shift_tl() {
    if (grad_shift_keep<DT, MAXD>() == 0) return 6;
    return MAXD <= 40 ? 18 : MAXD == 48 ? 15 : 11;
}
template <int DT, int MAXD, bool MASKED, int KEEP = grad_shift_keep<DT, MAXD>(), int TL = grad_shift_tl<DT, MAXD>()>
__device__ __forceinline__ void grad_shift_tile(
    const void* __restrict__ mpi, int D, int H, int W, int N, const hsgd_warp* __restrict__ warps,
    const float* __restrict__ images, const float* __restrict__ dimg, const uint64_t* __restrict__ mask,
    int kcap, float inv_n, float4* __restrict__ slots, float* __restrict__ partials, int ntx, int tile,
    unsigned tid) {
    // horizontal halves, two buffers of the tile (one wave row of padding in front, so that
    // the row above is at a constant distance below for every wave)
    __shared__ f32x4 s_h[kSX + 2 * kSX * kSY];
    __shared__ uint64_t s_bits[kSY];
    __shared__ float sred[kSX * kSY / 64];
    __shared__ f32x4 s_w[MAXD];                             // per plane: tap weights
    __shared__ uint32_t s_code[(MAXD + 3) / 4][kSX * kSY];  // rank bytes of 4 planes per thread
    // Transmittance in front of the first kTL planes: these live longest (from the start of
    // the front-to-back scan to the end of the back-to-front one), so they go to LDS instead
    // of registers, which would otherwise spill to scratch memory (whose reloads wait for
    // every load in flight, the look-ahead included).
    constexpr int kTL = TL;
    __shared__ float s_T[kTL > 0 ? kTL : 1][kSX * kSY];
    const int view = tile % N;
    const int t2 = tile / N;
    const int tx = t2 % ntx, ty = t2 / ntx;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xl = tx * kOX - 1;                 // x of lane 0
    const int x = xl + lane, y = ty * kOY - 1 + wv;
    const bool ray = lane < kSX - 1 && (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H;
    const bool owner = lane >= 1 && lane < kSX - 1 && wv >= 1;
    const int HW = H * W;

    // Plane tables, one entry per lane z < MAXD (read per plane with v_readlane, feeding
    // scalar address arithmetic):
    //   lrow  byte offset, within plane z, of this wave's upper tap row y + iy clamped into
    //         the plane, | 1 if that row lies in the plane, | 2 if the row below it does,
    //         | 4 if the row below is the plane's first row (the upper one lies above it);
    //   lcol  the integer column shift times the voxel size (ix * s).
    // A wave's tap columns are then x + ix for its lanes' x.
    // The bilinear weights of each plane (lerp_taps' four; the adjoint's as well) go to LDS,
    // read per plane as broadcasts: a tap outside the plane reads 0, so they hold for every
    // row. Planes z >= D repeat plane D - 1 with zero weights.
    constexpr int S = Vox<DT>::kBytes;
    const int rowbytes = W * S;
    const int dlast = __builtin_amdgcn_readfirstlane(D - 1);    // last plane, wave-uniform
    int lrow = 0, lcol = 0;
    if (lane < MAXD) {
        const hsgd_warp& w = warps[(size_t)view * D + min(lane, dlast)];
        const int Y0 = y + w.iy;
        const bool in0 = (unsigned)Y0 < (unsigned)H, in1 = (unsigned)(Y0 + 1) < (unsigned)H;
        lrow = min(max(Y0, 0), H - 1) * rowbytes | (in0 ? 1 : 0) | (in1 ? 2 : 0) | (Y0 == -1 ? 4 : 0);
        // (a shift beyond the frame and its halo only ever reads padding; clamping it there
        // keeps every lane's byte offset from wrapping into the row)
        lcol = min(max(w.ix, -(W + 64)), W + 64) * S;
        const f32x4 none = {0.0f, 0.0f, 0.0f, 0.0f};
        const f32x4 wt = {1.0f - w.fy, w.fy, 1.0f - w.fx, w.fx};
        if (wv == 0) s_w[lane] = lane < D ? wt : none;
    }
    // (the LDS addresses read per plane stay in registers: rebuilt from constants, as the
    // compiler would, they cost vector instructions, which bound this kernel)
    lds_f32x4* wts = (lds_f32x4*)s_w;
    lds_f32x4* halves = (lds_f32x4*)s_h + tid;              // the row above's; the own row's is kSX further
    asm volatile("" : "+v"(wts), "+v"(halves));
    const unsigned xs = (unsigned)x * (unsigned)S;                // wraps when x < 0: outside
    __syncthreads();

    // Both scans run over MAXD planes; planes z >= D sample plane D-1 with zero weights (a
    // transparent plane) and select nothing. The taps of plane z +- kAhead are loaded while
    // plane z is processed (see the end of each scan), and a scheduling fence per plane
    // keeps that look-ahead (and the register footprint) fixed. The second scan samples the
    // planes again (all but the last kKeep, below) instead of keeping them in registers: that
    // keeps the kernel small enough for several workgroups per CU, which hides the per-plane
    // barrier.
    struct Taps2 {
        typename Vox<DT>::Raw t00, t01;   // taps of rows y0 and y0 + 1, as stored (right-hand taps come from lane + 1)
        unsigned row;      // in-plane byte offset of the upper tap row, with lrow's flags
        unsigned col;      // the column shift in bytes (ix * s), wave-uniform
        // byte offset of this lane's tap column in a row: (x + ix) * s
        __device__ unsigned off(unsigned xs_) const { return xs_ + col; }
    };
    // zstride: the plane stride in voxels (H W), passed laundered to the second scan so that
    // the compiler cannot prove its loads equal the first scan's and keep those alive instead.
    // Taps come through buffer resources over the two tap rows: a column outside the
    // plane, or a whole row outside it, reads as 0 -- the zero padding -- so neither the
    // addresses nor the weights need per-lane range checks.
    auto fetch = [&](int z, int zstride) {
        Taps2 f;
        f.row = (unsigned)rl(lrow, z);
        f.col = (unsigned)rl(lcol, z);
        const char* plane = reinterpret_cast<const char*>(mpi) + (size_t)((unsigned)min(z, dlast) * (unsigned)zstride) * S;
        const char* row0 = plane + (f.row & ~7u);
        const char* row1 = row0 + ((f.row & 4u) ? 0u : (unsigned)rowbytes);
        const unsigned off = f.off(xs);
        f.t00 = Vox<DT>::load_raw(row_rsrc(row0, (f.row & 1u) ? rowbytes : 0), off);
        f.t01 = Vox<DT>::load_raw(row_rsrc(row1, (f.row & 2u) ? rowbytes : 0), off);
        return f;
    };
    // the owned cell's mask word (the cell is the upper tap row's voxel of this lane's
    // column), through a buffer resource over the cell's mask row: a cell outside the
    // plane reads 0, i.e. unselected
    auto fetch_mask = [&](const Taps2& f) -> uint64_t {
        if (!MASKED) return 0;
        const char* row = reinterpret_cast<const char*>(mask) + (f.row & ~7u) / (unsigned)(S / 8);
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(row_rsrc(row, (f.row & 1u) ? W * 8 : 0),
                                                            f.off(xs) / (unsigned)(S / 8), 0, 0);
        return ((uint64_t)v[1] << 32) | v[0];
    };
    auto sample = [&](const f32x4& wt, const Taps2& f) {
        const float4 a0 = Vox<DT>::decode(f.t00), a1 = Vox<DT>::decode(f.t01);
        float4 s;
        s.x = lerp_taps(a0.x, a1.x, wt);
        s.y = lerp_taps(a0.y, a1.y, wt);
        s.z = lerp_taps(a0.z, a1.z, wt);
        s.w = lerp_taps(a0.w, a1.w, wt);
        return s;
    };
    // planes of taps in flight: BF16 taps stay as stored (half the registers) until used,
    // which leaves room for a third plane; FP32 taps fill the same registers with two
    constexpr int kAhead = DT == HSGD_BF16 ? 3 : 2;
    // The samples of the last kKeep planes of the front-to-back scan stay in registers for
    // the back-to-front scan, which starts with them: 2 kKeep fewer row loads per wave (the
    // kernel then runs at 4 waves per SIMD, see grad_shift_keep).
    constexpr int kKeep = KEEP;
    float4 Sk[kKeep > 0 ? kKeep : 1];
    // Every plane iteration starts with a branch on an opaque, always-true value: the block
    // boundaries keep the compiler from moving each plane's setup code across planes (which
    // would keep all of it alive at once).
    int go = 1;

    float Ts[MAXD];
    uint32_t code = 0;                           // rank + 1 of the owned cell (or 0) per plane,
                                                 // 4 planes per word, flushed to s_code
    uint64_t own_bits = 0;                       // planes where an owned cell of this wave is selected
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    {
        Taps2 q[kAhead];
        uint64_t qm[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (i < MAXD) {
                q[i] = fetch(i, HW);
                qm[i] = fetch_mask(q[i]);
            }
#pragma unroll
        for (int z = 0; z < MAXD; ++z) {
            asm volatile("" : "+s"(go));
            if (!go) break;
            const Taps2 cur = q[z % kAhead];
            const uint64_t m = qm[z % kAhead];
            if (z + kAhead < MAXD) {
                q[z % kAhead] = fetch(z + kAhead, HW);
                qm[z % kAhead] = fetch_mask(q[z % kAhead]);
            }
            const f32x4 wt = wts[z];
            const float4 s = sample(wt, cur);
            if (kKeep > 0 && z >= MAXD - kKeep) Sk[z >= MAXD - kKeep ? z - (MAXD - kKeep) : 0] = s;
            if (z < kTL)
                s_T[z < kTL ? z : 0][tid] = T;
            else
                Ts[z] = T;
            const float wgt = T * s.w;
            c0 = __builtin_fmaf(wgt, s.x, c0);
            c1 = __builtin_fmaf(wgt, s.y, c1);
            c2 = __builtin_fmaf(wgt, s.z, c2);
            T *= 1.0f - s.w;
            // branch-free: n = rank + 1 of the owned cell's plane z if selected, else 0. With the
            // mask shifted so that bit z is the sign, the bits left count rank + 1. (A cell
            // outside the plane has a zero mask word; without a mask, check the range.)
            bool sel = owner && z < D;
            uint32_t n = z + 1;
            if (MASKED) {
                const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
                const uint32_t t = z < 32 ? lo << (31 - z) : hi << (63 - z);
                n = __popc(t) + (z < 32 ? 0 : __popc(lo));
                sel = sel && (int)t < 0;
            } else {
                sel = sel && (cur.row & 1u) && cur.off(xs) < (unsigned)rowbytes;
            }
            sel = sel && n <= (uint32_t)kcap;
            code |= (sel ? n : 0u) << ((z & 3) * 8);
            if ((z & 3) == 3 || z == MAXD - 1) {
                s_code[z >> 2][tid] = code;
                code = 0;
            }
            if (__builtin_amdgcn_ballot_w64(sel)) own_bits |= 1ull << z;
            __builtin_amdgcn_sched_barrier(0);
        }
        // The look-ahead loads are consumed on the path out of the loop as well, so that
        // each is issued before its plane's branch rather than sunk to its use planes later.
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            asm volatile("" ::"v"(q[i].t00.x), "v"(q[i].t01.x), "v"((uint32_t)qm[i]));
    }
    // planes where the wave below has selected cells: it needs this wave's adjoints
    if (lane == 0) s_bits[wv] = own_bits;
    __syncthreads();
    uint64_t below_bits = 0;
    if (wv + 1 < kSY) {
        const uint64_t b = s_bits[wv + 1];
        below_bits = ((uint64_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    }
    const uint64_t need_bits = own_bits | below_bits;

    float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f, sq = 0.0f;
    if (ray) {
        // (x again from the lane's tap offset, so that x itself need not stay live)
        const size_t pix = ((size_t)view * H + y) * W + (int)xs / S;
        if (images) {
            const float d0 = c0 - images[3 * pix + 0];
            const float d1 = c1 - images[3 * pix + 1];
            const float d2 = c2 - images[3 * pix + 2];
            if (owner) sq = __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
            g0 = d0 * inv_n;
            g1 = d1 * inv_n;
            g2 = d2 * inv_n;
        }
        if (dimg) {
            g0 = dimg[3 * pix + 0];
            g1 = dimg[3 * pix + 1];
            g2 = dimg[3 * pix + 2];
        }
    }
    float b0 = 0.0f, b1 = 0.0f, b2 = 0.0f;   // composite behind plane z
    float4* __restrict__ vslots = slots + (size_t)view * kcap * HW;
    // launder what the second scan derives its taps from, so that nothing computed per
    // plane in the first scan is kept alive for it
    int HW2 = HW;
    asm volatile("" : "+s"(HW2), "+v"(lrow), "+v"(lcol));
    uint32_t rcode = 0;
    {
        // (the first planes sampled are those below the kept ones: their loads run while the
        // kept planes are processed)
        Taps2 q[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (i + kKeep < MAXD) q[i] = fetch(MAXD - 1 - kKeep - i, HW2);
#pragma unroll
        for (int zz = 0; zz < MAXD; ++zz) {
            const int z = MAXD - 1 - zz;
            asm volatile("" : "+s"(go));
            if (!go) break;
            Taps2 cur;
            float4 s;
            const f32x4 wt = wts[z];
            if (zz < kKeep) {
                cur.row = (unsigned)rl(lrow, z);
                cur.col = (unsigned)rl(lcol, z);
                s = Sk[zz < kKeep ? kKeep - 1 - zz : 0];
            } else {
                const int zk = zz - kKeep;
                cur = q[zk % kAhead];
                if (zz + kAhead < MAXD) q[zk % kAhead] = fetch(z - kAhead, HW2);
                s = sample(wt, cur);
            }
            if ((z & 3) == 3 || z == MAXD - 1) rcode = s_code[z >> 2][tid];
            lds_f32x4* const up = halves + (z & 1) * (kSX * kSY);
            lds_f32x4* const own = up + kSX;
            // the colour of plane z against the composite behind it: the alpha adjoint's
            // factor and the step of the behind composite, B <- B + a (c - B)
            const float d0 = s.x - b0, d1 = s.y - b1, d2 = s.z - b2;
            if ((need_bits >> z) & 1) {
                const float Tz = z < kTL ? s_T[z < kTL ? z : 0][tid] : Ts[z];
                const float ca = s.w * Tz;
                float4 a;
                a.x = g0 * ca;
                a.y = g1 * ca;
                a.z = g2 * ca;
                a.w = Tz * __builtin_fmaf(g2, d2, __builtin_fmaf(g1, d1, g0 * d0));
                // horizontal half of the transposed bilinear: this ray (1 - fx) and the
                // ray to the left (fx) both touch the owned cell's row
                const float gx = wt.z, fx = wt.w;
                f32x4 h;
                h.x = __builtin_fmaf(a.x, gx, lane_from_prev(a.x) * fx);
                h.y = __builtin_fmaf(a.y, gx, lane_from_prev(a.y) * fx);
                h.z = __builtin_fmaf(a.z, gx, lane_from_prev(a.z) * fx);
                h.w = __builtin_fmaf(a.w, gx, lane_from_prev(a.w) * fx);
                *own = h;
            }
            b0 = __builtin_fmaf(s.w, d0, b0);
            b1 = __builtin_fmaf(s.w, d1, b1);
            b2 = __builtin_fmaf(s.w, d2, b2);
            __syncthreads();
            if ((own_bits >> z) & 1) {
                const int rc = (int)((rcode >> ((z & 3) * 8)) & 0xffu);
                if (rc) {
                    // this row's and the row above's horizontal halves, both from LDS (the
                    // own half is not kept in registers across the barrier)
                    const f32x4 h = *own, hu = *up;
                    const float gy = wt.x, fy = wt.y;
                    float4 c;
                    c.x = __builtin_fmaf(hu.x, fy, h.x * gy);
                    c.y = __builtin_fmaf(hu.y, fy, h.y * gy);
                    c.z = __builtin_fmaf(hu.z, fy, h.z * gy);
                    c.w = __builtin_fmaf(hu.w, fy, h.w * gy);
                    // slot (rank, cell): the cell's byte offset in an FP32 RGBA plane is its
                    // tap offsets scaled from the storage's voxel size to 16 bytes
                    const unsigned cell16 = ((cur.row & ~7u) + cur.off(xs)) * (unsigned)(16 / S);
                    const unsigned idx = (unsigned)(rc - 1) * (unsigned)HW * 16u + cell16;
                    *reinterpret_cast<float4*>(reinterpret_cast<char*>(vslots) + idx) = c;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (i + kKeep < MAXD) asm volatile("" ::"v"(q[i].t00.x), "v"(q[i].t01.x));
    }
    if (partials) {
        const float tot = block_sum(sq, sred);
        if (threadIdx.x == 0) partials[tile] = tot;
    }
}

// Waves per SIMD as grad_shift_waves gives them, without spills (the first planes'
// transmittance is kept in LDS).
template <int DT, int MAXD, bool MASKED>
__global__ __launch_bounds__(kSX * kSY) __attribute__((amdgpu_waves_per_eu(grad_shift_waves<DT, MAXD>()))) void k_grad_shift(
    const void* __restrict__ mpi, int D, int H, int W, int N, const hsgd_warp* __restrict__ warps,
    const float* __restrict__ images, const float* __restrict__ dimg, const uint64_t* __restrict__ mask,
    int kcap, float inv_n, float4* __restrict__ slots, float* __restrict__ partials, int ntx) {
    grad_shift_tile<DT, MAXD, MASKED>(mpi, D, H, W, N, warps, images, dimg, mask, kcap, inv_n, slots, partials,
                                      ntx, xcd_tile(flat_block(), flat_blocks()), threadIdx.x);
}

// ------------------------------------------------------------------------------------
// render, translation warps: the gradient kernel's front-to-back scan on its own
// ------------------------------------------------------------------------------------
// One workgroup = 63 x 8 rays of one view (lane 63 of each wave only supplies the right-
// hand taps of lane 62): per plane two row loads through buffer resources (hardware zero
// padding), per-wave tap weights from an LDS table, the right column through DPP, two
// planes of loads in flight.
template <int DT, int MAXD>
__global__ __launch_bounds__(kSX * kSY) void k_render_shift(const void* __restrict__ mpi, int D, int H, int W,
                                                            int N, const hsgd_warp* __restrict__ warps,
                                                            const float* __restrict__ images,
                                                            float* __restrict__ out_rgb,
                                                            float* __restrict__ partials, int ntx) {
    __shared__ float4 s_w[kSY][MAXD];
    __shared__ float sred[kSX * kSY / 64];
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int view = tile % N;
    const int t2 = tile / N;
    const int tx = t2 % ntx, ty = t2 / ntx;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xl = tx * kShiftRX;
    const int x = xl + lane, y = ty * kShiftRY + wv;
    const bool ray = lane < kShiftRX && x < W && y < H;
    int lx = 0, ly = 0;
    if (lane < MAXD) {
        float4 wt = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lane < D) {
            const hsgd_warp& w = warps[(size_t)view * D + lane];
            lx = w.ix;
            ly = w.iy;
            const int Y0 = y + ly;
            const float gy = (unsigned)Y0 < (unsigned)H ? 1.0f - w.fy : 0.0f;
            const float hy = (unsigned)(Y0 + 1) < (unsigned)H ? w.fy : 0.0f;
            wt = make_float4(gy, hy, 1.0f - w.fx, w.fx);
        }
        s_w[wv][lane] = wt;
    }
    __syncthreads();
    const int HW = H * W;
    const int rb = W * Vox<DT>::kBytes;
    struct Taps2 {
        float4 t00, t01;
    };
    auto fetch = [&](int z) {
        Taps2 f;
        const int ix = rl(lx, z), iy = rl(ly, z);
        const int zb = min(z, D - 1) * HW;
        const int Y0 = y + iy;
        const unsigned off = (unsigned)(x + ix) * (unsigned)Vox<DT>::kBytes;
        const bool r0 = (unsigned)Y0 < (unsigned)H, r1 = (unsigned)(Y0 + 1) < (unsigned)H;
        f.t00 = Vox<DT>::load_buf(row_rsrc(Vox<DT>::row_ptr(mpi, zb + (r0 ? Y0 : 0) * W), r0 ? rb : 0), off);
        f.t01 = Vox<DT>::load_buf(row_rsrc(Vox<DT>::row_ptr(mpi, zb + (r1 ? Y0 + 1 : 0) * W), r1 ? rb : 0), off);
        return f;
    };
    constexpr int kAhead = 2;
    int go = 1;
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    {
        Taps2 q[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (i < MAXD) q[i] = fetch(i);
#pragma unroll
        for (int z = 0; z < MAXD; ++z) {
            asm volatile("" : "+v"(go));
            if (!__builtin_amdgcn_readfirstlane(go)) break;
            const Taps2 f = q[z % kAhead];
            if (z + kAhead < MAXD) q[z % kAhead] = fetch(z + kAhead);
            const float4 wt = s_w[wv][z];
            float4 s;
            s.x = lerp_taps(f.t00.x, f.t01.x, wt);
            s.y = lerp_taps(f.t00.y, f.t01.y, wt);
            s.z = lerp_taps(f.t00.z, f.t01.z, wt);
            s.w = lerp_taps(f.t00.w, f.t01.w, wt);
            const float wgt = T * s.w;
            c0 = __builtin_fmaf(wgt, s.x, c0);
            c1 = __builtin_fmaf(wgt, s.y, c1);
            c2 = __builtin_fmaf(wgt, s.z, c2);
            T *= 1.0f - s.w;
            __builtin_amdgcn_sched_barrier(0);
        }
        // keep the look-ahead loads ahead of each plane's branch (see the gradient kernel)
        asm volatile("" ::"v"(q[0].t00.x), "v"(q[0].t01.x), "v"(q[1].t00.x), "v"(q[1].t01.x));
    }
    float sq = 0.0f;
    if (ray) {
        const size_t pix = ((size_t)view * H + y) * W + x;
        if (out_rgb) {
            out_rgb[3 * pix + 0] = c0;
            out_rgb[3 * pix + 1] = c1;
            out_rgb[3 * pix + 2] = c2;
        }
        if (partials) {
            const float d0 = c0 - images[3 * pix + 0];
            const float d1 = c1 - images[3 * pix + 1];
            const float d2 = c2 - images[3 * pix + 2];
            sq = __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
        }
    }
    if (partials) {
        const float tot = block_sum(sq, sred);
        if (threadIdx.x == 0) partials[tile] = tot;
    }
}

// The same for calls of many waves: a wave takes R rows of rays. Bound by the L1's rate on
// unaligned 16-byte taps and by vector instructions: a row of the plane is loaded once for the
// two rows of rays it lies between instead of twice, and the plane's addresses and weights are
// prepared once for R rows. FP32, 512 x 384 x 32, 18 views: 175 us by single rows, 132 at R = 2,
// 118 at 4, 114 at 8; BF16, 1440 x 1080 x 64, 5 views: 802, 679, 638, 570.
template <int DT, int R>
__global__ __launch_bounds__(64 * kRenderWaves) void k_render_shift_rows(
    const void* __restrict__ mpi, int D, int H, int W, int N, const hsgd_warp* __restrict__ warps,
    const float* __restrict__ images, float* __restrict__ out_rgb, float* __restrict__ partials, int ntx) {
    __shared__ f32x4 s_w[kMaxD];
    __shared__ float sred[kRenderWaves];
    constexpr int S = Vox<DT>::kBytes;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int view = tile % N;
    const int t2 = tile / N;
    const int tx = t2 % ntx, ty = t2 / ntx;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = tx * kShiftRX + lane, y = (ty * kRenderWaves + wv) * R;
    // per plane, one entry per lane: the integer shift (clamped where every tap is padding
    // anyway, so that no offset wraps into the plane)
    const hsgd_warp& w = warps[(size_t)view * D + min(lane, D - 1)];
    const int lx = min(max(w.ix, -(W + 64)), W + 64) * S;
    const int ly = min(max(w.iy, -(H + 64)), H + 64);
    if (wv == 0) s_w[lane] = f32x4{1.0f - w.fy, w.fy, 1.0f - w.fx, w.fx};
    __syncthreads();
    const int rowbytes = W * S;
    const unsigned xs = (unsigned)x * (unsigned)S;
    struct Rows {
        typename Vox<DT>::Raw t[R + 1];
    };
    // the R + 1 tap rows, through buffer resources: a column outside the plane, or a whole
    // row outside it (a resource of no bytes), reads as 0
    auto fetch = [&](int z) {
        Rows f;
        const int Y0 = y + rl(ly, z);
        const unsigned off = xs + (unsigned)rl(lx, z);
        const uint64_t plane = (uint64_t)(uintptr_t)mpi + (uint64_t)((unsigned)z * (unsigned)(H * W)) * S;
        uint64_t row = plane + (uint64_t)((int64_t)Y0 * rowbytes);
#pragma unroll
        for (int r = 0; r <= R; ++r) {
            const bool in = (unsigned)(Y0 + r) < (unsigned)H;
            f.t[r] = Vox<DT>::load_raw(row_rsrc(reinterpret_cast<const char*>(row), in ? rowbytes : 0), off);
            row += (unsigned)rowbytes;
        }
        return f;
    };
    float T[R], c0[R], c1[R], c2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        T[r] = 1.0f;
        c0[r] = c1[r] = c2[r] = 0.0f;
    }
    auto blend = [&](int z, const Rows& f) {
        const f32x4 wt = s_w[z];
        float4 a0 = Vox<DT>::decode(f.t[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float4 a1 = Vox<DT>::decode(f.t[r + 1]);
            const float alpha = lerp_taps(a0.w, a1.w, wt);
            const float wgt = T[r] * alpha;
            c0[r] = __builtin_fmaf(wgt, lerp_taps(a0.x, a1.x, wt), c0[r]);
            c1[r] = __builtin_fmaf(wgt, lerp_taps(a0.y, a1.y, wt), c1[r]);
            c2[r] = __builtin_fmaf(wgt, lerp_taps(a0.z, a1.z, wt), c2[r]);
            T[r] *= 1.0f - alpha;
            a0 = a1;
        }
    };
    // the next plane's rows are in flight while a plane is blended
    Rows q0 = fetch(0);
    for (int z = 0; z < D; z += 2) {
        const Rows q1 = fetch(min(z + 1, D - 1));
        __builtin_amdgcn_sched_barrier(0);
        blend(z, q0);
        __builtin_amdgcn_sched_barrier(0);
        if (z + 1 >= D) break;
        q0 = fetch(min(z + 2, D - 1));
        __builtin_amdgcn_sched_barrier(0);
        blend(z + 1, q1);
        __builtin_amdgcn_sched_barrier(0);
    }
    float sq = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (lane >= kShiftRX || x >= W || y + r >= H) continue;
        const size_t pix = ((size_t)view * H + y + r) * W + x;
        if (out_rgb) {
            out_rgb[3 * pix + 0] = c0[r];
            out_rgb[3 * pix + 1] = c1[r];
            out_rgb[3 * pix + 2] = c2[r];
        }
        if (partials) {
            const float d0 = c0[r] - images[3 * pix + 0];
            const float d1 = c1[r] - images[3 * pix + 1];
            const float d2 = c2[r] - images[3 * pix + 2];
            sq += __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
        }
    }
    if (partials) {
        const float tot = block_sum(sq, sred);
        if (threadIdx.x == 0) partials[tile] = tot;
    }
}

__global__ __launch_bounds__(256) void k_fill_zero(float4* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = i; j < n; j += stride) p[j] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// One thread per pixel: for each selected plane (rank r < kcap) sum the view slices, then
// apply the clamped descent step in place and/or write the gradient out. With shift
// warps, view v wrote voxel (z, p) only if p lies in v's owner coverage for plane z;
// outside it no ray of v reaches the voxel and the slot is not read. Workgroup 0 also
// reduces the loss partials of the gradient kernel (fixed order, FP64).
// Workgroup blk of the update over one MPI level (256 / RS pixels: with RS > 1 the RS
// groups of 256 / RS threads take the selected planes of rank r = group (mod RS) of the
// same pixels, so the ranks of a pixel are updated in parallel); s_off is LDS for the
// [nslices][D] shifts. Every thread of the 256-thread workgroup calls it.
template <int DT, bool SHIFT, int RS = 1>
__device__ __forceinline__ void update_block(void* __restrict__ mpi, int D, int H, int W,
                                             const uint64_t* __restrict__ mask, int kcap,
                                             const float4* __restrict__ slots, int nslices,
                                             const hsgd_warp* __restrict__ warps, int cover_w,
                                             int cover_h, float lr_rgb, float lr_a, int do_update,
                                             float4* __restrict__ grad_out,
                                             const float* __restrict__ partials, int64_t nparts,
                                             double loss_scale, float* __restrict__ out_loss, float prior,
                                             int blk, int2* __restrict__ s_off) {
    if (SHIFT) {
        for (int i = threadIdx.x; i < nslices * D; i += blockDim.x) s_off[i] = make_int2(warps[i].ix, warps[i].iy);
        __syncthreads();
    }
    if (out_loss && blk == 0) {
        __shared__ double sh[256];
        double acc = 0.0;
        for (int64_t i = threadIdx.x; i < nparts; i += 256) acc += (double)partials[i];
        sh[threadIdx.x] = acc;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) *out_loss = (float)(sh[0] * loss_scale);
    }
    static_assert(256 % RS == 0, "whole pixel groups");
    constexpr int kPix = 256 / RS;
    const int HW = H * W;
    const int p = blk * kPix + (int)(threadIdx.x % kPix);
    const int q = (int)(threadIdx.x / kPix);
    if (p >= HW) return;
    const int Y = p / W, X = p - Y * W;
    const uint64_t m = (mask ? mask[p] : ~0ull) & plane_bits(D);
    // Sum of the view slices of rank r (plane z), in view order. The loads of 8 views are
    // issued together through one buffer resource per view slice: a view whose owners do
    // not cover the cell (its slot holds stale data), or past the last view, gets an offset
    // outside the resource and reads 0 without touching memory.
    const unsigned slice_bytes = (unsigned)kcap * (unsigned)HW * 16u;
    auto grad_of = [&](int z, int r) {
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
        const unsigned off = ((unsigned)r * (unsigned)HW + (unsigned)p) * 16u;
        for (int v0 = 0; v0 < nslices; v0 += 8) {
            float4 t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int v = min(v0 + j, nslices - 1);
                bool ok = v0 + j < nslices;
                if (SHIFT) {
                    const int2 o = s_off[v * D + z];
                    ok = ok && (unsigned)(X - o.x) < (unsigned)cover_w && (unsigned)(Y - o.y) < (unsigned)cover_h;
                }
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float4*>(slots + (size_t)v * kcap * HW), (short)0, (int)slice_bytes, kBufWord3);
                const auto u = __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? off : 0xfffffff0u, 0, 0);
                t[j] = make_float4(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]),
                                   __uint_as_float(u[3]));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                g.x += t[j].x;
                g.y += t[j].y;
                g.z += t[j].z;
                g.w += t[j].w;
            }
        }
        return g;
    };
    uint64_t b = m;
    int r = 0;
    while (b && r < kcap) {
        const int z = __ffsll((unsigned long long)b) - 1;
        b &= b - 1;
        const int rank = r++;
        if (RS > 1 && rank % RS != q) continue;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (do_update || prior != 0.0f) v = Vox<DT>::load(mpi, z * HW + p);   // in flight with the slices
        float4 g = grad_of(z, rank);
        if (prior != 0.0f) {
            // sparsity prior: d/da log(1.5 - |0.5 - a|) = sign(0.5 - a) / (1.5 - |0.5 - a|)
            const float d = 0.5f - v.w;
            const float sg = d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f);
            g.w = __builtin_fmaf(prior, sg / (1.5f - fabsf(d)), g.w);
        }
        if (grad_out) grad_out[(size_t)z * HW + p] = g;
        if (do_update) {
            v.x = fminf(fmaxf(__builtin_fmaf(-lr_rgb, g.x, v.x), 0.0f), 1.0f);
            v.y = fminf(fmaxf(__builtin_fmaf(-lr_rgb, g.y, v.y), 0.0f), 1.0f);
            v.z = fminf(fmaxf(__builtin_fmaf(-lr_rgb, g.z, v.z), 0.0f), 1.0f);
            v.w = fminf(fmaxf(__builtin_fmaf(-lr_a, g.w, v.w), 0.0f), 1.0f);
            Vox<DT>::store(mpi, z * HW + p, v);
        }
    }
}

// the selected planes of a pixel split over 4 thread groups (64 pixels per workgroup)
constexpr int kUpdateRS = 4;
template <int DT, bool SHIFT>
__global__ __launch_bounds__(256) void k_update(void* __restrict__ mpi, int D, int H, int W,
                                                const uint64_t* __restrict__ mask, int kcap,
                                                const float4* __restrict__ slots, int nslices,
                                                const hsgd_warp* __restrict__ warps, int cover_w,
                                                int cover_h, float lr_rgb, float lr_a, int do_update,
                                                float4* __restrict__ grad_out,
                                                const float* __restrict__ partials, int64_t nparts,
                                                double loss_scale, float* __restrict__ out_loss, float prior) {
    extern __shared__ int2 s_off[];   // [nslices][D] (ix, iy) when SHIFT
    update_block<DT, SHIFT, kUpdateRS>(mpi, D, H, W, mask, kcap, slots, nslices, warps, cover_w, cover_h, lr_rgb, lr_a,
                            do_update, grad_out, partials, nparts, loss_scale, out_loss, prior, blockIdx.x, s_off);
}

// ------------------------------------------------------------------------------------
// hierarchy
// ------------------------------------------------------------------------------------
// Source pair and fraction of output coordinate x of a 2x upsampling along an axis of n
// source samples: the sample point (x + 1/2) / 2 - 1/2, clamped to [0, n - 1].
__device__ __forceinline__ void up_axis(int x, int n, int& i0, int& i1, float& f) {
    const float sx = fminf(fmaxf((x + 0.5f) * 0.5f - 0.5f, 0.0f), (float)(n - 1));
    i0 = (int)sx;
    i1 = min(i0 + 1, n - 1);
    f = sx - i0;
}

struct UpW {
    float w00, w10, w01, w11;
};
__device__ __forceinline__ UpW up_weights(float fx, float fy) {
    return UpW{(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy};
}
// The bilinear blend of taps a (x0, y0), b (x1, y0), c (x0, y1), d (x1, y1): the one
// expression every upsampling path evaluates, so that they agree bit for bit.
__device__ __forceinline__ float4 up_blend(const UpW& w, const float4& a, const float4& b, const float4& c,
                                           const float4& d) {
    auto f = [&](float a_, float b_, float c_, float d_) {
        return __builtin_fmaf(w.w11, d_, __builtin_fmaf(w.w01, c_, __builtin_fmaf(w.w10, b_, w.w00 * a_)));
    };
    return make_float4(f(a.x, b.x, c.x, d.x), f(a.y, b.y, c.y, d.y), f(a.z, b.z, c.z, d.z), f(a.w, b.w, c.w, d.w));
}

// The four source taps of output voxel i of plane z of the 2x upsampling of a [D][h][w]
// level, and their weights.
template <int DT>
struct UpTaps {
    float4 a, b, c, d;
    UpW w;
};
template <int DT>
__device__ __forceinline__ UpTaps<DT> upsample_taps(const void* __restrict__ src, int h, int w, int z, int i) {
    const int W2 = 2 * w;
    const int x = i % W2, y = i / W2;
    int x0, x1, y0, y1;
    float fx, fy;
    up_axis(x, w, x0, x1, fx);
    up_axis(y, h, y0, y1, fy);
    const int base = z * h * w;
    UpTaps<DT> t;
    t.a = Vox<DT>::load(src, base + y0 * w + x0);
    t.b = Vox<DT>::load(src, base + y0 * w + x1);
    t.c = Vox<DT>::load(src, base + y1 * w + x0);
    t.d = Vox<DT>::load(src, base + y1 * w + x1);
    t.w = up_weights(fx, fy);
    return t;
}

// Blends the taps, stores output voxel i of plane z and returns the value as stored (BF16:
// rounded).
template <int DT>
__device__ __forceinline__ float4 upsample_store(const UpTaps<DT>& t, void* __restrict__ dst, int H2W2, int z,
                                                 int i) {
    const float4 o = up_blend(t.w, t.a, t.b, t.c, t.d);
    Vox<DT>::store(dst, z * H2W2 + i, o);
    return Vox<DT>::stored(o);
}

// Output voxel i of plane z of the 2x upsampling of a [D][h][w] level; returns the value
// as stored, or 0 past the level's end.
template <int DT>
__device__ __forceinline__ float4 upsample_voxel(const void* __restrict__ src, int h, int w,
                                                 void* __restrict__ dst, int z, int i) {
    if (i >= 4 * w * h) return make_float4(0.f, 0.f, 0.f, 0.f);
    return upsample_store<DT>(upsample_taps<DT>(src, h, w, z, i), dst, 4 * w * h, z, i);
}

template <int DT>
__global__ __launch_bounds__(256) void k_upsample(const void* __restrict__ src, int h, int w,
                                                  void* __restrict__ dst) {
    upsample_voxel<DT>(src, h, w, dst, blockIdx.y, blockIdx.x * blockDim.x + threadIdx.x);
}

constexpr int kUpWaves = 4;

// Planes a wave of the fused kernels below loads together: its planes in whole groups.
constexpr int up_group(int planes) {
    return planes < 4 ? planes : planes % 4 == 0 ? 4 : planes % 3 == 0 ? 3 : 5;
}

// Upsampling fused with the first selection at the new level, for levels of few
// workgroups. A block covers 64 output pixels (lane = pixel) and its four waves split the
// planes: each upsamples and stores a
// quarter of them and puts the alpha it stored (the storage-rounded value) in LDS; the
// first wave then scores every plane of its pixel front to back and writes the mask, which
// equals what k_select computes from the stored level. Splitting the planes shortens each
// thread's chain of dependent tap loads and gives the small levels four times the waves.
template <int DT, int MAXD>
__global__ __launch_bounds__(64 * kUpWaves) void k_upsample_select(const void* __restrict__ src, int D, int h,
                                                                   int w, void* __restrict__ dst, int k,
                                                                   float tau, int rule,
                                                                   uint64_t* __restrict__ mask) {
    constexpr int kPW = (MAXD + kUpWaves - 1) / kUpWaves;   // planes per wave
    constexpr int kG = up_group(kPW);                        // tap loads of kG planes in flight together
    static_assert(kPW % kG == 0, "whole load groups");
    __shared__ float s_a[kUpWaves * kPW][64];
    const int n = 4 * w * h;
    const int lane = threadIdx.x & 63;
    const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = blockIdx.x * 64 + lane;
    if (i < n) {
#pragma unroll
        for (int j0 = 0; j0 < kPW; j0 += kG) {
            // plane index clamped, so the loads need no guard
            UpTaps<DT> t[kG];
#pragma unroll
            for (int j = 0; j < kG; ++j) t[j] = upsample_taps<DT>(src, h, w, min(q * kPW + j0 + j, D - 1), i);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                const int z = q * kPW + j0 + j;
                if (z < D) s_a[z][lane] = upsample_store<DT>(t[j], dst, n, z, i).w;
            }
        }
    }
    __syncthreads();
    if (q == 0 && i < n) {
        float A[MAXD];
        float T = 1.0f;
#pragma unroll
        for (int z = 0; z < MAXD; ++z)
            if (z < D) A[z] = score_step(s_a[z][lane], T);
        mask[i] = topk_bits<MAXD>(A, D, k, tau, rule);
    }
}

// Upsampling fused with the first selection at the new level, for large levels. A
// workgroup takes one source row Y and 62 source columns (lane = source column X = X0 - 1 + lane; lanes 0 and 63 only
// supply taps to their neighbours) and writes the 2 x 2 output voxels of each of its owner
// columns: per plane it loads source rows Y - 1, Y and Y + 1 (clamped) of its column and
// takes the columns X - 1 and X + 1 from the neighbouring lanes, so a loaded voxel serves
// four outputs. The taps, weights and blend of every output are those of upsample_taps
// (the same source voxels, the same expression). The four waves split the planes and put
// the alpha they stored (storage-rounded) in LDS; then each wave scores and selects a
// quarter of the 248 output pixels front to back, as k_select does on the stored level.
// Below this many workgroups (8 per CU) the 2 x 2 kernel has too few waves to hide its
// longer per-wave work, and the per-pixel kernel is the faster one.
constexpr int64_t kUpBlkMinGroups = 2048;
constexpr int kUpPix = 4 * kUpCols;       // output pixels per workgroup (2 rows x 124)

// alpha as the selection reads it back from LDS: FP32, or the stored BF16 bits (exact)
template <int DT>
struct UpAlpha {
    using T = float;
    static __device__ __forceinline__ T put(float a) { return a; }
    static __device__ __forceinline__ float get(T v) { return v; }
};
template <>
struct UpAlpha<HSGD_BF16> {
    using T = uint16_t;
    static __device__ __forceinline__ T put(float a) { return (uint16_t)(__float_as_uint(a) >> 16); }
    static __device__ __forceinline__ float get(T v) { return __uint_as_float((uint32_t)v << 16); }
};

__device__ __forceinline__ float4 lane_prev4(const float4& v) {
    return make_float4(lane_from_prev(v.x), lane_from_prev(v.y), lane_from_prev(v.z), lane_from_prev(v.w));
}
__device__ __forceinline__ float4 lane_next4(const float4& v) {
    return make_float4(lane_from_next(v.x), lane_from_next(v.y), lane_from_next(v.z), lane_from_next(v.w));
}
__device__ __forceinline__ float4 pick4(bool c, const float4& a, const float4& b) {
    return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}

// Block bx of source row Y; every thread of the workgroup calls it.
template <int DT, int MAXD>
__device__ __forceinline__ void upsample_select_block(const void* __restrict__ src, int D, int h, int w,
                                                      void* __restrict__ dst, int k, float tau, int rule,
                                                      uint64_t* __restrict__ mask, int bx, int Y,
                                                      typename UpAlpha<DT>::T (*__restrict__ s_a)[kUpPix]) {
    constexpr int kPW = (MAXD + kUpWaves - 1) / kUpWaves;   // planes per wave
    constexpr int kG = up_group(kPW);                        // planes of loads in flight
    static_assert(kPW % kG == 0, "whole load groups");
    const int lane = threadIdx.x & 63;
    const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int X = bx * kUpCols - 1 + lane;
    const int Xc = min(max(X, 0), w - 1);
    const bool own = lane >= 1 && lane <= kUpCols && X < w;
    const int hw = h * w, W2 = 2 * w, n = 4 * hw;
    const int row0 = max(Y - 1, 0) * w + Xc, row1 = Y * w + Xc, row2 = min(Y + 1, h - 1) * w + Xc;
    // Output column 2X + a and row 2Y + b take source columns / rows x0, x1 / y0, y1 (up_axis).
    // For an owner column these are X - 1 or X (x0, a = 0), X or X + 1 (x1, a = 0), X
    // (x0, a = 1), X + 1 or X (x1, a = 1), and likewise for the rows: the flags below say
    // which, and a neighbour's column is always inside the level when it is used.
    bool xl0, xr0, xr1, yu0, yd0, yd1;
    UpW wt[2][2];
    {
        int i0, i1, j0, j1;
        float fx[2], fy[2];
        up_axis(2 * X, w, i0, i1, fx[0]);
        xl0 = i0 < X;
        xr0 = i1 > X;
        up_axis(2 * X + 1, w, i0, i1, fx[1]);
        xr1 = i1 > X;
        up_axis(2 * Y, h, j0, j1, fy[0]);
        yu0 = j0 < Y;
        yd0 = j1 > Y;
        up_axis(2 * Y + 1, h, j0, j1, fy[1]);
        yd1 = j1 > Y;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) wt[b][a] = up_weights(fx[a], fy[b]);
    }
    // a wave whose owner columns and row are all inside the level (taps X - 1, X, X + 1 and
    // Y - 1, Y, Y + 1, as for every column and row but the first and last) skips the picks
    const bool inner = __builtin_amdgcn_ballot_w64(own && !(xl0 && !xr0 && xr1)) == 0 && yu0 && !yd0 && yd1;
    const int out0 = 2 * Y * W2 + 2 * X;    // output voxel (2Y, 2X) of plane 0
    const int pix = 2 * (lane - 1);         // LDS column of output pixel (2Y, 2X)
    // wave q takes the planes z = q mod 4, so that the waves share any D evenly
#pragma unroll
    for (int j0 = 0; j0 < kPW; j0 += kG) {
        if (j0 * kUpWaves + q >= D) break;
        float4 m[kG][3];
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            // plane index clamped, so the loads need no guard
            const int base = min((j0 + j) * kUpWaves + q, D - 1) * hw;
            m[j][0] = Vox<DT>::load(src, base + row0);
            m[j][1] = Vox<DT>::load(src, base + row1);
            m[j][2] = Vox<DT>::load(src, base + row2);
        }
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int z = (j0 + j) * kUpWaves + q;
            float4 L[3], R[3];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                L[r] = lane_prev4(m[j][r]);
                R[r] = lane_next4(m[j][r]);
            }
            float4 o00, o01, o10, o11;
            if (inner) {
                o00 = up_blend(wt[0][0], L[0], m[j][0], L[1], m[j][1]);
                o01 = up_blend(wt[0][1], m[j][0], R[0], m[j][1], R[1]);
                o10 = up_blend(wt[1][0], L[1], m[j][1], L[2], m[j][2]);
                o11 = up_blend(wt[1][1], m[j][1], R[1], m[j][2], R[2]);
            } else {
                // per source row r: the taps of columns x0 / x1 for a = 0 and x1 for a = 1
                float4 c00[3], c01[3], c11[3];
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    c00[r] = pick4(xl0, L[r], m[j][r]);
                    c01[r] = pick4(xr0, R[r], m[j][r]);
                    c11[r] = pick4(xr1, R[r], m[j][r]);
                }
                // rows y0 / y1: b = 0 takes rows (0 or 1) and (1 or 2), b = 1 rows 1 and (2 or 1)
                o00 = up_blend(wt[0][0], yu0 ? c00[0] : c00[1], yu0 ? c01[0] : c01[1], yd0 ? c00[2] : c00[1],
                               yd0 ? c01[2] : c01[1]);
                o01 = up_blend(wt[0][1], yu0 ? m[j][0] : m[j][1], yu0 ? c11[0] : c11[1], yd0 ? m[j][2] : m[j][1],
                               yd0 ? c11[2] : c11[1]);
                o10 = up_blend(wt[1][0], c00[1], c01[1], yd1 ? c00[2] : c00[1], yd1 ? c01[2] : c01[1]);
                o11 = up_blend(wt[1][1], m[j][1], c11[1], yd1 ? m[j][2] : m[j][1], yd1 ? c11[2] : c11[1]);
            }
            if (own && z < D) {
                Vox<DT>::store2(dst, z * n + out0, o00, o01);
                Vox<DT>::store2(dst, z * n + out0 + W2, o10, o11);
                s_a[z][pix] = UpAlpha<DT>::put(Vox<DT>::stored(o00).w);
                s_a[z][pix + 1] = UpAlpha<DT>::put(Vox<DT>::stored(o01).w);
                s_a[z][kUpPix / 2 + pix] = UpAlpha<DT>::put(Vox<DT>::stored(o10).w);
                s_a[z][kUpPix / 2 + pix + 1] = UpAlpha<DT>::put(Vox<DT>::stored(o11).w);
            }
        }
    }
    __syncthreads();
    // selection: output pixel e of the workgroup (row 2Y + e / 124, column 2 X0 + e % 124)
    const int e = q * 64 + lane;
    const int ox = 2 * bx * kUpCols + e % (kUpPix / 2);
    if (e < kUpPix && ox < W2) {
        const int oy = 2 * Y + e / (kUpPix / 2);
        float A[MAXD];
        float T = 1.0f;
#pragma unroll
        for (int z = 0; z < MAXD; ++z)
            if (z < D) A[z] = score_step(UpAlpha<DT>::get(s_a[z][e]), T);
        mask[oy * W2 + ox] = topk_bits<MAXD>(A, D, k, tau, rule);
    }
}

template <int DT, int MAXD>
__global__ __launch_bounds__(64 * kUpWaves) void k_upsample_select_blk(const void* __restrict__ src, int D, int h,
                                                                       int w, void* __restrict__ dst, int k,
                                                                       float tau, int rule,
                                                                       uint64_t* __restrict__ mask, int nbx) {
    __shared__ typename UpAlpha<DT>::T s_a[MAXD][kUpPix];
    const int g = blockIdx.x;
    upsample_select_block<DT, MAXD>(src, D, h, w, dst, k, tau, rule, mask, g % nbx, g / nbx, s_a);
}

// The 2x2 box mean of a (x, y), b (x + 1, y), c (x, y + 1), d (x + 1, y + 1): the one
// expression every downsampling path evaluates.
__device__ __forceinline__ float box4(float a, float b, float c, float d) { return ((a + b) + (c + d)) * 0.25f; }

// Output pixel i of view n of the 2x2 box mean of [N][H][W][3] images.
__device__ __forceinline__ void downsample_pixel(const float* __restrict__ img, int H, int W,
                                                 float* __restrict__ out, int n, int i) {
    const int h = H / 2, w = W / 2;
    if (i >= h * w) return;
    const int x = i % w, y = i / w;
    const float* s = img + ((size_t)n * H + 2 * y) * W * 3 + 6 * x;
    float* o = out + ((size_t)n * h * w + i) * 3;
    for (int c = 0; c < 3; ++c) o[c] = box4(s[c], s[3 + c], s[3 * W + c], s[3 * W + 3 + c]);
}

// NL successive 2x2 box means of [N][H][W][3] images (H and W multiples of 2^NL) in one
// launch: a thread takes one pixel of the coarsest result, reads its 2^NL x 2^NL block once
// and writes its share of every level (out[j]: level j + 1), each level the box means of
// the one above as downsample_pixel computes them.
template <int NL>
__device__ __forceinline__ void pyramid_block(const float* __restrict__ img, int H, int W, float* __restrict__ out0,
                                              float* __restrict__ out1, float* __restrict__ out2, int n, int bx) {
    constexpr int S = 1 << NL;
    const int hc = H >> NL, wc = W >> NL;
    const int i = bx * 256 + threadIdx.x;
    if (i >= hc * wc) return;
    const int x = i % wc, y = i / wc;
    float cur[S / 2][S / 2][3];
#pragma unroll
    for (int r = 0; r < S / 2; ++r) {
        const float* s0 = img + (((size_t)n * H + y * S + 2 * r) * W + (size_t)x * S) * 3;
        const float* s1 = s0 + (size_t)W * 3;
#pragma unroll
        for (int c = 0; c < S / 2; ++c)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                cur[r][c][ch] = box4(s0[6 * c + ch], s0[6 * c + 3 + ch], s1[6 * c + ch], s1[6 * c + 3 + ch]);
    }
    float* const outs[3] = {out0, out1, out2};
#pragma unroll
    for (int l = 1; l <= NL; ++l) {
        const int E = S >> l;                       // this thread's block edge at level l
        const int Hl = H >> l, Wl = W >> l;
        float* o = outs[l - 1];
#pragma unroll
        for (int r = 0; r < E; ++r)
#pragma unroll
            for (int c = 0; c < E; ++c)
#pragma unroll
                for (int ch = 0; ch < 3; ++ch)
                    o[(((size_t)n * Hl + y * E + r) * Wl + (size_t)x * E + c) * 3 + ch] = cur[r][c][ch];
        if (l < NL) {
#pragma unroll
            for (int r = 0; r < E / 2; ++r)
#pragma unroll
                for (int c = 0; c < E / 2; ++c)
#pragma unroll
                    for (int ch = 0; ch < 3; ++ch)
                        cur[r][c][ch] = box4(cur[2 * r][2 * c][ch], cur[2 * r][2 * c + 1][ch],
                                             cur[2 * r + 1][2 * c][ch], cur[2 * r + 1][2 * c + 1][ch]);
        }
    }
}

template <int NL>
__global__ __launch_bounds__(256) void k_pyramid(const float* __restrict__ img, int H, int W,
                                                 float* __restrict__ out0, float* __restrict__ out1,
                                                 float* __restrict__ out2) {
    pyramid_block<NL>(img, H, W, out0, out1, out2, blockIdx.y, blockIdx.x);
}

// The first selection of the coarsest level and the target pyramid are independent: one
// launch runs both, its first nsel blocks selecting (as k_select) and the others reducing
// (as k_pyramid, block b of view n at nsel + n * nbx + b), so neither waits for the other.
template <int DT, int MAXD, int NL>
__global__ __launch_bounds__(256) void k_select_pyramid(const void* __restrict__ mpi, int D, int HW, int k,
                                                        float tau, int rule, uint64_t* __restrict__ mask,
                                                        int nsel, const float* __restrict__ img, int H, int W,
                                                        float* __restrict__ out0, float* __restrict__ out1,
                                                        float* __restrict__ out2, int nbx) {
    const int b = blockIdx.x;
    if (b < nsel) {
        const int p = b * 256 + threadIdx.x;
        if (p < HW) mask[p] = select_bits<DT, MAXD>(mpi, D, HW, p, k, tau, rule);
    } else {
        const int j = b - nsel;
        pyramid_block<NL>(img, H, W, out0, out1, out2, j / nbx, j % nbx);
    }
}

__global__ __launch_bounds__(256) void k_downsample(const float* __restrict__ img, int H, int W,
                                                    float* __restrict__ out) {
    downsample_pixel(img, H, W, out, blockIdx.y, blockIdx.x * blockDim.x + threadIdx.x);
}

template <int SDT, int DDT>
__global__ __launch_bounds__(256) void k_convert(const void* __restrict__ src, void* __restrict__ dst,
                                                 int64_t n) {
    const int64_t i = (int64_t)flat_block() * 256 + threadIdx.x;
    if (i >= n) return;
    float v;
    if (SDT == HSGD_FP32) v = reinterpret_cast<const float*>(src)[i];
    else v = __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(src)[i] << 16);
    if (DDT == HSGD_FP32) reinterpret_cast<float*>(dst)[i] = v;
    else reinterpret_cast<uint16_t*>(dst)[i] = (uint16_t)f32_to_bf16_bits(v);
}

// ------------------------------------------------------------------------------------
// batched serving step: kernels over the work items of every in-flight request
// ------------------------------------------------------------------------------------
// Each kernel is launched over exactly its items of the step: workgroup g takes item g of
// the list concatenated over the requests (a list of 2^32 threads or more in rows over y, the
// last of which may end past it).
// Slot of flat work item g of kernel kk (prefix counts are non-decreasing; uniform result).
__device__ __forceinline__ int batch_slot_of(const BatchTable* __restrict__ t, int kk, int g) {
    int s = 0;
    for (int j = 1; j < t->nslot; ++j) s += g >= t->pre[kk][j] ? 1 : 0;
    return __builtin_amdgcn_readfirstlane(s);
}

// The step's table from the pinned memory it was written to: a kernel on the stream's own
// queue, 10 us between two steps' work with the step's event (a copy engine's hand-over and
// an event that frees the staging buffer: 15).
__global__ __launch_bounds__(256) void k_batch_table(const uint4* __restrict__ src, uint4* __restrict__ dst, int n) {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = src[i];
}

// The front of a step, one launch for what does not depend on each other: the slots at the
// start of a level above the coarsest upsample into it and select there (2 x 2 blocks, as
// k_upsample_select_blk), the others select on the MPI they have, and a request's first step
// also reduces its targets (as k_pyramid). A slot's first front_main items are the former,
// the rest the pyramid's. Bound by memory traffic: the level is written once and its alphas
// are scored from LDS. Eight requests (2 of 1008 x 756 x 32, 3 of 512 x 384 x 32, 3 of
// 256 x 192 x 16, BF16), as three box means, upsampling by pixel and selection from the stored
// level in five launches: 488 us at their finest level, 115 one below; here 212 and 65. (Items
// in launch order: grouping them by XCD took 221 us.)
template <int DT, int MAXD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DT == HSGD_FP32 && MAXD > 16 ? 2 : 4))) void k_batch_front(
    const BatchTable* __restrict__ t) {
    static_assert(64 * kUpWaves == 256, "one workgroup size");
    __shared__ typename UpAlpha<DT>::T s_a[MAXD][kUpPix];
    const int g = flat_block();
    if (g >= t->total[BK_FRONT]) return;
    const int sl = batch_slot_of(t, BK_FRONT, g);
    const BatchSlot& b = t->slot[sl];
    const int j = g - t->pre[BK_FRONT][sl];
    if (j >= b.front_main) {
        const int e = j - b.front_main;
        const int nb = ((b.pyr_h >> b.pyr_nl) * (b.pyr_w >> b.pyr_nl) + 255) / 256;
        const int n = e / nb, bx = e - n * nb;
        if (b.pyr_nl == 1)
            pyramid_block<1>(b.pyr_src, b.pyr_h, b.pyr_w, b.pyr_dst[0], nullptr, nullptr, n, bx);
        else if (b.pyr_nl == 2)
            pyramid_block<2>(b.pyr_src, b.pyr_h, b.pyr_w, b.pyr_dst[0], b.pyr_dst[1], nullptr, n, bx);
        else
            pyramid_block<3>(b.pyr_src, b.pyr_h, b.pyr_w, b.pyr_dst[0], b.pyr_dst[1], b.pyr_dst[2], n, bx);
    } else if (b.up_src) {
        const int nbx = (b.uw + kUpCols - 1) / kUpCols;
        upsample_select_block<DT, MAXD>(b.up_src, b.D, b.uh, b.uw, b.mpi, b.k, b.tau, b.rule, b.mask, j % nbx, j / nbx,
                                        s_a);
    } else {
        const int p = j * 256 + threadIdx.x;
        const int HW = b.H * b.W;
        if (p < HW) b.mask[p] = select_bits<DT, MAXD>(b.mpi, b.D, HW, p, b.k, b.tau, b.rule);
    }
}

// Tiles are taken in the XCD-grouped order of the flat item list, so neighbouring tiles of
// one request share an XCD's L2. The forms are k_grad_shift's (as a persistent loop over the
// items, which needs registers of its own, the eight requests of k_batch_front took 1425 us at their finest level, here 1188; now 1165).
template <int DT, int MAXD>
__global__ __launch_bounds__(kSX * kSY) __attribute__((amdgpu_waves_per_eu(grad_shift_waves<DT, MAXD>()))) void k_batch_grad(
    const BatchTable* __restrict__ t, int kk) {
    const int total = t->total[kk];
    if (flat_block() >= total) return;
    const int g = xcd_tile(flat_block(), total);
    const int sl = batch_slot_of(t, kk, g);
    const BatchSlot& b = t->slot[sl];
    grad_shift_tile<DT, MAXD, true>(b.mpi, b.D, b.H, b.W, b.N, b.warps, b.images, nullptr, b.mask, b.kcap,
                                    1.0f / (float)b.N, b.slots, b.partials, b.ntx, g - t->pre[kk][sl], threadIdx.x);
}

template <int DT>
__global__ __launch_bounds__(256) void k_batch_update(const BatchTable* __restrict__ t) {
    extern __shared__ int2 s_off[];
    const int g = blockIdx.x;
    const int sl = batch_slot_of(t, BK_UPDATE, g);
    const BatchSlot& b = t->slot[sl];
    update_block<DT, true>(b.mpi, b.D, b.H, b.W, b.mask, b.kcap, b.slots, b.N, b.warps, b.ntx * kOX, b.nty * kOY,
                           b.lr_rgb, b.lr_alpha, 1, nullptr, b.partials, (int64_t)b.ntx * b.nty * b.N, 0.5 / b.N,
                           b.loss_out, b.prior, g - t->pre[BK_UPDATE][sl], s_off);
}

// Plane-count classes: the kernels unroll their plane loops to MAXD planes and run the
// planes z >= D as transparent ones, at full cost, so the classes lie 8 apart up to 48. FP32,
// 512 x 378 x 40 planes, 3 views: gradient 173 us as 64 planes, 121 as 40; selection 32 and
// 24, upsampling with selection 45 and 35 (24 planes, 4 views: gradient 107 us as 32, 87).
constexpr int kClasses[kNumClasses] = {8, 16, 24, 32, 40, 48, 64};
int maxd_class(int D) {
    return kClasses[batch_class(D)];
}

#define HSGD_DISPATCH_D(D, BODY)                         \
    switch (maxd_class(D)) {                             \
        case 8: { constexpr int MD = 8; BODY; } break;   \
        case 16: { constexpr int MD = 16; BODY; } break; \
        case 24: { constexpr int MD = 24; BODY; } break; \
        case 32: { constexpr int MD = 32; BODY; } break; \
        case 40: { constexpr int MD = 40; BODY; } break; \
        case 48: { constexpr int MD = 48; BODY; } break; \
        default: { constexpr int MD = 64; BODY; } break; \
    }

#define HSGD_DISPATCH_T(dt, BODY)                                  \
    if ((dt) == HSGD_FP32) { constexpr int DT = HSGD_FP32; BODY; } \
    else { constexpr int DT = HSGD_BF16; BODY; }

}  // namespace

// ------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------
static int launch_scan_compact(const ActiveSet& as, int D, int HW, int* plane_off, hipStream_t s) {
    const int64_t n = (int64_t)D * as.nblk;
    {
        ProfScope ps(HSGD_K_SCAN, s);
        hipLaunchKernelGGL(k_scan_seg, dim3((unsigned)as.nseg), dim3(256), 0, s, as.off, n, as.seg);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, as.off, as.nblk, D, as.seg, (int)as.nseg,
                           plane_off, as.nact);
    }
    ProfScope ps(HSGD_K_COMPACT, s);
    hipLaunchKernelGGL(k_compact, dim3((unsigned)ceil_div(as.nblk * 64, 256)), dim3(256), 0, s, as.bal, as.off,
                       as.seg, D, HW, as.nblk, as.ids, as.cap);
    return (int)hipGetLastError();
}

int launch_select(const hsgd_mpi& m, int k, float tau, int rule, uint64_t* mask, const ActiveSet* as,
                  int32_t* plane_off, hipStream_t s) {
    const int HW = m.H * m.W;
    const dim3 grid((unsigned)ceil_div(HW, 256));
    {
        ProfScope ps(HSGD_K_SELECT, s);
        HSGD_DISPATCH_T(m.dtype, HSGD_DISPATCH_D(m.D, hipLaunchKernelGGL((k_select<DT, MD>), grid, dim3(256), 0, s,
                                                                        m.rgba, m.D, HW, k, tau, rule, mask,
                                                                        as ? as->bal : nullptr,
                                                                        as ? as->off : nullptr,
                                                                        as ? as->nblk : (int64_t)0)));
    }
    if (!as) return (int)hipGetLastError();
    return launch_scan_compact(*as, m.D, HW, plane_off, s);
}

int launch_render(const hsgd_mpi& m, const hsgd_views& v, float* out_rgb, float* out_loss,
                  void* ws, hipStream_t s) {
    const RenderWs L = render_ws(m.H, m.W, v.N);
    float* partials = out_loss ? reinterpret_cast<float*>((char*)ws + L.partial_off) : nullptr;
    int64_t nparts;
    if (v.flags & HSGD_VIEWS_SHIFT_ONLY) {
        const int ntx = (int)ceil_div(m.W, kShiftRX), nty = (int)ceil_div(m.H, kShiftRY);
        nparts = (int64_t)ntx * nty * v.N;
        const int rows = render_rows(m.D, m.H, m.W, v.N);
        ProfScope ps(HSGD_K_RENDER, s);
        if (rows > 1) {
            nparts = (int64_t)ntx * ceil_div(m.H, rows * kRenderWaves) * v.N;
#define HSGD_RENDER_ROWS(R)                                                                                        \
    HSGD_DISPATCH_T(m.dtype, hipLaunchKernelGGL((k_render_shift_rows<DT, R>), dim3((unsigned)nparts),                \
                                                dim3(64 * kRenderWaves), 0, s, m.rgba, m.D, m.H, m.W, v.N, v.warps, \
                                                v.images, out_rgb, partials, ntx))
            if (rows == 8) {
                HSGD_RENDER_ROWS(8);
            } else {
                HSGD_RENDER_ROWS(4);
            }
#undef HSGD_RENDER_ROWS
        } else {
            HSGD_DISPATCH_T(m.dtype, HSGD_DISPATCH_D(m.D, hipLaunchKernelGGL((k_render_shift<DT, MD>), dim3((unsigned)nparts),
                                                                            dim3(kSX * kSY), 0, s, m.rgba, m.D, m.H, m.W,
                                                                            v.N, v.warps, v.images, out_rgb, partials,
                                                                            ntx)));
        }
    } else {
        const int ntx = (int)ceil_div(m.W, kTileW);
        const int64_t each = ntx * ceil_div(m.H, kTileH);
        nparts = each * v.N;
        ProfScope ps(HSGD_K_RENDER, s);
        const int nty = (int)(each / ntx);
        const bool few = m.D <= kRenderFew && nty <= 65535;
        const dim3 grid = few ? dim3((unsigned)ntx, (unsigned)nty, (unsigned)v.N) : split_grid(each, v.N, kBlock);
#define HSGD_RENDER_GENERAL(FEW)                                                                                     \
    HSGD_DISPATCH_T(m.dtype, hipLaunchKernelGGL((k_render<DT, FEW>), grid, dim3(kBlock), 0, s, m.rgba, m.D, m.H, m.W, \
                                                v.N, v.warps, v.images, out_rgb, partials, ntx))
        if (few) {
            HSGD_RENDER_GENERAL(true);
        } else {
            HSGD_RENDER_GENERAL(false);
        }
#undef HSGD_RENDER_GENERAL
    }
    if (out_loss) {
        ProfScope ps(HSGD_K_REDUCE, s);
        hipLaunchKernelGGL(k_reduce, dim3(1), dim3(256), 0, s, partials, nparts, 0.5 / v.N, out_loss);
    }
    return (int)hipGetLastError();
}

int launch_grad_step(const hsgd_mpi& m, const hsgd_views& v, const uint64_t* mask, int kcap,
                     const float* dimg, float lr_rgb, float lr_alpha, float lambda_s, float* grad_out,
                     float* out_loss, float4* slots, float* partials, hipStream_t s) {
    const float prior = (float)((double)lambda_s / ((double)m.D * m.H * m.W));
    const int HW = m.H * m.W;
    const float inv_n = 1.0f / (float)v.N;
    const bool shift = (v.flags & HSGD_VIEWS_SHIFT_ONLY) != 0;
    int64_t nparts;
    int cover_w = 0, cover_h = 0;
    // (without a mask every entry is selected, and the update writes them all: 8 us of 50 for
    // 256 x 192 x 16, 3 views)
    if (grad_out && mask) {
        ProfScope ps(HSGD_K_FILL, s);
        const int64_t n = (int64_t)m.D * HW;
        hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)std::min<int64_t>(ceil_div(n, 256), 8192)), dim3(256), 0, s,
                           reinterpret_cast<float4*>(grad_out), n);
    }
    if (shift) {
        const int ntx = (int)ceil_div(m.W + 1, kOX), nty = (int)ceil_div(m.H + 1, kOY);
        cover_w = ntx * kOX;
        cover_h = nty * kOY;
        const int64_t each = (int64_t)ntx * nty;
        nparts = each * v.N;
        const dim3 grid = split_grid(each, v.N, kSX * kSY);
        ProfScope ps(HSGD_K_GRAD, s);
        if (mask) {
            HSGD_DISPATCH_T(m.dtype, HSGD_DISPATCH_D(m.D, hipLaunchKernelGGL((k_grad_shift<DT, MD, true>), grid,
                                                                            dim3(kSX * kSY), 0, s, m.rgba, m.D, m.H, m.W,
                                                                            v.N, v.warps, v.images, dimg, mask, kcap,
                                                                            inv_n, slots, out_loss ? partials : nullptr,
                                                                            ntx)));
        } else {
            HSGD_DISPATCH_T(m.dtype, HSGD_DISPATCH_D(m.D, hipLaunchKernelGGL((k_grad_shift<DT, MD, false>), grid,
                                                                            dim3(kSX * kSY), 0, s, m.rgba, m.D, m.H, m.W,
                                                                            v.N, v.warps, v.images, dimg, mask, kcap,
                                                                            inv_n, slots, out_loss ? partials : nullptr,
                                                                            ntx)));
        }
    } else {
        {
            ProfScope ps(HSGD_K_FILL, s);
            const int64_t n = (int64_t)kcap * HW;
            hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)std::min<int64_t>(ceil_div(n, 256), 8192)), dim3(256), 0, s,
                               slots, n);
        }
        const int ntx = (int)ceil_div(m.W, kGenOX);
        const int64_t each = ceil_div(m.H, kGenY) * ntx;
        nparts = each * v.N;
        const dim3 grid = split_grid(each, v.N, kGenThreads);
        ProfScope ps(HSGD_K_GRAD, s);
        const float* im = v.images;
        float* parts = out_loss ? partials : nullptr;
#define HSGD_GRAD_GENERAL(MD)                                                                                       \
    HSGD_DISPATCH_T(m.dtype, hipLaunchKernelGGL((k_grad<DT, MD>), grid, dim3(kGenThreads), 0, s, m.rgba, m.D, m.H, m.W, \
                                                v.N, v.warps, im, dimg, mask, kcap, inv_n, slots, parts, ntx))
        // The LDS of the transmittances sets the residency: two workgroups per CU up to 32 planes,
        // one above. A step of 512x384, 4 tilted views, k = 4 in FP32 takes 427 us with 33 planes
        // and 656 with 64 (736 and 932 before the kernel had its present form).
        if (m.D <= 32) {
            HSGD_GRAD_GENERAL(32);
        } else {
            HSGD_GRAD_GENERAL(64);
        }
#undef HSGD_GRAD_GENERAL
    }
    const int do_update = (lr_rgb != 0.0f || lr_alpha != 0.0f) ? 1 : 0;
    if (do_update || grad_out || out_loss) {
        ProfScope ps(HSGD_K_UPDATE, s);
        const dim3 grid((unsigned)ceil_div(HW, 256 / kUpdateRS));
        const size_t lds = shift ? sizeof(int2) * (size_t)v.N * m.D : 0;
        HSGD_DISPATCH_T(m.dtype, if (shift) {
            hipLaunchKernelGGL((k_update<DT, true>), grid, dim3(256), lds, s, m.rgba, m.D, m.H, m.W, mask, kcap,
                               slots, v.N, v.warps, cover_w, cover_h, lr_rgb, lr_alpha, do_update,
                               reinterpret_cast<float4*>(grad_out), partials, nparts, 0.5 / v.N, out_loss, prior);
        } else {
            hipLaunchKernelGGL((k_update<DT, false>), grid, dim3(256), 0, s, m.rgba, m.D, m.H, m.W, mask, kcap,
                               slots, 1, v.warps, 0, 0, lr_rgb, lr_alpha, do_update,
                               reinterpret_cast<float4*>(grad_out), partials, nparts, 0.5 / v.N, out_loss, prior);
        });
    }
    return (int)hipGetLastError();
}

int launch_upsample(const hsgd_mpi& c, const hsgd_mpi& f, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div((int64_t)f.H * f.W, 256), (unsigned)c.D);
    ProfScope ps(HSGD_K_UPSAMPLE, s);
    HSGD_DISPATCH_T(c.dtype, hipLaunchKernelGGL((k_upsample<DT>), grid, dim3(256), 0, s, c.rgba, c.H, c.W, f.rgba));
    return (int)hipGetLastError();
}

int launch_upsample_select(const hsgd_mpi& c, const hsgd_mpi& f, int k, float tau, int rule, uint64_t* mask,
                           hipStream_t s) {
    ProfScope ps(HSGD_K_UPSAMPLE, s);
    const int nbx = (int)ceil_div(c.W, kUpCols);
    const dim3 blk((unsigned)((int64_t)nbx * c.H));
    if ((int64_t)blk.x >= kUpBlkMinGroups) {
        HSGD_DISPATCH_T(c.dtype, HSGD_DISPATCH_D(c.D, hipLaunchKernelGGL((k_upsample_select_blk<DT, MD>), blk,
                                                                        dim3(64 * kUpWaves), 0, s, c.rgba, c.D, c.H,
                                                                        c.W, f.rgba, k, tau, rule, mask, nbx)));
    } else {
        const dim3 grid((unsigned)ceil_div((int64_t)f.H * f.W, 64));
        HSGD_DISPATCH_T(c.dtype, HSGD_DISPATCH_D(c.D, hipLaunchKernelGGL((k_upsample_select<DT, MD>), grid,
                                                                        dim3(64 * kUpWaves), 0, s, c.rgba, c.D, c.H,
                                                                        c.W, f.rgba, k, tau, rule, mask)));
    }
    return (int)hipGetLastError();
}

int launch_pyramid(const float* img, int N, int H, int W, int nl, float* const* out, hipStream_t s) {
    const int hc = H >> nl, wc = W >> nl;
    const dim3 grid((unsigned)ceil_div((int64_t)hc * wc, 256), (unsigned)N);
    ProfScope ps(HSGD_K_DOWNSAMPLE, s);
    if (nl == 1)
        hipLaunchKernelGGL(k_pyramid<1>, grid, dim3(256), 0, s, img, H, W, out[0], nullptr, nullptr);
    else if (nl == 2)
        hipLaunchKernelGGL(k_pyramid<2>, grid, dim3(256), 0, s, img, H, W, out[0], out[1], nullptr);
    else
        hipLaunchKernelGGL(k_pyramid<3>, grid, dim3(256), 0, s, img, H, W, out[0], out[1], out[2]);
    return (int)hipGetLastError();
}

int launch_select_pyramid(const hsgd_mpi& m, int k, float tau, int rule, uint64_t* mask, const float* img, int N,
                          int H, int W, int nl, float* const* out, hipStream_t s) {
    const int HW = m.H * m.W;
    const int nsel = (int)ceil_div(HW, 256);
    const int nbx = (int)ceil_div((int64_t)(H >> nl) * (W >> nl), 256);
    const dim3 grid((unsigned)(nsel + nbx * N));
    ProfScope ps(HSGD_K_SELECT, s);
    HSGD_DISPATCH_T(m.dtype, HSGD_DISPATCH_D(m.D, {
        if (nl == 1)
            hipLaunchKernelGGL((k_select_pyramid<DT, MD, 1>), grid, dim3(256), 0, s, m.rgba, m.D, HW, k, tau, rule,
                               mask, nsel, img, H, W, out[0], nullptr, nullptr, nbx);
        else if (nl == 2)
            hipLaunchKernelGGL((k_select_pyramid<DT, MD, 2>), grid, dim3(256), 0, s, m.rgba, m.D, HW, k, tau, rule,
                               mask, nsel, img, H, W, out[0], out[1], nullptr, nbx);
        else
            hipLaunchKernelGGL((k_select_pyramid<DT, MD, 3>), grid, dim3(256), 0, s, m.rgba, m.D, HW, k, tau, rule,
                               mask, nsel, img, H, W, out[0], out[1], out[2], nbx);
    }));
    return (int)hipGetLastError();
}

int launch_downsample(const float* img, int N, int H, int W, float* out, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div((int64_t)(H / 2) * (W / 2), 256), (unsigned)N);
    ProfScope ps(HSGD_K_DOWNSAMPLE, s);
    hipLaunchKernelGGL(k_downsample, grid, dim3(256), 0, s, img, H, W, out);
    return (int)hipGetLastError();
}

int launch_convert(const void* src, int sdt, void* dst, int ddt, size_t n, hipStream_t s) {
    const dim3 grid = items_grid(ceil_div((int64_t)n, 256), 256);
    ProfScope ps(HSGD_K_CONVERT, s);
    if (sdt == HSGD_FP32 && ddt == HSGD_FP32)
        hipLaunchKernelGGL((k_convert<HSGD_FP32, HSGD_FP32>), grid, dim3(256), 0, s, src, dst, (int64_t)n);
    else if (sdt == HSGD_FP32)
        hipLaunchKernelGGL((k_convert<HSGD_FP32, HSGD_BF16>), grid, dim3(256), 0, s, src, dst, (int64_t)n);
    else if (ddt == HSGD_FP32)
        hipLaunchKernelGGL((k_convert<HSGD_BF16, HSGD_FP32>), grid, dim3(256), 0, s, src, dst, (int64_t)n);
    else
        hipLaunchKernelGGL((k_convert<HSGD_BF16, HSGD_BF16>), grid, dim3(256), 0, s, src, dst, (int64_t)n);
    return (int)hipGetLastError();
}

int batch_class(int D) {
    return D <= 8 ? 0 : D <= 16 ? 1 : D <= 24 ? 2 : D <= 32 ? 3 : D <= 40 ? 4 : D <= 48 ? 5 : 6;
}

int launch_batch_step(const BatchTable* staged, BatchTable* t, int dtype, hipStream_t s) {
    const int words = (int)((offsetof(BatchTable, slot) + sizeof(BatchSlot) * (size_t)staged->nslot + 15) / 16);
    hipLaunchKernelGGL(k_batch_table, dim3(1), dim3(256), 0, s, reinterpret_cast<const uint4*>(staged),
                       reinterpret_cast<uint4*>(t), words);
    int max_d = 1;
    size_t shifts = 0;
    for (int i = 0; i < staged->nslot; ++i) {
        max_d = std::max(max_d, staged->slot[i].D);
        shifts = std::max(shifts, (size_t)staged->slot[i].N * staged->slot[i].D);
    }
    HSGD_DISPATCH_T(dtype, HSGD_DISPATCH_D(max_d, hipLaunchKernelGGL((k_batch_front<DT, MD>),
                                                                     items_grid(staged->total[BK_FRONT], 256), dim3(256), 0,
                                                                     s, t)));
    for (int c = 0; c < kNumClasses; ++c)
        if (staged->total[BK_GRAD + c])
            HSGD_DISPATCH_T(dtype, HSGD_DISPATCH_D(kClasses[c], hipLaunchKernelGGL((k_batch_grad<DT, MD>),
                                                                                   items_grid(staged->total[BK_GRAD + c], kSX * kSY),
                                                                                   dim3(kSX * kSY), 0, s, t, BK_GRAD + c)));
    HSGD_DISPATCH_T(dtype, hipLaunchKernelGGL((k_batch_update<DT>), dim3((unsigned)staged->total[BK_UPDATE]), dim3(256),
                                              sizeof(int2) * shifts, s, t));
    return (int)hipGetLastError();
}
}  // namespace hsgd
