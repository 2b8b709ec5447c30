// Plane-sweep volume of libhsgd for gfx950 (wave64).
//
//  k_plane_sweep  the source images inverse-warped onto every reference plane and box-
//                 downsampled level by level (Sec. 3.2, Hierarchical PSV Construction)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hsgd_device.h"
#include "hsgd_internal.h"

namespace hsgd {
namespace {

// ------------------------------------------------------------------------------------
// plane-sweep volume and its pyramid (Sec. 3.2, Hierarchical PSV Construction): a
// workgroup samples one 64 x 16 reference tile of one (view, plane) from the source image
// (4 consecutive pixels of a row per thread), stores it, then reduces it 2x2 level by level
// in LDS and stores each level from there: no level is read back from memory.
// ------------------------------------------------------------------------------------
constexpr int kPsvTW = 64, kPsvTH = 16;
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct PsvOut {
    void* p[kPsvMaxL];
    bool meet;                     // an FP32 level 1 through the caches
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool NT, typename T>
__device__ __forceinline__ void st_stream(T v, T* p) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Store the valid vh x vw pixels of a TH x TW tile, row-major in LDS (FP32), to rows of Wl
// pixels at dst (the tile's first pixel) in the output type OT. 16-byte runs when every row
// start is 16-byte aligned (FP32: Wl % 4 == 0; BF16: Wl % 8 == 0 and 16-byte tile rows; vw
// is then a multiple of the run's pixels too), else one pixel per lane; consecutive lanes
// write consecutive addresses either way. BF16 rounds to nearest even. NT: past the caches
// (through them 768x512x32, 2 tilted views, FP32 took 98 us instead of 72).
template <int TH, int TW, int OT, bool NT>
__device__ __forceinline__ void psv_store_tile(const float* __restrict__ s, int vh, int vw, void* __restrict__ dst,
                                               int Wl, int t) {
    if (OT == HSGD_FP32 && (Wl & 3) == 0) {
        float* o = reinterpret_cast<float*>(dst);
        constexpr int RQ = TW * 3 / 4;                      // float4 per tile row
        const int vq = vw * 3 / 4;
#pragma unroll
        for (int e0 = 0; e0 < TH * RQ; e0 += 256) {
            const int e = e0 + t, r = e / RQ, c = e - r * RQ;
            if ((TH * RQ % 256 == 0 || e < TH * RQ) && r < vh && c < vq) {
                const float4 q = reinterpret_cast<const float4*>(s)[e];
                st_stream<NT>(f32x4{q.x, q.y, q.z, q.w}, reinterpret_cast<f32x4*>(o + (size_t)r * Wl * 3) + c);
            }
        }
    } else if (OT == HSGD_BF16 && TW * 6 % 16 == 0 && (Wl & 7) == 0) {
        uint16_t* o = reinterpret_cast<uint16_t*>(dst);
        constexpr int RQ = TW * 3 / 8;                      // 8 values (16 bytes) per run
        const int vq = vw * 3 / 8;
#pragma unroll
        for (int e0 = 0; e0 < TH * RQ; e0 += 256) {
            const int e = e0 + t, r = e / RQ, c = e - r * RQ;
            if ((TH * RQ % 256 == 0 || e < TH * RQ) && r < vh && c < vq) {
                const float4 a = reinterpret_cast<const float4*>(s)[2 * e];
                const float4 b = reinterpret_cast<const float4*>(s)[2 * e + 1];
                const u32x4 q{f32x2_to_bf16x2(a.x, a.y), f32x2_to_bf16x2(a.z, a.w), f32x2_to_bf16x2(b.x, b.y),
                              f32x2_to_bf16x2(b.z, b.w)};
                st_stream<NT>(q, reinterpret_cast<u32x4*>(o + (size_t)r * Wl * 3) + c);
            }
        }
    } else {
#pragma unroll
        for (int e0 = 0; e0 < TH * TW; e0 += 256) {
            const int e = e0 + t, r = e / TW, c = e - r * TW;
            if ((TH * TW % 256 == 0 || e < TH * TW) && r < vh && c < vw) {
                const size_t at = ((size_t)r * Wl + c) * 3;
                if (OT == HSGD_FP32) {
                    float* o = reinterpret_cast<float*>(dst) + at;
                    st_stream<NT>(s[3 * e], o);
                    st_stream<NT>(s[3 * e + 1], o + 1);
                    st_stream<NT>(s[3 * e + 2], o + 2);
                } else {
                    uint16_t* o = reinterpret_cast<uint16_t*>(dst) + at;
                    st_stream<NT>((uint16_t)f32_to_bf16_bits(s[3 * e]), o);
                    st_stream<NT>((uint16_t)f32_to_bf16_bits(s[3 * e + 1]), o + 1);
                    st_stream<NT>((uint16_t)f32_to_bf16_bits(s[3 * e + 2]), o + 2);
                }
            }
        }
    }
}

__device__ __forceinline__ float3 bilerp(float w00, float w10, float w01, float w11, float3 a, float3 b,
                                         float3 c, float3 d) {
    return make_float3(w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x,
                       w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y,
                       w00 * a.z + w10 * b.z + w01 * c.z + w11 * d.z);
}

__device__ __forceinline__ float3 lds_rgb(const float* p) { return make_float3(p[0], p[1], p[2]); }

// The source patch of a tile under a translation map: source rows sy0 .. sy0 + 16 and
// pixels sx0 .. sx0 + 64 (the taps of 16 x 64 reference pixels), staged in LDS by coalesced
// dword loads (consecutive lanes, consecutive dwords of a row) through one buffer resource
// over the image: positions outside the image read 0, the zero padding.
constexpr int kPsvSrcRow = (kPsvTW + 1) * 3;                // dwords per patch row
constexpr int kPsvSrcN = (kPsvTH + 1) * kPsvSrcRow;         // dwords per patch
__device__ __forceinline__ void psv_stage_patch(const float* __restrict__ im, int H, int W, int sx0, int sy0,
                                                float* __restrict__ sp, int t) {
    const auto rs = row_rsrc(reinterpret_cast<const char*>(im), H * W * 12);
#pragma unroll
    for (int k = 0; k < (kPsvSrcN + 255) / 256; ++k) {
        const int e = t + 256 * k;
        const int r = e / kPsvSrcRow, c = e - r * kPsvSrcRow;
        const int row = sy0 + r, col = sx0 * 3 + c;
        const bool in = (unsigned)row < (unsigned)H && (unsigned)col < (unsigned)(3 * W);
        const float v = __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(rs, in ? (unsigned)(row * W * 3 + col) * 4u : 0x80000000u, 0, 0));
        if (k < kPsvSrcN / 256 || e < kPsvSrcN) sp[e] = v;
    }
}

// Bilinear samples of a thread's 4 consecutive reference pixels from the staged patch: its
// patch row ly (and ly + 1), patch pixels 4 gx .. 4 gx + 4.
__device__ __forceinline__ void psv_blend_patch(const hsgd_warp& wp, const float* __restrict__ sp, int gx, int ly,
                                                float3 (&v)[4]) {
    const float fx = wp.fx, fy = wp.fy, gxw = 1.0f - fx, gyw = 1.0f - fy;
    const float w00 = gxw * gyw, w10 = fx * gyw, w01 = gxw * fy, w11 = fx * fy;
    const float* r0 = sp + ly * kPsvSrcRow + 12 * gx;
    const float* r1 = r0 + kPsvSrcRow;
    float3 a[5], c[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        a[j] = lds_rgb(r0 + 3 * j);
        c[j] = lds_rgb(r1 + 3 * j);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = bilerp(w00, w10, w01, w11, a[j], a[j + 1], c[j], c[j + 1]);
}

__device__ __forceinline__ float3 psv_tap(__amdgpu_buffer_rsrc_t rs, unsigned off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, off, 0, 0);
    return make_float3(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]));
}

__device__ __forceinline__ RowMap psv_row(const hsgd_warp& w, int y) {
    return w.is_shift ? shift_row(w, (double)y) : row_map(w.G, (double)y);
}

// The samples of a tile under a general map, straight to level 0 in LDS: a wave takes one row
// of 64 pixels at a time (rows wv, wv + 4, ...), so that the lanes of a tap load read
// neighbouring pixels. Four consecutive pixels per lane, as the translation path has them,
// spread each load over 24 cache lines instead of 6-7 (1008x756, 32 planes, 5 views, 3
// levels, BF16 volume: 622 us a launch that way with an IEEE division per position, 511 us
// this way with the cheaper positions, 345 us with the packed rounding to BF16 as well). A tile has four positions per lane, so they are checked
// one by one (free here; checking the map first as plane_map does cost 2 to 3%).
__device__ __forceinline__ void psv_sample_general(const float* __restrict__ im, const hsgd_warp& wp, int tx, int ty,
                                                   int H, int W, float* __restrict__ s_lv, int t) {
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const auto rs = row_rsrc(reinterpret_cast<const char*>(im), H * W * 12);
    const double x = (double)(tx * kPsvTW + lane);
    // the rows' parts of the map, by lanes 0..3 through LDS (only this wave reads them)
    __shared__ double s_row[4][4][3];
    if (lane < 4) {
        const RowMap m = psv_row(wp, ty * kPsvTH + 4 * lane + wv);
        s_row[wv][lane][0] = m.b0;
        s_row[wv][lane][1] = m.b1;
        s_row[wv][lane][2] = m.b2;
    }
    wave_lds_fence();
    RowMap m = psv_row(wp, 0);                              // its a0, a1, a2
    MapPos p[4];
    float3 a[4], b[4], c[4], d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        m.b0 = s_row[wv][j][0];
        m.b1 = s_row[wv][j][1];
        m.b2 = s_row[wv][j][2];
        p[j] = map_pos<true>(m, x);
        const TapOffs o = tap_offsets<12>(p[j], W, H);
        a[j] = psv_tap(rs, o.o00);
        b[j] = psv_tap(rs, o.o10);
        c[j] = psv_tap(rs, o.o01);
        d[j] = psv_tap(rs, o.o11);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float gx = 1.0f - p[j].fx, gy = 1.0f - p[j].fy;
        const float3 v = bilerp(gx * gy, p[j].fx * gy, gx * p[j].fy, p[j].fx * p[j].fy, a[j], b[j], c[j], d[j]);
        float* s = s_lv + ((4 * j + wv) * kPsvTW + lane) * 3;
        s[0] = v.x;
        s[1] = v.y;
        s[2] = v.z;
    }
}

// Level l of a plane's tile (TH x TW pixels at LDS offset OFF) to memory, then level l + 1
// reduced from it into LDS (2x2 means), recursively up to level L - 1.
template <int L, int l, int OFF, int OT>
__device__ __forceinline__ void psv_level(float* __restrict__ s_lv, const PsvOut& out, int iz, int tx, int ty,
                                          int H, int W, int vh0, int vw0, int t) {
    constexpr int TH = kPsvTH >> l, TW = kPsvTW >> l;
    __syncthreads();                                        // level l complete in LDS
    const int Hl = H >> l, Wl = W >> l;
    if (out.p[l]) {
        const size_t at = (((size_t)iz * Hl + ty * TH) * Wl + tx * TW) * 3;
        void* dst = OT == HSGD_FP32 ? (void*)(reinterpret_cast<float*>(out.p[l]) + at)
                                    : (void*)(reinterpret_cast<uint16_t*>(out.p[l]) + at);
        if (l != 1 || OT == HSGD_BF16 || !out.meet) {
            psv_store_tile<TH, TW, OT, true>(s_lv + OFF, vh0 >> l, vw0 >> l, dst, Wl, t);
        } else {
            // (the clobbers keep the compiler from making one store, plain, of both branches')
            asm volatile("" ::: "memory");
            psv_store_tile<TH, TW, OT, false>(s_lv + OFF, vh0 >> l, vw0 >> l, dst, Wl, t);
            asm volatile("" ::: "memory");
        }
    }
    if constexpr (l + 1 < L) {
        constexpr int NH = TH / 2, NW = TW / 2, DST = OFF + TH * TW * 3;
#pragma unroll
        for (int e0 = 0; e0 < NH * NW; e0 += 256) {
            const int e = e0 + t;
            if (NH * NW % 256 == 0 || e < NH * NW) {
                const int ey = e / NW, ex = e - ey * NW;
                const float* a = s_lv + OFF + ((2 * ey) * TW + 2 * ex) * 3;
                const float3 p0 = lds_rgb(a), p1 = lds_rgb(a + 3), p2 = lds_rgb(a + TW * 3), p3 = lds_rgb(a + TW * 3 + 3);
                float* d = s_lv + DST + e * 3;
                d[0] = ((p0.x + p1.x) + (p2.x + p3.x)) * 0.25f;
                d[1] = ((p0.y + p1.y) + (p2.y + p3.y)) * 0.25f;
                d[2] = ((p0.z + p1.z) + (p2.z + p3.z)) * 0.25f;
            }
        }
        psv_level<L, l + 1, DST, OT>(s_lv, out, iz, tx, ty, H, W, vh0, vw0, t);
    }
}

// One plane's tile from the threads' samples v to every level in memory: level l of the
// tile ((16 >> l) x (64 >> l) pixels) is packed after level l - 1 in s_lv.
template <int L, int OT>
__device__ __forceinline__ void psv_tile_levels(const float3 (&v)[4], float* __restrict__ s_lv,
                                                const PsvOut& out, int iz, int tx, int ty, int H, int W,
                                                int vh0, int vw0, int t) {
    {
        const int gx = t & 15, ly = t >> 4;
        float4* s4 = reinterpret_cast<float4*>(s_lv + (ly * kPsvTW + 4 * gx) * 3);
        s4[0] = make_float4(v[0].x, v[0].y, v[0].z, v[1].x);
        s4[1] = make_float4(v[1].y, v[1].z, v[2].x, v[2].y);
        s4[2] = make_float4(v[2].z, v[3].x, v[3].y, v[3].z);
    }
    psv_level<L, 0, 0, OT>(s_lv, out, iz, tx, ty, H, W, vh0, vw0, t);
}

// A workgroup takes one 64 x 16 reference tile of one (view, plane), 4 consecutive pixels
// of a row per thread. Blocks run tile column fastest, then plane, then tile row: the
// workgroups resident on an XCD write whole 16-row bands of a plane (long contiguous runs
// per image row) and sweep the planes of one band, whose source rows stay in its L2.
template <bool SHIFT, int L, int OT>
__global__ __launch_bounds__(256) void k_plane_sweep(const float* __restrict__ img,
                                                     const hsgd_warp* __restrict__ warps, int D, int H, int W,
                                                     PsvOut out, int ntx, int nty) {
    // levels 0.. of the tile, packed one after another: 3 * (1024 + 256 + 64 + 16 + 4)
    // floats; before them, the source patch of a translation map (3315 floats)
    __shared__ __align__(16) float s_lv[3 * (1024 + 256 + 64 + 16 + 4)];
    static_assert(kPsvSrcN <= 3 * (1024 + 256 + 64 + 16 + 4), "source patch exceeds the LDS tile");
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const int tx = b % ntx, r = b / ntx;
    const int z = r % D, r2 = r / D;
    const int ty = r2 % nty, i = r2 / nty;
    const int iz = i * D + z;
    const hsgd_warp& wp = warps[iz];
    const int t = threadIdx.x;
    const float* im = img + (size_t)i * H * W * 3;
    // valid part of the tile; H and W are multiples of 2^(L-1), so every coarse pixel of it
    // has its whole 2x2 block inside the image
    const int vh0 = min(kPsvTH, H - ty * kPsvTH), vw0 = min(kPsvTW, W - tx * kPsvTW);
    if (SHIFT) {
        float3 v[4];
        psv_stage_patch(im, H, W, tx * kPsvTW + wp.ix, ty * kPsvTH + wp.iy, s_lv, t);
        __syncthreads();
        psv_blend_patch(wp, s_lv, t & 15, t >> 4, v);
        __syncthreads();                                    // the patch is overwritten below
        psv_tile_levels<L, OT>(v, s_lv, out, iz, tx, ty, H, W, vh0, vw0, t);
    } else {
        psv_sample_general(im, wp, tx, ty, H, W, s_lv, t);
        psv_level<L, 0, 0, OT>(s_lv, out, iz, tx, ty, H, W, vh0, vw0, t);
    }
}

}  // namespace

// The sweep of N views x D planes whose workgroups one launch holds.
static void sweep_part(const float* images, const hsgd_warp* warps, int N, int D, int H, int W, int L, int out_dtype,
                       bool shift, const PsvOut& o, hipStream_t s) {
    const int ntx = (int)ceil_div(W, kPsvTW), nty = (int)ceil_div(H, kPsvTH);
    const dim3 grid((unsigned)((int64_t)ntx * nty * N * D));
#define HSGD_PSV_LAUNCH(SH, LV)                                                                                \
    if (out_dtype == HSGD_FP32)                                                                                \
        hipLaunchKernelGGL((k_plane_sweep<SH, LV, HSGD_FP32>), grid, dim3(256), 0, s, images, warps, D, H, W, o, \
                           ntx, nty);                                                                          \
    else                                                                                                       \
        hipLaunchKernelGGL((k_plane_sweep<SH, LV, HSGD_BF16>), grid, dim3(256), 0, s, images, warps, D, H, W, o, \
                           ntx, nty)
    switch (L * 2 + (shift ? 1 : 0)) {
        case 2: HSGD_PSV_LAUNCH(false, 1); break;
        case 3: HSGD_PSV_LAUNCH(true, 1); break;
        case 4: HSGD_PSV_LAUNCH(false, 2); break;
        case 5: HSGD_PSV_LAUNCH(true, 2); break;
        case 6: HSGD_PSV_LAUNCH(false, 3); break;
        case 7: HSGD_PSV_LAUNCH(true, 3); break;
        case 8: HSGD_PSV_LAUNCH(false, 4); break;
        case 9: HSGD_PSV_LAUNCH(true, 4); break;
        case 10: HSGD_PSV_LAUNCH(false, 5); break;
        default: HSGD_PSV_LAUNCH(true, 5); break;
    }
#undef HSGD_PSV_LAUNCH
}

int launch_plane_sweep(const hsgd_views& src, int D, int L, int out_dtype, void* const* out, hipStream_t s) {
    const bool shift = (src.flags & HSGD_VIEWS_SHIFT_ONLY) != 0;
    // A grid dimension holds fewer than 2^32 threads: as many views a launch as fit, or as many
    // planes of one. (A grid that goes on in y instead cost small sweeps 2%, in every workgroup's
    // start.)
    const int64_t most = (int64_t)UINT32_MAX / 256, tiles = ceil_div(src.W, kPsvTW) * ceil_div(src.H, kPsvTH);
    const int nv = (int)std::min<int64_t>(src.N, std::max<int64_t>(1, most / (tiles * D)));
    const int nd = nv > 1 ? D : (int)std::min<int64_t>(D, most / tiles);
    const int one = out_dtype == HSGD_FP32 ? 12 : 6;
    // Level 1 of an FP32 volume with rows of no multiple of 64 bytes, the size of a write request:
    // a tile ends inside a request in nearly every row, and under general maps, whose workgroups
    // are many per CU, the parts that two tiles write left L2 one by one. Through the caches they
    // meet there: 1000x704x24, 4 views, 4 levels 335 us streamed and 282 this way, 308x220x40, 3
    // views, 3 levels 42.8 and 35.5. What of it is still in L2 at the kernel's end is written back
    // then, about 1 us, so small volumes stream on (32 MB at level 0, 264x144x16, 4 views: 13.4
    // and 14.3; 65 MB, 464x244x24, 2 views: 22.4 and 23.3; but 80 MB, 742x562x16, one: 28.8 and
    // 24.1), and so do translations (272x216x24, 2 views: 13.8 and 15.5).
    const bool meet = !shift && (src.W / 2) * 12 % 64 != 0 &&
                      (int64_t)src.N * D * src.H * src.W * 12 >= (int64_t)64 << 20;
    ProfScope ps(HSGD_K_PSV, s);
    for (int i = 0; i < src.N; i += nv)
        for (int z = 0; z < D; z += nd) {
            PsvOut o{};
            o.meet = meet;
            const size_t at = (size_t)i * D + z;
            for (int l = 0; l < L; ++l)
                if (out[l]) o.p[l] = (char*)out[l] + at * (size_t)(src.H >> l) * (size_t)(src.W >> l) * one;
            sweep_part(src.images + (size_t)i * src.H * src.W * 3, src.warps + at, std::min(nv, src.N - i),
                       std::min(nd, D - z), src.H, src.W, L, out_dtype, shift, o, s);
        }
    return (int)hipGetLastError();
}

}  // namespace hsgd
