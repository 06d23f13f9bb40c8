// Kernels of the learned warm start's 3-D U-Net (gfx950): BF16 MFMA implicit-GEMM
// 3x3x3 convolutions with FP32 accumulation, their backward passes, pooling,
// upsampling, the output head, the masked MSE loss and Adam.  The C ABI is in
// include/unet.h.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <algorithm>
#include <type_traits>

#include "../../include/unet.h"
#include "unet_kernels.h"

namespace {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float f32x4 __attribute__((__vector_size__(4 * sizeof(float))));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest even, NaN kept quiet: the conversion instruction (equal to the integer
// form, bits + 0x7fff + bit 16, over all 2^32 inputs)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

__host__ __device__ __forceinline__ int kpad_of(int cin) { return (27 * cin + 31) / 32 * 32; }

// elements of a layer's weights in fragment order (k_pack)
constexpr int64_t packed_len(int cin, int cout) { return (int64_t)(cin / 16) * (cout / 16) * 14 * 512; }

int status(hipError_t e) { return e == hipSuccess ? 0 : -6; }

// ------------------------------------------------------------------ conv3d forward
//
// Implicit GEMM: rows = voxels, columns = output channels, K = 27 taps x cin, on
// v_mfma_f32_16x16x32_bf16.  Fragment mapping (pinned by unet_mfma_selftest):
//   A[m][k]: lane l holds m = l % 16, k = 8 (l / 16) + j;  B[k][n]: n = l % 16, same k;
//   D[m][n]: lane l holds m = 4 (l / 16) + i, n = l % 16.
// K runs over stages of 16 input channels, in a stage over 14 chunks of two taps (the
// 28th tap is zero).  The weights are the MFMA's A operand and the inputs its B operand,
// so a lane's result is four consecutive output channels of one voxel, which leave as
// one 8-byte store.
//
// A wave owns four rows of 16 voxels in y of each plane and 16 output channels.  What
// bounded the product was the LDS: a chunk's input fragment (1 KB) read for every product
// is 256 bytes per cycle and CU at the matrix cores' rate, twice what the LDS gives.  So
// a wave takes an input plane at a time and reads each of its fragments once: chunks 0-3
// of the output plane above, 4-8 of the one at its height and 9-13 of the one below use
// the same three kinds of fragment (two neighbours in x, or the end of a row with the
// start of the next) of the wave's six halo rows.  19 reads serve 56 products, and every
// output still adds its chunks in the order 0 .. 13 of stage after stage.
//
// A workgroup is four waves: S slices of 16 output channels times 4 / S row groups of a
// tile of 16 x 16 / S voxels, so that the input copied into LDS serves S slices.
struct ConvArgs {
    const uint16_t *x;
    const uint16_t *w;
    const float *b;
    uint16_t *y;
    float *y32;
    int ldx, offx, ldy, offy;
    int nz, ny, nx, cin, cout, kpad, relu;
    uint32_t xbytes, plane_bytes;  // bytes of x and of one of its planes
    uint32_t wbytes;               // bytes of w
    // Input channels [cin1, cin) come from x2 instead (the concatenation of a skip
    // tensor and an upsampled one, never stored): rows of ldx2 at offset offx2, at
    // half resolution in every direction when up2 (nearest upsampling).
    const uint16_t *x2;
    int ldx2, offx2, cin1, up2;
    uint32_t x2bytes, plane2_bytes;
    // The network's 1x1x1 head fused into the last convolution (z-marching form,
    // 16 channels): hout[v] = hb + hbase[v] + sum_c hw[c] y[v, c] on the BF16 outputs,
    // which are then not stored.
    const float *hw, *hb, *hbase;
    float *hout;
    // The ReLU mask of the tensor written (backward): y is zeroed where m is not positive.
    const uint16_t *m;
    int ldm, offm;
    int packed;  // w is in the order of k_pack rather than in rows of kpad
};

typedef __attribute__((address_space(3))) void lds_void;

// four BF16 values with those zeroed whose mask value is not positive (not > 0: negative,
// zero or NaN)
__device__ __forceinline__ uint32_t mask_pair(uint32_t v, uint32_t m) {
    const bool lo = __uint_as_float(m << 16) > 0.f, hi = __uint_as_float(m & 0xffff0000u) > 0.f;
    return (lo ? v & 0xffffu : 0u) | (hi ? v & 0xffff0000u : 0u);
}
__device__ __forceinline__ uint2 mask4(uint2 v, uint2 m) { return make_uint2(mask_pair(v.x, m.x), mask_pair(v.y, m.y)); }

// dword 3 of a raw (untyped, unswizzled) buffer resource on the gfx9 family
constexpr int kRawBuffer = 0x00020000;
// Input planes and weights are read through buffer resources with 32-bit offsets:
// x and w stay below 2 GiB so that kNoOff lies past their ends, and a load at kNoOff
// returns zeros (the staged entries outside the grid, the weights past the 27th tap).
constexpr int64_t kMaxX = ((int64_t)1 << 31) - 16;
constexpr uint32_t kNoOff = 0x80000000u;

constexpr int kCC = 16;                  // input channels per stage
constexpr int kVS = 16;  // LDS elements per voxel: the 16 channels, unpadded.  A 32-byte voxel
                         // stride reads at the full LDS rate on gfx950 (the lanes' 16-byte
                         // reads tile whole 512-byte spans); a padded 48-byte stride ran 1.5x slower
constexpr int64_t kConvSlots = 512;       // workgroups a chip holds: two on each of 256 CUs
constexpr int kKC = 14;  // K chunks of 32 per stage: 27 taps x 16 channels, the last half empty
// s_waitcnt vmcnt(n), the other counters not waited for (gfx9 encoding)
constexpr int wait_vmcnt(int n) { return 0x0F70 | (n & 15) | (n >> 4) << 14; }
constexpr int kWaitVmcnt0 = wait_vmcnt(0);
// Around a wait whose count says which of this wave's copies, stores and loads may still be
// out: nothing is moved from one side of it to the other, or the count would not hold.
__device__ __forceinline__ void pin() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The tile of this workgroup: x and y origin, chunk of planes and group of channel slices.
// The grid is (x-y tiles, chunks, groups).  Workgroups reach the 8 XCDs round-robin by
// launch index b; XCD b % 8 takes a contiguous eighth of the tile order, so that tiles
// sharing input rows and planes run together under one L2.  Within a group the tiles go in
// bands of 16 rows in y: x fastest, then y within the band, then the chunks, then the bands
// (the last band may be shorter).
struct ConvTile {
    int x0, y0, zc, slice;
};
template <int TX, int TY>
__device__ __forceinline__ ConvTile conv_tile(int nx) {
    const int nxt = (nx + TX - 1) / TX;
    const int nblk = (int)(gridDim.x * gridDim.y * gridDim.z);
    const int b = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
    const int xcd = b % 8, per = nblk / 8, extra = nblk % 8;
    const int t = xcd * per + min(xcd, extra) + b / 8;
    constexpr int kYB = 16 / TY;
    const int nyt = (int)gridDim.x / nxt, nzc = (int)gridDim.y;
    const int per_slice = (int)gridDim.x * nzc;
    const int slice = t / per_slice, rem = t % per_slice;
    const int band = rem / (nxt * kYB * nzc), in_band = rem % (nxt * kYB * nzc);
    const int h = min(kYB, nyt - band * kYB);
    const int xt = in_band % nxt, yin = (in_band / nxt) % h, zc = in_band / (nxt * h);
    return ConvTile{xt * TX, (band * kYB + yin) * TY, zc, slice};
}

// A workgroup's tile: S channel slices times 4 / S waves of four rows of 16 voxels each, XG
// of them side by side in x and the others on top of each other in y.
template <int S, int XG>
struct Tile {
    static constexpr int TX = 16 * XG, TY = 16 / (S * XG);
    static constexpr int BX = TX + 2, PLANE = BX * (TY + 2);  // an input plane, halo included
    int x, y, slice;  // this wave's first voxel in the tile, and its slice of the workgroup's
    __device__ __forceinline__ explicit Tile(int wave)
        : x(16 * (wave % XG)), y(4 * (wave % (4 / S) / XG)), slice(wave / (4 / S)) {}
};

__device__ __forceinline__ bf16x8 lane_select(bool second, bf16x8 x, bf16x8 y) {
    const uint4 a = __builtin_bit_cast(uint4, x), b = __builtin_bit_cast(uint4, y);
    return __builtin_bit_cast(bf16x8, make_uint4(second ? a.x : b.x, second ? a.y : b.y, second ? a.z : b.z, second ? a.w : b.w));
}

// Fragments of one input plane for a wave's four rows of 16 voxels, halo rows 0 .. 5:
// a[r] holds taps x, x + 1 of row r, b[r] taps x + 1, x + 2, and c[r + 1] tap x + 2 of row r
// with tap x of row r + 1 (the two taps of a chunk lie in the two halves of the lanes);
// p: the rows 2 .. 5 of c of the plane before.
struct Frags {
    bf16x8 a[6], b[6], c[7], p[4];
};
// where a lane reads them (LDS elements from the plane's start); BX: voxels of a halo row
template <int BX>
struct FragAt {
    int a, c, d;
    __device__ __forceinline__ FragAt(int row, int x, int kb) {
        const int chan = 8 * (kb & 1), g = kb >> 1;
        a = (row * BX + x + g) * kVS + chan;
        c = (g ? (row + 1) * BX + x : row * BX + x + 2) * kVS + chan;
        d = (row * BX + x) * kVS + chan;
    }
};
__device__ __forceinline__ bf16x8 frag(const uint16_t *p, int voxel) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p + voxel * kVS));
}
template <int BX>
__device__ __forceinline__ void read_a(Frags &F, const uint16_t *plane, const FragAt<BX> &at) {
#pragma unroll
    for (int r = 0; r < 6; ++r) F.a[r] = frag(plane + at.a, r * BX);
}
template <int BX>
__device__ __forceinline__ void read_b(Frags &F, const uint16_t *plane, const FragAt<BX> &at) {
#pragma unroll
    for (int r = 0; r < 6; ++r) F.b[r] = frag(plane + at.a, r * BX + 1);
}
template <int BX>
__device__ __forceinline__ void read_c(Frags &F, const uint16_t *plane, const FragAt<BX> &at) {
    F.c[0] = frag(plane + at.d, 0);
#pragma unroll
    for (int r = 0; r < 5; ++r) F.c[r + 1] = frag(plane + at.c, r * BX);
    F.c[6] = frag(plane + at.d, 5 * BX + 2);
}
// The products of one input plane: chunks 0 .. 3 of the output plane above it (D0), 4 .. 8
// of the one at its height (D1), 9 .. 13 of the one below (D2).  Expects a and c read;
// next_a() and next_c() run once a and c are no longer needed.
template <bool D0, bool D1, bool D2, int BX, class NextA, class NextC>
__device__ __forceinline__ void plane_products(Frags &F, const uint16_t *plane, const FragAt<BX> &at, bool second,
                                               const bf16x8 (&B)[kKC], f32x4 (&above)[4], f32x4 (&level)[4],
                                               f32x4 (&below)[4], NextA next_a, NextC next_c) {
    auto mm = [&](int q, bf16x8 x, f32x4 &c) { c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B[q], x, c, 0, 0, 0); };
    const bf16x8 zero = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
    read_b(F, plane, at);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D0) mm(0, F.a[t], above[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D2) mm(9, F.a[t], below[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D0) mm(1, F.c[t + 1], above[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D2) mm(10, F.c[t + 1], below[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D1) mm(4, lane_select(second, F.c[t], F.p[t]), level[t]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D0) mm(2, F.b[t + 1], above[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D2) mm(11, F.b[t + 1], below[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D1) mm(5, F.b[t], level[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D0) mm(3, F.a[t + 2], above[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D2) mm(12, F.a[t + 2], below[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D1) mm(6, F.a[t + 1], level[t]);
    __builtin_amdgcn_sched_barrier(0);
    next_a();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D1) mm(7, F.c[t + 2], level[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D2) mm(13, lane_select(second, zero, F.c[t + 3]), below[t]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) F.p[t] = F.c[t + 3];
    next_c();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) if (D1) mm(8, F.b[t + 2], level[t]);
    __builtin_amdgcn_sched_barrier(0);
}
// All of them for the ZC + 2 planes of a slab, one stage; next(from, to): the weights of
// chunks from .. to - 1 are no longer needed.
template <int I, int ZC, int PLANE, int BX, class Next>
__device__ __forceinline__ void slab_products(Frags &F, const uint16_t *slab, const FragAt<BX> &at, bool second,
                                              const bf16x8 (&B)[kKC], f32x4 (&acc)[ZC][4], Next next) {
    constexpr bool D0 = I < ZC, D1 = I >= 1 && I <= ZC, D2 = I >= 2;
    const uint16_t *plane = slab + I * PLANE * kVS, *after = plane + PLANE * kVS;
    plane_products<D0, D1, D2>(
        F, plane, at, second, B, acc[D0 ? I : 0], acc[D1 ? I - 1 : 0], acc[D2 ? I - 2 : 0],
        [&]() __attribute__((always_inline)) { if (I <= ZC) read_a(F, after, at); },
        [&]() __attribute__((always_inline)) { if (I <= ZC) read_c(F, after, at); });
    if (I == ZC - 1) next(0, 4);
    if (I == ZC) next(4, 9);
    if (I == ZC + 1) next(9, kKC);
    if constexpr (I <= ZC) slab_products<I + 1, ZC, PLANE>(F, slab, at, second, B, acc, next);
}

// ZC output planes per workgroup; a stage's ZC + 2 input planes are copied straight from
// global memory into LDS, all in flight at once, then multiplied.  The weights of a chunk
// are fetched for the next stage as soon as its last product is out.  Two workgroups per CU
// (160 .. 241 VGPRs, 10 .. 62 KB of LDS), one's copies under the other's products.
// us before (one 4 x 64 tile and slice per workgroup, fragments read per product) and now
// with packed weights: 96 -> 32 channels at 96^3 307 -> 144 (1.0 PFLOP/s), 192 -> 64 at 48^3
// 164 -> 67, 64 -> 64 at 48^3 63 -> 26 (rows of kpad 31), 192 -> 64 at 24^3 57 -> 23,
// 128 -> 128 at 12^3 39 -> 12.4.
template <int S, int ZC, int XG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_slab(ConvArgs a) {
    constexpr int BX = Tile<S, XG>::BX, PLANE = Tile<S, XG>::PLANE, NE = 2 * PLANE, PS = (NE + 255) / 256;
    constexpr int kSlab = (ZC + 2) * PLANE * kVS;
    __shared__ __attribute__((aligned(16))) uint16_t slab[kSlab];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Tile<S, XG> W(wave);
    const ConvTile T = conv_tile<Tile<S, XG>::TX, Tile<S, XG>::TY>(a.nx);
    const int x0 = T.x0, y0 = T.y0, z0 = T.zc * ZC, co0 = 16 * (T.slice * S + W.slice);
    const int m = lane & 15, kb = lane >> 4, chan = 8 * (kb & 1);
    const bool second = kb >> 1;
    f32x4 acc[ZC][4];
#pragma unroll
    for (int p = 0; p < ZC; ++p)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[p][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.w), (short)0, (int)a.wbytes, kRawBuffer);
    // this lane's weights, and the bytes from one chunk, one stage to the next
    const uint32_t wlane = a.packed ? 2u * (uint32_t)((co0 / 16) * (a.cin / kCC) * kKC * 512 + 8 * lane)
                                    : 2u * (uint32_t)((co0 + m) * a.kpad + (kb >> 1) * a.cin + chan);
    const uint32_t wchunk = a.packed ? 1024u : 4u * (uint32_t)a.cin, wstage = a.packed ? kKC * 1024u / kCC : 2u;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x), (short)0, (int)a.xbytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rx2 =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x2), (short)0, (int)a.x2bytes, kRawBuffer);
    uint32_t poff[PS];
    auto source_offsets = [&](bool from2) __attribute__((always_inline)) {
        const int sh = from2 && a.up2 ? 1 : 0, ld = from2 ? a.ldx2 : a.ldx, off = from2 ? a.offx2 : a.offx;
#pragma unroll
        for (int it = 0; it < PS; ++it) {
            const int e = tid + 256 * it, bv = e >> 1, h = e & 1;
            const int xx = x0 + bv % BX - 1, yy = y0 + bv / BX - 1;
            const bool in = xx >= 0 && xx < a.nx && yy >= 0 && yy < a.ny;
            poff[it] = in ? 2u * (uint32_t)(((yy >> sh) * (a.nx >> sh) + (xx >> sh)) * ld + off + 8 * h) : kNoOff;
        }
    };
    auto copy_stage = [&](int c0) __attribute__((always_inline)) {
        if (c0 == 0 || c0 == a.cin1) source_offsets(c0 >= a.cin1);
        const bool from2 = c0 >= a.cin1;
#pragma unroll
        for (int s = 0; s < ZC + 2; ++s) {
            const int zz = z0 - 1 + s;
            const bool zin = zz >= 0 && zz < a.nz;  // else the whole plane reads as zeros
            const uint32_t zoff = !zin    ? 0u
                                  : from2 ? (uint32_t)(a.up2 ? zz >> 1 : zz) * a.plane2_bytes + 2u * (uint32_t)(c0 - a.cin1)
                                          : (uint32_t)zz * a.plane_bytes + 2u * (uint32_t)c0;
#pragma unroll
            for (int it = 0; it < PS; ++it) {
                const int e0 = 256 * it + 64 * wave, e = e0 + lane;
                if (e0 >= NE) break;  // wave-uniform
                const uint32_t off = zin ? poff[it] : kNoOff;
                uint16_t *to = slab + s * PLANE * kVS + 8 * e0;
                if (e < NE) __builtin_amdgcn_raw_ptr_buffer_load_lds(from2 ? rx2 : rx, (lds_void *)to, 16, off, zoff, 0, 0);
            }
        }
    };
    const FragAt<BX> at(W.y, W.x + m, kb);
    Frags F{};
    bf16x8 B[kKC];
    auto load_weights = [&](int c0, int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int q = from; q < to; ++q) {
            const int tap = 2 * q + (kb >> 1);  // past the 27th tap the offset lies past w: zeros
            const uint32_t off = tap < 27 ? wlane : kNoOff;
            B[q] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, off, wchunk * q + wstage * c0, 0));
        }
    };
    load_weights(0, 0, kKC);
    for (int c0 = 0; c0 < a.cin; c0 += kCC) {
        if (c0) __syncthreads();  // the previous stage's reads of the slab are done
        copy_stage(c0);
        __syncthreads();  // waits for the copies (vmcnt) and publishes them
        read_a(F, slab, at);
        read_c(F, slab, at);
        slab_products<0, ZC, PLANE>(F, slab, at, second, B, acc, [&](int from, int to) __attribute__((always_inline)) {
            if (c0 + kCC < a.cin) load_weights(c0 + kCC, from, to);
        });
    }
    const int xx = x0 + W.x + m, c = co0 + 4 * kb;
    if (xx >= a.nx) return;
    float bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i] = a.b ? a.b[c + i] : 0.f;
#pragma unroll
    for (int p = 0; p < ZC; ++p) {
        const int zz = z0 + p;
        if (zz >= a.nz) break;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int yy = y0 + W.y + t;
            if (yy >= a.ny) break;
            const int64_t vm = ((int64_t)zz * a.ny + yy) * a.nx + xx;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = acc[p][t][i] + bias[i];
                if (a.relu) v[i] = fmaxf(v[i], 0.f);
            }
            uint2 o = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
            if (a.m) o = mask4(o, *reinterpret_cast<const uint2 *>(a.m + vm * a.ldm + a.offm + c));
            *reinterpret_cast<uint2 *>(a.y + vm * a.ldy + a.offy + c) = o;
            if (a.y32) *reinterpret_cast<float4 *>(a.y32 + vm * a.cout + c) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

// The same with the LDS planes as a ring over (stage, plane): as soon as every wave is done
// with a plane, the next stage's plane of that place is copied into it, ZC + 1 steps before
// it is read.  For 16 output channels on large grids, where a copy serves one slice only and
// comes from beyond the L2: 48 -> 16 at 192^3 445 -> 371 us (558 before either).  Elsewhere a
// barrier per plane costs what the overlap gives (96 -> 32 at 96^3 144 and 143 us, 64 -> 64 at
// 48^3 26 and 28, 128 -> 128 at 12^3 12.4 and 14).
template <int S, int ZC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_ring(ConvArgs a) {
    constexpr int XG = 1, BX = Tile<S, XG>::BX, PLANE = Tile<S, XG>::PLANE, C = (2 * PLANE + 255) / 256, SLOT = 256 * C * 8;
    __shared__ __attribute__((aligned(16))) uint16_t slab[(ZC + 2) * SLOT];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Tile<S, XG> W(wave);
    const ConvTile T = conv_tile<Tile<S, XG>::TX, Tile<S, XG>::TY>(a.nx);
    const int x0 = T.x0, y0 = T.y0, z0 = T.zc * ZC, co0 = 16 * (T.slice * S + W.slice);
    const int m = lane & 15, kb = lane >> 4;
    const bool second = kb >> 1;
    f32x4 acc[ZC][4];
#pragma unroll
    for (int p = 0; p < ZC; ++p)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[p][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.w), (short)0, (int)a.wbytes, kRawBuffer);
    // this lane's weights, and the bytes from one chunk, one stage to the next
    const uint32_t wlane = a.packed ? 2u * (uint32_t)((co0 / 16) * (a.cin / kCC) * kKC * 512 + 8 * lane)
                                    : 2u * (uint32_t)((co0 + m) * a.kpad + (kb >> 1) * a.cin + 8 * (kb & 1));
    const uint32_t wchunk = a.packed ? 1024u : 4u * (uint32_t)a.cin, wstage = a.packed ? kKC * 1024u / kCC : 2u;
    bf16x8 B[kKC];
    auto load_weights = [&](int c0, int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int q = from; q < to; ++q) {
            const int tap = 2 * q + (kb >> 1);  // past the 27th tap the offset lies past w: zeros
            const uint32_t off = tap < 27 ? wlane : kNoOff;
            B[q] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, off, wchunk * q + wstage * c0, 0));
        }
    };
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x), (short)0, (int)a.xbytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rx2 =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x2), (short)0, (int)a.x2bytes, kRawBuffer);
    uint32_t poff[C];
    auto source_offsets = [&](bool from2) __attribute__((always_inline)) {
        const int sh = from2 && a.up2 ? 1 : 0, ld = from2 ? a.ldx2 : a.ldx, off = from2 ? a.offx2 : a.offx;
#pragma unroll
        for (int it = 0; it < C; ++it) {
            const int e = tid + 256 * it, bv = e >> 1, h = e & 1;
            const int xx = x0 + bv % BX - 1, yy = y0 + bv / BX - 1;
            const bool in = bv < PLANE && xx >= 0 && xx < a.nx && yy >= 0 && yy < a.ny;
            poff[it] = in ? 2u * (uint32_t)(((yy >> sh) * (a.nx >> sh) + (xx >> sh)) * ld + off + 8 * h) : kNoOff;
        }
    };
    // plane `slot` of the stage of channels c0 ..: C copies by every wave, so that the waits
    // can count them (the entries past the plane land in the slot's tail)
    auto copy_plane = [&](int c0, int slot) __attribute__((always_inline)) {
        const bool from2 = c0 >= a.cin1;
        const int zz = z0 - 1 + slot;
        const bool zin = zz >= 0 && zz < a.nz;  // else the whole plane reads as zeros
        const uint32_t zoff = !zin    ? 0u
                              : from2 ? (uint32_t)(a.up2 ? zz >> 1 : zz) * a.plane2_bytes + 2u * (uint32_t)(c0 - a.cin1)
                                      : (uint32_t)zz * a.plane_bytes + 2u * (uint32_t)c0;
#pragma unroll
        for (int it = 0; it < C; ++it) {
            const uint32_t off = zin ? poff[it] : kNoOff;
            uint16_t *to = slab + slot * SLOT + 8 * (256 * it + 64 * wave);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(from2 ? rx2 : rx, (lds_void *)to, 16, off, zoff, 0, 0);
        }
    };
    const FragAt<BX> at(W.y, W.x + m, kb);
    Frags F{};
    source_offsets(false);
    load_weights(0, 0, kKC);
#pragma unroll
    for (int s = 0; s <= ZC; ++s) copy_plane(0, s);
    auto step = [&](auto I, int c0, bool last) __attribute__((always_inline)) {
        constexpr int s = decltype(I)::value;
        constexpr bool D0 = s < ZC, D1 = s >= 1 && s <= ZC, D2 = s >= 2;
        // This wave's copies of the plane have landed when no more than the younger loads are
        // out: ZC planes' copies and the weights fetched since (in the first stage the weights
        // came first), or what is left of this stage's copies in the last
        constexpr int kYounger = ZC * C, kTail = ZC > s ? (ZC - s) * C : 0;
        constexpr int kWeights = (s + 1 <= ZC - 1 ? 4 : 0) + (s + 1 <= ZC ? 5 : 0) + (s + 1 <= ZC + 1 ? 5 : 0);
        pin();
        if (last)
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(kTail));
        else if (c0 == 0)
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(kYounger));
        else
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(kYounger + kWeights));
        __builtin_amdgcn_s_barrier();  // everyone's have, and everyone is done with the plane before
        pin();
        if (s == 0) {
            copy_plane(c0, ZC + 1);
        } else if (!last) {
            if (s == 1 && c0 + kCC == a.cin1) source_offsets(true);
            copy_plane(c0 + kCC, s - 1);
        }
        const uint16_t *plane = slab + s * SLOT;
        read_a(F, plane, at);
        read_c(F, plane, at);
        plane_products<D0, D1, D2>(F, plane, at, second, B, acc[D0 ? s : 0], acc[D1 ? s - 1 : 0], acc[D2 ? s - 2 : 0],
                                   []() {}, []() {});
        if (!last) {
            if (s == ZC - 1) load_weights(c0 + kCC, 0, 4);
            if (s == ZC) load_weights(c0 + kCC, 4, 9);
            if (s == ZC + 1) load_weights(c0 + kCC, 9, kKC);
        }
    };
    for (int c0 = 0; c0 < a.cin; c0 += kCC) {
        const bool last = c0 + kCC >= a.cin;
        step(std::integral_constant<int, 0>{}, c0, last);
        step(std::integral_constant<int, 1>{}, c0, last);
        step(std::integral_constant<int, 2>{}, c0, last);
        if constexpr (ZC >= 2) step(std::integral_constant<int, 3>{}, c0, last);
        if constexpr (ZC >= 3) step(std::integral_constant<int, 4>{}, c0, last);
        if constexpr (ZC >= 4) step(std::integral_constant<int, 5>{}, c0, last);
    }
    const int xx = x0 + W.x + m, c = co0 + 4 * kb;
    if (xx >= a.nx) return;
    float bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i] = a.b ? a.b[c + i] : 0.f;
#pragma unroll
    for (int p = 0; p < ZC; ++p) {
        const int zz = z0 + p;
        if (zz >= a.nz) break;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int yy = y0 + W.y + t;
            if (yy >= a.ny) break;
            const int64_t vm = ((int64_t)zz * a.ny + yy) * a.nx + xx;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = acc[p][t][i] + bias[i];
                if (a.relu) v[i] = fmaxf(v[i], 0.f);
            }
            uint2 o = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
            if (a.m) o = mask4(o, *reinterpret_cast<const uint2 *>(a.m + vm * a.ldm + a.offm + c));
            *reinterpret_cast<uint2 *>(a.y + vm * a.ldy + a.offy + c) = o;
            if (a.y32) *reinterpret_cast<float4 *>(a.y32 + vm * a.cout + c) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

// The head on a wave's four rows of results (o[r]: row r, this lane's four channels): the
// 16-lane groups' quarters and the rows change places, so that each lane has all 16 channels
// of its voxel in row lane / 16 and adds them in channel order, as unet_head_fwd does.  (The
// sum handed from group to group, row by row, took the last convolution at 192^3 154 us; now
// it takes 119.)
__device__ __forceinline__ float head_of_rows(const uint2 (&o)[4], const float (&hw)[16], float sum) {
    uint32_t q[4][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        auto half = [&](int r) { return h ? o[r].y : o[r].x; };
        const auto ac = __builtin_amdgcn_permlane32_swap(half(0), half(2), false, false);
        const auto bd = __builtin_amdgcn_permlane32_swap(half(1), half(3), false, false);
        const auto lo = __builtin_amdgcn_permlane16_swap(ac[0], bd[0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(ac[1], bd[1], false, false);
        q[0][h] = lo[0];
        q[1][h] = lo[1];
        q[2][h] = hi[0];
        q[3][h] = hi[1];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t w = q[i / 4][i / 2 % 2];
        sum = fmaf(hw[i], __uint_as_float(i % 2 ? w & 0xffff0000u : w << 16), sum);
    }
    return sum;
}

// Single-stage form for 16 input channels: a workgroup marches through a run of zr output
// planes of its tile, one input plane per step, three output planes in flight in registers.
// Input plane z0 - 1 + i lives in ring slot i % 4 (four distinct LDS arrays, chosen at
// compile time by a loop unrolled four times, or the compiler waits for every copy before
// every read); each plane is copied once per run, three steps before it is read.  A finished
// plane is stored in the next step.  Bound by the copies' and stores' way to memory at 192^3
// (64 bytes per voxel: 4.2 TB/s).  236 VGPRs: two workgroups per CU.  HEAD: the head is
// applied in the epilogue and only its FP32 output is stored.  MASK: a.m is not null.
// Before (4 x 64 tiles, fragments read per product) and now: 16 -> 16 at 192^3 176 -> 108 us,
// at 96^3 37 -> 20; 16 -> 32 at 96^3 56 -> 31.
template <int S, bool HEAD, bool MASK, int XG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_march(ConvArgs a, int zr) {
    constexpr int BX = Tile<S, XG>::BX, PLANE = Tile<S, XG>::PLANE, NE = 2 * PLANE, PS = (NE + 255) / 256;
    __shared__ __attribute__((aligned(16))) uint16_t s0[PLANE * kVS], s1[PLANE * kVS], s2[PLANE * kVS], s3[PLANE * kVS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Tile<S, XG> W(wave);
    const ConvTile T = conv_tile<Tile<S, XG>::TX, Tile<S, XG>::TY>(a.nx);
    const int x0 = T.x0, y0 = T.y0, z0 = T.zc * zr, co0 = 16 * (T.slice * S + W.slice);
    const int n = min(zr, a.nz - z0);
    const int m = lane & 15, kb = lane >> 4, c = co0 + 4 * kb, xx = x0 + W.x + m, yw = y0 + W.y;
    const bool second = kb >> 1;
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.w), (short)0, (int)a.wbytes, kRawBuffer);
    const uint32_t wlane = a.packed ? 2u * (uint32_t)((co0 / 16) * kKC * 512 + 8 * lane)
                                    : 2u * (uint32_t)((co0 + m) * a.kpad + (kb >> 1) * a.cin + 8 * (kb & 1));
    const uint32_t wchunk = a.packed ? 1024u : 4u * (uint32_t)a.cin;
    bf16x8 B[kKC];
#pragma unroll
    for (int q = 0; q < kKC; ++q) {
        const uint32_t off = 2 * q + (kb >> 1) < 27 ? wlane : kNoOff;
        B[q] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, off, wchunk * q, 0));
    }
    float bias[4], hw[16], hb = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bias[i] = a.b ? a.b[c + i] : 0.f;
    }
    if (HEAD) {
        hb = a.hb[0];
#pragma unroll
        for (int i = 0; i < 16; ++i) hw[i] = a.hw[i];
    }
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x), (short)0, (int)a.xbytes, kRawBuffer);
    uint32_t poff[PS];
#pragma unroll
    for (int it = 0; it < PS; ++it) {
        const int e = tid + 256 * it, bv = e >> 1, h = e & 1;
        const int xq = x0 + bv % BX - 1, yq = y0 + bv / BX - 1;
        const bool in = xq >= 0 && xq < a.nx && yq >= 0 && yq < a.ny;
        poff[it] = in ? 2u * (uint32_t)((yq * a.nx + xq) * a.ldx + a.offx + 8 * h) : kNoOff;
    }
    auto copy_plane = [&](int zz, uint16_t *slot) __attribute__((always_inline)) {
        const bool zin = zz >= 0 && zz < a.nz;  // else the plane reads as zeros
        const uint32_t zoff = zin ? (uint32_t)zz * a.plane_bytes : 0u;
#pragma unroll
        for (int it = 0; it < PS; ++it) {
            const int e0 = 256 * it + 64 * wave, e = e0 + lane;
            if (e0 >= NE) break;  // wave-uniform
            const uint32_t off = zin ? poff[it] : kNoOff;
            uint16_t *to = slot + 8 * e0;
            if (e < NE) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)to, 16, off, zoff, 0, 0);
        }
    };
    uint2 pend[4];
    float hpend = 0.f;  // HEAD: the output of this lane's voxel of row kb
    int pend_z = -1;
    auto flush = [&]() __attribute__((always_inline)) {
        if (pend_z < 0 || xx >= a.nx) return;
        const int64_t vm = ((int64_t)pend_z * a.ny + yw) * a.nx + xx;
        if (HEAD) {
            if (yw + kb < a.ny) a.hout[vm + (int64_t)kb * a.nx] = hpend;
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (yw + t >= a.ny) break;
            *reinterpret_cast<uint2 *>(a.y + (vm + (int64_t)t * a.nx) * a.ldy + a.offy + c) = pend[t];
        }
    };
    auto ring = [&](int i) __attribute__((always_inline)) -> uint16_t * {
        i &= 3;
        return i == 0 ? s0 : i == 1 ? s1 : i == 2 ? s2 : s3;
    };
    const FragAt<BX> at(W.y, W.x + m, kb);
    Frags F{};
    f32x4 above[4], level[4], below[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) above[t] = level[t] = below[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const bool full = yw + 4 <= a.ny && x0 + W.x < a.nx;  // this wave stores all four rows
    constexpr int kMinCopies = NE / 256, kStores = HEAD ? 1 : 4;  // of every wave for a plane
    copy_plane(z0 - 1, s0);
    copy_plane(z0, s1);
    copy_plane(z0 + 1, s2);
    // weights and the first planes: waited for here, or the compiler waits for the weights
    // (and with them for every copy issued since) in each trip of the loop
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    for (int i0 = 0; i0 < n + 2; i0 += 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + k;
            if (i >= n + 2) break;
            // this wave's copies of this plane have landed: in the steady state two planes'
            // copies (at least kMinCopies per wave each) and two planes' stores are younger
            pin();
            if (i < n && i >= 5 && full)
                __builtin_amdgcn_s_waitcnt(wait_vmcnt(2 * kStores + 2 * kMinCopies));
            else if (i < n)
                __builtin_amdgcn_s_waitcnt(wait_vmcnt(2 * kMinCopies));
            else
                __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            __builtin_amdgcn_s_barrier();
            pin();
            const int pz = z0 + i - 2;  // the output plane this step completes
            float hbase = 0.f;
            uint2 mask[4];
            if (HEAD && a.hbase && i >= 2 && xx < a.nx && yw + kb < a.ny)
                hbase = a.hbase[((int64_t)pz * a.ny + yw + kb) * a.nx + xx];
            if (MASK && i >= 2 && xx < a.nx) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int64_t vm = ((int64_t)pz * a.ny + yw + t) * a.nx + xx;
                    const bool in = yw + t < a.ny;
                    mask[t] = in ? *reinterpret_cast<const uint2 *>(a.m + vm * a.ldm + a.offm + c) : make_uint2(0u, 0u);
                }
            }
            flush();
            if (i + 3 < n + 2) copy_plane(z0 - 1 + i + 3, ring(k + 3));
            uint16_t *slot = ring(k);
            read_a(F, slot, at);
            read_c(F, slot, at);
            plane_products<true, true, true>(F, slot, at, second, B, above, level, below, []() {}, []() {});
            if (i >= 2) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        v[j] = below[t][j] + bias[j];
                        if (a.relu) v[j] = fmaxf(v[j], 0.f);
                    }
                    uint2 o = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
                    if (MASK) o = mask4(o, mask[t]);
                    pend[t] = o;
                    if (a.y32 && yw + t < a.ny && xx < a.nx)
                        *reinterpret_cast<float4 *>(a.y32 + (((int64_t)pz * a.ny + yw + t) * a.nx + xx) * a.cout + c) =
                            make_float4(v[0], v[1], v[2], v[3]);
                }
                if (HEAD) hpend = head_of_rows(pend, hw, hb + hbase);
                pend_z = pz;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                below[t] = level[t];
                level[t] = above[t];
                above[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    flush();
}

// wt[ci][tap' * cout + co] = w[co][(26 - tap') * cin + ci]
__global__ void k_wtrans(const uint16_t *w, uint16_t *wt, int cin, int cout, int kpad_in, int kpad_out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)cin * kpad_out) return;
    const int ci = (int)(i / kpad_out), kk = (int)(i % kpad_out);
    uint16_t v = 0;
    if (kk < 27 * cout) {
        const int tp = kk / cout, co = kk % cout;
        v = w[(int64_t)co * kpad_in + (26 - tp) * cin + ci];
    }
    wt[i] = v;
}

// Weights in fragment order, for the layers of a table (blockIdx.y the layer): the 14 chunks
// of each 16-channel stage of each 16-channel slice of the outputs, every chunk the 16
// bytes of each lane in turn.  A wave's fragment is then one run of 1 KB; from rows of
// kpad it takes 32 pieces of 32 bytes out of as many cache lines.
__global__ void k_pack(const uint16_t *w, uint16_t *packed, unet::PackTable t) {
    const unet::PackLayer L = t.l[blockIdx.y];
    const int stages = L.cin / 16;
    const uint16_t *src = w + L.from;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < packed_len(L.cin, L.cout) / 8;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (int)(i % 64), q = (int)(i / 64 % kKC), st = (int)(i / (64 * kKC) % stages);
        const int n = 16 * (int)(i / (64 * kKC * stages)) + lane % 16;         // output channel
        const int tap = 2 * q + lane / 32, k = 16 * st + 8 * (lane / 16 % 2);  // tap and first input channel
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (tap < 27) {
            if (!L.transposed) {
                v = *reinterpret_cast<const uint4 *>(src + (int64_t)n * kpad_of(L.cin) + tap * L.cin + k);
            } else {  // the roles of the channels and the taps reversed; w has L.cin outputs
                const uint16_t *p = src + (int64_t)k * kpad_of(L.cout) + (26 - tap) * L.cout + n;
                uint32_t e[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) e[j] = p[(int64_t)j * kpad_of(L.cout)];
                v = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
            }
        }
        *reinterpret_cast<uint4 *>(packed + L.to + 8 * i) = v;
    }
}

// ------------------------------------------------------------------ conv3d weight gradient
//
// dw[co][k] += sum_v dy[v][co] X(v, k) with X the im2col view of x: a GEMM whose
// reduction runs over the voxels.  On the 16x16x32 BF16 MFMA: M = output channel,
// N = k, K = 32 voxels per instruction.  A workgroup (4 waves) owns 16*NCO output
// channels x 128 k over a voxel range; per stage it stages 32 voxels of dy and of
// X into LDS transposed (voxels fastest), so each lane reads its 8-voxel fragment
// with one 16-byte LDS load; each wave accumulates NCO x 2 tiles of 16 x 16 in FP32
// and adds them to dw atomically at the end.
constexpr int kWgStage = 32;  // voxels per stage (the MFMA's K)
constexpr int kWgK = 128;     // k per workgroup
constexpr int kWgPad = 40;    // LDS row length (bf16): 32 voxels + 8 against bank conflicts

template <int NCO>
__global__ __launch_bounds__(256) void k_wgrad(const uint16_t *x, int ldx, int offx, const uint16_t *dy, int lddy,
                                               int offdy, int nz, int ny, int nx, int cin, int cout, int kpad,
                                               int64_t vper, float *dw, float *db) {
    __shared__ __attribute__((aligned(16))) uint16_t XT[kWgK][kWgPad];
    __shared__ __attribute__((aligned(16))) uint16_t DT[16 * NCO][kWgPad];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k0 = blockIdx.x * kWgK, co0 = blockIdx.z * 16 * NCO;
    const int K = 27 * cin;
    const int64_t nvox = (int64_t)nz * ny * nx;
    const int64_t v0 = (int64_t)blockIdx.y * vper;
    const int64_t v1 = min(nvox, v0 + vper);
    // staging roles: X: voxel sv = tid / 8, two 8-wide k chunks c = tid % 8 and + 8
    const int sv = tid >> 3, sc = tid & 7;
    int ck[2], cdz[2], cdy[2], cdx[2], cci[2];
    bool cok[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int k = k0 + 8 * (sc + 8 * h);
        cok[h] = k < K;
        const int tap = cok[h] ? k / cin : 0;
        ck[h] = 8 * (sc + 8 * h);
        cci[h] = k - tap * cin;
        cdz[h] = tap / 9 - 1;
        cdy[h] = (tap / 3) % 3 - 1;
        cdx[h] = tap % 3 - 1;
    }
    // dy: voxel sv, channels 8 * sc .. when 8 * sc < 16 * NCO
    const bool dact = 8 * sc < 16 * NCO;
    f32x4 acc[NCO][2];
#pragma unroll
    for (int c = 0; c < NCO; ++c)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[c][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float bacc = 0.f;
    const int m = lane & 15, q = lane >> 4;
    for (int64_t vs = v0; vs < v1; vs += kWgStage) {
        const int64_t v = vs + sv;
        const bool vok = v < v1;
        int xx = 0, yy = 0, zz = 0;
        if (vok) {
            xx = (int)(v % nx);
            const int64_t r = v / nx;
            yy = (int)(r % ny);
            zz = (int)(r / ny);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint4 val = make_uint4(0u, 0u, 0u, 0u);
            const int z2 = zz + cdz[h], y2 = yy + cdy[h], x2 = xx + cdx[h];
            if (vok && cok[h] && z2 >= 0 && z2 < nz && y2 >= 0 && y2 < ny && x2 >= 0 && x2 < nx) {
                const int64_t nb = ((int64_t)z2 * ny + y2) * nx + x2;
                val = *reinterpret_cast<const uint4 *>(x + nb * ldx + offx + cci[h]);
            }
            const uint16_t *e = reinterpret_cast<const uint16_t *>(&val);
#pragma unroll
            for (int i = 0; i < 8; ++i) XT[ck[h] + i][sv] = e[i];
        }
        if (dact) {
            uint4 val = make_uint4(0u, 0u, 0u, 0u);
            if (vok) val = *reinterpret_cast<const uint4 *>(dy + v * lddy + offdy + co0 + 8 * sc);
            const uint16_t *e = reinterpret_cast<const uint16_t *>(&val);
#pragma unroll
            for (int i = 0; i < 8; ++i) DT[8 * sc + i][sv] = e[i];
        }
        __syncthreads();
        bf16x8 A[NCO];
#pragma unroll
        for (int c = 0; c < NCO; ++c)
            A[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&DT[16 * c + m][8 * q]));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x8 B =
                __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&XT[16 * (2 * wave + t) + m][8 * q]));
#pragma unroll
            for (int c = 0; c < NCO; ++c) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[c], B, acc[c][t], 0, 0, 0);
        }
        if (db && blockIdx.x == 0 && tid < 16 * NCO)
            for (int i = 0; i < kWgStage; ++i) bacc += bf2f(DT[tid][i]);
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < NCO; ++c)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int k = k0 + 16 * (2 * wave + t) + m;
            if (k >= K) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = co0 + 16 * c + 4 * q + i;
                const float v = acc[c][t][i];
                if (v != 0.f) atomicAdd(&dw[(int64_t)co * kpad + k], v);
            }
        }
    if (db && blockIdx.x == 0 && tid < 16 * NCO) atomicAdd(&db[co0 + tid], bacc);
}

// The same for inputs that can be copied into LDS (16-byte aligned, below 2 GiB): a
// workgroup marches through a run of planes of one tile of 8 rows of 32 voxels, for 16
// input channels, 16 NCO output channels and all 27 taps.  Input planes (halo included)
// sit in a four-slot ring and gradient planes in a two-slot one, copied straight from
// global memory in their own layout (voxel by voxel, 16 channels) under the products of
// the plane before; each input plane is copied once per run, not once per tap.  The
// reduction runs over voxels, so both operands are needed voxel-fastest: the LDS
// transpose read (4 voxels of a channel per lane) does that on the way to the
// registers.  A row of 32 voxels is one MFMA's K, in the order 4 (l / 16) + j and 16 +
// 4 (l / 16) + j for j = 0 .. 3, the same for both operands.  The taps are shared out to
// the four waves (7, 7, 7, 6), the last one's spare product sums the gradient itself (db).
// Bound by the copies (35 of 41 us for 16 -> 16 at 96^3 with the products taken out).
// Staging both operands transposed by 2-byte LDS writes, once per group of taps, took
// 388 us there; the 14 layers of a 96^3 step went from 2.19 ms to 0.44.
struct WgradArgs {
    const uint16_t *x, *dy;
    float *dw, *db;
    int ldx, offx, ldd, offd;
    int nz, ny, nx, cin, cout, kpad, zr;
    uint32_t xbytes, xplane, dbytes, dplane;
};
constexpr int kWX = 32, kWY = 8;                 // a tile's voxels in each plane
constexpr int kWBX = kWX + 2, kWBY = kWY + 2;    // with the halo
constexpr int kWPlane = kWBX * kWBY * kCC;       // elements of an input plane in LDS
constexpr int kWD = kWX * kWY * kCC;             // elements of 16 channels of a gradient plane

typedef short s16x4 __attribute__((__vector_size__(4 * sizeof(short))));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 32 voxels x 16 channels at p (voxel-major): this lane's channel l % 16 of its 8 voxels
__device__ __forceinline__ bf16x8 read_transposed(const uint16_t *p, int lane) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * lane));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 16 * kCC + 4 * lane));
    typedef short s16x8 __attribute__((__vector_size__(8 * sizeof(short))));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}

template <int NCO, int WAVE, bool RAGGED>
__device__ __forceinline__ void wgrad_plane(const uint16_t *x0, const uint16_t *x1, const uint16_t *x2, const uint16_t *d,
                                            int rows, int lane, const uint4 &keep, f32x4 (&acc)[7][NCO]) {
    for (int r = 0; r < rows; ++r) {
        bf16x8 A[NCO];
#pragma unroll
        for (int c = 0; c < NCO; ++c) A[c] = read_transposed(d + c * kWD + r * kWX * kCC, lane);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            constexpr int kOne = 0x3f803f80;  // two BF16 ones
            const int tap = 7 * WAVE + i;
            bf16x8 B;
            if (tap < 27) {
                const uint16_t *plane = tap / 9 == 0 ? x0 : tap / 9 == 1 ? x1 : x2;
                B = read_transposed(plane + ((r + (tap / 3) % 3) * kWBX + tap % 3) * kCC, lane);
                if (RAGGED) {  // voxels past the row's end: the gradient there is zero, the input may not be finite
                    uint4 u = __builtin_bit_cast(uint4, B);
                    u = make_uint4(u.x & keep.x, u.y & keep.y, u.z & keep.z, u.w & keep.w);
                    B = __builtin_bit_cast(bf16x8, u);
                }
            } else {
                B = __builtin_bit_cast(bf16x8, make_uint4(kOne, kOne, kOne, kOne));
            }
#pragma unroll
            for (int c = 0; c < NCO; ++c) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[c], B, acc[i][c], 0, 0, 0);
        }
    }
}

template <int NCO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_zm(WgradArgs a) {
    __shared__ __attribute__((aligned(16))) uint16_t s0[kWPlane], s1[kWPlane], s2[kWPlane], s3[kWPlane];
    __shared__ __attribute__((aligned(16))) uint16_t g0[NCO * kWD], g1[NCO * kWD];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups reach the 8 XCDs round robin; each XCD takes a contiguous eighth of the
    // order slice, x tile, y tile, run, so that one L2 serves the slices of a tile
    const int nxt = (a.nx + kWX - 1) / kWX, nyt = (a.ny + kWY - 1) / kWY, nci = a.cin / 16, nsl = nci * (a.cout / (16 * NCO));
    int t = (int)blockIdx.x;
    {
        const int n = (int)gridDim.x, per = n / 8, extra = n % 8, xcd = t % 8;
        t = xcd * per + min(xcd, extra) + t / 8;
    }
    const int slice = t % nsl;
    t /= nsl;
    const int ci0 = slice % nci * 16, co0 = slice / nci * 16 * NCO;
    const int x0 = t % nxt * kWX, y0 = t / nxt % nyt * kWY, z0 = t / (nxt * nyt) * a.zr;
    const int n = min(a.zr, a.nz - z0), rows = min(kWY, a.ny - y0);
    const bool ragged = x0 + kWX > a.nx;
    uint32_t km[4];  // which of this lane's 8 voxels lie inside the row
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int v = x0 + 16 * (k >> 1) + 4 * (lane >> 4) + 2 * (k & 1);
        km[k] = (v < a.nx ? 0xffffu : 0u) | (v + 1 < a.nx ? 0xffff0000u : 0u);
    }
    const uint4 keep = make_uint4(km[0], km[1], km[2], km[3]);
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x), (short)0, (int)a.xbytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rd =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.dy), (short)0, (int)a.dbytes, kRawBuffer);
    // this thread's byte offsets within a plane: input entries (16 bytes, two per voxel)
    // and gradient entries, kNoOff (zeros) outside the grid
    constexpr int kXE = 2 * kWBX * kWBY, kXI = (kXE + 255) / 256;
    uint32_t xo[kXI], go[2];
#pragma unroll
    for (int it = 0; it < kXI; ++it) {
        const int e = tid + 256 * it, v = e >> 1, xx = x0 + v % kWBX - 1, yy = y0 + v / kWBX - 1;
        const bool in = xx >= 0 && xx < a.nx && yy >= 0 && yy < a.ny;
        xo[it] = in ? 2u * (uint32_t)((yy * a.nx + xx) * a.ldx + a.offx + ci0 + 8 * (e & 1)) : kNoOff;
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int e = tid + 256 * it, v = e >> 1, xx = x0 + v % kWX, yy = y0 + v / kWX;
        go[it] = xx < a.nx && yy < a.ny ? 2u * (uint32_t)((yy * a.nx + xx) * a.ldd + a.offd + co0 + 8 * (e & 1)) : kNoOff;
    }
    auto copy_x = [&](int zz, uint16_t *slot) __attribute__((always_inline)) {
        const bool zin = zz >= 0 && zz < a.nz;
        const uint32_t zoff = zin ? (uint32_t)zz * a.xplane : 0u;
#pragma unroll
        for (int it = 0; it < kXI; ++it) {
            const int e0 = 256 * it + 64 * wave;
            if (e0 >= kXE) break;  // wave-uniform
            if (e0 + lane < kXE)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(slot + 8 * e0), 16, zin ? xo[it] : kNoOff, zoff, 0, 0);
        }
    };
    auto copy_g = [&](int zz, uint16_t *slot) __attribute__((always_inline)) {
        const uint32_t zoff = (uint32_t)zz * a.dplane;
#pragma unroll
        for (int c = 0; c < NCO; ++c)
#pragma unroll
            for (int it = 0; it < 2; ++it)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (lds_void *)(slot + c * kWD + 8 * (256 * it + 64 * wave)), 16,
                                                         go[it] == kNoOff ? kNoOff : go[it] + 32u * c, zoff, 0, 0);
    };
    auto ring = [&](int i) -> uint16_t * {
        i &= 3;
        return i == 0 ? s0 : i == 1 ? s1 : i == 2 ? s2 : s3;
    };
    f32x4 acc[7][NCO];
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int c = 0; c < NCO; ++c) acc[i][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    copy_x(z0 - 1, s0);
    copy_x(z0, s1);
    copy_x(z0 + 1, s2);
    copy_g(z0, g0);
    for (int p0 = 0; p0 < n; p0 += 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // plane z0 + p: input slots k, k + 1, k + 2, gradient slot k & 1
            const int p = p0 + k;
            if (p >= n) break;
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // this wave's copies; the barrier waits for the others'
            __syncthreads();
            if (p + 1 < n) {
                copy_x(z0 + p + 2, ring(k + 3));
                copy_g(z0 + p + 1, k & 1 ? g0 : g1);
            }
            const uint16_t *d = k & 1 ? g1 : g0;
            auto plane = [&](auto w) __attribute__((always_inline)) {
                if (ragged)
                    wgrad_plane<NCO, decltype(w)::value, true>(ring(k), ring(k + 1), ring(k + 2), d, rows, lane, keep, acc);
                else
                    wgrad_plane<NCO, decltype(w)::value, false>(ring(k), ring(k + 1), ring(k + 2), d, rows, lane, keep, acc);
            };
            if (wave == 0)
                plane(std::integral_constant<int, 0>{});
            else if (wave == 1)
                plane(std::integral_constant<int, 1>{});
            else if (wave == 2)
                plane(std::integral_constant<int, 2>{});
            else
                plane(std::integral_constant<int, 3>{});
        }
    }
    const int m = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int tap = 7 * wave + i;
#pragma unroll
        for (int c = 0; c < NCO; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int co = co0 + 16 * c + 4 * q + j;
                const float v = acc[i][c][j];
                if (tap < 27) {
                    if (v != 0.f) atomicAdd(&a.dw[(int64_t)co * a.kpad + tap * a.cin + ci0 + m], v);
                } else if (a.db && ci0 == 0 && m == 0) {
                    atomicAdd(&a.db[co], v);
                }
            }
    }
}

// ------------------------------------------------------------------ elementwise layers

__global__ void k_relu_bwd(const uint16_t *y, int ldy, int offy, uint16_t *d, int ldd, int offd, int64_t nvox, int c) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nvox * c) return;
    const int64_t v = i / c;
    const int ch = (int)(i % c);
    if (!(bf2f(y[v * ldy + offy + ch]) > 0.f)) d[v * ldd + offd + ch] = 0;
}

__global__ void k_pool_fwd(const uint16_t *x, int ldx, int offx, uint16_t *y, int ldy, int offy, int nz, int ny,
                           int nx, int c) {
    const int hz = nz / 2, hy = ny / 2, hx = nx / 2;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)hz * hy * hx * c) return;
    const int ch = (int)(i % c);
    const int64_t p = i / c;
    const int X = (int)(p % hx), Y = (int)((p / hx) % hy), Z = (int)(p / ((int64_t)hx * hy));
    float s = 0.f;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx)
                s += bf2f(x[(((int64_t)(2 * Z + dz) * ny + 2 * Y + dy) * nx + 2 * X + dx) * ldx + offx + ch]);
    y[p * ldy + offy + ch] = f2bf(0.125f * s);
}

__global__ void k_pool_bwd(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, int nz, int ny,
                           int nx, int c) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)nz * ny * nx * c) return;
    const int ch = (int)(i % c);
    const int64_t v = i / c;
    const int x = (int)(v % nx), y = (int)((v / nx) % ny), z = (int)(v / ((int64_t)nx * ny));
    const int64_t p = ((int64_t)(z / 2) * (ny / 2) + y / 2) * (nx / 2) + x / 2;
    uint16_t *o = dx + v * ldx + offx + ch;
    *o = f2bf(bf2f(*o) + 0.125f * bf2f(dy[p * ldy + offy + ch]));
}

__global__ void k_up_fwd(const uint16_t *x, int ldx, int offx, uint16_t *y, int ldy, int offy, int nz, int ny, int nx,
                         int c) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)nz * ny * nx * c) return;
    const int ch = (int)(i % c);
    const int64_t v = i / c;
    const int xx = (int)(v % nx), yy = (int)((v / nx) % ny), zz = (int)(v / ((int64_t)nx * ny));
    const int64_t p = ((int64_t)(zz / 2) * (ny / 2) + yy / 2) * (nx / 2) + xx / 2;
    y[v * ldy + offy + ch] = x[p * ldx + offx + ch];
}

__global__ void k_up_bwd(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, int nz, int ny,
                         int nx, int c) {
    const int hz = nz / 2, hy = ny / 2, hx = nx / 2;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)hz * hy * hx * c) return;
    const int ch = (int)(i % c);
    const int64_t p = i / c;
    const int X = (int)(p % hx), Y = (int)((p / hx) % hy), Z = (int)(p / ((int64_t)hx * hy));
    float s = 0.f;
    for (int dz = 0; dz < 2; ++dz)
        for (int dyy = 0; dyy < 2; ++dyy)
            for (int ddx = 0; ddx < 2; ++ddx)
                s += bf2f(dy[(((int64_t)(2 * Z + dz) * ny + 2 * Y + dyy) * nx + 2 * X + ddx) * ldy + offy + ch]);
    dx[p * ldx + offx + ch] = f2bf(s);
}

// The same three layers on runs of 8 channels (16 bytes) per thread, for channel
// counts, row lengths and offsets that are multiples of 8 (every call the network
// makes); 32-bit index arithmetic (grids below 2^32 voxel-runs).
__device__ __forceinline__ void bf8_to_f(uint4 u, float (&f)[8]) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = __uint_as_float(w[k] << 16);
        f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
}

__global__ void k_pool_fwd8(const uint16_t *x, int ldx, int offx, uint16_t *y, int ldy, int offy, uint32_t nz,
                            uint32_t ny, uint32_t nx, uint32_t c8) {
    const uint32_t hy = ny / 2, hx = nx / 2;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if ((uint64_t)i >= (uint64_t)(nz / 2) * hy * hx * c8) return;
    const uint32_t g = i % c8, p = i / c8;
    const uint32_t X = p % hx, Y = (p / hx) % hy, Z = p / (hx * hy);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const uint64_t v = ((uint64_t)(2 * Z + (d >> 2)) * ny + 2 * Y + ((d >> 1) & 1)) * nx + 2 * X + (d & 1);
        float f[8];
        bf8_to_f(*reinterpret_cast<const uint4 *>(x + v * ldx + offx + 8 * g), f);
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] += f[k];
    }
    uint16_t o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = f2bf(0.125f * s[k]);
    *reinterpret_cast<uint4 *>(y + (uint64_t)p * ldy + offy + 8 * g) = *reinterpret_cast<const uint4 *>(o);
}

__global__ void k_up_fwd8(const uint16_t *x, int ldx, int offx, uint16_t *y, int ldy, int offy, uint32_t nz,
                          uint32_t ny, uint32_t nx, uint32_t c8) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if ((uint64_t)i >= (uint64_t)nz * ny * nx * c8) return;
    const uint32_t g = i % c8, v = i / c8;
    const uint32_t xx = v % nx, yy = (v / nx) % ny, zz = v / (nx * ny);
    const uint64_t p = ((uint64_t)(zz / 2) * (ny / 2) + yy / 2) * (nx / 2) + xx / 2;
    *reinterpret_cast<uint4 *>(y + (uint64_t)v * ldy + offy + 8 * g) =
        *reinterpret_cast<const uint4 *>(x + p * ldx + offx + 8 * g);
}

__device__ __forceinline__ uint4 f_to_bf8(const float (&f)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = f2bf2(f[2 * k], f[2 * k + 1]);
    return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ uint4 mask8(uint4 v, uint4 m) {
    return make_uint4(mask_pair(v.x, m.x), mask_pair(v.y, m.y), mask_pair(v.z, m.z), mask_pair(v.w, m.w));
}

// Pooling's and upsampling's adjoints on runs of 8 channels, with an optional ReLU mask m
// on what is written.  Bound by memory: pooling's reads and writes the fine tensor and
// reads the mask.  The one-channel kernels moved 2 bytes per thread and the mask was a
// pass of its own (13 us): 23.5 + 13 -> 15.8 us and 9.4 + 13 -> 9.3 us, means of the three
// calls of a 96^3 step.
__global__ void k_pool_bwd8(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m,
                            int ldm, int offm, uint32_t nz, uint32_t ny, uint32_t nx, uint32_t c8) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if ((uint64_t)i >= (uint64_t)nz * ny * nx * c8) return;
    const uint32_t g = i % c8, v = i / c8;
    const uint32_t xx = v % nx, yy = (v / nx) % ny, zz = v / (nx * ny);
    const uint64_t p = ((uint64_t)(zz / 2) * (ny / 2) + yy / 2) * (nx / 2) + xx / 2;
    uint4 *o = reinterpret_cast<uint4 *>(dx + (uint64_t)v * ldx + offx + 8 * g);
    float a[8], b[8];
    bf8_to_f(*o, a);
    bf8_to_f(*reinterpret_cast<const uint4 *>(dy + p * ldy + offy + 8 * g), b);
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] += 0.125f * b[k];
    uint4 r = f_to_bf8(a);
    if (m) r = mask8(r, *reinterpret_cast<const uint4 *>(m + (uint64_t)v * ldm + offm + 8 * g));
    *o = r;
}

__global__ void k_up_bwd8(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m,
                          int ldm, int offm, uint32_t nz, uint32_t ny, uint32_t nx, uint32_t c8) {
    const uint32_t hy = ny / 2, hx = nx / 2;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if ((uint64_t)i >= (uint64_t)(nz / 2) * hy * hx * c8) return;
    const uint32_t g = i % c8, p = i / c8;
    const uint32_t X = p % hx, Y = (p / hx) % hy, Z = p / (hx * hy);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const uint64_t v = ((uint64_t)(2 * Z + (d >> 2)) * ny + 2 * Y + ((d >> 1) & 1)) * nx + 2 * X + (d & 1);
        float f[8];
        bf8_to_f(*reinterpret_cast<const uint4 *>(dy + v * ldy + offy + 8 * g), f);
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] += f[k];
    }
    uint4 r = f_to_bf8(s);
    if (m) r = mask8(r, *reinterpret_cast<const uint4 *>(m + (uint64_t)p * ldm + offm + 8 * g));
    *reinterpret_cast<uint4 *>(dx + (uint64_t)p * ldx + offx + 8 * g) = r;
}

__global__ void k_head_fwd8(const uint16_t *x, int ldx, const float *w, const float *b, const float *base, float *out,
                            int64_t nvox, int c8) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    float s = b[0] + (base ? base[v] : 0.f);
    for (int g = 0; g < c8; ++g) {
        float f[8];
        bf8_to_f(*reinterpret_cast<const uint4 *>(x + v * ldx + 8 * g), f);
#pragma unroll
        for (int k = 0; k < 8; ++k) s = fmaf(w[8 * g + k], f[k], s);
    }
    out[v] = s;
}

__global__ void k_head_fwd(const uint16_t *x, int ldx, const float *w, const float *b, const float *base, float *out,
                           int64_t nvox, int c) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    float s = b[0] + (base ? base[v] : 0.f);
    for (int ch = 0; ch < c; ++ch) s = fmaf(w[ch], bf2f(x[v * ldx + ch]), s);
    out[v] = s;
}

__device__ __forceinline__ float block_sum(float v, float *red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
    __syncthreads();
    return t;
}

constexpr int kHeadMaxC = 32;  // channels of the 1x1x1 head (the first U-Net level)

// Grid-stride over the voxels with per-thread channel partials in registers, so
// each workgroup reduces and adds to dw / db once (not once per 256 voxels).
__global__ __launch_bounds__(256) void k_head_bwd(const uint16_t *x, int ldx, const float *w, const float *dout,
                                                  uint16_t *dx, float *dw, float *db, int64_t nvox, int c) {
    __shared__ float red[4];
    float part[kHeadMaxC];
#pragma unroll
    for (int ch = 0; ch < kHeadMaxC; ++ch) part[ch] = 0.f;
    float gsum = 0.f;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (int64_t)gridDim.x * blockDim.x) {
        const float g = dout[v];
        gsum += g;
#pragma unroll
        for (int ch = 0; ch < kHeadMaxC; ++ch) {
            if (ch < c) {
                part[ch] += g * bf2f(x[v * ldx + ch]);
                dx[v * c + ch] = f2bf(g * w[ch]);
            }
        }
    }
#pragma unroll
    for (int ch = 0; ch < kHeadMaxC; ++ch) {
        if (ch < c) {
            const float s = block_sum(part[ch], red);
            if (threadIdx.x == 0) atomicAdd(&dw[ch], s);
        }
    }
    const float s = block_sum(gsum, red);
    if (threadIdx.x == 0) atomicAdd(db, s);
}

// The same for 16 channels in 16-byte pieces, one reduction per workgroup for all 17 sums
// (252 -> 23 us at 96^3: the general form reads and writes 2 bytes at a time and reduces
// channel after channel).  RELU: dx is zeroed where x is not positive.
template <bool RELU>
__global__ __launch_bounds__(256) void k_head_bwd16(const uint16_t *x, int ldx, const float *w, const float *dout,
                                                    uint16_t *dx, float *dw, float *db, int64_t nvox) {
    __shared__ float red[4][17];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float wr[16], part[17];
#pragma unroll
    for (int c = 0; c < 16; ++c) wr[c] = w[c];
#pragma unroll
    for (int c = 0; c < 17; ++c) part[c] = 0.f;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (int64_t)gridDim.x * 256) {
        const float g = dout[v];
        part[16] += g;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint4 u = *reinterpret_cast<const uint4 *>(x + v * ldx + 8 * h);
            float f[8], o[8];
            bf8_to_f(u, f);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                part[8 * h + k] += g * f[k];
                o[k] = g * wr[8 * h + k];
            }
            uint4 r = f_to_bf8(o);
            if (RELU) r = mask8(r, u);
            *reinterpret_cast<uint4 *>(dx + v * 16 + 8 * h) = r;
        }
    }
#pragma unroll
    for (int c = 0; c < 17; ++c) {
        float s = part[c];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) red[wave][c] = s;
    }
    __syncthreads();
    if (threadIdx.x < 17) {
        const int c = threadIdx.x;
        atomicAdd(c < 16 ? &dw[c] : db, ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c]);
    }
}

// Bound by memory (17 to 21 bytes per voxel) once few workgroups add to the one loss: with
// a workgroup per 256 voxels their atomics stood in line, 47 us at 96^3; 512 take 16.
__global__ __launch_bounds__(256) void k_mse(const float *pred, const float *target, const uint8_t *mask,
                                             const float *weight, float *dout, float *loss, int64_t nvox,
                                             float inv_count) {
    __shared__ float red[4];
    float e = 0.f;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (int64_t)gridDim.x * 256) {
        const float d = mask[v] ? pred[v] - target[v] : 0.f;
        const float wd = (weight ? weight[v] : 1.f) * d;
        dout[v] = 2.f * wd * inv_count;
        e += wd * d * inv_count;
    }
    const float s = block_sum(e, red);
    if (threadIdx.x == 0) atomicAdd(loss, s);
}

__global__ void k_adam(float *p, float *m, float *v, const float *g, uint16_t *pb, int64_t n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = f2bf(pi);
}

__global__ void k_to_bf16(const float *s, uint16_t *d, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = f2bf(s[i]);
}

__global__ void k_zero(uint32_t *d, int64_t nwords) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nwords) d[i] = 0u;
}

// Bound by the 32 bytes written per voxel: 79 -> 63 us at 192^3 with every store a
// run of whole lines (two stores of alternate 16-byte pieces before).
__global__ void k_features(const uint8_t *active, const uint8_t *ncat, const float *omega, float tau_ref,
                           uint16_t *feat, float *weight, float weight_power, float weight_cap, int nz, int ny,
                           int nx) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)nz * ny * nx;
    const int x = (v >> 32) == 0 ? (int)((uint32_t)v % (uint32_t)nx) : (int)(v % nx);
    // distances to the inlet and outlet faces in voxels, not fractions of the length,
    // so that a network trained on short domains transfers to longer ones
    const float xi = (float)x, xo = (float)(nx - 1 - x);
    float f[6] = {0.f, 0.f, 0.f, expf(-xi / 24.f), expf(-xi / 96.f), expf(-xo / 24.f)};
    float w = 0.f;
    if (v < n && active[v]) {
        f[0] = 1.f;
        const float tau = 1.f / omega[v];
        const float drel = fmaxf((tau - 0.5f) / (tau_ref - 0.5f), 1e-9f);
        f[1] = log10f(drel) / 3.f;
        f[2] = ncat ? (float)ncat[v] / 6.f : 0.f;
        if (weight) w = fminf(weight_cap, powf(1.f / drel, weight_power));
    }
    if ((reinterpret_cast<uintptr_t>(feat) & 15) == 0) {
        // whole lines per store: the wave's 128 pieces of 16 bytes in order, the even ones
        // the channels of a voxel computed by lane piece / 2
        const int lane = threadIdx.x & 63;
        const uint32_t a = f2bf2(f[0], f[1]), b = f2bf2(f[2], f[3]), c = f2bf2(f[4], f[5]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int from = 32 * h + lane / 2;
            const uint32_t ha = __shfl(a, from, 64), hb = __shfl(b, from, 64), hc = __shfl(c, from, 64);
            const bool low = lane % 2 == 0;
            if (v - lane + from < n)
                reinterpret_cast<uint4 *>(feat)[2 * (v - lane) + 64 * h + lane] =
                    make_uint4(low ? ha : 0u, low ? hb : 0u, low ? hc : 0u, 0u);
        }
    }
    if (v >= n) return;
    if (reinterpret_cast<uintptr_t>(feat) & 15) {
        uint16_t *o = feat + v * 16;
        for (int c = 0; c < 16; ++c) o[c] = c < 6 ? f2bf(f[c]) : (uint16_t)0;
    }
    if (weight) weight[v] = w;
}

// y = ln(max(c, 0) + eps), or its inverse c = min(cmax, max(0, exp(y) - eps))
__global__ void k_log_map(const float *src, float *dst, int64_t n, float eps, int inverse, float cmax) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = src[i];
    dst[i] = inverse ? fminf(cmax, fmaxf(0.f, expf(v) - eps)) : logf(fmaxf(v, 0.f) + eps);
}

// start field of the solver from the network's log-space output: the prediction
// where the pore depth is at most depth_max, zero (the cold start) elsewhere
__global__ void k_start_field(const float *y, const uint8_t *depth, int depth_max, float eps, float cmax, float *c,
                              int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    c[i] = (int)depth[i] <= depth_max ? fminf(cmax, fmaxf(0.f, expf(y[i]) - eps)) : 0.f;
}

// corrector of the effective-diffusivity problem: the field minus the linear profile
// between the two Dirichlet faces, in units of the mean gradient (or its inverse)
__global__ void k_corrector(const float *src, float *dst, int64_t n, int nx, float c_in, float c_out, int inverse,
                            float cmax) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = (float)(i % nx);
    const float lin = c_in + (c_out - c_in) * (x + 0.5f) / (float)nx;
    const float scale = (float)nx / (c_in - c_out);
    dst[i] = inverse ? fminf(cmax, fmaxf(0.f, lin + src[i] / scale)) : (src[i] - lin) * scale;
}

// D = A B (16x32 by 32x16) through the conv kernel's fragment mapping
__global__ void k_mfma_selftest(const float *a, const float *b, float *d) {
    const int lane = threadIdx.x;
    const int m = lane & 15, kb = lane >> 4;
    uint16_t av[8], bv[8];
    for (int j = 0; j < 8; ++j) {
        av[j] = f2bf(a[m * 32 + 8 * kb + j]);
        bv[j] = f2bf(b[(8 * kb + j) * 16 + m]);
    }
    const bf16x8 A = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(av));
    const bf16x8 B = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(bv));
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B, acc, 0, 0, 0);
    for (int i = 0; i < 4; ++i) d[(4 * kb + i) * 16 + m] = acc[i];
}

dim3 grid1(int64_t n, int bs = 256) { return dim3((unsigned)((n + bs - 1) / bs)); }

bool ch_ok(int ld, int off, int c) { return ld > 0 && off >= 0 && c > 0 && off + c <= ld; }

// channel count, row lengths and offsets all in runs of 8 (16-byte loads and stores)
bool runs8(int c, int ld1, int off1, int ld2, int off2) { return ((c | ld1 | off1 | ld2 | off2) & 7) == 0; }

}  // namespace

static bool aligned16(const void *a, const void *b, const void *c) {
    return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c)) & 15) == 0;
}

template <bool RELU>
static int head_bwd(const uint16_t *x, int32_t ldx, const float *w, const float *dout, uint16_t *dx, float *dw, float *db,
                    int64_t nvox, int32_t c, void *stream) {
    if (!x || !w || !dout || !dx || !dw || !db || nvox <= 0 || c <= 0 || c > kHeadMaxC || ldx < c) return -1;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (c == 16 && ldx % 8 == 0 && aligned16(x, dx, nullptr)) {
        const dim3 g((unsigned)std::min<int64_t>((nvox + 255) / 256, 512));
        hipLaunchKernelGGL(k_head_bwd16<RELU>, g, dim3(256), 0, st, x, ldx, w, dout, dx, dw, db, nvox);
        return status(hipGetLastError());
    }
    if (RELU) return -1;
    const dim3 g((unsigned)std::min<int64_t>((nvox + 255) / 256, 1024));
    hipLaunchKernelGGL(k_head_bwd, g, dim3(256), 0, st, x, ldx, w, dout, dx, dw, db, nvox, c);
    return status(hipGetLastError());
}

// Planes per run of the marching form: each run costs its planes, two more to fill and about
// three of start, in rounds of kConvSlots workgroups.
static int march_planes(int64_t tiles, int nz) {
    int best = nz;
    int64_t cost = INT64_MAX;
    for (int runs = 1; runs <= std::max(1, nz / 4); ++runs) {
        const int zr = (nz + runs - 1) / runs;
        const int64_t c = (tiles * ((nz + zr - 1) / zr) + kConvSlots - 1) / kConvSlots * (zr + 5);
        if (c < cost) cost = c, best = zr;
    }
    return best;
}

// Planes of a slab: the busiest CU's workgroups times their planes, weighed by what a plane
// costs in a slab of that many (halo planes and weights are shared by its planes: measured
// over 12^3 .. 192^3; rows of kpad make the weights dearer), and by 1.25 where a CU has one
// workgroup, whose copies nothing covers.  At 64 -> 64 channels, packed: 12^3 best at 1
// (7.9 us; 11.7 at 2), 24^3 at 1 (10 us; 16 at 4), 48^3 at 4 (26 us; 32 at 1).
static int slab_planes(int64_t tiles, int nz, int s, bool packed) {
    static const double kCost[3][4] = {{1.17, 1.12, 1.0, 1.0}, {1.2, 1.0, 1.02, 1.1}, {2.2, 1.5, 1.15, 1.0}};
    const double *w = kCost[!packed ? 2 : s == 1 ? 1 : 0];
    int best = 1;
    double cost = 0.;
    for (int zc = 1; zc <= 4; ++zc) {
        const int64_t n = (tiles * ((nz + zc - 1) / zc) + kConvSlots / 2 - 1) / (kConvSlots / 2);
        const double c = (double)n * zc * w[zc - 1] * (n == 1 ? 1.25 : 1.);
        if (zc == 1 || c < cost) cost = c, best = zc;
    }
    return best;
}

template <int S, int XG>
static void launch_slab(int zc, dim3 g, hipStream_t st, const ConvArgs &a) {
    const dim3 blk(256);
    if (zc == 1) hipLaunchKernelGGL((k_conv_slab<S, 1, XG>), g, blk, 0, st, a);
    else if (zc == 2) hipLaunchKernelGGL((k_conv_slab<S, 2, XG>), g, blk, 0, st, a);
    else if (zc == 3) hipLaunchKernelGGL((k_conv_slab<S, 3, XG>), g, blk, 0, st, a);
    else hipLaunchKernelGGL((k_conv_slab<S, 4, XG>), g, blk, 0, st, a);
}

// Workgroups in a plane for s channel slices each; flat: with their waves side by side in x
// (tiles of 4 rows of 64 / s voxels) instead of on top of each other (16 / s rows of 16).
static int64_t tiles_xy(int nx, int ny, int s, bool flat) {
    const int tx = flat ? 64 / s : 16, ty = flat ? 4 : 16 / s;
    return (int64_t)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty);
}

template <int XG>
static void launch_march(dim3 g, hipStream_t st, const ConvArgs &a, int s, int zr) {
    const dim3 blk(256);
    if (a.hout) hipLaunchKernelGGL((k_conv_march<1, true, false, XG>), g, blk, 0, st, a, zr);
    else if (a.m) hipLaunchKernelGGL((k_conv_march<1, false, true, XG>), g, blk, 0, st, a, zr);
    else if (s == 1) hipLaunchKernelGGL((k_conv_march<1, false, false, XG>), g, blk, 0, st, a, zr);
    else hipLaunchKernelGGL((k_conv_march<2, false, false, XG == 4 ? 2 : 1>), g, blk, 0, st, a, zr);
}

extern "C" {

int32_t unet_kpad(int32_t cin) { return kpad_of(cin); }

// both convolution entry points: a.x2 is a.x and a.cin1 a.cin for a single input
static int launch_conv(ConvArgs a, int64_t nx2, int64_t ny2, int64_t nz2, void *stream) {
    const int nx = a.nx, ny = a.ny, nz = a.nz, cin = a.cin, cout = a.cout;
    if (!a.x || !a.x2 || !a.w || (!a.y && !a.hout) || nz <= 0 || ny <= 0 || nx <= 0 || cin % 16 || a.cin1 % 16 ||
        a.cin1 <= 0 || a.cin1 > cin || !ch_ok(a.ldx, a.offx, a.cin1) || (a.cin1 < cin && !ch_ok(a.ldx2, a.offx2, cin - a.cin1)) ||
        !ch_ok(a.ldy, a.offy, cout) || (a.ldx % 8) || (a.offx % 8) || (a.ldx2 % 8) || (a.offx2 % 8) || (a.ldy % 8) ||
        (a.offy % 8))
        return -1;
    if (cout % 16 || nz > 65535) return -1;
    if ((reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.x2) | reinterpret_cast<uintptr_t>(a.w) |
         reinterpret_cast<uintptr_t>(a.y) | reinterpret_cast<uintptr_t>(a.y32)) & 15)
        return -1;  // 16-byte vector loads and stores
    const int tiles = cout / 16;
    const int64_t plane_bytes = 2 * (int64_t)ny * nx * a.ldx, xbytes = plane_bytes * nz;
    const int64_t plane2_bytes = 2 * ny2 * nx2 * a.ldx2, x2bytes = plane2_bytes * nz2;
    const int64_t wbytes = a.packed ? 2 * packed_len(cin, cout) : 2 * (int64_t)cout * kpad_of(cin);
    if (xbytes > kMaxX || x2bytes > kMaxX || wbytes > kMaxX) return -1;
    a.kpad = kpad_of(cin);
    a.xbytes = (uint32_t)xbytes;
    a.plane_bytes = (uint32_t)plane_bytes;
    a.x2bytes = (uint32_t)x2bytes;
    a.plane2_bytes = (uint32_t)plane2_bytes;
    a.wbytes = (uint32_t)wbytes;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 blk(256);
    // slices per workgroup: as many as share the copies evenly
    int s = tiles % 4 == 0 ? 4 : tiles % 2 == 0 ? 2 : 1;
    // Few rows leave the upper waves of a tile without any: tiles lie flat where that saves a
    // quarter of them.  us upright / flat at 512 planes of rows of 512: 16 -> 16 channels, 4 rows
    // 49 / 22.5, 8 51 / 34.5, 12 55 / 47.5, 16 58 / 60, 20 107 / 80, 28 (an eighth saved) 120 / 112;
    // 48 -> 16 148 / 60, 154 / 112, 188 / 189, 232 / 258, 414 / 328, 433 / 453.
    auto flat = [&](int sl) { return sl < 4 && 3 * tiles_xy(nx, ny, sl, false) >= 4 * tiles_xy(nx, ny, sl, true); };
    if (tiles_xy(nx, ny, s, flat(s)) > 0x7fffffff) return -1;
    (void)hipGetLastError();
    // One stage: march where a chip full of workgroups (two per CU) has at least five planes
    // each.  Below that the run's first two planes cost more than they save (16 -> 32 at 48^3,
    // 1.7 planes: 10.0 us against 7.5 in slabs; 16 -> 16 at 96^3, 6.8: 20.4 against 22.9), as on
    // grids of fewer planes than that (512 x 512 rows, 16 -> 48: one plane 42 against 34, four 72.3
    // against 70.1, six 96 against 116; 16 -> 16 four 27 against 24.4, six 33 against 37).
    const int sm = s > 1 && !a.m && !a.hout ? 2 : 1;
    const int64_t tm = tiles_xy(nx, ny, sm, flat(sm));
    if (cin == kCC && a.cin1 == cin && (a.hout || (nz >= 5 && tm * (tiles / sm) * nz >= 5 * kConvSlots))) {
        const int zr = march_planes(tm * (tiles / sm), nz);
        const dim3 g((unsigned)tm, (unsigned)((nz + zr - 1) / zr), (unsigned)(tiles / sm));
        if (flat(sm)) launch_march<4>(g, st, a, sm, zr);
        else launch_march<1>(g, st, a, sm, zr);
        return status(hipGetLastError());
    }
    const bool f = flat(s);
    const int64_t txy = tiles_xy(nx, ny, s, f), t = txy * (tiles / s);
    // 16 output channels and eight rounds of workgroups: see k_conv_ring
    const bool ring = s == 1 && !f && t * ((nz + 3) / 4) >= 8 * kConvSlots;
    const int zc = ring ? 4 : slab_planes(t, nz, s, a.packed);
    const dim3 g((unsigned)txy, (unsigned)((nz + zc - 1) / zc), (unsigned)(tiles / s));
    if (ring) hipLaunchKernelGGL((k_conv_ring<1, 4>), g, blk, 0, st, a);
    else if (s == 4) launch_slab<4, 1>(zc, g, st, a);
    else if (s == 2 && f) launch_slab<2, 2>(zc, g, st, a);
    else if (s == 2) launch_slab<2, 1>(zc, g, st, a);
    else if (f) launch_slab<1, 4>(zc, g, st, a);
    else launch_slab<1, 1>(zc, g, st, a);
    return status(hipGetLastError());
}

int unet_conv3d_fwd(const uint16_t *x, int32_t ldx, int32_t offx, const uint16_t *w, const float *b, uint16_t *y,
                    int32_t ldy, int32_t offy, float *y32, int32_t nz, int32_t ny, int32_t nx, int32_t cin,
                    int32_t cout, int32_t relu, void *stream) {
    ConvArgs a{x, w, b, y, y32, ldx, offx, ldy, offy, nz, ny, nx, cin, cout, 0, relu, 0, 0, 0,
               x, ldx, offx, cin, 0, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, 0};
    return launch_conv(a, nx, ny, nz, stream);
}

int unet_conv3d_fwd_head(const uint16_t *x, int32_t ldx, int32_t offx, const uint16_t *w, const float *b,
                         const float *hw, const float *hb, const float *base, float *out, int32_t nz, int32_t ny,
                         int32_t nx, void *stream) {
    if (!hw || !hb || !out) return -1;
    // 16 -> 16 channels with ReLU, then the head; the BF16 outputs are not stored
    ConvArgs a{x, w, b, nullptr, nullptr, ldx, offx, 16, 0, nz, ny, nx, 16, 16, 0, 1, 0, 0, 0,
               x, ldx, offx, 16, 0, 0, 0, hw, hb, base, out, nullptr, 0, 0, 0};
    return launch_conv(a, nx, ny, nz, stream);
}

int unet_conv3d_fwd_cat(const uint16_t *x, int32_t ldx, int32_t offx, int32_t cin1, const uint16_t *x2, int32_t ldx2,
                        int32_t offx2, const uint16_t *w, const float *b, uint16_t *y, int32_t ldy, int32_t offy,
                        float *y32, int32_t nz, int32_t ny, int32_t nx, int32_t cin, int32_t cout, int32_t relu,
                        void *stream) {
    if (nz % 2 || ny % 2 || nx % 2) return -1;  // x2 holds the half-resolution grid
    ConvArgs a{x, w, b, y, y32, ldx, offx, ldy, offy, nz, ny, nx, cin, cout, 0, relu, 0, 0, 0,
               x2, ldx2, offx2, cin1, 1, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, 0};
    if (cin1 >= cin) return -1;
    return launch_conv(a, nx / 2, ny / 2, nz / 2, stream);
}

int unet_conv3d_wtrans(const uint16_t *w, uint16_t *wt, int32_t cin, int32_t cout, void *stream) {
    if (!w || !wt || cin <= 0 || cout <= 0) return -1;
    const int64_t n = (int64_t)cin * kpad_of(cout);
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_wtrans, grid1(n), dim3(256), 0, static_cast<hipStream_t>(stream), w, wt, cin, cout,
                       kpad_of(cin), kpad_of(cout));
    return status(hipGetLastError());
}

int unet_conv3d_wgrad(const uint16_t *x, int32_t ldx, int32_t offx, const uint16_t *dy, int32_t lddy, int32_t offdy,
                      int32_t nz, int32_t ny, int32_t nx, int32_t cin, int32_t cout, float *dw, float *db,
                      void *stream) {
    if (!x || !dy || !dw || nz <= 0 || ny <= 0 || nx <= 0 || !ch_ok(ldx, offx, cin) || !ch_ok(lddy, offdy, cout))
        return -1;
    if (cin % 16 || cout % 16 || ldx % 8 || offx % 8 || lddy % 8 || offdy % 8) return -1;
    const int64_t nvox = (int64_t)nz * ny * nx;
    const int64_t xplane = 2 * (int64_t)ny * nx * ldx, dplane = 2 * (int64_t)ny * nx * lddy;
    // The marching form, in runs of planes: about one workgroup per CU, up to two where the runs
    // stay 24 planes long (a run copies two planes beyond its own and adds its sums
    // atomically).  The 14 layers of a 96^3 step: 514 / 444 / 477 / 515 / 675 us with 128 / 256 /
    // 384 / 512 / 768 workgroups each; the 48 -> 16 layer alone 115 / 78 / 56 / 74 / 61.
    const int two = cout % 32 == 0 ? 2 : 1;
    const int64_t tiles = (int64_t)((nx + kWX - 1) / kWX) * ((ny + kWY - 1) / kWY) * (cin / 16) * (cout / (16 * two));
    const int64_t runs = std::max(std::max<int64_t>(1, 256 / tiles), std::min<int64_t>(512 / tiles, nz / 24));
    int64_t zr = (nz + runs - 1) / runs;
    // Tiny grids of one tile keep to two runs, whose two sums have no order; the general form
    // has as many there.
    const bool few = nvox <= 1024 && nx <= kWX && ny <= kWY;
    if (few) zr = std::max<int64_t>(zr, (nz + 1) / 2);
    // Not where long runs go through tiles that are mostly empty (us there / in the general
    // form, 512 x 512 rows: 1 voxel 138 / 83 (16 -> 16 channels), 750 / 180 (32 -> 64); 2: 138 / 160,
    // 750 / 361; 3: 139 / 230, 751 / 568; 4: 139 / 317, 749 / 706; 6: 139 / 455, 750 / 1133; runs of
    // 1 to 5 planes of 28 x 106 rows of 1 16 / 23, 13 x 73 of 4 22 / 28), nor where the two
    // runs of a tiny grid are long (planes of 8 x 8: 15 of them 15.5 / 23, 22 / 26; 20 of 7 x 7 17 /
    // 23, 24 / 26; 60 of 4 x 4 30 / 23, 42 / 26; 1000 of one voxel 227 / 22).
    // Nor long runs, or very many of them, of a few voxels a plane (2000 of 1 x 8 32 -> 64: 32 /
    // 25; 500 of 2 x 6 15 / 24; 2000 of 3 x 5 16 -> 16 in 250 runs: 29 / 24).
    const bool thin = nx < (two == 2 ? 5 : 3), sliver = (int64_t)nx * ny <= 16;
    const int64_t blocks = tiles * ((nz + zr - 1) / zr);
    if (((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy)) & 15) == 0 && xplane * nz <= kMaxX &&
        dplane * nz <= kMaxX && blocks <= 0x7fffffff && (!thin || zr <= 6) && (!sliver || zr <= (two == 2 ? 16 : 6)) &&
        (!few || zr <= 10)) {
        const WgradArgs a{x, dy, dw, db, ldx, offx, lddy, offdy, nz, ny, nx, cin, cout, kpad_of(cin), (int)zr,
                          (uint32_t)(xplane * nz), (uint32_t)xplane, (uint32_t)(dplane * nz), (uint32_t)dplane};
        (void)hipGetLastError();
        if (two == 2)
            hipLaunchKernelGGL(k_wgrad_zm<2>, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream), a);
        else
            hipLaunchKernelGGL(k_wgrad_zm<1>, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream), a);
        return status(hipGetLastError());
    }
    const int nco = cout % 64 == 0 ? 4 : (cout % 32 == 0 ? 2 : 1);
    // enough workgroups to fill the device: the voxel range per workgroup shrinks
    // for layers with few (k, channel) tiles
    const int64_t slices = (int64_t)((27 * cin + kWgK - 1) / kWgK) * (cout / (16 * nco));
    int64_t vper = 4096;
    while (vper > 512 && slices * ((nvox + vper - 1) / vper) < 2048) vper >>= 1;
    const dim3 g((unsigned)((27 * cin + kWgK - 1) / kWgK), (unsigned)((nvox + vper - 1) / vper),
                 (unsigned)(cout / (16 * nco)));
    (void)hipGetLastError();
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const int kp = kpad_of(cin);
    switch (nco) {
        case 4: hipLaunchKernelGGL(k_wgrad<4>, g, dim3(256), 0, st, x, ldx, offx, dy, lddy, offdy, nz, ny, nx, cin, cout, kp, vper, dw, db); break;
        case 2: hipLaunchKernelGGL(k_wgrad<2>, g, dim3(256), 0, st, x, ldx, offx, dy, lddy, offdy, nz, ny, nx, cin, cout, kp, vper, dw, db); break;
        default: hipLaunchKernelGGL(k_wgrad<1>, g, dim3(256), 0, st, x, ldx, offx, dy, lddy, offdy, nz, ny, nx, cin, cout, kp, vper, dw, db); break;
    }
    return status(hipGetLastError());
}

int unet_relu_bwd(const uint16_t *y, int32_t ldy, int32_t offy, uint16_t *dy, int32_t ldd, int32_t offd, int64_t nvox,
                  int32_t c, void *stream) {
    if (!y || !dy || !ch_ok(ldy, offy, c) || !ch_ok(ldd, offd, c) || nvox <= 0) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_relu_bwd, grid1(nvox * c), dim3(256), 0, static_cast<hipStream_t>(stream), y, ldy, offy, dy,
                       ldd, offd, nvox, c);
    return status(hipGetLastError());
}

int unet_pool_fwd(const uint16_t *x, int32_t ldx, int32_t offx, uint16_t *y, int32_t ldy, int32_t offy, int32_t nz,
                  int32_t ny, int32_t nx, int32_t c, void *stream) {
    if (!x || !y || (nz | ny | nx) & 1 || nz <= 0 || !ch_ok(ldx, offx, c) || !ch_ok(ldy, offy, c)) return -1;
    (void)hipGetLastError();
    if (runs8(c, ldx, offx, ldy, offy) && (int64_t)nz * ny * nx / 8 * (c / 8) < ((int64_t)1 << 32))
        hipLaunchKernelGGL(k_pool_fwd8, grid1((int64_t)nz * ny * nx / 8 * (c / 8)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), x, ldx, offx, y, ldy, offy, (uint32_t)nz, (uint32_t)ny,
                           (uint32_t)nx, (uint32_t)(c / 8));
    else
        hipLaunchKernelGGL(k_pool_fwd, grid1((int64_t)nz * ny * nx / 8 * c), dim3(256), 0,
                           static_cast<hipStream_t>(stream), x, ldx, offx, y, ldy, offy, nz, ny, nx, c);
    return status(hipGetLastError());
}

int unet_pool_bwd(const uint16_t *dy, int32_t ldy, int32_t offy, uint16_t *dx, int32_t ldx, int32_t offx, int32_t nz,
                  int32_t ny, int32_t nx, int32_t c, void *stream) {
    return unet::pool_bwd_relu(dy, ldy, offy, dx, ldx, offx, nullptr, 0, 0, nz, ny, nx, c, stream);
}

int unet_up_fwd(const uint16_t *x, int32_t ldx, int32_t offx, uint16_t *y, int32_t ldy, int32_t offy, int32_t nz,
                int32_t ny, int32_t nx, int32_t c, void *stream) {
    if (!x || !y || (nz | ny | nx) & 1 || nz <= 0 || !ch_ok(ldx, offx, c) || !ch_ok(ldy, offy, c)) return -1;
    (void)hipGetLastError();
    if (runs8(c, ldx, offx, ldy, offy) && (int64_t)nz * ny * nx * (c / 8) < ((int64_t)1 << 32))
        hipLaunchKernelGGL(k_up_fwd8, grid1((int64_t)nz * ny * nx * (c / 8)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), x, ldx, offx, y, ldy, offy, (uint32_t)nz, (uint32_t)ny,
                           (uint32_t)nx, (uint32_t)(c / 8));
    else
        hipLaunchKernelGGL(k_up_fwd, grid1((int64_t)nz * ny * nx * c), dim3(256), 0, static_cast<hipStream_t>(stream),
                           x, ldx, offx, y, ldy, offy, nz, ny, nx, c);
    return status(hipGetLastError());
}

int unet_up_bwd(const uint16_t *dy, int32_t ldy, int32_t offy, uint16_t *dx, int32_t ldx, int32_t offx, int32_t nz,
                int32_t ny, int32_t nx, int32_t c, void *stream) {
    return unet::up_bwd_relu(dy, ldy, offy, dx, ldx, offx, nullptr, 0, 0, nz, ny, nx, c, stream);
}

int unet_head_fwd(const uint16_t *x, int32_t ldx, const float *w, const float *b, const float *base, float *out,
                  int64_t nvox, int32_t c, void *stream) {
    if (!x || !w || !b || !out || nvox <= 0 || c <= 0 || ldx < c) return -1;
    (void)hipGetLastError();
    if (runs8(c, ldx, 0, 8, 0))
        hipLaunchKernelGGL(k_head_fwd8, grid1(nvox), dim3(256), 0, static_cast<hipStream_t>(stream), x, ldx, w, b,
                           base, out, nvox, c / 8);
    else
        hipLaunchKernelGGL(k_head_fwd, grid1(nvox), dim3(256), 0, static_cast<hipStream_t>(stream), x, ldx, w, b, base,
                           out, nvox, c);
    return status(hipGetLastError());
}

int unet_head_bwd(const uint16_t *x, int32_t ldx, const float *w, const float *dout, uint16_t *dx, float *dw,
                  float *db, int64_t nvox, int32_t c, void *stream) {
    return head_bwd<false>(x, ldx, w, dout, dx, dw, db, nvox, c, stream);
}

int unet_mse(const float *pred, const float *target, const uint8_t *mask, const float *weight, float *dout,
             float *loss, int64_t nvox, int64_t count, void *stream) {
    if (!pred || !target || !mask || !dout || !loss || nvox <= 0 || count <= 0) return -1;
    (void)hipGetLastError();
    const dim3 g((unsigned)std::min<int64_t>((nvox + 255) / 256, 512));
    hipLaunchKernelGGL(k_mse, g, dim3(256), 0, static_cast<hipStream_t>(stream), pred, target, mask, weight,
                       dout, loss, nvox, 1.0f / (float)count);
    return status(hipGetLastError());
}

int unet_adam(float *p, float *m, float *v, const float *g, uint16_t *pb, int64_t n, float lr, float beta1,
              float beta2, float eps, int32_t t, void *stream) {
    if (!p || !m || !v || !g || n <= 0 || t < 1) return -1;
    const float c1 = 1.f / (1.f - powf(beta1, (float)t)), c2 = 1.f / (1.f - powf(beta2, (float)t));
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_adam, grid1(n), dim3(256), 0, static_cast<hipStream_t>(stream), p, m, v, g, pb, n, lr, beta1,
                       beta2, eps, c1, c2);
    return status(hipGetLastError());
}

int unet_to_bf16(const float *src, uint16_t *dst, int64_t n, void *stream) {
    if (!src || !dst || n <= 0) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_to_bf16, grid1(n), dim3(256), 0, static_cast<hipStream_t>(stream), src, dst, n);
    return status(hipGetLastError());
}

int unet_zero(void *dst, int64_t bytes, void *stream) {
    if (!dst || bytes < 0 || (bytes & 3)) return -1;
    if (bytes == 0) return 0;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_zero, grid1(bytes / 4), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint32_t *>(dst), bytes / 4);
    return status(hipGetLastError());
}

int unet_features(const uint8_t *active, const uint8_t *n_cat, const float *omega, float tau_ref, uint16_t *feat,
                  float *weight, float weight_power, float weight_cap, int32_t nz, int32_t ny, int32_t nx,
                  void *stream) {
    if (!active || !omega || !feat || nz <= 0 || ny <= 0 || nx <= 0 || !(tau_ref > 0.5f)) return -1;
    if (weight && !(weight_cap >= 1.f && weight_power >= 0.f && weight_power <= 4.f)) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_features, grid1((int64_t)nz * ny * nx), dim3(256), 0, static_cast<hipStream_t>(stream),
                       active, n_cat, omega, tau_ref, feat, weight, weight_power, weight_cap, nz, ny, nx);
    return status(hipGetLastError());
}

int unet_log_map(const float *src, float *dst, int64_t n, float eps, int32_t inverse, float cmax, void *stream) {
    if (!src || !dst || n <= 0 || !(eps > 0.f) || !(cmax > 0.f)) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_log_map, grid1(n), dim3(256), 0, static_cast<hipStream_t>(stream), src, dst, n, eps,
                       inverse ? 1 : 0, cmax);
    return status(hipGetLastError());
}

int unet_start_field(const float *y, const uint8_t *depth, int32_t depth_max, float eps, float cmax, float *c,
                     int64_t n, void *stream) {
    if (!y || !depth || !c || n <= 0 || depth_max < 0 || !(eps > 0.f) || !(cmax > 0.f)) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_start_field, grid1(n), dim3(256), 0, static_cast<hipStream_t>(stream), y, depth, depth_max,
                       eps, cmax, c, n);
    return status(hipGetLastError());
}

int unet_corrector_map(const float *src, float *dst, int64_t nvox, int32_t nx, float c_in, float c_out,
                       int32_t inverse, float cmax, void *stream) {
    if (!src || !dst || nvox <= 0 || nx <= 0 || nvox % nx || !(c_in != c_out) || !(cmax > 0.f)) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_corrector, grid1(nvox), dim3(256), 0, static_cast<hipStream_t>(stream), src, dst, nvox, nx,
                       c_in, c_out, inverse ? 1 : 0, cmax);
    return status(hipGetLastError());
}

int unet_mfma_selftest(const float *a, const float *b, float *d, void *stream) {
    if (!a || !b || !d) return -1;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_mfma_selftest, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), a, b, d);
    return status(hipGetLastError());
}

}  // extern "C"

namespace unet {

int conv3d(const Conv &c, int nz, int ny, int nx, int cin, int cout, void *stream) {
    if (c.m && (c.ldm % 8 || c.offm % 8 || !ch_ok(c.ldm, c.offm, cout) || !aligned16(c.m, nullptr, nullptr))) return -1;
    const bool cat = c.x2 != nullptr;
    if (cat && (nz % 2 || ny % 2 || nx % 2 || c.cin1 >= cin)) return -1;
    ConvArgs a{c.x, c.w, c.b, c.y, nullptr, c.ldx, 0, c.ldy, 0, nz, ny, nx, cin, cout, 0, c.relu, 0, 0, 0,
               cat ? c.x2 : c.x, cat ? c.ldx2 : c.ldx, 0, cat ? c.cin1 : cin, cat ? 1 : 0, 0, 0,
               nullptr, nullptr, nullptr, nullptr, c.m, c.ldm, c.offm, 1};
    const int h = cat ? 2 : 1;
    return launch_conv(a, nx / h, ny / h, nz / h, stream);
}

int pool_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                  int offm, int nz, int ny, int nx, int c, void *stream) {
    if (!dy || !dx || (nz | ny | nx) & 1 || nz <= 0 || !ch_ok(ldx, offx, c) || !ch_ok(ldy, offy, c)) return -1;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (runs8(c, ldx | ldm, offx | offm, ldy, offy) && aligned16(dy, dx, m) && (int64_t)nz * ny * nx * (c / 8) < ((int64_t)1 << 32)) {
        hipLaunchKernelGGL(k_pool_bwd8, grid1((int64_t)nz * ny * nx * (c / 8)), dim3(256), 0, st, dy, ldy, offy, dx, ldx,
                           offx, m, ldm, offm, (uint32_t)nz, (uint32_t)ny, (uint32_t)nx, (uint32_t)(c / 8));
        return status(hipGetLastError());
    }
    if (m) return -1;
    hipLaunchKernelGGL(k_pool_bwd, grid1((int64_t)nz * ny * nx * c), dim3(256), 0, st, dy, ldy, offy, dx, ldx, offx, nz,
                       ny, nx, c);
    return status(hipGetLastError());
}

int up_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                int offm, int nz, int ny, int nx, int c, void *stream) {
    if (!dy || !dx || (nz | ny | nx) & 1 || nz <= 0 || !ch_ok(ldx, offx, c) || !ch_ok(ldy, offy, c)) return -1;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (runs8(c, ldx | ldm, offx | offm, ldy, offy) && aligned16(dy, dx, m) &&
        (int64_t)nz * ny * nx / 8 * (c / 8) < ((int64_t)1 << 32)) {
        hipLaunchKernelGGL(k_up_bwd8, grid1((int64_t)nz * ny * nx / 8 * (c / 8)), dim3(256), 0, st, dy, ldy, offy, dx, ldx,
                           offx, m, ldm, offm, (uint32_t)nz, (uint32_t)ny, (uint32_t)nx, (uint32_t)(c / 8));
        return status(hipGetLastError());
    }
    if (m) return -1;
    hipLaunchKernelGGL(k_up_bwd, grid1((int64_t)nz * ny * nx / 8 * c), dim3(256), 0, st, dy, ldy, offy, dx, ldx, offx, nz,
                       ny, nx, c);
    return status(hipGetLastError());
}

int head_bwd_relu(const uint16_t *x, int ldx, const float *w, const float *dout, uint16_t *dx, float *dw, float *db,
                  int64_t nvox, int c, void *stream) {
    return head_bwd<true>(x, ldx, w, dout, dx, dw, db, nvox, c, stream);
}

int64_t conv3d_packed_len(int cin, int cout) { return packed_len(cin, cout); }

int conv3d_pack(const uint16_t *w, uint16_t *packed, const PackTable &t, void *stream) {
    if (!w || !packed || t.n <= 0 || t.n > kMaxPack || !aligned16(w, packed, nullptr)) return -1;
    int64_t most = 0;
    for (int l = 0; l < t.n; ++l) {
        if (t.l[l].cin % 16 || t.l[l].cout % 16 || t.l[l].from % 8 || t.l[l].to % 8) return -1;
        most = std::max(most, packed_len(t.l[l].cin, t.l[l].cout) / 8);
    }
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_pack, dim3((unsigned)std::min<int64_t>((most + 255) / 256, 256), (unsigned)t.n), dim3(256), 0,
                       static_cast<hipStream_t>(stream), w, packed, t);
    return status(hipGetLastError());
}

}  // namespace unet
