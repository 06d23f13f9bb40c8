// Structure characterisation on the device (Chen et al., arXiv 1410.1914,
// Section 2.1.3): the 13-direction pore size behind the Knudsen diffusivity
// (Eqs. 8-9), and the reach of the transport phases from the Dirichlet faces.
// These are the two host steps of lbm_create whose cost grows with the voxel
// count; here they run on maps already resident in HBM.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <numeric>

#include "kernels.h"
#include "prep.h"

namespace {

// The 13 directions of Section 2.1.3 (one of each opposite pair), in the order in
// which their contributions are summed, with |d| and, for directions without an
// x component, the number of voxels on their closed loop under the y/z wrap.
struct Dir13 {
    int d[13][3];
    double len[13];
    int64_t cap[13];
};

constexpr int kDirs[13][3] = {{1, 0, 0},  {0, 1, 0},  {0, 0, 1}, {1, 1, 0},  {1, -1, 0}, {1, 0, 1},  {1, 0, -1},
                              {0, 1, 1},  {0, 1, -1}, {1, 1, 1}, {1, 1, -1}, {1, -1, 1}, {-1, 1, 1}};

__device__ __forceinline__ int mbcnt64(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int wrap1(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// Length in voxels of the run of pore voxels through (x, y, z) along direction d, walked
// both ways: bounded by the x faces, at most one loop when the line closes on itself.
__device__ __forceinline__ int64_t walk_run(const uint8_t *__restrict__ pore, int nx, int ny, int nz, const Dir13 &D,
                                            int d, int x, int y, int z) {
    const int dx = D.d[d][0], dy = D.d[d][1], dz = D.d[d][2];
    const int64_t cap = D.cap[d];
    int64_t count = 1;
    for (int s = -1; s <= 1; s += 2) {
        int cx = x, cy = y, cz = z;
        while (count < cap) {
            cx += s * dx;
            cy = wrap1(cy + s * dy, ny);
            cz = wrap1(cz + s * dz, nz);
            if (cx < 0 || cx >= nx) break;
            if (!pore[((int64_t)cz * ny + cy) * nx + cx]) break;
            ++count;
        }
    }
    return count;
}

// Pore size of every voxel by walking: the mean over the 13 directions of its run times
// |d|.  The products and sums are kept apart (no fused multiply-add), as in a plain
// FP64 evaluation.  For grids whose sheets (below) do not fit LDS.
__global__ __launch_bounds__(256) void k_pore_size(const uint8_t *__restrict__ pore, int nx, int ny, int nz, Dir13 D,
                                                   double *__restrict__ dp) {
    const int64_t N = (int64_t)nx * ny * nz;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    if (!pore[v]) {
        dp[v] = 0.0;
        return;
    }
    const int x = (int)(v % nx);
    const int64_t row = v / nx;
    const int y = (int)(row % ny), z = (int)(row / ny);
    double sum = 0.0;
    for (int d = 0; d < 13; ++d) {
        const int64_t count = walk_run(pore, nx, ny, nz, D, d, x, y, z);
        {
#pragma clang fp contract(off)
            sum = sum + (double)count * D.len[d];
        }
    }
    dp[v] = sum / 13.0;
}

// ------------------------------------------------------------------ pore size by sheets
//
// A sheet is a set of x rows r = 0 .. R - 1 that closes on itself: the rows of a z plane
// (kind 0), of a y plane (1), or of the planes y = c + z (2) and y = c - z (3), with the
// y/z wrap.  Every direction of Dir13 lies in one kind: along the rows' x, up the sheet
// (the next row, same x) or along one of its two diagonals.  A workgroup holds one sheet
// as bits in LDS and lays the lines of each direction out as bit strings, so a voxel's
// run is a count of leading and trailing ones in the bits either side of it:
//   P[k][r]   x rows (word k of row r)           V[k][x]   columns (a ring of R rows)
//   U[k][l]   diagonals r - x = l (mod R)        W[k][l]   diagonals r + x = l (mod R)
// Strings have a margin on both sides: two words of zeros beyond the x faces, kRingWords of
// the ring's other end for columns.  Kinds 1, 2, 3 leave their three counts in the voxel's own output word (7 bits
// each, 127: too long, walked again); kind 0 adds its four and sums in Dir13's order.
// Walking every voxel's 26 half lines through the byte map took 3.05 ms at 256^3 NPMC, the
// four kinds take 0.44 ms: bound by the instructions of the counting (three quarters of
// it), not by the 0.94 GB they move.
constexpr int kSheetThreads = 1024;
constexpr int kLong = 127;
constexpr int kRingWords = 4;  // margin of a ring's string, in words

struct SheetGeom {
    int nx, ny, nz, rows;
};

template <int KIND>
__device__ __forceinline__ void sheet_row(const SheetGeom &g, int sheet, int r, int &y, int &z) {
    if (KIND == 0) {
        y = r;
        z = sheet;
    } else if (KIND == 1) {
        y = sheet;
        z = r;
    } else {
        const bool square = g.ny == g.nz;  // then r < ny
        z = square ? r : r % g.nz;
        const int t = square ? r : r % g.ny;
        y = wrap1(KIND == 2 ? sheet + t : sheet - t, g.ny);
    }
}

// words of a line of x (two words of zeros before it), and of a ring of rows with
// kRingWords words of its other end on both sides
template <class T>
__host__ __device__ __forceinline__ T sheet_words(T nx) { return nx / 32 + 5; }
template <class T>
__host__ __device__ __forceinline__ T ring_words(T rows) { return rows / 32 + 1 + 2 * kRingWords; }

// Run of ones through a set bit of a string.  m: the string's word that holds the bit 63
// places below it, words `step` apart; sh: where in that word.  64 bits on either side
// are counted without a branch; longer runs loop on, inside the string's margins.
template <bool RING>
__device__ __forceinline__ int run_at(const uint32_t *m, int step, int sh, int ring) {
    const uint32_t w0 = m[0], w1 = m[step], w2 = m[2 * step], w3 = m[3 * step], w4 = m[4 * step];
    const uint32_t d0 = ~__builtin_amdgcn_alignbit(w2, w1, sh), d1 = ~__builtin_amdgcn_alignbit(w1, w0, sh);
    const uint32_t u0 = ~__builtin_amdgcn_alignbit(w3, w2, sh), u1 = ~__builtin_amdgcn_alignbit(w4, w3, sh);
    int a = d0 ? __builtin_clz(d0) : 32 + __builtin_clz(d1);  // set below where all 64 are ones
    int b = u0 ? __builtin_ctz(u0) : 32 + __builtin_ctz(u1);
    if ((d0 | d1) == 0u) {
        uint32_t w = 0u;
        int k = 2;
        for (; w == 0u && k < (RING ? kRingWords : 1 << 20); ++k)
            w = ~__builtin_amdgcn_alignbit(m[(2 - k) * step], m[(1 - k) * step], sh);
        a = 32 * k - (w ? 32 - __builtin_clz(w) : 0);
    }
    if ((u0 | u1) == 0u) {
        uint32_t w = 0u;
        int k = 2;
        for (; w == 0u && k < (RING ? kRingWords : 1 << 20); ++k)
            w = ~__builtin_amdgcn_alignbit(m[(3 + k) * step], m[(2 + k) * step], sh);
        b = 32 * k - (w ? 32 - __builtin_ctz(w) : 0);
    }
    return RING ? min(a + b, ring) : a + b;
}

template <int KIND>
__global__ __launch_bounds__(kSheetThreads) void k_pore_sheet(const uint8_t *__restrict__ pore, SheetGeom g, Dir13 D,
                                                              double *__restrict__ dp) {
    extern __shared__ uint32_t lds[];
    // P's columns go on past row R - 1 with the ring's first rows, so that 32 rows in a row
    // are read without a wrap
    const int nx = g.nx, R = g.rows, RP = R + 32, nk = sheet_words(nx), nr = ring_words(R);
    uint32_t *P = lds, *U = P + nk * RP, *W = U + nk * R, *V = W + nk * R;
    const int tid = threadIdx.x, lane = tid & 63, sheet = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kWaves = kSheetThreads / 64, kMlp = 8, kOut = 4;
    // waves take chunks of 64 x (cw at a time) and, per chunk, every `rstep`-th row
    const int nch = (nx + 63) / 64, cw = min(nch, kWaves), rstep = kWaves / cw;
    const int c_first = wave % cw, r_first = wave / cw < rstep ? wave / cw : R;
    for (int i = tid; i < 2 * RP; i += kSheetThreads) P[i] = 0u;
    for (int i = 2 * (nch + 1) * RP + tid; i < nk * RP; i += kSheetThreads) P[i] = 0u;
    for (int c = c_first; c < nch; c += cw) {
        const int x = c * 64 + lane;
        for (int r0 = r_first; r0 < R; r0 += rstep * kMlp) {  // kMlp rows' loads in flight
            uint8_t b[kMlp];
#pragma unroll
            for (int q = 0; q < kMlp; ++q) {
                int y, z;
                sheet_row<KIND>(g, sheet, min(r0 + q * rstep, R - 1), y, z);
                b[q] = x < nx ? pore[((int64_t)z * g.ny + y) * nx + x] : (uint8_t)0;
            }
#pragma unroll
            for (int q = 0; q < kMlp; ++q) {
                const uint64_t m = __ballot(b[q] != 0);
                const int k = 2 * (c + 1) + lane;
                if (lane < 2 && k < nk) P[k * RP + min(r0 + q * rstep, R - 1)] = (uint32_t)(m >> (32 * lane));
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < nk * 32; i += kSheetThreads) P[(i >> 5) * RP + R + (i & 31)] = P[(i >> 5) * RP + (i & 31) % R];
    __syncthreads();
    for (int i = tid; i < nk * R; i += kSheetThreads) {  // both diagonals of word k through line l
        const int k = i / R, l = i - k * R;
        uint32_t u = 0u, w = 0u;
        if (k > 1) {
            const int x0 = 32 * (k - 2) % R, x1 = (x0 + 31) % R;
            int ru = l + x0, rw = l - x1;  // rows of bit 0 of u and of bit 31 of w
            if (ru >= R) ru -= R;
            if (rw < 0) rw += R;
            const uint32_t *pu = P + k * RP + ru, *pw = P + k * RP + rw;
#pragma unroll
            for (int b = 0; b < 32; ++b) {
                u |= pu[b] & (1u << b);
                w |= pw[31 - b] & (1u << b);
            }
        }
        U[i] = u;
        W[i] = w;
    }
    for (int i = tid; i < nr * nx; i += kSheetThreads) {  // columns: string bit s is row s - 32 kRingWords of the ring
        const int k = i / nx, x = i - k * nx, sh = x & 31;
        const uint32_t *col = P + ((x >> 5) + 2) * RP + ((32 * (k - kRingWords)) % R + R) % R;
        uint32_t v = 0u;
#pragma unroll
        for (int b = 0; b < 32; ++b) v |= ((col[b] >> sh) & 1u) << b;
        V[i] = v;
    }
    __syncthreads();
    uint8_t *todo = reinterpret_cast<uint8_t *>(V + nr * nx) + wave * (64 * kOut);
    // this workgroup's share of the sheet's rows
    const int r_lo = R * (int)blockIdx.y / (int)gridDim.y, r_hi = R * ((int)blockIdx.y + 1) / (int)gridDim.y;
    for (int c = c_first; c < nch; c += cw) {
        const int xc = c * 64 + lane;
        for (int r0 = r_lo + r_first; r0 < r_hi; r0 += rstep * kOut) {
            // the pore voxels of kOut rows, packed to the front: less than half of the lanes
            // of a row are pore, and the counting below is bound by its instructions
            int64_t base[kOut];
            int n = 0;
#pragma unroll
            for (int q = 0; q < kOut; ++q) {
                const int r = r0 + q * rstep;
                int y, z;
                sheet_row<KIND>(g, sheet, min(r, R - 1), y, z);
                base[q] = ((int64_t)z * g.ny + y) * nx + c * 64;
                const bool in = r < r_hi && xc < nx;
                const bool set = in && ((P[((xc >> 5) + 2) * RP + r] >> (xc & 31)) & 1u) != 0u;
                const uint64_t m = __ballot(set);
                if (set) todo[n + mbcnt64(m)] = (uint8_t)(q * 64 + lane);
                if (KIND == 0 && in && !set) dp[base[q] + lane] = 0.0;
                n += __popcll(m);
            }
            uint64_t old[kOut];
            int64_t vox[kOut];
            int rr[kOut], xx[kOut];
#pragma unroll
            for (int q = 0; q < kOut; ++q) {  // every packed voxel's stored counts in flight
                old[q] = 0u;
                if (q * 64 + lane >= n) continue;
                const int e = todo[q * 64 + lane], f = e >> 6;
                static_assert(kOut == 4, "the selection below");
                rr[q] = r0 + f * rstep;
                xx[q] = c * 64 + (e & 63);
                vox[q] = (f & 2 ? (f & 1 ? base[3] : base[2]) : (f & 1 ? base[1] : base[0])) + (e & 63);
                if (KIND != 1) old[q] = reinterpret_cast<const uint64_t *>(dp)[vox[q]];
            }
#pragma unroll
            for (int q = 0; q < kOut; ++q) {
                if (q * 64 + lane >= n) continue;
                const int r = rr[q], x = xx[q], xr = nx <= R ? x : x % R, wx = (x + 1) >> 5, sx = (x + 1) & 31;
                int lu = r - xr, lw = r + xr;
                if (lu < 0) lu += R;
                if (lw >= R) lw -= R;
                const int sr = r + 32 * kRingWords - 63, at = __mul24(wx, R);
                const int cv = run_at<true>(V + __mul24(sr >> 5, nx) + x, nx, sr & 31, R);
                const int cu = run_at<false>(U + at + lu, R, sx, 0), cd = run_at<false>(W + at + lw, R, sx, 0);
                if constexpr (KIND != 0) {
                    const uint64_t k =
                        (uint64_t)min(cv, kLong) | (uint64_t)min(cu, kLong) << 7 | (uint64_t)min(cd, kLong) << 14;
                    reinterpret_cast<uint64_t *>(dp)[vox[q]] = old[q] | k << (21 * (KIND - 1));
                } else {
                    // Dir13's order; the stored counts: kind 1 z, (1,0,1), (1,0,-1); kind 2 (0,1,1),
                    // (1,1,1), (-1,1,1); kind 3 (0,1,-1), (1,-1,1), (1,1,-1)
                    const int own[4] = {run_at<false>(P + __mul24(wx, RP) + r, RP, sx, 0), cv, cu, cd};
                    constexpr int kFrom[13] = {-1, -2, 0, -3, -4, 1, 2, 3, 6, 4, 8, 7, 5};
                    // a ring longer than the string's margins: counts from kLong on are walked
                    double sum = 0.0;
#pragma unroll
                    for (int d = 0; d < 13; ++d) {
                        int k = kFrom[d] < 0 ? own[-1 - kFrom[d]] : (int)((old[q] >> (7 * kFrom[d])) & 127u);
                        if ((kFrom[d] >= 0 || d == 1) && k >= kLong)
                            k = (int)walk_run(pore, nx, g.ny, g.nz, D, d, x, r, sheet);
                        {
#pragma clang fp contract(off)
                            sum = sum + (double)k * D.len[d];
                        }
                    }
                    dp[vox[q]] = sum / 13.0;
                }
            }
        }
    }
}

size_t sheet_lds(int64_t nx, int64_t rows) {
    return 4 * (size_t)(sheet_words(nx) * (3 * rows + 32) + ring_words(rows) * nx) + 4 * kSheetThreads;
}
constexpr size_t kMaxLds = 160 << 10;

// Lets a kernel's launches ask for up to `bytes` of dynamic LDS.  The limit belongs to the
// process: every call sets the one value that all sizes share, so that calls of other host
// threads never find it lowered between here and their launch.
hipError_t allow_lds(const void *kernel, size_t bytes) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int KIND>
hipError_t launch_pore_sheet(const uint8_t *pore, int nx, int ny, int nz, const Dir13 &D, double *dp, hipStream_t st) {
    const int gcd = std::gcd(ny, nz);
    const SheetGeom g{nx, ny, nz, KIND == 0 ? ny : KIND == 1 ? nz : ny / gcd * nz};
    const size_t lds = sheet_lds(nx, g.rows);
    const hipError_t e = allow_lds(reinterpret_cast<const void *>(k_pore_sheet<KIND>), kMaxLds);
    if (e != hipSuccess) return e;
    // Few sheets leave CUs idle: several workgroups then share one, each laying out all of its
    // lines (25 us of a kind's 85-140 us at 256^3) and counting four rows or more.  128^3: 158
    // us with one, 124 with two; 64^3: 70 with one, 59 with four; 256^3: 441 with one, 508 with
    // two; 48 x 50 x 50 (two sheets of 1200 rows): 182 with three, 136 with 128.
    const int sheets = KIND == 0 ? nz : KIND == 1 ? ny : gcd, share = std::max(1, std::min(256 / sheets, g.rows / 4));
    hipLaunchKernelGGL(k_pore_sheet<KIND>, dim3(sheets, share), dim3(kSheetThreads), lds, st, pore, g, D, dp);
    return hipGetLastError();
}

// Whether the pore size is counted by sheets.  They have to fit LDS, and the lines that a
// workgroup lays out for itself must not take longer than walking: yz diagonals that close
// late make a few very long sheets, which each workgroup on them lays out whole.  By sheets:
// the four launches take 45 us, the lines 6.5 ns a word along x and the diagonals and 2 a
// word of a column (within 15% over the sizes below).  Walking: about 57 us and 1 us for
// 10500 voxels in random maps of 45% pore, 85 us and 1 us for 8000 in grown structures, whose
// runs are longer; the line lies between the two, and lower where rows are so short that no
// run along x is long.  us by sheets / walked, grown and random: 50^3 56 / 97, 62; 40 x 50 x 50
// (ten sheets of 200 rows) 66 / 93, 61; 48 x 60 x 64 70 / 93, 64; 16 x 24 x 240 74 / 96, 59; 80 x
// 100 x 64 97 / 157, 97; 55 x 60 x 57 (five of 660) 100 / -, 58; 3 x 300 x 100 103 / 104, 57; 48 x
// 50 x 50 (two of 1200) 136 / 93, 62; 32 x 31 x 100 (one of 992) 181 / 99, 59.  Random, short
// rows: 8^3 48 / 48, 39 x 4 x 8 57 / 46, 7 x 10 x 1 48 / 26.
bool by_sheets(int64_t nx, int64_t ny, int64_t nz) {
    const int64_t ring = std::lcm(ny, nz);
    if (sheet_lds(nx, std::max({ny, nz, ring})) > kMaxLds) return false;
    const int64_t lines = sheet_words(nx) * (ny + nz + 2 * ring);
    const int64_t columns = nx * (ring_words(ny) + ring_words(nz) + 2 * ring_words(ring));
    const double walk = (70.0 + (double)(nx * ny * nz) / 9000.0) * std::min(1.0, 0.3 + 0.7 * (double)nx / 15.0);
    return 45.0 + 0.0065 * (double)lines + 0.002 * (double)columns <= walk;
}

// Seeds of the reach: pass voxels on the selected x faces.
__global__ __launch_bounds__(256) void k_reach_seed(const uint8_t *__restrict__ pass, int nx, int ny, int nz, int faces,
                                                    uint8_t *__restrict__ hit) {
    const int64_t N = (int64_t)nx * ny * nz;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const int x = (int)(v % nx);
    hit[v] = (uint8_t)(pass[v] && (((faces & 1) && x == 0) || ((faces & 2) && x == nx - 1)));
}

// One sweep along `axis` (0 x, 1 y, 2 z): one thread per line, walked forward and
// then backward, carrying reach along the line and taking it from the four
// neighbours across the line.  Reach only ever turns on, so threads racing on a
// voxel agree; a sweep that turns nothing on leaves *changed untouched.
__global__ __launch_bounds__(256) void k_reach_sweep(const uint8_t *__restrict__ pass, uint8_t *hit, int nx, int ny,
                                                     int nz, int axis, int *changed) {
    const int n[3] = {nx, ny, nz};
    const int a1 = axis == 0 ? 1 : 0, a2 = axis == 2 ? 1 : 2;  // the two axes across the line
    const int64_t lines = (int64_t)n[a1] * n[a2];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= lines) return;
    int c[3];
    c[a1] = (int)(t % n[a1]);
    c[a2] = (int)(t / n[a1]);
    const int L = n[axis];
    auto at = [&](int cx, int cy, int cz) { return ((int64_t)cz * ny + cy) * nx + cx; };
    auto across = [&](int i) -> bool {  // reach of a neighbour across the line, with the y/z wrap
        int p[3] = {c[0], c[1], c[2]};
        p[axis] = i;
        const int cx = p[0], cy = p[1], cz = p[2];
        bool h = false;
        if (axis != 0) {
            if (cx > 0) h = h || hit[at(cx - 1, cy, cz)];
            if (cx + 1 < nx) h = h || hit[at(cx + 1, cy, cz)];
        }
        if (axis != 1) h = h || hit[at(cx, wrap1(cy - 1, ny), cz)] || hit[at(cx, wrap1(cy + 1, ny), cz)];
        if (axis != 2) h = h || hit[at(cx, cy, wrap1(cz - 1, nz))] || hit[at(cx, cy, wrap1(cz + 1, nz))];
        return h;
    };
    bool any = false;
    for (int pass_dir = 0; pass_dir < 2; ++pass_dir) {
        bool carry = false;
        for (int k = 0; k < L; ++k) {
            const int i = pass_dir ? L - 1 - k : k;
            int p[3] = {c[0], c[1], c[2]};
            p[axis] = i;
            const int64_t v = at(p[0], p[1], p[2]);
            if (!pass[v]) {
                carry = false;
                continue;
            }
            bool h = hit[v] != 0;
            if (!h && (carry || across(i))) {
                hit[v] = 1;
                h = true;
                any = true;
            }
            carry = h;
        }
    }
    if (any) *changed = 1;
}

// Bits of p in a run (maximal block of consecutive set bits) that holds a bit of
// h (h within p): adding h to p carries from the lowest such bit to the run's end,
// the same on reversed bits covers the run's start.
__device__ __forceinline__ uint64_t fill_runs(uint64_t p, uint64_t h) {
    const uint64_t up = ((p + h) ^ p) & p;
    const uint64_t pr = __brevll(p), hr = __brevll(h);
    const uint64_t down = __brevll(((pr + hr) ^ pr) & pr);
    return up | down | h;
}

// The x sweep with one wave per x line: 64 voxels at a time as bit masks (pass,
// reach including the four neighbours across the line), runs filled with
// fill_runs, and reach carried across 64-voxel chunks forward and then backward.
__global__ __launch_bounds__(256) void k_reach_sweep_x(const uint8_t *__restrict__ pass, uint8_t *hit, int nx,
                                                       int ny, int nz, int *changed) {
    const int lane = threadIdx.x & 63;
    const int64_t line = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (line >= (int64_t)ny * nz) return;  // whole waves leave together
    const int y = (int)(line % ny), z = (int)(line / ny);
    const int64_t base = line * nx;
    const int64_t ym = ((int64_t)z * ny + wrap1(y - 1, ny)) * nx, yp = ((int64_t)z * ny + wrap1(y + 1, ny)) * nx;
    const int64_t zm = ((int64_t)wrap1(z - 1, nz) * ny + y) * nx, zp = ((int64_t)wrap1(z + 1, nz) * ny + y) * nx;
    const int nch = (nx + 63) / 64;
    bool any = false;
    for (int dir = 0; dir < 2; ++dir) {
        bool carry = false;  // the voxel next to this chunk, on the side already swept, is reached
        for (int k = 0; k < nch; ++k) {
            const int c = dir ? nch - 1 - k : k;
            const int x = c * 64 + lane;
            const bool in = x < nx;
            const bool ps = in && pass[base + x];
            const bool h0 = ps && hit[base + x];
            const bool ac = ps && (hit[ym + x] || hit[yp + x] || hit[zm + x] || hit[zp + x]);
            const uint64_t P = __ballot(ps);
            uint64_t H = __ballot(h0 || ac);
            if (carry) H |= dir ? (P & (1ull << 63)) : (P & 1ull);
            const uint64_t R = P ? fill_runs(P, H) : 0ull;
            const bool now = (R >> lane) & 1ull;
            if (now && !h0) {
                hit[base + x] = 1;
                any = true;
            }
            const int edge = dir ? 0 : 63;  // the chunk's last voxel in sweep order
            carry = ((R >> edge) & 1ull) != 0 && (dir ? c * 64 : c * 64 + 63) < nx;
        }
    }
    if (any) *changed = 1;
}

// ------------------------------------------------------------------ reach by sheets
//
// While it runs, a byte of `hit` holds bit 0: reached, bit 1: pass.  A workgroup takes
// one sheet of x rows (all y of a z plane, or all z of a y plane) into LDS as bit words,
// [word][row], and fills it in up to kReachRounds rounds: rows by carry arithmetic, a word
// at a time, and columns by doubling, 64 rows to a wave.  Either half reads one copy of
// the reached bits and writes the other, so the state after every launch, and with it
// the number of cycles, is the same every time.  A cycle is a launch over the z planes
// and one over the y planes; one that turns nothing on has found the exact answer.
// One thread per line in y and z, bytes read one by one: 0.6 ms a sweep at 256^3.
constexpr int kReachThreads = 1024;
// Rounds of rows and columns per launch: 2D paths are far longer than 3D ones, so filling
// a sheet to the end is wasted on the first cycles.  256^3 NPMC: 534 us in 12 cycles with
// one round, 338 / 6 with four, 312 / 5 with eight, 352 / 5 with 32, 420 / 5 without a
// limit (9.2 ms in 7 cycles of line sweeps over the bytes).
constexpr int kReachRounds = 8;
constexpr int kReachRows = 4;  // columns fill 2 kReachRows - 1 rows at a time: most runs, in half the shuffles of 64

__device__ __forceinline__ uint64_t spread8(uint32_t b) {  // 8 bits to 8 bytes of 0 / 1
    const uint64_t t = (uint64_t)(b & 255u) * 0x0101010101010101ull & 0x8040201008040201ull;
    return (t + 0x7f7f7f7f7f7f7f7full) >> 7 & 0x0101010101010101ull;
}
__device__ __forceinline__ uint32_t gather8(uint64_t u) {  // 8 bytes of 0 / 1 to 8 bits
    return (uint32_t)(u * 0x0102040810204080ull >> 56);
}
__device__ __forceinline__ uint64_t nonzero8(uint64_t u) {  // bytes to 0 / 1
    return (((u & 0x7f7f7f7f7f7f7f7full) + 0x7f7f7f7f7f7f7f7full) | u) >> 7 & 0x0101010101010101ull;
}

struct ReachArgs {
    const uint8_t *pass;
    uint8_t *hit;
    int64_t row_stride, sheet_stride;
    int nx, rows, faces;
    int *changed;
};

// FIRST: the state from the pass map and the face seeds.  WIDE: rows lie on 8-byte
// boundaries and are moved 8 voxels at a time, otherwise voxel by voxel.
template <bool FIRST, bool WIDE>
__global__ __launch_bounds__(kReachThreads) void k_reach_sheet(ReachArgs a) {
    extern __shared__ uint64_t sheet_bits[];
    const int R = a.rows, nw = (a.nx + 63) / 64, tid = threadIdx.x, nth = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nwv = nth >> 6;
    uint64_t *P = sheet_bits, *H = P + nw * R, *G = H + nw * R;
    uint8_t *hit = a.hit + blockIdx.x * a.sheet_stride;
    const uint8_t *src = FIRST ? a.pass + blockIdx.x * a.sheet_stride : hit;
    if constexpr (WIDE) {
        const int n8 = a.nx / 8, m8 = nw * 8;  // the 8-bit parts of a row, stored and in all
        uint8_t *P8 = reinterpret_cast<uint8_t *>(P), *H8 = reinterpret_cast<uint8_t *>(H);
#pragma unroll 4
        for (int i = tid; i < m8 * R; i += nth) {
            const int r = i / m8, c = i - r * m8;
            uint64_t u = 0ull;
            if (c < n8) u = *reinterpret_cast<const uint64_t *>(src + r * a.row_stride + 8 * c);
            const uint32_t p = gather8(FIRST ? nonzero8(u) : u >> 1 & 0x0101010101010101ull);
            uint32_t h = FIRST ? 0u : gather8(u & 0x0101010101010101ull);
            if (FIRST && (a.faces & 1) && c == 0) h |= p & 1u;
            if (FIRST && (a.faces & 2) && c == n8 - 1) h |= p & 128u;
            const int at = ((c >> 3) * R + r) * 8 + (c & 7);
            P8[at] = (uint8_t)p;
            H8[at] = (uint8_t)h;
        }
    } else {
        for (int t = wave; t < R * nw; t += nwv) {
            const int r = t / nw, w = t - r * nw, x = 64 * w + lane;
            const uint32_t u = x < a.nx ? src[r * a.row_stride + x] : 0u;
            const bool p = FIRST ? u != 0u : (u & 2u) != 0u;
            const bool h = FIRST ? p && (((a.faces & 1) && x == 0) || ((a.faces & 2) && x == a.nx - 1)) : (u & 1u) != 0u;
            const uint64_t pm = __ballot(p), hm = __ballot(h);
            if (lane == 0) {
                P[w * R + r] = pm;
                H[w * R + r] = hm;
            }
        }
    }
    __syncthreads();
    bool grew = false;  // this thread turned something on
    const int nc = (R + 63) / 64;
    int more = 1;
    for (int round = 0; more && round < kReachRounds; ++round) {
        bool turned = false;
        for (int i = tid; i < nw * R; i += nth) {  // rows, H to G: a word, and what the words beside it bring in
            const uint64_t p = P[i], h = H[i];
            uint64_t n = h;
            if (i >= R) n |= p & H[i - R] >> 63;
            if (i < (nw - 1) * R) n |= p & H[i + R] << 63;
            if (n != 0ull && n != p) n = fill_runs(p, n);
            turned = turned || n != h;
            G[i] = n;
        }
        __syncthreads();
        for (int t = wave; t < nw * nc; t += nwv) {  // columns, G to H: 64 rows of one word to a wave
            const int w = t / nc, r = (t - w * nc) * 64 + lane;
            const bool in = r < R;
            const uint64_t p = in ? P[w * R + r] : 0ull, h = in ? G[w * R + r] : 0ull;
            uint64_t g = h;
            if (in && (lane == 0 || r == R - 1 || lane == 63)) {  // from the rows beside these (the ring's other end)
                if (lane == 0) g |= p & G[w * R + (r == 0 ? R - 1 : r - 1)];
                if (lane == 63 || r == R - 1) g |= p & G[w * R + (r == R - 1 ? 0 : r + 1)];
            }
            const uint64_t up = __shfl_up((unsigned long long)g, 1, 64), dn = __shfl_down((unsigned long long)g, 1, 64);
            if (__any((((lane > 0 ? up : 0ull) | (lane < 63 ? dn : 0ull)) & p & ~g) != 0ull)) {
                uint64_t q = p;
                for (int s = 1; s <= kReachRows; s <<= 1) {
                    const uint64_t gs = __shfl_up((unsigned long long)g, s, 64), qs = __shfl_up((unsigned long long)q, s, 64);
                    if (lane >= s) g |= q & gs;
                    q = lane >= s ? q & qs : 0ull;
                }
                q = p;
                for (int s = 1; s <= kReachRows; s <<= 1) {
                    const uint64_t gs = __shfl_down((unsigned long long)g, s, 64),
                                   qs = __shfl_down((unsigned long long)q, s, 64);
                    if (lane + s < 64) g |= q & gs;
                    q = lane + s < 64 ? q & qs : 0ull;
                }
            }
            turned = turned || g != h;
            if (in) H[w * R + r] = g;
        }
        grew = grew || turned;
        more = __syncthreads_or(turned);
    }
    const int any = __syncthreads_or(grew);
    if (any && tid == 0) *a.changed = 1;
    if (!FIRST && !any) return;  // nothing to store
    if constexpr (WIDE) {
        const int n8 = a.nx / 8;
        const uint8_t *P8 = reinterpret_cast<const uint8_t *>(P), *H8 = reinterpret_cast<const uint8_t *>(H);
        for (int i = tid; i < n8 * R; i += nth) {
            const int r = i / n8, c = i - r * n8, at = ((c >> 3) * R + r) * 8 + (c & 7);
            *reinterpret_cast<uint64_t *>(hit + r * a.row_stride + 8 * c) = spread8(P8[at]) << 1 | spread8(H8[at]);
        }
    } else {
        for (int t = wave; t < R * nw; t += nwv) {
            const int r = t / nw, w = t - r * nw, x = 64 * w + lane;
            const uint64_t p = P[w * R + r], h = H[w * R + r];
            if (x < a.nx) hit[r * a.row_stride + x] = (uint8_t)((p >> lane & 1ull) << 1 | (h >> lane & 1ull));
        }
    }
}

// The reached bit alone, the output's form.
__global__ __launch_bounds__(256) void k_reach_done(uint8_t *hit, int64_t n, int wide) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (wide) {
        if (i < n / 8) reinterpret_cast<uint64_t *>(hit)[i] &= 0x0101010101010101ull;
    } else if (i < n) {
        hit[i] &= 1u;
    }
}

// Clears n counters of the allocation-free reach's scratch (a kernel, not a
// memset, so the call stays free of memset nodes if a caller ever records it).
__global__ void k_zero_i32(int32_t *p, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = 0;
}

}  // namespace

// Scratch of lbm_reach_device_static: counters in device memory that the library
// never allocates.  Slots 0 and 1 are the change flags of the sweep cycles under way;
// the rest is reserved.  Each device holds its own copy for the life of the process.
constexpr int kReachScratchInts = 64;  // 256 bytes
static __device__ __align__(256) int32_t scratch[kReachScratchInts];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t *g_scratch_dev[kMaxDevices];  // device address of `scratch`, per device

// The device address of this device's `scratch`, looked up once per device with
// that device current (the symbol's host-side name is not a device address).
hipError_t reach_scratch(int32_t **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = static_cast<int32_t *>(ptr);
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

constexpr int kReachAhead = 2;  // cycles enqueued before their flags are read

size_t reach_lds(int64_t nx, int64_t rows) { return 24 * (size_t)((nx + 63) / 64 * rows); }
// What a sheet may take: k_reach_sheet's block-wide ORs have LDS of their own (256 bytes as
// compiled), which the launch adds to the sheet's.
constexpr size_t kMaxReachLds = kMaxLds - 1024;

template <bool FIRST, bool WIDE>
hipError_t launch_reach_t(const ReachArgs &a, int sheets, hipStream_t st) {
    const size_t lds = reach_lds(a.nx, a.rows);
    // few words: a wave to each 64 rows is enough
    const int threads = (a.nx + 63) / 64 * a.rows >= 512 ? kReachThreads : 256;
    hipLaunchKernelGGL((k_reach_sheet<FIRST, WIDE>), dim3(sheets), dim3(threads), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_reach(const ReachArgs &a, bool first, bool wide, int sheets, hipStream_t st) {
    if (first) return wide ? launch_reach_t<true, true>(a, sheets, st) : launch_reach_t<true, false>(a, sheets, st);
    return wide ? launch_reach_t<false, true>(a, sheets, st) : launch_reach_t<false, false>(a, sheets, st);
}

hipError_t allow_reach(bool wide) {
    const void *first = wide ? reinterpret_cast<const void *>(k_reach_sheet<true, true>)
                             : reinterpret_cast<const void *>(k_reach_sheet<true, false>);
    const void *next = wide ? reinterpret_cast<const void *>(k_reach_sheet<false, true>)
                            : reinterpret_cast<const void *>(k_reach_sheet<false, false>);
    const hipError_t e = allow_lds(first, kMaxReachLds);
    return e == hipSuccess ? allow_lds(next, kMaxReachLds) : e;
}

// Cycles until one turns nothing on: the loop both reach entry points share.  `flag_dev`
// holds kReachAhead change flags the kernels set; flag(true, nullptr) clears them,
// flag(false, v) waits for the work and reads them into v.  Sheets that do not
// fit LDS (planes of more than about 430,000 voxels) take line sweeps through the byte
// map instead.
template <class Flag>
hipError_t reach_cycles(const uint8_t *pass_dev, int32_t nx, int32_t ny, int32_t nz, int32_t faces, uint8_t *hit_dev,
                        hipStream_t st, int32_t *flag_dev, Flag &&flag, int32_t *n_cycles) {
    const int64_t N = (int64_t)nx * ny * nz;
    (void)hipGetLastError();
    if (reach_lds(nx, std::max(ny, nz)) <= kMaxReachLds) {
        const bool wide = nx % 8 == 0 && ((reinterpret_cast<uintptr_t>(pass_dev) | reinterpret_cast<uintptr_t>(hit_dev)) & 7) == 0;
        ReachArgs z{pass_dev, hit_dev, nx, (int64_t)ny * nx, nx, ny, faces, flag_dev};  // the rows of a z plane
        ReachArgs y{pass_dev, hit_dev, (int64_t)ny * nx, nx, nx, nz, faces, flag_dev};  // the rows of a y plane
        hipError_t e = allow_reach(wide);
        *n_cycles = 0;
        // two cycles to a wait: waiting costs about as much as a cycle of a small grid, and a
        // cycle after the last one changes nothing
        bool more = true;
        for (int64_t cyc = 0; e == hipSuccess && more && cyc <= N; cyc += kReachAhead) {
            e = flag(true, nullptr);
            for (int k = 0; k < kReachAhead; ++k) {
                z.changed = y.changed = flag_dev + k;
                if (e == hipSuccess) e = launch_reach(z, cyc + k == 0, wide, nz, st);
                if (e == hipSuccess) e = launch_reach(y, false, wide, ny, st);
            }
            int32_t changed[kReachAhead] = {};
            if (e == hipSuccess) e = flag(false, changed);
            for (int k = 0; k < kReachAhead && more; ++k) {
                ++*n_cycles;
                more = changed[k] != 0;
            }
        }
        if (e == hipSuccess) {
            const int64_t n = wide ? N / 8 : N;
            hipLaunchKernelGGL(k_reach_done, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, hit_dev, N, wide ? 1 : 0);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipStreamSynchronize(st);
        }
        return e;
    }
    hipLaunchKernelGGL(k_reach_seed, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, pass_dev, nx, ny, nz, faces,
                       hit_dev);
    hipError_t e = hipGetLastError();
    *n_cycles = 0;
    // every productive cycle turns at least one voxel on, so at most N + 1 cycles run
    for (int64_t cyc = 0; e == hipSuccess && cyc <= N; ++cyc) {
        e = flag(true, nullptr);
        if (e != hipSuccess) break;
        {
            const int64_t lines = (int64_t)ny * nz;  // x: one wave per line
            hipLaunchKernelGGL(k_reach_sweep_x, dim3((unsigned)((lines + 3) / 4)), dim3(256), 0, st, pass_dev, hit_dev,
                               nx, ny, nz, flag_dev);
            e = hipGetLastError();
        }
        for (int axis = 1; axis < 3 && e == hipSuccess; ++axis) {  // y, z: one thread per line
            const int64_t lines = axis == 1 ? (int64_t)nx * nz : (int64_t)nx * ny;
            hipLaunchKernelGGL(k_reach_sweep, dim3((unsigned)((lines + 255) / 256)), dim3(256), 0, st, pass_dev, hit_dev,
                               nx, ny, nz, axis, flag_dev);
            e = hipGetLastError();
        }
        int32_t changed[kReachAhead] = {};
        if (e == hipSuccess) e = flag(false, changed);
        ++*n_cycles;
        if (e != hipSuccess || !changed[0]) break;
    }
    return e;
}

}  // namespace

extern "C" {

int lbm_pore_size_device(const uint8_t *pore_dev, int32_t nx, int32_t ny, int32_t nz, double *dp_dev, void *stream) {
    if (!pore_dev || !dp_dev || nx <= 0 || ny <= 0 || nz <= 0) return LBM_ERR_INVALID_ARG;
    const int64_t N = (int64_t)nx * ny * nz;
    if ((N + 255) / 256 > INT32_MAX) return LBM_ERR_INVALID_ARG;
    Dir13 D{};
    for (int d = 0; d < 13; ++d) {
        const int dx = kDirs[d][0], dy = kDirs[d][1], dz = kDirs[d][2];
        for (int k = 0; k < 3; ++k) D.d[d][k] = kDirs[d][k];
        D.len[d] = std::sqrt((double)(dx * dx + dy * dy + dz * dz));
        D.cap[d] = dx != 0 ? INT64_MAX : (dy != 0 && dz != 0 ? std::lcm((int64_t)ny, (int64_t)nz) : (dy ? ny : nz));
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    hipError_t e = hipSuccess;
    if (by_sheets(nx, ny, nz)) {
        e = launch_pore_sheet<1>(pore_dev, nx, ny, nz, D, dp_dev, st);
        if (e == hipSuccess) e = launch_pore_sheet<2>(pore_dev, nx, ny, nz, D, dp_dev, st);
        if (e == hipSuccess) e = launch_pore_sheet<3>(pore_dev, nx, ny, nz, D, dp_dev, st);
        if (e == hipSuccess) e = launch_pore_sheet<0>(pore_dev, nx, ny, nz, D, dp_dev, st);
    } else {
        hipLaunchKernelGGL(k_pore_size, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, pore_dev, nx, ny, nz, D,
                           dp_dev);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    return cl::record_error(e, "lbm_pore_size_device");
}

int lbm_reach_device(const uint8_t *pass_dev, int32_t nx, int32_t ny, int32_t nz, int32_t faces, uint8_t *hit_dev,
                     int32_t *cycles, void *stream) {
    if (!pass_dev || !hit_dev || nx <= 0 || ny <= 0 || nz <= 0 || faces < 1 || faces > 3) return LBM_ERR_INVALID_ARG;
    const int64_t N = (int64_t)nx * ny * nz;
    if ((N + 255) / 256 > INT32_MAX) return LBM_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int *changed = nullptr;  // a flag per cycle, in pinned host memory the device writes directly
    hipError_t e = hipHostMalloc((void **)&changed, kReachAhead * sizeof(int), hipHostMallocMapped);
    int *changed_dev = nullptr;
    if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&changed_dev, changed, 0);
    int32_t n_cycles = 0;
    if (e == hipSuccess) {
        auto flag = [&](bool zero, int32_t *value) -> hipError_t {
            if (zero) {
                for (int k = 0; k < kReachAhead; ++k) changed[k] = 0;
                return hipSuccess;
            }
            const hipError_t se = hipStreamSynchronize(st);
            for (int k = 0; k < kReachAhead; ++k) value[k] = changed[k];
            return se;
        };
        e = reach_cycles(pass_dev, nx, ny, nz, faces, hit_dev, st, changed_dev, flag, &n_cycles);
    }
    if (changed) (void)hipHostFree(changed);
    if (cycles) *cycles = n_cycles;
    return cl::record_error(e, "lbm_reach_device");
}

int lbm_reach_device_static(const uint8_t *pass_dev, int32_t nx, int32_t ny, int32_t nz, int32_t faces,
                            uint8_t *hit_dev, int32_t *cycles, void *stream) {
    if (!pass_dev || !hit_dev || nx <= 0 || ny <= 0 || nz <= 0 || faces < 1 || faces > 3) return LBM_ERR_INVALID_ARG;
    const int64_t N = (int64_t)nx * ny * nz;
    if ((N + 255) / 256 > INT32_MAX) return LBM_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int32_t *flag_dev = nullptr;
    hipError_t e = reach_scratch(&flag_dev);
    int32_t n_cycles = 0;
    if (e == hipSuccess) {
        auto flag = [&](bool zero, int32_t *value) -> hipError_t {
            if (zero) {
                hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, st, flag_dev, kReachAhead);
                return hipGetLastError();
            }
            hipError_t ce = hipMemcpyAsync(value, flag_dev, kReachAhead * sizeof(int32_t), hipMemcpyDeviceToHost, st);
            if (ce == hipSuccess) ce = hipStreamSynchronize(st);
            return ce;
        };
        e = reach_cycles(pass_dev, nx, ny, nz, faces, hit_dev, st, flag_dev, flag, &n_cycles);
    }
    if (cycles) *cycles = n_cycles;
    return cl::record_error(e, "lbm_reach_device_static");
}

}  // extern "C"
