// The dense weight gradient of a 3x3 layer (stride 1, zero padding 1) on the
// matrix cores, for the primal step of the data-free ADMM loop (Sec. 4.3,
// Eq. 4) and, gathered at the kept taps, for the masked gradient of the
// retraining (Sec. 3.3):
//   dW[f][c][q] = sum over images and pixels p of g[n, f, p] x[n, c, p + off(q)]
// is a GEMM with M = filters, N = (tap, input channel) and K = pixels.
//
// fp16 values multiply by v_mfma_f32_32x32x16_f16 (exact products, fp32
// sums).  fp32 values split into three bf16 parts, a = a1 + a2 + a3 (each the
// rounding of what the ones before leave, so the sum is exact), and six of the
// nine products a_i b_j, i + j <= 4, by v_mfma_f32_32x32x16_bf16; what is
// dropped is below 2^-24 of a product (|a2| <= 2^-8 |a|, |a3| <= 2^-17 |a|; one
// rounding of fp32).  Six of those cost 0.38 of the fp32 MFMAs they replace.
// The six products of 16 pixels are summed from the smallest up, from zero, and
// only that sum is added to the accumulator: one rounding at the accumulator's
// size per 16 pixels, where the fp32 MFMA had four.
// Measured (dv + db of a layer, 60 % of the kernels dropped, vector kernels
// first, us): fp16 128 @ 28x28 b32 118 -> 52, 64 @ 32x32 b256 304 -> 104;
// fp32 256 @ 8x8 b256 254 -> 157, 64 @ 56x56 b32 148 -> 116; dense fp32
// 64 @ 32x32 b32 (fp32 MFMA first) 57 -> 53.
//
// A wave owns 32 filters x 32 channels x 9 taps (9 accumulators).  WT = 2: a
// block owns 64 x 64, four waves of the same pixels; WT = 1: 32 x 32, its
// waves take a quarter of the rows each and meet in LDS at the end (fewer
// partial sums where a layer has few channels).  K runs over tiles of RT rows
// x GT groups of 8 columns; rows count through the images with one zero row
// before each.  A tile is staged in LDS as 16-byte units of 8 columns,
//   dy[row][group][filter][8],  x[row][group][channel][8],
// which neighbouring lanes read from neighbouring addresses.  A unit is what
// one lane supplies to an MFMA; the columns beside it are one word of each
// neighbour, shifted in by v_alignbit.  The two halves of a wave take
// different rows.  Tiles are split over KS blocks whose partial sums go to KS
// workspace slots, added afterwards in slot order (deterministic).
//
// Range.  Parts are whole down to 2^-133 (subnormals are kept): a value of 2^-110
// or more is exactly the sum of its parts, a smaller one within 2^-134.  With
// factors below 2^29, n products are so within n 2^-105 of those of fp32, 2^-25 n
// of a sum of 2^-80.  A block with a sum that is not finite (also for the zero
// columns that stand beside the image), a nonzero sum below 2^-80, or an fp32
// value of 2^29 or more takes its sums again with fp32 multiply-adds over the
// pixels of the image alone.
#include "common.h"
#include "launch.h"

namespace psc {
namespace {

constexpr int kMaxKS = 128;             // workspace slots at most

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef uint16_t us2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f16v mfma(const u4& a, const u4& b, const f16v& c, IntC<DT_F16>) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f16v mfma(const u4& a, const u4& b, const f16v& c, IntC<DT_F32>) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// 8 columns of a row: fp16 as they are, fp32 split into three bf16 parts;
// the columns from `left` on read zero.
template <int DT> struct Raw { uint32_t w[DT == DT_F32 ? 8 : 4]; };

template <int DT>
__device__ __forceinline__ void finish_unit(Raw<DT>& v, int left, u4 (&parts)[DT == DT_F32 ? 3 : 1], us2& top) {
    if constexpr (DT == DT_F16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v.w[k] = left >= 2 * k + 2 ? v.w[k] : left == 2 * k + 1 ? v.w[k] & 0xffffu : 0;
        parts[0] = u4{v.w[0], v.w[1], v.w[2], v.w[3]};
    } else {
        uint32_t w[3][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f2 r = {2 * k < left ? __builtin_bit_cast(float, v.w[2 * k]) : 0.f,
                    2 * k + 1 < left ? __builtin_bit_cast(float, v.w[2 * k + 1]) : 0.f};
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                w[s][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, b2));
                r.x -= __builtin_bit_cast(float, w[s][k] << 16);
                r.y -= __builtin_bit_cast(float, w[s][k] & 0xffff0000u);
            }
            top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, w[0][k] & 0x7fff7fffu));
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) parts[s] = u4{w[s][0], w[s][1], w[s][2], w[s][3]};
    }
}

// v / d for 0 <= v < 2^16 by m = 2^32 / d rounded up (all ones: d = 1)
__device__ __forceinline__ int quot(int v, uint32_t m) { return m == 0xffffffffu ? v : int(__umulhi(uint32_t(v), m)); }

// The sizes of a call, kept in LDS for sum_again: in registers they would take
// scalars from the hot loop (1 to 1.5 % of its time).  For the same reason
// sum_again is a call (inlined: 512 @ 14x14 b64 fp16 183 us, 177 so) and comes
// after the store.
struct Sizes {
    int64_t tiles;
    int n, cin, H, W, cout, RT, GT, DU, U, gtiles, KS;
    uint32_t gt_m;
};

// The sums of a block that the matrix cores cannot give: the tiles staged
// again, whole, and summed by fp32 multiply-adds, 4 filters x 9 taps a lane (a
// quarter of the filters a wave, or with WT = 2 the wave's own in four goes).
// All that names a pixel is the same for the wave, so what lies outside the
// image is skipped and not multiplied.  Measured, dv + db with one infinity in
// the inputs, and in all of them (us; vector kernels, pixels read from memory
// one by one, here): fp16 128 @ 28x28 b32 120, 1773, 126 and 120, 4055, 277; fp32
// 256 @ 8x8 b256 255, 10245, 492 and 255, 12182, 558.
template <int DT, int WT>
__device__ __attribute__((noinline, cold)) void sum_again(const typename Elt<DT>::T* x, const typename Elt<DT>::T* g,
                                                          const Sizes& sz, float* out, char* lds) {
    using E = typename Elt<DT>::T;
    constexpr int NP = DT == DT_F32 ? 3 : 1, T = 32 * WT;
    auto u = [](int v) { return __builtin_amdgcn_readfirstlane(v); };    // the same in every lane
    const int n = u(sz.n), cin = u(sz.cin), H = u(sz.H), W = u(sz.W), cout = u(sz.cout);
    const int RT = u(sz.RT), GT = u(sz.GT), DU = u(sz.DU), U = u(sz.U), gtiles = u(sz.gtiles), KS = u(sz.KS);
    const uint32_t gt_m = u(sz.gt_m);
    const int f0 = blockIdx.x * T, c0 = blockIdx.y * T, ks = blockIdx.z;
    const int64_t t0 = sz.tiles * ks / KS, t1 = sz.tiles * (ks + 1) / KS;
    float* const dst = out + int64_t(ks) * cout * cin * 9;
    const int uo = U > GT ? 1 : 0, last = RT * GT - 1, dy_plane = DU * T * 16, x_plane = (RT + 2) * U * T * 16;
    char* const ldsG = lds;
    char* const ldsX = lds + NP * dy_plane;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wf = WT == 2 ? (wave & 1) * 32 : 0, wc = WT == 2 ? (wave >> 1) * 32 : 0;
    // the units of a tile as they are (fp32: columns 4 to 7 in the second plane)
    auto stage = [&](const E* p, int ch0, int chs, int row0, int grp0, int per, int units, char* to, int plane_bytes) {
        for (int e = int(threadIdx.x); e < units * T; e += 256) {
            const int u = e / T, ch = e - u * T, r = u / per, R = row0 + r, col = 8 * (grp0 + u - r * per);
            const int im = R < 0 ? -1 : R / (H + 1), i = R - im * (H + 1) - 1;
            const bool in = im >= 0 && im < n && i >= 0 && ch0 + ch < chs && col >= 0;
            const int64_t at = in ? (int64_t(im) * chs + ch0 + ch) * (H * W) + i * W + col : 0;
            E v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = in && col + k < W ? p[at + k] : E(0);
            __builtin_memcpy(to + e * 16, v, 16);
            if constexpr (DT == DT_F32) __builtin_memcpy(to + plane_bytes + e * 16, v + 4, 16);
        }
    };
    // the 8 columns of a unit
    auto columns = [&](const char* unit, int plane_bytes, float* v) {
        const u4 lo = *reinterpret_cast<const u4*>(unit);
        if constexpr (DT == DT_F16) {
            const h8 h = __builtin_bit_cast(h8, lo);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = float(h[e]);
        } else {
            const u4 hi = *reinterpret_cast<const u4*>(unit + plane_bytes);
            __builtin_memcpy(v, &lo, 16);
            __builtin_memcpy(v + 4, &hi, 16);
        }
    };
    auto column = [&](const char* unit, int plane_bytes, int e) {
        if constexpr (DT == DT_F16) return Elt<DT>::load(reinterpret_cast<const uint16_t*>(unit), e);
        else return reinterpret_cast<const float*>(unit + (e >> 2) * plane_bytes)[e & 3];
    };
    const int w0 = WT == 2 ? 0 : wave;
    const char* const xb = ldsX + (wc + (lane & 31)) * 16;
#pragma unroll 1
    for (int part = w0; part < (WT == 2 ? 4 : w0 + 1); ++part) {
        const int fl = wf + 8 * part + 4 * (lane >> 5);
        float sum[9][4] = {};
        for (int64_t t = t0; t < t1; ++t) {
            const int rt = int(t / gtiles), grp0 = int(t - int64_t(rt) * gtiles) * GT;
            __syncthreads();
            stage(g, f0, cout, rt * RT, grp0, GT, last + 1, ldsG, dy_plane);
            stage(x, c0, cin, rt * RT - 1, grp0 - uo, U, (RT + 2) * U, ldsX, x_plane);
            __syncthreads();
#pragma unroll 1
            for (int u = 0; u <= last; ++u) {
                const int r = quot(u, gt_m), grp = u - r * GT, R = rt * RT + r;
                const int im = R / (H + 1), i = R - im * (H + 1) - 1, j0 = 8 * (grp0 + grp);
                if (im >= n || i < 0 || j0 >= W) continue;
                const int cols = W - j0 < 8 ? W - j0 : 8;
                const bool left = j0 > 0, right = j0 + 8 < W;
                float gv[4][8];
#pragma unroll
                for (int f = 0; f < 4; ++f) columns(ldsG + (u * T + fl + f) * 16, dy_plane, gv[f]);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (i + q < 1 || i + q > H) continue;        // the row i + q - 1
                    const char* const xu = xb + ((r + q) * U + grp + uo) * T * 16;
                    float xv[10];                                // columns j0 - 1 ...
                    columns(xu, x_plane, xv + 1);
                    xv[0] = left ? column(xu - T * 16, x_plane, 7) : 0.f;
                    xv[9] = right ? column(xu + T * 16, x_plane, 0) : 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        if (e >= cols) break;
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            if (e > 0 || left) sum[3 * q][f] = fmaf(gv[f][e], xv[e], sum[3 * q][f]);
                            sum[3 * q + 1][f] = fmaf(gv[f][e], xv[e + 1], sum[3 * q + 1][f]);
                            if (e + 1 < cols || right) sum[3 * q + 2][f] = fmaf(gv[f][e], xv[e + 2], sum[3 * q + 2][f]);
                        }
                    }
                }
            }
        }
        const int c = c0 + wc + (lane & 31);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if (c < cin && f0 + fl + f < cout) dst[(int64_t(f0 + fl + f) * 9 + q) * cin + c] = sum[q][f];
    }
}

template <int DT, int WT>
__global__ __launch_bounds__(256, 2) void k_wgrad_mfma(
    const typename Elt<DT>::T* __restrict__ x, const typename Elt<DT>::T* __restrict__ g, int n, int cin, int H,
    int W, int cout, DenseWPlan pl, float* __restrict__ out) {
    constexpr int NP = DT == DT_F32 ? 3 : 1, T = 32 * WT;
    constexpr int NS = WT == 2 ? 2 : 8;                  // units in flight: one per half-wave of the same tile
    extern __shared__ __align__(16) char lds[];
    __shared__ Sizes sizes;
    if (threadIdx.x == 0) {
        sizes.n = n, sizes.cin = cin, sizes.H = H, sizes.W = W, sizes.cout = cout;
        sizes.RT = pl.RT, sizes.GT = pl.GT, sizes.DU = pl.DU, sizes.U = pl.U, sizes.gtiles = pl.gtiles, sizes.KS = pl.KS;
        sizes.tiles = pl.tiles, sizes.gt_m = pl.gt_m;
    }
    const int GT = pl.GT, U = pl.U, uo = U > GT ? 1 : 0;
    const int dy_plane = pl.DU * T * 16, x_plane = (pl.RT + 2) * U * T * 16;
    char* const ldsG = lds;
    char* const ldsX = lds + NP * dy_plane;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int f0 = blockIdx.x * T, c0 = blockIdx.y * T, ks = blockIdx.z;
    const int64_t t0 = pl.tiles * ks / pl.KS, t1 = pl.tiles * (ks + 1) / pl.KS;
    const int plane = H * W;
    const int64_t g_total = int64_t(n) * cout * plane, x_total = int64_t(n) * cin * plane;

    us2 top = {0, 0};                                    // the largest magnitudes of fp32 values, as bf16
    using E = typename Elt<DT>::T;
    auto stage = [&](const E* p, int64_t total, int ch0, int chs, int row0, int grp0, int per, uint32_t per_m,
                     int live, int units, char* dst, int dst_plane) {
        constexpr int NB = 4;
        // image and row of padded row row0 (-1: the row before the first image)
        const int im0 = row0 < 0 ? -1 : row0 / (H + 1), i0 = row0 - im0 * (H + 1);
#pragma unroll
        for (int h = 0; h < WT; ++h) {
            const int ch = (tid & 7) + 8 * (tid >> 6) + 32 * h;
            for (int u0 = (tid >> 3) & 7; u0 < units; u0 += 8 * NB) {
                Raw<DT> raw[NB];
                int left[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const int u = u0 + 8 * k, r = quot(u, per_m), grp = grp0 + u - r * per;
                    const int d = quot(i0 + r, pl.h_m), im = im0 + d, i = i0 + r - d * (H + 1) - 1;
                    const bool in = u < live && im >= 0 && i >= 0 && im < n && ch0 + ch < chs && grp >= 0 && 8 * grp < W;
                    left[k] = in ? W - 8 * grp : 0;
                    const int64_t at = in ? (int64_t(im) * chs + ch0 + ch) * plane + i * W + 8 * grp : 0;
                    if (at + 8 <= total) {
                        __builtin_memcpy(raw[k].w, p + at, 8 * sizeof(E));
                    } else {                             // the end of the tensor
                        E one[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) one[e] = at + e < total ? p[at + e] : E(0);
                        __builtin_memcpy(raw[k].w, one, sizeof one);
                    }
                }
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const int u = u0 + 8 * k;
                    if (u >= units) continue;
                    u4 parts[NP];
                    finish_unit<DT>(raw[k], left[k], parts, top);
#pragma unroll
                    for (int s = 0; s < NP; ++s)
                        *reinterpret_cast<u4*>(dst + s * dst_plane + (u * T + ch) * 16) = parts[s];
                }
            }
        }
    };

    // this half-wave's filters, channels and units
    const int wf = WT == 2 ? (wave & 1) * 32 : 0, wc = WT == 2 ? (wave >> 1) * 32 : 0;
    const int stream = WT == 2 ? lane >> 5 : wave * 2 + (lane >> 5);
    const int steps = pl.DU / NS, last = pl.RT * GT - 1;
    f16v acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;

    // The matrix cores' sums lean to one side a little (measured: the error of
    // a long sum grew with its length, 7e-7 at 10^5 pixels).  So CH steps are
    // summed from zero, every other time of -dy, and added to or subtracted
    // from the accumulator: 1.5e-7 there, as with fp32 multiply-adds
    constexpr int CH = DT == DT_F32 ? 1 : 2;
    float sign = 1.f;
    for (int64_t t = t0; t < t1; ++t) {
        const int rt = int(t / pl.gtiles), grp0 = int(t - int64_t(rt) * pl.gtiles) * GT, row0 = rt * pl.RT;
        if (t > t0) __syncthreads();
        stage(g, g_total, f0, cout, row0, grp0, GT, pl.gt_m, last + 1, pl.DU, ldsG, dy_plane);
        stage(x, x_total, c0, cin, row0 - 1, grp0 - uo, U, pl.u_m, (pl.RT + 2) * U, (pl.RT + 2) * U, ldsX, x_plane);
        __syncthreads();
        for (int k0 = 0; k0 < steps; k0 += CH) {
            sign = -sign;
            const uint32_t flip = sign < 0.f ? 0x80008000u : 0u;
            u4 av[CH][NP];
            const char* xp[CH];
            bool lok[CH], hok[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const bool more = k0 + k < steps;
                const int u = (more ? k0 + k : k0) * NS + stream, ux = u < last ? u : last;
                const int r = quot(ux, pl.gt_m), grp = ux - r * GT;
                lok[k] = uo || grp > 0;
                hok[k] = uo || grp + 1 < GT;
                xp[k] = ldsX + ((r * U + grp + uo) * T + wc + (lane & 31)) * 16;
#pragma unroll
                for (int s = 0; s < NP; ++s) {
                    const u4 v = *reinterpret_cast<const u4*>(ldsG + s * dy_plane + (u * T + wf + (lane & 31)) * 16);
                    av[k][s] = more ? v ^ flip : u4{0, 0, 0, 0};
                }
            }
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                u4 bv[CH][3][NP];
#pragma unroll
                for (int k = 0; k < CH; ++k)
#pragma unroll
                    for (int s = 0; s < NP; ++s) {
                        const char* const at = xp[k] + s * x_plane + r * U * T * 16;
                        const u4 c = *reinterpret_cast<const u4*>(at);
                        uint32_t lo = *reinterpret_cast<const uint32_t*>(at - T * 16 + 12);
                        uint32_t hi = *reinterpret_cast<const uint32_t*>(at + T * 16);
                        lo = lok[k] ? lo : 0;
                        hi = hok[k] ? hi : 0;
                        const uint32_t w0 = c.x, w1 = c.y, w2 = c.z, w3 = c.w;
                        const uint32_t m1 = __builtin_amdgcn_alignbit(w1, w0, 16),
                                       m2 = __builtin_amdgcn_alignbit(w2, w1, 16),
                                       m3 = __builtin_amdgcn_alignbit(w3, w2, 16);
                        bv[k][0][s] = u4{__builtin_amdgcn_alignbit(w0, lo, 16), m1, m2, m3};
                        bv[k][1][s] = c;
                        bv[k][2][s] = u4{m1, m2, m3, __builtin_amdgcn_alignbit(hi, w3, 16)};
                    }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    f16v part;
                    if constexpr (DT == DT_F16) {
                        part = mfma(av[0][0], bv[0][q][0], f16v{}, IntC<DT>{});
#pragma unroll
                        for (int k = 1; k < CH; ++k) part = mfma(av[k][0], bv[k][q][0], part, IntC<DT>{});
                    } else {
                        constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
                        part = mfma(av[0][0], bv[0][q][2], f16v{}, IntC<DT>{});
#pragma unroll
                        for (int o = 1; o < 6; ++o) part = mfma(av[0][ia[o]], bv[0][q][ib[o]], part, IntC<DT>{});
                    }
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[3 * r + q][e] = fmaf(part[e], sign, acc[3 * r + q][e]);
                }
            }
        }
    }

    // the four waves' sums of a 32 x 32 block: wave o finishes taps o and 4 + o
    // and a quarter of tap 8, adding the others' in a fixed order
    auto owns = [&](int q, int r) { return WT == 2 || wave == (q < 8 ? q & 3 : r >> 2); };
    if constexpr (WT == 1) {
        float* const red = reinterpret_cast<float*>(lds) + lane;
#pragma unroll
        for (int ph = 0; ph < 3; ++ph) {
            __syncthreads();
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                if (wave == o) continue;
                const int slot = o * 3 + (wave < o ? wave : wave - 1);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    if (ph < 2) red[(slot * 16 + r) * 64] = acc[4 * ph + o][r];
                    else if (r / 4 == o) red[(slot * 4 + r % 4) * 64] = acc[8][r];
                }
            }
            __syncthreads();
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                if (wave != o) continue;
#pragma unroll
                for (int s = 0; s < 3; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        if (ph < 2) acc[4 * ph + o][r] += red[((o * 3 + s) * 16 + r) * 64];
                        else if (r / 4 == o) acc[8][r] += red[((o * 3 + s) * 4 + r % 4) * 64];
                    }
            }
        }
    }
    bool again = top.x >= 0x4e00 || top.y >= 0x4e00;     // 2^29
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (owns(q, r)) {
                const float v = acc[q][r];               // a bit cast of the element itself gives element 0
                const uint32_t u = __builtin_bit_cast(uint32_t, v) << 1;
                // 2 * 0x7f800000, and 2 * the bits of 2^-80 less one
                again |= u >= 0xff000000u || (DT == DT_F32 && u - 1 < 2u * 0x17800000u - 1);
            }
    float* const dst = out + int64_t(ks) * cout * cin * 9;
    // asked before the store: a barrier after it would wait for it
    const int redo = __builtin_amdgcn_readfirstlane(__syncthreads_or(int(again)));
    // D[i][j] of tap q: filter f0 + wf + i, channel c0 + wc + j
    const int c = c0 + wc + (lane & 31);
    if (c < cin) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int f = f0 + wf + 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
            if (f >= cout) continue;
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if (owns(q, r)) dst[(int64_t(f) * 9 + q) * cin + c] = acc[q][r];
        }
    }
    // over what was just written, so that the sums need no registers any more
    if (redo)
        sum_again<DT, WT>(x, g, sizes, out, lds);
}

// dw[f][c][q] = the sum of the KS slots part[s][f][q][c] in a fixed order:
// four chains (s % 4), then their sum.
__global__ __launch_bounds__(256) void k_sum_slots(const float* __restrict__ part, int KS, int cin, int64_t n,
                                                   float* __restrict__ dw) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= n) return;
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s + 4 <= KS; s += 4)
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] += part[(s + t) * n + e];
    for (; s < KS; ++s) a[0] += part[s * n + e];
    const int64_t fq = e / cin, f = fq / 9;
    dw[(f * cin + (e - fq * cin)) * 9 + (fq - 9 * f)] = (a[0] + a[1]) + (a[2] + a[3]);
}

// The masked weight gradient (Sec. 3.3) from the KS partial sums of a dense
// one, added in a
// fixed order: for stored kernel k of reordered filter i
// (original filter perm[i], channel cin_idx[k], library pattern pat_id[k]),
// dv[4k + j] = sum over s of part[s][perm[i]][q_j][cin_idx[k]], q_j the j-th
// kept position of the pattern in ascending order -- the order of the stored
// weights.  One value per lane, one block per 64 kernels of a reordered
// filter.  A malformed channel or pattern index gives zeros, a malformed
// filter index reads filter 0.
__global__ __launch_bounds__(256) void k_gather_masked(const float* __restrict__ part, int KS,
                                                       const int32_t* __restrict__ perm,
                                                       const int32_t* __restrict__ filter_ptr,
                                                       const int32_t* __restrict__ cin_idx,
                                                       const uint8_t* __restrict__ pat_id, PatTable tab, int cin,
                                                       int cout, float* __restrict__ dv) {
    const int i = blockIdx.x;
    const int f = perm[i] >= 0 && perm[i] < cout ? perm[i] : 0;
    const int k0 = filter_ptr[i], k1 = filter_ptr[i + 1];
    const int64_t slot = int64_t(cout) * cin * 9;
    for (int k = k0 + int(blockIdx.y * 64 + threadIdx.x / 4); k < k1; k += 64 * gridDim.y) {
        const int c = cin_idx[k], p = pat_id[k], j = threadIdx.x & 3;
        uint32_t mask = (c >= 0 && c < cin && p < tab.m) ? tab.mask[p] : 0u;
        for (int t = 0; t < j; ++t) mask &= mask - 1;
        float v = 0.f;
        if (mask) {
            const float* src = part + (int64_t(f) * 9 + __builtin_ctz(mask)) * cin + c;
            float a[4] = {0.f, 0.f, 0.f, 0.f};
            int s = 0;
            for (; s + 4 <= KS; s += 4)
#pragma unroll
                for (int t = 0; t < 4; ++t) a[t] += src[(s + t) * slot];
            for (; s < KS; ++s) a[0] += src[s * slot];
            v = (a[0] + a[1]) + (a[2] + a[3]);
        }
        dv[int64_t(k) * 4 + j] = v;
    }
}

}  // namespace

// Layers of at least 16 input channels.
bool dense_wgrad_mfma_plan(int n, int cin, int cout, int h, int w, int dtype, DenseWPlan* p) {
    if (cin < 16 || n <= 0 || cout <= 0 || h <= 0 || w <= 0) return false;
    DenseWPlan q{};
    const int np = dtype == DT_F32 ? 3 : 1;
    const int64_t big = int64_t((cout + 63) / 64) * ((cin + 63) / 64);
    // 64 x 64 tiles only where those alone give every CU a quarter of a block,
    // and (fp32, whose three parts fill the LDS) where a row is one group of
    // columns: 512 -> 512 @ 4x4 b256, fp16: 120 us, against 138 in 32 x 32
    q.WT = big >= 64 && (dtype == DT_F16 ? int64_t(n) * h * w >= 4096 : w <= 8) ? 2 : 1;
    const int T = 32 * q.WT, NS = q.WT == 2 ? 2 : 8;
    q.fb = (cout + T - 1) / T;
    q.cb = (cin + T - 1) / T;
    const int64_t fc = int64_t(q.fb) * q.cb, rows = int64_t(n) * (h + 1);
    if (rows + 64 > 0x7fffffff || h >= 65000) return false;
    // LDS of a tile: the gradient's units, padded to whole steps, the input's
    // with the rows above and below (and a group on each side where a row
    // takes several tiles), and one unit past the end
    const int64_t unit = int64_t(T) * 16 * np, budget = 80 * 1024 - 1024;
    auto bytes = [&](int64_t rt, int64_t gt, int64_t u) {
        return ((rt * gt + NS - 1) / NS * NS + (rt + 2) * u) * unit + T * 16;
    };
    const int G = (w + 7) / 8;
    int least = G > 4 ? 4 : 8;                           // rows that a tile of whole rows should have
    q.gtiles = 1;
    q.GT = q.U = G;
    while (least > 4 && bytes(least, G, G) > budget) --least;
    if (bytes(least, G, G) > budget) {
        for (q.gtiles = 2;; ++q.gtiles) {
            q.GT = (G + q.gtiles - 1) / q.gtiles;
            q.U = q.GT + 2;
            if (bytes(4, q.GT, q.U) <= budget || q.GT == 1) break;
        }
        q.gtiles = (G + q.GT - 1) / q.GT;
    }
    int64_t rt = rows < 512 ? rows : 512;
    while (rt > 1 && bytes(rt, q.GT, q.U) > budget) --rt;
    // two blocks per CU, each with at least 256 pixels
    int64_t ks = 512 / fc;
    const int64_t px = int64_t(n) * h * w;
    if (ks > px / 256) ks = px / 256;
    if (ks > kMaxKS) ks = kMaxKS;
    if (ks < 1) ks = 1;
    // rows of a tile: the fewest clocks of the block with the most tiles, with
    // about 3000 of a tile's barriers and latency, and per half-wave unit of
    // MFMAs and of staging what these take on a shared SIMD
    {
        const int64_t step = dtype == DT_F32 ? 3500 : 1200, copy = dtype == DT_F32 ? 700 : 400;
        int64_t best = rt, least_cost = INT64_MAX;
        for (int64_t r = rt; r >= 1; --r) {
            const int64_t tiles = (rows + r - 1) / r * q.gtiles;
            const int64_t cost = (tiles + ks - 1) / ks * (3000 + (r * q.GT + NS - 1) / NS * step +
                                                         (r * q.GT + (r + 2) * q.U) * q.WT / 8 * copy);
            if (cost < least_cost) least_cost = cost, best = r;
        }
        rt = best;
        q.clocks = least_cost;
    }
    q.RT = int(rt);
    q.DU = int((rt * q.GT + NS - 1) / NS * NS);
    q.tiles = (rows + rt - 1) / rt * q.gtiles;
    if (ks > q.tiles) ks = q.tiles;
    q.KS = int(ks);
    auto inv = [](int d) { return uint32_t(((uint64_t(1) << 32) + d - 1) / d); };
    q.gt_m = q.GT == 1 ? 0xffffffffu : inv(q.GT);
    q.u_m = q.U == 1 ? 0xffffffffu : inv(q.U);
    q.h_m = inv(h + 1);
    const int64_t red = q.WT == 1 ? 4 * 3 * 16 * 64 * 4 : 0, st = bytes(rt, q.GT, q.U);
    q.lds = int(st > red ? st : red);
    if (p) *p = q;
    return true;
}

size_t dense_wgrad_mfma_workspace(const DenseWPlan& p, int cin, int cout) {
    return size_t(p.KS) * size_t(cout) * size_t(cin) * 9 * sizeof(float);
}

hipError_t launch_dense_wgrad_mfma(const DenseWPlan& p, int dtype, const void* x, const void* g, int n, int cin,
                                   int h, int w, int cout, float* dst, hipStream_t stream) {
    const dim3 grid(unsigned(p.fb), unsigned(p.cb), unsigned(p.KS));
    auto go = [&](auto dt, auto wt) {
        constexpr int DT = decltype(dt)::value, WT = decltype(wt)::value;
        using T = typename Elt<DT>::T;
        hipLaunchKernelGGL((k_wgrad_mfma<DT, WT>), grid, dim3(256), unsigned(p.lds), stream, static_cast<const T*>(x),
                           static_cast<const T*>(g), n, cin, h, w, cout, p, dst);
    };
    if (dtype == DT_F16)
        p.WT == 2 ? go(IntC<DT_F16>{}, IntC<2>{}) : go(IntC<DT_F16>{}, IntC<1>{});
    else
        p.WT == 2 ? go(IntC<DT_F32>{}, IntC<2>{}) : go(IntC<DT_F32>{}, IntC<1>{});
    return hipGetLastError();
}

hipError_t launch_sum_slots(const DenseWPlan& p, const float* part, int cin, int cout, float* dw,
                            hipStream_t stream) {
    const int64_t n = int64_t(cout) * cin * 9;
    hipLaunchKernelGGL(k_sum_slots, dim3(unsigned((n + 255) / 256)), dim3(256), 0, stream, part, p.KS, cin, n, dw);
    return hipGetLastError();
}

hipError_t launch_gather_masked(const PatTable& tab, const PackedView& pk, int cout, int cin, int64_t keep,
                                const float* part, int KS, float* dv, hipStream_t stream) {
    const int64_t per = (keep + cout - 1) / cout;        // kernels of a filter, about
    const unsigned gy = unsigned(per < 64 ? 1 : per / 64 > 64 ? 64 : per / 64);
    hipLaunchKernelGGL(k_gather_masked, dim3(unsigned(cout), gy), dim3(256), 0, stream, part, KS, pk.filter_perm,
                       pk.filter_ptr, pk.cin_idx, pk.pat_id, tab, cin, cout, dv);
    return hipGetLastError();
}

}  // namespace psc
