// fp32 3x3 convolutions on the 16-bit matrix cores: the dense layer of the
// ADMM loop (Sec. 4.3), and pattern-sparse calls (Sec. 4.1 Eq. 1) on which the
// vector kernels are slow (stride 2, odd widths).
//
// Every fp32 value is split into three bf16 parts, a = a1 + a2 + a3, each the
// rounding of what the ones before leave (24 bits: the sum is exact).  Of the
// nine products a_i b_j the six with i + j <= 4 are taken, by
// v_mfma_f32_32x32x16_bf16; what is dropped is below 2^-24 of a product
// (|a2| <= 2^-8 |a|, |a3| <= 2^-17 |a|; one rounding of fp32).  Six of those
// MFMAs cost 0.38 of the fp32 MFMAs of the same product.  The six products of 16
// channels at one tap are summed from the smallest up, from zero, every other
// time of -w; only that sum meets the accumulator (one rounding per 16 channels
// and tap, and a lean of the matrix cores' sums to one side cancels).
//
// The layout is that of the fp16 kernel: k_split_* write the weights of 64
// filters x 16 channels as three planes in LDS order, and a block of 8 waves
// owns 64 filters x NT pixels, staging the three planes of its input rows per
// 16 channels: 9 KB of LDS reads for the 12 MFMAs of a wave and tap (NT = 256).
// Counters (stride-2 entries, b256): MFMAs busy 24 to 28 % of the time, HBM 1.8
// TB/s, 1.8 to 2.9 conflict clocks per active LDS clock; the rest is the chain of
// stages between barriers.
//
// Range.  Parts are whole down to 2^-133 (subnormals are kept): a value of 2^-110
// or more is exactly the sum of its parts, a smaller one within 2^-134.  With the
// other factors below 2^19, n products are so within n 2^-115 of those of fp32,
// 2^-25 n of a sum of 2^-90.  A block computes its outputs again with fp32
// multiply-adds of the kept weights if a sum is not finite, or nonzero below
// 2^-90, or if inputs below 2^-110 meet weights of 2^19 or more or the other way
// round: k_split_* write what the weights are, and the inputs are looked at only
// where it matters (weights outside 2^-110 .. 2^19).
//
// Measured (us a call, fp32 MFMA first): dense 64 @ 32x32 b32 42 -> 22,
// 128 @ 28x28 b32 128 -> 64, 256 @ 14x14 b32 147 -> 60; error against 64 bits
// 3.9e-7 -> 1.1e-7 on the first.  The dispatch rule has the sparse calls.
#include "conv_mfma.h"

namespace psc {
namespace {
using namespace cm;

constexpr int kC = 16;                          // channels of a stage
constexpr int kQ = kC / 8;
constexpr int kT = 512;                         // threads
constexpr int kAU = 3 * 9 * kQ * kF;            // 16-byte units of a weight tile
constexpr int kAJ = (kAU + kT - 1) / kT;

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Eight values as three units of bf16 parts.
__device__ __forceinline__ void split8(const float (&v)[8], u4 (&o)[3]) {
    uint32_t w[3][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f2 r = {v[2 * k], v[2 * k + 1]};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            w[s][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, b2));
            r.x -= __builtin_bit_cast(float, w[s][k] << 16);
            r.y -= __builtin_bit_cast(float, w[s][k] & 0xffff0000u);
        }
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) o[s] = u4{w[s][0], w[s][1], w[s][2], w[s][3]};
}

// The smallest nonzero and the largest magnitude of some values, as twice their
// bits (less one, so that zero is the largest).
struct Range {
    uint32_t lo = ~0u, hi = 0;
    __device__ __forceinline__ void add(float v) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v) << 1;
        lo = u - 1 < lo ? u - 1 : lo;
        hi = u > hi ? u : hi;
    }
    // some below 2^-110: 1; some of 2^19 or more: 2
    __device__ __forceinline__ uint32_t bits() const {
        return (lo < 2u * 0x08800000u - 1 ? 1u : 0u) | (hi >= 2u * 0x49000000u ? 2u : 0u);
    }
};

// The range of a wave's weights to its word of `flags`; at most kFlags words for
// each 64 filters x 16 channels.  Waves write and read by themselves: a
// reduction over the block took 4 us of 90 (64->128 @ 32x32, stride 2, b256).
constexpr int kFlags = 64;
__device__ __forceinline__ uint32_t wave_or(uint32_t bits) {
    return (__ballot(bits & 1) ? 1u : 0u) | (__ballot(bits & 2) ? 2u : 0u);
}
__device__ __forceinline__ void put_range(const Range& range, uint32_t* block) {
    const uint32_t r = wave_or(range.bits());
    if ((threadIdx.x & 63) == 0) block[threadIdx.x >> 6] = r;
}

// The weight tiles wt[f / 64][c / 16][part][tap][(c / 8) % 2][f % 64][c % 8],
// zero past cin and cout.
__device__ __forceinline__ void put_unit(u4* wt, int nst, int f, int c8, int q, const float (&v)[8]) {
    u4 o[3];
    split8(v, o);
#pragma unroll
    for (int s = 0; s < 3; ++s)
        wt[(((int64_t(f / kF) * nst + c8 / kQ) * 3 + s) * 9 + q) * (kQ * kF) + (c8 % kQ) * kF + f % kF] = o[s];
}

// Dense weights w[f][c][9]: one unit (f, 8 channels, tap) per thread, 64
// filters per blockIdx.y.
__global__ __launch_bounds__(256) void k_split_dense(const float* __restrict__ w, int cin, int cout, int nst,
                                                     u4* __restrict__ wt, uint32_t* __restrict__ flags) {
    const int per = nst * kQ * 9, e = int(blockIdx.x * 256 + threadIdx.x);
    const int fl = e / per, f = int(blockIdx.y) * kF + fl, u = e - fl * per, c8 = u / 9, q = u - 9 * c8;
    Range range;
    if (fl < kF) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int c = 8 * c8 + k;
            v[k] = f < cout && c < cin ? w[(int64_t(f) * cin + c) * 9 + q] : 0.f;
            range.add(v[k]);
        }
        put_unit(wt, nst, f, c8, q, v);
    }
    put_range(range, flags + int64_t(blockIdx.y) * (kFlags * nst) + blockIdx.x * 4);
}

// Compressed weights: 4 reordered filters x 128 channels per block, scattered
// through LDS.
constexpr int kDF = 4, kDC = 128;
__global__ __launch_bounds__(256) void k_split_packed(const int32_t* __restrict__ fptr,
                                                      const int32_t* __restrict__ cin_idx,
                                                      const uint8_t* __restrict__ pat_id,
                                                      const float* __restrict__ values, MGeo g, int nst,
                                                      u4* __restrict__ wt, uint32_t* __restrict__ flags) {
    __shared__ __align__(16) float t[kDF][9 * kDC];
    const int f0 = blockIdx.x * kDF, c0 = blockIdx.y * kDC;
    for (int e = threadIdx.x; e < kDF * 9 * kDC / 4; e += 256) reinterpret_cast<u4*>(t)[e] = u4{0, 0, 0, 0};
    __syncthreads();
    const int lane = threadIdx.x & 63, fl = threadIdx.x >> 6;
    if (f0 + fl < g.cout) {
        const int k0 = fptr[f0 + fl] > 0 ? fptr[f0 + fl] : 0;
        const int k1 = fptr[f0 + fl + 1] < g.keep ? fptr[f0 + fl + 1] : g.keep;
        // four kernels a lane in flight, weights with their indices
        for (int kb = k0; kb < k1; kb += 256) {
            int c[4], p[4];
            float v[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = kb + 64 * i + lane < k1 ? kb + 64 * i + lane : k0;
                c[i] = cin_idx[k] - c0;
                p[i] = pat_id[k];
                __builtin_memcpy(v[i], values + 4 * int64_t(k), 16);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kb + 64 * i + lane >= k1 || uint32_t(c[i]) >= uint32_t(kDC) || c0 + c[i] >= g.cin || p[i] >= g.m)
                    continue;
                const uint32_t tp = g.taps[p[i]];
#pragma unroll
                for (int j = 0; j < 4; ++j) t[fl][((tp >> (4 * j)) & 15) * kDC + c[i]] = v[i][j];
            }
        }
    }
    __syncthreads();
    Range range;
    for (int e = threadIdx.x; e < kDF * 9 * kDC / 8; e += 256) {
        const int f = e % kDF, u = e / kDF, cg = u % (kDC / 8), q = u / (kDC / 8);
        if (c0 / kC + cg / kQ >= nst) continue;
        float v[8];
        __builtin_memcpy(v, &t[f][q * kDC + cg * 8], 32);
#pragma unroll
        for (int k = 0; k < 8; ++k) range.add(v[k]);
        put_unit(wt, nst, f0 + f, c0 / 8 + cg, q, v);
    }
    put_range(range, flags + int64_t(f0 / kF) * (kFlags * nst) + (blockIdx.y * (kF / kDF) + f0 % kF / kDF) * 4);
}

struct Packed {                                  // null perm: dense weights in `values`
    const int32_t* perm;
    const int32_t* fptr;
    const int32_t* cin_idx;
    const uint8_t* pat_id;
    const float* values;
};

template <int NT, bool ALIGNED>
__global__ __launch_bounds__(kT, 2) void k_conv_split(const float* __restrict__ x, const u4* __restrict__ wtiles,
                                                      const uint32_t* __restrict__ flags, int nflags, Packed pk,
                                                      const float* __restrict__ bias, MGeo g, int nst,
                                                      float* __restrict__ y) {
    // 8 waves: 2 x 4 of 32 filters x NT / 4 pixels
    constexpr int NI = NT / 128;
    extern __shared__ __align__(16) char lds[];
    char* const ldsA = lds;                              // kAU units
    char* const ldsX = lds + kAU * 16;                   // 3 planes of kQ * Lst units
    __shared__ int perm_s[kF];
    __shared__ float bias_s[kF];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // blocks go to the 8 XCDs in turn: an XCD takes consecutive tiles, pixels
    // first, so that its L2 holds few filters' weights
    const int per = (g.nblocks + 7) / 8;
    const int b = int(blockIdx.x % 8) * per + int(blockIdx.x / 8);
    if (b >= g.nblocks || int(blockIdx.x / 8) >= per) return;
    const int pts = g.ptiles * g.CT;
    const int ft = b / pts, pt = b - ft * pts;
    const int strip = pt / g.ptiles, o0 = (pt - strip * g.ptiles) * NT;
    const int j0 = strip * g.TW, f0 = ft * kF;
    const int plane = g.H * g.W, rowp = g.H + 1, per_img = g.OH * g.TW;
    uint32_t wrange = 0;                                 // loaded first: the values' latency covers it
    for (int e = lane; e < nflags; e += 64) wrange |= flags[int64_t(ft) * (kFlags * nst) + e];

    // padded row img * (H + 1) + i + 1 holds image row i
    auto prow = [&](int o, int& img, int& i, int& j) {
        img = o / per_img;
        const int r = o - img * per_img;
        i = r / g.TW;
        j = r - i * g.TW;
        return img * rowp + g.S * i + 1;
    };
    int img, i, j;
    const int olast = (o0 + NT < g.slots ? o0 + NT : g.slots) - 1;
    const int row_lo = prow(o0, img, i, j) - 1;
    const int rows = prow(olast, img, i, j) + 1 - row_lo + 1;

    int xbase[NI], ybase[NI];
    bool live[NI];
    const int wf = (wave & 1) * 32, wn = (wave >> 1) * (NT / 4);
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const int o = o0 + wn + 32 * t + (lane & 31);
        live[t] = o < g.slots;
        const int pr = prow(live[t] ? o : olast, img, i, j);
        live[t] = live[t] && j0 + j < g.OW;
        xbase[t] = ((pr - 1 - row_lo) * g.P + g.S * j + (lane >> 5) * g.Lst) * 16;
        ybase[t] = img * g.cout * g.OH * g.OW + i * g.OW + j0 + j;
    }

    // zero the X tile once: padding rows and columns are never written
    for (int e = tid; e < 3 * kQ * g.Lst; e += kT) *reinterpret_cast<u4*>(ldsX + e * 16) = u4{0, 0, 0, 0};
    if (tid < kF) {
        const int p = f0 + tid >= g.cout ? -1 : pk.perm ? pk.perm[f0 + tid] : f0 + tid;
        perm_s[tid] = p;
        bias_s[tid] = bias && p >= 0 ? bias[p] : 0.f;
    }

    // staging slot of this thread: 4 columns x 8 channels (the last vector of
    // a row ends with the row and may overlap the one before), and a halo
    // column of a strip
    const auto xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), int16_t(0), g.x_bytes, 0x00020000);
    uint32_t goff = 0x80000000u, hgoff = 0x80000000u;
    int loff = -1, hloff = -1;
    {
        const int tw = g.S * g.TW, nv = (tw + 3) / 4;
        const int cols = g.W - g.S * j0 < tw ? g.W - g.S * j0 : tw;      // at least 4
        const int v = tid % nv, r = (tid / nv) % rows, kq = tid / (nv * rows);
        const int gr = row_lo + r, im = gr / rowp, ir = gr - im * rowp - 1;
        const int rel = 4 * v < cols - 4 ? 4 * v : cols - 4;
        if (kq < kQ && ir >= 0 && im < g.n && 4 * v < cols) {
            goff = uint32_t((im * g.cin + 8 * kq) * plane + ir * g.W + g.S * j0 + rel) * 4u;
            loff = (kq * g.Lst + r * g.P + 1 + rel) * 16;
        }
    }
    const bool halo = g.CT > 1;
    if (halo && tid < kQ * rows * 2) {
        const int side = tid & 1, r = (tid >> 1) % rows, kq = (tid >> 1) / rows;
        const int gr = row_lo + r, im = gr / rowp, ir = gr - im * rowp - 1;
        const int col = side ? g.S * (j0 + g.TW) : g.S * j0 - 1;
        if (ir >= 0 && im < g.n && col >= 0 && col < g.W) {
            hgoff = uint32_t((im * g.cin + 8 * kq) * plane + ir * g.W + col) * 4u;
            hloff = (kq * g.Lst + r * g.P + (side ? g.P - 1 : 0)) * 16;
        }
    }
    const int xplane = kQ * g.Lst * 16;
    float xv[8][4], hv[8];
    u4 wv[kAJ];
    const u4* const wt = wtiles + int64_t(ft) * nst * kAU + tid;
    auto fetch = [&](int st) {
        // channels past cin read what follows (their weights are zero) or,
        // past x, zero
        const uint32_t so = uint32_t(st * kC * plane) * 4u, cs = uint32_t(plane) * 4u;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t vo = goff + (so + uint32_t(c) * cs);
            if constexpr (ALIGNED) {
                const u4 t = __builtin_amdgcn_raw_buffer_load_b128(xr, int(vo), 0, 0);
                __builtin_memcpy(xv[c], &t, 16);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) xv[c][k] = 0.f;
                if (vo + 16u <= uint32_t(g.x_bytes))
                    __builtin_memcpy(xv[c], reinterpret_cast<const char*>(x) + vo, 16);
            }
        }
        if (halo) {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                hv[c] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(xr, int(hgoff + (so + uint32_t(c) * cs)), 0, 0));
        }
#pragma unroll
        for (int e = 0; e < kAJ; ++e)
            if (tid + e * kT < kAU) wv[e] = wt[int64_t(st) * kAU + e * kT];
    };
    auto stage = [&]() {
        if (loff >= 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float v[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = xv[c][k];
                u4 o[3];
                split8(v, o);
#pragma unroll
                for (int s = 0; s < 3; ++s) *reinterpret_cast<u4*>(ldsX + s * xplane + loff + k * 16) = o[s];
            }
        }
        if (halo && hloff >= 0) {
            u4 o[3];
            split8(hv, o);
#pragma unroll
            for (int s = 0; s < 3; ++s) *reinterpret_cast<u4*>(ldsX + s * xplane + hloff) = o[s];
        }
#pragma unroll
        for (int e = 0; e < kAJ; ++e)
            if (tid + e * kT < kAU) *reinterpret_cast<u4*>(ldsA + (tid + e * kT) * 16) = wv[e];
    };

    f16v acc[NI];
#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    const char* const abase = ldsA + ((lane >> 5) * kF + wf + (lane & 31)) * 16;
    fetch(0);
    bool again = false;
    wrange = wave_or(wrange);
    if (wrange) {                                        // a look at the inputs
        Range range;
#pragma unroll 1
        for (int st = 0; st < nst; ++st) {
            fetch(st);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) range.add(loff >= 0 ? xv[c][k] : 0.f);
                range.add(halo && hloff >= 0 ? hv[c] : 0.f);
            }
        }
        const uint32_t x = range.bits();
        again = ((wrange & 1) && (x & 2)) || ((wrange & 2) && (x & 1));
        fetch(0);
    }
    __syncthreads();                                     // X zeroed
    for (int st = 0; st < nst; ++st) {
        stage();
        __syncthreads();
        if (st + 1 < nst) fetch(st + 1);                 // in flight during the MFMAs
        const char* xk = ldsX;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const bool neg = (st + q) & 1;
            const uint32_t flip = neg ? 0x80008000u : 0u;
            const float sign = neg ? -1.f : 1.f;
            u4 av[3];
#pragma unroll
            for (int s = 0; s < 3; ++s)
                av[s] = *reinterpret_cast<const u4*>(abase + (s * 9 + q) * (kQ * kF * 16)) ^ flip;
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                b8 bv[3];
#pragma unroll
                for (int s = 0; s < 3; ++s)
                    bv[s] = *reinterpret_cast<const b8*>(xk + s * xplane + xbase[t] + (q % 3) * 16);
                constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
                f16v part{};
#pragma unroll
                for (int o = 0; o < 6; ++o)
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, av[ia[o]]), bv[ib[o]], part,
                                                                   0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = fmaf(part[r], sign, acc[t][r]);
            }
            if (q % 3 == 2) xk += g.P * 16;
        }
        __syncthreads();
    }

#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = acc[t][r];                   // a bit cast of the element itself gives element 0
            const uint32_t u = __builtin_bit_cast(uint32_t, v) << 1;
            // 2 * 0x7f800000, and 2 * the bits of 2^-90 less one
            again |= u >= 0xff000000u || u - 1 < 2u * 0x12800000u - 1;
        }
    const int oplane = g.OH * g.OW;
    if (__syncthreads_or(int(again))) {
        for (int e = tid; e < kF * NT; e += kT) {
            const int f = e / NT, o = o0 + e % NT;
            if (f0 + f >= g.cout || o >= g.slots) continue;
            prow(o, img, i, j);
            if (j0 + j >= g.OW) continue;
            float s = 0.f;
            auto tap = [&](const float* xp, int q, float wgt) {
                const int ih = g.S * i + q / 3 - 1, iw = g.S * (j0 + j) + q % 3 - 1;
                if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) s = fmaf(wgt, xp[ih * g.W + iw], s);
            };
            if (pk.perm) {
                const int k1 = pk.fptr[f0 + f + 1] < g.keep ? pk.fptr[f0 + f + 1] : g.keep;
                for (int k = pk.fptr[f0 + f] > 0 ? pk.fptr[f0 + f] : 0; k < k1; ++k) {
                    const int c = pk.cin_idx[k], p = pk.pat_id[k];
                    if (uint32_t(c) >= uint32_t(g.cin) || p >= g.m) continue;
                    const uint32_t tp = g.taps[p];
                    for (int t = 0; t < 4; ++t)
                        tap(x + (int64_t(img) * g.cin + c) * plane, (tp >> (4 * t)) & 15, pk.values[4 * int64_t(k) + t]);
                }
            } else {
                for (int c = 0; c < g.cin; ++c)
                    for (int q = 0; q < 9; ++q)
                        tap(x + (int64_t(img) * g.cin + c) * plane, q, pk.values[(int64_t(f0 + f) * g.cin + c) * 9 + q]);
            }
            s += bias_s[f];
            if (g.relu) s = s > 0.f ? s : 0.f;
            y[(int64_t(img) * g.cout + perm_s[f]) * oplane + i * g.OW + j0 + j] = s;
        }
        return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int f = wf + 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
        if (f0 + f >= g.cout) continue;
        const float bv = bias_s[f];
        float* const yf = y + int64_t(perm_s[f]) * oplane;
#pragma unroll
        for (int t = 0; t < NI; ++t)
            if (live[t]) {
                float v = acc[t][r] + bv;
                if (g.relu) v = v > 0.f ? v : 0.f;
                yf[ybase[t]] = v;
            }
    }
}

// Host only.
bool tile_plan(const ConvArgs& a, int m, int NT, MPlan& p) {
    int64_t rows;
    // 32-bit byte offsets into x, and up to 24 channels past it
    if ((int64_t(a.n) * a.cin + 64) * a.h * a.w * 4 >= (int64_t(1) << 31)) return false;
    if (!geometry(a, m, NT, p, rows)) return false;
    const MGeo& g = p.g;
    if (kQ * rows * ((g.S * g.TW + 3) / 4) > kT || (g.CT > 1 && kQ * rows * 2 > kT)) return false;
    p.lds = size_t(kAU) * 16 + size_t(3 * kQ) * g.Lst * 16;
    return p.lds <= 158 * 1024;
}

// The larger tile where it still gives about a block per CU.
bool plan_split(const ConvArgs& a, int m, MPlan& p) {
    std::memset(&p, 0, sizeof p);
    if (tile_plan(a, m, 256, p) && p.g.nblocks >= 200) return true;
    return tile_plan(a, m, 128, p);
}

// The flags stand behind the tiles in the scratch.
uint32_t* flags_of(const ConvArgs& a) {
    const size_t tiles = size_t((a.cout + kF - 1) / kF) * size_t((a.cin + kC - 1) / kC) * kAU * 16;
    return reinterpret_cast<uint32_t*>(static_cast<char*>(a.ws) + tiles);
}

// After k_split_* of nflags waves for each 64 filters.
hipError_t launch(const MPlan& p, const Packed& pk, const ConvArgs& a, int nflags, hipStream_t s) {
    const u4* const wt = static_cast<const u4*>(a.ws);
    const uint32_t* const flags = flags_of(a);
    const int nst = (a.cin + kC - 1) / kC;
    const dim3 grid(unsigned((p.g.nblocks + 7) / 8 * 8));
    auto go = [&](auto nt, auto al) {
        hipLaunchKernelGGL((k_conv_split<decltype(nt)::value, decltype(al)::value != 0>), grid, dim3(kT), unsigned(p.lds),
                           s, static_cast<const float*>(a.x), wt, flags, nflags, pk, static_cast<const float*>(a.bias),
                           p.g, nst, static_cast<float*>(a.y));
    };
    if (p.NT == 256)
        p.aligned ? go(IntC<256>{}, IntC<1>{}) : go(IntC<256>{}, IntC<0>{});
    else
        p.aligned ? go(IntC<128>{}, IntC<1>{}) : go(IntC<128>{}, IntC<0>{});
    return hipGetLastError();
}

}  // namespace

size_t split_tiles_bytes(int cout, int cin) {
    return size_t((cout + kF - 1) / kF) * size_t((cin + kC - 1) / kC) * (kAU * 16 + kFlags * 4);
}

bool conv_split_takes(const PatTable& tab, const ConvArgs& a) {
    if (a.dtype != DT_F32 || a.pool || a.cin < 16 || a.cout < 32 || a.keep > 0x0fffffff) return false;
    // Against the vector kernels: those take about 7 us and, of nonzero
    // multiply-adds, 11 TFLOP/s at stride 2 (3 at odd widths), 16 on rows that
    // are no multiple of 4 columns (25 up to 16 columns) and 45 otherwise; this
    // path about 6 us (two launches) and the larger of 3.5 us per 16 channels
    // (one tile's chain of stages) and 700 TFLOP/s of its six bf16 products.
    // Measured both ways on 25 layers (us, vector first): stride 2 at batch 256
    // 64->128 @ 32x32 119, 86; 128->256 @ 16x16 97, 80; 256->512 @ 8x8 91, 77;
    // 64 @ 30x30 b32 51, 21; 64->128 @ 33x35 b32 91, 66; 64 @ 56x56 b32 all
    // kept 86, 68, at 40 % kept 47, 68.
    const double outs = double(a.n) * ((a.h - 1) / a.stride + 1) * ((a.w - 1) / a.stride + 1);
    const double rate = a.stride == 2 ? (a.w % 2 ? 3 : 11) : a.w % 4 == 0 ? 45 : a.w <= 16 ? 25 : 16;
    const double valu_us = 7.0 + 8.0 * outs * double(a.keep) / (rate * 1e6);
    const double padded = double((a.cin + 15) / 16 * 16) * ((a.cout + 63) / 64 * 64);
    const double dense_us = 6 * 18.0 * outs * padded / 700e6, chain_us = 3.5 * ((a.cin + kC - 1) / kC);
    if (1.1 * (6.0 + (dense_us > chain_us ? dense_us : chain_us)) > valu_us) return false;
    MPlan p;
    return plan_split(a, tab.m, p);
}

hipError_t launch_conv_split(const PatTable& tab, const PackedView& pk, const ConvArgs& a, hipStream_t s) {
    MPlan p;
    if (!a.ws || a.ws_bytes < split_tiles_bytes(a.cout, a.cin) || !conv_split_takes(tab, a) || !plan_split(a, tab.m, p))
        return hipErrorNotSupported;
    pack_taps(tab, p.g);
    const int nst = (a.cin + kC - 1) / kC;
    const dim3 grid(unsigned(p.g.ftiles * kF / kDF), unsigned((a.cin + kDC - 1) / kDC));
    hipLaunchKernelGGL(k_split_packed, grid, dim3(256), 0, s, pk.filter_ptr, pk.cin_idx, pk.pat_id,
                       static_cast<const float*>(pk.values), p.g, nst, static_cast<u4*>(a.ws), flags_of(a));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch(p, Packed{pk.filter_perm, pk.filter_ptr, pk.cin_idx, pk.pat_id, static_cast<const float*>(pk.values)},
                  a, int(grid.y) * (kF / kDF) * 4, s);
}

// Layers of at least 16 channels and 32 filters (half a block's); `ws` holds
// split_tiles_bytes bytes.
hipError_t launch_dense_split(const ConvArgs& a, const void* w, hipStream_t s) {
    MPlan p;
    if (a.dtype != DT_F32 || a.cin < 16 || a.cout < 32 || !a.ws || a.ws_bytes < split_tiles_bytes(a.cout, a.cin) ||
        !plan_split(a, 0, p))
        return hipErrorNotSupported;
    const int nst = (a.cin + kC - 1) / kC;
    const dim3 grid(unsigned((kF * nst * kQ * 9 + 255) / 256), unsigned(p.g.ftiles));
    hipLaunchKernelGGL(k_split_dense, grid, dim3(256), 0, s, static_cast<const float*>(w), a.cin, a.cout, nst,
                       static_cast<u4*>(a.ws), flags_of(a));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch(p, Packed{nullptr, nullptr, nullptr, nullptr, static_cast<const float*>(w)}, a, int(grid.x) * 4, s);
}

}  // namespace psc
