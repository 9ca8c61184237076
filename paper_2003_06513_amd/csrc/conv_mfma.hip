// The pattern-sparse 3x3 convolution (Sec. 4.1 Eq. 1) on the matrix cores,
// for fp16 calls of enough output pixels: an implicit GEMM with M = reordered
// filters, N = output pixels and K = (channel, tap), in two launches.
//   k_weight_tiles  decodes the compressed storage (Sec. 3.4) into dense tiles
//                   in the order in which the next kernel stages them,
//   k_conv_mfma     multiplies them.
//
// Why dense tiles of a sparse layer: a kept kernel is 4 taps of 9, so they
// cost 9 / (4 keep) times the multiply-adds (5.6 at keep 0.4), but
// v_mfma_f32_32x32x16_f16 does 16 times those of v_fmac_f32 a clock, and a
// staged input feeds all filters of the block.  The vector kernels are bound
// by the vector-memory path that brings each kernel's rows to the registers.
// Measured (fp16, 60 % dropped, us a call, vector kernel first):
// 512 @ 28x28 b64 866 -> 250, 512 @ 7x7 b32 42.5 -> 29.1, 256 @ 14x14 b32
// 36.1 -> 22.7, 128 @ 28x28 b32 48.0 -> 20.5, 64 @ 56x56 b32 49.4 -> 24.0.
// Decoding inside the convolution instead (each block scattering its filters'
// kernels into its weight tile) measured 342 on the first and 62 on the
// second: the scatter repeats for every pixel tile.
//
// A block owns kF filters x NT output pixels (consecutive in raster order
// over the images of a column strip).  Per stage, G groups of 4 waves take 32
// channels each from LDS:
//   X[c / 8][position][8]       the input rows the tile needs, channels innermost,
//   A[c / 32][tap][c / 8][filter][8]   the weights,
// both in 16-byte units that neighbouring lanes read from neighbouring
// addresses.  A tap is an offset of positions, so one X tile serves all nine.
// The next stage's values load into registers while the MFMAs of this one run.
// Counters (ResNet-50 layers, b32): MFMAs busy 12 to 16 % of the time, HBM 0.8 to
// 2 TB/s, 1.1 to 1.6 conflict clocks per active LDS clock: it is bound by its
// chain of stages, each a register round trip between two barriers with 4 KB of
// LDS reads for 4 MFMAs of a wave.
//
// Infinities and NaNs: the dense tile multiplies pruned weights (zero) by
// every staged input, which must not turn a non-finite input that no kept
// weight reads into NaN.  A block that staged one goes over its channels four
// times more, by the matrix cores again: for the sums, with 1 or -1 in its
// place; for the number of terms that are infinite or NaN; and twice for the
// signs of the infinite ones, from which the outputs that read one follow.  A
// kept weight that is zero is -0 in the tile, a pruned one 0.  Measured with one
// infinity in the input, and with all of it infinite (us a call; vector
// kernels, kept weights from memory one by one, here): 128 @ 28x28 b32 47, 1256,
// 100 and 47, 1445, 110; 512 @ 28x28 b64 882, 10867, 521 and 882, 62963, 2175.
//
// Layout of v_mfma_f32_32x32x16_f16: lane l supplies A[l % 32][8 (l / 32) + j]
// and B[8 (l / 32) + j][l % 32], j = 0..7; register r of the result holds
// D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
#include "conv_mfma.h"

namespace psc {
namespace {
using namespace cm;

constexpr int kKC = 32, kQ = kKC / 8;   // channels of a weight chunk and per four waves and stage

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// The weight tiles of a call, decoded from the compressed storage:
//   wt[f / 64][c / 32][tap][(c / 8) % 4][f % 64][c % 8],
// zero where pruned and past cin and cout, a kept zero as -0; f counts
// reordered filters.  A
// block owns 8 filters x 128 channels: each of its waves scans a filter's
// kernels, scatters the weights to LDS, and all write 16-byte units.
constexpr int kDF = 8, kDC = 128;

__global__ __launch_bounds__(512) void k_weight_tiles(const int32_t* __restrict__ fptr,
                                                      const int32_t* __restrict__ cin_idx,
                                                      const uint8_t* __restrict__ pat_id,
                                                      const uint16_t* __restrict__ values, MGeo g,
                                                      uint16_t* __restrict__ wt) {
    __shared__ __align__(16) uint16_t t[kDF][9 * kDC];
    const int f0 = blockIdx.x * kDF, c0 = blockIdx.y * kDC;
    for (int e = threadIdx.x; e < kDF * 9 * kDC / 8; e += 512) reinterpret_cast<u4*>(t)[e] = u4{0, 0, 0, 0};
    __syncthreads();
    const int lane = threadIdx.x & 63, fl = threadIdx.x >> 6;
    if (f0 + fl < g.cout) {
        const int k0 = fptr[f0 + fl] > 0 ? fptr[f0 + fl] : 0;
        const int k1 = fptr[f0 + fl + 1] < g.keep ? fptr[f0 + fl + 1] : g.keep;
        // four kernels a lane in flight, weights with their indices: one
        // memory latency where a filter keeps up to 256 kernels
        for (int kb = k0; kb < k1; kb += 256) {
            int c[4], p[4];
            uint32_t v[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = kb + 64 * j + lane < k1 ? kb + 64 * j + lane : k0;
                c[j] = cin_idx[k] - c0;
                p[j] = pat_id[k];
                __builtin_memcpy(v[j], values + 4 * int64_t(k), 8);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (kb + 64 * j + lane >= k1 || uint32_t(c[j]) >= uint32_t(kDC) || c0 + c[j] >= g.cin || p[j] >= g.m)
                    continue;
                const uint32_t tp = g.taps[p[j]];
                auto kept = [](uint32_t h) { return uint16_t(h & 0x7fffu ? h : 0x8000u); };
                t[fl][(tp & 15) * kDC + c[j]] = kept(v[j][0]);
                t[fl][((tp >> 4) & 15) * kDC + c[j]] = kept(v[j][0] >> 16);
                t[fl][((tp >> 8) & 15) * kDC + c[j]] = kept(v[j][1]);
                t[fl][(tp >> 12) * kDC + c[j]] = kept(v[j][1] >> 16);
            }
        }
    }
    __syncthreads();
    // unit (filter, tap, 8 channels): neighbouring lanes take the 8 filters
    const int nst = g.chunks;
    for (int e = threadIdx.x; e < kDF * 9 * kDC / 8; e += 512) {
        const int fl = e % kDF, u = e / kDF, cg = u % (kDC / 8), q = u / (kDC / 8);
        const int f = f0 + fl, st = c0 / kKC + cg / (kKC / 8);
        if (st >= nst) continue;
        const int64_t at = (((int64_t(f / kF) * nst + st) * 9 + q) * (kKC / 8) + cg % (kKC / 8)) * kF + f % kF;
        reinterpret_cast<u4*>(wt)[at] = *reinterpret_cast<const u4*>(&t[fl][q * kDC + cg * 8]);
    }
}

// Two fp16 values: all ones in each half whose bit 15 is set in t.
__device__ __forceinline__ uint32_t halves(uint32_t t) { return ((t & 0x80008000u) >> 15) * 0xffffu; }
__device__ __forceinline__ uint32_t not_finite(uint32_t w) { return halves((w & 0x7c007c00u) + 0x04000400u); }
__device__ __forceinline__ uint32_t signed_one(uint32_t w) { return (w & 0x80008000u) | 0x3c003c00u; }

// Inputs and weights as the sweeps multiply them.  0: the sums, a non-finite
// input as 1 or -1.  1: 1 for each non-finite input and kept weight (the number
// of such terms); 2: the sign of each infinite input and of each weight; 3:
// the same, times -2.  After 1 and 2 a sum is twice the +infinities plus the
// NaNs, after 3 twice the -infinities plus the NaNs.
__device__ __forceinline__ uint32_t sweep_x(uint32_t w, int sweep) {
    const uint32_t m = not_finite(w);
    if (sweep == 0) return (w & ~m) | (m & signed_one(w));
    if (sweep == 1) return m & 0x3c003c00u;
    const uint32_t inf = m & ~halves(((w & 0x03ff03ffu) + 0x03ff03ffu) << 5);
    return inf & (sweep == 2 ? signed_one(w) : signed_one(~w) + 0x04000400u);
}
__device__ __forceinline__ uint32_t sweep_w(uint32_t w, int sweep) {
    const uint32_t mag = w & 0x7fff7fffu, nonzero = mag + 0x7fff7fffu;
    if (sweep == 0) return w;
    if (sweep == 1) return halves(nonzero | w) & 0x3c003c00u;
    return halves(nonzero) & ~halves(mag + 0x03ff03ffu) & signed_one(w);
}

template <int NT, int G, bool ALIGNED, int MI>
__global__ __launch_bounds__(256 * G, 2) void k_conv_mfma(const uint16_t* __restrict__ x,
                                                          const uint16_t* __restrict__ wtiles,
                                                          const int32_t* __restrict__ perm,
                                                          const uint16_t* __restrict__ bias, MGeo g,
                                                          uint16_t* __restrict__ y) {
    constexpr int kThreads = 256 * G, KC = kKC * G, KQ = KC / 8;
    // four waves each take 32 channels of a stage: 256 pixels: 4 of 64 filters x 64 pixels; 128: 2 x 2 of 32 x 64;
    // 64: 2 x 2 of 32 x 32
    constexpr int WF = NT == 256 ? 1 : 2, WN = 4 / WF;
    constexpr int FI = kF / WF / 32, NI = NT / WN / 32;
    extern __shared__ __align__(16) char lds[];
    char* const ldsA = lds;                              // 9 * KQ * kF * 16 bytes
    char* const ldsX = lds + 9 * KQ * kF * 16;           // KQ * Lst * 16 bytes
    __shared__ int perm_s[kF];
    __shared__ float bias_s[kF];

    const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) & 3, grp = tid >> 8;
    // blocks go to the 8 XCDs in turn: an XCD takes consecutive tiles, pixels
    // first, so that its L2 holds few filters' weights (512 @ 7x7 b32: 34.2 us
    // with filters first, 29.8 so)
    const int per = (g.nblocks + 7) / 8;
    const int b = int(blockIdx.x % 8) * per + int(blockIdx.x / 8);
    if (b >= g.nblocks || int(blockIdx.x / 8) >= per) return;
    const int pts = g.ptiles * g.CT;
    const int ft = b / pts, pt = b - ft * pts;
    const int strip = pt / g.ptiles, o0 = (pt - strip * g.ptiles) * NT;
    const int j0 = strip * g.TW;                         // first output column of the strip
    const int f0 = ft * kF;
    const int plane = g.H * g.W, rowp = g.H + 1, per_img = g.OH * g.TW;

    // the tile's rows: padded row img * (H + 1) + i + 1 holds image row i
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

    // this lane's output pixels
    int xbase[NI], ybase[NI];
    bool live[NI];
    const int wf = (wave % WF) * (kF / WF), wn = (wave / WF) * (NT / WN);
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
    auto zero_x = [&]() {
        for (int e = tid; e < KQ * g.Lst; e += kThreads) *reinterpret_cast<u4*>(ldsX + e * 16) = u4{0, 0, 0, 0};
    };
    zero_x();
    if (tid < kF) {
        const int p = f0 + tid < g.cout ? perm[f0 + tid] : -1;
        perm_s[tid] = p;
        bias_s[tid] = bias && p >= 0 ? Elt<DT_F16>::load(bias, p) : 0.f;
    }

    // staging slots of this thread: 4 columns x 8 channels.  The last vector
    // of a row ends with the row (or the strip) and may overlap the one before
    const auto xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x), int16_t(0), g.x_bytes, 0x00020000);
    uint32_t goff[MI];
    int loff[MI];
    const int tw = g.S * g.TW, nv = (tw + 3) / 4, items = KQ * rows * nv;
    {
        const int cols = g.W - g.S * j0 < tw ? g.W - g.S * j0 : tw;      // at least 4
#pragma unroll
        for (int s = 0; s < MI; ++s) {
            const int e = tid + kThreads * s;
            goff[s] = 0x80000000u;
            loff[s] = -1;
            if (e < items) {
                const int v = e % nv, r = (e / nv) % rows, kq = e / (nv * rows);
                const int gr = row_lo + r, im = gr / rowp, ir = gr - im * rowp - 1;
                const int rel = 4 * v < cols - 4 ? 4 * v : cols - 4;
                if (ir >= 0 && im < g.n && 4 * v < cols) {
                    goff[s] = uint32_t((im * g.cin + 8 * kq) * plane + ir * g.W + g.S * j0 + rel) * 2u;
                    loff[s] = (kq * g.Lst + r * g.P + 1 + rel) * 16;
                }
            }
        }
    }
    // halo columns of a strip: one column x 8 channels
    const bool halo = g.CT > 1;
    uint32_t hgoff = 0x80000000u;
    int hloff = -1;
    if (halo && tid < KQ * rows * 2) {
        const int side = tid & 1, r = (tid >> 1) % rows, kq = (tid >> 1) / rows;
        const int gr = row_lo + r, im = gr / rowp, ir = gr - im * rowp - 1;
        const int col = side ? g.S * (j0 + g.TW) : g.S * j0 - 1;
        if (ir >= 0 && im < g.n && col >= 0 && col < g.W) {
            hgoff = uint32_t((im * g.cin + 8 * kq) * plane + ir * g.W + col) * 2u;
            hloff = (kq * g.Lst + r * g.P + (side ? g.P - 1 : 0)) * 16;
        }
    }
    u2 xv[MI][8];
    uint32_t hv[8];
    uint32_t bad = 0;
    const uint32_t cs = uint32_t(plane) * 2u;
    // channels past cin read what follows (their weights are zero) or, past
    // x, zero
    auto load = [&](uint32_t at, uint32_t so, u2 (&v)[8]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t vo = at + (so + uint32_t(c) * cs);
            if constexpr (ALIGNED) {
                v[c] = __builtin_amdgcn_raw_buffer_load_b64(xr, int(vo), 0, 0);
            } else {
                v[c] = u2{0, 0};
                if (vo + 8u <= uint32_t(g.x_bytes))
                    __builtin_memcpy(&v[c], reinterpret_cast<const char*>(x) + vo, 8);
            }
        }
    };
    auto load_halo = [&](uint32_t at, uint32_t so, uint32_t (&v)[8]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = __builtin_amdgcn_raw_buffer_load_b16(xr, int(at + (so + uint32_t(c) * cs)), 0, 0);
    };
    auto fetch = [&](int c0) {
#pragma unroll
        for (int s = 0; s < MI; ++s)
            if (kThreads * s < items) load(goff[s], uint32_t(c0) * cs, xv[s]);       // the same for the whole block
        if (halo) load_halo(hgoff, uint32_t(c0) * cs, hv);
    };
    // exponent all ones in either half sets bit 15 or 31
    auto test = [&](uint32_t w) {
        bad |= (w & 0x7c007c00u) + 0x04000400u;
        return w;
    };
    // 4 columns x 8 channels, and a halo column's 8, to LDS through `as`
    auto put = [&](int at, const u2 (&v)[8], auto as) {
        uint32_t w[2][8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            w[0][c] = as(v[c].x);
            w[1][c] = as(v[c].y);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            u4 o;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                o[c] = __builtin_amdgcn_perm(w[e / 2][2 * c + 1], w[e / 2][2 * c], e & 1 ? 0x07060302u : 0x05040100u);
            *reinterpret_cast<u4*>(ldsX + at + e * 16) = o;
        }
    };
    auto put_halo = [&](int at, const uint32_t (&v)[8], auto as) {
        u4 o;
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = as(__builtin_amdgcn_perm(v[2 * c + 1], v[2 * c], 0x05040100u));
        *reinterpret_cast<u4*>(ldsX + at) = o;
    };
    auto stage_x = [&]() {
#pragma unroll
        for (int s = 0; s < MI; ++s)
            if (loff[s] >= 0) put(loff[s], xv[s], test);
        if (halo && hloff >= 0) put_halo(hloff, hv, test);
    };

    // the stage's weight tile: 36 KiB in the LDS order, 9 x 16 bytes a thread
    constexpr int AJ = 9 * KQ * kF / kThreads;
    const int nst = g.chunks / G;
    const u4* const wt = reinterpret_cast<const u4*>(wtiles) + int64_t(ft) * nst * (AJ * kThreads) + tid;
    u4 wv[AJ];
    auto fetch_a = [&](int st) {
#pragma unroll
        for (int e = 0; e < AJ; ++e) wv[e] = wt[int64_t(st) * (AJ * kThreads) + e * kThreads];
    };
    auto stage_a = [&]() {
#pragma unroll
        for (int e = 0; e < AJ; ++e) *reinterpret_cast<u4*>(ldsA + (tid + e * kThreads) * 16) = wv[e];
    };

    f16v acc[FI][NI];
#pragma unroll
    for (int a = 0; a < FI; ++a)
#pragma unroll
        for (int t = 0; t < NI; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][t][r] = 0.f;

    const char* const abase = ldsA + (grp * 9 * kQ * kF + (lane >> 5) * kF + wf + (lane & 31)) * 16;
    const char* const xgrp = ldsX + grp * kQ * g.Lst * 16;
    auto mfma = [&](int ks) {                            // 16 channels, nine taps
        const char* xk = xgrp + 2 * ks * g.Lst * 16;
        const char* const ak = abase + 2 * ks * kF * 16;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                h8 av[FI], bv[NI];
#pragma unroll
                for (int a = 0; a < FI; ++a)
                    av[a] = *reinterpret_cast<const h8*>(ak + ((3 * r + s) * kQ * kF + 32 * a) * 16);
#pragma unroll
                for (int t = 0; t < NI; ++t) bv[t] = *reinterpret_cast<const h8*>(xk + xbase[t] + s * 16);
#pragma unroll
                for (int a = 0; a < FI; ++a)
#pragma unroll
                    for (int t = 0; t < NI; ++t)
                        acc[a][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[a], bv[t], acc[a][t], 0, 0, 0);
            }
            xk += g.P * 16;
        }
    };
    fetch(0);
    fetch_a(0);
    __syncthreads();                                     // X zeroed
    for (int c0 = 0; c0 < g.cin; c0 += KC) {
        stage_x();
        stage_a();
        __syncthreads();
        if (c0 + KC < g.cin) {                           // in flight during the MFMAs
            fetch(c0 + KC);
            fetch_a(c0 / KC + 1);
        }
#pragma unroll
        for (int ks = 0; ks < kKC / 16; ++ks) mfma(ks);
        __syncthreads();
    }

    // the second group's sums go to the first through LDS
    auto meet = [&]() {
        if constexpr (G == 2) {
            float* const red = reinterpret_cast<float*>(lds) + wave * (FI * NI * 1024) + lane;
#pragma unroll
            for (int a = 0; a < FI; ++a)
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (grp) red[((a * NI + t) * 16 + r) * 64] = acc[a][t][r];
            __syncthreads();
#pragma unroll
            for (int a = 0; a < FI; ++a)
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (!grp) acc[a][t][r] += red[((a * NI + t) * 16 + r) * 64];
        }
    };
    // each output of this lane: its number, filter, place
    const int oplane = g.OH * g.OW;
    auto outputs = [&](int lane, auto put) {
#pragma unroll
        for (int a = 0; a < FI; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int f = wf + 32 * a + 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
                if (f0 + f >= g.cout) continue;
                uint16_t* const yf = y + int64_t(perm_s[f]) * oplane;
                const float bv = bias_s[f];
#pragma unroll
                for (int t = 0; t < NI; ++t)
                    if (live[t]) put(a, t, r, bv, yf + ybase[t]);
            }
    };
    auto store = [&](int lane) {
        if (grp == 0)
            outputs(lane, [&](int a, int t, int r, float bv, uint16_t* to) {
                float v = acc[a][t][r] + bv;
                if (g.relu) v = v > 0.f ? v : 0.f;
                *to = Elt<DT_F16>::from_f(v);
            });
    };
    // asked before the store: a barrier after it would wait for it
    const int again = __builtin_amdgcn_readfirstlane(__syncthreads_or(int(bad & 0x80008000u)));
    meet();
    store(lane);
    if (!again) return;

    // the lane once more, so that nothing of the first store is kept for the
    // next (the registers are the hot loop's)
    auto again_lane = [&]() {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // the outputs of this lane whose sum is infinite above and below (NaN:
    // both), a bit each; by integers, so that no lane masks pile up
    constexpr int MW = (FI * NI + 1) / 2;
    uint32_t pos[MW] = {}, neg[MW] = {};
    auto mark = [&](auto add) {
#pragma unroll
        for (int a = 0; a < FI; ++a)
#pragma unroll
            for (int t = 0; t < NI; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float v = acc[a][t][r];
                    add(__builtin_bit_cast(uint32_t, v), (a * NI + t) / 2, ((a * NI + t) % 2) * 16 + r);
                }
    };
#pragma unroll 1
    for (int sweep = 0; sweep < 4; ++sweep) {
        if (sweep < 2) {
#pragma unroll
            for (int a = 0; a < FI; ++a)
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[a][t][r] = 0.f;
        }
        __syncthreads();
        zero_x();                                        // meet() may have used its place
#pragma unroll 1
        for (int c0 = 0; c0 < g.cin; c0 += KC) {
            __syncthreads();
            auto as = [&](uint32_t w) { return sweep_x(w, sweep); };
#pragma unroll
            for (int s = 0; s < MI; ++s) {
                u2 v[8];
                if (kThreads * s < items) load(goff[s], uint32_t(c0) * cs, v);
                if (loff[s] >= 0) put(loff[s], v, as);
            }
            if (halo) {
                uint32_t v[8];
                load_halo(hgoff, uint32_t(c0) * cs, v);
                if (hloff >= 0) put_halo(hloff, v, as);
            }
#pragma unroll
            for (int e = 0; e < AJ; ++e) {
                u4 v = wt[int64_t(c0 / KC) * (AJ * kThreads) + e * kThreads];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = sweep_w(v[k], sweep);
                *reinterpret_cast<u4*>(ldsA + (tid + e * kThreads) * 16) = v;
            }
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < kKC / 16; ++ks) mfma(ks);
        }
        if (sweep == 0) {
            __syncthreads();
            meet();
            mark([&](uint32_t u, int i, int k) {
                const uint32_t mag = u & 0x7fffffffu, inf = (mag + 0x00800000u) >> 31, nan = (mag + 0x007fffffu) >> 31;
                pos[i] |= (inf & (nan | ~(u >> 31))) << k;
                neg[i] |= (inf & (nan | (u >> 31))) << k;
            });
            store(again_lane());
        } else if (sweep == 2) {                         // whole numbers, none negative
            mark([&](uint32_t u, int i, int k) { pos[i] |= (u < 1u ? u : 1u) << k; });
        } else if (sweep == 3) {
            mark([&](uint32_t u, int i, int k) { neg[i] |= (u < 1u ? u : 1u) << k; });
        }
    }
    if constexpr (G == 2) {                              // each group has seen half of the channels
        uint32_t* const red = reinterpret_cast<uint32_t*>(lds) + (tid & 255);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MW; ++i)
            if (grp) red[512 * i] = pos[i], red[512 * i + 256] = neg[i];
        __syncthreads();
        if (grp) return;
#pragma unroll
        for (int i = 0; i < MW; ++i) pos[i] |= red[512 * i], neg[i] |= red[512 * i + 256];
    }
    outputs(again_lane(), [&](int a, int t, int r, float, uint16_t* to) {
        const int i = (a * NI + t) / 2, k = ((a * NI + t) % 2) * 16 + r;
        const bool p = (pos[i] >> k) & 1, n = (neg[i] >> k) & 1;
        if (p || n) *to = g.relu ? (p && !n ? 0x7c00 : 0) : n ? (p ? 0x7e00 : 0xfc00) : 0x7c00;
    });
}

// A tile of NT pixels and G groups of waves; false when the kernel does not
// take it.  Host only.
bool tile_plan(const ConvArgs& a, int m, int NT, int G, MPlan& p) {
    const int kThreads = 256 * G, KC = kKC * G;
    int64_t rows;
    if (!geometry(a, m, NT, p, rows)) return false;
    MGeo& g = p.g;
    const int64_t items = (KC / 8) * rows * ((g.S * g.TW + 3) / 4);
    const int64_t per = (items + kThreads - 1) / kThreads;
    p.MI = per <= 2 ? 2 : 4;
    if (per > p.MI || (g.CT > 1 && (KC / 8) * rows * 2 > kThreads)) return false;
    p.G = G;
    p.lds = size_t(9 * (KC / 8) * kF * 16) + size_t(KC / 8) * g.Lst * 16;
    return p.lds <= 136 * 1024;
}

bool plan_conv_mfma(const PatTable& tab, const ConvArgs& a, MPlan& p) {
    if (a.dtype != DT_F16 || a.pool || a.cin < 16 || a.cout < 32) return false;
    // 32-bit byte offsets into x, and up to 64 channels past it
    if ((int64_t(a.n) * a.cin + 64) * a.h * a.w * 2 >= (int64_t(1) << 31) || a.keep > 0x0fffffff) return false;
    // Against the vector kernels: those take about 7 us and 30 TFLOP/s of
    // nonzero multiply-adds on small and middle calls (48 on the largest);
    // this path about 6 us (two launches) and the larger of 3 us per 64
    // channels (the latency of one tile's chain of stages) and 700 TFLOP/s of
    // dense work.  Measured both ways on 30 layers; those within 15 % stay.
    const double outs = double(a.n) * ((a.h - 1) / a.stride + 1) * ((a.w - 1) / a.stride + 1);
    const double valu_us = 7.0 + 8.0 * outs * double(a.keep) / 30e6;
    const double padded = double((a.cin + 31) / 32 * 32) * ((a.cout + 63) / 64 * 64);
    const double dense_us = 18.0 * outs * padded / 700e6, chain_us = 3.0 * ((a.cin + 63) / 64);
    if (1.15 * (6.0 + (dense_us > chain_us ? dense_us : chain_us)) > valu_us) return false;
    std::memset(&p, 0, sizeof p);
    pack_taps(tab, p.g);
    // The largest tile that still gives each CU about 1.5 blocks (2 fit);
    // else about one block per CU, of 8 waves that take 64 channels a stage
    // (256 @ 14x14 at batch 32: 22.7 us, against 24.5 in 4-wave blocks of half
    // the pixels; 512 @ 7x7: 29.8 against 33.7).
    if (tile_plan(a, tab.m, 256, 1, p) && p.g.nblocks >= 384) return true;
    if (tile_plan(a, tab.m, 128, 1, p) && p.g.nblocks >= 384) return true;
    if (p.g.nblocks >= 160 && p.g.nblocks <= 256 && tile_plan(a, tab.m, 128, 2, p)) return true;
    if (tile_plan(a, tab.m, 64, 2, p) && p.g.nblocks <= 256) return true;
    return tile_plan(a, tab.m, 64, 1, p);
}

template <int NT, int G, bool ALIGNED, int MI>
hipError_t launch(const MPlan& p, const PackedView& pk, const ConvArgs& a, hipStream_t s) {
    const int grid = (p.g.nblocks + 7) / 8 * 8;
    hipLaunchKernelGGL((k_conv_mfma<NT, G, ALIGNED, MI>), dim3(unsigned(grid)), dim3(256 * G), unsigned(p.lds), s,
                       static_cast<const uint16_t*>(a.x), static_cast<const uint16_t*>(a.ws), pk.filter_perm,
                       static_cast<const uint16_t*>(a.bias), p.g, static_cast<uint16_t*>(a.y));
    return hipGetLastError();
}

template <int NT, int G>
hipError_t launch_nt(const MPlan& p, const PackedView& pk, const ConvArgs& a, hipStream_t s) {
    if (p.aligned) return p.MI == 2 ? launch<NT, G, true, 2>(p, pk, a, s) : launch<NT, G, true, 4>(p, pk, a, s);
    return p.MI == 2 ? launch<NT, G, false, 2>(p, pk, a, s) : launch<NT, G, false, 4>(p, pk, a, s);
}

}  // namespace

size_t conv_workspace_bytes(int dtype, int cout, int cin) {
    if (cin < 16 || cout < 32) return 0;
    if (dtype == DT_F32) return split_tiles_bytes(cout, cin);
    return size_t((cout + kF - 1) / kF) * size_t((cin + 63) / 64 * 2) * (9 * kKC * kF * 2);
}

bool conv_mfma_takes(const PatTable& tab, const ConvArgs& a) {
    if (a.dtype == DT_F32) return conv_split_takes(tab, a);
    MPlan p;
    return plan_conv_mfma(tab, a, p);
}

hipError_t launch_conv_mfma(const PatTable& tab, const PackedView& pk, const ConvArgs& a, hipStream_t s) {
    MPlan p;
    if (!a.ws || a.ws_bytes < conv_workspace_bytes(a.dtype, a.cout, a.cin) || !plan_conv_mfma(tab, a, p))
        return hipErrorNotSupported;
    const dim3 grid(unsigned((p.g.ftiles * kF) / kDF), unsigned((a.cin + kDC - 1) / kDC));
    hipLaunchKernelGGL(k_weight_tiles, grid, dim3(512), 0, s, pk.filter_ptr, pk.cin_idx, pk.pat_id,
                       static_cast<const uint16_t*>(pk.values), p.g, static_cast<uint16_t*>(a.ws));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.NT == 256) return launch_nt<256, 1>(p, pk, a, s);
    if (p.NT == 128) return p.G == 1 ? launch_nt<128, 1>(p, pk, a, s) : launch_nt<128, 2>(p, pk, a, s);
    return p.G == 1 ? launch_nt<64, 1>(p, pk, a, s) : launch_nt<64, 2>(p, pk, a, s);
}

}  // namespace psc
