// Offline preparation kernels: pattern projection (Sec. 4.3, Eq. 6),
// connectivity pruning (Sec. 4.4), filter kernel reorder + compressed weight
// storage (Sec. 3.4) and the dense unpacker.  All results are integer or bit
// copies except the fp64 energies, which are sums of exact squares added in a
// fixed order, so every output is bit-exact and run-to-run deterministic.
#include <mutex>

#include "common.h"
#include "launch.h"

// Products of fp32 values are exact in fp64, so contraction could not change
// a result here; keep it off anyway so each add is a plain rounded add.
#pragma clang fp contract(off)

namespace psc {
namespace {

// ---------------------------------------------------------------- projection
constexpr int kProjBlock = 256;

template <int DT>
__global__ __launch_bounds__(kProjBlock) void k_project(const typename Elt<DT>::T* __restrict__ w,
                                                       int64_t n_kernels, PatTable tab,
                                                       uint8_t* __restrict__ pat,
                                                       double* __restrict__ energy) {
    __shared__ float tile[kProjBlock * 9];
    const int64_t k0 = int64_t(blockIdx.x) * kProjBlock;
    const int nk = int(min<int64_t>(kProjBlock, n_kernels - k0));
    // coalesced staging of the block's nk*9 contiguous weights
    for (int i = threadIdx.x; i < nk * 9; i += kProjBlock) tile[i] = Elt<DT>::load(w + k0 * 9, i);
    __syncthreads();
    const int t = threadIdx.x;
    if (t >= nk) return;
    double sq[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const double v = double(tile[t * 9 + q]);  // stride 9: conflict-free
        sq[q] = v * v;
    }
    int best_p = 0;
    double best_e = 0.0;
    for (int p = 0; p < tab.m; ++p) {
        const unsigned mk = tab.mask[p];
        double e = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q)
            if ((mk >> q) & 1u) e = e + sq[q];
        if (p == 0 || e > best_e) {
            best_e = e;
            best_p = p;
        }
    }
    pat[k0 + t] = uint8_t(best_p);
    energy[k0 + t] = best_e;
}

// ---------------------------------------------------------------- top-beta
// Selection over the uint64 images of the non-negative fp64 energies
// (order-preserving).  Here the form for more than kSelFastMax kernels: 8
// bits per pass from the top, then an index-ordered rank of the keys equal to
// the threshold; the forms of smaller layers follow below.
struct SelState {
    uint64_t prefix;     // digits of the threshold found so far
    uint64_t mask;       // which bits of prefix are decided
    int64_t remaining;   // kernels still to keep among keys matching prefix
    int64_t pad;
};
constexpr int kSelChunk = 1024;     // keys per block in count/mark
constexpr size_t kSelHistOff = 0;   // 256 x u32
constexpr size_t kSelStateOff = 1024;
constexpr size_t kSelCountOff = 1280;

// The digit of one radix pass, by threads 0..255 of the block (every thread
// of the block calls it): with S(d) the number of candidate keys whose digit
// is d or more, the digit is the largest d >= 1 with S(d) >= r (r = kernels
// still to keep), else 0 -- the first digit from the top at which the
// running count reaches r -- and S(d + 1) keys rank above it.  Suffix sums
// in LDS instead of a serial walk over the 256 bins.  Returns the digit and
// sets *above (both valid in every thread).
__device__ __forceinline__ int sel_digit(const uint32_t* hist, int64_t r, uint64_t* sfx, int* s_d, int64_t* above) {
    const int t = threadIdx.x;
    if (t < 256) sfx[t] = hist[t];
    if (t == 0) {
        sfx[256] = 0;
        *s_d = 0;
    }
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint64_t v = t < 256 && t + off < 256 ? sfx[t + off] : 0u;
        __syncthreads();
        if (t < 256) sfx[t] += v;
        __syncthreads();
    }
    if (t >= 1 && t < 256 && int64_t(sfx[t]) >= r) atomicMax(s_d, t);
    __syncthreads();
    const int d = *s_d;
    *above = int64_t(sfx[d + 1]);
    return d;
}

__global__ __launch_bounds__(256) void k_sel_init(uint32_t* __restrict__ hist, SelState* __restrict__ st,
                                                  int64_t keep) {
    hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        st->prefix = 0;
        st->mask = 0;
        st->remaining = keep;
        st->pad = 0;
    }
}

__global__ __launch_bounds__(256) void k_sel_hist(const uint64_t* __restrict__ keys, int64_t n,
                                                  int shift, const SelState* __restrict__ st,
                                                  uint32_t* __restrict__ hist) {
    __shared__ uint32_t lh[256];
    lh[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t prefix = st->prefix, mask = st->mask;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const uint64_t key = keys[i];
        if ((key & mask) == prefix) atomicAdd(&lh[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    const uint32_t c = lh[threadIdx.x];
    if (c) atomicAdd(&hist[threadIdx.x], c);
}

__global__ __launch_bounds__(256) void k_sel_pick(uint32_t* __restrict__ hist, SelState* __restrict__ st,
                                                  int shift) {
    __shared__ uint64_t sfx[257];
    __shared__ int s_d;
    const int64_t r = st->remaining;
    int64_t above;
    const int d = sel_digit(hist, r, sfx, &s_d, &above);
    if (threadIdx.x == 0) {
        st->remaining = r - above;
        st->prefix |= uint64_t(d) << shift;
        st->mask |= uint64_t(255) << shift;
    }
    hist[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void k_sel_count(const uint64_t* __restrict__ keys, int64_t n,
                                                   const SelState* __restrict__ st,
                                                   uint32_t* __restrict__ blk) {
    __shared__ uint32_t red[256];
    const uint64_t T = st->prefix;
    const int64_t base = int64_t(blockIdx.x) * kSelChunk + threadIdx.x * 4;
    uint32_t c = 0;
    for (int j = 0; j < 4; ++j) {
        const int64_t i = base + j;
        if (i < n && keys[i] == T) ++c;
    }
    red[threadIdx.x] = c;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) blk[blockIdx.x] = red[0];
}

// In-place exclusive scan of n u32 values with one block of 1024 threads,
// each owning a contiguous run (so the result is in index order).
__global__ __launch_bounds__(1024) void k_scan_excl_u32(uint32_t* __restrict__ a, int64_t n) {
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int64_t per = (n + 1023) / 1024;
    const int64_t beg = min<int64_t>(n, t * per), end = min<int64_t>(n, beg + per);
    uint32_t s = 0;
    for (int64_t i = beg; i < end; ++i) s += a[i];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t run = part[t] - s;
    for (int64_t i = beg; i < end; ++i) {
        const uint32_t v = a[i];
        a[i] = run;
        run += v;
    }
}

__global__ __launch_bounds__(256) void k_sel_mark(const uint64_t* __restrict__ keys, int64_t n,
                                                  const SelState* __restrict__ st,
                                                  const uint32_t* __restrict__ blk_off,
                                                  uint8_t* __restrict__ keep) {
    __shared__ uint32_t part[256];
    const uint64_t T = st->prefix;
    const int64_t r = st->remaining;
    const int t = threadIdx.x;
    const int64_t base = int64_t(blockIdx.x) * kSelChunk + t * 4;
    uint64_t kv[4];
    uint32_t c = 0;
    for (int j = 0; j < 4; ++j) {
        const int64_t i = base + j;
        kv[j] = i < n ? keys[i] : 0;
        if (i < n && kv[j] == T) ++c;
    }
    part[t] = c;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t rank = int64_t(blk_off[blockIdx.x]) + (part[t] - c);
    for (int j = 0; j < 4; ++j) {
        const int64_t i = base + j;
        if (i >= n) break;
        uint8_t v = 0;
        if (kv[j] > T) {
            v = 1;
        } else if (kv[j] == T) {
            v = rank < r ? 1 : 0;
            ++rank;
        }
        keep[i] = v;
    }
}

// ---- Selection without the fixed 8 passes (layers of at most kSelFastMax
// kernels).  A block narrows a set of candidate keys to the threshold T: each
// round takes the bits that all candidates share as decided, histograms the
// next 11, and keeps the bin in which the count from the top reaches r.  It
// ends as soon as a bin is kept whole (T is then the bin's lower end) or all
// candidates are equal; random energies take two or three rounds.  Among the
// keys equal to T the lowest indices are kept, up to an index `cut`, so the
// keep mask is the same bit for bit.  Bound by launches and by the latency of
// a round's barriers, not by the keys (2 MB at 512 x 512).  Measured against 8
// passes of 8 bits: 4096 kernels 37 -> 9 us in one block, 262144 kernels 19
// launches and 105 us -> 6 and 25.
constexpr int kSelBins = 2048;
// Lines: one block 38 us at 16384 tied keys where the grid takes 40 (random 23,
// 22); above 2^20 kernels (4096 a block of pass 0) the radix passes stay, 132 us
// there.
constexpr int64_t kSelOneBlockMax = 16384, kSelFastMax = int64_t(1) << 20;

struct SelCut {
    uint64_t T;      // threshold
    int64_t cut;     // keep key > T, and key == T up to this index
};

struct SelShared {
    uint32_t hist[kSelBins];
    uint64_t w_and[16], w_or[16];
    uint32_t part[1024];
    uint32_t wsum[16];
    int digit;
    int64_t above, cut;
};

// The largest bin d with S(d) >= r, S(d) the count of bins d and up, and
// S(d + 1), from `bins` counters (a multiple of 1024; S(0) >= r).  Every
// thread of a 1024-thread block calls it.
__device__ __forceinline__ void sel_bin(const uint32_t* hist, int bins, int64_t r, SelShared& sh) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, per = bins / 1024;
    // thread t owns the bins from the top down: per * t .. per * t + per - 1
    uint32_t own = 0;
    for (int j = 0; j < per; ++j) own += hist[bins - 1 - per * t - j];
    uint32_t inc = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_up(inc, off);
        if (lane >= off) inc += v;
    }
    if (lane == 63) sh.wsum[wave] = inc;
    __syncthreads();
    for (int w = 0; w < wave; ++w) inc += sh.wsum[w];
    const uint32_t before = inc - own;
    if (int64_t(before) < r && int64_t(inc) >= r) {      // one thread
        int64_t run = before;
        int d = bins - 1 - per * t;
        while (run + int64_t(hist[d]) < r) run += hist[d--];
        sh.digit = d;
        sh.above = run;
    }
    __syncthreads();
}

// T and cut of the r largest of n candidates (those that match the decided
// bits `mask` of `prefix`; 1 <= r <= their number).  each(f) calls f on the
// thread's share of the keys; key(i) and index(i) name the i-th key and its
// index, for ties; `ordered`: index(i) ascends with i.  All 1024 threads call
// it.
template <typename Each, typename Key, typename Index>
__device__ SelCut sel_narrow(Each each, Key key, Index index, bool ordered, int64_t n, int64_t r, uint64_t prefix, uint64_t mask,
                             SelShared& sh) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint64_t T = 0;
    bool all = false;                                    // every candidate that is left is kept
    for (;;) {
        uint64_t va = ~uint64_t(0), vo = 0;
        each([&](uint64_t k) {
            if ((k & mask) == prefix) va &= k, vo |= k;
        });
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            va &= uint64_t(__shfl_xor((unsigned long long)va, off));
            vo |= uint64_t(__shfl_xor((unsigned long long)vo, off));
        }
        if (lane == 0) sh.w_and[wave] = va, sh.w_or[wave] = vo;
        for (int b = t; b < kSelBins; b += 1024) sh.hist[b] = 0;
        __syncthreads();
        for (int w = 0; w < 16; ++w) va &= sh.w_and[w], vo |= sh.w_or[w];
        const uint64_t diff = va ^ vo;
        if (diff == 0) {
            T = va;
            break;
        }
        const int hb = 63 - __clzll((long long)diff), shift = hb > 10 ? hb - 10 : 0;
        const uint64_t low = (uint64_t(2) << hb) - 1;    // all ones for hb = 63
        mask = ~low;
        prefix = va & mask;
        each([&](uint64_t k) {
            if ((k & mask) == prefix) atomicAdd(&sh.hist[(k & low) >> shift], 1u);
        });
        __syncthreads();
        sel_bin(sh.hist, kSelBins, r, sh);
        const int d = sh.digit;
        r -= sh.above;
        prefix |= uint64_t(d) << shift;
        mask = shift ? ~((uint64_t(1) << shift) - 1) : ~uint64_t(0);
        all = int64_t(sh.hist[d]) == r;
        __syncthreads();
        if (all || shift == 0) {
            T = prefix;
            break;
        }
    }
    if (all) return SelCut{T, INT64_MAX};
    // the r-th lowest index of the keys equal to T
    if (t == 0) sh.cut = INT64_MAX;
    __syncthreads();
    if (ordered) {
        const int64_t per = (n + 1023) / 1024, beg = min<int64_t>(n, t * per), end = min<int64_t>(n, beg + per);
        uint32_t c = 0;
        for (int64_t i = beg; i < end; ++i) c += key(i) == T;
        sh.part[t] = c;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const uint32_t v = t >= off ? sh.part[t - off] : 0u;
            __syncthreads();
            sh.part[t] += v;
            __syncthreads();
        }
        int64_t rank = int64_t(sh.part[t]) - c;
        if (rank < r && rank + c >= r)
            for (int64_t i = beg; i < end; ++i)
                if (key(i) == T && ++rank == r) sh.cut = index(i);
    } else {
        for (int64_t i = t; i < n; i += 1024) {
            if (key(i) != T) continue;
            const int64_t at = index(i);
            int64_t rank = 0;
            for (int64_t j = 0; j < n; ++j) rank += key(j) == T && index(j) < at;
            if (rank == r - 1) sh.cut = at;
        }
    }
    __syncthreads();
    return SelCut{T, sh.cut};
}

// The whole selection in one workgroup, KPT keys in each thread's registers:
// one launch, where the grid's way below takes six (about 3 us of host time
// each, which small layers feel).
template <int KPT>
__global__ __launch_bounds__(1024) void k_sel_one(const uint64_t* __restrict__ keys, int64_t n, int64_t keep,
                                                  uint8_t* __restrict__ out) {
    __shared__ SelShared sh;
    uint64_t kv[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int64_t i = threadIdx.x + 1024 * j;
        kv[j] = i < n ? keys[i] : 0;
    }
    // ties are ranked over contiguous runs, from memory
    const SelCut c = sel_narrow(
        [&](auto f) {
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if (threadIdx.x + 1024 * j < n) f(kv[j]);
        },
        [&](int64_t i) { return keys[i]; }, [](int64_t i) { return i; }, true, n, keep, 0, 0, sh);
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int64_t i = threadIdx.x + 1024 * j;
        if (i < n) out[i] = kv[j] > c.T || (kv[j] == c.T && i <= c.cut);
    }
}

// More keys: two histograms of 12 bits (sign and exponent, then the top of
// the mantissa) over the whole grid, the keys of the bin that is left in a
// list, T and cut from the list in one block, then the mask: 6 launches.  Each
// block takes the digit of the pass before from its histogram.  Where the bin
// holds more keys than the list (thousands of equal leading bits: weights
// already pruned, or of few values), pass 2 goes on over the whole grid in
// rounds of 10 bits (one, where the keys of the bin are all equal) and then
// ranks the ties, instead of the list.
// Measured (half kept; 8 passes of 8 bits first, then one block going over all
// the keys, then the rounds, us): 262144 kernels random 92, 24, 24; all equal
// 147, 252, 53; 70 % zeros 142, 250, 53; eight values 141, 244, 52; equal in 32
// leading bits 136, 365, 93; 1048576 kernels random 133, 31, 31; all equal 247,
// 1211, 92; equal in 32 bits 235, 2257, 163.
constexpr int kSelWide = 4096, kSelList = 2560, kSelRounds = 4, kSelChunks = 32;
struct SelStage {                                // each counter in a line of its own
    uint32_t claim, pad[63], done, pad2[63];
};
struct SelTail {                                 // of pass 2 without a list
    uint32_t hist[kSelRounds][1024];
    uint32_t ties[kSelChunks];                   // keys equal to T, by chunk
    unsigned long long ones, zeros;              // bits set, and clear, in some key of the bin
    SelStage stage[kSelRounds + 2];
};
struct SelWide {
    uint32_t hist[2][kSelWide];
    uint32_t count;
    uint32_t pad[63];
    SelCut cut;
    uint64_t pad2[30];
    union {
        struct {
            uint64_t key[kSelList];
            uint32_t index[kSelList];
        };
        SelTail tail;                            // zeroed by pass 1
    };
};
static_assert(sizeof(SelWide) <= 64 * 1024, "the scratch of psc_select_noalloc");

__global__ __launch_bounds__(1024) void k_selw_clear(SelWide* __restrict__ s) {
    for (int i = threadIdx.x; i < 2 * kSelWide; i += 1024) (&s->hist[0][0])[i] = 0;
    if (threadIdx.x == 0) s->count = 0;
}

// One more in `bin` of each active lane's; one addition for the wave where
// they are all the same bin (ties), which LDS would serve one by one.
__device__ __forceinline__ void hist_add(uint32_t* h, uint32_t bin) {
    const uint64_t on = __ballot(1);
    const int first = __builtin_ctzll(on);
    if (__ballot(bin == uint32_t(__shfl(int(bin), first))) == on) {
        if (int(threadIdx.x & 63) == first) atomicAdd(&h[bin], uint32_t(__popcll(on)));
    } else {
        atomicAdd(&h[bin], 1u);
    }
}

template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The next item of a stage of k_selw_pass<2>'s rounds, in every thread of the
// block.
__device__ __forceinline__ uint32_t sel_claim(SelTail* tl, int stage, uint32_t* item) {
    __syncthreads();                             // every thread has read the last one
    if (threadIdx.x == 0) *item = atomicAdd(&tl->stage[stage].claim, 1u);
    __syncthreads();
    return *item;
}

// What the block wrote for an item is seen by every block that waits for the
// stage.
__device__ __forceinline__ void sel_finish(SelTail* tl, int stage) {
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(&tl->stage[stage].done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Until all items of a stage are done.  A block comes here only when every
// item is claimed, and a block that has claimed one finishes it without
// waiting for any other: the wait ends however few blocks run at a time.
__device__ __forceinline__ void sel_wait(const SelTail* tl, int stage, uint32_t items) {
    if (threadIdx.x == 0) {
        while (load_agent(&tl->stage[stage].done) < items) __builtin_amdgcn_s_sleep(4);
        __threadfence();
    }
    __syncthreads();
}

// Pass 2 without a list: T and cut of the r largest of the keys that match
// `prefix` in their upper 24 bits.  The keys are cut into at most kSelChunks
// chunks, which the first as many blocks take as they come to them (a stage
// costs about 0.3 us a block in traffic on its counters: equal in 32 leading
// bits, 262144 kernels, 93 us in 32 chunks, 130 in 64).
__device__ __forceinline__ void sel_rounds(const uint64_t* __restrict__ keys, int64_t n, int64_t r, uint64_t prefix,
                                           SelWide* s, uint32_t* lh, SelShared& sh) {
    __shared__ uint32_t item;
    SelTail* const tl = &s->tail;
    const uint32_t chunks = gridDim.x < kSelChunks ? gridDim.x : kSelChunks;
    if (blockIdx.x >= chunks) return;
    const int64_t per = (n + chunks - 1) / chunks;
    const int t = threadIdx.x;
    bool all = false;                            // every key that is left is kept
    int round = 0;
    for (; round < kSelRounds && !all; ++round) {
        const int shift = 10 * (kSelRounds - 1 - round), up = shift + 10;
        for (uint32_t c; (c = sel_claim(tl, round, &item)) < chunks;) {
            lh[t] = 0;
            __syncthreads();
            const int64_t end = min<int64_t>(n, (c + 1) * per);
            unsigned long long ones = 0, zeros = 0;
            for (int64_t i = c * per + t; i < end; i += 1024) {
                const uint64_t k = keys[i];
                if (k >> up != prefix) continue;
                hist_add(lh, (k >> shift) & 1023);
                ones |= k;
                zeros |= ~k;
            }
            __syncthreads();
            if (lh[t]) atomicAdd(&tl->hist[round][t], lh[t]);
            if (round == 0) {
                for (int off = 32; off > 0; off >>= 1) {
                    ones |= __shfl_xor(ones, off);
                    zeros |= __shfl_xor(zeros, off);
                }
                if ((t & 63) == 0) sh.w_and[t >> 6] = ones, sh.w_or[t >> 6] = zeros;
                __syncthreads();
                if (t == 0) {
                    for (int w = 1; w < 16; ++w) ones |= sh.w_and[w], zeros |= sh.w_or[w];
                    atomicOr(&tl->ones, ones);
                    atomicOr(&tl->zeros, zeros);
                }
            }
            sel_finish(tl, round);
        }
        sel_wait(tl, round, chunks);
        if (round == 0) {                        // all equal: no further digit
            const uint64_t ones = load_agent(&tl->ones);
            if ((ones & load_agent(&tl->zeros)) == 0) {
                prefix = ones;
                break;
            }
        }
        lh[t] = load_agent(&tl->hist[round][t]);
        __syncthreads();
        sel_bin(lh, 1024, r, sh);
        r -= sh.above;
        prefix = prefix << 10 | uint64_t(sh.digit);
        all = int64_t(lh[sh.digit]) == r;
        __syncthreads();                         // every thread has read sh and lh
    }
    if (all) {                                   // T is the lower end of the bin
        if (sel_claim(tl, kSelRounds + 1, &item) == 0 && t == 0)
            s->cut = SelCut{prefix << (10 * (kSelRounds - round)), INT64_MAX};
        return;
    }
    // the r-th lowest index of the keys equal to T: by chunk, then inside one
    const uint64_t T = prefix;
    for (uint32_t c; (c = sel_claim(tl, kSelRounds, &item)) < chunks;) {
        const int64_t end = min<int64_t>(n, (c + 1) * per);
        int own = 0;
        for (int64_t i = c * per + t; i < end; i += 1024) own += keys[i] == T;
        for (int off = 32; off > 0; off >>= 1) own += __shfl_xor(own, off);
        if ((t & 63) == 0) sh.wsum[t >> 6] = own;
        __syncthreads();
        if (t == 0) {
            uint32_t sum = 0;
            for (int w = 0; w < 16; ++w) sum += sh.wsum[w];
            __hip_atomic_store(&tl->ties[c], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        sel_finish(tl, kSelRounds);
    }
    sel_wait(tl, kSelRounds, chunks);
    if (sel_claim(tl, kSelRounds + 1, &item) != 0) return;
    // inclusive sums of `part` over the block
    auto scan = [&](uint32_t v) {
        sh.part[t] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const uint32_t b = t >= off ? sh.part[t - off] : 0u;
            __syncthreads();
            sh.part[t] += b;
            __syncthreads();
        }
        return sh.part[t];
    };
    const uint32_t v = t < int(chunks) ? load_agent(&tl->ties[t]) : 0u, inc = scan(v);
    if (int64_t(inc) >= r && int64_t(inc - v) < r) {     // one thread
        sh.digit = t;
        sh.above = inc - v;
    }
    __syncthreads();
    const int64_t beg = sh.digit * per, end = min<int64_t>(n, beg + per), quarter = (per + 1023) / 1024;
    r -= sh.above;
    const int64_t lo = min<int64_t>(end, beg + t * quarter), hi = min<int64_t>(end, lo + quarter);
    uint32_t own = 0;
    for (int64_t i = lo; i < hi; ++i) own += keys[i] == T;
    int64_t rank = int64_t(scan(own)) - own;
    if (rank < r && rank + own >= r)                     // one thread
        for (int64_t i = lo; i < hi; ++i)
            if (keys[i] == T && ++rank == r) s->cut = SelCut{T, i};
}

// Pass 0 or 1, or (pass 2) the list of the keys that match both digits, or the
// rounds.
template <int PASS>
__global__ __launch_bounds__(1024) void k_selw_pass(const uint64_t* __restrict__ keys, int64_t n, int64_t keep,
                                                    SelWide* s) {
    __shared__ SelShared sh;
    __shared__ uint32_t lh[PASS < 2 ? kSelWide : 1024];
    int64_t r = keep;
    uint64_t prefix = 0;
#pragma unroll
    for (int p = 0; p < PASS; ++p) {
        sel_bin(s->hist[p], kSelWide, r, sh);
        r -= sh.above;
        prefix = prefix << 12 | uint64_t(sh.digit);
        __syncthreads();
    }
    if (PASS < 2) {
        for (int b = threadIdx.x; b < kSelWide; b += 1024) lh[b] = 0;
        if (PASS == 1 && blockIdx.x == 0)
            for (int b = threadIdx.x; b < int(sizeof(SelTail) / 4); b += 1024) reinterpret_cast<uint32_t*>(&s->tail)[b] = 0;
        __syncthreads();
    } else if (s->hist[1][prefix & 4095] > kSelList) {
        sel_rounds(keys, n, r, prefix, s, lh, sh);
        return;
    }
    for (int64_t i = int64_t(blockIdx.x) * 1024 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 1024) {
        const uint64_t k = keys[i];
        if (PASS == 0) {
            atomicAdd(&lh[k >> 52], 1u);
        } else if (PASS == 1) {
            if (k >> 52 == prefix) hist_add(lh, (k >> 40) & 4095);
        } else if (k >> 40 == prefix) {
            const uint32_t at = atomicAdd(&s->count, 1u);
            if (at < kSelList) s->key[at] = k, s->index[at] = uint32_t(i);
        }
    }
    if (PASS < 2) {
        __syncthreads();
        for (int b = threadIdx.x; b < kSelWide; b += 1024)
            if (lh[b]) atomicAdd(&s->hist[PASS][b], lh[b]);
    }
}

__global__ __launch_bounds__(1024) void k_selw_cut(int64_t keep, SelWide* __restrict__ s) {
    __shared__ SelShared sh;
    int64_t r = keep;
    uint64_t prefix = 0;
    for (int p = 0; p < 2; ++p) {
        sel_bin(s->hist[p], kSelWide, r, sh);
        r -= sh.above;
        prefix = prefix << 12 | uint64_t(sh.digit);
        __syncthreads();
    }
    if (s->hist[1][prefix & 4095] > kSelList) return;    // pass 2 has written it
    const int64_t count = s->count;
    const SelCut c = sel_narrow(
        [&](auto f) {
            for (int64_t i = threadIdx.x; i < count; i += 1024) f(s->key[i]);
        },
        [&](int64_t i) { return s->key[i]; }, [&](int64_t i) { return int64_t(s->index[i]); }, false, count, r,
        prefix << 40, ~((uint64_t(1) << 40) - 1), sh);
    if (threadIdx.x == 0) s->cut = c;
}

__global__ __launch_bounds__(256) void k_selw_mark(const uint64_t* __restrict__ keys, int64_t n,
                                                   const SelWide* __restrict__ s, uint8_t* __restrict__ out) {
    const SelCut c = s->cut;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const uint64_t k = keys[i];
        out[i] = k > c.T || (k == c.T && i <= c.cut);
    }
}

__global__ __launch_bounds__(256) void k_fill_u8(uint8_t* __restrict__ p, int64_t n, uint8_t v) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) p[i] = v;
}

// ---------------------------------------------------------------- packing
// Per filter: kept count and per-pattern counts.  One wave per filter.
__global__ __launch_bounds__(64) void k_pack_count(const uint8_t* __restrict__ pat,
                                                   const uint8_t* __restrict__ keep, int cin, int m,
                                                   int32_t* __restrict__ cnt, int32_t* __restrict__ nf) {
    __shared__ int32_t c_s[kMaxPatterns];
    const int f = blockIdx.x, lane = threadIdx.x;
    for (int p = lane; p < m; p += 64) c_s[p] = 0;
    __syncthreads();
    int n = 0;
    for (int c0 = 0; c0 < cin; c0 += 64) {
        const int ci = c0 + lane;
        bool kept = false;
        int pp = 0;
        if (ci < cin) {
            const int64_t k = int64_t(f) * cin + ci;
            kept = keep[k] != 0;
            pp = pat[k];
        }
        n += __popcll(__ballot(kept));
        if (kept && pp < m) atomicAdd(&c_s[pp], 1);
    }
    __syncthreads();
    for (int p = lane; p < m; p += 64) cnt[int64_t(f) * m + p] = c_s[p];
    if (lane == 0) nf[f] = n;
}

// Rank of each filter under (count desc, per-pattern counts lexicographically
// desc, index asc); the key is a total order, so ranks form a permutation.
// One block per filter f: its threads compare f with every other filter g
// (g = t, t + 256, ...) and the block adds up how many come first.
__global__ __launch_bounds__(256) void k_pack_rank(const int32_t* __restrict__ cnt,
                                                   const int32_t* __restrict__ nf, int cout, int m,
                                                   int32_t* __restrict__ perm,
                                                   int32_t* __restrict__ nf_sorted) {
    __shared__ int part[4];
    const int f = blockIdx.x;
    const int nff = nf[f];
    const int32_t* cf = cnt + int64_t(f) * m;
    int rank = 0;
    for (int g = threadIdx.x; g < cout; g += 256) {
        if (g == f) continue;
        const int ng = nf[g];
        bool before;
        if (ng != nff) {
            before = ng > nff;
        } else {
            before = g < f;
            const int32_t* cg = cnt + int64_t(g) * m;
            for (int p = 0; p < m; ++p) {
                if (cg[p] != cf[p]) {
                    before = cg[p] > cf[p];
                    break;
                }
            }
        }
        rank += before ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) rank += __shfl_xor(rank, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = rank;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int r = part[0] + part[1] + part[2] + part[3];
        perm[r] = f;
        nf_sorted[r] = nff;
    }
}

// out[0..n] = exclusive prefix sums of in[0..n-1], out[n] = total.
__global__ __launch_bounds__(1024) void k_scan_excl_i32(const int32_t* __restrict__ in,
                                                        int32_t* __restrict__ out, int n) {
    __shared__ int32_t part[1024];
    const int t = threadIdx.x;
    const int per = (n + 1023) / 1024;
    const int beg = min(n, t * per), end = min(n, beg + per);
    int32_t s = 0;
    for (int i = beg; i < end; ++i) s += in[i];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int32_t v = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int32_t run = part[t] - s;
    for (int i = beg; i < end; ++i) {
        out[i] = run;
        run += in[i];
    }
    if (t == 1023) out[n] = part[1023];
}

__global__ __launch_bounds__(256) void k_pack_seg(const int32_t* __restrict__ cnt,
                                                  const int32_t* __restrict__ perm,
                                                  const int32_t* __restrict__ fptr, int cout, int m,
                                                  int32_t* __restrict__ seg) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= cout) return;
    const int f = perm[i];
    int32_t s = fptr[i];
    for (int p = 0; p < m; ++p) {
        seg[int64_t(i) * (m + 1) + p] = s;
        s += cnt[int64_t(f) * m + p];
    }
    seg[int64_t(i) * (m + 1) + m] = fptr[i + 1];
}

// What the lanes of a wave did to memory before it happens before what they do
// after it.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Scatter of one reordered filter per block: a kernel's slot is the start of
// its pattern's segment + kept kernels of that pattern at lower ci.
template <typename B>
__global__ __launch_bounds__(256) void k_pack_scatter(const B* __restrict__ w,
                                                      const uint8_t* __restrict__ pat,
                                                      const uint8_t* __restrict__ keep, int cin,
                                                      int64_t n_keep, PatTable tab, const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ seg,
                                                      int32_t* __restrict__ cin_idx,
                                                      uint8_t* __restrict__ pat_id,
                                                      B* __restrict__ values) {
    // wave w takes the w-th quarter of the channels; cur[w][p]: the position
    // of its next kernel of pattern p.  Bound by the latency of a chain of
    // loads and ballots: 512 filters of 512 channels 25 us in one wave each
    // with two barriers per pattern, 8 so
    __shared__ int32_t cur[4][kMaxPatterns];
    __shared__ uint16_t msk[kMaxPatterns];
    const int i = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = tab.m;
    const int f = perm[i];
    for (int p = threadIdx.x; p < m; p += 256) msk[p] = tab.mask[p];
    for (int p = lane; p < m; p += 64) cur[wave][p] = 0;
    __syncthreads();
    const int per = (cin + 255) / 256 * 64, lo = min(cin, wave * per), hi = min(cin, lo + per);
    for (int ci = lo + lane; ci < hi; ci += 64) {
        const int64_t k = int64_t(f) * cin + ci;
        const int pp = pat[k];
        if (keep[k] && pp < m) atomicAdd(&cur[wave][pp], 1);
    }
    __syncthreads();
    for (int p = threadIdx.x; p < m; p += 256) {
        int32_t at = seg[int64_t(i) * (m + 1) + p];
        for (int v = 0; v < 4; ++v) {
            const int32_t c = cur[v][p];
            cur[v][p] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int c0 = lo; c0 < hi; c0 += 64) {
        const int ci = c0 + lane;
        const int64_t k = int64_t(f) * cin + ci;
        const int pp = ci < hi ? pat[k] : kMaxPatterns;
        const bool kept = ci < hi && keep[k] && pp < m;
        // the lanes of one pattern at a time, from the pattern's cursor in
        // lane order; the wave's barriers order the lanes' reads of a cursor
        // against the one lane's update of it (no instruction waits for them:
        // a wave's LDS accesses are served in order)
        uint64_t todo = __ballot(kept);
        int pos = -1;
        while (todo) {
            const int p = __shfl(pp, __builtin_ctzll(todo));
            const uint64_t b = __ballot(kept && pp == p);
            if (kept && pp == p) pos = cur[wave][p] + __popcll(b & ((uint64_t(1) << lane) - 1));
            wave_order();
            if (lane == __builtin_ctzll(b)) cur[wave][p] += __popcll(b);
            wave_order();
            todo &= ~b;
        }
        if (kept && pos >= 0 && pos < n_keep) {   // a keep mask with too many ones writes nothing past the arrays
            cin_idx[pos] = ci;
            pat_id[pos] = uint8_t(pp);
            unsigned mk = msk[pp];
            B v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = w[k * 9 + __builtin_ctz(mk | 0x200u)];
                mk &= mk - 1;
            }
            __builtin_memcpy(values + int64_t(pos) * 4, v, sizeof v);
        }
    }
}

template <typename B>
__global__ __launch_bounds__(256) void k_fill_zero(B* __restrict__ p, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) p[i] = 0;
}

template <typename B>
__global__ __launch_bounds__(256) void k_unpack(const int32_t* __restrict__ perm,
                                                const int32_t* __restrict__ fptr,
                                                const int32_t* __restrict__ cin_idx,
                                                const uint8_t* __restrict__ pat_id,
                                                const B* __restrict__ values, int cin, PatTable tab,
                                                B* __restrict__ dense) {
    __shared__ uint16_t msk[kMaxPatterns];
    for (int p = threadIdx.x; p < tab.m; p += 256) msk[p] = tab.mask[p];
    __syncthreads();
    const int i = blockIdx.x;
    const int f = perm[i];
    for (int k = fptr[i] + threadIdx.x; k < fptr[i + 1]; k += 256) {
        const int ci = cin_idx[k];
        const int p = pat_id[k];
        if (unsigned(ci) >= unsigned(cin) || p >= tab.m) continue;   // malformed storage
        const unsigned mk = msk[p];
        int j = 0;
        for (int q = 0; q < 9; ++q)
            if ((mk >> q) & 1u) dense[(int64_t(f) * cin + ci) * 9 + q] = values[int64_t(k) * 4 + j++];
    }
}

int grid_for(int64_t n, int per_block, int cap) {
    const int64_t g = (n + per_block - 1) / per_block;
    return int(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

hipError_t launch_project(const PatTable& tab, int dtype, const void* w, int64_t n_kernels,
                          uint8_t* pat, double* energy, hipStream_t stream) {
    if (n_kernels == 0) return hipSuccess;
    const dim3 grid(unsigned((n_kernels + kProjBlock - 1) / kProjBlock));
    if (dtype == DT_F16)
        hipLaunchKernelGGL(k_project<DT_F16>, grid, dim3(kProjBlock), 0, stream,
                           static_cast<const uint16_t*>(w), n_kernels, tab, pat, energy);
    else
        hipLaunchKernelGGL(k_project<DT_F32>, grid, dim3(kProjBlock), 0, stream,
                           static_cast<const float*>(w), n_kernels, tab, pat, energy);
    return hipGetLastError();
}

size_t select_workspace_bytes(int64_t n_kernels) {
    const int64_t nblk = (n_kernels + kSelChunk - 1) / kSelChunk;
    const bool wide = n_kernels > kSelOneBlockMax && n_kernels <= kSelFastMax;
    const size_t b = wide ? sizeof(SelWide) : kSelCountOff + size_t(nblk) * 4;
    return (b + 255) / 256 * 256;
}

hipError_t launch_select(int64_t n, int64_t keep, const double* energy, uint8_t* keep_out, void* ws,
                         hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (keep == 0 || keep == n) {
        hipLaunchKernelGGL(k_fill_u8, dim3(grid_for(n, 256, 4096)), dim3(256), 0, stream, keep_out, n,
                           uint8_t(keep == n ? 1 : 0));
        return hipGetLastError();
    }
    if (n <= kSelOneBlockMax) {
        const uint64_t* const k = reinterpret_cast<const uint64_t*>(energy);
        if (n <= 4096)
            hipLaunchKernelGGL(k_sel_one<4>, dim3(1), dim3(1024), 0, stream, k, n, keep, keep_out);
        else
            hipLaunchKernelGGL(k_sel_one<16>, dim3(1), dim3(1024), 0, stream, k, n, keep, keep_out);
        return hipGetLastError();
    }
    if (n <= kSelFastMax) {
        const uint64_t* const k = reinterpret_cast<const uint64_t*>(energy);
        SelWide* const s = static_cast<SelWide*>(ws);
        const dim3 g(unsigned(grid_for(n, 4096, 256)));
        hipLaunchKernelGGL(k_selw_clear, dim3(1), dim3(1024), 0, stream, s);
        hipLaunchKernelGGL(k_selw_pass<0>, g, dim3(1024), 0, stream, k, n, keep, s);
        hipLaunchKernelGGL(k_selw_pass<1>, g, dim3(1024), 0, stream, k, n, keep, s);
        hipLaunchKernelGGL(k_selw_pass<2>, g, dim3(1024), 0, stream, k, n, keep, s);
        hipLaunchKernelGGL(k_selw_cut, dim3(1), dim3(1024), 0, stream, keep, s);
        hipLaunchKernelGGL(k_selw_mark, dim3(unsigned(grid_for(n, 256, 2048))), dim3(256), 0, stream, k, n, s, keep_out);
        return hipGetLastError();
    }
    char* base = static_cast<char*>(ws);
    uint32_t* hist = reinterpret_cast<uint32_t*>(base + kSelHistOff);
    SelState* st = reinterpret_cast<SelState*>(base + kSelStateOff);
    uint32_t* blk = reinterpret_cast<uint32_t*>(base + kSelCountOff);
    const uint64_t* keys = reinterpret_cast<const uint64_t*>(energy);
    const int nblk = int((n + kSelChunk - 1) / kSelChunk);
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, stream, hist, st, keep);
    const int hg = grid_for(n, 256, 2048);
    for (int pass = 7; pass >= 0; --pass) {
        hipLaunchKernelGGL(k_sel_hist, dim3(hg), dim3(256), 0, stream, keys, n, pass * 8, st, hist);
        hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, stream, hist, st, pass * 8);
    }
    hipLaunchKernelGGL(k_sel_count, dim3(nblk), dim3(256), 0, stream, keys, n, st, blk);
    hipLaunchKernelGGL(k_scan_excl_u32, dim3(1), dim3(1024), 0, stream, blk, int64_t(nblk));
    hipLaunchKernelGGL(k_sel_mark, dim3(nblk), dim3(256), 0, stream, keys, n, st, blk, keep_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- static scratch
// The select workspace of the entry point that allocates nothing: one array
// in the library's device code.  Each GPU holds its own copy at its own
// address; in host code the array's name is only a stand-in, so kernels get
// the address hipGetSymbolAddress reports for the current device.
constexpr size_t kSelScratchBytes = 64 * 1024;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint8_t scratch[kSelScratchBytes];

size_t select_scratch_bytes() { return kSelScratchBytes; }

hipError_t select_scratch(void** out) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // with this device current
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

// Pack workspace: cnt[cout*m] | nf[cout] | nf_sorted[cout], each 256-aligned.
size_t pack_workspace_bytes(int cout, int m) {
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    return al(size_t(cout) * m * 4) + al(size_t(cout) * 4) + al(size_t(cout) * 4);
}

hipError_t launch_pack(const PatTable& tab, int dtype, int cout, int cin, int64_t n_keep, const void* w,
                       const uint8_t* pat, const uint8_t* keep, const PackedOut& out, void* ws,
                       hipStream_t stream) {
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    char* base = static_cast<char*>(ws);
    int32_t* cnt = reinterpret_cast<int32_t*>(base);
    int32_t* nf = reinterpret_cast<int32_t*>(base + al(size_t(cout) * tab.m * 4));
    int32_t* nfs = reinterpret_cast<int32_t*>(base + al(size_t(cout) * tab.m * 4) + al(size_t(cout) * 4));
    const int m = tab.m;
    const unsigned g256 = unsigned((cout + 255) / 256);
    hipLaunchKernelGGL(k_pack_count, dim3(cout), dim3(64), 0, stream, pat, keep, cin, m, cnt, nf);
    hipLaunchKernelGGL(k_pack_rank, dim3(unsigned(cout)), dim3(256), 0, stream, cnt, nf, cout, m,
                       out.filter_perm, nfs);
    hipLaunchKernelGGL(k_scan_excl_i32, dim3(1), dim3(1024), 0, stream, nfs, out.filter_ptr, cout);
    hipLaunchKernelGGL(k_pack_seg, dim3(g256), dim3(256), 0, stream, cnt, out.filter_perm,
                       out.filter_ptr, cout, m, out.seg_ptr);
    if (dtype == DT_F16)
        hipLaunchKernelGGL(k_pack_scatter<uint16_t>, dim3(cout), dim3(256), 0, stream,
                           static_cast<const uint16_t*>(w), pat, keep, cin, n_keep, tab, out.filter_perm,
                           out.seg_ptr, out.cin_idx, out.pat_id, static_cast<uint16_t*>(out.values));
    else
        hipLaunchKernelGGL(k_pack_scatter<uint32_t>, dim3(cout), dim3(256), 0, stream,
                           static_cast<const uint32_t*>(w), pat, keep, cin, n_keep, tab, out.filter_perm,
                           out.seg_ptr, out.cin_idx, out.pat_id, static_cast<uint32_t*>(out.values));
    return hipGetLastError();
}

hipError_t launch_unpack(const PatTable& tab, int dtype, int cout, int cin, int64_t keep,
                         const PackedView& pk, void* dense, hipStream_t stream) {
    const int64_t total = int64_t(cout) * cin * 9;
    if (dtype == DT_F16) {
        hipLaunchKernelGGL(k_fill_zero<uint16_t>, dim3(grid_for(total, 256, 4096)), dim3(256), 0, stream,
                           static_cast<uint16_t*>(dense), total);
        if (keep > 0)
            hipLaunchKernelGGL(k_unpack<uint16_t>, dim3(cout), dim3(256), 0, stream, pk.filter_perm,
                               pk.filter_ptr, pk.cin_idx, pk.pat_id,
                               static_cast<const uint16_t*>(pk.values), cin, tab,
                               static_cast<uint16_t*>(dense));
    } else {
        hipLaunchKernelGGL(k_fill_zero<uint32_t>, dim3(grid_for(total, 256, 4096)), dim3(256), 0, stream,
                           static_cast<uint32_t*>(dense), total);
        if (keep > 0)
            hipLaunchKernelGGL(k_unpack<uint32_t>, dim3(cout), dim3(256), 0, stream, pk.filter_perm,
                               pk.filter_ptr, pk.cin_idx, pk.pat_id,
                               static_cast<const uint32_t*>(pk.values), cin, tab,
                               static_cast<uint32_t*>(dense));
    }
    return hipGetLastError();
}

}  // namespace psc
