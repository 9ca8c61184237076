// What the two matrix-core convolutions (conv_mfma.hip: fp16; conv_split.hip:
// fp32 in bf16 parts) share: the geometry of a call.
#pragma once
#include <cstring>

#include "common.h"
#include "launch.h"

namespace psc {
namespace cm {

constexpr int kF = 64;         // filters per block

struct MGeo {
    int n, cin, H, W, cout, m, relu, keep;
    int S;              // stride
    int OH, OW;
    int CT, TW;         // column strips and output columns of one
    int P;              // positions of a tile row: S * TW + 2
    int Lst;            // positions of the X tile (its stride between channel groups)
    int slots;          // output slots of a strip: n * OH * TW
    int ptiles;         // pixel tiles of a strip
    int ftiles;
    int nblocks;
    int chunks;         // 32-channel chunks of the weight tiles: an even number
    int x_bytes;
    uint16_t taps[kMaxPatterns];   // a pattern's 4 taps, 4 bits each, ascending
};

struct MPlan {
    MGeo g;
    int NT, G, MI;
    bool aligned;
    size_t lds;
};

// Column strips, tiles and the X tile's size for tiles of NT output pixels;
// false where a strip would be narrower than one vector of 4 columns.
inline bool geometry(const ConvArgs& a, int m, int NT, MPlan& p, int64_t& rows) {
    MGeo& g = p.g;
    const int esz = a.dtype == DT_F16 ? 2 : 4;
    g.n = a.n;
    g.cin = a.cin;
    g.H = a.h;
    g.W = a.w;
    g.cout = a.cout;
    g.m = m;
    g.relu = a.relu;
    g.keep = int(a.keep);
    g.chunks = (a.cin + 63) / 64 * 2;
    g.S = a.stride;
    g.OH = (a.h - 1) / a.stride + 1;
    g.OW = (a.w - 1) / a.stride + 1;
    g.x_bytes = int(int64_t(a.n) * a.cin * a.h * a.w * esz);
    // strips of at most 32 output columns; 4-column loads are aligned where
    // rows and strips are multiples of 4 columns
    g.CT = (g.OW + 31) / 32;
    g.TW = (g.OW + g.CT - 1) / g.CT;
    p.aligned = a.w % 4 == 0 && reinterpret_cast<uintptr_t>(a.x) % (4 * esz) == 0;
    if (p.aligned && g.CT > 1) g.TW = (g.TW + 3) / 4 * 4;
    g.CT = (g.OW + g.TW - 1) / g.TW;
    if (a.w - g.S * (g.CT - 1) * g.TW < 4) return false;     // a strip narrower than one vector
    g.P = g.S * g.TW + 2;
    const int64_t slots = int64_t(a.n) * g.OH * g.TW;
    if (slots * g.CT > 0x3fffffff) return false;
    g.slots = int(slots);
    g.ptiles = int((slots + NT - 1) / NT);
    g.ftiles = (a.cout + kF - 1) / kF;
    const int64_t blocks = int64_t(g.ptiles) * g.CT * g.ftiles;
    if (blocks > 0x3fffffff) return false;
    g.nblocks = int(blocks);
    // padded rows of the largest tile: NT slots touch at most orows output
    // rows and cross at most `cross` image boundaries
    int64_t orows = (NT - 2) / g.TW + 2;
    if (orows > int64_t(a.n) * g.OH) orows = int64_t(a.n) * g.OH;
    const int64_t cross = (orows + g.OH - 2) / g.OH;
    rows = g.S * (orows - 1) + 3 + cross * (a.h + 1 - g.S * g.OH);
    g.Lst = int(rows * g.P);
    p.NT = NT;
    return true;
}

inline void pack_taps(const PatTable& tab, MGeo& g) {
    for (int i = 0; i < tab.m; ++i) {
        uint32_t t = 0, k = 0;
        for (uint32_t q = 0; q < 9; ++q)
            if ((tab.mask[i] >> q) & 1) t |= q << (4 * k++);
        g.taps[i] = uint16_t(t);
    }
}

}  // namespace cm
}  // namespace psc
