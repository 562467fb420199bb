// Which rows and columns the staged loads of the fp32 matrix-core kernels touch: plain integer
// rules, shared by the kernels and by the host code that checks them.
#ifndef PSF_F32_INDEX_H
#define PSF_F32_INDEX_H

#ifdef __HIP__
#include <hip/hip_runtime.h>
#define PSF_HD __host__ __device__ __forceinline__
#else
#define PSF_HD inline
#endif

namespace psf {

// Element a thread of a staged tile loads its four columns from: row `row`, column c of a tile whose
// rows are ld apart, or the tile's first piece where that place is not there.  The first piece has to
// exist: nvalid and width are at least 1.
PSF_HD unsigned tile_piece(int row, int c, int ld, int nvalid, int width)
{
    return row < nvalid && c < width ? (unsigned)row * (unsigned)ld + (unsigned)c : 0u;
}

// Tokens of a span that a workgroup of the state kernel walks for the value columns from c0 on: none
// where there are no such columns (dv <= 64 beside wider keys), whose sums are zero.
struct TokenRange { int begin, end; };
PSF_HD TokenRange state_tokens(int n, int span_tokens, int span, int dv, int c0)
{
    const int begin = span * span_tokens, end = begin + span_tokens < n ? begin + span_tokens : n;
    return {begin, c0 < dv ? end : begin};
}

// Grid of a launch that numbers its workgroups (256 threads) through: a dimension holds fewer than 2^32
// threads, so more than 2^23 workgroups (2^29 rows of 64 a workgroup) go into rows of 2^23.  The last
// row may hold numbers that are not there.
constexpr unsigned kGridRow = 1u << 23;
struct FlatGrid { unsigned x, y; };
PSF_HD FlatGrid flat_grid(unsigned long long groups)
{
    if (groups <= kGridRow) return {(unsigned)groups, 1u};
    return {kGridRow, (unsigned)((groups + kGridRow - 1) / kGridRow)};
}

// Which rows a workgroup of the row kernels takes: the k-th block of rows of a span of a unit.
// Workgroups go to the eight dies in turn, and the ones of a span read the same state record and
// keys; so with kDieGroups spans of all units or more, a span's workgroups follow each other on one
// die and find them in its cache.  With fewer, the k-th blocks of all spans follow each other, which
// fills the chip evenly.  Either way a span's longest walks come first (k counts from them).
// False: a number that is not there.
struct RowPlace { int unit, span, k; };
constexpr int kDieGroups = 64;
PSF_HD unsigned long long row_groups(int units, int spans, int per_span)
{
    const long long groups = (long long)units * spans;
    return (unsigned long long)(groups >= kDieGroups ? (groups + 7) / 8 * 8 : groups) * (unsigned long long)per_span;
}
PSF_HD bool row_place(unsigned flat, int units, int spans, int per_span, RowPlace &at)
{
    const long long groups = (long long)units * spans;
    long long group;
    if (groups >= kDieGroups) {
        const unsigned turn = flat / 8;
        group = (long long)(turn / (unsigned)per_span) * 8 + flat % 8;
        at.k = (int)(turn % (unsigned)per_span);
    } else {
        group = flat % (unsigned)groups;
        at.k = (int)(flat / (unsigned)groups);
    }
    at.unit = (int)(group % units);
    at.span = (int)(group / units);
    return group < groups && at.k < per_span;
}

// How many workgroups of 64 rows the row kernels have in hand, counted as if each walked as far as the longest:
// in a causal call the k-th block of a span walks k blocks of keys.  state_walk: blocks of keys that applying
// a state is worth (0: no states).  Not causal: every block walks alike.
PSF_HD double row_walks(int units, int spans, int per_span, int causal, double state_walk)
{
    const double blocks = (double)units * spans * per_span;
    return causal ? blocks * ((per_span + 1) / 2.0 + state_walk) / (per_span + state_walk) : blocks;
}

// Rows whose keys several workgroups share (see f32_row_share): a block of 16 rows walks `tiles` tiles of 128 keys of
// its unit, `share` of them a workgroup.  A block of one workgroup finishes its rows itself; the others leave
// their sums in slots, numbered unit by unit, block by block, slice by slice.
PSF_HD int row_slices(int block, int n, int share, int causal)
{
    const int tiles = causal ? block / 8 + 1 : (n + 127) / 128;
    return (tiles + share - 1) / share;
}
PSF_HD int row_slots_before(int block, int n, int share, int causal)    // of the blocks 0 .. block - 1 of a unit
{
    if (!causal) {
        const int s = row_slices(0, n, share, 0);
        return s > 1 ? block * s : 0;
    }
    const int per = 8 * share, q = block / per;                         // blocks of q + 1 slices come `per` together
    return q < 1 ? 0 : per * ((q - 1) * (q + 2) / 2) + (block - q * per) * (q + 1);
}

// Tiles a workgroup takes where few rows' keys are shared out; 0: they are not.  As few as leave no more workgroups than run
// at once and as many slots as there is room for.  One workgroup fills a CU's LDS: without a mask, where all walk alike, 256.
// Under the mask the last slices are short: from three tiles on a second round of 32 costs little; workgroups of one
// tile all last as long, and 240 of them took longer than no sharing.  A tile is 2.8 to 3.4 us of a workgroup's chain and
// the launch that adds the sums 3, so at least two tiles shorter; 2.2 us for rows and at most 32 sketch columns in bf16 (`light`): three.
// us a call, shared and not: causal, 6 units of 384 tokens (288 workgroups of a tile), r = 16 23.1, 18.8; 3 of 512 (240), r = 64 26.6,
// 25.4; 2 of 1536 (288 of six) 35.7, 51.6; no mask, 3 of 768 (288 of three) 36.2, 30.9, 2 of 768 (192) 24.2, 30.5; 1 of 384, bf16, r = 32
// (two tiles shorter) 16.2, 15.0.
inline int row_share(int units, int n, int causal, bool light, unsigned long long room)
{
    const int tiles = (n + 127) / 128, blocks = (n + 15) / 16;
    for (int share = 1; share + (light ? 3 : 2) <= tiles; ++share) {
        const long long slots = row_slots_before(blocks, n, share, causal);
        const long long whole = causal ? (blocks < 8 * share ? blocks : 8 * share) : 0;
        const long long most = !causal ? 256 : 192 + 32 * (share < 3 ? share : 3);
        if (units * (whole + slots) <= most && (unsigned long long)(units * slots) <= room) return share;
    }
    return 0;
}

}  // namespace psf
#endif
