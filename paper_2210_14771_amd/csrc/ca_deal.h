// How a launch over the learned scorers' half strips is divided: the entries of a
// list that a half strip makes, and the waves' shares of the list.  Host and
// device agree on it by these functions.
#pragma once

#include <stdint.h>

namespace ca {

constexpr int kStep = 64;           // positions a wave advances by
constexpr int kStripWaves = 8;      // waves of a workgroup
constexpr int kStripGroups = 256;   // most workgroups of a launch
constexpr int kXcds = 8;

// The half strips of all frames make one list, of which every workgroup takes an
// equal, contiguous share, and of that every wave: it may begin and end within a
// half strip.  An entry is a step; or, where the waves suffice for one each, a
// piece of `grain` steps.  Against 1, 2, 4 or 8 waves to a half strip, by turns of
// workgroups (calls, 2-D network and 1-D): 16 x 1080p, 32 + 32 strips, 78.6 -> 68.5
// and 64.0 -> 56.8 us; 17 x 2390x1201, 17 + 32, 89.9 -> 63.1 and 71.0 -> 53.2; 7 x
// 1623x882, 8 + 15, 31.7 -> 26.0 and 28.2 -> 24.3; 24 SD and 8 4K frames 256 -> 105
// and 191 -> 87; 64 x 1080p, where turns fit, 216 -> 217 and 169 -> 171.
struct StripDeal {
    int32_t groups;        // workgroups per XCD
    int32_t cut;           // least steps of a wave's share (an estimate); 0: pieces
    int32_t grain;         // steps of an entry
    int32_t row, col;      // entries of half a row, of half a column
    int32_t each;          // of a frame; 0 where frames differ: counted by the kernel
    int32_t share, extra;  // every workgroup's entries; this many take `more` more
    int32_t more;
};

// Entries of a half strip of len positions, which needs `halo` more at both ends
// of every piece it is cut into.  Shares of `cut` steps or more cut s steps into
// at most 2 + (s - 2) / cut pieces: those of a half strip that no share holds fit
// the steps dealt for them; of a shorter one, which few shares' ends cut, the
// second piece may take a step more.
constexpr int half_entries(int len, int halo, int cut, int grain)
{
    if (cut == 0) {
        const int fit = kStep * grain - 2 * halo;
        return (len + fit - 1) / fit;
    }
    int s = (len + 2 * halo + kStep - 1) / kStep;
    while (s > cut) {
        int pieces = 2 + (s - 2) / cut;
        pieces = pieces < s ? pieces : s;
        const int need = (len + 2 * halo * pieces + kStep - 1) / kStep;
        if (need <= s)
            break;
        s = need;
    }
    return s;
}
// of the longer half of a row or column
constexpr int extent_entries(int extent, int halo, const StripDeal &d)
{
    return half_entries(extent - extent / 2, halo, d.cut, d.grain);
}
// Where the piece of a half strip of len positions begins that starts at its
// entry `at`, after `before` cuts.
constexpr int piece_start(int len, int halo, int at, int before, int grain)
{
    const int p = kStep * grain * at - 2 * halo * before;
    return p < len ? p : len;
}

// Shares of a list: part k's first entry, and the part that takes an entry, where
// parts take `share` entries and the first `extra` `more` more.
constexpr int share_start(int share, int extra, int more, int k)
{
    return k * share + (k < extra ? k : extra) * more;
}
constexpr int share_of(int share, int extra, int more, int entry)
{
    const int longer = extra * (share + more);
    return entry < longer ? entry / (share + more) : extra + (entry - longer) / share;
}
// The same of the workgroups of a deal, and of its waves, numbered through them.
constexpr int group_of(const StripDeal &d, int entry)
{
    return share_of(d.share, d.extra, d.more, entry);
}
constexpr int wave_start(const StripDeal &d, int wave)
{
    const int group = wave / kStripWaves, k = wave % kStripWaves;
    const int mine = d.share + (group < d.extra ? d.more : 0);
    return share_start(d.share, d.extra, d.more, group)
           + share_start(mine / kStripWaves, mine % kStripWaves, 1, k);
}
constexpr int wave_of(const StripDeal &d, int entry)
{
    const int group = group_of(d, entry);
    const int mine = d.share + (group < d.extra ? d.more : 0);
    return group * kStripWaves
           + share_of(mine / kStripWaves, mine % kStripWaves, 1,
                      entry - share_start(d.share, d.extra, d.more, group));
}

// Cuts of a half strip before its entry `at`, with which a wave's share begins or
// ends, `waves` after the one that has its first entry: shares of a workgroup
// below its waves leave some without any, and none more than one.
constexpr int cuts_before(int share, int at, int waves)
{
    return share < kStripWaves ? at : waves;
}

// A frame's half strips in the list: row and column strips in turn while there are
// both.  Their half strips differ in length, and each costs a wave about the time
// of half a step to begin, so waves that took only columns would end last (64 x
// 1080p, 1-D network: rows and then columns 5 % slower).
struct StripPlace {
    int32_t strip, half;   // strip of its kind
    bool horizontal;
    int32_t at, entries;   // the half strip's entry, of so many
};
constexpr StripPlace strip_place(const StripDeal &d, int n_h, int n_v, int entry)
{
    StripPlace p = {0, 0, true, 0, 0};
    const int both = 2 * (n_h < n_v ? n_h : n_v), two = d.row + d.col;
    int k = 0;
    if (entry < both * two) {
        k = entry / two;
        entry -= k * two;
        p.horizontal = entry < d.row;
        p.at = entry - (p.horizontal ? 0 : d.row);
        p.entries = p.horizontal ? d.row : d.col;
    } else {
        p.horizontal = n_h > n_v;
        p.entries = p.horizontal ? d.row : d.col;
        entry -= both * two;
        k = entry / p.entries;
        p.at = entry - k * p.entries;
        k += both;
    }
    p.strip = k >> 1;
    p.half = k & 1;
    return p;
}
// The half strip that follows, without a division; false at the frame's end, where
// it is the next frame's first (of the same deal).
constexpr bool strip_next(const StripDeal &d, int n_h, int n_v, StripPlace &p)
{
    const int both = n_h < n_v ? n_h : n_v, all = n_h < n_v ? n_v : n_h;
    bool more = true;
    if (p.horizontal && p.strip < both) {
        p.horizontal = false;
    } else {
        p.strip += p.half;
        p.half ^= 1;
        more = p.strip < all;
        p.strip = more ? p.strip : 0;
        p.horizontal = p.strip < both || n_h > n_v;
    }
    p.at = 0;
    p.entries = p.horizontal ? d.row : d.col;
    return more;
}

// The deal of `frames` (at most kDealFrames, so that the list's entries are counted
// in 32 bits) of the n_all frames of these shapes, at most `resident` workgroups
// per XCD.  Shape: W, H, count.
constexpr int kDealFrames = 16384;
template <class Shape>
StripDeal strip_deal(const Shape *shapes, int n_shapes, int frames, int n_all, int n_h, int n_v,
                     int resident, int halo)
{
    if (resident > kStripGroups / kXcds)
        resident = kStripGroups / kXcds;
    const int64_t waves = kXcds * kStripWaves * (int64_t)resident;
    StripDeal d = {resident, 1 << 30, 1, 0, 0, 0, 0, 0, 1};
    auto total = [&] {
        int64_t sum = 0;
        for (int k = 0; k < n_shapes; ++k) {
            d.row = extent_entries(shapes[k].W, halo, d);
            d.col = extent_entries(shapes[k].H, halo, d);
            sum += 2 * ((int64_t)n_h * d.row + (int64_t)n_v * d.col) * shapes[k].count;
        }
        return sum * frames / n_all;
    };
    const int64_t least = total() / waves;
    d.cut = least > 1 ? (int32_t)least : 1;
    int64_t list = total();
    // A piece each, where the last wave takes no more steps then: a wave that ends
    // one half strip and begins another spends about a step's time between (4 x
    // 1080p, four steps a wave: 2-D network 35.7 us a call by steps, 32.9 so).
    if (2 * (int64_t)(n_h + n_v) * frames <= waves) {
        const StripDeal steps = d;
        const int64_t most = (list + waves - 1) / waves;
        d.cut = 0;
        while (d.grain < most && total() > waves)
            ++d.grain;
        const int64_t pieces = total();
        if (pieces <= waves) {
            list = pieces;
        } else {
            d = steps;
        }
    }
    // (few entries spread over the compute units)
    int64_t groups = (list + kXcds - 1) / kXcds;
    d.groups = groups < resident ? (int32_t)groups : resident;
    if (n_shapes > 1)
        return d;
    // Pieces: workgroups that take whole half strips need not meet in the edge
    // words (2 x 1080p, 2-D network: 27.2 us a call otherwise, 26.5 so).  Every half strip
    // makes 1, 2, 4 or 8 entries then, some of them empty.
    const int64_t halves = 2 * (int64_t)(n_h + n_v) * frames;
    const int32_t longer = d.row > d.col ? d.row : d.col;
    const int32_t even = longer <= 2 ? longer : longer <= 4 ? 4 : 8;
    if (d.cut == 0 && longer <= 8 && halves * even <= waves) {
        d.row = d.col = d.more = even;
        list = halves * even;
        groups = (halves + kXcds - 1) / kXcds;
        d.groups = groups < resident ? (int32_t)groups : resident;
    }
    const int all = kXcds * d.groups;
    d.each = 2 * (n_h * d.row + n_v * d.col);
    d.share = (int32_t)(list / d.more / all) * d.more;
    d.extra = (int32_t)(list / d.more % all);
    return d;
}

}  // namespace ca
