// How a d = 128 bf16 attention launch shares its last tiles, and the scratch
// that it shares them in.  Plain C++, no HIP: host rules and host tests use it
// as the kernels' launchers do.
#pragma once

#include <algorithm>
#include <cstdint>

namespace hcms {

// Every query visits its keys as kKeySegments fixed segments of whole key
// blocks, or as one where there are fewer than kKeySegmentMinBlocks blocks.
inline constexpr int kKeySegments = 3;
inline constexpr int kKeySegmentMinBlocks = 12;

// Scratch for splitting a launch's last round of tiles over several
// workgroups (d = 128 bf16): `slots` partial states of
// attention_split_slot_bytes() bytes each (part: slots x 64 KiB, ml: slots x
// 4 KiB, 16-byte aligned) and `counters` ints that are zero between launches.
// part NULL: none, and no tile is split by segments.  At most one launch may
// use one scratch at a time (launches on one stream are ordered).
struct SplitScratch {
    void *part;
    void *ml;
    int *count;
    int slots, counters;
    int n_cu;
    // Tiles at the end of the launch to split: -1 for the launch's own last
    // round (W mod n_cu); otherwise this many (at most W), for a launch whose
    // last tiles close a round that other launches' workgroups share.
    int64_t tail = -1;
};

// A context's scratch: regions of 2 n_cu, n_cu and 3/4 n_cu slots, as many
// counters each.  On 256 CUs that is 63.8 MiB: an allocation of more than 64
// takes 27 us, and 260 to free, 11 and 20 up to there.
inline constexpr int kSplitRegions = 3;
inline int split_slots(int r, int n_cu) { return r == 0 ? 2 * n_cu : r == 1 ? n_cu : n_cu * 3 / 4; }
inline int64_t split_slots_before(int r, int n_cu) {
    int64_t n = 0;
    for (int i = 0; i < r; ++i) n += split_slots(i, n_cu);
    return n;
}
inline int64_t split_slots_all(int n_cu) { return split_slots_before(kSplitRegions, n_cu); }
// Bytes of all of it with states of slot_bytes (4 KiB of them for ml), and
// their part that has to start at zero: the counters, at the end.
inline int64_t split_bytes(int n_cu, int64_t slot_bytes) { return split_slots_all(n_cu) * (slot_bytes + 4); }
inline int64_t split_counter_bytes(int n_cu) { return split_slots_all(n_cu) * 4; }
// Region r of it; mem NULL (none could be had): an empty scratch, with which
// launches split no tile by segments and give the same results.
inline SplitScratch split_region(void *mem, int r, int n_cu, int64_t slot_bytes) {
    SplitScratch s{};
    s.n_cu = n_cu;
    if (!mem) return s;
    char *const base = static_cast<char *>(mem);
    const int64_t first = split_slots_before(r, n_cu);
    s.slots = s.counters = split_slots(r, n_cu);
    s.part = base + first * slot_bytes;
    s.ml = base + first * slot_bytes + s.slots * (slot_bytes - 4096);
    s.count = reinterpret_cast<int *>(base + split_slots_all(n_cu) * slot_bytes + first * 4);
    return s;
}

// Which stream a region belongs to.  Two launches may be in one region only
// one after the other, so a region serves the launches of one stream, and
// moves to another stream behind an event recorded after its last use.  A
// context used on one main and one compute stream, the ordinary one, records
// none: its streams take regions 0 and 1.  Events begin with the first launch
// that finds its region taken; that one takes region 2.  A region used in a
// capture stays with its stream, since its launches are replayed whenever the
// program likes, and a launch in a capture waits for no event from outside.
// A launch that gets no region splits no tile by segments.
class SplitPool {
public:
    // The region for a launch on `stream`, -1: none.  role: 0 for the main
    // stream, 1 for the compute stream.  *wait: the launch's stream has to
    // wait for the region's event first.  own() then makes it the stream's.
    int find(const void *stream, int role, bool capturing, bool *wait) {
        *wait = false;
        for (int r = 0; r < kSplitRegions; ++r)
            if (at_[r].owned && at_[r].stream == stream) return r;
        const int order[2] = {role, 2};
        for (int r : order)
            if (!at_[r].owned) {
                shared_ = shared_ || r != role;
                return r;
            }
        shared_ = true;
        for (int r : order)
            if (at_[r].recorded && !capturing) {
                *wait = true;
                return r;
            }
        return -1;
    }
    void own(int r, const void *stream) { at_[r].owned = true, at_[r].stream = stream; }
    // After a launch in region r: whether to record its event behind it, and
    // that this was done (or failed).
    bool records(int r, bool capturing) {
        at_[r].captured = at_[r].captured || capturing;
        at_[r].recorded = false;
        return shared_ && !at_[r].captured;
    }
    void recorded(int r) { at_[r].recorded = true; }

private:
    struct Use {
        const void *stream = nullptr;
        bool owned = false, recorded = false, captured = false;
    };
    Use at_[kSplitRegions];
    bool shared_ = false;   // some launch found its region taken
};

// Tiles shared by several workgroups (the launch's last, partial round of
// tiles; see plan_split).  Of the `units` = n_split * halves * ways workgroups
// after the whole tiles', workgroup u takes part u % parts, parts = n_split *
// halves: with halves = 2 the first or second 128 queries of tile n_whole +
// part / 2, else the whole tile n_whole + part; and of it with ways = 3 key
// segment u / parts, with ways = 1 all of them.  With 3 ways each writes its
// partial state (the normalised output in the stash layout, and (m, l, E) per
// query) to slot u and counts itself in on its part's counter; the last to
// arrive merges the part's states in segment order, writes the output and
// sets the counter back to zero.
struct TailSplit {
    char *part;      // units slots of 64 KiB (ways = 3)
    char *ml;        // units slots of 256 (m, l, E, 0) per query
    int *count;      // a counter per part, zero between launches
    int n_whole;     // tiles computed whole by one workgroup: the first n_whole
    int n_split;     // tiles split: the last n_split
    int halves;      // 1 or 2
    int ways;        // 1 or 3
    int units() const { return n_split * halves * ways; }
};

// The split of a d = 128 bf16 launch of W tiles on n_cu CUs (one workgroup
// per CU), over nkb key blocks: the last round's t = W mod n_cu tiles are
// shared by more workgroups where that shortens it, in the first of these ways
// that fits (times of launches of t tiles at S = 4096, which take 92 us whole
// with 32 tiles and 97 with 128):
//   three key segments of halves of 128 queries   32 us with 32 tiles
//   three key segments                            49 with 64, 53 with 80
//   halves (half the waves only load)             69 with 96, 77 with 128
//   three key segments in two rounds              90 with 144 and 94 with 160
// Segments need scratch (none: halves or whole tiles, the same results).  The
// last way pays the merge, some 4 us, twice, and gains a tenth of a round:
// with 160 tiles 70 us against 71 whole at S = 2560 and 64 against 61 at 2048,
// with 168 tiles 127 against 135 at S = 6000, 89 against 88 at 3584 and 57
// against 51 at 1536, so it is taken from 40 key blocks on, from 64 with more
// than 5/8 of a round.  With sp->tail >= 0, t is that and the last
// min(tail, W) tiles are split: a launch whose last round is shared with
// another stream's launch splits the tiles that close the pooled rounds, and
// not over two rounds, since both launches' shares are in them: in lanes
// {11, 10} of S = 4971 took 339 us so, 294 with whole tiles, {4, 4} of S =
// 12986 747 and 649; of 36 such chunkings 8 were faster so, by up to 3 %.
struct SplitForm {
    int halves, ways, rounds;   // rounds that the shares may take
};
inline constexpr SplitForm kSplitForms[] = {{2, 3, 1}, {1, 3, 1}, {2, 1, 1}, {1, 3, 2}, {1, 1, 1}};

// Tiles of the last round, which the launch may share.
inline int64_t split_tiles(int64_t W, int n_cu, const SplitScratch *sp) {
    return n_cu < 2 ? 0 : sp && sp->tail >= 0 ? sp->tail : W % n_cu;
}
// Whether a last round of t tiles (rem of them this launch's) can take form f.
inline bool split_fits(SplitForm f, int64_t t, int64_t rem, int nkb, int n_cu, const SplitScratch *sp) {
    if (f.halves * f.ways * t > int64_t{f.rounds} * n_cu) return false;
    if (f.rounds == 2 && ((sp && sp->tail >= 0) || nkb < (8 * t <= 5 * int64_t{n_cu} ? 40 : 64))) return false;
    return f.ways == 1 || (sp && sp->part && nkb >= kKeySegmentMinBlocks &&
                           rem * f.halves * f.ways <= sp->slots && rem * f.halves <= sp->counters);
}
inline TailSplit split_as(SplitForm f, int64_t W, int64_t rem, const SplitScratch *sp) {
    TailSplit p{nullptr, nullptr, nullptr, static_cast<int>(W), 0, 1, 1};
    if (f.halves * f.ways == 1) return p;
    p.halves = f.halves;
    p.ways = f.ways;
    if (p.ways > 1) {
        p.part = static_cast<char *>(sp->part);
        p.ml = static_cast<char *>(sp->ml);
        p.count = sp->count;
    }
    p.n_whole = static_cast<int>(W - rem);
    p.n_split = static_cast<int>(rem);
    return p;
}
inline TailSplit plan_split(int64_t W, int nkb, int n_cu, const SplitScratch *sp) {
    const int64_t t = split_tiles(W, n_cu, sp), rem = std::min(t, W);
    if (rem > 0)
        for (const SplitForm &f : kSplitForms)
            if (split_fits(f, t, rem, nkb, n_cu, sp)) return split_as(f, W, rem, sp);
    return split_as(SplitForm{1, 1, 1}, W, 0, sp);
}

// Compute units that the last round of a launch of these tiles leaves idle.
inline int64_t idle_cus(const TailSplit &p, int n_cu) {
    const int64_t units = int64_t{p.n_whole} + p.units();
    return (n_cu - units % n_cu) % n_cu;
}

// About how long a last round of t tiles takes in form f, in full rounds
// (those run at a lower clock: 160 whole tiles take 0.75 of 256), and, for S =
// 64 nkb keys, how long a full round takes in us.  Launches of 16 to 170 tiles
// of S = 2048 to 75776: six workgroups a tile 0.18 to 0.25, thirds 0.26 (40
// tiles) to 0.36 (80), halves 0.47 to 80 tiles and 0.58 with 128, thirds over
// two rounds 0.64 to 0.72, whole 0.73 to 0.77; 256 tiles of S = 4096 127 us,
// of S = 65536 1700.
inline double form_rounds(SplitForm f, int64_t t, int n_cu) {
    const double x = static_cast<double>(t) / n_cu;
    if (f.ways == 3 && f.halves == 2) return 0.20 + 0.3 * x;
    if (f.ways == 3 && f.rounds == 1) return 0.26 + 0.3 * x;
    if (f.halves == 2) return 0.47 + 0.53 * std::max(0.0, x - 0.31);
    if (f.ways == 3) return 0.65 + 0.6 * std::max(0.0, x - 0.59);
    return 0.73 + 0.65 * std::max(0.0, x - 0.59);
}
inline double round_us(int nkb) { return 1.65 * nkb + 20.0; }

// The split of a launch that copies could ride in, and whether they do.
// Copies that ride take no time of their own, but a tail shared by more
// workgroups leaves them fewer CUs and ends earlier.  Of the forms that fit,
// riding or not, the one expected to end first.  Fitted to the fused and the
// serial plan of 144 chunkings of S = 1400 to 37000 (1.3 % of the pass off, rms):
// a copy kernel moves 9 TB/s, read and written, and takes 2 us more, an idle
// CU copies 12 GB/s.  Two chunks of 12 heads of S = 3178 take 174 us with
// whole tiles, 199 with the segments over two rounds that a launch without
// copies takes.
struct RidingSplit {
    TailSplit split;
    bool ride;
};
inline RidingSplit plan_riding(int64_t W, int nkb, int n_cu, const SplitScratch *sp, double copy_bytes,
                               int n_copies) {
    RidingSplit best{plan_split(W, nkb, n_cu, sp), false};
    const int64_t t = split_tiles(W, n_cu, sp), rem = std::min(t, W);
    if (rem == 0) return best;
    double t_best = 0;
    bool first = true;
    for (const SplitForm &f : kSplitForms) {
        if (!split_fits(f, t, rem, nkb, n_cu, sp)) continue;
        const double tail = form_rounds(f, t, n_cu) * round_us(nkb);
        if (first) t_best = tail + 2 * copy_bytes / 9e6 + 2 * n_copies;   // the copies behind it
        first = false;
        const TailSplit p = split_as(f, W, rem, sp);
        const int64_t idle = idle_cus(p, n_cu);
        if (idle < std::max(1, n_cu / 8)) continue;
        const double end = std::max(tail, tail * (f.rounds - 1) / f.rounds + copy_bytes / (12e3 * idle));
        if (end < t_best) {
            t_best = end;
            best = RidingSplit{p, true};
        }
    }
    return best;
}

}  // namespace hcms
