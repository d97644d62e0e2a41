// Where the rows of a segment come from in one decode step, and which unit a wavefront of a ranked launch works on.  Plain
// integer rules, apart from the kernels so that they can be compiled and enumerated on the host.
#pragma once

#include "fast_div.hpp"

namespace pkv {

// Virtual row numbering of a segment under pruning: rows [0, perm) are the permanent slots, rows
// perm + j are ring slot j (the last d+1 slots of the segment).  r_new is the row of the token stored
// in this step, r_mask the row of a token pruned in this step (-1 if none).
struct RingMap {
    int shift;    // ring slot j is physical slot perm + j + shift
    int r_new;
    int r_mask;
};

struct RowSource {
    bool valid;      // the row takes part in this step
    bool from_new;   // read from k_new / v_new instead of `slot`
    int slot;        // slot of the segment
};

// Row r of the block that starts at row r0 < len.  len_old rows were stored before this step (under pruning: permanent
// ones); app: the step stores a token.  A row that does not take part is read like the block's first one and ignored, so
// that a load needs no branch: no load of the step reads the slot that the step writes.
template <bool EV>
__device__ __forceinline__ RowSource row_source(int r, int r0, int len, int len_old, bool app, const RingMap& ring) {
    RowSource s;
    s.valid = r < len && (!EV || r != ring.r_mask);
    const int x = s.valid ? r : r0;
    s.from_new = EV ? x == ring.r_new : app && x == len_old;
    s.slot = EV && x >= len_old ? x + ring.shift : x;
    return s;
}

// The slot that a wavefront reads for row r of the block that starts at row r0 < len, where the new row (r_new, -1: none) does not
// come from the cache: its own, and for the new row and rows that take no part the block's first one or, if that is the new one, a
// neighbour of it.  No slot that the step writes; len > 1 or r_new < 0.
template <bool EV>
__host__ __device__ __forceinline__ int row_slot(int r, int r0, int len, int len_old, int r_new, const RingMap& ring) {
    const int other = r0 != r_new ? r0 : r0 > 0 ? r0 - 1 : 1;
    const int x = r < len && (!EV || r != ring.r_mask) && r != r_new ? r : other;
    return EV && x >= len_old ? x + ring.shift : x;
}

// How many units the unit counts in at its segment: of the `units` consecutive ones of a workgroup, of which it is number `at` and
// unit hu of the HU of its segment, the first of each segment speaks for all of that segment, the others for none.  (Units of one
// segment are alive together.)
__host__ __device__ __forceinline__ int counted_units(int at, int units, int hu, int HU) {
    if (at > 0 && hu > 0) return 0;
    return units - at < HU - hu ? units - at : HU - hu;
}

// Rows that a step attends to in a segment of cap slots, len_old of them stored before (under pruning: permanent ones), and whether
// the step stores a token: without pruning while a slot is left, with it if the ring of d + 1 slots fits behind the kept entries.
struct StepRows { bool app; int rows; };
template <bool EV>
__host__ __device__ __forceinline__ StepRows step_rows(int len_old, int cap, int base, bool append, int t, int d) {
    if (!EV) { const bool app = append && len_old < cap; return {app, len_old + (app ? 1 : 0)}; }
    const int ring0 = cap - (d + 1);
    const bool app = base >= 0 && ring0 >= base && len_old <= ring0;
    return {app, app ? len_old + (t < d + 1 ? t : d + 1) : 0};
}

// Whether `entries` >= 2 are within the target of step t, max(1, floor((2 base (N + t) + N) / (2 N))): without the division, which
// took some two hundred instructions at the start of every unit.
__host__ __device__ __forceinline__ bool within_target(int entries, int base, int N, int t) {
    return 2ll * N * entries <= 2ll * base * ((long long)N + t) + N;
}

// Ranked launches: the segments are cut into groups of gsz; in each the units (HU per segment) of the n4 longest get four
// wavefronts, those of the next n2 two and the others one; `by_length` false: in index order instead.  Workgroups of four
// wavefronts; the units of a class follow each other without gaps, so a workgroup may hold units of two segments, and the
// last of a class fewer than fit.
struct RankedShape { int gsz, n4, n2; bool by_length, large = false; };   // large: keys of more than 192 KB per head

// The shape of a launch of `units` units (more than four per compute unit) on `cus` compute units, each with room for `resident`
// wavefronts (20 of the plain bf16 step, else 16); N prompt positions with rows of row_bytes, gsz given.  More wavefronts per unit
// shorten the longest units, with which a launch ends; but each start costs, and a launch loses most on a second round that is
// nearly empty.  Only the prompt's length is known here, so the rules have to hold for long rows and for short ones.  Times
// against a quarter of the segments with four wavefronts and the others with two up to 1638 units, an eighth to a sixteenth each up
// to 8192, one each beyond, with a count of each unit by itself; 256 compute units, bf16, D 128, lengths of the segments within a
// factor 30 / 3 / equal:
//   prompts of more than 4096 positions with keys of more than 1 MB per head, while a quarter with four and the others with two are no more
//     than a third over a round of 16: those, except where they just fit a round of 20 (1707 to 2275 units: 2048, 400 rows, x1.11, an
//     eighth each 1.03; 2240, 250 rows 1.12 and 0.98), and for keys of more than 192 KB up to 4.9 units per compute unit.  Other shapes have fewer
//     workgroups, each of which counts, and win on few rows, but not on the many that such prompts keep, against a quarter and the others:
//     3200 units, an eighth, N5000, 250 rows 0.93, 400 1.01, 500 1.10, 1000 1.11; 2560, 1000 rows 1.07; 1120 units, 3/16, N818, 40 rows 0.88, 160 rows 1.01,
//     400 rows 1.04, N2000, 1000 rows 1.12; 1200, N1000, 400 rows 1.12;
//   of keys of more than 192 KB from there to 7.1 units per compute unit, a quarter each: with the others two / a quarter each / 3/16 each
//     1280 units, 40 rows x1.11 / 0.89 / 0.84, 400 rows 1.00 / 1.05 / 1.09; 1440 of 60 rows 1.13 / 0.88 / 0.83, of 400 1.01 / 0.96 / 0.99; 1760 of 60 1.16 / 0.92 /
//     0.81, of 400 1.06 / 1.00 / 1.04, an eighth 1.10;
//   shorter prompts of up to 6.4 units per compute unit, 3/16 with four and as many with two, the rest one: 1600 units of 136 rows
//     x0.87 / 0.95 / 0.85 (a quarter and the others 0.89 / 0.92 / 0.90), of 41 0.72 / 0.73 / 0.77 (0.86 / 1.12 / 0.80);
//   from 8.6 to 11.4 units per compute unit (9.1 for keys of more than 192 KB), where an eighth each is a fifth over a round of 16: a quarter with two, the others
//     one: 2400 units, N400, 40 rows an eighth 1.02 on average, at worst 1.10, a quarter with two 0.91, 1.01; 160 rows 0.99 and 0.95; 2560, 40 rows 1.02
//     and 0.91; 2880, N1000 0.99 and 0.97;
//   beyond, an eighth each while that fits one round of 16, then what does, but a sixteenth: 2048 units of 136 rows x0.90 / 0.91 / 0.90,
//     of 26 0.65 / 0.64 / 0.66; 3648 of 300 an eighth 0.98 on average, a sixteenth 0.97, none 0.99; 4096 of 136 fp32 rows 0.98, none 1.11;
//   the sixteenth up to two rounds of 16, except for the plain bf16 step on keys of up to 192 KB, which has what fits its own round
//     and then one each: 6144 units of 300 rows 0.97 on average, none 0.98 (8 % apart for lengths within a factor 30); of 136 rows 0.90,
//     none 0.90, of 41 0.70 and 0.64;
//   all others one each, and from 16 units per compute unit on prompts with keys of up to 96 KB per head in index order: finding
//     the rank costs too much there, 8192 units of 26 rows x0.65, by length 0.75, of 41 rows 0.78 and 0.85.
constexpr int kRankedResident = 20;
inline void ranked_shape(RankedShape& s, long long units, long long cus, int N, int row_bytes, int resident = 16) {
    const double per_unit = 16.0 * cus / units;               // wavefronts of one round of 16 for each unit
    const bool large = s.large = N * row_bytes > 192 << 10;
    double f4 = 0, f2 = 0;
    s.by_length = N * row_bytes > 96 << 10 || units < 16 * cus;
    const bool longest = N > 4096 && N * row_bytes > 1 << 20;
    if (longest ? per_unit >= 0.75 && (per_unit <= 1.8 || per_unit >= 2.4) : large && per_unit >= 3.25) { f4 = 0.25; f2 = 0.75; }
    else if (large && per_unit >= 2.25) f4 = f2 = 0.25;
    else if (per_unit >= 2.5) f4 = f2 = 0.1875;
    else if (per_unit >= 1.4 && per_unit <= (large ? 1.75 : 1.85)) f2 = 0.25;
    else if (s.by_length && per_unit >= (large || resident == 16 ? 0.5 : 1)) f4 = f2 = per_unit > 1.5 ? 0.125 : per_unit < 1.25 ? 0.0625 : (per_unit - 1) / 4;
    else if (s.by_length && units <= resident * cus) f4 = f2 = ((double)resident * cus / units - 1) / 4;
    s.n4 = (int)(s.gsz * f4 + 0.5);
    s.n2 = (int)(s.gsz * f2 + 0.5);
    if (s.n2 > s.gsz - s.n4) s.n2 = s.gsz - s.n4;
}

// LDS that a bf16 launch of `waves` wavefronts asks for beyond its own 2 KB, to have four workgroups resident and not five.
// Launches of several rounds of long rows are bound by memory, and that serves fewer streams of rows faster: lengths within a factor
// 30, four against five, 6144 units of 300 rows x0.986, 9216 0.973, 12 800 1.00, of 500 0.985, 0.977, 0.991; less unequal ones x0.99 ...
// 1.01.  Shorter rows wait for their starts (5440 units of 41 rows x1.11, 12 800 1.03), and up to an eighth over one round filling it
// counts more.
inline int ranked_lds(const RankedShape& s, long long waves, long long cus) {
    const long long round = kRankedResident * cus;
    return s.large && s.by_length && 8 * waves > 9 * round ? 31 << 10 : 0;
}

__host__ __device__ __forceinline__ int ranked_blocks(const RankedShape& s, int HU) {   // per group
    return s.n4 * HU + (s.n2 * HU + 1) / 2 + ((s.gsz - s.n4 - s.n2) * HU + 3) / 4;
}

// Grouped launches: a workgroup of W wavefronts takes as many units of a segment as its rows leave wavefronts for.  A unit has one
// wavefront up to kSpread blocks of rows, two up to twice as many, and so on, and no fewer than leave the HU units of a segment with
// a workgroup's.  (1024 units of 32 segments, 3 / 4 / 5 / 6 blocks, us: N200 14.3 / 12.2 / 12.2 / 12.2 at 50 %, 10.9 / 10.0 / 10.2 / 10.4 at 30 %; N300 16.4 /
// 16.4 / 14.8 / 14.8 and 13.6 / 14.1 / 12.2 / 12.6, 19.1 / 17.9 / 19.3 / 19.1 for lengths within a factor 3; 960 of 40, N250 16.1 / 15.2 / 16.2 / 16.3.)
constexpr int kSpread = 4;
__host__ __device__ __forceinline__ int active_waves(int blocks, int HU, int W) {
    int n = 1;
    while (n < W && (blocks > n * kSpread || n * HU < W)) n *= 2;
    return n;
}
// Workgroups of W wavefronts for a segment whose units (HU) have `waves` each, and the unit of a wavefront of one of them.  The last
// workgroup of a segment may have wavefronts to spare: they stay for its barriers and read what the segment's last unit reads.
__host__ __device__ __forceinline__ int grouped_blocks(int HU, int waves, int W) { return (HU * waves + W - 1) / W; }
struct GroupedUnit { int hu; bool live; };
__host__ __device__ __forceinline__ GroupedUnit grouped_unit(int block_of_segment, int wv, int waves, int W, int HU) {
    const int sh = __builtin_ctz(waves), u = block_of_segment * (W >> sh) + (wv >> sh);   // (a division each at the start of every unit otherwise)
    return {u < HU ? u : HU - 1, u < HU};
}
// Workgroup (x, y) of n_seg * HU: the first units of all segments, then the next ones, so that the counts of a segment come apart and the
// workgroups that are not needed come last.  Its segment: an even number of them is turned by one from y to y, else each would be on
// one or two XCDs.
inline int grouped_turn(int n_seg) { return n_seg % 2 == 0; }
__host__ __device__ __forceinline__ int grouped_segment(int x, int y, int turn, FastDiv n_seg) { return div_mod(x + turn * y, n_seg).r; }
// Whether a launch is grouped.  The units of a segment are counted by atomics on its word of lens, and a cache line of these words
// takes about 8 ns for each: 1024 units of 18 rows in one line 13.4 us, without the count 6.2.  A grouped launch counts less where the
// capacity leaves few wavefronts to a unit; where it does not (much room for new tokens, which the launch does not know) it has the order of
// its workgroups alone.  So on keys of up to 26 KB per head where three quarters of a unit per compute unit are counted in a line, up to 50 KB
// where one is, at least half of the launch's, and a segment has 16 units, and up to 76 where more than 1.5 and half are and the launch has
// more than 2, 100 where it has more than 2.75.  us per step, one unit per workgroup / grouped, room for 8 tokens and for 256, D 128, 40 % within a factor 3:
//   1024 units of 32 segments, N60 13.3 / 7.3 and 13.1 / 10.8, N130 14.2 / 9.3 and 13.5 / 12.4, N200 14.7 / 12.6 and 14.9 / 14.3, N300 17.7 / 16.6 and 17.7 /
//     16.8, N400 19.8 / 20.2 and 19.9 / 19.7, at 10 % 14.4 / 7.9; 960 of 40, N300 15.4 / 15.1 and 15.6 / 15.0, N400 17.5 / 18.4 and 17.9 / 17.9, at 10 % x0.66; fp32 N130 17.6 /
//     16.0 and 18.0 / 16.7;
//   768 of 24, N60 10.8 / 7.1 and 10.3 / 10.5, N200 12.9 / 10.4 and 12.6 / 12.0, N300 14.7 / 12.6 and 14.7 / 14.0; 608 of 19, N60 10.6 / 7.0 and 10.1 /
//     10.5, N300 13.3 / 13.2 and 12.9 / 13.7, at a factor 30 11.4 / 10.3 and 10.7 / 12.1, but N400 of that 12.8 / 16.1;
//   512 of 16, N60 10.5 / 6.9 and 9.9 / 10.3, N200 11.3 / 9.2 and 10.8 / 10.9, N300 12.3 / 11.4 and 11.5 / 11.9 (factor 30 with room, N200 10.3 / 11.0, N300 10.7 /
//     11.2); 416 of 13, N60 9.4 / 6.7 and 8.7 / 9.2, N200 9.7 / 8.7 and 9.3 / 9.5;
//   longer prompts gain too where few rows are kept, and lose where many of unequal lengths are: 864 units of 36 segments, N350 at a factor 30 14.1 / 16.3; of 400 ... 3000 positions 832 of 26
//     x0.92 ... 1.11 on average, at worst 1.09 ... 1.28, 960 of 40 0.91 ... 1.05 and 1.04 ... 1.10;
//   fewer in a line, on average and at worst of 7 spreads, budgets and rooms: 192 of 192 units, N100 x0.96 and 1.03, N200 1.02, 1.07; 256 of 256 0.90, 1.02 and 0.96, 1.03; 288 of 288 (24
//     segments of 12), N100 0.93, 1.02 and N200 1.02, 1.12; 384 of 960 (80 of 12) 0.83, 1.02 and 0.95, 1.17; 256 of 1024 (128 of 8), N100 0.93, 1.03, N130 0.97, 1.16; 512 of 1024 (64 of
//     16), N200 0.87, 1.07; 128 of 1024 (eight sequences, 4 of 32 layers), N60 7.0 / 7.6 us, N200 11.7 / 14.4; 1024 segments of one unit, N60 6.7 / 7.6.
inline bool units_grouped(long long n_seg, int HU, int nl, int L, long long cus, int N, int row_bytes) {
    const long long units = n_seg * HU, apart = nl == L ? 32 : nl < 32 ? nl : 32, line = (n_seg < apart ? n_seg : apart) * HU;   // units in a line of lens
    const long long keys = (long long)N * row_bytes;
    if (units > 4 * cus) return false;
    if (keys <= 26 << 10) return 4 * line >= 3 * cus;
    if (keys <= 50 << 10) return line >= cus && 2 * line >= units && HU >= 16;
    return units > 2 * cus && 2 * line > 3 * cus && 2 * line > units && keys <= (4 * units > 11 * cus ? 100 : 76) << 10;
}

// Length class of a segment: quarter octaves of its capacity below that of the longest one, the last class open.
constexpr int kLengthClasses = 16;
__host__ __device__ __forceinline__ int length_class(int cap, int longest) {
    const auto quarters = [](int x) { return (int)(__builtin_bit_cast(unsigned, (float)x) >> 21); };   // exponent, two bits
    const int d = quarters(longest) - quarters(cap);
    return d < kLengthClasses - 1 ? d : kLengthClasses - 1;
}

struct RankedUnit {
    bool live;       // the wavefront has a unit
    int UW;          // wavefronts that share it (the same for the whole workgroup)
    int first, n;    // the group's first segment and number of segments
    int rank, hu;    // which of them, longest first, and which unit of it
};

__device__ __forceinline__ RankedUnit ranked_unit(int block, int wv, const RankedShape& s, int HU, int n_seg) {
    RankedUnit x;
    const int b4 = s.n4 * HU, b2 = (s.n2 * HU + 1) / 2, bpg = ranked_blocks(s, HU);
    const int grp = block / bpg, j = block - grp * bpg;
    int r0, nc, u;                                        // the class's first rank and segments, the unit in it
    if (j < b4) { x.UW = 4; r0 = 0; nc = s.n4; u = j; }
    else if (j < b4 + b2) { x.UW = 2; r0 = s.n4; nc = s.n2; u = 2 * (j - b4) + wv / 2; }
    else { x.UW = 1; r0 = s.n4 + s.n2; nc = s.gsz - r0; u = 4 * (j - b4 - b2) + wv; }
    x.first = grp * s.gsz;
    x.n = n_seg - x.first < s.gsz ? n_seg - x.first : s.gsz;
    const int r = u / HU;
    x.hu = u - r * HU;
    x.rank = r0 + r;
    x.live = r < nc && x.rank < x.n;
    return x;
}

// Blocks of a grouped-query unit; one without rows has an output too.
__host__ __device__ __forceinline__ int row_blocks(int rows, int block) { return rows < 1 ? 1 : (rows + block - 1) / block; }

// Fewest blocks of a wavefront of a grouped-query launch.  A wavefront costs a start and a partial result of `width` numerators to
// add up.  One block each while the launch is a wait on chains, up to half the wavefronts, and the merge has up to 16 pieces for
// each of its 2048 / width groups; else two.  us per call with two / one, D 128: 64 units of width 512, 200 blocks 12.7 / 10.0, 900 12.1 /
// 11.0, 1400 13.0 / 13.1; 8 units, 400 12.0 / 11.2, 700 12.0 / 12.7, 2000 16.0 / 20.7; width 1024, 16 units, 200 13.5 / 11.7, 700 15.3 / 16.7,
// 128 units, 900 15.2 / 13.9, 1100 14.7 / 15.6.  (B4 H32/8 N8192, one layer a call, 2300 blocks: four 8 % slower than two.)
__host__ __device__ __forceinline__ int gqa_least(int all, int waves, int units, int width) {
    return 2ll * all <= waves && (long long)all * width <= 32768ll * units ? 1 : 2;
}
// Blocks of a wavefront when the `all` blocks are dealt out evenly.
__host__ __device__ __forceinline__ int gqa_share(int all, int waves, int least = 2) {
    const int even = (int)(((long long)all + waves - 1) / waves);
    return even < least ? least : even;
}

// The stream of blocks of a grouped-query launch: segment by segment, the head groups (HU) of a segment one after the other, nb
// blocks each, `first` blocks per head group in the segments before.  Wavefront w has blocks [w * share, (w + 1) * share).
struct GqaPlace { int hu, blk; };
__host__ __device__ __forceinline__ GqaPlace gqa_place(int x, int first, int nb, int HU) {   // of block x, which lies in the segment
    const int rem = x - first * HU, hu = rem / nb;
    return {hu, rem - hu * nb};
}
enum class GqaNext { block, head, segment };             // what the following block is the next of
__host__ __device__ __forceinline__ GqaNext gqa_next(int& blk, int& hu, int& seg, int nb, int HU) {
    if (++blk < nb) return GqaNext::block;
    blk = 0;
    if (++hu < HU) return GqaNext::head;
    hu = 0;
    ++seg;
    return GqaNext::segment;
}
// Where wavefront w leaves what it has of a unit that it shares with others: along the stream one of the two goes up from one
// piece to the next, so no two pieces share a slot.
__host__ __device__ __forceinline__ int gqa_slot(int w, int seg, int hu, int HU) { return w + seg * HU + hu; }
struct GqaPieces { int wave, n; };                       // the first wavefront that has some of a unit, and how many do
__host__ __device__ __forceinline__ GqaPieces gqa_pieces(int first, int nb, int hu, int HU, int share) {
    const int b0 = first * HU + hu * nb, w = b0 / share;
    return {w, (b0 + nb - 1) / share - w + 1};
}
// Workspace in words: [0] the share, from kGqaHdr the first block / HU of every segment and their total (n_seg + 1), then, 16-word
// aligned, the slots: [G][D] numerators, [G][2] max and denominator.
constexpr int kGqaHdr = 16;
__host__ __device__ inline int gqa_partial_word(int n_seg) { return (kGqaHdr + n_seg + 1 + 15) / 16 * 16; }

// The workspace of a grouped-query launch starts at the first multiple of 16 in the caller's, which may have any address: partial
// results are written and read by 16 bytes.  The size query adds kGqaWsAlign bytes for it.
constexpr int kGqaWsAlign = 16;
inline unsigned long long gqa_ws_base(unsigned long long address) { return (address + kGqaWsAlign - 1) / kGqaWsAlign * kGqaWsAlign; }

}  // namespace pkv
