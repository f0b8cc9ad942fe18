// Tile-schedule arithmetic shared by the kernels and their launchers: plain
// constexpr integer functions (no HIP types), so that the same definitions
// compile for the GPU and, in the tests, with the host C++ compiler.
#pragma once

namespace cattn {

constexpr int imin(int a, int b) { return a < b ? a : b; }
constexpr int imax(int a, int b) { return a > b ? a : b; }

// Rows per (batch, head) of each backward workspace row: S padded to a
// multiple of 32 (padding entries hold zeros), so that 32-row tiles of it can
// be copied whole.
constexpr int ws_rows(int S) { return (S + 31) / 32 * 32; }

// Ring of LDS buffers streamed over iterations 0 .. L-1 by `split` parts, each
// of which copies one tile per iteration (a part without a tile of its own in
// the last one copies another's).  The tiles of iteration x are copied at the
// top of iteration x - ahead (iterations 0 .. ahead-1 before the loop), each
// wave issuing the same number of copies per part tile, and a wave's copies
// complete in issue order.  Iteration i reads the tiles of iterations
// i .. i+need.  At the top of iteration i a wave may therefore leave in flight
// the part tiles of iterations i+need+1 .. i+ahead-1; this is their number.
constexpr int ring_in_flight(int i, int L, int split, int ahead, int need) {
  int k = 0;
  for (int x = i + need + 1; x <= i + ahead - 1; ++x) k += x < L ? split : 0;
  return k;
}
// The common case, when all of those iterations exist (i + ahead <= L): a
// compile-time count.
constexpr int ring_in_flight_full(int split, int ahead, int need) { return (ahead - 1 - need) * split; }

// The bf16 attention kernels: forward, dQ, dK/dV.
enum class Pass { kFwd, kDq, kDkdv };

// Parts (1, 2 or 4) that a bf16 work group's four waves split the other axis
// into.  A split work group owns 64 (two parts) or 32 (four) rows instead of
// 128, so that a grid of few work groups fills the GPU and its heaviest wave's
// run over the other axis is a half or a quarter as long; the price is as many
// rings to copy, the LDS for them and the parts' merge.  What decides is
//  * the tiles to share, nt: with one or two a part has none or one, and the
//    merge costs more than the run it shortens;
//  * 32-row groups per CU, g = BH nt / CUs: up to 1 (2 at D = 64) the four-part
//    work groups are resident from the start, up to 4 the two-part ones (LDS,
//    registers);
//  * with the mask, nt again: a long sequence's heaviest tile runs alone at the
//    end of the grid, so the shorter run pays even where work groups queue.
// Measured, unsplit / two / four parts, us (F forward, Q dQ, K dK/dV; c causal):
//   few tiles  c S64 D64, g 1: F 4.2 / 4.6 / 4.6, K 4.9 / 5.6 / 5.5; c S128 D64, g 1: F 5.2 / 5.1 / 4.7,
//              K 6.8 / 6.2 / 5.5, g 2: F 5.3 / 5.3 / 5.7, K 7.0 / 6.5 / 7.5; c S384 D64, g 1.5: K - / 8.8 / 7.7
//   four, two  S256 D64, g 2: F 7.1 / 6.0 / 5.8, Q 8.3 / 7.0 / 8.0; c S512 D64, g 2: Q 10.8 / 8.9 / 8.7;
//              S1024 D64, g 2: Q 17.8 / 12.9 / 12.9; c S2048 D64, g 3: F 28.5 / 18.1 / 16.9,
//              K 41.6 / 25.8 / 25.1; S2048 D64, g 3: F 27.9 / 23.0 / 24.5; c S128 D128, g 2: F 7.9 / 7.0 / 10.7
//   two, none  c S512 D64, g 4: F 10.2 / 8.3, Q 12.1 / 11.2, K 14.5 / 12.4; c S1024 D64, g 6: F 16.9 / 13.6,
//              Q 18.2 / 19.9, K 24.4 / 23.9, g 7: F 17.4 / 16.4, K 24.5 / 26.1; c S4096 D64, g 9: F 57.8 / 54.2,
//              g 7: Q 59.4 / 58.2, K 82.4 / 68.7; S2048 D64, g 6: F 38.2 / 33.7, Q 45.8 / 45.8, K 61.2 / 57.7,
//              g 7: F 40.1 / 43.3, K 64.5 / 69.3; c S256 D128, g 3: F 10.7 / 9.4, Q 13.7 / 13.6, K 16.6 / 15.0;
//              c S222 D64, g 2.3: F 6.8 / 6.3; c S154 D64, g 2: K 8.7 / 7.6; c S147 D64, g 2.6: K 8.9 / 8.9; c S2855
//              D64, g 6.3: Q 43.3 / 38.2; c S1659 D64, g 6.3: K 37.9 / 34.8; S261 D64, g 2.3: F 8.1 / 7.5, K 11.0 /
//              10.1; S187 D64, g 3.5 (298 work groups of 128): F 7.9 / 7.5, K 11.1 / 10.2; S371 D64, 72 heads: K
//              13.1 / 12.4, S377, 75 heads: 13.6 / 15.4;
//              S256 D128, g 3: F 11.1 / 11.6, Q 14.5 / 16.1; S512 D128, g 4: F 16.7 / 16.8, Q 21.4 / 22.9,
//              K 36.9 / 26.5; S2048 D128, g 5: F 59.1 / 61.5, K 102 / 105
constexpr int split_parts(Pass pass, int D, bool causal, int BH, int S, int cus) {
  const int nt = (S + 31) / 32;
  if (nt < 3) return 1;
  // largest g of four parts, and twice that of two
  int four = 1, two = 4;
  if (D == 128) {
    if (nt >= (causal ? 8 : 16) || (causal && pass == Pass::kFwd && nt >= 4)) two = 8;
  } else if (pass == Pass::kFwd) {
    if (nt >= (causal ? 8 : 16)) four = 2;
    if (causal && nt >= 8) two = 8;
    if (nt >= 10) two = 12;
    if (causal && nt >= 32) two = nt >= 128 ? 20 : nt >= 64 ? 18 : 14;
    if (causal && nt == 7) two = 6;
    if (!causal && nt == 9) two = 5;
  } else if (pass == Pass::kDq) {
    if (nt >= (causal ? 16 : 32)) four = 2;
    if (causal && nt >= 12) two = 6;
    if (nt >= 16) two = 8;
    if (causal && nt >= 20) two = nt >= 40 ? 12 : nt >= 36 ? 11 : nt >= 32 ? 10 : 9;
    if (causal && nt >= 64) two = nt >= 112 ? 16 : nt >= 88 ? 14 : 13;
  } else {
    if (nt >= (causal ? 8 : 32)) four = 2;
    if (causal && nt >= 5) two = nt >= 12 ? 9 : nt >= 8 ? 8 : 6;
    if (!causal && nt >= 16) two = 8;
    if (nt >= 24) two = causal && nt >= 64 ? 16 : causal && nt >= 48 ? 13 : 12;
    if (!causal && (nt == 5 || nt == 7 || nt == 9)) two = nt == 5 ? 6 : 5;
    // (a head's work groups then share a chiplet, or two of them)
    if (!causal && nt >= 7 && BH % 4 == 0) two = imax(two, 8);
  }
  if (D == 64 && causal && nt >= 48) four = 3;
  const long long g32 = (long long)BH * nt, g64 = (long long)BH * ((S + 63) / 64);
  if (g32 <= (long long)four * cus) return 4;
  // (a short last tile can give an unsplit grid a second round where two parts need no third)
  if (pass != Pass::kDq && D == 64 && !causal && nt >= 5 && (long long)BH * ((S + 127) / 128) > cus &&
      g64 <= 2LL * cus)
    return 2;
  // (an odd tile over: up to an eighth more 64-row groups than CUs is no loss yet)
  if (two == 4 && nt >= 8) return g32 <= 2LL * cus ? 2 : 1;
  // (a short last tile can give an unsplit grid a third round where two parts need no fifth:
  // forward without the mask, B1 H40 S1568 D64 40.2 / 35.1)
  if (pass == Pass::kFwd && D == 64 && !causal && nt >= 12 && (long long)BH * ((S + 127) / 128) > 2LL * cus &&
      g64 <= 4LL * cus)
    return 2;
  return 4 * g64 <= (long long)two * cus ? 2 : 1;
}

// Order in which a grid of n work groups takes the work items, when items are
// ranked heaviest first (rank 0 = most work).  Work groups are placed on the
// GPU in rounds of `band` (one per compute unit): group b shares its compute
// unit with groups b +- band, b +- 2 band, ...  Every other round walks the
// ranks backwards, so that a compute unit that receives one of the heaviest
// items in one round receives one of the lightest of the next.  Round 0 walks
// forwards, except in a grid of two rounds (with `pair_up`): there it walks
// backwards and the second round, which falls on the first units, forwards, so
// that it reaches those with the least before it.  Over 800 shapes of one to
// two rounds that was 0-20% faster than round 0 forwards (dQ, dK/dV; the
// forward 0-8%); in grids of three to four rounds, where the last round starts
// as units fall free, it was up to 14% slower (dQ, B1 H104 S1024 D128).  The
// walk is backwards in steps of kXcdGroup, keeping each rank's position within its
// group of kXcdGroup: work groups are dealt to the GPU's kXcdGroup chiplets
// (each with its own L2) round-robin by index, and a rank keeps the chiplet of
// the same-numbered group, so the tiles of one head, which share K/V or
// Q/dO, stay in one L2.  band <= 0 keeps the plain heaviest-first order.  A
// permutation of [0, n).
constexpr int kXcdGroup = 8;
constexpr int banded_rank(int bid, int n, int band, bool pair_up = true) {
  if (band <= 0) return bid;
  const int r = bid / band, p = bid % band;
  const int first_back = pair_up && n > band && n - band <= band ? 0 : 1;
  if (((r - first_back) & 1) != 0) return bid;
  const int size = n - r * band < band ? n - r * band : band;
  if (size % kXcdGroup != 0 || band % kXcdGroup != 0) return r * band + size - 1 - p;
  return r * band + (size / kXcdGroup - 1 - p / kXcdGroup) * kXcdGroup + p % kXcdGroup;
}

// The `band` argument of the causal forward and dQ for a grid of n work groups
// of 128/parts queries.  None for one round, where the order changes nothing
// but costs its arithmetic (1-2% of the smallest grids), and none for a split
// grid of over three rounds, which is not resident (forward, D = 64, two parts,
// banded / plain: 3-8% slower).  kNoPairUp is added where the heaviest-first
// ranks of a two-round grid are not heaviest first: the last of two or three
// unsplit tiles, if of at most 96 queries, has the longest run but idle waves,
// so less work than the tiles before it (forward, D = 128, paired up / round 0
// forwards: B1 H205 S160 16% slower, B1 H171 S192 12%, B1 H128 S300 10%; four
// tiles and more, whatever the last, 4-11% faster: B1 H80 S450 14.6 / 15.4 us).
constexpr int kNoPairUp = 1 << 24;
constexpr int query_band(long long n, int parts, int S, int cus) {
  if (n <= cus || (parts > 1 && n > 3LL * cus)) return 0;
  return cus + (parts == 1 && S < 384 && (S - 1) % 128 + 1 <= 96 ? kNoPairUp : 0);
}

// Order of a grid of BH heads x ntiles tiles that is too large to be resident
// at once: heads are taken hg at a time (the last group may be smaller), and
// inside a group the ranks 0 .. ntiles-1 of all its heads are dealt rank by
// rank.  Work groups that run together then share few enough heads for the
// streamed operands of those on one chiplet to stay in its L2.  A permutation
// of the heads' tiles for any hg >= 1; hg >= BH is the plain rank-by-rank order.
struct HeadRank {
  int bh, rank;
};
constexpr HeadRank grouped_rank(int bid, int BH, int ntiles, int hg) {
  const int g = bid / (hg * ntiles), rem = bid - g * (hg * ntiles);  // (hg * ntiles fits an int: work_order)
  const int n = imin(hg, BH - g * hg);
  return HeadRank{g * hg + rem % n, rem / n};
}

// The `order` argument of a grid of BH heads x n_tiles tiles, per_cu work
// groups resident per CU: `otherwise` (a band or 0), or the heads taken up to
// kHeadGroup at a time (the negative of their number), where the grid takes more
// than one round, there are at least three groups of heads and sequences are
// short enough that a group's heads (eight per chiplet) stream from its 4 MB L2.
// Forward + dQ + dK/dV, over all heads / 64 at a time, us: B16 H16 S512 D128 156 / 138, B16 H16
// S1024 D128 432 / 401, B32 H16 S200 D128 113 / 101, B32 H16 S512 D64 148 / 139,
// B16 H32 S1024 D64 417 / 406, B16 H16 S1024 D64 205 / 200; but B16 H12 S2048
// D64 498 / 522 (its longest tiles then start in every group's last round), B8
// H16 S1024 D64 (two groups) 109 / 116, and the forward of B16 H16 S512 D64
// (resident at once) 19.5 / 22.4.  The backward keeps `otherwise`
//  * in dK/dV without the mask at D = 128, where every work group streams the
//    whole head: B16 H16 S512 85 over all heads, 86-104 in groups;
//  * in grids of little more than a round, where heavy tiles of the last group
//    of heads would end the grid that light ones end in the order over all
//    heads: dK/dV with the mask at D = 128 up to 1.7 rounds (B1 H202 S320 26.2 /
//    32.5, B1 H208 S392 42.3 / 49.1; B1 H300 S384, 1.76, 53.5 / 51.1), with two
//    tiles up to two rounds (B1 H323 S186 24.9 / 29.7), at D = 64 with two tiles
//    in any number of rounds (B1 H942 S140 26.6 / 28.6) and with three, the last
//    at most 48 rows, up to 1.5 (B1 H340 S258 22.8 / 23.7); dQ at D = 128 with
//    the mask and three tiles up to 1.5 (B1 H210 S384 31.1 / 34.9, B1 H240 S264
//    26.8 / 28.8; B1 H300 S384 43.6 / 40.9), without it and two or three tiles,
//    the last at most 48 rows, up to two (B1 H340 S160 23.7 / 26.3, B1 H250 S300
//    39.4 / 41.4; B1 H340 S192 29.5 / 28.7).
// (One tile per head: both orders are the same.)  Groups are of the same size,
// a multiple of 8 so that a head keeps its chiplet: a small last one would start
// its heavy tiles last (dK/dV with the mask at D = 128, 64 and the rest / even:
// B1 H208 S540 63.0 / 58.2, B1 H202 S704 80.1 / 77.6, B1 H272 S668 107.7 / 102.3).
constexpr int kHeadGroup = 64;
constexpr int work_order(Pass pass, int D, bool causal, int BH, int S, int n_tiles, int per_cu, int cus,
                         int otherwise) {
  const long long n = (long long)BH * n_tiles, round = (long long)per_cu * cus;
  if (n_tiles < 2 || S > 1024 || BH < 3 * kHeadGroup || n <= round) return otherwise;
  const bool short_last = (long long)n_tiles * 128 - S >= 80;  // (no split grid of two or three tiles gets here)
  if (pass == Pass::kDkdv) {
    if (!causal && D == 128) return otherwise;
    if (causal && n_tiles == 2 && (D == 64 || n <= 2 * round)) return otherwise;
    if (causal && (D == 64 ? n_tiles == 3 && short_last && 2 * n <= 3 * round : 10 * n <= 17 * round)) return otherwise;
  }
  if (pass == Pass::kDq && D == 128 && n_tiles <= 3) {
    if (causal ? n_tiles == 3 && 2 * n <= 3 * round : short_last && n <= 2 * round) return otherwise;
  }
  const int groups = (BH + kHeadGroup - 1) / kHeadGroup;
  return -((BH + 8 * groups - 1) / (8 * groups) * 8);
}

// Ring with one barrier per group of G iterations (one part; G divides the
// ring depth NB): the prologue copies tiles 0 .. NB-G-1, and at the top of
// iteration i (i % G == 0) the copies of tiles i+NB-G .. i+NB-1 are issued
// into the slots of tiles i-G .. i-1, which every wave finished at the
// barrier.  Iterations i .. i+G-1 read tiles up to i+G-1+need, so the wait at
// the top of i (i > 0) may leave in flight the tiles issued before that lie
// beyond it: this is their number.  Needs NB >= 2 G + need (the tiles a
// group reads are then copied before its top).
// Iterations per barrier a ring of NB slots can take with `split` parts and
// `need` tiles of look-ahead: the largest g <= want that groups the ring (one
// part, NB a multiple of g, NB >= 2 g + need), else 1.
constexpr int ring_group(int split, int NB, int need, int want) {
  for (int g = want; g > 1; --g)
    if (split == 1 && NB % g == 0 && NB >= 2 * g + need) return g;
  return 1;
}
constexpr int ring_group_in_flight(int i, int L, int NB, int G, int need) {
  const int last_issued = imin(L - 1, i + NB - G - 1);
  const int d = last_issued - (i + G - 1 + need);
  return d > 0 ? d : 0;
}

}  // namespace cattn

