// Exhaustive check of the ring-schedule arithmetic of attn_sched.h against an
// explicit simulation of the copies, for every ring depth, number of parts and read
// depth the kernels use and every tile count up to 300.
#include <cstdio>
#include <initializer_list>

#include "attn_sched.h"
#include "lmhead_sched.h"
#include <vector>

using namespace cattn;

int main() {
  long bad = 0, checks = 0;
  // one barrier per iteration: n tiles dealt to the parts in turn, every part
  // copying one per iteration, in issue order
  for (int NB : {2, 3, 4, 6, 8}) {
    const int AH = NB - 1;
    for (int split : {1, 2, 4}) {
      for (int need : {0, 1}) {
        if (need >= AH) continue;
        for (int n = 1; n <= 300; ++n) {
          const int L = (n + split - 1) / split;
          std::vector<int> order;  // iteration of every part tile, in issue order
          auto copy = [&](int x) {
            for (int p = 0; p < split; ++p) order.push_back(x);
          };
          for (int x = 0; x < AH && x < L; ++x) copy(x);  // before the loop, which waits for all of them
          for (int i = 0; i < L; ++i) {
            ++checks;
            const int f = i == 0 ? 0 : ring_in_flight(i, L, split, AH, need);
            if (f < 0 || f > (int)order.size()) {
              ++bad;
              continue;
            }
            // everything older than the newest f has landed: no tile read by iterations i .. i+need is among those
            for (size_t x = order.size() - f; x < order.size(); ++x)
              if (order[x] <= i + need) ++bad;
            // ... and they have all been issued
            for (int x = i; x <= i + need && x < L; ++x)
              if (x > i - 1 + AH) ++bad;
            if (i > 0 && i + AH <= L && f != ring_in_flight_full(split, AH, need)) ++bad;
            // the copy issued at the top of iteration i (iteration i+AH) reuses the buffer
            // of iteration i-1, finished before the barrier, never one read at i .. i+need
            if (i + AH < L) {
              const int b = (i + AH) % NB;
              if (b != (i + NB - 1) % NB) ++bad;
              for (int k = 0; k <= need; ++k)
                if (b == (i + k) % NB) ++bad;
              copy(i + AH);
            }
          }
          if ((int)order.size() != L * split) ++bad;  // every tile of every part was copied
        }
      }
    }
  }
  // banded_rank is a permutation of [0, n) for every grid size and band, with
  // and without pairing up; only a grid of two rounds walks round 0 backwards
  for (int n = 1; n <= 1200; n += 7) {
    for (int band : {0, 1, 3, 80, 256, 304}) {
      for (bool pair_up : {false, true}) {
        static unsigned char seen[1200];
        for (int i = 0; i < n; ++i) seen[i] = 0;
        for (int b = 0; b < n; ++b) {
          ++checks;
          const int r = banded_rank(b, n, band, pair_up);
          if (r < 0 || r >= n || seen[r]) ++bad;
          else seen[r] = 1;
          if (band == 0) continue;
          // a unit's items: rounds alternate, so ranks within a round run one way or the other
          const bool back = b + kXcdGroup < n && b / band == (b + kXcdGroup) / band &&
                            banded_rank(b + kXcdGroup, n, band, pair_up) < r;
          const bool two = n > band && n <= 2 * band;
          if (band > kXcdGroup && b % band + kXcdGroup < band && b + kXcdGroup < n &&
              back != ((b / band + (pair_up && two ? 1 : 0)) % 2 == 1))
            ++bad;
        }
      }
    }
  }
  // the forward's and dQ's bands: none in one round or past three of a split
  // grid, no pairing up behind a short last one of two or three unsplit tiles
  for (int parts : {1, 2, 4})
    for (int S : {32, 96, 97, 128, 160, 224, 225, 300, 384, 450, 1024})
      for (long long n : {1LL, 256LL, 257LL, 512LL, 768LL, 769LL, 5000LL}) {
        ++checks;
        const bool short_last = S == 32 || S == 96 || S == 160 || S == 224 || S == 300;
        const int want = n <= 256 || (parts > 1 && n > 768) ? 0 : 256 + (parts == 1 && short_last ? kNoPairUp : 0);
        if (query_band(n, parts, S, 256) != want) ++bad;
      }
  for (int S = 1; S <= 5000; ++S) {
    const int p = ws_rows(S);
    if (p % 32 != 0 || p < S || p >= S + 32) ++bad;
  }
  // loss-head persistent grid: every (vocabulary tile, token tile) is taken by
  // exactly one work group, on the chiplet of its vocabulary tile, in bounds
  for (int N : {128, 256, 384, 1152, 2304, 50304, 65536 + 128}) {
    for (int M : {128, 256, 384, 8192}) {
      const int n_vt = lmh_vtiles(N), n_mt = lmh_mtiles(M);
      for (int per_xcd : {1, 3, 32}) {
        std::vector<int> seen((size_t)n_vt * n_mt, 0);
        for (int b = 0; b < lmh_grid(per_xcd); ++b) {
          const int x = b % kXcdGroup;
          for (int l = b / kXcdGroup; l < lmh_xcd_tiles(x, n_vt, n_mt); l += per_xcd) {
            ++checks;
            const int t = lmh_xcd_tile(x, l, n_vt, n_mt), vt = t >> 16, mt = t & 0xffff;
            if (vt < 0 || vt >= n_vt || mt < 0 || mt >= n_mt || vt % kXcdGroup != x) {
              ++bad;
              continue;
            }
            ++seen[(size_t)vt * n_mt + mt];
          }
        }
        for (int c : seen)
          if (c != 1) ++bad;
      }
    }
  }
  // grouped ring (one barrier per G iterations): every tile an iteration reads has landed at the
  // group's wait (copies complete in issue order), and no copy overwrites a tile still to be read
  for (int NB : {3, 4, 6, 8, 9, 12}) {
    for (int G : {1, 2, 3, 4})
    for (int need : {0, 1}) {
      const int pro = NB - G;
      if (NB % G || NB < 2 * G + need) continue;
      ++checks;
      if (ring_group(1, NB, need, G) != G || ring_group(2, NB, need, G) != 1) ++bad;
      for (int L = 1; L <= 70; ++L) {
        std::vector<int> order;  // tiles in issue order
        for (int t = 0; t < pro && t < L; ++t) order.push_back(t);
        std::vector<char> landed(L, 0);
        for (int t : order) landed[t] = 1;  // the prologue waits for everything
        for (int i = 0; i < L; i += G) {
          if (i > 0) {
            const int k = ring_group_in_flight(i, L, NB, G, need);
            ++checks;
            if (k < 0 || k > (int)order.size()) {
              ++bad;
              continue;
            }
            for (size_t x = 0; x + k < order.size(); ++x) landed[order[x]] = 1;
          }
          for (int g = 0; g < G; ++g) {
            const int t = i + pro + g;
            if (t >= L) continue;
            ++checks;
            const int prev = t - NB;  // the slot's previous tile: read by iterations prev - 1 and prev
            if (prev >= 0 && prev >= i) ++bad;
            order.push_back(t);
          }
          for (int j = i; j < i + G && j < L; ++j)
            for (int t = j; t <= j + need && t < L; ++t) {
              ++checks;
              if (!landed[t]) ++bad;
            }
        }
      }
    }
  }
  std::printf("checks=%ld bad=%ld\n", checks, bad);
  return bad != 0 || checks == 0;
}
