// How a decode step's attention is cut into work-groups: host-side, no GPU calls (exercised through
// include/areal_host.h).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <unordered_map>
#include <vector>

namespace areal {

constexpr int kDecodeUnit = 32;           // tokens a wave takes at a time
constexpr int kDecodeMaxUnits = 64;       // per segment: 128 block ids, two per lane
constexpr int kDecodeXcds = 8;

// A run of one row's tokens [t0, t0 + n), n > 0; the row's last segment holds the position it appends at.
// `slot` numbers the segments of a row.
struct DecodeSegment { int32_t row, t0, n, slot; };

struct DecodePlan {
  std::vector<DecodeSegment> segs;        // XCD by XCD: those of XCD x are [base[x], base[x + 1])
  int32_t base[kDecodeXcds + 1] = {};
  int depth = 0;                          // most segments of an XCD
  std::vector<int32_t> n_own;             // segments of each row
  int max_own = 0, max_units = 0;         // most segments of a row, longest segment
};

// Most bytes that the descriptors and block ids of the segments of n rows take, whatever their lengths up to
// `max_tokens`: 16 bytes a segment, and 4 for each of the longest one's blocks (rounded up to 4) in every segment.
// With X units in the longest row and segments of up to S units (4 <= S <= 64) a row has at most 1 + X / S of them, so that
// 24 bytes and 8 min(S, X) each are at most 24 + 24 X / S + 8 min(S, X) + 8 X, which no S in that range makes larger
// than the sum below.
inline uint64_t decode_segment_bytes(uint64_t n, uint64_t max_tokens) {
  const uint64_t X = (max_tokens + kDecodeUnit - 1) / kDecodeUnit;
  return n * (14 * X + 8 * std::min<uint64_t>(X, kDecodeMaxUnits) + 56);
}

// The cut replaces splits of one length for all rows (256 tokens and up, work-groups without tokens where a row was
// shorter than the longest, a remainder per row).  Attention launch of a step, 1.5B shape: 256 rows of 420 - 650 tokens
// 30.3 us and a merge of 4.9 -> 25.1 and none; 88 rows of 1,500 - 4,100 54.1 -> 51.1; 24 of 4,000 - 8,200 37.0 -> 32.5; one
// of 700 10.1 -> 7.3; 7B shape, 128 rows of 500 - 3,800 116.8 -> 106.4.
//
// Units of a row's segments (its last one may be shorter), aimed at `share`: cut evenly, then up to whole rounds of a
// work-group's four waves (a wave takes every fourth unit, so an uneven round leaves some without one).
inline int decode_segment_units(int units, int share) {
  const int k = (units + share - 1) / share;
  return k == 1 ? units : std::min(((units + k - 1) / k + 3) / 4 * 4, kDecodeMaxUnits);
}

// Units per segment, by price.  In microseconds: every unit of 32 tokens (16 KB a KV head) at 6.2 TB/s over the
// chip's 512 resident work-groups; a work-group's start (block ids, then tiles: two round trips), its end and its
// partials; what the last ones leave idle; and the merge launch if any row is cut at all.  Where all are resident at
// once, a compute unit that has two still takes 1.34 us for a unit of each, however few others there are (352
// work-groups of 51 units: 68 us, 880 of 24: 62), one that has one about 0.65.  With that and with whole rounds, against
// even cuts priced as if any number of work-groups streamed at the full rate: launches of 157 rows of 1,725 tokens
// 71.9 -> 61.8 us, 88 of 3,217 71.4 -> 66.4, 44 of 5,204 57.7 -> 53.0 (steps 3.52 -> 3.40 ms, 3.26 -> 3.14, 2.77 -> 2.62);
// rows of many lengths, as in the figures above, the same to 2 % better.
inline double decode_price(const std::vector<int>& units, int n_kv_heads, int share) {
  int64_t segs = 0, total = 0;
  int longest = 0;
  bool cut = false;
  for (int u : units) {
    const int len = decode_segment_units(u, share);
    segs += (u + len - 1) / len;
    total += u;
    longest = std::max(longest, len);
    cut |= len < u;
  }
  const double wgs = (double)segs * n_kv_heads, rounds = wgs / 512.0, mean = (double)total * n_kv_heads / wgs;
  const double streamed = (double)total * n_kv_heads * (1.34 / 512.0);
  double us;
  if (rounds > 1.0) {
    us = streamed + 1.5 * rounds + 0.25 * longest;
  } else {
    us = std::max(wgs > 256.0 ? 1.34 * mean : std::max(streamed, 0.65 * mean), 0.65 * longest + 3.4);
    us += rounds + 0.5 * (longest - mean);
  }
  return us + (cut ? 4.5 : 0.0);
}
inline int decode_share(const std::vector<int>& units, int n_kv_heads, int lo, int hi) {
  static const int steps[] = {4, 8, 12, 16, 20, 24, 28, 32, 40, 48, 64};
  int best = hi;
  double best_us = 1e30;
  for (int s : steps) {
    if (s < lo || s > hi) continue;
    const double us = decode_price(units, n_kv_heads, s);
    if (us < best_us) { best_us = us; best = s; }
  }
  return best;
}

// The share that gives about `target` work-groups (tuning): whole rounds of a work-group's four waves.
inline int decode_share_for(int64_t total_units, int n_kv_heads, int target, int min_tokens) {
  const int share = (int)((total_units * n_kv_heads + target - 1) / target);
  return (std::max(share, min_tokens / kDecodeUnit) + 3) / 4 * 4;
}

// own[i]: tokens of row i from its first own one to the one it appends (>= 1).  home[i]: the row's first KV block; rows
// with the same one hold leading blocks together.  Rows are cut into at most max_slots segments.  target > 0: so
// that there are about that many work-groups, no segment aimed shorter than min_tokens (tuning); 0: by price.
//
// Order: each XCD gets an eighth of the units, longest segments first.  Rows that share blocks are kept on as few XCDs
// as the balance allows (pieces of a sixteenth of the work), where their common blocks meet in one L2: 16
// prompts x 16 samples of 535 tokens, 288 shared, are 140 MB of K/V per layer, 69 MB of them distinct, of which 102
// would cross the fabric with the samples of a prompt on all XCDs.  No XCD gets more than a quarter above an eighth of the
// segments, and four: the launch has as many work-groups on each XCD as the one with the most segments needs, and among
// many rows of one unit the units alone would let one XCD have most of them (2,063 rows, 256 to a prompt, 1,637 of
// one unit: 12,512 work-groups a KV head without the limit, 2,160 with it).
inline DecodePlan plan_decode(const std::vector<int32_t>& own, const std::vector<int32_t>& home, int n_kv_heads,
                              int max_slots, int target, int min_tokens) {
  const int n = (int)own.size();
  DecodePlan p;
  std::vector<int> units(n);
  int64_t total = 0;
  int longest = 1;
  for (int i = 0; i < n; ++i) {
    units[i] = (own[i] + kDecodeUnit - 1) / kDecodeUnit;
    total += units[i];
    longest = std::max(longest, units[i]);
  }
  const int lo = (longest + max_slots - 1) / max_slots;
  const int aimed = target > 0 ? decode_share_for(total, n_kv_heads, target, min_tokens)
                               : decode_share(units, n_kv_heads, lo, kDecodeMaxUnits);
  const int share = std::min((std::max(aimed, lo) + 3) / 4 * 4, kDecodeMaxUnits);
  p.n_own.resize(n);
  std::vector<int> len(n);                                // units per segment of a row
  int64_t n_segs = 0;
  for (int i = 0; i < n; ++i) {
    len[i] = decode_segment_units(units[i], share);
    p.n_own[i] = (units[i] + len[i] - 1) / len[i];
    n_segs += p.n_own[i];
    p.max_own = std::max(p.max_own, (int)p.n_own[i]);
    p.max_units = std::max(p.max_units, len[i]);
  }
  const int64_t most = (n_segs + kDecodeXcds - 1) / kDecodeXcds * 5 / 4 + 4;       // segments of an XCD
  int64_t load[kDecodeXcds] = {}, count[kDecodeXcds] = {};
  // The XCD with the least to do among those with room for `segs` more (-1: none).
  auto least = [&](int64_t segs) {
    int x = -1;
    for (int k = 0; k < kDecodeXcds; ++k)
      if (count[k] + segs <= most && (x < 0 || load[k] < load[x])) x = k;
    return x;
  };
  // rows -> XCD, or -1: their segments go wherever there is room
  std::vector<int8_t> at(n, -1);
  {
    std::unordered_map<int32_t, std::vector<int>> by_home;
    for (int i = 0; i < n; ++i) by_home[home[i]].push_back(i);
    if ((int)by_home.size() < n) {
      struct Piece { int64_t load, segs; std::vector<int> rows; };
      std::vector<Piece> pieces;
      for (int i = 0; i < n; ++i) {                       // in row order, so that a plan does not depend on hashing
        auto& rows = by_home[home[i]];
        if (rows.size() < 2 || rows[0] != i) continue;
        Piece piece{0, 0, {}};
        for (int r : rows) {
          if (!piece.rows.empty() && (piece.load + units[r]) * 16 > total) {
            pieces.push_back(std::move(piece));
            piece = Piece{0, 0, {}};
          }
          piece.load += units[r];
          piece.segs += p.n_own[r];
          piece.rows.push_back(r);
        }
        pieces.push_back(std::move(piece));
      }
      std::stable_sort(pieces.begin(), pieces.end(), [](const Piece& a, const Piece& b) { return a.load > b.load; });
      for (const Piece& piece : pieces) {
        const int x = least(piece.segs);
        if (x < 0) continue;
        load[x] += piece.load;
        count[x] += piece.segs;
        for (int r : piece.rows) at[r] = (int8_t)x;
      }
      // more than a twentieth above an eighth of everything: the balance is worth more than the L2
      if (*std::max_element(load, load + kDecodeXcds) * 160 > total * 21) {
        std::fill(at.begin(), at.end(), (int8_t)-1);
        std::fill(load, load + kDecodeXcds, 0);
        std::fill(count, count + kDecodeXcds, 0);
      }
    }
  }
  std::vector<int> rows(n);
  for (int i = 0; i < n; ++i) rows[i] = i;
  std::stable_sort(rows.begin(), rows.end(), [&](int a, int b) { return len[a] > len[b]; });
  std::vector<DecodeSegment> queue[kDecodeXcds];
  for (int i : rows)
    for (int k = 0, u = 0; u < units[i]; ++k, u += len[i]) {
      const int m = std::min(len[i], units[i] - u);
      int x = at[i];
      if (x < 0) {
        x = least(1);
        load[x] += m;
        ++count[x];
      }
      queue[x].push_back(DecodeSegment{i, u * kDecodeUnit, m * kDecodeUnit, k});
    }
  p.segs.reserve(n_segs);
  for (int x = 0; x < kDecodeXcds; ++x) {
    p.segs.insert(p.segs.end(), queue[x].begin(), queue[x].end());
    p.base[x + 1] = (int32_t)p.segs.size();
    p.depth = std::max(p.depth, (int)queue[x].size());
  }
  return p;
}

}  // namespace areal
