// Host-only check of unit_shares and launch_shares (paper_2502_06155_amd/csrc/tile_attn_host.cpp), linked
// against the built library and run by tests/test_shares.py: the eight shares cover the
// units in order; a launch of few units with rows, or whose counts are even to within 3% of the work,
// keeps the equal counts; any other gets shares within one unit of an eighth of the work. Prints "<name>
// equal 0|1 most M" with M the largest share's work over an eighth of all. It also checks that
// append_fwd_schedule keeps the equal counts where it cuts units into parts.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "host_internal.h"
#include "tile_attn.h"
#include "unit_order.h"

using namespace ta::host;

// Heads cycle through the (g, form) pairs given.
static int check(const char* name, int B, int H, int F, int T, int P, int rows,
                 std::vector<std::pair<int, int>> kinds) {
  const int n_seg = F + (P > 0);
  std::vector<uint8_t> masks;
  for (int h = 0; h < H; ++h) {
    std::vector<uint8_t> m((size_t)F * F);
    tile_attn_make_mask(F, kinds[h % kinds.size()].first, kinds[h % kinds.size()].second, m.data());
    for (int i = 0; i < n_seg; ++i)
      for (int j = 0; j < n_seg; ++j) masks.push_back(i < F && j < F ? m[(size_t)i * F + j] : 1);
  }
  const HostWorkList hw = build_work_list(masks.data(), H, H, n_seg, true);
  const int nblk = (std::max(T, P) + rows - 1) / rows;
  uint32_t share[9];
  unit_shares(hw, B, nblk, rows, T, P, F, share);
  const uint32_t per_b = (uint32_t)hw.n_items * nblk, n = B * per_b;
  const int32_t *items = hw.words.data(), *cols = items + hw.off_cols;
  int64_t with_rows = 0;
  for (uint32_t u = 0; u < n; ++u)
    with_rows += (P > 0 && items[5 * ((u % per_b) / nblk) + 1] == F ? P : T) > (int)(u % nblk) * rows;
  auto work = [&](uint32_t u) -> double {
    const int32_t* it = items + 5 * ((u % per_b) / nblk);
    const int left = (P > 0 && it[1] == F ? P : T) - (int)(u % nblk) * rows;
    double t = it[3] * ((T + 63) / 64);
    if (P > 0 && it[3] > 0 && cols[it[2] + it[3] - 1] == F) t += (P + 63) / 64 - (T + 63) / 64;
    return left <= 0 ? 0 : left <= 32 ? t / 2 + 1 : t + 2;
  };
  double total = 0, longest = 0, most = 0, most_equal = 0;
  for (uint32_t u = 0; u < n; ++u) {
    total += work(u);
    longest = std::max(longest, work(u));
  }
  bool equal = true;
  if (share[0] != 0 || share[8] != n) return std::printf("%s: ends\n", name), 1;
  for (int x = 0; x < 8; ++x) {
    if (share[x] > share[x + 1]) return std::printf("%s: order\n", name), 1;
    equal = equal && share[x] == ta::share_start(n, x);
    double w = 0, we = 0;
    for (uint32_t u = share[x]; u < share[x + 1]; ++u) w += work(u);
    for (uint32_t u = ta::share_start(n, x); u < ta::share_start(n, x + 1); ++u) we += work(u);
    most = std::max(most, w);
    most_equal = std::max(most_equal, we);
  }
  const double even = total / 8;
  if (with_rows < kMinUnitsByWork && !equal) return std::printf("%s: few units not by count\n", name), 1;
  if (most_equal <= 1.0299 * even && !equal) return std::printf("%s: even counts not kept\n", name), 1;
  if (with_rows >= kMinUnitsByWork && most_equal > 1.0301 * even && most > even + longest + 8) return std::printf("%s: share of %.3f\n", name, most / even), 1;
  std::printf("%s equal %d most %.3f\n", name, (int)equal, most / even);
  return 0;
}

// launch_shares takes the equal counts or the cut by work, never one that is over half a percent
// longer: each XCD's units in order on 64 workgroups, the first that is free taking the next. Prints
// "<name> counts C work W chosen M", the tiles on the longest XCD.
static int check_choice(const char* name, int B, int H, int F, int T, int P, int rows, bool short_last,
                        std::vector<std::pair<int, int>> kinds) {
  const int n_seg = F + (P > 0);
  std::vector<uint8_t> masks;
  for (int h = 0; h < H; ++h) {
    std::vector<uint8_t> m((size_t)F * F);
    tile_attn_make_mask(F, kinds[h % kinds.size()].first, kinds[h % kinds.size()].second, m.data());
    for (int i = 0; i < n_seg; ++i)
      for (int j = 0; j < n_seg; ++j)
        masks.push_back(i < F && j < F ? m[(size_t)i * F + j] : 1);
  }
  const HostWorkList hw = build_work_list(masks.data(), H, H, n_seg, true);
  const int nblk = (std::max(T, P) + rows - 1) / rows;
  const uint32_t per_b = (uint32_t)hw.n_items * nblk, n = B * per_b;
  const int32_t *items = hw.words.data(), *cols = items + hw.off_cols;
  auto longest = [&](const uint32_t share[9]) {
    double end = 0;
    for (int x = 0; x < 8; ++x) {
      std::vector<double> slot(64, 0);
      for (int pass = 0; pass < 2; ++pass)  // the short blocks in a second pass of their own
        for (uint32_t u = share[x]; u < share[x + 1]; ++u) {
          const int32_t* it = items + 5 * ((u % per_b) / nblk);
          const int left = (P > 0 && it[1] == F ? P : T) - (int)(u % nblk) * rows;
          if (left <= 0 || pass != (int)(short_last && u % nblk == (uint32_t)nblk - 1)) continue;
          double t = it[3] * ((T + 63) / 64) + 2;
          if (P > 0 && it[3] > 0 && cols[it[2] + it[3] - 1] == F) t += (P + 63) / 64 - (T + 63) / 64;
          double& at = *std::min_element(slot.begin(), slot.end());
          at += left <= 32 ? t / 2 : t;
          end = std::max(end, at);
        }
    }
    return end;
  };
  uint32_t count[9], work[9], chosen[9];
  for (uint32_t x = 0; x <= 8; ++x) count[x] = ta::share_start(n, x);
  unit_shares(hw, B, nblk, rows, T, P, F, work);
  launch_shares(hw, B, nblk, rows, T, P, F, 64, short_last, false, chosen);
  if (!std::equal(chosen, chosen + 9, count) && !std::equal(chosen, chosen + 9, work))
    return std::printf("%s: neither cut\n", name), 1;
  const double c = longest(count), w = longest(work), m = longest(chosen);
  if (m > 1.005 * c || (n <= kMaxModelledUnits && m > 1.005 * w)) return std::printf("%s: %.0f of %.0f and %.0f\n", name, m, c, w), 1;
  std::printf("%s counts %.0f work %.0f chosen %.0f\n", name, c, w, m);
  return 0;
}

// A forward launch whose ragged round is cut into parts keeps the shares by count: they decide
// which units are cut, and with them how its sums are rounded. Only one that cuts nothing by
// count may take the shares by work, and then cuts nothing either. Prints "<name> cut U units
// by work 0|1", U the units cut.
static int check_cut(const char* name, int B, int H, int F, int T, int d, std::vector<std::pair<int, int>> kinds) {
  const int rows = d == 128 ? 128 : 256, nqb = (T + rows - 1) / rows;
  std::vector<uint8_t> masks((size_t)H * F * F);
  for (int h = 0; h < H; ++h)
    tile_attn_make_mask(F, kinds[h % kinds.size()].first, kinds[h % kinds.size()].second, masks.data() + (size_t)h * F * F);
  HostWorkList hw = build_work_list(masks.data(), H, H, F, true);
  const size_t words = hw.words.size();
  append_fwd_schedule(hw, B, nqb, rows, d, T, 0, F, 64, true);
  const uint32_t n = (uint32_t)B * hw.n_items * nqb;
  const int32_t* xcd = hw.words.data() + hw.off_xcd;
  if (hw.n_heavy != 0) return std::printf("%s: frames split\n", name), 1;
  bool equal = true;
  for (int x = 0; x < 8; ++x) {
    equal = equal && hw.share[x] == ta::share_start(n, x);
    if (xcd[4 * x] != (int)hw.share[x]) return std::printf("%s: shares of another schedule\n", name), 1;
  }
  if (hw.off_xcd != words || hw.share[8] != n) return std::printf("%s: layout\n", name), 1;
  if (!equal && (hw.n_cut_units > 0 || hw.n_part_slots > 0)) return std::printf("%s: cut by work\n", name), 1;
  std::printf("%s cut %d units by work %d\n", name, hw.n_cut_units, (int)!equal);
  return 0;
}

// A schedule formed on every call takes the cut by work only where a bound says so, or, with long
// units, the model. Prints "<name> every call work 0|1".
static int check_every_call(const char* name, int B, int H, int F, int T, int d, std::vector<std::pair<int, int>> kinds) {
  const int rows = d == 128 ? 128 : 256, nqb = (T + rows - 1) / rows;
  std::vector<uint8_t> masks((size_t)H * F * F);
  for (int h = 0; h < H; ++h)
    tile_attn_make_mask(F, kinds[h % kinds.size()].first, kinds[h % kinds.size()].second, masks.data() + (size_t)h * F * F);
  HostWorkList kept = build_work_list(masks.data(), H, H, F, true), hw = kept;
  append_fwd_schedule(kept, B, nqb, rows, d, T, 0, F, 64, false, false);
  append_fwd_schedule(hw, B, nqb, rows, d, T, 0, F, 64, false, false, true);
  const uint32_t n = (uint32_t)B * hw.n_items * nqb;
  bool equal = true;
  for (uint32_t x = 0; x <= 8; ++x) equal = equal && hw.share[x] == ta::share_start(n, x);
  if (!equal && !std::equal(hw.share, hw.share + 9, kept.share)) return std::printf("%s: another cut\n", name), 1;
  std::printf("%s every call work %d\n", name, (int)!equal);
  return 0;
}

// The grid of a launch holds every position and no workgroup past the last: units that just
// fit the grid limit (2^32 - 1 threads) launch whatever their number's remainder by eight.
static int check_grid(std::vector<uint32_t> cuts) {
  uint32_t count[8], last = 0;
  for (uint32_t x = 0; x < 8; ++x) {
    count[x] = cuts[x + 1] - cuts[x];
    if (count[x] > 0) last = std::max(last, 8 * (count[x] - 1) + x);
  }
  const uint32_t n = cuts[8], grid = ta::grid_of(count);
  if (grid != (n ? last + 1 : 0)) return std::printf("grid of %u units: %u\n", n, grid), 1;
  bool equal = true;
  for (uint32_t x = 0; x < 9; ++x) equal = equal && cuts[x] == ta::share_start(n, x);
  if (equal && grid != n) return std::printf("grid of %u units by count: %u\n", n, grid), 1;
  return 0;
}

int main() {
  const std::pair<int, int> col1{1, TA_MASK_COL}, sym1{1, TA_MASK_SYM}, sym2{2, TA_MASK_SYM}, col4{4, TA_MASK_COL};
  int bad = 0;
  bad |= check("uniform", 1, 24, 24, 3600, 0, 256, {col1});
  bad |= check("mixed-fwd", 1, 6, 24, 3600, 0, 256, {sym2, sym1, col4});
  bad |= check("mixed-bwd", 1, 6, 24, 3600, 0, 128, {sym2, sym1, col4});
  bad |= check("mixed-batch", 3, 5, 24, 333, 0, 128, {sym2, sym1, col4});
  bad |= check("share-sym", 1, 6, 24, 3600, 0, 256, {sym1});
  bad |= check("mmdit", 1, 5, 13, 1350, 226, 256, {sym2, col1});
  bad |= check("mmdit-long-text", 2, 3, 7, 40, 300, 128, {sym1, col1});
  bad |= check("one-unit", 1, 1, 1, 7, 0, 256, {col1});
  bad |= check("few-with-rows", 1, 5, 27, 90, 663, 128, {sym2});
  bad |= check("few", 1, 3, 2, 300, 0, 256, {col1});
  for (uint32_t n : {0u, 1u, 7u, 8u, 9u, 1000u, 16777208u, 16777209u, 16777215u}) {
    std::vector<uint32_t> cuts(9);
    for (uint32_t x = 0; x <= 8; ++x) cuts[x] = ta::share_start(n, x);
    bad |= check_grid(cuts);
  }
  bad |= check_grid({0, 0, 5, 5, 5, 9, 30, 30, 31});
  bad |= check_grid({0, 40, 41, 42, 43, 44, 45, 46, 46});
  bad |= check_cut("cut-d64", 1, 14, 9, 2883, 64, {{5, TA_MASK_SYM}});
  bad |= check_cut("cut-d96", 1, 18, 24, 555, 96, {{8, TA_MASK_SYM}});
  bad |= check_cut("cut-batch", 2, 3, 25, 2264, 64, {{7, TA_MASK_SYM}});
  bad |= check_cut("cut-d128", 1, 13, 4, 3231, 128, {{3, TA_MASK_SYM}});
  bad |= check_cut("cut-none", 3, 5, 17, 1936, 128, {{7, TA_MASK_COL}, col1, {14, TA_MASK_SYM}});
  bad |= check_every_call("every-share", 1, 6, 24, 3600, 96, {sym2, sym1, col4});
  bad |= check_every_call("every-long", 3, 5, 17, 1936, 128, {{7, TA_MASK_COL}, col1, {14, TA_MASK_SYM}});
  bad |= check_every_call("every-short", 2, 30, 40, 100, 96, {{3, TA_MASK_COL}, col1, {6, TA_MASK_SYM}});
  bad |= check_choice("choice-sym4", 1, 18, 24, 555, 0, 256, false, {{4, TA_MASK_SYM}});
  bad |= check_choice("choice-fwd", 2, 18, 8, 1056, 0, 256, true, {col1, {1, TA_MASK_COL}, sym2});
  bad |= check_choice("choice-d128", 1, 36, 15, 482, 0, 128, false, {{6, TA_MASK_COL}, col1, {12, TA_MASK_SYM}});
  bad |= check_choice("choice-tail", 1, 29, 9, 775, 0, 256, true, {{8, TA_MASK_COL}, col1, {9, TA_MASK_SYM}});
  bad |= check_choice("choice-share-heads", 1, 6, 24, 3600, 0, 256, true, {sym2, sym1, col4});
  bad |= check_choice("choice-share-sym", 1, 6, 24, 3600, 0, 256, true, {sym1});
  bad |= check_choice("choice-mmdit", 1, 27, 15, 1350, 226, 128, false, {sym1});
  bad |= check_choice("choice-many", 1, 41, 47, 3090, 0, 128, false, {col1, col1, sym2});
  return bad;
}
