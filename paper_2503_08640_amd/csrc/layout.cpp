// Host block-layout builder: pool structure (+ per-query group selections) ->
// per-Q-tile lists of KV tiles.  Integer work only, no GPU calls.
//
// Stage 1 (Sec. 2.1): a group attends the anchor, a fixed number of preceding
// groups, and itself causally, so the list of a Q tile is: every sink tile, every
// tile of the preceding groups in the window, and the own group's tiles that start
// at or before the tile's last row.  Stage 2 (Sec. 2.2): the selected groups' KV is
// used in place -- the list simply names their tiles behind the sink's -- followed
// by the query's own tiles up to the diagonal.
#include "layout.hpp"

#include <algorithm>
#include <climits>
#include <numeric>
#include <utility>

namespace {

struct Seg {
  int32_t begin, end;
};

inline int32_t pack_len_kind(int32_t len, int32_t kind) { return len | (kind << 16); }

// Append the tiles of [seg.begin, seg.end) cut every `bn` tokens, all with `kind`.
void push_whole_segment(std::vector<int32_t>& ent, Seg seg, int32_t bn, int32_t kind) {
  for (int64_t k0 = seg.begin; k0 < seg.end; k0 += bn) {
    ent.push_back(static_cast<int32_t>(k0));
    ent.push_back(pack_len_kind(static_cast<int32_t>(std::min<int64_t>(bn, seg.end - k0)), kind));
  }
}

// Append the tiles of `seg` a Q tile [q0, q0+qn) sees under a causal rule inside the
// segment: a tile is listed when its first key is not after the tile's last row; it
// needs no mask when its last key is not after the tile's first row.
void push_causal_segment(std::vector<int32_t>& ent, Seg seg, int32_t bn, int32_t q0, int32_t qn, int32_t kind_full,
                         int32_t kind_causal) {
  const int64_t q_last = static_cast<int64_t>(q0) + qn - 1;
  for (int64_t k0 = seg.begin; k0 < seg.end && k0 <= q_last; k0 += bn) {
    const int64_t kn = std::min<int64_t>(bn, seg.end - k0);
    const bool full = (k0 + kn - 1) <= q0;
    ent.push_back(static_cast<int32_t>(k0));
    ent.push_back(pack_len_kind(static_cast<int32_t>(kn), full ? kind_full : kind_causal));
  }
}

bool strictly_increasing(const int32_t* a, int64_t n) {
  for (int64_t i = 1; i < n; ++i)
    if (a[i] <= a[i - 1]) return false;
  return true;
}

}  // namespace

int dbsa_build_host_lists(const dbsa_pool_desc* pool, const dbsa_select_desc* sel, int32_t first_group, int32_t block_m, int32_t block_n,
                          dbsa_layout* L) {
  if (!pool || !L || block_m <= 0 || block_n <= 0 || block_n >= (1 << 16)) return DBSA_ERR_INVALID_ARG;
  if (!pool->demo_offsets || !pool->group_demo_offsets || pool->n_demos < 1 || pool->n_groups < 1 ||
      pool->sink_len < 0 || pool->prev_window < 0)
    return DBSA_ERR_INVALID_ARG;
  const int32_t S = pool->sink_len;
  const int32_t* doff = pool->demo_offsets;
  const int32_t* gdo = pool->group_demo_offsets;
  if (doff[0] != S || !strictly_increasing(doff, static_cast<int64_t>(pool->n_demos) + 1)) return DBSA_ERR_BAD_BOUNDS;
  if (gdo[0] != 0 || gdo[pool->n_groups] != pool->n_demos ||
      !strictly_increasing(gdo, static_cast<int64_t>(pool->n_groups) + 1))
    return DBSA_ERR_BAD_BOUNDS;

  const int32_t G = pool->n_groups;
  if (first_group >= 0 && (sel || first_group >= G)) return DBSA_ERR_INVALID_ARG;
  std::vector<Seg> group(G);
  for (int32_t g = 0; g < G; ++g) group[g] = Seg{doff[gdo[g]], doff[gdo[g + 1]]};
  const Seg sink{0, S};

  L->block_m = block_m;
  L->block_n = block_n;
  L->sink_len = S;
  L->n_tokens = doff[pool->n_demos];
  L->n_groups = G;
  L->prev_window = pool->prev_window;
  L->query_stage = (sel != nullptr);
  L->list_ptr.assign(1, 0);

  auto close_tile = [&](int32_t q0, int32_t qn, int32_t owner) {
    L->qtile_tab.insert(L->qtile_tab.end(), {q0, qn, owner, 0});
    L->list_ptr.push_back(static_cast<int64_t>(L->list_ent.size() / 2));
  };

  // where the segments sit in the tensors the query-stage calls will be given (the pool itself
  // unless the caller keeps groups in arena pages)
  Seg sink_at = sink;
  std::vector<Seg> group_at = group;

  if (!sel) {
    // ---- stage 1 ----
    // An appended group sees the sink, its window of preceding groups and itself; nothing
    // already encoded sees it (Sec. 2.1), so encoding it means walking its own Q tiles only.
    for (int64_t q0 = 0; q0 < S && first_group < 0; q0 += block_m) {
      const int32_t qn = static_cast<int32_t>(std::min<int64_t>(block_m, S - q0));
      push_causal_segment(L->list_ent, sink, block_n, static_cast<int32_t>(q0), qn, DBSA_TILE_FULL, DBSA_TILE_CAUSAL);
      close_tile(static_cast<int32_t>(q0), qn, -1);
    }
    for (int32_t g = std::max(first_group, 0); g < G; ++g) {
      const int32_t first_prev = std::max<int64_t>(0, static_cast<int64_t>(g) - pool->prev_window);
      for (int64_t q0 = group[g].begin; q0 < group[g].end; q0 += block_m) {
        const int32_t qn = static_cast<int32_t>(std::min<int64_t>(block_m, group[g].end - q0));
        push_whole_segment(L->list_ent, sink, block_n, DBSA_TILE_FULL);
        for (int32_t p = first_prev; p < g; ++p) push_whole_segment(L->list_ent, group[p], block_n, DBSA_TILE_FULL);
        push_causal_segment(L->list_ent, group[g], block_n, static_cast<int32_t>(q0), qn, DBSA_TILE_FULL,
                            DBSA_TILE_CAUSAL);
        close_tile(static_cast<int32_t>(q0), qn, g);
      }
    }
  } else {
    // ---- stage 2 ----
    if (sel->n_queries < 1 || !sel->cu_qlens || !sel->sel_ptr || sel->n_split < 0) return DBSA_ERR_INVALID_ARG;
    const int32_t B = sel->n_queries;
    if (sel->cu_qlens[0] != 0 || !strictly_increasing(sel->cu_qlens, static_cast<int64_t>(B) + 1))
      return DBSA_ERR_BAD_BOUNDS;
    if (sel->sel_ptr[0] != 0) return DBSA_ERR_BAD_BOUNDS;
    for (int32_t u = 0; u < B; ++u)
      if (sel->sel_ptr[u + 1] < sel->sel_ptr[u]) return DBSA_ERR_BAD_BOUNDS;
    if (sel->sel_ptr[B] > 0 && !sel->sel_idx) return DBSA_ERR_INVALID_ARG;
    std::vector<int32_t> seen(G, -1);
    for (int32_t u = 0; u < B; ++u)
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e) {
        const int32_t g = sel->sel_idx[e];
        if (g < 0 || g >= G || seen[g] == u) return DBSA_ERR_BAD_SELECTION;
        seen[g] = u;
      }

    if (sel->page_start) {
      const int32_t* ps = sel->page_start;
      std::vector<std::pair<int64_t, int64_t>> resident;
      if (S > 0) {
        if (ps[0] < 0) return DBSA_ERR_BAD_BOUNDS;  // the anchor is part of every query's cache
        sink_at = Seg{ps[0], ps[0] + S};
        resident.emplace_back(ps[0], static_cast<int64_t>(ps[0]) + S);
      }
      for (int32_t g = 0; g < G; ++g) {
        const int32_t len = group[g].end - group[g].begin;
        if (ps[g + 1] < 0) continue;
        if (static_cast<int64_t>(ps[g + 1]) + len > INT32_MAX) return DBSA_ERR_BAD_BOUNDS;
        group_at[g] = Seg{ps[g + 1], ps[g + 1] + len};
        resident.emplace_back(ps[g + 1], static_cast<int64_t>(ps[g + 1]) + len);
      }
      std::sort(resident.begin(), resident.end());
      for (size_t i = 1; i < resident.size(); ++i)
        if (resident[i].first < resident[i - 1].second) return DBSA_ERR_BAD_BOUNDS;
      for (int32_t e = 0; e < sel->sel_ptr[B]; ++e)
        if (ps[sel->sel_idx[e] + 1] < 0) return DBSA_ERR_BAD_SELECTION;
    }

    L->n_queries = B;
    L->n_query_tokens = sel->cu_qlens[B];
    L->dec_ptr.assign(1, 0);
    size_t shortest = SIZE_MAX;
    std::vector<int32_t> dec_shift;  // per decode-list entry of the current query
    for (int32_t u = 0; u < B; ++u) {
      // pool part, shared by all Q tiles of the query and by decode
      const size_t dec_begin = L->dec_ent.size();
      push_whole_segment(L->dec_ent, sink_at, block_n, DBSA_TILE_FULL);
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e)
        push_whole_segment(L->dec_ent, group_at[sel->sel_idx[e]], block_n, DBSA_TILE_FULL);
      L->dec_ptr.push_back(static_cast<int64_t>(L->dec_ent.size() / 2));
      shortest = std::min(shortest, (L->dec_ent.size() - dec_begin) / 2);
      // new ids (Sec. 2.2): the sink keeps 0 .. S-1, the k-th selected group follows the (k-1)-th,
      // the query follows the cache.  A run whose first key moves from id j to id j' leaves the
      // query row (at id cache_len + a) to be rotated at id cache_len + a - (j' - j).
      int64_t cache_len = S;
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e)
        cache_len += group[sel->sel_idx[e]].end - group[sel->sel_idx[e]].begin;
      L->cache_len.push_back(static_cast<int32_t>(cache_len));
      dec_shift.clear();
      dec_shift.insert(dec_shift.end(), (static_cast<size_t>(S) + block_n - 1) / block_n, static_cast<int32_t>(cache_len));
      int64_t new_first = S;
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e) {
        const Seg gs = group[sel->sel_idx[e]];
        const size_t n_t = (static_cast<size_t>(gs.end - gs.begin) + block_n - 1) / block_n;
        dec_shift.insert(dec_shift.end(), n_t, static_cast<int32_t>(cache_len - (new_first - gs.begin)));
        new_first += gs.end - gs.begin;
      }

      L->dec_shift.insert(L->dec_shift.end(), dec_shift.begin(), dec_shift.end());

      const Seg self{sel->cu_qlens[u], sel->cu_qlens[u + 1]};
      for (int64_t q0 = self.begin; q0 < self.end; q0 += block_m) {
        const int32_t qn = static_cast<int32_t>(std::min<int64_t>(block_m, self.end - q0));
        L->list_ent.insert(L->list_ent.end(), L->dec_ent.begin() + dec_begin, L->dec_ent.end());
        push_causal_segment(L->list_ent, self, block_n, static_cast<int32_t>(q0), qn, DBSA_TILE_SELF_FULL,
                            DBSA_TILE_SELF_CAUSAL);
        const int32_t a0 = static_cast<int32_t>(q0 - self.begin);  // local index of the tile's first row
        for (int32_t s : dec_shift) L->list_shift.push_back(s + a0);
        L->list_shift.resize(L->list_ent.size() / 2, a0);           // own keys sit at their local index
        close_tile(static_cast<int32_t>(q0), qn, u);
      }
    }
    // split count: enough (query, split) pairs to cover the chip a few times over
    // once multiplied by the KV heads, but never more splits than tiles.
    int32_t ns = sel->n_split;
    if (ns == 0) {
      ns = std::max(1, std::min(32, (256 + B - 1) / B));
      ns = static_cast<int32_t>(std::max<size_t>(1, std::min<size_t>(ns, shortest)));
    }
    L->n_split = ns;
    L->split_ptr.resize(static_cast<size_t>(B) * (ns + 1));
    for (int32_t u = 0; u < B; ++u) {
      const int64_t base = L->dec_ptr[u], len = L->dec_ptr[u + 1] - base;
      for (int32_t s = 0; s <= ns; ++s) L->split_ptr[static_cast<size_t>(u) * (ns + 1) + s] = base + (s * len) / ns;
    }
  }

  // runs cut to measure for the steps that run as a contraction (below): [segment][batch of 64 users] -> run
  // boundaries, the segments' users, the rotation shift of (query, segment), the share of rows that carry a query
  std::vector<std::vector<std::vector<int64_t>>> plan_cuts;
  std::vector<std::vector<int32_t>> plan_users;
  std::vector<int32_t> plan_shift;
  float plan_fill = 0.f;
  if (sel) {
    // ---- group-major decode schedule ----
    // Queries that selected the same group read the same KV, so at decode a chunk of a
    // segment (the sink, a group) is one work item for up to kItemQueries of its users:
    // its keys are fetched once and scored against all of them.  Every (item, user) pair
    // owns one partial-softmax slot; a query's last slot is for its own cached keys.
    constexpr int32_t kItemQueries = 32;
    const int32_t B = sel->n_queries;
    std::vector<std::vector<int32_t>> users(static_cast<size_t>(G) + 1);
    if (S > 0)
      for (int32_t u = 0; u < B; ++u) users[0].push_back(u);
    for (int32_t u = 0; u < B; ++u)
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e) users[sel->sel_idx[e] + 1].push_back(u);
    for (auto& v : users) std::sort(v.begin(), v.end());
    L->gm_seg_ptr.assign(1, 0);
    push_whole_segment(L->gm_seg_ent, sink_at, block_n, DBSA_TILE_FULL);
    L->gm_seg_ptr.push_back(static_cast<int64_t>(L->gm_seg_ent.size() / 2));
    for (int32_t g = 0; g < G; ++g) {
      push_whole_segment(L->gm_seg_ent, group_at[g], block_n, DBSA_TILE_FULL);
      L->gm_seg_ptr.push_back(static_cast<int64_t>(L->gm_seg_ent.size() / 2));
    }
    int64_t max_tiles = 1, tile_batches = 0;
    for (int32_t s = 0; s <= G; ++s) {
      const int64_t t = L->gm_seg_ptr[s + 1] - L->gm_seg_ptr[s];
      if (users[s].empty() || t == 0) continue;
      max_tiles = std::max(max_tiles, t);
      tile_batches += t * ((static_cast<int64_t>(users[s].size()) + kItemQueries - 1) / kItemQueries);
    }
    // single-wave workgroups the chip holds per KV head of an 8-KV-head model (six per compute
    // unit), three quarters of them for pool runs: the rest is for the queries' own caches and for
    // items that take a second batch of queries
    const int64_t run_slots = std::max<int64_t>(1, static_cast<int64_t>(L->compute_units) * 6 / 8 * 3 / 4);
    int64_t chunk = sel->n_split > 0 ? (max_tiles + sel->n_split - 1) / sel->n_split
                                     : std::min<int64_t>(32, (tile_batches + run_slots - 1) / run_slots);
    chunk = std::max<int64_t>(1, chunk);
    // Steps that will run their pool items as a contraction (64 queries per wave, one persistent
    // workgroup per compute unit and KV head: mx_rec below) are bound by arithmetic, and what counts is
    // that every worker gets the same work.  Runs of ONE length cannot do that (90 runs of 32 tiles over
    // 32 workers: three rounds for 2.8 rounds of work), so such a layout cuts its runs to measure: the
    // (segment, 64 queries) units are walked in order and dealt to W workers (W = compute units / 8 per
    // KV head, fewer when a worker's share would fall below kMinShare tiles), each taking tiles until
    // its cost (tiles + kRunCost per run, what starting and finishing a run costs in tiles) reaches the
    // mean; a unit that does not fit is cut there, but no run is shorter than kSnap tiles: a worker
    // rather stops a little early or takes the few tiles that are left.  Worker c takes the runs
    // mx_plan_ptr[c] .. mx_plan_ptr[c+1]-1, in order.  plan_cuts[s][b] = the run boundaries of the b-th
    // batch of 64 queries of segment s.
    if (sel->n_split == 0) {
      double rows = 0.0, used = 0.0;
      int64_t line = 0, n_units = 0;
      for (int32_t s = 0; s <= G; ++s) {
        const int64_t t = L->gm_seg_ptr[s + 1] - L->gm_seg_ptr[s];
        const int64_t n_u = static_cast<int64_t>(users[s].size());
        if (n_u == 0 || t == 0) continue;
        rows += 64.0 * static_cast<double>(t) * static_cast<double>((n_u + 63) / 64);
        used += static_cast<double>(t) * static_cast<double>(n_u);
        line += t * ((n_u + 63) / 64);
        n_units += (n_u + 63) / 64;
      }
      if (rows > 0.0 && used / rows >= kMatrixRowFill) {
        constexpr int64_t kMinShare = 12, kSnap = 4;
        constexpr double kRunCost = 4.5;
        const int64_t nominal = std::max<int64_t>(1, L->compute_units / 8);
        const int64_t workers = std::max<int64_t>(1, std::min<int64_t>(nominal, line / kMinShare));
        int64_t n_rec = 0, longest = 1;
        // one walk for a given share; returns what is left for the last worker, who takes the rest
        auto deal = [&](double target) {
          plan_cuts.assign(static_cast<size_t>(G) + 1, {});
          L->mx_plan_ptr.assign(1, 0);
          n_rec = 0;
          longest = 1;
          double acc = 0.0;
          auto next_worker = [&]() {
            L->mx_plan_ptr.push_back(static_cast<int32_t>(n_rec));
            acc = 0.0;
          };
          for (int32_t s = 0; s <= G; ++s) {
            const int64_t t0 = L->gm_seg_ptr[s], t = L->gm_seg_ptr[s + 1] - t0;
            const int64_t n_u = static_cast<int64_t>(users[s].size());
            if (n_u == 0 || t == 0) continue;
            for (int64_t b = 0; b < (n_u + 63) / 64; ++b) {
              std::vector<int64_t> bounds(1, t0);
              int64_t pos = 0;
              while (pos < t) {
                const bool last = static_cast<int64_t>(L->mx_plan_ptr.size()) >= workers;
                const double room = target - acc - kRunCost;
                const int64_t rem = t - pos;
                if (last || static_cast<double>(rem) <= room + static_cast<double>(kSnap)) {
                  acc += kRunCost + static_cast<double>(rem);  // the rest of the unit is one run
                  longest = std::max(longest, rem);
                  pos = t;
                } else if (room < static_cast<double>(kSnap) && acc > 0.0) {
                  next_worker();  // no room worth a run
                } else {
                  const int64_t take = std::min(rem - kSnap, std::max<int64_t>(kSnap, static_cast<int64_t>(room)));
                  pos += take;
                  bounds.push_back(t0 + pos);
                  longest = std::max(longest, take);
                  n_rec += 1;
                  next_worker();
                }
              }
              bounds.push_back(t0 + t);
              n_rec += 1;
              plan_cuts[static_cast<size_t>(s)].push_back(std::move(bounds));
            }
          }
          const double last_cost = static_cast<int64_t>(L->mx_plan_ptr.size()) >= workers ? acc : 0.0;
          while (static_cast<int64_t>(L->mx_plan_ptr.size()) < workers) L->mx_plan_ptr.push_back(static_cast<int32_t>(n_rec));
          L->mx_plan_ptr.push_back(static_cast<int32_t>(n_rec));
          return last_cost;
        };
        L->mx_plan_workers = static_cast<int32_t>(nominal);
        // the smallest share with which the last worker is left no more than the others (the number of
        // runs, and with it the total cost, depends on the share itself)
        double lo = static_cast<double>(line) / static_cast<double>(workers);
        // (a worker stops less than kRunCost + kSnap short of the share, and there are at most units + W runs:
        // with this share the last worker is sure to be left no more than the others)
        double hi = (static_cast<double>(line) + kRunCost * static_cast<double>(n_units + workers)) / static_cast<double>(workers) +
                    kRunCost + 2.0 * static_cast<double>(kSnap);
        for (int it = 0; it < 24; ++it) {
          const double mid = 0.5 * (lo + hi);
          (deal(mid) <= mid + static_cast<double>(kSnap) ? hi : lo) = mid;
        }
        deal(hi);
        plan_fill = static_cast<float>(used / rows);
      }
    }
    L->gm_chunk_tiles = static_cast<int32_t>(chunk);
    // displacement of segment s for user u, as in list_shift but without a tile offset
    std::vector<int32_t> seg_shift(static_cast<size_t>(B) * (G + 1), 0);
    for (int32_t u = 0; u < B; ++u) {
      seg_shift[static_cast<size_t>(u) * (G + 1)] = L->cache_len[u];
      int64_t new_first = S;
      for (int32_t e = sel->sel_ptr[u]; e < sel->sel_ptr[u + 1]; ++e) {
        const int32_t g = sel->sel_idx[e];
        seg_shift[static_cast<size_t>(u) * (G + 1) + g + 1] = static_cast<int32_t>(L->cache_len[u] - (new_first - group[g].begin));
        new_first += group[g].end - group[g].begin;
      }
    }
    std::vector<int64_t> n_slots(B, 0);
    // first pass: count slots per query; second pass: emit items with absolute slot numbers
    for (int pass = 0; pass < 2; ++pass) {
      std::vector<int64_t> next(B, 0);
      if (pass == 1) {
        L->gm_slot_ptr.assign(static_cast<size_t>(B) + 1, 0);
        for (int32_t u = 0; u < B; ++u) L->gm_slot_ptr[u + 1] = L->gm_slot_ptr[u] + n_slots[u] + 1;  // + own cache
      }
      for (int32_t s = 0; s <= G; ++s) {
        const int64_t t0 = L->gm_seg_ptr[s], t1 = L->gm_seg_ptr[s + 1];
        if (users[s].empty()) continue;
        // the segment's tiles are cut into ceil(tiles / chunk) runs of equal length (to within one
        // tile): a short last run would leave its workgroup idle while the full ones finish
        const int64_t n_runs = (t1 - t0 + chunk - 1) / chunk;
        for (int64_t run = 0; run < n_runs; ++run) {
          const int64_t c0 = t0 + run * (t1 - t0) / n_runs, c1 = t0 + (run + 1) * (t1 - t0) / n_runs;
          for (size_t b0 = 0; b0 < users[s].size(); b0 += kItemQueries) {
            const size_t b1 = std::min(users[s].size(), b0 + kItemQueries);
            if (pass == 1)
              L->gm_items.insert(L->gm_items.end(),
                                 {static_cast<int32_t>(c0), static_cast<int32_t>(c1 - c0),
                                  static_cast<int32_t>(L->gm_qrefs.size() / 2), static_cast<int32_t>(b1 - b0)});
            for (size_t k = b0; k < b1; ++k) {
              const int32_t u = users[s][k];
              if (pass == 0)
                ++n_slots[u];
              else {
                L->gm_qrefs.push_back(u);
                L->gm_qrefs.push_back(static_cast<int32_t>(L->gm_slot_ptr[u] + next[u]++));
                L->gm_qshift.push_back(seg_shift[static_cast<size_t>(u) * (G + 1) + s]);
              }
            }
          }
        }
      }
    }
    if (!plan_cuts.empty()) {
      plan_users = users;
      plan_shift = seg_shift;
    }
  }

  for (size_t i = 3; i < L->gm_items.size(); i += 4) L->gm_max_queries = std::max(L->gm_max_queries, L->gm_items[i]);
  for (const int32_t shift : L->gm_qshift) L->max_decode_shift = std::max<int64_t>(L->max_decode_shift, shift);
  if (!plan_cuts.empty()) {
    // Records of the runs cut to measure, with references and slots of their own (the work items above keep
    // their runs of one length for the steps that do not run as a contraction): per unit, run by run, the
    // unit's users with one slot each; a query's last slot is again its own cache.
    const int32_t B = L->n_queries;
    std::vector<int64_t> n_slots(static_cast<size_t>(B), 0), next(static_cast<size_t>(B), 0);
    for (int pass = 0; pass < 2; ++pass) {
      if (pass == 1) {
        L->mx_slot_ptr.assign(static_cast<size_t>(B) + 1, 0);
        for (int32_t u = 0; u < B; ++u) L->mx_slot_ptr[u + 1] = L->mx_slot_ptr[u] + n_slots[u] + 1;
      }
      for (size_t s = 0; s < plan_cuts.size(); ++s)
        for (size_t b = 0; b < plan_cuts[s].size(); ++b)
          for (size_t run = 0; run + 1 < plan_cuts[s][b].size(); ++run) {
            const size_t b0 = 64 * b, b1 = std::min(plan_users[s].size(), b0 + 64);
            if (pass == 1)
              L->mx_rec.insert(L->mx_rec.end(),
                               {static_cast<int32_t>(L->mx_qrefs.size() / 2), static_cast<int32_t>(b1 - b0),
                                static_cast<int32_t>(plan_cuts[s][b][run]),
                                static_cast<int32_t>(plan_cuts[s][b][run + 1] - plan_cuts[s][b][run])});
            for (size_t k = b0; k < b1; ++k) {
              const int32_t u = plan_users[s][k];
              if (pass == 0) {
                ++n_slots[static_cast<size_t>(u)];
              } else {
                L->mx_qrefs.push_back(u);
                L->mx_qrefs.push_back(static_cast<int32_t>(L->mx_slot_ptr[u] + next[static_cast<size_t>(u)]++));
                L->mx_qshift.push_back(plan_shift[static_cast<size_t>(u) * plan_cuts.size() + s]);
              }
            }
          }
    }
    L->mx_row_fill = plan_fill;
  } else {
    // No plan: the work items' runs with up to 64 queries each: consecutive items of one run (its batches of
    // 32 queries, whose references follow each other) are taken in pairs.  Slots do not change.
    const size_t n_items = L->gm_items.size() / 4;
    double rows = 0.0, used = 0.0;
    for (size_t it = 0; it < n_items; ++it) {
      const int32_t* a = &L->gm_items[4 * it];
      int32_t n_q = a[3];
      if (it + 1 < n_items) {
        const int32_t* b = a + 4;
        if (b[0] == a[0] && b[1] == a[1] && b[2] == a[2] + a[3] && a[3] == 32) {
          n_q += b[3];
          ++it;
        }
      }
      L->mx_rec.insert(L->mx_rec.end(), {a[2], n_q, a[0], a[1]});
      rows += 64.0 * a[1];
      used += static_cast<double>(n_q) * a[1];
    }
    L->mx_row_fill = rows > 0.0 ? static_cast<float>(used / rows) : 0.f;
  }
  {
    const size_t n_items = L->gm_items.size() / 4;
    L->gm_item_run.resize(n_items * 4);
    L->gm_ref_pad.resize(n_items * 32 * 4);
    for (size_t it = 0; it < n_items; ++it) {
      const int32_t ent_begin = L->gm_items[4 * it], ent_count = L->gm_items[4 * it + 1];
      const int32_t ref_begin = L->gm_items[4 * it + 2], n_q = L->gm_items[4 * it + 3];
      // tiles of one segment follow each other without gaps and all but the last are full
      L->gm_item_run[4 * it + 0] = L->gm_seg_ent[2 * ent_begin];
      L->gm_item_run[4 * it + 1] = block_n * (ent_count - 1) + (L->gm_seg_ent[2 * (ent_begin + ent_count - 1) + 1] & 0xFFFF);
      L->gm_item_run[4 * it + 2] = n_q;
      L->gm_item_run[4 * it + 3] = 0;
      for (int32_t j = 0; j < 32; ++j) {
        const int32_t ref = ref_begin + std::min(j, n_q - 1);
        int32_t* dst = &L->gm_ref_pad[(it * 32 + j) * 4];
        dst[0] = L->gm_qrefs[2 * ref];
        dst[1] = L->gm_qrefs[2 * ref + 1];
        dst[2] = L->gm_qshift[ref];
        dst[3] = 0;
      }
    }
  }
  if (L->query_stage) {
    const int32_t n_items = static_cast<int32_t>(L->gm_items.size() / 4);
    const int32_t pool_blocks = (n_items + 7) / 8;
    for (int k = 0; k < 6; ++k) {
      const int32_t per_wave = 32 >> k;
      std::vector<int32_t> batches(static_cast<size_t>(pool_blocks), 0);
      int64_t more = 0;
      for (int32_t b = 0; b < pool_blocks; ++b) {
        int32_t most = 0;
        for (int32_t it = 8 * b; it < std::min(n_items, 8 * b + 8); ++it) most = std::max(most, L->gm_items[4 * it + 3]);
        batches[static_cast<size_t>(b)] = (most + per_wave - 1) / per_wave;
        more += batches[static_cast<size_t>(b)] - 1;
      }
      // While few blocks have a second batch the first batches need no table (one look-up less in front of the first
      // tiles); otherwise the batches of a block stay next to each other, all in the table.  us with the table / without:
      // no second batches, 32/8 heads, one question 25.9 / 25.7, 8 questions 81.1 / 80.8; for 0.09 of the blocks, 24 of 100
      // groups 83.2 / 80.8; 0.10, 16 questions 86.1 / 85.8; 0.20, 20 questions 87.4 / 87.9; 0.35, 22 questions 91.6 / 94.4.
      L->gm_direct[k] = 4 * more <= pool_blocks ? pool_blocks : 0;
      L->gm_rows_off[k] = static_cast<int32_t>(L->gm_rows.size());
      for (int32_t b = 0; b < pool_blocks; ++b)
        for (int32_t z = L->gm_direct[k] ? 1 : 0; z < batches[static_cast<size_t>(b)]; ++z) L->gm_rows.push_back((b << 8) | z);
      // how often a key of the pool items is walked when a wave takes per_wave queries
      double keys = 0.0, walked = 0.0;
      for (int32_t it = 0; it < n_items; ++it) {
        const double n = L->gm_item_run[4 * it + 1];
        keys += n;
        walked += n * ((L->gm_item_run[4 * it + 2] + per_wave - 1) / per_wave);
      }
      L->gm_walks_per_key[k] = keys > 0.0 ? static_cast<float>(walked / keys) : 1.f;
    }
    L->gm_rows_off[6] = static_cast<int32_t>(L->gm_rows.size());
  }
  L->shortest_list = INT64_MAX;
  for (int64_t t = 0; t < L->n_qtiles(); ++t) {
    L->shortest_list = std::min(L->shortest_list, L->list_ptr[t + 1] - L->list_ptr[t]);
    L->longest_list = std::max(L->longest_list, L->list_ptr[t + 1] - L->list_ptr[t]);
    L->largest_tile = std::max(L->largest_tile, L->qtile_tab[4 * t + 1]);
    if (!L->list_shift.empty())
      for (int64_t e = L->list_ptr[t]; e < L->list_ptr[t + 1]; ++e)
        L->max_rotation_id = std::max<int64_t>(L->max_rotation_id,
                                               static_cast<int64_t>(L->list_shift[e]) + L->qtile_tab[4 * t + 1] - 1);
  }
  if (L->n_qtiles() == 0) L->shortest_list = 0;

  // launch order: owner by owner (a group at pre-encoding, a query at the query stage), the
  // longest list of an owner first.  Q tiles of one owner walk the same KV, so keeping them
  // adjacent keeps that KV in the L2 of the XCD that runs them.
  // At the query stage the owners themselves are put in the order of their selections (the lists
  // of selected groups compared word by word, then the query index): queries that start with the
  // same groups then run side by side and walk the same keys at about the same time, which is what
  // lets many queries with small selections share the L2 of the XCD that serves a KV head.
  const int64_t nt = L->n_qtiles();
  std::vector<int32_t> owner_rank;
  if (L->query_stage && sel) {
    std::vector<int32_t> by_sel(static_cast<size_t>(sel->n_queries));
    std::iota(by_sel.begin(), by_sel.end(), 0);
    std::stable_sort(by_sel.begin(), by_sel.end(), [&](int32_t a, int32_t b) {
      return std::lexicographical_compare(sel->sel_idx + sel->sel_ptr[a], sel->sel_idx + sel->sel_ptr[a + 1],
                                          sel->sel_idx + sel->sel_ptr[b], sel->sel_idx + sel->sel_ptr[b + 1]);
    });
    owner_rank.resize(by_sel.size());
    for (size_t i = 0; i < by_sel.size(); ++i) owner_rank[static_cast<size_t>(by_sel[i])] = static_cast<int32_t>(i);
  }
  auto rank_of = [&](int32_t owner) {
    return owner >= 0 && static_cast<size_t>(owner) < owner_rank.size() ? owner_rank[static_cast<size_t>(owner)] : owner;
  };
  L->order.resize(nt);
  std::iota(L->order.begin(), L->order.end(), 0);
  std::stable_sort(L->order.begin(), L->order.end(), [&](int32_t a, int32_t b) {
    const int32_t oa = rank_of(L->qtile_tab[4 * a + 2]), ob = rank_of(L->qtile_tab[4 * b + 2]);
    if (oa != ob) return oa < ob;
    return (L->list_ptr[a + 1] - L->list_ptr[a]) > (L->list_ptr[b + 1] - L->list_ptr[b]);
  });
  for (int64_t i = nt; i > 0 && L->qtile_tab[4 * L->order[static_cast<size_t>(i - 1)] + 2] == L->qtile_tab[4 * L->order.back() + 2]; --i)
    L->last_owner_tiles += 1;
  return DBSA_OK;
}

void dbsa_balance_records(const std::vector<int32_t>& rec_in, int32_t n_classes, std::vector<int32_t>* class_ptr,
                          std::vector<int32_t>* rec) {
  const int64_t nt = static_cast<int64_t>(rec_in.size() / 4);
  std::vector<int64_t> load(static_cast<size_t>(n_classes), 0);
  std::vector<std::vector<int32_t>> recs_of(static_cast<size_t>(n_classes));
  std::vector<int32_t> round, by_load(static_cast<size_t>(n_classes));
  auto entries = [&](int32_t t) { return static_cast<int64_t>(rec_in[4 * static_cast<size_t>(t) + 3]); };
  for (int64_t a = 0; a < nt; a += n_classes) {
    const int64_t b = std::min<int64_t>(nt, a + n_classes);
    round.resize(static_cast<size_t>(b - a));
    std::iota(round.begin(), round.end(), static_cast<int32_t>(a));
    std::stable_sort(round.begin(), round.end(), [&](int32_t x, int32_t y) { return entries(x) > entries(y); });
    std::iota(by_load.begin(), by_load.end(), 0);
    std::stable_sort(by_load.begin(), by_load.end(), [&](int32_t x, int32_t y) { return load[x] < load[y]; });
    for (size_t i = 0; i < round.size(); ++i) {
      const int32_t c = by_load[i];
      recs_of[c].push_back(round[i]);
      load[c] += entries(round[i]) + kTileCost;
    }
  }
  class_ptr->assign(static_cast<size_t>(n_classes) + 1, 0);
  rec->clear();
  rec->reserve(rec_in.size());
  for (int32_t c = 0; c < n_classes; ++c) {
    for (int32_t t : recs_of[c]) rec->insert(rec->end(), rec_in.begin() + 4 * static_cast<size_t>(t), rec_in.begin() + 4 * static_cast<size_t>(t) + 4);
    (*class_ptr)[c + 1] = static_cast<int32_t>(rec->size() / 4);
  }
}

namespace {
// the first n Q tiles in launch order as records
std::vector<int32_t> tile_records(const dbsa_layout* L, int64_t n) {
  std::vector<int32_t> rec;
  rec.reserve(static_cast<size_t>(n) * 4);
  for (int64_t i = 0; i < n; ++i) {
    const int32_t t = L->order[static_cast<size_t>(i)];
    rec.push_back(L->qtile_tab[4 * t + 0]);
    rec.push_back(L->qtile_tab[4 * t + 1]);
    rec.push_back(static_cast<int32_t>(L->list_ptr[t]));
    rec.push_back(static_cast<int32_t>(L->list_ptr[t + 1] - L->list_ptr[t]));
  }
  return rec;
}
}  // namespace

void dbsa_balance_schedule(const dbsa_layout* L, int32_t n_classes, std::vector<int32_t>* class_ptr,
                           std::vector<int32_t>* rec) {
  dbsa_balance_records(tile_records(L, L->n_qtiles()), n_classes, class_ptr, rec);
}

int64_t dbsa_cut_workers(const dbsa_layout* L, int64_t n_classes) {
  // (a share of fewer entries than it costs to start, finish and merge a piece is not worth a worker)
  constexpr int64_t kMinShare = 6;
  return std::max<int64_t>(1, std::min<int64_t>(n_classes, L->n_ent() / kMinShare));
}

namespace {
// Lists dealt to workers: the first n_whole tiles of `tiles` whole, in rounds, the others cut to measure.
struct CutPlan {
  struct Piece {
    int64_t tile, first, take, worker;  // tile: index in `tiles`
  };
  std::vector<int32_t> whole_ptr, whole_rec;
  std::vector<Piece> pieces;
  double cost = 0.0;  // of the busiest worker
};

// stray: cost of an entry of a piece over that of a whole tile's
CutPlan plan_cuts(const std::vector<int32_t>& tiles, int64_t n_whole, int64_t workers, double stray) {
  CutPlan plan;
  const int64_t nt = static_cast<int64_t>(tiles.size() / 4);
  plan.whole_ptr.assign(static_cast<size_t>(workers) + 1, 0);
  if (n_whole > 0)
    dbsa_balance_records(std::vector<int32_t>(tiles.begin(), tiles.begin() + 4 * n_whole), static_cast<int32_t>(workers),
                         &plan.whole_ptr, &plan.whole_rec);
  std::vector<int64_t> load(static_cast<size_t>(workers), 0);
  int64_t total = 0, rest = 0;
  for (size_t c = 0; c < load.size(); ++c) {
    for (int32_t k = plan.whole_ptr[c]; k < plan.whole_ptr[c + 1]; ++k) load[c] += plan.whole_rec[4 * static_cast<size_t>(k) + 3] + kTileCost;
    total += load[c];
  }
  const int64_t heaviest = *std::max_element(load.begin(), load.end());
  for (int64_t i = n_whole; i < nt; ++i) rest += tiles[4 * static_cast<size_t>(i) + 3];
  // One walk over the rest for a given share; returns the load of the last worker, who takes what is left.
  auto deal = [&](int64_t share) {
    plan.pieces.clear();
    int64_t w = 0, acc = load[0];
    for (int64_t i = n_whole; i < nt; ++i) {
      const int64_t first = tiles[4 * static_cast<size_t>(i) + 2], n = tiles[4 * static_cast<size_t>(i) + 3];
      for (int64_t pos = 0; pos < n;) {
        const int64_t room = share - acc - kPieceCost, rem = n - pos;
        int64_t take = rem;
        if (w + 1 < workers && rem > room) {
          // cut here, or leave the tile to the next worker where a piece would come out too short; a worker
          // that has nothing yet always takes something
          take = std::min(room, rem - kMinPiece);
          if (take < kMinPiece && acc > 0) {
            acc = load[static_cast<size_t>(++w)];
            continue;
          }
          if (take < kMinPiece) take = rem < 2 * kMinPiece ? rem : kMinPiece;
        }
        acc += kPieceCost + take;
        plan.pieces.push_back({i, first + pos, take, w});
        pos += take;
        if (w + 1 < workers && acc + kPieceCost + kMinPiece > share) acc = load[static_cast<size_t>(++w)];
      }
    }
    return w + 1 < workers ? int64_t{0} : acc;
  };
  // The smallest share with which the last worker is left no more than the others.  (With `hi` it surely is: a
  // worker stops less than kPieceCost + 2 kMinPiece short of its share, and there are at most nt + workers records.)
  int64_t lo = (total + rest) / workers - 1;
  int64_t hi = heaviest + (rest + kPieceCost * (nt + workers)) / workers + kPieceCost + 2 * kMinPiece + 1;
  while (lo + 1 < hi) {
    const int64_t mid = (lo + hi) / 2;
    (deal(mid) <= mid ? hi : lo) = mid;
  }
  deal(hi);
  std::vector<double> cost(load.begin(), load.end());
  for (const CutPlan::Piece& x : plan.pieces) cost[static_cast<size_t>(x.worker)] += stray * static_cast<double>(x.take) + kPieceCost;
  plan.cost = *std::max_element(cost.begin(), cost.end());
  return plan;
}
}  // namespace

// With several Q tiles per worker, whole tiles go round first and only what does not fill a round is cut.  Tiles next to
// each other in launch order selected the same groups, and in a round the workers walk them side by side: a group is
// fetched once for all of them.  Cutting the whole order to measure instead, a stretch of it to each worker, sends
// every worker through other groups: 300 questions of 32 tokens over 64 workers 1443 us against 1182 with whole tiles
// (4.7 rounds) and 1190 in rounds, 140 questions 707 / 659 / 574, 70 questions 362 / 433 / 311.  An entry of a piece
// costs about 1.13 times what it costs in step, 1.4 times where everything is cut over several tiles per worker, which
// only lists of very different lengths are worth.
void dbsa_cut_schedule(const dbsa_layout* L, int32_t n_classes) {
  const int64_t nt = L->n_qtiles(), workers = dbsa_cut_workers(L, n_classes);
  const std::vector<int32_t> tiles = tile_records(L, nt);
  CutPlan plan = plan_cuts(tiles, nt / workers * workers, workers, 1.13);
  if (nt >= workers && plan.cost > 1.4 * static_cast<double>(L->n_ent() / workers + kPieceCost)) {
    CutPlan all = plan_cuts(tiles, 0, workers, 1.4);
    if (all.cost < plan.cost) plan = std::move(all);
  }
  // ---- a worker's whole tiles, then its pieces; the pieces of a cut tile get partial rows ----
  L->cut_rec.clear();
  L->cut_part.clear();
  L->cut_tab.clear();
  L->cut_rows = 0;
  std::vector<int64_t> part(plan.pieces.size(), -1);
  for (size_t a = 0, b; a < part.size(); a = b) {
    for (b = a + 1; b < part.size() && plan.pieces[b].tile == plan.pieces[a].tile;) ++b;
    if (b - a == 1) continue;
    const int32_t* tile = &tiles[4 * static_cast<size_t>(plan.pieces[a].tile)];
    L->cut_tab.insert(L->cut_tab.end(), {tile[0], tile[1], static_cast<int32_t>(L->cut_rows), static_cast<int32_t>(b - a)});
    for (size_t k = a; k < b; ++k, L->cut_rows += tile[1]) part[k] = L->cut_rows;
  }
  L->cut_ptr.assign(static_cast<size_t>(n_classes) + 1, 0);
  size_t k = 0;
  for (int64_t c = 0; c < n_classes; ++c) {
    if (c < workers) {
      L->cut_rec.insert(L->cut_rec.end(), plan.whole_rec.begin() + 4 * plan.whole_ptr[static_cast<size_t>(c)],
                        plan.whole_rec.begin() + 4 * plan.whole_ptr[static_cast<size_t>(c) + 1]);
      L->cut_part.resize(L->cut_rec.size() / 4, -1);
      for (; k < part.size() && plan.pieces[k].worker == c; ++k) {
        const int32_t* tile = &tiles[4 * static_cast<size_t>(plan.pieces[k].tile)];
        L->cut_rec.insert(L->cut_rec.end(), {tile[0], tile[1], static_cast<int32_t>(plan.pieces[k].first),
                                             static_cast<int32_t>(plan.pieces[k].take)});
        L->cut_part.push_back(static_cast<int32_t>(part[k]));
      }
    }
    L->cut_ptr[static_cast<size_t>(c) + 1] = static_cast<int32_t>(L->cut_part.size());
  }
  L->cut_cost = plan.cost;
  // the same workers with whole Q tiles, for dbsa_cut_worth
  L->cut_whole = 0;
  if (nt >= 2 * n_classes) {
    std::vector<int32_t> ptr, rec;
    dbsa_balance_schedule(L, n_classes, &ptr, &rec);
    for (int32_t c = 0; c < n_classes; ++c) {
      int64_t load = 0;
      for (int32_t k = ptr[static_cast<size_t>(c)]; k < ptr[static_cast<size_t>(c) + 1]; ++k) load += rec[4 * static_cast<size_t>(k) + 3] + kTileCost;
      L->cut_whole = std::max(L->cut_whole, load);
    }
  }
  L->cut_classes = n_classes;
}

namespace {
// what an entry costs with two waves to a SIMD (1.74 us beside another wave), in entries of a wave alone (1.21)
constexpr double kBesideCost = 1.44;
}  // namespace

// Two waves fill each other's gaps, but a list beside another runs at 0.7 of its speed: it takes work for most of the places,
// and a launch whose longest list decides only loses.  16/16 heads, 128-token tiles, encoding two groups of 3650 tokens 78 us
// with one wave to a SIMD and 94 with two, of 4500 115 / 128, of 5500 169 / 155; twenty groups of 450 tokens 35 / 33;
// 32/8 heads, one group of 4400 tokens 104 / 100, of 5200 139 / 129, of 3600 76 / 77; four groups of 900 38 / 29.  Questions
// without a workspace: 48 of 64 tokens over 64 workers 289 / 245, 66 427 / 375, 100 of 20 tokens over 128 305 / 250 (nothing
// below three quarters was measured); one that selects 16 times as many groups as the 55 others 158 / 165.  Lists that can
// be cut to measure take four fifths: over 64 workers 40 questions 195 cut for one wave each, 48 231 / 245, 52 253 / 250,
// 60 292 / 262; fewer gain or lose and keep one wave (1 question of 64 tokens 30.6 / 22.3, 5 39.9 / 41.6, 20 118 / 108,
// 30 149 / 154; 1 of 400 51.6 / 48.8, 4 153 / 139; 5 ragged ones 67 / 66).  More workers than a schedule can name leave the launch to the order of the lists, or their cuts to half
// the places: 4/1 heads, 1200 questions of 30 tokens 114 / 167, encoding 60000 tokens 127 / 143; with one list per worker
// they gain, 900 questions 88 / 80, 32000 tokens 63 / 53.
bool dbsa_crowd_worth(const dbsa_layout* L, int64_t classes, bool cuts) {
  const int64_t nt = L->n_qtiles(), alone = classes / 2;
  if (nt == 0 || alone < 1) return false;
  const bool encoding = !L->query_stage, listed = classes <= kMaxSchedClasses;
  if (encoding ? 10 * nt < 9 * classes : cuts ? 5 * nt < 4 * classes : 4 * nt < 3 * classes) return false;
  if (!listed && nt > classes && (encoding || cuts)) return false;
  if (cuts) return true;
  // entries of the busiest of n workers, by the longest list, by all entries, and by how many lists it takes
  auto busiest = [&](int64_t n, int64_t per_tile) {
    return std::max({static_cast<double>(L->longest_list + per_tile), static_cast<double>(L->n_ent() + per_tile * nt) / static_cast<double>(n),
                     static_cast<double>((nt + n - 1) / n * (L->shortest_list + per_tile))});
  };
  // one wave to a SIMD; without a schedule the lists start in launch order, those of the last owner when the work of the
  // others is nearly done
  const bool dealt = nt >= 2 * alone;
  double single = busiest(alone, dealt ? kTileCost : kPieceCost);
  const int64_t before = nt - L->last_owner_tiles;
  if (!dealt && encoding && before >= alone)
    single = std::max(single, static_cast<double>(L->n_ent() + kPieceCost * nt) / static_cast<double>(alone) * static_cast<double>(before) /
                                      static_cast<double>(nt) + static_cast<double>(L->longest_list));
  // two: beside the longest list lies one of middling length (the lists are dealt longest first)
  const double beside = static_cast<double>(L->n_ent() + kTileCost * nt) / static_cast<double>(classes);
  double both = busiest(classes, kTileCost) + (kBesideCost - 1.0) * beside;
  if (!encoding && nt > classes && (!listed || nt < 2 * classes)) {  // no schedule: rounds, the last one perhaps not full
    const int64_t rounds = (nt + classes - 1) / classes;
    const double fill = static_cast<double>(nt - (rounds - 1) * classes) / static_cast<double>(classes);
    const double cost = kBesideCost * static_cast<double>(rounds - 1) + 1.0 + (kBesideCost - 1.0) * std::min(1.0, 4.0 * fill);
    both = std::max(both, cost * static_cast<double>(L->shortest_list + kPieceCost));
  }
  return both < single;
}

// Against whole Q tiles dealt to the same workers, and while there are fewer tiles than workers against runs of one length,
// one per workgroup, which walk in step and have one record each to start and finish: 29 questions of 64 tokens over 32
// workers take 713 us whole and 779 cut to measure, 14 take 378 in two runs each and 390 cut, one takes 58 in 32 pieces.
// The partial states of either are priced by their bytes.  An entry costs `crowd` times as much with every place taken as
// with few: a K/V pair serves 32 rows per row block, and 256 rows keep the matrix pipes busy at the rate the pairs
// arrive.  Two small workgroups per compute unit fetch a pair per 128 rows each and are bound by that traffic (512 of them
// move 7.4 TB/s; 50 questions of 20 tokens on 400 of 512 places: whole lists 771 us, all places with cut lists 803).
// Eight row blocks with two waves to a SIMD are priced like one: with kBesideCost instead 41 prefills of 52 to 800 questions
// took the same time to 1 % (200 of 20 tokens 456 us so and 468 with it, 220 of them 509 and 501).
bool dbsa_cut_worth(const dbsa_layout* L, int row_blocks) {
  const int64_t nt = L->n_qtiles();
  const double crowd = row_blocks == 8 ? 1.0 : row_blocks == 4 ? 1.5 : 3.0;
  const double classes = static_cast<double>(L->cut_classes), heads = std::max(1, row_blocks * 32 / std::max(1, L->block_m));
  auto per_entry = [&](int64_t busy) { return std::max(1.0, crowd * std::min(1.0, static_cast<double>(busy) / classes)); };
  auto merge = [&](int64_t rows) { return rows > 0 ? static_cast<double>(rows) * heads / classes * kStateCost + 2.0 : 0.0; };
  const double cut = 1.03 * (L->cut_cost * per_entry(dbsa_cut_workers(L, L->cut_classes)) + merge(L->cut_rows));
  if (nt >= 2 * L->cut_classes) return cut < static_cast<double>(L->cut_whole) * per_entry(nt);
  // (query_runs() splits lists only while whole ones leave places free)
  const int64_t top = nt < L->cut_classes ? std::max<int64_t>(1, std::min(kMaxQuerySplit, L->shortest_list / kMinRun)) : 1;
  double other = 1e30;
  for (int64_t runs = 1; runs <= top; ++runs)
    other = std::min(other, static_cast<double>((nt * runs + L->cut_classes - 1) / L->cut_classes) *
                                    (static_cast<double>(L->longest_list) / static_cast<double>(runs) * per_entry(nt * runs) + kPieceCost) +
                                merge(runs > 1 ? runs * L->n_query_tokens : 0));
  return cut < other;
}
