// Host side of the library: tree metadata (dta_tree_build and friends) and the
// DFS tile schedule.  Integer work only; nothing here touches the GPU.
//
// The tree is the rollout prefix tree of paper section 3 (problem formulation):
// nodes are token segments, root-to-leaf paths are rollouts, and path length is
// counted in tokens.  Nodes are packed in DFS preorder (any DFS order is valid,
// section 4); in that order the tokens that can see key k form the contiguous
// range [k, kend[k]) where kend[k] is the end of the subtree of k's node, which
// is what the kernels use as their visibility mask.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <new>
#include <numeric>
#include <type_traits>

#include "dta_internal.h"

namespace {

int build_impl(const int32_t* parent, const int32_t* seg_len, int32_t n, dta_tree* t) {
  t->n_nodes = n;
  t->parent.assign(parent, parent + n);
  t->seg_len.assign(seg_len, seg_len + n);

  int64_t total = 0;
  for (int32_t i = 0; i < n; ++i) {
    if (parent[i] < -1 || parent[i] >= n || parent[i] == i) return DTA_ERR_BAD_TREE;
    if (seg_len[i] < 1) return DTA_ERR_BAD_TREE;
    total += seg_len[i];
  }
  // leave room so that tile-padded indices still fit in int32
  if (total > (int64_t)std::numeric_limits<int32_t>::max() - 4096) return DTA_ERR_BAD_TREE;

  // children in CSR form; filling in ascending i keeps each list ascending
  std::vector<int32_t> child_ptr(n + 1, 0), child(n > 0 ? n : 1), roots;
  for (int32_t i = 0; i < n; ++i) {
    if (parent[i] >= 0) child_ptr[parent[i] + 1]++;
    else roots.push_back(i);
  }
  for (int32_t i = 0; i < n; ++i) child_ptr[i + 1] += child_ptr[i];
  {
    std::vector<int32_t> fill(child_ptr.begin(), child_ptr.end() - 1);
    for (int32_t i = 0; i < n; ++i)
      if (parent[i] >= 0) child[fill[parent[i]]++] = i;
  }

  // iterative preorder; nodes on a parent cycle are never reached from a root
  t->dfs_order.clear();
  t->dfs_order.reserve(n);
  {
    std::vector<int32_t> stack;
    for (auto it = roots.rbegin(); it != roots.rend(); ++it) stack.push_back(*it);
    while (!stack.empty()) {
      int32_t u = stack.back();
      stack.pop_back();
      t->dfs_order.push_back(u);
      for (int32_t c = child_ptr[u + 1] - 1; c >= child_ptr[u]; --c) stack.push_back(child[c]);
    }
  }
  if ((int32_t)t->dfs_order.size() != n) return DTA_ERR_BAD_TREE;

  t->node_offset.assign(n, 0);
  t->node_start_depth.assign(n, 0);
  t->subtree_tokens.assign(n, 0);
  std::vector<int32_t> depth_nodes(n, 1);
  int64_t pos = 0;
  for (int32_t r = 0; r < n; ++r) {
    int32_t u = t->dfs_order[r];
    t->node_offset[u] = pos;
    pos += seg_len[u];
    int32_t p = parent[u];
    if (p >= 0) {
      t->node_start_depth[u] = t->node_start_depth[p] + seg_len[p];
      depth_nodes[u] = depth_nodes[p] + 1;
    }
  }
  for (int32_t r = n - 1; r >= 0; --r) {
    int32_t u = t->dfs_order[r];
    t->subtree_tokens[u] += seg_len[u];
    if (parent[u] >= 0) t->subtree_tokens[parent[u]] += t->subtree_tokens[u];
  }

  // per-node ancestor key intervals, root first, merged when contiguous
  t->anc_ptr.assign(n + 1, 0);
  t->anc_seg_off.clear();
  t->anc_seg_len.clear();
  {
    std::vector<int32_t> path;
    for (int32_t u = 0; u < n; ++u) {
      path.clear();
      for (int32_t a = parent[u]; a >= 0; a = parent[a]) path.push_back(a);
      size_t first = t->anc_seg_off.size();
      for (auto it = path.rbegin(); it != path.rend(); ++it) {
        int64_t off = t->node_offset[*it], len = seg_len[*it];
        if (t->anc_seg_off.size() > first &&
            t->anc_seg_off.back() + t->anc_seg_len.back() == off) {
          t->anc_seg_len.back() += len;
        } else {
          t->anc_seg_off.push_back(off);
          t->anc_seg_len.push_back(len);
        }
      }
      t->anc_ptr[u + 1] = (int64_t)t->anc_seg_off.size();
    }
  }

  t->token_kend.resize((size_t)total);
  t->token_node.resize((size_t)total);
  for (int32_t u = 0; u < n; ++u) {
    int64_t off = t->node_offset[u];
    int32_t kend = (int32_t)(off + t->subtree_tokens[u]);
    for (int32_t j = 0; j < seg_len[u]; ++j) {
      t->token_kend[(size_t)(off + j)] = kend;
      t->token_node[(size_t)(off + j)] = u;
    }
  }

  dta_tree_info_t& inf = t->info;
  std::memset(&inf, 0, sizeof(inf));
  inf.n_nodes = n;
  inf.n_tokens = total;
  inf.n_roots = (int64_t)roots.size();
  for (int32_t u = 0; u < n; ++u) {
    int64_t len = seg_len[u], sd = t->node_start_depth[u], end = sd + len;
    bool leaf = child_ptr[u + 1] == child_ptr[u];
    inf.unique_pairs += len * sd + len * (len + 1) / 2;
    inf.rollout_tokens_full += end;
    inf.dense_pairs_full += end * (end + 1) / 2;
    if (leaf) {
      inf.n_leaves++;
      inf.rollout_tokens += end;
      inf.dense_pairs += end * (end + 1) / 2;
    }
    inf.max_path_tokens = std::max(inf.max_path_tokens, end);
    inf.max_depth_nodes = std::max<int64_t>(inf.max_depth_nodes, depth_nodes[u]);
  }
  return DTA_OK;
}

}  // namespace

namespace dta {

namespace {
// Work items are launched longest first (the hardware hands out blocks in index
// order), but only by power-of-two cost class: inside a class the DFS order is
// kept, so blocks that run at the same time stream neighbouring rows.
int64_t order_key(int64_t cost) {
  int64_t b = 0;
  while ((cost >> b) > 1) ++b;
  return b;
}
}  // namespace

// Both work lists cut the packed token order into fixed runs of bm (bn) tokens,
// whatever the node boundaries.  A tile pays for all of its padded rows anyway,
// and the keys (queries) a run of consecutive DFS tokens needs are the union of
// nested / adjacent intervals, never more than the sum over separate per-node
// tiles, so cutting at node boundaries could only add work.  What a mixed tile
// must not do is let a row see a key outside its own root path: the kernels
// mask with kend[] wherever a key interval is not visible to every row.
namespace {
// adds the chunks a query tile streams, for both chunk sizes of the forward kernel
void count_chunks(QueryTiles& s, const QTile& qt) {
  auto add = [&](int64_t len, bool full) {
    s.fwd_chunks64 += (len + 63) / 64;
    s.fwd_chunks128 += (len + 127) / 128;
    if (!full) s.fwd_masked64 += (len + 63) / 64;
  };
  for (int32_t i = qt.seg_begin; i < qt.seg_end; ++i)
    add(s.segs[(size_t)i].end - s.segs[(size_t)i].start, s.segs[(size_t)i].full != 0);
  add(qt.t1 - qt.t0, false);
}
}  // namespace

namespace {
// copies each tile's first key interval into its record
void fill_first_intervals(QueryTiles& s) {
  for (QTile& t : s.q_tiles)
    t.first = t.seg_begin < t.seg_end ? s.segs[(size_t)t.seg_begin] : KeySeg{t.t0, t.t0, 0, 0};
}
}  // namespace

namespace {
// Cuts the walks of the query tiles into steps (KeyStep).  A step ends early when its
// pieces would lie further apart than the kernels' 32-bit offsets reach.
void cut_steps(QueryTiles& s, int hkv) {
  const int64_t reach = (int64_t)0xffffffff / ((int64_t)hkv * 256) - 32;   // keys; a K/V row is at most 256 bytes per head
  for (const QTile& t : s.q_tiles) {
    StepTile st{};
    st.t0 = t.t0;
    st.t1 = t.t1;
    st.step_begin = (int32_t)s.steps.size();
    KeyStep cur{};
    int used = 0;
    bool first = true;
    auto flush = [&] {
      if (used == 0) return;
      for (; used < 4; ++used) {
        cur.c0[used] = cur.c0[0];
        cur.n[used] = kFullPiece;   // no keys
      }
      if (first) st.first = cur;
      else s.steps.push_back(cur);
      first = false;
      used = 0;
    };
    auto add = [&](int32_t start, int32_t end, int32_t full) {
      for (int32_t c = start; c < end; c += 32) {
        if (used == 4 || (used > 0 && c - (int64_t)cur.c0[0] > reach)) flush();
        cur.c0[used] = c;
        cur.n[used] = std::min(32, end - c) + (full ? kFullPiece : 0);
        ++used;
      }
    };
    for (int32_t i = t.seg_begin; i < t.seg_end; ++i)
      add(s.segs[(size_t)i].start, s.segs[(size_t)i].end, s.segs[(size_t)i].full);
    add(t.t0, t.t1, 0);
    flush();
    st.step_end = (int32_t)s.steps.size();
    s.step_tiles.push_back(st);
  }
}
}  // namespace

size_t partial_bytes(const Schedule& s, int head_dim) {
  return (size_t)s.n_slots * (size_t)s.hkv * 2u * (size_t)s.kv_keys * (size_t)head_dim * sizeof(float);
}

namespace {
// query tiles of bm tokens over the whole tree
void cut_query_tiles(const dta_tree* tree, int bm, QueryTiles& s) {
  const int64_t T = tree->info.n_tokens;
  const auto& parent = tree->parent;
  std::vector<int64_t> cost;
  std::vector<int32_t> path;
  for (int64_t t0 = 0; t0 < T; t0 += bm) {
    int64_t t1 = std::min<int64_t>(T, t0 + bm);
    QTile qt;
    qt.t0 = (int32_t)t0;
    qt.t1 = (int32_t)t1;
    qt.seg_begin = (int32_t)s.segs.size();
    int32_t u0 = tree->token_node[(size_t)t0];
    path.clear();
    for (int32_t a = parent[u0]; a >= 0; a = parent[a]) path.push_back(a);
    int64_t keys = t1 - t0;
    auto add = [&](int64_t start, int64_t end, int64_t kend) {
      int32_t full = kend >= t1 ? 1 : 0;
      if ((int32_t)s.segs.size() > qt.seg_begin && s.segs.back().end == start &&
          s.segs.back().full == full) {
        s.segs.back().end = (int32_t)end;
      } else {
        s.segs.push_back(KeySeg{(int32_t)start, (int32_t)end, full, 0});
      }
      keys += end - start;
    };
    for (auto a = path.rbegin(); a != path.rend(); ++a) {
      int64_t off = tree->node_offset[*a];
      add(off, off + tree->seg_len[*a], off + tree->subtree_tokens[*a]);
    }
    int64_t off0 = tree->node_offset[u0];
    if (t0 > off0) add(off0, t0, off0 + tree->subtree_tokens[u0]);
    qt.seg_end = (int32_t)s.segs.size();
    s.q_tiles.push_back(qt);
    cost.push_back(keys);
    s.fwd_tile_pairs += keys * bm;
    count_chunks(s, qt);
  }
  {
    std::vector<size_t> order(s.q_tiles.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](size_t a, size_t b) { return order_key(cost[a]) > order_key(cost[b]); });
    std::vector<QTile> sorted;
    sorted.reserve(order.size());
    for (size_t i : order) sorted.push_back(s.q_tiles[i]);
    s.q_tiles.swap(sorted);
  }
  fill_first_intervals(s);
}
}  // namespace

Schedule& get_schedule(dta_tree* tree, int bm, int bn, int hkv, int group, const KvWalk& kw) {
  const uint64_t key = schedule_key(bm, bn, hkv, group, kw);
  const int q_rows = kw.q_rows;
  auto it = tree->schedules.find(key);
  if (it != tree->schedules.end()) return it->second;
  // built aside and moved into the map when complete: an allocation failure half
  // way must not leave a partial schedule behind that a later call would use
  Schedule s;
  s.bm = bm;
  s.bn = bn;
  s.q_rows = q_rows;
  s.hkv = hkv;
  s.group = group;
  const int64_t T = tree->info.n_tokens;
  std::vector<int64_t> cost;

  // ---- query tiles (dQ and forward)
  cut_query_tiles(tree, bm, s);
  if (kw.key_steps) cut_steps(s, hkv);
  if (kw.fwd_bm != 0) cut_query_tiles(tree, kw.fwd_bm, s.fwd);

  // ---- key tiles (dK/dV): runs of at most bn consecutive packed keys.  A block
  // walks the union of the query ranges of its keys, [k0, max kend), so a run that
  // mixes keys of small nodes with disjoint or much shorter ranges (leaves of a
  // forest of short segments) keeps its four waves waiting for each other.  The
  // cuts are therefore chosen, by dynamic programming over the packed order, to
  // minimise the summed block time  sum over tiles of (fixed cost + walk steps):
  // a tile either ends at a node boundary or is bn keys long.  On trees of long
  // segments this reproduces the plain cut every bn keys.
  // (the rows of a walk step are a constant of the loop below, the innermost one of the
  // host part: 47 617 tokens in 3795 nodes take 1.8 ms, 2.3 ms with a division by q_rows)
  auto cut_key_tiles_at = [&](int keys, auto rows_per_step) {
    constexpr int64_t kRows = decltype(rows_per_step)::value;
    cost.clear();
    s.kv_tiles.clear();
    s.bwd_tile_pairs = 0;
    s.kv_keys = keys;
    constexpr int64_t kFixedSteps = 7;   // a block's prologue and epilogue cost about 7 walk steps
    const int64_t INF = std::numeric_limits<int64_t>::max() / 4;
    std::vector<int64_t> best((size_t)T + 1, INF);
    std::vector<int32_t> from((size_t)T + 1, -1);
    best[0] = 0;
    const std::vector<int32_t>& order = tree->dfs_order;
    size_t rank_of_q = 0;   // DFS rank of the node that holds position q
    for (int64_t q = 0; q < T; ++q) {
      while (tree->node_offset[(size_t)order[rank_of_q]] + tree->seg_len[(size_t)order[rank_of_q]] <= q) ++rank_of_q;
      const int64_t base = best[(size_t)q];
      if (base == INF) continue;
      int64_t mx = 0;
      const int64_t limit = std::min<int64_t>(T, q + keys);
      for (size_t r = rank_of_q; r < order.size(); ++r) {
        const int32_t u = order[r];
        const int64_t off = tree->node_offset[(size_t)u];
        if (off >= limit) break;
        mx = std::max(mx, off + tree->subtree_tokens[(size_t)u]);
        // the tile ends with this node, or after bn keys inside it
        const int64_t p = std::min(limit, off + tree->seg_len[(size_t)u]);
        const int64_t c = base + kFixedSteps + (mx - q + kRows - 1) / kRows * group;
        if (c < best[(size_t)p]) {   // (on ties the earlier start, visited first, stays)
          best[(size_t)p] = c;
          from[(size_t)p] = (int32_t)q;
        }
      }
    }
    std::vector<int64_t> cuts;
    for (int64_t p = T; p > 0; p = from[(size_t)p]) cuts.push_back(p);
    cuts.push_back(0);
    std::reverse(cuts.begin(), cuts.end());
    for (size_t i = 0; i + 1 < cuts.size(); ++i) {
      const int64_t k0 = cuts[i], k1 = cuts[i + 1];
      int32_t mx = 0, mn = std::numeric_limits<int32_t>::max();
      for (int64_t k = k0; k < k1; ++k) {
        mx = std::max(mx, tree->token_kend[(size_t)k]);
        mn = std::min(mn, tree->token_kend[(size_t)k]);
      }
      s.kv_tiles.push_back(KvTile{(int32_t)k0, (int32_t)k1, mx, mn, (int32_t)k0, {0, 0, 0}});
      cost.push_back(mx - k0);
      s.bwd_tile_pairs += (int64_t)(mx - k0) * keys;
    }
    std::vector<size_t> by_cost(s.kv_tiles.size());
    std::iota(by_cost.begin(), by_cost.end(), 0);
    std::stable_sort(by_cost.begin(), by_cost.end(),
                     [&](size_t a, size_t b) { return order_key(cost[a]) > order_key(cost[b]); });
    std::vector<KvTile> sorted;
    sorted.reserve(by_cost.size());
    for (size_t i : by_cost) sorted.push_back(s.kv_tiles[i]);
    s.kv_tiles.swap(sorted);
  };
  auto cut_key_tiles = [&](int keys) {
    if (q_rows == 32) cut_key_tiles_at(keys, std::integral_constant<int, 32>{});
    else cut_key_tiles_at(keys, std::integral_constant<int, 64>{});
  };
  cut_key_tiles(bn);

  // ---- dK/dV launch items: cut the longest walks so that no block becomes the
  // critical path.  The chip holds `resident` blocks of this kernel (512 of four
  // waves, 256 of eight); a piece of a cut walk is at most 2/3 of the work one of
  // those slots gets on average, and only walks longer than that are cut.  Finer pieces balance no better and cost
  // more (every item pays its prologue, the masked steps of its diagonal and,
  // when cut, fp32 partial sums): with pieces of 1/4 of a slot's share the dK/dV
  // launch of the 16-response tree (configuration 2) was 5 % slower, coarser
  // ones (a whole share) let a single piece decide the end of the launch.
  // A launch with at least 8 rounds of items runs as resident blocks that draw
  // the items from queues and take over work from slower XCDs (see the kernel);
  // what they can take over is whole items, so where the items are long the
  // walks are cut four times finer (1/6 of a share): measured on the deep tree with its 128
  // root tiles of 17 344 steps per kv head, 3 % faster than uncut walks handed
  // out block by block, while the same queues over uncut walks are 2.5 % slower.
  auto cut_items = [&](int64_t target_items) {
    s.kv_items.clear();
    s.kv_reduce.clear();
    s.n_slots = 0;
    s.kv_item_iters = 0;
    auto iters_of = [&](const KvTile& t) {
      return (int64_t)((t.q_end - t.k0 + q_rows - 1) / q_rows) * group;
    };
    int64_t total = 0;
    for (const KvTile& t : s.kv_tiles) total += iters_of(t);
    const int64_t target = std::max<int64_t>(kw.min_piece, (total * hkv + target_items - 1) / target_items);
    std::vector<int64_t> icost;
    for (const KvTile& t : s.kv_tiles) {
      const int64_t iters = iters_of(t);
      int64_t nparts = 1;
      if (iters > target) nparts = (iters + target - 1) / target;
      if (nparts > 1) s.kv_reduce.push_back(KvReduce{t.k0, t.k1, (int32_t)s.n_slots, (int32_t)nparts});
      for (int64_t p = 0; p < nparts; ++p) {
        KvItem it{t.k0, t.k1, t.q_end, t.q_full_end, (int32_t)(iters * p / nparts),
                  (int32_t)(iters * (p + 1) / nparts), nparts > 1 ? (int32_t)(s.n_slots + p) : -1,
                  t.q_begin};
        s.kv_items.push_back(it);
        icost.push_back(it.it_end - it.it_begin);
        s.kv_item_iters += it.it_end - it.it_begin;
      }
      if (nparts > 1) s.n_slots += nparts;
    }
    std::vector<size_t> order(s.kv_items.size());
    std::iota(order.begin(), order.end(), 0);
    // same cost class: parts that cover the same slice of the walk next to each
    // other (they stream the same query rows), then DFS order
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) {
      const int64_t ka = order_key(icost[a]), kb = order_key(icost[b]);
      if (ka != kb) return ka > kb;
      return s.kv_items[a].it_begin < s.kv_items[b].it_begin;
    });
    std::vector<KvItem> sorted;
    sorted.reserve(order.size());
    for (size_t i : order) sorted.push_back(s.kv_items[i]);
    s.kv_items.swap(sorted);
  };
  // items for a launch shape that keeps `resident` blocks on the chip
  auto cut_for = [&](int64_t resident) {
    cut_items(resident * 3 / 2);
    s.kv_queues = (int64_t)s.kv_items.size() * hkv >= 8 * resident;
    // (forests of short items, under 384 steps on average, have nothing to gain from
    // finer pieces and would only pay for more partial sums)
    if (s.kv_queues && s.kv_item_iters > 384 * (int64_t)s.kv_items.size()) cut_items(resident * 6);
  };
  if (kw.queues) cut_for(kw.resident);
  else cut_items((int64_t)kw.resident * 3 / 2);
  constexpr int64_t kWideMinIters = 256;
  if (kw.queues && wide_key_tiles && s.kv_item_iters > kWideMinIters * (int64_t)s.kv_tiles.size()) {
    // Long walks (256 steps per 128-key tile and more): tiles of 256 keys for the
    // eight-wave form of the kernel, one block per CU.  Every streamed 64-row
    // chunk then meets twice the keys, which halves the copies L2 -> LDS per
    // product; the steps of a walk, and so the piece lengths in steps, stay what
    // they are with 128 keys.  Measured on MI355X (dK/dV launch): the deep tree
    // -3.8 %, the multi-turn forest (374 steps per tile) -2 %, 16 long answers
    // -1.3 %; forests of short segments (130 steps per tile and fewer) take the
    // same time either way (+-0.5 %) with more of the block's waves idle, so
    // they stay on the two-blocks-per-CU form.
    cut_key_tiles(256);
    cut_for((int64_t)kNumCUs);
  }
  return tree->schedules.emplace(key, std::move(s)).first->second;
}

Schedule& get_segment_schedule(dta_tree* tree, int bm, int bn, int hkv, int group,
                               int64_t t_begin, int64_t t_end, const KvWalk& kw) {
  const int q_rows = kw.q_rows;
  const std::array<uint64_t, 3> key = {schedule_key(bm, bn, hkv, group, kw), (uint64_t)t_begin,
                                       (uint64_t)t_end};
  auto it = tree->segment_schedules.find(key);
  if (it != tree->segment_schedules.end()) {
    it->second.last_used = ++tree->use_counter;
    return it->second;
  }
  Schedule s;   // built aside, see get_schedule
  s.last_used = ++tree->use_counter;
  s.bm = bm;
  s.bn = bn;
  s.q_rows = q_rows;
  s.kv_keys = bn;
  s.hkv = hkv;
  s.group = group;

  // The keys the rows see: the segments of the ancestors (root first), then the
  // node's own tokens before t_begin; every row sees all of them.  Adjacent
  // pieces are merged.
  const int32_t u0 = tree->token_node[(size_t)t_begin];
  std::vector<int32_t> path;
  for (int32_t a = tree->parent[u0]; a >= 0; a = tree->parent[a]) path.push_back(a);
  std::vector<KeySeg> prefix;
  auto add = [&](int64_t start, int64_t end) {
    if (start >= end) return;
    if (!prefix.empty() && prefix.back().end == start) prefix.back().end = (int32_t)end;
    else prefix.push_back(KeySeg{(int32_t)start, (int32_t)end, 1, 0});
  };
  for (auto a = path.rbegin(); a != path.rend(); ++a) {
    const int64_t off = tree->node_offset[*a];
    add(off, off + tree->seg_len[*a]);
  }
  add(tree->node_offset[u0], t_begin);
  int64_t prefix_keys = 0;
  for (const KeySeg& ks : prefix) prefix_keys += ks.end - ks.start;

  // ---- query tiles over the rows; a tile also sees the rows before it
  auto cut_rows = [&](int tokens, QueryTiles& qs) {
    for (int64_t t0 = t_begin; t0 < t_end; t0 += tokens) {
      const int64_t t1 = std::min<int64_t>(t_end, t0 + tokens);
      QTile qt;
      qt.t0 = (int32_t)t0;
      qt.t1 = (int32_t)t1;
      qt.seg_begin = (int32_t)qs.segs.size();
      for (const KeySeg& ks : prefix) qs.segs.push_back(ks);
      if (t0 > t_begin) {
        if (!prefix.empty() && qs.segs.back().end == t_begin) qs.segs.back().end = (int32_t)t0;
        else qs.segs.push_back(KeySeg{(int32_t)t_begin, (int32_t)t0, 1, 0});
      }
      qt.seg_end = (int32_t)qs.segs.size();
      qs.q_tiles.push_back(qt);
      qs.fwd_tile_pairs += (prefix_keys + (t1 - t_begin)) * tokens;
      count_chunks(qs, qt);
    }
    std::reverse(qs.q_tiles.begin(), qs.q_tiles.end());   // the last tile sees the most keys
    fill_first_intervals(qs);
  };
  cut_rows(bm, s);
  if (kw.key_steps) cut_steps(s, hkv);
  if (kw.fwd_bm != 0) cut_rows(kw.fwd_bm, s.fwd);

  // ---- key tiles: the prefix pieces (walk = all rows, no mask beyond padding),
  // then the rows themselves (causal)
  auto add_tiles = [&](int64_t start, int64_t end, bool own) {
    for (int64_t k0 = start; k0 < end; k0 += bn) {
      const int64_t k1 = std::min<int64_t>(end, k0 + bn);
      const int64_t qb = own ? k0 : t_begin;
      s.kv_tiles.push_back(KvTile{(int32_t)k0, (int32_t)k1, (int32_t)t_end, (int32_t)t_end,
                                  (int32_t)qb, {0, 0, 0}});
      s.bwd_tile_pairs += (t_end - qb) * bn;
    }
  };
  add_tiles(t_begin, t_end, true);
  for (const KeySeg& ks : prefix) add_tiles(ks.start, ks.end, false);
  for (const KvTile& t : s.kv_tiles) {
    const int64_t iters = (int64_t)((t.q_end - t.q_begin + q_rows - 1) / q_rows) * group;
    s.kv_items.push_back(KvItem{t.k0, t.k1, t.q_end, t.q_full_end, 0, (int32_t)iters, -1, t.q_begin});
    s.kv_item_iters += iters;
  }
  // keep the cache bounded: drop the least recently used schedule; its device
  // block may still be read by a launch in flight, so it is only set aside here
  // (whoever uploads into it next orders that copy behind the tree's launches)
  if (tree->segment_schedules.size() >= max_segment_schedules(tree->n_nodes)) {
    auto lru = tree->segment_schedules.begin();
    for (auto e = tree->segment_schedules.begin(); e != tree->segment_schedules.end(); ++e)
      if (e->second.last_used < lru->second.last_used) lru = e;
    if (lru->second.d_blob)
      tree->retired.push_back(dta_tree::RetiredBlock{lru->second.d_blob, lru->second.d_blob_cap, lru->second.device});
    tree->segment_schedules.erase(lru);
  }
  return tree->segment_schedules.emplace(key, std::move(s)).first->second;
}

int validate_params(const dta_attn_params_t* p) {
  if (!p) return DTA_ERR_INVALID_ARG;
  if (p->n_q_heads < 1 || p->n_kv_heads < 1) return DTA_ERR_INVALID_ARG;
  // finite and nonzero (the bf16 backward divides by it)
  if (!(p->softmax_scale == p->softmax_scale) || p->softmax_scale == 0.f ||
      p->softmax_scale - p->softmax_scale != 0.f)
    return DTA_ERR_INVALID_ARG;
  if (p->n_q_heads % p->n_kv_heads != 0) return DTA_ERR_UNSUPPORTED;
  if (p->dtype == DTA_F32) {
    if (p->head_dim != 64 && p->head_dim != 128) return DTA_ERR_UNSUPPORTED;
  } else if (p->dtype == DTA_BF16) {
    if (p->head_dim != 64 && p->head_dim != 128) return DTA_ERR_UNSUPPORTED;
  } else {
    return DTA_ERR_UNSUPPORTED;
  }
  return DTA_OK;
}

namespace {
// Which form of the bf16 kernels a call takes.  Forward and dQ have three: blocks of 8
// row tiles, blocks of 4 row tiles x 2 groups that share out the keys (split), blocks of
// 2 x 4 (small, dta_bf16_small.hip); dK/dV has two.  The row tile is what a block of
// 8 waves holds one wave for, so 2048 row tiles are one round of blocks on the 256 CUs
// for the first form, 1024 for the second, 512 for the third; what shares out the keys
// costs more per pair and gains where the other form's round would be left half empty.
// Measured on MI355X, head_dim 128, in us, small / split / 8 row tiles:
//   forward of a tree   500 row tiles 15 / 16 / 20 (32/8 heads), 15 / 21 / 32 (16/16);
//             600: 20 / 16 / 20, 22 / 20 / 30; 1000: 25 / 21 / 26, 30 / 26 / 40;
//             1200: 32 / 28 / 26, 41 / 35 / 37; 2400: 66 / 55 / 50
//   forward of a segment under 1024 keys   500: 29 / 35 / 50; 1000: 58 / 45 / 63;
//             2000: 124 / 87 / 93 (32/8), 100 / 72 / 71 (64/8), 170 / 123 / 137 (16/16);
//             2500: 168 / 133 / 117
//             Above 1024 row tiles the split form has blocks left for a second round, which takes as long as the
//             first where the rows see mostly what lies before them: 1100, 16/1 heads, 2200 rows after 512 keys
//             68 / 52 / 74, 2048: 118 / 91 / 108, 8192: 327 / 281 / 245, 16 384: 598 / 532 / 431; 1500, 32/8, 1500 rows
//             after 512 66 / 50 / 61, 2048: 117 / 98 / 93, 8192: 325 / 288 / 238; 2000, 4/4, 16 000 rows after
//             8192 753 / 544 / 603, 16 384: 1108 / 809 / 832
//   backward of a tree (4 row tiles x 2 with the large dK/dV)   1600: 86 / 90 / 92 (32/8), 66 / 70 / 70
//             (64/8); 2000: 118 / 112 / 121, 171 / 150 / 149 (16/16); 3000: 196 / 185 / 199, 298 / 251 / 272;
//             3500: 257 / 214 / 222; dQ alone at 4000: 163 / 133 / 130; head_dim 64, 2000: 80 / 77 / 70,
//             3500: 166 / 144 / 138.  Below 1800 the small form loses where its blocks are many rounds:
//             with few heads per group, 400 key tiles, a prompt with answers 135 / 126 / 123 (16/16),
//             195 / 181 / 177 (8/8), short segments 114 / 99 / 99, at 300 key tiles 101 / 130 / 131 and
//             92 / 94 / 96; and where few heads walk far, 1600, a prompt with answers 605 / 578 / 551 (2/1,
//             25 600 tokens), one segment 1270 / 1179 / 1406, while 4/1, 12 800 tokens, has 323 / 360 / 342
//   dK/dV of a tree, small / large   the walks are cut, so few key tiles fill the chip as well if their walks
//             are long: what decides is the work.  In walk steps of the small form per CU (2^21 pairs each),
//             1800 row tiles and more: 19 91 / 117 (16/1), 76 / 79 (32/8); 44 142 / 164 (16/1), 135 / 121 (32/8);
//             69 192 / 212 (16/2), 190 / 190 (64/8); 82 229 / 276 (16/1); 100 295 / 294 (16/1); 125 333 / 332
//             (32/2); 138 348 / 300 (8/2); 156 418 / 365 (16/2), 410 / 370 (64/8); 313 785 / 655 (32/4);
//             625 1555 / 1269 (16/1); 1250 3196 / 2648 (32/2); at and above 200 key tiles only the large form is taken
//   backward of a segment (whose dK/dV walks are never cut)   1600 rows, small / 8 row tiles, under
//             2048 keys 300 / 335 (32/8) and 570 / 609 (64/8); 2000 row tiles under 1024 keys, 16/16:
//             418 / 386 / 412; 2500: 623 / 599 / 588.  The large dK/dV takes what its longest walk takes, with
//             one block per CU up to 256 key tiles and two up to 512; the small one takes the sum of its walks.
//             So the small form wins while many walks are short or many slots empty, and loses where most
//             rows see a full round of key tiles.  1790 row tiles, 16/1 heads, key tiles seen by the average
//             row: 86 1226 / 2048 / 2070, 236 3227 / 2843 / 2795, 336 4638 / 4239 / 4132, 436 5993 / 4924 / 4771;
//             64/8: 217 467 / 574 / 599 (2100 row tiles), 222 411 / 387 / 393, 422 733 / 645 / 645.
//             Blocks of 4 row tiles are one round up to 1024 row tiles, of 8 up to 2048: 16/1, 450 key tiles,
//             500 row tiles 1706 / 1759 / 2472, 800: 2953 / 2270 / 2933, 1200: 3860 / 4037 / 3619; 250 key tiles,
//             2100: 3546 / 3754 / 3956, 2600: 4549 / 4170 / 4425, 3000: 5225 / 4683 / 4755, 3900: 6553 / 6215 / 5975
void choose_forms(const CallShape& c, const dta_attn_params_t* p, TileChoice* out) {
  const int64_t row_tiles = c.rows / 32 * p->n_q_heads, key_tiles = c.keys / 128 * p->n_kv_heads;
  if (!c.backward) {
    out->q_small = row_tiles <= 512;
    out->q_split = !out->q_small && (row_tiles <= 1024 || (c.segment && row_tiles <= 2048 && c.keys <= 2 * c.rows));
    out->k_small = false;
    return;
  }
  if (c.segment) {
    const double seen = (double)c.pairs / (double)c.rows * p->n_kv_heads / 128;   // key tiles seen by the average row
    const bool k_full = seen >= 280 || (key_tiles <= 256 && seen >= 218);   // the large dK/dV fills its rounds
    const bool q_full = (row_tiles >= 600 && row_tiles < 1800) || row_tiles >= 2900;   // ... and the large or split dQ
    out->q_small = (row_tiles < 1800 || (row_tiles < 4000 && key_tiles < 350)) && !(k_full && q_full);
    out->q_split = !out->q_small && (row_tiles <= 1024 || (row_tiles >= 1800 && row_tiles <= 2048));
    out->k_small = out->q_small;
    return;
  }
  const double work = (double)c.pairs * p->n_q_heads / (1 << 21);   // walk steps of the small dK/dV per CU
  out->q_small = row_tiles < 1800 && key_tiles < 380 && (row_tiles < 1000 || work <= 128);
  out->q_split = !out->q_small && row_tiles < (p->head_dim == 128 ? 3600 : 1800);
  out->k_small = out->q_small || (key_tiles < 200 && work <= 100);
}
}  // namespace

namespace {
// Which form of the fp32 kernels a call takes: products on the fp32 instruction in blocks that
// share out the keys (small, dta_f32_kernels.hip), or on the bf16 one with operands in three
// parts (planes, dta_f32_planes.hip), whose blocks of 8 row tiles of 16 and 128-key tiles need a
// launch that fills the chip.  Measured on MI355X, in us, small / planes:
//   trees (a prompt with 8 answers), forward + backward, heads of 128   1000 row tiles: 39 + 121 / 50 + 125 (16/16),
//             24 + 81 / 29 + 76 (32/8), 18 + 53 / 20 + 64 (64/8), 63 + 187 / 74 + 180 (8/2); 1200: 50 + 142 / 56 + 134,
//             36 + 92 / 32 + 99, 25 + 73 / 23 + 69, 80 + 242 / 85 + 206, 36 + 96 / 32 + 108 (32/1); 1600: 77 + 224 / 65 + 171,
//             50 + 137 / 35 + 123, 38 + 106 / 27 + 95, 146 + 352 / 107 + 271; 2000: 111 + 323 / 81 + 227, 65 + 204 / 45 + 154,
//             45 + 143 / 30 + 108; of 64   1000: 29 + 82 / 34 + 78, 22 + 56 / 19 + 50, 20 + 42 / 13 + 43, 41 + 114 / 49 + 114;
//             1200: 37 + 100 / 38 + 86, 29 + 64 / 21 + 65, 25 + 50 / 15 + 47, 56 + 141 / 57 + 130
//   forward of a tree with few branches, whose longest walk is twice the average one: one segment, 1200 row tiles 52 / 74
//             (16/16 heads of 64), 91 / 142 (8/2), 68 / 98 (12/4), 96 / 112 (16/16 of 128), 185 / 216 (8/2); 1600: 82 / 98, 149 / 188,
//             52 / 52 (32/8), 135 / 148, 257 / 285 (8/2 of 128), 47 / 46 (64/8); 2000: 119 / 121, 222 / 234, 233 / 183
//   forward of a segment, heads of 128   after 512 keys, 1200: 134 / 157 (16/16, 1200 rows), 112 / 107 (32/8, 600 rows);
//             1800: 221 / 211, 155 / 134, 338 / 367 (8/2, 3600 rows); after 2048, 1000: 197 / 233 (32/8), 1200: 337 / 241,
//             388 / 396 (8/2), 351 / 291 (16/16); of 64   after 512, 1200: 91 / 104, 72 / 70; after 2048, 1200: 178 / 159 (32/8),
//             198 / 192 (16/16), 207 / 214 (12/4, 1600 rows), 233 / 260 (8/2, 2400 rows); 1450: 269 / 288 (8/2, 2900 rows)
//   backward of a segment, whose dK/dV walks are not cut: with one block per CU up to 256 key tiles of 128 the planes
//             form takes what its longest walk takes however many tiles there are, the small one the sum of its walks.  What
//             decides is the number of key tiles that the average row sees, at any number of rows: 60 to
//             70 tiles 1276 / 1762 (8/2 heads of 64, 2060 row tiles), 2709 / 3870 (32/1), 591 / 730 (32/8 of 128); 79 to 94
//             607 / 643, 1012 / 1034 (32/8, 3000), 5072 / 5384 (8/2 of 64, 6000), 4716 / 4535 (8/2 of 128, 4000 after 2048);
//             102 to 114 -2 to +21 % for small; 126 1276 / 1005 (12/4 of 128, 3000); 159 2673 / 1656 (64/8 of 128, 4000), 1534 / 1021 (of 64)
// One form for both directions: what the backward recomputes from an LSE of the other form's scores, whose roundings are
// others, is further from 64 bits: dV of queries 3 / 8 / 30 times N(0,1), one segment of 1300 tokens, 16/16 heads of 64, 5.3 / 8.6 / 22e-7
// small, 4.1 / 7.2 / 21e-7 planes, 7.2 / 21 / 80e-7 small forward and planes backward (N(0,1): 3.1, 2.5, 2.6e-7).
// (The planes' softmax multiplies by |softmax_scale| log2 e, which has to be a normal number: scales beyond 2^100 or
// below 2^-100 stay on the fp32 instruction.)
bool f32_planes(const CallShape& c, const dta_attn_params_t* p) {
  const float scale = std::fabs(p->softmax_scale);
  if (!(scale >= 0x1p-100f && scale <= 0x1p100f)) return false;
  const int64_t row_tiles = c.rows / 16 * p->n_q_heads;
  if (row_tiles < 1200) return false;
  if (!c.segment) {
    if (row_tiles >= 2048 || c.path == 0) return true;
    // One round of blocks: the planes form takes what its longest walk takes (1.85 us per 32 keys, 2.9 with heads of
    // 128), the small one the sum of its walks.  A prompt with answers has walks of like length, a chain does not.  (The
    // backward gains more: a tenth more of the forward's time, a twentieth with heads of 128, is allowed for.)
    if (4 * c.path * c.rows < 7 * c.pairs) return p->head_dim == 64 || row_tiles >= 1250;
    const double path = (double)c.path, pairs = (double)c.pairs * p->n_q_heads / 16e6;
    return p->head_dim == 64 ? 5 + 0.058 * path < 1.1 * (12 + 54 * pairs) : 6 + 0.09 * path < 1.05 * (10 + 100 * pairs);
  }
  // (From 3500 row tiles on the small form's forward would take up to 1.4 times what it took on the fp32 instruction in
  // blocks that fill the chip, below no longer.)
  if (row_tiles >= 3500) return true;
  // (a row sees the keys before the segment and half of its own rows' on average)
  const int64_t seen = (2 * c.keys - c.rows) * p->n_kv_heads / 256;
  if (seen < 95) return false;
  if (row_tiles >= 2048) return true;
  // (heads of 64: the longest walk against their sum, as above)
  const bool one_round = p->head_dim == 128 || c.keys >= 2 * c.rows ||
                         5 + 0.055 * c.keys < 12 + 51e-6 * row_tiles * (c.keys - 0.5 * c.rows);
  return one_round && 2 * c.keys >= 3 * c.rows;
}
}  // namespace

int choose_tiles(const dta_attn_params_t* p, TileChoice* out, const CallShape& call) {
  int st = validate_params(p);
  if (st != DTA_OK) return st;
  int G = p->n_q_heads / p->n_kv_heads;
  if (p->dtype == DTA_F32) {
    // Eight waves of 16 rows: R row tiles (hb q heads x 16-row blocks) x `split`
    // groups that share out the streamed keys where the launch does not fill the chip.  Where even blocks of four
    // waves are no more than the CUs, a block is four: one wave per SIMD.  Measured on MI355X, backward, four / eight waves,
    // in us: 256 row tiles of 16, head_dim 128, 32/8 heads 35 / 53, 16/16 34 / 51; 512: 43 / 56,
    // 56 / 63; head_dim 64, 8/2 heads, 256: 32 / 37.  Above, a CU gets two such blocks one after
    // the other: 16/16 heads of 64, 256 row and 256 key blocks in one launch, 29 / 23.
    TileChoice t{};
    t.planes = f32_planes(call, p);
    t.q_small = t.k_small = !t.planes;
    const int split = t.planes ? 1 : p->head_dim == 64 ? 4 : 2;
    const int64_t row_tiles = call.rows / 16 * p->n_q_heads;
    const int64_t row_blocks = row_tiles * split / 4, key_blocks = call.keys / 16 * p->n_kv_heads * split / 4;
    t.tiny = t.q_small && row_blocks <= kNumCUs && (p->head_dim == 128 || row_blocks + key_blocks <= kNumCUs * 4 / 3);
    const int R = (t.tiny ? 4 : 8) / split;
    t.hb = 1;
    while (t.hb < R && G % (2 * t.hb) == 0) t.hb *= 2;
    t.hblocks = G / t.hb;
    t.bm = 16 * (R / t.hb);
    t.bn = t.planes ? 128 : 16 * R;
    t.walk = KvWalk{32, 4 * split, kNumCUs};   // an iteration takes a wave several microseconds, so cut walks may be short
    *out = t;
  } else {
    // eight waves per block: hb q heads of the group x (R/hb) 32-row query blocks
    TileChoice f{}, b{};
    auto choose = [&](bool backward, TileChoice* t) {
      CallShape c = call;
      c.backward = backward;
      choose_forms(c, p, t);
      const int R = t->q_small ? 2 : t->q_split ? 4 : 8;
      t->hb = 1;
      while (t->hb < R && G % (2 * t->hb) == 0) t->hb *= 2;
      t->hblocks = G / t->hb;
      return 32 * (R / t->hb);
    };
    const int fwd_bm = choose(false, &f);
    b.bm = choose(true, &b);
    b.bn = b.k_small ? 64 : 128;
    b.walk = b.k_small ? KvWalk{32, 32, kNumCUs} : KvWalk{64, 32, 2 * kNumCUs};
    b.walk.queues = !b.k_small;
    // (a launch small enough for the forward's steps is small for dQ too, and then the tiles are the same)
    b.walk.key_steps = b.q_small;
    b.walk.fwd_bm = fwd_bm == b.bm ? 0 : fwd_bm;
    f.bm = b.bm;
    f.bn = b.bn;
    f.walk = b.walk;
    *out = call.backward ? b : f;
  }
  return DTA_OK;
}

}  // namespace dta

extern "C" {

int dta_tree_build(const int32_t* parent, const int32_t* seg_len, int32_t n_nodes,
                   uint32_t flags, dta_tree_t** out) {
  if (out) *out = nullptr;
  if (!parent || !seg_len || !out || n_nodes < 1 || flags != 0) return DTA_ERR_INVALID_ARG;
  dta_tree* t = new (std::nothrow) dta_tree();
  if (!t) return DTA_ERR_ALLOC;
  int st;
  try {
    st = build_impl(parent, seg_len, n_nodes, t);
  } catch (const std::bad_alloc&) {
    st = DTA_ERR_ALLOC;
  }
  if (st != DTA_OK) {
    delete t;
    return st;
  }
  *out = t;
  return DTA_OK;
}

int dta_tree_info(const dta_tree_t* tree, dta_tree_info_t* out) {
  if (!tree || !out) return DTA_ERR_INVALID_ARG;
  *out = tree->info;
  return DTA_OK;
}

int dta_tree_layout(const dta_tree_t* tree, dta_tree_layout_t* out) {
  if (!tree || !out) return DTA_ERR_INVALID_ARG;
  out->dfs_order = tree->dfs_order.data();
  out->node_offset = tree->node_offset.data();
  out->node_start_depth = tree->node_start_depth.data();
  out->subtree_tokens = tree->subtree_tokens.data();
  out->anc_ptr = tree->anc_ptr.data();
  out->anc_seg_off = tree->anc_seg_off.data();
  out->anc_seg_len = tree->anc_seg_len.data();
  out->token_kend = tree->token_kend.data();
  return DTA_OK;
}

static size_t schedule_bytes(const dta::Schedule& s) {
  return (s.q_tiles.size() + s.fwd.q_tiles.size()) * sizeof(dta::QTile) +
         (s.segs.size() + s.fwd.segs.size()) * sizeof(dta::KeySeg) + s.step_tiles.size() * sizeof(dta::StepTile) + s.steps.size() * sizeof(dta::KeyStep) +
         s.kv_items.size() * sizeof(dta::KvItem) + s.kv_reduce.size() * sizeof(dta::KvReduce);
}

int dta_tree_schedule_info(dta_tree_t* tree, const dta_attn_params_t* params,
                           dta_schedule_info_t* out) {
  if (!tree || !out) return DTA_ERR_INVALID_ARG;
  dta::TileChoice tc;
  int st = dta::choose_tiles(params, &tc, dta::whole_tree(tree, true));
  if (st != DTA_OK) return st;
  try {
    std::lock_guard<std::mutex> lock(tree->mu);
    const int group = params->n_q_heads / params->n_kv_heads;
    const dta::Schedule& b = dta::get_schedule(tree, tc.bm, tc.bn, params->n_kv_heads, group, tc.walk);
    const dta::QueryTiles& f = b.forward_tiles();
    out->fwd_q_tile_tokens = tc.walk.fwd_bm != 0 ? tc.walk.fwd_bm : tc.bm;
    out->fwd_work_items = (int64_t)f.q_tiles.size();
    out->fwd_tile_pairs = f.fwd_tile_pairs;
    out->bwd_kv_tile_tokens = b.kv_keys;
    out->bwd_work_items = (int64_t)b.kv_items.size();
    out->bwd_tile_pairs = b.bwd_tile_pairs;
    out->metadata_bytes = (int64_t)(tree->token_kend.size() * sizeof(int32_t) + schedule_bytes(b));
  } catch (const std::bad_alloc&) {
    return DTA_ERR_ALLOC;
  }
  return DTA_OK;
}

const char* dta_status_string(int status) {
  switch (status) {
    case DTA_OK: return "DTA_OK";
    case DTA_ERR_INVALID_ARG: return "DTA_ERR_INVALID_ARG";
    case DTA_ERR_BAD_TREE: return "DTA_ERR_BAD_TREE";
    case DTA_ERR_UNSUPPORTED: return "DTA_ERR_UNSUPPORTED";
    case DTA_ERR_ALLOC: return "DTA_ERR_ALLOC";
    case DTA_ERR_HIP: return "DTA_ERR_HIP";
    case DTA_ERR_WORKSPACE: return "DTA_ERR_WORKSPACE";
    default: return "DTA_ERR_UNKNOWN";
  }
}

}  // extern "C"
