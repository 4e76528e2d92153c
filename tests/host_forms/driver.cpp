// Prints which form of the kernels a call takes, one line per line of stdin:
//   Hq Hkv head_dim dtype backward segment rows keys pairs path
// Built and read by tests/test_host_forms.py, together with dta_tree.cpp.
#include <iostream>
#include <set>
#include <vector>

#include "dta_internal.h"

extern "C" void dta_tree_destroy(dta_tree_t* tree) { delete tree; }   // (no device copies here)

// Schedules that differ in any part have different keys.
static bool keys_tell_schedules_apart() {
  const dta::KvWalk base;
  std::vector<dta::KvWalk> walks(7, base);
  walks[1].q_rows = 32;
  walks[2].min_piece = 60;
  walks[3].resident = 256;
  walks[4].key_steps = true;
  walks[5].fwd_bm = 256;
  walks[6].queues = true;
  std::set<uint64_t> keys;
  for (const dta::KvWalk& w : walks) keys.insert(dta::schedule_key(128, 128, 8, 4, w));
  keys.insert(dta::schedule_key(256, 128, 8, 4, base));
  keys.insert(dta::schedule_key(128, 256, 8, 4, base));
  keys.insert(dta::schedule_key(128, 128, 4, 4, base));
  keys.insert(dta::schedule_key(128, 128, 8, 8, base));
  return keys.size() == walks.size() + 4;
}

int main() {
  if (!keys_tell_schedules_apart()) return 2;
  dta_attn_params_t p{};
  p.softmax_scale = 0.125f;
  dta::CallShape c;
  while (std::cin >> p.n_q_heads >> p.n_kv_heads >> p.head_dim >> p.dtype >> c.backward >> c.segment >> c.rows >>
         c.keys >> c.pairs >> c.path) {
    dta::TileChoice t{};
    if (dta::choose_tiles(&p, &t, c) != DTA_OK) return 1;
    const char* q = t.tiny ? "tiny" : t.q_small ? "small" : t.q_split ? "split" : "large";
    std::cout << q << ' ' << (t.k_small ? "small" : "large") << ' ' << t.bm << ' ' << t.bn << ' ' << t.walk.fwd_bm
              << '\n';
  }
  return 0;
}
