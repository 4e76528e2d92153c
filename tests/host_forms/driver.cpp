// Prints which form of the kernels a call takes, one line per line of stdin:
//   Hq Hkv head_dim dtype backward segment rows keys pairs path
// Built and read by tests/test_host_forms.py, together with dta_tree.cpp.
#include <iostream>

#include "dta_internal.h"

extern "C" void dta_tree_destroy(dta_tree_t* tree) { delete tree; }   // (no device copies here)

int main() {
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
