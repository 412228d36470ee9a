// Test harness: what the host library derives from a graph (compact template
// records, bursts of ready nodes), without a device (built with g++ beside the launch
// stand-ins of gts_host_only.cpp).
#include "../paper_2607_11262_amd/csrc/gts_host.cpp"

// After the checks alone (a size query, a validation): record words built.
extern "C" int64_t gts_test_words_after_check(const gts_graph_host* h) {
  Derived d;
  if (check_graph(h, &d)) return -1;
  int64_t n = (int64_t)d.crec.size();
  for (const KTemplate& t : d.ktmpl) n += t.slots;
  return n;
}

// Nodes that one event readies on one SM, at least.
extern "C" int64_t gts_test_burst(const gts_graph_host* h) {
  Derived d;
  if (check_graph(h, &d)) return -1;
  return h->n_nodes ? (int64_t)ready_burst(h, d) : 0;
}

// Whether a burst surely outgrows the team kernel's lists.
extern "C" int gts_test_team_overflows(uint32_t burst, uint32_t qp, uint32_t max_nsm) {
  return team_overflows(burst, qp, max_nsm);
}

// Per kernel {template nodes, first record, state slots}, then the record
// words into rec (at most cap); returns their number.
extern "C" int64_t gts_test_compact(const gts_graph_host* h, uint32_t* kernels, uint32_t* rec, uint64_t cap) {
  Derived d;
  if (check_graph(h, &d)) return -1;
  compact_templates(h, &d);
  for (uint32_t k = 0; k < h->n_kernels; ++k) {
    kernels[3 * k] = d.ktmpl[k].t_n;
    kernels[3 * k + 1] = d.ktmpl[k].t_base;
    kernels[3 * k + 2] = d.ktmpl[k].slots;
  }
  for (uint64_t i = 0; i < d.crec.size() && i < cap; ++i) rec[i] = d.crec[i];
  return (int64_t)d.crec.size();
}
