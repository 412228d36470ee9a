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

// Nodes, and loads and stores in one cycle, that one event readies on one SM,
// at least.
extern "C" int gts_test_burst(const gts_graph_host* h, uint32_t* out) {
  Derived d;
  if (const int rc = check_graph(h, &d)) return rc;
  const Burst b = ready_burst(h, d);
  out[0] = b.nodes;
  out[1] = b.mem;
  return 0;
}

// Whether bursts surely outgrow the team kernel's lists or rings.
extern "C" int gts_test_team_overflows(uint32_t nodes, uint32_t mem, uint32_t qp, uint32_t ring, uint32_t max_nsm) {
  return team_overflows(Burst{nodes, mem}, qp, ring, max_nsm);
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
