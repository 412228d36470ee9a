// gts_team.hip — team simulation kernel for gfx950 (MI355X): one workgroup
// of one to four wavefronts simulates one (graph, hardware record) pair, one
// thread per simulated SM.
//
// It advances a simulation through the time windows of the windowed kernel
// (gts_window.hip states why that order equals one event at a time), but
// spreads each window over the workgroup:
//
//   local phase: a thread issues its own SM's ready nodes, smallest (cycle,
//       node id) first, straight from that SM's list; the SMs of one wave
//       advance side by side and the waves do not wait for each other (inside
//       a window SMs share nothing);
//   memory phase: every thread puts its SM's due arrivals into one batch;
//       each arrival finds its place in the batch's (cycle, id) order by
//       counting the smaller keys, one thread per arrival; every wave then
//       walks the ordered batch through the L2 and DRAM servers (a max-plus
//       scan in doubles, which hold these whole numbers exactly) and
//       completes its own SMs' arrivals, so that no wave waits for another's
//       results;
//   retirement and dispatch: the first wave, and only in windows that retire
//       a CTA.
//
// What bounds it: a simulation is a chain of windows, and a window a chain of
// dependent LDS and L1 / L2 accesses and of the instructions between them; a
// batch of few simulations leaves the chip idle, so what counts is the length
// of that chain and not the work per CU.  With one wave per simulation the
// chain holds the packing of the taken nodes, two or three SMs per lane and a
// 256-key sorting network; here each of them is spread over the waves or
// gone.  Windowed kernel / this one: one 784-node GEMM 266 / 141 us, one
// 82,944-node attention 16.6 / 4.4 ms, 64 decoder layers of 2.56 M nodes
// 641 / 279 ms.  The windowed kernel takes fewer wave instructions per node,
// and stays the faster one for large batches that overlap.  The compiler
// spills 306-347 scalar registers to lanes of the 147-153 vector ones (none to
// memory), and reads them back lane by lane inside those chains.
//
// Memory: the ready list, memory-arrival ring, servers and counts of an SM
// lie in LDS, strided by the workgroup's threads; what does not fit goes to
// the windowed kernel's scratch regions.  A kernel with compact template
// records (gts_dev.h) runs from LDS alone when its records and the state
// slots of as many CTAs as can be resident fit there: its entries name {CTA,
// node, the CTA's place}, a step is straight-line code whose LDS accesses
// overlap, and finished nodes are logged per wave and written (and digested)
// 64 at a time.  Other kernels use the windowed kernel's records and state in
// global memory, where loads and stores return in order, so that every load
// also waits for the stores before it.  A simulation that overflows a list is
// handed back.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/gts.h"
#include "gts_common.h"
#include "gts_dev.h"
#include "gts_wave.h"

namespace gts {

namespace {

constexpr uint32_t kBadOverflow = 1u, kBadQueue = 2u;
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr int kWaveShr1 = 0x138;

extern __shared__ uint32_t team_lds_words[];
// A pointer into LDS (address space 3): 32-bit address arithmetic.
template <typename T>
using lmem = __attribute__((address_space(3))) T;
// four words of LDS at a 16-B boundary
using word4 = uint32_t __attribute__((ext_vector_type(4)));

// Waits for v here: a value that comes from global memory on one path and from
// LDS on the other would otherwise make both wait for all global accesses
// where the paths meet.
__device__ __forceinline__ uint32_t arrived(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ uint64_t arrived(uint64_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ uint4 arrived(uint4 v) { return make_uint4(arrived(v.x), arrived(v.y), arrived(v.z), arrived(v.w)); }

// f(x) = max(x, a) + o on whole numbers below 2^53, or (MaxPlus32) below 2^30
struct MaxPlus32 {
  int32_t a, o;
};
constexpr int32_t kNeg32 = -(1 << 30);
__device__ __forceinline__ MaxPlus32 after(MaxPlus32 f, MaxPlus32 g) {  // g after f
  const int32_t ga = g.a - f.o;
  return MaxPlus32{f.a > ga ? f.a : ga, f.o + g.o};
}
template <int ctrl, int row_mask = 0xF>
__device__ __forceinline__ MaxPlus32 dpp_mp(MaxPlus32 c) {  // lanes without a source get the identity
  uint32_t a = dpp<ctrl, row_mask>((uint32_t)kNeg32, (uint32_t)c.a), o = dpp<ctrl, row_mask>(0u, (uint32_t)c.o);
  // kept apart from their use: folded into the subtraction of after() (a
  // reversed subtract with a DPP operand), lanes without a source came out as
  // 0 - o instead of a - 0
  asm volatile("" : "+v"(a), "+v"(o));
  return MaxPlus32{(int32_t)a, (int32_t)o};
}
struct MaxPlus {
  double a, o;
};
constexpr double kNegInf = -__builtin_inf();
__device__ __forceinline__ MaxPlus after(MaxPlus f, MaxPlus g) {  // g after f
  return MaxPlus{__builtin_fmax(f.a, g.a - f.o), f.o + g.o};
}
template <int ctrl, int row_mask = 0xF>
__device__ __forceinline__ double dpp_f64(double old, double v) {
  const uint64_t ob = __builtin_bit_cast(uint64_t, old), vb = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = dpp<ctrl, row_mask>((uint32_t)ob, (uint32_t)vb);
  const uint32_t hi = dpp<ctrl, row_mask>((uint32_t)(ob >> 32), (uint32_t)(vb >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int ctrl, int row_mask = 0xF>
__device__ __forceinline__ MaxPlus dpp_mp(MaxPlus c) {  // lanes without a source get the identity
  return MaxPlus{dpp_f64<ctrl, row_mask>(kNegInf, c.a), dpp_f64<ctrl, row_mask>(0.0, c.o)};
}
__device__ __forceinline__ double lane_f64(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, ((uint64_t)lane_u32((uint32_t)(b >> 32), l) << 32) | lane_u32((uint32_t)b, l));
}
template <typename MP>
__device__ __forceinline__ MP wave_incl_mp(MP c) {
  c = after(dpp_mp<kRowShr1>(c), c);
  c = after(dpp_mp<kRowShr2>(c), c);
  c = after(dpp_mp<kRowShr4>(c), c);
  c = after(dpp_mp<kRowShr8>(c), c);
  c = after(dpp_mp<kRowBcast15, 0xA>(c), c);
  c = after(dpp_mp<kRowBcast31, 0xC>(c), c);
  return c;
}
// Cycles past the last one stay at 2^32 - 1, which is never due.  Were they to
// wrap, they could come up again in the same window, where the counts beside
// them in the state slots are no longer whole: each level of joins could be
// ready twice as often as the one before.
__device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }

// Barrier that orders LDS only.  Global memory is private to a thread's SM,
// atomic, handed over at a full barrier, or written by a thread that waits for
// its write before it comes here (push, ret_push).
template <uint32_t NW>
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <uint32_t NW>
struct TSim {
  static constexpr uint32_t TH = 64u * NW;
  Image G;
  const uint32_t* hw;
  uint32_t b, x, lane, wave, nsm, nsub, smem_w, sync_w, QF, RL, qcap, retl, rec_cap, own_cap, st_cap;
  bool nocont, ofin, mem_only, sink_ret, want_digest;
  // LDS: op table (then the template class x slot entries), servers, ready
  // lists, rings, pending retirements, compact records, state slots, CTA
  // places (class of each, then the free ones), the wave's log
  lmem<uint4>* optab;
  lmem<uint32_t>*srv, *q_cnt, *q_min, *res, *own, *log;
  lmem<uint4>*rg, *rec_l;  // rg: {entry, cycle, op, 0}
  lmem<uint64_t>*q, *ret_l;
  lmem<uint32_t>* st_l;
  // scratch
  uint64_t* state;
  CtaState* cst;
  uint32_t* mq_g;
  gmem<uint64_t>* q_g;
  gmem<uint64_t>* ret_g;
  uint32_t* out_cycles;
  // the running kernel: its template (as in the windowed kernel), the
  // reciprocal of its nodes per CTA; hot: it runs from LDS (t_places CTA
  // places of t_slots state slots each), its entries CTA << (nb + pb) | node
  // << pb | place.  rk_base, rk_shift, rk32: an entry's place in node order as
  // (entry - rk_base) >> rk_shift, whether that fits 22 bits
  uint32_t run_k, staged_k, t_n, t_rcp, t_node0, t_kc0, t_nc, t_base, t_ops, t_nslot;
  bool hot, rk32;
  uint32_t t_slots, t_places, nb, pb, rk_base, rk_shift;
  uint32_t t_cyc;  // cycle its slots count from: released in-edges << kSlotBits | latest release - t_cyc
  static constexpr uint32_t kSlotBits = 27, kSlotMask = (1u << kSlotBits) - 1u;
  double l2_av, dram_av;
  // this SM's ring: first entry and count in LDS, then in scratch
  uint32_t rh, rc, gh, gc;
  uint32_t red_next;  // LDS word: earliest cycle pushed for the next window
  uint32_t log_n, log_h;  // this wave's log: entries and the first one (uniform)
  uint64_t digest;
  uint32_t makespan, nfin, bad, n_issued;

  __device__ __forceinline__ static lmem<uint32_t>* lds() { return (lmem<uint32_t>*)team_lds_words; }
  __device__ __forceinline__ static lmem<uint64_t>* lds64(uint32_t w) { return (lmem<uint64_t>*)(lds() + w); }
  __device__ __forceinline__ static uint32_t lds_add(lmem<uint32_t>* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ static void lds_min(lmem<uint32_t>* p, uint32_t v) {
    __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // four words of LDS in one access
  __device__ __forceinline__ static uint4 get4(const lmem<uint4>* p) {
    const word4 v = *(const lmem<word4>*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  __device__ __forceinline__ static void set4(lmem<uint4>* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    *(lmem<word4>*)p = word4{a, b, c, d};
  }
  // Of the workgroup's NW waves (enough for the batch's largest machine), the
  // nw that this record's SMs need stay.  SM s runs on thread (s mod nw) * 64
  // + s / nw: consecutive SMs on different waves, so the waves carry the same
  // number of them.
  uint32_t nw;
  __device__ __forceinline__ uint32_t sm_of(uint32_t t) const { return (t & 63u) * nw + (t >> 6); }
  __device__ __forceinline__ uint32_t thread_of(uint32_t s) const { return (s % nw) * 64u + s / nw; }

  // ---- ready list of thread t's SM: entries cycle << 32 | node (or as above),
  // [0, QF) in LDS and the rest in scratch, in no order; q_min a lower bound
  // of the cycles outside the local phase
  __device__ __forceinline__ uint64_t q_get(uint32_t t, uint32_t i) const {
    return i < QF ? q[i * TH + t] : arrived((uint64_t)q_g[(i - QF) * TH + t]);
  }
  __device__ __forceinline__ void q_set(uint32_t t, uint32_t i, uint64_t k) {
    if (i < QF)
      q[i * TH + t] = k;
    else
      q_g[(i - QF) * TH + t] = k;
  }
  // outside the local phase any thread may push to any SM's list; its owner
  // reads it behind a barrier that orders LDS only, so an entry that goes to
  // scratch is waited for here
  __device__ __forceinline__ void push(uint32_t t, uint32_t cyc, uint32_t low) {
    const uint32_t i = lds_add(&q_cnt[t], 1u);
    if (i < qcap) {
      q_set(t, i, ((uint64_t)cyc << 32) | low);
      if (i >= QF) mem_wait();
      lds_min(&q_min[t], cyc);
    } else {
      bad |= kBadQueue;
    }
  }

  // ---- pending retirements (cycle << 32 | thread << 24 | the CTA's place), the
  // first retl in LDS
  __device__ __forceinline__ uint64_t ret_get(uint32_t i) const {
    return i < retl ? ret_l[i] : arrived((uint64_t)ret_g[i - retl]);
  }
  __device__ __forceinline__ void ret_set(uint32_t i, uint64_t k) {
    if (i < retl)
      ret_l[i] = k;
    else
      ret_g[i - retl] = k;
  }
  __device__ __forceinline__ void ret_push(uint32_t cyc, uint32_t place) {
    const uint32_t i = lds_add(lds() + kTeamRetCnt, 1u);
    if (i < kRetireCap) {
      ret_set(i, ((uint64_t)cyc << 32) | (x << 24) | place);
      if (i >= retl) mem_wait();  // the first wave reads it after a barrier that orders LDS only
      lds_min(lds() + red_next + 1u, cyc);
    } else {
      bad |= kBadQueue;
    }
  }

  __device__ __forceinline__ void record(uint32_t v, uint32_t s, uint32_t f) {
    const uint64_t w = ((uint64_t)f << 32) | s;
    if (out_cycles) ((gmem<uint64_t>*)out_cycles)[(uint64_t)b * G.n_nodes + v] = w;
    if (want_digest) digest += mix64((((uint64_t)s << 32) | f) ^ mix64((uint64_t)v + 1));
    makespan = f > makespan ? f : makespan;
    ++nfin;
  }
  // ---- the wave's log of finished nodes {node, start, finish}: every lane
  // calls with whether it has one; 64 of them are recorded at a time, one per
  // lane (the lanes of a step or a completion round are few)
  __device__ __forceinline__ void log_node(bool has, uint32_t v, uint32_t s, uint32_t f) {
    const uint64_t m = __ballot(has);
    if (has) {
      lmem<uint32_t>* const e = log + ((log_h + log_n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))) & (kTeamLog - 1u)) * 3u;
      e[0] = v;
      e[1] = s;
      e[2] = f;
    }
    log_n += (uint32_t)__popcll(m);
    if (log_n >= 64u) log_flush(64u);
  }
  __device__ __forceinline__ void log_flush(uint32_t k) {
    wsync();
    if (lane < k) {
      const lmem<uint32_t>* const e = log + ((log_h + lane) & (kTeamLog - 1u)) * 3u;
      record(e[0], e[1], e[2]);
    }
    log_h += k;
    log_n -= k;
    wsync();
  }

  // ---- node records: expanded, or the running kernel's template; the op
  // field becomes an index into the LDS op table
  __device__ __forceinline__ Rec rec_of(uint32_t v) const {
    if (t_n == 0) return load_rec(G.nodes, v);
    const uint32_t rel = v >= t_node0 ? v - t_node0 : 0u;  // idle lanes pass node 0
    uint32_t ci = __umulhi(rel, t_rcp);                     // the quotient or one below it
    uint32_t loc = rel - ci * t_n;
    if (loc >= t_n) {
      ++ci;
      loc -= t_n;
    }
    if (ci >= t_nc || loc >= t_n) ci = loc = 0u;
    Rec r = load_rec(G.tnodes, t_base + loc);
    const uint32_t cq = G.cclass[t_kc0 + ci];
    const uint32_t base = t_node0 + ci * t_n;
    r.a.x = (r.a.x & 0xFFFF0000u) | (G.n_ops + t_ops + cq * t_nslot + (r.a.x & 0xFFFFu));
    r.a.y = t_kc0 + ci;
    r.a.w += base;
    r.b.x += base;
    r.b.y += base;
    return r;
  }
  __device__ __forceinline__ void load_template(uint32_t k) {
    const KernelDev kd = G.kernels[k];
    run_k = k;
    t_n = uni(kd.t_n);
    t_rcp = t_n > 1u ? uni((uint32_t)(0x100000000ull / t_n)) : 0xFFFFFFFFu;
    t_node0 = uni(kd.node_begin);
    t_kc0 = uni(kd.cta_begin);
    t_nc = uni(kd.cta_end) - t_kc0;
    t_base = uni(kd.t_base);
    t_ops = uni(kd.t_ops & 0xFFFFu);
    t_nslot = uni(kd.t_ops >> 16);
    sink_ret = uni(kd.sink_ret) != 0;
    t_slots = uni(kd.t_slots);
    // it runs from LDS if its records, and places for as many CTAs as can be
    // resident, fit there and its entries fit 32 bits
    const uint64_t slots = uni64(kernel_slots(kd, hw)), most = slots * nsm;  // slots <= 2^32, nsm <= 256
    t_places = most < t_nc ? (uint32_t)most : t_nc;
    nb = t_n > 1u ? 32u - (uint32_t)__builtin_clz(t_n - 1u) : 0u;
    pb = t_places > 1u ? 32u - (uint32_t)__builtin_clz(t_places - 1u) : 0u;
    const uint32_t cb = t_nc > 1u ? 32u - (uint32_t)__builtin_clz(t_nc - 1u) : 0u;
    hot = t_slots != 0u && t_n <= rec_cap && t_places <= own_cap && t_places * t_slots <= st_cap && !ofin &&
          nsub <= 4u && QF >= 8u && cb + nb + pb <= 32u;
    rk_base = hot ? 0u : t_node0;
    rk_shift = hot ? pb : 0u;
    const uint32_t nodes = t_n ? t_nc * t_n : G.n_nodes - t_node0;
    rk32 = hot ? cb + nb <= 22u : nodes <= 1u << 22;
  }
  // Setup of a kernel that runs from LDS, every thread: its records and
  // zeroed state slots.
  __device__ __forceinline__ void stage_template() {
    if (hot) {
      if (x == 0) lds()[kTeamCount] += 1u;
      const gmem<const uint32_t>* src = (const gmem<const uint32_t>*)G.crec + (uint64_t)t_base * kCompactWords;
      for (uint32_t i = x; i < t_n * (kCompactWords / 4u); i += 64u * nw) {
        const uint4 w = ld4(src + 4u * i);
        set4(rec_l + i, w.x, w.y, w.z, w.w);
      }
      for (uint32_t i = x; i < t_places * t_slots; i += 64u * nw) st_l[i] = 0u;
      t_cyc = uni((uint32_t)lds()[kTeamCtl + 6u]);  // its first CTAs were dispatched then
    }
    staged_k = run_k;
    lds_barrier<NW>();
  }

  // ---- local phase: the earliest due entry is in `best`, the others in this
  // SM's list as [due | later]: n entries, the first nd of them due, mn the
  // earliest of the rest
  uint32_t n, nd, mn;
  uint64_t best;
  __device__ __forceinline__ void push_own(uint32_t cyc, uint32_t low, uint32_t H) {
    if (n >= qcap) {
      bad |= kBadQueue;
      return;
    }
    uint64_t k = ((uint64_t)cyc << 32) | low;
    if (cyc < H) {
      if (k < best) {
        const uint64_t o = best;
        best = k;
        k = o;
      }
      if (k == ~0ull) return;
      if (n < QF) {
        if (nd != n) q[n * TH + x] = q[nd * TH + x];
        q[nd * TH + x] = k;
      } else {
        if (nd != n) q_set(x, n, q_get(x, nd));
        q_set(x, nd, k);
      }
      ++nd;
    } else {
      q_set(x, n, k);
      mn = cyc < mn ? cyc : mn;
    }
    ++n;
  }
  // Entries [i0, end) of the list eight (scratch) or four (LDS) at a time, all
  // of them read before the first is used: f(entry, key), past the end the last
  // one again.  The two parts are read in loops of their own: a read that takes
  // either waits for its value before the next one is sent.  Joins of 160
  // nodes on one SM, x 64 / x 4096: 5.0 / 18.0 ms, one entry at a time 10.5 /
  // 49.3 (the windowed kernel: 8.3 / 23.3).
  template <typename F>
  __device__ __forceinline__ void scan_lds(uint32_t end, F f) const {
    for (uint32_t i0 = 0; i0 < end; i0 += 4) {
      uint64_t kk[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) kk[u] = q[(i0 + u < end ? i0 + u : end - 1u) * TH + x];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) f(i0 + u, kk[u]);
    }
  }
  template <typename F>
  __device__ __forceinline__ void scan_scratch(uint32_t end, F f) const {
    for (uint32_t i0 = QF; i0 < end; i0 += 8) {
      uint64_t kk[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) kk[u] = q_g[((i0 + u < end ? i0 + u : end - 1u) - QF) * TH + x];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) f(i0 + u, kk[u]);
    }
  }
  // The smallest due entry of the list moves to `best`; LDS: the whole list
  // is there.
  template <bool LDS>
  __device__ __forceinline__ void take_best() {
    uint32_t at = 0;
    auto least = [&](uint32_t i, uint64_t k) {
      const bool t = k < best;
      best = t ? k : best;
      at = t ? i : at;
    };
    scan_lds(LDS || nd < QF ? nd : QF, least);
    if constexpr (!LDS) scan_scratch(nd, least);
    --nd;  // the last due entry takes its place, the last entry that one's
    --n;
    if constexpr (LDS) {
      if (at != nd) q[at * TH + x] = q[nd * TH + x];
      if (nd != n) q[nd * TH + x] = q[n * TH + x];
    } else {
      if (at != nd) q_set(x, at, q_get(x, nd));
      if (nd != n) q_set(x, nd, q_get(x, n));
    }
  }
  // The due entries to the front of the list (a swap writes at or below the
  // entry at hand).
  template <bool LDS>
  __device__ __forceinline__ void split_due(uint32_t H) {
    mn = kNone;
    const uint32_t l = LDS || n < QF ? n : QF;
    scan_lds(l, [&](uint32_t i, uint64_t k) {
      if (i >= l) return;
      const uint32_t c = (uint32_t)(k >> 32);
      if (c >= H) {
        mn = c < mn ? c : mn;
        return;
      }
      if (i != nd) {
        q[i * TH + x] = q[nd * TH + x];
        q[nd * TH + x] = k;
      }
      ++nd;
    });
    if constexpr (!LDS)
      scan_scratch(n, [&](uint32_t i, uint64_t k) {
        if (i >= n) return;
        const uint32_t c = (uint32_t)(k >> 32);
        if (c >= H) {
          mn = c < mn ? c : mn;
          return;
        }
        if (i != nd) {
          q_set(x, i, q_get(x, nd));
          q_set(x, nd, k);
        }
        ++nd;
      });
  }
  __device__ __forceinline__ void next_best() {
    best = ~0ull;
    if (nd == 0) return;
    if (n <= QF)
      take_best<true>();
    else
      take_best<false>();
  }

  // Release along one edge into a shared node (atomics; the target may be in
  // another CTA on another SM).  H: the window end in the local phase (the
  // target is then on this SM), 0 in the memory phase.
  __device__ __forceinline__ void release_shared(uint32_t w, uint32_t r, uint32_t src_cta, uint32_t H) {
    atomicMax(st_acc(&state[w]), r);
    mem_wait();
    const uint32_t old = atomicAdd(st_cnt(&state[w]), 1u);
    if (old + 1u != (uint32_t)G.indeg[w]) return;
    const uint32_t acc = gld(st_acc(&state[w]));
    const uint32_t cw = G.nodes[w].cta;
    if (cw == src_cta) {
      ready(acc, w, H);
    } else if (cw < uni((uint32_t)lds()[kTeamNextCta])) {  // dispatched: ready at max(release, launch)
      const uint32_t launch = gld(&cst[cw].launch), t = gld(&cst[cw].sm);
      const uint32_t cyc = acc > launch ? acc : launch;
      push(t, cyc, w);
      lds_min(lds() + red_next, cyc);  // its owner may have taken its minimum already
    }
  }
  __device__ __forceinline__ void ready(uint32_t cyc, uint32_t low, uint32_t H) {
    if (H)
      push_own(cyc, low, H);
    else
      push(x, cyc, low);
  }

  // Releases of a node, the edges of `which` (1: released at issue, 2: at
  // completion, 3: both), in two halves: the states of its inline successors
  // set out before the node's stores (loads and stores return in order, so a
  // load behind a store waits for it), and the releases once it is timed (s1:
  // start + 1, f: finish, H as above).
  struct Succ {
    uint64_t sv[kInlineSucc];
    bool sel[kInlineSucc], slow;
  };
  __device__ __forceinline__ Succ load_succ(const Rec& rec, uint32_t which) const {
    const uint32_t nout = rec.nsucc();
    Succ z;
    z.slow = nout > kInlineSucc;
#pragma unroll
    for (uint32_t k = 0; k < kInlineSucc; ++k) {
      const uint32_t bits = rec.succ(k) >> GTS_EDGE_KIND_SHIFT;
      const bool at_issue = (bits & kDevOrder) && !ofin;
      const bool in = k < nout;
      z.slow |= in && (bits & kDevShared);
      z.sel[k] = in && !(bits & kDevShared) && (which & (at_issue ? 1u : 2u)) != 0u;
      z.sv[k] = 0;
      // a node with one in-edge needs no state: this release readies it
      if (z.sel[k] && rec.sindeg(k) != 1) z.sv[k] = state[rec.succ(k) & GTS_EDGE_TARGET_MASK];
    }
    return z;
  }
  __device__ __forceinline__ void release(const Rec& rec, const Succ& z, uint32_t which, uint32_t s1, uint32_t f,
                                          uint32_t H) {
#pragma unroll
    for (uint32_t k = 0; k < kInlineSucc; ++k) {
      if (!z.sel[k]) continue;
      const uint32_t bits = rec.succ(k) >> GTS_EDGE_KIND_SHIFT, w = rec.succ(k) & GTS_EDGE_TARGET_MASK;
      const uint32_t r = ((bits & kDevOrder) && !ofin) ? s1 : f;
      const uint32_t cnt = (uint32_t)(z.sv[k] >> 32) + 1u;
      uint32_t acc = (uint32_t)z.sv[k];
      acc = r > acc ? r : acc;
      if (cnt == rec.sindeg(k))
        ready(acc, w, H);  // its state is not read again
      else
        state[w] = ((uint64_t)cnt << 32) | acc;
    }
    if (z.slow) release_more(rec, rec.nsucc(), which, s1, f, H);
  }
  // Successors beyond the inline three, four at a time (their entries, then
  // in-degrees, then states in flight together; a node's successors are
  // distinct), and inline ones into shared nodes.
  __device__ __forceinline__ void release_more(const Rec& rec, uint32_t nout, uint32_t which, uint32_t s1, uint32_t f,
                                               uint32_t H) {
    for (uint32_t k = 0; k < kInlineSucc && k < nout; ++k) {
      const uint32_t ent = rec.succ(k), bits = ent >> GTS_EDGE_KIND_SHIFT;
      const bool at_issue = (bits & kDevOrder) && !ofin;
      if ((bits & kDevShared) && (which & (at_issue ? 1u : 2u)))
        release_shared(ent & GTS_EDGE_TARGET_MASK, at_issue ? s1 : f, rec.cta(), H);
    }
    const uint32_t base = t_n ? t_node0 + (rec.cta() - t_kc0) * t_n : 0u;
    const gmem<const uint32_t>* sp = (const gmem<const uint32_t>*)(t_n ? G.tsucc : G.succ) + rec.sb();
    const gmem<const uint16_t>* ip = (const gmem<const uint16_t>*)(t_n ? G.tindeg + t_base : G.indeg);
    for (uint32_t k0 = kInlineSucc; k0 < nout; k0 += 4) {
      uint32_t ent[4], ind[4];
      uint64_t sv[4];
      bool sel[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) ent[u] = k0 + u < nout ? sp[k0 + u] : 0u;
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        const bool at_issue = ((ent[u] >> GTS_EDGE_KIND_SHIFT) & kDevOrder) && !ofin;
        sel[u] = k0 + u < nout && (which & (at_issue ? 1u : 2u)) != 0u;
        ind[u] = sel[u] ? (uint32_t)ip[ent[u] & GTS_EDGE_TARGET_MASK] : 0u;
      }
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        sv[u] = 0;
        if (sel[u] && ind[u] != 1 && !((ent[u] >> GTS_EDGE_KIND_SHIFT) & kDevShared))
          sv[u] = state[(ent[u] & GTS_EDGE_TARGET_MASK) + base];
      }
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        if (!sel[u]) continue;
        const uint32_t bits = ent[u] >> GTS_EDGE_KIND_SHIFT, w = (ent[u] & GTS_EDGE_TARGET_MASK) + base;
        const uint32_t r = ((bits & kDevOrder) && !ofin) ? s1 : f;
        if (bits & kDevShared) {
          release_shared(w, r, rec.cta(), H);
          continue;
        }
        const uint32_t cnt = (uint32_t)(sv[u] >> 32) + 1u;
        uint32_t acc = (uint32_t)sv[u];
        acc = r > acc ? r : acc;
        if (cnt == ind[u])
          ready(acc, w, H);
        else
          state[w] = ((uint64_t)cnt << 32) | acc;
      }
    }
  }

  // ---- memory arrivals of this SM, in cycle order: RL entries in LDS, those
  // behind them in scratch
  __device__ __forceinline__ uint32_t ring_at(uint32_t i) const {  // the i-th entry's place, i <= RL
    const uint32_t p = rh + i;
    return (p >= RL ? p - RL : p) * TH + x;
  }
  __device__ __forceinline__ void ring_push(uint32_t cyc, uint32_t low, uint32_t op) {
    if (gc == 0 && rc < RL) {
      set4(rg + ring_at(rc), low, cyc, op, 0u);
      ++rc;
    } else if (gc < kRing) {
      uint32_t* e = mq_g + (x * kRing + (gh + gc) % kRing) * kRingWords;
      e[0] = low;
      e[1] = cyc;
      e[2] = op;
      ++gc;
    } else {
      bad |= kBadQueue;
    }
  }
  // d entries leave the front; the LDS part fills up again from scratch
  __device__ __forceinline__ void ring_pop(uint32_t d) {
    rh += d;
    rh = rh >= RL ? rh - RL : rh;
    rc -= d;
    while (gc != 0 && rc < RL) {
      const uint32_t* e = mq_g + (x * kRing + gh) * kRingWords;
      set4(rg + ring_at(rc), arrived(e[0]), arrived(e[1]), arrived(e[2]), 0u);
      ++rc;
      gh = (gh + 1u) % kRing;
      --gc;
    }
  }

  // Issue the ready nodes of this SM with cycle < H, in (cycle, id) order;
  // returns the steps this wave took.
  __device__ __forceinline__ uint32_t local_phase(uint32_t H) {
    n = q_cnt[x];
    n = n < qcap ? n : qcap;
    mn = q_min[x];
    nd = 0;
    best = ~0ull;
    if (__ballot(mn < H)) {
      if (!__ballot(n > 4u) && QF >= 4u) {
        start_short(H);
      } else {
        if (mn < H) {  // due entries to the front
          if (n <= QF)
            split_due<true>(H);
          else
            split_due<false>(H);
        }
        next_best();
      }
    }
    uint32_t steps = 0;
    if (hot) {
      steps = nsub == 1u ? hot_steps<1>(H) : hot_steps<4>(H);
    } else {
      while (__ballot(best != ~0ull)) {
        ++steps;
        if (best != ~0ull) step(H);
      }
    }
    q_cnt[x] = n;
    q_min[x] = mn;
    return steps;
  }
  // split_due and next_best of lists of at most four entries, straight-line.
  __device__ __forceinline__ void start_short(uint32_t H) {
    uint64_t kk[4];
    uint32_t dues = 0, at = 4;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) kk[u] = q[u * TH + x];
    mn = kNone;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t c = u < n ? (uint32_t)(kk[u] >> 32) : kNone;  // kNone: no entry
      const bool due = c < H;
      dues += due ? 1u : 0u;
      const bool t = due && kk[u] < best;
      best = t ? kk[u] : best;
      at = t ? u : at;
      mn = !due && c < mn ? c : mn;
    }
    nd = dues ? dues - 1u : 0u;
    uint32_t di = 0, li = nd;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {  // back in order [due | later], without the best one
      const bool stay = u < n && u != at;
      const bool due = (uint32_t)(kk[u] >> 32) < H;
      const uint32_t p = due ? di : li;
      di += stay && due ? 1u : 0u;
      li += stay && !due ? 1u : 0u;
      lmem<uint64_t>* const to = stay ? q + p * TH + x : lds64(kTeamSpare);
      *to = kk[u];
    }
    n = li;
  }

  // Timing of a node ready at t on the SM's servers: it holds its class's
  // subpartition lanes (compute), the shared-memory pipe or the global-memory
  // engine (memory nodes; L2 / DRAM follow in the memory phase), SYNC nothing;
  // every held server becomes free at start + occupancy.  False past the last
  // cycle.
  __device__ __forceinline__ bool time_node(const uint4& od, uint32_t t, uint32_t& st, uint32_t& fin) {
    const uint32_t cls = od.w & 7u;
    const bool comp = cls <= C_SFU, is_mem = cls == C_GLOAD || cls == C_GSTORE;
    lmem<uint32_t>* Sv = srv + (comp ? (od.w >> 16) : smem_w + (is_mem ? 1u : 0u)) * TH + x;
    st = t;
    if (nsub == 1u || !comp) {
      if (cls != C_SYNC) {
        const uint32_t a = nocont ? 0u : (uint32_t)Sv[0];
        st = a > st ? a : st;
      }
    } else if (!nocont) {
      for (uint32_t l = 0; l < nsub; ++l) {
        const uint32_t a = Sv[l * TH];
        st = (od.w >> (8u + l)) & 1u && a > st ? a : st;
      }
    }
    const uint64_t fr = (uint64_t)st + od.x;
    const uint64_t f = fr + (is_mem ? 0u : od.z);
    if (f > kMaxCycle) {
      bad |= kBadOverflow;
      return false;
    }
    if (nsub == 1u || !comp) {
      if (cls != C_SYNC) Sv[0] = (uint32_t)fr;
    } else {
      for (uint32_t l = 0; l < nsub; ++l)
        if ((od.w >> (8u + l)) & 1u) Sv[l * TH] = (uint32_t)fr;
    }
    fin = (uint32_t)f;
    ++n_issued;
    return true;
  }

  // One step of a kernel in global memory.
  __device__ __forceinline__ void step(uint32_t H) {
    const uint32_t t = (uint32_t)(best >> 32), v = (uint32_t)best;
    const Rec rec = rec_of(v);
    next_best();
    const uint32_t op = rec.op();
    const uint4 od = get4(optab + op);
    const uint32_t cls = od.w & 7u;
    const bool is_mem = cls == C_GLOAD || cls == C_GSTORE, book = !is_mem && !mem_only && !sink_ret;
    const uint32_t which = is_mem ? 1u : 3u;
    const Succ z = load_succ(rec, which);
    uint4 cs = make_uint4(0, 0, 0, 0);
    if (book) cs = *reinterpret_cast<const uint4*>(&cst[rec.cta()]);
    uint32_t st, f;
    if (!time_node(od, t, st, f)) return;
    if (is_mem) ring_push(st, v, op);
    release(rec, z, which, st + 1u, f, H);
    if (!is_mem) record(v, st, f);
    if (book) {  // a compute node never completes its CTA
      const uint32_t mf = f > cs.w ? f : cs.w;
      *reinterpret_cast<uint2*>(&cst[rec.cta()].left) = make_uint2(cs.z - 1u, mf);
    }
  }

  // A memory node of a kernel in global memory finishes at f: outputs, CTA
  // bookkeeping, releases.
  __device__ __forceinline__ void complete(uint32_t v, uint32_t s, uint32_t f) {
    const Rec rec = rec_of(v);
    const Succ z = load_succ(rec, 2u);
    uint4 cs = make_uint4(0, 0, 0, 0);
    if (!sink_ret) cs = *reinterpret_cast<const uint4*>(&cst[rec.cta()]);
    release(rec, z, 2u, 0u, f, 0u);
    record(v, s, f);
    if (sink_ret) {
      if ((rec.b.w >> 16) & kRecSink) ret_push(f, 0u);  // the sink finishes last
    } else {
      const uint32_t left = cs.z - 1u;
      const uint32_t mf = f > cs.w ? f : cs.w;
      *reinterpret_cast<uint2*>(&cst[rec.cta()].left) = make_uint2(left, mf);
      if (left == 0) ret_push(mf, 0u);  // the CTA retires at its largest finish
    }
  }

  // ---- kernels that run from LDS
  __device__ __forceinline__ uint32_t node_of(uint32_t low) const {
    return t_node0 + (low >> (nb + pb)) * t_n + ((low >> pb) & ((1u << nb) - 1u));
  }
  __device__ __forceinline__ lmem<uint4>* rec_at(uint32_t low) const {
    return rec_l + ((low >> pb) & ((1u << nb) - 1u)) * 2u;
  }
  __device__ __forceinline__ lmem<uint32_t>* slots_of(uint32_t low) const {
    return st_l + (low & ((1u << pb) - 1u)) * t_slots;
  }
  // Releases into the successors w[0..C): s1 the start + 1, f the finish; H:
  // the window's end, or 0 in the memory phase (nothing is due then).  SPILL:
  // the list may run past its LDS part.  sb: the CTA's slots, keep: the
  // entry without its node.
  template <uint32_t C, bool SPILL>
  __device__ __forceinline__ void release_hot(const uint32_t (&w)[C], uint32_t s1, uint32_t f, uint32_t H,
                                              lmem<uint32_t>* sb, uint32_t keep) {
    uint32_t sv[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) sv[k] = sb[(w[k] >> 12) & 1023u];
    uint64_t key[C];
    uint32_t dcyc[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) {
      const uint32_t r = ((w[k] >> 27) & 1u ? s1 : f) - t_cyc;
      const uint32_t cnt = (sv[k] >> kSlotBits) + 1u;
      uint32_t acc = sv[k] & kSlotMask;
      acc = r > acc ? r : acc;
      const bool rdy = cnt == ((w[k] >> 22) & 31u);
      sb[(w[k] >> 12) & 1023u] = rdy ? 0u : cnt << kSlotBits | acc;  // back to zero for the slot's next node
      acc += t_cyc;
      const uint32_t low = keep | (w[k] & 0xFFFu) << pb;
      key[k] = ((uint64_t)acc << 32) | low;
      if constexpr (SPILL) {
        dcyc[k] = kNone;
        if (rdy) push_own(acc, low, H);
      } else {
        // to the list's end, where it stays if it is a later one
        const uint32_t cyc = rdy ? acc : kNone;
        const bool due = cyc < H, later = rdy && !due;
        q[n * TH + x] = key[k];
        n += later ? 1u : 0u;
        mn = later && cyc < mn ? cyc : mn;
        dcyc[k] = due ? cyc : kNone;
      }
    }
    if (SPILL || H == 0u) return;
    bool more = false;
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) {
      const bool due = dcyc[k] != kNone;
      const bool lt = due && key[k] < best;
      const uint64_t o = lt ? best : key[k];  // the later one of the two stays in the list
      best = lt ? key[k] : best;
      key[k] = o;
      dcyc[k] = due && o != ~0ull ? 0u : kNone;
      more |= dcyc[k] == 0u;
    }
    if (__ballot(more)) {
#pragma unroll
      for (uint32_t k = 0; k < C; ++k)
        if (dcyc[k] == 0u) {
          if (nd != n) q[n * TH + x] = q[nd * TH + x];
          q[nd * TH + x] = key[k];
          ++nd;
          ++n;
        }
    }
  }
  // Releases into the first cnt successors of c (words 0-3 of the record, with
  // the others in words 4-7), two at a time while any lane has them.
  template <bool SPILL>
  __device__ __forceinline__ void release_words(const uint4& c, uint32_t cnt, uint32_t s1, uint32_t f, uint32_t H,
                                                lmem<uint32_t>* sb, uint32_t keep) {
    const uint32_t w0[2] = {c.x, c.y}, w1[2] = {c.z, c.w};
    release_hot<2, SPILL>(w0, s1, f, H, sb, keep);
    if (__ballot(cnt > 2u)) release_hot<2, SPILL>(w1, s1, f, H, sb, keep);
  }
  // Most successors a step or a completion pushes.
  static constexpr uint32_t kPushes = 8;

  // Steps until no node is due.  NS: server words per compute class, 1 or (at
  // most) 4.
  template <uint32_t NS>
  __device__ __forceinline__ uint32_t hot_steps(uint32_t H) {
    uint32_t steps = 0;
    while (true) {
      const bool act = best != ~0ull;
      if (!__ballot(act)) return steps;
      ++steps;
      if (__ballot(act && (n + kPushes > QF || rc >= RL)))
        hot_step<NS, true>(H, act);
      else
        hot_step<NS, false>(H, act);
    }
  }
  template <uint32_t NS, bool SPILL>
  __device__ __forceinline__ void hot_step(uint32_t H, bool act) {
    uint32_t v = 0, st = 0, f = 0;
    bool is_mem = true;
    if (act) {
      const uint32_t t = (uint32_t)(best >> 32), low = (uint32_t)best;
      const lmem<uint4>* const rp = rec_at(low);
      const uint4 a = get4(rp);
      const uint32_t cq = own[low & ((1u << pb) - 1u)];
      best = ~0ull;
      if (nd != 0) {
        if (!SPILL || n <= QF)
          take_best<true>();
        else
          take_best<false>();
      }
      const uint32_t op = G.n_ops + t_ops + cq * t_nslot + ((a.x >> 28) | (a.y >> 28 & 7u) << 4);
      const uint4 od = get4(optab + op);
      is_mem = (a.w >> 28) & 1u;
      const uint32_t cls = od.w & 7u;
      const bool comp = cls <= C_SFU;
      // SYNC nodes go through a word of their own with no occupancy: nodes
      // come in cycle order, so it never delays one
      const uint32_t word = comp ? od.w >> 16 : cls == C_SYNC ? sync_w : smem_w + (is_mem ? 1u : 0u);
      lmem<uint32_t>* const Sv = srv + word * TH + x;
      const uint32_t held = comp ? od.w >> 8 : 1u;
      st = t;
      uint32_t busy[NS];
#pragma unroll
      for (uint32_t l = 0; l < NS; ++l) busy[l] = Sv[l * TH];
#pragma unroll
      for (uint32_t l = 0; l < NS; ++l) {
        const bool h = NS == 1 || ((held >> l) & 1u) != 0u;
        st = h && !nocont && busy[l] > st ? busy[l] : st;
      }
      const uint32_t fr = add_sat(st, od.x), s1 = add_sat(st, 1u);
      f = add_sat(fr, is_mem ? 0u : od.z);
      bad |= f > kMaxCycle ? kBadOverflow : 0u;
      bad |= f - t_cyc > kSlotMask ? kBadQueue : 0u;
#pragma unroll
      for (uint32_t l = 0; l < NS; ++l) {
        lmem<uint32_t>* const to = NS == 1 || ((held >> l) & 1u) != 0u ? Sv + l * TH : lds() + kTeamSpare;
        *to = fr;
      }
      ++n_issued;
      if constexpr (SPILL) {
        if (is_mem) ring_push(st, low, op);
      } else {
        lmem<uint4>* const to = is_mem ? rg + ring_at(rc) : (lmem<uint4>*)(lds() + kTeamSpare);
        set4(to, low, st, op, 0u);
        rc += is_mem ? 1u : 0u;
      }
      lmem<uint32_t>* const sb = slots_of(low);
      const uint32_t keep = low & ~(((1u << nb) - 1u) << pb), cnt = a.z >> 28;
      release_words<SPILL>(a, cnt, s1, f, H, sb, keep);
      if (__ballot(cnt > 4u)) {
        if (cnt > 4u) release_words<SPILL>(get4(rp + 1), cnt - 4u, s1, f, H, sb, keep);
      }
      v = node_of(low);
    }
    log_node(act && !is_mem, v, st, f);
  }
  // This SM's d arrivals of the batch, from slot p on, complete in order.
  __device__ __forceinline__ void hot_finish(uint32_t p, uint32_t d) {
    best = ~0ull;
    nd = 0;
    for (uint32_t u = 0; __ballot(u < d); ++u) {
      if (__ballot(u < d && n + kPushes > QF))
        hot_complete<true>(p + u, u < d);
      else
        hot_complete<false>(p + u, u < d);
    }
    q_cnt[x] = n;
    q_min[x] = mn;
  }
  template <bool SPILL>
  __device__ __forceinline__ void hot_complete(uint32_t i, bool act) {
    uint32_t v = 0, c = 0, f = 0;
    if (act) {
      const uint64_t key = lds64(kTeamKey)[i];
      const uint4 od = get4(optab + lds()[kTeamOp + i]);
      const uint32_t m = lds()[kTeamMend + i];
      const uint32_t low = (uint32_t)key;
      c = (uint32_t)(key >> 32);
      const lmem<uint4>* const rp = rec_at(low);
      const uint4 a = get4(rp), w = get4(rp + 1);
      const uint32_t e = add_sat(c, od.x), g = e > m ? e : m;
      f = add_sat(g, od.z);
      bad |= f > kMaxCycle ? kBadOverflow : 0u;
      bad |= f - t_cyc > kSlotMask ? kBadQueue : 0u;
      release_words<SPILL>(w, a.w >> 29, f, f, 0u, slots_of(low), low & ~(((1u << nb) - 1u) << pb));
      if (a.y >> 31) ret_push(f, low & ((1u << pb) - 1u));  // the sink finishes last
      v = node_of(low);
    }
    log_node(act, v, c, f);
  }

  // The ordered batch (M arrivals, position lane * E + r) through the servers:
  // the end of each one's memory service to LDS, for the slots of this wave.
  // Relative to the window start T in 32 bits when `small` (occupancies and
  // the servers' backlog then sum to less than 2^30), else in doubles.
  template <uint32_t E, bool SMALL>
  __device__ __forceinline__ void serve(uint32_t M, uint32_t base, uint32_t cnt, uint32_t T) {
    using MP = std::conditional_t<SMALL, MaxPlus32, MaxPlus>;
    using Num = std::conditional_t<SMALL, int32_t, double>;
    const Num zero = 0;
    const lmem<uint4>* const srt = (const lmem<uint4>*)(lds() + kTeamSorted);
    lmem<uint32_t>* const mend = lds() + kTeamMend;
    auto most = [](Num a, Num b) { return a > b ? a : b; };
    Num cyc[E], occ[E];
    uint32_t sl[E];
    bool in[E], dram[E];
    bool any_l2 = false, any_dr = false;
#pragma unroll
    for (uint32_t r = 0; r < E; ++r) {
      const uint32_t p = lane * E + r;
      in[r] = p < M;
      const uint4 e = get4(srt + (in[r] ? p : 0u));
      cyc[r] = (Num)(e.x - T);
      occ[r] = (Num)e.z;
      sl[r] = e.y & 0x7FFFFFFFu;
      dram[r] = (e.y >> 31) != 0u;
      any_l2 |= in[r] && !dram[r];
      any_dr |= in[r] && dram[r];
    }
#pragma unroll
    for (uint32_t d = 0; d < 2; ++d) {
      if (!__ballot(d ? any_dr : any_l2)) continue;
      double& av = d ? dram_av : l2_av;
      const double late = av - (double)T;  // its backlog at the window start
      const Num from = (Num)(late > 0.0 ? late : 0.0);
      MP f;
      f.a = SMALL ? (Num)kNeg32 : (Num)kNegInf;
      f.o = zero;
#pragma unroll
      for (uint32_t r = 0; r < E; ++r)
        if (in[r] && dram[r] == (d != 0)) f = after(f, MP{cyc[r], occ[r]});
      const MP inc = wave_incl_mp(f);
      const MP exc = dpp_mp<kWaveShr1>(inc);
      Num y = most(from, exc.a) + exc.o;
      if (!nocont) {
        Num ta, to;
        if constexpr (SMALL) {
          ta = (Num)lane_u32((uint32_t)inc.a, 63);
          to = (Num)lane_u32((uint32_t)inc.o, 63);
        } else {
          ta = lane_f64(inc.a, 63);
          to = lane_f64(inc.o, 63);
        }
        av = (double)T + (double)(most(from, ta) + to);
      }
#pragma unroll
      for (uint32_t r = 0; r < E; ++r)
        if (in[r] && dram[r] == (d != 0)) {
          const Num m = nocont ? cyc[r] : most(y, cyc[r]);
          y = m + occ[r];
          uint32_t end;
          if constexpr (SMALL) {
            end = T + (uint32_t)y;
            end = end < T ? 0xFFFFFFFFu : end;
          } else {
            end = (uint32_t)__builtin_fmin((double)T + y, 4294967295.0);
          }
          if (sl[r] - base < cnt) mend[sl[r]] = end;
        }
    }
    wsync();
  }

  // ---- dispatch at cycle t (first wave only): up to 64 CTAs at a time are
  // placed on SMs (most free slots, lowest id), then set up by one lane each
  __device__ __forceinline__ void dispatch(uint32_t t) {
    lmem<uint32_t>* const ctl = lds() + kTeamCtl;
    uint32_t next_cta = uni((uint32_t)ctl[0]), cur_k = uni((uint32_t)ctl[2]), k_begin = uni((uint32_t)ctl[3]), k_end = uni((uint32_t)ctl[4]);
    const uint32_t retired = uni((uint32_t)ctl[1]);
    if (next_cta >= G.n_ctas) return;
    uint32_t kstart_k = uni((uint32_t)ctl[5]), kstart_t = uni((uint32_t)ctl[6]);
    uint64_t slots = uni64((uint64_t)*(lmem<uint64_t>*)(ctl + 8));
    while (next_cta < G.n_ctas) {
      while (next_cta >= k_end) {
        ++cur_k;
        const KernelDev kd = G.kernels[cur_k];
        k_begin = uni(kd.cta_begin);
        k_end = uni(kd.cta_end);
        slots = uni64(kernel_slots(kd, hw));
      }
      if (retired < k_begin) break;  // the previous kernel is still running
      // every CTA before next_cta is dispatched and `retired` of them have
      // retired, all of the running kernel: its free slots are known
      const uint64_t cap = (uint64_t)nsm * slots, busy = next_cta - retired;
      const uint64_t room = cap > busy ? cap - busy : 0u;
      uint32_t lim = k_end - next_cta < 64u ? k_end - next_cta : 64u;
      lim = room < lim ? (uint32_t)room : lim;
      if (lim == 0) break;
      // the records of the CTAs to place, in flight during the placement
      const uint32_t c = next_cta + lane;
      uint4 c0 = make_uint4(0, 0, 0, 0), c1 = make_uint4(0, 0, 0, 0);
      if (lane < lim) {
        const gmem<const uint32_t>* p = (const gmem<const uint32_t>*)(G.ctas + c);
        c0 = ld4(p);      // node_begin, node_count, root_begin, root_count
        c1 = ld4(p + 4);  // memory nodes, first three roots
      }
      // an SM's key: fewest resident CTAs, then lowest id; 0 when full
      uint32_t rs[NW], key[NW], mysm = 0;
      auto key_of = [&](uint32_t j) {
        const uint32_t s = lane * nw + j;
        return j < nw && s < nsm && rs[j] < slots ? ((0xFFFFFFu - rs[j]) << 8) | (255u - s) : 0u;
      };
#pragma unroll
      for (uint32_t j = 0; j < NW; ++j) {
        rs[j] = res[lane + 64u * j];
        key[j] = key_of(j);
      }
      uint32_t k = 0;
      while (k < lim) {
        uint32_t best = key[0];
#pragma unroll
        for (uint32_t j = 1; j < NW; ++j) best = key[j] > best ? key[j] : best;
        best = wave_max_u32(best);
        if (best == 0) break;  // every SM is full
        const uint32_t s = 255u - (best & 255u);
        if (lane == k) mysm = thread_of(s);
#pragma unroll
        for (uint32_t j = 0; j < NW; ++j) {
          rs[j] += key[j] == best ? 1u : 0u;
          key[j] = key_of(j);
        }
        ++k;
      }
#pragma unroll
      for (uint32_t j = 0; j < NW; ++j) res[lane + 64u * j] = rs[j];
      if (k == 0) break;
      if (run_k != cur_k) {  // the first CTAs of a kernel: it is now the running one
        load_template(cur_k);
        if (hot) {
          for (uint32_t i = lane; i < t_places; i += 64) own[own_cap + i] = i;
          if (lane == 0) lds()[kTeamFree] = t_places;
          wsync();
        }
      }
      if (kstart_k != cur_k) {
        kstart_k = cur_k;
        kstart_t = t;
      }
      const uint64_t launch = (uint64_t)t + uni((uint32_t)ctl[14]) + (kstart_t == t ? uni((uint32_t)ctl[15]) : 0u);
      if (launch > kMaxCycle) {
        bad |= kBadOverflow;
        break;
      }
      uint32_t place = 0, cls = 0;
      if (hot) {
        // a free place each (at most t_places CTAs are resident; its slots
        // are at zero)
        const uint32_t free = uni((uint32_t)lds()[kTeamFree]);
        if (k > free) {  // cannot happen
          bad |= kBadQueue;
          break;
        }
        if (lane < k) {
          place = own[own_cap + free - 1u - lane];
          cls = ((const gmem<const uint8_t>*)G.cclass)[c];
        }
        if (lane == 0) lds()[kTeamFree] = free - k;
      } else {
        zero_ctas(k, c0);
      }
      if (lane < k) start_cta(c, mysm, (uint32_t)launch, place, c0, c1, cls);
      next_cta += k;
      wsync();
    }
    if (lane == 0) {
      ctl[0] = next_cta;
      ctl[2] = cur_k;
      ctl[3] = k_begin;
      ctl[4] = k_end;
      ctl[5] = kstart_k;
      ctl[6] = kstart_t;
      *(lmem<uint64_t>*)(ctl + 8) = slots;
      ctl[10] = run_k;
    }
    wsync();
  }

  // dp retirements (due_l, at most 64) of a full machine: each one's SM takes
  // the next pending CTA at its cycle, in the order (cycle, SM id) -- the only
  // free slot of its cycle, or one of as many equally free SMs as retire then.
  // The new CTA inherits the place.  False (nothing done) if one SM retires
  // two CTAs in one cycle.  Lane l holds the records of CTA first + l.
  __device__ __forceinline__ bool refill(uint32_t dp, uint32_t first, const uint4& c0, const uint4& c1, uint32_t cls) {
    lmem<uint64_t>* const due_l = lds64(kTeamKey);
    lmem<uint32_t>* const ctl = lds() + kTeamCtl;
    const uint64_t mine = lane < dp ? due_l[lane] : ~0ull;
    const uint64_t key = lane < dp ? (mine & ~0xFF000000ull) | (uint64_t)sm_of((uint32_t)mine >> 24) << 24 : ~0ull;
    uint32_t rank = 0;
    bool twice = false;
    for (uint32_t j = 0; j < dp; ++j) {
      const uint64_t kj = ((uint64_t)lane_u32((uint32_t)(key >> 32), (int)j) << 32) | lane_u32((uint32_t)key, (int)j);
      rank += kj < key ? 1u : 0u;
      twice |= lane < dp && j != lane && (kj >> 24) == (key >> 24);
    }
    if (__ballot(twice)) return false;
    const uint32_t cta_lat = uni((uint32_t)ctl[14]), k_lat = uni((uint32_t)ctl[15]), kstart_t = uni((uint32_t)ctl[6]);
    wsync();
    if (lane < dp) due_l[rank] = mine;
    wsync();
    if (lane < dp) {
      const uint64_t e = due_l[lane];
      const uint32_t t = (uint32_t)(e >> 32), sm = (uint32_t)e >> 24, place = (uint32_t)e & 0xFFFFFFu;
      const uint64_t launch = (uint64_t)t + cta_lat + (kstart_t == t ? k_lat : 0u);
      if (launch > kMaxCycle) {
        bad |= kBadOverflow;
      } else {
        start_cta(first + lane, sm, (uint32_t)launch, place, c0, c1, cls);
      }
    }
    if (!hot) zero_ctas(dp, c0);
    return true;
  }
  // CTA c (records c0, c1, class) starts on thread sm's SM at cycle launch: its
  // state, and its ready roots.
  __device__ __forceinline__ void start_cta(uint32_t c, uint32_t sm, uint32_t launch, uint32_t place, const uint4& c0,
                                            const uint4& c1, uint32_t cls) {
    const uint32_t nroots = c0.w & ~kCtaShared;
    if (hot) {
      own[place] = cls;
      for (uint32_t r = 0; r < nroots; ++r) {
        const uint32_t v = r == 0 ? c1.y : r == 1 ? c1.z : r == 2 ? c1.w : G.roots[c0.z + r];
        push(sm, launch, (c - t_kc0) << (nb + pb) | (v - c0.x) << pb | place);
      }
      return;
    }
    if (!sink_ret)  // a CTA that retires with its sink keeps no state
      *reinterpret_cast<uint4*>(&cst[c]) = make_uint4(sm, launch, mem_only ? c1.x : c0.y, 0u);
    for (uint32_t r = 0; r < nroots; ++r) {
      const uint32_t v = r == 0 ? c1.y : r == 1 ? c1.z : r == 2 ? c1.w : G.roots[c0.z + r];
      if (!(c0.w & kCtaShared)) {  // no in-edges at all
        push(sm, launch, v);
      } else {
        const uint64_t sv = gld(&state[v]);
        if ((uint32_t)(sv >> 32) == (uint32_t)G.indeg[v]) {
          const uint32_t acc = (uint32_t)sv;
          push(sm, acc > launch ? acc : launch, v);
        }
      }
    }
  }
  // Node state of the unshared CTAs whose records lanes [0, k) hold (shared
  // ones were zeroed at start).
  __device__ __forceinline__ void zero_ctas(uint32_t k, const uint4& c0) {
    for (uint32_t j = 0; j < k; ++j) {
      const uint32_t n0 = lane_u32(c0.x, (int)j), nc = lane_u32(c0.y, (int)j), fl = lane_u32(c0.w, (int)j);
      if (!(fl & kCtaShared))
        for (uint32_t i = lane; i < nc; i += 64) state[n0 + i] = 0ull;
    }
  }

  // ---- retirement phase (first wave only): retirements below H, in cycle
  // order, each distinct cycle followed by dispatch.  More than kTeamCap of
  // them lower H; the new H goes to LDS.
  __device__ __forceinline__ void retire(uint32_t T, uint32_t H) {
    lmem<uint32_t>* const ctl = lds() + kTeamCtl;
    lmem<uint64_t>* const due_l = lds64(kTeamKey);
    uint32_t cnt = uni((uint32_t)lds()[kTeamRetCnt]);
    cnt = cnt < kRetireCap ? cnt : kRetireCap;
    // the records of the next CTAs, one per lane, in flight while the
    // retirements are counted
    const uint32_t first = uni((uint32_t)ctl[0]);
    uint4 c0 = make_uint4(0, 0, 0, 0), c1 = make_uint4(0, 0, 0, 0);
    uint32_t cls = 0;
    if (first + lane < G.n_ctas) {
      const gmem<const uint32_t>* p = (const gmem<const uint32_t>*)(G.ctas + first + lane);
      c0 = ld4(p);      // node_begin, node_count, root_begin, root_count
      c1 = ld4(p + 4);  // memory nodes, first three roots
      cls = ((const gmem<const uint8_t>*)G.cclass)[first + lane];
    }
    // a CTA leaves its SM and its place (its slots are back at zero)
    auto leave = [&](uint32_t who) {
      lds_add(&res[who >> 24], ~0u);
      if (hot) own[own_cap + lds_add(lds() + kTeamFree, 1u)] = who & 0xFFFFFFu;
    };
    auto below = [&](uint32_t X) {
      uint32_t c = 0;
      for (uint32_t i = lane; i < cnt; i += 64) c += (uint32_t)(ret_get(i) >> 32) < X;
      return wave_sum_u32(c);
    };
    uint32_t D = below(H);
    if (D > kTeamCap) {
      uint32_t lo = T + 1u, hi = H;
      while (hi - lo > 1u) {
        const uint32_t mid = lo + (hi - lo) / 2u;
        if (below(mid) <= kTeamCap)
          lo = mid;
        else
          hi = mid;
      }
      H = lo;
      D = below(H);
    }
    // more than kTeamCap at cycle T alone: released together
    const bool single = D > kTeamCap;
    uint32_t dp = 0, kp = 0, kmin = kNone;
    for (uint32_t base = 0; base < cnt; base += 64) {
      const uint32_t i = base + lane;
      const uint64_t k = i < cnt ? ret_get(i) : ~0ull;
      const bool due = i < cnt && (uint32_t)(k >> 32) < H;
      const bool keep = i < cnt && !due;
      const uint64_t bd = __ballot(due), bk = __ballot(keep);
      if (due) {
        if (single)
          leave((uint32_t)k);
        else
          due_l[dp + lanes_below(bd, lane)] = k;
      }
      if (keep) {
        const uint32_t dst = kp + lanes_below(bk, lane);
        if (dst != i) ret_set(dst, k);
        kmin = (uint32_t)(k >> 32) < kmin ? (uint32_t)(k >> 32) : kmin;
      }
      dp += (uint32_t)__popcll(bd);
      kp += (uint32_t)__popcll(bk);
    }
    kmin = wave_min_u32(kmin);
    wsync();
    if (lane == 0) {
      lds()[kTeamRetCnt] = kp;
      lds()[kTeamRetMin] = kmin;
      ctl[11] = H;
    }
    uint32_t retired = uni((uint32_t)ctl[1]);
    if (single) {
      retired += dp;
      if (lane == 0) ctl[1] = retired;
      wsync();
      dispatch(T);
      return;
    }
    // the usual case: the machine is full and stays full (every retirement
    // makes room for one pending CTA of the running kernel)
    if (dp <= 64u && first < G.n_ctas && uni((uint32_t)ctl[2]) == run_k &&
        uni((uint32_t)ctl[4]) - first >= dp && uni((uint32_t)ctl[4]) > first) {
      const uint64_t room = (uint64_t)nsm * uni64((uint64_t)*(const lmem<uint64_t>*)(ctl + 8));
      if (room == first - retired && refill(dp, first, c0, c1, cls)) {
        if (lane == 0) {
          ctl[0] = first + dp;
          ctl[1] = retired + dp;
        }
        wsync();
        return;
      }
    }
    // up to kTeamCap due ones, four per lane; the earliest cycle each time
    uint32_t rcyc[kTeamCap / 64], rx[kTeamCap / 64];
#pragma unroll
    for (uint32_t u = 0; u < kTeamCap / 64; ++u) {
      const uint32_t i = u * 64u + lane;
      const uint64_t k = i < dp ? due_l[i] : ~0ull;
      rcyc[u] = (uint32_t)(k >> 32);
      rx[u] = (uint32_t)k;
    }
    while (dp) {
      uint32_t m = rcyc[0];
#pragma unroll
      for (uint32_t u = 1; u < kTeamCap / 64; ++u) m = rcyc[u] < m ? rcyc[u] : m;
      m = wave_min_u32(m);
      uint32_t c = 0;
#pragma unroll
      for (uint32_t u = 0; u < kTeamCap / 64; ++u) {
        const bool now = rcyc[u] == m;
        if (now) {
          leave(rx[u]);
          rcyc[u] = kNone;
        }
        c += (uint32_t)__popcll(__ballot(now));
      }
      dp -= c;
      retired += c;
      wsync();
      if (lane == 0) ctl[1] = retired;
      wsync();
      dispatch(m);
      if (__ballot(bad != 0)) break;
    }
  }
};

template <uint32_t NW>
__device__ __forceinline__ void team_body(const Launch& L) {
  constexpr uint32_t TH = 64u * NW, GQ = kTeamHeads;
  const uint32_t b = blockIdx.x;
  if (b >= L.B) return;
  TSim<NW> S;
  lmem<uint32_t>* const lds = S.lds();
  S.G = L.img;
  S.hw = L.hw + (uint64_t)b * HW_WORDS;
  S.b = b;
  S.x = threadIdx.x;
  S.lane = S.x & 63u;
  S.wave = uni(S.x >> 6);
  S.nocont = (L.flags & GTS_NO_CONTENTION) != 0;
  S.ofin = (L.flags & GTS_ORDER_AT_FINISH) != 0;
  S.mem_only = (L.img.props & kGraphComputeFeedsData) != 0;
  S.want_digest = L.out_digest != nullptr;
  S.nsm = S.hw[HW_NSM];
  S.nsub = L.srv_one ? 1u : S.hw[HW_NSUB];
  const uint32_t sstride = server_stride(S.G.props, S.nsub);
  S.smem_w = sstride - 2u;
  S.sync_w = sstride;  // a word beyond the servers
  S.QF = L.qp;
  S.RL = L.team_ring;
  S.retl = L.team_ret;
  S.qcap = S.QF + kPoolSpill * 64u / TH;
  const uint32_t x = S.x, lane = S.lane;
  uint8_t* sim = L.sims + (uint64_t)b * L.layout.stride;
  S.state = reinterpret_cast<uint64_t*>(sim + L.layout.off_state);
  S.cst = reinterpret_cast<CtaState*>(sim + L.layout.off_cta);
  S.mq_g = reinterpret_cast<uint32_t*>(sim + L.layout.off_mq);
  S.q_g = (gmem<uint64_t>*)(sim + L.layout.off_rp);
  S.ret_g = (gmem<uint64_t>*)(sim + L.layout.off_ret);
  const TeamLds W = team_lds(TH, S.G.n_ops + S.G.n_tops, server_stride(S.G.props, L.srv_one ? 1u : L.max_nsub), L.qp,
                             L.team_ring, L.team_ret, L.team_rec, L.team_own, L.team_st);
  S.optab = (lmem<uint4>*)(lds + W.optab);
  S.srv = lds + W.srv;
  S.q_cnt = lds + W.q_cnt;
  S.q_min = lds + W.q_min;
  S.res = lds + W.res;
  S.q = (lmem<uint64_t>*)(lds + W.q);
  S.rg = (lmem<uint4>*)(lds + W.ring);
  S.ret_l = (lmem<uint64_t>*)(lds + W.ret);
  S.rec_l = (lmem<uint4>*)(lds + W.rec);
  S.st_l = lds + W.st;
  S.own = lds + W.own;
  S.log = lds + W.log + S.wave * 3u * kTeamLog;
  S.rec_cap = L.team_rec;
  S.own_cap = L.team_own;
  S.st_cap = L.team_st;
  S.out_cycles = (L.flags & GTS_OUT_NODES) ? L.out_cycles : nullptr;
  lmem<uint64_t>* const w_key = S.lds64(kTeamKey);
  lmem<uint32_t>* const w_k32 = lds + kTeamKey32;
  lmem<uint32_t>* const w_op = lds + kTeamOp;
  lmem<uint4>* const srt = (lmem<uint4>*)(lds + kTeamSorted);
  lmem<uint32_t>* const ctl = lds + kTeamCtl;

  // a kernel whose CTA fits nowhere makes the simulation infeasible
  bool infeasible = false;
  for (uint32_t k = lane; k < S.G.n_kernels; k += 64) infeasible |= kernel_slots(S.G.kernels[k], S.hw) == 0;
  if (__ballot(infeasible)) {  // every wave sees the same
    if (x == 0) {
      L.out_makespan[b] = 0xFFFFFFFFu;
      L.out_status[b] = GTS_SIM_INFEASIBLE;
      if (L.out_digest) L.out_digest[b] = 0;
    }
    return;
  }

  // waves without SMs end here (a barrier waits for the others only)
  S.nw = uni((S.nsm + 63u) / 64u);
  if (S.wave >= S.nw) return;
  const uint32_t nthr = 64u * S.nw;

  // Setup: duration table (every wave goes through all of it for the
  // smallest delays, thread x writes entries x, x + nthr, ...), idle servers,
  // empty queues.
  uint64_t lm_l2 = ~0ull, lm_dr = ~0ull, occ_max = 0;
  for (uint32_t p = lane; p < S.G.n_ops; p += 64) {
    uint4 e = op_entry(S.G.ops[p], S.hw, S.G.props);
    const uint32_t cls = e.w & 7u;
    if (L.srv_one && cls <= C_SFU)  // the class's single word: lane 0 of its slot
      e.w = (e.w & 0xFFu) | (1u << 8) | (compute_slot(S.G.props, cls) << 16);
    if ((p >> 6) % S.nw == S.wave) S.set4(S.optab + p, e.x, e.y, e.z, e.w);
    if (cls == C_GLOAD || cls == C_GSTORE) {
      const uint64_t d = (uint64_t)e.y + e.z;
      uint64_t& lm = (e.w >> 3) & 1u ? lm_dr : lm_l2;
      lm = d < lm ? d : lm;
      occ_max = e.y > occ_max ? e.y : occ_max;
    }
  }
  // memory occupancies whose sum over a batch stays below 2^29
  const bool small_occ = wmax64(occ_max) <= (1u << 29) / kTeamCap;
  lm_l2 = wmin64(lm_l2);
  lm_dr = wmin64(lm_dr);
  const double dmin_l2 = lm_l2 == ~0ull ? __builtin_inf() : (double)lm_l2;
  const double dmin_dr = lm_dr == ~0ull ? __builtin_inf() : (double)lm_dr;
  for (uint32_t i = 0; i < sstride + (L.team_rec ? 1u : 0u); ++i) S.srv[i * TH + x] = 0;
  S.q_cnt[x] = 0;
  S.q_min[x] = kNone;
  S.res[x] = 0;
  if (x < kTeamFixedInit) lds[kTeamCtl + x] = 0;
  if (x < 8u) S.set4((lmem<uint4>*)(lds + kTeamExch) + x, 0u, ~0u, ~0u, 0u);  // no arrivals of absent waves
  __syncthreads();
  for (uint32_t p = x; p < S.G.n_tops; p += nthr) {
    const uint4 e = S.get4(S.optab + S.G.tops[p]);
    S.set4(S.optab + S.G.n_ops + p, e.x, e.y, e.z, e.w);
  }
  if (x == 0) {
    const KernelDev kd = S.G.kernels[0];
    ctl[3] = kd.cta_begin;
    ctl[4] = kd.cta_end;
    ctl[5] = kNone;  // no kernel has started
    *(lmem<uint64_t>*)(ctl + 8) = kernel_slots(kd, S.hw);
    ctl[10] = kNone;
    ctl[14] = S.hw[HW_CTALAT];
    ctl[15] = S.hw[HW_KLAT];
    lds[kTeamRetMin] = kNone;
    for (uint32_t i = 0; i < 4; ++i) lds[kTeamRed + i] = kNone;
  }
  if (S.G.props & kGraphHasShared) {
    for (uint32_t c = x; c < S.G.n_ctas; c += nthr) {
      const CtaDev cd = S.G.ctas[c];
      if (cd.root_count & kCtaShared)
        for (uint32_t i = 0; i < cd.node_count; ++i) S.state[cd.node_begin + i] = 0ull;
    }
  }
  S.run_k = S.staged_k = kNone;  // no CTA dispatched yet
  S.t_n = 0;
  S.sink_ret = S.hot = S.rk32 = false;
  S.log_n = S.log_h = 0;
  S.l2_av = 0.0;
  S.dram_av = 0.0;
  S.rh = S.rc = S.gh = S.gc = 0;
  S.digest = 0;
  S.makespan = 0;
  S.nfin = 0;
  S.bad = 0;
  S.n_issued = 0;
  const bool clk = L.clocks != 0;
  uint64_t ck[5] = {0, 0, 0, 0, 0};
  uint32_t windows = 0, steps = 0, arrivals = 0, most = 0;
  uint32_t rb = 0;  // which half of the exchange words is next

  // Per-wave counts (and the smallest key bound) across the workgroup.
  auto exchange = [&](uint32_t cnt, uint64_t kb, uint32_t& total, uint32_t& base) -> uint64_t {
    lmem<uint32_t>* const e = lds + kTeamExch + rb * 16u;
    rb ^= 1u;
    if constexpr (NW > 1) {
      if (lane == 0) S.set4((lmem<uint4>*)(e + S.wave * 4u), cnt, (uint32_t)kb, (uint32_t)(kb >> 32), 0u);
      lds_barrier<NW>();
      total = base = 0;
      uint64_t k = ~0ull;
#pragma unroll
      for (uint32_t w = 0; w < NW; ++w) {
        const uint4 v = S.get4((lmem<uint4>*)(e + w * 4u));
        const uint64_t kw = ((uint64_t)v.z << 32) | v.y;
        total += v.x;
        base += w < S.wave ? v.x : 0u;
        k = kw < k ? kw : k;
      }
      total = uni(total);
      base = uni(base);
      return uni64(k);
    } else {
      total = cnt;
      base = 0;
      return kb;
    }
  };

  // the kernel whose CTAs were dispatched last is the running one
  auto follow = [&] {
    const uint32_t k = uni((uint32_t)ctl[10]);
    if (k == S.staged_k) return;
    if (k != S.run_k) S.load_template(k);
    S.stage_template();
  };

  __syncthreads();
  if (S.wave == 0) S.dispatch(0);
  __syncthreads();
  if (uni((uint32_t)ctl[10]) != kNone) follow();

  while (true) {
    const uint64_t c0 = clk ? __builtin_amdgcn_s_memtime() : 0ull;
    // T: the earliest pending event.  Each wave's minimum goes to this
    // window's words {ready or arrival, retirement}, which pushes to other
    // SMs lower as well.
    const uint32_t par = (windows & 1u) * 2u;
    {
      uint32_t m = S.q_min[x];
      if (S.rc) {
        const uint32_t h = S.get4(S.rg + S.rh * TH + x).y;
        m = h < m ? h : m;
      }
      m = wave_min_u32(m);
      const bool any_bad = __ballot(S.bad != 0) != 0;
      if (lane == 0) {
        S.lds_min(lds + kTeamRed + par, m);
        if (S.wave == 0) S.lds_min(lds + kTeamRed + par + 1u, lds[kTeamRetMin]);
        if (any_bad) ctl[12] = 1u;
      }
    }
    lds_barrier<NW>();
    const uint32_t rmin = uni((uint32_t)lds[kTeamRed + par + 1u]);
    uint32_t T = uni((uint32_t)lds[kTeamRed + par]);
    if (uni((uint32_t)ctl[12])) break;
    T = rmin < T ? rmin : T;
    if (T == kNone) break;  // cycles stop at kMaxCycle
    S.red_next = kTeamRed + (par ^ 2u);
    if (x == 0) {
      lds[S.red_next] = kNone;
      lds[S.red_next + 1u] = kNone;
      lds[kTeamRetMin] = rmin;
    }
    ++windows;
    bool small;
    // H: no arrival of this window completes before it.  An arrival waits
    // for its server, so a busy server's backlog lengthens the window.
    uint32_t H;
    {
      const double t = (double)T;
      const double a = S.nocont ? t : __builtin_fmax(t, S.l2_av), d = S.nocont ? t : __builtin_fmax(t, S.dram_av);
      double h = __builtin_fmin(a + dmin_l2, d + dmin_dr);
      h = __builtin_fmin(h, t + (double)kWindowMax);
      H = uni((uint32_t)__builtin_fmin(h, 4294967295.0));
      small = small_occ && __builtin_fmax(a, d) - t < (double)(1 << 29);
    }
    const uint64_t c1 = clk ? __builtin_amdgcn_s_memtime() : 0ull;
    if (rmin < H) {
      if (S.wave == 0) S.retire(T, H);
      __syncthreads();
      H = uni((uint32_t)ctl[11]);
      follow();
    }
    const uint64_t c2 = clk ? __builtin_amdgcn_s_memtime() : 0ull;
    steps += S.local_phase(H);
    const uint64_t c3 = clk ? __builtin_amdgcn_s_memtime() : 0ull;

    // Memory phase: the arrivals whose key (cycle, id) is below K <= H << 32,
    // at most kTeamCap of them, from the first GQ of each SM's ring.
    uint32_t ec[GQ], ev[GQ], eo[GQ];  // cycle, entry, op
    const uint32_t ld = S.rc < GQ ? S.rc : GQ;
    uint32_t d = 0;
#pragma unroll
    for (uint32_t u = 0; u < GQ; ++u) {
      const uint4 e = S.get4(S.rg + S.ring_at(u < S.RL ? u : 0u));
      ev[u] = e.x;
      ec[u] = u < ld ? e.y : kNone;
      eo[u] = e.z;
      d += ec[u] < H ? 1u : 0u;
    }
    auto due = [&](uint64_t K) -> uint32_t {
      uint32_t c = 0;
#pragma unroll
      for (uint32_t u = 0; u < GQ; ++u) c += (((uint64_t)ec[u] << 32) | ev[u]) < K;
      return c;
    };
    uint64_t K = (uint64_t)H << 32, kb = K;
    if (__ballot(d == ld && S.rc + S.gc > ld)) {  // more than were loaded may be due
#pragma unroll
      for (uint32_t u = 0; u < GQ; ++u)
        if (u + 1u == ld && d == ld && S.rc + S.gc > ld) kb = (((uint64_t)ec[u] << 32) | ev[u]) + 1u;
      kb = wmin64(kb);
    }
    uint32_t M, wbase;
    uint32_t cw = wave_sum_u32(d);
    const uint64_t Kx = exchange(cw, kb, M, wbase);
    if (Kx < K) {  // some SM has more arrivals than were loaded
      K = Kx;
      d = due(K);
      cw = wave_sum_u32(d);
      exchange(cw, 0, M, wbase);
    }
    if (M > kTeamCap) {
      // the largest cycle boundary that keeps kTeamCap, or, when cycle T
      // alone holds more, a boundary between the keys of cycle T
      const uint64_t Kmax = K;
      auto count = [&](uint64_t k) -> uint32_t {
        uint32_t m, wb;
        exchange(wave_sum_u32(due(k)), 0, m, wb);
        return m;
      };
      uint64_t lo = T, hi = Kmax >> 32;
      if (count(hi << 32) <= kTeamCap) {
        lo = hi;
      } else {
        while (hi - lo > 1) {
          const uint64_t mid = lo + (hi - lo) / 2;
          if (count(mid << 32) <= kTeamCap)
            lo = mid;
          else
            hi = mid;
        }
      }
      K = lo << 32;
      if (lo == T) {
        uint64_t klo = (uint64_t)T << 32, khi = ((uint64_t)T + 1) << 32;
        khi = Kmax < khi ? Kmax : khi;
        while (khi - klo > 1) {
          const uint64_t mid = klo + (khi - klo) / 2;
          if (count(mid) <= kTeamCap)
            klo = mid;
          else
            khi = mid;
        }
        K = klo;
      }
      d = due(K);
      cw = wave_sum_u32(d);
      exchange(cw, 0, M, wbase);
    }
    const uint64_t c4 = clk ? __builtin_amdgcn_s_memtime() : 0ull;
    if (M) {
      const uint32_t p = wbase + wave_excl_scan_u32(d);
#pragma unroll
      for (uint32_t u = 0; u < GQ; ++u)
        if (u < d) {
          w_key[p + u] = ((uint64_t)ec[u] << 32) | ev[u];
          // a window spans at most kWindowMax = 2^10 cycles
          w_k32[p + u] = (ec[u] - T) << 22 | ((ev[u] - S.rk_base) >> S.rk_shift);
          w_op[p + u] = eo[u];
        }
      if (x < kTeamPad) {  // the counts read many keys at a time
        w_key[M + x] = ~0ull;
        w_k32[M + x] = ~0u;
      }
      if (d) S.ring_pop(d);
      lds_barrier<NW>();
      for (uint32_t i = x; i < M; i += nthr) {
        const uint4 od = S.get4(S.optab + w_op[i]);
        const uint64_t mine = w_key[i];
        uint32_t r = 0;
        if (S.rk32) {
          const uint32_t m32 = w_k32[i];
          for (uint32_t j = 0; j < M; j += 16) {
            uint4 kk[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) kk[u] = S.get4((lmem<uint4>*)(w_k32 + j + 4u * u));
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
              r += kk[u].x < m32 ? 1u : 0u;
              r += kk[u].y < m32 ? 1u : 0u;
              r += kk[u].z < m32 ? 1u : 0u;
              r += kk[u].w < m32 ? 1u : 0u;
            }
          }
        } else {
          if (i == 0) lds[kTeamCount + 2u] += 1u;
          for (uint32_t j = 0; j < M; j += 8) {
            uint4 kk[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) kk[u] = S.get4((lmem<uint4>*)(w_key + j + 2u * u));
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
              r += (((uint64_t)kk[u].y << 32) | kk[u].x) < mine ? 1u : 0u;
              r += (((uint64_t)kk[u].w << 32) | kk[u].z) < mine ? 1u : 0u;
            }
          }
        }
        S.set4(srt + r, (uint32_t)(mine >> 32), i | ((od.w >> 3) & 1u) << 31, od.y, 0u);
      }
      lds_barrier<NW>();
      if (small) {
        if (M <= 64)
          S.template serve<1, true>(M, wbase, cw, T);
        else if (M <= 128)
          S.template serve<2, true>(M, wbase, cw, T);
        else
          S.template serve<4, true>(M, wbase, cw, T);
      } else {
        if (x == 0) lds[kTeamCount + 1u] += 1u;
        S.template serve<4, false>(M, wbase, cw, T);
      }
      // this SM's arrivals, in order
      if (S.hot) {  // its edges stay inside their CTA: only this thread pushes to its list
        S.hot_finish(p, d);
      } else {
        for (uint32_t u = 0; __ballot(u < d); ++u) {
          if (u < d) {
            const uint64_t key = w_key[p + u];
            const uint4 od = S.get4(S.optab + w_op[p + u]);
            const uint32_t c = (uint32_t)(key >> 32);
            const uint64_t e = (uint64_t)c + od.x, m = lds[kTeamMend + p + u];
            const uint64_t f = (e > m ? e : m) + od.z;
            if (f > kMaxCycle)
              S.bad |= kBadOverflow;
            else
              S.complete((uint32_t)key, c, (uint32_t)f);
          }
        }
      }
      arrivals += M;
      most = M > most ? M : most;
    }
    if (clk) {
      const uint64_t c5 = __builtin_amdgcn_s_memtime();
      ck[0] += c1 - c0;
      ck[1] += c2 - c1;
      ck[2] += c3 - c2;
      ck[3] += c4 - c3;
      ck[4] += c5 - c4;
    }
  }

  if (S.log_n) S.log_flush(S.log_n);
  // Results: per-wave sums, then the first wave's lane adds them up.
  uint64_t dg = S.digest;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) dg += __shfl_xor(dg, o, 64);
  const uint32_t mk = wave_max_u32(S.makespan);
  const uint32_t nf = wave_sum_u32(S.nfin), ni = wave_sum_u32(S.n_issued);
  const bool queue = __ballot((S.bad & kBadQueue) != 0) != 0, ovf = __ballot((S.bad & kBadOverflow) != 0) != 0;
  __syncthreads();
  lmem<uint32_t>* const fin = lds + kTeamSorted;
  if (lane == 0) {
    lmem<uint32_t>* const e = fin + S.wave * 8u;
    e[0] = (uint32_t)dg;
    e[1] = (uint32_t)(dg >> 32);
    e[2] = mk;
    e[3] = nf;
    e[4] = ni;
    e[5] = (queue ? 1u : 0u) | (ovf ? 2u : 0u);
    e[6] = steps;
  }
  __syncthreads();
  if (x == 0) {
    uint64_t dsum = 0;
    uint32_t mmax = 0, fsum = 0, isum = 0, why = 0;
    uint64_t ssum = 0;
    for (uint32_t w = 0; w < S.nw; ++w) {
      const lmem<uint32_t>* const e = fin + w * 8u;
      dsum += ((uint64_t)e[1] << 32) | e[0];
      mmax = e[2] > mmax ? e[2] : mmax;
      fsum += e[3];
      isum += e[4];
      why |= e[5];
      ssum += e[6];
    }
    uint64_t* stats = reinterpret_cast<uint64_t*>(sim + L.layout.stride - kStatsBytes);
    stats[0] = windows;
    stats[1] = ssum;  // of all waves, as the nodes issued
    stats[2] = isum;
    stats[3] = arrivals;
    stats[4] = ctl[1];
    stats[5] = most;
    for (uint32_t i = 0; i < 5; ++i) stats[6 + i] = ck[i];
    stats[11] = S.nw;  // wavefronts of the simulation
    stats[12] = why;
    for (uint32_t i = 0; i < 3; ++i) stats[13 + i] = lds[kTeamCount + i];
    int32_t st = GTS_SIM_OK;
    if (why & 1u)
      st = kStatusRetry;
    else if (why & 2u)
      st = GTS_SIM_OVERFLOW;
    else if (fsum != S.G.n_nodes)
      st = GTS_SIM_DEADLOCK;
    L.out_status[b] = st;
    L.out_makespan[b] = st == GTS_SIM_OK ? mmax : 0xFFFFFFFFu;
    if (L.out_digest) L.out_digest[b] = st == GTS_SIM_OK ? dsum : 0ull;
  }
}

}  // namespace

extern "C" __global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void gts_sim_team1(Launch L) { team_body<1>(L); }
extern "C" __global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(3))) void gts_sim_team2(Launch L) { team_body<2>(L); }
extern "C" __global__ __launch_bounds__(192) __attribute__((amdgpu_waves_per_eu(3))) void gts_sim_team3(Launch L) { team_body<3>(L); }
extern "C" __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gts_sim_team4(Launch L) { team_body<4>(L); }

hipError_t launch_team(const Launch& L, uint32_t lds_bytes, hipStream_t stream) {
  if (L.B == 0) return hipSuccess;
  const uint32_t nw = (L.max_nsm + 63) / 64;
  void (*const k[4])(Launch) = {gts_sim_team1, gts_sim_team2, gts_sim_team3, gts_sim_team4};
  hipLaunchKernelGGL(k[nw - 1u], dim3(L.B), dim3(64u * nw), lds_bytes, stream, L);
  return hipGetLastError();
}

}  // namespace gts
