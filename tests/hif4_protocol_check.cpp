// Host-side check of the HiF4 GEMM's LDS stage protocol, for every configuration the kernel
// instantiates (RESQ_HIF4_CONFIGS, one and two activation terms), with the kernel's own geometry
// and copy assignment (gemm_hif4_geo.h) and a model of its half-step loop:
// limits; every LDS byte a wave reads is written by exactly one copy of the same K step, from
// the source byte the reader takes it for (or zeros past the edge); and, for every K-step count
// up to a few unrolls, each read finds its stage complete and published by a barrier, and no
// buffer is refilled before a barrier that follows its last read.
//
// Usage: hif4_protocol_check [plant]; plant = 1 waits for one copy too few, plant = 2 refills a
// stage before the barrier, plant = 3 moves a padding copy onto an A fragment: each must be
// reported.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "gemm_hif4_geo.h"

using namespace resq;

static int g_plant = 0;
static int g_errors = 0;

#define FAIL(...)                   \
  do {                              \
    if (g_errors < 20) {            \
      std::printf("  FAIL: ");      \
      std::printf(__VA_ARGS__);     \
      std::printf("\n");            \
    }                               \
    ++g_errors;                     \
  } while (0)

// Source of an LDS byte: buffer (0 none, 1 A, 2 B, 3 zero) and byte offset.
struct Src {
  int buf = 0;
  int64_t off = 0;
  bool operator==(const Src& o) const { return buf == o.buf && (buf == 3 || off == o.off); }
};

template <class G>
void check_dataflow(const char* name, bool edge) {
  SlotArgs a{};
  a.a_frag0 = 0;
  a.a_frag1 = 1u << 24;
  a.a_sc0 = 1u << 26;
  a.a_sc1 = (1u << 26) + (1u << 22);
  a.b_frag_off = 0;
  a.b_sc_off = 1u << 26;
  a.T0 = 8;
  a.N0 = 16;
  a.nkb = 40;
  a.mt = edge ? a.T0 + 1 : 1u << 20;  // edge: only the first row and column tile exist
  a.nt = edge ? a.N0 + 1 : 1u << 20;
  std::vector<Src> lds(G::STAGE);
  std::vector<int> writes(G::STAGE, 0);
  auto put = [&](const HiSlot& c, int lane, int bytes, const char* cls) {
    if (c.lds == (uint32_t)G::DUMP_OFF && c.voff == kBad) {  // a padding copy
      if (G::DUMP_OFF + bytes * 64 > G::STAGE) FAIL("%s %s: padding copy overruns the dump area", name, cls);
      return;
    }
    if (c.voff != kBad && c.voff % 4) FAIL("%s %s: source offset %u is not dword aligned", name, cls, c.voff);
    for (int b = 0; b < bytes; ++b) {
      const int64_t at = (int64_t)c.lds + bytes * lane + b;
      if (at >= G::DUMP_OFF) {
        FAIL("%s %s: copy writes LDS byte %lld outside the K-step images", name, cls, (long long)at);
        return;
      }
      if (at / G::BLK != c.kk) FAIL("%s %s: copy of K step %u writes the image of another", name, cls, c.kk);
      ++writes[at];
      lds[at] = c.voff == kBad ? Src{3, 0} : Src{c.is_a ? 1 : 2, (int64_t)c.voff + b};
    }
  };
  for (int w = 0; w < G::W; ++w)
    for (int x = 0; x < G::JW; ++x) {
      const bool f = x < G::XF;
      const HiSlot c0 = f ? hi_slot_f<G>(w, x, 0, a) : hi_slot_s<G>(w, x - G::XF, 0, a);
      for (int lane = 0; lane < 64; ++lane) {
        HiSlot c = f ? hi_slot_f<G>(w, x, lane, a) : hi_slot_s<G>(w, x - G::XF, lane, a);
        if (c.is_a != c0.is_a || c.lds != c0.lds || c.kk != c0.kk)
          FAIL("%s: wave %d copy %d is not wave-uniform", name, w, x);
        if (g_plant == 3 && w == G::W - 1 && x == G::JW - 1 && c.lds == (uint32_t)G::DUMP_OFF) {
          c.lds = 0;  // planted: a padding copy lands on the first A fragment
          c.voff = c.kk = 0;
        }
        put(c, lane, f ? 16 : 4, f ? "fragment" : "scale");
      }
    }
  for (int i = 0; i < G::DUMP_OFF; ++i)
    if (writes[i] > 1) {
      FAIL("%s: LDS byte %d written by %d copies", name, i, writes[i]);
      break;
    }
  // every wave's reads (the kernel's read_a / read_b: same addresses)
  for (int wave = 0; wave < G::W; ++wave) {
    const int kg = wave / G::WT, wt = wave % G::WT, wm = wt % G::WM, wn = wt / G::WM;
    const int64_t base = (int64_t)kg * G::BLK;
    for (int lane = 0; lane < 64; ++lane) {
      auto expect = [&](int64_t at, int bytes, Src want, const char* what) {
        for (int b = 0; b < bytes; ++b, ++at, ++want.off) {
          if (writes[at] != 1) FAIL("%s: %s reads LDS byte %lld that no copy writes", name, what, (long long)at);
          else if (!(lds[at] == want))
            FAIL("%s: %s reads LDS byte %lld holding source (%d, %lld), expected (%d, %lld)", name, what,
                 (long long)at, lds[at].buf, (long long)lds[at].off, want.buf, (long long)want.off);
          else continue;
          return;
        }
      };
      // the pieces of a fragment at LDS byte f and source byte s
      auto fragment = [&](int64_t f, int64_t s, int buf, bool lo, const char* what) {
        const int64_t o[3] = {lane * 16, kHiTail + lane * 8, kHiLo + lane * 16};
        for (int q = 0; q < (lo ? 3 : 2); ++q) expect(f + o[q], q == 1 ? 8 : 16, Src{buf, buf == 3 ? 0 : s + o[q]}, what);
      };
      for (int j = 0; j < G::TN; ++j) {
        const int lj = wn * G::TN + j;
        const bool in = a.N0 + lj < a.nt;
        const int64_t rec = (int64_t)(a.N0 + lj) * a.nkb + kg;
        fragment(base + G::B_OFF + lj * kHiBFrag, a.b_frag_off + rec * kHiBFrag, in ? 2 : 3, false, "B fragment");
        expect(base + G::SB_OFF + lj * 64 + lane, 1, in ? Src{2, a.b_sc_off + rec * 64 + lane} : Src{3, 0}, "B scale");
      }
      for (int t = 0; t < G::NT; ++t)
        for (int i = 0; i < G::TM; ++i) {
          const int li = wm * G::TM + i;
          const bool in = a.T0 + li < a.mt;
          const int64_t rec = (int64_t)(a.T0 + li) * a.nkb + kg;
          fragment(base + (t * G::MTW + li) * kHiAFrag, a.frag_a(t) + rec * kHiAFrag, in ? 1 : 3, true, "A fragment");
          expect(base + G::SA_OFF + (t * G::SAJ * 4 + li) * 64 + lane, 1,
                 in ? Src{1, a.scale_a(t) + rec * 64 + lane} : Src{3, 0}, "A scale");
        }
    }
  }
}

// Event model of the loop: read = all operands that half step (k, i) loads.
enum Ev { kIssue, kWait, kBarrier, kRead };
struct Event {
  Ev e;
  int a, b;  // issue: buffer, stage; wait: N; read: buffer, stage
};

template <class G>
std::vector<Event> schedule(int nsteps) {
  constexpr int NS = G::NS;
  std::vector<Event> ev;
  const int wait_n = (NS - 2) * G::JW + (g_plant == 1 ? 1 : 0);
  for (int s = 0; s < NS; ++s) ev.push_back({kIssue, s, s});
  ev.push_back({kWait, (NS - 1) * G::JW, 0});
  ev.push_back({kBarrier, 0, 0});
  ev.push_back({kRead, 0, 0});
  for (int k0 = 0; k0 < nsteps; k0 += G::U)
    for (int u = 0; u < G::U; ++u)
      for (int i = 0; i < G::TM; ++i) {
        const int k = k0 + u;
        if (i < G::TM - 1) {
          ev.push_back({kRead, u % NS, k});
          continue;
        }
        ev.push_back({kWait, wait_n, 0});
        if (g_plant == 2) ev.push_back({kIssue, u % NS, k + NS});
        ev.push_back({kBarrier, 0, 0});
        if (g_plant != 2) ev.push_back({kIssue, u % NS, k + NS});
        ev.push_back({kRead, (u + 1) % NS, k + 1});
      }
  ev.push_back({kWait, 0, 0});
  ev.push_back({kBarrier, 0, 0});
  return ev;
}

template <class G>
void check_schedule(const char* name) {
  constexpr int NS = G::NS, JW = G::JW, U = G::U;
  for (int nsteps = 1; nsteps <= 3 * U + 2; ++nsteps) {
    const auto ev = schedule<G>(nsteps);
    std::vector<int> issued;              // stage of each copy, in issue order (JW per issue)
    int completed = 0;                    // copies known complete (a prefix)
    int visible_below = 0;                // copies complete before the last barrier
    std::vector<int> content(NS, -1);     // stage last issued into each buffer
    std::vector<int> last_read(NS, -1);   // event index of the last read of each buffer
    int last_barrier = -1;
    std::vector<int> stage_end;           // copy count after each stage's issue
    auto stage_done_by = [&](int stage, int copies) {
      return stage < (int)stage_end.size() && stage_end[stage] <= copies;
    };
    for (int i = 0; i < (int)ev.size(); ++i) {
      const Event& e = ev[i];
      if (e.e == kIssue) {
        if (last_read[e.a] > last_barrier)
          FAIL("%s nsteps %d: stage %d is copied into buffer %d before every wave is done reading it", name,
               nsteps, e.b, e.a);
        if (e.b != (int)stage_end.size()) FAIL("%s: stages issued out of order", name);
        for (int c = 0; c < JW; ++c) issued.push_back(e.b);
        stage_end.push_back((int)issued.size());
        content[e.a] = e.b;
      } else if (e.e == kWait) {
        if (e.a < 0 || e.a >= 64) FAIL("%s: vmcnt(%d) outside the 6-bit field", name, e.a);
        const int done = (int)issued.size() - e.a;
        if (done > completed) completed = done;
      } else if (e.e == kBarrier) {
        last_barrier = i;
        visible_below = completed;  // every wave has completed this many of its copies
      } else {
        if (content[e.a] != e.b)
          FAIL("%s nsteps %d: step %d reads buffer %d, which holds stage %d", name, nsteps, e.b, e.a, content[e.a]);
        else if (!stage_done_by(e.b, visible_below))
          FAIL("%s nsteps %d: step %d reads stage %d before every wave's copies of it are complete and a "
               "barrier has followed", name, nsteps, e.b, e.b);
        last_read[e.a] = i;
      }
      if (g_errors > 20) return;
    }
    if (completed != (int)issued.size()) FAIL("%s: copies still outstanding at the end", name);
  }
}

template <class G>
void check_config(const char* name) {
  if (G::LDS > 160 * 1024) FAIL("%s: LDS %zu bytes > 160 KB", name, (size_t)G::LDS);
  if ((G::NS - 1) * G::JW >= 64) FAIL("%s: vmcnt wait %d beyond the 6-bit field", name, (G::NS - 1) * G::JW);
  check_dataflow<G>(name, false);
  check_dataflow<G>(name, true);
  check_schedule<G>(name);
}

int main(int argc, char** argv) {
  g_plant = argc > 1 ? std::atoi(argv[1]) : 0;
  int configs = 0;
#define RESQ_CHECK(C, WM, WN, TM, TN, NS, KG)                                                             \
  for (int nt = 1; nt <= 2; ++nt) {                                                                       \
    char name[128];                                                                                       \
    std::snprintf(name, sizeof(name), "cfg %d %dx%d waves, %dx%d tiles, NS %d, KG %d, %d term(s)",        \
                  C, WM, WN, TM, TN, NS, KG, nt);                                                         \
    const int before = g_errors;                                                                          \
    if (nt == 1) check_config<HiGeo<WM, WN, TM, TN, 1, NS, KG>>(name);                                    \
    else check_config<HiGeo<WM, WN, TM, TN, 2, NS, KG>>(name);                                            \
    std::printf("%s %s\n", g_errors == before ? "ok  " : "FAIL", name);                                   \
    ++configs;                                                                                            \
  }
  RESQ_HIF4_CONFIGS(RESQ_CHECK)
#undef RESQ_CHECK
  std::printf("%d configurations, %d errors\n", configs, g_errors);
  return g_errors == 0 ? 0 : 1;
}
