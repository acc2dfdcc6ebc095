// Host-side checks of the launch planner over the supported shape domain,
// built with AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_host_planner.py. Exits nonzero (and names the shape) on the
// first broken invariant.
//
// Invariants checked for every plan:
//   - workspace regions are 256-byte aligned, ordered and large enough for
//     the call's flags and counters;
//   - counter offsets depend on (H, I, E) only, so calls of any batch, rank,
//     block length or expert-weight form can share a workspace;
//   - the gate/up splits cover the joint axis [H inputs | r ranks] exactly,
//     in order, with no empty split; down splits lie in [1, I/32];
//   - the gate/up item mapping is a bijection from positions onto
//     (active expert, gate|up, column group, split) for several grid sizes,
//     and a position takes a code split exactly when its split index is
//     below ns_v;
//   - the item LDS of the expert kernel holds the largest item that the call
//     has, and no more than that;
//   - the routing tables hold the records of every routing, a record no more
//     rows than a pass;
//   - sizes that must fit 32-bit offsets do;
//   - the layers of a stack share one layout, whichever neighbours they chain
//     to and whatever their bases.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <vector>

#include "../../paper_2609_21137_amd/csrc/cardan_plan.h"

using namespace cardan;

static int g_fail = 0;
static char g_ctx[256];

#define CHECK(c)                                                               \
  do {                                                                         \
    if (!(c)) {                                                                \
      fprintf(stderr, "FAIL %s: %s (line %d)\n", g_ctx, #c, __LINE__);         \
      if (++g_fail > 20) exit(1);                                              \
    }                                                                          \
  } while (0)

static int cdiv(int a, int b) { return (a + b - 1) / b; }

struct Counters {
  size_t rc, zc, gu, dn, rl;
};

// the first, a middle and the last layer of a stack: the step checks and lays
// out its workspace with the middle one's plan
static void check_step_layout(const cardan_shape& s, int B) {
  const int all = F_ROUTE | F_Z | F_GROUP | F_EXPERTS;
  const Plan P = make_plan(&s, B, 1, all | F_NORM_IN | F_SSQ_OUT);
  for (int z_sep = 0; z_sep < 2; ++z_sep)
    for (int chain : {(int)F_SSQ_OUT, (int)F_NORM_IN, F_NORM_IN | F_SSQ_OUT, F_NORM_IN | F_SSQ_OUT | F_PREFETCH}) {
      const Plan Q = make_plan(&s, B, z_sep, (s.r > 0 ? all : all & ~F_Z) | chain);
      snprintf(g_ctx, sizeof g_ctx, "H=%d I=%d E=%d k=%d d=%d K=%d r=%d B=%d z_sep=%d chain=%d", s.H, s.I, s.E,
               s.top_k, s.d, s.K, s.r, B, z_sep, chain);
      CHECK(Q.total == P.total && Q.o_z == P.o_z && combine_col_tiles(Q) == combine_col_tiles(P));
    }
}

// a call of few tiles has no longer tiles than the splits by bytes give
static void check_few_tiles(const cardan_shape& s, int B, int flags) {
  const Plan P = make_plan(&s, B, 0, flags), Q = make_plan(&s, B, 0, flags | F_BYTE_SPLITS);
  snprintf(g_ctx, sizeof g_ctx, "H=%d I=%d E=%d k=%d d=%d K=%d r=%d B=%d flags=%d few tiles", s.H, s.I, s.E, s.top_k,
           s.d, s.K, s.r, B, flags);
  // every selection an expert of its own, every eight a record: no more tiles than this
  const double records = P.max_act + P.S / 8.0;
  if (records * (n_proj(P) * P.ncg * Q.ns + P.ncgh * Q.nsd + P.ncgr * Q.nsdl) > 400.0) return;
  CHECK(P.ns_v >= Q.ns_v && P.ns - P.ns_v >= Q.ns - Q.ns_v && P.nsd >= Q.nsd);
  if (P.ncgr > 0) CHECK(P.nsdl >= Q.nsdl);
}

// Most records that S selections of E experts make with 1 << rs rows each: an
// expert's first selection makes one, and so do every 1 << rs after it, so with
// all experts used the rest fills records best on one of them.
static int most_records(int S, int E, int rs) {
  const int used = std::min(S, E);
  return used - 1 + (S - used + 1 + (1 << rs) - 1) / (1 << rs);
}

static void check_plan(const cardan_shape& s, int B, int z_sep, int flags, Counters* ref) {
  const Plan P = make_plan(&s, B, z_sep, flags);
  snprintf(g_ctx, sizeof g_ctx, "H=%d I=%d E=%d k=%d d=%d K=%d r=%d B=%d z_sep=%d flags=%d", s.H, s.I, s.E,
           s.top_k, s.d, s.K, s.r, B, z_sep, flags);
  const int mode = expert_mode(P);
  const int KSX = P.H / 32, KSZ = cdiv(P.r, 32), KSD = P.I / 32;
  // layout: aligned, ordered, every region large enough
  const size_t offs[] = {P.o_ctr, P.o_rc_flag, P.o_zc_flag, P.o_gu_tick, P.o_dn_done, P.o_rl,
                         P.o_zp,  P.o_z,       P.o_gu,      P.o_dn,      P.o_uap,     P.total};
  for (size_t i = 0; i < sizeof offs / sizeof offs[0]; ++i) {
    CHECK(offs[i] % 256 == 0);
    if (i) CHECK(offs[i] >= offs[i - 1]);
  }
  CHECK(P.o_rc_flag - P.o_ctr >= (size_t)C_NUM * kCtrStride * 4);
  CHECK(P.n_rc <= P.n_rc_flags && P.n_zc <= P.n_zc_flags);
  CHECK(P.o_zc_flag - P.o_rc_flag >= (size_t)P.n_rc_flags * kTickPad * 4);
  CHECK(P.o_gu_tick - P.o_zc_flag >= (size_t)P.n_zc_flags * kTickPad * 4);
  CHECK(P.o_dn_done - P.o_gu_tick >= (size_t)P.E * P.ncg * kTickPad * 4);
  CHECK(P.o_rl - P.o_dn_done >= (size_t)P.E * (P.ncgh + 1) * kTickPad * 4);
  CHECK(P.o_zp - P.o_rl >= (size_t)P.nch_r * B * P.E * 8);
  CHECK(P.o_z - P.o_zp >= (size_t)2 * P.nq_z * B * P.r * 4);
  CHECK(P.nq_z * 4 >= P.nch_z && (P.nq_z - 1) * 4 < P.nch_z);
  CHECK(P.o_gu - P.o_z >= (size_t)2 * B * P.r * 4);
  CHECK(P.o_dn - P.o_gu >= (size_t)P.S * 2 * P.ns * P.I * 4);
  CHECK(P.o_uap - P.o_dn >= (size_t)P.nsd * P.S * P.H * 4);
  CHECK(P.total - P.o_uap >= (size_t)P.nsdl * P.S * P.r * 4);
  // counter offsets shared by every call on the shape's workspace
  const Counters c = {P.o_rc_flag, P.o_zc_flag, P.o_gu_tick, P.o_dn_done, P.o_rl};
  if (ref->rc == (size_t)-1) *ref = c;
  CHECK(c.rc == ref->rc && c.zc == ref->zc && c.gu == ref->gu && c.dn == ref->dn && c.rl == ref->rl);
  // splits
  CHECK(P.ns_v >= 1 && P.ns_v <= P.ns && P.ns_v <= KSX);
  CHECK(P.ns - P.ns_v <= KSZ);
  int prev = 0;
  for (int sp = 0; sp < P.ns; ++sp) {
    int k0, k1;
    joint_split(sp, P.ns, P.ns_v, KSX, KSZ, k0, k1);
    CHECK(k0 == prev);
    CHECK(k1 > k0);
    if (sp < P.ns_v) CHECK(k0 < KSX);  // a code split starts among the code steps
    prev = k1;
  }
  CHECK(prev == KSX + KSZ);
  CHECK(P.nsd >= 1 && P.nsd <= KSD);
  if (P.r > 0 && mode == 0) CHECK(P.nsdl >= 1 && P.nsdl <= KSD);
  // no long low-rank down tile (I/32 K-steps round to tiles of about 12, so one
  // of up to 17 remains)
  if (P.ncgr > 0 && !(flags & (F_BYTE_SPLITS | F_NORM_IN | F_SSQ_OUT)) && P.total < 0x80000000ull &&
      P.lds_expert - book_bytes(P) <= kLdsMax)
    CHECK(cdiv(KSD, P.nsdl) <= (P.d == 8 ? 24 : 17));
  CHECK(P.nt_max >= 1 && P.nt_max <= kTokPass && P.nt_max <= B);
  CHECK(P.tpc >= 1 && P.tpc <= kTokPass);
  CHECK(P.max_act >= 1 && P.max_act <= P.E && P.max_act <= P.S);
  // records of the routing tables: no longer than a pass (a pass is a record
  // wherever an expert of B distinct tokens needs several and the tables fit),
  // and as many as the most that any routing of S selections makes
  const int rs = record_shift(P), nrec = max_records(P);
  if (rs != kOneRecord) {
    CHECK(1 << rs <= P.nt_max && 2 << rs > P.nt_max && P.nt_max < B);
  } else if (P.nt_max < B) {
    int pass = 0;
    while (2 << pass <= P.nt_max) ++pass;
    const size_t tables = (size_t)std::min(P.S, P.max_act + (P.S >> pass)) * 16 + (size_t)4 * P.S * 4;
    CHECK(((tables + 255) & ~(size_t)255) + (P.lds_expert - P.lds_routing - book_bytes(P)) > kLdsMax);
  }
  CHECK(P.S < 1 << kOneRecord);  // a record of kOneRecord holds every selection
  CHECK(nrec >= most_records(P.S, P.E, rs) && (nrec <= P.S));
  CHECK(P.lds_routing >= (size_t)nrec * 16 + (size_t)4 * P.S * 4);
  // packed fields: expert | records << 16 of a slot, slots and records of a scan
  CHECK(P.E < 1 << 16 && P.S < 1 << 15 && nrec < 1 << 15);
  // item LDS: operand rows of the gate/up, down and (where the call has them)
  // low-rank down tiles, the combine, the grouping scratch, T rows
  size_t rows = 0, item = combine_lds(P) + ((P.flags & F_CB_SPLITK) ? kSplitKRed : 0);
  for (int sp = 0; sp < P.ns; ++sp) {
    int k0, k1;
    joint_split(sp, P.ns, P.ns_v, KSX, KSZ, k0, k1);
    const int x = std::min(k1, KSX) - std::min(k0, KSX), z = std::max(k1, KSX) - std::max(k0, KSX);
    rows = std::max(rows, (size_t)(x * 4 + 1 + z * 8 + 1));
    if (sp < P.ns_v && (P.flags & F_TBOOK)) item = std::max(item, (size_t)x * (32 / P.d) * P.K * 4);
  }
  rows = std::max(rows, (size_t)cdiv(KSD, P.nsd) * 8 + 1);
  if (P.ncgr > 0) rows = std::max(rows, (size_t)cdiv(KSD, P.nsdl) * 8 + 1);
  item = std::max({item, rows * P.nt_max * 16, (size_t)8 * P.S + 16 * P.E + 32});
  // book lines in dynamic LDS where the kernel that the plan runs reads lines
  const bool xpre_kernel = (P.flags & F_XPRE) && !(P.flags & F_DN_WIDE);
  CHECK(book_bytes(P) == (mode == 2 || P.d == 4 || xpre_kernel ? 0 : 4096 << book_shift(P)) &&
        book_shift(P) <= kBookShiftMax);
  const size_t fixed = P.lds_routing + book_bytes(P) + ((P.flags & F_XPRE) ? kXpreBytes : 0);
  CHECK(P.lds_expert >= fixed + item && P.lds_expert < fixed + item + 256);
  if (P.flags & F_XPRE) CHECK(B == 1 && mode == 0 && P.H <= 8 * kXpreXGroups);
  if (P.flags & F_DN_WIDE) CHECK(mode == 0 && P.d == 8);
  // projection code book: code splits whose T rows fit the tile's LDS area,
  // low-rank steps in splits of their own, the table last in the workspace
  if (P.flags & F_TBOOK) {
    const int bps = 32 / P.d;
    CHECK(mode == 0 && P.K % 4 == 0 && (P.flags & F_ROUTE) && !(P.flags & F_NORM_IN));
    CHECK(P.d != 2 && !(P.flags & F_DN_WIDE));
    CHECK(tbook_offset(P) >= P.o_uap + (size_t)P.nsdl * P.S * P.r * 4);
    CHECK(P.total == tbook_offset(P) + tbook_bytes(P) && tbook_bytes(P) <= kTBookMaxBytes);
    CHECK(P.n_tb == B * n_proj(P) * tbook_groups(P));
    CHECK(P.n_pre == P.n_rc + P.n_zc + P.n_sel + P.n_zr + P.n_tb);
    for (int sp = 0; sp < P.ns_v; ++sp) {
      int k0, k1;
      joint_split(sp, P.ns, P.ns_v, KSX, KSZ, k0, k1);
      CHECK(k1 <= KSX && (k1 - k0) * bps <= kTBookTileBlocks);
      CHECK((size_t)(k1 - k0) * bps * P.K * 4 <=
            P.lds_expert - P.lds_routing - book_bytes(P) - ((P.flags & F_XPRE) ? kXpreBytes : 0));
    }
  } else {
    CHECK(P.n_tb == 0);
  }
  // item counts fit the kernels' int arithmetic
  const double items = (double)nrec * (gateup_tiles_per_expert(P) + down_tiles_per_expert(P)) + P.n_cb;
  CHECK(items < 2.0e9);
  // gate/up item mapping: a bijection for several grids and record counts
  const int n_tiles = gateup_tiles_per_expert(P);
  const int nacts[] = {1, nrec, P.max_act, (P.max_act + 1) / 2};
  const int grids[] = {1, 2, 7, 256, 512, 1024};
  std::vector<unsigned char> seen;
  for (int nact : nacts) {
    for (int G : grids) {
      const int n = nact * n_tiles;
      if (n > 200000) continue;
      seen.assign(n, 0);
      for (int p = 0; p < n; ++p) {
        const GateUpTile t = gateup_at(P, p, nact, P.ns_v, G);
        const bool ok = t.a >= 0 && t.a < nact && (t.pj == 0 || t.pj == 1) && t.cg >= 0 && t.cg < P.ncg &&
                        t.s >= 0 && t.s < P.ns && (t.pj == 1 || !(P.flags & F_UP_RELU2));
        CHECK(ok);
        if (!ok) continue;
        const int np = n_proj(P), id = ((t.a * np + (np == 2 ? t.pj : 0)) * P.ncg + t.cg) * P.ns + t.s;
        CHECK(!seen[id]);
        seen[id] = 1;
      }
    }
  }
}

int main(int argc, char** argv) {
  const int n_random = argc > 1 ? atoi(argv[1]) : 400;
  std::mt19937 rng(12345);
  auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + rng() % v.size()); };
  long plans = 0;
  // named shapes of the workloads, then random shapes over the domain
  std::vector<cardan_shape> shapes = {
      {256, 128, 8, 2, 4, 16, 8},      {2048, 768, 128, 8, 8, 256, 128}, {4096, 1536, 64, 6, 8, 256, 256},
      {2048, 1408, 64, 6, 8, 256, 384}, {2048, 1024, 64, 8, 4, 256, 256}, {2816, 704, 128, 8, 8, 256, 384},
      {2688, 1856, 128, 6, 8, 256, 128}, {2688, 1856, 128, 6, 8, 256, 512}, {64, 32, 1, 1, 2, 1, 0},        {8192, 4096, 1024, 32, 8, 256, 512}};
  for (int i = 0; i < n_random; ++i) {
    cardan_shape s;
    s.d = pick({2, 4, 8});
    s.H = 64 * (1 + rng() % 96);
    s.I = 32 * (1 + rng() % 96);
    s.E = pick({1, 2, 8, 60, 64, 128, 256, 300, 1024});
    s.top_k = 1 + rng() % (s.E < 32 ? s.E : 32);
    s.K = pick({1, 2, 16, 255, 256});
    s.r = 8 * (rng() % 65);
    shapes.push_back(s);
  }
  for (const cardan_shape& s : shapes) {
    Counters ref = {(size_t)-1, 0, 0, 0, 0};
    const int all = F_ROUTE | F_Z | F_GROUP | F_EXPERTS;
    const int batches[] = {1, 2, 3, 4, 8, 9, 15, 16, 17, 32, 63, 64};
    for (int B : batches) {
      for (int z_sep = 0; z_sep < 2; ++z_sep) {
        check_plan(s, B, z_sep, all | (s.r > 0 ? 0 : 0), &ref);
        ++plans;
      }
      check_plan(s, B, 0, F_ROUTE | F_GROUP | F_EXPERTS | F_DN_DENSE | F_Z, &ref);
      check_plan(s, B, 0, F_ROUTE | F_GROUP | F_EXPERTS | F_DN_DENSE | F_GU_DENSE, &ref);
      check_plan(s, B, 1, F_ROUTE, &ref);
      check_plan(s, B, 1, F_Z, &ref);
      check_plan(s, B, 1, F_GROUP | F_EXPERTS, &ref);
      // up-only squared-ReLU experts, compressed and dense
      check_plan(s, B, 0, all | F_UP_RELU2, &ref);
      check_plan(s, B, 0, F_ROUTE | F_GROUP | F_EXPERTS | F_DN_DENSE | F_GU_DENSE | F_UP_RELU2, &ref);
      // projection-code-book gate/up tiles (gated and up-only)
      check_plan(s, B, 0, all | F_TBOOK, &ref);
      check_plan(s, B, 1, all | F_TBOOK | F_UP_RELU2, &ref);
      // the scratch array's layout, and the layers of a stack (its first, a middle
      // and its last, gated with compressed weights)
      for (int more : {(int)F_BYTE_SPLITS, F_BYTE_SPLITS | F_UP_RELU2, (int)F_SSQ_OUT, F_NORM_IN | F_SSQ_OUT,
                       (int)F_NORM_IN}) {
        check_plan(s, B, 1, all | more, &ref);
        ++plans;
      }
      check_step_layout(s, B);
      for (int act : {0, (int)F_UP_RELU2}) check_few_tiles(s, B, all | act);
      check_few_tiles(s, B, all | F_DN_DENSE);
      plans += 9;
    }
  }
  // a layer that a GPU test takes for its book lines of 64 bytes
  for (int d : {2, 8}) {
    const cardan_shape s = {2432, 288, 100, 8, d, 256, 256};
    snprintf(g_ctx, sizeof g_ctx, "H=2432 I=288 E=100 k=8 d=%d r=256 B=16", d);
    CHECK(book_shift(make_plan(&s, 16, 0, F_ROUTE | F_Z | F_GROUP | F_EXPERTS)) == 2);
  }
  {  // and one for its tiles of two column groups at batch 1
    const cardan_shape s = {3968, 32, 32, 32, 8, 256, 256};
    snprintf(g_ctx, sizeof g_ctx, "H=3968 I=32 E=32 k=32 d=8 r=256 B=1");
    const Plan P = make_plan(&s, 1, 0, F_ROUTE | F_Z | F_GROUP | F_EXPERTS);
    CHECK((P.flags & F_DN_WIDE) && (P.flags & F_XPRE));
  }
  // layers that GPU tests take for the tiles of two column groups of a large
  // batch, for a stack's passes of four rows, and for their LDS
  const int all = F_ROUTE | F_Z | F_GROUP | F_EXPERTS;
  for (int relu2 = 0; relu2 < 2; ++relu2)
    for (int H : {512, 576}) {
      const cardan_shape s = {H, relu2 ? 1280 : 1024, 96, 8, 8, 256, relu2 ? 136 : 24};
      snprintf(g_ctx, sizeof g_ctx, "H=%d I=%d E=96 k=8 d=8 r=%d B=64", s.H, s.I, s.r);
      const Plan P = make_plan(&s, 64, 0, all | (relu2 ? F_UP_RELU2 : 0));
      CHECK((P.flags & F_DN_WIDE) && record_shift(P) == 3);
    }
  {
    const cardan_shape s = {4416, 32, 300, 2, 8, 256, 80};
    snprintf(g_ctx, sizeof g_ctx, "H=4416 I=32 E=300 k=2 d=8 r=80 B=16");
    for (int chain : {(int)F_SSQ_OUT, (int)F_NORM_IN}) CHECK(record_shift(make_plan(&s, 16, 0, all | chain)) == 2);
  }
  const cardan_shape near[] = {{64, 672, 64, 32, 4, 256, 424}, {64, 1152, 64, 16, 2, 256, 512}, {1536, 416, 64, 29, 8, 256, 504}};
  for (const cardan_shape& s : near) {
    snprintf(g_ctx, sizeof g_ctx, "H=%d I=%d E=64 k=%d d=%d r=%d B=64", s.H, s.I, s.top_k, s.d, s.r);
    const Plan P = make_plan(&s, 64, 0, all);
    CHECK(P.lds_expert >= 76 * 1024 && P.lds_expert - book_bytes(P) <= kLdsMax);
  }
  printf("%ld plans checked, %d failures\n", plans, g_fail);
  return g_fail ? 1 : 0;
}
