// Launch planner of one layer call: split counts, tile shapes, item counts,
// workspace layout and LDS sizes, from the layer shape, the batch and the
// call's flags. Host code only (no HIP calls), so it also builds as a plain
// C++ translation unit for host-side checks.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "cardan_plan.h"

namespace cardan {

namespace {

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int ceil_div(int a, int b) { return (a + b - 1) / b; }


constexpr size_t kLdsBudget = 60 * 1024;  // operand staging limit when sizing the K splits

int ks_max(int total, int splits) { return ceil_div(total, splits); }

// Largest x/z staging of a gate/up split (uint4 per token row).
int gateup_ld(int KSX, int KSZ, int ns, int ns_v) {
  int best = 0;
  for (int s = 0; s < ns; ++s) {
    int k0, k1;
    joint_split(s, ns, ns_v, KSX, KSZ, k0, k1);
    const int x = std::min(k1, KSX) - std::min(k0, KSX);
    const int z = std::max(k1, KSX) - std::max(k0, KSX);
    best = std::max(best, (x * 4 + 1) + (z * 8 + 1));
  }
  return best;
}

size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

constexpr double kSlots = 512.0;  // nominal grid: two workgroups per CU
constexpr double kFewTiles = 400.0, kFewTiles2 = 460.0;  // see choose_splits

// Splits of the compressed gate/up tiles and of the down tiles.
//
// Gate/up: of the splits of an (expert, projection, 256 columns) into code and
// low-rank tiles whose expected number fits one round of the nominal grid, the
// one whose longest tile is shortest; one tile for the whole joint axis where
// more do not fit. A second round costs each workgroup a tile's set-up again
// (3 to 4 us of loads before the first product), which longer tiles save:
// measured per call with the splits that the bytes alone gave and with these,
// DeepSeek-V2-Lite B=8 69.4 -> 57.0 us (1 code + 2 low-rank -> 1), B=32 119.6 ->
// 83.8, Gemma-4 B=16 87.2 -> 75.2, OLMoE B=32 82.1 -> 74.2, wide B=2 42.3 -> 34.5
// (1 + 1 -> 2 + 1). kCode and kLr: microseconds per K-step of a code and a
// low-rank tile while the grid is full; kSplit: of each split's partial sums
// in the down tiles' staging.
//
// Down: tiles of about 24 code K-steps (16 at d = 2, which reads four words for
// one) and 12 low-rank ones (4 KB instead of 1 KB of weights per wave and step)
// fill many rounds evenly. While finer ones
// fit one round, the code tiles take as many splits as do, down to 7 K-steps
// (less than that is set-up), and the low-rank tiles 8 K-steps, or 4 where
// their ranks fill only two waves. Dense down tiles (16 KB per K-step) go down to
// 8 K-steps, and to 2 while they leave half of the round free (I=480, 4 of 8
// experts, B=1: one tile of 15 steps 23.1 us, fifteen 20.4).
//
// records: expected records of the routing tables (tiles of an expert's passes).
void compressed_splits(Plan& P, double exp_act, double records, double npj, int KSX, int KSZ, int KSD, int mode) {
  const double kCode = P.d == 2 ? 0.2 : 0.13, kLr = 0.6, kSplit = 0.33;
  const double t1 = exp_act * npj * P.ncg;  // tiles with one split
  P.ns_v = P.ns = 1;
  double best = kCode * KSX + kLr * KSZ + kSplit;
  // (a whole axis of less than a tile's set-up stays one tile)
  for (int nv = 1; best > 3.0 && nv <= 8 && (nv == 1 || nv * 12 <= KSX); ++nv)
    for (int nl = 0; nl <= std::min(4, KSZ); ++nl) {
      // one code and one low-rank tile may exceed the grid by 30 %, priced by
      // the second round: worth it where both parts are long (Nemotron B=8 80.5
      // -> 76.7 us, OLMoE B=8 would go 54.2 -> 58.1)
      const double n = t1 * (nv + nl);
      const bool second = n > kSlots && n <= 1.3 * kSlots && nv == 1 && nl == 1;
      if (n > kSlots && !second) continue;
      // (with no low-rank split the last code tile takes those steps too)
      const double longest = nl > 0 ? std::max(kCode * KSX / nv, kLr * KSZ / nl) : kCode * KSX / nv + kLr * KSZ;
      const double cost = longest * (second ? 1.55 : 1.0) + kSplit * (nv + nl);
      if (cost < best) {
        best = cost;
        P.ns_v = nv;
        P.ns = nv + nl;
      }
    }
  if (mode == 1) {
    P.nsd = ceil_div(KSD, kDenseDownSteps);
    auto fits = [&](int n) {
      return exp_act * P.ncgh * n <= kSlots &&
             KSD / n >= (records * P.ncgh * n <= kSlots / 2 ? 2 : kDenseDownSteps / 3);
    };
    while (P.nsd < KSD && fits(P.nsd + 1)) ++P.nsd;
    return;
  }
  P.nsd = std::max(1, (int)lround(KSD / (P.d == 2 ? 16.0 : 24.0)));
  P.nsdl = P.r > 0 ? std::max(1, (int)lround(KSD / 12.0)) : 1;
  const int nl_fine = P.r > 0 ? ceil_div(KSD, P.r > 128 ? 8 : kLrDownSteps) : 1;
  // (where one code tile per column group is enough, fewer low-rank tiles are
  // tried too before a second round, but none of more than 16 K-steps, 24 at
  // d = 8: that one tile ends the down phase. One tile and the usual two or
  // three: H=3520, I=1024, r=504, 32 experts, B=22 84.9 and 65.9 us; with d = 4
  // OLMoE B=13 to 16 67 to 71, 5 % less; H=1344, I=640, up-only, B=9 56.8 and
  // 50.6. At d = 8 and 22 K-steps the few tiles of a second round cost as much
  // or more: Gemma-4 B=5 44.0 and 46.7 over 20 routings)
  const int lr_long = P.d == 8 ? kLrDownLong8 : kLrDownLong;
  const int nl_least = P.nsd == 1 ? std::min(nl_fine, ceil_div(KSD, lr_long)) : nl_fine;
  for (int nl = nl_fine; nl >= nl_least; --nl) {
    int n = 0;
    while (KSD / (n + 1) >= 7 && exp_act * (P.ncgh * (n + 1) + P.ncgr * nl) <= kSlots) ++n;
    if (n > 0) {
      P.nsd = std::max(P.nsd, n);
      P.nsdl = nl;
      break;
    }
  }
}

// Splits by bytes, for the all-dense layer, the stacked step, F_BYTE_SPLITS and calls of few tiles: the expected
// active experts' weight bytes spread over the nominal grid, kept between 16
// and 128 KB per tile, so small batches run every tile in one round and large
// ones stream long tiles (a VQ down K-step counts double). Dense tiles grow to
// 512 KB once the nominal tile passes two of 128 KB (a tile's set-up and
// pipeline drain then recur less often; measured 154 -> 143 us for the dense
// layer at batch 16). While the items fit the grid and a quarter more, code
// splits of at most 1, 2 or 4 pipeline depths.
void byte_splits(Plan& P, double exp_act, double npj, int KSX, int KSZ, int KSD, int mode) {
  const double code_bytes = mode == 2 ? 256.0 * P.H * 2 : 256.0 * (KSX * 32 / P.d);
  const double lr_bytes = 256.0 * P.r * 2;
  const double gu_expert = mode == 2 ? npj * P.H * P.I * 2 : npj * P.H * P.I / P.d + npj * P.I * P.r * 2;
  const double dn_expert = mode >= 1 ? (double)P.I * P.H * 2 : (double)P.H * P.I / P.d + (double)P.I * P.r * 2;
  const double nominal = exp_act * (gu_expert + dn_expert) / kSlots;
  const double tile_max = (mode != 0 && nominal > 2 * 128.0 * 1024 ? 512.0 : 128.0) * 1024;
  double tile = fmin(tile_max, fmax(16.0 * 1024, nominal));
  auto splits = [&](double bytes, int max_splits) {
    return std::max(1, std::min(max_splits, (int)(bytes / tile + 0.5)));
  };
  for (;;) {
    if (tile >= 0.75 * (code_bytes + lr_bytes)) {
      P.ns_v = P.ns = 1;  // one tile holds the whole joint axis
    } else {
      P.ns_v = splits(code_bytes, KSX);
      P.ns = P.ns_v + (KSZ > 0 ? splits(lr_bytes, KSZ) : 0);
    }
    P.nsd = mode >= 1 ? splits(256.0 * P.I * 2, KSD) : splits(2.0 * 256.0 * P.I / P.d, KSD);
    P.nsdl = P.r > 0 ? splits((double)std::min(P.r, kColsPerGroup) * P.I * 2, KSD) : 1;
    const double items = exp_act * (npj * P.ncg * P.ns + P.ncgh * P.nsd + P.ncgr * P.nsdl);
    if (items <= kSlots || tile >= tile_max) break;
    tile *= 1.05;
  }
  if (P.ns > 1) {
    const int pd = mode == 2 ? kPdDenseW : kPdVq;
    const int nl_fine = KSZ > 0 ? ceil_div(KSZ, kPdDense) : 0, nl_keep = P.ns - P.ns_v;
    bool done = false;
    for (int mult = 1; mult <= 4 && !done; mult *= 2) {
      const int nv = std::max(P.ns_v, ceil_div(KSX, pd * mult));
      for (const int nl : {nl_fine, nl_keep}) {
        const double items = exp_act * (npj * P.ncg * (nv + nl) + P.ncgh * P.nsd + P.ncgr * P.nsdl);
        if (items <= 1.25 * kSlots) {
          P.ns_v = nv;
          P.ns = nv + nl;
          done = true;
          break;
        }
      }
    }
  }
  P.nsdl = std::min(P.nsdl, ceil_div(KSD, kLrDownSteps));
}

// Splits of the compressed forms: compressed_splits, but for calls of few tiles
// the finer of those and of the splits by bytes, part by part. While few
// workgroups are busy a tile's length is the call's: its set-up overlaps the
// others' and costs no round. Few: the tiles split by bytes take at most 400 of
// the 512 workgroups of a round (460 at d = 2, whose K-steps take about twice as
// long). Measured over 1295 drawn calls and calls of the models' shapes against
// compressed_splits alone: 138 more than 1.5 % faster (H=576, I=1792, d=2, r=232,
// 2 of 39 experts 25.9 -> 22.5 us; H=640, I=288, d=2, r=328, 8 of 216 29.0 -> 26.1;
// H=448, I=384, d=4, up-only, B=4 25.2 -> 22.7), six more than 1.5 % slower (2 to
// 3.6 %).
void choose_splits(Plan& P, double exp_act, double npj, int KSX, int KSZ, int KSD, int mode) {
  // an expert has a record per 8 tokens: this many more if they were all in full ones
  const double records = exp_act + std::max(0.0, P.S - exp_act) / 8.0;
  const double few = P.d == 2 ? kFewTiles2 : kFewTiles;
  compressed_splits(P, exp_act, records, npj, KSX, KSZ, KSD, mode);
  // (more tiles than that with one split each: no need to see the splits by bytes)
  if (records * (npj * P.ncg + P.ncgh + P.ncgr) > few) return;
  Plan Q = P;
  byte_splits(Q, exp_act, npj, KSX, KSZ, KSD, mode);
  const double tiles = records * (npj * P.ncg * Q.ns + P.ncgh * Q.nsd + P.ncgr * Q.nsdl);
  if (tiles > few) return;
  const int nl = std::max(P.ns - P.ns_v, Q.ns - Q.ns_v);
  P.ns_v = std::max(P.ns_v, Q.ns_v);
  P.ns = P.ns_v + nl;
  P.nsd = std::max(P.nsd, Q.nsd);
  P.nsdl = std::max(P.nsdl, Q.nsdl);
}

// Dynamic LDS of k_route for a plan.
size_t lds_route(const Plan& P) {
  const int KSX = P.H / 32;
  size_t need = (size_t)kRouterTok * kRowsRouter * 4 + (size_t)4 * kRouterTok * 64 * 8 + 16;  // router chunk
  need = std::max(need, (size_t)kMaxE * 8 + kMaxK * (8 + 8 + 4 + 4) + (size_t)kWG * 8);  // select
  need = std::max(need, (size_t)(kMaxB * kMaxK + 2 * kMaxE + 4) * 4);   // grouping
  if (P.flags & F_Z)
    need = std::max(need, (size_t)4 * kTokPass * (ks_max(KSX, P.nch_z) * 4 + 1) * 16 + kZRed + kTokPass * 4);
  return round256(need);
}

// Dynamic LDS of k_expert for a plan.
size_t lds_expert(const Plan& P) {
  const int KSX = P.H / 32, KSZ = ceil_div(P.r, 32), KSD = P.I / 32;
  size_t need = (size_t)P.nt_max * gateup_ld(KSX, KSZ, P.ns, P.ns_v) * 16;
  // down: p operand rows (of the low-rank tiles where the call has them)
  const int ksd = std::max(ks_max(KSD, P.nsd), P.ncgr > 0 ? ks_max(KSD, P.nsdl) : 0);
  need = std::max(need, (size_t)P.nt_max * (ksd * 8 + 1) * 16);
  need = std::max(need, combine_lds(P) + ((P.flags & F_CB_SPLITK) ? kSplitKRed : 0));
  // T-path gate/up tiles: the T rows of their blocks for one token
  if (P.flags & F_TBOOK) need = std::max(need, (size_t)ks_max(KSX, P.ns_v) * (32 / P.d) * P.K * 4);
  return round256(need);
}

Plan plan_once(const cardan_shape* s, int B, int z_sep, int flags) {
  Plan P;
  memset(&P, 0, sizeof P);
  P.H = s->H; P.I = s->I; P.E = s->E; P.k = s->top_k; P.d = s->d; P.K = s->K; P.r = s->r;
  P.B = B;
  P.flags = flags;
  const int mode = expert_mode(P);
  if (mode == 2) P.r = 0;
  P.S = B * P.k;
  P.max_act = P.E < P.S ? P.E : P.S;
  P.nch_r = ceil_div(P.H, kRowsRouter);
  P.n_eg = ceil_div(P.E, 64);
  P.z_sep = z_sep;
  // token rows a tile stages per pass: 8 above batch 8 (the hi and lo halves of
  // a split operand fill one MFMA's 16 rows), which also keeps the operand
  // staging small enough for the code book's lines; an expert with more tokens
  // has a record, and tiles, per pass
  P.nt_max = B > 8 ? 8 : B;
  // combine tiles of few tokens, so that the final gather is spread over more
  // workgroups: B/32 each (OLMoE B=32 1 token instead of 2: 2 us less), and up
  // to two where the low-rank gather is short (r <= 128: one token each is 1 %
  // slower there)
  P.tpc = (flags & F_BYTE_SPLITS) ? ceil_div(B, 16) : P.r > 128 ? ceil_div(B, 32) : std::min(2, ceil_div(B, 16));
  const int KSX = P.H / 32, KSZ = ceil_div(P.r, 32), KSD = P.I / 32;
  P.nch_z = std::max(1, KSX / 2);                  // two K-steps of U per z unit (one wave)
  P.nq_z = ceil_div(P.nch_z, 4);                   // four units per z item, summed in LDS
  const double exp_act = fmax(1.0, P.E * (1.0 - pow(1.0 - (double)P.k / P.E, (double)B)));
  const double npj = n_proj(P);  // gate and up, or up alone
  P.ncg = ceil_div(P.I, kColsPerGroup);
  P.ncgh = ceil_div(P.H, kColsPerGroup);
  P.ncgr = mode == 0 ? ceil_div(P.r, kColsPerGroup) : 0;  // low-rank down column groups
  P.nsdl = 1;
  // (the stacked step keeps the order of its sums: see kTwoProducts)
  const bool by_bytes = mode == 2 || (P.flags & (F_BYTE_SPLITS | F_NORM_IN | F_SSQ_OUT));
  if (by_bytes)
    byte_splits(P, exp_act, npj, KSX, KSZ, KSD, mode);
  else
    choose_splits(P, exp_act, npj, KSX, KSZ, KSD, mode);
  // routing tables: records and four per-slot arrays (here with as many records
  // as the fewest rows of a pass could make)
  P.lds_routing = round256((size_t)std::min(P.S, P.max_act + P.S / 2) * 16 + (size_t)4 * P.S * 4);
  const size_t budget = by_bytes ? kLdsBudget : std::min(kLdsBudget, kLdsMax - std::min(kLdsMax, P.lds_routing));
  // Operand staging that does not fit LDS: split the codes (up to four ways)
  // before halving the token rows of a pass (down to 4), since experts with
  // more tokens than one pass stream and decode their weights again per pass
  // (the wide layer with 8 hot experts at B = 8: 78 us in passes of 4 rows, 55
  // in two splits of 8).
  auto staging = [&]() { return (size_t)P.nt_max * gateup_ld(KSX, KSZ, P.ns, P.ns_v) * 16; };
  while (!by_bytes && P.nt_max > 4 && P.ns_v < std::min(4, KSX) && staging() > budget) {
    ++P.ns_v;
    ++P.ns;
  }
  while (P.nt_max > 4 && (size_t)P.nt_max * gateup_ld(KSX, KSZ, P.ns, P.ns_v) * 16 > budget)
    P.nt_max = (P.nt_max + 1) / 2;
  while (P.ns_v < KSX && (size_t)P.nt_max * gateup_ld(KSX, KSZ, P.ns, P.ns_v) * 16 > budget) {
    if (P.ns == P.ns_v && KSZ > 0) ++P.ns;  // give the low-rank steps their own split first
    else {
      ++P.ns_v;
      ++P.ns;
    }
  }
  // Projection code book: only for whole-layer calls on compressed weights
  // with d = 4 or 8, K % 4 == 0 (16-byte T rows) and a table of at most
  // kTBookMaxBytes, in the narrow expert kernel (no F_DN_WIDE); its code splits hold at most the
  // K-steps whose T rows fit kTBookTileBlocks blocks of 1 KB (K = 256), and
  // the low-rank steps get splits of their own (a T-path tile has no MFMA
  // accumulators to add them to)
  if ((P.flags & F_TBOOK) &&
      (mode != 0 || !(P.flags & F_ROUTE) || (P.flags & F_NORM_IN) || P.d == 2 || P.K % 4 ||
       tbook_bytes(P) > kTBookMaxBytes))
    P.flags &= ~F_TBOOK;
  if (P.flags & F_TBOOK) {
    const int bps = 32 / P.d;
    const int nbt = std::min(kTBookTileBlocks, (int)(48 * 1024 / ((size_t)P.K * 4)));
    const int ks_t = std::max(1, nbt / bps);
    const int nl = KSZ > 0 ? std::max(1, P.ns - P.ns_v) : 0;
    P.ns_v = std::min(KSX, std::max(P.ns_v, ceil_div(KSX, ks_t)));
    P.ns = P.ns_v + nl;
  }
  // (the splits by bytes leave 8 KB more free: fewer splits would change the
  // order of the stacked step's sums and the layers the scratch array takes)
  auto down_fits = [&](int n) {
    return (size_t)P.nt_max * (ks_max(KSD, n) * 8 + 1) * 16 + (by_bytes ? 8192 : 0) <= budget;
  };
  while (P.nsd < KSD && !down_fits(P.nsd)) ++P.nsd;
  while (P.ncgr > 0 && P.nsdl < KSD && !down_fits(P.nsdl)) ++P.nsdl;
  // Items for more than two rounds of the nominal grid (throughput-bound):
  // VQ down tiles over two column groups, so that each K-step's activation
  // reads serve twice the columns and the down tiles take half the
  // workgroup slots (fewer rounds, longer tiles)
  const double items_all = exp_act * (npj * P.ncg * P.ns + P.ncgh * P.nsd + P.ncgr * P.nsdl);
  if (mode == 0 && items_all > 2 * kSlots && P.ncgh > 1 && P.d == 8 && !(P.flags & F_TBOOK)) P.flags |= F_DN_WIDE;

  // Small batches at ranks above 128: B^T u streams more of B than a
  // combine tile primes before its wait, so the tiles shrink to 64 columns
  // with the ranks split over their four waves (each wave's share primed).
  if (mode == 0 && P.r > 128 && B <= 4) P.flags |= F_CB_SPLITK;
  P.n_cb = P.ncgh * ceil_div(B, P.tpc) * ((P.flags & F_CB_SPLITK) ? 4 : 1);
  // Batch 1: every gate/up tile's operands are the one token's x and z rows,
  // so each workgroup stages them once while it builds its routing tables
  if (mode == 0 && B == 1 && P.H <= 8 * kXpreXGroups) P.flags |= F_XPRE;

  // token groups of the shared projection side by side, one flag per item
  P.n_zc_flags = 2 * ceil_div(kMaxR, 64) * P.nq_z;
  const int z_group = z_items_per_group(P);
  P.n_zc = (flags & F_Z) && P.r > 0 ? z_group * std::min(ceil_div(B, kTokPass), P.n_zc_flags / z_group) : 0;
  P.n_rc = (flags & F_ROUTE) ? P.nch_r * P.n_eg * ceil_div(B, kRouterTok) : 0;
  P.n_sel = (flags & F_ROUTE) ? B : 0;
  P.n_zr = (flags & F_Z) ? ceil_div(2 * B * P.r, kWG) : 0;
  P.n_tb = (P.flags & F_TBOOK) ? B * n_proj(P) * tbook_groups(P) : 0;
  P.n_pre = P.n_rc + P.n_zc + P.n_sel + P.n_zr + P.n_tb;

  // Counters first, at offsets that depend only on H, I and E (not on B,
  // r or the expert-weight form): a call leaves its expert ticks set until
  // the next call's k_route clears them, so every call on a workspace must
  // find them at the same place.
  P.n_rc_flags = P.nch_r * P.n_eg * ceil_div(kMaxB, kRouterTok);
  size_t o = 0;
  P.o_ctr = o; o = align256(o + (size_t)C_NUM * kCtrStride * 4);
  P.o_rc_flag = o; o = align256(o + (size_t)P.n_rc_flags * kTickPad * 4);
  P.o_zc_flag = o; o = align256(o + (size_t)P.n_zc_flags * kTickPad * 4);
  P.o_gu_tick = o; o = align256(o + (size_t)P.E * ceil_div(P.I, kColsPerGroup) * kTickPad * 4);
  P.o_dn_done = o; o = align256(o + (size_t)P.E * (ceil_div(P.H, kColsPerGroup) + 1) * kTickPad * 4);
  P.o_rl = o; o = align256(o + (size_t)P.nch_r * B * P.E * 8);
  P.o_zp = o; o = align256(o + (size_t)2 * P.nq_z * B * P.r * 4);
  P.o_z = o; o = align256(o + (size_t)2 * B * P.r * 4);
  P.o_gu = o; o = align256(o + (size_t)P.S * 2 * P.ns * P.I * 4);
  P.o_dn = o; o = align256(o + (size_t)P.nsd * P.S * P.H * 4);
  P.o_uap = o; o = align256(o + (size_t)P.nsdl * P.S * P.r * 4);
  if (P.flags & F_TBOOK) o = tbook_offset(P) + tbook_bytes(P);
  P.total = o;
  P.lds_route = lds_route(P);
  // item LDS, also the grouping scratch at the start of the kernel
  const size_t group_scratch = round256((size_t)2 * P.S * 4 + (size_t)4 * P.E * 4 + 32);
  const size_t items = std::max(lds_expert(P), group_scratch) + ((P.flags & F_XPRE) ? kXpreBytes : 0);
  auto routing = [&]() { return round256((size_t)max_records(P) * 16 + (size_t)4 * P.S * 4); };
  int rs = kOneRecord;
  if (P.nt_max < B)
    for (rs = 0; 2 << rs <= P.nt_max;) ++rs;
  P.flags |= rs << kRecordShiftPos;
  P.lds_routing = routing();
  if (P.lds_routing + items > kLdsMax) {
    P.flags = (P.flags & ~(15 << kRecordShiftPos)) | kOneRecord << kRecordShiftPos;
    P.lds_routing = routing();
  }
  P.lds_expert = P.lds_routing + items;
  // the large-batch kernel only where two workgroups with at least 64-byte
  // book lines fit a CU (80 KB each)
  constexpr size_t kLdsHalf = 80 * 1024 - 512;
  if ((P.flags & F_DN_WIDE) && P.lds_expert + (256 * 16 << 2) > kLdsHalf) P.flags &= ~F_DN_WIDE;
  // the longest book lines that still let two workgroups share a CU
  if (book_in_lines(P)) {
    int bs = kBookShiftMax;
    while (bs > 0 && P.lds_expert + ((size_t)256 * 16 << bs) > kLdsHalf) --bs;
    P.flags |= bs << kBookShiftPos;
    P.lds_expert += book_bytes(P);
  }
  return P;
}

}  // namespace

// Launch plan, item counts and workspace layout; depends only on
// (shape, B, z_sep, flags). F_GU_DENSE plans take r = 0. A plan whose partial
// sums would pass the 2 GiB that offsets reach, or whose term tables the LDS
// limit, is made again with the splits by bytes.
Plan make_plan(const cardan_shape* s, int B, int z_sep, int flags) {
  const Plan P = plan_once(s, B, z_sep, flags);
  const bool fits = P.total < 0x80000000ull && P.lds_expert - book_bytes(P) <= kLdsMax;
  if (fits || (flags & F_BYTE_SPLITS)) return P;
  return plan_once(s, B, z_sep, flags | F_BYTE_SPLITS);
}

}  // namespace cardan
