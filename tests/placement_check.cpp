// Host check of the persistent kernels' workgroup placement (wr_layout.h):
// for every plan shape and each of the 64 candidates (heads on XCD hx, units
// on XCD ux, or spread over all when ux == hx), every head, mirror and unit
// role is taken by exactly one block of the grid, heads and then mirrors sit
// on blocks 8 i + hx, units only on admitted XCDs, the last block of the grid
// is busy (the grid is no larger than needed) and the default candidate 0 is
// the original dealing (lead i at block 8 i, units on the remaining blocks in
// order).
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "wr_layout.h"

static int check(const char* what, PersistPlan P) {
  int bad = 0;
  for (int i = 0; i < 64; ++i) {
    const int hx = i / 8, ux = i % 8, uxm = ux == hx ? 255 : 1 << ux;
    wr_place(&P, hx, uxm);
    const int NL = P.NH + P.NM;   // heads, then mirrors
    std::vector<int> seen(NL + P.NU, 0);
    for (int b = 0; b < P.grid; ++b) {
      const int r = wr_role(P, b);
      if (r < 0) continue;
      if (r >= NL + P.NU) { ++bad; continue; }
      ++seen[r];
      if (r < NL && (b % 8 != hx || b / 8 != r)) ++bad;
      if (r >= NL && (!(uxm >> (b % 8) & 1) || (b % 8 == hx && b / 8 < NL))) ++bad;
      if (i == 0 && r >= NL) {   // original dealing: unit k at block k + leads below it
        const int before = (b + 7) / 8 < NL ? (b + 7) / 8 : NL;
        if (r - NL != b - before) ++bad;
      }
    }
    for (int r = 0; r < NL + P.NU; ++r) bad += seen[r] != 1;
    if (wr_role(P, P.grid - 1) < 0) ++bad;
  }
  if (bad) printf("%s: %d violations\n", what, bad);
  return bad;
}

// A launch's workgroups per XCD are the roles its blocks take, at every candidate
// placement and moved by any number of XCDs; moved, heads and units go along.
static int check_load(const char* what, PersistPlan P) {
  int bad = 0;
  for (int i = 0; i < 64; ++i)
    for (int rot = 0; rot < 8; ++rot) {
      const int hx = i / 8, ux = i % 8;
      wr_place_rot(&P, hx, ux == hx ? 255 : 1 << ux, rot);
      const XcdLoad l = wr_load(P);
      int n[8] = {};
      for (int b = 0; b < wr_rows(P.grid); ++b) n[b % 8] += wr_role(P, b) >= 0;   // (a grid is whole rows)
      for (int x = 0; x < 8; ++x) bad += n[x] != l.n[x];
      bad += P.hx != (hx + rot) % 8 || (ux != hx && P.uxm != 1 << (ux + rot) % 8);
    }
  if (bad) printf("%s: %d wrong loads\n", what, bad);
  return bad;
}

// Launches of separate models at their default placements and moved (32 CUs an
// XCD, one workgroup a CU), as a call beside others in flight is placed.
static int check_beside() {
  PersistPlan D, F;
  BatchPlan B;
  if (!persist_plan(896, &D) || !fused_plan(896, &F)) return 1;
  auto dense = [&](int rot) { wr_place_rot(&D, 0, 255, rot); return wr_load(D); };
  auto fused = [&](int rot) { wr_place_rot(&F, 0, 1, rot); return wr_load(F); };
  auto score = [&](int G) { return [G](int rot) { return wr_load(G, 896 / 32, rot); }; };
  XcdLoad held = {};
  auto add = [&](auto&& load, int expect) {   // the first placement that fits, -1: none
    int r = 0;
    for (; r < 8; ++r) {
      XcdLoad s = held;
      wr_load_add(&s, load(r));
      if (wr_load_fits(s, 32)) break;
    }
    if (r < 8) wr_load_add(&held, load(r));
    return (r < 8 ? r : -1) != expect;
  };
  int bad = 0;
  for (int i = 0; i < 8; ++i) bad += add(fused, i);      // eight fused models, an XCD each
  bad += add(fused, -1);
  held = {};
  bad += add(dense, 0);
  bad += add(score(1), 1);                               // one scored utterance beside a dense call
  bad += add(fused, 2);                                  // and a fused call
  held = {};
  bad += add(score(3), 0) + add(score(4), 3) + add(score(2), -1) + add(score(1), 7);
  held = {};
  for (int G = 1; G <= 8; ++G) {                         // the groups of a batched launch, its blocks moved with it
    if (!batch_plan(896, G * 8, &B)) return 1;
    for (int rot = 0; rot < 8; ++rot) {
      B.rot = rot;
      int n[8] = {}, g = 0;
      std::vector<int> seen(B.G * (B.NH + B.NU), 0);
      for (int b = 0; b < B.grid; ++b) {
        const int r = wr_batch_role(B, b, &g);
        if (r < 0) continue;
        ++n[b % 8];
        ++seen[g * (B.NH + B.NU) + r];
        bad += b % 8 != (g + rot) % 8;
      }
      for (int s : seen) bad += s != 1;
      const XcdLoad l = wr_load(B.G, B.NH + B.NU, rot);
      for (int x = 0; x < 8; ++x) bad += n[x] != l.n[x];
    }
  }
  if (bad) printf("beside: %d violations\n", bad);
  return bad;
}

// Side-by-side launches of a dense plan (n = 2 .. 4 utterances, launch i's
// heads and mirrors on XCD 8 i / n, units spread, as the library places them):
// every XCD of 32 CUs holds the busy blocks of all n grids.
static int check_fan(PersistPlan P) {
  int bad = 0;
  for (int n = 2; n <= 4; ++n) {
    int busy[8] = {};
    for (int i = 0; i < n; ++i) {
      wr_place(&P, 8 * i / n, 255);
      for (int b = 0; b < P.grid; ++b)
        if (wr_role(P, b) >= 0) ++busy[b % 8];
    }
    for (int x = 0; x < 8; ++x)
      if (busy[x] > 32) {
        printf("H=%d: %d launches put %d workgroups on XCD %d\n", P.H, n, busy[x], x);
        ++bad;
      }
  }
  return bad;
}

int main() {
  int bad = 0, plans = 0;
  PersistPlan P;
  for (int H = 128; H <= 896; H += 128) {
    if (persist_plan(H, &P)) {
      if (P.NM != P.NH || P.NM * WR_MTILES != P.NCT) ++bad;   // the mirrors cover every coarse row tile
      bad += check("dense", P) + check_load("dense", P);
      bad += check_fan(P);
      ++plans;
    }
    if (fused_plan(H, &P)) { bad += check("fused", P) + check_load("fused", P); ++plans; }
  }
  for (int H : {256, 512, 1024, 2048})
    for (int SR : {16, 32, 64, 128})
      for (int bh : {4, 16})
        if (sparse_plan(H, SR, bh, bh == 4 ? 4 : 1, 8, 8, &P)) { bad += check("sparse", P) + check_load("sparse", P); ++plans; }
  bad += check_beside();
  printf("%d plans, %d violations\n", plans, bad);
  return bad != 0 || plans < 20;
}
