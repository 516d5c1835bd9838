#include <cstdio>
#include <algorithm>
struct JointTab { int w[32]; };
constexpr int kMaxBodies=16,kMaxJoints=16,kMaxBodyJoints=8,kPairCap=96,kPairWords=6,kRecWords=12,kThreads=512,kThreadsWide=768,kMip=4,kPatch=28,kPatchBlocks=7;
namespace old {
constexpr int kVS = 7, kCS = 7, kJS = 13;
constexpr int kPairHitMin = 256;   // (gap, key) words a workgroup keeps at least

struct LdsPlan {
  int pos, vel, iw, nb, tq, push, outj, outc, tjs, rec, list, surv, lam, u, obs, lim, count, patch, mip, porg, org, tslot, tbody, tin, tjoint, total;
  int pq, po, pnear, pbs, pcount, pbcnt, pblist;  // capsule-capsule contacts (only with pairs != 0)
  int phit, hit_cap;                              // their (gap, key) words: offset (64-bit aligned) and capacity
  int wj, wc;                                     // kept impulses of joints and slots (only with warm != 0)
  int nu, nred, nsum;                             // Newton solver: body vectors, reduction entries, partial sums
};

// pairs: 0 = no capsule-capsule contacts, else the interaction group size (1 = self-collision only)
 inline LdsPlan make_plan(int B, int J, int S, int D, int F, int E, int with_patch, int pairs = 0,
                                             int threads = kThreads, int warm = 0, int newton = 0) {
  LdsPlan p;
  int o = 0;
  p.pos = o; o += B * 7 * E;
  p.vel = o; o += B * kVS * E;
  p.iw = o; o += B * kVS * E;
  p.nb = o; o += B * E;
  p.tq = o; o += J * 3 * E;
  p.push = o; o += 3 * E;
  o += o & 1;  // the search results kept in the copy arrays are 64-bit words
  p.outj = o; o += J * kJS * E;
  p.outc = o; o += S * kCS * E;
  p.rec = o; o += S * kRecWords * E;
  p.list = o; o += S * E;
  p.surv = o; o += S * E;
  p.lam = o;   // (with the warm start these impulses live in the per-slot array below)
  o += warm ? 0 : 3 * (S * E > threads - ((2 * J * E + 63) / 64) * 64 ? S * E - (threads - ((2 * J * E + 63) / 64) * 64) : 0);
  p.u = o; o += (D > 0 ? D : 1) * E;
  p.obs = o; o += (11 + 3 * D + F) * E;
  p.lim = o; o += (D > 0 ? D : 1) * E;
  p.count = o; o += 8;
  p.porg = o; o += 2 * E;
  p.org = o; o += 3 * E;
  p.tjs = o; o += B * (kMaxBodyJoints + 3);  // tjs .. tjoint: one block, copied from Model::table_image
  p.tslot = o; o += 2 * S;
  p.tbody = o; o += 4 * B;
  p.tin = o; o += 6 * B;
  p.tjoint = o; o += J * (int)(sizeof(JointTab) / 4);
  p.patch = o; o += with_patch ? E * kPatch * kPatch : 0;
  p.mip = o; o += with_patch ? E * kPatchBlocks * kPatchBlocks : 0;
  p.pq = o; o += pairs ? kPairCap * kPairWords : 0;   // sorted queue of the substep's contacts
  p.po = o; o += pairs ? (kPairCap + 1) * 12 : 0;     // weighted velocity copies of their two bodies; the last entry stays zero
  p.pnear = o; o += pairs ? (E * pairs) / 2 + 1 : 0;  // agent pairs whose bounding spheres overlap
  p.pbs = o; o += pairs ? E : 0;                      // bounding radius of every agent about its root
  p.pcount = o; o += pairs ? 4 : 0;
  p.pbcnt = o; o += pairs ? B * E : 0;                  // per body: how many of them touch it
  p.pblist = o; o += pairs ? (B * E * 6 + 3) / 4 : 0;  // per body: up to six of them, one byte each
  // one 64-bit (gap, key) word per capsule-capsule contact found, for the choice of those that stay
  // when a workgroup finds more than it holds: in the space of the terrain search's candidate list
  // (idle by then) where that holds kPairHitMin words, else in a region of their own
  p.hit_cap = ((J * kJS + S * kCS) * E - 5 * S * E - 2) / 2;
  p.phit = p.outj + ((5 * S * E + 1) & ~1);
  if (pairs && p.hit_cap < kPairHitMin) {
    o += o & 1;
    p.phit = o; o += 2 * kPairHitMin;
    p.hit_cap = kPairHitMin;
  }
  p.wj = o; o += warm ? J * 6 * E : 0;
  p.wc = o; o += warm ? S * 3 * E : 0;
  p.nu = o; o += newton ? B * kVS * E : 0;
  p.nred = o; o += newton ? 3 * (J + S) * E : 0;
  p.nsum = o; o += newton ? 3 * 8 * E : 0;
  p.total = o;
  return p;
}
}
namespace head {
constexpr int kVS = 7, kCS = 7, kJS = 13;
constexpr int kPairHitMin = 256;   // (gap, key) words a workgroup keeps at least

struct LdsPlan {
  int pos, vel, iw, nb, tq, push, outj, outc, zero, tjs, rec, list, surv, lam, u, obs, lim, count, patch, mip, porg, org, tslot, tbody, tin, tjoint, total;
  int pq, po, pnear, pbs, pcount, pbcnt, pblist;  // capsule-capsule contacts (only with pairs != 0)
  int phit, hit_cap;                              // their (gap, key) words: offset (64-bit aligned) and capacity
  int half, cand, cand_cap;                       // terrain search: half segments of the bodies, lists (in the copies' space)
  int wj, wc;                                     // kept impulses of joints and slots (only with warm != 0)
  int nu, nred, nsum;                             // Newton solver: body vectors, reduction entries, partial sums
};

// pairs: 0 = no capsule-capsule contacts, else the interaction group size (1 = self-collision only)
 inline LdsPlan make_plan(int B, int J, int S, int D, int F, int E, int with_patch, int pairs = 0,
                                             int threads = kThreads, int warm = 0, int newton = 0) {
  LdsPlan p;
  int o = 0;
  p.pos = o; o += B * 7 * E;
  p.vel = o; o += B * kVS * E;
  p.iw = o; o += B * kVS * E;
  p.nb = o; o += pairs ? B * E : 0;
  p.tq = o; o += J * 3 * E;
  p.push = o; o += 3 * E;
  o += o & 1;  // the search results kept in the copy arrays are 64-bit words
  // The sweep copies.  The terrain search, which is over before the first sweep, keeps its results there:
  // a 64-bit minimum per slot, half the segment of every body and the lists of rows and cells.
  const int copies = (J * kJS + S * kCS) * E, search = (2 * S + 3 * B) * E;
  p.outj = o;
  p.outc = o + J * kJS * E;
  p.half = o + 2 * S * E;
  p.cand = o + search;
  p.cand_cap = copies - search > 32 * E ? copies - search : 32 * E;
  o += copies > search + p.cand_cap ? copies : search + p.cand_cap;
  p.rec = o; o += S * kRecWords * E;
  p.list = o; o += S * E;
  p.surv = o; o += S * E;   // slots near the heightfield: end spheres from the front, mid-segments from the back
  p.lam = o;   // (with the warm start these impulses live in the per-slot array below)
  o += warm ? 0 : 3 * (S * E > threads - ((2 * J * E + 63) / 64) * 64 ? S * E - (threads - ((2 * J * E + 63) / 64) * 64) : 0);
  p.u = o; o += (D > 0 ? D : 1) * E;
  p.obs = o; o += (11 + 3 * D + F) * E;
  p.zero = p.obs;   // (six of them are zeros until the observation is packed)
  p.lim = o; o += (D > 0 ? D : 1) * E;
  if (with_patch) o = (o + 3) & ~3;   // (written four samples at a time)
  p.patch = o; o += with_patch ? E * kPatch * kPatch : 0;
  p.mip = o; o += with_patch ? E * kPatchBlocks * kPatchBlocks : 0;
  p.count = o; o += 8;
  p.porg = o; o += 2 * E;
  p.org = o; o += 3 * E;
  p.tjs = o; o += B * (kMaxBodyJoints + 3);  // tjs .. tjoint: one block, copied from Model::table_image
  p.tslot = o; o += 2 * S;
  p.tbody = o; o += 4 * B;
  p.tin = o; o += 6 * B;
  p.tjoint = o; o += J * (int)(sizeof(JointTab) / 4);
  p.pq = o; o += pairs ? kPairCap * kPairWords : 0;   // sorted queue of the substep's contacts
  p.po = o; o += pairs ? (kPairCap + 1) * 12 : 0;     // weighted velocity copies of their two bodies; the last entry stays zero
  p.pnear = o; o += pairs ? (E * pairs) / 2 + 1 : 0;  // agent pairs whose bounding spheres overlap
  p.pbs = o; o += pairs ? E : 0;                      // bounding radius of every agent about its root
  p.pcount = o; o += pairs ? 4 : 0;
  p.pbcnt = o; o += pairs ? B * E : 0;                  // per body: how many of them touch it
  p.pblist = o; o += pairs ? (B * E * 6 + 3) / 4 : 0;  // per body: up to six of them, one byte each
  // one 64-bit (gap, key) word per capsule-capsule contact found, for the choice of those that stay
  // when a workgroup finds more than it holds: in the space of the terrain search's candidate list
  // (idle by then) where that holds kPairHitMin words, else in a region of their own
  p.hit_cap = (p.cand_cap - 2) / 2;
  p.phit = (p.cand + 1) & ~1;
  if (pairs && p.hit_cap < kPairHitMin) {
    o += o & 1;
    p.phit = o; o += 2 * kPairHitMin;
    p.hit_cap = kPairHitMin;
  }
  p.wj = o; o += warm ? J * 6 * E : 0;
  p.wc = o; o += warm ? S * 3 * E : 0;
  p.nu = o; o += newton ? B * kVS * E : 0;
  p.nred = o; o += newton ? 3 * (J + S) * E : 0;
  p.nsum = o; o += newton ? 3 * 8 * E : 0;
  p.total = o;
  return p;
}
}
namespace nw {
constexpr int kVS = 7, kCS = 7, kJS = 13;
constexpr int kPairHitMin = 256;   // (gap, key) words a workgroup keeps at least
constexpr int kLdsWords = 160 * 1024 / 4;

struct LdsPlan {
  int pos, vel, iw, nb, tq, push, outj, outc, zero, tjs, rec, list, surv, lam, u, obs, lim, count, patch, mip, porg, org, tslot, tbody, tin, tjoint, total;
  int pq, po, pnear, pbs, pcount, pbcnt, pblist;  // capsule-capsule contacts (only with pairs != 0)
  int phit, hit_cap;                              // their (gap, key) words: offset (64-bit aligned) and capacity
  int half, cand, cand_cap;                       // terrain search: half segments of the bodies, lists
  int wj, wc;                                     // kept impulses of joints and slots (only with warm != 0)
  int nu, nred, nsum;                             // Newton solver: body vectors, reduction entries, partial sums
};

// field: 0 = plane, 1 = heightfield, 2 = heightfield of which every env keeps a copy
// pairs: 0 = no capsule-capsule contacts, else the interaction group size (1 = self-collision only)
 inline LdsPlan make_plan(int B, int J, int S, int D, int F, int E, int field, int pairs = 0,
                                             int threads = kThreads, int warm = 0, int newton = 0) {
  LdsPlan p;
  int o = 0;
  const bool with_patch = field == 2;
  p.pos = o; o += B * 7 * E;
  p.vel = o; o += B * kVS * E;
  p.iw = o; o += B * kVS * E;
  p.nb = o; o += pairs ? B * E : 0;
  p.tq = o; o += J * 3 * E;
  p.push = o; o += 3 * E;
  o += o & 1;  // the search results kept in the copy arrays are 64-bit words
  // The sweep copies.  The terrain search, which is over before the first sweep, keeps its results there:
  // a 64-bit minimum per slot and half the segment of every body (together never more than the copies,
  // since every body has a slot), and behind them the lists of rows and cells.  So does the search for
  // capsule-capsule contacts its spheres (one 16-byte word per body, an odd number of them per env).
  const int copies = (J * kJS + S * kCS) * E, search = field ? (2 * S + 3 * B) * E : 0;
  const int spheres = pairs ? 4 * (B | 1) * E + 3 : 0;
  p.outj = o;
  p.outc = o + J * kJS * E;
  p.half = o + 2 * S * E;
  p.cand = o + search;
  p.cand_cap = copies - search;
  o += copies > spheres ? copies : spheres;
  p.rec = o; o += S * kRecWords * E;
  p.list = o; o += S * E;
  p.surv = o; o += S * E;   // slots near the heightfield: end spheres from the front, mid-segments from the back
  p.lam = o;   // (with the warm start these impulses live in the per-slot array below)
  o += warm ? 0 : 3 * (S * E > threads - ((2 * J * E + 63) / 64) * 64 ? S * E - (threads - ((2 * J * E + 63) / 64) * 64) : 0);
  p.u = o; o += (D > 0 ? D : 1) * E;
  p.obs = o; o += (11 + 3 * D + F) * E;
  p.zero = p.obs;   // (six of them are zeros until the observation is packed)
  p.lim = o; o += (D > 0 ? D : 1) * E;
  if (with_patch) o = (o + 3) & ~3;   // (written four samples at a time)
  p.patch = o; o += with_patch ? E * kPatch * kPatch : 0;
  p.mip = o; o += with_patch ? E * kPatchBlocks * kPatchBlocks : 0;
  p.count = o; o += 8;
  p.porg = o; o += 2 * E;
  p.org = o; o += 3 * E;
  p.tjs = o; o += B * (kMaxBodyJoints + 3);  // tjs .. tjoint: one block, copied from Model::table_image
  p.tslot = o; o += 2 * S;
  p.tbody = o; o += 4 * B;
  p.tin = o; o += 6 * B;
  p.tjoint = o; o += J * (int)(sizeof(JointTab) / 4);
  p.pq = o; o += pairs ? kPairCap * kPairWords : 0;   // sorted queue of the substep's contacts
  p.po = o; o += pairs ? (kPairCap + 1) * 12 : 0;     // weighted velocity copies of their two bodies; the last entry stays zero
  p.pnear = o; o += pairs ? E * (pairs - 1) / 2 : 0;  // agent pairs whose bounding spheres overlap: at most all of them
  p.pbs = o; o += pairs ? E : 0;                      // bounding radius of every agent about its root
  p.pcount = o; o += pairs ? 4 : 0;
  p.pbcnt = o; o += pairs ? B * E : 0;                  // per body: how many of them touch it
  p.pblist = o; o += pairs ? (B * E * 6 + 3) / 4 : 0;  // per body: up to six of them, one byte each
  // one 64-bit (gap, key) word per capsule-capsule contact found, for the choice of those that stay
  // when a workgroup finds more than it holds: in the space of the terrain search's candidate list
  // (idle by then) where that holds kPairHitMin words, else in a region of their own
  p.hit_cap = (p.cand_cap - 2) / 2;
  p.phit = (p.cand + 1) & ~1;
  if (pairs && p.hit_cap < kPairHitMin) {
    o += o & 1;
    p.phit = o; o += 2 * kPairHitMin;
    p.hit_cap = kPairHitMin;
  }
  p.wj = o; o += warm ? J * 6 * E : 0;
  p.wc = o; o += warm ? S * 3 * E : 0;
  p.nu = o; o += newton ? B * kVS * E : 0;
  p.nred = o; o += newton ? 3 * (J + S) * E : 0;
  p.nsum = o; o += newton ? 3 * 8 * E : 0;
  // 32 list words per env are enough for the search; a robot without joints has no such space behind its
  // copies.  Its lists go to the end, as long as LDS has room: full lists only cost time (the direct search),
  // and no form is refused for them.
  if ((field || pairs) && p.cand_cap < 32 * E) {
    const int room = kLdsWords - o, cap = room < 32 * E ? room : 32 * E;
    if (cap > p.cand_cap) {
      p.cand = o; p.cand_cap = cap; o += cap;
      if ((cap - 2) / 2 > p.hit_cap) { p.phit = (p.cand + 1) & ~1; p.hit_cap = (cap - 2) / 2; }
    }
  }
  p.total = o;
  return p;
}
}

int main(){ long forms=0, lostHead=0, lostNew=0, lessHit=0, badFit=0, newOverOld=0, grow=0, lessList=0, diffHead=0;
 const int LIM=40960;
 for(int field=0;field<3;++field) for(int B=1;B<=16;++B) for(int caps=0;caps<=B;++caps) for(int J=0;J<=16;++J) for(int dk=0;dk<4;++dk) for(int F=0;F<=4;F+=2)
 for(int var=0;var<9;++var){ int pairs= var==1?1: var==2?2: var==3?4: var==4?8: var==5?16: var==8?1:0; int warm = var==6||var==8, newton = var==7;
  int per = field? 3:2, S = B-caps + caps*per, D = dk*J; if (S>48) continue;
  for(int E=1;E<=512;++E){ if(E*B>512||2*E*J>448) break; if(pairs>1&&E%pairs) continue;
   for(int wide=0;wide<(E==16&&!pairs&&!warm&&!newton?2:1);++wide){ int t=wide?768:512;
   if(newton){ int jt=((2*J*E+63)/64)*64; if(!(E<=8&&S*E<=512-jt&&2*B*E<=512)) continue; }
   auto o=old::make_plan(B,J,S,D,F,E,field==2,pairs,t,warm,newton); auto h=head::make_plan(B,J,S,D,F,E,field==2,pairs,t,warm,newton); auto n=nw::make_plan(B,J,S,D,F,E,field,pairs,t,warm,newton);
   ++forms; bool fo=o.total<=LIM, fh=h.total<=LIM, fn=n.total<=LIM;
   if(fo&&!fh) ++lostHead; if((fo||fh)&&!fn) { if(lostNew<5) printf("lost B%d S%d J%d D%d F%d E%d field%d pairs%d warm%d newton%d: %d %d %d\n",B,S,J,D,F,E,field,pairs,warm,newton,o.total,h.total,n.total); ++lostNew; }
   if(fn && pairs && n.hit_cap<o.hit_cap) ++lessHit;
   if(fn){ if(n.cand_cap<0||(n.cand+n.cand_cap>n.total)||(field&&n.half+3*B*E>n.cand&&n.cand>n.outj&&n.cand<n.rec)) ++badFit;
     if(pairs&&(n.phit&1)) ++badFit; if(pairs&&n.phit+2*n.hit_cap>n.total) ++badFit; if(pairs && n.phit<n.rec && n.phit+2*n.hit_cap>n.rec) ++badFit;
     if(pairs && ((n.outj+3)&~3)+4*(B|1)*E>n.rec) ++badFit;
     if(n.phit+2*n.hit_cap>n.rec && n.phit<n.total && pairs && n.phit<n.pq+kPairCap*kPairWords && n.phit>=n.rec) ++badFit;
     if((n.half+3*B*E>n.rec)&&field) ++badFit;
     if(field && n.cand_cap<32*E) ++lessList;
     if(E<=16 && J>=8 && B>=9 && (n.cand_cap!=h.cand_cap||n.total!=h.total||n.phit!=h.phit)&&field) ++diffHead; } } } }
 printf("forms %ld: refused at head %ld, refused now %ld, fewer hits than old %ld, misfits %ld, heightfield forms with lists under 32 E %ld, ant/humanoid-like field layouts that differ from head %ld\n",forms,lostHead,lostNew,lessHit,badFit,lessList,diffHead); }
