// Fused env-step kernel: every substep of one sim_step plus obs/reward packing
// in a single launch.
//
// Mapping.  One workgroup owns E consecutive environments for the whole step.
// All LDS arrays are laid out [item][component][E] with the env index fastest,
// and every thread role uses e = tid % E, so the lanes of a wavefront that work
// on the same item of neighbouring envs touch consecutive LDS banks and
// consecutive global addresses of the [field][body][env] state arrays.
// Roles (a thread can hold several):
//   body thread  (e, b): owns pose and velocity of one body in registers,
//   joint threads       : two neighbouring lanes own the six rows of one joint, one lane per
//                         body (parent, child); a row's J v is the sum of the two lanes' parts
//                         (four lanes in small workgroups, one where collisions share a large one),
//   contact thread      : owns the three rows of one active contact slot (constants in
//                         registers); a workgroup's contacts beyond one per thread are
//                         rebuilt from their LDS record every sweep,
//   pair-side threads   : (collision variant) two lanes per capsule-capsule contact,
//   env thread   (e)    : packs root observations, reward and done, applies the task rules.
// The joint-side threads fill the low wavefronts, the contact threads the high ones, so that a
// wavefront runs either the joint or the contact branch of a sweep.
//
// Per substep (Section 3.1 of the paper: maximal coordinates, torque control,
// speculative unilateral contacts, isotropic Coulomb friction, restitution 0):
//   A  body threads publish pose, world inverse inertia and half segment
//   B  contact generation per slot; joint threads turn actions into torques.  On the heightfield the
//      search by rows of cells, with the gravity / torque / gyroscopic term integrated beside the records
//   P  (collision variant) capsule-capsule contacts within an agent and within a group; on the plane
//      the forces are integrated beside them
//   C  (collision variant) body threads sum up the weights of their blocks; without capsule pairs the
//      lanes that need such a sum form it themselves
//   D  joint / contact threads build row constants; on the plane without capsule pairs the contact
//      wavefronts integrate the forces beside the joint rows
//   S  (warm-start variant: sweep -1 applies the impulses kept from the last substep)
//      `iterations` sweeps: every block relaxes its rows one after another, as on a
//      private copy of its bodies taken from the shared snapshot; a body is
//      shared out among its blocks by weight (joint 1, contact a ramp from 0 at
//      the margin to 1 at half the margin) and acts inside block c with inverse
//      mass scaled by W / w_c; then every body takes the weighted average of the
//      copies, which is the plain sum of what the blocks' impulses change in its
//      velocity (those changes are what the blocks leave in LDS), in static order
//      (no atomics)
//   E  damping, angular-velocity cap, position integration
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "contact_gen.hpp"
#include "model.hpp"

namespace sim355 {

constexpr int kThreads = 512;       // threads per workgroup every shape fits (host-side limits)
constexpr int kThreadsWide = 768;   // the wider workgroup the big heightfield batches are run with
constexpr int kGroup = 8;  // lanes that share the fine terrain search of one slot
constexpr int kPatchBlocks = (kPatch + kMip - 1) / kMip;

struct StepArgs {
  const Model* M;
  const float* heights;
  const float* coarse;   // block maxima of the heightfield
  const float* origins;  // [N][3]
  float* targets;  // [N][2]
  float* state;          // [13][B][N]
  int32_t* steps;        // [N]
  const float* actions;  // [N][D] or null
  float* obs;            // [N][obs_dim]
  float* reward;         // [N]
  uint8_t* done;         // [N]
  int32_t* recs;         // [N][S][12] or null
  int N, E, substeps, iterations, count_step;
  float h;
  float* obs_out;        // caller arrays for obs / reward / done (sim_step_obs) that replace the library's, or null
  float* reward_out;
  uint8_t* done_out;
  TaskParams task;       // task logic (enabled = 0: off)
  int32_t* task_i;       // [N][4]: frames below the threshold, target age, frame of the next push, episode
  float* push;           // [N][3]: force on the root body during this step
  long long* dbg;        // phase-timing slots (diagnostic build only)
  float* lam_j;          // warm start: [J*6][N] joint row impulses at the end of the last substep
  float* lam_s;          //             [S*3][N] terrain slot impulses (0 for slots that were inactive)
  int32_t* pair_recs;    // [grid][kPairCap][8] capsule-capsule contacts of the last substep, or null
  int32_t* pair_count;   // [grid] their number per workgroup
  int32_t* pair_dropped; // [1] contacts dropped because a workgroup found more than kPairCap
  const uint8_t* reset_mask; // sim_reset (a launch without substeps): which envs (null: all), the seed, and whether
  uint64_t reset_seed;
  int reset;
  const int32_t* place_env;  // [N] agent standing at every place of the launch, or null: agent = place
};

// Rows (E consecutive floats) per item of the velocity, inverse-inertia and change arrays.  Odd
// counts, so that neighbouring items start in different LDS banks when E is 16.
// The two sides of a joint lie an odd number of rows apart as well: neighbouring lanes store to both at once.
constexpr int kVS = 7, kCS = 7, kJS = 13, kSide = 7;
constexpr int kPairHitMin = 256;   // (gap, key) words a workgroup keeps at least
// Words of LDS a workgroup can ask for: 160 KiB without the 256 bytes that the compiler takes for the barrier
// that also says whether an env was reset.
constexpr int kLdsWords = (160 * 1024 - 256) / 4;

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
// lanes: lanes that relax one joint (1, 2 or 4)
__host__ __device__ inline LdsPlan make_plan(int B, int J, int S, int D, int F, int E, int field, int pairs = 0,
                                             int threads = kThreads, int warm = 0, int newton = 0, int lanes = 2) {
  LdsPlan p;
  int o = 0;
  const bool with_patch = field == 2;
  p.pos = o; o += B * 7 * E;
  p.vel = o; o += B * kVS * E;
  p.iw = o; o += B * kVS * E;
  p.nb = o; o += pairs ? B * E : 0;
  p.tq = o; o += J * 3 * E;
  p.push = o; o += 3 * E;
  o += o & 1;  // the search results kept in the change arrays are 64-bit words
  // The sweeps' changes of velocity.  The terrain search, which is over before the first sweep, keeps its results there:
  // a 64-bit minimum per slot and half the segment of every body (together never more than the changes,
  // since every body has a slot), and behind them the lists of rows and cells, for which 32 words per env are
  // enough.  So does the search for capsule-capsule contacts its spheres (one 16-byte word per body, an
  // odd number of them per env).  A robot with few joints has less room than that behind its results: up to
  // 16 envs the changes' space is then made larger, which LDS always has room for.  With more of them (which only
  // a caller asks for) nothing is reserved that the ground does not need, and the lists take what is left at
  // the end: full lists only cost time (the direct search), and no form is refused for them.
  const bool many = E > 16;
  const int changes = (J * kJS + S * kCS) * E, search = many && !field ? 0 : (2 * S + 3 * B) * E;
  const int spheres = pairs ? 4 * (B | 1) * E + 3 : 0;
  p.outj = o;
  p.outc = o + J * kJS * E;
  p.half = o + 2 * S * E;
  p.cand = o + search;
  p.cand_cap = changes - search > 32 * E ? changes - search : (many ? changes - search : 32 * E);
  o += changes > search + p.cand_cap ? changes : search + p.cand_cap;
  o += many && spheres > changes ? spheres - changes : 0;
  p.rec = o; o += S * kRecWords * E;
  p.list = o; o += S * E;
  p.surv = o; o += S * E;   // slots near the heightfield: end spheres from the front, mid-segments from the back
  p.lam = o;   // (with the warm start these impulses live in the per-slot array below)
  const int contact_threads = threads - ((lanes * J * E + 63) / 64) * 64;
  o += warm ? 0 : 3 * (S * E > contact_threads ? S * E - contact_threads : 0);
  p.u = o; o += (D > 0 ? D : 1) * E;
  p.obs = o; o += (11 + 3 * D + F) * E;
  p.zero = p.obs;   // (the first six rows are zeros while the sweeps run)
  p.lim = o; o += (D > 0 ? D : 1) * E;   // (one count per env is in use; the room decides which numbers of envs fit, and stays)
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
  p.po = o; o += pairs ? (kPairCap + 1) * 12 : 0;     // changes of their two bodies' velocities; the last entry stays zero
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
  if (many && (field || pairs) && p.cand_cap < 32 * E) {
    const int room = kLdsWords - o, cap = room < 32 * E ? room : 32 * E;
    if (cap > p.cand_cap) {
      p.cand = o; p.cand_cap = cap; o += cap;
      if ((cap - 2) / 2 > p.hit_cap) { p.phit = (p.cand + 1) & ~1; p.hit_cap = (cap - 2) / 2; }
    }
  }
  p.total = o;
  return p;
}

// The arithmetic of the substeps is written out down to the single rounded operation: contraction is off
// and every fused multiply-add is spelled, so that the forms of the kernel give the same bits whatever the
// compiler inlines, hoists or splits into blocks around them.  A sum of products is
// a0 b0 + a1 b1 + a2 b2 = fma(a2, b2, fma(a0, b0, a1 b1)).  Left to the compiler are the Newton solve by the whole
// workgroup (robots with more rows than a wavefront has lanes) and what follows the substeps: the
// observation, the reward and the poses of a reset.
#pragma clang fp contract(off)
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ float sum2(float a0, float b0, float a1, float b1) { return fma_(a0, b0, a1 * b1); }
__device__ __forceinline__ float diff2(float a0, float b0, float a1, float b1) { return fma_(a0, b0, -(a1 * b1)); }
__device__ __forceinline__ float sum3(float a0, float b0, float a1, float b1, float a2, float b2) {
  return fma_(a2, b2, sum2(a0, b0, a1, b1));
}

__device__ __forceinline__ void quat_to_mat(const float q[4], float R[9]) {
  // R[3*r + c]: row r, column c; column c is the image of body axis c
  float w = q[0], x = q[1], y = q[2], z = q[3];
  R[0] = fma_(-2.0f, sum2(y, y, z, z), 1.0f); R[1] = 2.0f * diff2(x, y, w, z); R[2] = 2.0f * sum2(x, z, w, y);
  R[3] = 2.0f * sum2(x, y, w, z); R[4] = fma_(-2.0f, sum2(x, x, z, z), 1.0f); R[5] = 2.0f * diff2(y, z, w, x);
  R[6] = 2.0f * diff2(x, z, w, y); R[7] = 2.0f * sum2(y, z, w, x); R[8] = fma_(-2.0f, sum2(x, x, y, y), 1.0f);
}
__device__ __forceinline__ void mat_vec(const float R[9], const float a[3], float o[3]) {
  o[0] = sum3(R[0], a[0], R[1], a[1], R[2], a[2]);
  o[1] = sum3(R[3], a[0], R[4], a[1], R[5], a[2]);
  o[2] = sum3(R[6], a[0], R[7], a[1], R[8], a[2]);
}
__device__ __forceinline__ void mat_t_vec(const float R[9], const float a[3], float o[3]) {
  o[0] = sum3(R[0], a[0], R[3], a[1], R[6], a[2]);
  o[1] = sum3(R[1], a[0], R[4], a[1], R[7], a[2]);
  o[2] = sum3(R[2], a[0], R[5], a[1], R[8], a[2]);
}
// symmetric 3x3 (xx,xy,xz,yy,yz,zz) times vector
__device__ __forceinline__ void sym_vec(const float S[6], const float a[3], float o[3]) {
  o[0] = sum3(S[0], a[0], S[1], a[1], S[2], a[2]);
  o[1] = sum3(S[1], a[0], S[3], a[1], S[4], a[2]);
  o[2] = sum3(S[2], a[0], S[4], a[1], S[5], a[2]);
}
__device__ __forceinline__ void cross(const float a[3], const float b[3], float o[3]) {
  o[0] = diff2(a[1], b[2], a[2], b[1]);
  o[1] = diff2(a[2], b[0], a[0], b[2]);
  o[2] = diff2(a[0], b[1], a[1], b[0]);
}
__device__ __forceinline__ float dot(const float a[3], const float b[3]) {
  return sum3(a[0], b[0], a[1], b[1], a[2], b[2]);
}
// (r x e_k) . w for the unit vector e_k, zero terms left out
__device__ __forceinline__ float cross_unit_dot(const float r[3], int k, const float w[3]) {
  return k == 0 ? diff2(r[2], w[1], r[1], w[2]) : (k == 1 ? diff2(r[0], w[2], r[2], w[0]) : diff2(r[1], w[0], r[0], w[1]));
}
// r x e_k
__device__ __forceinline__ void cross_unit(const float r[3], int k, float o[3]) {
  if (k == 0) { o[0] = 0.0f; o[1] = r[2]; o[2] = -r[1]; }
  else if (k == 1) { o[0] = -r[2]; o[1] = 0.0f; o[2] = r[0]; }
  else { o[0] = r[1]; o[1] = -r[0]; o[2] = 0.0f; }
}
// rotation vector of conj(qa) * qb, short way round
// atan2(y, x) for y >= 0, x >= 0 (not both zero), to about 2 ulp: the argument is brought into
// [0, tan(pi/8)] by the identities atan(t) = pi/2 - atan(1/t) and atan(t) = pi/4 + atan((t-1)/(t+1)),
// where an odd polynomial of degree 9 does (the classic single-precision arctangent of the Cephes
// library; coefficients as published there).  Runs once per joint side and substep, on the path
// everybody waits for, where the general library routine and two correctly rounded divisions
// cost several times as much.
__device__ __forceinline__ float atan2_first_quadrant(float y, float x) {
  const bool big = y > 2.414213562373095f * x, mid = y > 0.4142135623730950f * x;
  // t = y / x, or -x / y, or (y - x) / (y + x)
  const float num = big ? -x : (mid ? y - x : y), den = big ? y : (mid ? y + x : x);
  const float t = num * __builtin_amdgcn_rcpf(den);
  const float base = big ? 1.5707963267948966f : (mid ? 0.7853981633974483f : 0.0f);
  const float z = t * t;
  const float p = fma_(fma_(fma_(fma_(8.05374449538e-2f, z, -1.38776856032e-1f), z, 1.99777106478e-1f), z, -3.33329491539e-1f) * z, t, t);
  return base + p;
}

__device__ __forceinline__ void rel_rotvec(const float qa[4], const float qb[4], float phi[3]) {
  float w = fma_(qa[3], qb[3], sum3(qa[0], qb[0], qa[1], qb[1], qa[2], qb[2]));
  float x = fma_(qa[3], qb[2], fma_(-qa[2], qb[3], diff2(qa[0], qb[1], qa[1], qb[0])));
  float y = fma_(-qa[3], qb[1], fma_(-qa[2], qb[0], sum2(qa[0], qb[2], qa[1], qb[3])));
  float z = fma_(-qa[3], qb[0], fma_(qa[2], qb[1], diff2(qa[0], qb[3], qa[1], qb[2])));
  if (w < 0.0f) { w = -w; x = -x; y = -y; z = -z; }
  const float s2 = sum3(x, x, y, y, z, z);
  const float inv_s = __builtin_amdgcn_rsqf(fmaxf(s2, 1e-30f)), s = s2 * inv_s;
  float k = (s < 1e-12f) ? 2.0f : 2.0f * atan2_first_quadrant(s, w) * inv_s;
  phi[0] = k * x; phi[1] = k * y; phi[2] = k * z;
}

// Height of the heightfield surface under a world xy (plane of the containing triangle): the cell
// and the place within it, then the height from the cell's four samples.
struct HeightCell {
  int at;          // sample (i, j)
  float fx, fy;
};
__device__ __forceinline__ HeightCell height_cell(int nx, int ny, float cell, float hox, float hoy, float wx, float wy) {
  float ux = (wx - hox) / cell, uy = (wy - hoy) / cell;
  float fi = floorf(ux), fj = floorf(uy);
  float mi = (float)(nx - 2), mj = (float)(ny - 2);
  fi = fminf(fmaxf(fi, 0.0f), mi); fj = fminf(fmaxf(fj, 0.0f), mj);
  HeightCell c;
  c.at = (int)fj * nx + (int)fi;
  c.fx = fminf(fmaxf(ux - fi, 0.0f), 1.0f); c.fy = fminf(fmaxf(uy - fj, 0.0f), 1.0f);
  return c;
}
__device__ __forceinline__ float height_in_cell(float fx, float fy, float h00, float h10, float h11, float h01) {
  if (fx >= fy) return fma_(fy, h11 - h10, fma_(fx, h10 - h00, h00));
  return fma_(fy, h01 - h00, fma_(fx, h11 - h01, h00));
}

__device__ __forceinline__ void store_record(float* Lrec, int* Lreci, int s, int ee, int E, const ContactOut& co) {
  Lreci[(s * kRecWords + 0) * E + ee] = co.active;
  Lreci[(s * kRecWords + 1) * E + ee] = co.kind;
  Lreci[(s * kRecWords + 2) * E + ee] = co.feat;
  Lrec[(s * kRecWords + 3) * E + ee] = co.d;
  Lrec[(s * kRecWords + 4) * E + ee] = co.n.x;
  Lrec[(s * kRecWords + 5) * E + ee] = co.n.y;
  Lrec[(s * kRecWords + 6) * E + ee] = co.n.z;
  Lrec[(s * kRecWords + 7) * E + ee] = co.rc.x;
  Lrec[(s * kRecWords + 8) * E + ee] = co.rc.y;
  Lrec[(s * kRecWords + 9) * E + ee] = co.rc.z;
  Lrec[(s * kRecWords + 10) * E + ee] = co.w;
}

// Rows of one joint as seen from ONE of its two bodies (a joint is relaxed by a pair of
// neighbouring lanes, one per side; a row's J v is the sum of the two lanes' parts, exchanged
// with a DPP lane swap, and each lane then leaves its own body's change of velocity).  sg = -1 for
// the parent side, +1 for the child side; all signs are folded into the stored vectors.
// The rows of a block are relaxed one after another, each on the velocities the ones before it left.
// All six J v are taken from the snapshot at once, and what an earlier row of the block adds to a later
// row's is its impulse times an entry of J M^-1 J^T (both bodies scaled by W / w), known since the set-up:
// the sequence is then a triangular one over impulses instead of a trip through both velocities per row.
struct SideRows {
  float sr[3];             // sg * lever arm from the own centre to the shared impulse point
  float sv;                // sg / m_o: own linear response per unit impulse
  float sg;
  float Y[3][3];           // own angular response per unit impulse of positional row k
  float pme[3], pnb[3];    // -m_eff and -m_eff * bias of the positional rows (world x, y, z)
  float sax[3][3];         // sg * joint axis k (sign of an upper limit folded in)
  float Z[3][3];           // own angular response per unit impulse of angular row k
  float ame[3], anb[3];
  float pp[3];             // -m_eff (J M^-1 J^T) of rows (1, 0), (2, 0), (2, 1)
  float ap[3][3];          //                     of angular row k and positional row c
  float aa[3];             //                     of angular rows (1, 0), (2, 0), (2, 1)
  float nl[3];             // lower bound of the next increment of angular row k: minus the impulse so
                           // far for a limit row (impulse >= 0), -infinity for a locked axis
  float lam[3];            // impulses of the angular rows so far (only the warm start keeps them)
  float pD[3], pb[3];      // (Newton solver) diagonal of J M^-1 J^T and bias of the positional rows
  float aD[3], ab[3];      //                 and of the angular rows
  int onesided;            // bit k set: angular row k is a limit row (impulse >= 0)
  int upper;               // bit k set: that limit row stands for the upper limit
};
// value of the neighbouring lane (lane ^ 1), one DPP move
__device__ __forceinline__ float lane_swap1(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, true));
}

// value of another lane of the same four: lane i takes that of lane (kCtrl >> 2 i) & 3
template <int kCtrl>
__device__ __forceinline__ float quad_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
}

// All six rows of a joint in one lane: what SideRows holds of both sides ([0] parent, [1] child; signs folded in).
struct JointRows {
  float sr[2][3], sv[2], Y[2][3][3], sax[2][3][3], Z[2][3][3];
  float pme[3], pnb[3], ame[3], anb[3], pp[3], ap[3][3], aa[3], nl[3], lam[3];
  int onesided, upper;
};

// The three rows of one lane of four (see the sweeps): positional or angular ones of one side of a joint.
struct QuadRows {
  float K[3][3], kv;       // J on the side's angular velocity; on its linear velocity (angular rows: 0)
  float me[3], nb[3];      // -m_eff, -m_eff * bias
  float t1[3], t2[3];      // -m_eff (J M^-1 J^T) among positional, among angular rows (0 in the other kind's lanes)
  float ap[3][3];          //                     of angular with positional rows (positional: 0)
  float nl[3], lam[3];     // lower bound of the next increments; impulses so far (warm start)
  float R[3][3], sv;       // the side's angular response, its linear one
};

// lane_swap1 through the LDS crossbar (no memory is touched): twice the latency of a DPP move for a wavefront that has
// its SIMD to itself, but a DPP move holds up the SIMD's other wavefronts
__device__ __forceinline__ float lane_swap1_crossbar(float x) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x041F /* lane ^ 1 */));
}

// maximum without the instruction that quietens a signalling NaN first, which the compiler puts before
// every fmaxf whose operand comes from an earlier round of a loop
__device__ __forceinline__ float max_of(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Sum over the 64 lanes of a wavefront, the same in all of them (a fixed tree of DPP moves: pairs, fours,
// eights and sixteens within a row, then across the rows into the last lane).
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, kRows, 0xF, false));
}
__device__ __forceinline__ void wave_sum3(float& a, float& b, float& c) {
  a = dpp_add<0x111, 0xF>(a); b = dpp_add<0x111, 0xF>(b); c = dpp_add<0x111, 0xF>(c);   // row_shr:1
  a = dpp_add<0x112, 0xF>(a); b = dpp_add<0x112, 0xF>(b); c = dpp_add<0x112, 0xF>(c);   // row_shr:2
  a = dpp_add<0x114, 0xF>(a); b = dpp_add<0x114, 0xF>(b); c = dpp_add<0x114, 0xF>(c);   // row_shr:4
  a = dpp_add<0x118, 0xF>(a); b = dpp_add<0x118, 0xF>(b); c = dpp_add<0x118, 0xF>(c);   // row_shr:8
  a = dpp_add<0x142, 0xA>(a); b = dpp_add<0x142, 0xA>(b); c = dpp_add<0x142, 0xA>(c);   // row_bcast:15
  a = dpp_add<0x143, 0xC>(a); b = dpp_add<0x143, 0xC>(b); c = dpp_add<0x143, 0xC>(c);   // row_bcast:31
  a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 63));
  b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 63));
  c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), 63));
}

struct ContactRows {
  float dir[3][3];   // n, t1, t2
  float rc[3];       // lever arm
  float ang[3][3];   // rc x dir
  float Y[3][3];     // angular response
  float ls;          // linear response 1 / m
  float meff[3], bias, lam[3];
  float tn[2];       // -m_eff (J M^-1 J^T) of the tangent rows and the normal row, see SideRows
  float D[3];        // (Newton solver) diagonal of J M^-1 J^T
  int slot_e;        // slot * E + e
  int body;
};

// Phase timing (diagnostic build, -DSIM_PHASE_TIMING): thread 0 of workgroup 7 adds the cycles
// since the previous mark to slot k of a small buffer in the workspace.
// Each mark costs a few hundred cycles itself, so marks are kept out of the sweep loop.
#ifdef SIM_PHASE_TIMING
#define TMARK(k) do { if (tid == 0 && blockIdx.x == 7) { long long _t = clock64(); a.dbg[k] += _t - t_last; t_last = _t; } } while (0)
#else
#define TMARK(k) do { } while (0)
#endif

// Row constants of one active contact slot from its LDS record (d, n, rc, weight), the
// body's world inverse inertia, weight sum and inverse mass.
__device__ __forceinline__ void build_contact_rows(ContactRows& c, const float* Lrec, const float* Liw,
                                                   float nb, int s, int ee, int E, int body, float imb,
                                                   float h, float beta_c, float v_depen, bool whole_body = false) {
  c.body = body;
  c.slot_e = s * E + ee;
  float d = Lrec[(s * kRecWords + 3) * E + ee];
  float n[3], rc[3], iwb[6];
  for (int k = 0; k < 3; ++k) { n[k] = Lrec[(s * kRecWords + 4 + k) * E + ee]; rc[k] = Lrec[(s * kRecWords + 7 + k) * E + ee]; }
  for (int k = 0; k < 6; ++k) iwb[k] = Liw[(body * kVS + k) * E + ee];
  float nbb = nb / Lrec[(s * kRecWords + 10) * E + ee];
  if (whole_body) nbb = 1.0f;   // (the Newton solver does not split the body among its blocks)
  float t1[3], t2[3];
  if (fabsf(n[0]) < 0.57735f) { t1[0] = 0.0f; t1[1] = n[2]; t1[2] = -n[1]; }
  else { t1[0] = -n[2]; t1[1] = 0.0f; t1[2] = n[0]; }
  float inv = 1.0f / sqrtf(dot(t1, t1));
  for (int k = 0; k < 3; ++k) t1[k] *= inv;
  cross(n, t1, t2);
  for (int k = 0; k < 3; ++k) { c.dir[0][k] = n[k]; c.dir[1][k] = t1[k]; c.dir[2][k] = t2[k]; }
  for (int k = 0; k < 3; ++k) c.rc[k] = rc[k];
  c.ls = imb;
  for (int r = 0; r < 3; ++r) {
    cross(rc, c.dir[r], c.ang[r]);
    sym_vec(iwb, c.ang[r], c.Y[r]);
    float keff = nbb * (imb + dot(c.ang[r], c.Y[r]));
    c.meff[r] = keff > 0.0f ? 1.0f / keff : 0.0f;
    c.D[r] = keff;
    if (r > 0) c.tn[r - 1] = -c.meff[r] * (nbb * dot(c.ang[r], c.Y[0]));   // (n and t are orthogonal: no linear part)
    c.lam[r] = 0.0f;
  }
  c.bias = d >= 0.0f ? d / h : fmaxf(beta_c * d / h, -v_depen);
}

// Friction pair (l1, l2) brought back onto the disc of radius lim >= 0 (Section 3.1: isotropic
// Coulomb friction).  Runs in every sweep of every contact, so the test compares squares and the
// scale lim / |l| comes from the hardware's reciprocal square root (1 ulp) instead of a correctly
// rounded square root and division; the floor keeps a denormal |l|^2 from turning into infinity.
__device__ __forceinline__ void project_on_disc(float& l1, float& l2, float lim) {
  const float n2 = sum2(l1, l1, l2, l2);
  const float on_disc = lim * __builtin_amdgcn_rsqf(fmaxf(n2, 1e-30f));
  const float sc = n2 > lim * lim ? on_disc : 1.0f;
  l1 *= sc; l2 *= sc;
}

// What the impulses d of a contact's rows change in its body's velocity.
__device__ __forceinline__ void contact_response(const ContactRows& c, const float d[3], float vv[3], float ww[3]) {
  for (int k = 0; k < 3; ++k) {
    vv[k] = c.ls * sum3(c.dir[0][k], d[0], c.dir[1][k], d[1], c.dir[2][k], d[2]);
    ww[k] = sum3(c.Y[0][k], d[0], c.Y[1][k], d[1], c.Y[2][k], d[2]);
  }
}

// One sweep of a contact block from the snapshot (vv, ww) of the body velocity, which the change it makes
// replaces: normal row (impulse >= 0), then the friction pair projected on the disc mu * lambda_n.
__device__ __forceinline__ void relax_contact(ContactRows& c, float mu, float vv[3], float ww[3]) {
  // velocity of the contact point
  const float u[3] = {fma_(ww[1], c.rc[2], fma_(-ww[2], c.rc[1], vv[0])), fma_(ww[2], c.rc[0], fma_(-ww[0], c.rc[2], vv[1])),
                      fma_(ww[0], c.rc[1], fma_(-ww[1], c.rc[0], vv[2]))};
  const float b1 = fma_(-c.meff[1], dot(c.dir[1], u), c.lam[1]), b2 = fma_(-c.meff[2], dot(c.dir[2], u), c.lam[2]);
  const float ln = fmaxf(fma_(-c.meff[0], dot(c.dir[0], u) + c.bias, c.lam[0]), 0.0f);
  float d[3];
  d[0] = ln - c.lam[0];
  float l1 = fma_(c.tn[0], d[0], b1), l2 = fma_(c.tn[1], d[0], b2);
  project_on_disc(l1, l2, mu * ln);
  d[1] = l1 - c.lam[1]; d[2] = l2 - c.lam[2];
  c.lam[0] = ln; c.lam[1] = l1; c.lam[2] = l2;
  contact_response(c, d, vv, ww);
}

// Rows of one capsule-capsule contact (Section 3.1: contacts among bodies; Section 4.1:
// inter-agent collisions) as seen from ONE of its two bodies: normal and two tangents between
// body A (+J) and body B (-J), one contact point for both (midway between the closest surface
// points, so the pair of opposite impulses carries no net torque).  Like a joint, a contact is
// relaxed by two neighbouring lanes, one per body; a row's J v is the sum of the two lanes'
// parts, both lanes compute the same impulse and each leaves its own body's change of velocity.  All
// signs (+1 for A, -1 for B) are folded into the stored vectors.
struct PairSide {
  float sd[3][3];    // sg * (n, t1, t2); n points from B to A
  float sa[3][3];    // sg * (lever arm x direction)
  float Y[3][3];     // own angular response per unit impulse
  float ls;          // own linear response per unit impulse along sd
  float meff[3], bias, lam[3];
  float tn[2];       // -m_eff (J M^-1 J^T) of the tangent rows and the normal row, see SideRows
  int off;           // own body's velocity rows in LDS: body * kVS * E + env
};

// Builds side `side` (0: body A, 1: body B) of queue entry k from the poses, the segment
// parameters (s, t) the contact search found, the body's world inverse inertia and weight sum.
// Both lanes evaluate the same geometry with the same operations.
__device__ __forceinline__ void build_pair_side(PairSide& c, int side, const float* Lpq, const float* Lpos,
                                                const float* Liw, const float* Lnb, const float* Lorg,
                                                const float* Ltbody, int k, int E, float h, float beta_c,
                                                float v_depen) {
  const int refs = __float_as_int(Lpq[k * kPairWords + 1]);
  const int ra = refs & 0xffff, rb = (refs >> 16) & 0xffff;
  const int ba = ra / E, ea = ra - ba * E, bb = rb / E, eb = rb - bb * E;
  const float sp = Lpq[k * kPairWords + 2], tp = Lpq[k * kPairWords + 3], wk = Lpq[k * kPairWords + 4];
  // the closest points as seen from the two centres: ca, cb; df from B's to A's
  float qa[4], qb[4];
  for (int i = 0; i < 4; ++i) { qa[i] = Lpos[(ba * 7 + 3 + i) * E + ea]; qb[i] = Lpos[(bb * 7 + 3 + i) * E + eb]; }
  const float radA = Ltbody[4 * ba], hlA = Ltbody[4 * ba + 1];
  const float radB = Ltbody[4 * bb], hlB = Ltbody[4 * bb + 1];
  const int axA = __float_as_int(Ltbody[4 * ba + 2]), axB = __float_as_int(Ltbody[4 * bb + 2]);
  float Ra[9], Rb[9], ca[3], cb[3], df[3];
  quat_to_mat(qa, Ra);
  quat_to_mat(qb, Rb);
  for (int i = 0; i < 3; ++i) {
    ca[i] = (2.0f * sp - 1.0f) * (Ra[3 * i + axA] * hlA);
    cb[i] = (2.0f * tp - 1.0f) * (Rb[3 * i + axB] * hlB);
    const float dx = (Lpos[(ba * 7 + i) * E + ea] - Lpos[(bb * 7 + i) * E + eb]) - (Lorg[i * E + eb] - Lorg[i * E + ea]);
    df[i] = dx + (ca[i] - cb[i]);
  }
  const float dist = sqrtf(dot(df, df));
  float n[3] = {0.0f, 0.0f, 1.0f};
  if (dist >= 1e-9f) { const float inv = 1.0f / dist; for (int i = 0; i < 3; ++i) n[i] = df[i] * inv; }
  const float d = dist - radA - radB;
  // own body
  const int bo = side ? bb : ba, eo = side ? eb : ea;
  const float sg = side ? -1.0f : 1.0f;
  float arm[3], iwo[6];
  for (int i = 0; i < 3; ++i) {
    // midway between the two surface points, seen from the own centre (the other side's closest point is df away)
    arm[i] = fma_(0.5f, fma_(n[i], radB - radA, side ? df[i] : -df[i]), side ? cb[i] : ca[i]);
  }
  for (int i = 0; i < 6; ++i) iwo[i] = Liw[(bo * kVS + i) * E + eo];
  const float imo = Ltbody[4 * bo + 3];
  const float nbo = Lnb[bo * E + eo] / wk;
  float t1[3], t2[3];
  if (fabsf(n[0]) < 0.57735f) { t1[0] = 0.0f; t1[1] = n[2]; t1[2] = -n[1]; }
  else { t1[0] = -n[2]; t1[1] = 0.0f; t1[2] = n[0]; }
  const float inv = 1.0f / sqrtf(dot(t1, t1));
  for (int i = 0; i < 3; ++i) t1[i] *= inv;
  cross(n, t1, t2);
  for (int i = 0; i < 3; ++i) { c.sd[0][i] = sg * n[i]; c.sd[1][i] = sg * t1[i]; c.sd[2][i] = sg * t2[i]; }
  c.ls = imo;
  for (int r = 0; r < 3; ++r) {
    cross(arm, c.sd[r], c.sa[r]);
    sym_vec(iwo, c.sa[r], c.Y[r]);
    const float kp = nbo * (imo + dot(c.sa[r], c.Y[r]));
    const float keff = kp + lane_swap1(kp);
    c.meff[r] = keff > 0.0f ? 1.0f / keff : 0.0f;
    if (r > 0) {
      const float kt = nbo * dot(c.sa[r], c.Y[0]);
      c.tn[r - 1] = -c.meff[r] * (kt + lane_swap1(kt));
    }
    c.lam[r] = 0.0f;
  }
  c.bias = d >= 0.0f ? d / h : fmaxf(beta_c * d / h, -v_depen);
  c.off = bo * kVS * E + eo;
}

// One sweep of one side of a capsule-capsule block from the snapshot (v, w) of the own body's velocity, which
// the change it makes replaces.
__device__ __forceinline__ void relax_pair_side(PairSide& c, float mu, float v[3], float w[3]) {
  const float p0 = dot(c.sd[0], v) + dot(c.sa[0], w), p1 = dot(c.sd[1], v) + dot(c.sa[1], w), p2 = dot(c.sd[2], v) + dot(c.sa[2], w);
  const float jv0 = p0 + lane_swap1(p0), jv1 = p1 + lane_swap1(p1), jv2 = p2 + lane_swap1(p2);
  const float b1 = fma_(-c.meff[1], jv1, c.lam[1]), b2 = fma_(-c.meff[2], jv2, c.lam[2]);
  const float ln = fmaxf(fma_(-c.meff[0], jv0 + c.bias, c.lam[0]), 0.0f);
  const float d0 = ln - c.lam[0];
  float l1 = fma_(c.tn[0], d0, b1), l2 = fma_(c.tn[1], d0, b2);
  project_on_disc(l1, l2, mu * ln);
  const float d1 = l1 - c.lam[1], d2 = l2 - c.lam[2];
  c.lam[0] = ln; c.lam[1] = l1; c.lam[2] = l2;
  for (int k = 0; k < 3; ++k) {
    v[k] = c.ls * sum3(c.sd[0][k], d0, c.sd[1][k], d1, c.sd[2][k], d2);
    w[k] = sum3(c.Y[0][k], d0, c.Y[1][k], d1, c.Y[2][k], d2);
  }
}

// EC > 0: envs per workgroup fixed at compile time (LDS offsets become immediates);
// EC == 0: taken from the launch arguments.  NJ: compile-time bound on the joints one body
// belongs to (the per-body average reads NJ joint entries without branching).
#pragma clang fp contract(fast)
// counter-based uniform draw: one 64-bit mixing finaliser per (seed, env, index)
__device__ inline float reset_uniform(uint64_t seed, uint64_t env, uint64_t idx) {
  uint64_t z = seed + env * 0x632BE59BD9B4E019ULL + idx * 0xD1B54A32D192ED03ULL;
  z += 0x9E3779B97F4A7C15ULL;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  z ^= z >> 31;
  return (float)(z >> 40) * (1.0f / 16777216.0f);
}
// draws of the task logic, keyed by (seed, episode, env, frame, k): k = 0 push magnitude,
// 1 push direction, 2 frames to the next push, 3 target distance, 4 target direction
__device__ inline float task_u(const TaskParams& t, int env, int episode, int frame, int k) {
  return reset_uniform(t.seed + (uint64_t)episode * kEpisodeStride, (uint64_t)env, (uint64_t)(1024 + 8 * frame + k));
}
__device__ inline int task_interval(const TaskParams& t, int env, int episode, int frame) {
  const int span = t.push_max_f - t.push_min_f + 1;
  const int d = t.push_min_f + (int)floorf(task_u(t, env, episode, frame, 2) * (float)span);
  return d > t.push_max_f ? t.push_max_f : d;
}
__device__ inline void task_draw_target(const TaskParams& t, int env, int episode, int frame, float rx, float ry,
                                        float* target_xy) {
  const float r = t.radius * sqrtf(task_u(t, env, episode, frame, 3));
  const float phi = 6.283185307179586f * task_u(t, env, episode, frame, 4);
  target_xy[0] = rx + r * cosf(phi);
  target_xy[1] = ry + r * sinf(phi);
}

// Seeded reset (Section 4.1: positions, velocities, joint angles and joint angular velocities
// perturbed slightly): the rest pose displaced by a uniform offset, every hinge angle and every
// hinge rate drawn uniformly (angles clamped to their limits), bodies placed parents-first
// through the joint list; the top of the tree gets one uniform linear velocity and no spin, a
// child turns with its parent plus its hinge rates and moves so that the two anchor points of its
// joint share one velocity (the world as a parent stands still).
// In the step kernel by a thread per body and joint: a joint's draws depend on nothing else, its child's pose
// on the parent's, so the joints are placed level by level (Model::joint_level).  In reset_kernel (sim_reset of
// many envs) by one thread per env, in the joints' order.
template <class Poses>
__device__ __forceinline__ void reset_place_body(const Model& M, int b, int env, uint64_t seed, Poses P) {
  const float noise = M.reset_noise;
  for (int c = 0; c < 3; ++c) {
    P.X(b, c) = fma_(noise, 2.0f * reset_uniform(seed, env, c) - 1.0f, M.bodies[b].rest_pos[c]);
    P.V(b, c) = noise * (2.0f * reset_uniform(seed, env, 3 + c) - 1.0f);
    P.W(b, c) = 0.0f;
  }
  for (int c = 0; c < 4; ++c) P.Q(b, c) = c == 0 ? 1.0f : 0.0f;
}
struct ResetDraw {
  float dq[4], rate[3];   // rotation of the child in the parent's frame, hinge rates
};
__device__ __forceinline__ void reset_draw_joint(const Model& M, int j, int env, uint64_t seed, ResetDraw& d) {
  const float a = M.reset_noise;
  const JointTab& jt = M.joints[j];
  float phi[3] = {0, 0, 0};
  for (int k = 0; k < 3; ++k) {
    d.rate[k] = 0.0f;
    if (jt.mode[k] != 1) continue;
    float th = a * (2.0f * reset_uniform(seed, env, 8 + 3 * j + k) - 1.0f);
    th = fminf(fmaxf(th, jt.lo[k]), jt.hi[k]);
    for (int c = 0; c < 3; ++c) phi[c] += th * jt.axes[k][c];
    d.rate[k] = a * (2.0f * reset_uniform(seed, env, 256 + 3 * j + k) - 1.0f);
  }
  const float ang = sqrtf(dot(phi, phi));
  if (ang < 1e-12f) { d.dq[0] = 1.0f; d.dq[1] = 0.5f * phi[0]; d.dq[2] = 0.5f * phi[1]; d.dq[3] = 0.5f * phi[2]; }
  else { const float sn = sinf(0.5f * ang) / ang; d.dq[0] = cosf(0.5f * ang); d.dq[1] = sn * phi[0]; d.dq[2] = sn * phi[1]; d.dq[3] = sn * phi[2]; }
}
// where the poses and velocities are built: in LDS, or in the state itself (its column of one env)
struct LdsPoses {
  float* Lpos; float* Lvel; int E, ee;
  __device__ float& X(int b, int c) { return Lpos[(b * 7 + c) * E + ee]; }
  __device__ float& Q(int b, int c) { return Lpos[(b * 7 + 3 + c) * E + ee]; }
  __device__ float& V(int b, int c) { return Lvel[(b * kVS + c) * E + ee]; }
  __device__ float& W(int b, int c) { return Lvel[(b * kVS + 3 + c) * E + ee]; }
};
struct StatePoses {
  float* st; size_t body, field;   // floats from one body, from one component to the next
  __device__ float& X(int b, int c) { return st[c * field + b * body]; }
  __device__ float& Q(int b, int c) { return st[(3 + c) * field + b * body]; }
  __device__ float& V(int b, int c) { return st[(7 + c) * field + b * body]; }
  __device__ float& W(int b, int c) { return st[(10 + c) * field + b * body]; }
};
// the child of one joint, from its parent
template <class Poses>
__device__ __forceinline__ void reset_place_joint(const JointTab& jt, const ResetDraw& d, Poses P) {
  float qa[4] = {1, 0, 0, 0}, xa[3] = {0, 0, 0}, va[3] = {0, 0, 0}, wa[3] = {0, 0, 0};
  if (jt.parent >= 0) {
    for (int c = 0; c < 4; ++c) qa[c] = P.Q(jt.parent, c);
    for (int c = 0; c < 3; ++c) { xa[c] = P.X(jt.parent, c); va[c] = P.V(jt.parent, c); wa[c] = P.W(jt.parent, c); }
  }
  const float* dq = d.dq;
  float qb[4];
  qb[0] = qa[0] * dq[0] - qa[1] * dq[1] - qa[2] * dq[2] - qa[3] * dq[3];
  qb[1] = qa[0] * dq[1] + qa[1] * dq[0] + qa[2] * dq[3] - qa[3] * dq[2];
  qb[2] = qa[0] * dq[2] - qa[1] * dq[3] + qa[2] * dq[0] + qa[3] * dq[1];
  qb[3] = qa[0] * dq[3] + qa[1] * dq[2] - qa[2] * dq[1] + qa[3] * dq[0];
  const float inv = 1.0f / sqrtf(qb[0] * qb[0] + qb[1] * qb[1] + qb[2] * qb[2] + qb[3] * qb[3]);
  for (int c = 0; c < 4; ++c) qb[c] *= inv;
  float Ra[9], Rb[9], t0[3], t1[3];
  quat_to_mat(qa, Ra);
  quat_to_mat(qb, Rb);
  mat_vec(Ra, jt.la, t0);
  mat_vec(Rb, jt.lb, t1);
  for (int c = 0; c < 4; ++c) P.Q(jt.child, c) = qb[c];
  for (int c = 0; c < 3; ++c) P.X(jt.child, c) = xa[c] + t0[c] - t1[c];
  float wb[3] = {wa[0], wa[1], wa[2]};
  for (int k = 0; k < 3; ++k) {
    if (jt.mode[k] != 1) continue;
    float ak[3];
    mat_vec(Ra, jt.axes[k], ak);
    for (int c = 0; c < 3; ++c) wb[c] += d.rate[k] * ak[c];
  }
  float ca[3], cb[3];
  cross(wa, t0, ca);
  cross(wb, t1, cb);
  for (int c = 0; c < 3; ++c) { P.W(jt.child, c) = wb[c]; P.V(jt.child, c) = va[c] + ca[c] - cb[c]; }
}
// Start of an episode for the task logic (Section 4.1): counters cleared, first push time and
// (flagrun) first target drawn around the root.
__device__ inline void task_begin_episode(const TaskParams& t, int32_t* __restrict__ task_i, float* __restrict__ targets,
                                          int env, int episode, float rx, float ry) {
  task_i[4 * env + 0] = 0; task_i[4 * env + 1] = 0;
  task_i[4 * env + 2] = t.push_max_f > 0 ? task_interval(t, env, episode, 0) : -1;
  task_i[4 * env + 3] = episode;
  if (t.period > 0) task_draw_target(t, env, episode, 0, rx, ry, targets + 2 * env);
}
// (squared distance, feature id) as one 64-bit word whose unsigned order is the lexicographic
// order of the pair (squared distances are non-negative, ids non-negative)
__device__ __forceinline__ unsigned long long pack_best(float d2, int id) {
  return ((unsigned long long)__float_as_uint(d2) << 32) | (unsigned)id;
}

// Number of set bits of a 64-bit lane mask below the calling lane.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}
// Reserves n (0 .. 2^kBits - 1) consecutive entries of a list for each active lane with one
// atomic per wavefront; every active lane has to call it.  Returns the lane's first index.
template <int kBits>
__device__ __forceinline__ int wave_alloc(int n, int* counter) {
  int before = 0, total = 0;
#pragma unroll
  for (int bit = 0; bit < kBits; ++bit) {
    const unsigned long long bm = __ballot((n >> bit) & 1);
    before += lanes_below(bm) << bit;
    total += __popcll(bm) << bit;
  }
  int base = 0;
  if (total > 0) {
    if (lanes_below(__ballot(1)) == 0) base = atomicAdd(counter, total);
    base = __builtin_amdgcn_readfirstlane(base);
  }
  return base + before;
}

#pragma clang fp contract(off)
// The same address of constant memory, as one that the compiler knows nothing about: what is read
// through it is read here, through the scalar cache.
template <class T>
__device__ __forceinline__ const T* reload_constant(const T* p) {
  auto c = (const __attribute__((address_space(4))) T*)p;
  asm volatile("" : "+s"(c));
  return (const T*)c;
}

// PC != 0: capsule-capsule contacts (within an agent and between the agents of a group) compiled in.
// NT: threads per workgroup.
// NS != 0: the rows are solved by the non-smooth Newton / conjugate-residual solver instead of
// the Jacobi sweeps (at most 8 envs per workgroup, every slot has a contact thread of its own).
// JL: lanes that relax one joint: one, two (one per side) or four (one per side and kind of row).
template <int EC, int NJ, int PC = 0, int NT = kThreads, int WS = 0, int NS = 0, int JL = 2>
__global__ __launch_bounds__(NT) void step_kernel(StepArgs a) {
  constexpr int kThreads = NT;   // (shadows the namespace-scope default inside the kernel)
#ifdef SIM_PHASE_TIMING
  long long t_last = clock64();
#endif
  extern __shared__ float lds[];
  const Model& M = *a.M;
  const int B = M.B, J = M.J, S = M.S, D = M.D, F = M.F;
  const int E = EC > 0 ? EC : a.E, N = a.N;
  const int tid = threadIdx.x;
  const int e = tid % E, idx = tid / E;
  const int env = blockIdx.x * E + e;   // the thread's place in the launch: a workgroup holds E consecutive places
  const bool env_ok = env < N;
  // Which agent stands at a place: the agent of the same number, unless the interaction groups were
  // chosen from the agents' positions (capsule-capsule variants only).  Everything in global memory
  // is indexed by agent, everything in LDS by the place within the workgroup.
  auto agent_at = [&](int place) -> int {
    if constexpr (PC != 0) { if (a.place_env && place < N) return a.place_env[place]; }
    return place;
  };
  const int agent = agent_at(env);
  const bool is_body = idx < B && env_ok;
  const bool is_joint = idx < J && env_ok;
  const int obs_dim = 11 + 3 * D + F;                                      // staged in LDS
  // model scalars the loops below use, read once (before the kernel's first store, so they come
  // through the scalar cache and stay in scalar registers)
  const int m_terrain = M.terrain_kind, m_contacts = M.contacts;
  const Field H0 = make_field(M, a.heights, a.coarse);
  const bool use_patch = m_terrain == 1 && H0.nx >= kPatch && H0.ny >= kPatch;
  const int m_group = PC ? (M.group > 1 ? M.group : 1) : 1, m_npairs = PC ? M.n_pairs : 0, m_nap = PC ? M.n_agent_pairs : 0;
  const LdsPlan P = make_plan(B, J, S, D, F, E, use_patch ? 2 : (m_terrain == 1 ? 1 : 0), PC ? m_group : 0, NT, WS, NS, JL);
  float* Lpos = lds + P.pos;
  float* Lvel = lds + P.vel;
  float* Liw = lds + P.iw;
  float* Lnb = lds + P.nb;
  float* Loutj = lds + P.outj;
  float* Loutc = lds + P.outc;
  int* Ltjs = reinterpret_cast<int*>(lds + P.tjs);  // body table: joint-side count, slot0, slot count, joint sides
  float* Lrec = lds + P.rec;
  int* Lreci = reinterpret_cast<int*>(lds + P.rec);
  int* Llist = reinterpret_cast<int*>(lds + P.list);
  int* Lsurv = reinterpret_cast<int*>(lds + P.surv);
  float* Llam = lds + P.lam;                         // impulses of the contacts beyond one per thread
  // fine search: per slot (index s * E + env) the minimum of (squared distance, feature id) packed in 64 bits,
  // half of every body's segment, and four lists (rows of cells and single cells, each for the end
  // spheres and for the mid-segments); all of it lives in the space of the changes the sweeps use
  unsigned long long* Lbest64 = reinterpret_cast<unsigned long long*>(lds + P.outj);
  float* Lhalf = lds + P.half;                       // [B][3][E]: from the centre to the segment's second end
  unsigned* Lcell_e = reinterpret_cast<unsigned*>(lds + P.cand);
  const int cap32 = P.cand_cap / 32, cell_e_cap = 6 * cap32, cell_m_cap = 10 * cap32, row_e_cap = 6 * cap32, row_m_cap = 10 * cap32;
  unsigned* Lcell_m = Lcell_e + cell_e_cap;
  unsigned* Lrow_e = Lcell_m + cell_m_cap;
  unsigned* Lrow_m = Lrow_e + row_e_cap;
  // Candidate pairs of the capsule-capsule search, in the space the observations are staged in at the end.
  unsigned* Lpair = reinterpret_cast<unsigned*>(lds + P.obs);
  const int pair_cap = (11 + 3 * D + F) * E;
  float* Ltq = lds + P.tq;                           // joint torques, [J][3][E]
  float* Lpush = lds + P.push;                       // external force on the root body, [3][E]
  float* Lu = lds + P.u;
  float* Lobs = lds + P.obs;
  int* Llim = reinterpret_cast<int*>(lds + P.lim);
  int* Lcount = reinterpret_cast<int*>(lds + P.count);
  int* Lporg = reinterpret_cast<int*>(lds + P.porg);
  float* Lpatch = lds + P.patch;
  float* Lmip = lds + P.mip;
  float* Lorg = lds + P.org;                          // env origins, [3][E]
  int* Ltslot = reinterpret_cast<int*>(lds + P.tslot);  // slot table: body, kind
  float* Ltbody = lds + P.tbody;                      // body table: radius, half length, axis, 1/mass
  float* Ltin = lds + P.tin;                          // body table: inertia(3), inverse inertia(3)
  const JointTab* Ltjoint = reinterpret_cast<const JointTab*>(lds + P.tjoint);  // joint table
  float* Lpq = lds + P.pq;                            // capsule-capsule contacts, kPairWords each, sorted by key
  float* Lpo = lds + P.po;                            // what they change: A (v, w), B (v, w)
  int* Lmeet = reinterpret_cast<int*>(lds + P.pnear);
  int* Lbs = reinterpret_cast<int*>(lds + P.pbs);     // bounding radii as float bits (ordered like ints)
  int* Lpcount = reinterpret_cast<int*>(lds + P.pcount);  // contacts found, near agent pairs
  int* Lpbcnt = reinterpret_cast<int*>(lds + P.pbcnt);
  uint8_t* Lpblist = reinterpret_cast<uint8_t*>(lds + P.pblist);
  // Warm start (WS != 0): the impulse every joint row ([J*6][E]; a limit row's carries the limit it
  // stood for in its sign, minus = upper) and every terrain slot row ([S*3][E]) ended the last
  // substep with.  Slots that were not active then hold zero.
  float* Lwj = lds + P.wj;
  float* Lwc = lds + P.wc;
  const float p_warm = WS ? M.warm : 0.0f;
  const float h = a.h;

  // ---- load: body state into registers, clipped actions into LDS
  // The heightfield samples around an env's root body are copied by a share of the threads of its own
  // (the whole robot stays within them during one step; anything outside falls back to global memory).
  // What decides where the copy starts is asked for before everything else, so that two trips to
  // memory, not three, lie between the launch and the copy.
  const bool copy_field = use_patch && a.substeps > 0;   // (a launch without substeps never searches the terrain)
  const int tpe = kThreads / E, pe = tid / tpe, pl = tid - pe * tpe;
  float root_wx = 0.0f, root_wy = 0.0f;
  if (copy_field && pe < E && blockIdx.x * E + pe < N) {
    const int ag = agent_at(blockIdx.x * E + pe);
    const float* st = a.state + (size_t)M.root * N + ag;
    root_wx = st[0] + a.origins[3 * ag]; root_wy = st[(size_t)B * N] + a.origins[3 * ag + 1];
  }
  float x[3] = {0, 0, 0}, q[4] = {1, 0, 0, 0}, v[3] = {0, 0, 0}, w[3] = {0, 0, 0};
  const int b = idx;
  if (is_body) {
    const float* st = a.state + (size_t)b * N + agent;
    const size_t fs = (size_t)B * N;
    x[0] = st[0 * fs]; x[1] = st[1 * fs]; x[2] = st[2 * fs];
    q[0] = st[3 * fs]; q[1] = st[4 * fs]; q[2] = st[5 * fs]; q[3] = st[6 * fs];
    v[0] = st[7 * fs]; v[1] = st[8 * fs]; v[2] = st[9 * fs];
    w[0] = st[10 * fs]; w[1] = st[11 * fs]; w[2] = st[12 * fs];
  }
  // First words of the small arrays (actions, origins, tables): asked for here, so that their trips to memory run beside
  // those of the state and of the heightfield instead of one after the other behind them.
  const int n_act = E * D, n_tab = M.table_words;
  const float inv_d = __builtin_amdgcn_rcpf((float)(D > 0 ? D : 1));
  auto action_of = [&](int i) -> float {   // (i < E D < 2^14, D <= 32: the quotient is exact)
    const int ee = (int)(((float)i + 0.5f) * inv_d), d = i - ee * D, env_i = blockIdx.x * E + ee;
    return env_i < N && a.actions ? a.actions[(size_t)agent_at(env_i) * D + d] : 0.0f;
  };
  auto origin_of = [&](int i) -> float {
    const int c = i / E, ee = i - c * E, env_i = blockIdx.x * E + ee;
    return env_i < N ? a.origins[3 * agent_at(env_i) + c] : 0.0f;
  };
  float act_0 = 0.0f, org_0 = 0.0f;
  if (tid < n_act) act_0 = action_of(tid);
  if (tid < 3 * E) org_0 = origin_of(tid);
  int tab_0 = M.table_image[tid < n_tab ? tid : 0], tab_1 = M.table_image[tid + kThreads < n_tab ? tid + kThreads : 0];
  if (copy_field && pe < E) {
    // four samples at a time (a row of the copy is seven of them; rows start at any sample), all of a
    // thread's reads in flight together
    constexpr int kQuads = kPatch * kPatch / 4, kShare = EC > 0 ? kThreads / EC : 64, kInFlight = (kQuads + kShare - 1) / kShare;
    typedef float quad __attribute__((ext_vector_type(4), aligned(4)));
    typedef float quad16 __attribute__((ext_vector_type(4)));
    float ci = floorf((root_wx - M.hox) * M.inv_cell), cj = floorf((root_wy - M.hoy) * M.inv_cell);
    ci = fminf(fmaxf(ci - (float)(kPatch / 2), 0.0f), (float)(M.nx - kPatch));
    cj = fminf(fmaxf(cj - (float)(kPatch / 2), 0.0f), (float)(M.ny - kPatch));
    const int i0 = (int)ci, j0 = (int)cj;
    if (pl == 0) { Lporg[2 * pe] = i0; Lporg[2 * pe + 1] = j0; }
    const float* h0 = a.heights + j0 * H0.nx + i0;
    for (int k0 = pl; k0 < kQuads; k0 += kInFlight * tpe) {
      quad hv[kInFlight];
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) {
        const int i = k0 + k * tpe < kQuads ? k0 + k * tpe : k0, row = i / (kPatch / 4), c4 = i - row * (kPatch / 4);
        hv[k] = *reinterpret_cast<const quad*>(h0 + row * H0.nx + 4 * c4);
      }
#pragma unroll
      for (int k = 0; k < kInFlight; ++k)
        if (k0 + k * tpe < kQuads) *reinterpret_cast<quad16*>(Lpatch + pe * (kPatch * kPatch) + 4 * (k0 + k * tpe)) = hv[k];
    }
  }
  // uniform parameters and this thread's joint, read once
  const float g0 = M.g[0], g1 = M.g[1], g2 = M.g[2];
  const float p_mu = M.mu, p_margin = M.margin, p_beta_j = M.beta_j, p_beta_c = M.beta_c;
  const float p_vdepen = M.v_depen, p_clin = M.c_lin, p_cang = M.c_ang, p_wmax = M.w_max;
  const int p_gyro = M.gyro;
  // small copies of what the per-slot code looks up all the time
  asm volatile("" : "+v"(act_0), "+v"(org_0), "+v"(tab_0), "+v"(tab_1));   // (all four on their way before the first store)
  auto put_action = [&](int i, float u) {
    const int ee = (int)(((float)i + 0.5f) * inv_d);
    Lu[(i - ee * D) * E + ee] = fminf(fmaxf(u, -1.0f), 1.0f);
  };
  int* const Ltab = reinterpret_cast<int*>(lds + P.tjs);
  if (tid < n_act) put_action(tid, act_0);
  if (tid < 3 * E) Lorg[tid] = org_0;
  if (tid < n_tab) Ltab[tid] = tab_0;
  if (tid + kThreads < n_tab) Ltab[tid + kThreads] = tab_1;
  for (int i = tid + kThreads; i < n_act; i += kThreads) put_action(i, action_of(i));
  for (int i = tid + kThreads; i < 3 * E; i += kThreads) Lorg[i] = origin_of(i);
  for (int i = tid + 2 * kThreads; i < n_tab; i += kThreads) Ltab[i] = M.table_image[i];
  // external pushes (Section 4.1): is this frame the env's next push?
  if (tid < E) {
    const bool env_t_ok = blockIdx.x * E + tid < N;
    const int env_t = agent_at(blockIdx.x * E + tid);
    float fx = 0.0f, fy = 0.0f;
    if (a.task.enabled && a.task.push_max_f > 0 && a.count_step && env_t_ok) {
      const int f = a.steps[env_t], ep = a.task_i[4 * env_t + 3];
      if (f == a.task_i[4 * env_t + 2]) {
        const float mag = a.task.push_min_n + (a.task.push_max_n - a.task.push_min_n) * task_u(a.task, env_t, ep, f, 0);
        const float phi = 6.283185307179586f * task_u(a.task, env_t, ep, f, 1);
        fx = mag * cosf(phi); fy = mag * sinf(phi);
        a.task_i[4 * env_t + 2] = f + task_interval(a.task, env_t, ep, f);
      }
    }
    Lpush[0 * E + tid] = fx; Lpush[1 * E + tid] = fy; Lpush[2 * E + tid] = 0.0f;
    if (a.task.enabled && a.count_step && env_t_ok) { a.push[3 * env_t] = fx; a.push[3 * env_t + 1] = fy; a.push[3 * env_t + 2] = 0.0f; }
  }
  if constexpr (PC == 0)
    for (int i = tid; i < 6 * E; i += kThreads) lds[P.zero + i] = 0.0f;
  if (tid < 8) Lcount[tid] = 0;
  if constexpr (WS != 0) {
    for (int i = tid; i < J * 6 * E; i += kThreads) {
      const int env_i = blockIdx.x * E + i % E;
      Lwj[i] = env_i < N ? a.lam_j[(size_t)(i / E) * N + agent_at(env_i)] : 0.0f;
    }
    for (int i = tid; i < S * 3 * E; i += kThreads) {
      const int env_i = blockIdx.x * E + i % E;
      Lwc[i] = env_i < N ? a.lam_s[(size_t)(i / E) * N + agent_at(env_i)] : 0.0f;
    }
  }
  if constexpr (PC != 0) {
    if (tid < 12) Lpo[kPairCap * 12 + tid] = 0.0f;   // the entry unused list slots point at
  }
  // a step without substeps packs "no contact" (otherwise the contact phase clears what it does not set)
  if (a.substeps == 0)
    for (int i = tid; i < S * E; i += kThreads) Lreci[(i / E * kRecWords + 0) * E + i % E] = 0;

  if (copy_field) {
    __syncthreads();
    for (int i = tid; i < E * kPatchBlocks * kPatchBlocks; i += kThreads) {
      int ee = i / (kPatchBlocks * kPatchBlocks), r = i - ee * (kPatchBlocks * kPatchBlocks);
      int bj = r / kPatchBlocks, bi = r - bj * kPatchBlocks;
      // (kMip+1)^2 samples, indices clamped into the copy, all reads issued before the first use
      float hv[(kMip + 1) * (kMip + 1)];
#pragma unroll
      for (int dj = 0; dj <= kMip; ++dj)
#pragma unroll
        for (int di = 0; di <= kMip; ++di) {
          const int pj = bj * kMip + dj < kPatch ? bj * kMip + dj : kPatch - 1;
          const int pi = bi * kMip + di < kPatch ? bi * kMip + di : kPatch - 1;
          hv[dj * (kMip + 1) + di] = Lpatch[ee * (kPatch * kPatch) + pj * kPatch + pi];
        }
      __builtin_amdgcn_sched_group_barrier(0x100, (kMip + 1) * (kMip + 1), 0);
      float hm = -INFINITY;
#pragma unroll
      for (int k = 0; k < (kMip + 1) * (kMip + 1); ++k) hm = fmaxf(hm, hv[k]);
      Lmip[i] = hm;
    }
  }

  // phase A reads what other wavefronts copied (tables, counters, block maxima)
  __syncthreads();
  TMARK(0);
  // wavefronts [0, joint_threads/64) hold the joint-side threads; contact k of a workgroup goes
  // to thread kThreads-1-k as long as that thread is not in a joint wavefront (n_reg contacts)
  const int joint_threads = ((JL * J * E + 63) / 64) * 64;
  const int n_reg = kThreads - joint_threads;
  const bool joint_wave = __builtin_amdgcn_readfirstlane(tid) < joint_threads;
  // joint-side role: JL neighbouring lanes for pair p = (joint, env); the lowest bit says whether a lane is on the
  // parent's or the child's side, with four lanes the next one whether it has the positional or the angular rows
  const int js_side = JL > 1 ? tid & 1 : 0, js_kind = JL == 4 ? (tid >> 1) & 1 : 0, js_e = (tid / JL) % E, js_j = (tid / JL) / E;
  const bool js_on = js_j < J && blockIdx.x * E + js_e < N;

  // the heightfield with the env's copy of it
  auto field_of = [&](int ee) -> Field {
    Field H = H0;
    if (use_patch) {
      H.patch = (const lds_float*)(Lpatch + ee * (kPatch * kPatch)); H.mip = (const lds_float*)(Lmip + ee * (kPatchBlocks * kPatchBlocks));
      H.pi0 = Lporg[2 * ee]; H.pj0 = Lporg[2 * ee + 1]; H.ps = kPatch;
    }
    return H;
  };
  // geometry of one slot, from what phase A left in LDS
  auto listed_geom = [&](int bb, int ee, int kind) -> SlotGeom {
    const float bx[3] = {Lpos[(bb * 7 + 0) * E + ee], Lpos[(bb * 7 + 1) * E + ee], Lpos[(bb * 7 + 2) * E + ee]};
    const float bo[3] = {Lorg[ee], Lorg[E + ee], Lorg[2 * E + ee]};
    const float* lh = Lhalf + bb * 3 * E + ee;
    return slot_geom_from_half(Ltbody[4 * bb], p_margin, bx, f3{lh[0], lh[E], lh[2 * E]}, kind, bo);
  };

  // Capsule-capsule candidates of this thread, the same in every substep: its first four body pairs within its
  // agent (a byte each) and its agent pair.  Read from the model's tables in global memory inside the
  // substep, each of them was a trip to the cache that the whole workgroup waited for.
  const int pair_stride = kThreads / E;
  unsigned my_pairs = 0;
  int my_meet = 0;
  if constexpr (PC != 0) {
    if (idx < pair_stride)
      for (int k = 0; k < 4; ++k)
        if (idx + k * pair_stride < m_npairs)
          my_pairs |= (unsigned)(M.pair_a[idx + k * pair_stride] << 4 | M.pair_b[idx + k * pair_stride]) << (8 * k);
    const int t = kThreads - 1 - tid;
    if (m_group > 1 && t < (E / m_group) * m_nap) {
      const int gi = t / m_nap, pi = t - gi * m_nap;
      my_meet = (gi * m_group + M.agent_pair_a[pi]) | ((gi * m_group + M.agent_pair_b[pi]) << 16);
    }
  }
  const int tid_o = tid, e_o = e, idx_o = idx;
  const float h_o = h;
  for (int sub = 0; sub < a.substeps; ++sub) {
    // In the variants that are short of registers (capsule-capsule collisions, or the wide workgroup
    // with its 170 VGPRs per thread) the thread's indices and the time step are passed through empty
    // asm statements at the top of each substep: what is derived from them (LDS addresses, h-scaled
    // constants) is then recomputed per substep instead of being computed once before the loop and
    // kept alive across it.  The others have registers to spare and let the compiler hoist.
    // row constants of this substep (declared here: nothing of them is carried into the next one)
    SideRows jr;
    ContactRows cr;
    PairSide pr;
    bool has_contact = false;  // this thread owns an active contact this substep
    int tid = tid_o, e = e_o, idx = idx_o;
    float h = h_o;
    if constexpr (PC != 0 || NT > 512 || NS != 0) {
      asm volatile("" : "+v"(tid), "+v"(e), "+v"(idx));
      asm volatile("" : "+s"(h));
    }
    const int b = idx;
    // ---- A: publish pose and world inverse inertia
    if (tid == 0) Lcount[0] = 0;
    if constexpr (PC != 0) {
      if (tid < 4) Lpcount[tid] = 0;
      if (tid < E) Lbs[tid] = 0;
      for (int i = tid; i < B * E; i += kThreads) Lpbcnt[i] = 0;
    }
    if (is_body) {
      for (int c = 0; c < 3; ++c) Lpos[(b * 7 + c) * E + e] = x[c];
      for (int c = 0; c < 4; ++c) Lpos[(b * 7 + 3 + c) * E + e] = q[c];
      // velocities are parked in LDS as well: nothing of the body stays in registers while the
      // contact phases run
      for (int c = 0; c < 3; ++c) { Lvel[(b * kVS + c) * E + e] = v[c]; Lvel[(b * kVS + 3 + c) * E + e] = w[c]; }
      float R[9], invIb[3];
      quat_to_mat(q, R);
      for (int c = 0; c < 3; ++c) invIb[c] = Ltin[6 * b + 3 + c];
      float iw[6];
      iw[0] = sum3(R[0] * R[0], invIb[0], R[1] * R[1], invIb[1], R[2] * R[2], invIb[2]);
      iw[1] = sum3(R[0] * R[3], invIb[0], R[1] * R[4], invIb[1], R[2] * R[5], invIb[2]);
      iw[2] = sum3(R[0] * R[6], invIb[0], R[1] * R[7], invIb[1], R[2] * R[8], invIb[2]);
      iw[3] = sum3(R[3] * R[3], invIb[0], R[4] * R[4], invIb[1], R[5] * R[5], invIb[2]);
      iw[4] = sum3(R[3] * R[6], invIb[0], R[4] * R[7], invIb[1], R[5] * R[8], invIb[2]);
      iw[5] = sum3(R[6] * R[6], invIb[0], R[7] * R[7], invIb[1], R[8] * R[8], invIb[2]);
      for (int c = 0; c < 6; ++c) Liw[(b * kVS + c) * E + e] = iw[c];
      if (m_terrain == 1) {
        const f3 a = body_half(q, Ltbody[4 * b + 1], __float_as_int(Ltbody[4 * b + 2]));
        Lhalf[(b * 3 + 0) * E + e] = a.x; Lhalf[(b * 3 + 1) * E + e] = a.y; Lhalf[(b * 3 + 2) * E + e] = a.z;
      }
    }
    __syncthreads();

    TMARK(1);
    // ---- B: joint torques (stored once per joint; the body applies the sign) by the threads from tq_base on
    auto torques = [&](int tq_base) {
      const int tj = (tid - tq_base) / E, te = (tid - tq_base) % E;
      if (tid >= tq_base && tj < J && blockIdx.x * E + te < N) {
        const JointTab& jt = Ltjoint[tj];
        float qa[4] = {1, 0, 0, 0};
        if (jt.parent >= 0)
          for (int c = 0; c < 4; ++c) qa[c] = Lpos[(jt.parent * 7 + 3 + c) * E + te];
        float Ra[9];
        quat_to_mat(qa, Ra);
        float tq[3] = {0, 0, 0};
        for (int k = 0; k < 3; ++k) {
          if (jt.mode[k] != 1) continue;
          float ak[3];
          mat_vec(Ra, jt.axes[k], ak);
          float t = jt.gear[k] * Lu[jt.act[k] * E + te];
          for (int c = 0; c < 3; ++c) tq[c] = fma_(t, ak[c], tq[c]);
        }
        for (int c = 0; c < 3; ++c) Ltq[(tj * 3 + c) * E + te] = tq[c];
      }
    };
    // forces -> velocities (torques, gravity, push, explicit gyroscopic term): needs the joint torques and
    // nothing of the contacts.  Threads from t0 up; entry i is body i / E of env i % E.
    auto forces = [&](int t0) {
     for (int i = tid - t0; i >= 0 && i < B * E; i += kThreads - t0) {
      const int e = i % E, b = i / E;
      if (blockIdx.x * E + e >= N) continue;
      float tau[3] = {0, 0, 0};
      const int njs = Ltjs[b * (kMaxBodyJoints + 3)];
      for (int k = 0; k < njs; ++k) {
        const int js = Ltjs[b * (kMaxBodyJoints + 3) + 3 + k];
        const float sg = (js & 1) ? 1.0f : -1.0f;
        for (int c = 0; c < 3; ++c) tau[c] = fma_(sg, Ltq[((js >> 1) * 3 + c) * E + e], tau[c]);
      }
      float R[9], qq[4], Ib[3], invIb[3], v[3], w[3];
      for (int c = 0; c < 4; ++c) qq[c] = Lpos[(b * 7 + 3 + c) * E + e];
      quat_to_mat(qq, R);
      for (int c = 0; c < 3; ++c) { Ib[c] = Ltin[6 * b + c]; invIb[c] = Ltin[6 * b + 3 + c]; }
      for (int c = 0; c < 3; ++c) { v[c] = Lvel[(b * kVS + c) * E + e]; w[c] = Lvel[(b * kVS + 3 + c) * E + e]; }
      if (a.task.enabled && b == M.root) {
        const float him = h * Ltbody[4 * b + 3];
        for (int c = 0; c < 3; ++c) v[c] = fma_(him, Lpush[c * E + e], v[c]);
      }
      v[0] = fma_(h, g0, v[0]); v[1] = fma_(h, g1, v[1]); v[2] = fma_(h, g2, v[2]);
      float wb[3], tb[3];
      mat_t_vec(R, w, wb);
      mat_t_vec(R, tau, tb);
      float Iw[3] = {Ib[0] * wb[0], Ib[1] * wb[1], Ib[2] * wb[2]};
      float gy[3];
      cross(wb, Iw, gy);
      if (!p_gyro) { gy[0] = gy[1] = gy[2] = 0.0f; }
      // only the increment goes back to the world frame (the velocity itself is not rotated
      // there and back, which would round it six times more)
      float dwb[3], dww[3];
      for (int c = 0; c < 3; ++c) dwb[c] = h * (tb[c] - gy[c]) * invIb[c];
      mat_vec(R, dwb, dww);
      for (int c = 0; c < 3; ++c) w[c] += dww[c];
      for (int c = 0; c < 3; ++c) { Lvel[(b * kVS + c) * E + e] = v[c]; Lvel[(b * kVS + 3 + c) * E + e] = w[c]; }
     }
    };
    // bounding radius of every agent about its root, for the pairs of agents below
    auto agent_radius = [&](int t0) {
      for (int i = tid - t0; i >= 0 && i < B * E; i += kThreads - t0) {
        const int e = i % E, b = i / E;
        if (blockIdx.x * E + e >= N) continue;
        float dx[3];
        for (int c = 0; c < 3; ++c) dx[c] = Lpos[(b * 7 + c) * E + e] - Lpos[(M.root * 7 + c) * E + e];
        const float rad = __builtin_amdgcn_sqrtf(dot(dx, dx)) * 1.000001f + Ltbody[4 * b + 1] + Ltbody[4 * b];
        atomicMax(&Lbs[e], __float_as_int(rad));
      }
    };
    if (m_terrain == 0) {
      // plane: the torques from the lower end of the workgroup, every slot's contact from the upper one
      torques(0);
      if (PC != 0 && m_group > 1) agent_radius(0);
      for (int i = kThreads - 1 - tid; i < S * E; i += kThreads) {
        const int ee = i % E, s = i / E;
        ContactOut co = no_contact();
        if (blockIdx.x * E + ee < N && m_contacts) {
          const SlotTab sl{Ltslot[2 * s], Ltslot[2 * s + 1]};
          float bx[3], bq[4], bo[3];
          for (int c = 0; c < 3; ++c) bx[c] = Lpos[(sl.body * 7 + c) * E + ee];
          for (int c = 0; c < 4; ++c) bq[c] = Lpos[(sl.body * 7 + 3 + c) * E + ee];
          for (int c = 0; c < 3; ++c) bo[c] = Lorg[c * E + ee];
          const SlotGeom g = slot_geom(Ltbody[4 * sl.body], Ltbody[4 * sl.body + 1], __float_as_int(Ltbody[4 * sl.body + 2]),
                                       p_margin, bx, bq, sl.kind, bo);
          co = plane_contact(g, p_margin);
        }
        if (co.active) {
          store_record(Lrec, Lreci, s, ee, E, co);
          Llist[atomicAdd(&Lcount[0], 1)] = i;
        } else {
          Lreci[(s * kRecWords + 0) * E + ee] = 0;      // the other words of an inactive record are not read
          Lrec[(s * kRecWords + 10) * E + ee] = 0.0f;
        }
      }
      TMARK(2);
    } else {
      // ---- B1: one thread per slot (end spheres, then mid-segments in wavefronts of their own): reach
      //          box against the block maxima of the heightfield copy.  A slot that may touch the field is
      //          queued (end spheres from the front of the queue, mid-segments from the back) and the rows
      //          of its box are listed; an end sphere's box is first cut down to what can be nearer than
      //          the ground straight below its centre.  Box and reach stay in the slot's unused record.
      {
        const int t_mid = (2 * B * E + 63) & ~63;
        for (int t = tid; t < t_mid + B * E; t += kThreads) {
          const bool mid = t >= t_mid;
          if (!mid && t >= 2 * B * E) continue;
          const int r = mid ? t - t_mid : t, ee = r % E, bk = r / E, bb = mid ? bk : bk >> 1;
          const int s0 = Ltjs[bb * (kMaxBodyJoints + 3) + 1], ns = Ltjs[bb * (kMaxBodyJoints + 3) + 2];
          // a capsule's slots are its two ends and its interior, a sphere has the second end's alone
          const int kind = mid ? 2 : bk & 1;
          bool on = mid ? ns == 3 : ns > 1 || kind == 1;
          const int s = s0 + (ns == 1 ? 0 : kind), i = s * E + ee;
          int n_rows = 0;
          if (on) {
            Lreci[(s * kRecWords + 0) * E + ee] = 0;      // the other words of an inactive record are not read
            Lrec[(s * kRecWords + 10) * E + ee] = 0.0f;
            on = false;
            if (blockIdx.x * E + ee < N && m_contacts) {
              const Field H = field_of(ee);
              SlotGeom g = listed_geom(bb, ee, kind);
              if (slot_reach(H, g)) {
                on = true;
                float r2;
                const bool search = slot_search_box(H, g, r2);
                const int ni = g.i1 - g.i0 + 1, nj = g.j1 - g.j0 + 1;
                const bool fits = ni >= 1 && ni <= 15 && nj >= 1 && nj <= 15 && g.i0 < 4096 && g.j0 < 4096;
                Lreci[(s * kRecWords + 1) * E + ee] = g.i0 | (g.j0 << 12) | (ni << 24) | (nj << 28);
                Lrec[(s * kRecWords + 2) * E + ee] = r2;
                Lreci[(s * kRecWords + 8) * E + ee] = search && !fits ? 1 : 0;   // 1: search this slot the slow way
                if (search && !fits) Lcount[4] = 1;
                n_rows = search && fits ? nj : 0;
                Lbest64[i] = ~0ull;
              }
            }
          }
          if (on) Lsurv[mid ? S * E - 1 - atomicAdd(&Lcount[2], 1) : atomicAdd(&Lcount[1], 1)] = i;
          const int cap = mid ? row_m_cap : row_e_cap, r0 = wave_alloc<4>(n_rows, &Lcount[mid ? 6 : 5]);
          unsigned* U = mid ? Lrow_m : Lrow_e;
          if (r0 + n_rows <= cap) {
            for (int k = 0; k < n_rows; ++k) U[r0 + k] = (unsigned)i | ((unsigned)k << 20);
          } else {
            for (int k = r0; k < cap; ++k) U[k] = (unsigned)i | (15u << 20);   // (a row past every box)
            Lreci[(s * kRecWords + 8) * E + ee] = 1;
            Lcount[4] = 1;
          }
        }
      }
      torques(kThreads - ((J * E + 63) & ~63));   // (beside the slots; 2 J E threads fit below)
      TMARK(2);
      __syncthreads();
      TMARK(24);
      // ---- B2: fine search in two stages.  Stage 1: one row of a box per thread: which of its cells can
      //          hold a triangle within reach of the end sphere, or an edge within reach of the segment
      //          (conservative tests, from the corner heights).  Those are listed.  Stage 2: one triangle /
      //          edge of a listed cell per thread: exact distance, minimum of (d2, id) per slot with a
      //          64-bit LDS atomic.
      const int n_end = Lcount[1], n_mid = Lcount[2];
      {
        const int n_re = Lcount[5] < row_e_cap ? Lcount[5] : row_e_cap, n_rm = Lcount[6] < row_m_cap ? Lcount[6] : row_m_cap;
        const int t_mid = (n_re + 63) & ~63;
        for (int t = tid; t < t_mid + n_rm; t += kThreads) {
          const bool mid = t >= t_mid;
          if (!mid && t >= n_re) continue;
          const unsigned uw = mid ? Lrow_m[t - t_mid] : Lrow_e[t];
          const int i = uw & 4095, row = (int)(uw >> 20), ee = i % E, s = i / E, bb = Ltslot[2 * s];
          const unsigned box = (unsigned)Lreci[(s * kRecWords + 1) * E + ee];
          const float r2 = Lrec[(s * kRecWords + 2) * E + ee];
          const int i0 = box & 4095, j0 = (box >> 12) & 4095, ni = (box >> 24) & 15, nj = box >> 28;
          const Field H = field_of(ee);
          const SlotGeom g = listed_geom(bb, ee, mid ? 2 : Ltslot[2 * s + 1]);
          if (row >= nj) continue;
          const int cells = mid ? kSegCells : kEndCells;
          for (int col = 0; col < ni; col += cells) {
            unsigned m = mid ? cells_near_segment(H, g, r2, i0 + col, j0 + row, ni - col)
                             : cells_near_sphere(H, g.kind == 0 ? g.P0 : g.P1, r2, i0 + col, j0 + row, ni - col);
            int pos = wave_alloc<3>(__popc(m), &Lcount[mid ? 7 : 3]);
            const int cap = mid ? cell_m_cap : cell_e_cap;
            unsigned* C = mid ? Lcell_m : Lcell_e;
            unsigned cw = (unsigned)i | ((unsigned)row << 20) | ((unsigned)col << 16);
            if (m && pos + __popc(m) > cap) {
              // list full: the slot is searched again by the fallback below
              for (; pos < cap; ++pos) C[pos] = cw;
              Lreci[(s * kRecWords + 8) * E + ee] = 1;
              Lcount[4] = 1;
              m = 0;
            }
            for (; m; m &= m - 1) C[pos++] = cw + ((unsigned)(__ffs(m) - 1) << 16);
          }
        }
      }
      TMARK(10);
      __syncthreads();
      TMARK(25);
      {
        const int t_end = 2 * (Lcount[3] < cell_e_cap ? Lcount[3] : cell_e_cap), t_mid = (t_end + 63) & ~63;
        const int t_all = t_mid + 3 * (Lcount[7] < cell_m_cap ? Lcount[7] : cell_m_cap);
        for (int t = tid; t < t_all; t += kThreads) {
          const bool mid = t >= t_mid;
          if (!mid && t >= t_end) continue;
          const int c = mid ? (t - t_mid) / 3 : t >> 1, k = mid ? (t - t_mid) - 3 * c : t & 1;
          const unsigned cw = mid ? Lcell_m[c] : Lcell_e[c];
          const int i = cw & 4095, ee = i % E, s = i / E, bb = Ltslot[2 * s];
          const unsigned box = (unsigned)Lreci[(s * kRecWords + 1) * E + ee];
          const int ci = (int)(box & 4095) + (int)((cw >> 16) & 15), cj = (int)((box >> 12) & 4095) + (int)((cw >> 20) & 15);
          const Field H = field_of(ee);
          const SlotGeom g = listed_geom(bb, ee, mid ? 2 : Ltslot[2 * s + 1]);
          float d2;
          if (!mid) {
            if (sphere_tri_d2(H, g.kind == 0 ? g.P0 : g.P1, ci, cj, k, d2))
              atomicMin(&Lbest64[i], pack_best(d2, 2 * (cj * (H.nx - 1) + ci) + k));
          } else if ((k == 1 || ci < H.nx - 1) && (k == 0 || cj < H.ny - 1)) {   // (the last row and column have no cell of their own)
            if (segment_edge_d2(H, g.P0, g.P1, ci, cj, k, d2)) atomicMin(&Lbest64[i], pack_best(d2, 3 * (cj * H.nx + ci) + k));
          }
        }
      }
      __syncthreads();
      TMARK(13);
      if (Lcount[4]) {
        // rare: a box too large for the packed indices, or a full list: those slots are searched
        // directly, kGroup lanes per slot
        const int grp = tid / kGroup, gl = tid % kGroup;
        for (int sv = grp; sv < n_end + n_mid; sv += kThreads / kGroup) {
          const int i = Lsurv[sv < n_end ? sv : S * E - 1 - (sv - n_end)];
          const int ee = i % E, s = i / E;
          if (!Lreci[(s * kRecWords + 8) * E + ee]) continue;
          const Field H = field_of(ee);
          SlotGeom g = listed_geom(Ltslot[2 * s], ee, Ltslot[2 * s + 1]);
          slot_range(H, g);
          float best = INFINITY;
          int best_id = -1;
          if (g.kind < 2) {
            const f3 Pc = g.kind == 0 ? g.P0 : g.P1;
            const int ni = g.i1 - g.i0 + 1, nc = ni * (g.j1 - g.j0 + 1);
            for (int c = gl; c < nc; c += kGroup) sphere_cell(H, Pc, g.Rq, g.i0 + c % ni, g.j0 + c / ni, best, best_id);
          } else {
            const int ni = g.i1 - g.i0 + 2, nc = ni * (g.j1 - g.j0 + 2);
            const SegCull sc = seg_cull(g);
            for (int c = gl; c < nc; c += kGroup) segment_vertex(H, g, sc, g.i0 + c % ni, g.j0 + c / ni, best, best_id);
          }
          if (best_id >= 0) atomicMin(&Lbest64[i], pack_best(best, best_id));
        }
        __syncthreads();
      }
#ifdef SIM_PHASE_TIMING
      if (tid == 0 && blockIdx.x == 7) { a.dbg[14] += Lcount[5]; a.dbg[20] += Lcount[6]; a.dbg[15] += Lcount[3]; a.dbg[11] += Lcount[7]; a.dbg[21] += n_end; a.dbg[22] += n_mid; }
#endif
      // ---- B3: one thread per queued slot turns the selected feature into a contact record (end spheres,
      //          then mid-segments in wavefronts of their own, so that a wavefront follows one path), from
      //          the lower end of the workgroup up, while the forces are integrated from its upper end down
      {
        const int t_mid = (n_end + 63) & ~63;
          for (int x = tid; x < t_mid + n_mid; x += kThreads) {
            const bool mids = x >= t_mid;
            if (!mids && x >= n_end) continue;
            const int i = Lsurv[mids ? S * E - 1 - (x - t_mid) : x], ee = i % E, s = i / E;
            const SlotGeom g = listed_geom(Ltslot[2 * s], ee, Ltslot[2 * s + 1]);
            const Field H = field_of(ee);
            ContactOut co = no_contact();
            const unsigned long long bw = Lbest64[i];
            const float bestd = __uint_as_float((unsigned)(bw >> 32));
            const int besti = (int)(unsigned)bw;
            if (!mids) {
              // a centre underneath the surface overrides the nearest-triangle search
              if (!underneath_contact(H, g, p_margin, co)) co = finish_sphere(H, g, p_margin, bestd, besti);
            } else {
              co = finish_segment(H, g, p_margin, bestd, besti);
            }
            if (co.active) {
              store_record(Lrec, Lreci, s, ee, E, co);
              Llist[atomicAdd(&Lcount[0], 1)] = i;
            }
          }
        TMARK(12);
        forces(kThreads - ((B * E + 63) & ~63));
        if (PC != 0 && m_group > 1) agent_radius(kThreads - ((B * E + 63) & ~63));
      }
    }
    __syncthreads();
    TMARK(3);

    // ---- P: capsule-capsule contacts from the poses published in phase A (Section 3.1: contacts
    //         among bodies; Section 4.1: inter-agent collisions).  Candidates: the listed body pairs
    //         of every agent, and every body pair of two agents of one group whose bounding spheres
    //         overlap.  A candidate passes a bounding-sphere test (stage 1, which compacts the
    //         survivors into a list), then the segment-segment test in the fixed operation order
    //         (stage 2, one survivor per lane); hits are queued and the queue is sorted by key, so
    //         that the order in which the bodies later add up their contacts does not depend on which
    //         wavefront found what first.
    int n_pc = 0;
    if constexpr (PC != 0) {
      const bool search = m_contacts && (m_npairs > 0 || m_group > 1);
      // (plane: the torques are complete by now, and most of the workgroup has no candidate in stage 2)
      auto plane_forces = [&]() {
        if (m_terrain == 0) forces(kThreads - ((B * E + 63) & ~63));
      };
      if (!search) plane_forces();
      if (search) {
        // Bounding spheres of the bodies for stage 1: centre relative to the group's first origin, radius
        // (enlarged by what the centre's two roundings can be off), one 16-byte word each, env after env
        // with an odd stride, so that a candidate costs two reads from LDS instead of sixteen and neighbouring
        // lanes fall on different banks.  They lie where the terrain search was and the sweeps' changes will be.
        float4* const Lsph = reinterpret_cast<float4*>(lds + ((P.outj + 3) & ~3));
        const int sph_e = B | 1;
        for (int i = tid; i < B * E; i += kThreads) {
          const int e = i % E, b = i / E, e0 = e - e % m_group;
          float4 w;
          w.x = Lpos[(b * 7 + 0) * E + e] + (Lorg[0 * E + e] - Lorg[0 * E + e0]);
          w.y = Lpos[(b * 7 + 1) * E + e] + (Lorg[1 * E + e] - Lorg[1 * E + e0]);
          w.z = Lpos[(b * 7 + 2) * E + e] + (Lorg[2 * E + e] - Lorg[2 * E + e0]);
          w.w = fma_(0x1p-22f, fabsf(w.x) + fabsf(w.y) + fabsf(w.z), (Ltbody[4 * b] + Ltbody[4 * b + 1]) + 0.5f * p_margin + 1e-3f);
          Lsph[e * sph_e + b] = w;
        }
        // agents of one group whose bounding spheres overlap, from the upper end of the workgroup
        if (m_group > 1) {
          const int n_ap = (E / m_group) * m_nap;
          for (int t = kThreads - 1 - tid; t < n_ap; t += kThreads) {
            int pr = my_meet;
            if (t >= kThreads) {   // (more pairs than threads)
              const int gi = t / m_nap, pi = t - gi * m_nap;
              pr = (gi * m_group + M.agent_pair_a[pi]) | ((gi * m_group + M.agent_pair_b[pi]) << 16);
            }
            const int ea = pr & 0xffff, eb = pr >> 16;
            bool near = false;
            if (blockIdx.x * E + eb < N) {   // (ea < eb)
              float dd = 0.0f;
              for (int c = 0; c < 3; ++c) {
                const float dc = (Lpos[(M.root * 7 + c) * E + eb] + Lorg[c * E + eb]) - (Lpos[(M.root * 7 + c) * E + ea] + Lorg[c * E + ea]);
                dd += dc * dc;
              }
              const float rr = __int_as_float(Lbs[ea]) + __int_as_float(Lbs[eb]) + p_margin + 2e-3f;
              near = dd <= rr * rr;
            }
            const int pos = wave_alloc<1>(near ? 1 : 0, &Lpcount[1]);
            if (near) Lmeet[pos] = pr;
          }
        }
        float* Ltmp = Lpo;   // unsorted queue; the changes are not in use yet
        // Every hit also leaves (gap, key) as one 64-bit word whose unsigned order is that of the
        // pair: when a workgroup finds more than it can hold, the kPairCap contacts with the smallest
        // gap stay (ties: smaller key), whichever wavefront found what first.  Where they live:
        // see make_plan.
        unsigned long long* Lhit = reinterpret_cast<unsigned long long*>(lds + P.phit);
        const int hit_cap = P.hit_cap;
        // the segment-segment test of one candidate pair from the poses of phase A
        auto eval_pair = [&](int ea, int ba, int eb, int bb, float& sp, float& tp, float& gap) -> bool {
          float xa[3], xb[3], off[3];
          for (int c = 0; c < 3; ++c) {
            off[c] = Lorg[c * E + eb] - Lorg[c * E + ea];
            xa[c] = Lpos[(ba * 7 + c) * E + ea];
            xb[c] = Lpos[(bb * 7 + c) * E + eb];
          }
          const float radA = Ltbody[4 * ba], hlA = Ltbody[4 * ba + 1], radB = Ltbody[4 * bb], hlB = Ltbody[4 * bb + 1];
          float dd = 0.0f;
          for (int c = 0; c < 3; ++c) { const float dc = (xb[c] + off[c]) - xa[c]; dd += dc * dc; }
          const float reach = (radA + hlA) + (radB + hlB) + p_margin + 2e-3f;
          if (!(dd <= reach * reach)) return false;
          float qa[4], qb[4];
          for (int c = 0; c < 4; ++c) { qa[c] = Lpos[(ba * 7 + 3 + c) * E + ea]; qb[c] = Lpos[(bb * 7 + 3 + c) * E + eb]; }
          f3 p0, p1, q0, q1;
          body_ends(xa, qa, hlA, __float_as_int(Ltbody[4 * ba + 2]), p0, p1);
          body_ends(xb, qb, hlB, __float_as_int(Ltbody[4 * bb + 2]), q0, q1);
          return pair_in_contact(p0, p1, q0, q1, off, radA, radB, p_margin, sp, tp, gap);
        };
        auto store_hit = [&](int pos, int ea, int ba, int eb, int bb, unsigned key, float sp, float tp, float gap) {
          Ltmp[pos * kPairWords + 0] = __uint_as_float(key);
          Ltmp[pos * kPairWords + 1] = __int_as_float((ba * E + ea) | ((bb * E + eb) << 16));
          Ltmp[pos * kPairWords + 2] = sp;
          Ltmp[pos * kPairWords + 3] = tp;
          Ltmp[pos * kPairWords + 4] = block_weight(p_margin, gap, 1.0f);
          Ltmp[pos * kPairWords + 5] = gap;
        };
        auto test_pair = [&](int ea, int ba, int eb, int bb, unsigned key, bool valid) {
          float sp = 0.0f, tp = 0.0f, gap = 0.0f;
          const bool hit = valid && eval_pair(ea, ba, eb, bb, sp, tp, gap);
          const int pos = wave_alloc<1>(hit ? 1 : 0, &Lpcount[0]);
          if (hit && pos < kPairCap) store_hit(pos, ea, ba, eb, bb, key, sp, tp, gap);
          if (hit && pos < hit_cap) {
            const unsigned gb = __float_as_uint(gap);
            const unsigned ordered = (gb & 0x80000000u) ? ~gb : (gb | 0x80000000u);   // unsigned order = float order
            Lhit[pos] = ((unsigned long long)ordered << 32) | key;
          }
        };
        // Stage 1: bounding spheres of the two capsules only; what passes is listed as a packed word
        // (env and body of A, env and body of B: also the sort key of a hit).  The list lives where
        // the observations are staged at the end of the step.
        unsigned* Lc2 = Lpair;
        auto near_pair = [&](int ea, int ba, int eb, int bb) -> bool {
          const float4 sa = Lsph[ea * sph_e + ba], sb = Lsph[eb * sph_e + bb];
          const float dx = sb.x - sa.x, dy = sb.y - sa.y, dz = sb.z - sa.z, reach = sa.w + sb.w;
          return sum3(dx, dx, dy, dy, dz, dz) <= reach * reach;
        };
        auto pair_key = [&](int ea, int ba, int eb, int bb) -> unsigned {
          return ((unsigned)ea << 20) | ((unsigned)eb << 8) | (unsigned)(ba << 4) | (unsigned)bb;
        };
        // Four candidates of a thread at a time: their reads from LDS are in flight together and they take
        // their places in the list with one atomic add per wavefront.  One after the other, with sixteen
        // reads each, they were bound by those reads: 9500 cycles per substep for 16 humanoids in groups of
        // four, 5800 so (1000 humanoids in groups of 16: 151 to 142 us a step with the changes around it).
        // Where an agent has at least as many threads as a robot can have pairs (up to four envs per
        // workgroup), a thread has one of its own at most, and the reads of three that are not there were in
        // its way: 512 self-colliding humanoids on the plane, 4 x 8 sweeps, 53.8 to 52.5 us a step, on the
        // heightfield 62.9 to 61.0 us, 512 chains of 16 links on the plane 51.2 to 50.2 us.
        constexpr int kCull = 4, kOwn = EC > 0 && kThreads / (EC > 0 ? EC : 1) >= kMaxPairs ? 1 : kCull;
        auto list_pairs = [&](auto count, const bool* pass, const unsigned* key) {
          constexpr int NC = decltype(count)::value;
          int n = 0;
#pragma unroll
          for (int k = 0; k < NC; ++k) n += pass[k] ? 1 : 0;
          int pos = wave_alloc<NC == 1 ? 1 : 3>(n, &Lpcount[2]);
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            if (!pass[k]) continue;
            if (pos < pair_cap) Lc2[pos] = key[k];
            else Lpcount[3] = 1;   // list full: everything is tested the slow way below
            ++pos;
          }
        };
        __syncthreads();
        // the listed pairs of every agent: thread (idx, e) takes pairs idx, idx + stride, ...
        if (idx < pair_stride)
          for (int p0 = idx; p0 < m_npairs; p0 += kOwn * pair_stride) {
            bool pass[kOwn];
            unsigned key[kOwn];
#pragma unroll
            for (int k = 0; k < kOwn; ++k) {
              const int pp = p0 + k * pair_stride;
              const bool valid = env_ok && pp < m_npairs;
              int ab = (my_pairs >> (8 * k)) & 255u;
              if (p0 != idx) ab = valid ? (M.pair_a[pp] << 4 | M.pair_b[pp]) : 0;   // (more than four per thread)
              pass[k] = near_pair(e, ab >> 4, e, ab & 15) && valid;
              key[k] = pair_key(e, ab >> 4, e, ab & 15);
            }
            list_pairs(std::integral_constant<int, kOwn>{}, pass, key);
          }
        // agents of one group: 256 lanes per near agent pair, lane = (body of A) * 16 + (body of B)
        int n_near = 0;
        if (m_group > 1) {
          n_near = Lpcount[1];
          const int cb = tid & 255, ba = cb >> 4, bb = cb & 15;
          const bool valid = ba < B && bb < B;
          const int sa = ba < B ? ba : 0, sb = bb < B ? bb : 0;
          for (int n0 = tid >> 8; n0 < n_near; n0 += kCull * (kThreads >> 8)) {
            bool pass[kCull];
            unsigned key[kCull];
#pragma unroll
            for (int k = 0; k < kCull; ++k) {
              const int nn = n0 + k * (kThreads >> 8);
              const int pr = Lmeet[nn < n_near ? nn : n0];
              pass[k] = near_pair(pr & 0xffff, sa, pr >> 16, sb) && valid && nn < n_near;
              key[k] = pair_key(pr & 0xffff, sa, pr >> 16, sb);
            }
            list_pairs(std::integral_constant<int, kCull>{}, pass, key);
          }
        }
        __syncthreads();
        // Stage 2: the segment-segment test, one listed candidate per lane
        plane_forces();
        if (!Lpcount[3]) {
          const int n_c2 = Lpcount[2];
          for (int c = tid; c < n_c2; c += kThreads) {
            const unsigned wd = Lc2[c];
            test_pair((int)(wd >> 20), (int)((wd >> 4) & 15u), (int)((wd >> 8) & 0xfffu), (int)(wd & 15u), wd, true);
          }
        } else {
          if (idx < pair_stride)
            for (int pp = idx; pp < m_npairs; pp += pair_stride)
              test_pair(e, M.pair_a[pp], e, M.pair_b[pp], pair_key(e, M.pair_a[pp], e, M.pair_b[pp]), env_ok);
          for (int nn = tid >> 8; nn < n_near; nn += kThreads >> 8) {
            const int cb = tid & 255, ba = cb >> 4, bb = cb & 15;
            const int pr = Lmeet[nn], ea = pr & 0xffff, eb = pr >> 16;
            test_pair(ea, ba, eb, bb, pair_key(ea, ba, eb, bb), ba < B && bb < B);
          }
        }
        __syncthreads();
        const int n_raw = Lpcount[0];
        n_pc = n_raw < kPairCap ? n_raw : kPairCap;
        const int n_hit = n_raw < hit_cap ? n_raw : hit_cap;
        if (n_raw > kPairCap) {
          // more than the workgroup holds: the kPairCap smallest (gap, key) words stay; each is
          // found by its rank among all words and its contact worked out again from its key
          for (int i = tid; i < n_hit; i += kThreads) {
            const unsigned long long wi = Lhit[i];
            int rank = 0;
            for (int k = 0; k < n_hit; ++k) rank += Lhit[k] < wi ? 1 : 0;
            if (rank < kPairCap) {
              const unsigned key = (unsigned)wi;
              const int ea = (int)(key >> 20), eb = (int)((key >> 8) & 0xfffu), ba = (int)((key >> 4) & 15u), bb = (int)(key & 15u);
              float sp = 0.0f, tp = 0.0f, gap = 0.0f;
              eval_pair(ea, ba, eb, bb, sp, tp, gap);
              store_hit(rank, ea, ba, eb, bb, key, sp, tp, gap);
            }
          }
          __syncthreads();
        }
        if (tid < n_pc) {
          // (eight keys in flight at a time: one after the other the loop waits for LDS n_pc times)
          const unsigned key = __float_as_uint(Ltmp[tid * kPairWords]);
          int rank = 0;
          static_assert(kPairCap % 8 == 0, "");
          for (int k0 = 0; k0 < n_pc; k0 += 8) {
            unsigned other[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) other[k] = __float_as_uint(Ltmp[(k0 + k) * kPairWords]);
#pragma unroll
            for (int k = 0; k < 8; ++k) rank += (int)(k0 + k < n_pc) & (int)(other[k] < key);
          }
          for (int wd = 0; wd < kPairWords; ++wd) Lpq[rank * kPairWords + wd] = Ltmp[tid * kPairWords + wd];
          // every contact enters the lists of its two bodies (the order in which they arrive does not
          // matter: the averaging threads sort their list)
          const int refs = __float_as_int(Ltmp[tid * kPairWords + 1]);
          const int ra = refs & 0xffff, rb = (refs >> 16) & 0xffff;
          const int slot_a = atomicAdd(&Lpbcnt[ra], 1), slot_b = atomicAdd(&Lpbcnt[rb], 1);
          if (slot_a < 6) Lpblist[ra * 6 + slot_a] = (uint8_t)(2 * rank);
          if (slot_b < 6) Lpblist[rb * 6 + slot_b] = (uint8_t)(2 * rank + 1);
        }
        if (tid == 0 && n_raw > kPairCap) atomicAdd(a.pair_dropped, n_raw - kPairCap);
        __syncthreads();
      }
    }
    TMARK(16);
    // The sums of a body are split over several threads when the workgroup has room: thread (e, b * kParts + p)
    // takes part p of the six velocity components of body b.  Short threads beat a long one, and the parts of a
    // body lie next to each other: their rows do too, so that neighbouring lanes read different banks, and a
    // wavefront holds few bodies, so that few have to go by the one with the most joints or contacts.  The number
    // of parts is the largest that always fits (kMaxBodies bodies); the general form has two or one.
    constexpr int kParts = EC == 0 ? 2 : (6 * kMaxBodies * EC <= NT ? 6 : (3 * kMaxBodies * EC <= NT ? 3 : 2));
    constexpr int kPartC = 6 / kParts;   // components of a part
    const bool g_split = (EC > 0 && kParts * kMaxBodies * EC <= NT) || kParts * B * E <= kThreads;
    // (threads behind the last body's last part, where the wavefront has work at all, do what its threads do, to the
    // last bit: E divides 64 in the compiled forms, so that part lies in the same wavefront)
    constexpr bool g_all = EC > 0 && NS == 0;
    const int g_items = (g_split ? kParts : 1) * B, g_item = g_all && idx >= g_items ? g_items - 1 : idx;
    const int g_b = g_split ? g_item / kParts : g_item, g_part = g_split ? g_item - g_b * kParts : 0;
    const bool g_on = g_all || (env_ok && g_b < B);
    const bool g_wave = !g_all || __builtin_amdgcn_readfirstlane(idx) < g_items;
    const int g_ref = g_b * E + e;
    // capsule-capsule contacts of body g_b: where their changes will be (up to kPairList
    // of them; a body with more walks the queue in every sweep), and the sum of their weights
    constexpr int kPairList = 6;   // (the list in LDS and the sorting network below are made for six)
    int gp_off[kPairList];
#pragma unroll
    for (int j = 0; j < kPairList; ++j) gp_off[j] = kPairCap * 12;
    bool gp_many = false;
    float gp_wsum = 0.0f;
    int gp_cnt = 0;
    if constexpr (PC != 0) {
      if (g_on) {
        const int cnt = n_pc > 0 ? Lpbcnt[g_ref] : 0;
        gp_cnt = cnt;
        if (cnt > 0 && cnt <= kPairList) {
          // the body's list (bytes 2 * queue index + side), sorted into queue order
          int v[kPairList];
#pragma unroll
          for (int j = 0; j < kPairList; ++j) v[j] = j < cnt ? (int)Lpblist[g_ref * 6 + j] : 255;
          auto cx = [&](int i, int j) { const int lo = min(v[i], v[j]), hi = max(v[i], v[j]); v[i] = lo; v[j] = hi; };
          cx(0, 5); cx(1, 3); cx(2, 4); cx(1, 2); cx(3, 4); cx(0, 3); cx(2, 5); cx(0, 1); cx(2, 3); cx(4, 5); cx(1, 2); cx(3, 4);
#pragma unroll
          for (int j = 0; j < kPairList; ++j) {
            const bool used = v[j] != 255;
            gp_off[j] = used ? v[j] * 6 : kPairCap * 12;
            const float wj = Lpq[(used ? v[j] >> 1 : 0) * kPairWords + 4];
            gp_wsum += used ? wj : 0.0f;
          }
        } else if (cnt > kPairList) {
          // more than the list holds: the weights by a walk over the queue (as in every sweep)
          for (int k = 0; k < n_pc; ++k) {
            const int refs = __float_as_int(Lpq[k * kPairWords + 1]);
            if ((refs & 0xffff) == g_ref || ((refs >> 16) & 0xffff) == g_ref) gp_wsum += Lpq[k * kPairWords + 4];
          }
        }
        gp_many = cnt > kPairList;
      }
    }
    // no body of this wavefront has more than two capsule-capsule contacts (the usual case): its
    // averages read two list entries instead of six
    // (only where a wavefront holds few bodies: with four envs per workgroup it holds sixteen, the
    // short forms are never taken and the choice itself costs 5 %)
    constexpr bool g_variants = EC >= 8;
    constexpr int kPairFew = 2;
    const bool gp_few = g_variants && PC != 0 && __ballot(gp_cnt > kPairFew) == 0ull;
    // ---- C: a body's sum of block weights.  With capsule-capsule contacts the body threads work it out for
    //         everybody; without, the lanes that need it add up the body's three slots themselves, which
    //         saves a phase and its barrier.
    if constexpr (PC != 0) {
      if (g_on && g_part == 0) {
        const int* tb = Ltjs + g_b * (kMaxBodyJoints + 3);
        float nbf = (float)tb[0];
        for (int k = 0; k < tb[2]; ++k) nbf += Lrec[((tb[1] + k) * kRecWords + 10) * E + e];
        Lnb[g_ref] = nbf + gp_wsum;
      }
    }
    auto weight_sum = [&](int bb, int ee) -> float {
      if constexpr (PC != 0) return Lnb[bb * E + ee];
      const int* tb = Ltjs + bb * (kMaxBodyJoints + 3);
      const int slot0 = tb[1], nslots = tb[2];
      float wk[3], nbf = (float)tb[0];
#pragma unroll
      for (int k = 0; k < 3; ++k) wk[k] = Lrec[((slot0 + (k < nslots ? k : 0)) * kRecWords + 10) * E + ee];
#pragma unroll
      for (int k = 0; k < 3; ++k) nbf += k < nslots ? wk[k] : 0.0f;
      return nbf;
    };
    if (tid > 0 && tid < 8) Lcount[tid] = 0;   // for the next substep's search
    if (a.recs && sub == a.substeps - 1) {
      // export the records of the last substep, [N][S][12] words
      for (int i = tid; i < S * E * kRecWords; i += kThreads) {
        int wd = i % kRecWords, rest = i / kRecWords, s = rest % S, ee = rest / S;
        int env_i = blockIdx.x * E + ee;
        if (env_i < N) {
          int word = Lreci[(s * kRecWords + wd) * E + ee];
          if (!Lreci[(s * kRecWords + 0) * E + ee]) word = (wd == 1 || wd == 2) ? -1 : 0;   // inactive: canonical record
          if (wd == kRecWords - 1) word = 0;   // (not in use)
          a.recs[((size_t)agent_at(env_i) * S + s) * kRecWords + wd] = word;
        }
      }
    }
    if constexpr (PC != 0) {
      if (a.pair_recs && sub == a.substeps - 1) {
        if (tid == 0) a.pair_count[blockIdx.x] = n_pc;
        if (tid < n_pc) {
          const int refs = __float_as_int(Lpq[tid * kPairWords + 1]);
          const int ra = refs & 0xffff, rb = (refs >> 16) & 0xffff;
          int32_t* o = a.pair_recs + ((size_t)blockIdx.x * kPairCap + tid) * 8;
          o[0] = agent_at(blockIdx.x * E + ra % E); o[1] = ra / E; o[2] = agent_at(blockIdx.x * E + rb % E); o[3] = rb / E;
          o[4] = __float_as_int(Lpq[tid * kPairWords + 2]); o[5] = __float_as_int(Lpq[tid * kPairWords + 3]);
          o[6] = __float_as_int(Lpq[tid * kPairWords + 5]); o[7] = __float_as_int(Lpq[tid * kPairWords + 4]);
        }
      }
      // The candidates of the search were here (last read before the barrier ahead of the sorted queue).  In front of
      // the barrier, as the first sweep already reads these rows: the world's velocity, where one lane relaxes a joint.
      for (int i = tid; i < 6 * E; i += kThreads) lds[P.zero + i] = 0.0f;
      __syncthreads();
    }

    TMARK(4);
    // ---- D: row constants
    const int n_active = __builtin_amdgcn_readfirstlane(Lcount[0]);
    // The joint rows and the contact rows are built inside the wavefront-uniform branches that use
    // them, so that the two sets of registers are never alive together.  Every lane of the
    // wavefronts concerned builds rows, the idle ones from a clamped index: a value assigned on
    // every path is not carried from one substep into the next in registers, as a conditionally
    // assigned one is.
    auto build_joint_side = [&](int js_j, int js_e, int js_side) {
     {
      const JointTab& jt = Ltjoint[js_j < J ? js_j : J - 1];
      const int e = js_e;
      const int ob = js_side ? jt.child : jt.parent;     // own body; -1: the static world
      const bool ghost = ob < 0;
      const int bo = ghost ? 0 : ob;                     // loads stay unconditional
      const float sg = js_side ? 1.0f : -1.0f;
      float xo[3], qo[4], iwo[6];
      for (int c = 0; c < 3; ++c) xo[c] = Lpos[(bo * 7 + c) * E + e];
      for (int c = 0; c < 4; ++c) qo[c] = Lpos[(bo * 7 + 3 + c) * E + e];
      for (int c = 0; c < 6; ++c) iwo[c] = Liw[(bo * kVS + c) * E + e];
      float no = NS ? 1.0f : weight_sum(bo, e), imo = Ltbody[4 * bo + 3];   // (Newton: no mass splitting)
      if (ghost) {
        for (int c = 0; c < 3; ++c) xo[c] = 0.0f;
        qo[0] = 1.0f; qo[1] = qo[2] = qo[3] = 0.0f;
        for (int c = 0; c < 6; ++c) iwo[c] = 0.0f;
        no = 0.0f; imo = 0.0f;
      }
      // The other side's centre and anchor come through the lane swap.  The separation of the anchors
      // and the lever arm are put together from differences of centres and of arms, which round at
      // the size of a body and not at that of its distance from the origin.
      float Ro[9], lo[3], t0[3], C[3], r[3];
      quat_to_mat(qo, Ro);
      for (int c = 0; c < 3; ++c) lo[c] = js_side ? jt.lb[c] : jt.la[c];
      mat_vec(Ro, lo, t0);
      for (int c = 0; c < 3; ++c) {
        C[c] = sg * ((xo[c] - lane_swap1(xo[c])) + (t0[c] - lane_swap1(t0[c])));   // child anchor minus parent anchor
        r[c] = fma_(-0.5f * sg, C[c], t0[c]);            // impulses act at the midpoint
      }
      // the world's side of a joint adds nothing to J v (whatever velocity its lane reads)
      const float sgl = ghost ? 0.0f : sg;
      for (int c = 0; c < 3; ++c) jr.sr[c] = sgl * r[c];
      jr.sg = sgl;
      jr.sv = sg * imo;
      const float inv_h = __builtin_amdgcn_rcpf(h), bh = p_beta_j * inv_h;
      float y[3][3], yn[3][3], zn[3][3];   // responses of the rows, and times the body's share
      for (int k = 0; k < 3; ++k) {
        float cr[3];
        cross_unit(r, k, cr);
        sym_vec(iwo, cr, y[k]);
        for (int c = 0; c < 3; ++c) yn[k][c] = no * y[k][c];
        const float kp = fma_(no, imo, cross_unit_dot(r, k, yn[k]));
        const float keff = kp + lane_swap1(kp);
        jr.pme[k] = keff > 0.0f ? -__builtin_amdgcn_rcpf(keff) : 0.0f;
        jr.pnb[k] = jr.pme[k] * (bh * C[k]);
        jr.pD[k] = keff; jr.pb[k] = bh * C[k];
        for (int c = 0; c < 3; ++c) jr.Y[k][c] = sg * y[k][c];
        if constexpr (NS == 0)
          for (int c = 0; c < k; ++c) {
            const float kc = cross_unit_dot(r, k, yn[c]);
            jr.pp[k + c - 1] = jr.pme[k] * (kc + lane_swap1(kc));
          }
      }
      // joint angles from both orientations; axes live in the parent frame
      float qx[4], qa[4], qb[4], Ra[9], phi[3];
      for (int c = 0; c < 4; ++c) qx[c] = lane_swap1(qo[c]);
      for (int c = 0; c < 4; ++c) { qa[c] = js_side ? qx[c] : qo[c]; qb[c] = js_side ? qo[c] : qx[c]; }
      quat_to_mat(qa, Ra);
      rel_rotvec(qa, qb, phi);
      jr.onesided = 0;
      jr.upper = 0;
      for (int k = 0; k < 3; ++k) {
        float ak[3], z[3];
        mat_vec(Ra, jt.axes[k], ak);
        float th = dot(jt.axes[k], phi);
        float sgn = 1.0f, bias;
        if (jt.mode[k] == 0) {
          bias = bh * th;
        } else {
          float glo = th - jt.lo[k], ghi = jt.hi[k] - th, g;
          if (glo < ghi) { g = glo; } else { g = ghi; sgn = -1.0f; jr.upper |= 1 << k; }
          bias = g >= 0.0f ? g * inv_h : bh * g;
          jr.onesided |= 1 << k;
        }
        for (int c = 0; c < 3; ++c) ak[c] *= sgn;
        sym_vec(iwo, ak, z);
        const float kp = no * dot(ak, z);
        const float keff = kp + lane_swap1(kp);
        jr.ame[k] = keff > 0.0f ? -__builtin_amdgcn_rcpf(keff) : 0.0f;
        jr.anb[k] = jr.ame[k] * bias;
        jr.aD[k] = keff; jr.ab[k] = bias;
        jr.lam[k] = 0.0f;
        jr.nl[k] = jt.mode[k] == 0 ? -INFINITY : 0.0f;
        for (int c = 0; c < 3; ++c) { jr.sax[k][c] = sgl * ak[c]; jr.Z[k][c] = sg * z[c]; }
        if constexpr (NS == 0) {
          for (int c = 0; c < 3; ++c) zn[k][c] = no * z[c];
          for (int c = 0; c < 3; ++c) {
            const float kc = cross_unit_dot(r, c, zn[k]);
            jr.ap[k][c] = jr.ame[k] * (kc + lane_swap1(kc));
          }
          for (int c = 0; c < k; ++c) {
            const float kc = dot(ak, zn[c]);
            jr.aa[k + c - 1] = jr.ame[k] * (kc + lane_swap1(kc));
          }
        }
      }
     }
    };
    // The same with both sides in one lane: the same operations on the same numbers, without lane swaps.
    auto build_joint = [&](JointRows& R, int js_j, int e) {
      const JointTab& jt = Ltjoint[js_j < J ? js_j : J - 1];
      float xo[2][3], qo[2][4], iwo[2][6], no[2], imo[2], t0[2][3], r[2][3], C[3];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int ob = s ? jt.child : jt.parent;           // -1: the static world
        const bool ghost = ob < 0;
        const int bo = ghost ? 0 : ob;
        for (int c = 0; c < 3; ++c) xo[s][c] = Lpos[(bo * 7 + c) * E + e];
        for (int c = 0; c < 4; ++c) qo[s][c] = Lpos[(bo * 7 + 3 + c) * E + e];
        for (int c = 0; c < 6; ++c) iwo[s][c] = Liw[(bo * kVS + c) * E + e];
        no[s] = weight_sum(bo, e); imo[s] = Ltbody[4 * bo + 3];
        if (ghost) {
          for (int c = 0; c < 3; ++c) xo[s][c] = 0.0f;
          qo[s][0] = 1.0f; qo[s][1] = qo[s][2] = qo[s][3] = 0.0f;
          for (int c = 0; c < 6; ++c) iwo[s][c] = 0.0f;
          no[s] = 0.0f; imo[s] = 0.0f;
        }
      }
      float Ra[9], Rb[9];
      quat_to_mat(qo[0], Ra);
      quat_to_mat(qo[1], Rb);
      mat_vec(Ra, jt.la, t0[0]);
      mat_vec(Rb, jt.lb, t0[1]);
      for (int c = 0; c < 3; ++c) {
        C[c] = (xo[1][c] - xo[0][c]) + (t0[1][c] - t0[0][c]);   // child anchor minus parent anchor
        r[0][c] = fma_(0.5f, C[c], t0[0][c]); r[1][c] = fma_(-0.5f, C[c], t0[1][c]);   // impulses act at the midpoint
      }
      for (int c = 0; c < 3; ++c) { R.sr[0][c] = -r[0][c]; R.sr[1][c] = r[1][c]; }
      R.sv[0] = -imo[0]; R.sv[1] = imo[1];
      const float inv_h = __builtin_amdgcn_rcpf(h), bh = p_beta_j * inv_h;
      float yn[2][3][3], zn[2][3][3];
      for (int k = 0; k < 3; ++k) {
        float kp[2], y[2][3];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float cr[3];
          cross_unit(r[s], k, cr);
          sym_vec(iwo[s], cr, y[s]);
          for (int c = 0; c < 3; ++c) { yn[s][k][c] = no[s] * y[s][c]; R.Y[s][k][c] = s ? y[s][c] : -y[s][c]; }
          kp[s] = fma_(no[s], imo[s], cross_unit_dot(r[s], k, yn[s][k]));
        }
        const float keff = kp[0] + kp[1];
        R.pme[k] = keff > 0.0f ? -__builtin_amdgcn_rcpf(keff) : 0.0f;
        R.pnb[k] = R.pme[k] * (bh * C[k]);
        for (int c = 0; c < k; ++c)
          R.pp[k + c - 1] = R.pme[k] * (cross_unit_dot(r[0], k, yn[0][c]) + cross_unit_dot(r[1], k, yn[1][c]));
      }
      float phi[3];
      rel_rotvec(qo[0], qo[1], phi);
      R.onesided = 0;
      R.upper = 0;
      for (int k = 0; k < 3; ++k) {
        float ak[3], z[2][3], kp[2];
        mat_vec(Ra, jt.axes[k], ak);
        const float th = dot(jt.axes[k], phi);
        float sgn = 1.0f, bias;
        if (jt.mode[k] == 0) {
          bias = bh * th;
        } else {
          float glo = th - jt.lo[k], ghi = jt.hi[k] - th, g;
          if (glo < ghi) { g = glo; } else { g = ghi; sgn = -1.0f; R.upper |= 1 << k; }
          bias = g >= 0.0f ? g * inv_h : bh * g;
          R.onesided |= 1 << k;
        }
        for (int c = 0; c < 3; ++c) ak[c] *= sgn;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          sym_vec(iwo[s], ak, z[s]);
          kp[s] = no[s] * dot(ak, z[s]);
          for (int c = 0; c < 3; ++c) { zn[s][k][c] = no[s] * z[s][c]; R.Z[s][k][c] = s ? z[s][c] : -z[s][c]; R.sax[s][k][c] = s ? ak[c] : -ak[c]; }
        }
        const float keff = kp[0] + kp[1];
        R.ame[k] = keff > 0.0f ? -__builtin_amdgcn_rcpf(keff) : 0.0f;
        R.anb[k] = R.ame[k] * bias;
        R.lam[k] = 0.0f;
        R.nl[k] = jt.mode[k] == 0 ? -INFINITY : 0.0f;
        for (int c = 0; c < 3; ++c)
          R.ap[k][c] = R.ame[k] * (cross_unit_dot(r[0], c, zn[0][k]) + cross_unit_dot(r[1], c, zn[1][k]));
        for (int c = 0; c < k; ++c)
          R.aa[k + c - 1] = R.ame[k] * (dot(ak, zn[0][c]) + dot(ak, zn[1][c]));
      }
    };
    // The same for one kind of row of one side (four lanes per joint): positional and angular lanes run through the
    // same instructions, the three directions u_k (lever arm x world axis, or joint axis) and what goes with them
    // chosen per lane, so that a lane builds three rows instead of six and has nothing to pick apart afterwards (us a
    // step: 64 planned humanoids 216.8 to 212.6 for three, 1024 ants 50.4 to 49.5, 1024 humanoids 52.0 to 51.5).
    auto build_quad = [&](QuadRows& R, int jj, int e, int side, bool ang, int& onesided, int& upper) {
      const JointTab& jt = Ltjoint[jj];
      const int ob = side ? jt.child : jt.parent;        // own body; -1: the static world
      const bool ghost = ob < 0;
      const int bo = ghost ? 0 : ob;
      const float sg = side ? 1.0f : -1.0f, sgl = ghost ? 0.0f : sg;
      float xo[3], qo[4], iwo[6];
      for (int c = 0; c < 3; ++c) xo[c] = Lpos[(bo * 7 + c) * E + e];
      for (int c = 0; c < 4; ++c) qo[c] = Lpos[(bo * 7 + 3 + c) * E + e];
      for (int c = 0; c < 6; ++c) iwo[c] = Liw[(bo * kVS + c) * E + e];
      float no = weight_sum(bo, e), imo = Ltbody[4 * bo + 3];
      if (ghost) {
        for (int c = 0; c < 3; ++c) xo[c] = 0.0f;
        qo[0] = 1.0f; qo[1] = qo[2] = qo[3] = 0.0f;
        for (int c = 0; c < 6; ++c) iwo[c] = 0.0f;
        no = 0.0f; imo = 0.0f;
      }
      float Ro[9], Ra[9], lo[3], t0[3], C[3], r[3], qx[4], qa[4], qb[4], phi[3];
      quat_to_mat(qo, Ro);
      for (int c = 0; c < 3; ++c) lo[c] = side ? jt.lb[c] : jt.la[c];
      mat_vec(Ro, lo, t0);
      for (int c = 0; c < 3; ++c) {
        C[c] = sg * ((xo[c] - lane_swap1(xo[c])) + (t0[c] - lane_swap1(t0[c])));   // child anchor minus parent anchor
        r[c] = fma_(-0.5f * sg, C[c], t0[c]);            // impulses act at the midpoint
      }
      for (int c = 0; c < 4; ++c) qx[c] = lane_swap1(qo[c]);
      for (int c = 0; c < 4; ++c) { qa[c] = side ? qx[c] : qo[c]; qb[c] = side ? qo[c] : qx[c]; }
      for (int c = 0; c < 9; ++c) { const float rx = lane_swap1(Ro[c]); Ra[c] = side ? rx : Ro[c]; }   // the parent's
      rel_rotvec(qa, qb, phi);
      const float inv_h = __builtin_amdgcn_rcpf(h), bh = p_beta_j * inv_h;
      R.kv = ang ? 0.0f : sgl;
      R.sv = sg * imo;
      onesided = 0;
      upper = 0;
      float yn[3][3];
      for (int k = 0; k < 3; ++k) {
        float ak[3], u[3], y[3];
        mat_vec(Ra, jt.axes[k], ak);
        const float th = dot(jt.axes[k], phi);
        float sgn = 1.0f, bias;
        if (jt.mode[k] == 0) {
          bias = bh * th;
        } else {
          float glo = th - jt.lo[k], ghi = jt.hi[k] - th, g;
          if (glo < ghi) { g = glo; } else { g = ghi; sgn = -1.0f; upper |= 1 << k; }
          bias = g >= 0.0f ? g * inv_h : bh * g;
          onesided |= 1 << k;
        }
        cross_unit(r, k, u);
        for (int c = 0; c < 3; ++c) u[c] = ang ? ak[c] * sgn : u[c];
        sym_vec(iwo, u, y);
        for (int c = 0; c < 3; ++c) { yn[k][c] = no * y[c]; R.K[k][c] = sgl * u[c]; R.R[k][c] = sg * y[c]; }
        // (each kind's products in the order the other forms have)
        const float kp_pos = fma_(no, imo, cross_unit_dot(r, k, yn[k])), kp_ang = no * dot(u, y), kp = ang ? kp_ang : kp_pos;
        const float keff = kp + lane_swap1(kp);
        R.me[k] = keff > 0.0f ? -__builtin_amdgcn_rcpf(keff) : 0.0f;
        R.nb[k] = R.me[k] * (ang ? bias : bh * C[k]);
        R.nl[k] = ang && jt.mode[k] != 0 ? 0.0f : -INFINITY;
        R.lam[k] = 0.0f;
        for (int c = 0; c < k; ++c) {
          const float kc_pos = cross_unit_dot(r, k, yn[c]), kc_ang = dot(u, yn[c]), kc = ang ? kc_ang : kc_pos;
          const float v = R.me[k] * (kc + lane_swap1(kc));
          R.t1[k + c - 1] = ang ? 0.0f : v;
          R.t2[k + c - 1] = ang ? v : 0.0f;
        }
        const float me_ang = ang ? R.me[k] : 0.0f;
        for (int c = 0; c < 3; ++c) {
          const float kc = cross_unit_dot(r, c, yn[k]);
          R.ap[k][c] = me_ang * (kc + lane_swap1(kc));
        }
      }
    };
    // contact k of the workgroup's list goes to thread kThreads-1-k (the joint threads sit at
    // the low end); contacts beyond one per thread start from zero impulse in LDS
    auto build_contact = [&]() {
      const int li = kThreads - 1 - tid;
      has_contact = li < n_active && li < n_reg;
      if (n_active > 0) {
        const int i = Llist[li < n_active ? li : n_active - 1];
        const int ee = i % E, sl = i / E, body = Ltslot[2 * sl];
        build_contact_rows(cr, Lrec, Liw, NS ? 1.0f : weight_sum(body, ee), sl, ee, E, body, Ltbody[4 * body + 3], h, p_beta_c, p_vdepen, NS != 0);
        if constexpr (WS != 0)
          for (int r = 0; r < 3; ++r) cr.lam[r] = p_warm * Lwc[(sl * 3 + r) * E + ee];
      } else {
        cr = ContactRows{};
      }
    };
    // capsule-capsule contact k of the sorted queue goes to two neighbouring lanes (body A, body B).
    // The contact lanes start right above the joint wavefronts (whose registers are busy with the
    // joint rows) and go up; what does not fit there goes below, into the joint wavefronts.
    const int pk_up = (kThreads - joint_threads) >> 1;
    const int pk = tid >= joint_threads ? (tid - joint_threads) >> 1 : pk_up + ((joint_threads - 1 - tid) >> 1);
    const bool has_pair = PC != 0 && pk < n_pc;
    // (in the compiled forms there is room above the joint wavefronts for all that a workgroup can hold)
    constexpr bool kPairsInJoints = PC != 0 && (EC == 0 || (NT - ((JL * kMaxJoints * EC + 63) / 64) * 64) / 2 < kPairCap);
    auto build_pair = [&]() {
      if constexpr (PC != 0) {
        if (n_pc > 0) build_pair_side(pr, tid & 1, Lpq, Lpos, Liw, Lnb, Lorg, Ltbody, pk < n_pc ? pk : n_pc - 1, E, h, p_beta_c, p_vdepen);
        else pr = PairSide{};
      }
    };
    // impulses of the contacts beyond one per thread: slot k of a small array, or (warm start) the
    // contact's own place in the per-slot array, which already holds what was kept
    auto overflow_lam = [&](int k, int r) -> float& {
      if constexpr (WS != 0) { const int i = Llist[k]; return Lwc[(i / E * 3 + r) * E + i % E]; }
      else return Llam[3 * (k - n_reg) + r];
    };

    TMARK(5);
    // What a body adds up: the changes of NJ joint sides and of its contact slots.  Entries that are not in use
    // point at zeros (P.zero; the changes share their space with the terrain search, so only those that a block
    // writes in every sweep are read).  The slots that hold a contact come first.
    // (Newton's method with a wavefront per env has lists of its own)
    const bool env_per_wave = NS != 0 && 2 * J + S <= 64;
    int gat_off[NJ], gat_slot[3], g_njs = 0, g_nc = 0;
#pragma unroll
    for (int k = 0; k < NJ; ++k) gat_off[k] = P.zero;
    gat_slot[0] = gat_slot[1] = gat_slot[2] = P.zero;
    if (!env_per_wave) {
      const int* tb = Ltjs + (g_on ? g_b : 0) * (kMaxBodyJoints + 3);
      g_njs = g_on ? tb[0] : 0;
      const int g_slot0 = tb[1], g_nslots = tb[2], zero = P.zero + e;
#pragma unroll
      for (int k = 0; k < NJ; ++k) {
        const bool used = k < g_njs;
        int js = used ? tb[3 + k] : 0;
        gat_off[k] = used ? P.outj + ((js >> 1) * kJS + (js & 1) * kSide) * E + e : zero;
      }
      bool on[3];
      int at[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int sl = g_slot0 + (k < g_nslots ? k : 0);
        on[k] = g_on && k < g_nslots && Lrec[(sl * kRecWords + 10) * E + e] != 0.0f;
        at[k] = P.outc + sl * kCS * E + e;
      }
      gat_slot[0] = on[0] ? at[0] : (on[1] ? at[1] : (on[2] ? at[2] : zero));
      gat_slot[1] = on[0] && on[1] ? at[1] : ((on[0] || on[1]) && on[2] ? at[2] : zero);
      gat_slot[2] = on[0] && on[1] && on[2] ? at[2] : zero;
      g_nc = (int)on[0] + (int)on[1] + (int)on[2];
    }
    // The sums of a wavefront read no more entries than its bodies have (the same in all lanes, so the choice is a
    // scalar branch): two joint entries instead of NJ, no, one or three slots.  An entry is a read from LDS, of
    // which a wavefront issues one in about eight cycles.
    const bool g_few = NJ > 2 && __ballot(g_njs > 2) == 0ull;
    const bool g_noc = __ballot(g_nc > 0) == 0ull, g_onec = __ballot(g_nc > 1) == 0ull, g_twoc = __ballot(g_nc > 2) == 0ull;
    // ---- S: sweeps
    // What bounds a sweep is the length of one wavefront's chain, twice: rows, then sums, a barrier behind each.  On
    // this chip an instruction that needs the result of the one before it takes 8 cycles, an independent one 5, a
    // taken branch 22, a branch around a masked region 27, a read from LDS 70 plus 8 for every further one, and a
    // lane swap costs another 16 to 30 while a second wavefront of the SIMD computes.  Hence: impulses from a
    // triangular system instead of a trip through the velocities for every row (48 to 17 instructions waiting for
    // each other), changes of velocity instead of copies (one addition per entry instead of two operations), no
    // more entries read than the wavefront's bodies have, loops without branches or masks, four lanes per joint
    // where the SIMDs have room.  Cycles per sweep, before and now: 64 humanoids (2 envs per workgroup) 869 to 747,
    // 1024 on the plane (4) 964 to 770, 1500 (8) 1105 to 1000, 4096 (16) 1305 to 1200 and on the plane 1260 to 1150,
    // 4096 that collide in groups of 4 2260 to 1770.
    // Wavefronts that hold joint threads run only the joint rows, the others only the contact
    // rows (a wave-uniform branch, so neither path carries the other's registers); both paths
    // execute the same two barriers per sweep.
    // components [c0, c0 + NC) of the new velocity of body g_b (0..2 linear, 3..5 angular), from KJ joint entries
    // and HC slots' entries
    auto gather_part = [&](auto nc_tag, int c0, auto kj_tag, auto hc_tag) {
      constexpr int NC = decltype(nc_tag)::value, KJ = decltype(kj_tag)::value, HC = decltype(hc_tag)::value;
      if (g_on) {
        // The weighted average of the copies of a body, one per block and each scaled by W / w, is its velocity
        // plus the plain sum of what the blocks' impulses change in it.
        // Every load is unconditional: unused entries read P.zero.  All reads are issued before the first use so
        // their LDS latency is paid once; sums of sums, so that few additions wait for each other (in one order for
        // every KJ and HC: what is left out is zero).
        // (two components: a linear and an angular one, so that the parts' rows lie one apart)
        constexpr int kApart = NC == 2 ? 3 : 1;
        const int ho = c0 * E;
        float v0[NC], acc[NC], val[KJ + HC][NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v0[c] = Lvel[(g_b * kVS + c * kApart) * E + e + ho];
#pragma unroll
        for (int k = 0; k < KJ; ++k)
#pragma unroll
          for (int c = 0; c < NC; ++c) val[k][c] = lds[gat_off[k] + ho + c * kApart * E];
#pragma unroll
        for (int k = 0; k < HC; ++k)
#pragma unroll
          for (int c = 0; c < NC; ++c) val[KJ + k][c] = lds[gat_slot[k] + ho + c * kApart * E];
        __builtin_amdgcn_sched_group_barrier(0x100, NC == 3 ? (KJ + 1 + HC) * 2 : KJ + 1 + HC, 0);  // the DS reads first
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          float js[KJ];
#pragma unroll
          for (int k = 0; k < KJ; ++k) js[k] = val[k][c];
#pragma unroll
          for (int step = 1; step < KJ; step *= 2)
#pragma unroll
            for (int k = 0; k + step < KJ; k += 2 * step) js[k] += js[k + step];
          acc[c] = js[0];
          if constexpr (HC == 1) acc[c] += val[KJ][c];
          if constexpr (HC == 2) acc[c] += val[KJ][c] + val[KJ + 1][c];
          if constexpr (HC == 3) acc[c] += (val[KJ][c] + val[KJ + 1][c]) + val[KJ + 2][c];
        }
        if constexpr (PC != 0) {
          if (n_pc > 0) {
            if (gp_many) {
              // more contacts on this body than the list holds: walk the queue
              for (int k = 0; k < n_pc; ++k) {
                const int refs = __float_as_int(Lpq[k * kPairWords + 1]);
                if ((refs & 0xffff) == g_ref)
                  for (int c = 0; c < NC; ++c) acc[c] += Lpo[k * 12 + c0 + c * kApart];
                if (((refs >> 16) & 0xffff) == g_ref)
                  for (int c = 0; c < NC; ++c) acc[c] += Lpo[k * 12 + 6 + c0 + c * kApart];
              }
            } else {
              // the entries of the listed contacts (the list holds the used ones first; the others point at zeros)
              auto sum_pairs = [&](auto kp_tag) {
                constexpr int KP = decltype(kp_tag)::value;
                float pv[KP][NC];
#pragma unroll
                for (int j = 0; j < KP; ++j)
#pragma unroll
                  for (int c = 0; c < NC; ++c) pv[j][c] = Lpo[gp_off[j] + c0 + c * kApart];
#pragma unroll
                for (int j = 0; j < KP; ++j)
#pragma unroll
                  for (int c = 0; c < NC; ++c) acc[c] += pv[j][c];
              };
              if constexpr (g_variants) {
                if (gp_few) sum_pairs(std::integral_constant<int, kPairFew>{});
                else sum_pairs(std::integral_constant<int, kPairList>{});
              } else {
                sum_pairs(std::integral_constant<int, kPairList>{});
              }
            }
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) Lvel[(g_b * kVS + c * kApart) * E + e + ho] = v0[c] + acc[c];
      }
    };
    // one sweep of this thread's side of a capsule-capsule contact, if it has one
    // (a capsule-capsule contact starts every substep without impulses: in the warm start's
    // sweep -1 it changes nothing)
    auto pair_sweep = [&](bool relax) {
      if constexpr (PC != 0) {
        if (has_pair) {
          float vo[3] = {0.0f, 0.0f, 0.0f}, wo[3] = {0.0f, 0.0f, 0.0f};
          if (relax) {
            for (int c = 0; c < 3; ++c) { vo[c] = Lvel[pr.off + c * E]; wo[c] = Lvel[pr.off + (3 + c) * E]; }
            relax_pair_side(pr, p_mu, vo, wo);
          }
          const int po = (2 * pk + (tid & 1)) * 6;
          for (int c = 0; c < 3; ++c) { Lpo[po + c] = vo[c]; Lpo[po + 3 + c] = wo[c]; }
        }
      }
    };
    auto gather = [&](auto kj_tag, auto hc_tag) {
      gather_part(std::integral_constant<int, kPartC>{}, (kPartC == 2 ? 1 : kPartC) * g_part, kj_tag, hc_tag);
      if constexpr (kParts == 2) {
        if (!g_split) gather_part(std::integral_constant<int, kPartC>{}, kPartC, kj_tag, hc_tag);   // one thread per body
      }
    };
    // All sweeps of a wavefront: rows(it) relaxes what its lanes hold and leaves the changes in LDS, then the sums.
    // Which form of the sums the wavefront needs is the same in all sweeps, so the choice lies outside the loop
    // (a branch that is taken costs 22 cycles or more, about as much as four additions).
    auto sweeps = [&](auto rows) {
      using std::integral_constant;
      constexpr int kFew = NJ > 2 ? 2 : NJ;
      auto loop = [&](auto kj_tag, auto hc_tag) {
        for (int it = WS ? -1 : 0; it < a.iterations; ++it) {
          rows(it);
          __syncthreads();
          if constexpr (decltype(kj_tag)::value > 0) gather(kj_tag, hc_tag);
          __syncthreads();
        }
      };
      auto by_slots = [&](auto kj_tag) {
        if (g_noc) loop(kj_tag, integral_constant<int, 0>{});
        else if (g_onec) loop(kj_tag, integral_constant<int, 1>{});
        else if (g_twoc) loop(kj_tag, integral_constant<int, 2>{});
        else loop(kj_tag, integral_constant<int, 3>{});
      };
      if (!g_wave) loop(integral_constant<int, 0>{}, integral_constant<int, 0>{});
      else if (g_few) by_slots(integral_constant<int, kFew>{});
      else by_slots(integral_constant<int, NJ>{});
    };
    // Warm start: sweep -1 relaxes nothing; every block applies the impulses it starts from (the
    // kept ones times the share), as a sweep does with the increments.
    if (NS != 0 && env_per_wave) {
      // ---- S (Newton), where the rows of an env fit one wavefront: the solve of the block below with a
      // wavefront for every env.  Lane l < 2 J is side l & 1 of joint l >> 1, the lanes above hold the
      // contact slots.  Blocks and bodies still meet in LDS, but a wavefront's LDS instructions stay in
      // their order, so nothing waits at a barrier, and the dot products are sums over the lanes: an inner
      // iteration is one wavefront's chain instead of four phases of the whole workgroup.
      // Bound by that chain (LDS round trips and the sums' lane crossings).  1024 humanoids on the
      // heightfield, 3 Newton x 8 inner iterations x 4 substeps: 184 us with the block below, 135 us here
      // An env of more rows keeps the block below: two wavefronts per env would need barriers again.
      if constexpr (NS != 0) {
      if (m_terrain == 0) { forces(0); __syncthreads(); }
      const int we = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
      if (we < E && blockIdx.x * E + we < N) {
        float* LU = lds + P.nu;        // [B][kVS][E]: M^-1 J^T x (plus v* when asked for)
        const float p_reg = M.newton_reg;
        const int n_kry = M.krylov;
        constexpr float kFrictionEps = 1e-3f;   // m/s
        const bool jrole = lane < 2 * J;
        const int w_j = jrole ? lane >> 1 : 0, w_side = lane & 1;
        const int w_s = !jrole && lane - 2 * J < S ? lane - 2 * J : 0;
        const bool has = !jrole && lane - 2 * J < S && Lreci[(w_s * kRecWords + 0) * E + we] != 0;
        // The row constants of either role in one array, so that the two roles share registers:
        //   joint side: K[0..2] lever arm, K[3] linear response, K[4] sign, K[5..13] angular response of
        //               the positional rows, K[14..22] the three axes, K[23..31] their angular response;
        //   contact:    K[0..8] directions n, t1, t2, K[9..17] lever x direction, K[18..26] angular
        //               response, K[27] linear response.
        float K[32], Dg[6], bs[6], lam[6];
        int ones = 0, uppers = 0, ob = -1;
        for (int k = 0; k < 32; ++k) K[k] = 0.0f;
        for (int k = 0; k < 6; ++k) Dg[k] = bs[k] = lam[k] = 0.0f;
        if (jrole) {
          build_joint_side(w_j, we, w_side);
          for (int k = 0; k < 3; ++k) {
            K[k] = jr.sr[k];
            for (int c = 0; c < 3; ++c) { K[5 + 3 * k + c] = jr.Y[k][c]; K[14 + 3 * k + c] = jr.sax[k][c]; K[23 + 3 * k + c] = jr.Z[k][c]; }
            Dg[k] = jr.pD[k]; bs[k] = jr.pb[k]; Dg[3 + k] = jr.aD[k]; bs[3 + k] = jr.ab[k];
          }
          K[3] = jr.sv; K[4] = jr.sg;
          ones = jr.onesided; uppers = jr.upper;
          ob = w_side ? Ltjoint[w_j].child : Ltjoint[w_j].parent;
          if constexpr (WS != 0) {
            // Warm start: the first iterate is the share of what the rows ended the last substep with
            // (a limit row only if it stands for the same limit as then).
            for (int k = 0; k < 3; ++k) lam[k] = p_warm * Lwj[(w_j * 6 + k) * E + we];
            for (int k = 0; k < 3; ++k) {
              const float kept = Lwj[(w_j * 6 + 3 + k) * E + we];
              float l0 = p_warm * kept;
              if ((ones >> k) & 1) {
                const bool was_upper = __float_as_int(kept) < 0, is_upper = (uppers >> k) & 1;
                l0 = was_upper == is_upper ? fabsf(l0) : 0.0f;
              }
              lam[3 + k] = l0;
            }
          }
        } else if (has) {
          ob = Ltslot[2 * w_s];
          build_contact_rows(cr, Lrec, Liw, 1.0f, w_s, we, E, ob, Ltbody[4 * ob + 3], h, p_beta_c, p_vdepen, true);
          for (int r = 0; r < 3; ++r) {
            for (int c = 0; c < 3; ++c) { K[3 * r + c] = cr.dir[r][c]; K[9 + 3 * r + c] = cr.ang[r][c]; K[18 + 3 * r + c] = cr.Y[r][c]; }
            Dg[r] = cr.D[r];
            if constexpr (WS != 0) lam[r] = p_warm * Lwc[(w_s * 3 + r) * E + we];   // (a slot that was not active then holds zero)
          }
          bs[0] = cr.bias; K[27] = cr.ls;
        }
        const bool active = jrole || has, counts = has || (jrole && w_side == 0);   // (a joint's rows are counted once)
        const int nr = jrole ? 6 : 3, vo = (ob < 0 ? 0 : ob) * kVS * E + we;
        float* out = jrole ? Loutj + (w_j * kJS + w_side * kSide) * E + we : Loutc + w_s * kCS * E + we;
        // gathering lanes: three per body, two velocity components each
        const int g_b = lane / 3, g_c = 2 * (lane - 3 * g_b);
        const bool g_on = g_b < B;
        int g_src[NJ + 3];
        {
          const int* tb = Ltjs + (g_on ? g_b : 0) * (kMaxBodyJoints + 3);
          const int n_js = tb[0], slot0 = tb[1], n_slots = tb[2];
#pragma unroll
          for (int k = 0; k < NJ; ++k) {
            const int js = k < n_js ? tb[3 + k] : 0;
            g_src[k] = (g_on && k < n_js ? P.outj + ((js >> 1) * kJS + (js & 1) * kSide) * E : P.zero) + g_c * E + we;
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const bool used = g_on && k < n_slots && Lreci[((slot0 + (k < n_slots ? k : 0)) * kRecWords + 0) * E + we] != 0;
            g_src[NJ + k] = (used ? P.outc + (slot0 + k) * kCS * E : P.zero) + g_c * E + we;
          }
        }
        // stores of this wavefront's lanes before, loads after
        auto in_order = [&]() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
        auto scatter = [&](const float* xv) {
          float dv[3], dw[3];
          if (jrole) {
            for (int c = 0; c < 3; ++c) {
              dv[c] = K[3] * xv[c];
              dw[c] = sum3(K[5 + c], xv[0], K[8 + c], xv[1], K[11 + c], xv[2]);
              dw[c] = fma_(K[23 + c], xv[3], dw[c]); dw[c] = fma_(K[26 + c], xv[4], dw[c]); dw[c] = fma_(K[29 + c], xv[5], dw[c]);
            }
          } else {
            for (int c = 0; c < 3; ++c) {
              dv[c] = K[27] * sum3(K[c], xv[0], K[3 + c], xv[1], K[6 + c], xv[2]);
              dw[c] = sum3(K[18 + c], xv[0], K[21 + c], xv[1], K[24 + c], xv[2]);
            }
          }
          if (ob >= 0)
            for (int c = 0; c < 3; ++c) { out[c * E] = dv[c]; out[(3 + c) * E] = dw[c]; }
          in_order();
        };
        // every body: the plain sum of its blocks' contributions (in static order), on top of the
        // velocities the solve started from when `with_base`
        auto gather_sum = [&](bool with_base, float* dst) {
          if (g_on) {
            float val[NJ + 3][2], acc[2];
#pragma unroll
            for (int k = 0; k < NJ + 3; ++k) { val[k][0] = lds[g_src[k]]; val[k][1] = lds[g_src[k] + E]; }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              acc[c] = val[0][c];
#pragma unroll
              for (int k = 1; k < NJ + 3; ++k) acc[c] += val[k][c];
              const int o = (g_b * kVS + g_c + c) * E + we;
              dst[o] = with_base ? Lvel[o] + acc[c] : acc[c];
            }
          }
          in_order();
        };
        auto rows_of = [&](const float* src, float* y) {
          float uv[3], uw[3];
          for (int c = 0; c < 3; ++c) { uv[c] = src[vo + c * E]; uw[c] = src[vo + (3 + c) * E]; }
          float pj[6], pc[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            pj[k] = fma_(K[4], uv[k], cross_unit_dot(K, k, uw));
            pj[3 + k] = sum3(K[14 + 3 * k], uw[0], K[15 + 3 * k], uw[1], K[16 + 3 * k], uw[2]);
            pc[k] = dot(K + 3 * k, uv) + dot(K + 9 + 3 * k, uw);
          }
#pragma unroll
          for (int k = 0; k < 6; ++k) {
            const float both = pj[k] + lane_swap1(pj[k]);
            y[k] = jrole ? both : (k < 3 ? pc[k] : 0.0f);
          }
          in_order();
        };
        for (int it = 0; it < a.iterations; ++it) {
          float sres[6], known[6], cp[6], ipd[6], tmp[6];
          int on = 0;
          // residual of the current iterate
          scatter(lam);
          gather_sum(true, LU);
          rows_of(LU, sres);
          for (int k = 0; k < 6; ++k) { sres[k] += bs[k]; known[k] = 0.0f; cp[k] = 0.0f; }
          // the branch every row is on
          if (jrole) {
            on = 7;
            for (int k = 0; k < 3; ++k) {
              const bool one = (ones >> k) & 1;
              const bool s_branch = !one || (Dg[3 + k] > 0.0f && lam[3 + k] - sres[3 + k] / Dg[3 + k] > 0.0f);
              if (s_branch) on |= 8 << k; else known[3 + k] = -lam[3 + k];
            }
          } else {
            if (Dg[0] > 0.0f && lam[0] - sres[0] / Dg[0] > 0.0f) on |= 1; else known[0] = -lam[0];
            const float rad = p_mu * lam[0];
            if (rad > 0.0f) {
              on |= 6;
              cp[1] = cp[2] = sqrtf(sum3(sres[1], sres[1], sres[2], sres[2], kFrictionEps, kFrictionEps)) / rad;
            } else { known[1] = -lam[1]; known[2] = -lam[2]; }
          }
          // (ipd: inverse of the preconditioner's diagonal on the rows of the "s" branch, 0 elsewhere)
          for (int k = 0; k < 6; ++k) {
            const float pdk = fma_(Dg[k], 1.0f + p_reg, cp[k]);
            if (!(pdk > 0.0f) || k >= nr || !active) on &= ~(1 << k);
            ipd[k] = ((on >> k) & 1) ? 1.0f / pdk : 0.0f;
          }
          // right-hand side of the rows on the "s" branch: -s - c lambda - A known
          scatter(known);
          gather_sum(false, LU);
          rows_of(LU, tmp);
          float x[6], z[6], pv[6], q[6], az[6], damp[6];
          for (int k = 0; k < 6; ++k) {
            const float rhs = ((on >> k) & 1) ? fma_(-cp[k], lam[k], -sres[k]) - tmp[k] : 0.0f;
            x[k] = 0.0f; z[k] = rhs * ipd[k]; pv[k] = z[k];
            damp[k] = fma_(p_reg, Dg[k], cp[k]);
          }
          // (A + reg D + c) z on the rows of the "s" branch
          auto apply_hat = [&](const float* xv, float* y) {
            scatter(xv);
            gather_sum(false, LU);
            rows_of(LU, y);
            for (int k = 0; k < 6; ++k) y[k] = ((on >> k) & 1) ? fma_(damp[k], xv[k], y[k]) : 0.0f;
          };
          // z.Az, Az.Az / pd, Az.q / pd over the rows of the env
          auto products = [&](float& ta, float& tb, float& tc) {
            ta = tb = tc = 0.0f;
            for (int k = 0; k < 6; ++k) {
              const float ap = az[k] * ipd[k];
              ta = fma_(z[k], az[k], ta); tb = fma_(az[k], ap, tb); tc = fma_(ap, q[k], tc);
            }
            if (!counts) { ta = 0.0f; tb = 0.0f; tc = 0.0f; }
            wave_sum3(ta, tb, tc);
          };
          apply_hat(z, az);
          for (int k = 0; k < 6; ++k) q[k] = az[k];
          float gamma, den, unused;
          products(gamma, den, unused);
          const float gamma0 = gamma;
          for (int kk = 0; kk < n_kry; ++kk) {
            if (!(den > 0.0f) || !(gamma > 1e-12f * gamma0)) break;
            const float alpha = gamma / den;
            for (int k = 0; k < 6; ++k) { x[k] = fma_(alpha, pv[k], x[k]); z[k] = fma_(-alpha * q[k], ipd[k], z[k]); }   // (all zero off the "s" branch)
            if (kk == n_kry - 1) break;       // (the last iteration's operator product would not be used)
            apply_hat(z, az);
            float ta, tb, tc;
            products(ta, tb, tc);
            const float beta = ta / gamma;
            for (int k = 0; k < 6; ++k) { pv[k] = fma_(beta, pv[k], z[k]); q[k] = fma_(beta, q[k], az[k]); }
            den = fma_(beta * beta, den, fma_(2.0f * beta, tc, tb));     // q . q / pd of the new q
            gamma = ta;
          }
          // update, then back into the feasible set
          for (int k = 0; k < 6; ++k) lam[k] += ((on >> k) & 1) ? x[k] : known[k];
          if (jrole) {
            for (int k = 0; k < 3; ++k) if ((ones >> k) & 1) lam[3 + k] = fmaxf(lam[3 + k], 0.0f);
          } else {
            lam[0] = fmaxf(lam[0], 0.0f);
            const float rad = p_mu * lam[0], nrm = sqrtf(sum2(lam[1], lam[1], lam[2], lam[2]));
            if (nrm > rad) { const float sc = nrm > 0.0f ? rad / nrm : 0.0f; lam[1] *= sc; lam[2] *= sc; }
          }
        }
        // the solved velocities: v* + M^-1 J^T lambda
        scatter(lam);
        gather_sum(true, Lvel);
        if constexpr (WS != 0) {
          // kept for the next substep (both lanes of a joint hold the same impulses)
          if (jrole) {
            if (w_side == 0) {
              for (int k = 0; k < 3; ++k) Lwj[(w_j * 6 + k) * E + we] = lam[k];
              for (int k = 0; k < 3; ++k)
                Lwj[(w_j * 6 + 3 + k) * E + we] = ((ones & uppers) >> k) & 1 ? -lam[3 + k] : lam[3 + k];
            }
          } else if (lane - 2 * J < S) {
            for (int r = 0; r < 3; ++r) Lwc[(w_s * 3 + r) * E + we] = has ? lam[r] : 0.0f;   // (an inactive slot hands nothing on)
          }
        }
      }
      __syncthreads();
      }
    } else if constexpr (NS != 0) {
#pragma clang fp contract(fast)
      // ---- S (Newton): the paper's solver (Section 3.1), a non-smooth Newton method whose every
      // iteration is solved by a fixed number of preconditioned conjugate-residual iterations.
      // Unknowns: the impulses lambda of all rows; u = v* + M^-1 J^T lambda; residual s = J u + bias.
      // Bilateral rows ask for s = 0; one-sided rows for min(lambda, s / D) = 0 (D the diagonal of
      // J M^-1 J^T); a friction pair follows the smooth isotropic Coulomb law lambda_t = -mu lambda_n
      // s_t / |s_t|_eps, which enters an iteration as a damper s_t + c lambda_t = 0 with the
      // compliance c = |s_t|_eps / (mu lambda_n) of the current iterate.  The operator is applied
      // through the bodies in the two phases of a Jacobi sweep: every block writes the velocity
      // change its rows' impulses give its bodies (scatter), a barrier, every body adds up its
      // blocks' contributions (gather), a barrier, every row takes J times the result.  Every row's
      // vectors stay in the registers of its lane (both lanes of a joint hold the same values).
      // Dot products over the rows of an env: every block leaves its partial sum in an LDS entry of
      // its own, one thread per env adds them up in block order, so the result does not depend on
      // which wavefront ran first.
      float* LU = lds + P.nu;        // [B][kVS][E]: M^-1 J^T x (plus v* when asked for)
      float* Lred = lds + P.nred;    // [3][J + S][E]: partial sums of the blocks
      float* Lsum = lds + P.nsum;    // [3][8][E]: sums over an eighth of the blocks each
      const int nblk = J + S;
      const float p_reg = M.newton_reg;
      const int n_kry = M.krylov;
      constexpr float kFrictionEps = 1e-3f;   // m/s
      constexpr int kRedParts = 4;            // (J + S <= 64 blocks: at most sixteen per part)
      const bool jrole = joint_wave;
      if constexpr (WS != 0) {
        // a slot that is not active in this substep hands nothing on to the next one
        for (int i = tid; i < S * E; i += kThreads)
          if (!Lreci[(i / E * kRecWords + 0) * E + i % E])
            for (int r = 0; r < 3; ++r) Lwc[(i / E * 3 + r) * E + i % E] = 0.0f;
      }
      if (m_terrain == 0 && !jrole) forces(joint_threads);   // (the first gather is behind a barrier)
      if (jrole) build_joint_side(js_j, js_e, js_side); else build_contact();
      for (int i = tid; i < 3 * nblk * E; i += kThreads) Lred[i] = 0.0f;   // inactive slots contribute nothing
      const int nr = jrole ? 6 : 3;
      const bool active = jrole ? js_on : has_contact;      // this lane holds rows
      // The row constants of either role in one array, so that the two roles share registers:
      //   joint side: K[0..2] lever arm, K[3] linear response, K[4] sign, K[5..13] angular response of
      //               the positional rows, K[14..22] the three axes, K[23..31] their angular response;
      //   contact:    K[0..8] directions n, t1, t2, K[9..17] lever x direction, K[18..26] angular
      //               response, K[27] linear response.
      float K[32], Dg[6], bs[6];
      int ones = 0, uppers = 0, c_body = 0, c_slot_e = 0;
      if (jrole) {
        for (int k = 0; k < 3; ++k) {
          K[k] = jr.sr[k];
          for (int c = 0; c < 3; ++c) { K[5 + 3 * k + c] = jr.Y[k][c]; K[14 + 3 * k + c] = jr.sax[k][c]; K[23 + 3 * k + c] = jr.Z[k][c]; }
          Dg[k] = jr.pD[k]; bs[k] = jr.pb[k]; Dg[3 + k] = jr.aD[k]; bs[3 + k] = jr.ab[k];
        }
        K[3] = jr.sv; K[4] = jr.sg;
        ones = jr.onesided;
        uppers = jr.upper;
      } else {
        for (int r = 0; r < 3; ++r) {
          for (int c = 0; c < 3; ++c) { K[3 * r + c] = cr.dir[r][c]; K[9 + 3 * r + c] = cr.ang[r][c]; K[18 + 3 * r + c] = cr.Y[r][c]; }
          Dg[r] = cr.D[r]; bs[r] = r == 0 ? cr.bias : 0.0f; Dg[3 + r] = 0.0f; bs[3 + r] = 0.0f;
        }
        K[27] = cr.ls; K[28] = K[29] = K[30] = K[31] = 0.0f;
        c_body = cr.body; c_slot_e = cr.slot_e;
      }
      const int my_e = jrole ? js_e : (c_slot_e % E);
      const int my_blk = jrole ? (js_j < J ? js_j : 0) : J + c_slot_e / E;
      const bool writes_partial = jrole ? (js_on && js_side == 0) : has_contact;
      const int j_ob = jrole ? (js_side ? Ltjoint[js_j < J ? js_j : 0].child : Ltjoint[js_j < J ? js_j : 0].parent) : 0;
      const int j_bo = j_ob < 0 ? 0 : j_ob;
      // the velocity change of the lane's own body from the impulses xv of its rows -> its copy
      auto scatter = [&](const float* xv) {
        if (jrole) {
          if (js_on && j_ob >= 0) {
            float dw[3] = {0.0f, 0.0f, 0.0f};
            for (int k = 0; k < 3; ++k)
              for (int c = 0; c < 3; ++c) dw[c] += K[5 + 3 * k + c] * xv[k] + K[23 + 3 * k + c] * xv[3 + k];
            for (int c = 0; c < 3; ++c) {
              Loutj[(js_j * kJS + js_side * kSide + c) * E + js_e] = K[3] * xv[c];
              Loutj[(js_j * kJS + js_side * kSide + 3 + c) * E + js_e] = dw[c];
            }
          }
        } else if (has_contact) {
          const int ee = c_slot_e % E, sl = c_slot_e / E;
          float dv[3] = {0.0f, 0.0f, 0.0f}, dw[3] = {0.0f, 0.0f, 0.0f};
          for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) { dv[c] += K[27] * K[3 * r + c] * xv[r]; dw[c] += K[18 + 3 * r + c] * xv[r]; }
          for (int c = 0; c < 3; ++c) { Loutc[(sl * kCS + c) * E + ee] = dv[c]; Loutc[(sl * kCS + 3 + c) * E + ee] = dw[c]; }
        }
      };
      // every body: the plain sum of its blocks' contributions (in static order), on top of the
      // velocities the solve started from when `with_base`
      // (split like the average of a sweep: the host only picks launch shapes where 2 B E threads
      //  exist; all reads are issued before the first use)
      auto gather_sum = [&](bool with_base, float* dst) {
        if (!g_on) return;
        const int ho = kPartC * g_part * E;
        float val[NJ + 3][kPartC], base[kPartC];
#pragma unroll
        for (int c = 0; c < kPartC; ++c) base[c] = with_base ? Lvel[(g_b * kVS + c) * E + e + ho] : 0.0f;
#pragma unroll
        for (int k = 0; k < NJ; ++k)
#pragma unroll
          for (int c = 0; c < kPartC; ++c) val[k][c] = lds[gat_off[k] + ho + c * E];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int c = 0; c < kPartC; ++c) val[NJ + k][c] = lds[gat_slot[k] + ho + c * E];
#pragma unroll
        for (int c = 0; c < kPartC; ++c) {
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < NJ + 3; ++k) acc += val[k][c];
          dst[(g_b * kVS + c) * E + e + ho] = base[c] + acc;
        }
      };
      // y = J (body vectors in src) for the lane's rows
      auto rows_of = [&](const float* src, float* y) {
        const int bo = jrole ? j_bo : c_body, ee = my_e;
        float uv[3], uw[3];
        for (int c = 0; c < 3; ++c) { uv[c] = src[(bo * kVS + c) * E + ee]; uw[c] = src[(bo * kVS + 3 + c) * E + ee]; }
        if (jrole) {
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const float p0 = K[4] * uv[k] + cross_unit_dot(K, k, uw);
            y[k] = p0 + lane_swap1(p0);
            const float p1 = K[14 + 3 * k] * uw[0] + K[15 + 3 * k] * uw[1] + K[16 + 3 * k] * uw[2];
            y[3 + k] = p1 + lane_swap1(p1);
          }
        } else {
          for (int r = 0; r < 3; ++r) {
            y[r] = (K[3 * r] * uv[0] + K[3 * r + 1] * uv[1] + K[3 * r + 2] * uv[2]) +
                   (K[9 + 3 * r] * uw[0] + K[10 + 3 * r] * uw[1] + K[11 + 3 * r] * uw[2]);
            y[3 + r] = 0.0f;
          }
        }
      };
      // totals over the rows of the lane's env of up to three products
      // (indices of the adding threads, worked out once)
      const bool red_on = tid < 3 * kRedParts * E;
      const int red_q = tid / (kRedParts * E), red_r = tid - red_q * (kRedParts * E), red_part = red_r / E, red_e = red_r - red_part * E;
      const int red_per = (nblk + kRedParts - 1) / kRedParts;
      const int red_src = (red_q * nblk + red_part * red_per) * E + red_e, red_n = min(red_per, nblk - red_part * red_per);
      const int red_dst = (red_q * kRedParts + red_part) * E + red_e;
      auto reduce3 = [&](float pa, float pb, float pc, float& ta, float& tb, float& tc) {
        if (writes_partial) {
          Lred[(0 * nblk + my_blk) * E + my_e] = pa; Lred[(1 * nblk + my_blk) * E + my_e] = pb; Lred[(2 * nblk + my_blk) * E + my_e] = pc;
        }
        __syncthreads();
        // four threads per product and env add up a quarter of the blocks each (reads issued together)
        if (red_on) {
          float vals[16];
#pragma unroll
          for (int k = 0; k < 16; ++k) vals[k] = k < red_n ? Lred[red_src + k * E] : 0.0f;
          float sm = 0.0f;
#pragma unroll
          for (int k = 0; k < 16; ++k) sm += vals[k];
          Lsum[red_dst] = sm;
        }
        __syncthreads();
        // every lane adds the four partial sums of its env, in order
        float vals[3 * kRedParts];
#pragma unroll
        for (int k = 0; k < 3 * kRedParts; ++k) vals[k] = Lsum[k * E + my_e];
        ta = (vals[0] + vals[1]) + (vals[2] + vals[3]);
        tb = (vals[4] + vals[5]) + (vals[6] + vals[7]);
        tc = (vals[8] + vals[9]) + (vals[10] + vals[11]);
      };
      float lam[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (WS != 0) {
        // Warm start: the first iterate is the share of what the rows ended the last substep with
        // (a limit row only if it stands for the same limit as then; a slot that was not active
        // then holds zero).
        if (jrole) {
          if (js_on) {
            for (int k = 0; k < 3; ++k) lam[k] = p_warm * Lwj[(js_j * 6 + k) * E + js_e];
            for (int k = 0; k < 3; ++k) {
              const float kept = Lwj[(js_j * 6 + 3 + k) * E + js_e];
              float l0 = p_warm * kept;
              if ((ones >> k) & 1) {
                const bool was_upper = __float_as_int(kept) < 0, is_upper = (uppers >> k) & 1;
                l0 = was_upper == is_upper ? fabsf(l0) : 0.0f;
              }
              lam[3 + k] = l0;
            }
          }
        } else if (has_contact) {
          for (int r = 0; r < 3; ++r) lam[r] = cr.lam[r];
        }
      }
      for (int it = 0; it < a.iterations; ++it) {
        float sres[6], known[6], cp[6], ipd[6], tmp[6];
        int on = 0;
        // residual of the current iterate
        scatter(lam);
        __syncthreads();
        gather_sum(true, LU);
        __syncthreads();
        rows_of(LU, sres);
        for (int k = 0; k < 6; ++k) { sres[k] += bs[k]; known[k] = 0.0f; cp[k] = 0.0f; }
        // the branch every row is on
        if (jrole) {
          on = 7;
          for (int k = 0; k < 3; ++k) {
            const bool one = (ones >> k) & 1;
            const bool s_branch = !one || (Dg[3 + k] > 0.0f && lam[3 + k] - sres[3 + k] / Dg[3 + k] > 0.0f);
            if (s_branch) on |= 8 << k; else known[3 + k] = -lam[3 + k];
          }
        } else {
          if (Dg[0] > 0.0f && lam[0] - sres[0] / Dg[0] > 0.0f) on |= 1; else known[0] = -lam[0];
          const float rad = p_mu * lam[0];
          if (rad > 0.0f) {
            on |= 6;
            cp[1] = cp[2] = sqrtf(sres[1] * sres[1] + sres[2] * sres[2] + kFrictionEps * kFrictionEps) / rad;
          } else { known[1] = -lam[1]; known[2] = -lam[2]; }
        }
        // (ipd: inverse of the preconditioner's diagonal on the rows of the "s" branch, 0 elsewhere)
        for (int k = 0; k < 6; ++k) {
          const float pdk = Dg[k] * (1.0f + p_reg) + cp[k];
          if (!(pdk > 0.0f) || k >= nr || !active) on &= ~(1 << k);
          ipd[k] = ((on >> k) & 1) ? 1.0f / pdk : 0.0f;
        }
        // right-hand side of the rows on the "s" branch: -s - c lambda - A known
        scatter(known);
        __syncthreads();
        gather_sum(false, LU);
        __syncthreads();
        rows_of(LU, tmp);
        float x[6], z[6], pv[6], q[6], az[6];
        for (int k = 0; k < 6; ++k) {
          const bool o = (on >> k) & 1;
          const float rhs = o ? -sres[k] - cp[k] * lam[k] - tmp[k] : 0.0f;
          x[k] = 0.0f; z[k] = rhs * ipd[k]; pv[k] = z[k];
        }
        // (A + reg D + c) z on the rows of the "s" branch
        auto apply_hat = [&](const float* xv, float* y) {
          scatter(xv);
          __syncthreads();
          gather_sum(false, LU);
          __syncthreads();
          rows_of(LU, y);
          for (int k = 0; k < 6; ++k) y[k] = ((on >> k) & 1) ? y[k] + (p_reg * Dg[k] + cp[k]) * xv[k] : 0.0f;
        };
        apply_hat(z, az);
        float gamma, den, unused;
        {
          float pa = 0.0f, pb = 0.0f;
          for (int k = 0; k < 6; ++k) { q[k] = az[k]; pa += z[k] * az[k]; pb += az[k] * az[k] * ipd[k]; }
          reduce3(pa, pb, 0.0f, gamma, den, unused);
        }
        const float gamma0 = gamma;
        bool done = false;
        for (int kk = 0; kk < n_kry; ++kk) {
          done = done || !(den > 0.0f) || !(gamma > 1e-12f * gamma0);
          const float alpha = done ? 0.0f : gamma / den;
          for (int k = 0; k < 6; ++k) { x[k] += alpha * pv[k]; z[k] -= alpha * q[k] * ipd[k]; }   // (all zero off the "s" branch)
          if (kk == n_kry - 1) break;       // (the last iteration's operator product would not be used)
          apply_hat(z, az);
          float pa = 0.0f, pb = 0.0f, pc = 0.0f, ta, tb, tc;
          for (int k = 0; k < 6; ++k) {
            pa += z[k] * az[k];
            pb += az[k] * az[k] * ipd[k]; pc += az[k] * q[k] * ipd[k];
          }
          reduce3(pa, pb, pc, ta, tb, tc);
          if (!done) {
            const float beta = ta / gamma;
            for (int k = 0; k < 6; ++k) { pv[k] = z[k] + beta * pv[k]; q[k] = az[k] + beta * q[k]; }
            den = tb + 2.0f * beta * tc + beta * beta * den;     // q . q / pd of the new q
            gamma = ta;
          }
        }
        // update, then back into the feasible set
        for (int k = 0; k < 6; ++k) lam[k] += ((on >> k) & 1) ? x[k] : known[k];
        if (jrole) {
          for (int k = 0; k < 3; ++k) if ((ones >> k) & 1) lam[3 + k] = fmaxf(lam[3 + k], 0.0f);
        } else {
          lam[0] = fmaxf(lam[0], 0.0f);
          const float rad = p_mu * lam[0], nrm = sqrtf(lam[1] * lam[1] + lam[2] * lam[2]);
          if (nrm > rad) { const float sc = nrm > 0.0f ? rad / nrm : 0.0f; lam[1] *= sc; lam[2] *= sc; }
        }
      }
      // the solved velocities: v* + M^-1 J^T lambda
      scatter(lam);
      __syncthreads();
      gather_sum(true, Lvel);
      __syncthreads();
      if constexpr (WS != 0) {
        // kept for the next substep (both lanes of a joint hold the same impulses; everybody has
        // read the old ones before the barriers above)
        if (jrole) {
          if (js_on && js_side == 0) {
            for (int k = 0; k < 3; ++k) Lwj[(js_j * 6 + k) * E + js_e] = lam[k];
            for (int k = 0; k < 3; ++k)
              Lwj[(js_j * 6 + 3 + k) * E + js_e] = ((ones & uppers) >> k) & 1 ? -lam[3 + k] : lam[3 + k];
          }
        } else if (has_contact) {
          const int ee = c_slot_e % E, sl = c_slot_e / E;
          for (int r = 0; r < 3; ++r) Lwc[(sl * 3 + r) * E + ee] = lam[r];
        }
      }
    } else
    if (joint_wave) {
      // (lanes behind the last joint do what its lanes do, to the last bit)
      const int jj = js_j < J ? js_j : J - 1;
      JointRows jw;
      QuadRows qr;
      int q_onesided = 0, q_upper = 0;
      if constexpr (JL == 1) build_joint(jw, js_j, js_e);
      else if constexpr (JL == 4) build_quad(qr, jj, js_e, js_side, js_kind != 0, q_onesided, q_upper);
      else build_joint_side(js_j, js_e, js_side);
      if constexpr (kPairsInJoints) build_pair();
      if (PC == 0 && m_terrain == 0) __syncthreads();   // (the velocities, which the other wavefronts integrate meanwhile)
      TMARK(17);
      float acc[3] = {0.0f, 0.0f, 0.0f};   // impulses of the positional rows so far (kept for the next substep)
      if constexpr (WS != 0 && JL == 4) {
        for (int k = 0; k < 3; ++k) {
          const float kept = Lwj[(jj * 6 + 3 * js_kind + k) * E + js_e];
          float l0 = p_warm * kept;
          if (js_kind && (q_onesided & (1 << k))) {
            // kept for the other limit: it would push the wrong way
            const bool was_upper = __float_as_int(kept) < 0, is_upper = (q_upper >> k) & 1;
            l0 = was_upper == is_upper ? fabsf(l0) : 0.0f;
            qr.nl[k] = -l0;
          }
          qr.lam[k] = l0;
        }
      } else if constexpr (WS != 0) {
        for (int k = 0; k < 3; ++k) acc[k] = p_warm * Lwj[(jj * 6 + k) * E + js_e];
        for (int k = 0; k < 3; ++k) {
          const float kept = Lwj[(jj * 6 + 3 + k) * E + js_e];
          const int onesided = JL == 1 ? jw.onesided : jr.onesided, upper = JL == 1 ? jw.upper : jr.upper;
          float l0 = p_warm * kept;
          if (onesided & (1 << k)) {
            const bool was_upper = __float_as_int(kept) < 0, is_upper = (upper >> k) & 1;
            l0 = was_upper == is_upper ? fabsf(l0) : 0.0f;
          }
          (JL == 1 ? jw.lam[k] : jr.lam[k]) = l0;
          if (onesided & (1 << k)) (JL == 1 ? jw.nl[k] : jr.nl[k]) = -l0;
        }
      }
      // own body's velocity rows, found once (the world's side of a joint reads body 0's): looked up
      // inside the loop, the body index costs every sweep an LDS round trip
      // ahead of the reads that depend on it
      const int js_ob = js_side ? Ltjoint[jj].child : Ltjoint[jj].parent;
      const int js_voff = P.vel + ((js_ob < 0 ? 0 : js_ob) * kVS + 3 * js_kind) * E + js_e;
      const int js_out = P.outj + (jj * kJS + js_side * kSide + 3 * js_kind) * E + js_e;
      // Where a robot can have more joint wavefronts than there are SIMDs, they share SIMDs with each other and with the
      // contacts (16 envs with two lanes per joint: a humanoid has six; 4096 of them, cycles per sweep with DPP moves and
      // through the crossbar: 1274 and 1198, with the warm start, in 512 threads, 1330 and 1225); three of a smaller
      // workgroup have theirs to themselves.
      constexpr bool kSharedSimd = JL * kMaxJoints * EC > 4 * 64;
      constexpr int kC = JL == 4 ? 3 : (JL == 2 ? 6 : 12);   // velocity components of a lane
      // (one lane per joint: the child's rows besides; the world's velocity is read from the zeros)
      const int js_voff0 = JL == 1 && js_ob < 0 ? P.zero + js_e : js_voff;
      const int js_voff1 = P.vel + Ltjoint[jj].child * kVS * E + js_e;
      sweeps([&](int it) {
        const bool start_only = WS != 0 && it < 0;
        float own[kC], mine[kC];
#pragma unroll
        for (int c = 0; c < kC; ++c) own[c] = lds[JL == 1 && c >= 6 ? js_voff1 + (c - 6) * E : js_voff0 + c * E];
        if constexpr (JL == 1) {
          float d[3], dl[3];
          if (start_only) {
            for (int k = 0; k < 3; ++k) { d[k] = acc[k]; dl[k] = jw.lam[k]; }
          } else {
            const float *va = own, *wa = own + 3, *vb = own + 6, *wb = own + 9;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
              const float pa = cross_unit_dot(jw.sr[0], k, wa) - va[k], pb = cross_unit_dot(jw.sr[1], k, wb) + vb[k];
              const float qa = fma_(jw.sax[0][k][k], wa[k], fma_(jw.sax[0][k][k1], wa[k1], jw.sax[0][k][k2] * wa[k2]));
              const float qb = fma_(jw.sax[1][k][k], wb[k], fma_(jw.sax[1][k][k1], wb[k1], jw.sax[1][k][k2] * wb[k2]));
              d[k] = fma_(pa + pb, jw.pme[k], jw.pnb[k]);
              dl[k] = fma_(qa + qb, jw.ame[k], jw.anb[k]);
            }
            d[1] = fma_(jw.pp[0], d[0], d[1]);
            d[2] = fma_(jw.pp[2], d[1], fma_(jw.pp[1], d[0], d[2]));
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
              for (int k = 0; k < 3; ++k) dl[k] = fma_(jw.ap[k][c], d[c], dl[k]);
            dl[0] = max_of(dl[0], jw.nl[0]);
            dl[1] = max_of(fma_(jw.aa[0], dl[0], dl[1]), jw.nl[1]);
            dl[2] = max_of(fma_(jw.aa[2], dl[1], fma_(jw.aa[1], dl[0], dl[2])), jw.nl[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              jw.nl[k] -= dl[k];
              if constexpr (WS != 0) { acc[k] += d[k]; jw.lam[k] += dl[k]; }
            }
          }
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              mine[6 * s + c] = jw.sv[s] * d[c];
              mine[6 * s + 3 + c] = sum3(jw.Y[s][0][c], d[0], jw.Y[s][1][c], d[1], jw.Y[s][2][c], d[2]) +
                                    sum3(jw.Z[s][0][c], dl[0], jw.Z[s][1][c], dl[1], jw.Z[s][2][c], dl[2]);
            }
        } else if constexpr (JL == 2) {
          float d[3], dl[3];   // impulses of the positional and of the angular rows
          if (start_only) {
            for (int k = 0; k < 3; ++k) { d[k] = acc[k]; dl[k] = jr.lam[k]; }
          } else {
            const float *vo = own, *wo = own + 3;
            float jv[6];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
              jv[k] = fma_(jr.sg, vo[k], cross_unit_dot(jr.sr, k, wo));
              jv[3 + k] = fma_(jr.sax[k][k], wo[k], fma_(jr.sax[k][k1], wo[k1], jr.sax[k][k2] * wo[k2]));
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) jv[k] += kSharedSimd ? lane_swap1_crossbar(jv[k]) : lane_swap1(jv[k]);
#pragma unroll
            for (int k = 0; k < 3; ++k) { d[k] = fma_(jv[k], jr.pme[k], jr.pnb[k]); dl[k] = fma_(jv[3 + k], jr.ame[k], jr.anb[k]); }
            d[1] = fma_(jr.pp[0], d[0], d[1]);
            d[2] = fma_(jr.pp[2], d[1], fma_(jr.pp[1], d[0], d[2]));
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
              for (int k = 0; k < 3; ++k) dl[k] = fma_(jr.ap[k][c], d[c], dl[k]);
            // a limit row's impulse stays >= 0: max(lam + dl, 0) - lam = max(dl, -lam)
            dl[0] = max_of(dl[0], jr.nl[0]);
            dl[1] = max_of(fma_(jr.aa[0], dl[0], dl[1]), jr.nl[1]);
            dl[2] = max_of(fma_(jr.aa[2], dl[1], fma_(jr.aa[1], dl[0], dl[2])), jr.nl[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              jr.nl[k] -= dl[k];
              if constexpr (WS != 0) { acc[k] += d[k]; jr.lam[k] += dl[k]; }
            }
          }
          // (the world's side of a joint responds to nothing and nobody reads its entry)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            mine[c] = jr.sv * d[c];
            mine[3 + c] = sum3(jr.Y[0][c], d[0], jr.Y[1][c], d[1], jr.Y[2][c], d[2]) +
                          sum3(jr.Z[0][c], dl[0], jr.Z[1][c], dl[1], jr.Z[2][c], dl[2]);
          }
        } else {
          // lanes 0, 1 of the four hold the positional rows and v of either side, lanes 2, 3 the angular rows and w
          float d[3];
          if (start_only) {
            for (int k = 0; k < 3; ++k) d[k] = qr.lam[k];
          } else {
            float w[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c] = quad_move<0xEE>(own[c]);   // from lane 2, 3, 2, 3
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
              float y;
              if (k == 0) y = fma_(qr.K[k][0], w[0], fma_(qr.K[k][1], w[1], qr.K[k][2] * w[2]));
              else y = fma_(qr.K[k][k], w[k], fma_(qr.K[k][k1], w[k1], qr.K[k][k2] * w[k2]));
              d[k] = fma_(qr.kv, own[k], y);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) d[k] += lane_swap1(d[k]);
#pragma unroll
            for (int k = 0; k < 3; ++k) d[k] = fma_(d[k], qr.me[k], qr.nb[k]);
            d[1] = fma_(qr.t1[0], d[0], d[1]);
            d[2] = fma_(qr.t1[2], d[1], fma_(qr.t1[1], d[0], d[2]));
            float dp[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) dp[c] = quad_move<0x44>(d[c]);    // from lane 0, 1, 0, 1
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
              for (int k = 0; k < 3; ++k) d[k] = fma_(qr.ap[k][c], dp[c], d[k]);
            d[0] = max_of(d[0], qr.nl[0]);
            d[1] = max_of(fma_(qr.t2[0], d[0], d[1]), qr.nl[1]);
            d[2] = max_of(fma_(qr.t2[2], d[1], fma_(qr.t2[1], d[0], d[2])), qr.nl[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              qr.nl[k] -= d[k];
              if constexpr (WS != 0) qr.lam[k] += d[k];
            }
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float r = sum3(qr.R[0][c], d[0], qr.R[1][c], d[1], qr.R[2][c], d[2]);
            const float both = r + quad_move<0x44>(r);
            mine[c] = js_kind ? both : qr.sv * d[c];
          }
        }
#pragma unroll
        for (int c = 0; c < kC; ++c) lds[js_out + (c < 6 ? c : c - 6 + kSide) * E] = mine[c];
        if constexpr (kPairsInJoints) pair_sweep(!start_only);
      });
      if constexpr (WS != 0) {
        // (both lanes of a joint hold the same impulses; the two sit in one wavefront, so the
        // parent side's stores follow both lanes' reads above)
        if (js_on && js_side == 0) {
          if constexpr (JL == 4) {
            for (int k = 0; k < 3; ++k)
              Lwj[(js_j * 6 + 3 * js_kind + k) * E + js_e] = js_kind && (((q_onesided & q_upper) >> k) & 1) ? -qr.lam[k] : qr.lam[k];
          } else {
            const int uppers = JL == 1 ? jw.onesided & jw.upper : jr.onesided & jr.upper;
            for (int k = 0; k < 3; ++k) Lwj[(js_j * 6 + k) * E + js_e] = acc[k];
            for (int k = 0; k < 3; ++k) {
              const float l = JL == 1 ? jw.lam[k] : jr.lam[k];
              Lwj[(js_j * 6 + 3 + k) * E + js_e] = (uppers >> k) & 1 ? -l : l;
            }
          }
        }
      }
    } else {
      if constexpr (WS != 0) {
        // a slot that is not active in this substep hands nothing on to the next one (nobody
        // reads its entries now; the records are final since the barrier after the contact search)
        for (int i = tid - joint_threads; i < S * E; i += n_reg)
          if (!Lreci[(i / E * kRecWords + 0) * E + i % E])
            for (int r = 0; r < 3; ++r) Lwc[(i / E * 3 + r) * E + i % E] = 0.0f;
      }
      if (PC == 0 && m_terrain == 0) {
        // plane: the torques are complete only now; the forces are integrated beside the joint rows
        forces(joint_threads);
      }
      build_contact();
      build_pair();
      if (PC == 0 && m_terrain == 0) __syncthreads();
      {
        // (a lane without a contact of its own does what the last contact's lane of its wavefront does, to the last bit)
        // (up to four envs have a contact thread for every slot a robot can have)
        constexpr bool kMoreContacts = EC == 0 || kMaxSlots * EC > NT - ((JL * kMaxJoints * EC + 63) / 64) * 64;
        const bool contacts_here = __ballot(has_contact) != 0ull, more_contacts = kMoreContacts && n_active > n_reg;
        if constexpr (kMoreContacts) {
          // the starting impulses of the contacts beyond one per thread are set by the thread that
          // relaxes them in every sweep below (same index mapping), so no other thread's store is read
          for (int k = n_reg + (kThreads - 1 - tid); k < n_active; k += n_reg)
            for (int r = 0; r < 3; ++r) overflow_lam(k, r) = WS ? p_warm * overflow_lam(k, r) : 0.0f;
        }
        const int c_e = cr.slot_e % E, c_out = P.outc + (cr.slot_e / E) * kCS * E + c_e, c_voff = P.vel + cr.body * kVS * E + c_e;
        auto own_contact = [&](int it) {
            float vv[3], ww[3];
            for (int k = 0; k < 3; ++k) { vv[k] = lds[c_voff + k * E]; ww[k] = lds[c_voff + (3 + k) * E]; }
            if (WS != 0 && it < 0) contact_response(cr, cr.lam, vv, ww);
            else relax_contact(cr, p_mu, vv, ww);
            for (int k = 0; k < 3; ++k) { lds[c_out + k * E] = vv[k]; lds[c_out + (3 + k) * E] = ww[k]; }
        };
        if (more_contacts) sweeps([&](int it) {
          own_contact(it);
          for (int k = n_reg + (kThreads - 1 - tid); k < n_active; k += n_reg) {
            // rare: more active contacts in the workgroup than threads; rows rebuilt from the record
            const int i = Llist[k];
            const int ee = i % E, sl = i / E, body = Ltslot[2 * sl];
            ContactRows c2;
            build_contact_rows(c2, Lrec, Liw, weight_sum(body, ee), sl, ee, E, body, Ltbody[4 * body + 3], h, p_beta_c, p_vdepen);
            for (int r = 0; r < 3; ++r) c2.lam[r] = overflow_lam(k, r);
            float vv[3], ww[3];
            for (int r = 0; r < 3; ++r) { vv[r] = Lvel[(body * kVS + r) * E + ee]; ww[r] = Lvel[(body * kVS + 3 + r) * E + ee]; }
            if (WS != 0 && it < 0) contact_response(c2, c2.lam, vv, ww);
            else relax_contact(c2, p_mu, vv, ww);
            for (int r = 0; r < 3; ++r) overflow_lam(k, r) = c2.lam[r];
            for (int r = 0; r < 3; ++r) { Loutc[(sl * kCS + r) * E + ee] = vv[r]; Loutc[(sl * kCS + 3 + r) * E + ee] = ww[r]; }
          }
          pair_sweep(!(WS != 0 && it < 0));
        });
        else if (contacts_here) sweeps([&](int it) { own_contact(it); pair_sweep(!(WS != 0 && it < 0)); });
        else sweeps([&](int it) { pair_sweep(!(WS != 0 && it < 0)); });
      }
      if constexpr (WS != 0) {
        if (has_contact) {
          const int ee = cr.slot_e % E, sl = cr.slot_e / E;
          for (int r = 0; r < 3; ++r) Lwc[(sl * 3 + r) * E + ee] = cr.lam[r];
        }
      }
    }

    TMARK(6);
    // ---- E: damping, angular-velocity cap, positions
    if (is_body) {
      // the pose was parked in LDS during the sweeps (unchanged since phase A)
      for (int c = 0; c < 3; ++c) x[c] = Lpos[(b * 7 + c) * E + e];
      for (int c = 0; c < 4; ++c) q[c] = Lpos[(b * 7 + 3 + c) * E + e];
      // the solved velocities were left in LDS by the threads that averaged them
      for (int c = 0; c < 3; ++c) { v[c] = Lvel[(b * kVS + c) * E + e]; w[c] = Lvel[(b * kVS + 3 + c) * E + e]; }
      float dl = __builtin_amdgcn_rcpf(fma_(h, p_clin, 1.0f)), da = __builtin_amdgcn_rcpf(fma_(h, p_cang, 1.0f));
      for (int c = 0; c < 3; ++c) { v[c] *= dl; w[c] *= da; }
      const float w2 = dot(w, w);
      if (w2 > p_wmax * p_wmax) { float sc = p_wmax * __builtin_amdgcn_rsqf(w2); for (int c = 0; c < 3; ++c) w[c] *= sc; }
      for (int c = 0; c < 3; ++c) x[c] = fma_(h, v[c], x[c]);
      float dq[4];
      dq[0] = fma_(-w[2], q[3], diff2(-w[0], q[1], w[1], q[2]));
      dq[1] = fma_(-w[2], q[2], sum2(w[0], q[0], w[1], q[3]));
      dq[2] = fma_(w[2], q[1], sum2(-w[0], q[3], w[1], q[0]));
      dq[3] = fma_(w[2], q[0], diff2(w[0], q[2], w[1], q[1]));
      float hh = 0.5f * h;
      for (int c = 0; c < 4; ++c) q[c] = fma_(hh, dq[c], q[c]);
      float inv = __builtin_amdgcn_rsqf(fma_(q[3], q[3], sum3(q[0], q[0], q[1], q[1], q[2], q[2])));
      for (int c = 0; c < 4; ++c) q[c] *= inv;
    }
    // Phase A of the next substep follows without a barrier: since the last sweep's barrier a body's pose
    // and velocity are touched by its own thread alone.  (Without a sweep there was none.)
    if (a.iterations <= 0) __syncthreads();
    TMARK(7);
  }

  // ---- store state, publish final pose/velocity for packing
  // What the end of the step needs of the launch arguments and of the model is read again here (two trips
  // through the scalar cache) instead of being kept in scalar registers through all substeps.
  {
  const StepArgs& a = *reload_constant(reinterpret_cast<const StepArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()));
  const Model& M = *reload_constant(a.M);
  const Field H0 = make_field(M, a.heights, a.coarse);
  const int N = a.N, m_root = M.root, m_terrain = M.terrain_kind;
  const int obs_row = obs_dim + (M.height_map ? kHmRows * kHmCols : 0);   // row of the caller's array
  int m_feet = 0;   // the feet's bodies, a byte each
#pragma unroll
  for (int f = 0; f < kMaxFeet; ++f) m_feet |= (f < F ? M.feet[f] : 0) << (8 * f);
  auto agent_at = [&](int place) -> int {
    if constexpr (PC != 0) { if (a.place_env && place < N) return a.place_env[place]; }
    return place;
  };
  const int agent = agent_at(env);
  __syncthreads();
  TMARK(8);
  if (tid < E) Llim[tid] = 0;   // joints of the env at their limits
  if (is_body) {
    float* st = a.state + (size_t)b * N + agent;
    const size_t fs = (size_t)B * N;
    if (a.substeps > 0) {
      st[0 * fs] = x[0]; st[1 * fs] = x[1]; st[2 * fs] = x[2];
      st[3 * fs] = q[0]; st[4 * fs] = q[1]; st[5 * fs] = q[2]; st[6 * fs] = q[3];
      st[7 * fs] = v[0]; st[8 * fs] = v[1]; st[9 * fs] = v[2];
      st[10 * fs] = w[0]; st[11 * fs] = w[1]; st[12 * fs] = w[2];
    }
    for (int c = 0; c < 3; ++c) Lpos[(b * 7 + c) * E + e] = x[c];
    for (int c = 0; c < 4; ++c) Lpos[(b * 7 + 3 + c) * E + e] = q[c];
    for (int c = 0; c < 3; ++c) { Lvel[(b * kVS + c) * E + e] = v[c]; Lvel[(b * kVS + 3 + c) * E + e] = w[c]; }
  }
  __syncthreads();

  // The observation is packed once for every env (pass 0).  With the task logic's auto-reset, an
  // env whose episode ends in pass 0 is put back to a fresh initial state right here, and pass 1
  // packs the observation of that state for it (no action, no contact), so the caller gets the
  // finished step's reward and done flag next to the first observation of the next episode.
  // sim_reset is a launch without substeps that goes straight to the reset and packs every env in pass 1.
  // (Two copies of the packing: as a loop over the passes the addresses of both are computed ahead of it,
  // 1.3 us of a step of 16 ants.)
  int* Lrst = reinterpret_cast<int*>(Lpush);   // [E]: env is reset (the pushes are no longer read)
  const bool may_reset = a.task.enabled && a.task.auto_reset && a.count_step;
  const bool only_reset = a.substeps == 0 && a.reset;
  // ---- observation vector (Table 2 "Ours"), per joint part
  auto pack_joints = [&](auto pass_c) {
#pragma clang fp contract(fast)
  constexpr int pass = decltype(pass_c)::value;
  if (is_joint && (pass == 0 || only_reset || Lrst[e])) {
    const JointTab& jt = Ltjoint[idx];
    const int pa = jt.parent, pb = jt.child;
    float qa[4] = {1, 0, 0, 0}, wa[3] = {0, 0, 0}, qb[4], wb[3];
    if (pa >= 0) {
      for (int c = 0; c < 4; ++c) qa[c] = Lpos[(pa * 7 + 3 + c) * E + e];
      for (int c = 0; c < 3; ++c) wa[c] = Lvel[(pa * kVS + 3 + c) * E + e];
    }
    for (int c = 0; c < 4; ++c) qb[c] = Lpos[(pb * 7 + 3 + c) * E + e];
    for (int c = 0; c < 3; ++c) wb[c] = Lvel[(pb * kVS + 3 + c) * E + e];
    float Ra[9], phi[3];
    quat_to_mat(qa, Ra);
    rel_rotvec(qa, qb, phi);
    float dw[3] = {wb[0] - wa[0], wb[1] - wa[1], wb[2] - wa[2]};
    int at_limit = 0;
    for (int k = 0; k < 3; ++k) {
      if (jt.mode[k] != 1) continue;
      int ai = jt.act[k];
      float ak[3];
      mat_vec(Ra, jt.axes[k], ak);
      float th = dot(jt.axes[k], phi);
      Lobs[e * obs_dim + 11 + ai] = th;
      Lobs[e * obs_dim + 11 + D + ai] = dot(ak, dw);
      Lobs[e * obs_dim + 11 + 2 * D + ai] = pass ? 0.0f : Lu[ai * E + e];
      float g = fminf(th - jt.lo[k], jt.hi[k] - th);
      at_limit += g <= 0.0f ? 1 : 0;
    }
    if (at_limit) atomicAdd(&Llim[e], at_limit);
  }
  };
  // ---- root part.  One thread per env for all of it is a chain of many hundred instructions (two unit
  // directions, an arctangent, an arcsine, and reads from global memory) that every other wavefront
  // waits for, so its independent parts go to a wavefront each, above the joint threads; where there
  // are not enough wavefronts the first one takes what is left.  What the reward needs of them is left
  // in LDS (the inverse inertias are no longer read).
  float* Lsc = Liw;       // [5][E]: speed towards the target, distance to it, sums of |u| and u^2, feet on the ground
  float* Lhm = Loutj;     // [5][E]: centre of mass (world), cosine and sine of the yaw (the sweeps' changes are free by now)
  const bool m_height_map = obs_row > obs_dim;
  auto pack_root = [&](auto pass_c) {
#pragma clang fp contract(fast)
  constexpr int pass = decltype(pass_c)::value;
  const int part_0 = (J * E + 63) & ~63, part_n = (E + 63) & ~63;
  auto part_env = [&](int part) -> int {   // env of this thread in that part, or -1
    int t0 = part_0 + part * part_n;
    if (t0 + part_n > kThreads) t0 = 0;
    const int ee = tid - t0;
    if (ee < 0 || ee >= E || blockIdx.x * E + ee >= N) return -1;
    return pass == 0 || only_reset || Lrst[ee] ? ee : -1;
  };
  // Cosine and sine of the direction of (x, y), as the arctangent has it: the null vector points along x, an infinite
  // component outweighs a finite one, NaN stays NaN (a pose that is none must show).  The larger component is scaled
  // into [0.5, 1) by its exponent first, so that no square overflows or vanishes.
  auto direction_of = [&](float x, float y, float& c, float& sn) {
    if (isinf(x) || isinf(y)) {
      x = isinf(x) ? copysignf(1.0f, x) : 0.0f * x; y = isinf(y) ? copysignf(1.0f, y) : 0.0f * y;
    }
    const int up = -__builtin_amdgcn_frexp_expf(fmaxf(fabsf(x), fabsf(y)));
    x = __builtin_amdgcn_ldexpf(x, up); y = __builtin_amdgcn_ldexpf(y, up);
    const float n = sqrtf(x * x + y * y);
    c = n == 0.0f ? 1.0f : x / n; sn = n == 0.0f ? 0.0f : y / n;
  };
  // cosine and sine of the heading (the yaw of the ZYX Euler angles; looking straight up or down it counts as zero)
  auto heading_of = [&](int ee, float& c, float& sn) {
    const float qw = Lpos[(m_root * 7 + 3) * E + ee], qx = Lpos[(m_root * 7 + 4) * E + ee];
    const float qy = Lpos[(m_root * 7 + 5) * E + ee], qz = Lpos[(m_root * 7 + 6) * E + ee];
    direction_of(1.0f - 2.0f * (qy * qy + qz * qz), 2.0f * (qw * qz + qx * qy), c, sn);
  };
  if (const int ee = part_env(0); ee >= 0) {
    // target in the root's frame, speed towards it
    const int env_e = agent_at(blockIdx.x * E + ee);
    const float gx = a.targets[2 * env_e], gy = a.targets[2 * env_e + 1];
    const float rx = Lpos[(m_root * 7 + 0) * E + ee], ry = Lpos[(m_root * 7 + 1) * E + ee];
    float cy, sy;
    heading_of(ee, cy, sy);
    const float rv0 = Lvel[(m_root * kVS + 0) * E + ee], rv1 = Lvel[(m_root * kVS + 1) * E + ee];
    const float tx = gx - rx, ty = gy - ry;
    const float tn = sqrtf(tx * tx + ty * ty);
    // sine and cosine of the difference of two directions from their components: no angle is formed (the two
    // arctangents and the sine and cosine of their difference were the longest chain of this phase)
    float ux, uy;
    direction_of(tx, ty, ux, uy);
    Lobs[ee * obs_dim + 9] = uy * cy - ux * sy; Lobs[ee * obs_dim + 10] = ux * cy + uy * sy;
    Lsc[0 * E + ee] = tn > 0.0f ? (rv0 * tx + rv1 * ty) / tn : 0.0f;
    Lsc[1 * E + ee] = tn;
  }
  if (const int ee = part_env(1); ee >= 0) {
    // height above the ground
    const float rx = Lpos[(m_root * 7 + 0) * E + ee], ry = Lpos[(m_root * 7 + 1) * E + ee];
    float height = Lpos[(m_root * 7 + 2) * E + ee];
    if (m_terrain == 1) {
      const HeightCell c = height_cell(H0.nx, H0.ny, H0.cell, H0.ox, H0.oy, rx + Lorg[ee], ry + Lorg[E + ee]);
      const float* hs = a.heights + c.at;
      height = height + Lorg[2 * E + ee] - height_in_cell(c.fx, c.fy, hs[0], hs[1], hs[H0.nx + 1], hs[H0.nx]);
    }
    Lobs[ee * obs_dim] = height;
  }
  if (const int ee = part_env(2); ee >= 0) {
    // roll and pitch, velocities
    const float qw = Lpos[(m_root * 7 + 3) * E + ee], qx = Lpos[(m_root * 7 + 4) * E + ee];
    const float qy = Lpos[(m_root * 7 + 5) * E + ee], qz = Lpos[(m_root * 7 + 6) * E + ee];
    for (int c = 0; c < 6; ++c) Lobs[ee * obs_dim + 3 + c] = Lvel[(m_root * kVS + c) * E + ee];
    Lobs[ee * obs_dim + 1] = atan2f(2.0f * (qw * qx + qy * qz), 1.0f - 2.0f * (qx * qx + qy * qy));
    Lobs[ee * obs_dim + 2] = asinf(fminf(fmaxf(2.0f * (qw * qy - qz * qx), -1.0f), 1.0f));
  }
  if (const int ee = part_env(3); ee >= 0) {
    // feet on the ground: the records of all their slots are read together (slot after slot, with a branch around
    // each, this part was what everybody waited for: 4600 cycles of two ants' 6300 between state and reward)
    int active[kMaxFeet][3], slots[kMaxFeet];
    float gap[kMaxFeet][3];
#pragma unroll
    for (int f = 0; f < kMaxFeet; ++f) {
      const int fb = (m_feet >> (8 * f)) & 255;   // (body 0 for feet that there are not)
      const int s0 = Ltjs[fb * (kMaxBodyJoints + 3) + 1];
      slots[f] = Ltjs[fb * (kMaxBodyJoints + 3) + 2];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int sl = s0 + (k < slots[f] ? k : 0);
        active[f][k] = Lreci[(sl * kRecWords + 0) * E + ee];
        gap[f][k] = Lrec[(sl * kRecWords + 3) * E + ee];
      }
    }
    int n_feet = 0;
#pragma unroll
    for (int f = 0; f < kMaxFeet; ++f) {
      bool down = false;
#pragma unroll
      for (int k = 0; k < 3; ++k) down = down || (pass == 0 && k < slots[f] && active[f][k] != 0 && gap[f][k] <= 0.005f);
      if (f < F) Lobs[ee * obs_dim + 11 + 3 * D + f] = down ? 1.0f : 0.0f;
      n_feet += f < F && down ? 1 : 0;
    }
    Lsc[4 * E + ee] = (float)n_feet;
  }
  if (const int ee = part_env(5); ee >= 0) {
    // sums over the actions (eight reads in flight at a time)
    float l1 = 0.0f, l2 = 0.0f;
    for (int d0 = 0; d0 < D; d0 += 8) {
      float uu[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) uu[k] = Lu[(d0 + k < D ? d0 + k : D - 1) * E + ee];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (d0 + k < D) { l1 += fabsf(uu[k]); l2 += uu[k] * uu[k]; }
    }
    Lsc[2 * E + ee] = l1; Lsc[3 * E + ee] = l2;
  }
  if (m_height_map) {
    if (const int ee = part_env(4); ee >= 0) {
      // centre of mass and heading for the height map
      float cx = 0.0f, cy = 0.0f, cz = 0.0f;
      for (int bb = 0; bb < B; ++bb) {
        const float mf = M.body_mass_frac[bb];
        cx += mf * Lpos[(bb * 7 + 0) * E + ee]; cy += mf * Lpos[(bb * 7 + 1) * E + ee]; cz += mf * Lpos[(bb * 7 + 2) * E + ee];
      }
      Lhm[0 * E + ee] = cx + Lorg[ee]; Lhm[1 * E + ee] = cy + Lorg[E + ee]; Lhm[2 * E + ee] = cz + Lorg[2 * E + ee];
      heading_of(ee, Lhm[3 * E + ee], Lhm[4 * E + ee]);
    }
  }
  };
  // ---- reward (Eq. 1-3), done (Section 4.1), one thread per env; returns whether the env was reset
  // (what it needs from memory is read early, so that the trip passes while the observation is packed)
  const int m_max_steps = M.max_steps;
  const float m_alive = M.alive_bonus, m_term_height = M.term_height;
  int steps_before = 0;
  if (tid < E && (blockIdx.x * E + tid) < N) {
    steps_before = a.steps[agent_at(blockIdx.x * E + tid)];
  }
  auto finish_env = [&]() -> bool {
#pragma clang fp contract(fast)
  bool reset_now = false;
  if (tid < E && (blockIdx.x * E + tid) < N) {
    const int ee = tid, env_e = agent_at(blockIdx.x * E + tid);
    const int rb = m_root;
    const float height = Lobs[ee * obs_dim], cps = Lobs[ee * obs_dim + 10];
    const float speed = Lsc[0 * E + ee], tn = Lsc[1 * E + ee], l1 = Lsc[2 * E + ee], l2 = Lsc[3 * E + ee];
    const float n_feet = Lsc[4 * E + ee];
    const float qx = Lpos[(rb * 7 + 4) * E + ee], qy = Lpos[(rb * 7 + 5) * E + ee];
    const int n_lim = Llim[ee];
    float r_head = cps > 0.8f ? 1.0f : cps / 0.8f;
    float cvert = 1.0f - 2.0f * (qx * qx + qy * qy);
    float r_stand = cvert > 0.93f ? 1.0f : 0.0f;
    int steps = steps_before + (a.count_step ? 1 : 0);
    a.steps[env_e] = steps;
    const float rew = m_alive + speed + 0.5f * r_head + 0.05f * r_stand - 4.0f * l1 - 0.5f * l2 -
                      0.2f * (float)n_lim - n_feet;
    uint8_t dn = (height < m_term_height || steps >= m_max_steps) ? 1 : 0;
    if (a.task.enabled && a.count_step) {
      // Section 4.1: termination only after `grace` consecutive frames below the threshold;
      // flagrun target re-drawn every `period` frames or when reached; finished envs start
      // their next episode below
      int fall = a.task_i[4 * env_e + 0], age = a.task_i[4 * env_e + 1];
      const int ep = a.task_i[4 * env_e + 3];
      fall = height < m_term_height ? fall + 1 : 0;
      dn = (fall > a.task.grace || steps >= m_max_steps) ? 1 : 0;
      if (a.task.period > 0) {
        age += 1;
        if (age >= a.task.period || tn < a.task.reach) {
          float txy[2];
          task_draw_target(a.task, env_e, ep, steps, Lpos[(rb * 7 + 0) * E + ee], Lpos[(rb * 7 + 1) * E + ee], txy);
          a.targets[2 * env_e] = txy[0]; a.targets[2 * env_e + 1] = txy[1];
          age = 0;
        }
      }
      a.task_i[4 * env_e + 0] = fall; a.task_i[4 * env_e + 1] = age;
      reset_now = dn && a.task.auto_reset;
    }
    // (one copy each: the caller's array when there is one, else the library's)
    (a.reward_out ? a.reward_out : a.reward)[env_e] = rew;
    (a.done_out ? a.done_out : a.done)[env_e] = dn;
  }
  return reset_now;
  };
  // The marked envs start from the reset recipe (after a barrier behind Lrst; nothing of the sweeps'
  // changes is needed any more).
  auto reset_envs = [&](const StepArgs& a, const Model& M) {
#pragma clang fp contract(fast)
    const bool fresh = env_ok && Lrst[e];
    if (tid < E) Llim[tid] = 0;
    auto seed_of = [&](int ag) -> uint64_t {
      return only_reset ? a.reset_seed : a.task.seed + (uint64_t)(a.task_i[4 * ag + 3] + 1) * kEpisodeStride;
    };
    ResetDraw d;
    int level = -1;
    if (fresh && idx < B) reset_place_body(M, idx, agent, seed_of(agent), LdsPoses{Lpos, Lvel, E, e});
    if (fresh && idx < J) { reset_draw_joint(M, idx, agent, seed_of(agent), d); level = M.joint_level[idx]; }
    __syncthreads();
    for (int l = 0; l < M.n_levels; ++l) {
      if (level == l) reset_place_joint(Ltjoint[idx], d, LdsPoses{Lpos, Lvel, E, e});
      __syncthreads();
    }
    if (is_body && fresh) {
      float* st = a.state + (size_t)b * N + agent;
      const size_t fs = (size_t)B * N;
      for (int c = 0; c < 7; ++c) st[c * fs] = Lpos[(b * 7 + c) * E + e];
      for (int c = 0; c < 6; ++c) st[(7 + c) * fs] = Lvel[(b * kVS + c) * E + e];
    }
    if (!only_reset && tid < E && (blockIdx.x * E + tid) < N && Lrst[tid]) {
      const int ag = agent_at(blockIdx.x * E + tid);
      a.steps[ag] = 0;
      task_begin_episode(a.task, a.task_i, a.targets, ag, a.task_i[4 * ag + 3] + 1, Lpos[(m_root * 7 + 0) * E + tid], Lpos[(m_root * 7 + 1) * E + tid]);
    }
    __syncthreads();
  };
  bool resetting = only_reset;
  if (!resetting) {
    pack_joints(std::integral_constant<int, 0>{});
    pack_root(std::integral_constant<int, 0>{});
    __syncthreads();
    const bool reset_now = finish_env();
    if (may_reset) {
      if (tid < E) Lrst[tid] = reset_now ? 1 : 0;
      resetting = __syncthreads_or(reset_now);
    }
  }
  if (__builtin_expect(resetting, false)) {
    const StepArgs& a = *reload_constant(reinterpret_cast<const StepArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()));
    const Model& M = *reload_constant(a.M);   // (nothing of this is fetched ahead of the branch)
    if (only_reset) {
      if (tid < E && (blockIdx.x * E + tid) < N) {
        const int ag = agent_at(blockIdx.x * E + tid);
        const bool fresh = !a.reset_mask || a.reset_mask[ag];
        Lrst[tid] = fresh ? 1 : 0;
        if (fresh) steps_before = 0;
      }
      __syncthreads();
    }
    reset_envs(a, M);
    pack_joints(std::integral_constant<int, 1>{});
    pack_root(std::integral_constant<int, 1>{});
    __syncthreads();
    if (only_reset) finish_env();
  }
  if constexpr (WS != 0) {
    // the kept impulses go back to the workspace for the next launch; an env that was just reset
    // starts its episode without any
    if (a.substeps > 0) {
      for (int i = tid; i < (J * 6 + S * 3) * E; i += kThreads) {
        const int ee = i % E, env_i = blockIdx.x * E + ee;
        if (env_i >= N) continue;
        const bool fresh = may_reset && Lrst[ee];
        const int ag = agent_at(env_i);
        if (i < J * 6 * E) a.lam_j[(size_t)(i / E) * N + ag] = fresh ? 0.0f : Lwj[i];
        else a.lam_s[(size_t)((i - J * 6 * E) / E) * N + ag] = fresh ? 0.0f : Lwc[i - J * 6 * E];
      }
    }
  }
  {
    const int env0 = blockIdx.x * E;
    const int n_here = min(E, N - env0);
    float* const obs_dst = a.obs_out ? a.obs_out : a.obs;   // one copy: the caller's array when there is one
    const float inv_dim = __builtin_amdgcn_rcpf((float)obs_dim);
    for (int i = tid; i < n_here * obs_dim; i += kThreads) {
      const float o = Lobs[i];
      const int ee = (int)(((float)i + 0.5f) * inv_dim), k = i - ee * obs_dim;   // (i < 2^16, at most 512 envs: exact)
      obs_dst[(size_t)agent_at(env0 + ee) * obs_row + k] = o;
    }
    if (m_height_map) {
      // Height map (Section 4.1, complex-terrain task): terrain height under a 15 x 11 grid that
      // follows the centre of mass and is aligned with the root's heading, minus the height of
      // the centre of mass; written straight to the output rows (it is not staged in LDS).
      // Six points per thread at a time, their samples all in flight together: one point after the
      // other costs a trip to L2 each.
      constexpr int kHm = kHmRows * kHmCols, kPoints = 6;
      for (int i0 = tid; i0 < n_here * kHm; i0 += kPoints * kThreads) {
        float hz[kPoints], fx[kPoints], fy[kPoints], hs[kPoints][4];
        if (m_terrain == 1) {
#pragma unroll
          for (int u = 0; u < kPoints; ++u) {
            const int i = min(i0 + u * kThreads, n_here * kHm - 1);
            const int ee = i / kHm, k = i - ee * kHm, hi = k / kHmCols, hj = k - hi * kHmCols;
            const float fw = M.hm_fwd[hi], lt = M.hm_lat[hj], c = Lhm[3 * E + ee], sn = Lhm[4 * E + ee];
            const float wx = Lhm[0 * E + ee] + (c * fw - sn * lt), wy = Lhm[1 * E + ee] + (sn * fw + c * lt);
            const HeightCell hc = height_cell(H0.nx, H0.ny, H0.cell, H0.ox, H0.oy, wx, wy);
            fx[u] = hc.fx; fy[u] = hc.fy;
            const float* hp = a.heights + hc.at;
            hs[u][0] = hp[0]; hs[u][1] = hp[1]; hs[u][2] = hp[H0.nx + 1]; hs[u][3] = hp[H0.nx];
          }
#pragma unroll
          for (int u = 0; u < kPoints; ++u) hz[u] = height_in_cell(fx[u], fy[u], hs[u][0], hs[u][1], hs[u][2], hs[u][3]);
        } else {
#pragma unroll
          for (int u = 0; u < kPoints; ++u) hz[u] = 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kPoints; ++u) {
          const int i = i0 + u * kThreads;
          if (i >= n_here * kHm) break;
          const int ee = i / kHm, k = i - ee * kHm;
          obs_dst[(size_t)agent_at(env0 + ee) * obs_row + obs_dim + k] = hz[u] - Lhm[2 * E + ee];
        }
      }
    }
  }
  }
  TMARK(9);
}
#pragma clang fp contract(fast)

}  // namespace sim355
