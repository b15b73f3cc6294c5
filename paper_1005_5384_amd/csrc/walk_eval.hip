// Fused group walk + list evaluation (Sec. 2.2 + 2.3) for gfx950.
//
// The paper builds the lists with two walks (count, then write, with a host
// prefix sum between them) and evaluates them in separate kernels.  Here one
// 64-lane wavefront per work item (a group, or a chunk of 32 of its targets)
// walks the tree breadth-first itself, up to 64 candidates per step, and evaluates
// the accepted cells and opened leaves in LDS tiles of up to 64 as soon as a
// tile fills.  The lists never reach HBM, the walk needs no block barrier
// (each wave owns its LDS area, wave-ordered), and with 6.9 KB of LDS per
// wave 20 walks are in flight per CU, so their dependent gathers overlap
// other waves' arithmetic.  The waves are persistent: work items (whose
// costs differ by orders of magnitude) are handed out through per-XCD
// counters, which removed the tail of the one-block-per-item launch (11 %).
//
// The walk is the same as the two-pass walk (same test, same breadth-first
// order, ballot compaction in lane order), so the cell and leaf lists are
// identical; an export mode writes them at offsets from the count walk for
// the parity tests.  Each candidate costs one 32-byte gather (boundary +
// topology).  The frontier FIFO holds one word per opened cell (its
// children are consecutive cells); a step takes eight entries and gives each
// eight lanes, one per child.  Evaluation: the wave splits into S = floor(64 / n)
// slices of n lanes; every slice holds all n targets and takes every S-th
// source of a tile; plain FP32 per tile is folded into compensated pairs;
// slices are added up pairwise in a fixed order.
//
// Bound: VALU issue.  Measured costs per wave instruction and SIMD with four
// waves (cycles): 2.4 for FP32 and integer additions and FP32 multiplies on
// vector registers or constants, 4.2 for compares, selects, shifts, min / max,
// lane counts and anything with a scalar-register operand, 8.3 for v_rsq_f32;
// the clock falls to about 2.1 GHz under this load.  So the loops below keep
// uniform operands in vector registers, count in scalar registers and build
// lane masks there.  2^20 Plummer points, theta = 0.5: 2.01e9 -> 1.74e9
// vector instructions, 5.6 -> 4.9 million cycles, 2.53 -> 2.33 ms.
//
// A work item whose frontier outgrows its LDS queue aborts before writing any
// result and is redone by the next tier: 512-entry LDS queues, then
// 2048-entry LDS queues, then queues in global memory sized so that they
// cannot overflow.
//
// Learned acceptance criterion (LEARNED): candidates the test at theta_lo
// accepts are accepted, those the test at theta_hi opens are opened, and for
// the band in between the wave computes the 12 features of its band lanes,
// stages them as consecutive rows in LDS and runs the network on the matrix
// cores over ceil(rows / 16) tiles; a candidate is accepted iff the predicted
// log10 error is at most log10 tau_pair.  The accepted band candidates' predicted errors add up
// (FP64, sqrt of the sum of squares) into the group's budget; a work item
// whose group exceeds it drops its accumulators and walks again with the
// call's theta.  Every work item of a group makes the same decisions (same
// candidates, same network arithmetic, same reduction order).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "mlp_device.h"
#include "octgrav_internal.h"

namespace octgrav {
namespace {

using namespace dev;

constexpr int kLanes = 64;
constexpr int kTileW = 64;   // sources per tile
constexpr int kRingW = 128;  // pending cells / leaves (two tiles)

// Frontier entry: first child << 3 | (children - 1) of an opened cell (cell
// ids < 2^29).
template <int QCAP>
struct WShared {
  static constexpr int kRing = kRingW;
  int q[QCAP];
  int cring[kRingW];
  int2 lring[kRingW];  // (first particle, n particles) of opened leaves
  // Source tile: cells (com, M) [64], (Qxx, Qyy, Qzz, Qxy) [64], (Qxz, Qyz,
  // -, -) [64], or particles [64]; the network's rows; a wave's sums.
  float4 tile[3 * kTileW];
  int mark[kTileW];
};

// Orders this wave's LDS accesses: lanes read what other lanes of the same
// wave wrote before (LDS executes a wave's instructions in order).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS frontier queue of one wave.
struct LQueue {
  int* p;
  __device__ int get(uint32_t i) const { return p[i]; }
  __device__ void put(uint32_t i, int x) const { p[i] = x; }
};

typedef float v2f32 __attribute__((ext_vector_type(2)));

// One 16-byte LDS read (member-wise copies of a float4 may be split).
__device__ __forceinline__ float4 load_f4(const float4* p) {
  const v4f32 v = *reinterpret_cast<const v4f32*>(p);
  return make_float4(v[0], v[1], v[2], v[3]);
}

// Sums of the four values of lanes 0 ... 31 in a fixed order, stored by lanes 0
// ... 3 (each step halves the values a lane carries: 12 word exchanges
// instead of 40).
__device__ __forceinline__ void store_item_sums(const double* d, int lane, double* out) {
  const bool b0 = lane & 1, b1 = lane & 2;
  double k0 = b0 ? d[2] : d[0], k1 = b0 ? d[3] : d[1];
  k0 += __shfl_xor(b0 ? d[0] : d[2], 1);
  k1 += __shfl_xor(b0 ? d[1] : d[3], 1);
  double v = b1 ? k1 : k0;
  v += __shfl_xor(b1 ? k0 : k1, 2);
#pragma unroll
  for (int o = 4; o < 32; o <<= 1) v += __shfl_xor(v, o);
  if (lane < 4) out[((lane & 1) << 1) | (lane >> 1)] = v;
}

// The targets of one work item and their accumulators.  The wave splits into
// S = floor(64 / n) slices of n lanes; a tile is T = S c sources (c =
// floor(64 / S), T in [60, 64]) and slice s evaluates sources s, s + S, ...,
// so every lane runs the same number of terms, the loop counter is a scalar
// and one vector addition per term moves the LDS address (S adjacent entries
// per read: no bank conflicts; c consecutive entries per slice would need no
// addition but conflicted on a third of the LDS cycles).  A per-lane bound
// and index arithmetic on scalar operands cost four slow instructions
// per term before: compares and every instruction with a scalar-register
// operand issue at half the rate of arithmetic on vector registers.
template <bool PLAIN, int TEAM, typename SH>
struct WItem {
  const DevTree& T;
  SH& sh;
  float eps2;  // in a vector register
  int lane, nt, S, slice, c;
  int step;  // 16 S, in a vector register
  bool active, do_eval;
  float4 xi;
  Sum4 acc4;
  int64_t nsrc = 0;
  int stamp;  // last value written to sh.mark (never reused by this wave)
  int turn = 0;  // tiles of leaves until this wave evaluates one (teams)

  // Whether the next tile of leaves is this wave's: the waves of a team take turns.
  __device__ bool mine() {
    if constexpr (TEAM == 1) return true;
    const bool m = turn == 0;
    turn = m ? TEAM - 1 : turn - 1;
    return m;
  }

  // n targets from particle first on.
  __device__ void targets(int lane_, int n, int first, bool do_eval_, int stamp_) {
    lane = lane_;
    nt = n;
    S = kLanes / nt;
    c = kLanes / S;
    step = in_vgpr(16 * S);
    stamp = stamp_;
    slice = lane / nt;
    active = slice < S;
    do_eval = do_eval_;
    xi = reinterpret_cast<const float4*>(T.part)[first + lane % nt];
    acc4.zero();
  }

  __device__ int tile_size() const { return S * c; }

  // Terms per slice of a tile of cnt sources.
  __device__ int terms(int cnt) const { return cnt == S * c ? c : uni((cnt + S - 1) / S); }

  __device__ void flush_cells(uint32_t start, int cnt) {
    if (!do_eval) return;
    const float4* mp = reinterpret_cast<const float4*>(T.mp);
    const int k = terms(cnt);
    if (lane < S * k) {
      // The last entries of a partial tile repeat its last cell without mass.
      const int64_t id = sh.cring[(start + min(lane, cnt - 1)) & (SH::kRing - 1)];
      float4 a = mp[3 * id], b = mp[3 * id + 1];
      float2 d = *reinterpret_cast<const float2*>(mp + 3 * id + 2);
      if (lane >= cnt) {
        a.w = 0.f;
        b = make_float4(0.f, 0.f, 0.f, 0.f);
        d = make_float2(0.f, 0.f);
      }
      sh.tile[lane] = a;
      sh.tile[kTileW + lane] = b;
      *reinterpret_cast<float2*>(sh.tile + 2 * kTileW + lane) = d;
    }
    wave_lds_sync();
    if (active) {
      float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
      const char* t = reinterpret_cast<const char*>(sh.tile + slice);
      auto term = [&]() {
        const float4* e = reinterpret_cast<const float4*>(t);
        const v2f32 d = *reinterpret_cast<const v2f32*>(e + 2 * kTileW);
        pc_term(xi, load_f4(e), load_f4(e + kTileW), make_float4(d[0], d[1], 0.f, 0.f), eps2, ax,
                ay, az, ph);
        t += step;
      };
      int j = 0;
      for (; j + 2 <= k; j += 2) {
        term();
        term();
      }
      if (j < k) term();
      acc4.template fold<PLAIN>(ax, ay, az, ph);
    }
    wave_lds_sync();
  }

  // Adds r + q to s + e.
  __device__ static void add(float* s, float* e, const float* r, const float* q) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (PLAIN) {
        s[k] += r[k];
      } else {
        neu_add(s[k], e[k], r[k]);
        neu_add(s[k], e[k], q[k]);
      }
    }
  }

  // The slices of each target added up (in lane < nt), the upper half to the
  // lower until one is left: six steps at most.  (One after the other in
  // one lane, the 64 slices of a single target took 22 us, the eight of seven
  // targets 3.5 us.)
  __device__ void combine_slices(float* s, float* e) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s[k] = acc4.s[k];
      e[k] = PLAIN ? 0.f : acc4.c[k];
    }
    for (int n = S; n > 1;) {
      const int h = (n + 1) >> 1, from = lane + h * nt;
      float r[4], q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        r[k] = __shfl(s[k], from);
        q[k] = PLAIN ? 0.f : __shfl(e[k], from);
      }
      if (slice < n - h) add(s, e, r, q);
      n = h;
    }
  }

  // Results of the targets (lane < nt; o: its place in the input), and the item's
  // diagnostic sums.
  __device__ void store(const WalkBufs& B, int64_t w, int64_t o, float* s, float* e,
                        float* __restrict__ acc, float* __restrict__ pot) {
    double d[4] = {0.0, 0.0, 0.0, 0.0};  // m a, 1/2 m phi of this lane's target
    if (lane < nt) {
      // The target itself is in its own leaf: its self term added -m_i/eps to
      // the potential and nothing to the acceleration; remove that same value.
      const float self = self_term(xi.w, eps2);
      if (PLAIN) s[3] += self;
      else neu_add(s[3], e[3], self);
      const float a[4] = {s[0] + e[0], s[1] + e[1], s[2] + e[2], s[3] + e[3]};
      acc[3 * o + 0] = a[0];
      acc[3 * o + 1] = a[1];
      acc[3 * o + 2] = a[2];
      const double m = xi.w;
      for (int k = 0; k < 3; ++k) d[k] = m * (double)a[k];
      if (pot) {
        pot[o] = a[3];
        d[3] = 0.5 * m * (double)a[3];
      }
    }
    if (B.dpart) store_item_sums(d, lane, B.dpart + 4 * w);
  }

  // The leaves [start, start + lc) of the ring: their particles, flattened in
  // list order, tile by tile.  A leaf marks the lane at which its particles
  // begin in the tile; a ballot of the marks gives every lane its leaf.
  __device__ void flush_leaves(uint32_t start, int lc) {
    int first = 0, ln = 0;
    if (lane < lc) {
      const int2 fl = sh.lring[(start + lane) & (SH::kRing - 1)];
      first = fl.x;
      ln = fl.y;
    }
    const int incl = wave_inclusive_sum(ln);
    const int total = __builtin_amdgcn_readlane(incl, kLanes - 1);
    nsrc += total;
    if (!do_eval) return;
    const float4* part = reinterpret_cast<const float4*>(T.part);
    const int ex = incl - ln, rel = first - ex, tile = tile_size();
    for (int u0 = 0; u0 < total; u0 += tile) {
      if (!mine()) continue;
      const int cnt = min(tile, total - u0);
      const int k = terms(cnt);
      ++stamp;
      if (ln > 0 && incl > u0 && ex < u0 + kTileW) sh.mark[max(ex - u0, 0)] = stamp;
      wave_lds_sync();
      const bool mk = sh.mark[lane] == stamp;
      const int before = __popcll(__ballot(lane < lc && incl <= u0));  // leaves used up
      const int own = before + rank_below(__ballot(mk)) + (mk ? 0 : -1);
      int src = __shfl(rel, own) + u0 + lane;
      const int last = __builtin_amdgcn_readlane(src, cnt - 1);
      if (lane >= cnt) src = last;  // without mass below
      if (lane < S * k) {
        float4 p = part[src];
        if (lane >= cnt) p.w = 0.f;
        sh.tile[lane] = p;
      }
      wave_lds_sync();
      if (active) {
        float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
        const char* t = reinterpret_cast<const char*>(sh.tile + slice);
        auto term = [&]() {
          pp_term(xi, load_f4(reinterpret_cast<const float4*>(t)), eps2, ax, ay, az, ph);
          t += step;
        };
        int j = 0;
        for (; j + 4 <= k; j += 4) {
          term();
          term();
          term();
          term();
        }
        for (; j < k; ++j) term();
        acc4.template fold<PLAIN>(ax, ay, az, ph);
      }
      wave_lds_sync();
    }
  }
};

enum : int { kOverflow = 0, kDone = 1, kFallBack = 2 };

// Walks and evaluates work item w with one wave.  Returns kOverflow
// (uniformly, before writing any result) if the frontier outgrows the queue;
// with LEARNED, kFallBack (nothing written but the trace) if the group's
// budget is exceeded, *nband = band candidates visited.  cw is the value of
// cnt[g].w written by a walk with the theta test.
template <bool PLAIN, bool LEARNED, typename SH, typename Q>
__device__ int walk_eval_item(const DevTree& T, const WalkBufs& B, SH& sh, int64_t w,
                              float th2, float eps2, float* __restrict__ acc,
                              float* __restrict__ pot, Q q, uint32_t qmask, bool gmem_q,
                              bool do_eval, int cw, int* nband_out, int* stamp,
                              const MlpView* mv) {
  const int lane = threadIdx.x & (kLanes - 1);
  // Per-item constants; with the learned criterion they are held in scalar
  // registers (its network needs the vector registers).
  auto U = [](auto v) {
    if constexpr (LEARNED) return uni(v);
    else return v;
  };
  const int2 wk0 = reinterpret_cast<const int2*>(T.wwork)[w];
  const int2 wk = make_int2(U(wk0.x), U(wk0.y));
  const int64_t g = wk.x;
  const int4 gi = U(reinterpret_cast<const int4*>(T.ginfo)[g]);
  const float4* gbox = reinterpret_cast<const float4*>(T.gbox);
  const float4 gmin = U(gbox[2 * g]), gmax = U(gbox[2 * g + 1]);
  const float4* rec = reinterpret_cast<const float4*>(T.wrec);

  WItem<PLAIN, 1, SH> it{T, sh, in_vgpr(eps2)};
  const int first = gi.x + wk.y;
  it.targets(lane, uni(min(kChunk, gi.y - wk.y)), first, do_eval, *stamp);

  const bool exp = B.export_lists && wk.y == 0;
  // learned criterion state
  const bool trace = LEARNED && B.tr_s != nullptr && wk.y == 0;
  const int64_t trb = trace ? U(B.tr_off[g]) : 0, tre = trace ? U(B.tr_off[g + 1]) : 0;
  const MacGroup mg = mac_group(gmin, gmax);
  double sum2 = 0.0;
  int nband = 0;
  const int64_t xcb = exp ? U(B.c_off[g]) : 0, xce = exp ? U(B.c_off[g + 1]) : 0;
  const int64_t xlb = exp ? U(B.l_off[g]) : 0, xle = exp ? U(B.l_off[g + 1]) : 0;

  // Frontier: entries [rhead, rtail) of q.  A step takes up to eight entries
  // and gives each eight lanes, one per possible child, so no candidate has to
  // look for its entry (trees average 7 to 8 children per split cell; the
  // candidates keep their breadth-first order).
  uint32_t rhead = 0, rtail = 0;
  uint32_t chead = 0, ctail = 0, lhead = 0, ltail = 0;
  const int4 root = reinterpret_cast<const int4*>(rec)[1];
  if (root.y == 0) {  // the root is a leaf: its particles are the whole list
    if (lane == 0) {
      sh.lring[0] = make_int2(root.z, root.w);
      if (exp && xlb < xle) B.l_ids[xlb] = 0;
    }
    ltail = 1;
  } else {
    if (lane == 0) q.put(0, (root.x << 3) | (root.y - 1));
    rtail = 1;
  }
  if (gmem_q) __threadfence_block();  // queue stores complete before other lanes read
  wave_lds_sync();
  const int lent = lane >> 3, lchild = lane & 7;
  const uint32_t tile = (uint32_t)it.tile_size();
  const float th2v = in_vgpr(th2);

  // Candidate of each lane in the window of the next min(8, rtail - rh)
  // entries from rh; 0 (the root, never a candidate) for lanes without one.
  auto take = [&](uint32_t rh) {
    const int e = q.get((rh + lent) & qmask);
    const bool has = lchild <= (e & 7) && (uint32_t)lent < rtail - rh;
    return has ? (int)((uint32_t)e >> 3) + lchild : 0;
  };
  // Learned criterion: a step that runs the network also scores the next
  // step's band candidates when all of them are queued already (they come
  // before anything this step queues), so one network call serves two steps
  // with fuller tiles; the next step then reuses the candidates, tests and
  // scores kept here.
  bool have_next = false;
  int c_next = 0;
  float y_next = 0.0f;
  uint64_t mO_next = 0, mB_next = 0;

  // One walk step: tests a window of candidates and appends the accepted
  // cells, the opened leaves and the opened cells' entries.  False if the
  // queue cannot hold them.
  auto step = [&]() -> bool {
    const int c = LEARNED && have_next ? c_next : take(rhead);
    const bool valid = c != 0;
    rhead += min(8u, rtail - rhead);

    const int4 tp = reinterpret_cast<const int4*>(rec)[2 * (int64_t)c + 1];
    uint64_t mOp;
    if (LEARNED) {
      bool olo, band, accb = false;
      uint64_t mB;
      float yh = 0.0f;
      uint16_t* xs = reinterpret_cast<uint16_t*>(sh.tile);
      if (have_next) {
        have_next = false;
        olo = (mO_next >> lane) & 1;
        band = (mB_next >> lane) & 1;
        mB = mB_next;
        yh = y_next;
      } else {
        const float4* fc = reinterpret_cast<const float4*>(T.fcell);
        {
          const float4 ge = rec[2 * (int64_t)c];
          const float4 fc0 = fc[2 * (int64_t)c], fc1 = fc[2 * (int64_t)c + 1];
          olo = valid && open_cell(gmin, gmax, ge, B.mac_lo2);
          band = olo && !open_cell(gmin, gmax, ge, B.mac_hi2);
          mB = __ballot(band);
          // Band lanes stage their features as consecutive rows.
          if (band) {
            float f[kMlpIn];
            mac_features(mg, ge, fc0, fc1, f);
            mlp_stage(xs, kXsLd, rank_below(mB), f);
          }
        }
        if (mB) {
          const int ra = __popcll(mB);
          int rows = ra;
          if (rtail - rhead >= 8u) {  // the next step's eight entries are queued
            const int c2 = take(rhead);
            const float4 ge = rec[2 * (int64_t)c2];
            const float4 fc0 = fc[2 * (int64_t)c2], fc1 = fc[2 * (int64_t)c2 + 1];
            const bool olo2 = c2 != 0 && open_cell(gmin, gmax, ge, B.mac_lo2);
            const bool band2 = olo2 && !open_cell(gmin, gmax, ge, B.mac_hi2);
            const uint64_t mB2 = __ballot(band2);
            if (ra + __popcll(mB2) <= kLanes) {  // every row's score lands in its own lane
              if (band2) {
                float f[kMlpIn];
                mac_features(mg, ge, fc0, fc1, f);
                mlp_stage(xs, kXsLd, ra + rank_below(mB2), f);
              }
              rows += __popcll(mB2);
              have_next = true;
              c_next = c2;
              mO_next = __ballot(olo2);
              mB_next = mB2;
            }
          }
          // The network runs on ceil(rows / 16) tiles; lane l receives row l's output.
          wave_lds_sync();
          const float yrow = mlp_scores(*mv, xs, kXsLd, lane, (rows + 15) >> 4);
          wave_lds_sync();
          yh = __shfl(yrow, rank_below(mB));
          if (have_next) y_next = __shfl(yrow, ra + rank_below(mB_next));
        }
      }
      if (mB) {
        accb = band && yh <= B.mac_ltau;
        // 10^(2 y) = 2^(2 log2(10) y) on the FP32 exp unit; summed in FP64
        if (accb) sum2 += (double)__builtin_amdgcn_exp2f(yh * 6.64385618977472f);
        if (band && trace) {
          const int64_t k = trb + nband + rank_below(mB);
          if (k < tre) {
            B.tr_c[k] = c;
            B.tr_s[k] = yh;
          }
        }
        nband += __popcll(mB);
      }
      mOp = __ballot(olo && !accb);
    } else {
      const float4 ge = rec[2 * (int64_t)c];
      mOp = __ballot(valid) & open_mask(gmin, gmax, ge, th2v);
    }
    // The three destinations as lane masks (scalar registers): accepted cells,
    // opened leaves, opened cells with children.
    const uint64_t mLeaf = __ballot(tp.y == 0);
    const uint64_t mC = __ballot(valid) & ~mOp, mL = mOp & mLeaf, mQ = mOp & ~mLeaf;
    const uint32_t nq = (uint32_t)__popcll(mQ);
    if ((rtail + nq) - rhead > qmask + 1) return false;
    if (__builtin_amdgcn_inverse_ballot_w64(mC)) {
      const uint32_t k = ctail + rank_below(mC);
      sh.cring[k & (kRingW - 1)] = c;
      if (exp && xcb + k < xce) B.c_ids[xcb + k] = c;
    }
    if (__builtin_amdgcn_inverse_ballot_w64(mL)) {
      const uint32_t k = ltail + rank_below(mL);
      sh.lring[k & (kRingW - 1)] = make_int2(tp.z, tp.w);
      if (exp && xlb + k < xle) B.l_ids[xlb + k] = c;
    }
    if (__builtin_amdgcn_inverse_ballot_w64(mQ))
      q.put((rtail + rank_below(mQ)) & qmask, (tp.x << 3) | (tp.y - 1));
    ctail += __popcll(mC);
    ltail += __popcll(mL);
    rtail += nq;
    if (gmem_q) __threadfence_block();
    wave_lds_sync();
    return true;
  };

  // At most 63 + 64 cells or leaves are ever pending, two tiles of as few as 60.
  bool fits = true;
  if constexpr (LEARNED) {
    // Every step is followed by the evaluations it filled (with the loop below
    // the learned call took 4 % longer, 1.59 against 1.53 ms at 2^20).
    while (rhead != rtail) {
      fits = step();
      if (!fits) break;
      while (ctail - chead >= tile) {
        it.flush_cells(chead, (int)tile);
        chead += tile;
      }
      if (ltail - lhead >= (uint32_t)kTileW) {
        it.flush_leaves(lhead, kTileW);
        lhead += kTileW;
      }
    }
    if (fits) {
      while (ctail != chead) {
        const int n = (int)min(tile, ctail - chead);
        it.flush_cells(chead, n);
        chead += n;
      }
      while (ltail != lhead) {
        const int n = (int)min((uint32_t)kTileW, ltail - lhead);
        it.flush_leaves(lhead, n);
        lhead += n;
      }
    }
  } else {
    // Steps until a tile of cells or 64 leaves are pending, then one
    // evaluation, so that the accumulators stay in their registers through the
    // walk's loop (evaluating inside it cost 16 moves a step); at the end the
    // remainders.
    for (;;) {
      while (rhead != rtail && ctail - chead < tile && ltail - lhead < (uint32_t)kTileW) {
        fits = step();
        if (!fits) break;
      }
      if (!fits) break;
      const bool last = rhead == rtail;
      const uint32_t pc = ctail - chead, pl = ltail - lhead;
      if (pc >= tile || (last && pc != 0)) {
        const uint32_t n = min(tile, pc);
        it.flush_cells(chead, (int)n);
        chead += n;
      } else if (pl >= (uint32_t)kTileW || (last && pl != 0)) {
        const uint32_t n = min((uint32_t)kTileW, pl);
        it.flush_leaves(lhead, (int)n);
        lhead += n;
      } else {
        break;
      }
    }
  }
  *stamp = it.stamp;
  if (!fits) return kOverflow;

  if (LEARNED) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum2 += __shfl_xor(sum2, o);
    if (sqrt(sum2) > B.mac_budget) {
      *nband_out = nband;
      return kFallBack;
    }
    cw = 2 * nband;
  }
  if (lane == 0 && wk.y == 0)  // per-group counts; the totals are reduced afterwards
    reinterpret_cast<int4*>(B.cnt)[g] = make_int4((int)ctail, (int)ltail, (int)it.nsrc, cw);
  if (!do_eval) return kDone;

  float v[4], e[4];
  it.combine_slices(v, e);
  it.store(B, w, T.perm[first + lane % it.nt], v, e, acc, pot);
  wave_lds_sync();
  return kDone;
}

// One work item, with the theta re-walk of a group over its budget.
template <bool PLAIN, bool LEARNED, typename SH, typename Q>
__device__ int walk_eval_one(const DevTree& T, const WalkBufs& B, SH& sh, int64_t w, float th2,
                             float eps2, float* acc, float* pot, Q q, uint32_t qmask, bool gmem_q,
                             bool do_eval, int* stamp, const MlpView* mv) {
  int nb = 0;
  const int st = walk_eval_item<PLAIN, LEARNED>(T, B, sh, w, th2, eps2, acc, pot, q, qmask, gmem_q,
                                                do_eval, 0, &nb, stamp, mv);
  if (!LEARNED || st != kFallBack) return st;
  return walk_eval_item<PLAIN, false>(T, B, sh, w, th2, eps2, acc, pot, q, qmask, gmem_q, do_eval,
                                      2 * nb + 1, &nb, stamp, mv);
}

// Next work index from a shared counter, one atomic per wave.
__device__ __forceinline__ int take_work(int32_t* ctr, int lane) {
  int k = 0;
  if (lane == 0) k = atomicAdd(ctr, 1);
  return uni(__shfl(k, 0));
}

// Persistent blocks of NW independent waves (with the learned criterion
// they share one LDS copy of the network, loaded once per block).  Without
// FROM_LIST each XCD owns runs of consecutive (Morton-ordered) work items, handed
// out one at a time through a per-XCD counter (work items differ a lot in
// cost), and a wave whose XCD's items are exhausted helps the other XCDs;
// with FROM_LIST the items are the *src_n entries of src (the overflows of
// an earlier tier), handed out through one counter.  Items whose frontier
// outgrows this kernel's LDS queue are appended to (ovl, ovn).  Blocks of 16
// waves (the learned criterion: one network copy per CU) are held to 128
// VGPRs so that four waves per SIMD fit; the few registers this spills are
// outside the loops (the same lists took 13 % longer than in the opening-
// angle kernel at three waves per SIMD, 6 % at four).
template <bool PLAIN, int QCAP, bool LEARNED, int NW, bool FROM_LIST>
__global__ __launch_bounds__(NW * kLanes) __attribute__((amdgpu_waves_per_eu(NW == 16 ? 4 : 1)))
void walk_eval_persistent_kernel(
    DevTree T, WalkBufs B, float th2, float eps2, float* acc, float* pot, int do_eval,
    const int32_t* src, const int32_t* src_n, int32_t* ovl, int32_t* ovn) {
  __shared__ WShared<QCAP> shw[NW];
  __shared__ std::conditional_t<LEARNED, MlpLds, char> ml;
  if (FROM_LIST && *src_n == 0) return;
  MlpView V{};
  if constexpr (LEARNED) {
    mlp_load_lds(ml, B.mlp, threadIdx.x, blockDim.x);
    __syncthreads();
    V = mlp_lds(ml);
  }
  const int wv = uni((int)threadIdx.x / kLanes), lane = threadIdx.x & (kLanes - 1);
  // lds_qcap counts candidates; an entry holds up to eight
  const uint32_t qmask = (uint32_t)min(B.lds_qcap / 8, QCAP) - 1;
  const LQueue q{shw[wv].q};
  shw[wv].mark[lane] = 0;
  int stamp = 0;
  if constexpr (FROM_LIST) {
    for (;;) {
      const int k = take_work(B.wctr + 64 * 8, lane);
      if (k >= *src_n) break;
      const int32_t w = src[k];
      if (walk_eval_one<PLAIN, LEARNED>(T, B, shw[wv], w, th2, eps2, acc, pot, q, qmask, false,
                                        do_eval != 0, &stamp, &V) == kOverflow &&
          lane == 0)
        ovl[atomicAdd(ovn, 1)] = w;
    }
  } else {
    // Runs of kDeal consecutive items are dealt to the XCDs in turn: equal
    // shares of dense and sparse regions, and neighbours that share an L2.
    // (One contiguous range per XCD left its slowest XCD to the others' help: 260
    // against 249 us on a 200k galaxy at theta = 0.75; runs of 1 or 512 items cost
    // 1 % more at 2^20 and above.)  A wave's first item is its rank among its XCD's
    // waves (no atomic before any work), the next ones come from that XCD's
    // counter, then from the other XCDs' in turn.  A block notes the counters it
    // found used up, so that its other waves do not try them again.
    constexpr int kDeal = 64;
    __shared__ int used_up;
    if (threadIdx.x == 0) used_up = 0;
    __syncthreads();
    const int waves = (int)(gridDim.x >> 3) * NW;
    const int n = (int)((T.nw + 8 * kDeal - 1) / (8 * kDeal)) * kDeal;
    int first = (int)(blockIdx.x >> 3) + wv * (int)(gridDim.x >> 3);
    for (int s = 0; s < 8; ++s) {
      const int x = (blockIdx.x + s) & 7;
      for (;;) {
        int k = first;
        if (k < 0) {
          if (uni(*(volatile int*)&used_up) >> x & 1) break;
          k = take_work(B.wctr + 64 * x, lane) + waves;
        }
        first = -1;
        if (k >= n) {
          if (lane == 0) atomicOr(&used_up, 1 << x);
          break;
        }
        const int64_t w = ((int64_t)(k / kDeal) * 8 + x) * kDeal + k % kDeal;
        if (w >= T.nw) continue;
        if (walk_eval_one<PLAIN, LEARNED>(T, B, shw[wv], w, th2, eps2, acc, pot, q, qmask, false,
                                          do_eval != 0, &stamp, &V) == kOverflow &&
            lane == 0)
          ovl[atomicAdd(ovn, 1)] = (int32_t)w;
      }
    }
  }
}

// One block of NW waves per work item, for trees with too few items to fill
// the chip with a wave each: the item's latency is what counts.  The waves walk
// the tree together, NW windows of eight entries a step from one queue: a step
// takes about a microsecond (a dependent gather and two barriers) whatever
// its width, and a level of a small tree is one or two steps.  Every wave
// counts what its window appends and, after a barrier, writes it behind that of the
// waves before it, so the lists keep the order of the one-wave walk.  The tiles
// are its tiles too: of cells one per wave whenever all have one, and what there
// is at the end; of each 64 leaves in turns.  The first wave adds the partial
// sums in wave order, another order than the one-wave walk's, so the results agree
// with its to rounding: compensated ones nearly always bit for bit, plain ones
// not.  At 1000 bodies an item takes 13 us, of which 4.4 are seven steps
// and 4 its sources; with every wave walking alone and evaluating every NW-th
// tile, calls took 54 us for 5003 bodies (now 47), 75 for 16384 (67).
// (Remainders shared evenly by the waves were 1 to 2 us faster, but are other
// tiles, with other roundings.)
// Blocks go to the XCDs in turn, so consecutive items, which cost alike, do
// too (contiguous ranges per XCD: 10 % longer).
template <int QCAP, int NW>
struct TeamShared {
  int q[QCAP];
  int cring[128 * NW];  // before a step fewer than 64 NW are pending; it adds up to 64 NW
  int2 lring[128 * NW];
  float4 tile[NW][3 * kTileW];
  int mark[NW][kTileW];
  int count[NW];
};
// A wave's part of it, as WItem reads it.
template <int NW>
struct TeamView {
  static constexpr int kRing = 128 * NW;
  int* cring;
  int2* lring;
  float4* tile;
  int* mark;
};
template <bool PLAIN, int QCAP, int NW>
__global__ __launch_bounds__(NW * kLanes) void walk_eval_team_kernel(DevTree T, WalkBufs B, float th2,
                                                                     float eps2,
                                                                     float* __restrict__ acc,
                                                                     float* __restrict__ pot) {
  static_assert(NW <= 8, "counts of a step in ten bits each");
  __shared__ TeamShared<QCAP, NW> sh;
  const int64_t w = blockIdx.x;
  const int lane = threadIdx.x & (kLanes - 1), wave = uni((int)threadIdx.x / kLanes);
  const uint32_t qmask = (uint32_t)min(B.lds_qcap / 8, QCAP) - 1;
  const int2 wk = reinterpret_cast<const int2*>(T.wwork)[w];
  const int64_t g = wk.x;
  const int4 gi = reinterpret_cast<const int4*>(T.ginfo)[g];
  const float4* gbox = reinterpret_cast<const float4*>(T.gbox);
  const float4 gmin = gbox[2 * g], gmax = gbox[2 * g + 1];
  const float4* rec = reinterpret_cast<const float4*>(T.wrec);
  TeamView<NW> view{sh.cring, sh.lring, sh.tile[wave], sh.mark[wave]};
  view.mark[lane] = 0;
  WItem<PLAIN, NW, TeamView<NW>> it{T, view, in_vgpr(eps2)};
  it.turn = wave;
  const int first = gi.x + wk.y;
  it.targets(lane, uni(min(kChunk, gi.y - wk.y)), first, true, 0);
  const int64_t place = T.perm[first + lane % it.nt];

  uint32_t rhead = 0, rtail = 0, chead = 0, ctail = 0, lhead = 0, ltail = 0;
  const int4 root = reinterpret_cast<const int4*>(rec)[1];
  if (root.y == 0) {  // the root is a leaf: its particles are the whole list
    if (threadIdx.x == 0) sh.lring[0] = make_int2(root.z, root.w);
    ltail = 1;
  } else {
    if (threadIdx.x == 0) sh.q[0] = (root.x << 3) | (root.y - 1);
    rtail = 1;
  }
  __syncthreads();
  const uint32_t ent = 8 * wave + (lane >> 3);
  const int child = lane & 7;
  const uint32_t tile = (uint32_t)it.tile_size();
  const float th2v = in_vgpr(th2);
  for (;;) {
    // (every condition is the same in all waves)
    while (rhead != rtail && ctail - chead < NW * tile && ltail - lhead < (uint32_t)(NW * kTileW)) {
      const uint32_t avail = rtail - rhead;
      uint64_t mC = 0, mL = 0, mQ = 0;
      int c = 0;
      int4 tp = make_int4(0, 0, 0, 0);
      if (8u * wave < avail) {
        const int e = sh.q[(rhead + ent) & qmask];
        c = ent < avail && child <= (e & 7) ? (int)((uint32_t)e >> 3) + child : 0;
        tp = reinterpret_cast<const int4*>(rec)[2 * (int64_t)c + 1];
        const float4 ge = rec[2 * (int64_t)c];
        const uint64_t mV = __ballot(c != 0);
        const uint64_t mOp = mV & open_mask(gmin, gmax, ge, th2v), mLeaf = __ballot(tp.y == 0);
        mC = mV & ~mOp;
        mL = mOp & mLeaf;
        mQ = mOp & ~mLeaf;
      }
      rhead += min(8u * NW, avail);
      if (lane == 0) sh.count[wave] = __popcll(mC) | __popcll(mL) << 10 | __popcll(mQ) << 20;
      __syncthreads();
      const int incl = wave_inclusive_sum(lane < NW ? sh.count[lane] : 0);
      const uint32_t all = (uint32_t)__builtin_amdgcn_readlane(incl, NW - 1);
      const uint32_t own = wave == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane(incl, max(wave - 1, 0));
      if ((rtail + (all >> 20)) - rhead > qmask + 1) {
        if (threadIdx.x == 0) B.ovf_list[atomicAdd(B.ovf_count, 1)] = (int32_t)w;
        return;
      }
      if (__builtin_amdgcn_inverse_ballot_w64(mC))
        sh.cring[(ctail + (own & 1023) + rank_below(mC)) & (128 * NW - 1)] = c;
      if (__builtin_amdgcn_inverse_ballot_w64(mL))
        sh.lring[(ltail + (own >> 10 & 1023) + rank_below(mL)) & (128 * NW - 1)] = make_int2(tp.z, tp.w);
      if (__builtin_amdgcn_inverse_ballot_w64(mQ))
        sh.q[(rtail + (own >> 20) + rank_below(mQ)) & qmask] = (tp.x << 3) | (tp.y - 1);
      ctail += all & 1023;
      ltail += all >> 10 & 1023;
      rtail += all >> 20;
      __syncthreads();
    }
    const bool last = rhead == rtail;
    const uint32_t pc = ctail - chead, pl = ltail - lhead;
    if (pc >= NW * tile || (last && pc != 0)) {
      const uint32_t from = min(pc, tile * wave);
      const uint32_t n = min(tile, pc - from);
      if (n != 0) it.flush_cells(chead + from, (int)n);
      // the leaves' turns go on after the last tile (a full round leaves them)
      const int used = uni((int)((min(pc, tile * NW) + tile - 1) / tile));
      it.turn = it.turn >= used ? it.turn - used : it.turn - used + NW;
      chead += min(pc, tile * NW);
    } else if (pl >= (uint32_t)(NW * kTileW) || (last && pl != 0)) {
      const uint32_t n = min((uint32_t)kTileW, pl);
      it.flush_leaves(lhead, (int)n);
      lhead += n;
    } else {
      break;
    }
  }

  // The waves' sums, in their tiles: [32][8] floats.
  float v[4], e[4];
  it.combine_slices(v, e);
  auto sums = [&](int k) { return reinterpret_cast<float*>(sh.tile[k]) + lane * 8; };
  float* own = sums(wave);
  if (lane < it.nt && wave != 0)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      own[k] = v[k];
      own[4 + k] = e[k];
    }
  __syncthreads();
  if (wave != 0) return;
  if (lane < it.nt)
    for (int k = 1; k < NW; ++k)
      it.add(v, e, sums(k), sums(k) + 4);
  if (lane == 0 && wk.y == 0)
    reinterpret_cast<int4*>(B.cnt)[g] = make_int4((int)ctail, (int)ltail, (int)it.nsrc, 0);
  it.store(B, w, place, v, e, acc, pot);
}

// Global-memory queues: written and read by different lanes of one wave, so
// they are accessed as volatile (no stale L1 copies) and fenced.
struct GQueue {
  volatile int32_t* p;
  __device__ int get(uint32_t i) const { return p[i]; }
  __device__ void put(uint32_t i, int x) const { p[i] = x; }
};

// Last tier: the *src_n items of src with global-memory frontier queues of
// 2 x (widest tree level) entries, which a breadth-first FIFO cannot exceed
// (its candidates span at most two consecutive levels, and every queued
// entry holds at least one of them).
template <bool PLAIN, bool LEARNED>
__global__ __launch_bounds__(kLanes) void walk_eval_fallback_kernel(DevTree T, WalkBufs B,
                                                                    float th2, float eps2,
                                                                    float* acc, float* pot,
                                                                    int do_eval,
                                                                    const int32_t* src,
                                                                    const int32_t* src_n) {
  __shared__ WShared<64> sh;
  __shared__ std::conditional_t<LEARNED, MlpLds, char> ml;
  const int n = *src_n;
  if (n == 0) return;
  MlpView V{};
  if constexpr (LEARNED) {
    mlp_load_lds(ml, B.mlp, threadIdx.x, blockDim.x);
    __syncthreads();
    V = mlp_lds(ml);
  }
  GQueue q{B.gq + (int64_t)blockIdx.x * B.gq_cap};
  sh.mark[threadIdx.x] = 0;
  int stamp = 0;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const int st = walk_eval_one<PLAIN, LEARNED>(T, B, sh, src[i], th2, eps2, acc, pot, q,
                                                 (uint32_t)(B.gq_cap - 1), true, do_eval != 0, &stamp, &V);
    if (st == kOverflow && threadIdx.x == 0)
      atomicOr(reinterpret_cast<unsigned long long*>(&B.tot[5]), 1ull);
  }
}

// The counters a call starts from, by threads [0, 64) of one block.  (Not the
// last tier's overflow, B.tot[5], which the host may read after them.)
__device__ __forceinline__ void reset_counters(const WalkBufs& B, int t) {
  if (t < 9) B.wctr[64 * t] = 0;
  if (t == 0) {
    *B.ovf_count = 0;
    *B.ovf_count2 = 0;
    *B.ticket = 0;
    B.c_off[0] = 0;  // base of an offsets scan of the counts the walk writes
    B.l_off[0] = 0;
  }
}

__global__ void fused_init_kernel(WalkBufs B) {
  if (threadIdx.x < 8) B.tot[threadIdx.x] = 0;
  reset_counters(B, threadIdx.x);
}

// End of a call in one launch: totals and diagnostics summed per block over a
// contiguous range of work items, then by the last block to finish over the
// blocks in order (both fixed orders), written to the device, to the host's
// page-locked copy, and the counters reset for the next call.  Replaces an
// initial reset, a totals kernel, two diagnostics kernels over the particles
// (21 + 5 us at 2^20, bound by the gather of the masses) and a copy.
constexpr int kFinT = 1024, kFinBlocks = 256;
struct FinRec {
  double d[4];
  int64_t t[4];
};

// Sum over the wave of four values per lane; lane l < 4 gets that of value
// ((l & 1) << 1) | (l >> 1).
template <typename V>
__device__ __forceinline__ V wave_sum4(const V* d, int lane) {
  const bool b0 = lane & 1, b1 = lane & 2;
  V k0 = b0 ? d[2] : d[0], k1 = b0 ? d[3] : d[1];
  k0 += __shfl_xor(b0 ? d[0] : d[2], 1);
  k1 += __shfl_xor(b0 ? d[1] : d[3], 1);
  V v = b1 ? k1 : k0;
  v += __shfl_xor(b1 ? k0 : k1, 2);
#pragma unroll
  for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o);
  return v;
}

struct FinShared {
  double d[4][kFinT / 64];
  int64_t t[4][kFinT / 64];
};

// Sum over the block, in thread t < 4 for components t of both.
__device__ __forceinline__ void block_sum_rec(FinRec& r, double* d, int64_t* n, FinShared& sh) {
  const int t = threadIdx.x, lane = t & 63;
  const double sd = wave_sum4(r.d, lane);
  const int64_t st = wave_sum4((const long long*)r.t, lane);
  if (lane < 4) {
    const int k = ((lane & 1) << 1) | (lane >> 1);
    sh.d[k][t >> 6] = sd;
    sh.t[k][t >> 6] = st;
  }
  __syncthreads();
  if (t < 4) {
    *d = 0.0;
    *n = 0;
    for (int w = 0; w < kFinT / 64; ++w) {
      *d += sh.d[t][w];
      *n += sh.t[t][w];
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(kFinT) void finish_kernel(DevTree T, WalkBufs B, FinRec* rec,
                                                       double* diag, int64_t* host, int last) {
  __shared__ FinShared sh;
  __shared__ int is_last;
  const int t = threadIdx.x, nb = gridDim.x;
  const int64_t per = (T.nw + nb - 1) / nb;
  const int64_t lo = blockIdx.x * per, hi = lo + per < T.nw ? lo + per : T.nw;
  FinRec r{};
  for (int64_t i0 = lo + t; i0 < hi; i0 += 4 * kFinT) {  // four items' loads at a time
    int2 wk[4];
    double2 a[4], b[4];
    int4 c[4];
    int sz[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = i0 + q * kFinT < hi ? i0 + q * kFinT : hi - 1;
      wk[q] = reinterpret_cast<const int2*>(T.wwork)[i];
      const double2* dp = reinterpret_cast<const double2*>(B.dpart + 4 * i);
      a[q] = dp[0];
      b[q] = dp[1];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c[q] = reinterpret_cast<const int4*>(B.cnt)[wk[q].x];
      sz[q] = T.ginfo[4 * (int64_t)wk[q].x + 1];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i0 + q * kFinT >= hi) break;
      r.d[0] += a[q].x;
      r.d[1] += a[q].y;
      r.d[2] += b[q].x;
      r.d[3] += b[q].y;
      if (wk[q].y == 0) {
        r.t[0] += c[q].x;
        r.t[1] += c[q].y;
        r.t[2] += (int64_t)sz[q] * c[q].x;
        r.t[3] += (int64_t)sz[q] * c[q].z;
      }
    }
  }
  double sd;
  int64_t st;
  block_sum_rec(r, &sd, &st, sh);
  if (nb > 1) {
    if (t < 4) {
      __hip_atomic_store(&rec[blockIdx.x].d[t], sd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&rec[blockIdx.x].t[t], st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The record is written and read by agent-scope atomics, which do not rest
    // in this XCD's L2; thread 0's wave wrote it and waits for that, so the ticket
    // needs no release (which would write the whole L2 back: 5 us).
    if (t == 0) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      is_last = __hip_atomic_fetch_add(B.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1;
    }
    __syncthreads();
    if (!is_last) return;
    r = FinRec{};
    if (t < nb)  // nb <= kFinT
      for (int k = 0; k < 4; ++k) {
        r.d[k] = __hip_atomic_load(&rec[t].d[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r.t[k] = __hip_atomic_load(&rec[t].t[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    block_sum_rec(r, &sd, &st, sh);
  }
  const int left = *B.ovf_count;
  if (t < 4) {
    diag[t] = sd;
    B.tot[t] = st;
  }
  if (host) {
    if (t < 4) host[t] = st;
    else if (t < 8) host[t] = B.tot[t];
    else if (t == 8) host[t] = left;
  }
  if (t == 0) *B.ticket = 0;  // also when the later tiers and a second finish follow
  __syncthreads();
  if (last || left == 0) reset_counters(B, t);
}

}  // namespace

int launch_walk_eval(const DevTree& T, const WalkBufs& B, float theta, float eps, bool plain,
                     bool do_eval, float* acc, float* pot, void* stream, int parts) {
  hipStream_t s = (hipStream_t)stream;
  const float th2 = theta * theta, eps2 = eps * eps;
  if (parts & kWalkInit) fused_init_kernel<<<1, 64, 0, s>>>(B);
  // The breadth-first FIFO holds about two tree levels of the group's walk,
  // which grow like theta^-3, as entries of up to eight children: 512 entries
  // (2 KB) held every walk of the 2^20 Plummer sphere and the 4M clumps at
  // theta 0.3 ... 0.5.  Tiers: 512-entry LDS queues (20 waves per CU), then
  // the overflows with 2048-entry LDS queues (one wave per block, 10 per CU, all
  // that its LDS holds: with 7, calls of 16384 single particles as groups took
  // 2330 us at theta 0.1, now 1847, and of 2^20 particles 38.0 ms at theta 0.2,
  // now 30.0), then global-memory queues.
  const bool learned = B.mlp != nullptr;
  // Waves per work item.  With fewer than about 11000 items (two for each of the
  // 5120 waves the chip holds) one wave per item leaves a long tail, or most of
  // the chip idle; measured with 1 / 2 / 4 / 8 waves per item, in us: 79 items (1000
  // bodies) 100 / 44 / 39 / 37, 368 items 154 / 74 / 54 / 47, 655 items 173 / 88 / 61 / 55,
  // 1042 items 186 / 98 / 68 / 71, 1198 items 216 / 121 / 80 / 81, 2590 items 201 / 123 / 111 /
  // 131 and 125 / 76 / 77 / 101, 5008 items 248 / 201 / 189 / 235 and 137 / 112 / 119 / 172, 7580
  // items 165 / 149 / 164 / 250, 12641 items 219 / 233 / 259 / 402.  (Not
  // with the learned criterion: every wave would run the network.)
  // Below theta 0.3, where the frontiers outgrow 512 entries, a team of two has a
  // queue of 1024: calls of 5003 and 10000 single particles as groups took 387 and
  // 1149 us at theta 0.1 without, with the second tier redoing a quarter and
  // more of their items, and 241 and 629 with it.  From 0.3 up the two blocks per CU
  // less that its LDS then holds cost 1 to 2 % (5003 74.1 / 75.3 us at theta 0.5,
  // 9644 items 168 / 171 at 0.75).
  int team = 1;
  if (!learned && do_eval && !B.export_lists)
    team = T.nw <= 1000 ? 8 : T.nw <= 3500 ? 4 : T.nw <= 11000 ? 2 : 1;
  auto go = [&](auto plain_tag, auto learned_tag) {
    constexpr bool P = decltype(plain_tag)::value, L = decltype(learned_tag)::value;
    if (parts & kWalkFirst) {
      if constexpr (L)  // one block of 16 waves per CU (16 x 6.9 KB frontiers + 12 KB network,
                        // 122.5 KB of LDS), four per SIMD at <= 128 VGPRs
        walk_eval_persistent_kernel<P, 512, L, 16, false><<<8 * 32, 16 * kLanes, 0, s>>>(
            T, B, th2, eps2, acc, pot, do_eval, nullptr, nullptr, B.ovf_list, B.ovf_count);
      else if (team == 8)
        walk_eval_team_kernel<P, 512, 8><<<(unsigned)T.nw, 8 * kLanes, 0, s>>>(T, B, th2, eps2, acc, pot);
      else if (team == 4)
        walk_eval_team_kernel<P, 512, 4><<<(unsigned)T.nw, 4 * kLanes, 0, s>>>(T, B, th2, eps2, acc, pot);
      else if (team == 2 && theta < 0.3f)
        walk_eval_team_kernel<P, 1024, 2><<<(unsigned)T.nw, 2 * kLanes, 0, s>>>(T, B, th2, eps2, acc, pot);
      else if (team == 2)
        walk_eval_team_kernel<P, 512, 2><<<(unsigned)T.nw, 2 * kLanes, 0, s>>>(T, B, th2, eps2, acc, pot);
      else  // 5 blocks of 4 waves per CU (four: 2.36 against 2.32 ms at 2^20)
        walk_eval_persistent_kernel<P, 512, L, 4, false><<<8 * 160, 4 * kLanes, 0, s>>>(
            T, B, th2, eps2, acc, pot, do_eval, nullptr, nullptr, B.ovf_list, B.ovf_count);
    }
    if (parts & kWalkRest) {
      walk_eval_persistent_kernel<P, 2048, L, 1, true><<<8 * 320, kLanes, 0, s>>>(
          T, B, th2, eps2, acc, pot, do_eval, B.ovf_list, B.ovf_count, B.ovf_list2, B.ovf_count2);
      walk_eval_fallback_kernel<P, L><<<B.gq_waves, kLanes, 0, s>>>(
          T, B, th2, eps2, acc, pot, do_eval, B.ovf_list2, B.ovf_count2);
    }
  };
  if (learned) {
    if (plain) go(std::true_type{}, std::true_type{});
    else go(std::false_type{}, std::true_type{});
  } else {
    if (plain) go(std::true_type{}, std::false_type{});
    else go(std::false_type{}, std::false_type{});
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_finish(const DevTree& T, const WalkBufs& B, double* scratch, double* diag, int64_t* host,
                  bool last, void* stream) {
  // One block up to four items per thread (4.2 us at 79 items, 4.9 at 1042, 23 at
  // 16300); more blocks need the second level, a ticket and the records' way
  // through memory (about 6 us).
  static_assert(kFinBlocks <= kFinT, "the last block reads one record per thread");
  const int nb = T.nw <= 4 * kFinT ? 1 : (int)std::min<int64_t>(kFinBlocks, (T.nw + kFinT - 1) / kFinT);
  finish_kernel<<<nb, kFinT, 0, (hipStream_t)stream>>>(T, B, reinterpret_cast<FinRec*>(scratch), diag,
                                                       host, last);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace octgrav
