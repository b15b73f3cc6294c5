// What the walk and evaluation kernels are compiled from besides their own
// sources: work items, the packed network, a tree and the walk's buffers on
// the device.  (Apart from octgrav_internal.h, so that a change elsewhere leaves
// the counter records of these kernels valid.)
#pragma once

#include <cstdint>

namespace octgrav {

constexpr int kChunk = 32;      // targets per evaluation work item
// Work items by targets, the classes that are handed out one after the other
// (0 first): more than 24, more than 16, more than 8, the rest.
constexpr int kItemClasses = 4;
constexpr int kItemBound[3] = {24, 16, 8};
constexpr int item_class(int targets) {
  return targets > kItemBound[0] ? 0 : targets > kItemBound[1] ? 1 : targets > kItemBound[2] ? 2 : 3;
}

// ------------------------------------------------------------------ network
// Learned acceptance criterion: 12 -> 64 -> 64 -> 1 with ReLU.
constexpr int kMlpIn = 12, kMlpInPad = 16, kMlpH = 64;
constexpr int kMlpParams = kMlpH * kMlpIn + kMlpH + kMlpH * kMlpH + kMlpH + kMlpH + 1;  // 5057
// FP32 parameter vector offsets: W1 [64 x 12] row-major, b1, W2 [64 x 64], b2, w3, b3.
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kMlpH * kMlpIn, kOffW2 = kOffB1 + kMlpH,
              kOffB2 = kOffW2 + kMlpH * kMlpH, kOffW3 = kOffB2 + kMlpH, kOffB3 = kOffW3 + kMlpH;

// Packed inference image (one device buffer), byte offsets.
constexpr int kPkW1 = 0;                              // BF16 [64][16]
constexpr int kPkW2 = kPkW1 + kMlpH * kMlpInPad * 2;  // BF16 [64][64]
constexpr int kPkB1 = kPkW2 + kMlpH * kMlpH * 2;      // FP32 [64]
constexpr int kPkB2 = kPkB1 + kMlpH * 4;              // FP32 [64]
constexpr int kPkW3 = kPkB2 + kMlpH * 4;              // BF16 [64]
constexpr int kPkB3 = kPkW3 + kMlpH * 2;              // FP32
constexpr int kPkBytes = kPkB3 + 256;

// ------------------------------------------------------------------ device
struct DevTree {
  const float* part;     // float4 [n]
  const int32_t* perm;   // [n]
  const int32_t* topo;   // int4 [nc]
  const float* geo;      // float4 [nc]  boundary; the side's sign bit marks leaves
  const float* wrec;     // float4 x2 [nc] walk record: boundary (as geo) | topo
  const float* fcell;    // float4 x2 [nc] learned-criterion features of the cell alone:
                         // f1, f2, f4, f5 | f6, f10, f11, 0 (see mac_features)
  const int32_t* iperm;  // [n] caller index -> sorted position
  const float* mp;       // float4 x3 [nc]
  const int32_t* ginfo;  // int4 [ng]
  const float* gbox;     // float4 x2 [ng]
  const int32_t* work;   // int2 [nw] {group, first target in it}, in group order
  // The same items as the fused wave kernels take them: class by class
  // (item_class), each in group order.  An item's time grows with its targets (64 /
  // slices terms per tile), and the last items to start should be short ones.
  const int32_t* wwork;
  int64_t n, nc, ng, nw;
};

struct WalkBufs {
  int32_t* cnt;        // int4 [ng]: |C|, |L|, n_src(L), frontier-overflow flag
  int64_t* c_off;      // [ng+1]
  int64_t* l_off;      // [ng+1]
  int32_t* c_ids;      // [cap_c]
  int32_t* l_ids;      // [cap_l]
  int64_t cap_c, cap_l;
  int64_t* tot;        // [8]: n_c, n_l, N_pc, N_pp, capacity-overflow, fallback-overflow
  int64_t* blk;        // scan scratch: 2 per scan block
  int32_t* ovf_list;   // [max(ng, nw)] groups / work items whose LDS frontier overflowed
  int32_t* ovf_count;  // [1]
  int32_t* ovf_list2;  // [max(ng, nw)] second-tier overflows (fused wave kernels)
  int32_t* ovf_count2; // [1]
  int32_t* wctr;       // [9 x 64]: work counters (stride 64) of persistent kernels:
                       // 8 per-XCD ranges, 1 overflow list
  int32_t* ticket;     // [1]: blocks of finish_kernel that are done
  double* dpart;       // [4 nw]: FP64 sums (m a, 1/2 m phi) of each work item's targets,
                       // written by the fused wave kernels (NULL: not written)
  int32_t* gq;         // global frontier queues for the fallback walk: gq_cap words each
  int64_t gq_cap;      // entries per queue (power of two)
  int32_t gq_waves;    // queues (waves) of the fallback walk
  int32_t lds_qcap;    // cap on the LDS frontier in candidates (power of two >= 64; test
                       // hook); the fused wave walk's entries of up to eight children use
                       // lds_qcap / 8 of them
  int32_t export_lists;  // fused walk: also write the lists at c_off / l_off
  // Slotted lists (walk mode 2, > 0): group g's lists start at g * slot_c /
  // g * slot_l and their lengths are cnt[g].x / .y; 0 = CSR offsets.
  int64_t slot_c, slot_l;
  // Band collection (band != 0): the "cell list" records the candidates the
  // walk's test opens and the test at band_hi2 (squared angle) does not.
  int32_t band;
  float band_hi2;
  // Learned acceptance criterion (fused wave walk; mlp == NULL: the theta
  // test).  Candidates the test at mac_lo2 accepts are accepted, those the
  // test at mac_hi2 opens are opened, the network decides the rest (accept
  // iff its output <= mac_ltau); a group whose accepted band candidates give
  // sqrt(sum 10^(2 y)) > mac_budget is walked again with the call's theta.
  // cnt[g].w = 2 * (band candidates visited) + (1 if the group fell back).
  const uint8_t* mlp;  // packed network image (mlp_device.h)
  float mac_lo2, mac_hi2, mac_ltau;
  double mac_budget;
  // Decision trace of the learned walks (test export; tr_s == NULL: off):
  // group g's band candidates at [tr_off[g], tr_off[g + 1]).
  const int64_t* tr_off;
  int32_t* tr_c;
  float* tr_s;
};

}  // namespace octgrav
