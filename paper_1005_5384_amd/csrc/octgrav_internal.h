// Internal declarations shared by the library's host and device sources.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "walk_types.h"

namespace octgrav {

constexpr int kMaxDepth = 21;   // levels below the root cube (63-bit Morton keys)

// Host tree (Sec. 2.1), FP64 geometry and moments, FP32 device images.
struct HostTree {
  int64_t n = 0;
  int n_leaf = 0, n_group = 0;
  double corner[3] = {0, 0, 0}, side = 1;   // root cube
  int max_depth = 0;
  int64_t max_level_cells = 0;
  int64_t n_leaves = -1;         // counted by the device build (-1: count from topo)
  std::vector<int32_t> perm;     // [n] sorted position -> input index
  std::vector<float> part;       // [n*4] sorted x, y, z, m
  std::vector<int32_t> topo;     // [nc*4] first_child, n_child, first, n
  std::vector<int32_t> depth;    // [nc]
  std::vector<double> box;       // [nc*6] tight box
  std::vector<double> mp64;      // [nc*10] M, com, Q (xx yy zz xy xz yz)
  std::vector<float> geo;        // [nc*4] f32 boundary centre, side
  std::vector<float> mp;         // [nc*12] f32 com, M | Qxx Qyy Qzz Qxy | Qxz Qyz 0 0
  std::vector<int32_t> groups;   // [ng] cell id
  std::vector<int32_t> ginfo;    // [ng*4] first, n, cell, 0
  std::vector<float> gbox;       // [ng*8] gmin xyz 0, gmax xyz 0
  std::vector<int32_t> work;     // [nw*2] group, first target offset within group
  // Counts of a device build whose depth / groups / work arrays stay on the
  // device until an export fetches them (-1: the vectors' sizes).
  int64_t nc_dev = -1, ng_dev = -1, nw_dev = -1;
  int64_t n_cells() const { return nc_dev >= 0 ? nc_dev : (int64_t)depth.size(); }
  int64_t n_groups() const { return ng_dev >= 0 ? ng_dev : (int64_t)groups.size(); }
  int64_t n_work() const { return nw_dev >= 0 ? nw_dev : (int64_t)work.size() / 2; }
};

// Builds the host tree; returns false with a message on bad input.
bool build_host_tree(const float* pos, const float* mass, int64_t n, int n_leaf, int n_group,
                     HostTree& out, std::string& err);
// Pieces shared by the host and device builds.
bool validate_inputs(const float* pos, const float* mass, int64_t n, int n_leaf, int n_group,
                     std::string& err);
void root_cube(const double lo[3], const double hi[3], double corner[3], double* side);

// Kernel launchers (device sources).  mode 0 = count, 1 = write at the
// offsets, 2 = count and write into per-group slots.  Ranges
// are [g0, g0 + ng) groups / [w0, w0 + nw) work items (ng, nw < 0: to the end).
int launch_walk(const DevTree& T, const WalkBufs& B, float theta, int mode, void* stream,
                int64_t g0 = 0, int64_t ng = -1, bool init = true);
int launch_scan(const DevTree& T, const WalkBufs& B, void* stream, int64_t g0 = 0, int64_t ng = -1);
// Interaction totals and longest lists from the per-group counts.
int launch_totals(const DevTree& T, const WalkBufs& B, void* stream, int64_t g0 = 0, int64_t ng = -1);
int launch_eval(const DevTree& T, const WalkBufs& B, float eps, bool plain, float* acc,
                float* pot, void* stream, int64_t w0 = 0, int64_t nw = -1);
// Fused wave walk + evaluation.  parts: kWalkInit resets the counters, kWalkFirst
// is the first tier (every work item), kWalkRest the later tiers (the items whose
// frontier outgrew it).
constexpr int kWalkInit = 1, kWalkFirst = 2, kWalkRest = 4, kWalkAll = 7;
int launch_walk_eval(const DevTree& T, const WalkBufs& B, float theta, float eps, bool plain,
                     bool do_eval, float* acc, float* pot, void* stream, int parts = kWalkAll);
// After a fused wave evaluation: interaction totals (B.tot) and the FP64
// diagnostics (diag[4]) from the per-item and per-group records, copied to
// host (device pointer of page-locked memory, kFinishHost entries: the totals,
// then the number of items the first tier left over; or NULL).  Unless items
// were left over and !last, it also resets the counters as kWalkInit does, but
// for B.tot[5]: a call that reports it is followed by kWalkInit.
constexpr int kFinishHost = 9;
int launch_finish(const DevTree& T, const WalkBufs& B, double* scratch, double* diag, int64_t* host,
                  bool last, void* stream);
int launch_walk_eval_block(const DevTree& T, const WalkBufs& B, float theta, float eps, bool plain,
                           bool do_eval, float* acc, float* pot, void* stream);
// Walk records (nc x 32 B, the layout of DevTree::wrec) of the centre-of-mass
// offset opening test at theta: boundary (com, l + theta |com - cb|), topology.
int launch_com_records(const DevTree& T, float theta, float* out, void* stream);
// FP32 compensated direct sum for targets (caller indices, device array, or
// NULL = all); outputs in target order.  scratch: direct_scratch_bytes of
// device memory for the partial sums of several particle ranges per target,
// or NULL (one range).
int launch_direct(const DevTree& T, const int32_t* targets, int64_t nt, float eps, float* acc,
                  float* pot, void* scratch, void* stream);
int64_t direct_scratch_bytes(int64_t n, int64_t nt);
// Features (12, FP32) and labels of the band pairs of the listed groups
// (pair p of listed group s sits at out_off[s] + k); also each pair's ids.
int launch_mac_labels(const DevTree& T, const WalkBufs& B, const int32_t* groups, int64_t ngs,
                      const int64_t* out_off, const float* acc_direct, float eps, float* feat,
                      float* label, int32_t* gout, int32_t* cout, int64_t npairs, void* stream);
// Network of the learned criterion: pack FP32 parameters into the BF16
// inference image; batch forward; loss + gradient of a batch (hgrad / hloss:
// device addresses of page-locked host copies, or NULL); Adam step, which also
// updates the image.
int launch_mlp_pack(const float* P, void* pk, void* stream);
int launch_mlp_forward(const void* pk, const float* x, int64_t B, float* y, void* stream);
int launch_mlp_loss_grad(const void* pk, const float* x, const float* tgt, int64_t B, float tau,
                         float* scratch, float* grad, double* loss, float* hgrad, double* hloss,
                         void* stream);
int64_t mlp_train_scratch_floats(int64_t B);  // scratch of launch_mlp_loss_grad
int launch_mlp_adam(float* P, float* m, float* v, const float* g, void* pk, float lr, float b1,
                    float b2, float eps, float c1, float c2, void* stream);
// Device tree build (same result as build_host_tree, computed on the GPU).
// The persistent arrays are allocated through DevAlloc (owned by the
// caller); DeviceArrays receives the FP64 boxes / moments, the unsigned
// boundary image, the depths and the group cells, which stay on the device.
// Fills h with the scalars and the counts (nc_dev, ng_dev, nw_dev); every
// array stays on the device.  A build with pools makes two host round trips
// (the level counts, then the group and work counts).
struct DevAlloc {
  virtual int alloc(void** p, size_t bytes) = 0;
  // The next allocations add up to about this much.
  virtual void expect(size_t) {}
  virtual ~DevAlloc() = default;
};
// hipMalloc, with the tests' limit on its size (capi.cpp); a hipError_t.
int device_malloc(void** p, size_t bytes);
// Device buffers cut from a few large allocations that are freed together: a
// tree set up with one hipMalloc and hipFree per array spent 3 of 4 ms on
// about 75 of them (250k points; a hipFree takes 15 to 400 us).
struct Arena {
  std::vector<void*> chunks;
  char* at = nullptr;
  size_t left = 0, next = 0;
  // The next chunk is at least this large.
  void expect(size_t bytes) { next = bytes; }
  void* take(size_t bytes);  // nullptr when the device allocation fails
  Arena() = default;
  Arena(const Arena&) = delete;
  Arena& operator=(const Arena&) = delete;
  ~Arena();
};
// Device buffers handed out in request order and kept for the next round of
// requests in the same order: a repeated build (time integration) finds its
// buffers in place and only a request that outgrows its slot reallocates it.
struct SeqPool {
  std::vector<void*> ptr;
  std::vector<size_t> cap;
  size_t next = 0;
  void* take(size_t bytes);  // nullptr when the device allocation fails
  void rewind() { next = 0; }
  SeqPool() = default;
  SeqPool(const SeqPool&) = delete;
  SeqPool& operator=(const SeqPool&) = delete;
  ~SeqPool();
};
// Scratch of the device build kept between builds: whole-build arrays and
// the cell arrays.
struct BuildPools {
  SeqPool outer, cells;
  void* pinned = nullptr;  // page-locked host copy of the build's scalars (tree_gpu.hip)
  BuildPools() = default;
  BuildPools(const BuildPools&) = delete;
  BuildPools& operator=(const BuildPools&) = delete;
  ~BuildPools();
};
struct DeviceArrays {
  const double* box = nullptr;     // [nc * 6]
  const double* mp64 = nullptr;    // [nc * 10]
  const float* geo_host = nullptr; // [nc * 4]
  const int32_t* depth = nullptr;  // [nc]
  const int32_t* groups = nullptr; // [ng]
};
// Most cells of a tree (kMaxCells), and what is said of one with more.
int64_t max_cells();
std::string too_many_cells(int64_t nc);
// Inputs are host arrays (copied) or, with inputs_on_device, device arrays
// (checked on the device).  0, kBuildRefused (err: what is wrong with the input,
// or the tree's size) or another error.
constexpr int kBuildRefused = -2;
int build_device_tree(const float* pos_in, const float* mass_in, bool inputs_on_device, int64_t n,
                      int n_leaf, int n_group, HostTree& h, DevTree& dt, DeviceArrays& out,
                      DevAlloc& alloc, void* stream, std::string& err,
                      BuildPools* pools = nullptr);

// Leapfrog pieces: v += h a, x += dt v, and FP64 (1/2 sum m v^2, sum m v).
int launch_kick(float* vel, const float* acc, int64_t n, float h, void* stream);
// v += h a (twice with both), x += dt v
int launch_kick_drift(float* pos, float* vel, const float* acc, int64_t n, float h, float dt,
                      bool both, void* stream);
int launch_kinetic(const float* mass, const float* vel, int64_t n, double* part, double* out4,
                   void* stream);
int64_t kinetic_scratch_entries();

int launch_diag(const DevTree& T, const float* acc, const float* pot, double* part_sums,
                double* out4, void* stream);
int64_t scan_scratch_entries(int64_t ng);
int64_t diag_scratch_entries(int64_t n);  // also of launch_finish

// The file-scope device scratch array of octgrav_forces_noalloc: its size,
// and its device address on the current device (looked up on the first call
// per device, then cached).  0 on success.
size_t noalloc_scratch_bytes();
int noalloc_scratch(void** ptr, std::string& err);

}  // namespace octgrav
