// Internal declarations of the runtime shared by runtime.cpp (single-handle
// entry points) and batch.cpp (lock-step batches of handles): device plans,
// the handle itself and the helpers that enqueue its work.
#pragma once
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "attn.h"
#include "kernels.hpp"
#include "launch.hpp"
#include "model.hpp"

namespace rt {
using namespace attn;


struct HipFail {
  hipError_t e;
  const char* what;
};

#define HIPCHK(x)                                 \
  do {                                            \
    hipError_t _e = (x);                          \
    if (_e != hipSuccess) throw HipFail{_e, #x};  \
  } while (0)

struct StatusFail {
  attn_status st;
  std::string msg;
};

// Device memory handed out in order and taken back by marks, kept from one
// call to the next (an allocation of the size a call needs costs up to
// hundreds of milliseconds: 8 x 8 m = 32 correlation matrix, 90 to 600 ms a call,
// 33 ms with it).  Every user runs in order on one stream.  Blocks that nobody
// uses and that are too small for a request are freed before it gets a new one, so
// growing requests do not add up.  After a call at most kKeep bytes stay; the
// rest is freed, after a call that failed all of it, and with the handle.
struct Workspace {
  static constexpr size_t kKeep = (size_t)256 << 20;
  struct Block { char* p; size_t cap, used; };
  struct Mark { size_t cur, used; };
  std::vector<Block> blocks;   // those behind cur are unused
  size_t cur = 0;              // block that serves the next request
  size_t held() const {
    size_t total = 0;
    for (auto& b : blocks) total += b.cap;
    return total;
  }
  void* get(size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    if (blocks.empty() || blocks[cur].used + bytes > blocks[cur].cap) {
      if (!blocks.empty() && blocks[cur].used > 0) cur++;   // its rest is left until the scope ends
      size_t k = cur;                                       // the first unused block that holds the request
      while (k < blocks.size() && blocks[k].cap < bytes) k++;
      if (k < blocks.size()) {
        std::swap(blocks[cur], blocks[k]);
      } else {
        pop_to(cur);   // all too small
        const size_t cap = std::max(bytes, std::min<size_t>(std::max<size_t>(held(), (size_t)4 << 20), (size_t)128 << 20));
        void* p = nullptr;
        const hipError_t e = hipMalloc(&p, cap);
        if (e != hipSuccess) {
          if (cur > 0) cur--;
          throw HipFail{e, "hipMalloc of a workspace"};
        }
        blocks.push_back({(char*)p, cap, 0});
      }
      blocks[cur].used = 0;
    }
    void* r = blocks[cur].p + blocks[cur].used;
    blocks[cur].used += bytes;
    return r;
  }
  Mark mark() const { return {cur, blocks.empty() ? 0 : blocks[cur].used}; }
  void reset(Mark m) {
    cur = m.cur;
    if (cur < blocks.size()) blocks[cur].used = m.used;
    else cur = blocks.empty() ? 0 : blocks.size() - 1;   // the unused block of the mark is gone
  }
  // frees the blocks from index n on (hipFree waits for the work that uses them)
  void pop_to(size_t n) {
    while (blocks.size() > n) {
      (void)hipFree(blocks.back().p);
      blocks.pop_back();
    }
  }
  // frees blocks from the last one until at most `keep` bytes are left (nothing in use)
  void trim(size_t keep) {
    size_t n = blocks.size(), total = held();
    while (n > 0 && total > keep) total -= blocks[--n].cap;
    pop_to(n);
    cur = 0;
  }
};

// One run over two workspaces: when it ends they keep at most kKeep each, and
// nothing if it failed.  Declared before the scopes that use them.
struct WorkspaceRun {
  Workspace &a, &b;
  bool ok = false;
  WorkspaceRun(Workspace& x, Workspace& y) : a(x), b(y) {}
  WorkspaceRun(const WorkspaceRun&) = delete;
  ~WorkspaceRun() {
    a.trim(ok ? Workspace::kKeep : 0);
    b.trim(ok ? Workspace::kKeep : 0);
  }
};

// Uploads of work lists through pinned memory, asynchronous and in stream order.
struct Stage {
  static constexpr size_t kCap = (size_t)4 << 20;
  char* p = nullptr;
  size_t used = 0;
  void upload(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return;
    if (!p) HIPCHK(hipHostMalloc((void**)&p, kCap, hipHostMallocDefault));
    for (size_t at = 0; at < bytes;) {
      if (used == kCap) {   // full: what was staged has to leave first
        HIPCHK(hipStreamSynchronize(s));
        used = 0;
      }
      const size_t n = std::min(bytes - at, kCap - used);
      std::memcpy(p + used, (const char*)src + at, n);
      HIPCHK(hipMemcpyAsync((char*)dst + at, p + used, n, hipMemcpyHostToDevice, s));
      used += n;
      at += n;
    }
  }
  void release() {
    if (p) (void)hipHostFree(p);
    p = nullptr;
  }
};

// A sandwich launch group: tasks with the same (ma, mb).
struct SWGroup {
  int ma = 0, mb = 0;
  int fmt = 0;        // low-precision plans: 1 = FP32 blocks, 2 = split-BF16 blocks
  int wg_strips = 0;  // row strips of a work unit on the matrix cores (set at upload)
  double flops = 0;   // algorithmic flops of one launch
  std::vector<SWTask> tasks;
  std::vector<SWItem> items;
  std::vector<int4> wus;
  std::vector<SWOut> outs;   // tasks with several outputs
  SWTask* d_tasks = nullptr;
  SWItem* d_items = nullptr;
  int4* d_wus = nullptr;
  SWOut* d_outs = nullptr;
};

// Row strips that one workgroup takes of a slice on the matrix cores, in a launch of
// `slices` slices: all of them (one staging serves up to eight), but at most four
// where even halves leave every workgroup a CU of its own.  More than four strips
// share the matrix pipes of four SIMDs, and the rest of the chip has nothing to do
// (FP64 matvec at the 8 x 8 root of m = 80,
// 96, 128: 71, 128 and 389 us in one workgroup a slice, 51, 84 and 218 this way).
inline int sw_wg_strips(int strips, int64_t slices) { return strips > 4 && slices <= 128 ? 4 : strips; }

// The items of one task or output, from `first` on, into the order that the
// FP64 and FP32 kernels rely on: those without B first (their loop over the rest
// loads through B without looking).  The plans list them so already.
inline void items_without_b_first(std::vector<SWItem>& v, size_t first) {
  std::stable_partition(v.begin() + first, v.end(), [](const SWItem& it) { return !it.B; });
}

struct MPGroup {
  int mj = 0;
  bool mfma = false;
  std::vector<MPTask> tasks;
  std::vector<MPJob> jobs;
  std::vector<int2> wus;
  MPTask* d_tasks = nullptr;
  MPJob* d_jobs = nullptr;
  int2* d_wus = nullptr;
};

struct CBPlan {
  std::vector<CBTask> tasks;
  std::vector<CBTerm> terms;
  CBTask* d_tasks = nullptr;
  CBTerm* d_terms = nullptr;
  int maxn = 0;
};

struct GRPlan {
  int mj = 0;
  bool mfma = false;
  GramForm form = GRAM_RAGGED;
  std::vector<GRTask> tasks;
  std::vector<GRReduce> reds;
  GRTask* d_tasks = nullptr;
  GRReduce* d_reds = nullptr;
};

struct MVDev {
  TinyPlan* d_plan = nullptr;   // every item written out (dense tiny H_eff, diagonal)
  TinyPlan* d_tiny = nullptr;   // == d_plan when the whole eigensolve runs in one workgroup
  std::vector<SWItem> tiny_items;
  int tiny_item0[3] = {0, 0, 0}, tiny_nitem[3] = {0, 0, 0};
  std::vector<Item3> tiny_items3;
  CBPlan comb;
  std::vector<SWGroup> sw;
  std::vector<MPGroup> chainA, chainB, chainC;   // one group per mj
  // the last stage with its jobs cut into several outputs (FP64; chainC writes
  // the first output of each leg), and the sources chainC leaves out
  std::vector<MPGroup> chainS;
  std::vector<const void*> split_outs;
  std::vector<RDSrc> srcs;
  RDSrc* d_srcs = nullptr;
  // low-precision plans: conversions that refresh the mirrors the lists read
  CVTask* d_cv = nullptr;
  int n_cv = 0;
  int64_t cv_max = 0;
  bool need_xt = false;
  int dims[3] = {0, 0, 0};
};

struct EnvChunk {
  std::vector<SWGroup> sw;
  GRPlan gr;
  std::vector<std::pair<double*, int64_t>> zero_blocks;
};

struct EnvDev {
  bool present = false;
  bool transpose = false;
  int dims[3] = {0, 0, 0};
  CBPlan comb;
  std::vector<EnvChunk> chunks;
  int node = -1, leg = -1, out_edge = -1, out_dir = 0;
};

// QR of a node tensor with one leg as the column index (three CholeskyQR passes)
struct QRDev {
  bool present = false;
  int mj = 0, nfc = 0, nwus = 0;
  bool gmf = false, mmf = false;
  GramForm gform = GRAM_RAGGED;
  int64_t rows = 0, Msz = 0;
  GRTask* d_gt[3] = {nullptr, nullptr, nullptr};
  GRReduce* d_gr = nullptr;
  MPTask* d_mt[3] = {nullptr, nullptr, nullptr};
  MPJob* d_mj[3] = {nullptr, nullptr, nullptr};
  int2* d_wus = nullptr;
  std::vector<GRTask> h_gt[3];
  std::vector<GRReduce> h_gr;
  MPGroup h_mp[3];   // host copies for validation
};

// T <- R x_leg T, in place on the matrix cores, through a temporary otherwise
struct ABDev {
  bool present = false;
  int mj = 0, nwus = 0;
  bool mmf = false;
  int64_t Msz = 0;
  MPTask* d_mt = nullptr;
  MPJob* d_mj = nullptr;
  int2* d_wus = nullptr;
  MPGroup h_mp;   // host copy for validation
};

// Matrix-core mode products: whole tiles, and ragged legs above half a tile
// over at least one tile of free indices (smaller ones are a few loads per
// output entry, one thread each).  Tensors are addressed by 32-bit byte offsets.
inline bool mode_mfma_ok(int mj, int64_t M) {
  return mj <= 128 && M < ((int64_t)1 << 27) && ((mj % 16 == 0 && (M / mj) % 64 == 0) || (mj > 8 && M / mj >= 16));
}
inline int64_t mode_blocks(int mj, int64_t M) { return (M / mj + 63) / 64; }
inline bool gram_mfma_ok(int mj, int64_t M) { return mode_mfma_ok(mj, M); }
// Free indices per gram work unit (whole 64-wide blocks, the last unit takes
// what is left): at most `parts` units, about that many where the free range
// allows it.
inline int64_t gram_chunk(int64_t F, int parts) {
  int64_t c = std::max<int64_t>(64, ((F + parts - 1) / parts + 63) / 64 * 64);
  if (F % 64 == 0)
    while (F % c) c += 64;   // equal units
  return c;
}
inline int gram_parts(int64_t F, int parts) {
  const int64_t c = gram_chunk(F, parts);
  return (int)((F + c - 1) / c);
}
// Parts of the grams of effective-operator updates and of QRs: enough workgroups,
// few partial sums to add up.
constexpr int kEnvGramParts = 8, kQrGramParts = 32;

}  // namespace rt

using namespace attn;   // internal header: the runtime sources use both namespaces
using namespace rt;

// Host copy of the problem a handle was built from (every array deep-copied),
// kept for the problem hash of checkpoints and for rebuilding the rotated
// terms when the disentanglers change.
struct ProblemCopy {
  int32_t n_sites = 0, d = 0, m = 0;
  std::vector<int32_t> leaf_order, term_nsites, term_sites, de_sites;
  std::vector<double> term_ops, term_coef, de_u;
  uint32_t flags = 0;
  int32_t device = 0;
  void assign(const attn_problem* p);
  attn_problem view() const;
  // FNV-1a over everything that fixes the tree and the Hamiltonian: sizes,
  // leaf order, terms, disentangler sites and the strict flag (not the
  // disentangler matrices, which the optimisation changes, and not the device)
  uint64_t hash() const;
};

struct StoreRange {   // addresses of one effective-operator store
  uintptr_t begin, end;
  int dir, edge;
};

struct attn_handle {
  Model M;
  ProblemCopy prob;
  uint64_t problem_hash = 0;
  std::vector<double> sweep_energies;   // theta at the last node of every attn_sweep sweep
  std::string err;
  bool host_only = false;
  bool dryrun = false;
  bool dead = false;
  uintptr_t fake_next = (uintptr_t)1 << 40;
  std::vector<std::pair<uintptr_t, size_t>> allocs;
  int device = 0;
  std::vector<void*> owned;
  // tensors
  double* d_T = nullptr;
  std::vector<int64_t> T_off;
  std::vector<int64_t> T_len;
  // effective-operator stores per edge and direction
  std::vector<double*> store[2];
  std::vector<char> valid[2];
  std::vector<int> iso;       // per node: leg it is isometric toward, -1 = centre
  int center = -1;
  bool state_ready = false;
  // scratch
  int64_t Mmax = 0;
  int kcap = 65;   // at most 64 Krylov vectors (+1)
  double* d_V = nullptr;      // (kcap) x Mmax
  double* d_w = nullptr;
  double* d_xt = nullptr;
  double* d_tmp = nullptr;
  double* d_tmp2 = nullptr;
  float* d_x32 = nullptr;
  float* d_y32 = nullptr;
  double* d_part = nullptr;   // mv partial outputs
  int64_t part_cap = 0;
  double* d_chain = nullptr;
  int64_t chain_cap = 0;
  double* d_mvcomb = nullptr;
  double* d_envcomb = nullptr;
  double* d_Z = nullptr;
  double* d_grpart = nullptr;   // partial grams of one chunk of outputs
  int64_t grpart_cap = 0;
  double* d_red = nullptr;    // 128 x kRedBlocks
  double* d_qrmat = nullptr;  // G, R0, R1, R2, Rinv, Rt (mmax^2 each), Cholesky workspace
  double* d_qrR = nullptr;    // R of the last QR (absorbed into the neighbour)
  int mmax = 1;
  KrylovState* d_st = nullptr;
  // sweeps: per-node status checks stay on the device (no host round trip per
  // node); every failure status also lands in d_st->sticky, read once per sweep
  bool defer_status = false;
  KJob* d_kjobs64 = nullptr;  // per node: eigensolve descriptors (FP64 / with FP32 copy)
  KJob* d_kjobs32 = nullptr;
  TJob* d_tjobs = nullptr;    // per node: dense tiny-node eigensolve
  std::vector<KJob> h_kjobs;  // host copies for validation
  // Davidson form (allocated at its first use)
  DJob* d_djobs = nullptr;    // per node
  std::vector<DJob> h_djobs;
  DavState* d_dav = nullptr;
  void* d_mlp = nullptr;      // FP16 parameters of the learned correction model
  bool mlp_ready = false;
  double jacobi_rate = 0.9;   // running per-iteration residual reduction of Jacobi-mode solves
  int64_t n_dav_iter = 0, n_fallback = 0;
  double last_rnorm = 0;
  std::vector<TJob> h_tjobs;
  // plans
  std::vector<MVDev> mv;
  // low-precision forms: 4-byte-per-element mirrors of the FP64 stores (FP32,
  // or BF16 hi/lo planes per block) and copies of every matvec work list
  bool lowp_ready[2] = {false, false};
  std::vector<void*> mir[2][2];     // [format - 1][direction][edge]
  std::vector<int64_t> store_elems[2];
  std::vector<StoreRange> store_ranges;   // the stores by address
  void* comb_lp[2] = {nullptr, nullptr};
  int64_t mvcomb_elems = 0;
  std::vector<MVDev> mvlp[2];
  std::vector<EnvDev> env_up, env_down[2];
  std::vector<QRDev> qr[3];   // per leg, per node
  std::vector<ABDev> ab[3];   // absorb into node along leg
  // FP64 Lanczos sweeps captured as HIP graphs (attn_sweep_opts.use_graphs):
  // a graph replays the launches of one whole sweep from the host state it was
  // captured in (centre, isometry legs, valid stores) and leaves the state it
  // left then, so it is replayed only from an identical start state
  struct SweepState {
    int center = -1;
    std::vector<int> iso;
    std::vector<char> valid0, valid1;
    bool operator==(const SweepState& o) const {
      return center == o.center && iso == o.iso && valid0 == o.valid0 && valid1 == o.valid1;
    }
  };
  struct SweepGraph {
    hipGraphExec_t exec = nullptr;
    int krylov_k = 0;
    SweepState pre, post;
    int64_t d_matvec = 0, d_env = 0, d_qr = 0;
    double d_flops = 0;
  };
  hipStream_t gstream = nullptr;
  std::vector<SweepGraph> sgraphs;   // at most two (the first sweep from a fresh state, then the steady one)
  // observables: memory of a whole run, of its scopes, and the upload stage
  Workspace xkeep, xtmp;
  Stage xstage;
  // counters
  int64_t n_matvec = 0, n_env = 0, n_qr = 0;
  double mv_flops = 0;
  // live timing of the matvec sandwich launches (HIP events on the launch stream)
  bool prof = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  struct ProfRec { int a, b; double flops; int ma, mb, dtype; };
  std::vector<ProfRec> prof_recs;
};


// ---------------------------------------------------------------- shared helpers (runtime.cpp)
namespace rt {
void* dev_alloc(attn_handle* h, size_t bytes);
template <typename T>
T* upload(attn_handle* h, const std::vector<T>& v) {
  if (v.empty()) return nullptr;
  void* p = dev_alloc(h, v.size() * sizeof(T));
  if (!h->dryrun) HIPCHK(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return (T*)p;
}
double* block_ptr(attn_handle* h, const BRef& b, double* comb_base, const std::vector<int64_t>& comb_off);
void slice_geom(int spect, const int* dm, int& ma, int& mb, int& ns, int64_t& sl, int64_t& row);
// item chunks per spectator of the matvec plan of a node with dims dm
// (target workgroups per launch, per spectator's slice shape)
// Matvec work units per spectator group (three groups per node).  Four strips
// (the full nodes): 3 x 1024 = three rounds of the 1024 workgroups resident at
// four per CU; measured at the heaviest 16 x 16 m = 64 node (contraction + sum of
// the partial outputs) 1141 + 43 us, against 1158 + 34 with 768 and 1178 + 29
// with 683.  Fewer strips: 768, where the launches are shorter than the spread
// of their workgroups; and off the matrix cores (legs above 128: 4 x 4 m = 256, root,
// 21.3 ms with 768 and 28.4 with 1024, whose workgroups walk more blocks at once
// than the L2 holds).  The batched form takes the same split unless it is autotuned.
inline int64_t mv_target(int ma, int mb) { return sw_strips(ma) >= 4 && sw_on_mfma(ma, mb) ? 1024 : 768; }
inline void mv_targets(const int* dm, int64_t target[3]) {
  for (int sp = 0; sp < 3; sp++) {
    int ma, mb, ns;
    int64_t sl, row;
    slice_geom(sp, dm, ma, mb, ns, sl, row);
    target[sp] = mv_target(ma, mb);
  }
}
void mv_chunks(const MatvecPlan& P, const int* dm, const int64_t target[3], int out[3]);
bool sw_mfma(int ma, int mb);
// Doubles of the QR matrices of a handle whose widest link is mmax: G, R0, R1,
// R2, R^-1, R products (mmax^2 each) and the Cholesky workspace of links wider
// than 128 (two packed triangles, mmax (mmax + 1)).
inline int64_t qrmat_doubles(int64_t mmax) { return 6 * mmax * mmax + mmax * (mmax + 1); }
// Most item chunks (workgroup sets with their own partial output) of one
// sandwich group of a matvec: small nodes get more, so that their few slices
// still spread over the chip.
inline int64_t chunk_cap(int64_t Msz) {
  return Msz >= 65536 ? 32 : std::min<int64_t>(128, std::max<int64_t>(32, ((int64_t)1 << 19) / Msz));
}
// C chunks shared out over n spectators in proportion to their item counts by
// largest remainders, at least one each.
inline void chunk_shares(int64_t C, const int64_t* items, int n, int64_t* c) {
  int64_t tot = 0, rem[3], sum = 0;
  for (int g = 0; g < n; g++) tot += items[g];
  for (int g = 0; g < n; g++) {
    c[g] = C * items[g] / tot;
    rem[g] = C * items[g] - c[g] * tot;   // remainder of the exact share, in units of 1 / tot
    if (c[g] == 0) { c[g] = 1; rem[g] -= tot; }   // every spectator with items gets a chunk
    sum += c[g];
  }
  while (sum < C) {   // the largest remainders get one more chunk (lowest spectator first on ties)
    int best = 0;
    for (int g = 1; g < n; g++)
      if (rem[g] > rem[best]) best = g;
    c[best]++;
    rem[best] -= tot;
    sum++;
  }
  while (sum > C) {   // the smallest remainders among spectators with two chunks or more give one back
    int worst = -1;
    for (int g = 0; g < n; g++)
      if (c[g] > 1 && (worst < 0 || rem[g] < rem[worst])) worst = g;
    if (worst < 0) break;
    c[worst]--;
    rem[worst] += tot;
    sum--;
  }
}
// Chunks of a launch whose slices have more than four strips.  Few such
// workgroups are resident (two per CU at five and six strips, one at seven
// and eight), and a chunk is as many of them as the spectator has slices, so
// a fixed count leaves the last round part empty (128 slices x 9 chunks on 256
// slots: 4.5 rounds).  The count with the shortest list schedule is taken,
// between two and eight rounds: a workgroup lasts its items and one more (its
// slice in and out), and a chunk costs the write and the later read of a
// partial output, 50 / m items of the whole chip (16 bytes per entry at
// 4.75 TB/s against 4 m flops per entry and item at 60 TFLOP/s).  Counts past the
// most chunks that the spectators may have (cap each) are not tried: at a node
// with one slice there would be thousands (building the lists of an 8 x 8 m = 96
// handle: 300 ms with them, 36 without).
inline int64_t wide_chunks(const int64_t* items, int n, int64_t units, int m, int strips, int64_t cap) {
  const int64_t slots = 256 * (strips <= 6 ? 2 : 1);
  int64_t most = 0;
  for (int g = 0; g < n; g++) most += std::min(items[g], cap);
  const int64_t lo = std::min(most, std::max<int64_t>(n, 2 * slots / units));
  const int64_t hi = std::min(most, std::max<int64_t>(lo, 8 * slots / units));
  double best = 0;
  int64_t bestC = lo;
  for (int64_t C = lo; C <= hi; C++) {
    int64_t c[3];
    chunk_shares(C, items, n, c);
    std::vector<int64_t> len;
    for (int g = 0; g < n; g++)
      for (int64_t k = 0; k < c[g]; k++) len.push_back(items[g] * (k + 1) / c[g] - items[g] * k / c[g]);
    std::sort(len.rbegin(), len.rend());
    std::map<double, int64_t> idle;   // slots by the time they become free
    idle[0.0] = slots;
    double end = 0;
    for (int64_t l : len)
      for (int64_t left = units; left > 0;) {
        const auto it = idle.begin();
        const double t = it->first;
        const int64_t k = std::min(left, it->second);
        it->second -= k;
        if (it->second == 0) idle.erase(it);
        idle[t + (double)l + 1.0] += k;
        end = std::max(end, t + (double)l + 1.0);
        left -= k;
      }
    const double cost = end + (double)C * units / slots * (50.0 / m);
    if (C == lo || cost < best) { best = cost; bestC = C; }
  }
  return bestC;
}
// Item chunks per spectator of a matvec plan.  Spectators whose slices have
// the same shape share one launch; the launch gets C = (number of such
// spectators) x target / units item chunks in total (units = workgroups per
// chunk), shared out in proportion to the spectators' item counts by largest
// remainders, so that every chunk carries about the same number of items and
// the chunks add up to exactly C (a launch of C x units workgroups: with the
// default target, whole rounds of the chip's workgroup slots, and no round
// that starts only a few of them).  nitems[sp] = 0: no chunk.
inline void mv_chunk_counts(const int64_t nitems[3], const int ma[3], const int mb[3], const int64_t units[3],
                            int64_t Msz, const int64_t target[3], int out[3]) {
  for (int sp = 0; sp < 3; sp++) out[sp] = 0;
  bool done[3] = {false, false, false};
  for (int sp = 0; sp < 3; sp++) {
    if (nitems[sp] <= 0 || done[sp]) continue;
    int grp[3], ng = 0;
    int64_t it[3], c[3];
    for (int q = 0; q < 3; q++)
      if (nitems[q] > 0 && ma[q] == ma[sp] && mb[q] == mb[sp]) { it[ng] = nitems[q]; grp[ng++] = q; done[q] = true; }
    int64_t C = ng * std::max<int64_t>(1, target[sp] / std::max<int64_t>(1, units[sp]));
    if (sw_on_mfma(ma[sp], mb[sp]) && sw_strips(ma[sp]) > 4)
      C = wide_chunks(it, ng, units[sp], ma[sp], sw_strips(ma[sp]), chunk_cap(Msz));
    chunk_shares(C, it, ng, c);
    for (int g = 0; g < ng; g++) {
      const int q = grp[g];
      out[q] = (int)std::max<int64_t>(1, std::min<int64_t>(c[g], std::min<int64_t>(nitems[q], chunk_cap(Msz))));
    }
  }
}
void run_comb(CBPlan& P, hipStream_t s);
void* to_mirror(attn_handle* h, const void* p, int fmt);
void ensure_lowp(attn_handle* h, int dtype);
std::vector<CVTask> lowp_conversions(attn_handle* h, int n, int dtype);
int leg_toward(const Tree& tr, int a, int b);
void run_env(attn_handle* h, EnvDev& D, hipStream_t s);
void qr_node(attn_handle* h, int n, int leg, hipStream_t s);
void absorb(attn_handle* h, int q, int leg, hipStream_t s);
attn_status guard(attn_handle* h, const std::function<attn_status()>& f);
attn_status need_device(attn_handle* h);
void check_state(attn_handle* h, hipStream_t s, const char* where);
void reset_state(attn_handle* h, int kmax, hipStream_t s);
// Mark every effective-operator store stale, then recompute every store that
// points toward the current centre (children before parents off the centre's
// path, then down the path from the root).  Requires every node other than the
// centre to be isometric toward the centre.
void rebuild_envs(attn_handle* h, hipStream_t s);
}  // namespace rt
