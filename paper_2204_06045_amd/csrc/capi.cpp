// C ABI (include/qtn.h): network build, planning, schedule and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "device.hpp"
#include "kernels.hpp"
#include "mlp.hpp"
#include "plan.hpp"
#include "qtn.h"

using namespace qtn;

namespace {

thread_local std::string g_err;

int set_err(int code, const std::string &msg) {
  g_err = msg;
  return code;
}

#define QTN_HIP(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess)                                                          \
      return set_err(QTN_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Status of the exception being handled, at the C ABI, which no C++
// exception crosses: QTN_ENOMEM for a failed host allocation, QTN_EINVAL
// ("internal error: ...") for anything else.
int exception_status() {
  try {
    throw;
  } catch (const std::bad_alloc &) {
    return set_err(QTN_ENOMEM, "host allocation failed");
  } catch (const std::exception &e) {
    return set_err(QTN_EINVAL, std::string("internal error: ") + e.what());
  } catch (...) {
    return set_err(QTN_EINVAL, "internal error");
  }
}

uint32_t pext32(uint32_t x, uint32_t mask) {
  uint32_t r = 0, d = 0;
  for (int b = 0; b < 32; b++)
    if ((mask >> b) & 1u) r |= ((x >> b) & 1u) << d++;
  return r;
}

// Runs f(i) for i in [0, n) on up to hardware_concurrency threads.
template <class F>
void parallel_for(int n, F f) {
  int nt = (int)std::min<unsigned>(std::max(1u, std::thread::hardware_concurrency()), 32u);
  nt = std::min(nt, n);
  if (nt <= 1) {
    for (int i = 0; i < n; i++) f(i);
    return;
  }
  std::atomic<int> next{0};
  std::vector<std::thread> th;
  for (int t = 0; t < nt; t++)
    th.emplace_back([&] {
      for (int i = next++; i < n; i = next++) f(i);
    });
  for (auto &x : th) x.join();
}

struct Task {
  int kind;        // QTN_K_BLOCK: range index; QTN_K_WIDE: group index
  int index;
  uint32_t n_units;
  int variant;     // wide groups: mapping variant
  double bytes, flops;
  double ms = -1;  // the cost model's time (-1: none)
};

// Workspace of a schedule: byte offsets of its parts.
struct Layout {
  size_t off_res = 0, off_angles = 0, off_desc = 0, off_fills = 0, off_groups = 0, off_ops = 0,
         off_stab = 0, off_uperm = 0, off_ranges = 0, off_prog = 0, off_csb = 0, off_ncb = 0,
         off_cns = 0, off_step_tasks = 0, off_items = 0, off_steps = 0, off_item_task = 0,
         off_task_next = 0, off_task_first = 0, off_task_need = 0, off_queue = 0, off_ctl = 0,
         off_data = 0, total = 0;
};

// Device layout and launch list of one or more planned networks.
struct Schedule : Layout {
  int prec = 0;        // QTN_C128, QTN_C64 or QTN_MIXED
  int scalar_prec = 0;  // storage of the scalar slots
  std::vector<DevGroup> groups;
  std::vector<DevOp> ops;
  // segments: groups [x, y), program at word z of prog (-1: group by group);
  // first n_cones: each cone's leading small groups
  std::vector<int4> ranges;
  std::vector<uint32_t> prog;  // segment programs (device.hpp)
  size_t prog_more = 0;        // words kept free behind them
  int lead_prec = -1;          // arithmetic of the leading segments if all are
                               // programs of one precision, else -1
  std::vector<int> csb, ncb;
  std::vector<int> cns;       // slices per light cone (index slicing; 1: none)
  // hybrid executor: cones whose groups after the leading segment run by
  // per-group launches after the persistent launch (they may take the cell
  // mapping)
  std::vector<char> cone_heavy;
  std::vector<FillDesc> fills;
  std::vector<int32_t> stab;  // serial-offset tables of streaming operands
  std::vector<uint8_t> uperm; // 32 bytes per group: union bit of each unit bit
  std::vector<int> group_cone, group_index;  // plan position of each group
  // place of each group in the device's group array, which leaves out the
  // groups that run as segment programs (-1)
  std::vector<int> dev_group;
  std::vector<size_t> stab_at;  // first stab entry of each group
  // groups also given one-group ranges (tuning): from singles_range0 on, each
  // one's program (if it has one), then each one by its mapping
  std::vector<int> singles;
  int singles_range0 = 0;
  std::vector<std::vector<Task>> cone_tasks;  // after the leading small groups
  int n_cones = 0, n_nets = 0, n_angles = 0;
  size_t set_bytes = 0;  // data of one angle set
  int64_t scalar_off = 0, scalar_sstride = 0;
  int n_sets = 1;  // angle sets evaluated per launch (one copy of the data each)
  // step launches: the j-th task of every light cone (after the leading
  // segment) in one launch; tasks of other mappings follow one by one
  struct Step {
    int first = 0, n = 0, blocks = 0;  // tasks [first, first + n) of step_tasks
    int threads = 0;                   // of a workgroup
    size_t lds = 0;
    std::vector<Task> single;
  };
  std::vector<Step> steps;
  std::vector<int4> step_tasks;
  std::vector<char> desc_blob;  // bytes [off_desc, off_data)
  uint64_t serial = 0;          // distinct for every schedule built
  int item_order = 0;           // lockstep steps: 0 costliest cone's items first, 1 reversed
  double bytes[QTN_NKERNELS] = {}, flops[QTN_NKERNELS] = {};
  double init_bytes = 0, init_flops = 0;
  // persistent executors: work items in step order; the task (one cone's
  // segment or wide group) of each item, each task's predecessor in its cone
  // (-1: none) and its item count
  std::vector<int4> items;
  std::vector<int> step_begin, item_task, task_dep, task_need, task_next, task_first;
  int n_steps = 0, n_tasks = 0, n_init = 0;
  int n_ctl = 0;
};

// Device memory that the library keeps for descriptors, all together.  A batch's
// lives until one of its networks is planned anew or freed, so a program that
// forms batch after batch of the same networks would otherwise fill the card;
// past the bound, this part of the device's memory, a call sends its
// descriptors into the workspace.  A batch of 64 graphs of 20 to 200 vertices,
// depths 2 to 4, takes 236 MB: nine of them on a card of 288 GB.
constexpr size_t kDescPart = 128;
std::atomic<size_t> g_desc_bytes{0};

// Memory of the current device, asked for once per device (0: unknown).
size_t device_bytes() {
  constexpr int kMaxDevices = 64;
  static std::atomic<size_t> known[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  size_t all = known[dev];
  if (!all && hipDeviceTotalMem(&all, dev) == hipSuccess) known[dev] = all;
  return all;
}

// Null past the bound, and where the device has none left (*none).
char *desc_alloc(size_t bytes, bool *none) {
  char *p = nullptr;
  *none = false;
  const size_t held = g_desc_bytes.fetch_add(bytes) + bytes, all = device_bytes();
  if (!all || (held <= all / kDescPart && hipMalloc((void **)&p, bytes) != hipSuccess)) {
    (void)hipGetLastError();
    *none = true;
    p = nullptr;
  }
  if (p) return p;
  g_desc_bytes -= bytes;
  return nullptr;
}

void desc_free(char *p, size_t bytes) {
  if (!p) return;
  (void)hipFree(p);
  g_desc_bytes -= bytes;
}

// Streams, events, pinned staging and the captured graph of one schedule.
struct Runtime {
  int device = -1;
  hipStream_t main = nullptr;
  std::vector<hipStream_t> side;
  hipEvent_t ev_in = nullptr, ev_fork = nullptr;
  std::vector<hipEvent_t> ev_join;
  double *pinned = nullptr;
  size_t pinned_n = 0;
  void *ws = nullptr;  // workspace the captured graph was recorded for
  // the schedule's descriptors in device memory of the library's own, uploaded
  // once per schedule (the workspace's contents are the caller's between
  // calls); null where that allocation failed: then they go up into the
  // workspace before every evaluation
  char *dev_desc = nullptr;
  size_t dev_desc_cap = 0;
  uint64_t dev_serial = 0;    // schedule whose descriptors dev_desc holds
  uint64_t no_dev_serial = 0; // schedule for which there was no memory
  char *desc_base = nullptr;  // offsets off_desc..off_data count from here
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  int persist_blocks = 0;
  uint32_t *pinned_err = nullptr;

  void release() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    exec = nullptr;
    graph = nullptr;
    for (auto s : side) (void)hipStreamDestroy(s);
    side.clear();
    for (auto e : ev_join) (void)hipEventDestroy(e);
    ev_join.clear();
    if (ev_in) (void)hipEventDestroy(ev_in);
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (main) (void)hipStreamDestroy(main);
    if (pinned) (void)hipHostFree(pinned);
    if (pinned_err) (void)hipHostFree(pinned_err);
    desc_free(dev_desc, dev_desc_cap);
    pinned_err = nullptr;
    dev_desc = desc_base = nullptr;
    dev_desc_cap = 0;
    dev_serial = 0;
    persist_blocks = 0;
    ev_in = ev_fork = nullptr;
    main = nullptr;
    pinned = nullptr;
    pinned_n = 0;
    ws = nullptr;
    device = -1;
  }
  // The captured graph and the uploaded descriptors belong to one schedule.
  void forget_schedule() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    exec = nullptr;
    graph = nullptr;
    ws = nullptr;
    dev_serial = 0;
  }
  // Takes over o's streams, events and pinned buffers (o is left empty), for
  // a new schedule of the same network: streams are not torn down and
  // re-created when a plan is re-tuned.
  void take(Runtime &o) {
    if (&o == this) return;
    release();
    device = o.device;
    main = o.main;
    side.swap(o.side);
    ev_in = o.ev_in;
    ev_fork = o.ev_fork;
    ev_join.swap(o.ev_join);
    pinned = o.pinned;
    pinned_n = o.pinned_n;
    persist_blocks = o.persist_blocks;
    pinned_err = o.pinned_err;
    dev_desc = o.dev_desc;
    dev_desc_cap = o.dev_desc_cap;
    exec = o.exec;
    graph = o.graph;
    o.exec = nullptr;
    o.graph = nullptr;
    o.main = nullptr;
    o.ev_in = o.ev_fork = nullptr;
    o.pinned = nullptr;
    o.pinned_n = 0;
    o.pinned_err = nullptr;
    o.dev_desc = o.desc_base = nullptr;
    o.dev_desc_cap = 0;
    o.dev_serial = 0;
    o.persist_blocks = 0;
    o.ws = nullptr;
    o.device = -1;
    forget_schedule();
  }
  Runtime() = default;
  Runtime(const Runtime &) = delete;
  Runtime &operator=(const Runtime &) = delete;
  ~Runtime() { release(); }
};

struct Exec {
  Schedule sched;
  Runtime rt;
  bool persistent = false;
  bool dataflow = false;  // persistent: per-task dependencies instead of lockstep
  bool hybrid = false;    // persistent lockstep for light cones, launches for heavy ones
  bool lead_per_cone = false;
  bool steps = false;     // executor 0: step launches where the schedule has them
  uint32_t spin_limit = 1u << 22;
  int grid_quarters = 4;  // persistent grid: this many quarters of the resident blocks
};

std::atomic<uint64_t> g_sched_serial{0};  // Schedule::serial source

}  // namespace

struct qtn_network {
  Graph g;
  int p = 0;
  std::vector<double> gamma, beta;
  PlanOptions opt;
  int n_streams = 4;
  bool eager = false;
  int lane_sum_bits = 2;  // streaming: summed bits spread over lanes
  int order_trials = 0;   // >1: best of this many randomized min-fill orders
  int hybrid_width = 20;  // executor 5: cones with a bucket wider than this are heavy
  int executor = 0;       // 0 streams + per-group launches, 1 persistent lockstep
  uint32_t spin_limit = 1u << 22;
  int variant = 0;        // 0 auto, 1 generic only, 2 streaming where possible,
                          // 3 matrix form where possible, 4 cells where possible
  std::vector<LightCone> cones;
  std::vector<std::vector<int>> minfill;
  std::mutex minfill_lock;
  bool planned = false;
  int precision = 0;
  uint64_t version = 0;
  std::vector<ConePlan> plans;
  std::unique_ptr<Exec> exec;
  std::vector<qtn_launch_rec> launch_log;
  std::vector<qtn_tune_rec> tune_log;
  size_t tune_workspace = 0;
  // angle-set batches: a schedule with one data copy per set, rebuilt when
  // the set count or the plan changes; [1]: with the plan's order of
  // operations (derivatives in complex64)
  struct AngleExec {
    std::unique_ptr<Exec> exec;
    int sets = 0;
    uint64_t version = 0;
  } angle_exec[2];
};

namespace {

std::mutex g_batch_lock;
std::map<std::vector<std::pair<const qtn_network *, uint64_t>>, std::unique_ptr<Exec>> g_batch;

void drop_batches_with(const qtn_network *net) {
  std::lock_guard<std::mutex> lk(g_batch_lock);
  for (auto it = g_batch.begin(); it != g_batch.end();) {
    bool has = false;
    for (auto &kv : it->first) has |= kv.first == net;
    it = has ? g_batch.erase(it) : std::next(it);
  }
}

const std::vector<int> &get_minfill(qtn_network *net, int e) {
  std::lock_guard<std::mutex> lk(net->minfill_lock);
  if (net->minfill[e].empty()) net->minfill[e] = minfill_order(net->cones[e]);
  return net->minfill[e];
}

// Element offset of a gate's values in the gate table.  A gate cut by index
// slicing reads the block whose bit 0 is its remaining axis, at the row of
// the fixed axis's value (bit cut_slot of the slice number).
int64_t gate_offset(const Gate &gt, bool transposed, int p, uint32_t slice = 0) {
  int t = transposed ? 4 : 0;
  if (gt.cut >= 0) t = (gt.cut == 1 ? 4 : 0) + 2 * (int)((slice >> gt.cut_slot) & 1u);
  switch (gt.kind) {
    case kH: return 32LL * p;
    case kZ: return 32LL * p + 2;
    case kP: return 32LL * gt.layer + 0 + t;
    case kPc: return 32LL * gt.layer + 8 + t;
    case kR: return 32LL * gt.layer + 16 + t;
    default: return 32LL * gt.layer + 24 + t;
  }
}

// Bytes of the largest operand of a group (gate tables count in the group's
// precision).  The streaming and cell mappings address the lane and cell
// parts of an operand with 32-bit byte offsets, so they take only groups
// whose operands all fit in 4 GiB; the generic mapping addresses elements
// with 64-bit indices and takes any group.
double max_operand_bytes(const Group &G, const ConePlan &pl) {
  double mx = 0;
  for (const Operand &o : G.ops) {
    const Tensor &t = pl.tensors[o.tensor];
    const int prec = t.gate >= 0 ? G.prec : t.prec;
    mx = std::max(mx, std::ldexp(prec == 1 ? 8.0 : 16.0, (int)t.vars.size()));
  }
  return mx;
}
constexpr double kOffset32Bytes = 4294967296.0;

// Candidate kernel configuration the autotuner forces on every wide group.
struct Force {
  int place;    // -1 keep, 0 workgroup segment, 1 own launch
  int variant;  // 1 generic, 2 streaming, 3 matrix form, 4 cells
  int rls;      // streaming: lane-summed bits; cells: register bits
};

constexpr int kTuneSingleWidth = 16;

// Configurations measured by the autotuner: every group in its own launch
// with the generic mapping, with the streaming mapping at 1, 2, 3
// lane-summed bits, in matrix form (groups that have one), or with
// the cell mapping at 3 or 4 cell bits (groups wide enough for it; 2 cell
// bits were measured too and never won on the N=30 p=4 network).
const std::vector<Force> &tune_candidates() {
  static const std::vector<Force> c = {{1, 1, 2}, {1, 2, 1}, {1, 2, 2}, {1, 2, 3},
                                       {1, 3, 2}, {1, 4, 3}, {1, 4, 4}};
  return c;
}

// A tuned or learned pick of the cell mapping where no cell kernel runs (the
// persistent executors): the generic mapping up to this union width, past it
// the width rule.  Persistent batches with learned picks, milliseconds by the
// rule alone, up to 16, 20 and 32 bits: 6 graphs of 10 to 40 vertices, depths to 3,
// complex128 1.61, 1.41, 1.34, 1.32, complex64 1.66, 1.47, 1.44, 1.44; 4 graphs of
// 10 to 24 vertices, depths to 4, 6.32, 6.29, 5.97, 6.55 and 6.41, 6.19, 5.84, 6.28.
constexpr int kNoCellWidth = 20;

// Where a group's operands and output live (bytes from the data base) and
// the kernel configuration requested for it.
struct GroupEnv {
  int64_t out_off = 0, out_sstride = 0;   // output (tensor or scalar slot), set 0
  int64_t arena = 0, arena_sstride = 0;   // intermediates sit at arena + Tensor::offset
  int64_t table[2] = {-1, -1};            // gate tables: complex128, complex64
  int64_t table_sstride[2] = {0, 0};
  const std::vector<Gate> *gates = nullptr;  // gates of the group's gate operands
  uint32_t slice = 0;                     // index slicing: the slice's number
  int p = 0;                              // QAOA depth (gate table layout)
  int var_req = 0, rls_req = 2;           // mapping requested (0: the width rule)
  bool is_small = false;                  // runs inside a workgroup segment
  bool persistent = false;                // the schedule runs in a persistent executor
  bool in_order = false;                  // complex64 groups keep the plan's operand order
};

// Device descriptor of one group: chooses its mapping, appends its operands
// to s.ops (their tables to s.stab, its unit-bit order to s.uperm) and
// returns the group record with its algorithmic bytes and flops.
int describe_group(const Group &G, const ConePlan &pl, const GroupEnv &env, Schedule &s,
                   DevGroup *dg_out, double *bytes_out, double *flops_out) {
  auto es = [](int prec) { return prec == 1 ? (int64_t)8 : (int64_t)16; };
  DevGroup dg;
  std::memset(&dg, 0, sizeof dg);
  dg.out_off = env.out_off;
  dg.out_sstride = env.out_sstride;
  dg.prec = (uint8_t)G.prec;
  dg.op_begin = (int32_t)s.ops.size();
  dg.w = (uint8_t)G.w;
  dg.L = (uint8_t)G.L;
  dg.n_ops = (uint8_t)G.ops.size();
  double in_bytes = 0;
  std::vector<int> per_level(G.L, 0);
  for (const Operand &o : G.ops) {
    per_level[o.level]++;
    const Tensor &t = pl.tensors[o.tensor];
    in_bytes += std::ldexp(1.0, (int)t.vars.size()) * es(t.gate >= 0 ? G.prec : t.prec);
  }
  int var_req = env.var_req, rls_req = env.rls_req;
  const bool is_small = env.is_small, persistent = env.persistent;
  const int rls = std::min(G.L - 1, rls_req);
  const int sl = G.L - 1 - rls;
  const bool off32 = max_operand_bytes(G, pl) <= kOffset32Bytes;
  const bool stream_ok = (int)G.ops.size() <= kStreamMaxOps && sl <= kStreamMaxSerial && off32;
  // matrix form: groups that split into two sides (gemm_shape), requested or
  // picked by tuning; complex128 tiles take more LDS than the workgroup and
  // persistent kernels hold, so complex128 groups take it in own launches only
  GemmShape gsh;
  const bool mfma = var_req == 3 && (G.prec == 1 || (!is_small && !persistent)) &&
                    gemm_shape(G, pl, &gsh);
  if (var_req == 3 && !mfma) var_req = 0;
  // cells: lanes on union bits 0..5, cb cell bits in registers (the
  // summed bits above bit 5, then rb kept bits); own launches only (the
  // kernel is not part of the workgroup and persistent paths).  Taken
  // when requested, and by the rule for every own-launch group it fits
  const int low = std::max(G.L, 6);
  auto cell_fits = [&](int cbits) {
    const int r = cbits - std::max(0, G.L - 6);
    return !is_small && !persistent && off32 && (int)G.ops.size() <= kCellMaxOps &&
           G.L - 6 <= kCellMaxSerial && r >= 0 && G.w - low >= r;
  };
  int cb = 0;
  bool cell = false;
  if (var_req == 4) {
    cb = rls_req >= kCellMinCB && rls_req <= kCellMaxCB ? rls_req : kCellRuleCB;
    cell = cell_fits(cb);
    if (!cell) var_req = 0;
  }
  if (var_req == 0 && !mfma && cell_fits(kCellRuleCB)) {
    cb = kCellRuleCB;
    cell = true;
  }
  const int rb = cell ? cb - std::max(0, G.L - 6) : 0;
  // otherwise the streaming mapping once a lane walks >= 2 serial bits
  const bool stream =
      !mfma && !cell && stream_ok && (var_req == 2 || (var_req == 0 && sl >= 2));
  std::vector<int> order(G.ops.size());
  std::vector<int> cls(G.ops.size(), 0);
  for (size_t k = 0; k < G.ops.size(); k++) order[k] = (int)k;
  dg.in_order = cell && env.in_order && G.prec == 1;
  if (mfma) {
    dg.variant = kVarMfma;
    // [side A..., side B...]
    std::vector<int> side[2];
    for (int k = 0; k < (int)G.ops.size(); k++) side[gsh.role[k]].push_back(k);
    order.clear();
    for (auto &sd : side) order.insert(order.end(), sd.begin(), sd.end());
    dg.n_unit = (uint8_t)side[0].size();
    dg.n_step = (uint8_t)side[1].size();
    dg.n_serial = 0;
    dg.n_mb = (uint8_t)gsh.mbits.size();
    dg.n_nb = (uint8_t)gsh.nbits.size();
    dg.n_bb = (uint8_t)gsh.bbits.size();
    // column blocks of 16 per tile: as many as the n range fills (n >= 4
    // bits) in own launches; one inside workgroups and the persistent
    // executors, whose kernels are compiled for that form only
    dg.rls = (uint8_t)(is_small || persistent ? 1 : (dg.n_nb >= 6 ? 4 : (dg.n_nb == 5 ? 2 : 1)));
    const uint64_t tn = 16ull * dg.rls;
    const uint64_t mt = ((1ull << dg.n_mb) + kMmTM - 1) / kMmTM;
    const uint64_t nt = ((1ull << dg.n_nb) + tn - 1) / tn;
    const uint64_t tiles = (1ull << dg.n_bb) * mt * nt;
    if (tiles > 0xFFFFFFFFull) return set_err(QTN_ERANGE, "matrix-form group too large");
    dg.n_units = (uint32_t)tiles;
    // the tile's rows and columns: union bits of the lowest 6 m (n) bits
    dg.gtab = (int32_t)s.stab.size();
    for (int pass = 0; pass < 2; pass++) {
      const std::vector<int> &bl = pass == 0 ? gsh.mbits : gsh.nbits;
      const int lim = pass == 0 ? kMmTM : kMmTN;
      for (int r = 0; r < lim; r++) {
        uint32_t I = 0;
        for (int j = 0; j < (int)bl.size() && j < 6; j++) I |= (uint32_t)((r >> j) & 1) << bl[j];
        s.stab.push_back((int32_t)I);
      }
    }
  } else if (cell) {
    dg.variant = kVarCell;
    dg.rls = (uint8_t)cb;
    dg.sl = (uint8_t)std::max(0, G.L - 6);
    dg.lk = (uint8_t)(6 - std::min(G.L, 6));
    // operands by the first summed bit above the lanes they hold (the
    // serial cells are summed in that order, each operand multiplying
    // only the cells still open at its level): bit 6, then bit 7, then
    // none; without serial bits every operand is at the first level
    std::vector<int> lev(G.ops.size(), 0);
    for (size_t k = 0; k < G.ops.size(); k++) {
      const uint32_t m = G.ops[k].mask;
      lev[k] = G.L <= 6 ? 0 : ((m >> 6) & 1u) ? 0 : (G.L > 7 && ((m >> 7) & 1u)) ? 1 : 2;
      cls[k] = lev[k] < 2 ? kClsStep : kClsUnit;
    }
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return lev[a] < lev[b]; });
    int n0 = 0, n1 = 0;
    for (int k : order) {
      n0 += lev[k] == 0 ? 1 : 0;
      n1 += lev[k] == 1 ? 1 : 0;
    }
    dg.n_step = (uint8_t)n0;
    dg.n_serial = (uint8_t)n1;
    dg.n_units = 1u << (G.w - low - rb);
  } else if (stream) {
    dg.variant = kVarStream;
    dg.rls = (uint8_t)rls;
    dg.sl = (uint8_t)sl;
    dg.lk = (uint8_t)(6 - rls);
    // lane-kept bits: the lowest kept bits, so that the lanes' output
    // writes are contiguous (positions past the union, in narrow
    // groups, give idle lanes).  Choosing instead the bits the large
    // operands lack, so that lanes share operand elements, measured
    // slower.
    for (int j = 0; j < dg.lk; j++) dg.lkpos[j] = (uint8_t)(G.L + j);
    uint32_t lane_kept = 0;
    for (int j = 0; j < dg.lk; j++)
      if (dg.lkpos[j] < 32) lane_kept |= 1u << dg.lkpos[j];
    const uint32_t serial_bits = ((1u << G.L) - 1u) & ~((1u << (1 + rls)) - 1u);
    const uint32_t lane_bits = (((1u << rls) - 1u) << 1) | lane_kept;
    for (size_t k = 0; k < G.ops.size(); k++) {
      const Operand &o = G.ops[k];
      if (o.level >= 1 + rls)
        cls[k] = (o.mask & lane_bits) ? kClsSerial : kClsUniform;
      else
        cls[k] = (o.mask & serial_bits) ? kClsStep : kClsUnit;
    }
    // step-class operands with bit 0 first: they fill the unrolled slots
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
      if (cls[a] != cls[b]) return cls[a] < cls[b];
      if (cls[a] == kClsStep) return (G.ops[a].mask & 1u) > (G.ops[b].mask & 1u);
      return false;
    });
    int nu = 0, ns = 0, nun = 0, nse = 0, ns0 = 0;
    for (int k : order) {
      if (cls[k] == kClsUnit) nu++;
      else if (cls[k] == kClsStep) {
        ns++;
        ns0 += (G.ops[k].mask & 1u) ? 1 : 0;
      }
      else if (cls[k] == kClsUniform) nun++;
      else nse++;
    }
    dg.n_unit = (uint8_t)nu;
    dg.n_step = (uint8_t)ns;
    dg.n_step0 = (uint8_t)ns0;
    dg.n_serial = (uint8_t)(nun + nse);
    dg.level_end[0] = (uint8_t)nun;
    const int kept_lanes = G.L + dg.lk;
    dg.n_units = G.w > kept_lanes ? 1u << (G.w - kept_lanes) : 1u;
  } else {
    dg.variant = kVarGeneric;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return G.ops[a].level < G.ops[b].level; });
    int cum = 0;
    for (int l = 0; l < kMaxLevels; l++) {
      if (l < G.L) cum += per_level[l];
      dg.level_end[l] = (uint8_t)cum;
    }
    const int bits = kGenRegBits + 6;
    dg.n_units = G.w > bits ? 1u << (G.w - bits) : 1u;
  }
  if (mfma) {
    // matrix form: m bits, then n bits, then batch bits
    uint8_t up[32];
    std::memset(up, 0, sizeof up);
    int j = 0;
    for (int q : gsh.mbits) up[j++] = (uint8_t)q;
    for (int q : gsh.nbits) up[j++] = (uint8_t)q;
    for (int q : gsh.bbits) up[j++] = (uint8_t)q;
    dg.n_ubits = 0;
    s.uperm.insert(s.uperm.end(), up, up + 32);
  } else {
    // wave-unit bits, those that large operands lack first (their data
    // is then reused by neighbouring units of the same block and XCD);
    // cells: the first rb of that order are the register bits (each
    // value of an operand lacking them serves several cells), first in
    // the table
    const int start = stream ? G.L : (cell ? low : kGenRegBits + 6);
    std::vector<std::pair<double, int>> sc;
    for (int b = start; b < G.w; b++) {
      bool lane = false;
      for (int j = 0; stream && j < dg.lk; j++) lane |= dg.lkpos[j] == b;
      if (lane) continue;
      double miss = 0;
      for (const Operand &o : G.ops)
        if (pl.tensors[o.tensor].gate < 0 && !((o.mask >> b) & 1u))
          miss += std::ldexp(1.0, (int)pl.tensors[o.tensor].vars.size());
      sc.push_back({-miss, b});
    }
    std::stable_sort(sc.begin(), sc.end());
    std::vector<int> regs;
    if (cell) {
      // register bits: one at a time, the kept bit that adds the fewest
      // loads (an operand is loaded once per distinct value of the cell
      // bits it holds), ties to the earlier bit of the order above
      // cell bits held so far: the serial bits still open at the
      // operand's level
      std::vector<uint32_t> held(G.ops.size(), 0);
      for (size_t k = 0; k < G.ops.size(); k++) {
        const uint32_t m = G.ops[k].mask;
        const int lv = G.L <= 6 ? 0 : ((m >> 6) & 1u) ? 0 : (G.L > 7 && ((m >> 7) & 1u)) ? 1 : 2;
        for (int t = lv; t < dg.sl; t++) held[k] += (m >> (6 + t)) & 1u;
      }
      for (int j = 0; j < rb; j++) {
        size_t bi = 0;
        double best_cost = -1;
        for (size_t q = 0; q < sc.size(); q++) {
          double cost = 0;
          for (size_t k = 0; k < G.ops.size(); k++)
            cost += std::ldexp(1.0, (int)held[k] + (int)((G.ops[k].mask >> sc[q].second) & 1u));
          if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            bi = q;
          }
        }
        for (size_t k = 0; k < G.ops.size(); k++) held[k] += (G.ops[k].mask >> sc[bi].second) & 1u;
        regs.push_back(sc[bi].second);
        sc.erase(sc.begin() + bi);
      }
      // with serial bits, the operands without them that hold no unit
      // bit go first: their product over the register cells is formed
      // once per angle set and reused by every unit (without serial
      // bits it would span every cell and cost more registers than it
      // saves)
      if (dg.sl > 0) {
        uint32_t unit_mask = 0;
        for (auto &q : sc) unit_mask |= 1u << q.second;
        const int last0 = dg.n_step + (dg.sl == 2 ? dg.n_serial : 0);
        std::stable_partition(order.begin() + last0, order.end(),
                              [&](int k) { return (G.ops[k].mask & unit_mask) == 0; });
        int nfix = 0;
        for (size_t i = last0; i < order.size(); i++)
          nfix += (G.ops[order[i]].mask & unit_mask) == 0 ? 1 : 0;
        dg.n_step0 = (uint8_t)nfix;
      } else {
        // without serial bits, the operands holding only lane bits go
        // first: their product, one value per lane, is formed once per
        // angle set and multiplies the cells once per unit
        std::stable_partition(order.begin(), order.end(),
                              [&](int k) { return (G.ops[k].mask & ~63u) == 0; });
        int nfix = 0;
        for (int k : order) nfix += (G.ops[k].mask & ~63u) == 0 ? 1 : 0;
        dg.n_step0 = (uint8_t)nfix;
      }
      // the cell mapping forms an operand's unit offset from its runs
      // over the unit bits; past kCellURuns of them, ascending order
      // (at most one run per two unit bits)
      int worst = 0;
      for (size_t t = 0; t <= G.ops.size(); t++) {
        const uint32_t mask = t < G.ops.size() ? G.ops[t].mask : ~((1u << G.L) - 1u);
        int runs = 0, prev = -2;
        for (size_t j = 0; j < sc.size(); j++) {
          const int q = sc[j].second;
          if (!((mask >> q) & 1u)) {
            prev = -2;
            continue;
          }
          const int rank = __builtin_popcount(mask & ((1u << q) - 1u));
          if (rank != prev + 1) runs++;
          prev = rank;
        }
        worst = std::max(worst, runs);
      }
      if (worst > kCellURuns)
        std::sort(sc.begin(), sc.end(),
                  [](const std::pair<double, int> &a, const std::pair<double, int> &b) {
                    return a.second < b.second;
                  });
    }
    uint8_t up[32];
    std::memset(up, 0, sizeof up);
    const int first = cell ? rb : 0;
    for (int j = 0; j < first; j++) up[j] = (uint8_t)regs[j];
    for (size_t j = 0; j < sc.size(); j++) up[first + j] = (uint8_t)sc[j].second;
    dg.n_ubits = (uint8_t)sc.size();
    s.uperm.insert(s.uperm.end(), up, up + 32);
  }
  // union bit of cell bit j: kept bits, then serial bits (serial cell bit
  // rb + t is union bit 6 + sl - 1 - t, bit 6 the highest, summed first)
  auto cell_bit = [&](int j) {
    const uint8_t *rp = s.uperm.data() + s.uperm.size() - 32;
    return j < rb ? (int)rp[j] : 6 + dg.sl - 1 - (j - rb);
  };
  if (cell) {
    // Operand order.  Every point multiplies all operands, but an operand
    // without cell bits is one value per lane: without serial bits those form
    // a product of their own, which meets the cells once.  Of the others, the
    // one with the most cell bits comes first (its values become the cells,
    // none copied) and the one with the fewest last (it takes that product).
    auto held = [&](int k) {
      int n = 0;
      for (int j = 0; j < cb; j++) n += (G.ops[k].mask >> cell_bit(j)) & 1u;
      return n;
    };
    auto most_first = [&](int x, int y) { return held(x) > held(y); };
    if (dg.in_order) {
      // the plan's order: of the operands without cell bits, those that come
      // before every other one are multiplied once per lane
      if (dg.sl == 0) {
        const auto first = order.begin() + dg.n_step0;
        dg.n_serial = (uint8_t)(std::find_if(first, order.end(), [&](int k) { return held(k) > 0; }) - first);
      }
    } else if (dg.sl == 0) {
      const auto first = order.begin() + dg.n_step0;
      const auto full = std::stable_partition(first, order.end(), [&](int k) { return held(k) == 0; });
      dg.n_serial = (uint8_t)(full - first);
      std::stable_sort(full, order.end(), most_first);
    } else {
      std::stable_sort(order.begin(), order.begin() + dg.n_step, most_first);
    }
  }
  // A cell group's table of a tensor holding the union bits of mask.
  auto cell_table = [&](uint32_t mask) -> int {
    const uint8_t *up = s.uperm.data() + s.uperm.size() - 32 + rb;
    uint16_t ur[kCellURuns];
    std::memset(ur, 0, sizeof ur);
    auto place = [&](int q) { return __builtin_popcount(mask & ((1u << q) - 1u)); };
    int nur = 0;
    for (int j = 0; j < dg.n_ubits;) {
      const int q = up[j];
      if (!((mask >> q) & 1u)) {
        j++;
        continue;
      }
      const int dst = place(q);
      int len = 1;
      while (j + len < dg.n_ubits && ((mask >> up[j + len]) & 1u) && place(up[j + len]) == dst + len)
        len++;
      if (nur == kCellURuns) return set_err(QTN_ERANGE, "cell mapping: unit runs");
      ur[nur++] = (uint16_t)(j | (len << 5) | (dst << 11));
      j += len;
    }
    dg.n_unit = (uint8_t)std::max<int>(dg.n_unit, nur);
    for (int w = 0; w < kCellURuns / 2; w++)
      s.stab.push_back((int32_t)((uint32_t)ur[2 * w] | ((uint32_t)ur[2 * w + 1] << 16)));
    uint32_t cm = 0;
    for (int j = 0; j < cb; j++) {
      const int q = cell_bit(j);
      if ((mask >> q) & 1u) cm |= (uint32_t)place(q) << (5 * j) | 1u << (20 + j);
    }
    s.stab.push_back((int32_t)cm);
    return QTN_OK;
  };
  if (cell) {
    // the output holds every kept bit
    dg.gtab = (int32_t)s.stab.size();
    const int rc = cell_table(~((1u << G.L) - 1u));
    if (rc) return rc;
  }
  for (int k : order) {
    const Operand &o = G.ops[k];
    const Tensor &t = pl.tensors[o.tensor];
    DevOp d;
    std::memset(&d, 0, sizeof d);
    if (t.gate >= 0) {
      // gate operands read the table of the group's own precision
      d.off = env.table[G.prec] +
              gate_offset((*env.gates)[t.gate], t.transposed, env.p, env.slice) * es(G.prec);
      d.sstride = env.table_sstride[G.prec];
      d.dt = (uint8_t)G.prec;
    } else {
      d.off = env.arena + t.offset;
      d.sstride = env.arena_sstride;
      d.dt = (uint8_t)t.prec;
    }
    d.mask = o.mask;
    d.level = (uint8_t)o.level;
    uint8_t rs[32], rl[32], rd[32];
    const int nr = mask_runs(o.mask, rs, rl, rd);
    if (nr > kOpRuns) return set_err(QTN_ERANGE, "operand index set too fragmented");
    d.nruns = (uint8_t)nr;
    for (int r = 0; r < nr; r++)
      d.run[r] = (uint16_t)(rs[r] | (rl[r] << 5) | (rd[r] << 11));
    d.cls = (uint8_t)cls[k];
    d.stab = -1;
    if (stream && cls[k] != kClsUnit) {
      d.stab = (int32_t)s.stab.size();
      for (uint32_t st = 0; st < (1u << dg.sl); st++)
        s.stab.push_back((int32_t)pext32(st << (1 + dg.rls), o.mask));
    }
    if (cell) {
      d.stab = (int32_t)s.stab.size();
      const int rc = cell_table(o.mask);
      if (rc) return rc;
    }
    if (mfma) {
      // the operand's element offsets of the tile's rows (side A) or
      // columns (side B), then of the summed indices
      d.stab = (int32_t)s.stab.size();
      const int sd = gsh.role[k];
      const int lim = sd == 0 ? kMmTM : kMmTN;
      const int32_t *rows = s.stab.data() + dg.gtab + (sd == 0 ? 0 : kMmTM);
      std::vector<int32_t> tab(lim + (1 << G.L));
      for (int r = 0; r < lim; r++) tab[r] = (int32_t)pext32((uint32_t)rows[r], o.mask);
      for (int kk = 0; kk < (1 << G.L); kk++) tab[lim + kk] = (int32_t)pext32((uint32_t)kk, o.mask);
      s.stab.insert(s.stab.end(), tab.begin(), tab.end());
    }
    if (d.dt != dg.prec) dg.cvt = 1;
    s.ops.push_back(d);
  }
  double gb = in_bytes + es(G.prec) * std::ldexp(1.0, G.w - G.L), gf = 0;
  for (int l = 0; l < G.L; l++) {
    int factors = per_level[l] + (l > 0 ? 1 : 0);
    gf += std::ldexp(1.0, G.w - l) * 6.0 * std::max(0, factors - 1) +
          std::ldexp(1.0, G.w - l - 1) * 2.0;
  }
  *dg_out = dg;
  *bytes_out = gb;
  *flops_out = gf;
  return QTN_OK;
}

// What a light cone's segment programs address, for angle set 0 and in bytes
// from the data base, with the bytes between angle sets.
struct ProgBases {
  int64_t table, table_stride, arena, arena_stride, scalar, scalar_stride;
  int table_elems;
};

// Units of a small group in a segment program, and the items it is cut into.
int prog_units(const DevGroup &G) { return 1 << std::max(0, G.w - 6 - prog_reg_bits(G.w, G.L)); }
int prog_pieces(const DevGroup &G) { return std::min(prog_units(G), kProgPieces); }

// End of the page that starts at group b of [b, g1); adds its operands to
// n_ops and the most words it takes to words.
int page_end(const Schedule &s, int b, int g1, int *n_ops, size_t *words) {
  int e = b, w = kPageHeader + 8;
  while (e < g1) {
    const int more = 4 * s.groups[e].n_ops + 4 * prog_pieces(s.groups[e]) + 1;
    if (e > b && w + more > kPageWords) break;
    w += more;
    *n_ops += s.groups[e].n_ops;
    e++;
  }
  *words += (size_t)w;
  return e;
}

// Compiles groups [g0, g1) of the schedule (one light cone's, in execution
// order) into a segment program (prog); false where a group does not fit the
// form (union wider than 16 bits, more than 64 operands, mixed arithmetic, a
// gate table too long for LDS): such a segment runs group by group.
//
// Groups of a page are put on levels: after the group that makes an operand,
// and, as the arena reuses memory along the execution order, after every
// group that reads or writes an arena region the group overwrites.  An
// intermediate made and read within the page takes LDS where it fits, for the
// levels it lives on, and then has no part in the arena's hazards.
bool compile_segment(const Schedule &s, int g0, int g1, const ProgBases &pb,
                     std::vector<uint32_t> &prog) {
  if (g1 <= g0) return false;
  const int prec = s.groups[g0].prec;
  const int64_t es = prec == 1 ? 8 : 16;
  if (pb.table < 0 || pb.table_elems > kProgTable) return false;
  const int64_t most = (int64_t)1 << 30;
  for (int g = g0; g < g1; g++) {
    const DevGroup &G = s.groups[g];
    if (G.prec != prec || G.w > kProgMaxWidth || G.n_ops < 1 || G.n_ops > kProgMaxOps) return false;
    const bool scalar = G.w == G.L;
    if (scalar ? (G.out_off - pb.scalar) / es >= most : (G.out_off - pb.arena) / 256 >= most) return false;
    for (int k = 0; k < G.n_ops; k++) {
      const DevOp &o = s.ops[G.op_begin + k];
      const bool gate = o.off >= pb.table && o.off < pb.table + pb.table_elems * es;
      if (!gate && (o.off < pb.arena || (o.off - pb.arena) % 256 || (o.off - pb.arena) / 256 >= most))
        return false;
    }
  }
  size_t prev_at = 0;
  bool first = true;
  for (int b = g0; b < g1;) {
    // groups [b, e) make the page
    int n_ops = 0;
    size_t words = 0;
    const int e = page_end(s, b, g1, &n_ops, &words);
    const int n = e - b;
    // who makes an operand: the last group of the page to write its address
    const int op0 = s.groups[b].op_begin;  // the page's operands are [op0, op0 + n_ops)
    std::vector<int> maker(n_ops, -1), reader(n, -1);
    for (int i = 0; i < n; i++) {
      const DevGroup &G = s.groups[b + i];
      for (int k = 0; k < G.n_ops; k++) {
        const int64_t off = s.ops[G.op_begin + k].off;
        if (off < pb.arena) continue;
        for (int q = i - 1; q >= 0; q--)
          if (s.groups[b + q].out_off == off && s.groups[b + q].w != s.groups[b + q].L) {
            maker[G.op_begin - op0 + k] = q;
            reader[q] = i;
            break;
          }
      }
    }
    auto out_bytes = [&](int i) { return es << (s.groups[b + i].w - s.groups[b + i].L); };
    std::vector<char> lds(n);
    for (int i = 0; i < n; i++) lds[i] = reader[i] >= 0 && out_bytes(i) <= kProgPoolBytes;
    std::vector<int> level(n), where(n, -1);
    for (bool again = true; again;) {
      again = false;
      struct Use {
        int64_t lo, hi;
        int level;
        bool write;
      };
      std::vector<Use> uses;  // arena regions touched by the groups so far
      for (int i = 0; i < n; i++) {
        const DevGroup &G = s.groups[b + i];
        int lv = 0;
        for (int k = 0; k < G.n_ops; k++)
          if (maker[G.op_begin - op0 + k] >= 0) lv = std::max(lv, level[maker[G.op_begin - op0 + k]] + 1);
        const bool writes = G.w != G.L && !lds[i];
        const int64_t lo = G.out_off, hi = lo + out_bytes(i);
        if (writes)
          for (const Use &u : uses)
            if (u.lo < hi && lo < u.hi) lv = std::max(lv, u.level + 1);
        level[i] = lv;
        for (int k = 0; k < G.n_ops; k++) {
          const DevOp &o = s.ops[G.op_begin + k];
          if (o.off < pb.arena || (maker[G.op_begin - op0 + k] >= 0 && lds[maker[G.op_begin - op0 + k]])) continue;
          const int64_t sz = (o.dt == 1 ? 8ll : 16ll) << __builtin_popcount(o.mask);
          uses.push_back({o.off, o.off + sz, lv, false});
        }
        if (writes) uses.push_back({lo, hi, lv, true});
      }
      // LDS: first fit among the intermediates alive on the same levels
      struct Slot {
        int at, end, from, to;
      };
      std::vector<Slot> pool;
      for (int i = 0; i < n && !again; i++) {
        if (!lds[i]) continue;
        const int size = (int)((out_bytes(i) + 15) / 16 * 16), from = level[i], to = level[reader[i]];
        int at = 0;
        for (bool moved = true; moved;) {
          moved = false;
          for (const Slot &q : pool)
            if (q.from <= to && from <= q.to && q.at < at + size && at < q.end) {
              at = q.end;
              moved = true;
            }
        }
        if (at + size > kProgPoolBytes) {
          lds[i] = 0;
          again = true;
        } else {
          where[i] = at;
          pool.push_back({at, at + size, from, to});
        }
      }
    }
    // emit
    while (prog.size() % 4) prog.push_back(0);
    const size_t at = prog.size();
    if (!first) prog[prev_at + kPgNext] = (uint32_t)(at - prev_at);
    first = false;
    prev_at = at;
    prog.resize(at + kPageHeader + 4 * n_ops, 0);
    auto put64 = [&](int w, int64_t v) {
      prog[at + w] = (uint32_t)v;
      prog[at + w + 1] = (uint32_t)((uint64_t)v >> 32);
    };
    put64(kPgTableOff, pb.table);
    put64(kPgTableStride, pb.table_stride);
    put64(kPgArenaOff, pb.arena);
    put64(kPgArenaStride, pb.arena_stride);
    put64(kPgScalarOff, pb.scalar);
    put64(kPgScalarStride, pb.scalar_stride);
    prog[at + kPgPrec] = (uint32_t)prec;
    prog[at + kPgTable] = (uint32_t)pb.table_elems;
    std::vector<int> op_at(n);
    size_t w = at + kPageHeader;
    for (int i = 0, k0 = 0; i < n; i++) {
      const DevGroup &G = s.groups[b + i];
      op_at[i] = k0;
      k0 += G.n_ops;
      for (int k = 0; k < G.n_ops; k++) {
        const DevOp &o = s.ops[G.op_begin + k];
        uint32_t loc;
        if (o.off < pb.table + pb.table_elems * es)
          loc = kLocLds | (uint32_t)(kProgTableAt + (o.off - pb.table)) << 2;
        else if (maker[G.op_begin - op0 + k] >= 0 && lds[maker[G.op_begin - op0 + k]])
          loc = kLocLds | (uint32_t)(kProgPoolAt + where[maker[G.op_begin - op0 + k]]) << 2;
        else
          loc = (o.dt == prec ? kLocArena : kLocArenaX) | (uint32_t)((o.off - pb.arena) / 256) << 2;
        // move masks of the compress (Hacker's Delight 7-4) of a 16-bit mask
        uint32_t m = o.mask & 0xFFFFu, mk = ~m << 1, mv[4];
        for (int q = 0; q < 4; q++) {
          uint32_t mp = mk ^ (mk << 1);
          mp ^= mp << 2;
          mp ^= mp << 4;
          mp ^= mp << 8;
          mp ^= mp << 16;
          mv[q] = mp & m & 0xFFFFu;
          m = ((m ^ mv[q]) | (mv[q] >> (1 << q))) & 0xFFFFu;
          mk &= ~mp;
        }
        prog[w++] = loc;
        prog[w++] = mv[0] | mv[1] << 16;
        prog[w++] = mv[2] | mv[3] << 16;
        prog[w++] = o.mask;
      }
    }
    const int n_levels = 1 + *std::max_element(level.begin(), level.end());
    std::vector<int> by_level(n);
    for (int i = 0; i < n; i++) by_level[i] = i;
    // the costliest groups of a level first
    auto cost = [&](int i) { return (double)s.groups[b + i].n_ops * std::ldexp(1.0, s.groups[b + i].w); };
    std::stable_sort(by_level.begin(), by_level.end(), [&](int x, int y) {
      return level[x] != level[y] ? level[x] < level[y] : cost(x) > cost(y);
    });
    prog[at + kPgLevels] = (uint32_t)n_levels;
    prog[at + kPgItems] = (uint32_t)(prog.size() - at);
    std::vector<uint32_t> begin(n_levels + 1, 0);
    uint32_t item = 0;
    for (int i : by_level) {
      const DevGroup &G = s.groups[b + i];
      const int np = prog_pieces(G), per = prog_units(G) / np;
      uint32_t out;
      if (G.w == G.L) out = kLocScalar | (uint32_t)((G.out_off - pb.scalar) / es) << 2;
      else if (lds[i]) out = kLocLds | (uint32_t)(kProgPoolAt + where[i]) << 2;
      else out = kLocArena | (uint32_t)((G.out_off - pb.arena) / 256) << 2;
      for (int q = 0; q < np; q++, item++) {
        prog.push_back((uint32_t)G.w | (uint32_t)G.L << 5 | (uint32_t)G.n_ops << 9 |
                         (uint32_t)op_at[i] << 16);
        prog.push_back(out);
        prog.push_back((uint32_t)(q * per) | (uint32_t)per << 16);
        prog.push_back((uint32_t)prog_reg_bits(G.w, G.L));
      }
      begin[level[i] + 1] = item;
    }
    prog[at + kPgLevelAt] = (uint32_t)(prog.size() - at);
    prog.insert(prog.end(), begin.begin(), begin.end());
    while (prog.size() % 4) prog.push_back(0);
    prog[at + kPgWords] = (uint32_t)(prog.size() - at);
    b = e;
  }
  return true;
}

// Arithmetic of segment `range` when it runs as a program, else -1.
int prog_prec(const Schedule &s, int range) {
  const int4 r = s.ranges[range];
  return r.z >= 0 ? s.groups[r.x].prec : -1;
}

// Step launches of the light cones' task chains, where the rule takes them.
constexpr double kAloneMs = 3.5e-3;      // a launch of one tiny group
constexpr double kStepUnits = 4;         // units a wave takes once those are busy: 40 vertices,
                                         // mixed, 6.21 ms with 1, 5.94 with 4, 6.18 with 16
constexpr double kStepMaxUnits = 16384;  // most units a task
void plan_steps(Schedule &s) {
  double units = 0;
  int64_t n_tasks = 0, n_other = 0;
  size_t n_steps = 0;
  for (const auto &tk : s.cone_tasks) {
    n_steps = std::max(n_steps, tk.size());
    for (const Task &t : tk) {
      n_tasks++;
      if (t.kind == QTN_K_BLOCK) {
        if (s.ranges[t.index].z < 0) n_other++;
      } else {
        units += (double)s.groups[t.index].n_units * s.n_sets;
        if (!step_group(s.groups[t.index])) n_other++;
      }
    }
  }
  // Above the line the groups fill the chip by themselves, and the four
  // streams overlap the ends of launches of unlike light cones, which a step
  // makes wait for each other.  Four streams against step launches, by units
  // a task: 17 (20 vertices, depth 3) 281 us against 159; 469 (27 sets of a
  // 22-vertex one) 342 against 269; 1,479 (quartic, 24 vertices, depth 3) 2.46
  // ms against 1.38; 3,912 (40 vertices, mixed precision) 6.80 against 5.94;
  // 10,984 (4 sets of the 30-vertex depth-4 one) 13.64 against 13.58; 15,268 (9
  // sets of a 16-vertex one) 6.58 against 6.36; 21,968 (8 sets of the 30-vertex
  // one) 25.7 against 26.0; 87,871 (32 sets) 99.3 against 99.9, in complex64
  // 62.0 against 71.8.  A schedule that is mostly other mappings keeps its
  // streams.
  if (n_tasks == 0 || n_other * 8 > n_tasks || units > kStepMaxUnits * (double)n_tasks) return;
  s.steps.resize(n_steps);
  std::vector<std::vector<const Task *>> in_step(n_steps);
  for (const auto &tk : s.cone_tasks)
    for (size_t j = 0; j < tk.size(); j++) in_step[j].push_back(&tk[j]);
  for (size_t j = 0; j < n_steps; j++) {
    Schedule::Step &st = s.steps[j];
    st.first = (int)s.step_tasks.size();
    std::vector<std::pair<int, int>> wide;  // (-workgroups, group)
    // a workgroup sets up its tables before its first unit: once the step
    // fills the chip, several units share a set-up
    double step_units = 0;
    for (const Task *t : in_step[j])
      if (t->kind == QTN_K_WIDE) step_units += (double)s.groups[t->index].n_units * s.n_sets;
    const double per_wave = std::min(kStepUnits, step_units / kStepWaves);
    // A segment is one workgroup's chain and wants many waves; groups that
    // fill the chip want small workgroups, which start and end singly.  256,
    // 512 and 1,024 threads: 40 vertices, mixed, 5.95, 6.11 and 6.26 ms; 9 sets
    // of a 16-vertex depth-4 network 6.35, 6.73 and 6.77; 20 vertices, depth 3,
    // 195, 157 and 148 us.  The cost model's times say where a segment outlasts
    // the groups all the same (quartic graphs of 171, 228 and 284 vertices at
    // depth 3, complex64: 612, 499 and 491 us, 500, 393 and 357, 516, 413 and
    // 375; by those times 470, 354 and 376).
    double seg_ms = 0, wide_ms = 0;
    for (const Task *t : in_step[j])
      (t->kind == QTN_K_BLOCK ? seg_ms : wide_ms) = std::max(t->kind == QTN_K_BLOCK ? seg_ms : wide_ms, t->ms);
    st.threads = seg_ms > wide_ms ? 1024 : (step_units >= 2 * kStepWaves ? 256 : 512);
    for (const Task *tp : in_step[j]) {
      const Task &t = *tp;
      if (t.kind == QTN_K_BLOCK && s.ranges[t.index].z >= 0) {
        // segments first: each is one workgroup's chain
        s.step_tasks.push_back(make_int4(-1, st.blocks, s.n_sets, s.ranges[t.index].z));
        st.blocks += s.n_sets;
        st.lds = std::max(st.lds, (size_t)kProgLdsBytes);
      } else if (t.kind == QTN_K_WIDE && step_group(s.groups[t.index])) {
        wide.push_back({-step_blocks(s.groups[t.index], s.n_sets, per_wave, st.threads), t.index});
        st.lds = std::max(st.lds, step_lds(s.groups[t.index]));
      } else {
        st.single.push_back(t);
      }
    }
    std::stable_sort(wide.begin(), wide.end());
    for (auto &w : wide) {
      const int nb = -w.first;
      // a grid of whole rounds over the XCDs starts on one
      if (nb >= 64) st.blocks = (st.blocks + 7) & ~7;
      s.step_tasks.push_back(make_int4(w.second, st.blocks, nb, 0));
      st.blocks += nb;
    }
    st.n = (int)s.step_tasks.size() - st.first;
  }
}

// Workspace of a schedule with this many device descriptors, program words and
// step tasks, for n_sets angle sets.
Layout lay_out(const Schedule &s, size_t n_groups, size_t n_ops, size_t n_stab, size_t n_uperm,
               size_t n_prog, size_t n_step_tasks, int n_sets) {
  Layout l;
  l.off_res = 0;
  l.off_angles = align_up(8 * (size_t)(2 * s.n_cones + s.n_nets) * n_sets, 256);
  l.off_desc = align_up(l.off_angles + 8 * (size_t)s.n_angles * n_sets, 256);
  l.off_fills = l.off_desc;
  l.off_groups = align_up(l.off_fills + sizeof(FillDesc) * s.fills.size(), 256);
  l.off_ops = align_up(l.off_groups + sizeof(DevGroup) * n_groups, 256);
  l.off_stab = align_up(l.off_ops + sizeof(DevOp) * n_ops, 256);
  l.off_uperm = align_up(l.off_stab + sizeof(int32_t) * n_stab, 256);
  l.off_ranges = align_up(l.off_uperm + n_uperm, 256);
  l.off_prog = align_up(l.off_ranges + sizeof(int4) * s.ranges.size(), 256);
  l.off_csb = align_up(l.off_prog + sizeof(uint32_t) * (n_prog), 256);
  l.off_ncb = align_up(l.off_csb + sizeof(int) * s.csb.size(), 256);
  l.off_cns = align_up(l.off_ncb + sizeof(int) * s.ncb.size(), 256);
  l.off_step_tasks = align_up(l.off_cns + sizeof(int) * s.cns.size(), 256);
  l.off_items = align_up(l.off_step_tasks + sizeof(int4) * n_step_tasks, 256);
  l.off_steps = align_up(l.off_items + sizeof(int4) * s.items.size(), 256);
  l.off_item_task = align_up(l.off_steps + sizeof(int) * s.step_begin.size(), 256);
  l.off_task_next = align_up(l.off_item_task + sizeof(int) * s.item_task.size(), 256);
  l.off_task_first = align_up(l.off_task_next + sizeof(int) * s.task_next.size(), 256);
  l.off_task_need = align_up(l.off_task_first + sizeof(int) * s.task_first.size(), 256);
  l.off_queue = align_up(l.off_task_need + sizeof(int) * s.task_need.size(), 256);
  l.off_ctl = align_up(l.off_queue + sizeof(uint32_t) * s.items.size(), 256);
  l.off_data = align_up(l.off_ctl + sizeof(uint32_t) * s.n_ctl, 256);
  l.total = l.off_data + s.set_bytes * n_sets;
  return l;
}

// Most bytes that a schedule built like s needs for n_sets angle sets, of its
// two forms: in the plan's order every group has its descriptors on the
// device; otherwise its small groups may be in programs, and tasks in steps.
size_t form_bytes(const Schedule &s, bool in_order, int n_sets) {
  size_t words = 0, tasks = 0;
  if (!in_order) {
    for (int r = 0, n_ops = 0; r < s.singles_range0; r++)
      for (int g = s.ranges[r].x; g < s.ranges[r].y;) g = page_end(s, g, s.ranges[r].y, &n_ops, &words);
    for (auto &tk : s.cone_tasks) tasks += tk.size();
  }
  return lay_out(s, s.groups.size(), s.ops.size(), s.stab.size(), s.uperm.size(), words, tasks, n_sets).total;
}

// persistent: the schedule runs in a persistent executor (every group inside
// a workgroup, so no group takes the cell mapping).  size_only: s.total is
// wanted alone; the programs of single groups are left out and an upper bound
// of their words is counted.  in_order: no segment programs, and complex64
// groups multiply and sum in the plan's order.
int build_schedule(qtn_network *const *nets, int n, Schedule *S, const Force *force = nullptr,
                   int singleton_width = 0, int n_sets = 1, bool persistent = false,
                   bool size_only = false, bool in_order = false) {
  Schedule &s = *S;
  s = Schedule();
  s.serial = ++g_sched_serial;
  s.n_sets = n_sets;
  s.prec = nets[0]->precision;
  s.scalar_prec = s.prec == kPrecC64 ? 1 : 0;
  auto al = [](int64_t bytes) { return (bytes + 255) / 256 * 256; };
  auto es = [](int prec) { return prec == 1 ? (int64_t)8 : (int64_t)16; };
  // every offset below is in bytes from the data base
  int64_t data = 0;
  int n_scalars = 0;
  for (int i = 0; i < n; i++) {
    if (nets[i]->precision != s.prec) return set_err(QTN_EINVAL, "batched networks differ in precision");
    // one copy of every table, scalar slot and arena per angle set
    FillDesc f{(int64_t)s.n_angles, -1, -1, 0, 0, nets[i]->p, 0};
    const int64_t tab = gate_table_elems(nets[i]->p);
    if (s.prec != kPrecC64) {
      f.table128 = data;
      f.sstride128 = al(tab * 16);
      data += n_sets * f.sstride128;
    }
    if (s.prec != kPrecC128) {
      f.table64 = data;
      f.sstride64 = al(tab * 8);
      data += n_sets * f.sstride64;
    }
    s.fills.push_back(f);
    s.n_angles += 2 * nets[i]->p;
    for (auto &pl : nets[i]->plans) n_scalars += pl.n_scalars * pl.n_slices;
  }
  s.scalar_off = data;
  s.scalar_sstride = al(n_scalars * es(s.scalar_prec));
  data += n_sets * s.scalar_sstride;
  int scalar_next = 0;
  struct Job {
    int g0, g1;
    ProgBases pb;
    int range;  // its segment, or -(i + 1) for the i-th single group
    std::vector<uint32_t> prog;
  };
  std::vector<Job> jobs;  // segment programs to compile
  s.ncb.push_back(0);
  for (int i = 0; i < n; i++) {
    const qtn_network *net = nets[i];
    const int64_t table[2] = {s.fills[i].table128, s.fills[i].table64};
    const int64_t table_sstride[2] = {s.fills[i].sstride128, s.fills[i].sstride64};
    for (size_t c = 0; c < net->plans.size(); c++) {
      const ConePlan &pl = net->plans[c];
      const std::vector<Gate> &gates = pl.gates.empty() ? net->cones[c].gates : pl.gates;
      const int64_t arena = data, arena_sstride = al(pl.arena_bytes);
      data += n_sets * arena_sstride;
      s.csb.push_back(scalar_next);
      s.cns.push_back(pl.n_slices);
      // hybrid executor (executor 5): a cone with a bucket wider than the
      // network's hybrid width runs by per-group launches
      const bool heavy = persistent && net->executor == 5 && pl.max_width > net->hybrid_width;
      // segments run as programs unless the network asks for one mapping
      const bool programs = !in_order && (net->variant == 0 || net->variant == 4);
      const int tab_prec = s.prec == kPrecC64 ? 1 : 0;
      const ProgBases pb = {table[tab_prec], table_sstride[tab_prec], arena, arena_sstride,
                            s.scalar_off, s.scalar_sstride, (int)gate_table_elems(net->p)};
      s.cone_heavy.push_back(heavy ? 1 : 0);
      std::vector<Task> tasks;
      int open_begin = -1;
      double seg_bytes = 0, seg_flops = 0, seg_ms = 0;
      auto close_segment = [&](int end) {
        if (open_begin < 0) return;
        if (programs) jobs.push_back({open_begin, end, pb, (int)s.ranges.size(), {}});
        s.ranges.push_back(make_int4(open_begin, end, -1, 0));
        tasks.push_back({QTN_K_BLOCK, (int)s.ranges.size() - 1, 0, 0, seg_bytes, seg_flops,
                         seg_ms < 0 ? -1 : seg_ms + kAloneMs});
        open_begin = -1;
        seg_bytes = seg_flops = seg_ms = 0;
      };
      // index slicing: the groups run once per slice, in order, on the one
      // arena; slice k's scalars take slots k * n_scalars onwards
      for (int slice = 0; slice < pl.n_slices; slice++)
      for (int gi : pl.exec_order) {
        const Group &G = pl.groups[gi];
        if (G.ops.size() > 255) return set_err(QTN_ERANGE, "bucket with more than 255 tensors");
        if (G.out_tensor < 0 && G.prec != s.scalar_prec)
          return set_err(QTN_EINVAL, "scalar group precision differs from the scalar slots");
        GroupEnv env;
        env.out_off = G.out_tensor >= 0
                          ? arena + pl.tensors[G.out_tensor].offset
                          : s.scalar_off + (int64_t)(scalar_next + slice * pl.n_scalars + G.scalar_slot) *
                                               es(s.scalar_prec);
        env.out_sstride = G.out_tensor >= 0 ? arena_sstride : s.scalar_sstride;
        env.arena = arena;
        env.arena_sstride = arena_sstride;
        for (int q = 0; q < 2; q++) {
          env.table[q] = table[q];
          env.table_sstride[q] = table_sstride[q];
        }
        env.gates = &gates;
        env.slice = (uint32_t)slice;
        env.p = net->p;
        // the mapping requested (network config, tuned pick or a tuning
        // candidate); 0 leaves it to the width rule
        env.var_req = net->variant;
        env.rls_req = net->lane_sum_bits;
        if (G.pick_variant > 0) {
          env.var_req = G.pick_variant;
          if (G.pick_rls >= 0) env.rls_req = G.pick_rls;
        }
        const bool is_small = force && force->place >= 0
                                  ? force->place == 0
                                  : (G.pick_place >= 0 ? G.pick_place == 0 : G.small);
        if (force) {
          env.var_req = force->variant;
          env.rls_req = force->rls;
        }
        env.is_small = is_small;
        env.persistent = persistent && !heavy;
        if (!force && env.persistent && G.pick_variant == 4 && G.w <= kNoCellWidth) env.var_req = 1;
        env.in_order = in_order;
        DevGroup dg;
        double gb = 0, gf = 0;
        s.stab_at.push_back(s.stab.size());
        const int rc = describe_group(G, pl, env, s, &dg, &gb, &gf);
        if (rc) return rc;
        const int gid = (int)s.groups.size();
        s.groups.push_back(dg);
        s.group_cone.push_back(s.n_cones);
        s.group_index.push_back(gi);
        if (singleton_width > 0 && G.w <= singleton_width) {
          s.singles.push_back(gid);
          if (size_only) s.prog_more += kPageHeader + 12 + 4 * dg.n_ops + 4 * kProgPieces;
          if (programs && !size_only) jobs.push_back({gid, gid + 1, pb, -(int)s.singles.size(), {}});
        }
        if (is_small) {
          if (open_begin < 0) open_begin = gid;
          seg_bytes += gb;
          seg_flops += gf;
          seg_ms = G.pred_ms < 0 || seg_ms < 0 ? -1 : seg_ms + std::max(0.0, G.pred_ms - kAloneMs);
        } else {
          close_segment(gid);
          tasks.push_back({QTN_K_WIDE, gid, dg.n_units, dg.variant, gb, gf, G.pred_ms});
        }
      }
      close_segment((int)s.groups.size());
      scalar_next += pl.n_scalars * pl.n_slices;
      s.cone_tasks.push_back(std::move(tasks));
      s.n_cones++;
    }
    s.ncb.push_back(s.n_cones);
  }
  s.csb.push_back(scalar_next);
  std::vector<int> single_prog(s.singles.size(), -1);
  auto compile = [&](int q) {
    if (!compile_segment(s, jobs[q].g0, jobs[q].g1, jobs[q].pb, jobs[q].prog)) jobs[q].prog.clear();
  };
  // about 20 us a segment: threads pay off from a few dozen
  if (jobs.size() >= 64)
    parallel_for((int)jobs.size(), compile);
  else
    for (int q = 0; q < (int)jobs.size(); q++) compile(q);
  for (const Job &j : jobs) {
    if (j.prog.empty()) continue;
    (j.range >= 0 ? s.ranges[j.range].z : single_prog[-j.range - 1]) = (int)s.prog.size();
    s.prog.insert(s.prog.end(), j.prog.begin(), j.prog.end());
  }
  // the first n_cones ranges are the leading small segments (possibly empty)
  std::vector<int4> lead(s.n_cones, make_int4(0, 0, -1, 0));
  for (int c = 0; c < s.n_cones; c++) {
    auto &tk = s.cone_tasks[c];
    if (!tk.empty() && tk[0].kind == QTN_K_BLOCK) {
      lead[c] = s.ranges[tk[0].index];
      s.init_bytes += tk[0].bytes;
      s.init_flops += tk[0].flops;
      tk.erase(tk.begin());
    }
  }
  for (auto &tk : s.cone_tasks)
    for (auto &t : tk)
      if (t.kind == QTN_K_BLOCK) t.index += s.n_cones;
  s.ranges.insert(s.ranges.begin(), lead.begin(), lead.end());
  for (int c = 0, none = 1; c < s.n_cones; c++) {
    if (lead[c].y <= lead[c].x) continue;
    const int pr = prog_prec(s, c);
    if (none) s.lead_prec = pr;
    else if (pr != s.lead_prec) s.lead_prec = -1;
    none = 0;
  }
  s.singles_range0 = (int)s.ranges.size();
  for (size_t i = 0; i < s.singles.size(); i++)
    s.ranges.push_back(make_int4(s.singles[i], s.singles[i] + 1, single_prog[i], 0));
  for (int g : s.singles) s.ranges.push_back(make_int4(g, g + 1, -1, 0));
  s.n_nets = n;
  // persistent work items: the j-th task of every cone forms step j (leading
  // segment first); inside a step the costlier cones come first.  The
  // lockstep executor runs the steps between grid barriers; the dataflow
  // executor takes items in the same order and waits only for the previous
  // task of the item's own cone.
  {
    std::vector<int> corder(s.n_cones);
    std::vector<double> ccost(s.n_cones, 0);
    for (int c = 0; c < s.n_cones; c++) {
      corder[c] = c;
      for (auto &t : s.cone_tasks[c]) ccost[c] += t.bytes;
    }
    std::stable_sort(corder.begin(), corder.end(), [&](int a, int b) { return ccost[a] > ccost[b]; });
    std::vector<std::vector<int4>> per_step;
    std::vector<std::vector<int>> per_step_task;
    for (int cn : corder) {
      // a heavy cone runs by launches after the persistent kernel; its
      // leading segment, which needs nothing, is a first-step item
      const bool heavy = s.cone_heavy[cn] != 0;
      int j = 0, prev = -1;
      auto put = [&](const int4 &it, int task) {
        if ((int)per_step.size() <= j) {
          per_step.resize(j + 1);
          per_step_task.resize(j + 1);
        }
        per_step[j].push_back(it);
        per_step_task[j].push_back(task);
      };
      auto new_task = [&]() {
        s.task_dep.push_back(prev);
        s.task_need.push_back(0);
        prev = (int)s.task_dep.size() - 1;
        return prev;
      };
      if (lead[cn].y > lead[cn].x) {
        const int tk = new_task();
        put(make_int4(lead[cn].x, lead[cn].y, lead[cn].z, 0), tk);
        s.task_need[tk]++;
        j++;
      }
      if (heavy) continue;
      for (const Task &t : s.cone_tasks[cn]) {
        const int tk = new_task();
        if (t.kind == QTN_K_BLOCK) {
          const int4 r = s.ranges[t.index];
          put(make_int4(r.x, r.y, r.z, 0), tk);
          s.task_need[tk]++;
        } else {
          const uint32_t nu = t.n_units;
          // at least four passes of the block's waves per item
          uint32_t chunk = std::max<uint32_t>(16u, nu / 1024u);
          for (uint32_t u = 0; u < nu; u += chunk) {
            put(make_int4(t.index, -1, (int)u, (int)std::min(nu, u + chunk)), tk);
            s.task_need[tk]++;
          }
        }
        j++;
      }
    }
    s.step_begin.push_back(0);
    for (size_t j = 0; j < per_step.size(); j++) {
      s.items.insert(s.items.end(), per_step[j].begin(), per_step[j].end());
      s.item_task.insert(s.item_task.end(), per_step_task[j].begin(), per_step_task[j].end());
      s.step_begin.push_back((int)s.items.size());
    }
    s.n_steps = (int)per_step.size();
    s.n_tasks = (int)s.task_dep.size();
    s.n_ctl = 4 + std::max(s.n_steps, s.n_tasks);
    // ready-queue tables: a task's items are contiguous (one cone's chunks of
    // one step); the first step holds the first task of every cone
    s.task_next.assign(s.n_tasks, -1);
    for (int t = 1; t < s.n_tasks; t++)
      if (s.task_dep[t] >= 0) s.task_next[s.task_dep[t]] = t;
    s.task_first.assign(s.n_tasks, -1);
    for (int i = (int)s.item_task.size() - 1; i >= 0; i--) s.task_first[s.item_task[i]] = i;
    s.n_init = s.n_steps > 0 ? s.step_begin[1] : 0;
  }
  // (the cell kernels of a step have no form in the plan's order)
  if (!force && !persistent && !in_order && nets[0]->executor == 0) plan_steps(s);
  s.bytes[QTN_K_BLOCK] = s.init_bytes;
  s.flops[QTN_K_BLOCK] = s.init_flops;
  // a wide launch walks the units of every set in one flat 31-bit index
  for (const DevGroup &g : s.groups)
    if ((uint64_t)g.n_units * (uint64_t)s.n_sets > 0x7FFFFFFFull)
      return set_err(QTN_ERANGE, "too many units over the angle sets for one launch");
  for (auto &tk : s.cone_tasks)
    for (auto &t : tk) {
      s.bytes[t.kind] += t.bytes;
      s.flops[t.kind] += t.flops;
    }

  // device descriptors of the groups that kernels read one by one
  std::vector<DevGroup> dev_groups;
  std::vector<DevOp> dev_ops;
  std::vector<int32_t> dev_stab;
  std::vector<uint8_t> dev_uperm;
  size_t n_groups = s.groups.size(), n_ops = s.ops.size(), n_stab = s.stab.size(),
         n_uperm = s.uperm.size();
  if (!size_only) {
    const size_t ng = s.groups.size();
    s.stab_at.push_back(s.stab.size());
    s.dev_group.assign(ng, 0);
    for (int r = 0; r < s.singles_range0; r++)
      if (s.ranges[r].z >= 0) std::fill(&s.dev_group[s.ranges[r].x], &s.dev_group[0] + s.ranges[r].y, -1);
    for (size_t g = 0; g < ng; g++) {
      if (s.dev_group[g] < 0) continue;
      s.dev_group[g] = (int)dev_groups.size();
      DevGroup G = s.groups[g];
      const int32_t shift = (int32_t)s.stab_at[g] - (int32_t)dev_stab.size();
      const int32_t first = G.op_begin;
      G.op_begin = (int32_t)dev_ops.size();
      if (G.variant == kVarMfma || G.variant == kVarCell) G.gtab -= shift;
      for (int k = 0; k < G.n_ops; k++) {
        DevOp o = s.ops[first + k];
        if (o.stab >= 0) o.stab -= shift;
        dev_ops.push_back(o);
      }
      dev_groups.push_back(G);
      dev_stab.insert(dev_stab.end(), s.stab.begin() + s.stab_at[g], s.stab.begin() + s.stab_at[g + 1]);
      dev_uperm.insert(dev_uperm.end(), s.uperm.begin() + 32 * g, s.uperm.begin() + 32 * (g + 1));
    }
  }
  if (!size_only) {
    n_groups = dev_groups.size();
    n_ops = dev_ops.size();
    n_stab = dev_stab.size();
    n_uperm = dev_uperm.size();
  }
  auto on_device = [&](int4 r) {  // a segment or work item with device group numbers
    const bool chunk = r.y < 0;
    if (!chunk && (r.z >= 0 || r.y <= r.x)) return r;
    const int n = r.y - r.x;
    r.x = s.dev_group[r.x];
    if (!chunk) r.y = r.x + n;
    return r;
  };
  std::vector<int4> dev_ranges;
  if (!size_only) {
    for (const int4 &r : s.ranges) dev_ranges.push_back(on_device(r));
    for (int4 &it : s.items) it = on_device(it);
    for (int4 &t : s.step_tasks)
      if (t.x >= 0) t.x = s.dev_group[t.x];
  }

  s.set_bytes = (size_t)data / n_sets;
  (Layout &)s = lay_out(s, n_groups, n_ops, n_stab, n_uperm, s.prog.size() + s.prog_more,
                        s.step_tasks.size(), n_sets);
  if (size_only) return QTN_OK;
  s.desc_blob.assign(s.off_data - s.off_desc, 0);
  auto put = [&](size_t off, const void *src, size_t bytes) {
    if (bytes) std::memcpy(s.desc_blob.data() + (off - s.off_desc), src, bytes);
  };
  put(s.off_fills, s.fills.data(), sizeof(FillDesc) * s.fills.size());
  put(s.off_groups, dev_groups.data(), sizeof(DevGroup) * dev_groups.size());
  put(s.off_ops, dev_ops.data(), sizeof(DevOp) * dev_ops.size());
  put(s.off_stab, dev_stab.data(), sizeof(int32_t) * dev_stab.size());
  put(s.off_uperm, dev_uperm.data(), dev_uperm.size());
  put(s.off_ranges, dev_ranges.data(), sizeof(int4) * dev_ranges.size());
  put(s.off_prog, s.prog.data(), sizeof(uint32_t) * s.prog.size());
  put(s.off_csb, s.csb.data(), sizeof(int) * s.csb.size());
  put(s.off_ncb, s.ncb.data(), sizeof(int) * s.ncb.size());
  put(s.off_cns, s.cns.data(), sizeof(int) * s.cns.size());
  put(s.off_step_tasks, s.step_tasks.data(), sizeof(int4) * s.step_tasks.size());
  put(s.off_items, s.items.data(), sizeof(int4) * s.items.size());
  put(s.off_steps, s.step_begin.data(), sizeof(int) * s.step_begin.size());
  put(s.off_item_task, s.item_task.data(), sizeof(int) * s.item_task.size());
  put(s.off_task_next, s.task_next.data(), sizeof(int) * s.task_next.size());
  put(s.off_task_first, s.task_first.data(), sizeof(int) * s.task_first.size());
  put(s.off_task_need, s.task_need.data(), sizeof(int) * s.task_need.size());
  return QTN_OK;
}

void drop_graph(Runtime &rt) {
  if (rt.exec) (void)hipGraphExecDestroy(rt.exec);
  if (rt.graph) (void)hipGraphDestroy(rt.graph);
  rt.exec = nullptr;
  rt.graph = nullptr;
}

int ensure_runtime(Runtime &rt, int n_streams, int n_res) {
  int dev = 0;
  QTN_HIP(hipGetDevice(&dev));
  if (rt.device >= 0 && rt.device != dev) rt.release();
  if (rt.device < 0) {
    rt.device = dev;
    QTN_HIP(hipStreamCreateWithFlags(&rt.main, hipStreamNonBlocking));
    for (int i = 0; i < n_streams; i++) {
      hipStream_t s;
      QTN_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
      rt.side.push_back(s);
      hipEvent_t e;
      QTN_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
      rt.ev_join.push_back(e);
    }
    QTN_HIP(hipEventCreateWithFlags(&rt.ev_in, hipEventDisableTiming));
    QTN_HIP(hipEventCreateWithFlags(&rt.ev_fork, hipEventDisableTiming));
    QTN_HIP(hipHostMalloc((void **)&rt.pinned_err, 4 * sizeof(uint32_t), hipHostMallocDefault));
    int n_cu = 0;
    QTN_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    rt.persist_blocks = persistent_blocks(kPrecC128, n_cu);
  }
  // a runtime first made for a one-stream pass (autotuning) grows to the
  // network's stream count
  while ((int)rt.side.size() < n_streams) {
    hipStream_t s;
    QTN_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
    rt.side.push_back(s);
    hipEvent_t e;
    QTN_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    rt.ev_join.push_back(e);
  }
  if (rt.pinned_n < (size_t)n_res) {
    drop_graph(rt);  // it holds the old buffer's address
    if (rt.pinned) QTN_HIP(hipHostFree(rt.pinned));
    rt.pinned = nullptr;
    rt.pinned_n = 0;
    QTN_HIP(hipHostMalloc((void **)&rt.pinned, sizeof(double) * n_res, hipHostMallocDefault));
    rt.pinned_n = n_res;
  }
  return QTN_OK;
}

struct Timer {
  bool on = false;
  struct Rec {
    int kind;
    hipEvent_t a, b;
    int group, n_groups;
    double bytes, flops;
  };
  std::vector<Rec> recs;
  // on_dispatch: the launch attaches the events to its kernel's dispatch
  // (t0(), t1()) instead of recording them around it on the stream
  int begin(int kind, hipStream_t s, int group = -1, int n_groups = 0, double bytes = 0,
            double flops = 0, bool on_dispatch = false) {
    if (!on) return QTN_OK;
    Rec r{kind, nullptr, nullptr, group, n_groups, bytes, flops};
    QTN_HIP(hipEventCreate(&r.a));
    QTN_HIP(hipEventCreate(&r.b));
    if (!on_dispatch) QTN_HIP(hipEventRecord(r.a, s));
    recs.push_back(r);
    return QTN_OK;
  }
  hipEvent_t t0() const { return on ? recs.back().a : nullptr; }
  hipEvent_t t1() const { return on ? recs.back().b : nullptr; }
  int end(hipStream_t s, bool on_dispatch = false) {
    if (!on || on_dispatch) return QTN_OK;
    QTN_HIP(hipEventRecord(recs.back().b, s));
    return QTN_OK;
  }
  ~Timer() {
    for (auto &r : recs) {
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
  }
};

// Blocks of the persistent launch: all that are resident at once, or the
// tuned share of them (whole rounds over the 8 XCDs, at least 8).
int persist_grid(const Exec &X) {
  const int full = X.rt.persist_blocks;
  if (X.grid_quarters >= 4 || full <= 8) return full;
  const int nb = full * X.grid_quarters / 4;
  return std::max(8, nb - nb % 8);
}

// Orders the items inside every lockstep step: 0 the costliest light cone's
// first (as built), 1 reversed.  The blob's copies are rewritten and the
// schedule takes a new serial, so the next run uploads them.
void set_item_order(Schedule &s, int order) {
  if (order == s.item_order) return;
  for (int j = 0; j < s.n_steps; j++) {
    std::reverse(s.items.begin() + s.step_begin[j], s.items.begin() + s.step_begin[j + 1]);
    std::reverse(s.item_task.begin() + s.step_begin[j],
                 s.item_task.begin() + s.step_begin[j + 1]);
  }
  if (!s.items.empty())
    std::memcpy(s.desc_blob.data() + (s.off_items - s.off_desc), s.items.data(),
                sizeof(int4) * s.items.size());
  if (!s.item_task.empty())
    std::memcpy(s.desc_blob.data() + (s.off_item_task - s.off_desc), s.item_task.data(),
                sizeof(int) * s.item_task.size());
  s.item_order = order;
  s.serial = ++g_sched_serial;
}

// Every launch of one evaluation, on rt.main and the side streams.
int enqueue(Exec &X, Timer &tm) {
  Schedule &s = X.sched;
  Runtime &rt = X.rt;
  char *ws = (char *)rt.ws;
  char *desc = rt.desc_base;
  void *data = ws + s.off_data;
  auto *groups = (const DevGroup *)(desc + s.off_groups);
  auto *ops = (const DevOp *)(desc + s.off_ops);
  auto *ranges = (const int4 *)(desc + s.off_ranges);
  auto *prog = (const uint32_t *)(desc + s.off_prog);
  auto *stab = (const int32_t *)(desc + s.off_stab);
  auto *uperm = (const uint8_t *)(desc + s.off_uperm);
  int rc;
  if ((rc = tm.begin(QTN_K_FILL, rt.main))) return rc;
  QTN_HIP(launch_fill(s.prec, data, rt.pinned + (2 * s.n_cones + s.n_nets) * s.n_sets,
                      (const FillDesc *)(desc + s.off_fills), s.n_nets, s.n_angles, s.n_sets,
                      rt.main));
  if ((rc = tm.end(rt.main))) return rc;
  const int NS = s.n_sets;  // launch records carry the bytes of every set
  if (X.persistent) {
    if (NS != 1) return set_err(QTN_EINVAL, "the persistent executors run one angle set");
    bool any_heavy = false;
    for (char h : s.cone_heavy) any_heavy |= h != 0;
    // the persistent launch runs alone: its grid barriers need every block
    // resident, which kernels running beside it could prevent (measured: with
    // the heavy cones' launches started beside a full-size persistent grid, a
    // barrier wait ran past its bound)
    const int nb = persist_grid(X);
    if (nb < 1) return set_err(QTN_EDEVICE, "persistent kernel does not fit on the device");
    double b_all = 0, f_all = 0;
    for (int k = 0; k < QTN_NKERNELS; k++) {
      b_all += s.bytes[k];
      f_all += s.flops[k];
    }
    const int K = tm.on ? 1 : (int)rt.side.size();
    if (X.hybrid && any_heavy) {
      // the heavy cones' share is not the persistent launch's
      for (int c = 0; c < s.n_cones; c++)
        if (s.cone_heavy[c]) {
          for (auto &t : s.cone_tasks[c]) {
            b_all -= t.bytes;
            f_all -= t.flops;
          }
        }
    }
    if ((rc = tm.begin(QTN_K_PERSISTENT, rt.main, 0, (int)s.groups.size(), b_all, f_all, true)))
      return rc;
    if (X.dataflow)
      QTN_HIP(launch_dataflow(data, groups, ops, stab, uperm, prog, (const int4 *)(desc + s.off_items),
                              (int)s.items.size(), s.n_init, (const int *)(desc + s.off_item_task),
                              (const int *)(desc + s.off_task_next),
                              (const int *)(desc + s.off_task_first),
                              (const int *)(desc + s.off_task_need), (uint32_t *)(desc + s.off_queue),
                              (uint32_t *)(desc + s.off_ctl), s.n_ctl, nb, X.spin_limit, rt.main,
                              tm.t0(), tm.t1()));
    else
      QTN_HIP(launch_persistent(s.prec, data, groups, ops, stab, uperm, prog,
                                (const int4 *)(desc + s.off_items), (const int *)(desc + s.off_steps),
                                s.n_steps, (uint32_t *)(desc + s.off_ctl), s.n_ctl, nb, X.spin_limit,
                                rt.main, tm.t0(), tm.t1()));
    if ((rc = tm.end(rt.main, true))) return rc;
    if (X.hybrid && any_heavy) {
      // after the persistent launch (which ran their leading segments): the
      // heavy cones, each cone's tasks in order on one side stream, heaviest
      // first, dealt to the least loaded stream
      QTN_HIP(hipEventRecord(rt.ev_fork, rt.main));
      for (int i = 0; i < K; i++) QTN_HIP(hipStreamWaitEvent(rt.side[i], rt.ev_fork, 0));
      std::vector<int> order;
      std::vector<double> cost(s.n_cones, 0);
      for (int c = 0; c < s.n_cones; c++)
        if (s.cone_heavy[c]) {
          order.push_back(c);
          for (auto &t : s.cone_tasks[c]) cost[c] += t.bytes;
        }
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
      std::vector<double> load(K, 0);
      for (int c : order) {
        const int st = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        load[st] += cost[c];
        hipStream_t hs = rt.side[st];
        for (auto &t : s.cone_tasks[c]) {
          const int g0 = t.kind == QTN_K_BLOCK ? s.ranges[t.index].x : t.index;
          const int ng = t.kind == QTN_K_BLOCK ? s.ranges[t.index].y - s.ranges[t.index].x : 1;
          if ((rc = tm.begin(t.kind, hs, g0, ng, t.bytes, t.flops, true))) return rc;
          if (t.kind == QTN_K_BLOCK)
            QTN_HIP(launch_block_groups(prog_prec(s, t.index), data, groups, ops, stab, uperm, prog,
                                        ranges, t.index, 1, NS, hs, tm.t0(), tm.t1()));
          else
            QTN_HIP(launch_wide_group(s.groups[t.index], data, groups, ops, stab, uperm,
                                      s.dev_group[t.index], NS, hs, tm.t0(), tm.t1()));
          if ((rc = tm.end(hs, true))) return rc;
        }
      }
      for (int i = 0; i < K; i++) {
        QTN_HIP(hipEventRecord(rt.ev_join[i], rt.side[i]));
        QTN_HIP(hipStreamWaitEvent(rt.main, rt.ev_join[i], 0));
      }
    }
  } else {
  // leading small segments: one launch for every cone before the fork, or
  // (lead_per_cone) each cone's own one-block launch on its stream
  if (!X.lead_per_cone) {
    if ((rc = tm.begin(QTN_K_BLOCK, rt.main, 0, (int)s.groups.size(), NS * s.init_bytes,
                       NS * s.init_flops, true)))
      return rc;
    QTN_HIP(launch_block_groups(s.lead_prec, data, groups, ops, stab, uperm, prog, ranges, 0,
                                s.n_cones, NS, rt.main, tm.t0(), tm.t1()));
    if ((rc = tm.end(rt.main, true))) return rc;
  }
  // timed runs serialize on one stream, so each event pair brackets one kernel
  const int K = tm.on ? 1 : (int)rt.side.size();
  bool any = X.lead_per_cone;
  for (auto &tk : s.cone_tasks) any |= !tk.empty();
  if (X.steps && !s.steps.empty() && !tm.on) {
    // the cones' chains in step launches
    auto *tasks = (const int4 *)(desc + s.off_step_tasks);
    for (const Schedule::Step &st : s.steps) {
      QTN_HIP(launch_step(s.prec, data, groups, ops, stab, uperm, prog, tasks + st.first, st.n,
                          st.blocks, st.threads, st.lds, NS, rt.main));
      for (const Task &t : st.single) {
        if (t.kind == QTN_K_BLOCK)
          QTN_HIP(launch_block_groups(prog_prec(s, t.index), data, groups, ops, stab, uperm, prog,
                                      ranges, t.index, 1, NS, rt.main));
        else
          QTN_HIP(launch_wide_group(s.groups[t.index], data, groups, ops, stab, uperm,
                                    s.dev_group[t.index], NS, rt.main));
      }
    }
  } else if (any) {
    QTN_HIP(hipEventRecord(rt.ev_fork, rt.main));
    for (int i = 0; i < K; i++) QTN_HIP(hipStreamWaitEvent(rt.side[i], rt.ev_fork, 0));
    // heaviest light cones first, dealt round-robin over the side streams
    std::vector<int> order(s.n_cones);
    std::vector<double> cost(s.n_cones, 0);
    for (int c = 0; c < s.n_cones; c++) {
      order[c] = c;
      for (auto &t : s.cone_tasks[c]) cost[c] += t.bytes;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    std::vector<double> load(K, 0);
    for (int c : order) {
      const bool lead = X.lead_per_cone && s.ranges[c].y > s.ranges[c].x;
      if (s.cone_tasks[c].empty() && !lead) continue;
      int st = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      load[st] += cost[c];
      hipStream_t hs = rt.side[st];
      if (lead) {
        if ((rc = tm.begin(QTN_K_BLOCK, hs, s.ranges[c].x, s.ranges[c].y - s.ranges[c].x, 0, 0,
                           true)))
          return rc;
        QTN_HIP(launch_block_groups(prog_prec(s, c), data, groups, ops, stab, uperm, prog, ranges, c,
                                    1, NS, hs,
                                    tm.t0(), tm.t1()));
        if ((rc = tm.end(hs, true))) return rc;
      }
      for (auto &t : s.cone_tasks[c]) {
        const int g0 = t.kind == QTN_K_BLOCK ? s.ranges[t.index].x : t.index;
        const int ng = t.kind == QTN_K_BLOCK ? s.ranges[t.index].y - s.ranges[t.index].x : 1;
        if ((rc = tm.begin(t.kind, hs, g0, ng, NS * t.bytes, NS * t.flops, true))) return rc;
        if (t.kind == QTN_K_BLOCK)
          QTN_HIP(launch_block_groups(prog_prec(s, t.index), data, groups, ops, stab, uperm, prog,
                                      ranges, t.index, 1, NS, hs, tm.t0(), tm.t1()));
        else
          QTN_HIP(launch_wide_group(s.groups[t.index], data, groups, ops, stab, uperm,
                                    s.dev_group[t.index], NS, hs, tm.t0(), tm.t1()));
        if ((rc = tm.end(hs, true))) return rc;
      }
    }
    for (int i = 0; i < K; i++) {
      QTN_HIP(hipEventRecord(rt.ev_join[i], rt.side[i]));
      QTN_HIP(hipStreamWaitEvent(rt.main, rt.ev_join[i], 0));
    }
  }
  }
  if ((rc = tm.begin(QTN_K_REDUCE, rt.main))) return rc;
  QTN_HIP(launch_reduce(s.scalar_prec == 1 ? kPrecC64 : kPrecC128, data, s.scalar_off,
                        s.scalar_sstride, (const int *)(desc + s.off_csb),
                        (const int *)(desc + s.off_ncb), (const int *)(desc + s.off_cns), s.n_cones,
                        s.n_nets, NS,
                        (double *)(ws + s.off_res), rt.pinned,
                        X.persistent ? (const uint32_t *)(desc + s.off_ctl) : nullptr,
                        rt.pinned_err, rt.main));
  if ((rc = tm.end(rt.main))) return rc;
  return QTN_OK;
}

// One evaluation: the angles are read from, and the results written to,
// page-locked host memory by the first and the last kernel, so that a call
// copies nothing once the schedule's descriptors are on the device.
// set_angles: n_sets * n_angles doubles (per set, per network gamma[p] then
// beta[p]); NULL: the networks' own angles (one set).
int run_exec(Exec &X, const std::vector<const qtn_network *> &nets, void *ws, size_t bytes,
             void *stream, int n_streams, bool eager, Timer &tm, std::vector<double> &res,
             const double *set_angles = nullptr) {
  Schedule &s = X.sched;
  Runtime &rt = X.rt;
  if (!ws) return set_err(QTN_EINVAL, "workspace is NULL");
  if (bytes < s.total)
    return set_err(QTN_ENOMEM, "workspace of " + std::to_string(bytes) + " bytes, plan needs " +
                                   std::to_string(s.total));
  if ((uintptr_t)ws % 256) return set_err(QTN_EINVAL, "workspace must be 256-byte aligned");
  if (!set_angles && s.n_sets != 1) return set_err(QTN_EINVAL, "angle sets missing");
  // a call waits for its results, which a capture does not allow: refused
  // before anything of it joins the caller's graph
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing((hipStream_t)stream, &capture) != hipSuccess) (void)hipGetLastError();
  else if (capture != hipStreamCaptureStatusNone)
    return set_err(QTN_EDEVICE, "the stream is being captured, and the call waits for its results");
  const int n_res = (2 * s.n_cones + s.n_nets) * s.n_sets;
  int rc = ensure_runtime(rt, n_streams, n_res + s.n_angles * s.n_sets);
  if (rc) return rc;
  const size_t n_desc = s.desc_blob.size();
  if (rt.dev_desc_cap < n_desc && rt.no_dev_serial != s.serial) {
    if (rt.dev_desc) drop_graph(rt);
    desc_free(rt.dev_desc, rt.dev_desc_cap);
    bool none;
    rt.dev_desc = desc_alloc(n_desc, &none);
    rt.dev_desc_cap = rt.dev_desc ? n_desc : 0;
    rt.dev_serial = 0;
    if (none) rt.no_dev_serial = s.serial;
  }
  // the captured graph holds the old addresses
  char *base = rt.dev_desc ? rt.dev_desc - s.off_desc : (char *)ws;
  if (rt.ws != ws || rt.desc_base != base) drop_graph(rt);
  rt.ws = ws;
  rt.desc_base = base;
  QTN_HIP(hipEventRecord(rt.ev_in, (hipStream_t)stream));
  QTN_HIP(hipStreamWaitEvent(rt.main, rt.ev_in, 0));
  if (!rt.dev_desc || rt.dev_serial != s.serial) {
    QTN_HIP(hipMemcpyAsync(base + s.off_desc, s.desc_blob.data(), n_desc, hipMemcpyHostToDevice,
                           rt.main));
    rt.dev_serial = 0;  // known to be there once the stream has been waited for
  }
  double *angles = rt.pinned + n_res;
  if (set_angles) {
    std::memcpy(angles, set_angles, sizeof(double) * s.n_angles * s.n_sets);
  } else {
    size_t a = 0;
    for (auto *net : nets) {
      for (int l = 0; l < net->p; l++) angles[a + l] = net->gamma[l];
      for (int l = 0; l < net->p; l++) angles[a + net->p + l] = net->beta[l];
      a += 2 * net->p;
    }
  }
  if (eager || tm.on) {
    if ((rc = enqueue(X, tm))) return rc;
  } else {
    if (!rt.exec) {
      QTN_HIP(hipStreamBeginCapture(rt.main, hipStreamCaptureModeThreadLocal));
      rc = enqueue(X, tm);
      hipGraph_t graph = nullptr;
      hipError_t ce = hipStreamEndCapture(rt.main, &graph);
      if (rc) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
      }
      if (ce != hipSuccess)
        return set_err(QTN_EDEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(ce));
      rt.graph = graph;
      QTN_HIP(hipGraphInstantiate(&rt.exec, rt.graph, nullptr, nullptr, 0));
    }
    QTN_HIP(hipGraphLaunch(rt.exec, rt.main));
  }
  QTN_HIP(hipStreamSynchronize(rt.main));
  rt.dev_serial = s.serial;
  if (X.persistent && rt.pinned_err[0] != 0)
    return set_err(QTN_EDEVICE, X.dataflow
                                    ? "persistent executor: a dependency wait exceeded its bound"
                                    : "persistent executor: a grid barrier wait exceeded its bound");
  res.assign(rt.pinned, rt.pinned + n_res);
  return QTN_OK;
}

bool finite_angles(int p, const double *g, const double *b) {
  for (int l = 0; l < p; l++)
    if (!std::isfinite(g[l]) || !std::isfinite(b[l])) return false;
  return true;
}

}  // namespace

extern "C" {

const char *qtn_last_error(void) { return g_err.c_str(); }

int qtn_network_build(int32_t n_vertices, int64_t n_edges, const int32_t *edges, int32_t p,
                      const double *gamma, const double *beta, const qtn_config *cfg,
                      qtn_network **out) {
  try {
    if (!out) return set_err(QTN_EINVAL, "out is NULL");
    if (p < 1 || p > 64) return set_err(QTN_EINVAL, "p must be in 1..64");
    if (!gamma || !beta) return set_err(QTN_EINVAL, "angles are NULL");
    if (!finite_angles(p, gamma, beta)) return set_err(QTN_EINVAL, "angles must be finite");
    std::unique_ptr<qtn_network> net(new qtn_network());
    std::string err = make_graph(n_vertices, n_edges, edges, &net->g);
    if (!err.empty()) return set_err(QTN_EINVAL, err);
    net->p = p;
    net->gamma.assign(gamma, gamma + p);
    net->beta.assign(beta, beta + p);
    if (cfg) {
      if (cfg->max_levels < 0 || cfg->max_levels > kMaxLevels)
        return set_err(QTN_EINVAL, "max_levels must be in 0..8");
      if (cfg->max_levels) net->opt.max_levels = cfg->max_levels;
      if (cfg->small_width < 0 || cfg->small_width > kMaxWidth)
        return set_err(QTN_EINVAL, "small_width must be in 0..32");
      if (cfg->small_width) net->opt.small_width = cfg->small_width;
      if (cfg->max_width < 0 || cfg->max_width > kMaxWidth)
        return set_err(QTN_EINVAL, "max_width must be in 0..32");
      if (cfg->max_width) net->opt.max_width = cfg->max_width;
      if (cfg->n_streams < 0 || cfg->n_streams > 16)
        return set_err(QTN_EINVAL, "n_streams must be in 0..16");
      if (cfg->n_streams) net->n_streams = cfg->n_streams;
      net->eager = cfg->eager != 0;
      if (cfg->lane_sum_bits < 0 || cfg->lane_sum_bits > 5)
        return set_err(QTN_EINVAL, "lane_sum_bits must be in 0..5");
      if (cfg->lane_sum_bits) net->lane_sum_bits = cfg->lane_sum_bits;
      if (cfg->variant < 0 || cfg->variant > 4) return set_err(QTN_EINVAL, "variant must be 0..4");
      net->variant = cfg->variant;
      if (cfg->order_trials < 0 || cfg->order_trials > 4096)
        return set_err(QTN_EINVAL, "order_trials must be in 0..4096");
      net->order_trials = cfg->order_trials;
      if (cfg->executor < 0 || cfg->executor > 5) return set_err(QTN_EINVAL, "executor must be 0..5");
      net->executor = cfg->executor;
      if (cfg->spin_limit > 0) net->spin_limit = (uint32_t)cfg->spin_limit;
      if (cfg->mixed_width < 0 || cfg->mixed_width > 32)
        return set_err(QTN_EINVAL, "mixed_width must be in 0..32");
      if (cfg->mixed_width > 0) net->opt.mixed_width = cfg->mixed_width;
      if (cfg->slice_width < 0 || cfg->slice_width > kMaxWidth)
        return set_err(QTN_EINVAL, "slice_width must be in 0..32");
      net->opt.slice_width = cfg->slice_width;
      if (cfg->order_weight < 0 || cfg->order_weight > 1000)
        return set_err(QTN_EINVAL, "order_weight must be in 0..1000");
      net->opt.order_weight = cfg->order_weight;
      if (cfg->hybrid_width < 0 || cfg->hybrid_width > kMaxWidth)
        return set_err(QTN_EINVAL, "hybrid_width must be in 0..32");
      if (cfg->hybrid_width > 0) net->hybrid_width = cfg->hybrid_width;
    }
    const int m = (int)n_edges;
    net->cones.resize(m);
    net->minfill.resize(m);
    qtn_network *raw = net.get();
    parallel_for(m, [&](int e) { raw->cones[e] = build_lightcone(raw->g, e, p); });
    *out = net.release();
    return QTN_OK;
  } catch (const std::bad_alloc &) {
    return set_err(QTN_ENOMEM, "host allocation failed");
  } catch (const std::exception &e) {
    return set_err(QTN_EINVAL, e.what());
  } catch (...) {
    return exception_status();
  }
}

int qtn_network_info(const qtn_network *cnet, int64_t edge, int32_t *n_vars, int32_t *n_tensors,
                     int32_t *width_minfill) {
  try {
    auto *net = const_cast<qtn_network *>(cnet);
    if (!net) return set_err(QTN_EINVAL, "network is NULL");
    if (edge < 0 || edge >= (int64_t)net->cones.size())
      return set_err(QTN_EINVAL, "edge out of range");
    const LightCone &lc = net->cones[edge];
    int32_t w = 0;
    if (width_minfill) {
      PlanOptions o = net->opt;
      o.max_levels = 1;
      o.max_width = 64;
      ConePlan pl;
      std::string err = plan_cone(lc, get_minfill(net, (int)edge), o, &pl);
      if (!err.empty()) return set_err(QTN_EINVAL, err);
      w = pl.max_width;
    }
    if (n_vars) *n_vars = lc.n_vars;
    if (n_tensors) *n_tensors = (int32_t)lc.gates.size();
    if (width_minfill) *width_minfill = w;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_order_minfill(const qtn_network *cnet, int64_t edge, int32_t *order_out) {
  try {
    auto *net = const_cast<qtn_network *>(cnet);
    if (!net || !order_out) return set_err(QTN_EINVAL, "NULL argument");
    if (edge < 0 || edge >= (int64_t)net->cones.size())
      return set_err(QTN_EINVAL, "edge out of range");
    const auto &o = get_minfill(net, (int)edge);
    std::copy(o.begin(), o.end(), order_out);
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_plan(qtn_network *net, const int32_t *const *orders, int32_t precision,
             size_t *workspace_bytes_out) {
  try {
    if (!net) return set_err(QTN_EINVAL, "network is NULL");
    if (precision != QTN_C128 && precision != QTN_C64 && precision != QTN_MIXED)
      return set_err(QTN_EINVAL, "precision must be QTN_C128, QTN_C64 or QTN_MIXED");
    const int m = (int)net->cones.size();
    std::vector<ConePlan> plans(m);
    std::vector<std::string> errs(m);
    PlanOptions o = net->opt;
    o.precision = precision;
    parallel_for(m, [&](int e) {
      const LightCone &lc = net->cones[e];
      const bool given = orders && orders[e];
      std::vector<int> ord;
      // order search by the merged plan's cost (order_weight > 0) or by the
      // sum of 2^width
      const PlanOptions *cost_opt = o.order_weight > 0 ? &o : nullptr;
      if (given)
        ord.assign(orders[e], orders[e] + lc.n_vars);
      else if (net->order_trials > 1)
        ord = search_order(lc, net->order_trials, cost_opt, o.order_weight);
      else
        ord = get_minfill(net, e);
      if (o.slice_width > 0 && order_width(lc, ord) > o.slice_width) {
        // index slicing: fix variables until the widest bucket fits the cap,
        // then plan the restricted light cone (a caller's order still applies:
        // the fixed variables are left with empty buckets)
        std::vector<int> cord;
        const std::vector<int> sv = choose_slices(lc, o.slice_width, kMaxSliceVars,
                                                  net->order_trials, &cord, cost_opt, o.order_weight);
        LightCone sc = lc;
        for (size_t k = 0; k < sv.size(); k++) sc = slice_cone(sc, sv[k], (int)k);
        if (!given) {
          // the full order search, unless it is wider than the order the
          // choice of slices reached
          ord = net->order_trials > 1 ? search_order(sc, net->order_trials, cost_opt, o.order_weight)
                                      : minfill_order(sc);
          if (order_width(sc, ord) > std::max(o.slice_width, order_width(sc, cord))) ord = cord;
        }
        errs[e] = plan_cone(sc, ord, o, &plans[e]);
        plans[e].slice_vars = sv;
        plans[e].n_slices = 1 << sv.size();
        plans[e].gates = sc.gates;
        return;
      }
      errs[e] = plan_cone(lc, ord, o, &plans[e]);
    });
    for (int e = 0; e < m; e++)
      if (!errs[e].empty()) {
        bool range = errs[e].find("exceeds") != std::string::npos;
        return set_err(range ? QTN_ERANGE : QTN_EINVAL, "edge " + std::to_string(e) + ": " + errs[e]);
      }
    auto ex = std::make_unique<Exec>();
    net->plans.swap(plans);
    net->precision = precision;
    qtn_network *one[1] = {net};
    int rc = build_schedule(one, 1, &ex->sched, nullptr, 0, 1,
                            net->executor == 2 || net->executor == 4 || net->executor == 5);
    if (rc) {
      net->plans.clear();
      net->planned = false;
      return rc;
    }
    drop_batches_with(net);
    ex->persistent = net->executor == 2 || net->executor == 4 || net->executor == 5;
    ex->hybrid = net->executor == 5;
    ex->dataflow = net->executor == 4;
    ex->lead_per_cone = net->executor == 3;
    ex->steps = net->executor == 0;
    {
      size_t mx = ex->sched.total;
      for (const Force &f : tune_candidates()) {
        Schedule tmp;
        if (build_schedule(one, 1, &tmp, &f, kTuneSingleWidth, 1, false, true) == QTN_OK)
          mx = std::max(mx, tmp.total);
      }
      net->tune_workspace = mx;
    }
    ex->spin_limit = net->spin_limit;
    if (net->exec) ex->rt.take(net->exec->rt);
    net->exec = std::move(ex);
    net->planned = true;
    net->version++;
    if (workspace_bytes_out) *workspace_bytes_out = net->tune_workspace;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_set_angles(qtn_network *net, const double *gamma, const double *beta) {
  if (!net || !gamma || !beta) return set_err(QTN_EINVAL, "NULL argument");
  if (!finite_angles(net->p, gamma, beta)) return set_err(QTN_EINVAL, "angles must be finite");
  net->gamma.assign(gamma, gamma + net->p);
  net->beta.assign(beta, beta + net->p);
  return QTN_OK;
}

static int record_timing(qtn_network *net, const Exec &X, const Timer &tm, qtn_timing *timing);

static int contract_impl(qtn_network *net, void *ws, size_t bytes, void *stream, double *zz,
                         double *zz_im, double *energy, qtn_timing *timing) {
  try {
    if (!net) return set_err(QTN_EINVAL, "network is NULL");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    Timer tm;
    tm.on = timing != nullptr;
    std::vector<double> res;
    int rc = run_exec(*net->exec, {net}, ws, bytes, stream, net->n_streams, net->eager, tm, res);
    if (rc) return rc;
    if (timing && (rc = record_timing(net, *net->exec, tm, timing))) return rc;
    const int m = net->exec->sched.n_cones;
    if (zz) std::copy(res.begin(), res.begin() + m, zz);
    if (zz_im) std::copy(res.begin() + m, res.begin() + 2 * m, zz_im);
    if (energy) *energy = res[2 * m];
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

// The launch log and per-class totals of a timed run of X (bytes and flops
// cover every angle set of the run).
static int record_timing(qtn_network *net, const Exec &X, const Timer &tm, qtn_timing *timing) {
    qtn_timing t;
    std::memset(&t, 0, sizeof t);
    {
      net->launch_log.clear();
      const Schedule &sc = X.sched;
      for (auto &r : tm.recs) {
        float ms = 0;
        QTN_HIP(hipEventElapsedTime(&ms, r.a, r.b));
        t.ms[r.kind] += ms;
        t.launches[r.kind]++;
        qtn_launch_rec lr;
        std::memset(&lr, 0, sizeof lr);
        lr.kind = r.kind;
        lr.group = r.group;
        lr.n_groups = r.n_groups;
        lr.ms = ms;
        lr.bytes = r.bytes;
        lr.flops = r.flops;
        if (r.group >= 0 && r.group < (int)sc.groups.size()) {
          const DevGroup &g = sc.groups[r.group];
          lr.w = g.w;
          lr.L = g.L;
          lr.n_ops = g.n_ops;
          lr.variant = g.variant;
          lr.n_units = (int32_t)g.n_units;
          lr.prec = g.prec;
          lr.cvt = g.cvt;
          lr.knob = g.variant == kVarStream || g.variant == kVarCell || g.variant == kVarMfma ? g.rls : 0;
          lr.serial = g.variant == kVarStream || g.variant == kVarCell ? g.sl : 0;
        }
        net->launch_log.push_back(lr);
      }
      for (int k = 0; k < QTN_NKERNELS; k++) {
        t.bytes[k] = X.sched.bytes[k] * X.sched.n_sets;
        t.flops[k] = X.sched.flops[k] * X.sched.n_sets;
      }
      if (X.persistent) {
        for (int k = 0; k < QTN_K_PERSISTENT; k++) {
          t.bytes[QTN_K_PERSISTENT] += t.bytes[k];
          t.flops[QTN_K_PERSISTENT] += t.flops[k];
          t.bytes[k] = t.flops[k] = 0;
        }
      }
    }
    *timing = t;
    return QTN_OK;
}

int qtn_contract(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                 double *zz_out, double *zz_imag_out, double *energy_out) {
  return contract_impl(net, d_workspace, bytes, hip_stream, zz_out, zz_imag_out, energy_out,
                       nullptr);
}

constexpr int kMaxAngleSets = 1024;

static Exec *angle_exec(qtn_network *net, int n_sets, bool in_order, int *rc) {
  qtn_network::AngleExec &slot = net->angle_exec[in_order];
  if (slot.exec && slot.sets == n_sets && slot.version == net->version) return slot.exec.get();
  auto ex = std::make_unique<Exec>();
  qtn_network *one[1] = {net};
  // the same kernel mappings as the network's own schedule (so that every
  // set equals its single-set evaluation), though launched per group
  *rc = build_schedule(one, 1, &ex->sched, nullptr, 0, n_sets, net->exec->persistent, false, in_order);
  if (*rc) return nullptr;
  // per-group launches (the persistent executors run one set)
  ex->lead_per_cone = net->executor == 3;
  ex->steps = net->executor == 0;
  ex->spin_limit = net->spin_limit;
  if (slot.exec) ex->rt.take(slot.exec->rt);
  slot.exec = std::move(ex);
  slot.sets = n_sets;
  slot.version = net->version;
  return slot.exec.get();
}

// Where a network computes in complex64 a gradient runs in the plan's order of
// operations, whatever order a mapping would choose for speed.  That keeps the
// results of earlier versions bit for bit, and nothing else: a central
// difference divides the rounding of its energies by 2 step, so that another
// order moves a derivative far more than it moves an energy.  It is not the more
// accurate order.  Derivatives of 24 graphs with step 1e-4 against complex128, rms
// of the relative error: complex64 1.4e-2 in the plan's order, 6.1e-3 in the
// other, mixed 1.3e-3 in both.
static bool gradient_in_order(const qtn_network *net) { return net->precision != kPrecC128; }

static int gradient_sets(const qtn_network *net) { return 4 * net->p + 1; }

int qtn_angles_workspace(qtn_network *net, int32_t n_sets, size_t *bytes_out) {
  try {
    if (!net || !bytes_out) return set_err(QTN_EINVAL, "NULL argument");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    if (n_sets < 1 || n_sets > kMaxAngleSets)
      return set_err(QTN_EINVAL, "n_sets must be in 1.." + std::to_string(kMaxAngleSets));
    int rc = QTN_OK;
    Exec *ex = angle_exec(net, n_sets, false, &rc);
    if (!ex) return rc;
    *bytes_out = ex->sched.total;
    // as many sets as a gradient takes, or more, serve the gradient too
    if (n_sets >= gradient_sets(net) && gradient_in_order(net))
      *bytes_out = std::max(*bytes_out, form_bytes(ex->sched, true, gradient_sets(net)));
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

static int contract_angles(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                           int32_t n_sets, bool in_order, const double *gamma, const double *beta,
                           double *zz_out, double *energy_out, qtn_timing *timing) {
  try {
    if (!net || !gamma || !beta) return set_err(QTN_EINVAL, "NULL argument");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    if (n_sets < 1 || n_sets > kMaxAngleSets)
      return set_err(QTN_EINVAL, "n_sets must be in 1.." + std::to_string(kMaxAngleSets));
    const int p = net->p;
    std::vector<double> ang((size_t)n_sets * 2 * p);
    for (int k = 0; k < n_sets; k++) {
      if (!finite_angles(p, gamma + (size_t)k * p, beta + (size_t)k * p))
        return set_err(QTN_EINVAL, "angles of set " + std::to_string(k) + " are not finite");
      std::copy(gamma + (size_t)k * p, gamma + (size_t)(k + 1) * p, ang.begin() + (size_t)k * 2 * p);
      std::copy(beta + (size_t)k * p, beta + (size_t)(k + 1) * p,
                ang.begin() + (size_t)k * 2 * p + p);
    }
    int rc = QTN_OK;
    Exec *ex = angle_exec(net, n_sets, in_order, &rc);
    if (!ex) return rc;
    Timer tm;
    tm.on = timing != nullptr;
    std::vector<double> res;
    rc = run_exec(*ex, {net}, d_workspace, bytes, hip_stream, net->n_streams, net->eager, tm, res,
                  ang.data());
    if (rc) return rc;
    if (timing && (rc = record_timing(net, *ex, tm, timing))) return rc;
    const int m = (int)net->cones.size(), per = 2 * m + 1;
    for (int k = 0; k < n_sets; k++) {
      if (zz_out) std::copy(res.begin() + (size_t)k * per, res.begin() + (size_t)k * per + m,
                            zz_out + (size_t)k * m);
      if (energy_out) energy_out[k] = res[(size_t)k * per + 2 * m];
    }
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_contract_angles(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                        int32_t n_sets, const double *gamma, const double *beta, double *zz_out,
                        double *energy_out, qtn_timing *timing) {
  return contract_angles(net, d_workspace, bytes, hip_stream, n_sets, false, gamma, beta, zz_out,
                         energy_out, timing);
}

int qtn_contract_timed(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                       double *zz_out, double *energy_out, qtn_timing *timing) {
  if (!timing) return set_err(QTN_EINVAL, "timing is NULL");
  return contract_impl(net, d_workspace, bytes, hip_stream, zz_out, nullptr, energy_out, timing);
}

static Exec *batch_exec(qtn_network *const *nets, int32_t n, int *rc) {
  std::vector<std::pair<const qtn_network *, uint64_t>> key;
  for (int i = 0; i < n; i++) {
    if (!nets[i]) {
      *rc = set_err(QTN_EINVAL, "NULL network in batch");
      return nullptr;
    }
    if (!nets[i]->planned) {
      *rc = set_err(QTN_ESTATE, "network " + std::to_string(i) + " is not planned");
      return nullptr;
    }
    key.push_back({nets[i], nets[i]->version});
  }
  std::lock_guard<std::mutex> lk(g_batch_lock);
  auto it = g_batch.find(key);
  if (it != g_batch.end()) return it->second.get();
  auto ex = std::make_unique<Exec>();
  // complex64: in the plan's order, for the same reason as gradients.  At
  // arbitrary angles a graph's <ZZ> can all be near zero, where rounding of 1e-8
  // is 6e-5 of them.  Errors of 120 graphs' <ZZ> against complex128: rms of a
  // graph's largest 2.5e-7 in the plan's order and 2.0e-7 in the other, rms
  // relative to a graph's norm 2.2e-5 and 8.0e-6.  What the order costs: 19.1 ms
  // for 16 cubic graphs of depths 2 to 4, 18.2 without it
  *rc = build_schedule(nets, n, &ex->sched, nullptr, 0, 1,
                       nets[0]->executor != 1 && nets[0]->executor != 3, false,
                       nets[0]->precision == kPrecC64);
  if (*rc) return nullptr;
  // batches default to the persistent executor
  ex->persistent = nets[0]->executor != 1 && nets[0]->executor != 3;
  ex->dataflow = nets[0]->executor == 4;
  ex->hybrid = nets[0]->executor == 5;
  ex->spin_limit = nets[0]->spin_limit;
  Exec *raw = ex.get();
  g_batch[key] = std::move(ex);
  return raw;
}

int qtn_batch_workspace(qtn_network *const *nets, int32_t n, size_t *workspace_bytes_out) {
  try {
    if (!nets || n < 1 || !workspace_bytes_out) return set_err(QTN_EINVAL, "bad batch arguments");
    int rc = QTN_OK;
    Exec *ex = batch_exec(nets, n, &rc);
    if (!ex) return rc;
    *workspace_bytes_out = ex->sched.total;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_contract_batch(qtn_network *const *nets, int32_t n, void *d_workspace, size_t bytes,
                       void *hip_stream, double *zz_out, double *energy_out) {
  try {
    if (!nets || n < 1) return set_err(QTN_EINVAL, "bad batch arguments");
    int rc = QTN_OK;
    Exec *ex = batch_exec(nets, n, &rc);
    if (!ex) return rc;
    std::vector<const qtn_network *> list(nets, nets + n);
    Timer tm;
    std::vector<double> res;
    rc = run_exec(*ex, list, d_workspace, bytes, hip_stream, nets[0]->n_streams, nets[0]->eager,
                  tm, res);
    if (rc) return rc;
    const int m = ex->sched.n_cones;
    if (zz_out) std::copy(res.begin(), res.begin() + m, zz_out);
    if (energy_out) std::copy(res.begin() + 2 * m, res.begin() + 2 * m + n, energy_out);
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_autotune_batch(qtn_network *const *nets, int32_t n, void *d_workspace, size_t bytes,
                       void *hip_stream, qtn_batch_tune_report *report) {
  try {
    if (!nets || n < 1) return set_err(QTN_EINVAL, "bad batch arguments");
    int rc = QTN_OK;
    Exec *ex = batch_exec(nets, n, &rc);
    if (!ex) return rc;
    if (!ex->persistent || ex->dataflow)
      return set_err(QTN_ESTATE, "batch autotuning needs the persistent lockstep or hybrid executor");
    std::vector<const qtn_network *> list(nets, nets + n);
    struct Cand {
      int quarters, order;
    };
    std::vector<Cand> cands;
    for (int order = 0; order < 2; order++)
      for (int q : {4, 3, 2}) cands.push_back({q, order});
    auto apply = [&](const Cand &c) {
      ex->grid_quarters = c.quarters;
      set_item_order(ex->sched, c.order);
      drop_graph(ex->rt);
    };
    std::vector<double> best(cands.size(), 1e300);
    std::vector<int> grid(cands.size(), 0);
    for (size_t i = 0; i < cands.size(); i++) {
      apply(cands[i]);
      // the first call captures the graph (or warms up): not timed
      for (int r = 0; r < 4; r++) {
        Timer tm;
        std::vector<double> res;
        const auto t0 = std::chrono::steady_clock::now();
        rc = run_exec(*ex, list, d_workspace, bytes, hip_stream, nets[0]->n_streams,
                      nets[0]->eager, tm, res);
        const auto t1 = std::chrono::steady_clock::now();
        if (rc) {
          apply(cands[0]);
          return rc;
        }
        if (r > 0) best[i] = std::min(best[i], std::chrono::duration<double, std::milli>(t1 - t0).count());
      }
      grid[i] = persist_grid(*ex);
    }
    // the built configuration unless another is more than 3% faster
    size_t pick = 0;
    for (size_t i = 1; i < cands.size(); i++)
      if (best[i] < best[pick]) pick = i;
    if (best[0] <= 1.03 * best[pick]) pick = 0;
    apply(cands[pick]);
    if (report) {
      qtn_batch_tune_report r;
      std::memset(&r, 0, sizeof r);
      r.n_candidates = (int32_t)cands.size();
      r.pick = (int32_t)pick;
      for (size_t i = 0; i < cands.size(); i++) {
        r.grid_blocks[i] = grid[i];
        r.item_order[i] = cands[i].order;
        r.ms[i] = best[i];
      }
      *report = r;
    }
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

// A group leaves the step launches' mapping when it takes more than this many
// milliseconds in a launch of its own; a shorter one is mostly launch there, and
// among other mappings the schedule loses its steps.  Choices by launches alone
// against cells for all short groups, autotuned: 20 vertices, depth 3, 209 us
// against 126; 16 vertices, depth 4, 1.60 ms against 0.92; quartic, 24 vertices,
// depth 3, complex64, 2.22 against 0.77.  By the cost model: 232 us against 112,
// 2.23 ms against 1.04; 40 vertices, quartic, 6.14 against 4.50.  The line itself
// matters little: from 0.02 to no limit these stay within 3%.
constexpr double kLeaveStepMs = 0.05;

// Workspace of autotuning over n_sets copies of the network's angles: the
// largest candidate schedule.
static int tune_workspace_bytes(qtn_network *net, int n_sets, size_t *bytes) {
  if (n_sets == 1) {
    *bytes = net->tune_workspace;
    return QTN_OK;
  }
  qtn_network *one[1] = {net};
  size_t mx = 0;
  for (const Force &f : tune_candidates()) {
    Schedule tmp;
    const int rc = build_schedule(one, 1, &tmp, &f, kTuneSingleWidth, n_sets, false, true);
    if (rc) return rc;
    mx = std::max(mx, tmp.total);
  }
  *bytes = mx;
  return QTN_OK;
}

// The autotuner; every candidate runs over n_sets copies of the network's
// current angles (n_sets 1: one evaluation).
static int autotune_sets(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                         int n_sets, qtn_tune_report *report) {
  try {
    if (!net) return set_err(QTN_EINVAL, "network is NULL");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    if (n_sets < 1 || n_sets > kMaxAngleSets)
      return set_err(QTN_EINVAL, "n_sets must be in 1.." + std::to_string(kMaxAngleSets));
    size_t need = 0;
    int wrc = tune_workspace_bytes(net, n_sets, &need);
    if (wrc) return wrc;
    if (bytes < need)
      return set_err(QTN_ENOMEM, "autotuning needs a workspace of " + std::to_string(need) +
                                     " bytes");
    // the angles of every set: the network's current ones
    std::vector<double> set_angles;
    if (n_sets > 1)
      for (int k = 0; k < n_sets; k++) {
        set_angles.insert(set_angles.end(), net->gamma.begin(), net->gamma.end());
        set_angles.insert(set_angles.end(), net->beta.begin(), net->beta.end());
      }
    const auto &cands = tune_candidates();
    const int nc = (int)cands.size();
    qtn_network *one[1] = {net};
    // per plan group: measured ms per candidate, own launch and inside a block,
    // and as a segment program (the fastest of the passes)
    struct Meas {
      double wide[8], block[8], prog;
    };
    std::map<std::pair<int, int>, Meas> meas;
    qtn_tune_report rep;
    std::memset(&rep, 0, sizeof rep);
    rep.n_candidates = nc;
    // one runtime for every candidate: the network's own streams
    Exec ex;
    ex.rt.take(net->exec->rt);
    auto give_back = [&]() { net->exec->rt.take(ex.rt); };
    constexpr int kPasses = 2;
    for (int pass = 0; pass < kPasses; pass++)
      for (int ci = 0; ci < nc; ci++) {
        int rc = build_schedule(one, 1, &ex.sched, &cands[ci], kTuneSingleWidth, n_sets);
        if (rc) {
          give_back();
          return rc;
        }
        ex.rt.forget_schedule();
        Timer tm;
        tm.on = true;
        std::vector<double> res;
        rc = run_exec(ex, {net}, d_workspace, bytes, hip_stream, 1, true, tm, res,
                      n_sets > 1 ? set_angles.data() : nullptr);
        if (rc) {
          give_back();
          return rc;
        }
        // the same groups again, each alone in one workgroup: by the candidate's
        // mapping, which runs where a schedule has no segment programs (in the
        // plan's order), and once as a program
        Timer tb, tp;
        tb.on = tp.on = true;
        char *ws = (char *)d_workspace, *desc = ex.rt.desc_base;
        const Schedule &s = ex.sched;
        const int n_single = (int)s.singles.size();
        auto alone = [&](Timer &t, int single, int range) -> int {
          int rc = t.begin(QTN_K_BLOCK, ex.rt.main, s.singles[single], 1, 0, 0, true);
          if (rc) return rc;
          QTN_HIP(launch_block_groups(
              prog_prec(s, range), ws + s.off_data, (const DevGroup *)(desc + s.off_groups),
              (const DevOp *)(desc + s.off_ops), (const int32_t *)(desc + s.off_stab),
              (const uint8_t *)(desc + s.off_uperm), (const uint32_t *)(desc + s.off_prog),
              (const int4 *)(desc + s.off_ranges), range, 1, n_sets, ex.rt.main, t.t0(), t.t1()));
          return t.end(ex.rt.main, true);
        };
        for (int i = 0; i < n_single && !rc; i++) {
          // the cell mapping, the complex128 matrix form and matrix-form
          // tiles wider than one column block only run in their own launch
          const DevGroup &dg = s.groups[s.singles[i]];
          const int prog = s.singles_range0 + i;
          if (dg.variant != kVarCell && !(dg.variant == kVarMfma && (dg.prec == 0 || dg.rls != 1)))
            rc = alone(tb, i, prog + n_single);
          if (!rc && ci == 0 && s.ranges[prog].z >= 0) rc = alone(tp, i, prog);
        }
        if (rc) {
          give_back();
          return rc;
        }
        hipError_t he = hipStreamSynchronize(ex.rt.main);
        if (he != hipSuccess) {
          give_back();
          return set_err(QTN_EDEVICE, std::string("autotune: ") + hipGetErrorString(he));
        }
        auto key_of = [&](int g) { return std::make_pair(s.group_cone[g], s.group_index[g]); };
        // a candidate only counts for the groups that ran its kernel
        auto ran = [&](int g) {
          if (cands[ci].variant == 3) return s.groups[g].variant == kVarMfma;
          if (cands[ci].variant == 4) return s.groups[g].variant == kVarCell;
          return true;
        };
        auto slot = [&](int g) -> Meas & {
          return meas.emplace(key_of(g), Meas{{-1, -1, -1, -1, -1, -1, -1, -1},
                                              {-1, -1, -1, -1, -1, -1, -1, -1}, -1})
              .first->second;
        };
        auto keep_min = [](double &dst, double v) { dst = dst < 0 ? v : std::min(dst, v); };
        for (auto &r : tm.recs) {
          if (r.kind != QTN_K_WIDE || !ran(r.group)) continue;
          float ms = 0;
          (void)hipEventElapsedTime(&ms, r.a, r.b);
          keep_min(slot(r.group).wide[ci], ms);
        }
        for (auto &r : tb.recs) {
          if (!ran(r.group)) continue;
          float ms = 0;
          (void)hipEventElapsedTime(&ms, r.a, r.b);
          keep_min(slot(r.group).block[ci], ms);
        }
        for (auto &r : tp.recs) {
          float ms = 0;
          (void)hipEventElapsedTime(&ms, r.a, r.b);
          keep_min(slot(r.group).prog, ms);
        }
      }
    for (auto &kv : meas)
      for (int ci = 0; ci < nc; ci++)
        if (kv.second.wide[ci] > 0) rep.cand_ms[ci] += kv.second.wide[ci];
    // per group: the fastest candidate for where the width rule places it;
    // the width rule's own configuration is kept unless another is faster by
    // more than the tolerance (near-ties are timing noise and would make the
    // tuned schedule differ from run to run).  Every group's timings go to
    // the tuning log.
    constexpr double kSwitchGain = 0.97;
    net->tune_log.clear();
    struct Chosen {
      Group *group;
      const Meas *meas;
      int alone, in_step;  // candidate for launches of its own, and among step launches
    };
    std::vector<Chosen> chosen;
    for (auto &kv : meas) {
      ConePlan &pl = net->plans[kv.first.first];
      Group &G = pl.groups[kv.first.second];
      const Meas &m = kv.second;
      const double *t = G.small ? m.block : m.wide;
      const int rls = std::min(G.L - 1, net->lane_sum_bits), sl = G.L - 1 - rls;
      const bool rule_stream = (int)G.ops.size() <= kStreamMaxOps && sl <= kStreamMaxSerial &&
                               sl >= 2 && net->variant != 1 &&
                               max_operand_bytes(G, pl) <= kOffset32Bytes;
      // the rule's own configuration: the cell mapping wherever it ran (own
      // launches of the per-group executors), else streaming or generic
      int rule_cell = -1;
      for (int ci = 0; ci < nc; ci++)
        if (!G.small && !net->exec->persistent && net->variant != 1 && net->variant != 2 &&
            cands[ci].variant == 4 && cands[ci].rls == kCellRuleCB && t[ci] >= 0)
          rule_cell = ci;
      int best = rule_cell;
      for (int ci = 0; ci < nc && rule_cell < 0; ci++)
        if (cands[ci].variant == (rule_stream ? 2 : 1) && (rule_stream ? cands[ci].rls == rls : true))
          if (t[ci] >= 0) best = ci;
      for (int ci = 0; ci < nc; ci++)
        if (t[ci] >= 0 && (best < 0 || t[ci] < kSwitchGain * t[best])) best = ci;
      const bool is_short = rule_cell >= 0 && m.wide[rule_cell] < kLeaveStepMs;
      if (best >= 0) chosen.push_back({&G, &m, best, is_short ? rule_cell : best});
      qtn_tune_rec tr;
      std::memset(&tr, 0, sizeof tr);
      group_features(G, pl, net->precision, tr.features);
      double mb = -1, ms_stream = -1, ms_mfma = -1;
      for (int ci = 0; ci < nc; ci++) {
        if (m.block[ci] >= 0 && (mb < 0 || m.block[ci] < mb)) mb = m.block[ci];
        if ((cands[ci].variant == 2 || cands[ci].variant == 4) && m.wide[ci] >= 0 &&
            (ms_stream < 0 || m.wide[ci] < ms_stream))
          ms_stream = m.wide[ci];
        if (cands[ci].variant == 3) ms_mfma = m.wide[ci];
      }
      if (m.prog >= 0) mb = m.prog;  // what a workgroup runs
      tr.ms[QTN_VAR_BLOCK] = mb;
      tr.ms[QTN_VAR_STREAM] = ms_stream;
      tr.ms[QTN_VAR_GENERIC] = m.wide[0];
      tr.ms[QTN_VAR_MFMA] = ms_mfma;
      net->tune_log.push_back(tr);
    }
    // the tuned schedule replaces the current one, on the same streams.  Step
    // launches run the cell mapping, and a group timed in a launch of its own is
    // mostly launch: so the short groups keep that mapping where they leave the
    // schedule (at this many angle sets) its steps.
    auto tuned = std::make_unique<Exec>();
    int rc = QTN_OK;
    for (bool in_step : {net->exec->steps, false}) {
      rep.tuned_ms = 0;
      rep.n_groups = 0;
      std::fill(rep.picks, rep.picks + nc, 0);
      for (const Chosen &c : chosen) {
        const int k = in_step ? c.in_step : c.alone;
        c.group->pick_variant = (int8_t)cands[k].variant;
        c.group->pick_rls = (int8_t)cands[k].rls;
        c.group->pred_ms = -1;
        if (c.group->small) continue;
        rep.tuned_ms += c.meas->wide[k];
        rep.picks[k]++;
        rep.n_groups++;
      }
      if (in_step && n_sets > 1) {
        Schedule many;
        if ((rc = build_schedule(one, 1, &many, nullptr, 0, n_sets))) break;
        if (many.steps.empty()) continue;
      }
      if ((rc = build_schedule(one, 1, &tuned->sched, nullptr, 0, 1, net->exec->persistent))) break;
      if (!in_step || n_sets > 1 || !tuned->sched.steps.empty()) break;
    }
    if (rc) {
      give_back();
      return rc;
    }
    tuned->persistent = net->exec->persistent;
    tuned->hybrid = net->exec->hybrid;
    tuned->dataflow = net->exec->dataflow;
    tuned->lead_per_cone = net->exec->lead_per_cone;
    tuned->steps = net->exec->steps;
    tuned->spin_limit = net->exec->spin_limit;
    tuned->rt.take(ex.rt);
    drop_batches_with(net);
    net->exec = std::move(tuned);
    net->version++;
    if (report) *report = rep;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

// FNV-1a over a group's width, summed count and operand index sets.
static uint32_t group_shape(const Group &G) {
  uint32_t h = 2166136261u;
  auto mix = [&](uint32_t v) {
    for (int k = 0; k < 4; k++) {
      h ^= (v >> (8 * k)) & 0xFFu;
      h *= 16777619u;
    }
  };
  mix((uint32_t)G.w);
  mix((uint32_t)G.L);
  mix((uint32_t)G.ops.size());
  for (const Operand &o : G.ops) {
    mix(o.mask);
    mix((uint32_t)o.level);
  }
  return h;
}

int qtn_tune_picks(const qtn_network *net, int64_t cap, qtn_tune_pick *out, int64_t *n_out) {
  if (!net || !n_out || (cap > 0 && !out)) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
  int64_t n = 0;
  for (size_t e = 0; e < net->plans.size(); e++)
    for (size_t g = 0; g < net->plans[e].groups.size(); g++, n++) {
      if (n >= cap) continue;
      const Group &G = net->plans[e].groups[g];
      qtn_tune_pick p;
      std::memset(&p, 0, sizeof p);
      p.edge = (int32_t)e;
      p.group = (int32_t)g;
      p.place = G.pick_place;
      p.variant = G.pick_variant;
      p.rls = G.pick_rls;
      p.shape = group_shape(G);
      out[n] = p;
    }
  *n_out = n;
  return QTN_OK;
}

int qtn_set_tune_picks(qtn_network *net, const qtn_tune_pick *picks, int64_t n) {
  try {
    if (!net || (n > 0 && !picks)) return set_err(QTN_EINVAL, "NULL argument");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    for (int64_t i = 0; i < n; i++) {
      const qtn_tune_pick &p = picks[i];
      if (p.edge < 0 || p.edge >= (int32_t)net->plans.size() || p.group < 0 ||
          p.group >= (int32_t)net->plans[p.edge].groups.size())
        return set_err(QTN_EINVAL, "pick " + std::to_string(i) + " names no group of this plan");
      if (group_shape(net->plans[p.edge].groups[p.group]) != p.shape)
        return set_err(QTN_EINVAL, "pick " + std::to_string(i) + " is for a different group");
      if (p.place < -1 || p.place > 1 || p.variant < -1 || p.variant > 4 || p.rls < -1 || p.rls > 5)
        return set_err(QTN_EINVAL, "pick " + std::to_string(i) + " is out of range");
    }
    for (int64_t i = 0; i < n; i++) {
      Group &G = net->plans[picks[i].edge].groups[picks[i].group];
      G.pick_place = picks[i].place;
      G.pick_variant = picks[i].variant;
      G.pick_rls = picks[i].rls;
      G.pred_ms = -1;
    }
    qtn_network *one[1] = {net};
    auto ex = std::make_unique<Exec>();
    int rc = build_schedule(one, 1, &ex->sched, nullptr, 0, 1, net->exec->persistent);
    if (rc) return rc;
    ex->rt.take(net->exec->rt);
    ex->persistent = net->exec->persistent;
    ex->hybrid = net->exec->hybrid;
    ex->dataflow = net->exec->dataflow;
    ex->lead_per_cone = net->exec->lead_per_cone;
    ex->steps = net->exec->steps;
    ex->spin_limit = net->exec->spin_limit;
    drop_batches_with(net);
    net->exec = std::move(ex);
    net->version++;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_autotune(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                 qtn_tune_report *report) {
  return autotune_sets(net, d_workspace, bytes, hip_stream, 1, report);
}

int qtn_gradient_workspace(qtn_network *net, size_t *workspace_bytes_out) {
  if (!net || !workspace_bytes_out) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned || !gradient_in_order(net))
    return qtn_angles_workspace(net, gradient_sets(net), workspace_bytes_out);
  try {
    // builds the gradient's schedule; serves as many sets of
    // qtn_contract_angles too
    int rc = QTN_OK;
    Exec *ex = angle_exec(net, gradient_sets(net), true, &rc);
    if (!ex) return rc;
    *workspace_bytes_out = std::max(ex->sched.total, form_bytes(ex->sched, false, gradient_sets(net)));
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_energy_gradient(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                        const double *gamma, const double *beta, double step, double *energy_out,
                        double *grad_gamma_out, double *grad_beta_out) {
  try {
    if (!net || !gamma || !beta || !energy_out || !grad_gamma_out || !grad_beta_out)
      return set_err(QTN_EINVAL, "NULL argument");
    if (!(step > 0.0) || !std::isfinite(step))
      return set_err(QTN_EINVAL, "step must be positive and finite");
    const int p = net->p, n = gradient_sets(net);
    // set 0: the angles; then gamma_l + h, gamma_l - h for every l, then the
    // same for beta_l
    std::vector<double> g((size_t)n * p), b((size_t)n * p), e(n);
    for (int k = 0; k < n; k++) {
      std::copy(gamma, gamma + p, g.begin() + (size_t)k * p);
      std::copy(beta, beta + p, b.begin() + (size_t)k * p);
    }
    for (int l = 0; l < p; l++) {
      g[(size_t)(1 + 2 * l) * p + l] += step;
      g[(size_t)(2 + 2 * l) * p + l] -= step;
      b[(size_t)(1 + 2 * p + 2 * l) * p + l] += step;
      b[(size_t)(2 + 2 * p + 2 * l) * p + l] -= step;
    }
    const int rc = contract_angles(net, d_workspace, bytes, hip_stream, n, gradient_in_order(net),
                                   g.data(), b.data(), nullptr, e.data(), nullptr);
    if (rc) return rc;
    *energy_out = e[0];
    for (int l = 0; l < p; l++) {
      grad_gamma_out[l] = (e[1 + 2 * l] - e[2 + 2 * l]) / (2.0 * step);
      grad_beta_out[l] = (e[1 + 2 * p + 2 * l] - e[2 + 2 * p + 2 * l]) / (2.0 * step);
    }
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_tune_angles_workspace(qtn_network *net, int32_t n_sets, size_t *bytes_out) {
  try {
    if (!net || !bytes_out) return set_err(QTN_EINVAL, "NULL argument");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    if (n_sets < 1 || n_sets > kMaxAngleSets)
      return set_err(QTN_EINVAL, "n_sets must be in 1.." + std::to_string(kMaxAngleSets));
    return tune_workspace_bytes(net, n_sets, bytes_out);
  } catch (...) {
    return exception_status();
  }
}

int qtn_autotune_angles(qtn_network *net, void *d_workspace, size_t bytes, void *hip_stream,
                        int32_t n_sets, qtn_tune_report *report) {
  return autotune_sets(net, d_workspace, bytes, hip_stream, n_sets, report);
}

int qtn_tune_log(const qtn_network *net, int64_t cap, qtn_tune_rec *out, int64_t *n_out) {
  if (!net || !n_out || (cap > 0 && !out)) return set_err(QTN_EINVAL, "NULL argument");
  const auto &lg = net->tune_log;
  const int64_t n = std::min<int64_t>(cap, (int64_t)lg.size());
  for (int64_t i = 0; i < n; i++) out[i] = lg[i];
  *n_out = (int64_t)lg.size();
  return QTN_OK;
}

int qtn_launch_log(const qtn_network *net, int64_t cap, qtn_launch_rec *out, int64_t *n_out) {
  if (!net || !n_out || (cap > 0 && !out)) return set_err(QTN_EINVAL, "NULL argument");
  const auto &lg = net->launch_log;
  const int64_t n = std::min<int64_t>(cap, (int64_t)lg.size());
  for (int64_t i = 0; i < n; i++) out[i] = lg[i];
  *n_out = (int64_t)lg.size();
  return QTN_OK;
}

int qtn_get_plan_stats(const qtn_network *net, qtn_plan_stats *out) {
  if (!net || !out) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
  qtn_plan_stats st;
  std::memset(&st, 0, sizeof st);
  for (const ConePlan &pl : net->plans) {
    st.n_buckets += pl.n_buckets;
    st.n_groups += (int64_t)pl.groups.size();
    for (const Group &G : pl.groups) st.n_wide += G.small ? 0 : 1;
    st.max_width = std::max(st.max_width, pl.max_width);
    for (int w : pl.bucket_width)
      if (w > 0 && w < 40) st.width_hist[w]++;
    st.paper_flops += pl.paper_flops * pl.n_slices;
    st.n_sliced += pl.n_slices > 1 ? 1 : 0;
    st.n_slices += pl.n_slices;
  }
  const Schedule &s = net->exec->sched;
  for (int k = 0; k < QTN_NKERNELS; k++) {
    st.bytes += s.bytes[k];
    st.flops += s.flops[k];
  }
  st.workspace = s.total;
  for (size_t gi = 0; gi < s.groups.size(); gi++) {
    const DevGroup &g = s.groups[gi];
    st.n_matrix += g.variant == kVarMfma ? 1 : 0;
    st.n_cell += g.variant == kVarCell ? 1 : 0;
    st.n_stream += g.variant == kVarStream ? 1 : 0;
    const ConePlan &pl = net->plans[s.group_cone[gi]];
    if (max_operand_bytes(pl.groups[s.group_index[gi]], pl) > kOffset32Bytes) {
      st.n_over4g++;
      st.n_over4g_generic += g.variant == kVarGeneric ? 1 : 0;
    }
  }
  *out = st;
  return QTN_OK;
}

int qtn_slice_vars(const qtn_network *net, int64_t edge, int32_t cap, int32_t *vars_out,
                   int32_t *n_out) {
  if (!net || !n_out || (cap > 0 && !vars_out)) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
  if (edge < 0 || edge >= (int64_t)net->plans.size()) return set_err(QTN_EINVAL, "edge out of range");
  const auto &sv = net->plans[edge].slice_vars;
  for (int k = 0; k < (int)sv.size() && k < cap; k++) vars_out[k] = sv[k];
  *n_out = (int32_t)sv.size();
  return QTN_OK;
}

int qtn_plan_order(const qtn_network *net, int64_t edge, int32_t *order_out) {
  if (!net || !order_out) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
  if (edge < 0 || edge >= (int64_t)net->plans.size()) return set_err(QTN_EINVAL, "edge out of range");
  const auto &o = net->plans[edge].order;
  std::copy(o.begin(), o.end(), order_out);
  return QTN_OK;
}

}  // extern "C"

// One bucket contraction of caller-given tensors: a one-group schedule whose
// descriptors address the caller's data buffer.
namespace {

// The bucket's descriptors in device memory of its own.  A small bucket's call
// is the upload of its descriptors and one kernel (the fixed contraction over
// four indices of size 16: 10.6 us a call with the upload, 7.3 without); a caller that repeats it need not
// upload them again, since they depend on the plan alone.  The copy is made
// after kCalls calls, when the uploads so far have cost about what it does
// (allocation, release): a bucket that runs a few times pays nothing for it.
// Until the copy is known to be complete, on a stream of another device, and
// where the allocation failed, a call uploads into its workspace.
class BucketDesc {
 public:
  ~BucketDesc() {
    RelaxedCapture relax;
    if (ev_) (void)hipEventDestroy(ev_);
    desc_free(dev_, bytes_);  // waits for the kernels that read it
  }
  // The device copy if a launch on st may read it, else null.
  char *get(hipStream_t st) {
    if (state_.load(std::memory_order_acquire) == kReady) return on_device(st) ? dev_ : nullptr;
    std::lock_guard<std::mutex> lk(lock_);
    if (state_.load(std::memory_order_relaxed) != kUploading) return nullptr;
    RelaxedCapture relax;
    const hipError_t e = hipEventQuery(ev_);
    if (e == hipSuccess) state_.store(kReady, std::memory_order_release);
    else (void)hipGetLastError();
    return e == hipSuccess && on_device(st) ? dev_ : nullptr;
  }
  // Counts a call that uploaded; starts the copy on st when it is due.
  void uploaded(const std::vector<char> &blob, hipStream_t st) {
    if (state_.load(std::memory_order_relaxed) != kNone) return;
    std::lock_guard<std::mutex> lk(lock_);
    if (state_.load(std::memory_order_relaxed) != kNone || ++calls_ < kCalls) return;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return;
    }
    RelaxedCapture relax;
    bool none;
    if (stream_device(st, &device_)) dev_ = desc_alloc(bytes_ = blob.size(), &none);
    const bool ok = dev_ && hipEventCreateWithFlags(&ev_, hipEventDisableTiming) == hipSuccess &&
                    hipMemcpyAsync(dev_, blob.data(), blob.size(), hipMemcpyHostToDevice, st) == hipSuccess &&
                    hipEventRecord(ev_, st) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    state_.store(ok ? kUploading : kOff, std::memory_order_release);
  }

 private:
  enum State { kNone, kUploading, kReady, kOff };
  static constexpr int kCalls = 16;
  // Allocations and event queries of this thread do not disturb a stream
  // capture of another one.
  struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };
  // The device st runs on; allocations go to the current one, so only where
  // that is the same.
  static bool stream_device(hipStream_t st, int *dev) {
    int cur = -1;
    hipDevice_t d = -1;
    if (hipGetDevice(&cur) != hipSuccess || (st && hipStreamGetDevice(st, &d) != hipSuccess)) {
      (void)hipGetLastError();
      return false;
    }
    *dev = cur;
    return !st || d == cur;
  }
  bool on_device(hipStream_t st) const {
    int d;
    return stream_device(st, &d) && d == device_;
  }
  std::mutex lock_;
  std::atomic<int> state_{kNone};
  int calls_ = 0, device_ = -1;
  char *dev_ = nullptr;
  size_t bytes_ = 0;
  hipEvent_t ev_ = nullptr;
};

}  // namespace

struct qtn_bucket {
  Schedule s;              // one group; s.desc_blob holds its descriptors
  DevGroup hg;             // host copy of the group record
  size_t off_groups = 0, off_ops = 0, off_stab = 0, off_uperm = 0;
  int64_t data_bytes = 0;  // end of the last tensor in the data buffer
  double bytes = 0, flops = 0;
  hipEvent_t ev[2] = {nullptr, nullptr};  // timed runs: start/stop of the dispatch
  mutable BucketDesc dev;
  ~qtn_bucket() {
    for (hipEvent_t &e : ev)
      if (e) (void)hipEventDestroy(e);
  }
};

namespace {

// Runs the bucket's kernel on the caller's data buffer, its descriptors
// uploaded to `desc` (device) unless they are in device memory already.
// may_alloc: the call may start that copy.
// t0, t1: events attached to the kernel's dispatch (timed runs), or null.
int bucket_run(const qtn_bucket *b, void *d_data, size_t data_bytes, char *desc, hipStream_t st,
               bool may_alloc, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr) {
  if ((int64_t)data_bytes < b->data_bytes)
    return set_err(QTN_ENOMEM, "data buffer smaller than the bucket's tensors");
  if (((uintptr_t)d_data & 255u) != 0) return set_err(QTN_EINVAL, "data buffer not 256-byte aligned");
  char *const dev = b->dev.get(st);
  if (dev)
    desc = dev;
  else
    QTN_HIP(hipMemcpyAsync(desc, b->s.desc_blob.data(), b->s.desc_blob.size(), hipMemcpyHostToDevice, st));
  QTN_HIP(launch_wide_group(b->hg, d_data, (const DevGroup *)(desc + b->off_groups),
                            (const DevOp *)(desc + b->off_ops), (const int32_t *)(desc + b->off_stab),
                            (const uint8_t *)(desc + b->off_uperm), 0, 1, st, t0, t1));
  if (!dev && may_alloc) b->dev.uploaded(b->s.desc_blob, st);
  return QTN_OK;
}

}  // namespace

extern "C" {

int qtn_bucket_plan(int32_t n_ops, const int32_t *ranks, const int32_t *labels,
                    const int64_t *offsets, int32_t n_out, const int32_t *out_labels,
                    int64_t out_offset, int32_t precision, int32_t variant, int32_t knob,
                    qtn_bucket **out) {
  if (!ranks || !labels || !offsets || !out || (n_out > 0 && !out_labels))
    return set_err(QTN_EINVAL, "NULL argument");
  if (n_ops < 1 || n_ops > 64) return set_err(QTN_EINVAL, "n_ops must be in 1..64");
  if (n_out < 0 || n_out > kMaxWidth) return set_err(QTN_EINVAL, "n_out must be in 0..32");
  if (precision != QTN_C128 && precision != QTN_C64)
    return set_err(QTN_EINVAL, "precision must be QTN_C128 or QTN_C64");
  if (variant < 0 || variant > 4) return set_err(QTN_EINVAL, "variant must be 0..4");
  try {
    // union order: the summed labels ascending, then the output labels
    std::map<int32_t, int> seen;  // label -> union position (-1 until placed)
    int64_t n_lab = 0;
    for (int k = 0; k < n_ops; k++) {
      if (ranks[k] < 0 || ranks[k] > kMaxWidth) return set_err(QTN_EINVAL, "operand rank out of range");
      for (int j = 0; j < ranks[k]; j++) seen[labels[n_lab + j]] = -1;
      n_lab += ranks[k];
    }
    for (int j = 0; j < n_out; j++) {
      auto it = seen.find(out_labels[j]);
      if (it == seen.end()) return set_err(QTN_EINVAL, "output label held by no operand");
      if (it->second != -1) return set_err(QTN_EINVAL, "repeated output label");
      it->second = -2;  // kept
    }
    int L = 0;
    for (auto &kv : seen)
      if (kv.second == -1) kv.second = L++;
    const int w = L + n_out;
    if (L < 1) return set_err(QTN_EINVAL, "no summed label: a bucket sums at least one index");
    if (L > kMaxLevels) return set_err(QTN_ERANGE, "more than 8 summed labels");
    if (w > kMaxWidth) return set_err(QTN_ERANGE, "union of more than 32 labels");
    for (int j = 0; j < n_out; j++) seen[out_labels[j]] = L + j;
    auto qb = std::make_unique<qtn_bucket>();
    const int64_t es = precision == QTN_C64 ? 8 : 16;
    ConePlan pl;
    Group G;
    G.w = w;
    G.L = L;
    G.prec = (int8_t)precision;
    std::vector<std::pair<int64_t, int64_t>> ranges;  // byte ranges of the inputs
    n_lab = 0;
    for (int k = 0; k < n_ops; k++) {
      uint32_t mask = 0;
      int prev = -1;
      for (int j = 0; j < ranks[k]; j++) {
        const int pos = seen[labels[n_lab + j]];
        if (pos <= prev)
          return set_err(QTN_EINVAL, "operand " + std::to_string(k) +
                                         ": labels repeated or not in union order (summed labels "
                                         "ascending, then the output labels in order)");
        prev = pos;
        mask |= 1u << pos;
      }
      n_lab += ranks[k];
      const int64_t size = es << ranks[k];
      if (offsets[k] < 0 || offsets[k] % es) return set_err(QTN_EINVAL, "operand offset not aligned");
      ranges.push_back({offsets[k], offsets[k] + size});
      qb->data_bytes = std::max(qb->data_bytes, offsets[k] + size);
      Tensor t;
      t.vars.assign(ranks[k], 0);
      t.offset = offsets[k];
      t.prec = (int8_t)precision;
      pl.tensors.push_back(t);
      // level: after the summed labels below the operand's lowest one
      const uint32_t summed = mask & ((1u << L) - 1u);
      const int level = summed ? __builtin_ctz(summed) : L - 1;
      G.ops.push_back({k, mask, level});
    }
    std::stable_sort(G.ops.begin(), G.ops.end(),
                     [](const Operand &a, const Operand &b) { return a.level < b.level; });
    const int64_t osize = es << n_out;
    if (out_offset < 0 || out_offset % es) return set_err(QTN_EINVAL, "output offset not aligned");
    for (auto &r : ranges)
      if (r.first < out_offset + osize && out_offset < r.second)
        return set_err(QTN_EINVAL, "output overlaps an operand");
    qb->data_bytes = std::max(qb->data_bytes, out_offset + osize);
    Tensor to;
    to.vars.assign(n_out, 0);
    to.offset = out_offset;
    to.prec = (int8_t)precision;
    pl.tensors.push_back(to);
    G.out_tensor = n_ops;
    GroupEnv env;
    env.out_off = out_offset;
    env.var_req = variant;
    env.rls_req = knob > 0 ? knob : (variant == 4 ? kCellRuleCB : 2);
    Schedule &s = qb->s;
    int rc = describe_group(G, pl, env, s, &qb->hg, &qb->bytes, &qb->flops);
    if (rc) return rc;
    if (qb->hg.n_units == 0 || qb->hg.n_units > 0x7FFFFFFFu)
      return set_err(QTN_ERANGE, "too many units for one launch");
    qb->hg.op_begin = 0;
    s.groups.assign(1, qb->hg);
    qb->off_groups = 0;
    qb->off_ops = align_up(sizeof(DevGroup), 256);
    qb->off_stab = align_up(qb->off_ops + sizeof(DevOp) * s.ops.size(), 256);
    qb->off_uperm = align_up(qb->off_stab + sizeof(int32_t) * s.stab.size(), 256);
    s.desc_blob.assign(align_up(qb->off_uperm + s.uperm.size(), 256), 0);
    std::memcpy(s.desc_blob.data() + qb->off_groups, s.groups.data(), sizeof(DevGroup));
    std::memcpy(s.desc_blob.data() + qb->off_ops, s.ops.data(), sizeof(DevOp) * s.ops.size());
    if (!s.stab.empty())
      std::memcpy(s.desc_blob.data() + qb->off_stab, s.stab.data(), sizeof(int32_t) * s.stab.size());
    std::memcpy(s.desc_blob.data() + qb->off_uperm, s.uperm.data(), s.uperm.size());
    *out = qb.release();
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_bucket_get_info(const qtn_bucket *b, qtn_bucket_info *out) {
  if (!b || !out) return set_err(QTN_EINVAL, "NULL argument");
  qtn_bucket_info r;
  std::memset(&r, 0, sizeof r);
  r.w = b->hg.w;
  r.L = b->hg.L;
  r.n_ops = b->hg.n_ops;
  r.variant = b->hg.variant;
  r.knob = b->hg.variant == kVarStream || b->hg.variant == kVarCell || b->hg.variant == kVarMfma ? b->hg.rls : 0;
  r.serial = b->hg.variant == kVarStream || b->hg.variant == kVarCell ? b->hg.sl : 0;
  r.n_units = b->hg.n_units;
  r.bytes = b->bytes;
  r.flops = b->flops;
  r.workspace_bytes = b->s.desc_blob.size();
  r.data_bytes = b->data_bytes;
  *out = r;
  return QTN_OK;
}

int qtn_bucket_contract(const qtn_bucket *b, void *d_data, size_t data_bytes, void *d_workspace,
                        size_t ws_bytes, void *hip_stream) {
  if (!b || !d_data || !d_workspace) return set_err(QTN_EINVAL, "NULL argument");
  if (ws_bytes < b->s.desc_blob.size()) return set_err(QTN_ENOMEM, "workspace too small");
  if (((uintptr_t)d_workspace & 255u) != 0) return set_err(QTN_EINVAL, "workspace not 256-byte aligned");
  try {
    return bucket_run(b, d_data, data_bytes, (char *)d_workspace, (hipStream_t)hip_stream, true);
  } catch (...) {
    return exception_status();
  }
}

int qtn_bucket_contract_timed(qtn_bucket *b, void *d_data, size_t data_bytes, void *d_workspace,
                              size_t ws_bytes, void *hip_stream, double *kernel_ms) {
  if (!b || !d_data || !d_workspace || !kernel_ms) return set_err(QTN_EINVAL, "NULL argument");
  if (ws_bytes < b->s.desc_blob.size()) return set_err(QTN_ENOMEM, "workspace too small");
  if (((uintptr_t)d_workspace & 255u) != 0) return set_err(QTN_EINVAL, "workspace not 256-byte aligned");
  try {
    for (hipEvent_t &e : b->ev)
      if (!e) QTN_HIP(hipEventCreate(&e));
    const int rc = bucket_run(b, d_data, data_bytes, (char *)d_workspace, (hipStream_t)hip_stream,
                              true, b->ev[0], b->ev[1]);
    if (rc) return rc;
    QTN_HIP(hipEventSynchronize(b->ev[1]));
    float ms = 0;
    QTN_HIP(hipEventElapsedTime(&ms, b->ev[0], b->ev[1]));
    *kernel_ms = ms;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_bucket_contract_noalloc(const qtn_bucket *b, void *d_data, size_t data_bytes,
                                void *hip_stream) {
  if (!b || !d_data) return set_err(QTN_EINVAL, "NULL argument");
  if (b->s.desc_blob.size() > kScratchBytes)
    return set_err(QTN_ERANGE, "bucket descriptors (" + std::to_string(b->s.desc_blob.size()) +
                                   " bytes) exceed the " + std::to_string(kScratchBytes) +
                                   "-byte device scratch");
  try {
    void *scr = nullptr;
    QTN_HIP(scratch_address(&scr));
    return bucket_run(b, d_data, data_bytes, (char *)scr, (hipStream_t)hip_stream, false);
  } catch (...) {
    return exception_status();
  }
}

void qtn_bucket_free(qtn_bucket *b) { delete b; }

int qtn_bucket_widths(const qtn_network *net, int64_t edge, int32_t *widths_out) {
  if (!net || !widths_out) return set_err(QTN_EINVAL, "NULL argument");
  if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
  if (edge < 0 || edge >= (int64_t)net->plans.size()) return set_err(QTN_EINVAL, "edge out of range");
  const auto &w = net->plans[edge].bucket_width;
  std::copy(w.begin(), w.end(), widths_out);
  return QTN_OK;
}

}  // extern "C"

struct qtn_costmodel {
  std::vector<float> params, m1, m2;
  float mean[kMlpIn], inv_std[kMlpIn];
  bool norm_set = false;
  int step = 0;
};

namespace {

// Standardised features.
void mlp_normalize(const qtn_costmodel *cm, const float *x, int64_t n, float *out) {
  for (int64_t i = 0; i < n; i++)
    for (int k = 0; k < kMlpIn; k++)
      out[i * kMlpIn + k] = (x[i * kMlpIn + k] - cm->mean[k]) * cm->inv_std[k];
}

int mlp_upload_inputs(const qtn_costmodel *cm, const float *x, int64_t n, const MlpBuffers &b,
                      bool normalize, hipStream_t s, std::vector<float> &stage) {
  stage.assign(x, x + n * kMlpIn);
  if (normalize) mlp_normalize(cm, x, n, stage.data());
  QTN_HIP(hipMemcpyAsync(b.x, stage.data(), sizeof(float) * n * kMlpIn, hipMemcpyHostToDevice, s));
  QTN_HIP(hipMemcpyAsync(b.params, cm->params.data(), sizeof(float) * kMlpParams,
                         hipMemcpyHostToDevice, s));
  return QTN_OK;
}

int mlp_check_ws(int64_t n, void *ws, size_t bytes) {
  if (n < 1) return set_err(QTN_EINVAL, "need at least one sample");
  if (!ws) return set_err(QTN_EINVAL, "workspace is NULL");
  if (bytes < mlp_buffers(ws, n).bytes) return set_err(QTN_ENOMEM, "cost-model workspace too small");
  return QTN_OK;
}

}  // namespace

extern "C" {

int qtn_costmodel_create(const float *params, qtn_costmodel **out) {
  if (!params || !out) return set_err(QTN_EINVAL, "NULL argument");
  try {
    auto *cm = new qtn_costmodel();
    cm->params.assign(params, params + kMlpParams);
    cm->m1.assign(kMlpParams, 0.0f);
    cm->m2.assign(kMlpParams, 0.0f);
    for (int k = 0; k < kMlpIn; k++) {
      cm->mean[k] = 0.0f;
      cm->inv_std[k] = 1.0f;
    }
    *out = cm;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_costmodel_params(const qtn_costmodel *cm, float *params_out) {
  if (!cm || !params_out) return set_err(QTN_EINVAL, "NULL argument");
  std::copy(cm->params.begin(), cm->params.end(), params_out);
  return QTN_OK;
}

int qtn_costmodel_normalization(const qtn_costmodel *cm, float *mean_out, float *inv_std_out) {
  if (!cm || !mean_out || !inv_std_out) return set_err(QTN_EINVAL, "NULL argument");
  std::copy(cm->mean, cm->mean + kMlpIn, mean_out);
  std::copy(cm->inv_std, cm->inv_std + kMlpIn, inv_std_out);
  return QTN_OK;
}

int qtn_costmodel_workspace(int64_t n, size_t *bytes_out) {
  if (n < 1 || !bytes_out) return set_err(QTN_EINVAL, "bad arguments");
  *bytes_out = mlp_buffers(nullptr, n).bytes;
  return QTN_OK;
}

int qtn_costmodel_train(qtn_costmodel *cm, const float *x, const double *ms, int64_t n,
                        int32_t epochs, float lr, void *d_ws, size_t bytes, void *hip_stream,
                        float *loss_history) {
  try {
    if (!cm || !x || !ms || epochs < 1 || !(lr > 0)) return set_err(QTN_EINVAL, "bad arguments");
    int rc = mlp_check_ws(n, d_ws, bytes);
    if (rc) return rc;
    if (!cm->norm_set) {
      for (int k = 0; k < kMlpIn; k++) {
        double s = 0, s2 = 0;
        for (int64_t i = 0; i < n; i++) {
          s += x[i * kMlpIn + k];
          s2 += (double)x[i * kMlpIn + k] * x[i * kMlpIn + k];
        }
        const double mu = s / n, var = std::max(0.0, s2 / n - mu * mu);
        cm->mean[k] = (float)mu;
        cm->inv_std[k] = (float)(1.0 / std::max(1e-3, std::sqrt(var)));
      }
      cm->norm_set = true;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    const MlpBuffers b = mlp_buffers(d_ws, n);
    // parameters, moments, inputs, targets and mask go up in one copy
    std::vector<float> stage(b.m + n * kMlpOut - b.params);
    std::copy(cm->params.begin(), cm->params.end(), stage.data());
    std::copy(cm->m1.begin(), cm->m1.end(), stage.data() + (b.m1 - b.params));
    std::copy(cm->m2.begin(), cm->m2.end(), stage.data() + (b.m2 - b.params));
    mlp_normalize(cm, x, n, stage.data() + (b.x - b.params));
    float *t = stage.data() + (b.t - b.params), *m = stage.data() + (b.m - b.params);
    for (int64_t q = 0; q < n * kMlpOut; q++) {
      m[q] = ms[q] > 0 ? 1.0f : 0.0f;
      t[q] = ms[q] > 0 ? (float)std::log(ms[q]) : 0.0f;
    }
    std::vector<float> hist(epochs);
    hipError_t he = hipMemcpyAsync(b.params, stage.data(), sizeof(float) * stage.size(),
                                   hipMemcpyHostToDevice, s);
    int step = cm->step;
    for (int e = 0; e < epochs && he == hipSuccess; e++) {
      const int slot = e % kMlpLosses;
      he = mlp_train_step(b, (int)n, ++step, lr, b.loss + slot, s);
      if (he == hipSuccess && (slot == kMlpLosses - 1 || e == epochs - 1))
        he = hipMemcpyAsync(hist.data() + (e - slot), b.loss, sizeof(float) * (slot + 1),
                            hipMemcpyDeviceToHost, s);
    }
    const size_t back = b.m2 + kMlpParams - b.params;
    if (he == hipSuccess)
      he = hipMemcpyAsync(stage.data(), b.params, sizeof(float) * back, hipMemcpyDeviceToHost, s);
    // also after an error: nothing queued may outlive the host buffers
    const hipError_t se = hipStreamSynchronize(s);
    if (he == hipSuccess) he = se;
    if (he != hipSuccess)
      return set_err(QTN_EDEVICE, std::string("cost-model training: ") + hipGetErrorString(he));
    if (loss_history) std::copy(hist.begin(), hist.end(), loss_history);
    std::copy(stage.data(), stage.data() + kMlpParams, cm->params.begin());
    std::copy(stage.data() + (b.m1 - b.params), stage.data() + (b.m1 - b.params) + kMlpParams,
              cm->m1.begin());
    std::copy(stage.data() + (b.m2 - b.params), stage.data() + (b.m2 - b.params) + kMlpParams,
              cm->m2.begin());
    cm->step = step;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_costmodel_predict(const qtn_costmodel *cm, const float *x, int64_t n, void *d_ws,
                          size_t bytes, void *hip_stream, float *y_out) {
  try {
    if (!cm || !x || !y_out) return set_err(QTN_EINVAL, "NULL argument");
    int rc = mlp_check_ws(n, d_ws, bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)hip_stream;
    const MlpBuffers b = mlp_buffers(d_ws, n);
    std::vector<float> stage, y(n * kMlpOut);
    if ((rc = mlp_upload_inputs(cm, x, n, b, true, s, stage))) return rc;
    QTN_HIP(mlp_forward(b, (int)n, s));
    QTN_HIP(hipMemcpyAsync(y.data(), b.y, sizeof(float) * n * kMlpOut, hipMemcpyDeviceToHost, s));
    QTN_HIP(hipStreamSynchronize(s));
    std::copy(y.begin(), y.end(), y_out);
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_costmodel_grad(const qtn_costmodel *cm, const float *x, const float *t, const float *m,
                       int64_t n, void *d_ws, size_t bytes, void *hip_stream, float *loss_out,
                       float *grad_out) {
  try {
    if (!cm || !x || !t || !m || !loss_out || !grad_out) return set_err(QTN_EINVAL, "NULL argument");
    int rc = mlp_check_ws(n, d_ws, bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)hip_stream;
    const MlpBuffers b = mlp_buffers(d_ws, n);
    std::vector<float> stage, g(kMlpParams);
    if ((rc = mlp_upload_inputs(cm, x, n, b, false, s, stage))) return rc;
    QTN_HIP(hipMemcpyAsync(b.t, t, sizeof(float) * n * kMlpOut, hipMemcpyHostToDevice, s));
    QTN_HIP(hipMemcpyAsync(b.m, m, sizeof(float) * n * kMlpOut, hipMemcpyHostToDevice, s));
    QTN_HIP(mlp_loss_grad(b, (int)n, s));
    float loss = 0;
    QTN_HIP(hipMemcpyAsync(g.data(), b.grad, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost, s));
    QTN_HIP(hipMemcpyAsync(&loss, b.loss, sizeof(float), hipMemcpyDeviceToHost, s));
    QTN_HIP(hipStreamSynchronize(s));
    *loss_out = loss;
    std::copy(g.begin(), g.end(), grad_out);
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_costmodel_adam_step(qtn_costmodel *cm, const float *grad, float lr, void *d_ws,
                            size_t bytes, void *hip_stream) {
  try {
    if (!cm || !grad || !(lr > 0)) return set_err(QTN_EINVAL, "bad arguments");
    int rc = mlp_check_ws(1, d_ws, bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)hip_stream;
    const MlpBuffers b = mlp_buffers(d_ws, 1);
    QTN_HIP(hipMemcpyAsync(b.params, cm->params.data(), sizeof(float) * kMlpParams, hipMemcpyHostToDevice, s));
    QTN_HIP(hipMemcpyAsync(b.grad, grad, sizeof(float) * kMlpParams, hipMemcpyHostToDevice, s));
    QTN_HIP(hipMemcpyAsync(b.m1, cm->m1.data(), sizeof(float) * kMlpParams, hipMemcpyHostToDevice, s));
    QTN_HIP(hipMemcpyAsync(b.m2, cm->m2.data(), sizeof(float) * kMlpParams, hipMemcpyHostToDevice, s));
    QTN_HIP(mlp_adam(b, cm->step + 1, lr, s));
    std::vector<float> p(kMlpParams), a(kMlpParams), q2(kMlpParams);
    QTN_HIP(hipMemcpyAsync(p.data(), b.params, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost, s));
    QTN_HIP(hipMemcpyAsync(a.data(), b.m1, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost, s));
    QTN_HIP(hipMemcpyAsync(q2.data(), b.m2, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost, s));
    QTN_HIP(hipStreamSynchronize(s));
    cm->params.swap(p);
    cm->m1.swap(a);
    cm->m2.swap(q2);
    cm->step++;
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

int qtn_apply_costmodel(qtn_network *net, const qtn_costmodel *cm, void *d_ws, size_t bytes,
                        void *hip_stream, int32_t *counts_out) {
  try {
    if (!net || !cm) return set_err(QTN_EINVAL, "NULL argument");
    if (!net->planned) return set_err(QTN_ESTATE, "qtn_plan has not been called");
    std::vector<float> feats;
    std::vector<Group *> gs;
    std::vector<const ConePlan *> gp;
    for (ConePlan &pl : net->plans)
      for (Group &G : pl.groups) {
        float f[kNumFeatures];
        group_features(G, pl, net->precision, f);
        feats.insert(feats.end(), f, f + kNumFeatures);
        gs.push_back(&G);
        gp.push_back(&pl);
      }
    const int64_t n = (int64_t)gs.size();
    std::vector<float> y(n * kMlpOut);
    int rc = qtn_costmodel_predict(cm, feats.data(), n, d_ws, bytes, hip_stream, y.data());
    if (rc) return rc;
    int32_t counts[4] = {0, 0, 0, 0};
    const bool steps = net->exec->steps && !net->exec->sched.steps.empty();
    for (int64_t i = 0; i < n; i++) {
      Group &G = *gs[i];
      const float *p = &y[i * kMlpOut];
      // placement stays with the width rule: a group's time inside a
      // workgroup segment is not the time of the same group alone in a
      // one-workgroup launch, which is what was measured.  Groups that get
      // their own launch take the kernel with the lowest predicted time, the
      // matrix form only where the group has one.
      G.pick_place = -1;
      if (G.small) {
        G.pick_variant = -1;
        G.pick_rls = -1;
        G.pred_ms = std::exp(p[QTN_VAR_BLOCK]);
        counts[QTN_VAR_BLOCK]++;
        continue;
      }
      int best = p[QTN_VAR_STREAM] <= p[QTN_VAR_GENERIC] ? QTN_VAR_STREAM : QTN_VAR_GENERIC;
      if (G.prec == 1 && p[QTN_VAR_MFMA] < p[best] && gemm_shape(G, *gp[i], nullptr))
        best = QTN_VAR_MFMA;
      // step launches run the cell mapping: the times are those of launches
      // of their own, and only a long group is worth one
      if (steps && p[QTN_VAR_STREAM] < std::log(kLeaveStepMs)) best = QTN_VAR_STREAM;
      G.pred_ms = std::exp(p[best]);
      counts[best]++;
      // the streaming family: the cell mapping where it fits, else the
      // lane-sum streaming mapping (the planner falls back by itself)
      G.pick_variant = best == QTN_VAR_STREAM ? 4 : (best == QTN_VAR_MFMA ? 3 : 1);
      G.pick_rls = best == QTN_VAR_STREAM ? kCellRuleCB : 2;
    }
    qtn_network *one[1] = {net};
    auto ex = std::make_unique<Exec>();
    if ((rc = build_schedule(one, 1, &ex->sched, nullptr, 0, 1, net->exec->persistent))) return rc;
    ex->rt.take(net->exec->rt);
    ex->persistent = net->exec->persistent;
    ex->hybrid = net->exec->hybrid;
    ex->dataflow = net->exec->dataflow;
    ex->lead_per_cone = net->exec->lead_per_cone;
    ex->steps = net->exec->steps;
    ex->spin_limit = net->exec->spin_limit;
    drop_batches_with(net);
    net->exec = std::move(ex);
    net->version++;
    if (counts_out) std::copy(counts, counts + 4, counts_out);
    return QTN_OK;
  } catch (...) {
    return exception_status();
  }
}

void qtn_costmodel_free(qtn_costmodel *cm) { delete cm; }

void qtn_network_free(qtn_network *net) {
  if (!net) return;
  drop_batches_with(net);
  delete net;
}

}  // extern "C"
