// md_engine.hip -- host runtime of the batched NEMD micro-solve: builds the
// flattened device layout of many channel systems, runs the step loop as
// direct launches or replays of a captured HIP graph, and reduces results.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <numeric>

#include "engine.h"
#include "md_kernels.h"
#include "series.h"

namespace hmd {

namespace {

constexpr double kTwo32 = 4294967296.0;

inline int blocks_for(int64_t n, int tpb) { return int((n + tpb - 1) / tpb); }

StateRef state_ref(hmd_batch* b, int which) {
  double** s = b->d_state[which];
  return StateRef{s[0], s[1], s[2], s[3], s[4], s[5]};
}

StepConst step_const(const hmd_batch* b, bool thermostat, bool energy) {
  const hmd_md_params& P = b->P;
  StepConst K{};
  K.dt = P.dt;
  K.hdt = 0.5 * P.dt;
  K.dt_tau = P.dt / P.tau_T;
  K.T0 = P.T0;
  K.n_equil = P.n_equil;
  K.rc2 = float(P.rc * P.rc);
  K.eps_wf = float(P.eps_wf);
  K.sig2_wf = float(P.sigma_wf * P.sigma_wf);
  const double ir6 = 1.0 / std::pow(P.rc, 6.0);
  K.ush_ff = float(4.0 * (ir6 * ir6 - ir6));
  const double sw6 = std::pow(P.sigma_wf / P.rc, 6.0);
  K.ush_wf = float(4.0 * P.eps_wf * (sw6 * sw6 - sw6));
  K.half_skin2 = float(0.25 * b->skin * b->skin);
  K.axis = P.thermo_axis;
  K.nb = int(b->nser);
  K.B = b->ser_B;
  K.r = b->ser_r;
  K.thermo_on = thermostat ? 1 : 0;
  K.bins_on = 1;
  K.energy_on = energy ? 1 : 0;
  K.press_on = P.pressure ? 1 : 0;
  return K;
}

template <typename T>
int dalloc(hmd_ctx* ctx, T** p, int64_t n) {
  HMD_HIP(ctx, hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * size_t(std::max<int64_t>(n, 1))));
  return HMD_OK;
}

// 3-D Morton code: bits of x, y, z interleaved (x lowest).
uint64_t morton3(uint32_t x, uint32_t y, uint32_t z) {
  uint64_t m = 0;
  for (int b = 0; b < 21; ++b) {
    m |= uint64_t((x >> b) & 1u) << (3 * b);
    m |= uint64_t((y >> b) & 1u) << (3 * b + 1);
    m |= uint64_t((z >> b) & 1u) << (3 * b + 2);
  }
  return m;
}

uint32_t fix_axis_host(double v, double scale) {
  double t = v * scale;
  t = t < 0.0 ? 0.0 : (t > 4294967295.0 ? 4294967295.0 : t);
  return uint32_t(t);
}

// Launches of one kind, optionally timed.  Direct launches: HIP events
// around each kernel (marks).  Captured graphs, where events cannot be timed:
// stamp kernels writing the device wall clock into b->d_stamps, one before a
// stamped step's first kernel and one after each of its kernels; spans
// records (kernel, stamp before, stamp after).
struct Launcher {
  hmd_batch* b;
  hipStream_t s;
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>>* marks;  // null: untimed
  int next_ev = 0;
  std::vector<std::array<int, 3>>* spans = nullptr;  // non-null: stamp mode
  int next_stamp = 0, last_stamp = -1;
  const int* flag = nullptr;  // stamp mode: rebuild flags, recorded in each stamp's bit 63
  StepRef R{nullptr, 0};      // stamp mode: the step being stamped

  void stamp() {
    hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, s, b->d_stamps + next_stamp, flag, R);
    last_stamp = next_stamp++;
  }
  void begin(int k) {
    if (spans) {
      if (last_stamp < 0) stamp();
      spans->push_back({k, last_stamp, next_stamp});
      return;
    }
    if (!marks) return;
    hipEvent_t e0 = b->ev[next_ev++], e1 = b->ev[next_ev++];
    (void)hipEventRecord(e0, s);
    marks->push_back({k, {e0, e1}});
  }
  void end() {
    if (spans) {
      stamp();
      return;
    }
    if (!marks) return;
    (void)hipEventRecord(marks->back().second.second, s);
  }
};

TileBuild tile_build(hmd_batch* b, StateRef from, StateRef to, const int* tag_from, int* tag_to, int global_out) {
  const float rl2 = float((b->P.rc + b->skin) * (b->P.rc + b->skin));
  return {b->list_cap, b->d_tiles,  b->d_sims,  b->d_slot_cell, b->d_pfix,    b->d_pos4, b->d_start,
          b->d_ncount, b->d_wstart, b->d_wcount, b->d_list,     b->d_nlist,   b->d_tilerec, from,
          to,          tag_from,    tag_to,      b->d_flag + 2, rl2,          global_out || b->force_gather ? 0 : b->stage_cap};
}

// Pair-list build (after a reorder into `from`: the build copies the state
// back into `to`; from == to copies nothing).
void launch_build(hmd_batch* b, hipStream_t s, const int* flag, StepRef R, StateRef from, StateRef to,
                  const int* tag_from, int* tag_to, int global_out) {
  const int nt = int(b->ntot), tpb = b->tpb, nb = blocks_for(nt, tpb);
  const float rl2 = float((b->P.rc + b->skin) * (b->P.rc + b->skin));
  if (b->path == 2) {
    hipLaunchKernelGGL(b->uniform ? k_build_tiles<1> : k_build_tiles<0>, dim3(b->ntiles), dim3(TILE_THREADS), 0, s, nt,
                       b->list_ld, tile_build(b, from, to, tag_from, tag_to, global_out), flag, R);
    return;
  }
  hipLaunchKernelGGL(k_build_list, dim3(nb), dim3(tpb), 0, s, nt, b->list_ld, b->list_cap, b->d_sims,
                     b->d_atom_sim, b->d_slot_cell, b->d_pfix, b->d_start, b->d_ncount, b->d_wstart, b->d_wcount,
                     b->d_list, b->d_nlist, from, to, tag_from, tag_to, b->d_flag + 2, flag, R, rl2);
}

// Counting sort of the current state by cell (flag null: unconditional), and
// unless left to the caller the pair lists.
void enqueue_sort(hmd_batch* b, Launcher& L, const StepConst& K, const int* flag, StepRef R, bool with_list = true) {
  hipStream_t s = L.s;
  const int nt = int(b->ntot), tpb = b->tpb, nb = blocks_for(nt, tpb);
  if (b->path == 0) {
    const int src = b->cur, dst = 1 - b->cur;
    if (!flag && R.base == nullptr && R.k < 0) {  // keys for a sort outside a time step
      hipLaunchKernelGGL((k_integrate<0, 0>), dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim,
                         state_ref(b, src), b->d_f4, b->d_key, b->d_count, b->d_rank, b->d_pfix, b->d_pbuild,
                         b->d_flag, b->acc, b->d_dstate, StepRef{nullptr, 0}, K, b->S == 1);
    }
    L.begin(K_SCAN);
    hipLaunchKernelGGL(k_scan, dim3(b->S), dim3(1024), 0, s, b->d_sims, b->d_count, b->d_start, b->d_ncount,
                       nullptr, R);
    L.end();
    L.begin(K_SCATTER);
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(tpb), 0, s, nt, b->d_key, b->d_start, b->d_rank, b->d_perm,
                       nullptr, R);
    L.end();
    L.begin(K_REORDER);
    hipLaunchKernelGGL(k_reorder<0>, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_cell_sim, b->d_key,
                       b->d_start, b->d_ncount, b->d_perm, 0u, state_ref(b, src), state_ref(b, dst), b->d_tag[src],
                       b->d_tag[dst], b->d_pos4, b->d_pfix, b->d_pbuild, b->d_slot_cell, nullptr, R);
    L.end();
    b->cur = dst;
    return;
  }
  // two kernels do the sort; the four they replace run where each kernel of
  // the step is timed on its own
  const bool whole = b->bucket_cap > 0 && !L.spans && !L.marks;
  if (whole) {
    hipLaunchKernelGGL(k_sort, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim, state_ref(b, 0), b->d_key,
                       b->d_count, b->d_bucket, b->bucket_cap, b->d_start, b->d_ncount, b->d_done, flag, R);
  } else {
    L.begin(K_KEYS);
    hipLaunchKernelGGL(k_keys, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim, state_ref(b, 0), b->d_key,
                       b->d_count, b->d_rank, flag, R);
    L.end();
    L.begin(K_SCAN);
    hipLaunchKernelGGL(k_scan, dim3(b->S), dim3(1024), 0, s, b->d_sims, b->d_count, b->d_start, b->d_ncount, flag,
                       R);
    L.end();
    L.begin(K_SCATTER);
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(tpb), 0, s, nt, b->d_key, b->d_start, b->d_rank, b->d_perm, flag,
                       R);
    L.end();
  }
  L.begin(K_REORDER);
  hipLaunchKernelGGL(k_reorder<1>, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_cell_sim, b->d_key, b->d_start,
                     b->d_ncount, whole ? b->d_bucket : b->d_perm, whole ? b->bucket_cap : 0u, state_ref(b, 0),
                     state_ref(b, 1), b->d_tag[0], b->d_tag[1], b->d_pos4, b->d_pfix, b->d_pbuild, b->d_slot_cell,
                     flag, R);
  L.end();
  if (with_list) {
    L.begin(K_LIST);
    launch_build(b, s, flag, R, state_ref(b, 1), state_ref(b, 0), b->d_tag[1], b->d_tag[0], 0);
    L.end();
  }
}

// Pair-path force kernels by variant index ((mode 2 + energy) 2 + uniform
// unit) 2 + wall parameters equal to the fluid's; sampling steps with the
// wall pressure recorded take the PR table, indexed (energy 2 + uniform) 2 +
// walls.
#define HMD_V(K, M, E, U, W) &K<M, E, U, W, 0>
#define HMD_VP(K, E, U, W) &K<1, E, U, W, 1>
#define HMD_VARIANTS_PR(K)                                                                                  \
  HMD_VP(K, 0, 0, 0), HMD_VP(K, 0, 0, 1), HMD_VP(K, 0, 1, 0), HMD_VP(K, 0, 1, 1), HMD_VP(K, 1, 0, 0),         \
      HMD_VP(K, 1, 0, 1), HMD_VP(K, 1, 1, 0), HMD_VP(K, 1, 1, 1)
#define HMD_VARIANTS(K)                                                                                   \
  HMD_V(K, 0, 0, 0, 0), HMD_V(K, 0, 0, 0, 1), HMD_V(K, 0, 0, 1, 0), HMD_V(K, 0, 0, 1, 1),               \
      HMD_V(K, 0, 1, 0, 0), HMD_V(K, 0, 1, 0, 1), HMD_V(K, 0, 1, 1, 0), HMD_V(K, 0, 1, 1, 1),           \
      HMD_V(K, 1, 0, 0, 0), HMD_V(K, 1, 0, 0, 1), HMD_V(K, 1, 0, 1, 0), HMD_V(K, 1, 0, 1, 1),           \
      HMD_V(K, 1, 1, 0, 0), HMD_V(K, 1, 1, 0, 1), HMD_V(K, 1, 1, 1, 0), HMD_V(K, 1, 1, 1, 1)
decltype(&k_force_tiles<0, 0, 0, 0, 0>) force_tiles_variant(int v, bool pr, bool tall) {
  using Fn = decltype(&k_force_tiles<0, 0, 0, 0, 0>);
  static const Fn tab[16] = {HMD_VARIANTS(k_force_tiles)}, tab_pr[8] = {HMD_VARIANTS_PR(k_force_tiles)};
  static const Fn ttab[16] = {HMD_VARIANTS(k_force_tall)}, ttab_pr[8] = {HMD_VARIANTS_PR(k_force_tall)};
  return tall ? (pr ? ttab_pr[v & 7] : ttab[v]) : (pr ? tab_pr[v & 7] : tab[v]);
}
decltype(&k_force_list<0, 0, 0, 0, 0>) force_list_variant(int v, bool pr) {
  static const decltype(&k_force_list<0, 0, 0, 0, 0>) tab[16] = {HMD_VARIANTS(k_force_list)};
  static const decltype(&k_force_list<0, 0, 0, 0, 0>) tab_pr[8] = {HMD_VARIANTS_PR(k_force_list)};
  return pr ? tab_pr[v & 7] : tab[v];
}
#undef HMD_VARIANTS
#undef HMD_VARIANTS_PR
#undef HMD_V
#undef HMD_VP

// List and force kernels of a step by variant index (uniform 2 + walls) 2 +
// pressure.
decltype(&k_list_force<0, 0, 0>) list_force_variant(int v) {
  static const decltype(&k_list_force<0, 0, 0>) tab[8] = {
      &k_list_force<0, 0, 0>, &k_list_force<0, 0, 1>, &k_list_force<0, 1, 0>, &k_list_force<0, 1, 1>,
      &k_list_force<1, 0, 0>, &k_list_force<1, 0, 1>, &k_list_force<1, 1, 0>, &k_list_force<1, 1, 1>};
  return tab[v];
}

void enqueue_force(hmd_batch* b, hipStream_t s, int mode, const StepConst& K, StepRef R) {
  const int nt = int(b->ntot), tpb = b->tpb, nb = blocks_for(nt, tpb);
  const int src = b->cur;
  if (b->path == 0) {
    if (mode == 0)
      hipLaunchKernelGGL(k_force_cell<0>, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim, b->d_pos4,
                         b->d_start, b->d_ncount, b->d_wpos4, b->d_wstart, b->d_wcount, b->d_f4, state_ref(b, src),
                         b->acc, b->d_dstate, R, K);
    else
      hipLaunchKernelGGL(k_force_cell<1>, dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim, b->d_pos4,
                         b->d_start, b->d_ncount, b->d_wpos4, b->d_wstart, b->d_wcount, b->d_f4, state_ref(b, src),
                         b->acc, b->d_dstate, R, K);
  } else {
    const int v = ((mode * 2 + (K.energy_on ? 1 : 0)) * 2 + (b->uniform ? 1 : 0)) * 2 + (b->walls_same ? 1 : 0);
    const bool pr = mode == 1 && K.press_on;
    if (b->path == 2) {
      hipLaunchKernelGGL(force_tiles_variant(v, pr, b->stage_cap > TILE_STAGE), dim3(b->ntiles), dim3(TILE_THREADS), 0,
                         s, nt, b->list_ld, b->d_tilerec, b->d_sims, b->d_pfix, b->d_list,
                         b->d_nlist, b->d_f4, state_ref(b, 0), b->acc, b->d_dstate, R, K);
    } else {
      hipLaunchKernelGGL(force_list_variant(v, pr), dim3(nb), dim3(tpb), 0, s, nt, b->list_ld, b->d_sims,
                         b->d_atom_sim, b->d_pfix, b->d_list, b->d_nlist, b->d_f4, state_ref(b, 0), b->acc,
                         b->d_dstate, R, K);
    }
  }
}

constexpr int kResidentTiles = 1280;

// One velocity-Verlet step over the whole batch.
void enqueue_step(hmd_batch* b, Launcher& L, const StepConst& K, StepRef R) {
  hipStream_t s = L.s;
  const int nt = int(b->ntot), tpb = b->tpb, nb = blocks_for(nt, tpb);
  L.begin(K_INTEGRATE);
  if (b->path == 0)
    hipLaunchKernelGGL((k_integrate<1, 0>), dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim,
                       state_ref(b, b->cur), b->d_f4, b->d_key, b->d_count, b->d_rank, b->d_pfix, b->d_pbuild,
                       b->d_flag, b->acc, b->d_dstate, R, K, b->S == 1);
  else
    hipLaunchKernelGGL((k_integrate<1, 1>), dim3(nb), dim3(tpb), 0, s, nt, b->d_sims, b->d_atom_sim,
                       state_ref(b, 0), b->d_f4, b->d_key, b->d_count, b->d_rank, b->d_pfix, b->d_pbuild, b->d_flag,
                       b->acc, b->d_dstate, R, K, b->S == 1);
  L.end();
  // lists and forces in one launch where all tiles are resident at once (five
  // per compute unit): it saves a launch of 2.5 to 4 us, but asks for the
  // rebuild flag in every workgroup, one after another on a compute unit once
  // there are more (39,189 atoms 1.75 -> 1.69 ms for 40 steps with results,
  // the density sweep's 1,040 tiles 60 -> 55 us a step; 2.1 M atoms in 9,660
  // tiles 17.9 -> 18.3 ms)
  if (b->path == 2 && b->ntiles <= kResidentTiles && b->stage_cap == TILE_STAGE && !L.spans && !L.marks &&
      !K.energy_on) {
    enqueue_sort(b, L, K, b->d_flag, R, false);
    const int v = (b->uniform ? 4 : 0) + (b->walls_same ? 2 : 0) + (K.press_on ? 1 : 0);
    hipLaunchKernelGGL(list_force_variant(v), dim3(b->ntiles), dim3(TILE_THREADS), 0, s, nt, b->list_ld,
                       tile_build(b, state_ref(b, 1), state_ref(b, 0), b->d_tag[1], b->d_tag[0], 0), b->d_flag, b->d_f4,
                       state_ref(b, 0), b->acc, b->d_dstate, R, K);
    return;
  }
  enqueue_sort(b, L, K, b->path == 0 ? nullptr : b->d_flag, R);
  L.begin(K_FORCE);
  enqueue_force(b, s, 1, K, R);
  L.end();
}

// Unconditional sort of the current positions (creation, new state).
void sort_now(hmd_batch* b, const StepConst& K) {
  Launcher L{b, b->ctx->stream, nullptr, 0};
  enqueue_sort(b, L, K, nullptr, StepRef{nullptr, -1});
}

// Forces for the current positions; potential energy and pair counts go to
// acc.pe[(done + 1) & 1] and acc.pairs (cleared first).
int forces_now(hmd_batch* b, bool energy) {
  hmd_ctx* ctx = b->ctx;
  hipStream_t s = ctx->stream;
  StepConst K = step_const(b, b->thermo_on, energy);
  const int p = int((b->done + 1) & 1);
  hipLaunchKernelGGL(k_clear_sums, dim3(1), dim3(256), 0, s, b->acc.pe[p], b->acc.ke[p], b->S, b->acc.pairs,
                     kPairCounters * kPairPitch);
  enqueue_force(b, s, 0, K, StepRef{nullptr, b->done});
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

void release_graphs(hmd_batch* b) {
  for (auto& kv : b->graphs) (void)hipGraphExecDestroy(kv.second);
  for (auto& kv : b->graph_defs) (void)hipGraphDestroy(kv.second);
  b->graphs.clear();
  b->graph_defs.clear();
  b->graph_spans.clear();
  b->graph_nstamps.clear();
}

int ensure_events(hmd_batch* b, size_t n) {
  while (b->ev.size() < n) {
    hipEvent_t e;
    HMD_HIP(b->ctx, hipEventCreate(&e));
    b->ev.push_back(e);
  }
  return HMD_OK;
}

int harvest(hmd_batch* b, std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>>& marks) {
  if (marks.empty()) return HMD_OK;
  HMD_HIP(b->ctx, hipEventSynchronize(marks.back().second.second));
  for (auto& m : marks) {
    float ms = 0.f;
    HMD_HIP(b->ctx, hipEventElapsedTime(&ms, m.second.first, m.second.second));
    b->kern_ms[m.first] += ms;
    b->kern_n[m.first] += 1;
  }
  marks.clear();
  return HMD_OK;
}

// Executable graph of `chunk` steps; its step indices are read from
// d_dstate[0], which its last node advances by `chunk`.  With timing on, the
// kernels of up to kStampedSteps evenly spaced steps (the last one among
// them) are bracketed by stamp kernels, and one more stamp after the last
// measures the gap of an empty interval.
int get_graph(hmd_batch* b, int chunk, const StepConst& K, hipGraphExec_t* out) {
  const int key = chunk * 4 + (K.thermo_on ? 1 : 0) + (b->timing ? 2 : 0);
  auto it = b->graphs.find(key);
  if (it != b->graphs.end()) {
    *out = it->second;
    return HMD_OK;
  }
  hmd_ctx* ctx = b->ctx;
  hipStream_t s = ctx->stream;
  const int cur0 = b->cur;
  auto& spans = b->graph_spans[key];
  spans.clear();
  const int every = std::max(1, chunk / kStampedSteps);
  Launcher L{b, s, nullptr, 0};
  HMD_HIP(ctx, hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  for (int k = 0; k < chunk; ++k) {
    const bool stamped = b->timing && (chunk - 1 - k) % every == 0 && (chunk - 1 - k) / every < kStampedSteps;
    L.spans = stamped ? &spans : nullptr;
    L.last_stamp = -1;
    L.flag = b->path == 0 ? nullptr : b->d_flag;
    L.R = StepRef{b->d_dstate, k};
    enqueue_step(b, L, K, StepRef{b->d_dstate, k});
  }
  if (b->timing) {  // calibration: an empty interval after the last stamp
    L.spans = &spans;
    L.stamp();
  }
  hipLaunchKernelGGL(k_add_i64, dim3(1), dim3(1), 0, s, b->d_dstate, int64_t(chunk));
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(s, &g);
  b->cur = cur0;  // capture did not execute anything
  if (e != hipSuccess) {
    ctx->err = std::string("graph capture: ") + hipGetErrorString(e);
    return HMD_EDEVICE;
  }
  if (b->timing) b->graph_nstamps[key] = L.next_stamp;
  hipGraphExec_t ex = nullptr;
  e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(g);
    ctx->err = std::string("graph instantiate: ") + hipGetErrorString(e);
    return HMD_EDEVICE;
  }
  b->graph_defs[key] = g;
  b->graphs[key] = ex;
  *out = ex;
  return HMD_OK;
}

}  // namespace

// Tiles of the tiled path: per system and z slab, runs of whole columns
// sized so that a tile holds about one to two workgroups of atoms and its
// staged neighbourhood fits the LDS capacity.
int make_tiles(hmd_batch* b) {
  hmd_ctx* ctx = b->ctx;
  constexpr int64_t kMinTiles = 512;
  b->stage_cap = TILE_STAGE;
  auto per_column = [&](int k, double n) { return n / double(b->sims[k].nx * b->sims[k].nz); };
  auto fluid_atoms = [&](int k, int nc) {
    return 3.0 * std::min(nc + 2, b->sims[k].nx) * per_column(k, double(b->sims[k].nf));
  };
  auto wall_atoms = [&](int k, int nc) {
    return 3.0 * std::min(nc + 2, b->sims[k].nx) * per_column(k, double(b->host[k].nw));
  };
  auto staged_atoms = [&](int k, int nc) { return fluid_atoms(k, nc) + wall_atoms(k, nc); };
  // Whether tiles of nc columns stay within an LDS capacity.  Below a liquid's
  // density the fluid gathers in places (between 0.1 and 0.56 it separates at
  // T = 1), and each tile that outgrows the capacity reads its neighbours from
  // memory.  Room for 5% more than the mean and for 40%, skin 0.2: 28 channels
  // of 16 sigma at density 0.4 174 and 121 us a step, 100 of 15 at 0.1 178 and
  // 142, of 30 237 and 200; the narrower tiles cost up to 7% where none outgrows
  // it (55 of 33 at 0.1, skin 0.3: 106 and 113)
  auto fits = [&](int k, int nc, int cap) {
    const SimDev& D = b->sims[k];
    const double rho = double(D.nf) / (D.Lx * D.Lz * D.h);
    const double swell = std::min(1.4, std::max(1.0, 0.65 / rho));
    return staged_atoms(k, nc) <= 0.95 * cap && fluid_atoms(k, nc) * swell + wall_atoms(k, nc) < cap;
  };
  // a channel whose narrowest tiles fit only the larger capacity asks for it
  // on behalf of the batch (32 channels of 10 sigma and one of 36: 168 us a
  // step, 272 with the one gathering from memory; alone 38 and 64), one that
  // exceeds both does not (8 of 10 sigma and one of 50: 144 us, 157 with it)
  for (int k = 0; k < b->S; ++k) {
    const double staged = staged_atoms(k, 1);
    if (staged > 0.95 * TILE_STAGE && staged < TILE_STAGE_TALL) b->stage_cap = TILE_STAGE_TALL;
  }
  // Whether the list build's cell table holds a tile's neighbourhood.  Tall
  // dilute channels keep to that width where it leaves two columns (four
  // channels of 150 sigma at density 0.05: 42 us a step with two columns, 54
  // with three and lists built cell by cell; of 200 sigma, where it leaves
  // one: 60 with one column, 53 with three).
  auto tabled = [&](int k, int nc) {
    return 3 * std::min(nc + 2, b->sims[k].nx) * (b->sims[k].ny + 2) <= TILE_CTAB;
  };
  // columns per tile: the most home atoms per unit of cost, cost being the
  // lanes of whole 256-lane passes and of a last one (half, a quarter or an
  // eighth of that where its lists are shared by lanes; the whole where they
  // are built by one thread per atom) plus tile_alpha + 1/4
  // per staged atom (a wider tile stages less halo per home atom); 2%
  // hysteresis keeps the narrower of two near-equal choices.  Without the
  // quarter, and with every pass counted whole: 64-channel batch, force 180
  // -> 173 us and list build 117 -> 108 us per step (1/2 and 3/4 as good);
  // density sweep 54 -> 51 us
  auto tile_cost = [&](int k, int nc) {
    const double atoms = nc * per_column(k, double(b->sims[k].nf)), left = std::fmod(atoms, double(TILE_THREADS));
    double last = left > 0.0 ? 256.0 : 0.0;
    if (tabled(k, nc) && left > 0.0 && left <= 128.0) last = left > 64.0 ? 128.0 : left > 32.0 ? 64.0 : 32.0;
    return atoms - left + last + (b->tile_alpha + 0.25) * staged_atoms(k, nc);
  };
  auto columns = [&](int k, int cap) {
    const SimDev& D = b->sims[k];
    int best = 1;
    double best_use = -1.0;
    for (int nc = 1; nc <= D.nx; ++nc) {
      if (nc > 1 && !fits(k, nc, cap)) break;
      if (nc > 2 && !tabled(k, nc) && tabled(k, 2)) break;
      const double use = nc * per_column(k, double(D.nf)) / tile_cost(k, nc);
      if (use > 1.02 * best_use) {
        best_use = use;
        best = nc;
      }
    }
    return best;
  };
  // The larger capacity also where it halves the tiles (channels with few atoms
  // beside their walls', which every tile stages), though a compute unit then
  // takes four: 76 channels of 12 sigma at density 0.2 131 -> 116 us a step, 61
  // of 20 at 0.15 116 -> 106.  Not where tiles get fewer by less (80 to 60 in a
  // channel: 0.98 to 1.07 times the time; 64-channel batch 8,440 to 6,220: 202
  // us of force for 176) or are few enough for the joined launch.
  auto plan = [&](int cap) {
    int64_t tiles = 0;
    double cost = 0.0;
    for (int k = 0; k < b->S; ++k) {
      const SimDev& D = b->sims[k];
      const int ntx = (D.nx + columns(k, cap) - 1) / columns(k, cap);
      tiles += int64_t(D.nz) * ntx;
      for (int t = 0; t < ntx; ++t) cost += D.nz * tile_cost(k, (t + 1) * D.nx / ntx - t * D.nx / ntx);
    }
    return std::make_pair(tiles, cost);
  };
  if (b->stage_cap == TILE_STAGE) {
    const auto small = plan(TILE_STAGE), tall = plan(TILE_STAGE_TALL);
    if (small.first > kResidentTiles && 1.8 * double(tall.first) < double(small.first) &&
        1.1 * tall.second < small.second)
      b->stage_cap = TILE_STAGE_TALL;
  }
  std::vector<int> cols(b->S, 1);
  for (int k = 0; k < b->S; ++k) cols[k] = columns(k, b->stage_cap);
  auto count = [&](int widest) {
    int64_t n = 0;
    for (int k = 0; k < b->S; ++k) {
      const int nc = std::min(cols[k], widest);
      n += int64_t(b->sims[k].nz) * ((b->sims[k].nx + nc - 1) / nc);
    }
    return n;
  };
  // fewer tiles than two per compute unit leave the chip idle: narrower ones
  // then, down to a column each, though each stages more halo (a step of the
  // 2,048-atom channel 37 -> 31 us with 49 tiles for 14, of the 39,189-atom
  // one 48.8 -> 48 us with 400 for 80: a list build 54 -> 47 us, a force
  // 13.9 -> 14.6 us; batches of nine hundred tiles gain nothing)
  int widest = *std::max_element(cols.begin(), cols.end());
  while (widest > 1 && count(widest) < kMinTiles) --widest;
  std::vector<int4> tiles;
  b->tile_first.assign(b->S + 1, 0);
  for (int k = 0; k < b->S; ++k) {
    b->tile_first[k] = int(tiles.size());
    const SimDev& D = b->sims[k];
    const int nc = std::min(cols[k], widest), ntx = (D.nx + nc - 1) / nc;
    for (int z = 0; z < D.nz; ++z)
      for (int t = 0; t < ntx; ++t) {  // columns split as evenly as possible
        const int x0 = int(int64_t(t) * D.nx / ntx), x1 = int(int64_t(t + 1) * D.nx / ntx);
        tiles.push_back(make_int4(k, z, x0, x1 - x0));
      }
  }
  b->ntiles = int(tiles.size());
  b->tile_first[b->S] = b->ntiles;
  for (const SimDev& D : b->sims) b->acc.tb_ld = std::max(b->acc.tb_ld, std::min(D.nbins, BIN_LDS));
  const size_t nbin = size_t(b->ntiles) * size_t(b->acc.tb_ld) * 2;
  HMD_TRY(dalloc(ctx, &b->d_tbins, int64_t(nbin)));
  HMD_HIP(ctx, hipMemsetAsync(b->d_tbins, 0, sizeof(double) * nbin, ctx->stream));
  HMD_TRY(dalloc(ctx, &b->d_tiles, b->ntiles));
  HMD_TRY(dalloc(ctx, &b->d_tilerec, int64_t(b->ntiles) * TILE_REC));
  HMD_HIP(ctx, hipMemcpyAsync(b->d_tiles, tiles.data(), sizeof(int4) * tiles.size(), hipMemcpyHostToDevice,
                              ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return HMD_OK;
}

int batch_create(hmd_ctx* ctx, const hmd_md_job* jobs, int n, hmd_batch** out) {
  if (!ctx || !out || !jobs || n < 1 || n > 65535) {
    if (ctx) ctx->err = "md batch: need 1..65535 jobs";
    return HMD_EINVAL;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  auto* b = new hmd_batch();
  b->ctx = ctx;
  b->P = ctx->params;
  b->S = n;
  b->n_sample = jobs[0].n_sample;
  const int64_t min_sample = std::max(2, b->P.n_blocks);
  for (int k = 0; k < n; ++k)
    if (jobs[k].n_sample != b->n_sample || jobs[k].n_sample < 0 ||
        (jobs[k].n_sample > 0 && jobs[k].n_sample < min_sample)) {
      ctx->err = "md batch: every job needs the same n_sample (0, or at least max(2, n_blocks))";
      delete b;
      return HMD_EINVAL;
    }
  if (b->n_sample > 0) {  // one series entry per sampled step up to the cap, then groups of B steps
    const int64_t B = (b->n_sample + kSeriesCap - 1) / kSeriesCap;
    b->ser_B = int(B);
    b->nser = b->n_sample / B;
    b->ser_r = int(b->n_sample - b->nser * B);
  }
  {
    const Config c = choose_config(ctx, jobs, n);
    b->path = c.path;
    b->skin = c.skin;
    b->tpb = c.tpb;
    b->tile_alpha = c.tile_alpha;
    b->cell_w = c.cell_w;
    b->chunk = c.chunk;
  }
  if (b->path == 3) {  // the tiled path with every tile on its gather fallback
    b->path = 2;
    b->force_gather = true;
  }
  const double wmin = std::max(b->path >= 1 ? b->P.rc + b->skin : b->P.rc, b->cell_w);
  b->host.resize(n);
  for (int k = 0; k < n; ++k) {
    hmd_md_params Pk = b->P;  // the job's own density, where it gives one
    if (jobs[k].rho > 0.0) Pk.rho = jobs[k].rho;
    int rc = build_system(Pk, jobs[k].h, jobs[k].g, jobs[k].seed, wmin, b->host[k], ctx->err);
    if (rc != HMD_OK) {
      delete b;
      return rc;
    }
  }
  // flattened layout
  b->sims.resize(n);
  int64_t a0 = 0, c0 = 0, wc0 = 0, bin0 = 0, w0 = 0;
  const double half = 0.5 * std::cbrt(4.0 / b->P.rho_wall);
  for (int k = 0; k < n; ++k) {
    const HostSystem& H = b->host[k];
    SimDev& D = b->sims[k];
    std::memset(&D, 0, sizeof(D));
    D.Lx = H.Lx; D.Lz = H.Lz; D.h = H.h;
    D.inv_x = H.inv_x; D.inv_y = H.inv_y; D.inv_z = H.inv_z;
    D.wx = H.wx; D.wy = H.wy; D.wz = H.wz;
    D.g = H.g;
    D.inv_area = 1.0 / (H.Lx * H.Lz);
    D.inv_bin = 1.0 / b->P.bin_dy;
    D.inv_nf = 1.0 / double(H.nf);
    const double margin = double(b->P.wall_layers) * half + 1.0;  // beyond the outermost wall layer
    D.y_lo = -margin;
    D.fix_x = kTwo32 / H.Lx;
    D.fix_z = kTwo32 / H.Lz;
    // y takes the x unit when the wall span fits in 2^32 of them (then, with
    // Lx = Lz, one unit serves every axis)
    const double span_y = H.h + 2.0 * margin;
    D.fix_y = span_y < H.Lx ? D.fix_x : kTwo32 / span_y;
    D.unit_x = float(H.Lx / kTwo32);
    D.unit_y = float(1.0 / D.fix_y);
    D.unit_z = float(H.Lz / kTwo32);
    D.inv_u = float(D.fix_x);
    D.inv_u2 = float(D.fix_x * D.fix_x);
    D.fwx = float(H.wx); D.fwy = float(H.wy); D.fwz = float(H.wz);
    D.nx = H.nx; D.ny = H.ny; D.nz = H.nz;
    D.a0 = int(a0); D.nf = int(H.nf);
    D.c0 = int(c0); D.ncell = H.nx * H.ny * H.nz;
    D.wc0 = int(wc0);
    D.w0 = int(w0);
    D.nbins = H.nbins; D.bin0 = int(bin0);
    a0 += H.nf;
    c0 += D.ncell;
    wc0 += 2 * int64_t(H.nx) * H.nz;
    bin0 += H.nbins;
    w0 += H.nw;
  }
  if (a0 + w0 >= (int64_t(1) << 31) || c0 >= (int64_t(1) << 31)) {
    ctx->err = "md batch: too many atoms or cells for one batch";
    delete b;
    return HMD_EINVAL;
  }
  b->ntot = a0; b->ncell = c0; b->nwcell = wc0; b->nbins = bin0; b->nwall = w0;
  b->walls_same = b->P.eps_wf == 1.0 && b->P.sigma_wf == 1.0;
  b->uniform = true;
  for (const SimDev& D : b->sims)
    b->uniform = b->uniform && D.fix_x == D.fix_y && D.fix_x == D.fix_z;
  // the pair-list build packs a position index into 24 bits
  if (b->path == 1 && b->ntot + b->nwall >= (int64_t(1) << 24)) b->path = 0;
  if (b->path == 2 && b->P.wall_layers < 1) b->path = 1;
  if (b->P.pressure && b->path == 0) {
    ctx->err = "md batch: the wall pressure needs a pair path (force_path 1 or 2)";
    delete b;
    return HMD_EINVAL;
  }
  // pair-list capacity: neighbours within rc + skin at twice the fluid density
  // plus a wall half-space, rounded up to a multiple of 32
  const double rl = b->P.rc + b->skin;
  double rho_max = b->P.rho;
  for (int k = 0; k < n; ++k) rho_max = std::max(rho_max, jobs[k].rho);
  const double est = 2.0 * std::max(rho_max, 0.8) * 4.18879 * rl * rl * rl +
                     2.0 * b->P.rho_wall * 2.0944 * rl * rl * rl;
  b->list_cap = b->path >= 1 ? int(32 * std::ceil(est / 32.0)) : 0;
  b->list_ld = int(64 * ((b->ntot + 63) / 64));

  int rc = HMD_OK;
  auto fail = [&](int code) {
    batch_free(b);
    return code;
  };
  if ((rc = dalloc(ctx, &b->d_sims, n)) || (rc = dalloc(ctx, &b->d_atom_sim, b->ntot)) ||
      (rc = dalloc(ctx, &b->d_cell_sim, b->ncell)) || (rc = dalloc(ctx, &b->d_f4, b->ntot)) ||
      (rc = dalloc(ctx, &b->d_key, b->ntot)) || (rc = dalloc(ctx, &b->d_count, b->ncell)) ||
      (rc = dalloc(ctx, &b->d_rank, b->ntot)) || (rc = dalloc(ctx, &b->d_start, b->ncell)) ||
      (rc = dalloc(ctx, &b->d_ncount, b->ncell)) || (rc = dalloc(ctx, &b->d_perm, b->ntot)) ||
      (rc = dalloc(ctx, &b->d_wpos4, b->nwall)) || (rc = dalloc(ctx, &b->d_wstart, b->nwcell)) ||
      (rc = dalloc(ctx, &b->d_wcount, b->nwcell)) || (rc = dalloc(ctx, &b->d_dstate, 4)) ||
      (rc = dalloc(ctx, &b->d_tag[0], b->ntot)) || (rc = dalloc(ctx, &b->d_tag[1], b->ntot)) ||
      (rc = dalloc(ctx, &b->d_stamps, kMaxStamps)))
    return fail(rc);
  if (b->path == 0) {
    if ((rc = dalloc(ctx, &b->d_pos4, b->ntot))) return fail(rc);
  } else {
    if ((rc = dalloc(ctx, &b->d_pfix, b->ntot + b->nwall)) || (rc = dalloc(ctx, &b->d_pbuild, b->ntot)) ||
        (rc = dalloc(ctx, &b->d_slot_cell, b->ntot)) || (rc = dalloc(ctx, &b->d_nlist, b->ntot)) ||
        (rc = dalloc(ctx, &b->d_list, int64_t(b->list_cap) * b->list_ld)))
      return fail(rc);
    // Buckets of the sort (a fuller cell is handled, slowly): room for twice a
    // system's mean cell and some, and for a cell of condensed fluid at 1.25
    // per sigma^3 (a droplet of 5,878 atoms in cells 4 sigma wide, pair lists:
    // 55 us a step, 109 where its cells overran the first of the two).  Bounded
    // by the size of the pair lists: very dilute systems keep the first, or
    // the separate kernels.  Those also sort where a system has no atoms (nobody
    // would scan it).
    bool all = true;
    double mean = 0.0, dense = 0.0;
    for (const SimDev& D : b->sims) {
      all = all && D.nf > 0;
      mean = std::max(mean, double(D.nf) / double(D.ncell));
      dense = std::max(dense, 1.25 * D.wx * D.wy * D.wz);
    }
    if (all) {
      const double room = double(b->list_cap) * double(b->list_ld) / double(b->ncell);
      for (double atoms : {std::max(2.0 * mean, dense), 2.0 * mean}) {
        const double cap = 8.0 * std::ceil((atoms + 16.0) / 8.0);
        if (cap <= room) {
          b->bucket_cap = uint32_t(cap);
          break;
        }
      }
    }
    if (b->bucket_cap) {
      if ((rc = dalloc(ctx, &b->d_bucket, b->ncell * int64_t(b->bucket_cap))) || (rc = dalloc(ctx, &b->d_done, n)))
        return fail(rc);
      HMD_HIP(ctx, hipMemsetAsync(b->d_done, 0, sizeof(int) * n, ctx->stream));
    }
    // screening reads whole blocks past the end of a range
    if (b->path == 2 && (rc = dalloc(ctx, &b->d_pos4, b->ntot + b->nwall + SCREEN_PAD))) return fail(rc);
  }
  for (int w = 0; w < 2; ++w)
    for (int a = 0; a < 6; ++a)
      if ((rc = dalloc(ctx, &b->d_state[w][a], b->ntot))) return fail(rc);
  // cell numbering of every system (rank tables, then inverses): Morton
  // order, or slab order (z, x, y) for the tiled path
  if ((rc = dalloc(ctx, &b->d_cellmap, 2 * b->ncell))) return fail(rc);
  b->cell_rank.assign(b->ncell, 0);
  std::vector<uint32_t> cell_lin(b->ncell);
  for (int k = 0; k < n; ++k) {
    SimDev& D = b->sims[k];
    std::vector<std::pair<uint64_t, uint32_t>> order(D.ncell);
    for (int lid = 0; lid < D.ncell; ++lid) {
      const uint32_t cx = lid % D.nx, cy = (lid / D.nx) % D.ny, cz = lid / (D.nx * D.ny);
      const uint64_t key = b->path == 2 ? (uint64_t(cz) * D.nx + cx) * D.ny + cy : morton3(cx, cy, cz);
      order[lid] = {key, uint32_t(lid)};
    }
    std::sort(order.begin(), order.end());
    for (int r = 0; r < D.ncell; ++r) {
      b->cell_rank[D.c0 + order[r].second] = uint32_t(r);
      cell_lin[D.c0 + r] = order[r].second;
    }
    D.rank = b->d_cellmap + D.c0;
    D.lin = b->d_cellmap + b->ncell + D.c0;
  }
  if (b->path == 2 && (rc = make_tiles(b))) return fail(rc);
  HMD_HIP(ctx, hipMemcpyAsync(b->d_cellmap, b->cell_rank.data(), 4 * b->ncell, hipMemcpyHostToDevice, ctx->stream));
  HMD_HIP(ctx, hipMemcpyAsync(b->d_cellmap + b->ncell, cell_lin.data(), 4 * b->ncell, hipMemcpyHostToDevice,
                              ctx->stream));
  // per-system sums: what the results read first, in one piece (energies,
  // temperature sums, series statistics, flags and status), then the series
  // and the profile.  Atomics on one 64-byte piece of memory wait for each
  // other unless one instruction makes them, so the thermostat and the
  // temperature sums start cache lines of their own (one channel of 78,400 atoms
  // on the list path: 69 us a step, 95 with the sums side by side)
  auto lines = [](int64_t words) { return (words + 15) / 16 * 16; };
  const int64_t n_sums = lines(6 * int64_t(n)), n_temp = lines(3 * int64_t(n)), n_stat = lines(8 * int64_t(n));
  b->small_n = n_sums + n_temp + n_stat + lines((n + 5) / 2);
  const int64_t nacc = b->small_n + 2 * int64_t(n) * b->nser + 2 * b->nbins;
  if ((rc = dalloc(ctx, &b->d_accbuf, nacc)) ||
      (rc = dalloc(ctx, &b->acc.pairs, kPairCounters * kPairPitch)))
    return fail(rc);
  if (b->n_sample > 0 && b->P.n_blocks == 0 && (rc = dalloc(ctx, &b->d_gam, int64_t(n) * b->nser)))
    return fail(rc);
  double* q = b->d_accbuf;
  for (int p = 0; p < 2; ++p) { b->acc.vc2[p] = q; q += n; }
  for (int p = 0; p < 2; ++p) { b->acc.ke[p] = q; q += n; }
  for (int p = 0; p < 2; ++p) { b->acc.pe[p] = q; q += n; }
  b->acc.tsum = b->d_accbuf + n_sums;
  b->d_sout = b->acc.tsum + n_temp;
  b->d_flag = reinterpret_cast<int*>(b->d_sout + n_stat);
  b->d_status = b->d_flag + 4;
  q = b->d_accbuf + b->small_n;
  b->acc.blocks = q; q += int64_t(n) * b->nser;
  b->acc.pblocks = q; q += int64_t(n) * b->nser;
  b->acc.binvx = q; q += b->nbins;
  b->acc.bincnt = q;
  b->acc.tbins = b->d_tbins;
  b->acc.status = b->d_status;

  hipStream_t s = ctx->stream;
  // host staging
  std::vector<double> hs[6];
  for (auto& v : hs) v.resize(b->ntot);
  std::vector<int> tag(b->ntot);
  std::vector<uint16_t> atom_sim(b->ntot), cell_sim(b->ncell);
  std::vector<float4> wpos(std::max<int64_t>(b->nwall, 1));
  std::vector<int4> wfix(std::max<int64_t>(b->nwall, 1));
  std::vector<uint32_t> wstart(b->nwcell), wcount(b->nwcell, 0);
  b->wall_id.assign(std::max<int64_t>(b->nwall, 1), 0);
  for (int k = 0; k < n; ++k) {
    HostSystem& H = b->host[k];
    const SimDev& D = b->sims[k];
    for (int64_t i = 0; i < H.nf; ++i) {
      const int64_t g = D.a0 + i;
      for (int a = 0; a < 3; ++a) {
        hs[a][g] = H.x[3 * i + a];
        hs[3 + a][g] = H.v[3 * i + a];
      }
      tag[g] = int(i);
      atom_sim[g] = uint16_t(k);
    }
    for (int c = 0; c < D.ncell; ++c) cell_sim[D.c0 + c] = uint16_t(k);
    // wall columns: slab 0 below the channel, 1 above; ascending wall id
    const int ncol = 2 * D.nx * D.nz;
    std::vector<int> wkey(H.nw);
    for (int64_t w = 0; w < H.nw; ++w) {
      const int cx = cell_coord(H.xw[3 * w], H.inv_x, H.nx);
      const int cz = cell_coord(H.xw[3 * w + 2], H.inv_z, H.nz);
      const int slab = H.xw[3 * w + 1] <= 0.0 ? 0 : 1;
      wkey[w] = (slab * H.nz + cz) * H.nx + cx;
      wcount[D.wc0 + wkey[w]]++;
    }
    uint32_t acc0 = uint32_t(D.w0);
    for (int c = 0; c < ncol; ++c) {
      wstart[D.wc0 + c] = acc0;
      acc0 += wcount[D.wc0 + c];
    }
    std::vector<uint32_t> fill(ncol, 0);
    for (int64_t w = 0; w < H.nw; ++w) {
      const int c = wkey[w];
      const uint32_t slot = wstart[D.wc0 + c] + fill[c]++;
      b->wall_id[slot] = int(w);
      const int cx = c % H.nx, cz = (c / H.nx) % H.nz, slab = c / (H.nx * H.nz);
      const double oy = slab == 0 ? -H.wy : double(H.ny) * H.wy;
      const double* p = &H.xw[3 * w];
      if (b->path == 2) {  // as k_reorder writes for the fluid
        const float px = float(p[0] - cell_origin(cx, H.wx)), py = float(p[1] - 0.5 * H.h),
                    pz = float(p[2] - cell_origin(cz, H.wz));
        wpos[slot] = make_float4(px, py, pz, px * px + py * py + pz * pz);
      } else {
        wpos[slot] = make_float4(float(p[0] - double(cx) * H.wx), float(p[1] - oy),
                                 float(p[2] - double(cz) * H.wz), 0.0f);
      }
      wfix[slot] = make_int4(int(fix_axis_host(p[0], D.fix_x)), int(fix_axis_host(p[1] - D.y_lo, D.fix_y)),
                             int(fix_axis_host(p[2], D.fix_z)), 0);
    }
    // the big host arrays are no longer needed
    H.x.clear(); H.x.shrink_to_fit();
    H.v.clear(); H.v.shrink_to_fit();
    H.xw.clear(); H.xw.shrink_to_fit();
  }
  const int64_t dstate[4] = {0, b->P.n_equil, 0, 0};
  auto up = [&](void* d, const void* h, size_t bytes) -> int {
    HMD_HIP(ctx, hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, s));
    return HMD_OK;
  };
  if ((rc = up(b->d_sims, b->sims.data(), sizeof(SimDev) * n)) ||
      (rc = up(b->d_atom_sim, atom_sim.data(), 2 * b->ntot)) ||
      (rc = up(b->d_cell_sim, cell_sim.data(), 2 * b->ncell)) || (rc = up(b->d_tag[0], tag.data(), 4 * b->ntot)) ||
      (rc = up(b->d_wpos4, wpos.data(), sizeof(float4) * b->nwall)) ||
      (rc = up(b->d_wstart, wstart.data(), 4 * b->nwcell)) ||
      (rc = up(b->d_wcount, wcount.data(), 4 * b->nwcell)) || (rc = up(b->d_dstate, dstate, sizeof(dstate))))
    return fail(rc);
  if (b->path >= 1 && (rc = up(b->d_pfix + b->ntot, wfix.data(), sizeof(int4) * b->nwall))) return fail(rc);
  if (b->path == 2) {
    if ((rc = up(b->d_pos4 + b->ntot, wpos.data(), sizeof(float4) * b->nwall))) return fail(rc);
    HMD_HIP(ctx, hipMemsetAsync(b->d_pos4 + b->ntot + b->nwall, 0, SCREEN_PAD * sizeof(float4), s));
  }
  for (int a = 0; a < 6; ++a)
    if ((rc = up(b->d_state[0][a], hs[a].data(), 8 * b->ntot))) return fail(rc);
  HMD_HIP(ctx, hipMemsetAsync(b->d_accbuf, 0, sizeof(double) * nacc, s));
  HMD_HIP(ctx, hipMemsetAsync(b->d_count, 0, 4 * b->ncell, s));
  b->cur = 0;
  StepConst K = step_const(b, true, true);
  sort_now(b, K);
  if ((rc = forces_now(b, true))) return fail(rc);
  HMD_HIP(ctx, hipStreamSynchronize(s));
  HMD_HIP(ctx, hipGetLastError());
  *out = b;
  return HMD_OK;
}

void batch_free(hmd_batch* b) {
  if (!b) return;
  release_graphs(b);
  for (auto e : b->ev) (void)hipEventDestroy(e);
  void* ptrs[] = {b->d_sims, b->d_atom_sim, b->d_cell_sim, b->d_f4, b->d_pos4, b->d_pfix, b->d_pbuild,
                  b->d_slot_cell, b->d_list, b->d_nlist, b->d_key, b->d_count, b->d_rank, b->d_start, b->d_ncount,
                  b->d_perm, b->d_bucket, b->d_done, b->d_wpos4, b->d_wstart, b->d_wcount, b->d_dstate, b->d_tag[0],
                  b->d_tag[1], b->d_accbuf, b->acc.pairs, b->d_cellmap, b->d_tiles,
                  b->d_tilerec, b->d_tbins, b->d_gam, b->d_stamps};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  for (int w = 0; w < 2; ++w)
    for (int a = 0; a < 6; ++a)
      if (b->d_state[w][a]) (void)hipFree(b->d_state[w][a]);
  delete b;
}

int batch_run(hmd_batch* b, int64_t steps, int graph_chunk, bool thermostat, double* energy_trace) {
  hmd_ctx* ctx = b->ctx;
  if (steps < 0 || graph_chunk < 0 || (graph_chunk & 1)) {
    ctx->err = "md run: steps >= 0 and an even graph chunk";
    return HMD_EINVAL;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = ctx->stream;
  b->thermo_on = thermostat;
  const bool energy = energy_trace != nullptr;
  const StepConst K = step_const(b, thermostat, energy);
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> marks;
  const int per_sync = 32;
  if (b->timing) HMD_TRY(ensure_events(b, size_t(2 * K_COUNT) * per_sync + 2));
  Launcher L{b, s, b->timing ? &marks : nullptr, 2};

  auto direct_step = [&](int64_t k) -> int {
    enqueue_step(b, L, K, StepRef{nullptr, b->done});
    if (energy) {
      HMD_HIP(ctx, hipStreamSynchronize(s));
      const int p = int((b->done + 1) & 1);
      double pe = 0, ke = 0, vc2 = 0;
      HMD_HIP(ctx, hipMemcpy(&pe, b->acc.pe[p], sizeof(double), hipMemcpyDeviceToHost));
      HMD_HIP(ctx, hipMemcpy(&ke, b->acc.ke[p], sizeof(double), hipMemcpyDeviceToHost));
      HMD_HIP(ctx, hipMemcpy(&vc2, b->acc.vc2[p], sizeof(double), hipMemcpyDeviceToHost));
      const double nf = double(b->sims[0].nf);
      double lam2 = 1.0;
      if (thermostat) lam2 = 1.0 + K.dt_tau * (K.T0 / (vc2 / nf) - 1.0);
      energy_trace[k] = (0.5 * (ke + (lam2 - 1.0) * vc2) + pe) / nf;
    }
    b->done += 1;
    if (b->timing && int(marks.size()) >= per_sync * (K_COUNT - 1)) {
      HMD_TRY(harvest(b, marks));
      L.next_ev = 2;
    }
    return HMD_OK;
  };

  int64_t k = 0;
  if (graph_chunk > 0 && !energy && steps >= graph_chunk) {
    if (b->cur != 0) HMD_TRY(direct_step(k++));
    if (b->timing) {
      HMD_TRY(harvest(b, marks));
      L.next_ev = 2;
    }
    // timing mode: one replay in kStampEvery is the stamped graph (timed
    // by events, then its stamps read back); the others replay the plain
    // graph with no host synchronisation, as outside timing mode
    hipGraphExec_t ex = nullptr, ex_plain = nullptr;
    HMD_TRY(get_graph(b, graph_chunk, K, &ex));
    if (b->timing) {
      b->timing = false;
      const int rc = get_graph(b, graph_chunk, K, &ex_plain);
      b->timing = true;
      HMD_TRY(rc);
    }
    const int gkey = graph_chunk * 4 + (K.thermo_on ? 1 : 0) + (b->timing ? 2 : 0);
    if (b->timing && b->clock_khz <= 0.0) {
      int khz = 0;
      HMD_HIP(ctx, hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, ctx->device));
      if (khz <= 0) {
        ctx->err = "md run: the device reports no wall-clock rate for timed graph replays";
        return HMD_EDEVICE;
      }
      b->clock_khz = double(khz);
    }
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, b->d_dstate, b->done);
    for (int64_t rep = 0; steps - k >= graph_chunk; ++rep) {
      if (b->timing && rep % kStampEvery == 0) {
        hipEvent_t e0 = b->ev[0], e1 = b->ev[1];
        HMD_HIP(ctx, hipEventRecord(e0, s));
        HMD_HIP(ctx, hipGraphLaunch(ex, s));
        HMD_HIP(ctx, hipEventRecord(e1, s));
        HMD_HIP(ctx, hipEventSynchronize(e1));
        float ms = 0.f;
        HMD_HIP(ctx, hipEventElapsedTime(&ms, e0, e1));
        b->graph_ms += ms;
        b->graph_steps += graph_chunk;
        // the stamped steps of the replay: each kernel's time is the span
        // between its stamps less the gap of the empty interval at the end
        // the list build's time is also kept apart for steps that rebuild
        // and steps that do not (bit 63 of its opening stamp)
        const auto& spans = b->graph_spans[gkey];
        const int ns = b->graph_nstamps[gkey];
        unsigned long long st[kMaxStamps];
        HMD_HIP(ctx, hipMemcpy(st, b->d_stamps, sizeof(unsigned long long) * size_t(ns), hipMemcpyDeviceToHost));
        constexpr unsigned long long kClock = ~(1ull << 63);
        const double gap = double((st[ns - 1] & kClock) - (st[ns - 2] & kClock));
        for (const auto& sp : spans) {
          const double ticks = std::max(0.0, double((st[sp[2]] & kClock) - (st[sp[1]] & kClock)) - gap);
          b->kern_ms[sp[0]] += ticks / b->clock_khz;
          b->kern_n[sp[0]] += 1;
          if (sp[0] == K_LIST) {
            const int r = (st[sp[1]] >> 63) ? 1 : 0;
            b->list_ms[r] += ticks / b->clock_khz;
            b->list_n[r] += 1;
          }
        }
      } else {
        HMD_HIP(ctx, hipGraphLaunch(b->timing ? ex_plain : ex, s));
      }
      k += graph_chunk;
      b->done += graph_chunk;
    }
  }
  while (k < steps) HMD_TRY(direct_step(k++));
  if (b->timing) HMD_TRY(harvest(b, marks));
  b->pending = thermostat && b->done > 0;
  HMD_HIP(ctx, hipGetLastError());
  HMD_HIP(ctx, hipStreamSynchronize(s));
  return HMD_OK;
}

namespace {

// Pinned host memory of the context for downloads, at least `bytes` (null: not
// to be had; its earlier contents are dropped).  A copy into memory of the
// caller's costs 15 to 25 us of staging each; allocating it anew for every
// batch took 40 us and now and then near a millisecond of the first download.
void* stage(hmd_ctx* ctx, size_t bytes) {
  constexpr size_t kMaxStage = size_t(64) << 20;
  if (bytes > kMaxStage) return nullptr;
  if (bytes > ctx->stage_bytes) {
    if (ctx->h_stage) (void)hipHostFree(ctx->h_stage);
    const size_t want = std::min(kMaxStage, std::max({bytes, 2 * ctx->stage_bytes, size_t(1) << 16}));
    ctx->stage_bytes = 0;
    if (hipHostMalloc(&ctx->h_stage, want, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      ctx->h_stage = nullptr;
      return nullptr;
    }
    ctx->stage_bytes = want;
  }
  return ctx->h_stage;
}

}  // namespace

int batch_results(hmd_batch* b, hmd_md_result* out) {
  hmd_ctx* ctx = b->ctx;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  HMD_TRY(forces_now(b, true));
  const int n = b->S;
  // the sampling window is complete once every one of its n_sample steps ran
  const bool complete = b->n_sample > 0 && b->done - b->P.n_equil >= b->n_sample;
  hipStream_t s = ctx->stream;
  double* const d_pout = b->d_sout + 4 * size_t(n);
  if (complete && b->P.pressure)
    series_stats_enqueue(s, b->acc.pblocks, n, b->nser, b->nser, 1.0 / double(b->ser_B), b->P.n_blocks, b->d_gam,
                         d_pout);
  if (complete)
    series_stats_enqueue(s, b->acc.blocks, n, b->nser, b->nser, 1.0 / double(b->ser_B), b->P.n_blocks, b->d_gam,
                         b->d_sout);
  std::vector<double> pageable;
  double* h = static_cast<double*>(stage(ctx, 8 * size_t(b->small_n)));
  if (!h) {
    pageable.resize(b->small_n);
    h = pageable.data();
  }
  HMD_HIP(ctx, hipMemcpyAsync(h, b->d_accbuf, 8 * size_t(b->small_n), hipMemcpyDeviceToHost, s));
  auto host = [&](const void* d) { return h + (static_cast<const double*>(d) - b->d_accbuf); };
  const double *sout = host(b->d_sout), *pout = host(d_pout), *tsum = host(b->acc.tsum),
               *pe = host(b->acc.pe[(b->done + 1) & 1]);
  const int* const flags = reinterpret_cast<const int*>(host(b->d_flag));
  const int* const status = flags + 4;
  HMD_HIP(ctx, hipStreamSynchronize(s));
  HMD_HIP(ctx, hipGetLastError());
  for (int k = 0; k < n; ++k) {
    hmd_md_result& R = out[k];
    std::memset(&R, 0, sizeof(R));
    const SimDev& D = b->sims[k];
    R.n_fluid = D.nf;
    R.pe = pe[k] * D.inv_nf;
    // an overflowing pair list drops interactions: every result is suspect
    int st = (status[k] & 1) || flags[2] > 0 ? HMD_EUNSTABLE : HMD_OK;
    if (complete) {
      const double* so = &sout[4 * size_t(k)];
      R.flux = so[0];
      R.flux_se = so[1];
      R.jflux = so[0] / D.h;
      if (b->P.pressure) {
        R.p = pout[4 * size_t(k)];
        R.p_se = pout[4 * size_t(k) + 1];
      }
      // temperatures are summed over every sampled step
      for (int a = 0; a < 3; ++a) R.T[a] = tsum[3 * k + a] / double(b->n_sample);
      // non-convergence (critical shear, Sec. 3.2): the two halves of the
      // series differ by more than 8 SE, or the spanwise temperature runs away
      if (st == HMD_OK && (std::fabs(so[3] - so[2]) > 8.0 * R.flux_se || R.T[2] > 1.5 * b->P.T0))
        st = HMD_ENOTCONV;
    } else if (st == HMD_OK) {
      st = HMD_EINVAL;  // sampling window not complete
    }
    R.status = st;
  }
  if (flags[2] > 0)
    ctx->err = flags[2] >= (1 << 30) ? std::string("pair list build: a cell holds more than 255 atoms")
                                     : "pair list overflow: " + std::to_string(flags[2]) + " > capacity";
  return HMD_OK;
}

// The sampled q' series of one system: nser entries (each the mean of ser_B
// consecutive sampled steps), as far as sampling has reached.
int batch_series(hmd_batch* b, int sim, double* q, int64_t* n, int which) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S || b->n_sample <= 0 || which < 0 || which > 1 || (which == 1 && !b->P.pressure)) {
    ctx->err = "md series: need a valid system of a batch with n_sample > 0 (pressure series: pressure on)";
    return HMD_EINVAL;
  }
  if (n) *n = b->nser;
  if (!q) return HMD_OK;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  const double* src = which ? b->acc.pblocks : b->acc.blocks;
  double* h = static_cast<double*>(stage(ctx, 8 * size_t(b->nser)));
  if (!h) h = q;
  HMD_HIP(ctx, hipMemcpyAsync(h, src + int64_t(sim) * b->nser, 8 * size_t(b->nser), hipMemcpyDeviceToHost,
                              ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int64_t k = 0; k < b->nser; ++k) q[k] = h[k] / double(b->ser_B);
  return HMD_OK;
}

// ---------------------------------------------------------------------------
// state of every system at once, and single-system hooks (`sim` selects the
// system of the batch)
// ---------------------------------------------------------------------------
namespace {

int download_state(hmd_batch* b, std::vector<double> (&hs)[6], std::vector<int>& tag) {
  hmd_ctx* ctx = b->ctx;
  hipStream_t s = ctx->stream;
  for (int a = 0; a < 6; ++a) {
    hs[a].resize(b->ntot);
    HMD_HIP(ctx, hipMemcpyAsync(hs[a].data(), b->d_state[b->cur][a], 8 * b->ntot, hipMemcpyDeviceToHost, s));
  }
  tag.resize(b->ntot);
  HMD_HIP(ctx, hipMemcpyAsync(tag.data(), b->d_tag[b->cur], 4 * b->ntot, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  return HMD_OK;
}

}  // namespace

int batch_get_all_states(hmd_batch* b, std::vector<std::vector<double>>& x, std::vector<std::vector<double>>& v) {
  hmd_ctx* ctx = b->ctx;
  std::vector<double> hs[6];
  std::vector<int> tag;
  HMD_TRY(download_state(b, hs, tag));
  std::vector<double> vc2(b->S, 0.0);
  if (b->pending)  // the device holds velocities before the last Berendsen factor
    HMD_HIP(ctx, hipMemcpy(vc2.data(), b->acc.vc2[b->done & 1], 8 * size_t(b->S), hipMemcpyDeviceToHost));
  x.assign(b->S, {});
  v.assign(b->S, {});
  for (int k = 0; k < b->S; ++k) {
    const SimDev& D = b->sims[k];
    const double lam =
        b->pending ? std::sqrt(1.0 + (b->P.dt / b->P.tau_T) * (b->P.T0 / (vc2[k] * D.inv_nf) - 1.0)) : 1.0;
    x[k].resize(3 * size_t(D.nf));
    v[k].resize(3 * size_t(D.nf));
    for (int i = 0; i < D.nf; ++i) {
      const int64_t g = D.a0 + i;
      const int id = tag[g];
      for (int a = 0; a < 3; ++a) {
        x[k][3 * id + a] = hs[a][g];
        v[k][3 * id + a] = hs[3 + a][g] * (a == b->P.thermo_axis ? lam : 1.0);
      }
    }
  }
  return HMD_OK;
}

int batch_set_all_states(hmd_batch* b, const std::vector<std::vector<double>>& x,
                         const std::vector<std::vector<double>>& v) {
  hmd_ctx* ctx = b->ctx;
  if (int(x.size()) != b->S || int(v.size()) != b->S) return HMD_EINVAL;
  std::vector<double> hs[6];
  std::vector<int> tag;
  HMD_TRY(download_state(b, hs, tag));
  for (int k = 0; k < b->S; ++k) {
    const SimDev& D = b->sims[k];
    if (x[k].empty() && v[k].empty()) continue;  // this system keeps its state
    if (int64_t(x[k].size()) != 3 * int64_t(D.nf) || int64_t(v[k].size()) != 3 * int64_t(D.nf)) return HMD_EINVAL;
    for (int i = 0; i < D.nf; ++i) {
      const int64_t g = D.a0 + i;
      const int id = tag[g];
      for (int a = 0; a < 3; ++a) {
        hs[a][g] = x[k][3 * id + a];
        hs[3 + a][g] = v[k][3 * id + a];
      }
    }
  }
  hipStream_t s = ctx->stream;
  for (int a = 0; a < 6; ++a)
    HMD_HIP(ctx, hipMemcpyAsync(b->d_state[b->cur][a], hs[a].data(), 8 * b->ntot, hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, b->d_dstate + 3, int64_t(0));
  b->pending = false;
  StepConst K = step_const(b, b->thermo_on, true);
  sort_now(b, K);
  HMD_TRY(forces_now(b, true));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  return HMD_OK;
}

int batch_get_state(hmd_batch* b, int sim, double* x, double* v) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S) return HMD_EINVAL;
  const SimDev& D = b->sims[sim];
  const size_t n = size_t(D.nf), bytes = 8 * (6 * n + 1) + 4 * n;
  std::vector<char> pageable;
  char* h = static_cast<char*>(stage(ctx, bytes));
  if (!h) {
    pageable.resize(bytes);
    h = pageable.data();
  }
  // x y z vx vy vz, the sum behind a Berendsen factor still to come, atom ids
  double* const hs = reinterpret_cast<double*>(h);
  int* const tag = reinterpret_cast<int*>(hs + 6 * n + 1);
  hipStream_t s = ctx->stream;
  for (int a = 0; a < 6; ++a)
    if (a < 3 ? x != nullptr : v != nullptr)
      HMD_HIP(ctx, hipMemcpyAsync(hs + a * n, b->d_state[b->cur][a] + D.a0, 8 * n, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(tag, b->d_tag[b->cur] + D.a0, 4 * n, hipMemcpyDeviceToHost, s));
  if (b->pending)
    HMD_HIP(ctx, hipMemcpyAsync(hs + 6 * n, b->acc.vc2[b->done & 1] + sim, 8, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  // the device holds velocities before the last Berendsen factor
  const double lam =
      b->pending ? std::sqrt(1.0 + (b->P.dt / b->P.tau_T) * (b->P.T0 / (hs[6 * n] * D.inv_nf) - 1.0)) : 1.0;
  for (size_t i = 0; i < n; ++i) {
    const size_t id = size_t(tag[i]);
    for (int a = 0; a < 3; ++a) {
      if (x) x[3 * id + a] = hs[a * n + i];
      if (v) v[3 * id + a] = hs[(3 + a) * n + i] * (a == b->P.thermo_axis ? lam : 1.0);
    }
  }
  return HMD_OK;
}

int batch_set_state(hmd_batch* b, int sim, const double* x, const double* v) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S || !x || !v) return HMD_EINVAL;
  std::vector<double> hs[6];
  std::vector<int> tag;
  HMD_TRY(download_state(b, hs, tag));
  const SimDev& D = b->sims[sim];
  for (int i = 0; i < D.nf; ++i) {
    const int64_t g = D.a0 + i;
    const int id = tag[g];
    for (int a = 0; a < 3; ++a) {
      hs[a][g] = x[3 * id + a];
      hs[3 + a][g] = v[3 * id + a];
    }
  }
  hipStream_t s = ctx->stream;
  for (int a = 0; a < 6; ++a)
    HMD_HIP(ctx, hipMemcpyAsync(b->d_state[b->cur][a], hs[a].data(), 8 * b->ntot, hipMemcpyHostToDevice, s));
  // the new velocities are final: no Berendsen factor is pending
  hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, b->d_dstate + 3, int64_t(0));
  b->pending = false;
  StepConst K = step_const(b, b->thermo_on, true);
  sort_now(b, K);
  HMD_TRY(forces_now(b, true));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  return HMD_OK;
}

int batch_forces(hmd_batch* b, int sim, float* f, double* pe) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S) return HMD_EINVAL;
  HMD_TRY(forces_now(b, true));
  std::vector<float4> f4(b->ntot);
  std::vector<int> tag(b->ntot);
  hipStream_t s = ctx->stream;
  HMD_HIP(ctx, hipMemcpyAsync(f4.data(), b->d_f4, sizeof(float4) * b->ntot, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(tag.data(), b->d_tag[b->cur], 4 * b->ntot, hipMemcpyDeviceToHost, s));
  double pes = 0.0;
  HMD_HIP(ctx, hipMemcpyAsync(&pes, b->acc.pe[(b->done + 1) & 1] + sim, 8, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  const SimDev& D = b->sims[sim];
  for (int i = 0; i < D.nf; ++i) {
    const int64_t g = D.a0 + i;
    const int id = tag[g];
    if (f) {
      f[3 * id + 0] = f4[g].x;
      f[3 * id + 1] = f4[g].y;
      f[3 * id + 2] = f4[g].z;
    }
  }
  if (pe) *pe = pes;
  return HMD_OK;
}

int batch_cells(hmd_batch* b, int sim, uint32_t* cell_of, uint32_t* counts, uint32_t* order) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S) return HMD_EINVAL;
  const SimDev& D = b->sims[sim];
  std::vector<int> tag(b->ntot);
  std::vector<uint32_t> nc(D.ncell), cell(b->ntot);
  hipStream_t s = ctx->stream;
  if (b->path == 0) {
    std::vector<float4> p4(b->ntot);
    HMD_HIP(ctx, hipMemcpyAsync(p4.data(), b->d_pos4, sizeof(float4) * b->ntot, hipMemcpyDeviceToHost, s));
    HMD_HIP(ctx, hipStreamSynchronize(s));
    for (int64_t g = 0; g < b->ntot; ++g) {
      int lc;
      std::memcpy(&lc, &p4[g].w, 4);
      cell[g] = uint32_t(lc);
    }
  } else {
    // slots carry the Morton-ordered cell; report the row-major id
    std::vector<uint32_t> lin(D.ncell);
    for (int lid = 0; lid < D.ncell; ++lid) lin[b->cell_rank[D.c0 + lid]] = uint32_t(lid);
    HMD_HIP(ctx, hipMemcpyAsync(cell.data(), b->d_slot_cell, 4 * b->ntot, hipMemcpyDeviceToHost, s));
    HMD_HIP(ctx, hipStreamSynchronize(s));
    for (int64_t g = D.a0; g < D.a0 + D.nf; ++g) cell[g] = lin[cell[g] - uint32_t(D.c0)];
  }
  std::vector<uint32_t> st(D.ncell);
  HMD_HIP(ctx, hipMemcpyAsync(tag.data(), b->d_tag[b->cur], 4 * b->ntot, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(nc.data(), b->d_ncount + D.c0, 4 * size_t(D.ncell), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(st.data(), b->d_start + D.c0, 4 * size_t(D.ncell), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  if (cell_of)
    for (int i = 0; i < D.nf; ++i) cell_of[tag[D.a0 + i]] = cell[D.a0 + i];
  // counts and members are stored in Morton order of the cells; report them
  // in row-major cell order, members in the library's order inside a cell
  int64_t w = 0;
  for (int lid = 0; lid < D.ncell; ++lid) {
    const uint32_t key = b->cell_rank[D.c0 + lid];
    if (counts) counts[lid] = nc[key];
    for (uint32_t m = 0; m < nc[key]; ++m, ++w)
      if (order) order[w] = uint32_t(tag[st[key] + m]);
  }
  return HMD_OK;
}

int batch_neighbors(hmd_batch* b, int sim, uint32_t* counts, uint32_t* idx, int64_t cap, int64_t* total) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S || b->path == 0) return HMD_EINVAL;
  const SimDev& D = b->sims[sim];
  std::vector<uint32_t> nl(b->ntot), list(size_t(b->list_cap) * b->list_ld);
  std::vector<int> tag(b->ntot);
  hipStream_t s = ctx->stream;
  // tiled lists hold LDS indices: rebuild them with position indices to read
  // them out, then rebuild them as they were
  if (b->path == 2)
    launch_build(b, s, nullptr, StepRef{nullptr, -1}, state_ref(b, 0), state_ref(b, 0), b->d_tag[0],
                 b->d_tag[0], 1);
  HMD_HIP(ctx, hipMemcpyAsync(nl.data(), b->d_nlist, 4 * b->ntot, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(list.data(), b->d_list, 4 * list.size(), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(tag.data(), b->d_tag[0], 4 * b->ntot, hipMemcpyDeviceToHost, s));
  if (b->path == 2)
    launch_build(b, s, nullptr, StepRef{nullptr, -1}, state_ref(b, 0), state_ref(b, 0), b->d_tag[0],
                 b->d_tag[0], 0);
  HMD_HIP(ctx, hipStreamSynchronize(s));
  // per atom id: neighbour ids (fluid ids, or N_f + wall index of the system)
  std::vector<std::vector<uint32_t>> per(D.nf);
  int64_t tot = 0;
  for (int i = 0; i < D.nf; ++i) {
    const int64_t g = D.a0 + i;
    auto& v = per[tag[g]];
    for (uint32_t k = 0; k < nl[g]; ++k) {
      const uint32_t j = list[(size_t(k >> 2) * b->list_ld + size_t(g)) * 4 + (k & 3u)];
      v.push_back(j < uint32_t(b->ntot) ? uint32_t(tag[j])
                                        : uint32_t(D.nf) + uint32_t(b->wall_id[j - uint32_t(b->ntot)]));
    }
    tot += int64_t(v.size());
  }
  int64_t w = 0;
  for (int id = 0; id < D.nf; ++id) {
    auto& v = per[id];
    std::sort(v.begin(), v.end());
    if (counts) counts[id] = uint32_t(v.size());
    for (uint32_t j : v) {
      if (idx && w < cap) idx[w] = j;
      ++w;
    }
  }
  if (total) *total = tot;
  return HMD_OK;
}

int batch_pairs(hmd_batch* b, int64_t* ff, int64_t* wf) {
  hmd_ctx* ctx = b->ctx;
  HMD_TRY(forces_now(b, true));
  unsigned long long h[kPairCounters * kPairPitch], sum[2] = {0, 0};
  HMD_HIP(ctx, hipMemcpyAsync(h, b->acc.pairs, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int k = 0; k < kPairCounters * kPairPitch; ++k)
    if (k % kPairPitch < 2) sum[k % kPairPitch] += h[k];
  if (ff) *ff = int64_t(sum[0]);
  if (wf) *wf = int64_t(sum[1]);
  return HMD_OK;
}

int batch_list_builds(hmd_batch* b, int64_t* builds) {
  hmd_ctx* ctx = b->ctx;
  int flags[4] = {0, 0, 0, 0};
  HMD_HIP(ctx, hipMemcpyAsync(flags, b->d_flag, sizeof(flags), hipMemcpyDeviceToHost, ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (builds) *builds = b->path >= 1 ? int64_t(flags[3]) : 0;
  return HMD_OK;
}

int batch_profile(hmd_batch* b, int sim, double* mvx, double* cnt) {
  hmd_ctx* ctx = b->ctx;
  if (sim < 0 || sim >= b->S) return HMD_EINVAL;
  const SimDev& D = b->sims[sim];
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  // per-system bins plus, on the tiled path, the system's per-tile bins, which
  // come down together
  const size_t nb = size_t(D.nbins), ld = size_t(b->acc.tb_ld) * 2;
  const size_t ntb = b->d_tbins ? size_t(b->tile_first[sim + 1] - b->tile_first[sim]) : 0;
  const size_t words = 2 * nb + ntb * ld;
  std::vector<double> pageable;
  double* h = static_cast<double*>(stage(ctx, 8 * words));
  if (!h) {
    pageable.resize(words);
    h = pageable.data();
  }
  double *const a = h, *const c = a + nb, *const tb = c + nb;
  hipStream_t s = ctx->stream;
  HMD_HIP(ctx, hipMemcpyAsync(a, b->acc.binvx + D.bin0, 8 * nb, hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipMemcpyAsync(c, b->acc.bincnt + D.bin0, 8 * nb, hipMemcpyDeviceToHost, s));
  if (ntb > 0)
    HMD_HIP(ctx, hipMemcpyAsync(tb, b->d_tbins + size_t(b->tile_first[sim]) * ld, 8 * ntb * ld, hipMemcpyDeviceToHost,
                                s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  for (size_t t = 0; t < ntb; ++t)
    for (size_t k = 0; k < std::min(nb, ld / 2); ++k) {
      a[k] += tb[t * ld + 2 * k];
      c[k] += tb[t * ld + 2 * k + 1];
    }
  if (mvx) std::copy(a, a + nb, mvx);
  if (cnt) std::copy(c, c + nb, cnt);
  return HMD_OK;
}

}  // namespace hmd
