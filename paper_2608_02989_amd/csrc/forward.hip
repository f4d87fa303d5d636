// Grouped SwiGLU expert FFN over the restricted routing (Sec. 3.1, Eq. 2):
// only experts that receive a token are streamed, each once.
//
// Column path (smaller blocks, use_col_path):
//   gate_up    per (active expert, pair of 16-row tiles of I): X_e W_g^T and
//              X_e W_u^T on MFMA (tokens on the 16-wide M side), SwiGLU in
//              registers, the activation written once; the per-expert token
//              lists are derived in the workgroups
//   down       per 16-column tile of H (and half of I), act_e W_d^T for every
//              dispatched (expert, 16-token block), scaled by the gates and
//              summed per token in LDS, then written to out -- no per-slot
//              buffer, no combine pass
// Grouped path (larger blocks):
//   dispatch   per-expert token lists in node order (CSR) and the GEMM items
//   gate_up, down   grouped.hip; down writes gate-scaled rows per slot
//   combine    out_t = sum over the k slots of token t, in slot order
//
// Weights are read in the packed fragment layout (see
// acceptmoe_pack_expert_weights): one wave load = one contiguous 1 KiB block.
#include <type_traits>

#include "ffn_common.hpp"
#include "grouped_plan.hpp"

namespace amoe {

namespace {

constexpr int kDispatchThreads = 1024;
constexpr int kDispatchChunk = 256;   // nodes whose positions a dispatch workgroup finds at a time
constexpr int kDispatchMaxWgs = 256;

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// ---------------------------------------------------------------------------
// weight packing: [E, N, K] row-major -> [E][N/16][K/KF][64 lanes][16 B]
// ---------------------------------------------------------------------------
__global__ void pack_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int E, int N,
                            int rowbytes) {
  const int chunks_per_row = rowbytes / 64;  // 64-byte K chunks per row
  const size_t total = static_cast<size_t>(E) * N * chunks_per_row * 4;  // 16-B pieces
  for (size_t c = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; c < total;
       c += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const int lane = static_cast<int>(c & 63);
    size_t f = c >> 6;  // fragment index = ((e * NT) + nt) * KC + kc
    const int kc = static_cast<int>(f % chunks_per_row);
    f /= chunks_per_row;
    const int nt = static_cast<int>(f % (N / 16));
    const int e = static_cast<int>(f / (N / 16));
    const int row = nt * 16 + (lane & 15);
    const size_t byte = (static_cast<size_t>(e) * N + row) * rowbytes + kc * 64 + (lane >> 4) * 16;
    dst[c] = src[byte / 16];
  }
}

// gate and up stacks [E, I, H] -> [E][I/32 tile pairs][K/KF][4][64 lanes][16 B]:
// fragments gate 2p, gate 2p+1, up 2p, up 2p+1 of each K chunk side by side;
// the second tile of the last pair is zero when I/16 is odd.
__global__ void pack_gate_up_kernel(const uint4* __restrict__ gate, const uint4* __restrict__ up,
                                    uint4* __restrict__ dst, int E, int I, int rowbytes) {
  const int chunks_per_row = rowbytes / 64;
  const int npairs = (I / 16 + 1) / 2;
  const size_t total = static_cast<size_t>(E) * npairs * chunks_per_row * 4 * 64;  // 16-B pieces
  for (size_t c = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; c < total;
       c += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const int lane = static_cast<int>(c & 63);
    const int f = static_cast<int>((c >> 6) & 3);
    size_t q = c >> 8;
    const int kc = static_cast<int>(q % chunks_per_row);
    q /= chunks_per_row;
    const int pair = static_cast<int>(q % npairs);
    const int e = static_cast<int>(q / npairs);
    const int row = (2 * pair + (f & 1)) * 16 + (lane & 15);
    const uint4* src = (f >> 1) ? up : gate;
    dst[c] = row < I ? src[((static_cast<size_t>(e) * I + row) * rowbytes + kc * 64 + (lane >> 4) * 16) / 16]
                     : make_uint4(0u, 0u, 0u, 0u);
  }
}

// Exclusive scan of per-expert counts and compaction of the active experts,
// in index order (one wave, lane = tid < 64).  Returns the number of active
// experts; off[E] = total dispatched slots.
__device__ __forceinline__ int scan_experts(const int* cnt, int* off, int* active, int E, int tid) {
  int base = 0, abase = 0;
  for (int e0 = 0; e0 < E; e0 += kWave) {
    const int e = e0 + tid;
    const int c = e < E ? cnt[e] : 0;
    const int incl = wave_incl_scan_i32(c);
    if (e < E) off[e] = base + incl - c;
    const uint64_t am = __ballot(c > 0);
    if (c > 0) active[abase + popc64(am & lanes_below(tid))] = e;
    abase += popc64(am);
    base += lane_value(incl, kWave - 1);
  }
  if (tid == 0) off[E] = base;
  return abase;
}

// Down-pass items (expert, first CSR row, rows) per block of p.item_rows
// tokens of each active expert, in active-expert order, and their count (one
// wave).
__device__ __forceinline__ void write_down_items(const ForwardParams& p, const int* cnt, const int* off,
                                                 const int* active, int na, int tid) {
  const int ir = p.item_rows;
  int base = 0;
  for (int a0 = 0; a0 < na; a0 += kWave) {
    const int a = a0 + tid;
    const int e = a < na ? active[a] : 0;
    const int c = a < na ? cnt[e] : 0;
    const int nb = (c + ir - 1) / ir;
    const int incl = wave_incl_scan_i32(nb);
    for (int m = 0; m < nb; ++m)
      p.items[base + incl - nb + m] = make_int4(e, off[e] + ir * m, min(ir, c - ir * m), 0);
    base += lane_value(incl, kWave - 1);
  }
  if (tid == 0) *p.n_items = base;
}

// Items (expert, first CSR row, rows) of the grouped GEMMs, as split_rows cuts
// each active expert's rows, and their count (one wave).  The big items, which
// take longest, come first (their count goes to n_big), each group in
// active-expert order.
__device__ __forceinline__ void write_grouped_items(const ForwardParams& p, const int* cnt, const int* off,
                                                    const int* active, int na, int tid) {
  int base = 0;
  for (int big = 1; big >= 0; --big) {
    for (int a0 = 0; a0 < na; a0 += kWave) {
      const int a = a0 + tid;
      const int e = a < na ? active[a] : 0;
      const int c = a < na ? cnt[e] : 0;
      const ItemSplit sp = split_rows(c, p.is_bf16 ? 2 : 4);
      const int first = big != 0 ? 0 : sp.big, n = (big != 0 ? sp.big : sp.items) - first;
      const int incl = wave_incl_scan_i32(n);
      for (int m = first; m < first + n; ++m)
        p.items[base + incl - n + m - first] = make_int4(e, off[e] + sp.rows * m, min(sp.rows, c - sp.rows * m), 0);
      base += lane_value(incl, kWave - 1);
    }
    if (big != 0 && tid == 0) *p.n_big = base;
  }
  if (tid == 0) *p.n_items = base;
}

// ---------------------------------------------------------------------------
// dispatch of the grouped path: CSR of (expert -> slot ids in node order) and
// the items of the grouped GEMMs.  A workgroup writes the lists of
// nodes_per_wg nodes, one chunk of kDispatchChunk after the other: one chunk up to
// kDispatchMaxWgs of them (a workgroup per CU), more chunks beyond, because every
// workgroup counts all rows and a second round of them would count them again
// (whole forward of 1,048,560 nodes, H = I = 64, 64 experts, top-2: 2.4 ms, with one
// chunk per workgroup at any size 16.1 ms; H = 64, I = 32, 512 experts, top-8: 7.2
// and 60.7 ms).
// Every workgroup counts all routing rows, so no workgroup waits for another:
// its own nodes go into per-expert bitmasks, which give both their count and
// their positions (in node order, so the result is deterministic), the nodes
// before and after into counters.  That is one LDS atomic per slot; a wave's
// atomics on a popular expert run one after the other and bound the kernel.
// A wave beyond those that write the lists writes the items (workgroup 0).
// ---------------------------------------------------------------------------
template <int KMAX>
__global__ __launch_bounds__(kDispatchThreads) void dispatch_kernel(ForwardParams p, int nodes_per_wg) {
  constexpr int words = kDispatchChunk / 32;
  constexpr int kItemWave = kDispatchChunk / kWave;  // the first wave without a node of its own
  __shared__ int s_cnt[kMaxExperts];
  __shared__ int s_before[kMaxExperts];
  __shared__ int s_off[kMaxExperts + 1];
  __shared__ int s_active[kMaxExperts];
  __shared__ uint32_t s_mask[kMaxExperts * words];
  __shared__ int s_nact;
  const int tid = threadIdx.x;
  const int E = p.E, k = p.k, T = p.T;
  int c0 = blockIdx.x * nodes_per_wg;  // first node of the current chunk
  const int c_end = min(T, c0 + nodes_per_wg);
  // the node whose list entries this thread writes, loaded beside the clearing
  int own[KMAX];
  uint32_t own_valid = 0u;
  auto load_own = [&]() {
    own_valid = 0u;
    if (tid < kDispatchChunk && c0 + tid < c_end)
      own_valid = load_route_row<KMAX>(p.topk_idx + static_cast<size_t>(c0 + tid) * k, k, E, own);
  };
  auto mark_own = [&]() {
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (own_valid & (1u << j)) atomicOr(&s_mask[own[j] * words + (tid >> 5)], 1u << (tid & 31));
  };
  load_own();
  for (int e = tid; e < E; e += kDispatchThreads) s_cnt[e] = s_before[e] = 0;
  for (int i = tid; i < E * words; i += kDispatchThreads) s_mask[i] = 0u;
  __syncthreads();
  mark_own();
  // the other nodes: i counts the T nodes without the first chunk
  const int n_own = min(kDispatchChunk, c_end - c0);
  for (int i = tid; i < T - n_own; i += kDispatchThreads) {
    const int t = i < c0 ? i : i + n_own;
    int* cnt = i < c0 ? s_before : s_cnt;
    int ev[KMAX];
    const uint32_t valid = load_route_row<KMAX>(p.topk_idx + static_cast<size_t>(t) * k, k, E, ev);
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (valid & (1u << j)) atomicAdd(&cnt[ev[j]], 1);
  }
  __syncthreads();
  for (int e = tid; e < E; e += kDispatchThreads) {
    int c = s_cnt[e] + s_before[e];
#pragma unroll
    for (int w = 0; w < words; ++w) c += __popc(s_mask[e * words + w]);
    s_cnt[e] = c;
  }
  __syncthreads();
  if (tid < kWave) {
    const int na = scan_experts(s_cnt, s_off, s_active, E, tid);
    if (tid == 0) s_nact = na;
  }
  __syncthreads();
  if (blockIdx.x == 0 && wave_id() == kItemWave) write_grouped_items(p, s_cnt, s_off, s_active, s_nact, lane_id());
  for (;;) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (own_valid & (1u << j)) {
        const uint32_t* m = s_mask + own[j] * words;
        int pos = s_off[own[j]] + s_before[own[j]] + __popc(m[tid >> 5] & ((1u << (tid & 31)) - 1u));
#pragma unroll
        for (int w = 0; w < words; ++w) pos += w < (tid >> 5) ? __popc(m[w]) : 0;
        p.ent_slot[pos] = (c0 + tid) * k + j;
      }
    }
    c0 += kDispatchChunk;
    if (c0 >= c_end) break;
    __syncthreads();
    // the finished chunk's nodes come before those of the next
    for (int e = tid; e < E; e += kDispatchThreads) {
      int c = 0;
#pragma unroll
      for (int w = 0; w < words; ++w) {
        c += __popc(s_mask[e * words + w]);
        s_mask[e * words + w] = 0u;
      }
      s_before[e] += c;
    }
    load_own();
    __syncthreads();
    mark_own();
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// In-workgroup dispatch for blocks of up to kSelfMaxT tokens: every gate/up
// workgroup builds the same CSR in LDS from the routing rows (one row per
// thread), so no separate dispatch launch is needed; workgroup 0 also
// publishes it (and the down items) for the down pass.
// ---------------------------------------------------------------------------
constexpr int kSelfMaxT = 256;
constexpr int kSelfMaxSlots = 2048;
constexpr int kSelfWords = kSelfMaxT / 32;

struct SelfDispatch {
  int cnt[kMaxExperts];
  int off[kMaxExperts + 1];
  int active[kMaxExperts];
  uint32_t mask[kMaxExperts * kSelfWords];  // per-expert token bitmasks
  int ent[kSelfMaxSlots];                   // CSR: slot ids grouped by expert, token order
  int nact;
};

// blockDim.x == 256 >= T
template <int KMAX>
__device__ __forceinline__ void self_dispatch(const ForwardParams& p, SelfDispatch& sd, int tid) {
  const int E = p.E, k = p.k, T = p.T;
  const int words = (T + 31) / 32;
  // the routing row first, so its latency overlaps the LDS clearing
  int ev[KMAX];
  uint32_t valid = 0u;
  if (tid < T) valid = load_route_row<KMAX>(p.topk_idx + static_cast<size_t>(tid) * k, k, E, ev);
  for (int i = tid; i < E; i += 256) sd.cnt[i] = 0;
  for (int i = tid; i < E * words; i += 256) sd.mask[i] = 0u;
  __syncthreads();
  if (tid < T) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (valid & (1u << j)) {
        atomicAdd(&sd.cnt[ev[j]], 1);
        atomicOr(&sd.mask[ev[j] * words + (tid >> 5)], 1u << (tid & 31));
      }
    }
  }
  __syncthreads();
  if (tid < kWave) {
    const int na = scan_experts(sd.cnt, sd.off, sd.active, E, tid);
    if (tid == 0) sd.nact = na;
  }
  __syncthreads();
  if (tid < T) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (valid & (1u << j)) {
        const uint32_t* m = sd.mask + ev[j] * words;
        int before = __popc(m[tid >> 5] & ((1u << (tid & 31)) - 1u));
        for (int w = 0; w < (tid >> 5); ++w) before += __popc(m[w]);
        sd.ent[sd.off[ev[j]] + before] = tid * k + j;
      }
    }
  }
  __syncthreads();
}

// Per-item dispatch of the gate/up pass: a workgroup needs only the expert of
// its item (the a-th routed expert in index order, from the block's routed
// mask), that expert's slot ids in node order, its count n_e and its first
// CSR row o_e (the dispatched slots of lower experts) -- a few ballots over
// the routing rows, so the weight stream starts early.
template <int KMAX>
struct ItemDispatch {
  uint32_t emask[kMaxExperts / 32];  // routed experts of the block
  int wcnt[4], wless[4];             // per wave: its tokens of e, its slots below e
  int ent[kSelfMaxT];                // slot ids of e (one per token at most)
  int row[kSelfMaxT][KMAX];          // routing rows, kept here rather than in registers
  uint32_t valid[kSelfMaxT];         // their dispatched slots (load_route_row)
};

// the a-th set bit of mask[0 .. words) (a < number of set bits)
__device__ __forceinline__ int nth_set_bit(const uint32_t* mask, int words, int a) {
  int w = 0;
  for (; w + 1 < words; ++w) {
    const int c = __popc(mask[w]);
    if (a < c) break;
    a -= c;
  }
  uint32_t m = mask[w];
  for (int i = 0; i < a; ++i) m &= m - 1u;  // drop the a lowest set bits
  return 32 * w + __builtin_ctz(m);
}

// CSR rows and down items to the workspace
__device__ __forceinline__ void publish_dispatch(const ForwardParams& p, const SelfDispatch& sd, int tid) {
  const int n_rows = sd.off[p.E];
  for (int i = tid; i < n_rows; i += 256) p.ent_slot[i] = sd.ent[i];
  if (tid == 0) *p.n_rows = n_rows;
  if (tid < kWave) write_down_items(p, sd.cnt, sd.off, sd.active, sd.nact, tid);
}

// k-steps per pipeline stage of the gate/up stream; two stages are kept in flight
constexpr int kGateUpKU = 1;

// sum[nb][mt] += sum over the K chunks c_i = c_first + i * c_step, 0 <= i < n,
// of x[mt] (A, tokens) times w[nb] (B, weight rows).  w[nb] is the wave-uniform
// start of a weight run of wbytes bytes, in which chunk c's fragment sits at
// piece c * wstride + lane; x[mt] points at this lane's 16-byte piece of chunk
// 0 and chunk c sits c * 4 pieces further.  Loads run two stages ahead of the
// MFMAs and carry no branches, so the only waits are the in-order vmcnt
// waits on the stage being consumed.  kSums: sums of 16 of the chunks, then the
// sums (see col_sums); the branch for it sits behind a stage's MFMAs.
template <class P, int MT, int NB, int kPolicy, bool kSums>
__device__ __forceinline__ void stream_tiles(const uint4* const (&w)[NB], int wbytes, const uint4* const (&x)[MT],
                                             int c_first, int c_step, int n, int wstride, floatx4 (&sum)[NB][MT]) {
  constexpr int kU = kGateUpKU;
  floatx4 part[NB][MT];
  floatx4 (&acc)[NB][MT] = kSums ? part : sum;
  if (kSums) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) part[nb][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  auto flush = [&]() {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sum[nb][mt][q] += part[nb][mt][q];
          part[nb][mt][q] = 0.f;
        }
  };
  const int lane = lane_id();
  uint4 wb0[kU][NB], wb1[kU][NB], xb0[kU][MT], xb1[kU][MT];
  auto load0 = [&](int i) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int c = c_first + (i + u) * c_step;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) wb0[u][nb] = load_weight<kPolicy>(w[nb], wbytes, c * wstride + lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xb0[u][mt] = x[mt][c * 4];
    }
  };
  auto load1 = [&](int i) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int c = c_first + (i + u) * c_step;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) wb1[u][nb] = load_weight<kPolicy>(w[nb], wbytes, c * wstride + lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xb1[u][mt] = x[mt][c * 4];
    }
  };
  auto comp0 = [&]() {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nb][mt] = P::mma(xb0[u][mt], wb0[u][nb], acc[nb][mt]);
  };
  auto comp1 = [&]() {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nb][mt] = P::mma(xb1[u][mt], wb1[u][nb], acc[nb][mt]);
  };
  // Steady state without branches: the prefetch of the next stage is issued
  // unconditionally before the current stage is consumed, so the wait-count
  // pass sees straight-line code and only waits for the stage being used.
  // The scheduling barriers keep the compiler from sinking a prefetch below
  // the MFMAs of the stage before it (which would drain the pipeline: the
  // waits for the current stage would then come before the next loads).
  // The last one or two stages are peeled off after the loop.
  const int nst = n / kU;
  if (nst > 0) {
    load0(0);
    int st = 0;
    for (; st + 2 < nst; st += 2) {
      load1((st + 1) * kU);
      __builtin_amdgcn_sched_barrier(0);
      comp0();
      load0((st + 2) * kU);
      __builtin_amdgcn_sched_barrier(0);
      comp1();
      if (kSums && st % 16 == 14) flush();
    }
    if (st + 1 < nst) {
      load1((st + 1) * kU);
      __builtin_amdgcn_sched_barrier(0);
      comp0();
      comp1();
    } else {
      comp0();
    }
  }
  for (int i = nst * kU; i < n; ++i) {
    const int c = c_first + i * c_step;
    uint4 wt[NB], xt[MT];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wt[nb] = load_weight<kPolicy>(w[nb], wbytes, c * wstride + lane);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xt[mt] = x[mt][c * 4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nb][mt] = P::mma(xt[mt], wt[nb], acc[nb][mt]);
  }
  if (kSums) flush();
}

// ---------------------------------------------------------------------------
// Gate/up pass (blocks of up to kSelfMaxT tokens).  A workgroup (4 waves) owns
// one pair of 16-row tiles of I of one active expert, gate and up.  Its waves
// split the K chunks round-robin (wave s takes chunks s, s + 4, ...; the
// workgroup reads the pair's weight run front to back, which keeps the DRAM
// accesses of the whole chip in far fewer open rows than per-wave K ranges)
// and add their partial tiles in LDS in a fixed order (deterministic).  The
// gate and up fragments of a pair are adjacent in the packed layout
// ([E][I/32][K chunk][gate 2p, gate 2p+1, up 2p, up 2p+1]), so a K chunk of
// the pair is one 4 KiB run.  A = gathered hidden rows; SwiGLU -> act (bf16
// for the bf16 path, fp32 otherwise), written once per token row.
// ---------------------------------------------------------------------------
constexpr int kGateUpKS = 4;       // waves splitting K
constexpr int kTilesPerWG = 2;     // one tile pair
constexpr int kGateUpFrags = 4;    // weight fragments per K chunk

// ent_e: the n_e slot ids of expert e in node order; o_e: its first row in act
template <class P, int MT, bool kSums>
__device__ __forceinline__ void gate_up_pass(const ForwardParams& p, const int32_t* ent_e, int e, int tile0, int n_e,
                                             int o_e, int m0, floatx4 (*red)[kWave][4]) {
  constexpr int NB = kGateUpFrags, KS = kGateUpKS;
  const int wave = wave_id(), lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  const int ntiles = p.I / 16;
  const int KC = p.H / P::kKF;
  const int rowq = p.H * P::kElemBytes / 16;

  const uint4* x[MT];
  const uint4* hid = static_cast<const uint4*>(p.hidden);
  const int tok0 = ent_e[0] / p.k;  // rows past n_e read a valid row; their outputs are dropped
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m0 + mt * 16 + r;
    const int tok = m < n_e ? ent_e[m] / p.k : tok0;
    x[mt] = hid + static_cast<size_t>(tok) * rowq + g;
  }
  // wave-uniform starts of the weight runs
  const int npairs = (ntiles + 1) / 2;
  const uint4* base = uniform_ptr(static_cast<const uint4*>(p.w_gate_up) +
                                  (static_cast<size_t>(e) * npairs + tile0 / 2) * KC * 4 * kWave);
  const uint4* w[NB];
  w[0] = base;              // gate, tile 2 pair
  w[1] = base + 2 * kWave;  // up, tile 2 pair
  w[2] = base + kWave;      // gate, tile 2 pair + 1
  w[3] = base + 3 * kWave;  // up, tile 2 pair + 1
  const int wstride = 4 * kWave;                                // 16-byte pieces from one K chunk to the next
  const int wbytes = KC * 4 * kWave * 16 - 3 * kWave * 16;      // the last fragment of w[3] ends the pair's run
  floatx4 acc[NB][MT];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nb][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  stream_tiles<P, MT, NB, kPolicyStream, kSums>(w, wbytes, x, wave, KS, (KC - wave + KS - 1) / KS, wstride, acc);

  // fixed-order sum of the KS partial tiles, four fragments per LDS round
#pragma unroll
  for (int q0 = 0; q0 < NB * MT; q0 += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][lane][q] = acc[(q0 + q) / MT][(q0 + q) % MT];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int s2 = 1; s2 < KS; ++s2)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const floatx4 v = red[s2][lane][q];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[(q0 + q) / MT][(q0 + q) % MT][i] += v[i];
        }
    }
    __syncthreads();
  }
  if (wave == 0) {
#pragma unroll
    for (int j = 0; j < kTilesPerWG; ++j) {
      const int tile = tile0 + j;
      if (tile >= ntiles) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = m0 + mt * 16 + 4 * g + i;
          if (m < n_e) {
            const float v = silu_mul(acc[2 * j][mt][i], acc[2 * j + 1][mt][i]);
            const size_t idx = static_cast<size_t>(o_e + m) * p.I + tile * 16 + r;
            if (P::kElemBytes == 2)
              static_cast<uint16_t*>(p.act)[idx] = float_to_bf16_bits(v);
            else
              static_cast<float*>(p.act)[idx] = v;
          }
        }
      }
    }
  }
}

// the full CSR is built only by the publishing workgroup
template <int KMAX>
union DispatchSlot {
  SelfDispatch sd;
  ItemDispatch<KMAX> id;
};

// Work item i = (active expert i / wg_per_expert, tile run i % wg_per_expert).
// A grid of up to kSelfGridMult times the workgroups resident at once (H >= 4096; once otherwise) takes items blockIdx.x,
// blockIdx.x + gridDim.x, ..., each with its own per-item dispatch.  The
// workgroups beyond the resident ones start on whichever CU frees a slot
// first, which evens out the CUs' finish times (CUs stream at up to 20 %
// different rates): at H = 4096, T = 64 the pass took 121.1 us with a
// resident-sized grid and 117.8 us with three times that.  The shorter items
// of H = 2048 (256 KiB) do not repay the prologue each extra workgroup
// repeats: the 48-layer pass at T = 60 ran 4951, 4990 and 5054 us per block
// with one, two and three times the resident grid.  Workgroups left without
// an item exit after the prologue.  Workgroup 0 takes no item: it builds the
// full CSR and publishes it for the down pass, beside the others' streams
// (after an item of its own that work ended 2-3 us behind every other
// workgroup: one token's gate/up pass 12.8 us, of it 10.4 for the items).
// (Claiming items from a device-wide counter was measured no better.)
constexpr int kSelfGridMult = 3;

// Occupancy floor: three workgroups per CU for up to two M-tiles, two for
// more (the register budget the streaming loop is tuned to).
template <class P, int MTMAX, int KMAX, bool kSums>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MTMAX <= 2 ? 3 : 2))) void gate_up_kernel(
    ForwardParams p) {
  __shared__ floatx4 red[kGateUpKS][kWave][4];
  __shared__ DispatchSlot<KMAX> ds;
  const int ntiles = p.I / 16;
  const int wg_per_expert = (ntiles + kTilesPerWG - 1) / kTilesPerWG;
  if (p.zero_out) {
    // the column-tile down pass adds its two halves of I into out
    float4* o4 = reinterpret_cast<float4*>(p.out);
    const size_t n4 = static_cast<size_t>(p.T) * p.H / 4;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
         i += static_cast<size_t>(gridDim.x) * blockDim.x)
      o4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  auto run_expert = [&](int tile0, int e, int n_e, int o_e, const int32_t* ent_e) {
    for (int m0 = 0; m0 < n_e; m0 += 16 * MTMAX) {
      const int mt = min(MTMAX, (n_e - m0 + 15) / 16);
      if (mt == 1) gate_up_pass<P, 1, kSums>(p, ent_e, e, tile0, n_e, o_e, m0, red);
      else if (MTMAX >= 2 && mt == 2) gate_up_pass<P, (MTMAX >= 2 ? 2 : 1), kSums>(p, ent_e, e, tile0, n_e, o_e, m0, red);
      else if (MTMAX >= 3 && mt == 3) gate_up_pass<P, (MTMAX >= 3 ? 3 : 1), kSums>(p, ent_e, e, tile0, n_e, o_e, m0, red);
      else gate_up_pass<P, MTMAX, kSums>(p, ent_e, e, tile0, n_e, o_e, m0, red);
    }
  };
  const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  if (blockIdx.x == 0) {
    SelfDispatch& sd = ds.sd;
    self_dispatch<KMAX>(p, sd, tid);
    publish_dispatch(p, sd, tid);
    return;
  }
  ItemDispatch<KMAX>& id = ds.id;
  const int T = p.T, k = p.k, E = p.E, words = (E + 31) / 32;
  if (tid < kMaxExperts / 32) id.emask[tid] = 0u;
  {
    int ev[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) ev[j] = -1;
    uint32_t valid = 0u;
    if (tid < T) {
      valid = load_route_row<KMAX>(p.topk_idx + static_cast<size_t>(tid) * k, k, E, ev);
#pragma unroll
      for (int j = 0; j < KMAX; ++j) id.row[tid][j] = ev[j];
      id.valid[tid] = valid;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (valid & (1u << j)) atomicOr(&id.emask[ev[j] >> 5], 1u << (ev[j] & 31));
  }
  __syncthreads();
  // workgroup-uniform values go to scalar registers (the streaming loop
  // needs every vector register it can get)
  int nact = 0;
  for (int w = 0; w < words; ++w) nact += __popc(id.emask[w]);
  nact = __builtin_amdgcn_readfirstlane(nact);
  const int n_items = nact * wg_per_expert;
  for (int item = blockIdx.x - 1; item < n_items; item += gridDim.x - 1) {
    const int e = __builtin_amdgcn_readfirstlane(nth_set_bit(id.emask, words, item / wg_per_expert));
    // this thread's token: its slot of e, and its slots of lower experts
    int slot = -1, less = 0;
    if (tid < T) {
      const uint32_t valid = id.valid[tid];
#pragma unroll
      for (int j = 0; j < KMAX; ++j) {
        const int ej = id.row[tid][j];
        if (valid & (1u << j)) {
          slot = ej == e ? static_cast<int>(tid) * k + j : slot;
          less += ej < e ? 1 : 0;
        }
      }
    }
    const uint64_t hm = __ballot(slot >= 0);
    const int wless = wave_sum_i32(less);
    __syncthreads();  // the previous item's list is no longer read
    if (lane == 0) {
      id.wcnt[wave] = popc64(hm);
      id.wless[wave] = wless;
    }
    __syncthreads();
    int before = 0, n_e = 0, o_e = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      before += w < wave ? id.wcnt[w] : 0;
      n_e += id.wcnt[w];
      o_e += id.wless[w];
    }
    if (slot >= 0) id.ent[before + popc64(hm & lanes_below(lane))] = slot;
    __syncthreads();
    run_expert((item % wg_per_expert) * kTilesPerWG, e, __builtin_amdgcn_readfirstlane(n_e),
               __builtin_amdgcn_readfirstlane(o_e), id.ent);
  }
}

// ---------------------------------------------------------------------------
// Column-tile down pass (blocks of up to kColMaxT tokens).  A workgroup owns
// NB adjacent 16-column tiles of H and one of `ksplit` (1 or 2) parts of I.
// It streams those tiles' rows of W_d for every down item (expert e, block of
// up to 16 MTI tokens of e's list): the items are dealt round-robin to the
// waves, and each wave runs one continuous two-stage load pipeline across its
// items.  The MTI M-tiles of an item share every weight fragment, so an
// expert's slice of W_d is streamed once per 16 MTI tokens (an expert with 17
// to 32 tokens took two passes over it with 16-token items; the second mostly
// from L2, yet the pass ran at 4.6 instead of 5.9 TB/s).  A second M-tile with
// no token reads a valid row again (a cache hit); its products are dropped.
// After an item's last stage the wave adds gate * (act_e W_d^T) into its own
// LDS accumulator out_w[t, 16 NB columns] (a token appears once per expert, so
// the lanes of one item never collide).  At the end the waves' accumulators are
// summed in wave order and written to out, or added into the zeroed out when
// I is split in two (two fp32 additions onto zero commute, so the result
// does not depend on which half lands first).  Every workgroup does the same
// work; its LDS footprint keeps it alone on its CU.  Each workgroup reads
// every dispatched activation row once, so NB = 2 halves that traffic per
// column for wide H.
// ---------------------------------------------------------------------------
constexpr int kColLanes = 8;  // waves x NB: the accumulators take kColLanes x kColMaxT x 16 floats
constexpr int kColMaxT = 256;
constexpr int kColMaxSlots = 2048;
constexpr int kColMaxItems = kMaxExperts + kColMaxSlots / 16;

struct ColShared {
  float acc[kColLanes * kColMaxT * 16];  // per-wave token accumulators [wave][t][16 NB]
  int tok[kColMaxSlots];                 // CSR row -> token
  float gw[kColMaxSlots];                // CSR row -> gate of that slot
  int4 items[kColMaxItems];
};

template <class P, int kU, int NB, int MTI, bool kSums>
__global__ __launch_bounds__(kColLanes / NB * kWave) void down_col_kernel(ForwardParams p, int ksplit) {
  constexpr int kWaves = kColLanes / NB;
  constexpr int kThreads = kWaves * kWave;
  constexpr int kCols = 16 * NB;
  __shared__ ColShared sh;
  const int tid = threadIdx.x;
  const int wave = wave_id(), lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  const int T = p.T, H = p.H, k = p.k;
  const int ntiles = H / 16;
  const int ngroups = ntiles / NB;
  const int ht0 = (blockIdx.x % ngroups) * NB, part = blockIdx.x / ngroups;
  const int KC = p.I / P::kKF;
  const int kc0 = part * KC / ksplit;
  const int L = (KC / ksplit) / kU;  // pipeline stages per item
  const int rowq = p.I * P::kElemBytes / 16;
  const int n_items = *p.n_items;
  const int n_rows = *p.n_rows;
  // this wave's first item straight from the workspace, so the first stage's
  // loads are in flight while the lists are staged in LDS
  int4 first = make_int4(0, 0, 1, 0);
  if (wave < n_items) first = p.items[wave];
  for (int i = tid; i < kWaves * T * kCols; i += kThreads) sh.acc[i] = 0.f;
  for (int i = tid; i < n_rows; i += kThreads) {
    const int slot = p.ent_slot[i];
    sh.tok[i] = slot / k;
    sh.gw[i] = p.topk_gate[slot];
  }
  for (int i = tid; i < n_items; i += kThreads) sh.items[i] = p.items[i];

  const uint4* wd = static_cast<const uint4*>(p.w_down);
  const uint4* act = static_cast<const uint4*>(p.act);
  float* accw = sh.acc + wave * T * kCols;
  // items wave, wave + kWaves, ...; stage = (item, q), q in [0, L)
  const int my_items = n_items > wave ? (n_items - wave + kWaves - 1) / kWaves : 0;
  const int nst = my_items * L;
  struct Cursor {
    int it, q, e, row0, nrows;
  };
  auto fetch = [&](Cursor& c) {
    if (c.it < n_items) {
      const int4 d = sh.items[c.it];
      c.e = d.x;
      c.row0 = d.y;
      c.nrows = d.z;
    }
  };
  auto advance = [&](Cursor& c) {
    if (++c.q == L) {
      c.q = 0;
      c.it += kWaves;
      fetch(c);
    }
  };
  uint4 w0[kU][NB], x0[kU][MTI], w1[kU][NB], x1[kU][MTI];
  auto load = [&](uint4 (&wv)[kU][NB], uint4 (&xv)[kU][MTI], const Cursor& c) {
    const int kc = kc0 + c.q * kU;
    const uint4* xp[MTI];
#pragma unroll
    for (int mt = 0; mt < MTI; ++mt)
      xp[mt] = act + static_cast<size_t>(c.row0 + min(16 * mt + r, c.nrows - 1)) * rowq + g + kc * 4;
    const uint4* wrun = uniform_ptr(wd + (static_cast<size_t>(c.e) * ntiles + ht0) * KC * kWave);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        wv[u][nb] = load_weight<NB == 2 ? kPolicyPlain : kPolicyStream>(wrun, NB * KC * kWave * 16,
                                                                        (nb * KC + kc + u) * kWave + lane);
#pragma unroll
      for (int mt = 0; mt < MTI; ++mt) xv[u][mt] = xp[mt][u * 4];
    }
  };
  constexpr int kRun = 16 / kU > 0 ? 16 / kU : 1;  // stages of a sum
  floatx4 acc[NB][MTI], sum[NB][MTI];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mt = 0; mt < MTI; ++mt) acc[nb][mt] = sum[nb][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](uint4 (&wv)[kU][NB], uint4 (&xv)[kU][MTI], Cursor& c) {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MTI; ++mt) acc[nb][mt] = P::mma(xv[u][mt], wv[u][nb], acc[nb][mt]);
    if (kSums && (c.q % kRun == kRun - 1 || c.q == L - 1)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MTI; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            sum[nb][mt][i] += acc[nb][mt][i];
            acc[nb][mt][i] = 0.f;
          }
    }
    if (c.q == L - 1) {
      // item done: out_w[t] += gate * row, rows 16 mt + 4g .. +3 of the item, column r of each tile
#pragma unroll
      for (int mt = 0; mt < MTI; ++mt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = 16 * mt + 4 * g + i;
          if (m < c.nrows) {
            const int row = c.row0 + m;
            float* dst = accw + sh.tok[row] * kCols + r;
            const float gt = sh.gw[row];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) dst[16 * nb] += gt * (kSums ? sum : acc)[nb][mt][i];
          }
        }
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MTI; ++mt) acc[nb][mt] = sum[nb][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    advance(c);
  };
  Cursor lc{wave, 0, first.x, first.y, first.z}, cc{wave, 0, first.x, first.y, first.z};
  if (nst > 0) load(w0, x0, lc);
  __syncthreads();  // lists staged, accumulators cleared (advance reads the staged items)
  if (nst > 0) {
    advance(lc);
    int st = 0;
    for (; st + 2 < nst; st += 2) {
      load(w1, x1, lc);
      advance(lc);
      compute(w0, x0, cc);
      load(w0, x0, lc);
      advance(lc);
      compute(w1, x1, cc);
    }
    if (st + 1 < nst) {
      load(w1, x1, lc);
      compute(w0, x0, cc);
      compute(w1, x1, cc);
    } else {
      compute(w0, x0, cc);
    }
  }
  __syncthreads();
  // fixed-order sum over the waves, then out (or out += for a half of I)
  for (int i = tid; i < T * kCols; i += kThreads) {
    float v = sh.acc[i];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += sh.acc[w * T * kCols + i];
    float* o = p.out + static_cast<size_t>(i / kCols) * H + ht0 * 16 + (i % kCols);
    if (ksplit == 2) atomicAdd(o, v);
    else *o = v;
  }
}

// ---------------------------------------------------------------------------
// combine: out[t, h] = sum over the dispatched slots of token t, in slot order.
// The routing row and all k expert rows are loaded before any is used (rows
// of skipped slots are read but discarded).  Workgroup b covers token
// b / hblocks, float4 columns 256 (b % hblocks) ..; a one-dimensional grid, so
// any T fits.
// ---------------------------------------------------------------------------
template <int KMAX>
__global__ __launch_bounds__(256) void combine_kernel(ForwardParams p, int hblocks) {
  const int t = blockIdx.x / hblocks;
  const int h4 = (blockIdx.x % hblocks) * blockDim.x + threadIdx.x;  // float4 column
  const int H = p.H, k = p.k;
  if (h4 * 4 >= H) return;
  int ev[KMAX];
  const uint32_t valid = load_route_row<KMAX>(p.topk_idx + static_cast<size_t>(t) * k, k, p.E, ev);
  float4 v[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    const int jj = j < k ? j : k - 1;
    v[j] = reinterpret_cast<const float4*>(p.ys + (static_cast<size_t>(t) * k + jj) * H)[h4];
  }
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    if (valid & (1u << j)) {
      s.x += v[j].x;
      s.y += v[j].y;
      s.z += v[j].z;
      s.w += v[j].w;
    }
  }
  reinterpret_cast<float4*>(p.out + static_cast<size_t>(t) * H)[h4] = s;
}

// Workgroups of kernel `Kern` (256 threads) resident on the current device at
// once, computed on first use per kernel and device (a template per kernel, so
// kernels of different register or LDS needs keep separate counts).
template <auto Kern>
int resident_workgroups() {
  constexpr int kMaxDevices = 64;
  static int cached[kMaxDevices] = {};
  const auto kernel = Kern;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  if (cached[dev] == 0) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1;
    cached[dev] = per_cu * cus;
  }
  return cached[dev];
}

// Rows of 9 to 16 slots have an instantiation of their own: the search for
// repeated experts grows with the square of the row (512 experts, top-10,
// T = 64: 9.7 us before the first weight with rows of 32, pass 93.5 -> 82.7 us).
template <class P, int MTMAX, bool kSums = false>
hipError_t launch_gate_up(const ForwardParams& p, int cap, hipStream_t stream) {
  const int items = cap * ((p.I / 16 + kTilesPerWG - 1) / kTilesPerWG);
  if (p.k <= 8) {
    constexpr auto kern = &gate_up_kernel<P, MTMAX, 8, kSums>;
    const int res = (p.H >= 4096 ? kSelfGridMult : 1) * resident_workgroups<kern>();
    kern<<<dim3((items < res ? items : res) + 1), 256, 0, stream>>>(p);
  } else if (p.k <= 16) {
    constexpr auto kern = &gate_up_kernel<P, MTMAX, 16, kSums>;
    const int res = (p.H >= 4096 ? kSelfGridMult : 1) * resident_workgroups<kern>();
    kern<<<dim3((items < res ? items : res) + 1), 256, 0, stream>>>(p);
  } else {
    constexpr auto kern = &gate_up_kernel<P, MTMAX, kMaxTopK, kSums>;
    const int res = (p.H >= 4096 ? kSelfGridMult : 1) * resident_workgroups<kern>();
    kern<<<dim3((items < res ? items : res) + 1), 256, 0, stream>>>(p);
  }
  return hipGetLastError();
}

// Column-tile down pass shape: I split in two when that keeps the grid near
// 256 workgroups, two column tiles per workgroup for wide H, k-steps per
// pipeline stage: the largest of 12, 8, 6, 4, 3, 2, 1 dividing the part of I,
// at most 12 with one column tile (two stages in flight then fit the
// registers of one 8-wave workgroup per CU, and the deeper stages keep more
// bytes in flight: 12 vs 4 k-steps measured 0.6 us faster at H = 2048,
// I = 768) and at most 4 with two (whose stages already carry twice the
// weight bytes; 8 measured slower at H = 4096, I = 1536).  Thin parts of I
// (one GPU's share of a tensor-parallel split) give lengths like 3, where
// 3-step stages ran 11 % faster than single steps.
struct ColShape {
  int ksplit, ku, nb, mti;
};

// M-tiles per down item: two (items of up to 32 tokens) for blocks of more
// than 32 tokens when the workgroup owns two column tiles, whose stages are
// capped at 4 k-steps either way (H = 4096, T = 64: forward 188.7 -> 182.9 us);
// with one column tile a second M-tile would halve the 12-k-step stages, which
// cost more than it saves where experts receive ~10 tokens (H = 2048, T = 60:
// 48-layer pass 4926 -> 5063 us per block).
ColShape col_shape(int T, int H, int I, int is_bf16) {
  const int KC = I / (is_bf16 ? Bf16Path::kKF : F32Path::kKF);
  const int ntiles = H / 16;
  ColShape c;
  c.nb = (ntiles >= 256 && ntiles % 2 == 0) ? 2 : 1;
  c.mti = T > 32 && c.nb == 2 ? 2 : 1;
  c.ksplit = (ntiles / c.nb <= 128 && KC % 2 == 0) ? 2 : 1;
  const int len = KC / c.ksplit;
  const int ku_max = c.nb == 1 ? 12 : 4;
  c.ku = 1;
  for (const int u : {12, 8, 6, 4, 3, 2}) {
    if (len % u == 0 && u <= ku_max) {
      c.ku = u;
      break;
    }
  }
  return c;
}

// Column path (gate/up with its own dispatch, then the column-tile down pass)
// or grouped path (dispatch, grouped GEMMs, combine).  The column path's lists
// hold 256 tokens and 2048 slots; up to 96 tokens (fp32: 192), or with a thin I,
// which leaves the grouped gate/up one or two workgroups per expert, that path is
// taken.  Beyond, the line is where two costs meet.  Every workgroup of the
// column path's down pass reads all slots' activations, so it is behind once
// slots x I per down workgroup is large (three times earlier where the down
// stages are single k-steps).  The grouped path pays two more launches, the slot
// rows and, with few rows per expert, M-tiles that are mostly padding; from 12
// rows per expert on it gains in bf16 whatever the rest (both projections re-read
// an expert's rows once per 128 or 256 outputs, not once per 32 or 16), but not in
// fp32, whose products leave no such slack.  Whole steps, us, column / grouped:
//   H = 2048, I = 768    E = 128: k = 1, T = 160 102 / 121; k = 2, T = 100 91 / 113; k = 8, T = 160 210 / 201
//                        E = 64: k = 2, T = 160 96 / 115; k = 8, T = 256 225 / 154
//                        E = 16, k = 1: T = 100 46 / 57, T = 256 64 / 60
//   H = 1024, I = 512    E = 64: k = 1, T = 100 39 / 45; k = 8, T = 100 78 / 66
//   H = 4096, I = 1536   E = 128: k = 1, T = 100 202 / 221; k = 8, T = 256 822 / 764
//   fp32, H = 2048, I = 768   E = 64: k = 1, T = 200 162 / 197; k = 8, T = 256 456 / 329
//   fp32, H = 3584, I = 256   E = 160, k = 8, T = 195 262 / 285
// and below 96 tokens, E = 128, k = 8: H = 2048, I = 768, T = 72 117 / 128, T = 96
// 130 / 134; H = 4096, I = 1536, T = 72 323 / 330, T = 96 353 / 349.
// Over 789 (fp32: 448) layers and blocks of 97 (193) to 256 tokens, drawn and on a
// grid of H, I, E and k, this choice is 0.24 % (0.8 %) behind the faster path on
// average and in fp32 at most 8 % behind the column path; the grouped path
// throughout is 1.3 % (1.2 %) behind, up to 38 % (39 %).
bool use_col_path(int T, int H, int I, int E, int k, int is_bf16) {
  const long long slots = static_cast<long long>(T) * k;
  if (T > kColMaxT || T > kSelfMaxT || slots > kColMaxSlots || slots > kSelfMaxSlots) return false;
  if (T <= (is_bf16 ? 96 : 192) || I < 256) return true;
  if (is_bf16 && slots > 12ll * E) return false;
  const ColShape c = col_shape(T, H, I, is_bf16);
  const long long down_wgs = static_cast<long long>(H / 16 / c.nb) * c.ksplit;
  return slots * I <= (c.ku == 1 ? 640 : 1920) * down_wgs;
}

// fp32 blocks of more than 192 tokens on the column path add sums of 16 chunks, as
// the grouped path does for the blocks beside them: error against 64 bits 4.9e-7,
// 5.1e-7 grouped, 6.9e-7 with one running sum (200 tokens, 128 experts, top-1,
// H = 2048, I = 768).  The second accumulators leave room for three M-tiles in
// gate/up.  Smaller blocks keep one running sum: a few tokens are up to 4 % slower
// with sums.
constexpr int kColSumsT = 192;
bool col_sums(const ForwardParams& p) { return !p.is_bf16 && p.T > kColSumsT; }

template <class P, int NB, int MTI, bool kSums = false>
hipError_t launch_down_col_nb(const ForwardParams& p, const ColShape& c, hipStream_t stream) {
  const dim3 grid((p.H / 16 / NB) * c.ksplit);
  constexpr int threads = kColLanes / NB * kWave;
  if constexpr (NB == 1) {  // deeper stages only with one column tile (col_shape)
    if (c.ku > 4) {
      if (c.ku == 12) down_col_kernel<P, 12, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
      else if (c.ku == 8) down_col_kernel<P, 8, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
      else down_col_kernel<P, 6, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
      return hipGetLastError();
    }
  }
  if (c.ku == 4) down_col_kernel<P, 4, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
  else if (c.ku == 3) down_col_kernel<P, 3, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
  else if (c.ku == 2) down_col_kernel<P, 2, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
  else down_col_kernel<P, 1, NB, MTI, kSums><<<grid, threads, 0, stream>>>(p, c.ksplit);
  return hipGetLastError();
}

template <class P>
hipError_t launch_down_col(const ForwardParams& p, const ColShape& c, hipStream_t stream) {
  if constexpr (P::kElemBytes == 4)
    if (col_sums(p))  // more than 32 tokens, so mti = nb
      return c.nb == 2 ? launch_down_col_nb<P, 2, 2, true>(p, c, stream) : launch_down_col_nb<P, 1, 1, true>(p, c, stream);
  if (c.nb == 1) return launch_down_col_nb<P, 1, 1>(p, c, stream);
  return c.mti == 2 ? launch_down_col_nb<P, 2, 2>(p, c, stream) : launch_down_col_nb<P, 2, 1>(p, c, stream);
}

}  // namespace

size_t packed_gate_up_bytes(int is_bf16, int E, int I, int H) {
  return static_cast<size_t>(E) * ((I / 16 + 1) / 2) * 32 * H * (is_bf16 ? 2 : 4) * 2;
}

hipError_t launch_pack_gate_up(const void* gate, const void* up, int is_bf16, int E, int I, int H, void* dst,
                               hipStream_t stream) {
  const size_t pieces = packed_gate_up_bytes(is_bf16, E, I, H) / 16;
  const int block = 256;
  const size_t want = (pieces + block - 1) / block;
  const int grid = static_cast<int>(want < 65536 ? want : 65536);
  pack_gate_up_kernel<<<grid, block, 0, stream>>>(static_cast<const uint4*>(gate), static_cast<const uint4*>(up),
                                                  static_cast<uint4*>(dst), E, I, H * (is_bf16 ? 2 : 4));
  return hipGetLastError();
}

hipError_t launch_pack(const void* src, int is_bf16, int E, int N, int K, void* dst, hipStream_t stream) {
  const int rowbytes = K * (is_bf16 ? 2 : 4);
  const size_t pieces = static_cast<size_t>(E) * N * rowbytes / 16;
  const int block = 256;
  const size_t want = (pieces + block - 1) / block;
  const int grid = static_cast<int>(want < 65536 ? want : 65536);
  pack_kernel<<<grid, block, 0, stream>>>(static_cast<const uint4*>(src), static_cast<uint4*>(dst), E,
                                          N, rowbytes);
  return hipGetLastError();
}

int max_grouped_items(int T, int E, int k, int is_bf16) {
  return grouped_max_items(T * k, E, grouped_item_rows(is_bf16 ? 2 : 4));
}

// workspace: [n_items | n_big | n_rows] ints, CSR slot
// ids, activations, then the items of the grouped GEMMs and the per-slot
// output rows (grouped path) or the down items (column-tile path)
size_t forward_workspace_bytes(int T, int H, int I, int E, int k, int is_bf16) {
  const size_t slots = static_cast<size_t>(T) * k;
  const size_t eb = is_bf16 ? 2 : 4;
  const size_t head = align256(sizeof(int32_t) * 3) +
                      align256(sizeof(int32_t) * slots) + align256(slots * I * eb);
  if (use_col_path(T, H, I, E, k, is_bf16)) {
    const size_t items = (slots + 15) / 16 + (static_cast<size_t>(E) < slots ? E : slots);
    return head + align256(items * sizeof(int4));
  }
  return head + align256(static_cast<size_t>(max_grouped_items(T, E, k, is_bf16)) * sizeof(int4)) +
         align256(slots * H * sizeof(float));
}

void forward_carve(void* ws, ForwardParams& p) {
  char* c = static_cast<char*>(ws);
  const size_t slots = static_cast<size_t>(p.T) * p.k;
  const size_t eb = p.is_bf16 ? 2 : 4;
  int32_t* ints = reinterpret_cast<int32_t*>(c);
  p.n_items = ints;
  p.n_big = ints + 1;
  p.n_rows = ints + 2;
  c += align256(sizeof(int32_t) * 3);
  p.ent_slot = reinterpret_cast<int32_t*>(c);
  c += align256(sizeof(int32_t) * slots);
  p.act = c;
  c += align256(slots * p.I * eb);
  if (use_col_path(p.T, p.H, p.I, p.E, p.k, p.is_bf16)) {
    p.items = reinterpret_cast<int4*>(c);
    p.ys = nullptr;
  } else {
    p.items = reinterpret_cast<int4*>(c);
    c += align256(static_cast<size_t>(max_grouped_items(p.T, p.E, p.k, p.is_bf16)) * sizeof(int4));
    p.ys = reinterpret_cast<float*>(c);
  }
}

hipError_t launch_forward(ForwardParams p, hipStream_t stream) {
  hipError_t err = hipSuccess;
  if (use_col_path(p.T, p.H, p.I, p.E, p.k, p.is_bf16)) {
    const ColShape cs = col_shape(p.T, p.H, p.I, p.is_bf16);
    p.zero_out = cs.ksplit == 2;
    p.item_rows = 16 * cs.mti;
    // upper bound on active experts: min(E, T*k)
    const int cap = p.E < p.T * p.k ? p.E : p.T * p.k;
    const bool small_t = p.T <= 32;
    if (p.is_bf16)
      err = small_t ? launch_gate_up<Bf16Path, 2>(p, cap, stream) : launch_gate_up<Bf16Path, 4>(p, cap, stream);
    else
      err = small_t ? launch_gate_up<F32Path, 2>(p, cap, stream)
            : col_sums(p) ? launch_gate_up<F32Path, 3, true>(p, cap, stream) : launch_gate_up<F32Path, 4>(p, cap, stream);
    if (err != hipSuccess) return err;
    return p.is_bf16 ? launch_down_col<Bf16Path>(p, cs, stream) : launch_down_col<F32Path>(p, cs, stream);
  }
  const int chunks = (p.T + kDispatchChunk - 1) / kDispatchChunk;
  const int per_wg = (chunks + kDispatchMaxWgs - 1) / kDispatchMaxWgs * kDispatchChunk;
  const int wgs = (p.T + per_wg - 1) / per_wg;
  if (p.k <= 8)
    dispatch_kernel<8><<<wgs, kDispatchThreads, 0, stream>>>(p, per_wg);
  else if (p.k <= 16)
    dispatch_kernel<16><<<wgs, kDispatchThreads, 0, stream>>>(p, per_wg);
  else
    dispatch_kernel<kMaxTopK><<<wgs, kDispatchThreads, 0, stream>>>(p, per_wg);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  err = launch_grouped(p, max_grouped_items(p.T, p.E, p.k, p.is_bf16), stream);
  if (err != hipSuccess) return err;
  const int hblocks = (p.H / 4 + 255) / 256;
  const dim3 cgrid(static_cast<unsigned>(hblocks) * static_cast<unsigned>(p.T));
  if (p.k <= 8)
    combine_kernel<8><<<cgrid, 256, 0, stream>>>(p, hblocks);
  else if (p.k <= 16)
    combine_kernel<16><<<cgrid, 256, 0, stream>>>(p, hblocks);
  else
    combine_kernel<kMaxTopK><<<cgrid, 256, 0, stream>>>(p, hblocks);
  return hipGetLastError();
}

}  // namespace amoe
