// Grouped expert GEMMs for larger blocks: gate/up with SwiGLU, and down into
// gate-scaled slot rows.
//
// A workgroup of 4 waves takes one item (expert, up to 192 of its dispatched
// rows, fp32: 64) and one run of output tiles, or half or a quarter of one (see
// grouped_kernel).  Each wave streams the weights of its own tiles straight into
// registers (4 fragments per K chunk: a gate/up tile pair, or four 16-column tiles
// of the down projection; 2 in smaller runs); the item's rows are staged in LDS,
// once for the four waves, and every fragment read from there meets those weight
// fragments.  The rows are fetched once per 128 rows of I (256 columns of H), by
// half and quarter runs once per 64 and 32 (128 and 64).
//
// What bounds it: the weight stream at 15 to 60 tokens per expert (8 trees x
// 64 nodes, H = 4096, I = 1536: gate/up streams 3.0 GB in 468 us = 6.4 TB/s,
// 0.9 of a plain read; replacing the products by an XOR or the row gathers by
// one row changed nothing), the weight stream and the work per stage together
// at 120 (32 x 60 nodes, H = 2048, I = 768: 200 us; with whole runs everywhere
// 215, of it 128 with weights from L2).  Against the passes before it (K split over
// the waves, rows gathered by every wave): gate/up 611 -> 468 and down 363 -> 270 us
// on the wide layer, 412 -> 200 and 289 -> 122 us at 32 x 60.  fp32: the matrix
// instructions.  No better, with whole runs at the same shapes: two tiles
// per wave at three workgroups per CU (482 / 240 us gate/up), four weight
// stages in flight (484 / 223), K split two ways (486 / 245) or four ways
// (533 / 376), two M groups for every item (615 / 248).
#include <type_traits>

#include "ffn_common.hpp"
#include "grouped_plan.hpp"

namespace amoe {

namespace {

constexpr int kGrpStage = 2;  // K chunks per LDS stage (128 bytes of each row)

enum class Grouped { GateUp, Down };

// M-tiles per wave: the accumulators of 8 M-tiles x 4 fragments are half of
// the registers two workgroups per CU leave a wave.  With two M groups each
// thread also holds twice the rows in flight: 6.  The fp32 path keeps a second
// accumulator set (below): 2 (3 x 4 fragments spill 64 registers).  One bf16
// kernel holds all M-tile counts at the 256 registers; the compiler spills 6 of
// them in gate/up and 2 in down.
template <class P>
constexpr int kGrpTileM = grouped_tile_m(P::kElemBytes);
template <class P>
constexpr int kGrpTileM2 = grouped_tile_m2(P::kElemBytes);
template <class P>
constexpr int kGrpMaxRows = grouped_item_rows(P::kElemBytes);

// Adds the products of `rows` rows of one item into acc and returns with the
// workgroup's LDS free.  w[f] / wbytes[f]: run of weight fragment f (a run of
// 0 bytes reads as zeros and costs no traffic); chunk c of it sits wstride
// 16-byte pieces after chunk c - 1.
//
// Stage i (kGrpStage chunks): the rows of stage i + 1, loaded one stage
// earlier, go to the other LDS buffer, then the loads of the rows of stage
// i + 2 and of the weights of stage i + 1 are issued, then stage i is
// multiplied.  The row loads are issued before the weights of the same
// round, so waiting for them leaves the weight stream in flight.
template <class P, int MT, int MG, int FR, int KS>
__device__ __forceinline__ void grouped_product(const uint4* const (&w)[FR], const int (&wbytes)[FR],
                                                int wstride, const uint4* const (&xrow)[(MG * MT + 1) / 2], int KC,
                                                int mt0, uint4* lds, floatx4 (&acc)[FR][MT]) {
  constexpr int kLoads = (MG * MT + 1) / 2;   // 16-byte row pieces per thread and stage
  constexpr int kChunk = 2 * kLoads * kWave;  // pieces of one chunk of the item's rows in LDS
  constexpr int kBuf = kGrpStage * kChunk;
  const int tid = threadIdx.x, lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  // thread tid loads piece tid % 8 of rows tid / 8 + 32 s; a row's pieces of
  // one stage fill two fragments.  Row r of a fragment's piece group sits at
  // r ^ 2 * piece, so the eight pieces of a row fall into different banks.
  const int piece = tid & 7;
  const int srow = tid >> 3;
  const int dst = (piece >> 2) * kChunk + (srow >> 4) * kWave + (piece & 3) * 16 + ((srow & 15) ^ (2 * piece));
  const int src0 = g * 16 + (r ^ (2 * g));
  const int src1 = g * 16 + (r ^ (2 * (g + 4)));
  constexpr int kMine = kGrpStage / KS;  // chunks of a stage that this wave multiplies
  const int part = KS == 1 ? 0 : (wave_id() & 1);
  const int nst = (KC + kGrpStage - 1) / kGrpStage;
  uint4 ra[kLoads];
  uint4 wb[2][kMine][FR];
  auto load_rows = [&](int st) {
    const int kc = min(min(st, nst - 1) * kGrpStage + (piece >> 2), KC - 1);  // in range; see store_rows
#pragma unroll
    for (int s = 0; s < kLoads; ++s) ra[s] = xrow[s][kc * 4 + (piece & 3)];
  };
  auto store_rows = [&](int st, int buf) {
    const bool in = st * kGrpStage + (piece >> 2) < KC;  // past the last chunk: zeros
#pragma unroll
    for (int s = 0; s < kLoads; ++s) lds[buf * kBuf + s * 2 * kWave + dst] = in ? ra[s] : make_uint4(0u, 0u, 0u, 0u);
  };
  auto load_w = [&](int st, uint4 (&v)[kMine][FR]) {
#pragma unroll
    for (int u = 0; u < kMine; ++u)
#pragma unroll
      for (int f = 0; f < FR; ++f)
        v[u][f] = load_weight<MG == 1 ? kPolicyStream : kPolicyPlain>(w[f], wbytes[f], (st * kGrpStage + part + u) * wstride + lane);
  };
  auto multiply = [&](int buf, const uint4 (&v)[kMine][FR], floatx4 (&a)[FR][MT]) {
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int src = (part + u) * kChunk + (part + u != 0 ? src1 : src0);
      uint4 x[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) x[mt] = lds[buf * kBuf + (mt0 + mt) * kWave + src];
#pragma unroll
      for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[f][mt] = P::mma(x[mt], v[u][f], a[f][mt]);
    }
  };
  load_rows(0);
  load_w(0, wb[0]);
  store_rows(0, 0);
  load_rows(1);
  __syncthreads();
  auto stage = [&](int i, auto cur, floatx4 (&a)[FR][MT]) {
    constexpr int c = decltype(cur)::value;
    store_rows(i + 1, c ^ 1);
    load_rows(i + 2);
    load_w(i + 1, wb[c ^ 1]);
    __builtin_amdgcn_sched_barrier(0);  // the loads above stay above the products
    multiply(c, wb[c], a);
    __syncthreads();
  };
  if constexpr (P::kElemBytes == 4) {
    // fp32 products: sums of 16 chunks, then the sums (shorter chains of
    // roundings than one running sum over K)
    constexpr int kFlush = 8 * KS;  // stages
    floatx4 part[FR][MT];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) part[f][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto flush = [&]() {
#pragma unroll
      for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            acc[f][mt][q] += part[f][mt][q];
            part[f][mt][q] = 0.f;
          }
    };
    for (int i = 0;;) {
      stage(i, std::integral_constant<int, 0>{}, part);
      if (++i == nst) break;
      stage(i, std::integral_constant<int, 1>{}, part);
      if (i % kFlush == kFlush - 1) flush();
      if (++i == nst) break;
    }
    flush();
  } else {
    for (int i = 0;;) {
      stage(i, std::integral_constant<int, 0>{}, acc);
      if (++i == nst) break;
      stage(i, std::integral_constant<int, 1>{}, acc);
      if (++i == nst) break;
    }
  }
}

template <class P>
struct GroupedRows {  // an item's slots and their gates
  int slot[kGrpMaxRows<P>];
  float gate[kGrpMaxRows<P>];
};

// 16-byte pieces of LDS: two stages of an item's rows (M-tiles rounded up to an
// even number, see grouped_product), or four waves' M-tiles of 4 x 16 floats and a
// padding piece per row on their way out, whichever is more.
template <class P>
constexpr int kGrpStaging = 2 * kGrpStage * 2 * ((2 * kGrpTileM2<P> + 1) / 2) * kWave;
constexpr int kGrpOut = 4 * 16 * 17;
template <class P>
constexpr int kGrpLds = kGrpStaging<P> > kGrpOut ? kGrpStaging<P> : kGrpOut;

// MT M-tiles per wave, FR weight fragments.  MG = 2: the item has 2 MT M-tiles
// and the four waves are two M groups over half as many output tiles.  MG = 2
// or FR = 2: `run` counts half runs.  KS = 2 (with FR = 2): two waves share a
// tile, each over every other K chunk, and `run` counts quarter runs.
template <class P, Grouped F, int MT, int MG, int FR, int KS = 1>
__device__ __forceinline__ void grouped_item(const ForwardParams& p, int e, int row0, int rows, int run, uint4* lds,
                                             GroupedRows<P>& gr) {
  constexpr int kLoads = (MG * MT + 1) / 2;
  constexpr int kTiles = F == Grouped::GateUp ? FR / 2 : FR;  // output tiles per wave
  int tid = threadIdx.x;
  // opaque per instantiation: the compiler otherwise hoists the address
  // arithmetic of every M-tile count above the branch between them and spills
  asm volatile("" : "+v"(tid), "+s"(row0), "+s"(rows));
  const int wave = wave_id(), lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  const int K = F == Grouped::GateUp ? p.H : p.I;
  const int KC = K / P::kKF;
  const int rowq = K * P::kElemBytes / 16;
  const int ntiles = (F == Grouped::GateUp ? p.I : p.H) / 16;
  const int mt0 = MG == 1 ? 0 : (wave & 1) * MT;  // this wave's first M-tile
  const int tile0 = (run * (4 / (MG * KS)) + wave / (MG * KS)) * kTiles;

  const uint4* w[FR];
  int wbytes[FR];
  int wstride;
  if (F == Grouped::GateUp) {
    const int npairs = (ntiles + 1) / 2, pair = tile0 / 2;
    const bool in = pair < npairs;
    const uint4* base = uniform_ptr(static_cast<const uint4*>(p.w_gate_up) +
                                    (static_cast<size_t>(e) * npairs + (in ? pair : 0)) * KC * 4 * kWave);
    wstride = 4 * kWave;
    // fragments gate 2p, gate 2p + 1, up 2p, up 2p + 1 of a chunk lie side by
    // side; one tile takes its gate and its up fragment
#pragma unroll
    for (int f = 0; f < FR; ++f) {
      const int pos = FR == 4 ? f : 2 * f + (tile0 & 1);
      w[f] = base + pos * kWave;
      wbytes[f] = in ? (KC * 4 - pos) * kWave * 16 : 0;
    }
  } else {
    wstride = kWave;
#pragma unroll
    for (int f = 0; f < FR; ++f) {
      const bool in = tile0 + f < ntiles;
      w[f] = uniform_ptr(static_cast<const uint4*>(p.w_down) +
                         (static_cast<size_t>(e) * ntiles + (in ? tile0 + f : 0)) * KC * kWave);
      wbytes[f] = in ? KC * kWave * 16 : 0;
    }
  }
  // rows past the item's last read its first row; their outputs are dropped
  const uint4* xrow[kLoads];
#pragma unroll
  for (int s = 0; s < kLoads; ++s) {
    const int m = (tid >> 3) + 32 * s;
    const int row = row0 + (m < rows ? m : 0);
    xrow[s] = F == Grouped::GateUp
                  ? static_cast<const uint4*>(p.hidden) + static_cast<size_t>(p.ent_slot[row] / p.k) * rowq
                  : static_cast<const uint4*>(p.act) + static_cast<size_t>(row) * rowq;
  }
  if (F == Grouped::Down && tid < rows) {
    const int slot = p.ent_slot[row0 + tid];
    gr.slot[tid] = slot;
    gr.gate[tid] = p.topk_gate[slot];
  }
  floatx4 acc[FR][MT];
#pragma unroll
  for (int f = 0; f < FR; ++f)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[f][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  grouped_product<P, MT, MG, FR, KS>(w, wbytes, wstride, xrow, KC, mt0, lds, acc);
  if constexpr (KS == 2) {
    static_assert(MG == 1 && 2 * FR * MT * kWave <= kGrpLds<P>, "the odd chunks' sums of two tile groups fit");
    floatx4* red = reinterpret_cast<floatx4*>(lds) + (wave / 2) * FR * MT * kWave + lane;
    if (wave & 1) {
#pragma unroll
      for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) red[(f * MT + mt) * kWave] = acc[f][mt];
    }
    __syncthreads();
    if (!(wave & 1)) {
#pragma unroll
      for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const floatx4 v = red[(f * MT + mt) * kWave];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[f][mt][q] += v[q];
        }
    }
    __syncthreads();
    if (wave & 1) return;  // no barrier follows
  }

  // Lane (r, g) holds rows 4g .. 4g + 3 of column r of each tile.  Each M-tile
  // goes through this wave's part of the LDS, so the rows leave in 16-byte
  // pieces, whole 256 bytes (down) or 64 / 128 bytes (gate/up) per row (down
  // at 32 x 60 nodes 173 -> 135 us against one 4-byte store per value).
  constexpr int kOutEb = F == Grouped::GateUp ? P::kElemBytes : 4;
  constexpr int kRowPieces = kTiles * kOutEb;           // 16-byte pieces per row
  constexpr int kRowStride = kRowPieces * 16 + 16;      // bytes, padded
  constexpr int kRowsPerStore = kWave / kRowPieces < 16 ? kWave / kRowPieces : 16;
  static_assert(16 * kRowStride * 4 <= kGrpLds<P> * 16, "one M-tile per wave fits");
  char* mine = reinterpret_cast<char*>(lds) + wave * 16 * kRowStride;
  const int nt = min(kTiles, ntiles - tile0);  // valid tiles of this wave (may be <= 0)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m0 = (mt0 + mt) * 16;
    if (m0 >= rows) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      char* row = mine + (4 * g + i) * kRowStride + r * kOutEb;
      if (F == Grouped::GateUp) {
#pragma unroll
        for (int j = 0; j < kTiles; ++j) {
          const float v = silu_mul(acc[j][mt][i], acc[kTiles + j][mt][i]);
          if (P::kElemBytes == 2)
            *reinterpret_cast<uint16_t*>(row + 16 * j * kOutEb) = float_to_bf16_bits(v);
          else
            *reinterpret_cast<float*>(row + 16 * j * kOutEb) = v;
        }
      } else {
        const float gate = gr.gate[min(m0 + 4 * g + i, rows - 1)];
#pragma unroll
        for (int f = 0; f < FR; ++f) *reinterpret_cast<float*>(row + 16 * f * kOutEb) = gate * acc[f][mt][i];
      }
    }
    wave_lds_sync();
    const int pc = lane % kRowPieces;
#pragma unroll
    for (int q = 0; q < 16 / kRowsPerStore; ++q) {
      const int lr = q * kRowsPerStore + lane / kRowPieces;
      const int m = m0 + lr;
      const uint4 v = *reinterpret_cast<const uint4*>(mine + min(lr, 15) * kRowStride + pc * 16);
      if (lane < kRowsPerStore * kRowPieces && m < rows && pc < nt * kOutEb) {
        if (F == Grouped::GateUp)
          reinterpret_cast<uint4*>(static_cast<char*>(p.act) +
                                   (static_cast<size_t>(row0 + m) * p.I + tile0 * 16) * kOutEb)[pc] = v;
        else
          reinterpret_cast<uint4*>(p.ys + static_cast<size_t>(gr.slot[m]) * p.H + tile0 * 16)[pc] = v;
      }
    }
    wave_lds_sync();
  }
}

// One output run (or half run) of an item of up to kGrpTileM M-tiles.
template <class P, Grouped F, int FR>
__device__ __forceinline__ void grouped_small(const ForwardParams& p, int e, int row0, int rows, int run, uint4* lds,
                                              GroupedRows<P>& gr) {
  const int mt = (rows + 15) / 16;
  if (mt == 1) grouped_item<P, F, 1, 1, FR>(p, e, row0, rows, run, lds, gr);
  else if (kGrpTileM<P> == 2 || mt == 2) grouped_item<P, F, 2, 1, FR>(p, e, row0, rows, run, lds, gr);
  else if constexpr (kGrpTileM<P> > 2) {
    if (mt == 3) grouped_item<P, F, 3, 1, FR>(p, e, row0, rows, run, lds, gr);
    else if (mt == 4) grouped_item<P, F, 4, 1, FR>(p, e, row0, rows, run, lds, gr);
    else if (mt <= 6) grouped_item<P, F, 6, 1, FR>(p, e, row0, rows, run, lds, gr);
    else grouped_item<P, F, 8, 1, FR>(p, e, row0, rows, run, lds, gr);
  }
}

// A quarter run of an fp32 item (see grouped_kernel).
template <class P, Grouped F>
__device__ __forceinline__ void grouped_quarter(const ForwardParams& p, int e, int row0, int rows, int run, uint4* lds,
                                                GroupedRows<P>& gr) {
  if (rows <= 16) grouped_item<P, F, 1, 1, 2, 2>(p, e, row0, rows, run, lds, gr);
  else if (rows <= 32) grouped_item<P, F, 2, 1, 2, 2>(p, e, row0, rows, run, lds, gr);
  else if (rows <= 48) grouped_item<P, F, 3, 1, 2, 2>(p, e, row0, rows, run, lds, gr);
  else grouped_item<P, F, 4, 1, 2, 2>(p, e, row0, rows, run, lds, gr);
}

// Items come in groups of the workgroups that share one item's rows, group
// after group round-robin over the XCDs (workgroup b runs on XCD b % 8), so
// the rows are read from one XCD's L2.  An item of more than kGrpTileM M-tiles
// runs two M groups over one weight stream, so its weights come from HBM once;
// those loads use the default cache policy (the second M group reads the same
// lines: 229 -> 215 us at 32 x 60 nodes), all others are non-temporal (478
// against 530 us on the wide layer).
//
// A workgroup covers one of an item's `nblocks` runs, or half a run for the big
// items, which come first, and for the last n_split items: shorter workgroups
// at the end even out the finish.  With whole runs everywhere, on average 365
// (4 x 60 nodes, H = 2048, I = 768) to 430 (8 x 64, H = 4096, I = 1536) of the
// 512 resident workgroups were at work.  Steps, us, whole / half runs: 4 x 60
// 210 / 199, 32 x 60 413 / 403, 7 x 60 with H = 256, I = 1664, top-4 89 / 75;
// 8 x 64 (H = 4096) even.
template <class P, Grouped F>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void grouped_kernel(ForwardParams p,
                                                                                              int nblocks,
                                                                                              int n_split) {
  __shared__ uint4 lds[kGrpLds<P>];
  __shared__ GroupedRows<P> gr;
  const int n_items = *p.n_items, n_big = *p.n_big;
  const GroupedShare sh = grouped_share(blockIdx.x, n_items, n_big, n_split, nblocks, P::kElemBytes);
  if (sh.item >= n_items) return;
  const int4 d = p.items[sh.item];
  const int run = __builtin_amdgcn_readfirstlane(sh.run);  // without this the gate/up kernel spills 65 registers, not 6
  const int e = __builtin_amdgcn_readfirstlane(d.x);
  const int row0 = __builtin_amdgcn_readfirstlane(d.y);
  const int rows = __builtin_amdgcn_readfirstlane(d.z);
  if constexpr (P::kElemBytes == 4) {
    if (sh.parts == 4) {
      grouped_quarter<P, F>(p, e, row0, rows, run, lds, gr);
      return;
    }
  }
  if (sh.item >= n_big) {
    if (sh.parts == 2) grouped_small<P, F, 2>(p, e, row0, rows, run, lds, gr);
    else grouped_small<P, F, 4>(p, e, row0, rows, run, lds, gr);
  } else if constexpr (kGrpTileM<P> > 2) {
    if (rows <= 160) grouped_item<P, F, 5, 2, 4>(p, e, row0, rows, run, lds, gr);
    else grouped_item<P, F, 6, 2, 4>(p, e, row0, rows, run, lds, gr);
  } else {
    // three M-tiles in a half run of narrower waves rather than four
    if (rows <= 48) grouped_item<P, F, 3, 1, 2>(p, e, row0, rows, run, lds, gr);
    else grouped_item<P, F, 2, 2, 4>(p, e, row0, rows, run, lds, gr);
  }
}

// Items sorted by rows as well measured 3 % faster at 4 x 60 nodes, but up to 2 %
// slower at 8 x 64 (H = 4096).
template <class P, Grouped F>
hipError_t launch_grouped_pass(const ForwardParams& p, int max_items, int nblocks, hipStream_t stream) {
  const long long grid = grouped_workgroups(p.T * p.k, max_items, nblocks, P::kElemBytes);
  // far beyond what the slot rows of one device's memory allow
  if (grid > 0x7fffffffll) return hipErrorInvalidValue;
  grouped_kernel<P, F><<<static_cast<unsigned>(grid), 256, 0, stream>>>(p, nblocks, grouped_split_items(nblocks));
  return hipGetLastError();
}

template <class P>
hipError_t launch_grouped_path(const ForwardParams& p, int max_items, hipStream_t stream) {
  const hipError_t err = launch_grouped_pass<P, Grouped::GateUp>(p, max_items, (p.I / 16 + 7) / 8, stream);
  return err != hipSuccess ? err : launch_grouped_pass<P, Grouped::Down>(p, max_items, (p.H / 16 + 15) / 16, stream);
}

}  // namespace

hipError_t launch_grouped(const ForwardParams& p, int max_items, hipStream_t stream) {
  return p.is_bf16 ? launch_grouped_path<Bf16Path>(p, max_items, stream)
                   : launch_grouped_path<F32Path>(p, max_items, stream);
}

}  // namespace amoe
