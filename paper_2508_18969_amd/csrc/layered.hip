// Layer-by-layer path of the chemistry update for networks whose weights do
// not fit the on-chip design of the fused kernel - e.g. the ODENet of the
// paper's runs, 20-2048-4096-2048-1024-512-17 (Sec. 4, network sizes table;
// 38.9 MFLOP and 19.4M parameters per cell): its 38.9 MB of BF16 weights
// exceed the 4 MB L2 of an XCD, so every 64-cell tile of the fused kernel
// would stream them from the Infinity Cache.  Here each layer is one large
// matrix product over a chunk of cells, with 256 x 256 output tiles whose
// operands are staged in LDS, so every weight byte fetched serves 256 cells.
//
//   first_kernel   steps 1-2 (power transform, Z-score) and the first layer
//   layer_kernel   a hidden layer, Zt = GELU(W At + b)
//   last_kernel    the output layer and steps 4-7 (FP64 update)
//
// each writing the next layer's B fragments.
//
// Batches of the fused networks too small to fill the chip with the fused
// kernel's tiles run through the same kernels, on its packed weights.
//
// The property networks of the supercritical flame (PRNet, Sec. 2 and the
// network sizes of Sec. 4: 3-1024-512-256-1 and 3-2048-1024-512-4) run on the
// same kernels with their own input and output maps (Z-score of the input
// fields; the output affine map in FP64).
//
// Activations live in HBM between layers as "B fragments": for k-step q and
// cell-block cb (16 cells) a 1 KiB block of 64 lanes x 16 bytes, lane
// (cell cl, group g) holding input features frag_feature(KS, q, g, j); blocks
// are ordered [q][cb], so the 16 cell-blocks of a tile are 16 consecutive
// KiB.  Weights use the fused kernel's packed layout ([row-block][k-step]).
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace chemdnn {

namespace {

constexpr int FB = 64 * 16;        // bytes of one fragment (64 lanes x 16 bytes)

// Waits until at most N vector-memory operations of this wave are in flight.
// Direct-to-LDS copies are not tracked by the compiler's own wait insertion;
// the memory clobber keeps LDS reads from moving above the wait.
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Waits until at most PER * min(k, MAXK) vector-memory operations are in
// flight (k >= 0 at run time; PER, MAXK compile-time).
template <int PER, int MAXK>
__device__ __forceinline__ void wait_vmem_upto(int k) {
  if constexpr (MAXK <= 0) {
    wait_vmem<0>();
  } else {
    if (k >= MAXK) wait_vmem<PER * MAXK>();
    else wait_vmem_upto<PER, MAXK - 1>(k);
  }
}
// Every wave of the workgroup has finished its LDS reads (one wave: its own).
template <int NW> __device__ __forceinline__ void stage_barrier() {
  if constexpr (NW > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Fragments are copied through buffer resources: one per-lane offset and a
// wave-uniform offset in an SGPR, no vector address arithmetic; reads past
// the matrix return zero.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t layer_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
// One wave copies the 1 KiB fragment at byte offset off to dst (LDS), lane
// l's 16 bytes to dst + 16 l, without passing through registers.
__device__ __forceinline__ void dma_frag(rsrc_t r, uint32_t off, uint8_t *dst, int lane) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16,
                                           lane * 16, (int)off, 0, 0);
}

// Calls f(U), f(U - 1), ..., f(1) with compile-time arguments.
template <int U, class F> __device__ __forceinline__ void layer_tail(F &&f) {
  if constexpr (U >= 1) {
    f(std::integral_constant<int, U>{});
    layer_tail<U - 1>(f);
  }
}

// Tiles: rows x cells per workgroup, waves in a WR x WC grid of WRB x WCB
// 16x16 blocks each, ST stages of KG k-steps.
template <int WRB_, int WR_, int WCB_, int WC_, int ST_, int KG_> struct Tile {
  static constexpr int WRB = WRB_, WR = WR_, WCB = WCB_, WC = WC_, ST = ST_, KG = KG_;
  static constexpr int TRB = WRB * WR, TCB = WCB * WC, NT = 64 * WR * WC;
  static constexpr int LDS = ST * KG * (TRB + TCB) * FB;
  static_assert(LDS <= 160 * 1024, "LDS budget");
};
using T256 = Tile<4, 4, 8, 2, 4, 1>;   // 256 x 256, eight waves of 64 x 128
using T128 = Tile<2, 4, 4, 2, 4, 1>;   // 128 x 128, eight waves of 32 x 64
using T128S = Tile<2, 4, 4, 1, 8, 1>;  // 128 x 64, four waves of 32 x 64
using T64 = Tile<2, 2, 2, 2, 4, 2>;    // 64 x 64, four waves of 32 x 32
using T32 = Tile<2, 1, 2, 2, 4, 2>;    // 32 x 64, two waves of 32 x 32
using T16 = Tile<2, 1, 1, 1, 8, 2>;    // 32 x 16, one wave

// GELU of the row-blocks rb .. of one k-step (accumulators y), written as the
// next layer's B fragment of cell-block cb: output row 16 rb + 4 g + r is
// input feature of k-step rb / RPQ, slot 4 (rb % RPQ) + r.  Row-blocks past R
// are zero.
template <class Op>
__device__ __forceinline__ void put_hidden(uint8_t *Y, int rb, int R, int NCB, int cb, int lane,
                                           const f4 (&acc)[Op::KS / 16]) {
  constexpr int RPQ = Op::KS / 16;
  __attribute__((aligned(16))) uint8_t buf[16];
#pragma unroll
  for (int k = 0; k < RPQ; ++k) {
    f4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      y[r] = gelu(acc[k][r]);
      // an FP32 value before it is rounded to 16 bits, whatever the
      // compiler could fuse (v_fma_mix rounds the last product once)
      asm("" : "+v"(y[r]));
    }
    Op::store4(buf + 4 * k * Op::EB, y);
  }
  i4 v = *(const i4 *)buf;
  if (RPQ == 2 && rb + 1 >= R) v[2] = v[3] = 0;
  *(i4 *)(Y + ((size_t)(rb / RPQ) * NCB + cb) * FB + lane * 16) = v;
}

}  // namespace

// ------------------------------------------------------------------ layer
// Workgroup tile: TRB = WRB*WR row-blocks x TCB = WCB*WC cell-blocks; NW = WR WC
// waves in a WR x WC grid, each computing WRB x WCB 16x16 output blocks.  Per
// stage (KG k-steps) the tile's weight and activation fragments are copied to
// LDS (wave w copies the fragments w + NW k of each k-step); each wave then
// reads its fragments from LDS into registers one stage ahead, between the
// products of the current stage.  ST stages: the copies of stage t + ST - 1
// are issued once every wave has read the fragments of stage t (and so is done
// with the LDS space of stage t - 1).
// Tiles may reach past the matrix: fragments past its last row- or cell-block
// are read from the last one, and cell-blocks past NCB are not written;
// row-blocks R .. RO - 1 (the rest of the next layer's last k-step) are
// written as zeros.
// DBG (hidden layers): the accumulators are also written to a.dbg_acc.
//
// Large chunks are bound by the matrix cores' power (a 256 x 256 tile's k-step
// takes 580 ns alone and 870 ns with every CU busy; 1,024 cycles of products
// against 768 of LDS reads); small ones by the k-step's chain of wait, barrier
// and LDS read, and by how many CUs have a tile.  The steady loop has no
// branches (constant waits, the copies' offsets in SGPRs), and its reads are
// placed between the products: 4096 -> 2048 over 32,768 cells in BF16 takes
// 450 us (1.22 PFLOP/s) against 518 with a branching loop whose products the
// compiler had moved behind the next stage's barrier.
template <class Op, class T, bool DBG = false>
__global__ __launch_bounds__(T::NT, 1) void layer_kernel(LayerArgs a) {
  constexpr int WRB = T::WRB, WR = T::WR, WCB = T::WCB, WC = T::WC, ST = T::ST, KG = T::KG;
  constexpr int NW = WR * WC;                         // waves
  static_assert(Op::FRAG == 16, "16-byte fragments");
  using frag_t = typename Op::frag_t;
  constexpr int TRB = T::TRB, TCB = T::TCB, NF = TRB + TCB;
  static_assert(TRB % NW == 0 && TCB % NW == 0, "every wave copies as many fragments");
  constexpr int PER = KG * NF / NW;                   // copies per wave per stage
  static_assert(PER * (ST - 2) < 64, "copies in flight fit the wait counter");
  constexpr int SB = KG * NF * FB;                    // bytes of a stage
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w % WR, wc = w / WR;
  const int nrt = (a.R + TRB - 1) / TRB;
  const int rt = blockIdx.x % nrt, ct = blockIdx.x / nrt;
  const int rb0 = rt * TRB, cb0 = ct * TCB;

  // this wave's copies: fragments f = w + NW k of the NF of a k-step, as byte
  // offsets at k-step 0 (weights advance by one fragment per k-step,
  // activations by NCB fragments)
  const rsrc_t Wr = layer_rsrc(a.W, (uint32_t)a.R * a.NQ * FB);
  const rsrc_t Xr = layer_rsrc(a.X, (uint32_t)a.NQ * a.NCB * FB);
  uint32_t wo[TRB / NW], xo[TCB / NW];
#pragma unroll
  for (int k = 0; k < TRB / NW; ++k) {
    const int rb = rb0 + w + NW * k;
    wo[k] = (uint32_t)((rb < a.R ? rb : a.R - 1) * a.NQ) * FB;
  }
#pragma unroll
  for (int k = 0; k < TCB / NW; ++k) {
    const int cb = cb0 + w + NW * k;
    xo[k] = (uint32_t)(cb < a.NCB ? cb : a.NCB - 1) * FB;
  }
  const int N = (a.NQ + KG - 1) / KG;                 // stages
  const uint32_t xstep = (uint32_t)a.NCB * FB;
  // the next stage to copy: its k-step and LDS offset
  int qi = 0, ws = 0;
  auto issue = [&]() {
#pragma unroll
    for (int u = 0; u < KG; ++u) {
      const uint32_t q = KG == 1 || qi + u < a.NQ ? qi + u : a.NQ - 1;
      uint8_t *dst = smem + ws + (u * NF + w) * FB;
#pragma unroll
      for (int k = 0; k < TRB / NW; ++k) dma_frag(Wr, wo[k] + q * FB, dst + NW * k * FB, lane);
#pragma unroll
      for (int k = 0; k < TCB / NW; ++k) dma_frag(Xr, xo[k] + q * xstep, dst + (TRB + NW * k) * FB, lane);
    }
    qi += KG;
    ws = ws + SB == ST * SB ? 0 : ws + SB;
  };
  // the fragments of the next stage: part i of NP
  constexpr int NP = KG * (WRB + WCB);
  struct Regs { frag_t a[KG][WRB], b[KG][WCB]; };
  Regs rg[2];
  int rs = 0;                                         // LDS offset of the next stage to read
  auto read = [&](Regs &d, const uint8_t *pa, const uint8_t *pb, int i) {
    const int u = i / (WRB + WCB), k = i % (WRB + WCB);
    if (k < WRB) d.a[u][k] = *(const frag_t *)(pa + (u * NF + k) * FB);
    else d.b[u][k - WRB] = *(const frag_t *)(pb + (u * NF + k - WRB) * FB);
  };

  // accumulators start at the bias (rows 16 rb + 4 g + r)
  f4 acc[WRB][WCB];
#pragma unroll
  for (int i = 0; i < WRB; ++i) {
    const int rb = rb0 + wr * WRB + i;
    const f4 b = *(const f4 *)(a.bias + 16 * (rb < a.R ? rb : a.R - 1) + 4 * g);
#pragma unroll
    for (int j = 0; j < WCB; ++j) acc[i][j] = b;
  }

  // one stage: with NEXT the fragments of the next stage are read between the
  // products (WAIT: copies that may stay in flight then), with ISSUE the copies
  // of stage + ST - 1 go out; `half`: the stage holds one k-step only
  auto stage = [&](auto NEXT, auto ISSUE, auto WAIT, const Regs &cur, Regs &nxt, bool half) {
    const uint8_t *pa = nullptr, *pb = nullptr;
    if constexpr (NEXT()) {
      wait_vmem<WAIT()>();
      stage_barrier<NW>();
      pa = smem + rs + wr * WRB * FB + lane * 16;
      pb = smem + rs + (TRB + wc * WCB) * FB + lane * 16;
      rs = rs + SB == ST * SB ? 0 : rs + SB;
    }
    if constexpr (ISSUE()) issue();
    constexpr int NM = WRB * WCB, M = KG * NM;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if constexpr (NEXT()) {
#pragma unroll
        for (int i = m * NP / M; i < (m + 1) * NP / M; ++i) read(nxt, pa, pb, i);
      }
      if (KG > 1 && m >= NM && half) continue;
      const int u = m / NM, i = m % NM / WCB, j = m % WCB;
      acc[i][j] = Op::mma(cur.a[u][i], cur.b[u][j], acc[i][j]);
    }
    // a read (or more) after each product, so that neither the matrix cores
    // nor the LDS wait for the other's whole batch; nothing of the next stage
    // moves up (its wait would come before these products)
    if constexpr (NEXT()) {
#pragma unroll
      for (int m = 0; m < M; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, (NP + M - 1) / M, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using std::integral_constant;
  constexpr std::true_type YES{};
  constexpr std::false_type NO{};

  // stages 0 .. ST - 2 in flight; stage 0 in registers
  for (int t = 0; t < ST - 1 && t < N; ++t) issue();
  {
    const int issued = N < ST - 1 ? N : ST - 1;
    wait_vmem_upto<PER, ST - 2>(issued - 1);
    stage_barrier<NW>();
    const uint8_t *pa = smem + wr * WRB * FB + lane * 16, *pb = smem + (TRB + wc * WCB) * FB + lane * 16;
#pragma unroll
    for (int i = 0; i < NP; ++i) read(rg[0], pa, pb, i);
    rs = SB;
  }
  integral_constant<int, PER * (ST - 3)> steady;
  int t = 0;
  // two stages per trip, so the register sets need no dynamic index
  for (; t + ST < N; t += 2) {
    stage(YES, YES, steady, rg[0], rg[1], false);
    stage(YES, YES, steady, rg[1], rg[0], false);
  }
  if (t + ST - 1 < N) {
    stage(YES, YES, steady, rg[0], rg[1], false);
    rg[0] = rg[1];
    ++t;
  }
  // the last rem <= ST - 1 stages: all their copies are out
  const int rem = N - t;
  if ((ST - 1 - rem) & 1) rg[1] = rg[0];
  const bool half = KG > 1 && (a.NQ % KG) != 0;
  layer_tail<ST - 1>([&](auto U) {
    constexpr int u = U();                            // stages left, this one included
    constexpr int s = (ST - 1 - u) & 1;
    if (rem >= u) {
      if constexpr (u > 1) stage(YES, NO, integral_constant<int, PER *(u - 2)>{}, rg[s], rg[s ^ 1], false);
      else stage(NO, NO, integral_constant<int, 0>{}, rg[s], rg[s ^ 1], half);
    }
  });

  if constexpr (DBG) {
#pragma unroll
    for (int i = 0; i < WRB; ++i)
#pragma unroll
      for (int j = 0; j < WCB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * (rb0 + wr * WRB + i) + 4 * g + r;
          const int cell = 16 * (cb0 + wc * WCB + j) + cl;
          if (row < a.dbg_rows && cell < a.dbg_n) a.dbg_acc[row * a.dbg_ld + cell] = acc[i][j][r];
        }
  }
  // GELU, then the next layer's B fragments: output row 16 rb + 4 g + r is
  // input feature of k-step rb / RPQ, slot 4 (rb % RPQ) + r
  constexpr int RPQ = Op::KS / 16;
  static_assert(WRB % RPQ == 0, "row-blocks of a k-step in one wave");
#pragma unroll
  for (int i = 0; i < WRB; i += RPQ) {
    const int rb = rb0 + wr * WRB + i;
    if (rb >= a.RO) continue;
#pragma unroll
    for (int j = 0; j < WCB; ++j) {
      const int cb = cb0 + wc * WCB + j;
      if (cb >= a.NCB) continue;
      f4 y[RPQ];
#pragma unroll
      for (int k = 0; k < RPQ; ++k) y[k] = acc[i + k][j];
      put_hidden<Op>(a.Y, rb, a.R, a.NCB, cb, lane, y);
    }
  }
}

// ------------------------------------------------------------------ first layer
// The first hidden layer with its input.  A workgroup's four waves compute the
// features of FWCB cell-blocks, two slots of every lane each, into the B
// fragments (lane: cell cl, group g holds the features frag_feature(KS, q, g,
// j)) in LDS - power transform and Z-score for the chemistry networks, Z-score
// in FP64 for the property networks (PROP), zero past the inputs and for cells
// past the chunk - then RPW row-blocks of the layer each.  Its 32 inputs are
// one or two k-steps, so there is nothing else to stage: bound by the GELUs
// and by the writes.  The workgroups of a cell group recompute its features,
// which replaces a launch and a pass over memory: 32,768 cells x 2048 rows in
// BF16 take 40 us (67 M GELUs take 25 us of issue, the 134 MB written 27), with
// a feature kernel before it and the layer on the tiled kernel 43 us.  With
// every wave computing all its features, 4,096 cells x 1600 rows took 11.3 us
// (now 9.0), 30,011 x 2048 of a property network 37.5 (33.5), 1,000 x 2048 7.1
// (6.4), 16 x 1600 4.3 (3.7).
//
// FUSED: the features are rounded as in the fused kernel (T, P and the species
// of their slots through FP32), for its networks' small batches.  The property
// networks' inputs are rounded once, FP64 to the operand format, on both paths
// (in the fused kernel the compiler folds the two conversions).
constexpr int FWCB = 2;
template <class Op, bool PROP, bool FUSED, bool DBG = false>
__global__ __launch_bounds__(256) void first_kernel(FirstArgs a) {
  using frag_t = typename Op::frag_t;
  constexpr int NQ = 32 / Op::KS, NE = 16 / Op::EB, RPQ = Op::KS / 16;
  __shared__ __align__(16) uint8_t feat[FWCB * NQ * FB];
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a workgroup: four row parts of one cell group
  const int parts = (a.RO + a.RPW - 1) / a.RPW, quads = (parts + 3) / 4;
  const int r0 = (blockIdx.x % quads * 4 + v) * a.RPW, cb0 = blockIdx.x / quads * FWCB;
  const int r1 = r0 + a.RPW < a.RO ? r0 + a.RPW : a.RO;
  const rsrc_t Wr = layer_rsrc(a.W, (uint32_t)a.R * NQ * FB);
  // slots 2 v and 2 v + 1 of every lane
  const int f0 = 16 * (v >> 1) + 4 * g + 2 * (v & 1);
#pragma unroll
  for (int c = 0; c < FWCB; ++c) {
    const int cell = 16 * (cb0 + c) + cl;
    const bool valid = cell < a.nc;
    const int64_t i = a.n0 + (valid ? cell : 0);
    double in[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = f0 + j;
      if constexpr (PROP) {
        in[j] = a.x[(int64_t)(f < a.D ? f : a.D - 1) * a.ld + i];
      } else {
        const int s = f - 2 < a.D - 2 ? f - 2 : a.D - 3;
        in[j] = *(f == 0 ? a.T + i : f == 1 ? a.P + i : a.x + (int64_t)s * a.ld + i);
      }
    }
    typedef decltype(Op::feature(0.0)) elem_t;
    __attribute__((aligned(8))) elem_t buf[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = f0 + j;
      const bool used = valid && f < a.D;
      elem_t z;
      if constexpr (PROP) {
        z = Op::feature((in[j] - a.dc[PConst::IN_MU + f]) * a.dc[PConst::IN_IS + f]);
      } else {
        const float u = ypow(in[j], a.fc[FConst::LAM]), za = a.fc[FConst::ZA + f], zc = a.fc[FConst::ZC + f];
        z = Op::feature(u, za, zc);
        if (v == 0) {
          const double tp = (in[j] - a.dc[j == 0 ? DConst::T_MU : DConst::P_MU]) *
                            a.dc[j == 0 ? DConst::T_IS : DConst::P_IS];
          if constexpr (FUSED) {
            float zf = __builtin_fmaf(u, za, zc);
            zf = g == 0 ? (float)tp : zf;
            asm("" : "+v"(zf));
            z = (elem_t)zf;
          } else {
            z = g == 0 ? Op::feature(tp) : z;
          }
        }
      }
      z = used ? z : (elem_t)0.0f;
      if constexpr (DBG)
        if (used && blockIdx.x % quads == 0) a.dbg_in[f * a.dbg_ld + cell] = (float)z;
      buf[j] = z;
    }
    uint8_t *const p = feat + (c * NQ + 2 * v / NE) * FB + lane * 16 + 2 * v % NE * Op::EB;
    if constexpr (Op::EB == 2) *(uint32_t *)p = *(const uint32_t *)buf;
    else *(uint64_t *)p = *(const uint64_t *)buf;
  }
  __syncthreads();
  if (r0 >= a.RO) return;
  frag_t x[FWCB][NQ];
#pragma unroll
  for (int c = 0; c < FWCB; ++c)
#pragma unroll
    for (int q = 0; q < NQ; ++q) x[c][q] = *(const frag_t *)(feat + (c * NQ + q) * FB + lane * 16);
  auto load = [&](frag_t (&wf)[RPQ][NQ], f4 (&b)[RPQ], int rb) {
#pragma unroll
    for (int k = 0; k < RPQ; ++k) {
      const int r = rb + k < a.R ? rb + k : a.R - 1;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        wf[k][q] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                  Wr, lane * 16, (r * NQ + q) * FB, 0));
      b[k] = *(const f4 *)(a.bias + 16 * r + 4 * g);
    }
  };
  frag_t wf[RPQ][NQ];
  f4 bias[RPQ];
  load(wf, bias, r0);
  for (int rb = r0; rb < r1; rb += RPQ) {
    f4 acc[RPQ][FWCB];
#pragma unroll
    for (int k = 0; k < RPQ; ++k)
#pragma unroll
      for (int c = 0; c < FWCB; ++c) {
        acc[k][c] = bias[k];
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[k][c] = Op::mma(wf[k][q], x[c][q], acc[k][c]);
      }
    load(wf, bias, rb + RPQ < r1 ? rb + RPQ : rb);
#pragma unroll
    for (int c = 0; c < FWCB; ++c) {
      const int cb = cb0 + c;
      if (cb >= a.NCB) continue;
      if constexpr (DBG)
#pragma unroll
        for (int k = 0; k < RPQ; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * (rb + k) + 4 * g + r, cell = 16 * cb + cl;
            if (row < a.dbg_rows && cell < a.nc) a.dbg_acc[row * a.dbg_ld + cell] = acc[k][c][r];
          }
      f4 y[RPQ];
#pragma unroll
      for (int k = 0; k < RPQ; ++k) y[k] = acc[k][c];
      put_hidden<Op>(a.Y, rb, a.R, a.NCB, cb, lane, y);
    }
  }
}

// ------------------------------------------------------------------ last layer
// The output layer (32 rows) and what follows it, a wave per cell-block: the
// accumulators of its lanes are the rows 16 h + 4 g + r of cell cl, which the
// chemistry networks' post-processing takes as it does in the fused kernel
// (post.inc; output rows shifted by two), the property networks' (PROP) as
// y = o sigma + mu in FP64.  Weights and activations go straight
// to registers, PF k-steps ahead (the weights of a workgroup's four waves
// come through its L1).  Bound by the state's and the activations' loads and
// by the FP64 post-processing, whose four lanes per cell run it in a quarter
// of the time of one: 1,000 cells of the 512-wide layer take 8 us, 32,768
// 15 us, against 27 and 35 us in a tiled layer and a thread per cell.
template <class Op, bool PROP, bool DBG = false>
__global__ __launch_bounds__(256) void last_kernel(LastArgs a) {
  using frag_t = typename Op::frag_t;
  constexpr int PF = 8;
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int cb = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (cb >= a.NCB) return;
  const int cell = 16 * cb + cl;
  const bool valid = cell < a.nc;
  const int64_t i = a.n0 + (valid ? cell : 0);
  double T = 0.0, P = 0.0, Yc[8];
  if constexpr (!PROP && !DBG) {
    T = a.T[i];
    P = a.P[i];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int s = 16 * (j >> 2) + 4 * g + (j & 3) - 2;
      Yc[j] = a.x[(int64_t)(s < 0 ? 0 : s < a.S ? s : a.S - 1) * a.ld + i];
    }
  }
  const rsrc_t Wr = layer_rsrc(a.W, (uint32_t)2 * a.NQ * FB);
  const rsrc_t Xr = layer_rsrc(a.X, (uint32_t)a.NQ * a.NCB * FB);
  frag_t wf[PF][2], xf[PF];
  auto load = [&](int u, int q) {
    const int qc = q < a.NQ ? q : a.NQ - 1;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      wf[u][h] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                Wr, lane * 16, (h * a.NQ + qc) * FB, 0));
    xf[u] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(
                                           Xr, lane * 16, (int)((uint32_t)(qc * a.NCB + cb) * FB), 0));
  };
  f4 o[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) o[h] = *(const f4 *)(a.bias + 16 * h + 4 * g);
#pragma unroll
  for (int u = 0; u < PF; ++u) load(u, u);
  int q = 0;
  for (; q + PF <= a.NQ; q += PF)
#pragma unroll
    for (int u = 0; u < PF; ++u) {
#pragma unroll
      for (int h = 0; h < 2; ++h) o[h] = Op::mma(wf[u][h], xf[u], o[h]);
      load(u, q + u + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (q + u < a.NQ) {
#pragma unroll
      for (int h = 0; h < 2; ++h) o[h] = Op::mma(wf[u][h], xf[u], o[h]);
    }
  if constexpr (DBG) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 16 * h + 4 * g + r - 2;
        if (valid && s >= 0 && s < a.S) a.dbg_acc[s * a.dbg_ld + cell] = o[h][r];
      }
  } else if constexpr (PROP) {
    if (!valid) return;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * h + 4 * g + r - a.shift;
        if (k >= 0 && k < a.S)
          a.Y_out[(int64_t)k * a.ld + i] =
              __builtin_fma((double)o[h][r], a.dc[PConst::OUT_SD + k], a.dc[PConst::OUT_MU + k]);
      }
  } else {
    constexpr int FRAG = Op::FRAG;
    const double *const dcl = a.dc;
    const float *const fcl = a.fc;
    const float lam = fcl[FConst::LAM], inv_lam = fcl[FConst::INV_LAM];
    // (row offsets: a uniform part and one product per lane)
#define POST_SLOTS 8
#define POST_R(h) 4
#define POST_ROW(h, r, g) (16 * (h) + 4 * (g) + (r))
#define POST_AT(h, r, g, s) ((int64_t)(16 * (h) + (r) - 2) * a.ld + ((int64_t)(4 * (g)) * a.ld + i))
#include "post.inc"
  }
}

// ------------------------------------------------------------------ debug
// Operand value of feature f < K of cell c < n in the B fragments X
// ([NQ][NCB] fragments of 64 lanes x 16 bytes), decoded to FP32: the
// inverse of frag_feature within a k-step, f = KS q + 16 (j / 4) + 4 g + j % 4.
template <class Op>
__global__ __launch_bounds__(256) void frag_decode_kernel(const uint8_t *X, int NCB, int K, int n,
                                                          float *out, int64_t ld) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)K * n) return;
  const int f = (int)(t / n), c = (int)(t % n);
  const int q = f / Op::KS, rr = f % Op::KS;
  const int j = 4 * (rr / 16) + rr % 4, g = (rr % 16) / 4;
  const uint8_t *p = X + ((size_t)(q * NCB + c / 16) * 64 + g * 16 + c % 16) * 16 + j * Op::EB;
  out[f * ld + c] = (float)*(const decltype(Op::feature(0.0)) *)p;
}

// ------------------------------------------------------------------ launchers
namespace {

template <class K>
hipError_t set_lds(K kern, int bytes) {
  return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <class Op, class T, bool DBG = false>
hipError_t launch_tile(const LayerArgs &a, hipStream_t s) {
  auto k = layer_kernel<Op, T, DBG>;
  const int grid = ((a.R + T::TRB - 1) / T::TRB) * ((a.NCB + T::TCB - 1) / T::TCB);
  hipLaunchKernelGGL(k, dim3(grid), dim3(T::NT), T::LDS, s, a);
  return hipGetLastError();
}

// The tile of a hidden layer.  A launch of G workgroups puts c = ceil(G / CUs)
// of them on the fullest CU; a k-step then takes about lat ns for c = 1 and
// c thr for more, where lat is the k-step of one workgroup per CU (waits,
// barrier and products) and thr its share of a CU with several (products, LDS
// and L2 reads).
// Measured on the layers of 19-2048-4096-2048-1024-512-17 at 16 to 32,768 cells
// (lat from 16 cells, thr from the largest sizes of each tile).  The small
// tiles fill the chip for small chunks, the large ones read each operand
// fewer times: at 1,000 cells the 4096 -> 2048 layer takes 77 us on 32
// workgroups of 256 x 256 and 26 us on 512 of 64 x 64; at 32,768 cells 450 us
// against 940 us.
struct TileCost { int trb, tcb, lat, thr; };
// 128 x 64 tiles (16 bits) are for the launches that they fill in one round:
// 4096 -> 2048 over 1,000 cells 23.5 us on 256 of them, 26.3 on 512 of 64 x 64.
constexpr TileCost kCost16[6] = {{T256::TRB, T256::TCB, 870, 870}, {T128::TRB, T128::TCB, 270, 270},
                                 {T64::TRB, T64::TCB, 96, 92}, {T32::TRB, T32::TCB, 94, 70},
                                 {T16::TRB, T16::TCB, 77, 50}, {T128S::TRB, T128S::TCB, 178, 215}};
constexpr TileCost kCost32[5] = {{T256::TRB, T256::TCB, 3540, 3540}, {T128::TRB, T128::TCB, 920, 910},
                                 {T64::TRB, T64::TCB, 280, 245}, {T32::TRB, T32::TCB, 275, 230},
                                 {T16::TRB, T16::TCB, 165, 110}};
template <int N>
int pick_tile(const TileCost (&cost)[N], const LayerArgs &a) {
  int best = 0;
  int64_t tb = INT64_MAX;
  for (int k = 0; k < N; ++k) {
    const int64_t G = (int64_t)((a.R + cost[k].trb - 1) / cost[k].trb) *
                      ((a.NCB + cost[k].tcb - 1) / cost[k].tcb);
    const int64_t c = (G + a.n_cu - 1) / a.n_cu;
    const int64_t u = c > 1 ? c * cost[k].thr : cost[k].lat;
    if (u < tb) tb = u, best = k;
  }
  return best;
}

template <class Op>
hipError_t launch_layer_op(const LayerArgs &a, hipStream_t s) {
  int k;
  if constexpr (Op::EB == 4) k = pick_tile(kCost32, a);
  else k = pick_tile(kCost16, a);
  switch (k) {
    case 0: return launch_tile<Op, T256>(a, s);
    case 1: return launch_tile<Op, T128>(a, s);
    case 2: return launch_tile<Op, T64>(a, s);
    case 3: return launch_tile<Op, T32>(a, s);
    case 4: return launch_tile<Op, T16>(a, s);
    default:
      if constexpr (Op::EB == 2) return launch_tile<Op, T128S>(a, s);
      return hipErrorInvalidValue;
  }
}

// the layer dump: the same tiles with the accumulators written out
template <class Op>
hipError_t launch_layer_dbg_op(const LayerArgs &a, hipStream_t s) {
  int k;
  if constexpr (Op::EB == 4) k = pick_tile(kCost32, a);
  else k = pick_tile(kCost16, a);
  switch (k) {
    case 0: return launch_tile<Op, T256, true>(a, s);
    case 1: return launch_tile<Op, T128, true>(a, s);
    case 2: return launch_tile<Op, T64, true>(a, s);
    case 3: return launch_tile<Op, T32, true>(a, s);
    case 4: return launch_tile<Op, T16, true>(a, s);
    default:
      if constexpr (Op::EB == 2) return launch_tile<Op, T128S, true>(a, s);
      return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_layer_dbg(int fmt, const LayerArgs &a, hipStream_t s) {
  switch (fmt) {
    case 0: return launch_layer_dbg_op<OpF32>(a, s);
    case 1: return launch_layer_dbg_op<OpBF16>(a, s);
    case 2: return launch_layer_dbg_op<OpF16>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_frag_decode(int fmt, const uint8_t *X, int NCB, int K, int n, float *out,
                              int64_t ld, hipStream_t s) {
  const int64_t total = (int64_t)K * n;
  if (total <= 0) return hipSuccess;
  const dim3 grid((unsigned)((total + 255) / 256));
  switch (fmt) {
    case 0: hipLaunchKernelGGL(frag_decode_kernel<OpF32>, grid, dim3(256), 0, s, X, NCB, K, n, out, ld); break;
    case 1: hipLaunchKernelGGL(frag_decode_kernel<OpBF16>, grid, dim3(256), 0, s, X, NCB, K, n, out, ld); break;
    case 2: hipLaunchKernelGGL(frag_decode_kernel<OpF16>, grid, dim3(256), 0, s, X, NCB, K, n, out, ld); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The layer kernels use more than the default 64 KiB of LDS.
template <class Op, class T, bool DBG = false> static hipError_t prepare_tile() {
  return set_lds(layer_kernel<Op, T, DBG>, T::LDS);
}
template <class Op> static hipError_t prepare_op() {
  hipError_t e = prepare_tile<Op, T256>();   // (the other tiles: at most 64 KiB)
  if (e == hipSuccess) e = prepare_tile<Op, T256, true>();
  if constexpr (Op::EB == 2) {
    if (e == hipSuccess) e = prepare_tile<Op, T128S>();
    if (e == hipSuccess) e = prepare_tile<Op, T128S, true>();
  }
  static_assert(T128::LDS <= 65536 && T64::LDS <= 65536 && T32::LDS <= 65536 && T16::LDS <= 65536, "LDS");
  return e;
}
hipError_t layered_prepare(int fmt) {
  return fmt == 0 ? prepare_op<OpF32>() : fmt == 1 ? prepare_op<OpBF16>() : prepare_op<OpF16>();
}

hipError_t launch_layer(int fmt, const LayerArgs &a, hipStream_t s) {
  switch (fmt) {
    case 0: return launch_layer_op<OpF32>(a, s);
    case 1: return launch_layer_op<OpBF16>(a, s);
    case 2: return launch_layer_op<OpF16>(a, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {

template <class Op> hipError_t launch_first_op(const FirstArgs &a0, bool prop, bool fused, bool dbg, hipStream_t s) {
  FirstArgs a = a0;
  // row-blocks per wave: few enough that about 16 waves per CU have work, at
  // most 32; the row parts in whole fours, a workgroup's waves
  const int64_t groups = (a.NCB + FWCB - 1) / FWCB;
  const int64_t rpw = groups * a.RO / (16 * (int64_t)a.n_cu), r = rpw < 4 ? 4 : rpw > 32 ? 32 : rpw;
  const int64_t quads = (a.RO + 2 * r) / (4 * r), q = quads < 1 ? 1 : quads;
  a.RPW = (int)((a.RO + 8 * q - 1) / (8 * q) * 2);
  const int64_t parts = (a.RO + a.RPW - 1) / a.RPW;
  const dim3 grid((unsigned)(groups * ((parts + 3) / 4)));
  auto k = prop ? first_kernel<Op, true, false>
           : fused ? (dbg ? first_kernel<Op, false, true, true> : first_kernel<Op, false, true>)
           : dbg ? first_kernel<Op, false, false, true> : first_kernel<Op, false, false>;
  hipLaunchKernelGGL(k, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}
template <class Op> hipError_t launch_last_op(const LastArgs &a, bool prop, bool dbg, hipStream_t s) {
  auto k = prop ? last_kernel<Op, true> : dbg ? last_kernel<Op, false, true> : last_kernel<Op, false>;
  hipLaunchKernelGGL(k, dim3((a.NCB + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_first(int fmt, const FirstArgs &a, bool prop, bool fused, bool dbg, hipStream_t s) {
  switch (fmt) {
    case 0: return launch_first_op<OpF32>(a, prop, fused, dbg, s);
    case 1: return launch_first_op<OpBF16>(a, prop, fused, dbg, s);
    case 2: return launch_first_op<OpF16>(a, prop, fused, dbg, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_last(int fmt, const LastArgs &a, bool prop, bool dbg, hipStream_t s) {
  switch (fmt) {
    case 0: return launch_last_op<OpF32>(a, prop, dbg, s);
    case 1: return launch_last_op<OpBF16>(a, prop, dbg, s);
    case 2: return launch_last_op<OpF16>(a, prop, dbg, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace chemdnn
