// Layer-by-layer path of the chemistry update for networks whose weights do
// not fit the on-chip design of the fused kernel - e.g. the ODENet of the
// paper's runs, 20-2048-4096-2048-1024-512-17 (Sec. 4, network sizes table;
// 38.9 MFLOP and 19.4M parameters per cell): its 38.9 MB of BF16 weights
// exceed the 4 MB L2 of an XCD, so every 64-cell tile of the fused kernel
// would stream them from the Infinity Cache.  Here each layer is one large
// matrix product over a chunk of cells, with 256 x 256 output tiles whose
// operands are staged in LDS, so every weight byte fetched serves 256 cells.
//
//   prep_kernel    steps 1-2 (power transform, Z-score) -> layer-1 B fragments
//   layer_kernel   one layer, Zt = W At (+ b, GELU for hidden layers); the
//                  output goes straight into the next layer's B fragments
//   post_kernel    steps 4-7 per cell (one thread per cell, FP64 update)
//
// The property networks of the supercritical flame (PRNet, Sec. 2 and the
// network sizes of Sec. 4: 3-1024-512-256-1 and 3-2048-1024-512-4) run on the
// same layer kernel between their own input and output maps
// (prop_prep_kernel: Z-score of the input fields; prop_post_kernel: the
// output affine map in FP64).
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
using T64 = Tile<2, 2, 2, 2, 4, 2>;    // 64 x 64, four waves of 32 x 32
using T32 = Tile<2, 1, 2, 2, 4, 2>;    // 32 x 64, two waves of 32 x 32
using T16 = Tile<2, 1, 1, 1, 8, 2>;    // 32 x 16, one wave

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
template <class Op, class T, bool ACT, bool DBG = false>
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
          if (row < a.dbg_rows && cell < a.dbg_n) a.dbg_acc[(size_t)row * a.dbg_n + cell] = acc[i][j][r];
        }
  }
  if constexpr (ACT) {
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
        __attribute__((aligned(16))) uint8_t buf[16];
#pragma unroll
        for (int k = 0; k < RPQ; ++k) {
          f4 y;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            y[r] = gelu(acc[i + k][j][r]);
            // an FP32 value before it is rounded to 16 bits, whatever the
            // compiler could fuse (v_fma_mix rounds the last product once)
            asm("" : "+v"(y[r]));
          }
          Op::store4(buf + 4 * k * Op::EB, y);
        }
        i4 v = *(const i4 *)buf;
        if (RPQ == 2 && rb + 1 >= a.R) v[2] = v[3] = 0;
        *(i4 *)(a.Y + ((size_t)(rb / RPQ) * a.NCB + cb) * FB + lane * 16) = v;
      }
    }
  } else {
    // output layer: FP32 [row][cell]
#pragma unroll
    for (int i = 0; i < WRB; ++i)
#pragma unroll
      for (int j = 0; j < WCB; ++j) {
        const int rb = rb0 + wr * WRB + i, cb = cb0 + wc * WCB + j;
        if (rb >= a.R || cb >= a.NCB) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          a.O[(size_t)(16 * rb + 4 * g + r) * a.ldo + 16 * cb + cl] = acc[i][j][r];
      }
  }
}

// ------------------------------------------------------------------ prep
// Writes the 32 features z of cell c of the chunk into the layer-1 B
// fragments X ([32 / KS][NCB] fragments).
template <class Op>
__device__ __forceinline__ void store_layer1(const float (&z)[32], uint8_t *X, int NCB, int c) {
  const int cb = c >> 4, cl = c & 15;
  constexpr int NE = 16 / Op::EB;                          // slots per lane
#pragma unroll
  for (int q = 0; q < 32 / Op::KS; ++q)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      __attribute__((aligned(16))) uint8_t buf[16];
#pragma unroll
      for (int j0 = 0; j0 < NE; j0 += 4) {
        f4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = z[frag_feature(Op::KS, q, g, j0 + r)];
        Op::store4(buf + j0 * Op::EB, y);
      }
      *(i4 *)(X + ((size_t)q * NCB + cb) * FB + (g * 16 + cl) * 16) = *(const i4 *)buf;
    }
}

// Thread per cell c of the chunk (cells past the chunk give zero features):
// z_f of steps 1-2 for f < 32, written into the layer-1 B fragments.
template <class Op>
__global__ __launch_bounds__(256) void prep_kernel(PrepArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= 16 * a.NCB) return;
  const int64_t i = a.n0 + c;
  const bool valid = c < a.nc;
  const int64_t ii = valid ? i : 0;
  const float lam = a.fc[FConst::LAM];
  float z[32];
#pragma unroll
  for (int f = 0; f < 32; ++f) {
    float v = 0.0f;
    if (valid) {
      if (f == 0) {
        v = (float)((a.T[ii] - a.dc[DConst::T_MU]) * a.dc[DConst::T_IS]);
      } else if (f == 1) {
        v = (float)((a.P[ii] - a.dc[DConst::P_MU]) * a.dc[DConst::P_IS]);
      } else if (f - 2 < a.S) {
        v = __builtin_fmaf(ypow(a.Y[(int64_t)(f - 2) * a.ld + ii], lam), a.fc[FConst::ZA + f],
                           a.fc[FConst::ZC + f]);
      }
    }
    z[f] = v;
  }
  store_layer1<Op>(z, a.X, a.NCB, c);
}

// Property network input: thread per cell c of the chunk, z_f = (x_f - mu_f) /
// sigma_f in FP64 for the n_in input fields (zero for f >= n_in and for cells
// past the chunk), rounded to FP32 and written into the layer-1 B fragments.
template <class Op>
__global__ __launch_bounds__(256) void prop_prep_kernel(PropPrepArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= 16 * a.NCB) return;
  const bool valid = c < a.nc;
  const int64_t i = valid ? a.n0 + c : 0;
  float z[32];
#pragma unroll
  for (int f = 0; f < 32; ++f)
    z[f] = (valid && f < a.D)
               ? (float)((a.x[(int64_t)f * a.ld + i] - a.pc[PConst::IN_MU + f]) * a.pc[PConst::IN_IS + f])
               : 0.0f;
  store_layer1<Op>(z, a.X, a.NCB, c);
}

// ------------------------------------------------------------------ post
// Thread per cell: steps 4-7 from the FP32 network output O[s][cell].  The
// species loops are unrolled to the 30-species maximum (guarded by S), so
// the updated fractions stay in registers between the passes.
__global__ __launch_bounds__(256) void post_kernel(PostArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= a.nc) return;
  const int64_t i = a.n0 + c;
  const float lam = a.fc[FConst::LAM], inv_lam = a.fc[FConst::INV_LAM];
  const double T = a.T[i], P = a.P[i], t_ref = a.dc[DConst::T_REF];
  bool bad = !__builtin_isfinite(T) || !__builtin_isfinite(P);
  constexpr int SMAX = 30;
  double y[SMAX], yh[SMAX];
  double ssum = 0.0, h0 = 0.0, ry = 0.0;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    y[s] = 0.0;
    yh[s] = 0.0;
    if (s >= a.S) continue;
    const int rho = s + 2;
    y[s] = a.Y[(int64_t)s * a.ld + i];
    bad |= !__builtin_isfinite(y[s]);
    const float o = a.O[(size_t)s * a.ldo + c];
    const float wv = __builtin_fmaf(o, a.fc[FConst::PA + rho], a.fc[FConst::PB + rho]);
    const double v = y[s] + inv_change(y[s], wv, lam, inv_lam);
    // a NaN network output or a non-finite result flags the cell (the inverse
    // transform takes a NaN base like a negative one; the clamp turns NaN into 0)
    bad |= __builtin_isnan(wv) || !__builtin_isfinite(v);
    yh[s] = v > 0.0 ? v : 0.0;
    ssum += yh[s];
    h0 += y[s] * (a.dc[DConst::HF + rho] + a.dc[DConst::CP + rho] * (T - t_ref));
    ry += y[s] * a.dc[DConst::WINV + rho];
  }
  const double rsum = 1.0 / ssum;
  double hn = 0.0, cn = 0.0;
  bool nonfin = false;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    if (s >= a.S) continue;
    const double yn = yh[s] * rsum;
    nonfin |= !__builtin_isfinite(yn);
    hn += yn * a.dc[DConst::HF + s + 2];
    cn += yn * a.dc[DConst::CP + s + 2];
  }
  const double Tn = a.thermo ? t_ref + (h0 - hn) / cn : T;
  const bool okc = !bad && !nonfin && ssum > 0.0 && __builtin_isfinite(ssum) && __builtin_isfinite(Tn);
  const double rho_dt = a.omega && okc ? P / (kRGas * T * ry) * a.inv_dt : 0.0;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    if (s >= a.S) continue;
    const double yn = okc ? yh[s] * rsum : y[s];
    a.Y_out[(int64_t)s * a.ld + i] = yn;
    if (a.omega) a.omega[(int64_t)s * a.ld + i] = okc ? rho_dt * (yn - y[s]) : 0.0;
  }
  if (a.T_out) a.T_out[i] = okc ? Tn : T;
  if (!okc && a.n_bad) atomicAdd(a.n_bad, 1u);
}

// Property network output: y_k = o_k sigma_k + mu_k in FP64, thread per
// (output k, cell c); FP32 network output O[k][ldo] of the chunk.
__global__ __launch_bounds__(256) void prop_post_kernel(PropPostArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x, k = blockIdx.y;
  if (c >= a.nc) return;
  const double o = a.O[(size_t)k * a.ldo + c];
  a.y[(int64_t)k * a.ld + a.n0 + c] = __builtin_fma(o, a.pc[PConst::OUT_SD + k], a.pc[PConst::OUT_MU + k]);
}

// ------------------------------------------------------------------ debug
// Operand value of feature f < K of cell c < n in the B fragments X
// ([NQ][NCB] fragments of 64 lanes x 16 bytes), decoded to FP32: the
// inverse of frag_feature within a k-step, f = KS q + 16 (j / 4) + 4 g + j % 4.
template <class Op>
__global__ __launch_bounds__(256) void frag_decode_kernel(const uint8_t *X, int NCB, int K, int n,
                                                          float *out) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)K * n) return;
  const int f = (int)(t / n), c = (int)(t % n);
  const int q = f / Op::KS, rr = f % Op::KS;
  const int j = 4 * (rr / 16) + rr % 4, g = (rr % 16) / 4;
  const uint8_t *p = X + ((size_t)(q * NCB + c / 16) * 64 + g * 16 + c % 16) * 16 + j * Op::EB;
  float v;
  if constexpr (__is_same(Op, OpF32)) v = *(const float *)p;
  else if constexpr (__is_same(Op, OpBF16)) v = (float)*(const __bf16 *)p;
  else v = (float)*(const _Float16 *)p;
  out[t] = v;
}

__global__ __launch_bounds__(256) void copy_rows_kernel(const float *src, int ld_src, int rows, int n,
                                                        float *dst) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)rows * n) return;
  dst[t] = src[(t / n) * (int64_t)ld_src + t % n];
}

// ------------------------------------------------------------------ launchers
namespace {

template <class K>
hipError_t set_lds(K kern, int bytes) {
  return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <class Op, class T, bool ACT, bool DBG = false>
hipError_t launch_tile(const LayerArgs &a, hipStream_t s) {
  auto k = layer_kernel<Op, T, ACT, DBG>;
  const int grid = ((a.R + T::TRB - 1) / T::TRB) * ((a.NCB + T::TCB - 1) / T::TCB);
  hipLaunchKernelGGL(k, dim3(grid), dim3(T::NT), T::LDS, s, a);
  return hipGetLastError();
}

// The tile of a hidden layer.  A launch of G workgroups puts c = ceil(G / CUs)
// of them on the fullest CU; a k-step then takes about max(lat, c thr) ns,
// where lat is a lone workgroup's k-step (waits, barrier and the products of
// one wave) and thr its share of a full CU (products, LDS and L2 reads).
// Measured on the layers of 19-2048-4096-2048-1024-512-17 at 16 to 32,768 cells
// (lat from 16 cells, thr from the largest sizes of each tile).  The small
// tiles fill the chip for small chunks, the large ones read each operand
// fewer times: at 1,000 cells the 4096 -> 2048 layer takes 77 us on 32
// workgroups of 256 x 256 and 26 us on 512 of 64 x 64; at 32,768 cells 450 us
// against 940 us.
struct TileCost { int trb, tcb, lat, thr; };
constexpr TileCost kCost16[5] = {{T256::TRB, T256::TCB, 580, 870}, {T128::TRB, T128::TCB, 210, 270},
                                 {T64::TRB, T64::TCB, 96, 92}, {T32::TRB, T32::TCB, 94, 70},
                                 {T16::TRB, T16::TCB, 77, 50}};
constexpr TileCost kCost32[5] = {{T256::TRB, T256::TCB, 3540, 3540}, {T128::TRB, T128::TCB, 920, 910},
                                 {T64::TRB, T64::TCB, 280, 245}, {T32::TRB, T32::TCB, 275, 230},
                                 {T16::TRB, T16::TCB, 165, 110}};
int pick_tile(const TileCost (&cost)[5], const LayerArgs &a) {
  int best = 0;
  int64_t tb = INT64_MAX;
  for (int k = 0; k < 5; ++k) {
    const int64_t G = (int64_t)((a.R + cost[k].trb - 1) / cost[k].trb) *
                      ((a.NCB + cost[k].tcb - 1) / cost[k].tcb);
    const int64_t c = (G + a.n_cu - 1) / a.n_cu, t = c * cost[k].thr;
    const int64_t u = t > cost[k].lat ? t : cost[k].lat;
    if (u < tb) tb = u, best = k;
  }
  return best;
}

template <class Op>
hipError_t launch_layer_op(const LayerArgs &a, bool hidden, hipStream_t s) {
  if (!hidden) return launch_tile<Op, T32, false>(a, s);
  switch (pick_tile(Op::EB == 4 ? kCost32 : kCost16, a)) {
    case 0: return launch_tile<Op, T256, true>(a, s);
    case 1: return launch_tile<Op, T128, true>(a, s);
    case 2: return launch_tile<Op, T64, true>(a, s);
    case 3: return launch_tile<Op, T32, true>(a, s);
    default: return launch_tile<Op, T16, true>(a, s);
  }
}

// the layer dump: the same tiles with the accumulators written out
template <class Op>
hipError_t launch_layer_dbg_op(const LayerArgs &a, hipStream_t s) {
  switch (pick_tile(Op::EB == 4 ? kCost32 : kCost16, a)) {
    case 0: return launch_tile<Op, T256, true, true>(a, s);
    case 1: return launch_tile<Op, T128, true, true>(a, s);
    case 2: return launch_tile<Op, T64, true, true>(a, s);
    case 3: return launch_tile<Op, T32, true, true>(a, s);
    default: return launch_tile<Op, T16, true, true>(a, s);
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
                              hipStream_t s) {
  const int64_t total = (int64_t)K * n;
  if (total <= 0) return hipSuccess;
  const dim3 grid((unsigned)((total + 255) / 256));
  switch (fmt) {
    case 0: hipLaunchKernelGGL(frag_decode_kernel<OpF32>, grid, dim3(256), 0, s, X, NCB, K, n, out); break;
    case 1: hipLaunchKernelGGL(frag_decode_kernel<OpBF16>, grid, dim3(256), 0, s, X, NCB, K, n, out); break;
    case 2: hipLaunchKernelGGL(frag_decode_kernel<OpF16>, grid, dim3(256), 0, s, X, NCB, K, n, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_copy_rows(const float *src, int ld_src, int rows, int n, float *dst, hipStream_t s) {
  const int64_t total = (int64_t)rows * n;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src,
                     ld_src, rows, n, dst);
  return hipGetLastError();
}

// The layer kernels use more than the default 64 KiB of LDS.
template <class Op, class T, bool ACT, bool DBG = false> static hipError_t prepare_tile() {
  return set_lds(layer_kernel<Op, T, ACT, DBG>, T::LDS);
}
template <class Op> static hipError_t prepare_op() {
  hipError_t e = prepare_tile<Op, T256, true>();   // (the other tiles: at most 64 KiB)
  if (e == hipSuccess) e = prepare_tile<Op, T256, true, true>();
  static_assert(T128::LDS <= 65536 && T64::LDS <= 65536 && T32::LDS <= 65536 && T16::LDS <= 65536, "LDS");
  return e;
}
hipError_t layered_prepare() {
  hipError_t e = prepare_op<OpF32>();
  if (e == hipSuccess) e = prepare_op<OpBF16>();
  if (e == hipSuccess) e = prepare_op<OpF16>();
  return e;
}

hipError_t launch_layer(int fmt, const LayerArgs &a, bool hidden, hipStream_t s) {
  switch (fmt) {
    case 0: return launch_layer_op<OpF32>(a, hidden, s);
    case 1: return launch_layer_op<OpBF16>(a, hidden, s);
    case 2: return launch_layer_op<OpF16>(a, hidden, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_prep(int fmt, const PrepArgs &a, hipStream_t s) {
  const int blocks = (16 * a.NCB + 255) / 256;
  switch (fmt) {
    case 0: hipLaunchKernelGGL(prep_kernel<OpF32>, dim3(blocks), dim3(256), 0, s, a); break;
    case 1: hipLaunchKernelGGL(prep_kernel<OpBF16>, dim3(blocks), dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL(prep_kernel<OpF16>, dim3(blocks), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prop_prep(int fmt, const PropPrepArgs &a, hipStream_t s) {
  const int blocks = (16 * a.NCB + 255) / 256;
  switch (fmt) {
    case 0: hipLaunchKernelGGL(prop_prep_kernel<OpF32>, dim3(blocks), dim3(256), 0, s, a); break;
    case 1: hipLaunchKernelGGL(prop_prep_kernel<OpBF16>, dim3(blocks), dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL(prop_prep_kernel<OpF16>, dim3(blocks), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prop_post(const PropPostArgs &a, hipStream_t s) {
  if (a.nc <= 0 || a.K <= 0) return hipSuccess;
  hipLaunchKernelGGL(prop_post_kernel, dim3((a.nc + 255) / 256, a.K), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_post(const PostArgs &a, hipStream_t s) {
  if (a.nc <= 0) return hipSuccess;
  hipLaunchKernelGGL(post_kernel, dim3((a.nc + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace chemdnn
