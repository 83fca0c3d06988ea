// The chemistry update of the small network, 19-400-200-100-17, with its
// weights resident in a workgroup.
//
// One workgroup of eight waves per CU, persistent over tiles of CB blocks of
// 16 cells, four phases per tile with a barrier after each:
//
//   layer 1   25 row-blocks: three per wave, the last one's cell-blocks on
//             the upper four waves
//   layer 2   13 row-blocks: one per wave, one more on each of the lower four
//             waves, the last one's cell-blocks on the upper four
//   layer 3   7 row-blocks: one per wave
//   layer 4 and post-processing on the lower waves, a cell-block each; input
//             transform of the next tile on the upper waves
//
// so every SIMD (waves w and w + 4) has as many products and GELUs as the
// others in layers 1 and 2, and the FP64 work of both ends runs side by side.
// The layer-2 and layer-3 weights of a wave stay in its registers (16-bit and
// FP8 operands: 132 / 80 of the 256; layer 3's are reloaded from L2 a phase
// ahead), those of layers 1 and 4 in LDS.  FP32 weights are too large for that:
// layers 1 and 3 stay in registers, layer 2 comes from L2 for each tile, PF
// k-steps ahead, layer 4 lies in LDS.
//
// The fused kernel (step_kernel.h) has these weights stream through four waves
// in chunks of layer 1, one barrier per chunk, and a tile of it takes the same
// time whatever its cells.  The products, their order and their roundings are
// the same here; the FP64 sums of the post-processing run in another order.
//
// A tile of 64 cells in BF16 takes 19.8 thousand cycles: 4.5 in layer 1, 6.8 in
// layer 2, 3.2 in layer 3 and 5.3 in the last phase, bound by the issue of
// GELUs (700 per cell, about 60 cycles per wave and value) and of the FP64
// ends; LDS reads (a fragment per 1 to 3 products) come next.  A tile of 16 has
// 9.8 thousand, half of them the post-processing's 1,000 instructions in one
// wave.  16 / 4,096 / 16,384 / 262,144 cells, fused and here, us: BF16 16.1 /
// 17.0 / 17.9 / 199 and 8.7 / 10.0 / 15.8 / 155; FP8 16.5 / 17 / 31 / 289 and
// 8.8 / 9.9 / 14.9 / 142; FP32 28.7 / 30.6 / 57 / 808 and 17.3 / 19.4 / 47 / 642
// (FP32 is bound by the matrix cores: 12.8 thousand cycles of layer 2 alone on
// the SIMD with four row-blocks); BF16 with the FP32 table 27.4 / 28.5 / 29.5 /
// 375 and 10.3 / 11.8 / 20.1 / 211.
#pragma once
#include "step_kernel.h"

namespace chemdnn {

// C: the fused kernel's configuration (packed layout) of the same network; GT:
// the hidden activation - 0 the tanh form, 1 the FP32 table, 2 the FP16 table.
template <class C_, int CB_, int GT_> struct Small {
  using C = C_;
  static constexpr int CB = CB_, NW = 8, MC = 16 * CB, GT = GT_;
  static constexpr int FRAG = C::FRAG, RPQ = C::RPQ, FB = 64 * FRAG;
  static constexpr bool STREAM = C::EB == 4;         // FP32: weights from L2
  // row-blocks with rows of the network, and k-steps that hold any
  static constexpr int RB1 = (C::H1 + 15) / 16, RB2 = (C::H2 + 15) / 16, RB3 = (C::H3 + 15) / 16;
  static constexpr int NQ1 = C::NQ1, K2 = (RB1 + RPQ - 1) / RPQ, K3 = (RB2 + RPQ - 1) / RPQ,
                       K4 = (RB3 + RPQ - 1) / RPQ;
  static_assert(RB1 == 25 && RB2 == 13 && RB3 == 7 && CB <= 4, "the split of the row-blocks");
  static_assert(K2 <= C::NQ2 && K3 <= C::NQ3 && K4 <= C::NQ4, "k-steps of the packed layout");
  static constexpr int NBIAS = 16 * (RB1 + RB2 + RB3 + 2);
  static constexpr int LDS_DC = roundup(NBIAS * 4, 16);
  static constexpr int LDS_FC = LDS_DC + DConst::N * 8;
  static constexpr int LDS_W4 = roundup(LDS_FC + FConst::N * 4, 256);
  static constexpr int LDS_W1 = LDS_W4 + 2 * K4 * FB;
  static constexpr int LDS_ST = LDS_W1 + (STREAM ? 0 : RB1 * NQ1 * FB);  // FP64 state of two tiles
  static constexpr int STL = 6;                      // doubles per lane (five slots)
  static constexpr int ST_BYTES = CB * 64 * STL * 8;
  static constexpr int LDS_A0 = LDS_ST + 2 * ST_BYTES;
  static constexpr int LDS_A1 = LDS_A0 + NQ1 * CB * FB;
  // layer 4's input takes the place of layer 2's (whose rows past the network
  // lie in its last k-step and stay zero)
  static constexpr int LDS_A3 = LDS_A1;
  static_assert(K4 < K2, "the zero rows of layer 2's input stay");
  static constexpr int LDS_A2 = LDS_A1 + K2 * CB * FB;
  static constexpr int LDS_TAB = LDS_A2 + K3 * CB * FB;
  static constexpr int LDS_BYTES = LDS_TAB + C::tab_bytes(GT);
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  // FP32: layer-2 k-steps in flight (one block of 4,096 cells: six 20.7 us, eight
  // 19.4, ten 19.7, twelve spill and take 21.7; two blocks are bound by products)
  static constexpr int PF = CB == 1 ? 8 : 6;
};

// DBG: layer dump, as in the fused kernel - input operand values as they were
// stored (decoded to FP32) and accumulators of every layer; no post-processing.
template <class S, bool DBG = false>
__global__ __launch_bounds__(S::NW * 64, 2) void small_step_kernel(StepArgs a) {
  using C = typename S::C;
  using Op = typename C::Op;
  using frag_t = typename C::frag_t;
  constexpr int CB = S::CB, FRAG = S::FRAG, RPQ = S::RPQ, EB = C::EB, FB = S::FB;
  constexpr int NQ1 = S::NQ1, K2 = S::K2, K3 = S::K3, K4 = S::K4, PF = S::PF;
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t *const A0 = smem + S::LDS_A0, *const A1 = smem + S::LDS_A1;
  uint8_t *const A2 = smem + S::LDS_A2, *const A3 = smem + S::LDS_A3;
  int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15, voff = lane * FRAG;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool low = w < 4;
  const int uc = w - 4;                              // upper waves: their cell-block
  const rsrc_t W1 = weight_rsrc(a.w[0], C::wbytes(0)), W2 = weight_rsrc(a.w[1], C::wbytes(1));
  const rsrc_t W3 = weight_rsrc(a.w[2], C::wbytes(2));

  // the lane's indices anew, from an opaque copy: addresses built on them are
  // recomputed per phase instead of being kept, or spilled, across the tiles
  auto renew = [&]() {
    lane = opaque_v(lane);
    g = lane >> 4;
    cl = lane & 15;
    voff = lane * FRAG;
  };

  // A cell's fields f (T, P, Y_(f-2)), up to 20, are spread over its four
  // lanes in five slots: slot j < 4 of lane group g is field 4 g + j, slot 4
  // field 16 + g.  (The fused kernels' eight slots, field 16 h + 4 g + r, would
  // leave nine of the last sixteen idle.)
  constexpr int SLOTS = 5;
  auto row_of = [](int h, int r, int gr) { return h == 0 ? 4 * gr + r : 16 + gr; };
  auto row_at = [&](int h, int r, int gr, int64_t c) {
    return h == 0 ? (int64_t)(r - 2) * a.ld + ((int64_t)(4 * gr) * a.ld + c) : (int64_t)(14 + gr) * a.ld + c;
  };
  // the state is loaded a tile ahead by the upper waves, from valid addresses
  // (cells past the batch read cell 0, fields past the network row 0)
  double xin[SLOTS];
  auto load_xin = [&](int64_t t) {
    const int64_t i = t * S::MC + 16 * uc + cl;
    const int64_t ii = (t < a.ntiles && i < a.n) ? i : 0;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      const double *p = a.Y + (row_of(j >> 2, j & 3, g) - 2 < a.S ? row_at(j >> 2, j & 3, g, ii) : ii);
      if (j < 2) p = g == 0 ? (j == 0 ? a.T : a.P) + ii : p;
      xin[j] = __builtin_nontemporal_load(p);
    }
  };
  const bool pre = !low && uc < CB;
  if (pre) load_xin(blockIdx.x);

  // weights of layers 2 and 3 (packed row-blocks of C::NQ2 / C::NQ3 k-steps)
  const int rb2b = low ? 8 + w : 12, rb3 = w < S::RB3 ? w : S::RB3 - 1;
  frag_t w2[2][S::STREAM ? PF : K2], w3[K3], w1[S::STREAM ? 4 : 1][NQ1];
  auto load_w2 = [&](int u, int q, bool second) {
    w2[0][u] = ldb_frag<frag_t>(W2, w * C::NQ2 + q, voff);
    if (second) w2[1][u] = ldb_frag<frag_t>(W2, rb2b * C::NQ2 + q, voff);
  };
  auto load_w3 = [&]() {
#pragma unroll
    for (int q = 0; q < K3; ++q) w3[q] = ldb_frag<frag_t>(W3, rb3 * C::NQ3 + q, voff);
  };
  auto load_w1 = [&]() {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < NQ1; ++q)
        w1[k][q] = ldb_frag<frag_t>(W1, (k < 3 ? 3 * w + k : 24) * NQ1 + q, voff);
  };

  // constants, biases, the small layers' weights; rows past the network zero
  const float lam = a.fc[FConst::LAM], inv_lam = a.fc[FConst::INV_LAM];
  float inv_sa0 = 1.0f, sout[4], sa[4];
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    sa[l] = Op::SCALED ? a.fc[FConst::ASCALE + l] : 1.0f;
    sout[l] = Op::SCALED ? a.fc[FConst::SOUT + l] : 1.0f;
  }
  if (Op::SCALED) inv_sa0 = a.fc[FConst::INV_SA];
  constexpr int NT = S::NW * 64;
  float *const B1 = (float *)smem, *const B2 = B1 + 16 * S::RB1, *const B3 = B2 + 16 * S::RB2;
  float *const B4 = B3 + 16 * S::RB3;
  double *const dcl = (double *)(smem + S::LDS_DC);
  float *const fcl = (float *)(smem + S::LDS_FC);
  if constexpr (S::STREAM) {
    load_w3();
    load_w1();
  } else {
#pragma unroll
    for (int q = 0; q < K2; ++q) load_w2(q, q, true);
    for (int i = threadIdx.x; i < S::RB1 * NQ1 * FB / 16; i += NT)
      ((i4 *)(smem + S::LDS_W1))[i] = ((const i4 *)a.w[0])[i];
  }
  // layer 4's second row-block has row 16 + k at row 4 k, the row of slot 4 of
  // lane group k
  for (int i = threadIdx.x; i < 2 * K4 * FB / 16; i += NT) {
    constexpr int RB = K4 * FB / 16, PL = FRAG / 16;   // (packed row-blocks of C::NQ4 k-steps)
    const int h = i / RB, l = i % RB / PL;
    const int src = h == 0 ? l : (l & ~15) | (l & 15) >> 2;
    const bool used = h == 0 || (l & 3) == 0;
    const i4 v = ((const i4 *)a.w[3])[h * (C::NQ4 * FB / 16) + src * PL + i % PL];
    ((i4 *)(smem + S::LDS_W4))[i] = used ? v : i4{0, 0, 0, 0};
  }
  for (int i = threadIdx.x; i < S::NBIAS; i += NT) {
    constexpr int E1 = 16 * S::RB1, E2 = E1 + 16 * S::RB2, E3 = E2 + 16 * S::RB3, E4 = E3 + 16;
    B1[i] = i < E1 ? a.b[0][i] : i < E2 ? a.b[1][i - E1] : i < E3 ? a.b[2][i - E2]
            : i < E4 ? a.b[3][i - E3] : (i & 3) == 0 ? a.b[3][16 + (i - E4) / 4] : 0.0f;
  }
  for (int i = threadIdx.x; i < DConst::N; i += NT) dcl[i] = a.dc[i];
  for (int i = threadIdx.x; i < FConst::N; i += NT) fcl[i] = a.fc[i];
  for (int i = threadIdx.x; i < NQ1 * CB * FB / 16; i += NT) ((i4 *)A0)[i] = i4{0, 0, 0, 0};
  for (int i = threadIdx.x; i < C::tab_bytes(S::GT) / 16; i += NT)
    ((i4 *)(smem + S::LDS_TAB))[i] = ((const i4 *)a.gtab)[i];
  if constexpr (RPQ > 1) {
    for (int i = threadIdx.x; i < CB * FB / 16; i += NT) {
      ((i4 *)(A1 + (K2 - 1) * CB * FB))[i] = i4{0, 0, 0, 0};
      ((i4 *)(A2 + (K3 - 1) * CB * FB))[i] = i4{0, 0, 0, 0};
    }
  }
  __syncthreads();

  // debug mode: value v of row `row` (0 .. rows - 1) of a cell into
  // buf[(row0 + row) * dbg_ld + cell]
  auto dbg_put = [&](float *buf, int row0, int row, int rows, int64_t cell, float v) {
    dump_store(buf, a.dbg_ld, row0 + row, cell, row >= 0 && row < rows && cell < a.n, v);
  };
  int64_t cell0 = 0;                                   // first cell of the tile

  // input transform of the tile whose fields are in xin: state to LDS for the
  // post-processing, features to A0 (rounded as in the fused kernel), where
  // fields 16 .. 19 are slots 4 .. 7 (FP32: slots of the second k-step) of
  // lane group 0; the other groups' stay zero
  auto preprocess = [&](int64_t t, int buf) {
    double *st = (double *)(smem + S::LDS_ST + buf * S::ST_BYTES) + (uc * 64 + lane) * S::STL;
#pragma unroll
    for (int j = 0; j < 4; j += 2) *(double2v *)(st + j) = double2v{xin[j], xin[j + 1]};
    st[4] = xin[4];
    const bool valid = t * S::MC + 16 * uc + cl < a.n;
    uint8_t *const own = A0 + uc * FB + voff;
    uint8_t *const tail = A0 + ((NQ1 - 1) * CB + uc) * FB + cl * FRAG + ((NQ1 == 1 ? 4 : 0) + g) * EB;
    f4 v = {0.f, 0.f, 0.f, 0.f};                       // slots 0 .. 3 (FP8, FP32)
    __attribute__((aligned(8))) uint8_t own4[8];         // (16-bit operands)
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      const int f = row_of(j >> 2, j & 3, g);
      const double x = xin[j];
      const bool used = valid && f - 2 < a.S;
      const float u = ypow(x, lam), za = fcl[FConst::ZA + f], zc = fcl[FConst::ZC + f];
      float z = __builtin_fmaf(u, za, zc);
      if (j < 2) {
        const float ztp = j == 0 ? (float)((x - dcl[DConst::T_MU]) * dcl[DConst::T_IS])
                                 : (float)((x - dcl[DConst::P_MU]) * dcl[DConst::P_IS]);
        z = g == 0 ? ztp : z;
      }
      if constexpr (EB == 2) {
        typedef decltype(Op::feature(0.0)) elem_t;
        elem_t e;
        if (j < 2) {
          asm("" : "+v"(z));
          e = (elem_t)z;
        } else {
          e = Op::feature(u, za, zc);
        }
        e = used ? e : (elem_t)0.0f;
        if (j < 4) ((elem_t *)own4)[j] = e;
        else *(elem_t *)tail = e;
      } else {
        z = used ? z : 0.0f;
        if constexpr (Op::SCALED) z *= inv_sa0;
        if (j < 4) {
          v[j] = z;
        } else if constexpr (Op::SCALED) {
          *tail = (uint8_t)Op::pack4(f4{z, 0.f, 0.f, 0.f});
        } else {
          *(float *)tail = z;
        }
      }
    }
    if constexpr (EB == 2) *(uint64_t *)own = *(const uint64_t *)own4;
    else Op::store4(own, v);
    if constexpr (DBG)
#pragma unroll
      for (int j = 0; j < SLOTS; ++j)
        dbg_put(a.dbg_in, a.dbg_in_row[0], row_of(j >> 2, j & 3, g), a.S + 2, t * S::MC + 16 * uc + cl,
                j < 4 ? stored_operand<Op>(own, j) : stored_operand<Op>(tail, 0));
  };

  using std::integral_constant;
  // z[u] += wf[u] x[u] of N blocks (FP32: four dependent products each, the
  // blocks' chains side by side)
  auto mma = [&](auto N, auto wf, auto x, auto z) {
    if constexpr (EB == 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < N(); ++u)
          z(u) = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f4, wf(u))[r],
                                                      __builtin_bit_cast(f4, x(u))[r], z(u), 0, 0, 0);
    } else {
#pragma unroll
      for (int u = 0; u < N(); ++u) z(u) = Op::mma(wf(u), x(u), z(u));
    }
  };
  // hidden activation of the first n blocks
  auto act = [&](auto &z, int n) {
    if constexpr (S::GT == 0) {
      gelu_stages(z, n);
    } else {
#pragma unroll
      for (int u = 0; u < (int)(sizeof(z) / sizeof(f4)); ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (u < n)
            z[u][r] = S::GT == 1 ? gelu_tab(z[u][r], (const f4 *)(smem + S::LDS_TAB))
                                 : gelu_tab16(z[u][r], (const h4v *)(smem + S::LDS_TAB));
    }
  };
  // a row-block's starting accumulators, scaled result, and store of layer l's
  // activations y as the next layer's input
  auto init = [&](const float *B, int rb) {
    return Op::SCALED ? f4{0.f, 0.f, 0.f, 0.f} : *(const f4 *)(B + 16 * rb + 4 * g);
  };
  auto put = [&](f4 y, int l, int rb, int cb, uint8_t *A) {
    if constexpr (!Op::SCALED)
#pragma unroll
      for (int r = 0; r < 4; ++r) asm("" : "+v"(y[r]));
    uint8_t *const p = A + ((unsigned)rb / RPQ * CB + cb) * FB + voff + 4 * ((unsigned)rb % RPQ) * EB;
    Op::store4s(p, y, sa[l + 1]);
    if constexpr (DBG)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        dbg_put(a.dbg_in, a.dbg_in_row[l + 1], 16 * rb + 4 * g + r, l == 0 ? C::H1 : l == 1 ? C::H2 : C::H3,
                cell0 + 16 * cb + cl, stored_operand<Op>(p, r));
  };
  // debug mode: layer l's accumulators z
  auto dump_acc = [&](f4 z, int l, int rb, int cb) {
    if constexpr (DBG)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // (the output layer's second row-block: row 16 + g in slot 0)
        const int row = l < 3 ? 16 * rb + 4 * g + r : rb == 0 || r == 0 ? row_of(rb, r, g) - 2 : -1;
        const int H = l == 0 ? C::H1 : l == 1 ? C::H2 : l == 2 ? C::H3 : a.S;
        dbg_put(a.dbg_acc, a.dbg_acc_row[l], row, H, cell0 + 16 * cb + cl, z[r]);
      }
  };
  auto scale = [&](f4 &y, int l, const float *B, int rb) {
    if constexpr (Op::SCALED) {
      const f4 b = *(const f4 *)(B + 16 * rb + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = __builtin_fmaf(y[r], sout[l], b[r]);
    }
  };

  int buf = 0;
  if (pre) {
    preprocess(blockIdx.x, 0);
    load_xin((int64_t)blockIdx.x + gridDim.x);
  }
  lds_barrier();

  for (int64_t tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x, buf ^= 1) {
    renew();
    if constexpr (DBG) cell0 = tile * S::MC;
    // ------------------------------------------------------------ layer 1
    if constexpr (S::STREAM) {
      if (low || pre) {
#pragma unroll
        for (int u = 0; u < PF; ++u) load_w2(u, u, true);
      } else {
#pragma unroll
        for (int u = 0; u < PF; ++u) load_w2(u, u, false);
      }
    }
    {
      frag_t xq[NQ1][CB];
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int q = 0; q < NQ1; ++q) xq[q][c] = lds_frag<frag_t>(A0, q * CB + c, lane);
      auto wfrag = [&](int k, int q) {
        if constexpr (S::STREAM) return w1[k][q];
        else return lds_frag<frag_t>(smem + S::LDS_W1, (k < 3 ? 3 * w + k : 24) * NQ1 + q, lane);
      };
      // G row-blocks at a time, and the upper waves' block of the last one with
      // the last group
      constexpr int G = CB == 4 ? 1 : 3;
      auto rows = [&](auto K0, auto EXTRA) {
        constexpr int k0 = K0(), N = G * CB + EXTRA();
        f4 z[N];
#pragma unroll
        for (int u = 0; u < N; ++u) z[u] = init(B1, u < G * CB ? 3 * w + k0 + u / CB : 24);
#pragma unroll
        for (int q = 0; q < NQ1; ++q) {
          frag_t wf[G + 1], xe;
#pragma unroll
          for (int k = 0; k < G; ++k) wf[k] = wfrag(k0 + k, q);
          if constexpr (EXTRA()) wf[G] = wfrag(3, q), xe = lds_frag<frag_t>(A0, q * CB + uc, lane);
          mma(integral_constant<int, N>{}, [&](int u) { return wf[u / CB]; },
              [&](int u) { return u < G * CB ? xq[q][u % CB] : xe; }, [&](int u) -> f4 & { return z[u]; });
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int rb = u < G * CB ? 3 * w + k0 + u / CB : 24;
          dump_acc(z[u], 0, rb, u < G * CB ? u % CB : uc);
          scale(z[u], 0, B1, rb);
        }
        act(z, N);
#pragma unroll
        for (int u = 0; u < N; ++u)
          if (u < G * CB) put(z[u], 0, 3 * w + k0 + u / CB, u % CB, A1);
          else put(z[u], 0, 24, uc, A1);
      };
      if constexpr (G == 1) {
        rows(integral_constant<int, 0>{}, integral_constant<int, 0>{});
        rows(integral_constant<int, 1>{}, integral_constant<int, 0>{});
      }
      if (pre) rows(integral_constant<int, 3 - G>{}, integral_constant<int, 1>{});
      else rows(integral_constant<int, 3 - G>{}, integral_constant<int, 0>{});
    }
    lds_barrier();
    // ------------------------------------------------------------ layer 2
    {
      if constexpr (!S::STREAM) load_w3();
      // blocks of the wave's second row-block: all (lower waves) or one
      f4 z0[CB], z1[CB];
#pragma unroll
      for (int c = 0; c < CB; ++c) z0[c] = init(B2, w), z1[c] = init(B2, rb2b);
      // (the three forms in loops of their own: branches within the k-steps
      // would keep each one's LDS reads behind the previous products)
      auto run = [&](auto KIND) {
        auto kstep = [&](int q, int u) {
          frag_t x[CB];
#pragma unroll
          for (int c = 0; c < CB; ++c) x[c] = lds_frag<frag_t>(A1, q * CB + c, lane);
          frag_t xe;
          if constexpr (KIND() == 1) xe = lds_frag<frag_t>(A1, q * CB + uc, lane);
          mma(integral_constant<int, KIND() == 2 ? 2 * CB : CB + KIND()>{},
              [&](int k) { return w2[k / CB][u]; },
              [&](int k) { return k < CB ? x[k] : KIND() == 2 ? x[k % CB] : xe; },
              [&](int k) -> f4 & { return k < CB ? z0[k] : z1[k - CB]; });
        };
        if constexpr (S::STREAM) {
          constexpr int NF = K2 / PF * PF;
          for (int q0 = 0; q0 < NF; q0 += PF)
#pragma unroll
            for (int u = 0; u < PF; ++u) {
              kstep(q0 + u, u);
              const int qn = q0 + u + PF;
              load_w2(u, qn < K2 ? qn : K2 - 1, KIND() > 0);
            }
#pragma unroll
          for (int u = 0; u < K2 - NF; ++u) kstep(NF + u, u);
        } else {
#pragma unroll
          for (int q = 0; q < K2; ++q) kstep(q, q);
        }
      };
      if (low) run(integral_constant<int, 2>{});
      else if (pre) run(integral_constant<int, 1>{});
      else run(integral_constant<int, 0>{});
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        dump_acc(z0[c], 1, w, c);
        if (low) dump_acc(z1[c], 1, rb2b, c);
        else if (pre && c == 0) dump_acc(z1[0], 1, rb2b, uc);
        scale(z0[c], 1, B2, w), scale(z1[c], 1, B2, rb2b);
      }
      act(z0, CB);
#pragma unroll
      for (int c = 0; c < CB; ++c) put(z0[c], 1, w, c, A2);
      if (low) {
        act(z1, CB);
#pragma unroll
        for (int c = 0; c < CB; ++c) put(z1[c], 1, rb2b, c, A2);
      } else if (pre) {
        act(z1, 1);
        put(z1[0], 1, rb2b, uc, A2);
      }
    }
    lds_barrier();
    // ------------------------------------------------------------ layer 3
    {
      f4 z[CB];
      if (w < S::RB3) {
#pragma unroll
        for (int c = 0; c < CB; ++c) z[c] = init(B3, w);
#pragma unroll
        for (int q = 0; q < K3; ++q) {
          frag_t x[CB];
#pragma unroll
          for (int c = 0; c < CB; ++c) x[c] = lds_frag<frag_t>(A2, q * CB + c, lane);
          mma(integral_constant<int, CB>{}, [&](int) { return w3[q]; }, [&](int c) { return x[c]; },
              [&](int c) -> f4 & { return z[c]; });
        }
#pragma unroll
        for (int c = 0; c < CB; ++c) dump_acc(z[c], 2, w, c), scale(z[c], 2, B3, w);
        act(z, CB);
#pragma unroll
        for (int c = 0; c < CB; ++c) put(z[c], 2, w, c, A3);
      } else if (RPQ > 1) {
#pragma unroll
        for (int c = 0; c < CB; ++c) put(f4{0.f, 0.f, 0.f, 0.f}, 2, w, c, A3);
      }
    }
    lds_barrier();
    // ------------------------------------------- layer 4, post-processing; next tile's input
    renew();
    if (w < CB) {
      f4 o[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) o[h] = init(B4, h);
#pragma unroll
      for (int q = 0; q < K4; ++q) {
        const frag_t x = lds_frag<frag_t>(A3, q * CB + w, lane);
        frag_t wf[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) wf[h] = lds_frag<frag_t>(smem + S::LDS_W4, h * K4 + q, lane);
        mma(integral_constant<int, 2>{}, [&](int h) { return wf[h]; }, [&](int) { return x; },
            [&](int h) -> f4 & { return o[h]; });
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) dump_acc(o[h], 3, h, w), scale(o[h], 3, B4, h);
      const int64_t i = tile * S::MC + 16 * w + cl;
      const bool valid = i < a.n;
      if constexpr (!DBG) {
      const double *st = (const double *)(smem + S::LDS_ST + buf * S::ST_BYTES) + w * 64 * S::STL;
      const double T = st[cl * S::STL], P = st[cl * S::STL + 1];
      double Yc[SLOTS];
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) Yc[j] = st[lane * S::STL + j];
#define POST_SLOTS SLOTS
#define POST_R(h) ((h) == 0 ? 4 : 1)
#define POST_ROW(h, r, g) row_of(h, r, g)
#define POST_AT(h, r, g, s) row_at(h, r, g, i)
#include "post.inc"
      }
    } else if (pre && tile + gridDim.x < a.ntiles) {
      preprocess(tile + gridDim.x, buf ^ 1);
      load_xin(tile + 2 * (int64_t)gridDim.x);
    }
    lds_barrier();
  }
}

template <class S, bool DBG> static hipError_t launch_small(const StepArgs &a0, int n_cu, hipStream_t s) {
  StepArgs a = a0;
  a.ntiles = (a.n + S::MC - 1) / S::MC;
  const int grid = (int)(a.ntiles < n_cu ? a.ntiles : n_cu);
  hipLaunchKernelGGL((small_step_kernel<S, DBG>), dim3(grid), dim3(S::NW * 64), S::LDS_BYTES, s, a);
  return hipGetLastError();
}

// The tile: a block of 16 cells while every CU has one at most, then two, then
// MAXCB (four; two in FP32, whose four blocks do not fit the LDS).  A tile of one
// / two / four blocks takes 4.0 / 5.8 / 8.9 us in BF16, 4.1 / 5.3 / 8.5 in FP8,
// 13.8 / 20.8 in FP32, so the fewest rounds are the fastest.
template <class C, int MAXCB, int GT, bool DBG = false>
static hipError_t small_step(const StepArgs &a, int n_cu, hipStream_t s) {
  const int64_t blocks = (a.n + 15) / 16;
  if (blocks <= n_cu) return launch_small<Small<C, 1, GT>, DBG>(a, n_cu, s);
  if (MAXCB == 2 || blocks <= 2 * n_cu) return launch_small<Small<C, 2, GT>, DBG>(a, n_cu, s);
  return launch_small<Small<C, MAXCB, GT>, DBG>(a, n_cu, s);
}

template <class S, bool DBG> static hipError_t small_lds() {
  return hipFuncSetAttribute((const void *)small_step_kernel<S, DBG>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             S::LDS_BYTES);
}
template <class C, int MAXCB, int GT, bool DBG = false> static hipError_t small_prepare() {
  hipError_t e = small_lds<Small<C, 1, GT>, DBG>();
  if (e == hipSuccess) e = small_lds<Small<C, 2, GT>, DBG>();
  if (e == hipSuccess && MAXCB > 2) e = small_lds<Small<C, MAXCB, GT>, DBG>();
  return e;
}
template <class C, bool WITH_CALIB, int MAXCB> static void fill_small_layout(NetLayout *L) {
  fill_layout<C, WITH_CALIB>(L);
  L->pick[0] = small_step<C, MAXCB, 0>;
  L->pick[1] = small_step<C, MAXCB, 1>;
  L->pick[2] = small_step<C, MAXCB, 2>;
  L->pick_prepare[0] = small_prepare<C, MAXCB, 0>;
  L->pick_prepare[1] = small_prepare<C, MAXCB, 1>;
  L->pick_prepare[2] = small_prepare<C, MAXCB, 2>;
  L->pick_dbg = small_step<C, MAXCB, 0, true>;
  L->pick_dbg_prepare = small_prepare<C, MAXCB, 0, true>;
  L->pick_species = 18;                              // its slots
}

}  // namespace chemdnn
