// Training of the small network (hidden widths 400, 200, 100) by tiles of
// samples: forward, loss gradient and the gradients of every pre-activation
// in one kernel per batch, then all weight gradients in one, then their
// reduction with the Adam update.
//
// FP32 products on the BF16 matrix cores: each operand is the sum of three
// BF16 numbers (v = hi + mid + lo, each the rounding of what the earlier ones
// leave: 24 bits and their signs), and a product is the sum of the six terms
// down to 2^-18 of it, lo hi, hi lo, mid mid, mid hi, hi mid, and hi hi.  The
// dropped terms are below 2^-26.  Six 16x16x32 products take 96 cycles where
// the FP32 instruction takes 256.  The five small terms have an FP32
// accumulator of their own, so that the sum of the large ones is rounded once
// per 32 terms: in one accumulator the instruction's roundings, a few
// thousandths of an ulp off centre, added up over a batch (bias gradients
// 2.7e-6 off at 40,000 samples, against 2.1e-7).  Against 64 bits the results
// are closer than with FP32 products: output 1.5e-7 of its norm against
// 3.8e-7, gradients 1.5e-7 to 2.6e-7 against 2.7e-7 to 3.7e-7 (batches of 300
// to 65,536).  The range ends sooner than FP32's: operands that round to BF16
// infinity (above 3.39e38, and infinities) give NaN, and below 1e-33 the low
// parts become subnormal and lose bits (first layer's sums of operands of 1e-30
// / 1e-33 / 1e-36 / 1e-39: 3.3e-8 / 3.9e-8 / 2.7e-5 / 2.6e-2 of their norm off).
//
// Kernels of one training step on a batch (or chunk):
//   split_pack_kernel  weights and transposed weights -> fragments (once)
//   tile_kernel        32 samples at a time: input features, forward, loss,
//                      dZ_3, dZ_2, dZ_1; writes the activations and the dZ
//   dw_split_kernel    dW_l = dZ_l a_(l-1)^T and db_l over fixed batch splits
//   finish_kernel      sums the splits in order, updates the parameters
// No floating-point atomics: results are bitwise reproducible.
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "train.h"

namespace chemdnn {

namespace {

typedef __bf16 b4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

constexpr int FB = 1024;            // one BF16 fragment: 64 lanes x 16 bytes
constexpr int TF = 3 * FB;          // its three parts
constexpr int NW = 8;               // waves of a workgroup
constexpr int MC = 32;              // samples of a scratch block

// The compiled shape: hidden widths, row-blocks of 16 and k-steps of 32.
constexpr int H1 = 400, H2 = 200, H3 = 100, HT = H1 + H2 + H3;
constexpr int R1 = (H1 + 15) / 16, R2 = (H2 + 15) / 16, R3 = (H3 + 15) / 16;
constexpr int Q1 = (H1 + 31) / 32, Q2 = (H2 + 31) / 32, Q3 = (H3 + 31) / 32;

// Fragment offsets (in triples) of the packed matrices: forward W_l
// [row-block][k-step], then the transposed ones for the gradients.
constexpr int P1 = 0, P2 = P1 + R1, P3 = P2 + R2 * Q1, P4 = P3 + R3 * Q2, T4 = P4 + 2 * Q3,
              T3 = T4 + R3, T2 = T3 + R2 * Q3, T1 = T2 + R1 * Q2, PEND = T1 + 2 * Q1;

// v = hi + mid + lo, each rounded to nearest even.
struct Split4 { b4 p[3]; };
__device__ __forceinline__ Split4 split4(f4 v) {
  Split4 s;
  // an FP32 value, whatever product it comes from (v - hi could be contracted
  // to a fused multiply-add with that product)
#pragma unroll
  for (int r = 0; r < 4; ++r) asm("" : "+v"(v[r]));
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int r = 0; r < 4; ++r) s.p[k][r] = (__bf16)v[r];
    if (k < 2)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] -= (float)s.p[k][r];
  }
  return s;
}

// c += a b of split operands (parts 0, 1, 2: hi, mid, lo), small terms first.
constexpr int kTermA[6] = {2, 0, 1, 1, 0, 0}, kTermB[6] = {0, 2, 1, 0, 1, 0};
__device__ __forceinline__ f4 mma(i4 a, i4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b),
                                                 c, 0, 0, 0);
}

// LDS traffic only (global loads stay in flight).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The scratch between the tiles and the weight gradients: per 32-sample tile a
// block of rows of 32 floats - the input, the activations of the three hidden
// layers, dZ_1, dZ_2, dZ_3 and dO - so that a tile's results are contiguous,
// as is every fragment of 16 rows that a weight gradient reads.  (Rows of the
// whole batch, a power of two apart, made both sides wait for memory: the
// weight gradients of 65,536 samples took 239 us instead of 177.)
__host__ __device__ constexpr int row_a(int D) { return D; }
__host__ __device__ constexpr int row_dz(int D) { return D + HT; }
__host__ __device__ constexpr int row_do(int D) { return D + 2 * HT; }
__host__ __device__ constexpr int rows(int D, int S) { return D + 2 * HT + S; }

// GELU and its derivative at z: y = z s, s = 1/(1 + e^(-2v)) as in gelu(), and
// GELU' = s + z s (1 - s) 2 v', v' = sqrt(2/pi) (1 + 3 * 0.044715 z^2).
__device__ __forceinline__ void gelu_both(float z, float &y, float &d) {
  const float z2 = z * z;
  const float s = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * __builtin_fmaf(z2, kG3, kG1)));
  const float dv = __builtin_fmaf(z2, (float)(6.0 * kSqrt2OverPi * kGeluCubic), (float)(2.0 * kSqrt2OverPi));
  y = z * s;
  d = __builtin_fmaf(y * (1.0f - s), dv, s);
}

}  // namespace

// ------------------------------------------------------------------ packing
struct PackMat { int64_t src; int M, K, sm, sk, Q, begin; };   // element (m, k) at src + m sm + k sk
struct PackArgs { const float *params; uint8_t *dst; PackMat m[8]; };

// Thread per (triple, lane): eight values of one row, split and stored in the
// slots of their k-step; zero past the matrix.
__global__ __launch_bounds__(256) void split_pack_kernel(PackArgs a) {
  const int t = blockIdx.x * 256 + threadIdx.x, f = t >> 6, lane = t & 63;
  if (f >= PEND) return;
  int k = 7;
  while (f < a.m[k].begin) --k;
  const PackMat m = a.m[k];
  const int rb = (f - m.begin) / m.Q, q = (f - m.begin) % m.Q;
  const int row = 16 * rb + (lane & 15);
  uint8_t *const d = a.dst + (size_t)f * TF + lane * 16;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = frag_feature(32, q, lane >> 4, 4 * h + r);
      v[r] = row < m.M && c < m.K ? a.params[m.src + (int64_t)row * m.sm + (int64_t)c * m.sk] : 0.0f;
    }
    const Split4 s = split4(v);
#pragma unroll
    for (int p = 0; p < 3; ++p) *(b4 *)(d + p * FB + h * 8) = s.p[p];
  }
}

// ------------------------------------------------------------------ tiles
// What a tile starts and ends with.
enum {
  TILE_TRAIN = 0,      // FP64 state -> features -> forward -> loss gradient -> backward
  TILE_FWD = 1,        // x -> forward; out, and the pre-activations if wanted
  TILE_BWD_SAVED = 2,  // saved pre-activations, grad_out -> backward
  TILE_BWD = 3         // x -> forward again, grad_out -> backward
};

struct TileArgs {
  const double *T, *P, *Y;       // TRAIN: state, [D - 2][ld] mass fractions
  const float *x;                // other modes: input [D][ld]
  const float *go;               // TRAIN: target; BWD: grad_out; [S][ld]
  const float *z;                // BWD_SAVED: pre-activations [HT][ld]
  int64_t ld;                    // leading dimension of all of the above, out, zs and gx
  float *out, *zs, *gx;          // FWD: output, pre-activations or NULL; BWD: input gradient
  const float *params;
  const uint8_t *pack;
  float *blk;                    // scratch: per tile rows(D, S) rows of 32 samples
  float *lpart;                  // TRAIN: sum of squares per tile
  float inv;                     // TRAIN: 2 / (batch x species)
  int64_t B;
  int D, S;
  const float *fc;
  const double *dc;
};

// Weight fragments of NI row-blocks over Q k-steps, two k-steps in flight.
template <int NI, int Q> struct WStream {
  static constexpr int PF = Q < 2 ? Q : 2;
  i4 w[PF][NI][3];
  int off[NI];
  __device__ __forceinline__ void load(rsrc_t r, int voff, int u, int q) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        w[u][i][p] = __builtin_bit_cast(i4, __builtin_amdgcn_raw_buffer_load_b128(
                                                r, voff, off[i] + q * TF + p * FB, 0));
  }
  // the first k-steps of the row-blocks rb0, rb0 + 8 of the matrix at triple P
  __device__ __forceinline__ void start(rsrc_t r, int voff, int P, int rb0) {
#pragma unroll
    for (int i = 0; i < NI; ++i) off[i] = (P + (rb0 + NW * i) * Q) * TF;
#pragma unroll
    for (int u = 0; u < PF; ++u) load(r, voff, u, u);
  }
  // acc[i][c] += W B for the cell-blocks c0 .. c0 + NC - 1; B: triples [q][CB] in LDS
  template <int CB, int NC>
  __device__ __forceinline__ void run(rsrc_t r, int voff, const uint8_t *B, int c0, int lane,
                                      f4 (&acc)[NI][NC]) {
    i4 b[2][NC][3];
    f4 lo[NI][NC];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) lo[i][c] = f4{0.f, 0.f, 0.f, 0.f};
    const uint8_t *Bl = B + c0 * TF + lane * 16;
    auto read = [&](int u, const uint8_t *p) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < 3; ++k) b[u][c][k] = *(const i4 *)(p + c * TF + k * FB);
    };
    // k-step q from register sets u; the next one's operands are read and
    // the weights of q + 2 loaded behind its products
    auto step = [&](int u, int q, bool next) {
      if (next) read(u ^ 1, Bl + CB * TF);
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            f4 &d = t < 5 ? lo[i][c] : acc[i][c];
            d = mma(w[u][i][kTermA[t]], b[u][c][kTermB[t]], d);
          }
      if (next) load(r, voff, u, q + 2 < Q ? q + 2 : Q - 1);
      Bl += CB * TF;
      __builtin_amdgcn_sched_barrier(0);
    };
    read(0, Bl);
    if constexpr (Q > 1) {
#pragma nounroll
      for (int q = 0; q + 2 < Q; q += 2) {
        step(0, q, true);
        step(1, q + 1, true);
      }
      if constexpr (Q % 2 == 0) step(0, Q - 2, true);
    }
    step((Q - 1) & 1, Q - 1, false);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[i][c] += lo[i][c];
  }
};

// One workgroup of eight waves (two per SIMD) per 32-sample tile, grid-stride
// over the tiles.  Wave w owns the row-blocks w, w + 8, ... of every layer, in
// the forward and in the backward pass, so GELU'(z) of its rows waits in
// registers.  Operands sit in LDS as split fragments, written by the lanes
// that computed them; weights stream from L2 into registers.  A tile's eight
// products are a chain of barriers in which all waves multiply at the same
// time and then all evaluate: of its 60k cycles, 23k are products, 16k the
// GELUs, splits and stores, the rest waits and the uneven share of the last
// row-block (65,536 samples: 248 us in a trace of single steps, 113 TFLOP/s of
// FP32 products, 285 under a continuous load's lower clock; the layer-by-layer
// FP32 kernels took 570 us for the same part of the step).
//   LDS: A  a_1; then dO, dZ_3 (and dZ_1 for the input gradient)
//        B  a_2; then dZ_2
//        C  a_3
//        X  the input of the tile, then of the next one
// Tiles of ts samples: those of whole scratch blocks (samples past the batch
// have zero gradients).
__host__ __device__ constexpr int64_t tiles_of(int64_t n, int ts) { return (n + MC - 1) / MC * (MC / ts); }

template <int CB> struct TileLds {
  static constexpr int A = 0, B = A + Q1 * CB * TF, C = B + Q2 * CB * TF, BIAS = C + Q3 * CB * TF;
  static constexpr int NBIAS = 16 * (R1 + R2 + R3 + 2);
  static constexpr int RED = BIAS + NBIAS * 4, X = RED + 64, BYTES = X + CB * TF;
  static constexpr int DO = A, D3 = DO + CB * TF, D2 = B;
  static_assert(D3 + Q3 * CB * TF <= B && X % 16 == 0 && BYTES <= 160 * 1024, "LDS budget");
};

template <int MODE, bool GX, int CB>
__global__ __launch_bounds__(NW * 64, 1) void tile_kernel(TileArgs a) {
  using L = TileLds<CB>;
  constexpr int TS = 16 * CB;         // samples of a tile
  constexpr bool FWD = MODE != TILE_BWD_SAVED, BWD = MODE != TILE_FWD;
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t *const A = smem + L::A, *const Bq = smem + L::B, *const Cq = smem + L::C;
  float *const bias = (float *)(smem + L::BIAS), *const red = (float *)(smem + L::RED);
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15, voff = lane * 16;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void *)a.pack, (short)0, PEND * TF, 0x00020000);
  const int64_t ntiles = tiles_of(a.B, TS);

  if constexpr (FWD) {
    const int64_t o1 = (int64_t)a.D * H1, o2 = o1 + H1 + (int64_t)H1 * H2, o3 = o2 + H2 + H2 * H3,
                  o4 = o3 + H3 + (int64_t)H3 * a.S;
    for (int i = threadIdx.x; i < L::NBIAS; i += NW * 64) {
      const int k = i < 16 * R1 ? i : i < 16 * (R1 + R2) ? i - 16 * R1
                  : i < 16 * (R1 + R2 + R3) ? i - 16 * (R1 + R2) : i - 16 * (R1 + R2 + R3);
      const int n = i < 16 * R1 ? H1 : i < 16 * (R1 + R2) ? H2 : i < 16 * (R1 + R2 + R3) ? H3 : a.S;
      const int64_t o = i < 16 * R1 ? o1 : i < 16 * (R1 + R2) ? o2 : i < 16 * (R1 + R2 + R3) ? o3 : o4;
      bias[i] = k < n ? a.params[o + k] : 0.0f;
    }
  }

  // split values of row-block rb, cell-block c, as operand of the next product;
  // the second half of the last k-step is zero where the row-blocks end in it
  auto put = [&](uint8_t *base, int rb, int R, int c, f4 v) {
    uint8_t *const p = base + ((rb >> 1) * CB + c) * TF + lane * 16 + (rb & 1) * 8;
    const Split4 s = split4(v);
#pragma unroll
    for (int k = 0; k < 3; ++k) *(b4 *)(p + k * FB) = s.p[k];
    if (rb == R - 1 && !(rb & 1))
#pragma unroll
      for (int k = 0; k < 3; ++k) *(u2 *)(p + k * FB + 8) = u2{0u, 0u};
  };
  // rows of row-block rb (of H rows, the first at row r0) from column col on, in
  // the tile's scratch block: a resource at the block's first element, one
  // per-lane offset
  float *blk = a.blk;
  auto block_of = [&](int64_t t) { return a.blk + t * TS / MC * rows(a.D, a.S) * MC + t * TS % MC; };
  auto store = [&](int r0, int rb, int H, int col, f4 v) {
    const rsrc_t o = __builtin_amdgcn_make_buffer_rsrc(blk + (r0 + 16 * rb) * MC + col, (short)0, -1, 0x00020000);
    const int vo = (4 * g * MC + cl) * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * rb + 15 < H || 16 * rb + 4 * g + r < H)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)v[r]), o, vo, r * MC * 4, 0);
  };
  // the same rows of one of the caller's arrays (leading dimension a.ld): 64-bit
  // addresses, since sixteen rows pass 4 GiB from ld = 71.6 million on
  auto store_to = [&](float *dst, int r0, int rb, int H, int64_t col, bool ok, f4 v) {
    float *const p = dst + (int64_t)(r0 + 16 * rb + 4 * g) * a.ld + (col + cl);
    if (!ok) return;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * rb + 15 < H || 16 * rb + 4 * g + r < H) p[r * a.ld] = v[r];
  };

  // Wave w owns the row-blocks v = w, w + 8, ...  The input of a tile is made
  // by the last four waves, cell-block XC and features 16 XH .. 16 XH + 15
  // each, while the others do the output layer of the tile before it.
  const int v = w, XC = CB > 1 ? w & 1 : 0, XH = (w >> 1) & 1;
  const bool XW = w >= NW / 2 && (w & 1) < CB;
  typedef std::conditional_t<MODE == TILE_TRAIN, double, float> in_t;
  in_t xin[4];
  auto load_x = [&](int64_t t) {
    const int64_t i0 = t * TS + 16 * XC + cl, i = i0 < a.B ? i0 : 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int f = 16 * XH + 4 * g + r, fc = f < a.D ? f : a.D - 1;
      if constexpr (MODE == TILE_TRAIN)
        xin[r] = *(fc == 0 ? a.T + i : fc == 1 ? a.P + i : a.Y + (int64_t)(fc - 2) * a.ld + i);
      else
        xin[r] = a.x[(int64_t)fc * a.ld + i];
    }
  };
  // the features of tile t: operand of layer 1, and (for its weight gradient)
  // into the tile's scratch block
  auto make_x = [&](int64_t t) {
    const bool valid = t * TS + 16 * XC + cl < a.B;
    f4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int f = 16 * XH + 4 * g + r;
      float z;
      if constexpr (MODE == TILE_TRAIN) {
        // the arithmetic of the inference kernel's preprocessing
        z = __builtin_fmaf(ypow(xin[r], a.fc[FConst::LAM]), a.fc[FConst::ZA + f], a.fc[FConst::ZC + f]);
        if (r < 2) {
          const float tp = (float)((xin[r] - a.dc[r == 0 ? DConst::T_MU : DConst::P_MU]) *
                                   a.dc[r == 0 ? DConst::T_IS : DConst::P_IS]);
          z = g == 0 && XH == 0 ? tp : z;
        }
      } else {
        z = xin[r];
      }
      y[r] = valid && f < a.D ? z : 0.0f;
    }
    if constexpr (FWD) put(smem + L::X, XH, 2, XC, y);
    if constexpr (BWD) {
      blk = block_of(t);
      store(0, XH, a.D, 16 * XC, y);
    }
  };
  if (XW && FWD) {
    load_x(blockIdx.x);
    make_x(blockIdx.x);
  }
  __syncthreads();

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t s0 = tile * TS;
    if constexpr (BWD) blk = block_of(tile);
    // a hidden layer's epilogue: activation, its derivative (kept), operand, stores
    auto hidden = [&](f4 z, int r0, int rb, int H, int R, int c, uint8_t *dst, f4 &d) {
      const int64_t cell = s0 + 16 * c + cl;
      f4 y;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float yy, dd;
        gelu_both(z[r], yy, dd);
        y[r] = yy;
        d[r] = dd;
      }
      if constexpr (FWD) put(dst, rb, R, c, y);
      if constexpr (MODE == TILE_FWD) {
        if (a.zs) store_to(a.zs, r0, rb, H, s0 + 16 * c, cell < a.B, z);
      } else {
        store(row_a(a.D) + r0, rb, H, 16 * c, y);
      }
    };
    f4 g1[4][CB], g2[2][CB], g3[CB];
    // the output layer's waves: row-block w & 1, cell-block w >> 1
    const int orb = w & 1, ocb = CB > 1 ? (w >> 1) & 1 : 0;
    const bool OW = w < 2 * CB;
    const int64_t ocell = s0 + 16 * ocb + cl;
    f4 tgt = {0.f, 0.f, 0.f, 0.f};
    auto load_target = [&]() {
      if constexpr (BWD)
        if (OW)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * orb + 4 * g + r;
            tgt[r] = row < a.S && ocell < a.B ? a.go[(int64_t)row * a.ld + ocell] : 0.0f;
          }
    };

    if constexpr (FWD) {
      WStream<2, 1> w1;
      w1.start(wr, voff, P1, v);
      // ---------------------------------------------------------- layer 1
#pragma unroll
      for (int ps = 0; ps < 2; ++ps) {
        const int rb0 = v + 2 * NW * ps;
        f4 acc[2][CB];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int rb = rb0 + NW * i;
          const f4 b = *(const f4 *)(bias + 16 * (rb < R1 ? rb : 0) + 4 * g);
#pragma unroll
          for (int c = 0; c < CB; ++c) acc[i][c] = b;
        }
        w1.template run<CB, CB>(wr, voff, smem + L::X, 0, lane, acc);
        if (ps == 0) w1.start(wr, voff, P1, v + 2 * NW);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int rb = rb0 + NW * i;
          if (rb < R1)
#pragma unroll
            for (int c = 0; c < CB; ++c) hidden(acc[i][c], 0, rb, H1, R1, c, A, g1[2 * ps + i][c]);
        }
      }
      // ---------------------------------------------------------- layer 2
      auto layer2 = [&](auto NI) {
        constexpr int N = NI();
        WStream<N, Q1> s;
        s.start(wr, voff, P2, v);
        lds_barrier();
        f4 acc[N][CB];
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const f4 b = *(const f4 *)(bias + 16 * (R1 + v + NW * i) + 4 * g);
#pragma unroll
          for (int c = 0; c < CB; ++c) acc[i][c] = b;
        }
        s.template run<CB, CB>(wr, voff, A, 0, lane, acc);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int c = 0; c < CB; ++c) hidden(acc[i][c], H1, v + NW * i, H2, R2, c, Bq, g2[i][c]);
      };
      if (v + NW < R2) layer2(std::integral_constant<int, 2>{});
      else layer2(std::integral_constant<int, 1>{});
      // ---------------------------------------------------------- layer 3
      WStream<1, Q2> w3;
      w3.start(wr, voff, P3, v < R3 ? v : 0);
      load_target();
      if (XW) load_x(tile + gridDim.x < ntiles ? tile + gridDim.x : tile);
      lds_barrier();
      if (v < R3) {
        f4 acc[1][CB];
        const f4 b = *(const f4 *)(bias + 16 * (R1 + R2 + v) + 4 * g);
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[0][c] = b;
        w3.template run<CB, CB>(wr, voff, Bq, 0, lane, acc);
#pragma unroll
        for (int c = 0; c < CB; ++c) hidden(acc[0][c], H1 + H2, v, H3, R3, c, Cq, g3[c]);
      }
    } else {
      // ---------------------------------------------------------- saved z
      load_target();
      // (64-bit addresses, as in store_to; rows and samples past the batch read
      // the last row, the first sample)
      auto load_z = [&](int r0, int rb, int H, int c) {
        const bool ok = s0 + 16 * c + cl < a.B;
        const float *const p = a.z + (ok ? s0 + 16 * c + cl : 0);
        const int go = opaque_v(g);
        f4 z;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * rb + 4 * go + r;
          z[r] = p[(int64_t)(r0 + (16 * rb + 15 < H || row < H ? row : H - 1)) * a.ld];
          if (!ok || !(16 * rb + 15 < H || row < H)) z[r] = 0.0f;
        }
        __builtin_amdgcn_sched_barrier(0);
        return z;
      };
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c)
          if (v + NW * i < R1) g1[i][c] = load_z(0, v + NW * i, H1, c);
#pragma unroll
      for (int c = 0; c < CB; ++c) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (v + NW * i < R2) g2[i][c] = load_z(H1, v + NW * i, H2, c);
        if (v < R3) g3[c] = load_z(H1 + H2, v, H3, c);
      }
#pragma unroll
      for (int c = 0; c < CB; ++c) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (v + NW * i < R1) hidden(g1[i][c], 0, v + NW * i, H1, R1, c, nullptr, g1[i][c]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (v + NW * i < R2) hidden(g2[i][c], H1, v + NW * i, H2, R2, c, nullptr, g2[i][c]);
        if (v < R3) hidden(g3[c], H1 + H2, v, H3, R3, c, nullptr, g3[c]);
      }
      if (XW) {
        load_x(tile);
        make_x(tile);
      }
    }

    // ------------------------------------------------------------ output layer
    WStream<1, Q3> w4;
    if constexpr (FWD) {
      if (OW) w4.start(wr, voff, P4, orb);
      lds_barrier();
    }
    if (OW) {
      f4 o[1][1];
      if constexpr (FWD) {
        o[0][0] = *(const f4 *)(bias + 16 * (R1 + R2 + R3 + orb) + 4 * g);
        w4.template run<CB, 1>(wr, voff, Cq, ocb, lane, o);
      }
      if constexpr (MODE == TILE_FWD) {
        store_to(a.out, 0, orb, a.S, s0 + 16 * ocb, ocell < a.B, o[0][0]);
      } else {
        f4 d = tgt;
        if constexpr (MODE == TILE_TRAIN) {
          float s = 0.0f;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bool ok = 16 * orb + 4 * g + r < a.S && ocell < a.B;
            const float e = ok ? o[0][0][r] - tgt[r] : 0.0f;
            s = __builtin_fmaf(e, e, s);
            d[r] = e * a.inv;
          }
#pragma unroll
          for (int k = 32; k >= 1; k >>= 1) s += __shfl_xor(s, k);
          if (lane == 0) red[w] = s;
        }
        put(smem + L::DO, orb, 2, ocb, d);
        store(row_do(a.D), orb, a.S, 16 * ocb, d);
      }
    }
    if constexpr (FWD)
      if (XW && tile + gridDim.x < ntiles) {
        make_x(tile + gridDim.x);
        if constexpr (BWD) blk = block_of(tile);
      }
    if constexpr (!BWD) {
      lds_barrier();
      continue;
    }
    // ------------------------------------------------------------ dZ_3
    WStream<1, 1> t4;
    t4.start(wr, voff, T4, v < R3 ? v : 0);
    lds_barrier();
    if constexpr (MODE == TILE_TRAIN)
      if (threadIdx.x == 0) a.lpart[tile] = CB > 1 ? ((red[0] + red[1]) + red[2]) + red[3] : red[0] + red[1];
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    if (v < R3) {
      f4 acc[1][CB];
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[0][c] = zero;
      t4.template run<CB, CB>(wr, voff, smem + L::DO, 0, lane, acc);
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const f4 d = acc[0][c] * g3[c];
        put(smem + L::D3, v, R3, c, d);
        store(row_dz(a.D) + H1 + H2, v, H3, 16 * c, d);
      }
    }
    // ------------------------------------------------------------ dZ_2
    auto dz2 = [&](auto NI) {
      constexpr int N = NI();
      WStream<N, Q3> s;
      s.start(wr, voff, T3, v);
      lds_barrier();
      f4 acc[N][CB];
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[i][c] = zero;
      s.template run<CB, CB>(wr, voff, smem + L::D3, 0, lane, acc);
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const f4 d = acc[i][c] * g2[i][c];
          put(smem + L::D2, v + NW * i, R2, c, d);
          store(row_dz(a.D) + H1, v + NW * i, H2, 16 * c, d);
        }
    };
    if (v + NW < R2) dz2(std::integral_constant<int, 2>{});
    else dz2(std::integral_constant<int, 1>{});
    // ------------------------------------------------------------ dZ_1
    auto dz1 = [&](auto NI, int ps, auto &s) {
      constexpr int N = NI();
      f4 acc[N][CB];
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[i][c] = zero;
      s.template run<CB, CB>(wr, voff, smem + L::D2, 0, lane, acc);
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const f4 d = acc[i][c] * (ps == 0 ? g1[i][c] : g1[2 + i][c]);
          store(row_dz(a.D), v + NW * (2 * ps + i), H1, 16 * c, d);
          // (the input gradient's operand, in the place of the derivative)
          if constexpr (GX) (ps == 0 ? g1[i][c] : g1[2 + i][c]) = d;
        }
    };
    {
      WStream<2, Q2> s;
      s.start(wr, voff, T2, v);
      lds_barrier();
      dz1(std::integral_constant<int, 2>{}, 0, s);
    }
    if (v + 3 * NW < R1) {
      WStream<2, Q2> s;
      s.start(wr, voff, T2, v + 2 * NW);
      dz1(std::integral_constant<int, 2>{}, 1, s);
    } else if (v + 2 * NW < R1) {
      WStream<1, Q2> s;
      s.start(wr, voff, T2, v + 2 * NW);
      dz1(std::integral_constant<int, 1>{}, 1, s);
    }
    // ------------------------------------------------------------ input gradient
    if constexpr (GX) {
      lds_barrier();
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (v + NW * i < R1)
#pragma unroll
          for (int c = 0; c < CB; ++c) put(A, v + NW * i, R1, c, g1[i][c]);
      lds_barrier();
      if (OW) {
        WStream<1, Q1> s;
        s.start(wr, voff, T1, orb);
        f4 acc[1][1] = {{zero}};
        s.template run<CB, 1>(wr, voff, A, ocb, lane, acc);
        store_to(a.gx, 0, orb, a.D, s0 + 16 * ocb, ocell < a.B, acc[0][0]);
      }
      lds_barrier();      // (A is written again)
    }
  }
}

// ------------------------------------------------------------------ weight gradients
struct DwLayer {
  int A, B;                // rows of dZ_l and a_(l-1) in a tile's block
  int M, N;                // how many
  int64_t out, bout;       // offsets of W_l and b_l in the parameter vector
  int wm, tm, tn;          // waves along M (the others along N); workgroup tiles
  int kc, begin;           // 32-sample blocks per split; the first workgroup
};
struct DwArgs {
  DwLayer l[4];
  const float *blk;        // the tiles' blocks, `rows` rows of 32 floats each
  int rows, nk;            // blocks
  float *part;             // [splits][np]
  int64_t np;
};

constexpr int DF = 24;                // most operand fragments of a workgroup tile

// Partial dW tile of one batch split: eight waves share out its blocks of 16 x
// 16, WM along the rows.  Per 32 samples the tile's operand fragments (16 rows
// x 32 samples, one 2 KiB piece of a block) are shared out over the waves,
// which load them two blocks ahead, split them and put the parts into one of
// two LDS buffers while the other's products run; each operand is loaded and
// split once per workgroup.  (Four waves that load and split their own
// operands read 1.1 GB for 65,536 samples and spend as long on the splits as
// on the products: 177 us for 65,536 samples, against 155 in a trace of single
// steps now, 181 under a continuous load's lower clock.)  db_l: the row sums of
// the dZ_l fragments, by the waves that load them, in the tiles of the first
// column.
//
// NI x NJ: the most blocks of a wave (the last waves' missing ones are computed
// on other rows and not written).
template <int NI, int NJ>
__device__ __forceinline__ void dw_tile(const DwArgs &a, const DwLayer &L, uint8_t (*ops)[DF * TF]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = (blockIdx.x - L.begin) % (L.tm * L.tn), zt = (blockIdx.x - L.begin) / (L.tm * L.tn);
  const int by = tile / L.tn, bx = tile % L.tn, RM = (L.M + 15) / 16, RN = (L.N + 15) / 16;
  // blocks of the workgroup tile, shared evenly, and this wave's
  const int m0 = by * RM / L.tm, n0 = bx * RN / L.tn;
  const int na = (by + 1) * RM / L.tm - m0, nb = (bx + 1) * RN / L.tn - n0;
  const int wn = NW / L.wm, wi = w % L.wm, wj = w / L.wm;
  const int i0 = wi * na / L.wm, j0 = wj * nb / wn;
  const int ni = (wi + 1) * na / L.wm - i0, nj = (wj + 1) * nb / wn - j0;
  const int k0 = zt * L.kc, k1 = k0 + L.kc < a.nk ? k0 + L.kc : a.nk;

  // fragment f = w + 8 u < na + nb of the tile: rows of dZ first, then of the
  // activation (waves without a u-th one load the last, and do not store it)
  constexpr int NL = DF / NW;
  const int vo = c16 * MC + 4 * g;
  int fo[NL];
  bool fv[NL];
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    fv[u] = w + NW * u < na + nb;
    const int f = fv[u] ? w + NW * u : na + nb - 1;
    fo[u] = (f < na ? L.A + 16 * (m0 + f) : L.B + 16 * (n0 + f - na)) * MC;
  }
  f4 raw[2][NL][2];
  auto load = [&](int s, int k) {
    const float *const blk = a.blk + (int64_t)(k < k1 ? k : k1 - 1) * a.rows * MC;
#pragma unroll
    for (int u = 0; u < NL; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) raw[s][u][h] = *(const f4 *)(blk + fo[u] + 16 * h + vo);
  };
  float rs[NL] = {0.f, 0.f, 0.f};
  // splits raw set s into LDS buffer s; the row sums
  auto stage = [&](int s) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      if (!fv[u]) break;
      const f4 *const r = raw[s][u];
      const Split4 x = split4(r[0]), y = split4(r[1]);
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const u2 lo = __builtin_bit_cast(u2, x.p[p]), hi = __builtin_bit_cast(u2, y.p[p]);
        *(i4 *)(ops[s] + (w + NW * u) * TF + p * FB + lane * 16) =
            i4{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
      }
      rs[u] += ((r[0][0] + r[0][1]) + (r[0][2] + r[0][3])) + ((r[1][0] + r[1][1]) + (r[1][2] + r[1][3]));
    }
  };
  f4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  // products of LDS buffer s
  auto products = [&](int s) {
    const uint8_t *const pa = ops[s] + i0 * TF + lane * 16, *const pb = ops[s] + (na + j0) * TF + lane * 16;
    i4 fa[NI][3], fb[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) fb[0][p] = *(const i4 *)(pb + p * FB);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) fa[i][p] = *(const i4 *)(pa + (i < ni ? i : 0) * TF + p * FB);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (j >= nj) break;
      if (j + 1 < NJ)
#pragma unroll
        for (int p = 0; p < 3; ++p) fb[(j + 1) & 1][p] = *(const i4 *)(pb + (j + 1 < nj ? j + 1 : 0) * TF + p * FB);
      f4 lo[NI];
#pragma unroll
      for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int i = 0; i < NI; ++i)
          lo[i] = mma(fa[i][kTermA[t]], fb[j & 1][kTermB[t]], t == 0 ? f4{0.f, 0.f, 0.f, 0.f} : lo[i]);
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i][j] = mma(fa[i][0], fb[j & 1][0], acc[i][j]);
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i][j] += lo[i];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // block k from buffer s; block k + 1 is put into the other one, block k + 3 loaded
  // - the four waves of a SIMD's first half before their products, those of
  // the other half after them, so that one's splits run beside the other's
  // products
  auto step = [&](int s, int k) {
    lds_barrier();
    auto next = [&]() {
      if (k + 1 < k1) {
        stage(s ^ 1);
        load(s ^ 1, k + 3);
      }
    };
    if (w < NW / 2) next();
    products(s);
    if (w >= NW / 2) next();
  };
  load(0, k0);
  load(1, k0 + 1);
  stage(0);
  load(0, k0 + 2);
  for (int k = k0; k < k1; k += 2) {
    step(0, k);
    if (k + 1 < k1) step(1, k + 1);
  }
  float *const C = a.part + (int64_t)zt * a.np;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (i >= ni || j >= nj) continue;
      const int n = 16 * (n0 + j0 + j) + c16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * (m0 + i0 + i) + 4 * g + r;
        if (m < L.M && n < L.N) C[L.out + (int64_t)m * L.N + n] = acc[i][j][r];
      }
    }
  if (bx == 0)
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int f = w + NW * u;
      float t = rs[u];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (f < na && g == 0 && 16 * (m0 + f) + c16 < L.M) C[L.bout + 16 * (m0 + f) + c16] = t;
    }
}

__global__ __launch_bounds__(512, 1) void dw_split_kernel(DwArgs a) {
  __shared__ __align__(16) uint8_t ops[2][DF * TF];
  int l = 3;
  while ((int)blockIdx.x < a.l[l].begin) --l;
  switch (l) {
    case 0: dw_tile<2, 2>(a, a.l[0], ops); break;
    case 1: dw_tile<4, 4>(a, a.l[1], ops); break;
    case 2: dw_tile<4, 4>(a, a.l[2], ops); break;
    default: dw_tile<2, 1>(a, a.l[3], ops);
  }
}

// ------------------------------------------------------------------ finish
struct FinishArgs {
  const float *part;       // [splits][np]
  int64_t np, end[4];      // end of each layer's parameters
  int nsplit[4], accum;    // splits per layer; accum: add to the gradient (a later chunk)
  float *grads;
  float *p, *m, *v;        // Adam update, or p = NULL
  float lr, c1, c2;
  const float *lpart;      // loss: nl partial sums of this chunk, or NULL
  int64_t nl;
  double *closs;           // sum of the chunks so far
  double denom;
  float *loss;             // after the last chunk, else NULL
};

// The gradient: 64 outputs per workgroup, its four waves sum a quarter of the
// splits each in increasing order, the quarters in wave order; then Adam on
// the sum.  The last workgroup sums the loss (fixed order, FP64).  Bound by the
// latency of the loads, so several of each lane's are in flight together (one
// after the other, and one wave for the loss: 12.6 us at 65,536 samples; so 7).
__global__ __launch_bounds__(256) void finish_kernel(FinishArgs a) {
  __shared__ float q[4][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t o = blockIdx.x * (int64_t)64 + l;
  if (blockIdx.x * (int64_t)64 >= a.np) {
    // (the loss: all four waves, eight loads of each lane in flight)
    __shared__ double qs[4];
    double s = 0.0;
    for (int64_t i0 = threadIdx.x; i0 < a.nl; i0 += 8 * 256) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = i0 + 256 * u < a.nl ? a.lpart[i0 + 256 * u] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) s += (double)v[u];
    }
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) s += __shfl_xor(s, k);
    if (l == 0) qs[w] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      s = ((qs[0] + qs[1]) + qs[2]) + qs[3];
      if (a.accum) s += *a.closs;
      if (a.loss) *a.loss = (float)(s / a.denom);
      else *a.closs = s;
    }
    return;
  }
  const bool valid = o < a.np;
  const int ns = o < a.end[0] ? a.nsplit[0] : o < a.end[1] ? a.nsplit[1] : o < a.end[2] ? a.nsplit[2] : a.nsplit[3];
  const int zq = (ns + 3) / 4, z0 = w * zq, z1 = z0 + zq < ns ? z0 + zq : ns;
  float acc = 0.0f;
  if (valid)
    for (int z = z0; z < z1; z += 4) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = a.part[(int64_t)(z + u < z1 ? z + u : z1 - 1) * a.np + o];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = z + u < z1 ? acc + v[u] : acc;
    }
  q[w][l] = acc;
  __syncthreads();
  if (w == 0 && valid) {
    float t = ((q[0][l] + q[1][l]) + q[2][l]) + q[3][l];
    if (a.accum) t += a.grads[o];
    a.grads[o] = t;
    if (a.p) {
      const float mi = 0.9f * a.m[o] + 0.1f * t;
      const float vi = 0.999f * a.v[o] + 0.001f * t * t;
      a.m[o] = mi;
      a.v[o] = vi;
      a.p[o] -= a.lr * (mi * a.c1) / (__builtin_sqrtf(vi * a.c2) + 1e-8f);
    }
  }
}

// ------------------------------------------------------------------ host
namespace {

size_t up256(size_t b) { return (b + 255) / 256 * 256; }
int64_t chunk_samples(int64_t cap, int64_t chunk) { return chunk > 0 && chunk < cap ? chunk : cap; }
int64_t whole_tiles(int64_t n) { return (n + MC - 1) / MC * MC; }
int64_t params_of(const int *w) {
  int64_t o = 0;
  for (int l = 0; l < 4; ++l) o += (int64_t)w[l] * w[l + 1] + w[l + 1];
  return o;
}

// Splits of the weight gradients' batch of nk 32-sample blocks: at most 34 of
// the second and third layer (with their tiles and the other layers' fewer,
// longer splits, one round of workgroups on 256 CUs), one block at least; 27 up
// to 293 blocks, where the partial sums of more (0.43 MB a split) would outgrow
// the static scratch of the allocation-free step (293 blocks, 9,376 samples: the
// largest chunk of one species that it takes; 9,184 of 17).  Never more for
// fewer blocks: the scratch is sized by the largest chunk, and a batch's last
// chunk is smaller.  64 / 4,096 / 8,192 samples a step: at most 24 splits of two
// blocks at least 47.2 / 58.9 / 74.6 us, so 45.0 / 57.5 / 73.5.
int64_t max_splits(int64_t nk) {
  const int64_t most = nk <= 293 ? 27 : 34;
  return nk < most ? nk : most;
}
int split_blocks(int64_t nk) {
  const int64_t most = max_splits(nk), k = (nk + most - 1) / most;
  return (int)(k < 1 ? 1 : k);
}

// Tiles of 16 samples while they fit one round of workgroups (the chain of a
// tile's eight products takes 18 us with 16 samples and 29 with 32), of 32
// beyond (whose weights are read half as often).
int tile_samples(int64_t n, int n_cu) { return n <= 16 * (int64_t)n_cu ? 16 : 32; }

template <int MODE, bool GX, int CB> hipError_t tile_launch_cb(const TileArgs &a, int n_cu, hipStream_t s) {
  const int64_t nt = tiles_of(a.B, 16 * CB);
  hipLaunchKernelGGL((tile_kernel<MODE, GX, CB>), dim3((unsigned)(nt < n_cu ? nt : n_cu)), dim3(NW * 64),
                     TileLds<CB>::BYTES, s, a);
  return hipGetLastError();
}
template <int MODE, bool GX> hipError_t tile_launch(const TileArgs &a, int n_cu, hipStream_t s) {
  return tile_samples(a.B, n_cu) == 16 ? tile_launch_cb<MODE, GX, 1>(a, n_cu, s)
                                       : tile_launch_cb<MODE, GX, 2>(a, n_cu, s);
}
template <int MODE, bool GX> hipError_t tile_prepare() {
  hipError_t e = hipFuncSetAttribute((const void *)tile_kernel<MODE, GX, 1>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, TileLds<1>::BYTES);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void *)tile_kernel<MODE, GX, 2>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, TileLds<2>::BYTES);
}

hipError_t pack(const int *w, const float *params, uint8_t *dst, hipStream_t s) {
  const int64_t o1 = 0, o2 = o1 + (int64_t)w[0] * H1 + H1, o3 = o2 + (int64_t)H1 * H2 + H2,
                o4 = o3 + (int64_t)H2 * H3 + H3;
  PackArgs a{params, dst,
             {{o1, H1, w[0], w[0], 1, 1, P1}, {o2, H2, H1, H1, 1, Q1, P2}, {o3, H3, H2, H2, 1, Q2, P3},
              {o4, w[4], H3, H3, 1, Q3, P4}, {o4, H3, w[4], 1, H3, 1, T4}, {o3, H2, H3, 1, H2, Q3, T3},
              {o2, H1, H2, 1, H1, Q2, T2}, {o1, w[0], H1, 1, w[0], Q1, T1}}};
  hipLaunchKernelGGL(split_pack_kernel, dim3((PEND * 64 + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Weight and bias gradients of n samples in the scratch, summed into `f`.
hipError_t weight_grads(const int *w, int64_t n, const TileScratch *t, FinishArgs f, hipStream_t s) {
  DwArgs d{};
  const int D = w[0];
  const int A[4] = {row_dz(D), row_dz(D) + H1, row_dz(D) + H1 + H2, row_do(D)};
  const int B[4] = {0, row_a(D), row_a(D) + H1, row_a(D) + H1 + H2};
  int64_t off = 0;
  d.blk = t->blk;
  d.rows = rows(w[0], w[4]);
  d.nk = (int)((n + MC - 1) / MC);
  const int kc = split_blocks(d.nk);
  // waves along M, tiles and the length of a split per layer, by what a block
  // of 32 samples costs its workgroup: 33 block pairs on the busiest SIMD for
  // the second layer, 28 for the third, 8 and 2 for the thin ones
  constexpr int WM[4] = {8, 4, 2, 1}, TM[4] = {2, 1, 1, 1}, TN[4] = {1, 4, 1, 1}, KL[4] = {5, 4, 4, 5};
  int grid = 0;
  for (int l = 0; l < 4; ++l) {
    const int M = w[l + 1], N = w[l];
    d.l[l] = DwLayer{A[l], B[l], M, N, off, off + (int64_t)M * N, WM[l], TM[l], TN[l], kc * KL[l] / 4, grid};
    off += (int64_t)M * N + M;
    f.end[l] = off;
    f.nsplit[l] = (d.nk + d.l[l].kc - 1) / d.l[l].kc;
    if (f.nsplit[l] > t->splits) return hipErrorInvalidValue;
    grid += TM[l] * TN[l] * f.nsplit[l];
  }
  d.part = t->part;
  d.np = off;
  hipLaunchKernelGGL(dw_split_kernel, dim3((unsigned)grid), dim3(NW * 64), 0, s, d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  f.part = t->part;
  f.np = off;
  hipLaunchKernelGGL(finish_kernel, dim3((unsigned)((off + 63) / 64 + (f.lpart ? 1 : 0))), dim3(256), 0, s, f);
  return hipGetLastError();
}

}  // namespace

bool tile_shape(const int *w) {
  return w[0] <= 32 && w[1] == H1 && w[2] == H2 && w[3] == H3 && w[4] <= 32;
}

// Scratch blocks of n samples (whole tiles), and the rows that a ragged
// fragment at the end of the last block reads past it.
static size_t block_bytes(const int *w, int64_t n) {
  return up256(((size_t)n * rows(w[0], w[4]) + 16 * MC) * 4);
}

size_t tile_scratch_bytes(const int *w, int64_t cap, int64_t chunk) {
  size_t b = up256((size_t)PEND * TF);
  if (cap <= 0) return b;
  const int64_t c = chunk_samples(cap, chunk), n = whole_tiles(c);
  return b + block_bytes(w, n) + up256((size_t)max_splits(n / MC) * params_of(w) * 4) +
         up256((size_t)(n / 16) * 4) + up256(sizeof(double));
}

void tile_scratch_layout(TileScratch *t, uint8_t *base, const int *w, int64_t cap, int64_t chunk) {
  *t = TileScratch{};
  auto take = [&](size_t bytes) {
    uint8_t *p = base;
    base += up256(bytes);
    return p;
  };
  t->pack = take((size_t)PEND * TF);
  t->cap = cap;
  if (cap <= 0) return;
  t->chunk = chunk_samples(cap, chunk);
  const int64_t n = whole_tiles(t->chunk);
  t->blk = (float *)take(block_bytes(w, n));
  t->splits = max_splits(n / MC);
  t->part = (float *)take((size_t)t->splits * params_of(w) * 4);
  t->lpart = (float *)take((size_t)(n / 16) * 4);
  t->closs = (double *)base;
}

hipError_t tile_prepare_all() {
  hipError_t e = tile_prepare<TILE_TRAIN, false>();
  if (e == hipSuccess) e = tile_prepare<TILE_FWD, false>();
  if (e == hipSuccess) e = tile_prepare<TILE_BWD_SAVED, false>();
  if (e == hipSuccess) e = tile_prepare<TILE_BWD_SAVED, true>();
  if (e == hipSuccess) e = tile_prepare<TILE_BWD, false>();
  if (e == hipSuccess) e = tile_prepare<TILE_BWD, true>();
  return e;
}

// Forward over B samples of x [D][ld]; the pre-activations go to `saved`
// ([HT][ld]) if given.
hipError_t tile_mlp_forward(const int *w, int64_t B, int64_t ld, const float *x, const float *params,
                            float *out, float *saved, const TileScratch *t, int n_cu, hipStream_t s) {
  hipError_t e = pack(w, params, t->pack, s);
  if (e != hipSuccess) return e;
  TileArgs a{};
  a.x = x;
  a.ld = ld;
  a.out = out;
  a.zs = saved;
  a.params = params;
  a.pack = t->pack;
  a.B = B;
  a.D = w[0];
  a.S = w[4];
  return tile_launch<TILE_FWD, false>(a, n_cu, s);
}

// Backward over B samples, chunk by chunk, from the saved pre-activations or
// from recomputed ones (the same bits: the same products in the same order).
hipError_t tile_mlp_backward(const int *w, int64_t B, int64_t ld, const float *x, const float *params,
                             const float *saved, const float *grad_out, float *grad_params,
                             float *grad_x, const TileScratch *t, int n_cu, hipStream_t s) {
  if (B > t->cap) return hipErrorInvalidValue;
  if (B <= 0) return hipSuccess;
  hipError_t e = pack(w, params, t->pack, s);
  for (int64_t c0 = 0; c0 < B && e == hipSuccess; c0 += t->chunk) {
    const int64_t n = B - c0 < t->chunk ? B - c0 : t->chunk;
    TileArgs a{};
    a.x = x + c0;
    a.go = grad_out + c0;
    a.z = saved ? saved + c0 : nullptr;
    a.ld = ld;
    a.gx = grad_x ? grad_x + c0 : nullptr;
    a.params = params;
    a.pack = t->pack;
    a.blk = t->blk;
    a.B = n;
    a.D = w[0];
    a.S = w[4];
    if (saved)
      e = grad_x ? tile_launch<TILE_BWD_SAVED, true>(a, n_cu, s) : tile_launch<TILE_BWD_SAVED, false>(a, n_cu, s);
    else
      e = grad_x ? tile_launch<TILE_BWD, true>(a, n_cu, s) : tile_launch<TILE_BWD, false>(a, n_cu, s);
    if (e != hipSuccess) return e;
    FinishArgs f{};
    f.accum = c0 > 0;
    f.grads = grad_params;
    e = weight_grads(w, n, t, f, s);
  }
  return e;
}

// One training step, chunk by chunk; the loss and Adam with the last chunk's
// gradient.
hipError_t tile_train_step(const int *w, int64_t B, int64_t ld, const double *T, const double *P,
                           const double *Y, const float *target, float *params, float *grads,
                           float *adam_m, float *adam_v, float lr, float c1, float c2, float *loss,
                           const float *fc, const double *dc, const TileScratch *t, int n_cu,
                           hipStream_t s) {
  if (B > t->cap) return hipErrorInvalidValue;
  hipError_t e = pack(w, params, t->pack, s);
  const double denom = (double)B * w[4];
  for (int64_t c0 = 0; c0 < B && e == hipSuccess; c0 += t->chunk) {
    const int64_t n = B - c0 < t->chunk ? B - c0 : t->chunk;
    TileArgs a{};
    a.T = T + c0;
    a.P = P + c0;
    a.Y = Y + c0;
    a.go = target + c0;
    a.ld = ld;
    a.params = params;
    a.pack = t->pack;
    a.blk = t->blk;
    a.lpart = t->lpart;
    a.inv = 2.0f / (float)denom;
    a.B = n;
    a.D = w[0];
    a.S = w[4];
    a.fc = fc;
    a.dc = dc;
    e = tile_launch<TILE_TRAIN, false>(a, n_cu, s);
    if (e != hipSuccess) return e;
    FinishArgs f{};
    f.accum = c0 > 0;
    f.grads = grads;
    f.lpart = t->lpart;
    f.nl = tiles_of(n, tile_samples(n, n_cu));
    f.closs = t->closs;
    if (c0 + n >= B) {
      f.p = params;
      f.m = adam_m;
      f.v = adam_v;
      f.lr = lr;
      f.c1 = c1;
      f.c2 = c2;
      f.denom = denom;
      f.loss = loss;
    }
    e = weight_grads(w, n, t, f, s);
  }
  return e;
}

}  // namespace chemdnn
