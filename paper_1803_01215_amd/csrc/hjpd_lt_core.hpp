// Register-resident iteration of the linear-tanh family, shared by the forward
// kernel and the reverse sweep's recompute (hjpd_lintanh.hip).
//
// Layout.  A point's stacked state X, P, Z (nodes 1..N by d coordinates) stays
// in registers in the matrix-core accumulator layout: column tile t, lane
// (lr = lane & 15, lk = lane >> 4), element r holds node NT lr + t + 1 and
// coordinate 16 (row tile) + 4 lk + r.  A lane so holds NT consecutive nodes,
// like the lanes of the other families' kernels: the neighbour z_{j-1} or
// p_{j+1} is another of its own registers except at its first or last node,
// where one DPP row shift fetches it.  Node 0 (x_0, z_0) lives in the lanes
// lr = 0 and is zero in the others.
//
// d = 16, 32: one wave holds all rows of a point.  The k index of a matrix
// product may be taken in any order as long as both operands agree; with
// k = 16 (row tile) + 4 lk + r the state registers themselves are the B
// operands of v_mfma_f32_16x16x4_f32, and an iteration touches no LDS and
// needs no barrier.
//
// d = 100, 128: one wave per row tile (7 or 8).  A product needs every
// coordinate of a node, so each wave writes its rows of X (of P) to an LDS
// image and reads all of it back as B operands.  The image holds each FP32
// value as three bfloat16 pieces, x = h + m + l (8 significand bits each, the
// sum exact up to the smallest normal numbers), and a product sums the six
// piece products down to 2^-16 on v_mfma_f32_16x16x32_bf16; what is left out
// (m l, l m, l l) is at most 2^-25 of each term, below FP32's own rounding.
// The five small products of every k-step are summed first and the h h products
// last, so only d / 32 roundings happen at the size of the result, where the
// FP32 instruction rounds d / 4 times.  Six products of K = 32 take 96 cycles
// of the matrix unit where eight FP32 products of K = 4 take 256.  With
// d = 100 the last four coordinates are one FP32 product of their own.
//
// What bounds it, and what it measured.  A SIMD runs matrix and vector
// instructions almost one after the other (a probe of two waves a SIMD: 17.7
// cycles a bfloat16 product, 4.3 a vector instruction, together 31.5 for one
// product and four vector instructions), so the time is their sum: at d = 100,
// N = 50 each of two waves a SIMD issues 152 products and 540 vector
// instructions an iteration, 10,100 cycles measured against 10,200 of issue;
// LDS is busy for 4,200 of them.  The 22 % of columns and of the last row tile
// that are padding are what is left.  16,384 points of 500 iterations: 286 ms
// with the state in LDS and FP32 products, 136 ms; d = 32, N = 24, 512 points
// of 100 iterations 0.70 -> 0.22 ms; d = 16, N = 12, 5 points 228 -> 50 us.
#pragma once

#include <type_traits>

#include "hjpd_device.hpp"
#include "hjpd_lintanh.hpp"

namespace hjpd {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma32(bf8 a, bf8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// tanh from the exponential, tanh|x| = 1 - 2 / (exp(2|x|) + 1), sign restored:
// one hardware exp and one reciprocal; absolute error at FP32 rounding level.
__device__ __forceinline__ float tanh_fast(float x) {
  const float e = __expf(2.f * fabsf(x));
  const float t = 1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f);
  return copysignf(t, x);
}

// Two floats rounded to nearest bfloat16, packed (first in the low half).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, bf2));
}
// x = h + m + l in bfloat16 pieces; the differences are exact in FP32.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack_bf16(a, b);
  const float a1 = a - __uint_as_float(h << 16), b1 = b - __uint_as_float(h & 0xffff0000u);
  m = pack_bf16(a1, b1);
  l = pack_bf16(a1 - __uint_as_float(m << 16), b1 - __uint_as_float(m & 0xffff0000u));
}

// Register element r of the previous / next lane of the 16-lane row (0 at the row's end).
__device__ __forceinline__ f4 row_prev(f4 v) {
  return f4{dpp_f<kDppRowShr1>(v[0]), dpp_f<kDppRowShr1>(v[1]), dpp_f<kDppRowShr1>(v[2]), dpp_f<kDppRowShr1>(v[3])};
}
__device__ __forceinline__ f4 row_next(f4 v) {
  return f4{dpp_f<kDppRowShl1>(v[0]), dpp_f<kDppRowShl1>(v[1]), dpp_f<kDppRowShl1>(v[2]), dpp_f<kDppRowShl1>(v[3])};
}

struct LtArgs {
  const float* x;
  const float* t;
  const int32_t* N;
  const float* hp;  // [eps, A (d*d)]
  const float* Q;   // [d*d]
  const float* M;   // (I + tau Q_s)^{-1}
  float* phi;
  float* xtraj;
  float* ptraj;
  int32_t* iters;
  int32_t* status;
  int32_t* head;
  int64_t n;
  float sigma, tau, theta, tol;
  int max_iter, fixed, N_max;
  uint64_t seed;
  // checkpoints: per point n_ckpt + 1 snapshots of (X, P, Z), each 3 (N_max+1) d;
  // snapshot c holds the state before iteration c E, the last one the final state
  float* ckpt;
  int ckpt_every;
  int n_ckpt;
};

template <int D, int NT>
struct LtShape {
  static_assert(D % 4 == 0 && (D <= 32 ? D % 16 == 0 : D % 32 == 0 || D % 32 == 4), "built for d in {16, 32, 100, 128}");
  static constexpr int RT = (D + 15) / 16;
  static constexpr bool kReg = D <= 32;     // one wave holds every row of a point
  static constexpr int RPW = kReg ? RT : 1; // row tiles per wave
  static constexpr bool kAux = !kReg && RT < 8;  // a wave of its own steps node 0
  static constexpr int W = kReg ? 1 : RT + kAux;  // waves per workgroup
  static constexpr int kThreads = 64 * W;
  static constexpr int KB = kReg ? 0 : D / 32;       // bfloat16 k-steps of a product
  static constexpr bool kTail = !kReg && D % 32 != 0; // one FP32 k-step of 4 after them
  static constexpr int ROWS = 16 * NT;               // image rows (columns of a product)
  // An image piece is laid out [k / 8][row][8] (M: [k / 4][row][4]): the 16-byte
  // reads of any 16 lanes with distinct rows, and the 8-byte writes of 32 lanes,
  // cover the 64 banks once.  Rows padded to 16 bytes over a power of two lost
  // 2,850 of 6,240 LDS cycles an iteration to conflicts (d = 100, N = 50).
  static constexpr int PIECE = 32 * KB * ROWS;  // bfloat16 per piece
  static constexpr int MR = D;                  // rows of M in LDS
  // LDS in floats: two images (X, P), their FP32 tails, M, the node-0 vector, reduction slots
  static constexpr int kImg = kReg ? 0 : 3 * PIECE / 2;
  static constexpr int kTailF = kTail ? 4 * ROWS : 0;
  static constexpr int kM = kReg ? 0 : D * MR;
  static constexpr int kVec = 16 * RT;
  // tanh(x_j) from the dual step to the primal step, where it fits beside the rest
  static constexpr bool kThLds = !kReg && D < 128;
  static constexpr int kTh = kThLds ? 256 * RT * NT : 0;
  static constexpr int kLdsFloats = 2 * kImg + 2 * kTailF + kM + 4 * kVec + kTh + 2 * W + 2;
};

// A matrix's rows of one wave as A operands.
template <int D, int NT>
struct LtFrag {
  using S = LtShape<D, NT>;
  float f[S::kReg ? S::RPW : 1][S::kReg ? 4 * S::RPW : 1];  // FP32 operands (kReg), or the tail's
  bf8 h[S::kReg ? 1 : S::KB], m[S::kReg ? 1 : S::KB], l[S::kReg ? 1 : S::KB];

  // entry (row, k) at a[row * rs + k * ks]
  __device__ void load(const float* a, int rs, int ks, int wave, int lr, int lk) {
    if constexpr (S::kReg) {
#pragma unroll
      for (int ro = 0; ro < S::RPW; ro++)
#pragma unroll
        for (int q = 0; q < 4 * S::RPW; q++)
          f[ro][q] = a[(16 * ro + lr) * rs + (16 * (q / 4) + 4 * lk + q % 4) * ks];
    } else {
      const int row = 16 * wave + lr;
      const bool ok = row < D;
#pragma unroll
      for (int s = 0; s < S::KB; s++) {
        uint32_t hh[4], mm[4], ll[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int k = 32 * s + 8 * lk + 2 * e;
          const float u = ok ? a[row * rs + k * ks] : 0.f, v = ok ? a[row * rs + (k + 1) * ks] : 0.f;
          split_pair(u, v, hh[e], mm[e], ll[e]);
        }
        h[s] = __builtin_bit_cast(bf8, hh);
        m[s] = __builtin_bit_cast(bf8, mm);
        l[s] = __builtin_bit_cast(bf8, ll);
      }
      if constexpr (S::kTail) f[0][0] = ok ? a[row * rs + (32 * S::KB + lk) * ks] : 0.f;
    }
  }
};

// Kinds of wave.  Each runs code of its own, from the point loop down: with
// one code and a branch per step the compiler joined the state's registers
// after every branch, 70 copies and spills an iteration.
enum : int {
  kRowWave = 0,   // rows of every column tile
  kTailWave = 1,  // the same, for the rows past the last bfloat16 k-step (d = 100)
  kAuxWave = 2,   // node 0 (d = 100, whose seven row tiles leave an eighth wave)
};

// One point's iteration, by one wave; every wave of the workgroup runs it together.
template <int D, int NT, int KIND>
struct LtCore {
  using S = LtShape<D, NT>;
  using Frag = LtFrag<D, NT>;
  static constexpr int RPW = S::RPW;
  static constexpr bool kRows = KIND != kAuxWave;
  typedef f4 Tiles[RPW][NT];

  int tid, wave, lr, lk;
  // LDS (d > 32): bfloat16 images of X and P, their tails, M, a vector, reduction slots
  uint16_t *imgX, *imgP;
  float *tailX, *tailP, *sM, *sTh;
  float *sX0, *sZ0, *sV, *sW;  // x_0, z_0, p_1 (also scratch), x_0 + tau p_1
  float* sRed;
  uint32_t put_at, get_at;  // this lane's element offsets into an image
  Frag fA, fAt;
  float fM[S::kReg ? S::RPW : 1][S::kReg ? 4 * S::RPW : 1];

  // state of the current point
  Tiles X, P, Z;
  f4 x0[RPW], z0[RPW];  // d <= 32; otherwise node 0 is in LDS
  int Np;
  float delta, lam, c1;

  __device__ int coord(int ri) const { return 16 * (S::kReg ? ri : wave) + 4 * lk; }  // of element r = 0
  __device__ int node(int t) const { return NT * lr + t + 1; }
  __device__ bool rows_ok(int ri) const { return S::kReg || D % 16 == 0 || coord(ri) < D; }

  __device__ void setup(const LtArgs& a, float* lds) {
    tid = threadIdx.x;
    wave = S::W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    lr = tid & 15;
    lk = (tid & 63) >> 4;
    if constexpr (kRows) {
      fA.load(a.hp + 1, D, 1, wave, lr, lk);
      fAt.load(a.hp + 1, 1, D, wave, lr, lk);
    }
    imgX = reinterpret_cast<uint16_t*>(lds);
    imgP = reinterpret_cast<uint16_t*>(lds + S::kImg);
    tailX = lds + 2 * S::kImg;
    tailP = tailX + S::kTailF;
    sM = tailP + S::kTailF;
    sTh = sM + S::kM;
    sX0 = sTh + S::kTh;
    sZ0 = sX0 + S::kVec;
    sV = sZ0 + S::kVec;
    sW = sV + S::kVec;
    sRed = sW + S::kVec;
    put_at = ((2 * wave + (lk >> 1)) * S::ROWS + lr) * 8 + (lk & 1) * 4;
    get_at = (lk * S::ROWS + lr) * 8;
    if constexpr (S::kReg) {
#pragma unroll
      for (int ro = 0; ro < RPW; ro++)
#pragma unroll
        for (int q = 0; q < 4 * RPW; q++) fM[ro][q] = a.M[(16 * ro + lr) * D + 16 * (q / 4) + 4 * lk + q % 4];
    } else {
      for (int e = tid; e < D * S::MR; e += S::kThreads) {
        const int k = e / (4 * S::MR) * 4 + e % 4, row = e / 4 % S::MR;
        sM[e] = row < D ? a.M[row * D + k] : 0.f;
      }
      for (int e = tid; e < 4 * S::kVec; e += S::kThreads) sX0[e] = 0.f;  // entries past d stay zero
      __syncthreads();
    }
  }

  // This wave's rows of column tile t into an image (the tail wave: into the FP32 tail).
  __device__ __forceinline__ void put(uint16_t* img, float* tail, int t, f4 v) const {
    if constexpr (KIND == kRowWave) {
      u2 h, m, l;
      uint32_t a0, a1, b0, b1, g0, g1;
      split_pair(v[0], v[1], a0, b0, g0);
      split_pair(v[2], v[3], a1, b1, g1);
      h = u2{a0, a1};
      m = u2{b0, b1};
      l = u2{g0, g1};
      uint16_t* q = img + put_at + t * 16 * 8;
      *reinterpret_cast<u2*>(q) = h;
      *reinterpret_cast<u2*>(q + S::PIECE) = m;
      *reinterpret_cast<u2*>(q + 2 * S::PIECE) = l;
    } else if (lk == 0) {
      *reinterpret_cast<f4*>(tail + (16 * t + lr) * 4) = v;
    }
  }

  // Rows of this wave of (matrix) x (column tile t of the image): the small
  // products and the h h products summed apart.  `p` holds the pieces of the
  // first k-steps, read ahead.
  struct Pieces { bf8 h, m, l; };
  static constexpr int kAhead = 2;  // k-steps read ahead
  __device__ __forceinline__ Pieces get(const uint16_t* img, int t, int s) const {
    const uint16_t* q = img + get_at + t * 16 * 8 + s * 32 * S::ROWS;
    return {*reinterpret_cast<const bf8*>(q), *reinterpret_cast<const bf8*>(q + S::PIECE),
            *reinterpret_cast<const bf8*>(q + 2 * S::PIECE)};
  }
  __device__ __forceinline__ f4 product(const Frag& F, const uint16_t* img, const float* tail, int t,
                                        const Pieces (&p)[kAhead]) const {
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (!S::kReg) {
      Pieces rest[S::KB - kAhead];
#pragma unroll
      for (int s = kAhead; s < S::KB; s++) rest[s - kAhead] = get(img, t, s);
      float last = 0.f;
      if constexpr (S::kTail) last = tail[(16 * t + lr) * 4 + lk];
      auto piece = [&](int s) -> const Pieces& { return s < kAhead ? p[s < kAhead ? s : 0] : rest[s < kAhead ? 0 : s - kAhead]; };
#pragma unroll
      for (int s = 0; s < S::KB; s++) {
        const Pieces& b = piece(s);
        v = mfma32(F.l[s], b.h, v);
        v = mfma32(F.h[s], b.l, v);
        v = mfma32(F.m[s], b.m, v);
        v = mfma32(F.m[s], b.h, v);
        v = mfma32(F.h[s], b.m, v);
      }
#pragma unroll
      for (int s = 0; s < S::KB; s++) v = mfma32(F.h[s], piece(s).h, v);
      if constexpr (S::kTail) v = mfma4(F.f[0][0], last, v);
    }
    return v;
  }
  // The same from the state registers (d <= 32): row tile ro, column tile t.
  __device__ __forceinline__ f4 product_reg(const float (&f)[S::kReg ? S::RPW : 1][S::kReg ? 4 * S::RPW : 1],
                                            const f4 (&B)[RPW], int ro) const {
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (S::kReg) {
#pragma unroll
      for (int q = 0; q < 4 * RPW; q++) acc = mfma4(f[ro][q], B[q / 4][q % 4], acc);
    }
    return acc;
  }
  // Node 0 with d > 32: x_0 <- M (x_0 + tau p_1) from p_1 in sV, z_0 with it.
  // d = 100 leaves an eighth wave without rows: it takes the whole product, two
  // outputs to a lane, while the others run the primal product (the row waves
  // would each spend 60 instructions and two cross-lane sums on it, and hold
  // 56 registers).  d = 128: lane (lr, lk) of a row wave sums the terms
  // k = 4 lk .. 4 lk + 3 (mod 16) of row lr.
  template <bool kRes>
  __device__ __forceinline__ void node0(float tau, float theta, float& rx) const {
    auto finish = [&](int i, float xn) {
      const float xo = sX0[i], dx = xn - xo;
      if constexpr (kRes) rx += dx * dx;
      sX0[i] = xn;
      sZ0[i] = xn + theta * dx;
    };
    if constexpr (S::kAux) {
      const int i = tid & 63, i2 = 64 + i < D ? 64 + i : D - 1;
      sW[i] = sX0[i] + tau * sV[i];
      if (64 + i < D) sW[64 + i] = sX0[64 + i] + tau * sV[64 + i];
      __builtin_amdgcn_wave_barrier();
      float u = 0.f, v = 0.f;
#pragma unroll 5
      for (int k = 0; k < D; k += 4) {
        const f4 w = *reinterpret_cast<const f4*>(sW + k);
        const f4 a = *reinterpret_cast<const f4*>(sM + k * S::MR + 4 * i);
        const f4 b = *reinterpret_cast<const f4*>(sM + k * S::MR + 4 * i2);
#pragma unroll
        for (int r = 0; r < 4; r++) {
          u += a[r] * w[r];
          v += b[r] * w[r];
        }
      }
      finish(i, u);
      if (64 + i < D) finish(64 + i, v);
    } else {
      float part = 0.f;
#pragma unroll 2
      for (int k = 4 * lk; k < D; k += 16) {
        const f4 mm = *reinterpret_cast<const f4*>(sM + k * S::MR + 4 * (16 * wave + lr));
        const f4 vv = *reinterpret_cast<const f4*>(sV + k);
#pragma unroll
        for (int r = 0; r < 4; r++) part += mm[r] * vv[r];
      }
      part += __shfl_xor(part, 16, 64);
      part += __shfl_xor(part, 32, 64);
      if (lk == 0) finish(16 * wave + lr, part);
    }
  }

  // Sums over the workgroup of two values (all lanes get them).  The slots are
  // written before and read after one barrier; two barriers lie between uses.
  __device__ __forceinline__ void sum2(float& u, float& v) const {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      u += __shfl_xor(u, m, 64);
      v += __shfl_xor(v, m, 64);
    }
    if constexpr (S::W > 1) {
      if ((tid & 63) == 0) {
        sRed[2 * wave] = u;
        sRed[2 * wave + 1] = v;
      }
      __syncthreads();
      u = v = 0.f;
#pragma unroll
      for (int w = 0; w < S::W; w++) {
        u += sRed[2 * w];
        v += sRed[2 * w + 1];
      }
      __syncthreads();
    }
  }

  __device__ void set_point(const LtArgs& a, int64_t pt) {
    // the same in every lane, kept in scalar registers
    auto uniform = [](float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); };
    Np = __builtin_amdgcn_readfirstlane(a.N[pt]);
    delta = uniform(a.t[pt] / float(Np));
    lam = uniform(a.sigma * delta);
    c1 = uniform(1.f / (1.f + lam));
  }

  // Random start (section 6 set-up); nodes past N are zero.
  __device__ void start(const LtArgs& a, int64_t pt) {
    if constexpr (!S::kReg)
      for (int i = tid; i < D; i += S::kThreads)
        sX0[i] = sZ0[i] = float(double(a.x[pt * D + i]) + start_noise(a.seed, uint64_t(pt), kArrX, 0, i));
    if constexpr (kRows)
#pragma unroll
    for (int ri = 0; ri < RPW; ri++) {
      const int i0 = coord(ri);
      f4 xt = f4{0.f, 0.f, 0.f, 0.f};
      if (rows_ok(ri))
#pragma unroll
        for (int r = 0; r < 4; r++) xt[r] = a.x[pt * D + i0 + r];
      if constexpr (S::kReg) {
        x0[ri] = f4{0.f, 0.f, 0.f, 0.f};
        if (lr == 0)
#pragma unroll
          for (int r = 0; r < 4; r++)
            x0[ri][r] = float(double(xt[r]) + start_noise(a.seed, uint64_t(pt), kArrX, 0, i0 + r));
        z0[ri] = x0[ri];
      }
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const int j = node(t);
        X[ri][t] = P[ri][t] = f4{0.f, 0.f, 0.f, 0.f};
        if (j <= Np && rows_ok(ri))
#pragma unroll
          for (int r = 0; r < 4; r++) {
            X[ri][t][r] =
                j < Np ? float(double(xt[r]) + start_noise(a.seed, uint64_t(pt), kArrX, j, i0 + r)) : xt[r];
            P[ri][t][r] = float(start_noise(a.seed, uint64_t(pt), kArrP, j, i0 + r));
          }
        Z[ri][t] = X[ri][t];
        fence();
      }
    }
    put_all(imgX, tailX, X);
  }
  // A whole image, ready to be read.
  __device__ __forceinline__ void put_all(uint16_t* img, float* tail, const Tiles& V) const {
    if constexpr (!S::kReg) {
      if constexpr (kRows)
#pragma unroll
        for (int t = 0; t < NT; t++) put(img, tail, t, V[0][t]);
      __syncthreads();
    }
  }

  // Node 0 of this lane's rows: x_0, z_0 in the lanes lr = 0, zero in the others.
  __device__ __forceinline__ f4 x0_of(int ri) const {
    if constexpr (S::kReg) return x0[ri];
    else return first_col(*reinterpret_cast<const f4*>(sX0 + (rows_ok(0) ? coord(0) : 0)));
  }
  __device__ __forceinline__ f4 z0_of(int ri) const {
    if constexpr (S::kReg) return z0[ri];
    else return first_col(*reinterpret_cast<const f4*>(sZ0 + (rows_ok(0) ? coord(0) : 0)));
  }
  __device__ __forceinline__ f4 first_col(f4 v) const {
    const bool on = lr == 0 && rows_ok(0);
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = on ? v[r] : 0.f;
    return v;
  }

  // Snapshot (compact, [N_max+1][d] per array) of X, P, Z.
  __device__ void save(float* dst, int N_max) const {
    const int64_t CK = int64_t(N_max + 1) * D;
    if constexpr (kRows)
#pragma unroll
    for (int ri = 0; ri < RPW; ri++) {
      if (!rows_ok(ri)) continue;
      const int i0 = coord(ri);
      if (lr == 0) {
        *reinterpret_cast<f4*>(dst + i0) = x0_of(ri);
        *reinterpret_cast<f4*>(dst + CK + i0) = f4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f4*>(dst + 2 * CK + i0) = z0_of(ri);
      }
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const int j = node(t);
        if (j > Np) continue;
        float* q = dst + j * D + i0;
        *reinterpret_cast<f4*>(q) = X[ri][t];
        *reinterpret_cast<f4*>(q + CK) = P[ri][t];
        *reinterpret_cast<f4*>(q + 2 * CK) = Z[ri][t];
      }
    }
  }

  // Keeps the compiler from starting the next column tile's reads early: the
  // registers they would hold are what is short.
  __device__ __forceinline__ static void fence() { __builtin_amdgcn_sched_barrier(0); }

  // One iteration of the splitting (dual, node 0, primal, extrapolation).  The
  // image of X is current on entry and on return.  With kRes the squared
  // changes are added to rx and rp.
  template <bool kRes>
  __device__ __forceinline__ void iterate(const LtArgs& a, float eps, float& rx, float& rp) {
    const float sigma = a.sigma, tau = a.tau, theta = a.theta;
    // opaque, so that the per-column masks below are compared again in every
    // iteration instead of being held in registers
    int np = __builtin_amdgcn_readfirstlane(Np);
    asm volatile("" : "+s"(np));
    Tiles TH;
    if constexpr (kRows) {
      // ---- dual step: p_j <- (p_j + sigma (z_j - z_{j-1}) + lam (A x_j + eps tanh x_j)) c1 ----
      f4 zl[RPW];  // z of the node before the lane's first
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) zl[ri] = row_prev(Z[ri][NT - 1]) + z0_of(ri);
      sweep(fA, imgX, tailX, X, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
        const float c1t = node(t) <= np ? c1 : 0.f;  // nodes past N keep p = 0
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          const f4 zp = t > 0 ? Z[ri][t > 0 ? t - 1 : 0] : zl[ri];
          f4 tht;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const float th = tanh_fast(X[ri][t][r]);
            tht[r] = th;
            const float pv = P[ri][t][r];
            const float v = pv + sigma * (Z[ri][t][r] - zp[r]);
            const float pn = (v + lam * (acc[ri][r] + eps * th)) * c1t;
            if constexpr (kRes) rp += (pn - pv) * (pn - pv);
            P[ri][t][r] = pn;
          }
          if constexpr (S::kThLds) *reinterpret_cast<f4*>(sTh + 4 * (tid + 64 * S::RT * t)) = tht;
          else TH[ri][t] = tht;
          if constexpr (!S::kReg) put(imgP, tailP, t, P[ri][t]);
        }
      });
      if constexpr (!S::kReg)
        if (lr == 0 && rows_ok(0)) {
          f4 v = P[0][0];
          if constexpr (!S::kAux) v = *reinterpret_cast<const f4*>(sX0 + coord(0)) + tau * v;
          *reinterpret_cast<f4*>(sV + coord(0)) = v;
        }
    }
    // ---- node 0: x_0 <- M (x_0 + tau p_1) --------------------------------------------
    f4 xn0[RPW];
    if constexpr (S::kReg) {
      f4 v0[RPW];
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) v0[ri] = x0[ri] + tau * P[ri][0];
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) xn0[ri] = product_reg(fM, v0, ri);
    } else {
      __syncthreads();
      if constexpr (!S::kAux || KIND == kAuxWave) node0<kRes>(tau, theta, rx);
    }
    // ---- primal step, j = 1..N-1 -------------------------------------------------------
    if constexpr (kRows) {
      f4 pl[RPW];  // p of the node after the lane's last
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) pl[ri] = row_next(P[ri][0]);
      sweep(fAt, imgP, tailP, P, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
        const float tt = node(t) < np ? tau : 0.f;  // x_N and the nodes past it do not move
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          const f4 pn = t < NT - 1 ? P[ri][t < NT - 1 ? t + 1 : t] : pl[ri];
          f4 tht;
          if constexpr (S::kThLds) tht = *reinterpret_cast<const f4*>(sTh + 4 * (tid + 64 * S::RT * t));
          else tht = TH[ri][t];
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const float xv = X[ri][t][r], pv = P[ri][t][r], th = tht[r];
            const float g = acc[ri][r] + eps * ((1.f - th * th) * pv);  // -grad_x H
            const float dx = -tt * ((pv - pn[r]) + delta * g);
            if constexpr (kRes) rx += dx * dx;
            Z[ri][t][r] = xv + (1.f + theta) * dx;
            X[ri][t][r] = xv + dx;
          }
          if constexpr (!S::kReg) put(imgX, tailX, t, X[ri][t]);
        }
      });
    }
    if constexpr (S::kReg) {
#pragma unroll
      for (int ri = 0; ri < RPW; ri++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const float dx = lr == 0 ? xn0[ri][r] - x0[ri][r] : 0.f;
          if constexpr (kRes) rx += dx * dx;
          z0[ri][r] = x0[ri][r] + (1.f + theta) * dx;
          x0[ri][r] += dx;
        }
    } else {
      __syncthreads();
    }
  }

  // Products of every column tile, each handed to f(t, product).
  template <class Fn>
  __device__ __forceinline__ void sweep(const Frag& F, const uint16_t* img, const float* tail, const Tiles& B,
                                        const Fn& f) const {
    if constexpr (S::kReg) {
#pragma unroll
      for (int t = 0; t < NT; t++) {
        f4 acc[RPW], col[RPW];
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) col[ri] = B[ri][t];
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) acc[ri] = product_reg(F.f, col, ri);
        f(t, acc);
        fence();
      }
    } else {
      // A tile's matrix instructions are issued between the instructions of the
      // previous tile's f, one to three: a SIMD runs the two kinds one after the
      // other except for about three vector instructions behind each matrix one.
      f4 acc[1];
#pragma unroll
      for (int t = 0; t <= NT; t++) {
        Pieces p[kAhead];
        if (t < NT)
#pragma unroll
          for (int s = 0; s < kAhead; s++) p[s] = get(img, t, s);
        f4 next = f4{0.f, 0.f, 0.f, 0.f};
        if (t < NT) next = product(F, img, tail, t, p);
        if (t > 0) f(t - 1, acc);
        if (t > 0 && t < NT) {
          __builtin_amdgcn_sched_group_barrier(0x100, 7, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);
#pragma unroll
          for (int i = 0; i < 19; i++) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            if (i == 2) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
          }
        }
        fence();
        acc[0] = next;
      }
    }
  }
};

}  // namespace hjpd
