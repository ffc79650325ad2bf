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

// LDS pointers keep their address space, so that an address is one register
// and a constant part of it an instruction's offset.
typedef __attribute__((address_space(3))) float lds_f;
typedef __attribute__((address_space(3))) f4 lds_f4;
typedef __attribute__((address_space(3))) u2 lds_u2;
typedef __attribute__((address_space(3))) bf8 lds_bf8;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
// Global pointers that pass through an opaque step (and would come out generic).
typedef const __attribute__((address_space(1))) float glb_f;
typedef const __attribute__((address_space(1))) f4 glb_f4;
typedef const __attribute__((address_space(1))) bf8 glb_bf8;
__device__ __forceinline__ f4 ld4(glb_f* p) { return *(glb_f4*)p; }
// A pointer that is the same in every lane, kept in scalar registers.
template <class T>
__device__ __forceinline__ T* scalar(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  uint64_t u = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32)))) << 32) |
               uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v)));
  asm volatile("" : "+s"(u));
  return reinterpret_cast<T*>(u);
}
__device__ __forceinline__ f4 ld4(const float* p) { return *reinterpret_cast<const f4*>(p); }
__device__ __forceinline__ f4 ld4(const lds_f* p) { return *(const lds_f4*)p; }
__device__ __forceinline__ void st4(float* p, f4 v) { *reinterpret_cast<f4*>(p) = v; }
__device__ __forceinline__ void st4(lds_f* p, f4 v) { *(lds_f4*)p = v; }

// The lane's number, formed anew where it is used.
__device__ __forceinline__ uint32_t lane_now() {
  uint32_t v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// base + off as an LDS address that the compiler neither sees through nor
// keeps from one loop to the next: otherwise it holds a register (and soon a
// spill slot) for every constant offset in a loop.
// Only the reverse sweep needs that (the forward kernel's registers suffice,
// and it is 8 % slower with the extra instructions).
template <bool kOpaque, class P>
__device__ __forceinline__ P* at(P* base, uint32_t off) {
  if constexpr (kOpaque) asm volatile("" : "+v"(off));
  P* p = base + off;
  if constexpr (kOpaque) asm volatile("" : "+v"(p));
  return p;
}

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
  const float* Mc;  // (I + tau Q_s)^{-1} as [column / 4][row][4]
  const float* Qs;  // (Q + Q^T) / 2
  const float* packed;  // A, A^T (and M, d <= 32) as operands, LtFrag
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

template <int D, int NT, bool BACK = false>
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
  // An image piece is laid out [k / 8][row][8], the rows of odd chunks taken
  // with bits 2 and 3 flipped (M: [k / 4][row][4]): the 16-byte reads and 8-byte
  // writes of a wave then cover the 64 banks evenly, and so do the transposed
  // reads of the reverse sweep, which take two neighbouring chunks at once.
  // Rows padded to 16 bytes over a power of two lost 2,850 of 6,240 LDS cycles
  // an iteration to conflicts (d = 100, N = 50).
  static constexpr int CH = kReg ? 0 : 4 * KB + 2 * (BACK && kTail);  // chunks; the reverse sweep's outer products take the tail's row tile too
  static constexpr int PIECE = 8 * CH * ROWS;   // bfloat16 per piece
  static constexpr int MR = D;                  // rows of M
  // LDS in floats.  Forward: two images (X, P), their FP32 tails, M, vectors,
  // reduction slots.  Reverse sweep: three images (the third also holds the
  // recompute's tanh), M stays in global memory, and the multipliers' adjoint.
  static constexpr int kImg = kReg ? 0 : 3 * PIECE / 2;
  static constexpr int kImgs = BACK ? 3 : 2;
  static constexpr int kTailF = kTail ? 4 * ROWS : 0;
  static constexpr int kM = kReg || BACK ? 0 : D * MR;
  static constexpr int kVec = 16 * RT, kVecs = BACK ? 8 : 4;
  // tanh(x_j) from the dual step to the primal step, where it fits beside the rest
  static constexpr bool kThLds = !kReg && D < 128;
  static constexpr int kTh = kThLds && !BACK ? 256 * RT * NT : 0;
  static constexpr bool kPbLds = BACK && !kReg && D < 128;
  static constexpr int kPb = kPbLds ? 256 * RT * NT : 0;
  // d <= 32: rows of two operands of an outer product, row length an odd multiple of 16 (conflict-free columns)
  static constexpr int LDW = D == 16 ? 16 : 48;
  static constexpr int kScratch = BACK && kReg ? 2 * ROWS * LDW : 0;
  static constexpr int kLdsFloats = kImgs * kImg + 2 * kTailF + kM + kVecs * kVec + kTh + kPb + kScratch + 2 * W + 2;
};

// A matrix's rows of one wave as A operands, read from a packed copy that the
// set-up kernel makes (every load 1 KB a wave, shared by all workgroups and so
// in L2): the reverse sweep holds one matrix at a time and reads it again in
// every step, where the compiler otherwise kept both through scratch memory,
// which is per workgroup and does not fit L2.
template <int D>
struct LtFrag {
  using S = LtShape<D, 1>;
  static constexpr int kWave = S::kReg ? S::RPW * S::RPW * 256 : 3 * S::KB * 256 + 64;  // floats of one wave's rows
  static constexpr int kMatrix = kWave * (S::kReg ? 1 : S::RT);
  float f[S::kReg ? S::RPW : 1][S::kReg ? 4 * S::RPW : 1];  // FP32 operands (kReg), or the tail's
  bf8 h[S::kReg ? 1 : S::KB], m[S::kReg ? 1 : S::KB], l[S::kReg ? 1 : S::KB];

  // matrix: 0 = A, 1 = A^T, 2 = M (d <= 32).  The opaque address keeps the reads where they are written.
  __device__ __forceinline__ void load(const float* packed, int matrix, int wave, int lane) {
    glb_f* q = (glb_f*)packed + (matrix * kMatrix + wave * kWave);
    asm volatile("" : "+s"(q));
    if constexpr (S::kReg) {
#pragma unroll
      for (int ro = 0; ro < S::RPW; ro++)
#pragma unroll
        for (int e = 0; e < S::RPW; e++) {
          const f4 v = ld4(q + (ro * S::RPW + e) * 256 + lane * 4);
#pragma unroll
          for (int r = 0; r < 4; r++) f[ro][4 * e + r] = v[r];
        }
    } else {
#pragma unroll
      for (int s = 0; s < S::KB; s++) {
        h[s] = *(glb_bf8*)(q + (3 * s + 0) * 256 + lane * 4);
        m[s] = *(glb_bf8*)(q + (3 * s + 1) * 256 + lane * 4);
        l[s] = *(glb_bf8*)(q + (3 * s + 2) * 256 + lane * 4);
      }
      if constexpr (S::kTail) f[0][0] = q[3 * S::KB * 256 + lane];
    }
  }
  // Entry (row, k) of a matrix at its place in the packed copy (one thread per
  // entry, k < D; with d > 32 pairs of entries: call it for even k with both).
  __device__ static void pack(float* packed, int matrix, int row, int k, float u, float v) {
    float* q = packed + matrix * kMatrix;
    const int lr = row % 16;
    if constexpr (S::kReg) {
      q[((row / 16) * S::RPW + k / 16) * 256 + (16 * (k % 16 / 4) + lr) * 4 + k % 4] = u;
    } else {
      q += (row / 16) * kWave;
      if (k < 32 * S::KB) {
        uint32_t hml[3];
        split_pair(u, v, hml[0], hml[1], hml[2]);
        const int lane = 16 * (k % 32 / 8) + lr;
#pragma unroll
        for (int c = 0; c < 3; c++)
          reinterpret_cast<uint32_t*>(q)[(3 * (k / 32) + c) * 256 + lane * 4 + k % 8 / 2] = hml[c];
      } else {
        q[3 * S::KB * 256 + 16 * (k - 32 * S::KB) + lr] = u;
        q[3 * S::KB * 256 + 16 * (k + 1 - 32 * S::KB) + lr] = v;
      }
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
template <int D, int NT, int KIND, bool BACK = false>
struct LtCore {
  using S = LtShape<D, NT, BACK>;
  using Frag = LtFrag<D>;
  static constexpr int RPW = S::RPW;
  static constexpr bool kRows = KIND != kAuxWave;
  typedef f4 Tiles[RPW][NT];

  int tid, wave, lr, lk;
  // LDS (d > 32): bfloat16 images of X and P, their tails, M, a vector, reduction slots
  lds_u16 *imgX, *imgP, *img3;
  lds_f *tailX, *tailP, *sTh, *sPb, *sScr;
  std::conditional_t<BACK, glb_f*, const lds_f*> Mc;         // M in chunks of four columns, in LDS or (reverse sweep) in global memory
  lds_f *sX0, *sZ0, *sV, *sW;  // x_0, z_0, p_1 (also scratch), x_0 + tau p_1
  lds_f *sXb0, *sZb0, *sE, *sWb;  // reverse sweep: node 0's adjoints, XB_0 and M XB_0
  lds_f* sRed;
  uint32_t put_at, get_at;  // this lane's element offsets into an image
  Frag fA, fAt;
  Frag fM;  // d <= 32

  // state of the current point
  Tiles X, P, Z;
  f4 x0[RPW], z0[RPW];  // d <= 32; otherwise node 0 is in LDS
  int Np;
  float delta, lam, c1;

  __device__ int coord(int ri) const { return 16 * (S::kReg ? ri : wave) + 4 * lk; }  // of element r = 0
  __device__ int coord_now() const { return 16 * wave + 4 * (BACK ? int(lane_now() >> 4) : lk); }  // the same, d > 32
  __device__ int node(int t) const { return NT * lr + t + 1; }
  __device__ int node_now() const { return NT * (BACK ? int(lane_now() & 15) : lr) + 1; }           // node(0)
  __device__ bool rows_ok(int ri) const { return S::kReg || D % 16 == 0 || coord(ri) < D; }

  __device__ void setup(const LtArgs& a, float* shared) {
    lds_f* lds = (lds_f*)shared;
    tid = threadIdx.x;
    wave = S::W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    lr = tid & 15;
    lk = (tid & 63) >> 4;
    if constexpr (kRows && !BACK) load_matrices(a);
    imgX = (lds_u16*)lds;
    imgP = (lds_u16*)(lds + S::kImg);
    img3 = (lds_u16*)(lds + 2 * S::kImg);
    tailX = lds + S::kImgs * S::kImg;
    tailP = tailX + S::kTailF;
    lds_f* sM = tailP + S::kTailF;
    sTh = BACK ? lds + 2 * S::kImg : sM + S::kM;
    sPb = sM + S::kM + S::kTh;
    sScr = sPb + S::kPb;
    sX0 = sScr + S::kScratch;
    sZ0 = sX0 + S::kVec;
    sV = sZ0 + S::kVec;
    sW = sV + S::kVec;
    sXb0 = sW + S::kVec;
    sZb0 = sXb0 + S::kVec;
    sE = sZb0 + S::kVec;
    sWb = sE + S::kVec;
    sRed = sX0 + S::kVecs * S::kVec;
    put_at = ((2 * wave + (lk >> 1)) * S::ROWS + (lr ^ (lk & 2 ? 12 : 0))) * 8 + (lk & 1) * 4;
    get_at = (lk * S::ROWS + (lr ^ (lk & 1 ? 12 : 0))) * 8;
    if constexpr (BACK) Mc = (glb_f*)a.Mc;
    if constexpr (!S::kReg) {
      if constexpr (!BACK) {
        for (int e = tid; e < D * S::MR; e += S::kThreads) sM[e] = a.Mc[e];
        Mc = sM;
      }
      for (int e = tid; e < S::kVecs * S::kVec; e += S::kThreads) sX0[e] = 0.f;  // entries past d stay zero
      __syncthreads();
    }
  }

  __device__ __forceinline__ void load_matrices(const LtArgs& a) {
    fA.load(a.packed, 0, wave, tid & 63);
    fAt.load(a.packed, 1, wave, tid & 63);
    if constexpr (S::kReg) fM.load(a.packed, 2, wave, tid & 63);
  }

  // This wave's rows of column tile t into an image (the tail wave: into the FP32 tail).
  __device__ __forceinline__ void put(lds_u16* img, lds_f* tail, int t, f4 v) const {
    if (KIND == kRowWave || BACK) {  // (rows past d are zero)
      u2 h, m, l;
      uint32_t a0, a1, b0, b1, g0, g1;
      split_pair(v[0], v[1], a0, b0, g0);
      split_pair(v[2], v[3], a1, b1, g1);
      h = u2{a0, a1};
      m = u2{b0, b1};
      l = u2{g0, g1};
      lds_u16* q = at<BACK>(img, put_at) + t * 16 * 8;
      *(lds_u2*)q = h;
      *(lds_u2*)(q + S::PIECE) = m;
      *(lds_u2*)(q + 2 * S::PIECE) = l;
    }
    if (KIND == kTailWave && lk == 0 && tail) st4(at<BACK>(tail, lr * 4) + 64 * t, v);
  }

  // Rows of this wave of (matrix) x (column tile t of the image): the small
  // products and the h h products summed apart.  `p` holds the pieces of the
  // first k-steps, read ahead.
  struct Pieces { bf8 h, m, l; };
  static constexpr int kAhead = BACK ? 1 : 2;  // k-steps read ahead (the reverse sweep has fewer registers to spare)
  // (img, tail: with this lane's offset)
  __device__ __forceinline__ Pieces get(const lds_u16* img, int t, int s) const {
    const lds_u16* q = img + t * 16 * 8 + s * 32 * S::ROWS;
    return {*(const lds_bf8*)q, *(const lds_bf8*)(q + S::PIECE), *(const lds_bf8*)(q + 2 * S::PIECE)};
  }
  __device__ __forceinline__ f4 product(const Frag& F, const lds_u16* img, const lds_f* tail, int t,
                                        const Pieces (&p)[kAhead]) const {
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (!S::kReg) {
      Pieces rest[S::KB - kAhead];
#pragma unroll
      for (int s = kAhead; s < S::KB; s++) rest[s - kAhead] = get(img, t, s);
      float last = 0.f;
      if constexpr (S::kTail) last = tail[64 * t];
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
  __device__ __forceinline__ f4 product_reg(const Frag& F, const f4 (&B)[RPW], int ro) const {
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (S::kReg) {
#pragma unroll
      for (int q = 0; q < 4 * RPW; q++) acc = mfma4(F.f[ro][q], B[q / 4][q % 4], acc);
    }
    return acc;
  }
  // Node 0 with d > 32: x_0 <- M (x_0 + tau p_1) from p_1 in sV, z_0 with it.
  // d = 100 leaves an eighth wave without rows: it takes the whole product, two
  // outputs to a lane, while the others run the primal product (the row waves
  // would each spend 60 instructions and two cross-lane sums on it, and hold
  // 56 registers).  d = 128: lane (lr, lk) of a row wave sums the terms
  // k = 4 lk .. 4 lk + 3 (mod 16) of row lr.
  // M times the vector w in LDS (entries past d zero), each entry i handed to
  // out(i, value) by the lane that has it.
  template <class Out>
  __device__ __forceinline__ void gemv(const lds_f* w, const Out& out) const {
    if constexpr (S::kAux) {
      const int i = tid & 63, i2 = 64 + i < D ? 64 + i : D - 1;
      float u = 0.f, v = 0.f;
      auto m = Mc;  // opaque: the addresses of the unrolled reads are not kept
      if constexpr (BACK) asm volatile("" : "+s"(m));
#pragma unroll(BACK ? 25 : 5)  // from global memory: all reads in flight together
      for (int k = 0; k < D; k += 4) {
        const f4 x = ld4(w + k);
        const f4 a = ld4(m + k * S::MR + 4 * i);
        const f4 b = ld4(m + k * S::MR + 4 * i2);
#pragma unroll
        for (int r = 0; r < 4; r++) {
          u += a[r] * x[r];
          v += b[r] * x[r];
        }
      }
      out(i, u);
      if (64 + i < D) out(64 + i, v);
    } else {
      float part = 0.f;
#pragma unroll 2
      for (int k = 4 * lk; k < D; k += 16) {
        const f4 mm = ld4(Mc + k * S::MR + 4 * (16 * wave + lr));
        const f4 x = ld4(w + k);
#pragma unroll
        for (int r = 0; r < 4; r++) part += mm[r] * x[r];
      }
      part += __shfl_xor(part, 16, 64);
      part += __shfl_xor(part, 32, 64);
      if (lk == 0) out(16 * wave + lr, part);
    }
  }
  template <bool kRes>
  __device__ __forceinline__ void node0(float tau, float theta, float& rx) const {
    if constexpr (S::kAux) {
      const int i = tid & 63;
      sW[i] = sX0[i] + tau * sV[i];
      if (64 + i < D) sW[64 + i] = sX0[64 + i] + tau * sV[64 + i];
      __builtin_amdgcn_wave_barrier();
    }
    gemv(S::kAux ? sW : sV, [&](int i, float xn) {
      const float xo = sX0[i], dx = xn - xo;
      if constexpr (kRes) rx += dx * dx;
      sX0[i] = xn;
      sZ0[i] = xn + theta * dx;
    });
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
  __device__ __forceinline__ void put_all(lds_u16* img, lds_f* tail, const Tiles& V) const {
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
    else return first_col(ld4(sX0 + coord_now()));
  }
  __device__ __forceinline__ f4 z0_of(int ri) const {
    if constexpr (S::kReg) return z0[ri];
    else return first_col(ld4(sZ0 + coord_now()));
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
        st4(dst + i0, x0_of(ri));
        st4(dst + CK + i0, f4{0.f, 0.f, 0.f, 0.f});
        st4(dst + 2 * CK + i0, z0_of(ri));
      }
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const int j = node(t);
        if (j > Np) continue;
        float* q = dst + j * D + i0;
        st4(q, X[ri][t]);
        st4(q + CK, P[ri][t]);
        st4(q + 2 * CK, Z[ri][t]);
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
    const int n0 = node_now();
    if constexpr (kRows) {
      // ---- dual step: p_j <- (p_j + sigma (z_j - z_{j-1}) + lam (A x_j + eps tanh x_j)) c1 ----
      f4 zl[RPW];  // z of the node before the lane's first
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) zl[ri] = row_prev(Z[ri][NT - 1]) + z0_of(ri);
      sweep(fA, imgX, tailX, X, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
        const float c1t = n0 + t <= np ? c1 : 0.f;  // nodes past N keep p = 0
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
          if constexpr (S::kThLds) st4(at<BACK>(sTh, 4 * tid) + 256 * S::RT * t, tht);
          else TH[ri][t] = tht;
          if constexpr (!S::kReg) put(imgP, tailP, t, P[ri][t]);
        }
      });
      if constexpr (!S::kReg)
        if (lr == 0 && rows_ok(0)) {
          f4 v = P[0][0];
          const int i = coord_now();
          if constexpr (!S::kAux) v = ld4(sX0 + i) + tau * v;
          st4(sV + i, v);
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
        const float tt = n0 + t < np ? tau : 0.f;  // x_N and the nodes past it do not move
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          const f4 pn = t < NT - 1 ? P[ri][t < NT - 1 ? t + 1 : t] : pl[ri];
          f4 tht;
          if constexpr (S::kThLds) tht = ld4(at<BACK>(sTh, 4 * tid) + 256 * S::RT * t);
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
  __device__ __forceinline__ void sweep(const Frag& F, const lds_u16* img, const lds_f* tail, const Tiles& B,
                                        const Fn& f) const {
    if constexpr (S::kReg) {
#pragma unroll
      for (int t = 0; t < NT; t++) {
        f4 acc[RPW], col[RPW];
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) col[ri] = B[ri][t];
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) acc[ri] = product_reg(F, col, ri);
        f(t, acc);
        fence();
      }
    } else {
      // A tile's matrix instructions are issued between the instructions of the
      // previous tile's f, one to three: a SIMD runs the two kinds one after the
      // other except for about three vector instructions behind each matrix one.
      img = at<BACK>(img, get_at);
      if constexpr (S::kTail) tail = at<BACK>(tail, 4 * lr + lk);
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
          __builtin_amdgcn_sched_group_barrier(0x100, 3 * kAhead + 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);
#pragma unroll
          for (int i = 0; i < 19; i++) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            if (i == 2 || (BACK && i == 8)) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
          }
        }
        fence();
        acc[0] = next;
      }
    }
  }
};

}  // namespace hjpd
