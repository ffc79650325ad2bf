// Reverse sweep of the linear-tanh family (k_lt_backward), on the register
// layout of hjpd_lt_core.hpp.
//
// Per point the kernel goes through the segments of E iterations from the last
// to the first: it recomputes a segment forward from its checkpoint, keeping
// x^k and p^{k+1} of every step in a buffer of its workgroup, and then applies
// the transposed Jacobian of each iteration (x', p', z' adjoints XB, PB, ZB):
//   z' = x' + theta (x' - x)        XB += (1+theta) ZB;  Xpre = -theta ZB   (z'_N = x_N: Xpre_N = ZB_N + XB_N)
//   x'_0 = M w, w = x_0 + tau p'_1  wbar = M XB_0;  Xpre_0 += wbar;  PB_1 += tau wbar;  dM += XB_0 w^T
//   x'_j = x_j - tau (p'_j - p'_{j+1}) - tau delta (A^T p'_j + eps (1 - th_j^2) p'_j),  j < N:
//        Xpre_j += XB_j + 2 tau delta eps (1 - th_j^2) th_j p'_j XB_j
//        PB_j += -tau XB_j - tau delta (A XB)_j - tau delta eps (1 - th_j^2) XB_j + tau XB_{j-1}
//        dA += -tau delta p'_j XB_j^T;  deps += -tau delta sum (1 - th^2) p' XB
//   p'_j = c1 (p_j + sigma (z_j - z_{j-1}) + lam (A x_j + eps th_j)):
//        vbar = c1 PB;  Ppre = vbar;  Zpre_j = sigma (vbar_j - vbar_{j+1})
//        Xpre_j += lam (A^T vbar)_j + lam eps (1 - th_j^2) vbar_j;  dA += lam vbar_j x_j^T;  deps += lam th vbar
//
// x_N does not move, so its adjoint, most of dphi/dx, only ever grows, by terms
// far smaller than itself.  At node N those terms are gathered in the z adjoint
// first (which the next step adds to the x adjoint whole), so each step rounds
// once at the size of the sum: dphi/dx is 2.7e-7 (rms) from 64 bits after 100
// iterations at d = 32, where adding the terms one by one left 5.7e-7.
//
// XB and ZB stay in registers.  d > 32: a step has two barriers.  Between them
// the waves read the images of XB and of their own rows of -tau delta p' (A XB,
// the outer product p' XB^T) and write those of vbar and lam x; after the
// second they read the latter (A^T vbar, the outer product vbar x^T).  The
// outer products contract over the nodes, along the rows of an image, and read
// it with the transposing LDS loads (ds_read_b64_tr_b16) that gfx950 has for
// this; both add into the same accumulators, row tile by all columns.  Node 0's
// product M XB_0 of a step is formed during the second half of the step before
// (its XB_0 is known there), by the wave without rows at d = 100.
//
// Why this form: what bounds a step is the instruction issue of a SIMD's two
// waves, matrix instructions and vector ones nearly one after the other
// (7,900 cycles of the former and 1,700 instructions of the latter a row wave,
// 36,400 cycles a step and point at d = 100, N = 50; LDS 12,500).  So products
// run on bfloat16 pieces (six matrix instructions where FP32 ones need eight
// of twice the length), nothing is read back for elementwise work, and a wave
// holds one matrix at a time.  d <= 32: products straight from the state
// registers on FP32 matrix instructions, outer products by way of LDS rows of
// one wave, no barrier.  Before, products on FP32 matrix instructions from
// staged rows with the state in LDS: 2,048 points x 500 iterations at d = 100
// took 128 ms, now 68 ms; d = 128 (512 points, N = 40, 100 iterations) 7.7, now
// 4.4 ms; d = 32 (777 points, N = 24, 200 iterations) 8.4, now 1.4 ms.  Errors from
// 64 bits (rms) at the first, before and now: dphi/dx 2.2e-6, 1.5e-6; deps and dA
// together 8.3e-6, 0.8e-7; dQ 2.4e-7, 0.8e-7.
#pragma once

#include "hjpd_lt_core.hpp"

namespace hjpd {

typedef short sh4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) sh4 lds_sh4;

struct LtBwdArgs {
  LtArgs f;
  const float* grad_phi;  // [n]
  float* dphi_dx;         // [n][d]
  float* seg;             // per workgroup: E steps of (x^k, p^{k+1}), the saved adjoint, E pairs (XB_0, w)
  float* part;            // per workgroup: dA (d*d), dM (d*d), dQ direct (d*d), deps (1)
  int K;
};

// Floats of one array (x^k or p^{k+1}, all row and column tiles) of a workgroup's buffer.
constexpr int64_t lt_tiles(int d, int N_max) { return 256 * int64_t((d + 15) / 16) * ((N_max + 15) / 16); }
constexpr int64_t lt_seg_floats(int d, int N_max, int E) {
  return int64_t(E) * 2 * lt_tiles(d, N_max) + 2 * lt_tiles(d, N_max) + int64_t(E) * 2 * d;
}

template <int D, int NT, int KIND>
struct LtBack : LtCore<D, NT, KIND, true> {
  using Core = LtCore<D, NT, KIND, true>;
  using S = typename Core::S;
  using Tiles = typename Core::Tiles;
  using Core::lr, Core::lk, Core::tid, Core::wave, Core::Np, Core::delta, Core::lam, Core::c1;
  static constexpr int RPW = S::RPW, RT = S::RT, KS = NT / 2;
  static constexpr bool kHalf = NT % 2, kRows = Core::kRows;

  // Adjoints between steps: of z in XB, of x in ZB (a step turns one into the
  // other), of p (vbar of the step before) in PB, or in LDS where kPbLds.
  Tiles XB, ZB, PB;
  f4 dA[RPW][RT];
  f4 dM[S::kReg ? RPW : 1][S::kReg ? RT : 1];
  float deps;  // in units of 2^e_all
  // The adjoints are linear in the point's output weight w.  bfloat16 pieces lose
  // their low bits below about 2^-110 (w = 1e-35: dphi/dx 3e-7 -> 5e-6 from 64 bits),
  // so the sweep runs with w 2^-e_w in [1/2, 1), dA's and deps' terms are taken
  // relative to 2^e_all, the largest w delta of the workgroup's points, and dM's
  // relative to 2^e_dM, the largest w.  All are powers of two: the same bits.
  int e_w, e_all, e_dM;
  float ds;  // delta 2^(e_w - e_all)
  uint32_t tr0, tr1, tr2;  // transposed-read offsets: nodes 8 lk, 8 lk + 4, 4 lk

  __device__ void setup_back(const LtArgs& a, float* lds) {
    this->setup(a, lds);
    const int par = (lr & 3) >> 1, half = (lr & 1) * 4, n = lr >> 2, sw = par ? 12 : 0;
    auto at = [&](int node) { return uint32_t((par * S::ROWS + (node ^ sw)) * 8 + half); };
    tr0 = at(8 * (lk & 1) + n) + (lk >> 1) * 16 * 8;
    tr1 = at(8 * (lk & 1) + 4 + n) + (lk >> 1) * 16 * 8;
    tr2 = at(4 * lk + n);
    deps = 0.f;
    e_w = e_all = e_dM = 0;
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int ct = 0; ct < RT; ct++) dA[ri][ct] = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (S::kReg)
#pragma unroll
      for (int ri = 0; ri < RPW; ri++)
#pragma unroll
        for (int ct = 0; ct < RT; ct++) dM[ri][ct] = f4{0.f, 0.f, 0.f, 0.f};
  }

  // e_all and e_dM of the points first, first + step, ... (every wave for itself)
  __device__ void scale_of_all(const LtBwdArgs& b, int64_t first, int64_t step) {
    constexpr int kNone = -1024;
    int e = kNone, em = kNone;
    for (int64_t pt = first + (tid & 63) * step; pt < b.f.n; pt += 64 * step) {
      const float w = b.grad_phi[pt], t = b.f.t[pt];
      const int N = b.f.N[pt];
      if (w != 0.f && __builtin_isfinite(w) && t > 0.f && __builtin_isfinite(t) && N >= 1 && N <= b.f.N_max) {
        const int ew = __builtin_amdgcn_frexp_expf(w);
        em = max(em, ew);
        e = max(e, ew + __builtin_amdgcn_frexp_expf(t / float(N)));
      }
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      e = max(e, __shfl_xor(e, m, 64));
      em = max(em, __shfl_xor(em, m, 64));
    }
    e_all = __builtin_amdgcn_readfirstlane(e == kNone ? 0 : e);
    e_dM = __builtin_amdgcn_readfirstlane(em == kNone ? 0 : em);
  }
  // Takes the point's scales from its weight (after set_point) and returns the weight to sweep with.
  __device__ float scale_of_point(float w) {
    e_w = __builtin_amdgcn_readfirstlane(__builtin_isfinite(w) ? __builtin_amdgcn_frexp_expf(w) : 0);
    ds = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(ldexpf(delta, e_w - e_all))));
    return ldexpf(w, -e_w);
  }
  // An entry of XB_0 as dM takes it.
  __device__ __forceinline__ float for_dM(float v) const { return ldexpf(v, e_w - e_dM); }

  // ---- outer products over the nodes (d > 32) -------------------------------------------
  // One row tile of an image as an operand: coordinate lr, the nodes along k.
  // Step s covers nodes 32 s .. 32 s + 31 (the last one of an odd tile count, 16 of them, in q).
  struct Op { bf8 p[3]; sh4 q[3]; };  // pieces h, m, l
  struct At { const lds_u16 *a, *b, *c; };  // an image with this lane's offsets
  __device__ __forceinline__ At at_of(const lds_u16* img) const {
    At q;
    if constexpr (KS > 0) {
      q.a = at<true>(img, tr0);
      q.b = at<true>(img, tr1);
    }
    if constexpr (kHalf) q.c = at<true>(img, tr2);
    return q;
  }
  __device__ __forceinline__ void read_op(Op& o, const At& q, int ct, int s) const {
    const int off = 2 * ct * S::ROWS * 8 + s * 32 * 8;
    if (s < KS) {
#pragma unroll
      for (int c = 0; c < 3; c++) {
        const sh4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sh4*)(q.a + off + c * S::PIECE));
        const sh4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sh4*)(q.b + off + c * S::PIECE));
        o.p[c] = __builtin_bit_cast(bf8, __builtin_shufflevector(u, v, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    } else {
#pragma unroll
      for (int c = 0; c < 3; c++)
        o.q[c] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sh4*)(q.c + off + c * S::PIECE));
    }
  }
  // dA += (this wave's rows of U) (all columns of V)^T, by six piece products.
  // Added straight to dA, each of them rounds at dA's size, and not evenly: over
  // all steps and points that left dA up to 3.4 times further from 64 bits than
  // FP32 products do.  With up to two column tiles the six are summed apart;
  // with more there are no registers for that (42 % slower at N = 50), and dA is
  // added to the partial sums in memory and cleared every kFlush steps.
  // rms error of dA at d = 100 with FP32 products, straight, and so: 9.0e-7, 2.4e-6,
  // 1.8e-7 (1,442 points, N 19 to 25, 90 iterations); 1.4e-6, 4.6e-6, 5.9e-7 (700
  // points, N = 50, 100 iterations).
  static constexpr bool kApart = NT <= 2;
  static constexpr int kFlush = S::kReg || kApart ? 1 << 30 : 16;
  __device__ __forceinline__ void outer(const lds_u16* U, const lds_u16* V) {
    // this wave's rows: its own row tile
    const At au = at_of(U + 2 * wave * S::ROWS * 8), av = at_of(V);
#pragma unroll
    for (int s = 0; s < KS + kHalf; s++) {
      Op a;
      read_op(a, au, 0, s);
      Op b;
      read_op(b, av, 0, s);
#pragma unroll
      for (int ct = 0; ct < RT; ct++) {
        Op next;  // the next tile's reads, under this tile's products
        if (ct + 1 < RT) read_op(next, av, ct + 1, s);
        this->fence();
        f4 v = kApart ? f4{0.f, 0.f, 0.f, 0.f} : dA[0][ct];
        // piece pairs (a, b), small products first
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; q++) {
          if (s < KS) v = mfma32(a.p[pa[q]], b.p[pb[q]], v);
          else v = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.q[pa[q]], b.q[pb[q]], v, 0, 0, 0);
        }
        if (kApart) dA[0][ct] += v;
        else dA[0][ct] = v;
        if (ct + 1 < RT) b = next;
      }
    }
  }
  // d <= 32: the operands' rows go through LDS in FP32 (which = 0, 1).
  __device__ __forceinline__ void scratch_put(int which, int ri, int t, f4 v) const {
    st4(at<true>(this->sScr, lr * S::LDW + 4 * lk) + (which * S::ROWS + 16 * t) * S::LDW + 16 * ri, v);
  }
  __device__ __forceinline__ void outer_scratch() {
    if constexpr (S::kReg) {
      const lds_f *su = at<true>(this->sScr, lk * S::LDW + lr), *sv = su + S::ROWS * S::LDW;
#pragma unroll
      for (int s = 0; s < 4 * NT; s++) {
        float u[RPW], v[RT];
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          u[ri] = su[4 * s * S::LDW + 16 * ri];
          v[ri] = sv[4 * s * S::LDW + 16 * ri];
        }
#pragma unroll
        for (int ri = 0; ri < RPW; ri++)
#pragma unroll
          for (int ct = 0; ct < RT; ct++) dA[ri][ct] = mfma4(u[ri], v[ct], dA[ri][ct]);
        if (s % 4 == 3) this->fence();
      }
    }
  }

  // ---- buffers --------------------------------------------------------------------------
  // Every lane stores and loads (zeros past N): a mask would be a branch around
  // each.  Addresses are a scalar base and the lane's offset.
  __device__ __forceinline__ uint32_t lane_at() const { return lane_now() * 4; }
  __device__ __forceinline__ int tile_at(int ri, int t) const { return ((S::kReg ? ri : wave) * NT + t) * 256; }
  __device__ __forceinline__ void store_tiles(float* q, const Tiles& V) const {
    q = scalar(q);
    const uint32_t o = lane_at();
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int t = 0; t < NT; t++)
        *(__attribute__((address_space(1))) f4*)((__attribute__((address_space(1))) float*)(q + tile_at(ri, t)) + o) = V[ri][t];
  }
  __device__ __forceinline__ f4 load_tile(const float* q, int ri, int t) const {
    return ld4((glb_f*)scalar(q + tile_at(ri, t)) + lane_at());
  }
  __device__ __forceinline__ void load_tiles(const float* q, Tiles& V) const {
    q = scalar(q);
    const uint32_t o = lane_at();
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int t = 0; t < NT; t++) V[ri][t] = ld4((glb_f*)(q + tile_at(ri, t)) + o);
  }
  // One load a lane that covers the 128-byte lines of this wave's x^k: the
  // step's own loads then find them in L2, a tile ahead of their use.  The
  // caller consumes the value late.
  __device__ __forceinline__ float touch(const float* q) const {
    const uint32_t o = min(lane_now(), uint32_t(8 * NT * RPW - 1)) * 32;
    return ((glb_f*)scalar(q + (S::kReg ? 0 : wave) * NT * 256))[o];
  }
  // A snapshot's arrays ([N_max+1][d] each); node 0 to LDS or registers.
  __device__ void load_nodes(const float* src, Tiles& V) const {
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int t = 0; t < NT; t++) {
        V[ri][t] = f4{0.f, 0.f, 0.f, 0.f};
        if (this->node(t) <= Np && this->rows_ok(ri))
          V[ri][t] = ld4(src + this->node(t) * D + this->coord(ri));
      }
  }
  __device__ void load_snapshot(const float* src, int N_max) {
    const int64_t CK = int64_t(N_max + 1) * D;
    if constexpr (kRows) {
      load_nodes(src, this->X);
      load_nodes(src + CK, this->P);
      load_nodes(src + 2 * CK, this->Z);
    }
    if constexpr (S::kReg) {
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) {
        this->x0[ri] = this->z0[ri] = f4{0.f, 0.f, 0.f, 0.f};
        if (lr == 0) {
          this->x0[ri] = ld4(src + this->coord(ri));
          this->z0[ri] = ld4(src + 2 * CK + this->coord(ri));
        }
      }
    } else {
      for (int i = tid; i < D; i += S::kThreads) {
        this->sX0[i] = src[i];
        this->sZ0[i] = src[2 * CK + i];
      }
    }
  }

  // ---- node 0 (d > 32) --------------------------------------------------------------------
  // Entry i of node 0's adjoints after a step with vbar_1 = vb, and XB_0 of the
  // next step (sE); this step's XB_0 goes to st for dM.
  __device__ __forceinline__ void node0_entry(int i, float vb, float sigma, float theta, float* st) const {
    st[i] = for_dM(this->sE[i]);
    const float xb = -theta * this->sZb0[i] + this->sWb[i], zb = -sigma * vb;
    this->sXb0[i] = xb;
    this->sZb0[i] = zb;
    this->sE[i] = xb + (1.f + theta) * zb;
  }
  __device__ __forceinline__ void node0_product() const {
    this->gemv(this->sE, [&](int j, float v) { this->sWb[j] = v; });
  }

  // ---- one step of the sweep ----------------------------------------------------------------
  // st: this step's pair (XB_0, w) for dM; cur: its (x^k, p^{k+1}), prev: the
  // next step's, or null; pk: p^{k+1}, read ahead.  s1, s2 collect sum (1 - th^2) p' XB and sum th vbar.
  __device__ __forceinline__ void step(const LtArgs& a, float eps, float* st, float* cur, float* prev, Tiles& pk,
                                       float& touched, f4 (&xb0)[RPW], f4 (&zb0)[RPW], float& s1, float& s2) {
    const float sigma = a.sigma, tau = a.tau, theta = a.theta, td = tau * delta;
    const float td_s = tau * ds, lam_s = sigma * ds;  // for the outer products
    int np = __builtin_amdgcn_readfirstlane(Np);
    asm volatile("" : "+s"(np));
    const int n0 = this->node_now();
    // (A) extrapolation transposed: XB_j (zero at j = N, where x is fixed), and
    // Xpre_j's XB_j - theta ZB_j = x' + z' in one rounding
    asm volatile("" ::"v"(touched));
    if constexpr (kRows)
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const bool mid = n0 + t < np;
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const float xb = ZB[ri][t][r], zb = XB[ri][t][r];
            XB[ri][t][r] = mid ? xb + (1.f + theta) * zb : 0.f;
            ZB[ri][t][r] = xb + zb;
          }
          if constexpr (S::kReg) scratch_put(1, ri, t, XB[ri][t]);
          else this->put(this->imgX, this->tailX, t, XB[ri][t]);
        }
      }
    if constexpr (!S::kReg) __syncthreads();
    // (B) dA += -tau delta p' XB^T; primal and dual step transposed
    f4 wb[RPW], xn[RPW], pn[RPW];
    if constexpr (kRows)
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) {
        xn[ri] = load_tile(cur, ri, 0);
        pn[ri] = load_tile(cur + tiles_floats(), ri, 0);
      }
    typename Core::Frag fr;  // the matrix in use
    const int lane = tid & 63;
    if constexpr (S::kReg) {
      fr.load(a.packed, 2, 0, lane);
      f4 e[RPW];
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) e[ri] = xb0[ri] + (1.f + theta) * zb0[ri];
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) {
        const f4 v = this->product_reg(fr, e, ri);
        if (lr == 0) st4(st + this->coord(ri), f4{for_dM(e[ri][0]), for_dM(e[ri][1]), for_dM(e[ri][2]), for_dM(e[ri][3])});
#pragma unroll
        for (int r = 0; r < 4; r++) wb[ri][r] = lr == 0 ? v[r] : 0.f;
        xb0[ri] = wb[ri] - theta * zb0[ri];
      }
#pragma unroll
      for (int ri = 0; ri < RPW; ri++)
#pragma unroll
        for (int t = 0; t < NT; t++) scratch_put(0, ri, t, -td_s * pk[ri][t]);
      outer_scratch();
      fr.load(a.packed, 0, 0, lane);
    } else if constexpr (kRows) {
#pragma unroll
      for (int t = 0; t < NT; t++) this->put(this->img3, nullptr, t, -td_s * pk[0][t]);
      fr.load(a.packed, 0, wave, lane);  // arrives during the outer product
      this->fence();
      outer(this->img3, this->imgX);
      this->fence();
      wb[0] = this->first_col(ld4(this->sWb + this->coord_now()));
    }
    if constexpr (kRows) {
      f4 xbm[RPW], vfirst[RPW], vlast[RPW], end[RPW];
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) xbm[ri] = row_prev(XB[ri][NT - 1]) + wb[ri];
      this->sweep(fr, this->imgX, this->tailX, XB, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
        const bool last = n0 + t == np;
        const float le = last ? 0.f : lam * eps, le_end = last ? lam * eps : 0.f;
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          const f4 xk = xn[ri], pt = pn[ri];
          if (t + 1 < NT) {  // the next tile's, a tile ahead
            xn[ri] = load_tile(cur, ri, t + 1);
            pn[ri] = load_tile(cur + tiles_floats(), ri, t + 1);
          }
          f4 pb;
          if constexpr (S::kPbLds) pb = ld4(at<true>(this->sPb, 4 * tid) + 256 * RT * t);
          else pb = PB[ri][t];
          f4 vb, ve;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const float xb = XB[ri][t][r], pp = pt[r], th = tanh_fast(xk[r]);
            const float om = 1.f - th * th, q = om * xb, s = pp * q;
            const float v = (pb[r] + (tau * (xbm[ri][r] - xb) - td * (acc[ri][r] + eps * q))) * c1;
            vb[r] = v;
            ZB[ri][t][r] += (2.f * td * eps) * (th * s) + le * (om * v);
            ve[r] = le_end * (om * v);
            s1 += s;
            s2 += th * v;
          }
          xbm[ri] = XB[ri][t];
          if (t > 0) XB[ri][t > 0 ? t - 1 : 0] = sigma * (vlast[ri] - vb) + end[ri];
          else vfirst[ri] = vb;
          vlast[ri] = vb;
          end[ri] = ve;
          if constexpr (S::kPbLds) st4(at<true>(this->sPb, 4 * tid) + 256 * RT * t, vb);
          else PB[ri][t] = vb;
          if constexpr (S::kReg) {
            scratch_put(0, ri, t, vb);
            scratch_put(1, ri, t, lam_s * xk);
          } else {
            this->put(this->imgP, this->tailP, t, vb);
            this->put(this->img3, nullptr, t, lam_s * xk);
          }
        }
      });
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) {
        XB[ri][NT - 1] = sigma * (vlast[ri] - row_next(vfirst[ri])) + end[ri];
        if constexpr (S::kReg) {
#pragma unroll
          for (int r = 0; r < 4; r++) zb0[ri][r] = lr == 0 ? -sigma * vfirst[ri][r] : 0.f;
        } else if (lr == 0 && this->rows_ok(0)) {
          if constexpr (S::kAux) st4(this->sV + this->coord_now(), vfirst[0]);
          else
#pragma unroll
            for (int r = 0; r < 4; r++) node0_entry(this->coord(0) + r, vfirst[0][r], sigma, theta, st);
        }
      }
    }
    if constexpr (!S::kReg) __syncthreads();
    // (C) A^T vbar; dA += lam vbar x^T; node 0 of the next step
    if constexpr (S::kAux && KIND == kAuxWave) {
      const int i = tid & 63;
      node0_entry(i, this->sV[i], sigma, theta, st);
      if (64 + i < D) node0_entry(64 + i, this->sV[64 + i], sigma, theta, st);
      __builtin_amdgcn_wave_barrier();
      node0_product();
    } else if constexpr (kRows) {
      // the matrix first: a wave waits for its loads in order, and the next
      // step's tiles come from memory
      fr.load(a.packed, 1, wave, lane);
      this->fence();
      if (prev) {
        load_tiles(prev + tiles_floats(), pk);
        touched = touch(prev);
      }
      if constexpr (!S::kReg && !S::kAux) node0_product();
      this->fence();
      if constexpr (S::kReg) outer_scratch();
      else outer(this->imgP, this->img3);
      this->fence();
      this->sweep(fr, this->imgP, this->tailP, PB, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
        const bool last = n0 + t == np;
        const float la = last ? 0.f : lam, la_end = last ? lam : 0.f;
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          ZB[ri][t] += la * acc[ri];
          XB[ri][t] += la_end * acc[ri];
        }
      });
    }
  }
  static constexpr int64_t tiles_floats() { return 256 * int64_t(RT) * NT; }
};

}  // namespace hjpd
