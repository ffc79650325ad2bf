// Linear-tanh family with quadratic initial cost, dense d (differentiation
// workload).  H = -<p, A x + eps tanh x> + |p|^2/2 (paper convention, section
// 2.1), g = x^T Q_s x / 2, Algorithm 1 with:
//   dual   p_j <- (p_j + sigma (z_j - z_{j-1}) + lam (A x_j + eps tanh x_j)) / (1 + lam),
//          lam = sigma delta                                   (closed-form prox)
//   node 0 x_0 <- M (x_0 + tau p_1),  M = (I + tau Q_s)^{-1}
//   primal x_j <- x_j - tau (p_j - p_{j+1}) - tau delta (A^T p_j + eps (1 - tanh^2 x_j) p_j)
//   extrapolation z = x_new + theta (x_new - x_old).
//
// Forward kernel (k_lt_forward): the iteration of hjpd_lt_core.hpp on a state
// that stays in registers, one point per wave (d = 16, 32) or per workgroup of
// eight waves (d = 100, 128).  Workgroups are persistent and pop points from a
// counter; the kernel is compiled for one to four 16-node column tiles.
//
// Reverse mode (hjpd_value_grad): the forward pass stores the state every E
// iterations; the reverse kernel (k_lt_backward; the step is hjpd_lt_back.hpp's)
// recomputes each segment from its checkpoint and applies the transposed
// Jacobian of every iteration from the last one down.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "hjpd_lt_back.hpp"

namespace hjpd {

constexpr int kLtCounters = 8;
constexpr int kLtPackBlocks = 16;

// t > 0, 1 <= N <= N_max, x finite; the whole wave calls it for one point.
template <int D>
__device__ __forceinline__ bool lt_bad_point(const LtArgs& a, int64_t pt) {
  const int lane = threadIdx.x & 63;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < (D + 63) / 64; i++) bad = bad || (lane + 64 * i < D && !__builtin_isfinite(a.x[pt * D + lane + 64 * i]));
  const float t = a.t[pt];
  const int N = a.N[pt];
  return __any(bad || !(t > 0.f) || !__builtin_isfinite(t) || N < 1 || N > a.N_max);
}

template <int D, int NT, int KIND>
__device__ __forceinline__ void lt_forward_wave(const LtArgs& a, float* smem, int* s_pt) {
  using S = LtShape<D, NT>;
  LtCore<D, NT, KIND> c;
  c.setup(a, smem);
  const float eps = a.hp[0];
  const int64_t slot = 3 * int64_t(a.N_max + 1) * D;
  for (;;) {
    int pop = 0;
    if (c.tid == 0) pop = atomicAdd(a.head, 1);
    if constexpr (S::W > 1) {
      if (c.tid == 0) *s_pt = pop;
      __syncthreads();
      pop = *s_pt;
      __syncthreads();
    }
    const int64_t pt = __builtin_amdgcn_readfirstlane(pop);
    if (pt >= a.n) break;
    if (lt_bad_point<D>(a, pt)) {
      if (c.tid == 0) {
        if (a.phi) a.phi[pt] = NAN;
        a.iters[pt] = 0;
        a.status[pt] = kBadInput;
      }
      continue;
    }
    c.set_point(a, pt);
    c.start(a, pt);
    float* snap = a.ckpt ? a.ckpt + pt * (a.n_ckpt + 1) * slot : nullptr;
    int k = 0, st = kMaxIter, next_snap = 0, snaps = 0;
    auto snapshot = [&]() {
      if (snap && k == next_snap && snaps < a.n_ckpt) {
        c.save(snap + snaps * slot, a.N_max);
        snaps++;
        next_snap += a.ckpt_every;
      }
    };
    float rx = 0.f, rp = 0.f;
    if (a.fixed)  // residuals only of the last iteration
      for (; k + 1 < a.max_iter; k++) {
        snapshot();
        c.template iterate<false>(a, eps, rx, rp);
      }
    for (bool done = false; !done;) {
      snapshot();
      rx = rp = 0.f;
      c.template iterate<true>(a, eps, rx, rp);
      k++;
      c.sum2(rx, rp);
      done = k >= a.max_iter;
      if (!__builtin_isfinite(rx + rp)) {
        st = kNonFinite;
        done = true;
      } else if (rx < a.tol && rp < a.tol && (!a.fixed || done)) {
        st = kConverged;
        done = true;
      }
    }
    if (snap) c.save(snap + a.n_ckpt * slot, a.N_max);

    // ---- value: g(x_0) + sum <p_j, x_j - x_{j-1}> - delta sum H(x_j, p_j) ----------
    float val = 0.f, badf = 0.f;
    if constexpr (S::kReg)
      if (c.lr == 0)
#pragma unroll
        for (int ri = 0; ri < S::RPW; ri++) st4(c.sX0 + c.coord(ri), c.x0[ri]);
    if constexpr (c.kRows)
      c.sweep(c.fA, c.imgX, c.tailX, c.X, [&](int t, const f4(&acc)[S::RPW]) __attribute__((always_inline)) {
#pragma unroll
        for (int ri = 0; ri < S::RPW; ri++) {
          const f4 xm = t > 0 ? c.X[ri][t > 0 ? t - 1 : 0] : row_prev(c.X[ri][NT - 1]) + c.x0_of(ri);
#pragma unroll
          for (int r = 0; r < 4; r++) {
            // nodes past N have x = p = 0 and add nothing
            const float xv = c.X[ri][t][r], pv = c.P[ri][t][r];
            const float f = acc[ri][r] + eps * tanh_fast(xv);
            val += pv * (xv - xm[r]) - c.delta * (0.5f * pv * pv - pv * f);
            if (!(__builtin_isfinite(xv) && __builtin_isfinite(pv))) badf = 1.f;
          }
        }
      });
    __syncthreads();
    // x_0^T Q x_0 / 2 (the symmetric part of Q is all that counts), a column of Q to a thread
    for (int i = c.tid; i < D; i += S::kThreads) {
      float qx = 0.f;
#pragma unroll 10
      for (int kq = 0; kq < D; kq++) qx += a.Q[kq * D + i] * c.sX0[kq];
      val += 0.5f * c.sX0[i] * qx;
      if (!__builtin_isfinite(c.sX0[i])) badf = 1.f;
    }
    c.sum2(val, badf);
    if (badf > 0.f || !__builtin_isfinite(val)) st = kNonFinite;
    if (c.tid == 0) {
      if (a.phi) a.phi[pt] = val;
      a.iters[pt] = k;
      a.status[pt] = st;
    }
    if constexpr (c.kRows)
      if (a.xtraj || a.ptraj) {
        const int64_t base = pt * int64_t(a.N_max + 1) * D;
#pragma unroll
        for (int ri = 0; ri < S::RPW; ri++) {
          if (!c.rows_ok(ri)) continue;
          const int i0 = c.coord(ri);
          const f4 x0 = c.x0_of(ri);
#pragma unroll
          for (int t = -1; t < NT; t++) {
            const int j = t < 0 ? 0 : c.node(t);
            if (t < 0 ? c.lr != 0 : j > c.Np) continue;
#pragma unroll
            for (int r = 0; r < 4; r++) {
              if (a.xtraj) a.xtraj[base + j * D + i0 + r] = t < 0 ? x0[r] : c.X[ri][t < 0 ? 0 : t][r];
              if (a.ptraj) a.ptraj[base + j * D + i0 + r] = t < 0 ? 0.f : c.P[ri][t < 0 ? 0 : t][r];
            }
          }
        }
      }
    __syncthreads();
  }
}

template <int D, int NT>
__global__ void __launch_bounds__((LtShape<D, NT>::kThreads), 2) k_lt_forward(LtArgs a) {
  using S = LtShape<D, NT>;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  __shared__ int s_pt;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (S::kAux && wave == S::RT) lt_forward_wave<D, NT, S::kAux ? kAuxWave : kRowWave>(a, smem, &s_pt);
  else if (S::kTail && wave == S::RT - 1) lt_forward_wave<D, NT, S::kTail ? kTailWave : kRowWave>(a, smem, &s_pt);
  else lt_forward_wave<D, NT, kRowWave>(a, smem, &s_pt);
}

template <int D, int NT, int KIND>
__device__ __forceinline__ void lt_backward_wave(const LtBwdArgs& b, float* smem) {
  using C = LtBack<D, NT, KIND>;
  using S = typename C::S;
  constexpr int RPW = C::RPW, RT = C::RT, LD = D + 1;
  constexpr int64_t DD = int64_t(D) * D, TF = C::tiles_floats();
  const LtArgs& a = b.f;
  C c;
  c.setup_back(a, smem);
  const int tid = c.tid, lr = c.lr, lk = c.lk;
  const float eps = a.hp[0], tau = a.tau;
  const int E = a.ckpt_every;
  const int64_t CK = int64_t(a.N_max + 1) * D, slot = 3 * CK;
  float* seg = b.seg + int64_t(blockIdx.x) * (int64_t(E) * (2 * TF + 2 * D) + 2 * TF);
  float* adj = seg + int64_t(E) * 2 * TF;
  float* stage = adj + 2 * TF;  // per step of a segment: XB_0 and w = x_0 + tau p'_1
  // dA is summed in registers (with many column tiles, C::kFlush steps at a
  // time); the direct dQ term and (d > 32) dM in this workgroup's partial block
  float* part = b.part + int64_t(blockIdx.x) * (3 * DD + 1);
  for (int e = tid; e < DD; e += S::kThreads) part[e] = part[DD + e] = part[2 * DD + e] = 0.f;
  __syncthreads();

  // dA into the partial block (every entry has one lane that adds to it)
  auto flush_dA = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int ct = 0; ct < RT; ct++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int row = c.coord(ri) + r, col = 16 * ct + lr;
          if (row < D && col < D) part[row * D + col] += ldexpf(c.dA[ri][ct][r], c.e_all);
          c.dA[ri][ct][r] = 0.f;
        }
  };

  // Points are dealt to the workgroups in a fixed order (every point costs
  // the same K iterations), so each workgroup's partial sums of dA, dM, dQ and
  // deps, and with them the gradients, are the same from call to call.
  c.scale_of_all(b, blockIdx.x, gridDim.x);
  for (int64_t pt = blockIdx.x; pt < a.n; pt += gridDim.x) {
    const float w_out = b.grad_phi[pt];
    if (w_out == 0.f || lt_bad_point<D>(a, pt)) {
      for (int i = tid; i < D; i += S::kThreads) b.dphi_dx[pt * D + i] = 0.f;
      continue;
    }
    c.set_point(a, pt);
    const float w = c.scale_of_point(w_out);
    const float* ck_pt = a.ckpt + pt * (a.n_ckpt + 1) * slot;
    f4 xb0[RPW], zb0[RPW];  // node 0's adjoints (d <= 32)
    float s1 = 0.f, s2 = 0.f;

    // ---- adjoint of the value at the final iterate: XB, PB; dA += w delta sum p_j x_j^T ----
    {
      const float* last = ck_pt + a.n_ckpt * slot;
      const float wd = w * c.ds;
      for (int i = tid; i < D; i += S::kThreads) c.sX0[i] = last[i];
      if constexpr (C::kRows) {
        c.load_nodes(last, c.X);
        c.load_nodes(last + CK, c.P);
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          if (lr == 0 && c.rows_ok(ri)) st4(c.sV + c.coord(ri), c.P[ri][0]);
          if constexpr (!S::kReg)
#pragma unroll
            for (int t = 0; t < NT; t++) {
              c.put(c.imgX, c.tailX, t, c.X[0][t]);
              c.put(c.imgP, c.tailP, t, c.P[0][t]);
              c.put(c.img3, nullptr, t, wd * c.X[0][t]);
            }
        }
      }
      __syncthreads();
      for (int i = tid; i < D; i += S::kThreads) {
        float qx = 0.f;
#pragma unroll 10
        for (int k = 0; k < D; k++) qx += a.Qs[k * D + i] * c.sX0[k];
        const float xb = w * (qx - c.sV[i]);
        c.sXb0[i] = c.sE[i] = xb;
        c.sZb0[i] = 0.f;
      }
      for (int e = tid; e < DD; e += S::kThreads) part[2 * DD + e] += 0.5f * w_out * c.sX0[e / D] * c.sX0[e % D];
      if constexpr (C::kRows) {
        float sp = 0.f;
        c.load_matrices(a);
        c.sweep(c.fA, c.imgX, c.tailX, c.X, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
          const float wj = c.node(t) <= c.Np ? w : 0.f;
#pragma unroll
          for (int ri = 0; ri < RPW; ri++) {
            f4 x0 = f4{0.f, 0.f, 0.f, 0.f}, pb;
            if (t == 0 && lr == 0 && c.rows_ok(ri)) x0 = ld4(c.sX0 + c.coord(ri));
            const f4 xm = t > 0 ? c.X[ri][t > 0 ? t - 1 : 0] : row_prev(c.X[ri][NT - 1]) + x0;
#pragma unroll
            for (int r = 0; r < 4; r++) {
              const float xv = c.X[ri][t][r], pv = c.P[ri][t][r], th = tanh_fast(xv);
              pb[r] = wj * (xv - xm[r] + c.delta * (acc[ri][r] + eps * th - pv));
              sp += pv * th;
            }
            if constexpr (S::kPbLds) st4(at<true>(c.sPb, 4 * tid) + 256 * RT * t, pb);
            else c.PB[ri][t] = pb;
          }
        });
        c.deps += wd * sp;
        c.sweep(c.fAt, c.imgP, c.tailP, c.P, [&](int t, const f4(&acc)[RPW]) __attribute__((always_inline)) {
#pragma unroll
          for (int ri = 0; ri < RPW; ri++) {
            const f4 pn = t < NT - 1 ? c.P[ri][t < NT - 1 ? t + 1 : t] : row_next(c.P[ri][0]);
#pragma unroll
            for (int r = 0; r < 4; r++) {
              const float pv = c.P[ri][t][r], th = tanh_fast(c.X[ri][t][r]);
              c.ZB[ri][t][r] = w * (pv - pn[r] + c.delta * (acc[ri][r] + eps * ((1.f - th * th) * pv)));
              c.XB[ri][t][r] = 0.f;
            }
          }
        });
        if constexpr (S::kReg) {
#pragma unroll
          for (int ri = 0; ri < RPW; ri++)
#pragma unroll
            for (int t = 0; t < NT; t++) {
              c.scratch_put(0, ri, t, c.P[ri][t]);
              c.scratch_put(1, ri, t, wd * c.X[ri][t]);
            }
          c.outer_scratch();
        } else {
          c.outer(c.imgP, c.img3);
        }
      }
      __syncthreads();
      if constexpr (S::kReg) {
#pragma unroll
        for (int ri = 0; ri < RPW; ri++) {
          xb0[ri] = zb0[ri] = f4{0.f, 0.f, 0.f, 0.f};
          if (lr == 0) xb0[ri] = ld4(c.sXb0 + c.coord(ri));
        }
      } else if constexpr (!S::kAux || KIND == kAuxWave) {
        c.node0_product();
      }
    }

    // ---- segments, last to first ------------------------------------------------------
    const int nseg = (b.K + E - 1) / E;
    for (int sg = nseg - 1; sg >= 0; sg--) {
      const int k0 = sg * E, nk = min(b.K, k0 + E) - k0;
      // save the adjoint, recompute the segment forward from its checkpoint
      if constexpr (C::kRows) {
        c.store_tiles(adj, c.XB);
        c.store_tiles(adj + TF, c.ZB);
      }
      c.load_snapshot(ck_pt + sg * slot, a.N_max);
      if constexpr (C::kRows) c.load_matrices(a);
      c.put_all(c.imgX, c.tailX, c.X);
      for (int k = 0; k < nk; k++) {
        float* q = seg + int64_t(k) * 2 * TF;
        float* st = stage + int64_t(k) * 2 * D;
        float rx = 0.f, rp = 0.f;
        f4 x0[RPW];
        if constexpr (C::kRows) {
          c.store_tiles(q, c.X);
          if constexpr (!S::kAux)
#pragma unroll
            for (int ri = 0; ri < RPW; ri++) x0[ri] = c.x0_of(ri);
        }
        c.template iterate<false>(a, eps, rx, rp);
        if constexpr (S::kAux && KIND == kAuxWave)
          for (int i = tid & 63; i < D; i += 64) st[D + i] = c.sW[i];
        if constexpr (C::kRows) {
          c.store_tiles(q + TF, c.P);
          if constexpr (!S::kAux)
            if (lr == 0)
#pragma unroll
              for (int ri = 0; ri < RPW; ri++)
                st4(st + D + c.coord(ri), x0[ri] + tau * c.P[ri][0]);
        }
      }
      if constexpr (C::kRows) {
        c.load_tiles(adj, c.XB);
        c.load_tiles(adj + TF, c.ZB);
      }
      float touched = 0.f;
      typename C::Tiles pk;
      if constexpr (C::kRows) c.load_tiles(seg + int64_t(nk - 1) * 2 * TF + TF, pk);
      for (int k1 = nk; k1 > 0; k1 -= C::kFlush) {
        for (int k = k1 - 1; k >= max(k1 - C::kFlush, 0); k--) {
          float* cur = seg + int64_t(k) * 2 * TF;
          c.step(a, eps, stage + int64_t(k) * 2 * D, cur, k > 0 ? cur - 2 * TF : nullptr, pk, touched, xb0, zb0, s1, s2);
        }
        if constexpr (C::kRows && C::kFlush < 1 << 30) flush_dA();
      }
      // dM += sum over the segment's steps of XB_0 w^T, in FP32 from the kept pairs
      if constexpr (S::kReg) {
        __threadfence_block();
        for (int j0 = 0; j0 < nk; j0 += 4) {
          float u[RPW], v[RPW];
          const bool ok = j0 + lk < nk;
          const float* st = stage + int64_t(ok ? j0 + lk : 0) * 2 * D;
#pragma unroll
          for (int ri = 0; ri < RPW; ri++) {
            u[ri] = ok ? st[16 * ri + lr] : 0.f;
            v[ri] = ok ? st[D + 16 * ri + lr] : 0.f;
          }
#pragma unroll
          for (int ri = 0; ri < RPW; ri++)
#pragma unroll
            for (int ct = 0; ct < RT; ct++) c.dM[ri][ct] = mfma4(u[ri], v[ct], c.dM[ri][ct]);
        }
      } else {
        constexpr int R = 32;  // steps per pass: two [R][d + 1] arrays fit the smallest images
        static_assert(2 * R * LD <= 3 * S::kImg, "staging fits the images");
        float *S0 = smem, *S1 = smem + R * LD;
        for (int r0 = 0; r0 < nk; r0 += R) {
          const int nr = min(R, nk - r0);
          __syncthreads();
          for (int e = tid; e < R * LD; e += S::kThreads) {
            const int j = e / LD, i = e - j * LD;
            const bool ok = j < nr && i < D;
            const float* st = stage + int64_t(r0 + j) * 2 * D;
            S0[e] = ok ? st[i] : 0.f;
            S1[e] = ok ? st[D + i] : 0.f;
          }
          __syncthreads();
          if constexpr (C::kRows) {
            const int row = 16 * c.wave + lr, rc = row < D ? row : D;
            f4 acc[RT];
#pragma unroll
            for (int ct = 0; ct < RT; ct++) acc[ct] = f4{0.f, 0.f, 0.f, 0.f};
            for (int j = lk; j < R; j += 4) {
              const float u = S0[j * LD + rc];
#pragma unroll
              for (int ct = 0; ct < RT; ct++) {
                const int col = 16 * ct + lr;
                acc[ct] = mfma4(u, S1[j * LD + (col < D ? col : D)], acc[ct]);
              }
            }
            float* pm = part + DD + int64_t(16 * c.wave + 4 * lk) * D + lr;
#pragma unroll
            for (int ct = 0; ct < RT; ct++)
#pragma unroll
              for (int r = 0; r < 4; r++)
                if (16 * c.wave + 4 * lk + r < D && 16 * ct + lr < D) pm[r * D + 16 * ct] += ldexpf(acc[ct][r], c.e_dM);
          }
        }
        __syncthreads();
      }
    }
    c.deps += a.sigma * c.ds * s2 - tau * c.ds * s1;
    // d phi / d x: every x_j^0 = x + noise (j < N), x_N = x, z^0 = x^0
    if constexpr (C::kRows)
#pragma unroll
      for (int ri = 0; ri < RPW; ri++) {
        f4 g;
        if constexpr (S::kReg) g = xb0[ri] + zb0[ri];
        else g = c.first_col(ld4(c.sXb0 + (c.rows_ok(0) ? c.coord(0) : 0)) +
                             ld4(c.sZb0 + (c.rows_ok(0) ? c.coord(0) : 0)));
#pragma unroll
        for (int t = 0; t < NT; t++) g += c.XB[ri][t] + c.ZB[ri][t];
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const float v = group_sum<16>(g[r]);
          if (lr == 0 && c.rows_ok(ri)) b.dphi_dx[pt * D + c.coord(ri) + r] = ldexpf(v, c.e_w);
        }
      }
    __syncthreads();
  }
  // ---- per-workgroup partial parameter gradients ----------------------------------------
  if constexpr (C::kRows) flush_dA();
  if constexpr (S::kReg)
#pragma unroll
    for (int ri = 0; ri < RPW; ri++)
#pragma unroll
      for (int ct = 0; ct < RT; ct++)
#pragma unroll
        for (int r = 0; r < 4; r++)
          part[DD + (c.coord(ri) + r) * D + 16 * ct + lr] = ldexpf(c.dM[ri][ct][r], c.e_dM);
  float zero = 0.f;
  c.sum2(c.deps, zero);
  if (tid == 0) part[3 * DD] = ldexpf(c.deps, c.e_all);
}

template <int D, int NT>
__global__ void __launch_bounds__((LtShape<D, NT>::kThreads), 2) k_lt_backward(LtBwdArgs b) {
  using S = LtShape<D, NT, true>;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (S::kAux && wave == S::RT) lt_backward_wave<D, NT, S::kAux ? kAuxWave : kRowWave>(b, smem);
  else if (S::kTail && wave == S::RT - 1) lt_backward_wave<D, NT, S::kTail ? kTailWave : kRowWave>(b, smem);
  else lt_backward_wave<D, NT, kRowWave>(b, smem);
}

// Sum the per-workgroup partials (fixed order: deterministic).  A block takes
// 64 entries; its 16 waves sum every 16th partial each, all loads independent,
// and the sums meet in LDS.  Bound by memory latency: one thread per entry over
// all partials in turn took 99 us for 256 partials of d = 100 (184 us for 777
// of d = 32); this takes 9.5 us (5.4 us).
constexpr int kRedWaves = 16;
__global__ void __launch_bounds__(64 * kRedWaves) k_lt_reduce_parts(const float* part, int nwg, int d,
                                                                    float* out /* [3 d^2 + 1] */) {
  __shared__ float s[kRedWaves][64];
  const int64_t DD = int64_t(d) * d, W = 3 * DD + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t e = int64_t(blockIdx.x) * 64 + lane;
  float v = 0.f;
  if (e < W)
#pragma unroll 16
    for (int g = wave; g < nwg; g += kRedWaves) v += part[g * W + e];
  s[wave][lane] = v;
  __syncthreads();
  if (wave == 0 && e < W) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kRedWaves; w++) t += s[w][lane];
    out[e] = t;
  }
}

// Row blockIdx.x of S = scale M dM M: u = M[row] dM, then u M; four groups of
// threads take a quarter of the terms each.  (Two launches of a thread per
// entry took 26 us each at d = 100; this takes 5 us.)
__global__ void __launch_bounds__(4 * kLtMaxD) k_lt_mdm(const float* M, const float* dM, int d, float scale, float* S) {
  __shared__ float s_u[kLtMaxD], s_part[4][kLtMaxD];
  const int c = threadIdx.x % kLtMaxD, g = threadIdx.x / kLtMaxD, q = d / 4;
  auto vec_mat = [&](const float* B, auto u) {
    float v = 0.f;
    if (c < d)
#pragma unroll 8
      for (int k = g * q; k < (g + 1) * q; k++) v += u(k) * B[k * d + c];
    s_part[g][c] = v;
    __syncthreads();
    return (s_part[0][c] + s_part[1][c]) + (s_part[2][c] + s_part[3][c]);
  };
  const float u = vec_mat(dM, [&](int k) { return M[blockIdx.x * d + k]; });
  if (g == 0) s_u[c] = u;
  __syncthreads();
  const float v = vec_mat(M, [&](int k) { return s_u[k]; });
  if (g == 0 && c < d) S[blockIdx.x * d + c] = scale * v;
}

// dh = [deps, dA]; dg = dQ_direct + sym(S) with S = -tau M dM M.
__global__ void k_lt_grad_out(const float* sums, const float* S, int d, float* dh, float* dg) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t DD = int64_t(d) * d;
  if (e == 0) dh[0] = sums[3 * DD];
  if (e >= d * d) return;
  const int r = e / d, c = e - r * d;
  dh[1 + e] = sums[e];
  dg[e] = sums[2 * DD + e] + 0.5f * (S[r * d + c] + S[c * d + r]);
}

// Set-up of a call: block 0 inverts, the others pack A's operands.
//
// (I + tau Q_s)^{-1} by Gauss-Jordan exchange steps with row pivoting in double
// precision, one workgroup, the matrix in registers: thread (tr, tc) holds rows
// tr + TR u and columns tc + 16 m.  Also clears the solve's counters.
//
// The elimination is a chain of d steps, so what bounds it is the latency of
// one step: a barrier after the pivot column's entries reach LDS, a wave-wide
// maximum that every wave forms for itself (no second pass over LDS), a barrier
// after the pivot row, and D*D / threads updates per thread.  Rows are not
// exchanged: a row that has served as pivot is marked, and the permutation is
// undone on output.  With the matrix in global memory and thread 0 searching
// the pivot alone it took 29 / 124 / 2,350 / 4,600 us at d = 16 / 32 / 100 / 128;
// this form takes 8 / 17 / 112 / 154 us.
template <int D>
struct LtInv {
  static constexpr int TR = D <= 32 ? 16 : 64;  // row groups (16 column groups): 256 or 1,024 threads
  static constexpr int RU = (D + TR - 1) / TR, CM = (D + 15) / 16, kThreads = 16 * TR;
};

template <int D>
__global__ void __launch_bounds__(LtInv<D>::kThreads) k_lt_setup(const float* Q, const float* hp, double tau, float* Mout,
                                                                 float* Mc, float* Qs, float* packed,
                                                                 int32_t* counters) {
  constexpr int TR = LtInv<D>::TR, RU = LtInv<D>::RU, CM = LtInv<D>::CM;
  __shared__ double s_col[2][D], s_row[2][16 * CM];  // alternate between steps: one barrier each way is enough
  __shared__ int s_piv[D];
  const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15, lane = tid & 63;
  using Frag = LtFrag<D>;
  if (blockIdx.x > 0) {  // A and A^T as operands, rows past d zero
    constexpr int kRows = LtShape<D, 1>::RT * 16, kPairs = D / 2;
    const float* A = hp + 1;
    for (int e = (blockIdx.x - 1) * LtInv<D>::kThreads + tid; e < 2 * kRows * kPairs;
         e += (gridDim.x - 1) * LtInv<D>::kThreads) {
      const int matrix = e / (kRows * kPairs), row = e / kPairs % kRows, k = 2 * (e % kPairs);
      const int rs = matrix ? 1 : D, ks = matrix ? D : 1;
      const float u = row < D ? A[row * rs + k * ks] : 0.f, v = row < D ? A[row * rs + (k + 1) * ks] : 0.f;
      Frag::pack(packed, matrix, row, k, u, v);
      if constexpr (LtShape<D, 1>::kReg) Frag::pack(packed, matrix, row, k + 1, v, v);
    }
    return;
  }
  if (tid < kLtCounters) counters[tid] = 0;
  double T[RU][CM];
#pragma unroll
  for (int u = 0; u < RU; u++)
#pragma unroll
    for (int m = 0; m < CM; m++) {
      const int r = tr + TR * u, c = tc + 16 * m;
      T[u][m] = (r < D && c < D) ? (r == c ? 1.0 : 0.0) + tau * 0.5 * (double(Q[r * D + c]) + double(Q[c * D + r])) : 0.0;
    }
  bool used0 = lane >= D, used1 = lane + 64 >= D;  // rows lane and lane + 64 have served (or do not exist)
#pragma unroll
  for (int mc = 0; mc < CM; mc++) {
    for (int cc = 0; cc < 16; cc++) {
      const int c = 16 * mc + cc;
      if (c >= D) break;
      double* col = s_col[c & 1];
      double* row = s_row[c & 1];
      if (tc == cc)
#pragma unroll
        for (int u = 0; u < RU; u++)
          if (tr + TR * u < D) col[tr + TR * u] = T[u][mc];
      __syncthreads();
      // largest entry among the rows that have not served: the top bits of its
      // magnitude with 127 - row in the last seven (entries within 2^-13 of the
      // largest count as equal, the lowest row wins; a NaN counts as zero)
      auto key_of = [&](int r) {
        const uint32_t hi = uint32_t(__double_as_longlong(col[r]) >> 32) & 0x7fffffffu;
        return int(((hi <= 0x7ff00000u ? hi : 0u) & ~127u) | uint32_t(127 - r));
      };
      int key = used0 ? -1 : key_of(lane);
      if (!used1) key = max(key, key_of(lane + 64));
      auto exchange = [&](auto ctrl) {
        key = max(key, __builtin_amdgcn_update_dpp(0, key, decltype(ctrl)::value, 0xf, 0xf, true));
      };
      exchange(std::integral_constant<int, kDppQuad1032>{});
      exchange(std::integral_constant<int, kDppQuad2301>{});
      exchange(std::integral_constant<int, kDppRowHalfMirror>{});
      exchange(std::integral_constant<int, kDppRowMirror>{});
      key = max(key, __shfl_xor(key, 16, 64));
      key = max(key, __shfl_xor(key, 32, 64));
      const int pr = 127 - (__builtin_amdgcn_readfirstlane(key) & 127);
      used0 |= pr == lane;
      used1 |= pr == lane + 64;
      const double inv = 1.0 / col[pr];
      if (tid == 0) {
        s_piv[c] = pr;
        if (!(fabs(col[pr]) > 0.0)) counters[1] = 1;
      }
      if (tr == pr % TR)
#pragma unroll
        for (int u = 0; u < RU; u++)
          if (tr + TR * u == pr)
#pragma unroll
            for (int m = 0; m < CM; m++) row[tc + 16 * m] = T[u][m];
      __syncthreads();
      // exchange y_pr and x_c: the pivot row becomes -row / a (1 / a at c), every
      // other row T - T[.][c] row / a (T[.][c] / a at c)
#pragma unroll
      for (int u = 0; u < RU; u++) {
        const int r = tr + TR * u;
        const bool piv = r == pr;
        const double f = r < D ? (piv ? 0.0 : col[r]) : 0.0;
#pragma unroll
        for (int m = 0; m < CM; m++) {
          const double q = row[tc + 16 * m] * inv;
          const bool here = m == mc && tc == cc;
          if (here) T[u][m] = piv ? inv : T[u][m] * inv;
          else T[u][m] = piv ? -q : T[u][m] - f * q;
        }
      }
    }
  }
  __syncthreads();
  // row pr_c of the tableau is x_c, column c' stands for y at row pr_c'
  __shared__ int s_var[D];  // row -> the variable it holds
  if (tid < D) s_var[s_piv[tid]] = tid;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < RU; u++)
#pragma unroll
    for (int m = 0; m < CM; m++) {
      const int r = tr + TR * u, c = tc + 16 * m;
      if (r < D && c < D) {
        const int i = s_var[r], j = s_piv[c];
        Mout[i * D + j] = float(T[u][m]);
        Mc[(j / 4 * D + i) * 4 + j % 4] = float(T[u][m]);
        Qs[r * D + c] = 0.5f * (Q[r * D + c] + Q[c * D + r]);
        if constexpr (LtShape<D, 1>::kReg) Frag::pack(packed, 2, i, j, float(T[u][m]), 0.f);
      }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

struct LtState {
  int d = 0;
  int n_cu = 0;
  float* M = nullptr;           // M, M in chunks of four columns, Q_s (d*d each), packed operands
  int32_t* counters = nullptr;  // [0] forward head, [1] inverse failure
  int32_t* scratch_i = nullptr; // iterations and statuses of the forward pass in value_grad
  size_t scratch_bytes = 0;
  float* ckpt = nullptr;
  size_t ckpt_bytes = 0;
  float* seg = nullptr;
  size_t seg_bytes = 0;
  float* part = nullptr;
  size_t part_bytes = 0;
  float* sums = nullptr;  // 3 d^2 + 1
  float* tmp = nullptr;   // d^2
};

typedef const void* KernelPtr;

// Floats of the largest packed copy (d = 128: two matrices; d = 32: three).
constexpr size_t kLtPacked = 2 * LtFrag<128>::kMatrix;
static_assert(kLtPacked >= 3 * size_t(LtFrag<32>::kMatrix) && kLtPacked >= 2 * size_t(LtFrag<100>::kMatrix), "packed operands fit");

// A kernel for (d, N_max): its column tiles cover N_max.
struct LtKernel {
  KernelPtr fn = nullptr;
  int threads = 0;
  size_t lds = 0;
};

template <int D, int NT>
static LtKernel kernel_of(bool back) {
  if (back)
    return {reinterpret_cast<KernelPtr>(&k_lt_backward<D, NT>), LtShape<D, NT>::kThreads,
            sizeof(float) * LtShape<D, NT, true>::kLdsFloats};
  return {reinterpret_cast<KernelPtr>(&k_lt_forward<D, NT>), LtShape<D, NT>::kThreads,
          sizeof(float) * LtShape<D, NT>::kLdsFloats};
}
template <int D>
static LtKernel kernel_tiles(int N_max, bool back) {
  switch ((N_max + 15) / 16) {
    case 1: return kernel_of<D, 1>(back);
    case 2: return kernel_of<D, 2>(back);
    case 3: return kernel_of<D, 3>(back);
    case 4:
      if constexpr (D < 128) return kernel_of<D, 4>(back);  // d = 128 is built for N_max <= 48
  }
  return {};
}
static LtKernel lt_kernel(int d, int N_max, bool back) {
  switch (d) {
    case 16: return kernel_tiles<16>(N_max, back);
    case 32: return kernel_tiles<32>(N_max, back);
    case 100: return kernel_tiles<100>(N_max, back);
    case 128: return kernel_tiles<128>(N_max, back);
  }
  return {};
}

#define LT_HIP(expr, what)                                                                                    \
  do {                                                                                                        \
    hipError_t e_ = (expr);                                                                                   \
    if (e_ != hipSuccess) return hjpd_fail(HJPD_EDEVICE, (std::string(what) + ": " + hipGetErrorString(e_)).c_str()); \
  } while (0)

int lt_create(LtState** out, const hjpd_desc& desc) {
  *out = nullptr;
  if (!lt_kernel(desc.d, 1, false).fn) return hjpd_fail(HJPD_EUNSUPPORTED, "LINEAR_TANH is built for d in {16,32,100,128}");
  if (desc.N_max > kLtMaxN) return hjpd_fail(HJPD_EUNSUPPORTED, "LINEAR_TANH is built for N_max <= 64");
  const LtKernel fwd = lt_kernel(desc.d, desc.N_max, false), bwd = lt_kernel(desc.d, desc.N_max, true);
  if (!fwd.fn) return hjpd_fail(HJPD_EDEVICE, "cannot reserve LDS for the linear-tanh kernels (d = 128: N_max <= 48)");
  LtState* s = new LtState();
  s->d = desc.d;
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    delete s;
    return hjpd_fail(HJPD_EDEVICE, "device query failed");
  }
  s->n_cu = prop.multiProcessorCount;
  if (hipFuncSetAttribute(fwd.fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(fwd.lds)) != hipSuccess ||
      hipFuncSetAttribute(bwd.fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bwd.lds)) != hipSuccess) {
    delete s;
    return hjpd_fail(HJPD_EDEVICE, "cannot reserve LDS for the linear-tanh kernels");
  }
  const size_t dd = size_t(desc.d) * desc.d;
  if (hipMalloc(&s->M, sizeof(float) * (3 * dd + kLtPacked))  != hipSuccess ||
      hipMalloc(&s->counters, sizeof(int32_t) * kLtCounters) != hipSuccess ||
      hipMalloc(&s->sums, sizeof(float) * (3 * dd + 1)) != hipSuccess ||
      hipMalloc(&s->tmp, sizeof(float) * dd) != hipSuccess) {
    lt_destroy(s);
    return hjpd_fail(HJPD_ENOMEM, "linear-tanh workspace");
  }
  *out = s;
  return HJPD_OK;
}

void lt_destroy(LtState* s) {
  if (!s) return;
  if (s->M) (void)hipFree(s->M);
  if (s->counters) (void)hipFree(s->counters);
  if (s->scratch_i) (void)hipFree(s->scratch_i);
  if (s->ckpt) (void)hipFree(s->ckpt);
  if (s->seg) (void)hipFree(s->seg);
  if (s->part) (void)hipFree(s->part);
  if (s->sums) (void)hipFree(s->sums);
  if (s->tmp) (void)hipFree(s->tmp);
  delete s;
}

static int lt_grid(LtState* st, KernelPtr k, int threads, size_t lds, int64_t n) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, threads, lds) != hipSuccess || nb < 1) nb = 1;
  return int(std::min<int64_t>(int64_t(nb) * st->n_cu, n));
}

static void fill_args(LtArgs& a, LtState* st, const hjpd_desc& d, int64_t n, const void* x, const void* t,
                      const int32_t* N, const void* hp, const void* gp, void* phi, void* xtraj, void* ptraj,
                      int32_t* iters, int32_t* status, int max_iter, bool fixed) {
  std::memset(&a, 0, sizeof(a));
  a.x = (const float*)x;
  a.t = (const float*)t;
  a.N = N;
  a.hp = (const float*)hp;
  a.Q = (const float*)gp;
  a.Mc = st->M + size_t(d.d) * d.d;
  a.Qs = st->M + 2 * size_t(d.d) * d.d;
  a.packed = st->M + 3 * size_t(d.d) * d.d;
  a.phi = (float*)phi;
  a.xtraj = (float*)xtraj;
  a.ptraj = (float*)ptraj;
  a.iters = iters;
  a.status = status;
  a.head = st->counters;
  a.n = n;
  a.sigma = float(d.sigma);
  a.tau = float(d.tau);
  a.theta = float(d.theta);
  a.tol = float(d.tol);
  a.max_iter = max_iter;
  a.fixed = fixed ? 1 : 0;
  a.N_max = d.N_max;
  a.seed = d.seed;
  a.ckpt_every = 1;
}

static int lt_setup(LtState* st, const hjpd_desc& d, const void* hp, const void* gp, hipStream_t s) {
  const size_t dd = size_t(d.d) * d.d;
  auto launch = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3(1 + kLtPackBlocks), dim3(threads), 0, s, (const float*)gp, (const float*)hp, d.tau,
                       st->M, st->M + dd, st->M + 2 * dd, st->M + 3 * dd, st->counters);
  };
  switch (d.d) {
    case 16: launch(k_lt_setup<16>, LtInv<16>::kThreads); break;
    case 32: launch(k_lt_setup<32>, LtInv<32>::kThreads); break;
    case 100: launch(k_lt_setup<100>, LtInv<100>::kThreads); break;
    default: launch(k_lt_setup<128>, LtInv<128>::kThreads); break;
  }
  LT_HIP(hipGetLastError(), "linear-tanh set-up kernel");
  return HJPD_OK;
}

int lt_solve(LtState* st, const hjpd_desc& d, int64_t n, const void* x, const void* t, const int32_t* N,
             const void* hp, const void* gp, void* phi, void* xtraj, void* ptraj, int32_t* iters, int32_t* status,
             hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, int* launches, bool* timing_valid) {
  int rc = lt_setup(st, d, hp, gp, s);
  if (rc) return rc;
  LtArgs a;
  fill_args(a, st, d, n, x, t, N, hp, gp, phi, xtraj, ptraj, iters, status, d.max_iter,
            (d.flags & HJPD_FIXED_ITERS) != 0);
  const LtKernel k = lt_kernel(d.d, d.N_max, false);
  void* args[] = {&a};
  if (ev0) LT_HIP(hipEventRecord(ev0, s), "hipEventRecord");
  LT_HIP(hipLaunchKernel(k.fn, dim3(lt_grid(st, k.fn, k.threads, k.lds, n)), dim3(k.threads), args, k.lds, s),
         "linear-tanh forward");
  if (ev1) LT_HIP(hipEventRecord(ev1, s), "hipEventRecord");
  if (launches) *launches = 1;
  if (timing_valid) *timing_valid = ev0 != nullptr;
  return HJPD_OK;
}

// Buffers grow on demand and are kept; earlier work on the context may still
// use one that is replaced, so the stream is finished first.
static int grow(void** p, size_t* cap, size_t need, hipStream_t s) {
  if (need <= *cap) return HJPD_OK;
  LT_HIP(hipStreamSynchronize(s), "hipStreamSynchronize");
  if (*p) (void)hipFree(*p);
  *p = nullptr;
  *cap = 0;
  if (hipMalloc(p, need) != hipSuccess) return hjpd_fail(HJPD_ENOMEM, "linear-tanh reverse-mode buffers");
  *cap = need;
  return HJPD_OK;
}

int lt_value_grad(LtState* st, const hjpd_desc& d, int64_t n, const void* x, const void* t, const int32_t* N,
                  const void* hp, const void* gp, const void* grad_phi, int K, int E, void* phi, void* dphi_dx,
                  void* dh, void* dg, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, int* launches,
                  bool* timing_valid) {
  if (timing_valid) *timing_valid = false;
  // a captured call would keep the addresses of buffers that a later call may replace
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  LT_HIP(hipStreamIsCapturing(s, &capture), "hipStreamIsCapturing");
  if (capture != hipStreamCaptureStatusNone) return hjpd_fail(HJPD_EDEVICE, "value_grad on a stream that is being captured");
  if (E > K) E = K;
  const int n_ckpt = (K + E - 1) / E;
  const size_t CK = size_t(d.N_max + 1) * d.d;
  const size_t dd = size_t(d.d) * d.d;
  int rc = grow((void**)&st->ckpt, &st->ckpt_bytes, sizeof(float) * size_t(n) * (n_ckpt + 1) * 3 * CK, s);
  if (rc) return rc;
  const LtKernel kb = lt_kernel(d.d, d.N_max, true);
  const size_t seg_wg = sizeof(float) * size_t(lt_seg_floats(d.d, d.N_max, E));
  // several small workgroups share a CU; with long segments their buffers are
  // held to 4 GiB together, down to one workgroup a CU
  const int64_t fit = std::max<int64_t>(st->n_cu, int64_t((size_t(4) << 30) / seg_wg));
  int grid_b = int(std::min<int64_t>(lt_grid(st, kb.fn, kb.threads, kb.lds, n), fit));
  // where they do not fit the GPU's free memory, fewer workgroups take the points
  while ((rc = grow((void**)&st->seg, &st->seg_bytes, seg_wg * size_t(grid_b), s)) == HJPD_ENOMEM && grid_b > 1) {
    (void)hipGetLastError();
    grid_b = (grid_b + 1) / 2;
  }
  if (rc) return rc;
  rc = grow((void**)&st->part, &st->part_bytes, sizeof(float) * size_t(grid_b) * (3 * dd + 1), s);
  if (rc) return rc;
  rc = grow((void**)&st->scratch_i, &st->scratch_bytes, sizeof(int32_t) * 2 * size_t(n), s);
  if (rc) return rc;
  rc = lt_setup(st, d, hp, gp, s);
  if (rc) return rc;
  LtArgs a;
  fill_args(a, st, d, n, x, t, N, hp, gp, phi, nullptr, nullptr, st->scratch_i, st->scratch_i + n, K, true);
  a.ckpt = st->ckpt;
  a.ckpt_every = E;
  a.n_ckpt = n_ckpt;
  const LtKernel kf = lt_kernel(d.d, d.N_max, false);
  void* fargs[] = {&a};
  LT_HIP(hipLaunchKernel(kf.fn, dim3(lt_grid(st, kf.fn, kf.threads, kf.lds, n)), dim3(kf.threads), fargs, kf.lds, s),
         "linear-tanh forward");
  LtBwdArgs b;
  b.f = a;
  b.f.phi = nullptr;
  b.grad_phi = (const float*)grad_phi;
  b.dphi_dx = (float*)dphi_dx;
  b.seg = st->seg;
  b.part = st->part;
  b.K = K;
  void* bargs[] = {&b};
  if (ev0) LT_HIP(hipEventRecord(ev0, s), "hipEventRecord");
  LT_HIP(hipLaunchKernel(kb.fn, dim3(grid_b), dim3(kb.threads), bargs, kb.lds, s), "linear-tanh backward");
  if (ev1) LT_HIP(hipEventRecord(ev1, s), "hipEventRecord");
  const int W = int(3 * dd + 1);
  hipLaunchKernelGGL(k_lt_reduce_parts, dim3((W + 63) / 64), dim3(64 * kRedWaves), 0, s, st->part, grid_b, d.d, st->sums);
  // S = -tau M dM M
  hipLaunchKernelGGL(k_lt_mdm, dim3(d.d), dim3(4 * kLtMaxD), 0, s, st->M, st->sums + dd, d.d, -float(d.tau), st->tmp);
  hipLaunchKernelGGL(k_lt_grad_out, dim3(int((dd + 255) / 256)), dim3(256), 0, s, st->sums, st->tmp, d.d, (float*)dh,
                     (float*)dg);
  LT_HIP(hipGetLastError(), "linear-tanh gradient kernels");
  if (ev0 && ev1) {
    if (launches) *launches = 1;
    if (timing_valid) *timing_valid = true;
  }
  return HJPD_OK;
}

}  // namespace hjpd
