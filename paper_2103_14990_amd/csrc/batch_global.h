// Kernels of the batched iteration through the plant's own recursions (included by
// batch_kernels.hip).
//
// Every vector in the range of a null basis N_j is a localised trajectory: x_0 = 0, x_t = A x_{t-1}
// + B u_{t-1} on the whole network (the ring equations keep it zero outside the patch), fixed by
// its input rows N_u,j. Hence with the plant's global recursions
//   sum_j N_j W_j = [x; U],  U = sum_j N_u,j W_j,  x_0 = 0, x_t = A x_{t-1} + B U_{t-1};
//   b = sum_c x0_c o_c is the trajectory from x(0) with the input rows b_u;
//   N_j' alpha = N_u,j' g,  g_t = alpha_{u,t} + B' lam_{t+1},  lam_t = alpha_{x,t} + A' lam_{t+1},
// with one g for all column subsystems. An iteration is four launches (three on small networks):
//   bsim_fwd_kernel    per instance: forward recursion and row update (alpha, s);
//   bsim_adj_kernel    per instance: adjoint recursion (g);   (bsim_both_kernel: both)
//   bstep_kernel       per column subsystem: eta = N_u' g, tau, W = ||x0_j||^2 (tau + eta) and the
//                      subsystem's own share N_u W of U, on the matrix cores in split bf16;
//   bgather_kernel     U = sum of the shares per row subsystem, and the stopping decisions.
// What bounds it: the dense products read nx T + nu (T - 1) rows of every basis twice per
// iteration (1.03 GB at d = 3, T = 15 on the 1024-node mesh); the input rows alone are 14 of 44
// there, and W_j is no longer re-read by every row subsystem of the patch.
// Measured per iteration, 64 instances of that mesh: 496 us through the dense products (bphi 221, bpsi
// 267, bdecide 8), 253 us here (32 + 27 + 174 + 20); 64 of the 16 x 16 boxed grid 63 -> 43 us.
// The recursions run in FP32; products accumulate over fewer rows, so the iterate is closer to
// the FP64 one than through the dense bases (u(0) after 50 iterations on the 16 x 16 boxed grid:
// 4.8e-7 against 2.1e-6 relative). A plant whose A^t grows over the horizon amplifies the rounding of
// U in x; such plants keep the dense products (see kMaxGrowth in batch_kernels.hip).
#pragma once

constexpr int kSimThreads = 1024;
constexpr int kSimNE = 8;         // entries of a state row of A (or A') kept in registers
constexpr int kSimParts = 8;      // parts of an instance's row update at most
constexpr int kStepThreads = 512;
constexpr int kStepWaves = kStepThreads / 64;
constexpr int kStepRing = 4;      // K steps of basis fragments in flight per wave
constexpr int kSimStates = 4096;  // states of the network at most (two LDS buffers this far apart)

// Workgroup barrier that orders LDS accesses only: global loads and stores stay in flight across
// it (a full __syncthreads waits for every outstanding store, once per step of a recursion).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// State rows r = c N + m of A (or its transpose): a thread's own rows r = tid + i blockDim, the
// first kSimNE entries of each in registers (zero past a row's end). The count is taken per wave, so
// that the loop over the entries has no lane masks; states are two LDS buffers kSimStates apart.
template <int RPT>
struct RowEll {
  int e0[RPT], n[RPT], nw[RPT], idx[RPT][kSimNE];  // idx: byte offsets of the states
  float val[RPT][kSimNE];
  __device__ __forceinline__ void load(const int32_t *rp, const int32_t *col, const float *v, int NS) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = threadIdx.x + i * blockDim.x;
      e0[i] = r < NS ? rp[r] : 0;
      n[i] = r < NS ? rp[r + 1] - e0[i] : 0;
      int w = min(n[i], kSimNE);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, 64));
      nw[i] = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
      for (int e = 0; e < kSimNE; ++e) {
        idx[i][e] = e < n[i] ? col[e0[i] + e] * int(sizeof(float)) : 0;
        val[i][e] = e < n[i] ? v[e0[i] + e] : 0.f;
      }
    }
  }
  __device__ __forceinline__ float dot(int i, const float *x, const int32_t *col, const float *v) const {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < kSimNE; ++e) {
      if (e >= nw[i]) break;
      s += val[i][e] * *reinterpret_cast<const float *>(reinterpret_cast<const char *>(x) + idx[i][e]);
    }
    for (int e = kSimNE; e < n[i]; ++e) s += v[e0[i] + e] * x[col[e0[i] + e]];
    return s;
  }
};

// ------------------------------------------------------------------ row update between the recursions

// Block (instance b, part q of a.sim_q): forward recursion of coef b + sum_j N_j W_j over all
// states (threads over the state rows of one time step; row vectors are stored time step by time
// step, [b][l][m], so every access is coalesced), and the explicit clipped row update of the time
// steps and input rows that are q modulo a.sim_q. Streamed joins and set-up passes run the
// recursion on their own vectors and write q = M p (see BArgs phase).
// Bound by the instructions of one CU: the update of a step costs several times the recursion's,
// so the parts repeat the recursion and share the update (64 instances: 4 blocks each on 256 CUs).
template <int NX, int RPT>
__global__ __launch_bounds__(kSimThreads) void bsim_fwd_kernel(BArgs a) {
  if (a.ctl->stop) return;
  extern __shared__ __align__(16) float sim_lds[];
  const int b = blockIdx.x, part = blockIdx.y, nq = gridDim.y, tid = threadIdx.x, bd = blockDim.x;
  if (b >= a.ctl->batch) return;
  const bool cgm = a.phi_mode != 0;
  const int ph = a.phase[b];
  const bool adm = !cgm && ph < 0;
  if (!cgm && (a.ictl[b].stop || ph == 0 || ph > a.ctl->cg_k)) return;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu, nuT = nu * (T - 1), NU = N * nuT;
  const int64_t R = int64_t(N) * a.rs, plane = int64_t(a.Bmax) * R;
  const bool warm = a.ctl->warm != 0;
  const int it = a.ctl->iters + 1, cur = it & 1;
  const bool cold1 = !warm && it == 1;
  float *xa = sim_lds, *xb = xa + kSimStates, *uv = xb + kSimStates;  // two state buffers, input rows [m][nuT]
  const float coef = !adm ? 0.f : (warm ? 1.f : (it == 1 ? 0.f : (it == 2 ? 2.f : 1.f)));
  const bool use_u = cgm || warm || it >= 3;  // from a cold start tau = eta = 0 before iteration 3
  RowEll<RPT> ell;
  ell.load(a.prp, a.pcol, a.pval, NS);
  {
    const float *us = a.usum + int64_t(b) * NU, *bs = a.bu + int64_t(b) * NU;
    for (int e0 = tid; e0 < NU; e0 += 8 * bd) {  // sixteen loads in flight
      float u[8], v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int e = min(e0 + q * bd, NU - 1);
        u[q] = us[e];
        v[q] = bs[e];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e0 + q * bd < NU) {
          float x = use_u ? u[q] : 0.f;
          if (coef != 0.f) x += coef * v[q];
          uv[e0 + q * bd] = x;
        }
    }
  }
  const float rho = adm ? a.rho_b[b] : 1.f;
  const float *ap0 = a.alpha + (cur ^ 1) * plane + b * R;
  float *al0 = a.alpha + cur * plane + b * R, *s0 = a.s + b * R, *q0 = a.cg_q + b * R;
  float *apz = a.alpha + (cur ^ 1) * plane + b * R;
  float nr[RPT], bk[RPT][2];
  int ub[RPT], xi[RPT];
  double dl[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = min(tid + i * bd, NS - 1), c = r / N, m = r - c * N;
    nr[i] = a.nrm[int64_t(b) * N + m];
    dl[i] = 0.0;
    ub[i] = m * nuT;
    xi[i] = m * NX + c;
#pragma unroll
    for (int k = 0; k < 2; ++k) bk[i][k] = k < nu ? a.b_blk[int64_t(xi[i]) * nu + k] : 0.f;
  }
  struct Pre { float ap[RPT], w[RPT], lo[RPT], hi[RPT]; } pre;  // row data of this part's next step
  auto fetch = [&](int t) {
    if (!adm || t >= T) return;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int o = t * NS + min(tid + i * bd, NS - 1);
      pre.ap[i] = cold1 ? 0.f : ap0[o];
      pre.w[i] = a.wT[o];
      pre.lo[i] = a.lbT[o];
      pre.hi[i] = a.ubT[o];
    }
  };
  // explicit row solution: new alpha and s from the row value av = y - n alpha_prev
  auto update = [&](int o, float y, float n, float ap, float w, float lo, float hi, double &d) {
    const float av = y - n * ap;
    float sv, al;
    if (n > 0.f) {
      sv = rho * av / (rho + 2.f * w * n);
      sv = sv < lo ? lo : (sv > hi ? hi : sv);
      al = (sv - av) / n;
    } else {
      sv = av;
      al = 0.f;
    }
    al0[o] = al;
    s0[o] = sv;
    if (cold1) apz[o] = 0.f;
    d += double(al - ap) * double(al - ap);
  };
  auto step = [&](int t, const float *src, float *dst, bool mine) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        float y;
        if (t == 0) {
          y = coef != 0.f ? coef * a.x0[int64_t(b) * NS + xi[i]] : 0.f;
        } else {
          y = ell.dot(i, src, a.pcol, a.pval);
          const float *u = uv + ub[i] + (t - 1) * nu;
          y += bk[i][0] * u[0];
          if (nu > 1) y += bk[i][1] * u[1];
          for (int k = 2; k < nu; ++k) y += a.b_blk[int64_t(xi[i]) * nu + k] * u[k];
        }
        dst[r] = y;
        if (mine) {
          const int o = t * NS + r;
          if (adm)
            update(o, y, nr[i], pre.ap[i], pre.w[i], pre.lo[i], pre.hi[i], dl[i]);
          else
            q0[o] = y;
        }
      }
    }
    if (mine) fetch(t + nq);
    lds_barrier();
  };
  fetch(part);
  int next = part;  // this part's next time step
  for (int t = 0; t < T; t += 2) {
    bool mine = t == next;
    next += mine ? nq : 0;
    step(t, xb, xa, mine);
    if (t + 1 < T) {
      mine = t + 1 == next;
      next += mine ? nq : 0;
      step(t + 1, xa, xb, mine);
    }
  }
  // input rows, four loads in flight; this part's sum of (alpha - alpha_prev)^2 of every subsystem
  double *dld = reinterpret_cast<double *>(sim_lds);
  if (adm) {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
      if (tid + i * bd < NS) dld[tid + i * bd] = dl[i];
  }
  lds_barrier();
  for (int m = tid; m < N; m += bd) {
    const float n = a.nrm[int64_t(b) * N + m];
    double d = 0.0;
    for (int i0 = part; i0 < nuT; i0 += 4 * nq) {
      float ap[4], w[4], lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = T * NS + min(i0 + e * nq, nuT - 1) * N + m;
        ap[e] = (adm && !cold1) ? ap0[o] : 0.f;
        w[e] = a.wT[o];
        lo[e] = a.lbT[o];
        hi[e] = a.ubT[o];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e * nq;
        if (i >= nuT) break;
        const int o = T * NS + i * N + m;
        if (adm)
          update(o, uv[m * nuT + i], n, ap[e], w[e], lo[e], hi[e], d);
        else
          q0[o] = uv[m * nuT + i];
      }
    }
    if (adm) {
#pragma unroll
      for (int c = 0; c < NX; ++c) d += dld[c * N + m];
      a.dlq[(int64_t(b) * nq + part) * N + m] = d;
    }
  }
}

// One block per instance: adjoint recursion of the vector that the products of this pass project
// (the new alpha; a set-up pass's source; a streamed join's CG vector, see BArgs phase) into g,
// and the sum of the parts' (alpha - alpha_prev)^2 of every row subsystem. A chain of T - 1 steps
// with one LDS barrier each bounds it; the rows of a step are loaded four steps ahead.
template <int NX, int RPT>
__global__ __launch_bounds__(kSimThreads) void bsim_adj_kernel(BArgs a) {
  if (a.ctl->stop) return;
  extern __shared__ __align__(16) float sim_lds[];
  const int b = blockIdx.x, tid = threadIdx.x, bd = blockDim.x;
  if (b >= a.ctl->batch) return;
  const bool initp = a.init_pass != 0;
  const int ph = a.phase[b], cg_k = a.ctl->cg_k;
  if (!initp && a.ictl[b].stop) return;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu, nuT = nu * (T - 1), NU = N * nuT;
  const int64_t R = int64_t(N) * a.rs, plane = int64_t(a.Bmax) * R;
  const bool warm = a.ctl->warm != 0;
  const int it = a.ctl->iters + 1, cur = it & 1;
  auto sum_parts = [&]() {
    if (initp || ph >= 0) return;
    for (int m = tid; m < N; m += bd) {
      double x[kSimParts], d = 0.0;  // all parts in flight
#pragma unroll
      for (int q = 0; q < kSimParts; ++q) x[q] = a.dlq[(int64_t(b) * a.sim_q + min(q, a.sim_q - 1)) * N + m];
#pragma unroll
      for (int q = 0; q < kSimParts; ++q) d += q < a.sim_q ? x[q] : 0.0;
      a.dlm[int64_t(b) * N + m] = d;
    }
  };
  if (!warm && it == 1 && !initp) return sum_parts();  // alpha^1 = 0
  const float *src = initp ? a.src + int64_t(b) * a.src_bs
                     : (ph < 0 || ph > cg_k) ? a.alpha + cur * plane + b * R
                     : ph < cg_k ? a.cg_p + b * R : a.cg_x + b * R;
  float *xa = sim_lds, *xb = xa + kSimStates, *uv = xb + kSimStates;
  int rr[RPT];  // this thread's state rows (clamped)
#pragma unroll
  for (int i = 0; i < RPT; ++i) rr[i] = min(tid + i * bd, NS - 1);
  constexpr int kAhead = 4;
  float v[kAhead][RPT];
  auto fetch = [&](int t, float *f) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) f[i] = t >= 0 ? src[t * NS + rr[i]] : 0.f;
  };
#pragma unroll
  for (int q = 0; q < kAhead; ++q) fetch(T - 1 - q, v[q]);
  RowEll<RPT> ell;
  ell.load(a.trp, a.tcol, a.tval, NS);
  float bc[RPT][NX][2];  // input blocks of this thread's subsystems tid + i blockDim (first two inputs)
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int c = 0; c < NX; ++c)
#pragma unroll
      for (int k = 0; k < 2; ++k)
        bc[i][c][k] = (k < nu && tid + i * bd < N) ? a.b_blk[(int64_t(tid + i * bd) * NX + c) * nu + k] : 0.f;
  for (int m = tid; m < N; m += bd)
    for (int i0 = 0; i0 < nuT; i0 += 8) {  // eight loads in flight
      float u[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = src[T * NS + min(i0 + q, nuT - 1) * N + m];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (i0 + q < nuT) uv[m * nuT + i0 + q] = u[q];
    }
  const bool want0 = !initp && !warm && it == 2;  // lam_0: offset terms of the second cold iteration
  const int tl = want0 ? 0 : 1;
  auto step = [&](int t, const float *prev, float *dst, float *f) {  // lam_t, then g_{t-1}
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        const float l = t + 1 < T ? f[i] + ell.dot(i, prev, a.tcol, a.tval) : f[i];
        dst[r] = l;
        if (t == 0) a.lam0[int64_t(b) * NS + r] = l;
      }
    }
    fetch(t - kAhead, f);
    lds_barrier();
    if (t == 0) return;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int m = tid + i * bd;
      if (m >= N) break;
      float *u = uv + m * nuT + (t - 1) * nu, l[NX];
#pragma unroll
      for (int c = 0; c < NX; ++c) l[c] = dst[c * N + m];
      float g0 = u[0], g1 = nu > 1 ? u[1] : 0.f;
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        g0 += bc[i][c][0] * l[c];
        g1 += bc[i][c][1] * l[c];
      }
      u[0] = g0;
      if (nu > 1) u[1] = g1;
      for (int k = 2; k < nu; ++k) {
        float g = u[k];
#pragma unroll
        for (int c = 0; c < NX; ++c) g += a.b_blk[(int64_t(m) * NX + c) * nu + k] * l[c];
        u[k] = g;
      }
    }
  };
  for (int t = T - 1; t >= tl; t -= 4) {
    step(t, xb, xa, v[0]);
    if (t - 1 >= tl) step(t - 1, xa, xb, v[1]);
    if (t - 2 >= tl) step(t - 2, xb, xa, v[2]);
    if (t - 3 >= tl) step(t - 3, xa, xb, v[3]);
  }
  sum_parts();
  lds_barrier();
  for (int e = tid; e < NU; e += bd) a.gu[int64_t(b) * NU + e] = uv[e];
}

// Both recursions of one instance in one block, for networks whose rows of an instance fit on chip
// (R floats; see kSimBothLds): forward recursion into LDS, the row update of all rows at once
// from there, the adjoint recursion of the new alpha in place. ADMM iterations only; set-up passes
// and iterations with streamed joins use the two kernels.
// Bound by the chain of 2 T steps and four rounds of dependent loads; against the two kernels it saves
// a launch, alpha's way through memory, and the parts' repeated recursion: 8 x 8 grid (T = 10, 5
// instances) 9.1 + 9.6 -> 13.4 us, 16 x 16 boxed grid (T = 10, 64 instances) 15.9 + 11.6 -> 18.8 us.
// Issuing the row data's loads ahead of the recursion, or all loads ahead of the stop check,
// changed nothing.
template <int NX, int RPT>
__global__ __launch_bounds__(kSimThreads) void bsim_both_kernel(BArgs a) {
  if (a.ctl->stop) return;
  extern __shared__ __align__(16) float sim_lds[];
  __shared__ double red[kSimThreads];
  const int b = blockIdx.x, tid = threadIdx.x, bd = blockDim.x;
  if (b >= a.ctl->batch || a.ictl[b].stop) return;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu, nuT = nu * (T - 1), NU = N * nuT, rs = a.rs;
  const int64_t R = int64_t(N) * rs, plane = int64_t(a.Bmax) * R;
  const bool warm = a.ctl->warm != 0;
  const int it = a.ctl->iters + 1, cur = it & 1;
  const bool cold1 = !warm && it == 1;
  const float coef = warm ? 1.f : (it == 1 ? 0.f : (it == 2 ? 2.f : 1.f));
  const bool use_u = warm || it >= 3;  // from a cold start tau = eta = 0 before iteration 3
  float *y = sim_lds, *uv = y + T * NS;  // rows of the time steps [t][c][m], input rows [m][nuT]
  RowEll<RPT> ell, elt;
  ell.load(a.prp, a.pcol, a.pval, NS);
  {
    const float *us = a.usum + int64_t(b) * NU, *bs = a.bu + int64_t(b) * NU;
    for (int e0 = tid; e0 < NU; e0 += 4 * bd) {  // eight loads in flight
      float u[4], v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = min(e0 + q * bd, NU - 1);
        u[q] = us[e];
        v[q] = bs[e];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (e0 + q * bd < NU) {
          float x = use_u ? u[q] : 0.f;
          if (coef != 0.f) x += coef * v[q];
          uv[e0 + q * bd] = x;
        }
    }
  }
  float bk[RPT][2], bc[RPT][NX][2];  // first two inputs of the state rows, of the subsystems tid + i bd
  int ub[RPT], xi[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = min(tid + i * bd, NS - 1), c = r / N, m = r - c * N;
    ub[i] = m * nuT;
    xi[i] = m * NX + c;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      bk[i][k] = k < nu ? a.b_blk[int64_t(xi[i]) * nu + k] : 0.f;
#pragma unroll
      for (int q = 0; q < NX; ++q)
        bc[i][q][k] = (k < nu && tid + i * bd < N) ? a.b_blk[(int64_t(tid + i * bd) * NX + q) * nu + k] : 0.f;
    }
    if (tid + i * bd < NS) y[r] = coef != 0.f ? coef * a.x0[int64_t(b) * NS + xi[i]] : 0.f;
  }
  elt.load(a.trp, a.tcol, a.tval, NS);
  lds_barrier();
  for (int t = 1; t < T; ++t) {
    const float *src = y + (t - 1) * NS;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        float v = ell.dot(i, src, a.pcol, a.pval);
        const float *u = uv + ub[i] + (t - 1) * nu;
        v += bk[i][0] * u[0];
        if (nu > 1) v += bk[i][1] * u[1];
        for (int k = 2; k < nu; ++k) v += a.b_blk[int64_t(xi[i]) * nu + k] * u[k];
        y[t * NS + r] = v;
      }
    }
    lds_barrier();
  }
  // row update: thread (group g, subsystem m) takes the rows l = g, g + G, ... of m
  const float rho = a.rho_b[b];
  const float *ap0 = a.alpha + (cur ^ 1) * plane + b * R;
  float *al0 = a.alpha + cur * plane + b * R, *s0 = a.s + b * R, *apz = a.alpha + (cur ^ 1) * plane + b * R;
  const int G = bd / N, g = tid / N, m = tid - g * N;
  double d = 0.0;
  if (g < G) {
    const float n = a.nrm[int64_t(b) * N + m];
    for (int l0 = g; l0 < rs; l0 += 4 * G) {  // sixteen loads in flight
      float ap[4], w[4], lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = min(l0 + e * G, rs - 1) * N + m;
        ap[e] = cold1 ? 0.f : ap0[o];
        w[e] = a.wT[o];
        lo[e] = a.lbT[o];
        hi[e] = a.ubT[o];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int l = l0 + e * G;
        if (l >= rs) break;
        const int o = l * N + m;
        float *p = l < NX * T ? y + o : uv + m * nuT + (l - NX * T);
        const float av = *p - n * ap[e];
        float sv, al;
        if (n > 0.f) {
          sv = rho * av / (rho + 2.f * w[e] * n);
          sv = sv < lo[e] ? lo[e] : (sv > hi[e] ? hi[e] : sv);
          al = (sv - av) / n;
        } else {
          sv = av;
          al = 0.f;
        }
        al0[o] = al;
        s0[o] = sv;
        if (cold1) apz[o] = 0.f;
        *p = al;
        d += double(al - ap[e]) * double(al - ap[e]);
      }
    }
  }
  red[tid] = d;
  lds_barrier();
  if (tid < N) {
    for (int q = 1; q < G; ++q) d += red[q * N + tid];
    a.dlm[int64_t(b) * N + tid] = d;
  }
  if (cold1) return;  // alpha^1 = 0
  const int tl = !warm && it == 2 ? 0 : 1;  // lam_0: offset terms of the second cold iteration
  for (int t = T - 1; t >= tl; --t) {       // lam_t, then g_{t-1}
    float *lam = y + t * NS;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        float v = lam[r];
        if (t + 1 < T) v += elt.dot(i, lam + NS, a.tcol, a.tval);
        lam[r] = v;
        if (t == 0) a.lam0[int64_t(b) * NS + r] = v;
      }
    }
    lds_barrier();
    if (t == 0) break;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int mm = tid + i * bd;
      if (mm >= N) break;
      float *u = uv + mm * nuT + (t - 1) * nu;
      for (int k = 0; k < nu; ++k) {
        float x = u[k];
#pragma unroll
        for (int q = 0; q < NX; ++q)
          x += (k < 2 ? (k == 0 ? bc[i][q][0] : bc[i][q][1]) : a.b_blk[(int64_t(mm) * NX + q) * nu + k]) * lam[q * N + mm];
        u[k] = x;
      }
    }
  }
  lds_barrier();
  for (int e = tid; e < NU; e += bd) a.gu[int64_t(b) * NU + e] = uv[e];
}

// Trajectory start of slot slots[x] (or x): with the predicted input rows u of yhat, the state
// rows y from x(0) by the plant; r = y - b, which is the trajectory from 0 with the input rows
// u - b_u; p = r, x = 0, r'r; alpha^0 = -2 w y / rho into plane pl (both planes when pl < 0: a
// streamed join, read by whichever iteration starts).
template <int NX, int RPT>
__global__ __launch_bounds__(kSimThreads) void bsim_start_kernel(BArgs a, const int32_t *slots, int pl) {
  extern __shared__ __align__(16) float sim_lds[];
  __shared__ double red[kSimThreads / 64];
  const int b = slots ? slots[blockIdx.x] : blockIdx.x, tid = threadIdx.x, bd = blockDim.x;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu, nuT = nu * (T - 1), NU = N * nuT;
  const int64_t R = int64_t(N) * a.rs, plane = int64_t(a.Bmax) * R;
  float *ya = sim_lds, *yb = ya + kSimStates, *ra = yb + kSimStates, *rb = ra + kSimStates, *uv = rb + kSimStates;
  const float rho = a.rho_b[b];
  const float *yh = a.yhat + b * R;
  float *al = a.alpha + int64_t(pl < 0 ? 0 : pl) * plane + b * R;
  float *r0 = a.cg_r + b * R, *p0 = a.cg_p + b * R, *x0 = a.cg_x + b * R;
  double acc = 0.0;
  auto put = [&](int64_t o, float y, float r) {
    const float a0 = -2.f * a.wT[o] * y / rho;
    al[o] = a0;
    if (pl < 0) al[plane + o] = a0;
    r0[o] = r;
    p0[o] = r;
    x0[o] = 0.f;
    acc += double(r) * double(r);
  };
  for (int e = tid; e < NU; e += bd) {
    const int m = e / nuT, i = e - m * nuT;
    const float u = yh[int64_t(m) * a.rs + NX * T + i];
    uv[e] = u;
    put(int64_t(T) * NS + int64_t(i) * N + m, u, u - a.bu[int64_t(b) * NU + e]);
  }
  RowEll<RPT> ell;
  ell.load(a.prp, a.pcol, a.pval, NS);
  for (int t = 0; t < T; ++t) {
    const float *ys = (t & 1) ? ya : yb, *rsrc = (t & 1) ? ra : rb;
    float *yd = (t & 1) ? yb : ya, *rd = (t & 1) ? rb : ra;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        const int c = r / N, m = r - c * N;
        float y, d;
        if (t == 0) {
          y = a.x0[int64_t(b) * NS + m * NX + c];
          d = 0.f;
        } else {
          y = ell.dot(i, ys, a.pcol, a.pval);
          d = ell.dot(i, rsrc, a.pcol, a.pval);
          for (int k = 0; k < nu; ++k) {
            const float bc = a.b_blk[(int64_t(m) * NX + c) * nu + k];
            const int e = m * nuT + (t - 1) * nu + k;
            y += bc * uv[e];
            d += bc * (uv[e] - a.bu[int64_t(b) * NU + e]);
          }
        }
        yd[r] = y;
        rd[r] = d;
        put(int64_t(t) * NS + r, y, d);
      }
    }
    lds_barrier();
  }
  acc = wsum(acc);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < bd / 64; ++w) s += red[w];
    a.cg_rr[b] = a.cg_rrn[b] = s;
  }
}

// ------------------------------------------------------------------ products with the input rows

// One block per (column subsystem j, 16 NT instances): eta = N_u' g_j (k x instances), the k-space
// update and residual terms, W = ||x0_j||^2 (tau + eta), and j's share N_u W of the input rows.
// g_j (the input rows of j's patch) is staged once in LDS as bf16 hi + lo, then W in its place, so
// both products stream the basis fragments with no barrier inside; wave wm of kStepWaves / WN
// owns the M tiles wm, wm + kStepWaves / WN, ... for instance tiles wn NT / WN ... (WN = NT
// where the basis has so few tiles that waves would be idle).
// The instance halves of one j are dispatched 8 blocks apart: the same XCD, so the second finds
// the fragments in its L2. Bound by the bytes that miss the L2s (1024-node mesh, 64 instances: 560 MB
// read, of which the two fragment orders 375 MB, tau and eta 78 MB, and 165 MB written; 171 us).
template <int NX, int MT, int NT, int WN>
__global__ __launch_bounds__(kStepThreads) __attribute__((amdgpu_waves_per_eu(4))) void bstep_kernel(BArgs a) {
  if (a.ctl->stop) return;
  constexpr int NI = 16 * NT, NTW = NT / WN, WM = kStepWaves / WN;
  extern __shared__ __align__(16) unsigned char step_lds[];
  __shared__ int s_sub[kMaxPatch];
  __shared__ double red_e[kStepWaves][NI], red_d[kStepWaves][NI], red_l[kStepThreads / NI][NI], red_od[NI][NX];
  const int B = a.ctl->batch, nh = (a.Bmax + NI - 1) / NI;
  const int grp = blockIdx.x / (8 * nh), rem = blockIdx.x % (8 * nh);
  const int jj = grp * 8 + (rem & 7), b0 = (rem >> 3) * NI;
  if (jj >= a.N || b0 >= B) return;
  const StepDesc ds = a.sdesc[jj];
  const int j = ds.j, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave & (WN - 1), wm = wave / WN;
  const bool warm = a.ctl->warm != 0, initp = a.init_pass != 0;
  const int it = a.ctl->iters + 1, cur = it & 1, cg_k = a.ctl->cg_k;
  const bool cold2 = !warm && it == 2 && !initp;
  double *rr = a.rres;  // [Bmax][2][N] residual maxima of every column subsystem
  if (!warm && it == 1 && !initp) {  // alpha^1 = 0: Psi^1 = o, residuals ||o_c||, eta stays 0
    if (tid < NI && b0 + tid < B) {
      double mx = 0.0;
#pragma unroll
      for (int c = 0; c < NX; ++c) mx = fmax(mx, sqrt(a.onorm2[j * NX + c]));
      rr[int64_t(b0 + tid) * 2 * a.N + j] = mx;
      rr[(int64_t(b0 + tid) * 2 + 1) * a.N + j] = mx;
    }
    return;
  }
  const int64_t tb = ds.tb, koff = ds.koff;
  const int p = ds.p, nuT = a.nu * (a.T - 1), mu = p * nuT, k = ds.k;
  const int nks = (mu + 31) >> 5, mu32 = nks * 32, KS = mu32 + 8;
  const int nmt = (k + 15) >> 4, nk2 = (k + 31) >> 5, K2 = nk2 * 32 + 8;
  const int64_t NU = int64_t(a.N) * nuT;
  __bf16 *gh = reinterpret_cast<__bf16 *>(step_lds), *gl = gh + NI * KS;  // [NI][KS] each
  // Basis fragments: kStepRing K steps of this wave are in flight at any time (the first ones during
  // the staging of g); a slot is loaded again as soon as its step is done, and the last chunk of a
  // sequence loads nothing (conditional loads inside a chunk would cost the count in flight).
  const int nt_w = max(0, min(MT, (nmt - wm + WM - 1) / WM));  // tiles of this wave
  bf16x8 fh[kStepRing], fl[kStepRing];
  auto ld = [&](int q, const __bf16 *f) {
    fh[q] = load8(f);
    fl[q] = load8(f + 512);
  };
  const __bf16 *fu = a.ngu + ds.uo + int64_t(wm) * nks * 1024 + lane * 8;
  if (tid < p) s_sub[tid] = a.tile_rsub[tb + tid];
  if (nt_w > 0) {
#pragma unroll
    for (int q = 0; q < kStepRing; ++q) ld(q, fu + min(q, nks - 1) * 1024);
  }
  lds_barrier();
  // residual input: this thread's share of sum_{m in P(j)} ||(alpha - alpha_prev) on m||^2
  double sdl = 0.0;
  {
    const int bb = tid % NI;
    if (b0 + bb < B && !initp)
      for (int t = tid / NI; t < p; t += kStepThreads / NI) sdl += a.dlm[int64_t(b0 + bb) * a.N + s_sub[t]];
  }
  // staging: wave w takes instances w, w + 8, ..., lanes consecutive input rows (member-major)
  const float inv = 1.f / float(nuT);
  constexpr int NB = NI / kStepWaves;  // instances per wave
  for (int q0 = 0; q0 < mu32; q0 += 256) {
    float v[4][NB];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = q0 + 64 * q + lane;
      const bool ok = kk < mu;
      const int ti = ok ? int((float(kk) + 0.5f) * inv) : 0;
      const int64_t off = ok ? int64_t(s_sub[ti]) * nuT + (kk - ti * nuT) : 0;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int bb = b0 + wave + kStepWaves * i;
        const float x = a.gu[int64_t(bb < B ? bb : 0) * NU + off];
        v[q][i] = (ok && bb < B) ? x : 0.f;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = q0 + 64 * q + lane;
      if (kk < mu32)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const __bf16 h = static_cast<__bf16>(v[q][i]);
          gh[(wave + kStepWaves * i) * KS + kk] = h;
          gl[(wave + kStepWaves * i) * KS + kk] = static_cast<__bf16>(v[q][i] - static_cast<float>(h));
        }
    }
  }
  if (cold2) {
    // offset terms sum_rows alpha o_c = lam_0[j, c] + sum_rows g o_c over the input rows
    const int ld4 = (p * a.rs + 3) & ~3, nxT = NX * a.T;
    for (int i = 0; i < NB; ++i) {
      const int bb = b0 + wave + kStepWaves * i;
      double od[NX];
#pragma unroll
      for (int c = 0; c < NX; ++c) od[c] = 0.0;
      for (int kk = lane; kk < mu; kk += 64) {
        const int ti = kk / nuT, ii = kk - ti * nuT;
        const double g = bb < B ? double(a.gu[int64_t(bb) * NU + int64_t(s_sub[ti]) * nuT + ii]) : 0.0;
#pragma unroll
        for (int c = 0; c < NX; ++c)
          od[c] += g * double(a.off[ds.offp + int64_t(c) * ld4 + ti * a.rs + nxT + ii]);
      }
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        const double s = wsum(od[c]);
        if (lane == 0)
          red_od[wave + kStepWaves * i][c] = bb < B ? s + double(a.lam0[int64_t(bb) * a.N * NX + c * a.N + j]) : 0.0;
      }
    }
  }
  f32x4 acc[MT][NTW];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int n = 0; n < NTW; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  lds_barrier();
  const int kr = 8 * (lane >> 4);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if (t >= nt_w) break;
    auto mul = [&](int q, int ks) {
      if (ks >= nks) return;
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        const int row = ((wn * NTW + n) * 16 + (lane & 15)) * KS + ks * 32 + kr;
        const bf16x8 bh = *reinterpret_cast<const bf16x8 *>(gh + row);
        const bf16x8 bl = *reinterpret_cast<const bf16x8 *>(gl + row);
        acc[t][n] = mfma3(fh[q], fl[q], bh, bl, acc[t][n]);
      }
    };
    const __bf16 *ft = fu + t * WM * nks * 1024;
    int c0 = 0;
    for (; c0 + kStepRing < nks; c0 += kStepRing) {
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) {
        mul(q, c0 + q);
        ld(q, ft + min(c0 + kStepRing + q, nks - 1) * 1024);
        __builtin_amdgcn_sched_barrier(0);  // the reload stays ahead of the next products
      }
    }
    if (t + 1 < nt_w) {
      ft += WM * nks * 1024;
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) {
        mul(q, c0 + q);
        ld(q, ft + min(q, nks - 1) * 1024);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) mul(q, c0 + q);
    }
  }
  // k-space update: eta, tau, residual terms and W; lane holds basis rows 4 (lane / 16) + e of its
  // tile. W replaces g in LDS ([NI][K2] hi, then lo), zero past k.
  const bool want_w = !(initp && a.wmode == 0);
  const int64_t eplane = a.ktot * a.Bmax;
  float *tau0 = a.tau + koff * a.Bmax, *etac = a.eta + koff * a.Bmax + (cur ? eplane : 0);
  float *etap = a.eta + koff * a.Bmax + (cur ? 0 : eplane), *dst0 = a.dst_k + koff * a.Bmax;
  __bf16 *wh = reinterpret_cast<__bf16 *>(step_lds), *wl = wh + NI * K2;
  double e2[NTW], d2[NTW];
  float tv[MT][NTW][4], ev[MT][NTW][4];
#pragma unroll
  for (int n = 0; n < NTW; ++n) {
    e2[n] = d2[n] = 0.0;
    const int b = b0 + (wn * NTW + n) * 16 + (lane & 15);
    const bool act = b < B && (initp || !a.ictl[b].stop);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (t >= nt_w) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = (wm + WM * t) * 16 + 4 * (lane >> 4) + e;
        const bool ok = act && i < k && !cold2;  // tau = eta = 0 before the second cold iteration
        const int ki = ok ? i * a.Bmax + b : 0;
        const float tx = tau0[ki], ex = etap[ki];
        tv[t][n][e] = ok ? tx : 0.f;
        ev[t][n][e] = ok ? ex : 0.f;
      }
    }
  }
  lds_barrier();  // every read of g is done
#pragma unroll
  for (int n = 0; n < NTW; ++n) {
    const int bl_ = (wn * NTW + n) * 16 + (lane & 15), b = b0 + bl_;
    const bool act = b < B && (initp || !a.ictl[b].stop);
    const int ph = (initp || b >= B) ? -1 : a.phase[b];
    const float xj = b < B ? a.xn[int64_t(b) * a.N + j] : 0.f;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if ((wm + WM * t) * 16 >= nk2 * 32) break;  // past the padded k
      const int i0 = (wm + WM * t) * 16 + 4 * (lane >> 4);
      __bf16 h4[4], l4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e;
        float wv = 0.f;
        if (act && i < k) {
          const int ki = i * a.Bmax + b;
          const float en = acc[t][n][e];
          if (initp) {
            dst0[ki] = en;
            wv = xj * (a.wmode == 2 ? tv[t][n][e] + en : en);
          } else if (ph < 0) {
            const float tn = tv[t][n][e] + en;
            etac[ki] = en;
            tau0[ki] = tn;
            e2[n] += double(en) * double(en);
            d2[n] += double(en - ev[t][n][e]) * double(en - ev[t][n][e]);
            wv = xj * (tn + en);
          } else if (ph < cg_k) {  // streamed join: the start's projections, as the set-up passes do them
            etac[ki] = en;
            wv = xj * en;
          } else if (ph == cg_k) {
            tau0[ki] = en;
          } else {  // eta^0 into both planes: the joiner's first iteration may have either parity
            etac[ki] = en;
            etap[ki] = en;
            wv = xj * (tv[t][n][e] + en);
          }
        }
        h4[e] = static_cast<__bf16>(wv);
        l4[e] = static_cast<__bf16>(wv - static_cast<float>(h4[e]));
      }
      if (want_w) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<bf16x4 *>(wh + bl_ * K2 + i0) = bf16x4{h4[0], h4[1], h4[2], h4[3]};
        *reinterpret_cast<bf16x4 *>(wl + bl_ * K2 + i0) = bf16x4{l4[0], l4[1], l4[2], l4[3]};
      }
    }
  }
  if (!initp) {
#pragma unroll
    for (int n = 0; n < NTW; ++n) {  // lanes l, l^16, l^32, l^48 share an instance
      e2[n] += __shfl_xor(e2[n], 16, 64);
      e2[n] += __shfl_xor(e2[n], 32, 64);
      d2[n] += __shfl_xor(d2[n], 16, 64);
      d2[n] += __shfl_xor(d2[n], 32, 64);
      if (lane < 16) {
        red_e[wave][(wn * NTW + n) * 16 + lane] = e2[n];
        red_d[wave][(wn * NTW + n) * 16 + lane] = d2[n];
      }
    }
    red_l[tid / NI][tid % NI] = sdl;
  }
  // second product's first fragments (row tiles rt = wm, wm + WM, ... of N_u W)
  const int nrt = (mu + 15) >> 4;
  const __bf16 *fv = a.ngv + ds.vo + lane * 8;
  if (want_w && nk2 > 0 && wm < nrt) {
#pragma unroll
    for (int q = 0; q < kStepRing; ++q) ld(q, fv + (int64_t(wm) * nk2 + min(q, nk2 - 1)) * 1024);
  }
  lds_barrier();
  if (!initp && tid < NI && b0 + tid < B && !a.ictl[b0 + tid].stop && a.phase[b0 + tid] < 0) {
    const int b = b0 + tid, w0 = (tid / 16) / NTW;  // the waves wn that hold this instance's tile
    double se = 0.0, sd = 0.0, sl = 0.0;
    for (int w = w0; w < kStepWaves; w += WN) {
      se += red_e[w][tid];
      sd += red_d[w][tid];
    }
    for (int q = 0; q < kStepThreads / NI; ++q) sl += red_l[q][tid];
    double mp = 0.0, md = 0.0;
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      const double xc = double(a.x0[int64_t(b) * a.N * NX + j * NX + c]);
      const double rd = fabs(xc) * sqrt(se);
      const double rp2 = cold2 ? a.onorm2[j * NX + c] + 2.0 * xc * red_od[tid][c] + xc * xc * (sl - se)
                               : xc * xc * (sl - sd);
      const double rp = sqrt(fmax(rp2, 0.0));
      mp = (rp > mp || rp != rp || rp2 != rp2) ? (rp2 != rp2 ? rp2 : rp) : mp;
      md = (rd > md || rd != rd) ? rd : md;
    }
    rr[int64_t(b) * 2 * a.N + j] = mp;
    rr[(int64_t(b) * 2 + 1) * a.N + j] = md;
  }
  if (!want_w) return;
  for (int rt = wm; rt < nrt; rt += WM) {
    f32x4 c[NTW];
#pragma unroll
    for (int n = 0; n < NTW; ++n) c[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](int q, int ks) {
      if (ks >= nk2) return;
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        const int row = ((wn * NTW + n) * 16 + (lane & 15)) * K2 + ks * 32 + kr;
        const bf16x8 bh = *reinterpret_cast<const bf16x8 *>(wh + row);
        const bf16x8 bl = *reinterpret_cast<const bf16x8 *>(wl + row);
        c[n] = mfma3(fh[q], fl[q], bh, bl, c[n]);
      }
    };
    const __bf16 *ft = fv + rt * nk2 * 1024;
    int c0 = 0;
    for (; c0 + kStepRing < nk2; c0 += kStepRing) {
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) {
        mul(q, c0 + q);
        ld(q, ft + min(c0 + kStepRing + q, nk2 - 1) * 1024);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (rt + WM < nrt && nk2 > 0) {
      ft += WM * nk2 * 1024;
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) {
        mul(q, c0 + q);
        ld(q, ft + min(q, nk2 - 1) * 1024);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int q = 0; q < kStepRing; ++q) mul(q, c0 + q);
    }
#pragma unroll
    for (int n = 0; n < NTW; ++n) {
      const int col = b0 + (wn * NTW + n) * 16;
      if (col >= a.Bw) break;  // past the rows of the shares
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = rt * 16 + 4 * (lane >> 4) + e;
        if (row < mu) a.upart[(tb * nuT + row) * a.Bw + col + (lane & 15)] = c[n][e];
      }
    }
  }
}

// ------------------------------------------------------------------ sum of the shares, decisions

// Blocks 0..N-1: U of row subsystem m = sum over its tiles (column subsystems of its patch, in
// order) of their shares, [tile][nuT][Bw] -> [b][m][nuT] through LDS. Blocks N..: the stopping
// decision of one instance each from the residuals of every column subsystem; the last one to
// finish publishes the iteration count and the all-stopped flag (set-up passes: none).
__global__ __launch_bounds__(256) void bgather_kernel(BArgs a) {
  extern __shared__ __align__(16) float g_lds[];
  const int tid = threadIdx.x, B = a.ctl->batch, N = a.N;
  if (int(blockIdx.x) < N) {
    const int m = blockIdx.x, nuT = a.nu * (a.T - 1), B4 = (B + 3) >> 2, ldb = nuT | 1;
    const int64_t q0 = a.rt_ptr[m];
    const int pm = int(a.rt_ptr[m + 1] - q0);
    __shared__ int64_t s_t[kMaxPatch];
    __shared__ int s_stop;  // one read for the block: the launch's decisions may set it meanwhile
    if (tid == 0) s_stop = a.ctl->stop;
    if (tid < pm) s_t[tid] = a.rt_tile[q0 + tid] * nuT * a.Bw;
    __syncthreads();
    if (s_stop) return;
    for (int e = tid; e < nuT * B4; e += 256) {
      const int i = e / B4, b4 = e - i * B4;
      const float *src = a.upart + int64_t(i) * a.Bw + 4 * b4;
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
      for (int t = 0; t < pm; t += 8) {  // eight loads in flight, the last batch masked
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4 *>(src + s_t[min(t + u, pm - 1)]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (t + u < pm) s += v[u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) g_lds[(4 * b4 + u) * ldb + i] = s[u];
    }
    __syncthreads();
    const int64_t NU = int64_t(N) * nuT;
    for (int e = tid; e < B * nuT; e += 256) {
      const int b = e / nuT, i = e - b * nuT;
      a.usum[b * NU + int64_t(m) * nuT + i] = g_lds[b * ldb + i];
    }
    return;
  }
  if (a.init_pass || a.ctl->stop) return;  // (set after every deciding block has read it)
  const int b = blockIdx.x - N;
  if (b >= B) return;
  __shared__ double rm[2][4];
  Ctl *c = a.ctl;
  const int it = c->iters + 1;
  const double *rr = a.rres + int64_t(b) * 2 * N;
  double mp = 0.0, md = 0.0;
  auto worse = [](double x, double y) { return (y > x || y != y) ? y : x; };  // NaN propagates
  for (int j = tid; j < N; j += 256) {
    mp = worse(mp, rr[j]);
    md = worse(md, rr[N + j]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mp = worse(mp, __shfl_xor(mp, o, 64));
    md = worse(md, __shfl_xor(md, o, 64));
  }
  if ((tid & 63) == 0) {
    rm[0][tid >> 6] = mp;
    rm[1][tid >> 6] = md;
  }
  __syncthreads();
  if (tid != 0) return;
  for (int w = 1; w < 4; ++w) {
    mp = worse(mp, rm[0][w]);
    md = worse(md, rm[1][w]);
  }
  BCtl &ic = a.ictl[b];
  bool stop = ic.stop != 0;
  const int ph = a.phase[b];
  if (!stop && ph >= 0) {  // streamed join: its start runs; no decision yet
    if (ph + 1 > c->cg_k + 1) {
      a.phase[b] = -1;
      ic.it0 = it;  // its first ADMM iteration is the next one
    } else {
      a.phase[b] = ph + 1;
    }
  } else if (!stop) {
    const int iters = it - ic.it0;
    ic.iters = iters;
    ic.last_rp = mp;
    ic.last_rd = md;
    if (!(mp == mp) || !(md == md) || isinf(mp) || isinf(md)) {
      ic.numeric = 1;
      stop = true;
    } else if (mp <= c->eps && md <= c->eps) {
      ic.converged = 1;
      stop = true;
    } else if (iters >= c->max_iter) {
      stop = true;
    }
    if (stop) {
      ic.stop = 1;
    } else {
      atomicMax(&c->rp_bits, ord_bits(mp));
      atomicMax(&c->rd_bits, ord_bits(md));
    }
  }
  if (stop) atomicAdd(&c->n_stop, 1u);
  __threadfence();
  if (atomicAdd(&c->done_count, 1u) != unsigned(B) - 1) return;
  __threadfence();
  c->iters = it;
  c->last_rp = __longlong_as_double(static_cast<long long>(atomicExch(&c->rp_bits, 0ull)));
  c->last_rd = __longlong_as_double(static_cast<long long>(atomicExch(&c->rd_bits, 0ull)));
  if (atomicExch(&c->n_stop, 0u) == unsigned(B)) c->stop = 1;
  atomicExch(&c->done_count, 0u);
}

// ------------------------------------------------------------------ set-up

// Fragments of the input rows of every null basis (bf16 hi, lo 512 further): ngu (M = basis, K =
// input row) and ngv (M = input row, K = basis); input rows member-major.
__global__ void bgfrag_kernel(const double *__restrict__ nb, const int64_t *__restrict__ nb_off,
                              const int32_t *__restrict__ kdim, const int64_t *__restrict__ tile_off,
                              const int64_t *__restrict__ koff, const int64_t *__restrict__ ngu_off,
                              const int64_t *__restrict__ ngv_off, int rs, int nxT, __bf16 *__restrict__ ngu,
                              __bf16 *__restrict__ ngv) {
  const int j = blockIdx.x, nuT = rs - nxT;
  const int p = int(tile_off[j + 1] - tile_off[j]), D = p * rs, ld = (D + 3) & ~3, k = kdim[j], mu = p * nuT;
  const int nks = (mu + 31) >> 5, nk2 = int(koff[j + 1] - koff[j]) >> 5;
  const double *Nj = nb + nb_off[j];
  for (int64_t e = int64_t(blockIdx.y) * blockDim.x + threadIdx.x; e < int64_t(k) * mu;
       e += int64_t(gridDim.y) * blockDim.x) {
    const int i = int(e / mu), kk = int(e % mu), ti = kk / nuT;
    const float x = float(Nj[int64_t(i) * ld + ti * rs + nxT + (kk - ti * nuT)]);
    const __bf16 h = static_cast<__bf16>(x), lo = static_cast<__bf16>(x - static_cast<float>(h));
    const int64_t u = ngu_off[j] + (int64_t(i / 16) * nks + kk / 32) * 1024 + ((i % 16) + 16 * ((kk % 32) / 8)) * 8 + kk % 8;
    ngu[u] = h;
    ngu[u + 512] = lo;
    const int64_t v = ngv_off[j] + (int64_t(kk / 16) * nk2 + i / 32) * 1024 + ((kk % 16) + 16 * ((i % 32) / 8)) * 8 + i % 8;
    ngv[v] = h;
    ngv[v + 512] = lo;
  }
}
