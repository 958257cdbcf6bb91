// Single-instance iteration in the compact form of Algorithm 2 (included by admm_kernels.hip).
//
// From the cold start every iterate is Psi[:,c] = o_c + x0_c N_j tau_j, Lambda[:,c] = x0_c (I - N_j
// N_j') alpha with one row scalar alpha_r (Phi row = v + alpha_r x_r), eta_j = N_j' alpha and
// tau_j = the running sum of eta_j, so an iteration reads each basis for one vector instead of
// nx, touches no Phi, Psi or Lambda tile, and is two launches:
//   crow_kernel   per row subsystem: rows of b + sum_j ||x0_j||^2 N_j (tau_j + eta_j) - n alpha from
//                 the units' shares, the clipped row update; an extra block decides the
//                 previous iteration;
//   cstep_kernel  per unit of basis vectors: eta, tau, the residual sums, and the unit's share of
//                 the next row products from the same registers.
// On large networks the products run with the input rows of the bases, between the plant's global
// recursions (sum_j N_j W_j is one trajectory of the plant, N_j' alpha = N_u,j' g with one adjoint
// vector g for all j): csim_fwd_kernel, csim_adj_kernel, cstep_kernel, crow_kernel. On the smallest
// ones csolve_kernel runs a whole solve in one workgroup with the bases in LDS.
// After the stop cexpand_kernel writes Phi, Psi and Lambda (the certificate's and the caller's).
// The iterates are those of the standard form up to rounding: same counts in FP64.
// Measured, us per iteration, the standard form's best schedule -> here: 10-node chain FP64 (d = 1,
// T = 5) 14.6 -> 4.3 (one workgroup); paper's chain of 100 FP64 23.3 -> 11.4 (whole bases: crow 4.8 +
// cstep 6.7); 1024-node mesh (d = 3, T = 15) FP64 255 -> 148 and FP32 146 -> 85 (input rows: csim_fwd
// 30 / 24, csim_adj 28 / 19, cstep 81 / 36, crow 9 / 8; whole bases: 315 and 151).
// Which form a problem uses is chosen by timing at setup: whole bases win where the two
// recursions' 2 T dependent steps cost more than the state rows' bytes, one workgroup where a
// launch costs more than an iteration.
#pragma once

constexpr int kCRowThreads = 512;
constexpr int kCStepRegs = 2;     // vectors of rows per lane in registers
constexpr int kCSimThreads = 1024;
constexpr int kCSimNE = 8;        // entries of a state row of A (or A') kept in registers
constexpr int kCParts = 16;       // blocks that share the row update of csim_fwd_kernel
constexpr int kCMaxStates = 4096;

// One tile of a row subsystem (in the order of rt_tile): its rows' first element in the whole bases,
// stride and number of the basis vectors, their first k-space index, column subsystem.
struct CTile {
  uint32_t o;
  int32_t ld, k, ko, j, pad;
};

// Unit of basis vectors: column subsystem, first vector, patch size, null-space dimension, and the
// offsets of its tiles, basis, k-space vectors and share of the row products.
struct CUnit {
  int32_t j, i0, p, k;
  int64_t tb, bo, ko, so;
};

template <typename Tf>
struct CArgs {
  // rows per subsystem that the products read (rs: whole bases; nu (T - 1): input rows), the bases
  // in that form (column-major, leading dimension a multiple of 4), and the vectors in k-space
  int32_t rows, glob, n_units;
  const Tf *basis;
  const int64_t *boff;   // [N+1]
  const int64_t *koff;   // [N+1]
  const CUnit *unit;     // [n_units]
  const int32_t *ufirst; // [N+1] first unit of each column subsystem (units of one j consecutive)
  const int32_t *rsub;   // [n_tiles] row subsystem of each tile
  const CTile *ct;       // [n_tiles] row side (csolve_kernel)
  Tf *share;             // [units][patch rows] ||x0_j||^2 N_j (tau + eta) over the unit's vectors
  const int32_t *sptr;   // [N+1] row side: first entry of each row subsystem in soff
  const uint32_t *soff;  // rows of a row subsystem in the shares (tiles in order, units of each in order)
  const double *on2;     // [N nx] ||o_c||^2
  Tf *al;                // [3][R] row multipliers by iteration mod 3
  Tf *s;                 // [2][R] row values (Phi x0) by iteration parity
  Tf *bv;                // rows of b: [R], or its input rows [nuT][N]
  Tf *tau, *eta, *v;     // [K], [K], [2][K] (tau + eta by iteration parity)
  Tf *xn;                // [N] ||x0_j||^2
  Tf *us, *g;            // input rows [nuT][N] of the summed products, and of the adjoint recursion
  Tf *lam0;              // [nx][N]
  double *dlq;           // [1 + kCParts][N] sums of (alpha - alpha_prev)^2 of every row subsystem
  double *part;          // [n_units][2] sums of eta^2 and (eta - eta_prev)^2
  double *sdl, *od;      // [N], [N][nx]
  // state rows c N + m of A and A' (CSR), input blocks, row data in the order of alpha
  const int32_t *prp, *pcol, *trp, *tcol;
  const Tf *pval, *tval, *bblk, *w, *lb, *ub;
};

template <typename Tf>
__device__ __forceinline__ int64_t crow(const KArgs<Tf> &a, const CArgs<Tf> &c, int m, int l) {
  return c.glob ? int64_t(l) * a.N + m : int64_t(m) * a.rs + l;
}

// Column norms and maxima of iteration `it` from the units' sums: NaN propagates.
template <typename Tf, int NX>
__device__ __forceinline__ void cresiduals(const KArgs<Tf> &a, const CArgs<Tf> &c, int it, int j, double *mp,
                                           double *md) {
  double se = 0.0, sd = 0.0;
  const double sl = c.sdl[j];
  for (int u = c.ufirst[j]; u < c.ufirst[j + 1]; ++u) {
    se += c.part[2 * u];
    sd += c.part[2 * u + 1];
  }
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    double rp, rd;
    const double xc = double(a.x0f[j * NX + q]);
    if (it == 1) {
      rp = rd = sqrt(c.on2[j * NX + q]);
    } else {
      rd = fabs(xc) * sqrt(se);
      const double r2 = it == 2 ? c.on2[j * NX + q] + 2.0 * xc * c.od[j * NX + q] + xc * xc * (sl - se)
                                : xc * xc * (sl - sd);
      rp = r2 != r2 ? r2 : sqrt(fmax(r2, 0.0));
    }
    *mp = (rp > *mp || rp != rp) ? rp : *mp;
    *md = (rd > *md || rd != rd) ? rd : *md;
  }
}

// The decision of the latest finished iteration (c_psi), if it is still open; one block. With
// `advance` it also opens iteration c_psi + 1 for the products that follow.
// crow_kernel and csim_fwd_kernel decide in a block beside the ones that work, so `stop` can change
// under those: all of their blocks go by c_halt instead, which only cstep_kernel and
// cdecide_kernel write, in launches whose blocks do not read it. The launch that decides so always
// runs in full (its rows are of the iteration after the stop: planes that nothing reads), and the
// waves of a block agree at every barrier.
template <typename Tf, int NX>
__device__ __forceinline__ void cdecide(const KArgs<Tf> &a, const CArgs<Tf> &c, bool advance) {
  __shared__ double rp_s[16], rd_s[16];
  Ctl *k = a.ctl;
  const int it = k->c_psi, tid = threadIdx.x;
  if (it > k->iters) {
    double mp = 0.0, md = 0.0;
    for (int j = tid; j < a.N; j += blockDim.x) cresiduals<Tf, NX>(a, c, it, j, &mp, &md);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double op = __shfl_xor(mp, o, 64), od = __shfl_xor(md, o, 64);
      mp = (op > mp || op != op) ? op : mp;
      md = (od > md || od != od) ? od : md;
    }
    if ((tid & 63) == 0) {
      rp_s[tid >> 6] = mp;
      rd_s[tid >> 6] = md;
    }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < int(blockDim.x >> 6); ++w) {
        mp = (rp_s[w] > mp || rp_s[w] != rp_s[w]) ? rp_s[w] : mp;
        md = (rd_s[w] > md || rd_s[w] != rd_s[w]) ? rd_s[w] : md;
      }
      decide(k, it, mp, md);
    }
  }
  if (advance && tid == 0) k->c_phi = it + 1;
}

template <typename Tf, int NX>
__global__ __launch_bounds__(kCSimThreads) void cdecide_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  if (a.ctl->stop) return;  // (published by a cstep_kernel since)
  cdecide<Tf, NX>(a, c, false);
  if (threadIdx.x == 0) a.ctl->c_halt = a.ctl->stop;  // its own write
}

// Per row subsystem m: x0, ||x0_m||^2, ||x_r||^2 and the rows of b that the iteration reads;
// block 0 resets the control block.
template <typename Tf, int NX>
__global__ __launch_bounds__(kBlock) void cprep_kernel(KArgs<Tf> a, CArgs<Tf> c, const double *x0, int max_iter,
                                                       double eps, double rho) {
  const int m = blockIdx.x, tid = threadIdx.x, rs = a.rs;
  const int64_t q0 = a.rt_ptr[m];
  const int np = int(a.rt_ptr[m + 1] - q0);
  if (tid < NX) a.x0f[m * NX + tid] = static_cast<Tf>(x0[m * NX + tid]);
  if (tid == 0) {
    double sn = 0.0, sm = 0.0;
    for (int q = 0; q < np; ++q)
#pragma unroll
      for (int e = 0; e < NX; ++e) sn += x0[a.rt_col[q0 + q] * NX + e] * x0[a.rt_col[q0 + q] * NX + e];
#pragma unroll
    for (int e = 0; e < NX; ++e) sm += x0[m * NX + e] * x0[m * NX + e];
    a.nrm[m] = static_cast<Tf>(sn);
    c.xn[m] = static_cast<Tf>(sm);
  }
  const int l0 = c.glob ? NX * a.T : 0;
  for (int l = l0 + tid; l < rs; l += kBlock) {
    double b = 0.0;
    for (int q = 0; q < np; ++q) {
      const int j = a.rt_col[q0 + q];
      const int64_t t0 = a.tile_off[j];
      const int ld = (int(a.tile_off[j + 1] - t0) * rs + 3) & ~3;
      const Tf *o = a.off + a.off_ptr[j] + (a.rt_tile[q0 + q] - t0) * rs + l;
#pragma unroll
      for (int e = 0; e < NX; ++e) b += x0[j * NX + e] * double(o[int64_t(e) * ld]);
    }
    c.bv[c.glob ? int64_t(l - l0) * a.N + m : int64_t(m) * rs + l] = static_cast<Tf>(b);
  }
  if (m == 0 && tid == 0) {
    Ctl *k = a.ctl;
    k->iters = 0;
    k->stop = 0;
    k->converged = 0;
    k->numeric = 0;
    k->max_iter = max_iter;
    k->eps = eps;
    k->rho = rho;
    k->last_rp = INFINITY;
    k->last_rd = INFINITY;
    k->inner_iters = 0;
    k->objective = 0.0;
    k->bar_fail = 0u;
    k->c_phi = 0;
    k->c_psi = 0;
    k->c_halt = 0;
  }
}

// Explicit row solution from the row value av (Phi-comp): the new multiplier; sv the row value.
template <typename Tf>
__device__ __forceinline__ Tf crow_solve(Tf av, Tf n, Tf rho, Tf w, Tf lo, Tf hi, Tf *sv) {
  if (!(n > Tf(0))) {
    *sv = av;
    return Tf(0);
  }
  *sv = clip(rho * av / (rho + Tf(2) * w * n), lo, hi);
  return (*sv - av) / n;
}

// Rows of sum_j ||x0_j||^2 N_j (tau_j + eta_j) of one row subsystem: the sum of its rows of the
// units' shares, in a fixed order. Whole bases: the row update follows, and the block after the
// last decides the previous iteration; input rows: us is written.
// Bound by its chain of loads (list, shares): the shares are 1 / kP1Cols of the bases' bytes.
template <typename Tf, int NX>
__global__ __launch_bounds__(kCRowThreads) void crow_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  if (a.ctl->c_halt) return;
  if (blockIdx.x == unsigned(a.N)) {
    cdecide<Tf, NX>(a, c, true);
    return;
  }
  __shared__ Tf s_acc[kCRowThreads];
  __shared__ double s_d[kCRowThreads / 64];
  const int m = blockIdx.x, tid = threadIdx.x, rows = c.rows;
  const int q0 = c.sptr[m], q1 = c.sptr[m + 1];
  const int it = a.ctl->c_psi + 1;  // whole bases: the iteration whose rows this is
  const int G = max(1, kCRowThreads / rows);
  double dacc = 0.0;
  for (int l0 = 0; l0 < rows; l0 += kCRowThreads) {
    const int rl = min(rows - l0, kCRowThreads), g = tid / rl, l = tid - g * rl;
    const bool row = !c.glob && tid < rl;
    const int64_t R = int64_t(a.N) * a.rs, o = int64_t(m) * a.rs + l0 + tid;
    const Tf n = row ? a.nrm[m] : Tf(0), w = row ? a.w[o] : Tf(0), lo = row ? a.lb[o] : Tf(0);
    const Tf hi = row ? a.ub[o] : Tf(0), b = row ? c.bv[o] : Tf(0);
    const Tf ap = row && it > 1 ? c.al[((it - 1) % 3) * R + o] : Tf(0);
    Tf acc = Tf(0);
    if (g < G && it >= 3)  // tau = eta = 0 before iteration 3
      for (int q = q0 + g; q < q1; q += 8 * G) {  // eight loads in flight, the last ones masked
        uint32_t f[8];
        Tf x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = c.soff[min(q + e * G, q1 - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = c.share[int64_t(f[e]) + l0 + l];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += q + e * G < q1 ? x[e] : Tf(0);
      }
    if (l0 > 0) __syncthreads();  // s_acc is read by the previous rows
    s_acc[tid] = acc;
    __syncthreads();
    if (tid < rl) {
      Tf sum = Tf(0);
      for (int q = 0; q < G; ++q) sum += s_acc[q * rl + tid];
      if (c.glob) {
        c.us[int64_t(l0 + tid) * a.N + m] = sum;
      } else {
        const Tf rho = static_cast<Tf>(a.ctl->rho), coef = it == 1 ? Tf(0) : it == 2 ? Tf(2) : Tf(1);
        Tf sv;
        const Tf al = crow_solve((coef * b + sum) - n * ap, n, rho, w, lo, hi, &sv);
        c.al[(it % 3) * R + o] = al;
        c.s[(it & 1) * R + o] = sv;
        dacc += double(al - ap) * double(al - ap);
      }
    }
  }
  if (!c.glob) {
    dacc = wave_sum(dacc);
    if ((tid & 63) == 0) s_d[tid >> 6] = dacc;
    __syncthreads();
    if (tid == 0) {
      double d = 0.0;
      for (int q = 0; q < kCRowThreads / 64; ++q) d += s_d[q];
      c.dlq[m] = d;
    }
  }
}

// Workgroup barrier that orders LDS accesses only (global loads and stores stay in flight).
__device__ __forceinline__ void lds_barrier1() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Eight sums over the wave at once: lane l ends with the total of index 4 b5 + 2 b4 + b3 of its bits.
template <typename Tf>
__device__ __forceinline__ Tf wave_sum8(const Tf *x, int lane) {
  Tf y[4], z[2];
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
#pragma unroll
  for (int u = 0; u < 4; ++u) y[u] = (b5 ? x[u + 4] : x[u]) + __shfl_xor(b5 ? x[u] : x[u + 4], 32, 64);
#pragma unroll
  for (int u = 0; u < 2; ++u) z[u] = (b4 ? y[u + 2] : y[u]) + __shfl_xor(b4 ? y[u] : y[u + 2], 16, 64);
  Tf r = (b3 ? z[1] : z[0]) + __shfl_xor(b3 ? z[0] : z[1], 8, 64);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
  return r;
}

// eta = N_j' alpha (whole bases) or N_u,j' g (input rows) for kP1Cols basis vectors of one unit, tau,
// tau + eta, the unit's share ||x0_j||^2 N_j (tau + eta) of the row products, and its sums of eta^2
// and (eta - eta_prev)^2; the first unit of j adds up the rows' (alpha - alpha_prev)^2 over the
// patch and, in iteration 2, the offset terms. A wave holds the first kCStepRegs vectors of rows
// per lane of its kUC basis vectors in registers, so an iteration reads the bases once for both
// products (the rows past them twice, the second time from the L2).
// Bound by the bytes of the bases on large networks, by latency on small ones. Input rows of the
// 1024-node mesh (d = 3, T = 15; 41 M entries): 36 us FP32, 81 us FP64 (4.8 and 4.2 TB/s); with all rows in
// registers (four vectors, half the waves) 57 and 79 us; as two kernels that each read the bases
// 56 + 41 and 94 + 66 us.
template <typename Tf, int NX>
__global__ __launch_bounds__(kBlock) void cstep_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  if (a.ctl->stop) {
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->c_halt = 1;  // read by no block of this launch
    return;
  }
  using V = typename VecT<Tf>::type;
  constexpr int VN = VecT<Tf>::N;
  constexpr int kUC = 8, Q = kCStepRegs;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ V s_sh[kWaves][Q * 64];
  __shared__ double red[kWaves][2 + NX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int u = blockIdx.x;
  const CUnit cu = c.unit[u];
  const int j = cu.j, ibase = cu.i0, it = a.ctl->c_phi, rows = c.rows;
  const int64_t tb = cu.tb;
  const int p = cu.p, D = p * rows, ld = (D + 3) & ~3, nvec = ld / VN, k = cu.k;
  if (u == 0 && tid == 0) a.ctl->c_psi = it;  // read by no block of this launch
  Tf *src = reinterpret_cast<Tf *>(smem_raw);  // [ld]
  const int64_t R = int64_t(a.N) * a.rs, K = c.koff[a.N];
  const Tf *vec = c.glob ? c.g : c.al + (it % 3) * R;
  const int i0 = ibase + wave * kUC;
  const Tf *__restrict__ Nj = c.basis + cu.bo + int64_t(i0) * ld;
  V nv[Q][kUC];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int e = 0; e < kUC; ++e)
      nv[q][e] = (i0 + e < k && lane + 64 * q < nvec)
                     ? *reinterpret_cast<const V *>(Nj + int64_t(e) * ld + (lane + 64 * q) * VN)
                     : V(0);
  // basis vector whose sums this lane ends with
  const int i = i0 + ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
  const bool own = i < k;
  const int64_t ki = cu.ko + (own ? i : 0);
  const Tf eo = it > 2 ? c.eta[ki] : Tf(0), to = it > 2 ? c.tau[ki] : Tf(0), xn = c.xn[j];
  const float inv = 1.f / float(rows);
  for (int r = tid; r < ld; r += kBlock) {
    const int ti = int((float(r) + 0.5f) * inv), l = r - ti * rows;
    Tf x = Tf(0);
    if (r < D) {
      const int m = c.rsub[tb + ti];
      x = vec[c.glob ? int64_t(l) * a.N + m : int64_t(m) * rows + l];
    }
    src[r] = x;
  }
  double sdl = 0.0, od[NX];
#pragma unroll
  for (int q = 0; q < NX; ++q) od[q] = 0.0;
  if (ibase == 0 && it >= 2)
    for (int t = tid; t < p; t += kBlock) sdl += c.dlq[c.rsub[tb + t]];
  __syncthreads();
  if (it == 1) return;  // alpha^1 = 0: eta = tau = 0, residuals ||o_c||
  if (ibase == 0 && it == 2) {
    const int ldo = (p * a.rs + 3) & ~3, lo = a.rs - rows;  // input rows follow the state rows
    for (int r = tid; r < D; r += kBlock) {
      const int ti = int((float(r) + 0.5f) * inv);
#pragma unroll
      for (int q = 0; q < NX; ++q)
        od[q] += double(src[r]) * double(a.off[a.off_ptr[j] + int64_t(q) * ldo + ti * a.rs + lo + (r - ti * rows)]);
    }
  }
  Tf acc[kUC];
#pragma unroll
  for (int e = 0; e < kUC; ++e) acc[e] = Tf(0);
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (lane + 64 * q < nvec) {
      const V vv = *reinterpret_cast<const V *>(src + (lane + 64 * q) * VN);
#pragma unroll
      for (int e = 0; e < kUC; ++e) acc[e] += hsum(nv[q][e] * vv);
    }
  if (i0 < k)
    for (int q = lane + 64 * Q; q < nvec; q += 64) {
      const V vv = *reinterpret_cast<const V *>(src + q * VN);
#pragma unroll
      for (int e = 0; e < kUC; ++e)
        if (i0 + e < k) acc[e] += hsum(*reinterpret_cast<const V *>(Nj + int64_t(e) * ld + q * VN) * vv);
    }
  const Tf en = wave_sum8(acc, lane);
  const Tf tn = to + en, vn = own ? tn + en : Tf(0);
  double e2 = 0.0, d2 = 0.0;
  if ((lane & 7) == 0 && own) {
    c.eta[ki] = en;
    c.tau[ki] = tn;
    c.v[(it & 1) * K + ki] = vn;
    e2 = double(en) * double(en);
    d2 = double(en - eo) * double(en - eo);
  }
  Tf y[kUC];
#pragma unroll
  for (int e = 0; e < kUC; ++e) y[e] = xn * __shfl(vn, (e & 4) * 8 + (e & 2) * 8 + (e & 1) * 8, 64);
  for (int q0 = 0; q0 < nvec; q0 += Q * 64) {  // the shares of the waves, Q * 64 vectors of rows at a time
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      V x = V(0);
      if (q0 > 0) {
        const int f = q0 + 64 * q + lane;
#pragma unroll
        for (int e = 0; e < kUC; ++e)
          nv[q][e] = (i0 + e < k && f < nvec) ? *reinterpret_cast<const V *>(Nj + int64_t(e) * ld + f * VN) : V(0);
      }
#pragma unroll
      for (int e = 0; e < kUC; ++e) x += nv[q][e] * y[e];
      s_sh[wave][64 * q + lane] = x;
    }
    lds_barrier1();
    for (int f = tid; f < min(nvec - q0, Q * 64); f += kBlock) {
      V x = s_sh[0][f];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) x += s_sh[w][f];
      *reinterpret_cast<V *>(c.share + cu.so + int64_t(q0 + f) * VN) = x;
    }
    if (q0 + Q * 64 < nvec) lds_barrier1();
  }
  e2 = wave_sum(e2);
  d2 = wave_sum(d2);
  if (ibase == 0) {
    sdl = wave_sum(sdl);
#pragma unroll
    for (int q = 0; q < NX; ++q) od[q] = wave_sum(od[q]);
  }
  __shared__ double red_s[kWaves];
  if (lane == 0) {
    red[wave][0] = e2;
    red[wave][1] = d2;
    red_s[wave] = sdl;
#pragma unroll
    for (int q = 0; q < NX; ++q) red[wave][2 + q] = od[q];
  }
  __syncthreads();
  if (tid < 2) {
    double s = 0.0;
    for (int w = 0; w < kWaves; ++w) s += red[w][tid];
    c.part[2 * u + tid] = s;
  }
  if (ibase == 0 && tid == 2) {
    double s = 0.0;
    for (int w = 0; w < kWaves; ++w) s += red_s[w];
    c.sdl[j] = s;
  }
  if (ibase == 0 && it == 2 && tid >= 8 && tid < 8 + NX) {
    const int q = tid - 8;
    double s = c.glob ? double(c.lam0[int64_t(q) * a.N + j]) : 0.0;
    for (int w = 0; w < kWaves; ++w) s += red[w][2 + q];
    c.od[j * NX + q] = s;
  }
}

// ------------------------------------------------------------------ global recursions

template <typename Tf, int RPT>
struct CEll {  // a thread's state rows r = tid + i blockDim of A or A', first entries in registers
  int e0[RPT], n[RPT], nw[RPT];
  uint32_t idx[RPT][kCSimNE / 2];  // byte offsets of the states, two to a word
  Tf val[RPT][kCSimNE];
  __device__ __forceinline__ void load(const int32_t *rp, const int32_t *col, const Tf *v, int NS) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = threadIdx.x + i * blockDim.x;
      e0[i] = r < NS ? rp[r] : 0;
      n[i] = r < NS ? rp[r + 1] - e0[i] : 0;
      int w = min(n[i], kCSimNE);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, 64));
      nw[i] = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
      for (int e = 0; e < kCSimNE; ++e) {
        const uint32_t o = e < n[i] ? uint32_t(col[e0[i] + e]) * uint32_t(sizeof(Tf)) : 0u;
        idx[i][e / 2] = e & 1 ? idx[i][e / 2] | o << 16 : o;
        val[i][e] = e < n[i] ? v[e0[i] + e] : Tf(0);
      }
    }
  }
  __device__ __forceinline__ Tf dot(int i, const Tf *x, const int32_t *col, const Tf *v) const {
    Tf s = Tf(0);
#pragma unroll
    for (int e = 0; e < kCSimNE; ++e) {
      if (e >= nw[i]) break;
      s += val[i][e] * *reinterpret_cast<const Tf *>(reinterpret_cast<const char *>(x) + (e & 1 ? idx[i][e / 2] >> 16 : idx[i][e / 2] & 0xffffu));
    }
    for (int e = kCSimNE; e < n[i]; ++e) s += v[e0[i] + e] * x[col[e0[i] + e]];
    return s;
  }
};

// Forward recursion of coef b + sum_j N_j W_j (states from x(0), input rows coef b_u + us) by every
// block, the row update of the time steps and input rows that are blockIdx.x modulo kCParts by
// each; the last block decides the previous iteration.
// Bound by T dependent steps, each an LDS barrier and a gather of A's entries from LDS (2 us per step
// for 2048 FP64 states, of which the LDS reads and FP64 products are about half); 16 blocks repeat the
// recursion so that the row update's loads and stores (three row vectors read, two written) are
// off that chain. 1024 threads: 512 with twice the registers and no spills took 47 against 29 us.
template <typename Tf, int NX, int RPT, int KU, int BD>
__global__ __launch_bounds__(BD) void csim_fwd_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  if (a.ctl->c_halt) return;
  if (int(blockIdx.x) == kCParts) {
    cdecide<Tf, NX>(a, c, true);
    return;
  }
  __shared__ Tf xa[BD * RPT], xb[BD * RPT];
  __shared__ double dld[BD * RPT];
  constexpr int np = kCParts;
  const int part = blockIdx.x, tid = threadIdx.x, bd = blockDim.x;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu, nuT = nu * (T - 1);
  const int64_t R = int64_t(N) * a.rs;
  const int it = a.ctl->c_psi + 1;
  const Tf coef = it == 1 ? Tf(0) : it == 2 ? Tf(2) : Tf(1), rho = static_cast<Tf>(a.ctl->rho);
  const bool prod = it >= 3;
  const Tf *ap0 = c.al + ((it - 1) % 3) * R;
  Tf *al0 = c.al + (it % 3) * R, *s0 = c.s + (it & 1) * R;
  CEll<Tf, RPT> ell;
  ell.load(c.prp, c.pcol, c.pval, NS);
  Tf nr[RPT], bk[RPT][KU];
  int mm[RPT], xi[RPT];
  double dl[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = min(tid + i * bd, NS - 1), q = r / N;
    mm[i] = r - q * N;
    nr[i] = a.nrm[mm[i]];
    xi[i] = mm[i] * NX + q;
    dl[i] = 0.0;
#pragma unroll
    for (int k = 0; k < KU; ++k) bk[i][k] = c.bblk[int64_t(xi[i]) * nu + k];
  }
  auto uval = [&](int i, int m) {  // input row i of coef b + sum_j N_j W_j
    const Tf x = prod ? c.us[int64_t(i) * N + m] : Tf(0);
    return coef != Tf(0) ? x + coef * c.bv[int64_t(i) * N + m] : x;
  };
  constexpr int kAhead = sizeof(Tf) == 8 ? 2 : 4;  // steps loaded ahead (as many as the registers hold)
  Tf uq[kAhead][RPT][KU];  // inputs of the next steps
  auto fetch = [&](int t, Tf (*f)[KU]) {  // inputs u_{t-1} of step t
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int k = 0; k < KU; ++k) f[i][k] = (t >= 1 && t < T) ? uval((t - 1) * nu + k, mm[i]) : Tf(0);
  };
#pragma unroll
  for (int q = 0; q < kAhead; ++q) fetch(q + 1, uq[q]);
  auto step = [&](int t, const Tf *src, Tf *dst, Tf (*f)[KU]) {
    const bool mine = t % np == part;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        Tf y;
        if (t == 0) {
          y = coef != Tf(0) ? coef * a.x0f[xi[i]] : Tf(0);
        } else {
          y = ell.dot(i, src, c.pcol, c.pval);
#pragma unroll
          for (int k = 0; k < KU; ++k) y += bk[i][k] * f[i][k];
          for (int k = KU; k < nu; ++k) y += c.bblk[int64_t(xi[i]) * nu + k] * uval((t - 1) * nu + k, mm[i]);
        }
        dst[r] = y;
        if (mine) {
          const int o = t * NS + r;
          const Tf ap = it == 1 ? Tf(0) : ap0[o];
          Tf sv;
          const Tf al = crow_solve(y - nr[i] * ap, nr[i], rho, c.w[o], c.lb[o], c.ub[o], &sv);
          al0[o] = al;
          s0[o] = sv;
          dl[i] += double(al - ap) * double(al - ap);
        }
      }
    }
    if (t > 0) fetch(t + kAhead, f);
    lds_barrier1();
  };
  step(0, xb, xa, uq[0]);
  for (int t = 1; t < T; t += 4) {
    step(t, xa, xb, uq[0]);
    if (t + 1 < T) step(t + 1, xb, xa, uq[1]);
    if (t + 2 < T) step(t + 2, xa, xb, uq[2 % kAhead]);
    if (t + 3 < T) step(t + 3, xb, xa, uq[3 % kAhead]);
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    if (tid + i * bd < NS) dld[tid + i * bd] = dl[i];
  lds_barrier1();
  for (int m = tid; m < N; m += bd) {
    const Tf n = a.nrm[m];
    double d = 0.0;
    for (int i = part; i < nuT; i += np) {
      const int o = T * NS + i * N + m;
      const Tf ap = it == 1 ? Tf(0) : ap0[o];
      Tf sv;
      const Tf al = crow_solve(uval(i, m) - n * ap, n, rho, c.w[o], c.lb[o], c.ub[o], &sv);
      al0[o] = al;
      s0[o] = sv;
      d += double(al - ap) * double(al - ap);
    }
#pragma unroll
    for (int q = 0; q < NX; ++q) d += dld[q * N + m];
    c.dlq[int64_t(1 + part) * N + m] = d;
  }
}

// Adjoint recursion of the new alpha into g, one block; the parts' (alpha - alpha_prev)^2 summed.
// Bound like csim_fwd_kernel. State offsets are packed two to a register and the input rows' registers
// cover a thread's subsystems only: FP64 at 2048 states 43 -> 28 us, most of it spills.
template <typename Tf, int NX, int RPT, int KU, int BD>
__global__ __launch_bounds__(BD) void csim_adj_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  if (a.ctl->stop) return;
  __shared__ Tf xa[BD * RPT], xb[BD * RPT];
  const int tid = threadIdx.x, bd = blockDim.x;
  const int N = a.N, NS = N * NX, T = a.T, nu = a.nu;
  const int64_t R = int64_t(N) * a.rs;
  const int it = a.ctl->c_phi;
  if (it == 1) return;  // alpha^1 = 0
  const Tf *src = c.al + (it % 3) * R;
  constexpr int kAhead = sizeof(Tf) == 8 ? 2 : 4;  // steps loaded ahead (as many as the registers hold)
  constexpr int MPT = (RPT + NX - 1) / NX;  // subsystems of a thread
  Tf v[kAhead][RPT], uq[kAhead][MPT][KU], bc[MPT][NX][KU];
  CEll<Tf, RPT> ell;
  ell.load(c.trp, c.tcol, c.tval, NS);
  int rr[RPT], mr[MPT];  // this thread's state rows and subsystems (clamped)
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    rr[i] = min(tid + i * bd, NS - 1);
    if (i < MPT) mr[i] = min(tid + i * bd, N - 1);
  }
  auto fetch = [&](int t, Tf *f, Tf (*u)[KU]) {  // rows of step t and the input rows of g_{t-1}
    const Tf *st = src + t * NS, *ut = src + T * NS + (t - 1) * nu * N;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      f[i] = t >= 0 ? st[rr[i]] : Tf(0);
      if (i < MPT)
#pragma unroll
        for (int k = 0; k < KU; ++k) u[i][k] = t >= 1 ? ut[k * N + mr[i]] : Tf(0);
    }
  };
#pragma unroll
  for (int q = 0; q < kAhead; ++q) fetch(T - 1 - q, v[q], uq[q]);
#pragma unroll
  for (int i = 0; i < MPT; ++i)
#pragma unroll
    for (int q = 0; q < NX; ++q)
#pragma unroll
      for (int k = 0; k < KU; ++k)
        bc[i][q][k] = tid + i * bd < N ? c.bblk[(int64_t(tid + i * bd) * NX + q) * nu + k] : Tf(0);
  const int tl = it == 2 ? 0 : 1;  // lam_0: offset terms of the second iteration
  auto step = [&](int t, const Tf *prev, Tf *dst, Tf *f, Tf (*u)[KU]) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = tid + i * bd;
      if (r < NS) {
        const Tf l = t + 1 < T ? f[i] + ell.dot(i, prev, c.tcol, c.tval) : f[i];
        dst[r] = l;
        if (t == 0) c.lam0[r] = l;
      }
    }
    lds_barrier1();
    if (t > 0) {
#pragma unroll
      for (int i = 0; i < MPT; ++i) {
        const int m = tid + i * bd;
        if (m < N) {
          Tf l[NX];
#pragma unroll
          for (int q = 0; q < NX; ++q) l[q] = dst[q * N + m];
          Tf *g = c.g + int64_t((t - 1) * nu) * N + m;
#pragma unroll
          for (int k = 0; k < KU; ++k) {
            Tf gk = u[i][k];
#pragma unroll
            for (int q = 0; q < NX; ++q) gk += bc[i][q][k] * l[q];
            g[int64_t(k) * N] = gk;
          }
          for (int k = KU; k < nu; ++k) {
            Tf gk = src[int64_t(T) * NS + ((t - 1) * nu + k) * N + m];
#pragma unroll
            for (int q = 0; q < NX; ++q) gk += c.bblk[(int64_t(m) * NX + q) * nu + k] * l[q];
            g[int64_t(k) * N] = gk;
          }
        }
      }
    }
    fetch(t - kAhead, f, u);
  };
  for (int t = T - 1; t >= tl; t -= 4) {
    step(t, xb, xa, v[0], uq[0]);
    if (t - 1 >= tl) step(t - 1, xa, xb, v[1], uq[1]);
    if (t - 2 >= tl) step(t - 2, xb, xa, v[2 % kAhead], uq[2 % kAhead]);
    if (t - 3 >= tl) step(t - 3, xa, xb, v[3 % kAhead], uq[3 % kAhead]);
  }
  for (int m = tid; m < N; m += bd) {
    double x[kCParts], d = 0.0;  // all parts in flight
#pragma unroll
    for (int q = 0; q < kCParts; ++q) x[q] = c.dlq[int64_t(1 + q) * N + m];
#pragma unroll
    for (int q = 0; q < kCParts; ++q) d += x[q];
    c.dlq[m] = d;
  }
}

// ------------------------------------------------------------------ one workgroup

// A whole solve in one workgroup: bases, multipliers, k-space vectors and index lists in LDS, three LDS
// barriers per iteration. kCS1 lanes share a row of the first product (its terms, one per basis
// vector of the row's tiles, as (address, vector) pairs), kCS2 a basis vector of the second (its terms
// are the support rows) and a column subsystem's residuals; every thread takes the stop decision
// from the waves' maxima. For networks whose bases fit on chip; bound by the LDS latency of two
// short sums of products, their shuffles and the barriers.
constexpr int kCS1 = 4, kCS2 = 8;
constexpr int kCSolveThreads = 1024;

struct CSolveLds {  // byte offsets into the dynamic LDS
  uint32_t basis, al, ap, s, bv, w, lb, ub, d, tau, eta, v, cw, e2, d2, rt, tm, sp, sr, vj, cj, nr, total;
};

template <typename Tf, int NX>
__global__ __launch_bounds__(kCSolveThreads) void csolve_kernel(KArgs<Tf> a, CArgs<Tf> c, CSolveLds o) {
  extern __shared__ __align__(16) unsigned char sm[];
  __shared__ double rp_s[16], rd_s[16];
  Tf *Bs = reinterpret_cast<Tf *>(sm + o.basis), *al = reinterpret_cast<Tf *>(sm + o.al);
  Tf *ap = reinterpret_cast<Tf *>(sm + o.ap), *s = reinterpret_cast<Tf *>(sm + o.s);
  Tf *bv = reinterpret_cast<Tf *>(sm + o.bv), *w = reinterpret_cast<Tf *>(sm + o.w);
  Tf *lb = reinterpret_cast<Tf *>(sm + o.lb), *ub = reinterpret_cast<Tf *>(sm + o.ub);
  Tf *tau = reinterpret_cast<Tf *>(sm + o.tau), *eta = reinterpret_cast<Tf *>(sm + o.eta);
  Tf *v = reinterpret_cast<Tf *>(sm + o.v), *cw = reinterpret_cast<Tf *>(sm + o.cw);  // [2][K]; ||x0_j||^2 (tau + eta)
  double *d = reinterpret_cast<double *>(sm + o.d), *e2 = reinterpret_cast<double *>(sm + o.e2);
  double *d2 = reinterpret_cast<double *>(sm + o.d2);
  int *rt = reinterpret_cast<int *>(sm + o.rt);    // [N+1] first term of each row subsystem
  int2 *tm = reinterpret_cast<int2 *>(sm + o.tm);  // terms: address of the row subsystem's first row, vector
  int *sp = reinterpret_cast<int *>(sm + o.sp);    // [N+1] first support row of each column subsystem
  int *sr = reinterpret_cast<int *>(sm + o.sr);    // support rows
  int4 *vj = reinterpret_cast<int4 *>(sm + o.vj);  // [K] basis vectors: address, column subsystem, first row, rows
  int2 *cj = reinterpret_cast<int2 *>(sm + o.cj);  // [N] first vector, vectors
  Tf *nr = reinterpret_cast<Tf *>(sm + o.nr);      // [N] ||x_r||^2
  Ctl *k = a.ctl;
  const int tid = threadIdx.x, bd = blockDim.x;
  const int s1 = tid & (kCS1 - 1), g1 = tid / kCS1, n1 = bd / kCS1, s2 = tid & (kCS2 - 1), g2 = tid / kCS2, n2 = bd / kCS2;
  const int N = a.N, rs = a.rs, R = N * rs, K = int(c.koff[N]);
  const int64_t nb = c.boff[N];
  for (int64_t e = tid; e < nb; e += bd) Bs[e] = c.basis[e];
  for (int r = tid; r < R; r += bd) {
    bv[r] = c.bv[r];
    w[r] = a.w[r];
    lb[r] = a.lb[r];
    ub[r] = a.ub[r];
    al[r] = ap[r] = Tf(0);
  }
  for (int i = tid; i < K; i += bd) tau[i] = eta[i] = v[i] = v[K + i] = cw[i] = Tf(0);
  for (int j = tid; j < N; j += bd) {
    const int tb = int(a.tile_off[j]), p = int(a.tile_off[j + 1]) - tb, kj = a.kdim[j], ko = int(c.koff[j]);
    const int ld = (p * rs + 3) & ~3;
    cj[j] = int2{ko, kj};
    nr[j] = a.nrm[j];
    sp[j] = tb * rs;
    for (int t = 0; t < p; ++t)
      for (int l = 0; l < rs; ++l) sr[(tb + t) * rs + l] = c.rsub[tb + t] * rs + l;
    for (int i = 0; i < kj; ++i) vj[ko + i] = int4{int(c.boff[j]) + i * ld, j, tb * rs, p * rs};
    int at = 0;  // terms of the row subsystems before j
    for (int q = 0; q < int(a.rt_ptr[j]); ++q) at += c.ct[q].k;
    rt[j] = at;
    for (int q = int(a.rt_ptr[j]); q < int(a.rt_ptr[j + 1]); ++q) {
      const CTile t = c.ct[q];
      for (int i = 0; i < t.k; ++i) tm[at++] = int2{int(t.o) + i * t.ld, t.ko + i};
    }
    if (j == N - 1) {
      rt[N] = at;
      sp[N] = int(a.tile_off[N]) * rs;
    }
  }
  const Tf rho = static_cast<Tf>(k->rho);
  const double eps = k->eps;
  const int max_iter = k->max_iter, nw = min(bd / 64, (N * kCS2 + 63) / 64);  // waves that hold residuals
  __syncthreads();
  for (int it = 1;; ++it) {
    const Tf coef = it == 1 ? Tf(0) : it == 2 ? Tf(2) : Tf(1);
    for (int r0 = 0; r0 < R; r0 += n1) {
      const int r = r0 + g1;
      const bool ok = r < R;
      const int m = ok ? r / rs : 0, l = r - m * rs;
      Tf acc = Tf(0);
      if (ok && it >= 3) {
        const int q1 = rt[m + 1];
        for (int q = rt[m] + s1; q < q1; q += 8 * kCS1) {  // eight terms in flight
          int2 t[8];
          Tf x[8], y[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) t[e] = tm[min(q + e * kCS1, q1 - 1)];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            x[e] = Bs[t[e].x + l];
            y[e] = cw[t[e].y];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (q + e * kCS1 < q1) acc += x[e] * y[e];
        }
      }
#pragma unroll
      for (int x = kCS1 / 2; x > 0; x >>= 1) acc += __shfl_xor(acc, x, 64);
      if (ok && s1 == 0) {
        const Tf n = nr[m], a0 = al[r];
        Tf sv;
        const Tf a1 = crow_solve((coef * bv[r] + acc) - n * a0, n, rho, w[r], lb[r], ub[r], &sv);
        ap[r] = a0;
        al[r] = a1;
        s[r] = sv;
        d[r] = double(a1 - a0) * double(a1 - a0);
      }
    }
    lds_barrier1();
    if (it >= 2)
      for (int u0 = 0; u0 < K; u0 += n2) {
        const int ki = u0 + g2;
        const bool ok = ki < K;
        Tf acc = Tf(0);
        const int4 t = vj[ok ? ki : 0];
        if (ok)
          for (int r = s2; r < t.w; r += 8 * kCS2) {
            int q[8];
            Tf x[8], y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int rr = min(r + e * kCS2, t.w - 1);
              q[e] = sr[t.z + rr];
              x[e] = Bs[t.x + rr];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = al[q[e]];
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (r + e * kCS2 < t.w) acc += x[e] * y[e];
          }
#pragma unroll
        for (int x = kCS2 / 2; x > 0; x >>= 1) acc += __shfl_xor(acc, x, 64);
        if (ok && s2 == 0) {
          const Tf eo = eta[ki], tn = tau[ki] + acc, vn = tn + acc;
          eta[ki] = acc;
          tau[ki] = tn;
          v[(it & 1) * K + ki] = vn;
          cw[ki] = c.xn[t.y] * vn;
          e2[ki] = double(acc) * double(acc);
          d2[ki] = double(acc - eo) * double(acc - eo);
        }
      }
    lds_barrier1();
    double mp = 0.0, md = 0.0;  // squares of the column norms
    for (int j0 = 0; j0 < N; j0 += n2) {
      const int j = j0 + g2;
      double se = 0.0, sd = 0.0, sl = 0.0, od[NX];
#pragma unroll
      for (int q = 0; q < NX; ++q) od[q] = 0.0;
      if (j < N && it >= 2) {
        const int2 t = cj[j];
        for (int i = s2; i < t.y; i += kCS2) {
          se += e2[t.x + i];
          sd += d2[t.x + i];
        }
        const int r0 = sp[j], r1 = sp[j + 1];
        for (int r = r0 + s2; r < r1; r += 8 * kCS2) {
          int q[8];
          double y[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) q[e] = sr[min(r + e * kCS2, r1 - 1)];
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = d[q[e]];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (r + e * kCS2 < r1) sl += y[e];
        }
        if (it == 2) {
          const int ld = (r1 - r0 + 3) & ~3;
          for (int r = s2; r < r1 - r0; r += kCS2)
#pragma unroll
            for (int q = 0; q < NX; ++q)
              od[q] += double(al[sr[r0 + r]]) * double(a.off[a.off_ptr[j] + int64_t(q) * ld + r]);
        }
      }
#pragma unroll
      for (int x = kCS2 / 2; x > 0; x >>= 1) {
        se += __shfl_xor(se, x, 64);
        sd += __shfl_xor(sd, x, 64);
        sl += __shfl_xor(sl, x, 64);
        if (it == 2)
#pragma unroll
          for (int q = 0; q < NX; ++q) od[q] += __shfl_xor(od[q], x, 64);
      }
      if (j < N)
#pragma unroll
        for (int q = 0; q < NX; ++q) {
          const double xc = double(a.x0f[j * NX + q]), x2 = xc * xc, on = c.on2[j * NX + q];
          const double rd = it == 1 ? on : x2 * se;
          const double rp = it == 1 ? on : it == 2 ? on + 2.0 * xc * od[q] + x2 * (sl - se) : x2 * (sl - sd);
          mp = (rp > mp || rp != rp) ? rp : mp;
          md = (rd > md || rd != rd) ? rd : md;
        }
    }
#pragma unroll
    for (int x = 32; x >= kCS2; x >>= 1) {
      const double op = __shfl_xor(mp, x, 64), oq = __shfl_xor(md, x, 64);
      mp = (op > mp || op != op) ? op : mp;
      md = (oq > md || oq != oq) ? oq : md;
    }
    if ((tid & 63) == 0) {
      rp_s[tid >> 6] = mp;
      rd_s[tid >> 6] = md;
    }
    lds_barrier1();
    mp = rp_s[0];
    md = rd_s[0];
    for (int x = 1; x < nw; ++x) {
      mp = (rp_s[x] > mp || rp_s[x] != rp_s[x]) ? rp_s[x] : mp;
      md = (rd_s[x] > md || rd_s[x] != rd_s[x]) ? rd_s[x] : md;
    }
    mp = sqrt(mp);
    md = sqrt(md);
    const bool bad = !(mp == mp) || !(md == md) || isinf(mp) || isinf(md);
    if (bad || (mp <= eps && md <= eps) || it >= max_iter) {  // the same on every thread
      if (tid == 0) {
        decide(k, it, mp, md);
        k->c_psi = it;
      }
      // the state where cexpand_kernel and the output read it
      for (int r = tid; r < R; r += bd) {
        c.al[(it % 3) * int64_t(R) + r] = al[r];
        c.al[((it + 2) % 3) * int64_t(R) + r] = ap[r];
        c.s[(it & 1) * int64_t(R) + r] = s[r];
      }
      for (int i = tid; i < K; i += bd) {
        c.tau[i] = tau[i];
        c.eta[i] = eta[i];
        c.v[i] = v[i];
        c.v[K + i] = v[K + i];
      }
      return;
    }
  }
}

// ------------------------------------------------------------------ after the stop

// Phi, Psi and Lambda of the stopping iterate K on the tiles of column subsystem j, and (rows of
// subsystem j) y = Phi x0 in library order: with z = N_j (tau + eta)^{K-1} (K >= 3),
//   Phi = c o + x0_c (z - alpha^{K-1} + alpha^K) (c = 0, 2, 1 for K = 1, 2, >= 3),
//   Psi = o + x0_c N_j tau, Lambda = x0_c (alpha - N_j eta) (K = 1: -o).
// Rows of j over the threads, the basis vectors streamed once for the three products.
template <typename Tf, int NX>
__global__ __launch_bounds__(kBlock) void cexpand_kernel(KArgs<Tf> a, CArgs<Tf> c) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int j = a.psi_order[blockIdx.x], tid = threadIdx.x, rs = a.rs;
  const int it = a.ctl->iters, k = a.kdim[j];
  const int64_t tb = a.tile_off[j], R = int64_t(a.N) * rs, K = c.koff[a.N];
  const int D = int(a.tile_off[j + 1] - tb) * rs, ld = (D + 3) & ~3;
  Tf *z = reinterpret_cast<Tf *>(smem_raw), *tt = z + k, *ee = tt + k;
  for (int i = tid; i < k; i += kBlock) {
    z[i] = it >= 3 ? c.v[((it - 1) & 1) * K + c.koff[j] + i] : Tf(0);
    tt[i] = it >= 2 ? c.tau[c.koff[j] + i] : Tf(0);
    ee[i] = it >= 2 ? c.eta[c.koff[j] + i] : Tf(0);
  }
  __syncthreads();
  const Tf *__restrict__ Nj = a.nb + a.nb_off[j];
  const Tf coef = it == 1 ? Tf(0) : it == 2 ? Tf(2) : Tf(1);
  for (int r = tid + kBlock * blockIdx.y; r < D; r += kBlock * gridDim.y) {
    Tf s0 = Tf(0), s1 = Tf(0), s2 = Tf(0);
    int i = 0;
    for (; i + 8 <= k; i += 8) {
      Tf x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = Nj[int64_t(i + e) * ld + r];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        s0 += x[e] * z[i + e];
        s1 += x[e] * tt[i + e];
        s2 += x[e] * ee[i + e];
      }
    }
    for (; i < k; ++i) {
      const Tf x = Nj[int64_t(i) * ld + r];
      s0 += x * z[i];
      s1 += x * tt[i];
      s2 += x * ee[i];
    }
    const int ti = r / rs, l = r - ti * rs, m = c.rsub[tb + ti];
    const int64_t ro = crow(a, c, m, l);
    const Tf an = it >= 2 ? c.al[(it % 3) * R + ro] : Tf(0), ao = it >= 3 ? c.al[((it - 1) % 3) * R + ro] : Tf(0);
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const Tf o = a.off[a.off_ptr[j] + int64_t(q) * ld + r], x = a.x0f[j * NX + q];
      const int64_t e = (tb * rs + r) * NX + q;
      a.phi[e] = coef * o + x * (s0 - ao + an);
      a.psi[e] = o + x * s1;
      a.lam[e] = it == 1 ? -o : x * (an - s2);
    }
    if (m == j) a.y[int64_t(j) * rs + l] = c.s[(it & 1) * R + ro];
  }
}
