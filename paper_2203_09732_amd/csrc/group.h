// MINRES of one realization on a group of workgroups of one XCD, every
// recurrence vector on chip: the form for sectors that are too large for one
// compute unit and small enough for the 32 of an XCD (L = 14, 16, 18).
//
// Why one XCD: its compute units share an L2, so what one workgroup stores the
// others can load from there, with no write-back or invalidation. Across XCDs
// the same hand-over needs device-scope fences (measured with two fenced grid
// barriers per iteration: 12.6 us at L = 14, 17.2 at L = 16, 35 at L = 18).
// Workgroups are dispatched round-robin over the XCDs, so a group takes the
// blocks of one residue of blockIdx mod 8; the workgroups compare their XCC
// ids before they start, and use device-scope fences if they differ.
//
// What bounds it is the trip through the L2 (a store in one workgroup is seen
// by a load past the L1 in another after about 600 cycles; measured, a round
// trip is 1229 cycles, and 2358 if the store is also written through to
// device scope). As Alg. 2 is written an iteration makes two of them: the sums
// alpha_k (with beta_k's, formed an iteration earlier, in the same message),
// then the new q. With one or two rows per thread it makes one: M^{-1} p goes
// out beside the sums, and each workgroup forms the new q of its neighbours'
// rows too (L = 14: 1.92 -> 1.77 us per iteration on one machine; over machines
// 1.77 to 1.86). Neither waits for a drain or a separate flag:
// - an element of q is its own arrival flag: one not yet written holds a NaN
//   pattern that no arithmetic makes; three buffers rotate, and a workgroup
//   puts the pattern back into its rows one iteration before their next use;
// - a sum is one 16-byte slot per (receiver, sender), each half of the double
//   beside the iteration's tag.
// One wave keeps the sums and the scalars, the others own rows. Every wait is
// bounded (about one second), so the launch always ends. A workgroup may be done
// when another one's wait runs out, so a solve that counts as failed may have
// written its solution: never into what a second attempt starts from.
#pragma once

#include "resident.h"

namespace mbl {

constexpr int kGroupXcds = 8;

// What a group leaves: set by a wait that ran out of time, and the solve's
// iterations, phi and non-finite flag.
struct GroupOut {
  unsigned long long failed;
  int64_t k;
  double phi;
  int64_t bad;
};

// R realizations, each on one group of W workgroups (R = 1: the single form); a
// group takes the next one when its own is done. n-vectors of realization r
// have element i at i * R + r.
struct GroupArgs {
  const double* src;        // right-hand sides
  const double* ax0;        // (H - sigma) x0, or null for x0 = 0 (R = 1 only)
  double* x;                // out: the solution (less x0)
  const double* scale;      // R factors of src (0: not solved, x = 0), or null: scale1
  double scale1;
  const double* h;          // R x L fields, or null: the fields argument
  const double* c0;         // R: L / 4 + sum h / 2 - sigma, or null
  double* q[3];             // R x n doubles each: realization r at r * n
  GroupOut* out;            // R, zeroed before the launch
  unsigned long long* slots; // R x group_slots(W) words, zeroed before the launch
  const double* v;          // rank-one term theta v v^T (R = 1 only)
  double theta;
  double tol;
  int64_t kmax;
  int kind, R;
  int fenced;               // use device scope whatever the workgroups' XCDs
};

// Slot words of a group: three exchanges of W receivers x 2 values x W senders
// x 2 words. The sums of iteration k use exchange k mod 2:
// a workgroup may send those of k + 1 before a slow one has read those of k
// (it waits only for the q of its own neighbours), but those of k + 2 only
// after the slow one has sent its own of k + 1.
__host__ __device__ constexpr int group_xwords(int W) { return W * 2 * W * 2; }
__host__ __device__ constexpr int group_slots(int W) {
  return 3 * group_xwords(W);
}

constexpr uint64_t kNotYet = 0xfff4c0dec0de5eedull;   // a q element not yet written

__host__ __device__ constexpr uint32_t cbinom(int n, int k) {
  uint64_t v = 1;
  if (k < 0 || k > n) return 0;
  for (int t = 1; t <= k; ++t) v = v * (uint64_t)(n - k + t) / (uint64_t)t;
  return (uint32_t)v;
}

// A swap on bond b moves a row's rank by at most C(b, b / 2), so the
// neighbours on bonds 0 .. L - NG - 1 lie in a window of the own rows widened
// by that much on both sides; those on the last NG bonds (the periodic one
// among them) are "far". NG = 0: the window is the whole vector.
template <int L, int NG, int W>
struct GroupShape {
  static constexpr uint32_t n = cbinom(L, L / 2);
  static constexpr uint32_t kOwn = (n + W - 1) / W;   // rows of a workgroup
  static constexpr uint32_t kHalo = NG ? cbinom(L - NG - 1, (L - NG - 1) / 2) : 0;
  static constexpr uint32_t kWindow = NG && kOwn + 2 * kHalo < n ? kOwn + 2 * kHalo : n;
};

constexpr uint64_t kGroupTimeoutTicks = 100000000ull;   // ~1 s of the 100 MHz clock

// Bounded spinning of a wave: late() once about a second has passed or another
// wait has failed (then the flag is set for all).
struct GroupWait {
  unsigned long long* fail;
  uint64_t t0;
  uint32_t spin = 0;
  __device__ __forceinline__ explicit GroupWait(unsigned long long* f) : fail(f), t0(wall_clock64()) {}
  __device__ __forceinline__ bool late() {
    if ((++spin & 127u) != 0) return false;
    const bool over = wall_clock64() - t0 > kGroupTimeoutTicks;
    if (over) __hip_atomic_store(fail, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return over || __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  }
};

// Cache policies: a load past the L1; a store to the XCD's L2, or through it.
constexpr int kAuxDevice = 16;

__device__ __forceinline__ uint64_t peek64(__amdgpu_buffer_rsrc_t b, uint32_t off,
                                           uint32_t soff = 0) {
  const auto u = __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, (int)soff, kAuxDevice);
  uint64_t v;
  __builtin_memcpy(&v, &u, 8);
  return v;
}
__device__ __forceinline__ void poke64(__amdgpu_buffer_rsrc_t b, uint32_t off, uint64_t v,
                                       bool one_xcd, uint32_t soff = 0) {
  using U = decltype(__builtin_amdgcn_raw_buffer_load_b64(b, 0, 0, 0));
  U u;
  __builtin_memcpy(&u, &v, 8);
  if (one_xcd)
    __builtin_amdgcn_raw_buffer_store_b64(u, b, (int)off, (int)soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b64(u, b, (int)off, (int)soff, kAuxDevice);
}

// One wave: send values (lanes 0..31 value 0 in v, lanes 32..63 value 1) under
// `tag` to every workgroup's slots. xoff: byte offset of the exchange.
template <int W>
__device__ __forceinline__ void group_publish(__amdgpu_buffer_rsrc_t b, uint32_t xoff, int member,
                                              uint32_t tag, double v, int nval, bool one_xcd) {
  const int lane = threadIdx.x & 63, to = lane & 31, val = lane >> 5;
  if (to < W && val < nval) {
    using U = decltype(__builtin_amdgcn_raw_buffer_load_b128(b, 0, 0, 0));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t words[4] = {(uint32_t)u, tag, (uint32_t)(u >> 32), tag};
    U x;
    __builtin_memcpy(&x, words, 16);
    const int off = (int)(xoff + ((to * 2 + val) * W + member) * 16);
    if (one_xcd)
      __builtin_amdgcn_raw_buffer_store_b128(x, b, off, 0, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b128(x, b, off, 0, kAuxDevice);
  }
}
// One wave: wait for every workgroup's values; lane v * 32 + m returns value v
// of workgroup m (0 where there is none).
template <int W>
__device__ __forceinline__ bool group_poll(__amdgpu_buffer_rsrc_t b, uint32_t xoff,
                                           unsigned long long* fail, int member, uint32_t tag,
                                           int nval, double& out) {
  const int lane = threadIdx.x & 63, m = lane & 31, val = lane >> 5;
  const bool mine = m < W && val < nval;
  const int off = (int)(xoff + ((member * 2 + val) * W + m) * 16);
  uint32_t words[4] = {0, 0, 0, 0};
  GroupWait wait(fail);
  for (;;) {
    bool ok = true;
    if (mine) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, kAuxDevice);
      __builtin_memcpy(words, &x, 16);
      ok = words[1] == tag && words[3] == tag;
    }
    asm volatile("" ::: "memory");   // load again
    if (__all(ok)) break;
    if (wait.late()) return false;
  }
  out = mine ? __builtin_bit_cast(double, ((uint64_t)words[2] << 32) | words[0]) : 0.0;
  return true;
}

// sums over the two 32-lane halves (lanes without a value hold 0), fixed order
__device__ __forceinline__ void half_sums(double v, double& s0, double& s1) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  s0 = read_lane(v, 0) + read_lane(v, 16);
  s1 = read_lane(v, 32) + read_lane(v, 48);
}

// Realization r on the workgroups of a group; false when a wait ran out of time.
template <int L, int NG, int W, int RPT, int NT, bool DEFL>
__device__ __forceinline__ bool group_solve(const GroupArgs& A, const FieldArgs& F, int r,
                                            int member) {
  using Sh = GroupShape<L, NG, W>;
  constexpr uint32_t n = Sh::n;
  constexpr int NR = NT - 64, NWR = NR / 64;   // threads and waves that own rows
  static_assert(RPT * NR >= (int)Sh::kOwn && W <= 32, "rows do not fit the workgroup");
  constexpr int TW = (int)((Sh::kWindow + NR - 1) / NR);   // window elements per thread
  constexpr int NLB = L - NG;                  // bonds read from the LDS window
  constexpr int NPAIR = (NLB + 1) / 2;
  constexpr int NF = NG ? NG : 1;
  static_assert(Sh::kWindow < 65536, "window offsets are 16 bits");
  const int R = A.R;
  constexpr int BW = L / 2 + 2;
  // one trip per iteration where q_k and q_{k-1} of a thread's window and far
  // elements fit the registers beside its own rows (four rows: they do not);
  // v . q would take another trip and barrier (3 % slower than two trips)
  constexpr bool kOne = RPT <= 2 && !DEFL;
  __shared__ double win[Sh::kWindow + 1];      // q_k; the last place stays 0
  __shared__ uint32_t binom[(L + 1) * BW];
  __shared__ double red1[NWR], red2[NWR], red3[NWR];
  __shared__ ResidentCoef co;
  __shared__ double sh_alpha, sh_vq, sh_h[L];
  __shared__ int sh_ok;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)uni(tid >> 6);
  const bool rows = wave < NWR;                // the last wave keeps the scalars
  const uint32_t lo = Sh::kOwn * member < n ? Sh::kOwn * member : n;
  const uint32_t hi = lo + Sh::kOwn < n ? lo + Sh::kOwn : n;
  const uint32_t w0 = Sh::kWindow == n ? 0 : (lo > Sh::kHalo ? lo - Sh::kHalo : 0);
  const uint32_t w1 = Sh::kWindow == n ? n : (hi + Sh::kHalo < n ? hi + Sh::kHalo : n);
  for (int t = tid; t < (L + 1) * BW; t += NT) binom[t] = cbinom(t / BW, t % BW);
  if (tid < L) sh_h[tid] = A.h ? A.h[(size_t)r * L + tid] : F.h[tid];
  unsigned long long* slots = A.slots + (size_t)r * group_slots(W);
  GroupOut* out = A.out + r;
  unsigned long long* fail = &out->failed;
  // exchanges 0 and 1: the sums, by the tag's parity; 2: v . q
  const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
      slots, (short)0, 3 * group_xwords(W) * 8, 0x00020000);
  constexpr uint32_t kX = (uint32_t)group_xwords(W) * 8u;
  __amdgpu_buffer_rsrc_t qb[3];
#pragma unroll
  for (int b = 0; b < 3; ++b)
    qb[b] = __builtin_amdgcn_make_buffer_rsrc(A.q[b] + (size_t)r * n, (short)0, (int)(n * 8u),
                                              0x00020000);

  // ---- own rows of every buffer marked, then the workgroups' XCDs
  if (rows)
    for (uint32_t row = lo + tid; row < hi; row += NR)
      for (int b = 0; b < 3; ++b) poke64(qb[b], row * 8u, kNotYet, false);
  if (tid == 0) {
    sh_ok = 1;
    win[Sh::kWindow] = 0.0;
  }
  __threadfence();
  __syncthreads();
  if (!rows) {
    const uint32_t id = __builtin_amdgcn_s_getreg(20 | (3 << 11));   // XCC_ID
    group_publish<W>(xs, kX, member, 1u, (double)id, 1, false);
    double v = 0.0;
    const bool ok = group_poll<W>(xs, kX, fail, member, 1u, 1, v);
    const bool same = __all(lane >= W || v == (double)id);
    if (lane == 0) sh_ok = ok ? (same ? 1 : 2) : 0;
  }
  __syncthreads();
  const int xcds = sh_ok;
  __syncthreads();
  if (xcds == 0) return false;
  const bool one_xcd = uni((uint32_t)(xcds == 1 && !A.fenced)) != 0;
  __threadfence();
  // the marks of a buffer come before the sums that allow its use: by the
  // drain of the stores inside one XCD, by fences otherwise
  auto fence = [&] {
    if (!one_xcd) __threadfence();
  };

  // ---- own rows: state, neighbours, diagonal, preconditioner, right-hand side
  const double sc = A.scale ? A.scale[r] : A.scale1;
  const double c0 = A.c0 ? A.c0[r] : F.c0;
  constexpr uint32_t zero = Sh::kWindow;
  constexpr uint32_t kNone = 0xffffffffu;
  constexpr uint32_t kFarNone = 0x7ffffff8u;   // beyond the buffer: the load returns 0
  uint32_t nb[RPT][NPAIR], far[RPT][NF];
  double dg[RPT], rs[RPT], u[RPT], up[RPT], uo[RPT], d1[RPT], d0[RPT], x[RPT], v[DEFL ? RPT : 1];
  double m[kOne ? RPT : 1];    // one trip: M, and its inverse in rs
  double a2 = 0.0, av = 0.0;   // partial sums of u . u and v . q
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    __builtin_amdgcn_sched_barrier(0);   // one row at a time: few registers
    const uint32_t row = lo + i * NR + tid;
    dg[i] = rs[i] = u[i] = up[i] = uo[i] = d1[i] = d0[i] = x[i] = 0.0;
    if (DEFL) v[i] = 0.0;
    if (kOne) m[i] = 0.0;
#pragma unroll
    for (int b = 0; b < NPAIR; ++b) nb[i][b] = zero | (zero << 16);
#pragma unroll
    for (int b = 0; b < NF; ++b) far[i][b] = kFarNone;
    if (rows && row < hi) {
      uint32_t a = 0, rem = row;
      int k = L / 2;
      for (int b = L - 1; b >= 0; --b) {
        const uint32_t c = binom[b * BW + k];
        if (rem >= c) {
          a |= 1u << b;
          rem -= c;
          --k;
        }
      }
      const int na = __popc(a ^ (((a << 1) | (a >> (L - 1))) & ((1u << L) - 1u)));
      // nibble by nibble, as every other kernel sums the fields of a state: the
      // same bits, so the same operator
      double f = 0.0;
#pragma unroll
      for (int b = 0; b < L; b += 4) {
        double acc = 0.0;
#pragma unroll
        for (int t = b; t < b + 4 && t < L; ++t)
          acc += ((a >> t) & 1u) ? sh_h[t] : 0.0;
        f += acc;
      }
      dg[i] = c0 - 0.5 * (double)na - f;
      const double pm = precond_value(A.kind, dg[i], na);
      if (kOne) m[i] = pm;
      rs[i] = 1.0 / (kOne ? pm : sqrt(pm));
#pragma unroll
      for (int b = 0; b < L; ++b) {
        const uint32_t mask = b + 1 < L ? 3u << b : (1u | (1u << (L - 1)));
        const uint32_t two = a & mask;
        uint32_t to = kNone;
        if (two != 0 && two != mask) {
          if (b + 1 < L) {
            // the particle on bit b or b + 1 moves: the rank changes by C(b, .)
            const int below = __popc(a & ((2u << b) - 1u));
            to = ((a >> b) & 1u) ? row + binom[b * BW + below - 1] : row - binom[b * BW + below];
          } else {
            to = 0;
            int cnt = 0;
            for (int t = 0; t < L; ++t)
              if (((a ^ mask) >> t) & 1u) to += binom[t * BW + ++cnt];
          }
        }
        if (b < NLB) {
          const uint32_t w = to != kNone ? to - w0 : zero;
          nb[i][b / 2] = (b & 1) ? (nb[i][b / 2] & 0xffffu) | (w << 16)
                                 : (nb[i][b / 2] & 0xffff0000u) | w;
        } else {
          far[i][b - NLB] = to != kNone ? to * 8u : kFarNone;
        }
      }
      const size_t e = (size_t)row * R + r;
      double z = 0.0;
      if (sc != 0.0) z = sc * (A.src[e] - (A.ax0 ? A.ax0[e] : 0.0));
      double q1 = z * rs[i];
      if (!kOne) {
        u[i] = q1;
        a2 += u[i] * u[i];
        q1 = u[i] * rs[i];
      }
      if (DEFL) {
        v[i] = A.v[row];
        av += v[i] * q1;
      }
      poke64(qb[1], row * 8u, __builtin_bit_cast(uint64_t, q1), one_xcd);
    }
  }

  auto put = [&](double s, double* red) {
    s = wave_sum(s);
    if (lane == 0) red[wave] = s;
  };
  // lane w of the lower half: red_a[w]; of the upper half: red_b[w]; summed
  auto totals = [&](const double* ra, const double* rb) {
    const int w = lane & 31;
    double s0, s1;
    half_sums(w < NWR ? (lane < 32 ? ra[w] : rb[w]) : 0.0, s0, s1);
    return lane < 32 ? s0 : s1;
  };
  // the window's elements and the far neighbours of this thread's rows, as they
  // arrive in a buffer
  const uint32_t own = (lo + tid) * 8u, nown = hi - lo;   // row i at own + 8 i NR
  const uint32_t left = w1 - w0;
  auto await = [&](__amdgpu_buffer_rsrc_t q, uint64_t (&ww)[TW], uint64_t (&wf)[RPT][NF]) {
    GroupWait wait(fail);
    const uint32_t off = (w0 + tid) * 8u;
    for (;;) {
      bool ok = true;
#pragma unroll
      for (int t = 0; t < TW; ++t)
        ww[t] = peek64(q, t * NR + tid < left ? off + t * NR * 8u : kFarNone);
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int b = 0; b < NG; ++b) wf[i][b] = peek64(q, far[i][b]);
      asm volatile("" ::: "memory");   // load again
#pragma unroll
      for (int t = 0; t < TW; ++t) ok = ok && ww[t] != kNotYet;
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int b = 0; b < NG; ++b) ok = ok && wf[i][b] != kNotYet;
      if (__all(ok)) break;
      if (wait.late()) {
        if (lane == 0) sh_ok = 0;
        break;
      }
    }
  };
  // q's window goes to LDS and the far neighbours of this thread's rows to fv
  double fv[RPT][NF];
  // one trip: q_k (far: in fv) and q_{k-1} of the window and far elements
  double wq[kOne ? TW : 1], wqm[kOne ? TW : 1], fvm[kOne ? RPT : 1][NF];
  auto await_q = [&](__amdgpu_buffer_rsrc_t q) {
    uint64_t ww[TW], wf[RPT][NF];
    await(q, ww, wf);
#pragma unroll
    for (int t = 0; t < TW; ++t)
      if (t * NR + tid < left) win[t * NR + tid] = __builtin_bit_cast(double, ww[t]);
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int b = 0; b < NG; ++b) fv[i][b] = __builtin_bit_cast(double, wf[i][b]);
    if (kOne) {
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        wq[t] = __builtin_bit_cast(double, ww[t]);
        wqm[t] = 0.0;
      }
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int b = 0; b < NF; ++b) fvm[i][b] = 0.0;
    }
  };
  if (rows) {
    if (!kOne) put(a2, red2);
    if (DEFL) put(av, red3);
    await_q(qb[1]);
  }
  __syncthreads();
  if (!sh_ok) return false;
  ResidentScalars rec;
  int64_t k = 0;
  uint32_t tag = 1;
  __amdgpu_buffer_rsrc_t qn_ = qb[2], qa_ = qb[0], qp_ = qb[1];   // q_{k+1}, q_{k+2}, q_k
  // Iteration k on (u_k, u_{k-1}, d_{k-3}, d_{k-4}): u_{k-1} is overwritten by
  // u_{k+1} and goes to uo, d_{k-4} is overwritten by d_{k-2}. Returns false
  // when the solve had ended after iteration k - 1, or a wait has failed.
  auto iteration = [&](double (&uk)[RPT], double (&um)[RPT], double (&da)[RPT],
                       double (&db)[RPT]) {
    ++k;
    ++tag;
    double p[RPT], qi[RPT];
    if (rows) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        double off = 0.0, off2 = 0.0;
#pragma unroll
        for (int b = 0; b < NPAIR; ++b) {
          uint32_t w = nb[i][b];
          asm volatile("" : "+v"(w));   // keep the pair packed: unpacked in the loop, not before it
          off += win[w & 0xffffu];
          off2 += win[w >> 16];
        }
#pragma unroll
        for (int b = 0; b < NG; ++b) off += fv[i][b];
        qi[i] = uk[i] * rs[i];
        p[i] = dg[i] * qi[i] + 0.5 * (off + off2);
      }
    }
    if (DEFL) {
      if (!rows) {
        double val = totals(red3, red3), s0, s1;
        group_publish<W>(xs, 2 * kX, member, tag, val, 1, one_xcd);
        if (!group_poll<W>(xs, 2 * kX, fail, member, tag, 1, val) && lane == 0) sh_ok = 0;
        half_sums(val, s0, s1);
        if (lane == 0) sh_vq = s0;
      }
      __syncthreads();
      const double tv = A.theta * sh_vq;
#pragma unroll
      for (int i = 0; i < RPT; ++i) p[i] += tv * v[i];
    }
    if (rows) {
      double a1 = 0.0;
#pragma unroll
      for (int i = 0; i < RPT; ++i) a1 += qi[i] * p[i];
      put(a1, red1);
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the marks are in the L2
      fence();
    }
    __syncthreads();
    if (!rows) {
      double val = totals(red1, red2), s1, s2;
      const uint32_t xk = (tag & 1u) * kX;
      group_publish<W>(xs, xk, member, tag, val, 2, one_xcd);
      if (!group_poll<W>(xs, xk, fail, member, tag, 2, val) && lane == 0) sh_ok = 0;
      half_sums(val, s1, s2);
      ResidentCoef c;
      rec.lanczos(k, s2, c);
      const double alpha = s1 * c.ib * c.ib;
      if (lane == 0) {
        co.ib = c.ib;
        co.c3 = c.c3;
        sh_alpha = alpha;
      }
    } else if (k > 1) {
      // meanwhile the d/x update of iteration k - 2
      const double ibp = co.ibp, de = co.de, ep = co.ep, ig = co.ig, tau = co.tau;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const double d = (uo[i] * ibp - de * da[i] - ep * db[i]) * ig;
        db[i] = d;
        x[i] += tau * d;
      }
    }
    __syncthreads();
    fence();
    if (!sh_ok) return false;
    if (rows) {
      const double ib = co.ib, c3 = co.c3, c2 = sh_alpha * ib;
      double s2 = 0.0, s3 = 0.0;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const double un = ib * (p[i] * rs[i]) - c2 * uk[i] - c3 * um[i];
        const double qn = un * rs[i];
        if (i * NR + tid < nown)
          poke64(qn_, own, __builtin_bit_cast(uint64_t, qn), one_xcd, i * NR * 8u);
        s2 += un * un;
        if (DEFL) s3 += v[i] * qn;
        uo[i] = um[i];
        um[i] = un;
      }
      put(s2, red2);
      if (DEFL) put(s3, red3);
      await_q(qn_);
#pragma unroll
      for (int i = 0; i < RPT; ++i)
        if (i * NR + tid < nown) poke64(qa_, own, kNotYet, one_xcd, i * NR * 8u);
    } else {
      // the Givens step of iteration k - 1
      ResidentCoef c;
      rec.givens(k, A.tol, A.kmax, c);
      if (!c.done) rec.rotate(sh_alpha);   // (a done solve's alpha may be 0 / 0)
      if (lane == 0) {
        co.ibp = c.ibp;
        co.de = c.de;
        co.ep = c.ep;
        co.ig = c.ig;
        co.tau = c.tau;
        co.done = c.done;
      }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t t = qp_;
    qp_ = qn_;
    qn_ = qa_;
    qa_ = t;
    return sh_ok != 0 && co.done == 0;
  };
  // The same in one trip: M^{-1} p goes out beside the sums, and every workgroup
  // forms q_{k+1} of its window and far elements itself, with the operations
  // written out so that all of them hold the same bits. up holds q_{k-1} of the
  // own rows. The buffer of k - 1 is marked for k + 2: what it held was read
  // before the sums of k, and the marks are in the L2 before those of k + 1.
  auto one_trip = [&](const double (&da)[RPT], double (&db)[RPT]) {
    ++k;
    ++tag;
    double p[RPT], qi[RPT];
    uint64_t ww[TW], wf[RPT][NF];
    if (rows) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        qi[i] = win[i * NR + tid < nown ? lo - w0 + i * NR + tid : zero];
        double off = 0.0, off2 = 0.0;
#pragma unroll
        for (int b = 0; b < NPAIR; ++b) {
          uint32_t w = nb[i][b];
          asm volatile("" : "+v"(w));
          off += win[w & 0xffffu];
          off2 += win[w >> 16];
        }
#pragma unroll
        for (int b = 0; b < NG; ++b) off += fv[i][b];
        p[i] = dg[i] * qi[i] + 0.5 * (off + off2);
      }
    }
    if (rows) {
      double s1 = 0.0, s2 = 0.0;
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the marks are in the L2
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        if (i * NR + tid < nown)
          poke64(qn_, own, __builtin_bit_cast(uint64_t, p[i] * rs[i]), one_xcd, i * NR * 8u);
        s1 += qi[i] * p[i];
        s2 += qi[i] * (m[i] * qi[i]);
      }
      put(s1, red1);
      put(s2, red2);
      fence();
    }
    __syncthreads();
    if (!rows) {
      double val = totals(red1, red2), s1, s2;
      const uint32_t xk = (tag & 1u) * kX;
      group_publish<W>(xs, xk, member, tag, val, 2, one_xcd);
      if (!group_poll<W>(xs, xk, fail, member, tag, 2, val) && lane == 0) sh_ok = 0;
      half_sums(val, s1, s2);
      ResidentCoef c;
      rec.lanczos(k, s2, c);
      if (lane == 0) {
        co.ib = c.ib;
        co.c3 = c.c3;
        sh_alpha = s1 * c.ib * c.ib;
      }
    } else {
      if (k > 1) {
        const double ibp = co.ibp, de = co.de, ep = co.ep, ig = co.ig, tau = co.tau;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
          const double d = (uo[i] * ibp - de * da[i] - ep * db[i]) * ig;
          db[i] = d;
          x[i] += tau * d;
        }
      }
      await(qn_, ww, wf);
    }
    __syncthreads();
    fence();
    if (!sh_ok) return false;
    if (rows) {
      const double ib = co.ib, c3 = co.c3, c2 = sh_alpha * ib;
      auto next = [&](uint64_t w, double q, double qm) {
        return fma(-c3, qm, fma(-c2, q, ib * __builtin_bit_cast(double, w)));
      };
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        const double q = next(ww[t], wq[t], wqm[t]);
        if (t * NR + tid < left) win[t * NR + tid] = q;
        wqm[t] = wq[t];
        wq[t] = q;
      }
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
#pragma unroll
        for (int b = 0; b < NG; ++b) {
          const double q = next(wf[i][b], fv[i][b], fvm[i][b]);
          fvm[i][b] = fv[i][b];
          fv[i][b] = q;
        }
        uo[i] = up[i];
        up[i] = qi[i];
        if (i * NR + tid < nown) poke64(qp_, own, kNotYet, one_xcd, i * NR * 8u);
      }
    } else {
      ResidentCoef c;
      rec.givens(k, A.tol, A.kmax, c);
      if (!c.done) rec.rotate(sh_alpha);
      if (lane == 0) {
        co.ibp = c.ibp;
        co.de = c.de;
        co.ep = c.ep;
        co.ig = c.ig;
        co.tau = c.tau;
        co.done = c.done;
      }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t t = qp_;
    qp_ = qn_;
    qn_ = qa_;
    qa_ = t;
    return sh_ok != 0 && co.done == 0;
  };
  // the last d/x update, of iteration k - 1 where k is the last one begun
  auto last = [&](double (&da)[RPT], double (&db)[RPT]) {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
      x[i] += co.tau * ((uo[i] * co.ibp - co.de * da[i] - co.ep * db[i]) * co.ig);
  };
  for (;;) {
    if (!(kOne ? one_trip(d1, d0) : iteration(u, up, d1, d0))) {
      last(d0, d1);
      break;
    }
    if (!(kOne ? one_trip(d0, d1) : iteration(up, u, d0, d1))) {
      last(d1, d0);
      break;
    }
  }
  if (!sh_ok) return false;   // the failure flag is set
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const uint32_t row = lo + i * NR + tid;
    if (rows && row < hi) {
      const size_t e = (size_t)row * R + r;
      A.x[e] = kOne ? x[i] : x[i] * rs[i];
    }
  }
  if (member == 0 && !rows && lane == 0) {
    out->k = k - 1;
    out->phi = rec.phi;
    out->bad = rec.bad ? 1 : 0;
  }
  __syncthreads();
  return true;
}

template <int L, int NG, int W, int RPT, int NT, bool DEFL>
__global__ __launch_bounds__(NT) void k_minres_group(GroupArgs A, FieldArgs F) {
  const int xcd = blockIdx.x % kGroupXcds, place = blockIdx.x / kGroupXcds;
  const int groups = (int)gridDim.x / W;
  for (int r = (place / W) * kGroupXcds + xcd; r < A.R; r += groups)
    if (!group_solve<L, NG, W, RPT, NT, DEFL>(A, F, r, place % W)) return;
}

}  // namespace mbl
