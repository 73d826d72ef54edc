// Whole FP64 MINRES solves (Alg. 2) in one launch, single or for every
// realization of a batch: one workgroup per realization for sectors that fit a
// compute unit's LDS and registers (L <= 12, resident.h), one group of
// workgroups on one XCD for L = 14, 16, 18 (group.h).
#include "group.h"

#include <algorithm>

namespace mbl {

// One workgroup, one row per thread: L <= 10 with 256 threads (n <= 252),
// L = 12 with 1024 (n = 924). States and neighbours come from the basis.
template <int LB, int NT, bool DEFL>
__global__ __launch_bounds__(NT) void k_minres_lds(DevBasis B, FieldArgs F, GroupArgs A) {
  constexpr int NPAIR = LB / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double q[NT];
  __shared__ double red[3 * NT / 64];
  __shared__ ResidentCoef co;
  __shared__ FieldArgs fs;   // of realization r
  const int tid = threadIdx.x, n = (int)B.n, L = B.L, r = blockIdx.x, R = A.R;
  if (tid < kMaxL) fs.h[tid] = tid < L ? (A.h ? A.h[(size_t)r * L + tid] : F.h[tid]) : 0.0;
  if (tid == 0) fs.c0 = A.c0 ? A.c0[r] : F.c0;
  __syncthreads();
  const RowTables t = setup_tables(B, fs, smem);
  __syncthreads();
  const double sc = A.scale ? A.scale[r] : A.scale1;
  uint32_t nb[1][NPAIR];
  double dg[1] = {0.0}, rs[1] = {0.0}, u[1] = {0.0}, x[1], v[1] = {0.0};
  const uint32_t zero = (uint32_t)n * 8u;   // n < NT: a row that stays 0
#pragma unroll
  for (int b = 0; b < NPAIR; ++b) nb[0][b] = zero | (zero << 16);
  // this thread's state: its row's block is the last one that starts at or
  // before it (blocks that hold no state have offset 0xffffffff)
  if (tid < n) {
    uint32_t hi = 0, off = 0;
    for (uint32_t h = 0; h < (1u << B.nhi); ++h) {
      const uint32_t o = B.hi_off[h];
      if (o <= (uint32_t)tid) {
        hi = h;
        off = o;
      }
    }
    const uint32_t a = (hi << B.nlo) |
                       t.state[B.lo_coff[B.half - __popc(hi)] + (uint32_t)tid - off];
    int na;
    dg[0] = row_diag<0>(B, fs, t, a, na);
    rs[0] = 1.0 / sqrt(precond_value(A.kind, dg[0], na));
    const size_t e = (size_t)tid * R + r;
    if (sc != 0.0) u[0] = sc * (A.src[e] - (A.ax0 ? A.ax0[e] : 0.0)) * rs[0];
    if (DEFL) v[0] = A.v[tid];
#pragma unroll
    for (int b = 0; b < LB; ++b) {
      if (b >= L) continue;
      const uint32_t m = b + 1 < L ? 3u << b : (1u | (1u << (L - 1)));
      const uint32_t two = a & m;
      if (two != 0 && two != m) {
        const uint32_t c = a ^ m;
        const uint32_t to = (B.hi_off[c >> B.nlo] + t.rank[c & ((1u << B.nlo) - 1u)]) * 8u;
        nb[0][b / 2] = (b & 1) ? (nb[0][b / 2] & 0xffffu) | (to << 16)
                               : (nb[0][b / 2] & 0xffff0000u) | to;
      }
    }
  }
  int64_t it = 0;
  double phi = 0.0;
  bool bad = false;
  if constexpr (DEFL)
    resident_minres<NPAIR, 1, NT, true>(nb, dg, rs, u, x, q, red, &co, A.tol, A.kmax, it, phi, bad,
                                        v, A.theta);
  else
    resident_minres<NPAIR, 1, NT>(nb, dg, rs, u, x, q, red, &co, A.tol, A.kmax, it, phi, bad,
                                  {0.0}, 0.0);
  if (tid < n) {
    const size_t e = (size_t)tid * R + r;
    A.x[e] = x[0];
  }
  if (tid == 0) {
    GroupOut* out = A.out + r;
    out->failed = 0;
    out->k = it;
    out->phi = phi;
    out->bad = bad ? 1 : 0;
  }
}

constexpr int kOutWords = (int)(sizeof(GroupOut) / 8);

// Results and slots zeroed; the first `preset` words take the failure flag, one
// per result.
__global__ void k_zero_words(unsigned long long* p, int n, int preset) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    p[i] = i < preset && i % kOutWords == 0 ? 1ull : 0ull;
}

// Group shapes <far bonds, workgroups, rows per thread, threads> by chain
// length and batch width: a batch gives every XCD R / 8 realizations, whose
// groups share its 32 compute units; beyond that a group takes several in
// turn. As many workgroups as there is room for, so few rows per thread, until
// groups would take turns. Measured, us per iteration of all R:
// L = 14, R <= 16: 1.82 (16 workgroups of 320 threads; 8 of 512 1.95; with the
//   whole vector in each window 2.19); R = 32: 1.97 (8 of 512; 16 of 320, two
//   realizations in turn, 3.72);
// L = 16, R <= 8: 2.09 (32 of 512, one row per thread; 16 of 512 with two 2.83;
//   8 of 512 with four 4.14); R = 16: 2.82 (16 of 512; 8 of 512 4.16); R = 32:
//   4.16 (8 of 512, four rows, two trips; 16 of 512, two in turn, 5.66; 8 of 1024
//   with two rows and one trip 14.9: of the 128 registers that 16 waves leave it
//   spills 376 bytes a thread);
// L = 18: 4.73 (32 of 448; of 512 4.88; six far bonds instead of five 4.73; 832
//   threads with two rows and one trip 18.2: 504 bytes spilled).
template <int L, int NG, int W, int RPT, int NT>
static hipError_t launch_group(GroupArgs A, const FieldArgs& F, hipStream_t s) {
  static_assert(RPT * (NT - 64) * W >= (int)cbinom(L, L / 2), "group too small");
  const void* fn = (const void*)&k_minres_group<L, NG, W, RPT, NT, false>;
  if (A.v) {
    if constexpr (W == 32 || (L == 14 && W == 16)) fn = (const void*)&k_minres_group<L, NG, W, RPT, NT, true>;
    else return hipErrorInvalidValue;   // the single form only
  }
  const int words = kOutWords * A.R + group_slots(W) * A.R;   // results, then slots
  hipLaunchKernelGGL(k_zero_words, dim3(std::min(64, (words + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<unsigned long long*>(A.out), words,
                     minres_launch_is("refused") ? kOutWords * A.R : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  FieldArgs Fc = F;
  void* args[] = {&A, &Fc};
  const int per_xcd = std::min((A.R + kGroupXcds - 1) / kGroupXcds, 32 / W);
  // cooperative: the workgroups of a group wait for each other
  return hipLaunchCooperativeKernel(fn, dim3(kGroupXcds * per_xcd * W), dim3(NT), args, 0, s);
}

static hipError_t launch_for(int L, const GroupArgs& A, const FieldArgs& F, hipStream_t s) {
  switch (L) {
    case 14:
      return A.R <= 16 ? launch_group<14, 3, 16, 1, 320>(A, F, s)
                       : launch_group<14, 3, 8, 1, 512>(A, F, s);
    case 16:
      return A.R <= 8    ? launch_group<16, 4, 32, 1, 512>(A, F, s)
             : A.R <= 16 ? launch_group<16, 4, 16, 2, 512>(A, F, s)
                         : launch_group<16, 4, 8, 4, 512>(A, F, s);
    default:
      return launch_group<18, 5, 32, 4, 448>(A, F, s);
  }
}

// words of the results and slots of any launch of (L, R)
static size_t scratch_words(int L, int R) {
  return ((size_t)kOutWords + (L <= 12 ? 0 : group_slots(L == 14 ? 16 : 32))) * (size_t)R;
}

// A wait that ran out has cost a second (group.h), and what held it up, work of
// others on the same compute units, may last: the solves of the basis then pass
// this form by for ten, so that no more than a tenth of the time goes to waits.
constexpr std::chrono::seconds kChipPause(10);
static int64_t steady_ns() {
  return std::chrono::duration_cast<std::chrono::nanoseconds>(
             std::chrono::steady_clock::now().time_since_epoch()).count();
}
// A solve of very few iterations does not pay for a cooperative launch whose
// workgroups first work out their rows' states and neighbours. Measured, us on
// chip and in launches per iteration, for a limit of 1, 5 and 20 iterations:
// L = 14 99 and 82, 107 and 147; L = 16 142 and 72, 150 and 141, 181 and 314; L =
// 18 170 and 88, 186 and 173, 259 and 393; batches (whose launches per iteration
// cost more) of R = 2 at L = 16 120 and 66, 129 and 169; at L = 18 145 and 66, 163
// and 177; of R = 32 at L = 18, where a group takes four realizations in turn,
// 447 and 116, 523 and 308, 807 and 937.
static int64_t chip_kmax(int L, int R) {
  if (L <= 12) return 0;
  if (L == 14) return 3;
  if (R == 1) return 6;
  return L == 16 ? 4 : std::max(5, 3 * R / kGroupXcds + 1);
}
bool group_minres_serves(const mbl_basis_s* b, int64_t kmax, int R) {
  return b->L <= 18 && kmax >= chip_kmax(b->L, R) &&
         steady_ns() >= b->chip_from.load(std::memory_order_relaxed);
}

// Launches the solves of A with their results and slots in scratch (device);
// host: pinned, R results.
static mbl_status group_run(const mbl_basis_s* b, const FieldArgs& F, GroupArgs A, double* scratch,
                            double* host, hipStream_t s, MinresState* res, bool* refused) {
  A.fenced = minres_launch_is("fenced");
  A.out = reinterpret_cast<GroupOut*>(scratch);
  A.slots = reinterpret_cast<unsigned long long*>(A.out + A.R);
  if (b->L <= 12) {
    const DevBasis B = b->dev();
    const size_t lds = row_lds_for(b->nlo);
    const dim3 g(A.R);
    if (b->L <= 10) {
      if (A.v)
        hipLaunchKernelGGL((k_minres_lds<10, 256, true>), g, dim3(256), lds, s, B, F, A);
      else
        hipLaunchKernelGGL((k_minres_lds<10, 256, false>), g, dim3(256), lds, s, B, F, A);
    } else {
      if (A.v)
        hipLaunchKernelGGL((k_minres_lds<12, 1024, true>), g, dim3(1024), lds, s, B, F, A);
      else
        hipLaunchKernelGGL((k_minres_lds<12, 1024, false>), g, dim3(1024), lds, s, B, F, A);
    }
    MBL_HIP(hipGetLastError());
  } else {
    if (launch_for(b->L, A, F, s) != hipSuccess) {
      (void)hipGetLastError();
      *refused = true;
      return MBL_ERR_HIP;
    }
  }
  MBL_HIP(hipMemcpyAsync(host, A.out, sizeof(GroupOut) * A.R, hipMemcpyDeviceToHost, s));
  MBL_HIP(hipStreamSynchronize(s));
  const GroupOut* o = reinterpret_cast<const GroupOut*>(host);
  for (int r = 0; r < A.R; ++r) {
    // a workgroup waited a second for the others (say, for a compute unit that
    // another stream's kernel holds); some rows of A.x may be written
    if (o[r].failed) {
      b->chip_from.store(steady_ns() + std::chrono::nanoseconds(kChipPause).count(),
                         std::memory_order_relaxed);
      *refused = true;
      return MBL_ERR_HIP;
    }
    res[r].k = o[r].k;
    res[r].phi = o[r].phi;
    res[r].bad = (int32_t)o[r].bad;
  }
  return MBL_OK;
}

mbl_status group_minres(const mbl_basis_s* b, const FieldArgs& F, const double* src, double scale,
                        const double* ax0, double* x, double tol, int64_t kmax, int precond,
                        mbl_workspace_s* ws, const double* defl, double theta, hipStream_t s,
                        MinresState* out, bool* refused) {
  *refused = false;
  GroupArgs A{};
  A.src = src;
  A.ax0 = ax0;
  // x - x0 goes to a vector of the workspace, and into x once the solve counts:
  // the launches per iteration, the fallback, start from the x0 in x
  double* const dx = static_cast<double*>(ws->d[0]);
  A.x = ax0 ? dx : x;
  A.scale1 = scale;
  for (int i = 0; i < 3; ++i) A.q[i] = static_cast<double*>(ws->q[i]);
  static_assert(kOutWords + group_slots(32) <= kMaxPartials * 64, "scratch is the partial sums");
  A.v = defl;
  A.theta = theta;
  A.tol = tol;
  A.kmax = kmax;
  A.kind = precond;
  A.R = 1;
  const mbl_status st = group_run(b, F, A, ws->partials1, ws->h_red, s, out, refused);
  if (st == MBL_OK && ax0) MBL_HIP(launch_axpby(b->n, 1.0, dx, 1.0, x, s));
  return st;
}

mbl_status group_minres_batched(const mbl_basis_s* b, int R, const double* h, const double* c0,
                                const double* src, const double* scale, double* x, double* const* q,
                                double* scratch, double* host, double tol, int64_t kmax,
                                int precond, hipStream_t s, MinresState* out, bool* refused) {
  *refused = scratch_words(b->L, R) > (size_t)b->n * R;   // scratch is one batch vector
  if (*refused) return MBL_ERR_HIP;
  GroupArgs A{};
  A.src = src;
  A.x = x;
  A.scale = scale;
  A.h = h;
  A.c0 = c0;
  for (int i = 0; i < 3; ++i) A.q[i] = q[i];
  A.tol = tol;
  A.kmax = kmax;
  A.kind = precond;
  A.R = R;
  return group_run(b, FieldArgs{}, A, scratch, host, s, out, refused);
}

}  // namespace mbl
