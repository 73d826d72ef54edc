// Row kernels of the matrix-free Hamiltonian (Eq. (1)) on gfx950, and the
// dense vector helpers around them.
//
// Work decomposition. A state a = (hi << nlo) | lo. Rows sharing hi are one
// contiguous block; a chunk is up to 64 consecutive rows of one block and is
// processed by one wavefront, one row per lane. Inside a wavefront hi is
// uniform, so everything that depends on hi alone (block offsets of the
// neighbour blocks, which high bonds are antiparallel) is scalar work, and a
// hop on a bond inside the high bits reads a contiguous run of x from the
// neighbour block: a coalesced load. Hops on bonds inside the low bits stay
// in the same block (a few KB, cache resident); their targets come from the
// low-pattern rank table held in LDS. The two bonds that cross the split (the
// one between bit nlo-1 and bit nlo, and the periodic bond between bit L-1
// and bit 0) change the popcount of both halves and use both tables.
//
// Diagonal: a_aa - sigma = L/4 - N_anti/2 + (1/2) sum_j h_j - F(a) - sigma,
// where N_anti = popcount(a xor rotl_L(a, 1)) counts antiparallel bonds and
// F(a) = sum of h_j over set bits, summed from a per-nibble table in LDS.
//
// Reductions are per-workgroup partial sums written in a fixed order and
// reduced again in a fixed order, so results are bitwise reproducible.
#include "rows.h"

#include <algorithm>
#include <cstdlib>

namespace mbl {

// ---------------------------------------------------------------------------
// y = (H - sigma) x. MODE 0: plain; 1: partial sums of x.y; 2: partial sums of
// y.y. GUARD: the product of MINRES iteration k, which first takes the Givens
// step of iteration k - 1 (G; every workgroup the same, workgroup 0 stores
// it) and returns at once when the state is then done. (L, NLO) = (0, 0) is
// the runtime-split form.
template <typename T, int MODE, bool GUARD, int L, int NLO>
__global__ __launch_bounds__(kWG) void k_apply(DevBasis B, FieldArgs F, MinresGivens G,
                                               const T* __restrict__ x, T* __restrict__ y,
                                               double* __restrict__ partials, Defl D) {
  extern __shared__ __align__(16) unsigned char smem[];
  // the MINRES scalars and partial sums are loaded before the table fill, so
  // that the two latencies overlap
  PartialsPrefetch pq, pc;
  MinresState sp{};
  double al = 0.0;
  if (GUARD) {
    if (G.active) {
      prefetch_partials(G.part2, G.P2, pq);
      sp = *G.Sprev;
      al = *G.alpha;
    } else if (G.Scur->done) {
      return;
    }
    if (D.v) prefetch_partials(D.c_part, D.P, pc);
  }
  const RowTables t = setup_tables<L>(B, F, smem);
  __syncthreads();
  if (GUARD && G.active) {
    const double qz = reduce_prefetched(pq, G.P2, t.red);
    const MinresState so = minres_givens_step(sp, al, qz, G.tol, G.kmax);
    if (blockIdx.x == 0 && threadIdx.x == 0) *G.Scur = so;
    if (so.done) return;
  }
  // rank-one term theta v (v . x) of a deflated MINRES operator
  double dcoef = 0.0;
  if (GUARD && D.v) dcoef = D.theta * reduce_prefetched(pc, D.P, t.red);
  double acc = 0.0;
  for_rows(B, t, [&](uint32_t row, uint32_t hi, uint32_t lo, uint32_t j, uint32_t block0,
                     uint32_t a) {
    const double xi = (double)x[row];
    const double off = RowOps<T, L, NLO>::offdiag(B, t, x, hi, lo, j, block0);
    int na;
    const double dsh = row_diag<L>(B, F, t, a, na);
    double yv = dsh * xi + 0.5 * off;
    if (GUARD && D.v) yv += dcoef * D.v[row];
    const T yt = (T)yv;
    y[row] = yt;
    if (MODE == 1) acc += xi * (double)yt;
    if (MODE == 2) acc += (double)yt * (double)yt;
  });
  if (MODE != 0) {
    const double s = block_sum_all(acc, t.red);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------
// The same product for the split nlo = 13, by blocks: a workgroup stages a
// block of x (up to 1716 rows) in LDS by LDS DMA, the next block while it
// computes one, and takes the 12 low-bond neighbours from there, their places
// read as 16-bit halves from a table of the low patterns (coalesced, in L2).
// What is uniform over a block (rows of its high-bond neighbours, high fields)
// is read once, through the scalar cache; the high bonds are coalesced loads of
// the neighbour block's rows. Sums in the order of k_apply: the same bits.
//
// Counters at L = 26, k_apply and this: vector instructions per 64 rows 199 and
// 118 (FP32 227 and 147); address units busy 67 and 67 % of the time (55 and 60);
// read past the L2s 469 and 547 MB (190 and 212), beside 83 (42) MB written. So in
// FP64 the fabric bounds this one: 630 MB in 98 us is the 6.5 TB/s that gathers
// reach, x read 6.6 times by the high bonds that leave an XCD's part. In FP32 (254
// MB in 77 us) no one unit does. Measured, k_apply and this, us: FP64 L = 22 13.3
// and 9.8, L = 24 35.6 and 26.9, L = 26 134.8 and 99.0, L = 28 632 and 494, L = 30
// 2911 and 2340; FP32 12.0 and 9.4, 33.2 and 24.1, 119.5 and 77.8, 493 and 307, 2176
// and 1396. At L = 20 (6.2 and 7.0; FP32 6.1 and 5.9) the call is as long as its
// launch either way, and an iteration of MINRES 16.0 and 15.9.
constexpr int kBWT = 512;   // two (L <= 22) or three workgroups per compute unit

template <typename T, int MODE, bool GUARD, int L>
__global__ __launch_bounds__(kBWT, L > 22 ? 6 : 4) void k_apply_block(
    FieldArgs F, BlockPlan P, uint32_t n, MinresGivens G, const T* __restrict__ x,
    T* __restrict__ y, double* __restrict__ partials, Defl D) {
  constexpr int NLO = kBlockLoBits, NHI = L - NLO, NNIB = (L + 3) >> 2;
  constexpr int NP = block_pairs(NLO);
  constexpr uint32_t kZero = block_zero(NLO), kStride = block_stride(NLO);
  constexpr uint32_t kPer = 16 / sizeof(T);               // elements of a DMA piece
  constexpr uint32_t kBuf = kZero + 4;
  constexpr int kShift = sizeof(T) == 8 ? 3 : 2;
  __shared__ __align__(16) T buf[2 * kBuf];
  __shared__ double lut[NNIB * 16];   // field sums of the four-site groups
  __shared__ double lut01[256];       // and of the lowest two together
  __shared__ double red[kBWT / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = uni(tid >> 6);
  // the plan through the scalar cache (nothing writes it)
  typedef const __attribute__((address_space(4))) uint32_t plan_u32;
  constexpr int kItem = sizeof(BlockItem) / 4;
  plan_u32* item = (plan_u32*)(uintptr_t)P.items;
  plan_u32* const first = (plan_u32*)(uintptr_t)P.first;
  plan_u32* const end = item + kItem * first[blockIdx.x + 1];
  item += kItem * first[blockIdx.x];
  auto fetch = [&](plan_u32* p) {
    BlockItem v;
    v.hi = p[0], v.row0 = p[1], v.cnt = p[2], v.word0 = p[3], v.bnd = p[4], v.wrap = p[5];
#pragma unroll
    for (int b = 0; b + 1 < NHI; ++b) v.nb[b] = p[8 + b];
    return v;
  };
  auto group_sum = [&](int k, int bits) {
    double v = 0.0;
    for (int b = 0; b < 4; ++b)
      if (4 * k + b < L && ((bits >> b) & 1)) v += F.h[4 * k + b];
    return v;
  };
  for (int t = tid; t < NNIB * 16; t += kBWT) lut[t] = group_sum(t >> 4, t & 15);
  if (tid < 256) lut01[tid] = group_sum(0, tid & 15) + group_sum(1, tid >> 4);
  double dcoef = 0.0;
  if (GUARD) {
    bool live;
    if (G.active) {
      const double qz = reduce_partials(G.part2, G.P2, red);
      const MinresState so = minres_givens_step(*G.Sprev, *G.alpha, qz, G.tol, G.kmax);
      if (blockIdx.x == 0 && tid == 0) *G.Scur = so;
      live = !so.done;
    } else {
      live = !G.Scur->done;
    }
    if (!live) return;
    // rank-one term theta v (v . x) of a deflated MINRES operator
    if (D.v) dcoef = D.theta * reduce_partials(D.c_part, D.P, red);
  }
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(x), (short)0, (int)(n << kShift), 0x00020000);
  const __amdgpu_buffer_rsrc_t ry =
      __builtin_amdgcn_make_buffer_rsrc(y, (short)0, (int)(n << kShift), 0x00020000);
  const __amdgpu_buffer_rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(P.nbr), (short)0, (int)(4 * block_words(NLO) * kStride), 0x00020000);
  typedef __attribute__((address_space(3))) void lds_void;
  // rows row0 .. row0 + cnt - 1 into half b; row 0 lands at element row0 mod kPer
  auto stage = [&](uint32_t row0, uint32_t cnt, uint32_t b) {
    const uint32_t a0 = row0 & ~(kPer - 1), bytes = (row0 + cnt - a0) << kShift;
    for (uint32_t j = wave; j * 1024u < bytes; j += kBWT / 64) {
      const uint32_t off = j * 1024u + lane * 16u;
      if (off < bytes)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)((char*)(buf + b) + j * 1024u),
                                                 16, (int)off, (int)(a0 << kShift), 0, 0);
    }
  };
  auto load = [&](uint32_t voff, uint32_t soff) -> T {
    T v;
    if constexpr (sizeof(T) == 8) {
      const auto u = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)voff, (int)soff, 0);
      __builtin_memcpy(&v, &u, 8);
    } else {
      const auto u = __builtin_amdgcn_raw_buffer_load_b32(rx, (int)voff, (int)soff, 0);
      __builtin_memcpy(&v, &u, 4);
    }
    return v;
  };
  if (tid < 8) buf[(tid & 3) + kZero + (tid & 4 ? kBuf : 0u)] = (T)0;
  double acc = 0.0;
  BlockItem it{};
  uint32_t next_row0 = 0, next_cnt = 0;   // of the item after it
  if (item < end) {
    it = fetch(item);
    stage(it.row0, it.cnt, 0);
    if (item + kItem < end) {
      next_row0 = item[kItem + 1];
      next_cnt = item[kItem + 2];
    }
  }
  for (uint32_t cur = 0; item < end; item += kItem, cur = kBuf - cur) {
    const uint32_t hi = it.hi, cnt = it.cnt, row0 = it.row0;
    const uint32_t hflips = hi ^ (hi >> 1);
    uint32_t hb[NHI - 1];
#pragma unroll
    for (int b = 0; b + 1 < NHI; ++b) hb[b] = it.nb[b] << kShift;
    const uint32_t hb_bnd = it.bnd << kShift, hb_wrap = it.wrap << kShift;
    // the words of the first row, before the wait for the block
    const uint32_t vw = NP + 3 * ((hi & 1u) + 2 * (hi >> (NHI - 1)));
    uint32_t nb[NP], lo, r_bnd, r_wrap;
    auto words = [&](uint32_t j) {   // past the class: other words, not used
      const int off = (int)((it.word0 + j) << 2);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        nb[p] = __builtin_amdgcn_raw_buffer_load_b32(rn, off, (int)(4 * p * kStride), 0);
      lo = __builtin_amdgcn_raw_buffer_load_b32(rn, off, (int)(4 * vw * kStride), 0);
      r_bnd = __builtin_amdgcn_raw_buffer_load_b32(rn, off, (int)(4 * (vw + 1) * kStride), 0);
      r_wrap = __builtin_amdgcn_raw_buffer_load_b32(rn, off, (int)(4 * (vw + 2) * kStride), 0);
    };
    uint32_t j = tid;
    words(j);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's share of the block landed
    __syncthreads();                      // every wave's did, and the other half is free
    const uint32_t base = cur + (row0 & (kPer - 1));
    if (next_cnt) stage(next_row0, next_cnt, kBuf - cur);
    // uniform over the block: the field sums of the groups above the low bits
    double f_up[NNIB - 3];
#pragma unroll
    for (int k = 4; k < NNIB; ++k) f_up[k - 3] = lut[(k << 4) + ((hi >> (4 * k - NLO)) & 15u)];
    const uint32_t i3 = 48 + ((hi << 1) & 15u);
    const double f3_0 = lut[i3], f3_1 = lut[i3 + 1];
    const int na_hi = __popc(hflips & ((1u << (NHI - 1)) - 1u));
    for (; j < cnt; j += kBWT) {
      // the loads from memory first: high bonds, the split and periodic bonds
      T vh[NHI - 1];
#pragma unroll
      for (int b = 0; b + 1 < NHI; ++b)
        if ((hflips >> b) & 1u) vh[b] = load(j << kShift, hb[b]);
      const T v_bnd = load(r_bnd << kShift, hb_bnd), v_wrap = load(r_wrap << kShift, hb_wrap);
      const uint32_t low = lo;
      double off = 0.0;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const uint32_t w = nb[p] + base * 0x10001u;
        off += (double)buf[w & 0xffffu];
        off += (double)buf[w >> 16];
      }
      words(j + kBWT);
      const double xi = (double)buf[base + j];
      const int na = na_hi + (int)(low >> 16);
      double f = lut01[low & 255u] + lut[32 + ((low >> 8) & 15u)];
      f += (low & 4096u) ? f3_1 : f3_0;
#pragma unroll
      for (int k = 4; k < NNIB; ++k) f += f_up[k - 3];
      off += (double)v_bnd;
#pragma unroll
      for (int b = 0; b + 1 < NHI; ++b)
        if ((hflips >> b) & 1u) off += (double)vh[b];
      off += (double)v_wrap;
      double yv = (F.c0 - 0.5 * (double)na - f) * xi + 0.5 * off;
      if (GUARD && D.v) yv += dcoef * D.v[row0 + j];
      const T yt = (T)yv;
      if constexpr (sizeof(T) == 8) {
        unsigned long long u;
        __builtin_memcpy(&u, &yt, 8);
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{(uint32_t)u, (uint32_t)(u >> 32)}, ry,
                                              (int)(j << kShift), (int)(row0 << kShift), 0);
      } else {
        uint32_t u;
        __builtin_memcpy(&u, &yt, 4);
        __builtin_amdgcn_raw_buffer_store_b32(u, ry, (int)(j << kShift), (int)(row0 << kShift), 0);
      }
      if (MODE == 1) acc += xi * (double)yt;
      if (MODE == 2) acc += (double)yt * (double)yt;
    }
    if (item + kItem < end) it = fetch(item + kItem);
    next_cnt = 0;
    if (item + 2 * kItem < end) {
      next_row0 = item[2 * kItem + 1];
      next_cnt = item[2 * kItem + 2];
    }
  }
  if (MODE != 0) {
    const double s = block_sum_all(acc, red);
    if (tid == 0) partials[blockIdx.x] = s;
  }
}

__global__ __launch_bounds__(kWG) void k_precond(DevBasis B, FieldArgs F, int kind,
                                                 const double* z, double* q) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RowTables t = setup_tables(B, F, smem);
  __syncthreads();
  for_rows(B, t, [&](uint32_t row, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t a) {
    int na;
    const double dsh = row_diag<0>(B, F, t, a, na);
    q[row] = z[row] / precond_value(kind, dsh, na);
  });
}

// r = rhs - (H - sigma) x, partials[2g] = sum r^2 / m, partials[2g+1] = sum r^2
template <int L, int NLO>
__global__ __launch_bounds__(kWG) void k_residual(DevBasis B, FieldArgs F, int kind,
                                                  const double* __restrict__ rhs,
                                                  const double* __restrict__ x,
                                                  double* __restrict__ r,
                                                  double* __restrict__ partials) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RowTables t = setup_tables<L>(B, F, smem);
  __syncthreads();
  double am = 0.0, a2 = 0.0;
  for_rows(B, t, [&](uint32_t row, uint32_t hi, uint32_t lo, uint32_t j, uint32_t block0,
                     uint32_t a) {
    const double off = RowOps<double, L, NLO>::offdiag(B, t, x, hi, lo, j, block0);
    int na;
    const double dsh = row_diag<L>(B, F, t, a, na);
    const double ri = rhs[row] - (dsh * x[row] + 0.5 * off);
    r[row] = ri;
    am += ri * ri / precond_value(kind, dsh, na);
    a2 += ri * ri;
  });
  const double sm = block_sum_all(am, t.red);
  const double s2 = block_sum_all(a2, t.red);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = sm;
    partials[2 * blockIdx.x + 1] = s2;
  }
}

__global__ __launch_bounds__(kWG) void k_states(DevBasis B, uint32_t* states) {
  extern __shared__ __align__(16) unsigned char smem[];
  FieldArgs F{};
  const RowTables t = setup_tables(B, F, smem);
  __syncthreads();
  for_rows(B, t, [&](uint32_t row, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t a) {
    states[row] = a;
  });
}

__global__ __launch_bounds__(kWG) void k_rank(DevBasis B, const uint32_t* states, int64_t count,
                                              int64_t* ranks) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t a = states[i];
  const uint64_t top = (uint64_t)a >> B.L;
  int64_t out = -1;
  if (top == 0 && __popc(a) == B.half) {
    const uint32_t hi = a >> B.nlo, lo = a & ((1u << B.nlo) - 1u);
    out = (int64_t)B.hi_off[hi] + B.lo_rank[lo];
  }
  ranks[i] = out;
}

// Twist overlap partial sums. m(a) = 2 sum_{set bits p} (p + 1) - L(L+1)/2,
// u_a = exp(i pi m / L) from a 2L-entry table.
struct TwistTables {
  double c[2 * kMaxL];
  double s[2 * kMaxL];
};

__global__ __launch_bounds__(kWG) void k_twist(DevBasis B, TwistTables T, const double* psi,
                                               int64_t ld, double* partials) {
  extern __shared__ __align__(16) unsigned char smem[];
  FieldArgs F{};
  const RowTables t = setup_tables(B, F, smem);
  __syncthreads();
  const double* v = psi + (size_t)blockIdx.y * ld;
  const int twoL = 2 * B.L;
  const int base = (B.L * (B.L + 1)) / 2;
  double are = 0.0, aim = 0.0;
  for_rows(B, t, [&](uint32_t row, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t a) {
    int sum = 0;   // sum over set bits of (p + 1)
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      uint32_t w = 0;
      for (int p = 0; p < 32; ++p)
        if (((p + 1) >> k) & 1) w |= (1u << p);
      sum += __popc(a & w) << k;
    }
    int m = (2 * sum - base) % twoL;
    if (m < 0) m += twoL;
    const double c2 = v[row] * v[row];
    are += c2 * T.c[m];
    aim += c2 * T.s[m];
  });
  const double sr = block_sum_all(are, t.red);
  const double si = block_sum_all(aim, t.red);
  if (threadIdx.x == 0) {
    const size_t g = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    partials[2 * g] = sr;
    partials[2 * g + 1] = si;
  }
}

// ---------------------------------------------------------------------------
// dense helpers

constexpr int kDenseGrid = 512;

__global__ __launch_bounds__(kWG) void k_dot(int64_t n, const double* __restrict__ x,
                                             const double* __restrict__ y,
                                             double* __restrict__ partials) {
  __shared__ double red[kWavesPerWG];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    acc += x[i] * y[i];
  const double s = block_sum_all(acc, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// out[v] = sum_{g < nparts} partials[g * stride + v], one workgroup per v.
__global__ __launch_bounds__(kWG) void k_reduce(const double* __restrict__ partials, int nparts,
                                                int stride, double* __restrict__ out) {
  __shared__ double red[kWavesPerWG];
  const int v = blockIdx.x;
  double acc = 0.0;
  for (int g = threadIdx.x; g < nparts; g += blockDim.x) acc += partials[(size_t)g * stride + v];
  const double s = block_sum_all(acc, red);
  if (threadIdx.x == 0) out[v] = s;
}

__global__ __launch_bounds__(kWG) void k_axpby(int64_t n, double a, const double* __restrict__ x,
                                               double b, double* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    // BLAS convention: a zero coefficient does not read its operand
    const double ax = a != 0.0 ? a * x[i] : 0.0;
    y[i] = b != 0.0 ? ax + b * y[i] : ax;
  }
}

__global__ __launch_bounds__(kWG) void k_scale_copy(int64_t n, double a, const double* __restrict__ x,
                                                    double* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
}

__global__ __launch_bounds__(kWG) void k_fill(int64_t n, double v, double* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = v;
}

// SplitMix64 (Steele, Lea & Flood 2014) of seed + (i + 1) * golden gamma,
// top 53 bits mapped to [-1/2, 1/2).
__global__ __launch_bounds__(kWG) void k_splitmix(int64_t n, uint64_t seed, double* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    y[i] = (double)(z >> 11) * 0x1.0p-53 - 0.5;
  }
}

// ---------------------------------------------------------------------------
// host launch wrappers

int row_grid(const mbl_basis_s* b) {
  int g = (b->nchunks + kWavesPerWG - 1) / kWavesPerWG;
  if (g > kMaxPartials) g = kMaxPartials;
  if (g < 1) g = 1;
  return g >= 64 ? (g / 8) * 8 : g;   // whole XCD slices once the grid is large
}

size_t row_lds_bytes(const mbl_basis_s* b) { return row_lds_for(b->nlo); }

static int dense_grid(int64_t n) {
  int64_t g = (n + kWG - 1) / kWG;
  return (int)(g < 1 ? 1 : (g > kDenseGrid ? kDenseGrid : g));
}

// The block-staged product serves every chain that has a plan; LDS DMA moves 16
// bytes, so a vector that does not start on 16 bytes takes the row kernel.
static bool block_serves(const mbl_basis_s* b, const void* x) {
  return b->block.G > 0 && ((uintptr_t)x & 15u) == 0;
}

int minres_apply_grid(const mbl_basis_s* b) {
  return b->block.G > 0 ? b->block.G : row_grid(b);   // the solver's vectors are aligned
}

template <typename T, int MODE, bool GUARD>
static hipError_t block_dispatch(const mbl_basis_s* b, const FieldArgs& F, const MinresGivens& S,
                                 const T* x, T* y, double* partials, hipStream_t s,
                                 const Defl& D) {
  const dim3 g(b->block.G), blk(kBWT);
  const BlockPlan P = b->block.dev();
  const uint32_t n = (uint32_t)b->n;
  switch (b->L) {
#define MBL_BLOCK(LL)                                                                          \
  case LL:                                                                                     \
    hipLaunchKernelGGL((k_apply_block<T, MODE, GUARD, LL>), g, blk, 0, s, F, P, n, S, x, y,    \
                       partials, D);                                                           \
    break;
    MBL_BLOCK(20)
    MBL_BLOCK(22)
    MBL_BLOCK(24)
    MBL_BLOCK(26)
    MBL_BLOCK(28)
    MBL_BLOCK(30)
#undef MBL_BLOCK
  }
  return hipGetLastError();
}

// by blocks where the basis has a plan, else the (L, NLO) instance matching the
// basis, else the runtime form
template <typename T, int MODE, bool GUARD>
static hipError_t apply_dispatch(const mbl_basis_s* b, const FieldArgs& F, const MinresGivens& S,
                                 const T* x, T* y, double* partials, hipStream_t s,
                                 const Defl& D = Defl{}) {
  if (block_serves(b, x)) return block_dispatch<T, MODE, GUARD>(b, F, S, x, y, partials, s, D);
  const dim3 g(row_grid(b)), blk(kWG);
  const size_t lds = row_lds_bytes(b);
  const DevBasis B = b->dev();
  switch (b->L * 64 + b->nlo) {
#define MBL_CASE(LL, NN)                                                                     \
  case LL * 64 + NN:                                                                        \
    hipLaunchKernelGGL((k_apply<T, MODE, GUARD, LL, NN>), g, blk, lds, s, B, F, S, x, y,  \
                       partials, D);                                                        \
    return hipGetLastError();
    MBL_FAST_SPLITS(MBL_CASE)
#undef MBL_CASE
    default:
      hipLaunchKernelGGL((k_apply<T, MODE, GUARD, 0, 0>), g, blk, lds, s, B, F, S, x, y,
                         partials, D);
      return hipGetLastError();
  }
}

template <typename T>
hipError_t launch_apply(const mbl_basis_s* b, const FieldArgs& F, const T* x, T* y, int mode,
                        double* partials, int* nparts, hipStream_t s) {
  if (nparts) *nparts = block_serves(b, x) ? b->block.G : row_grid(b);
  if (mode == 0) return apply_dispatch<T, 0, false>(b, F, MinresGivens{}, x, y, partials, s);
  if (mode == 1) return apply_dispatch<T, 1, false>(b, F, MinresGivens{}, x, y, partials, s);
  return apply_dispatch<T, 2, false>(b, F, MinresGivens{}, x, y, partials, s);
}
template hipError_t launch_apply<double>(const mbl_basis_s*, const FieldArgs&, const double*,
                                         double*, int, double*, int*, hipStream_t);
template hipError_t launch_apply<float>(const mbl_basis_s*, const FieldArgs&, const float*, float*,
                                        int, double*, int*, hipStream_t);

template <typename T>
hipError_t launch_minres_apply(const mbl_basis_s* b, const FieldArgs& F, const MinresGivens& G,
                               const T* q, T* p, double* partials, const Defl& D, hipStream_t s) {
  return apply_dispatch<T, 1, true>(b, F, G, q, p, partials, s, D);
}
template hipError_t launch_minres_apply<double>(const mbl_basis_s*, const FieldArgs&,
                                                const MinresGivens&, const double*, double*,
                                                double*, const Defl&, hipStream_t);
template hipError_t launch_minres_apply<float>(const mbl_basis_s*, const FieldArgs&,
                                               const MinresGivens&, const float*, float*, double*,
                                               const Defl&, hipStream_t);

hipError_t launch_precond(const mbl_basis_s* b, const FieldArgs& F, int kind, const double* z,
                          double* q, hipStream_t s) {
  hipLaunchKernelGGL(k_precond, dim3(row_grid(b)), dim3(kWG), row_lds_bytes(b), s, b->dev(), F,
                     kind, z, q);
  return hipGetLastError();
}

hipError_t launch_residual(const mbl_basis_s* b, const FieldArgs& F, int precond,
                           const double* rhs, const double* x, double* r, double* partials,
                           int* nparts, hipStream_t s) {
  const int g = row_grid(b);
  if (nparts) *nparts = g;
  const size_t lds = row_lds_bytes(b);
  switch (b->L * 64 + b->nlo) {
#define MBL_CASE(LL, NN)                                                                    \
  case LL * 64 + NN:                                                                       \
    hipLaunchKernelGGL((k_residual<LL, NN>), dim3(g), dim3(kWG), lds, s, b->dev(), F,     \
                       precond, rhs, x, r, partials);                                      \
    return hipGetLastError();
    MBL_FAST_SPLITS(MBL_CASE)
#undef MBL_CASE
    default:
      hipLaunchKernelGGL((k_residual<0, 0>), dim3(g), dim3(kWG), lds, s, b->dev(), F, precond,
                         rhs, x, r, partials);
      return hipGetLastError();
  }
}

hipError_t launch_states(const mbl_basis_s* b, uint32_t* states, hipStream_t s) {
  hipLaunchKernelGGL(k_states, dim3(row_grid(b)), dim3(kWG), row_lds_bytes(b), s, b->dev(),
                     states);
  return hipGetLastError();
}

hipError_t launch_rank(const mbl_basis_s* b, const uint32_t* states, int64_t count,
                       int64_t* ranks, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const int64_t g = (count + kWG - 1) / kWG;
  hipLaunchKernelGGL(k_rank, dim3((unsigned)g), dim3(kWG), 0, s, b->dev(), states, count, ranks);
  return hipGetLastError();
}

hipError_t launch_twist(const mbl_basis_s* b, const double* psi, int64_t ld, int nvec,
                        const double* costab, const double* sintab, double* partials, int* nparts,
                        hipStream_t s) {
  TwistTables T{};
  for (int m = 0; m < 2 * b->L; ++m) {
    T.c[m] = costab[m];
    T.s[m] = sintab[m];
  }
  int g = row_grid(b);
  if (g * nvec > kMaxPartials * 32) g = (kMaxPartials * 32) / nvec;
  if (g < 1) g = 1;
  if (nparts) *nparts = g;
  hipLaunchKernelGGL(k_twist, dim3(g, nvec), dim3(kWG), row_lds_bytes(b), s, b->dev(), T, psi, ld,
                     partials);
  return hipGetLastError();
}

hipError_t launch_dot(int64_t n, const double* x, const double* y, double* partials, int* nparts,
                      hipStream_t s) {
  const int g = dense_grid(n);
  if (nparts) *nparts = g;
  hipLaunchKernelGGL(k_dot, dim3(g), dim3(kWG), 0, s, n, x, y, partials);
  return hipGetLastError();
}

hipError_t launch_reduce(const double* partials, int nparts, int stride, int nvals, double* out,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(nvals), dim3(kWG), 0, s, partials, nparts, stride, out);
  return hipGetLastError();
}

hipError_t launch_axpby(int64_t n, double a, const double* x, double b, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3(dense_grid(n)), dim3(kWG), 0, s, n, a, x, b, y);
  return hipGetLastError();
}

hipError_t launch_scale_copy(int64_t n, double a, const double* x, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_copy, dim3(dense_grid(n)), dim3(kWG), 0, s, n, a, x, y);
  return hipGetLastError();
}

hipError_t launch_fill(int64_t n, double v, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_fill, dim3(dense_grid(n)), dim3(kWG), 0, s, n, v, y);
  return hipGetLastError();
}

hipError_t launch_splitmix(int64_t n, uint64_t seed, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_splitmix, dim3(dense_grid(n)), dim3(kWG), 0, s, n, seed, y);
  return hipGetLastError();
}

}  // namespace mbl
