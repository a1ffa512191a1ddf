// reduce.hip -- per-token training-inference discrepancy, its segmented
// masked reductions, and the ACRL controller step.
//
//  * d = |pi(a_t) - mu(a_t)| on probabilities (Eq. distance_metric) and the
//    log-ratio log(pi/mu) (the log of rho in Sec. 2.2 / 4.1).
//  * Per response: |a_i|, sum d, sum log-ratio (log rho_i of sequence-level
//    MIS), mean d.  Per group (the G responses of a prompt): Y_g, the formula
//    of Y in Sec. 4.1.  Batch: mean of Y_g (the outer mean of X) and token
//    statistics (mean / max / population std of d, mean entropies).
//  * Controller (Eq. ACRL): weight = min((pi/mu)^alpha, C),
//    alpha = gamma sign(A) (1 - Y/X).
//
// Layout: slots [B, L] row-major, the usual right-padded response layout.
// One workgroup per response reads its L contiguous slots with coalesced
// loads; all sums are fp64 and combined by fixed-shape tree reductions, so
// results are deterministic (no floating-point atomics).  These kernels are
// HBM / latency bound; the controller is a plain grid-stride stream.
#include <mutex>
#include <type_traits>

#include "acrl_internal.h"

namespace acrl {
namespace {

constexpr int kRedThreads = 256;

// Per-response intermediate record in the workspace.
struct SeqRec {
  double n, sum_d, sum_lr, sum_hp, sum_hm, max_d, m2;  // m2 = sum (d - mean_i)^2
  double pad;
};

// Sum / maximum over groups of N = 4, 16 or 64 consecutive lanes: DPP inside
// each row of 16, lane exchanges across rows.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int N>
__device__ __forceinline__ double lane_sum(double v) {
  v += dpp_f64<0xB1>(v);                      // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);                      // quad_perm [2,3,0,1]
  if constexpr (N >= 16) {
    v += dpp_f64<0x124>(v);                   // row_ror:4
    v += dpp_f64<0x128>(v);                   // row_ror:8
  }
  if constexpr (N == 64) {
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
  }
  return v;
}
template <int N>
__device__ __forceinline__ double lane_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  if constexpr (N >= 16) {
    v = fmax(v, dpp_f64<0x124>(v));
    v = fmax(v, dpp_f64<0x128>(v));
  }
  if constexpr (N == 64) {
    v = fmax(v, __shfl_xor(v, 16));
    v = fmax(v, __shfl_xor(v, 32));
  }
  return v;
}

__device__ __forceinline__ double first_lane(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sums of NS values and the maximum of mx over a workgroup of NT = 64, 256 or
// 1024 threads, one barrier (none for a wavefront): trees inside each
// wavefront, then every thread's lane group of NT / 64 lanes takes one
// wavefront's result each and adds them by the same tree.  Deterministic.
// (The serial sum over the wavefronts, one dependent LDS read after another,
// made the 1024-thread batch statistics 13.5 us long.)
template <int NS, int NT>
struct BlockShared {
  double s[NT / 64][NS];
  double mx[NT / 64];
};
template <int NS, int NT>
__device__ __forceinline__ void block_stats(double (&v)[NS], double& mx, BlockShared<NS, NT>& sh) {
  constexpr int NW = NT / 64;
  static_assert(NW == 1 || NW == 4 || NW == 16, "1, 4 or 16 wavefronts");
#pragma unroll
  for (int k = 0; k < NS; ++k) v[k] = lane_sum<64>(v[k]);
  mx = lane_max<64>(mx);
  if constexpr (NW > 1) {
    const int w = threadIdx.x >> 6, q = threadIdx.x & (NW - 1);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < NS; ++k) sh.s[w][k] = v[k];
      sh.mx[w] = mx;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NS; ++k) v[k] = lane_sum<NW>(sh.s[q][k]);
    mx = lane_max<NW>(sh.mx[q]);
  }
}

// Count, mean and sum of squared deviations of a set of values; two sets
// combine exactly in real arithmetic (the pairwise update of Chan, Golub and
// LeVeque), so the squared deviations need no second pass over the slots.
struct Var {
  double n, mu, m2;
};
__device__ __forceinline__ Var var_merge(const Var& a, const Var& b) {
  if (b.n == 0.0) return a;
  if (a.n == 0.0) return b;
  const double n = a.n + b.n, d = b.mu - a.mu, f = b.n / n;
  return Var{n, a.mu + d * f, a.m2 + b.m2 + d * d * a.n * f};
}

// A thread's (n, mu, m2) as its share of the sum of squared deviations about
// the mean of all threads' values: m2 + n (mu - mean)^2.  The shares add up to
// the whole set's, so the threads combine by sums, without the pairwise
// update's division at each level of a tree.
__device__ __forceinline__ double var_about(const Var& v, double mean) {
  const double d = v.mu - mean;
  return v.n > 0.0 ? fma(v.n * d, d, v.m2) : 0.0;
}

__device__ __forceinline__ double token_distance(float lp_pi, float lp_mu) {
  return fabs(exp((double)lp_pi) - exp((double)lp_mu));
}

// Workgroup size of the per-response kernels and the slots of a thread: four
// per turn, consecutive (VEC: 16-byte loads, responses whose slots start
// 16-byte aligned) or NT apart.  64 threads take a response of up to 256
// slots in one turn, 256 or 1024 longer ones.  The size decides the order of a
// response's fp64 sums; the reduce's are outputs, so it goes by L alone there
// and a chunk of a batch has the sums of the batch.  1024 threads from L = 8193
// on, GPU time of the call in us, 256 against 1024 threads: 64 responses of
// 4096 slots 11.1 / 11.0, of 16384 25.2 / 20.5; 1024 responses, where 256
// threads fill the chip, of 4096 30.1 / 41.7, of 16384 83.9 / 90.3.
constexpr int kSlots = 4;
inline int reduce_threads(int64_t L) { return L <= 64 * kSlots ? 64 : L > 8192 ? 1024 : kRedThreads; }
// The surrogate's sums enter its one loss only: 1024 threads from the second
// turn on while that leaves no more than one workgroup per CU (64 responses of
// 4096 slots 9.7 us against 10.6, 256 of 16384 31.5 / 39.8, 1024 of 4096 38.3 /
// 35.0).
inline int surr_threads(int64_t B, int64_t L) {
  if (L <= 64 * kSlots) return 64;
  return L > kRedThreads * kSlots && B <= 256 ? 1024 : kRedThreads;
}
template <int NT, bool VEC>
__device__ __forceinline__ int64_t first_slot() {
  return VEC ? (int64_t)threadIdx.x * kSlots : (int64_t)threadIdx.x;
}
// The mask of the thread's slots from slot j on of the response at `base`
// (slots past L: 0) and four values of x there, 0 past L.
template <int NT, bool VEC>
__device__ __forceinline__ void load_mask(const uint8_t* __restrict__ mask, int64_t base, int64_t j, int64_t L,
                                          uint8_t (&m)[kSlots]) {
  if constexpr (VEC) {
    const uchar4 t = *reinterpret_cast<const uchar4*>(mask + base + j);
    m[0] = t.x; m[1] = t.y; m[2] = t.z; m[3] = t.w;
  } else {
#pragma unroll
    for (int k = 0; k < kSlots; ++k) m[k] = j + k * NT < L ? mask[base + j + k * NT] : (uint8_t)0;
  }
}
template <int NT, bool VEC>
__device__ __forceinline__ void load_slots(const float* __restrict__ x, int64_t base, int64_t j, int64_t L,
                                           float (&v)[kSlots]) {
  if constexpr (VEC) {
    const float4 t = *reinterpret_cast<const float4*>(x + base + j);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
#pragma unroll
    for (int k = 0; k < kSlots; ++k) v[k] = j + k * NT < L ? x[base + j + k * NT] : 0.0f;
  }
}

// One workgroup per response.  Every slot is loaded (masked ones too: no load
// waits on the mask).  The sums are plain fp64 sums in slot order; the squared
// deviations of each turn's four slots (about their own mean) merge into the
// thread's running Var.  Latency bound (turns of exponentials and divisions):
// 4 responses of 64 slots 5.6 us with 256 threads, 3.4 with 64.
template <int NT, bool VEC>
__global__ __launch_bounds__(NT) void reduce_seq_kernel(acrl_reduce_desc p, SeqRec* rec, uint32_t* unsorted) {
  __shared__ BlockShared<5, NT> sh;
  __shared__ BlockShared<1, NT> sh2;
  const int64_t i = blockIdx.x;
  const int64_t base = i * p.L;
  double v[5] = {0, 0, 0, 0, 0};  // n, sum d, sum log-ratio, sum H_pi, sum H_mu
  double mx = 0;
  Var var{0.0, 0.0, 0.0};
  for (int64_t j = first_slot<NT, VEC>(); j < p.L; j += NT * kSlots) {
    uint8_t m[kSlots];
    float a[kSlots], b[kSlots], hp[kSlots] = {}, hm[kSlots] = {};
    load_mask<NT, VEC>(p.mask, base, j, p.L, m);
    load_slots<NT, VEC>(p.logp_pi, base, j, p.L, a);
    load_slots<NT, VEC>(p.logp_mu, base, j, p.L, b);
    if (p.entropy_pi) load_slots<NT, VEC>(p.entropy_pi, base, j, p.L, hp);
    if (p.entropy_mu) load_slots<NT, VEC>(p.entropy_mu, base, j, p.L, hm);
    double dv[kSlots];
    float dt[kSlots];
    double pn = 0.0, ps = 0.0;
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      dt[k] = 0.0f;
      dv[k] = 0.0;
      if (m[k]) {
        dv[k] = token_distance(a[k], b[k]);
        v[0] += 1.0;
        v[1] += dv[k];
        v[2] += (double)a[k] - (double)b[k];
        v[3] += hp[k];
        v[4] += hm[k];
        mx = fmax(mx, dv[k]);
        dt[k] = (float)dv[k];
        pn += 1.0;
        ps += dv[k];
      }
    }
    if (pn > 0.0) {
      const double pm = ps / pn;
      double pm2 = 0.0;
#pragma unroll
      for (int k = 0; k < kSlots; ++k)
        if (m[k]) pm2 += (dv[k] - pm) * (dv[k] - pm);
      var = var_merge(var, Var{pn, pm, pm2});
    }
    if (p.d_tok) {
      if constexpr (VEC) {
        *reinterpret_cast<float4*>(p.d_tok + base + j) = make_float4(dt[0], dt[1], dt[2], dt[3]);
      } else {
#pragma unroll
        for (int k = 0; k < kSlots; ++k)
          if (j + k * NT < p.L) p.d_tok[base + j + k * NT] = dt[k];
      }
    }
  }
  block_stats<5, NT>(v, mx, sh);
  const double mean = v[0] > 0 ? v[1] / v[0] : 0.0;
  double m2[1] = {var_about(var, mean)}, unused = 0.0;
  block_stats<1, NT>(m2, unused, sh2);
  if (threadIdx.x == 0) {
    SeqRec r;
    r.n = v[0]; r.sum_d = v[1]; r.sum_lr = v[2]; r.sum_hp = v[3]; r.sum_hm = v[4]; r.max_d = mx; r.m2 = m2[0];
    r.pad = 0;
    rec[i] = r;
    if (p.seq_len) p.seq_len[i] = (int32_t)v[0];
    if (p.seq_sum_d) p.seq_sum_d[i] = v[1];
    if (p.seq_sum_logratio) p.seq_sum_logratio[i] = v[2];
    p.seq_mean_d[i] = (float)mean;
    // (no flag: one workgroup does all groups, in whatever order they come)
    if (unsorted && i + 1 < p.B && p.group_of_seq[i] > p.group_of_seq[i + 1]) atomicOr(unsorted, 1u);
  }
}

__global__ void clear_flag_kernel(uint32_t* f) { *f = 0u; }

// Per-group partial record (the groups partition the responses, so the
// batch statistics come from these).
struct GroupRec {
  double n, sum_d, sum_lr, sum_hp, sum_hm, max_d, nseq, mu, m2, y;
};
static_assert(sizeof(GroupRec) <= 128, "the workspace reserves 128 bytes");

// Sums over the responses of one group that a thread takes.
struct GroupSums {
  double v[7] = {0, 0, 0, 0, 0, 0, 0};  // sum of means, responses, n, sum d, sum log-ratio, sum H_pi, sum H_mu
  double mx = 0.0;
  Var var{0.0, 0.0, 0.0};
  __device__ __forceinline__ void add(const SeqRec& r) {
    if (r.n > 0) {
      const double mean = r.sum_d / r.n;
      v[0] += mean;
      v[1] += 1.0;
      v[2] += r.n;
      v[3] += r.sum_d;
      v[4] += r.sum_lr;
      v[5] += r.sum_hp;
      v[6] += r.sum_hm;
      mx = fmax(mx, r.max_d);
      var = var_merge(var, Var{r.n, mean, r.m2});
    }
  }
  __device__ __forceinline__ double mean_d() const { return v[2] > 0 ? v[3] / v[2] : 0.0; }
};

// Group g's outputs and record from its sums (mu, m2: its tokens' mean d and
// squared deviations).
__device__ __forceinline__ GroupRec store_group(const acrl_reduce_desc& p, int g, const GroupSums& t, double mu,
                                                double m2) {
  const double c = t.v[1];
  const double y = c > 0 ? t.v[0] / c : 0.0;
  p.group_y[g] = (float)y;
  if (p.group_nseq) p.group_nseq[g] = (int32_t)c;
  GroupRec r;
  r.n = t.v[2]; r.sum_d = t.v[3]; r.sum_lr = t.v[4]; r.sum_hp = t.v[5]; r.sum_hm = t.v[6]; r.max_d = t.mx; r.nseq = c;
  r.mu = mu; r.m2 = m2; r.y = y;
  return r;
}

// One workgroup per group: Y_g over the group's non-empty responses, and the
// group's share of the batch statistics.  When group_of_seq is non-decreasing
// (flag unsorted == 0, set by the per-response kernel) the group's responses are
// the range found by binary search; otherwise every response is scanned.
__global__ __launch_bounds__(kRedThreads) void reduce_group_kernel(acrl_reduce_desc p, const SeqRec* rec,
                                                                   const uint32_t* unsorted, GroupRec* grec) {
  __shared__ BlockShared<7, kRedThreads> sh;
  __shared__ BlockShared<1, kRedThreads> sh2;
  __shared__ int64_t range[2];
  const int g = blockIdx.x;
  const bool sorted = *unsorted == 0u;
  int64_t lo = 0, hi = p.B;
  if (sorted) {
    if (threadIdx.x == 0) {
      int64_t a = 0, b = p.B;
      while (a < b) {  // first response with group >= g
        const int64_t m = (a + b) >> 1;
        if (p.group_of_seq[m] < g) a = m + 1;
        else b = m;
      }
      range[0] = a;
      b = p.B;
      while (a < b) {  // first response with group > g
        const int64_t m = (a + b) >> 1;
        if (p.group_of_seq[m] <= g) a = m + 1;
        else b = m;
      }
      range[1] = a;
    }
    __syncthreads();
    lo = range[0];
    hi = range[1];
  }
  GroupSums t;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kRedThreads)
    if (sorted || p.group_of_seq[i] == g) t.add(rec[i]);
  block_stats<7, kRedThreads>(t.v, t.mx, sh);
  const double mu = t.mean_d();
  double m2[1] = {var_about(t.var, mu)}, unused = 0.0;
  block_stats<1, kRedThreads>(m2, unused, sh2);
  if (threadIdx.x == 0) grec[g] = store_group(p, g, t, mu, m2[0]);
}

// Batch statistics from the group records of the workgroup's threads.
struct BatchSums {
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // n, sum d, sum log-ratio, sum H_pi, sum H_mu, responses, sum Y_g, groups
  double mx = 0.0;
  Var var{0.0, 0.0, 0.0};
  __device__ __forceinline__ void add(const GroupRec& r) {
    v[0] += r.n;
    v[1] += r.sum_d;
    v[2] += r.sum_lr;
    v[3] += r.sum_hp;
    v[4] += r.sum_hm;
    v[5] += r.nseq;
    if (r.nseq > 0) {
      v[6] += r.y;
      v[7] += 1.0;
    }
    mx = fmax(mx, r.max_d);
    var = var_merge(var, Var{r.n, r.mu, r.m2});
  }
};
template <int NT>
__device__ __forceinline__ void batch_stats(const acrl_reduce_desc& p, BatchSums& t, BlockShared<8, NT>& sh,
                                            BlockShared<1, NT>& sh2) {
  block_stats<8, NT>(t.v, t.mx, sh);
  const double n = t.v[0], ng = t.v[7], mean = n > 0 ? t.v[1] / n : 0.0;
  double m2[1] = {var_about(t.var, mean)}, unused = 0.0;
  block_stats<1, NT>(m2, unused, sh2);
  if (threadIdx.x == 0) {
    double* st = p.stats;
    st[ACRL_STAT_Y_BATCH] = ng > 0 ? t.v[6] / ng : 0.0;
    st[ACRL_STAT_TOK_MEAN_D] = mean;
    st[ACRL_STAT_TOK_MAX_D] = t.mx;
    st[ACRL_STAT_TOK_STD_D] = n > 0 ? sqrt(m2[0] / n) : 0.0;
    st[ACRL_STAT_MEAN_H_PI] = n > 0 ? t.v[3] / n : 0.0;
    st[ACRL_STAT_MEAN_H_MU] = n > 0 ? t.v[4] / n : 0.0;
    st[ACRL_STAT_N_TOKENS] = n;
    st[ACRL_STAT_N_GROUPS] = ng;
    st[ACRL_STAT_TOK_MEAN_LOGRATIO] = n > 0 ? t.v[2] / n : 0.0;
    st[ACRL_STAT_N_SEQS] = t.v[5];
  }
}
constexpr int kBatchThreads = 1024;
__global__ __launch_bounds__(kBatchThreads) void reduce_batch_kernel(acrl_reduce_desc p, const GroupRec* grec) {
  __shared__ BlockShared<8, kBatchThreads> sh;
  __shared__ BlockShared<1, kBatchThreads> sh2;
  BatchSums t;
  for (int64_t g = threadIdx.x; g < p.n_groups; g += kBatchThreads) t.add(grec[g]);
  batch_stats<kBatchThreads>(p, t, sh, sh2);
}

// The groups and the batch in one workgroup, for up to kOneSeqs responses in
// up to kOneGroups groups: a wavefront takes a group at a time, its range where
// group_of_seq is non-decreasing, else what it finds in the responses' groups
// in LDS; the first wavefront then takes one group per lane.  Above, a
// workgroup per group searches for its range instead.  Where group_of_seq is
// non-decreasing lane k of either takes the group's k-th response, so a group
// of up to 64 has the same sums wherever it stands and whatever else is in the
// batch.  GPU time of the whole call, this against a workgroup per group, us:
// 64 responses in 8 groups 8.0 / 15.0, 1024 in 32 11.5 / 15.9, 1024 in 64 16.8 /
// 16.0 (the surrogate's 8.0 / 9.6, 9.8 / 10.9, 11.8 / 11.0); with 64 groups the
// launches less still save the host 4 us of 26 (of 21).
constexpr int kOneSeqs = 1024, kOneGroups = 64;
inline bool one_workgroup(int64_t B, int64_t n_groups) { return B <= kOneSeqs && n_groups <= kOneGroups; }
// Bit k: response lane + 64 k is in group g (-1 past the last response).
__device__ __forceinline__ uint32_t members(const int32_t* group_of, int g, int lane) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < kOneSeqs / 64; ++k) m |= (uint32_t)(group_of[lane + 64 * k] == g) << k;
  return m;
}
__global__ __launch_bounds__(1024) void reduce_groups_batch_kernel(acrl_reduce_desc p, const SeqRec* rec) {
  __shared__ int32_t group_of[kOneSeqs];
  __shared__ int lo[kOneGroups], hi[kOneGroups], disorder[16];
  __shared__ GroupRec grec[kOneGroups];
  __shared__ BlockShared<8, 64> sh;
  __shared__ BlockShared<1, 64> sh2;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // the groups' ranges lo .. hi - 1 where they are in order, noted by the
  // responses at their ends (those of a group without responses stay unwritten)
  const int i = threadIdx.x, ng = (int)p.n_groups, n = (int)p.B;
  const int mine = i < n ? p.group_of_seq[i] : -1;
  const int before = i > 0 && i < n ? p.group_of_seq[i - 1] : -1;
  const int after = i + 1 < n ? p.group_of_seq[i + 1] : -1;
  group_of[i] = mine;
  if (mine >= 0 && mine < ng) {
    if (mine != before) lo[mine] = i;
    if (mine != after) hi[mine] = i + 1;
  }
  const bool wrong = __any(i > 0 && i < n && mine < before);
  if (lane == 0) disorder[w] = wrong;
  __syncthreads();
  const bool sorted = !__any(disorder[lane & 15] != 0);
  for (int g = w; g < p.n_groups; g += 16) {
    GroupSums t;
    if (sorted) {
      const int first = lo[g] & (kOneSeqs - 1);  // (any value if the group has no response)
      const int last = group_of[first] == g ? hi[g] : 0;
      for (int k = first + lane; k < last; k += 64) t.add(rec[k]);
    } else {
      for (uint32_t m = members(group_of, g, lane); m; m &= m - 1) t.add(rec[lane + 64 * (__ffs(m) - 1)]);
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) t.v[k] = lane_sum<64>(t.v[k]);
    t.mx = lane_max<64>(t.mx);
    const double m2 = lane_sum<64>(var_about(t.var, first_lane(t.mean_d())));
    if (lane == 0) grec[g] = store_group(p, g, t, t.mean_d(), m2);
  }
  __syncthreads();
  if (w != 0) return;
  BatchSums t;
  if (lane < p.n_groups) t.add(grec[lane]);
  batch_stats<64>(p, t, sh, sh2);
}

// Element-wise controller.  alpha and the weight are evaluated in fp64 from
// the fp32 inputs (exact conversions), then rounded to fp32 once.  Modes:
// Eq. ACRL, token-level TIS (Eq. tis_objective), sequence-level MIS (Eq.
// mis_objective, from the fp64 per-sequence log-ratio sums of the reduce),
// and the continuous-reduction / fallback-to-GRPO ablations of Sec. 5.
// min(x, C) of an undefined x is undefined: a NaN log-ratio (an invalid
// token id) or a NaN Y (a group id outside [0, n_groups)) gives weight NaN,
// not the clip C.
__global__ __launch_bounds__(256) void controller_kernel(acrl_controller_desc p) {
  const int64_t n = p.B * p.L;
  const double X = p.X, gamma = p.gamma, lnC = log((double)p.C), C = p.C;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x) {
    float a_out = 0.0f, w_out = 0.0f;
    if (p.mask[t]) {
      const int64_t i = t / p.L;
      const double A = p.adv_per_token ? p.adv[t] : p.adv[i];
      const double sg = (A > 0) - (A < 0);
      const double lr = (double)p.logp_pi[t] - (double)p.logp_mu[t];  // ln(pi/mu)
      if (p.mode == ACRL_CTRL_MIS) {
        const double s = p.seq_sum_logratio[i];  // ln rho_i
        a_out = 1.0f;
        w_out = isnan(s) ? __builtin_nanf("") : (s <= lnC ? (float)exp(s) : 0.0f);
      } else if (p.mode == ACRL_CTRL_TIS) {
        a_out = 1.0f;
        w_out = isnan(lr) ? __builtin_nanf("") : (float)(lr < lnC ? exp(lr) : C);
      } else {
        double alpha;
        bool grpo = false;
        if (p.mode == ACRL_CTRL_CONTINUOUS) {
          alpha = -(double)p.k * sg;
        } else {
          double Y;
          if (p.y_level == ACRL_Y_SEQUENCE) Y = p.seq_mean_d[i];
          else if (p.y_level == ACRL_Y_GROUP) {
            const int32_t g = p.group_of_seq[i];
            Y = (g >= 0 && g < p.n_groups) ? (double)p.group_y[g] : __builtin_nan("");
          }
          else Y = p.stats[ACRL_STAT_Y_BATCH];
          grpo = p.mode == ACRL_CTRL_FALLBACK && Y < X;
          alpha = gamma * sg * (1.0 - Y / X);
        }
        if (grpo) {
          a_out = 0.0f;
          w_out = 1.0f;
        } else {
          const double e = alpha * lr;  // ln rho (NaN if alpha or lr is)
          a_out = (float)alpha;
          w_out = isnan(e) ? __builtin_nanf("") : (float)(e < lnC ? exp(e) : C);
        }
      }
    }
    if (p.alpha) p.alpha[t] = a_out;
    p.weight[t] = w_out;
  }
}

// ------------------------------------------------------------------ surrogate
// The ACRL-weighted clipped surrogate (Eq. ACRL on top of the GRPO objective
// of Sec. 2): J = mean over prompts of (1/G) sum_i (1/|a_i|) sum_t
// w_t min(r_t A_t, clip(r_t) A_t), r_t = exp(logp_new - logp_old); the
// prompts averaged are those with a non-empty response and G counts a
// prompt's non-empty responses.  loss = -J, coef_t = d loss / d logp_new_t.

struct SurrSeq {
  double n, J;  // |a_i| and sum_t w_t min(r A, clip(r) A)
};

// min(r A, clip(r) A), r and whether the unclipped term is the minimum (a tie
// counts as unclipped), in fp64 from the fp32 inputs.
__device__ __forceinline__ void surr_terms(const acrl_surrogate_desc& p, double logp_new, double logp_old, double A,
                                           double& r, double& m, bool& unclipped) {
  r = exp(logp_new - logp_old);
  const double rc = fmin(fmax(r, 1.0 - (double)p.eps_low), 1.0 + (double)p.eps_high);
  const double u = r * A, c = rc * A;
  unclipped = u <= c;
  m = unclipped ? u : c;
}

// One workgroup per response (slots as in reduce_seq_kernel: all loaded, no
// load waits on the mask up to 256 responses; 64 responses of 4096 slots 4.6 us, 10.8 one slot at
// a time behind its mask with 256 threads).
template <int NT, bool VEC>
__global__ __launch_bounds__(NT) void surr_seq_kernel(acrl_surrogate_desc p, SurrSeq* rec) {
  __shared__ BlockShared<2, NT> sh;
  const int64_t i = blockIdx.x;
  const int64_t base = i * p.L;
  double v[2] = {0, 0}, unused = 0.0;  // n, J
  for (int64_t j = first_slot<NT, VEC>(); j < p.L; j += NT * kSlots) {
    uint8_t m[kSlots];
    float ln[kSlots], lo[kSlots], w[kSlots] = {1.0f, 1.0f, 1.0f, 1.0f}, A[kSlots];
    load_mask<NT, VEC>(p.mask, base, j, p.L, m);
    // many workgroups a CU hide the wait, and what lies past a response's end is
    // not read
    if (p.B > 256 && !(m[0] | m[1] | m[2] | m[3])) continue;
    load_slots<NT, VEC>(p.logp_new, base, j, p.L, ln);
    load_slots<NT, VEC>(p.logp_old, base, j, p.L, lo);
    if (p.weight) load_slots<NT, VEC>(p.weight, base, j, p.L, w);
    if (p.adv_per_token) {
      load_slots<NT, VEC>(p.adv, base, j, p.L, A);
    } else {
#pragma unroll
      for (int k = 0; k < kSlots; ++k) A[k] = p.adv[i];
    }
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      if (!m[k]) continue;
      double r, mn;
      bool unc;
      surr_terms(p, ln[k], lo[k], A[k], r, mn, unc);
      v[0] += 1.0;
      v[1] += (double)w[k] * mn;
    }
  }
  block_stats<2, NT>(v, unused, sh);
  if (threadIdx.x == 0) rec[i] = SurrSeq{v[0], v[1]};
}

// One workgroup per group: G_g and the group's sum of per-response means.
__global__ __launch_bounds__(kRedThreads) void surr_group_kernel(acrl_surrogate_desc p, const SurrSeq* rec,
                                                                 double* gG, double* gJ) {
  __shared__ BlockShared<2, kRedThreads> sh;
  const int g = blockIdx.x;
  double v[2] = {0, 0}, unused = 0.0;  // G, J
  for (int64_t i = threadIdx.x; i < p.B; i += kRedThreads)
    if (p.group_of_seq[i] == g && rec[i].n > 0) {
      v[0] += 1.0;
      v[1] += rec[i].J / rec[i].n;
    }
  block_stats<2, kRedThreads>(v, unused, sh);
  if (threadIdx.x == 0) {
    gG[g] = v[0];
    gJ[g] = v[1];
  }
}

// The number of prompts and the loss from a thread's v = {prompts, J}.
template <int NT>
__device__ __forceinline__ void surr_loss(const acrl_surrogate_desc& p, double (&v)[2], BlockShared<2, NT>& sh,
                                          double* prompts) {
  double unused = 0.0;
  block_stats<2, NT>(v, unused, sh);
  if (threadIdx.x == 0) {
    prompts[0] = v[0];
    p.loss[0] = v[0] > 0 ? -v[1] / v[0] : 0.0;
  }
}
__global__ __launch_bounds__(kRedThreads) void surr_batch_kernel(acrl_surrogate_desc p, const double* gG,
                                                                 const double* gJ, double* prompts) {
  __shared__ BlockShared<2, kRedThreads> sh;
  double v[2] = {0, 0};
  for (int64_t g = threadIdx.x; g < p.n_groups; g += kRedThreads)
    if (gG[g] > 0) {
      v[0] += 1.0;
      v[1] += gJ[g] / gG[g];
    }
  surr_loss<kRedThreads>(p, v, sh, prompts);
}

// Both in one workgroup (see reduce_groups_batch_kernel): 64 responses 2.3 us
// (two launches of 2.2 each otherwise), 1024 in 64 groups 5.9 (3.8 + 2.6).
__global__ __launch_bounds__(1024) void surr_groups_batch_kernel(acrl_surrogate_desc p, const SurrSeq* rec,
                                                                 double* gG, double* prompts) {
  __shared__ int32_t group_of[kOneSeqs];
  __shared__ double G[kOneGroups], J[kOneGroups];
  __shared__ BlockShared<2, 64> sh;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  group_of[threadIdx.x] = threadIdx.x < p.B ? p.group_of_seq[threadIdx.x] : -1;
  __syncthreads();
  for (int g = w; g < p.n_groups; g += 16) {
    double n = 0, sum = 0;
    for (uint32_t m = members(group_of, g, lane); m; m &= m - 1) {
      const SurrSeq r = rec[lane + 64 * (__ffs(m) - 1)];
      if (r.n > 0) {
        n += 1.0;
        sum += r.J / r.n;
      }
    }
    n = lane_sum<64>(n);
    sum = lane_sum<64>(sum);
    if (lane == 0) {
      G[g] = n;
      J[g] = sum;
      gG[g] = n;
    }
  }
  __syncthreads();
  if (w != 0) return;
  double v[2] = {0, 0};
  if (lane < p.n_groups && G[lane] > 0) {
    v[0] = 1.0;
    v[1] = J[lane] / G[lane];
  }
  surr_loss<64>(p, v, sh, prompts);
}

// Element-wise: coef_t = -w_t r_t A_t / (prompts G_g |a_i|) where the
// unclipped term is the minimum, else 0 (the clipped term does not depend on
// logp_new); masked slots 0; a group id outside [0, n_groups) gives NaN.
__global__ __launch_bounds__(256) void surr_coef_kernel(acrl_surrogate_desc p, const SurrSeq* rec, const double* gG,
                                                        const double* prompts) {
  const int64_t n = p.B * p.L;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
    float out = 0.0f;
    if (p.mask[t]) {
      const int64_t i = t / p.L;
      const int32_t g = p.group_of_seq[i];
      if (g < 0 || g >= p.n_groups) {
        out = __builtin_nanf("");
      } else {
        const double A = p.adv_per_token ? p.adv[t] : p.adv[i];
        double r, m;
        bool unc;
        surr_terms(p, p.logp_new[t], p.logp_old[t], A, r, m, unc);
        if (unc) {
          const double c = 1.0 / (prompts[0] * gG[g] * rec[i].n);
          out = (float)(-c * (p.weight ? (double)p.weight[t] : 1.0) * r * A);
        }
      }
    }
    p.coef[t] = out;
  }
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline bool aligned(const void* q, uintptr_t a) { return ((uintptr_t)q & (a - 1)) == 0; }

// launch(workgroup size, 16-byte slots) of a per-response kernel of nt threads.
template <typename F>
inline void launch_seq(int nt, bool vec, F&& launch) {
  auto with = [&](auto n) {
    if (vec) launch(n, std::true_type{});
    else launch(n, std::false_type{});
  };
  switch (nt) {
    case 64: return with(std::integral_constant<int, 64>{});
    case 1024: return with(std::integral_constant<int, 1024>{});
    default: return with(std::integral_constant<int, kRedThreads>{});
  }
}

}  // namespace

size_t surrogate_workspace_bytes(int64_t B, int64_t n_groups) {
  return align_up((size_t)B * sizeof(SurrSeq), 256) + 2 * align_up((size_t)n_groups * sizeof(double), 256) + 256;
}

hipError_t launch_surrogate(const acrl_surrogate_desc& p, hipStream_t s) {
  uint8_t* ws = static_cast<uint8_t*>(p.workspace);
  SurrSeq* rec = reinterpret_cast<SurrSeq*>(ws);
  size_t off = align_up((size_t)p.B * sizeof(SurrSeq), 256);
  double* gG = reinterpret_cast<double*>(ws + off);
  off += align_up((size_t)p.n_groups * sizeof(double), 256);
  double* gJ = reinterpret_cast<double*>(ws + off);
  off += align_up((size_t)p.n_groups * sizeof(double), 256);
  double* prompts = reinterpret_cast<double*>(ws + off);
  if (p.B > 0) {
    const bool vec = p.L % kSlots == 0 && aligned(p.logp_new, 16) && aligned(p.logp_old, 16) && aligned(p.mask, 4) &&
                     aligned(p.weight, 16) && (!p.adv_per_token || aligned(p.adv, 16));
    launch_seq(surr_threads(p.B, p.L), vec, [&](auto nt, auto v) {
      constexpr int NT = decltype(nt)::value;
      hipLaunchKernelGGL((surr_seq_kernel<NT, decltype(v)::value>), dim3((unsigned)p.B), dim3(NT), 0, s, p, rec);
    });
  }
  if (one_workgroup(p.B, p.n_groups)) {
    hipLaunchKernelGGL(surr_groups_batch_kernel, dim3(1), dim3(1024), 0, s, p, (const SurrSeq*)rec, gG, prompts);
  } else {
    if (p.n_groups > 0)
      hipLaunchKernelGGL(surr_group_kernel, dim3((unsigned)p.n_groups), dim3(kRedThreads), 0, s, p,
                         (const SurrSeq*)rec, gG, gJ);
    hipLaunchKernelGGL(surr_batch_kernel, dim3(1), dim3(kRedThreads), 0, s, p, (const double*)gG, (const double*)gJ,
                       prompts);
  }
  const int64_t n = p.B * p.L;
  if (n > 0) {
    int64_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(surr_coef_kernel, dim3((unsigned)g), dim3(256), 0, s, p, (const SurrSeq*)rec,
                       (const double*)gG, (const double*)prompts);
  }
  return hipGetLastError();
}

size_t reduce_workspace_bytes(int64_t B, int64_t L, int64_t n_groups) {
  (void)L;
  // 144 bytes per group: the bound that the header states for the fixed scratch
  return align_up((size_t)B * sizeof(SeqRec), 256) + 2 * align_up((size_t)n_groups * sizeof(double), 256) +
         align_up((size_t)n_groups * 128, 256) + 256;
}

hipError_t launch_reduce(const acrl_reduce_desc& p, hipStream_t s) {
  uint8_t* ws = static_cast<uint8_t*>(p.workspace);
  SeqRec* rec = reinterpret_cast<SeqRec*>(ws);
  size_t off = align_up((size_t)p.B * sizeof(SeqRec), 256);
  GroupRec* grec = reinterpret_cast<GroupRec*>(ws + off);
  off += align_up((size_t)p.n_groups * sizeof(GroupRec), 256);
  uint32_t* unsorted = reinterpret_cast<uint32_t*>(ws + off);
  const bool one = one_workgroup(p.B, p.n_groups);
  if (!one) hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, s, unsorted);
  if (p.B > 0) {
    // 16-byte slot loads when every row of slots starts 16-byte aligned
    const bool vec = p.L % kSlots == 0 && aligned(p.logp_pi, 16) && aligned(p.logp_mu, 16) && aligned(p.mask, 4) &&
                     aligned(p.entropy_pi, 16) && aligned(p.entropy_mu, 16) && aligned(p.d_tok, 16);
    launch_seq(reduce_threads(p.L), vec, [&](auto nt, auto v) {
      constexpr int NT = decltype(nt)::value;
      hipLaunchKernelGGL((reduce_seq_kernel<NT, decltype(v)::value>), dim3((unsigned)p.B), dim3(NT), 0, s, p, rec,
                         one ? nullptr : unsorted);
    });
  }
  if (one) {
    hipLaunchKernelGGL(reduce_groups_batch_kernel, dim3(1), dim3(1024), 0, s, p, (const SeqRec*)rec);
  } else {
    if (p.n_groups > 0)
      hipLaunchKernelGGL(reduce_group_kernel, dim3((unsigned)p.n_groups), dim3(kRedThreads), 0, s, p,
                         (const SeqRec*)rec, (const uint32_t*)unsorted, grec);
    hipLaunchKernelGGL(reduce_batch_kernel, dim3(1), dim3(kBatchThreads), 0, s, p, (const GroupRec*)grec);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ fixed scratch
// Device memory for acrl_discrepancy_reduce_noalloc: the reduce's per-response
// and per-group records live here instead of in a caller workspace.  Each
// device holds its own copy for the life of the process; host code reaches
// it only through the address hipGetSymbolAddress returns for that device
// (the array's name is a host-side stand-in, not a device address).
static __device__ __align__(256) uint8_t scratch[kReduceScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices];  // device address of `scratch` per device, once looked up
}  // namespace

hipError_t reduce_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!a) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = a;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_controller(const acrl_controller_desc& p, hipStream_t s) {
  const int64_t n = p.B * p.L;
  if (n == 0) return hipSuccess;
  int64_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(controller_kernel, dim3((unsigned)g), dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace acrl
