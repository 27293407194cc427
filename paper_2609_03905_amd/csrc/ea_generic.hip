// ea_generic.hip -- the general einsum join-agg (Section 3.2, Definition
// "Implementation"): any spec, join MUL or ADD, aggregation NONE, SUM or MAX.
//
// One thread owns one element of one output block.  It walks its group's
// tuples in table order and, inside each tuple, every value of the contracted
// letters within the tuple blocks' intervals, applying the join to the
// inputs' elements and the aggregation to the running value in f32.  This is
// the slow, general path; two-operand products with a contracted letter take
// the matrix-core kernels, and reduce_kernel below takes the einsums of one or
// two inputs of one dtype with at most one contracted letter and four output
// letters (row and column reductions, sums of products that fill no tile,
// elementwise joins, broadcasts, transposes; not those over blocks of a few
// elements): element addresses from strides resolved when the plan is built,
// and the contracted letter shared between threads:
//   * lanes along the contracted letter where it is the input's contiguous one
//     ("ij->i") and long, or the outputs few: a wavefront, or four, per output;
//   * lanes along the output otherwise ("ij->j", "ij,ij->ij"): one, four or
//     sixteen wavefronts per 64 output elements.
// Both are bound by memory for large inputs and by latency (launch, three
// dependent loads, one pass) for small ones.  GPU time, general kernel ->
// this one (128-blocks):
//   "ij->i" max, 930 x 1668 bf16   972 -> 5.5 us   4096 x 2048 f32: 18 us
//   "ij->i" max, 162 x 85 bf16      51 -> 2.7 us
//   "ij->j" sum, 930 x 1668 f32            7.7 us   4096 x 2048 f32: 28 us
//   "ij,ij->ij", 4096 x 2048 f32            34 us (a copy of the bytes: 20 us)
#include <type_traits>

#include "ea_device.h"

namespace ea {

namespace {

__global__ __launch_bounds__(256) void generic_kernel(GenArgs a) {
  const GenDesc& g = *a.desc;
  const GenWork w = a.work[blockIdx.x];
  const DevBlk& ob = a.blk[g.n_in][w.block];
  int64_t n = 1;
  for (int d = 0; d < g.out_rank; ++d) n *= ob.ext[d];
  const int64_t e = (int64_t)w.start + threadIdx.x;
  if (e >= n) return;
  int32_t val[kMaxLetters];
  {
    int64_t rem = e;
    for (int d = g.out_rank - 1; d >= 0; --d) {
      val[g.out_letter[d]] = ob.lo[d] + (int32_t)(rem % ob.ext[d]);
      rem /= ob.ext[d];
    }
  }
  float acc = g.agg == EA_AGG_MAX ? -INFINITY : 0.0f;
  const int stride = g.n_in + 1;
  const int32_t t0 = a.goff[w.block], t1 = a.goff[w.block + 1];
  for (int32_t t = t0; t < t1; ++t) {
    const int32_t* tp = a.tuples + (int64_t)t * stride;
    int32_t clo[kMaxLetters], cext[kMaxLetters];
    int64_t ncomb = 1;
    for (int j = 0; j < g.n_contr; ++j) {
      const DevBlk& b = a.blk[g.contr_op[j]][tp[1 + g.contr_op[j]]];
      clo[j] = b.lo[g.contr_dim[j]];
      cext[j] = b.ext[g.contr_dim[j]];
      ncomb *= cext[j];
    }
    for (int64_t cc = 0; cc < ncomb; ++cc) {
      int64_t rem = cc;
      for (int j = g.n_contr - 1; j >= 0; --j) {
        val[g.contr_letter[j]] = clo[j] + (int32_t)(rem % cext[j]);
        rem /= cext[j];
      }
      float f = g.join == EA_JOIN_MUL ? 1.0f : 0.0f;
      for (int i = 0; i < g.n_in; ++i) {
        const DevBlk& b = a.blk[i][tp[1 + i]];
        int64_t idx = 0;
        for (int d = 0; d < g.in_rank[i]; ++d) idx = idx * b.ext[d] + (val[g.in_letter[i][d]] - b.lo[d]);
        const float x = ld_elem(a.in[i] + b.off, idx, g.dt_in[i]);
        f = g.join == EA_JOIN_MUL ? f * x : f + x;
      }
      if (g.agg == EA_AGG_MAX) acc = fmaxf(acc, f);
      else if (g.agg == EA_AGG_SUM) acc += f;
      else acc = f;
    }
  }
  if (g.has_res) acc += ld_elem(a.res + ob.off, e, g.dt_res);
  st_elem(a.out + ob.off, e, g.dt_out, acc);
}

// ---------------------------------------------------------------------------
// one or two inputs, at most one contracted letter
// ---------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ float ld_at(const char* base, uint32_t off) {
  if constexpr (DT == EA_F32) return *reinterpret_cast<const float*>(base + off);
  const uint16_t h = *reinterpret_cast<const uint16_t*>(base + off);
  return DT == EA_BF16 ? bf16_to_f32(h) : f16_to_f32(h);
}

// T threads; ROWS: lanes along the contracted letter, else along the output
template <int NIN, int DT, int T, bool ROWS>
__global__ __launch_bounds__(T) void reduce_kernel(const ReduceArgs a) {
  constexpr uint32_t ES = DT == EA_F32 ? 4 : 2;
  constexpr int W = T / 64;
  __shared__ float part[T];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RedWork* wp = a.work + blockIdx.x;
  const int gb = ld_uniform(&wp->gb), n = ld_uniform(&wp->n);
  const int64_t ooff = ld_uniform(&wp->ooff);
  int oext[kRedRank];
#pragma unroll
  for (int d = 0; d < kRedRank; ++d) oext[d] = ld_uniform(&wp->ext[d]);
  // R wavefronts share each output (ROWS) or each 64 outputs
  const int R = a.R, wr = wid % R, wg = wid / R;
  const int per = (W / R) * (ROWS ? 1 : 64);  // outputs of the workgroup per round
  // the key's tuples are shared out where there are enough, else the
  // contracted letter inside each
  const bool by_tuple = a.nt >= R;
  const int nt = a.nt, t_step = by_tuple ? R : 1, t0 = by_tuple ? wr : 0;
  const int c_lane = ROWS ? lane : 0, c_step = (ROWS ? 64 : 1) * (by_tuple ? 1 : R);
  const int c0 = c_lane + (by_tuple ? 0 : wr * (ROWS ? 64 : 1));
  const bool is_max = a.agg == EA_AGG_MAX, mul = a.join == EA_JOIN_MUL;
  // the identity of the aggregation (of NONE: -0, which leaves every value as it is)
  const float zero = is_max ? -INFINITY : a.agg == EA_AGG_NONE ? -0.0f : 0.0f;
  // products start from 1 and sums from 0, as on the general path (0 + -0 is 0)
  auto join2 = [&](float x, float y) {
    if constexpr (NIN == 1) return mul ? x : 0.0f + x;
    return mul ? x * y : (0.0f + x) + y;
  };
  auto add = [&](float acc, float f) { return is_max ? fmaxf(acc, f) : acc + f; };
  for (int k = 0; k < a.rounds; ++k) {
    const int e = ld_uniform(&wp->start) + k * per + (ROWS ? wg : wg * 64 + lane);
    const bool ok = e < n;
    // coordinates of the output element inside its block
    int co[kRedRank], rem = ok ? e : 0;
#pragma unroll
    for (int d = kRedRank - 1; d >= 0; --d) {
      co[d] = d > 0 ? rem % oext[d] : rem;
      if (d > 0) rem /= oext[d];
    }
    float acc = zero, acc1 = zero, acc2 = zero, acc3 = zero;
    for (int t = t0; t < nt; t += t_step) {
      const RedMeta* m = a.meta + gb + t;
      const char* base[NIN];
      uint32_t off[NIN], cs[NIN];
      const int cext = ld_uniform(&m->cext);
#pragma unroll
      for (int i = 0; i < NIN; ++i) {
        base[i] = a.in[i] + ld_uniform(&m->off[i]);
        uint32_t o = 0;
#pragma unroll
        for (int d = 0; d < kRedRank; ++d) o += (uint32_t)co[d] * (uint32_t)ld_uniform(&m->os[i][d]);
        cs[i] = (uint32_t)ld_uniform(&m->cs[i]) * ES;
        off[i] = o * ES + (uint32_t)c0 * cs[i];
      }
      auto term = [&](int u) {  // u steps ahead
        const float x = ld_at<DT>(base[0], off[0] + (uint32_t)(u * c_step) * cs[0]);
        return join2(x, NIN > 1 ? ld_at<DT>(base[NIN - 1], off[NIN - 1] + (uint32_t)(u * c_step) * cs[NIN - 1]) : 0.0f);
      };
      int c = c0;
      for (; c + 3 * c_step < cext; c += 4 * c_step) {  // four terms' loads in flight
        const float f0 = term(0), f1 = term(1), f2 = term(2), f3 = term(3);
        acc = add(acc, f0);
        acc1 = add(acc1, f1);
        acc2 = add(acc2, f2);
        acc3 = add(acc3, f3);
#pragma unroll
        for (int i = 0; i < NIN; ++i) off[i] += (uint32_t)(4 * c_step) * cs[i];
      }
      for (; c < cext; c += c_step) {
        acc = add(acc, term(0));
#pragma unroll
        for (int i = 0; i < NIN; ++i) off[i] += (uint32_t)c_step * cs[i];
      }
    }
    acc = add(add(acc, acc1), add(acc2, acc3));
    if constexpr (ROWS) acc = is_max ? wave_max(acc) : wave_sum(acc);
    if (R > 1) {  // the wavefronts' partials, in wavefront order
      if (k > 0) __syncthreads();
      part[threadIdx.x] = acc;
      __syncthreads();
      if (wr == 0)
        for (int q = 1; q < R; ++q) acc = add(acc, part[threadIdx.x + 64 * q]);
    }
    if (ok && wr == 0 && (!ROWS || lane == 0)) {
      if (a.res) acc += ld_elem(a.res + ooff, e, a.dt_out);
      st_elem(a.out + ooff, e, a.dt_out, acc);
    }
  }
}

__device__ __forceinline__ int32_t red_stride(const DevBlk& b, int rank, int d) {
  if (d < 0) return 0;
  int32_t s = 1;
  for (int x = d + 1; x < rank; ++x) s *= b.ext[x];
  return s;
}

// Plan time, after the join: one thread per tuple, then one per work item.
__global__ __launch_bounds__(256) void reduce_meta_kernel(const ReduceDims d, RedMeta* meta, const int32_t* count,
                                                          int64_t cap) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= cap || q >= *count) return;
  const int32_t* tp = d.tuples + q * (d.n_in + 1);
  RedMeta m = {};
  m.cext = 1;
  for (int i = 0; i < d.n_in; ++i) {
    const DevBlk& b = d.blk[i][tp[1 + i]];
    m.off[i] = b.off;
    for (int x = 0; x < kRedRank; ++x) m.os[i][x] = red_stride(b, d.rank[i], d.od[i][x]);
    m.cs[i] = red_stride(b, d.rank[i], d.cd[i]);
    if (d.cd[i] >= 0) m.cext = b.ext[d.cd[i]];
  }
  meta[q] = m;
}

__global__ __launch_bounds__(256) void reduce_work_kernel(const ReduceDims d, RedWork* work, int64_t n_work) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= n_work) return;
  RedWork& w = work[q];
  const DevBlk& b = d.blk[d.n_in][w.block];
  w.gb = d.goff[w.block];
  w.ooff = b.off;
  w.n = 1;
  for (int x = 0; x < kRedRank; ++x) {  // output letters right-aligned, leading extents 1
    const int dim = x - (kRedRank - d.out_rank);
    w.ext[x] = dim >= 0 ? b.ext[dim] : 1;
    w.n *= w.ext[x];
  }
}

template <int NIN, int DT>
void launch_reduce_t(const ReduceArgs& a, hipStream_t s) {
  const dim3 grid((uint32_t)a.n_work);
  if (a.rows) hipLaunchKernelGGL((reduce_kernel<NIN, DT, 256, true>), grid, dim3(256), 0, s, a);
  else if (a.threads == 1024) hipLaunchKernelGGL((reduce_kernel<NIN, DT, 1024, false>), grid, dim3(1024), 0, s, a);
  else hipLaunchKernelGGL((reduce_kernel<NIN, DT, 256, false>), grid, dim3(256), 0, s, a);
}

}  // namespace

hipError_t launch_generic(const GenArgs& a, hipStream_t s) {
  if (a.n_work == 0) return hipSuccess;
  hipLaunchKernelGGL(generic_kernel, dim3((uint32_t)a.n_work), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_reduce_prep(const ReduceDims& d, RedMeta* meta, RedWork* work, int64_t n_work, const int32_t* count,
                              int64_t tuple_cap, hipStream_t s) {
  if (tuple_cap > 0)
    hipLaunchKernelGGL(reduce_meta_kernel, dim3((uint32_t)((tuple_cap + 255) / 256)), dim3(256), 0, s, d, meta, count,
                       tuple_cap);
  if (n_work > 0)
    hipLaunchKernelGGL(reduce_work_kernel, dim3((uint32_t)((n_work + 255) / 256)), dim3(256), 0, s, d, work, n_work);
  return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs& a, hipStream_t s) {
  if (a.n_work == 0) return hipSuccess;
  switch (a.dt_in) {
    case EA_F32: a.n_in == 1 ? launch_reduce_t<1, EA_F32>(a, s) : launch_reduce_t<2, EA_F32>(a, s); break;
    case EA_BF16: a.n_in == 1 ? launch_reduce_t<1, EA_BF16>(a, s) : launch_reduce_t<2, EA_BF16>(a, s); break;
    default: a.n_in == 1 ? launch_reduce_t<1, EA_F16>(a, s) : launch_reduce_t<2, EA_F16>(a, s); break;
  }
  return hipGetLastError();
}

}  // namespace ea
