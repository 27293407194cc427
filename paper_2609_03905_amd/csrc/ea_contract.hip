// ea_contract.hip -- two-operand contractions on the fp32 matrix cores.
//
// Section 3.2, Example "Matrix multiply, decomposed": every tuple of an output
// key multiplies one block of A by one block of B and the products are summed
// (aggregation +).  These kernels take such join-aggs whose letters fall into
// one contracted letter (in both inputs), at most one row letter (A and
// output), at most one column letter (B and output), one of the two at least,
// and any batch letters (all three), whatever their order in the operands:
// "ij,jk->ik", "ij,kj->ik", "hqd,hkd->hqk", "bij,bjk->bik", "tj,j->t", ...  Left
// to others: blocks of 2 GiB and more (32-bit byte offsets), and products of
// which a tile holds few outputs, where reduction_faster in the host code
// estimates so.  f32, bf16 and f16 operands
// are widened to fp32 (exact) and multiplied by v_mfma_f32_*_f32, so products
// and sums keep fp32 precision; 16-bit products "ab,bc->ac" with 8-aligned
// blocks take the 16-bit matrix-core kernel instead.
//
// Both operands are seen alike: rows (m or n) and k, each with a stride.  An
// MFMA adds outer products over its k lanes, so any assignment of k values to
// (lane group, instruction) works as long as A and B share it: lane group h
// takes k = 4h .. 4h+3 over four consecutive MFMAs, which makes the four
// values of a lane one vector load where k is the contiguous letter.
//
// Two kernels, chosen per plan (contract_tile in the host code):
//   * contract_reg_kernel<16 or 32>: one TS x TS output tile per workgroup, the
//     K walk cut into four runs, one per wavefront, operands straight from
//     global memory into MFMA registers (no LDS, no barrier before the
//     end), 4 or 8 vector loads per operand in flight per lane; the four partial
//     tiles meet in LDS in wavefront order.  For small outputs, where latency
//     and idle CUs are the cost.
//   * contract_lds_kernel: a 64 x 64 tile, four wavefronts of 32 x 32, 32-deep
//     K steps double-buffered through LDS (one barrier per step), several
//     workgroups per CU.  It reads 1/4 of the operand bytes of a 16 x 16 tile
//     per FLOP (1/2 of a 32 x 32 one) and is bound by the fp32 MFMA rate.
//
// Measured against the kernels that took these calls before (a vector-ALU tile
// kernel for f32 "ab,bc->ac", one thread per element for the rest), GPU time:
//   f32 256^3 in 64-blocks               16.9 ->   3.7 us (latency: launch, three
//                                                dependent loads, 512 MFMA clocks)
//   f32 1536 x 2048 x 1160, 512-blocks    271 ->    84 us (87 TFLOP/s; 456 tiles
//                                                on 256 CUs, two rounds)
//   f32 2048^3                                     150 us (114 of 152 TFLOP/s)
//   bf16 scores of 8 heads, 256 x 128     423 ->   7.5 us
#include "ea_device.h"

namespace ea {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kWaves = kConWaves;
constexpr int kThreads = 64 * kWaves;

// Four consecutive-k values of one row, as stored: 16 bytes of f32 or 8 of a
// 16-bit type.
template <int DT>
struct Quad {
  uint32_t w[DT == EA_F32 ? 4 : 2];
  __device__ __forceinline__ float get(int i) const {
    if constexpr (DT == EA_F32) return __uint_as_float(w[i]);
    const uint16_t h = (uint16_t)(i & 1 ? w[i >> 1] >> 16 : w[i >> 1] & 0xffffu);
    return DT == EA_BF16 ? bf16_to_f32(h) : f16_to_f32(h);
  }
};

// Addresses are a wavefront-uniform block base plus a 32-bit byte offset (every
// operand block is below 2 GiB, a host guarantee): one add per load, where a
// 64-bit lane address takes several.  VEC: the four values are contiguous and
// aligned, n is 0 or 4.  Else four element loads `stride` bytes apart; values
// past n load the first one's address instead (always in bounds) and are
// zeroed by the caller's mask.
template <int DT, bool VEC>
__device__ __forceinline__ Quad<DT> load_quad(const char* base, uint32_t off, uint32_t stride, int n) {
  Quad<DT> q;
  if constexpr (VEC) {
    if constexpr (DT == EA_F32) {
      const uint4 v = *reinterpret_cast<const uint4*>(base + off);
      q.w[0] = v.x; q.w[1] = v.y; q.w[2] = v.z; q.w[3] = v.w;
    } else {
      const uint2 v = *reinterpret_cast<const uint2*>(base + off);
      q.w[0] = v.x; q.w[1] = v.y;
    }
  } else if constexpr (DT == EA_F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) q.w[i] = *reinterpret_cast<const uint32_t*>(base + (off + (i < n ? i * stride : 0u)));
  } else {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = *reinterpret_cast<const uint16_t*>(base + (off + (i < n ? i * stride : 0u)));
    q.w[0] = h[0] | (h[1] << 16);
    q.w[1] = h[2] | (h[3] << 16);
  }
  return q;
}

// Uniform copies of the plan's records, field by field with constant indexes:
// scalar loads into scalar registers.
__device__ __forceinline__ ConWork load_work(const ConWork* q) {
  ConWork w;
  w.m0 = ld_uniform(&q->m0);
  w.n0 = ld_uniform(&q->n0);
  w.batch = ld_uniform(&q->batch);
  w.gb = ld_uniform(&q->gb);
  w.mext = ld_uniform(&q->mext);
  w.next = ld_uniform(&q->next);
  w.som = ld_uniform(&q->som);
  w.son = ld_uniform(&q->son);
  w.coff = ld_uniform(&q->coff);
#pragma unroll
  for (int d = 0; d < kConMaxBatch; ++d) w.bext[d] = ld_uniform(&q->bext[d]);
  return w;
}

// the work item's batch index as one coordinate per batch letter
struct BatchIdx {
  int32_t c[kConMaxBatch];
};
__device__ __forceinline__ BatchIdx batch_index(const ContractArgs& p, const ConWork& w) {
  BatchIdx b;
  int rem = w.batch;
#pragma unroll
  for (int d = kConMaxBatch - 1; d >= 0; --d) {
    b.c[d] = 0;
    if (d < p.n_batch) {
      b.c[d] = d > 0 ? rem % w.bext[d] : rem;
      if (d > 0) rem /= w.bext[d];
    }
  }
  return b;
}

// element offset of the batch index under a block's batch strides
__device__ __forceinline__ int32_t batch_off(const ContractArgs& p, const BatchIdx& b, const int32_t* stride) {
  int32_t o = 0;
#pragma unroll
  for (int d = 0; d < kConMaxBatch; ++d)
    if (d < p.n_batch) o += b.c[d] * ld_uniform(stride + d);
  return o;
}

__device__ __forceinline__ void store_one(const ContractArgs& p, const ConWork& w, int32_t cbat, int gm, int gn, float v) {
  if (gm >= w.mext || gn >= w.next) return;
  const int32_t idx = cbat + gm * w.som + gn * w.son;
  if (p.res) v += ld_elem(p.res + w.coff, idx, p.dt_out);
  st_elem(p.c + w.coff, idx, p.dt_out, v);
}

// ---------------------------------------------------------------------------
// operands straight into registers, the K walk split over the wavefronts
// ---------------------------------------------------------------------------
template <int TS>
struct Acc;
template <>
struct Acc<16> { using T = f32x4_t; };
template <>
struct Acc<32> { using T = f32x16_t; };

template <int DT, int TS, bool VA, bool VB>
__global__ __launch_bounds__(kThreads) void contract_reg_kernel(const ContractArgs p) {
  constexpr int KG = 4 * 64 / TS;          // k values per group: four MFMAs
  constexpr int NR = TS * TS / 64;         // accumulators per lane
  constexpr int DEPTH = TS == 16 ? 4 : 8;  // groups in flight: 64 k values
  using AccT = typename Acc<TS>::T;
  __shared__ float part[kWaves][TS * TS];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane % TS, h = lane / TS;
  const ConWork w = load_work(p.work + blockIdx.x);
  const BatchIdx bi = batch_index(p, w);
  const int ra = min(w.m0 + r, w.mext - 1), rb = min(w.n0 + r, w.next - 1);  // rows past the edge are not stored

  // this wavefront's run of groups, and the tuple and group it starts at
  int left = p.run[wid].n;
  int t = w.gb + p.run[wid].t, kg = p.run[wid].g;
  constexpr uint32_t ES = DT == EA_F32 ? 4 : 2;
  uint32_t abase = 0, bbase = 0, ask = 0, bsk = 0;  // bytes
  int kext = 0;
  const char *pa = p.a, *pb = p.b;
  auto set_tuple = [&]() {
    const ConMeta* m = p.meta + t;
    pa = p.a + ld_uniform(&m->aoff);
    pb = p.b + ld_uniform(&m->boff);
    kext = ld_uniform(&m->kext);
    ask = ld_uniform(&m->ask) * ES;
    bsk = ld_uniform(&m->bsk) * ES;
    abase = ((uint32_t)batch_off(p, bi, m->abs_) + (uint32_t)ra * ld_uniform(&m->asr)) * ES;
    bbase = ((uint32_t)batch_off(p, bi, m->bbs) + (uint32_t)rb * ld_uniform(&m->bsr)) * ES;
  };
  Quad<DT> qa[DEPTH], qb[DEPTH];
  int nk[DEPTH];  // valid k values of the lane's quad
  // One group into slot s.  Past the run's last group the last one is loaded
  // again (never used): without a condition on the loads the compiler's
  // in-order waits let every slot but the one in use stay in flight.
  auto fetch = [&](int s) {
    const int k = kg * KG + 4 * h, n = min(max(kext - k, 0), 4), kc = n > 0 ? k : 0;
    qa[s] = load_quad<DT, VA>(pa, abase + kc * ask, ask, n);
    qb[s] = load_quad<DT, VB>(pb, bbase + kc * bsk, bsk, n);
    nk[s] = n;
    if (left > 1) {
      --left;
      ++kg;
      if (kg * KG >= kext) {
        ++t;
        kg = 0;
        set_tuple();
      }
    }
  };
  AccT acc{};
  const int n_groups = left;
  if (n_groups > 0) {
    set_tuple();
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) fetch(s);
    for (int g0 = 0; g0 < n_groups; g0 += DEPTH) {
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        if (g0 + s < n_groups) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bool ok = i < nk[s];
            const float a = ok ? qa[s].get(i) : 0.0f, b = ok ? qb[s].get(i) : 0.0f;
            if constexpr (TS == 16) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
            else acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
          }
        }
        fetch(s);
      }
    }
  }
  // accumulator v of a lane: 16 x 16: row 4 h + v, column r;
  // 32 x 32: row 8 (v / 4) + 4 h + v % 4, column r
#pragma unroll
  for (int v = 0; v < NR; ++v) {
    const int row = TS == 16 ? 4 * h + v : 8 * (v >> 2) + 4 * h + (v & 3);
    part[wid][row * TS + r] = acc[v];
  }
  __syncthreads();
  const int32_t cbat = batch_off(p, bi, p.work[blockIdx.x].obs);
#pragma unroll
  for (int e = 0; e < TS * TS / kThreads; ++e) {
    const int o = threadIdx.x + kThreads * e;
    float v = part[0][o];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) v += part[k][o];
    store_one(p, w, cbat, w.m0 + o / TS, w.n0 + o % TS, v);
  }
}

// ---------------------------------------------------------------------------
// 64 x 64 tiles through LDS
// ---------------------------------------------------------------------------
constexpr int kT = 64;       // tile rows and columns
constexpr int kK = 32;       // k values per step
constexpr int kPitchK = 36;  // [row][k] slices: floats per row (16-byte rows, spread over the banks)
constexpr int kPitchR = 72;  // [k][row] slices: floats per k

// A 64 x 32 slice of one operand: two quads per thread, along k where k is the
// operand's contiguous letter (RMAJ false), else along the rows, so that global
// loads run along memory; kept in LDS the way it was read.  Each thread's two
// quads keep their element offsets, advanced by one stride per step.
template <int DT, bool RMAJ, bool VEC>
struct Slice {
  static constexpr int kElems = RMAJ ? kK * kPitchR : kT * kPitchK;
  static constexpr uint32_t ES = DT == EA_F32 ? 4 : 2;
  Quad<DT> q[2][2];  // two steps in flight
  int n[2][2];       // valid values of each quad
  bool whole[2];     // (uniform) the slice lies inside the block: no masks
  const char* base;
  uint32_t off[2], home, stride, step;  // bytes
  int kext;
  __device__ __forceinline__ static int quad_row(int i) {
    const int e = threadIdx.x + kThreads * i;
    return RMAJ ? (e % (kT / 4)) * 4 : e / (kK / 4);
  }
  __device__ __forceinline__ static int quad_k(int i) {
    const int e = threadIdx.x + kThreads * i;
    return RMAJ ? e / (kT / 4) : (e % (kK / 4)) * 4;
  }
  __device__ __forceinline__ void set(const char* b, int32_t o, int r0, int rstride, int kstride, int ke) {
    base = b;
    home = (uint32_t)o * ES;
    stride = (uint32_t)(RMAJ ? rstride : kstride) * ES;
    step = (uint32_t)kstride * (kK * ES);
    kext = ke;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      off[i] = home + ((uint32_t)(r0 + quad_row(i)) * (uint32_t)rstride + (uint32_t)quad_k(i) * (uint32_t)kstride) * ES;
  }
  __device__ __forceinline__ void load(int set, int r0, int rext, int k0) {
    whole[set] = r0 + kT <= rext && k0 + kK <= kext;
    uint32_t at[2] = {off[0], off[1]};
    n[set][0] = n[set][1] = 4;
    if (!whole[set]) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int rows = rext - r0 - quad_row(i), ks = kext - k0 - quad_k(i);  // left from the quad's first value
        n[set][i] = RMAJ ? (ks > 0 ? min(max(rows, 0), 4) : 0) : (rows > 0 ? min(max(ks, 0), 4) : 0);
        at[i] = n[set][i] > 0 ? off[i] : home;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      q[set][i] = load_quad<DT, VEC>(base, at[i], stride, n[set][i]);
      off[i] += step;
    }
  }
  __device__ __forceinline__ void stash(int set, float* s) {
    float f[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) f[i][j] = q[set][i].get(j);
    if (!whole[set]) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) f[i][j] = j < n[set][i] ? f[i][j] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float* d = s + (RMAJ ? quad_k(i) * kPitchR + quad_row(i) : quad_row(i) * kPitchK + quad_k(i));
      *reinterpret_cast<float4*>(d) = make_float4(f[i][0], f[i][1], f[i][2], f[i][3]);
    }
  }
  // the lane's four k values (4h .. 4h+3 of group kg) of one row
  __device__ __forceinline__ static void frag(const float* s, int row, int kg, int h, float (&f)[4]) {
    const int k = kg * 8 + 4 * h;
    if constexpr (RMAJ) {
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = s[(k + j) * kPitchR + row];
    } else {
      const float4 v = *reinterpret_cast<const float4*>(s + row * kPitchK + k);
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
  }
};

template <int DT, bool RA, bool RB, bool VA, bool VB>
__global__ __launch_bounds__(kThreads) void contract_lds_kernel(const ContractArgs p) {
  using SA = Slice<DT, RA, VA>;
  using SB = Slice<DT, RB, VB>;
  __shared__ __attribute__((aligned(16))) float sA[2][SA::kElems];
  __shared__ __attribute__((aligned(16))) float sB[2][SB::kElems];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = 32 * (wid >> 1), wn = 32 * (wid & 1), r = lane & 31, h = lane >> 5;
  const ConWork w = load_work(p.work + blockIdx.x);
  const BatchIdx bi = batch_index(p, w);

  int t = w.gb, k0 = 0;
  const int te = w.gb + p.nt;
  SA la;
  SB lb;
  auto set_tuple = [&]() {
    const ConMeta* m = p.meta + t;
    const int ke = ld_uniform(&m->kext);
    la.set(p.a + ld_uniform(&m->aoff), batch_off(p, bi, m->abs_), w.m0, ld_uniform(&m->asr), ld_uniform(&m->ask), ke);
    lb.set(p.b + ld_uniform(&m->boff), batch_off(p, bi, m->bbs), w.n0, ld_uniform(&m->bsr), ld_uniform(&m->bsk), ke);
  };
  // The next step's slices into register set i; past the last step nothing
  // that is used: quads past the block's end load its first values (see fetch)
  auto load = [&](int i) {
    la.load(i, w.m0, w.mext, k0);
    lb.load(i, w.n0, w.next, k0);
    k0 += kK;
    if (k0 >= la.kext && t + 1 < te) {
      ++t;
      k0 = 0;
      set_tuple();
    }
  };
  auto stash = [&](int i) {
    la.stash(i, sA[i]);
    lb.stash(i, sB[i]);
  };
  f32x16_t acc{};
  // every operand of the step is read before its first MFMA, so that one LDS
  // latency covers the step's 16 MFMAs
  auto compute = [&](int i) {
    float fa[kK / 8][4], fb[kK / 8][4];
#pragma unroll
    for (int kg = 0; kg < kK / 8; ++kg) {
      SA::frag(sA[i], wm + r, kg, h, fa[kg]);
      SB::frag(sB[i], wn + r, kg, h, fb[kg]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kg = 0; kg < kK / 8; ++kg)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[kg][j], fb[kg][j], acc, 0, 0, 0);
  };
  // One barrier per step: step s is computed from buffer s % 2 while the loads
  // of step s + 1 (issued a step ago) and s + 2 are in flight; those of
  // s + 1 then go to the other buffer.  Two steps per iteration, so that
  // every index is a constant; an odd count ends with a step of zeros.
  const int n = p.n_steps;
  if (n > 0) {
    set_tuple();
    load(0);
    load(1);
    stash(0);
    __syncthreads();
    for (int s = 0; s < n; s += 2) {
      load(0);
      compute(0);
      stash(1);
      __syncthreads();
      load(1);
      compute(1);
      stash(0);
      __syncthreads();
    }
  }
  const int32_t cbat = batch_off(p, bi, p.work[blockIdx.x].obs);
#pragma unroll
  for (int v = 0; v < 16; ++v)
    store_one(p, w, cbat, w.m0 + wm + 8 * (v >> 2) + 4 * h + (v & 3), w.n0 + wn + r, acc[v]);
}

// Plan time, after the join.  One thread per tuple: its operand blocks'
// offsets, contracted extent and element strides.
__device__ __forceinline__ int32_t dim_stride(const DevBlk& b, int rank, int d) {
  if (d < 0) return 0;
  int32_t s = 1;
  for (int x = d + 1; x < rank; ++x) s *= b.ext[x];
  return s;
}

__global__ __launch_bounds__(256) void contract_meta_kernel(const ContractArgs p, const ContractDims d, ConMeta* meta,
                                                            const int32_t* count, int64_t cap) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= cap || q >= *count) return;
  const int32_t* tp = d.tuples + q * 3;
  const DevBlk& A = d.blk_a[tp[1 + d.a_op]];
  const DevBlk& B = d.blk_b[tp[2 - d.a_op]];
  ConMeta m;
  m.aoff = A.off;
  m.boff = B.off;
  m.kext = A.ext[d.ak];
  m.asr = dim_stride(A, d.a_rank, d.am);
  m.ask = dim_stride(A, d.a_rank, d.ak);
  m.bsr = dim_stride(B, d.b_rank, d.bn);
  m.bsk = dim_stride(B, d.b_rank, d.bk);
  m.pad = 0;
  for (int i = 0; i < kConMaxBatch; ++i) {
    m.abs_[i] = i < p.n_batch ? dim_stride(A, d.a_rank, d.ab[i]) : 0;
    m.bbs[i] = i < p.n_batch ? dim_stride(B, d.b_rank, d.bb[i]) : 0;
  }
  meta[q] = m;
}

// One thread per work item: its group's first tuple and its output block.
__global__ __launch_bounds__(256) void contract_work_kernel(const ContractArgs p, const ContractDims d, ConWork* work) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= p.n_work) return;
  ConWork& w = work[q];
  const DevBlk& C = d.blk_c[w.block];
  w.gb = d.goff[w.block];
  w.mext = d.cm >= 0 ? C.ext[d.cm] : 1;
  w.next = d.cn >= 0 ? C.ext[d.cn] : 1;
  w.coff = C.off;
  w.som = dim_stride(C, d.c_rank, d.cm);
  w.son = dim_stride(C, d.c_rank, d.cn);
  for (int i = 0; i < kConMaxBatch; ++i) {
    w.bext[i] = i < p.n_batch ? C.ext[d.cb[i]] : 1;
    w.obs[i] = i < p.n_batch ? dim_stride(C, d.c_rank, d.cb[i]) : 0;
  }
}

template <int DT, int TS>
void launch_reg(const ContractArgs& a, dim3 grid, hipStream_t s) {
  const bool va = a.vec_a && !a.rmaj_a, vb = a.vec_b && !a.rmaj_b;  // four consecutive k in one load
  if (va && vb) hipLaunchKernelGGL((contract_reg_kernel<DT, TS, true, true>), grid, dim3(kThreads), 0, s, a);
  else if (va) hipLaunchKernelGGL((contract_reg_kernel<DT, TS, true, false>), grid, dim3(kThreads), 0, s, a);
  else if (vb) hipLaunchKernelGGL((contract_reg_kernel<DT, TS, false, true>), grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL((contract_reg_kernel<DT, TS, false, false>), grid, dim3(kThreads), 0, s, a);
}

template <int DT, bool RA, bool RB>
void launch_lds(const ContractArgs& a, dim3 grid, hipStream_t s) {
  if (a.vec_a && a.vec_b)
    hipLaunchKernelGGL((contract_lds_kernel<DT, RA, RB, true, true>), grid, dim3(kThreads), 0, s, a);
  else if (a.vec_a)
    hipLaunchKernelGGL((contract_lds_kernel<DT, RA, RB, true, false>), grid, dim3(kThreads), 0, s, a);
  else if (a.vec_b)
    hipLaunchKernelGGL((contract_lds_kernel<DT, RA, RB, false, true>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((contract_lds_kernel<DT, RA, RB, false, false>), grid, dim3(kThreads), 0, s, a);
}

template <int DT>
hipError_t launch_dt(const ContractArgs& a, hipStream_t s) {
  const dim3 grid((uint32_t)a.n_work);
  if (a.tile == 16) launch_reg<DT, 16>(a, grid, s);
  else if (a.tile == 32) launch_reg<DT, 32>(a, grid, s);
  else if (a.rmaj_a && a.rmaj_b) launch_lds<DT, true, true>(a, grid, s);
  else if (a.rmaj_a) launch_lds<DT, true, false>(a, grid, s);
  else if (a.rmaj_b) launch_lds<DT, false, true>(a, grid, s);
  else launch_lds<DT, false, false>(a, grid, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_contract_prep(const ContractArgs& a, const ContractDims& d, ConMeta* meta, ConWork* work,
                                const int32_t* count, int64_t tuple_cap, hipStream_t s) {
  if (tuple_cap > 0)
    hipLaunchKernelGGL(contract_meta_kernel, dim3((uint32_t)((tuple_cap + 255) / 256)), dim3(256), 0, s, a, d, meta,
                       count, tuple_cap);
  if (a.n_work > 0)
    hipLaunchKernelGGL(contract_work_kernel, dim3((uint32_t)((a.n_work + 255) / 256)), dim3(256), 0, s, a, d, work);
  return hipGetLastError();
}

hipError_t launch_contract(const ContractArgs& a, hipStream_t s) {
  if (a.n_work == 0) return hipSuccess;
  switch (a.dt_in) {
    case EA_F32: return launch_dt<EA_F32>(a, s);
    case EA_BF16: return launch_dt<EA_BF16>(a, s);
    default: return launch_dt<EA_F16>(a, s);
  }
}

}  // namespace ea
