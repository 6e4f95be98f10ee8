// Linear kernels (Alg. 1 CallLinear): kick and drift, streaming over slots
// (SoA) or records (AoS), and the FP64 conservation reductions.
#include <algorithm>
#include <initializer_list>
#include <mutex>
#include <type_traits>

#include "sph_device.h"

namespace sph {
namespace {

constexpr int kThreads = 256;
constexpr int kReduceBlocks = 1024;
constexpr int kReduceVals = 8;

// The cell along one axis of a wrapped coordinate and, at depth sub_bits,
// the sub-cell inside it (the binning's definitions), as one integer.
__device__ __forceinline__ int cell_sub_axis(double xw, int n_c, int sub_bits) {
  const int c = cell_axis(xw, n_c);
  if (sub_bits == 0) return c;
  const int R = 1 << sub_bits;
  const double t = floor(xw * (double)(n_c * R));
  const int sa = (t == t) ? (int)fmin(fmax(t - (double)c * R, 0.0), (double)(R - 1)) : 0;
  return c * R + sa;
}

// Kick v and u with the FP32 rates, drift x in FP64 with the kicked v, wrap.
// Returns whether the particle's cell (or sub-cell at depth sub_bits)
// changed.
__device__ __forceinline__ bool kick_drift_one(double x[3], float v[3], float& u,
                                               const float a[3], float du, float dtk, double dtd,
                                               int n_c, int sub_bits) {
  bool moved = false;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    v[c] = __builtin_fmaf(a[c], dtk, v[c]);
    double xn = __builtin_fma((double)v[c], dtd, x[c]);
    xn = wrap01(xn);
    moved |= cell_sub_axis(wrap01(x[c]), n_c, sub_bits) != cell_sub_axis(xn, n_c, sub_bits);
    x[c] = xn;
  }
  u = __builtin_fmaf(du, dtk, u);
  return moved;
}

// Adds the block's count of moved particles to *counter: one atomic per
// block that has any.
__device__ __forceinline__ void count_moved(bool moved, int32_t* counter) {
  __shared__ int wsum[kThreads / 64];
  const uint64_t b = __ballot(moved);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = (int)__popcll(b);
  __syncthreads();
  if (threadIdx.x == 0 && counter) {
    int t = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += wsum[w];
    if (t) atomicAdd(counter, t);
  }
}

struct KickSoa {
  double* x[3];
  float* v[3];
  float* u;
  const float* a[3];
  const float* du;
};

// One slot per thread. Every field is streamed once (read, then written in
// place), so loads and stores are non-temporal: the lines go through the
// caches without displacing data that is reused (measured on 4M slots
// beyond the Infinity Cache: 4.1 -> 5.3 TB/s at 96 B per slot).
__global__ __launch_bounds__(kThreads) void k_kick_drift(KickSoa s, int n, int n_c, int sub_bits,
                                                          float dtk, double dtd, int32_t* moved) {
  const int k = blockIdx.x * kThreads + threadIdx.x;
  bool mv = false;
  if (k < n) {
    double x[3];
    float v[3], a[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c] = __builtin_nontemporal_load(s.x[c] + k);
      v[c] = __builtin_nontemporal_load(s.v[c] + k);
      a[c] = __builtin_nontemporal_load(s.a[c] + k);
    }
    float u = __builtin_nontemporal_load(s.u + k);
    const float du = __builtin_nontemporal_load(s.du + k);
    mv = kick_drift_one(x, v, u, a, du, dtk, dtd, n_c, sub_bits);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      __builtin_nontemporal_store(x[c], s.x[c] + k);
      __builtin_nontemporal_store(v[c], s.v[c] + k);
    }
    __builtin_nontemporal_store(u, s.u + k);
  }
  count_moved(mv, moved);
}

// Records' 32-bit or 64-bit fields of type RT (kRt: read from the layout)
constexpr int kRt = -1;
template <int RT>
struct RecField {
  using T = std::conditional_t<RT == DT_F64, double, float>;
  __device__ __forceinline__ static T load(const AosLayout& L, const char* rec, int f, int c) {
    if constexpr (RT == kRt) return rec_load32(rec, L.off[f], L.dt[f], c);
    else return reinterpret_cast<const T*>(rec + L.off[f])[c];
  }
  __device__ __forceinline__ static void store(const AosLayout& L, char* rec, int f, int c,
                                               float v) {
    if constexpr (RT == kRt) rec_store32(rec, L.off[f], L.dt[f], v, c);
    else reinterpret_cast<T*>(rec + L.off[f])[c] = v;
  }
};

// The type that all the given fields (of those present) have, or kRt
int common_type(const AosLayout& L, std::initializer_list<int> fields) {
  int dt = kRt;
  for (const int f : fields) {
    if (L.off[f] == kAbsent) continue;
    if (dt != kRt && L.dt[f] != dt) return kRt;
    dt = L.dt[f];
  }
  return dt == DT_F32 || dt == DT_F64 ? dt : kRt;
}

// One record per thread. With the types fixed all of a record's loads are in
// flight together; looked up at each load, a record cost one latency per field
// (262144 records of 200 bytes: 38 -> 22 us).
template <int RT>
__global__ __launch_bounds__(kThreads) void k_kick_drift_aos(char* __restrict__ aos, AosLayout L,
                                                              int n, int n_c, int sub_bits,
                                                              float dtk, double dtd,
                                                              int32_t* moved) {
  using F = RecField<RT>;
  const int k = blockIdx.x * kThreads + threadIdx.x;
  bool mv = false;
  if (k < n) {
    char* rec = aos + (size_t)k * L.stride;
    double* xp = reinterpret_cast<double*>(rec + L.off[SPH_A_X]);
    double x[3];
    typename F::T vr[3], ar[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c] = xp[c];
      vr[c] = F::load(L, rec, SPH_A_V, c);
      ar[c] = F::load(L, rec, SPH_A_A, c);
    }
    const typename F::T ur = F::load(L, rec, SPH_A_U, 0), dur = F::load(L, rec, SPH_A_DU, 0);
    float v[3], a[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c] = wrap01(x[c]);
      v[c] = (float)vr[c];
      a[c] = (float)ar[c];
    }
    float u = (float)ur;
    mv = kick_drift_one(x, v, u, a, (float)dur, dtk, dtd, n_c, sub_bits);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      xp[c] = x[c];
      F::store(L, rec, SPH_A_V, c, v[c]);
    }
    F::store(L, rec, SPH_A_U, 0, u);
  }
  count_moved(mv, moved);
}

// Inputs of the reductions at slot k: the SoA arrays (m and v in their
// storage formats), or the AoS records through the cell list (record
// perm[k]), in the same slot order, so FP32 storage and FP32 records give
// the same sums bit for bit. `load` only loads (formats MT, VT or RT fixed at
// compile time; kRt: read from the arguments) and `get` widens, so that all
// loads of a slot are in flight together: with the format looked up at each
// load, a slot cost one memory latency per field (262144 FP64 records of 200
// bytes: 36.6 -> 11.8 us; 3M FP32 slots: sums 28 -> 23, totals 21 -> 19).
template <int DT>
struct Stored {
  using Raw = std::conditional_t<DT == DT_F16 || DT == DT_BF16, uint16_t, float>;
  __device__ __forceinline__ static Raw load(const void* p, int rt, int k) {
    if constexpr (DT == kRt) return load_q(p, rt, k, 1.0f);
    else return static_cast<const Raw*>(p)[k];
  }
  __device__ __forceinline__ static float get(Raw v) {
    if constexpr (DT == DT_F16) return f16_bits_to_f32(v);
    else if constexpr (DT == DT_BF16) return bf16_bits_to_f32(v);
    else return v;
  }
};

struct RedVals {
  double m, v[3], a[3], du, ngb, nfrc;
};

template <int MT, int VT>
struct RedSoa {
  const void* m;
  int mhu_dt;
  float lm;
  const void* v[3];
  int vel_dt;
  const float* a[3];
  const float* du;
  const int32_t* nngb;
  const int32_t* nforce;

  struct Raw {
    typename Stored<MT>::Raw m;
    typename Stored<VT>::Raw v[3];
    float a[3], du;
    int32_t ngb, nfrc;
  };
  __device__ __forceinline__ Raw load(int k) const {
    Raw r{};
    if (m) r.m = Stored<MT>::load(m, mhu_dt, k);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r.v[c] = Stored<VT>::load(v[c], vel_dt, k);
      r.a[c] = a[c][k];
    }
    r.du = du[k];
    if (nngb) r.ngb = nngb[k];
    if (nforce) r.nfrc = nforce[k];
    return r;
  }
  __device__ __forceinline__ RedVals get(const Raw& r) const {
    RedVals x;
    x.m = m ? (double)(Stored<MT>::get(r.m) * lm) : 1.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x.v[c] = Stored<VT>::get(r.v[c]);
      x.a[c] = r.a[c];
    }
    x.du = r.du;
    x.ngb = (double)r.ngb;
    x.nfrc = (double)r.nfrc;
    return x;
  }
};

// RT: DT_F32 or DT_F64 where m, v, a and du all have that type
template <int RT>
struct RedAos {
  const char* aos;
  AosLayout L;
  const int32_t* perm;
  int n;

  using T = typename RecField<RT>::T;
  struct Raw {
    T m, v[3], a[3], du;
    int32_t ngb, nfrc;
  };
  __device__ __forceinline__ Raw load(int k) const {
    const char* rec = aos + (size_t)min(max(perm[k], 0), n - 1) * L.stride;
    Raw r{};
    if (L.off[SPH_A_M] != kAbsent) r.m = RecField<RT>::load(L, rec, SPH_A_M, 0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r.v[c] = RecField<RT>::load(L, rec, SPH_A_V, c);
      r.a[c] = RecField<RT>::load(L, rec, SPH_A_A, c);
    }
    r.du = RecField<RT>::load(L, rec, SPH_A_DU, 0);
    if (L.off[SPH_A_NNGB] != kAbsent)
      r.ngb = *reinterpret_cast<const int32_t*>(rec + L.off[SPH_A_NNGB]);
    if (L.off[SPH_A_NFORCE] != kAbsent)
      r.nfrc = *reinterpret_cast<const int32_t*>(rec + L.off[SPH_A_NFORCE]);
    return r;
  }
  __device__ __forceinline__ RedVals get(const Raw& r) const {
    RedVals x;
    x.m = L.off[SPH_A_M] != kAbsent ? (double)(float)r.m : 1.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x.v[c] = (float)r.v[c];
      x.a[c] = (float)r.a[c];
    }
    x.du = (float)r.du;
    x.ngb = (double)r.ngb;
    x.nfrc = (double)r.nfrc;
    return x;
  }
};

// Slots k0, k0 + stride, ... below n in order, the next one's loads issued
// before the arithmetic on this one: a block's time is the latency of its
// loads, a dozen slots in a row at 3M.
template <class S, class Add>
__device__ __forceinline__ void stream_slots(const S& s, int n, Add add) {
  const int stride = gridDim.x * kThreads;
  int k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= n) return;
  typename S::Raw r = s.load(k);
  while (n - k > stride) {
    k += stride;
    const typename S::Raw next = s.load(k);
    add(s.get(r));
    r = next;
  }
  add(s.get(r));
}

// The sum (minimum where q == mn) of each value over a wave
template <int mn>
__device__ __forceinline__ void wave_tree(double (&acc)[kReduceVals]) {
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int q = 0; q < kReduceVals; ++q) {
      const double w = __shfl_xor(acc[q], o);
      acc[q] = q == mn ? fmin(acc[q], w) : acc[q] + w;
    }
  }
}

// The block's eight values from its waves', in wave order, to out
template <int mn>
__device__ __forceinline__ void block_vals(double (&acc)[kReduceVals], double* __restrict__ out) {
  __shared__ double lds[kThreads / 64][kReduceVals];
  wave_tree<mn>(acc);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < kReduceVals; ++q) lds[threadIdx.x >> 6][q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x < kReduceVals) {
    const int q = threadIdx.x;
    double t = q == mn ? __builtin_inf() : 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t = q == mn ? fmin(t, lds[w][q]) : t + lds[w][q];
    out[q] = t;
  }
}

template <class R>
__global__ __launch_bounds__(kThreads) void k_reduce_partial(R s, int n,
                                                              double* __restrict__ part) {
  double acc[kReduceVals];
#pragma unroll
  for (int q = 0; q < kReduceVals; ++q) acc[q] = 0.0;
  stream_slots(s, n, [&](const RedVals& x) {
    double va = 0.0, an = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      acc[c] += x.m * x.a[c];
      va += x.v[c] * x.a[c];
      an += x.a[c] * x.a[c];
    }
    acc[3] += x.m * (va + x.du);
    acc[4] += x.m * sqrt(an);
    acc[5] += x.m * (fabs(va) + fabs(x.du));
    acc[6] += x.ngb;
    acc[7] += x.nfrc;
  });
  block_vals<-1>(acc, part + blockIdx.x * kReduceVals);
}

// Combines the nb (at most kReduceBlocks) per-block partials of each value
// in a fixed order: thread t takes partials t, t + 256, ..., then a fixed
// shuffle/LDS tree combines threads. All partials of a thread are loaded at
// once: one latency and one barrier instead of one of each per value (8.5 ->
// 4.0 us).
template <int mn>
__global__ __launch_bounds__(kThreads) void k_combine(const double* __restrict__ part, int nb,
                                                      double* __restrict__ out) {
  constexpr int kEach = kReduceBlocks / kThreads;
  double p[kEach][kReduceVals], acc[kReduceVals];
#pragma unroll
  for (int i = 0; i < kEach; ++i) {
    const int b = min((int)threadIdx.x + i * kThreads, nb - 1);
#pragma unroll
    for (int q = 0; q < kReduceVals; ++q) p[i][q] = part[b * kReduceVals + q];
  }
#pragma unroll
  for (int q = 0; q < kReduceVals; ++q) {
    acc[q] = q == mn ? __builtin_inf() : 0.0;
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
      const bool in = (int)threadIdx.x + i * kThreads < nb;
      const double t = q == mn ? fmin(acc[q], p[i][q]) : acc[q] + p[i][q];
      acc[q] = in ? t : acc[q];
    }
  }
  block_vals<mn>(acc, out);
}

// Blocks of a reduction over n slots: a block without a slot would add zero
// (4096 slots: 5.7 -> 4.0 us)
int reduce_blocks(int n) {
  return std::min(kReduceBlocks, std::max((n + kThreads - 1) / kThreads, 1));
}

// --- leapfrog support: predicted v, u; time step and conserved totals -----

struct PredIn {
  const float* v[3];      // kick view V (half-step values)
  const float* u;         // kick view UK
  void* vq[3];            // force view VQ (stored format)
  void* uq;               // U (stored format)
  int vel_dt, mhu_dt;
  float store_u;
  const int32_t* perm;
  const char* aos;
  AosLayout L;
};

// v and u predicted to the end of the step with the last rates (record
// fields A, DU of the slot's record), stored in the force/density formats.
__global__ __launch_bounds__(kThreads) void k_predict(PredIn s, int n, float dth) {
  const int k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= n) return;
  const char* rec = s.aos + (size_t)min(max(s.perm[k], 0), n - 1) * s.L.stride;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float a = rec_load32(rec, s.L.off[SPH_A_A], s.L.dt[SPH_A_A], c);
    store_q32(s.vq[c], s.vel_dt, k, __builtin_fmaf(a, dth, s.v[c][k]), 1.0f);
  }
  const float du = rec_load32(rec, s.L.off[SPH_A_DU], s.L.dt[SPH_A_DU]);
  store_q32(s.uq, s.mhu_dt, k, __builtin_fmaf(du, dth, s.u[k]), s.store_u);
}

template <int MT>
struct TotIn {
  const void* m;
  const void* h;
  int mhu_dt;
  float lm, lh;
  const float* v[3];
  const float* u;
  const float* vsig;
  double gk, cfl;

  struct Raw {
    typename Stored<MT>::Raw m, h;
    float v[3], u, vsig;
  };
  __device__ __forceinline__ Raw load(int k) const {
    Raw r;
    r.m = Stored<MT>::load(m, mhu_dt, k);
    r.h = Stored<MT>::load(h, mhu_dt, k);
#pragma unroll
    for (int c = 0; c < 3; ++c) r.v[c] = v[c][k];
    r.u = u[k];
    r.vsig = vsig[k];
    return r;
  }
  struct Vals {
    double m, h, v[3], u, vsig;
  };
  __device__ __forceinline__ Vals get(const Raw& r) const {
    return {(double)(Stored<MT>::get(r.m) * lm), (double)(Stored<MT>::get(r.h) * lh),
            {r.v[0], r.v[1], r.v[2]}, r.u, r.vsig};
  }
};

// Per-block partials: sums of m v (3), m |v|^2 / 2, m u, m, the count of
// slots with vsig > 0 (slot 7) and the minimum CFL step (slot 6).
template <class T>
__global__ __launch_bounds__(kThreads) void k_totals_partial(T s, int n,
                                                             double* __restrict__ part) {
  double acc[kReduceVals];
#pragma unroll
  for (int q = 0; q < kReduceVals; ++q) acc[q] = 0.0;
  acc[6] = __builtin_inf();
  stream_slots(s, n, [&](const typename T::Vals& x) {
    double v2 = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      acc[c] += x.m * x.v[c];
      v2 += x.v[c] * x.v[c];
    }
    acc[3] += 0.5 * x.m * v2;
    acc[4] += x.m * x.u;
    acc[5] += x.m;
    if (x.vsig > 0.0) {
      acc[6] = fmin(acc[6], s.cfl * (s.gk * x.h) / x.vsig);
      acc[7] += 1.0;
    }
  });
  block_vals<6>(acc, part + blockIdx.x * kReduceVals);
}

}  // namespace

hipError_t launch_predict(const sph_soa& soa, const Prec& p, const CellsDev& c, const void* aos,
                          const AosLayout& L, double dth, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  PredIn in;
  for (int a = 0; a < 3; ++a) {
    in.v[a] = static_cast<const float*>(soa.f[SPH_S_V_X + a]);
    in.vq[a] = soa.f[SPH_S_VQ_X + a];
  }
  in.u = static_cast<const float*>(soa.f[SPH_S_UK]);
  in.uq = soa.f[SPH_S_U];
  in.vel_dt = p.vel;
  in.mhu_dt = p.mhu;
  in.store_u = p.store_u;
  in.perm = c.perm;
  in.aos = static_cast<const char*>(aos);
  in.L = L;
  k_predict<<<(c.n + kThreads - 1) / kThreads, kThreads, 0, s>>>(in, c.n, (float)dth);
  return hipGetLastError();
}

namespace {

// f(format as an integral constant); packed codes take the run-time reader
template <class Fn>
hipError_t with_format(int dt, Fn f) {
  if (dt == DT_F32) return f(std::integral_constant<int, DT_F32>{});
  if (dt == DT_F16) return f(std::integral_constant<int, DT_F16>{});
  if (dt == DT_BF16) return f(std::integral_constant<int, DT_BF16>{});
  return f(std::integral_constant<int, kRt>{});
}

}  // namespace

hipError_t launch_step_totals(const sph_soa& soa, const Prec& p, int n, double gamma_k,
                              double c_cfl, double* out, void* ws, hipStream_t s) {
  double* part = static_cast<double*>(ws);
  return with_format(p.mhu, [&](auto mt) {
    TotIn<decltype(mt)::value> t;
    t.m = soa.f[SPH_S_M];
    t.h = soa.f[SPH_S_H];
    t.mhu_dt = p.mhu;
    t.lm = p.load_m;
    t.lh = p.load_h;
    for (int a = 0; a < 3; ++a) t.v[a] = static_cast<const float*>(soa.f[SPH_S_V_X + a]);
    t.u = static_cast<const float*>(soa.f[SPH_S_UK]);
    t.vsig = static_cast<const float*>(soa.f[SPH_S_VSIG]);
    t.gk = gamma_k;
    t.cfl = c_cfl;
    k_totals_partial<<<reduce_blocks(n), kThreads, 0, s>>>(t, n, part);
    k_combine<6><<<1, kThreads, 0, s>>>(part, reduce_blocks(n), out);
    return hipGetLastError();
  });
}

hipError_t launch_kick_drift(const sph_soa& soa, const CellsDev& c, double dtk, double dtd,
                             int32_t* moved, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  KickSoa k;
  for (int a = 0; a < 3; ++a) {
    k.x[a] = static_cast<double*>(soa.f[SPH_S_X_X + a]);
    k.v[a] = static_cast<float*>(soa.f[SPH_S_V_X + a]);
    k.a[a] = static_cast<const float*>(soa.f[SPH_S_A_X + a]);
  }
  k.u = static_cast<float*>(soa.f[SPH_S_UK]);
  k.du = static_cast<const float*>(soa.f[SPH_S_DU]);
  k_kick_drift<<<(c.n + kThreads - 1) / kThreads, kThreads, 0, s>>>(k, c.n, c.n_c, c.sub_bits,
                                                                     (float)dtk, dtd, moved);
  return hipGetLastError();
}

hipError_t launch_kick_drift_aos(void* aos, const AosLayout& L, int n, int n_c, int sub_bits,
                                 double dtk, double dtd, int32_t* moved, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int G = (n + kThreads - 1) / kThreads;
  const int rt = common_type(L, {SPH_A_V, SPH_A_A, SPH_A_U, SPH_A_DU});
  char* const a = static_cast<char*>(aos);
  if (rt == DT_F64)
    k_kick_drift_aos<DT_F64><<<G, kThreads, 0, s>>>(a, L, n, n_c, sub_bits, (float)dtk, dtd, moved);
  else if (rt == DT_F32)
    k_kick_drift_aos<DT_F32><<<G, kThreads, 0, s>>>(a, L, n, n_c, sub_bits, (float)dtk, dtd, moved);
  else
    k_kick_drift_aos<kRt><<<G, kThreads, 0, s>>>(a, L, n, n_c, sub_bits, (float)dtk, dtd, moved);
  return hipGetLastError();
}

size_t reduce_workspace_bytes(int n) {
  (void)n;
  return sizeof(double) * kReduceBlocks * kReduceVals;
}

// --- streaming probes of the HBM rate (the ceiling the streaming kernels are
// measured against): 16-byte non-temporal accesses, one per thread ----------
typedef float f4v __attribute__((ext_vector_type(4)));

namespace {

__global__ __launch_bounds__(kThreads) void k_probe_copy(const f4v* __restrict__ a,
                                                          f4v* __restrict__ b, size_t n) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(a + i), b + i);
}

__global__ __launch_bounds__(kThreads) void k_probe_write(f4v* __restrict__ b, size_t n) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) {
    const f4v v = {1.0f, 2.0f, 3.0f, (float)i};
    __builtin_nontemporal_store(v, b + i);
  }
}

// grid-stride read, four loads in flight per thread; one word is written only
// when the sum takes a value no input here produces, so the loads stay live
__global__ __launch_bounds__(kThreads) void k_probe_read(const f4v* __restrict__ a,
                                                          float* __restrict__ sink, size_t n) {
  const size_t stride = (size_t)gridDim.x * kThreads;
  size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  float acc = 0.0f;
  for (; i + 3 * stride < n; i += 4 * stride) {
    f4v v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(a + i + u * stride);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += v[u].x + v[u].y + v[u].z + v[u].w;
  }
  for (; i < n; i += stride) acc += a[i].x;
  if (acc == -1.5e38f) sink[0] = acc;
}

}  // namespace

hipError_t launch_hbm_probe(int mode, const void* src, void* dst, size_t bytes, hipStream_t s) {
  const size_t n = bytes / sizeof(f4v);
  if (n == 0) return hipSuccess;
  if (mode == SPH_PROBE_COPY) {
    k_probe_copy<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        static_cast<const f4v*>(src), static_cast<f4v*>(dst), n);
  } else if (mode == SPH_PROBE_WRITE) {
    k_probe_write<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        static_cast<f4v*>(dst), n);
  } else {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    k_probe_read<<<cus * 256, kThreads, 0, s>>>(static_cast<const f4v*>(src),
                                                static_cast<float*>(dst), n);
  }
  return hipGetLastError();
}

// Scratch of the allocation-free reduction (sph_reduce_static): the
// kReduceBlocks x kReduceVals partial sums, one copy on each device the
// library runs on. Host code never passes the array's name to a kernel: it
// resolves each device's address once, with that device current, and
// passes that address.
static __device__ __align__(256) double scratch[kReduceBlocks * kReduceVals];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

size_t reduce_scratch_bytes() { return sizeof(scratch); }

hipError_t reduce_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

namespace {

template <class R>
hipError_t reduce(const R& r, int n, double* out, void* ws, hipStream_t s) {
  double* part = static_cast<double*>(ws);
  k_reduce_partial<<<reduce_blocks(n), kThreads, 0, s>>>(r, n, part);
  k_combine<-1><<<1, kThreads, 0, s>>>(part, reduce_blocks(n), out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_reduce(const sph_soa& soa, const Prec& p, int n, double* out, void* ws,
                         hipStream_t s) {
  return with_format(p.mhu, [&](auto mt) {
    return with_format(p.vel, [&](auto vt) {
      RedSoa<decltype(mt)::value, decltype(vt)::value> r;
      r.m = soa.f[SPH_S_M];
      r.mhu_dt = p.mhu;
      r.lm = p.load_m;
      for (int a = 0; a < 3; ++a) {
        r.v[a] = soa.f[SPH_S_VQ_X + a];
        r.a[a] = static_cast<const float*>(soa.f[SPH_S_A_X + a]);
      }
      r.vel_dt = p.vel;
      r.du = static_cast<const float*>(soa.f[SPH_S_DU]);
      r.nngb = static_cast<const int32_t*>(soa.f[SPH_S_NNGB]);
      r.nforce = static_cast<const int32_t*>(soa.f[SPH_S_NFORCE]);
      return reduce(r, n, out, ws, s);
    });
  });
}

hipError_t launch_reduce_aos(const void* aos, const AosLayout& L, const CellsDev& c, double* out,
                             void* ws, hipStream_t s) {
  const char* rec = static_cast<const char*>(aos);
  const int dt = common_type(L, {SPH_A_M, SPH_A_V, SPH_A_A, SPH_A_DU});
  if (dt == DT_F64) return reduce(RedAos<DT_F64>{rec, L, c.perm, c.n}, c.n, out, ws, s);
  if (dt == DT_F32) return reduce(RedAos<DT_F32>{rec, L, c.perm, c.n}, c.n, out, ws, s);
  return reduce(RedAos<kRt>{rec, L, c.perm, c.n}, c.n, out, ws, s);
}

}  // namespace sph
