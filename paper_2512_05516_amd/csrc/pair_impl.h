// Quadratic kernels (implementation header, included by the pair_*.hip
// translation units): the density loop and the force loop over the cell list
// (Alg. 1 CallQuadratic; Eq. density, Eq. momentum, Eq. energy).
//
// One workgroup per (cell, chunk of TI particles): the chunk's particles i
// are held in registers, with one or more threads per particle (a chunk may also
// hold the particles of up to four sparse cells along x, with the cells around all
// of them as its neighbourhood). The workgroup walks the candidates j of the
// surrounding cells as one flattened index space and queues those whose
// distance to the chunk's bounding box is below the largest support radius (a
// conservative prune: every operation of the box distance is monotone in the
// same inputs as the pair test, so no accepted pair is ever dropped). The
// global loads of a window of rounds are issued before the first one is used.
//
// The queue is taken in LDS batches: the fields of a batch's candidates are
// loaded densely, then every wave runs two phases over its particles: (A) the
// support prefilter on the matrix cores, whose signs become bit masks and
// these the particles' lists of accepted candidates in LDS, and (B) the exact
// FP32 support test and the kernel sums over the lists only, so the pair
// arithmetic runs on accepted pairs instead of on every candidate. The
// partial sums of a particle are combined in a fixed tree: results are
// bit-identical run to run.
//
// What bounds the loops is vector issue (87 % of the cycles at 64x1 on the
// 128^3 lattice): the kernel sums take about half of it, the gather and its
// tables a quarter, tests and lists the rest. Against the version that tested
// with vector instructions, one candidate per lane and instruction, and kept
// gather state in registers across the pair phase (us, density / force):
//   128^3 lattice, 64 per cell   64x1  358 / 558 -> 342 / 539
//                                32x2  386 / 727 -> 388 / 668
//   0.88M lattice, 12 per cell   64x1  539 / 957 -> 315 / 516
//                                16x4  329 / 610 -> 306 / 510
//   clustered 1.5M, uneven       64x1  1286 / 2327 -> 728 / 1220
//                                32x2  883 / 1628 -> 714 / 1184
//   clustered 18170, 64x2              52 / 92   ->  50 / 100
// A cell that fills its tile gains least: its time is the kernel sums'. Launches
// of fewer chunks than the chip holds take the time of their longest chunk, most
// of it the sums over dense groups in one wave; there the queue's second round of
// loads and its barriers show, and the last line is the one kind of set found
// (a few tens of thousands of particles, uneven, 64x2) that lost time.
//
// The loaders (SoA views in compile-time or run-time storage formats, or
// AoS records) are the only difference between the SoA kernels and the
// plain-AoS kernels.
#pragma once
#include <cmath>
#include <type_traits>

#include "sph_device.h"

namespace sph {
namespace pairk {

// --------------------------------------------------------------------------
// Data sources
// --------------------------------------------------------------------------
// Element k of a stored array: format DT fixed at compile time, or taken
// from rt when DT < 0. A load is split from the arithmetic on its value, so
// that a phase issues the loads of several candidates before it waits for the
// first.
template <int DT>
struct Fmt {
  using Raw = std::conditional_t<DT == DT_F16 || DT == DT_BF16, uint16_t, float>;
  __device__ __forceinline__ static Raw load(const void* p, int rt, int64_t k) {
    if constexpr (DT < 0) return load_q(p, rt, k, 1.0f);
    else return static_cast<const Raw*>(p)[k];
  }
  __device__ __forceinline__ static float get(Raw v, float scale) {
    if constexpr (DT == DT_F16) return f16_bits_to_f32(v) * scale;
    else if constexpr (DT == DT_BF16) return bf16_bits_to_f32(v) * scale;
    else return v * scale;
  }
};

// Origin c / n_c of a cell per axis in FP64, where a source derives offsets
// from absolute positions: divided once per neighbour cell of a chunk, not
// once per candidate
struct CellOrigin {
  double x, y, z;
  __device__ __forceinline__ CellOrigin() = default;
  __device__ __forceinline__ CellOrigin(int cx, int cy, int cz, int n_c)
      : x((double)cx / (double)n_c), y((double)cy / (double)n_c), z((double)cz / (double)n_c) {}
};
struct NoOrigin {
  __device__ __forceinline__ NoOrigin() = default;
  __device__ __forceinline__ NoOrigin(int, int, int, int) {}
};

template <int PT, int VT, int MT>
struct SoaSrc {
  const void* off[3];
  const uint8_t* anc;     // anchor sub-cell codes (anchor >= SPH_ANCHOR_SUB(1))
  float anc_step;         // sub-cell side s 2^-b of the anchors
  int anchor;             // SPH_ANCHOR_CORNER or SPH_ANCHOR_SUB(b)
  const void* vq[3];
  const void* m;
  const void* h;
  const void* u;
  int pos_dt, vel_dt, mhu_dt;
  float lm, lh, lu;
  const float *rho, *f, *P, *c;
  float *o_rho, *o_wcount, *o_rho_dh, *o_f, *o_P, *o_c;
  int32_t* o_nngb;
  float *o_ax, *o_ay, *o_az, *o_du, *o_vsig;
  int32_t* o_nforce;

  using Origin = NoOrigin;
  struct Pos {
    typename Fmt<PT>::Raw x, y, z;
    uint32_t code;
  };
  struct Vel {
    typename Fmt<VT>::Raw x, y, z;
  };
  using Mhu = typename Fmt<MT>::Raw;
  __device__ __forceinline__ Pos load_pos(int k) const {
    Pos r;
    r.x = Fmt<PT>::load(off[0], pos_dt, k);
    r.y = Fmt<PT>::load(off[1], pos_dt, k);
    r.z = Fmt<PT>::load(off[2], pos_dt, k);
    r.code = 0u;
    if (anchor >= SPH_ANCHOR_SUB(1)) r.code = anc[k];   // uniform over the launch
    return r;
  }
  __device__ __forceinline__ Vel load_vel(int k) const {
    Vel r;
    r.x = Fmt<VT>::load(vq[0], vel_dt, k);
    r.y = Fmt<VT>::load(vq[1], vel_dt, k);
    r.z = Fmt<VT>::load(vq[2], vel_dt, k);
    return r;
  }
  __device__ __forceinline__ Mhu load_m(int k) const { return Fmt<MT>::load(m, mhu_dt, k); }
  __device__ __forceinline__ Mhu load_h(int k) const { return Fmt<MT>::load(h, mhu_dt, k); }
  // position relative to the cell corner: the stored offset plus its anchor
  // (the cell's origin is not needed)
  __device__ __forceinline__ void pos(const Pos& r, const Origin&, float& x, float& y,
                                      float& z) const {
    x = Fmt<PT>::get(r.x, 1.0f);
    y = Fmt<PT>::get(r.y, 1.0f);
    z = Fmt<PT>::get(r.z, 1.0f);
    if (anchor != SPH_ANCHOR_CORNER) {          // uniform over the launch
      const uint32_t c = r.code;
      x = __builtin_fmaf((float)(c & 3u) + 0.5f, anc_step, x);
      y = __builtin_fmaf((float)((c >> 2) & 3u) + 0.5f, anc_step, y);
      z = __builtin_fmaf((float)((c >> 4) & 3u) + 0.5f, anc_step, z);
    }
  }
  __device__ __forceinline__ void vel(const Vel& r, float& x, float& y, float& z) const {
    x = Fmt<VT>::get(r.x, 1.0f);
    y = Fmt<VT>::get(r.y, 1.0f);
    z = Fmt<VT>::get(r.z, 1.0f);
  }
  __device__ __forceinline__ float mass(Mhu r) const { return Fmt<MT>::get(r, lm); }
  __device__ __forceinline__ float hsml(Mhu r) const { return Fmt<MT>::get(r, lh); }
  __device__ __forceinline__ float uint(int k) const {
    return Fmt<MT>::get(Fmt<MT>::load(u, mhu_dt, k), lu);
  }
  __device__ __forceinline__ void dens_in(int k, float& r, float& ff, float& p,
                                          float& cs) const {
    r = rho[k];
    ff = f[k];
    p = P[k];
    cs = c[k];
  }
  __device__ __forceinline__ void dens_out(int k, float r, float wc, float dh, float ff, float p,
                                           float cs, int nn) const {
    o_rho[k] = r;
    o_wcount[k] = wc;
    o_rho_dh[k] = dh;
    o_f[k] = ff;
    o_P[k] = p;
    o_c[k] = cs;
    o_nngb[k] = nn;
  }
  __device__ __forceinline__ void force_out(int k, float ax, float ay, float az, float du,
                                            float vs, int nf) const {
    o_ax[k] = ax;
    o_ay[k] = ay;
    o_az[k] = az;
    o_du[k] = du;
    o_vsig[k] = vs;
    if (o_nforce) o_nforce[k] = nf;
  }
};

struct AosSrc {
  char* base;
  AosLayout L;
  const int32_t* perm;

  __device__ __forceinline__ char* rec(int k) const {
    return base + (size_t)perm[k] * L.stride;
  }
  using Origin = CellOrigin;
  struct Pos {
    double x, y, z;
  };
  struct Vel {
    float x, y, z;
  };
  using Mhu = float;
  __device__ __forceinline__ Pos load_pos(int k) const {
    const double* xp = reinterpret_cast<const double*>(rec(k) + L.off[SPH_A_X]);
    return {xp[0], xp[1], xp[2]};
  }
  __device__ __forceinline__ Vel load_vel(int k) const {
    const char* r = rec(k);
    return {rec_load32(r, L.off[SPH_A_V], L.dt[SPH_A_V], 0),
            rec_load32(r, L.off[SPH_A_V], L.dt[SPH_A_V], 1),
            rec_load32(r, L.off[SPH_A_V], L.dt[SPH_A_V], 2)};
  }
  __device__ __forceinline__ Mhu load_m(int k) const {
    return rec_load32(rec(k), L.off[SPH_A_M], L.dt[SPH_A_M]);
  }
  __device__ __forceinline__ Mhu load_h(int k) const {
    return rec_load32(rec(k), L.off[SPH_A_H], L.dt[SPH_A_H]);
  }
  // FP64 position less its cell's origin, rounded once (cell_offset)
  __device__ __forceinline__ void pos(const Pos& r, const Origin& o, float& x, float& y,
                                      float& z) const {
    x = (float)(wrap01(r.x) - o.x);
    y = (float)(wrap01(r.y) - o.y);
    z = (float)(wrap01(r.z) - o.z);
  }
  __device__ __forceinline__ void vel(const Vel& r, float& x, float& y, float& z) const {
    x = r.x;
    y = r.y;
    z = r.z;
  }
  __device__ __forceinline__ float mass(Mhu r) const { return r; }
  __device__ __forceinline__ float hsml(Mhu r) const { return r; }
  __device__ __forceinline__ float uint(int k) const {
    return rec_load32(rec(k), L.off[SPH_A_U], L.dt[SPH_A_U]);
  }
  __device__ __forceinline__ void dens_in(int k, float& rr, float& ff, float& p,
                                          float& cs) const {
    const char* r = rec(k);
    rr = rec_load32(r, L.off[SPH_A_RHO], L.dt[SPH_A_RHO]);
    ff = rec_load32(r, L.off[SPH_A_F], L.dt[SPH_A_F]);
    p = rec_load32(r, L.off[SPH_A_P], L.dt[SPH_A_P]);
    cs = rec_load32(r, L.off[SPH_A_C], L.dt[SPH_A_C]);
  }
  __device__ __forceinline__ void dens_out(int k, float rr, float wc, float dh, float ff,
                                           float p, float cs, int nn) const {
    char* r = rec(k);
    rec_store32(r, L.off[SPH_A_RHO], L.dt[SPH_A_RHO], rr);
    rec_store32(r, L.off[SPH_A_WCOUNT], L.dt[SPH_A_WCOUNT], wc);
    rec_store32(r, L.off[SPH_A_RHO_DH], L.dt[SPH_A_RHO_DH], dh);
    rec_store32(r, L.off[SPH_A_F], L.dt[SPH_A_F], ff);
    rec_store32(r, L.off[SPH_A_P], L.dt[SPH_A_P], p);
    rec_store32(r, L.off[SPH_A_C], L.dt[SPH_A_C], cs);
    rec_store_i32(r, L.off[SPH_A_NNGB], nn);
  }
  __device__ __forceinline__ void force_out(int k, float ax, float ay, float az, float du,
                                            float vs, int nf) const {
    char* r = rec(k);
    rec_store32(r, L.off[SPH_A_A], L.dt[SPH_A_A], ax, 0);
    rec_store32(r, L.off[SPH_A_A], L.dt[SPH_A_A], ay, 1);
    rec_store32(r, L.off[SPH_A_A], L.dt[SPH_A_A], az, 2);
    rec_store32(r, L.off[SPH_A_DU], L.dt[SPH_A_DU], du);
    rec_store32(r, L.off[SPH_A_VSIG], L.dt[SPH_A_VSIG], vs);
    rec_store_i32(r, L.off[SPH_A_NFORCE], nf);
  }
};

// The data source (a kernel's first argument) read again from the kernel
// arguments: its pointers then need registers only in the phase that uses
// them (kept from the kernel's start they overflow the scalar registers, and
// every use of a spilled one costs vector instructions).
template <class Src>
__device__ __forceinline__ Src kernel_src() {
  auto p = (const __attribute__((address_space(4))) Src*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Src*)p;
}

// A value the compiler must not carry derived quantities of across this
// point: what a phase computes from the thread index is cheaper computed
// again than kept in registers through the other phases.
__device__ __forceinline__ int again(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A value that is the same in every lane, in a scalar register
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

template <class Src>
struct PosH {
  typename Src::Pos pos;
  typename Src::Mhu h;
};

// Slot indices read from the cell table are clamped to [0, n], so a
// corrupted table can never send a load outside the particle arrays.
__device__ __forceinline__ int clamp_slot(int v, int n) { return min(max(v, 0), n); }

// Spread consecutive workgroups over the 8 XCDs in contiguous ranges: block b
// runs on XCD b % 8, so logical work item (b % 8) * per + b / 8 gives each
// XCD a contiguous slab of cells (shared neighbour cells stay in one L2).
__device__ __forceinline__ int xcd_remap(int b, int G) {
  int per = G >> 3;
  if (b >= (per << 3)) return b;
  return (b & 7) * per + (b >> 3);
}

// The K lanes of a particle lie P = 64 / K lanes apart in one wave (lane =
// kk P + particle): the layout in which the matrix instruction of the
// prefilter leaves the results of a particle.
template <int O>
__device__ __forceinline__ int lane_xor_i(int v) {
  if constexpr (O == 32) {
    const auto p = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return __lane_id() & 32 ? (int)p[0] : (int)p[1];
  } else if constexpr (O == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return __lane_id() & 16 ? (int)p[0] : (int)p[1];
  } else {
    return __shfl_xor(v, O);
  }
}
// Integers in the order of the floats (NaN excluded), and back
__device__ __forceinline__ int order_key(float v) {
  const int b = __float_as_int(v);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_float(int k) {
  return __int_as_float(k ^ ((k >> 31) & 0x7fffffff));
}

// Maximum over a wave, uniform: rotations inside the rows of 16 lanes (operand
// moves of the maximum itself), then row and half swaps. On integers: fmaxf on
// values moved between lanes canonicalises both operands first, which made the
// chunk box 150 vector instructions instead of 90.
template <int CTRL>
__device__ __forceinline__ int dpp_max(int v) {
  return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ int wave_max(int v) {
  v = dpp_max<0x128>(v);     // row_ror:8, 4, 2, 1
  v = dpp_max<0x124>(v);
  v = dpp_max<0x122>(v);
  v = dpp_max<0x121>(v);
  const auto p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  v = max((int)p[0], (int)p[1]);
  const auto q = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return __builtin_amdgcn_readfirstlane(max((int)q[0], (int)q[1]));
}

// Inclusive prefix sum over a wave: shifts inside the rows of 16 lanes, then
// the last lane of each row or half added to the rows after it
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, ROWS == 0xf);
}
__device__ __forceinline__ int row_scan(int v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  return dpp_add<0x118, 0xf>(v);
}
__device__ __forceinline__ int wave_scan(int v) {
  v = row_scan(v);
  v = dpp_add<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

// Position shift of the cell d cells away along an axis, relative to the
// chunk's cell: d * s in FP32 (-s, 0, s exactly), one expression wherever a
// position is shifted by d cells
__device__ __forceinline__ float cell_shift(int d, float s) { return (float)d * s; }

__device__ __forceinline__ float box_dist2(float x, float y, float z, float lox, float loy,
                                           float loz, float hix, float hiy, float hiz) {
#pragma clang fp contract(off)
  float bx = fmaxf(fmaxf(lox - x, x - hix), 0.0f);
  float by = fmaxf(fmaxf(loy - y, y - hiy), 0.0f);
  float bz = fmaxf(fmaxf(loz - z, z - hiz), 0.0f);
  float xx = bx * bx;
  return __builtin_fmaf(bz, bz, __builtin_fmaf(by, by, xx));
}

// Chunk bounding box of the valid particles and the largest H^2
struct ChunkBox {
  float lox, loy, loz, hix, hiy, hiz, h2max;
};

template <int NT>
__device__ __forceinline__ ChunkBox chunk_box(bool vi, float xi, float yi, float zi, float H2,
                                              int* red) {
  // the seven block maxima (minima as maxima of negated values) in one pass:
  // per value a wave maximum, then the wave results; two barriers. NaNs count
  // as absent.
  constexpr int NW = NT / 64;
  const float inf = __builtin_inff();
  const bool vx = vi && xi == xi, vy = vi && yi == yi, vz = vi && zi == zi;
  const float v[7] = {vx ? -xi : -inf, vy ? -yi : -inf, vz ? -zi : -inf, vx ? xi : -inf,
                      vy ? yi : -inf,  vz ? zi : -inf,  H2 == H2 ? H2 : -inf};
  int r[7];
#pragma unroll
  for (int k = 0; k < 7; ++k) r[k] = wave_max(order_key(v[k]));
  if constexpr (NW == 1) {
    (void)red;
    __syncthreads();
  } else {
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < 7; ++k) red[k * NW + wave] = r[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      r[k] = red[k * NW];
#pragma unroll
      for (int w = 1; w < NW; ++w) r[k] = max(r[k], red[k * NW + w]);
      r[k] = __builtin_amdgcn_readfirstlane(r[k]);
    }
    __syncthreads();
  }
  ChunkBox b;
  b.lox = -key_float(r[0]);
  b.loy = -key_float(r[1]);
  b.loz = -key_float(r[2]);
  b.hix = key_float(r[3]);
  b.hiy = key_float(r[4]);
  b.hiz = key_float(r[5]);
  b.h2max = key_float(r[6]);
  return b;
}

// Raises the status flag where a particle of the chunk has a support above the
// cell side: one thread, and only where the flag is not up yet. Smoothing
// lengths rounded up to their storage format can exceed the cell side in most
// chunks at once, and what such a launch then takes is the atomics on the one
// word, which are served one after the other: 113183 particles in FP16 at 64x4,
// an atomic per wave 530 us, this 298; in FP32, no flag to raise, 288.
__device__ __forceinline__ void flag_support(const CellsDev& cd, const ChunkBox& b, float s32) {
  if (threadIdx.x != 0 || !cd.status || !(b.h2max > s32 * s32)) return;
  if (!(__hip_atomic_load(cd.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
        SPH_FLAG_H_TOO_LARGE))
    atomicOr(cd.status, SPH_FLAG_H_TOO_LARGE);
}

// --------------------------------------------------------------------------
// Neighbour cells of a chunk's cells (m cells along x from the chunk's first
// cell, m = 1 unless the work list merges sparse cells): ids, the offsets
// (dx, dy, dz) of each from the chunk's first cell (its frame is shifted by
// cell_shift(delta, s) per axis), the support-radius bound of each (gamma_k * max h * (1 + 2^-8), covering
// storage rounding of h; the cell side when no bound table is given), and
// each cell's slot range. build_nbr issues all of its loads at once and
// ends without a barrier: the caller's next barrier (the chunk box's)
// publishes the table, so the chunk's own loads overlap these.
// --------------------------------------------------------------------------
constexpr int kMaxNbr = 9 * (kMaxMerge + 2);   // neighbour cells of a merged chunk
template <class Origin>
struct NbrCells {
  int cell[kMaxNbr];
  float hb[kMaxNbr];
  int st[kMaxNbr], cnt[kMaxNbr];   // first slot and particle count of each cell
  int d[kMaxNbr];   // offsets: (dx + 1) | (dy + 1) << 8 | (dz + 1) << 16
  float hbmax;      // largest hb over the nq cells
  int nq;           // neighbour cells: 9 (m + 2)
  Origin org[std::is_same_v<Origin, NoOrigin> ? 1 : kMaxNbr];

  __device__ __forceinline__ const Origin& origin(int q) const {
    return org[std::is_same_v<Origin, NoOrigin> ? 0 : q];
  }
  // shift of cell q's positions into the chunk's frame: d * s per axis as
  // cell_shift rounds it (fma(d + 1, s, -s) is d * s rounded once)
  __device__ __forceinline__ void shift(int q, float s, float& sx, float& sy, float& sz) const {
    const unsigned v = d[q];
    sx = __builtin_fmaf((float)(v & 0xffu), s, -s);
    sy = __builtin_fmaf((float)((v >> 8) & 0xffu), s, -s);
    sz = __builtin_fmaf((float)((v >> 16) & 0xffu), s, -s);
  }
  // whether q is one of the chunk's own m cells, and not a periodic image of
  // one (the cells around m > n_c - 2 cells hold images of them)
  __device__ __forceinline__ bool own(int q, int m) const {
    return (d[q] >> 8) == 0x0101 && (d[q] & 0xff) <= m && (d[q] & 0xff) != 0;
  }
  __device__ __forceinline__ void offsets(int q, int& dx, int& dy, int& dz) const {
    const int v = d[q];
    dx = (v & 0xff) - 1;
    dy = ((v >> 8) & 0xff) - 1;
    dz = (v >> 16) - 1;
  }
};

// Neighbour entry q of a chunk of w - 2 cells along x (w = 3 for a single
// cell): offsets dx in [-1, w - 2], dy, dz in [-1, 1], q = (dx + 1) +
// w ((dy + 1) + 3 (dz + 1)).
template <bool BMAX, class Origin>
__device__ __forceinline__ void build_nbr(NbrCells<Origin>& T, const CellsDev& cd, int cx, int cy,
                                          int cz, int m, float s32, float gk) {
  const int tid = again(threadIdx.x);
  if (tid >= 64) return;   // first wave (kMaxNbr <= 64)
  const int w = m + 2, nq = 9 * w, n_c = cd.n_c;
  float hbv = 0.0f;
  if (tid == 0) T.nq = nq;
  if (tid < nq) {
    // tid / w for tid < 64, w <= 6 through the FP32 reciprocal (v_rcp, 1 ulp):
    // exact, (tid + 1/2) / w lies at least 1 / 12 from an integer
    const int row = w == 3 ? tid / 3
                           : (int)(((float)tid + 0.5f) * __builtin_amdgcn_rcpf((float)w));
    const int dz = row / 3 - 1, dy = row - 3 * (dz + 1) - 1, dx = tid - w * row - 1;
    int nx = cx + dx, ny = cy + dy, nz = cz + dz;
    nx += (nx < 0) ? n_c : ((nx >= n_c) ? -n_c : 0);
    ny += (ny < 0) ? n_c : ((ny >= n_c) ? -n_c : 0);
    nz += (nz < 0) ? n_c : ((nz >= n_c) ? -n_c : 0);
    const int cn = nx + n_c * (ny + n_c * nz);
    const int a = clamp_slot(cd.start[cn], cd.n);
    const int b = clamp_slot(cd.start[cn + 1], cd.n);
    hbv = cd.hmax ? gk * cd.hmax[cn] * (1.0f + 0x1p-8f) : s32;
    T.d[tid] = (dx + 1) | ((dy + 1) << 8) | ((dz + 1) << 16);
    T.cell[tid] = cn;
    if constexpr (!std::is_same_v<Origin, NoOrigin>) T.org[tid] = Origin(nx, ny, nz, n_c);
    T.hb[tid] = hbv;
    T.st[tid] = a;
    T.cnt[tid] = max(b - a, 0);
  }
  if constexpr (BMAX) {
    const int mx = wave_max(__float_as_int(hbv));   // hbv >= 0: ordered as integers
    if (tid == 0) T.hbmax = __int_as_float(mx);
  }
}
static_assert(kMaxNbr <= 64, "the neighbour table is reduced by one wave");

// Block-wide exclusive scan of an int in thread order: returns this
// thread's prefix and sets tb to the block total. One barrier: the caller
// must pass another barrier before `lds` (NT / 64 ints) is written again.
template <int NT>
__device__ __forceinline__ int block_scan(int b, int& tb, int* lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ib = wave_scan(b);
  if constexpr (NW == 1) {
    tb = __builtin_amdgcn_readlane(ib, 63);
    __syncthreads();
    return ib - b;
  }
  if (lane == 63) lds[wave] = ib;
  __syncthreads();
  int pb = 0;
  tb = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int wb = lds[w];
    pb += (w < wave) ? wb : 0;
    tb += wb;
  }
  return pb + ib - b;
}

// Block-wide exclusive scan, in thread order, of a flag (0/1) and of an
// int; returns the block totals. One barrier: the caller must pass another
// barrier before `lds` (2 NT / 64 ints) is written again.
template <int NT>
__device__ __forceinline__ void block_scan2(bool flag, int b, int& ea, int& eb, int& ta, int& tb,
                                            int* lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t bal = __ballot(flag);
  const int xa = __popcll(bal & lanemask_lt());
  const int ib = wave_scan(b);
  if constexpr (NW == 1) {
    ta = __popcll(bal);
    tb = __builtin_amdgcn_readlane(ib, 63);
    ea = xa;
    eb = ib - b;
    __syncthreads();
    return;
  }
  if (lane == 63) {
    lds[wave] = __popcll(bal);
    lds[NW + wave] = ib;
  }
  __syncthreads();
  int pa = 0, pb = 0;
  ta = 0;
  tb = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int wa = lds[w], wb = lds[NW + w];
    pa += (w < wave) ? wa : 0;
    pb += (w < wave) ? wb : 0;
    ta += wa;
    tb += wb;
  }
  ea = pa + xa;
  eb = pb + ib - b;
}

// Position of each flagged thread when the flagged threads are ordered by
// class (0..3) and, within a class, by thread. One barrier: the caller must
// pass another barrier before `lds` (2 NT / 64 ints: a wave's four class
// counts, at most 64 each, as 16-bit halves) is written again.
template <int NT>
__device__ __forceinline__ int class_rank(bool flag, int cls, int* lds) {
  constexpr int NW = NT / 64;
  const int wave = threadIdx.x >> 6;
  uint64_t mine = 0;
  int cnt[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint64_t bal = __ballot(flag && cls == c);
    cnt[c] = __popcll(bal);
    mine = (cls == c) ? bal : mine;
  }
  if ((threadIdx.x & 63) == 0) {
    lds[wave] = cnt[0] | (cnt[1] << 16);
    lds[NW + wave] = cnt[2] | (cnt[3] << 16);
  }
  __syncthreads();
  int off = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int a = lds[w], b = lds[NW + w];
    const int v[4] = {a & 0xffff, a >> 16, b & 0xffff, b >> 16};
#pragma unroll
    for (int c = 0; c < 4; ++c) off += (c < cls || (c == cls && w < wave)) ? v[c] : 0;
  }
  return off + __popcll(mine & lanemask_lt());
}


// Range table of one batch of candidate ranges, and, per neighbour cell q, its
// entries: the whole cell, or its sub-cells inside the query box. wbits marks
// the last candidate of each range inside a gather window (KR rounds
// of NT flattened candidates), in two buffers by window parity: a buffer is
// zero again before the window after next marks it. An entry holds the
// range's first slot less its first flattened index (a candidate's slot is
// its flattened index plus this) and its cell's neighbour index.
template <int NT, int KR>
struct RangeTab {
  static constexpr int kWin = KR * NT / 64;   // 64-candidate words of a window
  uint2 wbits[2][kWin];
  int2 ent[NT];
  int scan[2 * (NT / 64)];
  int total;
  int split;                    // whether some cell is taken by its sub-cells
  int qpre[kMaxNbr + 1];        // prefix of the entry counts of the cells
  unsigned char qw[kMaxNbr];    // 1: whole cell, 0: sub-cells qr
  unsigned char qny[kMaxNbr];   // sub-cell range width along y
  alignas(4) unsigned char qr[kMaxNbr][4];   // local sub-cell range: x0, y0, z0, width nx

  __device__ __forceinline__ void clear() {
    const int t = threadIdx.x;
    if (t < 2 * kWin) wbits[t & 1][t >> 1] = make_uint2(0u, 0u);
  }
};

// A neighbour cell is split into its R^3 sub-cells only when it holds more
// than kSplitFactor * R^3 particles: below that, one range for the whole
// cell costs less than the table work of its sub-cells.
constexpr int kSplitFactor = 2;

// The candidate ranges of a chunk: for each of the nq neighbour cells q
// with bound(q) > 0, the sub-cells (R = 2^sub_bits per axis) of q whose
// boxes lie within bound(q) of the chunk box [lo, hi], or the whole of q
// (a superset) when q is sparse. Entries are processed in
// batches of at most NT: for each batch, `batch(tab, last)` gathers the
// particles of the batch's ranges. The per-cell index ranges are widened by
// 2^-7 of a sub-cell (twice the 2^-8 margin of the per-entry box test, which
// covers the rounding of stored offsets), so every entry that test keeps is
// enumerated.
// When a batch's ranges hold more than `spread` candidates (more than one
// LDS batch of the caller), they are placed class by class. The class of a
// sub-cell at sub-cell coordinates (gx, gy, gz) from the chunk's cell is its
// parity pattern (gx, gy, gz) & 1 taken together with the complementary
// pattern, ((gx ^ gz) & 1) | ((gy ^ gz) & 1) << 1 (a whole cell: the same of
// its cell offsets). Each class is spread evenly over the neighbourhood, so
// when the staged candidates fill several LDS batches every batch holds a
// similar share of each particle's neighbours, and the per-lane lists of a
// batch are of similar length (in enumeration order a batch covers one side
// of the neighbourhood, and particles on that side hold most of its pairs).
// `batch(end, last)` is called with each thread's range end (the flattened
// index after its last candidate, 0 for none). `pre` is NT ints of scratch.
template <int NT, int KR, class Origin, class Bound, class Batch>
__device__ __forceinline__ void for_sub_cells(const CellsDev& cd, const NbrCells<Origin>& T,
                                              RangeTab<NT, KR>& tab, int* pre, float s32,
                                              const ChunkBox& bx, int spread, Bound bound,
                                              Batch batch) {
  const int sb = cd.sub_bits, R = 1 << sb;
  const int tid = again(threadIdx.x);
  const int nq = T.nq;
  // Places this block's entries (one per thread where ok) in the table
  auto place = [&](bool ok, int st, int cnt, int q, int cls) {
    int e_idx, e_pre, ntab, total;
    block_scan2<NT>(ok, ok ? cnt : 0, e_idx, e_pre, ntab, total, tab.scan);
    int end = ok ? e_pre + cnt : 0;
    if (total > spread) {   // uniform: more than one LDS batch, order by class
      __syncthreads();
      e_idx = class_rank<NT>(ok, cls, tab.scan);
      if (ok) pre[e_idx] = cnt;
      __syncthreads();
      const int c_t = tid < ntab ? pre[tid] : 0;
      const int p_t = block_scan<NT>(c_t, total, tab.scan);
      end = tid < ntab ? p_t + c_t : 0;
      if (tid < ntab) pre[tid] = p_t;
      __syncthreads();
      if (ok) e_pre = pre[e_idx];
    }
    if (ok) tab.ent[e_idx] = make_int2(st - e_pre, q);
    if (tid == 0) tab.total = total;
    __syncthreads();
    return end;
  };
  int n = 0;          // entries of neighbour cell tid
  bool part = false;  // ... which are sub-cells of it
  if (tid < nq) {
    const int q = tid;
    int dx, dy, dz;
    T.offsets(q, dx, dy, dz);
    const float bq = bound(q);
    const int cnt = T.cnt[q];
    if (bq > 0.0f && cnt > 0) {
      const float inv = (float)R / s32;
      auto lo_i = [&](float v, int d) {
        return max((int)floorf((v - bq) * inv - 0x1p-7f) - d * R, 0);
      };
      auto hi_i = [&](float v, int d) {
        return min((int)floorf((v + bq) * inv + 0x1p-7f) - d * R, R - 1);
      };
      const int x0 = lo_i(bx.lox, dx), x1 = hi_i(bx.hix, dx);
      const int y0 = lo_i(bx.loy, dy), y1 = hi_i(bx.hiy, dy);
      const int z0 = lo_i(bx.loz, dz), z1 = hi_i(bx.hiz, dz);
      if (x0 <= x1 && y0 <= y1 && z0 <= z1) {
        part = sb > 0 && cnt > kSplitFactor * R * R * R;
        n = 1;
        if (part) {
          const int nx = x1 - x0 + 1;
          n = nx * (y1 - y0 + 1) * (z1 - z0 + 1);
          tab.qny[q] = (unsigned char)(y1 - y0 + 1);
          unsigned char* r = tab.qr[q];
          r[0] = (unsigned char)x0;
          r[1] = (unsigned char)y0;
          r[2] = (unsigned char)z0;
          r[3] = (unsigned char)nx;
        }
      }
      tab.qw[q] = part ? 0 : 1;
    }
  }
  bool split;
  if constexpr (NT == 64) {
    split = __any(part);
  } else {
    if (tid < 64 && __any(part) && tid == 0) tab.split = 1;
    else if (tid == 0) tab.split = 0;
    __syncthreads();
    split = __builtin_amdgcn_readfirstlane(tab.split) != 0;
  }
  int NQ = nq;
  if (split) {
    if (tid < 64) {     // first wave (nq <= 64): prefix of the entry counts
      const int inc = wave_scan(n);
      if (tid <= nq) tab.qpre[tid] = inc - n;   // lane nq holds the total
    }
    __syncthreads();
    NQ = __builtin_amdgcn_readfirstlane(tab.qpre[nq]);
  }
  const float ss = s32 / (float)R;
  for (int b0 = 0;; b0 += NT) {     // one call site of `batch`: it is large code
    const int t = b0 + tid;
    bool ok = split ? t < NQ : n > 0;
    int st = 0, cnt = 0, q = tid, cls = 0, dx = 0, dy = 0, dz = 0;
    if (ok) {
      if (split) {
        int lo = 0, hi = nq - 1;   // last q with qpre[q] <= t
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (tab.qpre[mid] <= t) lo = mid;
          else hi = mid - 1;
        }
        q = lo;
      }                            // else every entry is a whole cell, entry t is cell t
      T.offsets(q, dx, dy, dz);
      float bx0, bx1, by0, by1, bz0, bz1;
      if (!split || tab.qw[q]) {
        const float mg = s32 * 0x1p-8f;       // rounding margin of stored offsets
        bx0 = dx * s32 - mg, bx1 = (dx + 1) * s32 + mg;
        by0 = dy * s32 - mg, by1 = (dy + 1) * s32 + mg;
        bz0 = dz * s32 - mg, bz1 = (dz + 1) * s32 + mg;
        st = T.st[q];
        cnt = T.cnt[q];
        cls = ((dx ^ dz) & 1) | (((dy ^ dz) & 1) << 1);
      } else {
        const int e = t - tab.qpre[q];
        const uchar4 r = *reinterpret_cast<const uchar4*>(tab.qr[q]);
        // e = ex + nx (ey + ny ez), split through FP32 reciprocals (v_rcp,
        // 1 ulp): exact, as e < 2^9 and (e + 1/2) / w lies at least
        // 1 / (2 w) >= 2^-7 from an integer
        const int nx = r.w, nxy = nx * tab.qny[q];
        const int ez = (int)(((float)e + 0.5f) * __builtin_amdgcn_rcpf((float)nxy));
        const int rem = e - ez * nxy;
        const int ey = (int)(((float)rem + 0.5f) * __builtin_amdgcn_rcpf((float)nx));
        const int sx = r.x + (rem - ey * nx), sy = r.y + ey, sz = r.z + ez;
        const float mg = ss * 0x1p-8f;
        const int gx = dx * R + sx, gy = dy * R + sy, gz = dz * R + sz;
        cls = ((gx ^ gz) & 1) | (((gy ^ gz) & 1) << 1);
        bx0 = gx * ss - mg, bx1 = (gx + 1) * ss + mg;
        by0 = gy * ss - mg, by1 = (gy + 1) * ss + mg;
        bz0 = gz * ss - mg, bz1 = (gz + 1) * ss + mg;
        int m = 0;
        for (int b = 0; b < sb; ++b)
          m |= (((sx >> b) & 1) << (3 * b)) | (((sy >> b) & 1) << (3 * b + 1)) |
               (((sz >> b) & 1) << (3 * b + 2));
        const int key = (T.cell[q] << (3 * sb)) + m;
        st = clamp_slot(cd.sub_start[key], cd.n);
        cnt = max(clamp_slot(cd.sub_start[key + 1], cd.n) - st, 0);
      }
      const float ex = fmaxf(fmaxf(bx0 - bx.hix, bx.lox - bx1), 0.0f);
      const float ey = fmaxf(fmaxf(by0 - bx.hiy, bx.loy - by1), 0.0f);
      const float ez = fmaxf(fmaxf(bz0 - bx.hiz, bx.loz - bz1), 0.0f);
      const float bq = bound(q);     // 0: not a neighbour here
      ok = cnt > 0 && ex * ex + ey * ey + ez * ez < bq * bq * (1.0f + 0x1p-10f);
    }
    const bool last = b0 + NT >= NQ;
    batch(place(ok, st, cnt, q, cls), last);
    __syncthreads();
    if (last) break;
  }
}

constexpr int kMfmaTile = 16;    // candidates per matrix instruction
// Order of summation. A tile of TI particles and K lanes per particle stands
// for NT = TI K sums per chunk: candidate number x of a batch of the chunk
// belongs to lane x mod K of every particle, each lane adds up its accepted
// candidates in order, and the K lanes are added in a fixed tree. Batches are
// counted in rounds of NT flattened candidates: a round that would take the
// batch past batch_limit starts the next one at number 0. Results are defined
// by this order alone, bit for bit, not by which threads compute the terms,
// which loop the candidates are tested in, or how they are staged.
constexpr int batch_limit(int lists, int NT, int K) { return lists * NT - 8 * K; }

// Gathers the candidates of one table batch into the chunk's queue: those
// whose distance to the chunk box passes `keep(c)`, as slot and neighbour
// index. A window of KR rounds of NT candidates has all its loads
// in flight (`load(src, j)` the raw fields, which `get(src, raw, q, c)` turns
// into x, y, z relative to j's own cell and one more field for keep) and is compacted with one barrier, in (round, thread)
// order, so the queue is deterministic. Only the queue outlives a window:
// `flush(n)` runs the pair phase over the n queued candidates when the next
// window might not fit and at the end of the chunk's last table batch (one
// call site: the pair phase is large code, and no gather state is live in
// registers across it).
// Queue entry x belongs to lane x mod K: where a batch starts at number 0
// the entries up to the next multiple of K stay empty (kHole).
constexpr unsigned char kHole = 255;
template <int NT, int K, int KR>
struct Queue {
  static constexpr int CAP = 2 * KR * NT + (K > 1 ? KR * K : 0);   // two windows
  int slot[CAP];
  unsigned char q[CAP];     // neighbour index of its cell, or kHole
};
struct GatherState {
  int base = 0;    // queue entry of the current batch's number 0
  int num = 0;     // next number in the batch: the queue holds base + num entries
  int win = 0;     // windows so far (parity picks the buffers)
  int kept = 0;    // candidates queued for the chunk
};

template <class Src, int NT, int K, int KR, int LIMIT, class Load, class Get, class Keep,
          class Flush>
__device__ __forceinline__ void gather_batch(RangeTab<NT, KR>& tb,
                                             const NbrCells<typename Src::Origin>& T,
                                             Queue<NT, K, KR>& qu, int n, float s32, int* wtot,
                                             GatherState& gs, int my_end, bool last, Load load,
                                             Get get, Keep keep, Flush flush) {
  constexpr int NW = NT / 64, NWD = RangeTab<NT, KR>::kWin;
  const int total = __builtin_amdgcn_readfirstlane(tb.total);
  int nbefore = 0;               // ranges that end before the window
  for (int sbase = 0;;) {
    const bool done = sbase >= total;
    if (done ? last
             : gs.base + gs.num + min(KR * NT, total - sbase) + (K > 1 ? KR * K : 0) >
                   Queue<NT, K, KR>::CAP) {
      flush(gs.base + gs.num);
      gs.base = gs.num % K - gs.num;   // the batch goes on at its lane
      if constexpr (K > 1) {
        if ((int)threadIdx.x < gs.num % K) qu.q[threadIdx.x] = kHole;
      }
    }
    if (done) break;
    // A bit per window position where a range ends (ranges are non-empty, so
    // ends are distinct): candidate p belongs to the range whose number is the
    // count of ends before p, one mbcnt per 32-bit half on top of the count
    // before p's 64-candidate word.
    const Src src = kernel_src<Src>();
    const int tid = again(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    uint2* const wb = tb.wbits[gs.win & 1];
    const int p = my_end - 1 - sbase;
    if (my_end > 0 && p >= 0 && p < KR * NT)
      atomicOr(p & 32 ? &wb[p >> 6].y : &wb[p >> 6].x, 1u << (p & 31));
    __syncthreads();
    int excl = 0;                 // lane w < NWD: ends in the words before word w
    if constexpr (NW > 1) {
      const uint2 v = wb[min(lane, NWD - 1)];
      const int c = lane < NWD ? __popc(v.x) + __popc(v.y) : 0;
      const int inc = row_scan(c);
      excl = nbefore + inc - c;
      nbefore += __builtin_amdgcn_readlane(inc, NWD - 1);
    }
    decltype(load(src, 0)) raw[KR];
    int jj[KR], qq[KR];
#pragma unroll
    for (int r = 0; r < KR; ++r) {
      const int wd = r * NW + wave;
      const uint2 v = wb[wd];
      int e;
      if constexpr (NW > 1) {
        e = __builtin_amdgcn_mbcnt_hi(v.y,
                                      __builtin_amdgcn_mbcnt_lo(v.x, __shfl(excl, wd)));
      } else {
        e = __builtin_amdgcn_mbcnt_hi(v.y, __builtin_amdgcn_mbcnt_lo(v.x, nbefore));
        nbefore += __popc(v.x) + __popc(v.y);
      }
      // lanes past the last candidate repeat one: no branch between the loads.
      // The clamps give a table entry and a slot whatever the table holds.
      const int idx = min(sbase + r * NT + tid, total - 1);
      const int2 en = tb.ent[min(e, NT - 1)];
      jj[r] = min(max(idx + en.x, 0), n - 1);
      qq[r] = min(en.y & 0xff, kMaxNbr - 1);
      raw[r] = load(src, jj[r]);
    }
    bool ok[KR];
    int slot[KR], tot[KR];
    int* const wt = wtot + (gs.win & 1) * KR * NW;
#pragma unroll
    for (int r = 0; r < KR; ++r) {
      float4 c;
      float sx, sy, sz;
      get(src, raw[r], qq[r], c);
      T.shift(qq[r], s32, sx, sy, sz);
      c.x = shifted(c.x, sx);
      c.y = shifted(c.y, sy);
      c.z = shifted(c.z, sz);
      ok[r] = sbase + r * NT + tid < total && keep(c);
      const uint64_t bal = __ballot(ok[r]);
      slot[r] = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
      tot[r] = __popcll(bal);
      if (NW > 1 && lane == 0) wt[r * NW + wave] = tot[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KR; ++r) {
      if constexpr (NW > 1) {
        int sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const int t = wt[r * NW + w];
          slot[r] += (w < wave) ? t : 0;
          sum += t;
        }
        tot[r] = __builtin_amdgcn_readfirstlane(sum);
      }
      if (gs.num + tot[r] > LIMIT) {       // uniform: the next batch starts here
        const int hole = (K - gs.num % K) % K;
        if constexpr (K > 1) {
          if (tid < hole) qu.q[gs.base + gs.num + tid] = kHole;
        }
        gs.base += gs.num + hole;
        gs.num = 0;
      }
      slot[r] += gs.base + gs.num;
      gs.num += tot[r];
      gs.kept += tot[r];
    }
    if (tid < NWD) wb[tid] = make_uint2(0u, 0u);   // every lookup is done
#pragma unroll
    for (int r = 0; r < KR; ++r) {
      if (ok[r]) {
        qu.slot[slot[r]] = jj[r];
        qu.q[slot[r]] = (unsigned char)qq[r];
      }
    }
    sbase += KR * NT;
    ++gs.win;
  }
}

// Takes the n queue entries in LDS batches of at most CAP, as few as hold them
// and of even size: `fill(off, cnt, ntile)` stages entries [off, off + cnt), the
// r-th of lane k of the order at slot k CAP / K + r, and pads them to 16 KG
// ntile, an even number of matrix tiles for each of the KG groups of waves;
// `pairs(ntile)` runs the test and pair phases. Even batches keep the lists of a
// batch of similar length when the candidates come class by class. Sizes are
// even to a step of two matrix tiles per group, which pads the fewest
// candidates, or (EXACT, where `exact`) to the entry: then batches end where
// classes do, and the longest list of a wave, which its other lanes wait for, is
// shorter (force, one particle per lane, 64x1 on the 128^3 lattice: 72 -> 62
// entries a chunk, 560 -> 533 us; 140608 particles without a work list 61.3 ->
// 58.1). The density loop, whose lists cost less, gains nothing.
template <int CAP, int K, int KG, bool EXACT, class Fill, class Pairs>
__device__ __forceinline__ void for_lds_batches(int n, bool exact, Fill fill, Pairs pairs) {
  constexpr int kStep = 2 * kMfmaTile * KG;
  static_assert(CAP % kStep == 0 && CAP % K == 0, "whole steps");
  __syncthreads();     // the queue
  if constexpr (EXACT) {
    // ceil(n / parts), parts = 1 to 5, through v_rcp (1 ulp): exact, (n + parts - 1)
    // / parts + 2^-10 lies at least 2^-10 from an integer
    const int parts = (n + CAP - 1) / CAP;
    const int even = __builtin_amdgcn_readfirstlane(
        (int)((float)(n + parts - 1) * __builtin_amdgcn_rcpf((float)parts) + 0x1p-10f));
    const int unit = exact ? K : kStep;     // powers of two, multiples of K
    const int size = (even + unit - 1) & -unit;
    for (int off = 0; off < n; off += size) {
      const int cnt = min(size, n - off);
      const int ntile = (cnt + kStep - 1) / kStep * 2;
      fill(off, cnt, ntile);
      __syncthreads();
      pairs(ntile);
      __syncthreads();
    }
    return;
  }
  int steps = (n + kStep - 1) / kStep;
  int left = (steps + CAP / kStep - 1) / (CAP / kStep);     // batches left
  for (int off = 0; off < n; --left) {
    // ceil(steps / left), at most CAP / kStep: v_rcp (1 ulp) of a small count
    const int st = min(left > 1 ? __builtin_amdgcn_readfirstlane(
                                      (int)((float)(steps + left - 1) *
                                                __builtin_amdgcn_rcpf((float)left) +
                                            0x1p-10f))
                                : steps,
                       CAP / kStep);
    const int cnt = min(st * kStep, n - off);
    const int ntile = (cnt + kStep - 1) / kStep * 2;
    fill(off, cnt, ntile);
    __syncthreads();
    pairs(ntile);
    __syncthreads();
    off += cnt;
    steps -= st;
  }
}

constexpr float kFlatRatio = 1.02f;   // force: neighbour support bound^2 / chunk's largest H^2


// Candidate prefilter of phase A on the matrix cores. With p = x_i and
// q = x_j relative to the chunk's cell, r^2 = |p|^2 - 2 p.q + |q|^2: staging
// stores n2 = |q|^2 as q's fourth component, each particle has
// c = H^2 - |p|^2 + M, and a pair is accepted where
// t = n2 - 2 p.q - c < 0. That is a product of (x, y, z, n2) with
// (-2p, 1) plus the constant -c: one v_mfma_f32_16x16x4_f32 tests 16
// candidates against 16 particles in FP32, and the only vector instruction
// per test left is the one that shifts t's sign into a lane's mask. Phase B
// takes the exact FP32 support test (dist2) again on the accepted pairs, so
// the prefilter only has to accept a superset of it; M bounds the rounding of
// t, of c and of dist2. With |p|^2 <= Bi, |q|^2 <= Bj and H^2 <= Bj those
// errors add up to less than 19 * 2^-24 * (Bi + Bj); M = 2^-16 (Bi + Bj)
// leaves a factor 13. Bi, Bj follow from the chunk box: the candidates
// lie within one cell side s of it (H <= s, else the status flag is set).
__device__ __forceinline__ float prefilter_margin(const ChunkBox& b, float s) {
  const float ex = fmaxf(fabsf(b.lox), fabsf(b.hix));
  const float ey = fmaxf(fabsf(b.loy), fabsf(b.hiy));
  const float ez = fmaxf(fabsf(b.loz), fabsf(b.hiz));
  const float bi = ex * ex + ey * ey + ez * ez;
  const float bj = (ex + s) * (ex + s) + (ey + s) * (ey + s) + (ez + s) * (ez + s);
  return 0x1p-16f * (bi + bj);
}

typedef float f4v __attribute__((ext_vector_type(4)));

// Transposes a 4 x 4 matrix of (register, row of 16 lanes)
__device__ __forceinline__ void transpose4(unsigned (&w)[4]) {
  const auto p = __builtin_amdgcn_permlane16_swap(w[0], w[1], false, false);
  const auto q = __builtin_amdgcn_permlane16_swap(w[2], w[3], false, false);
  const auto u = __builtin_amdgcn_permlane32_swap(p[0], q[0], false, false);
  const auto v = __builtin_amdgcn_permlane32_swap(p[1], q[1], false, false);
  w[0] = u[0];
  w[1] = v[0];
  w[2] = u[1];
  w[3] = v[1];
}

// How a chunk's sums are laid out over the waves of a workgroup. A wave takes
// blocks of PB = 16, 32 or 64 particles for KC of the K lanes of the order of
// summation, and F threads share one sum: they compute the terms of F
// consecutive entries of its list and each adds all F in order. The lane of a
// wave is (kc PB + particle) F + f. A chunk with fewer particles than its tile
// is made for (cells of uneven occupancy, or smaller than the tile) has F > 1
// instead of lanes without a particle.
template <int TI, int K>
struct TileMap {
  static constexpr int NT = TI * K, NW = NT / 64;
  static constexpr int KC = K > NW ? K / NW : 1;   // lanes of the order per wave
  static constexpr int KG = K / KC;                // waves that share the particles
  static constexpr int Q = 64 / KC;                // PB F
  static constexpr int WP = NW / KG;               // waves that share the lanes
  // PB for a chunk of cnt particles
  __device__ __forceinline__ static int block(int cnt) {
    if (cnt <= 16 * WP) return 16;
    if (Q > 32 && cnt <= 32 * WP) return 32;
    return Q;
  }
};

// f(PB, F) as integral constants
template <int Q, class Fn>
__device__ __forceinline__ void with_block(int PB, Fn f) {
  if constexpr (Q == 64) {
    if (PB == 64) return f(std::integral_constant<int, 64>{}, std::integral_constant<int, 1>{});
  }
  if constexpr (Q >= 32) {
    if (PB == 32)
      return f(std::integral_constant<int, 32>{}, std::integral_constant<int, Q / 32>{});
  }
  f(std::integral_constant<int, 16>{}, std::integral_constant<int, Q / 16>{});
}

// A wave's operands of the prefilter for its PB particles, NB = PB / 16
// blocks: per lane component lane >> 4 of (-2p, 1) of the block's particle
// lane & 15, and its -c. F: threads per particle in the layout of the sums.
template <int PB, int F>
struct Prefilter {
  static constexpr int NB = PB / 16;
  float b[NB];

  __device__ __forceinline__ Prefilter(float m2x, float m2y, float m2z) {
    const int lane = threadIdx.x & 63, k = lane >> 4;
    if constexpr (NB == 4) {        // component per register -> component per lane row
      unsigned v[4] = {__float_as_uint(m2x), __float_as_uint(m2y), __float_as_uint(m2z),
                       __float_as_uint(1.0f)};
      transpose4(v);
#pragma unroll
      for (int q = 0; q < NB; ++q) b[q] = __uint_as_float(v[q]);
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int src = F * (16 * q + (lane & 15));
        const float x = __shfl(m2x, src), y = __shfl(m2y, src), z = __shfl(m2z, src);
        b[q] = k == 0 ? x : (k == 1 ? y : (k == 2 ? z : 1.0f));
      }
    }
  }

  // the value of each block's particle lane & 15, in every lane row
  __device__ __forceinline__ static void per_block(float v, float (&o)[NB]) {
    if constexpr (NB == 4) {
      const unsigned x = __float_as_uint(v);
      const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
      const auto e = __builtin_amdgcn_permlane32_swap(p[0], p[0], false, false);
      const auto f = __builtin_amdgcn_permlane32_swap(p[1], p[1], false, false);
      o[0] = __uint_as_float(e[0]);
      o[1] = __uint_as_float(f[0]);
      o[2] = __uint_as_float(e[1]);
      o[3] = __uint_as_float(f[1]);
    } else {
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int q = 0; q < NB; ++q) o[q] = __shfl(v, F * (16 * q + (lane & 15)));
    }
  }
};

// Signs of n2 - 2 p.q + c (with H2: n2 less h2 of the candidate) for the nt
// tiles (an even number, at most 8) of candidate group G of the wave's KC
// lanes of the order, as NB words per lane. The matrix result leaves rows 4 g
// .. 4 g + 3 of a tile in the 16 lanes of row g. The RG = 4 / KC row groups of
// a lane kc of the order cover its candidates: row 4 g + r of tile t, g = RG kc
// + x, is its candidate 32 RG G + 4 nt x + 4 t + r (staged at slot kc RC + its
// number), so a lane of row g collects one word per block, bit 4 t + r, of
// consecutive candidates. Lane rows and blocks are then exchanged: lane y has
// particle y mod PB and the words of row groups (y / PB) NB + j. The next
// tiles' operands are read ahead, and the results of a step's first matrix
// instruction are shifted in while the others run.
template <int NB, int KC, int RC, bool H2>
__device__ __forceinline__ void group_masks(const float4* cp, const float* ch2, int G, int nt,
                                            const float (&b)[NB], const float (&c)[NB],
                                            unsigned (&w)[NB]) {
  constexpr int TS = NB == 4 ? 1 : 2;                // tiles per step
  constexpr int RG = 4 / KC;
  const int lane = again(threadIdx.x) & 63;
  const int k = lane >> 4, g = (lane >> 2) & 3;
  const int sl0 = (g / RG) * RC + 32 * RG * G + 4 * nt * (g % RG) + (lane & 3);
  f4v cv[NB];          // made here: not kept through the other phases
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    float x = c[q];
    asm volatile("" : "+v"(x));
    cv[q] = f4v{x, x, x, x};
    w[q] = 0u;
  }
  auto arow = [&](int t) {
    const int sl = sl0 + 4 * max(t, 0);
    float a = reinterpret_cast<const float*>(cp + sl)[k];
    if constexpr (H2) {
      const float h2 = ch2[sl];
      a = k == 3 ? a - h2 : a;
    }
    return a;
  };
  float a[TS];
#pragma unroll
  for (int u = 0; u < TS; ++u) a[u] = arow(nt - 1 - u);
  for (int t = nt - 1; t >= 0; t -= TS) {
    f4v d[TS][NB];
#pragma unroll
    for (int u = 0; u < TS; ++u)
#pragma unroll
      for (int q = 0; q < NB; ++q)
        d[u][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[q], cv[q], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < TS; ++u) a[u] = arow(t - TS - u);
#pragma unroll
    for (int u = 0; u < TS; ++u)
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int r = 3; r >= 0; --r)
          w[q] = __builtin_amdgcn_alignbit(w[q], __float_as_uint(d[u][q][r]), 31);
  }
  if constexpr (NB == 2) {
    const auto p = __builtin_amdgcn_permlane16_swap(w[0], w[1], false, false);
    w[0] = p[0];
    w[1] = p[1];
  } else if constexpr (NB == 4) {
    transpose4(w);
  }
}

// A wave's neighbour lists of one LDS batch: 64 / F lists of 32 F entries,
// list kc PB + particle, entry e of list l at (64 / F) e + l, so that the F
// threads of a sum read entries F it + f at 64 it + their lane's place without
// conflicts.
constexpr int kListWave = 64 * 32;

// Phase A and B of one LDS batch for a wave's PB particles: `masks(G, nt, w)`
// gives the accepted candidates of group G; they are appended to the lists in
// order, and `consume(n)` runs phase B over the lists (n: entries of the list
// of this thread's sum), at the end and, where a list would overflow with the
// next group, before. A group too dense for the lists is taken 32 candidates at a
// time. PARTS says how:
//   kFill: the lists take words until one does not fit (the density loop, whose
//   sums per entry cost no more than the entry: 110592 particles, 64x2, 39.5 ->
//   37.5 us; clustered 1.5M, 64x1, 738 -> 730);
//   kDirect: where every lane has its own list, `bits(m, base)` runs phase B over
//   the bits of the word itself, in the same order, and there is no list to make
//   (force, 26617 clustered particles, 64x1, merged: 324 -> 295 us; filled lists
//   302);
//   kEach: a list per word (force, several threads per sum: as fast as kFill and
//   smaller).
enum : int { kFill, kDirect, kEach };
template <int PB, int F, int KC, int RC, int PARTS, class Masks, class Consume, class Bits>
__device__ __forceinline__ void test_and_consume(uint8_t* wl, int ntile, Masks masks,
                                                 Consume consume, Bits bits) {
  constexpr int NB = PB / 16, L = 64 / PB, NL = 64 / F, LP = kListWave / NL, RG = 4 / KC;
  static_assert(L == F * KC && RG == F * NB, "a wave holds PB F KC lanes");
  const int lane = threadIdx.x & 63;
  const int tr = lane / PB;         // this lane's place among the L of its particle
  uint8_t* const pl = wl + (tr / F) * PB + (lane & (PB - 1));
  unsigned w[NB];
  int n = 0;                        // entries of list (tr / F, lane mod PB)
  // over the F lanes that share a list: total, and the sum before this lane
  auto share = [&](int v, int& pre) {
    pre = 0;
    int tot = v;
    if constexpr (F == 4 || (F == 2 && KC == 2)) {
      const int o = lane_xor_i<16>(tot);
      pre += tr & 1 ? o : 0;
      tot += o;
    }
    if constexpr (F == 4 || (F == 2 && KC == 1)) {
      const int o = lane_xor_i<32>(tot);
      pre += tr & (F / 2) ? o : 0;
      tot += o;
    }
    return tot;
  };
  // the lowest and the highest bit of m in turn, which become entries from the
  // front and from the back of m's part of the list: two chains that do not wait
  // for each other (the last of an odd number is written twice)
  auto append = [&](unsigned m, uint8_t*& le, unsigned base) {
    const int k = NL * __popc(m);
    uint8_t *lo = le, *hi = le + k - NL;
    le += k;
    while (m) {
      const unsigned top = __builtin_clz(m);
      *lo = (uint8_t)((unsigned)__builtin_ctz(m) + base);
      *hi = (uint8_t)(31u - top + base);
      lo += NL;
      hi -= NL;
      m &= m - 1;
      m &= ~(0x80000000u >> top);
    }
  };
  // the list of this thread's sum was counted, and may have been written, by
  // other lanes, which write the next one when all have read this
  auto sums = [&] {
    wave_sync();
    consume(L == 1 ? n : __shfl(n, (lane / (F * PB)) * F * PB + (lane / F) % PB));
    wave_sync();
    n = 0;
  };
  for (int G = 0; 8 * G < ntile; ++G) {
    const int nt = min(ntile - 8 * G, 8);
    masks(G, nt, w);
    int add = 0, pre;
#pragma unroll
    for (int j = 0; j < NB; ++j) add += __popc(w[j]);
    const int tot = share(add, pre);
    // first entry of this lane's word j: row group tr NB + j
    auto base = [&](int j) {
      const int rg = tr * NB + j;
      return (unsigned)((rg / RG) * RC + 32 * RG * G + 4 * nt * (rg % RG));
    };
    const bool last = 8 * G + 8 >= ntile;
    if constexpr (PARTS == kFill) {
      int row = RG;                 // row groups of a group that is taken in parts
      if (__any(n + tot > LP)) {
        row = 0;
      } else {
        uint8_t* le = pl + (n + pre) * NL;
#pragma unroll
        for (int j = 0; j < NB; ++j) append(w[j], le, base(j));
        n += tot;
      }
      for (;; ++row) {              // one call site of the sums: they are large code
        unsigned m = 0u, b0 = 0u;
        int t = 0, p = 0;
        if (row < RG) {
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const bool mine = (tr * NB + j) % RG == row;
            m = mine ? w[j] : m;
            b0 = mine ? base(j) : b0;
          }
          t = share(__popc(m), p);
        }
        if (row < RG ? __any(n + t > LP) : last) sums();
        if (row == RG) break;
        uint8_t* le = pl + (n + p) * NL;
        append(m, le, b0);
        n += t;
      }
      continue;
    }
    for (int row = -1;;) {          // row groups of a group that is taken in parts
      if (row < 0 && !__any(n + tot > LP)) {
        uint8_t* le = pl + (n + pre) * NL;
#pragma unroll
        for (int j = 0; j < NB; ++j) append(w[j], le, base(j));
        n += tot;
        if (!last) break;
        row = RG;                   // done: the batch's sums
      } else if (RG > 1 && row >= 0) {
        // at most 32 entries of a list, from one of its lanes
        unsigned m = 0u, b0 = 0u;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const bool mine = (tr * NB + j) % RG == row;
          m = mine ? w[j] : m;
          b0 = mine ? base(j) : b0;
        }
        if constexpr (PARTS == kDirect && L == 1) {
          bits(m, b0);
          if (++row == RG) break;
          continue;
        }
        int p;
        uint8_t* le = pl;
        n = share(__popc(m), p);
        append(m, le, b0);
        ++row;
      } else {
        row = __any(n > 0) ? -1 : 0;   // empty the lists first
        if (row == 0) continue;
      }
      sums();
      if (row == RG) break;
    }
  }
}

// The F threads of a sum add the terms of F consecutive list entries in
// order: value of thread f of the group, in all of them
template <int F, int f>
__device__ __forceinline__ float of_thread(float v) {
  if constexpr (F == 1) return v;
  constexpr int ctrl = F == 4 ? f * 0x55 : (f == 0 ? 0xA0 : 0xF5);   // quad_perm
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true));
}
template <int F, class Fn>
__device__ __forceinline__ void in_order(Fn fn) {
  fn(std::integral_constant<int, 0>{});
  if constexpr (F >= 2) fn(std::integral_constant<int, 1>{});
  if constexpr (F == 4) {
    fn(std::integral_constant<int, 2>{});
    fn(std::integral_constant<int, 3>{});
  }
}

// Adds the K lanes of every particle's N sums in the fixed tree (lane x + lane
// x + K / 2, then K / 4, ...): the threads of lane 0 hold the result. `buf`:
// N NT floats of LDS.
template <int TI, int K, int N, class Add>
__device__ __forceinline__ void over_lanes(int kk, int gi, bool own, float (&v)[N], float* buf,
                                           Add add) {
  if constexpr (K > 1) {
    if (own) {
#pragma unroll
      for (int q = 0; q < N; ++q) buf[(q * K + kk) * TI + gi] = v[q];
    }
    __syncthreads();
    if (own && kk == 0) {
#pragma unroll
      for (int q = 0; q < N; ++q) {
        float t[K];
#pragma unroll
        for (int k = 0; k < K; ++k) t[k] = buf[(q * K + k) * TI + gi];
#pragma unroll
        for (int o = K / 2; o > 0; o >>= 1)
#pragma unroll
          for (int k = 0; k < o; ++k) t[k] = add(q, t[k], t[k + o]);
        v[q] = t[0];
      }
    }
  }
}

__device__ __forceinline__ float norm2(float x, float y, float z) {
  return __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
}

// dist2 with p given as -2p: fma(-2p, -1/2, -q) is p - q rounded once, the
// same value as dist2's subtraction, so the lanes need not keep p itself.
__device__ __forceinline__ float dist2_m2(float m2x, float m2y, float m2z, float qx, float qy,
                                          float qz, float& dx, float& dy, float& dz) {
#pragma clang fp contract(off)
  dx = __builtin_fmaf(m2x, -0.5f, -qx);
  dy = __builtin_fmaf(m2y, -0.5f, -qy);
  dz = __builtin_fmaf(m2z, -0.5f, -qz);
  float xx = dx * dx;
  return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, xx));
}

// Work distribution. No work list: one workgroup per cell, taking the
// cell's chunks of TI in turn. With a work list, items (cell, first slot)
// of XCD range x = blockIdx % 8 (workgroups are dispatched to the 8 XCDs in
// turn):
//   GRID / STATIC: workgroup l of its XCD takes items lo_x + l, + G/8, ...
//     (GRID launches about one workgroup per item, STATIC only as many as
//     stay resident);
//   DYNAMIC: resident workgroups take items from their XCD's queue with an
//     atomic counter and then steal from the other queues; the counter of
//     the next item is bumped while the current one is processed, so the
//     atomic's latency overlaps the work.
// A merged item (the work list's max_cells > 1) packs m - 1 into the bits
// of the cell id from kMergeShift up: its slots are those of the m cells
// cell, cell + 1, ... of one brick row, at most TI of them.
// The chunk callback takes (cell, m, c0, c1, only_q, out, obase): slots
// [c0, c1) of the m cells from `cell` along x, the neighbour cell index q
// (0..26) the j particles are restricted to (-1: all of them, -2: none; else
// only with m = 1), and the task result records (out == nullptr: the full loop's
// outputs) with slot i's record at out[obase + i].
// Position of slot i of a chunk over the m cells from `cell` along x,
// relative to `cell`: the stored offset in i's own cell, shifted by that
// cell's distance from `cell` with the same expression as the candidates'
// shifts, so that i meets its own candidate copy at r = 0 exactly.
template <class Src>
__device__ __forceinline__ void chunk_pos(const Src& src, const CellsDev& cd, int i, int cell,
                                          int m, float s32, float& x, float& y, float& z) {
  int d = 0;
  for (int k = 1; k < m; ++k) d += i >= clamp_slot(cd.start[cell + k], cd.n) ? 1 : 0;
  int cx, cy, cz;
  cell_coords(cell + d, cd.n_c, cx, cy, cz);
  src.pos(src.load_pos(i), typename Src::Origin(cx, cy, cz, cd.n_c), x, y, z);
  x = shifted(x, cell_shift(d, s32));
}

struct LoopItems {
  WorkDev wk;

  template <class Chunk>
  __device__ __forceinline__ void run(const CellsDev& cd, int TI, Chunk chunk) const {
  if (!wk.items) {   // one workgroup per cell, cells in brick order
    const int cell = brick_cell(xcd_remap(blockIdx.x, gridDim.x), cd.n_c);
    const int cs = clamp_slot(cd.start[cell], cd.n);
    const int ce = max(clamp_slot(cd.start[cell + 1], cd.n), cs);
    for (int base = cs; base < ce; base += TI)
      chunk(cell, 1, base, min(base + TI, ce), -1, (sph_task_result*)nullptr, 0);
    return;
  }
  const int C = cd.n_c * cd.n_c * cd.n_c;
  auto item = [&](int it) {
    const int2 v = wk.items[it];
    int cell = v.x, m = 1;
    if (wk.merge > 1) {
      cell = v.x & ((1 << kMergeShift) - 1);
      m = (int)((unsigned)v.x >> kMergeShift) + 1;
    }
    cell = min(max(cell, 0), C - 1);
    if (m > 1) {   // stay within the row (the list builder guarantees it)
      int cx, cy, cz;
      cell_coords(cell, cd.n_c, cx, cy, cz);
      m = min(min(m, kMaxMerge), cd.n_c - cx);
    }
    const int ce = max(clamp_slot(cd.start[cell + m], cd.n), 0);
    const int base = clamp_slot(v.y, ce);
    chunk(cell, m, base, min(base + TI, ce), -1, (sph_task_result*)nullptr, 0);
  };
  const int x = blockIdx.x & (kQueues - 1);
  const int total = min(wk.meta[0], wk.capacity);
  if (wk.sched != SPH_SCHED_DYNAMIC) {
    const int nl = gridDim.x / kQueues;
    const int lo = max(wk.meta[1 + x], 0), hi = min(wk.meta[2 + x], total);
    for (int it = lo + (int)(blockIdx.x / kQueues); it < hi; it += nl) item(it);
    return;
  }
  // more workgroups than items (small sets, filtered lists): the others would
  // only stand in line at the queues (4096 particles, 128x2, density / force us: 572
  // / 146, now 22 / 25)
  if ((int)blockIdx.x >= (total + kQueues - 1) / kQueues * kQueues) return;
  __shared__ int s_item;
  int qi = 0;   // thread 0: queue it takes items from, counted from its own
  // Item of the next queue that holds one. The queues are looked at first, all
  // at once, and an atomic goes to those with items left only (a queue found
  // empty stays so): at the end of a launch every workgroup comes by every
  // queue, and atomics on all of them, served one after the other, took longer
  // than the work (64000 particles, 128x2, density / force us: 534 / 365, now
  // 52 / 74; 512000: 808 / 731, now 366 / 427).
  auto grab = [&]() {
    unsigned open = 0u;
#pragma unroll
    for (int i = 0; i < kQueues; ++i) {
      const int q = (x + i) & (kQueues - 1);
      const int at =
          __hip_atomic_load(&wk.counters[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      open |= at < min(wk.meta[2 + q], total) ? 1u << i : 0u;
    }
    for (open &= ~0u << qi; open; open &= open - 1) {
      qi = __builtin_ctz(open);
      const int q = (x + qi) & (kQueues - 1);
      const int idx = atomicAdd(&wk.counters[q], 1);
      if (idx < min(wk.meta[2 + q], total)) return idx;
    }
    qi = kQueues;
    return -1;
  };
  if (threadIdx.x == 0) {
    const int first = atomicAdd(&wk.counters[x], 1);
    if (first < min(wk.meta[2 + x], total)) {
      s_item = first;
    } else {
      qi = 1;
      s_item = grab();
    }
  }
  __syncthreads();
  int it = __builtin_amdgcn_readfirstlane(s_item);
  while (it >= 0) {
    int nxt = -1, nq = 0;
    if (threadIdx.x == 0 && qi < kQueues) {
      nq = (x + qi) & (kQueues - 1);
      nxt = atomicAdd(&wk.counters[nq], 1);
    }
    __syncthreads();   // every thread has read s_item
    item(it);
    if (threadIdx.x == 0) {
      if (qi >= kQueues) {
        nxt = -1;
      } else if (nxt >= min(wk.meta[2 + nq], total)) {
        ++qi;
        nxt = grab();
      }
      s_item = nxt;
    }
    __syncthreads();
    it = __builtin_amdgcn_readfirstlane(s_item);
  }
}
};

// Neighbour index q = (dx+1) + 3 (dy+1) + 9 (dz+1) of cell cj seen from
// cell ci (periodic), or -2 if cj is not one of the 27 cells around ci.
__device__ __forceinline__ int nbr_index(int ci, int cj, int n_c) {
  int ax, ay, az, bx, by, bz;
  cell_coords(ci, n_c, ax, ay, az);
  cell_coords(cj, n_c, bx, by, bz);
  auto wrap = [&](int d) { return d > 1 ? d - n_c : (d < -1 ? d + n_c : d); };
  const int dx = wrap(bx - ax), dy = wrap(by - ay), dz = wrap(bz - az);
  if (dx < -1 || dx > 1 || dy < -1 || dy > 1 || dz < -1 || dz > 1) return -2;
  return (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
}

// Work items of a batch of cell-pair tasks: workgroup b takes item b =
// (task, first slot), i.e. up to TI slots of the task's i range against
// the task's neighbour cell only.
struct TaskItems {
  const sph_task* tasks;
  int ntasks;
  const int32_t* out_off;
  const int2* items;
  int nitems;
  sph_task_result* out;
  int n_out;

  template <class Chunk>
  __device__ __forceinline__ void run(const CellsDev& cd, int TI, Chunk chunk) const {
    const int b = blockIdx.x;
    if (b >= nitems) return;
    const int C = cd.n_c * cd.n_c * cd.n_c;
    const int2 it = items[b];
    const int ti_ = min(max(it.x, 0), ntasks - 1);
    const sph_task t = tasks[ti_];
    const int ci = min(max(t.ci, 0), C - 1), cj = min(max(t.cj, 0), C - 1);
    const int cs = clamp_slot(cd.start[ci], cd.n);
    const int ce = max(clamp_slot(cd.start[ci + 1], cd.n), cs);
    const int ib = min(max(t.i_begin, cs), ce), ie = min(max(t.i_end, ib), ce);
    const int c0 = min(max(it.y, ib), ie), c1 = min(c0 + TI, ie);
    const int o = min(max(out_off[ti_], 0), n_out);
    // records past n_out are dropped: clamp the range to what fits
    const int c1o = min(c1, c0 + max(n_out - (o + (c0 - ib)), 0));
    chunk(ci, 1, c0, c1o, nbr_index(ci, cj, cd.n_c), out, o - ib);
  }
};

// --------------------------------------------------------------------------
// Density
// --------------------------------------------------------------------------
// The second launch bound: the compiler reads it as waves per SIMD =
// blocks x ceil(waves per block / 4). Four waves per SIMD (at most 128
// VGPRs; tiles of 64 particles spill one to three) for every density tile,
// three (168 VGPRs; 64x2 spills three, on records the 64-particle tiles up to 17)
// for every force tile.
template <int NT>
constexpr int kDensityBlocks = 4;
template <int NT>
constexpr int kForceBlocks = 3;

template <int TI, int K, class Src, class Items, int KS>
__global__ __launch_bounds__(TI* K, kDensityBlocks<TI * K>) void k_density(Src, CellsDev cd, Phys ph,
                                                                    float s32, Items items) {
  using Shape = KernelShape<KS>;
  constexpr int NT = TI * K;
  // staged candidates: 2 NT leaves LDS for four waves per SIMD (64x1 on the
  // 128^3 lattice: 431 us with 256 candidates, 382 with 128)
  constexpr int CAP = 2 * NT;
  constexpr int kLimit = batch_limit(K == 1 ? 2 : 3, NT, K);
  // rounds of a gather window (and half the queue): fewer leave more LDS for
  // resident workgroups, more hide more latency (64x1 on the 128^3 lattice,
  // us: 2 rounds 391, 3 382, 4 374; clustered 32x2, 1.5M: 818, 798, 815; the
  // wider tiles: 64x4 on 0.88M, 64 per cell: 1 round 328, 2 286, 3 285)
  constexpr int KR = NT == 64 ? 3 : 2;
  using Map = TileMap<TI, K>;
  constexpr int RC = CAP / K;     // staged candidates of one lane of the order
  static_assert(Map::KC * RC <= 256, "list entries are bytes");
  __shared__ float4 cand[CAP];                 // x, y, z relative to this cell, |x|^2
  __shared__ float cmass[CAP];                 // m_j
  __shared__ alignas(16) uint8_t lst[kListWave * (NT / 64) + 64];
  __shared__ NbrCells<typename Src::Origin> T;
  __shared__ RangeTab<NT, KR> tab;
  __shared__ Queue<NT, K, KR> queue;
  __shared__ int wtot[2 * KR * (NT / 64)];
  __shared__ int red[7 * (NT / 64)];

  const int n_c = cd.n_c;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint8_t* const wl = lst + kListWave * wave;
  const int kg = wave % Map::KG, pg = wave / Map::KG;
  const float gk = ph.gamma_k;

  items.run(cd, TI, [&](int cell, int m, int c0, int c1, int only_q, sph_task_result* tout,
                        int tbase) {
    int cx, cy, cz;
    cell_coords(cell, n_c, cx, cy, cz);
    build_nbr<false>(T, cd, cx, cy, cz, m, s32, gk);
    tab.clear();     // published by the chunk box's barriers
    const int PB = Map::block(c1 - c0);
    const int F = Map::Q / PB, f = lane % F;      // 1, 2 or 4
    const int gi = pg * PB + (lane / F) % PB, kk = kg * Map::KC + lane / (F * PB);
    const int i = c0 + gi;
    const bool vi = i < c1;
    float xi = 0.f, yi = 0.f, zi = 0.f, hi = 0.f, ui = 0.f;
    if (vi) {
      const Src src = kernel_src<Src>();
      chunk_pos(src, cd, i, cell, m, s32, xi, yi, zi);
      hi = src.hsml(src.load_h(i));
      ui = src.uint(i);
    }
    const float H2 = vi ? support2(gk, hi) : 0.0f;
    const float Hinv = vi ? 1.0f / (gk * hi) : 0.0f;
    const ChunkBox bx = chunk_box<NT>(vi, xi, yi, zi, H2, red);
    flag_support(cd, bx, s32);
    const float bext = uniform(sqrtf(bx.h2max));
    const float m2x = -2.0f * xi, m2y = -2.0f * yi, m2z = -2.0f * zi;
    // -c of the prefilter; +inf (nothing accepted) without a particle or where
    // its position or support is NaN
    const float pp = norm2(xi, yi, zi);
    const float nc0 = pp - prefilter_margin(bx, s32) - H2;
    const bool usable = vi && pp < 1e30f && nc0 == nc0;
    const float negc = usable ? nc0 : __builtin_inff();

    float rho = 0.f, wsum = 0.f, dh = 0.f;
    int nn = 0;
    int gathered = 0;     // uniform: work counter of the chunk

    // candidates [off, off + cnt) of the queue into LDS, padded to whole
    // steps with entries no particle accepts
    auto fill = [&](int off, int cnt, int ntile) {
      const Src src = kernel_src<Src>();
      const int tid = again(threadIdx.x);
      typename Src::Pos pr[CAP / NT];
      typename Src::Mhu mr[CAP / NT];
      int qq[CAP / NT];
#pragma unroll
      for (int r = 0; r < CAP / NT; ++r) {   // threads past the end repeat an entry
        const int y = off + min(r * NT + tid, cnt - 1);
        const int j = min(max(queue.slot[y], 0), cd.n - 1);
        qq[r] = queue.q[y];
        pr[r] = src.load_pos(j);
        mr[r] = src.load_m(j);
      }
#pragma unroll
      for (int r = 0; r < CAP / NT; ++r) {
        const int x = r * NT + tid;
        float4 c;
        float sx, sy, sz;
        const int q = min(qq[r], kMaxNbr - 1);    // an empty entry reads some cell
        src.pos(pr[r], T.origin(q), c.x, c.y, c.z);
        T.shift(q, s32, sx, sy, sz);
        c.x = shifted(c.x, sx);
        c.y = shifted(c.y, sy);
        c.z = shifted(c.z, sz);
        // empty entries, and positions that are not finite (no pair test accepts
        // those), become entries the prefilter rejects
        c.w = norm2(c.x, c.y, c.z);
        if (!(x < cnt && (K == 1 || qq[r] != kHole) && c.w < 1e30f))
          c = make_float4(0.f, 0.f, 0.f, 1e30f);
        if (x < Map::KG * kMfmaTile * ntile) {
          const int sl = (x % K) * RC + x / K;
          cand[sl] = c;
          cmass[sl] = src.mass(mr[r]);
        }
      }
    };
    auto pairs = [&](int ntile) {
      if (pg * PB >= c1 - c0) return;   // no particle in this wave
      const float4* const cw = cand + kg * Map::KC * RC;
      const float* const mw = cmass + kg * Map::KC * RC;
      with_block<Map::Q>(PB, [&](auto pb, auto fc) {
        constexpr int PB = decltype(pb)::value, F = decltype(fc)::value, NB = PB / 16;
        const Prefilter<PB, F> pf(usable ? m2x : 0.0f, usable ? m2y : 0.0f, usable ? m2z : 0.0f);
        float nc[NB];
        pf.per_block(negc, nc);
        test_and_consume<PB, F, Map::KC, RC, kFill>(
            wl, ntile,
            [&](int G, int nt, unsigned(&w)[NB]) {
              group_masks<NB, Map::KC, RC, false>(cw, nullptr, G, nt, pf.b, nc, w);
            },
            [&](int n) {
              // the next list entry is read while one is processed
              const uint8_t* le = wl + f * (64 / F) + lane / F;
              int tn = *le;
              for (int it = 0; it < n; it += F) {
                const bool has = F == 1 || it + f < n;
                const int t = has ? tn : 0;
                const float4 q = cw[t];
                const float mj = mw[t];
                tn = *(le += 64);
                float dx, dy, dz;
                const float r2 = dist2_m2(m2x, m2y, m2z, q.x, q.y, q.z, dx, dy, dz);
                const bool in = r2 < H2 && has;       // the exact support test
                const float u = fast_sqrt(r2) * Hinv;
                float w, dw;
                Shape::w_dw(u, w, dw);
                w = in ? w : 0.0f;
                dw = in ? dw : 0.0f;
                nn += in ? 1 : 0;
                if constexpr (F == 1) {
                  rho = fmaf(mj, w, rho);
                  wsum += w;
                  dh = fmaf(mj, fmaf(u, dw, 3.0f * w), dh);
                } else {
                  float d = fmaf(u, dw, 3.0f * w);
                  d = in ? d : 0.0f;
                  const float m = has ? mj : 0.0f;
                  in_order<F>([&](auto k) {
                    constexpr int x = decltype(k)::value;
                    const float mk = of_thread<F, x>(m), wk = of_thread<F, x>(w);
                    rho = fmaf(mk, wk, rho);
                    wsum += wk;
                    dh = fmaf(mk, of_thread<F, x>(d), dh);
                  });
                }
              }
            },
            [](unsigned, unsigned) {});
      });
    };

    GatherState gs;
    for_sub_cells<NT, KR>(
        cd, T, tab, reinterpret_cast<int*>(lst), s32, bx, kLimit,
        [&](int q) { return (only_q == -1 || q == only_q) ? bext : 0.0f; },
        [&](int my_end, bool last) {
          gathered += __builtin_amdgcn_readfirstlane(tab.total);
          gather_batch<Src, NT, K, KR, kLimit>(
              tab, T, queue, cd.n, s32, wtot, gs, my_end, last,
              [&](const Src& src, int j) { return src.load_pos(j); },
              [&](const Src& src, const typename Src::Pos& r, int q, float4& c) {
                src.pos(r, T.origin(q), c.x, c.y, c.z);
              },
              [&](const float4& c) {
                return box_dist2(c.x, c.y, c.z, bx.lox, bx.loy, bx.loz, bx.hix, bx.hiy, bx.hiz) <
                       bx.h2max;
              },
              [&](int n) { for_lds_batches<CAP, K, Map::KG, false>(n, false, fill, pairs); });
        });

    if (cd.tally && tid == 0) {
      atomicAdd(cd.tally, (unsigned long long)(c1 - c0) * (unsigned long long)gs.kept);
      atomicAdd(cd.tally + 1, (unsigned long long)gathered);
    }
    if (F >= 2) nn += __shfl_xor(nn, 1);
    if (F == 4) nn += __shfl_xor(nn, 2);
    float sum[4] = {rho, wsum, dh, __int_as_float(nn)};
    over_lanes<TI, K>(kk, gi, vi && f == 0, sum, reinterpret_cast<float*>(cand),
                      [](int k, float a, float b) {
                        return k == 3 ? __int_as_float(__float_as_int(a) + __float_as_int(b))
                                      : a + b;
                      });
    rho = sum[0];
    wsum = sum[1];
    dh = sum[2];
    nn = __float_as_int(sum[3]);
    const bool out = vi && kk == 0 && f == 0;
    if (out && tout) {
      const float Hinv3 = Hinv * Hinv * Hinv;
      float4* r = reinterpret_cast<float4*>(tout + (tbase + i));
      r[0] = make_float4(rho * Hinv3, kFourPiThird * wsum, -gk * dh * Hinv3 * Hinv, 0.0f);
      r[1] = make_float4(0.0f, __int_as_float(nn), 0.0f, 0.0f);
    } else if (out) {
      const float Hinv3 = Hinv * Hinv * Hinv;
      const float rho_i = rho * Hinv3;
      const float rho_dh = -gk * dh * Hinv3 * Hinv;
      const float omega = 1.0f + hi * rho_dh / (3.0f * rho_i);
      const float f = ph.gradh ? 1.0f / omega : 1.0f;
      const float P = (ph.gamma - 1.0f) * rho_i * ui;
      const float c = sqrtf(ph.gamma * (ph.gamma - 1.0f) * ui);
      kernel_src<Src>().dens_out(i, rho_i, kFourPiThird * wsum, rho_dh, f, P, c, nn);
    }
    __syncthreads();
  });
}

// --------------------------------------------------------------------------
// Force
// --------------------------------------------------------------------------
template <int TI, int K, class Src, class Items, int KS>
__global__ __launch_bounds__(TI* K, kForceBlocks<TI * K>) void k_force(Src, CellsDev cd, Phys ph,
                                                                 float s32, Items items) {
  using Shape = KernelShape<KS>;
  constexpr int NT = TI * K;
  constexpr int CAP = 2 * NT;     // staged candidates
  constexpr int kLimit = batch_limit(2, NT, K);
  // rounds of a gather window: two keep the workgroup's LDS within 1/12 of
  // the CU's (64x1 on the 128^3 lattice, us: 2 rounds 606, 3 626; 32x2
  // 678, 719; 64x4 on 0.88M: 1 round 489, 2 411, 3 414). Workgroups of two waves
  // have room for four, and small launches wait for fewer windows (64x2: 4096
  // particles 34.7 -> 31.0, 9001 clustered 79 -> 76, 120001 clustered 191 -> 181);
  // records' positions, three FP64 values each, would take too many registers.
  constexpr int KR = NT == 128 && std::is_same_v<typename Src::Origin, NoOrigin> ? 4 : 2;
  using Map = TileMap<TI, K>;
  constexpr int RC = CAP / K;     // staged candidates of one lane of the order
  static_assert(Map::KC * RC <= 256, "list entries are bytes");
  __shared__ float4 cp[CAP];      // x, y, z (relative to this cell), |x|^2
  __shared__ float ch2[CAP];      // H_j^2
  __shared__ float4 cv[CAP];      // v_j, m_j
  __shared__ float4 cs4[CAP];     // 1/H_j, A_j, c_j, rho_j
  __shared__ int selfpos[TI];     // batch << 16 | slot of particle c0 + k, or -1
  __shared__ alignas(16) uint8_t lst[kListWave * (NT / 64) + 64];
  __shared__ NbrCells<typename Src::Origin> T;
  __shared__ RangeTab<NT, KR> tab;
  __shared__ Queue<NT, K, KR> queue;
  __shared__ int wtot[2 * KR * (NT / 64)];
  __shared__ int red[7 * (NT / 64)];

  const int n_c = cd.n_c;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint8_t* const wl = lst + kListWave * wave;
  const int kg = wave % Map::KG, pg = wave / Map::KG;
  const float gk = ph.gamma_k;
  const float alpha = ph.alpha, beta = ph.beta;

  items.run(cd, TI, [&](int cell, int m, int c0, int c1, int only_q, sph_task_result* tout,
                        int tbase) {
    int cx, cy, cz;
    cell_coords(cell, n_c, cx, cy, cz);
    build_nbr<true>(T, cd, cx, cy, cz, m, s32, gk);
    tab.clear();     // published by the chunk box's barriers
    if (tid < TI) selfpos[tid] = -1;
    const int PB = Map::block(c1 - c0);
    const int F = Map::Q / PB, f = lane % F;      // 1, 2 or 4
    const int gi = pg * PB + (lane / F) % PB, kk = kg * Map::KC + lane / (F * PB);
    const int i = c0 + gi;
    const bool vi = i < c1;
    // lanes without a particle sit far outside the box and accept nothing
    float xi = 1e30f, yi = 1e30f, zi = 1e30f, hi = 1.f, vxi = 0.f, vyi = 0.f, vzi = 0.f;
    float rhoi = 1.f, fi = 1.f, Pi_ = 0.f, ci = 0.f;
    if (vi) {
      const Src src = kernel_src<Src>();
      chunk_pos(src, cd, i, cell, m, s32, xi, yi, zi);
      src.vel(src.load_vel(i), vxi, vyi, vzi);
      hi = src.hsml(src.load_h(i));
      src.dens_in(i, rhoi, fi, Pi_, ci);
    }
    const float H2i = vi ? support2(gk, hi) : 0.0f;
    const float Hinvi = 1.0f / (gk * hi);
    const float Hinv2i = Hinvi * Hinvi;
    const float Hinv4i = Hinv2i * Hinv2i;
    const float Ai = (ph.gradh ? fi : 1.0f) * Pi_ / (rhoi * rhoi);
    const ChunkBox bx = chunk_box<NT>(vi, xi, yi, zi, H2i, red);
    flag_support(cd, bx, s32);
    const float bi = uniform(sqrtf(bx.h2max));
    // prefilter: r^2 < max(H_i^2, H_j^2) becomes
    // n2 - 2 p.q < max(H_i^2 - |p|^2 + M, H_j^2 - (|p|^2 - M))
    const float m2x = -2.0f * xi, m2y = -2.0f * yi, m2z = -2.0f * zi;
    const float mrg = prefilter_margin(bx, s32);
    const float pp = norm2(xi, yi, zi);
    const bool usable = vi && pp < 1e30f;    // nothing accepted otherwise
    const float ppm = usable ? pp - mrg : __builtin_inff();
    // Where no neighbour cell's support bound exceeds the chunk's largest
    // support by much, one threshold per lane replaces the per-candidate
    // max: t < max(H_i^2, Hn^2) - |p|^2 + M, with Hn bounding every H_j of
    // the 27 cells, accepts a superset of the pairs at a few extra entries,
    // and the consume phase applies the exact test to each of them.
    const float hn = uniform(only_q < 0 ? T.hbmax : T.hb[only_q]);
    const float hn2 = hn * hn;
    const bool flat = hn2 <= kFlatRatio * bx.h2max;   // uniform over the block
    const float nc0 = pp - mrg - (flat ? fmaxf(H2i, hn2) : H2i);
    const float negc = usable && nc0 == nc0 ? nc0 : __builtin_inff();

    float ax = 0.f, ay = 0.f, az = 0.f, du = 0.f, vsig = 0.f;
    int nf = 0;
    int gathered = 0;     // uniform: work counter of the chunk

    int nbatch = 0;   // uniform: LDS batches consumed so far in this chunk
    // candidates [off, off + cnt) of the queue into LDS, padded to whole
    // steps with entries no particle accepts
    auto fill = [&](int off, int cnt, int ntile) {
      constexpr int kFill = CAP / NT;     // rounds, their loads in flight together
      const Src src = kernel_src<Src>();
      const int tid = again(threadIdx.x);
      typename Src::Pos pr[kFill];
      typename Src::Vel vr[kFill];
      typename Src::Mhu mr[kFill], hr[kFill];
      float4 d4[kFill];
      int jj[kFill], qq[kFill];
#pragma unroll
      for (int r = 0; r < kFill; ++r) {      // threads past the end repeat an entry
        const int y = off + min(r * NT + tid, cnt - 1);
        const int j = min(max(queue.slot[y], 0), cd.n - 1);
        jj[r] = j;
        qq[r] = queue.q[y];
        pr[r] = src.load_pos(j);
        vr[r] = src.load_vel(j);
        mr[r] = src.load_m(j);
        hr[r] = src.load_h(j);
        src.dens_in(j, d4[r].x, d4[r].y, d4[r].z, d4[r].w);
      }
#pragma unroll
      for (int r = 0; r < kFill; ++r) {
        const int x = r * NT + tid;
        float4 c, v;
        float sx, sy, sz;
        const int q = min(qq[r], kMaxNbr - 1);    // an empty entry reads some cell
        src.pos(pr[r], T.origin(q), c.x, c.y, c.z);
        T.shift(q, s32, sx, sy, sz);
        c.x = shifted(c.x, sx);
        c.y = shifted(c.y, sy);
        c.z = shifted(c.z, sz);
        c.w = norm2(c.x, c.y, c.z);
        // empty entries, and positions that are not finite (no pair test accepts
        // those), become entries the prefilter rejects
        const bool real = x < cnt && (K == 1 || qq[r] != kHole) && c.w < 1e30f;
        if (!real) c = make_float4(0.f, 0.f, 0.f, 1e30f);
        src.vel(vr[r], v.x, v.y, v.z);
        v.w = src.mass(mr[r]);
        const float hj = src.hsml(hr[r]);
        if (x < Map::KG * kMfmaTile * ntile) {
          const int sl = (x % K) * RC + x / K;
          cp[sl] = c;
          ch2[sl] = real ? support2(gk, hj) : 0.0f;
          cv[sl] = v;
          // d4 = (rho, f, P, c) -> (1/H, A, c, rho)
          cs4[sl] = make_float4(1.0f / (gk * hj),
                                (ph.gradh ? d4[r].y : 1.0f) * d4[r].z / (d4[r].x * d4[r].x),
                                d4[r].w, d4[r].x);
          if (real && jj[r] >= c0 && jj[r] < c1 && T.own(qq[r], m))
            selfpos[jj[r] - c0] = (nbatch << 16) | sl;
        }
      }
    };

    auto pairs = [&](int ntile) {
      // i's own copy in this batch, or less than 0
      const int sp = selfpos[min(gi, TI - 1)];
      const int tself = (sp >> 16) == nbatch ? (sp & 0xffff) - kg * Map::KC * RC : -1;
      ++nbatch;
      if (pg * PB >= c1 - c0) return;   // no particle in this wave
      const float4 *const pw = cp + kg * Map::KC * RC, *const vw = cv + kg * Map::KC * RC,
                          *const sw = cs4 + kg * Map::KC * RC;
      const float* const hw = ch2 + kg * Map::KC * RC;
      // one accepted candidate: all its fields are read at once (one LDS round
      // trip), then `next` issues the read of the next list entry
      auto pair = [&](auto fcc, int t, bool has, auto next) {
        constexpr int F = decltype(fcc)::value;
        const float4 q0 = pw[t];
        const float h2j = hw[t];
        const float4 q1 = vw[t];
        const float4 q2 = sw[t];
        next();
        float dx, dy, dz;
        const float r2 = dist2_m2(m2x, m2y, m2z, q0.x, q0.y, q0.z, dx, dy, dz);
        // the exact support test, r2 < max(H_i^2, H_j^2), and not the
        // self pair; coincident stored positions (r2 = 0, j != i) stay:
        // w'(0) = 0 makes their terms vanish
        // (the empty asm keeps the force-only loads ahead of the branch,
        // where they overlap the position load)
        asm volatile("" ::"v"(q1.x), "v"(q1.y), "v"(q1.z), "v"(q1.w), "v"(q2.x),
                     "v"(q2.y), "v"(q2.z), "v"(q2.w));
        const bool skip = !((r2 < H2i) | (r2 < h2j)) | (t == tself) | !has;
        if (F == 1 && skip) return;
        const float r = fast_sqrt(r2);
        const float rinv = r2 > 0.0f ? fast_rcp(r) : 0.0f;
        const float ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
        const float gi_ = Shape::dw(r * Hinvi) * Hinv4i;
        const float hj2 = q2.x * q2.x;
        const float gj_ = Shape::dw(r * q2.x) * (hj2 * hj2);
        const float w = (vxi - q1.x) * ex + (vyi - q1.y) * ey + (vzi - q1.z) * ez;
        const float mu = fminf(w, 0.0f);
        const float vs = ci + q2.z - beta * mu;
        const float visc = -alpha * vs * mu * fast_rcp(rhoi + q2.w);
        const float gbar = 0.5f * (gi_ + gj_);
        const float kc = q1.w * (Ai * gi_ + q2.y * gj_ + visc * gbar);
        const float ke = q1.w * (Ai * gi_ + 0.5f * visc * gbar);
        if constexpr (F == 1) {
          ax = fmaf(-kc, ex, ax);
          ay = fmaf(-kc, ey, ay);
          az = fmaf(-kc, ez, az);
          du = fmaf(ke, w, du);
          // vs >= 0: the larger float is the larger int
          vsig = __int_as_float(max(__float_as_int(vsig), __float_as_int(vs)));
          ++nf;
        } else {      // a skipped entry adds zeros
          const float k0 = skip ? 0.0f : -kc, e0 = skip ? 0.0f : ke;
          const float x0 = skip ? 0.0f : ex, y0 = skip ? 0.0f : ey,
                      z0 = skip ? 0.0f : ez, w0 = skip ? 0.0f : w;
          in_order<F>([&](auto k) {
            constexpr int x = decltype(k)::value;
            const float kx = of_thread<F, x>(k0);
            ax = fmaf(kx, of_thread<F, x>(x0), ax);
            ay = fmaf(kx, of_thread<F, x>(y0), ay);
            az = fmaf(kx, of_thread<F, x>(z0), az);
            du = fmaf(of_thread<F, x>(e0), of_thread<F, x>(w0), du);
          });
          if (!skip) {
            vsig = __int_as_float(max(__float_as_int(vsig), __float_as_int(vs)));
            ++nf;
          }
        }
      };
      // two accepted candidates of one lane, t1 only where `two`: the terms of both
      // are computed side by side and added in order. Where few waves run, the loop
      // over a dense word is a chain of instructions that wait for each other (force,
      // 26617 clustered particles, 64x1, merged: 295 -> 282 us; 34295, 32x8: 338 ->
      // 318).
      auto pair2 = [&](int t0, int t1, bool two) {
        const int t[2] = {t0, t1};
        float4 q0[2], q1[2], q2[2];
        float h2j[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          q0[u] = pw[t[u]];
          h2j[u] = hw[t[u]];
          q1[u] = vw[t[u]];
          q2[u] = sw[t[u]];
        }
        float kc[2], ke[2], ex[2], ey[2], ez[2], w[2], vs[2];
        bool skip[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float dx, dy, dz;
          const float r2 = dist2_m2(m2x, m2y, m2z, q0[u].x, q0[u].y, q0[u].z, dx, dy, dz);
          skip[u] = !((r2 < H2i) | (r2 < h2j[u])) | (t[u] == tself) | (u == 1 && !two);
          const float r = fast_sqrt(r2);
          const float rinv = r2 > 0.0f ? fast_rcp(r) : 0.0f;
          ex[u] = dx * rinv, ey[u] = dy * rinv, ez[u] = dz * rinv;
          const float gi_ = Shape::dw(r * Hinvi) * Hinv4i;
          const float hj2 = q2[u].x * q2[u].x;
          const float gj_ = Shape::dw(r * q2[u].x) * (hj2 * hj2);
          w[u] = (vxi - q1[u].x) * ex[u] + (vyi - q1[u].y) * ey[u] + (vzi - q1[u].z) * ez[u];
          const float mu = fminf(w[u], 0.0f);
          vs[u] = ci + q2[u].z - beta * mu;
          const float visc = -alpha * vs[u] * mu * fast_rcp(rhoi + q2[u].w);
          const float gbar = 0.5f * (gi_ + gj_);
          kc[u] = q1[u].w * (Ai * gi_ + q2[u].y * gj_ + visc * gbar);
          ke[u] = q1[u].w * (Ai * gi_ + 0.5f * visc * gbar);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (skip[u]) continue;
          ax = fmaf(-kc[u], ex[u], ax);
          ay = fmaf(-kc[u], ey[u], ay);
          az = fmaf(-kc[u], ez[u], az);
          du = fmaf(ke[u], w[u], du);
          vsig = __int_as_float(max(__float_as_int(vsig), __float_as_int(vs[u])));
          ++nf;
        }
      };
      with_block<Map::Q>(PB, [&](auto pb, auto fc) {
        constexpr int PB = decltype(pb)::value, F = decltype(fc)::value, NB = PB / 16;
        const Prefilter<PB, F> pf(usable ? m2x : 0.0f, usable ? m2y : 0.0f, usable ? m2z : 0.0f);
        float nc[NB];
        pf.per_block(negc, nc);
        test_and_consume<PB, F, Map::KC, RC, F == 1 ? kDirect : kEach>(
            wl, ntile,
            [&](int G, int nt, unsigned(&w)[NB]) {
              group_masks<NB, Map::KC, RC, false>(pw, nullptr, G, nt, pf.b, nc, w);
              if (!flat) {    // or within the candidate's own support
                unsigned v[NB];
                float c2[NB];
                pf.per_block(ppm, c2);
                group_masks<NB, Map::KC, RC, true>(pw, hw, G, nt, pf.b, c2, v);
#pragma unroll
                for (int j = 0; j < NB; ++j) w[j] |= v[j];
              }
            },
            [&](int n) {
              // the next list entry is read while one is processed
              const uint8_t* le = wl + f * (64 / F) + lane / F;
              int tn = *le;
              for (int it = 0; it < n; it += F) {
                const bool has = F == 1 || it + f < n;
                pair(fc, has ? tn : 0, has, [&] { tn = *(le += 64); });
              }
            },
            [&](unsigned m, unsigned b0) {
              while (m) {      // two at a time; the last of an odd number twice
                const int t0 = (int)(b0 + __builtin_ctz(m));
                m &= m - 1;
                const int t1 = m ? (int)(b0 + __builtin_ctz(m)) : t0;
                pair2(t0, t1, m != 0u);
                m &= m - 1;
              }
            });
      });
    };

    GatherState gs;
    for_sub_cells<NT, KR>(
        cd, T, tab, reinterpret_cast<int*>(lst), s32, bx, kLimit,
        [&](int q) { return (only_q == -1 || q == only_q) ? fmaxf(bi, T.hb[q]) : 0.0f; },
        [&](int my_end, bool last) {
          gathered += __builtin_amdgcn_readfirstlane(tab.total);
          gather_batch<Src, NT, K, KR, kLimit>(
              tab, T, queue, cd.n, s32, wtot, gs, my_end, last,
              [&](const Src& src, int j) {
                return PosH<Src>{src.load_pos(j), src.load_h(j)};
              },
              [&](const Src& src, const PosH<Src>& r, int q, float4& c) {   // w: h_j
                src.pos(r.pos, T.origin(q), c.x, c.y, c.z);
                c.w = src.hsml(r.h);
              },
              [&](const float4& c) {
                return box_dist2(c.x, c.y, c.z, bx.lox, bx.loy, bx.loz, bx.hix, bx.hiy, bx.hiz) <
                       fmaxf(bx.h2max, support2(gk, c.w));
              },
              [&](int n) { for_lds_batches<CAP, K, Map::KG, true>(n, F == 1, fill, pairs); });
        });

    if (cd.tally && tid == 0) {
      atomicAdd(cd.tally, (unsigned long long)(c1 - c0) * (unsigned long long)gs.kept);
      atomicAdd(cd.tally + 1, (unsigned long long)gathered);
    }
    // over the threads of a sum as within one: the same integer maximum, which
    // keeps the NaN of a neighbour's sound speed however the chunk is laid out
    int vsi = __float_as_int(vsig);
    if (F >= 2) {
      vsi = max(vsi, __shfl_xor(vsi, 1));
      nf += __shfl_xor(nf, 1);
    }
    if (F == 4) {
      vsi = max(vsi, __shfl_xor(vsi, 2));
      nf += __shfl_xor(nf, 2);
    }
    vsig = __int_as_float(vsi);
    float sum[6] = {ax, ay, az, du, vsig, __int_as_float(nf)};
    over_lanes<TI, K>(kk, gi, vi && f == 0, sum, reinterpret_cast<float*>(cp),
                      [](int k, float a, float b) {
                        return k == 4 ? fmaxf(a, b)
                               : k == 5
                                   ? __int_as_float(__float_as_int(a) + __float_as_int(b))
                                   : a + b;
                      });
    ax = sum[0];
    ay = sum[1];
    az = sum[2];
    du = sum[3];
    vsig = sum[4];
    nf = __float_as_int(sum[5]);
    const bool out = vi && kk == 0 && f == 0;
    if (out && tout) {
      float4* r = reinterpret_cast<float4*>(tout + (tbase + i));
      r[0] = make_float4(ax, ay, az, du);
      r[1] = make_float4(vsig, __int_as_float(nf), 0.0f, 0.0f);
    } else if (out) {
      kernel_src<Src>().force_out(i, ax, ay, az, du, vsig, nf);
    }
    __syncthreads();
  });
}

template <int PT, int VT, int MT>
SoaSrc<PT, VT, MT> make_soa(const sph_soa& s, const Prec& p, int n_c) {
  SoaSrc<PT, VT, MT> r;
  for (int k = 0; k < 3; ++k) {
    r.off[k] = s.f[SPH_S_OFF_X + k];
    r.vq[k] = s.f[SPH_S_VQ_X + k];
  }
  r.anchor = p.anchor;
  r.anc = static_cast<const uint8_t*>(s.f[SPH_S_ANC]);
  // s 2^-b, exact: the kernels' cell side scaled by a power of two
  r.anc_step = p.anchor == SPH_ANCHOR_CORNER
                   ? 0.0f
                   : std::ldexp((float)(1.0 / (double)n_c), -(p.anchor - SPH_ANCHOR_SUB(0)));
  r.m = s.f[SPH_S_M];
  r.h = s.f[SPH_S_H];
  r.u = s.f[SPH_S_U];
  r.pos_dt = p.pos;
  r.vel_dt = p.vel;
  r.mhu_dt = p.mhu;
  r.lm = p.load_m;
  r.lh = p.load_h;
  r.lu = p.load_u;
  r.rho = static_cast<const float*>(s.f[SPH_S_RHO]);
  r.f = static_cast<const float*>(s.f[SPH_S_F]);
  r.P = static_cast<const float*>(s.f[SPH_S_P]);
  r.c = static_cast<const float*>(s.f[SPH_S_C]);
  r.o_rho = static_cast<float*>(s.f[SPH_S_RHO]);
  r.o_wcount = static_cast<float*>(s.f[SPH_S_WCOUNT]);
  r.o_rho_dh = static_cast<float*>(s.f[SPH_S_RHO_DH]);
  r.o_f = static_cast<float*>(s.f[SPH_S_F]);
  r.o_P = static_cast<float*>(s.f[SPH_S_P]);
  r.o_c = static_cast<float*>(s.f[SPH_S_C]);
  r.o_nngb = static_cast<int32_t*>(s.f[SPH_S_NNGB]);
  r.o_ax = static_cast<float*>(s.f[SPH_S_A_X]);
  r.o_ay = static_cast<float*>(s.f[SPH_S_A_Y]);
  r.o_az = static_cast<float*>(s.f[SPH_S_A_Z]);
  r.o_du = static_cast<float*>(s.f[SPH_S_DU]);
  r.o_vsig = static_cast<float*>(s.f[SPH_S_VSIG]);
  r.o_nforce = static_cast<int32_t*>(s.f[SPH_S_NFORCE]);
  return r;
}

// Resident workgroups (per CU times CUs), a multiple of the 8 XCDs
static int persistent_grid(const void* kernel, int block) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1024;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, block, 0) != hipSuccess ||
      per < 1)
    per = 1;
  return max(cus * per / kQueues, 1) * kQueues;
}

// Grid of a pair launch: cells, about one workgroup per item (rounded up to
// the 8 XCDs), or the resident workgroups.
static int pair_grid(const void* kernel, int block, int C, const WorkDev* w) {
  if (!w) return C;
  if (w->sched == SPH_SCHED_GRID) return (w->capacity + kQueues - 1) / kQueues * kQueues;
  return persistent_grid(kernel, block);
}

static __global__ void k_reset_queues(WorkDev w) {
  if (threadIdx.x < kQueues) w.counters[threadIdx.x] = w.meta[1 + threadIdx.x];
}

template <class S>
hipError_t run_density(const S& src, const CellsDev& c, const Phys& ph, int ti, int k,
                       const WorkDev* w, hipStream_t s) {
  WorkDev wv{};
  if (w) wv = *w;
  const int C = c.n_c * c.n_c * c.n_c;
  const float s32 = (float)(1.0 / (double)c.n_c);
  if (w && w->sched == SPH_SCHED_DYNAMIC) k_reset_queues<<<1, 64, 0, s>>>(*w);
#define SPH_DENS_CASE(TI_, K_)                                                        \
  if (ti == TI_ && k == K_) {                                                         \
    auto kern = ph.kernel == SPH_KERNEL_WENDLAND_C2                                   \
                    ? k_density<TI_, K_, S, LoopItems, SPH_KERNEL_WENDLAND_C2>        \
                    : k_density<TI_, K_, S, LoopItems, SPH_KERNEL_M4>;                \
    const int G = pair_grid((const void*)kern, TI_ * K_, C, w);                       \
    kern<<<G, TI_ * K_, 0, s>>>(src, c, ph, s32, LoopItems{wv});                      \
    return hipGetLastError();                                                         \
  }
  SPH_DENS_CASE(64, 4)
  SPH_DENS_CASE(32, 8)
  SPH_DENS_CASE(128, 2)
  SPH_DENS_CASE(64, 2)
  SPH_DENS_CASE(64, 1)
  SPH_DENS_CASE(16, 16)
  SPH_DENS_CASE(16, 4)
  SPH_DENS_CASE(32, 2)
#undef SPH_DENS_CASE
  return hipErrorInvalidValue;
}

template <class S>
hipError_t run_force(const S& src, const CellsDev& c, const Phys& ph, int ti, int k,
                       const WorkDev* w, hipStream_t s) {
  WorkDev wv{};
  if (w) wv = *w;
  const int C = c.n_c * c.n_c * c.n_c;
  const float s32 = (float)(1.0 / (double)c.n_c);
  if (w && w->sched == SPH_SCHED_DYNAMIC) k_reset_queues<<<1, 64, 0, s>>>(*w);
#define SPH_FORCE_CASE(TI_, K_)                                                       \
  if (ti == TI_ && k == K_) {                                                         \
    auto kern = ph.kernel == SPH_KERNEL_WENDLAND_C2                                   \
                    ? k_force<TI_, K_, S, LoopItems, SPH_KERNEL_WENDLAND_C2>          \
                    : k_force<TI_, K_, S, LoopItems, SPH_KERNEL_M4>;                  \
    const int G = pair_grid((const void*)kern, TI_ * K_, C, w);                       \
    kern<<<G, TI_ * K_, 0, s>>>(src, c, ph, s32, LoopItems{wv});                      \
    return hipGetLastError();                                                         \
  }
  SPH_FORCE_CASE(64, 4)
  SPH_FORCE_CASE(32, 8)
  SPH_FORCE_CASE(128, 2)
  SPH_FORCE_CASE(64, 2)
  SPH_FORCE_CASE(64, 1)
  SPH_FORCE_CASE(16, 16)
  SPH_FORCE_CASE(16, 4)
  SPH_FORCE_CASE(32, 2)
#undef SPH_FORCE_CASE
  return hipErrorInvalidValue;
}

// Task batches: one workgroup per item, density and force kernels
template <class S>
hipError_t run_tasks(const S& src, const CellsDev& c, const Phys& ph, int ti, int k,
                     const TaskItems& dens, const TaskItems& force, hipStream_t s) {
  const float s32 = (float)(1.0 / (double)c.n_c);
#define SPH_TASK_CASE(TI_, K_)                                                         \
  if (ti == TI_ && k == K_) {                                                          \
    const bool wc2 = ph.kernel == SPH_KERNEL_WENDLAND_C2;                                \
    auto kd = wc2 ? k_density<TI_, K_, S, TaskItems, SPH_KERNEL_WENDLAND_C2>             \
                  : k_density<TI_, K_, S, TaskItems, SPH_KERNEL_M4>;                     \
    auto kf = wc2 ? k_force<TI_, K_, S, TaskItems, SPH_KERNEL_WENDLAND_C2>               \
                  : k_force<TI_, K_, S, TaskItems, SPH_KERNEL_M4>;                       \
    if (dens.nitems > 0) kd<<<dens.nitems, TI_ * K_, 0, s>>>(src, c, ph, s32, dens);    \
    if (force.nitems > 0) kf<<<force.nitems, TI_ * K_, 0, s>>>(src, c, ph, s32, force); \
    return hipGetLastError();                                                          \
  }
  SPH_TASK_CASE(64, 4)
  SPH_TASK_CASE(32, 8)
  SPH_TASK_CASE(16, 16)
#undef SPH_TASK_CASE
  return hipErrorInvalidValue;
}

// instantiated in pair_*.hip
hipError_t run_density_dens_f32(const SoaSrc<DT_F32, DT_F32, DT_F32>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_density_dens_r(const SoaSrc<DT_F16, DT_BF16, DT_F16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_density_dens_h(const SoaSrc<DT_F16, DT_F16, DT_F16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_density_dens_b(const SoaSrc<DT_BF16, DT_BF16, DT_BF16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_density_dens_gen(const SoaSrc<-1, -1, -1>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_density_dens_aos(const AosSrc& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_f32(const SoaSrc<DT_F32, DT_F32, DT_F32>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_r(const SoaSrc<DT_F16, DT_BF16, DT_F16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_h(const SoaSrc<DT_F16, DT_F16, DT_F16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_b(const SoaSrc<DT_BF16, DT_BF16, DT_BF16>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_gen(const SoaSrc<-1, -1, -1>& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_force_force_aos(const AosSrc& src, const CellsDev& c, const Phys& ph, int ti, int k,
                  const WorkDev* w, hipStream_t s);
hipError_t run_tasks_f32(const SoaSrc<DT_F32, DT_F32, DT_F32>& src, const CellsDev& c,
                         const Phys& ph, int ti, int k, const TaskItems& dens,
                         const TaskItems& force, hipStream_t s);
hipError_t run_tasks_r(const SoaSrc<DT_F16, DT_BF16, DT_F16>& src, const CellsDev& c,
                       const Phys& ph, int ti, int k, const TaskItems& dens,
                       const TaskItems& force, hipStream_t s);
hipError_t run_tasks_gen(const SoaSrc<-1, -1, -1>& src, const CellsDev& c, const Phys& ph,
                         int ti, int k, const TaskItems& dens, const TaskItems& force,
                         hipStream_t s);

}  // namespace pairk
}  // namespace sph
