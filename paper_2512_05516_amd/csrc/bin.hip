// Cell binning: FP64 cell ids, a stable LSD radix sort by cell id, and the
// CSR cell_start table. The order is stable by (cell id, input index), so
// the permutation is identical on every run and on every device.
#include <algorithm>

#include "sph_device.h"

namespace sph {
namespace {

constexpr int kThreads = 256;
constexpr int kSortThreads = 1024;
constexpr int kRounds = 8;
constexpr int kTile = kSortThreads * kRounds; // keys per radix block
constexpr int kMaxBuckets = 512;             // radix buckets of the widest digit (9 bits)

// A gated launch does nothing when *gate == 0 (the cell list is kept: no
// particle changed its cell or sub-cell since it was built). The word is
// read at the start of each kernel; only the last kernel of the binning
// changes it.
__device__ __forceinline__ bool gated_off(const int32_t* gate) { return gate && *gate == 0; }

// Morton code of a sub-cell (bit b of sx at 3b, sy at 3b+1, sz at 3b+2)
__device__ __forceinline__ int morton3(int sx, int sy, int sz, int bits) {
  int m = 0;
  for (int b = 0; b < bits; ++b)
    m |= (((sx >> b) & 1) << (3 * b)) | (((sy >> b) & 1) << (3 * b + 1)) |
         (((sz >> b) & 1) << (3 * b + 2));
  return m;
}

// Largest record span staged through LDS by k_bin_keys (8-byte words)
constexpr int kSpanWords = 16;

// key = cell * R^3 + Morton(sub-cell); also h of each record for the
// per-cell maximum.
// nw > 0: the block first copies bytes [lo, lo + 8 nw) of each of its
// records into LDS with consecutive threads on consecutive words (x and h
// read from there), so every record line is fetched once and the loads
// coalesce; nw = 0: each thread reads its record's fields directly.
__global__ __launch_bounds__(kThreads) void k_bin_keys(const char* __restrict__ aos,
                                                        uint32_t stride, uint32_t offx,
                                                        uint32_t offh, int dth, uint32_t lo,
                                                        int nw, int n, int n_c, int sub_bits,
                                                        int32_t* __restrict__ keys,
                                                        float* __restrict__ hin,
                                                        int32_t* status, const int32_t* gate) {
  __shared__ uint2 span[kThreads * kSpanWords];
  if (gated_off(gate)) return;                 // uniform over the grid
  const int i0 = blockIdx.x * kThreads;
  const int i = i0 + threadIdx.x;
  const bool valid = i < n;   // no early exit: the whole block stages the records
  const char* rec;            // record bytes as seen at offsets offx, offh
  uint32_t rx = offx, rh = offh;
  if (nw > 0) {
    // every word of the block's spans: a thread's loads (at most
    // kSpanWords) are all issued before the first is stored to LDS
    const int nrec = min(kThreads, n - i0);
    const int nwords = nrec * nw;
    uint2 buf[kSpanWords];
#pragma unroll
    for (int q = 0; q < kSpanWords; ++q) {
      const int w = threadIdx.x + q * kThreads;
      buf[q] = make_uint2(0u, 0u);
      if (w < nwords) {
        const int r = w / nw, j = w - r * nw;
        buf[q] = *reinterpret_cast<const uint2*>(aos + (size_t)(i0 + r) * stride + lo + 8 * j);
      }
    }
#pragma unroll
    for (int q = 0; q < kSpanWords; ++q) {
      const int w = threadIdx.x + q * kThreads;
      if (w < nwords) span[w] = buf[q];
    }
    __syncthreads();
    rec = reinterpret_cast<const char*>(span + (valid ? threadIdx.x : 0) * nw);
    rx = offx - lo;
    rh = offh - lo;
  } else {
    rec = aos + (size_t)(valid ? i : 0) * stride;
  }
  const double* x = reinterpret_cast<const double*>(rec + rx);
  const int R = 1 << sub_bits;
  bool bad = false;
  int c[3], sc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double xv = x[k];
    bad |= !isfinite(xv);
    const double xw = wrap01(xv);
    c[k] = cell_axis(xw, n_c);
    const double t = floor(xw * (double)(n_c * R));
    int sa = (t == t) ? (int)fmin(fmax(t - (double)c[k] * R, 0.0), (double)(R - 1)) : 0;
    sc[k] = sa;
  }
  const int cell = c[0] + n_c * (c[1] + n_c * c[2]);
  if (valid) keys[i] = (cell << (3 * sub_bits)) + morton3(sc[0], sc[1], sc[2], sub_bits);
  // h of each input slot (0 where not positive): the per-cell maximum is
  // taken after the sort, where a wave's slots share few cells
  if (hin && valid) {
    const float h = rec_load32(rec, rh, dth);
    hin[i] = h > 0.0f ? h : 0.0f;
  }
  if (valid && bad && status) atomicOr(status, SPH_FLAG_BAD_POSITION);
}

// One pass of the sort, D-bit digits, NB = 2^D buckets, is three launches over
// tiles of kTile keys: the tiles' digit counts (hist[tile][digit]), their
// prefixes over the tiles, and the scatter; a list of one tile is one launch.
// Tiles are that large because a tile's run of a digit is what the scatter
// writes to consecutive addresses. 4.2M keys, 9-bit digits, us per pass: tiles
// of 2048 keys stored one by one 82, 32 with tiles of 8192 sorted in LDS first;
// counts and prefixes 37, now 11.
template <int D>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const int32_t* __restrict__ kin,
                                                              int32_t* __restrict__ hist, int n,
                                                              int shift, const int32_t* gate) {
  constexpr int NB = 1 << D;
  __shared__ int h[NB];
  if (gated_off(gate)) return;
  const int tid = threadIdx.x, t0 = blockIdx.x * kTile;
  if (tid < NB) h[tid] = 0;
  __syncthreads();
  int key[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int idx = t0 + r * kSortThreads + tid;
    key[r] = kin[min(idx, n - 1)];
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int idx = t0 + r * kSortThreads + tid;
    if (idx < n) atomicAdd(&h[(key[r] >> shift) & (NB - 1)], 1);
  }
  __syncthreads();
  if (tid < NB) hist[(size_t)blockIdx.x * NB + tid] = h[tid];
}

// Inclusive sum over the wave
__device__ __forceinline__ uint64_t wave_inclusive(uint64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t t = __shfl_up(v, o);
    v += lane >= o ? t : 0;
  }
  return v;
}

// Counts to exclusive prefixes over the tiles, per digit; the first tile's,
// which is zero, becomes the digit's total. A block takes 16 digits (one
// 64-byte segment of each tile's counts), 64 threads per digit.
constexpr int kScanDigits = 16;
__global__ __launch_bounds__(kSortThreads) void k_radix_prefix(int32_t* __restrict__ hist, int NB,
                                                                int nblk, const int32_t* gate) {
  constexpr int G = kSortThreads / kScanDigits;
  __shared__ int sum[kScanDigits][G + 1];
  if (gated_off(gate)) return;
  const int dl = threadIdx.x % kScanDigits, g = threadIdx.x / kScanDigits;
  const int d = blockIdx.x * kScanDigits + dl;
  const int per = (nblk + G - 1) / G;
  const int b0 = min(g * per, nblk), b1 = min(b0 + per, nblk);
  int s = 0;
#pragma unroll 8
  for (int b = b0; b < b1; ++b) s += hist[(size_t)b * NB + d];
  sum[dl][g] = s;
  __syncthreads();
  static_assert(G == 64, "a wave per digit");
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int v = sum[w][lane];
  const int inc = (int)wave_inclusive((uint64_t)v);
  sum[w][lane] = inc - v;
  if (lane == G - 1) sum[w][G] = inc;
  __syncthreads();
  int run = sum[dl][g];
#pragma unroll 8
  for (int b = b0; b < b1; ++b) {
    const size_t e = (size_t)b * NB + d;
    const int c = hist[e];
    hist[e] = b == 0 ? sum[dl][G] : run;
    run += c;
  }
}

// Stable scatter of one tile. A wave ranks its 512 consecutive keys in eight
// rounds: lanes with equal digits are found with D ballots, the wave's earlier
// rounds are counted in LDS, with no barrier between rounds. The waves' counts
// give every key its place in the tile sorted by digit, which is put together
// in LDS and written out digit run by digit run, so consecutive threads store
// consecutive addresses. vin == nullptr: the values are the key indices.
template <int D>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const int32_t* __restrict__ kin, const int32_t* __restrict__ vin, int32_t* __restrict__ kout,
    int32_t* __restrict__ vout, const int32_t* __restrict__ hist, int n, int shift,
    const int32_t* gate) {
  constexpr int NB = 1 << D, NW = kSortThreads / 64;
  static_assert(NB <= kSortThreads, "a thread per digit");
  __shared__ int2 tile[kTile];                 // (key, value) in the tile's digit order
  __shared__ uint16_t wcnt[NW][NB];            // a wave's keys of each digit, then their start
  __shared__ int gbase[NB];                    // a digit's first global position less its first here
  __shared__ uint64_t wsum[NW];
  if (gated_off(gate)) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b = blockIdx.x, t0 = b * kTile;
  const int ntile = min(kTile, n - t0);
  const int i0 = t0 + wave * (64 * kRounds) + lane;
  int key[kRounds], val[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int idx = min(i0 + 64 * r, n - 1);
    key[r] = kin[idx];
    val[r] = vin ? vin[idx] : idx;
  }
  int pre = 0, all = 0;       // of digit tid: keys in earlier tiles, and in all
  if (gridDim.x > 1 && tid < NB) {
    pre = b > 0 ? hist[(size_t)b * NB + tid] : 0;
    all = hist[tid];
  }
  for (int e = lane; e < NB; e += 64) wcnt[wave][e] = 0;
  wave_sync();
  int at[kRounds];            // keys of the same digit before it in the wave
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool valid = i0 + 64 * r < n;
    const int d = (key[r] >> shift) & (NB - 1);
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < D; ++bit) {
      const uint64_t bl = __ballot((d >> bit) & 1);
      m &= ((d >> bit) & 1) ? bl : ~bl;
    }
    const int rank = __popcll(m & lanemask_lt());
    const int before = wcnt[wave][d];
    at[r] = before + rank;
    wave_sync();     // every lane has read its count
    if (valid && rank == 0) wcnt[wave][d] = (uint16_t)(before + __popcll(m));
    wave_sync();
  }
  __syncthreads();
  int cnt = 0;
  if (tid < NB) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = wcnt[w][tid];
      wcnt[w][tid] = (uint16_t)cnt;
      cnt += c;
    }
    if (gridDim.x == 1) all = cnt;
  }
  // starts of the digits here (below 2^14) and over all keys
  const uint64_t v = (uint64_t)(uint32_t)all << 32 | (uint32_t)cnt;
  const uint64_t inc = wave_inclusive(v);
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint64_t st = inc - v;
#pragma unroll
  for (int w = 0; w < NW; ++w) st += w < wave ? wsum[w] : 0;
  if (tid < NB) {
    const int here = (int)(uint32_t)st;
    gbase[tid] = (int)(st >> 32) + pre - here;
#pragma unroll
    for (int w = 0; w < NW; ++w) wcnt[w][tid] = (uint16_t)(wcnt[w][tid] + here);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int d = (key[r] >> shift) & (NB - 1);
    if (i0 + 64 * r < n) tile[min(wcnt[wave][d] + at[r], kTile - 1)] = make_int2(key[r], val[r]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int t = r * kSortThreads + tid;
    if (t < ntile) {
      const int2 kv = tile[t];
      const int pos = min(max(gbase[(kv.x >> shift) & (NB - 1)] + t, 0), n - 1);
      kout[pos] = kv.x;
      vout[pos] = kv.y;
    }
  }
}

// CSR starts of the sorted keys: start[c] = first slot whose key is >= c,
// for c = 0 .. C (start[C] = n). Slot k writes the starts of the keys
// between its predecessor's key and its own; ranges of more than kOwnRange
// keys (empty regions, and sub-cells where there are many more than particles)
// are written by the whole wave (18.4M sub-cells, 4.2M slots: 62 -> 37 us).
constexpr int kOwnRange = 8;
__device__ __forceinline__ void fill_starts(int prev, int cur, int k, int32_t* __restrict__ start) {
  const bool own = cur - prev <= kOwnRange;
  if (own) {
    for (int c = prev + 1; c <= cur; ++c) start[c] = k;
  }
  const int lane = threadIdx.x & 63;
  for (uint64_t m = __ballot(!own); m; m &= m - 1) {
    const int l = __builtin_ctzll(m);
    const int p = __builtin_amdgcn_readlane(prev, l), q = __builtin_amdgcn_readlane(cur, l);
    const int kk = __builtin_amdgcn_readlane(k, l);
    for (int c = p + 1 + lane; c <= q; c += 64) start[c] = kk;
  }
}

// Cell ids of the sorted slots (key >> 3 sub_bits) and the CSR tables of
// cells and, with sub_bits > 0, of sub-cells, in one pass over the keys; also
// zero to the cells' largest h, for k_cell_hmax_sorted.
__global__ __launch_bounds__(kThreads) void k_cell_tables(const int32_t* __restrict__ skeys,
                                                           int n, int sub_bits, int C,
                                                           int32_t* __restrict__ cell,
                                                           int32_t* __restrict__ cell_start,
                                                           int32_t* __restrict__ sub_start,
                                                           float* __restrict__ hmax,
                                                           const int32_t* gate) {
  if (gated_off(gate)) return;
  const int k = blockIdx.x * kThreads + threadIdx.x;
  const int sh = 3 * sub_bits;
  const int key = k < n ? skeys[k] : (C << sh);
  const int pkey = k > n ? key : (k > 0 ? skeys[k - 1] : -1);   // past n: no range
  const int cur = key >> sh, prev = pkey >> sh;     // -1 >> sh is -1
  if (k < n && sub_bits) cell[k] = cur;
  fill_starts(prev, cur, k, cell_start);
  if (sub_bits) fill_starts(pkey, key, k, sub_start);
  if (hmax) {
    for (int c = blockIdx.x * kThreads + threadIdx.x; c < C; c += gridDim.x * kThreads)
      hmax[c] = 0.0f;
  }
}

// Largest h of each cell over its sorted slots: a thread per slot (h read
// through perm), a wave's slots of one cell combined first, so a cell's word
// takes one atomic per wave that holds slots of it; h >= 0, whose bits order as
// integers. A wave per cell instead took as long as its most crowded cell
// (4.2M slots, 287496 cells, us: 67, now 26; the zeroing is in k_cell_tables).
__global__ __launch_bounds__(kThreads) void k_cell_hmax_sorted(const int32_t* __restrict__ cell,
                                                                const int32_t* __restrict__ perm,
                                                                const float* __restrict__ hin,
                                                                int n, float* __restrict__ hmax,
                                                                const int32_t* gate) {
  if (gated_off(gate)) return;
  const int k = blockIdx.x * kThreads + threadIdx.x, lane = threadIdx.x & 63;
  const int c = k < n ? cell[k] : -1;
  int h = k < n ? __float_as_int(hin[perm[k]]) : 0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int oc = __shfl_up(c, o), oh = __shfl_up(h, o);
    if (lane >= o && oc == c) h = max(h, oh);
  }
  const int nc = __shfl_down(c, 1);
  if (k < n && (lane == 63 || nc != c)) atomicMax(reinterpret_cast<int*>(hmax) + c, h);
}

// Last kernel of a gated binning: [1] = whether this call rebuilt the list,
// [0] = 0 (the list now matches the records).
__global__ void k_rebin_done(int32_t* gate) {
  if (threadIdx.x == 0) {
    gate[1] = gate[0] != 0 ? 1 : 0;
    gate[0] = 0;
  }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct BinWs {
  int32_t *ka, *va, *kb, *vb, *hist;
  float* hin;   // h per input slot
};

// Workspace: four arrays of keys and values, the tiles' digit counts, h
size_t al(size_t b) { return (b + 255) & ~size_t(255); }
size_t hist_bytes(int n) {
  return al(sizeof(int32_t) * (size_t)kMaxBuckets * (size_t)std::max(cdiv(n, kTile), 1));
}

BinWs carve(void* ws, int n) {
  char* p = static_cast<char*>(ws);
  BinWs w;
  size_t nb = al(sizeof(int32_t) * (size_t)(n > 0 ? n : 1));
  w.ka = reinterpret_cast<int32_t*>(p); p += nb;
  w.va = reinterpret_cast<int32_t*>(p); p += nb;
  w.kb = reinterpret_cast<int32_t*>(p); p += nb;
  w.vb = reinterpret_cast<int32_t*>(p); p += nb;
  w.hist = reinterpret_cast<int32_t*>(p); p += hist_bytes(n);
  w.hin = reinterpret_cast<float*>(p);
  return w;
}

// One pass of the sort from (ks, vs) to (kd, vd); vs null: the indices
template <int D>
hipError_t radix_pass(const int32_t* ks, const int32_t* vs, int32_t* kd, int32_t* vd,
                      int32_t* hist, int n, int shift, const int32_t* gate, hipStream_t s) {
  const int nblk = cdiv(n, kTile);
  if (nblk > 1) {
    k_radix_hist<D><<<nblk, kSortThreads, 0, s>>>(ks, hist, n, shift, gate);
    k_radix_prefix<<<(1 << D) / kScanDigits, kSortThreads, 0, s>>>(hist, 1 << D, nblk, gate);
  }
  k_radix_scatter<D><<<nblk, kSortThreads, 0, s>>>(ks, vs, kd, vd, hist, n, shift, gate);
  return hipGetLastError();
}

}  // namespace

size_t bin_workspace_bytes(int n, int n_c, int sub_bits) {
  (void)n_c;
  (void)sub_bits;
  return 5 * al(sizeof(int32_t) * (size_t)(n > 0 ? n : 1)) + hist_bytes(n);
}

hipError_t launch_bin(const void* aos, const AosLayout& L, const CellsDev& c, int32_t* cell_start,
                      int32_t* perm, int32_t* cell, int32_t* sub_start, float* hmax, void* ws,
                      hipStream_t s) {
  const int n = c.n, n_c = c.n_c, sb = c.sub_bits;
  const int C = n_c * n_c * n_c;
  const int S = C << (3 * sb);
  BinWs w = carve(ws, n);
  const int32_t* gate = c.rebin;         // kept when no particle moved (may be null)
  const bool want_h = n > 0 && hmax && L.off[SPH_A_H] != kAbsent;
  int32_t* skeys = cell;                 // sorted keys (cell ids when sb == 0)
  if (n > 0) {
    // span of the record bytes the keys need: x, and h when hmax is wanted
    const uint32_t ox = L.off[SPH_A_X], oh = L.off[SPH_A_H];
    const uint32_t hsz = L.dt[SPH_A_H] == DT_F64 ? 8u : 4u;
    const uint32_t lo = (want_h ? min(ox, oh) : ox) & ~7u;
    const uint32_t hi = (max(ox + 24u, want_h ? oh + hsz : 0u) + 7u) & ~7u;
    const int nw = (hi - lo) / 8 <= (uint32_t)kSpanWords ? (int)((hi - lo) / 8) : 0;
    k_bin_keys<<<cdiv(n, kThreads), kThreads, 0, s>>>(
        static_cast<const char*>(aos), L.stride, ox, oh, L.dt[SPH_A_H], lo, nw, n, n_c, sb, w.ka,
        want_h ? w.hin : nullptr, c.status, gate);
    int bits = 1;
    while ((1 << bits) < S) ++bits;
    // 9-bit digits where they need fewer passes than 8-bit ones (keys of
    // 9, 17-18, 25-27 bits), else 8-bit digits
    const int passes = (bits + 8) / 9 < (bits + 7) / 8 ? (bits + 8) / 9 : (bits + 7) / 8;
    const int D = passes * 8 >= bits ? 8 : 9;
    int32_t *ks = w.ka, *vs = nullptr;
    for (int p = 0; p < passes; ++p) {
      int32_t* kd = ks == w.ka ? w.kb : w.ka;
      int32_t* vd = vs == w.vb ? w.va : w.vb;
      if (p == passes - 1) {
        kd = sb ? kd : cell;
        vd = perm;
      }
      const hipError_t e = D == 8 ? radix_pass<8>(ks, vs, kd, vd, w.hist, n, 8 * p, gate, s)
                                  : radix_pass<9>(ks, vs, kd, vd, w.hist, n, 9 * p, gate, s);
      if (e != hipSuccess) return e;
      ks = kd;
      vs = vd;
    }
    skeys = ks;
  }
  k_cell_tables<<<cdiv(n + 1, kThreads), kThreads, 0, s>>>(skeys, n, sb, C, cell, cell_start,
                                                           sub_start, hmax, gate);
  if (want_h)
    k_cell_hmax_sorted<<<cdiv(n, kThreads), kThreads, 0, s>>>(cell, perm, w.hin, n, hmax, gate);
  if (c.rebin) k_rebin_done<<<1, 64, 0, s>>>(c.rebin);
  return hipGetLastError();
}

}  // namespace sph
