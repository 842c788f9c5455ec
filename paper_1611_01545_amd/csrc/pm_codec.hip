// The compressed phase-space format of Sec. 2.4 on the GPU: encode from float
// particles, decode to bin centres, per-cell offsets of a compressed stream, the
// count/escape table, the byte stream and the float64 global reductions.
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "pm_codec.h"
#include "pm_scan.h"

using namespace pmscan;

namespace {

constexpr int T256 = 256;

__global__ void k_init_hdr(pm_shdr* h) {
  h->v_max = 0.f;
  h->j_min = 65536;
  h->j_max = -1;
  h->flags = 0;
  h->n_esc = 0;
  h->reserved = 0;
}

// ------------------------------------------------------------------------ encode --
// A stable LSD radix sort by cell whose items are the particles' codes themselves: the first
// pass reads x and v once, in order, and every pass moves whole records in runs. (Sorting
// indices and gathering x and v by them at the end fetched two cache lines per particle:
// 1.98 of 2.86 ms for 16.8 M particles in random order.)
//   k_encode_prep   v_max, the cell keys, the first pass's digit counts; clears the cell
//                   counts
//   k_sort_hist     digit counts of a later pass
//   k_sort_pass     one digit: ranks (a multi-split per wave, no barrier inside a wave's 512
//                   items), the tile ordered by digit in LDS, written in that order. The
//                   first pass makes the codes, the last one writes the species' arrays.
//   k_cell_counts   particles per cell, from the sorted keys
// Tiles of 4096 records in 76 KB of LDS (two on a CU): a digit's run of a tile is then 16
// records or more, which is 200 bytes written in one piece. The whole encode of 16.8 M
// particles takes 709 us (2860 with the gather).
constexpr int ST_T = 512, ST_I = 8, ST_TILE = ST_T * ST_I, ST_W = ST_T / 64;

__device__ __forceinline__ void load3(const float* p, float r[3]) {
  __builtin_memcpy(r, p, 12);
}

// v_max of a species: largest |v_a| (bit pattern of a non-negative float orders
// like an unsigned integer).
__global__ __launch_bounds__(ST_T) void k_encode_prep(const float* x, const float* v, int64_t n,
                                                     Geom g, uint32_t* keys, uint32_t mask,
                                                     uint32_t* hist, uint32_t* cnt, pm_shdr* h,
                                                     DevErr* err) {
  __shared__ uint32_t dc[256];
  __shared__ float wm[ST_W];
  if (threadIdx.x < 256) dc[threadIdx.x] = 0;
  if (cnt)
    for (int64_t i = (int64_t)blockIdx.x * ST_T + threadIdx.x; i < g.ncell3;
         i += (int64_t)gridDim.x * ST_T)
      cnt[i] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * ST_TILE + threadIdx.x;
  float m = 0.f;
  bool bad = false;
  float xx[ST_I][3], vv[ST_I][3];
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    const int64_t i = base + k * ST_T, j = i < n ? i : n - 1;  // n > 0
    load3(x + 3 * j, xx[k]);
    load3(v + 3 * j, vv[k]);
  }
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    const int64_t i = base + k * ST_T;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float q = fabsf(vv[k][a]);
      if (!(q <= 3.0e38f)) bad = true;
      else m = fmaxf(m, q);
    }
    uint32_t u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) bad |= !pos_code(xx[k][a], g.SL, g.S, u[a]);
    if (i < n) {
      const uint32_t key = cell_key(g, u[0] >> 8, u[1] >> 8, u[2] >> 8);
      keys[i] = key;
      atomicAdd(&dc[key & mask], 1u);
    }
  }
  for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x <= mask) hist[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = dc[threadIdx.x];
  if (threadIdx.x == 0) {
    for (int q = 1; q < ST_W; ++q) m = fmaxf(m, wm[q]);
    // most blocks find a larger one there: a plain read instead of an atomic
    const unsigned int b = __float_as_uint(m);
    unsigned int* vm = (unsigned int*)&h->v_max;
    if (b > __hip_atomic_load(vm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(vm, b);
  }
  if (bad) latch_error(err, ERRBIT_RANGE);
}

__global__ __launch_bounds__(ST_T) void k_sort_hist(const uint32_t* keys, int64_t n, int shift,
                                                   uint32_t mask, uint32_t* hist) {
  __shared__ uint32_t dc[256];
  if (threadIdx.x < 256) dc[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * ST_TILE + threadIdx.x;
  uint32_t key[ST_I];
#pragma unroll
  for (int k = 0; k < ST_I; ++k) key[k] = base + k * ST_T < n ? keys[base + k * ST_T] : 0u;
#pragma unroll
  for (int k = 0; k < ST_I; ++k)
    if (base + k * ST_T < n) atomicAdd(&dc[(key[k] >> shift) & mask], 1u);
  __syncthreads();
  if (threadIdx.x <= mask) hist[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = dc[threadIdx.x];
}

// The record of a particle: 3 P bytes of position codes, then 3 V of velocity codes, in words
// in LDS and registers. In memory every copy is a pair of arrays as a species holds them: one
// copy is the output itself, the other one the new codes of a step's re-sort, which are as
// large for as many particles. So an encode keeps no memory for records beyond a step's, and
// never replaces arrays that a captured step reads by larger ones. (Two buffers of records in
// whole words, 24 bytes a particle, take 761 us instead of 783 for 16.8 M particles.)
template <int P, int V>
constexpr int rec_words() { return (3 * (P + V) + 3) / 4; }

struct SortArgs {
  const float* x;  // first pass
  const float* v;
  Geom g;
  const uint32_t* kin;
  const void* pin;      // position and velocity codes (not the first pass)
  const void* vin;
  const uint32_t* iin;  // old indices (nullable)
  uint32_t* kout;
  void* pout;
  void* vout;
  uint32_t* iout;       // nullable: no permutation asked for
  const int64_t* hoff;  // destinations [digit][tile]
  int64_t n;
  int shift, bits;
  pm_shdr* h;
  int64_t* perm;        // last pass: nullable
};

// Codes in and out of a record's words at byte positions known at compile time. (A byte array
// filled in a function goes through scratch memory: first pass 157 us for 122.)
template <int B, int E>  // E bytes from byte B on
__device__ __forceinline__ void rec_put(uint32_t* w, uint32_t c) {
  w[B / 4] |= c << (8 * (B % 4));
  if constexpr (B % 4 + E > 4) w[B / 4 + 1] |= c >> (32 - 8 * (B % 4));
}
template <int B, int E>
__device__ __forceinline__ uint32_t rec_get(const uint32_t* w) {
  uint32_t c = w[B / 4] >> (8 * (B % 4));
  if constexpr (B % 4 + E > 4) c |= w[B / 4 + 1] << (32 - 8 * (B % 4));
  return c & ((1u << (8 * E)) - 1u);
}
template <int P, int V, typename PT, typename VT>
__device__ __forceinline__ void rec_load(uint32_t* w, const PT* p, const VT* v) {
#pragma unroll
  for (int q = 0; q < rec_words<P, V>(); ++q) w[q] = 0;
  rec_put<0, P>(w, p[0]);
  rec_put<P, P>(w, p[1]);
  rec_put<2 * P, P>(w, p[2]);
  rec_put<3 * P, V>(w, v[0]);
  rec_put<3 * P + V, V>(w, v[1]);
  rec_put<3 * P + 2 * V, V>(w, v[2]);
}
template <int P, int V, typename PT, typename VT>
__device__ __forceinline__ void rec_store(const uint32_t* w, PT* p, VT* v) {
  p[0] = (PT)rec_get<0, P>(w);
  p[1] = (PT)rec_get<P, P>(w);
  p[2] = (PT)rec_get<2 * P, P>(w);
  v[0] = (VT)rec_get<3 * P, V>(w);
  v[1] = (VT)rec_get<3 * P + V, V>(w);
  v[2] = (VT)rec_get<3 * P + 2 * V, V>(w);
}

template <int P, int V, bool FIRST>
__global__ __launch_bounds__(ST_T, 4) void k_sort_pass(SortArgs A) {
  using PT = typename PosCode<P>::T;
  using VT = typename VelCode<V>::T;
  constexpr int RW = rec_words<P, V>();
  __shared__ uint32_t skey[ST_TILE];       // the tile's keys, by digit
  __shared__ uint32_t srec[ST_TILE * RW];  // and records
  __shared__ uint32_t wcnt[ST_W][256];     // per wave: items per digit so far, then before it
  __shared__ int64_t dst0[256];            // destination of the digit's items less their slot
  __shared__ int wsum[ST_W];
  __shared__ int jmm[2];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t lt = lane ? ((~0ull) >> (64 - lane)) : 0ull;
  const uint32_t mask = (1u << A.bits) - 1u;
  for (int q = lane; q < 256; q += 64) wcnt[w][q] = 0;
  if (threadIdx.x == 0) {
    jmm[0] = 65536;
    jmm[1] = -1;
  }
  // an XCD's tiles follow one another: their runs of a digit are neighbours, which its L2 joins
  // into whole lines before they are written (16.8 M particles 782 -> 709 us)
  const int64_t tile = xcd_run(blockIdx.x, gridDim.x);
  // a wave's items are ST_I rounds of 64 consecutive ones
  const int64_t base = tile * ST_TILE + w * (64 * ST_I) + lane;
  const int64_t left = A.n - tile * ST_TILE;
  const int cnt = left < ST_TILE ? (int)left : ST_TILE;
  uint32_t key[ST_I], rec[ST_I][RW];
  int slot[ST_I];
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    const int64_t i = base + 64 * k, j = i < A.n ? i : A.n - 1;
    key[k] = A.kin[j];
    if constexpr (!FIRST) {
      rec_load<P, V>(rec[k], (const PT*)A.pin + 3 * j, (const VT*)A.vin + 3 * j);
    }
  }
  if constexpr (FIRST) {
    const int64_t S = A.g.S << (8 * (P - 1));
    const double SL = P == 1 ? A.g.SL : A.g.SL * 256.0;
    const float vmax = A.h->v_max;
    int jmn = 65536, jmx = -1;
    float xx[ST_I][3], vv[ST_I][3];
#pragma unroll
    for (int k = 0; k < ST_I; ++k) {
      const int64_t i = base + 64 * k, j = i < A.n ? i : A.n - 1;
      load3(A.x + 3 * j, xx[k]);
      load3(A.v + 3 * j, vv[k]);
    }
#pragma unroll
    for (int k = 0; k < ST_I; ++k) {
      PT pc[3];
      VT vc[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        uint32_t u;
        pos_code(xx[k][a], SL, S, u);
        const int c = vel_code_v<V>(vv[k][a], vmax);
        pc[a] = (PT)u;
        vc[a] = (VT)c;
        jmn = min(jmn, c);  // a repeated last particle changes nothing
        jmx = max(jmx, c);
      }
      rec_load<P, V>(rec[k], pc, vc);
    }
    for (int d = 32; d >= 1; d >>= 1) {
      jmn = min(jmn, __shfl_xor(jmn, d, 64));
      jmx = max(jmx, __shfl_xor(jmx, d, 64));
    }
    __syncthreads();  // jmm is set
    if (lane == 0) {
      atomicMin(&jmm[0], jmn);
      atomicMax(&jmm[1], jmx);
    }
  }
  // ranks inside the wave's items
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    const bool valid = base + 64 * k < A.n;
    const uint32_t d = (key[k] >> A.shift) & mask;
    uint64_t match = __ballot(valid);
    for (int b = 0; b < A.bits; ++b) {
      const uint64_t m = __ballot(valid && ((d >> b) & 1u));
      match &= ((d >> b) & 1u) ? m : ~m;
    }
    const uint32_t rk = (uint32_t)__popcll(match & lt);
    const uint32_t at = wcnt[w][d];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (valid && rk == 0) wcnt[w][d] = at + (uint32_t)__popcll(match);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    slot[k] = (int)(at + rk);
  }
  __syncthreads();
  // items of the digit in earlier waves, its first slot in the tile, its destination
  {
    uint32_t tot = 0;
    if (threadIdx.x < 256) {
#pragma unroll
      for (int q = 0; q < ST_W; ++q) {
        const uint32_t c = wcnt[q][threadIdx.x];
        wcnt[q][threadIdx.x] = tot;
        tot += c;
      }
    }
    const int start = block_excl_scan_i32((int)tot, wsum);
    if (threadIdx.x < 256) {
#pragma unroll
      for (int q = 0; q < ST_W; ++q) wcnt[q][threadIdx.x] += (uint32_t)start;
      if (threadIdx.x <= mask)
        dst0[threadIdx.x] = A.hoff[(int64_t)threadIdx.x * gridDim.x + tile] - start;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    if (base + 64 * k >= A.n) continue;
    slot[k] += (int)wcnt[w][(key[k] >> A.shift) & mask];
    skey[slot[k]] = key[k];
#pragma unroll
    for (int q = 0; q < RW; ++q) srec[RW * slot[k] + q] = rec[k][q];
  }
  __syncthreads();
  auto dest = [&](int sl) { return dst0[(skey[sl] >> A.shift) & mask] + sl; };
#pragma unroll
  for (int k = 0; k < ST_I; ++k) {
    const int sl = k * ST_T + (int)threadIdx.x;
    if (sl >= cnt) continue;
    const int64_t d = dest(sl);
    A.kout[d] = skey[sl];
    uint32_t rr[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) rr[q] = srec[RW * sl + q];
    rec_store<P, V>(rr, (PT*)A.pout + 3 * d, (VT*)A.vout + 3 * d);
  }
  if (A.iout || A.perm) {  // uniform: the old indices, the same way
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ST_I; ++k) {
      const int64_t i = base + 64 * k;
      if (i < A.n) srec[slot[k]] = FIRST ? (uint32_t)i : A.iin[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ST_I; ++k) {
      const int sl = k * ST_T + (int)threadIdx.x;
      if (sl >= cnt) continue;
      if (A.perm) A.perm[dest(sl)] = (int64_t)srec[sl];
      else A.iout[dest(sl)] = srec[sl];
    }
  }
  if constexpr (FIRST) {
    if (threadIdx.x == 0) {
      if (jmm[0] < __hip_atomic_load(&A.h->j_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMin(&A.h->j_min, jmm[0]);
      if (jmm[1] > __hip_atomic_load(&A.h->j_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&A.h->j_max, jmm[1]);
    }
  }
}

// Particles per cell: the lane that starts a wave's run of equal keys adds its length.
__global__ __launch_bounds__(T256) void k_cell_counts(const uint32_t* keys_sorted, int64_t n,
                                                     uint32_t* count32) {
  const int64_t j = (int64_t)blockIdx.x * T256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const uint32_t k = j < n ? keys_sorted[j] : 0xffffffffu;  // no cell key
  const uint32_t before = (uint32_t)__shfl_up((int)k, 1, 64);
  const bool head = lane == 0 || before != k;
  const uint64_t heads = __ballot(head);
  if (!head || j >= n) return;
  const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
  const int len = later ? __ffsll((unsigned long long)later) : 64 - lane;
  atomicAdd(&count32[k], (uint32_t)len);
}

// Per block of T256 cells: the byte counts, and the block's number of escapes in bcnt.
__global__ __launch_bounds__(T256) void k_count_bytes(const uint32_t* src, int64_t ncell,
                                                     uint8_t* count, uint32_t* bcnt) {
  const int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x;
  const uint32_t c = i < ncell ? src[i] : 0u;
  if (i < ncell) count[i] = (uint8_t)(c >= 255u ? 255u : c);
  const int ne = __syncthreads_count(c >= 255u);
  if (threadIdx.x == 0) bcnt[blockIdx.x] = (uint32_t)ne;
}

// The escape table in cell order: one thread per block of T256 cells writes that block's
// escapes from boff[b] (the exclusive prefix of the block counts, boff[nb] the total);
// blocks without escapes, nearly all of them, read one word.
__global__ __launch_bounds__(T256) void k_escapes(const uint32_t* src, int64_t ncell, int64_t nb,
                                                 const uint32_t* bcnt, const int64_t* boff,
                                                 uint64_t* esc, int64_t cap, pm_shdr* h,
                                                 DevErr* err) {
  const int64_t b = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (b == 0) {
    const int64_t ne = boff[nb];
    h->n_esc = ne;
    if (ne > cap) latch_error(err, ERRBIT_CAPACITY, ne);
  }
  if (b >= nb || bcnt[b] == 0) return;
  int64_t k = boff[b];
  const int64_t i1 = min((b + 1) * T256, ncell);
  for (int64_t i = b * T256; i < i1; ++i) {
    const uint32_t c = src[i];
    if (c >= 255u) {
      if (k < cap) {
        esc[2 * k] = (uint64_t)i;
        esc[2 * k + 1] = (uint64_t)c;
      }
      ++k;
    }
  }
}

__device__ inline int64_t find_cell(const int64_t* off, int64_t ncell, int64_t j) {
  // largest c with off[c] <= j (cells with zero particles are skipped)
  int64_t lo = 0, hi = ncell;  // off[lo] <= j < off[hi]
  while (hi - lo > 1) {
    int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= j) lo = mid; else hi = mid;
  }
  return lo;
}

template <int P, int V>
__global__ __launch_bounds__(T256) void k_decode(const void* pos_, const void* vel_,
                                                const pm_shdr* h, const int64_t* off,
                                                int64_t n, Geom g, float* x, float* v) {
  const typename PosCode<P>::T* pos = (const typename PosCode<P>::T*)pos_;
  const typename VelCode<V>::T* vel = (const typename VelCode<V>::T*)vel_;
  int64_t j = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (j >= n) return;
  uint32_t cell[3];
  key_cell(g, (uint32_t)find_cell(off, g.ncell3, j), cell[0], cell[1], cell[2]);
  float vmax = h->v_max;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const uint32_t u = (cell[a] << (8 * P)) | pos[3 * j + a];
    // 2-byte codes reach 2^26: the bin centre in float64, rounded once (as the 1-byte
    // form's float32 arithmetic is exact)
    x[3 * j + a] = P == 1 ? pos_decode(u, g.LS)
                          : (float)(((double)u + 0.5) * ((double)g.LS * 0x1p-8));
    v[3 * j + a] = vel_decode_v<V>(vel[3 * j + a], vmax);
  }
}

// ---------------------------------------------------------------- byte stream --
// Block sum of the checksum terms, stored at the block's index (integer: exact).
__device__ inline void block_sum_store(uint64_t s, uint64_t* part) {
  __shared__ uint64_t sm[T256 / 64];
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < T256 / 64; ++q) s += sm[q];
    part[blockIdx.x] = s;
  }
}

struct GetPackBytes {
  const int64_t* off;
  int64_t rb;  // record bytes: 3 (P + V)
  __device__ int64_t operator()(int64_t c) const {
    int64_t k = off[c + 1] - off[c];
    return 1 + (k >= 255 ? 4 : 0) + rb * k;
  }
};

__global__ __launch_bounds__(T256) void k_pack_cells(const int64_t* off, const int64_t* boff,
                                                    int64_t ncell, uint8_t* body,
                                                    int64_t cap_body, uint64_t* csum) {
  int64_t c = (int64_t)blockIdx.x * T256 + threadIdx.x;
  uint64_t s = 0;
  if (c < ncell && boff[ncell] <= cap_body) {
    int64_t k = off[c + 1] - off[c];
    int64_t o = boff[c];
    if (k >= 255) {
      uint8_t b[5] = {255, (uint8_t)(k & 255), (uint8_t)((k >> 8) & 255),
                      (uint8_t)((k >> 16) & 255), (uint8_t)((k >> 24) & 255)};
      for (int q = 0; q < 5; ++q) {
        body[o + q] = b[q];
        s += (2ull * (uint64_t)(o + q) + 1ull) * b[q];
      }
    } else {
      body[o] = (uint8_t)k;
      s += (2ull * (uint64_t)o + 1ull) * (uint64_t)k;
    }
  }
  block_sum_store(s, csum);
}

template <int P, int V>
__global__ __launch_bounds__(T256) void k_pack_records(const void* pos_, const void* vel_,
                                                      const int64_t* off, const int64_t* boff,
                                                      int64_t n, int64_t ncell, uint8_t* body,
                                                      int64_t cap_body, uint64_t* csum) {
  constexpr int RB = 3 * (P + V);  // record: x, y, z codes, then vx, vy, vz (little-endian)
  const typename PosCode<P>::T* pos = (const typename PosCode<P>::T*)pos_;
  const typename VelCode<V>::T* vel = (const typename VelCode<V>::T*)vel_;
  int64_t j = (int64_t)blockIdx.x * T256 + threadIdx.x;
  uint64_t s = 0;
  if (j < n && boff[ncell] <= cap_body) {
    int64_t c = find_cell(off, ncell, j);
    int64_t k = off[c + 1] - off[c];
    int64_t o = boff[c] + (k >= 255 ? 5 : 1) + RB * (j - off[c]);
    // counts inconsistent with n (latched by the offset check): write nothing
    if (o + RB > boff[ncell]) o = -1;
    uint8_t b[RB];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const uint32_t w = pos[3 * j + a];
#pragma unroll
      for (int q = 0; q < P; ++q) b[P * a + q] = (uint8_t)((w >> (8 * q)) & 255u);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const uint32_t w = vel[3 * j + a];
#pragma unroll
      for (int q = 0; q < V; ++q) b[3 * P + V * a + q] = (uint8_t)((w >> (8 * q)) & 255u);
    }
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      if (o < 0) break;
      body[o + q] = b[q];
      s += (2ull * (uint64_t)(o + q) + 1ull) * b[q];
    }
  }
  block_sum_store(s, csum);
}

// csum[0..nparts) -> csum[nparts] (sum mod 2^64, fixed order per thread, exact anyway)
__global__ __launch_bounds__(1024) void k_fold_sum(uint64_t* csum, int64_t nparts) {
  __shared__ uint64_t sm[16];
  uint64_t a = 0;
  for (int64_t i = threadIdx.x; i < nparts; i += 1024) a += csum[i];
  for (int d = 32; d >= 1; d >>= 1) a += __shfl_xor(a, d, 64);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < 16; ++q) a += sm[q];
    csum[nparts] = a;
  }
}

__global__ void k_pack_header(uint8_t* buf, int64_t cap, const int64_t* boff, int64_t ncell,
                              const uint64_t* csum, const pm_shdr* h, int32_t sid, int32_t B,
                              int64_t n, int64_t nc, double mass, uint32_t widths,
                              int64_t* used, DevErr* err) {
  int64_t body = boff[ncell];
  int64_t total = PM_STREAM_HEADER + body;
  *used = total;
  if (total > cap) {
    latch_error(err, ERRBIT_CAPACITY, total);
    return;
  }
  uint8_t hb[PM_STREAM_HEADER];
  for (int i = 0; i < PM_STREAM_HEADER; ++i) hb[i] = 0;
  auto put = [&](int o, const void* p, int len) {
    const uint8_t* q = (const uint8_t*)p;
    for (int i = 0; i < len; ++i) hb[o + i] = q[i];
  };
  const char magic[4] = {'P', 'M', 'C', '1'};
  uint32_t ver = 1, usid = (uint32_t)sid, ub = (uint32_t)B;
  const uint64_t cs = *csum;
  uint64_t un = (uint64_t)n, unc = (uint64_t)nc, ubl = (uint64_t)body;
  float vmax = h->v_max;
  put(0, magic, 4);
  put(4, &ver, 4);
  put(8, &usid, 4);
  put(12, &ub, 4);
  put(16, &un, 8);
  put(24, &unc, 8);
  put(32, &vmax, 4);
  put(36, &widths, 4);  // code widths, 0 for the paper's 1-byte positions, 2-byte velocities
  put(40, &mass, 8);
  put(48, &cs, 8);
  put(56, &ubl, 8);
  for (int i = 0; i < PM_STREAM_HEADER; ++i) buf[i] = hb[i];
}

// Checksum terms of body bytes [at, at + n), n of them at b: added to *csum (mod 2^64, so
// the order of the additions does not show). A thread takes 16 bytes in one load (b is
// 16-byte aligned).
constexpr int CS_BLOCKS = 2048;
__global__ __launch_bounds__(T256) void k_checksum(const uint8_t* b, int64_t n, int64_t at,
                                                  unsigned long long* csum) {
  uint64_t s = 0;
  for (int64_t i = ((int64_t)blockIdx.x * T256 + threadIdx.x) * 16; i < n;
       i += (int64_t)gridDim.x * T256 * 16) {
    if (i + 16 <= n) {
      const uint4 q = *(const uint4*)(b + i);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
      // sum (2 (at + i + k) + 1) b_k = (2 (at + i) + 1) sum b_k + 2 sum k b_k
      uint32_t s0 = 0, s1 = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const uint32_t v = (w[k >> 2] >> (8 * (k & 3))) & 255u;
        s0 += v;
        s1 += (uint32_t)k * v;
      }
      s += (2ull * (uint64_t)(at + i) + 1ull) * s0 + 2ull * s1;
    } else {
      for (int64_t k = i; k < n; ++k) s += (2ull * (uint64_t)(at + k) + 1ull) * b[k];
    }
  }
  __shared__ uint64_t sm[T256 / 64];
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < T256 / 64; ++q) s += sm[q];
    atomicAdd(csum, (unsigned long long)s);
  }
}

// Records of a byte stream into the species' arrays. A workgroup takes UT consecutive cells,
// whose first byte and first particle the host found as it walked the counts; the counts
// give the other cells' places. b: bytes from body byte `at` on; only the records that start
// in body bytes [at, end) are taken (all of them are there).
constexpr int UT = 64;
struct UnpackTile {
  int64_t byte, part;
};
template <int P, int V>
__global__ __launch_bounds__(T256) void k_unpack_cells(const uint8_t* b, int64_t at,
                                                      int64_t end, const UnpackTile* tiles,
                                                      int64_t cell0, int64_t ncell,
                                                      GetCount counts, void* pos_, void* vel_,
                                                      pm_shdr* h) {
  constexpr int RB = 3 * (P + V);
  typename PosCode<P>::T* pos = (typename PosCode<P>::T*)pos_;
  typename VelCode<V>::T* vel = (typename VelCode<V>::T*)vel_;
  __shared__ int64_t part[UT + 1], byte[UT];  // particles before a cell, its first record
  __shared__ int smn[T256 / 64], smx[T256 / 64];
  const UnpackTile t = tiles[blockIdx.x];
  const int64_t c0 = cell0 + (int64_t)blockIdx.x * UT;
  if (threadIdx.x < UT) {
    const int64_t c = c0 + threadIdx.x;
    const int64_t k = c < ncell ? counts(c) : 0;
    const int64_t len = c < ncell ? 1 + (k >= 255 ? 4 : 0) + RB * k : 0;
    const int64_t pk = wave_incl_scan(k), pl = wave_incl_scan(len);
    if (threadIdx.x == 0) part[0] = 0;
    part[threadIdx.x + 1] = pk;
    byte[threadIdx.x] = pl - RB * k;
  }
  __syncthreads();
  const uint8_t* src = b + (t.byte - at);
  int jmin = 65536, jmax = -1;
  // the tile's first record that starts at body byte p or later
  auto first_from = [&](int64_t p) -> int64_t {
    p -= t.byte;
    int c = 0;
#pragma unroll
    for (int d = UT / 2; d >= 1; d >>= 1) c += byte[c + d] <= p ? d : 0;
    const int64_t k = p > byte[c] ? (p - byte[c] + RB - 1) / RB : 0;
    return min(part[c] + k, part[c + 1]);
  };
  const int64_t q1 = first_from(end);
  for (int64_t q = first_from(at) + threadIdx.x; q < q1; q += T256) {
    int lo = 0;  // the largest cell with part[lo] <= q
#pragma unroll
    for (int d = UT / 2; d >= 1; d >>= 1) lo += part[lo + d] <= q ? d : 0;
    uint8_t r[RB];
    __builtin_memcpy(r, src + byte[lo] + RB * (q - part[lo]), RB);  // unaligned loads
    const int64_t j = t.part + q;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      uint32_t u = r[P * a], w = r[3 * P + V * a];
      if constexpr (P == 2) u |= (uint32_t)r[P * a + 1] << 8;
      if constexpr (V == 2) w |= (uint32_t)r[3 * P + V * a + 1] << 8;
      pos[3 * j + a] = (typename PosCode<P>::T)u;
      vel[3 * j + a] = (typename VelCode<V>::T)w;
      jmin = min(jmin, (int)w);
      jmax = max(jmax, (int)w);
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    jmin = min(jmin, __shfl_xor(jmin, d, 64));
    jmax = max(jmax, __shfl_xor(jmax, d, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    smn[threadIdx.x >> 6] = jmin;
    smx[threadIdx.x >> 6] = jmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < T256 / 64; ++q) {
      jmin = min(jmin, smn[q]);
      jmax = max(jmax, smx[q]);
    }
    // most workgroups find the extremes there already: a plain read instead of an atomic
    if (jmin < __hip_atomic_load(&h->j_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMin(&h->j_min, jmin);
    if (jmax > __hip_atomic_load(&h->j_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&h->j_max, jmax);
  }
}

// ------------------------------------------------------------------ reductions --
constexpr int RED_BLOCKS = 512;

__global__ __launch_bounds__(T256) void k_reduce_mesh(const float* rho, int64_t n,
                                                     double* part) {
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * T256)
    s += (double)rho[i];
  __shared__ double lw[T256 / 64];
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0) lw[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = lw[0] + lw[1] + lw[2] + lw[3];
}

// Per block: sum of v and of the CIC-interpolated acceleration a_i over one species'
// particles (decoded bin centres for compressed streams), in float64, stored at the
// block's index. off: cell offsets of a compressed stream (finds each particle's cell).
struct RedSpecies {
  pm_species sp;
  const int64_t* off;
};

__device__ inline void cic_accumulate(const float* acc, int64_t ng, const float xm[3],
                                      double a[3]) {
  int64_t i[3];
  float f[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float fl = floorf(xm[q]);
    f[q] = xm[q] - fl;
    int64_t k = (int64_t)fl % ng;
    i[q] = k < 0 ? k + ng : k;
  }
  const int64_t n3 = ng * ng * ng;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const float w = (dx ? f[0] : 1.f - f[0]) * (dy ? f[1] : 1.f - f[1]) *
                        (dz ? f[2] : 1.f - f[2]);
        const int64_t node = (((i[2] + dz) % ng) * ng + (i[1] + dy) % ng) * ng +
                             (i[0] + dx) % ng;
#pragma unroll
        for (int q = 0; q < 3; ++q) a[q] += (double)(w * acc[q * n3 + node]);
      }
}

template <int P, int V>
__global__ __launch_bounds__(T256) void k_reduce_particles(RedSpecies rs, const float* acc,
                                                          Geom g, double* part) {
  const pm_species& sp = rs.sp;
  const typename PosCode<P>::T* pos = (const typename PosCode<P>::T*)sp.pos;
  const typename VelCode<V>::T* vel = (const typename VelCode<V>::T*)sp.vel;
  double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const float fng = g.ngL;
  const float rs_cell = (float)g.r / 256.f;  // mesh cells per 1-byte position quantum
  for (int64_t j = (int64_t)blockIdx.x * T256 + threadIdx.x; j < sp.n;
       j += (int64_t)gridDim.x * T256) {
    float xm[3];
    if (sp.layout == PM_FLOAT) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s[a] += (double)sp.v[3 * j + a];
        xm[a] = sp.x[3 * j + a] * fng;  // mesh units (exact for a power-of-two box)
      }
    } else {
      uint32_t cell[3];
      key_cell(g, (uint32_t)find_cell(rs.off, g.ncell3, j), cell[0], cell[1], cell[2]);
      const float vmax = sp.hdr->v_max;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s[a] += (double)vel_decode_v<V>(vel[3 * j + a], vmax);
        const uint32_t u = (cell[a] << (8 * P)) | pos[3 * j + a];
        // bin centre in mesh units: exact in float32 for 1-byte codes, in float64 (then
        // rounded once) for 2-byte codes
        xm[a] = P == 1 ? ((float)u + 0.5f) * rs_cell
                       : (float)(((double)u + 0.5) * ((double)g.r * 0x1p-16));
      }
    }
    if (acc) cic_accumulate(acc, g.ng, xm, s + 3);
  }
  __shared__ double lw[6][T256 / 64];
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    for (int d = 32; d >= 1; d >>= 1) s[a] += __shfl_xor(s[a], d, 64);
    if ((threadIdx.x & 63) == 0) lw[a][threadIdx.x >> 6] = s[a];
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int a = threadIdx.x;
    part[6 * blockIdx.x + a] = lw[a][0] + lw[a][1] + lw[a][2] + lw[a][3];
  }
}

struct RedMeta {
  int n_sp;
  double mass[4];
  int64_t count[4];
};

// Fixed-order final sums (deterministic). out[0] mesh mass, out[1] particle mass,
// out[2..4] total momentum, out[5..7] total sum m a; per species s, out[8 + 6 s ..] =
// m_s sum v (3) and m_s sum a (3).
__global__ void k_reduce_final(const double* pmesh, int nmesh_part, double cell_vol,
                               const double* ppart, RedMeta meta, double* out) {
  double m = 0.0;
  for (int i = 0; i < nmesh_part; ++i) m += pmesh[i];
  out[0] = m * cell_vol;
  double mt = 0.0, tot[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int s = 0; s < meta.n_sp; ++s) {
    mt += meta.mass[s] * (double)meta.count[s];
    double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int b = 0; b < RED_BLOCKS; ++b) {
      const double* q = ppart + 6 * (int64_t)(s * RED_BLOCKS + b);
      for (int a = 0; a < 6; ++a) sum[a] += q[a];
    }
    for (int a = 0; a < 6; ++a) {
      out[8 + 6 * s + a] = meta.mass[s] * sum[a];
      tot[a] += meta.mass[s] * sum[a];
    }
  }
  out[1] = mt;
  for (int a = 0; a < 6; ++a) out[2 + a] = tot[a];
}

}  // namespace

// cell offsets of compressed streams and the check that the counts sum to n; bsum
// (nullable) holds the scan's block sums
static pm_status scan_counts_into(pm_context* c, const pm_species* sp, int n_sp,
                                  int64_t* const* off, int64_t* bsum) {
  ScanArgs<GetCount> A{};
  for (int s = 0; s < n_sp; ++s) {
    A.g[s] = GetCount{sp[s].count, sp[s].esc, sp[s].hdr};
    A.out[s] = off[s];
    A.want[s] = sp[s].n;
  }
  A.err = c->err;
  return scan_batch(c, A, n_sp, c->g.ncell3, bsum);
}

pm_status run_cell_offsets(pm_context* c, const pm_species* sp, int64_t* off) {
  ProfScope ps(c, ST_OFFSETS);
  return scan_counts_into(c, sp, 1, &off, nullptr);
}

pm_status run_species_offsets(pm_context* c, const pm_species* sp, int n_sp, int64_t** offs) {
  for (int s = 0; s < n_sp; ++s) {
    offs[s] = (int64_t*)scratch(c, SC_SPOFF0 + s, (size_t)(c->g.ncell3 + 1) * 8);
    if (!offs[s]) return PM_ERR_NOMEM;
  }
  ProfScope ps(c, ST_OFFSETS);
  return scan_counts_into(c, sp, n_sp, offs, nullptr);
}

pm_status run_finalize_counts(pm_context* c, const uint32_t* cnt32, pm_species* out) {
  const int64_t nc3 = c->g.ncell3;
  const int64_t nb = cdiv(nc3, T256);  // blocks of T256 cells
  uint32_t* bcnt = (uint32_t*)scratch(c, SC_FLAG, (size_t)nb * 4);
  int64_t* boff = (int64_t*)scratch(c, SC_FOFF, (size_t)(nb + 1) * 8);
  if (!bcnt || !boff) return PM_ERR_NOMEM;
  hipLaunchKernelGGL(k_count_bytes, dim3((unsigned)nb), dim3(T256), 0, c->stream, cnt32, nc3,
                     out->count, bcnt);
  PM_LAUNCH_CHECK();
  pm_status s = scan_u32(c, bcnt, nb, boff);
  if (s != PM_OK) return s;
  hipLaunchKernelGGL(k_escapes, dim3((unsigned)cdiv(nb, T256)), dim3(T256), 0, c->stream, cnt32,
                     nc3, nb, bcnt, boff, out->esc, out->cap_esc, out->hdr, c->err);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_encode(pm_context* c, const pm_species* in, pm_species* out, int64_t* perm) {
  ProfScope ps(c, ST_CODEC);
  const int64_t n = in->n;
  const Geom& g = c->g;
  hipLaunchKernelGGL(k_init_hdr, dim3(1), dim3(1), 0, c->stream, out->hdr);
  PM_LAUNCH_CHECK();
  uint32_t* cnt32 = (uint32_t*)scratch(c, SC_COUNT32, (size_t)g.ncell3 * 4);
  if (!cnt32) return PM_ERR_NOMEM;
  pm_status s;
  if (n == 0) {
    if ((s = launch_fill_u32(c, cnt32, g.ncell3, 0u)) != PM_OK) return s;
  } else {
    // digits of equal width, at most 8 bits (one pass of none for a single cell)
    const int bits = 3 * (g.lgB + g.lgnb);
    const int passes = bits > 8 ? (bits + 7) / 8 : 1, width = (bits + passes - 1) / passes;
    const int64_t nt = cdiv(n, ST_TILE);
    const uint32_t mask = (1u << width) - 1u;
    uint32_t* key[2] = {(uint32_t*)scratch(c, SC_KEYA, (size_t)n * 4),
                        (uint32_t*)scratch(c, SC_KEYB, (size_t)n * 4)};
    uint32_t* idx[2] = {nullptr, nullptr};
    bool have = key[0] && key[1];
    for (int q = 0; q < 2 && q < passes - 1 && perm; ++q)
      have = have && (idx[q] = (uint32_t*)scratch(c, q ? SC_VALB : SC_VALA, (size_t)n * 4));
    // the passes write the output and the scratch copy in turn, the last one the output
    void *cpos = nullptr, *cvel = nullptr;
    if (passes > 1) {
      cpos = scratch(c, SC_TPOS, (size_t)n * 3 * width_pos(*out));
      cvel = scratch(c, SC_TVEL, (size_t)n * 3 * width_vel(*out));
      have = have && cpos && cvel;
    }
    // digit counts, and behind their prefixes the scan's block sums (not in the scratch that
    // a step's scans use: the counts of many particles on few cells need more)
    uint32_t* hist = (uint32_t*)scratch(c, SC_HIST, (size_t)nt * 256 * 4);
    const int64_t nh = nt * 256 + 1;
    int64_t* hoff = (int64_t*)scratch(c, SC_HOFF, (size_t)(nh + cdiv(nh, SCAN_TILE)) * 8);
    if (!have || !hist || !hoff) return PM_ERR_NOMEM;
    // many more cells than particles: cleared by a grid of their own
    const bool apart = g.ncell3 > 4 * nt * ST_TILE;
    if (apart && (s = launch_fill_u32(c, cnt32, g.ncell3, 0u)) != PM_OK) return s;
    hipLaunchKernelGGL(k_encode_prep, dim3((unsigned)nt), dim3(ST_T), 0, c->stream, in->x, in->v,
                       n, g, key[0], mask, hist, apart ? nullptr : cnt32, out->hdr, c->err);
    PM_LAUNCH_CHECK();
    SortArgs A{};
    A.x = in->x;
    A.v = in->v;
    A.g = g;
    A.hoff = hoff;
    A.n = n;
    A.bits = width;
    A.h = out->hdr;
    for (int p = 0; p < passes; ++p) {
      const bool first = p == 0, last = p == passes - 1;
      A.shift = p * width;
      A.kin = key[p & 1];
      A.kout = key[(p + 1) & 1];
      const bool to_out = (passes - 1 - p) % 2 == 0;
      A.pin = to_out ? cpos : (void*)out->pos;
      A.vin = to_out ? cvel : (void*)out->vel;
      A.pout = to_out ? (void*)out->pos : cpos;
      A.vout = to_out ? (void*)out->vel : cvel;
      A.iin = first ? nullptr : idx[(p - 1) & 1];
      A.iout = last ? nullptr : idx[p & 1];
      A.perm = last ? perm : nullptr;
      if (!first)
        hipLaunchKernelGGL(k_sort_hist, dim3((unsigned)nt), dim3(ST_T), 0, c->stream, A.kin, n,
                           A.shift, mask, hist);
      if ((s = scan_u32(c, hist, nt * ((int64_t)mask + 1), hoff, hoff + nh)) != PM_OK) return s;
      s = width_dispatch(width_kind(*out), [&](auto P_, auto V_) {
        constexpr int P = decltype(P_)::value, V = decltype(V_)::value;
        auto launch = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, dim3((unsigned)nt), dim3(ST_T), 0, c->stream, A);
        };
        if (first) launch(k_sort_pass<P, V, true>);
        else launch(k_sort_pass<P, V, false>);
        return PM_OK;
      });
      if (s != PM_OK) return s;
      PM_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_cell_counts, dim3((unsigned)cdiv(n, T256)), dim3(T256), 0, c->stream,
                       (const uint32_t*)A.kout, n, cnt32);
    PM_LAUNCH_CHECK();
  }
  return run_finalize_counts(c, cnt32, out);
}

pm_status run_decode(pm_context* c, const pm_species* in, pm_species* out) {
  const int64_t n = in->n;
  int64_t* off = (int64_t*)scratch(c, SC_OFF, (size_t)(c->g.ncell3 + 1) * 8);
  if (!off) return PM_ERR_NOMEM;
  pm_status s = run_cell_offsets(c, in, off);
  if (s != PM_OK || n == 0) return s;
  s = width_dispatch(width_kind(*in), [&](auto P_, auto V_) {
    hipLaunchKernelGGL((k_decode<decltype(P_)::value, decltype(V_)::value>),
                       dim3((unsigned)cdiv(n, T256)), dim3(T256), 0, c->stream,
                       (const void*)in->pos, (const void*)in->vel, in->hdr, off, n, c->g,
                       out->x, out->v);
    return PM_OK;
  });
  if (s != PM_OK) return s;
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_pack(pm_context* c, const pm_species* sp, int32_t sid, uint8_t* buf,
                   int64_t cap, int64_t* used) {
  const int64_t nc3 = c->g.ncell3;
  int64_t* off = (int64_t*)scratch(c, SC_OFF, (size_t)(nc3 + 1) * 8);
  int64_t* boff = (int64_t*)scratch(c, SC_FOFF, (size_t)(nc3 + 1) * 8);
  const int64_t nbc = cdiv(nc3, T256), nbr = cdiv(sp->n, T256);
  uint64_t* csum = (uint64_t*)scratch(c, SC_PARTS, (size_t)(nbc + nbr + 1) * 8);
  if (!off || !boff || !csum) return PM_ERR_NOMEM;
  pm_status s = run_cell_offsets(c, sp, off);
  if (s != PM_OK) return s;
  const int64_t rb = 3 * (width_pos(*sp) + width_vel(*sp));
  s = scan_generic_pack(c, off, nc3, boff, rb);
  if (s != PM_OK) return s;
  int64_t cap_body = cap - PM_STREAM_HEADER;
  uint8_t* body = buf + PM_STREAM_HEADER;
  hipLaunchKernelGGL(k_pack_cells, dim3((unsigned)nbc), dim3(T256), 0, c->stream,
                     off, boff, nc3, body, cap_body, csum);
  if (nbr > 0) {
    s = width_dispatch(width_kind(*sp), [&](auto P_, auto V_) {
      hipLaunchKernelGGL((k_pack_records<decltype(P_)::value, decltype(V_)::value>),
                         dim3((unsigned)nbr), dim3(T256), 0, c->stream, (const void*)sp->pos,
                         (const void*)sp->vel, off, boff, sp->n, nc3, body, cap_body,
                         csum + nbc);
      return PM_OK;
    });
    if (s != PM_OK) return s;
  }
  hipLaunchKernelGGL(k_fold_sum, dim3(1), dim3(1024), 0, c->stream, csum, nbc + nbr);
  hipLaunchKernelGGL(k_pack_header, dim3(1), dim3(1), 0, c->stream, buf, cap, boff, nc3,
                     csum + nbc + nbr, sp->hdr, sid, c->g.B, sp->n, c->g.nc, sp->mass,
                     (uint32_t)sp->widths, used, c->err);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

namespace {
// What the host finds in a stream body: every cell's count byte and escape, and where each
// run of UT cells starts. False: the counts do not fit the body or the particle number.
struct BodyWalk {
  std::vector<uint8_t> count;
  std::vector<uint64_t> esc;
  std::vector<UnpackTile> tiles;
  int64_t largest = 0;  // bytes of the longest run
  bool ok = false, nomem = false;
  void run(const uint8_t* body, int64_t blen, int64_t ncell, uint64_t n, uint64_t rb) try {
    count.resize((size_t)ncell);
    tiles.reserve((size_t)cdiv(ncell, UT) + 1);
    const uint64_t len = (uint64_t)blen;
    uint64_t off = 0, p = 0;
    for (int64_t c = 0; c < ncell; ++c) {
      if (c % UT == 0) tiles.push_back({(int64_t)off, (int64_t)p});
      if (off >= len) return;
      uint64_t k = body[off++];
      if (k == 255) {
        if (off + 4 > len) return;
        uint32_t kk;
        std::memcpy(&kk, body + off, 4);
        off += 4;
        if (kk < 255) return;
        k = kk;
        esc.push_back((uint64_t)c);
        esc.push_back(k);
      }
      count[(size_t)c] = (uint8_t)(k >= 255 ? 255 : k);
      if (p + k > n || off + rb * k > len) return;
      p += k;
      off += rb * k;
    }
    tiles.push_back({(int64_t)off, (int64_t)p});
    for (size_t t = 1; t < tiles.size(); ++t)
      largest = std::max(largest, tiles[t].byte - tiles[t - 1].byte);
    ok = p == n && off == len;
  } catch (const std::bad_alloc&) {
    nomem = true;
  }
};
struct DevMem {
  void* p = nullptr;
  ~DevMem() {
    if (p) hipFree(p);
  }
};
// Device memory of an unpack: a table of cell runs, the checksum, and room for stream bytes
struct UnpackRoom {
  UnpackTile* tab;
  uint64_t* sum;
  uint8_t* buf;
  int64_t tabs, size;
  UnpackRoom(void* p, int64_t n, int64_t bytes) : tabs(n), size(bytes) {
    tab = (UnpackTile*)p;
    sum = (uint64_t*)(tab + n);
    buf = (uint8_t*)(sum + 2);
  }
  static size_t need(int64_t n, int64_t bytes) {
    return (size_t)n * sizeof(UnpackTile) + 16 + (size_t)bytes;
  }
};
constexpr int64_t ROOM_TABS = 4096, ROOM_BYTES = (int64_t)1 << 20;  // the context's own
}  // namespace

size_t unpack_room_bytes() { return UnpackRoom::need(ROOM_TABS, ROOM_BYTES); }

// Only the chain of counts is sequential: the host follows it (one byte per cell) while the
// body goes to the GPU, which sums it and takes the records apart. Two species of 256^3 and
// 128^3 particles on 128^3 cells (176 MB), with their decode: 11.2 ms, against 178 ms with
// the host's parse of every byte. What is left is the walk and the upload from pageable memory
// (30 GB/s), which run side by side. Bodies up to 1 MB go through the context's own room,
// larger ones through an allocation of up to 256 MB for the call, or, where the card has none
// left, through that room too; a body beyond the room goes through it in pieces, once to be
// summed and once to be parsed. Nothing of the destination is written before everything that
// can be refused has been looked at.
pm_status run_unpack(pm_context* c, const uint8_t* body, int64_t blen, uint64_t csum,
                     float vmax, pm_species* out) {
  constexpr int64_t CHUNK = (int64_t)256 << 20, CHUNK_TABS = 65536;
  const int64_t ncell = c->g.ncell3;
  const int P = width_pos(*out), V = width_vel(*out);
  BodyWalk w;
  std::thread helper;
  const bool apart = blen >= (1 << 20);  // a thread costs more than a short walk
  auto walk = [&] { w.run(body, blen, ncell, (uint64_t)out->n, 3 * (uint64_t)(P + V)); };
  bool walked = false;
  if (apart) {
    try {
      helper = std::thread(walk);
      walked = true;
    } catch (...) {
    }
  }
  struct Join {
    std::thread& t;
    ~Join() {
      if (t.joinable()) t.join();
    }
  } join{helper};
  if (!walked) walk();

  UnpackRoom r(c->room, ROOM_TABS, ROOM_BYTES);
  DevMem more;
  if (blen > r.size) {
    const int64_t tabs = std::min(cdiv(ncell, UT), CHUNK_TABS), size = std::min(blen, CHUNK);
    if (hipMalloc(&more.p, UnpackRoom::need(tabs, size)) == hipSuccess) {
      r = UnpackRoom(more.p, tabs, size);
    } else {
      more.p = nullptr;
      (void)hipGetLastError();
    }
  }
  auto up = [&](void* d, const void* s, int64_t n) {
    return hipMemcpyAsync(d, s, (size_t)n, hipMemcpyHostToDevice, c->stream);
  };
  hipLaunchKernelGGL(k_fill<uint64_t>, dim3(1), dim3(64), 0, c->stream, r.sum, (int64_t)1,
                     (uint64_t)0);
  for (int64_t at = 0; at < blen; at += r.size) {
    const int64_t n = std::min(r.size, blen - at);
    PM_HIP_CHECK(up(r.buf, body + at, n));
    hipLaunchKernelGGL(k_checksum, dim3((unsigned)std::min<int64_t>(cdiv(n, 16 * T256), CS_BLOCKS)),
                       dim3(T256), 0, c->stream, (const uint8_t*)r.buf, n, at,
                       (unsigned long long*)r.sum);
    PM_LAUNCH_CHECK();
  }
  uint64_t got = 0;
  PM_HIP_CHECK(hipMemcpyAsync(&got, r.sum, 8, hipMemcpyDeviceToHost, c->stream));
  PM_HIP_CHECK(hipStreamSynchronize(c->stream));
  if (helper.joinable()) helper.join();
  if (w.nomem) return PM_ERR_NOMEM;
  if (got != csum || !w.ok) return PM_ERR_CORRUPT;
  const int64_t n_esc = (int64_t)w.esc.size() / 2;
  if (n_esc > out->cap_esc) {
    c->last_detail = n_esc;
    return PM_ERR_CAPACITY;
  }

  pm_shdr h{};
  h.v_max = vmax;
  h.j_min = 65536;
  h.j_max = -1;
  h.n_esc = n_esc;
  PM_HIP_CHECK(up(out->hdr, &h, sizeof(h)));
  PM_HIP_CHECK(up(out->count, w.count.data(), ncell));
  if (n_esc > 0) PM_HIP_CHECK(up(out->esc, w.esc.data(), n_esc * 16));
  const int64_t nt = (int64_t)w.tiles.size() - 1;
  const int64_t over = 3 * (P + V) - 1;  // bytes of a record that may lie beyond a piece
  pm_status st = PM_OK;
  for (int64_t at = 0, t0 = 0, t1 = 0; st == PM_OK && out->n > 0 && at < blen;) {
    const int64_t n = std::min(r.size, blen - at);
    const int64_t end = at + n == blen ? blen : at + n - over;
    if (blen > r.size && up(r.buf, body + at, n) != hipSuccess) st = PM_ERR_DEVICE;
    while (t0 < nt && w.tiles[t0 + 1].byte <= at) ++t0;
    while (t1 < nt && w.tiles[t1].byte < end) ++t1;
    for (int64_t t = t0; t < t1 && st == PM_OK; t += r.tabs) {
      const int64_t m = std::min(r.tabs, t1 - t);
      if (up(r.tab, w.tiles.data() + t, m * (int64_t)sizeof(UnpackTile)) != hipSuccess) {
        st = PM_ERR_DEVICE;
        break;
      }
      st = width_dispatch(width_kind(*out), [&](auto P_, auto V_) {
        hipLaunchKernelGGL((k_unpack_cells<decltype(P_)::value, decltype(V_)::value>),
                           dim3((unsigned)m), dim3(T256), 0, c->stream, (const uint8_t*)r.buf, at,
                           end, (const UnpackTile*)r.tab, t * UT, ncell,
                           GetCount{out->count, out->esc, out->hdr}, (void*)out->pos,
                           (void*)out->vel, out->hdr);
        return hipGetLastError() == hipSuccess ? PM_OK : PM_ERR_DEVICE;
      });
    }
    at = end;
  }
  if (hipStreamSynchronize(c->stream) != hipSuccess && st == PM_OK) st = PM_ERR_DEVICE;
  return st;
}

pm_status scan_generic_pack(pm_context* c, const int64_t* off, int64_t n, int64_t* out,
                            int64_t rb) {
  return scan_generic(c, GetPackBytes{off, rb}, n, out);
}

namespace {
// Float64 reductions with the caller's choice of buffers: part (RED_BLOCKS * 25 doubles),
// off_of(s) the cell offsets of compressed species s ((ncell3 + 1) int64), bsum the scan's
// block sums (nullptr: the context's scratch).
template <typename OffOf>
pm_status reduce_core(pm_context* c, const pm_species* sp, int n_sp, const float* rho,
                      const float* acc, double* out, double* part, OffOf off_of,
                      int64_t* bsum) {
  if (n_sp < 0 || n_sp > 4) return PM_ERR_ARG;
  double* pmesh = part;
  double* ppart = part + RED_BLOCKS;
  RedMeta meta{};
  meta.n_sp = n_sp;
  int nmp = 0;
  if (rho) {
    nmp = RED_BLOCKS;
    hipLaunchKernelGGL(k_reduce_mesh, dim3(RED_BLOCKS), dim3(T256), 0, c->stream, rho,
                       c->g.ng * c->g.ng * c->g.ng, pmesh);
  }
  for (int s = 0; s < n_sp; ++s) {
    meta.mass[s] = sp[s].mass;
    meta.count[s] = sp[s].n;
    RedSpecies rs{sp[s], nullptr};
    if (sp[s].layout == PM_COMPRESSED) {
      int64_t* off = off_of(s);
      if (!off) return PM_ERR_NOMEM;
      pm_status st = scan_counts_into(c, &sp[s], 1, &off, bsum);
      if (st != PM_OK) return st;
      rs.off = off;
    }
    double* pp = ppart + 6 * (int64_t)s * RED_BLOCKS;
    const int kind = sp[s].layout == PM_COMPRESSED ? width_kind(sp[s]) : 0;
    pm_status st = width_dispatch(kind, [&](auto P_, auto V_) {
      hipLaunchKernelGGL((k_reduce_particles<decltype(P_)::value, decltype(V_)::value>),
                         dim3(RED_BLOCKS), dim3(T256), 0, c->stream, rs, acc, c->g, pp);
      return PM_OK;
    });
    if (st != PM_OK) return st;
  }
  const double dv = c->g.box * c->g.box * c->g.box / ((double)c->g.ng * c->g.ng * c->g.ng);
  hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(1), 0, c->stream, pmesh, nmp, dv, ppart,
                     meta, out);
  PM_LAUNCH_CHECK();
  return PM_OK;
}
}  // namespace

pm_status run_reduce(pm_context* c, const pm_species* sp, int n_sp, const float* rho,
                     const float* acc, double* out) {
  double* part = (double*)scratch(c, SC_MISC, (size_t)(RED_BLOCKS * (6 * 4 + 1)) * 8);
  if (!part) return PM_ERR_NOMEM;
  return reduce_core(c, sp, n_sp, rho, acc, out, part, [&](int s) {
    return (int64_t*)scratch(c, SC_SPOFF0 + s, (size_t)(c->g.ncell3 + 1) * 8);
  }, nullptr);
}

// ------------------------------------------------------- allocation-free reduce --
// For callers that cannot allocate device memory. Every buffer of pm_reduce_noalloc lives
// in one fixed array per device: the per-workgroup partial sums, the cell offsets of one
// compressed species at a time (species are reduced one after the other on the stream)
// and the block sums of their scan. Its device address is taken once per device, when a
// context is created there; calls that overlap on one device share the array and race.
namespace noalloc {
constexpr int64_t NC3_MAX = 32768;  // compressed species: n_cell^3 <= 32^3
constexpr size_t PART_BYTES = (size_t)RED_BLOCKS * (6 * 4 + 1) * 8;
constexpr size_t OFF_BYTES = (size_t)(NC3_MAX + 1) * 8;
constexpr size_t BSUM_BYTES = 256;  // cdiv(NC3_MAX + 1, 4096) int64 block sums
constexpr size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }
constexpr size_t BYTES = a256(PART_BYTES) + a256(OFF_BYTES) + BSUM_BYTES;
static __device__ __align__(256) unsigned char scratch[BYTES];

std::mutex mu;
unsigned char* addr[256] = {};
}  // namespace noalloc

pm_status noalloc_init(pm_context* c) {
  if (c->device < 0 || c->device >= 256) return PM_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(noalloc::mu);
  if (!noalloc::addr[c->device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc::scratch)) != hipSuccess || !p)
      return PM_ERR_DEVICE;
    noalloc::addr[c->device] = (unsigned char*)p;
  }
  c->na_scratch = noalloc::addr[c->device];
  return PM_OK;
}

pm_status run_reduce_noalloc(pm_context* c, const pm_species* sp, int n_sp,
                             const float* rho, const float* acc, double* out) {
  using namespace noalloc;
  if (!c->na_scratch) return PM_ERR_DEVICE;
  for (int s = 0; s < n_sp; ++s)
    if (sp[s].layout == PM_COMPRESSED && c->g.ncell3 > NC3_MAX) return PM_ERR_SHAPE;
  unsigned char* base = c->na_scratch;
  double* part = (double*)base;
  int64_t* off = (int64_t*)(base + a256(PART_BYTES));
  int64_t* bsum = (int64_t*)(base + a256(PART_BYTES) + a256(OFF_BYTES));
  return reduce_core(c, sp, n_sp, rho, acc, out, part, [&](int) { return off; }, bsum);
}
