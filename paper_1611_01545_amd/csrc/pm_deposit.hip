// Cloud-in-cell mass deposit (Sec. 2.1; CIC is named in Sec. 2.3), both species on
// one mesh (Sec. 2.1 footnote).
//
// Compressed particles are cell-sorted, so a workgroup owns a cube of R^3 mesh nodes
// (R = T r, T compression cells of r mesh cells each) and gathers exactly the
// particles that can reach those nodes: its own T^3 cells plus the one-cell shell
// on the -x/-y/-z faces, whose particles reach the tile's lowest node plane through
// their upper CIC corner. Every node has exactly one owner, so the tile is written
// with plain stores and no mesh-wide atomics or halo pass are needed. The paper's
// CPU code avoids write races with a strided loop over cells (Sec. 2.3); here the
// races inside the tile are resolved by LDS atomics.
//
// Weights are exact: a compressed position sits at the bin centre (2u+1)/(512 n_c),
// i.e. at (2u+1) r / 512 mesh cells, so each axis weight is an integer multiple of
// 1/512 and their product an integer multiple of 2^-27. Each species' weights are
// summed as 32-bit integers in LDS (exact, so independent of the order of the atomics).
// Each species' sum is scaled by its mass in FP64, rounded once to float and added in a
// fixed species order: every run, and the recomputation in the adjoint, gives
// bit-identical densities. A node that 32 particles' weight falls on wraps its sum; the
// tile's total shows it, and such a tile is summed again in 64 bits.
//
// The tile loop is bound by its instructions, about half of them per node and half per
// particle, and by the latency of two dependent loads (cell offsets, then codes). So both
// species are in flight together, with a sum each per node and one conversion pass; the
// nodes that a particle reaches outside the tile have (shared) slots of their own, which
// leaves no bounds test per corner; the atomics return nothing (a returned old value
// detected the wraps one by one before); and a wave finds its lanes' cells by a running
// maximum over marks instead of a binary search per particle. 512 threads and 47 (54) KB
// of LDS for tiles of 4^3 (8^3) cells of two species, three tiles on a CU, and 36 (45) KB of
// one, four (three); no register spilled (any scratch use doubled the time of these
// short-lived waves). A thread converts the nodes that it writes, straight from the slots.
// With the offset scans, two species of one and eight particles a cell: 39 us -> 12 on 64^3
// nodes, 281 -> 150 at 256^3, 429 -> 355 at 512^3, 3.02 -> 2.67 ms at 1024^3 (before: 32-bit
// words with a count of their wraps, and a search per particle). One species of one particle a
// cell: 36 us -> 32 on 256^3 nodes, but 211 -> 216 at 512^3 and 1.49 -> 1.63 ms at 1024^3.
#include "pm_codec.h"
#include "pm_scan.h"

namespace {

constexpr int MAX_SP = 4;

struct DepSpecies {
  int64_t n;           // particles (bounds guard against inconsistent counts)
  const void* pos;     // position codes, P bytes per axis
  const int64_t* off;  // [ncell3 + 1]
  double unit;         // density per weight unit 2^-27: m_s n_g^3 2^-27
};
struct DepArgs {
  DepSpecies sp[MAX_SP];
  int n_sp;
  int T;   // tile side in cells
  int r;   // mesh cells per compression cell
  int R;   // tile side in nodes: a power of two, 16 or (few cells) less
  int lgR;
  uint32_t rE;  // 2^16 / (T + 1), rounded up
  int lgt; // log2(tiles per box side)
};

// Node (x, y, z) of a tile of R nodes per side, -1 <= x, y, z <= R, is slot
// ((z + 1) Rp + y + 1) Rp + x + 1, Rp = R + 1: node R of a row falls on node -1 of the
// next one, and neither belongs to the tile, so a particle adds to its eight corners at
// constant slot distances without a bounds test.
__host__ __device__ constexpr int dep_slots(int R) {
  return (R + 1) * (R + 1) * (R + 1) + (R + 1) * (R + 1) + (R + 1) + 1;
}
// Particles per window, cell tables in LDS at once, type of a cell index of the tile.
// 16^3-node tiles of 4^3 cells hold few particles: both species' tables are there and their
// loads in flight together. Those of 8^3 cells take the species' tables one after the other
// (three tiles on a CU).
template <int TT> constexpr int dep_win() { return TT == 4 ? 1024 : TT == 8 ? 1536 : 2048; }
template <int TT, int SP> constexpr int dep_tabs() { return TT == 4 && SP != 1 ? 2 : 1; }
template <int TT> struct DepMark { using T = uint16_t; };
template <> struct DepMark<4> { using T = uint8_t; };  // 125 cells
constexpr int DEP_THREADS = 512;
// Node sums: 32 bits a slot and species, or one species' in 64 bits. Those of a single species
// are of the tile's own nodes alone, 32 KB, so that four tiles fit a CU: with room for a slot
// each, as two species have, three did, and 512^3 nodes with a particle per cell took 253 us
// instead of 218 (1.94 ms instead of 1.63 at 1024^3).
template <int SP>
__host__ __device__ constexpr int dep_node_bytes(int R) {
  const int narrow = (dep_slots(R) * 4 * (SP == 1 ? 1 : 2) + 15) & ~15, wide = R * R * R * 8;
  return narrow > wide ? narrow : wide;
}
template <int TT, int SP>
size_t dep_lds_bytes(int R, int NE) {
  constexpr int tabs = dep_tabs<TT, SP>();
  return (size_t)dep_node_bytes<SP>(R) + (size_t)tabs * (NE * 8 + (NE + 1) * 4) +
         (size_t)tabs * dep_win<TT>() * sizeof(typename DepMark<TT>::T);
}

// Sum over the 64 lanes of a wave by DPP (mod 2^64), in lane 63
__device__ inline uint64_t wave_sum_dpp(uint64_t v) {
  auto step = [&](auto ctrl, auto rows) {
    constexpr int C = decltype(ctrl)::value, M = decltype(rows)::value;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, C, M, 0xf, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), C, M, 0xf, false);
    v += ((uint64_t)hi << 32) | lo;
  };
  step(IC<0x111>{}, IC<0xf>{});
  step(IC<0x112>{}, IC<0xf>{});
  step(IC<0x114>{}, IC<0xf>{});
  step(IC<0x118>{}, IC<0xf>{});
  step(IC<0x142>{}, IC<0xa>{});
  step(IC<0x143>{}, IC<0xc>{});
  return v;
}

__device__ inline int wrapc(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

// Inclusive running maximum over the 64 lanes of a wave by DPP (values >= 0)
__device__ inline int wave_incl_max_dpp(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
  return v;
}

// The three codes of particle j of n: one unaligned load of 4 (8) bytes, moved back by
// `back` bytes from the array's end where it would pass it (shift the result down by as
// many); byte loads for a single particle.
template <int PB, typename CT>
__device__ __forceinline__ CT dep_codes(const void* pos, int64_t n, uint32_t j, int& back) {
  const uint8_t* p = (const uint8_t*)pos;
  const int64_t at = (int64_t)(3 * PB) * j, last = (int64_t)(3 * PB) * n - (int64_t)sizeof(CT);
  CT c = 0;
  back = 0;
  if (last >= 0) {  // two particles and more (uniform)
    const int64_t from = at < last ? at : last;
    back = (int)(at - from);
    __builtin_memcpy(&c, p + from, sizeof(CT));
  } else {
    for (int q = 0; q < 3 * PB; ++q) c |= (CT)p[at + q] << (8 * q);
  }
  return c;
}

// One particle's eight weights. put(dx, dy, dz, slots of the lower corner, weight); the weight
// units added, 0 for nothing to add or a particle of the shell that reaches no node of the tile.
template <int PB, typename CT, typename Put>
__device__ __forceinline__ uint32_t dep_weights(CT code, uint32_t org, int r, Put put) {
  constexpr int FB = 8 * PB + 1;  // fractional bits of a mesh coordinate
  constexpr int ONE = 1 << FB;    // one mesh cell
  int sl[3], f[3];
  code >>= 8 * (org >> 24);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    // position inside the cell in units of 2^-FB mesh cells (1/512 for PB = 1)
    const int c = (int)((uint32_t)(code >> (8 * PB * a)) & ((1u << (8 * PB)) - 1u));
    const int gl = (2 * c + 1) * r;
    sl[a] = (int)(int8_t)(org >> (8 * a)) + (gl >> FB);
    f[a] = gl & (ONE - 1);
  }
  if ((sl[0] | sl[1] | sl[2]) < 0) return 0;
  const uint32_t wx[2] = {(uint32_t)(ONE - f[0]), (uint32_t)f[0]},
                 wy[2] = {(uint32_t)(ONE - f[1]), (uint32_t)f[1]},
                 wz[2] = {(uint32_t)(ONE - f[2]), (uint32_t)f[2]};
  uint32_t sum = 0;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        uint32_t W;  // units of 2^-27
        if constexpr (PB == 1) {
          W = __umul24(__umul24(wx[dx], wy[dy]), wz[dz]);  // exact
        } else {
          const uint64_t w3 = (uint64_t)wx[dx] * (uint64_t)wy[dy] * (uint64_t)wz[dz];
          W = (uint32_t)((w3 + (1ull << 23)) >> 24);  // 2^-51 -> 2^-27, rounded
          sum += W;
        }
        put(dx, dy, dz, sl, W);
      }
  return PB == 1 ? 1u << 27 : sum;
}
// into slots of type NT
template <int PB, typename NT, typename CT>
__device__ __forceinline__ uint32_t dep_add(NT* node, CT code, uint32_t org, int r, int Rp) {
  return dep_weights<PB>(code, org, r, [&](int dx, int dy, int dz, const int (&sl)[3], uint32_t W) {
    atomicAdd(&node[(sl[2] * Rp + sl[1]) * Rp + sl[0] + (dz * Rp + dy) * Rp + dx], (NT)W);
  });
}
// into the tile's own nodes
template <int PB, typename NT, typename CT>
__device__ __forceinline__ void dep_add_own(NT* node, CT code, uint32_t org, int r, int lgR) {
  const uint32_t R = 1u << lgR;
  dep_weights<PB>(code, org, r, [&](int dx, int dy, int dz, const int (&sl)[3], uint32_t W) {
    const uint32_t x = (uint32_t)(sl[0] + dx - 1), y = (uint32_t)(sl[1] + dy - 1),
                   z = (uint32_t)(sl[2] + dz - 1);
    if (x < R && y < R && z < R) atomicAdd(&node[(((z << lgR) + y) << lgR) + x], (NT)W);
  });
}

// TT: tile side in cells (compile time, 0: runtime A.T); PB: position bytes per axis. With
// PB = 2 the offset inside a cell has 17 fractional bits of a mesh cell per axis, and each
// node's weight (the exact product, a multiple of 2^-51) is rounded to a multiple of
// 2^-27, the unit of the 1-byte form, so that the same integer sums apply.
// SP: one species, two, or (3) any larger number, in pairs.
template <int TT, int PB, int SP>
__global__ __launch_bounds__(DEP_THREADS, SP == 3 || (TT == 0 && PB == 2) ? 4 : 6) void k_deposit_tile(
    DepArgs A, Geom g, float* rho) {
  constexpr bool MORE = SP == 3;
  constexpr int SB = SP == 1 ? 1 : 2;  // species of a batch
  using CT = typename std::conditional<PB == 1, uint32_t, uint64_t>::type;
  constexpr int NT = DEP_THREADS, NW = NT / 64;
  constexpr int WIN = dep_win<TT>(), TABS = dep_tabs<TT, SP>();
  constexpr int U = WIN / NT;                 // chunks of 64 particles per wave and window
  using MT = typename DepMark<TT>::T;
  extern __shared__ __align__(16) unsigned char smem[];
  // compile-time tiles have T r = 16 nodes per side (T = 16 / r)
  const int T = TT ? TT : A.T, R = TT ? 16 : A.R, r = TT ? 16 / TT : A.r;
  const bool spread = !TT && r == 1;  // the coarse mesh of the two-level force
  const int lgR = TT ? 4 : A.lgR;
  const int E = T + 1;              // extended cells per side
  const int NE = E * E * E;
  const int Rp = R + 1, NS = TT ? dep_slots(16) : dep_slots(R);
  __shared__ int wsum[2][NW];
  __shared__ uint64_t lost[NW];  // weight units missing from the sums, per wave
  __shared__ int over[NW];       // the wave's cells: 1 beyond 32-bit sums, 2 perhaps so
  uint32_t* node = (uint32_t*)smem;                      // [SB][NS] weight sums per species
  unsigned long long* wide = (unsigned long long*)smem;  // one species' in 64 bits
  uint2* tab = (uint2*)(smem + dep_node_bytes<SP>(R));   // [TABS][NE] stream start, origin
  int* pre = (int*)(tab + TABS * NE);                    // [TABS][NE + 1] particles before
  MT* mark = (MT*)(pre + TABS * (NE + 1));               // [TABS][WIN] extended cells
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t ntm = (uint32_t)(1 << A.lgt) - 1u;  // tiles per side: a power of two
  const int tx = (int)((uint32_t)tile & ntm), ty = (int)((uint32_t)(tile >> A.lgt) & ntm),
            tz = (int)(tile >> (2 * A.lgt));
  const int ncs = (int)g.nc;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  constexpr int ZB = 4 / SB;  // slots of a 16-byte store
  for (int i = threadIdx.x; i < NS / ZB; i += NT) ((uint4*)node)[i] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < NS % ZB * SB) node[NS / ZB * 4 + threadIdx.x] = 0;
  for (int i = threadIdx.x; i < TABS * WIN * (int)sizeof(MT) / 4; i += NT)
    ((uint32_t*)mark)[i] = 0u;
  // Each thread's nodes of the tile: 16 nodes per side, four consecutive ones along x in planes
  // tid / 64 + NW k of row tid / 4 % 16; fewer nodes, one per thread. Their densities are summed
  // over the species in order.
  const bool full = TT || R == 16;
  const bool own = full || (int)threadIdx.x < R * R * R;
  const int lx = full ? 4 * (threadIdx.x & 3) : threadIdx.x & (R - 1),
            ly = full ? (threadIdx.x >> 2) & 15 : (threadIdx.x >> lgR) & (R - 1),
            lz = full ? threadIdx.x >> 6 : threadIdx.x >> (2 * lgR);
  constexpr int NPT = 4096 / NT;
  float racc[NPT];
  auto each = [&](auto f) {  // f(k, slot, node)
    if (!own) return;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      if (!full && k > 0) break;
      const int x = lx + (k & 3), z = lz + NW * (k >> 2);
      f(k, ((z + 1) * Rp + ly + 1) * Rp + x + 1, (((z << lgR) + ly) << lgR) + x);
    }
  };
#pragma unroll
  for (int k = 0; k < NPT; ++k) racc[k] = 0.0f;
  auto split = [&](int e, int& ex, int& ey, int& ez) {  // extended cell e < 2^10 (T <= 8)
    int q = e / E;
    if constexpr (!TT) q = (int)((uint32_t)e * A.rE >> 16);
    ex = e - q * E;
    ez = q / E;
    if constexpr (!TT) ez = (int)((uint32_t)q * A.rE >> 16);
    ey = q - ez * E;
  };

  const int n_sp = MORE ? A.n_sp : min(A.n_sp, 2);
  for (int s0 = 0; s0 < (MORE ? n_sp : min(n_sp, 1)); s0 += 2) {
    const int ns = SP == 1 ? 1 : min(2, n_sp - s0);
    // cells of both species: a thread takes K consecutive extended cells
    constexpr int KMAX = TT ? ((TT + 1) * (TT + 1) * (TT + 1) + NT - 1) / NT : 2;
    const int K = TT ? KMAX : (NE + NT - 1) / NT;
    const int e0 = threadIdx.x * K;
    const bool cells = wv * 64 * K < NE;  // this wave has any
    uint32_t start[2][KMAX];  // first particle and particle count of the thread's cells
    int cnt[2][KMAX];
    auto fetch = [&]() {
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        const int e = e0 + k;
        const bool in = k < K && e < NE;
        int ex, ey, ez;
        split(e, ex, ey, ez);
        const uint32_t key =
            in ? cell_key(g, wrapc(tx * T + ex - 1, ncs), wrapc(ty * T + ey - 1, ncs),
                          wrapc(tz * T + ez - 1, ncs))
               : 0u;
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          const int64_t* off = A.sp[s0 + (s < ns ? s : 0)].off;
          const int64_t o0 = off[key], o1 = off[key + 1];
          start[s][k] = (uint32_t)o0;
          cnt[s][k] = in && s < ns ? (int)(o1 - o0) : 0;
        }
      }
    };
    // A node of 32 particles' weight (2^32) passes a 32-bit slot, and such a tile is summed
    // again in 64 bits. These sums alone take 1.13 times as long as those in 32 bits with 4
    // mesh cells per compression cell and axis, 1.3 times with 2, so a tile starts with them
    // where a cell has 16 particles per node and some more: evenly spread, their nodes pass 32
    // about there. 8^3 cells of 2000 on 64^3 nodes 921 -> 529 us, 16^3 cells of 256 on as many
    // 968 -> 538, with the particles together in each cell 1980 -> 1016; 1024 particles a cell
    // in the former, which 32 bits just hold, 238 -> 281.
    const int most = 16 * r * r * r + 48;
    bool crowd = false, maybe = false;
    int before[2] = {0, 0}, loc[2] = {0, 0};
    if (cells) {
      fetch();
#pragma unroll
      for (int s = 0; s < SB; ++s) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          const int e = e0 + k;
          loc[s] += cnt[s][k];
          int ex, ey, ez;
          split(e, ex, ey, ez);
          if (cnt[s][k] > most) crowd |= ex && ey && ez;  // no shell cell
        }
        before[s] = pmscan::wave_incl_scan_dpp(loc[s]);
        // A node takes weight from 2^3 cells, four pairs of neighbours along x: with no pair of
        // more than 7 it cannot pass 28 particles, and the sums need no check. (Pairs across
        // waves by twice either count; those across rows do no harm.)
        const int last = K == KMAX ? cnt[s][KMAX - 1] : cnt[s][0];
        const int next = __shfl_down(cnt[s][0], 1, 64);
        maybe |= last + (lane == 63 ? last : next) > 7 || 2 * cnt[s][0] > 7 * (lane == 0 ? 1 : 2);
        for (int k = 0; k + 1 < KMAX; ++k) maybe |= k + 1 < K && cnt[s][k] + cnt[s][k + 1] > 7;
      }
    }
    const int wave_over = (__any(crowd) ? 1 : 0) | (__any(maybe) ? 2 : 0);
    if (lane == 63) {
      wsum[0][wv] = before[0];
      if (SP != 1) wsum[1][wv] = before[1];
      over[wv] = wave_over;
    }
    __syncthreads();  // also: the last pair is done with the tables
    int np[2] = {0, 0};  // particles of the tile and its shell
#pragma unroll
    for (int s = 0; s < SB; ++s) {
      before[s] -= loc[s];
      for (int w = 0; w * 64 * K < NE; ++w) {  // the waves with cells
        const int v = wsum[s][w];
        before[s] += w < wv ? v : 0;
        np[s] += v;
      }
      np[s] = __builtin_amdgcn_readfirstlane(np[s]);
    }
    int any_full = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any_full |= over[w];
    any_full = __builtin_amdgcn_readfirstlane(any_full);
    const bool dense = any_full & 1;
    // species s's table into slot t of the tables
    auto build = [&](int s, int t) {
      if (!cells) return;
      int at = s ? before[1] : before[0];
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        const int e = e0 + k;
        if (k < K && e < NE) {
          int ex, ey, ez;
          split(e, ex, ey, ez);
          // slot of the cell's first node per axis, a signed byte each: -r + 1 .. R
          const uint32_t ox = (uint32_t)((ex - 1) * r + 1) & 255u,
                         oy = (uint32_t)((ey - 1) * r + 1) & 255u,
                         oz = (uint32_t)((ez - 1) * r + 1) & 255u;
          tab[t * NE + e] =
              make_uint2((s ? start[1][k] : start[0][k]) - (uint32_t)at, ox | oy << 8 | oz << 16);
          pre[t * (NE + 1) + e] = at;
          at += s ? cnt[1][k] : cnt[0][k];
          if (e == NE - 1) pre[t * (NE + 1) + NE] = at;
        }
      }
    };
    // A window of WIN particles from particle rb of the tile (nw of them). Each cell marks its
    // first particle of the window and every 64th slot that it reaches, so that a wave finds
    // its lanes' cells by a running maximum.
    auto set_marks = [&](int t, int rb, int nw) {
      const int* pr = pre + t * (NE + 1);
      MT* mk = mark + t * WIN;
      for (int e = threadIdx.x; e < NE; e += NT) {
        const int lo = max(pr[e], rb) - rb, hi = min(pr[e + 1] - rb, nw);
        if (lo < hi) {
          mk[lo] = (MT)e;
          for (int m = (lo | 63) + 1; m < hi; m += 64) mk[m] = (MT)e;
        }
      }
    };
    struct Batch {
      CT code[U];
      uint32_t org[U];  // first slot per axis (bit 7 set: nothing to add), shift of the code
    };
    auto load = [&](int s, int t, int rb, int nw, Batch& B) {
      const DepSpecies& sp = A.sp[s0 + s];
      const uint2* tb = tab + t * NE;
      MT* mk = mark + t * WIN;
      const int lim = spread ? (nw + 511) & ~511 : nw;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        B.org[u] = 0x80u;
        B.code[u] = 0;
        const int b = wv * 64 + u * NT;
        if (b >= lim) continue;  // uniform across the wave
        const int l = b + lane;
        int e, q = l;
        if (spread) {
          // slot l of 512 takes particle (l % 8) 64 + l / 8: the lanes of one atomic then
          // hit the nodes of eight different cells (8 neutrinos per cell on one node each)
          // instead of the same eight nodes
          q = (l & ~511) + ((l & 7) << 6) + ((l & 511) >> 3);
          e = mk[q];
        } else {
          e = wave_incl_max_dpp((int)mk[l]);
          mk[l] = 0;  // read once: clear for the next window
        }
        const uint2 c = tb[e];
        const uint32_t j = c.x + (uint32_t)(rb + q);
        // counts inconsistent with n are latched by the offset check
        const bool ok = q < nw && (int64_t)j < sp.n;
        int back;
        B.code[u] = dep_codes<PB, CT>(sp.pos, sp.n, ok ? j : 0u, back);
        B.org[u] = ok ? c.y | (uint32_t)back << 24 : 0x80u;
      }
    };
    // the marks of a window, filled in for the spread order (all threads)
    auto marks_done = [&](int t, int nw) {
      __syncthreads();
      if (!spread) return;
      MT* mk = mark + t * WIN;
      for (int b = wv * 64; b < nw; b += NT)
        mk[b + lane] = (MT)wave_incl_max_dpp((int)mk[b + lane]);
      __syncthreads();
    };
    // species s's window at rb into B (all threads)
    auto window = [&](int s, int t, int rb, Batch& B) {
      const int nw = min(WIN, (s ? np[1] : np[0]) - rb);
      if (spread) {  // (the other order clears the marks as it reads them)
        __syncthreads();
        for (int l = threadIdx.x; l < WIN; l += NT) mark[t * WIN + l] = 0;
      }
      __syncthreads();
      set_marks(t, rb, nw);
      marks_done(t, nw);
      load(s, t, rb, nw, B);
    };
    uint64_t units = 0;  // weight units that this thread added
    auto narrow = [&](uint32_t* to) {
      return [&units, to, r, Rp](CT code, uint32_t org) {
        units += dep_add<PB>(to, code, org, r, Rp);
      };
    };
    auto add = [&](const Batch& B, auto put) {
#pragma unroll
      for (int u = 0; u < U; ++u) put(B.code[u], B.org[u]);
    };
    // the windows of species s from rb on
    auto rest = [&](int s, int t, int rb, auto put) {
      for (; rb < (s ? np[1] : np[0]) && rb >= 0; rb += WIN) {
        Batch B;
        window(s, t, rb, B);
        add(B, put);
      }
    };

    if constexpr (TABS == 2) {
      // the first windows of both species, their loads in flight together
      build(0, 0);
      if (SP != 1) build(1, 1);
      __syncthreads();
      if (!dense) {
        const int n0 = min(WIN, np[0]), n1 = min(WIN, np[1]);
        set_marks(0, 0, n0);
        if (SP != 1) set_marks(1, 0, n1);
        __syncthreads();
        Batch B0, B1;
        load(0, 0, 0, n0, B0);
        if (SP != 1) load(ns - 1, 1, 0, n1, B1);
        add(B0, narrow(node));
        if (SP != 1) add(B1, narrow(node + NS));
        rest(0, 0, WIN, narrow(node));
        if (SP != 1) rest(1, 1, WIN, narrow(node + NS));
      }
    } else if (!dense) {
      build(0, 0);
      rest(0, 0, 0, narrow(node));
      if (SP != 1 && ns > 1) {
        __syncthreads();
        build(1, 0);
        rest(1, 0, 0, narrow(node + NS));
      }
    }
    __syncthreads();
    // Where a sum passes 2^32 (a node of 32 particles' weight), the total falls short of the
    // weights added.
    const double unit0 = A.sp[s0].unit, unit1 = ns > 1 ? A.sp[s0 + 1].unit : 0.0;
    uint64_t all = 0;
    if (any_full) {
      uint64_t sum = 0;
#pragma unroll
      for (int k = 0; k < (dep_slots(16) + NT - 1) / NT; ++k) {
        const int i = threadIdx.x + k * NT;
        if (i < NS) {
          sum += node[i];
          if (SP != 1) sum += node[NS + i];  // 0 without a second species
        }
      }
      sum = wave_sum_dpp(units - sum);
      if (lane == 63) lost[wv] = sum;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) all += lost[w];
    }
    if (all == 0 && !dense) {
      each([&](int k, int slot, int) {
        racc[k] += (float)((double)node[slot] * unit0);
        if (SP != 1) racc[k] += (float)((double)node[NS + slot] * unit1);
      });
    } else {
      // again, one species at a time in 64-bit sums
#pragma unroll
      for (int s = 0; s < SB; ++s) {
        if (s >= ns) break;
        __syncthreads();
        for (int i = threadIdx.x; i < (SP == 1 ? 2 * R * R * R : 2 * NS); i += NT) node[i] = 0;
        if (TABS == 1) {
          if (cells) fetch();
          build(s, 0);
        }
        rest(s, TABS == 2 ? s : 0, 0, [&](CT code, uint32_t org) {
          if constexpr (SP == 1) dep_add_own<PB>(wide, code, org, r, lgR);
          else dep_add<PB>(wide, code, org, r, Rp);
        });
        __syncthreads();
        const double unit = s ? unit1 : unit0;
        each([&](int k, int slot, int own) {
          racc[k] += (float)((double)wide[SP == 1 ? own : slot] * unit);
        });
      }
    }
    if (MORE && s0 + 2 < n_sp) {  // the next pair's sums start at 0
      __syncthreads();
      for (int i = threadIdx.x; i < 2 * NS; i += NT) node[i] = 0;
    }
  }
  if (!own) return;
  const int64_t ng = g.ng;
  float* d = rho + (((int64_t)tz * R + lz) * ng + (int64_t)ty * R + ly) * ng + (int64_t)tx * R + lx;
  if (!full) {
    *d = racc[0];
    return;
  }
  const bool aligned = ((uintptr_t)rho & 15) == 0;  // the caller's pointer: any float
#pragma unroll
  for (int k = 0; k < NPT / 4; ++k, d += (int64_t)NW * ng * ng) {
    if (aligned) {
      *(float4*)d = make_float4(racc[4 * k], racc[4 * k + 1], racc[4 * k + 2], racc[4 * k + 3]);
    } else {
      for (int a = 0; a < 4; ++a) d[a] = racc[4 * k + a];
    }
  }
}

// ---------------------------------------------------------- float-layout path --
// Unsorted float particles: fixed-point weights accumulated with 64-bit global atomics
// (still order independent), then converted.
__global__ __launch_bounds__(256) void k_deposit_float(const float* x, int64_t n, int64_t ng,
                                                      float ngL, double scale,
                                                      unsigned long long* acc) {
  int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= n) return;
  int64_t i[3];
  double f[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double u = (double)(x[3 * p + a] * ngL);  // mesh units (exact for a power-of-two box)
    double fl = floor(u);
    f[a] = u - fl;
    int64_t k = (int64_t)fl % ng;
    i[a] = k < 0 ? k + ng : k;
  }
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        double w = (dx ? f[0] : 1.0 - f[0]) * (dy ? f[1] : 1.0 - f[1]) * (dz ? f[2] : 1.0 - f[2]);
        unsigned long long q = (unsigned long long)__double2ll_rn(w * scale);
        if (!q) continue;
        int64_t nz = (i[2] + dz) % ng, ny = (i[1] + dy) % ng, nx = (i[0] + dx) % ng;
        atomicAdd(&acc[(nz * ng + ny) * ng + nx], q);
      }
}

__global__ __launch_bounds__(256) void k_fixed_to_float(const unsigned long long* acc, int64_t n,
                                                       double unit, float* rho) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) rho[i] = (float)((double)acc[i] * unit);
}

}  // namespace

int deposit_tile_cells(const Geom& g) {
  // 16 nodes per tile side (T r = 16), except with one mesh cell per compression cell
  // (the coarse mesh of the two-level force): 8^3-cell tiles, since 16^3 cells would
  // hold 83 KB of LDS and run one workgroup per CU
  int T = g.r == 1 ? 8 : 16 / g.r;
  if (T < 1) T = 1;
  if (T > g.nc) T = (int)g.nc;
  return T;
}

pm_status run_deposit_tile(pm_context* c, const pm_species* sp, int n_sp,
                           int64_t* const* offs, float* rho) {
  const Geom& g = c->g;
  if (n_sp > MAX_SP) return PM_ERR_ARG;
  const double ng3 = (double)g.ng * g.ng * g.ng / (g.box * g.box * g.box);  // 1 / Delta^3
  DepArgs A{};
  A.n_sp = 0;
  for (int s = 0; s < n_sp; ++s) {
    if (sp[s].n == 0 || sp[s].mass == 0.0) continue;
    A.sp[A.n_sp].n = sp[s].n;
    A.sp[A.n_sp].pos = sp[s].pos;
    A.sp[A.n_sp].off = offs[s];
    A.sp[A.n_sp].unit = sp[s].mass * ng3 * 0x1p-27;
    A.n_sp++;
  }
  A.r = g.r;
  A.T = deposit_tile_cells(g);
  A.R = A.T * g.r;
  if (A.R > 16) return PM_ERR_SHAPE;  // at most 16 nodes per thread
  const int nt = (int)(g.nc / A.T);  // a power of two, as nc and T are
  while ((1 << A.lgt) < nt) ++A.lgt;
  while ((1 << A.lgR) < A.R) ++A.lgR;
  A.rE = (65536u + (uint32_t)A.T) / (uint32_t)(A.T + 1);
  const int ne = (A.T + 1) * (A.T + 1) * (A.T + 1);
  ProfScope ps(c, ST_DEPOSIT);
  const unsigned grid = (unsigned)((int64_t)nt * nt * nt);
  // the compile-time variants assume T r = 16; one position width for every species
  const int kind = common_width_kind(sp, n_sp);
  if (kind < 0) return PM_ERR_ARG;
  auto launch = [&](auto tt, auto pb) {
    constexpr int TT = decltype(tt)::value, PB = decltype(pb)::value;
    auto go = [&](auto kernel, size_t lds) {
      hipLaunchKernelGGL(kernel, dim3(grid), dim3(DEP_THREADS), lds, c->stream, A, g, rho);
    };
    if (A.n_sp > 2) go(k_deposit_tile<TT, PB, 3>, dep_lds_bytes<TT, 3>(A.R, ne));
    else if (A.n_sp == 2) go(k_deposit_tile<TT, PB, 2>, dep_lds_bytes<TT, 2>(A.R, ne));
    else go(k_deposit_tile<TT, PB, 1>, dep_lds_bytes<TT, 1>(A.R, ne));
  };
  if (width_pos(sp[0]) == 1) {
    if (A.T == 4 && A.r == 4) launch(IC<4>{}, IC<1>{});
    else if (A.T == 8 && A.r == 2) launch(IC<8>{}, IC<1>{});
    else launch(IC<0>{}, IC<1>{});
  } else {
    if (A.T == 4 && A.r == 4) launch(IC<4>{}, IC<2>{});
    else launch(IC<0>{}, IC<2>{});
  }
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_deposit(pm_context* c, const pm_species* sp, int n_sp, float* rho) {
  const Geom& g = c->g;
  if (n_sp <= 0 || n_sp > MAX_SP) return PM_ERR_ARG;
  int layout = sp[0].layout;
  for (int s = 1; s < n_sp; ++s)
    if (sp[s].layout != layout) return PM_ERR_ARG;
  if (layout == PM_COMPRESSED) {
    int64_t* offs[MAX_SP];
    const pm_status st = run_species_offsets(c, sp, n_sp, offs);
    if (st != PM_OK) return st;
    return run_deposit_tile(c, sp, n_sp, offs, rho);
  }
  ProfScope ps(c, ST_DEPOSIT);
  const unsigned long long* acc = nullptr;
  double unit = 0.0;
  const pm_status st = run_deposit_fixed(c, sp, n_sp, &acc, &unit);
  if (st != PM_OK) return st;
  const int64_t n3 = g.ng * g.ng * g.ng;
  hipLaunchKernelGGL(k_fixed_to_float, dim3((unsigned)cdiv(n3, 256)), dim3(256), 0, c->stream,
                     acc, n3, unit, rho);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_deposit_fixed(pm_context* c, const pm_species* sp, int n_sp,
                            const unsigned long long** fixed, double* unit) {
  const Geom& g = c->g;
  if (n_sp <= 0 || n_sp > MAX_SP) return PM_ERR_ARG;
  for (int s = 0; s < n_sp; ++s)
    if (sp[s].layout != PM_FLOAT) return PM_ERR_ARG;
  const int64_t n3 = g.ng * g.ng * g.ng;
  unsigned long long* acc = (unsigned long long*)scratch(c, SC_ACC64, (size_t)n3 * 8);
  if (!acc) return PM_ERR_NOMEM;
  const pm_status st = launch_fill_u64(c, (uint64_t*)acc, n3, 0ull);
  if (st != PM_OK) return st;
  double mmax = 0.0;
  for (int s = 0; s < n_sp; ++s) mmax = fmax(mmax, sp[s].mass);
  for (int s = 0; s < n_sp; ++s) {
    if (sp[s].n == 0 || sp[s].mass == 0.0) continue;
    double scale = 0x1p32 * (sp[s].mass / mmax);
    hipLaunchKernelGGL(k_deposit_float, dim3((unsigned)cdiv(sp[s].n, 256)), dim3(256), 0,
                       c->stream, sp[s].x, sp[s].n, g.ng, g.ngL, scale, acc);
  }
  PM_LAUNCH_CHECK();
  *fixed = acc;
  *unit = mmax > 0 ? mmax * 0x1p-32 * (double)n3 / (g.box * g.box * g.box) : 0.0;
  return PM_OK;
}
