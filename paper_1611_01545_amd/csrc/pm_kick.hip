// CIC force interpolation (Fig. 2 "inverse_force_interpolation"), kick and drift, fused
// with the re-encode of compressed particles and the stable re-sort of the stream into
// cell order (Sec. 2.4: particles are written cell by cell).
//
// Compressed path, per species:
//   k_kick_prep     v_max' = smallest power of two >= V + |c_k| A_max (V: largest
//                   decoded |v| of the input, from its extreme velocity codes; A_max:
//                   largest |a| on the mesh). Interpolation is a convex combination of
//                   mesh values, so no kicked component exceeds the bound. Clears the
//                   re-sort's counters.
//   k_kick_pair     two bricks adjacent along x per workgroup (R = 16 nodes per brick
//   k_kick_brick    side), or one brick of any shape: the force (or potential) nodes in LDS,
//                   then waves take 64-particle chunks independently (no barrier):
//                   decode, gather a from the 8 CIC nodes, v' = v + c_k a, fixed-point
//                   drift u' = u + floor(v' c_d S + 1/2), new codes, and the digit: the
//                   new cell inside the brick, or B^3 for a particle that leaves it (a
//                   "mover", whose new cell key is kept). Stayers are counted per new
//                   cell and movers per brick with LDS atomics, arrivals per brick with
//                   global ones.
//   k_brick_scan    first new stream position and first arrival of each brick.
//   k_list_arrivals the movers into their new bricks' lists, unordered.
//   k_place         per brick: its arrivals sorted by old index, then arrivals from
//                   earlier bricks, stayers and arrivals from later bricks written at
//                   their final stream positions, and the new count bytes.
//   k_place_rest    the cells of 255 particles and more; bricks that k_place leaves.
// Seven launches for all species on most meshes. The movers are few (1% of the
// neutrinos at the large workload), so grouping them by brick with one atomic each and
// sorting each brick's handful in LDS replaces a device-wide radix sort by cell: at
// 64^3 its 60 small launches took 170 of the step's 275 us.
#include <type_traits>

#include "pm_codec.h"
#include "pm_scan.h"

namespace {

constexpr int KT = 256;  // threads per workgroup

// ------------------------------------------------------------ float layout --
__global__ __launch_bounds__(KT) void k_kick_float(const float* x, const float* v, float* xo,
                                                  float* vo, int64_t n, const float* acc,
                                                  int64_t ng, float ngL, float box, float ck,
                                                  float cd) {
  int64_t p = (int64_t)blockIdx.x * KT + threadIdx.x;
  if (p >= n) return;
  const int64_t n3 = ng * ng * ng;
  int64_t i[3];
  float f[3], xv[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    xv[a] = x[3 * p + a];
    float u = xv[a] * ngL;  // mesh units (exact for a power-of-two box)
    float fl = floorf(u);
    f[a] = u - fl;
    int64_t k = (int64_t)fl % ng;
    i[a] = k < 0 ? k + ng : k;
  }
  float ax = 0.f, ay = 0.f, az = 0.f;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        float w = (dx ? f[0] : 1.f - f[0]) * (dy ? f[1] : 1.f - f[1]) * (dz ? f[2] : 1.f - f[2]);
        int64_t node = (((i[2] + dz) % ng) * ng + (i[1] + dy) % ng) * ng + (i[0] + dx) % ng;
        ax += w * acc[node];
        ay += w * acc[n3 + node];
        az += w * acc[2 * n3 + node];
      }
  const float a3[3] = {ax, ay, az};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float v1 = v[3 * p + a] + ck * a3[a];
    float x1 = xv[a] + cd * v1;
    x1 -= box * floorf(x1 / box);  // periodic wrap into [0, L)
    if (x1 >= box || x1 < 0.f) x1 = 0.f;
    vo[3 * p + a] = v1;
    xo[3 * p + a] = x1;
  }
}

// ------------------------------------------------------- compressed layout --
constexpr int MAXSP = 4;

struct PrepArgs {
  const pm_shdr* hin[MAXSP];
  pm_shdr* hout[MAXSP];
  int64_t n[MAXSP];
  int n_sp;
};
template <int VB = 2>  // velocity bytes per axis
__global__ __launch_bounds__(KT) void k_kick_prep(PrepArgs A, const float* amax, double ck,
                                                 uint32_t* clear, int64_t nclear) {
  for (int64_t i = (int64_t)blockIdx.x * KT + threadIdx.x; i < nclear; i += (int64_t)gridDim.x * KT)
    clear[i] = 0u;
  if (blockIdx.x || (int)threadIdx.x >= A.n_sp) return;
  const pm_shdr* hin = A.hin[threadIdx.x];
  pm_shdr* hout = A.hout[threadIdx.x];
  double V = 0.0;
  if (A.n[threadIdx.x] > 0 && hin->j_max >= 0) {
    double a = fabs((double)vel_decode_v<VB>((uint32_t)hin->j_min, hin->v_max));
    double b = fabs((double)vel_decode_v<VB>((uint32_t)hin->j_max, hin->v_max));
    V = a > b ? a : b;
  }
  double bound = V + fabs(ck) * (double)(*amax);
  float vm = 0.f;
  if (bound > 0.0) {
    int e;
    double m = frexp(bound, &e);
    vm = (float)(m == 0.5 ? bound : ldexp(1.0, e));
  }
  hout->v_max = vm;
  hout->j_min = 65536;
  hout->j_max = -1;
  hout->flags = 0;
  hout->n_esc = 0;
  hout->reserved = 0;
}

constexpr int KB = 512;  // threads per workgroup of the brick kicks
constexpr int NWK = KB / 64;

struct KickSpecies {
  int64_t n;
  const void* pos;     // position codes, P bytes per axis
  const void* vel;     // velocity codes, V bytes per axis
  const pm_shdr* hin;
  pm_shdr* hout;
  const int64_t* off;  // input cell offsets [ncell3 + 1]
  void* tpos;          // new codes, old stream order
  void* tvel;
  uint16_t* tdig;      // new local cell in the brick, or B^3 for movers
  uint32_t* mkey;      // movers: new cell key, at the old stream index
  uint32_t* cnt;       // stayers per cell
  uint32_t* mcnt;      // movers per brick
  uint32_t* acnt;      // arrivals per brick (2^apad words apart)
  int32_t* pmn;        // per-brick extreme new velocity codes, folded into hout
  int32_t* pmx;
  const float* app;    // nullable: per-particle acceleration added to the mesh force
};
struct KickArgs {
  KickSpecies sp[MAXSP];
  int n_sp;
  const float* acc;  // [3][ng^3], or the potential [ng^3] (k_kick_pair with PHI)
  float scale;       // of its difference: ng / 12
  int apad;
  float ck;
  double cdS;        // c_d S / L (position codes per unit velocity)
};

// Codec constants of one species (uniform), V velocity bytes per axis (half range
// H = 2^(8V - 1)): wd = v_max / H, ce = H / v_max' (v_max' a power of two: exponent
// field of 2^(8V - 1 - e) is 253 + 8V minus that of v_max').
struct Codec {
  float vmi, vmo, wd, ce;
};
template <int V>
__device__ inline Codec codec_of(const KickSpecies& S) {
  Codec k;
  k.vmi = S.hin->v_max;
  k.vmo = S.hout->v_max;
  k.wd = k.vmi * (V == 2 ? 0x1p-15f : 0x1p-7f);
  k.ce = __uint_as_float(((253u + 8u * V) - (__float_as_uint(k.vmo) >> 23)) << 23);
  return k;
}
// float32 codec forms valid for every species (see vel_code_p2, vel_decode_w)
__device__ inline bool codec_fast(const KickArgs& A) {
  bool fast = true;
  for (int s = 0; s < A.n_sp; ++s) {
    const float vi = A.sp[s].hin->v_max, vo = A.sp[s].hout->v_max;
    fast = fast && vi >= 0x1p-90f && vi <= 0x1p90f && vo >= 0x1p-90f && vo <= 0x1p90f &&
           (__float_as_uint(vo) & 0x7fffffu) == 0;
  }
  return fast;
}

// One lane kicks particle j of one species in one brick (jr: its index from the
// brick's first particle of that species): decode, gather a through `gather(li, f)`
// (node index inside the brick, CIC fractions), kick, fixed-point drift, new codes.
// Writes the new codes and the particle's digit (new local cell, or B^3 when it leaves
// the brick; movers also get their new cell key), counts stayers per new cell and movers
// in LDS, and folds the new velocity codes into the lane's running extremes jmn, jmx
// (reduced over the wave once per kernel, by VelExt). No barrier: waves are
// independent, and the lanes of a wave may take particles of different bricks. The cell
// search range [lo0, hi0) spans a power-of-two number of cells.
// P position bytes and V velocity bytes per axis (P = 1, V = 2: the paper's format).
template <bool FAST, int P, int V, typename Gather>
__device__ inline void kick_lane(const KickSpecies& S, const KickArgs& A, const Geom& g,
                                 const Codec& cd, int64_t j, uint32_t jr, const uint32_t* rel,
                                 int lo0, int hi0, const uint32_t bc[3], uint32_t* run,
                                 uint32_t* mvc, int& jmn, int& jmx, bool& bad, Gather gather) {
  using PC = typename PosCode<P>::T;
  using VC = typename VelCode<V>::T;
  constexpr int SH = 8 * P, FB = 8 * P + 1;  // offset bits, fractional bits of a mesh cell
  constexpr uint32_t FMASK = (1u << FB) - 1u, OMASK = (1u << SH) - 1u;
  constexpr float UNIT = 1.0f / (float)(1u << FB);
  const int B3 = g.B * g.B * g.B;
  const uint32_t mB = (uint32_t)g.B - 1;
  {
    const PC* pp = (const PC*)S.pos + 3 * j;
    const VC* vp = (const VC*)S.vel + 3 * j;
    uint32_t pb[3], vc[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      pb[a] = pp[a];
      vc[a] = vp[a];
    }
    int lo = lo0;  // local cell: largest l in [lo0, hi0) with rel[l] <= jr
    for (int st = (hi0 - lo0) >> 1; st > 0; st >>= 1) lo += rel[lo + st] <= jr ? st : 0;
    const uint32_t lc[3] = {(uint32_t)lo & mB, ((uint32_t)lo >> g.lgB) & mB,
                            (uint32_t)lo >> (2 * g.lgB)};
    int li[3];
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // position in 2^-FB mesh cells (1/512 for P = 1) from the brick's corner node
      const uint32_t gl = (2 * ((lc[a] << SH) | pb[a]) + 1) * (uint32_t)g.r;
      li[a] = (int)(gl >> FB);
      f[a] = (float)(gl & FMASK) * UNIT;
    }
    float acc3[3];
    gather(li, f, acc3);
    if (S.app) {
#pragma unroll
      for (int a = 0; a < 3; ++a) acc3[a] += S.app[3 * j + a];
    }
    const int64_t SP = g.S << (8 * (P - 1));  // position steps per box side
    const uint32_t Sm = (uint32_t)SP - 1;
    const double Sd = (double)SP, invS = 1.0 / Sd;  // powers of two
    PC* tp = (PC*)S.tpos + 3 * j;
    VC* tv = (VC*)S.tvel + 3 * j;
    uint32_t un[3], nl[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float v0 = FAST ? vel_decode_w_v<V>(vc[a], cd.wd) : vel_decode_v<V>(vc[a], cd.vmi);
      const float v1 = v0 + A.ck * acc3[a];
      const double d = floor((double)v1 * A.cdS + 0.5);
      const bool okd = fabs(d) < 4.0e15;
      bad |= !okd;
      // d mod S, exact in float64 (d is an integer below 2^52, S a power of two)
      const double dm = okd ? d - Sd * floor(d * invS) : 0.0;
      un[a] = ((((bc[a] + lc[a]) << SH) | pb[a]) + (uint32_t)dm) & Sm;
      nl[a] = (un[a] >> SH) - bc[a];  // new local cell (wraps above B when outside)
      const int jv = FAST ? vel_code_p2_v<V>(v1, cd.ce) : vel_code_v<V>(v1, cd.vmo);
      tp[a] = (PC)(un[a] & OMASK);
      tv[a] = (VC)jv;
      jmn = min(jmn, jv);
      jmx = max(jmx, jv);
    }
    if (nl[0] <= mB && nl[1] <= mB && nl[2] <= mB) {
      const uint32_t digit = (((nl[2] << g.lgB) | nl[1]) << g.lgB) | nl[0];
      S.tdig[j] = (uint16_t)digit;
      atomicAdd(&run[digit], 1u);
    } else {
      S.tdig[j] = (uint16_t)B3;
      const uint32_t key = cell_key(g, un[0] >> SH, un[1] >> SH, un[2] >> SH);
      S.mkey[j] = key;
      atomicAdd(mvc, 1u);
      atomicAdd(&S.acnt[(key >> (3 * g.lgB)) << A.apad], 1u);
    }
  }
}

// A workgroup-uniform 64-bit value read from LDS, moved to scalar registers.
__device__ inline int64_t uniform64(int64_t v) {
  const uint64_t u = (uint64_t)v;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Each lane's extreme new velocity codes per species over all the chunks it kicked
// (statically indexed, so they stay in registers), reduced over the wave and folded into
// the workgroup's smm[2 s], smm[2 s + 1] once at the end.
struct VelExt {
  int mn[MAXSP], mx[MAXSP];
  __device__ VelExt() {
#pragma unroll
    for (int t = 0; t < MAXSP; ++t) {
      mn[t] = 65536;
      mx[t] = -1;
    }
  }
  __device__ void fold(int s, int a, int b) {
#pragma unroll
    for (int t = 0; t < MAXSP; ++t)
      if (t == s) {
        mn[t] = min(mn[t], a);
        mx[t] = max(mx[t], b);
      }
  }
  __device__ void flush(int n_sp, int* smm) const {
#pragma unroll
    for (int t = 0; t < MAXSP; ++t) {
      if (t >= n_sp) break;
      int a = mn[t], b = mx[t];
      for (int d = 32; d >= 1; d >>= 1) {
        a = min(a, __shfl_xor(a, d, 64));
        b = max(b, __shfl_xor(b, d, 64));
      }
      if ((threadIdx.x & 63) == 0 && b >= 0) {
        atomicMin(&smm[2 * t], a);
        atomicMax(&smm[2 * t + 1], b);
      }
    }
  }
};

// Chunks of 64 particles over a list of segments (one species' particles in one brick,
// or in one z half of it), dealt to the waves of the workgroup in turn. seg(i) gives
// segment i's (species, brick slot, stream range, local cell search range).
struct Seg {
  int s, k;
  int64_t j0, j1;
  int lo, hi;
};

// ---- one brick per workgroup (any shape; R = B r nodes per side) ----
// With STAGE the brick's force nodes [b R, b R + R]^3 are copied to LDS first and every
// particle gathers its 8 CIC nodes from there.
// RS: staged tile side in nodes (compile time), or 0: gather from HBM; P, V: code widths
template <int RS, int P = 1, int V = 2>
__global__ __launch_bounds__(KB) void k_kick_brick(KickArgs A, Geom g, DevErr* err) {
  constexpr bool STAGE = RS > 0;
  const int B = g.B, B3 = B * B * B, L = B3 + 1;
  constexpr int R1 = RS + 1;
  extern __shared__ unsigned char smem[];
  float* F = (float*)smem;  // [3][R1^3] when STAGE
  const int fsz = STAGE ? 3 * R1 * R1 * R1 : 0;
  uint32_t* rel = (uint32_t*)(smem + fsz * 4);  // [MAXSP][L]
  uint32_t* run = rel + MAXSP * L;              // [MAXSP][L]
  __shared__ int64_t l0s[MAXSP];
  __shared__ uint32_t mvc[MAXSP];
  __shared__ int smm[2 * MAXSP];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = xcd_tile(blockIdx.x, g.nbrick);
  const uint32_t kbase = (uint32_t)(b * B3);
  const int64_t ng = g.ng, n3 = ng * ng * ng;
  uint32_t bc[3];
  key_cell(g, kbase, bc[0], bc[1], bc[2]);
  const int64_t ox = (int64_t)bc[0] * g.r, oy = (int64_t)bc[1] * g.r, oz = (int64_t)bc[2] * g.r;
  const int n_sp = A.n_sp;
  for (int i = threadIdx.x; i < n_sp * L; i += KB) {
    const int s = i / L, l = i - s * L;
    const int64_t v0 = A.sp[s].off[kbase];
    rel[i] = (uint32_t)(A.sp[s].off[kbase + l] - v0);
    run[i] = 0;
    if (l == 0) l0s[s] = v0;
  }
  if (threadIdx.x < MAXSP) mvc[threadIdx.x] = 0;
  if (threadIdx.x < 2 * MAXSP) smm[threadIdx.x] = (threadIdx.x & 1) ? -1 : 65536;
  if constexpr (STAGE) {
    // rows of RS nodes (x) as float4 loads, then the x = RS halo column; node (lz, ly)
    // of component c is row (c R1 + lz) R1 + ly. Rows past the end repeat the last row
    // (a duplicate load, not stored), so no load sits behind a branch.
    static_assert(RS % 4 == 0, "staged tile side must be a multiple of 4");
    constexpr int Q = RS / 4;
    constexpr int ROWS = 3 * R1 * R1;
    constexpr int NQ = ROWS * Q;
    constexpr int PQ = (NQ + KB - 1) / KB;
    constexpr int PH = (ROWS + KB - 1) / KB;
    constexpr int RR = R1 * R1;
    constexpr int DR = KB / Q;
    constexpr int DC = DR / RR, DLZ = (DR % RR) / R1, DLY = DR % R1;
    static_assert(KB % Q == 0, "a workgroup covers whole rows");
    const uint32_t mu = (uint32_t)(ng - 1), ngu = (uint32_t)ng;
    const uint32_t oxq = (uint32_t)ox + 4 * (threadIdx.x % Q);
    const uint32_t hx = ((uint32_t)ox + RS) & mu;
    const float* pc0 = A.acc;
    const float* pc1 = A.acc + n3;
    const float* pc2 = A.acc + 2 * n3;
    const int row0 = threadIdx.x / Q;
    float4 vq[PQ];
    float vh[PH];
    {
      int c = row0 / RR, lz = (row0 % RR) / R1, ly = row0 % R1;
#pragma unroll
      for (int k = 0; k < PQ; ++k) {
        const bool over = c >= 3;
        const int cc = over ? 2 : c, zz = over ? R1 - 1 : lz, yy = over ? R1 - 1 : ly;
        const float* pc = cc == 0 ? pc0 : (cc == 1 ? pc1 : pc2);
        const uint32_t gz = ((uint32_t)oz + zz) & mu, gy = ((uint32_t)oy + yy) & mu;
        vq[k] = *(const float4*)(pc + ((uint64_t)(gz * ngu + gy) * ngu + oxq));
        ly += DLY;
        lz += DLZ;
        c += DC;
        if (ly >= R1) { ly -= R1; ++lz; }
        if (lz >= R1) { lz -= R1; ++c; }
      }
    }
#pragma unroll
    for (int k = 0; k < PH; ++k) {
      const int row = min((int)threadIdx.x + k * KB, ROWS - 1);
      const int c = row / RR, rem = row - c * RR;
      const int lz = rem / R1, ly = rem - lz * R1;
      const float* pc = c == 0 ? pc0 : (c == 1 ? pc1 : pc2);
      const uint32_t gz = ((uint32_t)oz + lz) & mu, gy = ((uint32_t)oy + ly) & mu;
      vh[k] = pc[(uint64_t)(gz * ngu + gy) * ngu + hx];
    }
    {
      int c = row0 / RR, lz = (row0 % RR) / R1, ly = row0 % R1;
      const int q4 = 4 * (threadIdx.x % Q);
#pragma unroll
      for (int k = 0; k < PQ; ++k) {
        if (c < 3) {
          float* d = F + ((c * R1 + lz) * R1 + ly) * R1 + q4;
          d[0] = vq[k].x;
          d[1] = vq[k].y;
          d[2] = vq[k].z;
          d[3] = vq[k].w;
        }
        ly += DLY;
        lz += DLZ;
        c += DC;
        if (ly >= R1) { ly -= R1; ++lz; }
        if (lz >= R1) { lz -= R1; ++c; }
      }
    }
#pragma unroll
    for (int k = 0; k < PH; ++k) {
      const int row = threadIdx.x + k * KB;
      if (row < ROWS) F[row * R1 + RS] = vh[k];
    }
  }
  __syncthreads();

  auto gather = [&](const int li[3], const float f[3], float acc3[3]) {
    acc3[0] = acc3[1] = acc3[2] = 0.f;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
          const float wgt = (dx ? f[0] : 1.f - f[0]) * (dy ? f[1] : 1.f - f[1]) *
                            (dz ? f[2] : 1.f - f[2]);
          if constexpr (STAGE) {
            const int node = ((li[2] + dz) * R1 + (li[1] + dy)) * R1 + (li[0] + dx);
            acc3[0] += wgt * F[node];
            acc3[1] += wgt * F[R1 * R1 * R1 + node];
            acc3[2] += wgt * F[2 * R1 * R1 * R1 + node];
          } else {
            const int64_t m = ng - 1;
            const int64_t nz = (oz + li[2] + dz) & m, ny = (oy + li[1] + dy) & m,
                          nx = (ox + li[0] + dx) & m;
            const int64_t node = (nz * ng + ny) * ng + nx;
            acc3[0] += wgt * A.acc[node];
            acc3[1] += wgt * A.acc[n3 + node];
            acc3[2] += wgt * A.acc[2 * n3 + node];
          }
        }
  };
  bool bad = false;
  VelExt ext;
  auto run_all = [&](auto fast_tag) {
    constexpr bool FAST = decltype(fast_tag)::value;
    int64_t cbase = 0;  // chunks of the earlier species
    for (int s = 0; s < n_sp; ++s) {
      const KickSpecies& S = A.sp[s];
      const int64_t l0 = l0s[s];
      const int64_t j0 = min(l0, S.n), j1 = min(l0 + (int64_t)rel[s * L + B3], S.n);
      const int64_t nch = j1 > j0 ? (j1 - j0 + 63) >> 6 : 0;
      const Codec cd = codec_of<V>(S);
      // this wave's chunks of species s: global chunk index = cbase + c, dealt round-robin
      int64_t c = ((int64_t)w - cbase) % NWK;
      if (c < 0) c += NWK;
      int jmn = 65536, jmx = -1;
      for (; c < nch; c += NWK) {
        const int64_t j = j0 + 64 * c + (threadIdx.x & 63);
        if (j < j1)
          kick_lane<FAST, P, V>(S, A, g, cd, j, (uint32_t)(j - l0), rel + s * L, 0, B3, bc,
                                run + s * L, &mvc[s], jmn, jmx, bad, gather);
      }
      ext.fold(s, jmn, jmx);
      cbase += nch;
    }
  };
  if (codec_fast(A)) run_all(std::true_type{});
  else run_all(std::false_type{});
  ext.flush(n_sp, smm);
  __syncthreads();
  for (int i = threadIdx.x; i < n_sp * L; i += KB) {
    const int s = i / L, l = i - s * L;
    if (l < B3) A.sp[s].cnt[kbase + l] = run[i];
  }
  if ((int)threadIdx.x < n_sp) {
    const int s = threadIdx.x;
    A.sp[s].mcnt[b] = mvc[s];
    A.sp[s].pmn[b] = smm[2 * s];
    A.sp[s].pmx[b] = smm[2 * s + 1];
  }
  if (bad) latch_error(err, ERRBIT_RANGE);
}

// ---- two bricks adjacent along x per workgroup, R = 16, in NZ passes over z ----
// Pass h stages the force nodes x in [x0, x0 + 2R], y in [y0, y0 + R], z in
// [z0 + h R/NZ, z0 + (h + 1) R/NZ] (33 x 17 x 5 nodes for NZ = 4) and kicks the
// particles of both bricks' cells in that z slice (whole cell layers). Consecutive
// passes share a node layer, which stays in LDS: the layers form a ring, and passes
// after the first stage only their R/NZ new layers. Rows of the staged tile are 2R
// nodes long, which the memory system serves much faster than rows of R; with NZ = 4
// and 256 threads the tile is 34 KB and four workgroups share a CU, each staging while
// the others compute.
// PHI: the mesh is the potential, and a particle takes the fourth-order differences at its
// eight nodes itself (the same arithmetic as the force gradient pass, so the same bits).
// With a particle per seven nodes, as in this brick shape, that is less work than a pass
// over the nodes that writes three meshes and their staging here: the tile is x in [x0 - 4,
// x0 + 2R + 4), y in [y0 - 2, y0 + R + 2], and nine planes of z that go round like the
// layers above. At 1024^3 with 151 M particles 4.37 ms, and 1.25 for the maximum of the
// force, against 4.86 and 3.39 from the three meshes (512^3, 2-byte codes: 554 + 187 us
// against 634 + 440). Bound by the vector units (half the time) and by bank conflicts of the
// gather (56 words per particle, at random).
constexpr int PR = 16;
constexpr int FX = 2 * PR + 8, FY = PR + 5, FZ = 9;  // PHI: row, rows, planes
template <int NT, int NZ, bool PHI, int P = 1, int V = 2>  // threads, z passes, mesh, widths
__global__ __launch_bounds__(NT, 4) void k_kick_pair(KickArgs A, Geom g, DevErr* err) {
  constexpr int KB = NT, NWK = NT / 64;
  constexpr int X1 = 2 * PR + 1, Y1 = PR + 1, Z1 = PR / NZ + 1;
  constexpr int TS = X1 * Y1 * Z1;  // nodes per component
  static_assert(!PHI || PR / NZ + 5 == FZ, "planes of a z pass with their neighbours");
  const int B = g.B, B3 = B * B * B, L = B3 + 1, H = B3 / NZ;  // H: cells per z pass
  extern __shared__ unsigned char smem[];
  float* F = (float*)smem;                          // [3][Z1][Y1][X1], PHI: [FZ][FY][FX]
  uint32_t* rel = (uint32_t*)(smem + (PHI ? FX * FY * FZ : 3 * TS) * 4);  // [2][MAXSP][L]
  uint32_t* run = rel + 2 * MAXSP * L;              // [2][MAXSP][L]
  __shared__ int64_t l0s[2 * MAXSP];
  __shared__ uint32_t mvc[2 * MAXSP];
  __shared__ int smm[2 * MAXSP];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t p = xcd_tile(blockIdx.x, g.nbrick / 2);
  const int64_t b0 = 2 * p;  // bricks b0, b0 + 1 (x index even, same row)
  const uint32_t kb0 = (uint32_t)(b0 * B3);
  const int64_t ng = g.ng, n3 = ng * ng * ng;
  uint32_t bc0[3];
  key_cell(g, kb0, bc0[0], bc0[1], bc0[2]);
  const int64_t ox = (int64_t)bc0[0] * g.r, oy = (int64_t)bc0[1] * g.r,
                oz = (int64_t)bc0[2] * g.r;
  const int n_sp = A.n_sp;
  for (int i = threadIdx.x; i < 2 * MAXSP * L; i += KB) {
    const int k = i / (MAXSP * L), rem = i - k * (MAXSP * L);
    const int s = rem / L, l = rem - s * L;
    uint32_t v = 0;
    if (s < n_sp) {
      const int64_t v0 = A.sp[s].off[kb0 + k * B3];
      v = (uint32_t)(A.sp[s].off[kb0 + k * B3 + l] - v0);
      if (l == 0) l0s[k * MAXSP + s] = v0;
    }
    rel[i] = v;
    run[i] = 0;
  }
  if (threadIdx.x < 2 * MAXSP) {
    mvc[threadIdx.x] = 0;
    smm[threadIdx.x] = (threadIdx.x & 1) ? -1 : 65536;
  }
  const bool fast = codec_fast(A);
  bool bad = false;
  VelExt ext;

  // The z passes share their boundary layer: pass h needs node layers 4h..4h+4 (for
  // PR / NZ = 4), pass h + 1 starts at 4h + 4. F holds the Z1 layers as a ring, layer
  // 4h + lz in slot (4h + lz) mod Z1, so that pass 0 stages Z1 layers and every later
  // pass only the Z1 - 1 new ones.
  auto stage = [&](int h, auto nl_tag) {
    constexpr int NL = decltype(nl_tag)::value;  // layers loaded: Z1, or Z1 - 1
    constexpr int LZ0 = Z1 - NL;                  // first local layer loaded
    constexpr int Q = 2 * PR / 4;
    constexpr int ROWS = 3 * NL * Y1;
    constexpr int NQ = ROWS * Q;
    constexpr int PQ = (NQ + KB - 1) / KB;
    constexpr int PH = (ROWS + KB - 1) / KB;
    constexpr int RR = NL * Y1;
    constexpr int DR = KB / Q;
    constexpr int DC = DR / RR, DLZ = (DR % RR) / Y1, DLY = DR % Y1;
    static_assert(KB % Q == 0, "a workgroup covers whole rows");
    const uint32_t mu = (uint32_t)(ng - 1), ngu = (uint32_t)ng;
    const uint32_t oz2 = (uint32_t)oz + h * (PR / NZ) + LZ0;
    const int hb = (h * (PR / NZ) + LZ0) % Z1;  // slot of the first loaded layer
    const uint32_t oxq = (uint32_t)ox + 4 * (threadIdx.x % Q);
    const uint32_t hx = ((uint32_t)ox + 2 * PR) & mu;
    const float* pc0 = A.acc;
    const float* pc1 = A.acc + n3;
    const float* pc2 = A.acc + 2 * n3;
    const int row0 = threadIdx.x / Q;
    float4 vq[PQ];
    float vh[PH];
    {
      int c = row0 / RR, lz = (row0 % RR) / Y1, ly = row0 % Y1;
#pragma unroll
      for (int k = 0; k < PQ; ++k) {
        const bool over = c >= 3;
        const int cc = over ? 2 : c, zz = over ? NL - 1 : lz, yy = over ? Y1 - 1 : ly;
        const float* pc = cc == 0 ? pc0 : (cc == 1 ? pc1 : pc2);
        const uint32_t gz = (oz2 + zz) & mu, gy = ((uint32_t)oy + yy) & mu;
        vq[k] = *(const float4*)(pc + ((uint64_t)(gz * ngu + gy) * ngu + oxq));
        ly += DLY;
        lz += DLZ;
        c += DC;
        if (ly >= Y1) { ly -= Y1; ++lz; }
        if (lz >= NL) { lz -= NL; ++c; }
      }
    }
#pragma unroll
    for (int k = 0; k < PH; ++k) {
      const int row = min((int)threadIdx.x + k * KB, ROWS - 1);
      const int c = row / RR, rem = row - c * RR;
      const int lz = rem / Y1, ly = rem - lz * Y1;
      const float* pc = c == 0 ? pc0 : (c == 1 ? pc1 : pc2);
      const uint32_t gz = (oz2 + lz) & mu, gy = ((uint32_t)oy + ly) & mu;
      vh[k] = pc[(uint64_t)(gz * ngu + gy) * ngu + hx];
    }
    __syncthreads();  // the previous pass is done with the slots rewritten here
    {
      int c = row0 / RR, lz = (row0 % RR) / Y1, ly = row0 % Y1;
      const int q4 = 4 * (threadIdx.x % Q);
#pragma unroll
      for (int k = 0; k < PQ; ++k) {
        if (c < 3) {
          int sl = hb + lz;
          sl -= sl >= Z1 ? Z1 : 0;
          float* d = F + ((c * Z1 + sl) * Y1 + ly) * X1 + q4;
          d[0] = vq[k].x;
          d[1] = vq[k].y;
          d[2] = vq[k].z;
          d[3] = vq[k].w;
        }
        ly += DLY;
        lz += DLZ;
        c += DC;
        if (ly >= Y1) { ly -= Y1; ++lz; }
        if (lz >= NL) { lz -= NL; ++c; }
      }
    }
#pragma unroll
    for (int k = 0; k < PH; ++k) {
      const int row = threadIdx.x + k * KB;
      if (row < ROWS) {
        const int c = row / RR, rem = row - c * RR;
        const int lz = rem / Y1, ly = rem - lz * Y1;
        int sl = hb + lz;
        sl -= sl >= Z1 ? Z1 : 0;
        F[((c * Z1 + sl) * Y1 + ly) * X1 + 2 * PR] = vh[k];
      }
    }
    __syncthreads();
  };

  // PHI: plane q of the tile is z0 + q - 2 and lives in slot q mod FZ; pass h needs planes
  // 4h .. 4h + 8
  auto stage_phi = [&](int h, auto np_tag) {
    constexpr int NP = decltype(np_tag)::value;  // planes loaded: FZ, or PR / NZ
    constexpr int Q = FX / 4, NQ = NP * FY * Q, PQ = (NQ + KB - 1) / KB;
    const uint32_t mu = (uint32_t)(ng - 1), ngu = (uint32_t)ng;
    const int q0 = h * (PR / NZ) + (FZ - NP);
    const int sb = q0 % FZ;
    typedef float v4 __attribute__((ext_vector_type(4)));  // (float4 copies went to scratch)
    v4 vq[PQ];
#pragma unroll
    for (int k = 0; k < PQ; ++k) {
      const uint32_t i = min(threadIdx.x + k * KB, (unsigned)NQ - 1u);
      const uint32_t row = i / Q, seg = i - row * Q, pl = row / FY, ry = row - pl * FY;
      const uint32_t gz = ((uint32_t)oz + q0 + pl - 2u) & mu, gy = ((uint32_t)oy + ry - 2u) & mu,
                     gx = ((uint32_t)ox + 4u * seg - 4u) & mu;
      vq[k] = *(const v4*)(A.acc + ((uint64_t)(gz * ngu + gy) * ngu + gx));
    }
    __syncthreads();  // the previous pass is done with the slots rewritten here
#pragma unroll
    for (int k = 0; k < PQ; ++k) {
      const uint32_t i = threadIdx.x + k * KB;
      if (i < NQ) {
        const uint32_t row = i / Q, seg = i - row * Q, pl = row / FY, ry = row - pl * FY;
        int sl = sb + (int)pl;
        sl -= sl >= FZ ? FZ : 0;
        *(v4*)(F + (sl * FY + ry) * FX + 4 * seg) = vq[k];
      }
    }
    __syncthreads();
  };

  // A pass deals 64-particle chunks over each species' particles of the z slice, brick
  // b0's then brick b0 + 1's (the two ranges are apart in the stream), so that a lane's
  // brick k is its own: a species with few particles per slice (16 CDM particles per
  // brick at one per cell) fills one chunk instead of two part-empty ones.
  auto pass = [&](auto fast_tag, int h) {
    constexpr bool FAST = decltype(fast_tag)::value;
    int64_t cbase = 0;  // chunks of the earlier species of this pass
    const int lane = threadIdx.x & 63;
    {
      int k = 0;  // this lane's brick, set per chunk
      auto gather = [&](const int li[3], const float f[3], float acc3[3]) {
        const int tx = li[0] + k * PR, ty = li[1];
        if constexpr (PHI) {
          // slots of the planes z - 2 .. z + 3 around node z = li[2]
          int zo[6];
          int sl = li[2] - h * (PR / NZ) + (h * (PR / NZ)) % FZ;
          sl -= sl >= FZ ? FZ : 0;
#pragma unroll
          for (int q = 0; q < 6; ++q) {
            zo[q] = sl * (FX * FY) + (ty + 2) * FX + tx + 4;
            sl = sl + 1 == FZ ? 0 : sl + 1;
          }
          auto at = [&](int dx, int dy, int dz) { return F[zo[dz + 2] + dy * FX + dx]; };
          acc3[0] = acc3[1] = acc3[2] = 0.f;
#pragma unroll
          for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
              for (int dx = 0; dx < 2; ++dx) {
                const float wgt = (dx ? f[0] : 1.f - f[0]) * (dy ? f[1] : 1.f - f[1]) *
                                  (dz ? f[2] : 1.f - f[2]);
                const float gx = 8.f * (at(dx + 1, dy, dz) - at(dx - 1, dy, dz)) -
                                 (at(dx + 2, dy, dz) - at(dx - 2, dy, dz));
                const float gy = 8.f * (at(dx, dy + 1, dz) - at(dx, dy - 1, dz)) -
                                 (at(dx, dy + 2, dz) - at(dx, dy - 2, dz));
                const float gz = 8.f * (at(dx, dy, dz + 1) - at(dx, dy, dz - 1)) -
                                 (at(dx, dy, dz + 2) - at(dx, dy, dz - 2));
                acc3[0] += wgt * (-A.scale * gx);
                acc3[1] += wgt * (-A.scale * gy);
                acc3[2] += wgt * (-A.scale * gz);
              }
          return;
        }
        // ring slots of the node layers tz and tz + 1 (local to this pass)
        int z0 = li[2] - h * (PR / NZ) + (h * (PR / NZ)) % Z1;
        z0 -= z0 >= Z1 ? Z1 : 0;
        const int z1 = z0 + 1 == Z1 ? 0 : z0 + 1;
        acc3[0] = acc3[1] = acc3[2] = 0.f;
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
          for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
              const float wgt = (dx ? f[0] : 1.f - f[0]) * (dy ? f[1] : 1.f - f[1]) *
                                (dz ? f[2] : 1.f - f[2]);
              const int node = ((dz ? z1 : z0) * Y1 + (ty + dy)) * X1 + (tx + dx);
              acc3[0] += wgt * F[node];
              acc3[1] += wgt * F[TS + node];
              acc3[2] += wgt * F[2 * TS + node];
            }
      };
      for (int s = 0; s < n_sp; ++s) {
        const KickSpecies& S = A.sp[s];
        int64_t l0[2], j0[2], nk[2];  // per brick: first particle, slice start, slice size
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const uint32_t* rs = rel + (kk * MAXSP + s) * L;
          l0[kk] = uniform64(l0s[kk * MAXSP + s]);
          j0[kk] = min(l0[kk] + (int64_t)__builtin_amdgcn_readfirstlane(rs[h * H]), S.n);
          const int64_t j1 =
              min(l0[kk] + (int64_t)__builtin_amdgcn_readfirstlane(rs[(h + 1) * H]), S.n);
          nk[kk] = j1 > j0[kk] ? j1 - j0[kk] : 0;
        }
        const int64_t nt = nk[0] + nk[1];
        const int64_t nch = (nt + 63) >> 6;
        const Codec cd = codec_of<V>(S);
        int64_t c = ((int64_t)w - cbase) % NWK;
        if (c < 0) c += NWK;
        int jmn = 65536, jmx = -1;
        for (; c < nch; c += NWK) {
          const int64_t q = 64 * c + lane;  // position in the two slices, one after the other
          if (q < nt) {
            k = q >= nk[0];
            const int64_t j = k ? j0[1] + (q - nk[0]) : j0[0] + q;
            // brick b0 + 1 is brick b0's neighbour along x (b0 even)
            const uint32_t bc[3] = {bc0[0] + (uint32_t)(k * B), bc0[1], bc0[2]};
            const int sl = k * MAXSP + s;
            kick_lane<FAST, P, V>(S, A, g, cd, j, (uint32_t)(j - (k ? l0[1] : l0[0])),
                                  rel + sl * L, h * H, (h + 1) * H, bc, run + sl * L, &mvc[sl],
                                  jmn, jmx, bad, gather);
          }
        }
        ext.fold(s, jmn, jmx);
        cbase += nch;
      }
    }
  };
  if constexpr (PHI) stage_phi(0, std::integral_constant<int, FZ>{});
  else stage(0, std::integral_constant<int, Z1>{});
  if (fast) pass(std::true_type{}, 0);
  else pass(std::false_type{}, 0);
#pragma nounroll
  for (int h = 1; h < NZ; ++h) {
    if constexpr (PHI) stage_phi(h, std::integral_constant<int, PR / NZ>{});
    else stage(h, std::integral_constant<int, Z1 - 1>{});
    if (fast) pass(std::true_type{}, h);
    else pass(std::false_type{}, h);
  }
  ext.flush(n_sp, smm);
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * MAXSP * L; i += KB) {
    const int k = i / (MAXSP * L), rem = i - k * (MAXSP * L);
    const int s = rem / L, l = rem - s * L;
    if (s < n_sp && l < B3) A.sp[s].cnt[kb0 + k * B3 + l] = run[i];
  }
  if ((int)threadIdx.x < 2 * n_sp) {
    const int k = threadIdx.x / n_sp, s = threadIdx.x - k * n_sp;
    A.sp[s].mcnt[b0 + k] = mvc[k * MAXSP + s];
    A.sp[s].pmn[b0 + k] = smm[2 * s];
    A.sp[s].pmx[b0 + k] = smm[2 * s + 1];
  }
  if (bad) latch_error(err, ERRBIT_RANGE);
}

// ----------------------------------------------------------------- re-sort --
// Every kernel of the re-sort takes all species in one launch (grid.y).
struct PlaceSpecies {
  int64_t n;
  const int64_t* off;      // old cell offsets [ncell3 + 1]
  const uint16_t* tdig;    // per particle: new local cell, or B^3 for movers
  const uint32_t* mkey;    // movers: new cell key, at the old stream index
  const void* tpos;        // new codes, old stream order
  const void* tvel;
  uint32_t* cnt;           // stayers per cell; the new count of cells of 255 and more
  uint32_t* mcnt;          // movers per brick; after the scan: the bricks that k_place left
  uint32_t* acnt;          // arrivals per brick (counted down to 0 as they are listed)
  const int32_t* pmn;      // per-brick extreme new velocity codes
  const int32_t* pmx;
  int64_t* bstart;         // first new stream position of each brick [nbrick + 1]
  uint32_t* astart;        // first arrival of each brick [nbrick + 1]
  uint32_t* aidx;          // old stream indices of the arrivals, by brick
  uint32_t* abuf;          // the same size, for sorting long lists
  uint32_t* ecnt;          // cells of 255 and more per brick
  uint32_t* etile;         // the same per ET bricks
  uint32_t* tot;           // [0] their total, [1] crowded bricks, [2] bricks of long lists
  int64_t crowd;           // a brick of more stayers is crowded
  pm_shdr* hout;
  void* pos;
  void* vel;
  uint8_t* count;
  uint64_t* esc;
  int64_t cap_esc;
  int64_t* perm;           // nullable: new stream position -> old
};
struct PlaceArgs {
  PlaceSpecies sp[MAXSP];
  int apad;
};
constexpr int ET = 4096;
constexpr int64_t APAD_LEAST = 1 << 16, APAD_MOST = 1 << 20;

// First new stream position and first arrival of every brick: exclusive prefixes of the
// bricks' new particle counts (old particles less movers plus arrivals) and of their
// arrivals. One launch up to BS_TILE bricks; beyond that k_brick_sums first leaves each
// block's sums, and a block of k_brick_scan adds up those before its own (at most 2048: a kick
// of more than 2^21 bricks exceeds the largest grid). The extreme velocity codes ride along
// and end in the header. A brick per thread: the loads of distant offsets and counters are
// what takes the time (32768 bricks, sums and scan 36 us with four per thread, 18 with one).
constexpr int LONG = 1024;  // arrivals of a brick that one wave sorts
constexpr int BS_T = 1024, BS_I = 1, BS_TILE = BS_T * BS_I;
struct BrickSum {
  int64_t tot, arr;
  int32_t mn, mx;
};

__device__ inline void brick_items(const PlaceSpecies& S, int apad, int B3, int64_t nbrick, int64_t b0,
                                   uint32_t t[BS_I], uint32_t a[BS_I], int& mn, int& mx) {
  mn = 65536;
  mx = -1;
#pragma unroll
  for (int k = 0; k < BS_I; ++k) {
    const int64_t b = b0 + k;
    t[k] = a[k] = 0;
    if (b >= nbrick) continue;
    const int64_t j0 = min(S.off[b * B3], S.n), j1 = min(S.off[(b + 1) * B3], S.n);
    a[k] = S.acnt[b << apad];
    const int64_t v = (j1 > j0 ? j1 - j0 : 0) - (int64_t)S.mcnt[b] + (int64_t)a[k];
    t[k] = (uint32_t)(v > 0 ? v : 0);
    mn = min(mn, S.pmn[b]);
    mx = max(mx, S.pmx[b]);
  }
}

// block-wide extremes; sm: 2 x 16 ints of LDS. Valid in thread 0.
__device__ inline void block_extremes(int& mn, int& mx, int* sm) {
  for (int d = 32; d >= 1; d >>= 1) {
    mn = min(mn, __shfl_xor(mn, d, 64));
    mx = max(mx, __shfl_xor(mx, d, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sm[w] = mn;
    sm[16 + w] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int q = 1; q < (int)(blockDim.x >> 6); ++q) {
      mn = min(mn, sm[q]);
      mx = max(mx, sm[16 + q]);
    }
}

__global__ __launch_bounds__(BS_T) void k_brick_sums(PlaceArgs A, int B3, int64_t nbrick,
                                                     BrickSum* sums) {
  __shared__ int64_t lw[BS_T / 64 + 1];
  __shared__ int sm[32];
  uint32_t t[BS_I], a[BS_I];
  int mn, mx;
  brick_items(A.sp[blockIdx.y], A.apad, B3, nbrick, (int64_t)blockIdx.x * BS_TILE + threadIdx.x * BS_I,
              t, a, mn, mx);
  int64_t st = 0, sa = 0, tt, ta;
#pragma unroll
  for (int k = 0; k < BS_I; ++k) {
    st += t[k];
    sa += a[k];
  }
  pmscan::block_excl_scan(st, lw, &tt);
  pmscan::block_excl_scan(sa, lw, &ta);
  block_extremes(mn, mx, sm);
  if (threadIdx.x == 0) sums[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = BrickSum{tt, ta, mn, mx};
}

__global__ __launch_bounds__(BS_T) void k_brick_scan(PlaceArgs A, int B3, int64_t nbrick,
                                                     const BrickSum* sums) {
  __shared__ int64_t lw[BS_T / 64 + 1];
  __shared__ int sm[32];
  const PlaceSpecies& S = A.sp[blockIdx.y];
  const int64_t b0 = (int64_t)blockIdx.x * BS_TILE + threadIdx.x * BS_I;
  uint32_t t[BS_I], a[BS_I];
  int mn, mx;
  brick_items(S, A.apad, B3, nbrick, b0, t, a, mn, mx);
  int64_t pt = 0, pa = 0;  // the sums of the blocks before this one
  if (gridDim.x > 1) {
    const BrickSum* bs = sums + (int64_t)blockIdx.y * gridDim.x;
    const int nb = blockIdx.x == 0 ? (int)gridDim.x : (int)blockIdx.x;
    for (int i = threadIdx.x; i < nb; i += BS_T) {
      const BrickSum q = bs[i];
      pt += i < (int)blockIdx.x ? q.tot : 0;
      pa += i < (int)blockIdx.x ? q.arr : 0;
      mn = min(mn, q.mn);
      mx = max(mx, q.mx);
    }
    int64_t x;
    pmscan::block_excl_scan(pt, lw, &x);
    pt = x;
    pmscan::block_excl_scan(pa, lw, &x);
    pa = x;
  }
  if (blockIdx.x == 0) {  // it has seen every block's extremes
    block_extremes(mn, mx, sm);
    if (threadIdx.x == 0) {
      S.hout->j_min = mn;
      S.hout->j_max = mx;
    }
  }
  int64_t st = 0, sa = 0, tt, ta;
#pragma unroll
  for (int k = 0; k < BS_I; ++k) {
    st += t[k];
    sa += a[k];
  }
  int64_t et = pt + pmscan::block_excl_scan(st, lw, &tt);
  int64_t ea = pa + pmscan::block_excl_scan(sa, lw, &ta);
#pragma unroll
  for (int k = 0; k < BS_I; ++k) {
    const int64_t b = b0 + k;
    if (b < nbrick) {
      S.bstart[b] = et;
      S.astart[b] = (uint32_t)ea;
    }
    et += t[k];
    ea += a[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    S.bstart[nbrick] = pt + tt;
    S.astart[nbrick] = (uint32_t)(pa + ta);
  }
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same for global memory that only this wave's workgroup writes and reads. (A device-wide
// fence writes back and drops the XCD's L2 every time: bricks of 512 arrivals then took five
// times as long.)
__device__ __forceinline__ void wave_sync_global() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The movers into the lists of the bricks they arrive in, in no particular order (the
// brick's wave sorts its list by old index). A thread looks at MV particles' digits in one
// 16-byte load. A mover costs a chain of dependent accesses (key, its brick's counter, the
// list), and movers are a few per wave's 512 particles, so the wave first queues them in
// LDS and then takes 64 chains at a time instead of up to eight one after the other: 219 ->
// 112 us with 151 M particles in 262144 bricks, 78 -> 64 us with 18.9 M in 4096 (the rest
// is the atomics on few counters).
constexpr int MV = 8;
__global__ __launch_bounds__(KT) void k_list_arrivals(PlaceArgs A, int lgB3, int64_t nbrick,
                                                     DevErr* err) {
  __shared__ uint16_t queue[KT / 64][64 * MV];
  const PlaceSpecies& S = A.sp[blockIdx.y];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = ((int64_t)blockIdx.x * KT + (threadIdx.x & ~63)) * MV;  // the wave's first
  if (base >= S.n) return;
  const int64_t i = base + lane * MV;
  uint32_t d[MV];
  if (i + MV <= S.n) {  // tdig is 16-byte aligned
    const uint4 q = *(const uint4*)(S.tdig + i);
    const uint32_t v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < MV; ++k) d[k] = (v[k >> 1] >> (16 * (k & 1))) & 0xffffu;
  } else {
#pragma unroll
    for (int k = 0; k < MV; ++k) d[k] = i + k < S.n ? S.tdig[i + k] : 0u;
  }
  const uint32_t mover = 1u << lgB3;
  const uint64_t lt = lane ? ((~0ull) >> (64 - lane)) : 0ull;
  int m = 0;
#pragma unroll
  for (int k = 0; k < MV; ++k) {
    const uint64_t at = __ballot(d[k] == mover);
    if (d[k] == mover) queue[w][m + __popcll(at & lt)] = (uint16_t)(lane * MV + k);
    m += __popcll(at);
  }
  wave_sync();
  for (int q = lane; q < m; q += 64) {
    const int64_t j = base + queue[w][q];
    const int64_t b = S.mkey[j] >> lgB3;
    // counts inconsistent with n (latched by the offset check) leave stale digits
    const bool ok = b < nbrick;
    const uint32_t first = S.astart[ok ? b : 0];
    const uint32_t left = ok ? atomicSub(&S.acnt[b << A.apad], 1u) : 0u;
    const int64_t slot = left ? (int64_t)first + left - 1 : S.n;
    if (slot < S.n) S.aidx[slot] = (uint32_t)j;
    else latch_error(err, ERRBIT_CORRUPT);
  }
}

// Lanes of the wave whose `valid` digit equals this lane's.
__device__ __forceinline__ uint64_t wave_match(uint32_t d, bool valid, int nbits) {
  uint64_t match = __ballot(valid);
  for (int b = 0; b < nbits; ++b) {
    const uint64_t m = __ballot(valid && ((d >> b) & 1u));
    match &= ((d >> b) & 1u) ? m : ~m;
  }
  return match;
}

// Ascending bitonic sort of a[0, n) in LDS by one wave, n a power of two.
__device__ __forceinline__ void wave_sort_lds(uint32_t* a, int n) {
  const int lane = threadIdx.x & 63;
#pragma nounroll
  for (int run = 2; run <= n; run <<= 1) {
#pragma nounroll
    for (int d = run >> 1; d >= 1; d >>= 1) {
#pragma unroll 2
      for (int i = lane; i < n / 2; i += 64) {
        const int p = 2 * i - (i & (d - 1));
        const uint32_t x = a[p], y = a[p + d];
        const bool swap = (x > y) == !(p & run);
        a[p] = swap ? y : x;
        a[p + d] = swap ? x : y;
      }
      wave_sync();
    }
  }
}

// Ascending sort of a[0, m) in global memory by a workgroup of NW waves (stable 8-bit digit
// passes, an even number of them through b so that the result is in a): lists too long for
// k_place. Each wave takes a contiguous part. hist: [NW][256] words of LDS. bits: significant
// bits of the values.
template <int NW>
__device__ void block_sort_long(uint32_t* a, uint32_t* b, int64_t m, int bits, uint32_t* hist,
                                int* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t lt = lane ? ((~0ull) >> (64 - lane)) : 0ull;
  const int64_t per = ((m + NW - 1) / NW + 63) / 64 * 64;
  const int64_t i0 = min(w * per, m), i1 = min(i0 + per, m);
  uint32_t* my = hist + 256 * w;
  for (int shift = 0; shift < (bits <= 16 ? 16 : 32); shift += 8) {
    for (int q = lane; q < 256; q += 64) my[q] = 0;
    wave_sync();
    for (int64_t i = i0 + lane; i < i1; i += 64) atomicAdd(&my[(a[i] >> shift) & 255u], 1u);
    __syncthreads();
    uint32_t s = 0;
    if (threadIdx.x < 256)
      for (int q = 0; q < NW; ++q) s += hist[256 * q + threadIdx.x];
    uint32_t at = (uint32_t)pmscan::block_excl_scan_i32((int)s, wsum);
    if (threadIdx.x < 256)
      for (int q = 0; q < NW; ++q) {
        const uint32_t c = hist[256 * q + threadIdx.x];
        hist[256 * q + threadIdx.x] = at;
        at += c;
      }
    __syncthreads();
    for (int64_t j0 = i0; j0 < i1; j0 += 64) {
      const bool valid = j0 + lane < i1;
      const uint32_t v = valid ? a[j0 + lane] : 0u, d = (v >> shift) & 255u;
      const uint64_t match = wave_match(d, valid, 8);
      const uint32_t rk = (uint32_t)__popcll(match & lt);
      const uint32_t to = my[d];
      wave_sync();
      if (valid && rk == 0) my[d] = to + (uint32_t)__popcll(match);
      wave_sync();
      if (valid) b[to + rk] = v;
    }
    __syncthreads();  // the other waves read b next
    uint32_t* t = a;
    a = b;
    b = t;
  }
}

// One particle per valid lane to its cell's next positions, in lane order; run: the running
// positions, relative to `first`.
template <typename PC, typename VC>
__device__ __forceinline__ void place_put(const PlaceSpecies& S, uint32_t* run, int64_t first,
                                          int nbits, bool valid, uint32_t d, int64_t j,
                                          const PC (&p)[3], const VC (&v)[3], DevErr* err) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lane ? ((~0ull) >> (64 - lane)) : 0ull;
  const uint64_t match = wave_match(d, valid, nbits);
  const uint32_t rk = (uint32_t)__popcll(match & lt);
  uint32_t at = 0;
  if (valid) at = run[d];
  wave_sync();
  if (valid && rk == 0) run[d] = at + (uint32_t)__popcll(match);
  wave_sync();
  if (!valid) return;
  const int64_t dst = first + at + rk;
  if (dst < 0 || dst >= S.n) {
    latch_error(err, ERRBIT_CORRUPT);
    return;
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ((PC*)S.pos)[3 * dst + a] = p[a];
    ((VC*)S.vel)[3 * dst + a] = v[a];
  }
  if (S.perm) S.perm[dst] = j;
}

// Final stream positions. A brick's new particles, cell by cell, are its arrivals from
// earlier bricks, its stayers and its arrivals from later bricks, each in old stream
// order: one running position per cell serves them one after the other, and ranks within a
// chunk of 64 come from a multi-split by digit. NW = 1: one wave per brick, WB bricks per
// workgroup, no barrier; the stayers per cell are the kick's counts. NW > 1: a workgroup of
// NW waves per brick, each with a contiguous part of the stayers and its own running
// positions (from a first pass over the digits): for bricks of thousands of particles,
// which one wave takes 80 chunks for. The new count bytes are written here too, so that no
// pass over the cells follows. A brick of more than CAP arrivals or of many times the mean of
// stayers is only counted here and left to k_place_rest, whose code this kernel's waves then
// need not fetch (with it here a step at 64^3 took 92.0 us, 90.1 without).
constexpr int WB = 4;       // bricks per workgroup (NW = 1)
constexpr int PU = 4;       // chunks whose loads are issued together
constexpr int ACAP = 256;   // arrivals ranked in LDS, per wave
template <int P, int V, int NW>
__global__ __launch_bounds__(NW == 1 ? 64 * WB : 64 * NW) void k_place(
    PlaceArgs A, int B3, int nbits, int64_t nbrick, DevErr* err) {
  using PC = typename PosCode<P>::T;
  using VC = typename VelCode<V>::T;
  const PlaceSpecies& S = A.sp[blockIdx.y];
  const PC* tpos = (const PC*)S.tpos;
  const VC* tvel = (const VC*)S.tvel;
  constexpr int NT = 64 * NW, CAP = ACAP * NW;
  extern __shared__ uint32_t lds[];
  __shared__ int wsum[16];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tid = NW == 1 ? lane : (int)threadIdx.x;  // thread of the brick
  const int bw = NW == 1 ? 0 : wv;                    // wave of the brick
  // [CAP] arrivals (16-byte aligned)
  uint32_t* al = lds + (NW == 1 ? wv * (CAP + ((B3 + 3) & ~3)) : 0);
  uint32_t* runs = al + CAP;                             // [NW][B3] running positions
  uint32_t* run = runs + bw * B3;
  const int64_t b = (int64_t)blockIdx.x * (NW == 1 ? WB : 1) + (NW == 1 ? wv : 0);
  if (b >= nbrick) return;  // the whole wave (NW = 1)
  auto sync = [] {
    if constexpr (NW == 1) wave_sync();
    else __syncthreads();
  };
  const uint64_t lt = lane ? ((~0ull) >> (64 - lane)) : 0ull;
  const int64_t kbase = b * B3, n = S.n;
  const int64_t j0 = min(S.off[kbase], n), j1 = min(S.off[kbase + B3], n);
  const int64_t a0 = S.astart[b];
  const int64_t m = (int64_t)S.astart[b + 1] - a0;  // arrivals

  const bool crowded = j1 - j0 > S.crowd || m > LONG, rest = m > CAP || crowded;

  // the arrivals in old stream order: al[0, m) (aidx[a0, a0 + m), in no order, for the rest)
  for (int l = tid; l < NW * B3; l += NT) runs[l] = 0;
  if (!rest) {
    uint32_t v[ACAP / 64], r[ACAP / 64];
#pragma unroll
    for (int k = 0; k < ACAP / 64; ++k) {
      const int i = tid + k * NT;
      v[k] = i < m ? S.aidx[a0 + i] : 0xffffffffu;
      r[k] = 0;
      if (k * NT < m) al[i] = v[k];
    }
    sync();
    const int m4 = ((int)m + 3) & ~3;  // the slots up to the next multiple of NT are padding
    for (int q = 0; q < m4; q += 4) {
      const uint4 x = *(const uint4*)(al + q);
#pragma unroll
      for (int k = 0; k < ACAP / 64; ++k)
        r[k] += (x.x < v[k]) + (x.y < v[k]) + (x.z < v[k]) + (x.w < v[k]);
    }
    sync();
#pragma unroll
    for (int k = 0; k < ACAP / 64; ++k)
      if (tid + k * NT < m) al[r[k]] = v[k];
  }
  sync();
  auto arrival = [&](int64_t i) { return (int64_t)(rest ? S.aidx[a0 + i] : al[i]); };

  // arrivals per cell (those from earlier bricks count with the first wave, the others
  // with the last), and for NW > 1 each wave's stayers
  int64_t early = 0;  // arrivals from earlier bricks
  for (int64_t i = tid; i - tid < m; i += NT) {
    const int64_t j = i < m ? arrival(i) : n;
    const bool e = j < j0;
    if (j < n) {
      const uint32_t d = S.mkey[j] - (uint32_t)kbase;
      if (d < (uint32_t)B3) atomicAdd(&runs[(e || NW == 1 ? 0 : NW - 1) * B3 + d], 1u);
    }
    if constexpr (NW == 1) early += __popcll(__ballot(e));
    else early += __syncthreads_count(e);
  }
  // this wave's stayers: [s0, s1)
  const int64_t per = NW == 1 ? j1 - j0 : ((j1 - j0 + NW - 1) / NW + 63) / 64 * 64;
  const int64_t s0 = min(j0 + bw * per, j1), s1 = min(s0 + per, j1);
  if (NW > 1 && !rest) {
    for (int64_t base = s0; base < s1; base += 64 * PU) {
      uint32_t d[PU];
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const int64_t j = base + 64 * u + lane;
        d[u] = j < s1 ? S.tdig[j] : (uint32_t)B3;
      }
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (d[u] < (uint32_t)B3) atomicAdd(&run[d[u]], 1u);
    }
  }
  sync();
  // new counts, count bytes, escapes, and the running positions (relative to the brick's
  // first new position; exclusive prefix over the cells, then over the waves)
  const int64_t first = S.bstart[b];
  uint32_t carry = 0;
  int ne = 0;
  for (int l0 = 0; l0 < B3; l0 += NT) {
    const int l = l0 + tid;
    uint32_t x = 0;
    if (l < B3) {
      if (NW == 1 || rest) x = S.cnt[kbase + l];
#pragma unroll
      for (int q = 0; q < NW; ++q) x += runs[q * B3 + l];
      S.count[kbase + l] = (uint8_t)(x >= 255u ? 255u : x);
      if (x >= 255u) {
        S.cnt[kbase + l] = x;
        ++ne;
      }
    }
    uint32_t ex, tot;
    if constexpr (NW == 1) {
      const uint32_t inc = (uint32_t)pmscan::wave_incl_scan_dpp((int)x);
      ex = inc - x;
      tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    } else {
      ex = (uint32_t)pmscan::block_excl_scan_i32((int)x, wsum);
      tot = 0;
      for (int q = 0; q < NW; ++q) tot += (uint32_t)wsum[q];
      __syncthreads();
    }
    if (l < B3) {
      uint32_t at = carry + ex;
      if constexpr (NW == 1) {
        runs[l] = at;
      } else {
#pragma unroll
        for (int q = 0; q < NW; ++q) {
          const uint32_t c = runs[q * B3 + l];
          runs[q * B3 + l] = at;
          at += c;
        }
      }
    }
    carry += tot;
  }
  {
    for (int d = 32; d >= 1; d >>= 1) ne += __shfl_xor(ne, d, 64);
    if constexpr (NW > 1) {
      __syncthreads();
      if (lane == 0) wsum[bw] = ne;
      __syncthreads();
      ne = 0;
      for (int q = 0; q < NW; ++q) ne += wsum[q];
    }
    if (tid == 0) {
      S.ecnt[b] = (uint32_t)ne;
      if (ne) {
        atomicAdd(&S.tot[0], (uint32_t)ne);
        atomicAdd(&S.etile[b / ET], (uint32_t)ne);
      }
      // the crowded bricks from the front of the array, those of long lists from its end
      if (crowded) S.mcnt[atomicAdd(&S.tot[1], 1u)] = (uint32_t)b;
      else if (rest) S.mcnt[nbrick - 1 - atomicAdd(&S.tot[2], 1u)] = (uint32_t)b;
    }
  }
  if (rest) return;  // uniform: the wave (NW = 1) or the workgroup
  sync();
  auto put = [&](bool valid, uint32_t d, int64_t j, const PC (&p)[3], const VC (&v)[3]) {
    place_put(S, run, first, nbits, valid, d, j, p, v, err);
  };
  auto put_arrivals = [&](int64_t i0, int64_t i1) {
    for (int64_t i = i0; i < i1; i += 64) {
      const int64_t j = i + lane < i1 ? arrival(i + lane) : n;
      const uint32_t d = j < n ? S.mkey[j] - (uint32_t)kbase : (uint32_t)B3;
      const bool valid = d < (uint32_t)B3;
      PC p[3];
      VC v[3];
      const int64_t jj = valid ? j : 0;  // n > 0 whenever there are arrivals
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        p[a] = tpos[3 * jj + a];
        v[a] = tvel[3 * jj + a];
      }
      put(valid, d, j, p, v);
    }
  };
  if (bw == 0) put_arrivals(0, early);
  for (int64_t base = s0; base < s1; base += 64 * PU) {
    uint32_t d[PU];
    PC p[PU][3];
    VC v[PU][3];
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int64_t j = base + 64 * u + lane;
      const bool h = j < s1;
      const int64_t jj = h ? j : s0;
      d[u] = h ? S.tdig[jj] : (uint32_t)B3;  // past the end: not a stayer
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        p[u][a] = tpos[3 * jj + a];
        v[u][a] = tvel[3 * jj + a];
      }
    }
#pragma unroll
    for (int u = 0; u < PU; ++u)
      put(d[u] < (uint32_t)B3, d[u], base + 64 * u + lane, p[u], v[u]);
  }
  if (bw == NW - 1) put_arrivals(early, m);
}

// The escape table, then the bricks that k_place left. Without any of the two (the rule: cells
// of 255 particles and crowded bricks are rare) every workgroup returns after one load.
//
// Escapes in cell order: a workgroup takes ET bricks at a time; the escapes before them are the
// sum of the earlier tiles' counts, at most 512, one load per thread. (Adding up every earlier
// brick's count took the last workgroup 1024 rounds at 1024^3: 291 us with 400 escapes, now 36.)
//
// A brick's sequence of early arrivals, old particles and late arrivals is dealt to the waves in
// contiguous parts: a pass counts each wave's particles per cell, a prefix over cells and waves
// gives its running positions, a second pass places them. A brick of a long list takes one
// wave, a crowded one the whole workgroup: one wave takes 600 ns for a chunk of 64, all in one
// chain (1.9 M particles in one brick: 19.1 ms in k_place, 3.8 here).
constexpr int RT = 1024, RW = RT / 64;

// NW waves (all of the workgroup's, or this one alone) place brick b. lds: [NW][LONG].
template <int P, int V, int NW>
__device__ __forceinline__ void place_brick(const PlaceSpecies& S, int64_t b, int B3, int nbits,
                                            int nbits_idx, uint32_t* lds, int* wsum,
                                            DevErr* err) {
  using PC = typename PosCode<P>::T;
  using VC = typename VelCode<V>::T;
  const PC* tpos = (const PC*)S.tpos;
  const VC* tvel = (const VC*)S.tvel;
  const int lane = threadIdx.x & 63;
  const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tid = NW == 1 ? lane : (int)threadIdx.x;
  auto sync = [] {
    if constexpr (NW == 1) wave_sync();
    else __syncthreads();
  };
  const int64_t kbase = b * B3, n = S.n;
  const int64_t j0 = min(S.off[kbase], n), j1 = max(j0, min(S.off[kbase + B3], n));
  const int64_t a0 = S.astart[b], m = (int64_t)S.astart[b + 1] - a0;
  uint32_t* run = lds + w * B3;
  static_assert(LONG >= 512, "the cells of a brick and the digits of a sort fit");
  sync();  // the last brick is done with the LDS
  if constexpr (NW == 1) {
    const int full = m <= LONG / 2 ? LONG / 2 : LONG;
    for (int i = lane; i < full; i += 64) lds[i] = i < m ? S.aidx[a0 + i] : 0xffffffffu;
    wave_sync();
    wave_sort_lds(lds, full);
    for (int i = lane; i < m; i += 64) S.aidx[a0 + i] = lds[i];
    wave_sync_global();  // the wave reads them back
  } else {
    block_sort_long<NW>(S.aidx + a0, S.abuf + a0, m, nbits_idx, lds, wsum);
  }
  int64_t early = 0;  // arrivals from earlier bricks: before the first with index j0 or more
  for (int64_t hi = m; early < hi;) {
    const int64_t mid = (early + hi) >> 1;
    if ((int64_t)S.aidx[a0 + mid] < j0) early = mid + 1; else hi = mid;
  }
  for (int l = tid; l < NW * B3; l += 64 * NW) lds[l] = 0;
  sync();
  const int64_t all = m + (j1 - j0), late = early + (j1 - j0);
  const int64_t per = ((all + NW - 1) / NW + 63) / 64 * 64;
  const int64_t v0 = min(w * per, all), v1 = min(v0 + per, all);
  // element q of the sequence: its old stream index and digit (B3: none). An arrival's key lies
  // anywhere, so its digit is left in abuf for the second pass.
  auto item = [&](int64_t q, int64_t& j, bool again) -> uint32_t {
    if (q >= v1) return (uint32_t)B3;
    const bool old = q >= early && q < late;
    const int64_t i = a0 + (q < early ? q : q - (j1 - j0));
    j = old ? j0 + (q - early) : (int64_t)S.aidx[i];
    if (j >= n) return (uint32_t)B3;  // an inconsistent count (latched)
    if (old) return (uint32_t)S.tdig[j];
    if (again) return S.abuf[i];
    const uint32_t d = min(S.mkey[j] - (uint32_t)kbase, (uint32_t)B3);
    S.abuf[i] = d;
    return d;
  };
  for (int64_t q0 = v0; q0 < v1; q0 += 64 * PU) {
    uint32_t d[PU];
    int64_t j;
#pragma unroll
    for (int u = 0; u < PU; ++u) d[u] = item(q0 + 64 * u + lane, j, false);
#pragma unroll
    for (int u = 0; u < PU; ++u)
      if (d[u] < (uint32_t)B3) atomicAdd(&run[d[u]], 1u);
  }
  sync();
  uint32_t carry = 0;
  for (int l0 = 0; l0 < B3; l0 += 64 * NW) {  // (once, for a whole workgroup)
    const int l = l0 + tid;
    uint32_t x = 0;
    if (l < B3)
      for (int q = 0; q < NW; ++q) x += lds[q * B3 + l];
    uint32_t at = carry;
    if constexpr (NW == 1) {
      const uint32_t inc = (uint32_t)pmscan::wave_incl_scan_dpp((int)x);
      at += inc - x;
      carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    } else {
      at += (uint32_t)pmscan::block_excl_scan_i32((int)x, wsum);
    }
    if (l < B3)
      for (int q = 0; q < NW; ++q) {
        const uint32_t c = lds[q * B3 + l];
        lds[q * B3 + l] = at;
        at += c;
      }
  }
  if constexpr (NW == 1) wave_sync_global();  // the digits in abuf
  else __syncthreads();
  const int64_t first = S.bstart[b];
  for (int64_t q0 = v0; q0 < v1; q0 += 64 * PU) {
    uint32_t d[PU];
    int64_t j[PU];
    PC p[PU][3];
    VC v[PU][3];
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      j[u] = 0;  // n > 0: the brick has particles
      d[u] = item(q0 + 64 * u + lane, j[u], true);
      const int64_t jj = d[u] < (uint32_t)B3 ? j[u] : 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        p[u][a] = tpos[3 * jj + a];
        v[u][a] = tvel[3 * jj + a];
      }
    }
#pragma unroll
    for (int u = 0; u < PU; ++u)
      place_put(S, run, first, nbits, d[u] < (uint32_t)B3, d[u], j[u], p[u], v[u], err);
  }
}

template <int P, int V>
__global__ __launch_bounds__(RT, 8) void k_place_rest(PlaceArgs A, int B3, int nbits,
                                                     int64_t nbrick, int nbits_idx, DevErr* err) {
  const PlaceSpecies& S = A.sp[blockIdx.y];
  const uint32_t total = S.tot[0], crowded = S.tot[1], listed = S.tot[2];
  if ((total | crowded | listed) == 0) return;  // the header's n_esc is 0 already
  extern __shared__ uint32_t lds[];  // [RW][LONG]
  __shared__ int64_t lw[RW + 1];
  __shared__ int wsum[RW];
  if (total > 0) {
    const int64_t nt = (nbrick + ET - 1) / ET;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
      if (S.etile[t] == 0) continue;
      int64_t before = 0, tot;
      for (int64_t q = threadIdx.x; q < t; q += RT) before += S.etile[q];
      pmscan::block_excl_scan(before, lw, &tot);
      int64_t at = tot;
      const int64_t q1 = min((t + 1) * ET, nbrick);
      for (int64_t b0 = t * ET; b0 < q1; b0 += RT) {
        const int64_t b = b0 + threadIdx.x;
        const uint32_t ne = b < q1 ? S.ecnt[b] : 0u;
        int64_t k = at + pmscan::block_excl_scan((int64_t)ne, lw, &tot);
        at += tot;
        if (!ne) continue;
        for (int64_t i = b * B3; i < (b + 1) * B3; ++i)
          if (S.count[i] == 255) {
            if (k < S.cap_esc) {
              S.esc[2 * k] = (uint64_t)i;
              S.esc[2 * k + 1] = (uint64_t)S.cnt[i];
            }
            ++k;
          }
      }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      S.hout->n_esc = (int64_t)total;
      if ((int64_t)total > S.cap_esc) latch_error(err, ERRBIT_CAPACITY, (int64_t)total);
    }
  }
  for (uint32_t h = blockIdx.x; h < crowded; h += gridDim.x)
    place_brick<P, V, RW>(S, __builtin_amdgcn_readfirstlane(S.mcnt[h]), B3, nbits, nbits_idx, lds,
                          wsum, err);
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (uint32_t h = w * gridDim.x + blockIdx.x; h < listed; h += RW * gridDim.x)
    place_brick<P, V, 1>(S, __builtin_amdgcn_readfirstlane(S.mcnt[nbrick - 1 - h]), B3, nbits,
                         nbits_idx, lds + w * LONG, wsum, err);
}

}  // namespace

pm_status run_kick_float(pm_context* c, const pm_species* in, pm_species* out,
                         const float* acc, double ck, double cd) {
  if (in->n == 0) return PM_OK;
  ProfScope ps(c, ST_KICK);
  hipLaunchKernelGGL(k_kick_float, dim3((unsigned)cdiv(in->n, KT)), dim3(KT), 0, c->stream,
                     in->x, in->v, out->x, out->v, in->n, acc, c->g.ng, c->g.ngL,
                     (float)c->g.box, (float)ck, (float)cd);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

// two bricks per workgroup: R = 16, an even number of bricks per side, z quarters of
// whole cells
static size_t pair_bytes(const Geom& g) {
  return (size_t)3 * (2 * PR + 1) * (PR + 1) * (PR / 4 + 1) * 4 +
         (size_t)2 * MAXSP * (g.B * g.B * g.B + 1) * 4 * 2;
}
static bool pair_shape(const Geom& g) {
  return g.B * g.r == PR && g.lgnb >= 1 && (g.B % 4) == 0 && pair_bytes(g) <= 48 * 1024;
}

bool kick_takes_phi(const pm_context* c) { return pair_shape(c->g); }

// All species of a compressed state: one brick kernel launch, then one re-sort. offs[s]: input
// cell offsets; perm[s] (device int64 [n], nullable): new stream position -> old stream
// position. P, V: the species' code widths.
template <int P, int V>
static pm_status kick_compressed_t(pm_context* c, const pm_species* in, pm_species* out,
                                   int n_sp, int64_t* const* offs, const float* acc,
                                   const float* amax, double ck, double cd,
                                   int64_t* const* perm, const float* const* app, bool phi) {
  const Geom& g = c->g;
  if (phi && !kick_takes_phi(c)) return PM_ERR_ARG;
  if (n_sp <= 0 || n_sp > MAXSP) return PM_ERR_ARG;
  const int B3 = g.B * g.B * g.B;
  // the species' scratch arrays start at multiples of 8 particles (16-byte digit loads)
  int64_t ntot = 0, nbase[MAXSP];
  for (int s = 0; s < n_sp; ++s) {
    nbase[s] = ntot;
    ntot += (in[s].n + 7) & ~(int64_t)7;
  }
  const size_t nn = (size_t)(ntot > 0 ? ntot : 1);
  const int64_t nbrick = g.nbrick;
  uint32_t* cnt = (uint32_t*)scratch(c, SC_CNT, (size_t)g.ncell3 * 4 * n_sp);
  int64_t* bstart = (int64_t*)scratch(c, SC_OFF2, (size_t)(nbrick + 1) * 8 * n_sp);
  uint32_t* astart = (uint32_t*)scratch(c, SC_ASTART, (size_t)(nbrick + 1) * 4 * n_sp);
  // Arrival counters in cache lines of their own: atomics on one line follow one another. 4096
  // bricks, 16.8 M particles of which few leave them: listing 131 -> 34 us; all leave: listing
  // 2580 -> 540, kick 2550 -> 930. 32768 bricks, all leave: kick 1425 -> 735. But a line for few
  // arrivals costs more than it spares (32768 bricks of 64 particles, all leave: listing 48 us
  // side by side, 83 with 16 words' distance): 4 MB of them from 256 particles a brick on, else
  // 256 KB.
  int64_t most = 0;
  for (int s = 0; s < n_sp; ++s) most = std::max(most, in[s].n);
  const int64_t awords = most >= 256 * nbrick ? APAD_MOST : APAD_LEAST;
  int apad = 0;
  while (apad < 5 && nbrick << (apad + 1) <= awords) ++apad;
  // what every call clears: the arrival counters, and per species the escapes' tiles and total
  // and the numbers of bricks that k_place leaves
  const int64_t ntile = cdiv(nbrick, ET);
  const int64_t nclear = n_sp * ((nbrick << apad) + ntile + 3);
  uint32_t* acnt = (uint32_t*)scratch(c, SC_ACNT, (size_t)nclear * 4);
  uint32_t* ecnt = (uint32_t*)scratch(c, SC_ECNT, (size_t)nbrick * n_sp * 4);
  char* tpos = (char*)scratch(c, SC_TPOS, nn * 3 * P);
  char* tvel = (char*)scratch(c, SC_TVEL, nn * 3 * V);
  uint16_t* tdig = (uint16_t*)scratch(c, SC_TDST, nn * 2);
  uint32_t* mkey = (uint32_t*)scratch(c, SC_KEYA, nn * 4);
  uint32_t* aidx = (uint32_t*)scratch(c, SC_VALA, nn * 4);
  uint32_t* abuf = (uint32_t*)scratch(c, SC_VALB, nn * 4);
  uint32_t* mcnt = (uint32_t*)scratch(c, SC_MCNT, (size_t)nbrick * 4 * n_sp);
  int32_t* part = (int32_t*)scratch(c, SC_KPART, (size_t)nbrick * 8 * n_sp);
  const int64_t nbs = cdiv(nbrick, BS_TILE);
  BrickSum* bsum = (BrickSum*)scratch(c, SC_BSUM, (size_t)nbs * n_sp * sizeof(BrickSum));
  if (!cnt || !bstart || !astart || !acnt || !ecnt || !tpos || !tvel || !tdig || !mkey ||
      !aidx || !abuf || !mcnt || !part || !bsum)
    return PM_ERR_NOMEM;
  uint32_t* etile = acnt + n_sp * (nbrick << apad);
  uint32_t* tot = etile + n_sp * ntile;
  PrepArgs R{};
  R.n_sp = n_sp;
  PlaceArgs Q{};
  Q.apad = apad;
  int64_t nmax = 0;
  KickArgs A{};
  A.n_sp = n_sp;
  A.acc = acc;
  A.scale = grad_scale(g.ng);
  A.apad = apad;
  A.ck = (float)ck;
  A.cdS = cd * g.SL * (P == 1 ? 1.0 : 256.0);
  for (int s = 0; s < n_sp; ++s) {
    KickSpecies& S = A.sp[s];
    S.n = in[s].n;
    S.pos = in[s].pos;
    S.vel = in[s].vel;
    S.hin = in[s].hdr;
    S.hout = out[s].hdr;
    S.off = offs[s];
    S.tpos = tpos + 3 * P * nbase[s];
    S.tvel = tvel + 3 * V * nbase[s];
    S.tdig = tdig + nbase[s];
    S.cnt = cnt + (int64_t)s * g.ncell3;
    S.mkey = mkey + nbase[s];
    S.mcnt = mcnt + (int64_t)s * g.nbrick;
    S.acnt = acnt + (s * nbrick << apad);
    S.pmn = part + (int64_t)2 * s * g.nbrick;
    S.pmx = S.pmn + g.nbrick;
    S.app = app ? app[s] : nullptr;
    R.hin[s] = in[s].hdr;
    R.hout[s] = out[s].hdr;
    R.n[s] = in[s].n;
    nmax = std::max(nmax, in[s].n);
    PlaceSpecies& L = Q.sp[s];
    L.n = S.n;
    L.off = S.off;
    L.tdig = S.tdig;
    L.mkey = S.mkey;
    L.tpos = S.tpos;
    L.tvel = S.tvel;
    L.cnt = S.cnt;
    L.mcnt = S.mcnt;
    L.acnt = S.acnt;
    L.pmn = S.pmn;
    L.pmx = S.pmx;
    L.bstart = bstart + s * (nbrick + 1);
    L.astart = astart + s * (nbrick + 1);
    L.aidx = aidx + nbase[s];
    L.abuf = abuf + nbase[s];
    L.ecnt = ecnt + s * nbrick;
    L.etile = etile + s * ntile;
    L.tot = tot + 3 * s;
    // beyond 8 times the mean a brick is the last one to be done (and one wave takes 20 us for
    // 2048 stayers)
    L.crowd = std::max<int64_t>(B3 >= 512 ? 16384 : 2048, 8 * in[s].n / nbrick);
    L.hout = out[s].hdr;
    L.pos = out[s].pos;
    L.vel = out[s].vel;
    L.count = out[s].count;
    L.esc = out[s].esc;
    L.cap_esc = out[s].cap_esc;
    L.perm = perm ? perm[s] : nullptr;
  }
  {
    hipLaunchKernelGGL(k_kick_prep<V>, dim3((unsigned)std::min<int64_t>(cdiv(nclear, KT), 1024)),
                       dim3(KT), 0, c->stream, R, amax, ck, acnt, nclear);
    ProfScope ps(c, ST_KICK);
    const int RN = g.B * g.r;
    const size_t tail = (size_t)MAXSP * (B3 + 1) * 4 * 2;
    const size_t pbytes = pair_bytes(g);
    const size_t fbytes = (size_t)3 * (RN + 1) * (RN + 1) * (RN + 1) * 4;
    if (phi)
      hipLaunchKernelGGL((k_kick_pair<256, 4, true, P, V>), dim3((unsigned)(g.nbrick / 2)),
                         dim3(256), (size_t)FX * FY * FZ * 4 + 2 * tail, c->stream, A, g, c->err);
    else if (pair_shape(g))
      hipLaunchKernelGGL((k_kick_pair<256, 4, false, P, V>), dim3((unsigned)(g.nbrick / 2)),
                         dim3(256), pbytes, c->stream, A, g, c->err);
    else if (RN == 16 && fbytes + tail <= 96 * 1024)
      hipLaunchKernelGGL((k_kick_brick<16, P, V>), dim3((unsigned)g.nbrick), dim3(KB),
                         fbytes + tail, c->stream, A, g, c->err);
    else if (RN == 8)
      hipLaunchKernelGGL((k_kick_brick<8, P, V>), dim3((unsigned)g.nbrick), dim3(KB),
                         fbytes + tail, c->stream, A, g, c->err);
    else
      hipLaunchKernelGGL((k_kick_brick<0, P, V>), dim3((unsigned)g.nbrick), dim3(KB), tail,
                         c->stream, A, g, c->err);
    PM_LAUNCH_CHECK();
  }
  ProfScope ps(c, ST_RESORT);
  const unsigned ny = (unsigned)n_sp;
  if (nbs > 1)
    hipLaunchKernelGGL(k_brick_sums, dim3((unsigned)nbs, ny), dim3(BS_T), 0, c->stream, Q, B3,
                       nbrick, bsum);
  hipLaunchKernelGGL(k_brick_scan, dim3((unsigned)nbs, ny), dim3(BS_T), 0, c->stream, Q, B3,
                     nbrick, (const BrickSum*)bsum);
  if (nmax > 0)
    hipLaunchKernelGGL(k_list_arrivals, dim3((unsigned)cdiv(nmax, KT * MV), ny), dim3(KT), 0,
                       c->stream, Q, 3 * g.lgB, nbrick, c->err);
  PM_LAUNCH_CHECK();
  // bits of an old stream index (the long lists' sort)
  const int ibits = nmax > 65536 ? 32 : 16;
  // bricks of 8^3 cells hold thousands of particles: four waves each
  if (B3 >= 512)
    hipLaunchKernelGGL((k_place<P, V, 4>), dim3((unsigned)nbrick, ny), dim3(256),
                       (size_t)4 * (ACAP + B3) * 4, c->stream, Q, B3, 3 * g.lgB, nbrick, c->err);
  else
    hipLaunchKernelGGL((k_place<P, V, 1>), dim3((unsigned)cdiv(nbrick, WB), ny), dim3(64 * WB),
                       (size_t)WB * (ACAP + ((B3 + 3) & ~3)) * 4, c->stream, Q, B3, 3 * g.lgB,
                       nbrick, c->err);
  const unsigned nrest = (unsigned)std::min<int64_t>(cdiv(nbrick, 4), 512);
  hipLaunchKernelGGL((k_place_rest<P, V>), dim3(nrest, ny), dim3(RT), (size_t)RW * LONG * 4,
                     c->stream, Q, B3, 3 * g.lgB, nbrick, ibits, c->err);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_kick_compressed_all(pm_context* c, const pm_species* in, pm_species* out,
                                  int n_sp, int64_t* const* offs, const float* acc,
                                  const float* amax, double ck, double cd,
                                  int64_t* const* perm, const float* const* app, bool phi) {
  if (n_sp <= 0 || n_sp > MAXSP) return PM_ERR_ARG;
  const int kind = common_width_kind(in, n_sp);
  if (kind < 0) return PM_ERR_ARG;
  return width_dispatch(kind, [&](auto P_, auto V_) {
    return kick_compressed_t<decltype(P_)::value, decltype(V_)::value>(
        c, in, out, n_sp, offs, acc, amax, ck, cd, perm, app, phi);
  });
}
