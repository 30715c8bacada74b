// Atomic environment vectors (forward) and their adjoint with the force
// scatter, one wavefront per atom.
//
// The paper names the ANI atom-centered symmetry functions as the operation
// its optimized kernels compute (Methods, "Optimization Through NNPOps"); the
// definition implemented is the published ANI one restated in nnp.h.  Forces
// are the negative gradient of the energy (Methods, "PyTorch Model Support").
//
// Per atom the wave first loads its neighbor records into LDS (displacement,
// distance, cutoff values, species).  Both sums of the forward pass are
// products with a one-hot matrix, which the FP32 MFMA computes exactly (its
// products are a term times 1 or 0): the radial row G[s][m] is
// onehot(species x neighbors) * terms(neighbors x 16 shifts), four neighbors
// per v_mfma_f32_16x16x4f32, and the angular rows G[block][a z] are
// onehot(blocks x pairs) * terms(pairs x 32), four neighbor pairs per pass.
// Each lane computes one term per product; there are no per-block loops or
// cross-lane reductions, and the accumulator layout is the feature layout,
// so the results are stored straight from registers.  The angle term uses
// the identity
// cos(theta - theta_z) = kappa c cos(theta_z) + sqrt(1 - kappa^2 c^2) sin(theta_z)
// for theta = acos(kappa c); (1 + cos)/2 raised to zeta is exp2(zeta log2(.)).
//
// The adjoint recomputes the same terms and contracts them with g = dE/dG
// (read from the network backward pass, only the blocks the atom touches).
// Its radial part is pulled from both sides of a pair, so only the angular
// neighbors are scattered to.
#include <type_traits>

#include "kernels.h"
#include "energy_sum.h"

namespace nnp {

// sin(pi t) and cos(pi t) for t in [0, 1] from Taylor polynomials of sin and
// cos on u = pi (t - 1/2) in [-pi/2, pi/2] (cos(pi t) = -sin u,
// sin(pi t) = cos u); the truncation error is below 1e-8, under FP32 rounding.
__device__ __forceinline__ void sincos_pi01(float t, float& s, float& c) {
  const float u = 3.14159265358979f * (t - 0.5f);
  const float u2 = u * u;
  // sin u = u (1 - u^2/3! + u^4/5! - ... - u^12/13!)
  float ps = -1.6059043836821614e-10f;               // -1/13!
  ps = ps * u2 + 2.5052108385441720e-8f;              //  1/11!
  ps = ps * u2 - 2.7557319223985893e-6f;              // -1/9!
  ps = ps * u2 + 1.9841269841269841e-4f;              //  1/7!
  ps = ps * u2 - 8.3333333333333333e-3f;              // -1/5!
  ps = ps * u2 + 1.6666666666666667e-1f;              //  1/3!
  const float sinu = u - u * u2 * ps;
  // cos u = 1 - u^2/2! + u^4/4! - ... + u^12/12!
  float pc = 2.0876756987868099e-9f;                 //  1/12!
  pc = pc * u2 - 2.7557319223985891e-7f;              // -1/10!
  pc = pc * u2 + 2.4801587301587302e-5f;              //  1/8!
  pc = pc * u2 - 1.3888888888888889e-3f;              // -1/6!
  pc = pc * u2 + 4.1666666666666667e-2f;              //  1/4!
  pc = pc * u2 - 0.5f;                                // -1/2!
  const float cosu = 1.f + u2 * pc;
  c = -sinu;
  s = cosu;
}

// fc(r; R) = cos(pi r / R)/2 + 1/2 and its derivative -(pi/2R) sin(pi r/R).
__device__ __forceinline__ float cutoff_val(float r, float inv_rc, float& dfc, float pi_2rc) {
  float s, c;
  sincos_pi01(fminf(r * inv_rc, 1.f), s, c);
  dfc = -pi_2rc * s;
  return 0.5f * c + 0.5f;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// Records read before the neighbor count is known: enough for a molecule's
// atoms (up to 16 neighbors) without fetching the whole 64-entry window.
constexpr int kSpecRec = 16;

// v_sqrt_f32 (about 1 ulp): neighbor distances and the angle sine are
// normal numbers, so the IEEE-exact expansion (denormal scaling and two
// correction steps) buys nothing here
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Unordered pair t of the list prefix [0, na) -> entries a < b, row-major:
// row r starts at pair r (2 na - r - 1) / 2.  The row is the floor of the
// smaller root of that quadratic; the float square root (exact operands for
// na <= 2048) can put it one row off either way near a row start, which one
// compare-and-select step in each direction corrects.  Branch-free, so the
// lanes of a pass never diverge.
__device__ __forceinline__ void decode_pair(int t, int na, int& a, int& b) {
  const float c2 = (float)(2 * na - 1);
  int r = (int)((c2 - fast_sqrt(fmaxf(c2 * c2 - 8.f * (float)t, 0.f))) * 0.5f);
  r = r < 0 ? 0 : (r > na - 2 ? na - 2 : r);
  r = (r * (2 * na - r - 1)) >> 1 > t ? r - 1 : r;
  const bool up = (r + 1 <= na - 2) & ((((r + 1) * (2 * na - r - 2)) >> 1) <= t);
  r = up ? r + 1 : r;
  a = r;
  b = t - ((r * (2 * na - r - 1)) >> 1) + r + 1;
}

__device__ __forceinline__ int pair_block(int p, int q, int S) {
  const int lo = p < q ? p : q, hi = p < q ? q : p;
  return lo * S - lo * (lo - 1) / 2 + (hi - lo);
}

// LDS per wave (forward): per neighbor float4 (dx, dy, dz, r), float2 (fc_rad,
// species bits) and fc_ang; a table of 64 angular pairs (eight angle-shift
// weights, four distance Gaussians and the block of each).  The feature row is
// accumulated in registers and stored block by block, so no LDS row is needed.
constexpr int kPairChunk = 64;
constexpr int kFwdBytesPerNbr = 16 + 8 + 4;
// (the block is a byte: lists of 128 entries then leave LDS for six waves per
// SIMD, an int for five: 80 -> 78 us on the 23,001-atom water box)
constexpr int kFwdPairBytes = 32 + 16 + 1;

typedef float aev_f32x4 __attribute__((ext_vector_type(4)));

// acc += A * B for one 16 x 16 x 4 FP32 MFMA: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16] and holds C[4 * (l / 16) + r][l % 16], r = 0..3.  The
// forward pass passes the terms as A and the one-hot as B, so C is the
// transposed feature block: lane l holds features 4 (l / 16) .. +3 of
// species (or block) l % 16, stored as one vector.
__device__ __forceinline__ aev_f32x4 mfma4(float a, float b, aev_f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}

// Four atoms per wave.  When the lists of a wave's four atoms, each rounded up
// to whole passes, fit 64 entries ("quad" waves), the per-neighbor setup
// (distances, cutoffs, species) runs for all four at once, one 16-lane group
// per atom, and the pairs of angular neighbors of all four share one table
// while they fit it; the radial and angular passes, which fill the wave with
// (neighbor, shift) and (pair, shift) lanes, run atom by atom.  Other waves
// take their atoms one at a time with all 64 lanes.  Either way a wave's LDS
// region holds max(64, capacity) neighbor entries.
//
// Quads pay off where lists are short and waves are many; elsewhere a wave
// per atom keeps four times as many waves in flight to hide the latency of the
// per-atom passes.  The host does not see the lists, but long ones take large
// molecules: more than 16,384 atoms in molecules of at most 160 in the mean take
// quads, the others (and boxes) one atom.  Measured (us, one atom / four atoms
// per wave).  Molecules of 64 atoms, 8 neighbors per atom: 1,024 atoms 5.5 / 13.1,
// 8,192: 10.1 / 15.0, 16,640: 18.4 / 17.0, 32,768: 27.6 / 22.9; of 10 to 150:
// 77,163: 52 / 47; of 150: 18,000: 18.3 / 21.7, 75,000: 51 / 47.  Molecules three
// times as dense, whose lists mostly miss the 64 entries: of 64: 16,640: 31 / 36,
// 32,768: 51 / 51; of 10 to 150: 77,163: 90 / 104; of 150: 75,000: 104 / 113.
// Drops of 300 atoms (35 neighbors): 17,400: 45 / 58, 78,000: 148 / 165; one of
// 23,001: 74 / 99.
constexpr int kQuadNbr = 16;   // lanes per atom of a quad wave
constexpr int kQuadAtoms = 16384, kQuadMolecule = 160;

__host__ __device__ constexpr int aev_region(int cap) { return cap > 64 ? cap : 64; }

struct FwdLds {
  float4* nd;   // displacement, distance
  float2* fs;   // radial cutoff value, species
  float* fa;    // angular cutoff value
  float* pw;    // [kPairChunk][8]
  float* pg;    // [kPairChunk][4]: distance shifts 0, 2, 1, 3
  unsigned char* pblk;  // [kPairChunk]: block, 255 past the last pair
};

// The angular pair t of the na angular neighbors at entry `base`, to table
// slot `slot`: the factors of its 32 terms, computed once instead of in each of
// the 16 lanes of its pass: the angle-shift weights
// w[z] = 2 ((1 + cos(theta - theta_z)) / 2)^zeta fc_j fc_k and the distance
// Gaussians g[a] = exp(-eta_A ((r_j + r_k) / 2 - R_a)^2); term (a, z) = w[z] g[a].
// Returns the pair's block; not `valid`: the same terms with block -1, whose
// one-hot row is zero.
__device__ __forceinline__ int pair_geometry(int t, int na, bool valid, const AevConst& C,
                                             const FwdLds& L, int base, int slot) {
  int a, b;
  decode_pair(t, na, a, b);
  a += base;
  b += base;
  const float4 vj = L.nd[a], vk = L.nd[b];
  const float cs = (vj.x * vk.x + vj.y * vk.y + vj.z * vk.z) * fast_rcp(vj.w * vk.w);
  const float kc = C.kappa * cs;
  const float sn = fast_sqrt(fmaxf(1.f - kc * kc, 0.f));
  const float dbar = 0.5f * (vj.w + vk.w);
  const float fcc = L.fa[a] * L.fa[b];
  float w[kNZ];
#pragma unroll
  for (int z = 0; z < kNZ; ++z) {
    const float base_ = 0.5f + 0.5f * (kc * C.cos_z[z] + sn * C.sin_z[z]);
    w[z] = 2.f * fast_exp2(C.zeta * fast_log2(base_)) * fcc;
  }
  float g[kNA];
#pragma unroll
  for (int q = 0; q < kNA; ++q) {
    const float u = dbar - C.shf_a[q];
    g[q] = fast_exp2(-C.eta_a_l2e * u * u);
  }
  reinterpret_cast<float4*>(L.pw)[2 * slot] = make_float4(w[0], w[1], w[2], w[3]);
  reinterpret_cast<float4*>(L.pw)[2 * slot + 1] = make_float4(w[4], w[5], w[6], w[7]);
  reinterpret_cast<float4*>(L.pg)[slot] = make_float4(g[0], g[2], g[1], g[3]);
  const int blk = valid ? pair_block(__float_as_int(L.fs[a].y), __float_as_int(L.fs[b].y), C.S) : -1;
  L.pblk[slot] = (unsigned char)blk;
  return blk;
}

// The k-steps (32 feature columns) holding a block an atom touches, from the
// elements among its neighbors (bits 0-7 of `seen`), among its angular
// neighbors (8-15), and those at least twice among these (16-23): the radial
// blocks of the first, the angular blocks of the pairs of the second (a pair
// (x, x) needs two).  Every other feature is zero, and the adjoint reads no
// dE/dG column outside them.  For four atoms at once, one per 16 lanes (`seen`
// the same in all of them): lane 7 of each group returns its atom's.
__device__ __forceinline__ unsigned long long row_ksteps(unsigned seen, const AevConst& C) {
  const int S = C.S, x = lane_id() & 15;
  const unsigned rp = seen & 255u, ap = (seen >> 8) & 255u, ad = (seen >> 16) & 255u;
  // lane x: element x's row of the angular triangle, blocks (x, x + k), which
  // starts at block x S - x (x - 1) / 2
  const unsigned row = (((ap >> x) & ~1u) | ((ad >> x) & 1u)) & ((1u << (S - x > 0 ? S - x : 0)) - 1u);
  const unsigned long long bm =
      (ap >> x) & 1u ? (unsigned long long)row << (x * S - ((x * (x - 1)) >> 1)) : 0ull;
  int lo = (int)(unsigned)bm, hi = (int)(unsigned)(bm >> 32);
  lo |= __builtin_amdgcn_update_dpp(0, lo, 0x111, 0xf, 0xf, true);
  hi |= __builtin_amdgcn_update_dpp(0, hi, 0x111, 0xf, 0xf, true);
  lo |= __builtin_amdgcn_update_dpp(0, lo, 0x112, 0xf, 0xf, true);
  hi |= __builtin_amdgcn_update_dpp(0, hi, 0x112, 0xf, 0xf, true);
  lo |= __builtin_amdgcn_update_dpp(0, lo, 0x114, 0xf, 0xf, true);
  hi |= __builtin_amdgcn_update_dpp(0, hi, 0x114, 0xf, 0xf, true);
  const unsigned long long all = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
  const unsigned r2 = rp | (rp >> 1);  // k-step j holds elements 2j and 2j + 1
  const int k0 = C.A0 >> 5;  // block p spans k-step k0 + p (and k0 + p + 1 unaligned)
  return (unsigned long long)((r2 & 1u) | ((r2 >> 1) & 2u) | ((r2 >> 2) & 4u) | ((r2 >> 3) & 8u)) |
         (all << k0) | ((C.A0 & 31) ? all << (k0 + 1) : 0ull);
}

// Bits of `seen` for angular-first entry e of a list of nr, na of them angular.
__device__ __forceinline__ unsigned seen_bits(int e, int nr, int na, const float2* fs) {
  if (e >= nr) return 0u;
  const int s = __float_as_int(fs[e].y);
  // (angular entries are grouped by species: a second one is the next one)
  const bool twice = e + 1 < na && __float_as_int(fs[e + 1].y) == s;
  return (1u << s) | (e < na ? 1u << (8 + s) : 0u) | (twice ? 1u << (16 + s) : 0u);
}

// NT: 16-block tiles of the angular one-hot (ceil(S (S + 1) / 2 / 16): one
// for up to five elements, two for six or seven, three for eight).
//
// Bound by vector instructions.  So the passes do little else than their
// terms: lists and pair tables are padded to whole passes with entries whose
// one-hot row is zero (no lane is switched off), table reads have constant
// offsets, which tiles a pass touches is read from two wave-wide masks, and
// the row's k-steps come from one bitwise or over the entries and are formed
// for four atoms at once.  Measured: 23,001-atom water box 99 -> 78 us (1,456
// -> 976 vector instructions per atom), 4,500 atoms in FP32 32 -> 27 us, the
// 32,768-atom batch 23.9 -> 21.9 us, 77,163 mixed atoms 50.5 -> 46.4 us, 1,645
// atoms (a wave per atom now) 14.6 -> 5.9 us.
template <typename OutT, int NT, int Q>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT < 3 && Q == 1 ? 8 : 7, 8))) void
k_aev_fwd(const int* __restrict__ dims, AevConst C, const float4* __restrict__ rec,
          const int2* __restrict__ counts, int cap, const int* __restrict__ row_of,
          OutT* __restrict__ out, int ld, unsigned long long* __restrict__ kmask, int sparse) {
  extern __shared__ float4 lds4[];
  const int n = dims[0];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = lane_id();
  const int i0 = ((int)blockIdx.x * 4 + w) * Q;  // the wave's first atom
  if (i0 >= n) return;
  const int reg = aev_region(cap);
  FwdLds L;
  L.nd = lds4 + (size_t)w * reg;
  float2* fs0 = reinterpret_cast<float2*>(lds4 + (size_t)4 * reg);
  L.fs = fs0 + (size_t)w * reg;
  float* fa0 = reinterpret_cast<float*>(fs0 + (size_t)4 * reg);
  L.fa = fa0 + (size_t)w * reg;
  float* pw0 = fa0 + (size_t)4 * reg;
  L.pw = pw0 + w * kPairChunk * kNZ;
  float* pg0 = pw0 + 4 * kPairChunk * kNZ;
  L.pg = pg0 + w * kPairChunk * kNA;
  L.pblk = reinterpret_cast<unsigned char*>(pg0 + 4 * kPairChunk * kNA) + w * kPairChunk;

  // entry `slot`; past the list (not `in`): a species no one-hot row has
  auto setup = [&](int slot, const float4 q, bool in, bool ang) __attribute__((always_inline)) {
    const float r = fast_sqrt(dist2(q.x, q.y, q.z));
    float dfr, dfa;
    const float fr = cutoff_val(r, C.inv_rc_r, dfr, C.pi_2rc_r);
    L.nd[slot] = make_float4(q.x, q.y, q.z, r);
    L.fs[slot] = make_float2(fr, in ? q.w : __int_as_float(-1));
    if (ang) L.fa[slot] = cutoff_val(r, C.inv_rc_a, dfa, C.pi_2rc_a);
  };

  // group g (lanes 16 g .. 16 g + 15) reads the counts and first 16 records
  // of atom i0 + g (one atom per wave: every group reads atom i0)
  const int g = Q > 1 ? lane >> 4 : 0, l = lane & 15;
  const int ig = i0 + g;
  const bool gin = ig < n;
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  const float4 q0 = Q > 1 && gin ? rec[(size_t)ig * cap + l] : zero4;
  const int2 cn = gin ? counts[ig] : make_int2(0, 0);
  const int row_g = gin && row_of ? row_of[ig] : ig;
  const int nr_g = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
  const int na_g = cn.y < 0 ? 0 : (cn.y > nr_g ? nr_g : cn.y);
  // atom a's first entry slot (lists rounded up to whole passes)
  int eb[Q + 1];
  eb[0] = 0;
#pragma unroll
  for (int a = 0; a < Q; ++a)
    eb[a + 1] = eb[a] + ((__builtin_amdgcn_readlane(nr_g, kQuadNbr * a) + 3) & ~3);
  const bool quad = Q > 1 && eb[Q] <= 64;
  const int eb_g = Q > 1 ? (g == 0 ? eb[0] : (g == 1 ? eb[1] : (g == 2 ? eb[2] : eb[3]))) : 0;
  // quad waves whose pairs, each atom's rounded up to whole passes, fit the
  // table: one table for all four (atom a's from slot tb_a on)
  int tb[Q + 1];
  tb[0] = 0;
#pragma unroll
  for (int a = 0; a < Q; ++a) {
    const int k = __builtin_amdgcn_readlane(na_g, kQuadNbr * a);
    tb[a + 1] = tb[a] + (((k * (k - 1)) / 2 + 3) & ~3);
  }
  const bool joint = quad && tb[Q] <= kPairChunk;
  unsigned long long kb_g = 0;                // quad: lane 16 g + 7, the atom's k-steps
  unsigned long long blo = 0, bhi = 0, b3 = 0;  // table slots with blocks 0-15, 16-31, 32-47
  if (quad) {
    const int nr4 = (nr_g + 3) & ~3;
    if (l < nr4) setup(eb_g + l, l < nr_g ? q0 : zero4, l < nr_g, l < na_g);
    for (int e = l + kQuadNbr; __ballot(e < nr4) != 0; e += kQuadNbr) {
      if (e < nr4) {
        const bool in = e < nr_g;
        setup(eb_g + e, in ? rec[(size_t)ig * cap + e] : zero4, in, e < na_g);
      }
    }
    wave_lds_sync();
    if (kmask) {
      // or over the group, in its last lane
      int v = 0;
      for (int e = l; __ballot(e < nr_g) != 0; e += kQuadNbr)
        v |= (int)seen_bits(e, nr_g, na_g, L.fs + eb_g);
      v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
      v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
      v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
      v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
      kb_g = row_ksteps((unsigned)__shfl(v, lane | 15, kWave), C);
      if (l == 7 && gin) kmask[row_g] = kb_g;
    }
    if (joint) {
      int blk = -1;
      if (lane < tb[Q]) {
        int b = 0, t = lane, na = __builtin_amdgcn_readlane(na_g, 0);
#pragma unroll
        for (int q = 1; q < Q; ++q) {
          const bool past = lane >= tb[q];
          b = past ? eb[q] : b;
          t = past ? lane - tb[q] : t;
          na = past ? __builtin_amdgcn_readlane(na_g, kQuadNbr * q) : na;
        }
        const int T = (na * (na - 1)) / 2;
        blk = pair_geometry(t < T ? t : T - 1, na, t < T, C, L, b, lane);
      }
      blo = __ballot((unsigned)blk < 16u);
      bhi = NT > 1 ? __ballot((unsigned)(blk - 16) < 16u) : 0;
      b3 = NT > 2 ? __ballot((unsigned)(blk - 32) < 16u) : 0;
      wave_lds_sync();
    }
  }
  const int S = C.S;
  const int l16 = lane & 15, kq = lane >> 4;
  const float Rm = C.lane_tab[l16];
  const int z = l16 & 7, ah = l16 >> 3;
  const int nblk = S * (S + 1) / 2;

#pragma unroll 1
  for (int a = 0; a < Q; ++a) {
    const int i = i0 + a;
    if (i >= n) break;  // wave-uniform
    const int nr = __builtin_amdgcn_readlane(nr_g, kQuadNbr * a);
    const int na = __builtin_amdgcn_readlane(na_g, kQuadNbr * a);
    int base = 0;
    if constexpr (Q > 1) base = a == 0 ? eb[0] : (a == 1 ? eb[1] : (a == 2 ? eb[2] : eb[3]));
    if (!quad) {
      // this atom alone: every lane sets up its neighbors in slots [0, nr)
      base = 0;
      wave_lds_sync();  // the previous atom's passes have read the region
      const float4* arec = rec + (size_t)i * cap;
      const int nr4 = (nr + 3) & ~3;  // (at most cap, a multiple of 16)
      for (int e = lane; e < nr4; e += kWave) {
        const bool in = e < nr;
        setup(e, in ? arec[e] : zero4, in, e < na);
      }
      wave_lds_sync();
      if (kmask) {
        unsigned v = 0;
        for (int e = lane; e < nr; e += kWave) v |= seen_bits(e, nr, na, L.fs);
        kb_g = row_ksteps(wave_or(v), C);  // (in every group)
        if (lane == 7) kmask[__builtin_amdgcn_readlane(row_g, kQuadNbr * a)] = kb_g;
      }
    }
    const int orow_i = __builtin_amdgcn_readlane(row_g, kQuadNbr * a);
    OutT* orow = out + (size_t)orow_i * ld;
    // this lane's stores: its radial block, and block l16 of each angular tile
    unsigned kb_r = ~0u, kb_a[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) kb_a[u] = ~0u;
    if (sparse) {  // (the angular blocks are whole k-steps then)
      const int at = quad ? kQuadNbr * a + 7 : 7;
      const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)kb_g, at);
      const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(kb_g >> 32), at);
      kb_r = lo;
#pragma unroll
      for (int u = 0; u < NT; ++u)
        kb_a[u] = (unsigned)((((unsigned long long)hi << 32) | lo) >> ((C.A0 >> 5) + 16 * u));
    }
    // ---- radial: G[s][m] = sum over neighbors e of [species(e) == s] * term(e, m)
    // as MFMA products of a one-hot (species x 4 neighbors) with the terms
    // (4 neighbors x 16 shifts); lane (kq, l16) computes neighbor kq, shift l16
    {
      aev_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      const float4* nde = L.nd + base + kq;
      const float2* fse = L.fs + base + kq;
      for (int e0 = 0; e0 < nr; e0 += 16) {
#pragma unroll
        for (int q = 0; q < 16; q += 4) {
          if (q == 0 || e0 + q < nr) {  // wave-uniform
            const float u = nde[q].w - Rm;
            const float2 f = fse[q];
            const float term = C.cR * fast_exp2(-C.eta_r_l2e * u * u) * f.x;
            acc = mfma4(term, __float_as_int(f.y) == l16 ? 1.f : 0.f, acc);
          }
        }
        nde += 16;
        fse += 16;
      }
      // (element slots from S up to the angular blocks are the gap: zero)
      if (l16 < (C.A0 >> 4) && ((kb_r >> (l16 >> 1)) & 1u))
        Store<OutT>::put4(orow + l16 * kNR + 4 * kq, make_float4(acc[0], acc[1], acc[2], acc[3]));
    }

    // ---- angular: G[blk][a z] = sum over unordered pairs of angular
    // neighbors of [block(pair) == blk] * term(pair, a, z), four pairs per
    // pass.  Lane (kq, l16) takes pair kq and column l16 of each of the two
    // 16-column halves: angle shift z = l16 % 8 and radial shifts a = l16 / 8
    // and l16 / 8 + 2.  Tile u of the one-hot covers blocks 16 u .. 16 u + 15;
    // its products run only on passes that hold one of its blocks (pairs come
    // in species order, so most passes touch one tile).
    {
      const int T = na * (na - 1) / 2;
      aev_f32x4 c0[NT], c1[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        c0[u] = aev_f32x4{0.f, 0.f, 0.f, 0.f};
        c1[u] = c0[u];
      }
      for (int p0 = 0; p0 < T; p0 += kPairChunk) {
        int sl = 0;
        const int tn = T - p0 < kPairChunk ? T - p0 : kPairChunk;
        unsigned long long m0, m1 = 0, m2 = 0;
        if (joint) {
          if constexpr (Q > 1) sl = a == 0 ? tb[0] : (a == 1 ? tb[1] : (a == 2 ? tb[2] : tb[3]));
          m0 = blo >> sl;
          if (NT > 1) m1 = bhi >> sl;
          if (NT > 2) m2 = b3 >> sl;
        } else {
          wave_lds_sync();  // the previous chunk's passes have read the table
          int blk = -1;
          if (lane < ((tn + 3) & ~3)) {
            const int t = p0 + lane;
            blk = pair_geometry(t < T ? t : T - 1, na, t < T, C, L, base, lane);
          }
          m0 = __ballot((unsigned)blk < 16u);
          if (NT > 1) m1 = __ballot((unsigned)(blk - 16) < 16u);
          if (NT > 2) m2 = __ballot((unsigned)(blk - 32) < 16u);
          wave_lds_sync();
        }
        const float* pwe = L.pw + (sl + kq) * kNZ + z;
        const float2* pge = reinterpret_cast<const float2*>(L.pg) + (sl + kq) * 2 + ah;
        const unsigned char* pbe = L.pblk + sl + kq;
        for (int t0 = 0; t0 < tn; t0 += 16) {
#pragma unroll
          for (int q = 0; q < 16; q += 4) {
            if (q == 0 || t0 + q < tn) {  // wave-uniform
              const float wz = pwe[q * kNZ];
              const float2 gz = pge[q * 2];
              const int blk = pbe[q];
              const float b0 = wz * gz.x, b1 = wz * gz.y;
              if (NT == 1 || ((m0 >> q) & 15ull)) {
                const float hot = blk == l16 ? 1.f : 0.f;
                c0[0] = mfma4(b0, hot, c0[0]);
                c1[0] = mfma4(b1, hot, c1[0]);
              }
              if constexpr (NT > 1) {
                if ((m1 >> q) & 15ull) {
                  const float hot = blk == l16 + 16 ? 1.f : 0.f;
                  c0[1] = mfma4(b0, hot, c0[1]);
                  c1[1] = mfma4(b1, hot, c1[1]);
                }
              }
              if constexpr (NT > 2) {
                if ((m2 >> q) & 15ull) {
                  const float hot = blk == l16 + 32 ? 1.f : 0.f;
                  c0[2] = mfma4(b0, hot, c0[2]);
                  c1[2] = mfma4(b1, hot, c1[2]);
                }
              }
            }
          }
          pwe += 16 * kNZ;
          pge += 32;
          pbe += 16;
          m0 >>= 16;
          m1 >>= 16;
          m2 >>= 16;
        }
      }
      // column c of c0[u] is feature c of block 16 u + l16 (a = c / 8 for the
      // low radial shifts, z = c % 8); c1[u] holds features 16 + c
      OutT* ang = orow + C.A0 + l16 * 32 + 4 * kq;
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        if (u > 0 && (kb_a[u] & 0xffffu) == 0) continue;  // wave-uniform: no block of this tile
        if (l16 + 16 * u < nblk && ((kb_a[u] >> l16) & 1u)) {
          Store<OutT>::put4(ang + 512 * u, make_float4(c0[u][0], c0[u][1], c0[u][2], c0[u][3]));
          Store<OutT>::put4(ang + 512 * u + 16,
                            make_float4(c1[u][0], c1[u][1], c1[u][2], c1[u][3]));
        }
      }
    }
    for (int c = C.A0 + nblk * 32 + lane; c < ld; c += kWave) Store<OutT>::put(orow + c, 0.f);
  }
}

// Atoms and waves per workgroup of the molecule adjoint.
constexpr int kMolBlock = 64;
constexpr int kMolWaves = 8;

// LDS per wave (deterministic adjoint): per neighbor float4 (dx, dy, dz, r),
// float4 (fc_rad, fc_ang, dfc_rad, dfc_ang), float4 accumulated
// dE/d(displacement), int species.
constexpr int kBwdBytesPerNbr = 16 + 16 + 16 + 4;

// Sixteen consecutive dE/dG values (one radial species block) as floats.
template <typename GT> struct Load16;
template <> struct Load16<float> {
  __device__ __forceinline__ static void get(const float* p, float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 u = reinterpret_cast<const float4*>(p)[q];
      v[4 * q] = u.x;
      v[4 * q + 1] = u.y;
      v[4 * q + 2] = u.z;
      v[4 * q + 3] = u.w;
    }
  }
};
template <> struct Load16<bf16_t> {
  __device__ __forceinline__ static void get(const bf16_t* p, float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint4 u = reinterpret_cast<const uint4*>(p)[q];
      const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[8 * q + 2 * k] = __uint_as_float(w[k] << 16);
        v[8 * q + 2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
      }
    }
  }
};

// The 32 dE/dG values of one angular pair block (four distance shifts x
// eight angle shifts, a-major), kept as loaded (BF16: two per register) and
// converted where used.
template <typename GT> struct Block32;
template <> struct Block32<float> {
  float v[32];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 u = reinterpret_cast<const float4*>(p)[q];
      v[4 * q] = u.x;
      v[4 * q + 1] = u.y;
      v[4 * q + 2] = u.z;
      v[4 * q + 3] = u.w;
    }
  }
  __device__ __forceinline__ float at(int k) const { return v[k]; }
};
template <> struct Block32<bf16_t> {
  unsigned w[16];
  __device__ __forceinline__ void load(const bf16_t* p) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 u = reinterpret_cast<const uint4*>(p)[q];
      w[4 * q] = u.x;
      w[4 * q + 1] = u.y;
      w[4 * q + 2] = u.z;
      w[4 * q + 3] = u.w;
    }
  }
  __device__ __forceinline__ float at(int k) const {
    return __uint_as_float((k & 1) ? (w[k >> 1] & 0xffff0000u) : (w[k >> 1] << 16));
  }
};

// One neighbor entry of the adjoint's LDS region: displacement and
// distance, cutoff values and derivatives, species.
__device__ __forceinline__ void adjoint_setup(int slot, const float4 q, bool ang,
                                              const AevConst& C, float4* nd, float4* nf,
                                              int* nsp) {
  const float r = fast_sqrt(dist2(q.x, q.y, q.z));
  float dfr, dfa = 0.f;
  const float fr = cutoff_val(r, C.inv_rc_r, dfr, C.pi_2rc_r);
  const float fa = ang ? cutoff_val(r, C.inv_rc_a, dfa, C.pi_2rc_a) : 0.f;
  nd[slot] = make_float4(q.x, q.y, q.z, r);
  nf[slot] = make_float4(fr, fa, dfr, dfa);
  nsp[slot] = species_of(q);
}

// The radial and angular passes of one atom (nr neighbors, the first na
// angular, set up in nd, nf, nsp): dE/d(displacement) of every neighbor entry
// into grad (the radial pass stores, the angular pass adds), in an order that
// depends on the atom's own list only (deterministic mode): eight lanes per
// angular pair (one per angle shift), eight pairs per pass, whose terms are
// added one pair after the other.
template <typename GT>
__device__ __forceinline__ void adjoint_passes_ordered(int nr, int na, const AevConst& C,
                                                       const GT* __restrict__ grow,
                                                       const float4* nd, const float4* nf,
                                                       float4* grad, const int* nsp) {
  const int lane = lane_id();
  const int S = C.S;
  // ---- radial: dE/dr_ij per neighbor, reduced over the 16 shift lanes
  {
    const int gq = lane >> 4, m = lane & 15;
    const float Rm = C.lane_tab[m];
    for (int e0 = 0; e0 < nr; e0 += 4) {
      const int e = e0 + gq;
      float contrib = 0.f;
      float4 v = make_float4(0.f, 0.f, 0.f, 1.f);
      if (e < nr) {
        v = nd[e];
        const float4 f = nf[e];
        const float u = v.w - Rm;
        const float ex = C.cR * fast_exp2(-C.eta_r_l2e * u * u);
        contrib = Store<GT>::get(grow + nsp[e] * kNR + m) * ex * (f.z - C.eta_r2 * u * f.x);
      }
      contrib = group16_sum(contrib);
      if (e < nr && m == 0) {
        const float sc = contrib * fast_rcp(v.w);
        grad[e] = make_float4(v.x * sc, v.y * sc, v.z * sc, 0.f);
      }
    }
  }
  wave_lds_sync();
  // ---- angular: lanes (t, z), eight unordered pairs per pass
  {
    const int tz = lane & 7, tg = lane >> 3;
    const float cz = C.lane_tab[kNR + tz], sz = C.lane_tab[kNR + kNZ + tz];
    const float ra0 = C.shf_a[0], ra1 = C.shf_a[1], ra2 = C.shf_a[2], ra3 = C.shf_a[3];
    const int T = na * (na - 1) / 2;
    const GT* gang = grow + C.A0 + tz;
    for (int t0 = 0; t0 < T; t0 += 8) {
      // lanes past the last pair recompute it and contribute zero: every lane
      // runs the same straight-line code, with no branch around the terms
      const int t = t0 + tg;
      const bool valid = t < T;
      int ej, ek;
      decode_pair(valid ? t : T - 1, na, ej, ek);
      const float4 vj = nd[ej], vk = nd[ek];
      const float4 cj = nf[ej], ck = nf[ek];
      const float fj = cj.y, fk = ck.y, dfj = cj.w, dfk = ck.w;
      const GT* gb = gang + pair_block(nsp[ej], nsp[ek], S) * 32;
      const float g0 = Store<GT>::get(gb), g1 = Store<GT>::get(gb + 8),
                  g2 = Store<GT>::get(gb + 16), g3 = Store<GT>::get(gb + 24);
      const float rj = fast_rcp(vj.w), rk = fast_rcp(vk.w);
      const float cs = (vj.x * vk.x + vj.y * vk.y + vj.z * vk.z) * (rj * rk);
      const float kc = C.kappa * cs;
      const float sn = fast_sqrt(fmaxf(1.f - kc * kc, 1e-12f));
      const float base_ = 0.5f + 0.5f * (kc * cz + sn * sz);
      const float pw = fast_exp2(C.zeta * fast_log2(base_));
      const float f1 = 2.f * pw;
      // d f1 / d c = zeta base^(zeta-1) d(kappa c cos_z + sqrt(1-kappa^2 c^2) sin_z)/dc
      const float df1 = C.zeta * pw * fast_rcp(base_) * (C.kappa * (cz - kc * sz * fast_rcp(sn)));
      const float dbar = 0.5f * (vj.w + vk.w);
      float u, e2, A0 = 0.f, A1 = 0.f;
      u = dbar - ra0; e2 = fast_exp2(-C.eta_a_l2e * u * u); A0 += g0 * e2; A1 -= g0 * u * e2;
      u = dbar - ra1; e2 = fast_exp2(-C.eta_a_l2e * u * u); A0 += g1 * e2; A1 -= g1 * u * e2;
      u = dbar - ra2; e2 = fast_exp2(-C.eta_a_l2e * u * u); A0 += g2 * e2; A1 -= g2 * u * e2;
      u = dbar - ra3; e2 = fast_exp2(-C.eta_a_l2e * u * u); A0 += g3 * e2; A1 -= g3 * u * e2;
      float X0 = valid ? f1 * A0 : 0.f;
      float X1 = valid ? f1 * A1 * C.eta_a : 0.f;
      float Xc = valid ? df1 * A0 : 0.f;
      X0 = group8_sum(X0);
      X1 = group8_sum(X1);
      Xc = group8_sum(Xc);
      if (valid && tz == 0) {
        const float fcc = fj * fk;
        const float dEdc = Xc * fcc;
        const float dEdj = X1 * fcc + X0 * dfj * fk;
        const float dEdk = X1 * fcc + X0 * fj * dfk;
        const float aj = (dEdj - dEdc * cs * rj) * rj;
        const float ak = (dEdk - dEdc * cs * rk) * rk;
        const float bb = dEdc * rj * rk;
        for (int q = 0; q < 8; ++q) {
          if (tg == q) {
            float4 a = grad[ej];
            a.x += aj * vj.x + bb * vk.x;
            a.y += aj * vj.y + bb * vk.y;
            a.z += aj * vj.z + bb * vk.z;
            grad[ej] = a;
            float4 b = grad[ek];
            b.x += ak * vk.x + bb * vj.x;
            b.y += ak * vk.y + bb * vj.y;
            b.z += ak * vk.z + bb * vj.z;
            grad[ek] = b;
          }
          wave_lds_sync();
        }
      }
    }
  }
  wave_lds_sync();
}

// One unordered pair of angular neighbors (j, k) of an atom, in one lane: the
// derivative of the pair's 32 terms, contracted with the pair block's dE/dG
// values gb.at(8 a + z), as dE/dv_j = aj v_j + bb v_k and dE/dv_k = ak v_k +
// bb v_j.  What the terms share (cosine, sine, the four distance Gaussians) is computed once;
// base^(zeta - 1) serves the value (times base) and the derivative, so an
// angle shift costs one logarithm and one exponential.
template <typename Blk>
__device__ __forceinline__ void adjoint_pair(const AevConst& C, const Blk& gb, const float4 vj,
                                             const float4 vk, float fj, float dfj, float fk,
                                             float dfk, float& aj, float& ak, float& bb) {
  const float rj = fast_rcp(vj.w), rk = fast_rcp(vk.w);
  const float cs = (vj.x * vk.x + vj.y * vk.y + vj.z * vk.z) * (rj * rk);
  const float kc = C.kappa * cs;
  const float sn = fast_sqrt(fmaxf(1.f - kc * kc, 1e-12f));
  const float kci = kc * fast_rcp(sn);
  const float dbar = 0.5f * (vj.w + vk.w);
  float e2[kNA], ue2[kNA];
#pragma unroll
  for (int a = 0; a < kNA; ++a) {
    const float u = dbar - C.shf_a[a];
    e2[a] = fast_exp2(-C.eta_a_l2e * u * u);
    ue2[a] = u * e2[a];
  }
  const float zm1 = C.zeta - 1.f;
  float X0 = 0.f, X1 = 0.f, Xc = 0.f;
#pragma unroll
  for (int z = 0; z < kNZ; ++z) {
    float A0 = 0.f, A1 = 0.f;
#pragma unroll
    for (int a = 0; a < kNA; ++a) {
      A0 += gb.at(a * kNZ + z) * e2[a];
      A1 += gb.at(a * kNZ + z) * ue2[a];
    }
    const float base_ = 0.5f + 0.5f * (kc * C.cos_z[z] + sn * C.sin_z[z]);
    const float q = fast_exp2(zm1 * fast_log2(base_));
    const float qa = q * A0;
    X0 += qa * base_;
    X1 += (q * base_) * A1;
    Xc += qa * (C.cos_z[z] - kci * C.sin_z[z]);
  }
  X0 *= 2.f;
  X1 *= -2.f * C.eta_a;
  Xc *= C.zeta * C.kappa;
  const float fcc = fj * fk;
  const float dEdc = Xc * fcc;
  const float dEdj = X1 * fcc + X0 * dfj * fk;
  const float dEdk = X1 * fcc + X0 * fj * dfk;
  aj = (dEdj - dEdc * cs * rj) * rj;
  ak = (dEdk - dEdc * cs * rk) * rk;
  bb = dEdc * rj * rk;
}

// dE/dG values of an angular pair block staged in LDS as floats.
struct BlockLds {
  const float* p;
  __device__ __forceinline__ float at(int k) const { return p[k]; }
};

constexpr int kAdjEnt = 64;        // angular entries in LDS
constexpr int kAdjPairs = 192;     // pairs whose results the LDS holds at a time
constexpr int kAdjBlk = 6;         // staged pair blocks: three elements among the neighbors
constexpr int kAdjBlkStride = 36;  // floats (neighboring blocks start four banks apart)

// LDS of one wave of the adjoint, one atom at a time.
struct AdjLds {
  float4 nd[kAdjEnt];              // displacement, distance
  float2 nf[kAdjEnt];              // angular cutoff value and derivative
  int nj[kAdjEnt];                 // neighbor atom
  int nsp[kAdjEnt];                // element, or its rank among the neighbors' elements
  float tab[3][kAdjPairs];         // pair results, then the entries' vectors
  float gb[kAdjBlk * kAdjBlkStride];
};

// The radial derivative of one neighbor entry at displacement v, pulled: the
// derivative of E_i and E_j with respect to their distance is one sum over
// the 16 shifts of (dE_i/dG_i[s_j] + dE_j/dG_j[s_i]) times the term's
// derivative, so an atom adds both to its own force and writes to no
// neighbor.  Lists are symmetric (the predicate sees the negated
// displacement, the same distance), so every pair comes up from both sides.
// That fails only in a call whose status has a bit of kStAsym (`cut`): j's list
// need not hold i then, nor need the network have written j's block of dE/dG,
// so dE_i's part alone is returned, for the caller to scatter, as without PULL.
// (The second block is i's own then, times zero: with a branch around its loads
// the 23,001-atom box took 1.7 us more a call, so 0.9.)
constexpr uint32_t kStAsym = kStCapacity | kStOffsets;
template <typename GT, bool PULL>
__device__ __forceinline__ float radial_pull(const AevConst& C, const GT* __restrict__ gi,
                                             const GT* __restrict__ gj, bool cut, float r) {
  float gv[16], gw[16];
  Load16<GT>::get(gi, gv);
  if constexpr (PULL) Load16<GT>::get(cut ? gi : gj, gw);
  const float pull = cut ? 0.f : 1.f;
  float dfr;
  const float fr = cutoff_val(r, C.inv_rc_r, dfr, C.pi_2rc_r);
  float acc = 0.f;
#pragma unroll
  for (int m = 0; m < kNR; ++m) {
    const float u = r - C.shf_r[m];
    const float gm = PULL ? __builtin_fmaf(gw[m], pull, gv[m]) : gv[m];
    acc += gm * fast_exp2(-C.eta_r_l2e * u * u) * (dfr - C.eta_r2 * u * fr);
  }
  return C.cR * acc * fast_rcp(r);
}

// The adjoint of one atom by one wave; put(j, c, x) adds x to component c of
// atom j.  (23,001-atom water box, BF16: 148 -> 74 us against scattering every
// entry and adding the pairs by lane scans and LDS atomics, 4,500 atoms in
// FP32 38 -> 24 us; it is bound by vector instructions, 1,380 per atom of which
// 88 transcendental: 61 us at four and sixteen clocks each.)
//
// Radial part: pulled, one lane per entry.  Angular part: one lane per
// unordered pair of angular neighbors.  A pair leaves three numbers in LDS
// (aj, ak and bb of adjoint_pair), which the lanes of the entries then
// collect, several lanes per entry.  (LDS atomics, at two clocks per lane,
// took three quarters of the time of a version that added the pairs' results
// with them.)  The pair blocks of dE/dG that the neighbors' elements select
// are staged in LDS.  Only angular entries are scattered, component by
// component in consecutive lanes: a global atomic addition costs by the
// 64-byte line it goes to (one lane per entry with three additions in turn
// costs three times as much).  The LDS holds 64 angular entries and 192
// pairs; further pairs come in turn, and an atom with more than 64 angular
// neighbors scatters every pair's results directly.
template <typename GT, bool PULL, typename Put>
__device__ __forceinline__ void adjoint_one(int i, int n, const AevConst& C, int si,
                                            const float4* __restrict__ rec,
                                            const int* __restrict__ nbr, int nr, int na, int cap,
                                            const int* __restrict__ row_of,
                                            const GT* __restrict__ grow, const GT* __restrict__ g,
                                            int ldg, float sign, bool cut, AdjLds& L, Put&& put) {
  const int lane = lane_id();
  const int S = C.S;
  const size_t at0 = (size_t)i * cap;
  const int pairs = (na * (na - 1)) >> 1;
  const bool fits = na <= kAdjEnt;
  const GT* gang = grow + C.A0;
  float cx = 0.f, cy = 0.f, cz = 0.f;  // the lane's part of the centre's sum
  unsigned elems = 0;                   // elements among the angular neighbors
  for (int e = lane; e < nr; e += kWave) {
    const float4 v = rec[at0 + e];
    const int j = clampi(nbr[at0 + e], n);
    const int sp = species_of(v);
    const float r = fast_sqrt(dist2(v.x, v.y, v.z));
    const float sc = radial_pull<GT, PULL>(
        C, grow + sp * kNR, PULL ? g + (size_t)row_of[j] * ldg + si * kNR : nullptr, cut, r);
    if (!PULL || cut) {
      put(j, 0, -sign * v.x * sc);
      put(j, 1, -sign * v.y * sc);
      put(j, 2, -sign * v.z * sc);
    }
    cx += v.x * sc;
    cy += v.y * sc;
    cz += v.z * sc;
    if (e < na && fits) {
      float dfa;
      const float fa = cutoff_val(r, C.inv_rc_a, dfa, C.pi_2rc_a);
      L.nd[e] = make_float4(v.x, v.y, v.z, r);
      L.nf[e] = make_float2(fa, dfa);
      L.nj[e] = j;
      L.nsp[e] = sp;
      elems = 1u << sp;  // (angular entries are in the first 64)
    }
  }
  if (fits && pairs > 0) {
    // the blocks of the neighbors' elements: slot of ranks (a, b >= a) is
    // pair_block(a, b, ne)
    elems = wave_or(elems);
    const int ne = __popc(elems), nb = (ne * (ne + 1)) >> 1;
    const bool staged = nb <= kAdjBlk;
    const int np = staged ? ne : S;
    if (staged) {
      if (lane < na) L.nsp[lane] = __popc(elems & ((1u << L.nsp[lane]) - 1u));
      constexpr int EP = 16 / sizeof(GT), VB = 32 / EP;  // elements per 16 bytes, pieces per block
      if (lane < nb * VB) {
        const int slot = lane / VB, piece = lane % VB;
        int a = 0;
        while (a + 1 < ne && slot >= ((a + 1) * (2 * ne - a)) >> 1) ++a;
        const int b = slot - ((a * (2 * ne - a + 1)) >> 1) + a;
        const int blk = pair_block(nth_bit(elems, a), nth_bit(elems, b), S);
        const uint4 u = *reinterpret_cast<const uint4*>(gang + blk * 32 + piece * EP);
        float* d = L.gb + slot * kAdjBlkStride + piece * EP;
        if constexpr (sizeof(GT) == 4) {
          *reinterpret_cast<uint4*>(d) = u;
        } else {
          const unsigned w[4] = {u.x, u.y, u.z, u.w};
          float f[8];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            f[2 * k] = __uint_as_float(w[k] << 16);
            f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
          }
          reinterpret_cast<float4*>(d)[0] = make_float4(f[0], f[1], f[2], f[3]);
          reinterpret_cast<float4*>(d)[1] = make_float4(f[4], f[5], f[6], f[7]);
        }
      }
    }
    wave_lds_sync();
    // this lane's entry when results are collected: entry e, every nsub-th
    // partner from sub on
    const int nsub = kWave / na;
    const int sub = (int)(((float)lane + 0.5f) * fast_rcp((float)na));
    const int e = lane - sub * na;
    float gx = 0.f, gy = 0.f, gz = 0.f, ga = 0.f;
    for (int c0 = 0; c0 < pairs; c0 += kAdjPairs) {
      const int cn = pairs - c0 < kAdjPairs ? pairs - c0 : kAdjPairs;
      for (int k = lane; k < cn; k += kWave) {
        int ej, ek;
        decode_pair(c0 + k, na, ej, ek);
        const int blk = pair_block(L.nsp[ej], L.nsp[ek], np);
        const float2 cj = L.nf[ej], ck = L.nf[ek];
        float aj, ak, bb;
        if (staged) {
          const BlockLds gb{L.gb + blk * kAdjBlkStride};
          adjoint_pair(C, gb, L.nd[ej], L.nd[ek], cj.x, cj.y, ck.x, ck.y, aj, ak, bb);
        } else {
          Block32<GT> gb;
          gb.load(gang + blk * 32);
          adjoint_pair(C, gb, L.nd[ej], L.nd[ek], cj.x, cj.y, ck.x, ck.y, aj, ak, bb);
        }
        L.tab[0][k] = aj;
        L.tab[1][k] = ak;
        L.tab[2][k] = bb;
      }
      wave_lds_sync();
      if (sub < nsub) {
        for (int p = sub; p < na; p += nsub) {
          const int lo = p < e ? p : e, hi = p < e ? e : p;
          const int t = ((lo * (2 * na - lo - 1)) >> 1) + hi - lo - 1 - c0;
          if (p != e && t >= 0 && t < cn) {
            const float4 v = L.nd[p];
            const float bb = L.tab[2][t];
            ga += L.tab[p < e ? 1 : 0][t];
            gx += bb * v.x;
            gy += bb * v.y;
            gz += bb * v.z;
          }
        }
      }
      wave_lds_sync();
    }
    // the entry's sum over its lanes, and the scatter
    for (int s = 1; s < nsub; ++s) {
      const int from = e + s * na;
      const float ox = __shfl(gx, from, kWave), oy = __shfl(gy, from, kWave),
                  oz = __shfl(gz, from, kWave), oa = __shfl(ga, from, kWave);
      if (sub == 0) {
        gx += ox;
        gy += oy;
        gz += oz;
        ga += oa;
      }
    }
    if (lane < na) {
      const float4 v = L.nd[lane];
      gx += ga * v.x;
      gy += ga * v.y;
      gz += ga * v.z;
      L.tab[0][lane] = gx;
      L.tab[1][lane] = gy;
      L.tab[2][lane] = gz;
      cx += gx;
      cy += gy;
      cz += gz;
    }
    wave_lds_sync();
    for (int t = lane; t < 3 * na; t += kWave) {
      const int q = (t * 21846) >> 16, c = t - 3 * q;  // t / 3
      put(L.nj[q], c, -sign * L.tab[c][q]);
    }
  } else if (!fits) {
    for (int t = lane; t < pairs; t += kWave) {
      int ej, ek;
      decode_pair(t, na, ej, ek);
      float4 vj = rec[at0 + ej], vk = rec[at0 + ek];
      Block32<GT> gb;
      gb.load(gang + pair_block(species_of(vj), species_of(vk), S) * 32);
      vj.w = fast_sqrt(dist2(vj.x, vj.y, vj.z));
      vk.w = fast_sqrt(dist2(vk.x, vk.y, vk.z));
      float dj, dk;
      const float fj = cutoff_val(vj.w, C.inv_rc_a, dj, C.pi_2rc_a);
      const float fk = cutoff_val(vk.w, C.inv_rc_a, dk, C.pi_2rc_a);
      float aj, ak, bb;
      adjoint_pair(C, gb, vj, vk, fj, dj, fk, dk, aj, ak, bb);
      const float gj[3] = {aj * vj.x + bb * vk.x, aj * vj.y + bb * vk.y, aj * vj.z + bb * vk.z};
      const float gk[3] = {ak * vk.x + bb * vj.x, ak * vk.y + bb * vj.y, ak * vk.z + bb * vj.z};
      const int jj = clampi(nbr[at0 + ej], n), jk = clampi(nbr[at0 + ek], n);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        put(jj, c, -sign * gj[c]);
        put(jk, c, -sign * gk[c]);
      }
      cx += gj[0] + gk[0];
      cy += gj[1] + gk[1];
      cz += gj[2] + gk[2];
    }
  }
  cx = wave_sum_rows(cx);
  cy = wave_sum_rows(cy);
  cz = wave_sum_rows(cz);
  if (lane < 3) put(i, lane, sign * (lane == 0 ? cx : (lane == 1 ? cy : cz)));
}

// The adjoint of atoms i0 .. i0 + 4 H - 1 by one wave, for short lists
// (molecules): lane (g, l) of H rounds takes entries l, l + 16, ... of atom
// i0 + 4 h + g, so the atom's sums are sums over 16 lanes; the pairs of
// angular neighbors of all atoms form one list, one lane per pair, whose
// results go through LDS as in adjoint_one.  Needs at most 16 angular
// neighbors per atom; returns false (nothing done) otherwise.  (32,768-atom
// batch 18.8 -> 15.6 us, 77,163 atoms of mixed molecules 73.5 -> 40.4 us against
// eight lanes per pair, lists of at most 16 entries and LDS atomics: mixed
// molecules have longer lists now and then, which took the slow path.)
template <int H>
struct QuadLds {
  float4 nd[64 * H];
  float2 nf[64 * H];
  int nsp[64 * H];
  float tab[3][kAdjPairs];
};

template <typename GT, int H, bool PULL, typename Put>
__device__ __forceinline__ bool adjoint_quads(int i0, int n, const AevConst& C,
                                              const float4* __restrict__ xyzs,
                                              const float4* __restrict__ rec,
                                              const int* __restrict__ nbr,
                                              const int2* __restrict__ counts, int cap,
                                              const int* __restrict__ row_of,
                                              const GT* __restrict__ g, int ldg, float sign,
                                              QuadLds<H>& L, Put&& put) {
  constexpr int Q = 4 * H;
  const int lane = lane_id();
  const int S = C.S;
  const int gq = lane >> 4, l = lane & 15;
  int nr[H], na[H], row[H], si[H], jn[H];
  float4 v0[H];
  bool wide = false;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int i = i0 + 4 * h + gq;
    const bool in = i < n;
    const int2 cn = in ? counts[i] : make_int2(0, 0);
    v0[h] = in ? rec[(size_t)i * cap + l] : make_float4(0.f, 0.f, 0.f, 0.f);
    jn[h] = in ? nbr[(size_t)i * cap + l] : 0;
    row[h] = in ? row_of[i] : 0;
    si[h] = in ? species_of(xyzs[i]) : 0;
    nr[h] = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
    na[h] = cn.y < 0 ? 0 : (cn.y > nr[h] ? nr[h] : cn.y);
    wide |= na[h] > kQuadNbr;
  }
  if (__ballot(wide)) return false;
  float cen[H][3];
  float gx[H], gy[H], gz[H], ga[H];  // the lane's angular entry
#pragma unroll
  for (int h = 0; h < H; ++h) gx[h] = gy[h] = gz[h] = ga[h] = 0.f;
  int P[Q + 1];  // the atoms' first pairs in the list (uniform)
  P[0] = 0;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    cen[h][0] = cen[h][1] = cen[h][2] = 0.f;
    const size_t at = (size_t)(i0 + 4 * h + gq) * cap;
    for (int e = l; __ballot(e < nr[h]) != 0; e += kQuadNbr) {
      if (e < nr[h]) {
        const bool first = e < kQuadNbr;
        const float4 v = first ? v0[h] : rec[at + e];
        const int j = clampi(first ? jn[h] : nbr[at + e], n);
        const int sp = species_of(v);
        const float r = fast_sqrt(dist2(v.x, v.y, v.z));
        const float sc = radial_pull<GT, PULL>(
            C, g + (size_t)row[h] * ldg + sp * kNR,
            PULL ? g + (size_t)row_of[j] * ldg + si[h] * kNR : nullptr, false, r);
        if (!PULL) {
          if (e < na[h]) {  // (with the angular part)
            gx[h] = v.x * sc;
            gy[h] = v.y * sc;
            gz[h] = v.z * sc;
          } else {
            put(j, 0, -sign * v.x * sc);
            put(j, 1, -sign * v.y * sc);
            put(j, 2, -sign * v.z * sc);
          }
        }
        if (PULL || e >= na[h]) {
          cen[h][0] += v.x * sc;
          cen[h][1] += v.y * sc;
          cen[h][2] += v.z * sc;
        }
        if (e < na[h]) {
          float dfa;
          const float fa = cutoff_val(r, C.inv_rc_a, dfa, C.pi_2rc_a);
          const int slot = 64 * h + lane;
          L.nd[slot] = make_float4(v.x, v.y, v.z, r);
          L.nf[slot] = make_float2(fa, dfa);
          L.nsp[slot] = sp;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = __builtin_amdgcn_readlane(na[h], 16 * q);
      P[4 * h + q + 1] = P[4 * h + q] + ((k * (k - 1)) >> 1);
    }
  }
  wave_lds_sync();
  const int pairs = P[Q];
  for (int c0 = 0; c0 < pairs; c0 += kAdjPairs) {
    const int cn = pairs - c0 < kAdjPairs ? pairs - c0 : kAdjPairs;
    for (int k = lane; k < cn; k += kWave) {
      const int idx = c0 + k;
      int a = 0, start = 0, ka = __builtin_amdgcn_readlane(na[0], 0),
          ra = __builtin_amdgcn_readlane(row[0], 0);
#pragma unroll
      for (int q = 1; q < Q; ++q) {
        const bool past = idx >= P[q];
        a = past ? q : a;
        start = past ? P[q] : start;
        ka = past ? __builtin_amdgcn_readlane(na[q >> 2], 16 * (q & 3)) : ka;
        ra = past ? __builtin_amdgcn_readlane(row[q >> 2], 16 * (q & 3)) : ra;
      }
      int ej, ek;
      decode_pair(idx - start, ka, ej, ek);
      ej += kQuadNbr * a;
      ek += kQuadNbr * a;
      Block32<GT> gb;
      gb.load(g + (size_t)ra * ldg + C.A0 + pair_block(L.nsp[ej], L.nsp[ek], S) * 32);
      const float2 cj = L.nf[ej], ck = L.nf[ek];
      float aj, ak, bb;
      adjoint_pair(C, gb, L.nd[ej], L.nd[ek], cj.x, cj.y, ck.x, ck.y, aj, ak, bb);
      L.tab[0][k] = aj;
      L.tab[1][k] = ak;
      L.tab[2][k] = bb;
    }
    wave_lds_sync();
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int base = 64 * h + 16 * gq;
      const int t0 = (gq == 0 ? P[4 * h] : (gq == 1 ? P[4 * h + 1]
                                                    : (gq == 2 ? P[4 * h + 2] : P[4 * h + 3]))) - c0;
      if (l < na[h]) {
        for (int p = 0; p < na[h]; ++p) {
          const int lo = p < l ? p : l, hi = p < l ? l : p;
          const int t = ((lo * (2 * na[h] - lo - 1)) >> 1) + hi - lo - 1 + t0;
          if (p != l && t >= 0 && t < cn) {
            const float4 v = L.nd[base + p];
            const float bb = L.tab[2][t];
            ga[h] += L.tab[p < l ? 1 : 0][t];
            gx[h] += bb * v.x;
            gy[h] += bb * v.y;
            gz[h] += bb * v.z;
          }
        }
      }
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (l < na[h]) {
      gx[h] += ga[h] * v0[h].x;
      gy[h] += ga[h] * v0[h].y;
      gz[h] += ga[h] * v0[h].z;
      const int j = clampi(jn[h], n);
      put(j, 0, -sign * gx[h]);
      put(j, 1, -sign * gy[h]);
      put(j, 2, -sign * gz[h]);
    }
    const float x = group16_sum(cen[h][0] + gx[h]), y = group16_sum(cen[h][1] + gy[h]),
                z = group16_sum(cen[h][2] + gz[h]);
    const int i = i0 + 4 * h + gq;
    if (i < n && l < 3) put(i, l, sign * (l == 0 ? x : (l == 1 ? y : z)));
  }
  return true;
}

// Adjoint: g (rows of type GT, stride ldg) -> added into out (float32 [n][3]).
// sign = +1 writes forces (-dE/dr); sign = -1 writes the gradient dE/dr.
// With gidx, atom i's force goes to row gidx[i] of out ([n_total][3]; rows
// outside [0, n_total) are skipped; staging reports them).  Blocks from
// nb_adj on sum the molecular energies (one block per molecule), which need
// only the atomic energies of the forward pass: they fill the tail of the
// scatter instead of a launch of their own.
template <typename GT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_aev_bwd(
    const int* __restrict__ dims, AevConst C, const float4* __restrict__ xyzs,
    const float4* __restrict__ rec, const int* __restrict__ nbr, const int2* __restrict__ counts,
    int cap, const int* __restrict__ row_of, const GT* __restrict__ g, int ldg,
    float* __restrict__ out, float sign, const int* __restrict__ gidx, int n_total,
    const uint32_t* __restrict__ status, int nb_adj, EnergyArgs EA) {
  __shared__ AdjLds lds[4];
  if ((int)blockIdx.x >= nb_adj) {  // block-uniform: the molecular energy sums
    energy_block((int)blockIdx.x - nb_adj, dims, EA);
    return;
  }
  const int n = dims[0];
  const bool cut = (*status & kStAsym) != 0;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i = (int)blockIdx.x * 4 + w;
  if (i >= n) return;
  const int2 cn = counts[i];
  const int nr = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
  const int na = cn.y < 0 ? 0 : (cn.y > nr ? nr : cn.y);
  adjoint_one<GT, true>(i, n, C, species_of(xyzs[i]), rec, nbr, nr, na, cap, row_of,
                        g + (size_t)row_of[i] * ldg, g, ldg, sign, cut, lds[w],
                        [&](int j, int c, float x) {
                          if (gidx) {
                            j = gidx[j];
                            if (j < 0 || j >= n_total) return;
                          }
                          unsafeAtomicAdd(out + 3 * (size_t)j + c, x);
                        });
}

// Small systems (few waves, so the chain of dependent loads is the time): four
// atoms per wave on short lists, every entry scattered to global memory
// (pulling the radial part would put two more loads in the chain).  1,645
// atoms: 28.7 -> 9.0 us, 24 atoms in FP32: 11.5 -> 5.6 us, against 64-atom
// workgroups with windows.
template <typename GT>
__global__ __launch_bounds__(256) void k_aev_bwd_small(
    const int* __restrict__ dims, AevConst C, const float4* __restrict__ xyzs,
    const float4* __restrict__ rec, const int* __restrict__ nbr, const int2* __restrict__ counts,
    int cap, const int* __restrict__ row_of, const GT* __restrict__ g, int ldg,
    float* __restrict__ out, float sign, const int* __restrict__ gidx, int n_total,
    const uint32_t* __restrict__, int nb_adj, EnergyArgs EA) {
  __shared__ union {
    QuadLds<1> quad;
    AdjLds one;
  } lds[4];
  if ((int)blockIdx.x >= nb_adj) {  // block-uniform: the molecular energy sums
    energy_block((int)blockIdx.x - nb_adj, dims, EA);
    return;
  }
  const int n = dims[0];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i0 = ((int)blockIdx.x * 4 + w) * 4;
  if (i0 >= n) return;
  auto put = [&](int j, int c, float x) {
    if (gidx) {
      j = gidx[j];
      if (j < 0 || j >= n_total) return;
    }
    unsafeAtomicAdd(out + 3 * (size_t)j + c, x);
  };
  if (adjoint_quads<GT, 1, false>(i0, n, C, xyzs, rec, nbr, counts, cap, row_of, g, ldg, sign,
                                  lds[w].quad, put))
    return;
  for (int a = 0; a < 4 && i0 + a < n; ++a) {
    const int i = i0 + a;
    const int2 cn = counts[i];
    const int nr = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
    const int na = cn.y < 0 ? 0 : (cn.y > nr ? nr : cn.y);
    adjoint_one<GT, false>(i, n, C, 0, rec, nbr, nr, na, cap, row_of,
                           g + (size_t)row_of[i] * ldg, g, ldg, sign, false, lds[w].one, put);
    wave_lds_sync();  // the next atom reuses the LDS
  }
}

// Deterministic adjoint (gather mode): one atom per wave, as above, but the
// atom's dE/d(displacement) of every neighbor entry goes to pgrad[i * cap +
// e] instead of being scattered; a gather forms the forces from these rows
// (neighbors.hip).  Blocks from nb_adj on sum the molecular energies.
template <typename GT>
__global__ __launch_bounds__(256) void k_aev_bwd_det(const int* __restrict__ dims, AevConst C,
                                                     const float4* __restrict__ rec,
                                                     const int2* __restrict__ counts, int cap,
                                                     const int* __restrict__ row_of,
                                                     const GT* __restrict__ g, int ldg,
                                                     float4* __restrict__ pgrad, int nb_adj,
                                                     EnergyArgs EA) {
  extern __shared__ float4 lds4[];
  if ((int)blockIdx.x >= nb_adj) {  // block-uniform: the molecular energy sums
    energy_block((int)blockIdx.x - nb_adj, dims, EA);
    return;
  }
  const int n = dims[0];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i = (int)blockIdx.x * 4 + w;
  if (i >= n) return;
  const int lane = lane_id();
  const int reg = aev_region(cap);
  float4* nd = lds4 + (size_t)w * reg * 3;
  float4* nf = nd + reg;
  float4* grad = nd + 2 * reg;
  int* nsp = reinterpret_cast<int*>(lds4 + (size_t)4 * reg * 3) + w * reg;
  const int2 cn = counts[i];
  const int nr = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
  const int na = cn.y < 0 ? 0 : (cn.y > nr ? nr : cn.y);
  const float4* arec = rec + (size_t)i * cap;
  for (int e = lane; e < nr; e += kWave) adjoint_setup(e, arec[e], e < na, C, nd, nf, nsp);
  wave_lds_sync();
  adjoint_passes_ordered<GT>(nr, na, C, g + (size_t)row_of[i] * ldg, nd, nf, grad, nsp);
  for (int e = lane; e < nr; e += kWave) pgrad[(size_t)i * cap + e] = grad[e];
}

// Molecules (no box, no index map): a workgroup owns the kMolBlock atoms
// [b * kMolBlock, (b + 1) * kMolBlock), eight per wave, and
// adds every force into an LDS window over the atoms [b - 1, b + 2) *
// kMolBlock, which holds all neighbors of its atoms for molecules of up to
// kMolBlock + 1 atoms (neighbors outside it, in larger molecules, are added
// to global memory directly).  At the end each touched window atom is written
// once: with a plain store if its whole molecule lies inside the workgroup's
// atoms (nothing else adds to it; staging zeroed the output), else with one
// atomic add per component.  This replaces the contended per-entry global
// atomics of the per-atom kernel (about nine adds per atom on the same lines).
template <typename GT>
__global__ __launch_bounds__(64 * kMolWaves) __attribute__((amdgpu_waves_per_eu(4, 8))) void
k_aev_bwd_mol(const int* __restrict__ dims, AevConst C, const float4* __restrict__ xyzs,
              const float4* __restrict__ rec, const int* __restrict__ nbr,
              const int2* __restrict__ counts, int cap, const int* __restrict__ row_of,
              const GT* __restrict__ g, int ldg, float* __restrict__ out, float sign,
              const int2* __restrict__ mrange, const uint32_t* __restrict__ status, int nb_adj,
              EnergyArgs EA) {
  constexpr int kWin = 3 * kMolBlock;
  __shared__ union {
    QuadLds<2> quad;
    AdjLds one;
  } lds[kMolWaves];
  __shared__ float win[3 * kWin];
  if ((int)blockIdx.x >= nb_adj) {  // block-uniform: the molecular energy sums
    energy_block((int)blockIdx.x - nb_adj, dims, EA);
    return;
  }
  const int n = dims[0];
  const bool cut = (*status & kStAsym) != 0;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int base = (int)blockIdx.x * kMolBlock, w0 = base - kMolBlock;
  for (int t = threadIdx.x; t < 3 * kWin; t += blockDim.x) win[t] = 0.f;
  __syncthreads();
  auto put = [&](int j, int c, float x) {
    const int t = j - w0;
    if (t >= 0 && t < kWin)
      atomicAdd(win + 3 * t + c, x);
    else
      unsafeAtomicAdd(out + 3 * (size_t)j + c, x);
  };
  static_assert(kMolBlock == 8 * kMolWaves, "eight atoms per wave");
  const int i0 = base + 8 * w;
  auto one_by_one = [&](auto pull) __attribute__((always_inline)) {
    for (int a = 0; a < 8 && i0 + a < n; ++a) {
      const int i = i0 + a;
      const int2 cn = counts[i];
      const int nr = cn.x < 0 ? 0 : (cn.x > cap ? cap : cn.x);
      const int na = cn.y < 0 ? 0 : (cn.y > nr ? nr : cn.y);
      adjoint_one<GT, pull.value>(i, n, C, species_of(xyzs[i]), rec, nbr, nr, na, cap, row_of,
                                  g + (size_t)row_of[i] * ldg, g, ldg, sign, false, lds[w].one,
                                  put);
      wave_lds_sync();  // the next atom reuses the LDS
    }
  };
  if (__builtin_expect(cut, 0))
    one_by_one(std::false_type{});
  else if (i0 < n && !adjoint_quads<GT, 2, true>(i0, n, C, xyzs, rec, nbr, counts, cap, row_of, g,
                                                 ldg, sign, lds[w].quad, put))
    one_by_one(std::true_type{});
  __syncthreads();
  for (int t = threadIdx.x; t < kWin; t += blockDim.x) {
    const int j = w0 + t;
    if (j < 0 || j >= n) continue;
    const float x = win[3 * t], y = win[3 * t + 1], z = win[3 * t + 2];
    if (x == 0.f && y == 0.f && z == 0.f) continue;
    const int2 mr = mrange[j];
    if (mr.x >= base && mr.y <= base + kMolBlock) {
      out[3 * j] = x;
      out[3 * j + 1] = y;
      out[3 * j + 2] = z;
    } else {
      unsafeAtomicAdd(out + 3 * j, x);
      unsafeAtomicAdd(out + 3 * j + 1, y);
      unsafeAtomicAdd(out + 3 * j + 2, z);
    }
  }
}

// ----------------------------------------------------------------- launchers

template <typename OutT, int Q>
static void launch_aev_fwd_q(const int* dims, int n_cap, const AevConst& C, const float4* rec,
                             const int2* counts, int cap, const int* row_of, OutT* out, int ld,
                             unsigned long long* kmask, bool sparse, hipStream_t st) {
  const size_t lds = (size_t)4 * aev_region(cap) * kFwdBytesPerNbr +
                     (size_t)4 * kPairChunk * kFwdPairBytes;
  static const bool attr = (ensure_lds(k_aev_fwd<OutT, 1, Q>), ensure_lds(k_aev_fwd<OutT, 2, Q>),
                            ensure_lds(k_aev_fwd<OutT, 3, Q>), true);
  (void)attr;
  const int nblk = C.S * (C.S + 1) / 2;
  auto kern = nblk <= 16 ? k_aev_fwd<OutT, 1, Q>
                         : (nblk <= 32 ? k_aev_fwd<OutT, 2, Q> : k_aev_fwd<OutT, 3, Q>);
  const int per_block = 4 * Q;
  hipLaunchKernelGGL(kern, dim3((n_cap + per_block - 1) / per_block), dim3(256), lds, st, dims, C,
                     rec, counts, cap, row_of, out, ld, kmask, sparse ? 1 : 0);
}

template <typename OutT>
void launch_aev_fwd(const int* dims, int n_cap, int nmol_cap, const AevConst& C,
                    const float4* rec, const int2* counts, int cap, const int* row_of, OutT* out,
                    int ld, bool det, unsigned long long* kmask, bool sparse, hipStream_t st) {
  if (n_cap <= 0) return;
  const bool quads = n_cap > kQuadAtoms && n_cap / kQuadMolecule <= nmol_cap;
  sparse = sparse && kmask && ld <= 64 * 32;
  if (quads && !det)
    launch_aev_fwd_q<OutT, 4>(dims, n_cap, C, rec, counts, cap, row_of, out, ld, kmask, sparse,
                              st);
  else
    launch_aev_fwd_q<OutT, 1>(dims, n_cap, C, rec, counts, cap, row_of, out, ld, kmask, sparse,
                              st);
}
template void launch_aev_fwd<float>(const int*, int, int, const AevConst&, const float4*,
                                    const int2*, int, const int*, float*, int, bool,
                                    unsigned long long*, bool, hipStream_t);
template void launch_aev_fwd<bf16_t>(const int*, int, int, const AevConst&, const float4*,
                                     const int2*, int, const int*, bf16_t*, int, bool,
                                     unsigned long long*, bool, hipStream_t);

template <typename GT>
void launch_aev_bwd(const int* dims, int n_cap, const AevConst& C, const float4* xyzs,
                    const float4* rec, const int* nbr, const int2* counts, int cap, const int* row_of, const GT* g,
                    int ldg, float* out, float sign, const int* gidx, int n_total,
                    const int2* mrange, const uint32_t* status, const EnergyArgs* energy,
                    int nmol_cap, float4* pgrad, hipStream_t st) {
  if (pgrad) {
    const int nb_e = energy && energy->E && nmol_cap > 0 ? nmol_cap : 0;
    const EnergyArgs ea = nb_e ? *energy : EnergyArgs{};
    const int nb_adj = n_cap > 0 ? (n_cap + 3) / 4 : 0;
    if (nb_adj + nb_e == 0) return;
    const size_t lds = (size_t)4 * aev_region(cap) * kBwdBytesPerNbr;
    static const bool attr = (ensure_lds(k_aev_bwd_det<GT>), true);
    (void)attr;
    hipLaunchKernelGGL((k_aev_bwd_det<GT>), dim3(nb_adj + nb_e), dim3(256), lds, st, dims, C,
                       rec, counts, cap, row_of, g, ldg, pgrad, nb_adj, ea);
    return;
  }
  const int nb_e = energy && energy->E && nmol_cap > 0 ? nmol_cap : 0;
  const EnergyArgs ea = nb_e ? *energy : EnergyArgs{};
  // Molecules: above 10,000 atoms workgroups with LDS windows, below it four
  // atoms per wave and direct additions.  Measured, whole evaluation of
  // 64-atom molecules, seven elements, BF16 (us, direct / window): 1,024 atoms
  // 36.3 / 41.2, 8,192: 52.0 / 52.5, 12,288: 70.7 / 66.4, 32,768: 126 / 105.
  // Boxes (long lists) and large subsets: one atom per wave.
  const bool mol = mrange != nullptr;
  const bool window = mol && !gidx && n_cap > 10000;
  const bool small = mol && n_cap <= 10000;
  const int per_block = window ? kMolBlock : (small ? 16 : 4);
  const int nb_adj = n_cap > 0 ? (n_cap + per_block - 1) / per_block : 0;
  if (nb_adj + nb_e == 0) return;
  if (window)
    hipLaunchKernelGGL((k_aev_bwd_mol<GT>), dim3(nb_adj + nb_e), dim3(64 * kMolWaves), 0, st, dims,
                       C, xyzs, rec, nbr, counts, cap, row_of, g, ldg, out, sign, mrange, status,
                       nb_adj, ea);
  else
    hipLaunchKernelGGL(small ? k_aev_bwd_small<GT> : k_aev_bwd<GT>, dim3(nb_adj + nb_e), dim3(256),
                       0, st, dims, C, xyzs, rec, nbr, counts, cap, row_of, g, ldg, out, sign,
                       gidx, n_total, status, nb_adj, ea);
}
template void launch_aev_bwd<float>(const int*, int, const AevConst&, const float4*, const float4*, const int*,
                                    const int2*, int, const int*, const float*, int, float*, float,
                                    const int*, int, const int2*, const uint32_t*, const EnergyArgs*,
                                    int, float4*, hipStream_t);
template void launch_aev_bwd<bf16_t>(const int*, int, const AevConst&, const float4*, const float4*, const int*,
                                     const int2*, int, const int*, const bf16_t*, int, float*,
                                     float, const int*, int, const int2*, const uint32_t*,
                                     const EnergyArgs*, int, float4*, hipStream_t);

}  // namespace nnp
