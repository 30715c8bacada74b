// Dispatch of the fused network by operand type and hidden widths, and dE/dG
// of ensembles.
#include "mlp_net.h"

namespace nnp {

void launch_net_bf16_7(const NetArgs&, int, int, int, hipStream_t);
void launch_net_bf16_4(const NetArgs&, int, int, int, hipStream_t);
void launch_net_fp32_7(const NetArgs&, int, int, int, hipStream_t);
void launch_net_fp32_4(const NetArgs&, int, int, int, hipStream_t);

template <typename T>
bool launch_mlp_net(const int* width, const NetArgs& a, int n_rows, int rows_cap, int members,
                    hipStream_t st) {
  if (!net_widths(width, a.ldx) || !a.X || !a.kmask) return false;
  if (a.H1 && !(a.H2 && a.H3 && a.D3 && a.D2 && a.D1 && a.uprow)) return false;
  const bool seven = width[1] == 256;
  if constexpr (sizeof(T) == 2)
    (seven ? launch_net_bf16_7 : launch_net_bf16_4)(a, n_rows, rows_cap, members, st);
  else
    (seven ? launch_net_fp32_7 : launch_net_fp32_4)(a, n_rows, rows_cap, members, st);
  return true;
}
template bool launch_mlp_net<bf16_t>(const int*, const NetArgs&, int, int, int, hipStream_t);
template bool launch_mlp_net<float>(const int*, const NetArgs&, int, int, int, hipStream_t);

// Rows per tile.  A tile's chain of products takes about the same time
// whatever its rows (28 us with 64 rows, 15 us with 16 for BF16 in the idle
// GPU), so small systems spread over small tiles and large ones, whose tiles
// fill the 512 places on the GPU anyway, share the weight stream among more
// rows.  Measured, whole evaluation of 64-atom molecules of seven elements
// (rows: us with 16 / 32 / 64): BF16 2,048: 61.5 / 63.9 / 70.7; 8,192: 75.6 /
// 71.2 / 78.5; 12,288: 94.8 / 82.5 / 81.8; 32,768: 152 / 126 / 114.  FP32
// 2,048: 79.8 / 100.1 / 145.6; 6,144: 117.3 / 112.0 / 165.6; 32,768: 325 /
// 308 / 307 (64 rows of FP32 activations leave one workgroup per CU, and at
// 24,576 take 328 against 270: no use).  Ensembles: the members' tiles count
// for BF16; FP32 eight members 2,048: 229 / 244, 4,096: 384 / 399.  Rows sorted
// by k-steps make small FP32 tiles cheaper (network of seven elements, 16 / 32:
// 8,192: 48 / 52, 12,160: 85 / 97, 16,000: 105 / 105, 32,768: 178 / 163; BF16
// 32 / 64: 19,200: 29 / 29, 32,768: 40 / 33, as without).
template <typename T>
int net_tile(int n_rows, int members, bool ordered) {
  const long rows = (long)n_rows * members;
  if (sizeof(T) == 4) return n_rows <= 4096 || (ordered && rows <= 14336) ? 16 : 32;
  return rows <= 3072 ? 16 : (rows <= 10240 ? 32 : 64);
}
template int net_tile<float>(int, int, bool);
template int net_tile<bf16_t>(int, int, bool);

// ------------------------------------------------------------ the rows' order
//
// Layer 1 and dE/dG run over the union of a tile's k-steps.  Neighboring rows
// of a group belong to unlike atoms: 32 rows of one element in 512 conformers
// of 64 atoms have 13 k-steps together, a row alone 4.4.  Sorted by their masks
// as numbers (the k-steps of the rarest elements come last and lead the order)
// within windows of 1,024 rows they have 5.3; 64 rows of random molecules 10
// for 22.  A row's rank in its window is the number of smaller masks (equal
// ones: of earlier rows), so the order follows from the rows alone.  One
// workgroup ranks 64 rows, each wave against an eighth of the window from LDS
// (6 us for 8,192 rows, 7 for 32,768, 12 for 77,163: latencies, then the
// comparisons; four waves 8 / 8 / 11, sixteen 5 / 8 / 18, 128 rows at a time 10 /
// 10 / 14).
//
// The last rows of a window have the k-steps of rare elements and the most
// unlike masks: their tiles take up to twice the time of the others.  Eight
// more workgroups list the tiles of each XCD's range with the ends of all
// windows first, so that no long tile starts last (512 x 64 conformers in FP32,
// two rounds of tiles: 194 us with the tiles in order, now 166; 77,163 rows in
// BF16 96, now 81).
constexpr int kOrderWaves = 8;
__device__ __forceinline__ void order_tiles(const GroupTable* __restrict__ gt, int xcd,
                                            int tile_rows, int* __restrict__ tiles, int* bin) {
  // bin[p]: tiles p places before the end of their window
  const int per = kNetWindow / tile_rows, tid = threadIdx.x;
  const int nt = gt->total_rows / tile_rows;
  const int lo = xcd < nt ? xcd_tile(xcd, nt) : 0, m = xcd < nt ? (nt - xcd + 7) / 8 : 0;
  auto place = [&](int t) {
    const int row0 = t * tile_rows, s = tile_species(gt, row0), g0 = gt->pstart[s];
    const int len = (gt->cnt[s] + tile_rows - 1) / tile_rows, i = row0 / tile_rows - g0 / tile_rows;
    const int end = (i / per + 1) * per;
    const int p = (end < len ? end : len) - 1 - i;
    return p < 0 ? per - 1 : p;  // (tiles of padding only)
  };
  for (int p = tid; p < per; p += 64 * kOrderWaves) bin[p] = 0;
  __syncthreads();
  for (int j = tid; j < m; j += 64 * kOrderWaves) atomicAdd(&bin[place(lo + j)], 1);
  __syncthreads();
  if (tid < 64) {  // per <= 64: exclusive sums in place
    const int v = tid < per ? bin[tid] : 0;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int u = __shfl_up(x, d, 64);
      if (tid >= d) x += u;
    }
    if (tid < per) bin[tid] = x - v;
  }
  __syncthreads();
  for (int j = tid; j < m; j += 64 * kOrderWaves)
    tiles[lo + atomicAdd(&bin[place(lo + j)], 1)] = lo + j;
}

template <typename K>
__global__ __launch_bounds__(64 * kOrderWaves) void k_net_order(
    const GroupTable* __restrict__ gt, const unsigned long long* __restrict__ kmask,
    const int* __restrict__ perm, int nrank, int tile_rows, NetRow* __restrict__ order,
    int* __restrict__ tiles) {
  constexpr int W = kNetWindow, SL = W / kOrderWaves;  // keys per wave
  static_assert(SL % 64 == 0, "64 keys are the rows' own or none of them");
  __shared__ __attribute__((aligned(16))) K key[W];
  __shared__ int part[kOrderWaves][64];
  if ((int)blockIdx.x >= nrank) {
    order_tiles(gt, blockIdx.x - nrank, tile_rows, tiles, &part[0][0]);
    return;
  }
  const int row0 = blockIdx.x * 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (row0 >= gt->total_rows) return;
  const int s = tile_species(gt, row0);
  const int g0 = gt->pstart[s], g1 = g0 + gt->cnt[s];
  if (row0 >= g1) return;
  const int w0 = g0 + (row0 - g0) / W * W;
  const int cnt = g1 - w0 < W ? g1 - w0 : W;
  const int row = row0 + lane;
  const unsigned long long m = row < g1 ? kmask[row] : 0ull;
  const int atom = wv == 0 && row < g1 ? perm[row] : -1;
#pragma unroll
  for (int i = tid; i < W; i += 64 * kOrderWaves) key[i] = i < cnt ? (K)kmask[w0 + i] : (K)~(K)0;
  __syncthreads();
  const K mine = (K)m;
  const int own = row0 - w0;
  int n = 0;
  for (int k0 = wv * SL; k0 < (wv + 1) * SL && k0 < cnt; k0 += 64) {
    const K* k = key + k0;
    if (k0 < own) {
#pragma unroll 32
      for (int j = 0; j < 64; ++j) n += k[j] <= mine;
    } else if (k0 > own) {
#pragma unroll 32
      for (int j = 0; j < 64; ++j) n += k[j] < mine;
    } else {
#pragma unroll 32
      for (int j = 0; j < 64; ++j) n += k[j] < mine || (k[j] == mine && j < lane);
    }
  }
  part[wv][lane] = n;
  __syncthreads();
  if (wv == 0 && row < g1) {
    int at = 0;
#pragma unroll
    for (int w = 0; w < kOrderWaves; ++w) at += part[w][lane];
    order[w0 + at] = NetRow{m, row, atom};
  }
}

void launch_net_order(const GroupTable* gt, const unsigned long long* kmask, const int* perm,
                      int ldx, int rows_cap, int tile_rows, NetRow* order, int* tiles,
                      hipStream_t st) {
  const int nrank = rows_cap / 64;
  const dim3 grid(nrank + 8), block(64 * kOrderWaves);
  if (ldx <= 32 * 32)
    hipLaunchKernelGGL(k_net_order<unsigned>, grid, block, 0, st, gt, kmask, perm, nrank,
                       tile_rows, order, tiles);
  else
    hipLaunchKernelGGL(k_net_order<unsigned long long>, grid, block, 0, st, gt, kmask, perm, nrank,
                       tile_rows, order, tiles);
}

// ------------------------------------------------------- dE/dG of an ensemble
//
// One workgroup per 64-row tile and group of 4 UN active k-steps of the
// tile's rows (32 columns of G each, UN per wave): the members' delta1 stream
// through two LDS chunk buffers, the weights through the register ring.  The
// members are summed inside the FP32 accumulator, in member order.  Held to two
// waves per SIMD: left alone the compiler takes 278 registers for BF16 with two
// k-steps per wave and one wave per SIMD (eight members, 32,768 rows: 64 us,
// now 54; with unsorted rows 91 and 72).
template <typename T, int UN, int P>
struct GradRing {
  static constexpr int FB = 64 * 16;
  uint4 r[P][2 * UN];
  const unsigned char* base[UN];
  unsigned lane16, tile;
  int ns;
  __device__ __forceinline__ void init(const T* B, int K, int lane, const int (&q)[UN]) {
    ns = K / Frag<T>::KS;
    tile = (unsigned)ns * FB;
#pragma unroll
    for (int u = 0; u < UN; ++u)
      base[u] = reinterpret_cast<const unsigned char*>(B) + (size_t)(2 * q[u]) * tile;
    lane16 = (unsigned)lane * 16;
  }
  template <int U>
  __device__ __forceinline__ void load(int s) {
    const unsigned at = (unsigned)(s < ns ? s : ns - 1) * FB;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      r[U][2 * u] = *reinterpret_cast<const uint4*>(base[u] + at + lane16);
      r[U][2 * u + 1] = *reinterpret_cast<const uint4*>(base[u] + (at + tile) + lane16);
    }
  }
  template <int U = 0>
  __device__ __forceinline__ void prologue() {
    if constexpr (U < P) {
      load<U>(U);
      prologue<U + 1>();
    }
  }
};

template <typename T, int UN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_net_grad(NetGradArgs a) {
  constexpr int BM = 64, NTH = 256, ES = sizeof(T), TM = BM / 16;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BM * kNetChunkStride];
  __shared__ unsigned long long rmask[BM];
  __shared__ int rrow[BM];
  const GroupTable* gt = a.gt;
  const int nt = gt->total_rows / BM;
  if ((int)blockIdx.x >= nt) return;
  const int row0 = xcd_tile(blockIdx.x, nt) * BM;
  const int s = tile_species(gt, row0);
  const int row_end = gt->pstart[s] + gt->cnt[s];
  if (row0 >= row_end) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rl = lane & 15, cq = (lane >> 4) * 4;
  const int K = a.K, ldx = a.ldx;
  const int nks = ldx / 32;
  const unsigned long long all = nks >= 64 ? ~0ull : (1ull << nks) - 1ull;
  unsigned long long m = 0ull;
  int row = row0 + lane;
  if (row < row_end) {
    m = (a.order ? a.order[row].mask : a.kmask[row]) & all;
    if (a.order) row = a.order[row].row;
  }
  if (tid < BM) {
    rmask[tid] = m;
    rrow[tid] = row;
  }
  unsigned lo = (unsigned)m, hi = (unsigned)(m >> 32);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    lo |= __shfl_xor(lo, d, 64);
    hi |= __shfl_xor(hi, d, 64);
  }
  const unsigned long long U = ((unsigned long long)__builtin_amdgcn_readfirstlane(hi) << 32) |
                               (unsigned)__builtin_amdgcn_readfirstlane(lo);
  const int nact = __popcll(U);
  const int p0 = (int)blockIdx.y * 4 * UN;
  if (p0 >= nact) return;  // block-uniform
  const int qlist = nth_set_bit(U, lane);
  int q[UN];
#pragma unroll
  for (int u = 0; u < UN; ++u) {
    const int p = p0 + wv * UN + u;
    q[u] = __builtin_amdgcn_readlane(qlist, p < nact ? p : nact - 1);
  }

  // (the tile's rows only: an element's may be more bytes than a range can say)
  const int rows = row_end - row0 < BM ? row_end - row0 : BM;
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(static_cast<const T*>(a.D1) + (size_t)row0 * K), (short)0,
      rows * K * ES, kBufferRsrcWord3);
  constexpr int RPV = NTH / 16, NVA = BM / RPV;
  auto aload = [&](int c, uint4 (&ra)[NVA]) __attribute__((always_inline)) {
    const int col = c * (kNetChunk / ES) + (tid & 15) * (16 / ES);
#pragma unroll
    for (int v = 0; v < NVA; ++v) {
      const int r = (tid >> 4) + RPV * v;
      const unsigned off = col < K ? (unsigned)((r * K + col) * ES) : kOutOfRange;
      const u32x4_t val = __builtin_amdgcn_raw_buffer_load_b128(arsrc, off, 0, 0);
      ra[v] = make_uint4(val[0], val[1], val[2], val[3]);
    }
  };
  auto astore = [&](int buf, const uint4 (&ra)[NVA]) __attribute__((always_inline)) {
    unsigned char* base = smem + buf * BM * kNetChunkStride;
#pragma unroll
    for (int v = 0; v < NVA; ++v)
      *reinterpret_cast<uint4*>(base + ((tid >> 4) + RPV * v) * kNetChunkStride + (tid & 15) * 16) =
          ra[v];
  };
  GradRing<T, UN, 4> br;
  br.init(static_cast<const T*>(a.Wc) + (size_t)s * ldx * K, K, lane, q);
  br.prologue();
  uint4 ra0[NVA], ra1[NVA];
  const int nu = (K * ES + kNetChunk - 1) / kNetChunk;
  aload(0, ra0);
  aload(1 < nu ? 1 : 0, ra1);
  f32x4_t acc[TM][2 * UN];
  zero_acc(acc);
  astore(0, ra0);
  __syncthreads();
  const int arow = rl * kNetChunkStride + (lane >> 4) * 16;
  auto unit = [&](int u, uint4 (&r_next2)[NVA], const uint4 (&r_next1)[NVA])
                  __attribute__((always_inline)) {
    aload(u + 2 < nu ? u + 2 : nu - 1, r_next2);
    kgroup<T, TM, 2 * UN, 4>(smem + (u & 1) * BM * kNetChunkStride + arow, 16 * kNetChunkStride, br,
                             u * 4, acc);
    astore((u + 1) & 1, r_next1);
    __syncthreads();
  };
  for (int u = 0; u < nu; u += 2) {
    unit(u, ra0, ra1);
    if (u + 1 < nu) unit(u + 1, ra1, ra0);
  }
#pragma unroll
  for (int u = 0; u < UN; ++u) {
    if (p0 + wv * UN + u >= nact) break;  // wave-uniform
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = i * 16 + rl;
      if (row0 + r < row_end && ((rmask[r] >> q[u]) & 1ull)) {
        T* g = static_cast<T*>(a.G) + (size_t)rrow[r] * ldx + q[u] * 32 + cq;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4_t v = acc[i][2 * u + j];
          Store<T>::put4(g + j * 16, make_float4(v[0], v[1], v[2], v[3]));
        }
      }
    }
  }
}

// Small FP32 calls: one workgroup per 16-row tile and four active k-steps of
// it.  The tile's deltas all lie in LDS (16 rows of up to 8 KB), so the loop has
// no barriers, a ring of 16 steps keeps the weights' latency out of it, and no
// products run for 48 absent rows; the sums are those of the large form, step
// by step.  Eight members of 256 columns, 128 / 1,024 / 1,536 / 2,048 atoms: 71 /
// 72 / 73 / 73 us in the large form, whose tiles then run side by side, 27 / 54 /
// 77 / 102 here; eight of 160, 1,024 / 2,048 / 3,072: 48 / 48 / 48 and 36 / 38 /
// 53; two of 256, 1,536 / 2,048: 23 / 24 and 17 / 27.  BF16, half the bytes and an eighth of the matrix time, is faster in
// the large form, which multiplies while it loads (53 / 1,024 atoms 12 / 13 us,
// 14 / 15 here).
constexpr int kGradSmallRing = 16;
constexpr int kGradSmallRows = 1024;
template <typename T, int S = 0>
__device__ __forceinline__ void grad_steps(const unsigned char* ap, GradRing<T, 1, kGradSmallRing>& br,
                                           int s0, f32x4_t (&acc)[1][2], uint4 (&fe)[1],
                                           uint4 (&fo)[1]) {
  constexpr int P = kGradSmallRing, SB = Frag<T>::KS * sizeof(T);
  if constexpr (S < P) {
    if constexpr (S % 2 == 0)
      kstep<T, 1, 2, P, S, true, (S + 1 < P)>(ap + (S + 1) * SB, 0, br, s0 + S + P, acc, fe, fo);
    else
      kstep<T, 1, 2, P, S, true, (S + 1 < P)>(ap + (S + 1) * SB, 0, br, s0 + S + P, acc, fo, fe);
    grad_steps<T, S + 1>(ap, br, s0, acc, fe, fo);
  }
}

template <typename T>
constexpr int grad_small_steps(int K) {  // K in steps, whole rings
  return (K / Frag<T>::KS + kGradSmallRing - 1) / kGradSmallRing * kGradSmallRing;
}

template <typename T>
__global__ __launch_bounds__(256) void k_net_grad_small(NetGradArgs a) {
  constexpr int BM = 16, ES = sizeof(T), SB = Frag<T>::KS * ES;
  static_assert(SB == 64, "a step is four 16-byte pieces of a row");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ unsigned long long rmask[BM];
  __shared__ int rrow[BM];
  const GroupTable* gt = a.gt;
  const int nt = gt->total_rows / BM;
  if ((int)blockIdx.x >= nt) return;
  const int row0 = xcd_tile(blockIdx.x, nt) * BM;
  const int s = tile_species(gt, row0);
  const int row_end = gt->pstart[s] + gt->cnt[s];
  if (row0 >= row_end) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rl = lane & 15, cq = (lane >> 4) * 4;
  const int K = a.K, ldx = a.ldx, nks = ldx / 32;
  const unsigned long long all = nks >= 64 ? ~0ull : (1ull << nks) - 1ull;
  unsigned long long m = 0ull;
  int row = row0 + rl;
  if (row < row_end) {
    m = (a.order ? a.order[row].mask : a.kmask[row]) & all;
    if (a.order) row = a.order[row].row;
  }
  if (tid < BM) {
    rmask[tid] = m;
    rrow[tid] = row;
  }
  const unsigned long long U =
      ((unsigned long long)wave_or((unsigned)(m >> 32)) << 32) | wave_or((unsigned)m);
  const int nact = __popcll(U);
  const int p = (int)blockIdx.y * 4 + wv;
  if ((int)blockIdx.y * 4 >= nact) return;  // block-uniform
  int q[1];
  q[0] = __builtin_amdgcn_readlane(nth_set_bit(U, lane), p < nact ? p : nact - 1);
  GradRing<T, 1, kGradSmallRing> br;
  br.init(static_cast<const T*>(a.Wc) + (size_t)s * ldx * K, K, lane, q);
  br.prologue();
  const int nsp = grad_small_steps<T>(K), stride = nsp * SB + 16;
  const int rows = row_end - row0 < BM ? row_end - row0 : BM;
  const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(static_cast<const T*>(a.D1) + (size_t)row0 * K), (short)0,
      rows * K * ES, kBufferRsrcWord3);
  constexpr int NL = 8;
  const int pieces = nsp * 4;  // per row
  for (int c0 = tid; c0 < BM * pieces; c0 += 256 * NL) {
    u32x4_t v[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int c = c0 + 256 * k, r = c / pieces, at = (c - r * pieces) * 16;
      v[k] = __builtin_amdgcn_raw_buffer_load_b128(
          src, r < BM && at < K * ES ? (unsigned)(r * K * ES + at) : kOutOfRange, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int c = c0 + 256 * k, r = c / pieces, at = (c - r * pieces) * 16;
      if (r < BM)
        *reinterpret_cast<uint4*>(smem + r * stride + at) =
            make_uint4(v[k][0], v[k][1], v[k][2], v[k][3]);
    }
  }
  __syncthreads();
  f32x4_t acc[1][2];
  zero_acc(acc);
  const unsigned char* ap = smem + rl * stride + (lane >> 4) * 16;
  for (int s0 = 0; s0 < nsp; s0 += kGradSmallRing) {
    uint4 fe[1], fo[1];
    load_a<1>(ap, 0, fe);
    grad_steps<T>(ap, br, s0, acc, fe, fo);
    ap += kGradSmallRing * SB;
  }
  if (p >= nact) return;  // wave-uniform, no barrier after
  if (row0 + rl < row_end && ((rmask[rl] >> q[0]) & 1ull)) {
    T* g = static_cast<T*>(a.G) + (size_t)rrow[rl] * ldx + q[0] * 32 + cq;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      Store<T>::put4(g + j * 16, make_float4(acc[0][j][0], acc[0][j][1], acc[0][j][2], acc[0][j][3]));
  }
}

template <typename T>
void launch_net_grad(const NetGradArgs& a, int n_rows, int rows_cap, hipStream_t st) {
  const int tiles = rows_cap / 64, nks = a.ldx / 32;
  if constexpr (sizeof(T) == 4) {
    if (n_rows <= kGradSmallRows) {
      static const bool attr = (ensure_lds(k_net_grad_small<T>), true);
      (void)attr;
      const size_t lds = 16 * ((size_t)grad_small_steps<T>(a.K) * 64 + 16);
      hipLaunchKernelGGL(k_net_grad_small<T>, dim3(rows_cap / 16, (nks + 3) / 4), dim3(256), lds,
                         st, a);
      return;
    }
  }
  // two k-steps per wave where the tiles alone fill the GPU (the deltas are
  // read once per eight k-steps then), else one
  if (tiles >= 256)
    hipLaunchKernelGGL((k_net_grad<T, 2>), dim3(tiles, (nks + 7) / 8), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_net_grad<T, 1>), dim3(tiles, (nks + 3) / 4), dim3(256), 0, st, a);
}
template void launch_net_grad<bf16_t>(const NetGradArgs&, int, int, hipStream_t);
template void launch_net_grad<float>(const NetGradArgs&, int, int, hipStream_t);

}  // namespace nnp
