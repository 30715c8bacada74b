// The whole per-element network of one tile of species-sorted rows in one
// workgroup: layer 1, layer 2, the energy head and, with gradients, the
// adjoint of layers 3 and 2 and dE/dG.
//
//   H1 = CELU(X W0^T + b0)      X streamed through two LDS chunk buffers
//   H2 = CELU(H1 W1^T + b1)
//   z3 = H2 W2^T + b2;  E_i = w_out . CELU(z3) + b_out
//   D3 = up_i * w_out * CELU'(z3)
//   D2 = (D3 W2) * CELU'(z2)    over H2
//   D1 = (D2 W1) * CELU'(z1)    over H1
//   G  = D1 W0                  dE/dG, to global memory
//
// Activations and deltas never leave LDS (in the operand type T: BF16 or
// FP32); the weights stream from L2 into MFMA operand registers in fragment
// order (mfma_tile.h).  CELU'(z) is recovered from the stored activation: 1
// for h > 0, else 1 + h/alpha.
//
// Feature rows are sparse: an atom touches the blocks of the elements around
// it only.  With the rows' k-step masks (32 columns of X per bit) a tile runs
// layer 1 and dE/dG over the union of its rows' k-steps (a compacted list,
// one entry per lane), each row reads its own k-steps of X (the others load
// as zero through the buffer resource) and writes its own k-steps of dE/dG,
// which are all the symmetry-function adjoint reads.  The skipped steps would
// add exact zeros, so the results do not change.
//
// What bounds it: the chain of one tile.  On the 32,768-atom batch every tile
// is resident at once (two workgroups of 80 KB LDS per CU), and each of its
// products is short, so the time is the sum of the products' latencies and of
// the epilogues' vector work.  Hence: the next product's weight fragments are
// requested between the tiles of an epilogue (BF16: all of them; in one burst
// before it they queue for 1.6 us behind each other, 64 bytes per clock and
// CU, and the epilogue's arithmetic waits), biases, upstream gradients and
// row indices before the products that need them, CELU has no branch, and
// conversions to BF16 are packed.  Kernel time per evaluation (from traces, as
// all kernel times in these sources), BF16 batch: 42 -> 40 us; FP32 batch, which
// ran one GEMM per layer with activations through HBM: 342 -> 256 us, and 166
// with the rows sorted by k-steps (its products at the rate a large FP32 product
// reaches, 154 TFLOP/s, take 101); one 24-atom molecule in FP32: 108 -> 21 us;
// an eight-network ensemble with its dE/dG, which ran two launches per member:
// 603 -> 289 us on the batch, 245 with sorted rows, 402 -> 31 us on one 53-atom
// molecule.
//
// Every row's result is independent of the tile it sits in: the sums over K
// run in the same order for every tile size, and the energy's sum over the
// last hidden layer in one of two fixed orders (HEAD).
#pragma once
#include "mfma_tile.h"

namespace nnp {

constexpr int kNetWaves = 4;

// Waves of a product with N columns over BM rows: 4 column groups (2 by 2 row
// groups when N is not a multiple of 64).  16-row tiles give every wave all
// rows and deal the 16-column tiles out in turn (the last wave may have
// fewer).
template <int N, int BM>
struct NetProd {
  static constexpr int NW = kNetWaves;
  static constexpr int NT = N / 16;
  static constexpr bool spread = BM == 16;
  static constexpr int WN = spread ? NW : (N % 64 == 0 ? 4 : 2);
  static constexpr int WM = NW / WN;
  static constexpr int TM = BM / 16 / WM;
  static constexpr int TN = (NT + WN - 1) / WN;
  static constexpr bool even = TN * WN == NT;
  static_assert(WM * WN == NW && WM * TM * 16 == BM, "the waves cover the rows");
  static_assert(spread || even, "the waves cover the columns");
};

// Register ring of a product's weight fragments: slot u holds the wave's TN
// fragments of every k-step s with s % P == u.  The address is a uniform base
// plus the lane's 16 bytes.  Not EVEN: tiles past the last re-read it.
template <typename T, int TN, int P, bool EVEN>
struct NetRing {
  static constexpr int FB = 64 * 16;  // bytes of a fragment
  uint4 r[P][TN];
  const unsigned char* base;
  unsigned lane16;
  unsigned tile;  // bytes per 16-row tile (all k-steps)
  int jl;
  __device__ __forceinline__ void init(const T* B, int nt0, int nt, int K, int lane) {
    tile = (unsigned)(K / Frag<T>::KS) * FB;
    if constexpr (!EVEN) nt0 = nt0 < nt ? nt0 : nt - 1;
    jl = nt - 1 - nt0;
    base = reinterpret_cast<const unsigned char*>(B) + (size_t)nt0 * tile;
    lane16 = (unsigned)lane * 16;
  }
  template <int U>
  __device__ __forceinline__ void load(int s) {
    const unsigned char* p = base + (unsigned)s * FB;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const unsigned jj = EVEN ? (unsigned)j : (unsigned)(j < jl ? j : jl);
      r[U][j] = *reinterpret_cast<const uint4*>(p + (size_t)(jj * tile) + lane16);
    }
  }
  // fragment f of the first min(P, NS) steps (f a constant after unrolling):
  // the epilogue before the product asks for a few after each of its tiles
  __device__ __forceinline__ void fetch(int f) {
    const int u = f / TN, j = f % TN;
    const unsigned jj = EVEN ? (unsigned)j : (unsigned)(j < jl ? j : jl);
    const unsigned char* p = base + (unsigned)u * FB;
    r[u][j] = *reinterpret_cast<const uint4*>(p + (size_t)(jj * tile) + lane16);
  }
  // epilogue tile t of NE (0 .. NE - 1) asks for its share
  template <int NS, int NE>
  __device__ __forceinline__ void fetch_share(int t) {
    constexpr int NF = (P < NS ? P : NS) * TN, PER = (NF + NE - 1) / NE;
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (t * PER + q < NF) fetch(t * PER + q);
    __builtin_amdgcn_sched_barrier(0);
  }
};

// The same over the tile's compacted list of active k-steps of X: position s
// is fragment step s % R of the (s / R)-th active mask step (R = 1 for BF16,
// 2 for FP32, whose fragments hold 16 columns).  Positions past the end
// re-read the last one, so every access stays inside B and the loads in
// flight before a step are an exact count.
template <typename T, int TN, int P, bool EVEN>
struct NetRingQ {
  static constexpr int FB = 64 * 16;
  static constexpr int R = 32 / Frag<T>::KS;
  uint4 r[P][TN];
  const unsigned char* base;
  unsigned lane16;
  unsigned tile;
  int jl, nact, qlist;
  __device__ __forceinline__ void init(const T* B, int nt0, int nt, int K, int lane, int nact_,
                                       int qlist_) {
    tile = (unsigned)(K / Frag<T>::KS) * FB;
    if constexpr (!EVEN) nt0 = nt0 < nt ? nt0 : nt - 1;
    jl = nt - 1 - nt0;
    base = reinterpret_cast<const unsigned char*>(B) + (size_t)nt0 * tile;
    lane16 = (unsigned)lane * 16;
    nact = nact_;
    qlist = qlist_;
  }
  template <int U>
  __device__ __forceinline__ void load(int s) {
    const int m = s / R;
    const int q = __builtin_amdgcn_readlane(qlist, m < nact ? m : (nact > 0 ? nact - 1 : 0));
    const unsigned char* p = base + (unsigned)(q * R + s % R) * FB;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const unsigned jj = EVEN ? (unsigned)j : (unsigned)(j < jl ? j : jl);
      r[U][j] = *reinterpret_cast<const uint4*>(p + (size_t)(jj * tile) + lane16);
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

template <typename T> struct LdsV;
template <> struct LdsV<bf16_t> {
  __device__ __forceinline__ static void put(unsigned char* p, float4 v) {
    *reinterpret_cast<uint2*>(p) = make_uint2(f2bf2(v.x, v.y), f2bf2(v.z, v.w));
  }
  __device__ __forceinline__ static float4 get(const unsigned char* p) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                       __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
  }
};
template <> struct LdsV<float> {
  __device__ __forceinline__ static void put(unsigned char* p, float4 v) {
    *reinterpret_cast<float4*>(p) = v;
  }
  __device__ __forceinline__ static float4 get(const unsigned char* p) {
    return *reinterpret_cast<const float4*>(p);
  }
};

constexpr int kNetChunk = 256;                  // bytes of X per row and chunk (four fragments)
constexpr int kNetChunkStride = kNetChunk + 16;

template <typename T, int W1, int W2, int W3, int BM>
struct NetLds {
  static constexpr int ES = sizeof(T);
  static constexpr int S1 = W1 * ES + 16, S2 = W2 * ES + 16, S3 = W3 * ES + 16;
  static constexpr int SH = W3 * 4 + 16;                         // 16-row tiles: h3 in FP32
  static constexpr int EP = BM == 16 ? BM * SH : 2 * BM * 4;     // energy partials
  static constexpr int D3 = BM * S2 + EP;
  static constexpr int RA_MID = D3 + BM * S3;                    // region A after layer 1
  static constexpr int RA_L1 = 2 * BM * kNetChunkStride;         // ... during it
  static constexpr int RA = RA_MID > RA_L1 ? RA_MID : RA_L1;
  static constexpr int X1 = RA;                                  // H1, then D1
  static constexpr int MASKS = X1 + BM * S1;
  static constexpr size_t bytes = (size_t)MASKS + BM * 8;
  // the tile's row numbers sit in the padding of X1's rows (64 BF16 rows fill
  // half a CU's LDS to the byte)
  static constexpr int ROWS = X1 + W1 * ES;
  static_assert(RA % 16 == 0 && D3 % 16 == 0 && MASKS % 8 == 0, "aligned regions");
};

// CELU without a branch: the exponential of a positive z (possibly infinite)
// is computed and not selected.
__device__ __forceinline__ float net_celu(float z, float alpha, float ial2e) {
  const float ex = __builtin_amdgcn_exp2f(z * ial2e);
  const float neg = alpha * (ex - 1.f);
  return z > 0.f ? z : neg;
}

// BWD: also the adjoint (D1, and dE/dG when a.G).  STORE: keep H1, H2, H3,
// D3, D2, D1 and the upstream gradients in global memory for the weight
// gradients (H1's and D1's rows have W1 columns then).  blockIdx.y is the
// ensemble member; with a.D1 (and not STORE) its D1 goes to columns
// [member W1, ...) of a.D1's rows, which lie as the tiles take them.
// HEAD: the order of the energy's sum over the last hidden layer's columns.
//   false (BF16 with gradients): a lane adds its columns 16 j + 4 g + e of a
//     half in order of j, then e; then the four g, then the halves.
//   true: per column c of 16, the sum over j; then the 16 sums pairwise by
//     the bits of c from the lowest; then the halves.
template <typename T, int W1, int W2, int W3, int BM, bool BWD, bool STORE>
__global__ __launch_bounds__(64 * kNetWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_net(
    NetArgs a) {
  using LL = NetLds<T, W1, W2, W3, BM>;
  constexpr bool HEAD = !BWD || sizeof(T) == 4;
  constexpr int NTH = 64 * kNetWaves, ES = sizeof(T), KS = Frag<T>::KS, R = 32 / KS;
  constexpr int S1 = LL::S1, S2 = LL::S2, S3 = LL::S3;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* X2 = smem;
  float* epart = reinterpret_cast<float*>(smem + BM * S2);
  unsigned char* D3s = smem + LL::D3;
  unsigned char* X1 = smem + LL::X1;
  unsigned long long* rmask = reinterpret_cast<unsigned long long*>(smem + LL::MASKS);
  auto rrow = [&](int r) -> int& { return *reinterpret_cast<int*>(smem + LL::ROWS + r * S1); };

  const GroupTable* gt = a.gt;
  const int nt = gt->total_rows / BM;
  if ((int)blockIdx.x >= nt) return;
  int tile = xcd_tile(blockIdx.x, nt);
  if (a.order) tile = a.tiles[tile];
  const int row0 = tile * BM;
  const int s = tile_species(gt, row0);
  const int row_end = gt->pstart[s] + gt->cnt[s];
  if (row0 >= row_end) return;
  const int member = blockIdx.y;
  const int slot = member * a.S + s;  // weight slot
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rl = lane & 15, cq = (lane >> 4) * 4;
  const int K = a.ldx;
  const float alpha = a.alpha, ia = 1.f / a.alpha, ial2e = a.inv_alpha_l2e;

  // ---- the tile's k-steps: the union of its rows' masks, compacted into
  // qlist (lane l: the l-th active k-step); rows past the group have none
  const int nks = K / 32;
  const unsigned long long all = nks >= 64 ? ~0ull : (1ull << nks) - 1ull;
  // row r of the tile: by a.order, or the tile's rows as they lie
  auto net_row = [&](int r) -> NetRow {
    const int p = row0 + r;
    if (p >= row_end) return NetRow{0ull, p, -1};
    NetRow v = a.order ? a.order[p] : NetRow{a.kmask[p], p, a.perm[p]};
    v.mask &= all;
    return v;
  };
  static_assert(BM <= 64, "at most one row per lane");
  unsigned long long U;
  {
    unsigned long long m = 0ull;
    if (lane < BM) {
      const NetRow v = net_row(lane);
      m = v.mask;
      if (tid < BM) {
        rmask[tid] = m;
        rrow(tid) = v.row;
      }
    }
    unsigned lo = (unsigned)m, hi = (unsigned)(m >> 32);
#pragma unroll
    for (int d = 1; d < (BM < 64 ? BM : 64); d <<= 1) {
      lo |= __shfl_xor(lo, d, 64);
      hi |= __shfl_xor(hi, d, 64);
    }
    U = ((unsigned long long)__builtin_amdgcn_readfirstlane(hi) << 32) |
        (unsigned)__builtin_amdgcn_readfirstlane(lo);
  }
  const int nact = __popcll(U);
  const int qlist = nth_set_bit(U, lane);

  // the head's rows: their upstream gradients, and (threads < BM) the atom
  // each row's energy goes to, loaded here so that the head does not wait
  using C3 = NetProd<W3, BM>;
  float up[C3::TM];
#pragma unroll
  for (int i = 0; i < C3::TM; ++i) {
    up[i] = a.escale;
    if (BWD && a.dLdE) {
      const int atom = net_row((wv / C3::WN) * C3::TM * 16 + i * 16 + rl).atom;
      up[i] = atom >= 0 ? (float)a.dLdE[a.mol[atom]] * a.escale : 0.f;
    }
  }
  const bool erow_on = tid < (C3::spread ? BM * 16 : BM);
  const int erow_r = C3::spread ? tid >> 4 : tid;
  const int eatom = erow_on ? net_row(erow_r).atom : -1;

  // weight-ring depths: BF16 products are short, so all their fragments are
  // in flight over the previous product's epilogue; FP32 products are bound
  // by the MFMA rate and four steps cover a fragment's latency
  constexpr int P1 = ES == 2 ? (W1 / KS < 8 ? W1 / KS : 8) : 4;
  constexpr int P2 = ES == 2 ? (W2 / KS < 8 ? W2 / KS : 8) : 4;
  constexpr int P3 = ES == 2 ? (W3 / KS < 8 ? W3 / KS : 8) : 4;
  using C1 = NetProd<W1, BM>;
  using C2 = NetProd<W2, BM>;
  NetRing<T, C2::TN, P1, C2::even> br1;  // layer 2 (K = W1)

  // ---- layer 1 over the active k-steps, four fragments per chunk; thread t
  // loads 16-byte piece t % 16 of chunk rows t / 16 + (NTH / 16) v
  {
    constexpr int MS = 4 / R;           // mask steps per chunk
    constexpr int PPM = 16 / MS;        // 16-byte pieces per mask step
    constexpr int RPV = NTH / 16;       // rows per round of loads
    constexpr int NVA = (BM + RPV - 1) / RPV;
    // (an ordered tile's rows are of one window of its group)
    const int g0 = gt->pstart[s], win = g0 + (row0 - g0) / kNetWindow * kNetWindow;
    const int wrows = row_end - win < kNetWindow ? row_end - win : kNetWindow;
    const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(static_cast<const T*>(a.X) + (size_t)win * K), (short)0, wrows * K * ES,
        kBufferRsrcWord3);
    const int mslot = (tid & 15) / PPM, piece = (tid & 15) % PPM;
    unsigned long long rm[NVA];
    int xo[NVA];  // the row's offset in elements
#pragma unroll
    for (int v = 0; v < NVA; ++v) {
      const int r = (tid >> 4) + RPV * v;
      const NetRow w = r < BM ? net_row(r) : NetRow{0ull, win, -1};
      rm[v] = w.mask;
      xo[v] = (w.row - win) * K;
    }
    auto aload = [&](int c, uint4 (&ra)[NVA]) __attribute__((always_inline)) {
      const int pos = c * MS + mslot;
      const int q = __shfl(qlist, pos & 63, 64);
#pragma unroll
      for (int v = 0; v < NVA; ++v) {
        const bool on = pos < nact && ((rm[v] >> q) & 1ull);
        const unsigned off = on ? (unsigned)((xo[v] + q * 32) * ES + piece * 16) : kOutOfRange;
        const u32x4_t val = __builtin_amdgcn_raw_buffer_load_b128(arsrc, off, 0, 0);
        ra[v] = make_uint4(val[0], val[1], val[2], val[3]);
      }
    };
    auto astore = [&](int buf, const uint4 (&ra)[NVA]) __attribute__((always_inline)) {
      unsigned char* base = smem + buf * BM * kNetChunkStride;
#pragma unroll
      for (int v = 0; v < NVA; ++v) {
        const int r = (tid >> 4) + RPV * v;
        if (BM % RPV == 0 || r < BM)
          *reinterpret_cast<uint4*>(base + r * kNetChunkStride + (tid & 15) * 16) = ra[v];
      }
    };
    const int wm = wv / C1::WN, wn = wv % C1::WN;
    const int nu = nact > MS ? (nact + MS - 1) / MS : 1;
    const int arow = (wm * C1::TM * 16 + rl) * kNetChunkStride + (lane >> 4) * 16;
    uint4 ra0[NVA], ra1[NVA];
    aload(0, ra0);
    aload(1 < nu ? 1 : 0, ra1);
    NetRingQ<T, C1::TN, 4, C1::even> br;
    br.init(static_cast<const T*>(a.W0) + (size_t)slot * W1 * K, wn * C1::TN, C1::NT, K, lane,
            nact, qlist);
    br.prologue();
    float4 b[C1::TN];
#pragma unroll
    for (int j = 0; j < C1::TN; ++j) {
      const int ct = C1::even ? wn * C1::TN + j
                              : (wn * C1::TN + j < C1::NT ? wn * C1::TN + j : C1::NT - 1);
      b[j] = *reinterpret_cast<const float4*>(a.b0 + (size_t)slot * W1 + ct * 16 + cq);
    }
    f32x4_t acc[C1::TM][C1::TN];
    zero_acc(acc);
    astore(0, ra0);
    __syncthreads();
    auto unit = [&](int u, uint4 (&r_next2)[NVA], const uint4 (&r_next1)[NVA])
                    __attribute__((always_inline)) {
      aload(u + 2 < nu ? u + 2 : nu - 1, r_next2);
      kgroup<T, C1::TM, C1::TN, 4>(smem + (u & 1) * BM * kNetChunkStride + arow,
                                   16 * kNetChunkStride, br, u * 4, acc);
      astore((u + 1) & 1, r_next1);
      __syncthreads();
    };
    for (int u = 0; u < nu; u += 2) {
      unit(u, ra0, ra1);
      if (u + 1 < nu) unit(u + 1, ra1, ra0);
    }
    br1.init(static_cast<const T*>(a.W1) + (size_t)slot * W2 * W1, (wv % C2::WN) * C2::TN, C2::NT,
             W1, lane);
#pragma unroll
    for (int i = 0; i < C1::TM; ++i) {
      const int r = wm * C1::TM * 16 + i * 16 + rl;
#pragma unroll
      for (int j = 0; j < C1::TN; ++j) {
        const int ct = wn * C1::TN + j;
        if (C1::even || ct < C1::NT) {  // wave-uniform
          const int c = ct * 16 + cq;
          const float4 h = make_float4(net_celu(acc[i][j][0] + b[j].x, alpha, ial2e),
                                       net_celu(acc[i][j][1] + b[j].y, alpha, ial2e),
                                       net_celu(acc[i][j][2] + b[j].z, alpha, ial2e),
                                       net_celu(acc[i][j][3] + b[j].w, alpha, ial2e));
          LdsV<T>::put(X1 + r * S1 + c * ES, h);
          if (STORE) Store<T>::put4(static_cast<T*>(a.H1) + (size_t)rrow(r) * W1 + c, h);
        }
        br1.template fetch_share<W1 / KS, C1::TM * C1::TN>(i * C1::TN + j);
      }
    }
  }
  __syncthreads();  // H1 in X1; region A free

  // ---- H2 = CELU(H1 W1^T + b1)
  NetRing<T, C3::TN, P2, C3::even> br2;  // layer 3 (K = W2)
  {
    const int wm = wv / C2::WN, wn = wv % C2::WN;
    float4 b[C2::TN];
#pragma unroll
    for (int j = 0; j < C2::TN; ++j) {
      const int ct = wn * C2::TN + j < C2::NT ? wn * C2::TN + j : C2::NT - 1;
      b[j] = *reinterpret_cast<const float4*>(a.b1 + (size_t)slot * W2 + ct * 16 + cq);
    }
    f32x4_t acc[C2::TM][C2::TN];
    zero_acc(acc);
    uint4 fe[C2::TM], fo[C2::TM];
    ksteps_ct<T, C2::TM, C2::TN, P1, W1 / KS>(X1 + (wm * C2::TM * 16 + rl) * S1 + (lane >> 4) * 16,
                                              16 * S1, br1, acc, fe, fo);
    br2.init(static_cast<const T*>(a.W2) + (size_t)slot * W3 * W2, (wv % C3::WN) * C3::TN, C3::NT,
             W2, lane);
#pragma unroll
    for (int i = 0; i < C2::TM; ++i) {
      const int r = wm * C2::TM * 16 + i * 16 + rl;
#pragma unroll
      for (int j = 0; j < C2::TN; ++j) {
        const int ct = wn * C2::TN + j;
        if (C2::even || ct < C2::NT) {  // wave-uniform
          const int c = ct * 16 + cq;
          const float4 h = make_float4(net_celu(acc[i][j][0] + b[j].x, alpha, ial2e),
                                       net_celu(acc[i][j][1] + b[j].y, alpha, ial2e),
                                       net_celu(acc[i][j][2] + b[j].z, alpha, ial2e),
                                       net_celu(acc[i][j][3] + b[j].w, alpha, ial2e));
          LdsV<T>::put(X2 + r * S2 + c * ES, h);
          if (STORE) Store<T>::put4(static_cast<T*>(a.H2) + (size_t)rrow(r) * W2 + c, h);
        }
        br2.template fetch_share<W2 / KS, C2::TM * C2::TN>(i * C2::TN + j);
      }
    }
  }
  __syncthreads();

  // ---- z3 = H2 W2^T + b2: energies and D3
  NetRing<T, C2::TN, P3, C2::even> br3;  // adjoint of layer 3 (K = W3)
  {
    const int wm = wv / C3::WN, wn = wv % C3::WN;
    float4 b[C3::TN], w[C3::TN];
#pragma unroll
    for (int j = 0; j < C3::TN; ++j) {
      const int ct = wn * C3::TN + j < C3::NT ? wn * C3::TN + j : C3::NT - 1;
      b[j] = *reinterpret_cast<const float4*>(a.b2 + (size_t)slot * W3 + ct * 16 + cq);
      w[j] = *reinterpret_cast<const float4*>(a.wout + (size_t)slot * W3 + ct * 16 + cq);
    }
    f32x4_t acc[C3::TM][C3::TN];
    zero_acc(acc);
    uint4 fe[C3::TM], fo[C3::TM];
    ksteps_ct<T, C3::TM, C3::TN, P2, W2 / KS>(X2 + (wm * C3::TM * 16 + rl) * S2 + (lane >> 4) * 16,
                                              16 * S2, br2, acc, fe, fo);
    if (BWD)
      br3.init(static_cast<const T*>(a.W2T) + (size_t)slot * W2 * W3, (wv % C2::WN) * C2::TN,
               C2::NT, W3, lane);
#pragma unroll
    for (int i = 0; i < C3::TM; ++i) {
      const int r = wm * C3::TM * 16 + i * 16 + rl;
      float ep[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < C3::TN; ++j) {
        const int ct = wn * C3::TN + j;
        if (C3::even || ct < C3::NT) {  // wave-uniform
          const int c = ct * 16 + cq;
          const float bb[4] = {b[j].x, b[j].y, b[j].z, b[j].w};
          const float ww[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
          float h[4], d[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float z = acc[i][j][e] + bb[e];
            const float ex = __builtin_amdgcn_exp2f(fminf(z, 0.f) * ial2e);
            const float neg = alpha * (ex - 1.f);
            h[e] = z > 0.f ? z : neg;
            d[e] = up[i] * ww[e] * (z > 0.f ? 1.f : ex);
            float& sum = ep[HEAD ? e : 0];
            if (!C3::spread) sum = __builtin_fmaf(ww[e], h[e], sum);
          }
          const float4 h4 = make_float4(h[0], h[1], h[2], h[3]);
          const float4 d4 = make_float4(d[0], d[1], d[2], d[3]);
          if (BWD) LdsV<T>::put(D3s + r * S3 + c * ES, d4);
          if (C3::spread)
            *reinterpret_cast<float4*>(reinterpret_cast<unsigned char*>(epart) + r * LL::SH + c * 4) =
                h4;
          if (STORE) {
            Store<T>::put4(static_cast<T*>(a.H3) + (size_t)rrow(r) * W3 + c, h4);
            Store<T>::put4(static_cast<T*>(a.D3) + (size_t)rrow(r) * W3 + c, d4);
          }
        }
        if (BWD) br3.template fetch_share<W3 / KS, C3::TM * C3::TN>(i * C3::TN + j);
      }
      if (STORE && wn == 0 && lane < 16) a.uprow[rrow(r)] = row0 + r < row_end ? up[i] : 0.f;
      if constexpr (!C3::spread) {
        float e = HEAD ? (ep[0] + ep[1]) + (ep[2] + ep[3]) : ep[0];
        e += __shfl_xor(e, 16, 64);
        e += __shfl_xor(e, 32, 64);
        if (lane < 16) epart[wn * BM + r] = e;
      }
    }
  }
  __syncthreads();
  if (erow_on) {
    float e = a.bout[slot];
    if constexpr (C3::spread) {
      // 16 lanes per row: column c of 16 of each half, in either order
      const unsigned char* hrow = reinterpret_cast<unsigned char*>(epart) + erow_r * LL::SH;
      const float* wo = a.wout + (size_t)slot * W3;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float v = 0.f;
        if constexpr (HEAD) {
#pragma unroll
          for (int j = 0; j < W3 / 32; ++j) {
            const int c = q * (W3 / 2) + j * 16 + rl;
            v = __builtin_fmaf(wo[c], *reinterpret_cast<const float*>(hrow + c * 4), v);
          }
          v = group16_sum(v);
        } else {
          // lanes 4 g' hold the sums of lane groups g' (others repeat them)
          const int g4 = (rl & 3) * 4;
#pragma unroll
          for (int j = 0; j < W3 / 32; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int c = q * (W3 / 2) + j * 16 + g4 + k;
              v = __builtin_fmaf(wo[c], *reinterpret_cast<const float*>(hrow + c * 4), v);
            }
          v += dpp_get<0xb1>(v);  // groups g and g ^ 1, then g ^ 2
          v += dpp_get<0x4e>(v);
        }
        e += v;
      }
      if (rl == 0 && eatom >= 0) a.erow[(size_t)member * a.erow_stride + eatom] = e;
    } else {
#pragma unroll
      for (int q = 0; q < C3::WN; ++q) e += epart[q * BM + tid];
      if (eatom >= 0) a.erow[(size_t)member * a.erow_stride + eatom] = e;
    }
  }
  if constexpr (!BWD) return;

  // ---- D2 = (D3 W2) * CELU'(z2), over H2
  NetRing<T, C1::TN, P2, C1::even> br4;  // adjoint of layer 2 (K = W2)
  {
    const int wm = wv / C2::WN, wn = wv % C2::WN;
    f32x4_t acc[C2::TM][C2::TN];
    zero_acc(acc);
    uint4 fe[C2::TM], fo[C2::TM];
    ksteps_ct<T, C2::TM, C2::TN, P3, W3 / KS>(
        D3s + (wm * C2::TM * 16 + rl) * S3 + (lane >> 4) * 16, 16 * S3, br3, acc, fe, fo);
    br4.init(static_cast<const T*>(a.W1T) + (size_t)slot * W1 * W2, (wv % C1::WN) * C1::TN, C1::NT,
             W2, lane);
#pragma unroll
    for (int i = 0; i < C2::TM; ++i) {
      const int r = wm * C2::TM * 16 + i * 16 + rl;
#pragma unroll
      for (int j = 0; j < C2::TN; ++j) {
        const int ct = wn * C2::TN + j;
        if (C2::even || ct < C2::NT) {  // wave-uniform
          const int c = ct * 16 + cq;
          const float4 h = LdsV<T>::get(X2 + r * S2 + c * ES);
          const float4 d =
              make_float4(acc[i][j][0] * celu_slope(h.x, ia), acc[i][j][1] * celu_slope(h.y, ia),
                          acc[i][j][2] * celu_slope(h.z, ia), acc[i][j][3] * celu_slope(h.w, ia));
          LdsV<T>::put(X2 + r * S2 + c * ES, d);
          if (STORE) Store<T>::put4(static_cast<T*>(a.D2) + (size_t)rrow(r) * W2 + c, d);
        }
        br4.template fetch_share<W2 / KS, C2::TM * C2::TN>(i * C2::TN + j);
      }
    }
  }
  __syncthreads();

  // dE/dG runs over the active k-steps, one (two 16-column tiles) per wave
  // and pass: wave w takes positions w, w + GN, ...  FP32, whose products and
  // not its weights bound it, takes 16 rows of a k-step at a time, so that few
  // k-steps spread over the waves (4,500 atoms of water, 27.6 -> 26.6 us)
  constexpr int GN = kNetWaves, GM = sizeof(T) == 4 ? 1 : BM / 16, GU = BM / 16 / GM;
  const T* W0T = static_cast<const T*>(a.W0T) + (size_t)slot * K * W1;
  auto qat = [&](int pos) -> int {
    return __builtin_amdgcn_readlane(qlist, pos < nact ? pos : (nact > 0 ? nact - 1 : 0));
  };
  NetRing<T, 2, P1, true> br5;  // (K = W1)

  // ---- D1 = (D2 W1) * CELU'(z1), over H1
  {
    const int wm = wv / C1::WN, wn = wv % C1::WN;
    f32x4_t acc[C1::TM][C1::TN];
    zero_acc(acc);
    uint4 fe[C1::TM], fo[C1::TM];
    ksteps_ct<T, C1::TM, C1::TN, P2, W2 / KS>(X2 + (wm * C1::TM * 16 + rl) * S2 + (lane >> 4) * 16,
                                              16 * S2, br4, acc, fe, fo);
    if (a.G) br5.init(W0T, 2 * qat(wv / GU), K / 16, W1, lane);
#pragma unroll
    for (int i = 0; i < C1::TM; ++i) {
      const int r = wm * C1::TM * 16 + i * 16 + rl;
#pragma unroll
      for (int j = 0; j < C1::TN; ++j) {
        const int ct = wn * C1::TN + j;
        if (C1::even || ct < C1::NT) {  // wave-uniform
          const int c = ct * 16 + cq;
          const float4 h = LdsV<T>::get(X1 + r * S1 + c * ES);
          const float4 d =
              make_float4(acc[i][j][0] * celu_slope(h.x, ia), acc[i][j][1] * celu_slope(h.y, ia),
                          acc[i][j][2] * celu_slope(h.z, ia), acc[i][j][3] * celu_slope(h.w, ia));
          LdsV<T>::put(X1 + r * S1 + c * ES, d);
          if (STORE || a.D1)
            Store<T>::put4(static_cast<T*>(a.D1) + (size_t)(STORE ? rrow(r) : row0 + r) * a.ld_d1 +
                               member * W1 + c, d);
        }
        if (a.G) br5.template fetch_share<W1 / KS, C1::TM * C1::TN>(i * C1::TN + j);
      }
    }
  }
  if (!a.G) return;  // block-uniform: no dE/dG asked for here
  __syncthreads();   // D1 in X1

  // ---- dE/dG, each row on its own k-steps
  for (int p = wv; p < nact * GU; p += GN) {
    const int q = qat(p / GU), r0 = p % GU * GM * 16;
    f32x4_t acc[GM][2];
    zero_acc(acc);
    uint4 fe[GM], fo[GM];
    ksteps_ct<T, GM, 2, P1, W1 / KS>(X1 + (r0 + rl) * S1 + (lane >> 4) * 16, 16 * S1,
                                     br5, acc, fe, fo);
    br5.init(W0T, 2 * qat((p + GN) / GU), K / 16, W1, lane);
    if (p + GN < nact * GU) br5.template fetch_share<W1 / KS, 1>(0);
#pragma unroll
    for (int i = 0; i < GM; ++i) {
      const int r = r0 + i * 16 + rl;
      if (row0 + r < row_end && ((rmask[r] >> q) & 1ull)) {
        T* g = static_cast<T*>(a.G) + (size_t)rrow(r) * K + q * 32 + cq;
#pragma unroll
        for (int j = 0; j < 2; ++j)
          Store<T>::put4(g + j * 16,
                         make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]));
      }
    }
  }
}

template <typename T, int W1, int W2, int W3, int BM, bool BWD, bool STORE>
static void launch_net_t(const NetArgs& a, int rows_cap, int members, hipStream_t st) {
  constexpr size_t lds = NetLds<T, W1, W2, W3, BM>::bytes;
  auto kern = k_mlp_net<T, W1, W2, W3, BM, BWD, STORE>;
  static const bool attr = (ensure_lds(kern), true);
  (void)attr;
  hipLaunchKernelGGL(kern, dim3(rows_cap / BM, members), dim3(64 * kNetWaves), lds, st, a);
}

template <typename T, int W1, int W2, int W3, int BM>
static void launch_net_m(const NetArgs& a, int rows_cap, int members, hipStream_t st) {
  if (!a.bwd)
    launch_net_t<T, W1, W2, W3, BM, false, false>(a, rows_cap, members, st);
  else if (!a.H1)
    launch_net_t<T, W1, W2, W3, BM, true, false>(a, rows_cap, members, st);
  else
    launch_net_t<T, W1, W2, W3, BM, true, true>(a, rows_cap, members, st);
}

template <typename T, int W1, int W2, int W3>
static void launch_net_w(const NetArgs& a, int n_rows, int rows_cap, int members, hipStream_t st) {
  switch (net_tile<T>(n_rows, members, a.order != nullptr)) {
    case 16: launch_net_m<T, W1, W2, W3, 16>(a, rows_cap, members, st); return;
    case 32: launch_net_m<T, W1, W2, W3, 32>(a, rows_cap, members, st); return;
    default:
      if constexpr (sizeof(T) == 2) launch_net_m<T, W1, W2, W3, 64>(a, rows_cap, members, st);
  }
}

}  // namespace nnp
