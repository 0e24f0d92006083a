// Chunked prefill of the shared post-prefill state S_ctx (Sec. 3.1) on gfx950:
// Eq. 1 (Sec. 2.2) over a prompt, from S = 0, in chunks of C = 64 tokens.
//
// Inside a chunk that starts from state S_0, write Eq. 1 with the paper's
// correction term (Eq. 2), delta_t = beta_t (v_t - alpha_t S_{t-1} k_t), as
// S_t = alpha_t S_{t-1} + delta_t k_t^T.  Unrolling it with
// Gamma(t, i) = alpha_{i+1} ... alpha_t and gamma_t = Gamma(t, -1):
//   S_t     = gamma_t S_0 + sum_{i<=t} Gamma(t, i) delta_i k_i^T
//   delta_t = beta_t v_t - beta_t gamma_t S_0 k_t
//             - sum_{i<t} beta_t Gamma(t, i) (k_t . k_i) delta_i.
// With M the strictly lower C x C matrix M(t, i) = beta_t Gamma(t, i) (k_t.k_i)
// and T = (I + M)^{-1} (unit lower triangular), the deltas of the chunk are
//   D = T diag(beta) (V - diag(gamma) K S_0^T),
// and the state after the chunk is
//   S_C = g S_0 + D^T diag(sigma) K,   sigma_t = Gamma(C - 1, t),  g = gamma_{C-1},
// that is, with T' = diag(sigma) T diag(beta) and D' = T' (V - diag(gamma) K S_0^T),
//   S_C = g S_0 + D'^T K.
//
// bf16 keys and values (exact in one bf16 part each, so the products with
// fp32 factors split into three bf16 parts are exact):
//   prefill_factor_kernel: one workgroup per (request, value head, chunk)
//     forms gamma and T' (split in three parts) and stores only those;
//   prefill_scan_kernel: walks the chunks from the raw keys and values, 128 state
//     rows per workgroup, the prompt cut into segments that run at once
//     where the chip would otherwise be idle;
//   prefill_combine_kernel: chains the segments (only with more than one).
// Measured (one MI355X, 16 heads, d = 128; the launches by rocprofv3): 4096 tokens
// factors 13 us, scan 41, combination 11, against 57 + 98 for the two launches of the
// form below; 16 requests x 1000 tokens 36 + 78 against 229 + 207.
//
// fp32 keys and values:
//   prefill_chunk_kernel: one workgroup per (request, value head, chunk) forms T
//     by forward substitution (each column held in registers by a quad of
//     lanes), then W' = T' diag(gamma) K and U' = T' V, and stores W', K^T, U'^T
//     and g in the order the scan's lanes load them;
//   prefill_scan_f32_kernel: one workgroup per (request, value head, 16 state
//     rows) walks the chunks in order: X^T = W' S^T, D'^T = U'^T - X^T,
//     S^T <- g S^T + K^T D'^T, on v_mfma_f32_16x16x4f32.  Wave w owns the state
//     columns 16 w .. 16 w + 15 (a 16 x 16 fp32 accumulator tile that never
//     leaves registers); the contraction orders are chosen so that the tile is
//     directly the B operand of the next chunk's X and X's output is directly
//     the B operand of the update.  The partial X of the d_k / 16 waves are
//     summed through LDS, each token tile by d_k / 64 waves that take a share
//     of its accumulator components.
//
// No division: products of alpha are formed directly, so alpha = 0 is exact.  A
// ragged last chunk is padded with alpha = 1, beta = 0, k = v = 0, which leaves
// the state unchanged.
#include "device_common.h"
#include "internal.h"

namespace onela {
namespace {

constexpr int kC = kPrefillChunk;  // tokens per chunk
constexpr int kP1Threads = 256;

struct PrefillParams {
  const void* k;      // [R][P][HK][DK] io dtype
  const void* v;      // [R][P][HV][DV] io dtype
  const float* alpha; // [R][P][HV]
  const float* beta;
  float* s_out;       // [R][HV][DV][DK]
  // fp32 keys: per (request, value head, chunk), in phase 2's fragment order
  float* wb;          // [R*HV][nch][DK/16][4][64] f32x4   W' = diag(sigma) W
  float* ktb;         // [R*HV][nch][DK/16][4][64] f32x4   K^T
  float* utb;         // [R*HV][nch][DV/16][4][64] f32x4   U'^T = (diag(sigma) U)^T
  float* gb;          // [R*HV][nch][16]  g, repeated (phase 2 loads it per lane)
  // bf16 keys: per (request, value head, chunk) the factors of the scan
  uint4* tf;          // [R*HV][nch][6][3][64]  T' fragments, three bf16 parts each
  float* gam;         // [R*HV][nch][64]  gamma_t
  float* segb;        // [R*HV][nseg][DV][DK]  (nseg > 1)
  uint4* sega;        // [R*HV][nseg - 1][DK/16][DK/32][3][64]  A^T fragments, split
  int nseg, cps;      // segments of the scan, chunks per segment
  int HK, HV, P, nch;
  int xcd_map;  // phase 2: all row blocks of a unit on one XCD (units % 8 == 0)
};

// 8 consecutive fp32 elements at element i.
struct Io8 {
  uint4 u[2];
  __device__ void load(const void* base, long i) {
    const uint4* q = reinterpret_cast<const uint4*>(static_cast<const float*>(base) + i);
    u[0] = q[0];
    u[1] = q[1];
  }
  __device__ float get(int e) const { return __uint_as_float((&u[e >> 2].x)[e & 3]); }
};

// Fills dst[t][c] (t < kC, c < NCOL, row stride LD) from rows of an fp32
// array (row t at element row0(t) + c0, zero for t >= n), scaled by
// scale(t).  Every thread issues all of its loads before its first store.
template <int NCOL, int LD, typename RowFn, typename ScaleFn>
__device__ inline void fill_rows(float* dst, const void* src, int n, int c0, RowFn&& row0,
                                 ScaleFn&& scale) {
  constexpr int NV = kC * NCOL / 8;  // 8-element vectors
  constexpr int PER = (NV + kP1Threads - 1) / kP1Threads;
  Io8 buf[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int vi = threadIdx.x + q * kP1Threads;
    const int t = vi / (NCOL / 8), c = (vi - t * (NCOL / 8)) * 8;
    if (vi < NV && t < n) buf[q].load(src, row0(t) + c0 + c);
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int vi = threadIdx.x + q * kP1Threads;
    const int t = vi / (NCOL / 8), c = (vi - t * (NCOL / 8)) * 8;
    if (vi < NV) {
      const float sc = t < n ? scale(t) : 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[t * LD + c + e] = t < n ? sc * buf[q].get(e) : 0.f;
    }
  }
}

// ---- fp32 keys, phase 1 -------------------------------------------------------

// Rows are padded to a multiple of 4 words plus 4, so that the 16 rows x 4
// columns an MFMA operand read touches fall in distinct banks.
template <int DK>
struct P1Shared {
  static constexpr int KLD = DK + 4;
  float K[kC][KLD];       // the chunk's keys (padding rows zero)
  float T[kC][kC + 4];    // (I + M)^{-1}
  union {
    float M[kC][kC + 4];  // until T is formed
    float X[kC][128 + 4]; // then beta V (d_v <= 128)
  };
  float P[7][kC];         // P[k][t]: product of the 2^k decays ending at token t
  alignas(16) float be[kC], gam[kC], sig[kC];
};

// alpha_{i+1} ... alpha_t (t - i >= 0 factors; none: 1) from the doubling
// table, in blocks of 2^k decays, largest first.  Products only, so a zero
// decay gives an exact zero.
__device__ inline float decay(const float (&P)[7][kC], int t, int i) {
  float g = 1.f;
  int pos = t;
  const int L = t - i;
#pragma unroll
  for (int k = 6; k >= 0; --k)
    if ((L >> k) & 1) {
      g *= P[k][pos];
      pos -= 1 << k;
    }
  return g;
}

// Sum over the 4 lanes of a quad.
__device__ inline float quad_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1,
                                                             0xF, 0xF, false));  // [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E,
                                                             0xF, 0xF, false));  // [2,3,0,1]
  return x;
}

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The products of phase 1 run on v_mfma_f32_16x16x4f32 in 16 x 16 tiles: for
// D = A B, lane l supplies A(l % 16, k) and B(k, l % 16) with k = l / 16 of
// each 4-deep step and holds D(4 (l / 16) + r, l % 16), r = 0..3.
template <int DK, int DV>
__global__ __launch_bounds__(kP1Threads) void prefill_chunk_kernel(PrefillParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  using Sh = P1Shared<DK>;
  Sh& sh = *reinterpret_cast<Sh*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int c = blockIdx.x % p.nch, unit = blockIdx.x / p.nch;
  const int r = unit / p.HV, hv = unit - r * p.HV, hk = hv / (p.HV / p.HK);
  const int t0 = c * kC;
  const int n = min(kC, p.P - t0);
  const long tok0 = long(r) * p.P + t0;

  fill_rows<DK, Sh::KLD>(&sh.K[0][0], p.k, n, 0,
                                [&](int t) { return ((tok0 + t) * p.HK + hk) * DK; },
                                [](int) { return 1.f; });
  if (tid < kC) {
    const bool in = tid < n;
    const float al = in ? p.alpha[(tok0 + tid) * p.HV + hv] : 1.f;
    sh.be[tid] = in ? p.beta[(tok0 + tid) * p.HV + hv] : 0.f;
    // doubling table of decay products (lane t of wave 0 holds token t)
    float v = al;
    sh.P[0][tid] = v;
#pragma unroll
    for (int k = 1; k < 7; ++k) {
      const float u = __shfl_up(v, 1 << (k - 1));
      if (tid >= (1 << (k - 1))) v *= u;
      sh.P[k][tid] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // gamma_t = alpha_0 ... alpha_t; sigma_t = alpha_{t+1} ... alpha_{C-1}
    sh.gam[tid] = decay(sh.P, tid, -1);
    sh.sig[tid] = decay(sh.P, kC - 1, tid);
  }
  // M is zero above its diagonal 16 x 16 tiles (the product below fills the
  // rest)
  for (int e = tid; e < kC * kC; e += kP1Threads) {
    const int t = e / kC, i = e - t * kC;
    if ((i >> 4) > (t >> 4)) sh.M[t][i] = 0.f;
  }
  __syncthreads();
  // M(t, i) = beta_t Gamma(t, i) (k_t . k_i) for i < t, 0 for i >= t: the ten
  // tiles on or below the diagonal of K K^T
  for (int x = w; x < 10; x += 4) {
    const int a = (x >= 1) + (x >= 3) + (x >= 6), b = x - a * (a + 1) / 2;
    f32x4 acc4[4] = {};  // four independent chains over the key dimension
#pragma unroll 8
    for (int ks = 0; ks < DK / 4; ++ks)
      acc4[ks & 3] = mfma4(sh.K[16 * a + l16][4 * ks + l4], sh.K[16 * b + l16][4 * ks + l4],
                           acc4[ks & 3]);
    const f32x4 acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = 16 * a + 4 * l4 + q, i = 16 * b + l16;
      const float g = decay(sh.P, t, i < t ? i : t);  // (no factor on or above the diagonal)
      sh.M[t][i] = i < t ? sh.be[t] * g * acc[q] : 0.f;
    }
  }
  __syncthreads();
  // T = (I + M)^{-1} by forward substitution, T(t, j) = -sum_{i<t} M(t, i)
  // T(i, j) for t > j: column j = 16 w + lane / 4 is held in registers by the
  // quad of lanes 4 (j % 16) .. + 3, lane sub summing the rows i = sub mod 4
  {
    const int j = 16 * w + (lane >> 2), sub = lane & 3;
    float x[kC / 4];
#pragma unroll
    for (int m = 0; m < kC / 4; ++m) x[m] = 0.f;
#pragma unroll
    for (int t = 0; t < kC; ++t) {
      float sp[4] = {0.f, 0.f, 0.f, 0.f};  // rows not computed yet hold 0
#pragma unroll
      for (int m = 0; m < (t + 3) / 4; ++m) sp[m & 3] = fmaf(sh.M[t][sub + 4 * m], x[m], sp[m & 3]);
      const float s = quad_sum((sp[0] + sp[1]) + (sp[2] + sp[3]));
      const float val = t == j ? 1.f : (t > j ? -s : 0.f);
      if (sub == (t & 3)) x[t >> 2] = val;
    }
#pragma unroll
    for (int m = 0; m < kC / 4; ++m) sh.T[sub + 4 * m][j] = x[m];
  }
  __syncthreads();

  const long cu = long(unit) * p.nch + c;
  // The three operands of phase 2 are stored in the order its lanes load them
  // (16 bytes per lane, 1 KB per wave and fragment).  K^T: fragment (column
  // block b, token tile a) of lane l holds K(t = 16 a + 4 (l / 16) + j,
  // k = 16 b + l % 16), j = 0..3
  f32x4* kdst = reinterpret_cast<f32x4*>(p.ktb + cu * DK * kC);
  for (int e = tid; e < DK / 16 * 4 * 64; e += kP1Threads) {
    const int l = e & 63, a = (e >> 6) & 3, b = e >> 8;
    const int kk = 16 * b + (l & 15), t = 16 * a + 4 * (l >> 4);
    kdst[e] = f32x4{sh.K[t][kk], sh.K[t + 1][kk], sh.K[t + 2][kk], sh.K[t + 3][kk]};
  }
  // W' = diag(sigma) T diag(beta gamma) K, formed transposed so that a lane
  // holds 4 consecutive keys of one token: fragment (b, a) of lane l holds
  // W'(t = 16 a + l % 16, k = 16 b + 4 (l / 16) + i), i = 0..3
  f32x4* wdst = reinterpret_cast<f32x4*>(p.wb + cu * kC * DK);
  // (T is lower triangular: row block a needs k < 16 (a + 1))
  constexpr int NBW = DK / 16;
  for (int x = w; x < 4 * NBW; x += 4) {
    const int a = x / NBW, b = x - a * NBW;
    f32x4 acc4[4] = {};
    for (int ks = 0; ks < 4 * (a + 1); ks += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kk = 4 * (ks + u) + l4;
        acc4[u] = mfma4(sh.be[kk] * sh.gam[kk] * sh.K[kk][16 * b + l16], sh.T[16 * a + l16][kk],
                        acc4[u]);
      }
    }
    const f32x4 acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
    wdst[(b * 4 + a) * 64 + lane] = sh.sig[16 * a + l16] * acc;
  }
  // U' = diag(sigma) T diag(beta) V, as U'^T fragments: fragment (row block rb,
  // token tile a) of lane l holds U'^T(16 rb + l % 16, t = 16 a + 4 (l / 16) + j),
  // j = 0..3
  f32x4* udst = reinterpret_cast<f32x4*>(p.utb + cu * DV * kC);
  static_assert(DV <= 128, "beta V takes M's place in one piece");
  constexpr int NBU = DV / 16;
  fill_rows<DV, 128 + 4>(&sh.X[0][0], p.v, n, 0,
                         [&](int t) { return ((tok0 + t) * p.HV + hv) * DV; },
                         [&](int t) { return sh.be[t]; });
  __syncthreads();
  for (int x = w; x < 4 * NBU; x += 4) {
    const int a = x / NBU, b = x - a * NBU;
    f32x4 acc4[4] = {};
    for (int ks = 0; ks < 4 * (a + 1); ks += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kk = 4 * (ks + u) + l4;
        acc4[u] = mfma4(sh.T[16 * a + l16][kk], sh.X[kk][16 * b + l16], acc4[u]);
      }
    }
    const f32x4 acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
    const f32x4 sg = *reinterpret_cast<const f32x4*>(&sh.sig[16 * a + 4 * l4]);
    udst[(b * 4 + a) * 64 + lane] = sg * acc;
  }
  if (tid < 16) p.gb[cu * 16 + tid] = sh.gam[kC - 1];
}

// ---- fp32 keys, phase 2 -------------------------------------------------------

// Operands of one chunk for one lane, loaded from the workspace's fragment order.
template <int NU>
struct ScanOps {
  f32x4 w[4], k[4], u[NU];
  float g;
};

template <int N>
struct Vec {
  typedef float type __attribute__((ext_vector_type(N)));
};

// Components N g .. N g + N - 1 of v.
template <int N>
__device__ inline typename Vec<N>::type slice(const f32x4& v, int g) {
  static_assert(N == 4 || N == 2, "d_k <= 128");
  if constexpr (N == 4) {
    return v;
  } else {
    return g == 0 ? v.xy : v.zw;
  }
}

template <int DK, int DV>
__global__ __launch_bounds__(4 * DK) void prefill_scan_f32_kernel(PrefillParams p) {
  constexpr int NW = DK / 16;  // waves: state columns 16 w .. 16 w + 15
  // The NW partial X^T of a token tile are summed by NW / 4 waves, each taking
  // NCP of the 4 accumulator components a lane holds (with fewer than 4 waves
  // a wave sums TPW whole tiles).
  constexpr int TPW = NW >= 4 ? 1 : 4 / NW;
  constexpr int NCP = NW >= 4 ? 16 / NW : 4;
  constexpr int NG = 4 / NCP;
  using VN = typename Vec<NCP>::type;
  __shared__ VN xp[NW][4][NG][64];  // partial X^T tiles of every wave, by component group
  __shared__ f32x4 ds[4][64];       // D'^T tiles: U'^T minus the sums of the partials
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // The DV / 16 row blocks of a (request, value head) read the same W and
  // Kt of every chunk.  Workgroups are dispatched round-robin over the 8
  // XCDs (block i on XCD i % 8), so when the unit count is a multiple of 8
  // all row blocks of a unit are placed on one XCD and share its L2.
  constexpr int NRB = DV / 16;
  int rb, unit;
  if (p.xcd_map) {
    const int x = blockIdx.x & 7, slot = blockIdx.x >> 3;
    unit = x + 8 * (slot / NRB);
    rb = slot % NRB;
  } else {
    rb = blockIdx.x % NRB;
    unit = blockIdx.x / NRB;
  }
  const int row0 = 16 * rb;
  const int lr = lane & 15, lq = lane >> 4;
  // st[i] = S^T(k = 16 w + 4 lq + i, n = lr) = S(row0 + lr, 16 w + 4 lq + i)
  f32x4 st = {0.f, 0.f, 0.f, 0.f};
  float* dst = p.s_out + (long(unit) * DV + row0 + lr) * DK + 16 * w + 4 * lq;
  if (p.nch == 0) {  // empty prompt: S = 0, and there is no chunk to read
    *reinterpret_cast<f32x4*>(dst) = st;
    return;
  }
  // the token tiles whose D' this wave forms, and its component group
  const int g0 = NW >= 4 ? w >> 2 : 0;
  auto tile = [&](int i) { return NW >= 4 ? (w & 3) : w + NW * i; };
  // Loads are unconditional (past the end they re-read the last chunk) so
  // the compiler can count them and wait only for the set about to be used.
  // Every load is one lane's 16 bytes of a fragment stored contiguously by
  // phase 1, so a wave reads whole 1 KB blocks.
  auto load = [&](int c, ScanOps<TPW>& o) {
    const long cu = long(unit) * p.nch + (c < p.nch ? c : p.nch - 1);
    const f32x4* wc = reinterpret_cast<const f32x4*>(p.wb + cu * kC * DK);
    const f32x4* ut = reinterpret_cast<const f32x4*>(p.utb + cu * DV * kC);
    // g through the vector memory path (16 copies, one per lane of a row):
    // a scalar load would be waited for by the step's first LDS wait
    o.g = p.gb[cu * 16 + lr];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) o.w[mt] = wc[(w * 4 + mt) * 64 + lane];
    const f32x4* kt = reinterpret_cast<const f32x4*>(p.ktb + cu * DK * kC);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) o.k[mt] = kt[(w * 4 + mt) * 64 + lane];
#pragma unroll
    for (int i = 0; i < TPW; ++i) o.u[i] = ut[(rb * 4 + tile(i)) * 64 + lane];
  };
  auto step = [&](int c, const ScanOps<TPW>& o) {
    if (c >= p.nch) return;
    // partial X^T(t, n) over this wave's 16 state columns: four independent
    // accumulator chains, one per token tile
    f32x4 xa[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) xa[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
        xa[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.w[mt][i], st[i], xa[mt], 0, 0, 0);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int g = 0; g < NG; ++g) xp[w][mt][g][lane] = slice<NCP>(xa[mt], g);
    __syncthreads();
    // D'^T(t = 16 mt + 4 lq + j, n = lr) = U'^T - sum over the waves of X^T,
    // components NCP g0 .. of the tiles this wave forms
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int mt = tile(i);
      VN x = xp[0][mt][g0][lane];
#pragma unroll
      for (int v = 1; v < NW; ++v) x += xp[v][mt][g0][lane];
      *reinterpret_cast<VN*>(reinterpret_cast<float*>(&ds[mt][lane]) + NCP * g0) =
          slice<NCP>(o.u[i], g0) - x;
    }
    __syncthreads();
    // S^T <- g S^T + K^T D'^T
    // one fp32 chain per token tile, summed
    f32x4 up[4], dd[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      dd[mt] = ds[mt][lane];
      up[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
        up[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.k[mt][j], dd[mt][j], up[mt], 0, 0, 0);
    st = o.g * st + ((up[0] + up[1]) + (up[2] + up[3]));
  };
  // three operand sets in flight: chunk c + 2 is requested before chunk c is
  // processed.  (xp and ds are rewritten only after the next chunk's first
  // barrier, which every wave reaches after reading them.)  The scheduling
  // barriers keep every load group in program order, so the wait before a
  // step covers only its own (oldest) group.
  ScanOps<TPW> a, b, c3;
  load(0, a);
  __builtin_amdgcn_sched_barrier(0);
  load(1, b);
  for (int c = 0; c < p.nch; c += 3) {
    __builtin_amdgcn_sched_barrier(0);
    load(c + 2, c3);
    __builtin_amdgcn_sched_barrier(0);
    step(c, a);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 3, a);
    __builtin_amdgcn_sched_barrier(0);
    step(c + 1, b);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 4, b);
    __builtin_amdgcn_sched_barrier(0);
    step(c + 2, c3);
  }
  *reinterpret_cast<f32x4*>(dst) = st;
}

// ---- bf16 keys: factors of the chunks, then the scan over them ------------------

// x = hi + mid + lo (8 floats, three bf16 vectors; exact for normal x).
__device__ inline void split3(const float* x, uint4& hi, uint4& mid, uint4& lo) {
  unsigned h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
    const float r0 = x[2 * i] - bf16_lo_to_float(h[i]);
    const float r1 = x[2 * i + 1] - bf16_hi_to_float(h[i]);
    m[i] = pack_bf16x2(r0, r1);
    l[i] = pack_bf16x2(r0 - bf16_lo_to_float(m[i]), r1 - bf16_hi_to_float(m[i]));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  mid = make_uint4(m[0], m[1], m[2], m[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

__device__ inline void split3(const f32x4& x0, const f32x4& x1, uint4& hi, uint4& mid, uint4& lo) {
  const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
  split3(x, hi, mid, lo);
}

// x = hi + mid + lo exactly by truncation (8 of the 24 significant bits each),
// for products that use all three parts.  Byte permutes and masks in place of
// the conversions.
__device__ inline void cut3(const f32x4& x0, const f32x4& x1, uint4& hi, uint4& mid, uint4& lo) {
  const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
  unsigned h[4], m[4], l[4];
  auto top2 = [](float a, float b) {  // the upper halves, a's in the low half
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  };
  auto top = [](float a) { return __uint_as_float(__float_as_uint(a) & 0xffff0000u); };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = x[2 * i], b = x[2 * i + 1];
    const float a1 = a - top(a), b1 = b - top(b);
    h[i] = top2(a, b);
    m[i] = top2(a1, b1);
    l[i] = top2(a1 - top(a1), b1 - top(b1));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  mid = make_uint4(m[0], m[1], m[2], m[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// 16 bytes on their way through registers, as a native vector: arrays of the
// header's uint4 (a class) that are moved under a condition stay in memory
// (scratch, or LDS that the compiler adds).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ inline u32x4 keep(u32x4 v, bool in) {
  return in ? v : u32x4{0u, 0u, 0u, 0u};
}

// Fragment f of T' = diag(sigma) T diag(beta) covers the tokens (row tile) kTfRow[f] x
// (32-token column step) kTfStep[f]; the blocks above the diagonal are not stored.
constexpr int kTFrags = 6;
constexpr int kTChunk = kTFrags * 3 * 64;  // 16-byte pieces of one chunk's T'

template <int DK>
struct FactorShared {
  union {
    uint16_t K[kC][DK + 8];  // the chunk's keys (padding rows zero)
    float T[kC][kC + 4];     // then (I + M)^{-1}
  };
  float M[kC][kC + 4];  // M; the diagonal 16 x 16 blocks then hold those of (I + M)^{-1}
  alignas(16) float al[kC], be[kC], pre[kC], suf[kC], sig[kC];
};

// x of the lane N places back (forward) in the row of 16 lanes; 1 past its end.
template <int CTRL>
__device__ inline float row_shift1(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, 1.f),
                                                               __builtin_bit_cast(int, x), CTRL,
                                                               0xF, 0xF, false));
}

// Factors of one 64-token chunk of one (request, value head): the decays gamma_t
// and T' = diag(sigma) (I + M)^{-1} diag(beta), split into three bf16 parts, in
// the order the scan's lanes load it as an MFMA A operand.  Four waves.
//   Bound: latency of its serial steps (one dependent chain per chunk); the
// workgroup holds 36 KB of LDS up to d_k = 128, so four of them share a compute
// unit (52 KB and three at 256) and hide each other's chain.  The inverse is formed by 16-token blocks:
// the four diagonal blocks by forward substitution, one per wave with a column
// per lane (16 dependent steps instead of 64), then each wave the blocks below
// the diagonal block of its block column, T_ij = -T_ii sum_k M_ik T_kj, on
// v_mfma_f32_16x16x4f32 with T_kj kept in the accumulator layout (its component
// s is the B operand of the steps s, 4 lq + s).  Decay products are formed in
// registers without a branch: within a 16-token block by DPP scans and, for
// the diagonal tiles, down the tile's rows (looked up in a table of doubled
// products, each waited for by itself, the launch took 51 us at 16 x 16 heads x 16 chunks).
template <int DK>
__global__ __launch_bounds__(kP1Threads, DK == 256 ? 3 : 4) void prefill_factor_kernel(PrefillParams p) {
  using Sh = FactorShared<DK>;
  __shared__ __align__(16) Sh sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int c = blockIdx.x % p.nch, unit = blockIdx.x / p.nch;
  const int r = unit / p.HV, hv = unit - r * p.HV, hk = hv / (p.HV / p.HK);
  const int n = min(kC, p.P - c * kC);
  const long tok0 = long(r) * p.P + long(c) * kC;
  const long cu = long(unit) * p.nch + c;
  {  // raw 16-byte copies of the key rows (zero past the prompt)
    constexpr int PER = kC * DK / 8 / kP1Threads;
    u32x4 buf[PER];
    float al = 1.f, be = 0.f;
    if (w == 0) {  // lane t holds token t (alpha = 1, beta = 0 past the prompt)
      const long ti = (tok0 + min(lane, n - 1)) * p.HV + hv;
      al = p.alpha[ti];
      be = p.beta[ti];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int vi = tid + q * kP1Threads, t = vi / (DK / 8), cc = (vi - t * (DK / 8)) * 8;
      buf[q] = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(p.k) +
                                               ((tok0 + min(t, n - 1)) * p.HK + hk) * DK + cc);
    }
    if (w == 0) {
      al = lane < n ? al : 1.f;
      be = lane < n ? be : 0.f;
      // the decays of the token's 16-token block up to and including it, and
      // after it (products only, so a zero decay gives an exact zero)
      float pre = al;
      pre *= row_shift1<0x111>(pre);
      pre *= row_shift1<0x112>(pre);
      pre *= row_shift1<0x114>(pre);
      pre *= row_shift1<0x118>(pre);
      float suf = row_shift1<0x101>(al);
      suf *= row_shift1<0x101>(suf);
      suf *= row_shift1<0x102>(suf);
      suf *= row_shift1<0x104>(suf);
      suf *= row_shift1<0x108>(suf);
      auto block = [&](int b) {
        return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(pre), 16 * b + 15));
      };
      // gamma_t = alpha_0 ... alpha_t; sigma_t = alpha_{t+1} ... alpha_{C-1}
      const float p1 = block(0), p2 = p1 * block(1), p3 = p2 * block(2);
      const float s2 = block(3), s1 = s2 * block(2), s0 = s1 * block(1);
      p.gam[cu * kC + lane] = pre * (lq == 0 ? 1.f : lq == 1 ? p1 : lq == 2 ? p2 : p3);
      sh.sig[lane] = suf * (lq == 0 ? s0 : lq == 1 ? s1 : lq == 2 ? s2 : 1.f);
      sh.al[lane] = al;
      sh.be[lane] = be;
      sh.pre[lane] = pre;
      sh.suf[lane] = suf;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int vi = tid + q * kP1Threads, t = vi / (DK / 8), cc = (vi - t * (DK / 8)) * 8;
      *reinterpret_cast<u32x4*>(&sh.K[t][cc]) = keep(buf[q], t < n);
    }
  }
  __syncthreads();
  // M(t, i) = beta_t Gamma(t, i) (k_t . k_i) for i < t, from the tiles on and
  // below the diagonal of K K^T (exact products of bf16 keys)
  auto kk = [&](int a, int b) {
    f32x4 acc2[2] = {};
#pragma unroll
    for (int ks = 0; ks < DK / 32; ++ks)
      acc2[ks & 1] = mfma_bf16(*reinterpret_cast<const uint4*>(&sh.K[16 * a + lr][32 * ks + 8 * lq]),
                               *reinterpret_cast<const uint4*>(&sh.K[16 * b + lr][32 * ks + 8 * lq]),
                               acc2[ks & 1]);
    return acc2[0] + acc2[1];
  };
#pragma unroll
  for (int x = 0; x < 2; ++x) {  // (1, 0), (2, 0), (2, 1), (3, 0); (3, 1), (3, 2)
    if (x == 1 && w >= 2) break;
    const int a = x == 1 ? 3 : w == 0 ? 1 : w < 3 ? 2 : 3, b = x == 1 ? w + 1 : w == 2 ? 1 : 0;
    const f32x4 acc = kk(a, b);
    // Gamma(t, i): the rest of i's block, the blocks between, t's block up to t
    float mid = sh.suf[16 * b + lr];
    for (int m = b + 1; m < a; ++m) mid *= sh.pre[16 * m + 15];
    const f32x4 be = *reinterpret_cast<const f32x4*>(&sh.be[16 * a + 4 * lq]);
    const f32x4 pre = *reinterpret_cast<const f32x4*>(&sh.pre[16 * a + 4 * lq]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      sh.M[16 * a + 4 * lq + q][16 * b + lr] = be[q] * (pre[q] * mid) * acc[q];
  }
  // the diagonal block w, then column lr of its inverse in every lane of the column
  f32x4 tc[4];  // blocks (w + d, w) of T, rows 4 lq + component, column lr
  {
    const f32x4 acc = kk(w, w);
    const f32x4 be = *reinterpret_cast<const f32x4*>(&sh.be[16 * w + 4 * lq]);
    f32x4 gd = {0.f, 0.f, 0.f, 0.f};
    float g = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 al = *reinterpret_cast<const f32x4*>(&sh.al[16 * w + 4 * q]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // row 4 q + j: 0 on and above the diagonal
        const int t = 4 * q + j;
        g = lr == t - 1 ? al[j] : g * al[j];
        gd[j] = lq == q ? g : gd[j];
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      sh.M[16 * w + 4 * lq + q][16 * w + lr] = lr < 4 * lq + q ? be[q] * gd[q] * acc[q] : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float x[16];
    f32x4 m[16][4];
#pragma unroll
    for (int i = 1; i < 16; ++i)
#pragma unroll
      for (int q = 0; q < (i + 3) / 4; ++q)
        m[i][q] = *reinterpret_cast<const f32x4*>(&sh.M[16 * w + i][16 * w + 4 * q]);
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = i == lr ? 1.f : 0.f;
#pragma unroll
    for (int j = 0; j < 15; ++j)
#pragma unroll
      for (int i = j + 1; i < 16; ++i) x[i] = fmaf(-m[i][j >> 2][j & 3], x[j], x[i]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      tc[0][q] = lq == 0 ? x[q] : lq == 1 ? x[4 + q] : lq == 2 ? x[8 + q] : x[12 + q];
      sh.M[16 * w + 4 * lq + q][16 * w + lr] = tc[0][q];
    }
  }
  __syncthreads();  // (the keys are not read any more: T takes their place)
#pragma unroll
  for (int d = 1; d < 4; ++d) {
    if (w + d >= 4) break;
    const int i = w + d;
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
    for (int e = 0; e < d; ++e) {
      const f32x4 mm = *reinterpret_cast<const f32x4*>(&sh.M[16 * i + lr][16 * (w + e) + 4 * lq]);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        f32x4& acc = (s & 1) ? a1 : a0;
        acc = mfma4(mm[s], tc[e][s], acc);
      }
    }
    const f32x4 pr = a0 + a1;
    const f32x4 tt = *reinterpret_cast<const f32x4*>(&sh.M[16 * i + lr][16 * i + 4 * lq]);
    f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = b0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      f32x4& acc = (s & 1) ? b1 : b0;
      acc = mfma4(tt[s], pr[s], acc);
    }
    tc[d] = -(b0 + b1);
#pragma unroll
    for (int q = 0; q < 4; ++q) sh.T[16 * i + 4 * lq + q][16 * w + lr] = tc[d][q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    sh.T[16 * w + 4 * lq + q][16 * w + lr] = tc[0][q];
    // the blocks above the diagonal that a 32-token step covers
    if (w & 1) sh.T[16 * (w - 1) + 4 * lq + q][16 * w + lr] = 0.f;
  }
  __syncthreads();
  // T' fragments: lane (lr, lq) of (row tile a, step h) holds row 16 a + lr and
  // the columns 32 h + 4 lq + 0..3 and 32 h + 16 + 4 lq + 0..3, the order in
  // which the scan's accumulators hold the tokens
  uint4* const td = p.tf + cu * kTChunk;
  for (int f = w; f < kTFrags; f += 4) {
    const int a = f < 2 ? f : f < 4 ? 2 : 3, h = f < 2 ? 0 : f & 1;
    const int t = 16 * a + lr, s0 = 32 * h + 4 * lq;
    const float sg = sh.sig[t];
    const f32x4 t0 = *reinterpret_cast<const f32x4*>(&sh.T[t][s0]);
    const f32x4 t1 = *reinterpret_cast<const f32x4*>(&sh.T[t][s0 + 16]);
    const f32x4 e0 = *reinterpret_cast<const f32x4*>(&sh.be[s0]);
    const f32x4 e1 = *reinterpret_cast<const f32x4*>(&sh.be[s0 + 16]);
    uint4 hi, mid, lo;
    split3(sg * (t0 * e0), sg * (t1 * e1), hi, mid, lo);
    td[(f * 3 + 0) * 64 + lane] = hi;
    td[(f * 3 + 1) * 64 + lane] = mid;
    td[(f * 3 + 2) * 64 + lane] = lo;
  }
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Transposed LDS read: the 16 lanes of a group address four rows of four
// 8-byte pieces (lane s: row s / 4, piece s % 4); lane j receives element j of
// the 16 of each row.
__device__ inline uint2 lds_tr4(const uint16_t* a) {
  return __builtin_bit_cast(
      uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                 (__attribute__((address_space(3))) s16x4*)(const_cast<uint16_t*>(a))));
}

// Waves of a scan workgroup: 16 state rows each.
template <int DV>
constexpr int kScanWaves = DV / 16 < 8 ? DV / 16 : 8;

// 64 rows of COLS bf16 elements in LDS, addressed in pieces of 4 elements (8
// bytes).  The scan reads the keys in two ways: pieces of 16 consecutive rows
// (16 lanes, one piece column), and transposed, 4 rows x 4 neighbouring pieces
// (16 lanes, rows from a multiple of 4).  From 16 pieces per row on, the piece
// index is XORed with f(row) = the row's bits 1:0 above its bits 3:2, which gives
// the 16 lanes of either read 16 different slots of the 128-byte bank row
// (LDS bank conflicts of the scan: 12.6 M -> 2.4 M cycles at 16 requests x 1000
// tokens against padded rows; with 16 pieces per row only f's low 3 bits are used, so
// that the two pieces of a key operand stay a constant apart).  Narrower rows
// are padded instead.
template <int COLS>
struct Swz {
  static constexpr bool kXor = COLS >= 64;
  static constexpr int LD = kXor ? COLS : COLS + 16;
  uint16_t x[kC * LD];
  __device__ static int f(int row) {
    return (((row & 3) << 2) | ((row >> 2) & 3)) & (COLS >= 128 ? 15 : 7);
  }
  // Byte offset of (row, piece): f(row) has the four low bits, so the pieces
  // 4 j + m of one lane are the XOR of its piece m with 4 j, j < 4, and the rest
  // of the address is a constant.
  __device__ static int off(int row, int piece) {
    return 2 * LD * row + 8 * (kXor ? piece ^ f(row) : piece);
  }
  template <typename T>
  __device__ const T* at(int base, int j, int rest) const {
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(x) +
                                      (kXor ? base ^ (32 * (j & 3)) : base + 32 * (j & 3)) +
                                      128 * (j >> 2) + rest);
  }
  // stores the pieces 2 i and 2 i + 1 of a row
  __device__ void put(int row, int i, u32x4 v) {
    if constexpr (kXor) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      char* const b = reinterpret_cast<char*>(x);
      *reinterpret_cast<u32x2*>(b + off(row, 2 * i)) = v.xy;
      *reinterpret_cast<u32x2*>(b + off(row, 2 * i + 1)) = v.zw;
    } else {
      *reinterpret_cast<u32x4*>(x + row * LD + 8 * i) = v;
    }
  }
};

// The operands of two chunks.  The two chunks' keys come first and next to each other,
// so that (up to d_k = 256) both are reached from one lane address and a constant, as
// are the other pairs.  With one struct per chunk every address was held twice, and the
// compiler spilled 46 registers of a lane at d_k = 256 and 3 at 128 (now 16 and none;
// T' read late at 256, see kLateT): 7 chunks of 8 heads of 256 62 -> 54 us per call, 16 x 8
// heads x 1000 tokens 171 -> 139.
template <int DK, int NW>
struct ScanBufs {
  alignas(16) Swz<DK> K[2];
  alignas(16) Swz<16 * NW> V[2];
  uint4 T[2][kTChunk];
  alignas(16) float gam[2][kC];
};

// The scan over the chunks of one segment of one (request, value head): wave w
// carries 16 state rows (all d_k columns, S^T in d_k / 16 accumulator tiles)
// through its chunks,
//   Y = K S^T,  D0 = V - diag(gamma) Y,  D' = T' D0,  S^T <- g S^T + K^T D',
// on v_mfma_f32_16x16x32_bf16: keys and values are exact in bf16; S, D0 and D'
// are split exactly into three bf16 parts (S against one part of K: every
// product exact; T' D0: the six products above 2^-24).  All three
// products chain in registers: the tokens' and columns' order within a 32-deep
// step is that of the accumulators (slot 8 lq + i stands for 4 lq + i of the
// first tile, i < 4, and 4 lq + i - 4 of the second).
//   Segments.  The scan is one chain over the chunks, and 16 rows x 16 heads
// leave most of the chip idle for few heads, so the prompt is cut into nseg segments
// that run at once: S_out = S_in A + B, B from S_in = 0 and, for every segment
// but the first, A (d_k x d_k) from S_in = I with V = 0, by the same code (rows
// of the identity for rows of the state).  prefill_combine_kernel chains them.
//   Each wave reads 52 KB of operands from LDS per chunk (d_k = 128) and the
// eight waves share them; the next chunk's operands travel in registers from
// global memory (requested one chunk ahead) to the other LDS buffer, one barrier
// per chunk.
//   Bound: no one unit.  At 16 requests x 16 heads x 1000 tokens (78 us) the matrix cores are
// busy 38% of the time and the vector units with other instructions about 35%; a wave
// waits 27% of its cycles (LDS, the barrier) and is ready but not issued 36%, with two
// waves per SIMD.
template <int DK, int DV>
__global__ __launch_bounds__(64 * kScanWaves<DV>) void prefill_scan_kernel(PrefillParams p) {
  constexpr int NW = kScanWaves<DV>, TH = 64 * NW;
  constexpr int GB = DV / (16 * NW), GA = DK / (16 * NW);  // workgroups of B and of A
  constexpr int NB = DK / 16;
  // The 32-deep step h of Y covers the state tiles t0(h) and t0(h) + PS: PS = 4
  // puts a key operand's two pieces 128 bytes apart (one two-address read).
  constexpr int PS = NB / 2 < 4 ? NB / 2 : 4;
  auto t0 = [](int h) constexpr { return h / PS * (2 * PS) + h % PS; };
  constexpr int NK = kC * DK / 8 / TH, NT = (kTChunk + TH - 1) / TH, NV = 2;
  __shared__ __align__(16) ScanBufs<DK, NW> buf;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  // all workgroups of a unit on one XCD (block i runs on XCD i % 8)
  const int items = GB + (p.nseg - 1) * (GB + GA);
  int unit, item;
  if (p.xcd_map) {
    const int slot = blockIdx.x >> 3;
    unit = (blockIdx.x & 7) + 8 * (slot / items);
    item = slot % items;
  } else {
    unit = blockIdx.x / items;
    item = blockIdx.x % items;
  }
  int seg = 0, grp = item;
  if (item >= GB) {
    seg = 1 + (item - GB) / (GB + GA);
    grp = (item - GB) % (GB + GA);
  }
  const bool ident = grp >= GB;  // rows of A
  if (ident) grp -= GB;
  const int row0 = 16 * NW * grp + 16 * w;  // this wave's rows
  const int r = unit / p.HV, hv = unit - r * p.HV, hk = hv / (p.HV / p.HK);
  const int cb = seg * p.cps, ce = min(cb + p.cps, p.nch);

  f32x4 st[NB];  // st[b][i] = S^T(16 b + 4 lq + i, lr) = S(row0 + lr, 16 b + 4 lq + i)
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      st[b][i] = ident && 16 * b + 4 * lq + i == row0 + lr ? 1.f : 0.f;

  u32x4 rk[NK], rt[NT], rv[NV];
  float rg;
  // Byte offsets of this thread's pieces from a chunk's first token; the chunk
  // enters as the (scalar) base of a buffer that ends with its last token, so that
  // tokens past the prompt read as zeros without a comparison (and V's buffer
  // is empty for the rows of A).  Chunks past the segment's end re-read its last one.
  const unsigned ks = unsigned(p.HK) * (DK * 2), vs = unsigned(p.HV) * (DV * 2);
  unsigned ko[NK], vo[NV];
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const int e = tid + q * TH;
    ko[q] = unsigned(e / (DK / 8)) * ks + (e % (DK / 8)) * 16;
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int e = tid + q * TH;
    vo[q] = unsigned(e / (2 * NW)) * vs + (e % (2 * NW)) * 16;
  }
  const char* const kbase = static_cast<const char*>(p.k) + (long(r) * p.P * p.HK + hk) * (DK * 2);
  const char* const vbase = static_cast<const char*>(p.v) + (long(r) * p.P * p.HV + hv) * (DV * 2) +
                            (ident ? 0 : 32 * NW * grp);
  auto buffer = [](const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                             int(bytes), 0x00020000);
  };
  auto load = [&](int c) {
    c = min(c, ce - 1);
    const long cu = long(unit) * p.nch + c;
    const unsigned n = unsigned(min(kC, p.P - c * kC));
    const auto kr = buffer(kbase + long(c) * kC * ks, n * ks - unsigned(hk) * (DK * 2));
    const auto vr = buffer(vbase + long(c) * kC * vs,
                           ident ? 0u : n * vs - unsigned(hv) * (DV * 2) - 32u * NW * grp);
    const auto tr = buffer(p.tf + cu * kTChunk, kTChunk * 16);
#pragma unroll
    for (int q = 0; q < NK; ++q) rk[q] = __builtin_amdgcn_raw_buffer_load_b128(kr, ko[q], 0, 0);
#pragma unroll
    for (int q = 0; q < NV; ++q) rv[q] = __builtin_amdgcn_raw_buffer_load_b128(vr, vo[q], 0, 0);
#pragma unroll
    for (int q = 0; q < NT; ++q)
      rt[q] = __builtin_amdgcn_raw_buffer_load_b128(tr, tid * 16, q * TH * 16, 0);
    rg = p.gam[cu * kC + (tid & 63)];
  };
  auto store = [&](int x) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      const int e = tid + q * TH;
      buf.K[x].put(e / (DK / 8), e % (DK / 8), rk[q]);
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int e = tid + q * TH;
      buf.V[x].put(e / (2 * NW), e % (2 * NW), rv[q]);
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int e = tid + q * TH;
      if (kTChunk % TH == 0 || e < kTChunk) *reinterpret_cast<u32x4*>(&buf.T[x][e]) = rt[q];
    }
    if (tid < kC) buf.gam[x][tid] = rg;
  };
  // this lane's LDS offsets: key pieces of row lr from piece lq; transposed
  // keys and values, row 4 lq + lr / 4 from piece lr % 4
  const int kb = Swz<DK>::off(lr, lq), tb = Swz<DK>::off(4 * lq + (lr >> 2), lr & 3),
            vb = Swz<16 * NW>::off(4 * lq + (lr >> 2), 4 * w + (lr & 3));
  constexpr int KR = 32 * Swz<DK>::LD, VR = 32 * Swz<16 * NW>::LD;  // bytes of 16 rows
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
  // One chunk.  The LDS reads of a phase are issued in the phase before (the
  // scheduling barriers keep them there), and within a phase the products and
  // the vector work that prepares the next operands are independent, so that
  // the matrix core and the vector unit run together.
  auto step = [&](int x) __attribute__((always_inline)) {
    const Swz<DK>& sK = buf.K[x];
    const Swz<16 * NW>& sV = buf.V[x];
    const uint4* const sT = buf.T[x];
    const float* const sgam = buf.gam[x];
    f32x4 yh[4], yl[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) yh[a] = yl[a] = z;
    uint4 kf[2][4], sh[2], sm[2], sl[2];
    auto read_k = [&](int h, uint4(&f)[4]) {
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const char* const k = sK.template at<char>(kb, t0(h), KR * a);
        const uint2 k0 = *reinterpret_cast<const uint2*>(k),
                    k1 = *reinterpret_cast<const uint2*>(k + 32 * PS);
        f[a] = make_uint4(k0.x, k0.y, k1.x, k1.y);
      }
    };
    uint2 v[4];
    f32x4 g[4];
    uint4 tf[4][3];
    // (at d_k = 256 T' is read when its product comes: read ahead, as for fewer columns,
    // 27 registers of a lane spill in place of 16, 7 chunks of 8 heads 60 us against 54)
    constexpr bool kLateT = NB > 8;
    auto read_tf = [&]() {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 3; ++q) tf[a][q] = sT[(3 * (a < 2 ? a : 2 * a - 2) + q) * 64 + lane];
    };
    read_k(0, kf[0]);
    cut3(st[t0(0)], st[t0(0) + PS], sh[0], sm[0], sl[0]);
#pragma unroll
    for (int h = 0; h < DK / 32; ++h) {
      __builtin_amdgcn_sched_barrier(0);
      if (h + 1 < DK / 32) {
        read_k(h + 1, kf[(h + 1) & 1]);
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          v[a] = lds_tr4(sV.template at<uint16_t>(vb, 0, VR * a));
          g[a] = *reinterpret_cast<const f32x4*>(&sgam[16 * a + 4 * lq]);
        }
        if constexpr (!kLateT) read_tf();
      }
      __builtin_amdgcn_sched_barrier(0);
      const int e = h & 1;
#pragma unroll
      for (int a = 0; a < 4; ++a) yl[a] = mfma_bf16(kf[e][a], sl[e], yl[a]);
#pragma unroll
      for (int a = 0; a < 4; ++a) yh[a] = mfma_bf16(kf[e][a], sh[e], yh[a]);
#pragma unroll
      for (int a = 0; a < 4; ++a) yl[a] = mfma_bf16(kf[e][a], sm[e], yl[a]);
      if (h + 1 < DK / 32)
        cut3(st[t0(h + 1)], st[t0(h + 1) + PS], sh[e ^ 1], sm[e ^ 1], sl[e ^ 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // D0(t = 16 a + 4 lq + i, n = lr) = V - gamma_t Y
    auto d0 = [&](int a) {
      const f32x4 vf = {bf16_lo_to_float(v[a].x), bf16_hi_to_float(v[a].x),
                        bf16_lo_to_float(v[a].y), bf16_hi_to_float(v[a].y)};
      const f32x4 y = yh[a] + yl[a];
      f32x4 d;
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = fmaf(-g[a][i], y[i], vf[i]);
      return d;
    };
    uint4 dh[2], dm[2], dl[2], tg[2][3];
    f32x4 eh[4], el[4];
    if constexpr (kLateT) read_tf();
    // D' = T' D0: the first 32 tokens' products beside the split of the others
    auto read_tg = [&]() {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        tg[0][q] = sT[(3 * 3 + q) * 64 + lane];
        tg[1][q] = sT[(3 * 5 + q) * 64 + lane];
      }
    };
    if constexpr (!kLateT) read_tg();
    split3(d0(0), d0(1), dh[0], dm[0], dl[0]);
    __builtin_amdgcn_sched_barrier(0);
    // part by part over the tiles, so that no product waits for the one before
    auto apply = [&](const uint4(*t)[3], int h, int a0, int n) {
      auto part = [&](int q, const uint4& d, f32x4* e) {
#pragma unroll
        for (int a = 0; a < n; ++a) e[a0 + a] = mfma_bf16(t[a][q], d, e[a0 + a]);
      };
      part(2, dh[h], el);
      part(0, dh[h], eh);
      part(1, dm[h], el);
      part(0, dl[h], el);
      part(1, dh[h], el);
      part(0, dm[h], el);
    };
#pragma unroll
    for (int a = 0; a < 4; ++a) eh[a] = el[a] = z;
    apply(tf, 0, 0, 4);
    split3(d0(2), d0(3), dh[1], dm[1], dl[1]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kLateT) read_tg();
    // state tiles per group of the update (four at d_k = 256: with eight the
    // operands do not fit in the registers, 242 us against 162 at 4 x 8 heads x 2048 tokens
    // when it was chosen, 134 now)
    constexpr int NG = NB < 8 ? NB : NB == 8 ? 8 : 4;
    uint4 kt[NG][2];
    auto read_t = [&](int b0) {
#pragma unroll
      for (int b = 0; b < NG; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint2 k0 = lds_tr4(sK.template at<uint16_t>(tb, b0 + b, 2 * KR * h)),
                      k1 = lds_tr4(sK.template at<uint16_t>(tb, b0 + b, 2 * KR * h + KR));
          kt[b][h] = make_uint4(k0.x, k0.y, k1.x, k1.y);
        }
    };
    read_t(0);
    const float gc = sgam[kC - 1];
    __builtin_amdgcn_sched_barrier(0);
    uint4 ph[2], pm[2], pl[2];  // D' of the two token halves, split
    apply(tg, 1, 2, 2);
    cut3(eh[0] + el[0], eh[1] + el[1], ph[0], pm[0], pl[0]);
    __builtin_amdgcn_sched_barrier(0);
    // S^T <- g S^T + K^T D'
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += NG) {
      f32x4 lo[NG];
#pragma unroll
      for (int b = 0; b < NG; ++b) lo[b] = mfma_bf16(kt[b][0], pl[0], z);
#pragma unroll
      for (int b = 0; b < NG; ++b) lo[b] = mfma_bf16(kt[b][0], pm[0], lo[b]);
      if (b0 == 0) cut3(eh[2] + el[2], eh[3] + el[3], ph[1], pm[1], pl[1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < NG; ++b) lo[b] = mfma_bf16(kt[b][1], pl[1], lo[b]);
#pragma unroll
      for (int b = 0; b < NG; ++b) lo[b] = mfma_bf16(kt[b][1], pm[1], lo[b]);
      f32x4 hi[NG];
#pragma unroll
      for (int b = 0; b < NG; ++b) hi[b] = mfma_bf16(kt[b][0], ph[0], z);
#pragma unroll
      for (int b = 0; b < NG; ++b) hi[b] = mfma_bf16(kt[b][1], ph[1], hi[b]);
      if (b0 + NG < NB) {
        __builtin_amdgcn_sched_barrier(0);
        read_t(b0 + NG);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < NG; ++b) st[b0 + b] = gc * st[b0 + b] + (hi[b] + lo[b]);
    }
  };
  if (cb < ce) {  // (an empty prompt has no chunk: S = 0)
    // (the scheduling barriers keep the requests ahead of the step: left alone,
    // the compiler sinks them to its end and the next store waits for memory)
    auto turn = [&](int c, int x) __attribute__((always_inline)) {
      store(x ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      load(c + 2);
      __builtin_amdgcn_sched_barrier(0);
      step(x);
      __syncthreads();
    };
    load(cb);
    store(0);
    load(cb + 1);
    __syncthreads();
    for (int c = cb; c < ce; c += 2) {
      turn(c, 0);
      if (c + 1 == ce) break;
      turn(c + 1, 1);
    }
  }
  if (ident) {
    // A's rows 16 NW grp .. as A operands of the combination, A^T split into
    // three bf16 parts: through LDS (whose last reader passed the barrier
    // above, or there was none), a wave per 16 columns of A
    constexpr int LD = DK + 4;
    float* const x = reinterpret_cast<float*>(&buf);
    static_assert(sizeof(buf) >= sizeof(float) * 16 * NW * LD, "A's rows fit the operand buffers");
#pragma unroll
    for (int b = 0; b < NB; ++b)
      *reinterpret_cast<f32x4*>(x + (16 * w + lr) * LD + 16 * b + 4 * lq) = st[b];
    __syncthreads();
    uint4* const dst = p.sega + (long(unit) * (p.nseg - 1) + seg - 1) * (DK * DK * 3 / 8);
    for (int b = w; b < NB; b += NW)
#pragma unroll
      for (int h = 0; h < NW / 2; ++h) {
        f32x4 x0, x1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x0[j] = x[(32 * h + 4 * lq + j) * LD + 16 * b + lr];
          x1[j] = x[(32 * h + 16 + 4 * lq + j) * LD + 16 * b + lr];
        }
        uint4 f[3];
        split3(x0, x1, f[0], f[1], f[2]);
#pragma unroll
        for (int q = 0; q < 3; ++q)
          dst[((b * (DK / 32) + grp * (NW / 2) + h) * 3 + q) * 64 + lane] = f[q];
      }
    return;
  }
  float* const dst = p.nseg > 1 ? p.segb + (long(unit) * p.nseg + seg) * (DV * DK)
                                : p.s_out + long(unit) * (DV * DK);
#pragma unroll
  for (int b = 0; b < NB; ++b)
    *reinterpret_cast<f32x4*>(dst + (row0 + lr) * DK + 16 * b + 4 * lq) = st[b];
}

// S_ctx from the segments of one (request, value head, 16 state rows): S = B_0,
// then S <- S A_j + B_j for j = 1 .. nseg - 1.  Wave w holds the columns
// 16 w .. 16 w + 15 as an accumulator tile of S^T; the tiles, split into three bf16
// parts, are exchanged through LDS as B operands (one barrier per segment), A_j
// comes from the scan as split A operands, and the six products above 2^-24 run
// on v_mfma_f32_16x16x32_bf16.  Latency of the chain bounds it (about a memory
// round trip for the first operands, then the exchange and 6 d_k / 32 products
// per segment); the next segment's operands are requested one segment ahead.
template <int DK, int DV>
__global__ __launch_bounds__(4 * DK) void prefill_combine_kernel(PrefillParams p) {
  constexpr int NH = DK / 32, NRB = DV / 16;
  __shared__ uint4 xs[2][NH][3][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  int unit, rb;
  if (p.xcd_map) {
    const int slot = blockIdx.x >> 3;
    unit = (blockIdx.x & 7) + 8 * (slot / NRB);
    rb = slot % NRB;
  } else {
    unit = blockIdx.x / NRB;
    rb = blockIdx.x % NRB;
  }
  const long at = long(16 * rb + lr) * DK + 16 * w + 4 * lq;
  const float* bp = p.segb + long(unit) * p.nseg * (DV * DK) + at;
  const uint4* ap = p.sega + long(unit) * (p.nseg - 1) * (DK * DK * 3 / 8) + w * (NH * 3 * 64) + lane;
  f32x4 st = *reinterpret_cast<const f32x4*>(bp);
  u32x4 a[NH][3];
  auto load = [&](int j, int h) {
    const uint4* q = ap + long(min(j, p.nseg - 1) - 1) * (DK * DK * 3 / 8) + h * (3 * 64);
#pragma unroll
    for (int i = 0; i < 3; ++i) a[h][i] = *reinterpret_cast<const u32x4*>(q + i * 64);
  };
  f32x4 bn = *reinterpret_cast<const f32x4*>(bp + DV * DK);
#pragma unroll
  for (int h = 0; h < NH; ++h) load(1, h);
  for (int j = 1; j < p.nseg; ++j) {
    const int x = j & 1;
    uint4 d[3];
    split3(st, st, d[0], d[1], d[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      reinterpret_cast<uint2*>(&xs[x][w >> 1][i][lane])[w & 1] = make_uint2(d[i].x, d[i].y);
    __syncthreads();
    f32x4 hi[2] = {}, lo[4] = {};
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const uint4 dh = xs[x][h][0][lane], dm = xs[x][h][1][lane], dl = xs[x][h][2][lane];
      const uint4 t0 = __builtin_bit_cast(uint4, a[h][0]), t1 = __builtin_bit_cast(uint4, a[h][1]),
                  t2 = __builtin_bit_cast(uint4, a[h][2]);
      const int e = h & 1;
      hi[e] = mfma_bf16(t0, dh, hi[e]);
      lo[e] = mfma_bf16(t2, dh, lo[e]);
      lo[2 + e] = mfma_bf16(t1, dm, lo[2 + e]);
      lo[e] = mfma_bf16(t0, dl, lo[e]);
      lo[2 + e] = mfma_bf16(t1, dh, lo[2 + e]);
      lo[e] = mfma_bf16(t0, dm, lo[e]);
      load(j + 1, h);  // (into the registers just read)
    }
    st = bn + ((hi[0] + hi[1]) + ((lo[0] + lo[1]) + (lo[2] + lo[3])));
    bn = *reinterpret_cast<const f32x4*>(bp + long(min(j + 1, p.nseg - 1)) * (DV * DK));
  }
  *reinterpret_cast<f32x4*>(p.s_out + long(unit) * (DV * DK) + at) = st;
}

template <int DK, int DV>
hipError_t launch_bf16(const Shape& s, const PrefillParams& prm, hipStream_t st) {
  const unsigned units = unsigned(s.R * s.HV);
  constexpr int NW = kScanWaves<DV>;
  constexpr unsigned GB = DV / (16 * NW), GA = DK / (16 * NW);
  if (prm.nch > 0) {  // an empty prompt leaves S = 0 (the scan stores zeros)
    prefill_factor_kernel<DK><<<units * unsigned(prm.nch), kP1Threads, 0, st>>>(prm);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  prefill_scan_kernel<DK, DV><<<units * (GB + unsigned(prm.nseg - 1) * (GB + GA)), 64 * NW, 0, st>>>(prm);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || prm.nseg == 1) return e;
  prefill_combine_kernel<DK, DV><<<units * unsigned(DV / 16), 4 * DK, 0, st>>>(prm);
  return hipGetLastError();
}

template <int DK, int DV>
hipError_t launch_f32(const Shape& s, const PrefillParams& prm, hipStream_t st) {
  const unsigned units = unsigned(s.R * s.HV);
  const size_t lds = sizeof(P1Shared<DK>);
  auto k1 = prefill_chunk_kernel<DK, DV>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k1),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  if (prm.nch > 0) {  // an empty prompt leaves S = 0 (phase 2 stores zeros)
    k1<<<units * unsigned(prm.nch), kP1Threads, lds, st>>>(prm);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  prefill_scan_f32_kernel<DK, DV><<<units * unsigned(DV / 16), 4 * DK, 0, st>>>(prm);
  return hipGetLastError();
}

}  // namespace


hipError_t launch_prefill_chunked(const Shape& s, int prompt_len, const void* k, const void* v,
                                  const float* alpha, const float* beta, float* s0_out,
                                  void* workspace, hipStream_t st) {
  PrefillParams prm{};
  prm.k = k;
  prm.v = v;
  prm.alpha = alpha;
  prm.beta = beta;
  prm.s_out = s0_out;
  prm.HK = s.HK;
  prm.HV = s.HV;
  prm.P = prompt_len;
  prm.nch = (prompt_len + kC - 1) / kC;
  const size_t units = size_t(s.R) * s.HV, nch = size_t(prm.nch);
  prm.xcd_map = units % 8 == 0 ? 1 : 0;
  float* base = static_cast<float*>(workspace);
  prm.wb = base;
  float* const kt_base = prm.wb + units * nch * kC * s.dk;  // K^T region (fp32-sized)
  prm.ktb = kt_base;
  prm.utb = kt_base + units * nch * kC * s.dk;
  auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
  prm.gb = reinterpret_cast<float*>(static_cast<char*>(workspace) +
                                    up(units * nch * size_t(kC) * (2 * s.dk + s.dv) * 4));
  if (s.bf16) {
    prm.nseg = prefill_segments(s, prm.nch);
    prm.cps = (prm.nch + prm.nseg - 1) / prm.nseg;
    prm.tf = reinterpret_cast<uint4*>(workspace);
    prm.gam = reinterpret_cast<float*>(prm.tf + units * nch * kTChunk);
    prm.segb = prm.gam + units * nch * kC;
    prm.sega = reinterpret_cast<uint4*>(prm.segb + units * size_t(prm.nseg) * s.dv * s.dk);
  }
#define ONELA_PF_SHAPE(KIND, DK, DV) \
  if (s.dk == DK && s.dv == DV) return launch_##KIND<DK, DV>(s, prm, st);
  if (s.bf16) {
    ONELA_PF_SHAPE(bf16, 32, 32)
    ONELA_PF_SHAPE(bf16, 64, 64)
    ONELA_PF_SHAPE(bf16, 128, 128)
    ONELA_PF_SHAPE(bf16, 128, 256)
    ONELA_PF_SHAPE(bf16, 128, 512)
    ONELA_PF_SHAPE(bf16, 256, 256)
    ONELA_PF_SHAPE(bf16, 256, 512)
  } else {
    ONELA_PF_SHAPE(f32, 32, 32)
    ONELA_PF_SHAPE(f32, 64, 64)
    ONELA_PF_SHAPE(f32, 128, 128)
  }
#undef ONELA_PF_SHAPE
  return hipErrorInvalidValue;
}

}  // namespace onela
