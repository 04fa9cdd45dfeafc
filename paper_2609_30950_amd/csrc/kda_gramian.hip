// Gramian row weights of eq. gram (Sec. 2, Prop. 1) over a window of W
// tokens: the diagonal-erase estimate (a recursion per row, sequential in time)
// and the exact matrix recursion with the full KDA transition, the reference
// the paper compares its estimate with.  Float64.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kda_device.hpp"
#include "kda_kernels.hpp"
#include "kda_profile.hpp"

namespace kda {

// Windowed Gramian weights over tokens t = 1 .. W - 1 in order:
//   A <- lam_t (chi_{t-1} + A),  acc <- acc + q_t^2 A.
// Only this recursion is serial; lam_t = exp(-2 s_t - y_t) (a float64
// exponential, about nine tenths of the work) and q_t^2 are independent per
// token.  A block takes 64 rows of one head and WG_NW waves: per tile of
// WG_NW WG_U tokens each wave forms lam and q^2 of WG_U tokens into LDS with
// the next tile's inputs already requested, and wave 0 then runs the recursion
// over the tile (buffers by tile parity: one barrier per tile).  Bound by HBM
// reads of q, k and s beside the float64 exponentials; a grid of B H d_k / 64
// blocks holds about 16 MB of reads in flight, where one thread per row with
// its loads next to their use held 3 MB and waited for each token's: 988 ->
// 311 us (5.2 TB/s) at B = 32, H = 32, d_k = 128, W = 1024.
constexpr int WG_NW = 4;   // waves per block
constexpr int WG_U = 4;    // tokens per wave and tile
// Blocks per launch: a grid holds fewer than 2^32 threads, so calls of more than
// 2^30 rows (B H d_k; 2^28 in tiles) take several launches.
constexpr long long WG_GRID = 1ll << 22;

template <bool PER_HEAD, bool ERASE>
__global__ void __launch_bounds__(WG_NW* WAVE) k_window_gamma(long long first, int W, int H, int DKr, int C, const float* q,
                                                              const float* s, const float* beta,
                                                              const float* k, double* gamma) {
  constexpr int TILE = WG_NW * WG_U;
  __shared__ double lam[2][TILE][WAVE], q2[2][TILE][WAVE];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = lane_id();
  const int nrb = DKr / WAVE;
  const long long blk = first + blockIdx.x;
  const int bh = (int)(blk / nrb), i = (int)(blk % nrb) * WAVE + lane;
  const int b = bh / H, h = bh % H;
  float qv[WG_U], kv[WG_U], sv[WG_U], bv[WG_U];
  auto issue = [&](int t0) {   // inputs of this wave's tokens of the tile at t0 (clamped to the window)
#pragma unroll
    for (int u = 0; u < WG_U; ++u) {
      const int t = min(t0 + w * WG_U + u, W - 1);
      const size_t tok = ((size_t)b * W + t) * H + h;
      sv[u] = PER_HEAD ? s[tok] : s[tok * DKr + i];
      qv[u] = q[tok * DKr + i];
      if constexpr (ERASE) {
        kv[u] = k[tok * DKr + i];
        bv[u] = beta[tok];
      }
    }
  };
  double A = 0.0, acc = 0.0;
  int ph = 1 % C;   // t % C of the next token of the recursion (wave 0)
  issue(1);
  int par = 0;
  for (int t0 = 1; t0 < W; t0 += TILE, par ^= 1) {
#pragma unroll
    for (int u = 0; u < WG_U; ++u) {
      const double y = ERASE ? erase_sample(kv[u], bv[u]) : 0.0;
      const double qq = (double)qv[u];
      lam[par][w * WG_U + u][lane] = exp(-2.0 * (double)sv[u] - y);
      q2[par][w * WG_U + u][lane] = qq * qq;
    }
    if (t0 + TILE < W) issue(t0 + TILE);
    __syncthreads();
    if (w == 0) {
      const int n = min(TILE, W - t0);
      for (int j = 0; j < n; ++j) {
        const double chi = ph == 0 ? 1.0 : 0.0;   // write-back after token t - 1
        ph = ph + 1 == C ? 0 : ph + 1;
        A = lam[par][j][lane] * (chi + A);
        acc = acc + q2[par][j][lane] * A;
      }
    }
  }
  if (w == 0) gamma[(size_t)bh * DKr + i] = acc / (double)W;
}

// The same with one thread per row and the tokens in turn, for windows too short
// to fill tiles and grids large enough to hide a token's chain (launch_window_gamma).
template <bool PER_HEAD, bool ERASE>
__global__ void __launch_bounds__(WG_NW* WAVE) k_window_gamma_rows(long long first, long long rows, int W, int H, int DKr, int C,
                                                                    const float* q, const float* s, const float* beta,
                                                                    const float* k, double* gamma) {
  const long long id = (first + blockIdx.x) * (WG_NW * WAVE) + threadIdx.x;
  if (id >= rows) return;
  const int bh = (int)(id / DKr), i = (int)(id % DKr);
  const int b = bh / H, h = bh % H;
  double A = 0.0, acc = 0.0;
  int ph = 1 % C;   // t % C
  for (int t = 1; t < W; ++t) {
    const size_t tok = ((size_t)b * W + t) * H + h;
    const float sv = PER_HEAD ? s[tok] : s[tok * DKr + i];
    const double y = ERASE ? erase_sample(k[tok * DKr + i], beta[tok]) : 0.0;
    const double qq = (double)q[tok * DKr + i];
    const double chi = ph == 0 ? 1.0 : 0.0;   // write-back after token t - 1
    ph = ph + 1 == C ? 0 : ph + 1;
    A = exp(-2.0 * (double)sv - y) * (chi + A);
    acc = acc + (qq * qq) * A;
  }
  gamma[id] = acc / (double)W;
}

// Exact Gramian weights (eq. gram with the full transition
// F_t = (I - beta_t k_t k_t^T) diag(exp(-s_t)), the KDA erase): per head,
// backward over a window of W tokens,
//   M <- F_t^T (q_t q_t^T + M) F_t   for t = W-1 down to 1,
//   Gamma_i = (1/W) sum_t chi_{t-1} M_ii,
// chi_tau = 1 when a write-back follows token tau.  (I - beta k k^T) is
// symmetric, so with X = q q^T + M, u = X k and c = k^T u,
//   F^T X F = D (X - (beta k) u^T + (beta^2 c k - beta u) k^T) D
// (the two rank-one terms of the expansion merge), O(d_k^2) per token.
// Float64.  One block per head; thread t holds the 4 x 8 tile of M at rows
// 4 (t / G), columns 8 (t % G), G = d_k / 8 threads per row group (adjacent
// lanes of one wave), so each token's vectors are read from LDS once per
// tile row or column rather than once per element.  u is summed over the G
// tiles of a row by DPP pairings (every lane of the row ends with the same
// value); the thread whose tile holds the diagonal of its
// rows accumulates Gamma from it.
constexpr int XG_RT = 4;   // tile rows
constexpr int XG_CT = 8;   // tile columns

template <int DK>
constexpr int exact_gamma_threads() { return (DK / XG_RT) * (DK / XG_CT); }

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum over N = 8 or 16 adjacent lanes by DPP pairings (quad xor 1, quad
// xor 2, mirror within 8, mirror within 16): each step adds a partner's value
// and partners add the same two numbers, so every lane of the group ends with
// the same sum.
template <int N>
__device__ __forceinline__ double group_sum_d(double v) {
  static_assert(N == 8 || N == 16, "group size");
  v += dpp_d<0xB1>(v);
  v += dpp_d<0x4E>(v);
  v += dpp_d<0x141>(v);
  if constexpr (N == 16) v += dpp_d<0x140>(v);
  return v;
}

template <int DK>
__global__ void __launch_bounds__(exact_gamma_threads<DK>()) k_exact_gamma(
    int W, int H, int C, int per_head, int no_erase, const float* q, const float* s,
    const float* beta, const float* k, double* gamma) {
  constexpr int G = DK / XG_CT;
  constexpr int NT = exact_gamma_threads<DK>();
  constexpr int NW = NT / WAVE;
  static_assert((G == 8 || G == 16) && NT % WAVE == 0, "row groups within a wave");
  const int bh = blockIdx.x, b = bh / H, h = bh % H;
  const int t = threadIdx.x, r0 = (t / G) * XG_RT, c0 = (t % G) * XG_CT;
  const int w = t / WAVE, lane = lane_id();
  // the tile holding the diagonal of rows r0..r0+3, and where it sits in it
  const bool diag = (t % G) == r0 / XG_CT;
  const int dcol = r0 % XG_CT;   // 0 or XG_RT
  static_assert(XG_CT == 2 * XG_RT, "two tile row blocks per tile width");
  // token inputs double-buffered by token parity: writing token tt's while a
  // slower wave still reads token tt + 1's needs no barrier
  __shared__ __align__(16) double qb[2][DK], kb[2][DK], db[2][DK];
  __shared__ __align__(16) double uv[DK];
  __shared__ double part[NW];
  double M[XG_RT][XG_CT];
#pragma unroll
  for (int a = 0; a < XG_RT; ++a)
#pragma unroll
    for (int j = 0; j < XG_CT; ++j) M[a][j] = 0.0;
  // diagonal sums for both positions the diagonal can take in a tile (a
  // select between two register elements would be lowered to a memory index)
  double acc0[XG_RT] = {0.0, 0.0, 0.0, 0.0}, acc1[XG_RT] = {0.0, 0.0, 0.0, 0.0};
  // token inputs one token ahead in registers (loaded while the current token runs)
  float nq = 0.f, nk = 0.f, ns = 0.f, nb = 0.f;
  auto fetch = [&](int tt) {
    const size_t tok = ((size_t)b * W + tt) * H + h;
    if (t < DK) {
      nq = q[tok * DK + t];
      nk = k[tok * DK + t];
      ns = per_head ? s[tok] : s[tok * DK + t];
    }
    nb = beta[tok];
  };
  if (W > 1) fetch(W - 1);
  for (int tt = W - 1; tt >= 1; --tt) {
    double* qv = qb[tt & 1];
    double* kv = kb[tt & 1];
    double* dv = db[tt & 1];
    if (t < DK) {
      qv[t] = (double)nq;
      kv[t] = (double)nk;
      dv[t] = exp(-(double)ns);
    }
    const double bt = no_erase ? 0.0 : (double)nb;   // no erasure: F = D
    if (tt > 1) fetch(tt - 1);
    __syncthreads();
    double qr[XG_RT], kr[XG_RT], ur[XG_RT], kc[XG_CT];
#pragma unroll
    for (int a = 0; a < XG_RT; ++a) {
      qr[a] = qv[r0 + a];
      kr[a] = kv[r0 + a];
    }
#pragma unroll
    for (int j = 0; j < XG_CT; ++j) kc[j] = kv[c0 + j];
    // X = q q^T + M and this tile's part of u = X k
#pragma unroll
    for (int a = 0; a < XG_RT; ++a) ur[a] = 0.0;
#pragma unroll
    for (int j = 0; j < XG_CT; ++j) {
      const double qc = qv[c0 + j];
#pragma unroll
      for (int a = 0; a < XG_RT; ++a) {
        M[a][j] = __builtin_fma(qr[a], qc, M[a][j]);
        ur[a] = __builtin_fma(M[a][j], kc[j], ur[a]);
      }
    }
#pragma unroll
    for (int a = 0; a < XG_RT; ++a) ur[a] = group_sum_d<G>(ur[a]);
    // c = k^T u: the row group's first tile contributes its rows, summed over
    // the first tiles of the wave, then over waves in order
    double ct = 0.0;
    if (t % G == 0) {
#pragma unroll
      for (int a = 0; a < XG_RT; ++a) {
        ct += kr[a] * ur[a];
        uv[r0 + a] = ur[a];
      }
    }
#pragma unroll
    for (int o = G; o < WAVE; o <<= 1) ct += __shfl_xor(ct, o);
    if (lane == 0) part[w] = ct;
    __syncthreads();
    double cc = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) cc += part[i];
    double ar[XG_RT], fr[XG_RT], dr[XG_RT];
#pragma unroll
    for (int a = 0; a < XG_RT; ++a) {
      ar[a] = bt * kr[a];
      fr[a] = bt * bt * cc * kr[a] - bt * ur[a];
      dr[a] = dv[r0 + a];
    }
#pragma unroll
    for (int j = 0; j < XG_CT; ++j) {
      const double uc = uv[c0 + j], dc = dv[c0 + j];
#pragma unroll
      for (int a = 0; a < XG_RT; ++a) {
        M[a][j] = __builtin_fma(-ar[a], uc, M[a][j]);
        M[a][j] = __builtin_fma(fr[a], kc[j], M[a][j]);
        M[a][j] = M[a][j] * (dr[a] * dc);
      }
    }
    if (diag && tt % C == 0) {   // a write-back follows token tt - 1
#pragma unroll
      for (int a = 0; a < XG_RT; ++a) {
        acc0[a] += M[a][a];
        acc1[a] += M[a][XG_RT + a];
      }
    }
  }
  if (diag) {
#pragma unroll
    for (int a = 0; a < XG_RT; ++a)
      gamma[(size_t)bh * DK + r0 + a] = (dcol == 0 ? acc0[a] : acc1[a]) / (double)W;
  }
}

hipError_t launch_exact_gamma(const KParams& p, int W, int C, const float* q, const float* s,
                              const float* beta, const float* k, double* gamma, hipStream_t st) {
  const int nbh = p.B * p.H;
  if (p.dk == 64)
    return launch("weights", k_exact_gamma<64>, nbh, exact_gamma_threads<64>(), 0, st, W, p.H, C,
                  p.per_head, p.no_erase, q, s, beta, k, gamma);
  return launch("weights", k_exact_gamma<128>, nbh, exact_gamma_threads<128>(), 0, st, W, p.H, C,
                p.per_head, p.no_erase, q, s, beta, k, gamma);
}

hipError_t launch_window_gamma(const KParams& p, int W, int C, const float* q, const float* s,
                               const float* beta, const float* k, double* gamma, hipStream_t st) {
  // Rows in turn up to a token per 8192 rows of the call, at least four: a tile
  // is 16 tokens' exponentials and one trip to memory however few are left of
  // it, while with that many rows the threads' own chains overlap.  us, tiles
  // against rows in turn (rate per channel, with erasure), d = 128:
  //   2 tokens, heads 32: 3.4 3.2   1024: 7.0 3.3   8192: 38.8 7.3
  //   16 tokens,   256: 4.4 5.8     1024: 7.7 6.4   8192: 43.9 31.3
  //   32 tokens,  1024: 13.2 16.1   2048: 22.0 20.0   64 tokens, 4096: 84.3 78.4
  // With three arrays to read (q, k and s per channel) the turn comes at about 100
  // tokens however many the rows (16384 heads: 96 tokens 453 443, 128 tokens 588
  // 642); with one (rate per head, no erasure) at twice the length beyond 2^16
  // rows (4096 heads: 96 tokens 84 69; 512 heads: 16 tokens 4.9 5.4).
  const long long rows = (long long)p.B * p.H * p.dk;
  long long in_turn_max = rows >> 13 > 4 ? rows >> 13 : 4;
  if (!p.per_head && !p.no_erase && in_turn_max > 96) in_turn_max = 96;
  if (p.per_head && p.no_erase && rows > 1 << 16) in_turn_max *= 2;
  // launches of up to WG_GRID blocks of WG_NW waves
  const auto blocks = [](long long nblk, auto go) {
    hipError_t e = hipSuccess;
    for (long long first = 0; first < nblk && e == hipSuccess; first += WG_GRID)
      e = go(first, (unsigned)(nblk - first < WG_GRID ? nblk - first : WG_GRID));
    return e;
  };
  const auto tiled = [&](auto kernel) {
    return blocks(rows / WAVE, [&](long long first, unsigned n) {
      return launch("weights", kernel, n, WG_NW * WAVE, 0, st, first, W, p.H, p.dk, C, q, s, beta, k, gamma);
    });
  };
  const auto in_turn = [&](auto kernel) {
    return blocks((rows + WG_NW * WAVE - 1) / (WG_NW * WAVE), [&](long long first, unsigned n) {
      return launch("weights", kernel, n, WG_NW * WAVE, 0, st, first, rows, W, p.H, p.dk, C, q, s, beta, k, gamma);
    });
  };
  if (W <= in_turn_max) {
    if (p.per_head)
      return p.no_erase ? in_turn(k_window_gamma_rows<true, false>) : in_turn(k_window_gamma_rows<true, true>);
    return p.no_erase ? in_turn(k_window_gamma_rows<false, false>) : in_turn(k_window_gamma_rows<false, true>);
  }
  if (p.per_head) return p.no_erase ? tiled(k_window_gamma<true, false>) : tiled(k_window_gamma<true, true>);
  return p.no_erase ? tiled(k_window_gamma<false, false>) : tiled(k_window_gamma<false, true>);
}

}  // namespace kda
