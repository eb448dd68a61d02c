// The intra encoder: forward wavelet transform of every tile (Section 3.1;
// per level every column, then every row) and the uniform quantiser.
//
// Two kernels, each reading its samples once and writing its coefficients
// once:
//
//  * k_enc_strip (plane edges 512 and 256): the two finest levels in one pass
//    over the source.  One wave takes a strip of a tile across its whole
//    width, every lane owning C adjacent columns; the vertical lifting streams
//    down the rows with a few rows of state in registers, the horizontal
//    lifting takes one value per step from the neighbouring lane (DPP), and
//    the second level is fed row by row from the first.  The approximation
//    (1/16 of the samples) goes to a workspace.
//  * k_enc_tile (edges up to 128): a whole plane tile in LDS, all its
//    remaining levels in place, from the 8-bit source or from the workspace.
//
// What bounds it: HBM for 5/3 (the floor is a read of the source and a write
// of the coefficients, 3 bytes per sample: 302 MB of an 8192 x 8192 YUV420
// frame, 58 us at a copy's rate; the strip kernel takes 71 us, 4.4 TB/s), the
// float64 arithmetic for 9/7 (4096 x 4096: 47 us against 24).  One pass per
// level and direction through a workspace of every sample, allocated and freed
// by each call, moved about 30 (60) bytes per sample; whole calls: 1598 -> 107 us
// (5/3, 8192 x 8192, five levels), 2700 to 4560 (the allocations varied) -> 80 us
// (9/7, 4096 x 4096).
#include <algorithm>
#include <type_traits>

#include "wv_dev.h"
#include "wv_internal.h"

namespace wv {
namespace {

// a / b correctly rounded, from inv = 1 / b correctly rounded: one residual
// correction of the product (P. Markstein, IBM J. Res. Dev. 34, 1990), three
// operations where the general division takes a dozen.
__device__ __forceinline__ double div_by(double a, double b, double inv) {
  const double q = a * inv;
  return __builtin_fma(__builtin_fma(-q, b, a), inv, q);
}

// ------------------------------------------------------------ forward lifting
// One direction of one level, e_k = x[2k], o_k = x[2k+1].  Whole-sample
// symmetric extension makes every lifting step repeat its own end value:
// x[n] = x[n-2] gives e_M = e_(M-1) (and the updated even samples likewise),
// x[-1] = x[1] gives p_(-1) = p_0 (and the updated odd samples likewise).
struct Enc53 {
  using V = int;
  using CT = int16_t;
  static constexpr int LAG = 1;    // pairs between a pair's samples and its outputs
  static constexpr int WARM = 1;   // pairs ahead of the first output that it depends on
  static constexpr int LO = 2, HI = 1;   // samples before / after a run of pairs
  __device__ static __forceinline__ int high(int o, int e0, int e1) { return o - ((e0 + e1) >> 1); }
  __device__ static __forceinline__ int low(int e, int d0, int d1) { return e + ((d0 + d1 + 2) >> 2); }
  // NP pairs from x[-LO .. 2 NP + HI)
  template <int NP>
  __device__ static __forceinline__ void run(const int* x, int* s, int* d) {
    int p[NP + 1];
#pragma unroll
    for (int k = 0; k <= NP; ++k) p[k] = high(x[2 * k + 1], x[2 * k], x[2 * k + 2]);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      s[k] = low(x[2 * k + 2], p[k], p[k + 1]);
      d[k] = p[k + 1];
    }
  }
};

struct Enc97 {
  using V = double;
  using CT = float;
  static constexpr int LAG = 2, WARM = 2, LO = 4, HI = 3;
  __device__ static __forceinline__ double a(double o, double e0, double e1) { return o + WV_A97 * (e0 + e1); }
  __device__ static __forceinline__ double b(double e, double p0, double p1) { return e + WV_B97 * (p0 + p1); }
  __device__ static __forceinline__ double g(double p, double f0, double f1) { return p + WV_G97 * (f0 + f1); }
  __device__ static __forceinline__ double d(double f, double q0, double q1) { return f + WV_D97 * (q0 + q1); }
  __device__ static __forceinline__ double low(double v) { return div_by(v, WV_K97, 1.0 / WV_K97); }
  __device__ static __forceinline__ double high(double v) { return v * WV_K97; }
  template <int NP>
  __device__ static __forceinline__ void run(const double* x, double* s, double* dd) {
    double p[NP + 3], f[NP + 2], q[NP + 1];
#pragma unroll
    for (int k = 0; k < NP + 3; ++k) p[k] = a(x[2 * k + 1], x[2 * k], x[2 * k + 2]);   // pair k - 2
#pragma unroll
    for (int k = 0; k < NP + 2; ++k) f[k] = b(x[2 * k + 2], p[k], p[k + 1]);           // pair k - 1
#pragma unroll
    for (int k = 0; k < NP + 1; ++k) q[k] = g(p[k + 1], f[k], f[k + 1]);               // pair k - 1
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      s[k] = low(d(f[k + 1], q[k], q[k + 1]));
      dd[k] = high(q[k + 1]);
    }
  }
};

// ---------------------------------------------------------------- quantiser
// q = sign(c) floor(|c| / step + 1/2).  5/3: the index itself, the division
// of n = 2 |c| + step by 2 step as a multiplication: with s such that
// 2^s < 2 step <= 2^(s+1) and mul = ceil(2^(32+s) / (2 step)),
// n / (2 step) = (n mul) >> (32 + s) exactly for every n < 2^31.
// 9/7: step q in float64, stored as float32.
struct Quant {
  int step;
  uint32_t mul;
  int shift;
  double stepd, inv; // step and 1 / step
  int* overflow;     // set to 1 when an index falls outside int16
};
__device__ __forceinline__ int16_t quantise(int c, const Quant& q, bool& bad) {
  const int a = (int)(__umulhi((uint32_t)(2 * abs(c) + q.step), q.mul) >> q.shift);
  const int r = c < 0 ? -a : a;
  bad |= r != (int)(int16_t)r;
  return (int16_t)r;
}
__device__ __forceinline__ float quantise(double c, const Quant& q, bool&) {
  const double a = floor(div_by(fabs(c), q.stepd, q.inv) + 0.5);
  return (float)(q.stepd * (c < 0 ? -a : a));
}

// N consecutive values at p; the buffers need no more than their elements'
// alignment (packed types: the hardware's wide accesses may be unaligned).
template <class T, int N>
struct __attribute__((packed, aligned(sizeof(T)))) Vec { T v[N]; };

template <int N, class V, class CT>
__device__ __forceinline__ void put(CT* p, const V (&c)[N], const Quant& q, bool& bad) {
  Vec<CT, N> w;
#pragma unroll
  for (int k = 0; k < N; ++k) w.v[k] = quantise(c[k], q, bad);
  *(Vec<CT, N>*)p = w;
}

// ------------------------------------------------------------------ strips
// A lane's value in the previous / next lane; the first / last lane keeps its
// own edge value.
__device__ __forceinline__ int lane_left(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xf, 0xf, false);   // wave_shr:1
}
__device__ __forceinline__ int lane_right(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x130, 0xf, 0xf, false);   // wave_shl:1
}
__device__ __forceinline__ double lane_left(double edge, double v) {
  return __hiloint2double(lane_left(__double2hiint(edge), __double2hiint(v)),
                          lane_left(__double2loint(edge), __double2loint(v)));
}
__device__ __forceinline__ double lane_right(double edge, double v) {
  return __hiloint2double(lane_right(__double2hiint(edge), __double2hiint(v)),
                          lane_right(__double2loint(edge), __double2loint(v)));
}

// One row spread over the wave's 64 lanes, 2 H samples per lane.
template <class LF, int H>
struct RowFwd;
template <int H>
struct RowFwd<Enc53, H> {
  __device__ static __forceinline__ void run(const int (&x)[2 * H], int (&s)[H], int (&d)[H]) {
    const int er = lane_right(x[2 * H - 2], x[0]);
#pragma unroll
    for (int k = 0; k < H; ++k) d[k] = Enc53::high(x[2 * k + 1], x[2 * k], k + 1 < H ? x[2 * k + 2] : er);
    const int dl = lane_left(d[0], d[H - 1]);
#pragma unroll
    for (int k = 0; k < H; ++k) s[k] = Enc53::low(x[2 * k], k ? d[k - 1] : dl, d[k]);
  }
};
template <int H>
struct RowFwd<Enc97, H> {
  __device__ static __forceinline__ void run(const double (&x)[2 * H], double (&s)[H], double (&d)[H]) {
    double p[H], f[H], q[H];
    const double er = lane_right(x[2 * H - 2], x[0]);
#pragma unroll
    for (int k = 0; k < H; ++k) p[k] = Enc97::a(x[2 * k + 1], x[2 * k], k + 1 < H ? x[2 * k + 2] : er);
    const double pl = lane_left(p[0], p[H - 1]);
#pragma unroll
    for (int k = 0; k < H; ++k) f[k] = Enc97::b(x[2 * k], k ? p[k - 1] : pl, p[k]);
    const double fr = lane_right(f[H - 1], f[0]);
#pragma unroll
    for (int k = 0; k < H; ++k) q[k] = Enc97::g(p[k], f[k], k + 1 < H ? f[k + 1] : fr);
    const double ql = lane_left(q[0], q[H - 1]);
#pragma unroll
    for (int k = 0; k < H; ++k) {
      s[k] = Enc97::low(Enc97::d(f[k], k ? q[k - 1] : ql, q[k]));
      d[k] = Enc97::high(q[k]);
    }
  }
};

// Vertical lifting streamed down the rows: push(j, e_j, o_j) completes pair
// j - LAG (s, d).  Pairs before 0 and from m on stand outside the level: the
// values pushed for them do not matter, the extension is applied here.
template <class LF, int C>
struct ColFwd;
template <int C>
struct ColFwd<Enc53, C> {
  int e[C], o[C], dp[C];
  __device__ __forceinline__ void push(int j, int m, const int (&en)[C], const int (&on)[C], int (&s)[C],
                                       int (&d)[C]) {
    const bool top = j == 1, end = j >= m;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      d[c] = Enc53::high(o[c], e[c], end ? e[c] : en[c]);
      s[c] = Enc53::low(e[c], top ? d[c] : dp[c], d[c]);
      dp[c] = d[c];
      e[c] = en[c];
      o[c] = on[c];
    }
  }
};
template <int C>
struct ColFwd<Enc97, C> {
  double e[C], o[C], pp[C], fp[C], qp[C];
  __device__ __forceinline__ void push(int j, int m, const double (&en)[C], const double (&on)[C],
                                       double (&s)[C], double (&d)[C]) {
    const bool top = j == 1, end = j >= m, past = j > m, top2 = j == 2;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const double p = Enc97::a(o[c], e[c], end ? e[c] : en[c]);            // pair j - 1
      double f = Enc97::b(e[c], top ? p : pp[c], p);
      if (past) f = fp[c];
      const double q = Enc97::g(pp[c], fp[c], f);                            // pair j - 2
      s[c] = Enc97::low(Enc97::d(fp[c], top2 ? q : qp[c], q));
      d[c] = Enc97::high(q);
      pp[c] = p;
      fp[c] = f;
      qp[c] = q;
      e[c] = en[c];
      o[c] = on[c];
    }
  }
};

// One wave: rows [4 i0, 4 (i0 + n)) of a P x P plane tile, P = 64 C, NL = 1 or
// 2 levels.  Level 1 pairs t, level 2 pairs i.  The state is warmed up with
// the WARM pairs before the strip's first one at each level.
template <class LF, int C, int NL>
__device__ __forceinline__ void enc_strip(const uint8_t* src, typename LF::CT* dst, typename LF::V* ws,
                                          int i0, int n, const Quant& q) {
  using V = typename LF::V;
  using CT = typename LF::CT;
  constexpr int P = 64 * C, M1 = P / 2, M2 = P / 4, H1 = C / 2, H2 = C / 4, LAG = LF::LAG;
  const int lane = threadIdx.x & 63;
  using Row = Vec<uint8_t, C>;
  const Row* base = (const Row*)(src + lane * C);
  constexpr int RS = P / C;          // rows are RS lane vectors apart
  const int i1 = i0 + n;
  const int ts = NL == 2 ? 2 * max(i0 - LF::WARM, 0) : 2 * i0;   // first pair level 2 reads
  const int js = max(ts - LF::WARM, 0);
  const int u0 = (js - LAG) >> 1;    // pairs 2 u, 2 u + 1 are completed in step u
  const int u1 = NL == 2 ? i1 - 1 + LAG : i1 - 1;
  auto load = [&](int u, Row (&r)[4]) __attribute__((always_inline)) {
    const int j = 2 * u + LAG;       // the pairs pushed to complete 2 u and 2 u + 1
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = base[min(max(2 * j + k, 0), P - 1) * RS];
  };
  ColFwd<LF, C> c1;
  ColFwd<LF, NL == 2 ? H1 : 1> c2;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    c1.e[c] = c1.o[c] = V(0);
    if constexpr (LAG == 1) c1.dp[c] = V(0);
    else c1.pp[c] = c1.fp[c] = c1.qp[c] = V(0);
  }
  if constexpr (NL == 2)
#pragma unroll
    for (int c = 0; c < H1; ++c) {
      c2.e[c] = c2.o[c] = V(0);
      if constexpr (LAG == 1) c2.dp[c] = V(0);
      else c2.pp[c] = c2.fp[c] = c2.qp[c] = V(0);
    }
  bool bad = false;
  V ll[2][H1];
  Row nxt[4];
  load(u0, nxt);
  for (int u = u0; u <= u1; ++u) {
    Row cur[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) cur[k] = nxt[k];
    if (u < u1) load(u + 1, nxt);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int t = 2 * u + h, j = t + LAG;
      V en[C], on[C], s[C], d[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        en[c] = (V)cur[2 * h].v[c];
        on[c] = (V)cur[2 * h + 1].v[c];
      }
      c1.push(j, M1, en, on, s, d);
      V hl[H1];
      RowFwd<LF, H1>::run(s, ll[h], hl);
      if (u >= i0 && u < i1) {
        V lh[H1], hh[H1];
        RowFwd<LF, H1>::run(d, lh, hh);
        CT* row = dst + (size_t)t * P + lane * H1;
        if constexpr (NL == 1) put<H1>(row, ll[h], q, bad);
        put<H1>(row + M1, hl, q, bad);
        put<H1>(row + (size_t)M1 * P, lh, q, bad);
        put<H1>(row + (size_t)M1 * P + M1, hh, q, bad);
      }
    }
    if constexpr (NL == 2) {
      V s[H1], d[H1];
      c2.push(u, M2, ll[0], ll[1], s, d);
      const int i = u - LAG;
      if (i >= i0) {
        V l2[H2], hl[H2], lh[H2], hh[H2];
        RowFwd<LF, H2>::run(s, l2, hl);
        RowFwd<LF, H2>::run(d, lh, hh);
        CT* row = dst + (size_t)i * P + lane * H2;
        if (ws) {
#pragma unroll
          for (int k = 0; k < H2; ++k) ws[(size_t)i * M2 + lane * H2 + k] = l2[k];
        } else {
          put<H2>(row, l2, q, bad);
        }
        put<H2>(row + M2, hl, q, bad);
        put<H2>(row + (size_t)M2 * P, lh, q, bad);
        put<H2>(row + (size_t)M2 * P + M2, hh, q, bad);
      }
    }
  }
  if (bad) *q.overflow = 1;
}

struct StripArgs {
  const uint8_t* src[3];
  void* dst[3];
  void* ws[3];        // approximation after two levels, or NULL: there are no more
  int n_tiles;
  int rows;           // level 2 rows (4 source rows each) per strip
  int blocks0;        // workgroups of plane 0; planes 1 and 2 follow
  Quant q;
};

// Workgroups [0, blocks0) take plane 0 (edge 64 C), the others planes 1 and 2
// (edge 32 C, absent when C = 4 or for grey frames).  Four waves, a strip each.
template <class LF, int C, int NL>
__global__ __launch_bounds__(256) void k_enc_strip(const StripArgs a) {
  using V = typename LF::V;
  using CT = typename LF::CT;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto go = [&](auto CC, int p, int w) __attribute__((always_inline)) {
    constexpr int c = decltype(CC)::value, P = 64 * c, M2 = P / 4;
    const int per = M2 / a.rows, tile = w / per;
    if (tile >= a.n_tiles) return;
    const size_t off = (size_t)tile * P * P;
    V* ws = a.ws[p] ? (V*)a.ws[p] + off / 16 : nullptr;
    enc_strip<LF, c, NL>(a.src[p] + off, (CT*)a.dst[p] + off, ws, (w - tile * per) * a.rows, a.rows, a.q);
  };
  const int b = blockIdx.x;
  if (b < a.blocks0) {
    go(std::integral_constant<int, C>{}, 0, b * 4 + wave);
  } else if constexpr (C == 8) {
    const int nb = (gridDim.x - a.blocks0) / 2, r = b - a.blocks0, p = r >= nb;
    go(std::integral_constant<int, C / 2>{}, 1 + p, (r - p * nb) * 4 + wave);
  }
}

// -------------------------------------------------------------- whole tiles
// Pairs of one line per thread at a level of edge M: M lines of 8 runs.
constexpr int seg_len(int m) { return m >= 16 ? m / 8 : 2; }

// One direction of a level of edge M, in place over the top-left M x M of buf
// (row pitch PITCH, odd: lines along either direction fall into distinct
// banks): every sample is read into registers before any is written.
template <class LF, int M, int PITCH, bool ROWS>
__device__ __forceinline__ void tile_pass(typename LF::V* buf) {
  using V = typename LF::V;
  constexpr int S = seg_len(M), NP = S / 2;
  const int line = threadIdx.x % M, k0 = (threadIdx.x / M) * S;
  const bool on = k0 < M;
  auto at = [&](int i) -> V& { return ROWS ? buf[line * PITCH + i] : buf[i * PITCH + line]; };
  V x[S + LF::LO + LF::HI], s[NP], d[NP];
  if (on) {
#pragma unroll
    for (int i = 0; i < S + LF::LO + LF::HI; ++i) {
      const int j = k0 - LF::LO + i, b = abs(j);
      x[i] = at(M >= 8 ? min(b, 2 * M - 2 - b) : wss(j, M));   // one reflection is enough from 8 on
    }
    LF::template run<NP>(x, s, d);
  }
  __syncthreads();
  if (on) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      at(k0 / 2 + k) = s[k];
      at(M / 2 + k0 / 2 + k) = d[k];
    }
  }
  __syncthreads();
}

template <class LF, int M, int PITCH>
__device__ __forceinline__ void tile_levels(typename LF::V* buf, int n) {
  if constexpr (M >= 2) {
    if (n <= 0) return;
    tile_pass<LF, M, PITCH, false>(buf);
    tile_pass<LF, M, PITCH, true>(buf);
    tile_levels<LF, M / 2, PITCH>(buf, n - 1);
  }
}

struct TileArgs {
  const void* src[2];     // per plane: the 8-bit plane or the workspace, [n_tiles][E][E]
  void* dst[2];           // coefficient planes, tiles of edge p
  int p, levels;          // edge of the stored tile; levels to do on the E x E region
  Quant q;
};

// Levels of an E x E region of one plane tile per workgroup.  IN: uint8_t
// (the whole tile) or the workspace type.
template <class LF, int E, class IN>
__global__ __launch_bounds__(E * 8) void k_enc_tile(const TileArgs a) {
  using V = typename LF::V;
  using CT = typename LF::CT;
  constexpr int PITCH = E + 1, NT = E * 8, N4 = E * E / 4;
  __shared__ V buf[E * PITCH];
  const int tile = blockIdx.x, pl = blockIdx.y;
  const Vec<IN, 4>* src = (const Vec<IN, 4>*)((const IN*)a.src[pl] + (size_t)tile * E * E);
#pragma unroll
  for (int i0 = 0; i0 < N4; i0 += NT) {
    const int i = i0 + threadIdx.x;
    if (N4 % NT == 0 || i < N4) {
      const Vec<IN, 4> w = src[i];
#pragma unroll
      for (int k = 0; k < 4; ++k) buf[(4 * i / E) * PITCH + 4 * i % E + k] = (V)w.v[k];
    }
  }
  __syncthreads();
  tile_levels<LF, E, PITCH>(buf, a.levels);
  CT* dst = (CT*)a.dst[pl] + (size_t)tile * a.p * a.p;
  bool bad = false;
#pragma unroll
  for (int i0 = 0; i0 < N4; i0 += NT) {
    const int i = i0 + threadIdx.x;
    if (N4 % NT == 0 || i < N4) {
      const int r = 4 * i / E, c = 4 * i % E;
      V v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = buf[r * PITCH + c + k];
      put<4>(dst + (size_t)r * a.p + c, v, a.q, bad);
    }
  }
  if (bad) *a.q.overflow = 1;
}

// e: edges of 8 to 128 from the 8-bit source, of 64 and 128 from the workspace
// (a quarter of a strip plane's edge).
template <class LF, class IN>
hipError_t launch_tile(int e, int planes, int n_tiles, const TileArgs& a, hipStream_t s) {
  const dim3 g(n_tiles, planes);
  constexpr bool WS = !std::is_same<IN, uint8_t>::value;
  if (e == 128) {
    hipLaunchKernelGGL((k_enc_tile<LF, 128, IN>), g, dim3(1024), 0, s, a);
  } else if (e == 64) {
    hipLaunchKernelGGL((k_enc_tile<LF, 64, IN>), g, dim3(512), 0, s, a);
  } else {
    if constexpr (WS) return hipErrorInvalidValue;
    else if (e == 32) hipLaunchKernelGGL((k_enc_tile<LF, 32, IN>), g, dim3(256), 0, s, a);
    else if (e == 16) hipLaunchKernelGGL((k_enc_tile<LF, 16, IN>), g, dim3(128), 0, s, a);
    else if (e == 8) hipLaunchKernelGGL((k_enc_tile<LF, 8, IN>), g, dim3(64), 0, s, a);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Rows (of level 2) per strip: short strips give more waves, long ones read
// and transform fewer rows twice (the warm-up, 3 rows of 5/3 and 5 of 9/7).
// Strip kernel on 8192 x 8192 5/3 / 4096 x 4096 9/7 (us): 32 rows 80.7 / 86.3,
// 16 rows 72.1 / 54.1, 8 rows 71.2 / 47.5.
constexpr int kStripRows = 8;

template <class LF>
hipError_t launch_encode_t(int nplanes, int n_tiles, int tile, int levels, int qstep, const void* const* src,
                           void* const* dst, void* ws, int* overflow, hipStream_t s) {
  using V = typename LF::V;
  Quant q;
  q.step = qstep;
  q.stepd = qstep;
  q.inv = 1.0 / qstep;
  const uint64_t dv = 2u * (uint64_t)qstep;
  q.shift = 0;
  while ((2ull << q.shift) < dv) ++q.shift;
  q.mul = (uint32_t)(((1ull << (32 + q.shift)) + dv - 1) / dv);
  q.overflow = overflow;
  const int nl = std::min(levels, 2);
  V* wp[3] = {};
  const int strips = tile == 512 ? nplanes : tile == 256 ? 1 : 0;   // planes of edge 256 and more
  if (strips) {
    StripArgs a = {};
    size_t at = 0;
    for (int p = 0; p < strips; ++p) {
      const int e = p ? tile / 2 : tile;
      a.src[p] = (const uint8_t*)src[p];
      a.dst[p] = dst[p];
      wp[p] = (V*)ws + at;
      a.ws[p] = levels > 2 ? wp[p] : nullptr;
      at += (size_t)n_tiles * (e / 4) * (e / 4);
    }
    a.n_tiles = n_tiles;
    a.rows = kStripRows;
    a.q = q;
    auto groups = [&](int e) { return (n_tiles * (e / 4 / kStripRows) + 3) / 4; };
    a.blocks0 = groups(tile);
    const dim3 g(a.blocks0 + (strips == 3 ? 2 * groups(tile / 2) : 0));
    if (tile == 512 && nl == 2) hipLaunchKernelGGL((k_enc_strip<LF, 8, 2>), g, dim3(256), 0, s, a);
    else if (tile == 512) hipLaunchKernelGGL((k_enc_strip<LF, 8, 1>), g, dim3(256), 0, s, a);
    else if (nl == 2) hipLaunchKernelGGL((k_enc_strip<LF, 4, 2>), g, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_enc_strip<LF, 4, 1>), g, dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  for (int p = 0; p < nplanes; p += p ? 2 : 1) {   // luma, then both chroma planes
    const int n = p ? 2 : 1;
    TileArgs a = {};
    a.p = p ? tile / 2 : tile;
    a.q = q;
    const bool strip = p < strips;
    if (strip && levels <= 2) continue;
    for (int k = 0; k < n; ++k) {
      a.src[k] = strip ? (const void*)wp[p + k] : src[p + k];
      a.dst[k] = dst[p + k];
    }
    a.levels = strip ? levels - 2 : levels;
    const hipError_t e = strip ? launch_tile<LF, V>(a.p / 4, n, n_tiles, a, s)
                               : launch_tile<LF, uint8_t>(a.p, n, n_tiles, a, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

size_t encode_workspace_bytes(int wavelet, int nplanes, int n_tiles, int tile, int levels) {
  if (tile < 256 || levels <= 2) return 0;
  const size_t v = wavelet == WV_W53 ? sizeof(int) : sizeof(double);
  const size_t luma = (size_t)n_tiles * (tile / 4) * (tile / 4) * v;
  return tile == 512 && nplanes == 3 ? luma * 3 / 2 : luma;
}

hipError_t launch_encode(int wavelet, int nplanes, int n_tiles, int tile, int levels, int qstep,
                         const void* const* src, void* const* dst, void* ws, int* overflow, hipStream_t s) {
  if (wavelet == WV_W53)
    return launch_encode_t<Enc53>(nplanes, n_tiles, tile, levels, qstep, src, dst, ws, overflow, s);
  return launch_encode_t<Enc97>(nplanes, n_tiles, tile, levels, qstep, src, dst, ws, overflow, s);
}

}  // namespace wv
