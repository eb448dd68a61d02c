// Whole-tile fused decode for tiles of 64, 32 and 16: one workgroup takes a
// tile, all its planes in LDS, through every step of the decode (and, in the
// GOP form, through the frames of a GOP in order).
//
// A small tile fits on chip whole, so nothing is computed twice: the block and
// strip kernels recompute a dependency cone per block, which at these sizes is
// larger than the block.  The kept coefficients are read once (those of the
// next frames while these are transformed), the levels run in place -- every
// line of a level is split over 8 threads, which read their samples into
// registers before any is written back -- then residual, clip, reference,
// colour and output on four adjacent samples per thread.  The reference stays
// in registers between the frames of a GOP and is read and written only at its
// ends.
// What bounds it: a workgroup per tile, so fewer tiles than CUs leave the others
// idle (100 of 256 CUs in the case below); on a CU instruction issue (two
// wavefronts per SIMD, about 5000 instructions for four frames of a 64-sample
// tile), then latency.
// GOP of 8 frames, 1920 x 1920 YUV420, 64-sample tiles, 5/3, four levels,
// 110 x 110 degree viewport (100 tiles): 39 us a call (block kernel, a launch per
// frame: 256).
#include <type_traits>

#include "wv_fused_common.h"

namespace wv {
namespace {

template <class T, int N>
struct alignas(sizeof(T) * N) Group { T v[N]; };

// N 32-bit words (Clang vectors load and store through address-space pointers).
template <int N>
struct Words { typedef uint32_t T __attribute__((ext_vector_type(N))); };
template <>
struct Words<1> { typedef uint32_t T; };

// Four clipped samples as they are stored (bytes by permutes, see pack4).
__device__ __forceinline__ Group<uint8_t, 4> pack(const int (&v)[4]) {
  return __builtin_bit_cast(Group<uint8_t, 4>, pack4(v[0], v[1], v[2], v[3]));
}
__device__ __forceinline__ Group<float, 4> pack(const float (&v)[4]) { return {{v[0], v[1], v[2], v[3]}}; }

// Four values at element e of a plane.
template <class G4, class T>
__device__ __forceinline__ G4 get(const WV_G T* p, unsigned e) {
  using U = Words<sizeof(G4) / 4>;
  return __builtin_bit_cast(G4, *(const WV_G typename U::T*)at(p, e));
}
template <class G4, class T>
__device__ __forceinline__ void put(WV_G T* p, unsigned e, const G4& v) {
  using U = Words<sizeof(G4) / 4>;
  *(WV_G typename U::T*)at(p, e) = __builtin_bit_cast(typename U::T, v);
}

// RGB of two horizontally adjacent samples, which share a chroma sample.
__device__ __forceinline__ void rgb_pair(int y0, int y1, int cb, int cr, int (&o)[3][4], int i) {
  // (Y << 16) + t >> 16 == Y + (t >> 16)
  cb -= 128;
  cr -= 128;
  const int t[3] = {(91881 * cr + 32768) >> 16, (-22554 * cb - 46802 * cr + 32768) >> 16,
                    (116130 * cb + 32768) >> 16};
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    o[p][i] = clip255(y0 + t[p]);
    o[p][i + 1] = clip255(y1 + t[p]);
  }
}
__device__ __forceinline__ void rgb_pair(float y0, float y1, float cb, float cr, float (&o)[3][4], int i) {
  to_rgb(y0, cb, cr, o[0][i], o[1][i], o[2][i]);
  to_rgb(y1, cb, cr, o[0][i + 1], o[1][i + 1], o[2][i + 1]);
}

// Pairs of output samples per thread along a line of a level of edge M: M / 16
// (8 threads a line), and at least the samples a run reads beyond its ends.
template <class LF>
constexpr int tile_pairs(int m) {
  return m >= 16 * LF::D_LO ? m / 16 : m >= 2 * LF::D_LO ? LF::D_LO : 1;
}

// The samples of output pairs k0 .. k0 + NP - 1 of line `line`.  From M = 8 on
// only the first and the last run of a line reach over its ends, by no more
// than their own length, so every sample is at a constant offset from the
// run's start, one for the run at the end and one for the others.
template <class LF, int M, int PITCH, bool ROWS, int NP>
__device__ __forceinline__ void line_load(const typename LF::V* buf, int line, int k0, typename LF::V (&s)[NP + LF::NS - 1],
                                          typename LF::V (&d)[NP + LF::ND - 1]) {
  constexpr int STEP = ROWS ? 1 : PITCH, H = M / 2;
  if constexpr (M >= 8) {
    static_assert(NP >= LF::D_LO && NP >= LF::D_HI && NP >= LF::S_HI, "runs reach one run over their ends");
    const typename LF::V* b = buf + (ROWS ? line * PITCH + k0 : k0 * PITCH + line);
    const bool first = k0 == 0, last = k0 == H - NP;
    static_for<0, NP + LF::NS - 1>([&](auto I) {
      constexpr int o = decltype(I)::value - LF::S_LO;   // s[-m] = s[m], s[H + m] = s[H - 1 - m]
      if constexpr (o < 0) s[I] = b[(first ? -o : o) * STEP];
      else if constexpr (o >= NP) s[I] = b[(last ? 2 * NP - 1 - o : o) * STEP];
      else s[I] = b[o * STEP];
    });
    static_for<0, NP + LF::ND - 1>([&](auto I) {
      constexpr int o = decltype(I)::value - LF::D_LO;   // d[-m] = d[m - 1], d[H + m] = d[H - 2 - m]
      if constexpr (o < 0) d[I] = b[(H + (first ? -o - 1 : o)) * STEP];
      else if constexpr (o >= NP) d[I] = b[(H + (last ? 2 * NP - 2 - o : o)) * STEP];
      else d[I] = b[(H + o) * STEP];
    });
  } else {
    // two (M = 4) or more (M = 2) reflections
    auto at = [&](int i) { return ROWS ? buf[line * PITCH + i] : buf[i * PITCH + line]; };
    auto ext = [](int j) { return M == 2 ? j & 1 : abs(j) < M ? abs(j) : abs(2 * M - 2 - abs(j)); };
#pragma unroll
    for (int i = 0; i < NP + LF::NS - 1; ++i) s[i] = at(ext(2 * (k0 - LF::S_LO + i)) >> 1);
#pragma unroll
    for (int i = 0; i < NP + LF::ND - 1; ++i) d[i] = at(H + (ext(2 * (k0 - LF::D_LO + i) + 1) >> 1));
  }
}
template <class V, int PITCH, bool ROWS, int NP>
__device__ __forceinline__ void line_store(V* buf, int line, int k0, const V (&x)[2 * NP]) {
  V* b = buf + (ROWS ? line * PITCH + 2 * k0 : 2 * k0 * PITCH + line);
#pragma unroll
  for (int i = 0; i < 2 * NP; ++i) b[i * (ROWS ? 1 : PITCH)] = x[i];
}

// One direction of one level of every plane of F frames: luma edge M, chroma
// edge M / 2 (threads of the lower half take Cb, the others Cr).  A frame's
// planes are YS (luma) and CS (both chroma planes) values apart.
template <class LF, int T, int M, bool YUV, bool ROWS, int F>
__device__ __forceinline__ void tile_pass(typename LF::V* y, typename LF::V* c) {
  using V = typename LF::V;
  constexpr int PY = T + 1, PC = T / 2 + 1, MC = M / 2, YS = T * PY, CS = T * PC;
  constexpr int NY = tile_pairs<LF>(M), NC = tile_pairs<LF>(MC), HT = 4 * T;
  // opaque: the passes' addresses are formed where they are used instead of
  // being kept in registers across the frames (one frame at a time, tiles of
  // 64: 181 -> 94 registers)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  V sy[F][NY + LF::NS - 1], dy[F][NY + LF::ND - 1], sc[F][NC + LF::NS - 1], dc[F][NC + LF::ND - 1];
  const int ly = tid % M, ky = tid / M * NY;
  const bool on_y = ky < M / 2;
  V* cp = c + (tid >= HT ? (T / 2) * PC : 0);
  const int lc = tid % MC, kc = tid % HT / MC * NC;
  const bool on_c = YUV && kc < MC / 2;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    if (on_y) line_load<LF, M, PY, ROWS, NY>(y + f * YS, ly, ky, sy[f], dy[f]);
    if (on_c) line_load<LF, MC, PC, ROWS, NC>(cp + f * CS, lc, kc, sc[f], dc[f]);
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < F; ++f) {
    if (on_y) {
      V x[2 * NY];
      LF::template run<NY>(sy[f], dy[f], x);
      line_store<V, PY, ROWS, NY>(y + f * YS, ly, ky, x);
    }
    if (on_c) {
      V x[2 * NC];
      LF::template run<NC>(sc[f], dc[f], x);
      line_store<V, PC, ROWS, NC>(cp + f * CS, lc, kc, x);
    }
  }
  __syncthreads();
}

// Levels n .. 1 of a region of edge M and below, coarsest first.
template <class LF, int T, int M, bool YUV, int F>
__device__ __forceinline__ void tile_levels(typename LF::V* y, typename LF::V* c, int n) {
  if constexpr (M >= (YUV ? 4 : 2)) {
    if (n <= 0) return;
    tile_levels<LF, T, M / 2, YUV, F>(y, c, n - 1);
    tile_pass<LF, T, M, YUV, true, F>(y, c);
    tile_pass<LF, T, M, YUV, false, F>(y, c);
  }
}

// F: frames transformed side by side (1: calls of one frame).
template <class LF, int FMT, int T, int F>
__global__ __launch_bounds__(8 * T) void k_tile(const WorkArgs a) {
  using V = typename LF::V;
  using CT = typename CoefT<LF>::T;
  using RT = typename CoefT<LF>::R;
  using C4 = Group<CT, 4>;
  using R4 = Group<RT, 4>;
  constexpr bool YUV = FMT == WV_YUV420;
  constexpr int C = T / 2, PY = T + 1, PC = C + 1, NT = 8 * T, YS = T * PY, CS = T * PC;
  constexpr int QY = T * T / 4, QC = YUV ? 2 * C * C / 4 : 0;   // groups of four samples
  constexpr int GY = QY / NT > 1 ? QY / NT : 1, GC = QC / NT > 1 ? QC / NT : 1;
  __shared__ V sy[F * YS];
  __shared__ V sc[YUV ? F * CS : 1];
  const int tid = threadIdx.x;
  const int it = xcd_remap(blockIdx.x, gridDim.x);
  const Item item = a.items_dev ? a.items_dev[it] : a.items[it];
  const int nf = a.n_frames > 0 ? a.n_frames : 1, drop = a.levels - item.lc;
  // the kept region: everything outside the top-left edge >> drop is zero
  const int ey = T >> drop, ec = C >> drop;
  auto job_of = [&](int f) -> const Job& {
    const int j = a.n_frames > 0 ? f : item.job;
    return a.jobs_dev ? a.jobs_dev[j] : a.jobs[j];
  };
  // this tile's part of a plane, in global memory (a generic pointer would
  // make every access a FLAT instruction)
  auto plane = [&](auto* p, int n) {
    using E = std::remove_pointer_t<decltype(p)>;
    return uniform((WV_G E*)p + (size_t)item.tile * n);
  };
  // group q of the luma plane: row, column; of the chroma planes: plane, row, column
  auto ypos = [&](int q, int& r, int& c) { r = 4 * q / T; c = 4 * q % T; };
  auto cpos = [&](int q, int& p, int& r, int& c) {
    p = q / (C * C / 4);
    const int e = 4 * (q % (C * C / 4));
    r = e / C;
    c = e % C;
  };
  auto y_has = [&](int q) { return QY % NT == 0 || q < QY; };
  auto c_has = [&](int q) { return QC % NT == 0 || q < QC; };
  auto cut = [&](C4& w, int c, int edge) {   // a kept edge (a power of two) inside the group
    if (edge < 4)
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (c + k >= edge) w.v[k] = CT(0);
  };
  C4 wy[F][GY], wc[F][GC];
  auto load = [&](int f0) {   // the coefficients of frames f0 .. f0 + F - 1
#pragma unroll
    for (int k = 0; k < F; ++k) {
      const bool have = F == 1 || f0 + k < nf;
      const Job& job = job_of(have ? f0 + k : f0);
      const WV_G CT* cp = plane((const CT*)job.coef[0], T * T);
      const WV_G CT* c1 = plane((const CT*)job.coef[1], C * C);
      const WV_G CT* c2 = plane((const CT*)job.coef[2], C * C);
#pragma unroll
      for (int g = 0; g < GY; ++g) {
        const int q = tid + g * NT;
        int r, c;
        ypos(q, r, c);
        wy[k][g] = C4{};
        if (have && y_has(q) && r < ey && c < ey) {
          wy[k][g] = get<C4>(cp, q * 4);
          cut(wy[k][g], c, ey);
        }
      }
      if constexpr (YUV)
#pragma unroll
        for (int g = 0; g < GC; ++g) {
          const int q = tid + g * NT;
          int p, r, c;
          cpos(q, p, r, c);
          wc[k][g] = C4{};
          if (have && c_has(q) && r < ec && c < ec) {
            wc[k][g] = get<C4>(p ? c2 : c1, r * C + c);
            cut(wc[k][g], c, ec);
          }
        }
    }
  };
  load(0);
  R4 ry[GY], rc[GC];   // the reference: this thread's samples
  for (int f0 = 0; f0 < nf; f0 += F) {
    const int n = min(F, nf - f0);
#pragma unroll
    for (int k = 0; k < F; ++k) {
      const int qs = job_of(k < n ? f0 + k : f0).qstep;
#pragma unroll
      for (int g = 0; g < GY; ++g) {
        const int q = tid + g * NT;
        int r, c;
        ypos(q, r, c);
        if (y_has(q))
#pragma unroll
          for (int i = 0; i < 4; ++i) sy[k * YS + r * PY + c + i] = deq(wy[k][g].v[i], qs);
      }
      if constexpr (YUV)
#pragma unroll
        for (int g = 0; g < GC; ++g) {
          const int q = tid + g * NT;
          int p, r, c;
          cpos(q, p, r, c);
          if (c_has(q))
#pragma unroll
            for (int i = 0; i < 4; ++i) sc[k * CS + p * C * PC + r * PC + c + i] = deq(wc[k][g].v[i], qs);
        }
    }
    // what arrives while the levels run: the first frame's reference, the
    // next frames' coefficients
    if (f0 == 0 && !(job_of(0).flags & kJobIntra)) {
      const Job& job = job_of(0);
      const WV_G RT* r0 = plane((const RT*)job.ref[0], T * T);
      const WV_G RT* r1 = plane((const RT*)job.ref[1], C * C);
      const WV_G RT* r2 = plane((const RT*)job.ref[2], C * C);
#pragma unroll
      for (int g = 0; g < GY; ++g) {
        const int q = tid + g * NT;
        if (y_has(q)) ry[g] = get<R4>(r0, q * 4);
      }
      if constexpr (YUV)
#pragma unroll
        for (int g = 0; g < GC; ++g) {
          const int q = tid + g * NT;
          int p, r, c;
          cpos(q, p, r, c);
          if (c_has(q))
            rc[g] = get<R4>(p ? r2 : r1, r * C + c);
        }
    }
    if (f0 + F < nf) load(f0 + F);
    __syncthreads();
    tile_levels<LF, T, T, YUV, F>(sy, sc, a.levels);
    // residual and clip, frame after frame; four samples each
    auto finish = [&](bool intra, R4& ref, const V* p, V (&v)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = clip255(p[i] + (intra ? V(0) : (V)ref.v[i]));
      ref = pack(v);
    };
    if constexpr (YUV) {
      for (int k = 0; k < n; ++k) {
        const Job& job = job_of(f0 + k);
        const bool intra = (job.flags & kJobIntra) != 0, last = f0 + k == nf - 1;
        WV_G RT* r1 = plane((RT*)job.ref[1], C * C);
        WV_G RT* r2 = plane((RT*)job.ref[2], C * C);
#pragma unroll
        for (int g = 0; g < GC; ++g) {
          const int q = tid + g * NT;
          int p, r, c;
          cpos(q, p, r, c);
          if (!c_has(q)) continue;
          V* px = sc + k * CS + p * C * PC + r * PC + c;
          V v[4];
          finish(intra, rc[g], px, v);
          if (last) put(p ? r2 : r1, r * C + c, rc[g]);
#pragma unroll
          for (int i = 0; i < 4; ++i) px[i] = v[i];
        }
      }
      __syncthreads();
    }
    for (int k = 0; k < n; ++k) {
      const Job& job = job_of(f0 + k);
      const bool intra = (job.flags & kJobIntra) != 0, last = f0 + k == nf - 1;
      const bool has_out = (job.flags & kJobHasOut) != 0;
      WV_G RT* r0 = plane((RT*)job.ref[0], T * T);
      WV_G RT* out = uniform((WV_G RT*)job.out + (size_t)item.slot * (YUV ? 3 : 1) * T * T);
#pragma unroll
      for (int g = 0; g < GY; ++g) {
        const int q = tid + g * NT;
        int r, c;
        ypos(q, r, c);
        if (!y_has(q)) continue;
        V y[4];
        finish(intra, ry[g], sy + k * YS + r * PY + c, y);
        if (last) put(r0, q * 4, ry[g]);
        if (!has_out) continue;
        if constexpr (YUV) {
          V o[3][4];
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            const V* c0 = sc + k * CS + (r >> 1) * PC + ((c + i) >> 1);
            rgb_pair(y[i], y[i + 1], c0[0], c0[C * PC], o, i);
          }
#pragma unroll
          for (int p = 0; p < 3; ++p) put(out, p * T * T + q * 4, pack(o[p]));
        } else {
          put(out, q * 4, ry[g]);
        }
      }
    }
    if (f0 + F < nf) __syncthreads();   // the planes are read before the next coefficients land
  }
}

template <class LF, int FMT, int F>
hipError_t launch_f(int tile, const WorkArgs& a, hipStream_t s) {
  const dim3 g(a.total), b(8 * tile);
  switch (tile) {
    case 64: hipLaunchKernelGGL((k_tile<LF, FMT, 64, F>), g, b, 0, s, a); break;
    case 32: hipLaunchKernelGGL((k_tile<LF, FMT, 32, F>), g, b, 0, s, a); break;
    case 16: hipLaunchKernelGGL((k_tile<LF, FMT, 16, F>), g, b, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Four frames at a time as soon as there are two: the transforms of a GOP's
// frames do not depend on each other, and four of them share the barriers of
// one (120 tiles of 64, GOP of 8: 61.8 us one at a time, 36 four at a time).
template <class LF, int FMT>
hipError_t launch_t(int tile, const WorkArgs& a, hipStream_t s) {
  if (a.total <= 0) return hipSuccess;
  return a.n_frames > 1 ? launch_f<LF, FMT, 4>(tile, a, s) : launch_f<LF, FMT, 1>(tile, a, s);
}

}  // namespace

hipError_t launch_tile(int wavelet, int format, int tile, const WorkArgs& a, hipStream_t s) {
  if (wavelet == WV_W53)
    return format == WV_YUV420 ? launch_t<Inv53, WV_YUV420>(tile, a, s) : launch_t<Inv53, WV_GRAY8>(tile, a, s);
  return format == WV_YUV420 ? launch_t<Inv97, WV_YUV420>(tile, a, s) : launch_t<Inv97, WV_GRAY8>(tile, a, s);
}

}  // namespace wv
