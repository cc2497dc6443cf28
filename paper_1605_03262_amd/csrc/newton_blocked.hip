// Blocked LU and triangular solves of the Newton matrices I - h gamma J with
// more than 64 species (gfx950).
//
//  lu    : one workgroup per state.  The matrix is column-major, so that a
//          wavefront's lanes hold consecutive rows in every access of the
//          panel, of the trailing matrix and of the triangular solves.
//  solve : one wavefront per state, lane l holding rows l, l + 64, ...
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "newton_blocked.hpp"

namespace pyjac {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// 16x16x4 matrix-core products.  Both precisions take A[row = lane % 16][k =
// lane / 16] and B[k = lane / 16][col = lane % 16]; the result slot v of lane
// l holds column l % 16 and row row(l / 16, v), which differs between the FP32
// and the FP64 instruction (checked on gfx950 with one-hot operands).
template <typename T> struct Mfma;
template <> struct Mfma<float> {
  typedef floatx4 acc_t;
  __device__ static acc_t run(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int q, int v) { return 4 * q + v; }
};
template <> struct Mfma<double> {
  typedef doublex4 acc_t;
  __device__ static acc_t run(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int q, int v) { return q + 4 * v; }
};

// Compile-time loop: f(std::integral_constant<int, j>) for j in [B, E), so
// that register arrays are only ever indexed by constants.
template <int B, int E, typename F>
__device__ __forceinline__ void sfor(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    sfor<B + 1, E>(f);
  }
}

__device__ __forceinline__ unsigned mag_key(double v) {
  return (unsigned)((unsigned long long)__double_as_longlong(v) >> 32) & 0x7FFFFFFFu;
}
__device__ __forceinline__ unsigned mag_key(float v) { return (unsigned)__float_as_int(v) & 0x7FFFFFFFu; }

__device__ __forceinline__ double read_lane(double v, int lane) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float read_lane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// ---------------------------------------------------------------- LU
// Right-looking LU with partial pivoting in panels of NB columns; thread t is
// row position t (N <= NT).
//  1. Panel: every thread keeps its row of the panel in registers.  One step
//     per column: the largest |a| of each wavefront (compared on the high 32
//     bits of the FP64 pattern or the FP32 pattern, which order non-negative
//     values) writes its row to LDS, and after ONE barrier every thread takes
//     the best of them and eliminates (two LDS buffers in turn).  Rows are not
//     exchanged meanwhile.
//  2. The pivot rows move to the top of the panel and the rows they displace
//     to the places left, in every column at once: at most 2 NB values per
//     column, read and written by NB neighbouring lanes.
//  3. U12 = L11^-1 A12, one column per thread, in LDS.
//  4. Trailing matrix A22 -= L21 U12 on the matrix cores, transposed (the
//     instruction's rows are matrix columns), so that 16 lanes address 16
//     consecutive rows of a column.  L21 comes from memory (just written, so
//     from cache), U12 from LDS.
// What bounds it: the chain of a panel's steps (wavefront maximum, barrier,
// reciprocal, update) at 111 rows; at 360 rows also the trailing matrix, read
// and written once per panel, which is why a panel has 32 columns as far as
// U12 leaves room in LDS.  4,099 FP64 systems of 360 rows take 15.4 ms and
// 4,003 of 111 rows 0.75 ms, against 55.6 and 3.18 ms for panels of 16 columns
// kept in LDS with a workgroup-wide search, about ten barriers per column.
template <typename T> constexpr int lu_ps(int NB) { return NB + 16 / (int)sizeof(T); }   // LDS row of U12: no bank conflicts

template <typename T, int NT, int NB>
size_t lu_lds(int N) {
  const size_t up = N > NB ? (size_t)((N - NB + 15) / 16 * 16) : 0;
  return (up * lu_ps<T>(NB) + NB * NB + 2 * (NT / 64) * NB) * sizeof(T) + (4 * (NT / 64) + 3 * NB + NT + 4) * sizeof(int);
}

template <typename T, int NT, int NB>
__global__ __launch_bounds__(NT, NT >= 1024 ? 4 : 2) void lu_kernel(int N, int64_t n, T* __restrict__ Aall,
                                                                   int* __restrict__ pivall,
                                                                   const int* __restrict__ list,
                                                                   const int* __restrict__ count,
                                                                   int* __restrict__ status, int sing_code) {
  extern __shared__ __align__(16) char smem[];
  constexpr int NW = NT / 64, PS = lu_ps<T>(NB);
  const int64_t slot = blockIdx.x;
  const int64_t lim = count ? *count : n;
  if (slot >= lim) return;
  const int64_t st = list ? list[slot] : slot;
  if (status[st] == -3) return;
  T* A = Aall + slot * (int64_t)N * N;
  const int t = threadIdx.x, lane = t % 64, wave = t / 64;
  const int up = N > NB ? (N - NB + 15) / 16 * 16 : 0;
  T* Us = reinterpret_cast<T*>(smem);           // [up][PS]: U12, column by column
  T* Lt = Us + (size_t)up * PS;                 // [NB][NB]: L11 transposed
  T* cand = Lt + NB * NB;                       // [2][NW][NB]: pivot row candidates
  int* ckey = reinterpret_cast<int*>(cand + 2 * NW * NB);   // [2][NW]
  int* cpos = ckey + 2 * NW;                    // [2][NW]
  int* pvp = cpos + 2 * NW;                     // [NB] row position of each pivot of the panel
  int* dl = pvp + NB;                           // displaced rows' positions ...
  int* vl = dl + NB;                            // ... and where they go
  int* prm = vl + NB;                           // [NT] matrix row at each position
  int* nmv = prm + NT;                          // number of displaced rows
  int orig = t;
  bool sing = false;
  for (int k0 = 0; k0 < N; k0 += NB) {
    const int nb = min(NB, N - k0), W = N - k0 - nb;
    const bool inp = t >= k0 && t < N;
    T a[NB];
    sfor<0, NB>([&](auto j) { a[j] = (inp && j < nb) ? A[(int64_t)(k0 + j) * N + t] : T(0); });
    bool act = inp;
    int step = -1;
    sfor<0, NB>([&](auto c) {
      if (c < nb) {
        constexpr int buf = decltype(c)::value & 1;
        const unsigned key = act ? mag_key(a[c]) + 1u : 0u;
        const unsigned mk = __ockl_wfred_max_u32(key);
        const int p = (int)__builtin_ctzll(__ballot(key == mk));
        if (lane == p) {
          T* dst = cand + (buf * NW + wave) * NB;
          sfor<decltype(c)::value, NB>([&](auto j) { dst[j] = a[j]; });
          ckey[buf * NW + wave] = (int)mk;
          cpos[buf * NW + wave] = t;
        }
        __syncthreads();
        unsigned best = (unsigned)ckey[buf * NW];
        int bw = 0;
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          const unsigned k = (unsigned)ckey[buf * NW + w];
          if (k > best) { best = k; bw = w; }
        }
        const int pr = cpos[buf * NW + bw];
        const T* prow = cand + (buf * NW + bw) * NB;
        const T piv = prow[c];
        const T inv = piv != T(0) ? T(1) / piv : T(0);
        sing = sing || !(fabs(piv) > T(0));
        if (act && t == pr) {
          act = false;
          step = c;
        }
        const T l = act ? a[c] * inv : T(0);
        a[c] = act ? l : a[c];
        sfor<decltype(c)::value + 1, NB>([&](auto j) { a[j] = fma(-l, prow[j], a[j]); });
      }
    });
    // the panel's pivots go to positions k0 .. k0 + nb - 1 in pivot order; the
    // other rows that were there go, in order, to the positions left
    if (step >= 0) pvp[step] = t;
    __syncthreads();
    int rank = 0;
    if (wave == k0 / 64) {            // holds positions k0 .. k0 + nb - 1 (NB divides 64)
      const int c = t - k0;
      const bool in = c >= 0 && c < nb;
      const unsigned long long below = (1ull << lane) - 1ull;
      const unsigned long long md = __ballot(in && step < 0);
      rank = __popcll(md & below);
      if (in && step < 0) dl[rank] = t;
      const int pp = in ? pvp[c] : 0;
      const bool vac = in && pp >= k0 + nb;
      const unsigned long long mv = __ballot(vac);
      if (vac) vl[__popcll(mv & below)] = pp;
      if (lane == 0) *nmv = __popcll(md);
    }
    __syncthreads();
    const int nm = *nmv;
    if (inp) {
      const int np = step >= 0 ? k0 + step : (t < k0 + nb ? vl[rank] : t);
      sfor<0, NB>([&](auto j) {
        if (j < nb) A[(int64_t)(k0 + j) * N + np] = a[j];
      });
      prm[np] = orig;
      if (step >= 0)
        sfor<0, NB>([&](auto j) {
          if (j < step) Lt[j * NB + step] = a[j];
        });
    }
    // the same exchange in the other columns, four at a time; the pivot rows
    // of the trailing columns go to LDS
    {
      const int c = t % NB, cols = N - nb;
      constexpr int STEP = NT / NB, UN = 4;
      const int pc = c < nb ? pvp[c] : 0, dc = c < nm ? dl[c] : 0, vc = c < nm ? vl[c] : 0;
      for (int col0 = t / NB; col0 < cols; col0 += STEP * UN) {
        T v[UN], d[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int col = col0 + u * STEP;
          const T* base = A + (int64_t)(col < k0 ? col : col + nb) * N;
          v[u] = (col < cols && c < nb) ? base[pc] : T(0);
          d[u] = (col < cols && c < nm) ? base[dc] : T(0);
        }
        // every lane's reads of these columns are done before any write
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int col = col0 + u * STEP;
          if (col < cols) {
            T* base = A + (int64_t)(col < k0 ? col : col + nb) * N;
            if (c < nb) {
              if (col < k0) base[k0 + c] = v[u];
              else Us[(size_t)(col - k0) * PS + c] = v[u];
            }
            if (c < nm) base[vc] = d[u];
          }
        }
      }
    }
    __syncthreads();
    if (inp) orig = prm[t];
    if (W <= 0) break;
    // U12, one column per thread; rows up to a multiple of 16 columns are zero
    const int Wp = (W + 15) / 16 * 16;
    if (t < Wp) {
      T u[NB];
      T* row = Us + (size_t)t * PS;
      sfor<0, NB>([&](auto c) { u[c] = t < W ? row[c] : T(0); });
      sfor<0, NB>([&](auto s) {
        sfor<decltype(s)::value + 1, NB>([&](auto c) { u[c] = fma(-Lt[s * NB + c], u[s], u[c]); });
      });
      sfor<0, NB>([&](auto c) { row[c] = u[c]; });
    }
    __syncthreads();
    for (int e = t; e < W * NB; e += NT) A[(int64_t)(k0 + NB + e / NB) * N + k0 + e % NB] = Us[(size_t)(e / NB) * PS + e % NB];
    // trailing update: a row tile and up to CT column tiles per wavefront
    {
      constexpr int CT = 4, KS = NB / 4;
      const int tr = (W + 15) / 16, ncb = (tr + CT - 1) / CT, r16 = lane % 16, q = lane / 16, o = k0 + NB;
      for (int it = wave; it < tr * ncb; it += NW) {
        const int rt = it / ncb, cb = it % ncb;
        const int p = o + rt * 16 + r16;
        const bool pok = p < N;
        typename Mfma<T>::acc_t acc[CT];
        T b[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) b[k] = pok ? -A[(int64_t)(k0 + 4 * k + q) * N + p] : T(0);
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int col = o + (cb * CT + u) * 16 + Mfma<T>::row(q, v);
            acc[u][v] = (pok && col < N) ? A[(int64_t)col * N + p] : T(0);
          }
#pragma unroll
        for (int u = 0; u < CT; ++u) {
          const int ct = cb * CT + u;
          if (ct < tr) {
            const T* us = Us + (size_t)(ct * 16 + r16) * PS + q;
#pragma unroll
            for (int k = 0; k < KS; ++k) acc[u] = Mfma<T>::run(us[4 * k], b[k], acc[u]);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int col = o + ct * 16 + Mfma<T>::row(q, v);
              if (pok && col < N) A[(int64_t)col * N + p] = acc[u][v];
            }
          }
        }
      }
    }
    __syncthreads();
  }
  if (t < N) pivall[slot * (int64_t)N + t] = orig;
  if (t == 0 && sing) status[st] = sing_code;
}

// ---------------------------------------------------------------- solve
// One wavefront per state, four states per workgroup (no barrier: each
// wavefront goes at its own pace).  Lane l holds rows l, l + 64, ...; step k
// of the forward sweep broadcasts y_k (v_readlane) and subtracts column k of
// L, 512 contiguous bytes per load, and the backward sweep does the same with
// U.  Columns are read in blocks of CB, one block ahead of their use (CB and
// the wavefronts per SIMD such that both blocks stay in registers).  Bound by
// reading the factor once: 98 us for 4,003 FP64 systems of 111 rows (4.0 TB/s;
// 311 us with a reduction over the wavefront and a barrier per row) and 915 us
// for 4,099 of 360 rows (4.6 TB/s; 1,779 us).
template <typename T, int R, bool REFINE>
__global__ __launch_bounds__(256, R * sizeof(T) <= 16 ? 3 : 2) void solve_kernel(int N, int64_t n, int64_t ld, const T* __restrict__ Aall,
                                                    const int* __restrict__ pivall, const double* __restrict__ rhs,
                                                    const double* __restrict__ rbuf, double* __restrict__ xs,
                                                    double* __restrict__ xout, const int* __restrict__ list,
                                                    const int* __restrict__ count, int* __restrict__ status,
                                                    int sweep, double rtol, double* __restrict__ dprev) {
  const bool first = !REFINE || sweep == 0;           // right-hand side as given
  constexpr int CB = R * sizeof(T) <= 16 ? 8 : R * sizeof(T) <= 48 ? 4 : 2;
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const int64_t slot = (int64_t)blockIdx.x * 4 + wv;
  const int64_t lim = count ? *count : n;
  if (slot >= lim) return;
  const int64_t st = list ? list[slot] : slot;
  const int s0 = status[st];
  if (REFINE ? s0 != ST_UNSET : (s0 == -3 || s0 == -1 || s0 == ST_SING32)) return;
  const T* A = Aall + slot * (int64_t)N * N;
  const int* piv = pivall + slot * (int64_t)N;
  T b[R], rd[R], dg[R];
  sfor<0, R>([&](auto i) {
    const int r = lane + 64 * i;
    b[i] = T(0);
    dg[i] = T(1);
    if (r < N) {
      const int64_t row = piv[r];
      b[i] = first ? (T)rhs[row * ld + st] : (T)rbuf[row * n + st];
      dg[i] = A[(int64_t)r * N + r];
    }
    rd[i] = T(1) / dg[i];
  });
  // forward: unit lower
  sfor<0, R>([&](auto S) {
    constexpr int s = decltype(S)::value, RS = R - s;
    const int nk = min(64, N - 64 * s);
    T buf[2][RS][CB];
    auto load = [&](T (&f)[RS][CB], int kb) {
      sfor<0, CB>([&](auto j) {
        const int kk = kb + j;
        const T* col = A + (int64_t)(64 * s + kk) * N + lane + 64 * s;
        sfor<0, RS>([&](auto i) {
          f[i][j] = (kk < nk && lane + 64 * (s + i) < N && (i > 0 || lane > kk)) ? col[64 * i] : T(0);
        });
      });
    };
    auto apply = [&](const T (&f)[RS][CB], int kb) {
      sfor<0, CB>([&](auto j) {
        const T y = read_lane(b[s], (kb + j) & 63);
        sfor<0, RS>([&](auto i) { b[s + i] = fma(-f[i][j], y, b[s + i]); });
      });
    };
    load(buf[0], 0);
    for (int kb = 0; kb < nk; kb += 2 * CB) {
      load(buf[1], kb + CB);
      apply(buf[0], kb);
      load(buf[0], kb + 2 * CB);
      apply(buf[1], kb + CB);
    }
  });
  // backward: upper
  sfor<0, R>([&](auto S) {
    constexpr int s = R - 1 - decltype(S)::value, RS = s + 1;
    const int nk = min(64, N - 64 * s);
    T buf[2][RS][CB];
    const int kt = (nk + 2 * CB - 1) / (2 * CB) * (2 * CB);      // steps nk .. kt - 1 read nothing and change nothing
    auto load = [&](T (&f)[RS][CB], int kb) {                    // columns kb + CB - 1 down to kb
      sfor<0, CB>([&](auto j) {
        const int kk = kb + CB - 1 - j;
        const T* col = A + (int64_t)(64 * s + kk) * N + lane;
        sfor<0, RS>([&](auto i) { f[i][j] = (kk >= 0 && kk < nk && (i < s || lane < kk)) ? col[64 * i] : T(0); });
      });
    };
    auto apply = [&](const T (&f)[RS][CB], int kb) {
      sfor<0, CB>([&](auto j) {
        const int kk = kb + CB - 1 - j;
        // x_k = b_k / u_kk, the reciprocal's rounding corrected
        T x = b[s] * rd[s];
        const T e = fma(-dg[s], x, b[s]);
        const T xc = fma(e, rd[s], x);
        x = isfinite(xc) ? xc : x;
        const T xk = read_lane(x, kk & 63);
        if (lane == kk) b[s] = x;
        sfor<0, RS>([&](auto i) { b[i] = fma(-f[i][j], xk, b[i]); });
      });
    };
    load(buf[0], kt - CB);
    for (int kb = kt - CB; kb > 0; kb -= 2 * CB) {
      load(buf[1], kb - CB);
      apply(buf[0], kb);
      load(buf[0], kb - 2 * CB);
      apply(buf[1], kb - CB);
    }
  });
  bool fin = true;
  if constexpr (!REFINE) {
    sfor<0, R>([&](auto i) {
      const int r = lane + 64 * i;
      if (r < N) {
        xout[(int64_t)r * ld + st] = (double)b[i];
        fin = fin && isfinite((double)b[i]);
      }
    });
    fin = __all(fin);
    if (lane == 0 && s0 == ST_UNSET) status[st] = fin ? 0 : -1;
    return;
  }
  double dmax = 0.0, xmax = 0.0, xv[R];
  sfor<0, R>([&](auto i) {
    const int r = lane + 64 * i;
    xv[i] = 0.0;
    if (r < N) {
      const double d = (double)b[i];
      xv[i] = first ? d : xs[(int64_t)r * n + st] + d;
      xs[(int64_t)r * n + st] = xv[i];
      dmax = fmax(dmax, fabs(d));
      xmax = fmax(xmax, fabs(xv[i]));
      fin = fin && isfinite(xv[i]);
    }
  });
  if (first) return;
  for (int o = 32; o > 0; o >>= 1) {
    dmax = fmax(dmax, __shfl_xor(dmax, o));
    xmax = fmax(xmax, __shfl_xor(xmax, o));
  }
  fin = __all(fin);
  // converged when the correction is below rtol of the solution, or when
  // the contraction rho of the last two corrections (refinement converges
  // linearly) predicts the remaining error rho / (1 - rho) |d| below it
  const double dp = sweep >= 2 ? dprev[st] : 0.0;
  const double rho = dp > 0.0 ? dmax / dp : 1.0;
  const bool conv = fin && (dmax <= rtol * xmax || (rho < 0.5 && rho * dmax <= rtol * xmax * (1.0 - rho)));
  if (lane == 0) {
    if (conv) status[st] = sweep;
    dprev[st] = dmax;
  }
  if (conv)
    sfor<0, R>([&](auto i) {
      const int r = lane + 64 * i;
      if (r < N) xout[(int64_t)r * ld + st] = xv[i];
    });
}

template <typename T, int NT, int NB>
hipError_t launch_lu_t(int N, int64_t n, T* A, int* piv, const int* list, const int* count, int* status,
                       int sing_code, hipStream_t st) {
  const size_t lds = lu_lds<T, NT, NB>(N);
  auto k = lu_kernel<T, NT, NB>;
  const hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3((unsigned)n), dim3(NT), lds, st, N, n, A, piv, list, count, status, sing_code);
  return hipGetLastError();
}

template <typename T, bool REFINE>
hipError_t launch_solve(int N, int64_t n, int64_t ld, const T* A, const int* piv, const double* rhs,
                        const double* rbuf, double* xs, double* xout, const int* list, const int* count, int* status,
                        int sweep, double rtol, double* dprev, hipStream_t st) {
#define PYJAC_SOLVE(r)                                                                                              \
  if (N <= 64 * r) {                                                                                                \
    hipLaunchKernelGGL((solve_kernel<T, r, REFINE>), dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, N, n, ld, A,  \
                       piv, rhs, rbuf, xs, xout, list, count, status, sweep, rtol, dprev);                          \
    return hipGetLastError();                                                                                       \
  }
  PYJAC_SOLVE(2)
  PYJAC_SOLVE(3)
  PYJAC_SOLVE(4)
  PYJAC_SOLVE(6)
  PYJAC_SOLVE(8)
  PYJAC_SOLVE(10)
#undef PYJAC_SOLVE
  return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t launch_lu(int N, int64_t n, T* A, int* piv, const int* list, const int* count, int* status, int sing_code,
                     hipStream_t st) {
  if (N <= 128) return launch_lu_t<T, 128, 32>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= 256) return launch_lu_t<T, 256, 32>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= 512) return launch_lu_t<T, 512, 32>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= kBlockedMax) return launch_lu_t<T, 1024, 16>(N, n, A, piv, list, count, status, sing_code, st);
  return hipErrorInvalidValue;
}
template hipError_t launch_lu<float>(int, int64_t, float*, int*, const int*, const int*, int*, int, hipStream_t);
template hipError_t launch_lu<double>(int, int64_t, double*, int*, const int*, const int*, int*, int, hipStream_t);

template <typename T>
hipError_t launch_solve_direct(int N, int64_t n, int64_t ld, const T* A, const int* piv, const double* rhs,
                               double* xout, const int* list, const int* count, int* status, hipStream_t st) {
  return launch_solve<T, false>(N, n, ld, A, piv, rhs, nullptr, nullptr, xout, list, count, status, 0, 0.0, nullptr, st);
}
template hipError_t launch_solve_direct<double>(int, int64_t, int64_t, const double*, const int*, const double*,
                                                double*, const int*, const int*, int*, hipStream_t);

hipError_t launch_solve_refine(int N, int64_t n, int64_t ld, const float* A, const int* piv, const double* rhs,
                               const double* rbuf, double* xs, double* xout, int* status, int sweep, double rtol,
                               double* dprev, hipStream_t st) {
  return launch_solve<float, true>(N, n, ld, A, piv, rhs, rbuf, xs, xout, nullptr, nullptr, status, sweep, rtol, dprev,
                                   st);
}

}  // namespace pyjac
