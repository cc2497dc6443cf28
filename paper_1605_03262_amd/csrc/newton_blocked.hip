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

// The bits of |v|, which order as the magnitudes do.
__device__ __forceinline__ unsigned long long mag_key(double v) {
  return (unsigned long long)__double_as_longlong(v) & 0x7FFFFFFFFFFFFFFFull;
}
__device__ __forceinline__ unsigned mag_key(float v) { return (unsigned)__float_as_int(v) & 0x7FFFFFFFu; }

// The first lane that holds the wavefront's largest key; of 64-bit keys the low
// halves are looked at where several lanes share the largest high half.
__device__ __forceinline__ int first_max(unsigned key) {
  return (int)__builtin_ctzll(__ballot(key == __ockl_wfred_max_u32(key)));
}
__device__ __forceinline__ int first_max(unsigned long long key) {
  const unsigned hi = (unsigned)(key >> 32), mh = __ockl_wfred_max_u32(hi);
  unsigned long long m = __ballot(hi == mh);
  if (m & (m - 1)) {
    const unsigned lo = hi == mh ? (unsigned)key : 0u, ml = __ockl_wfred_max_u32(lo);
    m = __ballot(hi == mh && lo == ml);
  }
  return (int)__builtin_ctzll(m);
}

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
//     per column: the largest |a| of each wavefront goes to LDS; after a
//     barrier every wavefront sees whether its own is the largest (the first
//     of equal ones), and the winner's row, with the reciprocal of its pivot
//     (every thread has computed its own meanwhile), goes through LDS to all
//     threads, which eliminate.  Rows are not exchanged meanwhile.
//  2. The pivot rows move to the top of the panel and the rows they displace
//     to the places left.  In the columns to the right this is done with the
//     reads for U12; in the columns to the left it is put off to the end,
//     where every column block is read and written once (smap keeps each
//     panel's exchange).
//  3. U12 = L11^-1 A12, one column per thread, in LDS, CW columns at a time.
//  4. Trailing matrix A22 -= L21 U12 on the matrix cores, transposed (the
//     instruction's rows are matrix columns), so that 16 lanes address 16
//     consecutive rows of a column.  L21 comes from memory (just written, so
//     from cache), U12 from LDS.
// What bounds it: the chain of a panel's steps (wavefront maximum, barrier,
// update) at 111 rows; at 360 rows also the trailing matrix, read and written
// once per panel, which is why a panel has 32 columns as far as the registers
// allow.  1,024 FP64 systems of 360 rows take 3.94 ms (11 % of the FP64 matrix
// rate) and 4,003 of 111 rows 0.73 ms, against 4.51 and 0.82 ms with one
// candidate row per wavefront, the division after the barrier, and the left
// columns exchanged after every panel; FP32, 2.13 and 0.41 against 2.58 and
// 0.45 ms.
template <typename T> constexpr int lu_ps(int NB) { return NB + 16 / (int)sizeof(T); }   // LDS row of U12: no bank conflicts

// columns of U12 kept in LDS at a time
inline __host__ __device__ int lu_cols(int N, int NB, int CW) {
  const int up = N > NB ? (N - NB + 15) / 16 * 16 : 0;
  return up < CW ? up : CW;
}

// Least wavefronts per SIMD: three as far as 96 rows (4,003 FP64 systems of 80
// rows 0.383 ms, 0.465 ms with two); above, the registers for more loads in
// flight are worth more (111 rows 0.721 against 0.794 ms).
template <typename T, int NT, int CW>
constexpr int lu_waves() { return NT >= 1024 ? 4 : CW <= 64 ? 3 : sizeof(T) == 8 && NT <= 256 ? 1 : 2; }

template <typename T, int NT, int NB, int CW>
size_t lu_lds(int N) {
  const size_t panels = (N + NB - 1) / NB;
  return ((lu_cols(N, NB, CW) + 1) * lu_ps<T>(NB) + NB * NB) * sizeof(T) + NT / 64 * sizeof(unsigned long long) +
         (5 * NB + NT + 1) * sizeof(int) + panels * N * sizeof(unsigned short);
}

// 1 / x by the hardware estimate and Newton steps; by division near the ends
// of the range of the exponents; 0 of a zero.
__device__ __forceinline__ double recip(double x) {
  const double e = __builtin_amdgcn_rcp(x);
  double r = fma(e, fma(-x, e, 1.0), e);
  r = fma(r, fma(-x, r, 1.0), r);
  if (x != 0.0 && !(fabs(x) > 0x1p-1000 && fabs(x) < 0x1p1000)) r = 1.0 / x;
  return x != 0.0 ? r : 0.0;
}
__device__ __forceinline__ float recip(float x) {
  const float e = __builtin_amdgcn_rcpf(x);
  float r = fmaf(e, fmaf(-x, e, 1.0f), e);
  if (x != 0.0f && !(fabsf(x) > 0x1p-120f && fabsf(x) < 0x1p120f)) r = 1.0f / x;
  return x != 0.0f ? r : 0.0f;
}

// Marks every entry of a register array as modified (no code emitted): what
// was loaded into it is there before anything after this is stored.
template <int J, int NM, typename T>
__device__ __forceinline__ void opaque_regs(T (&a)[NM]) {
  if constexpr (J < NM) {
    __asm__ volatile("" : "+v"(a[J])::"memory");
    opaque_regs<J + 1, NM>(a);
  }
}

template <typename T, int NT, int NB, int CW>
__global__ __launch_bounds__(NT, (lu_waves<T, NT, CW>())) void lu_kernel(int N, int64_t n, T* __restrict__ Aall,
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
  const int uc = lu_cols(N, NB, CW);
  T* Us = reinterpret_cast<T*>(smem);           // [uc][PS]: U12, column by column
  T* Lt = Us + (size_t)uc * PS;                 // [NB][NB]: L11 transposed
  T* prow = Lt + NB * NB;                       // [PS]: pivot row, 1 / pivot at [NB]
  typedef decltype(mag_key(T())) key_t;
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(prow + PS);
  key_t* wkey = reinterpret_cast<key_t*>(keys); // [NW] largest key of each wavefront
  int* pvp = reinterpret_cast<int*>(keys + NW); // [NB] row position of each pivot of the panel
  int* dl = pvp + NB;                           // displaced rows' positions ...
  int* vl = dl + NB;                            // ... and where they go
  int* newp = vl + NB;                          // [NB] the same by position in the panel
  int* taken = newp + NB;                       // [NB] 1: the row at this place of the panel is a pivot
  int* prm = taken + NB;                        // [NT] matrix row at each position
  int* nmv = prm + NT;                          // number of displaced rows
  unsigned short* smap = reinterpret_cast<unsigned short*>(nmv + 1);   // [panels][N] position before the panel's exchange
  int orig = t;
  bool sing = false;
  for (int k0 = 0; k0 < N; k0 += NB) {
    const int nb = min(NB, N - k0), W = N - k0 - nb, o = k0 + NB;
    const bool inp = t >= k0 && t < N;
    bool act = inp;
    int step = -1;
    T a[NB];
    {
      const T* src = A + (int64_t)k0 * N + min(t, N - 1);
      sfor<0, NB>([&](auto j) { a[j] = src[min((int)j, nb - 1) * N]; });
    }
    sfor<0, NB>([&](auto c) {
      if (c < nb) {
        const key_t key = act ? mag_key(a[c]) + 1u : key_t(0);
        const T rc = recip(a[c]);
        const bool first = lane == first_max(key);
        if (first) wkey[wave] = key;
        __syncthreads();
        const int w = min(lane, NW - 1);
        const key_t mine = wkey[wave], other = wkey[w];
        const bool me = __ballot(other > mine || (other == mine && w < wave)) == 0 && first;
        if (me) {
          sfor<decltype(c)::value, NB>([&](auto j) { prow[j] = a[j]; });
          prow[NB] = rc;
        }
        __syncthreads();
        const T inv = prow[NB];
        sing = sing || !(fabs(prow[c]) > T(0));
        if (me) {
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
    if (wave == 0) {
      const bool in = lane < nb;
      const unsigned long long below = (1ull << lane) - 1ull;
      if (in) taken[lane] = 0;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      const int pp = in ? pvp[lane] : 0;
      const bool vac = in && pp >= k0 + nb;
      if (in && !vac) taken[pp - k0] = 1;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      const bool disp = in && taken[lane] == 0;
      const unsigned long long md = __ballot(disp), mv = __ballot(vac);
      const int rank = __popcll(md & below);
      if (disp) dl[rank] = k0 + lane;
      if (vac) vl[__popcll(mv & below)] = pp;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      if (disp) newp[lane] = vl[rank];
      if (lane == 0) *nmv = __popcll(md);
    }
    __syncthreads();
    const int nm = *nmv;
    unsigned short* map = smap + (size_t)(k0 / NB) * N;
    if (inp) {
      const int np = step >= 0 ? k0 + step : (t < k0 + nb ? newp[t - k0] : t);
      sfor<0, NB>([&](auto j) {
        if (j < nb) A[(int64_t)(k0 + j) * N + np] = a[j];
      });
      prm[np] = orig;
      map[np] = (unsigned short)t;
      if (step >= 0)
        sfor<0, NB>([&](auto j) {
          if (j < step) Lt[j * NB + step] = a[j];
        });
    } else if (t < N) {
      map[t] = (unsigned short)t;
    }
    for (int ch = 0; ch < W; ch += uc) {          // columns o + ch .. of the trailing matrix
      const int Wc = min(uc, W - ch);
      T* Ac = A + (int64_t)(o + ch) * N;
      // the same exchange in these columns, several at a time; the pivot rows go to LDS
      {
        constexpr int STEP = NT / NB, UN = lu_waves<T, NT, CW>() == 1 ? 12 : 4;
        const int c = t % NB, pc = pvp[c], dc = c < nm ? dl[c] : 0, vc = c < nm ? vl[c] : 0;
        for (int col0 = t / NB; col0 < Wc; col0 += STEP * UN) {
          T v[UN], d[UN];
#pragma unroll
          for (int u = 0; u < UN; ++u) {
            const T* base = Ac + (int64_t)min(col0 + u * STEP, Wc - 1) * N;
            v[u] = base[pc];
            d[u] = base[dc];
          }
          // every lane's reads of these columns are done before any write
          opaque_regs<0, UN>(v);
          opaque_regs<0, UN>(d);
#pragma unroll
          for (int u = 0; u < UN; ++u) {
            const int col = col0 + u * STEP;
            if (col < Wc) {
              Us[(size_t)col * PS + c] = v[u];
              if (c < nm) Ac[(int64_t)col * N + vc] = d[u];
            }
          }
        }
      }
      __syncthreads();
      // U12, one column per thread; rows up to a multiple of 16 columns are zero
      const int Wp = (Wc + 15) / 16 * 16;
      for (int col = t; col < Wp; col += NT) {
        T u[NB];
        T* row = Us + (size_t)col * PS;
        sfor<0, NB>([&](auto c) { u[c] = col < Wc ? row[c] : T(0); });
        sfor<0, NB>([&](auto s) {
          sfor<decltype(s)::value + 1, NB>([&](auto c) { u[c] = fma(-Lt[s * NB + c], u[s], u[c]); });
        });
        sfor<0, NB>([&](auto c) { row[c] = u[c]; });
      }
      __syncthreads();
      for (int e = t; e < Wc * NB; e += NT) Ac[(int64_t)(e / NB) * N + k0 + e % NB] = Us[(size_t)(e / NB) * PS + e % NB];
      // trailing update: a row tile and up to CT column tiles per wavefront.
      // Byte offsets into the matrix fit 32 bits (N <= kBlockedMax); a read
      // past the last column or row stays in the matrix and is not used.
      {
        constexpr int CT = 4, KS = NB / 4;
        const int tr = (W + 15) / 16, tc = (Wc + 15) / 16, ncb = (tc + CT - 1) / CT, r16 = lane % 16, q = lane / 16;
        char* Ab = reinterpret_cast<char*>(A);
        const unsigned cs = (unsigned)N * sizeof(T), top = (unsigned)(N * N - 1) * (unsigned)sizeof(T);
        const unsigned vs = cs * Mfma<T>::row(0, 1), qs = cs * Mfma<T>::row(1, 0);
        for (int it = wave; it < tr * ncb; it += NW) {
          const int rt = it / ncb, cb = it % ncb;
          const int p = o + rt * 16 + r16;
          const unsigned ro = (unsigned)p * (unsigned)sizeof(T), lo = (unsigned)(k0 + q) * cs + ro;
          const unsigned c0 = (unsigned)(o + ch + cb * CT * 16) * cs + q * qs + ro;
          typename Mfma<T>::acc_t acc[CT];
          T b[KS];
#pragma unroll
          for (int k = 0; k < KS; ++k) b[k] = *reinterpret_cast<const T*>(Ab + min(lo + 4 * k * cs, top));
#pragma unroll
          for (int u = 0; u < CT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][v] = *reinterpret_cast<const T*>(Ab + min(c0 + u * 16 * cs + v * vs, top));
#pragma unroll
          for (int u = 0; u < CT; ++u) {
            const int ct = cb * CT + u;
            if (ct < tc) {
              const T* us = Us + (size_t)(ct * 16 + r16) * PS + q;
#pragma unroll
              for (int k = 0; k < KS; ++k) acc[u] = Mfma<T>::run(-us[4 * k], b[k], acc[u]);
#pragma unroll
              for (int v = 0; v < 4; ++v)
                if (p < N && ct * 16 + Mfma<T>::row(q, v) < Wc)
                  *reinterpret_cast<T*>(Ab + (c0 + u * 16 * cs + v * vs)) = acc[u][v];
            }
          }
        }
      }
      __syncthreads();
    }
    if (W <= 0) __syncthreads();
    if (inp) orig = prm[t];
  }
  // the rows of L in their final order: the columns of panel p have seen the
  // exchanges of their own panel only
  int s = min(t, N - 1);
  for (int p = (N + NB - 1) / NB - 2; p >= 0; --p) {
    T v[NB];
    T* blk = A + (int64_t)(p * NB) * N;
    s = smap[(size_t)(p + 1) * N + s];
    sfor<0, NB>([&](auto j) { v[j] = blk[(int64_t)j * N + s]; });
    opaque_regs<0, NB>(v);
    __syncthreads();
    if (t >= (p + 1) * NB && t < N) sfor<0, NB>([&](auto j) { blk[(int64_t)j * N + t] = v[j]; });
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
  bool rdok = true;
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
    rdok = rdok && isfinite(rd[i]);
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
  // backward: upper.  A pivot whose reciprocal is not finite (below 2^-1024, in
  // FP32 2^-128) is divided by, in a plain loop.
  if (!__all(rdok)) sfor<0, R>([&](auto S) {
    constexpr int s = R - 1 - decltype(S)::value;
    for (int kk = min(64, N - 64 * s) - 1; kk >= 0; --kk) {
      const T* col = A + (int64_t)(64 * s + kk) * N + lane;
      const T x = b[s] / dg[s], xk = read_lane(x, kk);
      if (lane == kk) b[s] = x;
      sfor<0, s + 1>([&](auto i) {
        if (i < s || lane < kk) b[i] = fma(-col[64 * i], xk, b[i]);
      });
    }
  });
  else sfor<0, R>([&](auto S) {
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

template <typename T, int NT, int NB, int CW>
hipError_t launch_lu_t(int N, int64_t n, T* A, int* piv, const int* list, const int* count, int* status,
                       int sing_code, hipStream_t st) {
  const size_t lds = lu_lds<T, NT, NB, CW>(N);
  auto k = lu_kernel<T, NT, NB, CW>;
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
  // Columns of U12 at a time (1,024 systems of 360 rows): FP64, all of them
  // 3.94 ms, 192 4.11 ms; FP32, 96 2.13 ms, 192 2.49 ms.  600 rows: 128
  // 11.95 / 6.96 ms (512 systems, FP64 / FP32), 192 12.23 / 7.33 ms.
  constexpr bool f64 = sizeof(T) == 8;
  if (N <= 96) return launch_lu_t<T, 128, 32, 64>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= 128) return launch_lu_t<T, 128, 32, 96>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= 256) return launch_lu_t<T, 256, 32, 224>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= 512) return launch_lu_t<T, 512, 32, f64 ? 480 : 96>(N, n, A, piv, list, count, status, sing_code, st);
  if (N <= kBlockedMax) return launch_lu_t<T, 1024, 16, 128>(N, n, A, piv, list, count, status, sing_code, st);
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
