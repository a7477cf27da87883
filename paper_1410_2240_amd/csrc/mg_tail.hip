// The V(2,2) cycle on grids of 16^3 and below, by one workgroup (CDNA4).
//
// These grids hold less than a megabyte between them, so what they cost is latency: the
// loads of each half-sweep, a barrier after it, and the length of an update's chain.  The
// split follows from that.
//   16^3  Each of the 512 threads owns a 2 x 2 x 2 block, the children of one 8^3 cell.  It
//         holds the block's values, right-hand sides, faces, diagonals and their reciprocals
//         in registers for the whole cycle: nothing but the values of the three neighbours
//         outside the block is read in a half-sweep (12 LDS reads and 4 writes for 4
//         independent updates), and the restriction and prolongation are thread-local.
//   8^3   Each of 256 threads owns an x-pair, one cell of each colour, with the same things
//         in registers, or below a 16^3 grid in LDS; the values live in LDS.
//   4^3   The pseudo-inverse product, 8 threads to a row, its entries loaded at the start.
// All memory is read once, at the start, in one round of loads.  On the values of a 16^3
// grid rows are split by column parity and padded to 20 words, so that the neighbours of a
// wave's blocks fall in different banks.
//
// A cycle from 16^3 takes 12.4 us in FP64 and 10.7 us in FP32, launch included, and one
// from 8^3 7.6 us.  With a barrier-separated copy of the many-block kernels instead (each
// half-sweep reading its coefficients and six neighbours again) they took 26.1, 21.7 and
// 10.2 us.  The cycle's kernel has no spills (230 VGPRs in FP64).  The solve in one launch
// keeps more across its loop than there are registers: at 16^3 42 are spilled, most of them
// LDS offsets, about 30 loads a cycle.
#include "mg_kernels.h"
#include "mg_plan.h"

namespace mg {

namespace {

constexpr int kTailThreads = 512;
constexpr int kRow = 20;            // a 16-cell row: 8 even columns, 8 odd ones, 4 unused
constexpr int kPlane = 16 * kRow;

template <typename T>
struct Vec2of;
template <>
struct Vec2of<double> {
  using type = double2;
};
template <>
struct Vec2of<float> {
  using type = float2;
};

template <typename T>
__device__ __forceinline__ typename Vec2of<T>::type pair_at(const T* __restrict__ a, int c) {
  return *reinterpret_cast<const typename Vec2of<T>::type*>(a + c);
}

__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// gs_quotient in two parts: the reciprocal of a diagonal, kept for the whole cycle, and the
// quotient from it
__device__ __forceinline__ double diag_recip(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  return __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
}
__device__ __forceinline__ float diag_recip(float d) { return __builtin_amdgcn_rcpf(d); }
template <typename T>
__device__ __forceinline__ T quotient(T n, T d, T r) {
  const T q = n * r;
  return fma_t(fma_t(-d, q, n), r, q);
}

template <typename T, bool TOP16>
struct TailShared {
  T e0[TOP16 ? 16 * kPlane : 1];
  T e1[512], f1[512];
  T x[256];   // residuals of the 8^3 grid's pairs
  T e2[64];
  double fh[64];
  // what a thread's registers have no room for beside its block: each its own column
  double pinv[TOP16 ? 8 * kTailThreads : 1];
  T pair[TOP16 ? 8 : 1][2][TOP16 ? 256 : 1];   // faces, diagonal and reciprocal of its 8^3 pair
};

// One cell: faces, diagonal and its reciprocal, right-hand side (less its shift).
template <typename T>
struct TailCell {
  T xm, xp, ym, yp, zm, zp, D, r, f;
};

template <typename T, bool TOP16>
struct Tail {
  using V2 = typename Vec2of<T>::type;
  TailShared<T, TOP16>& s;
  const CoarseCycle<T>& a;
  const int tid;

  // the block of a 16^3 grid: [dz][dy][dx] values, faces by position along their direction
  T e[2][2][2], f[2][2][2], D[2][2][2], r[2][2][2];
  T fx[3][2][2], fy[3][2][2], fz[3][2][2];   // [x][dy][dz], [y][dx][dz], [z][dx][dy]
  unsigned live0 = 0;                        // bit dz 4 + dy 2 + dx: an active cell
  int o, oxm, oxp, oym, oyp, ozm, ozp;       // LDS offsets: the block, and to its neighbours
  // the pair of an 8^3 grid: cell of colour 0 and of colour 1
  TailCell<T> p1[TOP16 ? 1 : 2];   // (in LDS below a 16^3 grid)
  bool live1[2];
  int c1[2], xm1[2], xp1[2], ym1, yp1, zm1, zp1;
  double pv[TOP16 ? 1 : 8];
  bool act2 = false;

  static constexpr int L1 = TOP16 ? 1 : 0;   // the 8^3 grid's and the 4^3 grid's entry in a
  static constexpr int L2 = L1 + 1;

  __device__ Tail(TailShared<T, TOP16>& sh, const CoarseCycle<T>& args) : s(sh), a(args), tid(threadIdx.x) {}

  // every load of the cycle but the top grid's values
  __device__ __forceinline__ void load(T fs) {
    if constexpr (TOP16) {
      const int I = tid & 7, J = (tid >> 3) & 7, K = tid >> 6;
      const T* __restrict__ bx = a.bx[0];
      const T* __restrict__ by = a.by[0];
      const T* __restrict__ bz = a.bz[0];
      auto at = [](int i, int j, int k) { return (k << 8) + (j << 4) + i; };
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          const int c = at(2 * I, 2 * J + dy, 2 * K + dz);
          const V2 xv = pair_at(bx, c), fv = pair_at(a.f, c);
          fx[0][dy][dz] = xv.x;
          fx[1][dy][dz] = xv.y;
          fx[2][dy][dz] = bx[at((2 * I + 2) & 15, 2 * J + dy, 2 * K + dz)];
          f[dz][dy][0] = fv.x - fs;
          f[dz][dy][1] = fv.y - fs;
          const uchar2 mk = *reinterpret_cast<const uchar2*>(a.mask[0] + c);
          live0 |= (mk.x ? 1u : 0u) << (4 * dz + 2 * dy);
          live0 |= (mk.y ? 2u : 0u) << (4 * dz + 2 * dy);
        }
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const V2 v = pair_at(by, at(2 * I, (2 * J + b) & 15, 2 * K + dz));
          fy[b][0][dz] = v.x;
          fy[b][1][dz] = v.y;
        }
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          const bool in = 2 * K + c < 16;   // the top wall's face is 0, the bottom one's is stored as 0
          const V2 v = in ? pair_at(bz, at(2 * I, 2 * J + dy, 2 * K + c)) : V2{T(0), T(0)};
          fz[c][0][dy] = v.x;
          fz[c][1][dy] = v.y;
        }
      o = 2 * K * kPlane + 2 * J * kRow + I;
      oxm = 8 + ((I - 1) & 7) - I;          // column 2I-1, from column 2I
      oxp = ((I + 1) & 7) - I;              // column 2I+2, from column 2I
      oym = (((2 * J - 1) & 15) - 2 * J) * kRow;
      oyp = (((2 * J + 2) & 15) - 2 * J) * kRow;
      ozm = K > 0 ? -kPlane : 0;            // at a wall the cell itself: its face there is 0
      ozp = K < 7 ? 2 * kPlane : kPlane;
    }
    if (tid < 256) {
      const int ip = tid & 3, j = (tid >> 2) & 7, k = tid >> 5;
      const T* __restrict__ bx = a.bx[L1];
      const T* __restrict__ by = a.by[L1];
      const T* __restrict__ bz = a.bz[L1];
      ym1 = (((j - 1) & 7) - j) * 8;
      yp1 = (((j + 1) & 7) - j) * 8;
      zm1 = k > 0 ? -64 : 0;
      zp1 = k < 7 ? 64 : 0;
#pragma unroll
      for (int col = 0; col < 2; ++col) {
        const int i = 2 * ip + ((col + j + k) & 1);
        const int c = (k * 8 + j) * 8 + i;
        c1[col] = c;
        xm1[col] = c - i + ((i - 1) & 7);
        xp1[col] = c - i + ((i + 1) & 7);
        TailCell<T> q;
        q.xm = bx[c];
        q.xp = bx[xp1[col]];
        q.ym = by[c];
        q.yp = by[c + yp1];
        q.zm = bz[c];
        q.zp = k < 7 ? bz[c + 64] : T(0);
        live1[col] = a.mask[L1][c] != 0;
        q.D = q.xm + q.xp + q.ym + q.yp + q.zm + q.zp;
        q.r = diag_recip(q.D);
        if constexpr (TOP16) {
          const T v[8] = {q.xm, q.xp, q.ym, q.yp, q.zm, q.zp, q.D, q.r};
#pragma unroll
          for (int x = 0; x < 8; ++x) s.pair[x][col][tid] = v[x];
        } else {
          q.f = a.f[c] - fs;
          p1[col] = q;
        }
      }
    }
    if (tid < 64) act2 = a.mask[L2][tid] != 0;
    {
      const int row = tid >> 3, part = tid & 7;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const double v = a.pinv[row * 64 + part * 8 + c];
        if constexpr (TOP16) s.pinv[c * kTailThreads + tid] = v;
        else pv[c] = v;
      }
    }
    if constexpr (TOP16) {
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
          for (int dx = 0; dx < 2; ++dx) {
            const T d = fx[dx][dy][dz] + fx[dx + 1][dy][dz] + fy[dy][dx][dz] + fy[dy + 1][dx][dz] + fz[dz][dx][dy] +
                        fz[dz + 1][dx][dy];
            D[dz][dy][dx] = d;
            r[dz][dy][dx] = diag_recip(d);
          }
    }
  }

  // the 8^3 cell of colour col this thread (tid < 256) owns
  __device__ __forceinline__ TailCell<T> cell8(int col) const {
    if constexpr (TOP16) {
      return TailCell<T>{s.pair[0][col][tid], s.pair[1][col][tid], s.pair[2][col][tid], s.pair[3][col][tid],
                         s.pair[4][col][tid], s.pair[5][col][tid], s.pair[6][col][tid], s.pair[7][col][tid],
                         s.f1[c1[col]]};
    } else {
      return p1[col];
    }
  }

  // ---- 16^3

  __device__ __forceinline__ void load_e() {
    if constexpr (TOP16) {
      const int I = tid & 7, J = (tid >> 3) & 7, K = tid >> 6;
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          const V2 v = pair_at(a.e, ((2 * K + dz) << 8) + ((2 * J + dy) << 4) + 2 * I);
          e[dz][dy][0] = v.x;
          e[dz][dy][1] = v.y;
        }
    } else {
      s.e1[tid] = a.e[tid];
    }
  }

  __device__ __forceinline__ void store_e() {
    if constexpr (TOP16) {
      const int I = tid & 7, J = (tid >> 3) & 7, K = tid >> 6;
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
          *reinterpret_cast<V2*>(a.e + ((2 * K + dz) << 8) + ((2 * J + dy) << 4) + 2 * I) =
              V2{e[dz][dy][0], e[dz][dy][1]};
    } else {
      a.e[tid] = s.e1[tid];
    }
  }

  __device__ __forceinline__ int own(int dz, int dy, int dx) const { return o + dz * kPlane + dy * kRow + 8 * dx; }

  __device__ __forceinline__ void put_block() {   // every value of the block into LDS
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) s.e0[own(dz, dy, dx)] = e[dz][dy][dx];
  }

  struct Around {
    T xm, xp, ym, yp, zm, zp;
  };
  __device__ __forceinline__ Around around(int dz, int dy, int dx) const {
    const T* L = s.e0;
    const int row = o + dz * kPlane + dy * kRow;
    Around n;
    n.xm = dx ? e[dz][dy][0] : L[row + oxm];
    n.xp = dx ? L[row + oxp] : e[dz][dy][1];
    n.ym = dy ? e[dz][0][dx] : L[o + dz * kPlane + 8 * dx + oym];
    n.yp = dy ? L[o + dz * kPlane + 8 * dx + oyp] : e[dz][1][dx];
    n.zm = dz ? e[0][dy][dx] : L[o + dy * kRow + 8 * dx + ozm];
    n.zp = dz ? L[o + dy * kRow + 8 * dx + ozp] : e[1][dy][dx];
    return n;
  }

  template <int COL>
  __device__ __forceinline__ void half16() {
    const T h2 = a.h2[0];
    T v[4];
    int u = 0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy) {
        const int dx = (COL + dy + dz) & 1;
        const Around n = around(dz, dy, dx);
        const T S = fma_t(fz[dz + 1][dx][dy], n.zp, fma_t(fz[dz][dx][dy], n.zm, fma_t(fy[dy + 1][dx][dz], n.yp,
                    fma_t(fy[dy][dx][dz], n.ym, fma_t(fx[dx + 1][dy][dz], n.xp, fx[dx][dy][dz] * n.xm)))));
        const T q = quotient(fma_t(-h2, f[dz][dy][dx], S), D[dz][dy][dx], r[dz][dy][dx]);
        v[u++] = D[dz][dy][dx] > T(0) ? q : e[dz][dy][dx];
      }
    u = 0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy) {
        const int dx = (COL + dy + dz) & 1;
        e[dz][dy][dx] = v[u];
        s.e0[own(dz, dy, dx)] = v[u++];
      }
    __syncthreads();
  }

  __device__ __forceinline__ T residual16(int dz, int dy, int dx) const {
    const Around n = around(dz, dy, dx);
    const T pc = e[dz][dy][dx];
    const T S = fma_t(fz[dz + 1][dx][dy], n.zp - pc, fma_t(fz[dz][dx][dy], n.zm - pc,
                fma_t(fy[dy + 1][dx][dz], n.yp - pc, fma_t(fy[dy][dx][dz], n.ym - pc,
                fma_t(fx[dx + 1][dy][dz], n.xp - pc, fx[dx][dy][dz] * (n.xm - pc))))));
    return D[dz][dy][dx] > T(0) ? fma_t(-a.inv_h2[0], S, f[dz][dy][dx]) : T(0);
  }

  // the mean of the block's residuals: the right-hand side of 8^3 cell tid
  __device__ __forceinline__ void restrict16() {
    T sum = T(0);
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy) sum += residual16(dz, dy, 0) + residual16(dz, dy, 1);
    s.f1[tid] = sum * T(0.125);
    s.e1[tid] = T(0);
    __syncthreads();
  }

  // the trilinear correction from an edge-long grid's correction ec at cell (I, J, K) to its
  // child (dx, dy, dz): 1-D weights 3/4 and 1/4, x then y then z, each a fused multiply-add
  template <int EDGE>
  __device__ static __forceinline__ void around_coarse(const T* ec, int I, int J, int K, T (&ax)[3][3][2]) {
    constexpr int m = EDGE - 1;
    const int Ix[3] = {(I - 1) & m, I, (I + 1) & m}, Jy[3] = {(J - 1) & m, J, (J + 1) & m};
    const int Kz[3] = {K > 0 ? K - 1 : K, K, K < m ? K + 1 : K};
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const T* row = ec + (Kz[b] * EDGE + Jy[c]) * EDGE;
        const T e0 = row[Ix[0]], e1 = row[Ix[1]], e2 = row[Ix[2]];
        ax[b][c][0] = fma_t(T(0.75), e1, T(0.25) * e0);
        ax[b][c][1] = fma_t(T(0.75), e1, T(0.25) * e2);
      }
  }

  __device__ __forceinline__ void prolong16() {
    T ax[3][3][2];
    around_coarse<8>(s.e1, tid & 7, (tid >> 3) & 7, tid >> 6, ax);
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
          const T lo = fma_t(T(0.75), ax[1][1][dx], T(0.25) * ax[1][2 * dy][dx]);
          const T hi = fma_t(T(0.75), ax[2 * dz][1][dx], T(0.25) * ax[2 * dz][2 * dy][dx]);
          if (live0 >> (4 * dz + 2 * dy + dx) & 1) e[dz][dy][dx] += fma_t(T(0.75), lo, T(0.25) * hi);
        }
    put_block();
    __syncthreads();
  }

  // ---- 8^3

  template <int COL>
  __device__ __forceinline__ void half8() {
    if (tid < 256) {
      const TailCell<T> q = cell8(COL);
      const int c = c1[COL];
      const T* L = s.e1;
      const T S = fma_t(q.zp, L[c + zp1], fma_t(q.zm, L[c + zm1], fma_t(q.yp, L[c + yp1], fma_t(q.ym, L[c + ym1],
                  fma_t(q.xp, L[xp1[COL]], q.xm * L[xm1[COL]])))));
      if (q.D > T(0)) s.e1[c] = quotient(fma_t(-a.h2[L1], q.f, S), q.D, q.r);
    }
    __syncthreads();
  }

  __device__ __forceinline__ T residual8(int col) const {
    const TailCell<T> q = cell8(col);
    const int c = c1[col];
    const T* L = s.e1;
    const T pc = L[c];
    const T S = fma_t(q.zp, L[c + zp1] - pc, fma_t(q.zm, L[c + zm1] - pc, fma_t(q.yp, L[c + yp1] - pc,
                fma_t(q.ym, L[c + ym1] - pc, fma_t(q.xp, L[xp1[col]] - pc, q.xm * (L[xm1[col]] - pc))))));
    return q.D > T(0) ? fma_t(-a.inv_h2[L1], S, q.f) : T(0);
  }

  // the 8^3 grid's cycle on s.e1
  __device__ __forceinline__ void cycle8() {
    half8<0>();
    half8<1>();
    half8<0>();
    half8<1>();
    if (tid < 256) {
      const T ra = residual8(0), rb = residual8(1);
      s.x[tid] = ra + rb;
    }
    __syncthreads();
    // the 4^3 grid: e = A^+ (f - active mean of f) in FP64
    if (tid < 64) {
      const int I = tid & 3, J = (tid >> 2) & 3, K = tid >> 4;
      T sum = T(0);
#pragma unroll
      for (int d = 0; d < 4; ++d) sum += s.x[((2 * K + (d >> 1)) * 8 + 2 * J + (d & 1)) * 4 + I];
      const T f2 = sum * T(0.125);
      const double v = act2 ? static_cast<double>(f2) : 0.0;
      double total = v;
      for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
      const int cnt = __popcll(__ballot(act2));
      s.fh[tid] = act2 ? v - (cnt > 0 ? total / cnt : 0.0) : 0.0;
    }
    __syncthreads();
    {
      const int row = tid >> 3, part = tid & 7;
      double acc = 0.0;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        double v;
        if constexpr (TOP16) v = s.pinv[c * kTailThreads + tid];
        else v = pv[c];
        acc = __builtin_fma(v, s.fh[part * 8 + c], acc);
      }
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      acc += __shfl_xor(acc, 4, 64);
      if (part == 0) s.e2[row] = static_cast<T>(acc);
    }
    __syncthreads();
    if (tid < 256) {
      const int ip = tid & 3, j = (tid >> 2) & 7, k = tid >> 5;
      T ax[3][3][2];
      around_coarse<4>(s.e2, ip, j >> 1, k >> 1, ax);
      const int dy = j & 1, dz = k & 1;
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const T near = dy ? ax[1][2][dx] : ax[1][0][dx];
        const T far1 = dz ? ax[2][1][dx] : ax[0][1][dx];
        const T far2 = dz ? (dy ? ax[2][2][dx] : ax[2][0][dx]) : (dy ? ax[0][2][dx] : ax[0][0][dx]);
        const T lo = fma_t(T(0.75), ax[1][1][dx], T(0.25) * near);
        const T hi = fma_t(T(0.75), far1, T(0.25) * far2);
        const bool on = ((dx + j + k) & 1) ? live1[1] : live1[0];
        if (on) s.e1[(k * 8 + j) * 8 + 2 * ip + dx] += fma_t(T(0.75), lo, T(0.25) * hi);
      }
    }
    __syncthreads();
    half8<1>();
    half8<0>();
    half8<1>();
    half8<0>();
  }

  // one cycle; the top grid's values are in e (and in s.e0) or in s.e1, past a barrier
  __device__ __forceinline__ void cycle() {
    if constexpr (TOP16) {
      half16<0>();
      half16<1>();
      half16<0>();
      half16<1>();
      restrict16();
      cycle8();
      prolong16();
      half16<1>();
      half16<0>();
      half16<1>();
      half16<0>();
    } else {
      cycle8();
    }
  }
};

template <typename T, bool TOP16>
__global__ __launch_bounds__(kTailThreads) void k_coarse_cycle(CoarseCycle<T> a) {
  __shared__ TailShared<T, TOP16> s;
  Tail<T, TOP16> t(s, a);
  t.load_e();
  t.load(a.fshift ? static_cast<T>(*a.fshift) : T(0));
  if constexpr (TOP16) t.put_block();
  __syncthreads();
  t.cycle();
  t.store_e();
}

// The sum over the workgroup, in every thread; its barriers also end every wave's reads of
// the values the next half-sweep changes.
__device__ __forceinline__ double sum_all(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kTailThreads / 64; ++w) s += red[w];
  __syncthreads();
  return s;
}

// A whole solve: the cycle above with its residual norm, stopping test and history, so that
// a cycle costs neither launches nor a round trip to the host and the coefficients are
// read once per solve.  A cycle and its norm take 12 us at 16^3 and 6 us at 8^3; launched
// one by one, with the sums and the host's part, 28 and 22 us.
template <bool TOP16>
__global__ __launch_bounds__(kTailThreads) void k_small_solve(SmallSolve a) {
  __shared__ TailShared<double, TOP16> s;
  __shared__ double red[kTailThreads / 64];
  Tail<double, TOP16> t(s, a.cyc);
  const int tid = threadIdx.x;
  t.load_e();
  t.load(0.0);
  // per thread: f(term) over its active cells, summed
  auto over_f = [&](auto term) {
    double v = 0.0;
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (t.live0 >> c & 1) v += term(t.f[c >> 2][(c >> 1) & 1][c & 1]);
    } else if (tid < 256) {
#pragma unroll
      for (int col = 0; col < 2; ++col)
        if (t.live1[col]) v += term(t.p1[col].f);
    }
    return v;
  };
  auto subtract = [&](double m) {
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c) t.f[c >> 2][(c >> 1) & 1][c & 1] -= m;
    } else {
      t.p1[0].f -= m;
      t.p1[1].f -= m;
    }
  };
  // the guess, and at the end the solution less its mean: 0 on inactive cells
  auto gauge = [&](double m) {
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        double& v = t.e[c >> 2][(c >> 1) & 1][c & 1];
        v = (t.live0 >> c & 1) ? v - m : 0.0;
      }
    } else if (tid < 256) {
#pragma unroll
      for (int col = 0; col < 2; ++col) s.e1[t.c1[col]] = t.live1[col] ? s.e1[t.c1[col]] - m : 0.0;
    }
  };
  auto residual2 = [&]() {
    double v = 0.0;
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const double r = t.residual16(c >> 2, (c >> 1) & 1, c & 1);
        v = __builtin_fma(r, r, v);
      }
    } else if (tid < 256) {
      const double ra = t.residual8(0), rb = t.residual8(1);
      v = __builtin_fma(rb, rb, ra * ra);
    }
    return sum_all(v, red);
  };
  const double inv_active = 1.0 / a.active;
  const double mean = sum_all(over_f([](double v) { return v; }), red) * inv_active;
  subtract(mean);
  const double nf2 = sum_all(over_f([](double v) { return v * v; }), red);
  const double nf = sqrt(nf2), nf_all = sqrt(nf2 + a.active * mean * mean);
  gauge(0.0);
  if constexpr (TOP16) t.put_block();
  __syncthreads();
  int nh = 0, cycles = 0, how = kSmallDone;
  double r = 0.0, r0 = 0.0;
  auto record = [&](double v) {
    if (tid == 0) {
      a.hist[nh] = v;
      if (nh < a.host_cap) a.host_hist[nh] = v;
    }
    ++nh;
  };
  if (!(nf > a.zero_rhs * nf_all)) {   // P f = 0 to rounding: p = 0
    how = __builtin_isfinite(nf) ? kSmallZero : kSmallNotFinite;
    record(0.0);
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c) t.e[c >> 2][(c >> 1) & 1][c & 1] = 0.0;
    } else {
      s.e1[tid] = 0.0;
    }
  } else {
    r = r0 = sqrt(residual2()) / nf;
    record(r);
    if (!__builtin_isfinite(r)) how = kSmallBreakdown;   // (a guess that is not finite)
    while (__builtin_isfinite(r) && r > a.tol && cycles < a.max_cycles) {
      t.cycle();
      ++cycles;
      r = sqrt(residual2()) / nf;
      record(r);
      if (!__builtin_isfinite(r) || r > a.growth * fmax(r0, 1.0)) {
        how = kSmallBreakdown;
        break;
      }
    }
    if (how == kSmallDone && r > a.tol) how = kSmallNoConv;
    double v = 0.0;
    if constexpr (TOP16) {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (t.live0 >> c & 1) v += t.e[c >> 2][(c >> 1) & 1][c & 1];
    } else if (tid < 256) {
#pragma unroll
      for (int col = 0; col < 2; ++col)
        if (t.live1[col]) v += s.e1[t.c1[col]];
    }
    gauge(sum_all(v, red) * inv_active);
  }
  if constexpr (!TOP16) __syncthreads();
  t.store_e();
  if (tid == 0) {
    double* h = a.pub.host;
    h[0] = mean;
    h[1] = r;
    h[2] = r0;
    h[3] = nh;
    h[4] = cycles;
    h[5] = how;
    __threadfence_system();
    __hip_atomic_store(a.pub.ticket, a.pub.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---------------------------------------------------------------------------- setup

// The grids below 16^3 and the 4^3 pseudo-inverse, by one workgroup in one launch: the
// face products coarsened to 8^3 and 4^3 as k_coarsen does, the setup's counts added up,
// and A^+ of the 4^3 operator.  Its null space is known: the constant on each connected
// fluid region and one unit vector per inactive cell.  With Z that orthonormal basis,
// M = Z Z^T - A is symmetric positive definite and A^+ = Z Z^T - M^-1; M^-1 comes from
// Gauss-Jordan elimination in place, whose pivots need no exchange in a definite matrix.
// Lane r of wave w holds M's row r in columns 8w .. 8w+7, so a pivot row is a broadcast
// within each wave and only the pivot column goes through LDS, with one barrier per pivot.
// A pivot that is not positive is reported; the host then takes its own way.
// The launch takes 32 us; the elimination on the host, with the copies to it and back and
// a launch per grid and array before it, held every setup to 310 us at the least (68 now).
struct SetupLds {
  double x8[512], y8[512], z8[512];
  double x4[64], y4[64], z4[64];
  uint8_t m8[512], m4[64];
  double col[2][64], tiny;
  int comp[64], size[64];
  long long count[3][kTailThreads / 64];
};

// coarse cell (I, J, K) of the grid of edge 2^qc from the fine grid's accessors: its low
// faces and activity (k_coarsen's arithmetic)
template <typename BX, typename BY, typename BZ, typename M>
__device__ __forceinline__ void coarsen_cell(int qc, int I, int J, int K, BX bx, BY by, BZ bz, M mask, double& xm,
                                             double& ym, double& zm, bool& act) {
  const int mf = (2 << qc) - 1, mc = (1 << qc) - 1, i = 2 * I, j = 2 * J, k = 2 * K;
  auto fx = [&](int ii) { return 0.25 * (bx(ii, j, k) + bx(ii, j + 1, k) + bx(ii, j, k + 1) + bx(ii, j + 1, k + 1)); };
  auto fy = [&](int jj) { return 0.25 * (by(i, jj, k) + by(i + 1, jj, k) + by(i, jj, k + 1) + by(i + 1, jj, k + 1)); };
  auto fz = [&](int kk) { return 0.25 * (bz(i, j, kk) + bz(i + 1, j, kk) + bz(i, j + 1, kk) + bz(i + 1, j + 1, kk)); };
  xm = fx(i);
  ym = fy(j);
  zm = fz(k);
  const double xp = fx((i + 2) & mf), yp = fy((j + 2) & mf), zp = K < mc ? fz(k + 2) : 0.0;
  bool any = false;
#pragma unroll
  for (int d = 0; d < 8; ++d) any |= mask(i + (d & 1), j + ((d >> 1) & 1), k + (d >> 2));
  act = any && (xm + xp + ym + yp + zm + zp) > 0.0;
}

__device__ __forceinline__ double from_lane(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane(static_cast<unsigned>(b), lane);
  const unsigned hi = __builtin_amdgcn_readlane(static_cast<unsigned>(b >> 32), lane);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

__global__ __launch_bounds__(kTailThreads) void k_coarse_setup(CoarseSetup a) {
  __shared__ SetupLds s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int last = a.nlev - 1;
  auto keep = [](const CoarseSetup::Grid& g, int c, double xm, double ym, double zm, bool act) {
    g.bx[c] = xm;
    g.by[c] = ym;
    g.bz[c] = zm;
    g.mask[c] = act ? 1 : 0;
    if (g.bx32) {
      g.bx32[c] = static_cast<float>(xm);
      g.by32[c] = static_cast<float>(ym);
      g.bz32[c] = static_cast<float>(zm);
    }
  };
  // ---- the counts of the finest grid's setup, a set of partial ones per block
  long long cnt[3] = {0, 0, 0};
  for (int b = tid; b < a.nparts; b += kTailThreads) {
#pragma unroll
    for (int x = 0; x < 3; ++x) cnt[x] += a.parts[x * a.nparts + b];
  }
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    for (int off = 32; off > 0; off >>= 1) cnt[x] += __shfl_xor(cnt[x], off, 64);
    if (lane == 0) s.count[x][wave] = cnt[x];
  }
  // ---- 16^3 -> 8^3, or the 8^3 grid as it is
  if (a.nlev == 3) {
    const CoarseSetup::Grid& g = a.g[0];
    auto at = [](int i, int j, int k) { return (k << 8) + (j << 4) + i; };
    double xm, ym, zm;
    bool act;
    coarsen_cell(
        3, tid & 7, (tid >> 3) & 7, tid >> 6, [&](int i, int j, int k) { return g.bx[at(i, j, k)]; },
        [&](int i, int j, int k) { return g.by[at(i, j, k)]; }, [&](int i, int j, int k) { return g.bz[at(i, j, k)]; },
        [&](int i, int j, int k) { return g.mask[at(i, j, k)] != 0; }, xm, ym, zm, act);
    keep(a.g[1], tid, xm, ym, zm, act);
    s.x8[tid] = xm;
    s.y8[tid] = ym;
    s.z8[tid] = zm;
    s.m8[tid] = act;
  } else if (a.nlev == 2) {
    const CoarseSetup::Grid& g = a.g[0];
    s.x8[tid] = g.bx[tid];
    s.y8[tid] = g.by[tid];
    s.z8[tid] = g.bz[tid];
    s.m8[tid] = g.mask[tid] != 0;
  }
  __syncthreads();
  // ---- 8^3 -> 4^3, or the 4^3 grid as it is
  if (tid < 64) {
    if (a.nlev > 1) {
      auto at = [](int i, int j, int k) { return (k << 6) + (j << 3) + i; };
      double xm, ym, zm;
      bool act;
      coarsen_cell(
          2, tid & 3, (tid >> 2) & 3, tid >> 4, [&](int i, int j, int k) { return s.x8[at(i, j, k)]; },
          [&](int i, int j, int k) { return s.y8[at(i, j, k)]; }, [&](int i, int j, int k) { return s.z8[at(i, j, k)]; },
          [&](int i, int j, int k) { return s.m8[at(i, j, k)] != 0; }, xm, ym, zm, act);
      keep(a.g[last], tid, xm, ym, zm, act);
      s.x4[tid] = xm;
      s.y4[tid] = ym;
      s.z4[tid] = zm;
      s.m4[tid] = act;
    } else {
      const CoarseSetup::Grid& g = a.g[last];
      s.x4[tid] = g.bx[tid];
      s.y4[tid] = g.by[tid];
      s.z4[tid] = g.bz[tid];
      s.m4[tid] = g.mask[tid] != 0;
    }
    s.size[tid] = 0;
  }
  __syncthreads();
  // ---- row `lane` of A: neighbours and faces (every wave the same)
  const int i = lane & 3, j = (lane >> 2) & 3, k = lane >> 4;
  const bool act = s.m4[lane] != 0;
  const int nb[6] = {lane - i + ((i + 3) & 3),        lane - i + ((i + 1) & 3),
                     lane + 4 * (((j + 3) & 3) - j),  lane + 4 * (((j + 1) & 3) - j),
                     k > 0 ? lane - 16 : lane,        k < 3 ? lane + 16 : lane};
  double b[6] = {s.x4[lane], s.x4[nb[1]], s.y4[lane], s.y4[nb[3]], k > 0 ? s.z4[lane] : 0.0, k < 3 ? s.z4[nb[5]] : 0.0};
#pragma unroll
  for (int f = 0; f < 6; ++f) b[f] = act ? b[f] * a.inv_h2 : 0.0;
  double diag = 0.0;
#pragma unroll
  for (int f = 0; f < 6; ++f) diag -= b[f];
  if (wave == 0) {
    // connected regions of the active cells over open faces: the lowest cell of each
    int lab = act ? lane : -1;
    for (int round = 0; round < 64; ++round) {
      int low = lab;
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        const int other = __shfl(lab, nb[f], 64);
        if (act && b[f] > 0.0 && other >= 0) low = min(low, other);
      }
      const bool moved = low != lab;
      lab = low;
      if (!__any(moved)) break;
    }
    s.comp[lane] = lab;
    if (lab >= 0) atomicAdd(&s.size[lab], 1);
    double big = fabs(diag);
    for (int off = 32; off > 0; off >>= 1) big = fmax(big, __shfl_xor(big, off, 64));
    if (lane == 0) s.tiny = 1e-14 * fmax(big, 1.0);
  }
  __syncthreads();
  const int own = s.comp[lane];
  const double share = own >= 0 ? 1.0 / s.size[own] : 0.0;
  const double tiny = s.tiny;
  double zz[8], m[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int cc = wave * 8 + c;
    zz[c] = own >= 0 ? (s.comp[cc] == own ? share : 0.0) : (cc == lane ? 1.0 : 0.0);
    double v = 0.0;
#pragma unroll
    for (int f = 0; f < 6; ++f)
      if (nb[f] == cc) v += b[f];
    if (cc == lane) v = diag;
    m[c] = zz[c] - v;
  }
  bool bad = false;
  for (int kb = 0; kb < 8; ++kb) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int kp = kb * 8 + kk;
      if (wave == kb) s.col[kk & 1][lane] = m[kk];
      __syncthreads();
      const double p = s.col[kk & 1][kp], ci = s.col[kk & 1][lane];
      bad |= !(p > tiny);
      double inv = __builtin_amdgcn_rcp(p);   // two Newton steps: within an ulp, half the division's chain
      inv = __builtin_fma(inv, __builtin_fma(-p, inv, 1.0), inv);
      inv = __builtin_fma(inv, __builtin_fma(-p, inv, 1.0), inv);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const double rk = from_lane(m[c], kp) * inv;
        m[c] = lane == kp ? rk : __builtin_fma(-ci, rk, m[c]);
      }
      if (wave == kb) m[kk] = lane == kp ? inv : -ci * inv;
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) a.pinv[lane * 64 + wave * 8 + c] = zz[c] - m[c];
  // The host takes the ticket for the end of the setup, and may go on from another stream:
  // each wave waits here until its stores are in the L2 (the barrier alone orders LDS only),
  // which the fence before the ticket writes back.  A fence in every wave costs 2 us.
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      long long t = 0;
      for (int v = 0; v < kTailThreads / 64; ++v) t += s.count[x][v];
      a.pub.host[x] = static_cast<double>(t);
    }
    a.pub.host[3] = bad ? 1.0 : 0.0;
    __threadfence_system();
    __hip_atomic_store(a.pub.ticket, a.pub.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace

template <typename T>
hipError_t launch_coarse_cycle(const CoarseCycle<T>& a, hipStream_t s) {
  if (a.nlev == 3 && a.q[0] == 4)
    hipLaunchKernelGGL((k_coarse_cycle<T, true>), dim3(1), dim3(kTailThreads), 0, s, a);
  else if (a.nlev == 2 && a.q[0] == 3)
    hipLaunchKernelGGL((k_coarse_cycle<T, false>), dim3(1), dim3(kTailThreads), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_small_solve(const SmallSolve& a, hipStream_t s) {
  if (!a.hist || !a.pub.host || !a.pub.ticket || a.max_cycles < 0) return hipErrorInvalidValue;
  if (a.cyc.nlev == 3 && a.cyc.q[0] == 4)
    hipLaunchKernelGGL(k_small_solve<true>, dim3(1), dim3(kTailThreads), 0, s, a);
  else if (a.cyc.nlev == 2 && a.cyc.q[0] == 3)
    hipLaunchKernelGGL(k_small_solve<false>, dim3(1), dim3(kTailThreads), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_coarse_setup(const CoarseSetup& a, hipStream_t s) {
  if (a.nlev < 1 || a.nlev > 3 || a.nparts < 0 || !a.pinv || !a.pub.host || !a.pub.ticket) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_coarse_setup, dim3(1), dim3(kTailThreads), 0, s, a);
  return hipGetLastError();
}

template hipError_t launch_coarse_cycle<double>(const CoarseCycle<double>&, hipStream_t);
template hipError_t launch_coarse_cycle<float>(const CoarseCycle<float>&, hipStream_t);

}  // namespace mg
