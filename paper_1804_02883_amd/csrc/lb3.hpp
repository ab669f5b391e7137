// Three-dimensional lattice Boltzmann fluid: D3Q19, the scheme the paper
// names for three dimensions (end of Sec. II), with the collision and body
// force of the two-dimensional fluid (Sec. II, Eq. LB_prop and Eq. force_col
// at gamma_s = gamma_b = 0): pull streaming, BGK relaxation with time tau
// towards the second-order equilibrium, the second-order force term
//   (1 - 1/(2 tau)) w_i [3 (c_i - u).F + 9 (c_i.u)(c_i.F)],
// and u = (sum f_i c_i + F/2) / rho.
//
// Layout: 19 planes of nx*ny*nz values, [i][z][y][x], x contiguous, holding
// the deviations g_i = f_i - w_i from the rest state (FP32 keeps the small
// momentum of slow flows).  Force and velocity: 3 planes (x, y, z).
//
// The step moves 19 values in and 19 out per site plus the force: it is a
// streaming kernel bound by HBM.  Each value is read by exactly one site (the
// one its velocity points to), so the only reuse is the cache line that two
// neighbouring chunks share when a population moves along x; runs of 4,096 sites
// stay on one XCD, whose L2 then holds that line (192^3 / 256^3 FP32: 214.9 /
// 520 us a step; one run per XCD through the whole box 225.3 / 525, single
// blocks 218.1 / 505 but 128^3 FP64 138.8 against 133.9).  A lane takes one site,
// in the order of memory: every wave but the last is full whatever the row length,
// and all sites are in flight at once.  With a wave per row, in chunks of 64
// sites, a row of 70 left 45 % of the lanes idle.  Per step, before -> now: 192^3
// FP32 229.8 -> 214.9 us (5.4 TB/s); 190^3 FP32 331 -> 213; 100^3 FP64 70.0 -> 56.2;
// 70 x 45 x 33 FP64 11.9 -> 6.3; 32^3 FP32 3.6 -> 3.2.
#pragma once
#include "kernels.hpp"

namespace epdlb {
namespace lb3 {

constexpr int kQ = 19;
// Threads per block: one wave up to kSmall sites, where more CUs get a block
// (33 x 20 x 20 FP64: 3.2 us with 64 threads, 3.7 with 256), else 256 (128^3
// FP64: 136.7 us with 64, 125.7 with 256; the two are equal around kSmall).
constexpr int kThreads = 256;
constexpr int kThreadsSmall = 64;
constexpr long kSmall = 1 << 18;

// c_i: rest, +x, -x, +y, -y, +z, -z, then the face diagonals
// (1,1,0) (-1,-1,0) (1,-1,0) (-1,1,0) (1,0,1) (-1,0,-1) (1,0,-1) (-1,0,1)
// (0,1,1) (0,-1,-1) (0,1,-1) (0,-1,1); weights 1/3, 1/18 (axes), 1/36 (diagonals).
constexpr int kCx[kQ] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr int kCy[kQ] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr int kCz[kQ] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};

template <typename T> __device__ __forceinline__ T weight(int k) {
  return k == 0 ? T(1.0 / 3.0) : (k < 7 ? T(1.0 / 18.0) : T(1.0 / 36.0));
}

template <typename T> __device__ __forceinline__ T signed_term(int c, T v) { return c > 0 ? v : -v; }

// c_k . a with the zero components left out (k is a constant after unrolling).
template <typename T> __device__ __forceinline__ T cdot(int k, T ax, T ay, T az) {
  const int a = kCx[k], b = kCy[k], c = kCz[k];
  if (a != 0 && b != 0) return signed_term(a, ax) + signed_term(b, ay);
  if (a != 0 && c != 0) return signed_term(a, ax) + signed_term(c, az);
  if (b != 0 && c != 0) return signed_term(b, ay) + signed_term(c, az);
  if (a != 0) return signed_term(a, ax);
  if (b != 0) return signed_term(b, ay);
  if (c != 0) return signed_term(c, az);
  return T(0);
}

// i / d for i < 2^31 by one multiplication: with l = ceil(log2 d) and
// m = ceil(2^(31 + l) / d) < 2^32, floor(i m / 2^(31 + l)) = floor(i / d).
struct DivBy {
  unsigned m = 1u << 31, s = 31;
  DivBy() = default;
  explicit DivBy(unsigned d) {
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    s = 31 + l;
    m = unsigned(((1ull << s) + d - 1) / d);
  }
  __device__ __forceinline__ unsigned operator()(unsigned i) const { return unsigned((static_cast<unsigned long long>(i) * m) >> s); }
};

template <typename T> struct Lb3Args {
  const T* fin;  // 19 planes g* (post-collision of the previous step)
  T* fout;       // 19 planes
  const T* F;    // 3 planes
  T* rho;        // written when the kernel stores the moments
  T* u;          // 3 planes
  int nx, ny, nz;
  long n;        // nx ny nz
  T omega;       // 1/tau
  T fpre;        // 1 - 1/(2 tau)
  DivBy by_nx, by_ny;  // site -> row, row -> plane
  __device__ const Lb3Args& base() const { return *this; }
};

// The value at byte `o` of a plane.  Off: 32 bits for planes of less than 4 GiB
// (a scalar base plus a lane offset), else 64.
template <typename X, typename Off> __device__ __forceinline__ X load_at(const X* base, Off o) {
  return *reinterpret_cast<const X*>(reinterpret_cast<const char*>(base) + o);
}
template <typename X, typename Off> __device__ __forceinline__ void store_at(X* base, Off o, X v) {
  *reinterpret_cast<X*>(reinterpret_cast<char*>(base) + o) = v;
}

// One step of the site at byte o of each plane, from its streamed-in populations
// g and its force.
template <bool MOM, typename T, typename Off>
__device__ __forceinline__ void collide(const Lb3Args<T>& P, const T (&g)[kQ], Off o, T Fx, T Fy, T Fz) {
  // sum_i w_i = 1 and sum_i w_i c_i = 0: the deviations carry rho - 1 and the momentum
  T drho = T(0), jx = T(0), jy = T(0), jz = T(0);
#pragma unroll
  for (int k = 0; k < kQ; ++k) {
    drho += g[k];
    if (kCx[k] != 0) jx = kCx[k] > 0 ? jx + g[k] : jx - g[k];
    if (kCy[k] != 0) jy = kCy[k] > 0 ? jy + g[k] : jy - g[k];
    if (kCz[k] != 0) jz = kCz[k] > 0 ? jz + g[k] : jz - g[k];
  }
  const T rho = T(1) + drho;
  const T ir = T(1) / rho;
  const T ux = (jx + T(0.5) * Fx) * ir, uy = (jy + T(0.5) * Fy) * ir, uz = (jz + T(0.5) * Fz) * ir;
  const T usq = ux * ux + uy * uy + uz * uz;
  const T uF = ux * Fx + uy * Fy + uz * Fz;
#pragma unroll
  for (int k = 0; k < kQ; ++k) {
    const T w = weight<T>(k);
    const T cu = cdot(k, ux, uy, uz);
    const T cF = cdot(k, Fx, Fy, Fz);
    // f^eq - w = w (rho - 1) + w rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2)
    const T geq = w * drho + w * rho * (T(3) * cu + T(4.5) * cu * cu - T(1.5) * usq);
    const T s = w * (T(3) * (cF - uF) + T(9) * cu * cF);
    store_at(P.fout + long(k) * P.n, o, T(g[k] - (g[k] - geq) * P.omega + P.fpre * s));
  }
  if (MOM) {
    store_at(P.rho, o, rho);
    store_at(P.u, o, ux);
    store_at(P.u + P.n, o, uy);
    store_at(P.u + 2 * P.n, o, uz);
  }
}

// The block of sites a block takes.  Large boxes: runs of 4,096 sites on one XCD
// (block b starts on XCD b mod 8), the XCDs side by side through memory.  Small
// ones: one run per XCD, whose L2 then still holds most of what the last step
// wrote (70 x 45 x 33 FP64: 6.4 us, 8.2 in runs of 4,096).
template <int BLOCK> __device__ __forceinline__ unsigned site_block(unsigned b, unsigned blocks) {
  if constexpr (BLOCK == kThreadsSmall) return xcd_tile(b, blocks);
  constexpr unsigned run = 4096 / BLOCK, group = kNumXcd * run;
  if (b >= blocks / group * group) return b;
  const unsigned r = b % group;
  return b - r + (r % kNumXcd) * run + r / kNumXcd;
}

// One step at every site: ceil(n / BLOCK) blocks, rounded up to all XCDs.
template <typename T, typename Args, typename Off, bool MOM, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_lb3(Args A) {
  const Lb3Args<T>& P = A.base();
  const unsigned nx = P.nx, ny = P.ny, nz = P.nz;
  const unsigned i = site_block<BLOCK>(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
  if (i >= unsigned(P.n)) return;
  const unsigned r = P.by_nx(i), x = i - r * nx, z = P.by_ny(r), y = r - z * ny;
  // byte distance to the sites that populations with components +1, 0, -1 come
  // from (differences modulo the range of Off)
  const Off es = sizeof(T), row = es * nx, plane = row * ny;
  const Off dx[3] = {x == 0 ? es * (nx - 1) : -es, 0, x + 1 == nx ? -es * (nx - 1) : es};
  const Off dy[3] = {y == 0 ? row * (ny - 1) : -row, 0, y + 1 == ny ? -row * (ny - 1) : row};
  const Off dz[3] = {z == 0 ? plane * (nz - 1) : -plane, 0, z + 1 == nz ? -plane * (nz - 1) : plane};
  const Off o = es * i;
  T g[kQ];
#pragma unroll
  for (int k = 0; k < kQ; ++k)
    g[k] = load_at(P.fin + long(k) * P.n, Off(o + dx[1 - kCx[k]] + dy[1 - kCy[k]] + dz[1 - kCz[k]]));
  collide<MOM>(A, g, o, load_at(P.F, o), load_at(P.F + P.n, o), load_at(P.F + 2 * P.n, o));
}

// g = f^eq(rho, u) - w from the moments in P.rho and P.u, kThreads sites a block.
template <typename T> __global__ void __launch_bounds__(kThreads) k_lb3_equilibrium(Lb3Args<T> P) {
  const long i = long(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= P.n) return;
  const T rho = P.rho[i];
  const T ux = P.u[i], uy = P.u[P.n + i], uz = P.u[2 * P.n + i];
  const T usq = ux * ux + uy * uy + uz * uz;
#pragma unroll
  for (int k = 0; k < kQ; ++k) {
    const T w = weight<T>(k);
    const T cu = cdot(k, ux, uy, uz);
    P.fout[long(k) * P.n + i] = w * (rho - T(1)) + w * rho * (T(3) * cu + T(4.5) * cu * cu - T(1.5) * usq);
  }
}

}  // namespace lb3
}  // namespace epdlb
