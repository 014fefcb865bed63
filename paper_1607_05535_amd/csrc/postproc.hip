// Post-processing on pressure levels (the results of Sec. 7 are shown on
// pressure levels): per snapshot, every column's u, v, T and theta are
// interpolated linearly in pressure to the requested levels; latitude-band
// zonal means (area-weighted over the columns that have a value), the eddy
// fluxes [u'v'] and [v'T'] (eddies = deviations from the zonal mean) and the
// valid area fraction are added to running time sums; the result divides
// the sums by the number of snapshots with a value and adds the mass
// streamfunction Psi = 2 pi A cos(lat) / g * int_0^p [v] dp.  Beside them,
// the grid-imprinting map of the Held-Suarez results: per column, the time
// sum of w* = w - {w} in the first model layer, {w} the area-weighted mean
// of w over the column's latitude band.
//
// Readings: a level outside a column's [top-cell, bottom-cell] pressure
// range has no value in that column; band b covers latitudes
// [-90 + 180 b / n, -90 + 180 (b + 1) / n) degrees (the north pole in the
// last band); Psi uses the trapezoid rule with [v](p = 0) = [v](first level);
// the imprinting bracket is a zonal deviation followed by a time mean (a
// deviation from the time mean alone would average to zero).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <vector>

#include "internal.h"
#include "kernels.h"
#include "powd.h"
#include "state.h"

namespace thor {
namespace {

constexpr int kZq = 4;          // interpolated quantities: u, v, T, theta
constexpr int kZslot = kZq + 1; // + pressure, in LDS
constexpr int kZrec = 11;       // a tile's record: 2 areas, 4 sums, 2 co-moments, 3 remainders
constexpr int kZthreads = 256;  // threads of a workgroup
constexpr int kZcols = 16;      // columns per workgroup of the interpolation
constexpr int kZlev = 64;        // pressure levels per pass of the interpolation
constexpr int kZpitch = kZcols + 1;   // LDS row of one level over those columns, padded

bool zok(hipError_t e, const char *what) {
  if (e == hipSuccess) return true;
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return false;
}

// Sums over each 16 consecutive lanes (a DPP row, by rotations), to every one
// of them.
template <int ROT>
__device__ __forceinline__ double row_ror(double x) {
  union { double d; int i[2]; } u{x}, r;
  r.i[0] = __builtin_amdgcn_update_dpp(0, u.i[0], 0x120 + ROT, 0xf, 0xf, true);
  r.i[1] = __builtin_amdgcn_update_dpp(0, u.i[1], 0x120 + ROT, 0xf, 0xf, true);
  return r.d;
}
template <int NV>
__device__ __forceinline__ void lane16_sums(double v[NV]) {
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] += row_ror<8>(v[k]);
    v[k] += row_ror<4>(v[k]);
    v[k] += row_ror<2>(v[k]);
    v[k] += row_ror<1>(v[k]);
  }
}

// A tile of at most kZcols consecutive columns of the band-sorted list `cols`
// per workgroup, all of one band (tiles[w] = first position, count): p, u, v,
// T, theta of every level into LDS ([quantity][level][column], dynamic), then
// 16 lanes per pressure level, one a column, look for the lowest-index level
// pair whose pressures bracket the level.  What a band needs of the tile goes
// to P[j][w]: the area with a value there, the whole area, the area-weighted
// sums of u, v, T, theta, the co-moments u'v', v'T' about the tile's own
// (rounded) means and the sums of u, v, T less those means: k_zreduce merges
// them about the band's means as exactly as a second pass over the columns.
// Zw[pos] = w at the centre of the first layer (half the momentum of the first
// interior interface over rho; the ground interface carries none).
// Bound by reading the state (40 bytes per cell); g6 L32, 20 levels:
// 81 -> 30 us by columns in LDS, -> 28 by records instead of every value
// (33 MB) out and a scatter of each level pair to the pressure levels it
// brackets instead of a search through the pairs for each.  Twice the
// threads 37 us, more wavefronts per SIMD (7) 39, four levels per thread 30.
template <typename H>
__global__ __launch_bounds__(kZthreads) void k_zinterp(Fields<H> f, Consts c, const int32_t *cols, const int2 *tiles,
                                                       const double *area, const double *plev, int np, double *P,
                                                       double *Zw) {
  extern __shared__ double zs[];
  __shared__ int below[kZlev * kZcols];   // lower level of the bracketing pair, L if none
  __shared__ double pl[kZlev];
  const int2 tile = tiles[blockIdx.x];
  const int L = c.L, pos0 = tile.x, nc = tile.y;
  const int plane = L * kZpitch;   // one quantity
  for (int i = threadIdx.x; i < nc * L; i += kZthreads) {
    const int cb = i / L, lev = i - cb * L, col = cols[pos0 + cb];
    const size_t idx = (size_t)col * c.S + lev;   // state row stride
    const double rho = f.rho_t[idx], rth = f.rth_t[idx];
    const double p = c.p_ref * powd(c.Rd * rth / c.p_ref, c.gamma);
    double e[3], n[3];
    wind64(f, col, e, n);
    const double ir = rcpd(rho);
    const double vx = quot((double)f.Mx_t[idx], rho, ir), vy = quot((double)f.My_t[idx], rho, ir),
                 vz = quot((double)f.Mz_t[idx], rho, ir);
    double *o = zs + lev * kZpitch + cb;
    o[0] = p;
    o[plane] = e[0] * vx + e[1] * vy;
    o[2 * plane] = n[0] * vx + n[1] * vy + n[2] * vz;
    o[3 * plane] = p / (rho * c.Rd);
    o[4 * plane] = quot(rth, rho, ir);
    if (lev == 0) Zw[pos0 + cb] = L > 1 ? 0.5 * f.W_t[idx + 1] / rho : 0.0;
  }
  __syncthreads();
  for (int j0 = 0; j0 < np; j0 += kZlev) {
    const int nj = min(kZlev, np - j0);
    for (int i = threadIdx.x; i < kZlev * kZcols; i += kZthreads) below[i] = L;
    if (threadIdx.x < nj) pl[threadIdx.x] = plev[j0 + threadIdx.x];
    __syncthreads();
    // interval (k, k + 1) of a column holds the pressure levels from p of
    // k + 1 up to p of k (the levels ascend)
    for (int i = threadIdx.x; i < nc * (L - 1); i += kZthreads) {
      const int cb = i / (L - 1), k = i - cb * (L - 1);
      const double hi = zs[k * kZpitch + cb], lo = zs[(k + 1) * kZpitch + cb];
      int j = 0;
#pragma unroll
      for (int h = kZlev / 2; h > 0; h >>= 1)
        if (j + h <= nj && !(pl[j + h - 1] >= lo)) j += h;
      if (j == nj - 1 && !(pl[j] >= lo)) j = nj;
      for (; j < nj && pl[j] >= lo && pl[j] <= hi; ++j) atomicMin(&below[j * kZcols + cb], k);
    }
    __syncthreads();
    // whole wavefronts: four levels each (past the last one without a value)
    for (int i = threadIdx.x; i < (nj + 3) / 4 * 64; i += kZthreads) {
      const int jj = min(i / kZcols, nj - 1), cb = i % kZcols;
      const bool in = i / kZcols < nj && cb < nc;
      const double pj = pl[jj];
      const double *col = zs + min(cb, nc - 1);
      const int b = below[jj * kZcols + min(cb, nc - 1)], k = b < L ? b : -1;
      const bool has = in && k >= 0;
      const double p0 = col[max(k, 0) * kZpitch], p1 = col[min(max(k, 0) + 1, L - 1) * kZpitch];
      const double w = (pj - p1) / (p0 - p1);
      const double *q0 = col + max(k, 0) * kZpitch, *q1 = q0 + (k < 0 ? 0 : kZpitch);
      double x[kZq];   // u, v, T, theta
#pragma unroll
      for (int q = 1; q <= kZq; ++q) {
        const double up = q1[q * plane];
        x[q - 1] = has ? up + w * (q0[q * plane] - up) : 0.0;
      }
      const double A0 = in ? area[pos0 + cb] : 0.0, A = has ? A0 : 0.0;
      double m[2 + kZq] = {A, A0, A * x[0], A * x[1], A * x[2], A * x[3]};
      lane16_sums<2 + kZq>(m);
      const double iA = m[0] == 0.0 ? 0.0 : 1.0 / m[0];
      const double mu = m[2] * iA, mv = m[3] * iA, mT = m[4] * iA;   // as k_zreduce forms them
      const double du = x[0] - mu, dv = x[1] - mv, dT = x[2] - mT;
      double co[5] = {A * du * dv, A * dv * dT, A * du, A * dv, A * dT};
      lane16_sums<5>(co);
      if (cb < kZrec && i / kZcols < nj) {
        double v = m[0];
#pragma unroll
        for (int q = 1; q < kZrec; ++q)
          if (cb == q) v = q < 6 ? m[q < 6 ? q : 0] : co[q < 6 ? 0 : q - 6];
        P[((size_t)(j0 + jj) * gridDim.x + blockIdx.x) * kZrec + cb] = v;
      }
    }
    __syncthreads();   // the table is free
  }
}

// Sums of NV values per thread over the workgroup, in a fixed order (across
// the wavefront's lanes, then the wavefronts), to every thread.
template <int NV>
__device__ __forceinline__ void block_sums(double v[NV], double (*sm)[NV]) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], o, 64);
  __syncthreads();   // the previous sums have been read
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) sm[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = ((sm[0][k] + sm[1][k]) + sm[2][k]) + sm[3][k];
}

// A wavefront per band and pressure level: area-weighted means of the band's
// columns that have a value, then the eddy products, from the band's tiles
// toff[b] .. toff[b + 1] - 1 (lane t takes tiles t, t + 64, ...); added to the
// time sums S[b][j][0..6] = u, v, T, theta, [u'v'], [v'T'], valid fraction and
// to the snapshot count S[b][j][7].  The last workgroup of a band: the
// area-weighted mean of the first-layer w over all of its columns, then each
// column's deviation from it added to the time sum Wsum[column].
// Bound by latency; g6 L32, 20 levels, 36 bands: 14 us from every column's
// values, 8.5 from the records.
__global__ __launch_bounds__(kZthreads) void k_zreduce(const double *P, const double *Zw, int np, int n_tiles,
                                                       const int32_t *toff, const int32_t *off, const int32_t *cols,
                                                       const double *area, double *S, double *Wsum) {
  __shared__ double sm[kZthreads / 64][2];
  const int b = blockIdx.x, a0 = off[b], a1 = off[b + 1];
  if (a0 == a1) return;   // empty band (a snapshot of 4096 bands over 162 columns: 36 -> 12.5 us)
  if (blockIdx.y == gridDim.y - 1) {
    double s[2] = {0, 0};
    for (int i = a0 + threadIdx.x; i < a1; i += kZthreads) {
      s[0] += area[i];
      s[1] += area[i] * Zw[i];
    }
    block_sums<2>(s, sm);
    const double mw = s[1] / s[0];
    for (int i = a0 + threadIdx.x; i < a1; i += kZthreads) Wsum[cols[i]] += Zw[i] - mw;
    return;
  }
  const int j = blockIdx.y * (kZthreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= np) return;
  const int t0 = toff[b], t1 = toff[b + 1];
  const double *rec = P + (size_t)j * n_tiles * kZrec;
  double s[6] = {0, 0, 0, 0, 0, 0};   // A, band area, u, v, T, theta
  for (int t = t0 + lane; t < t1; t += 64)
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] += rec[(size_t)t * kZrec + k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] += __shfl_xor(s[k], o, 64);
  const double sA = s[0];
  if (sA == 0.0) return;   // uniform across the wavefront
  const double mu = s[2] / sA, mv = s[3] / sA, mT = s[4] / sA, mth = s[5] / sA, frac = sA / s[1];
  double e0 = 0.0, e1 = 0.0;
  for (int t = t0 + lane; t < t1; t += 64) {
    const double *r = rec + (size_t)t * kZrec;
    const double iA = r[0] == 0.0 ? 0.0 : 1.0 / r[0];
    // co-moments about the band's means: the tile's own, and the area times
    // the deviations of its means, which are the rounded means the tile used
    // and what its values leave over them
    const double tu = r[2] * iA, tv = r[3] * iA, tT = r[4] * iA;
    const double du = (tu - mu) + r[8] * iA, dv = (tv - mv) + r[9] * iA, dT = (tT - mT) + r[10] * iA;
    e0 += r[6] + r[0] * (du * dv);
    e1 += r[7] + r[0] * (dv * dT);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    e0 += __shfl_xor(e0, o, 64);
    e1 += __shfl_xor(e1, o, 64);
  }
  if (lane == 0) {
    double *o = S + ((size_t)b * np + j) * 8;
    o[0] += mu;
    o[1] += mv;
    o[2] += mT;
    o[3] += mth;
    o[4] += e0 / sA;
    o[5] += e1 / sA;
    o[6] += frac;
    o[7] += 1.0;
  }
}

__global__ void k_zzero(double *S, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) S[i] = 0.0;
}

size_t a256z(size_t x) { return (x + 255) & ~(size_t)255; }

// Partial sums per workgroup (4 wavefronts, lanes = levels) of the absolute
// angular momentum about the rotation axis of the state between large steps:
// per cell (R x rho v)_z with R = r_C rhat, plus rho Omega r_C^2 cos^2(lat),
// times the volume A_c r_C^2 dz; fixed reduction order.
template <typename H>
__global__ __launch_bounds__(256) void k_angmom(Fields<H> f, Consts c, double *out) {
  __shared__ double sm[4];
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int L = c.L, cpw = 64 / L;
  const int cw = lane / L, lev = lane - cw * L;
  const int col = wave * cpw + cw;
  double v = 0.0;
  if (cw < cpw && col < c.N) {
    const size_t idx = (size_t)col * c.S + lev;
    const double rC = c.radius + (lev + 0.5) * c.rdz;
    const H *rh = f.rhat + (size_t)col * 3;
    const double x = rh[0], y = rh[1];
    const double rel = rC * (x * (double)f.My_t[idx] - y * (double)f.Mx_t[idx]);
    const double plan = f.rho_t[idx] * c.omega * rC * rC * (x * x + y * y);
    v = (rel + plan) * f.area[col] * rC * rC * c.dz;
  }
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if (lane == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = ((sm[0] + sm[1]) + sm[2]) + sm[3];
}

}  // namespace

template <typename H>
void launch_angmom(const Fields<H> &f, const Consts &c, double *out, hipStream_t s, int *nblocks_out) {
  const long waves = (c.N + 64 / c.L - 1) / (64 / c.L);
  const int nb = (int)((waves + 3) / 4);
  *nblocks_out = nb;
  hipLaunchKernelGGL(k_angmom<H>, dim3(nb), dim3(256), 0, s, f, c, out);
}
template void launch_angmom<double>(const Fields<double> &, const Consts &, double *, hipStream_t, int *);
template void launch_angmom<float>(const Fields<float> &, const Consts &, double *, hipStream_t, int *);

}  // namespace thor

using namespace thor;

struct thor_zonal {
  thor_state *s = nullptr;
  int nb = 0, np = 0;
  std::vector<double> plev_h;
  double radius = 0, gravity = 0;
  double *plev = nullptr, *P = nullptr, *S = nullptr, *area = nullptr, *Zw = nullptr, *Wsum = nullptr;
  int32_t *off = nullptr, *cols = nullptr, *toff = nullptr;
  int2 *tiles = nullptr;
  int n_tiles = 0;
  int snapshots = 0;
};

namespace {

size_t zonal_layout(thor_zonal *z, size_t N, char *base) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char * {
    char *p = base ? base + off : nullptr;
    off += a256z(bytes);
    return p;
  };
  z->plev = (double *)take(z->np * sizeof(double));
  const size_t tiles = std::min(N, N / kZcols + z->nb);   // at most: one partly filled tile per band, none empty
  z->P = (double *)take(tiles * z->np * kZrec * sizeof(double));
  z->tiles = (int2 *)take(tiles * sizeof(int2));
  z->toff = (int32_t *)take((z->nb + 1) * sizeof(int32_t));
  z->S = (double *)take((size_t)z->nb * z->np * 8 * sizeof(double));
  z->area = (double *)take(N * sizeof(double));
  z->off = (int32_t *)take((z->nb + 1) * sizeof(int32_t));
  z->cols = (int32_t *)take(N * sizeof(int32_t));
  z->Zw = (double *)take(N * sizeof(double));
  z->Wsum = (double *)take(N * sizeof(double));
  return off;
}

bool zonal_args(const thor_state *s, int n_bands, const double *plev, int n_plev) {
  if (!s || !plev) { set_error("thor_zonal: NULL argument"); return false; }
  if (n_bands < 1 || n_bands > 4096 || n_plev < 1 || n_plev > 1024) {
    set_error("thor_zonal: need 1..4096 bands and 1..1024 pressure levels");
    return false;
  }
  for (int j = 0; j < n_plev; ++j)
    if (!(plev[j] > 0) || (j > 0 && !(plev[j] > plev[j - 1]))) {
      set_error("thor_zonal: pressure levels must be positive and strictly ascending");
      return false;
    }
  return true;
}

}  // namespace

extern "C" {

int thor_zonal_bytes(const thor_state *s, int n_bands, const double *plev, int n_plev, size_t *bytes) {
  clear_error();
  if (!bytes || !zonal_args(s, n_bands, plev, n_plev)) {
    if (!bytes) set_error("thor_zonal_bytes: NULL argument");
    return THOR_EINVAL;
  }
  thor_zonal z;
  z.nb = n_bands;
  z.np = n_plev;
  *bytes = zonal_layout(&z, (size_t)s->n_col, nullptr);
  return THOR_OK;
}

int thor_zonal_init(thor_state *s, const thor_grid *g, double radius, double gravity, int n_bands,
                    const double *plev, int n_plev, void *dev_buf, size_t dev_bytes, thor_zonal **out) {
  clear_error();
  if (!out || !g || !dev_buf) { set_error("thor_zonal_init: NULL argument"); return THOR_EINVAL; }
  *out = nullptr;
  if (!zonal_args(s, n_bands, plev, n_plev)) return THOR_EINVAL;
  if (g->g.n != s->n_col) { set_error("thor_zonal_init: grid does not match the state"); return THOR_EINVAL; }
  if (!(radius > 0 && gravity > 0)) { set_error("thor_zonal_init: radius and gravity must be positive"); return THOR_EINVAL; }
  if (((uintptr_t)dev_buf & 255) != 0) { set_error("thor_zonal_init: dev_buf must be 256-byte aligned"); return THOR_EINVAL; }
  thor_zonal *z = new (std::nothrow) thor_zonal;
  if (!z) { set_error("thor_zonal_init: out of host memory"); return THOR_ENOMEM; }
  z->s = s;
  z->nb = n_bands;
  z->np = n_plev;
  z->plev_h.assign(plev, plev + n_plev);
  z->radius = radius;
  z->gravity = gravity;
  const size_t N = (size_t)s->n_col;
  if (dev_bytes < zonal_layout(z, N, nullptr)) {
    delete z;
    set_error("thor_zonal_init: dev_bytes smaller than thor_zonal_bytes");
    return THOR_ENOMEM;
  }
  zonal_layout(z, N, (char *)dev_buf);
  // latitude bands, columns in increasing id within a band
  std::vector<int32_t> off(n_bands + 1, 0), cols(N);
  std::vector<int> band(N);
  for (size_t i = 0; i < N; ++i) {
    const double lat = std::asin(std::fmin(1.0, std::fmax(-1.0, g->g.pos[i].z)));
    int b = (int)std::floor((lat + M_PI / 2) / M_PI * n_bands);
    band[i] = std::min(std::max(b, 0), n_bands - 1);
    off[band[i] + 1] += 1;
  }
  for (int b = 0; b < n_bands; ++b) off[b + 1] += off[b];
  std::vector<int32_t> fill(off.begin(), off.end() - 1);
  for (size_t i = 0; i < N; ++i) cols[fill[band[i]]++] = (int32_t)i;
  std::vector<int32_t> toff(n_bands + 1, 0);
  std::vector<int2> tiles;
  for (int b = 0; b < n_bands; ++b) {
    for (int i = off[b]; i < off[b + 1]; i += kZcols) tiles.push_back(make_int2(i, std::min(kZcols, off[b + 1] - i)));
    toff[b + 1] = (int32_t)tiles.size();
  }
  z->n_tiles = (int)tiles.size();
  std::vector<double> area(N);   // in band order, as Zw
  for (size_t i = 0; i < N; ++i) area[i] = g->g.area[cols[i]];
  hipStream_t st = s->stream;
  const size_t ns = (size_t)n_bands * n_plev * 8;
  bool ok = zok(hipMemcpyAsync(z->plev, plev, n_plev * sizeof(double), hipMemcpyHostToDevice, st), "copy plev") &&
            zok(hipMemcpyAsync(z->area, area.data(), N * sizeof(double), hipMemcpyHostToDevice, st), "copy area") &&
            zok(hipMemcpyAsync(z->off, off.data(), off.size() * sizeof(int32_t), hipMemcpyHostToDevice, st), "copy off") &&
            zok(hipMemcpyAsync(z->toff, toff.data(), toff.size() * sizeof(int32_t), hipMemcpyHostToDevice, st), "copy toff") &&
            zok(hipMemcpyAsync(z->tiles, tiles.data(), tiles.size() * sizeof(int2), hipMemcpyHostToDevice, st), "copy tiles") &&
            zok(hipMemcpyAsync(z->cols, cols.data(), N * sizeof(int32_t), hipMemcpyHostToDevice, st), "copy cols");
  if (ok) {
    hipLaunchKernelGGL(k_zzero, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, st, z->S, ns);
    hipLaunchKernelGGL(k_zzero, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, z->Wsum, N);
    ok = zok(hipGetLastError(), "zero sums") && zok(hipStreamSynchronize(st), "zonal init synchronize");
  }
  if (!ok) { delete z; return THOR_EHIP; }
  *out = z;
  return THOR_OK;
}

int thor_zonal_accumulate(thor_zonal *z) {
  clear_error();
  if (!z) { set_error("thor_zonal_accumulate: NULL argument"); return THOR_EINVAL; }
  thor_state *s = z->s;
  const dim3 g((unsigned)z->n_tiles), t(kZthreads);
  const unsigned lds = (unsigned)(kZslot * s->c.L * kZpitch * sizeof(double));   // 43520 bytes at 64 levels
  if (s->precision == THOR_MIXED)
    hipLaunchKernelGGL(k_zinterp<float>, g, t, lds, s->stream, s->f32[s->parity], s->c, z->cols, z->tiles, z->area,
                       z->plev, z->np, z->P, z->Zw);
  else
    hipLaunchKernelGGL(k_zinterp<double>, g, t, lds, s->stream, s->f64[s->parity], s->c, z->cols, z->tiles, z->area,
                       z->plev, z->np, z->P, z->Zw);
  hipLaunchKernelGGL(k_zreduce, dim3(z->nb, (z->np + 3) / 4 + 1), t, 0, s->stream, z->P, z->Zw, z->np, z->n_tiles,
                     z->toff, z->off, z->cols, z->area, z->S, z->Wsum);
  if (!zok(hipGetLastError(), "zonal accumulate")) return THOR_EHIP;
  z->snapshots += 1;
  return THOR_OK;
}

int thor_zonal_result(thor_zonal *z, double *host_out, int *n_snapshots) {
  clear_error();
  if (!z || !host_out) { set_error("thor_zonal_result: NULL argument"); return THOR_EINVAL; }
  const int nb = z->nb, np = z->np;
  std::vector<double> S((size_t)nb * np * 8);
  if (!zok(hipMemcpyAsync(S.data(), z->S, S.size() * sizeof(double), hipMemcpyDeviceToHost, z->s->stream), "copy sums") ||
      !zok(hipStreamSynchronize(z->s->stream), "zonal result synchronize"))
    return THOR_EHIP;
  for (int b = 0; b < nb; ++b) {
    const double lat = -M_PI / 2 + (b + 0.5) * M_PI / nb;
    const double fac = 2.0 * M_PI * z->radius * std::cos(lat) / z->gravity;
    double integ = 0.0, v_prev = 0.0, p_prev = 0.0;
    for (int j = 0; j < np; ++j) {
      const double *s = &S[((size_t)b * np + j) * 8];
      double *o = host_out + ((size_t)b * np + j) * THOR_ZM_COUNT;
      const double n = s[7];
      for (int k = 0; k < 7; ++k) o[k] = n > 0 ? s[k] / n : 0.0;
      const double v = o[THOR_ZM_V];
      integ = j == 0 ? v * z->plev_h[0] : integ + 0.5 * (v + v_prev) * (z->plev_h[j] - p_prev);
      o[THOR_ZM_PSI] = fac * integ;
      o[THOR_ZM_SNAPSHOTS] = n;
      v_prev = v;
      p_prev = z->plev_h[j];
    }
  }
  if (n_snapshots) *n_snapshots = z->snapshots;
  return THOR_OK;
}

int thor_zonal_imprint(thor_zonal *z, double *host_out, int *n_snapshots) {
  clear_error();
  if (!z || !host_out) { set_error("thor_zonal_imprint: NULL argument"); return THOR_EINVAL; }
  const size_t N = (size_t)z->s->n_col;
  if (!zok(hipMemcpyAsync(host_out, z->Wsum, N * sizeof(double), hipMemcpyDeviceToHost, z->s->stream), "copy imprint") ||
      !zok(hipStreamSynchronize(z->s->stream), "zonal imprint synchronize"))
    return THOR_EHIP;
  const double n = z->snapshots;
  for (size_t i = 0; i < N; ++i) host_out[i] = n > 0 ? host_out[i] / n : 0.0;
  if (n_snapshots) *n_snapshots = z->snapshots;
  return THOR_OK;
}

int thor_zonal_reset(thor_zonal *z) {
  clear_error();
  if (!z) { set_error("thor_zonal_reset: NULL argument"); return THOR_EINVAL; }
  const size_t ns = (size_t)z->nb * z->np * 8;
  const size_t N = (size_t)z->s->n_col;
  hipLaunchKernelGGL(k_zzero, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, z->s->stream, z->S, ns);
  hipLaunchKernelGGL(k_zzero, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, z->s->stream, z->Wsum, N);
  z->snapshots = 0;
  return zok(hipGetLastError(), "zonal reset") ? THOR_OK : THOR_EHIP;
}

void thor_zonal_free(thor_zonal *z) { delete z; }

}  // extern "C"

// ===========================================================================
// Measurement aid: streaming kernel with a given read/write mix.
// ===========================================================================
namespace {
struct StreamPtrs {
  const double *src[16];
  double *dst[8];
};

// NS sources unrolled (every load issued before the sum uses it), the stores
// in a loop.
template <int NS>
__global__ __launch_bounds__(256) void k_stream_mix(StreamPtrs p, int n_dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) v[k] = p.src[k][i];
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < NS; ++k) acc += v[k];
  for (int k = 0; k < n_dst; ++k) p.dst[k][i] = acc + k;
}

template <int NS>
void launch_stream_mix(int n_src, const StreamPtrs &p, int n_dst, int64_t n, unsigned blocks, hipStream_t s) {
  if (n_src == NS) hipLaunchKernelGGL(k_stream_mix<NS>, dim3(blocks), dim3(256), 0, s, p, n_dst, n);
  else if constexpr (NS > 1) launch_stream_mix<NS - 1>(n_src, p, n_dst, n, blocks, s);
}
}  // namespace

extern "C" int thor_stream_mix(const double *const *src, int n_src, double *const *dst, int n_dst, int64_t n,
                               void *hip_stream) {
  thor::clear_error();
  if (!src || !dst || n_src < 1 || n_src > 16 || n_dst < 1 || n_dst > 8 || n < 1) {
    thor::set_error("thor_stream_mix: 1..16 sources, 1..8 destinations, n >= 1");
    return THOR_EINVAL;
  }
  StreamPtrs p{};
  for (int k = 0; k < n_src; ++k) {
    if (!src[k]) { thor::set_error("thor_stream_mix: NULL source"); return THOR_EINVAL; }
    p.src[k] = src[k];
  }
  for (int k = 0; k < n_dst; ++k) {
    if (!dst[k]) { thor::set_error("thor_stream_mix: NULL destination"); return THOR_EINVAL; }
    p.dst[k] = dst[k];
  }
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffff) { thor::set_error("thor_stream_mix: n too large"); return THOR_EINVAL; }
  launch_stream_mix<16>(n_src, p, n_dst, n, (unsigned)blocks, (hipStream_t)hip_stream);
  if (hipGetLastError() != hipSuccess) { thor::set_error("thor_stream_mix: launch failed"); return THOR_EHIP; }
  return THOR_OK;
}
