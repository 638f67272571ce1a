// Disc diagnostics of the paper's analysis (Sec. 4.2 and 5.2-5.4): heat of
// the disc with the mean circular velocity from radial bins of equal
// particle numbers, RMS thickness per bin, vertical density profile and
// velocity dispersions in an annulus.  The radial order is by FP64 radius,
// ties in the caller's particle order.  Every sum except the vertical profile
// is reduced in a fixed order.
#include <type_traits>

#include "ctx.h"

using namespace sbx;

namespace {

constexpr int kRsTile = 1024;  // elements per radix block (one wavefront, 16 chunks)
constexpr int kRsChunks = kRsTile / 64;
constexpr int kMaxBins = 2048;
constexpr int kMaxZ = 1024;
constexpr int kAnBlocks = 512;  // blocks of the heat / annulus pass
constexpr int kBulkBlocks = 1024;
// per-block partial row: heat, annulus count, sum vR, vR^2, vphi, vphi^2, vz, vz^2
constexpr int kAnVals = 8;

// ------------------------------------------------------------- selection --
// The disc particles are numbered in the caller's order (k = 0, 1, ...): a bit
// per particle, set at its caller's index, the popcounts of the words scanned.
// Bits instead of a word per particle keep the scattered writes of the 8.5M
// galaxy in 1 MB (169 -> 84 us).
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_mask(PartDev<T> p, int comp, int gal, uint32_t* __restrict__ mask) {
  const int lane = threadIdx.x & 63;
  const int64_t rounds = (p.n + 63) / 64;
  for (int64_t w = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6; w < rounds; w += (int64_t)gridDim.x * 4) {
    const int64_t i = w * 64 + lane;
    const bool in = i < p.n;
    const int32_t id = in ? p.id[i] : 0;
    const bool sel = in && p.comp[i] == comp && p.gal[i] == gal && !p.lost[i];
    const uint64_t bits = __ballot(sel);
    const int32_t id0 = __builtin_amdgcn_readfirstlane(id);
    const int here = p.n - w * 64 < 64 ? (int)(p.n - w * 64) : 64;
    if (__ballot(in && id != id0 + lane) == 0ull && (id0 & 63) == 0 && (here == 64 || id0 + here == p.n)) {
      // the caller's own order: this wavefront holds every number of its
      // words.  The last one, if it is not full, does so only where its
      // numbers are the highest: the rest of its words lies elsewhere else.
      if (in && (lane & 31) == 0) mask[id >> 5] = (uint32_t)(bits >> lane);
    } else if (sel) {
      __hip_atomic_fetch_or(mask + (id >> 5), 1u << (id & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

__global__ void __launch_bounds__(256)
    k_disc_popc(const uint32_t* __restrict__ mask, int64_t words, uint32_t* __restrict__ cnt) {
  const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (w <= words) cnt[w] = w < words ? (uint32_t)__popc(mask[w]) : 0u;
}

// One disc particle as it is held: x, y, z, vx, vy, vz, m, and its place in
// its radial bucket (bits).
template <typename T>
struct alignas(16) DiscRec {
  T v[8];
};
template <typename T>
__device__ __forceinline__ T put_bits(uint32_t u) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, u);
  else return __builtin_bit_cast(T, (uint64_t)u);
}
__device__ __forceinline__ uint32_t get_bits(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t get_bits(double v) { return (uint32_t)__builtin_bit_cast(uint64_t, v); }

template <typename T>
__device__ __forceinline__ DiscRec<T> load_rec(const DiscRec<T>* __restrict__ rec, size_t k) {
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int W = 16 / sizeof(T);
  DiscRec<T> r;
  const gp<const vec> s = glb((const vec*)(rec + k));
#pragma unroll
  for (int q = 0; q < 8 / W; ++q) {
    const vec x = s[q];
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[q * W + e] = x[e];
  }
  return r;
}

// The galaxy's centre: of the last solve (on the device), else as given.
struct Centre {
  const double* dev;
  double c[3];
  __device__ __forceinline__ double at(int k) const { return dev ? dev[k] : c[k]; }
};

// Cylindrical radius, each operation rounded (the radial order depends on it).
__device__ __forceinline__ double cyl_r(double dx, double dy) {
#pragma clang fp contract(off)
  return sqrt(dx * dx + dy * dy);
}

// Radial buckets: 2^bits per octave of R over 24 octaves up to `top`, what
// lies outside in the first and the last; a bucket's radii are all below the
// next one's.
struct Buckets {
  int base, shift, count;
  __device__ __forceinline__ int of(double r) const {
    const int hi = (int)(__double_as_longlong(r) >> 32) - base;
    const int b = hi < 0 ? 0 : hi >> shift;
    return b < count ? b : count - 1;
  }
};

// Records in the caller's order; each particle takes a place in its bucket.
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_compact(PartDev<T> p, int comp, int gal, const uint32_t* __restrict__ mask,
                   const uint32_t* __restrict__ cnt, Centre cen, Buckets bk, uint32_t* __restrict__ fill,
                   DiscRec<T>* __restrict__ rec) {
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int W = 16 / sizeof(T);
  const double cx = cen.at(0), cy = cen.at(1);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < p.n; i += (int64_t)gridDim.x * 256) {
    if (!(p.comp[i] == comp && p.gal[i] == gal && !p.lost[i])) continue;
    const uint32_t id = (uint32_t)p.id[i];
    DiscRec<T> r;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      r.v[k] = p.x[k][i];
      r.v[3 + k] = p.v[k][i];
    }
    r.v[6] = p.m[i];
    const uint32_t k = cnt[id >> 5] + (uint32_t)__popc(mask[id >> 5] & ((1u << (id & 31)) - 1u));
    const int b = bk.of(cyl_r((double)r.v[0] - cx, (double)r.v[1] - cy));
    r.v[7] = put_bits<T>(__hip_atomic_fetch_add(fill + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const gp<vec> d = glb((vec*)(rec + k));
#pragma unroll
    for (int q = 0; q < 8 / W; ++q) {
      vec x;
#pragma unroll
      for (int e = 0; e < W; ++e) x[e] = r.v[q * W + e];
      d[q] = x;
    }
  }
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Fixed-order sum of nv values over a 256-thread block into out[0..nv).
template <int NV>
__device__ __forceinline__ void block_rows(const double* vals, double* out) {
  __shared__ double red[4][NV];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double s = wsum(vals[k]);
    if (lane == 0) red[wave][k] = s;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < NV; k += blockDim.x) out[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
}

// column sums of rows x nv partials (one block per column, fixed order)
__global__ void __launch_bounds__(256)
    k_columns(const double* __restrict__ part, int rows, int nv, double* __restrict__ out) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  double s = 0.0;
  for (int r = threadIdx.x; r < rows; r += 256) s += part[(size_t)r * nv + c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[c] = red[0];
}

// Radial key (R >= 0: the bits order like the values) and number of a particle.
struct alignas(16) RadKey {
  uint64_t r;
  uint32_t k, pad;
};

// The records in order: keys to their buckets (start: the scanned counts),
// and the sums of m and m v over the disc (block partials).
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_keys(const DiscRec<T>* __restrict__ rec, int64_t n, Centre cen, Buckets bk,
                const uint32_t* __restrict__ start, RadKey* __restrict__ key, double* __restrict__ part) {
  const double cx = cen.at(0), cy = cen.at(1);
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const DiscRec<T> r = load_rec(rec, i);
    const double R = cyl_r((double)r.v[0] - cx, (double)r.v[1] - cy);
    const double m = (double)r.v[6];
    a[0] += m;
    a[1] += m * (double)r.v[3];
    a[2] += m * (double)r.v[4];
    a[3] += m * (double)r.v[5];
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const uint64_t u = (uint64_t)__double_as_longlong(R);
    glb((u4*)key)[start[bk.of(R)] + get_bits(r.v[7])] = u4{(uint32_t)u, (uint32_t)(u >> 32), (uint32_t)i, 0u};
  }
  block_rows<4>(a, part + 4 * (size_t)blockIdx.x);
}

// Every bucket sorted by (radius, number): its keys in the wavefront's LDS,
// a key's place the number of smaller ones.  Buckets of more than kBucketCap
// raise the flag and leave their part of the order unset: what reads the
// order does nothing while the flag stands, and the radix sort below then
// orders the whole disc.  Bound by the chain of each bucket (bounds, keys,
// comparisons): with a bucket per 64, 128 and 256 particles the whole call
// took 1.00, 0.97 and 1.01 ms.  Eight 8-bit radix passes of the 64-bit radii
// took 590 us for 2M particles; scattering the keys and this take 98 us.
constexpr int kBucketCap = 768;  // 36 KB of LDS a block: four on a CU
__global__ void __launch_bounds__(256)
    k_disc_order(const RadKey* __restrict__ key, const uint32_t* __restrict__ start, int buckets,
                 uint64_t* __restrict__ skey, uint32_t* __restrict__ order, uint32_t* __restrict__ flag) {
  __shared__ uint64_t rs[4][kBucketCap];
  __shared__ uint32_t ks[4][kBucketCap];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t* const R = rs[wave];
  uint32_t* const K = ks[wave];
  for (int b = (int)blockIdx.x * 4 + wave; b < buckets; b += (int)gridDim.x * 4) {
    const uint32_t s0 = start[b];
    const int m = (int)(start[b + 1] - s0);
    if (m == 0) continue;
    if (m > kBucketCap) {
      if (lane == 0) *flag = 1u;
      continue;
    }
    for (int e = lane; e < m; e += 64) {
      const RadKey q = key[s0 + e];
      R[e] = q.r;
      K[e] = q.k;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int e0 = 0; e0 < m; e0 += 128) {  // two keys a lane per walk
      const int ea = e0 + lane, eb = ea + 64;
      const uint64_t ra = R[ea < m ? ea : 0], rb = R[eb < m ? eb : 0];
      const uint32_t ka = K[ea < m ? ea : 0], kb = K[eb < m ? eb : 0];
      uint32_t pa = 0, pb = 0;
#pragma unroll 4
      for (int j = 0; j < m; ++j) {
        const uint64_t rj = R[j];
        const uint32_t kj = K[j];
        pa += (rj < ra || (rj == ra && kj < ka)) ? 1u : 0u;
        pb += (rj < rb || (rj == rb && kj < kb)) ? 1u : 0u;
      }
      if (ea < m) {
        skey[s0 + pa] = ra;
        order[s0 + pa] = ka;
      }
      if (eb < m) {
        skey[s0 + pb] = rb;
        order[s0 + pb] = kb;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Cylindrical quantities of a record relative to the disc's mean velocity.
struct Cyl {
  double R, vR, vphi, vz, dz;
};
template <typename T>
__device__ __forceinline__ Cyl cyl_of(const DiscRec<T>& r, const double* c, const double* b) {
#pragma clang fp contract(off)
  Cyl o;
  const double dx = (double)r.v[0] - c[0], dy = (double)r.v[1] - c[1];
  const double ux = (double)r.v[3] - b[0], uy = (double)r.v[4] - b[1];
  o.R = cyl_r(dx, dy);
  o.vR = o.R > 0.0 ? (dx * ux + dy * uy) / o.R : 0.0;
  o.vphi = o.R > 0.0 ? (dx * uy - dy * ux) / o.R : 0.0;
  o.vz = (double)r.v[5] - b[2];
  o.dz = (double)r.v[2] - c[2];
  return o;
}
__device__ __forceinline__ void frame(const Centre& cen, const double* bulk, double* c, double* b) {
  for (int k = 0; k < 3; ++k) {
    c[k] = cen.at(k);
    b[k] = bulk ? bulk[1 + k] / bulk[0] : 0.0;
  }
}

// keys of the whole disc in the caller's order, for the radix sort
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_radii(const DiscRec<T>* __restrict__ rec, int64_t n, Centre cen, uint64_t* __restrict__ key,
                 uint32_t* __restrict__ val) {
  const double cx = cen.at(0), cy = cen.at(1);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const DiscRec<T> r = load_rec(rec, i);
    key[i] = (uint64_t)__double_as_longlong(cyl_r((double)r.v[0] - cx, (double)r.v[1] - cy));
    val[i] = (uint32_t)i;
  }
}

// ------------------------------------------------------------ radix sort --
__device__ __forceinline__ int digit_of(uint64_t k, int shift) { return (int)((k >> shift) & 0xFF); }

// per-tile histogram of one 8-bit digit, stored digit-major: cnt[d * nb + b]
__global__ void __launch_bounds__(64)
    k_rs_hist(const uint64_t* __restrict__ key, int64_t n, int shift, int nb, uint32_t* __restrict__ cnt) {
  __shared__ uint32_t h[256];
  for (int d = threadIdx.x; d < 256; d += 64) h[d] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRsTile;
  for (int c = 0; c < kRsChunks; ++c) {
    const int64_t e = base + c * 64 + threadIdx.x;
    if (e < n) atomicAdd(h + digit_of(key[e], shift), 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < 256; d += 64) cnt[(size_t)d * nb + blockIdx.x] = h[d];
}

// stable scatter: within a tile, elements keep their order (chunks in
// order, lanes in order: rank among equal digits by ballots)
__global__ void __launch_bounds__(64)
    k_rs_scatter(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin, int64_t n,
                 int shift, int nb, const uint32_t* __restrict__ off, uint64_t* __restrict__ kout,
                 uint32_t* __restrict__ vout) {
  __shared__ uint32_t o[256];
  const int lane = threadIdx.x;
  for (int d = lane; d < 256; d += 64) o[d] = off[(size_t)d * nb + blockIdx.x];
  __syncthreads();
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int64_t base = (int64_t)blockIdx.x * kRsTile;
  for (int c = 0; c < kRsChunks; ++c) {
    const int64_t e = base + c * 64 + lane;
    const bool ok = e < n;
    const uint64_t k = ok ? kin[e] : 0ull;
    const int d = digit_of(k, shift);
    uint64_t match = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(ok && bit);
      match &= bit ? bb : ~bb;
    }
    const int rank = __popcll(match & lt);
    const uint32_t start = ok ? o[d] : 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (ok) {
      kout[start + rank] = k;
      vout[start + rank] = vin[e];
      if (rank == 0) o[d] = start + (uint32_t)__popcll(match);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// ------------------------------------------------------------------- bins --
// mean R, mean v_phi, RMS z over a bin's range of the sorted order (bin k:
// n / nbins items, plus one for k < n % nbins).  A bin is split over
// gridDim.y blocks (one block a bin left most of the chip idle), whose sums
// are added in order by k_disc_bins_end.
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_bins(const uint32_t* __restrict__ order, int64_t n, int nbins, const DiscRec<T>* __restrict__ rec,
                Centre cen, const double* __restrict__ bulk, const uint32_t* __restrict__ flag,
                double* __restrict__ part) {
  if (*flag) return;  // no order yet
  const int k = blockIdx.x;
  const int64_t q = n / nbins, r = n % nbins;
  const int64_t s0 = k * q + (k < r ? k : r);
  const int64_t s1 = s0 + q + (k < r ? 1 : 0);
  double c[3], b[3];
  frame(cen, bulk, c, b);
  double a[3] = {0.0, 0.0, 0.0};
  for (int64_t j = s0 + (int64_t)blockIdx.y * 256 + threadIdx.x; j < s1; j += (int64_t)gridDim.y * 256) {
    const Cyl y = cyl_of(load_rec(rec, order[j]), c, b);
    a[0] += y.R;
    a[1] += y.vphi;
    a[2] += y.dz * y.dz;
  }
  block_rows<3>(a, part + 3 * ((size_t)k * gridDim.y + blockIdx.y));
}

__global__ void __launch_bounds__(256)
    k_disc_bins_end(const double* __restrict__ part, int split, int64_t n, int nbins,
                    double* __restrict__ bin_r, double* __restrict__ bin_vc, double* __restrict__ bin_rz) {
  const int k = (int)blockIdx.x * 256 + threadIdx.x;
  if (k >= nbins) return;
  double s[3] = {0.0, 0.0, 0.0};
  for (int q = 0; q < split; ++q)
    for (int e = 0; e < 3; ++e) s[e] += part[3 * ((size_t)k * split + q) + e];
  const double c = (double)(n / nbins + (k < n % nbins ? 1 : 0));
  bin_r[k] = c > 0 ? s[0] / c : 0.0;
  bin_vc[k] = c > 0 ? s[1] / c : 0.0;
  bin_rz[k] = c > 0 ? sqrt(s[2] / c) : 0.0;
}

// heat with the interpolated circular velocity; annulus sums; z profile
template <typename T>
__global__ void __launch_bounds__(256)
    k_disc_heat(int64_t n, int nbins, const double* __restrict__ bin_r, const double* __restrict__ bin_vc,
                const DiscRec<T>* __restrict__ rec, Centre cen, const double* __restrict__ bulk, double lo,
                double hi, int nz, double zmax, double* __restrict__ part, double* __restrict__ zpart) {
  extern __shared__ double sh[];  // bin_r, bin_vc (nbins each), then nz profile bins
  double* br = sh;
  double* bv = sh + nbins;
  double* hz = sh + 2 * nbins;
  for (int k = threadIdx.x; k < nbins; k += 256) {
    br[k] = bin_r[k];
    bv[k] = bin_vc[k];
  }
  for (int k = threadIdx.x; k < nz; k += 256) hz[k] = 0.0;
  double cc[3], bb[3];
  frame(cen, bulk, cc, bb);
  __syncthreads();
  const double dz = 2.0 * zmax / nz;
  double a[kAnVals] = {};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const DiscRec<T> rc = load_rec(rec, i);
    const Cyl y = cyl_of(rc, cc, bb);
    const double r = y.R, m = (double)rc.v[6];
    // vbar_c(r): linear between the bins' mean radii, constant beyond the ends
    double vc;
    if (r <= br[0]) {
      vc = bv[0];
    } else if (r >= br[nbins - 1]) {
      vc = bv[nbins - 1];
    } else {
      int lo_k = 0, hi_k = nbins - 1;  // br[lo_k] < r < br[hi_k]
      while (hi_k - lo_k > 1) {
        const int mid = (lo_k + hi_k) >> 1;
        if (br[mid] <= r) lo_k = mid;
        else hi_k = mid;
      }
      const double t = (r - br[lo_k]) / (br[hi_k] - br[lo_k]);
      vc = bv[lo_k] + t * (bv[hi_k] - bv[lo_k]);
    }
    const double a_r = y.vR, a_p = y.vphi, a_z = y.vz;
    const double dp = a_p - vc;
    a[0] += 0.5 * m * ((a_r * a_r + dp * dp) + a_z * a_z);
    if (r >= lo && r < hi) {
      a[1] += 1.0;
      a[2] += a_r;
      a[3] += a_r * a_r;
      a[4] += a_p;
      a[5] += a_p * a_p;
      a[6] += a_z;
      a[7] += a_z * a_z;
      const double z = y.dz;
      if (z >= -zmax && z < zmax) {
        int k = (int)floor((z + zmax) / dz);
        k = k < nz - 1 ? k : nz - 1;
        atomicAdd(hz + k, m);
      }
    }
  }
  block_rows<kAnVals>(a, part + (size_t)kAnVals * blockIdx.x);
  __syncthreads();
  for (int k = threadIdx.x; k < nz; k += 256) zpart[(size_t)blockIdx.x * nz + k] = hz[k];
}

template <typename T>
PartDev<T> live_set(sbx_ctx* c) {
  const PSet& q = c->set[c->cur];
  PartDev<T> p;
  for (int k = 0; k < 3; ++k) {
    p.x[k] = (T*)q.x[k];
    p.v[k] = (T*)q.v[k];
  }
  p.m = (T*)q.m;
  p.comp = q.comp;
  p.gal = q.gal;
  p.lost = q.lost;
  p.id = q.id;
  p.n = c->n;
  return p;
}

// Work arrays carved from one device buffer of the context, kept between
// calls and grown when a call needs more (allocating and freeing some
// fifteen arrays took over half of a call).
struct Arena {
  sbx_ctx* c;
  size_t at = 0;
  size_t take(size_t bytes) {
    const size_t o = at;
    at += (bytes + 255) & ~(size_t)255;
    return o;
  }
  sbx_status reserve() {
    if (c->an_work_bytes >= at) return SBX_OK;
    SBX_HIP(hipStreamSynchronize(c->stream));
    free_ptr(c->an_work);
    c->an_work_bytes = 0;
    SBX_TRY(dev_alloc(&c->an_work, at));
    c->an_work_bytes = at;
    return SBX_OK;
  }
  template <typename P>
  P* ptr(size_t o) const {
    return (P*)((char*)c->an_work + o);
  }
};

// A prepared disc: records in the caller's order and the radial order.
template <typename T>
struct Disc {
  int64_t n = 0;
  DiscRec<T>* rec = nullptr;
  uint64_t* key = nullptr;    // sorted radius keys (FP64 bits)
  uint32_t* order = nullptr;  // number of the particle at each sorted place
  uint64_t* key2 = nullptr;   // the radix sort's other buffers
  uint32_t *order2 = nullptr, *cnt = nullptr, *ctmp = nullptr;
  double* bulk = nullptr;
  uint32_t* flag = nullptr;   // set when a bucket was too full: radix sort
  void* extra = nullptr;      // the caller's own part of the work buffer
  Centre cen;
};

int rs_blocks(int64_t n) { return (int)((n + kRsTile - 1) / kRsTile); }

// Select the disc (caller order), centre it on the galaxy, sort by radius.
// extra: bytes of work the caller wants for itself.
template <typename T>
sbx_status disc_prepare(sbx_ctx* c, int comp, int galaxy, size_t extra, Disc<T>& D) {
  const int64_t n = c->n, words = (n + 31) / 32;
  hipStream_t s = c->stream;
  const PartDev<T> p = live_set<T>(c);
  D.cen.dev = c->solved ? c->centres + 3 * galaxy : nullptr;
  for (int k = 0; k < 3; ++k) D.cen.c[k] = c->hh[galaxy].centre[k];
  Arena A{c};
  const size_t o_mask = A.take(4 * words), o_cnt = A.take(4 * (words + 1));
  const size_t o_tmp = A.take(4 * scan_tmp_elems(words + 1));
  SBX_TRY(A.reserve());
  uint32_t nd32 = 0;
  {
    uint32_t* mask = A.ptr<uint32_t>(o_mask);
    uint32_t* cnt = A.ptr<uint32_t>(o_cnt);
    SBX_TRY(launch_zero<uint32_t>(mask, words, s));
    hipLaunchKernelGGL((k_disc_mask<T>), dim3(2048), dim3(256), 0, s, p, comp, galaxy, mask);
    hipLaunchKernelGGL(k_disc_popc, dim3((unsigned)(words / 256 + 1)), dim3(256), 0, s, mask, words, cnt);
    SBX_TRY(exclusive_scan_u32(cnt, words + 1, A.ptr<uint32_t>(o_tmp), s));
    SBX_HIP(hipMemcpyAsync(&nd32, cnt + words, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    SBX_HIP(hipStreamSynchronize(s));
  }
  const int64_t nd = nd32;
  D.n = nd;
  if (nd == 0) {
    set_error("no live particles of the requested disc component");
    return SBX_ESTATE;
  }
  // about 2^bits = nd / 256 buckets per octave of the radius: near the peak of
  // a disc they hold some 200 particles; the top octave holds the far corner
  // of the grid
  int bits = 4;
  while (bits < 15 && (nd >> (bits + 8)) > 0) ++bits;
  const double span = c->hh[galaxy].lv[c->hh[galaxy].n_levels - 1].R;
  const int top = std::min(1023 + 1000, std::max(24, 1023 + std::ilogb(span) + 3));
  const Buckets bk{(top - 24) << 20, 20 - bits, 24 << bits};
  const int nb = rs_blocks(nd);
  const size_t ncnt = (size_t)256 * nb;
  const size_t o_fill = A.take(4 * ((size_t)bk.count + 1)), o_ftmp = A.take(4 * scan_tmp_elems(bk.count + 1));
  const size_t o_flag = A.take(4), o_rec = A.take(sizeof(DiscRec<T>) * nd);
  const size_t o_key = A.take(16 * nd);  // bucketed keys; the radix sort's second buffers and counts
  const size_t o_skey = A.take(8 * nd), o_ord = A.take(4 * nd);
  const size_t o_rcnt = A.take(4 * ncnt), o_rtmp = A.take(4 * scan_tmp_elems(ncnt));
  const size_t o_part = A.take(sizeof(double) * 4 * kBulkBlocks), o_bulk = A.take(sizeof(double) * 4);
  const size_t o_extra = A.take(extra);
  const bool grow = c->an_work_bytes < A.at;
  SBX_TRY(A.reserve());
  if (grow) return disc_prepare<T>(c, comp, galaxy, extra, D);  // a new buffer: select again
  uint32_t* fill = A.ptr<uint32_t>(o_fill);
  D.rec = A.ptr<DiscRec<T>>(o_rec);
  D.key = A.ptr<uint64_t>(o_skey);
  D.order = A.ptr<uint32_t>(o_ord);
  D.key2 = A.ptr<uint64_t>(o_key);
  D.order2 = (uint32_t*)(D.key2 + nd);
  D.cnt = A.ptr<uint32_t>(o_rcnt);
  D.ctmp = A.ptr<uint32_t>(o_rtmp);
  D.bulk = A.ptr<double>(o_bulk);
  D.flag = A.ptr<uint32_t>(o_flag);
  D.extra = A.ptr<void>(o_extra);
  double* part = A.ptr<double>(o_part);
  // counts and flag cleared together (they are neighbours)
  SBX_TRY(launch_zero<uint32_t>(fill, (o_flag - o_fill) / 4 + 1, s));
  hipLaunchKernelGGL((k_disc_compact<T>), dim3(4096), dim3(256), 0, s, p, comp, galaxy,
                     A.ptr<uint32_t>(o_mask), A.ptr<uint32_t>(o_cnt), D.cen, bk, fill, D.rec);
  SBX_TRY(exclusive_scan_u32(fill, (size_t)bk.count + 1, A.ptr<uint32_t>(o_ftmp), s));
  hipLaunchKernelGGL((k_disc_keys<T>), dim3(kBulkBlocks), dim3(256), 0, s, D.rec, nd, D.cen, bk, fill,
                     A.ptr<RadKey>(o_key), part);
  hipLaunchKernelGGL(k_columns, dim3(4), dim3(256), 0, s, part, kBulkBlocks, 4, D.bulk);
  hipLaunchKernelGGL(k_disc_order, dim3(4096), dim3(256), 0, s, A.ptr<RadKey>(o_key), fill, bk.count, D.key,
                     D.order, D.flag);
  SBX_HIP(hipGetLastError());
  return SBX_OK;
}

// The radial order by a stable radix sort of the whole disc (radii too
// crowded for the buckets).
template <typename T>
sbx_status disc_radix(sbx_ctx* c, const Disc<T>& D) {
  hipStream_t s = c->stream;
  const int nb = rs_blocks(D.n);
  hipLaunchKernelGGL((k_disc_radii<T>), dim3(1024), dim3(256), 0, s, D.rec, D.n, D.cen, D.key, D.order);
  uint64_t *ka = D.key, *kb = D.key2;
  uint32_t *va = D.order, *vb = D.order2;
  for (int shift = 0; shift < 64; shift += 8) {  // eight passes: the result is back in the first buffers
    hipLaunchKernelGGL(k_rs_hist, dim3(nb), dim3(64), 0, s, ka, D.n, shift, nb, D.cnt);
    SBX_TRY(exclusive_scan_u32(D.cnt, (size_t)256 * nb, D.ctmp, s));
    hipLaunchKernelGGL(k_rs_scatter, dim3(nb), dim3(64), 0, s, ka, va, D.n, shift, nb, D.cnt, kb, vb);
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  SBX_TRY(launch_zero<uint32_t>(D.flag, 1, s));  // the order stands
  SBX_HIP(hipGetLastError());
  return SBX_OK;
}

// Run `use(buf)`, which queues the passes that need the radial order and
// leaves `count` doubles at buf, and copy them to out; if the buckets
// overflowed, once more on the radix sort's order.
template <typename T, typename Fn>
sbx_status with_order(sbx_ctx* c, const Disc<T>& D, double* buf, size_t count, double* out, Fn&& use) {
  for (int attempt = 0; attempt < 2; ++attempt) {
    SBX_TRY(use());
    uint32_t flag = 0;
    SBX_HIP(hipMemcpyAsync(out, buf, sizeof(double) * count, hipMemcpyDeviceToHost, c->stream));
    if (attempt == 0) SBX_HIP(hipMemcpyAsync(&flag, D.flag, sizeof(flag), hipMemcpyDeviceToHost, c->stream));
    SBX_HIP(hipStreamSynchronize(c->stream));
    if (!flag) break;
    SBX_TRY(disc_radix<T>(c, D));
  }
  return SBX_OK;
}

template <typename T>
sbx_status disc_t(sbx_ctx* c, const sbx_disc_query* qy, sbx_disc_result* res, double* bin_r,
                  double* bin_vc, double* bin_rms_z, double* rho_z) {
  hipStream_t s = c->stream;
  Disc<T> D;
  const int nbins = qy->n_bins, nz = qy->n_z;
  const int split = std::max(1, std::min(32, 2048 / nbins));
  // results [annulus and heat 8][bulk 4][profile nz][bin r, vc, rms z], then partials
  const size_t nres = kAnVals + 4 + nz + 3 * (size_t)nbins;
  const size_t npart = 3 * (size_t)nbins * split + (size_t)kAnBlocks * (kAnVals + nz);
  auto body = [&]() -> sbx_status {
    SBX_TRY(disc_prepare<T>(c, qy->comp, qy->galaxy, sizeof(double) * (nres + npart), D));
    const int64_t nd = D.n;
    res->n_disc = nd;
    double* asum = (double*)D.extra;
    double *bsum = asum + kAnVals, *zsum = bsum + 4;
    double *br = zsum + nz, *bv = br + nbins, *bz = bv + nbins;
    double *bpart = bz + nbins, *apart = bpart + 3 * (size_t)nbins * split;
    double* zpart = apart + (size_t)kAnBlocks * kAnVals;
    std::vector<double> h(nres);
    const size_t shb = sizeof(double) * (2 * (size_t)nbins + nz);
    SBX_TRY(with_order<T>(c, D, asum, nres, h.data(), [&]() -> sbx_status {
      SBX_HIP(hipMemcpyAsync(bsum, D.bulk, sizeof(double) * 4, hipMemcpyDeviceToDevice, s));
      hipLaunchKernelGGL((k_disc_bins<T>), dim3(nbins, split), dim3(256), 0, s, D.order, nd, nbins, D.rec,
                         D.cen, D.bulk, D.flag, bpart);
      hipLaunchKernelGGL(k_disc_bins_end, dim3((nbins + 255) / 256), dim3(256), 0, s, bpart, split, nd, nbins,
                         br, bv, bz);
      hipLaunchKernelGGL((k_disc_heat<T>), dim3(kAnBlocks), dim3(256), shb, s, nd, nbins, br, bv, D.rec,
                         D.cen, D.bulk, qy->annulus[0], qy->annulus[1], nz, qy->z_max, apart, zpart);
      hipLaunchKernelGGL(k_columns, dim3(kAnVals), dim3(256), 0, s, apart, kAnBlocks, kAnVals, asum);
      hipLaunchKernelGGL(k_columns, dim3(nz), dim3(256), 0, s, zpart, kAnBlocks, nz, zsum);
      SBX_HIP(hipGetLastError());
      return SBX_OK;
    }));
    const double *a = h.data(), *b4 = a + kAnVals, *z = b4 + 4, *hb = z + nz;
    if (bin_r) std::copy(hb, hb + nbins, bin_r);
    if (bin_vc) std::copy(hb + nbins, hb + 2 * nbins, bin_vc);
    if (bin_rms_z) std::copy(hb + 2 * nbins, hb + 3 * nbins, bin_rms_z);
    res->e_heat = a[0];
    res->n_annulus = (int64_t)llround(a[1]);
    auto sd = [&](double s1, double s2) {
      if (a[1] <= 0) return 0.0;
      const double mu = s1 / a[1];
      return sqrt(std::max(s2 / a[1] - mu * mu, 0.0));
    };
    res->sig_R = sd(a[2], a[3]);
    res->sig_phi = sd(a[4], a[5]);
    res->sig_z = sd(a[6], a[7]);
    res->sig_tot2 = res->sig_R * res->sig_R + res->sig_phi * res->sig_phi + res->sig_z * res->sig_z;
    for (int k = 0; k < 3; ++k) res->bulk_v[k] = b4[1 + k] / b4[0];
    const double lo = qy->annulus[0], hi = qy->annulus[1];
    const double area = M_PI * (hi * hi - lo * lo), dz = 2.0 * qy->z_max / nz;
    if (rho_z)
      for (int k = 0; k < nz; ++k) rho_z[k] = z[k] / (area * dz);
    return SBX_OK;
  };
  const sbx_status rc = body();
  (void)hipStreamSynchronize(s);
  return rc;
}

// ------------------------------------------------------------ disc modes --
// first sorted position with R >= r (sorted radius keys)
__device__ __forceinline__ int64_t lower_bound_r(const uint64_t* key, int64_t n, double r) {
  const uint64_t kr = (uint64_t)__double_as_longlong(r);
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (key[mid] < kr) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Annular bin [k dR, (k+1) dR) split over gridDim.y blocks: sums over its
// particles of M cos(m phi) and -M sin(m phi), m = 0..MM, in a fixed order.
// The factors e^{i m phi} are products of e^{i phi} = (x + i y) / R, each of
// at most log2(m) + 1 factors, so that their rounding stays that of the
// angle itself; radii whose square leaves the normal range take the angle.
// One block a bin and a sincos per m took 884 us for 2M particles, 64 bins
// and m up to 4 (now 60 us).
template <typename T, int MM>
__global__ void __launch_bounds__(256)
    k_disc_modes(const uint64_t* __restrict__ key, const uint32_t* __restrict__ order, int64_t n,
                 const DiscRec<T>* __restrict__ rec, Centre cen, double dR, const uint32_t* __restrict__ flag,
                 double* __restrict__ part) {
  if (*flag) return;  // no order yet
  const int k = blockIdx.x;
  const int64_t s0 = lower_bound_r(key, n, k * dR), s1 = lower_bound_r(key, n, (k + 1) * dR);
  const double cx = cen.at(0), cy = cen.at(1);
  double a[2 * (MM + 1)] = {};
  for (int64_t j = s0 + (int64_t)blockIdx.y * 256 + threadIdx.x; j < s1; j += (int64_t)gridDim.y * 256) {
    const DiscRec<T> r = load_rec(rec, order[j]);
    const double dx = (double)r.v[0] - cx, dy = (double)r.v[1] - cy;
    const double m = (double)r.v[6];
    double re[MM + 1], im[MM + 1];
    re[0] = 1.0;
    im[0] = 0.0;
    if constexpr (MM > 0) {
      const double R = __longlong_as_double((long long)key[j]);
      if (R > 1e-140 && R < 1e140) {
        re[1] = dx / R;
        im[1] = dy / R;
      } else {
        sincos(atan2(dy, dx), &im[1], &re[1]);
      }
#pragma unroll
      for (int q = 2; q <= MM; ++q) {
        const int h = q / 2, g = q - h;
        re[q] = re[h] * re[g] - im[h] * im[g];
        im[q] = re[h] * im[g] + im[h] * re[g];
      }
    }
#pragma unroll
    for (int q = 0; q <= MM; ++q) {
      a[2 * q] += m * re[q];
      a[2 * q + 1] -= m * im[q];
    }
  }
  block_rows<2 * (MM + 1)>(a, part + ((size_t)k * gridDim.y + blockIdx.y) * 2 * (MM + 1));
}

// The blocks' sums of each bin added in order and divided by the bin area:
// out[(k * (mmax + 1) + m) * 2 + {0, 1}] = re, im.
__global__ void __launch_bounds__(256)
    k_disc_modes_end(const double* __restrict__ part, int split, int width, int mmax, int nr, double dR,
                     double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int w = 2 * (mmax + 1);
  if (i >= (int64_t)nr * w) return;
  const int k = (int)(i / w), q = (int)(i - (int64_t)k * w);
  double s = 0.0;
#pragma unroll 8
  for (int b = 0; b < split; ++b) s += part[((size_t)k * split + b) * width + q];
  const double S = M_PI * dR * dR * ((double)(k + 1) * (k + 1) - (double)k * k);
  out[i] = s / S;
}

template <typename T>
sbx_status modes_t(sbx_ctx* c, int comp, int galaxy, int nr, double rmax, int mmax, double* coeff) {
  hipStream_t s = c->stream;
  Disc<T> D;
  const int split = std::max(1, std::min(64, 4096 / nr));
  // sums for the least of 0, 2, 4, 8, 16 that covers mmax
  const int MM = mmax == 0 ? 0 : mmax <= 2 ? 2 : mmax <= 4 ? 4 : mmax <= 8 ? 8 : 16;
  const size_t width = 2 * (MM + 1), cnt = (size_t)nr * (mmax + 1) * 2;
  auto body = [&]() -> sbx_status {
    SBX_TRY(disc_prepare<T>(c, comp, galaxy, sizeof(double) * (cnt + (size_t)nr * split * width), D));
    double* out = (double*)D.extra;
    double* part = out + cnt;
    const double dR = rmax / nr;
    return with_order<T>(c, D, out, cnt, coeff, [&]() -> sbx_status {
      const dim3 g(nr, split), b(256);
      auto go = [&](auto mc) {
        hipLaunchKernelGGL((k_disc_modes<T, decltype(mc)::value>), g, b, 0, s, D.key, D.order, D.n, D.rec, D.cen,
                           dR, D.flag, part);
      };
      switch (MM) {
        case 0: go(std::integral_constant<int, 0>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        case 8: go(std::integral_constant<int, 8>()); break;
        default: go(std::integral_constant<int, 16>());
      }
      hipLaunchKernelGGL(k_disc_modes_end, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, part, split,
                         (int)width, mmax, nr, dR, out);
      SBX_HIP(hipGetLastError());
      return SBX_OK;
    });
  };
  const sbx_status rc = body();
  (void)hipStreamSynchronize(s);
  return rc;
}

}  // namespace

extern "C" {

sbx_status sbx_disc_analysis(sbx_ctx* c, const sbx_disc_query* q, sbx_disc_result* res,
                             double* bin_r, double* bin_vc, double* bin_rms_z, double* rho_z) {
  if (!c || !q || !res) {
    set_error("null argument");
    return SBX_EINVAL;
  }
  if (c->batch && c->batch->pending) {
    set_error("the context's batch has queued work: call sbx_batch_sync first");
    return SBX_ESTATE;
  }
  if (!c->built || c->n == 0) {
    set_error("build_grids and load_particles first");
    return SBX_ESTATE;
  }
  if (q->n_bins < 1 || q->n_bins > kMaxBins || q->n_z < 1 || q->n_z > kMaxZ ||
      !(q->z_max > 0.0) || !(q->annulus[1] > q->annulus[0]) || !(q->annulus[0] >= 0.0) ||
      q->comp < 0 || q->comp >= kNComp || q->galaxy < 0 || q->galaxy >= c->ngal) {
    set_error("bad disc query (1 <= n_bins <= 2048, 1 <= n_z <= 1024, z_max > 0, "
              "0 <= R_lo < R_hi, component and galaxy in range)");
    return SBX_EINVAL;
  }
  SBX_TRY(set_device(c->cfg.device));
  std::memset(res, 0, sizeof(*res));
  return c->cfg.prec == SBX_FP64 ? disc_t<double>(c, q, res, bin_r, bin_vc, bin_rms_z, rho_z)
                                 : disc_t<float>(c, q, res, bin_r, bin_vc, bin_rms_z, rho_z);
}

sbx_status sbx_disc_modes(sbx_ctx* c, int32_t comp, int32_t galaxy, int32_t n_rbins, double r_max,
                          int32_t m_max, double* coeff) {
  if (!c || !coeff) {
    set_error("null argument");
    return SBX_EINVAL;
  }
  if (c->batch && c->batch->pending) {
    set_error("the context's batch has queued work: call sbx_batch_sync first");
    return SBX_ESTATE;
  }
  if (!c->built || c->n == 0) {
    set_error("build_grids and load_particles first");
    return SBX_ESTATE;
  }
  if (n_rbins < 1 || n_rbins > 65536 || !(r_max > 0.0) || m_max < 0 || m_max > 16 || comp < 0 ||
      comp >= kNComp || galaxy < 0 || galaxy >= c->ngal) {
    set_error("bad mode query (1 <= n_rbins <= 65536, r_max > 0, 0 <= m_max <= 16)");
    return SBX_EINVAL;
  }
  SBX_TRY(set_device(c->cfg.device));
  return c->cfg.prec == SBX_FP64 ? modes_t<double>(c, comp, galaxy, n_rbins, r_max, m_max, coeff)
                                 : modes_t<float>(c, comp, galaxy, n_rbins, r_max, m_max, coeff);
}

}  // extern "C"
