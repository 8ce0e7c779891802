// sph_kernels.hip -- gfx950 kernels of the SPH hydrodynamics step.
//
//   keys + sort + permute ....... Sect. 3.1 (space-filling curve, sort)
//   tree + groups ............... Sect. 3.1 (chopping the curve)
//   group tree walk ............. Sect. 3.2 (breadth-first, one wave per group)
//   density + h iteration ....... Sect. 2.2 and Sect. 3.2.1
//   hydro force ................. Sect. 2.4 (eq:acc, eq:energy), 2.5, 2.6
//   leapfrog + Courant step ..... Sect. 2.4 (eq:predict_pos, eq:predict_vel,
//                                 eq:correct_vel, eq:timestep), Sect. 3.3
//
// Built with -ffp-contract=off: every fused multiply-add is an explicit fma().
#include <math.h>

#include <mutex>

#include <type_traits>

#include "sph_ctx.h"

namespace sph {

#define SPH_INF (__builtin_huge_val())

// ============================================================================
// Wave / block primitives (wave64)
// ============================================================================
// v moved across lanes by a DPP control (row_shr:n = 0x110 + n, row_bcast:15
// = 0x142, row_bcast:31 = 0x143); lanes without a source, or outside the
// enabled rows, read 0.  Called with every lane of the wavefront active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum over the 64 lanes: Hillis-Steele within each row of
// 16 lanes, then the row totals carried by the two row broadcasts.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  v += dpp_u32<0x111, 0xf>(v);
  v += dpp_u32<0x112, 0xf>(v);
  v += dpp_u32<0x114, 0xf>(v);
  v += dpp_u32<0x118, 0xf>(v);
  v += dpp_u32<0x142, 0xa>(v);
  v += dpp_u32<0x143, 0xc>(v);
  return v;
}

__device__ __forceinline__ double wave_max_f64(double v) { return seg_max<kWave>(v); }
__device__ __forceinline__ double wave_min_f64(double v) { return seg_min<kWave>(v); }

__device__ __forceinline__ uint32_t block256_excl_scan(uint32_t v, uint32_t* lds,
                                                       uint32_t* total) {
  const uint32_t inc = wave_incl_scan_u32(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 63) lds[w] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t s = lds[k];
    off += (k < w) ? s : 0u;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

// ============================================================================
// Device-wide exclusive scan of uint32 (three launches).  Tiles of 2048.
// ============================================================================
__global__ __launch_bounds__(256) void k_scan_partials(const uint32_t* __restrict__ in, int64_t n,
                                                        uint32_t* __restrict__ part) {
  __shared__ uint32_t lds[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) s += (base + k < n) ? in[base + k] : 0u;
  uint32_t tot;
  block256_excl_scan(s, lds, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// One block of 1024 threads scans nb partials in chunks; writes the total.
__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* __restrict__ part, int nb,
                                                    uint32_t* __restrict__ total_out) {
  __shared__ uint32_t lds[16];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int base = 0; base < nb; base += 1024) {
    const int i = base + threadIdx.x;
    const uint32_t v = (i < nb) ? part[i] : 0u;
    const uint32_t inc = wave_incl_scan_u32(v);
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int k = 0; k < 16; ++k) {
      uint32_t s = lds[k];
      off += (k < w) ? s : 0u;
      tot += s;
    }
    const uint32_t c0 = carry;
    if (i < nb) part[i] = c0 + off + inc - v;
    __syncthreads();
    if (threadIdx.x == 0) carry = c0 + tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total_out = carry;
}

__global__ __launch_bounds__(256) void k_scan_apply(const uint32_t* in, uint32_t* out, int64_t n,
                                                     const uint32_t* __restrict__ part) {
  __shared__ uint32_t lds[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
  uint32_t v[8];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0u;
    s += v[k];
  }
  uint32_t tot;
  uint32_t off = block256_excl_scan(s, lds, &tot) + part[blockIdx.x];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (base + k < n) out[base + k] = off;
    off += v[k];
  }
}

// Exclusive scan of up to kScanSingleMax uint32 (n a multiple of 4, data
// 16-byte aligned) by one block of 1024 threads in one launch: every thread
// owns a contiguous run of at most 16 uint4, loaded all at once.
constexpr int kScanSingleMax = 1024 * 64;

__global__ __launch_bounds__(1024) void k_scan_single(uint32_t* __restrict__ data, int n,
                                                       uint32_t* __restrict__ total_out) {
  __shared__ uint32_t lds[16];
  const int t = threadIdx.x;
  const int q = (n + 4095) / 4096;  // uint4 per thread, <= 16
  const int nq = n >> 2;
  uint4* d4 = reinterpret_cast<uint4*>(data);
  uint4 v[16];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int idx = t * q + k;
    v[k] = (k < q && idx < nq) ? d4[idx] : make_uint4(0u, 0u, 0u, 0u);
    s += v[k].x + v[k].y + v[k].z + v[k].w;
  }
  const uint32_t inc = wave_incl_scan_u32(s);
  const int w = t >> 6, lane = t & 63;
  if (lane == 63) lds[w] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const uint32_t x = lds[k];
    off += (k < w) ? x : 0u;
    tot += x;
  }
  off += inc - s;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int idx = t * q + k;
    if (k < q && idx < nq) {
      uint4 o;
      o.x = off;
      off += v[k].x;
      o.y = off;
      off += v[k].y;
      o.z = off;
      off += v[k].z;
      o.w = off;
      off += v[k].w;
      d4[idx] = o;
    }
  }
  if (t == 0) *total_out = tot;
}

static hipError_t scan_u32(sph_ctx* c, uint32_t* data, int64_t n, uint32_t* total) {
  if (n > 0 && n <= kScanSingleMax && (n & 3) == 0 && (reinterpret_cast<uintptr_t>(data) & 15) == 0) {
    hipLaunchKernelGGL(k_scan_single, dim3(1), dim3(1024), 0, c->stream, data, (int)n, total);
    return hipGetLastError();
  }
  const int nb = (int)((n + kScanTile - 1) / kScanTile);
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scan_partials, dim3(nb), dim3(256), 0, c->stream, data, n, c->scan_part);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, c->stream, c->scan_part, nb, total);
  hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(256), 0, c->stream, data, data, n,
                     c->scan_part);
  return hipGetLastError();
}

// ============================================================================
// Predict (optional) + Morton keys
// ============================================================================
__device__ __forceinline__ uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

// (x - lo) * scale, floored and clamped to [0, 2^21 - 1]; NaN -> 0.
__device__ __forceinline__ uint64_t quantise(double x, double lo, double scale) {
  double q = (x - lo) * scale;
  if (!(q >= 0.0)) return 0ull;
  q = floor(q);
  return (q > 2097151.0) ? 2097151ull : (uint64_t)q;
}

__device__ __forceinline__ double wrap_coord(double v, double lo, double len, int periodic) {
  if (periodic) {
    if (v >= lo + len)
      v -= len;
    else if (v < lo)
      v += len;
  }
  return v;
}

// Prediction of particle i (optional) and its key.
__device__ __forceinline__ uint64_t predict_key(const KParams& kp, const Parts& p, bool predict,
                                                double dt, int i, bool& bad) {
  double x = p.x[i], y = p.y[i], z = p.z[i];
  if (predict) {
    const double hdt2 = 0.5 * dt * dt;
    const double vx = p.vx[i], vy = p.vy[i], vz = p.vz[i];
    const double ax = p.ax[i], ay = p.ay[i], az = p.az[i];
    x = wrap_coord(x + (vx * dt + hdt2 * ax), kp.lo[0], kp.len[0], kp.periodic[0]);
    y = wrap_coord(y + (vy * dt + hdt2 * ay), kp.lo[1], kp.len[1], kp.periodic[1]);
    z = wrap_coord(z + (vz * dt + hdt2 * az), kp.lo[2], kp.len[2], kp.periodic[2]);
    p.x[i] = x;
    p.y[i] = y;
    p.z[i] = z;
    p.vx[i] = vx + ax * dt;
    p.vy[i] = vy + ay * dt;
    p.vz[i] = vz + az * dt;
    p.u[i] = p.u[i] + p.dudt[i] * dt;
  }
  bad |= !(isfinite(x) && isfinite(y) && isfinite(z));
  const uint64_t ix = quantise(x, kp.lo[0], kp.key_scale);
  const uint64_t iy = quantise(y, kp.lo[1], kp.key_scale);
  const uint64_t iz = quantise(z, kp.lo[2], kp.key_scale);
  return (spread3(ix) << 2) | (spread3(iy) << 1) | spread3(iz);
}

// Words of the radix sort besides the look-back status and the histograms.
struct SortHead {
  uint32_t tickets[8];     // next tile of every pass
  uint32_t ticket;         // next item of k_resort
  uint32_t done[10];       // items finished in every stage of k_resort
  uint32_t items;          // items of every stage of k_resort but the first
  uint32_t shift;          // lowest key bit the passes sort
  uint32_t resort;         // 1: a long run of equal sorted bits is out of order
  uint32_t runs;           // long runs listed
  uint32_t over;           // runs listed that are too long for one block
};

__device__ __forceinline__ uint64_t wave_or_u64(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor((unsigned long long)v, o);
  return v;
}

// Block 0 also clears the radix sort's digit histograms and tile tickets
// (the sort follows at once); every block leaves the key bits that are set in
// one of its keys and those that are clear in one (range[0], range[1]).
__global__ __launch_bounds__(256) void k_predict_keys(KParams kp, Parts p, int predict,
                                                       const DevState* __restrict__ ds,
                                                       uint64_t* __restrict__ keys,
                                                       uint32_t* __restrict__ vals,
                                                       uint32_t* __restrict__ ghist,
                                                       SortHead* __restrict__ head,
                                                       uint64_t* __restrict__ range,
                                                       uint32_t* __restrict__ err) {
  __shared__ uint64_t wr[4][2];
  if (blockIdx.x == 0) {
    for (int k = threadIdx.x; k < 8 * 256; k += blockDim.x) ghist[k] = 0u;
    uint32_t* hw = reinterpret_cast<uint32_t*>(head);
    if (threadIdx.x < sizeof(SortHead) / 4) hw[threadIdx.x] = 0u;
  }
  const int n = kp.n;
  const double dt = predict ? ds->dt_cur : 0.0;
  bool bad = false;
  uint64_t ones = 0ull, zeros = 0ull;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint64_t key = predict_key(kp, p, predict != 0, dt, i, bad);
    ones |= key;
    zeros |= ~key;
    keys[i] = key;
    vals[i] = (uint32_t)i;
  }
  if (bad) atomicOr(err, kErrNonFinite);
  ones = wave_or_u64(ones);
  zeros = wave_or_u64(zeros);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    wr[w][0] = ones;
    wr[w][1] = zeros;
  }
  __syncthreads();
  if (threadIdx.x < 2)
    range[2 * blockIdx.x + threadIdx.x] =
        wr[0][threadIdx.x] | wr[1][threadIdx.x] | wr[2][threadIdx.x] | wr[3][threadIdx.x];
}

// ============================================================================
// LSD radix sort of (key, index), 8 bits per pass, stable.
// ============================================================================
// Lanes (among `active`) whose 8-bit digit equals this lane's.
__device__ __forceinline__ uint64_t match_digit8(uint32_t d, uint64_t active) {
  uint64_t m = active;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bal = ballot64(bit);
    m &= bit ? bal : ~bal;
  }
  return m;
}

// Wave-aggregated increment of an LDS digit counter: when every active lane
// of the wavefront holds the same digit (the high digits of a curve-ordered
// tile) one lane adds the whole count.
__device__ __forceinline__ void lds_count_digit(uint32_t* cnt, uint32_t d, bool valid) {
  const uint64_t act = ballot64(valid);
  if (act == 0ull) return;
  const int lead = __builtin_ctzll(act);
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, lead);  // lead is uniform
  const uint64_t same = ballot64(valid && d == d0);
  if (same == act) {
    if (lane_id() == lead) atomicAdd(&cnt[d0], (uint32_t)popc64(act));
  } else if (valid) {
    atomicAdd(&cnt[d], 1u);
  }
}

// One-sweep radix sort of the keys' leading bits.  k_radix_prep counts the
// digits of all passes in one read of the keys (global histograms) and clears
// the look-back status of every pass; k_radix_pass then sorts one 8-bit digit
// per launch: each block takes the next tile (an atomic ticket, so every
// earlier tile belongs to a block that already runs), publishes its digit
// counts, and looks back over the earlier tiles' published counts or
// inclusive prefixes for its exclusive prefix (decoupled look-back), then
// scatters stably.  Status words: flag in the top two bits (1 count only, 2
// inclusive prefix), the count in the low 30 (n < 2^30).  A word carries
// nothing but itself, so relaxed device-scope atomics suffice (no
// acquire/release cache maintenance).
//
// A 63-bit key of n particles needs about log2 n bits to tell most particles
// apart, so the passes sort only the top bits from the highest one that
// varies (launch_sort chooses their number); k_sort_fix then orders the short
// runs that agree in all of them, and k_resort the longer ones.  What each pass
// costs is latency (tile count, look-back) at small n, and its 24 bytes per
// particle at large n: 8.3 us at 32^3, 13.3 at 294,912, 205 at 16.8M particles.
constexpr uint32_t kStAgg = 1u << 30, kStPre = 2u << 30, kStMask = (1u << 30) - 1u;
constexpr int kLookbackSpin = 1 << 22;  // bounded wait; the predecessors always publish
constexpr int kLookW = 16;               // earlier tiles read per look-back round

// Sorted bits start here: 8 npass bits up to the highest one that varies.
__device__ __forceinline__ uint32_t sort_shift(uint64_t varying, int npass) {
  const int top = varying ? 64 - __clzll((long long)varying) : 0;
  return (uint32_t)max(0, top - 8 * npass);
}

__device__ __forceinline__ void count_digits(const uint64_t* __restrict__ keys, int n, int base,
                                             uint32_t shift, int npass, uint32_t (*h)[256]) {
#pragma unroll
  for (int k = 0; k < kSortTile / 256; ++k) {
    const int i = base + k * 256 + threadIdx.x;
    const bool valid = i < n;
    const uint64_t key = valid ? keys[i] >> shift : 0ull;
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p < npass) lds_count_digit(h[p], (uint32_t)((key >> (8 * p)) & 255ull), valid);
  }
}

__global__ __launch_bounds__(256) void k_radix_prep(const uint64_t* __restrict__ keys, int n,
                                                     int nblk, int npass, int nrange,
                                                     const uint64_t* __restrict__ range,
                                                     uint32_t* __restrict__ status,
                                                     uint32_t* __restrict__ ghist,
                                                     SortHead* __restrict__ head) {
  __shared__ uint32_t h[8][256];
  __shared__ uint64_t wr[4][2];
  const int tid = threadIdx.x;
  uint64_t ones = 0ull, zeros = 0ull;
  for (int k = tid; k < nrange; k += 256) {
    ones |= range[2 * k];
    zeros |= range[2 * k + 1];
  }
#pragma unroll
  for (int p = 0; p < 8; ++p) h[p][tid] = 0u;
  ones = wave_or_u64(ones);
  zeros = wave_or_u64(zeros);
  if ((tid & 63) == 0) {
    wr[tid >> 6][0] = ones;
    wr[tid >> 6][1] = zeros;
  }
  __syncthreads();
  const uint32_t shift =
      sort_shift((wr[0][0] | wr[1][0] | wr[2][0] | wr[3][0]) &
                     (wr[0][1] | wr[1][1] | wr[2][1] | wr[3][1]),
                 npass);
  if (blockIdx.x == 0 && tid == 0) head->shift = shift;
  for (int t = blockIdx.x; t < nblk; t += gridDim.x) {
    for (int p = 0; p < npass; ++p) status[((int64_t)p * nblk + t) * 256 + tid] = 0u;
    count_digits(keys, n, t * kSortTile, shift, npass, h);
  }
  __syncthreads();
  for (int p = 0; p < npass; ++p)
    if (h[p][tid]) atomicAdd(&ghist[p * 256 + tid], h[p][tid]);
}

struct SortLds {
  // wc[d * NS + s]: keys of digit d in set s, then the tile's keys of digit d
  // before set s (at most kSortTile: 16 bits suffice);
  // the digit counts (16 KB), then the tile in digit order (24 KB)
  alignas(16) unsigned char buf[kSortTile * 12];
  uint32_t run[256];
  uint32_t lst[256];
  uint32_t lds4[4];
  int tile;
};

// Loads and stores of data that passes between blocks within one launch
// (AGENT): past the L2s, each of which belongs to one XCD.
template <bool AGENT, typename T>
__device__ __forceinline__ T tile_load(const T* p) {
  if constexpr (AGENT) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool AGENT, typename T>
__device__ __forceinline__ void tile_store(T* p, T v) {
  if constexpr (AGENT)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

// One tile of one pass: digits (key >> shift) & 255; st: the pass's status
// words, gh: this thread's digit of the pass's histogram.
template <bool AGENT>
__device__ __forceinline__ void radix_tile(SortLds& L, const uint64_t* __restrict__ kin,
                                           const uint32_t* __restrict__ vin,
                                           uint64_t* __restrict__ kout,
                                           uint32_t* __restrict__ vout, int n, uint32_t shift,
                                           int tile, uint32_t* __restrict__ st, uint32_t gh,
                                           uint32_t* __restrict__ err) {
  constexpr int PER = kSortTile / 256;
  constexpr int NS = PER * 4;  // (key slice, wavefront) sets of 64 keys, in key order
  static_assert(256 * NS * 2 <= kSortTile * 12, "digit counts fit the tile buffer");
  static_assert(kSortTile <= 65535, "16-bit tile offsets");
  uint16_t* wc = reinterpret_cast<uint16_t*>(L.buf);
  uint64_t* s_key = reinterpret_cast<uint64_t*>(L.buf);
  uint32_t* s_val = reinterpret_cast<uint32_t*>(L.buf + kSortTile * 8);
  const int tid = threadIdx.x, w = tid >> 6;
  const int base = tile * kSortTile;
  uint64_t key[PER];
  uint32_t val[PER], rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = base + k * 256 + tid;
    key[k] = i < n ? tile_load<AGENT>(kin + i) : 0ull;
    val[k] = i < n ? tile_load<AGENT>(vin + i) : 0u;
  }
  // rank of each key among the equal digits of its set (wave ballots), and
  // the count of every digit in every set
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const bool valid = base + k * 256 + tid < n;
    const uint32_t d = (uint32_t)((key[k] >> shift) & 255ull);
    const uint64_t m = match_digit8(d, ballot64(valid));
    rank[k] = (uint32_t)popc64(m & lanemask_lt());
    if (valid && rank[k] == 0) wc[d * NS + k * 4 + w] = (uint16_t)popc64(m);
  }
  __syncthreads();
  // thread d: exclusive offsets of digit d over the sets, and the tile's count
  uint32_t mine = 0u;
  {
    uint16_t c[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) c[q] = wc[tid * NS + q];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const uint32_t v = c[q];
      c[q] = (uint16_t)mine;
      mine += v;
    }
#pragma unroll
    for (int q = 0; q < NS; ++q) wc[tid * NS + q] = c[q];
  }
  // publish this tile's counts; scan the global digit counts while earlier
  // tiles publish theirs; then the exclusive prefix over earlier tiles
  __hip_atomic_store(&st[(int64_t)tile * 256 + tid], (tile == 0 ? kStPre : kStAgg) | mine,
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // start of every digit: keys with a smaller digit anywhere
  uint32_t all;
  const uint32_t gofs = block256_excl_scan(gh, L.lds4, &all);
  uint32_t excl = 0u;
  if (tile > 0) {
    // a window of kLookW earlier tiles per round: their loads are in flight
    // together, so a long chain of published counts costs one latency per
    // window rather than one per tile
    int t = tile - 1, spins = 0;
    while (t >= 0) {
      uint32_t v[kLookW];
#pragma unroll
      for (int q = 0; q < kLookW; ++q)
        v[q] = (t - q >= 0) ? __hip_atomic_load(&st[(int64_t)(t - q) * 256 + tid], __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT)
                            : kStPre;  // before tile 0: prefix 0
      int used = 0;
      bool done = false;
#pragma unroll
      for (int q = 0; q < kLookW; ++q) {
        if (done || used < q) continue;  // stopped at an earlier entry
        const uint32_t f = v[q] & ~kStMask;
        if (f == 0u) continue;  // not published yet: poll again from here
        excl += v[q] & kStMask;
        used = q + 1;
        done = f == kStPre;
      }
      if (done) break;
      t -= used;
      if (used == 0 && ++spins > kLookbackSpin) {
        atomicOr(err, kErrSort);
        break;
      }
    }
    __hip_atomic_store(&st[(int64_t)tile * 256 + tid], kStPre | (excl + mine), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  // the tile's keys in digit order in LDS first, so that each digit's run is
  // stored by consecutive lanes to consecutive addresses
  uint32_t tot2;
  const uint32_t ls = block256_excl_scan(mine, L.lds4, &tot2);  // tile-local start of digit tid
  L.lst[tid] = ls;
  L.run[tid] = gofs + excl - ls;  // global position of local position 0, for digit tid
  __syncthreads();
  uint32_t lp[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t d = (uint32_t)((key[k] >> shift) & 255ull);
    lp[k] = L.lst[d] + (uint32_t)wc[d * NS + k * 4 + w] + rank[k];
  }
  __syncthreads();  // the counts are overwritten by the sorted tile
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (base + k * 256 + tid < n) {
      s_key[lp[k]] = key[k];
      s_val[lp[k]] = val[k];
    }
  }
  __syncthreads();
  const int cnt = min(kSortTile, n - base);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int q = k * 256 + tid;
    if (q < cnt) {
      const uint64_t kk = s_key[q];
      const uint32_t d = (uint32_t)((kk >> shift) & 255ull);
      const uint32_t pos = L.run[d] + (uint32_t)q;
      tile_store<AGENT>(kout + pos, kk);
      tile_store<AGENT>(vout + pos, s_val[q]);
    }
  }
}

__device__ __forceinline__ void clear_counts(SortLds& L) {
  uint32_t* z = reinterpret_cast<uint32_t*>(L.buf);
#pragma unroll
  for (int q = 0; q < kSortTile / 128; ++q) z[q * 256 + threadIdx.x] = 0u;
}

__global__ __launch_bounds__(256) void k_radix_pass(const uint64_t* __restrict__ kin,
                                                     const uint32_t* __restrict__ vin,
                                                     uint64_t* __restrict__ kout,
                                                     uint32_t* __restrict__ vout, int n,
                                                     int pass, int nblk,
                                                     uint32_t* __restrict__ status,
                                                     const uint32_t* __restrict__ ghist,
                                                     SortHead* __restrict__ head,
                                                     uint32_t* __restrict__ err) {
  __shared__ SortLds L;
  const uint32_t gh = ghist[pass * 256 + threadIdx.x];  // in flight from the start
  const uint32_t shift = head->shift + 8u * (uint32_t)pass;
  clear_counts(L);
  if (threadIdx.x == 0) L.tile = (int)atomicAdd(&head->tickets[pass], 1u);
  __syncthreads();
  radix_tile<false>(L, kin, vin, kout, vout, n, shift, L.tile,
                    status + (int64_t)pass * nblk * 256, gh, err);
}

// After the passes: every run of keys that agree in the sorted bits is put in
// the order of the whole keys (stably, so that the result is that of all
// passes).  A block orders the runs that start in its tile, each of at most
// kRunMax keys: every key counts the keys of its run that go before it.
// Other blocks read the keys that a block moves only for their sorted bits,
// which the moves keep.  Longer runs are listed and, if one is out of order,
// left to k_resort.  TILE: 512 keys as long as a CU gets few tiles (8.5 against
// 4.3 us with 2048 and 512 at 30,000 particles, 8.6 against 6.0 at 10^6), 2048
// beyond (10.9 against 14.2 at 4 10^6: the halos).
// Bound by one read of the keys: runs are found from one bit
// per key (followed key by key, runs of clustered particles took 20 to 100 us).
constexpr int kRunMax = 64;
constexpr int kRunBlock = 4096;  // keys of a run that one block of k_resort sorts

// Scratch of the long runs (words, less than one per particle): the listed
// runs' starts; starts, lengths and first items of those longer than
// kRunBlock; words by which k_resort's blocks wait (one per kReadyLine words);
// digit counts.
constexpr int kReady = 64, kReadyLine = 32;
struct RunWs {
  uint32_t *runs, *start, *len, *item, *ready, *hist;
  __host__ __device__ RunWs(uint32_t* w, int n) {
    const int64_t nr = n / (kRunMax + 1) + 1, no = n / (kRunBlock + 1) + 1;
    runs = w;
    start = runs + nr;
    len = start + no;
    item = len + no;
    ready = item + no;
    hist = ready + kReady * kReadyLine;  // 8 x 256 of each
  }
};

template <int TILE>
__global__ __launch_bounds__(256) void k_sort_fix(uint64_t* __restrict__ keys,
                                                   uint32_t* __restrict__ vals, int n,
                                                   RunWs ws, SortHead* __restrict__ head) {
  constexpr int H = 64;                      // halo on both sides
  static_assert(kRunMax <= H, "a run of the tile lies within its halos");
  constexpr int W = TILE + kRunMax;     // positions looked at: the tile and what
                                             // its last run can hold beyond it
  constexpr int PER = (W + 255) / 256;
  constexpr int NK = TILE + 2 * H;
  __shared__ uint64_t s_key[NK + 64];
  __shared__ uint64_t s_first[NK / 64 + 1];  // bit t: position t begins a run
  __shared__ uint32_t s_runs, s_at;
  __shared__ int s_over;  // start of a run longer than kRunBlock (a tile begins one at most)
  const uint32_t shift = head->shift;
  if (shift == 0u) return;  // sorted by all bits that vary
  const int tid = threadIdx.x;
  const int base = blockIdx.x * TILE;
  if (tid == 0) {
    s_runs = 0u;
    s_over = -1;
  }
  if (blockIdx.x == 0 && tid < kReady) ws.ready[tid * kReadyLine] = 0u;
  // position t of the block is particle base - H + t; the first particle and
  // what lies past the last one begin a run
  for (int t = tid; t < NK + 64; t += 256) {
    const int j = base - H + t;
    const bool in = j >= 0 && j < n;
    const uint64_t kk = in ? keys[j] : 0ull, prev = in && j > 0 ? keys[j - 1] : 0ull;
    s_key[t] = kk;
    const uint64_t b = ballot64(j <= 0 || j >= n || (kk >> shift) != (prev >> shift));
    if ((t & 63) == 0) s_first[t >> 6] = b;
  }
  __syncthreads();
  int to[PER];
  uint64_t key[PER];
  uint32_t val[PER];
  bool longrun = false;
  int begins = 0;  // long runs that this thread's keys begin (bit k)
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = H + k * 256 + tid, i = base - H + t;
    to[k] = -1;
    key[k] = 0ull;
    if (t >= H + W) continue;
    // the words of this wavefront's 64 positions and of their neighbours
    const uint64_t here = s_first[t >> 6], before = s_first[(t >> 6) - 1],
                   after = s_first[(t >> 6) + 1];
    if (ballot64((here & (after << 63 | here >> 1)) != ~0ull) == 0ull) continue;  // all alone
    if (i >= n) continue;
    // the run's first position a at or before t, at most 64 back or more, and
    // its end e after t, at most 64 further or more
    const int u = t & 63;
    const uint64_t lo = here & (~0ull >> (63 - u)), hi = u < 63 ? here & (~0ull << (u + 1)) : 0ull;
    const int a = lo ? t - u + 63 - __clzll((long long)lo)
                     : before ? t - u - 1 - __clzll((long long)before) : t - kRunMax;
    const int e = hi ? t - u + __builtin_ctzll(hi)
                     : after ? t - u + 64 + __builtin_ctzll(after) : t + kRunMax + 1;
    if (e - a == 1) continue;  // alone
    const uint64_t kk = s_key[t];
    if (e - a > kRunMax) {
      longrun |= e > t + 1 && s_key[t + 1] < kk;
      if (a == t && t < H + TILE) begins |= 1 << k;
      continue;
    }
    if (a < H || a >= H + TILE) continue;  // another block's
    int r = a;
    for (int j = a; j < e; j += 4) {
      uint64_t o[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = s_key[min(j + q, e - 1)];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        r += j + q < e && (o[q] < kk || (o[q] == kk && j + q < t)) ? 1 : 0;
    }
    if (r != t) {
      to[k] = base - H + r;
      key[k] = kk;
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    val[k] = 0u;
    if (to[k] >= 0) val[k] = vals[base + k * 256 + tid];
  }
  if (longrun) head->resort = 1u;
  uint32_t at = begins ? atomicAdd(&s_runs, (uint32_t)__popc(begins)) : 0u;
  __syncthreads();  // all values read, all runs counted
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (to[k] >= 0) {
      keys[to[k]] = key[k];
      vals[to[k]] = val[k];
    }
  if (s_runs == 0u) return;
  if (tid == 0) s_at = atomicAdd(&head->runs, s_runs);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (begins & (1 << k)) {
      const int i = base + k * 256 + tid;
      // (other blocks move keys only within their runs)
      const bool over = i + kRunBlock < n &&
                        (keys[i + kRunBlock] >> shift) == (s_key[H + k * 256 + tid] >> shift);
      ws.runs[s_at + at++] = over ? ~0u : (uint32_t)i;
      if (over) s_over = i;
    }
  __syncthreads();
  if (s_over < 0) return;
  // its length, and cleared digit counts
  const int start = s_over;
  const uint64_t pre = keys[start] >> shift;
  int lo = kRunBlock, hi = n - start;  // start + lo is of the run, start + hi is not
  while (hi - lo > 1) {
    const int step = (hi - lo + 255) / 256, p = lo + tid * step;
    const int c = __syncthreads_count(tid > 0 && p < hi && (keys[start + p] >> shift) == pre);
    lo += c * step;
    hi = min(lo + step, hi);
  }
  if (tid == 0) {
    s_at = atomicAdd(&head->over, 1u);
    ws.start[s_at] = (uint32_t)start;
    ws.len[s_at] = (uint32_t)hi;
  }
  __syncthreads();
  const int words = (int)(shift + 7) / 8 * 256;
  for (int q = tid; q < words; q += 256) ws.hist[(int64_t)s_at * words + q] = 0u;
}

// A run of up to kRunBlock keys that agree from bit `shift` (at most 39: three
// passes or more) on, by one block in LDS.  A key's lower bits and its place in
// the run make one number, so that no two are equal and any order of additions
// will do: the keys fall into 4096 buckets by the 12 leading bits that vary,
// and each counts those of its bucket that go before it.  If a bucket holds
// more than kRunMax, the digits are sorted one by one, the lowest first.  Bound
// by latency: k_resort on eight runs of 3750 keys takes 25 us (35 by digits).
constexpr int kRunBits = 12;
static_assert(kRunBlock == 1 << kRunBits, "a key's place in its run");

struct RunLds {
  uint64_t key[kRunBlock];
  uint32_t cnt[kRunBlock];
  uint32_t lst[256];
  uint32_t lds4[4];
  uint64_t wr[4][2];
};

__device__ __forceinline__ void sort_run(RunLds& L, uint64_t* __restrict__ keys,
                                         uint32_t* __restrict__ vals, int n, uint32_t shift,
                                         int start) {
  constexpr int PER = kRunBlock / 256;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const uint64_t pre = keys[start] >> shift;
  // the run's length: its keys are consecutive
  auto same = [&](int p) { return start + p < n && (keys[start + p] >> shift) == pre; };
  const int c16 = __syncthreads_count(same(PER * tid)) - 1;
  const int len = PER * c16 + __syncthreads_count(tid < PER && same(PER * c16 + tid));
  const int per = (len + 255) >> 8;
  // a wavefront holds consecutive keys, a lane every 64th of them
  const int p0 = w * per * 64 + lane;
  auto holds = [&](int k) { return k < per && p0 + 64 * k < len; };
  uint64_t key[PER];
  uint32_t at[PER];
  uint64_t ones = 0ull, zeros = 0ull;
#pragma unroll
  for (int k = 0; k < PER; ++k) key[k] = holds(k) ? keys[start + p0 + 64 * k] : 0ull;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (holds(k)) {
      const uint64_t low = key[k] & ((1ull << shift) - 1ull);
      ones |= low;
      zeros |= ~low;
      key[k] = low << kRunBits | (uint64_t)(p0 + 64 * k);
      L.key[p0 + 64 * k] = key[k];
    }
  ones = wave_or_u64(ones);
  zeros = wave_or_u64(zeros);
  if (lane == 0) {
    L.wr[w][0] = ones;
    L.wr[w][1] = zeros;
  }
  for (int q = tid; q < kRunBlock; q += 256) L.cnt[q] = 0u;
  __syncthreads();
  bool out = false;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    out |= holds(k) && p0 + 64 * k + 1 < len && key[k] > L.key[p0 + 64 * k + 1];
  const uint64_t varying = (L.wr[0][0] | L.wr[1][0] | L.wr[2][0] | L.wr[3][0]) &
                           (L.wr[0][1] | L.wr[1][1] | L.wr[2][1] | L.wr[3][1]);
  if (!__syncthreads_or(out)) return;
  const int top = kRunBits + 64 - __clzll((long long)varying);
  const int bit0 = max(kRunBits, top - kRunBits);
  auto bucket = [&](uint64_t v) { return (uint32_t)(v >> bit0) & (uint32_t)(kRunBlock - 1); };
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    at[k] = 0u;
    if (holds(k)) at[k] = atomicAdd(&L.cnt[bucket(key[k])], 1u);
  }
  __syncthreads();
  // first places of the buckets (16 a thread)
  uint32_t mine = 0u, all;
  bool large = false;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t c = L.cnt[PER * tid + q];
    L.cnt[PER * tid + q] = mine;
    mine += c;
    large |= c > (uint32_t)kRunMax;
  }
  const uint32_t before = block256_excl_scan(mine, L.lds4, &all);
#pragma unroll
  for (int q = 0; q < PER; ++q) L.cnt[PER * tid + q] += before;
  if (!__syncthreads_or(large)) {
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (holds(k)) L.key[L.cnt[bucket(key[k])] + at[k]] = key[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (!holds(k)) continue;
      const uint32_t d = bucket(key[k]);
      const int a = (int)L.cnt[d], e = d + 1 < kRunBlock ? (int)L.cnt[d + 1] : len;
      int r = a;
      for (int j = a; j < e; ++j) r += L.key[j] < key[k] ? 1 : 0;
      at[k] = (uint32_t)r;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (holds(k)) L.key[at[k]] = key[k];
    __syncthreads();
  } else {
    uint32_t* cnt = L.cnt + 256 * w;  // this wavefront's digit counts
    for (int bit = kRunBits + __builtin_ctzll(varying); bit < top; bit += 8) {
      __syncthreads();
      for (int q = lane; q < 256; q += 64) cnt[q] = 0u;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        at[k] = 0u;
        if (k >= per) continue;
        const uint32_t d = (uint32_t)(key[k] >> bit) & 255u;
        const uint64_t m = match_digit8(d, ballot64(holds(k)));
        const uint32_t r = (uint32_t)popc64(m & lanemask_lt()), c = cnt[d];
        at[k] = c + r;
        if (holds(k) && r == 0u) cnt[d] = c + (uint32_t)popc64(m);
      }
      __syncthreads();
      mine = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t c = L.cnt[256 * q + tid];
        L.cnt[256 * q + tid] = mine;
        mine += c;
      }
      L.lst[tid] = block256_excl_scan(mine, L.lds4, &all);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k)
        if (holds(k)) {
          const uint32_t d = (uint32_t)(key[k] >> bit) & 255u;
          L.key[L.lst[d] + cnt[d] + at[k]] = key[k];
        }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k)
        if (holds(k)) key[k] = L.key[p0 + 64 * k];
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    key[k] = holds(k) ? L.key[p0 + 64 * k] : 0ull;
    at[k] = holds(k) ? vals[start + (int)(key[k] & (kRunBlock - 1))] : 0u;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) loaded(at[k]);
  __syncthreads();  // all values read
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (holds(k)) {
      keys[start + p0 + 64 * k] = pre << shift | key[k] >> kRunBits;
      vals[start + p0 + 64 * k] = at[k];
    }
}

// For keys with a long run out of order; without one it ends at once.  Runs of
// up to kRunBlock keys are sorted by a block each.  Longer ones are sorted by
// the bits below the passes', each as an array of its own: a stage of digit
// counts (1) and the passes (2 on).  Items (tiles of the runs: at most 3/2 of
// the array's tiles, for at most five passes, so that their status words fit
// the array's of eight) are taken in order by a ticket, and an item waits for
// the stage before its own to end: those items belong to blocks that already
// run, so the wait ends however many blocks are resident.
// Sort (all its launches) in random order: 30,000 particles of a Plummer sphere
// of 1/100 of the box 62 us, 10^6 168 (eight passes over everything: 80 and 236;
// uniform: 44 and 144); a body of 1/1000 of the box, its runs longer than
// kRunBlock from 33,000 particles on: 10^5 116 us, 10^6 267, 4 10^6 628 (91, 237,
// 546).
//
// Between stages data passes from one XCD's L2 to another's.  All of it is
// stored and loaded past them (tile_store, tile_load): a release and an acquire
// fence for every tile, each of which goes over an L2, took 15 us of a stage at
// 10^6 particles when one wavefront of a block made them, some 80 when all four
// did.  A stage there takes 18 us, a pass in a launch of its own 25.
//
// The last item of a stage tells the blocks that wait, by words of their own:
// polls of the counter itself hold up the additions to it (40 us a stage).
__device__ __forceinline__ void stage_end(SortHead* head, const RunWs& ws, int stage, int items) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's stores are done
  __syncthreads();
  if (threadIdx.x < kWave) {
    uint32_t before = 0u;
    if (threadIdx.x == 0)
      before = __hip_atomic_fetch_add(&head->done[stage], 1u, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane((int)before) == items - 1)
      tile_store<true>(ws.ready + (int)threadIdx.x * kReadyLine, (uint32_t)stage + 1u);
  }
}
static_assert(kReady == kWave, "one lane per word");

// All stages before `stage` have ended.
__device__ __forceinline__ void stage_wait(const RunWs& ws, int stage,
                                           uint32_t* __restrict__ err) {
  const uint32_t* p = ws.ready + (int)(blockIdx.x % kReady) * kReadyLine;
  int spins = 0;
  while ((int)tile_load<true>(p) < stage) {
    __builtin_amdgcn_s_sleep(4);
    if (++spins > kLookbackSpin) {
      atomicOr(err, kErrSort);
      break;
    }
  }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void k_resort(uint64_t* k0, uint32_t* v0, uint64_t* k1,
                                                 uint32_t* v1, int n, uint32_t* status, RunWs ws,
                                                 SortHead* head, uint32_t* __restrict__ err) {
  if (head->resort == 0u) return;
  __shared__ union {
    SortLds sort;
    RunLds run;
  } U;
  const int tid = threadIdx.x;
  const uint32_t shift = head->shift;
  const int nr = (int)head->runs;
  for (int r = blockIdx.x; r < nr; r += gridDim.x) {
    const uint32_t i = ws.runs[r];
    if (i == ~0u) continue;  // a longer one
    sort_run(U.run, k0, v0, n, shift, (int)i);
    __syncthreads();  // the LDS of the next
  }
  const int no = (int)head->over;
  if (no == 0) return;
  SortLds& L = U.sort;
  const int npass = (int)(shift + 7) / 8;
  const bool odd = npass & 1;  // the runs then begin in the second buffer
  // first item of every run: by each block for up to 256 of them, otherwise by
  // one for all (stage 0, ticket 0)
  __shared__ uint32_t s_item[256];
  const bool few = no <= 256;
  int items = 0;  // of every stage but 0 (0: not known yet)
  if (few) {
    uint32_t all;
    const uint32_t tiles = tid < no ? (ws.len[tid] + kSortTile - 1) / kSortTile : 0u;
    s_item[tid] = block256_excl_scan(tiles, L.lds4, &all);
    items = (int)all;
  }
  const int t0 = few ? 0 : 1;  // ticket of the first item
  for (;;) {
    __syncthreads();  // the LDS of the item before
    if (tid == 0) {
      const int t = (int)atomicAdd(&head->ticket, 1u);
      L.tile = t;
      if (t >= t0) {
        if (items == 0) {
          stage_wait(ws, 1, err);
          items = (int)tile_load<true>(&head->items);
        }
        const int stage = 1 + (t - t0) / items;
        if (stage > 1 && stage <= npass + 1) stage_wait(ws, stage, err);
      }
    }
    __syncthreads();
    const int t = L.tile;
    if (t < t0) {
      uint32_t before = 0u;
      for (int r0 = 0; r0 < no; r0 += 256) {
        const int r = r0 + tid;
        uint32_t all;
        const uint32_t o = block256_excl_scan(
            r < no ? (ws.len[r] + kSortTile - 1) / kSortTile : 0u, L.lds4, &all);
        if (r < no) tile_store<true>(ws.item + r, before + o);
        before += all;
      }
      if (tid == 0) tile_store<true>(&head->items, before);
      stage_end(head, ws, 0, 1);
      continue;
    }
    if (items == 0) items = (int)tile_load<true>(&head->items);
    const int stage = 1 + (t - t0) / items, item = (t - t0) % items;
    if (stage > npass + 1) return;
    // the run of the item: the last with no later first item
    int r = 0, first = 0;
    if (few) {
      r = __syncthreads_count(tid < no && (int)s_item[tid] <= item) - 1;
      first = (int)s_item[r];
    } else {
      for (int size = no; size > 1;) {
        const int step = (size + 255) / 256;
        const int c = __syncthreads_count(tid * step < size &&
                                          (int)tile_load<true>(ws.item + r + tid * step) <= item);
        r += (c - 1) * step;
        size = min(step, size - (c - 1) * step);
      }
      first = (int)tile_load<true>(ws.item + r);
    }
    const int start = (int)ws.start[r], len = (int)ws.len[r], tile = item - first;
    uint32_t* hist = ws.hist + (int64_t)r * npass * 256;
    if (stage == 1) {
      uint32_t(*h)[256] = reinterpret_cast<uint32_t(*)[256]>(L.buf);
      for (int p = 0; p < npass; ++p) {
        h[p][tid] = 0u;
        tile_store<true>(status + ((int64_t)p * items + item) * 256 + tid, 0u);
      }
      __syncthreads();
      count_digits(k0 + start, len, tile * kSortTile, 0u, npass, h);
      if (odd) {
        for (int i = tile * kSortTile + tid; i < min((tile + 1) * kSortTile, len); i += 256) {
          tile_store<true>(k1 + start + i, k0[start + i]);
          tile_store<true>(v1 + start + i, v0[start + i]);
        }
      }
      __syncthreads();
      for (int p = 0; p < npass; ++p)
        if (h[p][tid]) atomicAdd(&hist[p * 256 + tid], h[p][tid]);
    } else {
      const int pass = stage - 2;
      const uint32_t gh = tile_load<true>(&hist[pass * 256 + tid]);
      clear_counts(L);
      __syncthreads();
      const bool second = odd == ((pass & 1) == 0);
      radix_tile<true>(L, (second ? k1 : k0) + start, (second ? v1 : v0) + start,
                 (second ? k0 : k1) + start, (second ? v0 : v1) + start, len,
                 8u * (uint32_t)pass, tile, status + ((int64_t)pass * items + first) * 256, gh,
                 err);
    }
    stage_end(head, ws, stage, items);
  }
}

// Few particles: prediction, keys and sort by one block, keys in registers and
// LDS, PER per thread.  The leading npass digits first; if two neighbours are
// then out of order, all eight.  The separate launches take some 5 us each,
// whatever they do: 29 -> 9 us at 1000 particles, 37 -> 15 at 1728, 44 -> 29
// at 3375; its own time is that of one CU and doubles with n, so that beyond
// 4096 particles the launches win (47 us at 8000).
template <int PER>
__global__ __launch_bounds__(1024) void k_sort_small(KParams kp, Parts p, int predict, int npass,
                                                      const DevState* __restrict__ ds,
                                                      uint64_t* __restrict__ keys,
                                                      uint32_t* __restrict__ vals,
                                                      uint32_t* __restrict__ err) {
  constexpr int NS = PER * 16;  // (key slice, wavefront) sets of 64 keys, in key order
  __shared__ alignas(16) uint16_t wc[256 * NS];
  __shared__ uint64_t s_key[PER * 1024];
  __shared__ uint32_t s_val[PER * 1024];
  __shared__ uint32_t lst[256];
  __shared__ uint32_t wtot[4];
  __shared__ uint64_t wr[16][2];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int n = kp.n;
  const double dt = predict ? ds->dt_cur : 0.0;
  uint64_t key[PER];
  uint32_t val[PER];
  uint64_t ones = 0ull, zeros = 0ull;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * 1024 + tid;
    key[k] = 0ull;
    val[k] = (uint32_t)i;
    if (i < n) {
      key[k] = predict_key(kp, p, predict != 0, dt, i, bad);
      ones |= key[k];
      zeros |= ~key[k];
    }
  }
  if (bad) atomicOr(err, kErrNonFinite);
  ones = wave_or_u64(ones);
  zeros = wave_or_u64(zeros);
  if (lane == 0) {
    wr[w][0] = ones;
    wr[w][1] = zeros;
  }
  __syncthreads();
  for (int q = 0; q < 16; ++q) {
    ones |= wr[q][0];
    zeros |= wr[q][1];
  }
  uint32_t shift = sort_shift(ones & zeros, npass);
  for (;;) {
    for (int pass = 0; pass < npass; ++pass, shift += 8) {
      for (int q = tid; q < 256 * NS / 8; q += 1024)
        reinterpret_cast<uint4*>(wc)[q] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
      uint32_t rank[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const bool valid = k * 1024 + tid < n;
        const uint32_t d = (uint32_t)((key[k] >> shift) & 255ull);
        const uint64_t m = match_digit8(d, ballot64(valid));
        rank[k] = (uint32_t)popc64(m & lanemask_lt());
        if (valid && rank[k] == 0) wc[d * NS + k * 16 + w] = (uint16_t)popc64(m);
      }
      __syncthreads();
      // thread d < 256: exclusive offsets of digit d over the sets, its start
      uint32_t mine = 0u, inc = 0u;
      if (tid < 256) {
        uint16_t c[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) c[q] = wc[tid * NS + q];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          const uint32_t v = c[q];
          c[q] = (uint16_t)mine;
          mine += v;
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) wc[tid * NS + q] = c[q];
        inc = wave_incl_scan_u32(mine);
        if (lane == 63) wtot[w] = inc;
      }
      __syncthreads();
      if (tid < 256) {
        uint32_t off = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) off += q < w ? wtot[q] : 0u;
        lst[tid] = off + inc - mine;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const uint32_t d = (uint32_t)((key[k] >> shift) & 255ull);
        if (k * 1024 + tid < n) {
          const uint32_t at = lst[d] + (uint32_t)wc[d * NS + k * 16 + w] + rank[k];
          s_key[at] = key[k];
          s_val[at] = val[k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int i = k * 1024 + tid;
        key[k] = i < n ? s_key[i] : 0ull;
        val[k] = i < n ? s_val[i] : 0u;
      }
    }
    bool out = false;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = k * 1024 + tid;
      out |= i + 1 < n && key[k] > s_key[i + 1];
    }
    if (!__syncthreads_or(out)) break;
    npass = 8;  // equal keys are in the order of the particles and stay so
    shift = 0u;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * 1024 + tid;
    if (i < n) {
      keys[i] = key[k];
      vals[i] = val[k];
    }
  }
}

// ============================================================================
// Permute the particle fields into key order (gather, then copy back).
// ============================================================================
struct FieldSet {
  double* f[kMaxFields];
  int64_t* id;
  int nf;
  int im;           // index of m in f (x, y, z are f[0..2])
  double4* xyzm;    // packed x, y, z, m in the new order (FP64 density gathers), or null
};

__global__ __launch_bounds__(256) void k_gather(FieldSet fs, const uint32_t* __restrict__ perm,
                                                 double* __restrict__ tmp,
                                                 int64_t* __restrict__ tmp_id, int n,
                                                 int64_t stride) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const uint32_t j = perm[k];
    for (int f = 0; f < fs.nf; ++f) tmp[f * stride + k] = fs.f[f][j];
    if (fs.id) tmp_id[k] = fs.id[j];
  }
}

__global__ __launch_bounds__(256) void k_copy_back(FieldSet fs, const double* __restrict__ tmp,
                                                    const int64_t* __restrict__ tmp_id, int n,
                                                    int64_t stride) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    for (int f = 0; f < fs.nf; ++f) fs.f[f][k] = tmp[f * stride + k];
    if (fs.id) fs.id[k] = tmp_id[k];
    if (fs.xyzm)
      fs.xyzm[k] =
          make_double4(tmp[k], tmp[stride + k], tmp[2 * stride + k], tmp[fs.im * stride + k]);
  }
}

// Few particles: in place, one block per field (the last one: the ids), PER
// values per thread in registers between the reads and the writes.  One launch
// instead of two and no pass through memory in between: 11 -> 4 us at 1000
// particles, 12 -> 7 at 8000, 14 -> 9 at 15,625; a field's time is that of one
// CU and would pass the two launches' soon after 16,384.
template <int PER>
__global__ __launch_bounds__(1024) void k_permute_small(FieldSet fs,
                                                         const uint32_t* __restrict__ perm, int n) {
  const int f = (int)blockIdx.x, tid = threadIdx.x;
  uint32_t j[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) j[k] = k * 1024 + tid < n ? perm[k * 1024 + tid] : 0u;
  if (f == fs.nf) {
    int64_t v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] = fs.id[j[k]];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (k * 1024 + tid < n) fs.id[k * 1024 + tid] = v[k];
    return;
  }
  double* a = fs.f[f];
  double v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) v[k] = a[j[k]];
  __syncthreads();
  const int part = f == fs.im ? 3 : f;  // of the packed x, y, z, m
  double* q = fs.xyzm && part < 4 && (f < 3 || f == fs.im)
                  ? reinterpret_cast<double*>(fs.xyzm) + part
                  : nullptr;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * 1024 + tid;
    if (i < n) {
      a[i] = v[k];
      if (q) q[4 * i] = v[k];
    }
  }
}

// Packed x, y, z, m from the particle arrays (the density entry point: the
// caller may have changed m, or x with it, since the permute wrote them).
__global__ __launch_bounds__(256) void k_pack_xyzm(Parts p, int n, double4* __restrict__ xyzm) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    xyzm[k] = make_double4(p.x[k], p.y[k], p.z[k], p.m[k]);
}

// Node h_max refresh modes: 1 a new tree (boxes too), 2 always, 0 only while
// the neighbour lists of the tree are not valid for the force.
__device__ __forceinline__ bool h_refresh_needed(const DevState* ds, int mode) {
  return mode != 0 || ds->leaf_state != 1 || ds->lists_missing != 0;
}

// The mixed kernels' 16-byte gather records: position codes in the tree's
// frame (DevState::qf, set with the node boxes) and m (the density gather)
// or h (the list kernel's candidates) in FP32.  Rewritten with every refresh
// of the nodes' h_max (mode as there), so that a list pass sees the h the
// walk's radii were sized for.
__global__ __launch_bounds__(256) void k_pack_q(KParams kp, Parts p, int n,
                                                const DevState* __restrict__ ds, int mode,
                                                int4* __restrict__ qm, int4* __restrict__ qh) {
  if (!h_refresh_needed(ds, mode)) return;
  const QFrame f = ds->qf;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const int32_t qx = qcode(p.x[k], f, 0, kp.periodic[0]);
    const int32_t qy = qcode(p.y[k], f, 1, kp.periodic[1]);
    const int32_t qz = qcode(p.z[k], f, 2, kp.periodic[2]);
    qm[k] = make_int4(qx, qy, qz, __float_as_int((float)p.m[k]));
    qh[k] = make_int4(qx, qy, qz, __float_as_int((float)p.h[k]));
  }
}

// ============================================================================
// Tree and groups from the sorted keys, in three launches.
//
// d(s): level at which keys s-1 and s first differ (1..21; 22 if equal),
// d(0) = d(n) = 0.  The level-l cell containing s spans [a, b) with a the
// last index <= s and b the first index > s where d <= l.  A cell at level
// l is a node iff its parent holds more than n_leaf particles, i.e. iff the
// smallest level L(s) at which the cell containing s holds <= n_leaf
// particles is >= l.  So the nodes starting at s are the levels
// d(s)..L(s), and L(s) is found in a window of n_leaf keys on each side:
//   L(s) = min over s < b <= s+T, b-T <= a <= s of max(d(a), d(b)).
// ============================================================================
constexpr int kHalo = 64;  // n_leaf, n_group <= 64

__device__ __forceinline__ int diff_level(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  if (x == 0ull) return 22;
  return (__clzll((long long)x) + 2) / 3;
}

__device__ __forceinline__ int window_level(const uint8_t* d, int idx, int s, int n, int T) {
  int run = 22;  // d is 0 at the first particle and before
  int best = 22;
  for (int k = 0; k < T; k += 8) {  // loads of eight steps at a time
    int dl[8], dr[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = min(k + u, T - 1);
      dl[u] = d[idx - q];
      dr[u] = s + T - q <= n ? d[idx + T - q] : 22;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {  // a repeated last step changes nothing
      run = min(run, dl[u]);
      best = min(best, max(dr[u], run));
    }
  }
  return best;
}

// First index > s whose key leaves the level-l cell of s (galloping search).
__device__ __forceinline__ int cell_end(const uint64_t* __restrict__ keys, int n, int s, int l) {
  if (l == 0) return n;
  const int sh = 3 * (kKeyLevels - l);
  const uint64_t pre = keys[s] >> sh;
  int lo = s, step = 1;
  while (lo + step < n && (keys[lo + step] >> sh) == pre) {
    lo += step;
    step <<= 1;
  }
  int hi = min(lo + step, n);
  while (hi - lo > 1) {
    const int mid = lo + ((hi - lo) >> 1);
    if ((keys[mid] >> sh) == pre)
      lo = mid;
    else
      hi = mid;
  }
  return hi;
}

// Groups (Sect. 3.1): the group cells are the chopped cells of at most
// n_group particles (level lg >= 1, so their parent P holds more).
// Consecutive children of P that are group cells are packed, in curve order
// and greedily, into groups of at most n_group particles; a child that is
// chopped further ends a pack.  For the group cell starting at s: whether a
// group starts there, and its particle count.  D(j) is the level at which
// keys j-1 and j first differ (0 at j <= 0 and j >= n), so j begins a new
// level-l cell iff D(j) <= l.  The run of group-cell siblings around s is
// found from s outwards (at most eight children, each of at most n_group
// particles), then packed from its first cell.
template <typename DFn>
__device__ void group_pack(DFn D, int n, int s, int lg, int n_group, bool& start, int& count) {
  int rs = s;  // first particle of the run
  for (int k = 0; k < 7 && D(rs) > lg - 1; ++k) {
    int j = rs - 1;  // the previous sibling starts at the last boundary before rs
    while (j > rs - n_group && D(j) > lg) --j;
    if (D(j) > lg) break;  // that sibling holds more than n_group particles
    rs = j;
  }
  int acc = 0;      // particles of the open pack
  int pstart = -1;  // its first particle
  start = false;
  count = 0;
  for (int c0 = rs;;) {
    int c1 = c0 + 1;
    while (c1 < n && c1 <= c0 + n_group && D(c1) > lg) ++c1;
    if (c1 > c0 + n_group) break;  // a chopped sibling ends the run
    const int cc = c1 - c0;
    const bool joins = acc > 0 && acc + cc <= n_group;
    if (pstart == s && !joins) break;  // the pack that starts at s is complete
    if (joins) {
      acc += cc;
    } else {
      acc = cc;
      pstart = c0;
    }
    if (c0 == s && pstart != s) return;  // s's cell joined an earlier pack
    c0 = c1;
    if (c0 >= n || D(c0) <= lg - 1) break;  // P ends
  }
  start = pstart == s;
  count = start ? acc : 0;
}

// The same packing from 192-bit boundary masks over particles [w0, w0 + 192)
// (bit p: particle w0 + p begins a cell at the group level, bc, or at the
// parent level, bp); s sits at bit ps.  For n_group <= 8 every cell the
// packing of s inspects lies within 64 particles of s.
__device__ __forceinline__ bool bit3(const uint64_t (&m)[3], int p) {
  return (m[p >> 6] >> (p & 63)) & 1ull;
}
__device__ __forceinline__ int hi_below(const uint64_t (&m)[3], int p) {  // or -1
  for (int w = p >> 6; w >= 0; --w) {
    uint64_t v = m[w];
    if (w == (p >> 6)) v &= (p & 63) ? (~0ull >> (64 - (p & 63))) : 0ull;
    if (v != 0ull) return w * 64 + 63 - __builtin_clzll(v);
  }
  return -1;
}
__device__ __forceinline__ int lo_above(const uint64_t (&m)[3], int p) {  // or 192
  for (int w = (p + 1) >> 6; w < 3; ++w) {
    uint64_t v = m[w];
    if (w == ((p + 1) >> 6)) v &= ~0ull << ((p + 1) & 63);
    if (v != 0ull) return w * 64 + __builtin_ctzll(v);
  }
  return 192;
}
__device__ void group_pack_masks(const uint64_t (&bc)[3], const uint64_t (&bp)[3], int ps,
                                 int n_group, bool& start, int& count) {
  int rs = ps;
  for (int k = 0; k < 7 && !bit3(bp, rs); ++k) {
    const int pb = hi_below(bc, rs);
    if (pb < rs - n_group) break;  // that sibling holds more than n_group particles
    rs = pb;
  }
  int acc = 0, pstart = -1;
  start = false;
  count = 0;
  for (int c0 = rs;;) {
    const int c1 = lo_above(bc, c0);
    if (c1 - c0 > n_group) break;  // a chopped sibling ends the run
    const int cc = c1 - c0;
    const bool joins = acc > 0 && acc + cc <= n_group;
    if (pstart == ps && !joins) break;
    if (joins) {
      acc += cc;
    } else {
      acc = cc;
      pstart = c0;
    }
    if (c0 == ps && pstart != ps) return;
    c0 = c1;
    if (bit3(bp, c0)) break;  // P ends
  }
  start = pstart == ps;
  count = start ? acc : 0;
}

__global__ __launch_bounds__(256) void k_tree_levels(const uint64_t* __restrict__ keys, int n,
                                                      int n_leaf, int n_group,
                                                      uint8_t* __restrict__ dlev,
                                                      uint8_t* __restrict__ lleaf,
                                                      uint8_t* __restrict__ gsize,
                                                      uint8_t* __restrict__ gstart,
                                                      uint32_t* __restrict__ tree_cnt, int nblk,
                                                      int32_t* __restrict__ nnchild,
                                                      int64_t node_cap) {
  __shared__ uint8_t d[kTreeTile + 2 * kHalo + 1];
  // child counts of every node slot cleared for k_tree_emit's increments
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < node_cap;
       k += (int64_t)gridDim.x * blockDim.x)
    nnchild[k] = 0;
  __shared__ uint32_t lc[kLevels];
  __shared__ uint32_t gc;
  const int base = blockIdx.x * kTreeTile;
  for (int t = threadIdx.x; t < kTreeTile + 2 * kHalo + 1; t += blockDim.x) {
    const int j = base - kHalo + t;
    d[t] = (j <= 0 || j >= n) ? (uint8_t)0 : (uint8_t)diff_level(keys[j - 1], keys[j]);
  }
  if (threadIdx.x < kLevels) lc[threadIdx.x] = 0;
  if (threadIdx.x == 0) gc = 0;
  __syncthreads();
  const int s = base + threadIdx.x;
  const bool valid = s < n;
  const int idx = kHalo + threadIdx.x;
  int ds = 0, ll = 0, lg_raw = kLevels;
  if (valid) {
    ds = d[idx];
    ll = min(window_level(d, idx, s, n, n_leaf), kKeyLevels);
    lg_raw = window_level(d, idx, s, n, n_group);
  }
  bool start = false;
  int gcount = 0;
  const bool cell = valid && lg_raw <= kKeyLevels && ds <= lg_raw;  // s begins its group cell
  if (cell && lg_raw == 0) {
    start = true;
    gcount = n;  // the whole set is one group
  }
  if (n_group <= 8) {
    // per wavefront and group level L: boundary masks over the 192
    // particles around the wavefront's 64, from the LDS window
    const int lane = threadIdx.x & (kWave - 1);
    const int t0 = threadIdx.x - lane;  // window index of particle s - lane - 64
    uint64_t todo = ballot64(cell && lg_raw >= 1);
    while (todo != 0ull) {
      const int L = __builtin_amdgcn_readlane(lg_raw, __builtin_ctzll(todo));
      uint64_t bc[3], bp[3];
#pragma unroll
      for (int w = 0; w < 3; ++w) {
        const int dj = d[t0 + kWave * w + lane];
        bc[w] = ballot64(dj <= L);
        bp[w] = ballot64(dj <= L - 1);
      }
      const bool mine = cell && lg_raw == L;
      if (mine) group_pack_masks(bc, bp, lane + kWave, n_group, start, gcount);
      todo &= ~ballot64(mine);
    }
  } else if (cell && lg_raw >= 1) {
    // diff levels from the block's LDS window (it reaches kHalo particles
    // past the tile on both sides), else from the keys
    auto D = [&](int j) -> int {
      const int t = j - base + kHalo;
      if (t >= 0 && t < kTreeTile + 2 * kHalo + 1) return d[t];
      return (j <= 0 || j >= n) ? 0 : diff_level(keys[j - 1], keys[j]);
    };
    group_pack(D, n, s, lg_raw, n_group, start, gcount);
  }
  if (valid && lg_raw > kKeyLevels) {
    // level-21 cell with more than n_group identical keys: cut in chunks
    int a = s;
    while (a > 0 && keys[a - 1] == keys[a]) --a;
    start = ((s - a) % n_group) == 0;
    if (start) gcount = min(n_group, cell_end(keys, n, s, kKeyLevels) - s);
  }
  if (valid) {
    dlev[s] = (uint8_t)ds;
    lleaf[s] = (uint8_t)ll;
    gsize[s] = (uint8_t)gcount;
    gstart[s] = start ? 1 : 0;
    for (int l = ds; l <= ll; ++l) atomicAdd(&lc[l], 1u);
    if (start) atomicAdd(&gc, 1u);
  }
  __syncthreads();
  // the group counts follow the node counts of the levels, so that one scan
  // does both (its length rounded up with zeros)
  if (threadIdx.x < kLevels) tree_cnt[threadIdx.x * nblk + blockIdx.x] = lc[threadIdx.x];
  if (threadIdx.x == 0) tree_cnt[kLevels * nblk + blockIdx.x] = gc;
  if (blockIdx.x == 0 && threadIdx.x < 3) tree_cnt[(kLevels + 1) * nblk + threadIdx.x] = 0;
}

// State of the list kernels on a tree without groups: all particles flagged,
// the force left to the walk (of no group).
__device__ __forceinline__ void no_rows(DevState* ds) {
  ds->n_flag_rows = 1;
  ds->leaf_state = 2;
}

// tree_off: exclusive prefix of the node counts, level by level, then of the
// group counts; total: nodes and groups together.
__global__ __launch_bounds__(256) void k_tree_emit(
    const uint64_t* __restrict__ keys, int n, const uint8_t* __restrict__ dlev,
    const uint8_t* __restrict__ lleaf, const uint8_t* __restrict__ gsize,
    const uint8_t* __restrict__ gstart, const uint32_t* __restrict__ tree_off,
    const uint32_t* __restrict__ total, int nblk, int64_t node_cap,
    int32_t* __restrict__ nlevel, int32_t* __restrict__ nfirst, int32_t* __restrict__ ncount,
    int32_t* __restrict__ nparent, int32_t* __restrict__ nchild, int32_t* __restrict__ nnchild,
    int32_t* __restrict__ gfirst, int32_t* __restrict__ gcount, int32_t* __restrict__ nl_len,
    int32_t* __restrict__ grp_of, int32_t* __restrict__ gflag, DevState* __restrict__ ds) {
  __shared__ uint32_t wc[4][kLevels];
  __shared__ uint32_t first[4][kLevels];  // index of a wavefront's first node of a level
  __shared__ uint32_t gw[4];
  __shared__ uint8_t s_d[kTreeTile + kHalo];  // start levels from the tile's first particle on
  const int n_nodes = (int)tree_off[kLevels * nblk];
  // a tree that outgrew the node arrays is reported and left empty, so that no
  // later launch reads or writes past them; its particles have empty rows and
  // count as one flagged group that no list names, so that the list kernels
  // pass them over (no list kernel will write rows for them)
  const bool fits = n_nodes >= 0 && (int64_t)n_nodes <= node_cap;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ds->n_nodes = fits ? n_nodes : 0;
    ds->n_groups = fits ? (int)(*total - (uint32_t)n_nodes) : 0;
    if (!fits) atomicOr(&ds->err, kErrNodes);
  }
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int s = blockIdx.x * kTreeTile + tid;
  const bool valid = s < n;
  if (!fits) {
    if (valid) {
      nl_len[s] = 0;
      grp_of[s] = 0;
    }
    if (s == 0) {
      gflag[0] = 1;
      no_rows(ds);
    }
    return;
  }
  const int dsv = valid ? dlev[s] : 99;
  const int ll = valid ? lleaf[s] : -1;
  const bool gs = valid && gstart[s];
  const uint32_t off = tid < kLevels ? tree_off[tid * nblk + blockIdx.x] : 0u;
  s_d[tid] = valid ? (uint8_t)dsv : (uint8_t)0;  // a cell ends at the last particle
  if (tid < kHalo) {
    const int j = s + kTreeTile;
    s_d[kTreeTile + tid] = j < n ? dlev[j] : (uint8_t)0;
  }
  for (int l = 0; l < kLevels; ++l) {
    const uint64_t b = ballot64(valid && dsv <= l && l <= ll);
    if (lane == 0) wc[w][l] = (uint32_t)popc64(b);
  }
  const uint64_t bg = ballot64(gs);
  if (lane == 0) gw[w] = (uint32_t)popc64(bg);
  __syncthreads();
  if (tid < kLevels) {
    uint32_t f = off;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      first[q][tid] = f;
      f += wc[q][tid];
    }
  }
  __syncthreads();
  // only leaves need their particle count (the walk reads particles of leaves
  // only; inner counts are derived on the host for inspection).  A leaf that
  // starts here ends where a cell of its level or above starts next: within
  // n_leaf particles, unless it is a level-21 cell of coincident keys.
  // Latency bound at small n: what a level needs is in LDS before the level
  // loop (a galloping search of the keys from each leaf and a load of the
  // offset per level were chains of dependent loads: 12.5 -> 6.8 us at 1000
  // particles, 16.5 -> 11.0 at 294,912, 467 -> 295 at 16.8M).
  int leaf_count = 0;
  if (dsv <= ll) {
    int t = tid + 1;
    const int t1 = min(tid + kHalo, kTreeTile + kHalo - 1);
    while (t < t1 && (int)s_d[t] > ll) ++t;
    leaf_count = (int)s_d[t] <= ll ? t - tid : cell_end(keys, n, s, ll) - s;
  }
  int prev = -1, par_at_d = -1;
  for (int l = 0; l < kLevels; ++l) {
    if (ballot64(valid && dsv - 1 <= l && l <= ll) == 0ull) continue;
    const bool mem = valid && dsv <= l && l <= ll;
    const uint64_t b = ballot64(mem);
    const int idx = (int)(first[w][l] + (uint32_t)popc64(b & lanemask_lt()));
    if (valid && l == dsv - 1) par_at_d = idx - 1;  // last level-(d-1) node before s
    if (mem) {
      nlevel[idx] = l;
      nfirst[idx] = s;
      ncount[idx] = (l == ll) ? leaf_count : 0;
      const int parent = (l == 0) ? -1 : (l == dsv ? par_at_d : prev);
      nparent[idx] = parent;
      nchild[idx] = -1;
      if (l > dsv) nchild[prev] = idx;  // first child of (l-1, s) is (l, s)
      if (parent >= 0) atomicAdd(&nnchild[parent], 1);
      prev = idx;
    }
  }
  uint32_t rg = (uint32_t)popc64(bg & lanemask_lt());
  for (int q = 0; q < w; ++q) rg += gw[q];
  if (gs) {
    const int g = (int)(tree_off[kLevels * nblk + blockIdx.x] - (uint32_t)n_nodes + rg);
    gfirst[g] = s;
    gcount[g] = gsize[s];
  }
}

// ---- node and group boxes and largest h -----------------------------------
// Every leaf and group covers a contiguous range of the sorted particles:
// k_range_boxes reduces each one's particles (four per wavefront, 16 lanes
// each, so the particle loads coalesce; the lanes combine by DPP moves, as
// LDS permutes took most of it: 32 -> 23 us at 294,912 particles, 840 -> 600
// at 16.8M).  Inner nodes then take the union of
// their children's boxes and the largest of their h_max, one launch per
// level from the deepest up (k_level_boxes).  No atomics.  A leaf's or
// group's box is exactly the range's; an inner node's holds its children's
// conservative (rounded-up) boxes, so every box contains its particles.
// mode 1: boxes and h_max of a new tree; 0: h_max only, skipped on the device
// while the neighbour lists of the tree are valid; 2: h_max only, always.
struct Box7 {
  double lo[3], hi[3], hm;
};

__device__ __forceinline__ void box_empty(Box7& b) {
  for (int a = 0; a < 3; ++a) {
    b.lo[a] = SPH_INF;
    b.hi[a] = -SPH_INF;
  }
  b.hm = 0.0;
}

__device__ __forceinline__ float f32_up(double v) {
  float f = (float)v;
  if ((double)f < v) f = nextafterf(f, SPH_INF);
  return f;
}

__device__ __forceinline__ void write_node_box(const Box7& b, int it, int f, int e, int nc,
                                               const int32_t* __restrict__ nchild,
                                               WalkNode* __restrict__ wn, int do_bb) {
  if (do_bb) {
    WalkNode w;
    for (int a = 0; a < 3; ++a) {
      const double c = 0.5 * (b.lo[a] + b.hi[a]);
      w.c[a] = c;
      w.w[a] = f32_up(fmax(b.hi[a] - c, c - b.lo[a]));
    }
    w.hmax = f32_up(b.hm);
    w.first = f;
    w.count = e - f;
    w.child = nc ? nchild[it] : -1;
    w.nchild = nc;
    wn[it] = w;
  } else {
    wn[it].hmax = f32_up(b.hm);
  }
}

__device__ __forceinline__ void write_group_box(const Box7& b, int g, int f, int e,
                                                GroupInfo* __restrict__ gi, int do_bb) {
  if (do_bb) {
    GroupInfo G;
    for (int a = 0; a < 3; ++a) {
      G.c[a] = 0.5 * (b.lo[a] + b.hi[a]);
      G.w[a] = fmax(b.hi[a] - G.c[a], G.c[a] - b.lo[a]);
    }
    G.hmax = b.hm;
    G.first = f;
    G.count = e - f;
    gi[g] = G;
  } else {
    gi[g].hmax = b.hm;
  }
}

constexpr int kNoChunks = 2048;

// Small trees: every inner node by one wavefront, in the launch of the leaves
// and groups, from the particles of its range and the boxes of the whole
// kChunk-particle chunks inside it (k_chunk_boxes); its range ends where its
// next sibling starts, or, for a last child, where its parent's range ends.
// Up to kNoChunks particles the particles alone: the chunk boxes' launches take
// longer than the reads that they spare (boxes and refresh of a step: 16.6 ->
// 12.6 us at 1000 particles, 23 -> 18 at 1728; 22 -> 26 at 3375).
// One launch instead of one per level; on large trees the chunks' particles
// are read by many nodes of the lower levels, and the per-level launches win.
__device__ __forceinline__ void wave_box(Box7& b, int do_bb) {
  if (do_bb)
    for (int a = 0; a < 3; ++a) {
      b.lo[a] = wave_min_f64(b.lo[a]);
      b.hi[a] = wave_max_f64(b.hi[a]);
    }
  b.hm = wave_max_f64(b.hm);
}

// Lane-partial box of particles [a, e), lanes striding by 64.
__device__ __forceinline__ void add_particles(Box7& b, int a, int e, const double* __restrict__ x,
                                              const double* __restrict__ y,
                                              const double* __restrict__ z,
                                              const double* __restrict__ h, int do_bb) {
#pragma unroll 4
  for (int s = a + lane_id(); s < e; s += kWave) {
    if (do_bb) {
      const double px = x[s], py = y[s], pz = z[s];
      b.lo[0] = fmin(b.lo[0], px);
      b.hi[0] = fmax(b.hi[0], px);
      b.lo[1] = fmin(b.lo[1], py);
      b.hi[1] = fmax(b.hi[1], py);
      b.lo[2] = fmin(b.lo[2], pz);
      b.hi[2] = fmax(b.hi[2], pz);
    }
    b.hm = fmax(b.hm, h[s]);
  }
}

// cb: 8 doubles per chunk (lo xyz, hi xyz, h_max, unused).
__global__ __launch_bounds__(256) void k_chunk_boxes(const double* __restrict__ x,
                                                      const double* __restrict__ y,
                                                      const double* __restrict__ z,
                                                      const double* __restrict__ h, int n,
                                                      double* __restrict__ cb,
                                                      const DevState* __restrict__ ds, int mode) {
  if (!h_refresh_needed(ds, mode)) return;
  const int do_bb = mode == 1 ? 1 : 0;
  const int nch = (n + kChunk - 1) / kChunk;
  const int wpb = blockDim.x / kWave;
  for (int c = blockIdx.x * wpb + (int)(threadIdx.x / kWave); c < nch; c += gridDim.x * wpb) {
    Box7 b;
    box_empty(b);
    add_particles(b, c * kChunk, min(n, (c + 1) * kChunk), x, y, z, h, do_bb);
    wave_box(b, do_bb);
    if (lane_id() == 0) {
      double* o = cb + 8 * (int64_t)c;
      if (do_bb)
        for (int a = 0; a < 3; ++a) {
          o[a] = b.lo[a];
          o[3 + a] = b.hi[a];
        }
      o[6] = b.hm;
    }
  }
}

__device__ void inner_ranges(int blk, int nblocks, const double* __restrict__ x,
                             const double* __restrict__ y, const double* __restrict__ z,
                             const double* __restrict__ h, int n, const double* __restrict__ cb,
                             const int32_t* __restrict__ nfirst,
                             const int32_t* __restrict__ nparent,
                             const int32_t* __restrict__ nchild,
                             const int32_t* __restrict__ nnchild, WalkNode* __restrict__ wn,
                             int nn, int do_bb) {
  const int wpb = blockDim.x / kWave;
  const int nw = nblocks * wpb;
  for (int it = blk * wpb + (int)(threadIdx.x / kWave); it < nn; it += nw) {
    const int nc = nnchild[it];
    if (nc == 0) continue;
    const int f = nfirst[it];
    int e = n;
    int k = it;
    while (k > 0) {
      const int p = nparent[k];
      if (p < 0) break;
      if (k + 1 < nchild[p] + nnchild[p]) {
        e = nfirst[k + 1];
        break;
      }
      k = p;
    }
    Box7 b;
    box_empty(b);
    const int c0 = (f + kChunk - 1) / kChunk, c1 = e / kChunk;
    if (c1 > c0 && n > kNoChunks) {
      add_particles(b, f, c0 * kChunk, x, y, z, h, do_bb);
      for (int c = c0 + lane_id(); c < c1; c += kWave) {
        const double* q = cb + 8 * (int64_t)c;
        if (do_bb)
          for (int a = 0; a < 3; ++a) {
            b.lo[a] = fmin(b.lo[a], q[a]);
            b.hi[a] = fmax(b.hi[a], q[3 + a]);
          }
        b.hm = fmax(b.hm, q[6]);
      }
      add_particles(b, c1 * kChunk, e, x, y, z, h, do_bb);
    } else {
      add_particles(b, f, e, x, y, z, h, do_bb);
    }
    wave_box(b, do_bb);
    if (lane_id() == 0) write_node_box(b, it, f, e, nc, nchild, wn, do_bb);
  }
}

__global__ __launch_bounds__(256) void k_range_boxes(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ h, const int32_t* __restrict__ nfirst,
    const int32_t* __restrict__ ncount, const int32_t* __restrict__ nchild,
    const int32_t* __restrict__ nnchild, WalkNode* __restrict__ wn,
    const int32_t* __restrict__ gfirst, const int32_t* __restrict__ gcount,
    GroupInfo* __restrict__ gi, const DevState* __restrict__ ds, int mode, int nb_items, int n,
    const double* __restrict__ cb, const int32_t* __restrict__ nparent) {
  if (!h_refresh_needed(ds, mode)) return;
  const int do_bb = mode == 1 ? 1 : 0;
  const int nn = ds->n_nodes, ng = ds->n_groups;
  if ((int)blockIdx.x >= nb_items) {  // small trees: the inner nodes
    inner_ranges((int)blockIdx.x - nb_items, (int)gridDim.x - nb_items, x, y, z, h, n, cb,
                 nfirst, nparent, nchild, nnchild, wn, nn, do_bb);
    return;
  }
  // items 0..nn-1 are nodes (inner ones are left to k_level_boxes), the rest
  // groups; the trip count is uniform over the wavefront (its shuffles)
  const int seg = lane_id() >> 4, sub = lane_id() & 15;
  const int wpb = blockDim.x / kWave;
  const int nwv = nb_items * wpb;
  for (int base = (blockIdx.x * wpb + (int)(threadIdx.x / kWave)) * 4; base < nn + ng;
       base += nwv * 4) {
    const int it = base + seg;
    const bool is_node = it < nn;
    const bool item = it < nn + ng && !(is_node && nnchild[it] != 0);
    int f = 0, e = 0;
    if (item) {
      f = is_node ? nfirst[it] : gfirst[it - nn];
      e = f + (is_node ? ncount[it] : gcount[it - nn]);
    }
    Box7 b;
    box_empty(b);
    for (int s = f + sub; s < e; s += 16) {
      if (do_bb) {
        const double px = x[s], py = y[s], pz = z[s];
        b.lo[0] = fmin(b.lo[0], px);
        b.hi[0] = fmax(b.hi[0], px);
        b.lo[1] = fmin(b.lo[1], py);
        b.hi[1] = fmax(b.hi[1], py);
        b.lo[2] = fmin(b.lo[2], pz);
        b.hi[2] = fmax(b.hi[2], pz);
      }
      b.hm = fmax(b.hm, h[s]);
    }
    if (do_bb)
      for (int a = 0; a < 3; ++a) {
        b.lo[a] = seg_min<16>(b.lo[a]);
        b.hi[a] = seg_max<16>(b.hi[a]);
      }
    b.hm = seg_max<16>(b.hm);
    if (item && sub == 0) {
      if (is_node)
        write_node_box(b, it, f, e, 0, nchild, wn, do_bb);
      else
        write_group_box(b, it - nn, f, e, gi, do_bb);
    }
  }
}

// An inner node from its children (already final): the union of their boxes
// and the largest of their h_max; its range ends where its last child's ends.
__device__ __forceinline__ void inner_node(int it, const int32_t* __restrict__ nfirst,
                                           const int32_t* __restrict__ nchild,
                                           const int32_t* __restrict__ nnchild,
                                           WalkNode* __restrict__ wn, int mode) {
  const int nc = nnchild[it];
  if (nc == 0) return;
  const int c0 = nchild[it];
  double lo[3] = {SPH_INF, SPH_INF, SPH_INF}, hi[3] = {-SPH_INF, -SPH_INF, -SPH_INF};
  float hm = 0.f;
  int last_end = 0;
  for (int q = 0; q < nc; ++q) {
    const WalkNode w = wn[c0 + q];
    for (int a = 0; a < 3; ++a) {
      lo[a] = fmin(lo[a], w.c[a] - (double)w.w[a]);
      hi[a] = fmax(hi[a], w.c[a] + (double)w.w[a]);
    }
    hm = fmaxf(hm, w.hmax);
    last_end = w.first + w.count;
  }
  if (mode == 1) {
    WalkNode w;
    for (int a = 0; a < 3; ++a) {
      const double c = 0.5 * (lo[a] + hi[a]);
      w.c[a] = c;
      w.w[a] = f32_up(fmax(hi[a] - c, c - lo[a]));
    }
    w.hmax = hm;
    w.first = nfirst[it];
    w.count = last_end - w.first;
    w.child = c0;
    w.nchild = nc;
    wn[it] = w;
  } else {
    wn[it].hmax = hm;
  }
}

// Nodes are numbered level by level: level l is [off[l nblk], off[(l+1) nblk]).
__device__ __forceinline__ void level_range(int level, const uint32_t* __restrict__ off, int nblk,
                                            int nn, int& beg, int& end) {
  beg = (int)off[level * nblk];
  end = min(level + 1 < kLevels ? (int)off[(level + 1) * nblk] : nn, nn);
}

// The inner nodes of one level (large trees: one launch per level).
__global__ __launch_bounds__(256) void k_level_boxes(int level, const uint32_t* __restrict__ level_off,
                                                      int nblk, const int32_t* __restrict__ nfirst,
                                                      const int32_t* __restrict__ nchild,
                                                      const int32_t* __restrict__ nnchild,
                                                      WalkNode* __restrict__ wn,
                                                      const DevState* __restrict__ ds, int mode) {
  if (!h_refresh_needed(ds, mode)) return;
  int beg, end;
  level_range(level, level_off, nblk, ds->n_nodes, beg, end);
  for (int it = beg + blockIdx.x * blockDim.x + threadIdx.x; it < end;
       it += gridDim.x * blockDim.x)
    inner_node(it, nfirst, nchild, nnchild, wn, mode);
}

// Fixed-point frame of the mixed force records (QFrame) for the positions of
// the current tree: the box on periodic axes, the root node's box (a
// conservative one: its half-widths are rounded up) on open axes.
__global__ void k_qframe(KParams kp, const WalkNode* __restrict__ nodes,
                         DevState* __restrict__ ds) {
  if (threadIdx.x >= 3) return;
  const int a = threadIdx.x;
  QFrame& f = ds->qf;
  if (kp.periodic[a]) {
    f.o[a] = kp.lo[a];
    f.inv[a] = 4294967296.0 / kp.len[a];
    f.step[a] = (float)(kp.len[a] / 4294967296.0);
  } else {
    const bool any = ds->n_nodes > 0;
    const double c = any ? nodes[0].c[a] : 0.0;
    const double w = any ? (double)nodes[0].w[a] : 0.0;
    const double ext = w > 0.0 ? 2.0 * w : 1.0;
    f.o[a] = c - 0.5 * ext;
    f.inv[a] = 2147483648.0 / ext;
    f.step[a] = (float)(ext / 2147483648.0);
  }
}

// ============================================================================
// Group tree walk (Sect. 3.2): one wavefront per group, breadth-first.  The
// frontier lives in LDS; nodes are tested 64 at a time, opened inner nodes
// push their (contiguous) children, opened leaves append (first, count) to an
// LDS leaf list that is flushed through a candidate loop when it fills.  An
// inner node that lies wholly within the opening radius is appended whole
// (its particle range), which keeps the frontier to the nodes that straddle
// the edge of the search region.
// The opening test is conservative (a superset); the exact pair predicate is
// applied in the candidate loop.
// ============================================================================
constexpr int kFCap = 512;  // frontier entries per level in LDS
constexpr int kLCap = 128;  // leaves per flush
constexpr int kPMax = 128;  // pairs per particle slot
constexpr int kTile = 256;  // candidates staged in LDS at a time
constexpr int kFCapFb = 256, kTileFb = 128;  // of the flagged groups' density
constexpr int kSG = 8;      // groups sharing one super-group walk
constexpr int kSLCap = 256; // leaves a super-group walk may collect

// Nearest periodic image of a separation d (|d| < 1.5 len for positions in
// the box).  Branch-free: the two selects compile to conditional moves, so a
// wavefront does not split over the sign of d.
__device__ __forceinline__ double fold(double d, double len, double half, int periodic) {
  const double lp = periodic ? len : 0.0;
  double t = d > half ? d - lp : d;
  t = d < -half ? d + lp : t;
  return t;
}

// Largest squared distance between a point of the group box and a point of
// the node box, along the nearest periodic image of the centres (an upper
// bound of the minimum-image distance of every such pair).
__device__ __forceinline__ double box_far2(const WalkNode& nd, const GroupInfo& G,
                                           const KParams& kp) {
  double d2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double dc = nd.c[a] - G.c[a];
    if (kp.periodic[a]) dc = dc - kp.len[a] * rint(dc * kp.inv_len[a]);
    const double far = fabs(dc) + (double)nd.w[a] + G.w[a];
    d2 = d2 + far * far;
  }
  return d2;
}

// min-image squared distance between a node box and the group box
__device__ __forceinline__ double box_gap2(const WalkNode& nd, const GroupInfo& G,
                                           const KParams& kp) {
  double d2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double dc = nd.c[a] - G.c[a];
    if (kp.periodic[a]) dc = dc - kp.len[a] * rint(dc * kp.inv_len[a]);
    double gap = fabs(dc) - (double)nd.w[a] - G.w[a];
    gap = gap > 0.0 ? gap : 0.0;
    d2 = d2 + gap * gap;
  }
  return d2;
}

struct WalkLds {
  int lfirst[kLCap];
  int lcnt[kLCap];
  int lnode[kLCap];
  int loff[kLCap + 1];
};

// Candidate tile: up to kTile candidates of the flushed leaves.  FP64 path:
// absolute positions; FP32 path: positions relative to the group centre,
// folded to the nearest periodic image once, when staged.  `a` carries one
// more per-particle value (m_j for the density, h_j for the force), `j` the
// particle index.
template <typename T, int N = kTile>
struct TileOf {
  T x[N];
  T y[N];
  T z[N];
  T a[N];
  int j[N];
};

// Breadth-first walk.  open_r(node) returns the opening radius for a node;
// flush(nleaf) consumes the leaf list (loff filled).  A level's frontier
// holds FC entries in LDS and continues in this wavefront's region of
// global memory (`spill`, kSpill entries per level; search regions much
// larger than the local particle spacing need it).  Returns false on
// frontier overflow.
template <int FC, typename RadiusFn, typename FlushFn>
__device__ bool group_walk(const WalkNode* __restrict__ nodes, const GroupInfo& G,
                           const KParams& kp, WalkLds& L, int (&front)[2][FC],
                           int* __restrict__ spill, RadiusFn open_r, FlushFn flush) {
  const int lane = threadIdx.x;
  constexpr int cap = kFCap + kSpill;
  constexpr int stride = FC < kFCap ? 2 * kSpill : kSpill;  // spill entries per level
  static_assert(cap - FC <= stride, "a level's frontier fits LDS and its spill region");
  auto fget = [&](int lvl, int k) -> int {
    return k < FC ? front[lvl][k]
                  : __hip_atomic_load(&spill[lvl * stride + (k - FC)], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
  };
  auto fput = [&](int lvl, int k, int v) {
    if (k < FC)
      front[lvl][k] = v;
    else
      __hip_atomic_store(&spill[lvl * stride + (k - FC)], v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };
  int nf = 1, cur = 0, nleaf = 0;
  if (lane == 0) front[0][0] = 0;
  __syncthreads();
  bool ok = true;
  while (nf > 0) {
    int nn = 0;
    for (int base = 0; base < nf; base += kWave) {
      const int k = base + lane;
      const bool act = k < nf;
      WalkNode nd;
      bool open = false, inside = false;
      int id = 0;
      if (act) {
        id = fget(cur, k);
        nd = nodes[id];
        const double R = open_r(nd);
        open = box_gap2(nd, G, kp) < R * R;
        // an inner node wholly within the radius of every point of the group
        // box is taken whole, like a leaf, all of its leaves being opened
        inside = open && nd.nchild > 0 && box_far2(nd, G, kp) < R * R;
      }
      const bool leaf = open && (nd.nchild == 0 || inside);
      const bool inner = open && nd.nchild > 0 && !inside;
      const uint64_t lb = ballot64(leaf);
      const int nl = popc64(lb);
      if (nleaf + nl > kLCap) {
        flush(nleaf);
        nleaf = 0;
      }
      if (leaf) {
        const int pos = nleaf + popc64(lb & lanemask_lt());
        L.lfirst[pos] = nd.first;
        L.lcnt[pos] = nd.count;
        L.lnode[pos] = id;
      }
      nleaf += nl;
      const uint32_t nc = inner ? (uint32_t)nd.nchild : 0u;
      const uint32_t inc = wave_incl_scan_u32(nc);
      const uint32_t tot = __shfl(inc, kWave - 1, kWave);
      if (nn + (int)tot > cap) {
        ok = false;
      } else {
        const int o = nn + (int)(inc - nc);
        for (uint32_t q = 0; q < nc; ++q) fput(cur ^ 1, o + q, nd.child + (int)q);
        nn += (int)tot;
      }
      __syncthreads();
    }
    if (!ok) break;
    nf = nn;
    cur ^= 1;
  }
  if (nleaf > 0) flush(nleaf);
  return ok;
}

// The same leaf collection as group_walk, but over a list of leaves that a
// walk for an enclosing region already found (super-group walk): every listed
// leaf is tested against this group's box.
template <typename RadiusFn, typename FlushFn>
__device__ void list_walk(const WalkNode* __restrict__ nodes, const int* sl, int nsl,
                          const GroupInfo& G, const KParams& kp, WalkLds& L, RadiusFn open_r,
                          FlushFn flush) {
  const int lane = threadIdx.x;
  int nleaf = 0;
  for (int base = 0; base < nsl; base += kWave) {
    const int k = base + lane;
    WalkNode nd;
    bool open = false;
    if (k < nsl) {
      nd = nodes[sl[k]];
      const double R = open_r(nd);
      open = box_gap2(nd, G, kp) < R * R;
    }
    const uint64_t lb = ballot64(open);
    const int nl = popc64(lb);
    if (nleaf + nl > kLCap) {
      flush(nleaf);
      nleaf = 0;
    }
    if (open) {
      const int pos = nleaf + popc64(lb & lanemask_lt());
      L.lfirst[pos] = nd.first;
      L.lcnt[pos] = nd.count;
      L.lnode[pos] = sl[k];
    }
    nleaf += nl;
    __syncthreads();
  }
  if (nleaf > 0) flush(nleaf);
}

// Exclusive scan of the leaf counts into L.loff[0..nleaf].
__device__ __forceinline__ int leaf_offsets(WalkLds& L, int nleaf) {
  const int lane = threadIdx.x;
  uint32_t carry = 0;
  for (int base = 0; base < nleaf; base += kWave) {
    const int k = base + lane;
    const uint32_t v = (k < nleaf) ? (uint32_t)L.lcnt[k] : 0u;
    const uint32_t inc = wave_incl_scan_u32(v);
    if (k < nleaf) L.loff[k] = (int)(carry + inc - v);
    carry += __shfl(inc, kWave - 1, kWave);
  }
  if (lane == 0) L.loff[nleaf] = (int)carry;
  __syncthreads();
  return (int)carry;
}

// Stage candidates [c0, c0+cnt) of the flushed leaves into the LDS tile.
// Every lane resolves its candidates' particle indices first and then issues
// all their loads before storing any, so a whole tile costs about one
// memory latency instead of one per candidate step.
template <typename T, int N>
__device__ __forceinline__ void stage_tile(const WalkLds& L, int nleaf, int c0, int cnt,
                                           const double* __restrict__ px,
                                           const double* __restrict__ py,
                                           const double* __restrict__ pz,
                                           const double* __restrict__ pa, TileOf<T, N>& S,
                                           const GroupInfo& G, const KParams& kp) {
  constexpr int PER = N / kWave;
  const int lane = threadIdx.x;
  int jj[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int t = lane + q * kWave;
    jj[q] = -1;
    if (t < cnt) {
      const int c = c0 + t;
      int lo = 0, hi = nleaf;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (L.loff[mid] <= c)
          lo = mid;
        else
          hi = mid;
      }
      jj[q] = L.lfirst[lo] + (c - L.loff[lo]);
    }
  }
  double vx[PER], vy[PER], vz[PER], va[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int j = jj[q] >= 0 ? jj[q] : 0;
    vx[q] = px[j];
    vy[q] = py[j];
    vz[q] = pz[j];
    va[q] = pa[j];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int t = lane + q * kWave;
    if (jj[q] >= 0) {
      if constexpr (std::is_same<T, float>::value) {
        S.x[t] = (float)fold(vx[q] - G.c[0], kp.len[0], kp.half[0], kp.periodic[0]);
        S.y[t] = (float)fold(vy[q] - G.c[1], kp.len[1], kp.half[1], kp.periodic[1]);
        S.z[t] = (float)fold(vz[q] - G.c[2], kp.len[2], kp.half[2], kp.periodic[2]);
        S.a[t] = (float)va[q];
      } else {
        S.x[t] = vx[q];
        S.y[t] = vy[q];
        S.z[t] = vz[q];
        S.a[t] = va[q];
      }
      S.j[t] = jj[q];
    }
  }
  __syncthreads();
}

// Candidate loop over the flushed leaves, one staged tile at a time: lane
// `sub` of every slot visits tile entries sub, sub+LPI, ...;
// body(valid, c) is called by all lanes with c the tile index.
template <int LPI, typename T, int N, typename Body>
__device__ __forceinline__ void for_tiles(const WalkLds& L, int nleaf, int total, int sub,
                                          const double* __restrict__ px,
                                          const double* __restrict__ py,
                                          const double* __restrict__ pz,
                                          const double* __restrict__ pa, TileOf<T, N>& S,
                                          const GroupInfo& G, const KParams& kp, Body body) {
  for (int c0 = 0; c0 < total; c0 += N) {
    const int cnt = min(N, total - c0);
    stage_tile<T>(L, nleaf, c0, cnt, px, py, pz, pa, S, G, kp);
    for (int cb = 0; cb < cnt; cb += LPI) {
      const int c = cb + sub;
      body(c < cnt, c);
    }
    __syncthreads();
  }
}

// Load entries [b, b+nl) of a stored leaf list into the LDS leaf list.
__device__ __forceinline__ void load_leaves(WalkLds& L, const int2* __restrict__ pool, int off,
                                            int b, int nl) {
  for (int k = threadIdx.x; k < nl; k += kWave) {
    const int2 e = pool[off + b + k];
    L.lfirst[k] = e.x;
    L.lcnt[k] = e.y;
  }
  __syncthreads();
}

// ---- smoothing kernels of Sect. 2.3: W = C f(q) / h^3, q = r / h ----------
// M4 cubic spline (support 2, C = 1/pi), M6 quintic spline (support 3,
// C = 1/(120 pi)), Wendland C6 on the support H = 2h (C = 1365/(512 pi)).
// f(q) and f'(q); the kind is uniform over a launch.
template <typename T>
__device__ __forceinline__ void kern_f_df(int kind, T q, T& f, T& df) {
  if (kind == 1) {
    const T a = T(3) - q, b = T(2) - q, c = T(1) - q;
    const T t3 = a > T(0) ? a : T(0), t2 = b > T(0) ? b : T(0), t1 = c > T(0) ? c : T(0);
    const T s3 = t3 * t3, s2 = t2 * t2, s1 = t1 * t1;
    const T q3 = s3 * s3, q2 = s2 * s2, q1 = s1 * s1;  // fourth powers
    f = q3 * t3 - T(6) * q2 * t2 + T(15) * q1 * t1;
    df = T(-5) * q3 + T(30) * q2 - T(75) * q1;
  } else if (kind == 2) {
    const T u = T(1) - T(0.5) * q;
    const T s = u > T(0) ? u : T(0);
    const T s2 = s * s, s4 = s2 * s2, s7 = s4 * s2 * s;
    f = s7 * s * (((T(4) * q + T(6.25)) * q + T(4)) * q + T(1));
    df = T(-2.75) * q * ((T(8) * q + T(7)) * q + T(2)) * s7;
  } else {
    const T t = T(2) - q;
    const T tp = t > T(0) ? t : T(0);
    // inner branch (q < 1): 1 - 1.5 q^2 + 0.75 q^3 and -3q + 2.25 q^2
    const T fi = T(1) + q * q * (T(0.75) * q - T(1.5));
    const T dfi = q * (T(2.25) * q - T(3));
    // outer branch (1 <= q < 2): 0.25 (2-q)^3 and -0.75 (2-q)^2
    const T fo = T(0.25) * tp * tp * tp;
    const T dfo = T(-0.75) * tp * tp;
    const bool in = q < T(1);
    f = in ? fi : fo;
    df = in ? dfi : dfo;
  }
}

template <typename T>
__device__ __forceinline__ T kern_df(int kind, T q) {
  if (kind == 1) {
    const T a = T(3) - q, b = T(2) - q, c = T(1) - q;
    const T t3 = a > T(0) ? a : T(0), t2 = b > T(0) ? b : T(0), t1 = c > T(0) ? c : T(0);
    const T s3 = t3 * t3, s2 = t2 * t2, s1 = t1 * t1;
    return T(-5) * s3 * s3 + T(30) * s2 * s2 - T(75) * s1 * s1;
  }
  if (kind == 2) {
    const T u = T(1) - T(0.5) * q;
    const T s = u > T(0) ? u : T(0);
    const T s2 = s * s, s4 = s2 * s2;
    return T(-2.75) * q * ((T(8) * q + T(7)) * q + T(2)) * (s4 * s2 * s);
  }
  const T t = T(2) - q;
  const T tp = t > T(0) ? t : T(0);
  const T dfi = q * (T(2.25) * q - T(3));
  const T dfo = T(-0.75) * tp * tp;
  return q < T(1) ? dfi : dfo;
}

__device__ __forceinline__ float fast_sqrt(float v) { return __builtin_amdgcn_sqrtf(v); }
__device__ __forceinline__ float fast_rcp(float v) { return __builtin_amdgcn_rcpf(v); }

// The same shapes with the kind fixed at compile time (the list kernels are
// instantiated per kind, so their pair loops carry no branch on it) and the
// polynomials in fused multiply-adds.  M4 in one expression for both
// branches: f = t^3/4 - s^3, f' = 3 s^2 - 3 t^2/4, s = max(1-q, 0),
// t = max(2-q, 0).
template <int KIND, typename T>
__device__ __forceinline__ void kf_df(T q, T& f, T& df) {
  if constexpr (KIND == 1) {
    const T a = T(3) - q, b = T(2) - q, c = T(1) - q;
    const T t3 = a > T(0) ? a : T(0), t2 = b > T(0) ? b : T(0), t1 = c > T(0) ? c : T(0);
    const T s3 = t3 * t3, s2 = t2 * t2, s1 = t1 * t1;
    const T q3 = s3 * s3, q2 = s2 * s2, q1 = s1 * s1;  // fourth powers
    f = fma(T(15) * q1, t1, fma(T(-6) * q2, t2, q3 * t3));
    df = fma(T(-75), q1, fma(T(30), q2, T(-5) * q3));
  } else if constexpr (KIND == 2) {
    const T u = fma(T(-0.5), q, T(1));
    const T s = u > T(0) ? u : T(0);
    const T s2 = s * s, s4 = s2 * s2, s7 = s4 * s2 * s;
    f = (s7 * s) * fma(fma(fma(T(4), q, T(6.25)), q, T(4)), q, T(1));
    df = (T(-2.75) * q) * fma(fma(T(8), q, T(7)), q, T(2)) * s7;
  } else {
    const T a = T(2) - q, b = T(1) - q;
    const T t = a > T(0) ? a : T(0), s = b > T(0) ? b : T(0);
    const T t2 = t * t, s2 = s * s;
    f = fma(T(0.25) * t2, t, -(s2 * s));
    df = fma(T(3) * s, s, T(-0.75) * t2);
  }
}

template <int KIND, typename T>
__device__ __forceinline__ T kdf(T q) {
  if constexpr (KIND == 1) {
    const T a = T(3) - q, b = T(2) - q, c = T(1) - q;
    const T t3 = a > T(0) ? a : T(0), t2 = b > T(0) ? b : T(0), t1 = c > T(0) ? c : T(0);
    const T s3 = t3 * t3, s2 = t2 * t2, s1 = t1 * t1;
    return fma(T(-75) * s1, s1, fma(T(30) * s2, s2, T(-5) * s3 * s3));
  } else if constexpr (KIND == 2) {
    const T u = fma(T(-0.5), q, T(1));
    const T s = u > T(0) ? u : T(0);
    const T s2 = s * s, s4 = s2 * s2;
    return (T(-2.75) * q) * fma(fma(T(8), q, T(7)), q, T(2)) * (s4 * s2 * s);
  } else {
    const T a = T(2) - q, b = T(1) - q;
    const T t = a > T(0) ? a : T(0), s = b > T(0) ? b : T(0);
    return fma(T(3) * s, s, T(-0.75) * (t * t));
  }
}

// The exact FP64 pair predicate of both precisions: r^2 = fma(dz, dz,
// fma(dy, dy, dx dx)) of the nearest-image separation against
// (S max(h_i, h_j))^2 (force set, `force`) or (S h_i)^2 (density set).
__device__ __forceinline__ bool exact_pair(const KParams& kp, const double* __restrict__ x,
                                           const double* __restrict__ y,
                                           const double* __restrict__ z,
                                           const double* __restrict__ h, int i, int j,
                                           bool force) {
  const double dx = fold(x[i] - x[j], kp.len[0], kp.half[0], kp.periodic[0]);
  const double dy = fold(y[i] - y[j], kp.len[1], kp.half[1], kp.periodic[1]);
  const double dz = fold(z[i] - z[j], kp.len[2], kp.half[2], kp.periodic[2]);
  const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
  const double hi = h[i], hj = h[j];
  const double sr = kp.support * ((force && hj > hi) ? hj : hi);
  return r2 < sr * sr;
}

// The same, one axis at a time: a rare test inside a loop whose registers it
// must not raise.
__device__ __forceinline__ bool exact_pair_lean(const KParams& kp, const double* __restrict__ x,
                                                const double* __restrict__ y,
                                                const double* __restrict__ z,
                                                const double* __restrict__ h, int i, int j) {
  loaded(i);  // its addresses are not kept for the loop
  double r2;
  {
    const double d = fold(x[i] - x[j], kp.len[0], kp.half[0], kp.periodic[0]);
    r2 = d * d;
    loaded(r2);
  }
  {
    const double d = fold(y[i] - y[j], kp.len[1], kp.half[1], kp.periodic[1]);
    r2 = fma(d, d, r2);
    loaded(r2);
  }
  {
    const double d = fold(z[i] - z[j], kp.len[2], kp.half[2], kp.periodic[2]);
    r2 = fma(d, d, r2);
    loaded(r2);
  }
  const double hi = h[i], hj = h[j];
  const double sr = kp.support * (hj > hi ? hj : hi);
  return r2 < sr * sr;
}

// FP32 pair tests of the mixed mode lie within about 1e-6 (relative) of the
// FP64 ones; a test this close to the boundary is settled by exact_pair.
constexpr float kBorder = 4e-5f;

// ============================================================================
// Density: one wave per group (GS = 64/LPI particle slots of LPI lanes).
// Pair lists (r, m_j) for r < 2 h_i * margin are built once by the walk and
// kept in LDS while h is iterated; the walk is redone only if some h grows
// past its list radius.  Newton-Raphson on f(h) = S0(h) - m (hfact/h)^3 with
// a bracket; the group leaves the loop when a ballot shows every slot
// converged, after one more sum at the converged h.  A group whose lists
// would overflow sums on the fly during a walk at the current h instead.
// The first walk opens nodes with the force criterion widened by the margin
// and stores the group's leaf list, so that the force pass can replay it.
// ============================================================================

// This wavefront's set of counters.
__device__ __forceinline__ WaveTally& my_tally(DevState* ds) {
  return ds->tally[(blockIdx.x + gridDim.x * (threadIdx.x / kWave)) % kTallies];
}

// Courant minimum of a tally: the atomic is skipped when the stored value is
// already smaller (most wavefronts once the first ones have finished).
__device__ __forceinline__ void dt_min_update(WaveTally& t, double dm) {
  const unsigned long long e = enc_f64(dm);
  const unsigned long long cur =
      __hip_atomic_load(&t.dt_min_enc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (e < cur) atomicMin(&t.dt_min_enc, e);
}

// rho, Omega, P, c_s of particle i at its converged h (Sect. 2.2 and the
// ideal-gas closure), and the record the force loop reads for it (mixed: with
// the position codes qi, FP64: with the position); stored by the lane with
// `write`.
template <bool MIXED>
__device__ __forceinline__ void density_outputs(const KParams& kp, const Parts& p,
                                                void* __restrict__ frec_out, int i, double xi,
                                                double yi, double zi, const int4& qi, double mi,
                                                double h, double S0, double S1, double minhalf,
                                                uint32_t& err, bool write) {
  const double rho = S0;
  const double omega = 1.0 + h * S1 / (3.0 * rho);
  const double u = p.u[i];
  const double P = kp.gm1 * rho * u;
  const double cs = sqrt(kp.gamma * kp.gm1 * u);
  if (!(isfinite(rho) && isfinite(omega) && isfinite(P) && isfinite(cs))) err |= kErrNonFinite;
  if (kp.support * h >= minhalf) err |= kErrDomain;
  if (!write) return;
  p.h[i] = h;
  p.rho[i] = rho;
  p.omega[i] = omega;
  p.P[i] = P;
  p.cs[i] = cs;
  const double hinv = 1.0 / h;
  const double g = P / (rho * rho * omega);
  const double kk = 1.0 / (rho * omega);
  const double hinv4pi = hinv * hinv * hinv * hinv * kp.knorm;
  if constexpr (MIXED) {
    FRec32 r;
    r.qx = qi.x;
    r.qy = qi.y;
    r.qz = qi.z;
    r.m = (float)mi;
    r.h = (float)h;
    r.vx = (float)p.vx[i];
    r.vy = (float)p.vy[i];
    r.vz = (float)p.vz[i];
    r.u = (float)u;
    r.hinv = (float)hinv;
    r.hinv4pi = (float)hinv4pi;
    r.g = (float)g;
    r.k = (float)kk;
    r.c = (float)cs;
    r.P = (float)P;
    r.rho = (float)rho;
    reinterpret_cast<FRec32*>(frec_out)[i] = r;
  } else {
    FRec64 r;
    r.x = xi;
    r.y = yi;
    r.z = zi;
    r.m = mi;
    r.vx = p.vx[i];
    r.vy = p.vy[i];
    r.vz = p.vz[i];
    r.u = u;
    r.hinv = hinv;
    r.hinv4pi = hinv4pi;
    r.g = g;
    r.k = kk;
    r.c = cs;
    r.P = P;
    r.rho = rho;
    r.h = h;
    reinterpret_cast<FRec64*>(frec_out)[i] = r;
  }
}

// FB: only the groups of flag_list, which the neighbour-list kernels flagged,
// each with its own walk and without storing leaf lists.  A group's walks,
// staging and sums are serial chains of some 100 us, so what counts is how
// many wavefronts a CU holds: with a smaller frontier and tile in LDS (25 KB
// instead of 33 in FP64) and without the super-group code, six instead of
// four (3157 flagged groups of 30,011 particles: 369 -> 231 us).
template <bool MIXED, int LPI, bool FB>
__global__ __launch_bounds__(64) void k_density(KParams kp, Parts p,
                                                const WalkNode* __restrict__ nodes,
                                                const GroupInfo* __restrict__ groups,
                                                void* __restrict__ frec_out,
                                                int2* __restrict__ pool, int64_t pool_cap,
                                                int32_t* __restrict__ gl_off,
                                                int32_t* __restrict__ gl_cnt,
                                                const int32_t* __restrict__ flag_list,
                                                int32_t* __restrict__ walk_spill,
    DevState* __restrict__ ds) {
  // FB: half the wavefronts, each with twice the spill
  int* __restrict__ spill = walk_spill + (int64_t)blockIdx.x * (FB ? 4 : 2) * kSpill;
  using R = typename std::conditional<MIXED, float, double>::type;
  constexpr int GS = kWave / LPI;
  // (known only at run time in the form for all groups, which otherwise is laid
  // out 3 % slower: 3312 against 3192 us at 24^3, groups of 16, Wendland C6)
  const bool fb = FB || flag_list != nullptr;
  if (FB && ds->n_flagged == 0) return;
  __shared__ WalkLds L;
  __shared__ int s_front[2][FB ? kFCapFb : kFCap];
  __shared__ TileOf<R, FB ? kTileFb : kTile> T;
  __shared__ R s_r[kPMax * GS];
  __shared__ R s_m[kPMax * GS];
  __shared__ int s_sl[FB ? 1 : kSLCap];  // leaves found by the super-group walk

  const int lane = threadIdx.x;
  const int slot = lane / LPI, sub = lane % LPI;
  const int ng = ds->n_groups;
  // waves take super-groups of kSG consecutive groups; each XCD a contiguous
  // range of them, so that neighbouring groups share that XCD's L2
  // flagged groups are spread one per wavefront (they are few, and heavy)
  // (striped over all wavefronts of all XCDs)
  const int sgs = fb ? 1 : kSG;
  const int nsg = fb ? ds->n_flagged : (ng + sgs - 1) / sgs;
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;
  const int chunk = (nsg + 7) >> 3;
  const int sbeg = fb ? (int)blockIdx.x : xcd * chunk;
  const int send = fb ? nsg : min(sbeg + chunk, nsg);
  const int sstep = fb ? (int)gridDim.x : nloc;
  const double margin = kp.h_margin;
  double minhalf = SPH_INF;
  for (int a = 0; a < 3; ++a)
    if (kp.periodic[a]) minhalf = fmin(minhalf, kp.half[a]);
  // this wave's region of the leaf-list pool
  const int64_t rsize = pool_cap / gridDim.x;
  const int64_t rbase = (int64_t)blockIdx.x * rsize;
  int64_t rpos = 0;

  uint32_t err = 0;
  int it_max = 0;
  unsigned long long pairs_final = 0, sums = 0, cands = 0;
  int walks = 0;
  bool grew = false;

  for (int sg = fb ? sbeg : sbeg + local; sg < send; sg += sstep) {
   const int g0 = fb ? flag_list[sg] : sg * sgs, g1 = fb ? g0 + 1 : min(g0 + sgs, ng);
   // ---- super-group box (union of the group boxes) and largest start h
   GroupInfo SG;
   {
     const bool v = !fb && lane < g1 - g0;
     GroupInfo Gk;
     if (v) Gk = groups[g0 + lane];
     for (int a = 0; a < 3; ++a) {
       const double lo = wave_min_f64(v ? Gk.c[a] - Gk.w[a] : SPH_INF);
       const double hi = wave_max_f64(v ? Gk.c[a] + Gk.w[a] : -SPH_INF);
       SG.c[a] = 0.5 * (lo + hi);
       SG.w[a] = fmax(hi - SG.c[a], SG.c[a] - lo);
     }
     SG.hmax = wave_max_f64(v ? Gk.hmax : 0.0);
     SG.first = 0;
     SG.count = 0;
   }
   // ---- one walk for the super-group: every leaf any of its groups can need
   int nsl = 0;
   bool sok = true;
   {
     const double hs = margin * SG.hmax;
     auto sradius = [&](const WalkNode& nd) {
       return kp.support * fmax(hs, margin * (double)nd.hmax) * (1.0 + 4e-9);
     };
     auto sflush = [&](int nleaf) {
       if (nsl + nleaf <= kSLCap) {
         for (int q = lane; q < nleaf; q += kWave) s_sl[nsl + q] = L.lnode[q];
       } else {
         sok = false;
       }
       nsl += nleaf;
       __syncthreads();
     };
     if (fb) {
       sok = false;  // flagged groups walk on their own
     } else {
       if (!group_walk(nodes, SG, kp, L, s_front, spill, sradius, sflush)) sok = false;
       ++walks;
     }
   }
   for (int g = g0; g < g1; ++g) {
    if (fb && lane == 0) gl_cnt[g] = -1;  // its force pass walks
    const GroupInfo G = groups[g];
    const bool act = slot < G.count;
    const int i = G.first + (act ? slot : 0);
    const double xi = p.x[i], yi = p.y[i], zi = p.z[i], mi = p.m[i];
    double h = p.h[i];
    if (!(h > 0.0) || !isfinite(h)) {
      err |= kErrNonFinite;
      h = 1.0;
    }
    const double h0 = h;
    float xr = 0.f, yr = 0.f, zr = 0.f;  // FP32 path: position relative to the group centre
    if constexpr (MIXED) {
      xr = (float)fold(xi - G.c[0], kp.len[0], kp.half[0], kp.periodic[0]);
      yr = (float)fold(yi - G.c[1], kp.len[1], kp.half[1], kp.periodic[1]);
      zr = (float)fold(zi - G.c[2], kp.len[2], kp.half[2], kp.periodic[2]);
    }
    double hlim = h * margin;
    double hlo = 0.0, hhi = SPH_INF;
    bool conv = !act;
    bool need = true;
    bool store = !fb;  // the first walk stores the leaf list
    const int64_t gstart = rpos;
    bool gover = false;
    int npair = 0;
    int nit = 0;
    double S0 = 0.0, S1 = 0.0;
    uint32_t nnb = 0;
    bool failed = false;
    bool stream = false;  // group-wide: a pair list overflowed, sum on the fly instead
    while (true) {
      if (!stream && ballot64(act && need) != 0ull) {
        // ---- walk and fill the pair lists (r < 2 hlim_i)
        const double hm = wave_max_f64(act ? hlim : 0.0);
        const double rl = kp.support * hlim, rl2 = rl * rl;
        const float rl2f = (float)rl2 * 1.00001f;
        npair = 0;
        auto radius = [&](const WalkNode& nd) {
          const double r = store ? fmax(hm, margin * (double)nd.hmax) : hm;
          return kp.support * r * (1.0 + 4e-9);
        };
        auto flush = [&](int nleaf) {
          const int total = leaf_offsets(L, nleaf);
          if (store) {
            if (!gover && rpos + nleaf <= rsize) {
              for (int k = lane; k < nleaf; k += kWave)
                pool[rbase + rpos + k] = make_int2(L.lfirst[k], L.lcnt[k]);
              rpos += nleaf;
            } else {
              gover = true;
            }
          }
          cands += (unsigned long long)total * ((act && sub == 0) ? 1u : 0u);
          for_tiles<LPI, R>(L, nleaf, total, sub, p.x, p.y, p.z, p.m, T, G, kp,
                            [&](bool valid, int c) {
            bool pred = false;
            R rv = R(0), mj = R(0);
            if (valid && act) {
              if constexpr (MIXED) {
                const float dx = xr - T.x[c], dy = yr - T.y[c], dz = zr - T.z[c];
                const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                pred = r2 < rl2f;
                rv = fast_sqrt(r2);
              } else {
                const double dx = fold(xi - T.x[c], kp.len[0], kp.half[0], kp.periodic[0]);
                const double dy = fold(yi - T.y[c], kp.len[1], kp.half[1], kp.periodic[1]);
                const double dz = fold(zi - T.z[c], kp.len[2], kp.half[2], kp.periodic[2]);
                const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
                pred = r2 < rl2;
                if (pred) rv = sqrt(r2);
              }
              mj = T.a[c];
            }
            const uint64_t b = ballot64(pred);
            const uint32_t seg = (uint32_t)((b >> (slot * LPI)) & ((LPI == 64) ? ~0ull : ((1ull << LPI) - 1ull)));
            const int pos = npair + __popc(seg & ((1u << sub) - 1u));
            if (pred && pos < kPMax) {
              s_r[pos * GS + slot] = rv;
              s_m[pos * GS + slot] = mj;
            }
            npair += __popc(seg);
          });
          __syncthreads();
        };
        bool wok;
        if (!fb && store && sok)
          wok = true, list_walk(nodes, s_sl, nsl, G, kp, L, radius, flush);
        else
          wok = group_walk(nodes, G, kp, L, s_front, spill, radius, flush);
        if (!wok) {
          err |= kErrFrontier;
          failed = true;
        }
        if (store) {
          if (lane == 0) {
            gl_off[g] = (int32_t)(rbase + gstart);
            gl_cnt[g] = (gover || failed) ? -1 : (int32_t)(rpos - gstart);
            if (gover || failed) atomicOr(&ds->lists_missing, 1);
          }
          store = false;
        }
        if (ballot64(failed) != 0ull) {
          failed = true;
          break;
        }
        if (ballot64(npair > kPMax) != 0ull) stream = true;
        need = false;
        ++walks;
      }
      // ---- one density sum at the current h
      const double hinv = 1.0 / h;
      double a0 = 0.0, a1 = 0.0;
      uint32_t cnt = 0;
      if (stream) {
        // walk at the current h and accumulate the candidates directly
        const double Rg = kp.support * wave_max_f64(act ? h : 0.0) * (1.0 + 4e-9);
        const double twoh = kp.support * h, rl2 = twoh * twoh;
        const float rl2f = (float)rl2;
        const float hinvf = (float)hinv;
        auto radius = [&](const WalkNode&) { return Rg; };
        auto flush = [&](int nleaf) {
          const int total = leaf_offsets(L, nleaf);
          for_tiles<LPI, R>(L, nleaf, total, sub, p.x, p.y, p.z, p.m, T, G, kp,
                            [&](bool valid, int c) {
            if (valid && act) {
              if constexpr (MIXED) {
                const float dx = xr - T.x[c], dy = yr - T.y[c], dz = zr - T.z[c];
                const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                if (r2 < rl2f) {
                  const float m = T.a[c];
                  const float q = fast_sqrt(r2) * hinvf;
                  float f, df;
                  kern_f_df<float>(kp.kernel, q, f, df);
                  a0 += (double)(m * f);
                  a1 += (double)(m * (3.0f * f + q * df));
                  ++cnt;
                }
              } else {
                const double dx = fold(xi - T.x[c], kp.len[0], kp.half[0], kp.periodic[0]);
                const double dy = fold(yi - T.y[c], kp.len[1], kp.half[1], kp.periodic[1]);
                const double dz = fold(zi - T.z[c], kp.len[2], kp.half[2], kp.periodic[2]);
                const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
                if (r2 < rl2) {
                  const double mj = T.a[c];
                  const double q = sqrt(r2) * hinv;
                  double f, df;
                  kern_f_df<double>(kp.kernel, q, f, df);
                  a0 += mj * f;
                  a1 += mj * (3.0 * f + q * df);
                  ++cnt;
                }
              }
            }
          });
          __syncthreads();
        };
        if (!group_walk(nodes, G, kp, L, s_front, spill, radius, flush)) {
          err |= kErrFrontier;
          failed = true;
        }
        if (ballot64(failed) != 0ull) {
          failed = true;
          break;
        }
        ++walks;
      } else if (MIXED) {
        // each lane sums its few terms in FP32; lanes are combined in FP64
        const float hinvf = (float)hinv;
        const float twohf = (float)(kp.support * h);
        float s0 = 0.f, s1 = 0.f;
        for (int k = sub; k < npair; k += LPI) {
          const float r = (float)s_r[k * GS + slot], m = (float)s_m[k * GS + slot];
          const float q = r * hinvf;
          float f, df;
          kern_f_df<float>(kp.kernel, q, f, df);
          s0 = fmaf(m, f, s0);
          s1 = fmaf(m, fmaf(q, df, 3.0f * f), s1);
          cnt += (r < twohf) ? 1u : 0u;
        }
        a0 = (double)s0;
        a1 = (double)s1;
      } else {
        const double twoh = kp.support * h;
        for (int k = sub; k < npair; k += LPI) {
          const double r = (double)s_r[k * GS + slot], m = (double)s_m[k * GS + slot];
          const double q = r * hinv;
          double f, df;
          kern_f_df<double>(kp.kernel, q, f, df);
          a0 += m * f;
          a1 += m * (3.0 * f + q * df);
          cnt += (r < twoh) ? 1u : 0u;
        }
      }
      a0 = seg_sum<LPI>(a0);
      a1 = seg_sum<LPI>(a1);
      cnt = seg_sum_u32<LPI>(cnt);
      const double h3 = hinv * hinv * hinv;
      S0 = a0 * h3 * kp.knorm;
      S1 = -a1 * h3 * hinv * kp.knorm;
      nnb = cnt;
      sums += (act && sub == 0) ? (unsigned long long)cnt : 0ull;
      // ---- decide: a slot is done when the h-rho relation holds at its
      // current h to the tolerance (then S0, S1 above are its final sums);
      // otherwise it takes a safeguarded Newton step and is summed again
      bool moved = false;
      if (!conv) {
        const double t = kp.hfact * hinv;
        const double rh = mi * (t * t * t);
        const double f = S0 - rh;
        const double fp = S1 + 3.0 * rh * hinv;
        double hn = h;
        if (kp.fixed_passes) {
          hn = h - f / fp;
          if (!(fp > 0.0))
            hn = h;
          else if (hn > 1.2 * h)
            hn = 1.2 * h;
          else if (hn < 0.8 * h)
            hn = 0.8 * h;
          // three density computations (Sect. 3.2.1): two updates, then
          // rho and Omega from the third sum at the h it used
          conv = (nit + 1) >= 2;
          moved = true;
        } else if (fabs(f) <= 3.0 * kp.h_tol * rh) {
          // |f| / f' <= tol h (f' = 3 rho_h Omega / h): converged at this h
          conv = true;
        } else {
          if (f < 0.0)
            hlo = fmax(hlo, h);
          else
            hhi = fmin(hhi, h);
          hn = h - f / fp;
          const bool bad = !(fp > 0.0) || !(hn >= 0.8 * h) || !(hn <= 1.2 * h) ||
                           !(hn > hlo) || !(hn < hhi);
          if (bad) {
            if (hlo > 0.0 && hhi < SPH_INF)
              hn = 0.5 * (hlo + hhi);
            else
              hn = (f < 0.0) ? 1.2 * h : h / 1.2;
          }
          // a step at the rounding level of h: sum once more there and stop
          conv = fabs(hn - h) <= 4e-16 * h;
          moved = true;
        }
        if (moved) {
          h = hn;
          if (h > hlim) {
            hlim = h * margin;
            need = true;
          }
          ++nit;
          if (nit > kp.max_iter) {
            err |= kErrNoConv;
            conv = true;
          }
        }
      }
      if (ballot64(!conv || moved) == 0ull) break;  // every slot summed at its final h
    }
    it_max = max(it_max, nit + 1);
    if (act && !failed && h > h0 * margin) grew = true;
    if (act && !failed) {
      int4 qi = make_int4(0, 0, 0, 0);
      if constexpr (MIXED) {
        const QFrame& f = ds->qf;
        qi.x = qcode(xi, f, 0, kp.periodic[0]);
        qi.y = qcode(yi, f, 1, kp.periodic[1]);
        qi.z = qcode(zi, f, 2, kp.periodic[2]);
      }
      density_outputs<MIXED>(kp, p, frec_out, i, xi, yi, zi, qi, mi, h, S0, S1, minhalf, err,
                             sub == 0);
      if (sub == 0) {
        pairs_final += nnb;
      }
    }
   }
  }
  // one set of atomics per wave
  const bool ballot_any = ballot64(grew) != 0ull;
  const uint64_t b = ballot64(err != 0);
  uint32_t eall = err;
  for (int d = 32; d > 0; d >>= 1) eall |= __shfl_xor(eall, d, kWave);
  unsigned long long pf = pairs_final;
  for (int d = 32; d > 0; d >>= 1) pf += __shfl_xor(pf, d, kWave);
  unsigned long long cd = cands, sm = sums;
  for (int d = 32; d > 0; d >>= 1) {
    cd += __shfl_xor(cd, d, kWave);
    sm += __shfl_xor(sm, d, kWave);
  }
  sums = sm;
  if (lane == 0) {
    WaveTally& tally = my_tally(ds);
    if (b) atomicOr(&ds->err, eall);
    if (it_max > 0) atomicMax(&tally.max_iter, it_max);
    if (pf) atomicAdd(&tally.n_pairs_density, pf);
    if (sums) atomicAdd(&tally.n_sums_density, sums);
    if (sums && !fb) atomicAdd(&tally.tot_sums_density, sums);
    if (cd) atomicAdd(&tally.n_cand_density, cd);
    if (walks) atomicAdd(&tally.n_rewalk, walks);
    if (ballot_any) atomicMax(&ds->leaf_state, 2);
  }
}

// ============================================================================
// Force: one wave per group.  The walk opens a node if the group box comes
// within 2 max(h_max,group, h_max,node) of it; candidates j != i with
// r < 2 max(h_i, h_j) go to a per-slot LDS list of indices; the pair loop
// then reads each neighbour's record.
// ============================================================================
template <bool MIXED>
struct FRecOf {
  using T = FRec64;
};
template <>
struct FRecOf<true> {
  using T = FRec32;
};

template <bool MIXED, int LPI>
__global__ __launch_bounds__(64) void k_force(KParams kp, Parts p,
                                              const WalkNode* __restrict__ nodes,
                                              const GroupInfo* __restrict__ groups,
                                              const void* __restrict__ frec_in,
                                              const int2* __restrict__ pool,
                                              const int32_t* __restrict__ gl_off,
                                              const int32_t* __restrict__ gl_cnt,
                                              double* __restrict__ out_ax,
                                              double* __restrict__ out_ay,
                                              double* __restrict__ out_az,
                                              double* __restrict__ out_du,
                                              const int32_t* __restrict__ flag_list,
                                              int32_t* __restrict__ walk_spill,
    DevState* __restrict__ ds) {
  int* __restrict__ spill = walk_spill + (int64_t)blockIdx.x * 2 * kSpill;
  using Rec = typename FRecOf<MIXED>::T;
  using R = typename std::conditional<MIXED, float, double>::type;
  constexpr int GS = kWave / LPI;
  __shared__ WalkLds L;
  __shared__ int s_front[2][kFCap];
  __shared__ TileOf<R> T;
  __shared__ int s_j[kPMax * GS];
  const bool use_lists = ds->leaf_state == 1;
  const Rec* __restrict__ rec = reinterpret_cast<const Rec*>(frec_in);

  const int lane = threadIdx.x;
  const int slot = lane / LPI, sub = lane % LPI;
  const int ng = ds->n_groups;
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;
  const int chunk = (ng + 7) >> 3;
  const int gbeg = xcd * chunk, gend = min(gbeg + chunk, ng);
  uint32_t err = 0;
  unsigned long long pairs = 0, cands = 0;
  double dtmin = SPH_INF;

  // flag_list != nullptr while the neighbour lists hold every pair (leaf_state
  // 1): the list kernel does the unflagged groups, and the few flagged ones
  // are striped over all wavefronts
  const bool only_flagged = flag_list != nullptr && use_lists;
  if (only_flagged && ds->n_flagged == 0) return;
  const int g_first = only_flagged ? (int)blockIdx.x : gbeg + local;
  const int g_end = only_flagged ? ds->n_flagged : gend;
  const int g_step = only_flagged ? (int)gridDim.x : nloc;
  for (int gk = g_first; gk < g_end; gk += g_step) {
    const int g = only_flagged ? flag_list[gk] : gk;
    const GroupInfo G = groups[g];
    const bool act = slot < G.count;
    const int i = G.first + (act ? slot : 0);
    const double xi = p.x[i], yi = p.y[i], zi = p.z[i], hi = p.h[i];
    const Rec ri = rec[i];
    float xr = 0.f, yr = 0.f, zr = 0.f;  // FP32 path: position relative to the group centre
    const float hif = (float)hi;
    if constexpr (MIXED) {
      xr = (float)fold(xi - G.c[0], kp.len[0], kp.half[0], kp.periodic[0]);
      yr = (float)fold(yi - G.c[1], kp.len[1], kp.half[1], kp.periodic[1]);
      zr = (float)fold(zi - G.c[2], kp.len[2], kp.half[2], kp.periodic[2]);
    }
    double ax = 0.0, ay = 0.0, az = 0.0, du = 0.0, vmax = 0.0;
    int npair = 0;
    // ---- pair loop over the pending list entries of each slot
    auto compute = [&]() {
      if constexpr (MIXED) {
        const float al = (float)kp.alpha, be = (float)kp.beta, au = (float)kp.alpha_u;
        const float vxi = ri.vx, vyi = ri.vy, vzi = ri.vz;
        const float hinvi = ri.hinv, h4i = ri.hinv4pi, gi = ri.g, ki = ri.k, ci = ri.c;
        const float Pi = ri.P, rhoi = ri.rho, ui = ri.u;
        const float qsx = ds->qf.step[0], qsy = ds->qf.step[1], qsz = ds->qf.step[2];
        auto pair = [&](const Rec& rj) {
          const float dx = qsep(ri.qx, rj.qx, qsx);
          const float dy = qsep(ri.qy, rj.qy, qsy);
          const float dz = qsep(ri.qz, rj.qz, qsz);
          const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
          const float rinv = __builtin_amdgcn_rsqf(r2);
          const float r = r2 * rinv;
          const float ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
          const float w = fmaf(vzi - rj.vz, ez, fmaf(vyi - rj.vy, ey, (vxi - rj.vx) * ex));
          const float Fi = kern_df<float>(kp.kernel, r * hinvi) * h4i;
          const float Fj = kern_df<float>(kp.kernel, r * rj.hinv) * rj.hinv4pi;
          const float aw = fabsf(w);
          const bool app = w < 0.0f;
          const float vsi = fmaf(be, aw, al * ci);
          const float vsj = fmaf(be, aw, al * rj.c);
          const float ti = app ? fmaf(-0.5f * vsi * w, ki, gi) : gi;
          const float tj = app ? fmaf(-0.5f * vsj * w, rj.k, rj.g) : rj.g;
          const float pa = rj.m * fmaf(ti, Fi, tj * Fj);
          ax -= (double)(pa * ex);
          ay -= (double)(pa * ey);
          az -= (double)(pa * ez);
          const float mwF = rj.m * w * Fi;
          float e = gi * mwF;
          if (app) e = fmaf(-0.5f * ki * vsi * w, mwF, e);
          const float dP = fabsf(Pi - rj.P);
          const float vu = fast_sqrt(dP * fast_rcp(0.5f * (rhoi + rj.rho)));
          e = fmaf(rj.m * au * vu * (ui - rj.u), 0.5f * fmaf(Fi, ki, Fj * rj.k), e);
          du += (double)e;
          vmax = fmax(vmax, (double)vsi);
        };
        for (int k = sub; k < npair; k += 2 * LPI) {
          const int k2 = k + LPI;
          const bool two = k2 < npair;
          const int j1 = s_j[k * GS + slot];
          const int j2 = two ? s_j[k2 * GS + slot] : j1;
          const Rec r1 = rec[j1];
          const Rec r2 = rec[j2];
          pair(r1);
          if (two) pair(r2);
        }
      } else {
        const double al = kp.alpha, be = kp.beta, au = kp.alpha_u;
        const double vxi = ri.vx, vyi = ri.vy, vzi = ri.vz;
        const double hinvi = ri.hinv, h4i = ri.hinv4pi, gi = ri.g, ki = ri.k, ci = ri.c;
        const double Pi = ri.P, rhoi = ri.rho, ui = ri.u;
        auto pair = [&](const Rec& rj) {
          const double dx = fold(xi - rj.x, kp.len[0], kp.half[0], kp.periodic[0]);
          const double dy = fold(yi - rj.y, kp.len[1], kp.half[1], kp.periodic[1]);
          const double dz = fold(zi - rj.z, kp.len[2], kp.half[2], kp.periodic[2]);
          const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
          const double r = sqrt(r2);
          const double rinv = 1.0 / r;
          const double ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
          const double w = fma(vzi - rj.vz, ez, fma(vyi - rj.vy, ey, (vxi - rj.vx) * ex));
          const double Fi = kern_df<double>(kp.kernel, r * hinvi) * h4i;
          const double Fj = kern_df<double>(kp.kernel, r * rj.hinv) * rj.hinv4pi;
          const double aw = fabs(w);
          const bool app = w < 0.0;
          const double vsi = fma(be, aw, al * ci);
          const double vsj = fma(be, aw, al * rj.c);
          const double ti = app ? fma(-0.5 * vsi * w, ki, gi) : gi;
          const double tj = app ? fma(-0.5 * vsj * w, rj.k, rj.g) : rj.g;
          const double pa = rj.m * fma(ti, Fi, tj * Fj);
          ax -= pa * ex;
          ay -= pa * ey;
          az -= pa * ez;
          const double mwF = rj.m * w * Fi;
          double e = gi * mwF;
          if (app) e = fma(-0.5 * ki * vsi * w, mwF, e);
          const double vu = sqrt(fabs(Pi - rj.P) / (0.5 * (rhoi + rj.rho)));
          e = fma(rj.m * au * vu * (ui - rj.u), 0.5 * fma(Fi, ki, Fj * rj.k), e);
          du += e;
          vmax = fmax(vmax, vsi);
        };
        for (int k = sub; k < npair; k += 2 * LPI) {
          const int k2 = k + LPI;
          const bool two = k2 < npair;
          const int j1 = s_j[k * GS + slot];
          const int j2 = two ? s_j[k2 * GS + slot] : j1;
          const Rec r1 = rec[j1];
          const Rec r2 = rec[j2];
          pair(r1);
          if (two) pair(r2);
        }
      }
      pairs += (act && sub == 0) ? (unsigned long long)npair : 0ull;
      npair = 0;
    };
    const double hg = G.hmax;
    auto radius = [&](const WalkNode& nd) {
      return kp.support * fmax(hg, (double)nd.hmax) * (1.0 + 4e-9);
    };
    auto flush = [&](int nleaf) {
      const int total = leaf_offsets(L, nleaf);
      cands += (unsigned long long)total * ((act && sub == 0) ? 1u : 0u);
      for_tiles<LPI, R>(L, nleaf, total, sub, p.x, p.y, p.z, p.h, T, G, kp,
                        [&](bool valid, int c) {
        // one candidate step adds at most LPI entries per slot: empty the
        // lists through the pair loop before they can overflow
        if (ballot64(npair > kPMax - LPI) != 0ull) {
          __syncthreads();
          compute();
          __syncthreads();
        }
        bool pred = false;
        const int j = valid ? T.j[c] : -1;
        if (valid && act && j != i) {
          if constexpr (MIXED) {
            const float dx = xr - T.x[c], dy = yr - T.y[c], dz = zr - T.z[c];
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const float hj = T.a[c];
            const float sr = (float)kp.support * fmaxf(hif, hj);
            pred = r2 < sr * sr * 1.00001f;
          } else {
            const double dx = fold(xi - T.x[c], kp.len[0], kp.half[0], kp.periodic[0]);
            const double dy = fold(yi - T.y[c], kp.len[1], kp.half[1], kp.periodic[1]);
            const double dz = fold(zi - T.z[c], kp.len[2], kp.half[2], kp.periodic[2]);
            const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
            const double hj = T.a[c];
            const double sr = kp.support * (hi > hj ? hi : hj);
            pred = r2 < sr * sr;
          }
        }
        const uint64_t b = ballot64(pred);
        const uint32_t seg = (uint32_t)((b >> (slot * LPI)) & ((LPI == 64) ? ~0ull : ((1ull << LPI) - 1ull)));
        const int pos = npair + __popc(seg & ((1u << sub) - 1u));
        if (pred) s_j[pos * GS + slot] = j;
        npair += __popc(seg);
      });
      __syncthreads();
    };
    const int lcount = use_lists ? gl_cnt[g] : -1;
    if (lcount >= 0) {
      // replay the leaf list the density walk stored for this group
      const int off = gl_off[g];
      for (int b = 0; b < lcount; b += kLCap) {
        const int nl = min(kLCap, lcount - b);
        load_leaves(L, pool, off, b, nl);
        flush(nl);
      }
    } else if (!group_walk(nodes, G, kp, L, s_front, spill, radius, flush)) {
      err |= kErrFrontierForce;
    }
    __syncthreads();
    compute();
    ax = seg_sum<LPI>(ax);
    ay = seg_sum<LPI>(ay);
    az = seg_sum<LPI>(az);
    du = seg_sum<LPI>(du);
    vmax = seg_max<LPI>(vmax);
    if (act) {
      const double v0 = (kp.alpha == 0.0) ? (double)ri.c : kp.alpha * (double)ri.c;
      const double vs = fmax(vmax, v0);
      if (!(isfinite(ax) && isfinite(ay) && isfinite(az) && isfinite(du))) err |= kErrNonFinite;
      if (sub == 0) {
        out_ax[i] = ax;
        out_ay[i] = ay;
        out_az[i] = az;
        out_du[i] = du;
        p.vsig[i] = vs;
      }
      dtmin = fmin(dtmin, kp.c_cour * hi / vs);
    }
  }
  const uint64_t b = ballot64(err != 0);
  uint32_t eall = err;
  for (int d = 32; d > 0; d >>= 1) eall |= __shfl_xor(eall, d, kWave);
  unsigned long long pf = pairs, cd = cands;
  for (int d = 32; d > 0; d >>= 1) {
    pf += __shfl_xor(pf, d, kWave);
    cd += __shfl_xor(cd, d, kWave);
  }
  const double dm = wave_min_f64(dtmin);
  if (lane == 0) {
    WaveTally& tally = my_tally(ds);
    if (b) atomicOr(&ds->err, eall);
    if (pf) atomicAdd(&tally.n_pairs_force, pf);
    if (pf && flag_list == nullptr) atomicAdd(&tally.tot_pairs_force, pf);
    if (cd) atomicAdd(&tally.n_cand_force, cd);
    if (dm < SPH_INF) dt_min_update(tally, dm);
  }
}

// Groups of this wave under the XCD-aware static schedule: block b works on
// the contiguous eighth of the groups that belongs to XCD b mod 8.
struct GroupRange {
  int beg, end, step;
};
__device__ __forceinline__ GroupRange xcd_groups(int ng) {
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;
  const int chunk = (ng + 7) >> 3;
  const int gbeg = xcd * chunk;
  return GroupRange{gbeg + local, min(gbeg + chunk, ng), nloc};
}

// The same for blocks of WPB wavefronts, which take WPB consecutive items at a
// time: what their neighbourhoods share then stays in the CU's L1.
template <int WPB>
__device__ __forceinline__ GroupRange xcd_items(int n) {
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;
  const int chunk = (((n + 7) >> 3) + WPB - 1) / WPB * WPB;
  const int beg = xcd * chunk;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  return GroupRange{beg + local * WPB + wave, min(beg + chunk, n), nloc * WPB};
}

// ============================================================================
// Neighbour lists (Sect. 3.2), in two kernels.
//
// k_leaves: one wavefront per super-group of kSGL consecutive groups (aligned
// runs of the curve, hence compact) walks the tree once for all of them and
// writes every leaf that any of the groups can need to the super-group's leaf
// list, with one bit per group whose box and radius reach the leaf.  The walk
// starts from all nodes of levels 0 to 2 (at most 73) at once.  A super-group
// whose list or frontier overflows lets each of its groups walk on its own,
// into a list from the pool.
//
// k_rows: one wavefront per group takes the leaves that carry its bit, loads
// their particles, one candidate per lane, and for each of its particles i in
// turn appends the indices j of every candidate with
//     r_ij < S max(hl_i, hl_j),   hl = h_margin * (h at the start),
// to the fixed-capacity row i of nl_idx (self included): one ballot and one
// coalesced store per particle and 64 candidates, in candidate order (leaves
// by level, then along the curve).  As long as no h grows past its hl, a row
// is a superset of the density neighbours (r < S h_i) and of the force pairs
// (r < S max(h_i, h_j)); the density and force list kernels apply the exact
// predicates.  A group with an overflowing row or a failed walk is flagged
// (gflag = 1) and left to the walking kernels.  The group of every particle is
// kept (grp_of) for the list kernels, which work on chunks of consecutive
// particles instead of groups.
//
// Why two kernels: the walk is a chain of dependent loads (one level after
// another) and the row tests are VALU work; in one kernel the frontier, the
// leaf lists and the candidate tiles of both took 8.5 KB of LDS and 121
// registers per wavefront, and its 4 wavefronts per SIMD kept the VALU half
// idle.  k_leaves is bound by its loads' latency, k_rows by VALU and scalar
// issue.  One kernel -> k_leaves + k_rows: 16.8M mixed 11.2 -> 2.2 + 5.7 ms,
// 10^6 mixed 819 -> 150 + 316 us, 10^6 FP64 1322 -> 150 + 456, 294,912 mixed
// 176 -> 61 + 70, 32^3 FP64 65 -> 20 + 19 us.
// ============================================================================
constexpr int kSGLShift = 3;
constexpr int kSGL = 1 << kSGLShift;  // groups per super-group of the list kernels
constexpr int kSLCapL = 512;  // leaves a list-kernel walk may collect (trees of small leaves: more)
constexpr int kLeafPart = 64; // particles per leaf-list entry at most (>= the largest n_leaf)
constexpr int kRowWaves = 8;  // wavefronts per SIMD of k_rows
constexpr int kNoLeaves = -0x7fffffff;  // ll_cnt of a group whose walk failed

// The value a wave-uniform lane `l` holds, as a wave-uniform scalar.
__device__ __forceinline__ float lane_val(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Whether this lane's bit of a wave-uniform mask is set.
__device__ __forceinline__ bool lane_in(uint64_t m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

// Largest value of each aligned run of 8 lanes.
__device__ __forceinline__ float seg_max8(float v) {
  v = fmaxf(v, __uint_as_float(xor_lane_u32<4>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(xor_lane_u32<2>(__float_as_uint(v))));
  return fmaxf(v, __uint_as_float(xor_lane_u32<1>(__float_as_uint(v))));
}

// base + the number of set bits of m below this lane (mbcnt: two VALU ops)
__device__ __forceinline__ int rank_below(uint64_t m, int base) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
}

// Squared search radius (support * x)^2 of the list predicate with the slack
// of its FP32 test: 1e-5 relative, and 2e-6 w (support * x) for offsets that
// were rounded to FP32 at a distance of up to w (0 for position codes) beyond
// the radius from the group's centre.  Every step rounds monotonically, so
// the value at max(a, b) is the larger of the values at a and at b: the pair
// test compares r^2 with the larger of the particle's and the candidate's.
__device__ __forceinline__ float list_thr(float support, float x, float w) {
  const float s = support * x;
  return fmaf(2e-6f * w, s, s * s * 1.00001f);
}

// The FP32 tests of the list kernels take lengths times 2^e, e from a group's
// (or part's) own radius r: exact, so it changes no test, but the squares then
// neither overflow nor vanish in any unit of length (unscaled, radii beyond
// 1.8e19 or below 1e-22 lost neighbours).  e is 0 for r in 2^-32 .. 2^32, where
// FP32 holds the squares as they are, and otherwise brings r to 1 .. 2.
__device__ __forceinline__ int list_exponent(double r) {
  if (!(r > 0.0) || !isfinite(r)) return 0;
  const int e = -ilogb(r);
  return __builtin_amdgcn_readfirstlane(abs(e) <= 32 ? 0 : min(max(e, -1000), 1000));
}

// Groups per unit of k_leaves (its log2): kSGL, or fewer on sets too small to
// give every fourth wavefront a unit of that size.
__device__ __forceinline__ int unit_shift(int ng, int nwaves) {
  int u = kSGLShift;
  while (u > 0 && (ng >> u) < nwaves / 4) --u;
  return u;
}
// Entries of a unit's leaf list: an equal share of the list space, at most
// kSLCapL of them, or as many more as the space grows for small leaves.
__device__ __forceinline__ int leaf_list_cap(int64_t entries, int nu, int n_leaf) {
  return (int)min((int64_t)kSLCapL * leaf_list_factor(n_leaf), entries / max(nu, 1));
}

// Separation of a node's centre from c along the nearest periodic image, and
// the squared gap between the node's box and the box (c, w).
__device__ __forceinline__ double node_gap2(const WalkNode& nd, const double (&c)[3],
                                            const double (&w)[3], const KParams& kp,
                                            double (&dc)[3]) {
  double d2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double d = nd.c[a] - c[a];
    if (kp.periodic[a]) d = d - kp.len[a] * rint(d * kp.inv_len[a]);
    dc[a] = d;
    double gap = fabs(d) - (double)nd.w[a] - w[a];
    gap = gap > 0.0 ? gap : 0.0;
    d2 = d2 + gap * gap;
  }
  return d2;
}

// Breadth-first walk for the region within S max(hl, margin h_max(node)) of
// the box (c, w): visit(leaf, node, dc) is called by all lanes for every batch
// of up to 64 nodes, with leaf set in the lanes that hold an opened leaf, and
// ends the walk by returning false.  A level's frontier holds kFCap entries in
// LDS and continues in this wavefront's region of global memory (kSpill
// entries per level).  Returns false if the walk ended early or its frontier
// overflowed.
template <typename Visit>
__device__ __forceinline__ bool leaf_walk(const WalkNode* __restrict__ nodes, int n01, int n012,
                                          const double (&c)[3], const double (&w)[3], double hl,
                                          const KParams& kp, int (&front)[2][kFCap],
                                          int* __restrict__ spill, Visit visit) {
  const int lane = threadIdx.x;
  constexpr int cap = kFCap + kSpill;
  auto fget = [&](int lvl, int k) -> int {
    return k < kFCap ? front[lvl][k]
                     : __hip_atomic_load(&spill[lvl * kSpill + (k - kFCap)], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
  };
  auto fput = [&](int lvl, int k, int v) {
    if (k < kFCap)
      front[lvl][k] = v;
    else
      __hip_atomic_store(&spill[lvl * kSpill + (k - kFCap)], v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };
  // the first frontier: nodes 0 .. n012 - 1, of which the first n01 (levels 0
  // and 1) have their children in it already
  for (int k = lane; k < n012; k += kWave) front[0][k] = k;
  int nf = n012, cur = 0, no_push = n01;
  __syncthreads();
  while (nf > 0) {
    int nn = 0;
    for (int base = 0; base < nf; base += kWave) {
      const int k = base + lane;
      WalkNode nd;
      nd.nchild = 0;
      bool open = false;
      int id = 0;
      double dc[3] = {0.0, 0.0, 0.0};
      if (k < nf) {
        id = fget(cur, k);
        nd = nodes[id];
        const double R =
            kp.support * fmax(hl, kp.h_margin * (double)nd.hmax) * (1.0 + 4e-9);
        open = node_gap2(nd, c, w, kp, dc) < R * R;
      }
      if (!visit(open && nd.nchild == 0, nd, dc)) return false;
      const uint32_t nc = open && id >= no_push ? (uint32_t)nd.nchild : 0u;
      const uint32_t inc = wave_incl_scan_u32(nc);
      const int tot = __builtin_amdgcn_readlane((int)inc, kWave - 1);
      if (nn + tot > cap) return false;
      const int o = nn + (int)(inc - nc);
      for (uint32_t q = 0; q < nc; ++q) fput(cur ^ 1, o + (int)q, nd.child + (int)q);
      nn += tot;
      __syncthreads();
    }
    nf = nn;
    cur ^= 1;
    no_push = 0;
  }
  return true;
}

// sg_list: the units' leaf lists, `sg_entries` entries in all; entry: (first
// particle, particle count | group bits << 24), of at most kLeafPart
// particles (a level-21 leaf of more takes several).  pool: lists of groups
// that walked on their own; entry: (first particle, particle count).  Per group:
// ll_off, ll_cnt = its list's first entry and length (>= 0) in sg_list, or
// ll_cnt = ~length (< 0) in the pool, or kNoLeaves.
//
// A unit's groups are walked together unless they lie apart: where the curve
// jumps between two of them by more than their two search regions (an octant
// boundary of a high level), or where their list overflows, the run is cut,
// and the parts walk one after the other.  (Walked whole, such a unit's box
// spans the domain: its walk alone took 150 us at 294,912 particles, longer
// than all others together.)
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kLeafWaves)))
void k_leaves(KParams kp, const WalkNode* __restrict__ nodes,
              const GroupInfo* __restrict__ groups, const uint32_t* __restrict__ level_off,
              int nblk, int2* __restrict__ sg_list, int64_t sg_entries, int2* __restrict__ pool,
              int pool_cap, int32_t* __restrict__ ll_off, int32_t* __restrict__ ll_cnt,
              int32_t* __restrict__ gflag, int32_t* __restrict__ walk_spill, DevState* __restrict__ ds) {
  int* __restrict__ spill = walk_spill + (int64_t)blockIdx.x * 2 * kSpill;
  __shared__ int front[2][kFCap];
  __shared__ float4 s_g[kSGL][2];  // per group: box centre from the part's, h_l; half-widths
  const int lane = threadIdx.x;
  const int ng = ds->n_groups;
  const int ush = unit_shift(ng, (int)gridDim.x), usz = 1 << ush;
  const int nu = (ng + usz - 1) >> ush;
  const int cap = leaf_list_cap(sg_entries, nu, kp.n_leaf);
  const int n01 = (int)level_off[2 * nblk], n012 = (int)level_off[3 * nblk];
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;
  const int chunk = (nu + 7) >> 3;
  const int uend = min((xcd + 1) * chunk, nu);
  const float S = (float)kp.support, margin = (float)kp.h_margin;
  int walks = 0;

  for (int u = xcd * chunk + local; u < uend; u += nloc) {
    const int g0 = u * usz, ngs = min(usz, ng - g0);
    const bool isg = lane < ngs;
    const int glane = g0 + (isg ? lane : 0);
    if (isg) gflag[glane] = 0;
    // bit k: the search regions of groups k - 1 and k do not meet
    uint64_t jumps;
    {
      const GroupInfo Gk = groups[glane];
      const double reach = kp.support * kp.h_margin * Gk.hmax;
      const double before = __shfl_up(reach, 1, kWave);
      bool apart = false;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double cb = __shfl_up(Gk.c[a], 1, kWave), wb = __shfl_up(Gk.w[a], 1, kWave);
        apart |= fabs(Gk.c[a] - cb) - Gk.w[a] - wb > reach + before;
      }
      jumps = ballot64(apart && isg && lane > 0);
    }
    const int64_t base = (int64_t)u * cap;
    int used = 0;  // entries of the unit's space written so far
    for (int a0 = 0; a0 < ngs;) {
      const uint64_t ahead = jumps & (~0ull << (a0 + 1));
      int a1 = ahead ? min(__builtin_ctzll(ahead), ngs) : ngs;
      // The part [a0, a1) into the unit's list, halved until it fits (kUnit);
      // a single group that still does not fit counts its leaves (kCount) and
      // then writes them to space taken from the pool (kPool); more than
      // 512 leaves (1024 small ones) make it a case for the walking kernels: at
      // 24^3 particles, one per leaf and Wendland C6, some groups reach 690.
      enum { kUnit, kCount, kPool };
      int mode = kUnit, off = 0, room = cap - used;
      int2* __restrict__ list = sg_list + base + used;
      while (true) {
        const bool in = lane >= a0 && lane < a1;
        const GroupInfo Gk = groups[glane];
        double c[3], w[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double lo = wave_min_f64(in ? Gk.c[a] - Gk.w[a] : SPH_INF);
          const double hi = wave_max_f64(in ? Gk.c[a] + Gk.w[a] : -SPH_INF);
          c[a] = 0.5 * (lo + hi);
          w[a] = fmax(hi - c[a], c[a] - lo);
        }
        const double hl = kp.h_margin * wave_max_f64(in ? Gk.hmax : 0.0);
        const int se = list_exponent(hl);  // of the FP32 lengths below
        __syncthreads();
        if (in) {
          // FP32 offsets from the part's centre
          s_g[lane][0] = make_float4((float)ldexp(Gk.c[0] - c[0], se),
                                     (float)ldexp(Gk.c[1] - c[1], se),
                                     (float)ldexp(Gk.c[2] - c[2], se),
                                     (float)ldexp(kp.h_margin * Gk.hmax, se));
          s_g[lane][1] = make_float4((float)ldexp(Gk.w[0], se), (float)ldexp(Gk.w[1], se),
                                     (float)ldexp(Gk.w[2], se), 0.f);
        }
        // bound of the FP32 offsets' rounding within the part's reach
        const float eps =
            (float)ldexp(1e-6 * (fmax(w[0], fmax(w[1], w[2])) + kp.support * hl), se);
        __syncthreads();
        int n = 0;
        const bool fits =
            leaf_walk(nodes, n01, n012, c, w, hl, kp, front, spill,
                      [&](bool leaf, const WalkNode& nd, const double (&dc)[3]) {
          if (ballot64(leaf) == 0ull) return true;
          uint32_t bits = 0;
          if (mode == kUnit) {
            // FP32 on offsets from the part's centre, settled in FP64 within
            // its rounding of the boundary, and near half a periodic length,
            // where a group's nearest image may be another than the part's:
            // the leaves a group takes, and so the rows, do not depend on the
            // part it walks with
            bool amb = false;
#pragma unroll
            for (int a = 0; a < 3; ++a) amb |= kp.periodic[a] && fabs(dc[a]) + w[a] > kp.half[a];
            const float x = (float)ldexp(dc[0], se), y = (float)ldexp(dc[1], se),
                        z = (float)ldexp(dc[2], se);
            const float nwx = ldexpf(nd.w[0], se), nwy = ldexpf(nd.w[1], se),
                        nwz = ldexpf(nd.w[2], se), nh = margin * ldexpf(nd.hmax, se);
            const float e4 = 4.f * fmaf(1e-6f, fmaxf(nwx, fmaxf(nwy, nwz)), eps);
            uint32_t border = 0;
            for (int gk = a0; gk < a1; ++gk) {
              const float4 gc = s_g[gk][0], gw = s_g[gk][1];
              const float dx = fmaxf(fabsf(x - gc.x) - (nwx + gw.x), 0.f);
              const float dy = fmaxf(fabsf(y - gc.y) - (nwy + gw.y), 0.f);
              const float dz = fmaxf(fabsf(z - gc.z) - (nwz + gw.z), 0.f);
              const float R = S * fmaxf(gc.w, nh);
              const float t = fmaf(dz, dz, fmaf(dy, dy, dx * dx)) - R * R;
              const float tol = R * fmaf(4e-5f, R, e4);
              bits |= t < 0.f ? 1u << (24 + gk) : 0u;
              border |= fabsf(t) <= tol ? 1u << gk : 0u;
            }
            if (amb) border = (1u << a1) - (1u << a0);
            if (!leaf) border = 0u;
            while (ballot64(border != 0u) != 0ull) {
              if (border != 0u) {
                const int gk = __builtin_ctz(border);
                const GroupInfo G = groups[g0 + gk];
                const double rg = kp.support *
                                  fmax(kp.h_margin * G.hmax, kp.h_margin * (double)nd.hmax) *
                                  (1.0 + 4e-9);
                bits &= ~(1u << (24 + gk));
                if (box_gap2(nd, G, kp) < rg * rg) bits |= 1u << (24 + gk);
                border &= border - 1u;
              }
            }
            leaf = leaf && bits != 0u;
          }
          const uint64_t lb = ballot64(leaf);
          if (ballot64(leaf && nd.count > kLeafPart) == 0ull) {
            const int pos = rank_below(lb, n);
            if (leaf && pos < room && mode != kCount)
              list[pos] = make_int2(nd.first, (int)((uint32_t)nd.count | bits));
            n += popc64(lb);
          } else {  // leaves of coincident keys, in parts
            const uint32_t np = leaf ? (uint32_t)((nd.count + kLeafPart - 1) / kLeafPart) : 0u;
            const uint32_t inc = wave_incl_scan_u32(np);
            int pos = n + (int)(inc - np);
            if (mode != kCount)
              for (int f = 0; f < (int)np * kLeafPart && pos < room; f += kLeafPart, ++pos)
                list[pos] = make_int2(
                    nd.first + f, (int)((uint32_t)min(kLeafPart, nd.count - f) | bits));
            n += __builtin_amdgcn_readlane((int)inc, kWave - 1);
          }
          return n <= room;
        });
        ++walks;
        if (mode == kCount && fits) {
          // not past a full pool, so that the counter cannot wrap round
          if (lane == 0) {
            const int taken =
                __hip_atomic_load(&ds->pool_used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            off = (uint32_t)taken < (uint32_t)pool_cap ? atomicAdd(&ds->pool_used, n) : -1;
          }
          off = __builtin_amdgcn_readfirstlane(off);
          if (off >= 0 && off <= pool_cap - n) {
            list = pool + off;
            room = n;
            mode = kPool;
            continue;
          }
        } else if (mode == kUnit && !fits) {
          if (a1 - a0 > 1) {
            a1 = a0 + (a1 - a0) / 2;
          } else {
            mode = kCount;
            room = kp.n_leaf < 8 ? 2 * kSLCapL : kSLCapL;
          }
          continue;
        }
        if (in) {
          ll_off[glane] = mode == kUnit ? used : off;
          ll_cnt[glane] = mode == kUnit ? n : mode == kPool && fits ? ~n : kNoLeaves;
        }
        if (mode == kUnit) used += n;
        break;
      }
      a0 = a1;
    }
    __syncthreads();  // s_g and the frontier are refilled next
  }
  if (lane == 0 && walks) atomicAdd(&my_tally(ds).n_rewalk, walks);
}

// Candidates of a group are first tested against its box (with the largest
// radius of its particles); those that pass are packed in LDS, and every 128 of
// them meet the group's particles.  (Leaves bring in about twice the
// candidates that lie within reach of the group.)  2^psh wavefronts share a
// group, each with its share of the particles, where there are fewer groups
// than wavefronts.
template <bool MIXED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kRowWaves)))
void k_rows(KParams kp, const double* __restrict__ hp, const WalkNode* __restrict__ nodes,
            const GroupInfo* __restrict__ groups, const int2* __restrict__ sg_list,
            int64_t sg_entries, int leaf_grid, const int2* __restrict__ pool,
            const int32_t* __restrict__ ll_off, const int32_t* __restrict__ ll_cnt,
            int32_t* __restrict__ nl_idx, int32_t* __restrict__ nl_len,
            int32_t* __restrict__ gflag, int32_t* __restrict__ flag_list,
            int32_t* __restrict__ grp_of, const int4* __restrict__ qrec,
            const double4* __restrict__ xyzm, DevState* __restrict__ ds) {
  constexpr int PT = 2;                   // sets of 64 packed candidates per test
  constexpr int NPK = (PT + 1) * kWave;   // fewer than PT sets wait when the next is packed
  constexpr int NM = kWave * kLeafPart / kWave;
  __shared__ float4 s_c[NPK];  // packed candidates: offset from the centre, squared radius
  __shared__ int s_j[NPK];
  __shared__ int s_j0[kWave];  // first particle of each selected leaf less its first candidate
  __shared__ unsigned long long s_start[NM];  // bit c: a leaf's candidates start at c
  const int lane = threadIdx.x;
  const int ng = ds->n_groups;
  const int ush = unit_shift(ng, leaf_grid);
  const int ucap = leaf_list_cap(sg_entries, (ng + (1 << ush) - 1) >> ush, kp.n_leaf);
  int psh = 0;
  while (psh < 2 && (ng << (psh + 1)) <= (int)gridDim.x) ++psh;
  const GroupRange gr = xcd_groups(ng << psh);
  const float S = (float)kp.support, marginf = (float)kp.h_margin;
  const int cap = kp.nl_cap;
  const float stx = ds->qf.step[0], sty = ds->qf.step[1], stz = ds->qf.step[2];
  // reach bounds the list radius of every pair
  const double reach =
      kp.support * kp.h_margin * (ds->n_nodes > 0 ? (double)nodes[0].hmax : 0.0) * (1.0 + 1e-4);
  int nflag = 0;
  unsigned long long cands = 0;

  for (int it = gr.beg; it < gr.end; it += gr.step) {
    const int g = it >> psh, part = it & ((1 << psh) - 1);
    const double gcx = groups[g].c[0], gcy = groups[g].c[1], gcz = groups[g].c[2];
    const double gwx = groups[g].w[0], gwy = groups[g].w[1], gwz = groups[g].w[2];
    const int gcount = groups[g].count;
    // this wavefront's particles of the group
    const int s0 = (gcount * part) >> psh, cnt = ((gcount * (part + 1)) >> psh) - s0;
    const int gfirst = groups[g].first + s0;
    const int nl = ll_cnt[g];
    const bool own = nl < 0;
    const bool gok = nl != kNoLeaves;
    const int nlist = !gok ? 0 : own ? ~nl : nl;
    const int2* __restrict__ list =
        own ? pool + ll_off[g] : sg_list + ((int64_t)(g >> ush) * ucap + ll_off[g]);
    const uint32_t mybit = own ? ~0u : 1u << (24 + (g & ((1 << ush) - 1)));
    const uint32_t cmask = own ? ~0u : 0xffffffu;
    // Positions relative to the group's centre along the nearest image: code
    // differences in the tree's fixed-point frame (mixed), or rounded FP64
    // differences.  A pair's difference of offsets is then the pair's nearest
    // image whenever it lies within reach, unless the group's half-width and
    // the reach together come to half a periodic length on some axis (tiny
    // periodic boxes): that group folds every pair separation instead.
    const bool farx = kp.periodic[0] && gwx + reach >= kp.half[0];
    const bool fary = kp.periodic[1] && gwy + reach >= kp.half[1];
    const bool farz = kp.periodic[2] && gwz + reach >= kp.half[2];
    const bool amb = farx || fary || farz;
    // FP64: the lengths' power of two in the FP32 tests, and the distance at
    // which offsets may have been rounded
    int se = 0;
    float wr = 0.f;
    int32_t qgx = 0, qgy = 0, qgz = 0;
    if constexpr (MIXED) {
      const QFrame& qf = ds->qf;
      qgx = qcode(gcx, qf, 0, kp.periodic[0]);
      qgy = qcode(gcy, qf, 1, kp.periodic[1]);
      qgz = qcode(gcz, qf, 2, kp.periodic[2]);
    } else {
      se = list_exponent(groups[g].hmax);
      wr = (float)ldexp(fmax(gwx + (farx ? kp.len[0] : 0.0),
                             fmax(gwy + (fary ? kp.len[1] : 0.0), gwz + (farz ? kp.len[2] : 0.0))),
                        se);
    }
    // a particle as the tests take it: its offset and its squared radius
    struct Raw {
      int4 q;     // mixed
      double4 d;  // FP64
      double h;
    };
    auto load = [&](int j) {
      Raw r;
      if constexpr (MIXED) {
        r.q = qrec[j];
      } else {
        r.d = xyzm[j];
        r.h = hp[j];
      }
      return r;
    };
    auto offsets = [&](const Raw& r) {
      float4 c;
      if constexpr (MIXED) {
        c.x = qsep(r.q.x, qgx, stx);
        c.y = qsep(r.q.y, qgy, sty);
        c.z = qsep(r.q.z, qgz, stz);
        c.w = list_thr(S, marginf * __int_as_float(r.q.w), 0.f);
      } else {
        double dx = fold(r.d.x - gcx, kp.len[0], kp.half[0], kp.periodic[0]);
        double dy = fold(r.d.y - gcy, kp.len[1], kp.half[1], kp.periodic[1]);
        double dz = fold(r.d.z - gcz, kp.len[2], kp.half[2], kp.periodic[2]);
        double hl = kp.h_margin * r.h;
        if (__builtin_expect(se != 0, 0)) {
          dx = ldexp(dx, se);
          dy = ldexp(dy, se);
          dz = ldexp(dz, se);
          hl = ldexp(hl, se);
        }
        c.x = (float)dx;
        c.y = (float)dy;
        c.z = (float)dz;
        c.w = list_thr(S, (float)hl, wr);
      }
      return c;
    };
    // one particle per lane, read as scalars by the tests; the next entry of
    // its row, counted from the first particle's row
    const int pi = gfirst + (lane < cnt ? lane : 0);
    float4 me = offsets(load(pi));
    if constexpr (MIXED) me.w = list_thr(S, (float)(kp.h_margin * hp[pi]), 0.f);
    int npv = lane * cap;
    int32_t* __restrict__ rows = nl_idx + (int64_t)gfirst * cap;
    // the box of the particles about the group's centre with its test's own
    // rounding, and their largest squared radius (lanes 0 to 7 hold them all)
    float bx = seg_max8(fabsf(me.x)), by = seg_max8(fabsf(me.y)), bz = seg_max8(fabsf(me.z));
    float tmax = seg_max8(me.w);
    {
      const float e = 1e-6f * (bx + by + bz + fast_sqrt(tmax));
      bx = lane_val(bx + e, 0);
      by = lane_val(by + e, 0);
      bz = lane_val(bz + e, 0);
      tmax = amb ? (float)SPH_INF : lane_val(tmax, 0);  // folded pairs: no box test
    }
    int npk = 0;  // packed candidates waiting

    // the first PT sets of 64 packed candidates (or what is left of them)
    // against the particles: every particle's row gets the hits in order
    auto test = [&]() {
      float4 c[PT];
      int j[PT];
      uint64_t vm[PT];  // lanes that hold a candidate
#pragma unroll
      for (int q = 0; q < PT; ++q) {
        c[q] = s_c[q * kWave + lane];
        j[q] = s_j[q * kWave + lane];
        const int left = npk - q * kWave;
        vm[q] = left >= kWave ? ~0ull : left > 0 ? ~0ull >> (kWave - left) : 0ull;
      }
      auto pairs = [&](auto fold_pairs) {
        constexpr bool FOLD = decltype(fold_pairs)::value;
        int end = 0;  // of the particle's row
        for (int s = 0; s < cnt; ++s) {
          const float px = lane_val(me.x, s), py = lane_val(me.y, s), pz = lane_val(me.z, s);
          const float pt = lane_val(me.w, s);
          int n = __builtin_amdgcn_readlane(npv, s);
          end += cap;
#pragma unroll
          for (int q = 0; q < PT; ++q) {
            if (q > 0 && vm[q] == 0ull) break;
            float dx = px - c[q].x, dy = py - c[q].y, dz = pz - c[q].z;
            if constexpr (FOLD) {
              auto nearest = [&](float d, int a) {
                return kp.periodic[a] ? fmaf(-(float)ldexp(kp.len[a], se),
                                             rintf(d * (float)ldexp(kp.inv_len[a], -se)), d)
                                      : d;
              };
              dx = nearest(dx, 0);
              dy = nearest(dy, 1);
              dz = nearest(dz, 2);
            }
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            // r2 and the radii are >= 0: their bit patterns order like their
            // values (an integer max needs no NaN care)
            const uint64_t b =
                ballot64(__float_as_int(r2) < max(__float_as_int(pt), __float_as_int(c[q].w))) &
                vm[q];
            const int pos = rank_below(b, n);
            const uint64_t st = b & ballot64(pos < end);
            if (lane_in(st))
              *reinterpret_cast<int*>(reinterpret_cast<char*>(rows) + ((unsigned)pos << 2)) = j[q];
            n += popc64(b);
          }
          npv = lane_in(1ull << s) ? n : npv;
        }
      };
      if (amb)
        pairs(std::true_type{});
      else
        pairs(std::false_type{});
    };

    // 64 leaves at a time: those with this group's bit, their first candidate
    // in s_j0 and s_start; then their candidates, 64 at a time
    for (int base = 0; base < nlist || npk > 0; base += kWave) {
      int total = 0;
      if (base < nlist) {
        const int k = base + lane;
        const int2 e = list[min(k, nlist - 1)];
        const bool open = k < nlist && ((uint32_t)e.y & mybit) != 0u;
        const uint32_t c = open ? (uint32_t)e.y & cmask : 0u;
        const uint32_t inc = wave_incl_scan_u32(c);
        total = __builtin_amdgcn_readlane((int)inc, kWave - 1);
        __syncthreads();
        for (int m = lane; m * kWave < total; m += kWave) s_start[m] = 0ull;
        __syncthreads();
        if (open) {
          const int o = (int)(inc - c);
          s_j0[rank_below(ballot64(open), 0)] = e.x - o;
          atomicOr(&s_start[o >> 6], 1ull << (o & 63));
        }
        __syncthreads();
        if (part == 0) cands += (unsigned long long)total * (unsigned)gcount;
      }
      // leaves hold at least one particle each, so the leaf of candidate c is
      // the number of starts at or before c, less one
      int lt = -1;  // leaf of the candidate before the set
      for (int c0 = 0; c0 < total; c0 += kWave) {
        const unsigned long long starts = s_start[c0 >> 6];
        const uint64_t st =
            (uint64_t)__builtin_amdgcn_readfirstlane((int)starts) & 0xffffffffull |
            (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(starts >> 32)) << 32;
        const int left = total - c0;
        const uint64_t vm = left >= kWave ? ~0ull : ~0ull >> (kWave - left);
        const int lo = rank_below(st, lt) + (lane_in(st) ? 1 : 0);
        lt += popc64(st);
        const int j = lane_in(vm) ? s_j0[lo] + c0 + lane : gfirst;
        const float4 c = offsets(load(j));
        const float dx = fmaxf(fabsf(c.x) - bx, 0.f), dy = fmaxf(fabsf(c.y) - by, 0.f),
                    dz = fmaxf(fabsf(c.z) - bz, 0.f);
        const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        const uint64_t near =
            ballot64(__float_as_int(d2) < max(__float_as_int(tmax), __float_as_int(c.w))) & vm;
        if (lane_in(near)) {
          const int pos = rank_below(near, npk);
          s_c[pos] = c;
          s_j[pos] = j;
        }
        npk += popc64(near);
        __syncthreads();
        if (npk >= PT * kWave) {
          test();
          const float4 rc = s_c[PT * kWave + lane];  // the rest moves to the front
          const int rj = s_j[PT * kWave + lane];
          __syncthreads();
          s_c[lane] = rc;
          s_j[lane] = rj;
          npk -= PT * kWave;
          __syncthreads();
        }
      }
      if (base + kWave >= nlist && npk > 0) {
        test();
        npk = 0;
      }
    }
    const int len = npv - lane * cap;
    const bool bad = !gok || ballot64(lane < cnt && len > cap) != 0ull;
    if (lane < cnt) {
      nl_len[pi] = len;
      grp_of[pi] = g;
    }
    if (bad && lane == 0 && atomicCAS(&gflag[g], 0, 1) == 0) {
      flag_list[atomicAdd(&ds->n_flagged, 1)] = g;
      ++nflag;
    }
    __syncthreads();  // the packed candidates are refilled next
  }
  if (lane == 0) {
    WaveTally& tally = my_tally(ds);
    if (cands) atomicAdd(&tally.n_cand_density, cands);
    if (cands) atomicAdd(&tally.tot_cand_lists, cands);
    if (nflag) {
      atomicOr(&ds->lists_missing, 1);
      atomicAdd(&ds->n_flag_rows, nflag);
    }
  }
}

// ============================================================================
// Density from the neighbour lists (Sect. 2.2, Sect. 3.2.1): one wavefront
// per chunk, LPI lanes per particle.  Each lane gathers the separations and
// masses of its share of the row once (registers), then the h iteration
// re-sums them: Newton-Raphson on f(h) = S0(h) - m (hfact/h)^3 with the same
// safeguards as the walking kernel, a wavefront ballot deciding when the
// group is done.  A group in which some h passes hl (its rows may then miss
// neighbours) is flagged (gflag = 2) for the walking kernel, and the force
// pass then walks for every group (leaf_state 2).
//
// Bound by VALU issue and the gather's latency.  The entries sit in
// registers (E separations and E masses per lane): in LDS, where they were
// before, they cost two LDS reads and their addressing per pair sum and held
// FP64 rows of 256 entries to 1.25 wavefronts per SIMD.  Kernel time before
// and after: FP64 Wendland C6 294,912 particles 859 -> 395 us, mixed M6
// 294,912 292 -> 216 us, FP64 M4 10^6 945 -> 654 us, mixed M4 16.8M 6657 ->
// 5907 us.
// ============================================================================
// Wavefronts per SIMD the list density kernel is compiled for.
constexpr int density_waves(bool mixed, int entries) { return mixed ? (entries > 16 ? 3 : 4) : (entries > 16 ? 2 : 3); }

template <bool MIXED, int LPI, int CAP, int KIND>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(density_waves(MIXED, CAP / LPI))))
void k_density_lists(KParams kp, Parts p,
                                                      const GroupInfo* __restrict__ groups,
                                                      const int32_t* __restrict__ nl_idx,
                                                      const int32_t* __restrict__ nl_len,
                                                      int32_t* __restrict__ gflag,
                                                      int32_t* __restrict__ flag_list,
                                                      const int32_t* __restrict__ grp_of,
                                                      const void* __restrict__ pos,
                                                      void* __restrict__ frec_out,
                                                      DevState* __restrict__ ds) {
  using R = typename std::conditional<MIXED, float, double>::type;
  constexpr int E = CAP / LPI;  // row entries per lane (CAP = kp.nl_cap)
  constexpr int B = 4;          // entries per lane gathered and summed at a time
  static_assert(E % B == 0, "whole blocks of entries");
  const int lane = threadIdx.x;
  const int slot = lane / LPI, sub = lane % LPI;
  constexpr int CS = kWave / LPI;  // particles per chunk
  const int nch = (kp.n + CS - 1) / CS;
  const GroupRange gr = xcd_groups(nch);
  const double margin = kp.h_margin;
  double minhalf = SPH_INF;
  for (int a = 0; a < 3; ++a)
    if (kp.periodic[a]) minhalf = fmin(minhalf, kp.half[a]);
  uint32_t err = 0;
  int it_max = 0;
  unsigned long long pairs_final = 0, sums = 0;
  bool outgrew_any = false;
  int ngrew = 0;
  // gathered per row entry: x, y, z, m (FP64), or position codes and m (mixed)
  const double4* __restrict__ xyzm = reinterpret_cast<const double4*>(pos);
  const int4* __restrict__ qpos = reinterpret_cast<const int4*>(pos);
  const float qsx = ds->qf.step[0], qsy = ds->qf.step[1], qsz = ds->qf.step[2];

  // groups the list kernel flagged (1) are left to the walking kernel; their
  // flags are looked up only if there are any.  Those that this kernel flags
  // (2) are not looked at: whether one is seen in time would depend on the
  // order of the wavefronts, and with it where the walking kernel's iteration
  // starts and what it counts.
  const bool any_flag = ds->n_flag_rows != 0;

  for (int g = gr.beg; g < gr.end; g += gr.step) {
    const int first = g * CS, count = min(CS, kp.n - first);
    const bool inr = slot < count;
    const int i = first + (inr ? slot : 0);
    const bool act = inr && (!any_flag || gflag[grp_of[i]] != 1);
    if (any_flag && ballot64(act) == 0ull) continue;
    const double mi = p.m[i];
    double h = p.h[i];
    int len = nl_len[i];
    loaded(len);
    len = act ? len : 0;
    int4 qi = make_int4(0, 0, 0, 0);  // mixed: i's position codes
    double xi = 0.0, yi = 0.0, zi = 0.0;
    if constexpr (MIXED) {
      qi = qpos[i];
    } else {
      xi = p.x[i];
      yi = p.y[i];
      zi = p.z[i];
    }
    if (!(h > 0.0) || !isfinite(h)) {
      err |= kErrNonFinite;
      h = 1.0;
    }
    const double hl = margin * h;
    const int lmax = __builtin_amdgcn_readfirstlane(wave_max_i32(len));
    // ---- gather: separation and mass of every row entry into registers (a
    // lane reads no entry but its own), four entries per lane at a time (their
    // loads in flight together).  Entries past the row's end get a separation
    // beyond the support of any h up to hl and no mass: they add exactly zero.
    // Blocks past the chunk's longest row are neither loaded nor summed.
    // Short mixed rows keep the raw records of all their blocks in flight; the
    // others reduce a block to its separations before the next one is loaded
    // (the records would not fit the registers).
    const int32_t* __restrict__ row = nl_idx + ((int64_t)i * CAP + sub);
    R er[E], em[E];
    const R rpad = (R)(4.0 * hl);
    int iself = i;  // in place of entries past the row's end
    loaded(iself);
#pragma unroll
    for (int t0 = 0; t0 < E; t0 += B) {
      if (t0 * LPI >= lmax) break;
      int jj[B];
#pragma unroll
      for (int q = 0; q < B; ++q) jj[q] = row[LPI * (t0 + q)];  // within the row's CAP entries
#pragma unroll
      for (int q = 0; q < B; ++q) {
        loaded(jj[q]);
        jj[q] = sub + LPI * (t0 + q) < len ? jj[q] : iself;
      }
      if constexpr (MIXED) {
        int4 v[B];
#pragma unroll
        for (int q = 0; q < B; ++q) v[q] = qpos[jj[q]];
#pragma unroll
        for (int q = 0; q < B; ++q) {
          loaded(v[q].w);
          const float fx = qsep(qi.x, v[q].x, qsx);
          const float fy = qsep(qi.y, v[q].y, qsy);
          const float fz = qsep(qi.z, v[q].z, qsz);
          const float r = fast_sqrt(fmaf(fz, fz, fmaf(fy, fy, fx * fx)));
          const bool in = sub + LPI * (t0 + q) < len;
          er[t0 + q] = in ? r : rpad;
          em[t0 + q] = in ? __int_as_float(v[q].w) : 0.f;
          if constexpr (E > 16) loaded(er[t0 + q]);
        }
      } else {
        double4 v[B];
#pragma unroll
        for (int q = 0; q < B; ++q) v[q] = xyzm[jj[q]];
#pragma unroll
        for (int q = 0; q < B; ++q) {
          loaded(v[q].w);
          const double dx = fold(xi - v[q].x, kp.len[0], kp.half[0], kp.periodic[0]);
          const double dy = fold(yi - v[q].y, kp.len[1], kp.half[1], kp.periodic[1]);
          const double dz = fold(zi - v[q].z, kp.len[2], kp.half[2], kp.periodic[2]);
          const double r = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
          const bool in = sub + LPI * (t0 + q) < len;
          er[t0 + q] = in ? r : rpad;
          em[t0 + q] = in ? v[q].w : 0.0;
          loaded(er[t0 + q]);
        }
      }
    }
    // ---- h iteration over the gathered entries
    double hlo = 0.0, hhi = SPH_INF;
    bool conv = !act, outgrew = false;
    int nit = 0;
    double S0 = 0.0, S1 = 0.0;
    uint32_t nnb = 0;
    while (true) {
      const double hinv = 1.0 / h;
      // mixed: each lane sums its few terms in FP32; lanes are combined in FP64
      const R hinvr = (R)hinv, twoh = (R)(kp.support * h);
      R s0 = R(0), s1 = R(0);
      uint32_t cnt = 0;
#pragma unroll
      for (int t0 = 0; t0 < E; t0 += B) {
        if (t0 * LPI >= lmax) break;
#pragma unroll
        for (int q = 0; q < B; ++q) {
          const R r = er[t0 + q], m = em[t0 + q];
          const R w = r * hinvr;
          R f, df;
          kf_df<KIND, R>(w, f, df);
          s0 = fma(m, f, s0);
          s1 = fma(m, fma(w, df, R(3) * f), s1);
          cnt += (r < twoh) ? 1u : 0u;
        }
      }
      double a0 = (double)s0, a1 = (double)s1;
      a0 = seg_sum<LPI>(a0);
      a1 = seg_sum<LPI>(a1);
      cnt = seg_sum_u32<LPI>(cnt);
      const double h3 = hinv * hinv * hinv;
      S0 = a0 * h3 * kp.knorm;
      S1 = -a1 * h3 * hinv * kp.knorm;
      nnb = cnt;
      sums += (act && sub == 0) ? (unsigned long long)cnt : 0ull;
      bool moved = false;
      if (!conv) {
        const double t = kp.hfact * hinv;
        const double rh = mi * (t * t * t);
        const double f = S0 - rh;
        const double fp = S1 + 3.0 * rh * hinv;
        double hn = h;
        if (kp.fixed_passes) {
          hn = h - f / fp;
          if (!(fp > 0.0))
            hn = h;
          else if (hn > 1.2 * h)
            hn = 1.2 * h;
          else if (hn < 0.8 * h)
            hn = 0.8 * h;
          // three density computations (Sect. 3.2.1): two updates, then
          // rho and Omega from the third sum at the h it used
          conv = (nit + 1) >= 2;
          moved = true;
        } else if (fabs(f) <= 3.0 * kp.h_tol * rh) {
          conv = true;
        } else {
          if (f < 0.0)
            hlo = fmax(hlo, h);
          else
            hhi = fmin(hhi, h);
          hn = h - f / fp;
          const bool bad = !(fp > 0.0) || !(hn >= 0.8 * h) || !(hn <= 1.2 * h) ||
                           !(hn > hlo) || !(hn < hhi);
          if (bad) {
            if (hlo > 0.0 && hhi < SPH_INF)
              hn = 0.5 * (hlo + hhi);
            else
              hn = (f < 0.0) ? 1.2 * h : h / 1.2;
          }
          conv = fabs(hn - h) <= 4e-16 * h;
          moved = true;
        }
        if (moved) {
          h = hn;
          if (h > hl) outgrew = true;
          ++nit;
          if (nit > kp.max_iter) {
            err |= kErrNoConv;
            conv = true;
          }
        }
      }
      if (ballot64(outgrew) != 0ull) break;  // rows too short: the walking kernel redoes it
      if (ballot64(!conv || moved) == 0ull) break;
    }
    if (ballot64(outgrew) != 0ull) {
      // the groups of every particle of this chunk go to the walking kernel
      const int gi = grp_of[i];
      if (act && sub == 0 && atomicCAS(&gflag[gi], 0, 2) == 0) {
        flag_list[atomicAdd(&ds->n_flagged, 1)] = gi;
        ++ngrew;
      }
      outgrew_any = true;
      continue;
    }
    it_max = max(it_max, nit + 1);
    if (act) {
      density_outputs<MIXED>(kp, p, frec_out, i, xi, yi, zi, qi, mi, h, S0, S1, minhalf, err,
                             sub == 0);
      if (sub == 0) pairs_final += nnb;
    }
  }
  const uint64_t b = ballot64(err != 0);
  uint32_t eall = err;
  for (int d = 32; d > 0; d >>= 1) eall |= __shfl_xor(eall, d, kWave);
  unsigned long long pf = pairs_final, sm = sums;
  for (int d = 32; d > 0; d >>= 1) {
    pf += __shfl_xor(pf, d, kWave);
    sm += __shfl_xor(sm, d, kWave);
    ngrew += __shfl_xor(ngrew, d, kWave);
  }
  outgrew_any = ballot64(outgrew_any) != 0ull;
  if (lane == 0) {
    WaveTally& tally = my_tally(ds);
    if (b) atomicOr(&ds->err, eall);
    if (it_max > 0) atomicMax(&tally.max_iter, it_max);
    if (pf) atomicAdd(&tally.n_pairs_density, pf);
    if (sm) atomicAdd(&tally.n_sums_density, sm);
    if (sm) atomicAdd(&tally.tot_sums_density, sm);
    if (outgrew_any) {
      atomicMax(&ds->leaf_state, 2);
      atomicOr(&ds->lists_missing, 1);
      atomicAdd(&ds->n_flag_grew, ngrew);
    }
  }
}

// ============================================================================
// Force from the neighbour lists (Sect. 2.4-2.6): one wavefront per group,
// LPI lanes per particle, each lane walking its share of row i.  The exact
// pair predicate (j != i, r < 2 max(h_i, h_j) with the converged h) is applied
// to every entry; accepted pairs add the pressure, viscosity and conductivity
// terms.  Runs only while every row is complete (leaf_state 1); flagged
// groups are left to the walking kernel.
//
// Was bound by the L1's access rate (one access per cycle and CU, all cycles
// taken): each lane loaded its own 64- or 128-byte record, four or eight
// 16-byte loads of 64 scattered lanes each.  The records now come through LDS,
// a record's bytes loaded by neighbouring lanes (LdsGather); FP64 10^6 1207 ->
// 835 us, FP64 Wendland C6 294,912 792 -> 529, mixed 16.8M 7.46 -> 6.65 ms,
// mixed 10^6 460 -> 401 us, mixed M6 294,912 240 -> 218.  A second buffer per
// wavefront (the next records in flight during the pair terms) costs FP64 half
// its wavefronts (835 -> 998 us) and gains the mixed form nothing over a fifth
// wavefront per SIMD.
// ============================================================================
// Blocks of four wavefronts take neighbouring chunks, which share L1 lines
// (one wavefront per block: 3 % slower).
constexpr int kForceWpb = 4;
// Wavefronts per SIMD: what the registers allow without spilling.
constexpr int force_waves(bool mixed) { return mixed ? 5 : 4; }

template <bool MIXED, int LPI, int KIND>
__global__ __launch_bounds__(kWave * kForceWpb) __attribute__((amdgpu_waves_per_eu(force_waves(MIXED))))
void k_force_lists(KParams kp, Parts p,
                                                    const GroupInfo* __restrict__ groups,
                                                    const void* __restrict__ frec_in,
                                                    const int32_t* __restrict__ nl_idx,
                                                    const int32_t* __restrict__ nl_len,
                                                    const int32_t* __restrict__ gflag,
                                                    const int32_t* __restrict__ grp_of,
                                                    double* __restrict__ out_ax,
                                                    double* __restrict__ out_ay,
                                                    double* __restrict__ out_az,
                                                    double* __restrict__ out_du,
                                                    DevState* __restrict__ ds) {
  if (ds->leaf_state != 1) return;
  constexpr int RB = MIXED ? 4 : 8;   // 16-byte pieces of a record
  using Gather = LdsGather<RB>;
  __shared__ alignas(128) char s_rec[kForceWpb][Gather::kBytes];
  using Rec = typename FRecOf<MIXED>::T;
  const Rec* __restrict__ rec = reinterpret_cast<const Rec*>(frec_in);
  const int lane = threadIdx.x % kWave;
  const int slot = lane / LPI, sub = lane % LPI;
  constexpr int CS = kWave / LPI;  // particles per chunk
  const int nch = (kp.n + CS - 1) / CS;
  const GroupRange gr = xcd_items<kForceWpb>(nch);
  uint32_t err = 0;
  uint32_t pairs = 0, cands = 0;  // this lane's: n / (64 wavefronts) rows of at most 256
  double dtmin = SPH_INF;
  char* const rec_lds = s_rec[__builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave)];
  const Gather gather(rec, rec_lds, lane);
  const bool any_flag = ds->n_flagged != 0;

  for (int g = gr.beg; g < gr.end; g += gr.step) {
    const int first = g * CS, count = min(CS, kp.n - first);
    const bool inr = slot < count;
    const int i = first + (inr ? slot : 0);
    // particles of flagged groups are left to the walking kernel
    const bool act = inr && (!any_flag || gflag[grp_of[i]] == 0);
    if (any_flag && ballot64(act) == 0ull) continue;
    const Rec ri = rec[i];
    int len = nl_len[i];
    loaded(len);
    len = act ? len : 0;
    const int32_t* __restrict__ row = nl_idx + ((int64_t)i * kp.nl_cap + sub);
    const int lmax = __builtin_amdgcn_readfirstlane(wave_max_i32(len));
    cands += (act && sub == 0) ? (uint32_t)len : 0u;
    double ax = 0.0, ay = 0.0, az = 0.0, du = 0.0, vmax = 0.0;
    // body(record, index) for this lane's share of the row (index -1 past its
    // end), in order, one record per lane at a time; the indices are loaded
    // one set ahead.
    auto rows_loop = [&](auto body) {
      int k = sub;
      auto index = [&]() {     // of the next entry (within the row's nl_cap entries)
        const int j = row[0];
        k += LPI;
        row += k < kp.nl_cap ? LPI : 0;
        return j;
      };
      int next = index();
      for (int k0 = 0; k0 < lmax; k0 += LPI) {
        const int j = k - LPI < len ? next : -1;
        gather.start(rec_lds, j);
        next = index();
        Gather::wait();
        Piece pc[RB];
        gather.read(pc);
        body(__builtin_bit_cast(Rec, pc), j);
      }
    };
    if constexpr (MIXED) {
      const float al = (float)kp.alpha, be = (float)kp.beta, hau = (float)(0.5 * kp.alpha_u);
      const float vxi = ri.vx, vyi = ri.vy, vzi = ri.vz, hif = (float)p.h[i];
      const float hinvi = ri.hinv, h4i = ri.hinv4pi, gi = ri.g, ki = ri.k;
      const float Pi = ri.P, rhoi = ri.rho, ui = ri.u;
      const float aci = al * ri.c, nhki = -0.5f * ki, S = (float)kp.support;
      // per-lane sums in FP32 (a lane takes one in LPI of the row's pairs),
      // combined across the slot's lanes in FP64 below
      float fax = 0.f, fay = 0.f, faz = 0.f, fdu = 0.f, fvmax = 0.f;
      uint32_t npr = 0;
      // The pair terms of eq:acc and eq:energy with the switch w_ = min(w, 0)
      // of the approaching pairs (w = v_ij . e_ij):
      //   t_i = g_i - k_i vsig_i w_ / 2,  A_i = t_i m_j F_i,  pa = A_i + t_j m_j F_j,
      //   a_i -= pa e_ij,  du_i += w A_i + (alpha_u / 2) v^u (u_i - u_j)
      //                                   (k_i m_j F_i + k_j m_j F_j);
      // the viscous heating of an approaching pair is the w_ part of w A_i.
      // The FP32 support test is settled in FP64 near its boundary, so the
      // accepted pairs are those of the FP64 predicate.
      const float qsx = ds->qf.step[0], qsy = ds->qf.step[1], qsz = ds->qf.step[2];
      auto pair = [&](const Rec& rj, int j) {
        const float dx = qsep(ri.qx, rj.qx, qsx);
        const float dy = qsep(ri.qy, rj.qy, qsy);
        const float dz = qsep(ri.qz, rj.qz, qsz);
        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        const float sr = S * fmaxf(hif, rj.h);
        const float sr2 = sr * sr;
        bool in = r2 < sr2;
        const bool border = fabsf(r2 - sr2) <= kBorder * sr2;
        if (ballot64(border) != 0ull)
          if (border) in = exact_pair_lean(kp, p.x, p.y, p.z, p.h, i, j);
        if (!in) return;
        ++npr;
        const float rinv = __builtin_amdgcn_rsqf(r2);
        const float r = r2 * rinv;
        const float ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
        const float w = fmaf(vzi - rj.vz, ez, fmaf(vyi - rj.vy, ey, (vxi - rj.vx) * ex));
        const float mFi = rj.m * (kdf<KIND, float>(r * hinvi) * h4i);
        const float mFj = kdf<KIND, float>(r * rj.hinv) * (rj.m * rj.hinv4pi);
        const float aw = fabsf(w), wn = fminf(w, 0.f);
        const float vsi = fmaf(be, aw, aci);
        const float vsj = fmaf(be, aw, al * rj.c);
        const float ti = fmaf(nhki * vsi, wn, gi);
        const float tj = fmaf(-0.5f * rj.k * vsj, wn, rj.g);
        const float Ai = ti * mFi;
        const float pa = fmaf(tj, mFj, Ai);
        fax = fmaf(-pa, ex, fax);
        fay = fmaf(-pa, ey, fay);
        faz = fmaf(-pa, ez, faz);
        const float vu = fast_sqrt(fabsf(Pi - rj.P) * fast_rcp(0.5f * (rhoi + rj.rho)));
        const float X = fmaf(mFi, ki, mFj * rj.k);
        fdu = fmaf(w, Ai, fmaf(hau * vu * (ui - rj.u), X, fdu));
        fvmax = fmaxf(fvmax, vsi);
      };
      rows_loop([&](const Rec& rj, int j) {
        if (j >= 0 && j != i) pair(rj, j);
      });
      ax = fax;
      ay = fay;
      az = faz;
      du = fdu;
      vmax = fvmax;
      pairs += npr;
    } else {
      const double al = kp.alpha, be = kp.beta, au = kp.alpha_u;
      const double vxi = ri.vx, vyi = ri.vy, vzi = ri.vz;
      const double hinvi = ri.hinv, h4i = ri.hinv4pi, gi = ri.g, ki = ri.k, ci = ri.c;
      const double Pi = ri.P, rhoi = ri.rho, ui = ri.u;
      const double xi = ri.x, yi = ri.y, zi = ri.z, hi = p.h[i];
      auto pair = [&](const Rec& rj) {
        const double dx = fold(xi - rj.x, kp.len[0], kp.half[0], kp.periodic[0]);
        const double dy = fold(yi - rj.y, kp.len[1], kp.half[1], kp.periodic[1]);
        const double dz = fold(zi - rj.z, kp.len[2], kp.half[2], kp.periodic[2]);
        const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
        const double sr = kp.support * (hi > rj.h ? hi : rj.h);
        if (!(r2 < sr * sr)) return;
        ++pairs;
        const double r = sqrt(r2);
        const double rinv = 1.0 / r;
        const double ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
        const double w = fma(vzi - rj.vz, ez, fma(vyi - rj.vy, ey, (vxi - rj.vx) * ex));
        const double Fi = kdf<KIND, double>(r * hinvi) * h4i;
        const double Fj = kdf<KIND, double>(r * rj.hinv) * rj.hinv4pi;
        const double aw = fabs(w);
        const bool app = w < 0.0;
        const double vsi = fma(be, aw, al * ci);
        const double vsj = fma(be, aw, al * rj.c);
        const double ti = app ? fma(-0.5 * vsi * w, ki, gi) : gi;
        const double tj = app ? fma(-0.5 * vsj * w, rj.k, rj.g) : rj.g;
        const double pa = rj.m * fma(ti, Fi, tj * Fj);
        ax -= pa * ex;
        ay -= pa * ey;
        az -= pa * ez;
        const double mwF = rj.m * w * Fi;
        double e = gi * mwF;
        if (app) e = fma(-0.5 * ki * vsi * w, mwF, e);
        const double vu = sqrt(fabs(Pi - rj.P) / (0.5 * (rhoi + rj.rho)));
        e = fma(rj.m * au * vu * (ui - rj.u), 0.5 * fma(Fi, ki, Fj * rj.k), e);
        du += e;
        vmax = fmax(vmax, vsi);
      };
      rows_loop([&](const Rec& rj, int j) {
        if (j >= 0 && j != i) pair(rj);
      });
    }
    ax = seg_sum<LPI>(ax);
    ay = seg_sum<LPI>(ay);
    az = seg_sum<LPI>(az);
    du = seg_sum<LPI>(du);
    vmax = seg_max<LPI>(vmax);
    if (act) {
      const double v0 = (kp.alpha == 0.0) ? (double)ri.c : kp.alpha * (double)ri.c;
      const double vs = fmax(vmax, v0);
      if (!(isfinite(ax) && isfinite(ay) && isfinite(az) && isfinite(du))) err |= kErrNonFinite;
      if (sub == 0) {
        out_ax[i] = ax;
        out_ay[i] = ay;
        out_az[i] = az;
        out_du[i] = du;
        p.vsig[i] = vs;
      }
      dtmin = fmin(dtmin, kp.c_cour * p.h[i] / vs);
    }
  }
  const uint64_t b = ballot64(err != 0);
  uint32_t eall = err;
  for (int d = 32; d > 0; d >>= 1) eall |= __shfl_xor(eall, d, kWave);
  unsigned long long pf = pairs, cd = cands;
  for (int d = 32; d > 0; d >>= 1) {
    pf += __shfl_xor(pf, d, kWave);
    cd += __shfl_xor(cd, d, kWave);
  }
  const double dm = wave_min_f64(dtmin);
  if (lane == 0) {
    WaveTally& tally = my_tally(ds);
    if (b) atomicOr(&ds->err, eall);
    if (pf) atomicAdd(&tally.n_pairs_force, pf);
    if (pf) atomicAdd(&tally.tot_pairs_force, pf);
    if (cd) atomicAdd(&tally.n_cand_force, cd);
    if (dm < SPH_INF) dt_min_update(tally, dm);
  }
}

// ============================================================================
// The pairs the list kernels accept (Sect. 3.2), for inspection and for the
// adjoint's frozen neighbour sets: each particle's row filtered with the
// exact FP64 predicate at the h in p.h (the mixed force kernel settles its
// FP32 test in FP64 near the boundary, so it accepts the same pairs); mode
// 0: density set (r < S h_i, self included), 1: force set (j != i,
// r < S max(h_i, h_j)).  Particles of flagged groups (incomplete rows) get
// the count -1.  Indices are written at offsets[i] in row order.
// ============================================================================
template <int LPI>
__global__ __launch_bounds__(64) void k_row_sets(KParams kp, Parts p, int mode,
                                                 const int32_t* __restrict__ nl_idx,
                                                 const int32_t* __restrict__ nl_len,
                                                 const int32_t* __restrict__ gflag,
                                                 const int32_t* __restrict__ grp_of,
                                                 int32_t* __restrict__ counts,
                                                 int32_t* __restrict__ idx,
                                                 const int64_t* __restrict__ offsets) {
  const int lane = threadIdx.x;
  const int slot = lane / LPI, sub = lane % LPI;
  constexpr int CS = kWave / LPI;
  const int nch = (kp.n + CS - 1) / CS;
  const GroupRange gr = xcd_groups(nch);
  for (int g = gr.beg; g < gr.end; g += gr.step) {
    const int first = g * CS, count = min(CS, kp.n - first);
    const bool inr = slot < count;
    const int i = first + (inr ? slot : 0);
    const bool act = inr && gflag[grp_of[i]] == 0;
    const int len = act ? min(nl_len[i], kp.nl_cap) : 0;
    int lmax = len;
    for (int d = 32; d > 0; d >>= 1) lmax = max(lmax, __shfl_xor(lmax, d, kWave));
    const int32_t* __restrict__ row = nl_idx + (int64_t)i * kp.nl_cap;
    const int64_t base = (act && idx) ? offsets[i] : 0;
    int n = 0;  // accepted entries of this slot so far (uniform over the slot's lanes)
    for (int k0 = 0; k0 < lmax; k0 += LPI) {
      const int k = k0 + sub;
      bool hit = false;
      int j = i;
      if (k < len) {
        j = row[k];
        hit = exact_pair(kp, p.x, p.y, p.z, p.h, i, j, mode == 1) && (mode == 0 || j != i);
      }
      const uint64_t b = ballot64(hit);
      const uint32_t seg = (uint32_t)(b >> (slot * LPI)) & ((1u << LPI) - 1u);
      if (hit && idx) idx[base + n + __popc(seg & ((1u << sub) - 1u))] = j;
      n += __popc(seg);
    }
    if (inr && sub == 0) counts[i] = act ? n : -1;
  }
}

// ============================================================================
// Neighbour sets for inspection: the same walk, the exact FP64 predicates,
// counts (idx == nullptr) or indices written at offsets[i].
// ============================================================================
template <int LPI>
__global__ __launch_bounds__(64) void k_neighbours(KParams kp, Parts p, int mode,
                                                   const WalkNode* __restrict__ nodes,
                                                   const GroupInfo* __restrict__ groups,
                                                   int32_t* __restrict__ counts,
                                                   const int64_t* __restrict__ offsets,
                                                   int32_t* __restrict__ idx,
                                                   int32_t* __restrict__ walk_spill,
    DevState* __restrict__ ds) {
  int* __restrict__ spill = walk_spill + (int64_t)blockIdx.x * 2 * kSpill;
  __shared__ WalkLds L;
  __shared__ int s_front[2][kFCap];
  __shared__ TileOf<double> T;
  const int lane = threadIdx.x;
  const int slot = lane / LPI, sub = lane % LPI;
  const int ng = ds->n_groups;
  uint32_t err = 0;
  for (int g = blockIdx.x; g < ng; g += gridDim.x) {
    const GroupInfo G = groups[g];
    const bool act = slot < G.count;
    const int i = G.first + (act ? slot : 0);
    const double xi = p.x[i], yi = p.y[i], zi = p.z[i], hi = p.h[i];
    int cnt = 0;
    const double hg = G.hmax;
    auto radius = [&](const WalkNode& nd) {
      return kp.support * (mode == 1 ? fmax(hg, (double)nd.hmax) : hg) * (1.0 + 4e-9);
    };
    auto flush = [&](int nleaf) {
      const int total = leaf_offsets(L, nleaf);
      for_tiles<LPI, double>(L, nleaf, total, sub, p.x, p.y, p.z, p.h, T, G, kp,
                             [&](bool valid, int c) {
        bool pred = false;
        const int j = valid ? T.j[c] : -1;
        if (valid && act) {
          const double dx = fold(xi - T.x[c], kp.len[0], kp.half[0], kp.periodic[0]);
          const double dy = fold(yi - T.y[c], kp.len[1], kp.half[1], kp.periodic[1]);
          const double dz = fold(zi - T.z[c], kp.len[2], kp.half[2], kp.periodic[2]);
          const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
          if (mode == 0) {
            const double s = kp.support * hi;
            pred = r2 < s * s;
          } else {
            const double hj = T.a[c];
            const double s = kp.support * (hi > hj ? hi : hj);
            pred = (j != i) && r2 < s * s;
          }
        }
        const uint64_t b = ballot64(pred);
        const uint32_t seg = (uint32_t)((b >> (slot * LPI)) & ((LPI == 64) ? ~0ull : ((1ull << LPI) - 1ull)));
        const int pos = cnt + __popc(seg & ((1u << sub) - 1u));
        if (pred && idx) idx[offsets[i] + pos] = j;
        cnt += __popc(seg);
      });
      __syncthreads();
    };
    if (!group_walk(nodes, G, kp, L, s_front, spill, radius, flush)) err |= kErrFrontier;
    if (act && sub == 0 && !idx) counts[i] = cnt;
  }
  if (err) atomicOr(&ds->err, err);
}

// ============================================================================
// Integration and reductions (one thread per particle)
// ============================================================================
__global__ void k_set_leaf_state(DevState* ds, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ds->leaf_state = v;
    ds->lists_missing = 0;
    ds->n_flag_rows = 0;
    ds->n_flag_grew = 0;
    ds->n_flagged = 0;
    ds->pool_used = 0;
    if (ds->n_groups == 0) no_rows(ds);
  }
}

// The tallies, one per lane of the one wavefront that the next kernels run in.
static_assert(kTallies == kWave, "one lane per tally");

__global__ void k_reset_force_state(DevState* ds) {
  ds->tally[threadIdx.x].dt_min_enc = enc_f64(SPH_INF);
}

__device__ __forceinline__ void clear_counters(DevState* ds) {
  WaveTally& t = ds->tally[threadIdx.x];
  t.max_iter = 0;
  t.n_pairs_density = 0;
  t.n_pairs_force = 0;
  t.n_sums_density = 0;
  t.n_cand_density = 0;
  t.n_cand_force = 0;
  t.n_rewalk = 0;
  if (threadIdx.x == 0) {
    ds->leaf_state = 0;
    ds->lists_missing = 0;
    ds->n_flag_rows = 0;
    ds->n_flag_grew = 0;
    ds->n_flagged = 0;
    ds->pool_used = 0;
  }
}

__global__ void k_reset_counters(DevState* ds) { clear_counters(ds); }

// Start of a step: counters cleared; the step's dt (the host's, or the
// previous force pass's Courant minimum) taken before that minimum is reset
// for this step's force pass; neighbour lists wanted (leaf_state 1: the tree
// kernels before the density do not read it).
__global__ void k_step_begin(DevState* ds, double dt_host) {
  const double dt = wave_min_f64(dec_f64(ds->tally[threadIdx.x].dt_min_enc));
  ds->tally[threadIdx.x].dt_min_enc = enc_f64(SPH_INF);
  clear_counters(ds);
  if (threadIdx.x == 0) {
    ds->dt_cur = (dt_host > 0.0) ? dt_host : dt;
    ds->leaf_state = 1;
  }
}

// v1 = v_p + (a1 - a0) dt/2, u1 = u_p + (du1 - du0) dt/2; a0 <- a1.
__global__ __launch_bounds__(256) void k_correct(Parts p, int n, const double* __restrict__ a1,
                                                  int64_t stride, const DevState* __restrict__ ds) {
  const double hdt = 0.5 * ds->dt_cur;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const double nax = a1[i], nay = a1[stride + i], naz = a1[2 * stride + i],
                 ndu = a1[3 * stride + i];
    p.vx[i] = p.vx[i] + (nax - p.ax[i]) * hdt;
    p.vy[i] = p.vy[i] + (nay - p.ay[i]) * hdt;
    p.vz[i] = p.vz[i] + (naz - p.az[i]) * hdt;
    p.u[i] = p.u[i] + (ndu - p.dudt[i]) * hdt;
    p.ax[i] = nax;
    p.ay[i] = nay;
    p.az[i] = naz;
    p.dudt[i] = ndu;
  }
}

constexpr int kRedBlocks = 512;

// Fixed-order FP64 sums: thread t of block b owns particles b*256+t + k*stride.
__global__ __launch_bounds__(256) void k_reduce_part(Parts p, int n, double* __restrict__ part) {
  __shared__ double s[12][256];
  double acc[12];
  for (int q = 0; q < 12; ++q) acc[q] = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += kRedBlocks * 256) {
    const double m = p.m[i], vx = p.vx[i], vy = p.vy[i], vz = p.vz[i];
    const double ax = p.ax[i], ay = p.ay[i], az = p.az[i], du = p.dudt[i], u = p.u[i];
    const double v2 = vx * vx + vy * vy + vz * vz;
    const double va = vx * ax + vy * ay + vz * az;
    acc[1] += 0.5 * m * v2;
    acc[2] += m * u;
    acc[3] += m * vx;
    acc[4] += m * vy;
    acc[5] += m * vz;
    acc[6] += m * ax;
    acc[7] += m * ay;
    acc[8] += m * az;
    acc[9] += m * (va + du);
    acc[10] += m * sqrt(ax * ax + ay * ay + az * az);
    acc[11] += m * (fabs(va) + fabs(du));
  }
  for (int q = 0; q < 12; ++q) s[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int q = 0; q < 12; ++q) s[q][threadIdx.x] += s[q][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 12) part[blockIdx.x * 12 + threadIdx.x] = s[threadIdx.x][0];
}

// The block sums added in block order.  A chain of 512 dependent additions per
// sum: from LDS, where the whole block loads the partials first (read one by
// one from memory they took 13 us; 7 us so).
constexpr int kRedParts = kRedBlocks * 12;
__global__ __launch_bounds__(512) void k_reduce_final(const double* __restrict__ part,
                                                       double* __restrict__ out) {
  __shared__ double s[kRedParts];
  for (int k = threadIdx.x; k < kRedParts; k += 512) s[k] = part[k];
  __syncthreads();
  double a = 0.0;
  if (threadIdx.x < 12) {
#pragma unroll 32
    for (int b = 0; b < kRedBlocks; ++b) a += s[b * 12 + threadIdx.x];
  }
  // E = E_kin + E_th
  const double th = __shfl(a, 2, kWave), kin = __shfl(a, 1, kWave);
  if (threadIdx.x == 0) a = kin + th;
  if (threadIdx.x < 12) out[threadIdx.x] = a;
}

// ============================================================================
// Allocation-free reduction: the partial sums of k_reduce_part and the 12
// results of k_reduce_final in a file-scope device array instead of context
// scratch.  Each GPU the library runs on holds its own copy, until the
// process ends.  Host code never passes the array's name to a kernel or a
// copy: it takes the array's device address on each device once
// (hipGetSymbolAddress, with that device current) and uses that address.
// ============================================================================
constexpr int kRedScratch = kRedBlocks * 12 + 16;  // doubles: partials, then the 12 sums
static __device__ __align__(256) double scratch[kRedScratch];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device (looked up on the first
// call there).
static hipError_t scratch_address(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// ============================================================================
// Host-side launchers
// ============================================================================
static Parts parts_of(const sph_particles* s) {
  Parts p;
  p.id = s->id;
  p.x = s->x;
  p.y = s->y;
  p.z = s->z;
  p.vx = s->vx;
  p.vy = s->vy;
  p.vz = s->vz;
  p.m = s->m;
  p.u = s->u;
  p.h = s->h;
  p.ax = s->ax;
  p.ay = s->ay;
  p.az = s->az;
  p.dudt = s->dudt;
  p.rho = s->rho;
  p.omega = s->omega;
  p.P = s->P;
  p.cs = s->cs;
  p.vsig = s->vsig_dt;
  return p;
}

static int stream_blocks(int n) {
  int b = (n + 255) / 256;
  return b < 1 ? 1 : (b > 8192 ? 8192 : b);
}

// The radix sort's workspace: look-back status words of every pass and tile,
// then the digit histograms of the passes, then the head, then the key bits of
// every block of k_predict_keys.
struct SortWs {
  uint32_t *status, *ghist;
  SortHead* head;
  uint64_t* range;
};
static SortWs sort_ws(sph_ctx* c) {
  const int64_t nst = (int64_t)c->n_max_sort_blocks * 8 * 256;
  static_assert(sizeof(SortHead) <= 4 * kSortHeadWords, "the head fits its words");
  SortWs w;
  w.status = c->radix_cnt;
  w.ghist = c->radix_cnt + nst;
  w.head = reinterpret_cast<SortHead*>(w.ghist + 8 * 256);
  w.range = reinterpret_cast<uint64_t*>(w.ghist + 8 * 256 + kSortHeadWords);
  return w;
}

// Passes of the sort: enough of the leading key bits that a cell of them
// holds 2^-6 particles on average (the key bits of an axis shorter than the
// longest do not vary at the top and do not count), so that denser regions
// keep runs of a few particles.  Sort (all its launches) of 32^3 particles in
// a cube 40 us, of 294,912 in a box of 16:1:1 90, of 16.8M in a cube 983 with
// the 3, 5 and 4 passes this gives; 77, 119 and 1750 with all eight.
static int sort_passes(const sph_ctx* c) {
  int want = 6;
  for (int64_t m = c->n; m > 1; m = (m + 1) >> 1) ++want;
  int top = -1, have = 0;
  for (int bit = 3 * kKeyLevels - 1; bit >= 0; --bit) {
    const int axis = 2 - bit % 3, level = bit / 3;  // bit of cell coordinate
    if (!(c->kp.len[axis] * c->kp.key_scale > ldexp(1.0, level))) continue;
    if (top < 0) top = bit;
    if (++have == want) return (top - bit + 8) / 8;
  }
  return 8;
}

constexpr int kSortSmall = 4096, kPermuteSmall = 16384;

hipError_t launch_predict_keys(sph_ctx* c, const sph_particles* s, bool predict, double) {
  c->kp.n = c->n;
  if (c->n <= kSortSmall) {  // the sort too
    const auto kernel = c->n <= 1024   ? k_sort_small<1>
                        : c->n <= 2048 ? k_sort_small<2>
                                       : k_sort_small<4>;
    launch_last(c, kernel, dim3(1), dim3(1024), c->kp, parts_of(s), predict ? 1 : 0,
                sort_passes(c), c->ds, c->keys[0], c->vals[0], &c->ds->err);
    return hipGetLastError();
  }
  const SortWs w = sort_ws(c);
  const int src = sort_passes(c) & 1;
  hipLaunchKernelGGL(k_predict_keys, dim3(stream_blocks(c->n)), dim3(256), 0, c->stream, c->kp,
                     parts_of(s), predict ? 1 : 0, c->ds, c->keys[src], c->vals[src], w.ghist,
                     w.head, w.range, &c->ds->err);
  return hipGetLastError();
}

// Follows launch_predict_keys, which cleared the histograms and the head.
// The result is in buffer 0.
hipError_t launch_sort(sph_ctx* c) {
  const int n = c->n;
  if (n <= kSortSmall) return hipSuccess;
  const int nblk = (n + kSortTile - 1) / kSortTile;
  const SortWs w = sort_ws(c);
  const int pblocks = std::min(nblk, 4 * c->n_cu);
  const int npass = sort_passes(c);
  int src = npass & 1;
  hipLaunchKernelGGL(k_radix_prep, dim3(pblocks), dim3(256), 0, c->stream, c->keys[src], n, nblk,
                     npass, stream_blocks(n), w.range, w.status, w.ghist, w.head);
  for (int pass = 0; pass < npass; ++pass, src ^= 1) {
    const int dst = src ^ 1;
    hipLaunchKernelGGL(k_radix_pass, dim3(nblk), dim3(256), 0, c->stream, c->keys[src],
                       c->vals[src], c->keys[dst], c->vals[dst], n, pass, nblk, w.status, w.ghist,
                       w.head, &c->ds->err);
  }
  // the permute's staging space is free during the sort
  const RunWs ws(reinterpret_cast<uint32_t*>(c->gtmp), n);
  if (nblk < 4 * c->n_cu)
    hipLaunchKernelGGL(k_sort_fix<512>, dim3((n + 511) / 512), dim3(256), 0, c->stream, c->keys[0],
                       c->vals[0], n, ws, w.head);
  else
    hipLaunchKernelGGL(k_sort_fix<kSortTile>, dim3(nblk), dim3(256), 0, c->stream, c->keys[0],
                       c->vals[0], n, ws, w.head);
  // enough blocks for many runs at once, few enough to end quickly without one
  // (30,000 particles: 15 blocks 1.6 us without a run and 64 with a cluster's,
  // 128 blocks 1.7 and 9, 462 blocks 3.0)
  const int blocks = n > (1 << 17) ? 3 * c->n_cu : std::max(nblk + nblk / 2, c->n_cu / 2);
  launch_last(c, k_resort, dim3(std::min(blocks, 3 * c->n_cu)), dim3(256), c->keys[0], c->vals[0],
              c->keys[1], c->vals[1], n, w.status, ws, w.head, &c->ds->err);
  return hipGetLastError();
}

hipError_t launch_permute(sph_ctx* c, const sph_particles* s, bool outputs_too) {
  FieldSet fs;
  fs.nf = 0;
  double* all[] = {s->x,  s->y,  s->z,    s->vx,  s->vy,   s->vz, s->m,  s->u,     s->h,
                   s->ax, s->ay, s->az,   s->dudt, s->rho, s->omega, s->P, s->cs, s->vsig_dt};
  const int n_in = 13;  // x..dudt are state; the rest are outputs
  fs.im = -1;
  for (int k = 0; k < (int)(sizeof(all) / sizeof(all[0])); ++k) {
    if (!all[k]) continue;
    if (k >= n_in && !outputs_too) continue;
    if (all[k] == s->m) fs.im = fs.nf;
    fs.f[fs.nf++] = all[k];
  }
  fs.xyzm = c->kp.precision == SPH_PREC_MIXED ? nullptr : c->xyzm;
  fs.id = s->id;
  // in place only if no two fields share memory
  bool apart = true;
  for (int k = 0; k < fs.nf; ++k)
    for (int q = 0; q < k; ++q)
      apart = apart && (fs.f[q] + c->n <= fs.f[k] || fs.f[k] + c->n <= fs.f[q]);
  for (int k = 0; k < fs.nf && fs.id; ++k)
    apart = apart && ((double*)fs.id + c->n <= fs.f[k] || fs.f[k] + c->n <= (double*)fs.id);
  if (c->n <= kPermuteSmall && apart) {
    const auto kernel = c->n <= 1024   ? k_permute_small<1>
                        : c->n <= 4096 ? k_permute_small<4>
                                       : k_permute_small<16>;
    launch_last(c, kernel, dim3(fs.nf + (fs.id ? 1 : 0)), dim3(1024), fs, c->vals[0], c->n);
    return hipGetLastError();
  }
  const int nb = stream_blocks(c->n);
  hipLaunchKernelGGL(k_gather, dim3(nb), dim3(256), 0, c->stream, fs, c->vals[0], c->gtmp,
                     c->gtmp_id, c->n, (int64_t)c->n_max);
  launch_last(c, k_copy_back, dim3(nb), dim3(256), fs, c->gtmp, c->gtmp_id, c->n,
              (int64_t)c->n_max);
  return hipGetLastError();
}

// FP64 contexts: x, y, z, m packed for the density gather (the mixed code
// records are packed with each refresh of the nodes' h_max, node_props)
hipError_t launch_pack_xyzm(sph_ctx* c, const sph_particles* s) {
  if (c->kp.precision != SPH_PREC_MIXED)
    hipLaunchKernelGGL(k_pack_xyzm, dim3(stream_blocks(c->n)), dim3(256), 0, c->stream,
                       parts_of(s), c->n, c->xyzm);
  return hipGetLastError();
}

static void pack_q(sph_ctx* c, const sph_particles* s, int mode) {
  launch_last(c, k_pack_q, dim3(stream_blocks(c->n)), dim3(256), c->kp, parts_of(s), c->n, c->ds,
              mode, c->qxyzm, c->qrec);
}

hipError_t launch_tree(sph_ctx* c) {
  const int n = c->n;
  const int nblk = (n + kTreeTile - 1) / kTreeTile;
  hipLaunchKernelGGL(k_tree_levels, dim3(nblk), dim3(256), 0, c->stream, c->keys[0], n,
                     c->kp.n_leaf, c->kp.n_group, c->dlev, c->lleaf, c->gsize, c->gstart,
                     c->tree_cnt, nblk, c->node_nchild, c->node_cap);
  const int64_t counts = ((int64_t)(kLevels + 1) * nblk + 3) / 4 * 4;
  const hipError_t e = scan_u32(c, c->tree_cnt, counts, c->scan_total);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tree_emit, dim3(nblk), dim3(256), 0, c->stream, c->keys[0], n,
                     c->dlev, c->lleaf, c->gsize, c->gstart, c->tree_cnt,
                     c->scan_total, nblk, c->node_cap, c->node_level, c->node_first,
                     c->node_count, c->node_parent, c->node_child, c->node_nchild,
                     c->grp_first, c->grp_count, c->nl_len, c->grp_of, c->gflag, c->ds);
  return hipGetLastError();
}

// Node boxes (positions) and largest h; group boxes.  The positions are the
// current (sorted) ones; h may be the start value or the converged one.
static hipError_t node_props(sph_ctx* c, const sph_particles* s, int mode) {
  const int n = c->n;
  const bool small = n <= kSmallTree;
  // leaves and groups four per wavefront; small trees: their inner nodes one
  // per wavefront in the same launch (from chunk boxes), large trees: one
  // launch per level afterwards (the deepest first; the last level holds
  // leaves only; the level offsets are the scanned per-level node counts).
  if (small && n > kNoChunks) {
    const int nch = (n + kChunk - 1) / kChunk;
    hipLaunchKernelGGL(k_chunk_boxes, dim3((nch + 3) / 4), dim3(256), 0, c->stream, s->x, s->y,
                       s->z, s->h, n, c->chunk_box, c->ds, mode);
  }
  const int64_t items = c->node_cap + (int64_t)n;
  const int nb = (int)std::min<int64_t>(std::max<int64_t>((items / 4 + 15) / 16, 16), 4096);
  const int nbi =
      small ? (int)std::min<int64_t>(std::max<int64_t>((c->node_cap / 8 + 63) / 64, 16), 4096) : 0;
  // the last launch stamps a phase boundary: here, unless the mixed code
  // records follow
  const bool mixed = c->kp.precision == SPH_PREC_MIXED;
  const hipEvent_t mark = c->mark;
  c->mark = small && !mixed ? mark : nullptr;
  launch_last(c, k_range_boxes, dim3(nb + nbi), dim3(256), s->x, s->y, s->z, s->h, c->node_first,
              c->node_count, c->node_child, c->node_nchild, c->wnode, c->grp_first, c->grp_count,
              c->ginfo, c->ds, mode, nb, n, c->chunk_box, c->node_parent);
  if (!small) {
    const int nblk = (n + kTreeTile - 1) / kTreeTile;
    const int lb =
        (int)std::min<int64_t>(std::max<int64_t>((c->node_cap / 4 + 255) / 256, 1), 1024);
    for (int l = kLevels - 2; l >= 0; --l) {
      c->mark = l == 0 && !mixed ? mark : nullptr;
      launch_last(c, k_level_boxes, dim3(lb), dim3(256), l, c->tree_cnt, nblk, c->node_first,
                  c->node_child, c->node_nchild, c->wnode, c->ds, mode);
    }
  }
  // mixed: the code records with the current h and m (a new tree's after its
  // frame, below)
  if (mixed) {
    c->mark = mark;
    if (mode != 1) pack_q(c, s, mode);
  }
  return hipGetLastError();
}

hipError_t launch_node_h(sph_ctx* c, const sph_particles* s, bool always) {
  return node_props(c, s, always ? 2 : 0);
}
hipError_t launch_node_boxes(sph_ctx* c, const sph_particles* s) {
  const hipError_t e = node_props(c, s, 1);
  if (e != hipSuccess) return e;
  // the mixed code records and their frame (FP64 contexts have neither)
  if (c->kp.precision == SPH_PREC_MIXED) {
    hipLaunchKernelGGL(k_qframe, dim3(1), dim3(64), 0, c->stream, c->kp, c->wnode, c->ds);
    pack_q(c, s, 1);
  }
  return hipGetLastError();
}

// Density and force of groups of 4 or 8 particles go through the neighbour
// lists; larger groups (and flagged groups) through the walking kernels.
bool lists_mode(const sph_ctx* c) { return c->kp.n_group == 4 || c->kp.n_group == 8; }

#define SPH_LPI_SWITCH(NG, BODY)      \
  switch (NG) {                       \
    case 4: {                         \
      constexpr int LPI = 16;         \
      BODY;                           \
    } break;                          \
    case 8: {                         \
      constexpr int LPI = 8;          \
      BODY;                           \
    } break;                          \
    case 16: {                        \
      constexpr int LPI = 4;          \
      BODY;                           \
    } break;                          \
    default: {                        \
      constexpr int LPI = 2;          \
      BODY;                           \
    } break;                          \
  }

#define SPH_LPI_SWITCH_LISTS(NG, BODY) \
  switch (NG) {                        \
    case 4: {                          \
      constexpr int LPI = 16;          \
      BODY;                            \
    } break;                           \
    default: {                         \
      constexpr int LPI = 8;           \
      BODY;                            \
    } break;                           \
  }

// Wavefronts for the flagged groups: one for each that the tree can have, at
// most about what is resident at a time.
static int flagged_blocks(const sph_ctx* c) {
  return std::min((c->n + 7) / 8 * 8, c->walk_blocks / 2);
}

template <bool MIXED>
static hipError_t density_dispatch(sph_ctx* c, const sph_particles* s, const int32_t* gflag) {
  const Parts p = parts_of(s);
  if (gflag) {
    SPH_LPI_SWITCH_LISTS(c->kp.n_group,
                         launch_last(c, (k_density<MIXED, LPI, true>), dim3(flagged_blocks(c)),
                                     dim3(64), c->kp, p, c->wnode, c->ginfo, c->frec,
                                     c->leaf_pool, c->pool_cap, c->gl_off, c->gl_cnt, gflag,
                                     c->walk_spill, c->ds));
  } else {
    SPH_LPI_SWITCH(c->kp.n_group,
                   launch_last(c, (k_density<MIXED, LPI, false>), dim3(c->walk_blocks), dim3(64),
                               c->kp, p, c->wnode, c->ginfo, c->frec, c->leaf_pool, c->pool_cap,
                               c->gl_off, c->gl_cnt, gflag, c->walk_spill, c->ds));
  }
  return hipGetLastError();
}

hipError_t launch_density(sph_ctx* c, const sph_particles* s, bool flagged_only) {
  c->kp.n = c->n;
  const int32_t* gf = flagged_only ? c->flag_list : nullptr;
  return c->kp.precision == SPH_PREC_MIXED ? density_dispatch<true>(c, s, gf)
                                           : density_dispatch<false>(c, s, gf);
}

hipError_t launch_lists(sph_ctx* c, const sph_particles* s) {
  c->kp.n = c->n;
  const int nblk = (c->n + kTreeTile - 1) / kTreeTile;
  // the units' leaf lists take the walking density's leaf-list pool, which that
  // kernel fills only later; single groups' lists the permute's staging space,
  // which is free between two tree builds
  int2* sg_list = c->leaf_pool;
  const int64_t sg_entries = c->pool_cap;
  int2* pool = reinterpret_cast<int2*>(c->gtmp);
  // and the groups' offsets and lengths the sort's second buffers
  int32_t* ll_off = reinterpret_cast<int32_t*>(c->keys[1]);
  int32_t* ll_cnt = reinterpret_cast<int32_t*>(c->vals[1]);
  const int pool_cap = (int)std::min<int64_t>((int64_t)kMaxFields * c->n_max, 0x7fffffff);
  // As many wavefronts as are resident at once: the items go round them, and a
  // second generation of wavefronts would run alone at the end (k_rows asked
  // for 8 per SIMD with 6 resident: 428 us instead of 362 at 10^6 particles).
  const int grid = leaf_walk_waves(c->n_cu);
  const int row_grid = kRowWaves * 4 * c->n_cu / 8 * 8;
  hipLaunchKernelGGL(k_leaves, dim3(grid), dim3(64), 0, c->stream, c->kp, c->wnode, c->ginfo,
                     c->tree_cnt, nblk, sg_list, sg_entries, pool, pool_cap, ll_off, ll_cnt,
                     c->gflag, c->walk_spill, c->ds);
  const auto rows = c->kp.precision == SPH_PREC_MIXED ? k_rows<true> : k_rows<false>;
  launch_last(c, rows, dim3(row_grid), dim3(64), c->kp, s->h, c->wnode, c->ginfo, sg_list,
              sg_entries, grid, pool, ll_off, ll_cnt, c->nl_idx, c->nl_len, c->gflag,
              c->flag_list, c->grp_of, c->qrec, c->xyzm, c->ds);
  return hipGetLastError();
}

// The list kernels are instantiated per smoothing kernel (Sect. 2.3).
#define SPH_KIND_SWITCH(KD, BODY) \
  switch (KD) {                   \
    case 1: {                     \
      constexpr int KIND = 1;     \
      BODY;                       \
    } break;                      \
    case 2: {                     \
      constexpr int KIND = 2;     \
      BODY;                       \
    } break;                      \
    default: {                    \
      constexpr int KIND = 0;     \
      BODY;                       \
    } break;                      \
  }

template <bool MIXED, int CAP, int KIND>
static void density_lists_kind(sph_ctx* c, const Parts& p) {
  const dim3 grid(c->walk_blocks), block(64);
  SPH_LPI_SWITCH_LISTS(c->kp.n_group,
                       launch_last(c, (k_density_lists<MIXED, LPI, CAP, KIND>), grid, block,
                                   c->kp, p, c->ginfo, c->nl_idx, c->nl_len, c->gflag,
                                   c->flag_list, c->grp_of,
                                   MIXED ? (const void*)c->qxyzm : (const void*)c->xyzm, c->frec,
                                   c->ds));
}

template <bool MIXED, int CAP>
static void density_lists_dispatch(sph_ctx* c, const Parts& p) {
  SPH_KIND_SWITCH(c->kp.kernel, (density_lists_kind<MIXED, CAP, KIND>(c, p)));
}

hipError_t launch_density_lists(sph_ctx* c, const sph_particles* s) {
  c->kp.n = c->n;
  const Parts p = parts_of(s);
  const bool wide = c->kp.nl_cap > 128;
  if (c->kp.precision == SPH_PREC_MIXED) {
    if (wide)
      density_lists_dispatch<true, 256>(c, p);
    else
      density_lists_dispatch<true, 128>(c, p);
  } else {
    if (wide)
      density_lists_dispatch<false, 256>(c, p);
    else
      density_lists_dispatch<false, 128>(c, p);
  }
  return hipGetLastError();
}

template <bool MIXED>
static hipError_t force_dispatch(sph_ctx* c, const sph_particles* s, double* oax, double* oay,
                                 double* oaz, double* odu, const int32_t* gflag) {
  const Parts p = parts_of(s);
  // (with lists, every group walks once some h has outgrown its rows)
  const dim3 grid(gflag ? std::min((c->n + 7) / 8 * 8, c->walk_blocks) : c->walk_blocks), block(64);
  SPH_LPI_SWITCH(c->kp.n_group,
                 launch_last(c, (k_force<MIXED, LPI>), grid, block, c->kp, p, c->wnode, c->ginfo,
                             c->frec, c->leaf_pool, c->gl_off, c->gl_cnt, oax, oay, oaz, odu, gflag,
                             c->walk_spill, c->ds));
  return hipGetLastError();
}

static void force_outputs(sph_ctx* c, const sph_particles* s, bool step_mode, double** o) {
  o[0] = step_mode ? c->a1 : s->ax;
  o[1] = step_mode ? c->a1 + c->n_max : s->ay;
  o[2] = step_mode ? c->a1 + 2 * c->n_max : s->az;
  o[3] = step_mode ? c->a1 + 3 * c->n_max : s->dudt;
}

hipError_t launch_force(sph_ctx* c, const sph_particles* s, bool step_mode, bool flagged_only) {
  c->kp.n = c->n;
  double* o[4];
  force_outputs(c, s, step_mode, o);
  const int32_t* gf = flagged_only ? c->flag_list : nullptr;
  return c->kp.precision == SPH_PREC_MIXED ? force_dispatch<true>(c, s, o[0], o[1], o[2], o[3], gf)
                                           : force_dispatch<false>(c, s, o[0], o[1], o[2], o[3], gf);
}

// Lanes per particle: 64 / n_group, but 16 in FP64 as long as chunks of eight
// particles would leave SIMDs without a wavefront, and 32 for half of those
// sizes.  A wavefront alone on its SIMD waits for each block of gathered
// records, so half the row per lane is half the blocks: 8, 16 and 32 lanes
// 19.5, 13.4 and 10.2 us at 1000 particles, 19.5, 13.5 and 13.0 at 3375; 25.6
// and 26.6 with 8 and 16 at 13,824, worse beyond (230 and 251 at 262,144).
// The FP32 sums of the mixed mode keep their lanes.
template <bool MIXED, int KIND>
static void force_lists_kind(sph_ctx* c, const Parts& p, double* const* o) {
  const int n_group = !MIXED && c->n <= 8 * 4 * c->n_cu ? 4 : c->kp.n_group;
  const int waves = force_waves(MIXED) * 4 * c->n_cu;  // resident at once
  const dim3 grid(std::max(waves / kForceWpb / 8 * 8, 8)), block(kWave * kForceWpb);
  if constexpr (!MIXED) {
    if (c->n <= 8 * 2 * c->n_cu) {
      launch_last(c, (k_force_lists<MIXED, 32, KIND>), grid, block, c->kp, p, c->ginfo, c->frec,
                  c->nl_idx, c->nl_len, c->gflag, c->grp_of, o[0], o[1], o[2], o[3], c->ds);
      return;
    }
  }
  SPH_LPI_SWITCH_LISTS(n_group,
                       launch_last(c, (k_force_lists<MIXED, LPI, KIND>), grid, block, c->kp, p,
                                   c->ginfo, c->frec, c->nl_idx, c->nl_len, c->gflag, c->grp_of,
                                   o[0], o[1], o[2], o[3], c->ds));
}

hipError_t launch_force_lists(sph_ctx* c, const sph_particles* s, bool step_mode) {
  c->kp.n = c->n;
  double* o[4];
  force_outputs(c, s, step_mode, o);
  const Parts p = parts_of(s);
  if (c->kp.precision == SPH_PREC_MIXED) {
    SPH_KIND_SWITCH(c->kp.kernel, (force_lists_kind<true, KIND>(c, p, o)));
  } else {
    SPH_KIND_SWITCH(c->kp.kernel, (force_lists_kind<false, KIND>(c, p, o)));
  }
  return hipGetLastError();
}

// Each particle's pairs among its list row that pass the exact FP64
// predicate at the h in p->h (mode 0: density set, self included; 1: force
// set): counts, and the indices at offsets[i] when idx is given.
hipError_t launch_row_sets(sph_ctx* c, const sph_particles* s, int mode, int32_t* counts,
                           int32_t* idx, const int64_t* offsets) {
  c->kp.n = c->n;
  const Parts p = parts_of(s);
  const dim3 grid(c->walk_blocks), block(64);
  SPH_LPI_SWITCH_LISTS(c->kp.n_group,
                       hipLaunchKernelGGL((k_row_sets<LPI>), grid, block, 0, c->stream, c->kp, p,
                                          mode, c->nl_idx, c->nl_len, c->gflag, c->grp_of,
                                          counts, idx, offsets));
  return hipGetLastError();
}

hipError_t launch_leaf_state(sph_ctx* c, int v) {
  launch_last(c, k_set_leaf_state, dim3(1), dim3(64), c->ds, v);
  return hipGetLastError();
}

hipError_t launch_force_reset(sph_ctx* c) {
  launch_last(c, k_reset_force_state, dim3(1), dim3(64), c->ds);
  return hipGetLastError();
}

hipError_t launch_correct(sph_ctx* c, const sph_particles* s) {
  launch_last(c, k_correct, dim3(stream_blocks(c->n)), dim3(256), parts_of(s), c->n, c->a1,
              (int64_t)c->n_max, c->ds);
  return hipGetLastError();
}

// The sums of launch_reduce with the partials in `scratch` (its device
// address on the current device), copied into the host array out; the
// stream is synchronised.  Allocates nothing.
hipError_t reduce_noalloc(const sph_particles* s, hipStream_t stream, double* out) {
  double* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) return e;
  double* part = base;
  double* res = base + kRedBlocks * 12;
  hipLaunchKernelGGL(k_reduce_part, dim3(kRedBlocks), dim3(256), 0, stream, parts_of(s),
                     (int)s->n, part);
  hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(512), 0, stream, part, res);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(out, res, 12 * sizeof(double), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  return e;
}

// out: memory the device writes and the host reads (pinned).
hipError_t launch_reduce(sph_ctx* c, const sph_particles* s, double* out) {
  hipLaunchKernelGGL(k_reduce_part, dim3(kRedBlocks), dim3(256), 0, c->stream, parts_of(s),
                     (int)s->n, c->red_part);
  hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(512), 0, c->stream, c->red_part, out);
  return hipGetLastError();
}

hipError_t launch_step_begin(sph_ctx* c, double dt_host) {
  launch_last(c, k_step_begin, dim3(1), dim3(64), c->ds, dt_host);
  return hipGetLastError();
}

hipError_t launch_reset_counters(sph_ctx* c) {
  launch_last(c, k_reset_counters, dim3(1), dim3(64), c->ds);
  return hipGetLastError();
}

hipError_t launch_neighbours(sph_ctx* c, const sph_particles* s, int mode, int32_t* counts,
                             const int64_t* offsets, int32_t* idx) {
  c->kp.n = c->n;
  const Parts p = parts_of(s);
  const dim3 grid(c->walk_blocks), block(64);
  switch (c->kp.n_group) {
    case 4:
      hipLaunchKernelGGL((k_neighbours<16>), grid, block, 0, c->stream, c->kp, p, mode, c->wnode,
                         c->ginfo, counts, offsets, idx, c->walk_spill, c->ds);
      break;
    case 8:
      hipLaunchKernelGGL((k_neighbours<8>), grid, block, 0, c->stream, c->kp, p, mode, c->wnode,
                         c->ginfo, counts, offsets, idx, c->walk_spill, c->ds);
      break;
    case 16:
      hipLaunchKernelGGL((k_neighbours<4>), grid, block, 0, c->stream, c->kp, p, mode, c->wnode,
                         c->ginfo, counts, offsets, idx, c->walk_spill, c->ds);
      break;
    default:
      hipLaunchKernelGGL((k_neighbours<2>), grid, block, 0, c->stream, c->kp, p, mode, c->wnode,
                         c->ginfo, counts, offsets, idx, c->walk_spill, c->ds);
      break;
  }
  return hipGetLastError();
}

}  // namespace sph
