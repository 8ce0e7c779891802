// sph_internal.h -- device-side building blocks and the context layout of
// the gfx950 SPH library.  Not part of the public ABI (include/sph.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sph.h"

namespace sph {

constexpr int kKeyLevels = 21;  // 21 bits per axis -> levels 1..21
constexpr int kLevels = 22;     // tree levels 0..21
constexpr int kWave = 64;

// ---- device error word bits ------------------------------------------------
enum : uint32_t {
  kErrNoConv = 1u,
  kErrNodes = 2u,      // tree node capacity
  kErrFrontier = 4u,   // walk frontier capacity
  kErrPairs = 8u,      // per-particle pair list capacity
  kErrDomain = 16u,    // 2h >= L/2 on a periodic axis
  kErrNonFinite = 32u,
  kErrLeaves = 64u,
  kErrFrontierForce = 128u,  // walk frontier capacity in the force pass
  kErrIds = 256u,            // a particle id outside [0, n) (adjoint cotangent index)
  kErrSort = 512u,           // a radix-sort look-back wait ran out (should not happen)
};

// Fixed-point frame of the positions in the mixed-precision force records.
// Axis a maps x to the code floor((x - o[a]) inv[a]): on a periodic axis inv
// = 2^32 / L and the code is kept modulo 2^32, so the wrapped 32-bit
// difference of two codes is the nearest periodic image; on an open axis the
// frame spans the root node's box with 2^31 codes (clamped), so a difference
// never wraps.  Code difference times step[a] is the separation to within one
// step (L 2^-32 on a periodic axis), with no FP64 arithmetic and no fold.
struct QFrame {
  double o[3];
  double inv[3];
  float step[3];
  int32_t pad;
};

__device__ __forceinline__ int32_t qcode(double x, const QFrame& f, int a, int periodic) {
  const double t = floor((x - f.o[a]) * f.inv[a]);
  if (periodic) return (int32_t)(uint32_t)(uint64_t)(int64_t)t;  // modulo 2^32
  return (int32_t)fmin(fmax(t, 0.0), 2147483647.0);
}

// Separation a - b of two codes of one axis (wrapped 32-bit difference).
__device__ __forceinline__ float qsep(int32_t a, int32_t b, float step) {
  return (float)(int32_t)((uint32_t)a - (uint32_t)b) * step;
}

// Work counts and the Courant minimum, which every wavefront of the list and
// walk kernels adds to once, when it ends.  On small and mid-sized sets all of
// them end together, and their atomics on one set of counters queued up: 13 to
// 37 us of every such kernel (32^3 FP64: lists 86 -> 65 us, density 62 -> 26,
// force 75 -> 49 with the counts spread; 294,912 mixed: 193 -> 176, 111 -> 98,
// 161 -> 132).  So there are kTallies sets, 128 bytes apart; a block adds to
// set blockIdx mod kTallies (all blocks of a set run on one XCD), and the
// readers combine them.
constexpr int kTallies = 64;
struct alignas(128) WaveTally {
  unsigned long long n_pairs_density;   // true neighbours (r < 2h) at the final pass
  unsigned long long n_pairs_force;     // force pairs
  unsigned long long n_sums_density;    // sum over groups of (density passes * pairs)
  unsigned long long n_cand_density;    // candidate tests in the density walks
  unsigned long long n_cand_force;      // candidate tests in the force walks
  unsigned long long tot_sums_density;  // n_sums_density over every launch so far
  unsigned long long tot_pairs_force;   // n_pairs_force over every launch so far
  unsigned long long tot_cand_lists;    // candidate tests of the list kernel so far
  unsigned long long dt_min_enc;        // ordered encoding of min_i c_cour h_i / vsig_i
  int32_t max_iter;                     // most density sums any group needed
  int32_t n_rewalk;
};

// Device-resident scalars of one context.
struct DevState {
  int32_t n_nodes;
  int32_t n_groups;
  int32_t leaf_state;     // 0: no stored leaf lists, 1: valid for the force, 2: some h outgrew them
  int32_t lists_missing;  // some group needs the walking kernels (h refresh needed)
  int32_t n_flag_rows;    // groups whose neighbour-list rows overflowed (walking kernels)
  int32_t n_flag_grew;    // groups in which some h outgrew the rows (walking kernels)
  int32_t n_flagged;      // entries of the flagged-group list (both kinds)
  int32_t pool_used;      // entries taken from the pool of single groups' leaf lists
  double dt_cur;          // step used by the running sph_step
  alignas(256) uint32_t err;
  alignas(256) QFrame qf;  // frame of the mixed force records (set with each tree's node boxes)
  WaveTally tally[kTallies];
};

// Walk view of a tree node: centre, conservative half-widths, largest h.
struct alignas(16) WalkNode {
  double c[3];
  float w[3];    // half-widths rounded up
  float hmax;    // largest smoothing length, rounded up
  int32_t first;
  int32_t count;
  int32_t child;   // first child (children are contiguous); -1 for leaves
  int32_t nchild;  // 0 for leaves
};
static_assert(sizeof(WalkNode) == 56 || sizeof(WalkNode) == 64, "WalkNode layout");

struct alignas(16) GroupInfo {
  double c[3];
  double w[3];
  double hmax;
  int32_t first;
  int32_t count;
};

// Parameters as the kernels see them.
struct KParams {
  double lo[3];
  double len[3];
  double half[3];  // 0.5 * len (exact)
  double inv_len[3];
  int32_t periodic[3];
  double key_scale;  // 2^21 / max(len)
  double gamma, gm1, hfact, alpha, beta, alpha_u, c_cour;
  double h_tol;
  int32_t max_iter;
  int32_t fixed_passes;  // 1: three fixed passes (h_tol < 0)
  double h_margin;
  int32_t n;
  int32_t n_leaf;
  int32_t n_group;
  int32_t precision;
  int32_t kernel;   // 0 M4 cubic, 1 M6 quintic, 2 Wendland C6
  double support;   // kernel support in units of h (2, 3, 2)
  double knorm;     // 3D normalisation C of W = C f(r/h) / h^3
  int32_t nl_cap;   // entries per neighbour-list row (128 or 256)
};

// ---- small device helpers ---------------------------------------------------
__device__ __forceinline__ int lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
__device__ __forceinline__ uint64_t lanemask_lt() {
  int l = lane_id();
  return (l == 0) ? 0ull : (~0ull >> (64 - l));
}
__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }
__device__ __forceinline__ int popc64(uint64_t x) { return __popcll(x); }

// Marks a loaded value as used here whatever becomes of it, so that the
// compiler neither sinks its load into a later condition nor serialises a
// batch of loads that are meant to be in flight together.
template <typename T>
__device__ __forceinline__ void loaded(T& v) {
  asm volatile("" : "+v"(v));
}

// v of lane (l ^ D).  Distances below 16 stay within a row of 16 lanes and go
// by DPP (a VALU move, no LDS round trip): quad permutations for 1 and 2, the
// two row shifts by 4 on alternate banks of 4 lanes for 4, a row rotation by
// 8 for 8.  Called with every lane of the wavefront active.
template <int D>
__device__ __forceinline__ uint32_t xor_lane_u32(uint32_t v) {
  if constexpr (D == 1) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);
  } else if constexpr (D == 2) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);
  } else if constexpr (D == 4) {
    const int up = __builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xf, 0x5, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)v, 0x114, 0xf, 0xa, false);
  } else if constexpr (D == 8) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);
  } else {
    return (uint32_t)__shfl_xor((int)v, D, kWave);
  }
}
template <int D>
__device__ __forceinline__ double xor_lane_f64(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = xor_lane_u32<D>((uint32_t)b), hi = xor_lane_u32<D>((uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the LPI consecutive lanes of a particle slot (aligned segments),
// the farthest lanes first.  The two and four lanes of groups of 32 and 16, whose
// walking kernels wait for other things, take shuffles: their density is 7 and
// 1 % slower by DPP (16^3 mixed 523 against 484 us, 80^3 1602 against 1582).
template <int LPI>
__device__ __forceinline__ double seg_sum(double v) {
  if constexpr (LPI <= 4) {
#pragma unroll
    for (int d = LPI / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
  }
  if constexpr (LPI > 32) v += xor_lane_f64<32>(v);
  if constexpr (LPI > 16) v += xor_lane_f64<16>(v);
  if constexpr (LPI > 8) v += xor_lane_f64<8>(v);
  v += xor_lane_f64<4>(v);
  v += xor_lane_f64<2>(v);
  v += xor_lane_f64<1>(v);
  return v;
}
template <int LPI>
__device__ __forceinline__ double seg_max(double v) {
  if constexpr (LPI > 32) v = fmax(v, xor_lane_f64<32>(v));
  if constexpr (LPI > 16) v = fmax(v, xor_lane_f64<16>(v));
  if constexpr (LPI > 8) v = fmax(v, xor_lane_f64<8>(v));
  if constexpr (LPI > 4) v = fmax(v, xor_lane_f64<4>(v));
  if constexpr (LPI > 2) v = fmax(v, xor_lane_f64<2>(v));
  if constexpr (LPI > 1) v = fmax(v, xor_lane_f64<1>(v));
  return v;
}
template <int LPI>
__device__ __forceinline__ double seg_min(double v) {
  if constexpr (LPI > 32) v = fmin(v, xor_lane_f64<32>(v));
  if constexpr (LPI > 16) v = fmin(v, xor_lane_f64<16>(v));
  if constexpr (LPI > 8) v = fmin(v, xor_lane_f64<8>(v));
  if constexpr (LPI > 4) v = fmin(v, xor_lane_f64<4>(v));
  if constexpr (LPI > 2) v = fmin(v, xor_lane_f64<2>(v));
  if constexpr (LPI > 1) v = fmin(v, xor_lane_f64<1>(v));
  return v;
}
template <int LPI>
__device__ __forceinline__ uint32_t seg_sum_u32(uint32_t v) {
  if constexpr (LPI <= 4) {
#pragma unroll
    for (int d = LPI / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
  }
  if constexpr (LPI > 32) v += xor_lane_u32<32>(v);
  if constexpr (LPI > 16) v += xor_lane_u32<16>(v);
  if constexpr (LPI > 8) v += xor_lane_u32<8>(v);
  v += xor_lane_u32<4>(v);
  v += xor_lane_u32<2>(v);
  v += xor_lane_u32<1>(v);
  return v;
}
__device__ __forceinline__ int wave_max_i32(int v) {
  v = max(v, (int)xor_lane_u32<1>((uint32_t)v));
  v = max(v, (int)xor_lane_u32<2>((uint32_t)v));
  v = max(v, (int)xor_lane_u32<4>((uint32_t)v));
  v = max(v, (int)xor_lane_u32<8>((uint32_t)v));
  v = max(v, (int)xor_lane_u32<16>((uint32_t)v));
  v = max(v, (int)xor_lane_u32<32>((uint32_t)v));
  return v;
}

// ---- gathers of per-particle records through LDS ------------------------------
// A wavefront gathers one record of 16 RB bytes per lane.  Loaded by its own
// lane, a record costs the L1 an access per 16 bytes and lane (each dwordx4 of
// 64 scattered lanes takes the L1 about 40 cycles); here RB consecutive lanes
// load one record's bytes together, straight into LDS (64 bytes per access),
// and each lane then reads its record from there.  The pieces of a record sit
// permuted (slot = piece ^ key) so that the reads of 8 consecutive lanes fall
// in distinct banks of 32; over the 64 banks two of 16 lanes still meet, and the
// conflict counter shows it (3.7e8 per launch at 16.8M particles, 0 without LDS;
// the wait for LDS rose from 1.2e7 to 1.4e8).
typedef int Piece __attribute__((ext_vector_type(4)));

template <int RB>
struct LdsGather {
  static_assert(RB == 4 || RB == 8, "records of 64 or 128 bytes");
  static constexpr int kBytes = 64 * 16 * RB;  // LDS of one set of 64 records
  const char* base;  // the records, at this lane's piece
  int src;           // ds_bpermute address of the first load's source lane
  uint32_t at0;      // LDS address of this lane's piece 0

  // lds: this wavefront's buffer of kBytes, aligned to a record
  __device__ __forceinline__ LdsGather(const void* records, char* lds, int lane) {
    base = static_cast<const char*>(records) + 16 * ((lane & (RB - 1)) ^ ((lane >> 3) & (RB - 1)));
    src = 4 * (lane / RB);
    const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const int key = RB == 4 ? (lane >> 1) & 3 : lane & 7;
    at0 = a + 16u * (uint32_t)(RB * lane + key);
  }

  // Starts the loads of record j of every lane (none if j < 0) into the buffer
  // `buf`; every earlier read of it is complete (read() waits).
  __device__ __forceinline__ void start(char* buf, int j) const {
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int je = __builtin_amdgcn_ds_bpermute(src + q * (4 * 64 / RB), j);
      if (je >= 0)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(base + (int64_t)je * (16 * RB)),
            (__attribute__((address_space(3))) void*)(buf + q * 1024), 16, 0, 0);
    }
  }

  // All loads started so far are in LDS (and all other loads done).
  static __device__ __forceinline__ void wait() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }

  // This lane's record.  The reads and their wait are one statement: the next
  // start() overwrites the buffer.
  __device__ __forceinline__ void read(Piece (&r)[RB]) const {
    // piece k sits at slot k ^ key of the (aligned) record: its address is
    // piece 0's with the bits of 16 k flipped
    uint32_t at[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) at[k] = at0 ^ (16u * (uint32_t)k);
    if constexpr (RB == 4) {
      asm volatile(
          "ds_read_b128 %0, %4\n\t"
          "ds_read_b128 %1, %5\n\t"
          "ds_read_b128 %2, %6\n\t"
          "ds_read_b128 %3, %7\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
          : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3])
          : "memory");
    } else {
      asm volatile(
          "ds_read_b128 %0, %8\n\t"
          "ds_read_b128 %1, %9\n\t"
          "ds_read_b128 %2, %10\n\t"
          "ds_read_b128 %3, %11\n\t"
          "ds_read_b128 %4, %12\n\t"
          "ds_read_b128 %5, %13\n\t"
          "ds_read_b128 %6, %14\n\t"
          "ds_read_b128 %7, %15\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]),
            "=&v"(r[6]), "=&v"(r[7])
          : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]),
            "v"(at[7])
          : "memory");
    }
  }
};

// Order-preserving map of doubles to unsigned 64-bit integers, so that
// atomicMin / atomicMax on the integers implement min / max on the doubles.
__host__ __device__ __forceinline__ unsigned long long enc_f64(double x) {
  unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__host__ __device__ __forceinline__ double dec_f64(unsigned long long e) {
  unsigned long long b = (e >> 63) ? (e & 0x7fffffffffffffffull) : ~e;
  return __builtin_bit_cast(double, b);
}

}  // namespace sph

// Host-side launchers implemented in sph_kernels.hip.
struct sph_ctx;
namespace sph {
hipError_t launch_predict_keys(sph_ctx* c, const sph_particles* p, bool predict, double dt_host);
hipError_t launch_sort(sph_ctx* c);
hipError_t launch_permute(sph_ctx* c, const sph_particles* p, bool outputs_too);
hipError_t launch_tree(sph_ctx* c);
hipError_t launch_node_h(sph_ctx* c, const sph_particles* p, bool always);
bool lists_mode(const sph_ctx* c);
hipError_t launch_lists(sph_ctx* c, const sph_particles* p);
hipError_t launch_density_lists(sph_ctx* c, const sph_particles* p);
hipError_t launch_density(sph_ctx* c, const sph_particles* p, bool flagged_only);
hipError_t launch_force_lists(sph_ctx* c, const sph_particles* p, bool step_mode);
hipError_t launch_row_sets(sph_ctx* c, const sph_particles* p, int mode, int32_t* counts,
                           int32_t* idx, const int64_t* offsets);
hipError_t launch_force(sph_ctx* c, const sph_particles* p, bool step_mode, bool flagged_only);
hipError_t launch_correct(sph_ctx* c, const sph_particles* p);
hipError_t launch_reduce(sph_ctx* c, const sph_particles* p, double* out);
hipError_t reduce_noalloc(const sph_particles* p, hipStream_t stream, double* out);
hipError_t launch_neighbours(sph_ctx* c, const sph_particles* p, int mode, int32_t* counts,
                             const int64_t* offsets, int32_t* idx);
// implemented in sph_adjoint.hip
// part 0: seed, 1: force adjoint, 2: density adjoint and final combination
hipError_t launch_adjoint(sph_ctx* c, const sph_particles* p, const sph_cotangents* g, double dt,
                          bool step_mode, int part);
}  // namespace sph
