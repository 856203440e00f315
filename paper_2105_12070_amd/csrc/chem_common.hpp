// Shared definitions of the HIP path: packed mechanism layout (written by the
// host packer, read by the kernels), Rosenbrock tables, kernel arguments and
// wavefront primitives for gfx950 (wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace chem {

constexpr double RU = 8.314462618e7;  // gas constant, erg/(mol K)
constexpr double PATM = 1.01325e6;     // standard-state pressure, dyn/cm^2
constexpr int MAXTB = 8;               // non-unit third-body efficiencies per reaction
constexpr int WAVE = 64;

enum CellStatus { ST_OK = 0, ST_TOO_MANY = 1, ST_UNDERFLOW = 2, ST_SINGULAR = 3, ST_NONFINITE = 4, ST_TAPE = 5 };

// Packed mechanism.  Reactions are stored sorted by type: [0,R0) elementary,
// [R0,R1) third-body, [R1,R) Troe.  Empty molecule slots and unused efficiency
// slots point at the padding species index K, whose concentration is 1 and
// whose g/RT and h/RT are 0, so the kernels need no branches for them.
struct MechDims {
  int K, R, N, S;  // species, reactions, N = K+1, LDS row stride of J (odd, >= N+1)
  int R0, R1;      // type boundaries
  int L;           // species->reaction incidence entries
  // byte offsets inside the LDS-staged blob
  int o_lnA, o_b, o_th, o_sp, o_W, o_iW, o_cptr, o_cent;
  int o_tbp, o_tbs, o_tbd, o_troe;  // third-body lists and Troe data
  int lds_bytes;   // size of the staged blob (multiple of 16)
};

// Third-body / Troe reaction r >= R0 has the non-unit efficiencies
// tbs[e], 1 + tbd[e] for e in [tbp[r-R0], tbp[r-R0+1]) (at most MAXTB).
// Troe data per falloff reaction: alpha, 1/T***, 1/T*, T**, lnA0, b0, theta0, 0.
constexpr int TROE_STRIDE = 8;

// Rosenbrock method in the transformed form (Hairer & Wanner IV.7):
//   M = I/(gamma h) - J,  M K_i = f(y + sum_j a_ij K_j) + sum_j (c_ij/h) K_j,
//   y_new = y + sum m_i K_i,  err = sum e_i K_i.
// Stage i as the integrators walk it: the coefficients of K_{i-1}, K_{i-2},
// K_{i-3} (0 where there is no such stage), one aligned 64-byte row.  Bound:
// the latency of the scalar loads; six of them, each behind its own branch, and
// eight more for m and e took 19.8 ms for 1,024 cells of 10 species and 600 ms
// for 262,144 of 54, the rows 19.1 and 595.
struct alignas(64) RosStage {
  double a[3], c[3];
  int newf;         // stage i > 0 evaluates f at a point no earlier stage used
  int pad[3];
};
struct RosTable {
  RosStage stage[4];
  double mr[4], er[4];  // m and e, last stage first
  int s;
  int src[4];       // the stage whose f evaluation stage i uses
  double gamma;
  double a[4][4], c[4][4], m[4];  // the same by stage (the adjoint)
};

// 0: ROS4 with Shampine's parameters (as tabulated by Sandu et al. 1997),
// order 4 with an embedded order-3 estimate; 1: Rodas3 (Sandu et al. 1997),
// stiffly accurate, order 3(2).
constexpr RosTable ros_table(int s, const int (&newf)[4], const int (&src)[4], double gamma, const double (&a)[4][4],
                             const double (&c)[4][4], const double (&m)[4], const double (&e)[4]) {
  RosTable t{};
  t.s = s;
  t.gamma = gamma;
  for (int i = 0; i < 4; ++i) {
    t.src[i] = src[i];
    t.m[i] = m[i];
    t.stage[i].newf = i > 0 ? newf[i] : 0;
    for (int j = 0; j < 4; ++j) {
      t.a[i][j] = a[i][j];
      t.c[i][j] = c[i][j];
    }
    for (int j = 0; j < 3; ++j) {
      t.stage[i].a[j] = i > j ? a[i][i - 1 - j] : 0.0;
      t.stage[i].c[j] = i > j ? c[i][i - 1 - j] : 0.0;
    }
    t.mr[i] = i < s ? m[s - 1 - i] : 0.0;
    t.er[i] = i < s ? e[s - 1 - i] : 0.0;
  }
  return t;
}
__constant__ const RosTable kTables[2] = {
    ros_table(4, {0, 1, 1, 0}, {0, 1, 2, 2}, 0.57282,
              {{0, 0, 0, 0}, {2.0, 0, 0, 0}, {1.867943637803922, 0.2344449711399156, 0, 0},
               {1.867943637803922, 0.2344449711399156, 0.0, 0}},
              {{0, 0, 0, 0}, {-7.137615036412310, 0, 0, 0}, {2.580708087951457, 0.6515950076447975, 0, 0},
               {-2.137148994382534, -0.3214669691237626, -0.6949742501781779, 0}},
              {2.255570073418735, 0.2870493262186792, 0.4353179431840180, 1.093502252409163},
              {-0.2815431932141155, -0.07276199124938920, -0.1082196201495311, -1.093502252409163}),
    ros_table(4, {0, 0, 1, 1}, {0, 0, 2, 3}, 0.5,
              {{0, 0, 0, 0}, {0, 0, 0, 0}, {2.0, 0, 0, 0}, {2.0, 0, 1.0, 0}},
              {{0, 0, 0, 0}, {4.0, 0, 0, 0}, {1.0, -1.0, 0, 0}, {1.0, -1.0, -8.0 / 3.0, 0}},
              {2.0, 0.0, 1.0, 1.0}, {0.0, 0.0, 0.0, 1.0})};

struct Controller {
  int max_steps;
  double fac_safe, fac_min, fac_max, h_min;
};

// Arguments of the integration kernels.
struct IntArgs {
  const uint8_t* blob;      // LDS-staged part of the mechanism (global copy)
  const double* nasa;       // [K][16] Tmid, lo a1..a7, hi a1..a7, pad
  const uint32_t* jsched;   // [jsched_it][64] species-scatter schedule of the Jacobian (wavefront path)
  int jsched_it;
  MechDims d;
  int method;               // index into kTables
  double q;                 // controller exponent 1/q (4 ROS4, 3 Rodas3)
  Controller ctl;
  double* state;            // [N][ld]
  int64_t ld, ncells;
  double* h;                // [ncells]
  double p;                 // dyn/cm^2
  double dt, rtol, atol;
  int32_t* steps;
  int32_t* rejects;
  int32_t* status;
  int* queue;               // persistent work cursor (NULL: one cell per wave slot)
  const int32_t* order;     // optional cell order for the queue
  const int* nactive;       // optional device count of queue entries (default ncells)
  int cell_doubles;         // per-wave LDS workspace in doubles
  int pool_slots;           // Jacobian slots shared by the workgroup's waves (0: every wave has its own)
  // adjoint tape (NULL in the forward integrator)
  double* tape_h;           // [ncells][max_tape]
  double* tape_y;           // [ncells][max_tape/ckpt + 1][N]
  int max_tape, ckpt;
  unsigned long long* prof; // [ncells][8] per-phase cycle counts, or NULL
  unsigned long long* failed; // cells that ended with a nonzero status (counter), or NULL
  int64_t fail_lu_lo, fail_lu_hi; // cells in [lo, hi) see every factorisation of M as singular (testing)
  int jac_fd;               // ablation (instrumented kernel only): finite-difference Jacobian
  int lu_nopiv;             // ablation (instrumented kernel only): LU without pivoting
};

// ------------------------------------------------------------ wave primitives
__device__ __forceinline__ int lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

__device__ __forceinline__ double readlane(double x, int l) {
  unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
  unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ int uniform_int(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ double uniform_double(double x) { return readlane(x, 0); }

__device__ __forceinline__ unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

template <unsigned CTRL>
__device__ __forceinline__ unsigned dpp(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
template <unsigned CTRL>
__device__ __forceinline__ double dpp(double x) {
  unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  unsigned lo = dpp<CTRL>((unsigned)u), hi = dpp<CTRL>((unsigned)(u >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// DPP controls: quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror
constexpr unsigned DPP_QP1032 = 0xB1, DPP_QP2301 = 0x4E, DPP_HMIRROR = 0x141, DPP_MIRROR = 0x140;

// Wave sum in a fixed order: pairwise within each row of 16 lanes (both
// partners add the same two operands, and IEEE addition commutes, so all lanes
// of a row agree bitwise), then the four row sums combined as (r0+r1)+(r2+r3).
__device__ __forceinline__ double wave_sum(double x) {
  x += dpp<DPP_QP1032>(x);
  x += dpp<DPP_QP2301>(x);
  x += dpp<DPP_HMIRROR>(x);
  x += dpp<DPP_MIRROR>(x);
  const double r0 = readlane(x, 0), r1 = readlane(x, 16), r2 = readlane(x, 32), r3 = readlane(x, 48);
  return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ unsigned wave_max_u32(unsigned x) {
  x = max(x, dpp<DPP_QP1032>(x));
  x = max(x, dpp<DPP_QP2301>(x));
  x = max(x, dpp<DPP_HMIRROR>(x));
  x = max(x, dpp<DPP_MIRROR>(x));
  // lane 15 of each row into the next row (rows 1 and 3), then lane 31 into the
  // upper half: lane 63 has the maximum (0, the identity, where nothing moves)
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
  return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}

// v[q] of lane block t (lanes 16 t .. 16 t + 15) <-> v[t] of lane block q: a 4 x 4
// transpose between the lane blocks and the registers, eight lane-swap
// instructions.  It is its own inverse.
typedef double dbl4 __attribute__((ext_vector_type(4)));
template <bool SWAP32>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
  unsigned lo[2], hi[2];
  if constexpr (SWAP32) {  // upper half of a <-> lower half of b
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
  } else {  // odd blocks of a <-> even blocks of b
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
  }
  a = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]);
  b = __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ void block_transpose(double (&v)[4]) {
  lane_swap<false>(v[0], v[1]);
  lane_swap<false>(v[2], v[3]);
  lane_swap<true>(v[0], v[2]);
  lane_swap<true>(v[1], v[3]);
}

// x with lane l's value replaced by the wave-uniform v (l uniform): v_writelane_b32,
// which has no clang builtin.
__device__ int amdgcn_writelane(int v, int l, int x) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int writelane(int v, int l, int x) { return amdgcn_writelane(v, l, x); }
__device__ __forceinline__ double writelane(double v, int l, double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v), w = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)amdgcn_writelane((int)(unsigned)u, l, (int)(unsigned)w);
  const unsigned hi = (unsigned)amdgcn_writelane((int)(unsigned)(u >> 32), l, (int)(unsigned)(w >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// f(integral_constant I), I = B .. E - 1, in straight-line code.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>());
    static_for<B + 1, E>(f);
  }
}

// Orders the wave's LDS traffic between phases in which lanes read what
// other lanes wrote.
// Waits until the wave's outstanding LDS operations (atomics without return
// included) have completed: s_waitcnt lgkmcnt(0), the other counters at their
// maximum.  Placed after each loop of LDS atomic accumulations, before the
// sums are read.
__device__ __forceinline__ void lds_wait() { __builtin_amdgcn_s_waitcnt(0xc07f); }

__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace chem
