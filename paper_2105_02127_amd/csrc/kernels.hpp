// HIP kernels of the TENO residual for gfx950 (MI355X), FP64.
//
//   k_reconstruct  blocks of four or eight wavefronts, one tile of 16 cells
//                  each, four lanes per cell.  Least-squares phase (Sec. 2.2 eqs. 08-10)
//                  without stored operators (below).  Selection phase: lane g
//                  holds the full coefficient vectors of variable g, forms the
//                  smoothness indicators (Sec. 2.3), the strong scale
//                  separation and the two-step ENO-like selection
//                  (Sec. 3.2-3.3), and the face Gauss-point states, written
//                  once.
//  k_face_flux     one lane per face: rotated HLL flux with Einfeldt/Roe wave
//                  speeds (Sec. 4) at the face's Gauss point pairs and the
//                  face quadrature, written once per face.
//  k_cell_update   one lane per cell: gather of its three face fluxes into
//                  the residual (Sec. 2.1), optional SSP-RK3 stage combine
//                  (a gather in a fixed order: no atomics, deterministic).
//  k_cell_flux_update  both in one launch, for small meshes.
//  k_dt_*          constant-CFL step: per-block minima, then one block.
//  k_adj_*         adjoint of the residual with the selection frozen.
//
// Lane-to-work mapping and tile layout are described in internal.h.
#pragma once
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "internal.h"
#include "tables.h"

namespace teno {

struct DevDiag {
  unsigned long long nonphysical;
  unsigned long long near_ties;
  unsigned long long fallbacks;
  long long first_bad;  // LLONG_MAX when none
};

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of tiles so that its L2 holds the neighbourhood it gathers.
__device__ __forceinline__ int xcd_remap(int b, int nblk) {
  const int X = 8;
  const int q = nblk / X, r = nblk % X;
  const int x = b % X, local = b / X;
  return x * q + (x < r ? x : r) + local;
}

// ---------------------------------------------------------------------------
// Euler helpers
// ---------------------------------------------------------------------------
// HLL flux through unit normal (nx, ny): rotate into the face frame, HLL with
// S_L = min(u_L - c_L, u~ - c~), S_R = max(u_R + c_R, u~ + c~) from Roe
// averages (both velocity components in c~), rotate back.  The quotients
// share four reciprocals (1/rho_L, 1/rho_R, 1/(1 + sqrt(rho_R/rho_L)),
// 1/(S_R - S_L)): FP64 division is a long instruction sequence and this
// function is most of the flux kernel's work.
__device__ __forceinline__ void hll(const double uL[4], const double uR[4], double nx, double ny,
                                    double g, double out[4]) {
  const double L0 = uL[0], L1 = nx * uL[1] + ny * uL[2], L2 = nx * uL[2] + (-ny) * uL[1], L3 = uL[3];
  const double R0 = uR[0], R1 = nx * uR[1] + ny * uR[2], R2 = nx * uR[2] + (-ny) * uR[1], R3 = uR[3];
  const double iL = 1.0 / L0, iR = 1.0 / R0;
  const double unL = L1 * iL, utL = L2 * iL, unR = R1 * iR, utR = R2 * iR;
  const double pL = (g - 1.0) * (L3 - (0.5 * L0) * (unL * unL + utL * utL));
  const double pR = (g - 1.0) * (R3 - (0.5 * R0) * (unR * unR + utR * utR));
  const double cL = sqrt(g * pL * iL), cR = sqrt(g * pR * iR);
  const double HL = (L3 + pL) * iL, HR = (R3 + pR) * iR;
  const double D = sqrt(R0 * iL);
  const double iden = 1.0 / (1.0 + D);
  const double ut = (unL + D * unR) * iden, vt = (utL + D * utR) * iden, Ht = (HL + D * HR) * iden;
  const double ct = sqrt((g - 1.0) * (Ht - 0.5 * (ut * ut + vt * vt)));
  const double a1 = unL - cL, a2 = ut - ct;
  const double SL = a2 < a1 ? a2 : a1;
  const double b1 = unR + cR, b2 = ut + ct;
  const double SR = b2 > b1 ? b2 : b1;
  const double FL[4] = {L1, L1 * unL + pL, L1 * utL, unL * (L3 + pL)};
  const double FR[4] = {R1, R1 * unR + pR, R1 * utR, unR * (R3 + pR)};
  const double UL[4] = {L0, L1, L2, L3};
  const double UR[4] = {R0, R1, R2, R3};
  double F[4];
  if (SL >= 0.0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) F[c] = FL[c];
  } else if (SR <= 0.0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) F[c] = FR[c];
  } else {
    const double iS = 1.0 / (SR - SL);
#pragma unroll
    for (int c = 0; c < 4; ++c) F[c] = (SR * FL[c] - SL * FR[c] + SL * SR * (UR[c] - UL[c])) * iS;
  }
  out[0] = F[0];
  out[1] = nx * F[1] - ny * F[2];
  out[2] = ny * F[1] + nx * F[2];
  out[3] = F[3];
}

// Reverse mode of hll (the same flux, the same branches): adds
// ob^T d(out)/d(uL) to gL and ob^T d(out)/d(uR) to gR.  The speed selections
// and the flux case follow the primal values, as the flux does.  One pass
// forward, one back: both sides' adjoints for about three times the flux's
// arithmetic.
__device__ __forceinline__ void hll_vjp(const double uL[4], const double uR[4], double nx,
                                        double ny, double g, const double ob[4], double gL[4],
                                        double gR[4]) {
  const double gm = g - 1.0;
  // ---- primal, keeping what the reverse pass needs ----
  const double L0 = uL[0], L1 = nx * uL[1] + ny * uL[2], L2 = nx * uL[2] + (-ny) * uL[1], L3 = uL[3];
  const double R0 = uR[0], R1 = nx * uR[1] + ny * uR[2], R2 = nx * uR[2] + (-ny) * uR[1], R3 = uR[3];
  const double iL = 1.0 / L0, iR = 1.0 / R0;
  const double unL = L1 * iL, utL = L2 * iL, unR = R1 * iR, utR = R2 * iR;
  const double qL = unL * unL + utL * utL, qR = unR * unR + utR * utR;
  const double pL = gm * (L3 - (0.5 * L0) * qL), pR = gm * (R3 - (0.5 * R0) * qR);
  const double cL = sqrt(g * pL * iL), cR = sqrt(g * pR * iR);
  const double EL = L3 + pL, ER = R3 + pR;  // rho H
  const double HL = EL * iL, HR = ER * iR;
  const double D = sqrt(R0 * iL);
  const double iden = 1.0 / (1.0 + D);
  const double nu = unL + D * unR, nv = utL + D * utR, nH = HL + D * HR;
  const double ut = nu * iden, vt = nv * iden, Ht = nH * iden;
  const double ct = sqrt(gm * (Ht - 0.5 * (ut * ut + vt * vt)));
  const double a1 = unL - cL, a2 = ut - ct;
  const bool l2 = a2 < a1;
  const double SL = l2 ? a2 : a1;
  const double b1 = unR + cR, b2 = ut + ct;
  const bool r2 = b2 > b1;
  const double SR = r2 ? b2 : b1;
  const double FL[4] = {L1, L1 * unL + pL, L1 * utL, unL * EL};
  const double FR[4] = {R1, R1 * unR + pR, R1 * utR, unR * ER};
  const double UL[4] = {L0, L1, L2, L3}, UR[4] = {R0, R1, R2, R3};
  // ---- reverse ----
  // out = (F0, nx F1 - ny F2, ny F1 + nx F2, F3)
  const double Fb[4] = {ob[0], nx * ob[1] + ny * ob[2], nx * ob[2] - ny * ob[1], ob[3]};
  double FLb[4] = {0.0, 0.0, 0.0, 0.0}, FRb[4] = {0.0, 0.0, 0.0, 0.0};
  double Lb[4] = {0.0, 0.0, 0.0, 0.0}, Rb[4] = {0.0, 0.0, 0.0, 0.0};
  double SLb = 0.0, SRb = 0.0;
  if (SL >= 0.0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) FLb[c] = Fb[c];
  } else if (SR <= 0.0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) FRb[c] = Fb[c];
  } else {
    // F_c = N_c iS, N_c = SR FL_c - SL FR_c + SL SR (UR_c - UL_c), iS = 1 / (SR - SL)
    const double iS = 1.0 / (SR - SL);
    double iSb = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double dU = UR[c] - UL[c];
      const double N = SR * FL[c] - SL * FR[c] + SL * SR * dU;
      const double Nb = Fb[c] * iS;
      iSb += Fb[c] * N;
      FLb[c] = SR * Nb;
      FRb[c] = -SL * Nb;
      SRb += Nb * (FL[c] + SL * dU);
      SLb += Nb * (SR * dU - FR[c]);
      Rb[c] += SL * SR * Nb;
      Lb[c] -= SL * SR * Nb;
    }
    const double t = -iS * iS * iSb;  // d(iS) = -iS^2 d(SR - SL)
    SRb += t;
    SLb -= t;
  }
  // the physical fluxes
  Lb[1] += FLb[0] + FLb[1] * unL + FLb[2] * utL;
  Rb[1] += FRb[0] + FRb[1] * unR + FRb[2] * utR;
  double unLb = FLb[1] * L1 + FLb[3] * EL, unRb = FRb[1] * R1 + FRb[3] * ER;
  double utLb = FLb[2] * L1, utRb = FRb[2] * R1;
  double pLb = FLb[1], pRb = FRb[1];
  double ELb = FLb[3] * unL, ERb = FRb[3] * unR;
  // the wave-speed estimates
  const double a1b = l2 ? 0.0 : SLb, a2b = l2 ? SLb : 0.0;
  const double b1b = r2 ? 0.0 : SRb, b2b = r2 ? SRb : 0.0;
  unLb += a1b;
  const double cLb = -a1b;
  unRb += b1b;
  const double cRb = b1b;
  double utb = a2b + b2b;
  const double ctb = b2b - a2b;
  // ct = sqrt(X), X = (g - 1) (Ht - (ut^2 + vt^2) / 2)
  const double Xb = ctb * 0.5 / ct;
  const double Htb = gm * Xb;
  utb -= gm * ut * Xb;
  const double vtb = -gm * vt * Xb;
  // Roe averages: ut = nu iden, vt = nv iden, Ht = nH iden
  const double nub = utb * iden, nvb = vtb * iden, nHb = Htb * iden;
  const double idenb = utb * nu + vtb * nv + Htb * nH;
  unLb += nub;
  unRb += D * nub;
  utLb += nvb;
  utRb += D * nvb;
  const double HLb = nHb, HRb = D * nHb;
  double Db = unR * nub + utR * nvb + HR * nHb - iden * iden * idenb;
  // D = sqrt(R0 iL)
  const double Yb = Db * 0.5 / D;
  Rb[0] += Yb * iL;
  double iLb = Yb * R0, iRb = 0.0;
  // H = (E + p) / rho
  ELb += HLb * iL;
  iLb += HLb * EL;
  ERb += HRb * iR;
  iRb += HRb * ER;
  // c = sqrt(g p / rho)
  const double ZLb = cLb * 0.5 / cL, ZRb = cRb * 0.5 / cR;
  pLb += g * iL * ZLb + ELb;
  iLb += g * pL * ZLb;
  pRb += g * iR * ZRb + ERb;
  iRb += g * pR * ZRb;
  Lb[3] += ELb;
  Rb[3] += ERb;
  // p = (g - 1) (E - rho q / 2)
  Lb[3] += gm * pLb;
  Rb[3] += gm * pRb;
  Lb[0] -= 0.5 * gm * qL * pLb;
  Rb[0] -= 0.5 * gm * qR * pRb;
  const double qLb = -0.5 * gm * L0 * pLb, qRb = -0.5 * gm * R0 * pRb;
  unLb += 2.0 * unL * qLb;
  utLb += 2.0 * utL * qLb;
  unRb += 2.0 * unR * qRb;
  utRb += 2.0 * utR * qRb;
  // un = m_n / rho, ut = m_t / rho
  Lb[1] += unLb * iL;
  Lb[2] += utLb * iL;
  iLb += unLb * L1 + utLb * L2;
  Rb[1] += unRb * iR;
  Rb[2] += utRb * iR;
  iRb += unRb * R1 + utRb * R2;
  Lb[0] -= iL * iL * iLb;
  Rb[0] -= iR * iR * iRb;
  // the rotation into the face frame
  gL[0] += Lb[0];
  gL[1] += nx * Lb[1] - ny * Lb[2];
  gL[2] += ny * Lb[1] + nx * Lb[2];
  gL[3] += Lb[3];
  gR[0] += Rb[0];
  gR[1] += nx * Rb[1] - ny * Rb[2];
  gR[2] += ny * Rb[1] + nx * Rb[2];
  gR[3] += Rb[3];
}

// ---------------------------------------------------------------------------
// Least-squares phase (Sec. 2.2 eqs. 08-10), without stored operators.
//
// With rows A_s (moments of member s about the target, zero mean over it) and
// weights w_s = |V_s|^2, the coefficients of one stencil are
//   a = N sum_s w_s A_s (U_s - U_0),   N = (sum_s w_s A_s A_s^T)^-1.
// Stored operators a = M d are n_u x n_l doubles per cell and stage (4.6 KB at
// order 5) and bound this kernel to HBM: 461 us per launch on 524,288 cells at
// order 5 (5.7 TB/s).  N is symmetric (1.2 KB), and A_s follows from the
// member's own central moments by a Taylor shift, a few multiply-adds per entry
// from a record that the whole block shares: 285 to 315 us by state, bound by
// vector issue (67% of the SIMDs' cycles: 3,140 instructions a tile, seven tenths
// of them FP64) with memory at 3.5 TB/s.  At orders 3, 4, 6 (180,000 cells):
// 73, 105, 270 us stored, 49, 65, 165 us like this.
//
// Precision: the normal matrix squares the condition of A, so the basis is
// chosen to keep that small: moments in a frame that gives the block's
// displacements unit variance, of Hermite polynomials (they shift by the same
// binomial rule as monomials), about the mean of each stencil's members; N is
// formed and inverted in extended precision.  Against 128 bits the face values
// are closer than the stored operators' (rms error 0.44, 0.13, 0.07, 0.02 of
// theirs at orders 3-6 on jittered meshes).  Set-up bounds every stencil's error
// and leaves cells where it would exceed an operator's to k_reconstruct_kept.
//
// A block of wavefronts (16 cells each, four lanes per cell) stages the distinct
// members of all its stencils in LDS: about 190 records and states for four
// wavefronts and 300 for eight, 2.3 to 3 per cell, where one wavefront alone
// would stage 7.  Lane g of a cell owns rows 4j + g of each stencil and adds
// them for all four variables.  Its accumulators and differences are ordered by
// i = v xor g, so that the sum over the cell's four lanes hands lane g variable
// g by three DPP exchanges of whole registers, without selects.  The sum's order
// is fixed: results do not depend on timing.
// ---------------------------------------------------------------------------
struct BlockArgs {
  const int* __restrict__ boff;        // [n_blocks + 1] first member of a block
  const int* __restrict__ bmem;        // [block][mstride] member cells, the block's own first
  const double2* __restrict__ brec;    // geometry records (internal.h)
  const unsigned* __restrict__ bslot;  // [n_tiles][slot_words][64] row slots
  const double2* __restrict__ N;       // [n_tiles][normal_quads][64]
  const double2* __restrict__ jac;     // [n_pad][2]
  const float2* __restrict__ centre;   // [n_pad][4] centre of each stencil's basis
  const int* __restrict__ pack;        // [n_pad] cell of each packed position, -1: none or kept
  int bwaves;                          // wavefronts (tiles) per block
  int mstride;                         // members of the mesh's largest block
  int bmax;                            // of all the launch's meshes: lays out the LDS
  int nbuf;                            // staged blocks in LDS (2 or 1)
};

// Arguments in constant memory (a kernel's own, or a batch's descriptors):
// fields are loaded through the scalar cache where they are used.
#define TENO_CONST const __attribute__((address_space(4)))

// LDS of a reconstruction workgroup: nbuf staged blocks (states at 0, records at
// 32 bmax), then nbuf lists of member ids.  The stride is formed here and not
// loaded: the compiler has to know it for a multiple of 16 to read the records 16
// bytes at a time (8 at a time cost order 6 a quarter: 831 against 670 us a step
// on 204,800 cells).
template <int NU, bool CH>
__device__ __forceinline__ int stride_of(TENO_CONST BlockArgs& b) {
  if constexpr (CH) return 16 * (buffer_stride(NU, b.bmax, b.bwaves, true) / 16);
  else return block_lds_bytes(NU, b.bmax);
}
template <int NU, bool CH>
__device__ __forceinline__ unsigned buf_offset(TENO_CONST BlockArgs& b, int k) {
  return buffer_offset(stride_of<NU, CH>(b), b.nbuf, k);
}
template <int NU, bool CH>
__device__ __forceinline__ unsigned list_offset(TENO_CONST BlockArgs& b, int k) {
  return ids_offset(stride_of<NU, CH>(b), b.bmax, b.nbuf, k);
}

// Copies from memory straight to LDS (no registers): lane l's 16 (or 4) bytes
// go to lds + 16 l (4 l); lds is uniform.  The copies are counted with the
// wavefront's other memory operations and are complete after lds_copy_wait.
// In assembly, because the compiler waits for such a copy before any later LDS
// read; nothing is returned in a register.  m0 is named as clobbered because it is:
// the compiler warns that it will not save a reserved register, and need not.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_copy16(const void* src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(lds), "v"(src) : "m0", "memory");
}
__device__ __forceinline__ void lds_copy4(const void* src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :: "s"(lds), "v"(src) : "m0", "memory");
}
#pragma clang diagnostic pop
// A uniform load through the scalar cache (of data that no kernel writes); the
// copies' memory clobbers would otherwise turn it into a vector load.
__device__ __forceinline__ int scalar_load(const int* p, int i) {
  return ((const __attribute__((address_space(4))) int*)(uintptr_t)p)[i];
}
__device__ __forceinline__ void lds_copy_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int K>
__device__ __forceinline__ double quad_perm_dpp(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), K, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), K, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// Broadcast lane K of every group of four lanes (DPP quad permutation).
template <int K>
__device__ __forceinline__ double quad_bcast(double x) {
  constexpr int ctrl = K * 0x55;  // quad_perm(K, K, K, K)
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), ctrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), ctrl, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// x of lane g ^ I of the quad
template <int I>
__device__ __forceinline__ double quad_xor(double x) {
  if constexpr (I == 0) return x;
  else return quad_perm_dpp<I == 1 ? 0xB1 : (I == 2 ? 0x4E : 0x1B)>(x);
}

// Sum over the cell's four lanes of variable g, from sums x[i] of variable
// i ^ g.  Called with all four lanes active.
__device__ __forceinline__ double quad_sum(const double (&x)[4]) {
  return (x[0] + quad_xor<1>(x[1])) + (quad_xor<2>(x[2]) + quad_xor<3>(x[3]));
}

// A constant table behind an opaque pointer: its entries come through the
// scalar cache where they are used, instead of as literals that the compiler
// collects in scalar registers for all their uses and spills.
__device__ __forceinline__ TENO_CONST double* table(const double* p) {
  auto q = (TENO_CONST double*)(uintptr_t)p;
  asm volatile("" : "+s"(q));
  return q;
}

__device__ __forceinline__ void opaque(double& x) { asm volatile("" : "+v"(x)); }

// Index of X^(d-k) Y^k in the graded basis.
constexpr int mono(int d, int k) { return d * (d + 1) / 2 - 1 + k; }

// Starts the copies of block blk's records (to rec), and of its members' states
// (to st), whose ids are at mem, by nthr threads.
template <int NU>
__device__ __forceinline__ void copy_records(TENO_CONST BlockArgs& b, int blk, unsigned rec, int nthr) {
  constexpr int RU = rec_units(NU);
  const int m0 = scalar_load(b.boff, blk), n = (scalar_load(b.boff, blk + 1) - m0) * RU;
  const char* src = reinterpret_cast<const char*>(b.brec) + (size_t)m0 * (16 * RU);
  const unsigned w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  for (int i = 0; i < n; i += nthr)
    if (i + (int)threadIdx.x < n) lds_copy16(src + 16 * (i + threadIdx.x), rec + 16 * (i + w0));
}
__device__ __forceinline__ void copy_states(const double* __restrict__ U, const int* mem, int nm,
                                            unsigned st, int nthr) {
  const unsigned w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  // ids two passes at a time: one wait for both
  for (int i = 0; i < 2 * nm; i += 2 * nthr) {
    const int k = i + threadIdx.x, k2 = k + nthr;
    const int id = k < 2 * nm ? mem[k >> 1] : 0, id2 = k2 < 2 * nm ? mem[k2 >> 1] : 0;
    if (k < 2 * nm) lds_copy16(U + (size_t)id * 4 + (k & 1) * 2, st + 16 * (i + w0));
    if (k2 < 2 * nm) lds_copy16(U + (size_t)id2 * 4 + (k & 1) * 2, st + 16 * (i + nthr + w0));
  }
}
__device__ __forceinline__ void copy_ids(TENO_CONST BlockArgs& b, int blk, unsigned ids, int nthr) {
  const int nm = scalar_load(b.boff, blk + 1) - scalar_load(b.boff, blk);
  const int* __restrict__ mem = b.bmem + (size_t)blk * b.mstride;
  const unsigned w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  for (int i = 0; i < nm; i += nthr)
    if (i + (int)threadIdx.x < nm) lds_copy4(mem + i + threadIdx.x, ids + 4 * (i + w0));
}

// The lane's row slots: NG groups, BITS bits each, packed in words [word][64].
template <int NG, int BITS>
struct RowSlots {
  static constexpr int PER = 32 / BITS, NW = (NG + PER - 1) / PER;
  unsigned w[NW];
  __device__ __forceinline__ void load(const unsigned* __restrict__ p, int tile, int lane) {
    const unsigned* __restrict__ t = p + (size_t)tile * (NW * 64);  // uniform
    static_for<0, NW>([&](auto k) { w[k] = t[k * 64 + (unsigned)lane]; });
  }
  template <int G>
  __device__ __forceinline__ unsigned get() const {
    return (w[G / PER] >> (BITS * (G % PER))) & ((1u << BITS) - 1);
  }
};
template <int NL>
using MemberSlots = RowSlots<lane_groups(NL), kSlotBits>;

// Moments E[H_a(x + X) H_b(y + Y)], 1 <= a + b <= R, from central moments mu
// (the record's order): a binomial shift along x, then along y.
template <int R>
__device__ __forceinline__ void shift_moments(double x, double y, const double* mu, double* out) {
  double t[R + 1][R + 1];
  static_for<0, R + 1>([&](auto bc) {
    constexpr int b = bc, n = R - b;
    double v[n + 1];
    static_for<0, n + 1>([&](auto ac) {
      constexpr int a = ac;
      if constexpr (a + b >= 2) v[a] = mu[mono(a + b, b) - 2];
    });
    // first pass, with mu_00 = 1 and mu_10 = mu_01 = 0 folded in
    constexpr int first = b == 0 ? 3 : (b == 1 ? 2 : 1);
    static_for<0, n + 1>([&](auto ac) {
      constexpr int a = n - ac;
      if constexpr (a >= first) v[a] = fma(x, v[a - 1], v[a]);
    });
    if constexpr (b == 0) v[1] = x;
    static_for<2, n + 1>([&](auto ic) {
      constexpr int i = ic;
      static_for<0, n + 1 - i>([&](auto ac) {
        constexpr int a = n - ac;
        v[a] = fma(x, v[a - 1], v[a]);
      });
    });
    static_for<1, n + 1>([&](auto ac) { t[ac][b] = v[ac]; });
    if constexpr (b >= 2) t[0][b] = v[0];
  });
  static_for<0, R + 1>([&](auto ac) {
    constexpr int a = ac, n = R - a;
    double v[n + 1];
    static_for<0, n + 1>([&](auto bc) {
      constexpr int b = bc;
      if constexpr (a + b >= 2 || a == 1) v[b] = t[a][b];
    });
    constexpr int first = a == 0 ? 3 : 1;
    static_for<0, n + 1>([&](auto bc) {
      constexpr int b = n - bc;
      if constexpr (b >= first) v[b] = fma(y, v[b - 1], v[b]);
    });
    if constexpr (a == 0) v[1] = y;
    static_for<2, n + 1>([&](auto ic) {
      constexpr int i = ic;
      static_for<0, n + 1 - i>([&](auto bc) {
        constexpr int b = n - bc;
        v[b] = fma(y, v[b - 1], v[b]);
      });
    });
    static_for<0, n + 1>([&](auto bc) {
      constexpr int b = bc;
      if constexpr (a + b >= 1) out[mono(a + b, b)] = v[b];
    });
  });
}

// A block as one cell's lane sees it.
struct CellView {
  const double* us;      // LDS: member states
  const double* geo;     // LDS: records
  double x, y;           // the cell's centroid
  double u0[4];          // its means, u0[i] = variable i ^ g
  int g;
};

// c = N r of one stencil.  Each lane of a cell loads a quarter of the packed
// triangle (a wavefront load is 1 KB, each byte once) and broadcasts its
// entries to the quad as they are used: two DPP moves an entry, where loading
// every entry in all four lanes took four times the loads and, with no
// registers to hold them ahead, a round trip to memory per few entries.  Two
// chunks of CH quads are in registers, one in flight while one is used.
template <int N, int CH = sym_quads(N)>
struct NormalMatrix {
  typedef double v2d __attribute__((ext_vector_type(2)));
  static constexpr int NQ = sym_quads(N), NE = N * (N + 1) / 2, NC = (NQ + CH - 1) / CH;
  v2d w[NC > 1 ? 2 : 1][CH];
  // loads chunk K of the stencil's matrix (p: its first quad, uniform)
  template <int K>
  __device__ __forceinline__ void load(const double2* __restrict__ p, int lane) {
    static_for<0, CH>([&](auto i) {
      constexpr int q = K * CH + i;
      if constexpr (q < NQ)
        w[K % 2][i] =
            __builtin_nontemporal_load(reinterpret_cast<const v2d*>(&p[q * 64 + (unsigned)lane]));
    });
  }
  static constexpr int row_of(int e) {
    int i = 0;
    while (e >= N - i) e -= N - i++;
    return i;
  }
  static constexpr int col_of(int e) {
    int i = 0;
    while (e >= N - i) e -= N - i++;
    return i + e;
  }
  // load<0> must have been called; called with all four lanes of the cell active
  __device__ __forceinline__ void apply(const double2* __restrict__ p, int lane, const double* r,
                                        double* c) {
    static_for<0, N>([&](auto l) { c[l] = 0.0; });
    static_for<0, NC>([&](auto k) {
      if constexpr (k + 1 < NC) {
        load<k + 1>(p, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
      static_for<0, 8 * CH>([&](auto ec) {
        constexpr int e = 8 * CH * k + ec;
        if constexpr (e < NE) {
          constexpr int i = row_of(e), j = col_of(e);
          const v2d x2 = w[k % 2][ec / 8];
          const double x = quad_bcast<(e / 2) % 4>(e % 2 ? x2.y : x2.x);
          c[i] = fma(x, r[j], c[i]);
          if constexpr (i != j) c[j] = fma(x, r[i], c[j]);
        }
      });
      if constexpr (k + 1 < NC) __builtin_amdgcn_sched_barrier(0);
    });
  }
};

// The map from the block's frame to the basis, x = j0 X + j1 Y and
// y = j2 X + j3 Y: forms y^k, k = 2..R, shared by the degrees.
template <int R>
struct Frame {
  double j0, j1, j2, j3;
  double yp[R + 1][R + 1];
  __device__ __forceinline__ void init(double2 a, double2 b) {
    j0 = a.x;
    j1 = a.y;
    j2 = b.x;
    j3 = b.y;
    yp[1][0] = j2;
    yp[1][1] = j3;
    static_for<2, R + 1>([&](auto kc) {
      constexpr int k = kc;
      yp[k][0] = j2 * yp[k - 1][0];
      static_for<1, k>([&](auto ic) {
        constexpr int i = ic;
        yp[k][i] = fma(j2, yp[k - 1][i], j3 * yp[k - 1][i - 1]);
      });
      yp[k][k] = j3 * yp[k - 1][k - 1];
    });
  }
  // coefficients of x^a y^b -> coefficients of X^a Y^b, degree by degree, in
  // place: p_0 = c_0, p_k = p_{k-1} x + c_k y^k
  template <int D>
  __device__ __forceinline__ void to_basis(double* c) const {
    static_for<1, D + 1>([&](auto dc) {
      constexpr int d = dc;
      double p[d + 1];
      p[0] = c[mono(d, 0)];
      static_for<1, d + 1>([&](auto kc) {
        constexpr int k = kc;
        const double ck = c[mono(d, k)];
        p[k] = fma(ck, yp[k][k], j1 * p[k - 1]);
        static_for<1, k>([&](auto ic) {
          constexpr int i = k - ic;
          p[i] = fma(ck, yp[k][i], fma(j0, p[i], j1 * p[i - 1]));
        });
        p[0] = fma(ck, yp[k][0], j0 * p[0]);
      });
      static_for<0, d + 1>([&](auto kc) { c[mono(d, kc)] = p[kc]; });
    });
  }
  // its transpose (adjoints of basis coefficients -> of frame coefficients)
  template <int D>
  __device__ __forceinline__ void from_basis_adjoint(double* c) const {
    static_for<1, D + 1>([&](auto dc) {
      constexpr int d = dc;
      double p[d + 1];
      static_for<0, d + 1>([&](auto kc) { p[kc] = c[mono(d, kc)]; });
      static_for<0, d>([&](auto kc) {
        constexpr int k = d - kc;
        double s = p[0] * yp[k][0];
        static_for<1, k + 1>([&](auto ic) { s = fma(p[ic], yp[k][ic], s); });
        c[mono(d, k)] = s;
        static_for<0, k>([&](auto ic) {
          constexpr int i = ic;
          p[i] = fma(j0, p[i], j1 * p[i + 1]);
        });
      });
      c[mono(d, 0)] = p[0];
    });
  }
};

// The cell's own moments about the centre (cx, cy).
template <int R>
__device__ __forceinline__ void own_moments(const double* own, double cx, double cy, bool shift,
                                            double* h) {
  constexpr int N = (R + 1) * (R + 2) / 2 - 1;
  h[0] = h[1] = 0.0;
  static_for<2, N>([&](auto l) { h[l] = own[l + 1]; });
  if (shift) {
    double t[N];
    shift_moments<R>(-cx, -cy, h + 2, t);
    static_for<0, N>([&](auto l) { h[l] = t[l]; });
  }
}

// Coefficients of H_a(x - cx) H_b(y - cy) -> coefficients of x^a y^b, in place
// (the constant is not kept): shifted to the cell's centroid, then expanded.
template <int R>
__device__ __forceinline__ void hermite_to_monomials(double* c, double cx, double cy, bool shift) {
  if (shift) {
    static_for<0, R>([&](auto bc) {
      constexpr int b = bc, n = R - b;
      static_for<0, n>([&](auto ic) {
        static_for<0, n - ic>([&](auto jc) {
          constexpr int a = n - 1 - jc;
          if constexpr (a + b >= 1)
            c[mono(a + b, b)] = fma(-cx, c[mono(a + 1 + b, b)], c[mono(a + b, b)]);
        });
      });
    });
    static_for<0, R>([&](auto ac) {
      constexpr int a = ac, n = R - a;
      static_for<0, n>([&](auto ic) {
        static_for<0, n - ic>([&](auto jc) {
          constexpr int b = n - 1 - jc;
          if constexpr (a + b >= 1)
            c[mono(a + b, b)] = fma(-cy, c[mono(a + b + 1, b + 1)], c[mono(a + b, b)]);
        });
      });
    });
  }
  static_for<0, R>([&](auto bc) {
    static_for<0, R + 1 - bc>([&](auto ac) {
      constexpr int a = ac, b = bc, n = R - b;
      if constexpr (a + b >= 1 && a + 2 <= n) {
        double v = fma(cx_hermite(a + 2, 1), c[mono(a + 2 + b, b)], c[mono(a + b, b)]);
        if constexpr (a + 4 <= n) v = fma(cx_hermite(a + 4, 2), c[mono(a + 4 + b, b)], v);
        c[mono(a + b, b)] = v;
      }
    });
  });
  static_for<0, R>([&](auto ac) {
    static_for<0, R + 1 - ac>([&](auto bc) {
      constexpr int a = ac, b = bc, n = R - a;
      if constexpr (a + b >= 1 && b + 2 <= n) {
        double v = fma(cx_hermite(b + 2, 1), c[mono(a + b + 2, b + 2)], c[mono(a + b, b)]);
        if constexpr (b + 4 <= n) v = fma(cx_hermite(b + 4, 2), c[mono(a + b + 4, b + 4)], v);
        c[mono(a + b, b)] = v;
      }
    });
  });
}

// Its transpose (adjoints of monomial coefficients -> of the stencil's).
template <int R>
__device__ __forceinline__ void hermite_to_monomials_adjoint(double* c, double cx, double cy,
                                                             bool shift) {
  static_for<0, R>([&](auto ac) {
    static_for<0, R + 1 - ac>([&](auto jc) {
      constexpr int a = ac, b = R - a - jc;
      if constexpr (a + b >= 1 && b >= 2) {
        double v = c[mono(a + b, b)];
        if constexpr (a + b - 2 >= 1) v = fma(cx_hermite(b, 1), c[mono(a + b - 2, b - 2)], v);
        if constexpr (b >= 4 && a + b - 4 >= 1)
          v = fma(cx_hermite(b, 2), c[mono(a + b - 4, b - 4)], v);
        c[mono(a + b, b)] = v;
      }
    });
  });
  static_for<0, R>([&](auto bc) {
    static_for<0, R + 1 - bc>([&](auto jc) {
      constexpr int b = bc, a = R - b - jc;
      if constexpr (a + b >= 1 && a >= 2) {
        double v = c[mono(a + b, b)];
        if constexpr (a + b - 2 >= 1) v = fma(cx_hermite(a, 1), c[mono(a + b - 2, b)], v);
        if constexpr (a >= 4 && a + b - 4 >= 1)
          v = fma(cx_hermite(a, 2), c[mono(a + b - 4, b)], v);
        c[mono(a + b, b)] = v;
      }
    });
  });
  if (shift) {
    static_for<0, R>([&](auto ac) {
      constexpr int a = ac, n = R - a;
      static_for<0, n>([&](auto ic) {
        static_for<0, ic + 1>([&](auto jc) {
          constexpr int b = n - 1 - ic + jc;
          if constexpr (a + b >= 1)
            c[mono(a + b + 1, b + 1)] = fma(-cy, c[mono(a + b, b)], c[mono(a + b + 1, b + 1)]);
        });
      });
    });
    static_for<0, R>([&](auto bc) {
      constexpr int b = bc, n = R - b;
      static_for<0, n>([&](auto ic) {
        static_for<0, ic + 1>([&](auto jc) {
          constexpr int a = n - 1 - ic + jc;
          if constexpr (a + b >= 1)
            c[mono(a + b + 1, b)] = fma(-cx, c[mono(a + b, b)], c[mono(a + b + 1, b)]);
        });
      });
    });
  }
}

// Right-hand side of one stencil's normal equations: rhs[l] of the lane's
// variable g.  NR rows of degree R about the centre (cx, cy), slot groups
// G0...; the record of the cell itself is at own.  With S < R the rows are
// read twice, for the functions of degree S and less and for the others: the
// moments cost more, but fewer row sums are in registers at once.
template <int R, int NR, int G0, int NU, int S, class Slots>
__device__ __forceinline__ void stencil_sums(const CellView& cv, const Slots& slots,
                                             const double* own, double cx, double cy, bool shift,
                                             double* rhs) {
  constexpr int N = (R + 1) * (R + 2) / 2 - 1;
  constexpr int RS = 2 * rec_units(NU);
  const double x0 = cv.x + cx, y0 = cv.y + cy;
  double r0 = 0.0;
  static_for<0, S < R ? 2 : 1>([&](auto pc) {
    // degrees (D0, D1] in this pass, functions [L0, L1)
    constexpr int D0 = pc == 0 ? 0 : S, D1 = pc == 0 && S < R ? S : R;
    constexpr int L0 = mono(D0 + 1, 0), L1 = mono(D1, D1) + 1;
    double acc[L1 - L0][4], acc0[4];
    static_for<0, row_groups(NR)>([&](auto jc) {
      unsigned m = slots.template get<G0 + jc>();
      asm volatile("" : "+v"(m));  // each pass reads its records again
      const double* rec = cv.geo + m * RS;
      double q[L1 + 1], mo[L1], d[4];
      static_for<0, L1 + 1>([&](auto l) { q[l] = rec[l]; });
      const double* u = cv.us + m * 4;
      static_for<0, 4>([&](auto i) { d[i] = (u[cv.g ^ i] - cv.u0[i]) * q[2]; });
      shift_moments<D1>(q[0] - x0, q[1] - y0, q + 3, mo);
      static_for<0, 4>([&](auto i) {
        if constexpr (jc == 0) {
          acc0[i] = d[i];
          static_for<L0, L1>([&](auto l) { acc[l - L0][i] = mo[l] * d[i]; });
        } else {
          if constexpr (pc == 0) acc0[i] += d[i];
          static_for<L0, L1>([&](auto l) { acc[l - L0][i] = fma(mo[l], d[i], acc[l - L0][i]); });
        }
      });
      __builtin_amdgcn_sched_barrier(0);  // one group's record at a time in registers
    });
    // the pass ends here: an opaque use of each sum, or the compiler sinks the
    // rows' arithmetic past what follows and holds every record till then
    if constexpr (pc == 0) {
      r0 = quad_sum(acc0);
      opaque(r0);
    }
    static_for<L0, L1>([&](auto l) {
      rhs[l] = quad_sum(acc[l - L0]);
      opaque(rhs[l]);
    });
  });
  // rows have zero mean over the cell: less its own moments
  double h[N];
  own_moments<R>(own, cx, cy, shift, h);
  static_for<0, N>([&](auto l) { rhs[l] = fma(-h[l], r0, rhs[l]); });
}

// ---------------------------------------------------------------------------
// reconstruction
// ---------------------------------------------------------------------------
struct ReconArgs {
  const double* __restrict__ U;        // [n_cell][4]
  BlockArgs b;                         // stencils and least squares
  double* __restrict__ fp;             // [3 nq][n_pad][4]
  uint16_t* flags;                     // out, or in when frozen
  const int32_t* __restrict__ user_of; // [n_pad]
  const double* __restrict__ geo;      // [n_pad][10]: (nx, ny, len) x 3 edges, area
  const int4* __restrict__ nbinfo;     // [n_pad]: .w bit 6+e set when the cell is edge e's L side
  DevDiag* diag;
  int n_cell, n_tiles, n_pad;
  int frozen, variant, fallback, power;
  double ct, eps, gamma, tie_rel;
  double tie_lo, tie_hi;               // near-tie window ct (1 -+ tie_rel); empty when ct = 0
  double cw_dK, cw_ds;                 // CWENO linear weights: large, each small
};

// chi within the near-tie window around C_T (counted, never decided on).
__device__ __forceinline__ int near_tie(TENO_CONST ReconArgs& a, double chi) {
  return (chi >= a.tie_lo && chi <= a.tie_hi) ? 1 : 0;
}

__device__ __forceinline__ double gamma_k(double beta, double eps, int power) {
  const double x = beta + eps;
  double xp;
  if (power == 6) {  // the paper's q: the same products, in the same order, unrolled
    xp = x * x;
    xp *= x;
    xp *= x;
    xp *= x;
    xp *= x;
  } else {
    xp = 1.0;
    for (int t = 0; t < power; ++t) xp *= x;
  }
  return 1.0 / xp;
}

// beta = a^T B a from U, the upper triangle of B with its off-diagonal entries
// doubled.
template <int R>
__device__ __forceinline__ double smoothness(const double* a) {
  using S = SmoothForm<R>;
  constexpr int N = S::N;
  double s = 0.0;
  static_for<0, N>([&](auto lc) {
    constexpr int l = lc;
    double t = S::U.v[l][l] * a[l];
    static_for<l + 1, N>([&](auto m) { t = fma(S::U.v[l][m], a[m], t); });
    s = fma(a[l], t, s);
  });
  return s;
}

__device__ __forceinline__ double pick4(double t0, double t1, double t2, double t3, int g) {
  return g == 0 ? t0 : (g == 1 ? t1 : (g == 2 ? t2 : t3));
}

// LDS ordering between the lanes of one wavefront (staged indices).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Selection of one variable from its stencils' coefficients (Sec. 3.2-3.3):
// step one keeps the large stencil or not; where a lane of the wavefront
// rejects it, step two and the mean of the small stencils it keeps.  aK becomes
// the selected coefficients; returns the variable's 4-bit flag.
template <int P>
__device__ __forceinline__ unsigned teno_select(TENO_CONST ReconArgs& a, bool frozen, unsigned nib_in,
                                                const double (&as)[3][5],
                                                double (&aK)[OrderT<P>::NU], int& ties) {
  using O = OrderT<P>;
  unsigned nib = 8u;
  double gk[3] = {0.0, 0.0, 0.0}, ssum = 1.0;
  if (frozen) {
    nib = nib_in;
  } else if (a.variant == 0) {
    static_for<0, 3>([&](auto k) { gk[k] = gamma_k(smoothness<2>(as[k]), a.eps, a.power); });
    ssum = (gk[0] + gk[1]) + gk[2];
    const double gK = gamma_k(smoothness<O::R>(aK), a.eps, a.power);
    const double chiK = gK / (ssum + gK);
    ties += near_tie(a, chiK);
    nib = chiK >= a.ct ? 8u : 0u;
  }
  if (__any(!(nib & 8u))) {
    const bool rej = !(nib & 8u);
    if (rej && !frozen) {
      const double is = 1.0 / ssum;
      static_for<0, 3>([&](auto k) {
        const double x = gk[k] * is;
        ties += near_tie(a, x);
        nib |= x >= a.ct ? 1u << k : 0u;
      });
    }
    const int cnt = (int)(nib & 1u) + (int)((nib >> 1) & 1u) + (int)((nib >> 2) & 1u);
    const double inv = cnt == 3 ? 1.0 / 3.0 : (cnt == 2 ? 0.5 : (cnt == 1 ? 1.0 : 0.0));
    static_for<0, O::NU>([&](auto l) {
      double x = 0.0;
      if constexpr (l < 5) {
        if (nib & 1u) x += as[0][l];
        if (nib & 2u) x += as[1][l];
        if (nib & 4u) x += as[2][l];
        x *= inv;
      }
      aK[l] = rej ? x : aK[l];
    });
    if (rej) nib &= 7u;
  }
  return nib;
}

// CWENO (Sec. 2.4): P = (w_K/d_K)(P_K - sum_k d_k P_k) + sum_k w_k P_k with
// alpha_k = d_k / (beta_k + eps)^power, w = alpha / sum alpha.
template <int P>
__device__ __forceinline__ void cweno_combine(TENO_CONST ReconArgs& a, const double (&as)[3][5],
                                              double (&aK)[OrderT<P>::NU]) {
  using O = OrderT<P>;
  double w[3];
  static_for<0, 3>([&](auto k) { w[k] = a.cw_ds * gamma_k(smoothness<2>(as[k]), a.eps, a.power); });
  const double wK = a.cw_dK * gamma_k(smoothness<O::R>(aK), a.eps, a.power);
  const double iS = 1.0 / (((w[0] + w[1]) + w[2]) + wK);
  const double cK = wK / a.cw_dK;
  static_for<0, O::NU>([&](auto l) {
    if constexpr (l < 5) {
      const double dsm = a.cw_ds * ((as[0][l] + as[1][l]) + as[2][l]);
      const double asm_ = (w[0] * as[0][l] + w[1] * as[1][l]) + w[2] * as[2][l];
      aK[l] = (cK * (aK[l] - dsm) + asm_) * iS;
    } else {
      aK[l] = (cK * aK[l]) * iS;
    }
  });
}

// Whether a state held one variable per lane of the quad is physical (rho > 0
// and p > 0, false for NaN), tested as (g - 1)(rho E - (mx^2 + my^2) / 2) > 0
// so that the quad shares one sum and no division.  Each lane returns its part;
// the state is physical where all four lanes say so (quad_all).  Called with
// all four lanes active.
struct QuadPhysical {
  double cs;  // factor of the lane's own square
  double cp;  // factor of its product with lane v ^ 3 (rho E on lane 0)
  bool rho;
  __device__ __forceinline__ void init(int v, double g) {
    cs = (v == 1 || v == 2) ? -0.5 * (g - 1.0) : 0.0;
    cp = v == 0 ? g - 1.0 : 0.0;
    rho = v == 0;
  }
  __device__ __forceinline__ bool operator()(double x) const {
    double t = x * fma(cp, quad_xor<3>(x), cs * x);
    t += quad_xor<1>(t);
    t += quad_xor<2>(t);
    return t > 0.0 && (!rho || x > 0.0);
  }
};
__device__ __forceinline__ bool quad_all(bool ok, int lane) {
  return ((__ballot(!ok) >> (lane & 60)) & 15ull) == 0ull;
}

// Characteristic projection of lane variable v (Sec. 2.3): row v of L
// (char_lrow_lane) and row v of R (char_rrow), where R's columns are the right
// eigenvectors of the Euler flux Jacobian in direction (nx, ny) at the cell
// mean u (quad lanes 0..3), for the speeds u.n - c, u.n (entropy), u.n
// (shear), u.n + c, and L = R^-1 in closed form (b1 = (gamma-1)/c^2,
// b2 = b1 |u|^2 / 2).  A mean that is not physical keeps the conservative
// variables (identity rows).  The two are formed apart, each when needed,
// to keep fewer registers live.
// The normal-independent part of the projection state, formed once per cell.
struct CharState {
  double ux, uy, q2, c, ic, H, b1, b2;
};
__device__ __forceinline__ CharState char_state(double u0, double g) {
  const double rho = quad_bcast<0>(u0), mx = quad_bcast<1>(u0), my = quad_bcast<2>(u0),
               en = quad_bcast<3>(u0);
  CharState S;
  const double ir = 1.0 / rho;
  S.ux = mx * ir;
  S.uy = my * ir;
  S.q2 = S.ux * S.ux + S.uy * S.uy;
  const double p = (g - 1.0) * (en - 0.5 * rho * S.q2);
  S.c = sqrt(g * p * ir);
  S.ic = 1.0 / S.c;
  S.H = (en + p) * ir;
  S.b1 = (g - 1.0) * S.ic * S.ic;
  S.b2 = 0.5 * S.q2 * S.b1;
  return S;
}

// The part of the state that costs a division or a square root (u = m / rho,
// c, 1 / c), kept across a cell's edges where registers allow; the rest is
// formed again from it on each edge, with H = c^2 / (gamma - 1) + |u|^2 / 2.
struct CharCore {
  double ux, uy, c, ic;
};
__device__ __forceinline__ CharCore char_core(const CharState& S) { return {S.ux, S.uy, S.c, S.ic}; }
__device__ __forceinline__ CharState char_expand(CharCore K, double g) {
  // opaque copies: left visible, the expansion is the same on every edge
  // and the compiler forms it once and holds all of it
  asm volatile("" : "+v"(K.ux), "+v"(K.uy), "+v"(K.c), "+v"(K.ic));
  CharState S;
  S.ux = K.ux;
  S.uy = K.uy;
  S.q2 = K.ux * K.ux + K.uy * K.uy;
  S.c = K.c;
  S.ic = K.ic;
  S.H = K.c * K.c / (g - 1.0) + 0.5 * S.q2;
  S.b1 = (g - 1.0) * K.ic * K.ic;
  S.b2 = 0.5 * S.q2 * S.b1;
  return S;
}

__device__ __forceinline__ void char_rrow(const CharState& S, double nx, double ny, bool ok, int v,
                                          double (&rrow)[4]) {
  if (!ok) {
#pragma unroll
    for (int j = 0; j < 4; ++j) rrow[j] = (j == v) ? 1.0 : 0.0;
    return;
  }
  const double un = S.ux * nx + S.uy * ny, ut = S.uy * nx - S.ux * ny;
  const double R[4][4] = {{1.0, 1.0, 0.0, 1.0},
                          {S.ux - S.c * nx, S.ux, -ny, S.ux + S.c * nx},
                          {S.uy - S.c * ny, S.uy, nx, S.uy + S.c * ny},
                          {S.H - S.c * un, 0.5 * S.q2, ut, S.H + S.c * un}};
#pragma unroll
  for (int j = 0; j < 4; ++j) rrow[j] = pick4(R[0][j], R[1][j], R[2][j], R[3][j], v);
}

// sum_j row[j] x_j, x_j = lane j's x of this cell's quad.  Operand and
// result pass through opaque copies, which keep each product whole and in
// order: the broadcasts of a coefficient are the same on every edge, and
// left visible the compiler forms them all ahead of their use and holds
// four copies of every coefficient across the edges.
__device__ __forceinline__ double quad_dot(const double (&row)[4], double x) {
  asm volatile("" : "+v"(x));
  double s = row[0] * quad_bcast<0>(x);
  s = fma(row[1], quad_bcast<1>(x), s);
  s = fma(row[2], quad_bcast<2>(x), s);
  s = fma(row[3], quad_bcast<3>(x), s);
  asm volatile("" : "+v"(s));
  return s;
}

// Characteristic TENO (and Linear) without projecting the coefficients for
// the indicators.  For each stencil the Gram matrix G = sum_lm B_lm a_l a_m^T
// of the four variables' coefficient vectors (4 x 4, symmetric) is formed
// once per cell; the indicator of characteristic variable v on an edge is
// then L_v^T G L_v, which equals beta of the projected coefficients L_v a.
// The selection follows per variable.  Where the four variables of a cell
// select alike on an edge (every smooth cell, and any jump that all fields
// see), the projection cancels (R L = I) and the face states are the
// conservative combination of the same stencils; only cells whose fields
// select differently project the coefficients and map back.  The Gram
// matrices live in the block's staging LDS (16 cells x
// 4 stencils x 10 entries), which the least-squares phase no longer needs.
__device__ __forceinline__ int gram_off(int i, int j) {  // i <= j
  return i * 4 - (i * (i - 1)) / 2 + (j - i);
}

// Row v of the Gram matrix of one stencil, G_vj = (a^j)^T B a^v, from the
// factor B = L D L^T: with z = L^T a, G_vj = sum_l d_l z^v_l z^j_l.  One
// component of z at a time; the empty asm ties each step to the previous
// step's sums so that the compiler does not form all of z up front.
template <int R>
__device__ __forceinline__ void gram_rows(const double* a, int v, double* G) {
  using S = SmoothForm<R>;
  constexpr int N = S::N;
  double r0 = 0.0, r1 = 0.0, r2 = 0.0, r3 = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    double z = a[l];
    asm volatile("" : "+v"(z), "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3));
#pragma unroll
    for (int m = l + 1; m < N; ++m) z = fma(S::LDL.Lt[l][m], a[m], z);
    const double w = S::LDL.d[l] * z;
    r0 = fma(quad_bcast<0>(z), w, r0);
    r1 = fma(quad_bcast<1>(z), w, r1);
    r2 = fma(quad_bcast<2>(z), w, r2);
    r3 = fma(quad_bcast<3>(z), w, r3);
  }
  const double r[4] = {r0, r1, r2, r3};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j >= v) G[gram_off(v, j)] = r[j];
}

// Row v of the left eigenvector matrix for edge normal (nx, ny), formed
// directly for the lane's own variable: with
//   A = (b2, -b1 ux, -b1 uy, b1), B = (un, -nx, -ny, 0) / c, C = (-ut, -ny, nx, 0)
// the rows are A/2 + B/2 (v = 0), (1, 0, 0, 0) - A (v = 1), C (v = 2) and
// A/2 - B/2 (v = 3), the same matrix as char_lrow.
__device__ __forceinline__ void char_lrow_lane(const CharState& S, double nx, double ny, bool ok,
                                               int v, double (&lrow)[4]) {
  const double un = S.ux * nx + S.uy * ny, ut = S.uy * nx - S.ux * ny;
  const double ca = v == 1 ? -1.0 : (v == 2 ? 0.0 : 0.5);
  const double cb = v == 0 ? 0.5 : (v == 3 ? -0.5 : 0.0);
  const double cc = v == 2 ? 1.0 : 0.0;
  const double cd = v == 1 ? 1.0 : 0.0;
  const double A[4] = {S.b2, -S.b1 * S.ux, -S.b1 * S.uy, S.b1};
  const double B[4] = {un * S.ic, -nx * S.ic, -ny * S.ic, 0.0};
  const double Cv[4] = {-ut, -ny, nx, 0.0};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double r = fma(ca, A[j], fma(cb, B[j], cc * Cv[j])) + (j == 0 ? cd : 0.0);
    lrow[j] = ok ? r : (j == v ? 1.0 : 0.0);
  }
}

// The ten products of a row L that pair with the stored entries of G
// (diagonal once, off-diagonal doubled), in gram_off order.
__device__ __forceinline__ void gram_weights(const double (&L)[4], double (&q)[10]) {
  const double t0 = L[0] + L[0], t1 = L[1] + L[1], t2 = L[2] + L[2];
  q[0] = L[0] * L[0];
  q[1] = t0 * L[1];
  q[2] = t0 * L[2];
  q[3] = t0 * L[3];
  q[4] = L[1] * L[1];
  q[5] = t1 * L[2];
  q[6] = t1 * L[3];
  q[7] = L[2] * L[2];
  q[8] = t2 * L[3];
  q[9] = L[3] * L[3];
}

__device__ __forceinline__ double gram_dot(const double* G, const double (&q)[10]) {
  double s = q[0] * G[0];
#pragma unroll
  for (int k = 1; k < 10; ++k) s = fma(q[k], G[k], s);
  return s;
}

template <int P, int NQ>
__device__ __forceinline__ void char_edges_gram(TENO_CONST ReconArgs& a, const double (&as)[3][5],
                                                const double (&aK)[OrderT<P>::NU], double u0,
                                                int cell, bool live, int g, int v, int c, int lane,
                                                double* gram0) {
  using O = OrderT<P>;
  constexpr int NU = O::NU;
  QuadPhysical phys;
  phys.init(v, a.gamma);
  const bool avg_ok = quad_all(phys(u0), lane);
  const double* __restrict__ gc = a.geo + (size_t)(live ? cell : 0) * 10;
  const int side = a.nbinfo[live ? cell : 0].w;  // face normals point out of the L side
  // ---- Gram matrices of the four stencils (the staging LDS is free now) ----
  double* gram = gram0 + c * 40;
  wave_lds_sync();
  if (a.variant == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) gram_rows<2>(as[k], v, gram + 10 * k);
  }
  gram_rows<O::R>(aK, v, gram + 30);
  wave_lds_sync();
  int ties = 0;
  bool fp_ok = true;
  const CharCore core = char_core(char_state(u0, a.gamma));
  auto state = [&]() { return char_expand(core, a.gamma); };
  static_for<0, 3>([&](auto E) {
    constexpr int e = E;
    __builtin_amdgcn_sched_barrier(0);
    const double sg = ((side >> (6 + e)) & 1) ? 1.0 : -1.0;
    const double nx = sg * gc[3 * e], ny = sg * gc[3 * e + 1];
    double lrow[4];
    char_lrow_lane(state(), nx, ny, avg_ok, v, lrow);
    // ---- selection of characteristic variable v (Sec. 3.2-3.3) ----
    unsigned nib = 8u;
    if (a.variant == 0) {
      // an opaque offset per edge keeps the 40 Gram entries from being read
      // once and held in registers across the three edges
      int goff = c * 40;
      asm volatile("" : "+v"(goff));
      const double* gram = gram0 + goff;
      double q[10];
      gram_weights(lrow, q);
      const double g0 = gamma_k(gram_dot(gram, q), a.eps, a.power);
      const double g1 = gamma_k(gram_dot(gram + 10, q), a.eps, a.power);
      const double g2 = gamma_k(gram_dot(gram + 20, q), a.eps, a.power);
      const double ssum = (g0 + g1) + g2;
      const double is = 1.0 / ssum;
      const double x0 = g0 * is, x1 = g1 * is, x2 = g2 * is;
      const int st = near_tie(a, x0) + near_tie(a, x1) + near_tie(a, x2);
      const unsigned nsm = (x0 >= a.ct ? 1u : 0u) | (x1 >= a.ct ? 2u : 0u) | (x2 >= a.ct ? 4u : 0u);
      const double gK = gamma_k(gram_dot(gram + 30, q), a.eps, a.power);
      const double chiK = gK / (ssum + gK);
      ties += near_tie(a, chiK);
      const bool keepK = chiK >= a.ct;
      if (!keepK) ties += st;
      nib = keepK ? 8u : nsm;
    }
    // ---- do the cell's four variables select alike? ----
    const unsigned n0 = (unsigned)__builtin_amdgcn_mov_dpp((int)nib, 0x00, 0xF, 0xF, false);
    const unsigned n1 = (unsigned)__builtin_amdgcn_mov_dpp((int)nib, 0x55, 0xF, 0xF, false);
    const unsigned n2 = (unsigned)__builtin_amdgcn_mov_dpp((int)nib, 0xAA, 0xF, 0xF, false);
    const unsigned n3 = (unsigned)__builtin_amdgcn_mov_dpp((int)nib, 0xFF, 0xF, 0xF, false);
    const bool alike = n0 == n1 && n1 == n2 && n2 == n3;
    TENO_CONST double* fb = table(&FaceBasis<O::R, NQ>::P.v[e * NQ][0]);
    // the combined coefficients one at a time, straight into the face sums
    const int cnt = (int)(nib & 1u) + (int)((nib >> 1) & 1u) + (int)((nib >> 2) & 1u);
    const double inv = cnt == 3 ? 1.0 / 3.0 : (cnt == 2 ? 0.5 : (cnt == 1 ? 1.0 : 0.0));
    double val[NQ];
    if (alike) {
      // the conservative combination of the stencils every field selected
#pragma unroll
      for (int kq = 0; kq < NQ; ++kq) val[kq] = u0;
#pragma unroll
      for (int l = 0; l < NU; ++l) {
        double ab = aK[l];
        if (l < 5 && !(nib & 8u)) {
          double sm = 0.0;
          if (nib & 1u) sm += as[0][l];
          if (nib & 2u) sm += as[1][l];
          if (nib & 4u) sm += as[2][l];
          ab = sm * inv;
        } else if (!(nib & 8u)) {
          ab = 0.0;
        }
#pragma unroll
        for (int kq = 0; kq < NQ; ++kq) val[kq] = fma(ab, fb[kq * NU + l], val[kq]);
      }
    } else {
      // fields select differently: project, combine per variable, map back
      double dw[NQ];
#pragma unroll
      for (int kq = 0; kq < NQ; ++kq) dw[kq] = 0.0;
#pragma unroll
      for (int l = 0; l < NU; ++l) {
        // every lane of the quad takes part in each projection (the four
        // variables of a cell may select differently here)
        double xk = aK[l];
        asm volatile("" : "+v"(xk), "+v"(dw[0]), "+v"(dw[NQ - 1]));
        const double wk = quad_dot(lrow, xk);
        double ab = (nib & 8u) ? wk : 0.0;
        if (l < 5) {
          double x0 = as[0][l], x1 = as[1][l], x2 = as[2][l];
          asm volatile("" : "+v"(x0), "+v"(x1), "+v"(x2) : "v"(wk));
          const double w0 = quad_dot(lrow, x0), w1 = quad_dot(lrow, x1), w2 = quad_dot(lrow, x2);
          double sm = 0.0;
          if (nib & 1u) sm += w0;
          if (nib & 2u) sm += w1;
          if (nib & 4u) sm += w2;
          if (!(nib & 8u)) ab = sm * inv;
        }
#pragma unroll
        for (int kq = 0; kq < NQ; ++kq) dw[kq] = fma(ab, fb[kq * NU + l], dw[kq]);
      }
      double rrow[4];
      char_rrow(state(), nx, ny, avg_ok, v, rrow);
#pragma unroll
      for (int kq = 0; kq < NQ; ++kq) val[kq] = u0 + quad_dot(rrow, dw[kq]);
    }
#pragma unroll
    for (int kq = 0; kq < NQ; ++kq) {
      fp_ok = phys(val[kq]) && fp_ok;
      if (live) (a.fp + (size_t)(e * NQ + kq) * a.n_pad * 4)[4u * cell + v] = val[kq];
    }
    if (a.flags) {  // one word per local edge: flags[e][n_cell]
      unsigned f = nib << (4 * v);
      f |= __shfl_xor(f, 1);
      f |= __shfl_xor(f, 2);
      if (live && g == 0) a.flags[(size_t)e * a.n_cell + cell] = (uint16_t)f;
    }
  });
  __builtin_amdgcn_sched_barrier(0);
  // ---- non-physical states (all four lanes of a cell agree) ----
  fp_ok = quad_all(fp_ok, lane);
  if (live && g == 0 && !(avg_ok && fp_ok)) {
    atomicAdd(&a.diag->nonphysical, 1ull);
    atomicMin(&a.diag->first_bad, (long long)a.user_of[cell]);
  }
  if (!fp_ok && avg_ok && a.fallback) {
    if (live)
      for (int q = 0; q < 3 * NQ; ++q) a.fp[((size_t)q * a.n_pad + cell) * 4 + v] = u0;
    if (a.flags && live && g == 0)
      for (int e = 0; e < 3; ++e) a.flags[(size_t)e * a.n_cell + cell] = 0;
    if (live && g == 0) atomicAdd(&a.diag->fallbacks, 1ull);
  }
  if (live && ties) atomicAdd(&a.diag->near_ties, (unsigned long long)ties);
}

// Characteristic CWENO (Sec. 2.4 in the variables of Sec. 2.3) with the
// indicators of char_edges_gram: the weights of variable v on an edge come
// from L_v^T G_k L_v.  The CWENO polynomial is a linear combination of the
// stencils' polynomials, P = lK P_K + sum_k l_k p_k with lK = (w_K/d_K)/S and
// l_k = (alpha_k - d_k w_K/d_K)/S, so each stencil is evaluated at the edge's
// Gauss points in conservative variables and only those point values are
// projected (four stencils x NQ points instead of every coefficient).
template <int P, int NQ>
__device__ __forceinline__ void char_edges_cweno_gram(TENO_CONST ReconArgs& a,
                                                      const double (&as)[3][5],
                                                      const double (&aK)[OrderT<P>::NU],
                                                      double u0, int cell, bool live,
                                                      int g, int v, int c, int lane, double* gram0) {
  using O = OrderT<P>;
  constexpr int NU = O::NU;
  QuadPhysical phys;
  phys.init(v, a.gamma);
  const bool avg_ok = quad_all(phys(u0), lane);
  const double* __restrict__ gc = a.geo + (size_t)(live ? cell : 0) * 10;
  const int side = a.nbinfo[live ? cell : 0].w;  // face normals point out of the L side
  double* gram = gram0 + c * 40;
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 3; ++k) gram_rows<2>(as[k], v, gram + 10 * k);
  gram_rows<O::R>(aK, v, gram + 30);
  wave_lds_sync();
  bool fp_ok = true;
  const CharCore core = char_core(char_state(u0, a.gamma));
  auto state = [&]() { return char_expand(core, a.gamma); };
  static_for<0, 3>([&](auto E) {
    constexpr int e = E;
    __builtin_amdgcn_sched_barrier(0);
    const double sg = ((side >> (6 + e)) & 1) ? 1.0 : -1.0;
    const double nx = sg * gc[3 * e], ny = sg * gc[3 * e + 1];
    double lrow[4];
    char_lrow_lane(state(), nx, ny, avg_ok, v, lrow);
    int goff = c * 40;
    asm volatile("" : "+v"(goff));
    const double* gm = gram0 + goff;
    double q[10];
    gram_weights(lrow, q);
    const double w0 = a.cw_ds * gamma_k(gram_dot(gm, q), a.eps, a.power);
    const double w1 = a.cw_ds * gamma_k(gram_dot(gm + 10, q), a.eps, a.power);
    const double w2 = a.cw_ds * gamma_k(gram_dot(gm + 20, q), a.eps, a.power);
    const double wK = a.cw_dK * gamma_k(gram_dot(gm + 30, q), a.eps, a.power);
    const double iS = 1.0 / (((w0 + w1) + w2) + wK);
    const double cK = wK / a.cw_dK;
    const double lK = cK * iS;
    const double l0 = (w0 - cK * a.cw_ds) * iS, l1 = (w1 - cK * a.cw_ds) * iS,
                 l2 = (w2 - cK * a.cw_ds) * iS;
    double rrow[4];
    char_rrow(state(), nx, ny, avg_ok, v, rrow);
    TENO_CONST double* fb = table(&FaceBasis<O::R, NQ>::P.v[e * NQ][0]);
#pragma unroll
    for (int kq = 0; kq < NQ; ++kq) {
      // the four stencils' values of the lane's conservative variable
      double pK = 0.0, p0 = 0.0, p1 = 0.0, p2 = 0.0;
#pragma unroll
      for (int l = 0; l < NU; ++l) pK = fma(aK[l], fb[kq * NU + l], pK);
#pragma unroll
      for (int l = 0; l < 5; ++l) {
        p0 = fma(as[0][l], fb[kq * NU + l], p0);
        p1 = fma(as[1][l], fb[kq * NU + l], p1);
        p2 = fma(as[2][l], fb[kq * NU + l], p2);
      }
      const double dw = lK * quad_dot(lrow, pK) +
                        ((l0 * quad_dot(lrow, p0) + l1 * quad_dot(lrow, p1)) +
                         l2 * quad_dot(lrow, p2));
      const double val = u0 + quad_dot(rrow, dw);
      fp_ok = phys(val) && fp_ok;
      if (live) (a.fp + (size_t)(e * NQ + kq) * a.n_pad * 4)[4u * cell + v] = val;
    }
    if (a.flags && live && g == 0) a.flags[(size_t)e * a.n_cell + cell] = 0;
  });
  __builtin_amdgcn_sched_barrier(0);
  // ---- non-physical states (all four lanes of a cell agree) ----
  fp_ok = quad_all(fp_ok, lane);
  if (live && g == 0 && !(avg_ok && fp_ok)) {
    atomicAdd(&a.diag->nonphysical, 1ull);
    atomicMin(&a.diag->first_bad, (long long)a.user_of[cell]);
  }
  if (!fp_ok && avg_ok && a.fallback) {
    if (live)
      for (int q = 0; q < 3 * NQ; ++q) a.fp[((size_t)q * a.n_pad + cell) * 4 + v] = u0;
    if (live && g == 0) atomicAdd(&a.diag->fallbacks, 1ull);
  }
}

// Degree at which the large stencil's rows are split into two passes: one pass
// keeps (degree <= split) sums of four variables in registers, the other the
// rest.  Order 6 on 180,000 cells: 177.5 us split at degree 3, 185.1 at 4;
// order 5 on 262,088: 159.2 at 4, 170.3 at 3.
constexpr int split_degree(int p) { return p == 3 ? 2 : (p == 4 ? 3 : (p == 5 ? 4 : 3)); }
// 16-byte loads of the large normal matrix per chunk, two chunks in flight: as
// many as the registers hold beside the row sums (7 to 19 at order 5 and 5 to 9
// at order 6 measured within 3%).  Loading the first chunk a tile ahead costs
// order 3 its third wavefront per SIMD (53.3 against 48.8 us on 180,000 cells)
// and gains nothing at the others.
constexpr int solve_chunk(int p) { return p == 5 ? 14 : (p == 6 ? 9 : 99); }

// What a wavefront needs of its next tile before the first row: loaded while the
// previous tile's selection runs.
template <int P>
struct TileAhead {
  static constexpr int NU = OrderT<P>::NU, NL = OrderT<P>::NL;
  static constexpr int CH = solve_chunk(P) < sym_quads(NU) ? solve_chunk(P) : sym_quads(NU);
  MemberSlots<NL> slots;
  int cell;  // -1: none
  double2 ja, jb;
  float2 cen[4];
  __device__ __forceinline__ void load(TENO_CONST BlockArgs& b, int tile, int lane) {
    cell = (b.pack + (size_t)tile * kTile)[(unsigned)lane >> 2];
    slots.load(b.bslot, tile, lane);
    const unsigned c = (unsigned)lane >> 2;
    const float2* __restrict__ ce = b.centre + (size_t)tile * (4 * kTile);
    const double2* __restrict__ jc = b.jac + (size_t)tile * (2 * kTile);
    static_for<0, 4>([&](auto k) { cen[k] = ce[4 * c + k]; });
    ja = jc[2 * c];
    jb = jc[2 * c + 1];
  }
};

// Selection and face states of one cell per quad from its stencils' coefficients,
// in conservative variables.
template <int P, int NQ, bool CW>
__device__ __forceinline__ void select_and_store(TENO_CONST ReconArgs& a, bool frozen,
                                                 const double (&as)[3][5],
                                                 double (&aK)[OrderT<P>::NU], double u0, int cell,
                                                 bool live, int g, int v, int lane) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NP = 3 * NQ;
  const unsigned nib_in = (frozen && live) ? ((a.flags[cell] >> (4 * v)) & 0xFu) : 8u;
  int ties = 0;
  unsigned nib = 0u;
  if constexpr (CW)
    cweno_combine<P>(a, as, aK);
  else
    nib = teno_select<P>(a, frozen, nib_in, as, aK, ties);
  // ---- face Gauss points (variable v of this cell) ----
  double val[NP];
  static_for<0, NP>([&](auto q) {
    double s = u0;
    static_for<0, NU>([&](auto l) { s = fma(aK[l], FaceBasis<O::R, NQ>::P.v[q][l], s); });
    val[q] = s;
  });
  // ---- non-physical states (all four lanes of a cell agree) ----
  if (!frozen) {
    QuadPhysical phys;
    phys.init(v, a.gamma);
    const bool avg_ok = quad_all(phys(u0), lane);
    bool ok = true;
    static_for<0, NP>([&](auto q) { ok = phys(val[q]) && ok; });
    const bool fp_ok = quad_all(ok, lane);
    if (live && g == 0 && !(avg_ok && fp_ok)) {  // one lane per cell
      atomicAdd(&a.diag->nonphysical, 1ull);
      atomicMin(&a.diag->first_bad, (long long)a.user_of[cell]);
    }
    if (!fp_ok && avg_ok && a.fallback) {
      static_for<0, NP>([&](auto q) { val[q] = u0; });
      nib = 0u;
      if (live && g == 0) atomicAdd(&a.diag->fallbacks, 1ull);
    }
    if (live && ties) atomicAdd(&a.diag->near_ties, (unsigned long long)ties);
  }
  if (live)
    static_for<0, NP>([&](auto q) {
      (a.fp + (size_t)q * a.n_pad * 4)[4u * cell + v] = val[q];
    });
  if (!frozen && a.flags) {
    unsigned f = nib << (4 * v);
    f |= __shfl_xor(f, 1);
    f |= __shfl_xor(f, 2);
    if (live && g == 0) a.flags[cell] = (uint16_t)f;
  }
}

// Reconstruction of the blocks of a work list by one workgroup: items
// [k0, k1) in steps, item k = (arguments, block) from items(k).  Two blocks are
// staged in LDS: while one is computed, the next one's records and states are
// copied in behind it and the ids of the one after, so the only wait for
// memory is for the part of the large normal matrix that the registers cannot
// hold ahead.  (One block per workgroup and launch slot left the phases of the
// resident wavefronts aligned: at order 5 a quarter of a wavefront's time went to
// loading and a fifth of the slots stood empty between workgroups.)
template <int P, int NQ, bool CW, bool CH, class Items>
__device__ __forceinline__ void reconstruct_loop(const Items& items, int k0, int k1, int step,
                                                 char* lds) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NL = O::NL, R = O::R;
  constexpr int GS = row_groups(kSmallRows), QS = sym_quads(kSmallCoef);
  if (k0 >= k1) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nthr = blockDim.x;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  auto tile_of = [&](TENO_CONST ReconArgs& a, int blk) {  // the wavefront's tile, -1: none
    const int t = blk * a.b.bwaves + wave;
    return wave < a.b.bwaves && t < a.n_tiles ? t : -1;
  };
  // ---- the first block: ids straight from memory ----
  TileAhead<P> ta;
  int tile_n;  // the wavefront's tile of the next item
  {
    TENO_CONST ReconArgs& a = items.args(k0);
    const int blk = items.block(k0);
    // all of its places: the lists' lengths are one load further away
    copy_states(a.U, a.b.bmem + (size_t)blk * a.b.mstride, a.b.mstride, lds0, nthr);
    copy_records<NU>(a.b, blk, lds0 + 32 * a.b.bmax, nthr);
    if (k0 + step < k1) {
      TENO_CONST ReconArgs& n = items.args(k0 + step);
      copy_ids(n.b, items.block(k0 + step), lds0 + list_offset<NU, CH>(n.b, 1), nthr);
    }
    tile_n = tile_of(a, blk);
    ta.load(a.b, max(tile_n, 0), threadIdx.x & 63);
    lds_copy_wait();
  }
  int it = 0;
#pragma unroll 1
  for (int k = k0; k < k1; k += step, ++it) {
    TENO_CONST ReconArgs& a = items.args(k);
    const bool on = tile_n >= 0;
    const int tile = max(tile_n, 0);
    __syncthreads();  // this block is staged, the other buffer is no longer read
    // opaque, so that what derives from the lane is formed where it is used and
    // not held in registers across the items
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int c = lane >> 2, g = lane & 3, v = g;
    auto stage_next = [&]() {
      if (k + step < k1) {
        TENO_CONST ReconArgs& n = items.args(k + step);
        const int nb = items.block(k + step);
        const unsigned st = lds0 + buf_offset<NU, CH>(n.b, it + 1);
        const int* ids = reinterpret_cast<const int*>(lds + list_offset<NU, CH>(n.b, it + 1));
        copy_states(n.U, ids, scalar_load(n.b.boff, nb + 1) - scalar_load(n.b.boff, nb), st, nthr);
        copy_records<NU>(n.b, nb, st + 32 * n.b.bmax, nthr);
      }
    };
    if (a.b.nbuf == 2) {
      stage_next();
      if (k + 2 * step < k1) {
        TENO_CONST ReconArgs& n = items.args(k + 2 * step);
        copy_ids(n.b, items.block(k + 2 * step), lds0 + list_offset<NU, CH>(n.b, it), nthr);
      }
    }
    const char* buf = lds + buf_offset<NU, CH>(a.b, it);
    const int own_slot = min(wave, a.b.bwaves - 1) * kTile + c;
    const int cell = ta.cell;
    const bool live = on && cell >= 0;
    CellView cv;
    cv.us = reinterpret_cast<const double*>(buf);
    cv.geo = reinterpret_cast<const double*>(buf + 32 * a.b.bmax);
    cv.g = g;
    const double* own = cv.geo + own_slot * (2 * rec_units(NU));
    cv.x = own[0];
    cv.y = own[1];
    static_for<0, 4>([&](auto i) { cv.u0[i] = cv.us[own_slot * 4 + (g ^ i)]; });
    const double u0 = cv.u0[0];
    const bool frozen = a.frozen != 0;
    const double2* __restrict__ np = a.b.N + (size_t)tile * (normal_quads(NU) * 64);
    const bool small = CW || frozen || a.variant != 1;
    double aK[NU], as[3][5];
    NormalMatrix<kSmallCoef> ns[3];
    // ---- large stencil ----
    {
      double r[NU];
      const float2 ce = ta.cen[3];
      const bool shift = __any(ce.x != 0.0f || ce.y != 0.0f);
      stencil_sums<R, NL, 3 * GS, NU, split_degree(P)>(cv, ta.slots, own, ce.x, ce.y, shift, r);
      NormalMatrix<NU, TileAhead<P>::CH> nl;
      nl.template load<0>(np + 3 * QS * 64, lane);
      if (small) ns[0].template load<0>(np, lane);
      nl.apply(np + 3 * QS * 64, lane, r, aK);
      hermite_to_monomials<R>(aK, ce.x, ce.y, shift);
      Frame<R> fr;
      fr.init(ta.ja, ta.jb);
      fr.template to_basis<R>(aK);
      static_for<0, NU>([&](auto l) { opaque(aK[l]); });
    }
    // ---- small stencils; the linear scheme keeps the large stencil and never
    //      reads them ----
    if (small) {
      Frame<2> fr;
      fr.init(ta.ja, ta.jb);
      static_for<0, 3>([&](auto q) {
        double r[kSmallCoef];
        const float2 ce = ta.cen[q];
        if constexpr (q < 2) ns[q + 1].template load<0>(np + QS * (q + 1) * 64, lane);
        stencil_sums<2, kSmallRows, GS * q, NU, 2>(cv, ta.slots, own, ce.x, ce.y, true, r);
        ns[q].apply(np, lane, r, as[q]);
        hermite_to_monomials<2>(as[q], ce.x, ce.y, true);
        fr.template to_basis<2>(as[q]);
        static_for<0, 5>([&](auto l) { opaque(as[q][l]); });
      });
    } else {
      static_for<0, 3>([&](auto q) { static_for<0, 5>([&](auto l) { as[q][l] = 0.0; }); });
    }
    // every copy and load so far is complete (they return in order)
    lds_copy_wait();
    if (k + step < k1) {
      TENO_CONST ReconArgs& n = items.args(k + step);
      tile_n = tile_of(n, items.block(k + step));
      ta.load(n.b, max(tile_n, 0), lane);
    }
    if (a.b.nbuf == 1 && k + step < k1) {  // the next block in the same LDS
      TENO_CONST ReconArgs& n = items.args(k + step);
      __syncthreads();
      copy_ids(n.b, items.block(k + step), lds0 + list_offset<NU, CH>(n.b, 0), nthr);
      lds_copy_wait();
      __syncthreads();
      if constexpr (!CH) {
        stage_next();
        lds_copy_wait();
      }
    }
    if constexpr (CH) {
      __syncthreads();  // every wavefront is done with the staged members
      double* gram = reinterpret_cast<double*>(const_cast<char*>(buf)) + wave * kCharGramDoubles;
      if constexpr (CW)
        char_edges_cweno_gram<P, NQ>(a, as, aK, u0, cell, live, g, v, c, lane, gram);
      else
        char_edges_gram<P, NQ>(a, as, aK, u0, cell, live, g, v, c, lane, gram);
      if (a.b.nbuf == 1 && k + step < k1) {
        __syncthreads();
        stage_next();
        lds_copy_wait();
      }
      continue;
    }
    // (through a lambda: called outright, the loop spills 16 registers at order 3
    // instead of 12, 99.4 against 95.8 us on 352,800 cells)
    [&]() __attribute__((always_inline)) {
      select_and_store<P, NQ, CW>(a, frozen, as, aK, u0, cell, live, g, v, lane);
    }();
  }
}

// The blocks of one mesh, dealt to the workgroups of an XCD in turn: workgroups
// are dispatched round-robin over the 8 XCDs, and each XCD gets a contiguous
// range of blocks, so that its L2 holds the neighbourhood it gathers.
struct MeshItems {
  int first;
  // the kernel's first argument, through an opaque pointer: what an item reads
  // is not held in scalar registers across the items
  __device__ __forceinline__ TENO_CONST ReconArgs& args(int) const {
    auto p = (TENO_CONST ReconArgs*)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *p;
  }
  __device__ __forceinline__ int block(int k) const { return first + k; }
};
template <int P, int NQ, bool CW, bool CH>
__device__ __forceinline__ void reconstruct_mesh(int n_blocks) {
  extern __shared__ int4 lds[];
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3, G = gridDim.x;
  const int q = n_blocks / 8, r = n_blocks % 8;
  const MeshItems items{x * q + min(x, r)};
  reconstruct_loop<P, NQ, CW, CH>(items, j, q + (x < r ? 1 : 0), G / 8 + (x < G % 8 ? 1 : 0),
                                  reinterpret_cast<char*>(lds));
}

// Occupancy targets (waves per SIMD) of the reconstruction kernels: the third
// wavefront pays at order 3 (48.8 against 53.3 us on 180,000 cells); at order 4
// its 168 registers spill (97 against 68 us).
constexpr int recon_waves(int p) { return p == 3 ? 3 : 2; }

template <int P, int NQ, bool CW>
__global__ __launch_bounds__(64 * block_tiles(P))
__attribute__((amdgpu_waves_per_eu(recon_waves(P)))) void k_reconstruct(ReconArgs a,
                                                                         int n_blocks) {
  reconstruct_mesh<P, NQ, CW, false>(n_blocks);
}

// The same in characteristic variables.
template <int P, int NQ, bool CW>
__global__ __launch_bounds__(64 * block_tiles(P))
__attribute__((amdgpu_waves_per_eu(recon_waves(P)))) void k_reconstruct_char(ReconArgs a,
                                                                              int n_blocks) {
  reconstruct_mesh<P, NQ, CW, true>(n_blocks);
}

// ---------------------------------------------------------------------------
// Small meshes: one workgroup of four wavefronts per tile, a wavefront per stencil
// (0..2 small, 3 large) over the tile's staged block, whose coefficients the first
// one then selects from.  The same sums in the same order as above, so the same
// bits, from a quarter of the chain: where blocks of 64 or 128 cells leave compute
// units empty, a tile waits for its rows and not for its share of the chip.
// 2,048 cells, orders 3-6: 6.8, 6.8, 10.0, 14.6 us against 8.7, 9.5, 16.9, 24.3 us.
// ---------------------------------------------------------------------------
// Tiles up to which it is taken.  Small against blocks (us): order 3 8.4 / 9.9 at
// 1,013 tiles, 14.4 / 13.2 at 2,048; in characteristic variables, whose selection is
// most of the work, 24.2 / 25.0 at 2,048 and 40.6 / 41.9 at 4,050 (CWENO 25.0 / 22.5
// at 2,048).  Order 4 8.2 / 10.2 at 512, 13.7 / 10.6 at 1,013; order 5 11.6 / 17.2
// and 22.3 / 17.7; order 6 16.5 / 24.9 and 31.7 / 25.5: two or three workgroups fit
// a compute unit there.
constexpr int small_tiles(int order, bool characteristic_teno) {
  return order > 3 ? 512 : (characteristic_teno ? 4096 : 1024);
}
// wavefronts per SIMD: as many workgroups on a CU
constexpr int small_waves(int p) { return p == 3 ? 4 : 2; }

template <int P, int NQ, bool CW, bool CH>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(small_waves(P)))) void k_reconstruct_small(ReconArgs) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NL = O::NL, R = O::R;
  constexpr int GS = row_groups(kSmallRows), QS = sym_quads(kSmallCoef);
  typedef RowSlots<GS, kSlotBits> Small;
  static_assert(Small::NW == 1 && Small::PER == GS, "a word of slots per small stencil");
  extern __shared__ int4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  TENO_CONST ReconArgs& a = *(TENO_CONST ReconArgs*)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = lane >> 2, g = lane & 3;
  const int tile = xcd_remap(blockIdx.x, gridDim.x), blk = tile / a.b.bwaves;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  copy_states(a.U, a.b.bmem + (size_t)blk * a.b.mstride, a.b.mstride, lds0, 256);
  copy_records<NU>(a.b, blk, lds0 + 32 * a.b.bmax, 256);
  const int cell = a.b.pack[tile * kTile + c];
  const bool live = cell >= 0, frozen = a.frozen != 0;
  const bool small = CW || frozen || a.variant != 1;
  const unsigned* __restrict__ words = a.b.bslot + (size_t)tile * (slot_words(NL) * 64);
  const double2* __restrict__ np = a.b.N + (size_t)tile * (normal_quads(NU) * 64);
  const double2* __restrict__ jc = a.b.jac + (size_t)tile * (2 * kTile);
  const float2 ce = (a.b.centre + (size_t)tile * (4 * kTile))[4 * c + wave];
  const double2 ja = jc[2 * c], jb = jc[2 * c + 1];
  CellView cv;
  cv.us = reinterpret_cast<const double*>(lds);
  cv.geo = reinterpret_cast<const double*>(lds + 32 * a.b.bmax);
  cv.g = g;
  const int own_slot = (tile - blk * a.b.bwaves) * kTile + c;
  const double* own = cv.geo + own_slot * (2 * rec_units(NU));
  auto staged = [&]() {
    lds_copy_wait();
    __syncthreads();
    cv.x = own[0];
    cv.y = own[1];
    static_for<0, 4>([&](auto i) { cv.u0[i] = cv.us[own_slot * 4 + (g ^ i)]; });
  };
  double* ex = reinterpret_cast<double*>(lds) + lane;
  if (wave == 3) {
    double r[NU], aK[NU];
    RowSlots<row_groups(NL), kSlotBits> slots;
    static_for<0, slots.NW>([&](auto k) { slots.w[k] = words[(3 + k) * 64 + lane]; });
    NormalMatrix<NU, TileAhead<P>::CH> nl;
    nl.template load<0>(np + 3 * QS * 64, lane);
    staged();
    const bool shift = __any(ce.x != 0.0f || ce.y != 0.0f);
    stencil_sums<R, NL, 0, NU, split_degree(P)>(cv, slots, own, ce.x, ce.y, shift, r);
    nl.apply(np + 3 * QS * 64, lane, r, aK);
    hermite_to_monomials<R>(aK, ce.x, ce.y, shift);
    Frame<R> fr;
    fr.init(ja, jb);
    fr.template to_basis<R>(aK);
    __syncthreads();  // every wavefront is done with the staged members
    static_for<0, NU>([&](auto l) { ex[(3 * kSmallCoef + l) * 64] = aK[l]; });
  } else {
    double r[kSmallCoef], as[kSmallCoef];
    Small slots;
    slots.w[0] = words[wave * 64 + lane];
    NormalMatrix<kSmallCoef> ns;
    ns.template load<0>(np + QS * wave * 64, lane);
    staged();
    static_for<0, kSmallCoef>([&](auto l) { as[l] = 0.0; });
    if (small) {
      stencil_sums<2, kSmallRows, 0, NU, 2>(cv, slots, own, ce.x, ce.y, true, r);
      ns.apply(np, lane, r, as);
      hermite_to_monomials<2>(as, ce.x, ce.y, true);
      Frame<2> fr;
      fr.init(ja, jb);
      fr.template to_basis<2>(as);
    }
    __syncthreads();
    static_for<0, kSmallCoef>([&](auto l) { ex[(wave * kSmallCoef + l) * 64] = as[l]; });
  }
  __syncthreads();
  if (wave != 0) return;
  double as[3][5], aK[NU];
  static_for<0, 3>([&](auto q) { static_for<0, 5>([&](auto l) { as[q][l] = ex[(5 * q + l) * 64]; }); });
  static_for<0, NU>([&](auto l) { aK[l] = ex[(3 * kSmallCoef + l) * 64]; });
  double* gram = reinterpret_cast<double*>(lds) + (3 * kSmallCoef + NU) * 64;
  if constexpr (CH && CW)
    char_edges_cweno_gram<P, NQ>(a, as, aK, cv.u0[0], cell, live, g, g, c, lane, gram);
  else if constexpr (CH)
    char_edges_gram<P, NQ>(a, as, aK, cv.u0[0], cell, live, g, g, c, lane, gram);
  else
    select_and_store<P, NQ, CW>(a, frozen, as, aK, cv.u0[0], cell, live, g, g, lane);
}

// Cells solved with operators (internal.h), in sets of four.
struct KeptArgs {
  const int* __restrict__ cell;    // [4 n] -1: none
  const int* __restrict__ rows;    // [n][kept_groups][64]
  const double* __restrict__ ops;  // [n][kept_chunks][64]
  int n;
};

// Sum over a cell's sixteen lanes of variable g, from sums x[i] of variable i ^ g:
// the same bits in its four quads.
__device__ __forceinline__ double kept_sum(const double (&x)[4]) {
  double s = quad_sum(x);
  s += quad_perm_dpp<0x128>(s);  // row_ror:8
  s += quad_perm_dpp<0x124>(s);  // row_ror:4
  return s;
}

// Their reconstruction, one wavefront per set, operators and members' states from
// memory: sixteen lanes per cell, so that all loads of a wavefront are in flight at
// once (few cells: what counts is the chain of loads, not their number).  The
// selection is that of the other cells, done alike by the four quads of a cell, of
// which the first writes.  5 to 8 us after the main launch (8,192 cells of a graded
// sector, 1-5% of them kept, orders 3-6); four lanes per cell took 8 to 27.
template <int N, int NR>
__device__ __forceinline__ void operator_sums(const double* __restrict__ U,
                                              const int* __restrict__ rows,
                                              const double* __restrict__ M, int lane, int g,
                                              const double (&u0)[4], double* c) {
  double acc[N][4];
  static_for<0, kept_row_groups(NR)>([&](auto j) {
    const double* u = U + (size_t)rows[j * 64 + lane] * 4;
    double d[4];
    static_for<0, 4>([&](auto i) { d[i] = u[g ^ i] - u0[i]; });
    static_for<0, N>([&](auto l) {
      const double x = M[(j * N + l) * 64 + lane];
      static_for<0, 4>([&](auto i) { acc[l][i] = j == 0 ? x * d[i] : fma(x, d[i], acc[l][i]); });
    });
  });
  static_for<0, N>([&](auto l) { c[l] = kept_sum(acc[l]); });
}

template <int P, int NQ, bool CW, bool CH>
__device__ __forceinline__ void reconstruct_kept(TENO_CONST ReconArgs& a, const KeptArgs& k, int set,
                                                 double* gram) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NL = O::NL;
  constexpr int GS = kept_row_groups(kSmallRows), CS = GS * kSmallCoef;
  const int lane = threadIdx.x & 63, c = lane >> 2, g = lane & 3;
  const int at = k.cell[set * kKeptCells + (lane >> 4)];
  const int cell = max(at, 0);
  const bool live = at >= 0 && (lane & 15) < 4;
  const double* __restrict__ U = a.U;
  const int* __restrict__ rows = k.rows + (size_t)set * (kept_groups(NL) * 64);
  const double* __restrict__ M = k.ops + (size_t)set * (kept_chunks(NL, NU) * 64);
  double u0[4], aK[NU], as[3][5];
  static_for<0, 4>([&](auto i) { u0[i] = U[(size_t)cell * 4 + (g ^ i)]; });
  static_for<0, 3>([&](auto q) {
    operator_sums<kSmallCoef, kSmallRows>(U, rows + GS * q * 64, M + CS * q * 64, lane, g, u0, as[q]);
  });
  operator_sums<NU, NL>(U, rows + 3 * GS * 64, M + 3 * CS * 64, lane, g, u0, aK);
  if constexpr (CH && CW)
    char_edges_cweno_gram<P, NQ>(a, as, aK, u0[0], cell, live, g, g, c, lane, gram);
  else if constexpr (CH)
    char_edges_gram<P, NQ>(a, as, aK, u0[0], cell, live, g, g, c, lane, gram);
  else
    select_and_store<P, NQ, CW>(a, a.frozen != 0, as, aK, u0[0], cell, live, g, g, lane);
}

template <int P, int NQ, bool CW, bool CH>
__global__ __launch_bounds__(64) void k_reconstruct_kept(ReconArgs, KeptArgs k) {
  __shared__ double gram[CH ? kCharGramDoubles : 1];
  reconstruct_kept<P, NQ, CW, CH>(
      *(TENO_CONST ReconArgs*)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr(), k, blockIdx.x, gram);
}

// ---------------------------------------------------------------------------
// flux, residual, Runge-Kutta stage
// ---------------------------------------------------------------------------
// Flux and residual (Sec. 2.1, Sec. 4), in two launches.
//  face_flux    one lane per face (faces sorted by their L cell): rotated HLL
//               at the N_q point pairs (L point k with R point N_q-1-k),
//               Gauss quadrature, Phi_f = |A| sum_k w_k F_k, written once.
//  cell_update  one lane per cell: R = -(1/|V|) sum_e s_e Phi_f(e) over its
//               three faces in local-edge order (s = +1 on the L side), then
//               the optional SSP-RK3 stage combine.  A gather: no atomics.
struct FaceFluxArgs {
  const double* __restrict__ fp;       // [3 nq][n_pad][4]
  const int4* __restrict__ fcell;      // [n_face]: L, R, eL | eR << 2, boundary index or -1
  const double2* __restrict__ fgeo;    // [n_face][2]: (nx, ny), (|A|, 0)
  double* __restrict__ phi;            // [n_face][4]
  const int* __restrict__ bkind;       // [n_bface] TENO_BC_*
  const double* __restrict__ bstate;   // [n_bface][4] prescribed states
  double gamma;
  int n_face, n_pad;
};

// Outer state of boundary face b at one Gauss point (normal (nx, ny) out of
// the domain): transmissive copies the inner state, reflective reverses its
// normal momentum, prescribed takes the given state.
__device__ __forceinline__ void boundary_state(int kind, const double* __restrict__ bstate, int b,
                                               const double uL[4], double nx, double ny,
                                               double uR[4]) {
  if (kind == TENO_BC_PRESCRIBED) {
#pragma unroll
    for (int c = 0; c < 4; ++c) uR[c] = bstate[4 * (size_t)b + c];
  } else if (kind == TENO_BC_REFLECTIVE) {
    const double mn = uL[1] * nx + uL[2] * ny;
    uR[0] = uL[0];
    uR[1] = uL[1] - 2.0 * mn * nx;
    uR[2] = uL[2] - 2.0 * mn * ny;
    uR[3] = uL[3];
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) uR[c] = uL[c];
  }
}

// Phi of face f.  KIND 0: as if no face lay on the boundary; 1: f is boundary
// face b; 2: what the face's record says.
template <int NQ, int KIND>
__device__ __forceinline__ void face_phi(const FaceFluxArgs& a, int f, int b, double (&out)[4]) {
  const int4 fc = a.fcell[f];
  const double2 nrm = a.fgeo[2 * (size_t)f], len = a.fgeo[2 * (size_t)f + 1];
  const int eL = fc.z & 3, eR = (fc.z >> 2) & 3;
  const double2* fp2 = reinterpret_cast<const double2*>(a.fp);
  double phi[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const size_t oL = ((size_t)(eL * NQ + k) * a.n_pad + fc.x) * 2;
    const double2 l0 = fp2[oL], l1 = fp2[oL + 1];
    const double uL[4] = {l0.x, l0.y, l1.x, l1.y};
    double uR[4];
    if constexpr (KIND == 1) {
      boundary_state(a.bkind[b], a.bstate, b, uL, nrm.x, nrm.y, uR);
    } else {
      const size_t oR = ((size_t)(eR * NQ + NQ - 1 - k) * a.n_pad + fc.y) * 2;
      const double2 r0 = fp2[oR], r1 = fp2[oR + 1];
      uR[0] = r0.x;
      uR[1] = r0.y;
      uR[2] = r1.x;
      uR[3] = r1.y;
      if constexpr (KIND == 2)
        if (fc.w >= 0) boundary_state(a.bkind[fc.w], a.bstate, fc.w, uL, nrm.x, nrm.y, uR);
    }
    double F[4];
    hll(uL, uR, nrm.x, nrm.y, a.gamma, F);
#pragma unroll
    for (int c = 0; c < 4; ++c) phi[c] = phi[c] + FaceRule<NQ>::w[k] * F[c];
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) out[c] = phi[c] * len.x;
}

template <int NQ, bool BND = false>
__device__ __forceinline__ void face_flux(const FaceFluxArgs& a, int f, int b = -1) {
  double p[4];
  face_phi<NQ, BND ? 1 : 0>(a, f, b, p);
  double2* out = reinterpret_cast<double2*>(a.phi) + 2 * (size_t)f;
  out[0] = make_double2(p[0], p[1]);
  out[1] = make_double2(p[2], p[3]);
}

// Every face, boundary faces included as if their outer side were the cell
// itself; k_boundary_flux then rewrites the boundary faces.
template <int NQ>
__global__ __launch_bounds__(256) void k_face_flux(FaceFluxArgs a) {
  const int f = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (f < a.n_face) face_flux<NQ>(a, f);
}

// Boundary faces only (after k_face_flux, same stream): bf[b] is the face
// index of boundary face b, whose outer state comes from its condition.
template <int NQ>
__global__ __launch_bounds__(256) void k_boundary_flux(FaceFluxArgs a, const int* __restrict__ bf,
                                                       int n_bface) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < n_bface) face_flux<NQ, true>(a, bf[b], b);
}

struct CellUpdateArgs {
  const int4* __restrict__ cfaces;     // [n_pad]: faces of local edges 0..2, L bits
  const double* __restrict__ vol;      // [n_pad]
  const double* __restrict__ phi;      // [n_face][4]
  const double* Un;                    // [n][4]
  const double* Uk;                    // [n][4]
  double* out;                         // R or U^(k+1)
  const double* dt;                    // device scalar
  double ca, cb, cc;                   // out = ca Un + cb Uk + cc (dt R)
  int n_cell;
};

template <bool RK>
__device__ __forceinline__ void cell_update(const CellUpdateArgs& a, int t, double* kept = nullptr) {
  const int4 cf = a.cfaces[t];
  const double2* ph = reinterpret_cast<const double2*>(a.phi);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const size_t f = (size_t)(e == 0 ? cf.x : (e == 1 ? cf.y : cf.z));
    const bool isL = (cf.w >> e) & 1;
    const double2 x = ph[2 * f], y = ph[2 * f + 1];
    const double p[4] = {x.x, x.y, y.x, y.y};
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = isL ? acc[c] + p[c] : acc[c] - p[c];
  }
  const double ia = -1.0 / a.vol[t];
  double R[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) R[c] = acc[c] * ia;
  double* o = a.out + (size_t)t * 4;
  if (RK) {
    const double dt = *a.dt;
    const double* un = a.Un + (size_t)t * 4;
    const double* uk = a.Uk + (size_t)t * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double x = a.ca * un[c] + a.cb * uk[c] + a.cc * (dt * R[c]);
      o[c] = x;
      if (kept) kept[c] = x;
    }
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] = R[c];
  }
}

template <bool RK>
__global__ __launch_bounds__(256) void k_cell_update(CellUpdateArgs a) {
  const int t = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (t < a.n_cell) cell_update<RK>(a, t);
}

// ---------------------------------------------------------------------------
// time step
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_min(double x, double* sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmin(x, __shfl_xor(x, o));
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < (int)(blockDim.x >> 6); ++k) x = fmin(x, sh[k]);
    sh[0] = x;
  }
  __syncthreads();
  return sh[0];
}

// |V_i| / sum_j |A_ij| (|u_i . n_ij| + c_i) from the cell average u of cell t.
__device__ __forceinline__ double dt_limit_of(const double* u, const double* __restrict__ geo,
                                              int t, double g) {
  const double* gg = geo + (size_t)t * 10;
  const double vx = u[1] / u[0], vy = u[2] / u[0];
  const double p = (g - 1.0) * (u[3] - 0.5 * u[0] * (vx * vx + vy * vy));
  const double c = sqrt(g * p / u[0]);
  double den = 0.0;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const double un = vx * gg[3 * e] + vy * gg[3 * e + 1];
    den = den + gg[3 * e + 2] * (fabs(un) + c);
  }
  return gg[9] / den;
}

__device__ __forceinline__ double cell_dt_limit(const double* __restrict__ U,
                                                const double* __restrict__ geo, int t, double g) {
  return dt_limit_of(U + (size_t)t * 4, geo, t, g);
}

// The last stage's gather and update, fused with the first half of the
// constant-CFL step of the state it writes: each block's minimum of
// |V_i| / sum_j |A_ij| (|u_i . n_ij| + c_i) over its new cell averages, from
// the values in registers and with k_dt_partial's arithmetic, so that
// k_dt_final over these minima gives teno_max_dt of the new state bit for
// bit.  (The minima are reduced by a second launch, not by the last block
// to finish: on this multi-die GPU the device-scope fence that would order
// each block's minimum before its count writes back the block's whole L2.)
__global__ __launch_bounds__(256) void k_cell_update_dt(CellUpdateArgs a,
                                                        const double* __restrict__ geo, double g,
                                                        double* __restrict__ partial) {
  __shared__ double sh[4];
  const int t = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  double lim = INFINITY;
  if (t < a.n_cell) {
    double u[4];
    cell_update<true>(a, t, u);
    lim = dt_limit_of(u, geo, t, g);
  }
  const double m = block_min(lim, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

// Flux, gather and update in one launch, four lanes per cell: lane e < 3 forms
// the Phi of the cell's local edge e as the face's own lane would, and the four
// lanes add them in edge order, so the results are those of the separate kernels
// bit for bit.  Every face is formed twice (both its cells), which a small mesh
// does not notice: it waits for launches.  DT: also the block's minimum of the
// next step's limit, as k_cell_update_dt.
template <int NQ, bool RK, bool DT>
__global__ __launch_bounds__(256) void k_cell_flux_update(FaceFluxArgs fa, CellUpdateArgs a,
                                                          const double* __restrict__ geo,
                                                          double* __restrict__ partial) {
  const int t = xcd_remap(blockIdx.x, gridDim.x) * 64 + (threadIdx.x >> 2), e = threadIdx.x & 3;
  const bool live = t < a.n_cell;
  const int4 cf = a.cfaces[live ? t : 0];
  double p[4] = {0.0, 0.0, 0.0, 0.0};
  if (live && e < 3) face_phi<NQ, 2>(fa, e == 0 ? cf.x : (e == 1 ? cf.y : cf.z), -1, p);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  static_for<0, 3>([&](auto k) {
    static_for<0, 4>([&](auto c) {
      const double x = quad_bcast<k>(p[c]);
      acc[c] = (cf.w >> k) & 1 ? acc[c] + x : acc[c] - x;
    });
  });
  const double own = e == 0 ? acc[0] : (e == 1 ? acc[1] : (e == 2 ? acc[2] : acc[3]));
  double u = 0.0;
  if (live) {
    const double ia = -1.0 / a.vol[t];
    const double R = own * ia;
    const size_t o = 4 * (size_t)t + e;
    u = R;
    if (RK) u = a.ca * a.Un[o] + a.cb * a.Uk[o] + a.cc * (*a.dt * R);
    a.out[o] = u;
  }
  if constexpr (DT) {
    __shared__ double sh[4];
    double w[4];
    static_for<0, 4>([&](auto c) { w[c] = quad_bcast<c>(u); });
    const double m = block_min(live ? dt_limit_of(w, geo, t, fa.gamma) : INFINITY, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = m;
  }
}
// Taken up to 65,536 / nq cells.  Linear residuals (fused against separate, us),
// two points per face: 11.8 against 15.3 at 2,048 cells, 14.8 / 15.2 at 32,768,
// 24.7 / 22.9 at 65,522; three: 17.7 / 19.0 at 2,048, 20.6 / 21.5 at 14,450,
// 25.8 / 24.7 at 32,768.
constexpr bool fuse_update(int n_cell, int nq) { return n_cell <= 65536 / nq; }

__global__ __launch_bounds__(256) void k_dt_partial(const double* __restrict__ U,
                                                    const double* __restrict__ geo, int n,
                                                    double g, double* __restrict__ partial) {
  __shared__ double sh[4];
  const int t = blockIdx.x * 256 + threadIdx.x;
  const double lim = t < n ? cell_dt_limit(U, geo, t, g) : INFINITY;
  const double m = block_min(lim, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

__global__ __launch_bounds__(256) void k_dt_final(const double* __restrict__ partial, int n,
                                                  double cfl, double* __restrict__ dt) {
  __shared__ double sh[4];
  double x = INFINITY;
  for (int i = threadIdx.x; i < n; i += 256) x = fmin(x, partial[i]);
  const double m = block_min(x, sh);
  if (threadIdx.x == 0) *dt = cfl * m;
}

// ---------------------------------------------------------------------------
// adjoint of the residual (selection frozen)
// ---------------------------------------------------------------------------
// Phase 1 (one lane per face): adjoint of the face-point states.  Face f
// gets Phi_bar = lam_R/|V_R| - lam_L/|V_L| (scaled by `scale`); at each of
// its Gauss points the lane runs the reverse mode of the HLL flux (hll_vjp)
// and writes both sides' face-point adjoints.
struct AdjFaceArgs {
  const double* __restrict__ fp;      // [3 nq][n_pad][4]
  const int4* __restrict__ fcell;     // [n_face]: L, R, eL | eR << 2
  const double2* __restrict__ fgeo;   // [n_face][2]: (nx, ny), (|A|, 0)
  const double* __restrict__ vol;     // [n_pad]
  const double* __restrict__ lam;
  const double* scale_dev;            // device scalar multiplying lam (nullable = 1)
  double scale;
  double* __restrict__ fpbar;         // [3 nq][n_pad][4]
  const int* __restrict__ bkind;      // [n_bface] boundary conditions (meshes with open axes)
  const double* __restrict__ bstate;  // [n_bface][4] prescribed states
  double gamma;
  int n_face, n_pad;
};

template <int NQ>
__device__ __forceinline__ void adj_face(const AdjFaceArgs& a, int f) {
  const int4 fc = a.fcell[f];
  const double2 nrm = a.fgeo[2 * (size_t)f], len = a.fgeo[2 * (size_t)f + 1];
  const int L = fc.x, R = fc.y, eL = fc.z & 3, eR = (fc.z >> 2) & 3;
  const double sc = a.scale * (a.scale_dev ? *a.scale_dev : 1.0);
  const double aL = a.vol[L], aR = a.vol[R];
  double pb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    pb[c] = sc * (a.lam[(size_t)R * 4 + c] / aR - a.lam[(size_t)L * 4 + c] / aL);
  const double2* fp2 = reinterpret_cast<const double2*>(a.fp);
  double2* out2 = reinterpret_cast<double2*>(a.fpbar);
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int qL = eL * NQ + k, qR = eR * NQ + NQ - 1 - k;
    const size_t oL = ((size_t)qL * a.n_pad + L) * 2, oR = ((size_t)qR * a.n_pad + R) * 2;
    const double2 l0 = fp2[oL], l1 = fp2[oL + 1], r0 = fp2[oR], r1 = fp2[oR + 1];
    const double vl[4] = {l0.x, l0.y, l1.x, l1.y}, vr[4] = {r0.x, r0.y, r1.x, r1.y};
    double gL[4] = {0.0, 0.0, 0.0, 0.0}, gR[4] = {0.0, 0.0, 0.0, 0.0};
    hll_vjp(vl, vr, nrm.x, nrm.y, a.gamma, pb, gL, gR);
    const double w = len.x * FaceRule<NQ>::w[k];
    out2[oL] = make_double2(w * gL[0], w * gL[1]);
    out2[oL + 1] = make_double2(w * gL[2], w * gL[3]);
    out2[oR] = make_double2(w * gR[0], w * gR[1]);
    out2[oR + 1] = make_double2(w * gR[2], w * gR[3]);
  }
}

template <int NQ>
__global__ __launch_bounds__(256) void k_adj_faces(AdjFaceArgs a) {
  const int f = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (f >= a.n_face) return;
  adj_face<NQ>(a, f);
}

// Boundary faces only (after k_adj_faces, same stream; bf[b] is the face of
// boundary face b).  Only the inner cell's term enters the face's adjoint,
// and the outer state follows the inner one through the face's condition,
// so the inner side also takes the outer side's adjoint through that map,
// transposed: the identity (transmissive), the mirror I - 2 n n^T of the
// momentum (reflective, symmetric), nothing (prescribed).  Rewrites every
// face point of the edge, which k_adj_faces filled as if the cell were on
// both sides.
template <int NQ>
__global__ __launch_bounds__(256) void k_adj_boundary(AdjFaceArgs a, const int* __restrict__ bf,
                                                      int n_bface) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= n_bface) return;
  const int f = bf[b];
  const int4 fc = a.fcell[f];
  const double2 nrm = a.fgeo[2 * (size_t)f], len = a.fgeo[2 * (size_t)f + 1];
  const int L = fc.x, eL = fc.z & 3, kind = a.bkind[b];
  const double sc = a.scale * (a.scale_dev ? *a.scale_dev : 1.0);
  const double aL = a.vol[L];
  double pb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) pb[c] = -sc * (a.lam[(size_t)L * 4 + c] / aL);
  const double2* fp2 = reinterpret_cast<const double2*>(a.fp);
  double2* out2 = reinterpret_cast<double2*>(a.fpbar);
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const size_t oL = ((size_t)(eL * NQ + k) * a.n_pad + L) * 2;
    const double2 l0 = fp2[oL], l1 = fp2[oL + 1];
    const double uL[4] = {l0.x, l0.y, l1.x, l1.y};
    double uR[4];
    boundary_state(kind, a.bstate, b, uL, nrm.x, nrm.y, uR);
    double gL[4] = {0.0, 0.0, 0.0, 0.0}, gR[4] = {0.0, 0.0, 0.0, 0.0};
    hll_vjp(uL, uR, nrm.x, nrm.y, a.gamma, pb, gL, gR);
    if (kind == TENO_BC_TRANSMISSIVE) {
#pragma unroll
      for (int c = 0; c < 4; ++c) gL[c] += gR[c];
    } else if (kind == TENO_BC_REFLECTIVE) {
      const double gn = gR[1] * nrm.x + gR[2] * nrm.y;
      gL[0] += gR[0];
      gL[1] += gR[1] - 2.0 * gn * nrm.x;
      gL[2] += gR[2] - 2.0 * gn * nrm.y;
      gL[3] += gR[3];
    }
    const double w = len.x * FaceRule<NQ>::w[k];
    out2[oL] = make_double2(w * gL[0], w * gL[1]);
    out2[oL + 1] = make_double2(w * gL[2], w * gL[3]);
  }
}

// Phase 2 (one wavefront per tile, four lanes per cell): transpose of the
// reconstruction.  Lane v forms the adjoints of variable v's coefficients from
// its face points and, per stencil that a variable of the wavefront keeps,
// z = N times them (in the block's frame).  The cell's four lanes share z, and
// lane g takes rows 4j + g for all four variables, as the forward kernel does:
// the adjoint of difference d_s is w_s A_s^T z, with A_s from the staged
// records.  It goes to the tile's member slot of U_s, summed in LDS (one
// accumulator per distinct member of the tile and variable) in a fixed order:
// the lanes of a group of rows that name the same member add in rounds that
// set-up assigns, so no LDS instruction has two lanes on one address.  The
// tile's sums are written once to tbar; the cell's own part (the -U_0 of its
// differences and its face points) goes to own[n][4].
struct AdjReconArgs {
  const double* __restrict__ fpbar;
  const uint16_t* __restrict__ flags;
  BlockArgs b;
  const unsigned* __restrict__ aslot;  // [n_tiles][adj_words][64]: slot | round << 9
  double* __restrict__ tbar;      // [n_tiles][ustride][4], then [kept rows][4]
  double* __restrict__ own;       // [n_pad][4]
  int ustride;
  int n_cell, n_tiles, n_pad;
};

// Rows of one stencil: adjoints of its differences from z (the lane's own
// variable), added to acc; returns the lane's sums over its rows in dq.
// VP variables at a time: two passes form the moments twice, where the shared z
// of all four would not fit the registers.
template <int R, int NR, int G0, int NU, int VP, class Slots, class AdjSlots>
__device__ __forceinline__ void adj_rows(const CellView& cv, const Slots& slots,
                                         const AdjSlots& aslots, const double* own,
                                         double cx, double cy, bool shift, double* z,
                                         double* acc, double (&dq)[4]) {
  constexpr int N = (R + 1) * (R + 2) / 2 - 1;
  constexpr int RS = 2 * rec_units(NU);
  // zero mean of the rows over the cell
  double h[N];
  own_moments<R>(own, cx, cy, shift, h);
  double z0 = 0.0;
  static_for<0, N>([&](auto l) { z0 = fma(-h[l], z[l], z0); });
  const double x0 = cv.x + cx, y0 = cv.y + cy;
  static_for<0, 4 / VP>([&](auto pc) {
    constexpr int I0 = pc * VP;
    double zq[N][VP], z0q[VP];
    opaque(z0);  // (or every pass's exchange is formed ahead and held)
    static_for<0, N>([&](auto l) { opaque(z[l]); });
    static_for<0, VP>([&](auto i) {
      z0q[i] = quad_xor<I0 + i>(z0);
      static_for<0, N>([&](auto l) { zq[l][i] = quad_xor<I0 + i>(z[l]); });
    });
    static_for<0, row_groups(NR)>([&](auto jc) {
      unsigned m = slots.template get<G0 + jc>();
      asm volatile("" : "+v"(m));  // each pass reads its records again
      const unsigned w = aslots.template get<G0 + jc>();
      const double* rec = cv.geo + m * RS;
      double q[N + 1], mo[N], d[VP];
      static_for<0, N + 1>([&](auto l) { q[l] = rec[l]; });
      shift_moments<R>(q[0] - x0, q[1] - y0, q + 3, mo);
      const bool row = 4 * jc + cv.g < NR;
      static_for<0, VP>([&](auto i) {
        double t = z0q[i];
        static_for<0, N>([&](auto l) { t = fma(mo[l], zq[l][i], t); });
        d[i] = row ? t * q[2] : 0.0;
        dq[I0 + i] += d[i];
      });
      double* dst = acc + (w & 511) * 4;
      const int mine = row ? (int)(w >> 9) : -1;
      for (int r = 0; __any(mine >= r); ++r)
        if (mine == r) static_for<0, VP>([&](auto i) { atomicAdd(dst + (cv.g ^ (I0 + i)), d[i]); });
    });
  });
}

// The adjoint's: three at order 4 too, 44.5 against 50.1 us where most cells keep
// the large stencil alone (131,072 cells, random lines, which smooth out along a
// rollout) and 64.0 against 73.8 us where few do (random states of every cell).
constexpr int adj_waves(int p) { return p <= 4 ? 3 : 2; }

template <int P, int NQ>
__global__ __launch_bounds__(64 * block_tiles(P))
__attribute__((amdgpu_waves_per_eu(adj_waves(P)))) void k_adj_recon(AdjReconArgs a) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NL = O::NL, R = O::R;
  constexpr int NP = 3 * NQ;
  constexpr int GS = row_groups(kSmallRows), QS = sym_quads(kSmallCoef);
  extern __shared__ int4 lds4[];  // records, then bwaves x ustride x 4 doubles
  char* lds = reinterpret_cast<char*>(lds4);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = blk * a.b.bwaves + wave;
  double* accs = reinterpret_cast<double*>(lds + 16 * rec_units(NU) * a.b.bmax);
  for (int i = threadIdx.x; i < 4 * a.b.bwaves * a.ustride; i += blockDim.x) accs[i] = 0.0;
  copy_records<NU>(((TENO_CONST AdjReconArgs*)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr())->b,
                   blk, (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds,
                   blockDim.x);
  lds_copy_wait();
  __syncthreads();
  if (tile >= a.n_tiles) return;  // whole wavefront leaves together
  double* acc = accs + (size_t)wave * a.ustride * 4;
  const int c = lane >> 2, v = lane & 3;
  const int pos = tile * kTile + c, cell = a.b.pack[pos];
  const bool live = cell >= 0;
  const int cl = live ? cell : 0;
  MemberSlots<NL> slots;
  slots.load(a.b.bslot, tile, lane);
  RowSlots<lane_groups(NL), 16> aslots;
  aslots.load(a.aslot, tile, lane);
  CellView cv;
  cv.us = nullptr;
  cv.geo = reinterpret_cast<const double*>(lds);
  cv.g = v;
  const double* own = cv.geo + (wave * kTile + c) * (2 * rec_units(NU));
  cv.x = own[0];
  cv.y = own[1];
  const double2* __restrict__ np = a.b.N + (size_t)tile * (normal_quads(NU) * 64);
  const double2* __restrict__ jp = a.b.jac + 2 * (size_t)pos;
  const float2* __restrict__ cen = a.b.centre + 4 * (size_t)pos;
  Frame<R> fr;
  fr.init(jp[0], jp[1]);
  const unsigned nib = live ? ((a.flags[cl] >> (4 * v)) & 0xFu) : 0u;
  double gsum = 0.0;
  double ab[NU];
#pragma unroll
  for (int l = 0; l < NU; ++l) ab[l] = 0.0;
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const double gq = live ? a.fpbar[((size_t)q * a.n_pad + cl) * 4 + v] : 0.0;
    gsum += gq;
#pragma unroll
    for (int l = 0; l < NU; ++l) ab[l] = fma(FaceBasis<O::R, NQ>::P.v[q][l], gq, ab[l]);
  }
  // adjoints of the frame's coefficients (the small stencils' basis is the
  // first functions of the large one)
  static_for<0, NU>([&](auto l) { opaque(ab[l]); });
  fr.template from_basis_adjoint<R>(ab);
  static_for<0, NU>([&](auto l) { opaque(ab[l]); });
  const bool keepK = nib & 8u;
  const int cnt = (int)(nib & 1u) + (int)((nib >> 1) & 1u) + (int)((nib >> 2) & 1u);
  double dq[4] = {0.0, 0.0, 0.0, 0.0};
  // ---- small stencils: each kept one counts 1/cnt where step two decided ----
  static_for<0, 3>([&](auto k) {
    const bool kept = !keepK && ((nib >> k) & 1u);
    if (!__any(kept)) return;
    const double w = kept ? 1.0 / (double)cnt : 0.0;
    double r[kSmallCoef], z[kSmallCoef];
#pragma unroll
    for (int l = 0; l < kSmallCoef; ++l) r[l] = w * ab[l];
    const float2 ce = cen[k];
    hermite_to_monomials_adjoint<2>(r, ce.x, ce.y, true);
    NormalMatrix<kSmallCoef> nm;
    nm.template load<0>(np + QS * k * 64, lane);
    nm.apply(np, lane, r, z);
    static_for<0, kSmallCoef>([&](auto l) { opaque(z[l]); });
    adj_rows<2, kSmallRows, GS * k, NU, 4>(cv, slots, aslots, own, ce.x, ce.y, true, z, acc, dq);
  });
  // ---- large stencil ----
  if (__any(keepK)) {
    double z[NU];
#pragma unroll
    for (int l = 0; l < NU; ++l) ab[l] = keepK ? ab[l] : 0.0;
    const float2 ce = cen[3];
    const bool shift = __any(ce.x != 0.0f || ce.y != 0.0f);
    hermite_to_monomials_adjoint<R>(ab, ce.x, ce.y, shift);
    static_for<0, NU>([&](auto l) { opaque(ab[l]); });
    NormalMatrix<NU, TileAhead<P>::CH> nm;
    nm.template load<0>(np + 3 * QS * 64, lane);
    nm.apply(np + 3 * QS * 64, lane, ab, z);
    static_for<0, NU>([&](auto l) { opaque(z[l]); });  // (no part of it sinks past a branch)
    adj_rows<R, NL, 3 * GS, NU, (P >= 5 ? 2 : 4)>(cv, slots, aslots, own, ce.x, ce.y, shift, z, acc, dq);
  }
  const double dsum = quad_sum(dq);
  if (live) a.own[(size_t)cell * 4 + v] = gsum - dsum;
  wave_lds_sync();
  double* __restrict__ tb = a.tbar + (size_t)tile * a.ustride * 4;
  for (int i = lane; i < 4 * a.ustride; i += 64) tb[i] = acc[i];
}

// The same for the cells solved with operators, one wavefront per set of them.
// What a row adds to its member goes to a place of its own in tbar (after the
// tiles' sums), which the member's reverse list names.
template <int N, int NR>
__device__ __forceinline__ void adj_operator(const double* __restrict__ M, int lane, int g,
                                             const double* ab, double* __restrict__ out,
                                             double (&dq)[4]) {
  static_for<0, kept_row_groups(NR)>([&](auto j) {
    double d[4] = {0.0, 0.0, 0.0, 0.0};
    static_for<0, N>([&](auto l) {
      const double x = M[(j * N + l) * 64 + lane];
      static_for<0, 4>([&](auto i) { d[i] = fma(x, quad_xor<i>(ab[l]), d[i]); });
    });
    if (16 * j + (lane & 15) < NR) static_for<0, 4>([&](auto i) {
      dq[i] += d[i];
      out[(j * 64 + lane) * 4 + (g ^ i)] = d[i];
    });
  });
}

template <int P, int NQ>
__global__ __launch_bounds__(64) void k_adj_recon_kept(AdjReconArgs a, KeptArgs k) {
  using O = OrderT<P>;
  constexpr int NU = O::NU, NL = O::NL;
  constexpr int GS = kept_row_groups(kSmallRows), CS = GS * kSmallCoef;
  const int lane = threadIdx.x, v = lane & 3, set = blockIdx.x;
  const int cell = k.cell[set * kKeptCells + (lane >> 4)];
  const bool live = cell >= 0;
  const int cl = live ? cell : 0;
  const unsigned nib = live ? ((a.flags[cl] >> (4 * v)) & 0xFu) : 0u;
  double gsum = 0.0, ab[NU];
  static_for<0, NU>([&](auto l) { ab[l] = 0.0; });
  static_for<0, 3 * NQ>([&](auto q) {
    const double gq = live ? a.fpbar[((size_t)q * a.n_pad + cl) * 4 + v] : 0.0;
    gsum += gq;
    static_for<0, NU>([&](auto l) { ab[l] = fma(FaceBasis<O::R, NQ>::P.v[q][l], gq, ab[l]); });
  });
  const bool keepK = nib & 8u;
  const int cnt = (int)(nib & 1u) + (int)((nib >> 1) & 1u) + (int)((nib >> 2) & 1u);
  const double* __restrict__ M = k.ops + (size_t)set * (kept_chunks(NL, NU) * 64);
  double* __restrict__ out =
      a.tbar + ((size_t)a.n_tiles * a.ustride + (size_t)set * (kept_groups(NL) * 64)) * 4;
  double dq[4] = {0.0, 0.0, 0.0, 0.0};
  static_for<0, 3>([&](auto q) {
    const double w = !keepK && ((nib >> q) & 1u) ? 1.0 / (double)cnt : 0.0;
    double r[kSmallCoef];
    static_for<0, kSmallCoef>([&](auto l) { r[l] = w * ab[l]; });
    adj_operator<kSmallCoef, kSmallRows>(M + CS * q * 64, lane, v, r, out + GS * q * 256, dq);
  });
  static_for<0, NU>([&](auto l) { ab[l] = keepK ? ab[l] : 0.0; });
  adj_operator<NU, NL>(M + 3 * CS * 64, lane, v, ab, out + 3 * GS * 256, dq);
  const double dsum = kept_sum(dq);
  if (live && (lane & 15) < 4) a.own[(size_t)cell * 4 + v] = gsum - dsum;
}

// Phase 3 (four lanes per cell, lane q = variable q): U_bar[j] = own[j] +
// the tile sums of every tile member slot naming j and the rows of kept cells
// that do (reverse list rev_ptr[j] .. rev_ptr[j+1]-1), in list order: no atomics.  Then out = U_bar
// + beta * extra (extra nullable).
__global__ __launch_bounds__(256) void k_adj_gather(const double* __restrict__ own,
                                                    const double* __restrict__ tbar,
                                                    const int32_t* __restrict__ rev_ptr,
                                                    const int32_t* __restrict__ rev_ent,
                                                    int n_cell, const double* extra, double beta,
                                                    double* out) {
  const int gid = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  const int j = gid >> 2, q = gid & 3;
  if (j >= n_cell) return;
  const int b = rev_ptr[j], e = rev_ptr[j + 1];
  double s = 0.0;
  int t = b;
  for (; t + 3 < e; t += 4) {
    const int e0 = rev_ent[t], e1 = rev_ent[t + 1], e2 = rev_ent[t + 2], e3 = rev_ent[t + 3];
    const double x0 = tbar[(size_t)e0 * 4 + q], x1 = tbar[(size_t)e1 * 4 + q];
    const double x2 = tbar[(size_t)e2 * 4 + q], x3 = tbar[(size_t)e3 * 4 + q];
    s += x0;
    s += x1;
    s += x2;
    s += x3;
  }
  for (; t < e; ++t) s += tbar[(size_t)rev_ent[t] * 4 + q];
  double v = own[(size_t)j * 4 + q] + s;
  if (extra) v = v + beta * extra[(size_t)j * 4 + q];
  out[(size_t)j * 4 + q] = v;
}

// out = a1 x1 + a2 x2 (+ a3 x3), elementwise over n doubles.
__global__ __launch_bounds__(256) void k_lincomb(double* out, double a1, const double* x1,
                                                 double a2, const double* x2, double a3,
                                                 const double* x3, long n) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double s = a1 * x1[i];
  if (x2) s = s + a2 * x2[i];
  if (x3) s = s + a3 * x3[i];
  out[i] = s;
}

// ---------------------------------------------------------------------------
// batches of independent meshes
// ---------------------------------------------------------------------------
// One mesh of a batch: the arguments of its three RK stages.
struct BatchMeshDev {
  ReconArgs r[3];          // reconstruction input of stage k
  KeptArgs kept;           // cells solved with operators
  FaceFluxArgs ff;         // face fluxes (the same buffers every stage)
  CellUpdateArgs cu[3];    // gather and update of stage k
  const double* U;         // cell averages at the start of the step
  const double* geo;
  double* dt;              // this mesh's step (device scalar)
  const int* bface;        // [n_bface]: face of each boundary face
  double gamma;
  int pq;                  // order * 10 + face points
  int n_cell;
  int n_bface;
};

// Items of a batch's work list: (mesh, block).
struct BatchItems {
  const BatchMeshDev* __restrict__ meshes;
  const int2* __restrict__ items;
  int stage_k;
  __device__ __forceinline__ TENO_CONST ReconArgs& args(int k) const {
    const int m = scalar_load(reinterpret_cast<const int*>(items), 2 * k);
    return *(TENO_CONST ReconArgs*)(uintptr_t)&meshes[m].r[stage_k];
  }
  __device__ __forceinline__ int block(int k) const {
    return scalar_load(reinterpret_cast<const int*>(items), 2 * k + 1);
  }
};

// Reconstruction over items of one order and face-point count.  start: each
// workgroup takes the contiguous, cost-balanced range [start[w], start[w+1]);
// null: the n_items items are dealt out in turn.
template <int PQ>
__global__ __launch_bounds__(64 * block_tiles(PQ / 10))
__attribute__((amdgpu_waves_per_eu(recon_waves(PQ / 10)))) void k_batch_reconstruct(
    const BatchMeshDev* __restrict__ meshes, const int2* __restrict__ items,
    const int* __restrict__ start, int n_items, int stage_k) {
  extern __shared__ int4 lds[];
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const BatchItems it{meshes, items, stage_k};
  reconstruct_loop<PQ / 10, PQ % 10, false, false>(it, start ? start[w] : w,
                                                   start ? start[w + 1] : n_items,
                                                   start ? 1 : (int)gridDim.x,
                                                   reinterpret_cast<char*>(lds));
}

// One launch for every order: each item is dispatched by its mesh's order, one at
// a time (the pipeline of reconstruct_loop runs within one order).
__global__ __launch_bounds__(64 * kMaxBlockTiles) __attribute__((amdgpu_waves_per_eu(2)))
void k_batch_reconstruct_all(const BatchMeshDev* __restrict__ meshes,
                             const int2* __restrict__ items, const int* __restrict__ start,
                             int stage_k) {
  extern __shared__ int4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int i0 = start ? start[w] : w, i1 = start ? start[w + 1] : w + 1;
  for (int i = i0; i < i1; ++i) {
    if (i > i0) __syncthreads();  // the previous item's staged members are read
    const BatchItems it{meshes, items, stage_k};
    switch (meshes[__builtin_amdgcn_readfirstlane(items[i].x)].pq) {
      case 32: reconstruct_loop<3, 2, false, false>(it, i, i + 1, 1, lds); break;
      case 33: reconstruct_loop<3, 3, false, false>(it, i, i + 1, 1, lds); break;
      case 42: reconstruct_loop<4, 2, false, false>(it, i, i + 1, 1, lds); break;
      case 43: reconstruct_loop<4, 3, false, false>(it, i, i + 1, 1, lds); break;
      case 52: reconstruct_loop<5, 2, false, false>(it, i, i + 1, 1, lds); break;
      case 53: reconstruct_loop<5, 3, false, false>(it, i, i + 1, 1, lds); break;
      case 62: reconstruct_loop<6, 2, false, false>(it, i, i + 1, 1, lds); break;
      case 63: reconstruct_loop<6, 3, false, false>(it, i, i + 1, 1, lds); break;
      default: break;
    }
  }
}

// Cells solved with operators, over (mesh, set of them) items of every order.
__global__ __launch_bounds__(64) void k_batch_reconstruct_kept(
    const BatchMeshDev* __restrict__ meshes, const int2* __restrict__ items, int stage_k) {
  const int2 it = items[blockIdx.x];
  const int m = __builtin_amdgcn_readfirstlane(it.x);
  TENO_CONST ReconArgs& a = *(TENO_CONST ReconArgs*)(uintptr_t)&meshes[m].r[stage_k];
  const KeptArgs k = meshes[m].kept;
  switch (meshes[m].pq) {
    case 32: reconstruct_kept<3, 2, false, false>(a, k, it.y, nullptr); break;
    case 33: reconstruct_kept<3, 3, false, false>(a, k, it.y, nullptr); break;
    case 42: reconstruct_kept<4, 2, false, false>(a, k, it.y, nullptr); break;
    case 43: reconstruct_kept<4, 3, false, false>(a, k, it.y, nullptr); break;
    case 52: reconstruct_kept<5, 2, false, false>(a, k, it.y, nullptr); break;
    case 53: reconstruct_kept<5, 3, false, false>(a, k, it.y, nullptr); break;
    case 62: reconstruct_kept<6, 2, false, false>(a, k, it.y, nullptr); break;
    case 63: reconstruct_kept<6, 3, false, false>(a, k, it.y, nullptr); break;
    default: break;
  }
}

// Persistent face fluxes over (mesh, 64-face chunk) items.
__global__ __launch_bounds__(256) void k_batch_face_flux(const BatchMeshDev* __restrict__ meshes,
                                                         const int2* __restrict__ items,
                                                         const int* __restrict__ wave_start,
                                                         int n_waves) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int w = xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
  if (w >= n_waves) return;
  const int i0 = wave_start[w], i1 = wave_start[w + 1];
  for (int i = i0; i < i1; ++i) {
    const int2 it = items[i];
    const int m = __builtin_amdgcn_readfirstlane(it.x);
    const BatchMeshDev& d = meshes[m];
    const int f = it.y * 64 + lane;
    if (f >= d.ff.n_face) continue;
    if (d.pq % 10 == 2) face_flux<2>(d.ff, f);
    else face_flux<3>(d.ff, f);
  }
}

// Boundary faces over (mesh, 64-face chunk) items, one item per wavefront,
// after k_batch_face_flux: every face, then the boundary faces rewritten
// with their conditions, as for one mesh.
__global__ __launch_bounds__(256) void k_batch_boundary_flux(const BatchMeshDev* __restrict__ meshes,
                                                             const int2* __restrict__ items,
                                                             int n_items) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= n_items) return;
  const int2 it = items[w];
  const int m = __builtin_amdgcn_readfirstlane(it.x);
  const BatchMeshDev& d = meshes[m];
  const int b = it.y * 64 + lane;
  if (b >= d.n_bface) return;
  if (d.pq % 10 == 2) face_flux<2, true>(d.ff, d.bface[b], b);
  else face_flux<3, true>(d.ff, d.bface[b], b);
}

// Persistent gather + stage update over (mesh, 64-cell chunk) items.
__global__ __launch_bounds__(256) void k_batch_cell_update(const BatchMeshDev* __restrict__ meshes,
                                                           const int2* __restrict__ items,
                                                           const int* __restrict__ wave_start,
                                                           int n_waves, int stage_k) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int w = xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
  if (w >= n_waves) return;
  const int i0 = wave_start[w], i1 = wave_start[w + 1];
  for (int i = i0; i < i1; ++i) {
    const int2 it = items[i];
    const int m = __builtin_amdgcn_readfirstlane(it.x);
    const BatchMeshDev& d = meshes[m];
    const int t = it.y * 64 + lane;
    if (t >= d.n_cell) continue;
    cell_update<true>(d.cu[stage_k], t);
  }
}

// Per-mesh dt: one block per (mesh, 256-cell block) item, then one block per mesh.
__global__ __launch_bounds__(256) void k_batch_dt_partial(const BatchMeshDev* __restrict__ meshes,
                                                          const int2* __restrict__ items,
                                                          double* __restrict__ partial) {
  __shared__ double sh[4];
  const int2 it = items[blockIdx.x];
  const BatchMeshDev& d = meshes[it.x];
  const int t = it.y * 256 + threadIdx.x;
  const double lim = t < d.n_cell ? cell_dt_limit(d.U, d.geo, t, d.gamma) : INFINITY;
  const double m = block_min(lim, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

__global__ __launch_bounds__(256) void k_batch_dt_final(const BatchMeshDev* __restrict__ meshes,
                                                        const int* __restrict__ item_start,
                                                        const double* __restrict__ partial,
                                                        double cfl) {
  __shared__ double sh[4];
  double x = INFINITY;
  for (int i = item_start[blockIdx.x] + threadIdx.x; i < item_start[blockIdx.x + 1]; i += 256)
    x = fmin(x, partial[i]);
  const double m = block_min(x, sh);
  if (threadIdx.x == 0) *meshes[blockIdx.x].dt = cfl * m;
}

__global__ void k_diag_reset(DevDiag* d) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    d->nonphysical = 0;
    d->near_ties = 0;
    d->fallbacks = 0;
    d->first_bad = LLONG_MAX;
  }
}

}  // namespace teno
