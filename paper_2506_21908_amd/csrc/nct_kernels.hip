// HIP kernels of the non-collinear TDDFT step for gfx950 (MI355X), wave64.
//
// H application (Eq. HNC-SDFT / TDSDFT) as two passes over HBM, in one of two forms:
//   real space (the kinetic operator is a sum T_x + T_yz): k_xv, per column block and both spinor
//     components, forms T_x w and the 2x2 local potential V w = [v + b.sigma] w on the Taylor base;
//     k_plane_yz, per (spinor component, x-plane), adds T_yz w and the projector scatter rows, and
//     gathers the sphere rows of the result for the next projection.  Everything in FP64; in FP32
//     single applications and the steps and adjoint steps of large systems;
//   with (y,z)-transformed copies, FP32 only (the other steps, ground states): k_xpass (DFT_x ->
//     multiply 1/2|G|^2/N -> IDFT_x on the transformed states) and k_plane_stage2 / k_plane_stage_r
//     (IDFT_yz -> T w; V w; + scatter rows; Taylor update; sphere rows; DFT_yz of the result for the
//     next column pass).
// Densities, exchange, Hartree and reductions are FP64.  The projector
// contraction <beta|psi> and its scatter-back run on the matrix cores
// (v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "nct_fft.hpp"
#include "nct_internal.hpp"
#include "nct_tables.hpp"

// This file is compiled once per precision (in parallel): NCT_FP64_TU 1 holds the FP64 instantiations
// and everything that has no precision of its own, 0 the FP32 ones.
#ifndef NCT_FP64_TU
#error "compile with -DNCT_FP64_TU=1 and -DNCT_FP64_TU=0"
#endif

namespace nct {

// threads per plane workgroup: smallest power of two >= 64 with at most 9 points per thread
__host__ __device__ constexpr int plane_nt(int np) {
  int nt = 64;
  while (nt < 1024 && (np + nt - 1) / nt > 9) nt *= 2;
  return nt;
}
template <int NY, int NZ>
constexpr size_t plane_lds_bytes(size_t elem) {
  return (size_t(NY) * (NZ + 1) + NY + NZ) * elem;
}

// ---------------------------------------------------------------- block reductions
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red) {
  // wave64 butterfly then a fixed-order sum over waves: deterministic
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    for (int k = 0; k < NT / 64; ++k) s += red[k];
  }
  return s;  // valid on thread 0
}
// W sums at once, the same order: one barrier instead of two for each (k_fields with its twelve: 5.7
// against 6.3 us at 16^3).  Sum w goes to out[w].
template <int NT, int W>
__device__ __forceinline__ void block_sums(const double (&v)[W], double (&red)[NT / 64][W], double* out) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    double s = v[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (l == 0) red[w][k] = s;
  }
  __syncthreads();
  if (int(threadIdx.x) < W) {
    double s = 0.0;
    for (int k = 0; k < NT / 64; ++k) s += red[k][threadIdx.x];
    out[threadIdx.x] = s;
  }
}

// ---------------------------------------------------------------- streamed global access
// Cache policy of the large streamed operands (the state-sized buffers), chosen per system from
// the size of one state set: M = 0 plain loads and stores; M = 1 non-temporal (streaming)
// stores; M = 2 non-temporal loads as well.  Streaming keeps buffers that will not be re-read
// from the caches before eviction from displacing the shared fields and twiddles; for state
// sets small enough to stay cache-resident between passes plain accesses are faster.
template <int M, typename R>
__device__ __forceinline__ cpx<R> ld_stream(const cpx<R>* p) {
  if constexpr (M >= 2) {
    typedef R v2 __attribute__((ext_vector_type(2)));
    const v2 t = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
    return cpx<R>{t.x, t.y};
  } else {
    return *p;
  }
}
template <int M, typename R>
__device__ __forceinline__ void st_stream(cpx<R>* p, cpx<R> v) {
  if constexpr (M >= 1) {
    typedef R v2 __attribute__((ext_vector_type(2)));
    v2 t;
    t.x = v.x;
    t.y = v.y;
    __builtin_nontemporal_store(t, reinterpret_cast<v2*>(p));
  } else {
    *p = v;
  }
}

// Bloch phase exp(i q.d) of one sphere row (q: Bloch vector, d: the row's displacement from its
// atom).  Rows taken into the projections carry it, scattered rows its conjugate.
// (q passed as scalars: an addressable local array would live in scratch memory)
__device__ __forceinline__ cpx<double> bloch_phase(double q0, double q1, double q2, const double* d) {
  double sn, cs;
  sincos(q0 * d[0] + q1 * d[1] + q2 * d[2], &sn, &cs);
  return {cs, sn};
}
__device__ __forceinline__ cpx<float> bloch_phase(float q0, float q1, float q2, const float* d) {
  float sn, cs;
  sincosf(q0 * d[0] + q1 * d[1] + q2 * d[2], &sn, &cs);
  return {cs, sn};
}

// ---------------------------------------------------------------- plane pass, two halves
// FP32 stage in transformed form: inverse (y,z) transform of the column-pass output, 2x2 local
// potential on w, projector rows, Horner update out = alpha x + c H w, sphere rows of out, forward
// (y,z) transform of out.  The two spinor components of the (state, x-plane) are held as two LDS planes
// and transformed concurrently by the two halves of the workgroup; the pointwise 2x2 update then reads
// both planes.  Threads per spinor half: plane_nt's choice capped at NCT_PLANE2_NTH_MAX (tuning macro).
#ifndef NCT_PLANE2_NTH_MAX_F32
#define NCT_PLANE2_NTH_MAX_F32 512
#endif
template <typename R>
__host__ __device__ constexpr int plane2_nth(int np) {
  return plane_nt(np) > NCT_PLANE2_NTH_MAX_F32 ? NCT_PLANE2_NTH_MAX_F32 : plane_nt(np);
}
// Minimum waves per SIMD the register allocation of the two-half kernel must allow, where LDS
// admits more workgroups per CU than the registers would: 64^2, whose two 66 KB workgroups of 16
// waves need 8 waves per SIMD: at 68 VGPRs only one fitted, at 63 both do (measured 1159 -> 949 us
// per launch at 64^3 x 256).
template <typename R>
__host__ __device__ constexpr int plane2_min_waves(int np) {
  return np == 64 * 64 ? 8 : 1;
}
template <int NY, int NZ>
constexpr size_t plane2_lds_bytes(size_t elem) {
  return (size_t(2) * NY * (NZ + 1) + NY + NZ) * elem;
}

template <typename R, int NY, int NZ, int M>
__global__ __launch_bounds__(2 * plane2_nth<R>(NY* NZ), plane2_min_waves<R>(NY* NZ)) void k_plane_stage2(StageArgs<R> a, ProjTables pt,
                                                                          const cpx<R>* __restrict__ twy_g,
                                                                          const cpx<R>* __restrict__ twz_g,
                                                                          int S, int NX) {
  constexpr int NP = NY * NZ;
  constexpr int NTH = plane2_nth<R>(NP);
  constexpr int NT = 2 * NTH;
  constexpr int PZ = NZ + 1;
  constexpr int PL = NY * PZ;
  constexpr int PPH = (NP + NTH - 1) / NTH;
  constexpr int PPT = (NP + NT - 1) / NT;
#ifndef NCT_PLANE2_G_F32
#define NCT_PLANE2_G_F32 3
#endif
  constexpr int G = NCT_PLANE2_G_F32;  // pointwise points per load batch
  extern __shared__ double4 smem_d4[];
  cpx<R>* planes = reinterpret_cast<cpx<R>*>(smem_d4);
  cpx<R>* twy = planes + 2 * PL;
  cpx<R>* twz = twy + NY;
  const int tid = threadIdx.x;
  const int h = tid / NTH;
  const int th = tid - h * NTH;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / S;
  const int i = L - x * S;
  for (int k = tid; k < NY; k += NT) twy[k] = twy_g[k];
  for (int k = tid; k < NZ; k += NT) twz[k] = twz_g[k];
  const size_t N = size_t(NX) * NP;
  const size_t off0 = (size_t(2 * i) * NX + x) * NP;
  const size_t off1 = (size_t(2 * i + 1) * NX + x) * NP;
  const size_t offh = h ? off1 : off0;
  cpx<R>* pl = planes + h * PL;

  // 1) kinetic part: each half loads and inverse-transforms its spinor's plane (the first
  //    transform stage works on the loaded values)
  {
    const cpx<R>* __restrict__ tin = reinterpret_cast<const cpx<R>*>(a.tmp_in) + offh;
    plane_fft_inv_from<R, NY, NZ, PZ, NTH>(pl, twy, twz, th, [&](int g) { return ld_stream<M>(&tin[g]); });
  }

  // 2) 2x2 local potential and Taylor update over the whole plane (both spinors per point)
  {
    const cpx<R>* __restrict__ win = reinterpret_cast<const cpx<R>*>(a.w_in);
    const cpx<R>* __restrict__ xb = reinterpret_cast<const cpx<R>*>(a.x_base);
    const bool xsep = xb && (a.x_base != a.w_in);
    const R* __restrict__ F = a.fields;
    const R lx = a.lg[0] * R(x) + a.lg[3];  // laser potential of this plane, less its y, z terms
#pragma unroll
    for (int j0 = 0; j0 < PPT; j0 += G) {
      cpx<R> wu[G], wd[G], xu[G], xd[G];
      R fv[G], fx[G], fy[G], fz[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (j0 + g < PPT) {
          const int e = min(tid + (j0 + g) * NT, NP - 1);  // clamped: loads unconditional
          const size_t p = size_t(x) * NP + e;
          wu[g] = ld_stream<M>(&win[off0 + e]);
          wd[g] = ld_stream<M>(&win[off1 + e]);
          if (xsep) {
            xu[g] = ld_stream<M>(&xb[off0 + e]);
            xd[g] = ld_stream<M>(&xb[off1 + e]);
          } else {
            xu[g] = wu[g];
            xd[g] = wd[g];
          }
          fv[g] = F[p];
          fx[g] = F[N + p];
          fy[g] = F[2 * N + p];
          fz[g] = F[3 * N + p];
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int e = tid + (j0 + g) * NT;
        if (j0 + g < PPT && e < NP) {
          const int q = (e / NZ) * PZ + (e % NZ);
          const cpx<R> tu = planes[q], td = planes[PL + q];
          const R v = fv[g] + (lx + a.lg[1] * R(e / NZ) + a.lg[2] * R(e % NZ));
          const R bx = fx[g] + a.bext[0], by = fy[g] + a.bext[1], bz = fz[g] + a.bext[2];
          cpx<R> hu, hd;
          hu.x = tu.x + (v + bz) * wu[g].x + bx * wd[g].x + by * wd[g].y;
          hu.y = tu.y + (v + bz) * wu[g].y + bx * wd[g].y - by * wd[g].x;
          hd.x = td.x + bx * wu[g].x - by * wu[g].y + (v - bz) * wd[g].x;
          hd.y = td.y + bx * wu[g].y + by * wu[g].x + (v - bz) * wd[g].y;
          cpx<R> ou = {a.cre * hu.x - a.cim * hu.y, a.cre * hu.y + a.cim * hu.x};
          cpx<R> od = {a.cre * hd.x - a.cim * hd.y, a.cre * hd.y + a.cim * hd.x};
          if (xb) {
            ou.x += a.alpha * xu[g].x;
            ou.y += a.alpha * xu[g].y;
            od.x += a.alpha * xd[g].x;
            od.y += a.alpha * xd[g].y;
          }
          planes[q] = ou;
          planes[PL + q] = od;
        }
      }
    }
  }
  __syncthreads();

  // 3) projector rows, outputs, forward transform; each half its own spinor
  const cpx<R>* __restrict__ Y = reinterpret_cast<const cpx<R>*>(a.Y);
  cpx<R>* __restrict__ Wr = reinterpret_cast<cpx<R>*>(a.W);
  cpx<R>* __restrict__ wout = reinterpret_cast<cpx<R>*>(a.w_out);
  cpx<R>* __restrict__ acc = reinterpret_cast<cpx<R>*>(a.acc);
  cpx<R>* __restrict__ tout = reinterpret_cast<cpx<R>*>(a.tmp_out);
  const int r0 = pt.pr_off ? pt.pr_off[x] : 0;
  const int r1 = pt.pr_off ? pt.pr_off[x + 1] : 0;
  const size_t rowbase = size_t(2 * i + h) * pt.Jtot;
  const bool kq = a.kv != nullptr;
  R q0 = 0, q1 = 0, q2 = 0;
  if (kq) {
    const R* k0 = a.kv + 3 * (a.state_off + i);
    q0 = k0[0] + a.ka[0];
    q1 = k0[1] + a.ka[1];
    q2 = k0[2] + a.ka[2];
  }
  const R* disp = reinterpret_cast<const R*>(pt.disp);
  if (Y) {
    for (int r = r0; r < r1; ++r) {
      const int jb = pt.pr_begin[r], je = pt.pr_end[r];
      for (int J = jb + th; J < je; J += NTH) {
        const int e = pt.pidx[J];
        cpx<R> y = Y[rowbase + J];
        if (kq) y = cmulc(y, bloch_phase(q0, q1, q2, disp + 3 * J));
        cpx<R>& d = pl[(e / NZ) * PZ + (e % NZ)];
        d.x += a.cre * y.x - a.cim * y.y;
        d.y += a.cre * y.y + a.cim * y.x;
      }
      __syncthreads();
    }
  }
  if (Wr) {
    for (int r = r0; r < r1; ++r) {
      const int jb = pt.pr_begin[r], je = pt.pr_end[r];
      for (int J = jb + th; J < je; J += NTH) {
        const int e = pt.pidx[J];
        cpx<R> o = pl[(e / NZ) * PZ + (e % NZ)];
        if (kq) o = cmul(o, bloch_phase(q0, q1, q2, disp + 3 * J));
        Wr[rowbase + J] = o;
      }
    }
  }
  if (acc) {
    cpx<R> v[PPH];
#pragma unroll
    for (int j = 0; j < PPH; ++j) v[j] = acc[offh + min(th + j * NTH, NP - 1)];
#pragma unroll
    for (int j = 0; j < PPH; ++j) {
      const int e = th + j * NTH;
      if (e < NP) acc[offh + e] = v[j] + pl[(e / NZ) * PZ + (e % NZ)];
    }
  }
  if (wout) {
#pragma unroll
    for (int j = 0; j < PPH; ++j) {
      const int e = th + j * NTH;
      if (e < NP) st_stream<M>(&wout[offh + e], pl[(e / NZ) * PZ + (e % NZ)]);
    }
  }
  if (tout) {
    __syncthreads();
    cpx<R>* __restrict__ to = tout + offh;
    plane_fft_fwd_to<R, NY, NZ, PZ, NTH>(pl, twy, twz, th, [](int) { return 0; },
                                         [&](int g, int, cpx<R> v, int) { st_stream<M>(&to[g], v); });
  }
}

// ---------------------------------------------------------------- plane pass, one plane in LDS
// Same stage as k_plane_stage2 for planes where two LDS planes would admit only one workgroup per
// CU but one plane admits two (96^2: 76 KB).  The spinor components go
// through the single LDS plane one after the other: the up component's kinetic part waits in
// registers (PPT values per thread, the last of them in a private LDS slot per thread) while the
// down component is transformed; after the 2x2 update the up result waits there again while the
// down result is finished and transformed forward.
// Two resident workgroups per CU interleave their memory and transform phases.
// Threads per workgroup (tuning macro) and the point batch of the 2x2 update.
#ifndef NCT_PLANER_NT
#define NCT_PLANER_NT 512
#endif
// NCT_PLANER_OFF (tuning macro) keeps those planes on the two-plane kernel.
template <typename R, int NY, int NZ>
constexpr bool planer_use() {
#ifdef NCT_PLANER_OFF
  return false;
#else
  return plane2_lds_bytes<NY, NZ>(sizeof(cpx<R>)) > 80 * 1024 &&
         plane_lds_bytes<NY, NZ>(sizeof(cpx<R>)) <= 80 * 1024 - 512;
#endif
}

// Values per thread of the held spinor component that live in LDS left over by the plane
// (tuning macro NCT_PLANER_KL: at most that many, within the 80 KB of two workgroups per CU).
#ifndef NCT_PLANER_KL
#define NCT_PLANER_KL 1
#endif
template <typename R, int NY, int NZ>
constexpr int planer_kl() {
  constexpr size_t spare = 80 * 1024 - 512 - plane_lds_bytes<NY, NZ>(sizeof(cpx<R>));
  constexpr int fit = int(spare / (size_t(NCT_PLANER_NT) * sizeof(cpx<R>)));
  constexpr int ppt = (NY * NZ + NCT_PLANER_NT - 1) / NCT_PLANER_NT;
  constexpr int kl = NCT_PLANER_KL < fit ? NCT_PLANER_KL : fit;
  return kl < ppt ? kl : ppt;
}
template <typename R, int NY, int NZ>
constexpr size_t planer_lds_bytes() {
  return plane_lds_bytes<NY, NZ>(sizeof(cpx<R>)) + size_t(planer_kl<R, NY, NZ>()) * NCT_PLANER_NT * sizeof(cpx<R>);
}

template <typename R, int NY, int NZ, int M>
__global__ __launch_bounds__(NCT_PLANER_NT, 4) void k_plane_stage_r(StageArgs<R> a, ProjTables pt,
                                                                     const cpx<R>* __restrict__ twy_g,
                                                                     const cpx<R>* __restrict__ twz_g,
                                                                     int S, int NX) {
  constexpr int NP = NY * NZ;
  constexpr int NT = NCT_PLANER_NT;
  constexpr int PZ = NZ + 1;
  constexpr int PPT = (NP + NT - 1) / NT;
  constexpr int KR = PPT - planer_kl<R, NY, NZ>();  // held values in registers, the rest in LDS
  constexpr int G = 3;  // points per load batch of the 2x2 update
  extern __shared__ double4 smem_d4[];
  cpx<R>* pl = reinterpret_cast<cpx<R>*>(smem_d4);
  cpx<R>* twy = pl + NY * PZ;
  cpx<R>* twz = twy + NY;
  cpx<R>* kus = twz + NZ;  // [PPT - KR][NT]: each thread's own held values beyond KR
  const int tid = threadIdx.x;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / S;
  const int i = L - x * S;
  for (int k = tid; k < NY; k += NT) twy[k] = twy_g[k];
  for (int k = tid; k < NZ; k += NT) twz[k] = twz_g[k];
  const size_t N = size_t(NX) * NP;
  const size_t off0 = (size_t(2 * i) * NX + x) * NP;
  const size_t off1 = (size_t(2 * i + 1) * NX + x) * NP;
  const cpx<R>* __restrict__ tin = reinterpret_cast<const cpx<R>*>(a.tmp_in);

  // 1) kinetic part of the up component (inverse 2D transform), kept in registers (the first KR
  //    values of each thread) and in the thread's own LDS slots (the rest)
  plane_fft_inv_from<R, NY, NZ, PZ, NT>(pl, twy, twz, tid, [&](int g) { return ld_stream<M>(&tin[off0 + g]); });
  cpx<R> ku[KR > 0 ? KR : 1];
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    const int e = min(tid + j * NT, NP - 1);
    const cpx<R> v = pl[(e / NZ) * PZ + (e % NZ)];
    if (j < KR) ku[j < KR ? j : 0] = v;
    else kus[(j - KR) * NT + tid] = v;
  }
  __syncthreads();
  // 2) kinetic part of the down component, left in LDS
  plane_fft_inv_from<R, NY, NZ, PZ, NT>(pl, twy, twz, tid, [&](int g) { return ld_stream<M>(&tin[off1 + g]); });

  // 3) 2x2 local potential and Taylor update: up result back into ku, down result into LDS
  {
    const cpx<R>* __restrict__ win = reinterpret_cast<const cpx<R>*>(a.w_in);
    const cpx<R>* __restrict__ xb = reinterpret_cast<const cpx<R>*>(a.x_base);
    const bool xsep = xb && (a.x_base != a.w_in);
    const R* __restrict__ F = a.fields;
    const R lx = a.lg[0] * R(x) + a.lg[3];  // laser potential of this plane, less its y, z terms
#pragma unroll
    for (int j0 = 0; j0 < PPT; j0 += G) {
      cpx<R> wu[G], wd[G], xu[G], xd[G];
      R fv[G], fx[G], fy[G], fz[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (j0 + g < PPT) {
          const int e = min(tid + (j0 + g) * NT, NP - 1);  // clamped: loads unconditional
          const size_t p = size_t(x) * NP + e;
          wu[g] = ld_stream<M>(&win[off0 + e]);
          wd[g] = ld_stream<M>(&win[off1 + e]);
          if (xsep) {
            xu[g] = ld_stream<M>(&xb[off0 + e]);
            xd[g] = ld_stream<M>(&xb[off1 + e]);
          } else {
            xu[g] = wu[g];
            xd[g] = wd[g];
          }
          fv[g] = F[p];
          fx[g] = F[N + p];
          fy[g] = F[2 * N + p];
          fz[g] = F[3 * N + p];
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int j = j0 + g;
        const int e = tid + j * NT;
        if (j < PPT && e < NP) {
          const int q = (e / NZ) * PZ + (e % NZ);
          const cpx<R> tu = j < KR ? ku[j < KR ? j : 0] : kus[(j - KR) * NT + tid], td = pl[q];
          const R v = fv[g] + (lx + a.lg[1] * R(e / NZ) + a.lg[2] * R(e % NZ));
          const R bx = fx[g] + a.bext[0], by = fy[g] + a.bext[1], bz = fz[g] + a.bext[2];
          cpx<R> hu, hd;
          hu.x = tu.x + (v + bz) * wu[g].x + bx * wd[g].x + by * wd[g].y;
          hu.y = tu.y + (v + bz) * wu[g].y + bx * wd[g].y - by * wd[g].x;
          hd.x = td.x + bx * wu[g].x - by * wu[g].y + (v - bz) * wd[g].x;
          hd.y = td.y + bx * wu[g].y + by * wu[g].x + (v - bz) * wd[g].y;
          cpx<R> ou = {a.cre * hu.x - a.cim * hu.y, a.cre * hu.y + a.cim * hu.x};
          cpx<R> od = {a.cre * hd.x - a.cim * hd.y, a.cre * hd.y + a.cim * hd.x};
          if (xb) {
            ou.x += a.alpha * xu[g].x;
            ou.y += a.alpha * xu[g].y;
            od.x += a.alpha * xd[g].x;
            od.y += a.alpha * xd[g].y;
          }
          if (j < KR) ku[j < KR ? j : 0] = ou;
          else kus[(j - KR) * NT + tid] = ou;
          pl[q] = od;
        }
      }
    }
  }
  __syncthreads();

  // 4) per component (down, then up): projector rows, outputs, forward transform
  const cpx<R>* __restrict__ Y = reinterpret_cast<const cpx<R>*>(a.Y);
  cpx<R>* __restrict__ Wr = reinterpret_cast<cpx<R>*>(a.W);
  cpx<R>* __restrict__ wout = reinterpret_cast<cpx<R>*>(a.w_out);
  cpx<R>* __restrict__ acc = reinterpret_cast<cpx<R>*>(a.acc);
  cpx<R>* __restrict__ tout = reinterpret_cast<cpx<R>*>(a.tmp_out);
  const int r0 = pt.pr_off ? pt.pr_off[x] : 0;
  const int r1 = pt.pr_off ? pt.pr_off[x + 1] : 0;
  const bool kq = a.kv != nullptr;
  R q0 = 0, q1 = 0, q2 = 0;
  if (kq) {
    const R* k0 = a.kv + 3 * (a.state_off + i);
    q0 = k0[0] + a.ka[0];
    q1 = k0[1] + a.ka[1];
    q2 = k0[2] + a.ka[2];
  }
  const R* disp = reinterpret_cast<const R*>(pt.disp);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int h = 1 - pass;  // spinor component finished in this pass
    const size_t offh = h ? off1 : off0;
    if (pass == 1) {
      // the down component's forward transform has read LDS for the last time: reuse it for up
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        const int e = tid + j * NT;
        if (e < NP) pl[(e / NZ) * PZ + (e % NZ)] = j < KR ? ku[j < KR ? j : 0] : kus[(j - KR) * NT + tid];
      }
      __syncthreads();
    }
    const size_t rowbase = size_t(2 * i + h) * pt.Jtot;
    if (Y) {
      for (int r = r0; r < r1; ++r) {
        const int jb = pt.pr_begin[r], je = pt.pr_end[r];
        for (int J = jb + tid; J < je; J += NT) {
          const int e = pt.pidx[J];
          cpx<R> y = Y[rowbase + J];
          if (kq) y = cmulc(y, bloch_phase(q0, q1, q2, disp + 3 * J));
          cpx<R>& d = pl[(e / NZ) * PZ + (e % NZ)];
          d.x += a.cre * y.x - a.cim * y.y;
          d.y += a.cre * y.y + a.cim * y.x;
        }
        __syncthreads();
      }
    }
    if (Wr) {
      for (int r = r0; r < r1; ++r) {
        const int jb = pt.pr_begin[r], je = pt.pr_end[r];
        for (int J = jb + tid; J < je; J += NT) {
          const int e = pt.pidx[J];
          cpx<R> o = pl[(e / NZ) * PZ + (e % NZ)];
          if (kq) o = cmul(o, bloch_phase(q0, q1, q2, disp + 3 * J));
          Wr[rowbase + J] = o;
        }
      }
    }
    if (acc) {
      cpx<R> v[PPT];
#pragma unroll
      for (int j = 0; j < PPT; ++j) v[j] = acc[offh + min(tid + j * NT, NP - 1)];
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        const int e = tid + j * NT;
        if (e < NP) acc[offh + e] = v[j] + pl[(e / NZ) * PZ + (e % NZ)];
      }
    }
    if (wout) {
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        const int e = tid + j * NT;
        if (e < NP) st_stream<M>(&wout[offh + e], pl[(e / NZ) * PZ + (e % NZ)]);
      }
    }
    if (tout) {
      __syncthreads();
      cpx<R>* __restrict__ to = tout + offh;
      plane_fft_fwd_to<R, NY, NZ, PZ, NT>(pl, twy, twz, tid, [](int) { return 0; },
                                          [&](int g, int, cpx<R> v, int) { st_stream<M>(&to[g], v); });
    }
  }
}

// ---------------------------------------------------------------- real-space H stage
// The kinetic operator is a sum of one operator per axis, T = T_x + T_yz, so H is applied in real
// space on both sides, nothing kept in transformed form: the column pass (k_xv) writes
// r = alpha x + c (T_x + V) w, with V the 2x2 local potential, and the plane pass (k_plane_yz) adds
// c (T_yz w + projector rows) to it.  The two passes of a stage read w twice and r once and write r and
// out: 5 |psi| (6 where the Taylor base x is not w), against 7 |psi| with (y,z)-transformed copies of
// w.  V sits in the column pass because that pass holds both spinor components of a point at once in
// little LDS; in the plane pass it cost a second read of w (a plane of either component and the
// transforms leave no room to keep w), which misses L2 and counts on the fabric like HBM: 6.2 instead
// of 4.3 GB fetched per launch at 64^3 x 256, 1478 us.
//
// Element at a byte offset from a wave-uniform base: the base stays in scalar registers (the empty
// asm keeps the compiler from folding the offset into a 64-bit vector address per operand) and one
// 32-bit vector register addresses every operand of the same shape.  The pointer is named as global
// memory: an asm that hides where it points leaves flat loads with 64-bit address sums, which also
// count as LDS operations in every wait (64^3 x 128: column pass 377 against 414 us; 48^3 x 64: 92
// against 106).
template <typename T>
__device__ __forceinline__ T* at_bytes(T* base, uint32_t bytes) {
  typedef __attribute__((address_space(1))) char* gptr;  // in global memory, which the asm would hide
  gptr p = (gptr)base;
  asm volatile("" : "+s"(p));
  return (T*)(p + bytes);
}

// Value that is computed here, not where it is used next: the fences order memory operations only, and
// the operands of sums put off to their use spilled (96 points: 35 registers FP64, 39 FP32).
template <typename R>
__device__ __forceinline__ void pin(cpx<R>& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// Waves per workgroup of the plane pass and the waves per SIMD its registers must allow.
// FP64 64^2: eight waves in each of the two workgroups that the LDS holds (1055 us per pass at 64^3 x
// 256, 6.1 TB/s); more waves per SIMD than the four of 128 registers spill (48^2 with five 172 against
// 143 us at 48^3 x 64 with 4 atoms).  FP32 has half the registers per point: each wave takes twice the
// lines (64^2 four waves 553 us at 64^3 x 256, eight 650 to 746).  96^2: 74 KB (FP32) or 147 KB (FP64) of
// LDS allow 12 waves per CU, three per SIMD (FP32 with 24 waves of 80 registers 1413 to 1650 against
// 1282 us at 96^3 x 128).
template <typename R>
__host__ __device__ constexpr int real_nw(int ny, int nz) {
  if (ny == 64 && nz == 64) return sizeof(R) == 8 ? 8 : 4;
  if (ny == 48 && nz == 48) return sizeof(R) == 8 ? 6 : 3;
  if (ny == 96 && nz == 96) return sizeof(R) == 8 ? 12 : 6;
  if (ny == 32 && nz == 32) return 2;
  if (ny == 24 && nz == 24) return 3;
  if (ny * nz == 384) return 2;  // 16 x 24, 24 x 16
  return 1;
}
__host__ __device__ constexpr int real_mw(int ny, int nz) { return ny == 96 && nz == 96 ? 3 : 4; }
// r is loaded before the last stages, not along with w: at 96^2, whose twelve values per thread and
// operand leave few registers for the radix-12 stages (609 -> 566 us FP64 96^3 x 32, 1356 -> 1282 us FP32
// 96^3 x 128; no gain where the registers are there: 48^2 143 against 146 us, 64^2 583 against 588).
__host__ __device__ constexpr bool real_late(int ny, int nz) { return ny == 96 && nz == 96; }
// A stage whose base is w itself (product stages): the plane pass adds alpha w to r while it holds both, and w is
// rounded twice per stage, not three times with two of them in the column pass (one FP64 step at 16^3, K = 4,
// |z| E_max = 2.1, smooth states, against long double 1.78e-16 and 2.06e-16; the transformed form 2.01e-16).  The
// transforms then wait for r as well: 64^3 x 256 FP64 25.27 against 25.48 ms per step, 32^3 x 32 0.713 / 0.712,
// 24^3 x 64 0.769 / 0.764, 48^3 x 310 FP32 7.64 / 7.63.  Not at 96^2 (r is late) and not at 48^2 in FP64, whose six
// waves have less to run meanwhile (48^3 x 64 3.28 against 3.20 ms) and whose error is below the transformed form's
// either way (6.4e-16 against 6.5e-16 after two steps).
template <typename R>
__host__ __device__ constexpr bool plane_takes_base(int ny, int nz) {
  return !real_late(ny, nz) && !(sizeof(R) == 8 && ny == 48 && nz == 48);
}
template <typename R, int NY, int NZ>
constexpr size_t real_lds_bytes() {
  return (size_t(NY) * (NZ + 1) + NY + NZ) * sizeof(cpx<R>) + (NY + NZ) * sizeof(R);
}

// Plane pass: out = r + c (T_yz w + projector rows), with walpha w in r where the stage's base is w
// (plane_takes_base), one workgroup per (spinor component, x-plane), one LDS plane.  All loads (the
// thread's points of w and of r) are issued up front (but see real_late); r waits in registers while w
// goes through the plane.  out may be w.
//
// Each wave owns NZ / NW columns of the y transforms and NY / NW rows of the z transforms, so the
// stages of one axis run without a workgroup barrier (LDS operations of a wave stay in order); only
// the two changes of axis take one.  The last forward z stage, the kinetic factor and the first inverse
// z stage work on the same values and stay in registers.  Where the work items of a wave are no
// multiple of 64, the surplus lanes repeat the last item: they write the same values to the same places.
//
// The projector rows of a plane come in at the end: the map of its points is read before the last change
// of axis and the rows before the last stages, so neither wait stands before the transforms (64^3 x 128
// with 16 atoms 583 against 600 us per pass, without atoms 530; 48^3 x 64 with 4 atoms 143 against 162,
// without 131), and one read of the map serves the rows taken from out too.
//
// ACC: acc += out (the adjoint).
template <typename R, int NY, int NZ, int M, bool ACC>
__global__ __launch_bounds__(64 * real_nw<R>(NY, NZ), real_mw(NY, NZ)) void k_plane_yz(
    StageArgs<R> a, KinTables kt, ProjTables pt, const cpx<R>* __restrict__ twy_g,
    const cpx<R>* __restrict__ twz_g, int B, int NX) {
  using C = cpx<R>;
  constexpr int NP = NY * NZ, PZ = NZ + 1;
  constexpr int NW = real_nw<R>(NY, NZ), NT = 64 * NW;
  constexpr int CW = NZ / NW, RW = NY / NW;
  constexpr int FY = plane_plan(NY), FZ = plane_plan(NZ);
  constexpr int RY = plan_radix(FY, 0), MY = NY / RY;
  constexpr int ITEMS = CW * MY, IT = (ITEMS + 63) / 64;
  static_assert(NZ % NW == 0 && NY % NW == 0 && plan_nstages(FY) <= 2 && plan_nstages(FZ) <= 2, "plane split");
  extern __shared__ double4 smem_d4[];
  C* pl = reinterpret_cast<C*>(smem_d4);
  C* twy = pl + NY * PZ;
  C* twz = twy + NY;
  R* ty = reinterpret_cast<R*>(twz + NZ);
  R* tz = ty + NY;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / B;
  const int b = L - x * B;  // 2 state + component
  const size_t off = (size_t(b) * NX + x) * NP;
  const C* win = reinterpret_cast<const C*>(a.w_in);
  const C* __restrict__ rin = reinterpret_cast<const C*>(a.tmp_in);

  // sphere rows on this plane (pt.pmap): their scatter values go into r before the last stage
  const C* __restrict__ Y = reinterpret_cast<const C*>(a.Y);
  C* __restrict__ Wr = reinterpret_cast<C*>(a.W);
  const bool on_plane = (Y || Wr) && pt.pr_off[x + 1] > pt.pr_off[x];
  const int* __restrict__ pm = pt.pmap + size_t(x) * NP;
  const size_t rb = size_t(b) * pt.Jtot;

  // thread (column z, butterfly c) of the y transform holds the points y = c + q MY
  C v[IT][RY], r[IT][RY];
  const auto load_r = [&]() {
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      const int it = min(lane + 64 * u, ITEMS - 1);
      const uint32_t o = uint32_t((it / CW) * NZ + it % CW) * uint32_t(sizeof(C));
#pragma unroll
      for (int q = 0; q < RY; ++q) r[u][q] = ld_stream<M>(at_bytes(rin + off + (w * CW + q * MY * NZ), o));
    }
  };
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    const uint32_t o = uint32_t((it / CW) * NZ + it % CW) * uint32_t(sizeof(C));
#pragma unroll
    for (int q = 0; q < RY; ++q) v[u][q] = ld_stream<M>(at_bytes(win + off + (w * CW + q * MY * NZ), o));
  }
  if constexpr (!real_late(NY, NZ)) load_r();
  {
    const double ky = kt.shift(b >> 1, 1), kz = kt.shift(b >> 1, 2);
    for (int k = tid; k < NY; k += NT) {
      twy[k] = twy_g[k];
      const double g = kt.g[1][plan_position<FY>(k)] + ky;
      ty[k] = R(0.5 / NP * (g * g));
    }
    for (int k = tid; k < NZ; k += NT) {
      twz[k] = twz_g[k];
      const double g = kt.g[2][plan_position<FZ>(k)] + kz;
      tz[k] = R(0.5 / NP * (g * g));
    }
  }
  if constexpr (plane_takes_base<R>(NY, NZ)) {
    if (a.walpha != R(0)) {  // the base of this stage is w: added here, it is rounded once and once with c T_yz w
#pragma unroll
      for (int u = 0; u < IT; ++u)
#pragma unroll
        for (int q = 0; q < RY; ++q) {
          r[u][q].x += a.walpha * v[u][q].x;
          r[u][q].y += a.walpha * v[u][q].y;
        }
    }
  }
  group_sync<NW>();  // tables
  C* cols = pl + w * CW;       // this wave's columns
  C* rows = pl + w * RW * PZ;  // this wave's rows
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    {
      stage_butterfly<R, FY, 0, true>(v[u], twy, it / CW);
      C* p = cols + (it / CW) * PZ + it % CW;
#pragma unroll
      for (int q = 0; q < RY; ++q) p[q * MY * PZ] = v[u][q];
    }
  }
  if constexpr (plan_nstages(FY) > 1) {
    wave_sync();
    wave_stage<R, FY, 1, CW, 1, PZ, true>(cols, twy, lane);
  }
  group_sync<NW>();
  if constexpr (plan_nstages(FZ) > 1) {
    wave_stage<R, FZ, 0, RW, PZ, 1, true>(rows, twz, lane);
    wave_sync();
  }
  wave_middle<R, FZ, RW, PZ, 1>(rows, lane, [&](int line, int k) { return ty[w * RW + line] + tz[k]; });
  if constexpr (plan_nstages(FZ) > 1) {
    wave_sync();
    wave_stage<R, FZ, 0, RW, PZ, 1, false>(rows, twz, lane);
  }
  if constexpr (real_late(NY, NZ)) load_r();
  // the map of the plane's sphere rows, then the rows themselves, are under way during the last stages
  int J[IT][RY];
  if (on_plane) {
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      const int it = min(lane + 64 * u, ITEMS - 1);
      const uint32_t o = uint32_t((it / CW) * NZ + it % CW) * 4u;
#pragma unroll
      for (int q = 0; q < RY; ++q) J[u][q] = *at_bytes(pm + (w * CW + q * MY * NZ), o);
    }
  }
  group_sync<NW>();
  bool rows_here = false;  // (wave-uniform)
  C y[IT][RY];
  if (on_plane) {
    int any = J[0][0];
#pragma unroll
    for (int u = 0; u < IT; ++u)
#pragma unroll
      for (int q = 0; q < RY; ++q) any &= J[u][q];  // all negative (no row) only if every J is
    rows_here = __any(any >= 0);
    if (Y && rows_here) {
      // every load at once: points without a row read row 0 and drop it
#pragma unroll
      for (int u = 0; u < IT; ++u)
#pragma unroll
        for (int q = 0; q < RY; ++q) y[u][q] = Y[rb + (J[u][q] >= 0 ? (J[u][q] & kRowMask) : 0)];
    }
  }
  if constexpr (plan_nstages(FY) > 1) {
    wave_stage<R, FY, 1, CW, 1, PZ, false>(cols, twy, lane);
    wave_sync();
  }
  if (Y && rows_here) {
    int more = -1;
#pragma unroll
    for (int u = 0; u < IT; ++u)
#pragma unroll
      for (int q = 0; q < RY; ++q) {
        const C z = J[u][q] >= 0 ? y[u][q] : C{R(0), R(0)};
        r[u][q].x += a.cre * z.x - a.cim * z.y;
        r[u][q].y += a.cre * z.y + a.cim * z.x;
        more = max(more, J[u][q]);
      }
    if (__any(more > kRowMask)) {  // further rows at a point: overlapping spheres
#pragma unroll
      for (int u = 0; u < IT; ++u)
#pragma unroll
        for (int q = 0; q < RY; ++q)
          if (J[u][q] > kRowMask)
            for (int k = pt.rnext[J[u][q] & kRowMask]; k >= 0; k = pt.rnext[k]) {
              const C z = Y[rb + k];
              r[u][q].x += a.cre * z.x - a.cim * z.y;
              r[u][q].y += a.cre * z.y + a.cim * z.x;
            }
    }
  }

  // out = r + c T_yz w, and its sphere rows
  C* wout = reinterpret_cast<C*>(a.w_out);
  C* acc = reinterpret_cast<C*>(a.acc);
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    const uint32_t oc = uint32_t((it / CW) * NZ + it % CW) * uint32_t(sizeof(C));
    const C* p = cols + (it / CW) * PZ + it % CW;
#pragma unroll
    for (int q = 0; q < RY; ++q) v[u][q] = p[q * MY * PZ];
    stage_butterfly<R, FY, 0, false>(v[u], twy, it / CW);
#pragma unroll
    for (int q = 0; q < RY; ++q) {
      const C h = v[u][q];
      r[u][q].x += a.cre * h.x - a.cim * h.y;
      r[u][q].y += a.cre * h.y + a.cim * h.x;
      const int eu = w * CW + q * MY * NZ;
      st_stream<M>(at_bytes(wout + off + eu, oc), r[u][q]);
      if constexpr (ACC) {
        C* ap = at_bytes(acc + off + eu, oc);
        *ap = *ap + r[u][q];
      }
    }
    if (Wr && rows_here) {
#pragma unroll
      for (int q = 0; q < RY; ++q)
        if (J[u][q] >= 0) {
          Wr[rb + (J[u][q] & kRowMask)] = r[u][q];
          if (J[u][q] > kRowMask)
            for (int k = pt.rnext[J[u][q] & kRowMask]; k >= 0; k = pt.rnext[k]) Wr[rb + k] = r[u][q];
        }
    }
  }
}

// Sphere rows W[b][J] of B batch entries (state b / 2, spinor component b % 2): the rows the plane
// pass gathers from its own output, for states that no plane pass has just written.
template <typename R>
__global__ __launch_bounds__(256) void k_gather_rows(const cpx<R>* __restrict__ psi, cpx<R>* __restrict__ W,
                                                     ProjTables pt, size_t N) {
  const int b = blockIdx.x;
  for (int J = blockIdx.y * 256 + threadIdx.x; J < pt.Jtot; J += gridDim.y * 256)
    W[size_t(b) * pt.Jtot + J] = psi[size_t(b) * N + pt.rflat[J]];
}

// Column pass: r = alpha x + c (T_x + V) w, T_x = IDFT_x 1/2 (G_x + k_x)^2 / NX DFT_x, in real space along
// y and z.  Each wave takes CW (xv_cols) consecutive yz columns of one spinor component; the neighbouring wave takes the other component of the same columns, and the two swap
// their values of w through their LDS tiles for the 2x2 potential.  r waits in registers while w goes
// through the tile: the first forward stage works on the values as they are loaded, the last forward
// stage, the factor and the first inverse stage stay in registers.  No workgroup barrier is needed
// after the swap, so the waves' phases interleave freely.  Each XCD takes one eighth of the columns for
// every state (where the column blocks divide by eight): its eighth of the fields stays in its L2, and
// consecutive workgroups still read consecutive columns of one state.
// XS: the Taylor base x is another array than w (else alpha w is used).  It is loaded beside the last stage and
// added last: the sum of the small terms rounds at their own size and x is rounded once here, not twice
// (one FP64 step of smooth states at 16^3, |z| E_max = 0.95, against long double 1.14e-16, 1.35e-16 with x added
// first; Horner steps take as long, 64^3 x 128 FP64 13.49 against 13.47 ms, or less at 96 points, where x waits for
// no field, 96^3 x 32 FP64 12.9 against 13.3, 96^3 x 64 FP32 14.7 against 16.1).
// A wave's columns.  At least one 128-byte line per x-plane (FP32 with 64-byte halves 667 against 425 us per pass
// at 64^3 x 256), and on short lines as many as give the first stage a butterfly per lane: lines of 8, 12, 16 and 32
// points have 1 to 4 butterflies, so that 128 bytes of columns left 32 to 56 of a wave's lanes repeating the last one
// (FP64 8 x 96 x 96 x 60 3.50 -> 1.84 ms per step, 32^3 x 200 3.00 -> 2.64, 16^3 x 60 0.258 -> 0.245).  Lines of 24 take
// sixteen in FP64 too, two rounds of small butterflies (24^3 x 300 2.21 against 2.45 ms with eight, 2.18 with the 8 x
// 3 plan; 24^3 x 1500 9.17, 9.76, 9.28).  Where the plane's columns do not divide by 64 (12 x 12, lines of 8 points), 16.
template <typename R>
constexpr int xv_cols(int nx) {
  const int line = 128 / int(sizeof(cpx<R>)), m = nx / plan_radix(real_plan(nx), 0);
  const int lanes = m == 1 ? 64 : 16;
  return (line * m >= 48 && nx != 24) || lanes < line ? line : lanes;
}
// Column blocks per workgroup (two waves each): four blocks of lines of 48 and 64 points (FP64 64^3 x 256:
// 512 bytes of a row per workgroup, 824 against 862 us per pass with two, 1021 with one, all with the
// slower addressing above; 752 us = 5.7 TB/s now; FP32 373 us against 432 with two), two at 96 points (LDS) and on
// shorter lines where 4096 workgroups remain (FP64 steps with two against one: 24^3 x 300, 5400 workgroups,
// 2.36 / 2.48 ms with the 8 x 3 plan; 32^3 x 200, 6400, 2.64 / 2.78; 24 x 48 x 48 x 60, 4320, 1.306 / 1.319), one below (16^3 x 300, 2400,
// 1.035 / 1.025; 32^3 x 64, 2048, 1.053 / 1.047; 24^3 x 60, 1080, 0.491 / 0.485; 16^3 x 8 0.148 / 0.142).
constexpr int xv_pairs(int nx) { return nx == 48 || nx == 64 ? 4 : 2; }
constexpr size_t kXvTwoBlocksMin = 4096;
// waves per SIMD that the registers must allow
constexpr int xv_mw(int nx) { return nx == 96 ? 3 : 4; }
template <typename R, int NX, int CW, int PAIRS, int M, bool XS>
__global__ __launch_bounds__(128 * PAIRS, xv_mw(NX)) void k_xv(StageArgs<R> a, cpx<R>* __restrict__ dst, int NY, int NZ,
                                                       int S, const cpx<R>* __restrict__ twx_g, KinTables kt) {
  using C = cpx<R>;
  constexpr int FX = real_plan(NX);
  constexpr int RX = plan_radix(FX, 0), MX = NX / RX;
  constexpr int ITEMS = CW * MX, IT = (ITEMS + 63) / 64;
  static_assert(plan_nstages(NX) <= 2, "column split");
  __shared__ C tiles[2 * PAIRS][NX * CW];
  __shared__ C tw[NX];
  __shared__ R tx[NX];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int s = w & 1;
  const int NYZ = NY * NZ;
  const size_t N = size_t(NX) * NYZ;
  const int nblk = NYZ / (CW * PAIRS);
  int blk, i;
  if (nblk % 8 == 0) {
    const int per = nblk >> 3, j = blockIdx.x >> 3;
    i = j / per;
    blk = (blockIdx.x & 7) * per + (j - i * per);
  } else {
    i = blockIdx.x / nblk;
    blk = blockIdx.x - i * nblk;
  }
  const int q0 = (blk * PAIRS + (w >> 1)) * CW;
  const size_t off = size_t(2 * i + s) * N + q0;
  const C* __restrict__ win = reinterpret_cast<const C*>(a.w_in);
  const C* __restrict__ xb = reinterpret_cast<const C*>(a.x_base);
  const R* __restrict__ F = a.fields + q0;
  C* tile = tiles[w];
  const C* other = tiles[w ^ 1];
  C v[IT][RX], r[IT][RX];
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    const uint32_t o = uint32_t(it / CW * NYZ + it % CW) * uint32_t(sizeof(C));
#pragma unroll
    for (int q = 0; q < RX; ++q) v[u][q] = ld_stream<M>(at_bytes(win + (off + size_t(q * MX) * NYZ), o));
  }
  // the fields are loaded along with w where their registers allow, else FD points ahead of their use
  // (96: 350 us FP64 96^3 x 32, 452 with one point at a time)
  constexpr int NPT = IT * RX;
  constexpr int FD = NPT * int(sizeof(R)) <= 64 ? NPT : 32 / int(sizeof(R));
  constexpr bool PRE = FD == NPT;
  R f[FD][4];
  const auto load_f = [&](int p) {
    const int it = min(lane + 64 * (p / RX), ITEMS - 1);
    const uint32_t of = uint32_t(it / CW * NYZ + it % CW) * uint32_t(sizeof(R));
#pragma unroll
    for (int d = 0; d < 4; ++d) f[p % FD][d] = *at_bytes(F + d * N + size_t(p % RX * MX) * NYZ, of);
  };
#pragma unroll
  for (int p = 0; p < FD; ++p) load_f(p);
  const double kx = kt.shift(i, 0);
  for (int k = tid; k < NX; k += 128 * PAIRS) {
    tw[k] = twx_g[k];
    const double g = kt.g[0][plan_position<FX>(k)] + kx;
    tx[k] = R(0.5 / NX * (g * g));
  }
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    {
#pragma unroll
      for (int q = 0; q < RX; ++q) tile[it + q * MX * CW] = v[u][q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    const int x0 = it / CW, col = q0 + it % CW;
    // laser potential, less its x term
    const R lyz = a.lg[3] + a.lg[1] * R(col / NZ) + a.lg[2] * R(col % NZ);
#pragma unroll
    for (int q = 0; q < RX; ++q) {
      const int p = u * RX + q;
      R fq[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) fq[d] = f[p % FD][d];
      if (p + FD < NPT) load_f(p + FD);
      const R vl = fq[0] + (lyz + a.lg[0] * R(x0 + q * MX));
      const R bx = fq[1] + a.bext[0], by = fq[2] + a.bext[1], bz = fq[3] + a.bext[2];
      const C ws = v[u][q], wo = other[it + q * MX * CW];
      // up: (v+bz) up + (bx - i by) dn ; dn: (v-bz) dn + (bx + i by) up
      const R d = s ? vl - bz : vl + bz, e = s ? -by : by;
      const C h = {d * ws.x + bx * wo.x + e * wo.y, d * ws.y + bx * wo.y - e * wo.x};
      r[u][q] = {a.cre * h.x - a.cim * h.y, a.cre * h.y + a.cim * h.x};
      if constexpr (!XS) r[u][q] = {a.alpha * ws.x + r[u][q].x, a.alpha * ws.y + r[u][q].y};
      if (!PRE) {
        pin(r[u][q]);
        sched_fence();
      }
    }
  }
  __syncthreads();  // the other wave has read this tile
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    {
      stage_butterfly<R, FX, 0, true>(v[u], tw, it / CW);
      if constexpr (plan_nstages(NX) > 1) {
#pragma unroll
        for (int q = 0; q < RX; ++q) tile[it + q * MX * CW] = v[u][q];
      } else {  // one stage: all of a column's values are in this lane
#pragma unroll
        for (int q = 0; q < RX; ++q) v[u][q] = cscale(v[u][q], tx[q]);
      }
    }
    if (!PRE) sched_fence();
  }
  if constexpr (plan_nstages(NX) > 1) {
    wave_sync();
    wave_middle<R, FX, CW, 1, CW>(tile, lane, [&](int, int k) { return tx[k]; });
    wave_sync();
  }
  C* out = dst + off;
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int it = min(lane + 64 * u, ITEMS - 1);
    {
      const uint32_t o = uint32_t(it / CW * NYZ + it % CW) * uint32_t(sizeof(C));
      if constexpr (plan_nstages(NX) > 1) {
#pragma unroll
        for (int q = 0; q < RX; ++q) v[u][q] = tile[it + q * MX * CW];
      }
      C xv[RX];
      if constexpr (XS) {
#pragma unroll
        for (int q = 0; q < RX; ++q) xv[q] = ld_stream<M>(at_bytes(xb + (off + size_t(q * MX) * NYZ), o));
      }
      stage_butterfly<R, FX, 0, false>(v[u], tw, it / CW);
#pragma unroll
      for (int q = 0; q < RX; ++q) {
        const C h = v[u][q];
        C t = {r[u][q].x + (a.cre * h.x - a.cim * h.y), r[u][q].y + (a.cre * h.y + a.cim * h.x)};
        if constexpr (XS) t = {a.alpha * xv[q].x + t.x, a.alpha * xv[q].y + t.y};
        st_stream<M>(at_bytes(out + size_t(q * MX) * NYZ, o), t);
      }
    }
    if (!PRE) sched_fence();
  }
}

// (y,z) part of the kinetic energy: part[b][x] = sum over the plane of 1/2 |G_yz + k|^2 |X|^2 /
// (NY NZ), X the (y,z) transform of batch entry b (state b / 2) on plane x.
template <int NY, int NZ>
__global__ __launch_bounds__(plane_nt(NY* NZ)) void k_plane_energy(const cpx<double>* __restrict__ in,
                                                                    const cpx<double>* __restrict__ twy_g,
                                                                    const cpx<double>* __restrict__ twz_g, int B,
                                                                    int NX, double* __restrict__ part, KinTables kt) {
  constexpr int NP = NY * NZ;
  constexpr int NT = plane_nt(NP);
  constexpr int PZ = NZ + 1;
  extern __shared__ double4 smem_d4[];
  cpx<double>* plane = reinterpret_cast<cpx<double>*>(smem_d4);
  cpx<double>* twy = plane + NY * PZ;
  cpx<double>* twz = twy + NY;
  __shared__ double red[NT / 64];
  const int tid = threadIdx.x;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / B;
  const int b = L - x * B;
  for (int k = tid; k < NY; k += NT) twy[k] = twy_g[k];
  for (int k = tid; k < NZ; k += NT) twz[k] = twz_g[k];
  const size_t off = (size_t(b) * NX + x) * NP;
  for (int e = tid; e < NP; e += NT) plane[(e / NZ) * PZ + (e % NZ)] = in[off + e];
  __syncthreads();
  plane_fft_fwd<double, NY, NZ, PZ>(plane, twy, twz, tid, NT);
  const double ky = kt.shift(b / 2, 1), kz = kt.shift(b / 2, 2);
  double s = 0.0;
  for (int e = tid; e < NP; e += NT) {
    const double gy = kt.g[1][e / NZ] + ky, gz = kt.g[2][e % NZ] + kz;
    const cpx<double> v = plane[(e / NZ) * PZ + (e % NZ)];
    s += (gy * gy + gz * gz) * (v.x * v.x + v.y * v.y);
  }
  const double t = block_sum<NT>(s, red);
  if (tid == 0) part[size_t(b) * NX + x] = t * (0.5 / NP);
}

// x part of the kinetic energy and the norm: per (batch entry, tile of TC columns) sums of
// 1/2 (G_x + k_x)^2 |X|^2 / NX and |X|^2 / NX, X the x transform of the states.
template <int NX, int TC>
__global__ __launch_bounds__(256) void k_xkin_energy(const cpx<double>* __restrict__ src, int NYZ,
                                                     const cpx<double>* __restrict__ twx_g,
                                                     double* __restrict__ part, KinTables kt) {
  __shared__ cpx<double> tile[NX * TC];
  __shared__ cpx<double> tw[NX];
  __shared__ double red[4];
  const int tid = threadIdx.x;
  const int tiles = NYZ / TC;
  const int b = blockIdx.x / tiles;
  for (int k = tid; k < NX; k += 256) tw[k] = twx_g[k];
  const size_t base = size_t(b) * NX * NYZ + (blockIdx.x - b * tiles) * TC;
  constexpr int PER = (NX * TC + 255) / 256;
  {
    cpx<double> v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = min(tid + j * 256, NX * TC - 1);  // clamped: every load unconditional
      v[j] = src[base + size_t(e / TC) * NYZ + (e % TC)];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + j * 256;
      if (e < NX * TC) tile[e] = v[j];
    }
  }
  __syncthreads();
  lds_fft<double, NX, TC, 1, TC, true>(tile, tw, tid, 256);
  const double kx = kt.shift(b / 2, 0);
  double s1 = 0.0, s2 = 0.0;
  for (int e = tid; e < NX * TC; e += 256) {
    const double gx = kt.g[0][e / TC] + kx;
    const double a2 = tile[e].x * tile[e].x + tile[e].y * tile[e].y;
    s1 += gx * gx * a2;
    s2 += a2;
  }
  const double t1 = block_sum<256>(s1, red);
  const double t2 = block_sum<256>(s2, red);
  if (tid == 0) {
    part[size_t(blockIdx.x) * 2 + 0] = t1 * (0.5 / NX);
    part[size_t(blockIdx.x) * 2 + 1] = t2 * (1.0 / NX);
  }
}

// ---------------------------------------------------------------- plane pass: transform only
// SRC: what `in` holds: 0 complex values; 1 a spin density rho_v (real, [4][N]; the transform
// takes n = rho_uu + rho_dd), 2 a real array (the transform takes it as the real part).
template <typename R, int NY, int NZ, int SRC = 0>
__global__ __launch_bounds__(plane_nt(NY* NZ)) void k_plane_fwd(const cpx<R>* in, cpx<R>* out,
                                                                 cpx<R>* W, ProjTables pt,
                                                                 const cpx<R>* __restrict__ twy_g,
                                                                 const cpx<R>* __restrict__ twz_g,
                                                                 int B, int NX, KTables<R> kt) {
  constexpr int NP = NY * NZ;
  constexpr int NT = plane_nt(NP);
  constexpr int PZ = NZ + 1;
  extern __shared__ double4 smem_d4[];
  cpx<R>* plane = reinterpret_cast<cpx<R>*>(smem_d4);
  cpx<R>* twy = plane + NY * PZ;
  cpx<R>* twz = twy + NY;
  const int tid = threadIdx.x;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / B;
  const int b = L - x * B;
  for (int k = tid; k < NY; k += NT) twy[k] = twy_g[k];
  for (int k = tid; k < NZ; k += NT) twz[k] = twz_g[k];
  const size_t off = (size_t(b) * NX + x) * NP;
  if constexpr (SRC == 0) {
    for (int e = tid; e < NP; e += NT) plane[(e / NZ) * PZ + (e % NZ)] = in[off + e];
  } else {
    const R* rin = reinterpret_cast<const R*>(in);
    const size_t Nall = size_t(NX) * NP;
    for (int e = tid; e < NP; e += NT)
      plane[(e / NZ) * PZ + (e % NZ)] = cpx<R>{SRC == 1 ? rin[off + e] + rin[Nall + off + e] : rin[off + e], R(0)};
  }
  __syncthreads();
  if (W && pt.pr_off) {
    const size_t rowbase = size_t(b) * pt.Jtot;
    const bool kq = kt.kv != nullptr;
    R q0 = 0, q1 = 0, q2 = 0;
    if (kq) {
      const R* k0 = kt.kv + 3 * (kt.state_off + b / 2);
      q0 = k0[0] + kt.ka[0];
      q1 = k0[1] + kt.ka[1];
      q2 = k0[2] + kt.ka[2];
    }
    const R* disp = reinterpret_cast<const R*>(pt.disp);
    for (int r = pt.pr_off[x]; r < pt.pr_off[x + 1]; ++r) {
      for (int J = pt.pr_begin[r] + tid; J < pt.pr_end[r]; J += NT) {
        const int e = pt.pidx[J];
        cpx<R> o = plane[(e / NZ) * PZ + (e % NZ)];
        if (kq) o = cmul(o, bloch_phase(q0, q1, q2, disp + 3 * J));
        W[rowbase + J] = o;
      }
    }
    __syncthreads();
  }
  plane_fft_fwd<R, NY, NZ, PZ>(plane, twy, twz, tid, NT);
  for (int e = tid; e < NP; e += NT) out[off + e] = plane[(e / NZ) * PZ + (e % NZ)];
}

template <typename R, int NY, int NZ>
__global__ __launch_bounds__(plane_nt(NY* NZ)) void k_plane_inv(const cpx<R>* in, cpx<R>* out,
                                                                 R scale,
                                                                 const cpx<R>* __restrict__ twy_g,
                                                                 const cpx<R>* __restrict__ twz_g,
                                                                 int B, int NX) {
  constexpr int NP = NY * NZ;
  constexpr int NT = plane_nt(NP);
  constexpr int PZ = NZ + 1;
  extern __shared__ double4 smem_d4[];
  cpx<R>* plane = reinterpret_cast<cpx<R>*>(smem_d4);
  cpx<R>* twy = plane + NY * PZ;
  cpx<R>* twz = twy + NY;
  const int tid = threadIdx.x;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int x = L / B;
  const int b = L - x * B;
  for (int k = tid; k < NY; k += NT) twy[k] = twy_g[k];
  for (int k = tid; k < NZ; k += NT) twz[k] = twz_g[k];
  const size_t off = (size_t(b) * NX + x) * NP;
  for (int e = tid; e < NP; e += NT) plane[(e / NZ) * PZ + (e % NZ)] = in[off + e];
  __syncthreads();
  plane_fft_inv<R, NY, NZ, PZ>(plane, twy, twz, tid, NT);
  for (int e = tid; e < NP; e += NT) out[off + e] = cscale(plane[(e / NZ) * PZ + (e % NZ)], scale);
}

// ---------------------------------------------------------------- column pass along x
// widest column-pass tile (64, 32, 16 columns) whose LDS footprint stays within a budget
// (tuning macros, bytes per workgroup).  FP32 at 96 points takes 64 columns (48 KB, three
// 512-thread workgroups per CU): 4717 against 4535 GB/s with 32 columns (96^3 x 512).
#ifndef NCT_XPASS_TILE_MAX_F64
#define NCT_XPASS_TILE_MAX_F64 32768
#endif
#ifndef NCT_XPASS_TILE_MAX_F32
#define NCT_XPASS_TILE_MAX_F32 49152
#endif
template <typename R>
constexpr int xpass_tc(int nx) {
  const int b = int(sizeof(R)) * 2;
  const int cap = sizeof(R) == 8 ? NCT_XPASS_TILE_MAX_F64 : NCT_XPASS_TILE_MAX_F32;
  if (nx * 64 * b <= cap) return 64;
  if (nx * 32 * b <= cap) return 32;
  return 16;
}
constexpr int XP_NT = 256;  // threads of the energy column pass
// threads of the column pass per precision (tuning macros); FP32 tiles of 64 columns whose first
// stage has at least 512 butterflies take NCT_XPASS_NT_F32_WIDE: at 64 points 512 threads
// measured 4848 against 4571 GB/s (64^3 x 256), while the 48-point tile (384 butterflies) and
// the 32-column tile at 96 points lost with 512 (4324 against 4402, 4256 against 4543 GB/s), and
// the 64-column tile at 96 points with 256 (4159 against 4717 GB/s).  FP64 passes here are those of the
// Poisson solve, one box of a few us.
#ifndef NCT_XPASS_NT_F64
#define NCT_XPASS_NT_F64 256
#endif
#ifndef NCT_XPASS_NT_F32
#define NCT_XPASS_NT_F32 256
#endif
#ifndef NCT_XPASS_NT_F32_WIDE
#define NCT_XPASS_NT_F32_WIDE 512
#endif
template <typename R, int NX, int TC>
__host__ __device__ constexpr int xp_nt() {
  if constexpr (sizeof(R) == 4 && TC == 64 && TC * NX / plan_radix(NX, 0) >= 512) return NCT_XPASS_NT_F32_WIDE;
  return sizeof(R) == 8 ? NCT_XPASS_NT_F64 : NCT_XPASS_NT_F32;
}

// Column pass: one workgroup per tile of TC consecutive yz columns x NX planes of one batch
// entry (spinor component).  The first forward x stage works on the values as they are loaded.
template <typename R, int NX, int TC, int M>
__global__ __launch_bounds__((xp_nt<R, NX, TC>())) void k_xpass(const cpx<R>* src, cpx<R>* dst, int NYZ,
                                                 const R* __restrict__ g2x,
                                                 const R* __restrict__ g2yz, R kscale, int mode,
                                                 const cpx<R>* __restrict__ twx_g, KTables<R> kt) {
  __shared__ cpx<R> tile[NX * TC];
  __shared__ cpx<R> tw[NX];
  const int tid = threadIdx.x;
  const int tiles = NYZ / TC;
  const int b = blockIdx.x / tiles;
  const int q0 = (blockIdx.x - b * tiles) * TC;
  for (int k = tid; k < NX; k += xp_nt<R, NX, TC>()) tw[k] = twx_g[k];
  const cpx<R>* srcb = src + size_t(b) * NX * NYZ + q0;
  cpx<R>* dstb = dst + size_t(b) * NX * NYZ + q0;
  {
    // forward DFT along x; its last stage applies the kinetic (mode 0) or Poisson (mode 1)
    // factor as it writes back; the inverse DFT's last stage stores to dst
    constexpr int NS = plan_nstages(NX);
    if constexpr (NS > 1) {
      stage_from<R, NX, 0, TC, 1, TC, 1, TC, xp_nt<R, NX, TC>(), true>(
          tile, tw, tid, [&](int e) { return ld_stream<M>(&srcb[size_t(e / TC) * NYZ + (e % TC)]); });
    } else {
      for (int e = tid; e < NX * TC; e += xp_nt<R, NX, TC>()) tile[e] = ld_stream<M>(&srcb[size_t(e / TC) * NYZ + (e % TC)]);
      __syncthreads();
    }
    if constexpr (NS > 2) {
      lds_stage<R, NX, 1, TC, 1, TC, true>(tile, tw, tid, xp_nt<R, NX, TC>());
      __syncthreads();
    }
    stage_to<R, NX, NS - 1, TC, 1, TC, 1, TC, xp_nt<R, NX, TC>(), true>(
        tile, tw, tid, [](int) { return 0; }, [&](int e, int l, cpx<R> v, int) {
          R g;
          if (kt.kv) {  // |G + k|^2 of this spinor component's state
            const R* k = kt.kv + 3 * (kt.state_off + b / 2);
            const R gx = kt.gx[e / TC] + (k[0] + kt.ka[0]);
            const R gy = kt.gy[q0 + (e % TC)] + (k[1] + kt.ka[1]);
            const R gz = kt.gz[q0 + (e % TC)] + (k[2] + kt.ka[2]);
            g = gx * gx + gy * gy + gz * gz;
          } else {
            g = g2x[e / TC] + g2yz[q0 + (e % TC)];
          }
          R m;
          if (mode == 0) m = kscale * g;
          else m = g > R(0) ? kscale / g : R(0);
          tile[l] = cscale(v, m);
        });
    __syncthreads();
    if constexpr (NS > 2) {
      lds_stage<R, NX, 2, TC, 1, TC, false>(tile, tw, tid, xp_nt<R, NX, TC>());
      __syncthreads();
    }
    if constexpr (NS > 1) {
      lds_stage<R, NX, 1, TC, 1, TC, false>(tile, tw, tid, xp_nt<R, NX, TC>());
      __syncthreads();
    }
    stage_to<R, NX, 0, TC, 1, TC, 1, TC, xp_nt<R, NX, TC>(), false>(
        tile, tw, tid, [](int) { return 0; }, [&](int e, int, cpx<R> v, int) {
          st_stream<M>(&dstb[size_t(e / TC) * NYZ + (e % TC)], v);
        });
  }
}

template <typename R, int NX, int TC>
__global__ __launch_bounds__(XP_NT) void k_xpass_energy(const cpx<R>* src, int NYZ,
                                                        const R* __restrict__ g2x,
                                                        const R* __restrict__ g2yz, R kscale,
                                                        const cpx<R>* __restrict__ twx_g,
                                                        double* part, KTables<R> kt) {
  __shared__ cpx<R> tile[NX * TC];
  __shared__ cpx<R> tw[NX];
  __shared__ double red[XP_NT / 64];
  const int tid = threadIdx.x;
  const int tiles = NYZ / TC;
  const int b = blockIdx.x / tiles;
  const int tl = blockIdx.x - b * tiles;
  const int q0 = tl * TC;
  for (int k = tid; k < NX; k += XP_NT) tw[k] = twx_g[k];
  const size_t base = size_t(b) * NX * NYZ + q0;
  constexpr int PER = (NX * TC + XP_NT - 1) / XP_NT;
  {
    cpx<R> v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = min(tid + j * XP_NT, NX * TC - 1);  // clamped: every load unconditional
      v[j] = src[base + size_t(e / TC) * NYZ + (e % TC)];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + j * XP_NT;
      if (e < NX * TC) tile[e] = v[j];
    }
  }
  __syncthreads();
  lds_fft<R, NX, TC, 1, TC, true>(tile, tw, tid, XP_NT);
  double s1 = 0.0, s2 = 0.0;
  for (int e = tid; e < NX * TC; e += XP_NT) {
    const int xx = e / TC, c = e - (e / TC) * TC;
    double g;
    if (kt.kv) {
      const R* k = kt.kv + 3 * (kt.state_off + b / 2);
      const double gx = double(kt.gx[xx]) + double(k[0] + kt.ka[0]);
      const double gy = double(kt.gy[q0 + c]) + double(k[1] + kt.ka[1]);
      const double gz = double(kt.gz[q0 + c]) + double(k[2] + kt.ka[2]);
      g = gx * gx + gy * gy + gz * gz;
    } else {
      g = double(g2x[xx]) + double(g2yz[q0 + c]);
    }
    const double a2 = double(tile[e].x) * double(tile[e].x) + double(tile[e].y) * double(tile[e].y);
    s1 += double(kscale) * g * a2;
    s2 += a2;
  }
  const double t1 = block_sum<XP_NT>(s1, red);
  const double t2 = block_sum<XP_NT>(s2, red);
  if (tid == 0) {
    part[size_t(blockIdx.x) * 2 + 0] = t1;
    part[size_t(blockIdx.x) * 2 + 1] = t2;
  }
}

// ---------------------------------------------------------------- density (Eq. density4)
template <typename R>
__global__ __launch_bounds__(256) void k_density(const cpx<R>* __restrict__ psi,
                                                 const double* __restrict__ occ, int S, size_t N,
                                                 double* __restrict__ rho) {
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= N) return;
  double uu = 0, dd = 0, udr = 0, udi = 0;
#pragma unroll 4
  for (int i = 0; i < S; ++i) {
    const double f = occ[i];
    const cpx<R> u = psi[size_t(2 * i) * N + p];
    const cpx<R> d = psi[size_t(2 * i + 1) * N + p];
    const double ux = u.x, uy = u.y, dx = d.x, dy = d.y;
    uu += f * (ux * ux + uy * uy);
    dd += f * (dx * dx + dy * dy);
    udr += f * (ux * dx + uy * dy);   // Re(u d*)
    udi += f * (uy * dx - ux * dy);   // Im(u d*)
  }
  rho[p] = uu;
  rho[N + p] = dd;
  rho[2 * N + p] = udr;
  rho[3 * N + p] = udi;
}

// ---------------------------------------------------------------- exchange + fields (FP64)
// Locally collinear Slater exchange (Eqs. LC+ALDA2, LC+ALDA):
//   n_s = (n +/- |m|)/2, v_s = -(6/pi)^(1/3) n_s^(1/3), vbar = (v_up+v_dn)/2,
//   b_xc = (v_up - v_dn)/2 m/|m| (0 below threshold), e_x = -(3/4)(6/pi)^(1/3) sum n_s^(4/3).
// v_up - v_dn is evaluated as -(6/pi)^(1/3) (n_up - n_dn) / (n_up^(2/3) + (n_up n_dn)^(1/3) + n_dn^(2/3)).
// Dual number v + d e (e^2 = 0) for forward-mode derivatives of the correlation potentials in
// the adjoint; the elementary functions below take double or dual.  cbrt's derivative at 0 is
// taken as 0 (the one-sided value of the clamped channel).
struct dnum {
  double v, d;
};
__device__ __forceinline__ dnum operator+(dnum a, dnum b) { return {a.v + b.v, a.d + b.d}; }
__device__ __forceinline__ dnum operator-(dnum a, dnum b) { return {a.v - b.v, a.d - b.d}; }
__device__ __forceinline__ dnum operator*(dnum a, dnum b) { return {a.v * b.v, a.d * b.v + a.v * b.d}; }
__device__ __forceinline__ dnum operator/(dnum a, dnum b) {
  return {a.v / b.v, (a.d * b.v - a.v * b.d) / (b.v * b.v)};
}
__device__ __forceinline__ dnum operator+(double a, dnum b) { return {a + b.v, b.d}; }
__device__ __forceinline__ dnum operator+(dnum a, double b) { return {a.v + b, a.d}; }
__device__ __forceinline__ dnum operator-(double a, dnum b) { return {a - b.v, -b.d}; }
__device__ __forceinline__ dnum operator-(dnum a, double b) { return {a.v - b, a.d}; }
__device__ __forceinline__ dnum operator*(double a, dnum b) { return {a * b.v, a * b.d}; }
__device__ __forceinline__ dnum operator*(dnum a, double b) { return {a.v * b, a.d * b}; }
__device__ __forceinline__ dnum operator/(double a, dnum b) { return {a / b.v, -a * b.d / (b.v * b.v)}; }
__device__ __forceinline__ dnum operator/(dnum a, double b) { return {a.v / b, a.d / b}; }
__device__ __forceinline__ double xval(double x) { return x; }
__device__ __forceinline__ double xval(dnum x) { return x.v; }
__device__ __forceinline__ double xcbrt(double x) { return cbrt(x); }
__device__ __forceinline__ dnum xcbrt(dnum x) {
  const double c = cbrt(x.v);
  return {c, c != 0.0 ? x.d / (3.0 * c * c) : 0.0};
}
__device__ __forceinline__ double xsqrt(double x) { return sqrt(x); }
__device__ __forceinline__ dnum xsqrt(dnum x) {
  const double r = sqrt(x.v);
  return {r, x.d / (2.0 * r)};
}
__device__ __forceinline__ double xlog1p(double x) { return log1p(x); }
__device__ __forceinline__ dnum xlog1p(dnum x) { return {log1p(x.v), x.d / (1.0 + x.v)}; }
__device__ __forceinline__ double xclamp01(double x) { return fmin(fmax(x, 0.0), 1.0); }
__device__ __forceinline__ dnum xclamp01(dnum x) {
  if (x.v < 0.0) return {0.0, 0.0};
  if (x.v > 1.0) return {1.0, 0.0};
  return x;
}

// PW92 LSDA correlation (J. P. Perdew and Y. Wang, Phys. Rev. B 45, 13244 (1992)).
// G(rs) = -2A(1 + a1 rs) ln[1 + 1/(2A(b1 rs^1/2 + b2 rs + b3 rs^3/2 + b4 rs^2))] and dG/drs.
template <typename T>
__device__ __forceinline__ void pw92_g(T rs, T srs, double A, double a1, double b1, double b2, double b3,
                                       double b4, T& g, T& dg) {
  const T q0 = -2.0 * A * (1.0 + a1 * rs);
  const T q1 = 2.0 * A * (b1 * srs + b2 * rs + b3 * rs * srs + b4 * rs * rs);
  const T q1p = A * (b1 / srs + 2.0 * b2 + 3.0 * b3 * srs + 4.0 * b4 * rs);
  const T lg = xlog1p(1.0 / q1);
  g = q0 * lg;
  dg = -2.0 * A * a1 * lg - q0 * q1p / (q1 * q1 + q1);
}
// Locally collinear PW92 at density n and |m| = mu: vbar = (v_up + v_dn)/2, bmag = (v_up - v_dn)/2
// (the field along m/|m|), ec = n eps_c; zero where n <= 1e-30.  T = dnum carries the derivative
// along the direction given in n.d, mu.d; T = double is the plain evaluation.
template <typename T>
__device__ void pw92_lc(T n, T mu, T& vbar, T& bmag, T& ec) {
  vbar = bmag = ec = T{};
  if (!(xval(n) > 1e-30)) return;
  const T rs = xcbrt(0.75 / (3.14159265358979323846 * n));
  const T srs = xsqrt(rs);
  const T z = xclamp01(mu / n);
  T e0, d0, e1, d1, ma, dma;
  pw92_g(rs, srs, 0.031091, 0.21370, 7.5957, 3.5876, 1.6382, 0.49294, e0, d0);    // zeta = 0
  pw92_g(rs, srs, 0.015545, 0.20548, 14.1189, 6.1977, 3.3662, 0.62517, e1, d1);   // zeta = 1
  pw92_g(rs, srs, 0.016887, 0.11125, 10.357, 3.6231, 0.88026, 0.49671, ma, dma);  // -alpha_c
  const T ac = 0.0 - ma, dac = 0.0 - dma;
  const double fpp0 = 1.709921;
  const double fden = 0.5198420997897464;  // 2^(4/3) - 2
  const T cu = xcbrt(1.0 + z), cd = xcbrt(1.0 - z);
  const T f = ((1.0 + z) * cu + (1.0 - z) * cd - 2.0) / fden;
  const T fp = (4.0 / 3.0) * (cu - cd) / fden;
  const T z3 = z * z * z, z4 = z3 * z;
  const T eps = e0 + ac * f * (1.0 - z4) / fpp0 + (e1 - e0) * f * z4;
  const T drs = d0 * (1.0 - f * z4) + d1 * f * z4 + dac * f * (1.0 - z4) / fpp0;
  const T dz = 4.0 * z3 * f * (e1 - e0 - ac / fpp0) + fp * (z4 * (e1 - e0) + (1.0 - z4) * ac / fpp0);
  vbar = eps - rs / 3.0 * drs - z * dz;
  bmag = dz;
  ec = n * eps;
}
static __global__ __launch_bounds__(256) void k_fields(const double* __restrict__ rho,
                                                const double* __restrict__ vext,
                                                const double* __restrict__ vH, int xc, double thr,
                                                int ny, int nz, double hx, double hy, double hz,
                                                double cx, double cy, double cz, size_t N,
                                                double* __restrict__ fields,
                                                float* __restrict__ f32, double* __restrict__ part) {
  __shared__ double red[4][kFieldTot];
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  double n = 0, mx = 0, my = 0, mz = 0, eloc = 0, eh = 0, ex = 0, dx = 0, dy = 0, dz = 0;
  if (p < N) {
    const double ruu = rho[p], rdd = rho[N + p], rr = rho[2 * N + p], ri = rho[3 * N + p];
    n = ruu + rdd;
    mx = 2.0 * rr;
    my = -2.0 * ri;
    mz = ruu - rdd;
    const double ve = vext ? vext[p] : 0.0;
    const double vh = vH ? vH[2 * p] : 0.0;  // real part of the complex Poisson output
    double vbar = 0.0, bx = 0.0, by = 0.0, bz = 0.0;
    if (xc) {
      const double c = 1.2407009817988000;  // (6/pi)^(1/3)
      const double mu = sqrt(mx * mx + my * my + mz * mz);
      const double nu = fmax(0.5 * (n + mu), 0.0);
      const double nd = fmax(0.5 * (n - mu), 0.0);
      const double cu = cbrt(nu), cd = cbrt(nd);
      vbar = -0.5 * c * (cu + cd);
      ex = -0.75 * c * (nu * cu + nd * cd);
      double bmag = 0.0;
      if (mu >= thr) {
        const double den = cu * cu + cu * cd + cd * cd;
        bmag = den > 0.0 ? -0.5 * c * (nu - nd) / den : 0.0;
      }
      if (xc >= 2) {
        double vc, bc, ec;
        pw92_lc<double>(n, mu, vc, bc, ec);
        vbar += vc;
        ex += ec;
        if (mu >= thr) bmag += bc;
      }
      if (mu >= thr) {
        const double s = bmag / mu;
        bx = s * mx;
        by = s * my;
        bz = s * mz;
      }
    }
    const double v = ve + vh + vbar;
    fields[p] = v;
    fields[N + p] = bx;
    fields[2 * N + p] = by;
    fields[3 * N + p] = bz;
    if (f32) {
      f32[p] = float(v);
      f32[N + p] = float(bx);
      f32[2 * N + p] = float(by);
      f32[3 * N + p] = float(bz);
    }
    eloc = ve * n;
    eh = 0.5 * vh * n;
    const size_t nyz = size_t(ny) * nz;
    const int ix = int(p / nyz);
    const int rem = int(p - size_t(ix) * nyz);
    const int iy = rem / nz;
    const int iz = rem - iy * nz;
    dx = (ix * hx - cx) * n;
    dy = (iy * hy - cy) * n;
    dz = (iz * hz - cz) * n;
  }
  const double vals[kFieldTot] = {n, mx, my, mz, eloc, eh, ex, 0.0, dx, dy, dz, 0.0};
  block_sums<256>(vals, red, part + size_t(blockIdx.x) * kFieldTot);
}

// out[w] = sum_r part[r*width + w], fixed order, one workgroup per w; copy0, if given, receives out[0] as
// well.  (One workgroup that took the columns in turn was a chain of reads and barriers: 6.8
// against 2.4 us at 16^3, 5.9 against 4.0 at 32^3.)
static __global__ __launch_bounds__(256) void k_reduce_rows(const double* __restrict__ part, int nrows,
                                                     int width, double* __restrict__ out,
                                                     double* __restrict__ copy0) {
  __shared__ double red[4];
  const int w = blockIdx.x;
  double s = 0.0;
  for (int r = threadIdx.x; r < nrows; r += 256) s += part[size_t(r) * width + w];
  const double t = block_sum<256>(s, red);
  if (threadIdx.x == 0) {
    out[w] = t;
    if (w == 0 && copy0) *copy0 = t;
  }
}

static __global__ void k_add_bext(const double* __restrict__ f, int ny, int nz, size_t N, double b0,
                           double b1, double b2, double l0, double l1, double l2, double l3,
                           double* __restrict__ out) {
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p < N) {
    const size_t nyz = size_t(ny) * nz;
    const int ix = int(p / nyz);
    const int rem = int(p - size_t(ix) * nyz);
    const int iy = rem / nz;
    const int iz = rem - iy * nz;
    out[p] = f[p] + (l0 * ix + l1 * iy + l2 * iz + l3);
    out[N + p] = f[N + p] + b0;
    out[2 * N + p] = f[2 * N + p] + b1;
    out[3 * N + p] = f[3 * N + p] + b2;
  }
}
static __global__ void k_to_float(const double* __restrict__ in, size_t n, float* __restrict__ out) {
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p < n) out[p] = float(in[p]);
}

// ---------------------------------------------------------------- projectors on the matrix cores
typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <typename R>
struct mfma16;
// Output element r of lane l is D[row(r, l/16)][l%16]: the f64 instruction interleaves the
// four row groups across registers, the f32 one keeps four consecutive rows per lane.
template <>
struct mfma16<double> {
  typedef d4v acc;
  static __device__ __forceinline__ int row(int r, int kl) { return 4 * r + kl; }
  static __device__ __forceinline__ acc zero() { return acc{0.0, 0.0, 0.0, 0.0}; }
  static __device__ __forceinline__ acc op(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct mfma16<float> {
  typedef f4v acc;
  static __device__ __forceinline__ int row(int r, int kl) { return 4 * kl + r; }
  static __device__ __forceinline__ acc zero() { return acc{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ acc op(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// k-steps whose operands are loaded together.  Neither loaded ahead of the products before them nor eight at a time in
// FP32: that wins 1 % where a system is small (48^3 x 32 mixed with four atoms 1.120 against 1.119 ms, 96 x 24 x
// 24 x 40 0.801 against 0.805) and takes the registers of a wave per SIMD where it is not (32^3 x 200 mixed with two atoms
// 1.97 against 1.87 ms, contraction 34 against 21 us).
constexpr int KU = 4;

// Cpart[a][kc][p][i] = sum_{k in chunk} conj(beta[a][k][p]) W[i][k], k = 2 (J - off_a) + s.
// One wave: PP/16 output tiles of 16 projectors x 16 states; A/B operands as
// A[row = lane%16][k = lane/16], B[k = lane/16][col = lane%16]; D rows from mfma16::row.
// KQ: the rows of W are taken times the phases exp(i k.d) of PhaseTab (real-space form with Bloch vectors;
// in the transformed form the plane pass has put the phase on them).
template <typename R, int PP, bool KQ>
__global__ __launch_bounds__(64, 3) void k_proj_contract(ProjTables pt, const cpx<R>* __restrict__ W,
                                                      int S, cpx<double>* __restrict__ Cpart, PhaseTab ph) {
  using M = mfma16<R>;
  constexpr int NMT = PP / 16;
  const int a = blockIdx.x, nt = blockIdx.y, kc = blockIdx.z;
  const int off = pt.row_off[a];
  const int K = 2 * (pt.row_off[a + 1] - off);
  const int KC = pt.kc;
  if (kc * KC >= K) return;
  const int lane = threadIdx.x;
  const int col = lane & 15, kl = lane >> 4;
  const int i = nt * 16 + col;
  const cpx<R>* __restrict__ beta = reinterpret_cast<const cpx<R>*>(pt.beta);
  const cpx<R>* __restrict__ phase = nullptr;
  if constexpr (KQ) phase = ph.row<R>(min(i, S - 1), pt.Jtot);
  typename M::acc ar[NMT], ai[NMT];
#pragma unroll
  for (int mt = 0; mt < NMT; ++mt) {
    ar[mt] = M::zero();
    ai[mt] = M::zero();
  }
  const int kend = min(K, kc * KC + KC);
  for (int k0 = kc * KC; k0 < kend; k0 += 4 * KU) {
    cpx<R> bw[KU], bb[KU][NMT];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = k0 + 4 * u + kl;
      const bool ok = k < kend;
      const int kk = ok ? k : kc * KC;  // clamped index, value zeroed below
      const int J = off + (kk >> 1), s = kk & 1;
      cpx<R> w = W[size_t(2 * min(i, S - 1) + s) * pt.Jtot + J];
      if constexpr (KQ) w = cmul(w, phase[J]);
      bw[u] = (ok && i < S) ? w : cpx<R>{R(0), R(0)};
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt) {
        const cpx<R> v = beta[(size_t(2 * off) + kk) * PP + mt * 16 + col];
        bb[u][mt] = ok ? v : cpx<R>{R(0), R(0)};
      }
    }
#pragma unroll
    for (int u = 0; u < KU; ++u) {
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt) {
        ar[mt] = M::op(bb[u][mt].x, bw[u].x, ar[mt]);
        ar[mt] = M::op(bb[u][mt].y, bw[u].y, ar[mt]);
        ai[mt] = M::op(bb[u][mt].x, bw[u].y, ai[mt]);
        ai[mt] = M::op(-bb[u][mt].y, bw[u].x, ai[mt]);
      }
    }
  }
  const int nch = pt.max_kchunks;
#pragma unroll
  for (int mt = 0; mt < NMT; ++mt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int p = mt * 16 + M::row(r, kl);
      if (i < S)
        Cpart[((size_t(a) * nch + kc) * PP + p) * S + i] = {double(ar[mt][r]), double(ai[mt][r])};
    }
  }
}

// dV sum_kc Cpart[a][kc][p + 16 c][i] in chunk order, c < NC, sixteen reads in flight: the sums are short,
// and each wait for memory counts
template <int NC>
__device__ __forceinline__ void proj_sums(const ProjTables& pt, const cpx<double>* __restrict__ Cpart, int S, double dV,
                                          int a, int p, int i, cpx<double> (&out)[NC]) {
  constexpr int U = 16 / NC;
  const int K = 2 * (pt.row_off[a + 1] - pt.row_off[a]);
  const int nch_a = (K + pt.kc - 1) / pt.kc;
  const size_t stride = size_t(pt.PP) * S;
  const cpx<double>* src = Cpart + (size_t(a) * pt.max_kchunks * pt.PP + p) * S + i;
#pragma unroll
  for (int c = 0; c < NC; ++c) out[c] = {0.0, 0.0};
  for (int kc = 0; kc < nch_a; kc += U) {
    cpx<double> v[U][NC];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) v[u][c] = src[size_t(min(kc + u, nch_a - 1)) * stride + size_t(16 * c) * S];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (kc + u < nch_a) {
#pragma unroll
        for (int c = 0; c < NC; ++c) out[c] = out[c] + v[u][c];
      }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) out[c] = {out[c].x * dV, out[c].y * dV};
}
// C[a][p][i] of the observables
static __global__ __launch_bounds__(256) void k_proj_reduce(ProjTables pt, const cpx<double>* __restrict__ Cpart,
                                                            int S, double dV, cpx<double>* __restrict__ C) {
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= size_t(pt.natoms) * pt.PP * S) return;
  cpx<double> c[1];
  proj_sums<1>(pt, Cpart, S, dV, int(idx / (size_t(S) * pt.PP)), int((idx / S) % pt.PP), int(idx % S), c);
  C[idx] = c[0];
}

// EC[a][p][i] = E[a][p] C[a][p][i] of the scatter
template <typename R>
__global__ __launch_bounds__(256) void k_proj_coeffs(ProjTables pt, const cpx<double>* __restrict__ Cpart, int S,
                                                     double dV, cpx<R>* __restrict__ EC) {
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= size_t(pt.natoms) * pt.PP * S) return;
  const int a = int(idx / (size_t(S) * pt.PP)), p = int((idx / S) % pt.PP);
  cpx<double> c[1];
  proj_sums<1>(pt, Cpart, S, dV, a, p, int(idx % S), c);
  const double en = pt.energy[size_t(a) * pt.PP + p];
  EC[idx] = {R(en * c[0].x), R(en * c[0].y)};
}

// Y[i][s][J] = sum_p beta[J][s][p] E[a][p] C[a][p][i]; rows k = 2 (J - off_a) + s (KQ: times exp(-i k.d)).
// One workgroup per (atom, 16 states, share of the atom's row tiles).  SUMS: it first sums the chunk partials of its
// own 16 x PP coefficients, which all shares of an atom repeat.  That is for small systems, whose chain
// runs on the main stream: a launch of its own stands on the path that the plane pass waits for (5-39 us each
// time).  On a stream of its own the chain is hidden but for its share of memory and CUs, and there k_proj_coeffs
// sums once: repeated sums made 48^3 x 128 mixed with 16 atoms 4.56 ms per step (4.38 now), 48^3 x 64
// mixed with four 2.03 (2.00), and limiting the shares for them left four waves for all 111 row tiles of an atom.
// The projector values of the next row tile are loaded ahead (of the first one before the sums), and as in
// the contraction the register bound keeps the products out of accumulation registers: contraction and
// scatter together 17.2 against 17.8 us at 32^3 x 16 FP64, H application 32 x 16 x 24 x 39 with its density
// and fields 87 against 92 us.  Sixteen reads of partials in flight, not
// eight with the last ones singly: 8.6 -> 7.7 us at 16^3 x 8 mixed with two atoms.
// With the sums FP64 takes one coefficient per thread, FP32 256 threads (one or two); without, one wave.
template <typename R, int PP, bool SUMS>
constexpr int ps_nt() { return !SUMS ? 64 : (sizeof(R) == 8 ? 16 * PP : 256); }
template <typename R, int PP, bool KQ, bool SUMS>
__global__ __launch_bounds__((ps_nt<R, PP, SUMS>()), 4) void k_proj_scatter(ProjTables pt, const cpx<double>* __restrict__ Cpart,
                                                        const cpx<R>* __restrict__ EC, int S, double dV,
                                                        cpx<R>* __restrict__ Y, PhaseTab ph) {
  using M = mfma16<R>;
  constexpr int KS = PP / 4, NT = ps_nt<R, PP, SUMS>();
  __shared__ cpx<R> ecs[SUMS ? PP : 1][16];
  const int a = blockIdx.x, nt = blockIdx.y;
  const int off = pt.row_off[a];
  const int K2 = 2 * (pt.row_off[a + 1] - off);
  if (K2 == 0) return;  // (no grid point in the sphere)
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, kl = lane >> 4;
  const cpx<R>* __restrict__ beta = reinterpret_cast<const cpx<R>*>(pt.beta);
  cpx<R> xn[KS];  // projector values of the wave's next row tile
  const auto load = [&](int rt) {
    const int row = rt * 16 + col;
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      const cpx<R> bv = beta[(size_t(2 * off) + min(row, K2 - 1)) * PP + 4 * u + kl];
      xn[u] = row < K2 ? bv : cpx<R>{R(0), R(0)};
    }
  };
  const int rt0 = blockIdx.z * (NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = nt * 16 + col;
  cpx<R> ec[KS];
  if constexpr (!SUMS) {
    if (rt0 * 16 >= K2) return;  // (one wave per workgroup, no barrier below)
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      const cpx<R> ev = EC[(size_t(a) * PP + 4 * u + kl) * S + min(i, S - 1)];
      ec[u] = i < S ? ev : cpx<R>{R(0), R(0)};
    }
  }
  load(rt0);
  if constexpr (SUMS) {
    constexpr int NC = 16 * PP / NT;  // coefficients per thread
    const int p = threadIdx.x >> 4, c16 = threadIdx.x & 15, ic = nt * 16 + c16;
    cpx<double> c[NC];
    proj_sums<NC>(pt, Cpart, S, dV, a, p, min(ic, S - 1), c);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const double en = pt.energy[size_t(a) * PP + p + 16 * k];
      ecs[p + 16 * k][c16] = ic < S ? cpx<R>{R(en * c[k].x), R(en * c[k].y)} : cpx<R>{R(0), R(0)};
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KS; ++u) ec[u] = ecs[4 * u + kl][col];
  }
  const cpx<R>* __restrict__ phase = nullptr;
  if constexpr (KQ) phase = ph.row<R>(min(i, S - 1), pt.Jtot);
  for (int rt = rt0; rt * 16 < K2; rt += gridDim.z * (NT / 64)) {
    cpx<R> xb[KS];
#pragma unroll
    for (int u = 0; u < KS; ++u) xb[u] = xn[u];
    load(rt + gridDim.z * (NT / 64));  // (past the last tile: its last row, dropped)
    typename M::acc yr = M::zero(), yi = M::zero();
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      yr = M::op(xb[u].x, ec[u].x, yr);
      yr = M::op(-xb[u].y, ec[u].y, yr);
      yi = M::op(xb[u].x, ec[u].y, yi);
      yi = M::op(xb[u].y, ec[u].x, yi);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = rt * 16 + M::row(r, kl);
      if (rr < K2 && i < S) {
        const int J = off + (rr >> 1), sp = rr & 1;
        cpx<R> y = {yr[r], yi[r]};
        if constexpr (KQ) y = cmulc(y, phase[J]);
        Y[size_t(2 * i + sp) * pt.Jtot + J] = y;
      }
    }
  }
}

// Phases exp(i (k + A).d) of every sphere row for each run of states.  The runs are counted from the last state's
// in device memory (last_run null: one run), not from the grid: a launch recorded into a graph fills the table for
// the Bloch vectors of the moment, which may be more runs than when it was recorded.
template <typename R>
__global__ __launch_bounds__(256) void k_phases(const double* __restrict__ kruns, const int* __restrict__ last_run,
                                                double a0, double a1, double a2, const R* __restrict__ disp, int Jtot,
                                                cpx<R>* __restrict__ out) {
  const int nruns = last_run ? *last_run + 1 : 1;
  for (int run = blockIdx.x; run < nruns; run += gridDim.x) {
    const double* k = kruns + 3 * size_t(run);
    for (int J = blockIdx.y * 256 + threadIdx.x; J < Jtot; J += gridDim.y * 256)
      out[size_t(run) * Jtot + J] = bloch_phase(R(k[0] + a0), R(k[1] + a1), R(k[2] + a2), disp + 3 * J);
  }
}

// ---------------------------------------------------------------- adjoint kernels
// Pair reduction of one adjoint Taylor stage w_k = x + c H w_{k-1} with adjoint mu_k:
//   g[0][p] += Re c sum_i mu_i^dagger w_i,  g[1+q][p] += Re c sum_i mu_i^dagger sigma_q w_i
// i.e. dL = sum_r (g_v dv + g_b . db) for a perturbation dH = dv + db.sigma of the stage.  FP64 takes any
// c = cre + i cim.  RE: with the real parts (FP64 always takes them, FP32 for c off the imaginary axis: Horner
// stages have c = -i gamma, cim = -gamma).
template <typename R, bool RE>
__global__ __launch_bounds__(256) void k_pair(const cpx<R>* __restrict__ mu, const cpx<R>* __restrict__ w,
                                              int S, size_t N, double cre, double cim, double* __restrict__ g) {
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= N) return;
  const double gamma = -cim;
  double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
  double t0 = 0, t1 = 0, t2 = 0, t3 = 0;  // real parts
#pragma unroll 2
  for (int i = 0; i < S; ++i) {
    const cpx<R> mu_u = mu[size_t(2 * i) * N + p], mu_d = mu[size_t(2 * i + 1) * N + p];
    const cpx<R> w_u = w[size_t(2 * i) * N + p], w_d = w[size_t(2 * i + 1) * N + p];
    const double ar = mu_u.x, ai = mu_u.y, br = mu_d.x, bi = mu_d.y;
    const double ur = w_u.x, ui = w_u.y, dr = w_d.x, di = w_d.y;
    // Im(conj(a) u) = ar ui - ai ur, Re(conj(a) u) = ar ur + ai ui
    const double im_au = ar * ui - ai * ur, im_bd = br * di - bi * dr;
    const double im_ad = ar * di - ai * dr, im_bu = br * ui - bi * ur;
    const double re_ad = ar * dr + ai * di, re_bu = br * ur + bi * ui;
    s0 += im_au + im_bd;                 // 1
    s1 += im_ad + im_bu;                 // sigma_x: conj(a) d + conj(b) u
    s2 += -re_ad + re_bu;                // sigma_y: -i conj(a) d + i conj(b) u  -> Im = -Re(a*d) + Re(b*u)
    s3 += im_au - im_bd;                 // sigma_z
    if constexpr (RE) {
      const double re_au = ar * ur + ai * ui, re_bd = br * dr + bi * di;
      t0 += re_au + re_bd;
      t1 += re_ad + re_bu;
      t2 += im_ad - im_bu;               // Re(-i a*d + i b*u) = Im(a*d) - Im(b*u)
      t3 += re_au - re_bd;
    }
  }
  if constexpr (RE) {
    g[p] += gamma * s0 + cre * t0;
    g[N + p] += gamma * s1 + cre * t1;
    g[2 * N + p] += gamma * s2 + cre * t2;
    g[3 * N + p] += gamma * s3 + cre * t3;
  } else {
    g[p] += gamma * s0;
    g[N + p] += gamma * s1;
    g[2 * N + p] += gamma * s2;
    g[3 * N + p] += gamma * s3;
  }
}

// Transpose of the field map (v, b) <- (n, m) at the density rho, for gradients g = (g_v, g_b):
//   g_n = P g_v + dvbar/dn g_v + dbeta/dn (mhat.g_b)
//   g_m = [dvbar/dmu g_v + dbeta/dmu (mhat.g_b)] mhat + (beta/mu)(g_b - mhat (mhat.g_b))
// with beta = (v_up - v_dn)/2, v_s' = -(1/3)(6/pi)^(1/3) n_s^(-2/3) (0 on a clamped channel),
// b_xc = 0 (and its derivatives) below the |m| threshold.  pg = P g_v (Poisson) or null.
// part[blk][0..2] = block sums of g_b (for dL/dB_ext).
static __global__ __launch_bounds__(256) void k_field_adjoint(const double* __restrict__ rho,
                                                       const double* __restrict__ g,
                                                       const double* __restrict__ pg, int xc,
                                                       double thr, size_t N, double* __restrict__ gnm,
                                                       double* __restrict__ part) {
  __shared__ double red[4];
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  double gbx = 0, gby = 0, gbz = 0;
  if (p < N) {
    const double gv = g[p];
    gbx = g[N + p];
    gby = g[2 * N + p];
    gbz = g[3 * N + p];
    double gn = pg ? pg[2 * p] : 0.0;  // real part of the complex Poisson output
    double gmx = 0, gmy = 0, gmz = 0;
    if (xc) {
      // v = vbar(n, |m|), b = bmag(n, |m|) m/|m| (|m| >= thr); with J the Jacobian of
      // (vbar, bmag) in (n, |m|) and g_r = mhat.g_b:
      //   g_n += J00 g_v + J10 g_r,  g_m = (J01 g_v + J11 g_r) mhat + (bmag/|m|)(g_b - mhat g_r)
      const double c = 1.2407009817988000;  // (6/pi)^(1/3)
      const double ruu = rho[p], rdd = rho[N + p], rr = rho[2 * N + p], ri = rho[3 * N + p];
      const double n = ruu + rdd, mx = 2.0 * rr, my = -2.0 * ri, mz = ruu - rdd;
      const double mu = sqrt(mx * mx + my * my + mz * mz);
      const double nu = 0.5 * (n + mu), nd = 0.5 * (n - mu);
      const double cu = nu > 0 ? cbrt(nu) : 0.0, cd = nd > 0 ? cbrt(nd) : 0.0;
      // exchange: v_s depends on n_s alone, dv_s/dn_s = du, dd
      const double du = nu > 0 ? -(c / 3.0) / (cu * cu) : 0.0;
      const double dd = nd > 0 ? -(c / 3.0) / (cd * cd) : 0.0;
      double j00 = 0.25 * (du + dd), j01 = 0.25 * (du - dd), j10 = j01, j11 = j00;
      double bmag = 0.0;
      if (mu >= thr) {
        const double nuc = fmax(nu, 0.0), ndc = fmax(nd, 0.0);
        const double den = cu * cu + cu * cd + cd * cd;
        bmag = den > 0.0 ? -0.5 * c * (nuc - ndc) / den : 0.0;
      }
      if (xc >= 2) {  // PW92 correlation: its Jacobian from two dual evaluations
        dnum vb, bm, ec;
        pw92_lc<dnum>(dnum{n, 1.0}, dnum{mu, 0.0}, vb, bm, ec);
        j00 += vb.d;
        j10 += bm.d;
        pw92_lc<dnum>(dnum{n, 0.0}, dnum{mu, 1.0}, vb, bm, ec);
        j01 += vb.d;
        j11 += bm.d;
        if (mu >= thr) bmag += bm.v;
      }
      gn += j00 * gv;
      if (mu >= thr) {
        const double hx = mx / mu, hy = my / mu, hz = mz / mu;
        const double mg = hx * gbx + hy * gby + hz * gbz;
        const double bom = bmag / mu;
        gn += j10 * mg;
        const double radial = j01 * gv + j11 * mg;
        gmx = radial * hx + bom * (gbx - hx * mg);
        gmy = radial * hy + bom * (gby - hy * mg);
        gmz = radial * hz + bom * (gbz - hz * mg);
      }
    }
    gnm[p] = gn;
    gnm[N + p] = gmx;
    gnm[2 * N + p] = gmy;
    gnm[3 * N + p] = gmz;
  }
  const double v3[3] = {gbx, gby, gbz};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double t = block_sum<256>(v3[k], red);
    if (threadIdx.x == 0) part[size_t(blockIdx.x) * 4 + k] = t;
  }
  if (threadIdx.x == 0) part[size_t(blockIdx.x) * 4 + 3] = 0.0;
}

// lam_i (+)= 2 f_i [g_n + g_m . sigma] psi_i   (adjoint of n = sum f psi^dag psi, m = sum f psi^dag sigma psi)
template <typename R>
__global__ __launch_bounds__(256) void k_density_backprop(const cpx<R>* __restrict__ psi,
                                                          const double* __restrict__ occ,
                                                          const double* __restrict__ gnm, int S,
                                                          size_t N, int add, cpx<R>* __restrict__ lam) {
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= size_t(S) * N) return;
  const int i = int(idx / N);
  const size_t p = idx - size_t(i) * N;
  const double f = 2.0 * occ[i];
  const double gn = gnm[p], gx = gnm[N + p], gy = gnm[2 * N + p], gz = gnm[3 * N + p];
  const cpx<R> u = psi[size_t(2 * i) * N + p], d = psi[size_t(2 * i + 1) * N + p];
  const double ux = u.x, uy = u.y, dx = d.x, dy = d.y;
  // up' = (gn + gz) u + (gx - i gy) d ; dn' = (gx + i gy) u + (gn - gz) d
  double ox = (gn + gz) * ux + gx * dx + gy * dy;
  double oy = (gn + gz) * uy + gx * dy - gy * dx;
  double px = gx * ux - gy * uy + (gn - gz) * dx;
  double py = gx * uy + gy * ux + (gn - gz) * dy;
  cpx<R>& lu = lam[size_t(2 * i) * N + p];
  cpx<R>& ld = lam[size_t(2 * i + 1) * N + p];
  if (add) {
    ox = f * ox + double(lu.x);
    oy = f * oy + double(lu.y);
    px = f * px + double(ld.x);
    py = f * py + double(ld.y);
  } else {
    ox *= f;
    oy *= f;
    px *= f;
    py *= f;
  }
  lu = {R(ox), R(oy)};
  ld = {R(px), R(py)};
}


// ---------------------------------------------------------------- observables row
// One workgroup; a wave takes one state at a time, its lanes the state's partial sums (one thread per state
// read them in a chain: 66 against 29 us for 96 states of 48^3, 8.0 against 5.0 for 8 of 16^3).
constexpr int OBS_NT = 1024;
static __global__ __launch_bounds__(OBS_NT) void k_obs_row(ObsInputs in, double* __restrict__ row) {
  constexpr int NW = OBS_NT / 64;
  __shared__ double red[NW];
  __shared__ double maxerr[NW];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  double ekin = 0.0, mx = 0.0, enl = 0.0;
  const int per = 2 * in.ntiles, perp = 2 * in.nplanes;  // of one state, both components
  for (int i = w; i < in.S; i += NW) {
    double e = 0.0, nn = 0.0;
    const double* q = in.epart + size_t(i) * per * 2;
    for (int t = lane; t < per; t += 64) {
      e += q[2 * t];
      nn += q[2 * t + 1];
    }
    for (int t = lane; t < perp; t += 64) e += in.eplane[size_t(i) * perp + t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nn += __shfl_xor(nn, o, 64);
    ekin += in.occ[i] * e * in.dV;  // (the lanes' shares)
    mx = fmax(mx, fabs(nn * in.invN * in.dV - 1.0));
  }
  if (in.C) {
    const size_t total = size_t(in.natoms) * in.PP * in.S;
    const cpx<double>* C = reinterpret_cast<const cpx<double>*>(in.C);
    for (size_t idx = tid; idx < total; idx += OBS_NT) {
      const int i = int(idx % in.S);
      const int p = int((idx / in.S) % in.PP);
      const int a = int(idx / (size_t(in.S) * in.PP));
      const cpx<double> c = C[idx];
      enl += in.occ[i] * in.energy[size_t(a) * in.PP + p] * (c.x * c.x + c.y * c.y);
    }
  }
  const double Ekin = block_sum<OBS_NT>(ekin, red);
  const double Enl = block_sum<OBS_NT>(enl, red);
  if (lane == 0) maxerr[w] = mx;
  __syncthreads();
  if (tid == 0) {
    double m = 0.0;
    for (int k = 0; k < NW; ++k) m = fmax(m, maxerr[k]);
    const double* ft = in.field_tot;
    const double dV = in.dV;
    const double Ne = ft[0] * dV, Mx = ft[1] * dV, My = ft[2] * dV, Mz = ft[3] * dV;
    const double Eloc = (ft[4] + in.efield[0] * ft[8] + in.efield[1] * ft[9] + in.efield[2] * ft[10]) * dV;
    const double EH = ft[5] * dV, Exc = ft[6] * dV;
    const double EZ = in.muB_B[0] * Mx + in.muB_B[1] * My + in.muB_B[2] * Mz;
    row[0] = in.t;
    row[1] = Ne;
    row[2] = Mx;
    row[3] = My;
    row[4] = Mz;
    row[5] = Ekin + Eloc + Enl + EH + Exc + EZ;
    row[6] = Ekin;
    row[7] = Eloc;
    row[8] = Enl;
    row[9] = EH;
    row[10] = Exc;
    row[11] = EZ;
    row[12] = m;
  }
}

// ---------------------------------------------------------------- small pointwise kernels
// lam_i = scale f_i (w . sigma) psi_i
template <typename R>
__global__ void k_seed(const cpx<R>* __restrict__ psi, const double* __restrict__ occ, int S,
                       size_t N, double w0, double w1, double w2, double scale,
                       cpx<R>* __restrict__ lam) {
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= size_t(S) * N) return;
  const int i = int(idx / N);
  const size_t p = idx - size_t(i) * N;
  const double f = scale * occ[i];
  const cpx<R> u = psi[size_t(2 * i) * N + p];
  const cpx<R> d = psi[size_t(2 * i + 1) * N + p];
  // (w.sigma) (u, d) = (w2 u + (w0 - i w1) d, (w0 + i w1) u - w2 d)
  const double ux = u.x, uy = u.y, dx = d.x, dy = d.y;
  const double ox = w2 * ux + w0 * dx + w1 * dy;
  const double oy = w2 * uy + w0 * dy - w1 * dx;
  const double px = w0 * ux - w1 * uy - w2 * dx;
  const double py = w0 * uy + w1 * ux - w2 * dy;
  lam[size_t(2 * i) * N + p] = {R(f * ox), R(f * oy)};
  lam[size_t(2 * i + 1) * N + p] = {R(f * px), R(f * py)};
}

// y = (a_re + i a_im) x + b y
template <typename R>
__global__ void k_axpby(cpx<R>* __restrict__ y, const cpx<R>* __restrict__ x, size_t count,
                        R are, R aim, R b) {
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= count) return;
  const cpx<R> xv = x[idx];
  const cpx<R> yv = y[idx];
  y[idx] = {are * xv.x - aim * xv.y + b * yv.x, are * xv.y + aim * xv.x + b * yv.y};
}

// rows[S][2][Jtot] *= exp(i dA.d_J)
template <typename R>
__global__ __launch_bounds__(256) void k_rephase_rows(cpx<R>* __restrict__ rows, const R* __restrict__ disp,
                                                      int Jtot, size_t total, R a0, R a1, R a2) {
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= total) return;
  const int J = int(p % size_t(Jtot));
  rows[p] = cmul(rows[p], bloch_phase(a0, a1, a2, disp + 3 * J));
}

// ---------------------------------------------------------------- initial spin-density matrix
static __global__ __launch_bounds__(256) void k_dm_init(int nx, int ny, int nz, double hx, double hy,
                                                 double hz, double Lx, double Ly, double Lz, int natoms,
                                                 const double* __restrict__ atoms,
                                                 const double* __restrict__ moments,
                                                 double* __restrict__ rho) {
  const size_t N = size_t(nx) * ny * nz;
  const size_t p = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= N) return;
  const size_t nyz = size_t(ny) * nz;
  const int ix = int(p / nyz);
  const int rem = int(p - size_t(ix) * nyz);
  const int iy = rem / nz, iz = rem - (rem / nz) * nz;
  const double r[3] = {ix * hx, iy * hy, iz * hz};
  const double L[3] = {Lx, Ly, Lz};
  double best = 1e300;
  int owner = 0;
  for (int a = 0; a < natoms; ++a) {
    double d2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double d = __dsub_rn(r[k], atoms[6 * a + k]);
      d = __dsub_rn(d, __dmul_rn(L[k], rint(d / L[k])));
      d2 = __dadd_rn(d2, __dmul_rn(d, d));
    }
    if (d2 < best) {
      best = d2;
      owner = a;
    }
  }
  const double Z = atoms[6 * owner + 3], sg = atoms[6 * owner + 4];
  const double n = Z * pow(2.0 * 3.14159265358979323846 * sg * sg, -1.5) * exp(-best / (2.0 * sg * sg));
  const double mx = moments[3 * owner] / Z, my = moments[3 * owner + 1] / Z, mz = moments[3 * owner + 2] / Z;
  rho[p] = n * (1.0 + mz) / 2.0;
  rho[N + p] = n * (1.0 - mz) / 2.0;
  rho[2 * N + p] = n * mx / 2.0;
  rho[3 * N + p] = -n * my / 2.0;
}

// ---------------------------------------------------------------- orthonormalisation (ground state)
// Overlap of a run of states and the triangular change of basis that orthonormalises them.  Both
// are dense complex contractions on the matrix cores with FP64 operands and FP64 accumulation in
// either precision (the overlap is a norm reduction over 2N terms).

// Partial Gram matrices over K-chunks: part[c][i][j] = sum_{k in chunk c} conj(A[i][k]) A[j][k]
// for the tile pairs (ti <= tj) of 32 x 32 state tiles; A is [S][K] (states are rows of K = 2N
// complex values).  Four waves per workgroup, one 16 x 16 output tile each (the one below the diagonal
// is left out).  Bound by the matrix cores, so the next KB values are loaded while this iteration's
// products run, into the other of two LDS tiles, with one barrier per iteration; the pairs of a chunk run on
// one XCD and find each other's rows in its L2.  At least four waves per SIMD are asked for: with more
// registers allowed, the compiler keeps the sums in accumulation registers and copies them back and forth
// every iteration.  96 states of 48^3 FP64: 223 against 239 us (9.5 GFLOP of products, 43 TFLOP/s).
constexpr int GRAM_T = 32;   // output tile (states)
constexpr int GRAM_KB = 16;  // k values staged per iteration
template <typename R>
__global__ __launch_bounds__(256, 4) void k_gram_partial(const cpx<R>* __restrict__ A, int S, size_t K,
                                                      size_t kchunk, cpx<double>* __restrict__ part) {
  using M = mfma16<double>;
  constexpr int E = GRAM_T * GRAM_KB / 256;
  __shared__ cpx<double> sa[2][GRAM_T][GRAM_KB + 1];
  __shared__ cpx<double> sb[2][GRAM_T][GRAM_KB + 1];
  const int T = (S + GRAM_T - 1) / GRAM_T;
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int chunk = L / (T * (T + 1) / 2);
  int pidx = L - chunk * (T * (T + 1) / 2), ti = 0;
  while (pidx >= T - ti) {
    pidx -= T - ti;
    ++ti;
  }
  const int tj = ti + pidx;
  const size_t k0 = size_t(chunk) * kchunk;
  const size_t k1 = min(K, k0 + kchunk);
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wi = w >> 1, wj = w & 1;
  const int c = lane & 15, kl = lane >> 4;
  const bool below = ti == tj && wi > wj;
  M::acc cr = M::zero(), ci = M::zero();
  cpx<R> va[E], vb[E];
  const auto load = [&](size_t kb) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int r = (tid + 256 * e) / GRAM_KB;
      const size_t k = kb + (tid + 256 * e) % GRAM_KB, kc = min(k, k1 - 1);
      // rows past the last state repeat it: their products are not stored
      va[e] = A[size_t(min(ti * GRAM_T + r, S - 1)) * K + kc];
      vb[e] = A[size_t(min(tj * GRAM_T + r, S - 1)) * K + kc];
      if (k >= k1) va[e] = vb[e] = {R(0), R(0)};
    }
  };
  load(k0);
  int buf = 0;
  for (size_t kb = k0; kb < k1; kb += GRAM_KB, buf ^= 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int r = (tid + 256 * e) / GRAM_KB, kk = (tid + 256 * e) % GRAM_KB;
      sa[buf][r][kk] = {double(va[e].x), double(va[e].y)};
      sb[buf][r][kk] = {double(vb[e].x), double(vb[e].y)};
    }
    __syncthreads();  // also: every wave is past the products of the other buffer, written next
    load(kb + GRAM_KB);  // (past the end: the last values again, dropped)
    if (!below) {
#pragma unroll
    for (int ks = 0; ks < GRAM_KB; ks += 4) {
      const cpx<double> a = sa[buf][wi * 16 + c][ks + kl];  // A operand: row i, column k
      const cpx<double> b = sb[buf][wj * 16 + c][ks + kl];  // B operand: row k, column j
      cr = M::op(a.x, b.x, cr);
      ci = M::op(a.x, b.y, ci);
      cr = M::op(a.y, b.y, cr);
      ci = M::op(-a.y, b.x, ci);
    }
    }
  }
  if (below) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = ti * GRAM_T + wi * 16 + M::row(r, kl);
    const int j = tj * GRAM_T + wj * 16 + c;
    if (i < S && j < S) part[(size_t(chunk) * S + i) * S + j] = {cr[r], ci[r]};
  }
}

// out[i][j] = scale sum_c part[c][i][j] for j >= i, and its conjugate at [j][i].  Sixteen entries per
// workgroup, sixteen threads each: thread q adds the chunks c = q mod 16 in order, then the sixteen
// sums are added in order (one thread per entry was a chain of up to 256 reads on few CUs: 79 against 6.4 us for
// 96 states).
constexpr int GRAM_RED = 16;
static __global__ __launch_bounds__(256) void k_gram_reduce(const cpx<double>* __restrict__ part, int S, int nchunks,
                                                     double scale, cpx<double>* __restrict__ out) {
  __shared__ cpx<double> sums[GRAM_RED][GRAM_RED];
  const int e = threadIdx.x % GRAM_RED, q = threadIdx.x / GRAM_RED;
  const size_t idx = size_t(blockIdx.x) * GRAM_RED + e;
  const int i = int(idx / S), j = int(idx - size_t(i) * S);
  const bool mine = idx < size_t(S) * S && j >= i;
  double sr = 0.0, si = 0.0;
  if (mine)
    for (int cch = q; cch < nchunks; cch += GRAM_RED) {
      const cpx<double> v = part[(size_t(cch) * S + i) * S + j];
      sr += v.x;
      si += v.y;
    }
  sums[q][e] = {sr, si};
  __syncthreads();
  if (q != 0 || !mine) return;
  for (int k = 1; k < GRAM_RED; ++k) {
    sr += sums[k][e].x;
    si += sums[k][e].y;
  }
  out[size_t(i) * S + j] = {scale * sr, scale * si};
  if (j != i) out[size_t(j) * S + i] = {scale * sr, -scale * si};
}

// D[j][p] = sum_{i <= j} Mt[i][j] A[i][p] (Mt upper triangular, FP64): the states D_j = sum_i
// A_i M_ij.  One workgroup: 64 states j x 64 columns p; wave w owns 16 columns and four 16-state MFMA
// tiles.  Bound by the matrix cores: a tile of states takes only the i up to its own last j, which costs
// every wave the same, since each holds all four tiles; the waves read A's columns straight
// into the operand layout (four rows of 256 bytes per load) and share Mt through LDS, and both are loaded
// one block of i ahead (96 states of 48^3 FP64: 226 against
// 426 us with 16 states per wave and every i of the workgroup's block; blocks of 16 i, which leave three
// waves per SIMD instead of four, and all states of a column block at once, whose four shares take
// unequal time, 7.08 against 6.20 ms with the overlap for 256 states of 64^3, which started at 7.54).
constexpr int BT_J = 64;
constexpr int BT_P = 64;
constexpr int BT_KI = 8;
template <typename R>
__global__ __launch_bounds__(256, 4) void k_basis_transform(const cpx<R>* __restrict__ A,
                                                         const cpx<double>* __restrict__ Mt, int S,
                                                         size_t K, cpx<R>* __restrict__ D) {
  using M = mfma16<double>;
  constexpr int E = BT_KI * BT_J / 256;
  __shared__ cpx<double> sm[2][BT_J][BT_KI + 1];   // [j][i]
  const int jblocks = (S + BT_J - 1) / BT_J, pblocks = int((K + BT_P - 1) / BT_P);
  const int jb = blockIdx.x / pblocks, pb = blockIdx.x - jb * pblocks;
  const int j0 = (jblocks - 1 - jb) * BT_J;  // the longest first
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int c = lane & 15, kl = lane >> 4;
  const size_t pp = size_t(pb) * BT_P + w * 16 + c;
  const size_t pr = min(pp, K - 1);
  M::acc dr[4], di[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    dr[h] = M::zero();
    di[h] = M::zero();
  }
  const int iend = min(S, j0 + BT_J);
  cpx<double> vm[E];
  cpx<R> va[BT_KI / 4];
  const auto load = [&](int i0) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = i0 + (tid + 256 * e) / BT_J, j = j0 + (tid + 256 * e) % BT_J;
      vm[e] = Mt[size_t(min(i, S - 1)) * S + min(j, S - 1)];  // (states j >= S are not stored)
      if (i >= S) vm[e] = {0.0, 0.0};
    }
#pragma unroll
    for (int q = 0; q < BT_KI / 4; ++q) {
      const int i = i0 + 4 * q + kl;
      va[q] = A[size_t(min(i, S - 1)) * K + pr];
      if (i >= S) va[q] = {R(0), R(0)};
    }
  };
  load(0);
  int buf = 0;
  for (int i0 = 0; i0 < iend; i0 += BT_KI, buf ^= 1) {
    cpx<R> b[BT_KI / 4];
#pragma unroll
    for (int q = 0; q < BT_KI / 4; ++q) b[q] = va[q];
#pragma unroll
    for (int e = 0; e < E; ++e) sm[buf][(tid + 256 * e) % BT_J][(tid + 256 * e) / BT_J] = vm[e];
    __syncthreads();  // also: every wave is past the products of the other buffer, written next
    load(i0 + BT_KI);  // (past the last state: zeros)
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      // (wave-uniform) Mt is zero there, or no such states
      if (i0 >= j0 + 16 * (h + 1) || j0 + 16 * h >= S) continue;
#pragma unroll
      for (int q = 0; q < BT_KI / 4; ++q) {
        const cpx<double> a = sm[buf][h * 16 + c][4 * q + kl];  // A operand: row j, column i
        const double bx = double(b[q].x), by = double(b[q].y);  // B operand: row i, column p
        dr[h] = M::op(a.x, bx, dr[h]);
        di[h] = M::op(a.x, by, di[h]);
        dr[h] = M::op(-a.y, by, dr[h]);
        di[h] = M::op(a.y, bx, di[h]);
      }
    }
  }
  if (pp >= K) return;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = j0 + h * 16 + M::row(r, kl);
      if (j < S) D[size_t(j) * K + pp] = {R(dr[h][r]), R(di[h][r])};
    }
  }
}

// ---------------------------------------------------------------- static scratch
// Temporaries of the allocation-free entry point.  Host code never passes this name to a kernel:
// it takes the per-device address from static_scratch().
#if NCT_FP64_TU
static __device__ __align__(256) unsigned char scratch[NCT_STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {  // once per device, with that device current
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = NCT_STATIC_SCRATCH_BYTES;
  return hipSuccess;
}
#endif

// ================================================================ launchers
static inline unsigned nblocks(size_t n, unsigned bs) { return unsigned((n + bs - 1) / bs); }

#if NCT_FP64_TU
LaunchEvents& launch_events() {
  static thread_local LaunchEvents ev;
  return ev;
}
#endif

// Every dispatch goes through here: with timing events pending they ride on the dispatch itself.
template <typename F, typename... Args>
static void nct_launch(F kern, dim3 grid, dim3 block, size_t lds, hipStream_t st, Args... args) {
  LaunchEvents& ev = launch_events();
  if (ev.stop) {
    hipExtLaunchKernelGGL(kern, grid, block, std::uint32_t(lds), st, ev.used ? nullptr : ev.start,
                          ev.stop, 0u, args...);
    ev.used = true;
  } else {
    hipLaunchKernelGGL(kern, grid, block, lds, st, args...);
  }
}

#ifndef NCT_PLANE_PAIRS
#define NCT_PLANE_PAIRS(X) \
  X(8, 8) X(12, 12) X(16, 16) X(24, 24) X(32, 32) X(48, 48) X(64, 64) X(96, 96) \
  X(8, 16) X(16, 8) X(12, 16) X(16, 12) X(16, 24) X(24, 16)
#define NCT_LINES(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96)
#endif

#if NCT_FP64_TU
bool real_base_in_plane(int ny, int nz, bool fp64) {
  return fp64 ? plane_takes_base<double>(ny, nz) : plane_takes_base<float>(ny, nz);
}
bool plane_pair_supported(int ny, int nz) {
#define X(a, b) if (ny == a && nz == b) return true;
  NCT_PLANE_PAIRS(X)
#undef X
  return false;
}
bool line_supported(int n) {
#define X(a) if (n == a) return true;
  NCT_LINES(X)
#undef X
  return false;
}
#endif

template <typename K>
static hipError_t set_lds(K kern, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

// ---- real-space form
template <typename R, int A, int B, int M, bool ACC>
static hipError_t launch_plane_yz_m(int S, int NX, const StageArgs<R>& a, const KinTables& kt,
                                    const ProjTables& pt, const void* twy, const void* twz, hipStream_t st) {
  constexpr size_t lds = real_lds_bytes<R, A, B>();
  auto kern = k_plane_yz<R, A, B, M, ACC>;
  hipError_t e = set_lds(kern, lds);
  if (e != hipSuccess) return e;
  nct_launch(kern, dim3(2u * unsigned(S) * unsigned(NX)), dim3(64 * real_nw<R>(A, B)), lds, st, a, kt, pt,
             reinterpret_cast<const cpx<R>*>(twy), reinterpret_cast<const cpx<R>*>(twz), 2 * S, NX);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_plane_yz(const int n[3], int S, const StageArgs<R>& a, const KinTables& kt,
                           const ProjTables& pt, const void* twy, const void* twz, hipStream_t st) {
  // accumulation is for the adjoint, which takes this form in FP32 only for large states (cache mode 2)
  constexpr bool D = sizeof(R) == 8;
  if (a.acc && !D && a.cache_mode < 2) return hipErrorInvalidValue;
#define Y(A, B, M)                                                                             \
  return a.acc ? launch_plane_yz_m<R, A, B, M, D || M == 2>(S, n[0], a, kt, pt, twy, twz, st)  \
               : launch_plane_yz_m<R, A, B, M, false>(S, n[0], a, kt, pt, twy, twz, st)
#define X(A, B)                          \
  if (n[1] == A && n[2] == B) {          \
    if (a.cache_mode >= 2) Y(A, B, 2);   \
    if constexpr (!D) {                  \
      if (a.cache_mode == 1) Y(A, B, 1); \
    }                                    \
    Y(A, B, 0);                          \
  }
  NCT_PLANE_PAIRS(X)
#undef X
#undef Y
  return hipErrorInvalidValue;
}

template <typename R>
hipError_t launch_gather_rows(const ProjTables& pt, const void* psi, void* W, int B, size_t N, hipStream_t st) {
  if (pt.natoms == 0 || pt.Jtot == 0) return hipSuccess;
  nct_launch(k_gather_rows<R>, dim3(unsigned(B), tables::row_blocks(pt.Jtot, 256)), dim3(256), 0, st,
             reinterpret_cast<const cpx<R>*>(psi), reinterpret_cast<cpx<R>*>(W), pt, N);
  return hipGetLastError();
}

template <typename R, int NX, int CW, int PAIRS, int M>
static hipError_t launch_xv_m(const int n[3], int S, const StageArgs<R>& a, void* dst, const void* twx,
                              const KinTables& kt, hipStream_t st) {
  const dim3 grid(unsigned(n[1] * n[2] / (CW * PAIRS)) * unsigned(S)), block(128 * PAIRS);
  const auto d_ = reinterpret_cast<cpx<R>*>(dst);
  const auto t_ = reinterpret_cast<const cpx<R>*>(twx);
  if (a.x_base && a.x_base != a.w_in) nct_launch((k_xv<R, NX, CW, PAIRS, M, true>), grid, block, 0, st, a, d_, n[1], n[2], S, t_, kt);
  else nct_launch((k_xv<R, NX, CW, PAIRS, M, false>), grid, block, 0, st, a, d_, n[1], n[2], S, t_, kt);
  return hipGetLastError();
}
template <typename R, int NX, int CW, int PAIRS>
static hipError_t launch_xv_p(const int n[3], int S, const StageArgs<R>& a, void* dst, const void* twx,
                              const KinTables& kt, hipStream_t st) {
  if (a.cache_mode >= 2) return launch_xv_m<R, NX, CW, PAIRS, 2>(n, S, a, dst, twx, kt, st);
  if constexpr (sizeof(R) == 4) {  // FP64 has no streaming stores with plain loads
    if (a.cache_mode == 1) return launch_xv_m<R, NX, CW, PAIRS, 1>(n, S, a, dst, twx, kt, st);
  }
  return launch_xv_m<R, NX, CW, PAIRS, 0>(n, S, a, dst, twx, kt, st);
}
template <typename R>
hipError_t launch_xv(const int n[3], int S, const StageArgs<R>& a, void* dst, const void* twx,
                     const KinTables& kt, hipStream_t st) {
  // every built plane holds a multiple of 16 columns
#define X(A)                                                                             \
  if (n[0] == A) {                                                                       \
    constexpr int CW = xv_cols<R>(A), P = xv_pairs(A);                                      \
    const int cols = n[1] * n[2];                                                           \
    const bool two = A >= 48 || size_t(cols / (2 * CW)) * S >= kXvTwoBlocksMin;             \
    if (two && cols % (P * CW) == 0) return launch_xv_p<R, A, CW, P>(n, S, a, dst, twx, kt, st); \
    if constexpr (P > 2)                                                                    \
      if (cols % (2 * CW) == 0) return launch_xv_p<R, A, CW, 2>(n, S, a, dst, twx, kt, st); \
    if constexpr (CW > 16)                                                                  \
      if (cols % CW != 0) return launch_xv_p<R, A, 16, 1>(n, S, a, dst, twx, kt, st);       \
    if constexpr (P > 1) return launch_xv_p<R, A, CW, 1>(n, S, a, dst, twx, kt, st);        \
  }
  NCT_LINES(X)
#undef X
  return hipErrorInvalidValue;
}

#if NCT_FP64_TU
hipError_t launch_energy_real(const int n[3], int B, const void* src, const void* twx, const void* twy,
                              const void* twz, const KinTables& kt, double* part, double* eplane, int* ntiles_out,
                              hipStream_t st) {
  const int NYZ = n[1] * n[2];
  const auto s_ = reinterpret_cast<const cpx<double>*>(src);
  const auto t_ = reinterpret_cast<const cpx<double>*>(twx);
  hipError_t e = hipErrorInvalidValue;
#define X(A)                                                                                       \
  if (n[0] == A) {                                                                                 \
    constexpr int TC = xpass_tc<double>(A);                                                        \
    const int tc = NYZ % TC == 0 ? TC : 16;                                                        \
    *ntiles_out = NYZ / tc;                                                                        \
    const dim3 grid(unsigned(B) * unsigned(NYZ / tc));                                             \
    if (tc == TC) nct_launch((k_xkin_energy<A, TC>), grid, dim3(256), 0, st, s_, NYZ, t_, part, kt); \
    else nct_launch((k_xkin_energy<A, 16>), grid, dim3(256), 0, st, s_, NYZ, t_, part, kt);        \
    e = hipGetLastError();                                                                         \
  }
  NCT_LINES(X)
#undef X
  if (e != hipSuccess) return e;
#define X(A, BB)                                                                                   \
  if (n[1] == A && n[2] == BB) {                                                                   \
    constexpr size_t lds = plane_lds_bytes<A, BB>(sizeof(cpx<double>));                            \
    auto kern = k_plane_energy<A, BB>;                                                             \
    e = set_lds(kern, lds);                                                                        \
    if (e != hipSuccess) return e;                                                                 \
    nct_launch(kern, dim3(unsigned(B) * unsigned(n[0])), dim3(plane_nt(A * BB)), lds, st, s_,      \
               reinterpret_cast<const cpx<double>*>(twy), reinterpret_cast<const cpx<double>*>(twz), B, n[0], \
               eplane, kt);                                                                        \
    return hipGetLastError();                                                                      \
  }
  NCT_PLANE_PAIRS(X)
#undef X
  return hipErrorInvalidValue;
}
#else
// ---- transformed form (FP32)
template <typename R, int A, int B, int M>
static hipError_t launch_plane_stage_m(int S, int NX, const StageArgs<R>& a, const ProjTables& pt,
                                       const void* twy, const void* twz, hipStream_t st) {
  const unsigned grid = unsigned(S) * unsigned(NX);
  const auto ty = reinterpret_cast<const cpx<R>*>(twy);
  const auto tz = reinterpret_cast<const cpx<R>*>(twz);
  if constexpr (planer_use<R, A, B>()) {
    constexpr size_t ldsr = planer_lds_bytes<R, A, B>();
    auto kernr = k_plane_stage_r<R, A, B, M>;
    hipError_t er = set_lds(kernr, ldsr);
    if (er != hipSuccess) return er;
    nct_launch(kernr, dim3(grid), dim3(NCT_PLANER_NT), ldsr, st, a, pt, ty, tz, S, NX);
  } else {
    constexpr size_t lds2 = plane2_lds_bytes<A, B>(sizeof(cpx<R>));
    auto kern2 = k_plane_stage2<R, A, B, M>;
    hipError_t e2 = set_lds(kern2, lds2);
    if (e2 != hipSuccess) return e2;
    nct_launch(kern2, dim3(grid), dim3(2 * plane2_nth<R>(A * B)), lds2, st, a, pt, ty, tz, S, NX);
  }
  return hipGetLastError();
}

hipError_t launch_plane_stage(const int n[3], int S, const StageArgs<float>& a, const ProjTables& pt,
                              const void* twy, const void* twz, hipStream_t st) {
#define X(A, B)                                                                              \
  if (n[1] == A && n[2] == B) {                                                              \
    if (a.cache_mode >= 2) return launch_plane_stage_m<float, A, B, 2>(S, n[0], a, pt, twy, twz, st); \
    if (a.cache_mode == 1) return launch_plane_stage_m<float, A, B, 1>(S, n[0], a, pt, twy, twz, st); \
    return launch_plane_stage_m<float, A, B, 0>(S, n[0], a, pt, twy, twz, st);              \
  }
  NCT_PLANE_PAIRS(X)
#undef X
  return hipErrorInvalidValue;
}
#endif

#if !NCT_FP64_TU
template <typename R>
hipError_t launch_plane_fwd(const int n[3], int B, const void* in, void* out, void* W,
                            const ProjTables* pt, const void* twy, const void* twz, hipStream_t st,
                            KTables<R> kt) {
  const unsigned grid = unsigned(B) * unsigned(n[0]);
  ProjTables none;
  const ProjTables& p = pt ? *pt : none;
#define X(A, BB)                                                                            \
  if (n[1] == A && n[2] == BB) {                                                            \
    constexpr size_t lds = plane_lds_bytes<A, BB>(sizeof(cpx<R>));                          \
    auto kern = k_plane_fwd<R, A, BB>;                                                      \
    hipError_t e = set_lds(kern, lds);                                                      \
    if (e != hipSuccess) return e;                                                          \
    nct_launch(kern, dim3(grid), dim3(plane_nt(A * BB)), lds, st,                   \
                       reinterpret_cast<const cpx<R>*>(in), reinterpret_cast<cpx<R>*>(out),  \
                       reinterpret_cast<cpx<R>*>(W), p,                                     \
                       reinterpret_cast<const cpx<R>*>(twy), reinterpret_cast<const cpx<R>*>(twz), \
                       B, n[0], kt);                                                        \
    return hipGetLastError();                                                               \
  }
  NCT_PLANE_PAIRS(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_plane_fwd_real(const int n[3], const double* in, int src, void* out, const void* twy,
                                 const void* twz, hipStream_t st) {
  const unsigned grid = unsigned(n[0]);
#define X(A, BB)                                                                            \
  if (n[1] == A && n[2] == BB) {                                                            \
    constexpr size_t lds = plane_lds_bytes<A, BB>(sizeof(cpx<double>));                     \
    auto kern = src == 1 ? k_plane_fwd<double, A, BB, 1> : k_plane_fwd<double, A, BB, 2>;  \
    hipError_t e = set_lds(kern, lds);                                                      \
    if (e != hipSuccess) return e;                                                          \
    nct_launch(kern, dim3(grid), dim3(plane_nt(A * BB)), lds, st,                            \
               reinterpret_cast<const cpx<double>*>(in), reinterpret_cast<cpx<double>*>(out), \
               static_cast<cpx<double>*>(nullptr), ProjTables{},                             \
               reinterpret_cast<const cpx<double>*>(twy), reinterpret_cast<const cpx<double>*>(twz), \
               1, n[0], KTables<double>{});                                                  \
    return hipGetLastError();                                                               \
  }
  NCT_PLANE_PAIRS(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_dm_init(const int n[3], const double cell[3], int natoms, const double* atoms,
                          const double* moments, double* rho, hipStream_t st) {
  const size_t N = size_t(n[0]) * n[1] * n[2];
  nct_launch(k_dm_init, dim3(nblocks(N, 256)), dim3(256), 0, st, n[0], n[1], n[2], cell[0] / n[0],
             cell[1] / n[1], cell[2] / n[2], cell[0], cell[1], cell[2], natoms, atoms, moments, rho);
  return hipGetLastError();
}
#endif

#if !NCT_FP64_TU
template <typename R>
hipError_t launch_rephase_rows(const ProjTables& pt, void* rows, int S, const double dA[3],
                               hipStream_t st) {
  if (pt.natoms == 0 || pt.Jtot == 0) return hipSuccess;
  const size_t total = size_t(S) * 2 * pt.Jtot;
  nct_launch(k_rephase_rows<R>, dim3(nblocks(total, 256)), dim3(256), 0, st,
             reinterpret_cast<cpx<R>*>(rows), reinterpret_cast<const R*>(pt.disp), pt.Jtot, total,
             R(dA[0]), R(dA[1]), R(dA[2]));
  return hipGetLastError();
}
#endif

template <typename R>
hipError_t launch_plane_inv(const int n[3], int B, const void* in, void* out, R scale,
                            const void* twy, const void* twz, hipStream_t st) {
  const unsigned grid = unsigned(B) * unsigned(n[0]);
#define X(A, BB)                                                                            \
  if (n[1] == A && n[2] == BB) {                                                            \
    constexpr size_t lds = plane_lds_bytes<A, BB>(sizeof(cpx<R>));                          \
    auto kern = k_plane_inv<R, A, BB>;                                                      \
    hipError_t e = set_lds(kern, lds);                                                      \
    if (e != hipSuccess) return e;                                                          \
    nct_launch(kern, dim3(grid), dim3(plane_nt(A * BB)), lds, st,                   \
                       reinterpret_cast<const cpx<R>*>(in), reinterpret_cast<cpx<R>*>(out),  \
                       scale, reinterpret_cast<const cpx<R>*>(twy),                         \
                       reinterpret_cast<const cpx<R>*>(twz), B, n[0]);                      \
    return hipGetLastError();                                                               \
  }
  NCT_PLANE_PAIRS(X)
#undef X
  return hipErrorInvalidValue;
}

template <typename R, int NX, int TC>
static hipError_t launch_xpass_tc(int B, int NYZ, const void* src, void* dst, const R* g2x, const R* g2yz,
                                  R kscale, int mode, const void* twx, int cache_mode, hipStream_t st,
                                  KTables<R> kt) {
  const int tiles = NYZ / TC;
  const auto s_ = reinterpret_cast<const cpx<R>*>(src);
  const auto d_ = reinterpret_cast<cpx<R>*>(dst);
  const auto t_ = reinterpret_cast<const cpx<R>*>(twx);
  // one tile per workgroup (a second, prefetched tile per workgroup measured no faster on
  // MI355X and costs occupancy)
  const dim3 grid(unsigned(B) * unsigned(tiles));
  if constexpr (sizeof(R) == 4) {  // FP64 only runs the Poisson solve here: plain accesses
    if (cache_mode >= 2) {
      nct_launch((k_xpass<R, NX, TC, 2>), grid, dim3(xp_nt<R, NX, TC>()), 0, st, s_, d_, NYZ, g2x, g2yz, kscale, mode, t_, kt);
      return hipGetLastError();
    }
    if (cache_mode == 1) {
      nct_launch((k_xpass<R, NX, TC, 1>), grid, dim3(xp_nt<R, NX, TC>()), 0, st, s_, d_, NYZ, g2x, g2yz, kscale, mode, t_, kt);
      return hipGetLastError();
    }
  }
  nct_launch((k_xpass<R, NX, TC, 0>), grid, dim3(xp_nt<R, NX, TC>()), 0, st, s_, d_, NYZ, g2x, g2yz, kscale, mode, t_, kt);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_xpass(const int n[3], int B, const void* src, void* dst, const R* g2x,
                        const R* g2yz, R kscale, int mode, const void* twx, hipStream_t st,
                        int cache_mode, KTables<R> kt) {
  const int NYZ = n[1] * n[2];
#define X(A)                                                                                \
  if (n[0] == A) {                                                                          \
    constexpr int TCP = xpass_tc<R>(A);                                                     \
    if (NYZ % TCP == 0)                                                                     \
      return launch_xpass_tc<R, A, TCP>(B, NYZ, src, dst, g2x, g2yz, kscale, mode, twx, cache_mode, st, kt); \
    return launch_xpass_tc<R, A, 16>(B, NYZ, src, dst, g2x, g2yz, kscale, mode, twx, cache_mode, st, kt); \
  }
  NCT_LINES(X)
#undef X
  return hipErrorInvalidValue;
}

#if !NCT_FP64_TU
template <typename R>
hipError_t launch_xpass_energy(const int n[3], int B, const void* src, const R* g2x,
                               const R* g2yz, R kscale, const void* twx, double* part,
                               int* ntiles_out, hipStream_t st, KTables<R> kt) {
  const int NYZ = n[1] * n[2];
#define X(A)                                                                                \
  if (n[0] == A) {                                                                          \
    constexpr int TCP = xpass_tc<R>(A);                                                     \
    if (NYZ % TCP == 0) {                                                                   \
      *ntiles_out = NYZ / TCP;                                                              \
      nct_launch((k_xpass_energy<R, A, TCP>), dim3(unsigned(B) * unsigned(NYZ / TCP)), \
                         dim3(XP_NT), 0, st, reinterpret_cast<const cpx<R>*>(src), NYZ, g2x,  \
                         g2yz, kscale, reinterpret_cast<const cpx<R>*>(twx), part, kt);      \
    } else {                                                                                \
      *ntiles_out = NYZ / 16;                                                               \
      nct_launch((k_xpass_energy<R, A, 16>), dim3(unsigned(B) * unsigned(NYZ / 16)),  \
                         dim3(XP_NT), 0, st, reinterpret_cast<const cpx<R>*>(src), NYZ, g2x,  \
                         g2yz, kscale, reinterpret_cast<const cpx<R>*>(twx), part, kt);      \
    }                                                                                       \
    return hipGetLastError();                                                               \
  }
  NCT_LINES(X)
#undef X
  return hipErrorInvalidValue;
}
#endif

template <typename R>
hipError_t launch_density(const void* psi, const double* occ, int S, size_t N, double* rho,
                          hipStream_t st) {
  nct_launch((k_density<R>), dim3(nblocks(N, 256)), dim3(256), 0, st,
                     reinterpret_cast<const cpx<R>*>(psi), occ, S, N, rho);
  return hipGetLastError();
}

#if NCT_FP64_TU
hipError_t launch_fields(const double* rho, const double* vext, const double* vH, int xc,
                         double thr, const int n[3], const double cell[3], double* fields,
                         float* fields32, double* part, int* nblk_out, hipStream_t st) {
  const size_t N = size_t(n[0]) * n[1] * n[2];
  const unsigned nb = nblocks(N, 256);
  *nblk_out = int(nb);
  nct_launch(k_fields, dim3(nb), dim3(256), 0, st, rho, vext, vH, xc, thr, n[1], n[2],
                     cell[0] / n[0], cell[1] / n[1], cell[2] / n[2], 0.5 * cell[0], 0.5 * cell[1],
                     0.5 * cell[2], N, fields, fields32, part);
  return hipGetLastError();
}

hipError_t launch_reduce_rows(const double* part, int nrows, int width, double* out,
                              hipStream_t st, double* copy0) {
  nct_launch(k_reduce_rows, dim3(unsigned(width)), dim3(256), 0, st, part, nrows, width, out, copy0);
  return hipGetLastError();
}
hipError_t launch_add_bext(const double* fields, const int n[3], const double b[3],
                           const double lg[4], double* out, hipStream_t st) {
  const size_t N = size_t(n[0]) * n[1] * n[2];
  nct_launch(k_add_bext, dim3(nblocks(N, 256)), dim3(256), 0, st, fields, n[1], n[2], N,
                     b[0], b[1], b[2], lg[0], lg[1], lg[2], lg[3], out);
  return hipGetLastError();
}
hipError_t launch_to_float(const double* in, size_t n, float* out, hipStream_t st) {
  nct_launch(k_to_float, dim3(nblocks(n, 256)), dim3(256), 0, st, in, n, out);
  return hipGetLastError();
}
#endif

template <typename R, int PP, bool KQ>
static hipError_t launch_contract_pp(const ProjTables& pt, const void* W, int S, void* Cpart, const PhaseTab& ph,
                                     hipStream_t st) {
  const dim3 grid(pt.natoms, unsigned((S + 15) / 16), pt.max_kchunks);
  nct_launch((k_proj_contract<R, PP, KQ>), grid, dim3(64), 0, st, pt, reinterpret_cast<const cpx<R>*>(W), S,
             reinterpret_cast<cpx<double>*>(Cpart), ph);
  return hipGetLastError();
}
template <typename R>
hipError_t launch_proj_contract(const ProjTables& pt, const void* W, int S, void* Cpart, const PhaseTab& ph,
                                hipStream_t st) {
  if (pt.natoms == 0) return hipSuccess;
  if (ph.tab)
    return pt.PP == 16 ? launch_contract_pp<R, 16, true>(pt, W, S, Cpart, ph, st)
                       : launch_contract_pp<R, 32, true>(pt, W, S, Cpart, ph, st);
  return pt.PP == 16 ? launch_contract_pp<R, 16, false>(pt, W, S, Cpart, ph, st)
                     : launch_contract_pp<R, 32, false>(pt, W, S, Cpart, ph, st);
}
#if NCT_FP64_TU
hipError_t launch_proj_reduce(const ProjTables& pt, const void* Cpart, int S, double dV, void* C, hipStream_t st) {
  if (pt.natoms == 0) return hipSuccess;
  nct_launch(k_proj_reduce, dim3(nblocks(size_t(pt.natoms) * pt.PP * S, 256)), dim3(256), 0, st, pt,
             reinterpret_cast<const cpx<double>*>(Cpart), S, dV, reinterpret_cast<cpx<double>*>(C));
  return hipGetLastError();
}
#endif
template <typename R>
hipError_t launch_phases(const double* kruns, const int* last_run, int nruns, const double ka[3], const ProjTables& pt,
                         void* tab, hipStream_t st) {
  if (pt.natoms == 0 || pt.Jtot == 0) return hipSuccess;
  nct_launch(k_phases<R>, dim3(unsigned(nruns), tables::row_blocks(pt.Jtot, 256)), dim3(256), 0, st, kruns, last_run, ka[0],
             ka[1], ka[2], reinterpret_cast<const R*>(pt.disp), pt.Jtot, reinterpret_cast<cpx<R>*>(tab));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_proj_coeffs(const ProjTables& pt, const void* Cpart, int S, double dV, void* EC, hipStream_t st) {
  if (pt.natoms == 0) return hipSuccess;
  nct_launch(k_proj_coeffs<R>, dim3(nblocks(size_t(pt.natoms) * pt.PP * S, 256)), dim3(256), 0, st, pt,
             reinterpret_cast<const cpx<double>*>(Cpart), S, dV, reinterpret_cast<cpx<R>*>(EC));
  return hipGetLastError();
}

template <typename R, int PP, bool KQ, bool SUMS>
static hipError_t launch_scatter_pp(const ProjTables& pt, const void* Cpart, const void* EC, int S, double dV, void* Y,
                                    const PhaseTab& ph, hipStream_t st) {
  constexpr int NT = ps_nt<R, PP, SUMS>(), waves = NT / 64;
  const int ntile = (S + 15) / 16;
  // Shares of an atom's row tiles.  With the coefficients made: two tiles per wave (48^3 x 64 mixed with four atoms
  // 2.00 ms per step, 32^3 x 64 FP64 1.05; with eight 2.06 and 1.16; one per wave 64^3 x 256 mixed with 16 atoms 13.64
  // against 13.59).  With the sums in here, which every share repeats: one tile per wave where there
  // are few (atom, states) pairs, up to 512 workgroups (96 x 24 x 24 x 40 mixed 0.80 ms per step, 0.83 with 128).
  const int shares = SUMS ? std::max(1, std::min((pt.max_rowtiles + waves - 1) / waves, 512 / (pt.natoms * ntile)))
                          : std::max(1, (pt.max_rowtiles + 1) / 2);
  const dim3 grid(pt.natoms, unsigned(ntile), unsigned(shares));
  nct_launch((k_proj_scatter<R, PP, KQ, SUMS>), grid, dim3(unsigned(NT)), 0, st, pt,
             reinterpret_cast<const cpx<double>*>(Cpart), reinterpret_cast<const cpx<R>*>(EC), S, dV,
             reinterpret_cast<cpx<R>*>(Y), ph);
  return hipGetLastError();
}
template <typename R, bool SUMS>
static hipError_t launch_scatter_k(const ProjTables& pt, const void* Cpart, const void* EC, int S, double dV, void* Y,
                                   const PhaseTab& ph, hipStream_t st) {
  if (ph.tab)
    return pt.PP == 16 ? launch_scatter_pp<R, 16, true, SUMS>(pt, Cpart, EC, S, dV, Y, ph, st)
                       : launch_scatter_pp<R, 32, true, SUMS>(pt, Cpart, EC, S, dV, Y, ph, st);
  return pt.PP == 16 ? launch_scatter_pp<R, 16, false, SUMS>(pt, Cpart, EC, S, dV, Y, ph, st)
                     : launch_scatter_pp<R, 32, false, SUMS>(pt, Cpart, EC, S, dV, Y, ph, st);
}
template <typename R>
hipError_t launch_proj_scatter(const ProjTables& pt, const void* Cpart, const void* EC, int S, double dV, void* Y,
                               const PhaseTab& ph, hipStream_t st) {
  if (pt.natoms == 0) return hipSuccess;
  return EC ? launch_scatter_k<R, false>(pt, Cpart, EC, S, dV, Y, ph, st)
            : launch_scatter_k<R, true>(pt, Cpart, EC, S, dV, Y, ph, st);
}

#if NCT_FP64_TU
int gram_chunks(int S, size_t K) {
  const int T = (S + GRAM_T - 1) / GRAM_T;
  const size_t pairs = size_t(T) * (T + 1) / 2;
  size_t nc = std::max<size_t>(1, 1024 / pairs);                       // the four per CU that run at once
  nc = std::min<size_t>(nc, 512);
  nc = std::min<size_t>(nc, std::max<size_t>(1, (size_t(64) << 20) / (size_t(S) * S * 16)));  // partials <= 64 MiB
  nc = std::min<size_t>(nc, std::max<size_t>(1, K / (4 * GRAM_KB)));   // chunks of >= 64 values
  return int(std::max<size_t>(nc, 1));
}
#endif

template <typename R>
hipError_t launch_gram(const void* A, int S, size_t K, double scale, void* part, int nchunks, void* out,
                       hipStream_t st) {
  if (S <= 0 || nchunks <= 0) return hipErrorInvalidValue;
  const int T = (S + GRAM_T - 1) / GRAM_T;
  const unsigned pairs = unsigned(T) * unsigned(T + 1) / 2;
  size_t kchunk = (K + nchunks - 1) / nchunks;
  kchunk = (kchunk + GRAM_KB - 1) / GRAM_KB * GRAM_KB;
  const unsigned used = unsigned((K + kchunk - 1) / kchunk);
  nct_launch((k_gram_partial<R>), dim3(pairs * used), dim3(256), 0, st, reinterpret_cast<const cpx<R>*>(A), S, K,
             kchunk, reinterpret_cast<cpx<double>*>(part));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  nct_launch(k_gram_reduce, dim3(nblocks(size_t(S) * S, GRAM_RED)), dim3(256), 0, st,
             reinterpret_cast<const cpx<double>*>(part), S, int(used), scale, reinterpret_cast<cpx<double>*>(out));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_basis_transform(const void* A, const void* Mt, int S, size_t K, void* D, hipStream_t st) {
  if (S <= 0) return hipErrorInvalidValue;
  const dim3 grid(unsigned((K + BT_P - 1) / BT_P) * unsigned((S + BT_J - 1) / BT_J));
  nct_launch((k_basis_transform<R>), grid, dim3(256), 0, st, reinterpret_cast<const cpx<R>*>(A),
             reinterpret_cast<const cpx<double>*>(Mt), S, K, reinterpret_cast<cpx<R>*>(D));
  return hipGetLastError();
}

#if NCT_FP64_TU
hipError_t launch_obs_row(const ObsInputs& in, double* row, hipStream_t st) {
  nct_launch(k_obs_row, dim3(1), dim3(OBS_NT), 0, st, in, row);
  return hipGetLastError();
}
#endif

template <typename R>
hipError_t launch_seed(const void* psi, const double* occ, int S, size_t N, double w0, double w1,
                       double w2, double scale, void* lam, hipStream_t st) {
  nct_launch((k_seed<R>), dim3(nblocks(size_t(S) * N, 256)), dim3(256), 0, st,
                     reinterpret_cast<const cpx<R>*>(psi), occ, S, N, w0, w1, w2, scale,
                     reinterpret_cast<cpx<R>*>(lam));
  return hipGetLastError();
}
template <typename R>
hipError_t launch_axpby(void* y, const void* x, size_t count, R a_re, R a_im, R b,
                        hipStream_t st) {
  nct_launch((k_axpby<R>), dim3(nblocks(count, 256)), dim3(256), 0, st,
                     reinterpret_cast<cpx<R>*>(y), reinterpret_cast<const cpx<R>*>(x), count, a_re,
                     a_im, b);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_pair(const void* mu, const void* w, int S, size_t N, double cre, double cim, double* g,
                       hipStream_t st) {
  const auto kern = sizeof(R) == 8 || cre != 0.0 ? k_pair<R, true> : k_pair<R, false>;
  nct_launch(kern, dim3(nblocks(N, 256)), dim3(256), 0, st, reinterpret_cast<const cpx<R>*>(mu),
             reinterpret_cast<const cpx<R>*>(w), S, N, cre, cim, g);
  return hipGetLastError();
}
#if NCT_FP64_TU
hipError_t launch_field_adjoint(const double* rho, const double* g, const double* pg, int xc,
                                double thr, size_t N, double* gnm, double* part, int* nblk_out,
                                hipStream_t st) {
  const unsigned nb = nblocks(N, 256);
  *nblk_out = int(nb);
  nct_launch(k_field_adjoint, dim3(nb), dim3(256), 0, st, rho, g, pg, xc, thr, N, gnm, part);
  return hipGetLastError();
}
#endif
template <typename R>
hipError_t launch_density_backprop(const void* psi, const double* occ, const double* gnm, int S,
                                   size_t N, int add, void* lam, hipStream_t st) {
  nct_launch((k_density_backprop<R>), dim3(nblocks(size_t(S) * N, 256)), dim3(256), 0, st,
                     reinterpret_cast<const cpx<R>*>(psi), occ, gnm, S, N, add,
                     reinterpret_cast<cpx<R>*>(lam));
  return hipGetLastError();
}

// explicit instantiations
#define NCT_INST(R)                                                                                \
  template hipError_t launch_plane_yz<R>(const int*, int, const StageArgs<R>&, const KinTables&,   \
                                         const ProjTables&, const void*, const void*, hipStream_t); \
  template hipError_t launch_xv<R>(const int*, int, const StageArgs<R>&, void*, const void*,       \
                                   const KinTables&, hipStream_t);                                 \
  template hipError_t launch_gather_rows<R>(const ProjTables&, const void*, void*, int, size_t, hipStream_t); \
  template hipError_t launch_phases<R>(const double*, const int*, int, const double*, const ProjTables&, void*, \
                                       hipStream_t);                                                \
  template hipError_t launch_xpass<R>(const int*, int, const void*, void*, const R*, const R*, R,  \
                                      int, const void*, hipStream_t, int, KTables<R>);             \
  template hipError_t launch_density<R>(const void*, const double*, int, size_t, double*,          \
                                        hipStream_t);                                              \
  template hipError_t launch_proj_contract<R>(const ProjTables&, const void*, int, void*, const PhaseTab&, \
                                              hipStream_t);                                        \
  template hipError_t launch_proj_coeffs<R>(const ProjTables&, const void*, int, double, void*, hipStream_t); \
  template hipError_t launch_proj_scatter<R>(const ProjTables&, const void*, const void*, int, double, void*, \
                                             const PhaseTab&, hipStream_t);                        \
  template hipError_t launch_seed<R>(const void*, const double*, int, size_t, double, double,      \
                                     double, double, void*, hipStream_t);                          \
  template hipError_t launch_axpby<R>(void*, const void*, size_t, R, R, R, hipStream_t);          \
  template hipError_t launch_pair<R>(const void*, const void*, int, size_t, double, double, double*, \
                                     hipStream_t);                                               \
  template hipError_t launch_density_backprop<R>(const void*, const double*, const double*, int,  \
                                                 size_t, int, void*, hipStream_t);               \
  template hipError_t launch_gram<R>(const void*, int, size_t, double, void*, int, void*, hipStream_t); \
  template hipError_t launch_basis_transform<R>(const void*, const void*, int, size_t, void*, hipStream_t);
#if NCT_FP64_TU
NCT_INST(double)
template hipError_t launch_plane_inv<double>(const int*, int, const void*, void*, double, const void*, const void*,
                                             hipStream_t);
#else
NCT_INST(float)
template hipError_t launch_plane_fwd<float>(const int*, int, const void*, void*, void*, const ProjTables*,
                                            const void*, const void*, hipStream_t, KTables<float>);
template hipError_t launch_rephase_rows<float>(const ProjTables&, void*, int, const double*, hipStream_t);
template hipError_t launch_xpass_energy<float>(const int*, int, const void*, const float*, const float*, float,
                                               const void*, double*, int*, hipStream_t, KTables<float>);
#endif

}  // namespace nct
