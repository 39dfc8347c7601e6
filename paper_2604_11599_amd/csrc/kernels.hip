// gfx950 kernels of the dynamic-circuit state-vector path (complex128).
//
// State layout: shot s holds its 2^n amplitudes contiguously at
// state + s * stride (double2 = re, im; index i = sum_q b_q 2^q).
//
// Kernels:
//   k_bind_matrices   2x2 gate matrices (and their angle derivatives) from theta
//   k_init_state      |0...0> for every shot
//   k_tile_pass       one fused gate pass: each workgroup stages a 2^t tile in
//                     LDS, applies the pending collapse, the pass's guarded
//                     gates (in the shot's qubit-flip frame) and stores it back
//   k_site_reduce     per-workgroup probability histogram over <= 4 qubits
//   k_site_finalize   per shot: fixed-order sum of the histograms, Philox draws,
//                     outcomes, classical bits, flags, record, new pending collapse
//   k_site_fused      both for states of up to 14 qubits
//   k_resident        a whole shot of up to 12 qubits, its state in LDS
//   k_persistent      (request, shot) items of a batch, one workgroup each
//   k_pass_units      one gate pass of many requests' prefixes
//   k_materialize     the logical state of one shot (collapse + frame applied)
// The expectation-value and adjoint-gradient kernels are in adjoint.hip.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include "device_common.h"
#include "kernels.h"
#include "qsv.h"

namespace qsv {

// Philox4x64-10 (Salmon et al., SC'11): multipliers and Weyl increments of
// Philox4x64. One block for key (k0, k1) and counter (c0, c1, c2, c3), in place.
__device__ __forceinline__ void philox_block(uint64_t& c0, uint64_t& c1, uint64_t& c2, uint64_t& c3, uint64_t k0,
                                             uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
    uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
    uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += W0;
    k1 += W1;
  }
}

// A shot's word of measure/reset event e: counter (e / 4 + 1, 0, 0, 0) under key (seed, shot), word e % 4.

// ---------------------------------------------------------------------------
// Matrix binding (compile once, run many: angles are affine in theta)
// ---------------------------------------------------------------------------
__device__ void set2(double* m, double2 a, double2 b, double2 c, double2 d) {
  m[0] = a.x; m[1] = a.y; m[2] = b.x; m[3] = b.y; m[4] = c.x; m[5] = c.y; m[6] = d.x; m[7] = d.y;
}
__device__ __forceinline__ double2 cexpi(double t) {
  double s, c;
  sincos(t, &s, &c);
  return make_double2(c, s);
}

// theta extended by the derived parameters: out[b] = theta[b] (P values)
// followed by D values, derived k = sum of coef[e] * theta[b][in[e]] over
// e in [off[k], off[k + 1]) in that order.
__global__ void k_derive_params(const double* __restrict__ theta, uint32_t P, uint32_t D,
                                const uint32_t* __restrict__ off, const uint32_t* __restrict__ in,
                                const double* __restrict__ coef, uint32_t batch, double* __restrict__ out) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t W = P + D;
  if (idx >= (uint64_t)batch * W) return;
  const uint32_t b = (uint32_t)(idx / W), j = (uint32_t)(idx % W);
  const double* t = theta + (uint64_t)b * P;
  double v = 0.0;
  if (j < P) {
    v = t[j];
  } else {
    for (uint32_t e = off[j - P]; e < off[j - P + 1]; ++e) v += coef[e] * t[in[e]];
  }
  out[idx] = v;
}

hipError_t launch_derive_params(const double* theta, uint32_t P, uint32_t D, const uint32_t* off, const uint32_t* in,
                                const double* coef, uint32_t batch, double* out, hipStream_t st) {
  const uint64_t total = (uint64_t)batch * (P + D);
  if (!total) return hipSuccess;
  hipLaunchKernelGGL(k_derive_params, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, st, theta, P, D, off, in,
                     coef, batch, out);
  return hipGetLastError();
}

// One matrix slot from its source and a theta row: the 2x2 matrix at m and,
// when dm is set, its derivatives by each angle.
__device__ __forceinline__ void bind_slot(const GateSrc& g, const double* __restrict__ th, double* m, double* dm) {
  double a[3];
  for (int k = 0; k < 3; ++k) {
    a[k] = g.offset[k];
    if (g.param[k] != QSV_NONE) a[k] += g.scale[k] * th[g.param[k]];
  }
  const double2 Z0 = make_double2(0, 0), O1 = make_double2(1, 0), I1 = make_double2(0, 1);
  const double r2 = 0.70710678118654752440;
  if (dm)
    for (int k = 0; k < 3 * kMatStride; ++k) dm[k] = 0.0;
  switch (g.kind) {
    case QSV_G_X: case QSV_G_CX: set2(m, Z0, O1, O1, Z0); break;
    case QSV_G_Y: case QSV_G_CY: set2(m, Z0, make_double2(0, -1), I1, Z0); break;
    case QSV_G_Z: case QSV_G_CZ: set2(m, O1, Z0, Z0, make_double2(-1, 0)); break;
    case QSV_G_H: case QSV_G_CH:
      set2(m, make_double2(r2, 0), make_double2(r2, 0), make_double2(r2, 0), make_double2(-r2, 0));
      break;
    case QSV_G_S: set2(m, O1, Z0, Z0, I1); break;
    case QSV_G_SDG: set2(m, O1, Z0, Z0, make_double2(0, -1)); break;
    case QSV_G_T: set2(m, O1, Z0, Z0, make_double2(r2, r2)); break;
    case QSV_G_TDG: set2(m, O1, Z0, Z0, make_double2(r2, -r2)); break;
    case QSV_G_SX:
      set2(m, make_double2(0.5, 0.5), make_double2(0.5, -0.5), make_double2(0.5, -0.5), make_double2(0.5, 0.5));
      break;
    case QSV_G_SXDG:
      set2(m, make_double2(0.5, -0.5), make_double2(0.5, 0.5), make_double2(0.5, 0.5), make_double2(0.5, -0.5));
      break;
    case QSV_G_RX: case QSV_G_CRX: {
      double s, c;
      sincos(0.5 * a[0], &s, &c);
      set2(m, make_double2(c, 0), make_double2(0, -s), make_double2(0, -s), make_double2(c, 0));
      if (dm) set2(dm, make_double2(-0.5 * s, 0), make_double2(0, -0.5 * c), make_double2(0, -0.5 * c),
                   make_double2(-0.5 * s, 0));
      break;
    }
    case QSV_G_RY: case QSV_G_CRY: {
      double s, c;
      sincos(0.5 * a[0], &s, &c);
      set2(m, make_double2(c, 0), make_double2(-s, 0), make_double2(s, 0), make_double2(c, 0));
      if (dm) set2(dm, make_double2(-0.5 * s, 0), make_double2(-0.5 * c, 0), make_double2(0.5 * c, 0),
                   make_double2(-0.5 * s, 0));
      break;
    }
    case QSV_G_RZ: case QSV_G_CRZ: {
      double2 e0 = cexpi(-0.5 * a[0]), e1 = cexpi(0.5 * a[0]);
      set2(m, e0, Z0, Z0, e1);
      if (dm) set2(dm, make_double2(0.5 * e0.y, -0.5 * e0.x), Z0, Z0, make_double2(-0.5 * e1.y, 0.5 * e1.x));
      break;
    }
    case QSV_G_P: case QSV_G_CP: {
      double2 e = cexpi(a[0]);
      set2(m, O1, Z0, Z0, e);
      if (dm) set2(dm, Z0, Z0, Z0, make_double2(-e.y, e.x));
      break;
    }
    case QSV_G_U: {
      double s, c;
      sincos(0.5 * a[0], &s, &c);
      double2 ep = cexpi(a[1]), el = cexpi(a[2]), epl = cexpi(a[1] + a[2]);
      set2(m, make_double2(c, 0), cscale(el, -s), cscale(ep, s), cscale(epl, c));
      if (dm) {
        // d/dtheta, d/dphi, d/dlambda of U(theta, phi, lambda)
        set2(dm, make_double2(-0.5 * s, 0), cscale(el, -0.5 * c), cscale(ep, 0.5 * c), cscale(epl, -0.5 * s));
        set2(dm + kMatStride, Z0, Z0, cmul(I1, cscale(ep, s)), cmul(I1, cscale(epl, c)));
        set2(dm + 2 * kMatStride, Z0, cmul(I1, cscale(el, -s)), Z0, cmul(I1, cscale(epl, c)));
      }
      break;
    }
    default: set2(m, O1, Z0, Z0, O1); break;  // ID, SWAP (unused)
  }
}


// The first n_bind of each batch element's n_slots matrix slots (the others hold
// composed matrices, which k_compose_dense writes whole).
__global__ void k_bind_matrices(const GateSrc* __restrict__ src, uint32_t n_bind, uint32_t n_slots,
                                const double* __restrict__ theta, uint32_t n_params, uint32_t batch,
                                double* __restrict__ mats, double* __restrict__ dmats) {
  uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (uint64_t)n_bind * batch) return;
  const uint32_t b = (uint32_t)(idx / n_bind), slot = (uint32_t)(idx % n_bind);
  const uint64_t at = (uint64_t)b * n_slots + slot;
  bind_slot(src[slot], theta + (uint64_t)b * n_params, mats + at * kMatStride,
            dmats ? dmats + at * 3 * kMatStride : nullptr);
}

// The matrix slots of many programs at once (a batch of requests, each with its
// own theta row and matrices): one thread per slot; unit k covers slots
// [units[k].slot_begin, units[k + 1].slot_begin) of the flat range.
__global__ void k_bind_units(const BindUnit* __restrict__ units, uint32_t n_units, uint64_t n_total) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_total) return;
  uint32_t lo = 0, hi = n_units;  // the last unit whose slot_begin <= idx
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (units[mid].slot_begin <= idx) lo = mid;
    else hi = mid;
  }
  const BindUnit u = units[lo];
  const uint64_t slot = idx - u.slot_begin;
  bind_slot(u.src[slot], u.theta, u.mats + slot * kMatStride, nullptr);
}

hipError_t launch_bind_units(const BindUnit* units, uint32_t n_units, uint64_t n_total, hipStream_t st) {
  if (!n_total || !n_units) return hipSuccess;
  hipLaunchKernelGGL(k_bind_units, dim3((uint32_t)((n_total + 255) / 256)), dim3(256), 0, st, units, n_units,
                     n_total);
  return hipGetLastError();
}

hipError_t launch_bind_matrices(const GateSrc* src, uint32_t n_bind, uint32_t n_slots, const double* theta,
                                uint32_t n_params, uint32_t batch, double* mats, double* dmats,
                                hipStream_t st) {
  uint64_t total = (uint64_t)n_bind * batch;
  if (total == 0) return hipSuccess;
  uint32_t blocks = (uint32_t)((total + 255) / 256);
  hipLaunchKernelGGL(k_bind_matrices, dim3(blocks), dim3(256), 0, st, src, n_bind, n_slots, theta, n_params,
                     batch, mats, dmats);
  return hipGetLastError();
}

// Depolarizing slots of a call with rate p (one thread per shot and slot): the
// word of counter (noise[ctr[e]].ctr[0..2], 1) under key (key[0], key[1] + s),
// as u = (w >> 11) 2^-53, puts X (u < p/3), Y (u < 2p/3), Z (u < p) or the
// identity into matrix slot slot[e] of shot s. The fourth counter word is 0 in
// every measure/reset event's counter, so the two kinds of draws never meet.
// With dirty: a slot that draws a Pauli marks dirty[s * n_dense + nd[e]]
// (nd[e]: the dense phase holding slot e, or kNoDense), so that only those
// phases of the shot are composed again.
__global__ void k_noise_matrices(const uint32_t* __restrict__ slot, const uint32_t* __restrict__ ctr, uint32_t n,
                                 const qsv_noise* __restrict__ noise, const uint64_t* __restrict__ key, double p,
                                 uint32_t shots, uint64_t mat_stride, double* __restrict__ mats,
                                 const uint32_t* __restrict__ nd, uint32_t n_dense, uint8_t* __restrict__ dirty) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (uint64_t)n * shots) return;
  const uint32_t s = (uint32_t)(idx / n), e = (uint32_t)(idx % n);
  const qsv_noise c = noise[ctr[e]];
  uint64_t c0 = c.ctr[0], c1 = c.ctr[1], c2 = c.ctr[2], c3 = 1;
  philox_block(c0, c1, c2, c3, key[0], key[1] + s);
  const double u = (double)(c0 >> 11) * 0x1p-53;
  const double2 Z0 = make_double2(0, 0), O1 = make_double2(1, 0);
  double* m = mats + (uint64_t)s * mat_stride + (uint64_t)slot[e] * kMatStride;
  if (u < p && dirty && nd[e] != kNoDense) dirty[(uint64_t)s * n_dense + nd[e]] = 1;
  if (u >= p) set2(m, O1, Z0, Z0, O1);
  else if (u < p / 3.0) set2(m, Z0, O1, O1, Z0);
  else if (u < 2.0 * p / 3.0) set2(m, Z0, make_double2(0, -1), make_double2(0, 1), Z0);
  else set2(m, O1, Z0, Z0, make_double2(-1, 0));
}

// one workgroup clears n words (a fill kernel: safe to capture in a graph)
__global__ void k_zero_u32(uint32_t* p, uint32_t n);

hipError_t launch_noise_matrices(const uint32_t* slot, const uint32_t* ctr, uint32_t n, const qsv_noise* noise,
                                 const uint64_t* key, double p, uint32_t shots, uint64_t mat_stride, double* mats,
                                 const uint32_t* nd, uint32_t n_dense, uint8_t* dirty, hipStream_t st) {
  if (dirty && n_dense && shots) {
    const uint64_t words = ((uint64_t)shots * n_dense + 3) / 4;
    if (words > 0xFFFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(256), 0, st, reinterpret_cast<uint32_t*>(dirty), (uint32_t)words);
  }
  const uint64_t total = (uint64_t)n * shots;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_noise_matrices, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, st, slot, ctr, n, noise,
                     key, p, shots, mat_stride, mats, nd, n_dense, dirty);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Control blocks and state initialisation
// ---------------------------------------------------------------------------
__global__ void k_init_ctl(ShotCtl* ctl, uint64_t* creg, uint32_t cw, uint8_t* record, uint32_t max_record,
                           uint32_t shots) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= shots) return;
  ShotCtl c;
  c.flags = 0;
  c.pend_mask = 0;
  c.pend_val = 0;
  c.frame = 0;
  c.pend_scale = 1.0;
  c.record_prob = 1.0;
  c.n_events = 0;
  c.n_record = 0;
  c.status = 0;
  c.wg_done = 0;
  ctl[s] = c;
  for (uint32_t w = 0; w < cw; ++w) creg[(uint64_t)s * cw + w] = 0;
  if (record)
    for (uint32_t w = 0; w < max_record; ++w) record[(uint64_t)s * max_record + w] = 0;
}

hipError_t launch_init_ctl(ShotCtl* ctl, uint64_t* creg, uint32_t cw, uint8_t* record, uint32_t max_record,
                           uint32_t shots, hipStream_t st) {
  if (!shots) return hipSuccess;
  hipLaunchKernelGGL(k_init_ctl, dim3((shots + 255) / 256), dim3(256), 0, st, ctl, creg, cw, record, max_record,
                     shots);
  return hipGetLastError();
}

template <typename CT>
__global__ void k_init_state(CT* __restrict__ state, uint64_t stride, uint64_t dim, uint32_t shots) {
  uint64_t total = dim * shots;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * blockDim.x) {
    uint64_t s = i / dim, j = i % dim;
    state[s * stride + j] = cmake<CT>(j == 0 ? 1.0 : 0.0, 0.0);
  }
}

hipError_t launch_init_state(double2* state, uint64_t stride, uint32_t n, uint32_t shots, hipStream_t st, bool c64) {
  uint64_t total = (1ull << n) * shots;
  uint64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (c64)
    hipLaunchKernelGGL(k_init_state<float2>, dim3((uint32_t)blocks), dim3(256), 0, st,
                       reinterpret_cast<float2*>(state), stride, 1ull << n, shots);
  else
    hipLaunchKernelGGL(k_init_state<double2>, dim3((uint32_t)blocks), dim3(256), 0, st, state, stride, 1ull << n,
                       shots);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tile pass
// ---------------------------------------------------------------------------
// Applies one gate to the LDS tile (tile-local logical indices).
template <typename CT>
__device__ __forceinline__ void tile_apply(CT* __restrict__ tile, uint32_t t, const DGate& g,
                                           const double* __restrict__ m) {
  const uint32_t tid = threadIdx.x;
  switch (g.type) {
    case GT_DENSE1: case GT_DIAG1: {
      const M2x<CT> u = load_m2x<CT>(m, 0);
      const uint32_t np = 1u << (t - 1), bit = 1u << g.b0;
      if (g.type == GT_DIAG1) {
        for (uint32_t p = tid; p < np; p += kTileThreads) {
          uint32_t i0 = ins0(p, g.b0), i1 = i0 | bit;
          tile[i0] = cmul(u.a, tile[i0]);
          tile[i1] = cmul(u.d, tile[i1]);
        }
      } else {
        for (uint32_t p = tid; p < np; p += kTileThreads) {
          uint32_t i0 = ins0(p, g.b0), i1 = i0 | bit;
          CT x0 = tile[i0], x1 = tile[i1];
          tile[i0] = cmac2(u.a, x0, u.b, x1);
          tile[i1] = cmac2(u.c, x0, u.d, x1);
        }
      }
      break;
    }
    case GT_X1: {
      const uint32_t np = 1u << (t - 1), bit = 1u << g.b0;
      for (uint32_t p = tid; p < np; p += kTileThreads) {
        uint32_t i0 = ins0(p, g.b0), i1 = i0 | bit;
        CT x0 = tile[i0];
        tile[i0] = tile[i1];
        tile[i1] = x0;
      }
      break;
    }
    default: {  // two-qubit gates
      const uint32_t lo = g.b0 < g.b1 ? g.b0 : g.b1, hi = g.b0 < g.b1 ? g.b1 : g.b0;
      const uint32_t nq = 1u << (t - 2);
      const uint32_t B0 = 1u << g.b0, B1 = 1u << g.b1;
      if (g.type == GT_CX) {
        for (uint32_t p = tid; p < nq; p += kTileThreads) {
          uint32_t i = ins0(ins0(p, lo), hi) | B0;
          CT x = tile[i];
          tile[i] = tile[i | B1];
          tile[i | B1] = x;
        }
      } else if (g.type == GT_CTRL1) {
        const M2x<CT> u = load_m2x<CT>(m, 0);
        for (uint32_t p = tid; p < nq; p += kTileThreads) {
          uint32_t i = ins0(ins0(p, lo), hi) | B0;
          CT x0 = tile[i], x1 = tile[i | B1];
          tile[i] = cmac2(u.a, x0, u.b, x1);
          tile[i | B1] = cmac2(u.c, x0, u.d, x1);
        }
      } else if (g.type == GT_CPHASE) {
        const CT ph = cmake<CT>(m[6], m[7]);
        for (uint32_t p = tid; p < nq; p += kTileThreads) {
          uint32_t i = ins0(ins0(p, lo), hi) | B0 | B1;
          tile[i] = cmul(ph, tile[i]);
        }
      } else {  // GT_SWAP
        for (uint32_t p = tid; p < nq; p += kTileThreads) {
          uint32_t i = ins0(ins0(p, lo), hi);
          CT x = tile[i | B0];
          tile[i | B0] = tile[i | B1];
          tile[i | B1] = x;
        }
      }
      break;
    }
  }
}

template <typename CT>
__global__ __launch_bounds__(kTileThreads) void k_tile_pass(
    CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl,
    const DGate* __restrict__ gates, const double* __restrict__ mats, uint64_t mat_stride, PassArgs a) {
  extern __shared__ double2 qsv_lds[];
  CT* const tile = reinterpret_cast<CT*>(qsv_lds);
  const uint32_t shot = blockIdx.y, w = blockIdx.x, tid = threadIdx.x;
  ShotCtl* c = ctl + shot;
  if (c->status != 0) return;
  const uint64_t flags = c->flags, M = c->pend_mask, F = c->frame;
  const double s = c->pend_scale;
  const bool pending = M != 0 || s != 1.0;
  bool any = false;
  for (uint32_t i = 0; i < a.gate_count && !any; ++i) any = guard_ok(flags, gates[a.gate_begin + i].guard);
  if (!a.init && !any) return;  // the pending collapse stays owed to a later pass
  const uint64_t V = c->pend_val;
  // Tile w holds the logical indices whose non-tile bits spell w; amplitude i is
  // stored at memory index i ^ F (the shot's flip frame), so a workgroup reads
  // and writes one memory tile and gates act on logical indices.
  uint64_t base = 0;
  {
    uint32_t k = 0;
    for (uint32_t q = 0; q < a.n; ++q)
      if (!((a.tile_mask >> q) & 1ull)) base |= (uint64_t)((w >> k++) & 1u) << q;
  }
  CT* st = state + (uint64_t)shot * stride;
  const uint32_t T = 1u << a.t;
  for (uint32_t l = tid; l < T; l += kTileThreads) {
    uint64_t gi = base | local_to_global(l, a);
    CT v;
    if (a.init) {
      v = cmake<CT>(gi == 0 ? 1.0 : 0.0, 0.0);
    } else if ((gi & M) != V) {
      v = cmake<CT>(0.0, 0.0);
    } else {
      v = st[gi ^ F];
      if (pending) v = cscale(v, s);
    }
    tile[l] = v;
  }
  __syncthreads();
  const double* mb = mats + (uint64_t)shot * mat_stride;
  for (uint32_t i = 0; i < a.gate_count; ++i) {
    DGate g = gates[a.gate_begin + i];
    if (!guard_ok(flags, g.guard)) continue;
    tile_apply(tile, a.t, g, mb + (uint64_t)g.mat * kMatStride);
    __syncthreads();
  }
  for (uint32_t l = tid; l < T; l += kTileThreads) st[(base | local_to_global(l, a)) ^ F] = tile[l];
  if (pending) {
    // the last workgroup of this shot to finish clears the pending collapse
    __syncthreads();
    if (tid == 0) {
      __threadfence();
      uint32_t done = atomicAdd(&c->wg_done, 1u);
      if (done == a.tiles - 1) {
        c->pend_mask = 0;
        c->pend_val = 0;
        c->pend_scale = 1.0;
        c->wg_done = 0;
      }
    }
  }
}

template <typename CT>
__global__ __launch_bounds__(kTileThreads) void k_tile_pass_r(CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl,
                              const DGate* __restrict__ gates, const Phase* __restrict__ phases,
                              const double* __restrict__ mats, uint64_t mat_stride, PassArgs a, uint32_t shots);

hipError_t resident_grid(const void* kernel, uint32_t threads, size_t lds, size_t max_lds, uint32_t* out) {
  // (LDS sizes come in steps of at least 512 bytes up to a CU's 160 KiB, so the
  // table holds a few hundred entries per kernel at most)
  static std::map<std::tuple<int, const void*, uint32_t, size_t>, uint32_t> grids;
  static std::mutex mu;  // forked contexts launch from several host threads
  std::lock_guard<std::mutex> lk(mu);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const auto key = std::make_tuple(dev, kernel, threads, lds);
  const auto hit = grids.find(key);
  if (hit != grids.end()) {
    *out = hit->second;
    return hipSuccess;
  }
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds);
  if (e != hipSuccess) return e;
  int cus = 0, per = 0;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, (int)threads, lds);
  if (e != hipSuccess) return e;
  *out = grids[key] = (uint32_t)std::max(1, cus) * (uint32_t)std::max(1, per);
  return hipSuccess;
}

// Waves per SIMD the eight-wave dense pass is compiled for: two workgroups per
// CU with complex128 tiles (64 KiB of LDS each), three with complex64 tiles
// (32 KiB), so that the HBM, LDS and matrix-core work of different workgroups
// overlap.
// kPreload: the staged phases' descriptors are read once per workgroup into
// scalar registers (complex128; the complex64 build, held to 80 VGPRs for its
// third workgroup, spills more with them and runs slower).
template <typename CT> struct D8Waves;
template <> struct D8Waves<double2> { static constexpr int kMin = 4; static constexpr bool kPreload = true; };
template <> struct D8Waves<float2> { static constexpr int kMin = 6; static constexpr bool kPreload = false; };
template <typename CT>
__global__ __launch_bounds__(2 * kTileThreads, D8Waves<CT>::kMin) void k_tile_pass_d8(
    CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, const Phase* __restrict__ phases,
    const double* __restrict__ mats, uint64_t mat_stride, PassArgs a, uint32_t shots, uint32_t lds_mats);
// Tiles per resident workgroup from which complex64 passes take the register steps.
constexpr uint64_t kRegStepMinTiles = 4;
template <bool kStaged>
__global__ __launch_bounds__(kTileThreads, 4) void k_tile_pass_c64(
    float2* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, const RegStep* __restrict__ reg_steps,
    const double* __restrict__ mats, uint64_t mat_stride, PassArgs a, uint32_t shots);

template <typename CT>
static hipError_t tile_pass_t(const RunBuffers& rb, CT* state, const DGate* gates, const Phase* phases,
                              const RegStep* reg_steps, const double* mats, uint64_t mat_stride, const PassArgs& a, hipStream_t st) {
  dim3 grid(a.tiles, rb.shots);
  size_t lds = (size_t)sizeof(CT) << a.t;
  if (a.phase_count) {
    const uint64_t total = (uint64_t)a.tiles * rb.shots;
    const size_t mat_lds = (size_t)a.phase_count * 256u * sizeof(CT);
    const size_t max_lds = (sizeof(CT) << kTileMaxBits) + kLdsDensePhases * 256u * sizeof(CT);
    const uint32_t nthr = 1u << (a.t - kRegBits);
    uint32_t g = 0;
    hipError_t e = hipSuccess;
    // all-dense passes: eight amplitudes per thread and one LDS round trip per
    // phase. complex64 tiles in plenty take the register steps instead, sixteen
    // amplitudes per thread: 1.33 against 1.51 ms for four phases on 2^28
    // amplitudes, but with up to a tile per workgroup (20 qubits x 4 shots) 2 us
    // longer, since a thread's chain of products is twice as long. complex128
    // gains nothing (28 qubits x 4 shots: 346 against 336 ms in all such passes;
    // the clock falls to 2.2 GHz under FP64 products and HBM traffic together).
    if (a.all_dense && a.t >= kDenseMinTileBits && (sizeof(CT) == sizeof(double2) || !a.guard)) {
      const bool staged = a.phase_count <= kLdsDensePhases && mat_stride == 0;
      if constexpr (sizeof(CT) == sizeof(float2)) {
        const size_t l = (a.exchanges ? lds : 0) + (staged ? mat_lds : 0);
        const auto kernel = staged ? k_tile_pass_c64<true> : k_tile_pass_c64<false>;
        e = resident_grid((const void*)kernel, nthr, l, max_lds, &g);
        if (e != hipSuccess) return e;
        if (total >= kRegStepMinTiles * (uint64_t)g) {
          hipLaunchKernelGGL(kernel, dim3(g), dim3(nthr), l, st, state, rb.stride, rb.ctl, reg_steps, mats, mat_stride,
                             a, rb.shots);
          return hipGetLastError();
        }
      }
      const size_t l8 = lds + (staged ? mat_lds : 0);
      e = resident_grid((const void*)k_tile_pass_d8<CT>, 2 * nthr, l8, max_lds, &g);
      if (e != hipSuccess) return e;
      if ((uint64_t)g > total) g = (uint32_t)total;
      if (!g) return hipSuccess;
      hipLaunchKernelGGL(k_tile_pass_d8<CT>, dim3(g), dim3(2 * nthr), l8, st, state, rb.stride, rb.ctl, phases, mats,
                         mat_stride, a, rb.shots, staged ? 1u : 0u);
      return hipGetLastError();
    }
    e = resident_grid((const void*)k_tile_pass_r<CT>, nthr, lds, max_lds, &g);
    if (e != hipSuccess) return e;
    if ((uint64_t)g > total) g = (uint32_t)total;
    if (!g) return hipSuccess;
    k_tile_pass_r<CT><<<dim3(g), dim3(nthr), lds, st>>>(state, rb.stride, rb.ctl, gates, phases, mats, mat_stride, a,
                                                        rb.shots);
  } else {
    hipLaunchKernelGGL(k_tile_pass<CT>, grid, dim3(kTileThreads), lds, st, state, rb.stride, rb.ctl, gates,
                       mats, mat_stride, a);
  }
  return hipGetLastError();
}

hipError_t launch_tile_pass(const RunBuffers& rb, const DGate* gates, const Phase* phases, const RegStep* reg_steps,
                            const double* mats, uint64_t mat_stride, const PassArgs& a, hipStream_t st) {
  if (rb.c64)
    return tile_pass_t(rb, reinterpret_cast<float2*>(rb.state), gates, phases, reg_steps, mats, mat_stride, a, st);
  return tile_pass_t(rb, rb.state, gates, phases, reg_steps, mats, mat_stride, a, st);
}

// ---------------------------------------------------------------------------
// Register-blocked tile pass
//
// Each thread owns the 16 amplitudes of the tile that differ only in the
// phase's 4 register bits, applies the phase's gates to them in registers and
// hands them back through LDS, where the next phase picks up a different set
// of 4 bits. One LDS round trip per phase instead of one per gate.
// ---------------------------------------------------------------------------

// Composes every dense phase: column c of the phase's complex matrix M is the
// phase's gate list applied, in order, to the basis vector e_c (one thread per
// batch element, phase and column), stored in matrix-core operand order.
//
// Bound by the latency of the gate chain, so a workgroup is one wave that
// composes one phase: its gate list is wave-uniform (descriptors by scalar
// loads, the next gate's while one is applied; no divergence over gate types),
// also where the batch leaves three quarters of the lanes idle. The bound of 64
// threads gives the column's 16 amplitudes their registers; under the default
// of 1024 threads the kernels spilled 2900 of them. 1000 noisy 10-qubit shots
// (28 phases each): 192 us before, the call 800 us then and 697 us now; 32
// energies of 17 qubits (30 phases): 567 us and 498 us.
__device__ __forceinline__ void compose_column(const Phase& ph, const DGate* __restrict__ gates, double* mb,
                                               uint32_t c) {
  double2 a[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) a[k] = make_double2(k == (int)c ? 1.0 : 0.0, 0.0);
  DGate next = load_gate(gates + ph.gate_begin);
  for (uint32_t i = 0; i < ph.gate_count; ++i) {
    const DGate g = next;
    next = load_gate(gates + ph.gate_begin + (i + 1 < ph.gate_count ? i + 1 : i));
    r_apply(a, g.type, g.j0, g.j1, mb + (uint64_t)g.mat * kMatStride);
  }
  double2* A = reinterpret_cast<double2*>(mb + (uint64_t)ph.dense * kMatStride);
#pragma unroll
  for (uint32_t r = 0; r < (uint32_t)kR; ++r) A[dense_pos(r, c)] = a[r];
}

// With dirty: a phase whose slots all hold what they hold in the matrix set
// `clean` (dirty[b * n_dense + d] == 0) takes its column from clean's composed
// matrix, the same gate list applied to the same matrices, or with clean null
// is left out (its readers go to clean themselves).
// Workgroup d * ceil(batch / 4) + i: phase d of batch elements 4 i .. 4 i + 3.
__global__ __launch_bounds__(64) void k_compose_dense(const Phase* __restrict__ phases,
                                                      const uint32_t* __restrict__ dense,
                                                      const DGate* __restrict__ gates, uint32_t n_dense,
                                                      uint32_t batch, uint64_t mat_stride, double* __restrict__ mats,
                                                      const uint8_t* __restrict__ dirty,
                                                      const double* __restrict__ clean) {
  const uint32_t per = (batch + 3u) / 4u, d = blockIdx.x / per;
  const uint32_t c = threadIdx.x % kR, b = (blockIdx.x % per) * 4u + threadIdx.x / kR;
  if (b >= batch) return;
  const Phase ph = load_phase(phases + dense[d]);
  double* mb = mats + (uint64_t)b * mat_stride;
  if (dirty && !dirty[(uint64_t)b * n_dense + d]) {
    if (!clean) return;
    const double2* src = reinterpret_cast<const double2*>(clean + (uint64_t)ph.dense * kMatStride);
    double2* dst = reinterpret_cast<double2*>(mb + (uint64_t)ph.dense * kMatStride);
#pragma unroll
    for (uint32_t r = 0; r < (uint32_t)kR; ++r) dst[dense_pos(r, c)] = src[dense_pos(r, c)];
    return;
  }
  compose_column(ph, gates, mb, c);
}

// The same over the dense phases of many programs at once (a batch of
// requests, each with its own matrices): one workgroup of 16 threads per unit.
__global__ __launch_bounds__(64) void k_compose_units(const ComposeUnit* __restrict__ units) {
  const ComposeUnit u = units[blockIdx.x];
  compose_column(load_phase(u.phases + u.phase), u.gates, u.mats, threadIdx.x);
}

hipError_t launch_compose_units(const ComposeUnit* units, uint32_t n_units, hipStream_t st) {
  if (!n_units) return hipSuccess;
  hipLaunchKernelGGL(k_compose_units, dim3(n_units), dim3(kR), 0, st, units);
  return hipGetLastError();
}

hipError_t launch_compose_dense(const Phase* phases, const uint32_t* dense, uint32_t n_dense, const DGate* gates,
                                uint32_t batch, uint64_t mat_stride, double* mats, hipStream_t st,
                                const uint8_t* dirty, const double* clean) {
  const uint64_t blocks = (uint64_t)n_dense * ((batch + 3u) / 4u);
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(k_compose_dense, dim3((uint32_t)blocks), dim3(64), 0, st, phases, dense, gates, n_dense, batch,
                     mat_stride, mats, dirty, clean);
  return hipGetLastError();
}

// group bits 4..7 of a wave-uniform group index, scattered over the mask bits
__device__ __forceinline__ uint32_t udep_hi(const UBits& u, uint32_t g) {
  return (((g >> 4) & 1u) ? u.b[4] : 0u) | (((g >> 5) & 1u) ? u.b[5] : 0u) | (((g >> 6) & 1u) ? u.b[6] : 0u) |
         (((g >> 7) & 1u) ? u.b[7] : 0u);
}

// One dense phase on the matrix cores, for the 64 amplitude groups of this
// thread's wave (group g = tile-local indices with the non-register bits set
// to the bits of g). With M = A + iB and a block of 16 groups as X + iY (16
// components x 16 groups), the product is formed from three real 16x16
// products, P1 = A X, P2 = B Y, P3 = (A + B)(X + Y): real part P1 - P2,
// imaginary part P3 - P1 - P2 (three real multiplications per complex one
// instead of four). Each real product is 4 v_mfma_f64_16x16x4f64; that
// instruction takes A[l % 16][l / 16] and B[l / 16][l % 16] from lane l and
// returns D[4 v + l / 16][l % 16] in its result element v (the
// double-precision form interleaves the rows). So lane l needs M[l % 16][4 kb +
// l / 16] (kb = 0..3: the complex values at Mc[kb * 64 + l]), reads the
// components q + 4 kb (q = l / 16) of its group in each block and writes back
// the same components. The wave reads a block before it writes it, and the
// blocks of different waves are disjoint. xs: slots are XORed with it (the tile
// holds tile-local index l at slot swz(l) ^ xs).
// lane l's matrix-core operand of a phase matrix: Mc[kb * 64 + l], kb = 0..3;
// from LDS when the pass's matrices are staged there (in the amplitude type),
// else from HBM, rounded to it (two loops, so the compiler keeps the LDS reads
// as LDS reads)
template <typename CT>
__device__ __forceinline__ void load_mfrag(CT (&mf)[4], bool staged, const CT* __restrict__ lds_mats,
                                           const double2* __restrict__ gmat, uint32_t lane) {
  typedef typename CxT<CT>::R R;
  typedef __attribute__((address_space(3))) const R lds_r;
  typedef __attribute__((address_space(1))) const double glb_d;
  if (staged) {
    const lds_r* l = (const lds_r*)lds_mats;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      mf[kb].x = l[2 * (kb * 64 + (int)lane)];
      mf[kb].y = l[2 * (kb * 64 + (int)lane) + 1];
    }
  } else {
    const glb_d* g = (const glb_d*)gmat;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) mf[kb] = cmake<CT>(g[2 * (kb * 64 + (int)lane)], g[2 * (kb * 64 + (int)lane) + 1]);
  }
}

// One 16x16x4 product step on the matrix cores in the amplitude precision.
// kRowsInterleaved: result element v of lane l is row 4 v + l / 16 (the
// double-precision instruction) rather than row 4 (l / 16) + v (single).
template <typename CT> struct MfmaT;
template <> struct MfmaT<double2> {
  typedef double R;
  typedef qsv_d4 V4;
  static constexpr bool kRowsInterleaved = true;
  __device__ static V4 step(double a, double b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <> struct MfmaT<float2> {
  typedef float R;
  typedef qsv_f4 V4;
  static constexpr bool kRowsInterleaved = false;
  __device__ static V4 step(float a, float b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

template <int kBlocks, typename CT>
__device__ __forceinline__ void dense_phase_mfma(CT* __restrict__ tile, uint32_t T, uint32_t tid,
                                                 const Phase& ph, const CT (&mf)[4], uint32_t xs = 0u) {
  typedef MfmaT<CT> Mf;
  typedef typename Mf::R R;
  // this wave's groups: gbase + 16 cb + j, cb < kBlocks
  const uint32_t lane = tid & 63u, q = lane >> 4, j = lane & 15u;
  const uint32_t wbase = __builtin_amdgcn_readfirstlane(tid >> 6) * (16u * kBlocks);
  const uint32_t o0 = 1u << ph.r[0], o1 = 1u << ph.r[1], o2 = 1u << ph.r[2], o3 = 1u << ph.r[3];
  const UBits u = ubits((T - 1u) & ~(o0 | o1 | o2 | o3));
  R fa[4], fb[4], fs[4];  // fragments of A, B and A + B
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    fa[kb] = mf[kb].x;
    fb[kb] = mf[kb].y;
    fs[kb] = mf[kb].x + mf[kb].y;
  }
  // slot of component q + 4 k of group gbase + 16 cb + j: a per-lane part (group
  // bits 0..3, component bits of q) XOR a wave-uniform part (higher group bits,
  // component bits of k)
  const uint32_t rl = xs ^ swz(udep<4>(u, j) | ((q & 1u) ? o0 : 0u) | ((q & 2u) ? o1 : 0u));
  // where results go when the result rows are grouped: element v of lane l is
  // component 4 q + v (component bits 0..1 from v, bits 2..3 from q)
  const uint32_t rw = xs ^ swz(udep<4>(u, j) | ((q & 1u) ? o2 : 0u) | ((q & 2u) ? o3 : 0u));
  // software-pipelined over the blocks: the reads of block b + 1 are issued
  // before the writes of block b, so the LDS round trip of the next block
  // overlaps the tail of the current block's products
  uint32_t slot[2][4];
  CT x[2][4];
  {
    const uint32_t ug = udep_hi(u, wbase);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      slot[0][k] = rl ^ swz(ug | ((k & 1u) ? o2 : 0u) | ((k & 2u) ? o3 : 0u));
      x[0][k] = tile[slot[0][k]];
    }
  }
#pragma unroll
  for (uint32_t cb = 0; cb < (uint32_t)kBlocks; ++cb) {
    const uint32_t c = cb & 1u;
    typename Mf::V4 p1 = {0, 0, 0, 0}, p2 = {0, 0, 0, 0}, p3 = {0, 0, 0, 0};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      p1 = Mf::step(fa[kb], x[c][kb].x, p1);
      p2 = Mf::step(fb[kb], x[c][kb].y, p2);
      p3 = Mf::step(fs[kb], x[c][kb].x + x[c][kb].y, p3);
    }
    // the block's results go to the slots it read (every read of the block
    // is complete: its values entered the products above)
    uint32_t wslot[4];
    if (Mf::kRowsInterleaved) {
#pragma unroll
      for (int v = 0; v < 4; ++v) wslot[v] = slot[c][v];
    } else {
      const uint32_t ug = udep_hi(u, wbase + 16u * cb);
#pragma unroll
      for (uint32_t v = 0; v < 4; ++v) wslot[v] = rw ^ swz(ug | ((v & 1u) ? o0 : 0u) | ((v & 2u) ? o1 : 0u));
    }
    if (cb + 1 < (uint32_t)kBlocks) {
      const uint32_t ug = udep_hi(u, wbase + 16u * (cb + 1));
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        slot[c ^ 1u][k] = rl ^ swz(ug | ((k & 1u) ? o2 : 0u) | ((k & 2u) ? o3 : 0u));
        x[c ^ 1u][k] = tile[slot[c ^ 1u][k]];
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      CT o;
      o.x = p1[v] - p2[v];
      o.y = p3[v] - p1[v] - p2[v];
      tile[wslot[v]] = o;
    }
  }
}

// Runs the register phases of a pass on a tile of T amplitudes staged in LDS
// (slot swz(l) holds tile-local index l). Threads tid < nthr own 16 amplitudes
// per phase; every thread of the workgroup reaches the barriers.
// kDense: apply the composed matrix of dense phases on the matrix cores, and gate
// lists to the others; else gate lists to every phase. xs: as in dense_phase_mfma.
template <bool kDense, typename CT>
__device__ __forceinline__ void run_phases(CT* __restrict__ tile, uint32_t T, uint32_t tid, uint32_t nthr, uint64_t flags,
                           const Phase* __restrict__ phases, uint32_t pb, uint32_t pc,
                           const DGate* __restrict__ gates, const double* __restrict__ mb, uint32_t xs = 0u) {
  CT r[kR];
  for (uint32_t p = 0; p < pc; ++p) {
    const Phase ph = load_phase(phases + pb + p);
    bool act = false;
    for (uint32_t i = 0; i < ph.gate_count && !act; ++i) act = guard_ok(flags, cst(gates + ph.gate_begin + i)->guard);
    if (!act) continue;
    if (kDense && ph.dense != kNoDense && nthr >= 64u &&
        (sizeof(CT) == sizeof(double2) || cst(gates + ph.gate_begin)->guard == 0u)) {
      if (tid < nthr) {
        CT mf[4];
        load_mfrag(mf, false, static_cast<const CT*>(nullptr),
                   reinterpret_cast<const double2*>(mb + (uint64_t)ph.dense * kMatStride), tid & 63u);
        dense_phase_mfma<4>(tile, T, tid, ph, mf, xs);
      }
    } else if (tid < nthr) {
      const uint32_t o0 = 1u << ph.r[0], o1 = 1u << ph.r[1], o2 = 1u << ph.r[2], o3 = 1u << ph.r[3];
      const uint32_t lb = pdep32(tid, (T - 1u) & ~(o0 | o1 | o2 | o3));
#pragma unroll
      for (int k = 0; k < kR; ++k) {
        const uint32_t l = lb | ((k & 1) ? o0 : 0u) | ((k & 2) ? o1 : 0u) | ((k & 4) ? o2 : 0u) | ((k & 8) ? o3 : 0u);
        r[k] = tile[swz(l) ^ xs];
      }
      {
      // DGate words: [0] type | b0 | b1 | nang | j0 | j1 | q0 | q1, [1] mat | pad, [2] guard;
      // gate words and matrices are wave-uniform scalar loads, the next gate's
      // are requested before the current gate is applied
      const QSV_CONST uint64_t* gw = cst(reinterpret_cast<const uint64_t*>(gates + ph.gate_begin));
      const QSV_CONST double* mp = cst(mb + (uint64_t)ph.gate_begin * kMatStride);
      uint64_t w0n = gw[0], gdn = gw[2];
      double mn[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) mn[e] = mp[e];
      for (uint32_t i = 0; i < ph.gate_count; ++i) {
        const uint64_t w0 = w0n, gd = gdn;
        double m[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = mn[e];
        if (i + 1 < ph.gate_count) {
          w0n = gw[(uint64_t)(i + 1) * 4];
          gdn = gw[(uint64_t)(i + 1) * 4 + 2];
#pragma unroll
          for (int e = 0; e < 8; ++e) mn[e] = mp[(uint64_t)(i + 1) * kMatStride + e];
        }
        if (!guard_ok(flags, gd)) continue;
        r_apply(r, (uint8_t)(w0 & 0xFFu), (int)((w0 >> 32) & 0xFFu), (int)((w0 >> 40) & 0xFFu), m);
      }
      }
#pragma unroll
      for (int k = 0; k < kR; ++k) {
        const uint32_t l = lb | ((k & 1) ? o0 : 0u) | ((k & 2) ? o1 : 0u) | ((k & 4) ? o2 : 0u) | ((k & 8) ? o3 : 0u);
        tile[swz(l) ^ xs] = r[k];
      }
    }
    __syncthreads();
  }
}

// Tile-local index l = tid + k * 2^(t-4) (k = 0..15) of thread tid < 2^(t-4):
// its global index is base | (tid's bits over tq[0..t-5]) | (k's bits over
// tq[t-4..t-1]). Logical amplitude i is stored at memory index i ^ F (the
// shot's flip frame), so a workgroup reads and writes one memory tile while
// gates see logical indices.
__device__ __forceinline__ void store_tile16(const double2* __restrict__ tile, double2* __restrict__ st,
                                             const PassArgs& a, uint64_t base, uint32_t tid, uint64_t F) {
  const uint32_t nthr = 1u << (a.t - kRegBits);
  uint64_t gthr = base;
  for (uint32_t b = 0; b + kRegBits < a.t; ++b) gthr |= (uint64_t)((tid >> b) & 1u) << a.tq[b];
  const uint64_t h0 = 1ull << a.tq[a.t - 4], h1 = 1ull << a.tq[a.t - 3], h2 = 1ull << a.tq[a.t - 2],
                 h3 = 1ull << a.tq[a.t - 1];
  double2 r[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) r[k] = tile[swz(tid + (uint32_t)k * nthr)];
#pragma unroll
  for (int k = 0; k < kR; ++k) {
    const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull) |
                        ((k & 8) ? h3 : 0ull);
    st[gi ^ F] = r[k];
  }
}

// Whether the pass has work for a shot: the shot is alive and (the pass
// initialises the state, or some gate of the pass is enabled by its flags).
__device__ __forceinline__ bool pass_active(const ShotCtl* __restrict__ c, const PassArgs& a,
                                            const DGate* __restrict__ gates) {
  const QSV_CONST ShotCtl* cc = cst(c);
  if (cc->status != 0) return false;
  if (a.init || a.uncond) return true;
  const uint64_t flags = cc->flags;
  if (a.guard) return guard_ok(flags, a.guard);
  for (uint32_t i = 0; i < a.gate_count; ++i)
    if (guard_ok(flags, cst(gates + a.gate_begin + i)->guard)) return true;
  return false;
}

__device__ __forceinline__ uint64_t next_pass_item(uint64_t it, uint64_t total, uint64_t G, const ShotCtl* ctl,
                                                   const PassArgs& a, const DGate* __restrict__ gates,
                                                   uint32_t& last_shot, bool& last_active) {
  for (; it < total; it += G) {
    const uint32_t shot = (uint32_t)(it / a.tiles);
    if (shot != last_shot) {
      last_shot = shot;
      last_active = pass_active(ctl + shot, a, gates);
    }
    if (last_active) break;
  }
  return it;
}

// The 16 amplitudes of a thread (address bits gthr | subsets of h0..h3) in the
// load layout: logical amplitude i is stored at memory index i ^ F. Every
// amplitude is read (one straight run of loads); those outside a pending
// collapse are zeroed when staged.
template <typename CT>
__device__ __forceinline__ void fetch16(CT (&r)[kR], const CT* __restrict__ st, uint64_t gthr, uint64_t h0,
                                        uint64_t h1, uint64_t h2, uint64_t h3, bool init, uint64_t F) {
  if (init) {
#pragma unroll
    for (int k = 0; k < kR; ++k) {
      const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull) |
                          ((k & 8) ? h3 : 0ull);
      r[k] = cmake<CT>(gi == 0 ? 1.0 : 0.0, 0.0);
    }
  } else {
#pragma unroll
    for (int k = 0; k < kR; ++k) {
      const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull) |
                          ((k & 8) ? h3 : 0ull);
      r[k] = st[gi ^ F];
    }
  }
}

// the 16 amplitudes of a thread into LDS (load layout l = tid + k nthr), with
// the pending collapse's scale applied
template <typename CT>
__device__ __forceinline__ void stage16(CT* __restrict__ tile, const CT (&r)[kR], uint32_t tid,
                                        uint32_t nthr, uint64_t gthr, uint64_t h0, uint64_t h1, uint64_t h2,
                                        uint64_t h3, uint64_t M, uint64_t V, double s) {
  if (M == 0 && s == 1.0) {
#pragma unroll
    for (int k = 0; k < kR; ++k) tile[swz(tid + (uint32_t)k * nthr)] = r[k];
  } else {
#pragma unroll
    for (int k = 0; k < kR; ++k) {
      const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull) |
                          ((k & 8) ? h3 : 0ull);
      tile[swz(tid + (uint32_t)k * nthr)] = ((gi & M) == V) ? cscale(r[k], s) : cmake<CT>(0.0, 0.0);
    }
  }
}

// Persistent register-blocked pass. The grid holds as many workgroups as fit
// on the device at once; workgroup b takes the work items (shot, tile)
// b, b + G, b + 2G, ... (item = shot * tiles + tile) of shots the pass has work
// for. For passes with gate lists: their registers leave no room to hold the
// next tile meanwhile, so each tile is loaded when its turn comes.
template <typename CT>
__global__ __launch_bounds__(kTileThreads) void k_tile_pass_r(
    CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, const DGate* __restrict__ gates,
    const Phase* __restrict__ phases, const double* __restrict__ mats, uint64_t mat_stride, PassArgs a,
    uint32_t shots) {
  extern __shared__ double2 qsv_lds[];
  CT* const tile = reinterpret_cast<CT*>(qsv_lds);
  const uint32_t tid = threadIdx.x;
  const uint32_t nthr = 1u << (a.t - kRegBits), T = 1u << a.t;
  const uint64_t total = (uint64_t)a.tiles * shots, G = gridDim.x;
  const uint64_t free_mask = ~a.tile_mask & ((a.n >= 64) ? ~0ull : ((1ull << a.n) - 1ull));
  uint64_t tb = 0;  // this thread's bits over tile qubits tq[0..t-5]
  for (uint32_t b = 0; b + kRegBits < a.t; ++b) tb |= (uint64_t)((tid >> b) & 1u) << a.tq[b];
  const uint64_t h0 = 1ull << a.tq[a.t - 4], h1 = 1ull << a.tq[a.t - 3], h2 = 1ull << a.tq[a.t - 2],
                 h3 = 1ull << a.tq[a.t - 1];
  // next item at or after `it` (in steps of G) whose shot the pass has work for;
  // the answer for the last shot looked at is kept
  uint32_t last_shot = 0xFFFFFFFFu;
  bool last_active = false;
  CT nx[kR];
  uint64_t it = next_pass_item(blockIdx.x, total, G, ctl, a, gates, last_shot, last_active);
  if (it < total) {
    const uint32_t sh = (uint32_t)(it / a.tiles);
    const QSV_CONST ShotCtl* cc = cst(ctl + sh);
    const uint64_t g0 = tile_base(it % a.tiles, free_mask) | tb;
    fetch16(nx, state + (uint64_t)sh * stride, g0, h0, h1, h2, h3, a.init, cc->frame);
    stage16(tile, nx, tid, nthr, g0, h0, h1, h2, h3, cc->pend_mask, cc->pend_val, cc->pend_scale);
    __syncthreads();
  }
  while (it < total) {
    const uint32_t shot = (uint32_t)(it / a.tiles);
    ShotCtl* c = ctl + shot;
    const uint64_t flags = cst(c)->flags, F = cst(c)->frame;
    const bool pending = cst(c)->pend_mask != 0 || cst(c)->pend_scale != 1.0;
    const uint64_t base = tile_base(it % a.tiles, free_mask);
    const uint64_t nit = next_pass_item(it + G, total, G, ctl, a, gates, last_shot, last_active);
    const uint32_t nshot = (uint32_t)(nit / a.tiles);
    const uint64_t ngthr = nit < total ? tile_base(nit % a.tiles, free_mask) | tb : 0ull;
    run_phases<true>(tile, T, tid, nthr, flags, phases, a.phase_begin, a.phase_count, gates,
                           mats + (uint64_t)shot * mat_stride);
    {
      // back to HBM in the load layout (address bits computed once, above)
      CT* st = state + (uint64_t)shot * stride;
      const uint64_t gthr = base | tb;
      CT r[kR];
#pragma unroll
      for (int k = 0; k < kR; ++k) r[k] = tile[swz(tid + (uint32_t)k * nthr)];
#pragma unroll
      for (int k = 0; k < kR; ++k) {
        const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull) |
                            ((k & 8) ? h3 : 0ull);
        st[gi ^ F] = r[k];
      }
    }
    if (pending) {
      __syncthreads();
      if (tid == 0) {
        __threadfence();
        const uint32_t done = atomicAdd(&c->wg_done, 1u);
        if (done == a.tiles - 1) {
          c->pend_mask = 0;
          c->pend_val = 0;
          c->pend_scale = 1.0;
          c->wg_done = 0;
        }
      }
    }
    __syncthreads();
    if (nit < total) {
      // nit is a tile its shot has not finished, so that shot's pending
      // collapse is still in place
      const QSV_CONST ShotCtl* cn = cst(ctl + nshot);
      fetch16(nx, state + (uint64_t)nshot * stride, ngthr, h0, h1, h2, h3, a.init, cn->frame);
      stage16(tile, nx, tid, nthr, ngthr, h0, h1, h2, h3, cn->pend_mask, cn->pend_val, cn->pend_scale);
      __syncthreads();
    }
    it = nit;
  }
}

// Tile pass for passes made only of dense phases, on tiles of 2^t amplitudes
// (10 <= t <= 12), with 2^(t - 9) waves per tile: each thread stages and
// stores 8 amplitudes (load layout l = tid + k * 2^(t - 3)), each wave applies
// the phases to 2 blocks of 16 amplitude groups on the matrix cores, and at
// most 128 registers per thread let several workgroups share a CU (two of
// 2^12, three of 2^11, five of 2^10 amplitudes with their staged matrices),
// so that the waits of one workgroup (LDS, barriers, HBM) are covered by the
// others' matrix-core work. With
// lds_mats the pass's matrices (shared by every shot: mat_stride 0, at most
// kLdsDensePhases of them) are staged in LDS once; otherwise each phase reads
// its matrix from the shot's matrix slots.
template <typename CT>
__global__ __launch_bounds__(2 * kTileThreads, D8Waves<CT>::kMin) void k_tile_pass_d8(
    CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, const Phase* __restrict__ phases,
    const double* __restrict__ mats, uint64_t mat_stride, PassArgs a, uint32_t shots, uint32_t lds_mats) {
  extern __shared__ double2 qsv_lds[];
  CT* const tile = reinterpret_cast<CT*>(qsv_lds);
  constexpr uint32_t kA = 8;
  const uint32_t tid = threadIdx.x, T = 1u << a.t, lane = tid & 63u, nth = T / kA;  // nth = blockDim.x
  const uint64_t total = (uint64_t)a.tiles * shots, G = gridDim.x;
  const uint64_t free_mask = ~a.tile_mask & ((a.n >= 64) ? ~0ull : ((1ull << a.n) - 1ull));
  uint64_t tb = 0;  // this thread's bits over tile qubits tq[0..t-4]
  for (uint32_t b = 0; b + 3 < a.t; ++b) tb |= (uint64_t)((tid >> b) & 1u) << a.tq[b];
  const uint64_t h0 = 1ull << a.tq[a.t - 3], h1 = 1ull << a.tq[a.t - 2], h2 = 1ull << a.tq[a.t - 1];
  CT* const lmats = tile + T;
  if (lds_mats)
    for (uint32_t p = 0; p < a.phase_count; ++p) {
      const double2* src =
          reinterpret_cast<const double2*>(mats + (uint64_t)cst(phases + a.phase_begin + p)->dense * kMatStride);
      for (uint32_t e = tid; e < 256u; e += nth) lmats[p * 256u + e] = cmake<CT>(src[e].x, src[e].y);
    }
  // the first phases' descriptors, read once (wave-uniform, scalar registers):
  // every tile runs the same phases, and a descriptor read inside the tile
  // loop would make each phase wait for it, and for the matrix operand reads
  // issued with it, before any of its address work
  Phase pre[kLdsDensePhases];
  if constexpr (D8Waves<CT>::kPreload) {
#pragma unroll
    for (uint32_t p = 0; p < kLdsDensePhases; ++p)
      pre[p] = load_phase(phases + a.phase_begin + (p < a.phase_count ? p : 0u));
  }
  uint32_t last_shot = 0xFFFFFFFFu;
  bool last_active = false;
  uint64_t it = next_pass_item(blockIdx.x, total, G, ctl, a, nullptr, last_shot, last_active);
  while (it < total) {
    const uint32_t shot = (uint32_t)(it / a.tiles);
    ShotCtl* c = ctl + shot;
    const uint64_t F = cst(c)->frame, M = cst(c)->pend_mask, V = cst(c)->pend_val;
    const double sc = cst(c)->pend_scale;
    const bool pending = M != 0 || sc != 1.0;
    const uint64_t gthr = tile_base(it % a.tiles, free_mask) | tb;
    // amplitude k of this thread is at physical index (gthr | h_k) ^ F = lb + off(k):
    // flipping tile bit h moves by +h, or by -h where the frame holds that bit
    // (gthr never does), so the offsets are wave-uniform and only lb is per lane
    const int64_t d0 = (F & h0) ? -(int64_t)h0 : (int64_t)h0, d1 = (F & h1) ? -(int64_t)h1 : (int64_t)h1,
                  d2 = (F & h2) ? -(int64_t)h2 : (int64_t)h2;
    auto off = [&](int k) { return ((k & 1) ? d0 : 0) + ((k & 2) ? d1 : 0) + ((k & 4) ? d2 : 0); };
    CT* sp = state + (uint64_t)shot * stride + (gthr ^ F);
    CT r[kA];
#pragma unroll
    for (int k = 0; k < (int)kA; ++k) r[k] = a.init ? cmake<CT>(k == 0 && gthr == 0 ? 1.0 : 0.0, 0.0) : sp[off(k)];
#pragma unroll
    for (int k = 0; k < (int)kA; ++k) {
      const uint64_t gi = gthr | ((k & 1) ? h0 : 0ull) | ((k & 2) ? h1 : 0ull) | ((k & 4) ? h2 : 0ull);
      tile[swz(tid + (uint32_t)k * nth)] =
          !pending ? r[k] : (((gi & M) == V) ? cscale(r[k], sc) : cmake<CT>(0.0, 0.0));
    }
    __syncthreads();
    if (D8Waves<CT>::kPreload && lds_mats) {
      // staged matrices (at most kLdsDensePhases phases): descriptors and
      // operands from registers and LDS only
#pragma unroll
      for (uint32_t p = 0; p < kLdsDensePhases; ++p) {
        if (p >= a.phase_count) break;
        CT mf[4];
        load_mfrag(mf, true, lmats + (size_t)p * 256u, nullptr, lane);
        dense_phase_mfma<2>(tile, T, tid, pre[p], mf);
        __syncthreads();
      }
    } else {
      const double* ms = mats + (uint64_t)shot * mat_stride;
      for (uint32_t p = 0; p < a.phase_count; ++p) {
        const Phase ph = load_phase(phases + a.phase_begin + p);
        CT mf[4];
        load_mfrag(mf, lds_mats != 0u, lmats + (size_t)p * 256u,
                   reinterpret_cast<const double2*>(ms + (uint64_t)ph.dense * kMatStride), lane);
        dense_phase_mfma<2>(tile, T, tid, ph, mf);
        __syncthreads();
      }
    }
#pragma unroll
    for (int k = 0; k < (int)kA; ++k) r[k] = tile[swz(tid + (uint32_t)k * nth)];
#pragma unroll
    for (int k = 0; k < (int)kA; ++k) sp[off(k)] = r[k];
    if (pending) {
      __syncthreads();
      if (tid == 0) {
        __threadfence();
        const uint32_t done = atomicAdd(&c->wg_done, 1u);
        if (done == a.tiles - 1) {
          c->pend_mask = 0;
          c->pend_val = 0;
          c->pend_scale = 1.0;
          c->wg_done = 0;
        }
      }
    }
    // no barrier before the next tile: its staging writes go to the slots
    // swz(tid + k * nth) that this thread has just read for the stores
    // (one wave's LDS accesses complete in order), and the staging barrier
    // orders them before any other thread's reads
    it = next_pass_item(it + G, total, G, ctl, a, nullptr, last_shot, last_active);
  }
}

// ---------------------------------------------------------------------------
// complex64 all-dense tile pass: register steps (RegStep) on the matrix cores
// ---------------------------------------------------------------------------
// Position in a phase matrix (in operand order) of lane l's operand for kb = 0,
// M[row of l % 16][l / 16]; kb = 1..3 follow at distance 64. The row is l % 16
// with its bit pairs exchanged (see RegStep).
__device__ __forceinline__ uint32_t sp_pos(uint32_t l) { return (l & 48u) + ((l >> 2) & 3u) + ((l & 3u) << 2); }

// lane l's operand of a phase matrix for kb = 0..3: from the pass's staged
// copy (lane order), or from the matrix slots, rounded to single precision
template <bool kStaged>
__device__ __forceinline__ void sp_frag(float2 (&w)[4], const float2* __restrict__ lds_mat,
                                        const double* __restrict__ gmat, uint32_t lane) {
  typedef __attribute__((address_space(3))) const float lds_r;
  typedef __attribute__((address_space(1))) const double glb_d;
  if (kStaged) {
    const lds_r* l = (const lds_r*)lds_mat;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      w[kb].x = l[2 * (kb * 64 + (int)lane)];
      w[kb].y = l[2 * (kb * 64 + (int)lane) + 1];
    }
  } else {
    // a 32-bit offset per lane from a wave-uniform address
    const uint32_t e0 = 16u * sp_pos(lane);
#pragma unroll
    for (uint32_t kb = 0; kb < 4; ++kb) {
      const glb_d* g = (const glb_d*)((const __attribute__((address_space(1))) char*)gmat + (e0 + kb * 1024u));
      w[kb] = make_float2((float)g[0], (float)g[1]);
    }
  }
}

// The 4 x 256 amplitudes X + iY a wave holds: per lane, elements 0..3 of each
// block, real and imaginary parts apart, as the matrix cores leave them.
struct SpTile {
  qsv_f4 re[4], im[4];
};

// One phase on a wave's amplitudes in layout L(R, C): the matrix-core products
// with A + iB contract R and leave L(C, R). Each complex product is formed from
// three real ones, as in dense_phase_mfma and in the same order of sums:
// P1 = X A, P2 = Y B, P3 = (X + Y)(A + B), real = P1 - P2, imaginary = P3 - P1 - P2.
__device__ __forceinline__ void sp_contract(SpTile& x, const float2 (&w)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    qsv_f4 p1 = {0, 0, 0, 0}, p2 = {0, 0, 0, 0}, p3 = {0, 0, 0, 0};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      p1 = MfmaT<float2>::step(x.re[e][kb], w[kb].x, p1);
      p2 = MfmaT<float2>::step(x.im[e][kb], w[kb].y, p2);
      p3 = MfmaT<float2>::step(x.re[e][kb] + x.im[e][kb], w[kb].x + w[kb].y, p3);
    }
    x.re[e] = p1 - p2;
    x.im[e] = p3 - p1 - p2;
    // one block's three sums at a time (four waves per SIMD: 128 registers)
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A lane's bits 0..5 as masks (all ones where the bit is set).
struct SpLane {
  uint32_t m[6];
  __device__ __forceinline__ explicit SpLane(uint32_t lane) {
#pragma unroll
    for (int i = 0; i < 6; ++i) m[i] = 0u - ((lane >> i) & 1u);
  }
};
// A pass's steps, held by a wave: word i of step s in lane 16 (s % 4) + i of a
// register. A scalar load per step would stall the exchange between two steps
// for its latency (two exchanges per tile, timing copy of a complex128 build: 0.4
// of 8.4 ms).
static_assert(sizeof(RegStep) == 64, "a step is 16 words");
struct SpSteps {
  const uint32_t* p;
  uint32_t count, lane, d[2];
  __device__ __forceinline__ SpSteps(const RegStep* first, uint32_t n, uint32_t l)
      : p(reinterpret_cast<const uint32_t*>(first)), count(n), lane(l) {
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c) d[c] = c * 64u + l < count * 16u ? p[c * 64u + l] : 0u;
    // (here, before the tile loop, whose first use would otherwise wait for
    // every load in flight, the next tile's among them)
    asm volatile("" : "+v"(d[0]), "+v"(d[1]));
  }
  // the register that holds step s < count
  __device__ __forceinline__ uint32_t reg(uint32_t s) const {
    if (s < 4) return d[0];
    if (s < 8) return d[1];
    const uint32_t i = (s & ~3u) * 16u + lane;
    return i < count * 16u ? p[i] : 0u;
  }
};
__device__ __forceinline__ uint32_t sp_word(uint32_t reg, uint32_t s, uint32_t i) {
  return __builtin_amdgcn_readlane(reg, (s & 3u) * 16u + i);
}
constexpr uint32_t kSpOut = 0, kSpIn = 6, kSpMat = 12, kSpExchange = 13;  // words of a RegStep

// Byte offset in LDS of element k of block e of a lane in a layout (kSpIn or
// kSpOut of a step): a per-lane part (lane and wave bits) XOR a wave-uniform one.
struct SpAddr {
  uint32_t lane, b[4];
  __device__ __forceinline__ SpAddr(uint32_t reg, uint32_t s, uint32_t which, const SpLane& l, uint32_t wave) {
    uint32_t w[6], u = 0;
#pragma unroll
    for (uint32_t i = 0; i < 6; ++i) w[i] = sp_word(reg, s, which + i);
    auto bit = [&](int i) { return (i & 1) ? w[i >> 1] >> 16 : w[i >> 1] & 0xFFFFu; };
#pragma unroll
    for (int i = 0; i < 2; ++i) u ^= (0u - ((wave >> i) & 1u)) & bit(10 + i);
    lane = u;
#pragma unroll
    for (int i = 0; i < 6; ++i) lane ^= l.m[i] & bit(i);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = bit(6 + i);
  }
  __device__ __forceinline__ uint32_t at(int e, int k) const {
    uint32_t u = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) u ^= (((4 * e + k) >> i) & 1) ? b[i] : 0u;
    return lane ^ u;
  }
};
// The tile is at the start of a workgroup's LDS (no kernel that uses these has
// static LDS), so its byte offsets are LDS addresses.
__device__ __forceinline__ void sp_read(SpTile& x, const SpAddr& ad) {
  typedef float vec __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const vec v = *(const __attribute__((address_space(3))) vec*)(uintptr_t)ad.at(e, k);
      x.re[e][k] = v[0];
      x.im[e][k] = v[1];
    }
}
__device__ __forceinline__ void sp_write(const SpTile& x, const SpAddr& ad) {
  typedef __attribute__((address_space(3))) float lds_r;
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lds_r* p = (lds_r*)(uintptr_t)ad.at(e, k);
      p[0] = x.re[e][k];
      p[1] = x.im[e][k];
    }
}

// The work items (shot, tile) of an all-dense pass, for a workgroup that takes
// every step-th: an item's position holds the tile's index bits over the
// non-tile qubits and the shot's number above qubit n - 1, so that the next one
// is an addition whose carries pass over the tile's qubits. (Forming a tile's base
// bit by bit takes about 3000 cycles at 28 qubits, and sixteen-amplitude threads
// leave few waves to hide them.)
struct PassItem {
  uint64_t pos;
  uint32_t shot;
  uint64_t F, M, V;  // the shot's frame and pending collapse
  double sc;
};
struct PassItems {
  const ShotCtl* ctl;
  uint64_t tmask, step;
  uint32_t n, shots;
  __device__ __forceinline__ PassItems(const ShotCtl* c, const PassArgs& a, uint32_t s, uint32_t g)
      : ctl(c), tmask(a.tile_mask), step(tile_base(g, ~a.tile_mask)), n(a.n), shots(s) {}
  // w: the first item at or after w.pos (in steps) whose shot is alive; false past the last
  __device__ __forceinline__ bool seek(PassItem& w, uint32_t& known) const {
    for (;; w.pos = next(w.pos)) {
      w.shot = (uint32_t)(w.pos >> n);
      if (w.shot >= shots) return false;
      if (w.shot == known) return true;
      const QSV_CONST ShotCtl* c = cst(ctl + w.shot);
      if (c->status != 0) continue;
      known = w.shot;
      w.F = c->frame;
      w.M = c->pend_mask;
      w.V = c->pend_val;
      w.sc = c->pend_scale;
      return true;
    }
  }
  __device__ __forceinline__ uint64_t next(uint64_t pos) const { return ((pos | tmask) + step) & ~tmask; }
  __device__ __forceinline__ uint64_t base(const PassItem& w) const { return w.pos & ((1ull << n) - 1ull); }
  __device__ __forceinline__ bool first(PassItem& w, uint32_t& known) const {
    w.pos = tile_base(blockIdx.x, ~tmask);
    return seek(w, known);
  }
};

// Tiles of 2^t amplitudes (10 <= t <= 12), 2^(t - 10) waves per tile, sixteen
// amplitudes per thread, which stay in registers from one LDS exchange to the
// next: a tile comes straight from HBM and goes straight back, and LDS carries
// it only between register steps. With kStaged the pass's matrices (shared by
// every shot: mat_stride 0, at most kLdsDensePhases of them) are staged in LDS
// once, and the next tile's amplitudes are requested before the current tile's
// phases; otherwise each step requests the next one's operand from the shot's
// matrix slots. Up to four workgroups per CU (32 KiB tiles, 128 registers).
// Bound by the matrix cores and HBM in turn, at a clock that both pull down
// (25 qubits x 8 shots: 1.33 ms per four-phase pass, 1.51 with an LDS round
// trip per phase; 2.6 against 3.3 ms with nine phases).
template <bool kStaged>
__global__ __launch_bounds__(kTileThreads, 4) void k_tile_pass_c64(
    float2* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, const RegStep* __restrict__ reg_steps,
    const double* __restrict__ mats, uint64_t mat_stride, PassArgs a, uint32_t shots) {
  extern __shared__ double2 qsv_lds[];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SpLane lm(lane);
  const uint32_t N = a.step_count;
  const RegStep* const first = reg_steps + a.step_begin;
  const SpSteps steps(first, N, lane);
  float2* const lmats = reinterpret_cast<float2*>(qsv_lds) + (a.exchanges ? 1u << a.t : 0u);
  if (kStaged) {
    for (uint32_t s = 0, c = 0; s < N; ++s) {
      const uint32_t m = cst(first + s)->mat;
      if (m == kNoDense) continue;
      const double2* src = reinterpret_cast<const double2*>(mats + (uint64_t)m * kMatStride);
      for (uint32_t e = tid; e < 256u; e += blockDim.x) {
        const double2 v = src[(e & 192u) + sp_pos(e & 63u)];
        lmats[c * 256u + e] = make_float2((float)v.x, (float)v.y);
      }
      ++c;
    }
    __syncthreads();
  }
  // a thread's tile qubits in the layout whose global qubits are q
  auto thread_bits = [&](const uint8_t (&q)[kLayoutBits]) {
    uint64_t u = 0, g = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) u |= (uint64_t)((wave >> i) & 1u) << q[10 + i];
#pragma unroll
    for (int i = 0; i < 6; ++i) g |= (uint64_t)((lane >> i) & 1u) << q[i];
    return g | u;
  };
  const uint64_t gi = thread_bits(a.gin), go = thread_bits(a.gout);
  // Element i = 4 e + k of a thread is at physical index (g | h_i) ^ F =
  // (g ^ F) + off(i): flipping tile bit h moves by +h, or by -h where the frame
  // F holds that bit (g never does), so the offsets are wave-uniform.
  constexpr int kElems = 16;
  auto off = [&](const uint8_t (&q)[kLayoutBits], uint64_t F, int i) {
    int64_t d = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if ((i >> b) & 1) d += (int64_t)(((F >> q[6 + b]) & 1ull) ? ~0ull << q[6 + b] : 1ull << q[6 + b]);
    return d;
  };
  const PassItems items(ctl, a, shots, gridDim.x);
  // unstaged: a step's operand, requested a step ahead
  float2 wn[4];
  auto request = [&](uint32_t m, uint32_t shot) {  // (a step without a phase: any operand, not used)
    if (!kStaged)
      sp_frag<false>(wn, lmats, mats + (uint64_t)shot * mat_stride + (uint64_t)(m == kNoDense ? 0u : m) * kMatStride,
                     lane);
  };
  // staged: the next item's amplitudes, on their way while this one is worked on
  float2 nx[kElems];
  auto fetch = [&](const PassItem& w) {
    const float2* sp = state + (uint64_t)w.shot * stride + ((items.base(w) | gi) ^ w.F);
#pragma unroll
    for (int i = 0; i < kElems; ++i) nx[i] = sp[off(a.gin, w.F, i)];
  };
  uint32_t known = 0xFFFFFFFFu;  // the shot whose control block w holds
  PassItem w;
  if (!items.first(w, known)) return;
  request(sp_word(steps.d[0], 0, kSpMat), w.shot);
  if (kStaged && !a.init) fetch(w);
  for (;;) {
    const bool pending = w.M != 0 || w.sc != 1.0;
    const uint64_t g = items.base(w);
    PassItem nw = w;
    nw.pos = items.next(w.pos);
    const bool more = items.seek(nw, known);
    SpTile x;
    if (a.init) {
#pragma unroll
      for (int i = 0; i < kElems; ++i) {
        x.re[i >> 2][i & 3] = i == 0 && (g | gi) == 0 ? 1 : 0;
        x.im[i >> 2][i & 3] = 0;
      }
    } else {
      if (!kStaged) fetch(w);
#pragma unroll
      for (int i = 0; i < kElems; ++i) {
        x.re[i >> 2][i & 3] = nx[i].x;
        x.im[i >> 2][i & 3] = nx[i].y;
      }
      if (kStaged && more) fetch(nw);
    }
    if (pending) {
      const uint8_t(&q)[kLayoutBits] = a.gin;
      const uint64_t d = ((g | gi) & w.M) ^ w.V;  // the bits of M that the thread's amplitude 0 misses
#pragma unroll
      for (int i = 0; i < kElems; ++i) {
        uint64_t f = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) f |= ((i >> b) & 1) ? w.M & (1ull << q[6 + b]) : 0ull;
        x.re[i >> 2][i & 3] = d == f ? x.re[i >> 2][i & 3] * (float)w.sc : 0;
        x.im[i >> 2][i & 3] = d == f ? x.im[i >> 2][i & 3] * (float)w.sc : 0;
      }
    }
    uint32_t phase = 0;
    bool exchanged = false;
#pragma unroll 1
    for (uint32_t s = 0; s < N; ++s) {
      const uint32_t sr = steps.reg(s), m = sp_word(sr, s, kSpMat);
      float2 wf[4];
      if (!kStaged) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) wf[kb] = wn[kb];
        const bool last = s + 1 == N;
        request(last ? sp_word(steps.d[0], 0, kSpMat) : sp_word(steps.reg(s + 1), s + 1, kSpMat),
                last && more ? nw.shot : w.shot);
      }
      if (sp_word(sr, s, kSpExchange)) {
        const SpAddr out(sr, s, kSpOut, lm, wave);
        // a wave rewrites the slots it has read itself; only a tile's first
        // exchange follows other waves' reads (of the tile before)
        if (!exchanged) __syncthreads();
        exchanged = true;
        sp_write(x, out);
        const SpAddr in(sr, s, kSpIn, lm, wave);
        __syncthreads();
        sp_read(x, in);
      }
      if (m != kNoDense) {
        if (kStaged) sp_frag<true>(wf, lmats + 256u * phase++, nullptr, lane);
        sp_contract(x, wf);
      }
    }
    if (kStaged && !a.init && more) {
      // the next item is here before this one is stored: waiting for it later
      // would be waiting for the stores too
#pragma unroll
      for (int i = 0; i < kElems; ++i) asm volatile("" : "+v"(nx[i].x), "+v"(nx[i].y));
    }
    {
      float2* sp = state + (uint64_t)w.shot * stride + ((g | go) ^ w.F);
#pragma unroll
      for (int i = 0; i < kElems; ++i) {
        float2 v;
        v.x = x.re[i >> 2][i & 3];
        v.y = x.im[i >> 2][i & 3];
        sp[off(a.gout, w.F, i)] = v;
      }
    }
    if (pending) {
      __syncthreads();
      if (tid == 0) {
        ShotCtl* c = ctl + w.shot;
        __threadfence();
        const uint32_t n = atomicAdd(&c->wg_done, 1u);
        if (n == a.tiles - 1) {
          c->pend_mask = 0;
          c->pend_val = 0;
          c->pend_scale = 1.0;
          c->wg_done = 0;
        }
      }
    }
    if (!more) break;
    w = nw;
  }
}

// ---------------------------------------------------------------------------
// Measurement sites
// ---------------------------------------------------------------------------
// Histogram of |psi|^2 over the site's qubits (logical values), restricted to
// the pending collapse. Each workgroup covers a contiguous slice of the free
// (unrestricted) index space; every thread keeps its own 16 bins in LDS and
// the bins are summed in a fixed order, so the result does not depend on how
// many shots share the launch.
template <typename CT>
__device__ __forceinline__ double amp_prob(CT v, double s2) {
  const double vx = v.x, vy = v.y;
  return (vx * vx + vy * vy) * s2;
}

// The histogram of one block of one shot's state over the site's qubits (see
// k_site_reduce), summed in a fixed order; threads tid < kSiteBins return bin
// tid, the others 0. Every thread of the workgroup calls it (two barriers).
template <typename CT>
__device__ __forceinline__ double site_bins(const CT* __restrict__ state, uint64_t stride,
                                            const ShotCtl* __restrict__ c, const SiteArgs& a, uint32_t blk,
                                            uint64_t buf, uint32_t tid, double (*bins)[kRedThreads],
                                            double (*red)[kSiteBins]) {
  for (int b = 0; b < kSiteBins; ++b) bins[b][tid] = 0.0;
  if (c->status == 0) {
    const uint64_t M = c->pend_mask, F = c->frame, Vm = c->pend_val ^ (F & M);
    const double s2 = c->pend_scale * c->pend_scale;
    const uint32_t r = (uint32_t)__popcll(M);
    const uint64_t nfree = 1ull << (a.n - r);
    const uint64_t per = (nfree + a.blocks - 1) / a.blocks;
    const uint64_t j0 = per * blk, j1 = (j0 + per < nfree) ? j0 + per : nfree;
    const CT* st = state + buf * stride;
    uint32_t qbit[kSiteQubits];
    uint32_t fq = 0;
    for (uint32_t k = 0; k < a.nq; ++k) {
      qbit[k] = a.q[k];
      fq |= (uint32_t)((F >> a.q[k]) & 1ull) << k;
    }
    for (uint64_t j = j0 + tid; j < j1; j += kRedThreads) {
      uint64_t gi = j;
      if (M) {
        uint64_t mm = M;
        while (mm) {
          uint32_t b = __ffsll((long long)mm) - 1;
          mm &= mm - 1;
          gi = ins0_64(gi, b);
        }
        gi |= Vm;
      }
      const double p = amp_prob(st[gi], s2);
      uint32_t bin = 0;
      for (uint32_t k = 0; k < a.nq; ++k) bin |= (uint32_t)((gi >> qbit[k]) & 1ull) << k;
      bin ^= fq;
      bins[bin][tid] += p;
    }
  }
  __syncthreads();
  {
    const uint32_t b = tid & (kSiteBins - 1), part = tid / kSiteBins;
    double acc = 0.0;
    for (uint32_t k = 0; k < kSiteBins; ++k) acc += bins[b][part * kSiteBins + k];
    red[part][b] = acc;
  }
  __syncthreads();
  double acc = 0.0;
  if (tid < kSiteBins)
    for (uint32_t part = 0; part < kRedThreads / kSiteBins; ++part) acc += red[part][tid];
  return acc;
}

template <typename CT>
__global__ __launch_bounds__(kRedThreads) void k_site_reduce(
    const CT* __restrict__ state, uint64_t stride, const ShotCtl* __restrict__ ctl, SiteArgs a,
    double* __restrict__ partials, uint32_t pblocks, const uint32_t* __restrict__ buf_of) {
  __shared__ double bins[kSiteBins][kRedThreads];
  __shared__ double red[kRedThreads / kSiteBins][kSiteBins];
  const uint32_t shot = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
  const double v = site_bins(state, stride, ctl + shot, a, blk, buf_of ? buf_of[shot] : shot, tid, bins, red);
  if (tid < kSiteBins) partials[((uint64_t)shot * pblocks + blk) * kSiteBins + tid] = v;
}

// A classical expression (postfix code from code[pc] to its QSV_C_END) on one
// shot's classical bits, in 64-bit two's complement (include/qsv.h), by a wave
// whose lanes all do the same; s: kCStack words of LDS.
__device__ __forceinline__ int64_t cexec(const qsv_cop* __restrict__ code, uint64_t pc, const uint64_t* creg, int64_t* s) {
  int sp = 0;
  for (;; ++pc) {
    const qsv_cop c = code[pc];
    if (c.op == QSV_C_END) return s[sp - 1];
    if (c.op == QSV_C_IMM) {
      s[sp++] = c.imm;
      continue;
    }
    if (c.op == QSV_C_BITS) {
      uint64_t v = 0;
      for (uint32_t i = 0; i < c.width; ++i) {
        const uint32_t bit = c.lo + i;
        v |= ((creg[bit >> 6] >> (bit & 63)) & 1ull) << i;
      }
      if (c.sgn && c.width < 64 && ((v >> (c.width - 1)) & 1ull)) v |= ~0ull << c.width;
      s[sp++] = (int64_t)v;
      continue;
    }
    if (c.op == QSV_C_NEG || c.op == QSV_C_NOT || c.op == QSV_C_LNOT) {
      const uint64_t a = (uint64_t)s[sp - 1];
      s[sp - 1] = c.op == QSV_C_NEG ? (int64_t)(0ull - a) : c.op == QSV_C_NOT ? (int64_t)~a : (int64_t)(a == 0);
      continue;
    }
    const int64_t b = s[--sp], a = s[sp - 1];
    const uint64_t ua = (uint64_t)a, ub = (uint64_t)b;
    int64_t r;
    switch (c.op) {
      case QSV_C_ADD: r = (int64_t)(ua + ub); break;
      case QSV_C_SUB: r = (int64_t)(ua - ub); break;
      case QSV_C_MUL: r = (int64_t)(ua * ub); break;
      case QSV_C_DIV:  // truncation toward zero; INT64_MIN / -1 wraps to INT64_MIN
        r = b == 0 ? 0 : (b == -1 ? (int64_t)(0ull - ua) : a / b);
        break;
      case QSV_C_MOD: r = (b == 0 || b == -1) ? 0 : a % b; break;
      case QSV_C_AND: r = a & b; break;
      case QSV_C_OR: r = a | b; break;
      case QSV_C_XOR: r = a ^ b; break;
      case QSV_C_SHL: r = (b < 0 || b >= 64) ? 0 : (int64_t)(ua << b); break;
      case QSV_C_SHR: r = (b < 0 || b >= 64) ? (a < 0 ? -1 : 0) : (a >> b); break;
      case QSV_C_EQ: r = a == b; break;
      case QSV_C_NE: r = a != b; break;
      case QSV_C_LT: r = a < b; break;
      case QSV_C_GT: r = a > b; break;
      case QSV_C_LE: r = a <= b; break;
      case QSV_C_GE: r = a >= b; break;
      case QSV_C_LAND: r = (a != 0) && (b != 0); break;
      default: r = (a != 0) || (b != 0); break;
    }
    s[sp - 1] = r;
  }
}

// A comparison of a run of classical bits (not an expression).
__device__ __forceinline__ bool eval_cmp(const DPred& p, const uint64_t* creg) {
  if (p.cmp == QSV_CMP_TRUE) return true;
  uint64_t v = 0;
  for (uint32_t i = 0; i < p.width; ++i) {
    uint32_t bit = p.lo + i;
    v |= ((creg[bit >> 6] >> (bit & 63)) & 1ull) << i;
  }
  switch (p.cmp) {
    case QSV_CMP_EQ: return v == p.value;
    case QSV_CMP_NE: return v != p.value;
    case QSV_CMP_LT: return v < p.value;
    case QSV_CMP_GT: return v > p.value;
    case QSV_CMP_LE: return v <= p.value;
    default: return v >= p.value;
  }
}

__device__ __forceinline__ uint32_t uni32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) { return ((uint64_t)uni32((uint32_t)(v >> 32)) << 32) | uni32((uint32_t)v); }

// x of the lane r places on in its row of 16 (row_ror)
template <int r>
__device__ __forceinline__ double row_ror(double x) {
  uint64_t u;
  __builtin_memcpy(&u, &x, 8);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + r, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + r, 0xf, 0xf, false);
  u = ((uint64_t)hi << 32) | lo;
  __builtin_memcpy(&x, &u, 8);
  return x;
}
// The sum over the rows of 16 lanes, equal bit for bit in every lane of a row
// (each step adds the same two values in the two lanes that it joins).
__device__ __forceinline__ double row_sum(double x) {
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  x += row_ror<1>(x);
  return x;
}

// A shot's Philox words from `base` on: lane l of the wave holds words base + 4 l
// to base + 4 l + 3 (words of a block are drawn together), 256 in all once filled.
struct Draws {
  uint64_t w0, w1, w2, w3;
  uint32_t base, filled;
};
__device__ __forceinline__ uint64_t draw_word(const Draws& d, uint32_t e) {
  const uint32_t i = e - d.base;
  const uint64_t a = (i & 1u) ? d.w1 : d.w0, b = (i & 1u) ? d.w3 : d.w2, v = (i & 2u) ? b : a;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)(i >> 2));
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)(i >> 2));
  return ((uint64_t)hi << 32) | lo;
}

// The control block with its integers as wave-uniform values.
__device__ __forceinline__ ShotCtl load_ctl(const ShotCtl* p) {
  ShotCtl c = *p;
  c.flags = uni64(c.flags);
  c.pend_mask = uni64(c.pend_mask);
  c.pend_val = uni64(c.pend_val);
  c.frame = uni64(c.frame);
  c.n_events = uni32(c.n_events);
  c.n_record = uni32(c.n_record);
  c.status = (decltype(c.status))uni32((uint32_t)c.status);
  return c;
}

// The sequential events of a measurement site for one shot, given the
// histogram of |psi|^2 over the site's qubits (logical values, pending collapse
// applied; bin: that of bin l % 16 in lane l): Philox draws, outcomes (or
// forced ones), classical bits, flags, record, trajectory probability; then the
// site's collapse and flips are composed into the shot's pending collapse and
// flip frame. q4: the site's qubits, one a byte; stack: kCStack words of LDS.
//
// A whole wave runs it, every lane the same: a shot's events are one serial
// chain, so its cost is latency. Wave-uniform events are scalar loads (the next
// one's under way) and scalar branches, the sums over the bins four steps across
// a row instead of sixteen additions, and 64 lanes draw 256 words at once.
__device__ __forceinline__ void site_events(ShotCtl& cc, Draws& dr, double bin, uint32_t q4, const SiteEvent* ev,
                                            uint32_t ev_count, const DPred* preds, const qsv_cop* __restrict__ code,
                                            uint64_t* cr, uint8_t* rec, uint32_t max_record, const uint8_t* frow,
                                            uint32_t forced_len, uint64_t seed, uint64_t key1, double readout_err,
                                            double reset_err, int64_t* stack) {
  static_assert(sizeof(SiteEvent) == 24 && offsetof(SiteEvent, guard) == 16 && offsetof(SiteEvent, q) == 4, "words of SiteEvent");
  const uint32_t lane = __lane_id(), b = lane & (uint32_t)(kSiteBins - 1);
  uint32_t rm = 0, rv = 0;  // restriction on the bins (pre-site logical values)
  uint64_t xf = 0;          // flips applied during this site
  const double kZero = 0x1p-60;
  struct EvWords {
    uint32_t w0, w1, w2, w3;
    uint64_t guard;
  };
  auto fetch = [&](uint32_t e) {
    const QSV_CONST uint32_t* p = (const QSV_CONST uint32_t*)(ev + e);
    EvWords x;
    x.w0 = p[0];
    x.w1 = p[1];
    x.w2 = p[2];
    x.w3 = p[3];
    x.guard = ((const QSV_CONST uint64_t*)p)[2];
    return x;
  };
  EvWords nx = fetch(0);
  for (uint32_t e = 0; e < ev_count; ++e) {
    const EvWords E = nx;
    nx = fetch(e + 1 < ev_count ? e + 1 : e);
    const uint32_t op = E.w0 & 0xFFu, k = (E.w0 >> 8) & 0xFFu, flag = (E.w0 >> 16) & 0xFFu, q = E.w1,
                   cbit = E.w2;
    const bool active = guard_ok(cc.flags, E.guard);
    // (one place evaluates expressions, and its stack is the wave's: the code
    // stays small and free of scratch memory)
    DPred pr = {0, 0, 0, QSV_CMP_TRUE, 0};
    if (active && op == SE_SETF) {
      const QSV_CONST DPred* pp = cst(preds + E.w3);
      pr.lo = pp->lo;
      pr.width = pp->width;
      pr.value = pp->value;
      pr.cmp = pp->cmp;
    }
    int64_t x = 0;
    if (active && (op == SE_CSTORE || pr.cmp == QSV_CMP_EXPR))
      x = (int64_t)uni64((uint64_t)cexec(code, op == SE_CSTORE ? E.w3 : pr.value, cr, stack));
    if (op == SE_SETF) {
      const bool v = active && (pr.cmp == QSV_CMP_EXPR ? x != 0 : uni32(eval_cmp(pr, cr) ? 1u : 0u) != 0u);
      cc.flags = (cc.flags & ~(1ull << flag)) | ((uint64_t)v << flag);
      continue;
    }
    if (!active) continue;
    if (op == SE_CLRF) {
      cc.flags &= ~(1ull << flag);
    } else if (op == SE_SETB || op == SE_CLRB) {  // classical assignment of one bit
      const uint64_t m = 1ull << (cbit & 63u), o = cr[cbit >> 6];
      cr[cbit >> 6] = (op == SE_SETB) ? (o | m) : (o & ~m);
    } else if (op == SE_CSTORE) {  // classical assignment of a computed value
      const uint64_t v = (uint64_t)x;
      for (uint32_t i = 0; i < flag; ++i) {
        const uint32_t bit = cbit + i;
        const uint64_t m = 1ull << (bit & 63u), o = cr[bit >> 6];
        cr[bit >> 6] = ((v >> i) & 1ull) ? (o | m) : (o & ~m);
      }
    } else if (op == SE_X) {
      xf ^= 1ull << q;
    } else {  // measure or reset
      if (!dr.filled || cc.n_events + 2u > dr.base + 256u) {
        dr.base = cc.n_events & ~3u;
        dr.filled = 1u;
        dr.w0 = (uint64_t)(dr.base / 4u) + 1u + lane;
        dr.w1 = dr.w2 = dr.w3 = 0;
        philox_block(dr.w0, dr.w1, dr.w2, dr.w3, seed, key1);
      }
      const uint32_t fq = (uint32_t)((xf >> q) & 1ull), side = ((b >> k) & 1u) ^ fq;
      const double v = (b & rm) == rv ? bin : 0.0;
      const double p0 = row_sum(side ? 0.0 : v), p1 = row_sum(side ? v : 0.0);
      const double norm = p0 + p1, f0 = p0 / norm;
      const double u = (double)(draw_word(dr, cc.n_events) >> 11) * 0x1p-53;
      cc.n_events++;
      uint32_t o;
      double fo;
      if (op == SE_MEASURE && frow && cc.n_record < forced_len) {
        o = uni32(frow[cc.n_record] ? 1u : 0u);
        fo = o ? p1 / norm : f0;
        if (uni32(fo < kZero ? 1u : 0u)) {
          cc.status = QSV_ERR_FORCED_ZERO_PROB;
          return;
        }
      } else {
        o = uni32(u < f0 ? 0u : 1u);
        fo = o ? p1 / norm : f0;
      }
      cc.record_prob *= fo;
      rm |= 1u << k;
      rv |= (o ^ fq) << k;
      if (op == SE_MEASURE) {
        // readout error: the next word flips the recorded bit (the state keeps o)
        uint32_t r = o;
        if (readout_err > 0.0) {
          r ^= (double)(draw_word(dr, cc.n_events) >> 11) * 0x1p-53 < readout_err ? 1u : 0u;
          r = uni32(r);
          cc.n_events++;
        }
        if (cc.n_record < max_record) rec[cc.n_record] = (uint8_t)r;
        cc.n_record++;
        if (cbit != 0xFFFFFFFFu) {
          const uint64_t bitm = 1ull << (cbit & 63u), old = cr[cbit >> 6];
          cr[cbit >> 6] = r ? (old | bitm) : (old & ~bitm);
        }
      } else {
        if (o) xf ^= 1ull << q;  // reset: flip the qubit back to |0>
        // reset error: the next word leaves the qubit flipped
        if (reset_err > 0.0) {
          if (uni32((double)(draw_word(dr, cc.n_events) >> 11) * 0x1p-53 < reset_err ? 1u : 0u)) xf ^= 1ull << q;
          cc.n_events++;
        }
      }
    }
  }
  // compose the site's collapse with the incoming one (all in logical frames)
  uint64_t R = 0, RV = 0;
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kSiteQubits; ++k)
    if (rm >> k & 1u) {
      const uint32_t q = (q4 >> (8u * k)) & 63u;
      R |= 1ull << q;
      RV |= (uint64_t)((rv >> k) & 1u) << q;
    }
  if (rm) cc.pend_scale = cc.pend_scale / sqrt(row_sum((b & rm) == rv ? bin : 0.0));
  const uint64_t M = cc.pend_mask;
  cc.pend_val = ((cc.pend_val ^ (xf & M)) & M) | ((RV ^ (xf & R)) & R);
  cc.pend_mask = M | R;
  cc.frame ^= xf;
}

__device__ __forceinline__ uint32_t site_q4(const SiteArgs& a) {
  uint32_t w;
  __builtin_memcpy(&w, a.q, 4);
  return w;
}

// The site's events for one shot from its bins (bin l % 16 in lane l), by one wave.
__device__ __forceinline__ void finalize_shot(ShotCtl* __restrict__ c, double bin,
                                              const SiteArgs& a, const SiteEvent* __restrict__ ev,
                                              const DPred* __restrict__ preds, const qsv_cop* __restrict__ code,
                                              uint64_t* __restrict__ creg, uint32_t cw, uint8_t* __restrict__ record,
                                              uint32_t max_record, const uint8_t* __restrict__ forced,
                                              uint32_t forced_len, uint64_t seed, uint64_t shot_base, uint32_t shot,
                                              double readout_err, double reset_err,
                                              const uint64_t* __restrict__ key, int64_t* stack) {
  ShotCtl cc = load_ctl(c);
  if (cc.status != 0) return;
  if (key) {
    seed = cst(key)[0];
    shot_base = cst(key)[1];
  }
  Draws dr;
  dr.filled = 0;
  dr.base = 0;
  site_events(cc, dr, bin, site_q4(a), ev + a.ev_begin, a.ev_count, preds, code, creg + (uint64_t)shot * cw,
              record + (uint64_t)shot * max_record, max_record,
              forced ? forced + (uint64_t)shot * forced_len : nullptr, forced_len, seed, shot_base + shot, readout_err,
              reset_err, stack);
  if (__lane_id() == 0) *c = cc;
}

__global__ __launch_bounds__(64) void k_site_finalize(
    ShotCtl* __restrict__ ctl, SiteArgs a, const SiteEvent* __restrict__ ev,
    const DPred* __restrict__ preds, const qsv_cop* __restrict__ code, const double* __restrict__ partials,
    uint32_t pblocks,
    uint64_t* __restrict__ creg,
    uint32_t cw, uint8_t* __restrict__ record, uint32_t max_record, const uint8_t* __restrict__ forced,
    uint32_t forced_len, uint64_t seed, uint64_t shot_base, const uint32_t* __restrict__ slot_of, double readout_err,
    double reset_err, const uint64_t* __restrict__ key) {
  __shared__ double part[4][kSiteBins];
  __shared__ int64_t stack[kCStack];
  const uint32_t shot = blockIdx.x, tid = threadIdx.x;
  ShotCtl* c = ctl + shot;
  if (a.nq) {
    const double* pp = partials + (uint64_t)(slot_of ? slot_of[shot] : shot) * pblocks * kSiteBins;
    const uint32_t b = tid & (kSiteBins - 1), q = tid / kSiteBins;
    double acc = 0.0;
    // (one wave and up to kRedMaxBlocks / 4 additions in order: 16 loads at a time)
    uint32_t k = q;
    for (; k + 60u < a.blocks; k += 64) {
      double x[16];
#pragma unroll
      for (uint32_t m = 0; m < 16; ++m) x[m] = pp[(uint64_t)(k + 4u * m) * kSiteBins + b];
#pragma unroll
      for (uint32_t m = 0; m < 16; ++m) acc += x[m];
    }
    for (; k < a.blocks; k += 4) acc += pp[(uint64_t)k * kSiteBins + b];
    part[q][b] = acc;
  }
  __syncthreads();
  const uint32_t b = tid & (kSiteBins - 1);
  const double bin = a.nq ? ((part[0][b] + part[1][b]) + part[2][b]) + part[3][b] : 0.0;
  finalize_shot(c, bin, a, ev, preds, code, creg, cw, record, max_record, forced, forced_len, seed, shot_base, shot,
                readout_err, reset_err, key, stack);
}

// Both steps of a site whose histogram takes one block (states of up to 14
// qubits) and whose shots own their states: one workgroup per shot builds the
// bins as k_site_reduce does and its first thread runs the events. The bins
// equal those of the two launches (there each is the one block's sum plus
// three zeros).
template <typename CT>
__global__ __launch_bounds__(kRedThreads) void k_site_fused(
    const CT* __restrict__ state, uint64_t stride, ShotCtl* __restrict__ ctl, SiteArgs a,
    const SiteEvent* __restrict__ ev, const DPred* __restrict__ preds, const qsv_cop* __restrict__ code,
    uint64_t* __restrict__ creg, uint32_t cw, uint8_t* __restrict__ record, uint32_t max_record,
    const uint8_t* __restrict__ forced, uint32_t forced_len, uint64_t seed, uint64_t shot_base,
    const uint32_t* __restrict__ buf_of, double readout_err, double reset_err, const uint64_t* __restrict__ key) {
  __shared__ double bins[kSiteBins][kRedThreads];
  __shared__ double red[kRedThreads / kSiteBins][kSiteBins];
  __shared__ double fin[kSiteBins];
  __shared__ int64_t stack[kCStack];
  const uint32_t shot = blockIdx.x, tid = threadIdx.x;
  ShotCtl* c = ctl + shot;
  const double v = site_bins(state, stride, c, a, 0u, buf_of ? buf_of[shot] : shot, tid, bins, red);
  if (tid < kSiteBins) fin[tid] = v;
  __syncthreads();
  if (tid >= 64) return;
  finalize_shot(c, fin[tid & (kSiteBins - 1)], a, ev, preds, code, creg, cw, record, max_record, forced, forced_len, seed, shot_base, shot,
                readout_err, reset_err, key, stack);
}

hipError_t launch_site(const RunBuffers& rb, const SiteArgs& a, const SiteEvent* ev, const DPred* preds,
                       const qsv_cop* code, hipStream_t st) {
  if (a.nq && a.blocks == 1 && !rb.slot_of) {
    if (rb.c64)
      hipLaunchKernelGGL(k_site_fused<float2>, dim3(rb.shots), dim3(kRedThreads), 0, st,
                         reinterpret_cast<const float2*>(rb.state), rb.stride, rb.ctl, a, ev, preds, code, rb.creg,
                         rb.cw, rb.record, rb.max_record, rb.forced, rb.forced_len, rb.seed, rb.shot_base, rb.buf_of,
                         rb.readout_err, rb.reset_err, rb.key);
    else
      hipLaunchKernelGGL(k_site_fused<double2>, dim3(rb.shots), dim3(kRedThreads), 0, st, rb.state, rb.stride, rb.ctl,
                         a, ev, preds, code, rb.creg, rb.cw, rb.record, rb.max_record, rb.forced, rb.forced_len,
                         rb.seed, rb.shot_base, rb.buf_of, rb.readout_err, rb.reset_err, rb.key);
    return hipGetLastError();
  }
  if (a.nq) {
    // with trajectory sharing the histograms are taken per slot (slot control
    // blocks in site_ctl), the outcomes per shot
    const dim3 grid(a.blocks, rb.slot_of ? rb.site_slots : rb.shots);
    const ShotCtl* hc = rb.slot_of ? rb.site_ctl : rb.ctl;
    if (rb.c64)
      hipLaunchKernelGGL(k_site_reduce<float2>, grid, dim3(kRedThreads), 0, st,
                         reinterpret_cast<const float2*>(rb.state), rb.stride, hc, a, rb.partials, rb.pblocks,
                         rb.buf_of);
    else
      hipLaunchKernelGGL(k_site_reduce<double2>, grid, dim3(kRedThreads), 0, st, rb.state, rb.stride, hc, a,
                         rb.partials, rb.pblocks, rb.buf_of);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_site_finalize, dim3(rb.shots), dim3(64), 0, st, rb.ctl, a, ev, preds, code, rb.partials,
                     rb.pblocks, rb.creg, rb.cw, rb.record, rb.max_record, rb.forced, rb.forced_len, rb.seed,
                     rb.shot_base, rb.slot_of, rb.readout_err, rb.reset_err, rb.key);
  return hipGetLastError();
}

__global__ void k_ctl_gather(ShotCtl* __restrict__ dst, const ShotCtl* __restrict__ src,
                             const uint32_t* __restrict__ idx, uint32_t count) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[idx[i]];
}

hipError_t launch_ctl_gather(ShotCtl* dst, const ShotCtl* src, const uint32_t* idx, uint32_t count, hipStream_t st) {
  if (!count) return hipSuccess;
  hipLaunchKernelGGL(k_ctl_gather, dim3((count + 255) / 256), dim3(256), 0, st, dst, src, idx, count);
  return hipGetLastError();
}

// Copy-on-write of trajectory slots: buffer pairs[2k] takes the amplitudes of
// buffer pairs[2k + 1]. Sources are never destinations in one launch.
template <typename CT>
__global__ void k_buf_copy(CT* __restrict__ state, uint64_t stride, uint64_t dim,
                           const uint32_t* __restrict__ pairs, uint32_t n_pairs) {
  const uint64_t total = dim * n_pairs;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t k = i / dim, j = i % dim;
    state[(uint64_t)pairs[2 * k] * stride + j] = state[(uint64_t)pairs[2 * k + 1] * stride + j];
  }
}

hipError_t launch_buf_copy(double2* state, uint64_t stride, uint32_t n, const uint32_t* pairs, uint32_t n_pairs,
                           hipStream_t st, bool c64) {
  if (!n_pairs) return hipSuccess;
  const uint64_t total = (1ull << n) * n_pairs;
  uint64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (c64)
    hipLaunchKernelGGL(k_buf_copy<float2>, dim3((uint32_t)blocks), dim3(256), 0, st, reinterpret_cast<float2*>(state),
                       stride, 1ull << n, pairs, n_pairs);
  else
    hipLaunchKernelGGL(k_buf_copy<double2>, dim3((uint32_t)blocks), dim3(256), 0, st, state, stride, 1ull << n, pairs,
                       n_pairs);
  return hipGetLastError();
}

// Plain streaming copy (calibration of hardware byte counters).
__global__ void k_copy(double2* __restrict__ dst, const double2* __restrict__ src, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, uint64_t bytes, hipStream_t st) {
  const uint64_t n = bytes / 16;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3((uint32_t)blocks), dim3(256), 0, st, static_cast<double2*>(dst),
                     static_cast<const double2*>(src), n);
  return hipGetLastError();
}

// The logical state of one shot: psi[i] = cond(i) ? mem[i ^ frame] * scale : 0,
// as complex128 whatever the amplitude type.
template <typename CT>
__global__ void k_materialize(const CT* __restrict__ state, uint64_t stride, const ShotCtl* ctl,
                              uint32_t shot, uint64_t dim, double2* __restrict__ out) {
  const ShotCtl c = ctl[shot];
  const CT* st = state + (uint64_t)shot * stride;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
       i += (uint64_t)gridDim.x * blockDim.x) {
    double2 v = make_double2(0.0, 0.0);
    if ((i & c.pend_mask) == c.pend_val) {
      const CT x = st[i ^ c.frame];
      v = cscale(make_double2(x.x, x.y), c.pend_scale);
    }
    out[i] = v;
  }
}

hipError_t launch_materialize(const RunBuffers& rb, uint32_t n, uint32_t shot, double2* out, hipStream_t st) {
  uint64_t dim = 1ull << n;
  uint64_t blocks = (dim + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (rb.c64)
    hipLaunchKernelGGL(k_materialize<float2>, dim3((uint32_t)blocks), dim3(256), 0, st,
                       reinterpret_cast<const float2*>(rb.state), rb.stride, rb.ctl, shot, dim, out);
  else
    hipLaunchKernelGGL(k_materialize<double2>, dim3((uint32_t)blocks), dim3(256), 0, st, rb.state, rb.stride, rb.ctl,
                       shot, dim, out);
  return hipGetLastError();
}


__global__ void k_zero_u32(uint32_t* p, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Persistent interpreter: one launch runs every shot of every request.
//
// Workgroups pop work items (request, shot) from an atomic counter until the
// queue is empty, so trajectories of uneven length (loop exits, taken
// branches) and circuits of different widths share one launch. A state of
// n <= 12 qubits stays in LDS from the first gate to the last measurement; a
// larger one lives in the workgroup's HBM slot and every pass streams it tile
// by tile. Each item is processed by one workgroup in a fixed order, so its
// results do not depend on what else is in the batch.
// ---------------------------------------------------------------------------
// Deterministic workgroup sum of 16 per-thread bins (wave shuffles, then waves in order).
__device__ void wg_bins(double (&acc)[kSiteBins], double* red /* [4][16] in LDS */, double* out /* [16] */) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
#pragma unroll
  for (int b = 0; b < kSiteBins; ++b) {
    double v = acc[b];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) red[wave * kSiteBins + b] = v;
  }
  __syncthreads();
  if (tid < (uint32_t)kSiteBins) {
    double v = 0.0;
    for (uint32_t w = 0; w < blockDim.x / 64u; ++w) v += red[w * kSiteBins + tid];
    out[tid] = v;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kTileThreads) void k_persistent(
    const ReqDev* __restrict__ reqs, const uint32_t* __restrict__ item_req, uint32_t n_items,
    uint32_t* __restrict__ queue, double2* __restrict__ scratch, uint64_t slot_amps, ShotCtl* __restrict__ out_ctl,
    uint64_t* __restrict__ out_creg, uint32_t cw, uint8_t* __restrict__ out_rec, uint32_t rec_max) {
  extern __shared__ double2 tile[];
  __shared__ ShotCtl cs;
  __shared__ int64_t stack[kCStack];
  // algorithmic HBM bytes of the streamed (HBM-slot) states, summed over the
  // launch for the profile: queue[2..3] as one 64-bit counter
  unsigned long long* const hbm_bytes = reinterpret_cast<unsigned long long*>(queue + 2);
  __shared__ uint32_t item_s;
  __shared__ double red[4 * kSiteBins];
  __shared__ double bins[kSiteBins];
  const uint32_t tid = threadIdx.x;
  double2* const wg_slot = scratch + (uint64_t)blockIdx.x * slot_amps;
  for (;;) {
    if (tid == 0) item_s = atomicAdd(queue, 1u);
    __syncthreads();
    const uint32_t item = item_s;
    if (item >= n_items) break;  // every workgroup reaches this once the queue is drained
    const ReqDev R = reqs[item_req[item]];
    const uint32_t shot = item - R.item_begin, n = R.n;
    const bool resident = n <= (uint32_t)kResidentMaxBits;
    double2* const slot = R.state_out ? reinterpret_cast<double2*>(R.state_out) : wg_slot;
    const double2* const init_state = reinterpret_cast<const double2*>(R.init_state);
    uint64_t* cr = out_creg + (uint64_t)item * cw;
    uint8_t* rec = out_rec + (uint64_t)item * rec_max;
    for (uint32_t w = tid; w < cw; w += blockDim.x) cr[w] = R.init_creg ? R.init_creg[w] : 0ull;
    for (uint32_t w = tid; w < rec_max; w += blockDim.x) rec[w] = 0;
    if (tid == 0) {
      ShotCtl c;
      if (R.init_ctl) {
        c = *R.init_ctl;
      } else {
        c.flags = 0;
        c.pend_mask = 0;
        c.pend_val = 0;
        c.frame = 0;
        c.pend_scale = 1.0;
        c.record_prob = 1.0;
        c.n_events = 0;
        c.n_record = 0;
        c.status = 0;
      }
      c.wg_done = 0;
      cs = c;
    }
    const uint64_t dim = 1ull << n;
    if (init_state) {  // the request's shared prefix, computed once
      if (resident) {
        for (uint32_t l = tid; l < (uint32_t)dim; l += blockDim.x) tile[swz(l)] = init_state[l];
      } else {
        for (uint64_t j = tid; j < dim; j += blockDim.x) slot[j] = init_state[j];
        if (tid == 0) atomicAdd(hbm_bytes, 32ull * dim);
      }
    }
    __syncthreads();
    for (uint32_t k = R.step_begin; k < R.n_steps; ++k) {
      if (cs.status != 0) break;
      const DStep stp = R.steps[k];
      const uint64_t flags = cs.flags;
      if (stp.kind == 0) {  // |0...0>
        if (resident) {
          for (uint32_t l = tid; l < (uint32_t)dim; l += blockDim.x) tile[swz(l)] = make_double2(l == 0 ? 1.0 : 0.0, 0.0);
        } else {
          for (uint64_t j = tid; j < dim; j += blockDim.x) slot[j] = make_double2(j == 0 ? 1.0 : 0.0, 0.0);
          if (tid == 0) atomicAdd(hbm_bytes, 16ull * dim);
        }
        __syncthreads();
      } else if (stp.kind == 1) {  // gate pass
        const PassArgs a = R.passes[stp.index];
        bool any = a.init != 0 || (a.guard && guard_ok(flags, a.guard));
        for (uint32_t i = 0; !a.guard && i < a.gate_count && !any; ++i)
          any = guard_ok(flags, R.gates[a.gate_begin + i].guard);
        if (!any) continue;
        if (resident) {
          if (a.init) {
            for (uint32_t l = tid; l < (uint32_t)dim; l += blockDim.x) tile[swz(l)] = make_double2(l == 0 ? 1.0 : 0.0, 0.0);
            __syncthreads();
          }
          if (a.phase_count) {
            run_phases<true>(tile, (uint32_t)dim, tid, (uint32_t)dim >> kRegBits, flags, R.phases, a.phase_begin,
                       a.phase_count, R.gates, R.mats);
          } else {
            // fewer than 4 qubits: one LDS sweep per gate (slots are unswizzled for T < 16)
            for (uint32_t i = 0; i < a.gate_count; ++i) {
              const DGate g = R.gates[a.gate_begin + i];
              if (!guard_ok(flags, g.guard)) continue;
              tile_apply(tile, a.t, g, R.mats + (uint64_t)g.mat * kMatStride);
              __syncthreads();
            }
          }
        } else {
          // stream the HBM slot tile by tile; the pending collapse and frame
          // apply on staging. The 16 loads per thread of the next tile are
          // issued before the current tile's phases run (tiles of one pass
          // are disjoint), so they overlap its gate arithmetic.
          const uint64_t M = cs.pend_mask, V = cs.pend_val, F = cs.frame;
          const double sc = cs.pend_scale;
          const uint32_t T = 1u << a.t, nthr = T >> kRegBits;
          uint64_t tb = 0;  // this thread's bits over tile qubits tq[0..t-5]
          for (uint32_t b = 0; b + kRegBits < a.t; ++b) tb |= (uint64_t)((tid >> b) & 1u) << a.tq[b];
          const uint64_t h0 = 1ull << a.tq[a.t - 4], h1 = 1ull << a.tq[a.t - 3], h2 = 1ull << a.tq[a.t - 2],
                         h3 = 1ull << a.tq[a.t - 1];
          const uint64_t free_mask = ~a.tile_mask & ((n >= 64) ? ~0ull : ((1ull << n) - 1ull));
          double2 nx[kR];
          if (tid < nthr) fetch16(nx, slot, tile_base(0, free_mask) | tb, h0, h1, h2, h3, a.init != 0, F);
          for (uint32_t w = 0; w < a.tiles; ++w) {
            const uint64_t gthr = tile_base(w, free_mask) | tb;
            if (tid < nthr) stage16(tile, nx, tid, nthr, gthr, h0, h1, h2, h3, M, V, sc);
            __syncthreads();
            if (w + 1 < a.tiles && tid < nthr)
              fetch16(nx, slot, tile_base(w + 1, free_mask) | tb, h0, h1, h2, h3, a.init != 0, F);
            run_phases<true>(tile, T, tid, nthr, flags, R.phases, a.phase_begin, a.phase_count, R.gates, R.mats);
            if (tid < nthr) store_tile16(tile, slot, a, tile_base(w, free_mask), tid, F);
            __syncthreads();
          }
          if (tid == 0) {
            cs.pend_mask = 0;
            cs.pend_val = 0;
            cs.pend_scale = 1.0;
            atomicAdd(hbm_bytes, 32ull * dim);
          }
          __syncthreads();
        }
      } else {  // measurement site
        const SiteArgs sa = R.sites[stp.index];
        if (sa.nq) {
          double acc[kSiteBins];
#pragma unroll
          for (int b = 0; b < kSiteBins; ++b) acc[b] = 0.0;
          const uint64_t M = cs.pend_mask, V = cs.pend_val, F = cs.frame;
          const double s2 = cs.pend_scale * cs.pend_scale;
          const uint32_t r = (uint32_t)__popcll(M);
          const uint64_t nfree = 1ull << (n - r);
          for (uint64_t j = tid; j < nfree; j += blockDim.x) {
            uint64_t gi = j;
            if (M) {
              uint64_t mm = M;
              while (mm) {
                const uint32_t b = __ffsll((long long)mm) - 1;
                mm &= mm - 1;
                gi = ins0_64(gi, b);
              }
              gi |= V;
            }
            const double2 v = resident ? tile[swz((uint32_t)(gi ^ F))] : slot[gi ^ F];
            const double p = (v.x * v.x + v.y * v.y) * s2;
            uint32_t bin = 0;
            for (uint32_t q = 0; q < sa.nq; ++q) bin |= (uint32_t)((gi >> sa.q[q]) & 1ull) << q;
#pragma unroll
            for (int b = 0; b < kSiteBins; ++b) acc[b] += (bin == (uint32_t)b) ? p : 0.0;
          }
          wg_bins(acc, red, bins);
          if (!resident && tid == 0) atomicAdd(hbm_bytes, 16ull * nfree);
        }
        if (tid < 64) {
          ShotCtl c = load_ctl(&cs);
          Draws dr;
          dr.filled = 0;
          dr.base = 0;
          site_events(c, dr, sa.nq ? bins[tid & (kSiteBins - 1)] : 0.0, site_q4(sa), R.events + sa.ev_begin, sa.ev_count,
                      R.preds, R.code, cr, rec, rec_max, R.forced ? R.forced + (uint64_t)shot * R.forced_len : nullptr,
                      R.forced_len, R.seed, R.shot_offset + shot, R.readout_err, R.reset_err, stack);
          if (tid == 0) cs = c;
        }
        __syncthreads();
        if (resident && (cs.pend_mask != 0 || cs.pend_scale != 1.0 || cs.frame != 0)) {
          // materialise the collapse and the flips in LDS: psi[i] = cond(i) ? mem[i ^ F] * s : 0
          const uint64_t M = cs.pend_mask, V = cs.pend_val, F = cs.frame;
          const double sc = cs.pend_scale;
          for (uint32_t l = tid; l < (uint32_t)dim; l += blockDim.x) {
            const uint32_t m = l ^ (uint32_t)F;
            if (m < l) continue;  // each pair (l, l ^ F) is handled by its smaller index
            const double2 a0 = tile[swz(l)], a1 = tile[swz(m)];
            tile[swz(l)] = ((l & M) == V) ? cscale(a1, sc) : make_double2(0.0, 0.0);
            if (m != l) tile[swz(m)] = ((m & M) == V) ? cscale(a0, sc) : make_double2(0.0, 0.0);
          }
          __syncthreads();
          if (tid == 0) {
            cs.pend_mask = 0;
            cs.pend_val = 0;
            cs.pend_scale = 1.0;
            cs.frame = 0;
          }
          __syncthreads();
        }
      }
    }
    if (R.state_out && resident)
      for (uint32_t l = tid; l < (uint32_t)dim; l += blockDim.x) slot[l] = tile[swz(l)];
    if (tid == 0) out_ctl[item] = cs;
    __syncthreads();
  }
}

hipError_t launch_persistent(const ReqDev* reqs, const uint32_t* item_req, uint32_t n_items, uint32_t* queue,
                             double2* scratch, uint64_t slot_amps, uint32_t workgroups, ShotCtl* out_ctl,
                             uint64_t* out_creg, uint32_t cw, uint8_t* out_rec, uint32_t rec_max, hipStream_t st) {
  if (!n_items) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, st, queue, 4u);  // queue head and byte counter
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = sizeof(double2) << kResidentMaxBits;
  hipLaunchKernelGGL(k_persistent, dim3(workgroups), dim3(kTileThreads), lds, st, reqs, item_req, n_items, queue,
                     scratch, slot_amps, out_ctl, out_creg, cw, out_rec, rec_max);
  return hipGetLastError();
}

// One gate pass of many different programs' states at once, a workgroup a tile
// (see PassUnit): the deterministic prefixes of a batch, which as one persistent
// item per request left most of the chip idle behind the widest one. The tile is
// staged, run and stored as the persistent kernel does it (same results bit for
// bit). Bound by the chain of phases of a tile, a few hundred tiles a round.
// 17 prefixes of 13 to 17 qubits, 12 layers and the first body of a loop: 4.47
// ms as persistent items, 0.27 ms in 9 rounds.
__global__ __launch_bounds__(kTileThreads) void k_pass_units(const PassUnit* __restrict__ units, uint32_t n_units) {
  extern __shared__ double2 qsv_lds[];
  double2* const tile = qsv_lds;
  const uint32_t tid = threadIdx.x;
  uint32_t lo = 0, hi = n_units;  // the last unit whose tile_begin <= blockIdx.x
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (cst(units + mid)->tile_begin <= blockIdx.x) lo = mid;
    else hi = mid;
  }
  const QSV_CONST PassUnit* u = cst(units + lo);
  double2* const st = reinterpret_cast<double2*>(u->state);
  if (!u->pass) {
    const uint64_t at = ((uint64_t)blockIdx.x - u->tile_begin) << kTileMaxBits;
    for (uint32_t l = tid; l < (1u << kTileMaxBits); l += kTileThreads)
      st[at + l] = make_double2(at + l == 0 ? 1.0 : 0.0, 0.0);
    return;
  }
  const PassArgs& a = *u->pass;
  if (!pass_active(u->ctl, a, u->gates)) return;
  const uint64_t F = cst(u->ctl)->frame, flags = cst(u->ctl)->flags;
  const uint32_t T = 1u << a.t, nthr = T >> kRegBits;
  uint64_t tb = 0;  // this thread's bits over tile qubits tq[0..t-5]
  for (uint32_t b = 0; b + kRegBits < a.t; ++b) tb |= (uint64_t)((tid >> b) & 1u) << a.tq[b];
  const uint64_t h0 = 1ull << a.tq[a.t - 4], h1 = 1ull << a.tq[a.t - 3], h2 = 1ull << a.tq[a.t - 2],
                 h3 = 1ull << a.tq[a.t - 1];
  const uint64_t free_mask = ~a.tile_mask & ((1ull << a.n) - 1ull);
  const uint64_t base = tile_base((uint64_t)blockIdx.x - u->tile_begin, free_mask), gthr = base | tb;
  if (tid < nthr) {
    double2 r[kR];
    fetch16(r, st, gthr, h0, h1, h2, h3, a.init != 0, F);
    stage16(tile, r, tid, nthr, gthr, h0, h1, h2, h3, 0, 0, 1.0);
  }
  __syncthreads();
  run_phases<true>(tile, T, tid, nthr, flags, u->phases, a.phase_begin, a.phase_count, u->gates, u->mats);
  if (tid < nthr) store_tile16(tile, st, a, base, tid, F);
}

hipError_t launch_pass_units(const PassUnit* units, uint32_t n_units, uint32_t tiles, hipStream_t st) {
  if (!n_units || !tiles) return hipSuccess;
  const size_t lds = sizeof(double2) << kTileMaxBits;
  uint32_t g = 0;  // (for the LDS limit it raises)
  const hipError_t e = resident_grid((const void*)k_pass_units, kTileThreads, lds, lds, &g);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pass_units, dim3(tiles), dim3(kTileThreads), lds, st, units, n_units);
  return hipGetLastError();
}

// The control-only sites of a round, a workgroup of one wave each: bound by one
// site's chain of events, a few microseconds. A launch per request is bound by
// the host instead: 100 requests of 13 qubits with six such sites each 4.38 ms a
// batch, 1.22 ms here (as items of a persistent launch 1.29 ms).
__global__ __launch_bounds__(64) void k_site_units(const SiteUnit* __restrict__ units, uint32_t cw,
                                                   uint32_t max_record) {
  __shared__ int64_t stack[kCStack];
  const QSV_CONST SiteUnit* u = cst(units + blockIdx.x);
  finalize_shot(u->ctl, 0.0, *u->site, u->events, u->preds, u->code, u->creg, cw, u->record, max_record, nullptr, 0u,
                0u, 0u, 0u, 0.0, 0.0, nullptr, stack);
}

hipError_t launch_site_units(const SiteUnit* units, uint32_t n_units, uint32_t cw, uint32_t max_record,
                             hipStream_t st) {
  if (!n_units) return hipSuccess;
  hipLaunchKernelGGL(k_site_units, dim3(n_units), dim3(64), 0, st, units, cw, max_record);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Resident shots: the whole program for one shot of up to 2^12 amplitudes in one
// workgroup, the state in LDS from the first gate to the last measurement.
//
// One launch instead of one per pass and site: a 10-qubit state is 16 KiB, so
// passes and sites as launches spend their time on launch gaps, on operands
// fetched cold by every workgroup and on moving a state that fits its CU. Bound
// by the chain of phases and events of one shot (each phase waits for the one
// before), not by a unit; so descriptors are staged in LDS ahead of the chain,
// the next phase's matrix is under way during the current phase's products, and
// a site's events run on a whole wave. Arithmetic, its order, draws and the
// collapse that is applied when the next pass starts are those of the tile
// passes and of the site kernels, so that the results are the same bit for bit.
// Amplitude i of the frame-free state sits at slot swz(i ^ frame).
//
// Calls, launches per pass and site (with the same read-back before either)
// against this kernel: one shot of 3 qubits 117 and 84 us, 257 of 7 247 and 168
// us, 1000 of 10 (20 layers, 3 sites) 406 and 195 us, 3000 of 11 866 and 590 us,
// 3000 of 12 1.49 and 1.32 ms, 3000 of 12 in complex64 1.19 and 0.99 ms. At 10
// qubits a phase takes 4.6 k cycles of the chain, 2.1 k of them matrix-core
// work. From 13 qubits on a state no longer fits.
// ---------------------------------------------------------------------------
// Programs below kDenseMinTileBits qubits are gate lists throughout. From
// kListMinBits qubits, or up to kListMaxShots shots, a pass then runs as one list
// of phases: long lists are a serial chain, and descriptors taken from the staged
// copy phase by phase made it longer than the tile pass's (one shot of 200 layers
// on 8 qubits 1.35 ms there, 1.42 staged, 1.34 in one run). Many narrow shots
// run faster from the staged copy (4000 of 7 qubits, 60 layers: 1.35 ms, 1.63 in
// one run).
constexpr uint32_t kListMinBits = 8, kListMaxShots = 256;
constexpr uint32_t kResPhases = 64;  // phase descriptors staged at a time (one per thread of the smallest workgroup)
struct ResidentScratch {
  Phase ph[kResPhases];
  uint64_t mat[kResPhases];  // where each dense phase's matrix is
  double red[kSiteBins][kSiteBins];
  int64_t stack[kCStack];
  ShotCtl cs;
  uint32_t pad[2];
};

// The lowest k set bits of m.
__device__ __forceinline__ uint32_t low_bits(uint32_t m, int k) {
  uint32_t r = 0;
  for (int i = 0; i < k && m; ++i) {
    r |= m & (0u - m);
    m &= m - 1u;
  }
  return r;
}

// A site's histogram over a state of up to 2^14 amplitudes in LDS, with the
// sums in the order of site_bins, where thread j of 256 adds the amplitudes of
// unrestricted index j + 256 m (m ascending) and the threads' sums are added
// 16 part + k over k and then over the parts. Pair (part, bin b) here adds the
// amplitudes of its own bin only: the index bits are split over the free
// positions (those the pending collapse leaves) into k, part and m, each less
// the bits that the bin fixes.
template <typename CT>
__device__ __forceinline__ void resident_bins(const CT* __restrict__ tile, uint32_t nq, uint32_t q4, uint32_t T,
                                              uint32_t M, uint32_t Vm, uint32_t F, double s2, uint32_t tid,
                                              uint32_t nth, double (*red)[kSiteBins]) {
  const uint32_t open = (T - 1u) & ~M;
  const uint32_t km = low_bits(open, 4), pm = low_bits(open & ~km, 4), mm = open & ~(km | pm);
  uint32_t qm = 0;
  for (uint32_t k = 0; k < nq; ++k) qm |= 1u << ((q4 >> (8u * k)) & 31u);
  const uint32_t kf = km & ~qm, mf = mm & ~qm;
  for (uint32_t i = tid; i < (16u << nq); i += nth) {
    const uint32_t part = i & 15u, b = i >> 4;
    uint32_t want = 0;  // stored values of the site's qubits in bin b
    for (uint32_t k = 0; k < nq; ++k) want |= ((b >> k) & 1u) << ((q4 >> (8u * k)) & 31u);
    want ^= F & qm;
    const uint32_t pv = pdep32(part, pm);
    double acc = 0.0;
    if (part < (1u << __popc(pm)) && ((want ^ Vm) & M & qm) == 0u && ((want ^ pv) & pm & qm) == 0u) {
      const uint32_t at0 = swz(Vm | pv | want);
      uint32_t kk = 0;
      do {
        double v = 0.0;
        uint32_t m = 0;
#pragma unroll 4
        for (uint32_t c = 1u << __popc(mf); c; --c) {
          v += amp_prob(tile[at0 ^ swz(kk | m)], s2);
          m = ((m | ~mf) + 1u) & mf;
        }
        acc += v;
        kk = ((kk | ~kf) + 1u) & kf;
      } while (kk);
    }
    red[part][b] = acc;
  }
}

// kGates: the program has phases that are not dense (their registers halve the
// waves per SIMD). kWaves: waves per SIMD to leave registers for.
template <bool kGates, int kWaves, typename CT>
__global__ __launch_bounds__(2 * kTileThreads, kWaves) void k_resident(ResidentArgs R) {
  extern __shared__ double2 qsv_lds[];
  CT* const tile = reinterpret_cast<CT*>(qsv_lds);
  const uint32_t tid = threadIdx.x, nth = blockDim.x, n = R.n, T = 1u << n, shot = blockIdx.x;
  ResidentScratch& S = *reinterpret_cast<ResidentScratch*>(tile + (T < 16u ? 16u : T));
  uint64_t* const cr = reinterpret_cast<uint64_t*>(&S + 1);
  uint8_t* const rec = reinterpret_cast<uint8_t*>(cr + R.cw);
  for (uint32_t w = tid; w < R.cw; w += nth) cr[w] = 0;
  for (uint32_t w = tid; w < R.max_record; w += nth) rec[w] = 0;
  if (tid == 0) {
    ShotCtl c;
    c.flags = 0;
    c.pend_mask = 0;
    c.pend_val = 0;
    c.frame = 0;
    c.pend_scale = 1.0;
    c.record_prob = 1.0;
    c.n_events = 0;
    c.n_record = 0;
    c.status = 0;
    c.wg_done = 0;
    S.cs = c;
  }
  __syncthreads();
  Draws dr;  // (wave 0's)
  dr.filled = 0;
  dr.base = 0;
  const double* mb = R.mats + (uint64_t)shot * R.mat_stride;
  auto fill = [&]() {
    for (uint32_t l = tid; l < T; l += nth) tile[swz(l)] = cmake<CT>(l == 0 ? 1.0 : 0.0, 0.0);
    __syncthreads();
  };
  for (uint32_t k = 0; k < R.n_steps; ++k) {
    if (uni32((uint32_t)S.cs.status) != 0) break;
    const uint32_t kind = cst(R.steps + k)->kind, index = cst(R.steps + k)->index;
    const uint64_t F = uni64(S.cs.frame), M = uni64(S.cs.pend_mask), V = uni64(S.cs.pend_val);
    const double sc = S.cs.pend_scale;
    if (kind == 0) {  // |0...0>
      fill();
    } else if (kind == 1) {  // gate pass
      const QSV_CONST PassArgs* a = cst(R.passes + index);
      const uint64_t flags = uni64(S.cs.flags);
      if (!a->init && !a->uncond) {
        bool any = a->guard && guard_ok(flags, a->guard);
        for (uint32_t i = 0; !a->guard && i < a->gate_count && !any; ++i)
          any = guard_ok(flags, cst(R.gates + a->gate_begin + i)->guard);
        if (!any) continue;  // the pending collapse stays owed to a later pass
      }
      const uint32_t pb = a->phase_begin, pc = a->phase_count;
      // a phase in which the shot drew no Pauli takes the matrix of the clean set
      auto stage = [&](uint32_t p) {
        const Phase x = R.phases[p];
        const double* m = mb;
        if (R.dirty && x.dense != kNoDense &&
            !R.dirty[(uint64_t)shot * R.n_dense + (x.dense - R.dense0) / (uint32_t)kDenseSlots])
          m = R.clean;
        S.ph[tid] = x;
        S.mat[tid] = (uint64_t)(uintptr_t)(m + (uint64_t)x.dense * kMatStride);
      };
      if (tid < pc && tid < kResPhases) stage(pb + tid);
      if (a->init) {
        fill();
      } else if (M == 0 && sc == 1.0) {
        __syncthreads();
      } else {
        for (uint32_t l = tid; l < T; l += nth) {
          const uint32_t at = swz(l ^ (uint32_t)F);
          tile[at] = ((l & M) == V) ? cscale(tile[at], sc) : cmake<CT>(0.0, 0.0);
        }
        __syncthreads();  // (every thread has read the control block)
        if (tid == 0) {
          S.cs.pend_mask = 0;
          S.cs.pend_val = 0;
          S.cs.pend_scale = 1.0;
        }
      }
      const uint32_t xs = swz((uint32_t)F);
      const bool lists = kGates && n < kDenseMinTileBits && (n >= kListMinBits || gridDim.x <= kListMaxShots);
      if (kGates && lists)
        run_phases<false>(tile, T, tid, T >> kRegBits, flags, R.phases, pb, pc, R.gates, mb, xs);
      for (uint32_t c0 = 0; !lists && c0 < pc; c0 += kResPhases) {
        const uint32_t ne = pc - c0 < kResPhases ? pc - c0 : kResPhases;
        if (c0) {
          if (tid < ne) stage(pb + c0 + tid);
          __syncthreads();
        }
        auto phase_at = [&](uint32_t p) {
          uint64_t w[2];
          __builtin_memcpy(w, &S.ph[p < ne ? p : ne - 1], 16);
          w[0] = uni64(w[0]);
          w[1] = uni64(w[1]);
          Phase ph;
          __builtin_memcpy(&ph, w, 16);
          return ph;
        };
        auto mat_at = [&](uint32_t p) { return uni64(S.mat[p < ne ? p : ne - 1]); };
        auto request = [&](const Phase& p, uint64_t from, CT (&m)[4]) {
          if (p.dense != kNoDense)
            load_mfrag(m, false, static_cast<const CT*>(nullptr), reinterpret_cast<const double2*>((uintptr_t)from),
                       tid & 63u);
        };
        Phase ph = phase_at(0), nph = phase_at(1);
        uint64_t nmat = mat_at(1);
        CT mf[4];
        request(ph, mat_at(0), mf);
        for (uint32_t p = 0; p < ne; ++p) {
          CT nmf[4];
          request(nph, nmat, nmf);
          const Phase nnph = phase_at(p + 2);
          nmat = mat_at(p + 2);
          // (an all-dense pass runs under its one guard: all phases, or none)
          const uint64_t g = kGates && (!a->all_dense || a->guard) ? cst(R.gates + ph.gate_begin)->guard : 0u;
          if (ph.dense != kNoDense && (sizeof(CT) == sizeof(double2) || g == 0u)) {
            if (guard_ok(flags, g)) {
              dense_phase_mfma<2>(tile, T, tid, ph, mf, xs);
              __syncthreads();
            }
          } else if (kGates) {
            run_phases<false>(tile, T, tid, T >> kRegBits, flags, R.phases, pb + c0 + p, 1u, R.gates, mb,
                              xs);
          }
          ph = nph;
          nph = nnph;
#pragma unroll
          for (int e = 0; e < 4; ++e) mf[e] = nmf[e];
        }
        if (kGates) __syncthreads();  // (a phase without enabled gates has no barrier of its own)
      }
      if (kGates && lists) __syncthreads();  // (as above)
      if (kGates && pc == 0) {
        // fewer than 4 qubits: gate by gate on the frame-free state (slots are
        // unswizzled), one amplitude per thread where the frame is taken off and put
        // back; descriptors by scalar loads, the next gate's while one is applied (one
        // shot of 250 layers on 3 qubits: 365 us as launches, 402 with vector loads in
        // the chain, 338 so)
        auto flip = [&]() {
          const CT v = tid < T ? tile[tid ^ (uint32_t)F] : cmake<CT>(0.0, 0.0);
          __syncthreads();
          if (tid < T) tile[tid] = v;
          __syncthreads();
        };
        __syncthreads();  // (the control block is in place before the next step reads it)
        if (F) flip();
        const uint32_t gb = a->gate_begin, gc = a->gate_count;
        DGate next = load_gate(R.gates + gb);
        for (uint32_t i = 0; i < gc; ++i) {
          const DGate g = next;
          next = load_gate(R.gates + gb + (i + 1 < gc ? i + 1 : i));
          if (!guard_ok(flags, g.guard)) continue;
          tile_apply(tile, n, g, mb + (uint64_t)g.mat * kMatStride);
          __syncthreads();
        }
        if (F) flip();
      }
    } else {  // measurement site
      const QSV_CONST uint32_t* sw = (const QSV_CONST uint32_t*)(R.sites + index);
      static_assert(offsetof(SiteArgs, ev_begin) == 8 && offsetof(SiteArgs, q) == 24, "words of SiteArgs");
      const uint32_t nq = sw[0], ev_begin = sw[2], ev_count = sw[3], q4 = sw[6];
      if (nq) {
        resident_bins(tile, nq, q4, T, (uint32_t)M, (uint32_t)(V ^ (F & M)), (uint32_t)F, sc * sc, tid, nth, S.red);
        __syncthreads();
      }
      if (tid < 64) {
        const uint32_t b = tid & (uint32_t)(kSiteBins - 1);
        double bin = 0.0;
        if (b < (nq ? 1u << nq : 0u)) {
#pragma unroll
          for (uint32_t part = 0; part < 16; ++part) bin += S.red[part][b];
        }
        ShotCtl c = load_ctl(&S.cs);
        if (ev_count)
          site_events(c, dr, bin, q4, R.events + ev_begin, ev_count, R.preds, R.code, cr, rec, R.max_record,
                      R.forced ? R.forced + (uint64_t)shot * R.forced_len : nullptr, R.forced_len,
                      R.key ? cst(R.key)[0] : R.seed, (R.key ? cst(R.key)[1] : R.shot_base) + shot, R.readout_err, R.reset_err, S.stack);
        if (tid == 0) S.cs = c;
      }
      __syncthreads();
    }
  }
  __syncthreads();
  for (uint32_t w = tid; w < R.cw; w += nth) R.creg[(uint64_t)shot * R.cw + w] = cr[w];
  for (uint32_t w = tid; w < R.max_record; w += nth) R.record[(uint64_t)shot * R.max_record + w] = rec[w];
  if (tid == 0) R.ctl[shot] = S.cs;
  if (shot == 0 && R.state_out) {  // as k_materialize
    const uint64_t F = S.cs.frame, M = S.cs.pend_mask, V = S.cs.pend_val;
    const double sc = S.cs.pend_scale;
    for (uint32_t i = tid; i < T; i += nth) {
      double2 v = make_double2(0.0, 0.0);
      if ((i & M) == V) {
        const CT x = tile[swz(i ^ (uint32_t)F)];
        v = cscale(make_double2(x.x, x.y), sc);
      }
      R.state_out[i] = v;
    }
  }
}

// Dense programs in complex128 spill 26 registers at four waves per SIMD and none
// at two, so a call whose shots are all resident at once at two takes that build
// (1000 shots of 10 qubits 173 and 158 us, 64 of 12 188 and 173 us); with more
// shots the waves count for more (3000 of 12 qubits 1.33 and 1.69 ms).
template <bool kGates, int kWaves, typename CT>
static hipError_t resident_t(const ResidentArgs& R, uint32_t shots, hipStream_t st) {
  const uint32_t T = std::max(16u, 1u << R.n), nth = std::max(64u, (1u << R.n) >> 3);
  size_t lds = T * sizeof(CT) + sizeof(ResidentScratch) + R.cw * 8u + R.max_record;
  lds = (lds + 511) & ~(size_t)511;
  uint32_t g = 0;  // (also for the LDS limit it raises)
  const hipError_t e =
      resident_grid((const void*)k_resident<kGates, kWaves, CT>, nth, lds,
                    (sizeof(CT) << kResidentMaxBits) + sizeof(ResidentScratch) + kResidentMaxBytes + 512, &g);
  if (e != hipSuccess) return e;
  if constexpr (!kGates && kWaves == 2) {
    if (shots > g) return resident_t<false, 4, CT>(R, shots, st);
  }
  hipLaunchKernelGGL((k_resident<kGates, kWaves, CT>), dim3(shots), dim3(nth), lds, st, R);
  return hipGetLastError();
}

hipError_t launch_resident(const ResidentArgs& R, uint32_t shots, bool gates, bool c64, hipStream_t st) {
  if (!shots) return hipSuccess;
  if (R.n > (uint32_t)kResidentMaxBits || R.cw * 8u + R.max_record > kResidentMaxBytes) return hipErrorInvalidValue;
  if (c64) return gates ? resident_t<true, 2, float2>(R, shots, st) : resident_t<false, 4, float2>(R, shots, st);
  return gates ? resident_t<true, 2, double2>(R, shots, st) : resident_t<false, 2, double2>(R, shots, st);
}

// ---------------------------------------------------------------------------
// Fixed device scratch of the no-allocation entry point
// ---------------------------------------------------------------------------
// Every device the library runs on holds one copy of this array from the
// moment the code object is loaded there until the process ends. In host code
// the array's name is not a device address: each device's copy is reached only
// through the address hipGetSymbolAddress returns with that device current,
// taken once per device by noalloc_scratch_init (called when a context is
// created) and handed to the kernels as an ordinary buffer argument.
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kNoAllocMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current first
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  g_scratch_ptr[device] = p;
  return hipSuccess;
}

void* noalloc_scratch(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return g_scratch_ptr[device];
}

}  // namespace qsv
