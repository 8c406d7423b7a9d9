// gfx950 kernels of the light tracer and its three reverse modes.
//
// Every pass is a persistent kernel: each wave keeps all 64 lanes busy by
// fetching new path indices (one atomic per wave) as soon as lanes finish
// their path, so paths of uneven length do not idle the SIMD.  All path
// state lives in registers; the BVH traversal stack lives in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include "lt_path.h"

namespace lt {

#ifdef LT_COUNTERS
inline namespace counted {
#endif

// ---------------------------------------------------------------- forward
// Light tracing with a connection + splat at every Lambertian vertex
// (Eq. 1-2, Eq. 20).  RESV: streams valid connections through a capacity-1
// weighted reservoir (Eq. 8) and records/splats the selection (Eq. 9).
// TAPE: writes the per-vertex naive-AD tape.  SPL: writes the buffered
// two-pass splat records (u_i, C_i of every valid connection, a per-path
// header).  GS: writes each path's diffuse-guide training sample (its first
// guided Lambertian scatter: position, arrival-side normal, direction,
// density, S = sum of lum(C_i) over the later connections, component).
// Each loop iteration advances every live lane by one vertex; the splat is
// issued cooperatively by the whole wave after the step.
template <bool TAPE, bool RESV, bool SPL, bool GS, int SC>
__device__ __forceinline__ void trace_run(ArgsPtr P, int* lds) {
  const PassArgs& A = fresh(P);
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  const bool selected = (A.flags & 2u) != 0;
  bool alive = false, exhausted = false;
  uint32_t path = 0, sig = 0;
  int j = 0, nrec = 0;
  Ray r;
  f3 beta = {0.f, 0.f, 0.f};
  float Om = 0.f, omR = 0.f, uxR = 0.f, uyR = 0.f;
  int R = 0;
  f3 CR = {0.f, 0.f, 0.f};
  float fac = 0.f, Sl = 0.f;  // emission factor, path contribution sum_i lum(C_i)
  int klast = 0;              // SPL: last connection depth and validity bits
  uint64_t vmask = 0ull;
  f3 Le = ld3(A.Le);
  D3R iLe = {0.0, 0.0, 0.0};
  int etex = -1;
  float gs[12];  // GS: the sample being built (gs[10] accumulates S)
  bool gs_on = false;
  WorkQ wq = work_begin(A.counter, draws_ahead<SC>(A.n_paths));
  while (true) {
    const PassArgs& A = fresh(P);
    refill(A, wq, alive, exhausted, path, [&](uint32_t p) {
      if (GS)
        for (int q = 0; q < 12; ++q) A.gsamp[(size_t)p * 12 + q] = 0.f;
      if (SPL) { SplatHdr z{}; A.spl_hdr[p] = z; }
      if (TAPE) A.tape_len[p] = 0;
      if (RESV && A.res) { ResRec z{}; A.res[p] = z; }
      if (A.sig) A.sig[p] = 0u;
      if (A.contrib) A.contrib[p] = 0.f;
    });
    if (__ballot(alive) == 0ull) break;
    bool has = false;
    float sux = 0.f, suy = 0.f;
    f3 sC = {0.f, 0.f, 0.f};
    if (alive) {
      if (j == 0) {  // new path: vertex 0 on the emitter
        fac = emit_path(A, path, r);
        path_emitter(A, path, Le, iLe, etex);
        beta = Le * fac;
        j = 1; nrec = 0; sig = 0x811C9DC5u;
        Om = 0.f; omR = 0.f; R = 0; Sl = 0.f;
        klast = 0; vmask = 0ull;
        if (GS) {
          gs_on = false;
#pragma unroll
          for (int q = 0; q < 12; ++q) gs[q] = 0.f;
        }
      }
      Event ev = bounce<SC>(A, path, j, r, 1, stk, ss);
      if (A.sig) sig = sig_event(sig, ev);
      if (ev.kind == 1 && ev.valid) {
        f3 C = mul(beta, ev.rho) * ev.g;
        if (GS && gs_on) gs[10] += luminance(C);
        if (SPL) {
          SplatRec* o = A.spl + (size_t)(j - 1) * (size_t)A.n_paths + path;
          o->ux = ev.ux; o->uy = ev.uy; o->C[0] = C.x; o->C[1] = C.y; o->C[2] = C.z;
          klast = j; vmask |= 1ull << (j - 1);
        }
        if (!selected) { has = true; sux = ev.ux; suy = ev.uy; sC = C; }
        Sl += luminance(C);
        if (RESV) {
          float om = luminance(C);
          if (om > 0.0f) {
            Om += om;
            if (ev.u_res < om / Om) { R = j; omR = om; uxR = ev.ux; uyR = ev.uy; CR = C; }
          }
        }
      }
      if (TAPE && ev.kind != 0) {
        TapeRec t;
        if (ev.kind == 1)
          t.tf = (uint32_t)ev.texel | kTfLambert | (ev.valid ? kTfValid : 0u) | (ev.cont ? kTfScatter : 0u);
        else
          t.tf = kTfDielectric;
        t.g = ev.g; t.ux = ev.ux; t.uy = ev.uy;
        t.b[0] = beta.x; t.b[1] = beta.y; t.b[2] = beta.z; t.pad = fac;
        A.tape[(size_t)(j - 1) * (size_t)A.n_paths + path] = t;
        if (A.tape_gw) A.tape_gw[(size_t)(j - 1) * (size_t)A.n_paths + path] = ev.gw;
        LT_COUNT(8, 1);
        ++nrec;
      }
      if (ev.kind == 1 && ev.cont) beta = mul(beta, ev.rho) * ev.gw;
      if (GS && !gs_on && ev.kind == 1 && ev.cont && ev.gq > 0.f) {
        f3 na = ev.cos_in < 0.0f ? r.offn : r.offn * -1.0f;
        gs[0] = ev.x.x; gs[1] = ev.x.y; gs[2] = ev.x.z;
        gs[3] = na.x; gs[4] = na.y; gs[5] = na.z;
        gs[6] = r.w.x; gs[7] = r.w.y; gs[8] = r.w.z;
        gs[9] = ev.gq; gs[11] = (float)ev.gcomp;
        gs_on = true;
      }
      if (ev.cont) {
        ++j;
      } else {  // path finished
        if (GS)
          for (int q = 0; q < 12; ++q) A.gsamp[(size_t)path * 12 + q] = gs[q];
        float W = R > 0 ? Om / omR : 0.f;
        if (RESV && selected && R > 0) { has = true; sux = uxR; suy = uyR; sC = CR * W; }
        if (RESV && A.res) {
          ResRec rr;
          rr.R = R; rr.W = W; rr.ux = uxR; rr.uy = uyR;
          rr.S[0] = CR.x * W; rr.S[1] = CR.y * W; rr.S[2] = CR.z * W; rr.pad = 0.f;
          A.res[path] = rr;
        }
        if (TAPE) A.tape_len[path] = nrec;
        if (SPL) {
          SplatHdr hd;
          hd.klast = klast; hd.pad = 0; hd.vmask = vmask;
          A.spl_hdr[path] = hd;
        }
        if (A.sig) A.sig[path] = fnv1a(sig, (uint32_t)R);
        if (A.contrib) A.contrib[path] = Sl;
        alive = false; j = 0;
      }
    }
    if (!GS) {  // the sample pass writes no image
      keep_finite(A, has, sC);
      splat_wave(A.sc, A.image, A.cells, has, sux, suy, sC);
    }
  }
}

// At most 96 VGPRs (five waves per SIMD, with the default 10 x 128-thread
// workgroups per CU), where a few registers spill: the box forward runs 3.6%
// faster than at four waves.  The plain forward with the heightfield's grid
// walk holds four (128 VGPRs, few spills): the 128x128 caustic's runs 6.7%
// faster there (5.08 -> 4.74 ms).
template <bool TAPE, bool RESV, bool SPL, bool GS, int SC>
__global__ void __launch_bounds__(1024, ((SC & kScHf) && !TAPE && !RESV && !SPL && !GS) ? 4 : 5) k_trace(PassArgs) {
  extern __shared__ int lds[];
  trace_run<TAPE, RESV, SPL, GS, SC>(kernel_args(), lds);
}

// ---------------------------------------------------------------- naive AD
// Reverse sweep over the tape, exact chain rule (no inverses, no division):
//   C_j = beta_j rho_j g_j,  beta_{j+1} = beta_j rho_j s_j (Lambertian scatter,
//   s_j = 1, or cos / (pi q) from the tape's weight array when guided),
//   beta_1 = L_e * f, with the path's emission factor f taped in every record.
// Lanes of a wave walk their tapes in lock step, all at the same depth.
__global__ void __launch_bounds__(1024) k_naive_bwd(PassArgs) {
  const ArgsPtr P = kernel_args();
  const PassArgs& A = fresh(P);
  extern __shared__ int lds[];
  AGrad ga = agrad_begin(A, lds);
  float* le = legrad_begin(A, past_agrad(A, lds, 0));
  const size_t N = (size_t)A.n_paths;
  double gl0 = 0.0, gl1 = 0.0, gl2 = 0.0;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t rounds = (N + stride - 1) / stride;
  for (size_t rd = 0; rd < rounds; ++rd) {
    size_t path = first + rd * stride;
    bool live = path < N && !(A.mask && A.mask[path] == 0);
    int k = live ? min(max(A.tape_len_in[path], 0), A.D) : 0;
    int kmax = k;
    for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o));
    f3 bb = {0.f, 0.f, 0.f};  // adjoint of beta_{j+1}
    float fac = 0.f;
    // every lane at the same depth, so that a row of the tape is read in one
    // piece, and the next row's record on its way while this one is used
    TapeRec next;
    if (kmax >= 1 && kmax <= k) next = A.tape_in[(size_t)(kmax - 1) * N + path];
    for (int j = kmax; j >= 1; --j) {
      const PassArgs& A = fresh(P);
      bool has = false;
      int texel = 0;
      f3 gr = {0.f, 0.f, 0.f};
      const TapeRec t = next;
      if (j >= 2 && j - 1 <= k) next = A.tape_in[(size_t)(j - 2) * N + path];
      if (j <= k) {
        LT_COUNT(9, 1);
        fac = t.pad;
        if (t.tf & kTfLambert) {  // dielectric: weight 1, adjoint passes through
          texel = min((int)(t.tf & kTexMask), A.n_texels - 1);
          f3 rho = ld3(A.albedo + (size_t)texel * 3);
          f3 b = {t.b[0], t.b[1], t.b[2]};
          f3 bj = {0.f, 0.f, 0.f};
          if (t.tf & kTfValid) {
            f3 Lb = gather(A.sc, A.dI, t.ux, t.uy);
            gr = mul(Lb, b) * t.g;
            bj = mul(Lb, rho) * t.g;
          }
          if (t.tf & kTfScatter) {
            const float sw = A.tape_gw_in ? A.tape_gw_in[(size_t)(j - 1) * N + path] : 1.0f;
            gr = gr + mul(bb, b) * sw;
            bj = bj + mul(bb, rho) * sw;
          }
          bb = bj;
          has = true;
        }
      }
      keep_finite(A, has, gr);
      scatter_albedo(A, ga, has, texel, gr);
    }
    f3 Lp = ld3(A.Le);
    if (live) {
      D3R iLp = {0.0, 0.0, 0.0};
      int etex = -1;
      path_emitter(A, (uint32_t)path, Lp, iLp, etex);
      add_le(A, gl0, gl1, gl2, (double)bb.x * fac, (double)bb.y * fac, (double)bb.z * fac, etex, le);
    }
    // the path's adjoint-weighted contribution |delta_total| = sum_c |L_e,c f bb_c|
    if (A.contrib && path < N)
      A.contrib[path] = live ? fabsf(Lp.x * fac * bb.x) + fabsf(Lp.y * fac * bb.y) + fabsf(Lp.z * fac * bb.z) : 0.f;
  }
  flush_sums(A, gl0, gl1, gl2);
  agrad_end(A, ga);
  legrad_end(A, le);
}

// ---------------------------------------------------------------- ResLRB
// Replay each path up to its selected depth R and apply the log-derivative
// identity with weight w = dI(u_R) * S_hat (Eq. 11): the emitter factor
// gets w / L_e, every Lambertian factor rho_j (j < R scatter, j = R
// connection) gets w / rho_j.  No connection is re-evaluated.
template <int SC>
__global__ void __launch_bounds__(1024) k_reslrb_bwd(PassArgs) {
  const ArgsPtr P = kernel_args();
  const PassArgs& A = fresh(P);
  extern __shared__ int lds[];
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  AGrad ga = agrad_begin(A, lds + A.sc.stack_n * blockDim.x);
  float* le = legrad_begin(A, past_agrad(A, lds, A.sc.stack_n));
  bool alive = false, exhausted = false;
  uint32_t path = 0;
  int j = 0, R = 0;
  Ray r;
  f3 w = {0.f, 0.f, 0.f};
  f3 Le = ld3(A.Le);
  D3R iLe = recip_le(Le);
  int etex = -1;
  double gl0 = 0.0, gl1 = 0.0, gl2 = 0.0;
  WorkQ wq = work_begin(A.counter, draws_ahead<SC>(A.n_paths));
  while (true) {
    const PassArgs& A = fresh(P);
    refill(A, wq, alive, exhausted, path, [&](uint32_t) {});
    if (__ballot(alive) == 0ull) break;
    bool has = false;
    int texel = 0;
    f3 gv = {0.f, 0.f, 0.f};
    if (alive && j == 0) {
      ResRec rec = A.res_in[path];
      if (rec.R <= 0) {
        alive = false;
      } else {
        R = min(rec.R, A.D);
        f3 Lb = gather(A.sc, A.dI, rec.ux, rec.uy);
        w = mul(Lb, mk(rec.S[0], rec.S[1], rec.S[2]));
        path_emitter(A, path, Le, iLe, etex);
        add_le(A, gl0, gl1, gl2, (double)w.x * iLe.x, (double)w.y * iLe.y, (double)w.z * iLe.z, etex, le);
        emit_path(A, path, r);
        j = 1;
      }
    }
    if (alive) {
      Event ev = bounce<SC>(A, path, j, r, 0, stk, ss);
      if (ev.kind == 1) {
        texel = ev.texel;
        gv = {ev.rho.x > 0.f ? w.x / ev.rho.x : 0.f, ev.rho.y > 0.f ? w.y / ev.rho.y : 0.f,
              ev.rho.z > 0.f ? w.z / ev.rho.z : 0.f};
        has = true;
      }
      if (ev.cont && j < R) ++j;
      else { alive = false; j = 0; }
    }
    keep_finite(A, has, gv);
    scatter_albedo(A, ga, has, texel, gv);
  }
  flush_sums(A, gl0, gl1, gl2);
  agrad_end(A, ga);
  legrad_end(A, le);
}

// ---------------------------------------------------------------- LRB-3
// Pass 2 and Pass 3 fused per path (dI is read-only between them):
// phase 2 replays and accumulates delta_total = sum_i dI(u_i) * C_i
// (Eq. 14, FP64); phase 3 replays again: the splat term dI(u_i) * C_i / rho_i
// (Eq. 15), the subtraction delta_rem -= dI(u_i) * C_i (Eq. 16) and the
// log-derivative delta_rem / rho_i of the scatter factor (Eq. 17); the
// emitter gets delta_total / L_e.
// Phase 2 also keeps one bit per vertex (valid connection) and the depth of
// the last valid connection: phase 3 then re-evaluates only the connection
// geometry where the bit is set (no shadow rays) and stops at that depth,
// where delta_rem is exactly zero and nothing further contributes.
template <int SC>
__device__ __forceinline__ void lrb3_run(ArgsPtr P, int* lds) {
  const PassArgs& A = fresh(P);
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  AGrad ga = agrad_begin(A, lds + A.sc.stack_n * blockDim.x);
  float* le = legrad_begin(A, past_agrad(A, lds, A.sc.stack_n));
  bool alive = false, exhausted = false;
  uint32_t path = 0;
  int j = 0, phase = 2, klast = 0;
  uint64_t vmask = 0ull;
  Ray r;
  f3 beta = {0.f, 0.f, 0.f};
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;  // delta_total, then delta_rem
  f3 Le = ld3(A.Le);
  D3R iLe = recip_le(Le);
  int etex = -1;
  double gl0 = 0.0, gl1 = 0.0, gl2 = 0.0;
  WorkQ wq = work_begin(A.counter, draws_ahead<SC>(A.n_paths));
  while (true) {
    const PassArgs& A = fresh(P);
    refill(A, wq, alive, exhausted, path, [&](uint32_t p) { if (A.contrib) A.contrib[p] = 0.f; });
    if (__ballot(alive) == 0ull) break;
    bool has = false;
    int texel = 0;
    f3 gv = {0.f, 0.f, 0.f};
    if (alive) {
      if (j == 0) {
        float f = emit_path(A, path, r);
        path_emitter(A, path, Le, iLe, etex);
        beta = Le * f;
        j = 1;
        if (phase == 2) { d0 = d1 = d2 = 0.0; vmask = 0ull; klast = 0; }
      }
      const int cmode = phase == 2 ? 1 : (((vmask >> (j - 1)) & 1ull) ? 2 : 0);
      Event ev = bounce<SC>(A, path, j, r, cmode, stk, ss);
      if (phase == 3 && j >= klast) ev.cont = false;  // nothing after the last connection
      if (ev.kind == 1) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        if (ev.valid) {
          f3 C = mul(beta, ev.rho) * ev.g;
          f3 Lb = gather(A.sc, A.dI, ev.ux, ev.uy);
          a0 = (double)Lb.x * C.x; a1 = (double)Lb.y * C.y; a2 = (double)Lb.z * C.z;
          if (phase == 2) { vmask |= 1ull << (j - 1); klast = j; }
        }
        if (phase == 2) {
          d0 += a0; d1 += a1; d2 += a2;
        } else {
          d0 -= a0; d1 -= a1; d2 -= a2;
          if (j >= klast) { d0 = d1 = d2 = 0.0; }
          double g0 = a0, g1 = a1, g2 = a2;
          if (ev.cont) { g0 += d0; g1 += d1; g2 += d2; }
          texel = ev.texel;
          gv = {ev.rho.x > 0.f ? (float)g0 / ev.rho.x : 0.f, ev.rho.y > 0.f ? (float)g1 / ev.rho.y : 0.f,
                ev.rho.z > 0.f ? (float)g2 / ev.rho.z : 0.f};
          has = true;
        }
        if (ev.cont) beta = mul(beta, ev.rho) * ev.gw;
      }
      if (ev.cont) {
        ++j;
      } else if (phase == 2 && klast > 0 && (d0 != 0.0 || d1 != 0.0 || d2 != 0.0)) {  // consuming replay
        add_le(A, gl0, gl1, gl2, d0 * iLe.x, d1 * iLe.y, d2 * iLe.z, etex, le);
        // the path's adjoint-weighted contribution |delta_total|
        if (A.contrib) A.contrib[path] = (float)(fabs(d0) + fabs(d1) + fabs(d2));
        phase = 3; j = 0;
      } else {
        if (A.contrib && phase == 2) A.contrib[path] = 0.f;
        phase = 2; j = 0; alive = false;
      }
    }
    keep_finite(A, has, gv);
    scatter_albedo(A, ga, has, texel, gv);
  }
  flush_sums(A, gl0, gl1, gl2);
  agrad_end(A, ga);
  legrad_end(A, le);
  lds_grads_done(A);
}

template <int SC>
__global__ void __launch_bounds__(1024) k_lrb3_bwd(PassArgs) {
  extern __shared__ int lds[];
  lrb3_run<SC>(kernel_args(), lds);
}

// ---------------------------------------------------------------- buffered two-pass
// The buffered two-pass variant (lrb_2pass, Sec. 4.1 and Sec. 6): the forward
// stored every connection's film position and contribution in a buffer
// preallocated to the maximum depth, so delta_total = sum_i dI(u_i) C_i
// (Eq. 14) is read back without a traversal, and one replay (no shadow rays,
// no connection geometry: u_i and C_i come from the buffer) consumes it as
// LRB-3's pass 3 does (Eq. 15-17).  Memory is linear in depth, traversals
// two (forward and replay), the gradient naive AD's.
template <int SC>
__device__ __forceinline__ void lrb2_run(ArgsPtr P, int* lds) {
  const PassArgs& A = fresh(P);
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  AGrad ga = agrad_begin(A, lds + A.sc.stack_n * blockDim.x);
  float* le = legrad_begin(A, past_agrad(A, lds, A.sc.stack_n));
  const size_t N = (size_t)A.n_paths;
  bool alive = false, exhausted = false;
  uint32_t path = 0;
  int j = 0, klast = 0;
  uint64_t vmask = 0ull;
  Ray r;
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;
  f3 Le = ld3(A.Le);
  D3R iLe = recip_le(Le);
  int etex = -1;
  double gl0 = 0.0, gl1 = 0.0, gl2 = 0.0;
  WorkQ wq = work_begin(A.counter, draws_ahead<SC>(A.n_paths));
  while (true) {
    const PassArgs& A = fresh(P);
    refill(A, wq, alive, exhausted, path, [&](uint32_t p) { if (A.contrib) A.contrib[p] = 0.f; });
    if (__ballot(alive) == 0ull) break;
    bool has = false;
    int texel = 0;
    f3 gv = {0.f, 0.f, 0.f};
    if (alive && j == 0) {
      const SplatHdr hd = A.spl_hdr_in[path];
      klast = min(hd.klast, A.D);
      vmask = hd.vmask;
      d0 = d1 = d2 = 0.0;
      for (uint64_t m = vmask; m; m &= m - 1ull) {
        const int i = __ffsll((unsigned long long)m);  // 1-based vertex
        if (i > klast) break;
        const SplatRec rec = A.spl_in[(size_t)(i - 1) * N + path];
        LT_COUNT(9, 1);
        f3 Lb = gather(A.sc, A.dI, rec.ux, rec.uy);
        d0 += (double)Lb.x * rec.C[0]; d1 += (double)Lb.y * rec.C[1]; d2 += (double)Lb.z * rec.C[2];
      }
      if (klast > 0 && (d0 != 0.0 || d1 != 0.0 || d2 != 0.0)) {
        path_emitter(A, path, Le, iLe, etex);
        add_le(A, gl0, gl1, gl2, d0 * iLe.x, d1 * iLe.y, d2 * iLe.z, etex, le);
        if (A.contrib) A.contrib[path] = (float)(fabs(d0) + fabs(d1) + fabs(d2));
        emit_path(A, path, r);
        j = 1;
      } else {
        if (A.contrib) A.contrib[path] = 0.f;
        alive = false;
      }
    }
    if (alive) {
      Event ev = bounce<SC>(A, path, j, r, 0, stk, ss);
      const bool last = j >= klast;
      if (ev.kind == 1) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        if ((vmask >> (j - 1)) & 1ull) {
          const SplatRec rec = A.spl_in[(size_t)(j - 1) * N + path];
          LT_COUNT(9, 1);
          f3 Lb = gather(A.sc, A.dI, rec.ux, rec.uy);
          a0 = (double)Lb.x * rec.C[0]; a1 = (double)Lb.y * rec.C[1]; a2 = (double)Lb.z * rec.C[2];
        }
        d0 -= a0; d1 -= a1; d2 -= a2;
        if (last) { d0 = d1 = d2 = 0.0; }
        double g0 = a0, g1 = a1, g2 = a2;
        if (!last) { g0 += d0; g1 += d1; g2 += d2; }
        texel = ev.texel;
        gv = {ev.rho.x > 0.f ? (float)g0 / ev.rho.x : 0.f, ev.rho.y > 0.f ? (float)g1 / ev.rho.y : 0.f,
              ev.rho.z > 0.f ? (float)g2 / ev.rho.z : 0.f};
        has = true;
      }
      if (ev.cont && !last) ++j;
      else { alive = false; j = 0; }
    }
    keep_finite(A, has, gv);
    scatter_albedo(A, ga, has, texel, gv);
  }
  flush_sums(A, gl0, gl1, gl2);
  agrad_end(A, ga);
  legrad_end(A, le);
}

template <int SC>
__global__ void __launch_bounds__(1024) k_lrb2_bwd(PassArgs) {
  extern __shared__ int lds[];
  lrb2_run<SC>(kernel_args(), lds);
}

// ---------------------------------------------------------------- LRB-3, two kernels
// The same two replays as k_lrb3_bwd, each a kernel of its own with the
// method's per-path state handed over in memory (Lrb3Hand, 40 bytes per
// connected path, appended per class of the path index, flat in depth).
// Every wave then runs one phase: pass 2's shadow rays and pass 3's gradient
// scatters never share a wave, and pass 3 visits only the paths with a
// sensor connection, compacted by the append.

// Pass 2 (Eq. 14): replay with the sensor connections (shadow rays
// included), delta_total = sum_i dI(u_i) C_i in FP64, one bit per vertex for
// a valid connection, the depth of the last one.  A path whose delta_total is
// nonzero gets its emitter gradient delta_total / L_e here and a hand-off
// entry (appended to its class's region).
template <int SC>
__device__ __forceinline__ void lrb3_p2_run(ArgsPtr P, int* lds) {
  const PassArgs& A = fresh(P);
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  float* le = legrad_begin(A, past_agrad(A, lds, A.sc.stack_n));
  bool alive = false, exhausted = false;
  uint32_t path = 0;
  int j = 0, klast = 0;
  uint64_t vmask = 0ull;
  Ray r;
  f3 beta = {0.f, 0.f, 0.f};
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;
  f3 Le = ld3(A.Le);
  D3R iLe = recip_le(Le);
  int etex = -1;
  double gl0 = 0.0, gl1 = 0.0, gl2 = 0.0;
  WorkQ wq = work_begin(A.counter, draws_ahead<SC>(A.n_paths));
  while (true) {
    const PassArgs& A = fresh(P);
    refill(A, wq, alive, exhausted, path, [&](uint32_t p) { if (A.contrib) A.contrib[p] = 0.f; });
    if (__ballot(alive) == 0ull) break;
    bool put = false;
    if (alive) {
      if (j == 0) {
        const float f = emit_path(A, path, r);
        path_emitter(A, path, Le, iLe, etex);
        beta = Le * f;
        j = 1;
        d0 = d1 = d2 = 0.0; vmask = 0ull; klast = 0;
      }
      Event ev = bounce<SC>(A, path, j, r, 1, stk, ss);
      if (ev.kind == 1) {
        if (ev.valid) {
          f3 C = mul(beta, ev.rho) * ev.g;
          f3 Lb = gather(A.sc, A.dI, ev.ux, ev.uy);
          d0 += (double)Lb.x * C.x; d1 += (double)Lb.y * C.y; d2 += (double)Lb.z * C.z;
          vmask |= 1ull << (j - 1); klast = j;
        }
        if (ev.cont) beta = mul(beta, ev.rho) * ev.gw;
      }
      if (ev.cont) {
        ++j;
      } else {
        put = klast > 0 && (d0 != 0.0 || d1 != 0.0 || d2 != 0.0);
        if (put) add_le(A, gl0, gl1, gl2, d0 * iLe.x, d1 * iLe.y, d2 * iLe.z, etex, le);
        // the path's adjoint-weighted contribution |delta_total|
        if (A.contrib) A.contrib[path] = put ? (float)(fabs(d0) + fabs(d1) + fabs(d2)) : 0.f;
        alive = false; j = 0;
      }
    }
    const uint32_t slot = hand_append(A, put, path);
    if (put) {
      Lrb3Hand h;
      h.path = path; h.klast = klast; h.vmask = vmask; h.d[0] = d0; h.d[1] = d1; h.d[2] = d2;
      A.hand[slot] = h;
    }
  }
  flush_sums(A, gl0, gl1, gl2);
  legrad_end(A, le);
}

// Pass 3 (Eq. 15-17) over the handed-over paths: replay to the last
// connection re-evaluating only the connection geometry where the bit is
// set (no shadow rays), the splat term dI(u_i) C_i / rho_i, the subtraction
// from delta_rem and the scatter term delta_rem / rho_i.
template <int SC>
__device__ __forceinline__ void lrb3_p3_run(ArgsPtr P, int* lds) {
  const PassArgs& A = fresh(P);
  int* stk = lds + threadIdx.x;
  const int ss = blockDim.x;
  AGrad ga = agrad_begin(A, lds + A.sc.stack_n * blockDim.x);
  bool alive = false, exhausted = false;
  uint32_t item = 0, path = 0;
  int j = 0, klast = 0;
  uint64_t vmask = 0ull;
  Ray r;
  f3 beta = {0.f, 0.f, 0.f};
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;
  f3 Le = ld3(A.Le);
  D3R iLe = {0.0, 0.0, 0.0};
  int etex = -1;
  WorkQ wq = work_begin(A.counter3, draws_ahead<SC>(A.n_paths / 2));
  while (true) {
    const PassArgs& A = fresh(P);
    refill_hand(A, wq, alive, exhausted, item);
    if (__ballot(alive) == 0ull) break;
    bool has = false;
    int texel = 0;
    f3 gv = {0.f, 0.f, 0.f};
    if (alive) {
      if (j == 0) {
        const Lrb3Hand h = A.hand[item];
        path = h.path; klast = h.klast; vmask = h.vmask; d0 = h.d[0]; d1 = h.d[1]; d2 = h.d[2];
        const float f = emit_path(A, path, r);
        path_emitter(A, path, Le, iLe, etex);
        beta = Le * f;
        j = 1;
      }
      Event ev = bounce<SC>(A, path, j, r, ((vmask >> (j - 1)) & 1ull) ? 2 : 0, stk, ss);
      if (j >= klast) ev.cont = false;  // nothing after the last connection
      if (ev.kind == 1) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        if (ev.valid) {
          f3 C = mul(beta, ev.rho) * ev.g;
          f3 Lb = gather(A.sc, A.dI, ev.ux, ev.uy);
          a0 = (double)Lb.x * C.x; a1 = (double)Lb.y * C.y; a2 = (double)Lb.z * C.z;
        }
        d0 -= a0; d1 -= a1; d2 -= a2;
        if (j >= klast) { d0 = d1 = d2 = 0.0; }
        double g0 = a0, g1 = a1, g2 = a2;
        if (ev.cont) { g0 += d0; g1 += d1; g2 += d2; }
        texel = ev.texel;
        gv = {ev.rho.x > 0.f ? (float)g0 / ev.rho.x : 0.f, ev.rho.y > 0.f ? (float)g1 / ev.rho.y : 0.f,
              ev.rho.z > 0.f ? (float)g2 / ev.rho.z : 0.f};
        has = true;
        if (ev.cont) beta = mul(beta, ev.rho) * ev.gw;
      }
      if (ev.cont) ++j;
      else { alive = false; j = 0; }
    }
    keep_finite(A, has, gv);
    scatter_albedo(A, ga, has, texel, gv);
  }
  agrad_end(A, ga);
}

template <int SC>
__global__ void __launch_bounds__(1024) k_lrb3_p2(PassArgs) {
  extern __shared__ int lds[];
  lrb3_p2_run<SC>(kernel_args(), lds);
}
template <int SC>
__global__ void __launch_bounds__(1024) k_lrb3_p3(PassArgs) {
  extern __shared__ int lds[];
  lrb3_p3_run<SC>(kernel_args(), lds);
}

// ---------------------------------------------------------------- small kernels
// Pixel channel i of the film (row-major, 3 per pixel) summed over the four
// cells around it (see splat_wave).
__device__ __forceinline__ float film_pixel(const float* cells, int W, int i) {
  const int y = i / (3 * W), q = i - y * 3 * W, x = q / 3, ch = q - 3 * x;
  const float* c = cells + ((size_t)(y + 1) * (W + 1) + x + 1) * kCellFloats + ch;  // the cell whose tap (0, 0) it is
  const float* up = c - (size_t)(W + 1) * kCellFloats;
  return (c[0] + c[3 - kCellFloats]) + (up[6] + up[9 - kCellFloats]);
}
__global__ void __launch_bounds__(256) k_film_resolve(PassArgs A) {
  const int n = 3 * A.sc.W * A.sc.H;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    A.image[i] = film_pixel(A.cells, A.sc.W, i);
}

// Heightfield triangle q from the current heights, written at its slot.
// The edges are built from height differences and whole grid steps, not by
// subtracting rounded corner positions: base + h rounds to about 6e-8 at
// base 0.6, which on a 1/127 grid spacing would put ~1e-5 of error on every
// facet slope, whereas h_k - h_0 and (i_k - i_0) dx are exact or nearly so.
__device__ __forceinline__ void write_hf_tri(const DevScene& sc, const float* h, int q) {
  int gi[3], gj[3];
  float hv[3];
  for (int k = 0; k < 3; ++k) {
    hf_corner(sc.hf_G, sc.hf_rcells, q, k, gi[k], gj[k]);
    hv[k] = hget(h, sc.hf_G, gi[k], gj[k]);
  }
  Tri t;
  t.p0[0] = sc.hf_x0 + gi[0] * sc.hf_dx;
  t.p0[1] = sc.hf_base + hv[0];
  t.p0[2] = sc.hf_z0 + gj[0] * sc.hf_dx;
  t.prim = sc.n_static + q;
  t.e1[0] = (float)(gi[1] - gi[0]) * sc.hf_dx; t.e1[1] = hv[1] - hv[0]; t.e1[2] = (float)(gj[1] - gj[0]) * sc.hf_dx;
  t.e2[0] = (float)(gi[2] - gi[0]) * sc.hf_dx; t.e2[1] = hv[2] - hv[0]; t.e2[2] = (float)(gj[2] - gj[0]) * sc.hf_dx;
  t.mat = sc.hf_mat; t.par = sc.hf_par;
  const_cast<Tri*>(sc.tris)[sc.n_static + q] = t;  // the heightfield's slots follow the static triangles
}
// Least and greatest of the heights, into hb (see kHfRange).  Up to kHfOne
// heights workgroup 0 of the pass start forms them by itself; of more, kHfParts
// workgroups form a part each and a launch of one wave the whole.  Nothing is
// counted between workgroups, so nothing that a launch leaves behind can make
// a later one finish early; and a count's chain of three dependent atomics and
// 32 atomic reads is no shorter (with a count -> without, us a step: 33x33
// heights with taped AD, 100k paths, 149 -> 141; 64x64 bidirectional 896 -> 887;
// 128x128, 16M paths, 11.87 -> 11.86 ms).
__device__ __forceinline__ void hf_range(const float* h, int n, float* hb, int part) {
  __shared__ float lo[256], hi[256];
  const int parts = n <= kHfOne ? 1 : kHfParts;
  if (part >= parts) return;
  float a = 3.0e38f, b = -3.0e38f;
  for (int i = part * 256 + threadIdx.x; i < n; i += parts * 256) { a = fminf(a, h[i]); b = fmaxf(b, h[i]); }
  lo[threadIdx.x] = a; hi[threadIdx.x] = b;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      lo[threadIdx.x] = fminf(lo[threadIdx.x], lo[threadIdx.x + w]);
      hi[threadIdx.x] = fmaxf(hi[threadIdx.x], hi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  float* out = hb + (parts == 1 ? 0 : 2 + 2 * part);
  out[0] = lo[0]; out[1] = hi[0];
}
// the whole range from the parts: one wave
__device__ __forceinline__ void hf_whole(float* hb) {
  const int k = 2 + 2 * (threadIdx.x & (kHfParts - 1));
  float a = hb[k], b = hb[k + 1];
#pragma unroll
  for (int o = kHfParts / 2; o > 0; o >>= 1) { a = fminf(a, __shfl_xor(a, o)); b = fmaxf(b, __shfl_xor(b, o)); }
  if (threadIdx.x == 0) { hb[0] = a; hb[1] = b; }
}
__global__ void __launch_bounds__(64) k_hf_whole(float* hb) { hf_whole(hb); }
__global__ void __launch_bounds__(64) k_hf_whole_batch(const PassArgs* __restrict__ T) {
  const PassArgs& A = fresh(table_ptr(T, blockIdx.x));
  if (A.begin_hf && A.sc.hf_G * A.sc.hf_G > kHfOne) hf_whole(const_cast<float*>(A.sc.hf_hb));
}
// Start of a pass, one launch for everything it needs cleared or derived (it
// took five): the film, the heightfield's triangles, slopes and height range
// (a large heightfield's range takes one more).
__device__ __forceinline__ void begin_run(const PassArgs& A, int block, int blocks) {
  const size_t first = (size_t)block * blockDim.x + threadIdx.x, stride = (size_t)blocks * blockDim.x;
  if (A.cells) {
    const size_t n = (size_t)(A.sc.W + 1) * (A.sc.H + 1) * (kCellFloats / 4);
    for (size_t i = first; i < n; i += stride) reinterpret_cast<float4*>(A.cells)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  } else if (A.image) {
    const size_t n = (size_t)A.sc.W * A.sc.H * 3;
    for (size_t i = first; i < n; i += stride) A.image[i] = 0.f;
  }
  if (A.begin_hf) {
    const int n = 2 * (A.sc.hf_G - 1) * (A.sc.hf_G - 1);
    for (size_t q = first; q < (size_t)n; q += stride) write_hf_tri(A.sc, A.heights, (int)q);
    if (!A.nmap) {
      // central differences, once a pass: a shading normal took twelve heights
      // and six quotients (128x128 caustic, 16M paths, step 12.7 -> 11.9 ms)
      const int G = A.sc.hf_G;
      for (size_t v = first; v < (size_t)G * G; v += stride) {
        const int j = (int)(v / (size_t)G), i = (int)(v - (size_t)j * G);
        float2 s;
        hf_slope(A.heights, G, A.sc.hf_dx, A.sc.hf_idx, i, j, s.x, s.y);
        reinterpret_cast<float2*>(A.sc.slopes)[v] = s;
      }
    }
    hf_range(A.heights, A.sc.hf_G * A.sc.hf_G, const_cast<float*>(A.sc.hf_hb), block);
  }
}
__global__ void __launch_bounds__(256) k_begin(PassArgs A, unsigned int* counters, size_t n_counters) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_counters; i += (size_t)gridDim.x * blockDim.x)
    counters[i] = 0u;
  begin_run(A, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) k_begin_batch(const PassArgs* __restrict__ T, unsigned int* counters,
                                                     size_t n_counters) {
  const size_t block = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
  for (size_t i = block * blockDim.x + threadIdx.x; i < n_counters; i += (size_t)gridDim.x * gridDim.y * blockDim.x)
    counters[i] = 0u;
  begin_run(fresh(table_ptr(T, blockIdx.y)), blockIdx.x, gridDim.x);
}

// Mean squared error over n values and its adjoint.  The workgroups' FP64 sums
// go to kAccSlots slots, a line each (one address took 12 ns a workgroup);
// the last workgroup to finish writes the loss.  Slots and ticket are zero at
// launch.  cells: the image is first summed up from the film cells and stored.
__device__ __forceinline__ void loss_run(const float* I, float* image, const float* cells, int W, const float* T, size_t n,
                                         float* dI, double* acc, float* loss, int block, int blocks) {
  __shared__ double part[4];
  double s = 0.0;
  const double inv = 1.0 / (double)n;
  for (size_t i = (size_t)block * blockDim.x + threadIdx.x; i < n; i += (size_t)blocks * blockDim.x) {
    float v;
    if (cells) { v = film_pixel(cells, W, (int)i); image[i] = v; }
    else v = I[i];
    double d = (double)v - (double)T[i];
    s += d * d;
    dI[i] = (float)(2.0 * d * inv);
  }
  s = wave_sum(s);
  if (__lane_id() == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  unsigned int done = 0;
  if (threadIdx.x == 0) {
    unsigned int* ticket = reinterpret_cast<unsigned int*>(acc + 1);
    done_atomic(atomicAdd(acc + (block & (kAccSlots - 1)) * kAccStride, (part[0] + part[1]) + (part[2] + part[3])));
    done = atomicAdd(ticket, 1u);
  }
  done = (unsigned int)__builtin_amdgcn_readfirstlane((int)done);
  if (done != (unsigned int)blocks - 1u) return;
  // the slots, a lane each, read where the atomics execute
  double t = 0.0;
  if (threadIdx.x < kAccSlots)
    t = __longlong_as_double((long long)atomicAdd(reinterpret_cast<unsigned long long*>(acc + threadIdx.x * kAccStride), 0ull));
  t = wave_sum(t);
  if (threadIdx.x == 0) loss[0] = (float)(t / (double)n);
}
__global__ void __launch_bounds__(256) k_loss(const float* I, const float* T, size_t n, float* dI, double* acc,
                                              float* loss) {
  loss_run(I, nullptr, nullptr, 0, T, n, dI, acc, loss, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) k_loss_batch(const PassArgs* __restrict__ T) {
  const PassArgs& A = fresh(table_ptr(T, blockIdx.y));
  loss_run(A.image, A.image, A.cells, A.sc.W, A.target, (size_t)A.sc.W * A.sc.H * 3, A.d_image, A.loss_acc, A.loss,
           blockIdx.x, gridDim.x);
}

#include "lt_camera.inc"

// ---------------------------------------------------------------- batches
// One persistent launch over a table of instances (scenes, films, path
// counts and depths of their own).  Every wave walks the table in order and
// takes work tickets (path indices) from each instance's own counter; a wave
// moves on once its lanes have drained an instance, so an instance's
// arguments stay uniform across the wave and the cooperative splat and
// gradient scatter work unchanged.  Waves that finish an instance early start
// on the next one while others drain: no launch gaps, one tail per launch.
// SC: the kinds of scene among the entries (kScAny when some are in the tree)
template <int SC>
__global__ void __launch_bounds__(1024) k_trace_batch(const PassArgs* __restrict__ T, int n) {
  extern __shared__ int lds[];
  for (int i = 0; i < n; ++i) trace_run<false, false, false, false, SC>(table_ptr(T, i), lds);
}
// One table entry through the single-instance forward, at its register
// budget (five waves per SIMD without the heightfield walk, four with it).
// Batches run their largest instances' forwards through it.
template <int SC>
__global__ void __launch_bounds__(1024, (SC & kScHf) ? 4 : 5) k_trace_entry(const PassArgs* __restrict__ T) {
  extern __shared__ int lds[];
  trace_run<false, false, false, false, SC>(table_ptr(T, 0), lds);
}
template <int SC>
__global__ void __launch_bounds__(1024) k_lrb3_batch(const PassArgs* __restrict__ T, int n) {
  extern __shared__ int lds[];
  for (int i = 0; i < n; ++i) lrb3_run<SC>(table_ptr(T, i), lds);
}
// One detached entry of the table as the single-instance kernel runs it,
// without the loop over entries, which holds live state across the
// instances.  Batches run their large detached instances through it.
template <int SC>
__global__ void __launch_bounds__(1024) k_lrb3_entry(const PassArgs* __restrict__ T) {
  extern __shared__ int lds[];
  lrb3_run<SC>(table_ptr(T, 0), lds);
}

#ifdef LT_COUNTERS
}  // namespace counted
#endif

// ---------------------------------------------------------------- launchers
static size_t stack_bytes(const PassArgs& A, int block) { return (size_t)A.sc.stack_n * block * sizeof(int); }
static size_t agrad_bytes(const PassArgs& A) { return A.agrad_lds ? (size_t)A.n_texels * 3 * sizeof(float) : 0; }
static size_t legrad_bytes(const PassArgs& A) {
  return A.legrad_lds ? (size_t)A.sc.em_tex_res * A.sc.em_tex_res * 3 * sizeof(float) : 0;
}

// allow the backward kernels the device's full LDS per workgroup
static const std::initializer_list<const void*> kLdsKernels = {
    (const void*)k_naive_bwd,
    (const void*)k_reslrb_bwd<0>, (const void*)k_reslrb_bwd<1>, (const void*)k_reslrb_bwd<2>, (const void*)k_reslrb_bwd<3>,
    (const void*)k_lrb2_bwd<1>, (const void*)k_lrb2_bwd<3>,
    (const void*)k_lrb3_bwd<0>, (const void*)k_lrb3_bwd<1>, (const void*)k_lrb3_bwd<2>, (const void*)k_lrb3_bwd<3>,
    (const void*)k_lrb3_p2<1>, (const void*)k_lrb3_p2<3>, (const void*)k_lrb3_p3<1>, (const void*)k_lrb3_p3<3>,
    (const void*)k_lrb3_batch<kScBatch>, (const void*)k_lrb3_batch<1 | kScBatch>, (const void*)k_lrb3_batch<1 | kScAny | kScBatch>,
    (const void*)k_lrb3_entry<0>, (const void*)k_lrb3_entry<1>, (const void*)k_lrb3_entry<2>, (const void*)k_lrb3_entry<3>,
    (const void*)k_camera_prb<1>, (const void*)k_camera_prb<3>};
hipError_t set_lds_limit(int bytes) {
  for (const void* f : kLdsKernels) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  return set_lds_limit_att(bytes);
}

// Residency is asked of one instantiation of each kernel: those for the other
// kinds of scene hold the same number of waves (their launch bounds).
int resident_groups(BwdKernel k, int block, size_t lds) {
  // the answer depends only on the arguments and the device: cache it
  static std::mutex mu;
  static std::map<std::tuple<int, int, int, size_t>, int> memo;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) (void)hipGetLastError();
  const auto key = std::make_tuple(dev, (int)k, block, lds);
  {
    std::lock_guard<std::mutex> g(mu);
    auto it = memo.find(key);
    if (it != memo.end()) return it->second;
  }
  const void* f = nullptr;
  switch (k) {
    case BwdKernel::naive: f = (const void*)k_naive_bwd; break;
    case BwdKernel::reslrb: f = (const void*)k_reslrb_bwd<1>; break;
    case BwdKernel::lrb3: f = (const void*)k_lrb3_bwd<1>; break;
    case BwdKernel::lrb3_batch: f = (const void*)k_lrb3_batch<1 | kScBatch>; break;
    case BwdKernel::lrb3_entry: f = (const void*)k_lrb3_entry<1>; break;
    case BwdKernel::lrb3_p2: f = (const void*)k_lrb3_p2<1>; break;
    case BwdKernel::lrb3_p3: f = (const void*)k_lrb3_p3<1>; break;
    case BwdKernel::lrb2: f = (const void*)k_lrb2_bwd<1>; break;
    case BwdKernel::camera_prb: f = (const void*)k_camera_prb<1>; break;
    default: f = att_kernel(k); break;
  }
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, block, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  std::lock_guard<std::mutex> g(mu);
  memo[key] = n;
  return n;
}

hipError_t launch_trace_batch(const PassArgs* table, int n, int kind, int stack_n, int grid, int block, hipStream_t s) {
  hipLaunchKernelGGL((kind & kScTree) ? k_trace_batch<1 | kScAny | kScBatch> : k_trace_batch<1 | kScBatch>, dim3(grid), dim3(block),
                     (size_t)stack_n * block * sizeof(int), s, table, n);
  return hipGetLastError();
}
hipError_t launch_trace_entry(const PassArgs* entry, int kind, int stack_n, int grid, int block, hipStream_t s) {
  by_scene(kind, [&](auto sc) {
    hipLaunchKernelGGL(k_trace_entry<sc>, dim3(grid), dim3(block), (size_t)stack_n * block * sizeof(int), s, entry);
  });
  return hipGetLastError();
}
hipError_t launch_lrb3_batch(const PassArgs* table, int n, int kind, int stack_n, size_t grad_lds, int grid, int block,
                             hipStream_t s) {
  hipLaunchKernelGGL((kind & kScTree) ? k_lrb3_batch<1 | kScAny | kScBatch> : (kind & kScHf) ? k_lrb3_batch<1 | kScBatch> : k_lrb3_batch<kScBatch>,
                     dim3(grid), dim3(block),
                     (size_t)stack_n * block * sizeof(int) + grad_lds, s, table, n);
  return hipGetLastError();
}
hipError_t launch_lrb3_entry(const PassArgs* entry, int kind, int stack_n, size_t grad_lds, int grid, int block,
                             hipStream_t s) {
  by_scene(kind, [&](auto sc) {
    hipLaunchKernelGGL(k_lrb3_entry<sc>, dim3(grid), dim3(block), (size_t)stack_n * block * sizeof(int) + grad_lds, s,
                       entry);
  });
  return hipGetLastError();
}

hipError_t read_counters(uint64_t* out, bool reset, hipStream_t s) {
#ifdef LT_COUNTERS
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  e = hipMemcpyFromSymbol(out, HIP_SYMBOL(lt_counters), 16 * sizeof(uint64_t), 0, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = add_counters_att(out, reset);
  if (e != hipSuccess || !reset) return e;
  uint64_t z[16] = {0};
  return hipMemcpyToSymbol(HIP_SYMBOL(lt_counters), z, sizeof(z), 0, hipMemcpyHostToDevice);
#else
  (void)out; (void)reset; (void)s;
  return hipErrorNotSupported;
#endif
}

hipError_t launch_trace(const PassArgs& A, bool tape, bool resv, int grid, int block, hipStream_t s) {
  const size_t sh = stack_bytes(A, block);
  if (tape && resv)
    by_scene_hf(scene_kind(A.sc), [&](auto sc) {
      hipLaunchKernelGGL((k_trace<true, true, false, false, sc>), dim3(grid), dim3(block), sh, s, A);
    });
  else
    by_scene(scene_kind(A.sc), [&](auto sc) {
      if (tape) hipLaunchKernelGGL((k_trace<true, false, false, false, sc>), dim3(grid), dim3(block), sh, s, A);
      else if (resv) hipLaunchKernelGGL((k_trace<false, true, false, false, sc>), dim3(grid), dim3(block), sh, s, A);
      else hipLaunchKernelGGL((k_trace<false, false, false, false, sc>), dim3(grid), dim3(block), sh, s, A);
    });
  return hipGetLastError();
}

hipError_t launch_camera(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_camera<sc>, dim3(grid), dim3(block), stack_bytes(A, block), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_camera_prb(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_camera_prb<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A), s, A);
  });
  return hipGetLastError();
}

hipError_t launch_naive_bwd(const PassArgs& A, int grid, int block, hipStream_t s) {
  hipLaunchKernelGGL(k_naive_bwd, dim3(grid), dim3(block), agrad_bytes(A) + legrad_bytes(A), s, A);
  return hipGetLastError();
}

hipError_t launch_reslrb_bwd(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_reslrb_bwd<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A) + legrad_bytes(A), s,
                       A);
  });
  return hipGetLastError();
}

hipError_t launch_lrb3_bwd(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_lrb3_bwd<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A) + legrad_bytes(A), s,
                       A);
  });
  return hipGetLastError();
}

hipError_t launch_trace_splats(const PassArgs& A, bool resv, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    const size_t sh = stack_bytes(A, block);
    if (resv) hipLaunchKernelGGL((k_trace<false, true, true, false, sc>), dim3(grid), dim3(block), sh, s, A);
    else hipLaunchKernelGGL((k_trace<false, false, true, false, sc>), dim3(grid), dim3(block), sh, s, A);
  });
  return hipGetLastError();
}
hipError_t launch_trace_gsamples(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL((k_trace<false, false, false, true, sc>), dim3(grid), dim3(block), stack_bytes(A, block), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_lrb2_bwd(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_lrb2_bwd<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A) + legrad_bytes(A), s,
                       A);
  });
  return hipGetLastError();
}

hipError_t launch_lrb3_p2(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_lrb3_p2<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A) + legrad_bytes(A), s,
                       A);
  });
  return hipGetLastError();
}
hipError_t launch_lrb3_p3(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL(k_lrb3_p3<sc>, dim3(grid), dim3(block), stack_bytes(A, block) + agrad_bytes(A), s,
                       A);
  });
  return hipGetLastError();
}

static int blocks_for(size_t items, size_t most) {
  return (int)std::max<size_t>(1, std::min<size_t>((items + 255) / 256, most));
}
hipError_t launch_film_resolve(const PassArgs& A, hipStream_t s) {
  hipLaunchKernelGGL(k_film_resolve, dim3(blocks_for((size_t)A.sc.W * A.sc.H * 3, 4096)), dim3(256), 0, s, A);
  return hipGetLastError();
}
static size_t begin_items(const PassArgs& A) {
  return A.cells ? (size_t)(A.sc.W + 1) * (A.sc.H + 1) * (kCellFloats / 4) : A.image ? (size_t)A.sc.W * A.sc.H * 3 : 0;
}
static size_t hf_items(const PassArgs& A) { return A.begin_hf ? (size_t)2 * A.sc.hf_G * A.sc.hf_G : 0; }
hipError_t launch_begin(const PassArgs& A, unsigned int* counters, size_t n_counters, hipStream_t s) {
  const int grid = std::max(blocks_for(std::max(std::max(begin_items(A), hf_items(A)), n_counters), 4096),
                            A.begin_hf ? kHfParts : 1);
  hipLaunchKernelGGL(k_begin, dim3(grid), dim3(256), 0, s, A, counters, n_counters);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !A.begin_hf || A.sc.hf_G * A.sc.hf_G <= kHfOne) return e;
  hipLaunchKernelGGL(k_hf_whole, dim3(1), dim3(64), 0, s, const_cast<float*>(A.sc.hf_hb));
  return hipGetLastError();
}
hipError_t launch_begin_batch(const PassArgs* table, int n, size_t clear_floats, size_t hf_cells, unsigned int* counters,
                              size_t n_counters, hipStream_t s) {
  const int grid = std::max(blocks_for(std::max(clear_floats / 4, 2 * hf_cells), 1024), hf_cells ? kHfParts : 1);
  hipLaunchKernelGGL(k_begin_batch, dim3(grid, n), dim3(256), 0, s, table, counters, n_counters);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || hf_cells <= (size_t)kHfOne) return e;
  hipLaunchKernelGGL(k_hf_whole_batch, dim3(n), dim3(64), 0, s, table);
  return hipGetLastError();
}
hipError_t launch_loss(const float* I, const float* T, size_t n, float* dI, double* acc, float* loss, hipStream_t s) {
  // Every workgroup adds to the same eight lines at its end, so few of them,
  // until their loads in flight no longer fill the memory's bandwidth (from
  // about 20M values on, as 1024 groups): 3M values 22 us with 1024 groups and
  // 33 with 2048, 19M 47 and 56, 25M 78 and 70, 50M 146 and 123, 100M 285 and 225.
  const size_t most = n <= (size_t)20 << 20 ? 1024 : 2048;
  hipLaunchKernelGGL(k_loss, dim3(blocks_for((n + 3) / 4, most)), dim3(256), 0, s, I, T, n, dI, acc, loss);
  return hipGetLastError();
}
hipError_t launch_loss_batch(const PassArgs* table, int n, size_t largest, hipStream_t s) {
  hipLaunchKernelGGL(k_loss_batch, dim3(blocks_for((largest + 3) / 4, 512), n), dim3(256), 0, s, table);
  return hipGetLastError();
}

}  // namespace lt
