// Path code shared by the detached and the attached kernels: one vertex of a
// light path, the work distribution of the persistent loops and the gradient
// accumulators.  Included by one translation unit per kernel family.
#pragma once
#include "lt_device.h"
#include "lt_launch.h"

namespace lt {

// The instrumented build (event counters on) gives its kernels their own
// symbol names so that profiles keep the two builds apart.
#ifdef LT_COUNTERS
inline namespace counted {
#endif

// The pass arguments, re-read from here on.  They are constant, so the
// compiler moves every load of them (and what follows from them, such as the
// ten round keys of the random numbers) out of the persistent loops, runs out
// of scalar registers and keeps a hundred and more of them in lanes of vector
// registers (100-190 spilled in each traversal kernel, 300-1600 v_readlane in
// its code).  A pointer it cannot see through ties the loads to the loop
// iteration: they come back through the scalar cache where they are used.
// Measured: attached pass 3 with rough conductors 256 -> 237 vector registers
// and 28 -> 16 bytes of scratch, attached ResLRB 238 -> 195 registers; the
// 128x128 caustic's LRB-3 step at 16M paths 21.0 -> 18.0 ms, the 256x256 box's
// at depth 32 9.93 -> 9.49 ms.
typedef const __attribute__((address_space(4))) PassArgs* ArgsPtr;
__device__ __forceinline__ const PassArgs& fresh(ArgsPtr p) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(p));
#endif
  return *(const PassArgs*)p;
}
// the arguments of a kernel whose only parameter is a PassArgs
__device__ __forceinline__ ArgsPtr kernel_args() {
#if defined(__HIP_DEVICE_COMPILE__)
  return (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
#else
  return nullptr;  // host pass of the device function: never executed
#endif
}

// One vertex of a light path: closest hit, material dispatch, sensor
// connection geometry and the sampling of the next direction.
struct Event {
  int prim;        // hit primitive, -1 on a miss
  int kind;        // 0 path ended at this hit (miss/absorber), 1 Lambertian or rough
                   // conductor (a texel, a connection, a scatter linear in rho), 2 dielectric
  bool cond;       // kind 1 on a rough conductor
  int texel;       // Lambertian texel
  f3 rho;          // Lambertian albedo
  bool valid;      // sensor connection exists
  float ux, uy, g; // film position and connection factor (C = beta rho g)
  float cos_in;
  int lobe, fail;  // dielectric: lobe 2 reflect / 4 refract, fail 7/8; conductor: fail 9
                   // (arrived behind its shading normal), 7/8 (no reflection)
  bool cont;       // the path continues with the updated ray
  float u_res;     // reservoir uniform of this vertex
  int slot;        // hit triangle in BVH order
  float par;       // dielectric: refractive index; conductor: roughness; else 1
  f3 x;            // hit point
  float gw, gq;    // Lambertian scatter weight over rho (cos / (pi q) when guided, else 1)
                   // and the guided density q (0: cosine sampling)
  int gcomp;       // guided component (0 cosine, k + 1 lobe k)
  bool illc;       // ill-conditioned vertex for attached derivatives (grazing hit,
                   // refraction near the critical angle, short segment, or a
                   // connection next to a tent-filter kink)
};

__device__ __forceinline__ bool near_kink(float u) {
  float d = u - 0.5f;
  return fabsf(d - rintf(d)) < 1e-3f;
}

// cmode: 0 no sensor connection, 1 full connection test (with shadow
// ray), 2 connection geometry only (known visible from an earlier replay).
template <int SC>
__device__ __forceinline__ Event bounce(const PassArgs& A, uint32_t path, int j, Ray& r, int cmode,
                                        int* stk, int ss) {
  const DevScene& sc = A.sc;
  Event ev;
  ev.prim = -1; ev.kind = 0; ev.cond = false; ev.texel = -1; ev.rho = {0.f, 0.f, 0.f}; ev.valid = false;
  ev.ux = ev.uy = ev.g = 0.f; ev.lobe = 0; ev.fail = 0; ev.cont = false; ev.u_res = 1.0f; ev.cos_in = 0.f;
  ev.slot = -1; ev.x = {0.f, 0.f, 0.f}; ev.illc = false; ev.gw = 1.0f; ev.gq = 0.f; ev.gcomp = 0; ev.par = 1.0f;
  Hit h = closest_hit<SC>(sc, ray_origin(r), r.w, kTmin, 3.0e38f, stk, ss);
  if (h.tri < 0) return ev;
  Surf s = surface(sc, h.tri, r);
  ev.prim = s.prim;
  ev.slot = h.tri;
  ev.x = s.x;
  const int mt = s.mat & 3;
  if (mt == 0) return ev;
  ev.cos_in = dot(r.w, s.ng);
  // grazing hit (hit-point derivatives ~ 1/cos) or a short segment (the
  // segment direction carries position rounding amplified by 1/length)
  f3 seg = s.x - r.x;
  ev.illc = fabsf(ev.cos_in) < 0.02f || dot(seg, seg) < 4e-4f;
  u4f u = (mt != 2 || j < A.D) ? rng4(A.seed, path, (uint32_t)j, 0u) : u4f{0.f, 0.f, 0.f, 1.f};
  ev.u_res = u.u3;
  if (mt == 1 || mt == 3) {
    ev.kind = 1;
    ev.cond = mt == 3;
    ev.texel = texel_of(sc, s, s.mat >> 2);
    ev.rho = ld3(A.albedo + (size_t)ev.texel * 3);
    f3 nc = s.ng;  // conductor: arrival-side shading normal
    float rough = 0.f;
    if (ev.cond) {
      rough = s.par;
      ev.par = s.par;
      f3 ns = s.prim >= sc.n_static ? hf_shading_normal(sc, A.heights, A.slopes, s) : s.ng;
      nc = ev.cos_in < 0.0f ? ns : ns * -1.0f;
      if (!(dot(r.w, nc) < 0.0f)) { ev.fail = 9; return ev; }
    }
    if (cmode)
      ev.valid = connect<SC>(sc, s, r.w, A.Kfilm, ev.ux, ev.uy, ev.g, stk, ss, cmode == 2, ev.cond ? &nc : nullptr, rough);
    // the tent filter has kinks where u - 1/2 is an integer: within 1e-3 px
    // of one the splat-position derivative is one-sided (rounding picks the side)
    if (ev.valid && (near_kink(ev.ux) || near_kink(ev.uy))) ev.illc = true;
    if (j < A.D && ev.cond) {
      f3 wo;
      float wgt;
      int code = conductor_scatter(r.w * -1.0f, nc, s.ng, ev.cos_in < 0.0f ? 1.0f : -1.0f, rough, u.u0, u.u1, wo, wgt);
      if (code) { ev.fail = code; return ev; }
      ev.gw = wgt;
      r.w = wo; r.x = s.x; r.offn = s.ng; r.off = true;
      ev.cont = true;
      return ev;
    }
    if (j < A.D) {
      f3 na = ev.cos_in < 0.0f ? s.ng : s.ng * -1.0f;
      const float4* ge = A.gtab ? A.gtab + (size_t)(2 * ev.texel + (ev.cos_in < 0.0f ? 0 : 1)) * kGTabF4 : nullptr;
      if (ge && ge[1].w >= 0.f) {
        // guided scatter (component by u2, direction by u0, u1), weight
        // f cos / q = rho cos / (pi q) with q held fixed
        float q;
        int comp;
        f3 w = gtab_sample(ge, na, u.u2, u.u0, u.u1, q, comp);
        ev.gcomp = comp;
        float c = dot(w, na);
        if (!(q > 0.f && c > 0.f)) return ev;
        ev.gw = c / (3.14159265358979323846f * q);
        ev.gq = q;
        r.w = w;
      } else {
        r.w = cosine_dir(na, u.u0, u.u1);
      }
      r.x = s.x; r.offn = s.ng; r.off = true;
      ev.cont = true;
    }
    return ev;
  }
  ev.kind = 2;
  ev.par = s.par;
  if (j >= A.D) return ev;
  f3 ns = s.ng;
  if (s.prim >= sc.n_static) ns = hf_shading_normal(sc, A.heights, A.slopes, s);
  f3 wo; bool refl;
  float cos_t = 1.f;
  int code = dielectric(r.w, s.ng, ns, s.par, u.u2, wo, refl, cos_t);
  if (code == 7) { ev.fail = 7; return ev; }
  ev.lobe = refl ? 2 : 4;
  // refraction near the critical angle: d(cos_t) ~ 1/cos_t amplifies FP32
  // rounding of the primal direction by ~1/cos_t^2 in the derivatives
  if (cos_t < 0.1f) ev.illc = true;
  if (code == 8) { ev.fail = 8; return ev; }
  r.w = wo; r.x = s.x; r.offn = s.ng; r.off = true;
  ev.cont = true;
  return ev;
}

__device__ __forceinline__ uint32_t sig_event(uint32_t h, const Event& ev) {
  if (ev.prim < 0) return fnv1a(h, 0u);
  h = fnv1a(h, (uint32_t)ev.prim + 1u);
  if (ev.kind == 1) {
    h = fnv1a(h, (uint32_t)ev.texel + 1u);
    if (ev.fail == 9) return fnv1a(h, 9u);
    h = fnv1a(h, ev.valid ? 1u : 0u);
    if (ev.fail) h = fnv1a(h, (uint32_t)ev.fail);
  } else if (ev.kind == 2) {
    if (ev.fail == 7) return fnv1a(h, 7u);
    if (ev.lobe) h = fnv1a(h, (uint32_t)ev.lobe);
    if (ev.fail == 8) h = fnv1a(h, 8u);
  }
  return h;
}

// Work distribution.  Path indices are dealt out by eight counters,
// counter c handing out p = 8k + c (k = 0, 1, ...), each on a cache line of
// its own: with one counter for all the waves of the chip, its line was the
// busiest address of a pass and its returning atomics serialised (measured:
// the box forward 5.8 -> 4.3 ms, the fused LRB-3 backward 8.4 -> 6.8 ms).
// A wave starts on the counter of its XCD and, once that class is used up,
// moves to the next; having found all eight used up, it is done.  Every
// index below n_paths is handed out exactly once whatever the XCD reads.
// Paths that `accept` rejects (default: the path mask) get their per-path
// outputs cleared by `on_skip`.
// The same over any eight classes of work: class c holds limit(c) items,
// the k-th of them being index(c, k).
// In a long pass a wave draws 64 indices at a time and hands them out as its
// lanes fall free, so that the atomic's round trip comes once in about five
// steps of the wave, not in every one.  A wave then holds up to a path a lane
// that others could have taken at the end: from eight paths a lane on that is
// lost in the gain.  Path by path -> ahead, us, at two paths a lane a mesh's
// step 2070 -> 2340; at eight the 256x256 box at depth 32 forward 1046 -> 976,
// LRB-3 1345 -> 1297, the caustic attached 1486 -> 1487; at sixteen 1838 ->
// 1691, 2248 -> 2145 and 2741 -> 2695; at thirty-two 3405 -> 3115, 4042 ->
// 3817 and 5303 -> 5194.
constexpr unsigned int kDraw = 64;
template <int SC>
__device__ __forceinline__ bool draws_ahead(uint32_t n_paths) {
  return !(SC & kScBatch) && n_paths >> 3 >= gridDim.x * blockDim.x;
}
template <typename Limit, typename Index, typename Skip, typename Accept>
__device__ __forceinline__ void refill_classes(WorkQ& q, bool& alive, bool& exhausted, uint32_t& item, Limit limit,
                                               Index index, Skip on_skip, Accept accept) {
  if (q.ahead) {
    while (true) {
      const bool need = !alive && !exhausted;
      const uint64_t m = __ballot(need);
      if (m == 0ull) break;
      if (q.next == q.end) {
        if (q.tried == kWorkClasses) {  // every class used up
          if (need) exhausted = true;
          break;
        }
        const uint32_t lim = limit(q.cls);
        unsigned int k = 0;
        if (__lane_id() == 0) k = atomicAdd(q.base + q.cls * kCtrStride, kDraw);
        k = (unsigned int)__builtin_amdgcn_readfirstlane((int)k);
        q.next = k < lim ? k : lim;
        q.end = k < lim && lim - k > kDraw ? k + kDraw : lim;
        if (q.next == q.end) {  // this class is used up: the next one
          q.cls = (q.cls + 1) & (kWorkClasses - 1);
          ++q.tried;
          continue;
        }
      }
      const uint32_t mine = q.next + (uint32_t)__popcll(m & lanemask_lt());
      if (need && mine < q.end) {
        const uint32_t p = index(q.cls, mine);
        if (!accept(p)) on_skip(p);
        else { alive = true; item = p; }
      }
      const uint32_t left = q.end - q.next, asked = (uint32_t)__popcll(m);
      q.next += asked < left ? asked : left;
    }
    return;
  }
  while (true) {
    bool need = !alive && !exhausted;
    if (__ballot(need) == 0ull) break;
    if (q.tried == kWorkClasses) {  // every class used up
      if (need) exhausted = true;
      break;
    }
    const uint32_t k = fetch_paths(q.base + q.cls * kCtrStride, need);
    const bool over = need && k >= limit(q.cls);
    const uint32_t p = index(q.cls, k);
    if (__ballot(over) != 0ull) {  // this class is used up: the next one
      q.cls = (q.cls + 1) & (kWorkClasses - 1);
      ++q.tried;
    }
    if (need && !over) {
      if (!accept(p)) on_skip(p);
      else { alive = true; item = p; }
    }
  }
}
// paths: class c holds p = 8k + c below n_paths
template <typename Skip, typename Accept>
__device__ __forceinline__ void refill(const PassArgs& A, WorkQ& q, bool& alive, bool& exhausted, uint32_t& path,
                                       Skip on_skip, Accept accept) {
  const uint32_t N = (uint32_t)A.n_paths;
  refill_classes(
      q, alive, exhausted, path,
      [&](int c) { return N > (uint32_t)c ? (N - (uint32_t)c + (uint32_t)kWorkClasses - 1u) / (uint32_t)kWorkClasses : 0u; },
      [&](int c, uint32_t k) { return k * (uint32_t)kWorkClasses + (uint32_t)c; }, on_skip, accept);
}
template <typename Skip>
__device__ __forceinline__ void refill(const PassArgs& A, WorkQ& q, bool& alive, bool& exhausted, uint32_t& path,
                                       Skip on_skip) {
  refill(A, q, alive, exhausted, path, on_skip, [&](uint32_t p) { return !(A.mask && A.mask[p] == 0); });
}
// LRB-3 pass 3: the entries pass 2 appended, region by region
__device__ __forceinline__ void refill_hand(const PassArgs& A, WorkQ& q, bool& alive, bool& exhausted,
                                            uint32_t& item) {
  refill_classes(
      q, alive, exhausted, item, [&](int c) { return A.hand_app[c * kCtrStride]; },
      [&](int c, uint32_t k) { return (uint32_t)c * A.hand_region + k; }, [&](uint32_t) {},
      [&](uint32_t) { return true; });
}

// Pass 2's append of one entry per path that has one (`put`): grouped by the
// path's class, one atomic per class present in the wave; returns the
// entry's index (valid where put).  Every lane of the wave calls it.
__device__ __forceinline__ uint32_t hand_append(const PassArgs& A, bool put, uint32_t path) {
  const int c = (int)(path & (uint32_t)(kWorkClasses - 1));
  uint32_t slot = 0;
  bool todo = put;
  while (true) {
    const uint64_t m = __ballot(todo);
    if (m == 0ull) break;
    const int cl = __shfl(c, __ffsll((unsigned long long)m) - 1);
    const bool mine = todo && c == cl;
    const uint32_t k = fetch_paths(A.hand_app + cl * kCtrStride, mine);
    if (mine) { slot = (uint32_t)cl * A.hand_region + k; todo = false; }
  }
  return slot;
}

// Non-finite values (a division by a vanishing cosine, length or
// determinant on a degenerate path) never reach an atomic: they are dropped
// and counted in stats[1].
__device__ __forceinline__ void count_nonfinite(const PassArgs& A) {
  if (A.stats) atomicAdd(A.stats + 1, 1ull);
}
__device__ __forceinline__ void keep_finite(const PassArgs& A, bool& has, f3 v) {
  if (has && !(isfinite(v.x) && isfinite(v.y) && isfinite(v.z))) { has = false; count_nonfinite(A); }
}
// Textured-emitter gradients.  Every path adds to the texel it was emitted
// from, so a small texture takes all of them on a few cache lines, where
// the atomics serialize.  With A.legrad_lds each workgroup pre-reduces them
// in an LDS copy of the texture (`le`, past the albedo copy) and adds that
// to the caller's array once, at its end.  Every thread of the workgroup
// calls begin and end.
__device__ __forceinline__ float* legrad_begin(const PassArgs& A, int* lds) {
  float* le = reinterpret_cast<float*>(lds);
  if (!A.legrad_lds) return le;
  const int n = A.sc.em_tex_res * A.sc.em_tex_res * 3;
  for (int i = threadIdx.x; i < n; i += blockDim.x) le[i] = 0.f;
  __syncthreads();
  return le;
}
__device__ __forceinline__ void legrad_end(const PassArgs& A, float* le) {
  if (!A.legrad_lds) return;
  __syncthreads();
  if (!A.g_le_tex) return;
  const int n = A.sc.em_tex_res * A.sc.em_tex_res * 3;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    float v = le[i];
    if (v != 0.f) atomicAdd(A.g_le_tex + i, v);
  }
}

// emitter-gradient accumulation of one path, (a0, a1, a2) in place of zeros
// when any is non-finite: into the lane's FP64 sums (one radiance), or onto
// the path's texel of a textured emitter (texel >= 0; the workgroup's LDS
// copy `le` with A.legrad_lds)
__device__ __forceinline__ void add_le(const PassArgs& A, double& g0, double& g1, double& g2, double a0, double a1,
                                       double a2, int texel = -1, float* le = nullptr) {
  if (!(isfinite(a0) && isfinite(a1) && isfinite(a2))) { count_nonfinite(A); return; }
  if (texel >= 0) {
    if (!A.g_le_tex) return;
    if (A.legrad_lds) {
      float* d = le + 3 * texel;
      if (a0 != 0.0) atomicAdd(d + 0, (float)a0);
      if (a1 != 0.0) atomicAdd(d + 1, (float)a1);
      if (a2 != 0.0) atomicAdd(d + 2, (float)a2);
      return;
    }
    float* d = A.g_le_tex + 3 * texel;
    if (a0 != 0.0) atomicAdd(d + 0, (float)a0);
    if (a1 != 0.0) atomicAdd(d + 1, (float)a1);
    if (a2 != 0.0) atomicAdd(d + 2, (float)a2);
    return;
  }
  g0 += a0; g1 += a1; g2 += a2;
}

// Albedo gradients.  With A.agrad_lds each workgroup pre-reduces them in an
// LDS copy of the texture set and adds that to the caller's array once, at
// its end.  Without it (the set is large, or the copy would cost resident
// workgroups) they go to the caller's array through a one-entry
// write-combining cache per wave: sums for the texel most of the wave hits
// stay in registers while later scatters hit the same texel, so a constant
// or small texture takes one atomic per wave and texel change, not one per
// scatter.  Every thread of the workgroup calls begin and end, and every
// lane of a wave calls scatter.
// The LDS copy is addressed through a pointer derived only from the
// workgroup's LDS array, and the choice between it and the caller's array is
// a branch on the uniform flag, not a pointer select: each side then compiles
// to LDS or global atomics rather than flat ones.
struct AGrad {
  float* lds;
  int idx;  // cached texel (wave-uniform), -1 when empty
  float s0, s1, s2;
};
__device__ __forceinline__ AGrad agrad_begin(const PassArgs& A, int* lds) {
  AGrad g{reinterpret_cast<float*>(lds), -1, 0.f, 0.f, 0.f};
  if (!A.agrad_lds) return g;
  const int n = A.n_texels * 3;
  for (int i = threadIdx.x; i < n; i += blockDim.x) g.lds[i] = 0.f;
  __syncthreads();
  return g;
}
__device__ __forceinline__ void agrad_flush(const PassArgs& A, AGrad& g) {
  if (g.idx >= 0 && __lane_id() == 0) {
    float* d = A.g_albedo + (size_t)g.idx * 3;
    if (g.s0 != 0.f) atomicAdd(d + 0, g.s0);
    if (g.s1 != 0.f) atomicAdd(d + 1, g.s1);
    if (g.s2 != 0.f) atomicAdd(d + 2, g.s2);
  }
}
__device__ __forceinline__ void scatter_albedo(const PassArgs& A, AGrad& g, bool has, int texel, f3 v) {
  if (A.agrad_lds) {
    // Each lane adds its own triplet: gathering lanes for wider instructions,
    // as global atomics want it, costs more here than the LDS saves.  So does
    // summing the lanes of one texel first, even with one texel for all: LRB-3
    // of 1M paths, box 591 us against 596 summed, caustic of 4M 2259 and 2266,
    // detached 1082 and 1098; the tape sweep 164 and 167, 610 and 619 (the
    // tumbler's alone gains, 61 -> 52).  Nor is the sum less exact: against the
    // FP64 sum of 64 parts both are at 0.3-2e-6, which is the rounding of the
    // caller's FP32 array, with 256 copies as with 2560.
    if (has) {
      LT_COUNT(6, 3);
      float* q = g.lds + 3 * texel;
      atomicAdd(q, v.x);
      atomicAdd(q + 1, v.y);
      atomicAdd(q + 2, v.z);
    }
    return;
  }
  uint64_t m = __ballot(has);
  if (m == 0ull) return;
  const int lane = __lane_id();
  int lead = __ffsll((unsigned long long)m) - 1;
  int li = __shfl(texel, lead);
  bool mine = has && texel == li;
  uint64_t same = __ballot(mine);
  if (li == g.idx || __popcll(same) >= 8) {
    LT_COUNT(6, mine ? 3 : 0);
    float s0 = mine ? v.x : 0.f, s1 = mine ? v.y : 0.f, s2 = mine ? v.z : 0.f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {  // xor butterfly: every lane ends with the same sums
      s0 += __shfl_xor(s0, o); s1 += __shfl_xor(s1, o); s2 += __shfl_xor(s2, o);
    }
    if (li != g.idx) {
      agrad_flush(A, g);
      g.idx = li; g.s0 = 0.f; g.s1 = 0.f; g.s2 = 0.f;
    }
    g.s0 += s0; g.s1 += s1; g.s2 += s2;
    has = has && !mine;
    if (m == same) return;
  }
  scatter3_wave(A.g_albedo, has, texel, v);
}
__device__ __forceinline__ void agrad_end(const PassArgs& A, AGrad& g) {
  if (!A.agrad_lds) {
    agrad_flush(A, g);
    return;
  }
  __syncthreads();
  const int n = A.n_texels * 3;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    float v = g.lds[i];
    if (v != 0.f) atomicAdd(A.g_albedo + i, v);
  }
}

// The workgroup's next instance of a batch reuses the LDS past the traversal
// stacks: no wave may start on it before every wave has flushed the copies.
__device__ __forceinline__ void lds_grads_done(const PassArgs& A) {
  if (A.hgrad_lds || A.agrad_lds || A.legrad_lds) __syncthreads();
}
// LDS past the traversal stacks (stack_n entries per lane) and the albedo copy
__device__ __forceinline__ int* past_agrad(const PassArgs& A, int* lds, int stack_n) {
  return lds + stack_n * (int)blockDim.x + (A.agrad_lds ? A.n_texels * 3 : 0);
}

// End of a pass: the lanes' FP64 emitter-gradient sums and guard counts, summed
// over the workgroup and added to the workgroup's accumulator slot; the last
// workgroup to finish adds the slots to the caller's gradient (last_adds).
// Every thread calls it.  Atomics on one address serialise (about 12 ns each here),
// and the waves of a pass end together.  With one triplet a wave on one address
// the step took, before -> after: box with taped AD, 1M paths 809 -> 690 us
// (4096 waves in the sweep); 33x33 caustic with taped AD, 100k paths 223 -> 177
// us; bidirectional 1.10 -> 1.01 ms; 64x64 box, 16k paths 132 -> 123 us.
__device__ __forceinline__ void flush_sums(const PassArgs& A, double g0, double g1, double g2,
                                           unsigned long long guards = 0, bool last_adds = true) {
  __shared__ double part[16][4];
  static_assert(sizeof(part) <= kStaticLds, "LDS beside the launch's");
  g0 = wave_sum(g0); g1 = wave_sum(g1); g2 = wave_sum(g2);
  double gd = wave_sum((double)guards);  // whole numbers far below 2^53
  __syncthreads();  // the previous use of `part` (a batch's instance before) is over
  if (__lane_id() == 0) {
    double* p = part[threadIdx.x >> 6];
    p[0] = g0; p[1] = g1; p[2] = g2; p[3] = gd;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  if (threadIdx.x < 4) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += part[w][threadIdx.x];
    if (t != 0.0) {
      if (threadIdx.x < 3) {
        if (A.g_le) done_atomic(atomicAdd(A.g_Le_acc + (blockIdx.x & (kAccSlots - 1)) * kAccStride + threadIdx.x, t));
      } else if (A.stats) {
        atomicAdd(A.stats, (unsigned long long)t);
      }
    }
  }
  if (!last_adds || !A.g_le) return;
  // the pass's last workgroup adds the slots to the caller's gradient
  unsigned int done = 0;
  if (threadIdx.x == 0) done = atomicAdd(A.ticket, 1u);
  done = (unsigned int)__builtin_amdgcn_readfirstlane((int)done);
  if (done != gridDim.x - 1 || threadIdx.x >= 3) return;
  double t = 0.0;
  for (int k = 0; k < kAccSlots; ++k)  // read where the atomics execute
    t += atomicAdd(A.g_Le_acc + k * kAccStride + threadIdx.x, 0.0);
  if (t != 0.0) atomicAdd(A.g_le + threadIdx.x, (float)t);
}

// Reciprocal emitter radiance, zero where a channel is zero: the emitter
// gradient of a path is its adjoint sum times this (computed once, not a
// double division per path).
struct D3R { double x, y, z; };
__device__ __forceinline__ D3R recip_le(f3 Le) {
  return {Le.x > 0.f ? 1.0 / Le.x : 0.0, Le.y > 0.f ? 1.0 / Le.y : 0.0, Le.z > 0.f ? 1.0 / Le.z : 0.0};
}

// Emitter radiance of a path.  One radiance: Le, iLe as set once per kernel,
// texel -1.  A textured emitter: the texel of the path's emission point
// (quad coordinates u0 along e1, u1 along e2, nearest texel; computed on the
// 24-bit integers of the uniforms, so exactly floor(u R)), its radiance and
// reciprocal.
__device__ __forceinline__ void path_emitter(const PassArgs& A, uint32_t path, f3& Le, D3R& iLe, int& texel) {
  const int R = A.sc.em_tex_res;
  if (R <= 0) return;
  u4f u = rng4(A.seed, path, 0u, 0u);
  const uint64_t k0 = (uint64_t)(u.u0 * 16777216.0f), k1 = (uint64_t)(u.u1 * 16777216.0f);
  const int tx = (int)((k0 * (uint64_t)R) >> 24), ty = (int)((k1 * (uint64_t)R) >> 24);
  texel = ty * R + tx;
  Le = ld3(A.Le + 3 * texel);
  iLe = recip_le(Le);
}

// Vertex 0 of a path.  With a guide the emitted direction and its density q
// come from the per-path record of the guide pass (same position draw);
// beta_1 = L_e * A cos / q, the density held fixed in every derivative.
__device__ __forceinline__ float emit_path(const PassArgs& A, uint32_t path, Ray& r) {
  float f = emit(A.sc, A.seed, path, r);
  if (A.guide_rec) {
    float4 g = A.guide_rec[path];
    r.w = mk(g.x, g.y, g.z);
    float c = fmaxf(dot(r.w, ld3(A.sc.em_n)), 0.f);
    f = g.w > 0.f ? A.sc.em_area * c / g.w : 0.f;
  }
  return f;
}

__device__ __forceinline__ float luminance(f3 c) { return 0.2126f * c.x + 0.7152f * c.y + 0.0722f * c.z; }

// Pointers read from ordinary memory are generic to the compiler, so every
// access through them would be a flat instruction (address-space check,
// counted on both the vector-memory and LDS counters).  The table is
// read-only during a launch and is read through the constant address space,
// as kernel arguments are; pointers loaded from there are taken to be global
// memory, and loads, stores and atomics through them compile to global ones.
__device__ __forceinline__ ArgsPtr table_ptr(const PassArgs* T, int i) {
  return (ArgsPtr)T + i;
}

#ifdef LT_COUNTERS
}  // namespace counted
#endif

}  // namespace lt
