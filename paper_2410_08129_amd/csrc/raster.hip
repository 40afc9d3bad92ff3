// Tile rasterizer, forward and backward (Sec. 3.2 and Sec. 3.3).
//
// Forward: one workgroup per tile; each wave owns an 8x8 pixel block, one
// lane per pixel. The tile's instances are staged through LDS in batches of
// one record per lane; each wave then lists, for each 4x4 part of its block,
// the staged splats that can reach the part, and its four parts walk their
// lists side by side. For the Pluecker
// direction d and moment m of its pixel ray in splat space, rho^2 =
// |m|^2/|d|^2 (Eq. rho-pluecker), alpha = min(alpha_max, o exp(-rho^2/2)),
// and for fragments with alpha >= tau_K the view depth of the
// maximum-density point z = (M T [(d x m)/|d|^2; 1])_z (Sec. 3.3); since d
// and m are affine in the pixel offset, |d|^2, |m|^2 and R3 . (d x m) are
// quadratics in it, staged per (tile, splat) and evaluated per pixel. The
// fragments enter a register core of K (depth, list position) keys kept
// sorted by minima and maxima of doubles. Every fragment is
// added to running sums (sum alpha, sum alpha rgb, prod (1 - alpha)); at
// the end the core members are taken back out of them, which leaves the
// order-independent tail of everything that never entered the core or fell
// off its end. The composite is Eq. pixel_color_computation.
//
// Backward: one workgroup per tile. First each pixel's adjoint factors are
// built in LDS: the core terms T_i (c_i - B_i) . G and T_i by walking the
// stored core back to front, and the tail factors shared by every tail
// fragment of the pixel (Sec. 3.3, last paragraph). Then each wave takes 64
// of the tile's instances, one per lane, and loops over the tile's pixels
// (skipping 8x8 blocks no lane's rect touches), recomputing rho^2 and alpha
// (from the forward's staged forms in its operation order: the same bits, so
// exactly the fragments that the forward blended). Because d
// and m are affine in the pixel offset (lx, ly), the gradient w.r.t. their
// 18 affine coefficients follows
// from six moments of dL/d(rho^2)-weights per vector (sum of w, w lx, w ly,
// w lx^2, w lx ly, w ly^2), accumulated in registers. Each lane writes one
// partial per instance (the moments about the pixel at the centre of the
// Gaussian's tile rect, opacity and colour terms): no floating-point
// atomics, deterministic results.
//
// Launch times in the comments are HIP events around the launch over frames
// rendered one after another into kept buffers, once the clocks are steady.
// (The first few dozen steps after an idle time run 7% slower: a benchmark run
// of 20 steps after 5 gives 411 and 520 us for the 1080p launches, one of 200
// after 50 gives 382 and 491. Kernel tracing adds another 10%.)
#include <float.h>

#include <type_traits>

#include "common.h"

namespace htgs {

typedef float float4v __attribute__((ext_vector_type(4)));   // one 16-byte LDS read
typedef float float2v __attribute__((ext_vector_type(2)));
// two 16-bit list entries in one read (the compiler may not move it past the
// entries' stores)
typedef uint32_t __attribute__((may_alias)) list_pair;
typedef __attribute__((address_space(3))) const char *lds_bytes;   // a 32-bit LDS address
typedef __attribute__((address_space(3))) const float2v *lds_float2;
typedef __attribute__((address_space(3))) const float4v *lds_float4;

constexpr float kNegHalfLog2e = -0.72134752044448170368f;  // -1 / (2 ln 2)

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }

// Forward staging. The forward needs, per pixel ray, only |d|^2 and |m|^2
// (the cutoff test and alpha) and R3 . (d x m) (the depth of the maximum
// point). With d and m affine in the pixel offset (X, Y) from the tile
// centre (|X|, |Y| <= (tile size - 1) / 2), |d|^2 and R3 . (d x m) are
// quadratics in (X, Y) whose coefficients (1, X, Y, X^2, XY, Y^2) are
// formed per (tile, splat); a pixel evaluates each with five FMAs. |m|^2
// vanishes at the splat's centre, where its expanded quadratic would lose
// precision to cancellation, so it is staged as a sum of squares instead:
// with an orthonormal basis (q1, q2) of a plane holding Mu and Mv (q1
// along Mu), m = s1 q1 + s2 q2 + r with s1 = R11 X + R12 Y + k1,
// s2 = R22 Y + k2 and r constant and orthogonal to both, so
// |m|^2 = s1^2 + s2^2 + |r|^2 (five FMAs, cancellation only inside s1, s2,
// as in the vector form).
enum FwdStage {
  F_QD = 0,           // |d|^2
  F_QM = 6,           // |m|^2: |r|^2, R11, R12, k1, R22, k2
  F_RC = 12, F_O = 13, F_R = 14, F_G = 15, F_B = 16, F_MUZ = 17,
  F_QZ45 = 18, F_QZ = 20,   // R3 . (d x m): its last two coefficients, its first four
  F_FLOATS = 24, F_TEST4 = 4   // float4s read for the cutoff test and alpha
};

__device__ __forceinline__ void cross_f(const float a[3], const float b[3], float c[3]) {
  c[0] = fmaf(a[1], b[2], -a[2] * b[1]);
  c[1] = fmaf(a[2], b[0], -a[0] * b[2]);
  c[2] = fmaf(a[0], b[1], -a[1] * b[0]);
}

__device__ __forceinline__ float dot_f(const float a[3], const float b[3]) {
  return fmaf(a[2], b[2], fmaf(a[1], b[1], a[0] * b[0]));
}

// R3 . (a x b + e x f)
__device__ __forceinline__ float triple2(const float r[3], const float a[3], const float b[3],
                                         const float e[3], const float f[3]) {
  float c[3], g[3];
  cross_f(a, b, c);
  cross_f(e, f, g);
  return fmaf(r[2], c[2] + g[2], fmaf(r[1], c[1] + g[1], r[0] * (c[0] + g[0])));
}

// (cx2, cy2): twice the tile centre in pixel-index units (an integer).
__device__ __forceinline__ void stage_fwd(const float *__restrict__ rec, int cx2, int cy2,
                                          float *q) {
  const float dx = 0.5f * (float)(cx2 - 2 * __float_as_int(rec[R_IX]));
  const float dy = 0.5f * (float)(cy2 - 2 * __float_as_int(rec[R_IY]));
  float D0[3], Du[3], Dv[3], M0[3], Mu[3], Mv[3], R3[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Du[k] = rec[R_DU + k]; Dv[k] = rec[R_DV + k];
    Mu[k] = rec[R_MU + k]; Mv[k] = rec[R_MV + k];
    D0[k] = fmaf(dy, Dv[k], fmaf(dx, Du[k], rec[R_D0 + k]));
    M0[k] = fmaf(dy, Mv[k], fmaf(dx, Mu[k], rec[R_M0 + k]));
    R3[k] = rec[R_R3 + k];
  }
  q[F_QD + 0] = dot_f(D0, D0);
  q[F_QD + 1] = 2.f * dot_f(D0, Du);
  q[F_QD + 2] = 2.f * dot_f(D0, Dv);
  q[F_QD + 3] = dot_f(Du, Du);
  q[F_QD + 4] = 2.f * dot_f(Du, Dv);
  q[F_QD + 5] = dot_f(Dv, Dv);
  {
    // Gram-Schmidt (q1 along Mu; other unit vectors where Mu, or the part of
    // Mv orthogonal to it, vanishes). Float rounding of the basis only
    // perturbs |m|^2 relatively, by ~1e-7.
    float q1[3], q2[3];
    const float na2 = dot_f(Mu, Mu), nb2 = dot_f(Mv, Mv);
    if (na2 > 0.f) {
      const float s = __builtin_amdgcn_rsqf(na2);
      for (int k = 0; k < 3; ++k) q1[k] = Mu[k] * s;
    } else if (nb2 > 0.f) {
      const float s = __builtin_amdgcn_rsqf(nb2);
      for (int k = 0; k < 3; ++k) q1[k] = Mv[k] * s;
    } else {
      q1[0] = 1.f; q1[1] = 0.f; q1[2] = 0.f;
    }
    const float r12 = dot_f(q1, Mv);
    float v[3];
    for (int k = 0; k < 3; ++k) v[k] = fmaf(-r12, q1[k], Mv[k]);
    const float nv2 = dot_f(v, v);
    if (nv2 > 1e-12f * nb2 && nv2 > 0.f) {
      const float s = __builtin_amdgcn_rsqf(nv2);
      for (int k = 0; k < 3; ++k) q2[k] = v[k] * s;
    } else {
      // q1 x (the axis q1 is least along), normalised
      const float a0 = fabsf(q1[0]), a1 = fabsf(q1[1]), a2 = fabsf(q1[2]);
      float e[3] = {0.f, 0.f, 0.f};
      e[(a0 <= a1 && a0 <= a2) ? 0 : (a1 <= a2 ? 1 : 2)] = 1.f;
      cross_f(q1, e, q2);
      const float s = __builtin_amdgcn_rsqf(dot_f(q2, q2));
      for (int k = 0; k < 3; ++k) q2[k] *= s;
    }
    const float k1 = dot_f(q1, M0), k2 = dot_f(q2, M0);
    float r[3];
    for (int k = 0; k < 3; ++k) r[k] = fmaf(-k2, q2[k], fmaf(-k1, q1[k], M0[k]));
    q[F_QM + 0] = dot_f(r, r);
    q[F_QM + 1] = dot_f(q1, Mu);
    q[F_QM + 2] = r12;
    q[F_QM + 3] = k1;
    q[F_QM + 4] = dot_f(q2, Mv);
    q[F_QM + 5] = k2;
  }
  // d x m = D0xM0 + X (D0xMu + DuxM0) + Y (D0xMv + DvxM0) + X^2 DuxMu
  //         + XY (DuxMv + DvxMu) + Y^2 DvxMv
  float c[3];
  cross_f(D0, M0, c);
  q[F_QZ + 0] = dot_f(R3, c);
  q[F_QZ + 1] = triple2(R3, D0, Mu, Du, M0);
  q[F_QZ + 2] = triple2(R3, D0, Mv, Dv, M0);
  cross_f(Du, Mu, c);
  q[F_QZ + 3] = dot_f(R3, c);
  q[F_QZ45 + 0] = triple2(R3, Du, Mv, Dv, Mu);
  cross_f(Dv, Mv, c);
  q[F_QZ45 + 1] = dot_f(R3, c);
  q[F_RC] = rec[R_RC];
  q[F_O] = rec[R_O];
  q[F_MUZ] = rec[R_MUZ];
  q[F_R] = rec[R_RGB];
  q[F_G] = rec[R_RGB + 1];
  q[F_B] = rec[R_RGB + 2];
}

// Per-pixel constants of the quadratics: X, Y, X^2, XY, Y^2.
struct PixQ {
  float x, y, xx, xy, yy;
};

__device__ __forceinline__ float eval_q(const float *c, const PixQ &u) {
  return fmaf(u.yy, c[5], fmaf(u.xy, c[4], fmaf(u.xx, c[3], fmaf(u.y, c[2], fmaf(u.x, c[1], c[0])))));
}

// |d|^2 from its staged quadratic, the Y terms first (a pixel row shares
// them) and then the X terms: c0 + Y c2 + Y^2 c5 + X^2 c3 + X (c1 + Y c4).
// The backward evaluates it in the same order, row part once per row, so
// both passes get the same bits.
__device__ __forceinline__ float eval_dd(const float *c, const PixQ &u) {
  return fmaf(u.x, fmaf(u.y, c[4], c[1]), fmaf(u.xx, c[3], fmaf(u.yy, c[5], fmaf(u.y, c[2], c[0]))));
}

// |m|^2 = s1^2 + s2^2 + |r|^2 (see FwdStage).
__device__ __forceinline__ float eval_mm(const float *c, const PixQ &u) {
  const float s1 = fmaf(c[1], u.x, fmaf(c[2], u.y, c[3]));
  const float s2 = fmaf(c[4], u.y, c[5]);
  return fmaf(s1, s1, fmaf(s2, s2, c[0]));
}

// alpha = min(alpha_max, o exp(-rho^2 / 2)) with rho^2 = mm / dd (a median
// with 0: fminf canonicalizes its operands first).
__device__ __forceinline__ float frag_alpha(float o, float mm, float inv, float amax) {
  return __builtin_amdgcn_fmed3f(o * exp2_fast((mm * inv) * kNegHalfLog2e), 0.f, amax);
}

__device__ __forceinline__ bool is_fragment(float dd, float mm, float rc) {
  return (dd >= FLT_MIN) && (mm <= rc * dd);
}


__device__ __forceinline__ void load_record(const float *__restrict__ recs, uint32_t gid, float *rec) {
  const float4 *r4 = reinterpret_cast<const float4 *>(recs + (int64_t)gid * kRecFloats);
#pragma unroll
  for (int k = 0; k < kRecFloats / 4; ++k) {
    const float4 t = r4[k];
    rec[4 * k] = t.x; rec[4 * k + 1] = t.y; rec[4 * k + 2] = t.z; rec[4 * k + 3] = t.w;
  }
}

// The forward's state is written once and read once, in another launch, and
// it is larger than the caches: non-temporal, so that it does not push the
// records out of them (1080p, K = 8, 0.45 GB: backward 514 -> 498 us, forward
// 392 -> 387).
__device__ __forceinline__ void put_state(float *sp, int64_t i, float x) {
  __builtin_nontemporal_store(x, sp + i);
}
__device__ __forceinline__ float get_state(const float *sp, int64_t i) {
  return __builtin_nontemporal_load(sp + i);
}

struct TileInfo {
  int t, v, tx, ty;
};

// Float offset of a tile's forward state (tile-major layout: nval values
// of nt pixels per tile, tiles row-major inside their view).
__device__ __forceinline__ int64_t tile_state_off(const ViewParams &V, const TileInfo &ti,
                                                  int nval, int nt) {
  return V.state_off + ((int64_t)ti.ty * V.tiles_x + ti.tx) * nval * nt;
}

// The workgroup's tile; false past the last one. (The hardware hands the next
// workgroup to the first CU with room. Resident workgroups that took tiles
// from an atomic counter instead waited for it, 13 ns per tile however many
// asked: 582 against 425 us for the 1080p forward's 32,400 tiles, 996 against
// 734 us for the 70,752 of an 8-view batch.)
__device__ __forceinline__ bool tile_info(const ViewSet &vs, const KCfg &cfg, const Ws &w,
                                          TileInfo &ti) {
  const int slot = xcd_slot((int)blockIdx.x, cfg.xcd_shift);
  if (slot >= vs.total_tiles) return false;
  ti.t = cfg.cost_order ? (int)w.order[slot] : slot;
  ti.v = view_of_tile(vs, ti.t);
  const int lt = ti.t - vs.v[ti.v].tile_base;
  ti.tx = lt % vs.v[ti.v].tiles_x;
  ti.ty = lt / vs.v[ti.v].tiles_x;
  return true;
}

__device__ __forceinline__ bool rect_meets_block(const float *bb, int bx, int by) {
  return (__float_as_int(bb[2]) >= bx) && (__float_as_int(bb[0]) <= bx + 7) &&
         (__float_as_int(bb[3]) >= by) && (__float_as_int(bb[1]) <= by + 7);
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
// A wave owns an 8x8 pixel block, one lane per pixel, cut into kParts parts
// of 4 columns and kPartRows rows, 64 / kParts consecutive lanes each. Every
// part walks a list of its own, of the staged splats that can reach it, so a
// step of the wave handles up to kParts different splats. The walk is bound
// by VALU issue, and a step costs the same whatever share of its lanes hold
// a fragment: with one list per block 64% of the lanes of the 1080p frame
// (1M Gaussians, K = 8, 8x8 tiles, 205 splats per tile), with four lists 69%
// in 0.71 times the steps. Eight lists of 4x2 pixels shorten them further,
// but their rows' reads meet in the LDS banks and their lists cost more to
// build: 444 us against 419 for the launch at 1080p, 7.05 ms against 6.98 on
// a 3840x2160 frame of 6M Gaussians.
constexpr int kParts = 4;
constexpr int kPartRows = 16 / kParts;
constexpr int kPartLanes = 64 / kParts;
__device__ __forceinline__ int part_x(int lane) {
  return (lane & 3) | ((lane / kPartLanes) & 1) * 4;
}
__device__ __forceinline__ int part_y(int lane) {
  return ((lane % kPartLanes) >> 2) + (lane / (2 * kPartLanes)) * kPartRows;
}

// Parts of a TW x TH tile that a staged splat can reach: bit kParts b + p for
// part p of 8x8 block b. A pixel row of a part is missed when the smallest
// |m|^2 over its columns (X taken as continuous between the first and the
// last) exceeds rho_c times the largest |d|^2 over the tile (a bound from the
// coefficients' magnitudes; |d|^2 hardly changes over a tile). The slack
// (2e-6 of the terms of s1 and s2, 1e-4 of the bound) is far above the
// rounding of the per-pixel test, so no part with a fragment is left out.
template <int TW, int TH>
__device__ __forceinline__ uint32_t part_mask(const float *q) {
  constexpr int QX = TW / 4, QY = TH / kPartRows, BX = TW / 8, BY = 8 / kPartRows;
  const float hx = 0.5f * (float)(TW - 1), hy = 0.5f * (float)(TH - 1);
  const float *d = q + F_QD, *m = q + F_QM;
  const float ddmax = fmaf(hx, fabsf(d[1]), fmaf(hy, fabsf(d[2]), fmaf(hx * hy, fabsf(d[4]),
                      fmaf(hx * hx, d[3], fmaf(hy * hy, d[5], d[0])))));
  const float lim = fmaf(q[F_RC] * ddmax, 1.0001f, -m[0]);
  const float ax = fabsf(m[1]);
  const float h = fmaf(1.5f, ax, 2e-6f * fmaf(hx, ax, fmaf(hy, fabsf(m[2]), fabsf(m[3]))));
  const float e2 = 2e-6f * fmaf(hy, fabsf(m[4]), fabsf(m[5]));
  uint32_t mask = 0u;
#pragma unroll
  for (int qy = 0; qy < QY; ++qy) {
    float best[QX];   // smallest s1^2 + s2^2 - lim over the part's rows
#pragma unroll
    for (int r = 0; r < kPartRows; ++r) {
      const float y = (float)(kPartRows * qy + r) - hy;
      const float s2 = fmaxf(fabsf(fmaf(m[4], y, m[5])) - e2, 0.f);
      const float a = fmaf(m[2], y, m[3]);
      const float c = fmaf(s2, s2, -lim);
#pragma unroll
      for (int qx = 0; qx < QX; ++qx) {
        const float s1 = fmaxf(fabsf(fmaf(m[1], (float)(4 * qx) + 1.5f - hx, a)) - h, 0.f);
        const float v = fmaf(s1, s1, c);
        best[qx] = r == 0 ? v : fminf(best[qx], v);
      }
    }
#pragma unroll
    for (int qx = 0; qx < QX; ++qx) {
      const int bit = kParts * ((qy / BY) * BX + (qx >> 1)) + 2 * (qy % BY) + (qx & 1);
      if (!(best[qx] > 0.f)) mask |= 1u << bit;   // (kept where a form is not finite)
    }
  }
  return mask;
}

// Blocks of the tile whose pixels meet the covered pixel rect (b0, b1: the
// record's packed corners), kParts bits each. One-block tiles take them all.
template <int TW, int TH>
__device__ __forceinline__ uint32_t rect_block_mask(uint32_t b0, uint32_t b1, int px0, int py0) {
  constexpr uint32_t kAll = (1u << kParts) - 1u;
  if constexpr (TW * TH == 64) return kAll;
  uint32_t mask = 0u;
  const int x0 = (int)(b0 & 0xffffu) - px0, y0 = (int)(b0 >> 16) - py0;
  const int x1 = (int)(b1 & 0xffffu) - px0, y1 = (int)(b1 >> 16) - py0;
#pragma unroll
  for (int b = 0; b < TW * TH / 64; ++b) {
    const int bx = (b % (TW / 8)) * 8, by = (b / (TW / 8)) * 8;
    if (x1 >= bx && x0 <= bx + 7 && y1 >= by && y0 <= by + 7) mask |= kAll << (kParts * b);
  }
  return mask;
}

// A batch of staged splats in LDS and the parts' lists of them (byte offsets
// of the rows).
constexpr int kStageBytes = F_FLOATS * 4;
template <int TW, int TH, int NBATCH>
struct FwdLds {
  static constexpr int kWaves = TW * TH / 64;
  // one row per splat; the last row is all zeros (|d|^2 = 0: no fragment)
  float4 stage[(NBATCH + 1) * (F_FLOATS / 4)];
  union {
    uint16_t list[kWaves][kParts][NBATCH];
    uint2 fill[kWaves][kParts * NBATCH / 4];
  };
  uint32_t mask[kWaves > 1 ? NBATCH : 1];
  uint32_t reach[kWaves > 1 ? NBATCH : 1];
};

// A staged row in registers (opaque: otherwise each component is read by
// itself where it is used).
struct StagedRow {
  float4v q[F_FLOATS / 4];
};
__device__ __forceinline__ StagedRow read_row(const char *p) {
  StagedRow row;
#pragma unroll
  for (int k = 0; k < F_FLOATS / 4; ++k) {
    row.q[k] = *reinterpret_cast<const float4v *>(p + 16 * k);
    asm("" : "+v"(row.q[k]));
  }
  return row;
}

// What a wave knows about the staged batch as a whole.
struct BatchInfo {
  int nlist;     // length of its longest list, rounded up to an even number
  float reach;   // no fragment lies further in front of its splat's mean
};

// Largest of the wave's values. All 64 lanes.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#define HTGS_MAX_DPP(CTRL) \
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true))
  HTGS_MAX_DPP(0x111);   // row_shr:1, 2, 4, 8
  HTGS_MAX_DPP(0x112);
  HTGS_MAX_DPP(0x114);
  HTGS_MAX_DPP(0x118);
  HTGS_MAX_DPP(0x142);   // row_bcast:15, 31
  HTGS_MAX_DPP(0x143);
#undef HTGS_MAX_DPP
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// How far in front of its splat's mean a fragment's depth can lie (bits of a
// float that is not negative, or of a NaN): z = muz + R3 . (d x m) / |d|^2
// with |m| <= sqrt(rho_c) |d|, so |R3| sqrt(rho_c), and a quarter more, with
// 2^-20 of the depth, for the rounding of z.
__device__ __forceinline__ uint32_t depth_reach(const float *rec) {
  const float r2 = dot_f(rec + R_R3, rec + R_R3);
  return __float_as_uint(
      fmaf(1.25f, __builtin_amdgcn_sqrtf(r2 * rec[R_RC]), 9.6e-7f * fabsf(rec[R_MUZ]))) &
         0x7fffffffu;
}

// Stages one splat; returns the parts it can reach.
template <int TW, int TH, int NBATCH>
__device__ __forceinline__ uint32_t stage_splat(FwdLds<TW, TH, NBATCH> &L, int r,
                                                const float *__restrict__ recs, uint32_t gid,
                                                int px0, int py0, uint32_t *reach) {
  float rec[kRecFloats];
  load_record(recs, gid, rec);
  float st[F_FLOATS];
  stage_fwd(rec, 2 * px0 + TW - 1, 2 * py0 + TH - 1, st);
#pragma unroll
  for (int k = 0; k < F_FLOATS / 4; ++k)
    L.stage[r * (F_FLOATS / 4) + k] =
        make_float4(st[4 * k], st[4 * k + 1], st[4 * k + 2], st[4 * k + 3]);
  *reach = depth_reach(rec);
  return part_mask<TW, TH>(st) &
         rect_block_mask<TW, TH>(__float_as_uint(rec[R_BB0]), __float_as_uint(rec[R_BB1]), px0, py0);
}

// Adds the staged splat j of each lane (part bits m of this wave's block; 0
// past the batch) to the wave's lists; n: the lists' lengths. Called by all
// 64 lanes.
template <int NBATCH>
__device__ __forceinline__ void extend_lists(uint16_t (*list)[NBATCH], int j, uint32_t m, int *n) {
#pragma unroll
  for (int p = 0; p < kParts; ++p) {
    const bool hit = (m & (1u << p)) != 0u;
    const uint64_t mk = __ballot(hit);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, (uint32_t)n[p]));
    if (hit) list[p][at] = (uint16_t)(j * kStageBytes);
    n[p] += __popcll(mk);
  }
}

// The thread's splats of the batch from `base` on (0 past the list's end).
// They are read a batch ahead, while the batch before is walked, so that the
// records wait for one round trip and not for two: 6.28 -> 6.11 ms for the
// 4K frame's launch, 393 -> 388 us at 1080p. (A load that brings the records
// themselves nearer costs more than it hides: 411 us.)
template <int NT, int BM>
__device__ __forceinline__ void next_splats(const uint32_t *__restrict__ vals, uint32_t base,
                                            uint32_t end, int tid, uint32_t *gid) {
#pragma unroll
  for (int i = 0; i < BM; ++i) {
    const uint32_t j = base + (uint32_t)(i * NT + tid);
    gid[i] = j < end ? vals[j] : 0u;
  }
}

// Stages the batch's cnt splats (gid: this thread's, next_splats) and builds
// this wave's lists (padded with the zero row to the longest one's even
// length). All threads of the workgroup.
template <int TW, int TH, int NBATCH>
__device__ __forceinline__ BatchInfo stage_batch(FwdLds<TW, TH, NBATCH> &L,
                                                 const float *__restrict__ recs,
                                                 const uint32_t *gid, int cnt, int px0, int py0,
                                                 int wave, int lane) {
  constexpr int NT = TW * TH;
  int n[kParts];
  uint32_t reach = 0u;
#pragma unroll
  for (int p = 0; p < kParts; ++p) n[p] = 0;
  constexpr uint32_t kZeroRow = (uint32_t)(NBATCH * kStageBytes);
  constexpr uint32_t kZero2 = kZeroRow | (kZeroRow << 16);
  static_assert(kZeroRow < 65536u, "row offsets are 16 bits");
#pragma unroll
  for (int i = 0; i < kParts * NBATCH / 4; i += 64)
    if (i + lane < kParts * NBATCH / 4) L.fill[wave][i + lane] = make_uint2(kZero2, kZero2);
  __builtin_amdgcn_wave_barrier();
  if constexpr (NT == 64) {
#pragma unroll
    for (int r0 = 0; r0 < NBATCH; r0 += 64) {
      const int r = r0 + lane;
      uint32_t m = 0u, e = 0u;
      if (r < cnt) m = stage_splat(L, r, recs, gid[r0 / 64], px0, py0, &e);
      reach = max(reach, e);
      extend_lists<NBATCH>(L.list[0], r, m, n);
    }
    __syncthreads();
  } else {
    static_assert(NBATCH == NT, "one record per thread");
    const int r = wave * 64 + lane;
    if (r < cnt) {
      uint32_t e;
      L.mask[r] = stage_splat(L, r, recs, gid[0], px0, py0, &e);
      L.reach[r] = e;
    }
    __syncthreads();
    for (int j0 = 0; j0 < cnt; j0 += 64) {
      const int j = j0 + lane;
      const uint32_t m = j < cnt ? L.mask[j] >> (kParts * wave) : 0u;
      reach = max(reach, j < cnt ? L.reach[j] : 0u);
      extend_lists<NBATCH>(L.list[wave], j, m, n);
    }
    __builtin_amdgcn_wave_barrier();
  }
  int longest = 0;
#pragma unroll
  for (int p = 0; p < kParts; ++p) longest = max(longest, n[p]);
  return {(longest + 1) & ~1, __uint_as_float(wave_max(reach))};
}

// Core keys: depth in the high word, list position and alpha slot in the
// low word, as a double. Depths are below infinity (as float32 bits never a
// NaN of the double), so doubles compare like (depth, position), and one
// minimum and one maximum per entry insert a fragment. Of negative doubles the
// larger low word is the smaller number: behind the camera (a negative z_near
// lets such splats through) the position's bits are inverted.
__device__ __forceinline__ double core_key(uint32_t hi, uint32_t lo) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t key_hi(double k) {
  return (uint32_t)((unsigned long long)__double_as_longlong(k) >> 32);
}
__device__ __forceinline__ uint32_t key_lo(double k) {
  return (uint32_t)(unsigned long long)__double_as_longlong(k);
}
// The list position of a key with SB slot bits (BEHIND: inverted where the
// depth is negative).
template <int SB, bool BEHIND>
__device__ __forceinline__ uint32_t key_pos(double k) {
  if constexpr (!BEHIND) return key_lo(k) >> SB;
  return (key_lo(k) ^ (uint32_t)((int32_t)key_hi(k) >> 31)) >> SB;
}
// (fmin and fmax would canonicalize their operands first)
__device__ __forceinline__ double key_min(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double key_max(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Inserts x into the sorted keys; the last one drops out. (Four minima ahead
// of their maxima: no instruction waits for the one before it.)
template <int KMAX>
__device__ __forceinline__ void core_insert(double *key, double x) {
#pragma unroll
  for (int g = KMAX - 1; g >= 1; g -= 4) {
    double m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (g - i >= 1) m[i] = key_min(key[g - i], x);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (g - i >= 1) key[g - i] = key_max(key[g - i - 1], m[i]);
  }
  key[0] = key_min(key[0], x);
}

constexpr int log2_of(int x) { return x <= 1 ? 0 : 1 + log2_of(x / 2); }

// The wave's fragments to the forward's counter. All 64 lanes.
__device__ __forceinline__ void add_fragments(const Ws &w, uint32_t n, int lane) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off, 64);
  if (lane == 0 && n) count_add(w.frags, (unsigned long long)n);
}

// One tile. EXACT: K == KMAX, known at compile time. BEHIND: a view has a
// negative z_near, so that equal negative depths can meet (a test per insertion
// instead took 1 to 4% of the launch). Bound by VALU issue: an instruction per
// 3.5 cycles and SIMD at 1080p with K = 8 and per 3.8 on the 4K frame with K =
// 16, where float32 arithmetic takes 2.7 cycles and compares, selects, integer
// and float64 operations 4.4 (about 36 instructions per step of the walk, 36
// more where a lane inserts, 375 per staged batch), with 4.5 waves per SIMD,
// which LDS sets. 1080p, K = 8, 8x8 tiles: 525 us when each block walked one list
// and shifted its core by compares and selects, 384 now; 4K frame 8.30 -> 6.10
// ms, 8 views 1180 -> 687 us.
template <int KMAX, int TW, int TH, int BM, bool EXACT, bool BEHIND>
__device__ __forceinline__ void fwd_tile(const TileInfo &ti, const Ws &w, const ViewSet &vs,
                                         const KCfg &cfg, float *__restrict__ state,
                                         const uint32_t *__restrict__ vals) {
  constexpr int NT = TW * TH;
  constexpr int NBATCH = NT * BM;   // records staged per batch
  constexpr int NW = NT / 64;       // waves, one 8x8 block each
  constexpr int BX = TW / 8;
  __shared__ FwdLds<TW, TH, NBATCH> L;
  __shared__ float s_alpha[NW][KMAX][64];   // alphas of the core, by slot and lane

  const ViewParams &V = vs.v[ti.v];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lx = (wave % BX) * 8 + part_x(lane), ly = (wave / BX) * 8 + part_y(lane);
  const int px0 = ti.tx * TW, py0 = ti.ty * TH;
  const int px = px0 + lx, py = py0 + ly;
  const bool inside = (px < V.width) && (py < V.height);
  // a failed front end (overflow) leaves every
  // tile empty: background, and no list or record is read
  uint2 rg = front_failed(w) ? make_uint2(0u, 0u) : w.ranges[ti.t];
  rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
  rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
  PixQ u;
  u.x = (float)lx - 0.5f * (float)(TW - 1);
  u.y = (float)ly - 0.5f * (float)(TH - 1);
  u.xx = u.x * u.x; u.xy = u.x * u.y; u.yy = u.y * u.y;   // exact (half-integers)
  const int K = EXACT ? KMAX : cfg.K;
  // (K = 0: no alpha reaches the core)
  const float tau_core = K > 0 ? cfg.tau_core : 2.f, amax = cfg.alpha_max;
  const int no_tail = cfg.no_tail;
  const float *recs = w.records + (int64_t)ti.v * cfg.n * kRecFloats;

  // Core: the KMAX front-most fragments with alpha >= tau_K, sorted by
  // (depth, list position); with K < KMAX the first K are used. An entry's
  // alpha lies in LDS, in the slot its key names; a new entry takes the slot
  // of the one that drops out. Every fragment is added to the running sums
  // (alpha, alpha rgb, prod 1 - alpha); once the list is done the core
  // members are taken back out of them with the same alphas, which leaves
  // exactly the tail sums. Keys as doubles take 15 instructions per
  // insertion for K = 8; depth, position and alpha shifted by compares and
  // selects took 48.
  constexpr int SB = log2_of(KMAX);   // slot bits; list positions are below 2^27
  double key[KMAX];
#pragma unroll
  for (int i = 0; i < KMAX; ++i) key[i] = core_key(0x7f800000u, (uint32_t)i);
  float A = 0.f, S0 = 0.f, S1 = 0.f, S2 = 0.f, P = 1.f;
  uint32_t nfrag = 0;
  float *my_alpha = &s_alpha[wave][0][lane];
  if (tid < F_FLOATS / 4) L.stage[NBATCH * (F_FLOATS / 4) + tid] = make_float4(0.f, 0.f, 0.f, 0.f);

  uint32_t gid[BM];
  next_splats<NT, BM>(vals, rg.x, rg.y, tid, gid);
  for (uint32_t base = rg.x; base < rg.y; base += NBATCH) {
    const int cnt = (int)min((uint32_t)NBATCH, rg.y - base);
    __syncthreads();
    const BatchInfo batch = stage_batch(L, recs, gid, cnt, px0, py0, wave, lane);
    next_splats<NT, BM>(vals, base + NBATCH, rg.y, tid, gid);
    if (!inside) continue;
    // A splat whose mean lies at this depth or further back has no fragment
    // in front of the last core entry, and its depth is not evaluated (two
    // thirds of the steps of a wave with 786 splats per tile and K = 16, half
    // of them with 205 and K = 8: 7.01 -> 6.70 ms and 425 -> 411 us).
    float far = __uint_as_float(key_hi(key[KMAX - 1])) + batch.reach;
    const char *rows = reinterpret_cast<const char *>(L.stage);
    auto step = [&](uint32_t off, const StagedRow &row) {
      float e[12];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float4v t = row.q[k];
        e[4 * k] = t.x; e[4 * k + 1] = t.y; e[4 * k + 2] = t.z; e[4 * k + 3] = t.w;
      }
      const float4v f3 = row.q[F_RC / 4];   // rho_c, o, r, g
      const float4v f4 = row.q[F_B / 4];    // b, muz, qz4, qz5
      const float dd = eval_dd(e + F_QD, u);
      const float mm = eval_mm(e + F_QM, u);
      if (!is_fragment(dd, mm, f3.x)) return;
      ++nfrag;
      const float inv = rcp_fast(dd);
      const float alpha = frag_alpha(f3.y, mm, inv, amax);
      int nt = no_tail;
      asm volatile("" : "+s"(nt));   // (a scalar test here, not a saved lane mask)
      if (nt == 0) {
        A += alpha;
        S0 = fmaf(alpha, f3.z, S0);
        S1 = fmaf(alpha, f3.w, S1);
        S2 = fmaf(alpha, f4.x, S2);
        P *= 1.f - alpha;
      }
      // (also where a reach is not finite)
      if (!(f4.y >= far) && alpha >= tau_core) {
        const float4v f5 = row.q[F_QZ / 4];   // qz0..qz3
        const float qz[6] = {f5.x, f5.y, f5.z, f5.w, f4.z, f4.w};
        const float z = fmaf(eval_q(qz, u), inv, f4.y);
        if (z < __uint_as_float(key_hi(key[KMAX - 1]))) {
          const uint32_t slot = key_lo(key[KMAX - 1]) & (uint32_t)(KMAX - 1);
          // row / kStageBytes for whole rows
          uint32_t pos = (base - rg.x) + ((off * 683u) >> 16);
          my_alpha[slot * 64u] = alpha;
          if constexpr (BEHIND) pos ^= (uint32_t)(__float_as_int(z) >> 31);
          core_insert<KMAX>(key, core_key(__float_as_uint(z), (pos << SB) | slot));
          far = __uint_as_float(key_hi(key[KMAX - 1])) + batch.reach;
        }
      }
    };
    // Two splats per round, both rows read whole before the first is used (a
    // read where its values are needed leaves the wave waiting up to six
    // times per round: 411 against 395 us for the launch at 1080p with K = 8);
    // the next round's rows are looked up meanwhile (the last look-up lies
    // past the list, inside L, and is not used).
    const list_pair *list = reinterpret_cast<const list_pair *>(L.list[wave][lane / kPartLanes]);
    uint32_t next = list[0];
    for (int q = 0; q < batch.nlist; q += 2) {
      const uint32_t o = next;
      next = list[q / 2 + 1];
      const StagedRow r0 = read_row(rows + (o & 0xffffu)), r1 = read_row(rows + (o >> 16));
      step(o & 0xffffu, r0);
      step(o >> 16, r1);
    }
  }
  static_assert(kStageBytes == 96 && NBATCH <= 256, "row numbers from byte offsets");
  add_fragments(w, nfrag, lane);
  if (!inside) return;

  // Composite (Eq. pixel_color_computation): the core front to back, then
  // the tail behind it.
  float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
  float Ac = 0.f, Sc0 = 0.f, Sc1 = 0.f, Sc2 = 0.f;
  uint32_t ncore = 0;
  // tile-major state: this tile's values, value by value, each over the
  // tile's 8x8 blocks (this wave's block is block number `wave`)
  const int blk_pix = part_y(lane) * 8 + part_x(lane);
  float *sp = state ? state + tile_state_off(V, ti, state_values(K), NT) + wave * 64 + blk_pix
                    : nullptr;
  // One core member: composite, take it out of the sums, store it.
  auto core_entry = [&](int i, int gid, int pos, float a, float r, float g, float b) {
    if (gid >= 0) {
      const float wgt = a * T;
      C0 = fmaf(wgt, r, C0);
      C1 = fmaf(wgt, g, C1);
      C2 = fmaf(wgt, b, C2);
      T *= 1.f - a;
      Ac += a;
      Sc0 = fmaf(a, r, Sc0);
      Sc1 = fmaf(a, g, Sc1);
      Sc2 = fmaf(a, b, Sc2);
      ++ncore;
    }
    if (sp) {
      put_state(sp, (int64_t)i * NT, __int_as_float(gid));
      put_state(sp, (int64_t)(K + i) * NT, a);
      put_state(sp, (int64_t)(2 * K + i) * NT, __int_as_float(pos));
      put_state(sp, (int64_t)(3 * K + 3 * i) * NT, r);
      put_state(sp, (int64_t)(3 * K + 3 * i + 1) * NT, g);
      put_state(sp, (int64_t)(3 * K + 3 * i + 2) * NT, b);
    }
  };
  // Ids, then colours and alphas, eight entries at a time: the loads of a
  // group are independent of each other.
  constexpr int GR = KMAX < 8 ? KMAX : 8;
#pragma unroll
  for (int i0 = 0; i0 < KMAX; i0 += GR) {
    int gids[GR], pos[GR];
    float4 c[GR];
    float ca[GR];
#pragma unroll
    for (int i = 0; i < GR; ++i) {
      const bool got = i0 + i < K && key_hi(key[i0 + i]) != 0x7f800000u;
      const uint32_t lo = key_lo(key[i0 + i]);
      const uint32_t at = key_pos<SB, BEHIND>(key[i0 + i]);
      pos[i] = got ? (int)at : -1;
      gids[i] = got ? (int)vals[rg.x + at] : -1;
      ca[i] = got ? my_alpha[(lo & (uint32_t)(KMAX - 1)) * 64u] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < GR; ++i) {
      c[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (gids[i] >= 0)
        c[i] = reinterpret_cast<const float4 *>(recs + (int64_t)gids[i] * kRecFloats)[R_RGB / 4];
    }
#pragma unroll
    for (int i = 0; i < GR; ++i)
      if (i0 + i < K) core_entry(i0 + i, gids[i], pos[i], ca[i], c[i].x, c[i].y, c[i].z);
  }
  // Tail sums: everything minus the core; exactly empty when no fragment
  // is left over, or when the tail is left out (inference without the
  // tail, Sec. 4.3: the background lies right behind the core).
  if (no_tail || nfrag == ncore) {
    A = 0.f; S0 = S1 = S2 = 0.f; P = 1.f;
  } else {
    A = fmaxf(A - Ac, 0.f);
    S0 = fmaxf(S0 - Sc0, 0.f);
    S1 = fmaxf(S1 - Sc1, 0.f);
    S2 = fmaxf(S2 - Sc2, 0.f);
    P = T > 0.f ? fminf(P / T, 1.f) : 0.f;
  }
  float X0 = P * cfg.bg[0], X1 = P * cfg.bg[1], X2 = P * cfg.bg[2];
  if (A > 0.f) {
    const float k = (1.f - P) / A;
    X0 = fmaf(k, S0, X0);
    X1 = fmaf(k, S1, X1);
    X2 = fmaf(k, S2, X2);
  }
  const int64_t npix = (int64_t)V.width * V.height;
  const int64_t pix = (int64_t)py * V.width + px;
  V.out_rgb[pix] = fmaf(T, X0, C0);
  V.out_rgb[npix + pix] = fmaf(T, X1, C1);
  V.out_rgb[2 * npix + pix] = fmaf(T, X2, C2);
  if (sp) {
    put_state(sp, (int64_t)(6 * K) * NT, T);
    put_state(sp, (int64_t)(6 * K + 1) * NT, A);
    put_state(sp, (int64_t)(6 * K + 2) * NT, S0);
    put_state(sp, (int64_t)(6 * K + 3) * NT, S1);
    put_state(sp, (int64_t)(6 * K + 4) * NT, S2);
    put_state(sp, (int64_t)(6 * K + 5) * NT, P);
  }
}

// ---------------------------------------------------------------------------
// Forward, sorted blending
// ---------------------------------------------------------------------------
// The paper's "w/o per-pixel HT" configuration (Sec. 4.3, Table splat_eval):
// the per-pixel evaluation of Sec. 3.2 with plain alpha blending (Eq.
// alpha_blending) in the order of the tile's list, which the front end has
// sorted front to back by the view depth of the Gaussians' means. A pixel
// stops before the fragment that would take its transmittance below tau_T
// (the early stop plain alpha blending allows, Sec. 5), and the workgroup
// stops staging batches once every pixel of its tile has stopped.
template <int TW, int TH>
__device__ __forceinline__ void fwd_tile_sorted(const TileInfo &ti, const Ws &w,
                                                const ViewSet &vs, const KCfg &cfg,
                                                float *__restrict__ state,
                                                const uint32_t *__restrict__ vals) {
  constexpr int NT = TW * TH;
  constexpr int BX = TW / 8;
  __shared__ FwdLds<TW, TH, NT> L;

  const ViewParams &V = vs.v[ti.v];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lx = (wave % BX) * 8 + part_x(lane), ly = (wave / BX) * 8 + part_y(lane);
  const int px0 = ti.tx * TW, py0 = ti.ty * TH;
  const int px = px0 + lx, py = py0 + ly;
  const bool inside = (px < V.width) && (py < V.height);
  uint2 rg = front_failed(w) ? make_uint2(0u, 0u) : w.ranges[ti.t];
  rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
  rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
  PixQ u;
  u.x = (float)lx - 0.5f * (float)(TW - 1);
  u.y = (float)ly - 0.5f * (float)(TH - 1);
  u.xx = u.x * u.x; u.xy = u.x * u.y; u.yy = u.y * u.y;
  const float amax = cfg.alpha_max, tau_T = cfg.tau_T;
  const float *recs = w.records + (int64_t)ti.v * cfg.n * kRecFloats;

  float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
  bool done = !inside;
  int nb = 0, end_pos = 0, stop_pos = -1;
  if (tid < F_FLOATS / 4) L.stage[NT * (F_FLOATS / 4) + tid] = make_float4(0.f, 0.f, 0.f, 0.f);

  uint32_t gid[1];
  next_splats<NT, 1>(vals, rg.x, rg.y, tid, gid);
  for (uint32_t base = rg.x; base < rg.y; base += NT) {
    // (also the barrier before the stage is overwritten)
    if (__syncthreads_and(done)) break;
    const int cnt = (int)min((uint32_t)NT, rg.y - base);
    const int nlist = stage_batch(L, recs, gid, cnt, px0, py0, wave, lane).nlist;
    next_splats<NT, 1>(vals, base + NT, rg.y, tid, gid);
    if (done) continue;
    const char *rows = reinterpret_cast<const char *>(L.stage);
    auto step = [&](uint32_t off, const StagedRow &row) {
      float e[4 * F_TEST4];
#pragma unroll
      for (int k = 0; k < F_TEST4; ++k) {
        const float4v t = row.q[k];
        e[4 * k] = t.x; e[4 * k + 1] = t.y; e[4 * k + 2] = t.z; e[4 * k + 3] = t.w;
      }
      const float dd = eval_dd(e + F_QD, u);
      const float mm = eval_mm(e + F_QM, u);
      if (!is_fragment(dd, mm, e[F_RC])) return;
      const float alpha = frag_alpha(e[F_O], mm, rcp_fast(dd), amax);
      const float tn = T * (1.f - alpha);
      const int pos = (int)((base - rg.x) + ((off * 683u) >> 16));
      if (tn < tau_T) {
        done = true;
        stop_pos = pos;
        return;
      }
      const float wgt = alpha * T;
      C0 = fmaf(wgt, e[F_R], C0);
      C1 = fmaf(wgt, e[F_G], C1);
      C2 = fmaf(wgt, row.q[F_B / 4].x, C2);
      T = tn;
      ++nb;
      end_pos = pos + 1;
    };
    const list_pair *list = reinterpret_cast<const list_pair *>(L.list[wave][lane / kPartLanes]);
    for (int q = 0; q < nlist && !done; q += 2) {
      const uint32_t o = list[q / 2];
      const StagedRow r0 = read_row(rows + (o & 0xffffu)), r1 = read_row(rows + (o >> 16));
      step(o & 0xffffu, r0);
      if (!done) step(o >> 16, r1);
    }
  }
  add_fragments(w, (uint32_t)nb, lane);
  if (!inside) return;
  const int64_t npix = (int64_t)V.width * V.height;
  const int64_t pix = (int64_t)py * V.width + px;
  V.out_rgb[pix] = fmaf(T, cfg.bg[0], C0);
  V.out_rgb[npix + pix] = fmaf(T, cfg.bg[1], C1);
  V.out_rgb[2 * npix + pix] = fmaf(T, cfg.bg[2], C2);
  if (state) {
    float *sp = state + tile_state_off(V, ti, kSortedStateValues, NT) + wave * 64 +
                part_y(lane) * 8 + part_x(lane);
    put_state(sp, 0, T);
    put_state(sp, NT, C0);
    put_state(sp, 2 * NT, C1);
    put_state(sp, 3 * NT, C2);
    put_state(sp, 4 * NT, __int_as_float(end_pos));
    put_state(sp, 5 * NT, __int_as_float(nb));
    put_state(sp, 6 * NT, __int_as_float(stop_pos >= 0 ? (int)vals[rg.x + (uint32_t)stop_pos] : -1));
  }
}

template <int TW, int TH>
__global__ void __launch_bounds__(TW * TH)
    k_raster_fwd_sorted(Ws w, ViewSet vs, KCfg cfg, float *__restrict__ state,
                        const uint32_t *__restrict__ vals) {
  TileInfo ti;
  if (tile_info(vs, cfg, w, ti)) fwd_tile_sorted<TW, TH>(ti, w, vs, cfg, state, vals);
}

// ---------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------
// Per-pixel adjoint factors of the hybrid backward in LDS: G(3), w1, q1, q2,
// then per fragment code (0: tail, i + 1: core entry i) the pair (dL/dalpha
// of the core entry, dC/dc per alpha): (unused, w1), (T_i (c_i - B_i) . G,
// T_i), ... The core's list positions are read from the forward state when a
// chunk's code table is built.
template <int KMAX>
struct PixLayout {
  static constexpr int kPair = 6;
  // codes are stored as multiples of this (one byte): offsets of the pairs,
  // or half of them where 8 K does not fit a byte
  static constexpr int kCodeUnit = KMAX <= 16 ? 8 : 4;
  static constexpr int kStride = ((8 + 2 * KMAX) + 3) / 4 * 4;
};

// Gradient contribution of one fragment (lane's splat at the pixel whose
// factors lie at Pp, column c of its 8x8 block; c is a constant after
// unrolling) to the lane's accumulators; code: its fragment code times
// kCodeUnit. rs holds this row's sums of the d and m weights times (1, c,
// c^2). CLAMP false: no lane's opacity exceeds the alpha clamp.
template <int KMAX, bool CLAMP>
__device__ __forceinline__ void bwd_fragment(float op, const float *rgb, lds_bytes Pp, int c,
                                             float dd, float mm, uint32_t code, float amax,
                                             float *rs, float *acc) {
  using L = PixLayout<KMAX>;
  // alpha exactly as the forward's frag_alpha forms it
  const float inv = rcp_fast(dd);
  const float r2 = mm * inv;
  const float e = exp2_fast(r2 * kNegHalfLog2e);
  const float araw = op * e;
  float alpha = CLAMP ? __builtin_amdgcn_fmed3f(araw, 0.f, amax) : araw;
  asm("" : "+v"(alpha));   // (1 - alpha below from the rounded alpha, as the forward's)
  const float4v gw = *(lds_float4)Pp;            // G, w1
  const float2v q = *(lds_float2)(Pp + 16);      // q1, q2
  const float2v core = *(lds_float2)(Pp + (code * (8 / L::kCodeUnit)) + 4 * L::kPair);
  // tail: dC/dalpha = w1 (c - c_tail) - T P (c_bg - c_tail) / (1 - alpha),
  // dC/dc = w1 alpha; core: the pixel's precomputed T_i (c_i - B_i) and T_i
  const float gdc = fmaf(gw.z, rgb[2], fmaf(gw.y, rgb[1], gw.x * rgb[0]));
  const float tail = fmaf(gw.w, gdc, -q.x) - q.y * rcp_fast(1.f - alpha);
  const float dLda = code ? core.x : tail;
  const float wc = alpha * core.y;
  acc[13] = fmaf(wc, gw.x, acc[13]);
  acc[14] = fmaf(wc, gw.y, acc[14]);
  acc[15] = fmaf(wc, gw.z, acc[15]);
  // Where alpha is clamped, o and rho^2 receive no gradient.
  const float g = !CLAMP || araw <= amax ? dLda : 0.f;
  {
    acc[12] = fmaf(g, e, acc[12]);
    const float s1 = -alpha * g * inv;      // weight of m: 2 dL/drho^2 / |d|^2
    const float s2 = -s1 * r2;              // weight of d
    rs[0] += s2;
    rs[3] += s1;
    if (c >= 1) {
      const float fc = (float)c, fc2 = (float)(c * c);
      rs[1] = fmaf(fc, s2, rs[1]);
      rs[2] = fmaf(fc2, s2, rs[2]);
      rs[4] = fmaf(fc, s1, rs[4]);
      rs[5] = fmaf(fc2, s1, rs[5]);
    }
  }
}

// One instance partial: the lane's moments about the tile's first pixel
// (acc[0..5] for the d weights, acc[6..11] for the m weights) moved to
// an origin (a, b) pixels before it (dx = lx + a: sum w dx = S_x + a S,
// sum w dx^2 = S_xx + 2 a S_x + a^2 S, ...), then dL/do and dL/d(rgb).
__device__ __forceinline__ void form_partial(const float *acc, float a, float b, float *out) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float *S = acc + 6 * h;
    float *M = out + (h ? P_MM : P_MD);
    M[0] = S[0];
    M[1] = fmaf(a, S[0], S[1]);
    M[2] = fmaf(b, S[0], S[2]);
    M[3] = fmaf(a, fmaf(a, S[0], 2.f * S[1]), S[3]);
    M[4] = fmaf(a, fmaf(b, S[0], S[2]), fmaf(b, S[1], S[4]));
    M[5] = fmaf(b, fmaf(b, S[0], 2.f * S[2]), S[5]);
  }
  out[P_O] = acc[12];
  out[P_C] = acc[13];
  out[P_C + 1] = acc[14];
  out[P_C + 2] = acc[15];
}

// The wave's partials to their slots (kNoSlot: none), four lanes per 64-byte
// partial: a store of the wave then covers 16 partials instead of a quarter
// of 64, a quarter of the address work (6.6M partials to random slots take
// 174 instead of 247 us by themselves, the 1080p backward 517 instead of
// 549 us). buf: 4 KiB of LDS of the wave's own, row r's words rotated by
// r / 4 (no bank conflicts either way). STREAM: non-temporal stores, where the
// partials are far larger than the caches (the 4K frame's 6.5 GB: 7.42 ->
// 7.34 ms; sorted blending's sums read theirs back faster from the cache).
constexpr uint32_t kNoSlot = 0xffffffffu;
template <bool STREAM>
__device__ __forceinline__ void write_partials(const float *acc, float a, float b, uint32_t slot,
                                               float4 *buf, float *__restrict__ partials, int lane) {
  float out[kPartialFloats];
  form_partial(acc, a, b, out);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 4; ++k)
    buf[lane * 4 + (k ^ ((lane >> 2) & 3))] =
        make_float4(out[4 * k], out[4 * k + 1], out[4 * k + 2], out[4 * k + 3]);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = it * 16 + (lane >> 2);
    const uint32_t sl = (uint32_t)__shfl((int)slot, r, 64);
    const float4v v =
        *reinterpret_cast<const float4v *>(&buf[r * 4 + ((lane & 3) ^ ((r >> 2) & 3))]);
    float4v *dst =
        reinterpret_cast<float4v *>(partials) + ((int64_t)sl * (kPartialFloats / 4) + (lane & 3));
    if (sl != kNoSlot) {
      if constexpr (STREAM) __builtin_nontemporal_store(v, dst);
      else *dst = v;
    }
  }
  __builtin_amdgcn_wave_barrier();
}

// Waves per backward workgroup. A tile's 64-instance chunks are dealt to
// its waves round-robin, so waves whose share ends early idle until the
// tile is done; fewer waves idle less but stage the tile's per-pixel factors
// for fewer waves. One-block tiles with 1, 2, 3 and 4 waves: 516, 516, 532
// and 556 us at 1080p (205 instances per tile), 8.78, 7.80, 7.90 and 8.00 ms
// on the 4K frame (786 per tile).
// WIDE: for frames of few tiles, whose workgroups do not fill the chip, so
// that the chunks of a long list are walked side by side (the sums do not
// depend on which wave walks a chunk).
template <int TW, int TH, bool WIDE>
constexpr int bwd_waves() {
  return WIDE ? 8 : (TW * TH <= 64 ? 2 : 4);
}

// Target waves per SIMD of the backward (register budget; HIP's second
// launch-bounds argument is a minimum number of waves per execution unit).
// The walk of a one-block tile with K <= 8 fits 96 registers; at 80 it
// spills (630 against 516 us at 1080p; now 488). Tiles of several blocks with
// K <= 8, and tiles of up to two with K <= 16, fit 128 (16x16 with one register
// spilled); the others take 127 to 184, and LDS allows them no more
// than two or three waves anyway.
template <int KMAX, int TW, int TH>
constexpr int bwd_simd_waves() {
  return (TW * TH <= 64 && KMAX <= 8) ? 5 : ((KMAX <= 8 || (KMAX <= 16 && TW * TH <= 128)) ? 4 : 1);
}

// One tile of the backward. At 1080p (1M Gaussians, K = 8, 8x8 tiles) the
// walk's VALU work overlaps with the memory traffic (358 us with the walk left
// out: 143 of them for 0.42 GB of partials in random 64-byte slots, 40 for a
// 16-byte descriptor in a random line per instance, the rest 0.45 GB of state
// and 0.85 GB of records) to 488 us; on the 4K frame (K = 16) 5.6 of 7.4 ms
// remain without it. A SIMD issues an instruction per 3.5 cycles on both. The
// launch took 602 us with a branch per fragment that formed the code table's
// addresses lane by lane, tested the clamp and the smallest |d|^2 for every
// pixel and wrote 64 scattered partials per store, and 514 before the state and
// the partials became non-temporal; K = 16 with 16x8 tiles 941 -> 690 us, the 4K
// frame 8.83 -> 7.40 ms.
template <int KMAX, int TW, int TH, bool WIDE, bool EXACT>
__device__ __forceinline__ void bwd_tile(const TileInfo &ti, const Ws &w, const ViewSet &vs,
                                         const KCfg &cfg, const float *__restrict__ state,
                                         const uint32_t *__restrict__ vals, uint32_t &nfr) {
  constexpr int NT = TW * TH;
  constexpr int NB = NT / 64;
  constexpr int BX = TW / 8;
  using L = PixLayout<KMAX>;
  __shared__ float4 s_pix[NT * L::kStride / 4];
  constexpr int BW = bwd_waves<TW, TH, WIDE>();
  constexpr int BT = 64 * BW;
  // Per wave, for the 8x8 block being walked, the fragment codes of its
  // pixels by the chunk's instances: codes[wave][r][2 lane], [2 lane + 1]
  // hold the eight bytes of row r for instance `lane` (core index + 1, 0
  // where the instance is not in the core, times kCodeUnit). A lane reads
  // its codes once per row, without bank conflicts, and a pixel's byte is an
  // address offset as it stands. The table also carries the paired waves'
  // sums and the partials on their way out (16 floats per lane).
  __shared__ __attribute__((aligned(16))) uint32_t s_code[BW][8][128];
  static_assert(sizeof(s_code[0]) == 64 * 16 * sizeof(float), "one partial per lane");

  uint2 rg = w.ranges[ti.t];
  rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
  rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
  if (rg.x >= rg.y) return;   // nothing to differentiate
  const ViewParams &V = vs.v[ti.v];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px0 = ti.tx * TW, py0 = ti.ty * TH;
  const int K = EXACT ? KMAX : cfg.K;
  const float *recs = w.records + (int64_t)ti.v * cfg.n * kRecFloats;
  const int64_t npix = (int64_t)V.width * V.height;
  float *sp_all = reinterpret_cast<float *>(s_pix);

  // Per-pixel adjoint factors. Threads walk the pixels in the state's
  // order (8x8 blocks, row-major inside), so consecutive threads read
  // consecutive state words.
  const float *tstate = state + tile_state_off(V, ti, state_values(K), NT);
  for (int ps = tid; ps < NT; ps += BT) {
    const int lxp = ((ps >> 6) % BX) * 8 + (ps & 7), lyp = ((ps >> 6) / BX) * 8 + ((ps >> 3) & 7);
    const int p = lyp * TW + lxp;
    const int px = px0 + lxp, py = py0 + lyp;
    float *Pp = sp_all + p * L::kStride;
    float G[3] = {0.f, 0.f, 0.f}, w1 = 0.f, q1 = 0.f, q2 = 0.f;
    int pos[KMAX];
    float coef[KMAX], Ti[KMAX];
#pragma unroll
    for (int i = 0; i < KMAX; ++i) { pos[i] = -1; coef[i] = 0.f; Ti[i] = 0.f; }
    if (px < V.width && py < V.height) {
      const int64_t pix = (int64_t)py * V.width + px;
      for (int c = 0; c < 3; ++c) G[c] = V.grad_rgb[c * npix + pix];
      const float *sp = tstate + ps;
      float ca[KMAX], cc[KMAX][3];
#pragma unroll
      for (int i = 0; i < KMAX; ++i) {
        ca[i] = 0.f; cc[i][0] = cc[i][1] = cc[i][2] = 0.f;
        if (i < K) {
          // all loads independent of each other (one round trip); empty
          // entries (position -1) get alpha and colour 0 from the forward
          // (the positions are read again, chunk by chunk)
          ca[i] = get_state(sp, (int64_t)(K + i) * NT);
          pos[i] = __float_as_int(sp[(int64_t)(2 * K + i) * NT]);
          cc[i][0] = get_state(sp, (int64_t)(3 * K + 3 * i) * NT);
          cc[i][1] = get_state(sp, (int64_t)(3 * K + 3 * i + 1) * NT);
          cc[i][2] = get_state(sp, (int64_t)(3 * K + 3 * i + 2) * NT);
        }
      }
      const float A = sp[(int64_t)(6 * K + 1) * NT];
      const float S[3] = {sp[(int64_t)(6 * K + 2) * NT], sp[(int64_t)(6 * K + 3) * NT],
                          sp[(int64_t)(6 * K + 4) * NT]};
      const float Pt = sp[(int64_t)(6 * K + 5) * NT];
      float T = 1.f;
#pragma unroll
      for (int i = 0; i < KMAX; ++i) {
        if (i < K && pos[i] >= 0) {
          Ti[i] = T;
          T *= 1.f - ca[i];
        }
      }
      float X[3], ct[3] = {0.f, 0.f, 0.f};
      const bool has_tail = A > 0.f;
      for (int c = 0; c < 3; ++c) {
        X[c] = Pt * cfg.bg[c];
        if (has_tail) {
          ct[c] = S[c] / A;
          X[c] = fmaf(1.f - Pt, ct[c], X[c]);
        }
      }
      float B[3] = {X[0], X[1], X[2]};
#pragma unroll
      for (int i = KMAX - 1; i >= 0; --i) {
        if (i < K && pos[i] >= 0) {
          coef[i] = Ti[i] * (G[0] * (cc[i][0] - B[0]) + G[1] * (cc[i][1] - B[1]) +
                             G[2] * (cc[i][2] - B[2]));
          for (int c = 0; c < 3; ++c) B[c] = fmaf(ca[i], cc[i][c] - B[c], B[c]);
        }
      }
      if (has_tail) {
        w1 = T * (1.f - Pt) / A;
        q1 = w1 * (G[0] * ct[0] + G[1] * ct[1] + G[2] * ct[2]);
        q2 = T * Pt *
             (G[0] * (cfg.bg[0] - ct[0]) + G[1] * (cfg.bg[1] - ct[1]) + G[2] * (cfg.bg[2] - ct[2]));
      }
    }
    Pp[0] = G[0]; Pp[1] = G[1]; Pp[2] = G[2];
    Pp[3] = w1; Pp[4] = q1; Pp[5] = q2;
    Pp[L::kPair] = 0.f; Pp[L::kPair + 1] = w1;
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      Pp[L::kPair + 2 + 2 * i] = coef[i];
      Pp[L::kPair + 3 + 2 * i] = Ti[i];
    }
  }

  const uint32_t count = rg.y - rg.x;
  const uint32_t nch = (count + 63u) >> 6;
  const float amax = cfg.alpha_max;
  // Chunk schedule. In general a wave takes every BW-th chunk over all of
  // the tile's 8x8 blocks. With two blocks (16x8 tiles) a pair of waves
  // shares each chunk instead, one block each, and the pairs take the
  // chunks in turn; the block-1 wave hands its sums to the
  // block-0 wave, which writes the partial. A tile whose chunk count is not
  // a multiple of the wave count then leaves fewer waves idle.
  constexpr bool PAIRS = NB == 2;
  constexpr uint32_t NP = BW / 2;   // pairs
  const int myblk = PAIRS ? wave / (int)NP : -1;
  const uint32_t c_end = PAIRS ? NP * ((nch + NP - 1u) / NP) : nch;  // uniform when PAIRS
  const uint32_t c_step = PAIRS ? NP : (uint32_t)BW;
  const int cx2 = 2 * px0 + TW - 1, cy2 = 2 * py0 + TH - 1;
  const float hx = 0.5f * (float)(TW - 1), hy = 0.5f * (float)(TH - 1);
  // The factors are complete at the first chunk's barrier, behind its loads
  // and staging: the waves without pixels of their own do those meanwhile.
  bool ready = false;
  for (uint32_t c = PAIRS ? (uint32_t)wave % NP : (uint32_t)wave; c < c_end; c += c_step) {
    const uint32_t j = rg.x + c * 64u + lane;
    const bool active = c < nch && j < rg.y;
    // The forward's staged forms of |d|^2 and |m|^2 for this (tile, splat)
    // (stage_fwd, same arithmetic), so that every pixel's |d|^2, |m|^2,
    // fragment test and alpha are bit-identical to the forward's: the
    // backward differentiates exactly the fragments the image blended.
    float qd[6], qm[6], rc = -1.f, op = 0.f, rgb[3] = {0.f, 0.f, 0.f};
    int bb[4] = {1 << 20, 1 << 20, -1, -1};
#pragma unroll
    for (int k = 0; k < 6; ++k) { qd[k] = 0.f; qm[k] = 0.f; }
    uint32_t slot = 0, gid = 0;
    int ox = 0, oy = 0;   // moment origin: the record's reference pixel
    if (active) {
      gid = vals[j];
      float rec[kRecFloats];
      load_record(recs, gid, rec);
      float sf[F_FLOATS];
      stage_fwd(rec, cx2, cy2, sf);
#pragma unroll
      for (int k = 0; k < 6; ++k) { qd[k] = sf[F_QD + k]; qm[k] = sf[F_QM + k]; }
      rc = sf[F_RC];
      op = sf[F_O];
      rgb[0] = sf[F_R]; rgb[1] = sf[F_G]; rgb[2] = sf[F_B];
      const uint32_t b0 = __float_as_uint(rec[R_BB0]), b1 = __float_as_uint(rec[R_BB1]);
      bb[0] = (int)(b0 & 0xffffu) - px0;
      bb[1] = (int)(b0 >> 16) - py0;
      bb[2] = (int)(b1 & 0xffffu) - px0;
      bb[3] = (int)(b1 >> 16) - py0;
      if (myblk <= 0) {
        slot = tslot_slot(w.tslots[(int64_t)ti.v * cfg.n + gid], ti.tx, ti.ty);
        ox = __float_as_int(rec[R_IX]);
        oy = __float_as_int(rec[R_IY]);
      }
    }
    if (!ready) __syncthreads();
    ready = true;
    const float bbf[4] = {__int_as_float(bb[0]), __int_as_float(bb[1]), __int_as_float(bb[2]),
                          __int_as_float(bb[3])};
    // Whether every alpha of this splat stays below the clamp and |d|^2 above
    // the smallest normal float all over the tile (|d|^2 - |its value at the
    // centre| bounded by the coefficients' magnitudes): the walk then leaves
    // out both tests.
    const float ddmin = qd[0] - fmaf(hx, fabsf(qd[1]), fmaf(hy, fabsf(qd[2]), hx * hy * fabsf(qd[4])));
    const bool plain = op <= amax && ddmin > 1e-30f;
    // acc: d-moments (6), m-moments (6), dL/do, dL/drgb (3)
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.f;
    float nf = 0.f;   // this chunk's fragments
    for (int blk = 0; blk < NB; ++blk) {
      if (PAIRS && blk != myblk) continue;
      const int bx = (blk % BX) * 8, by = (blk / BX) * 8;
      const bool hitb = active && rect_meets_block(bbf, bx, by);
      if (__ballot(hitb) == 0ull) continue;
      // Core table of this block for this chunk: lane = block pixel.
      {
        // list positions of the pixel's core from the forward state
        // (opaque offset: the entries' addresses would be kept over the chunks)
        uint32_t off = (uint32_t)(blk * 64 + lane);
        asm volatile("" : "+v"(off));
        int cps[KMAX];
#pragma unroll
        for (int i = 0; i < KMAX; ++i)
          cps[i] = i < K ? __float_as_int(tstate[off + (uint32_t)((2 * K + i) * NT)]) : -1;
        uint4 *tab = reinterpret_cast<uint4 *>(&s_code[wave][0][0]);
#pragma unroll
        for (int k = 0; k < 4; ++k) tab[k * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_wave_barrier();
        // (opaque: the shifted codes would be kept over the chunks)
        uint32_t bit = (uint32_t)((lane & 3) * 8);
        asm volatile("" : "+v"(bit));
        uint32_t *row = &s_code[wave][lane >> 3][(lane >> 2) & 1];
#pragma unroll
        for (int i = 0; i < KMAX; ++i) {
          if (i < K) {
            const uint32_t dl = (uint32_t)(cps[i] - (int)(c * 64u));
            if (cps[i] >= 0 && dl < 64u) atomicOr(&row[2 * dl], (uint32_t)((i + 1) * L::kCodeUnit) << bit);
          }
        }
        __builtin_amdgcn_wave_barrier();
      }
      // Pixels of the block inside the image (the forward skips the rest).
      const int cols_in = V.width - (px0 + bx), rows_in = V.height - (py0 + by);
      // A row at a time: the row's parts of the two staged forms (Y, the
      // pixel's offset from the tile centre, fixed), then two FMAs per pixel
      // for each; the columns are unrolled, so for one-block tiles X is a
      // constant. The moments (1, lx, ly, lx^2, lx ly, ly^2) of the weights
      // follow from per-row sums over (1, c, c^2).
      const float fbx = (float)bx;
      auto walk = [&](auto rare) __attribute__((always_inline)) {
        constexpr bool RARE = decltype(rare)::value;
        for (int row = 0; row < 8; ++row) {
          const float ly = (float)(by + row);
          const float Y = ly - hy, YY = Y * Y;
          const float rd0 = fmaf(YY, qd[5], fmaf(Y, qd[2], qd[0]));
          const float rd1 = fmaf(Y, qd[4], qd[1]);
          const float s2 = fmaf(qm[4], Y, qm[5]);
          const float rm0 = fmaf(s2, s2, qm[0]);
          const float rm1 = fmaf(qm[2], Y, qm[3]);
          // (bitwise ands: both pixels of a column pair are tested before
          // either fragment path branches, and no test branches on its own)
          const bool row_in = hitb & (row < rows_in);
          float rs[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          // (rs[1] and rs[2] agree up to column 1: opaque, or they share a
          // register until they part in column 2's path)
          asm("" : "+v"(rs[2]), "+v"(rs[5]));
          const uint2 codes = reinterpret_cast<const uint2 *>(s_code[wave][row])[lane];
          auto code_of = [&](int col) -> uint32_t {
            return ((col < 4 ? codes.x : codes.y) >> (8 * (col & 3))) & 255u;
          };
          // (in a vector register: its reads take the column as their offset)
          lds_bytes P = (lds_bytes)(const char *)(sp_all + ((by + row) * TW + bx) * L::kStride);
          asm("" : "+v"(P));
#pragma unroll
          for (int col = 0; col < 8; col += 2) {
            const float X0 = (fbx + (float)col) - hx, X1 = X0 + 1.f;
            const float dd0 = fmaf(X0, rd1, fmaf(X0 * X0, qd[3], rd0));
            const float dd1 = fmaf(X1, rd1, fmaf(X1 * X1, qd[3], rd0));
            const float s10 = fmaf(qm[1], X0, rm1), s11 = fmaf(qm[1], X1, rm1);
            const float mm0 = fmaf(s10, s10, rm0), mm1 = fmaf(s11, s11, rm0);
            const bool f0 = row_in & (col < cols_in) & (!RARE || dd0 >= FLT_MIN) & (mm0 <= rc * dd0);
            const bool f1 = row_in & (col + 1 < cols_in) & (!RARE || dd1 >= FLT_MIN) & (mm1 <= rc * dd1);
            if (f0) {
              nf += 1.f;
              bwd_fragment<KMAX, RARE>(op, rgb, P + col * 4 * L::kStride, col, dd0, mm0, code_of(col), amax, rs, acc);
            }
            if (f1) {
              nf += 1.f;
              bwd_fragment<KMAX, RARE>(op, rgb, P + (col + 1) * 4 * L::kStride, col + 1, dd1, mm1,
                           code_of(col + 1), amax, rs, acc);
            }
          }
          if constexpr (BX > 1) {
            // sums over (1, c, c^2) -> over (1, lx, lx^2), lx = bx + c
            rs[2] = fmaf(fbx, fmaf(fbx, rs[0], 2.f * rs[1]), rs[2]);
            rs[1] = fmaf(fbx, rs[0], rs[1]);
            rs[5] = fmaf(fbx, fmaf(fbx, rs[3], 2.f * rs[4]), rs[5]);
            rs[4] = fmaf(fbx, rs[3], rs[4]);
          }
          const float ly2 = ly * ly;
          acc[0] += rs[0];
          acc[1] += rs[1];
          acc[2] = fmaf(ly, rs[0], acc[2]);
          acc[3] += rs[2];
          acc[4] = fmaf(ly, rs[1], acc[4]);
          acc[5] = fmaf(ly2, rs[0], acc[5]);
          acc[6] += rs[3];
          acc[7] += rs[4];
          acc[8] = fmaf(ly, rs[3], acc[8]);
          acc[9] += rs[5];
          acc[10] = fmaf(ly, rs[4], acc[10]);
          acc[11] = fmaf(ly2, rs[3], acc[11]);
        }
      };
      // (uniform over the wave)
      if (__ballot(hitb && !plain) != 0ull) walk(std::true_type{});
      else walk(std::false_type{});
      __builtin_amdgcn_wave_barrier();
    }
    nfr += (uint32_t)nf;
    if constexpr (PAIRS) {
      // The block-1 wave's code table is free now: it carries the sums.
      float *xch = reinterpret_cast<float *>(&s_code[PAIRS ? (int)NP + wave % (int)NP : 0][0][0]);
      if (myblk == 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) xch[k * 64 + lane] = acc[k];
      }
      __syncthreads();
      if (myblk == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] += xch[k * 64 + lane];
      }
      __syncthreads();  // before the block-1 waves rebuild their tables
    }
    if (myblk <= 0) {
      // The tile's moments (about its first pixel) moved to the record's
      // reference pixel, (a, b) pixels from it (near the splat's centre,
      // which keeps the moments small): with dx = lx + a,
      // sum w dx = S_x + a S, sum w dx^2 = S_xx + 2 a S_x + a^2 S, ...
      const bool out = active && (uint64_t)slot < (uint64_t)w.capacity;
      write_partials<true>(acc, (float)(px0 - ox), (float)(py0 - oy), out ? slot : kNoSlot,
                     reinterpret_cast<float4 *>(&s_code[wave][0][0]), w.partials, lane);
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (!ready) __syncthreads();   // (a wave without a chunk)
}

// Minimum waves per SIMD asked of the compiler for the forward (HIP's
// second launch bound): what LDS leaves room for (8x8 tiles with K = 8 take
// 8.8 KiB per wave, 18 waves per CU).
template <int KMAX, int TW, int TH, int BM>
constexpr int fwd_simd_waves() {
  return (KMAX > 8 || BM > 1 || TW * TH > 128) ? 1 : 4;
}

template <int KMAX, int TW, int TH, int BM, bool EXACT>
__global__ void __launch_bounds__((TW * TH), (fwd_simd_waves<KMAX, TW, TH, BM>()))
    k_raster_fwd(Ws w, ViewSet vs, KCfg cfg, float *__restrict__ state,
                 const uint32_t *__restrict__ vals) {
  TileInfo ti;
  if (tile_info(vs, cfg, w, ti))
    fwd_tile<KMAX, TW, TH, BM, EXACT, false>(ti, w, vs, cfg, state, vals);
}

// Views with a negative z_near (any K up to KMAX).
template <int KMAX, int TW, int TH>
__global__ void __launch_bounds__(TW * TH)
    k_raster_fwd_behind(Ws w, ViewSet vs, KCfg cfg, float *__restrict__ state,
                        const uint32_t *__restrict__ vals) {
  TileInfo ti;
  if (tile_info(vs, cfg, w, ti))
    fwd_tile<KMAX, TW, TH, 1, false, true>(ti, w, vs, cfg, state, vals);
}

template <int KMAX, int TW, int TH, bool WIDE, bool EXACT>
__global__ void __launch_bounds__((64 * bwd_waves<TW, TH, WIDE>()), (bwd_simd_waves<KMAX, TW, TH>()))
    k_raster_bwd(Ws w, ViewSet vs, KCfg cfg, const float *__restrict__ state,
                 const uint32_t *__restrict__ vals) {
  // the forward of a failed front end rendered empty tiles: nothing to do
  if (front_failed(w)) return;
  uint32_t nfr = 0;   // fragments this thread differentiated
  TileInfo ti;
  if (tile_info(vs, cfg, w, ti)) bwd_tile<KMAX, TW, TH, WIDE, EXACT>(ti, w, vs, cfg, state, vals, nfr);
  // one atomic per wave (a word of LDS would take the 8x8 and 16x8 kernels
  // past 16 and 32 KiB, one workgroup per CU fewer)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) nfr += (uint32_t)__shfl_xor((int)nfr, off, 64);
  if ((threadIdx.x & 63) == 0 && nfr) count_add(w.frags_bwd, (unsigned long long)nfr);
}

// ---------------------------------------------------------------------------
// Backward, sorted blending
// ---------------------------------------------------------------------------
// Inclusive scans over the 64 lanes of a wave: shifts by 1, 2, 4, 8 inside
// each row of 16 lanes, then lane 15 into rows 1 and 3 and lane 31 into rows
// 2 and 3, each one operation with a DPP operand (a move into the identity
// and an operation took three). Lanes without a source, and rows that are
// masked out, keep their value. A DPP operand needs two wait states after the
// write of its register. All 64 lanes. (1M Gaussians at 1280x720: the sorted
// backward 326 -> 285 us, with the partials' four-lane stores.)
#define HTGS_WAVE_SCAN(first, op, x)                                                  \
  asm(first                                                                           \
      "s_nop 1\n\t" op " %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"        \
      "s_nop 1\n\t" op " %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"        \
      "s_nop 1\n\t" op " %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"        \
      "s_nop 1\n\t" op " %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"     \
      "s_nop 1\n\t" op " %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"     \
      "s_nop 1"                                                                       \
      : "+v"(x))
__device__ __forceinline__ float wave_scan_mul(float x) {
  HTGS_WAVE_SCAN("s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t",
                 "v_mul_f32_dpp", x);
  return x;
}
// (of a b, the sum's first step as a multiply-add)
__device__ __forceinline__ float wave_scan_add(float a, float b) {
  float x = a * b;
  x = fmaf(a, b, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf,
                                                            false)));
  HTGS_WAVE_SCAN("", "v_add_f32_dpp", x);
  return x;
}
// The lane before's value; `first` in lane 0. All 64 lanes.
__device__ __forceinline__ float wave_shift(float x, float first) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(x),
                                                    0x138, 0xf, 0xf, false));   // wave_shr:1
}

// Adjoint of sorted blending. With the fragments of a pixel blended front
// to back, C = sum_i alpha_i T_i c_i + T c_bg, T_i = prod_{k<i} (1 -
// alpha_k):
//   dC/dc_i = alpha_i T_i,
//   dC/dalpha_i = T_i c_i - R_i / (1 - alpha_i),  R_i = sum_{k>i} alpha_k T_k
//                 c_k + T c_bg = C - (sum_{k<=i} alpha_k T_k c_k).
// The lanes of a wave hold 64 consecutive list entries (splats) of the tile
// and walk the pixels of their 8x8 block; at a pixel a wave scan over the
// lanes gives each lane T_i (product of 1 - alpha) and the dot product with
// G = dL/dC of the prefix colour sum, starting from the pixel's carry of the
// earlier chunks (kept in LDS), so the chunks of a tile run in list order.
// A lane's fragment is differentiated iff the forward blended it: its list
// position lies before the pixel's end position stored by the forward (the
// same staged forms and arithmetic give the same fragment test and alpha).
// Partials as in the hybrid backward: moments of the d and m weights, opacity
// and colour terms, one per instance. One wave per 8x8 block; with several
// blocks the waves add their sums in LDS and wave 0 writes the partial.
template <int TW, int TH>
__device__ __forceinline__ void bwd_tile_sorted(const TileInfo &ti, const Ws &w,
                                                const ViewSet &vs, const KCfg &cfg,
                                                const float *__restrict__ state,
                                                const uint32_t *__restrict__ vals, uint32_t &nfr) {
  constexpr int NT = TW * TH;
  constexpr int NB = NT / 64;
  constexpr int BX = TW / 8;
  // per pixel: G (3), G . C, then end position, T carry, (G . prefix) carry
  __shared__ float4 s_pg[NT], s_pc[NT];
  __shared__ float s_red[NB > 1 ? NB * 16 * 64 : 1];   // [block][value][lane]
  __shared__ float4 s_out[256];   // write_partials
  __shared__ int s_maxend;

  const ViewParams &V = vs.v[ti.v];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bx = (wave % BX) * 8, by = (wave / BX) * 8;
  const int px0 = ti.tx * TW, py0 = ti.ty * TH;
  const float *recs = w.records + (int64_t)ti.v * cfg.n * kRecFloats;
  const int64_t npix = (int64_t)V.width * V.height;
  if (tid == 0) s_maxend = 0;
  __syncthreads();
  {
    // this thread's pixel: block `wave`, lane = row-major pixel of the block
    const int lx = bx + (lane & 7), ly = by + (lane >> 3);
    const int px = px0 + lx, py = py0 + ly;
    float4 pg = make_float4(0.f, 0.f, 0.f, 0.f), pc = make_float4(0.f, 1.f, 0.f, 0.f);
    if (px < V.width && py < V.height) {
      const int64_t pix = (int64_t)py * V.width + px;
      const float *sp = state + tile_state_off(V, ti, kSortedStateValues, NT) + wave * 64 + lane;
      const float T = sp[0], S0 = sp[NT], S1 = sp[2 * NT], S2 = sp[3 * NT];
      const int end = __float_as_int(sp[4 * NT]);
      const float G0 = V.grad_rgb[pix], G1 = V.grad_rgb[npix + pix], G2 = V.grad_rgb[2 * npix + pix];
      const float gC = fmaf(G2, fmaf(T, cfg.bg[2], S2), fmaf(G1, fmaf(T, cfg.bg[1], S1),
                                                          G0 * fmaf(T, cfg.bg[0], S0)));
      pg = make_float4(G0, G1, G2, gC);
      pc = make_float4(__int_as_float(end), 1.f, 0.f, 0.f);
      if (end > 0) atomicMax(&s_maxend, end);
    }
    s_pg[ly * TW + lx] = pg;
    s_pc[ly * TW + lx] = pc;
  }
  __syncthreads();
  const uint2 rg = w.ranges[ti.t];
  // no pixel blends past max_end: later list entries get zero partials
  // (every instance's slot is written, as the preprocess backward sums them)
  const uint32_t stop = min(rg.y, rg.x + (uint32_t)s_maxend);
  const float amax = cfg.alpha_max;
  const int cx2 = 2 * px0 + TW - 1, cy2 = 2 * py0 + TH - 1;
  const float hx = 0.5f * (float)(TW - 1), hy = 0.5f * (float)(TH - 1);
  const int cols_in = V.width - (px0 + bx), rows_in = V.height - (py0 + by);
  for (uint32_t c0 = rg.x; c0 < rg.y; c0 += 64u) {
    const uint32_t j = c0 + lane;
    const bool active = j < rg.y;
    const bool work = j < stop;
    const int pos = (int)(j - rg.x);
    float qd[6], qm[6], rc = -1.f, op = 0.f, rgb[3] = {0.f, 0.f, 0.f};
    int bb[4] = {1 << 20, 1 << 20, -1, -1};
#pragma unroll
    for (int k = 0; k < 6; ++k) { qd[k] = 0.f; qm[k] = 0.f; }
    const uint32_t gid = active ? vals[j] : 0u;
    int ox = 0, oy = 0;   // moment origin: the record's reference pixel
    if (work) {
      float rec[kRecFloats];
      load_record(recs, gid, rec);
      ox = __float_as_int(rec[R_IX]);
      oy = __float_as_int(rec[R_IY]);
      float sf[F_FLOATS];
      stage_fwd(rec, cx2, cy2, sf);
#pragma unroll
      for (int k = 0; k < 6; ++k) { qd[k] = sf[F_QD + k]; qm[k] = sf[F_QM + k]; }
      rc = sf[F_RC];
      op = sf[F_O];
      rgb[0] = sf[F_R]; rgb[1] = sf[F_G]; rgb[2] = sf[F_B];
      const uint32_t b0 = __float_as_uint(rec[R_BB0]), b1 = __float_as_uint(rec[R_BB1]);
      bb[0] = (int)(b0 & 0xffffu) - px0;
      bb[1] = (int)(b0 >> 16) - py0;
      bb[2] = (int)(b1 & 0xffffu) - px0;
      bb[3] = (int)(b1 >> 16) - py0;
    }
    const float bbf[4] = {__int_as_float(bb[0]), __int_as_float(bb[1]), __int_as_float(bb[2]),
                          __int_as_float(bb[3])};
    const bool hitb = work && rect_meets_block(bbf, bx, by);
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.f;
    if (__ballot(hitb) != 0ull) {
      const float fbx = (float)bx;
      for (int row = 0; row < 8; ++row) {
        const float ly = (float)(by + row);
        const float Y = ly - hy, YY = Y * Y;
        const float rd0 = fmaf(YY, qd[5], fmaf(Y, qd[2], qd[0]));
        const float rd1 = fmaf(Y, qd[4], qd[1]);
        const float s2r = fmaf(qm[4], Y, qm[5]);
        const float rm0 = fmaf(s2r, s2r, qm[0]);
        const float rm1 = fmaf(qm[2], Y, qm[3]);
        const bool row_in = hitb & (row < rows_in);
        float rs[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int col = 0; col < 8; ++col) {
          const int p = (by + row) * TW + bx + col;
          const float4 pc = s_pc[p];
          const float X = (fbx + (float)col) - hx;
          const float dd = fmaf(X, rd1, fmaf(X * X, qd[3], rd0));
          const float s1 = fmaf(qm[1], X, rm1);
          const float mm = fmaf(s1, s1, rm0);
          const bool f = row_in & (col < cols_in) & (dd >= FLT_MIN) & (mm <= rc * dd) &
                         (pos < __float_as_int(pc.x));
          if (__ballot(f) == 0ull) continue;   // uniform: no blended fragment here
          const float4 pg = s_pg[p];
          // alpha exactly as the forward forms it (0 off the fragments)
          const float inv = rcp_fast(dd);
          const float r2 = mm * inv;
          const float e = exp2_fast(r2 * kNegHalfLog2e);
          const float araw = op * e;
          const bool unclamped = araw <= amax;
          const float alpha = f ? (unclamped ? araw : amax) : 0.f;
          const float om = 1.f - alpha;
          const float incl = wave_scan_mul(om);
          const float excl = wave_shift(incl, 1.f);
          const float Ti = pc.y * excl;
          const float gc = fmaf(pg.z, rgb[2], fmaf(pg.y, rgb[1], pg.x * rgb[0]));
          const float isum = wave_scan_add(alpha * Ti, gc);
          const float gP = pc.z + isum;   // G . (colour sum up to and including i)
          // the pixel's carries past this chunk
          const float tot_m = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(incl), 63));
          const float tot_s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(isum), 63));
          if (lane == 0) s_pc[p] = make_float4(pc.x, pc.y * tot_m, pc.z + tot_s, 0.f);
          if (f) {
            ++nfr;
            const float dLda = Ti * gc - (pg.w - gP) * rcp_fast(om);
            const float wc = alpha * Ti;
            acc[13] = fmaf(wc, pg.x, acc[13]);
            acc[14] = fmaf(wc, pg.y, acc[14]);
            acc[15] = fmaf(wc, pg.z, acc[15]);
            const float g = unclamped ? dLda : 0.f;
            acc[12] = fmaf(g, e, acc[12]);
            const float w1 = -alpha * g * inv;   // weight of m
            const float w2 = -w1 * r2;           // weight of d
            rs[0] += w2;
            rs[3] += w1;
            const float fc = (float)col, fc2 = (float)(col * col);
            rs[1] = fmaf(fc, w2, rs[1]);
            rs[2] = fmaf(fc2, w2, rs[2]);
            rs[4] = fmaf(fc, w1, rs[4]);
            rs[5] = fmaf(fc2, w1, rs[5]);
          }
        }
        if constexpr (BX > 1) {
          rs[2] = fmaf(fbx, fmaf(fbx, rs[0], 2.f * rs[1]), rs[2]);
          rs[1] = fmaf(fbx, rs[0], rs[1]);
          rs[5] = fmaf(fbx, fmaf(fbx, rs[3], 2.f * rs[4]), rs[5]);
          rs[4] = fmaf(fbx, rs[3], rs[4]);
        }
        const float ly2 = ly * ly;
        acc[0] += rs[0];
        acc[1] += rs[1];
        acc[2] = fmaf(ly, rs[0], acc[2]);
        acc[3] += rs[2];
        acc[4] = fmaf(ly, rs[1], acc[4]);
        acc[5] = fmaf(ly2, rs[0], acc[5]);
        acc[6] += rs[3];
        acc[7] += rs[4];
        acc[8] = fmaf(ly, rs[3], acc[8]);
        acc[9] += rs[5];
        acc[10] = fmaf(ly, rs[4], acc[10]);
        acc[11] = fmaf(ly2, rs[3], acc[11]);
      }
    }
    if constexpr (NB > 1) {
      // the blocks' sums for each instance, added in block order
#pragma unroll
      for (int k = 0; k < 16; ++k) s_red[(wave * 16 + k) * 64 + lane] = acc[k];
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          float t = s_red[k * 64 + lane];
#pragma unroll
          for (int b2 = 1; b2 < NB; ++b2) t += s_red[(b2 * 16 + k) * 64 + lane];
          acc[k] = t;
        }
      }
      __syncthreads();
    }
    if (wave == 0) {
      uint32_t slot = kNoSlot;
      if (active) slot = tslot_slot(w.tslots[(int64_t)ti.v * cfg.n + gid], ti.tx, ti.ty);
      if ((uint64_t)slot >= (uint64_t)w.capacity) slot = kNoSlot;
      // (lanes past the last blended position were not staged: their
      // moments are zero, so the origin does not matter)
      write_partials<false>(acc, (float)(px0 - ox), (float)(py0 - oy), slot, s_out, w.partials, lane);
    }
  }
}

template <int TW, int TH>
__global__ void __launch_bounds__(TW * TH)
    k_raster_bwd_sorted(Ws w, ViewSet vs, KCfg cfg, const float *__restrict__ state,
                        const uint32_t *__restrict__ vals) {
  if (front_failed(w)) return;
  uint32_t nfr = 0;
  TileInfo ti;
  if (tile_info(vs, cfg, w, ti)) bwd_tile_sorted<TW, TH>(ti, w, vs, cfg, state, vals, nfr);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) nfr += (uint32_t)__shfl_xor((int)nfr, off, 64);
  if ((threadIdx.x & 63) == 0 && nfr) count_add(w.frags_bwd, (unsigned long long)nfr);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Workgroups of a raster launch: one per tile slot, the slots in whole groups
// of eight XCD chunks.
static dim3 tile_grid(const ViewSet &vs, const KCfg &cfg) {
  const int group = 8 << cfg.xcd_shift;
  return dim3((unsigned)((vs.total_tiles + group - 1) / group * group));
}
template <int KMAX, int TW, int TH, int BM, bool EXACT>
static hipError_t fwd_launch_bm(const Ws &w, const ViewSet &vs, const KCfg &cfg, float *state,
                                const uint32_t *vals, hipStream_t s) {
  hipLaunchKernelGGL((k_raster_fwd<KMAX, TW, TH, BM, EXACT>), tile_grid(vs, cfg), dim3(TW * TH), 0, s, w, vs, cfg, state, vals);
  return hipGetLastError();
}

template <int KMAX, int TW, int TH, bool EXACT>
static hipError_t fwd_launch(const Ws &w, const ViewSet &vs, const KCfg &cfg, float *state,
                             const uint32_t *vals, hipStream_t s) {
  if (vs.behind) {
    hipLaunchKernelGGL((k_raster_fwd_behind<KMAX, TW, TH>), tile_grid(vs, cfg), dim3(TW * TH), 0, s, w, vs, cfg, state, vals);
    return hipGetLastError();
  }
  if constexpr (TW == 8) {
    if (cfg.batch_mult == 2) return fwd_launch_bm<KMAX, TW, TH, 2, EXACT>(w, vs, cfg, state, vals, s);
  }
  return fwd_launch_bm<KMAX, TW, TH, 1, EXACT>(w, vs, cfg, state, vals, s);
}

// Frames of up to 512 tiles take the wide backward where there is room for more
// than 64 instances per tile; with less there is nothing to share. (Room, not
// the lists' length, which the host does not know: short lists in a roomy
// workspace take 18.6 -> 20.4 us with 16x8 tiles and K = 16, within 0.5 us of
// the other form with 8x8 or 16x16 tiles and K = 8.) Up to 128 VGPRs two
// workgroups share a CU and all tiles run at once: 50k Gaussians, 256 and 504
// tiles of 8x8 with K = 8 275 -> 88 and 230 -> 97 us, 16x8 with K = 16 261 -> 172
// and 249 -> 207, 16x16 with K = 8 511 -> 304 and 450 -> 343; past 512 it loses
// where lists are short (1200 tiles of 16x16, K = 8: 84 -> 119 us with 50k
// Gaussians, 216 -> 178 with 300k; 2048 of 8x8 32 -> 42). The forms with more
// registers (K > 16, and 8 < K <= 16 with tiles of 256 pixels but for 32x8 with
// K = 16) run one workgroup per CU, 256 tiles at a time, and still win or draw
// up to 512 tiles (50k Gaussians, 504 tiles of 8x8 with K = 32 264 -> 117, of
// 16x16 with K = 12 478 -> 338, of 32x8 with K = 12 425 -> 415; with 5k 43 -> 37,
// 92 -> 95, 91 -> 64), except 16x8 with K > 16, whose four pairs of waves share
// less. K = 24 with 160, 300 to 350, 600 to 700 and 1500 to 1750 instances per
// tile: 59 -> 71, 88 -> 86, 144 -> 119 and 324 -> 209 us at 272 tiles, 58 -> 73,
// 85 -> 89, 146 -> 121 and 305 -> 236 at 304, 61 -> 75, 83 -> 91, 133 -> 148 and
// 299 -> 266 at 384, 61 -> 75, 87 -> 91, 132 -> 148 and 287 -> 306 at 448.
template <int KMAX, int TW, int TH>
static bool few_tiles(const Ws &w, const ViewSet &vs) {
  const int64_t tiles = vs.total_tiles;
  if (KMAX > 16 && TW * TH == 128 && tiles > 256)
    return tiles <= 384 && w.capacity > (tiles <= 320 ? 256 : 1024) * tiles;
  return tiles <= 512 && w.capacity > 64 * tiles;
}
template <int KMAX, int TW, int TH, bool EXACT>
static hipError_t bwd_launch(const Ws &w, const ViewSet &vs, const KCfg &cfg, const float *state,
                             const uint32_t *vals, hipStream_t s) {
  const bool wide = few_tiles<KMAX, TW, TH>(w, vs);
  auto *bwd = wide ? k_raster_bwd<KMAX, TW, TH, true, EXACT> : k_raster_bwd<KMAX, TW, TH, false, EXACT>;
  const int threads = 64 * (wide ? bwd_waves<TW, TH, true>() : bwd_waves<TW, TH, false>());
  hipLaunchKernelGGL(bwd, tile_grid(vs, cfg), dim3(threads), 0, s, w, vs, cfg, state, vals);
  return hipGetLastError();
}

int kmax_for(int K) {
  if (K <= 1) return 1;
  if (K <= 2) return 2;
  if (K <= 4) return 4;
  if (K <= 8) return 8;
  if (K <= 16) return 16;
  return 32;
}

#define HTGS_KX(FN, KM, TW_, TH_, ...)                                          \
  (cfg.K == (KM) ? FN<KM, TW_, TH_, true>(__VA_ARGS__) : FN<KM, TW_, TH_, false>(__VA_ARGS__))
#define HTGS_DISPATCH(FN, ...)                                                   \
  do {                                                                           \
    const int km = kmax_for(cfg.K);                                              \
    if (cfg.tile_w == 8 && cfg.tile_h == 8) {                                    \
      switch (km) {                                                              \
        case 1: return HTGS_KX(FN, 1, 8, 8, __VA_ARGS__);                        \
        case 2: return HTGS_KX(FN, 2, 8, 8, __VA_ARGS__);                        \
        case 4: return HTGS_KX(FN, 4, 8, 8, __VA_ARGS__);                        \
        case 8: return HTGS_KX(FN, 8, 8, 8, __VA_ARGS__);                        \
        case 16: return HTGS_KX(FN, 16, 8, 8, __VA_ARGS__);                      \
        default: return HTGS_KX(FN, 32, 8, 8, __VA_ARGS__);                      \
      }                                                                          \
    } else if (cfg.tile_w == 16 && cfg.tile_h == 8) {                            \
      switch (km) {                                                              \
        case 1: return HTGS_KX(FN, 1, 16, 8, __VA_ARGS__);                       \
        case 2: return HTGS_KX(FN, 2, 16, 8, __VA_ARGS__);                       \
        case 4: return HTGS_KX(FN, 4, 16, 8, __VA_ARGS__);                       \
        case 8: return HTGS_KX(FN, 8, 16, 8, __VA_ARGS__);                       \
        case 16: return HTGS_KX(FN, 16, 16, 8, __VA_ARGS__);                     \
        default: return HTGS_KX(FN, 32, 16, 8, __VA_ARGS__);                     \
      }                                                                          \
    } else if (cfg.tile_w == 32 && cfg.tile_h == 8) {                            \
      switch (km) {                                                              \
        case 1: return HTGS_KX(FN, 1, 32, 8, __VA_ARGS__);                       \
        case 2: return HTGS_KX(FN, 2, 32, 8, __VA_ARGS__);                       \
        case 4: return HTGS_KX(FN, 4, 32, 8, __VA_ARGS__);                       \
        case 8: return HTGS_KX(FN, 8, 32, 8, __VA_ARGS__);                       \
        default: return HTGS_KX(FN, 16, 32, 8, __VA_ARGS__);                     \
      }                                                                          \
    } else {                                                                     \
      switch (km) {                                                              \
        case 1: return HTGS_KX(FN, 1, 16, 16, __VA_ARGS__);                      \
        case 2: return HTGS_KX(FN, 2, 16, 16, __VA_ARGS__);                      \
        case 4: return HTGS_KX(FN, 4, 16, 16, __VA_ARGS__);                      \
        case 8: return HTGS_KX(FN, 8, 16, 16, __VA_ARGS__);                      \
        default: return HTGS_KX(FN, 16, 16, 16, __VA_ARGS__);                    \
      }                                                                          \
    }                                                                            \
  } while (0)

template <int TW, int TH>
static hipError_t fwd_sorted_launch(const Ws &w, const ViewSet &vs, const KCfg &cfg, float *state,
                                    const uint32_t *vals, hipStream_t s) {
  hipLaunchKernelGGL((k_raster_fwd_sorted<TW, TH>), tile_grid(vs, cfg), dim3(TW * TH), 0, s, w, vs, cfg, state, vals);
  return hipGetLastError();
}

hipError_t launch_raster_fwd(const Ws &w, const ViewSet &vs, const KCfg &cfg, float *state,
                             const uint32_t *vals, hipStream_t s) {
  if (cfg.sorted) {
    if (cfg.tile_w == 8 && cfg.tile_h == 8) return fwd_sorted_launch<8, 8>(w, vs, cfg, state, vals, s);
    if (cfg.tile_w == 16 && cfg.tile_h == 8) return fwd_sorted_launch<16, 8>(w, vs, cfg, state, vals, s);
    if (cfg.tile_w == 32 && cfg.tile_h == 8) return fwd_sorted_launch<32, 8>(w, vs, cfg, state, vals, s);
    return fwd_sorted_launch<16, 16>(w, vs, cfg, state, vals, s);
  }
  HTGS_DISPATCH(fwd_launch, w, vs, cfg, state, vals, s);
}

template <int TW, int TH>
static hipError_t bwd_sorted_launch(const Ws &w, const ViewSet &vs, const KCfg &cfg,
                                    const float *state, const uint32_t *vals, hipStream_t s) {
  hipLaunchKernelGGL((k_raster_bwd_sorted<TW, TH>), tile_grid(vs, cfg), dim3(TW * TH), 0, s, w, vs, cfg, state, vals);
  return hipGetLastError();
}

hipError_t launch_raster_bwd(const Ws &w, const ViewSet &vs, const KCfg &cfg, const float *state,
                             const uint32_t *vals, hipStream_t s) {
  if (cfg.sorted) {
    if (cfg.tile_w == 8 && cfg.tile_h == 8) return bwd_sorted_launch<8, 8>(w, vs, cfg, state, vals, s);
    if (cfg.tile_w == 16 && cfg.tile_h == 8) return bwd_sorted_launch<16, 8>(w, vs, cfg, state, vals, s);
    if (cfg.tile_w == 32 && cfg.tile_h == 8) return bwd_sorted_launch<32, 8>(w, vs, cfg, state, vals, s);
    return bwd_sorted_launch<16, 16>(w, vs, cfg, state, vals, s);
  }
  HTGS_DISPATCH(bwd_launch, w, vs, cfg, state, vals, s);
}

}  // namespace htgs
