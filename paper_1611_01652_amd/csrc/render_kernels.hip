// gfx950 kernels of the differentiable camera (paper section 3.4): one ray
// per pixel from a pinhole through the pixel's centre on the projection
// plane, the closest intersection in front of that plane among the env's
// spheres and the ground plane, and a bilinear sample of the object's
// texture; and the reverse of that map for the gradient of sum(w * image)
// with respect to every body's position and rotation.
//
// The ray of pixel (i, j) is C + s d, d = f e_z + u e_x + v e_y with (u, v)
// = ((i + 1/2 - W/2) p, (H/2 - j - 1/2) p), so the projection plane is s = 1.
// A sphere of centre c = p_b + R_b o and radius r is hit at the smallest root
// s >= 1 of |C + s d - c|^2 = r^2; the ground z = 0 at s = -C_z / d_z.  A
// sphere's texel coordinates are ((l_x + 1) (nx - 1) / 2, (l_y + 1) (ny - 1)
// / 2) for its body-frame direction l = R_b^T (h - c) / r, the ground's
// (h_x, h_y) / cell; texel (a, b) sits at integer coordinates, indices wrap.
//
// Reverse of a sphere hit, for the pixel's weight w: the bilinear piece's
// slopes give (u-bar, v-bar); l-bar = (u-bar kx, v-bar ky, 0); R-bar +=
// q l-bar^T / r and q-bar = R l-bar / r for q = h - c; h-bar = q-bar and
// c-bar = -q-bar; the root's derivative in the centre, ds/dc = q / (d . q)
// (implicit differentiation of the sphere equation), adds (d . h-bar) q /
// (d . q) to c-bar; c = p + R o gives p-bar += c-bar, R-bar += c-bar o^T.
// Which object a ray hits is decided on values: silhouettes carry no
// derivative.  The gradient is reduced per env in a fixed order (no float
// atomics), so it is bitwise reproducible.
#include <hip/hip_runtime.h>

#include "sim_internal.h"

namespace sim {

namespace {

struct RHit {
  int k;       // -2 nothing, -1 ground, >= 0 sphere (index within the env)
  float s;     // ray parameter of the hit
};

__device__ __forceinline__ int wrapi(int k, int n) {
  const int m = k % n;
  return m < 0 ? m + n : m;
}

// Texels a and a + 1 (wrapped) of a texture row of n >= 2, in one 8-byte load
// but at the wrap: a wave's texel loads go to up to 64 cache lines each, and
// their number bounds k_render.
struct alignas(4) texel2 { float x, y; };
__device__ __forceinline__ void texel_pair(const float* row, int a, int n, float* t0, float* t1) {
  const int am = a < n - 1 ? a : n - 2;
  const texel2 p = *reinterpret_cast<const texel2*>(row + am);
  *t0 = p.x;
  *t1 = p.y;
  if (am != a) {
    *t0 = p.y;
    *t1 = row[0];
  }
}

// bilinear sample and its slopes in the texel coordinates
__device__ __forceinline__ float bilinear(const float* T, int nx, int ny, float u, float v, float* du, float* dv) {
  const float fu0 = floorf(u), fv0 = floorf(v);
  const float fu = u - fu0, fv = v - fv0;
  const int a0 = wrapi((int)fu0, nx);
  const int b0 = wrapi((int)fv0, ny), b1 = wrapi((int)fv0 + 1, ny);
  float t00, t10, t01, t11;
  texel_pair(T + b0 * nx, a0, nx, &t00, &t10);
  texel_pair(T + b1 * nx, a0, nx, &t01, &t11);
  if (du) *du = (1.f - fv) * (t10 - t00) + fv * (t11 - t01);
  if (dv) *dv = (1.f - fu) * (t01 - t00) + fu * (t11 - t10);
  return (1.f - fu) * (1.f - fv) * t00 + fu * (1.f - fv) * t10 + (1.f - fu) * fv * t01 + fu * fv * t11;
}

// an integral double's index in [0, n).  Below 2^50 the quotient by a rounded
// reciprocal is off by at most one, and the remainder is formed exactly (one
// fused step, a result below 2 n in size); beyond, fmod is exact at any
// magnitude (its loop per bit of the quotient was a third of k_render).
__device__ __forceinline__ int wrapd(double k, int n, double inv_n) {
  double m;
  if (fabs(k) < 1125899906842624.0) {
    m = __builtin_fma(-floor(k * inv_n), (double)n, k);
    if (m >= (double)n) m -= (double)n;
  } else {
    m = fmod(k, (double)n);
  }
  if (m < 0.0) m += (double)n;
  const int r = (int)m;
  return r >= n ? 0 : r;
}

// reciprocals of the ground's cell and texel counts, formed once per thread
struct RenderInv { double cell, gnx, gny; };

// the ground's bilinear sample at FP64 texel coordinates (far from the
// camera they reach hundreds of texels): the floor and the fractions in FP64,
// the interpolation in FP32
__device__ __forceinline__ float ground_sample(const RenderTex& tex, const RenderInv& inv, double u, double v) {
  const double fu0 = floor(u), fv0 = floor(v);
  const float fu = (float)(u - fu0), fv = (float)(v - fv0);
  const int a0 = wrapd(fu0, tex.gnx, inv.gnx);
  const int b0 = wrapd(fv0, tex.gny, inv.gny), b1 = b0 + 1 == tex.gny ? 0 : b0 + 1;
  float t00, t10, t01, t11;
  texel_pair(tex.ground + b0 * tex.gnx, a0, tex.gnx, &t00, &t10);
  texel_pair(tex.ground + b1 * tex.gnx, a0, tex.gnx, &t01, &t11);
  return (1.f - fu) * (1.f - fv) * t00 + fu * (1.f - fv) * t10 + (1.f - fu) * fv * t01 + fu * fv * t11;
}

// The ray's direction is set up in FP64 and kept in both precisions: near the
// horizon the ground's hit point moves by s / |d_z| times any rounding of
// d_z, so the ground is intersected in FP64 (a few operations per pixel);
// the spheres take the direction rounded to FP32.
struct Ray {
  float c[3], d[3];
  double d64[3];
};

__device__ __forceinline__ Ray pixel_ray(const RenderCam& cam, int i, int j) {
  const double u = ((double)i + 0.5 - 0.5 * (double)cam.width) * (double)cam.pitch;
  const double v = (0.5 * (double)cam.height - (double)j - 0.5) * (double)cam.pitch;
  Ray r;
  for (int k = 0; k < 3; ++k) {
    r.c[k] = cam.pos[k];
    r.d64[k] = (double)cam.focal * (double)cam.axes[6 + k] + u * (double)cam.axes[k] + v * (double)cam.axes[3 + k];
    r.d[k] = (float)r.d64[k];
  }
  return r;
}

// the ground's hit parameter (FP64), or a negative value when the ray is
// parallel to the ground
__device__ __forceinline__ double ground_s(const Ray& ray) {
  return ray.d64[2] != 0.0 ? -(double)ray.c[2] / ray.d64[2] : -1.0;
}

// sphere k's centre from its body's state (x: [18][B], component-major)
__device__ __forceinline__ void sphere_centre(const float* x, int B, int b, const float* o, float* c) {
  for (int r = 0; r < 3; ++r)
    c[r] = x[r * B + b] + x[(3 + 3 * r) * B + b] * o[0] + x[(4 + 3 * r) * B + b] * o[1] +
           x[(5 + 3 * r) * B + b] * o[2];
}

// Spheres [g0, g1) of env order staged in LDS: centre p + R o and radius,
// one float4 each, made once per workgroup instead of once per pixel.
__device__ __forceinline__ void stage_spheres(const RenderScene& sc, const float* x, int g0, int g1, float4* cs) {
  for (int g = g0 + (int)threadIdx.x; g < g1; g += (int)blockDim.x) {
    const float4 so = sc.sph[g];
    const float o[3] = {so.x, so.y, so.z};
    float c[3];
    sphere_centre(x, sc.B, sc.sph_body[g], o, c);
    cs[g - g0] = make_float4(c[0], c[1], c[2], so.w);
  }
}

// The roots of |m + s d|^2 = r^2 (m = C - c) are s = t0 -/+ sqrt(D) with t0 =
// -(d . m) / a and D = (r^2 - |m + t0 d|^2) / a, a = |d|^2: the distance of
// the ray from the centre, m + t0 d, is formed first, so D does not come
// from the difference of two terms of the size |m|^2 |d|^2 (which loses
// every digit of a small D in FP32).  Both quotients by a use one
// reciprocal of a per pixel (ia).  Of the staged spheres those in the mask
// (the same in every lane) are tested, in env order (index k0 + bit); the
// first of equal nearest roots is kept.
__device__ __forceinline__ void trace_spheres(const float4* cs, unsigned long long mask, int k0, const Ray& ray,
                                              float ia, RHit& h) {
  for (; mask; mask &= mask - 1) {
    const int k = __ffsll(mask) - 1;
    const float4 cc = cs[k];
    const float m0 = ray.c[0] - cc.x, m1 = ray.c[1] - cc.y, m2 = ray.c[2] - cc.z;
    const float t0 = -(ray.d[0] * m0 + ray.d[1] * m1 + ray.d[2] * m2) * ia;
    const float p0 = m0 + t0 * ray.d[0], p1 = m1 + t0 * ray.d[1], p2 = m2 + t0 * ray.d[2];
    const float D = (cc.w * cc.w - (p0 * p0 + p1 * p1 + p2 * p2)) * ia;
    if (D < 0.f) continue;
    const float sq = sqrtf(D);
    const float s = t0 - sq >= 1.f ? t0 - sq : t0 + sq;
    if (s >= 1.f && s < h.s) { h.s = s; h.k = k0 + k; }
  }
}

// A wave's pixels: tiles of w() x h() = 64, lane l at column l % w(), row
// l / w().  16 x 4 (64-byte runs of an image row), a constant of the kernel, but
// for frames that fill those badly: the shape is then the frame's (tile_shape).
// Few of an env's spheres are in sight of so small a tile, so a wave first
// tests the staged spheres against the tile, one per lane, and traces only
// those left.
constexpr int kTileLg = 4;   // log2 of the usual tile's width
template <int LG>            // log2 of the tile's width; -1: the launch's choice
struct Tiles {
  int chosen;
  __host__ __device__ __forceinline__ int lg() const { return LG >= 0 ? LG : chosen; }
  __host__ __device__ __forceinline__ int w() const { return 1 << lg(); }
  __host__ __device__ __forceinline__ int h() const { return 64 >> lg(); }
  __host__ __device__ __forceinline__ int across(const RenderCam& cam) const { return (cam.width + w() - 1) >> lg(); }
  __host__ __device__ __forceinline__ int count(const RenderCam& cam) const {
    return across(cam) * ((cam.height + h() - 1) >> (6 - lg()));
  }
};
// Every ray of the tile has |d - dc| <= rho for the tile's centre ray dc and
// rho = half the pixel span along u and v (the triangle inequality: nothing
// is asked of the axes), so a hit at some s >= 1 needs |s dc - m| <= r + s rho
// for m = c - C: f(s) = A s^2 - 2 q s + g <= 0 with A = |dc|^2 - rho^2, q =
// dc . m + r rho, g = |m|^2 - r^2.  A sphere is left out when f has no root,
// or none that is positive, by margins (1e-5 of the terms) far above the FP32
// rounding here and in trace_spheres; anything not finite is kept.
template <int LG>
__device__ __forceinline__ bool sphere_in_tile(const float4 cc, const RenderCam& cam, Tiles<LG> tiles, int i0, int j0) {
  const float u = (((float)i0 + 0.5f * (float)tiles.w()) - 0.5f * (float)cam.width) * cam.pitch;
  const float v = (0.5f * (float)cam.height - ((float)j0 + 0.5f * (float)tiles.h())) * cam.pitch;
  float ex = 0.f, ey = 0.f, a = 0.f, b = 0.f, m2 = 0.f;
  const float c[3] = {cc.x, cc.y, cc.z};
  for (int k = 0; k < 3; ++k) {
    const float d = cam.focal * cam.axes[6 + k] + u * cam.axes[k] + v * cam.axes[3 + k], m = c[k] - cam.pos[k];
    ex += cam.axes[k] * cam.axes[k];
    ey += cam.axes[3 + k] * cam.axes[3 + k];
    a += d * d;
    b += d * m;
    m2 += m * m;
  }
  const float rho = 0.5005f * cam.pitch * ((float)tiles.w() * sqrtf(ex) + (float)tiles.h() * sqrtf(ey));
  const float A = a - rho * rho, q = b + cc.w * rho, g = m2 - cc.w * cc.w;
  const float disc = q * q - A * g;
  return !(A > 1e-3f * a && (disc < -1e-5f * (q * q + fabsf(A * g)) || (q < 0.f && g > 1e-5f * m2)));
}
// The staged spheres to trace in one tile, a lane each ...
template <int LG>
__device__ __forceinline__ unsigned long long tile_spheres(const float4* cs, int n, const RenderCam& cam,
                                                           Tiles<LG> tiles, int i0, int j0, int lane) {
  return __ballot(lane < n && sphere_in_tile(cs[lane], cam, tiles, i0, j0));
}
// ... or, of at most 16 spheres, in the four tiles tile, tile + step, ..: 16
// bits each.  (A test is 60 instructions, most of what a tile without spheres
// costs the gradient: 65 -> 51 us for 512 images.  The image, where every
// tile has the ground, got slower with it: 98 -> 111 us.)
template <int LG>
__device__ __forceinline__ unsigned long long tile_spheres_x4(const float4* cs, int n, const RenderCam& cam,
                                                              Tiles<LG> tiles, int tile, int step, int tx, int lane) {
  const int k = lane & 15, t = tile + (lane >> 4) * step;
  return __ballot(k < n && sphere_in_tile(cs[k], cam, tiles, t % tx * tiles.w(), t / tx * tiles.h()));
}

__device__ __forceinline__ void trace_ground(const RenderScene& sc, const Ray& ray, RHit& h) {
  if (sc.ground) {
    const double s = ground_s(ray);
    if (s >= 1.0 && s < (double)h.s) { h.s = (float)s; h.k = -1; }
  }
}

// 1 / |d|^2 of the ray
__device__ __forceinline__ float ray_ia(const Ray& ray) {
  return 1.f / (ray.d[0] * ray.d[0] + ray.d[1] * ray.d[1] + ray.d[2] * ray.d[2]);
}

// The colour of a ray: the nearest of its sphere hit and the ground.
__device__ __forceinline__ float pixel_colour(const RenderScene& sc, const float* x, const Ray& ray,
                                              const RenderTex& tex, const RenderInv& inv, int s0, RHit h) {
  trace_ground(sc, ray, h);
  if (h.k == -1) {
    const double sg = ground_s(ray);
    const double gu = ((double)ray.c[0] + sg * ray.d64[0]) * inv.cell;
    const double gv = ((double)ray.c[1] + sg * ray.d64[1]) * inv.cell;
    return ground_sample(tex, inv, gu, gv);
  }
  if (h.k < 0) return 0.f;
  const int g = s0 + h.k, b = sc.sph_body[g];
  const float4 so = sc.sph[g];
  const float o[3] = {so.x, so.y, so.z};
  float c[3], q[3];
  sphere_centre(x, sc.B, b, o, c);
  for (int k = 0; k < 3; ++k) q[k] = ray.c[k] + h.s * ray.d[k] - c[k];
  // l = R^T q / r (R row-major at x[3 + 3 r + i])
  const float lx = (x[3 * sc.B + b] * q[0] + x[6 * sc.B + b] * q[1] + x[9 * sc.B + b] * q[2]) / so.w;
  const float ly = (x[4 * sc.B + b] * q[0] + x[7 * sc.B + b] * q[1] + x[10 * sc.B + b] * q[2]) / so.w;
  return bilinear(tex.sphere, tex.snx, tex.sny, (lx + 1.f) * (0.5f * (float)(tex.snx - 1)),
                  (ly + 1.f) * (0.5f * (float)(tex.sny - 1)), nullptr, nullptr);
}

constexpr int kStage = 64;    // spheres staged in LDS at a time by k_render
constexpr int kTilesPerWave = 8;

// One pixel per lane; a workgroup of four waves takes 4 kTilesPerWave tiles
// of one env.  An env's spheres are staged once per workgroup (kStage at a
// time, again for each tile, where it has more).  Bound by instruction issue
// (the ground's FP64 intersection the largest part) and the texel loads.  512
// images of 288 x 96 over chains of 2..16 spheres: 98 us, 57 MB written; with
// every sphere tested per pixel, fmod and four texel loads 153 us.
template <int LG>
__global__ __launch_bounds__(256) void k_render(RenderScene sc, const float* x, RenderCam cam, Tiles<LG> tiles,
                                                RenderTex tex, float* image) {
  __shared__ float4 cs[kStage];
  const int e = blockIdx.y, lane = threadIdx.x & 63;
  const int n = cam.width * cam.height, tx = tiles.across(cam), nt = tiles.count(cam);
  const int s0 = sc.env_sph[e], s1 = sc.env_sph[e + 1];
  const RenderInv inv{1.0 / (double)tex.cell, 1.0 / (double)tex.gnx, 1.0 / (double)tex.gny};
  for (int q = 0; q < kTilesPerWave; ++q) {
    const int tile = (blockIdx.x * kTilesPerWave + q) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = tile % tx * tiles.w(), j0 = tile / tx * tiles.h();
    const int i = i0 + (lane & (tiles.w() - 1)), j = j0 + (lane >> tiles.lg());
    const Ray ray = pixel_ray(cam, i, j);
    RHit h{-2, INFINITY};
    for (int g0 = s0; g0 < s1; g0 += kStage) {
      const int g1 = g0 + kStage < s1 ? g0 + kStage : s1;
      if (q == 0 || s1 - s0 > kStage) {
        __syncthreads();
        stage_spheres(sc, x, g0, g1, cs);
        __syncthreads();
      }
      const unsigned long long mask = tile_spheres(cs, g1 - g0, cam, tiles, i0, j0, lane);
      if (mask) trace_spheres(cs, mask, g0 - s0, ray, ray_ia(ray), h);
    }
    if (tile < nt && i < cam.width && j < cam.height)
      image[(size_t)e * n + (size_t)j * cam.width + i] = pixel_colour(sc, x, ray, tex, inv, s0, h);
  }
}

// Sum over the wave's 64 lanes in a fixed order, valid in lane 63 (adds
// along rows of 16 lanes, then across the rows, without LDS).
__device__ __forceinline__ float wave_sum63(float v) {
#define SIM_ADD_DPP(ctrl, rows) \
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xf, true))
  SIM_ADD_DPP(0x111, 0xf);   // row_shr:1, 2, 4, 8
  SIM_ADD_DPP(0x112, 0xf);
  SIM_ADD_DPP(0x114, 0xf);
  SIM_ADD_DPP(0x118, 0xf);
  SIM_ADD_DPP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
  SIM_ADD_DPP(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef SIM_ADD_DPP
  return v;
}

constexpr int kGradWaves = 16;
static_assert(kRenderMaxSpheres <= 16, "a tile's mask is 16 bits");
constexpr int kGradThreads = 64 * kGradWaves;

// One workgroup of 16 waves per env (512 images of 288 x 96: 51 us; with four
// waves, each waiting for its own loads, every pixel traced and the sums by
// LDS butterflies 310 us).  Wave v takes every
// 16th tile from the v-th; a tile with no sphere in sight is done at once,
// its weights unread.  A lane whose pixel shows sphere k forms that pixel's
// 12 terms (the body's position 3, rotation 9); then, for each sphere that
// some lane of the wave shows (in the order of the lowest such lane), the
// wave adds those lanes' terms in a fixed order and lane 63 adds the sums to
// the wave's row for that sphere in LDS.  At the end the waves' rows are
// added in wave order and each sphere's sums go to its body, spheres in env
// order.  Every sum runs in an order fixed by the inputs, so the gradient is
// bitwise reproducible.
template <int LG>
__global__ __launch_bounds__(kGradThreads) void k_render_grad(RenderScene sc, const float* x, RenderCam cam,
                                                              Tiles<LG> tiles, RenderTex tex, const float* w,
                                                              float* g_x) {
  __shared__ float4 cs[kRenderMaxSpheres];
  __shared__ float rot[kRenderMaxSpheres][12];   // body rotation 9, sphere offset 3
  __shared__ float acc[kGradWaves][kRenderMaxSpheres][12];
  __shared__ float tot[kRenderMaxSpheres][12];
  const int e = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = cam.width * cam.height, tx = tiles.across(cam), nt = tiles.count(cam);
  const int s0 = sc.env_sph[e], ns = sc.env_sph[e + 1] - s0;
  for (int u = t; u < kGradWaves * kRenderMaxSpheres * 12; u += kGradThreads) (&acc[0][0][0])[u] = 0.f;
  stage_spheres(sc, x, s0, s0 + ns, cs);
  for (int u = t; u < ns * 12; u += kGradThreads) {
    const int k = u / 12, c = u % 12;
    rot[k][c] = c < 9 ? x[(size_t)(3 + c) * sc.B + sc.sph_body[s0 + k]]
                      : reinterpret_cast<const float*>(&sc.sph[s0 + k])[c - 9];
  }
  __syncthreads();
  const float kx = 0.5f * (float)(tex.snx - 1), ky = 0.5f * (float)(tex.sny - 1);
  unsigned long long four = 0;
  for (int tile = wv, q = 0; tile < nt; tile += kGradWaves, ++q) {
    if (q % 4 == 0) four = tile_spheres_x4(cs, ns, cam, tiles, tile, kGradWaves, tx, lane);
    const unsigned long long mask = four >> (16 * (q % 4)) & 0xffffull;
    if (mask == 0) continue;
    const int i0 = tile % tx * tiles.w(), j0 = tile / tx * tiles.h();
    const int i = i0 + (lane & (tiles.w() - 1)), j = j0 + (lane >> tiles.lg());
    int hk = -1;
    float v[12];
    for (int c = 0; c < 12; ++c) v[c] = 0.f;
    const float wt = i < cam.width && j < cam.height ? w[(size_t)e * n + (size_t)j * cam.width + i] : 0.f;
    if (wt != 0.f) {
      const Ray ray = pixel_ray(cam, i, j);
      RHit h{-2, INFINITY};
      trace_spheres(cs, mask, 0, ray, ray_ia(ray), h);
      if (h.k >= 0) trace_ground(sc, ray, h);
      // the ground and the background do not depend on the state
      if (h.k >= 0) {
        hk = h.k;
        const float4 cc = cs[h.k];
        const float c[3] = {cc.x, cc.y, cc.z};
        const float r = cc.w;
        float q[3], R[9], o[3];
        for (int k = 0; k < 9; ++k) R[k] = rot[h.k][k];
        for (int k = 0; k < 3; ++k) o[k] = rot[h.k][9 + k];
        for (int k = 0; k < 3; ++k) q[k] = ray.c[k] + h.s * ray.d[k] - c[k];
        const float lx = (R[0] * q[0] + R[3] * q[1] + R[6] * q[2]) / r;
        const float ly = (R[1] * q[0] + R[4] * q[1] + R[7] * q[2]) / r;
        float du, dv;
        (void)bilinear(tex.sphere, tex.snx, tex.sny, (lx + 1.f) * kx, (ly + 1.f) * ky, &du, &dv);
        const float lbx = wt * du * kx, lby = wt * dv * ky;
        // R-bar_{k i} = q_k l-bar_i / r (i = x, y); q-bar_k = (R_k0 l-bar_x + R_k1 l-bar_y) / r
        float qb[3];
        for (int k = 0; k < 3; ++k) {
          v[3 + 3 * k] = q[k] * lbx / r;
          v[4 + 3 * k] = q[k] * lby / r;
          qb[k] = (R[3 * k] * lbx + R[3 * k + 1] * lby) / r;
        }
        // h-bar = q-bar, c-bar = -q-bar + (d . h-bar) q / (d . q)
        const float dh = ray.d[0] * qb[0] + ray.d[1] * qb[1] + ray.d[2] * qb[2];
        const float dq = ray.d[0] * q[0] + ray.d[1] * q[1] + ray.d[2] * q[2];
        float cb[3];
        for (int k = 0; k < 3; ++k) cb[k] = -qb[k] + dh * q[k] / dq;
        // c = p + R o
        for (int k = 0; k < 3; ++k) {
          v[k] = cb[k];
          for (int m = 0; m < 3; ++m) v[3 + 3 * k + m] += cb[k] * o[m];
        }
      }
    }
    // (wave-uniform: the ballots are the same in every lane)
    unsigned long long todo = __ballot(hk >= 0);
    while (todo) {
      const int kk = __shfl(hk, __ffsll(todo) - 1);
      const bool mine = hk == kk;
      float r[12];
      for (int c = 0; c < 12; ++c) r[c] = mine ? v[c] : 0.f;
      for (int c = 0; c < 12; ++c) r[c] = wave_sum63(r[c]);
      if (lane == 63)
        for (int c = 0; c < 12; ++c) acc[wv][kk][c] += r[c];
      todo &= ~__ballot(mine);
    }
  }
  __syncthreads();
  for (int u = t; u < ns * 12; u += kGradThreads) {
    const int k = u / 12, c = u % 12;
    float s = acc[0][k][c];
    for (int q = 1; q < kGradWaves; ++q) s += acc[q][k][c];
    tot[k][c] = s;
  }
  __syncthreads();
  // the env's bodies: each sphere's sums added to its body in sphere order
  // (one thread per value)
  const int b0 = sc.env_body[e], b1 = sc.env_body[e + 1];
  for (int u = t; u < (b1 - b0) * 18; u += kGradThreads) {
    const int b = b0 + u / 18, c = u % 18;
    float s = 0.f;
    if (c < 12)
      for (int k = 0; k < ns; ++k)
        if (sc.sph_body[s0 + k] == b) s += tot[k][c];
    g_x[(size_t)c * sc.B + b] = s;
  }
}

// log2 of the width of the frame's tiles: 16, unless another width needs less
// than two thirds of the tiles, then the one that needs the fewest, the nearest
// to 16 of equal ones.  Frames one or a few pixels wide or high leave most
// lanes of a 16 x 4 tile idle (512 images and their gradient, 16 x 4 -> chosen:
// 1 x 2048 pixels 110 -> 44 us, 2048 x 1 73 -> 49 us).  As a constant of the
// kernels the 16 x 4 shape is 1 to 2 % faster than as an argument, so the usual
// frames have kernels of their own.
int tile_shape(const RenderCam& cam) {
  const long long whole = Tiles<kTileLg>{}.count(cam);
  long long least = whole;
  int lg = kTileLg;
  for (int k : {3, 5, 2, 6, 1, 0}) {
    const long long n = Tiles<-1>{k}.count(cam);
    if (3 * n < 2 * whole && n < least) {
      least = n;
      lg = k;
    }
  }
  return lg;
}

template <int LG>
void render_frame(const RenderScene& sc, const float* x, const RenderCam& cam, Tiles<LG> tiles, const RenderTex& tex,
                  float* image, hipStream_t st) {
  const dim3 grid((tiles.count(cam) + 4 * kTilesPerWave - 1) / (4 * kTilesPerWave), sc.E);
  hipLaunchKernelGGL(k_render<LG>, grid, dim3(256), 0, st, sc, x, cam, tiles, tex, image);
}

}  // namespace

hipError_t launch_render(const RenderScene& sc, const float* x, const RenderCam& cam, const RenderTex& tex,
                         float* image, hipStream_t st) {
  const int n = cam.width * cam.height;
  if (sc.E == 0 || n == 0) return hipSuccess;
  const int lg = tile_shape(cam);
  if (lg == kTileLg) render_frame(sc, x, cam, Tiles<kTileLg>{lg}, tex, image, st);
  else render_frame(sc, x, cam, Tiles<-1>{lg}, tex, image, st);
  return hipGetLastError();
}

hipError_t launch_render_grad(const RenderScene& sc, const float* x, const RenderCam& cam, const RenderTex& tex,
                              const float* w, float* g_x, hipStream_t st) {
  if (sc.E == 0) return hipSuccess;
  const int lg = tile_shape(cam);
  if (lg == kTileLg)
    hipLaunchKernelGGL(k_render_grad<kTileLg>, dim3(sc.E), dim3(kGradThreads), 0, st, sc, x, cam, Tiles<kTileLg>{lg},
                       tex, w, g_x);
  else
    hipLaunchKernelGGL(k_render_grad<-1>, dim3(sc.E), dim3(kGradThreads), 0, st, sc, x, cam, Tiles<-1>{lg}, tex, w,
                       g_x);
  return hipGetLastError();
}

}  // namespace sim
