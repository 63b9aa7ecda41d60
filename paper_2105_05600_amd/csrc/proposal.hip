// Inputs of the learned PST proposal: a low-resolution raycast of the TSDF
// at the previous pose and the depth residual against the current frame.
#include <algorithm>

#include "common.h"

namespace rose {

// trilinear psi at voxel-space point h = g - 1/2 (binary64; +1 when any of
// the 8 corners is outside the grid)
template <int FMT>
__device__ inline double trilinear64(const Grid& g, double hx, double hy, double hz) {
    const double h[3] = {hx, hy, hz};
    const int32_t n[3] = {g.nx, g.ny, g.nz};
    int64_t i0[3];
    double f[3];
    for (int c = 0; c < 3; ++c) {
        if (!(h[c] >= 0.0 && h[c] < (double)(n[c] - 1))) return 1.0;
        i0[c] = (int64_t)floor(h[c]);
        if (i0[c] + 1 >= n[c]) return 1.0;
        f[c] = h[c] - (double)i0[c];
    }
    double acc = 0.0;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const double w = (dx ? f[0] : 1.0 - f[0]) * (dy ? f[1] : 1.0 - f[1]) * (dz ? f[2] : 1.0 - f[2]);
                const uint32_t off =
                    brick_offset(g, (uint32_t)(i0[0] + dx), (uint32_t)(i0[1] + dy), (uint32_t)(i0[2] + dz));
                acc += w * (double)load_psi<FMT>(g.psi, off);
            }
    return acc;
}

struct RaycastArgs {
    Grid g;
    double R[9];
    double t[3];
    int32_t W, H;
    double fx, fy, cx, cy;
    double near_z, far_z, step;
    double inv_vox, kmax;  // 1 / vox; (far - near) / step + 2
    float* out;
};

// The point of a ray at depth z in voxels, and the value there, as a serial
// march computes them.
__device__ inline void ray_point(const RaycastArgs& a, const double dw[3], double z, double h[3]) {
    const double vox = (double)a.g.vox;
    for (int c = 0; c < 3; ++c) h[c] = (a.t[c] + z * dw[c] - (double)a.g.origin[c]) / vox - 0.5;
}

template <int FMT>
__device__ inline double ray_sample(const RaycastArgs& a, const double dw[3], double z) {
    double h[3];
    ray_point(a, dw, z, h);
    return trilinear64<FMT>(a.g, h[0], h[1], h[2]);
}

// What a sample of a ray can be.  Outside the grid it is +1; inside it is <= 0
// only if a corner is, and > 0 only if a corner is (the interpolation weights
// are >= 0 and not all 0; with a NaN corner it is NaN).  The voxel coordinates
// are i0 + f with the voxel i0 of a stretch's first sample and f = f0 + d b in
// binary32 (d below 128, |b| at most 8 voxels: within 1e-4 of ray_sample's),
// and ray_sample's own where those are so close to a voxel or grid boundary
// that the corners are not certain (every second sample of a camera along an
// axis with a half-voxel step: evaluating them cost 0.38 ms against 0.29 for
// evaluating all samples, 320 x 240 in 256^3 of free space).  Loads are
// unconditional (voxel 0 for the lanes that do not need theirs), so that
// those of several samples are in flight together.
struct RayTest {
    int v[8];  // the corners' signs: > 0 or <= 0 as the value (a NaN's by its sign bit)
    bool outside;
};

// sign of a voxel from its bits
__device__ inline int sign_of(uint32_t bits) { return (int)bits; }
__device__ inline int sign_of(unsigned short bits) { return (int16_t)bits; }

template <int FMT>
__device__ inline int load_sign(const void* psi, uint32_t off) {
    if constexpr (FMT == ROSE_TSDF_F32) return sign_of(((const uint32_t*)psi)[off]);
    else return sign_of(((const unsigned short*)psi)[off]);
}

template <int FMT, bool WIDE>
__device__ inline void ray_test_load(const RaycastArgs& a, __amdgpu_buffer_rsrc_t psi, const int i0[3],
                                     const float f0[3], const float fb[3], float d, const double dw[3], int k,
                                     RayTest& t) {
    constexpr float kEps = 1e-4f;
    const Grid& g = a.g;
    const int32_t n[3] = {g.nx, g.ny, g.nz};
    uint32_t i[3];
    bool unsure = false;
    t.outside = false;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float f = fmaf(d, fb[c], f0[c]), fl = floorf(f), fr = f - fl;
        const int h = i0[c] + (int)fl;
        const bool in = (uint32_t)h < (uint32_t)(n[c] - 1);
        t.outside = t.outside || !in;
        unsure = unsure || fr < kEps || fr > 1.0f - kEps;
        i[c] = in ? (uint32_t)h : 0u;
    }
    if (unsure) {
        double h[3];
        ray_point(a, dw, a.near_z + (double)k * a.step, h);
        t.outside = false;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bool in = h[c] >= 0.0 && h[c] < (double)(n[c] - 1);
            t.outside = t.outside || !in;
            i[c] = in ? (uint32_t)h[c] : 0u;
        }
    }
    const uint32_t x[2] = {(i[0] & ~7u) * 63u + i[0], ((i[0] + 1) & ~7u) * 63u + i[0] + 1};
    const uint32_t y[2] = {__umul24(i[1] & ~7u, (uint32_t)g.bstride_y) + 8 * i[1],
                           __umul24((i[1] + 1) & ~7u, (uint32_t)g.bstride_y) + 8 * (i[1] + 1)};
    const uint32_t z[2] = {__umul24(i[2] & ~7u, (uint32_t)g.bstride_z) + 64 * i[2],
                           __umul24((i[2] + 1) & ~7u, (uint32_t)g.bstride_z) + 64 * (i[2] + 1)};
    if constexpr (WIDE) {
#pragma unroll
        for (int e = 0; e < 8; ++e) t.v[e] = load_sign<FMT>(g.psi, x[e & 1] + y[(e >> 1) & 1] + z[e >> 2]);
        return;
    }
    // the two x neighbours of a corner row in one load, except across a brick
    // boundary (the lanes with i mod 8 = 7 load the second apart): gathers
    // are what the march waits for
    const bool split = (i[0] & 7u) == 7u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t off = x[0] + y[e & 1] + z[e >> 1];
        if constexpr (FMT == ROSE_TSDF_F32) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(psi, (int)(4u * off), 0, 0);
            t.v[2 * e] = sign_of(w[0]);
            t.v[2 * e + 1] = sign_of(w[1]);
        } else {  // the 4 values from the 4-byte boundary at or below
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(psi, (int)(2u * (off & ~1u)), 0, 0);
            const uint32_t pair = __builtin_amdgcn_alignbit(w[1], w[0], 16u * (off & 1u));
            t.v[2 * e] = sign_of((unsigned short)pair);
            t.v[2 * e + 1] = sign_of((unsigned short)(pair >> 16));
        }
    }
    if (split) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t off = x[1] + y[e & 1] + z[e >> 1];
            if constexpr (FMT == ROSE_TSDF_F32)
                t.v[2 * e + 1] = sign_of((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(psi, (int)(4u * off), 0, 0));
            else
                t.v[2 * e + 1] = sign_of((unsigned short)__builtin_amdgcn_raw_buffer_load_b16(psi, (int)(2u * off), 0, 0));
        }
    }
}

// whether the sample may be > 0 (POS) or <= 0
template <bool POS>
__device__ inline bool ray_may_be(const RayTest& t) {
    int m = t.v[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) m = POS ? max(m, t.v[e]) : min(m, t.v[e]);
    return !t.outside && (POS ? m > 0 : m <= 0);
}

// The fixed-step march of the rays: a wavefront takes a TP x TP patch of
// pixels and NS = 64 / TP^2 consecutive samples of each (z = near + k step,
// the same expression as a serial march, so the samples are identical), U
// such groups in flight together.  A crossing at k is a + to - change
// between samples k-1 and k inside the truncation band, so only a sample
// that may be <= 0 after one that may be > 0 needs a value, and that one
// with it: ray_may_be tells the others (free space, and the inside of solids,
// the bulk of every ray).  The first crossing in step order gives the depth
// by linear interpolation, exactly as a serial march stopping there would.
// Bound by the gathers' cache-line lookups (8 corners per sample in 4 loads;
// with one load per corner 258 us at 320 x 240, whatever the arithmetic
// around them).
template <int FMT, bool WIDE, int TP, int U>
__global__ __launch_bounds__(256) void k_raycast(RaycastArgs a) {
    constexpr int NS = kWave / (TP * TP);
    const int lane = threadIdx.x & 63, px = lane / NS, j = lane % NS;
    const int tiles_x = (a.W + TP - 1) / TP, tiles_y = (a.H + TP - 1) / TP;
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= tiles_x * tiles_y) return;  // whole wavefronts leave together
    const int u = (tile % tiles_x) * TP + px % TP, v = (tile / tiles_x) * TP + px / TP;
    const double dc[3] = {((double)u - a.cx) / a.fx, ((double)v - a.cy) / a.fy, 1.0};
    double dw[3];
    for (int i = 0; i < 3; ++i) dw[i] = a.R[3 * i + 0] * dc[0] + a.R[3 * i + 1] * dc[1] + a.R[3 * i + 2] * dc[2];
    const uint32_t bytes = (uint32_t)a.g.nx * (uint32_t)a.g.ny * (uint32_t)a.g.nz * (FMT == ROSE_TSDF_F32 ? 4u : 2u);
    const __amdgpu_buffer_rsrc_t psi = __builtin_amdgcn_make_buffer_rsrc(a.g.psi, (short)0, (int)bytes, 0x00020000);
    // voxel coordinates ha + k hb; where they are too large or too far apart
    // for RayTest's margin, every sample is evaluated
    double ha[3], hb[3];
    float fb[3];
    bool plain = false;
    const double inv = a.inv_vox, kmax = a.kmax;
    for (int c = 0; c < 3; ++c) {
        ha[c] = (a.t[c] + a.near_z * dw[c] - (double)a.g.origin[c]) * inv - 0.5;
        hb[c] = a.step * dw[c] * inv;
        fb[c] = (float)hb[c];
        plain = plain || !((fabs(a.t[c]) + fabs((double)a.g.origin[c])) * inv + kmax * fabs(hb[c]) +
                               fabs(a.near_z * dw[c]) * inv < 1e8) || !(fabs(hb[c]) <= 8.0);
    }
    // samples before the ray enters the grid and after it leaves it are +1
    // (the reciprocal's rounding is far below the margins of 1e-3 voxels and
    // 2 samples)
    double k0 = 0.0, k1 = kmax;
    if (!plain) {
        const int32_t n[3] = {a.g.nx, a.g.ny, a.g.nz};
        for (int c = 0; c < 3; ++c) {
            const double ib = 1.0 / hb[c];
            const double e0 = (-1e-3 - ha[c]) * ib, e1 = ((double)(n[c] - 1) + 1e-3 - ha[c]) * ib;
            if (hb[c] > 0.0) {
                k0 = fmax(k0, e0);
                k1 = fmin(k1, e1);
            } else if (hb[c] < 0.0) {
                k0 = fmax(k0, e1);
                k1 = fmin(k1, e0);
            }
        }
    }
    const int kend = (int)fmin(fmax(k1 + 2.0, 0.0), kmax);
    int base = (int)fmin(fmax(k0 - 2.0, 0.0), kmax);
    double out = 0.0;
    bool done = u >= a.W || v >= a.H || base > kend;
    // lanes that hold a pixel's first sample of a group
    constexpr uint64_t kFirst = NS == 64 ? 1ull : NS == 16 ? 0x0001000100010001ull : 0x1111111111111111ull;
    uint64_t carry = kFirst;  // of these, the ones whose sample before may be > 0
    for (; !done; base += U * NS, done = done || base > kend) {
        int i0[3];
        float f0[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double h = fma((double)base, hb[c], ha[c]), fl = floor(fmin(fmax(h, -1e8), 1e8));
            i0[c] = (int)fl;
            f0[c] = (float)(h - fl);
        }
        RayTest t[U];
#pragma unroll
        for (int q = 0; q < U; ++q)
            ray_test_load<FMT, WIDE>(a, psi, i0, f0, fb, (float)(q * NS + j), dw, base + q * NS + j, t[q]);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (done) break;
            const int k = base + q * NS + j;
            const double z = a.near_z + (double)k * a.step;
            const bool neg = k >= 1 && !(z > a.far_z) && (plain || ray_may_be<false>(t[q]));
            if (!__ballot(neg)) {  // free space: most groups
                carry = kFirst;
                continue;
            }
            const uint64_t pos = __ballot(plain || ray_may_be<true>(t[q]));
            const uint64_t after = ((pos << 1) & ~kFirst) | carry;
            carry = (pos >> (NS - 1)) & kFirst;
            double prev = 0.0, s = 1.0;
            bool cross = false;
            if (neg && __builtin_amdgcn_inverse_ballot_w64(after)) {
                s = ray_sample<FMT>(a, dw, z);
                if (s <= 0.0 && s > -1.0) {
                    prev = ray_sample<FMT>(a, dw, a.near_z + (double)(k - 1) * a.step);
                    cross = prev > 0.0 && prev < 1.0;
                }
            }
            // the pixel's lanes leave the loop together: they are all active here
            const uint64_t hits = (__ballot(cross) >> (px * NS)) & (NS == 64 ? ~0ull : (1ull << (NS & 63)) - 1ull);
            if (hits) {
                const int first = __ffsll((unsigned long long)hits) - 1;
                const double zp = a.near_z + (double)(k - 1) * a.step;
                const double o = zp + a.step * prev / (prev - s);
                out = __shfl(o, px * NS + first, kWave);
                done = true;
            }
        }
    }
    if (j == 0 && u < a.W && v < a.H) a.out[(int64_t)v * a.W + u] = (float)out;
}

// Every sample evaluated: a wavefront per pixel, lane j taking sample
// base + j, the sample before it from the lane below.
template <int FMT>
__global__ __launch_bounds__(256) void k_raycast_each(RaycastArgs a) {
    const int lane = threadIdx.x & 63;
    const int idx = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (idx >= a.W * a.H) return;  // whole wavefronts leave together
    const int u = idx % a.W, v = idx / a.W;
    const double dc[3] = {((double)u - a.cx) / a.fx, ((double)v - a.cy) / a.fy, 1.0};
    double dw[3];
    for (int i = 0; i < 3; ++i) dw[i] = a.R[3 * i + 0] * dc[0] + a.R[3 * i + 1] * dc[1] + a.R[3 * i + 2] * dc[2];
    double carry = 0.0, out = 0.0;  // sample base - 1 (from the round before)
    for (int base = 0;; base += kWave) {
        const int k = base + lane;
        const double z = a.near_z + (double)k * a.step;
        const bool valid = !(z > a.far_z);
        const double s = valid ? ray_sample<FMT>(a, dw, z) : 0.0;
        double prev = __shfl_up(s, 1, kWave);
        if (lane == 0) prev = carry;
        const uint64_t hits = __ballot(valid && k >= 1 && prev > 0.0 && s <= 0.0 && prev < 1.0 && s > -1.0);
        if (hits) {
            const double o = a.near_z + (double)(k - 1) * a.step + a.step * prev / (prev - s);
            out = __shfl(o, __ffsll((unsigned long long)hits) - 1, kWave);
            break;
        }
        if (__ballot(!valid)) break;  // past `far`: so are all later samples
        carry = __shfl(s, kWave - 1, kWave);
    }
    if (lane == 0) a.out[idx] = (float)out;
}

template <int FMT, bool WIDE>
static void launch_raycast(const RaycastArgs& a, hipStream_t s) {
    auto blocks = [&](int tp) { return dim3((unsigned)((((a.W + tp - 1) / tp) * ((a.H + tp - 1) / tp) + 3) / 4)); };
    // A patch of neighbouring rays shares lines that the samples along one ray
    // do not, but leaves fewer wavefronts, whose rounds follow one another;
    // with few samples per ray in a small image the rounds are few and each
    // one's setup and dependent loads count.  384 x 392 x 248, a room, us with
    // every sample evaluated / 1 / 4 / 16 pixels per wavefront:
    //   40 x 30, 1200 samples per ray 11 / 11 / 25 / 93
    //   120 x 90, 1200: 31 / 28 / 34 / 85, 400: 19 / 23 / 18 / 37
    //   160 x 120, 1200: 51 / 45 / 38 / 86, 200: 18 / 30 / 17 / 23, 55: 12 / 22 / 17 / 16
    //   320 x 240, 1200: 186 / - / 112 / 117, 55: 43 / - / 39 / 26
    //   640 x 480, 1200: 733 / - / - / 336, 55: 165 / - / - / 95
    const int64_t pixels = (int64_t)a.W * a.H;
    const double nx = a.g.nx, ny = a.g.ny, nz = a.g.nz;
    const double samples = std::min(a.kmax, sqrt(nx * nx + ny * ny + nz * nz) * (double)a.g.vox / a.step);
    if (pixels < 3000 || samples < (pixels < 15000 ? 1000.0 : pixels < 30000 ? 128.0 : 0.0))
        hipLaunchKernelGGL((k_raycast_each<FMT>), blocks(1), dim3(256), 0, s, a);
    else if (pixels < 15000) hipLaunchKernelGGL((k_raycast<FMT, WIDE, 1, 2>), blocks(1), dim3(256), 0, s, a);
    else if (pixels < (1 << 18)) hipLaunchKernelGGL((k_raycast<FMT, WIDE, 2, 2>), blocks(2), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_raycast<FMT, WIDE, 4, 2>), blocks(4), dim3(256), 0, s, a);
}

template <int FMT>
static void launch_raycast_fmt(const RaycastArgs& a, hipStream_t s) {
    const uint64_t bytes = (uint64_t)a.g.nx * a.g.ny * a.g.nz * (FMT == ROSE_TSDF_F32 ? 4u : 2u);
    // plain pointers for volumes past 32-bit offsets, and for a 16-bit buffer
    // that is not aligned to the pairs the buffer loads take
    if (bytes >= (uint64_t(1) << 32) || ((uintptr_t)a.g.psi & 3u)) launch_raycast<FMT, true>(a, s);
    else launch_raycast<FMT, false>(a, s);
}

struct FeatureArgs {
    const float* depth;
    int32_t W, H;
    const float* render;
    int32_t w, hgt, scale;
    double vel[6];
    int32_t dim;
    float* out;
};

// residual = clamp(D(scale u + scale/2, scale v + scale/2) - render(u, v),
// -0.5, 0.5) where both are valid, else 0; then the 6D velocity; zero pad
__global__ __launch_bounds__(256) void k_features(FeatureArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.dim) return;
    const int npx = a.w * a.hgt;
    float v = 0.0f;
    if (i < npx) {
        const int u = i % a.w, r = i / a.w;
        const int U = a.scale * u + a.scale / 2, V = a.scale * r + a.scale / 2;
        const float d = (U < a.W && V < a.H) ? a.depth[(int64_t)V * a.W + U] : 0.0f;
        const float m = a.render[i];
        if (d > 0.0f && m > 0.0f) v = fminf(0.5f, fmaxf(-0.5f, d - m));
    } else if (i < npx + 6) {
        v = (float)a.vel[i - npx];
    }
    a.out[i] = v;
}

}  // namespace rose

using namespace rose;

extern "C" {

rose_status tsdf_raycast(const rose_tsdf* h, const rose_pose* T_wc, const rose_camera* cam, double near_m,
                         double far_m, double step_m, float* depth_out_dev, hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(h && T_wc && cam && depth_out_dev, ROSE_E_ARG, "tsdf_raycast: NULL argument");
    ROSE_REQUIRE(cam->width > 0 && cam->height > 0 && (int64_t)cam->width * cam->height <= 1 << 20, ROSE_E_SHAPE,
                 "tsdf_raycast: image %dx%d out of range (at most 2^20 pixels)", cam->width, cam->height);
    ROSE_REQUIRE(cam->fx > 0 && cam->fy > 0, ROSE_E_ARG, "tsdf_raycast: focal lengths must be > 0");
    ROSE_REQUIRE(near_m > 0 && far_m > near_m && step_m > 0 && (far_m - near_m) / step_m <= 1e6, ROSE_E_ARG,
                 "tsdf_raycast: need 0 < near < far and 0 < step, at most 1e6 steps");
    RaycastArgs a;
    a.g = h->g;
    quat_rot(T_wc->q, a.R);
    for (int i = 0; i < 3; ++i) a.t[i] = T_wc->t[i];
    a.W = cam->width;
    a.H = cam->height;
    a.fx = cam->fx; a.fy = cam->fy; a.cx = cam->cx; a.cy = cam->cy;
    a.near_z = near_m; a.far_z = far_m; a.step = step_m;
    a.inv_vox = 1.0 / (double)h->g.vox;
    a.kmax = (far_m - near_m) / step_m + 2.0;
    a.out = depth_out_dev;
    if (h->g.fmt == ROSE_TSDF_F32) launch_raycast_fmt<ROSE_TSDF_F32>(a, s);
    else if (h->g.fmt == ROSE_TSDF_F16) launch_raycast_fmt<ROSE_TSDF_F16>(a, s);
    else launch_raycast_fmt<ROSE_TSDF_SN16>(a, s);
    ROSE_CHECK_HIP(hipGetLastError());
    return ROSE_OK;
}

rose_status proposal_features(const float* depth_dev, const rose_camera* cam, const float* render_dev,
                              const rose_camera* cam_low, int32_t scale, const double velocity[6], int32_t dim,
                              float* features_dev, hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(depth_dev && cam && render_dev && cam_low && velocity && features_dev, ROSE_E_ARG,
                 "proposal_features: NULL argument");
    ROSE_REQUIRE(scale >= 1 && cam->width > 0 && cam->height > 0 && cam_low->width > 0 && cam_low->height > 0,
                 ROSE_E_SHAPE, "proposal_features: bad sizes");
    const int npx = cam_low->width * cam_low->height;
    ROSE_REQUIRE(dim >= npx + 6 && dim <= (1 << 20), ROSE_E_SHAPE, "proposal_features: dim %d < pixels + 6", dim);
    FeatureArgs a;
    a.depth = depth_dev;
    a.W = cam->width;
    a.H = cam->height;
    a.render = render_dev;
    a.w = cam_low->width;
    a.hgt = cam_low->height;
    a.scale = scale;
    for (int i = 0; i < 6; ++i) a.vel[i] = velocity[i];
    a.dim = dim;
    a.out = features_dev;
    hipLaunchKernelGGL(k_features, dim3((dim + 255) / 256), dim3(256), 0, s, a);
    ROSE_CHECK_HIP(hipGetLastError());
    return ROSE_OK;
}

}  // extern "C"
