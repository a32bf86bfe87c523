// emergent.hip -- emergent intensity along parallel long characteristics
// (Osborne & Sannikov, arXiv:2408.14425, Sec. 3.9: a single-pass long
// characteristics solver for rays of any direction through the domain,
// traced front to back from the point where the emergent intensity is
// wanted).
//
// A beam of n_rays parallel rays of light direction w, one cell apart
// across the beam and centred on the domain, is traced from outside the
// domain back along -w with the FP64 cell walk and FP32 front-to-back update
// of the cascade march; what has accumulated when a ray leaves the far side
// is the intensity emerging towards the observer.
#include "march_rows.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace rcx {
namespace {

using march::kBlock;

// Every cell is crossed about 1.4 times by a beam, so the image costs one
// read of chi and eta (104 us for 1024^2 x 64 wavelengths at the rate of a
// large copy): they are read here as the caller holds them, without a pass
// that writes fields first (183 us, and the march of the fields another 152;
// now 205 us in all). A workgroup takes 64 neighbouring rays, one per lane, and
// a piece of 16 columns of the major axis. The rays' segments in those
// columns, the same for every wavelength, are found once, into LDS. Then each
// wavefront takes every 4th wavelength: the cells the rays cross in the piece
// (at most kMinor of the minor axis, as the rays lie at most sqrt(2) apart)
// are read in rows of consecutive cells, prepared, and staged in LDS 8 columns
// at a time (40 KB of LDS, so a CU holds 16 wavefronts; all 16 columns at
// once, 8 wavefronts, took 10 to 25 % longer); each lane steps along its ray,
// while the next wavelength's cells are read. The pieces' {I, T} are folded
// front to back by k_emergent_fold. What bounds it is the latency of the reads
// (2.7 TB/s) and of the division and exponentials of each cell.
constexpr int kRays = 64, kTile = 16;
constexpr int kMinor = 109;  // 63 sqrt(2) + 16 + 2 = 107.1 cells, odd against bank conflicts
constexpr int kHalf = kTile / 2, kNull = kHalf * kMinor;  // a staged cell with no opacity and no emission

struct Beam {
    double ox0, oz0, px, pz;  // origin of the beam's middle, unit step across it
    double4 d;                // march direction and its inverse
    int32_t n_rays, r0, r1;   // this launch's rays [r0, r1)
};

// Rays j of the beam: origin o0 + s_j p, s_j = j + 1/2 - n_rays/2 (cells
// across the beam), direction d = -w. blockIdx.x = piece x groups of 64 rays +
// group, .y = share of the wavelengths. part [piece][wavelength][ray - r0] {I, T}.
template <bool XMAJ>
__global__ __launch_bounds__(kBlock, 4) void k_emergent(int32_t nx, int32_t nz, Beam B, const float* __restrict__ chi,
                                                        const float* __restrict__ eta,
                                                        const uint8_t* __restrict__ mask, float voxel, int32_t n_wave,
                                                        int32_t groups, float2* __restrict__ part)
{
    constexpr int kWaves = kBlock / 64, kOwn = kTile / kWaves;  // kOwn: columns whose segments a thread finds
    // loads of a tile: rows of 16 columns x 4 minor cells, or 2 of 64 columns
    constexpr int kLoads = XMAJ ? (kMinor + 3) / 4 : 2 * kTile;
    __shared__ uint32_t key[kTile][kRays];  // staged cells of a column's two segments (16 bits each)
    __shared__ float2 len[kTile][kRays];    // and their lengths
    __shared__ float2 tile[kWaves][kNull + 1];
    __shared__ int lo_cell, hi_cell;         // first and last minor cell
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nm = XMAJ ? nx : nz, nn = XMAJ ? nz : nx;
    const double wm = XMAJ ? B.d.x : B.d.y, wn = XMAJ ? B.d.y : B.d.x;
    const int sm = wm > 0.0 ? 1 : -1, sn = wn > 0.0 ? 1 : -1;
    const int piece = (int)(blockIdx.x / (unsigned)groups), group = (int)blockIdx.x - piece * groups;
    const int q0 = piece * kTile;  // first column, counted along the march
    if (threadIdx.x == 0) {
        lo_cell = INT_MAX;
        hi_cell = -1;
    }
    tile[wave][kNull] = make_float2(0.0f, 0.0f);
    __syncthreads();

    // ---- the segments (walk_ray, march_rows.h: the same arithmetic)
    const int64_t j = (int64_t)B.r0 + group * kRays + lane;  // (beams of nearly 2^31 rays)
    const double s = (double)j + 0.5 - 0.5 * (double)B.n_rays;
    const double cx = B.ox0 + s * B.px, cz = B.oz0 + s * B.pz;
    const double kx = floor(cx), kz = floor(cz), fx = cx - kx, fz = cz - kz;
    const double ax = march::plane_t(0.0, kx, fx, B.d.z), bx = march::plane_t((double)nx, kx, fx, B.d.z);
    const double az = march::plane_t(0.0, kz, fz, B.d.w), bz = march::plane_t((double)nz, kz, fz, B.d.w);
    const double lo = fmax(0.0, fmax(fmin(ax, bx), fmin(az, bz))), hi = fmin(fmax(ax, bx), fmax(az, bz));
    const double km = XMAJ ? kx : kz, kn = XMAJ ? kz : kx, fm = XMAJ ? fx : fz, fn = XMAJ ? fz : fx;
    const double im_ = XMAJ ? B.d.z : B.d.w, in_ = XMAJ ? B.d.w : B.d.z;
    const int ikm = (int)km, ikn = (int)kn;
    const double qm0 = fm + lo * wm;
    int im0 = ikm + (wm > 0.0 ? (int)floor(qm0) : (int)ceil(qm0) - 1);
    im0 = min(max(im0, 0), nm - 1);
    const int mfirst = wm > 0.0 ? im0 + 1 : im0;
    const bool ray = j < B.r1 && lo < hi;
    int c0[kOwn], c1[kOwn];
    float2 ds[kOwn];
    int low = INT_MAX, high = -1;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int q = q0 + wave + i * kWaves, m = sm > 0 ? q : nm - 1 - q;
        const int jc = (m - im0) * sm;  // column of the ray
        const int pj = mfirst + (jc - 1) * sm;
        const double ta = jc == 0 ? lo : march::plane_t((double)(pj - ikm), 0.0, fm, im_);
        const double tb = fmin(march::plane_t((double)(pj + sm - ikm), 0.0, fm, im_), hi);
        const bool valid = ray && q < nm && jc >= 0 && ta < hi;
        const double qn = fn + ta * wn;
        int in0 = ikn + ((int)floor((double)sn * qn) ^ (sn > 0 ? 0 : -1));
        in0 = min(max(in0, 0), nn - 1);
        const double tn = march::plane_t((double)(in0 + (sn > 0 ? 1 : 0) - ikn), 0.0, fn, in_);
        const bool two = valid && tn < tb;
        const double tmid = fmax(tn, ta);
        const int in1 = min(max(in0 + sn, 0), nn - 1);
        ds[i] = make_float2(valid ? (float)fmax((two ? tmid : tb) - ta, 0.0) : 0.0f,
                            two ? (float)fmax(tb - tmid, 0.0) : 0.0f);
        c0[i] = valid ? in0 : -1;
        c1[i] = two ? in1 : -1;
        if (valid) low = min(low, two ? min(in0, in1) : in0);
        high = max(high, max(c0[i], c1[i]));
    }
#pragma unroll
    for (int m = 1; m < 64; m *= 2) {
        low = min(low, __shfl_xor(low, m));
        high = max(high, __shfl_xor(high, m));
    }
    if (lane == 0) {
        atomicMin(&lo_cell, low);
        atomicMax(&hi_cell, high);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int c = wave + i * kWaves, first = lo_cell;
        auto at = [&](int cell) {
            return cell < 0 ? kNull : (c % kHalf) * kMinor + min(cell - first, kMinor - 1);
        };
        key[c][lane] = (uint32_t)at(c0[i]) | ((uint32_t)at(c1[i]) << 16);
        len[c][lane] = ds[i];
    }
    __syncthreads();

    // ---- the wavelengths
    const int64_t ncell = (int64_t)nx * nz;
    const int step = kWaves * (int)gridDim.y;
    const int lo_n = __builtin_amdgcn_readfirstlane(lo_cell), hi_n = __builtin_amdgcn_readfirstlane(hi_cell);
    float2* own = tile[wave];
    float ch[kLoads], et[kLoads];
    // cell of load i: a lane's column and every 4th minor cell, or column i / 2
    // and 64 minor cells. What lies past the last cell (read by no ray) is that
    // cell again
    uint32_t at0, at1;
    if constexpr (XMAJ) {
        const int col = min(q0 + (lane & 15), nm - 1), m = sm > 0 ? col : nm - 1 - col;
        at0 = (uint32_t)((lo_n + (lane >> 4)) * nx + m);
        at1 = (uint32_t)(hi_n * nx + m);
    } else {
        at0 = (uint32_t)min(lo_n + lane, hi_n);
        at1 = (uint32_t)min(lo_n + lane + 64, hi_n);
    }
    auto cell_of = [&](int i) -> uint32_t {
        if constexpr (XMAJ) return min(at0 + 4u * (uint32_t)(i * nx), at1);
        const int col = min(q0 + (i >> 1), nm - 1);
        return (uint32_t)((sm > 0 ? col : nm - 1 - col) * nx) + (i & 1 ? at1 : at0);
    };
    auto load = [&](int lam) {
        const float* cp = chi + (int64_t)lam * ncell;
        const float* ep = eta + (int64_t)lam * ncell;
        asm("" : "+v"(at0), "+v"(at1));  // (the cells' offsets are formed again, not kept)
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const uint32_t c = cell_of(i);
            ch[i] = cp[c];
            et[i] = ep[c];
        }
    };
    const bool any = hi_n >= 0;
    int lam = wave + kWaves * (int)blockIdx.y;
    if (any && lam < n_wave) load(lam);
    for (; lam < n_wave; lam += step) {
        float I = 0.0f, T = 1.0f;
        if (any) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                float2 f = march::prep_value(ch[i], et[i], voxel);
                if (mask && !mask[cell_of(i)]) f = make_float2(0.0f, 0.0f);
                ch[i] = f.x;
                et[i] = f.y;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // a lane's loads lie in one half of the columns (XMAJ), or half
                // of them in each
                if (!XMAJ || ((lane >> 3) & 1) == h) {
#pragma unroll
                    for (int i = XMAJ ? 0 : h * kTile; i < (XMAJ ? kLoads : (h + 1) * kTile); ++i) {
                        const int n = XMAJ ? (lane >> 4) + 4 * i : lane + 64 * (i & 1);
                        const int at = (XMAJ ? lane & 7 : (i >> 1) - h * kHalf) * kMinor + n;
                        if (n < kMinor) own[at] = make_float2(ch[i], et[i]);
                    }
                }
                march::wave_sync();
                if (h == 1 && lam + step < n_wave) load(lam + step);
#pragma unroll 4
                for (int c = 0; c < kHalf; ++c) {
                    const uint32_t e = key[h * kHalf + c][lane];
                    const float2 l = len[h * kHalf + c][lane];
                    const float2 f0 = own[e & 0xffffu], f1 = own[e >> 16];
                    march::step(f0, l.x, I, T);
                    march::step(f1, l.y, I, T);
                }
                march::wave_sync();
            }
        }
        if (j < B.r1) part[((int64_t)piece * n_wave + lam) * (B.r1 - B.r0) + (j - B.r0)] = make_float2(I, T);
    }
}

// I[lam][r0 + j] of this launch's n rays, the pieces front to back.
__global__ __launch_bounds__(256) void k_emergent_fold(const float2* __restrict__ part, int32_t pieces, int32_t n,
                                                       int32_t r0, int32_t n_rays, int32_t n_wave,
                                                       float* __restrict__ out)
{
    const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    for (int32_t lam = blockIdx.y; lam < n_wave; lam += gridDim.y) {
        float I = 0.0f, T = 1.0f;
#pragma unroll 8
        for (int p = 0; p < pieces; ++p) {
            const float2 v = part[((int64_t)p * n_wave + lam) * n + j];
            I = fmaf(T, v.x, I);
            T *= v.y;
        }
        out[(int64_t)lam * n_rays + r0 + j] = I;
    }
}

}  // namespace
}  // namespace rcx

using namespace rcx;

extern "C" int32_t rcx_emergent(rcx_plan* p, int32_t n_wave, const float* chi, const float* eta, double wx,
                                double wz, int32_t n_rays, float* I, hipStream_t st)
{
    if (!p || !chi || !eta || !I) return fail(RCX_E_INVALID, "rcx_emergent: null argument");
    if (n_wave <= 0 || n_wave > p->max_wave) return fail(RCX_E_INVALID, "rcx_emergent: n_wave must be in [1, max_wave]");
    if (n_rays <= 0) return fail(RCX_E_INVALID, "rcx_emergent: n_rays must be positive");
    const double wn = std::hypot(wx, wz);
    if (!(wn > 0.0) || !std::isfinite(wn)) return fail(RCX_E_INVALID, "rcx_emergent: direction must be non-zero");
    wx /= wn;
    wz /= wn;
    const int32_t nx = p->grid.nx, nz = p->grid.nz;
    const int64_t ncell = (int64_t)nx * nz;
    if (p->prm.flags & RCX_FLAG_CHECK_INPUT) {
        unsigned int* flag = (unsigned int*)p->ws_own;  // read back before the march
        RCX_HIP_TRY(launch_zero_flag(flag, st));
        RCX_HIP_TRY(launch_check_f32(chi, (int64_t)n_wave * ncell, kCheckNonNegative, flag, st));
        RCX_HIP_TRY(launch_check_f32(eta, (int64_t)n_wave * ncell, kCheckNonNegative, flag, st));
        const int32_t rc = check_flag_result(flag, "rcx_emergent: chi or eta", st);
        if (rc != RCX_OK) return rc;
    }
    // beam: centred on the domain, starting outside it on the observer's
    // side; march direction -w (an axis-parallel ray gets a 1e-12 minor
    // component so its plane steps stay finite; its cells are unchanged)
    const double R = 0.5 * std::hypot((double)nx, (double)nz) + 2.0;
    const double ox0 = 0.5 * nx + R * wx, oz0 = 0.5 * nz + R * wz;
    double dx = -wx, dz = -wz;
    if (std::fabs(dx) < 1e-12) dx = dx < 0.0 ? -1e-12 : 1e-12;
    if (std::fabs(dz) < 1e-12) dz = dz < 0.0 ? -1e-12 : 1e-12;
    const double4 d = make_double4(dx, dz, 1.0 / dx, 1.0 / dz);
    // the pieces' {I, T} lie in the plan's own workspace, which holds 128 B per
    // cell and 16 wavelengths of max_wave at least, so one ray of every
    // wavelength and piece; a beam too wide for it (hundreds of domain widths),
    // or for a launch's grid, goes in slices
    const bool xmaj = std::fabs(d.x) >= std::fabs(d.y);
    const int32_t pieces = ((xmaj ? nx : nz) - 1) / kTile + 1;
    const int64_t room = (int64_t)(p->ws_own_bytes / sizeof(float2)) / ((int64_t)pieces * n_wave);
    const int32_t slice =
        (int32_t)std::min({(int64_t)n_rays, room, (int64_t)(kMaxGridX / (uint32_t)pieces) * kRays});
    Beam B{ox0, oz0, -wz, wx, d, n_rays, 0, 0};
    for (B.r0 = 0; B.r0 < n_rays; B.r0 = B.r1) {
        B.r1 = (int32_t)std::min<int64_t>((int64_t)B.r0 + slice, n_rays);
        const int32_t n = B.r1 - B.r0;
        const int32_t groups = (n - 1) / kRays + 1;
        // shares of the wavelengths: up to 3 rounds of the 1024 workgroups that
        // the chip holds, one wavelength per wavefront at least (2 at least are
        // 1 us faster on 512^2 x 16 and 4 us slower on 100 x 140 x 20)
        const int32_t shares = (int32_t)std::max<int64_t>(
            std::min({3072 / ((int64_t)groups * pieces), (int64_t)(n_wave + 3) / 4, (int64_t)65535}), 1);
        const dim3 grid((unsigned)groups * (unsigned)pieces, (unsigned)shares);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, st, nx, nz, B, chi, eta, p->mask_dev,
                               (float)p->grid.voxel_scale, n_wave, groups, (float2*)p->ws_own);
        };
        if (xmaj) go(k_emergent<true>);
        else go(k_emergent<false>);
        RCX_HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_emergent_fold, dim3((unsigned)((n - 1) / 256 + 1), (unsigned)std::min(n_wave, 65535)),
                           dim3(256), 0, st, (const float2*)p->ws_own, pieces, n, B.r0, n_rays, n_wave, I);
        RCX_HIP_TRY(hipGetLastError());
    }
    return RCX_OK;
}
