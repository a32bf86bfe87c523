// march_table.hip -- segment tables of a plan's cascades and the launches of
// the march that reads them (march_table.h; Osborne & Sannikov,
// arXiv:2408.14425, Secs. 2.2-2.3).
#include "march_table.h"
#include "segment_length.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

namespace rcx {

namespace {

using tab::DirTable;
using tab::Segment;

// Tables beyond this size (grids of about 4096^2 with three wide cascades
// stay below 1 GiB) are not built; such plans march with the cell walk.
constexpr size_t kTableMaxBytes = size_t(2) << 30;

struct LevelWalk {
    int32_t nd, odd;  // odd: probe centres at cell centres (spacing 1), else at cell corners
    int32_t nx;
    int32_t fix;      // 16 lists per direction (march_table.h, k_march_fix_table)
    double s;
    double ta, tb, dmax_x, dmax_z;  // largest distance from a probe to the exit planes
};

// The line a list follows: from (ox, oz) relative to the probe along (x, z),
// parameters [t0, t1) (t1 no later than where every probe's ray has left the
// domain).
struct Line {
    double x, z, ix, iz, ox, oz, t0, t1;
};

__host__ __device__ inline Line list_line(const LevelWalk& W, double4 d, int32_t cls)
{
    Line n;
    if (!W.fix) {
        n = Line{d.x, d.y, d.z, d.w, 0.0, 0.0, W.ta, 0.0};
        n.t1 = fmin(W.tb, fmin(W.dmax_x * fabs(d.z), W.dmax_z * fabs(d.w)) + 2.0);
        return n;
    }
    // from p + t_a w to q + t_b w; a ray of no length crosses nothing, and an
    // axis-parallel one gets a 1e-12 minor component (as march_fix_ray)
    n.ox = W.ta * d.x;
    n.oz = W.ta * d.y;
    const double dx = ((cls & 3) - 1.5) * W.s + W.tb * d.x - n.ox, dz = ((cls >> 2) - 1.5) * W.s + W.tb * d.y - n.oz;
    const double len = sqrt(dx * dx + dz * dz);
    n.x = 0.6;
    n.z = 0.8;
    if (len > 0.0) {
        n.x = dx / len;
        n.z = dz / len;
        if (fabs(n.x) < 1e-12) n.x = n.x < 0.0 ? -1e-12 : 1e-12;
        if (fabs(n.z) < 1e-12) n.z = n.z < 0.0 ? -1e-12 : 1e-12;
    }
    n.ix = 1.0 / n.x;
    n.iz = 1.0 / n.z;
    n.t0 = 0.0;
    const double ex = (W.dmax_x - (n.x > 0.0 ? n.ox : -n.ox)) * fabs(n.ix);
    const double ez = (W.dmax_z - (n.z > 0.0 ? n.oz : -n.oz)) * fabs(n.iz);
    n.t1 = fmin(len, fmin(ex, ez) + 2.0);
    return n;
}

// One thread per list: the walk of walk_ray (march_rows.h) from a probe
// in cell (0, 0) on an unbounded grid, with the same FP64 arithmetic, so a
// ray steps the same segments, in the same order, with the same lengths
// (with the bilinear fix to FP64 rounding: its rays start at p + t_a w).
// rest (nullable): what the FP32 lengths leave out.
__global__ void k_build_tables(LevelWalk W, const double4* __restrict__ dirs, DirTable* __restrict__ dt,
                               Segment* __restrict__ segs, uint32_t* __restrict__ idx, float* __restrict__ rest)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int nc = W.fix ? tab::kFixClasses : 1;
    if (k >= W.nd * nc) return;
    DirTable D = dt[k];
    const Line d = list_line(W, dirs[k / nc], k % nc);
    const double f = W.odd ? 0.5 : 0.0, fx = f + d.ox, fz = f + d.oz;
    const bool xmaj = fabs(d.x) >= fabs(d.z);
    const double wm = xmaj ? d.x : d.z, wn = xmaj ? d.z : d.x, im_ = xmaj ? d.ix : d.iz, in_ = xmaj ? d.iz : d.ix;
    const double fm = xmaj ? fx : fz, fn = xmaj ? fz : fx;
    const int sm = wm > 0.0 ? 1 : -1, sn = wn > 0.0 ? 1 : -1;
    const double T0 = d.t0, T1 = d.t1;
    const double qm0 = fm + T0 * wm;
    const int im0 = wm > 0.0 ? (int)floor(qm0) : (int)ceil(qm0) - 1;
    const int mfirst = wm > 0.0 ? im0 + 1 : im0;
    const double snd = (double)sn;
    const int nflip = sn > 0 ? 0 : -1, nadd = sn > 0 ? 1 : 0;
    const int sx = d.x > 0.0 ? 1 : -1, sz = d.z > 0.0 ? 1 : -1;

    int n = 0, px = 0, pz = 0;
    D.px0 = D.pz0 = 0;
    auto emit = [&](int dx, int dz, double len) {
        if (n >= D.cap) return;
        // progress never falls back (where a ray passes through a corner to
        // rounding), so a run's cells all lie inside the domain
        const int nx_ = n ? max(sx * dx, px) : sx * dx, nz_ = n ? max(sz * dz, pz) : sz * dz;
        if (n == 0) {
            D.px0 = px = nx_;
            D.pz0 = pz = nz_;
        }
        while (px < nx_) idx[D.ix + (uint32_t)(++px - D.px0)] = (uint32_t)n;
        while (pz < nz_) idx[D.iz + (uint32_t)(++pz - D.pz0)] = (uint32_t)n;
        // (entries that lie outside the domain for every probe may wrap: no ray reads them)
        segs[D.off + n] = Segment{(int)(uint32_t)(((int64_t)(sz * nz_) * W.nx + sx * nx_) * (tab::kLB * 8)), (float)len};
        if (rest) rest[D.off + n] = length_rest(len);
        ++n;
    };
    if (T0 < T1) {
        for (int j = 0;; ++j) {
            const int pj = mfirst + (j - 1) * sm;
            const double ta = j == 0 ? T0 : march::plane_t((double)pj, 0.0, fm, im_);
            if (!(ta < T1)) break;
            const double tb = fmin(march::plane_t((double)(pj + sm), 0.0, fm, im_), T1);
            const int im = im0 + j * sm;
            const double qn = fn + ta * wn;
            const int in0 = (int)floor(snd * qn) ^ nflip;
            const double tn = march::plane_t((double)(in0 + nadd), 0.0, fn, in_);
            const bool two = tn < tb;
            const double tmid = fmax(tn, ta);
            emit(xmaj ? im : in0, xmaj ? in0 : im, fmax((two ? tmid : tb) - ta, 0.0));
            if (two) emit(xmaj ? im : in0 + sn, xmaj ? in0 + sn : im, fmax(tb - tmid, 0.0));
            if (n >= D.cap) break;
        }
    }
    for (int q = 0; q < tab::kSegPad; ++q) segs[D.off + n + q] = Segment{0, 0.0f};
    D.n = n;
    D.px1 = px;
    D.pz1 = pz;
    D.xpos = sx > 0;
    D.zpos = sz > 0;
    // the same for the children of a cone (of 16 directions' cones, some lie on
    // both sides of a diagonal) and for a direction's lists: they march together
    const double4 mid = dirs[(k / nc & ~3) + 1];
    D.xmaj = fabs(mid.x) >= fabs(mid.y);
    dt[k] = D;
}

// ------------------------------------------------------------- windows
// The wide cascades' rays are hundreds of cells long, and the rays one XCD
// holds at a time, each at its own distance along its way, cover far more
// cells than its L2 holds: 60% of the L2's reads missed on the two widest
// cascades of a 1024^2 grid, 80 GB a launch at the fabric's rate. So these
// cascades are marched in windows of kWindow list entries, a launch each,
// and the workgroups of a window are sorted by the region of the grid their
// segments cross: a window's list walks the grid region by region, every
// region's cells are fetched about once per window, and a ray's {I, T} waits
// in memory between windows (16 B per window against 8 B per entry).
constexpr int kWindow = 128;
constexpr int kRegion = 64;    // cells per side (a workgroup's own segments spread over 100-230)
// bins of (window, region, wedge) at most, larger regions beyond (4096^2 takes
// 7e6, 3e7 with the fix; a 64 x 140000 strip would take 8e7 of the 64^2 ones)
constexpr size_t kMaxBins = size_t(1) << 25;
constexpr int kDirBins = 32;   // wedges of directions, in order within a region

struct WindowGeom {
    tab::LaunchArgs A;  // geometry, directions, lists, sub-blocks, flagged probes
    uint32_t n_sub, n_cone;
    int32_t region, nrx, nrz, n_win;  // n_win: of one tap
    int32_t fix;              // 4 taps, the sub-blocks of each parity
    double s, ta;
};

// Windows [w0, w1) of a workgroup (sub-block, cone, tap): those that hold
// entries of its rays, at least one; false when the sub-block holds no ray.
__device__ bool window_range(const WindowGeom& G, uint32_t sub, uint32_t cone, int tap, int& w0, int& w1, int& uc,
                             int& vc)
{
    const tab::LaunchArgs& A = G.A;
    int a_min = 1 << 30, e_max = 0;
    bool any = false;
    for (int j = 0; j < 4; ++j) {
        const int pu = sub & 1, pv = (sub >> 1) & 1;  // (fix)
        const DirTable D = G.fix ? A.dirs[(4 * cone + j) * tab::kFixClasses + tab::fix_class(pu, pv, tap & 1, tap >> 1)]
                                 : A.dirs[4 * cone + j];
        for (int row = 0; row < tab::kWinLong * tab::kWinShort; ++row) {
            int u, v;
            bool active;
            if (A.plist) {
                const uint32_t i = sub * (tab::kWinLong * tab::kWinShort) + (uint32_t)row;
                active = i < (uint32_t)A.n_active;
                const uint32_t p = active ? (uint32_t)A.plist[i] : 0u;
                v = (int)A.pxdiv.div(p);
                u = (int)(p - (uint32_t)v * A.pxdiv.d);
            } else if (G.fix) {
                tab::window_probe(A, sub >> 2, D.xmaj, row, u, v, active);
                u = 2 * u + pu;
                v = 2 * v + pv;
                active = active && u < A.full_px && v < A.full_pz &&
                         tab::FixTap(u, v, tap & 1, tap >> 1, A.qx, A.qz).in;
            } else {
                tab::window_probe(A, sub, D.xmaj, row, u, v, active);
            }
            if (!active) continue;
            if (!any) {
                uc = u;
                vc = v;
            }
            any = true;
            int a, e;
            tab::clip_run(D, A.idx, A.nx, A.nz, u * A.is + A.half, v * A.is + A.half, a, e);
            if (a >= e) continue;
            a_min = min(a_min, a);
            e_max = max(e_max, e);
        }
    }
    w0 = e_max > 0 ? a_min / kWindow : 0;
    w1 = e_max > 0 ? (e_max - 1) / kWindow + 1 : 1;
    return any;
}

// counts (fill == nullptr) or places the workgroups by (window, region, wedge):
// bins[((tap * n_win + w) * regions + r) * kDirBins + wedge] holds the count,
// then the next free place.
__global__ void k_windows(WindowGeom G, const double4* __restrict__ dirs, uint32_t* __restrict__ bins,
                          tab::Work* __restrict__ fill)
{
    const uint32_t id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= G.n_sub * G.n_cone) return;
    const uint32_t sub = id / G.n_cone, cone = id - sub * G.n_cone;
    const int tap = (int)blockIdx.y;
    int w0, w1, u, v;
    if (!window_range(G, sub, cone, tap, w0, w1, u, v)) return;
    const double4 d = dirs[4 * cone + 1];
    const double per = 1.0 / (fabs(d.x) + fabs(d.y));
    for (int w = w0; w < w1; ++w) {
        const double t = G.ta + (w + 0.5) * kWindow * per;
        const int x = (int)((u + 0.5) * G.s + t * d.x) / G.region, z = (int)((v + 0.5) * G.s + t * d.y) / G.region;
        const int rx = min(max(x, 0), G.nrx - 1), rz = min(max(z, 0), G.nrz - 1);
        const uint32_t bin = (uint32_t)(((tap * G.n_win + w) * G.nrz + rz) * G.nrx + rx) * kDirBins +
                             (uint32_t)((uint64_t)cone * kDirBins / G.n_cone);
        const uint32_t at = atomicAdd(&bins[bin], 1u);
        if (fill) fill[at] = tab::Work{sub, cone * 2u + (w + 1 == w1 ? 1u : 0u)};
    }
}

size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace

namespace {
hipError_t make_tables(const rcx_grid& g, const rcx_params& prm, const std::vector<LevelDesc>& levels,
                       bool top_skipped, const std::vector<double4>& dirs, const std::vector<int32_t>& dir_off,
                       const double4* dirs_dev, bool rests, std::vector<LevelTable>& tables, void** mem)
{
    const int32_t n_casc = (int32_t)levels.size();
    tables.assign(n_casc, LevelTable{});
    *mem = nullptr;
    if (prm.c0_dirs != 4) return hipSuccess;
    const bool fix = (prm.flags & RCX_FLAG_BILINEAR_FIX) != 0;
    struct Off {
        size_t dirs, segs, idx, rest;
    };
    std::vector<Off> off(n_casc);
    std::vector<DirTable> dt;  // every cascade's, copied at once
    std::vector<size_t> first(n_casc + 1, 0);
    std::vector<LevelWalk> lw(n_casc);
    size_t total = 0;
    for (int32_t i = 0; i < n_casc; ++i) {
        first[i + 1] = first[i] = dt.size();
        if (top_skipped && i == n_casc - 1) continue;
        const LevelDesc& L = levels[i];
        // 32-bit byte offsets of the fields, probe cells past a ragged edge included
        if (((double)L.pz * L.s + 1.0) * g.nx * tab::kLB * 8 >= 4294967296.0) return hipSuccess;
        // 32-bit places in a stored cascade of 16 wavelengths (every direction's
        // code, or the means of 4): long, narrow grids with wide cascades walk
        const double stored = (double)L.px * L.pz * L.nd / (prm.storage == RCX_STORE_F16_SCALED ? 1 : 4);
        if (i > 0 && stored * tab::kLB >= 4294967296.0) return hipSuccess;
        LevelWalk& W = lw[i];
        W.nd = L.nd;
        W.odd = L.s == 1.0;
        W.nx = g.nx;
        W.fix = fix && i + 1 < n_casc;
        W.s = L.s;
        W.ta = L.ta;
        W.tb = L.tb;
        W.dmax_x = std::max((L.px - 0.5) * L.s, g.nx - 0.5 * L.s);
        W.dmax_z = std::max((L.pz - 0.5) * L.s, g.nz - 0.5 * L.s);
        // furthest cell from a probe's own that a ray inside the domain crosses
        // (the last probes of a ragged grid lie past its far edge)
        const double far_x = std::max((L.px - 1) * L.s + std::floor(0.5 * L.s), g.nx - 1.0);
        const double far_z = std::max((L.pz - 1) * L.s + std::floor(0.5 * L.s), g.nz - 1.0);
        const int32_t nc = W.fix ? tab::kFixClasses : 1;
        // (before the host holds a header for every list)
        const double least = (sizeof(DirTable) + (8.0 + tab::kSegPad) * sizeof(Segment)) * L.nd * nc;
        if ((double)total + least > (double)kTableMaxBytes) return hipSuccess;
        dt.resize(first[i] + (size_t)L.nd * nc);
        first[i + 1] = dt.size();
        double n_seg = 0.0, n_idx = 0.0;
        for (int32_t k = 0; k < L.nd * nc; ++k) {
            const Line d = list_line(W, dirs[dir_off[i] + k / nc], k % nc);
            const double len = std::max(d.t1 - d.t0, 0.0), wx = std::fabs(d.x), wz = std::fabs(d.z);
            if (!(len * (wx + wz) < 1e9)) return hipSuccess;  // (intervals near the largest double, with the fix)
            // keys are 32-bit byte offsets with sign: where a ray can cross a
            // cell 2^24 cells away (within a few percent of the largest grids,
            // with probes past the edge) the plan walks
            const double reach = std::min(std::fabs(d.oz + d.z * d.t1) + 2.0, far_z) * g.nx +
                                 std::min(std::fabs(d.ox + d.x * d.t1) + 2.0, far_x);
            if (len > 0.0 && reach * (tab::kLB * 8) >= 2147483648.0) return hipSuccess;
            DirTable& D = dt[first[i] + k];
            D.cap = (int32_t)(len * (wx + wz)) + 8;
            tables[i].max_entries = std::max(tables[i].max_entries, D.cap);
            D.off = (uint32_t)n_seg;
            D.ix = (uint32_t)n_idx;
            D.iz = D.ix + (uint32_t)(len * wx) + 6;
            n_seg += D.cap + tab::kSegPad;
            n_idx = (double)D.iz + std::floor(len * wz) + 6;
            if (n_seg * sizeof(Segment) + n_idx * sizeof(uint32_t) > (double)kTableMaxBytes) return hipSuccess;
        }
        off[i].segs = total;
        total += up256(sizeof(Segment) * (size_t)n_seg);
        off[i].idx = total;
        total += up256(sizeof(uint32_t) * (size_t)n_idx);
        off[i].rest = total;
        if (rests) total += up256(sizeof(float) * (size_t)n_seg);
    }
    const size_t dirs_at = total;
    total += up256(sizeof(DirTable) * dt.size());
    if (total > kTableMaxBytes) return hipSuccess;
    hipError_t e = hipMalloc(mem, total);
    if (e != hipSuccess) return e;
    char* base = (char*)*mem;
    e = hipMemcpy(base + dirs_at, dt.data(), sizeof(DirTable) * dt.size(), hipMemcpyHostToDevice);
    for (int32_t i = 0; i < n_casc && e == hipSuccess; ++i) {
        const size_t n_list = first[i + 1] - first[i];
        if (n_list == 0) continue;
        off[i].dirs = dirs_at + sizeof(DirTable) * first[i];
        tables[i].dirs = base + off[i].dirs;
        tables[i].segs = base + off[i].segs;
        tables[i].idx = (const uint32_t*)(base + off[i].idx);
        if (rests) tables[i].rest = (const float*)(base + off[i].rest);
        hipLaunchKernelGGL(k_build_tables, dim3((unsigned)((n_list + 63) / 64)), dim3(64), 0, nullptr, lw[i],
                           dirs_dev + dir_off[i], (DirTable*)(base + off[i].dirs), (Segment*)(base + off[i].segs),
                           (uint32_t*)(base + off[i].idx), (float*)tables[i].rest);
        e = hipGetLastError();
    }
    // solves may run on any stream
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) {
        (void)hipFree(*mem);
        *mem = nullptr;
        tables.assign(n_casc, LevelTable{});
    }
    return e;
}
}  // namespace

hipError_t build_tables(const rcx_grid& g, const rcx_params& prm, const std::vector<LevelDesc>& levels,
                        bool top_skipped, const std::vector<double4>& dirs, const std::vector<int32_t>& dir_off,
                        const double4* dirs_dev, bool rests, std::vector<LevelTable>& tables, void** mem)
{
    try {
        return make_tables(g, prm, levels, top_skipped, dirs, dir_off, dirs_dev, rests, tables, mem);
    } catch (const std::bad_alloc&) {
        return hipErrorOutOfMemory;
    }
}

int32_t table_lanes(int32_t n)
{
    int32_t lanes = 1;
    while (lanes < n) lanes *= 2;
    return std::min(lanes, (int32_t)tab::kLB);
}

namespace {

// Launch arguments that depend on the cascade alone.
tab::LaunchArgs level_args(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz)
{
    tab::LaunchArgs A{};
    A.nx = nx;
    A.nz = nz;
    A.px = L.px;
    A.pz = L.pz;
    A.nd = L.nd;
    A.qx = L.qx;
    A.qz = L.qz;
    A.is = (int32_t)L.s;
    A.half = A.is >> 1;
    A.dirs = (const DirTable*)T.dirs;
    A.segs = (const Segment*)T.segs;
    A.idx = T.idx;
    A.plist = L.plist;
    A.n_active = L.n_active;
    A.pxdiv = make_fastdiv((uint32_t)L.px);
    A.pzdiv = make_fastdiv((uint32_t)L.pz);
    A.sub_x = make_fastdiv((uint32_t)((L.px + tab::kWinShort - 1) / tab::kWinShort));
    A.sub_z = make_fastdiv((uint32_t)((L.px + tab::kWinLong - 1) / tab::kWinLong));
    A.ncell = (int64_t)nx * nz;
    return A;
}

// Bilinear fix: the probe grid of the even parity.
void fix_probes(tab::LaunchArgs& A)
{
    A.full_px = A.px;
    A.full_pz = A.pz;
    A.px = (A.px + 1) / 2;
    A.pz = (A.pz + 1) / 2;
    A.sub_x = make_fastdiv((uint32_t)((A.px + tab::kWinShort - 1) / tab::kWinShort));
    A.sub_z = make_fastdiv((uint32_t)((A.px + tab::kWinLong - 1) / tab::kWinLong));
}

// Probes in plain order (along the directions' minor axis, PW at a time)
// where tiled sub-blocks would leave more than a fifth of their rows empty:
// 333x200 x 19 wavelengths 512 -> 468 us, x 3 209 -> 188, 100x140 x 32 124 ->
// 116; with less waste the tiles' locality is worth more (600x420 x 20 3.19
// ms in tiles, 3.29 plain from 8 % on, 3.51 from 2 %).
constexpr double kPlainWaste = 1.25;
template <int LB, int W, int OUT>
void set_plain(tab::LaunchArgs& A, const LevelDesc& L)
{
    constexpr int32_t PW = tab::wave_probes<LB, W>(), th = PW <= 4 ? 1 : PW <= 16 ? PW / 4 : 4, tw = PW / th;
    if (A.plist || OUT == tab::kOutJ || L.tile_p <= 0) return;
    auto pad = [](int32_t n, int32_t m) { return (double)((n + m - 1) / m * m); };
    const double padded = 0.5 * (pad(A.px, tw) * pad(A.pz, th) + pad(A.px, th) * pad(A.pz, tw));
    if (padded > kPlainWaste * A.px * A.pz) A.n_active = A.px * A.pz;
}

// The launch order of a cascade marched whole; returns its workgroups per
// wavelength batch.
template <int LB, int W, int OUT>
uint64_t set_order(tab::LaunchArgs& A, const LevelDesc& L)
{
    constexpr int PW = tab::wave_probes<LB, W>(), NS = tab::sub_blocks<LB, W, OUT>();
    // Sub-blocks: on the tiled (wide) cascades the probes of a wavefront run
    // along the direction's minor axis, where their rays end closest
    // together (up to 4 x 16 probes at few wavelengths); below, along x, so
    // neighbouring probes read and write neighbouring addresses.
    const bool tiled = L.tile_p > 0;
    uint32_t blocks_per_tile, n_tiles, wedge;
    const uint32_t cones = (uint32_t)L.nd / 4;
    if (A.plist || A.n_active) {
        const int32_t per = PW * NS;
        A.tile_x = tiled ? (L.tile_p * L.tile_p + per - 1) / per * per : per;
        A.tile_z = 0;
        blocks_per_tile = (uint32_t)(A.tile_x / per);
        n_tiles = (uint32_t)((A.n_active + A.tile_x - 1) / A.tile_x);
        A.tw_log2 = 0;
        A.th = 1;
        A.nb_long = make_fastdiv(1);
        A.ntx = make_fastdiv(1);
        A.orient = 0;
    } else {
        int32_t tw, th;
        if (tiled && OUT != tab::kOutJ) {
            th = PW <= 4 ? 1 : PW <= 16 ? PW / 4 : 4;
            tw = PW / th;
            const int32_t side = (L.tile_p + tw - 1) / tw * tw;
            A.tile_x = A.tile_z = side;
            A.orient = 1;
        } else {
            th = 1;
            tw = PW;
            A.tile_x = tw * NS;
            A.tile_z = 1;
            A.orient = 0;
        }
        A.tw_log2 = 0;
        while ((1 << A.tw_log2) < tw) ++A.tw_log2;
        A.th = th;
        A.nb_long = make_fastdiv((uint32_t)(A.tile_x / (tw * NS)));
        blocks_per_tile = A.nb_long.d * (uint32_t)(A.tile_z / th);
        const uint32_t ntx = (uint32_t)((A.px + A.tile_x - 1) / A.tile_x);
        A.ntx = make_fastdiv(ntx);
        n_tiles = ntx * (uint32_t)((A.pz + A.tile_z - 1) / A.tile_z);
    }
    wedge = tiled && L.tile_d >= 4 ? (uint32_t)L.tile_d / 4 : cones;
    const uint64_t blocks = (uint64_t)n_tiles * blocks_per_tile * cones;
    A.n_blocks = (uint32_t)blocks;
    A.per = make_fastdiv(blocks_per_tile * wedge);
    A.nwedge = make_fastdiv(cones / wedge);
    A.wd = make_fastdiv(wedge);
    A.chunk = make_fastdiv((uint32_t)L.xcd_chunk);
    A.chunk8 = make_fastdiv((uint32_t)L.xcd_chunk * march::kXcds);
    return blocks;
}

// Workgroups [0, blocks) of a march in launches of at most kMaxGridX:
// go(grid.x) with A.block0 set.
template <class Go>
hipError_t launch_blocks(tab::LaunchArgs& A, uint64_t blocks, Go&& go)
{
    if (blocks >= (1ull << 32) - march::kXcds) return hipErrorInvalidValue;
    const uint64_t all = (blocks + march::kXcds - 1) / march::kXcds * march::kXcds;
    for (uint64_t b = 0; b < all; b += kMaxGridX) {
        A.block0 = (uint32_t)b;
        go((unsigned)std::min<uint64_t>(all - b, kMaxGridX));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int LB, int W, int OUT, bool UPF16>
hipError_t launch_k(tab::LaunchArgs& A, const LevelDesc& L, int32_t n_batch, const tab::Slots<W>& sl, hipStream_t st)
{
    set_plain<LB, W, OUT>(A, L);
    const uint64_t blocks = set_order<LB, W, OUT>(A, L);
    return launch_blocks(A, blocks, [&](unsigned gx) {
        hipLaunchKernelGGL((tab::k_march_table<LB, W, OUT, UPF16, false>), dim3(gx, (unsigned)n_batch),
                           dim3(march::kBlock), 0, st, A, sl);
    });
}

template <int LB>
hipError_t launch_lb(tab::LaunchArgs& A, const LevelDesc& L, const TableLaunch& io, hipStream_t st)
{
    if (io.sc) {
        tab::Slots<kInclSlots> sl;
        for (int w = 0; w < kInclSlots; ++w) {
            sl.sc[w] = io.sc[w];
            sl.wt[w] = io.wt[w];
        }
        if (io.J) return launch_k<LB, kInclSlots, tab::kOutJ, false>(A, L, io.n_batch, sl, st);
        return launch_k<LB, kInclSlots, tab::kOutMean, false>(A, L, io.n_batch, sl, st);
    }
    const tab::Slots<1> sl;
    if (io.J) {
        if (io.f16) return launch_k<LB, 1, tab::kOutJ, true>(A, L, io.n_batch, sl, st);
        return launch_k<LB, 1, tab::kOutJ, false>(A, L, io.n_batch, sl, st);
    }
    if (io.f16) return launch_k<LB, 1, tab::kOutF16, true>(A, L, io.n_batch, sl, st);
    return launch_k<LB, 1, tab::kOutMean, false>(A, L, io.n_batch, sl, st);
}

// The windows of one cascade, a launch each (LB = 16).
template <int OUT, bool UPF16>
hipError_t launch_windows(tab::LaunchArgs& A, const LevelTable& T, int32_t n_batch, bool fix, hipStream_t st)
{
    const tab::Slots<1> sl;
    const size_t per_tap = (T.win_start.size() - 1) / (fix ? 4 : 1);
    for (size_t w = 0; w + 1 < T.win_start.size(); ++w) {
        A.n_blocks = T.win_start[w + 1] - T.win_start[w];
        if (A.n_blocks == 0) continue;
        A.work = (const tab::Work*)T.work + T.win_start[w];
        A.lo = (int32_t)(w % per_tap) * kWindow;
        A.hi = A.lo + kWindow;
        A.tap = (int32_t)(w / per_tap);
        const uint32_t per_xcd = (A.n_blocks + march::kXcds - 1) / march::kXcds;
        A.chunk = make_fastdiv(per_xcd);
        const hipError_t e = launch_blocks(A, A.n_blocks, [&](unsigned gx) {
            const dim3 grid(gx, (unsigned)n_batch);
            if (OUT == tab::kOutMean && fix)
                hipLaunchKernelGGL((tab::k_march_table<tab::kLB, 1, tab::kOutMean, false, true, true>), grid,
                                   dim3(march::kBlock), 0, st, A, sl);
            else
                hipLaunchKernelGGL((tab::k_march_table<tab::kLB, 1, OUT, UPF16, true>), grid, dim3(march::kBlock), 0,
                                   st, A, sl);
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

namespace {
tab::LaunchArgs launch_args(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, const TableLaunch& io)
{
    tab::LaunchArgs A = level_args(L, T, nx, nz);
    A.has_up = L.has_up && io.up;
    A.F = (const char*)io.F;
    A.f_stride = (uint64_t)A.ncell * io.lanes * sizeof(float2);
    A.f_bytes = (uint32_t)A.f_stride;
    A.up = io.up;
    A.out = io.out;
    A.casc_stride = (uint64_t)io.casc_stride;
    A.slot_stride = (uint64_t)io.slot_stride;
    A.ebias = io.ebias;
    A.J = io.J;
    A.n_wave = io.n_wave;
    return A;
}
}  // namespace

tab::LaunchArgs tab::row_args(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, bool plain)
{
    static_assert(wave_probes<kLB, kInclSlots>() == 4, "the order of 4-probe wavefronts");
    LaunchArgs A = level_args(L, T, nx, nz);
    if (plain) A.n_active = A.px * A.pz;
    set_order<kLB, kInclSlots, kOutMean>(A, L);
    return A;
}

namespace {
template <int LB>
hipError_t launch_fix(tab::LaunchArgs& A, LevelDesc L, const TableLaunch& io, hipStream_t st)
{
    // the order of the even probes, with the 4 parities within each place
    fix_probes(A);
    L.px = A.px;
    L.pz = A.pz;
    L.tile_p = (L.tile_p + 1) / 2;
    L.xcd_chunk *= 4;
    const uint64_t blocks = 4 * set_order<LB, 1, tab::kOutMean>(A, L);
    A.n_blocks = (uint32_t)blocks;
    return launch_blocks(A, blocks, [&](unsigned gx) {
        const dim3 grid(gx, (unsigned)io.n_batch);
        if (io.J)
            hipLaunchKernelGGL((tab::k_march_fix_table<LB, tab::kOutJ>), grid, dim3(march::kBlock), 0, st, A);
        else
            hipLaunchKernelGGL((tab::k_march_fix_table<LB, tab::kOutMean>), grid, dim3(march::kBlock), 0, st, A);
    });
}
}  // namespace

size_t table_task_bytes() { return sizeof(tab::Task); }

uint64_t table_task(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, const TableLaunch& io,
                    uint32_t block0, void* task)
{
    tab::Task t{launch_args(L, T, nx, nz, io), block0};
    if (!io.J) set_plain<tab::kLB, 1, tab::kOutMean>(t.A, L);
    const uint64_t blocks = io.J      ? set_order<tab::kLB, 1, tab::kOutJ>(t.A, L)
                            : io.f16 ? set_order<tab::kLB, 1, tab::kOutF16>(t.A, L)
                                     : set_order<tab::kLB, 1, tab::kOutMean>(t.A, L);
    std::memcpy(task, &t, sizeof(t));
    return blocks * (uint64_t)io.n_batch;
}

hipError_t launch_table_tasks(const void* tasks, int32_t n, uint32_t blocks, bool j, bool f16, hipStream_t st)
{
    const auto* t = (const tab::Task*)tasks;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(blocks), dim3(march::kBlock), 0, st, t, n); };
    if (j && f16) go(tab::k_march_tasks<tab::kOutJ, true>);
    else if (j) go(tab::k_march_tasks<tab::kOutJ, false>);
    else if (f16) go(tab::k_march_tasks<tab::kOutF16, true>);
    else go(tab::k_march_tasks<tab::kOutMean, false>);
    return hipGetLastError();
}

hipError_t launch_march_table(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, const TableLaunch& io,
                              hipStream_t st)
{
    tab::LaunchArgs A = launch_args(L, T, nx, nz, io);
    if (io.state) {
        A.state = io.state;
        if (io.fix) fix_probes(A);
        if (io.f16) return launch_windows<tab::kOutF16, true>(A, T, io.n_batch, false, st);
        return launch_windows<tab::kOutMean, false>(A, T, io.n_batch, io.fix, st);
    }
    if (io.fix) {
        switch (io.lanes) {
        case 1: return launch_fix<1>(A, L, io, st);
        case 2: return launch_fix<2>(A, L, io, st);
        case 4: return launch_fix<4>(A, L, io, st);
        case 8: return launch_fix<8>(A, L, io, st);
        case 16: return launch_fix<16>(A, L, io, st);
        }
        return hipErrorInvalidValue;
    }
    switch (io.lanes) {
    case 1: return launch_lb<1>(A, L, io, st);
    case 2: return launch_lb<2>(A, L, io, st);
    case 4: return launch_lb<4>(A, L, io, st);
    case 8: return launch_lb<8>(A, L, io, st);
    case 16: return launch_lb<16>(A, L, io, st);
    }
    return hipErrorInvalidValue;
}

namespace {
template <int LB, int OUT, bool UPF16>
hipError_t launch_two(tab::LaunchArgs& A, tab::LaunchArgs& B, const LevelDesc& L, int32_t n_batch, hipStream_t st)
{
    auto up8 = [](uint64_t b) { return (b + march::kXcds - 1) / march::kXcds * march::kXcds; };
    set_plain<tab::kLB, 1, OUT>(A, L);
    set_plain<LB, 1, OUT>(B, L);
    const uint64_t a = up8(set_order<tab::kLB, 1, OUT>(A, L)), b = up8(set_order<LB, 1, OUT>(B, L));
    if (a == 0) return hipSuccess;  // (nothing flagged)
    if (a * n_batch + b > kMaxGridX) {
        const hipError_t e = launch_k<tab::kLB, 1, OUT, UPF16>(A, L, n_batch, tab::Slots<1>{}, st);
        return e != hipSuccess ? e : launch_k<LB, 1, OUT, UPF16>(B, L, 1, tab::Slots<1>{}, st);
    }
    hipLaunchKernelGGL((tab::k_march_two<LB, OUT, UPF16>), dim3((unsigned)(a * n_batch + b)), dim3(march::kBlock), 0, st,
                       A, B, (uint32_t)b, make_fastdiv((uint32_t)a));
    return hipGetLastError();
}
template <int LB>
hipError_t launch_two_lb(tab::LaunchArgs& A, tab::LaunchArgs& B, const LevelDesc& L, const TableLaunch& io,
                         hipStream_t st)
{
    if (io.J && io.f16) return launch_two<LB, tab::kOutJ, true>(A, B, L, io.n_batch, st);
    if (io.J) return launch_two<LB, tab::kOutJ, false>(A, B, L, io.n_batch, st);
    if (io.f16) return launch_two<LB, tab::kOutF16, true>(A, B, L, io.n_batch, st);
    return launch_two<LB, tab::kOutMean, false>(A, B, L, io.n_batch, st);
}
}  // namespace

hipError_t launch_march_table2(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, const TableLaunch& io,
                               const TableLaunch& last, hipStream_t st)
{
    tab::LaunchArgs A = launch_args(L, T, nx, nz, io), B = launch_args(L, T, nx, nz, last);
    switch (last.lanes) {
    case 1: return launch_two_lb<1>(A, B, L, io, st);
    case 2: return launch_two_lb<2>(A, B, L, io, st);
    case 4: return launch_two_lb<4>(A, B, L, io, st);
    case 8: return launch_two_lb<8>(A, B, L, io, st);
    }
    return hipErrorInvalidValue;
}

namespace {
// Entries inside the domain of a cascade's rays that reach into it, on average
// (from 9 x 9 places in 32 directions).
double mean_run(const rcx_grid& g, const LevelDesc& L)
{
    constexpr int kPlaces = 9, kDirs = 32;
    double sum = 0.0, rays = 0.0;
    for (int k = 0; k < kDirs; ++k) {
        const double th = 2.0 * M_PI * (k + 0.5) / kDirs, c = std::cos(th), s = std::sin(th);
        for (int j = 0; j < kPlaces * kPlaces; ++j) {
            const double x = g.nx * (j % kPlaces + 0.5) / kPlaces, z = g.nz * (j / kPlaces + 0.5) / kPlaces;
            const double end = std::min(
                {L.tb, (c > 0.0 ? g.nx - x : x) / std::fabs(c), (s > 0.0 ? g.nz - z : z) / std::fabs(s)});
            if (end <= L.ta) continue;
            sum += (end - L.ta) * (std::fabs(c) + std::fabs(s));
            rays += 1.0;
        }
    }
    return rays > 0.0 ? sum / rays : 0.0;
}
}  // namespace

hipError_t build_windows(const rcx_grid& g, const LevelDesc& L, const double4* dirs, bool fix, LevelTable& T)
{
    T.win_start.clear();
    if (T.work) (void)hipFree(T.work);
    T.work = nullptr;
    if (!T.dirs || (L.plist && (fix || L.n_active == 0))) return hipSuccess;
    // windows pay where a cascade's rays are longer than a window and a
    // batch's fields larger than an XCD's L2 (4 MB). The length that counts is
    // that inside the domain, of the rays that reach into it: a widest cascade
    // that mostly points out of the domain fills its later windows with a few
    // rays each (one batch of 16 wavelengths on 256^2, cascade 4 of 99 entries
    // a ray: 152 us in windows, 123 whole; on 512^2, cascade 5 of 104: 286 and
    // 239), while 113 entries on 300 x 600 break even and 214 on 260 x 1000
    // gain (0.53 ms in windows, 1.2 whole)
    const double reach = std::min(L.tb, std::hypot((double)g.nx, (double)g.nz)) - L.ta;
    if (reach <= kWindow || mean_run(g, L) < kWindow || (int64_t)g.nx * g.nz * tab::kLB * 8 < (int64_t(8) << 20)) return hipSuccess;
    WindowGeom G{};
    G.A = level_args(L, T, g.nx, g.nz);
    G.fix = fix;
    const uint32_t taps = fix ? 4 : 1;
    if (fix) fix_probes(G.A);
    auto subs = [](int32_t a, int32_t b, int32_t na, int32_t nb) {
        return (uint32_t)((a + na - 1) / na) * (uint32_t)((b + nb - 1) / nb);
    };
    constexpr int32_t per = tab::kWinLong * tab::kWinShort;
    G.n_sub = L.plist ? (uint32_t)((L.n_active + per - 1) / per)
                      : std::max(subs(G.A.px, G.A.pz, tab::kWinShort, tab::kWinLong),
                                 subs(G.A.px, G.A.pz, tab::kWinLong, tab::kWinShort)) * taps;  // (fix: 4 parities)
    G.n_cone = (uint32_t)L.nd / 4;
    G.s = L.s;
    G.ta = L.ta;
    G.n_win = (T.max_entries - 1) / kWindow + 1;
    if ((uint64_t)G.n_sub * G.n_cone >= (1ull << 31)) return hipSuccess;
    size_t n_bin;
    for (G.region = kRegion;; G.region *= 2) {
        G.nrx = (g.nx + G.region - 1) / G.region;
        G.nrz = (g.nz + G.region - 1) / G.region;
        n_bin = (size_t)taps * G.n_win * G.nrx * G.nrz * kDirBins;
        if (n_bin <= kMaxBins || G.nrx * G.nrz == 1) break;
    }
    uint32_t* bins = nullptr;
    hipError_t e = hipMalloc(&bins, n_bin * sizeof(uint32_t));
    if (e != hipSuccess) return e;
    const unsigned grid = (G.n_sub * G.n_cone + 255) / 256;
    std::vector<uint32_t> h;
    try {
        h.resize(n_bin);
        T.win_start.reserve((size_t)taps * G.n_win + 1);
    } catch (const std::bad_alloc&) {
        (void)hipFree(bins);
        return hipErrorOutOfMemory;
    }
    e = hipMemset(bins, 0, n_bin * sizeof(uint32_t));
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_windows, dim3(grid, taps), dim3(256), 0, nullptr, G, dirs, bins, (tab::Work*)nullptr);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(h.data(), bins, n_bin * sizeof(uint32_t), hipMemcpyDeviceToHost);
    if (e == hipSuccess) {
        uint32_t at = 0;
        const size_t per_win = n_bin / (size_t)G.n_win / taps;
        for (size_t b = 0; b < n_bin; ++b) {
            if (b % per_win == 0) T.win_start.push_back(at);
            const uint32_t c = h[b];
            h[b] = at;
            at += c;
        }
        T.win_start.push_back(at);
        e = hipMalloc(&T.work, std::max<size_t>(at, 1) * sizeof(tab::Work));
        if (e == hipSuccess) e = hipMemcpy(bins, h.data(), n_bin * sizeof(uint32_t), hipMemcpyHostToDevice);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_windows, dim3(grid, taps), dim3(256), 0, nullptr, G, dirs, bins, (tab::Work*)T.work);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    }
    (void)hipFree(bins);
    if (e != hipSuccess) {
        if (T.work) (void)hipFree(T.work);
        T.work = nullptr;
        T.win_start.clear();
    }
    return e;
}

}  // namespace rcx
