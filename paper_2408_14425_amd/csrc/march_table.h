// march_table.h -- the radiance-interval march + merge of the field solves
// from per-direction segment tables (Osborne & Sannikov, arXiv:2408.14425,
// Secs. 2.2-2.3 and 3.2).
//
// The probes of a cascade sit whole cells apart, so every ray of one
// direction crosses the same cells relative to its probe's cell, with the
// same segment lengths: the list {cell offset, length} of a direction is
// walked once, in FP64, when the plan is made (k_build_tables), and a march
// reads it instead of walking. A wavefront marches one direction from
// 64 V / LB probes, LB wavelengths each (V per lane), so the list is read with scalar loads
// and a step's cell offset is added to the scalar base address of the load:
// no LDS, no FP64 and no per-lane address arithmetic in the step loop (10
// VALU instructions per step; the walking march issues 16.7 per step with
// its walk, set-up and merge). What a ray may step through is a run of the
// list, [first entry inside the domain, first entry beyond it), found from
// the plane-crossing indices of the direction (DirTable::ix, iz).
//
// A workgroup's 4 wavefronts are the 4 children 4g..4g+3 of one cone of the
// cascade below. The merge only ever reads the mean of those 4, so that mean
// is what the cascade buffers hold in FP32 (a quarter of the values written,
// 4 loads per ray instead of 16); with 16-bit cascades every direction's code
// is kept, as the walking march stores them.
//
// What bounds it: VALU issue on the cascades whose cells stay in the L2 (the
// step's 10 instructions, one of them a quarter-rate exponential, allow about
// 0.31 instructions per SIMD and cycle; cascade 3 of a 1024^2 grid reaches
// 0.25), then the L1's one access per cycle and CU: 16 wavelengths on 16
// lanes of 8 bytes took 16 accesses per wavefront load and bound the march;
// 8 lanes of 16 bytes (V = 2) take half, and serve 8 probes per wavefront.
// 1024^2 x 64 wavelengths, ms per solve (cascades 0..5): walking march 86.2
// (2.1 2.2 4.4 11.2 34 34), tables with V = 1 88 (1.3 1.6 3.1 10.2 35 43: the
// wide cascades bound by L2 misses), V = 2 97 (0.9 1.0 2.3 7.4 41 47),
// V = 2 in windows 60 (0.7 1.0 2.2 7.1 23 26; march_table.hip).
#pragma once

#include "march_rows.h"

namespace rcx {
namespace tab {

using march::kBlock;
using march::kLB;

// One direction's list: n entries at `off`, progress (cells crossed along
// +-x and +-z, from the probe's cell) of the first and last entry, and the
// first entry at progress >= P for P in (px0, px1] at idx[ix + P - px0]
// (likewise iz).
struct DirTable {
    uint32_t off;
    int32_t n;
    int32_t px0, px1, pz0, pz1;
    uint32_t ix, iz;
    int32_t xpos, zpos;  // 1 when the direction's x (z) component is positive
    int32_t xmaj;        // 1 when |x| >= |z| (of the cone: its 4 directions march from the same probes)
    int32_t cap;         // entries allocated (before the padding)
};
// a segment: cell offset x 128 B (the bytes of 16 wavelengths), length in cells
struct Segment {
    int32_t key;
    float ds;
};
// One workgroup of a windowed march: sub-block of probes, cone, and whether
// no later window holds entries of its rays (it then merges and stores them).
struct Work {
    uint32_t sub, cone_final;  // cone * 2 + final
};
constexpr int kSegPad = 8;  // entries readable past a list's end
static_assert(kMaxGridX % march::kXcds == 0, "launches start on the first XCD");

struct LaunchArgs {
    // geometry
    int32_t nx, nz, px, pz, nd, qx, qz, has_up;
    int32_t is, half;  // probe spacing; the probe's cell is (u is + half, v is + half)
    const DirTable* dirs;
    const Segment* segs;
    const uint32_t* idx;
    // launch order: workgroup -> (tile, wedge of cones) group, then cone
    // (fastest), then the sub-block of probes a wavefront takes
    uint32_t n_blocks;
    uint32_t block0 = 0;     // this launch's first workgroup (kMaxGridX at a time)
    FastDiv per, nwedge, wd, nb_long, ntx, chunk, chunk8;
    int32_t tile_x, tile_z;  // probes of a tile
    int32_t tw_log2, th;     // sub-block: 2^tw_log2 x th probes, x th <-> z on z-long sub-blocks
    int32_t orient;          // 1: sub-blocks run along the direction's minor axis
    const int32_t* plist;    // sparse: flagged probes (tile = tile_x consecutive entries)
    int32_t n_active;        // > 0 without a list: every probe, in plain order
    FastDiv pxdiv, pzdiv;
    // windowed march: this window's workgroups, entries [lo, hi) of every list
    const Work* work;
    int32_t lo, hi;
    FastDiv sub_x, sub_z;  // sub-blocks per row of probes: x-major directions, z-major ones
    float* state;          // {I, T} of every ray between windows, [ray][LB][2]
    // bilinear fix: px, pz above are those of the even probes
    int32_t full_px, full_pz;
    int32_t tap;           // windowed: the tap 2 z + x this launch traces
    // data; blockIdx.y = wavelength batch, strides in bytes (F) and elements
    const char* F;
    uint64_t f_stride;
    uint32_t f_bytes;
    const void* up;
    void* out;
    uint64_t casc_stride;  // elements between batches of the cascade buffers
    uint64_t slot_stride;  // elements between the inclination slots of one batch
    const int32_t* ebias;  // [batch][16]
    // J
    float* J;
    int64_t ncell;
    int32_t n_wave;        // wavelengths of this launch's batches
};

template <int W>
struct Slots {
    float sc[W], wt[W];
};
template <>
struct Slots<1> {};

// The sub-block of a workgroup in a windowed march: kWinLong x kWinShort
// probes, the long side along the directions' minor axis.
constexpr int kWinLong = 4, kWinShort = 2;

enum Out : int { kOutMean = 0, kOutJ = 1, kOutF16 = 2 };

// Wavelengths per lane V: 2 where a row has at least 2 (one 16-byte load per
// step and lane), 1 with the inclination slots, whose step already serves 8.
template <int LB, int W>
constexpr int lane_waves()
{
    return W == 1 && LB >= 2 ? 2 : 1;
}
// Probes of a wavefront: rows of LB / V lanes.
template <int LB, int W>
constexpr int wave_probes()
{
    return 64 / LB * lane_waves<LB, W>();
}
// Sub-blocks of probes a wavefront takes in turn. On cascade 0 a workgroup
// covers 16 consecutive cells, so J is written 64 bytes at a time.
template <int LB, int W, int OUT>
constexpr int sub_blocks()
{
    return OUT == kOutJ && wave_probes<LB, W>() < 16 ? 16 / wave_probes<LB, W>() : 1;
}

__device__ __forceinline__ Segment load_seg(const Segment* p)
{
    // read-only for the launch and wave-uniform: scalar loads
    typedef const __attribute__((address_space(4))) uint64_t* cptr;
    const uint64_t v = *(cptr)(uintptr_t)p;
    return Segment{(int32_t)(uint32_t)v, __uint_as_float((uint32_t)(v >> 32))};
}

// A read-only, wave-uniform struct by scalar loads.
template <class T>
__device__ __forceinline__ T load_uniform(const T* p)
{
    typedef const __attribute__((address_space(4))) uint32_t* cptr;
    static_assert(sizeof(T) % 4 == 0, "copied by words");
    const cptr src = (cptr)(uintptr_t)p;
    uint32_t words[sizeof(T) / 4];
#pragma unroll
    for (uint32_t i = 0; i < sizeof(T) / 4; ++i) words[i] = src[i];
    T t;
    __builtin_memcpy(&t, words, sizeof(T));
    return t;
}

// {optical depth per cell, S} of V wavelengths at base + key + voff: the uniform part is added
// on the scalar unit and stays there (the empty asm keeps the compiler from
// moving it into a 64-bit vector add per step), voff is the load's 32-bit
// vector offset.
template <int V>
struct Cell {
    typedef uint32_t raw __attribute__((ext_vector_type(2 * V)));
    raw r;
    __device__ __forceinline__ float2 get(int i) const
    {
        return make_float2(__uint_as_float(r[2 * i]), __uint_as_float(r[2 * i + 1]));
    }
};
template <int V>
__device__ __forceinline__ Cell<V> load_cell(const char* base, int32_t key, uint32_t voff)
{
    typedef const __attribute__((address_space(1))) char* gptr;
    typedef const __attribute__((address_space(1))) typename Cell<V>::raw* rptr;
    uint64_t b = (uint64_t)(uintptr_t)base + (uint64_t)(int64_t)key;
    asm("" : "+s"(b));
    return Cell<V>{*(rptr)((gptr)b + voff)};
}
template <int V>
__device__ __forceinline__ Cell<V> load_cell_checked(__amdgpu_buffer_rsrc_t rsrc, uint32_t off)
{
    if constexpr (V == 1)
        return Cell<V>{__builtin_bit_cast(typename Cell<V>::raw, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0))};
    else
        return Cell<V>{__builtin_bit_cast(typename Cell<V>::raw, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0))};
}

template <int LB>
constexpr int lb_log2()
{
    return LB == 16 ? 4 : LB == 8 ? 3 : LB == 4 ? 2 : LB == 2 ? 1 : 0;
}

// The run [a, e) of direction D's list inside the domain, for the probe in
// cell (X0, Z0). The domain and the path are convex and monotone, so it is
// one run; probes may lie past the far edge of a ragged grid (their rays can
// enter the domain later).
__device__ __forceinline__ void clip_run(const DirTable& D, const uint32_t* __restrict__ idx, int nx, int nz, int X0,
                                         int Z0, int& a, int& e)
{
    const int Ex = D.xpos ? nx - X0 : X0 + 1, Ez = D.zpos ? nz - Z0 : Z0 + 1;    // progress that leaves
    const int Nx = D.xpos ? -X0 : X0 - nx + 1, Nz = D.zpos ? -Z0 : Z0 - nz + 1;  // progress that has entered
    auto first = [&](int P, int p0, int p1, uint32_t base) {
        if (P <= p0) return 0;
        if (P > p1) return D.n;
        return (int)idx[base + (uint32_t)(P - p0)];
    };
    a = max(first(Nx, D.px0, D.px1, D.ix), first(Nz, D.pz0, D.pz1, D.iz));
    e = min(first(Ex, D.px0, D.px1, D.ix), first(Ez, D.pz0, D.pz1, D.iz));
    if (a >= e) a = e = 0;
}

// Probe of row `row` of sub-block `sub` in a windowed march (dense).
__device__ __forceinline__ void window_probe(const LaunchArgs& A, uint32_t sub, bool xmaj, int row, int& u, int& v,
                                             bool& active)
{
    const FastDiv& d = xmaj ? A.sub_x : A.sub_z;
    const int sv = (int)d.div(sub), su = (int)(sub - (uint32_t)sv * d.d);
    const int rl = row % kWinLong, rs = row / kWinLong;
    u = xmaj ? su * kWinShort + rs : su * kWinLong + rl;
    v = xmaj ? sv * kWinLong + rl : sv * kWinShort + rs;
    active = u < A.px && v < A.pz;
    u = min(u, A.px - 1);
    v = min(v, A.pz - 1);
}

template <int LPR>
__device__ __forceinline__ int rows_min(int x)
{
#pragma unroll
    for (int m = LPR; m < 64; m *= 2) x = min(x, __shfl_xor(x, m));
    return __builtin_amdgcn_readfirstlane(x);
}
template <int LPR>
__device__ __forceinline__ int rows_max(int x)
{
#pragma unroll
    for (int m = LPR; m < 64; m *= 2) x = max(x, __shfl_xor(x, m));
    return __builtin_amdgcn_readfirstlane(x);
}

template <int LB, int W>
struct Ray {
    static constexpr int V = lane_waves<LB, W>();
    float I[W * V], T[W * V];  // slot w of wavelength i at [w * V + i]
    __device__ __forceinline__ void step(const Cell<V>& c, float ds, const Slots<W>& sl)
    {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const float2 f = c.get(i);
            if constexpr (W == 1) {
                march::step(f, ds, I[i], T[i]);
            } else {
#pragma unroll
                for (int w = 0; w < W; ++w)
                    march::step(make_float2(f.x * sl.sc[w], f.y), ds, I[w * V + i], T[w * V + i]);
            }
        }
    }
    // entries [s, s + N) of the list, every row inside the domain
    template <int N>
    __device__ __forceinline__ void full(const Segment* seg, const char* Fb, uint32_t voff, const Slots<W>& sl)
    {
        Segment g[N];
        Cell<V> f[N];
#pragma unroll
        for (int q = 0; q < N; ++q) g[q] = load_seg(seg + q);
        // (tied to the group's entries, so its zero extension stays beside the
        // loads, where it folds into their scalar-base form)
        asm("" : "+v"(voff) : "s"(g[0].key));
#pragma unroll
        for (int q = 0; q < N; ++q) f[q] = load_cell<V>(Fb, g[q].key >> (4 - lb_log2<LB>()), voff);
#pragma unroll
        for (int q = 0; q < N; ++q) step(f[q], g[q].ds, sl);
    }
    // entries [s, e) where some rows are outside the domain (a null read:
    // no opacity, no emission)
    __device__ __forceinline__ void edge(const Segment* seg, int s, int e, __amdgpu_buffer_rsrc_t rsrc, uint32_t voff,
                                         int ra, int re, const Slots<W>& sl)
    {
        // entries past e belong to the other loops or to the padding
        const uint32_t len = (uint32_t)max(min(re, e) - ra, 0);
        for (; s < e; s += 4) {
            Cell<V> f[4];
            float ds[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const Segment g = load_seg(seg + s + q);  // at most 3 past the end (padded)
                ds[q] = g.ds;
                const bool in = (uint32_t)(s + q - ra) < len;
                const uint32_t o = in ? voff + (uint32_t)(g.key >> (4 - lb_log2<LB>())) : 0x80000000u;
                f[q] = load_cell_checked<V>(rsrc, o);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) step(f[q], ds[q], sl);
        }
    }
    // entries [s0, smax) of the list, of which a row takes [a, e): all rows'
    // in [s0, s1) when no ray of the wavefront leaves the domain (!part)
    __device__ __forceinline__ void run(const Segment* seg, const char* Fb, __amdgpu_buffer_rsrc_t rsrc, uint32_t voff,
                                        bool part, int s0, int s1, int smax, int a, int e, const Slots<W>& sl)
    {
        constexpr int LPR = LB / V;
        if (part) {
            int smin = s0;
            if (__ballot(a != smin) != 0) {
                s0 = rows_max<LPR>(a);
                smin = rows_min<LPR>(a);
            }
            s1 = rows_min<LPR>(e);
            smax = rows_max<LPR>(e);
            if (s0 >= s1) s0 = s1 = smax;
            edge(seg, smin, s0, rsrc, voff, a, e, sl);
        }
        int s = s0;
        constexpr int U = W == 1 ? 8 : 4;
#pragma unroll 1
        for (; s + U <= s1; s += U) full<U>(seg + s, Fb, voff, sl);
        if constexpr (U == 8)
            if (s + 4 <= s1) {
                full<4>(seg + s, Fb, voff, sl);
                s += 4;
            }
        if (s + 2 <= s1) {
            full<2>(seg + s, Fb, voff, sl);
            s += 2;
        }
        if (s < s1) full<1>(seg + s, Fb, voff, sl);
        edge(seg, s1, smax, rsrc, voff, a, e, sl);
    }
};

template <int V>
struct alignas(4 * V) Pack32 {
    float v[V];
};
template <int V>
struct alignas(2 * V) Pack16 {
    uint16_t v[V];
};

// Bilinear fix: tap (ax, az) of probe (u, v) of the cascade above. Where both
// taps of an axis clamp to the same probe, the inside one takes the weight of
// both and the other has no ray.
constexpr int kFixClasses = 16;  // lists per direction (k_march_fix_table)
struct FixTap {
    int qu, qv;
    float w;
    bool in, first;  // this tap has a ray; it is the probe's first one that has
    __host__ __device__ FixTap(int u, int v, int ax, int az, int qx, int qz)
    {
        const int bu = (u - 1) >> 1, bv = (v - 1) >> 1;
        qu = bu + ax;
        qv = bv + az;
        in = qu >= 0 && qu < qx && qv >= 0 && qv < qz;
        first = ax == (bu < 0) && az == (bv < 0);
        const int ou = bu + 1 - ax, ov = bv + 1 - az;
        const float fx = u & 1 ? 0.25f : 0.75f, fz = v & 1 ? 0.25f : 0.75f;
        w = (ou < 0 || ou >= qx ? 1.0f : ax ? fx : 1.0f - fx) * (ov < 0 || ov >= qz ? 1.0f : az ? fz : 1.0f - fz);
    }
};
__host__ __device__ __forceinline__ uint32_t fix_class(int pu, int pv, int ax, int az)
{
    return 4u * (uint32_t)(2 * az + pv) + (uint32_t)(2 * ax + pu);
}

// One workgroup: 4 directions of a cone from the probes of place lb in the
// launch order (windowed: of entry lb of the window's list), wavelength batch
// `batch`.
template <int LB, int W, int OUT, bool UPF16, bool WIN, bool TASK = false, bool FIX = false>
__device__ __forceinline__ void march_table(const LaunchArgs& A, const Slots<W>& sl, uint32_t lb, const uint32_t batch)
{
    static_assert(!WIN || (W == 1 && OUT != kOutJ && wave_probes<LB, W>() == kWinLong * kWinShort),
                  "windowed march: one sub-block per wavefront, flatland, cascades above 0");
    static_assert(!FIX || (WIN && OUT == kOutMean && !UPF16), "whole cascades with the fix: k_march_fix_table");
    constexpr int V = lane_waves<LB, W>(), LPR = LB / V;  // lanes per row
    constexpr int PW = wave_probes<LB, W>();
    constexpr int NS = sub_blocks<LB, W, OUT>();
    // [..][wavelength of the lane][lane]
    __shared__ float red[OUT == kOutMean ? W : 1][OUT == kOutF16 ? 1 : 4][NS][V][64];
    const int lane = threadIdx.x & 63, l = (lane & (LPR - 1)) * V, row = lane / LPR;  // l: first wavelength
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    uint32_t t = 0, cone, sb = 0, bl = 0, bs = 0, tz = 0, tx = 0;
    bool final = true;
    if constexpr (WIN) {
        const Work wk = A.work[lb];
        sb = wk.sub;
        cone = wk.cone_final >> 1;
        final = (wk.cone_final & 1u) != 0;
    } else {
        const uint32_t g = A.per.div(lb), rin = lb - g * A.per.d;
        t = A.nwedge.div(g);
        sb = A.wd.div(rin);
        cone = (g - t * A.nwedge.d) * A.wd.d + (rin - sb * A.wd.d);
        bl = A.nb_long.div(sb);
        bs = sb - bl * A.nb_long.d;
        tz = A.ntx.div(t);
        tx = t - tz * A.ntx.d;
    }
    const int k = (int)(4 * cone) + wave;
    DirTable D;
    if constexpr (TASK) D = load_uniform(A.dirs + k);
    else if constexpr (FIX) D = A.dirs[k * kFixClasses + fix_class(sb & 1, (sb >> 1) & 1, A.tap & 1, A.tap >> 1)];
    else D = A.dirs[k];
    const bool swap = A.orient && D.xmaj;

    const char* Fb = A.F + batch * A.f_stride;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Fb, 0, (int)A.f_bytes, 0x00020000);
    const Segment* seg = A.segs + D.off;
    int32_t B16[V] = {};
    if constexpr (UPF16 || OUT == kOutF16) {
#pragma unroll
        for (int i = 0; i < V; ++i) B16[i] = A.ebias[batch * kLB + l + i] * 1024;
    }

    int u = 0, v = 0;
    bool active = true;
#pragma unroll 1
    for (int ns = 0; ns < NS; ++ns) {
        if constexpr (FIX) {
            window_probe(A, sb >> 2, D.xmaj, row, u, v, active);
            u = 2 * u + (int)(sb & 1u);
            v = 2 * v + (int)((sb >> 1) & 1u);
            active = active && u < A.full_px && v < A.full_pz;
            u = min(u, A.full_px - 1);
            v = min(v, A.full_pz - 1);
        } else if (WIN && !A.plist) {
            window_probe(A, sb, D.xmaj, row, u, v, active);
        } else if (A.n_active) {
            const uint32_t i = t * (uint32_t)A.tile_x + (sb * NS + (uint32_t)ns) * PW + (uint32_t)row;
            active = i < (uint32_t)A.n_active;
            uint32_t p = active ? i : (uint32_t)A.n_active - 1u;
            if (A.plist) p = (uint32_t)A.plist[p];
            if (A.plist || !D.xmaj) {
                v = (int)A.pxdiv.div(p);
                u = (int)(p - (uint32_t)v * A.pxdiv.d);
            } else {
                u = (int)A.pzdiv.div(p);
                v = (int)(p - (uint32_t)u * A.pzdiv.d);
            }
        } else {
            const int tw = 1 << A.tw_log2;
            const int al = (int)(bs * NS + ns) * tw + (row & (tw - 1)), as = (int)bl * A.th + (row >> A.tw_log2);
            u = (int)tx * A.tile_x + (swap ? as : al);
            v = (int)tz * A.tile_z + (swap ? al : as);
            active = u < A.px && v < A.pz;
            u = min(u, A.px - 1);
            v = min(v, A.pz - 1);
        }
        const int X0 = u * A.is + A.half, Z0 = v * A.is + A.half;
        const uint32_t voff = (uint32_t)(Z0 * A.nx + X0) * (uint32_t)(LB * 8) + (uint32_t)l * 8u;

        Ray<LB, W> r;
#pragma unroll
        for (int w = 0; w < W * V; ++w) {
            r.I[w] = 0.0f;
            r.T[w] = 1.0f;
        }
        // the whole list of every row inside the domain (most rays of the
        // lower cascades), else the rows' runs
        const int Ex = D.xpos ? A.nx - X0 : X0 + 1, Ez = D.zpos ? A.nz - Z0 : Z0 + 1;
        bool whole = Ex > D.px1 && Ez > D.pz1 && X0 < A.nx && Z0 < A.nz;
        if constexpr (FIX) {  // (its rays do not start on their probe)
            const int Nx = D.xpos ? -X0 : X0 - A.nx + 1, Nz = D.zpos ? -Z0 : Z0 - A.nz + 1;
            active = active && FixTap(u, v, A.tap & 1, A.tap >> 1, A.qx, A.qz).in;
            whole = active && Ex > D.px1 && Ez > D.pz1 && Nx <= D.px0 && Nz <= D.pz0;
        }
        int s0 = WIN ? A.lo : 0, s1 = WIN ? min(D.n, A.hi) : D.n;
        int a = 0, e = D.n, smax = s1;
        bool more = false;  // windowed: this row has entries in this window
        const uint64_t so =
            WIN ? (((uint64_t)(uint32_t)(v * (FIX ? A.full_px : A.px) + u) * (uint32_t)A.nd + (uint32_t)k) * LB +
                   (uint32_t)l) * 2u
                : 0u;
        bool part = __ballot(!whole) != 0;
        if (!WIN && __ballot(active) == 0) {
            // no probe here (a sub-block past a ragged edge)
            part = false;
            s1 = smax = 0;
        }
        if (part) clip_run(D, A.idx, A.nx, A.nz, X0, Z0, a, e);
        if constexpr (FIX)
            if (!active) a = e = 0;
        if constexpr (WIN) {
            if (e > a && a < A.lo) {
                // marched up to lo by earlier windows
                const Pack32<2 * V> st = *reinterpret_cast<const Pack32<2 * V>*>(A.state + so);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    r.I[i] = st.v[2 * i];
                    r.T[i] = st.v[2 * i + 1];
                }
            }
            a = max(a, A.lo);
            e = min(e, A.hi);
            more = a < e;
            if (!more) a = e = A.lo;
            smax = max(s1, A.lo);
            s1 = smax;
        }
        r.run(seg, Fb, rsrc, voff, part, s0, s1, smax, a, e, sl);
        if constexpr (WIN) {
            if (!final) {
                if (more && active) {
                    Pack32<2 * V> st;
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        st.v[2 * i] = r.I[i];
                        st.v[2 * i + 1] = r.T[i];
                    }
                    *reinterpret_cast<Pack32<2 * V>*>(A.state + so) = st;
                }
                return;
            }
        }

        if (FIX && A.has_up) {
            const FixTap q(u, v, A.tap & 1, A.tap >> 1, A.qx, A.qz);
            const uint32_t pi = active ? (uint32_t)(q.qv * A.qx + q.qu) : 0u;
            const Pack32<V> c = *reinterpret_cast<const Pack32<V>*>(
                (const float*)A.up + batch * A.casc_stride + ((pi * (uint32_t)A.nd + (uint32_t)k) * LB + (uint32_t)l));
#pragma unroll
            for (int i = 0; i < V; ++i) r.I[i] = fmaf(r.T[i], c.v[i], r.I[i]);
        } else if (A.has_up) {
            // bilinear taps on the cascade above (as march_ray)
            const int bx0 = (u - 1) >> 1, bz0 = (v - 1) >> 1;
            const float fx = (u & 1) ? 0.25f : 0.75f, fz = (v & 1) ? 0.25f : 0.75f;
            const int txs[2] = {min(max(bx0, 0), A.qx - 1), min(max(bx0 + 1, 0), A.qx - 1)};
            const int tzs[2] = {min(max(bz0, 0), A.qz - 1), min(max(bz0 + 1, 0), A.qz - 1)};
            const float wxs[2] = {1.0f - fx, fx}, wzs[2] = {1.0f - fz, fz};
            float far[W * V];
#pragma unroll
            for (int w = 0; w < W * V; ++w) far[w] = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float wq = wzs[q >> 1] * wxs[q & 1];
                const uint32_t pi = (uint32_t)(tzs[q >> 1] * A.qx + txs[q & 1]);
                if constexpr (UPF16) {
                    const uint16_t* up = (const uint16_t*)A.up + batch * A.casc_stride;
                    const uint32_t o = (pi * (uint32_t)(4 * A.nd) + 4u * (uint32_t)k) * LB + (uint32_t)l;
                    Pack16<V> c[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) c[j] = *reinterpret_cast<const Pack16<V>*>(up + (o + j * LB));
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        const float c4 = march::dec_h16(c[0].v[i], B16[i]) + march::dec_h16(c[1].v[i], B16[i]) +
                                         march::dec_h16(c[2].v[i], B16[i]) + march::dec_h16(c[3].v[i], B16[i]);
                        far[i] = fmaf(wq, 0.25f * c4, far[i]);
                    }
                } else {
                    const float* up = (const float*)A.up + batch * A.casc_stride;
                    const uint32_t o = (pi * (uint32_t)A.nd + (uint32_t)k) * LB + (uint32_t)l;
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const Pack32<V> c = *reinterpret_cast<const Pack32<V>*>(up + (w * A.slot_stride + o));
#pragma unroll
                        for (int i = 0; i < V; ++i) far[w * V + i] = fmaf(wq, c.v[i], far[w * V + i]);
                    }
                }
            }
#pragma unroll
            for (int w = 0; w < W * V; ++w) r.I[w] = fmaf(r.T[w], far[w], r.I[w]);
        }
        if constexpr (OUT == kOutF16) {
            uint16_t* out = (uint16_t*)A.out + batch * A.casc_stride;
            Pack16<V> c;
#pragma unroll
            for (int i = 0; i < V; ++i) c.v[i] = march::enc_h16(r.I[i], B16[i]);
            if (active)
                *reinterpret_cast<Pack16<V>*>(
                    out + (((uint32_t)(v * A.px + u) * (uint32_t)A.nd + (uint32_t)k) * LB + (uint32_t)l)) = c;
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                if constexpr (OUT == kOutJ && W > 1) {
                    float j = 0.0f;
#pragma unroll
                    for (int w = 0; w < W; ++w) j = fmaf(sl.wt[w], r.I[w * V + i], j);
                    red[0][wave][ns][i][lane] = j;
                } else {
#pragma unroll
                    for (int w = 0; w < W; ++w) red[w][wave][ns][i][lane] = r.I[w * V + i];
                }
            }
        }
    }
    if constexpr (OUT == kOutMean) {
        __syncthreads();
        // the mean of the 4 children, slot by slot on the 4 wavefronts (all
        // hold the same probes)
        const uint32_t o =
            ((uint32_t)(v * (FIX ? A.full_px : A.px) + u) * (uint32_t)(A.nd / 4) + cone) * LB + (uint32_t)l;
        float* out = (float*)A.out + batch * A.casc_stride;
        for (int w = wave; w < W; w += 4) {
            Pack32<V> c;
#pragma unroll
            for (int i = 0; i < V; ++i)
                c.v[i] = 0.25f * (red[w][0][0][i][lane] + red[w][1][0][i][lane] + red[w][2][0][i][lane] +
                                  red[w][3][0][i][lane]);
            if constexpr (FIX) {
                // weighted, added to the taps before it
                const FixTap q(u, v, A.tap & 1, A.tap >> 1, A.qx, A.qz);
                if (active) {
                    Pack32<V> sum{};
                    if (!q.first) sum = *reinterpret_cast<const Pack32<V>*>(out + (w * A.slot_stride + o));
#pragma unroll
                    for (int i = 0; i < V; ++i) c.v[i] = fmaf(q.w, c.v[i], sum.v[i]);
                }
            }
            if (active) *reinterpret_cast<Pack32<V>*>(out + (w * A.slot_stride + o)) = c;
        }
    } else if constexpr (OUT == kOutJ) {
        __syncthreads();
        // J of NS x PW probes x LB wavelengths, probes fastest over the threads
        constexpr int P = NS * PW;
        for (int j = (int)threadIdx.x; j < P * LB; j += kBlock) {
            const int p = j & (P - 1), jl = j / P, js = p / PW, i = jl % V;
            const int jlane = (p & (PW - 1)) * LPR + jl / V;
            const float val = (red[0][0][js][i][jlane] + red[0][1][js][i][jlane]) +
                              (red[0][2][js][i][jlane] + red[0][3][js][i][jlane]);
            int64_t cell;
            bool ok;
            if (A.plist) {
                const uint32_t n = t * (uint32_t)A.tile_x + sb * (uint32_t)P + (uint32_t)p;
                ok = n < (uint32_t)A.n_active;
                cell = ok ? A.plist[n] : 0;
            } else {
                const int tw = 1 << A.tw_log2, q = p & (PW - 1);
                const int cu = (int)tx * A.tile_x + (int)(bs * NS + js) * tw + (q & (tw - 1));
                const int cv = (int)tz * A.tile_z + (int)bl * A.th + (q >> A.tw_log2);
                ok = cu < A.px && cv < A.pz;
                cell = (int64_t)cv * A.px + cu;
            }
            const int lam = (int)batch * LB + jl;
            if (ok && lam < A.n_wave) A.J[(int64_t)lam * A.ncell + cell] = 0.25f * val;
        }
    }
}

// Place in the launch order of workgroup b: chunks of workgroups per XCD
// (march_rows.h, xcd_block_chunked).
__device__ __forceinline__ uint32_t place(const LaunchArgs& A, uint32_t b)
{
    const uint32_t c8 = A.chunk8.d, full = A.chunk8.div(A.n_blocks) * c8;
    if (b >= full) return b;
    const uint32_t x = b % march::kXcds, slot = b / march::kXcds;
    const uint32_t q = A.chunk.div(slot);
    return q * c8 + x * A.chunk.d + (slot - q * A.chunk.d);
}

template <int LB, int W, int OUT, bool UPF16, bool WIN, bool FIX = false>
__global__ __launch_bounds__(kBlock, W == 1 ? 8 : 4) void k_march_table(LaunchArgs A, Slots<W> sl)
{
    uint32_t lb = A.block0 + blockIdx.x;
    if constexpr (WIN) {
        // XCD x takes the x-th eighth of the window's list (sorted by region)
        lb = (lb % march::kXcds) * A.chunk.d + lb / march::kXcds;
    } else {
        lb = place(A, lb);
    }
    if (lb >= A.n_blocks) return;
    march_table<LB, W, OUT, UPF16, WIN, false, FIX>(A, sl, lb, blockIdx.y);
}

// A cascade of the whole batches (A) and of the last, narrower one (B, rows of
// LB lanes) in one launch, B's workgroups first: alone, a few wavelengths'
// rays are too few for the chip, and the launch lasts as long as its longest
// chain of loads (3 wavelengths on 333 x 200 took 220 us after 430 us of 16).
// b_grid (a multiple of the XCDs) workgroups are B's, then a_grid per batch of A.
template <int LB, int OUT, bool UPF16>
__global__ __launch_bounds__(kBlock, 8) void k_march_two(LaunchArgs A, LaunchArgs B, uint32_t b_grid, FastDiv a_grid)
{
    if (blockIdx.x < b_grid) {
        const uint32_t lb = place(B, blockIdx.x);
        if (lb < B.n_blocks) march_table<LB, 1, OUT, UPF16, false>(B, Slots<1>{}, lb, 0);
        return;
    }
    const uint32_t b = blockIdx.x - b_grid, batch = a_grid.div(b);
    const uint32_t lb = place(A, b - batch * a_grid.d);
    if (lb < A.n_blocks) march_table<kLB, 1, OUT, UPF16, false>(A, Slots<1>{}, lb, batch);
}

// The same cascade of several small atmospheres in one launch: task t holds
// workgroups [block0, block0 of the next), n_blocks per wavelength batch.
struct Task {
    LaunchArgs A;
    uint32_t block0;
};
template <int OUT, bool UPF16>
__global__ __launch_bounds__(kBlock, 8) void k_march_tasks(const Task* __restrict__ tasks, int32_t n)
{
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (tasks[mid].block0 <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const Task T = load_uniform(tasks + __builtin_amdgcn_readfirstlane(lo));
    // pointers read from memory are generic: these are global ones
    auto global = [](const void* p) {
        __builtin_assume(!__builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)p));
        __builtin_assume(!__builtin_amdgcn_is_private((const __attribute__((address_space(0))) void*)p));
    };
    global(T.A.dirs);
    global(T.A.segs);
    global(T.A.idx);
    global(T.A.plist);
    global(T.A.up);
    global(T.A.out);
    global(T.A.ebias);
    global(T.A.J);
    const uint32_t b = blockIdx.x - T.block0, batch = b / T.A.n_blocks;
    march_table<kLB, 1, OUT, UPF16, false, true>(T.A, Slots<1>{}, b - batch * T.A.n_blocks, batch);
}

// ----------------------------------------------------------- bilinear fix
// A cascade below the top of a plan with the bilinear fix (march_rows.h,
// march_fix_ray): the interval of probe p along w_k is traced once per tap q
// of the cascade above, from p + t_a w_k to q + t_b w_k. q - p is
// (c - 3/2) s along each axis, c = 0 and 2 for the two taps of an even probe
// and 1 and 3 for those of an odd one, so a direction has 16 lists, one per
// class 4 c_z + c_x, which all probes share. At the grid's edge both taps
// clamp to the same q: the list of the tap that is inside serves, with the
// weight of both (the other tap's ray is left out).
//
// A workgroup takes probes of one parity (x and z) and a cone; its 4
// wavefronts are the 4 taps, which cross nearly the same cells at the same
// time, and each marches the cone's 4 children in turn. The sums over taps
// and children meet in LDS: the cascade keeps the mean of the children (J on
// cascade 0). LaunchArgs describes the probes of one parity (px, pz =
// those of the even one); the parity is the fastest part of the order. Wide
// cascades are marched in windows instead (k_march_table, FIX), tap by tap,
// so the rays' state stays that of one tap. The walk of every tap
// (k_march_fix) issued about twice the instructions per step: 512^2 x 32
// wavelengths 26.2 -> 17.1 ms, 256^2 x 16 2.1 -> 1.4, 1024^2 x 16 96 -> 69
// (marched whole 103: the taps' rays cross more cells than an L2 holds).
// What bounds it is VALU issue, as the march without the fix, on 4 times its
// steps; a wavefront's probes lie 2 spacings apart, so on the widest cascade
// their rays end far apart (1.2 to 1.7 entries issued per entry used).
template <int LB, int OUT>
__global__ __launch_bounds__(kBlock, 8) void k_march_fix_table(LaunchArgs A)
{
    constexpr int V = lane_waves<LB, 1>(), LPR = LB / V, PW = wave_probes<LB, 1>();
    __shared__ float red[4][V][64];
    const int lane = threadIdx.x & 63, l = (lane & (LPR - 1)) * V, row = lane / LPR;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    uint32_t lb = place(A, A.block0 + blockIdx.x);
    if (lb >= A.n_blocks) return;
    const uint32_t batch = blockIdx.y;
    const int pu = (int)(lb & 1u), pv = (int)((lb >> 1) & 1u);
    lb >>= 2;
    const uint32_t g = A.per.div(lb), rin = lb - g * A.per.d;
    const uint32_t t = A.nwedge.div(g), sb = A.wd.div(rin);
    const uint32_t cone = (g - t * A.nwedge.d) * A.wd.d + (rin - sb * A.wd.d);
    const uint32_t bl = A.nb_long.div(sb), bs = sb - bl * A.nb_long.d;
    const uint32_t tz = A.ntx.div(t), tx = t - tz * A.ntx.d;
    const bool swap = A.orient && A.dirs[(4 * cone + 1) * kFixClasses + 5].xmaj;
    const int tw = 1 << A.tw_log2;
    const int al = (int)bs * tw + (row & (tw - 1)), as = (int)bl * A.th + (row >> A.tw_log2);
    int u = 2 * ((int)tx * A.tile_x + (swap ? as : al)) + pu, v = 2 * ((int)tz * A.tile_z + (swap ? al : as)) + pv;
    const bool active = u < A.full_px && v < A.full_pz;
    u = min(u, A.full_px - 1);
    v = min(v, A.full_pz - 1);

    const FixTap q(u, v, wave & 1, wave >> 1, A.qx, A.qz);  // this wavefront's tap
    const bool tap = active && q.in;
    const uint32_t cls = fix_class(pu, pv, wave & 1, wave >> 1);
    const uint32_t qi = tap ? (uint32_t)(q.qv * A.qx + q.qu) : 0u;

    const char* Fb = A.F + batch * A.f_stride;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Fb, 0, (int)A.f_bytes, 0x00020000);
    const int X0 = u * A.is + A.half, Z0 = v * A.is + A.half;
    const uint32_t voff = (uint32_t)(Z0 * A.nx + X0) * (uint32_t)(LB * 8) + (uint32_t)l * 8u;
    float sum[V];
#pragma unroll
    for (int i = 0; i < V; ++i) sum[i] = 0.0f;
#pragma unroll 1
    for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t k = 4u * cone + j;
        const DirTable D = A.dirs[k * kFixClasses + cls];
        Ray<LB, 1> r;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            r.I[i] = 0.0f;
            r.T[i] = 1.0f;
        }
        const int Ex = D.xpos ? A.nx - X0 : X0 + 1, Ez = D.zpos ? A.nz - Z0 : Z0 + 1;
        const int Nx = D.xpos ? -X0 : X0 - A.nx + 1, Nz = D.zpos ? -Z0 : Z0 - A.nz + 1;
        const bool whole = tap && Ex > D.px1 && Ez > D.pz1 && Nx <= D.px0 && Nz <= D.pz0;
        int a = 0, e = D.n;
        const bool part = __ballot(!whole) != 0;
        if (part) {
            clip_run(D, A.idx, A.nx, A.nz, X0, Z0, a, e);
            if (!tap) a = e = 0;
        }
        r.run(A.segs + D.off, Fb, rsrc, voff, part, 0, D.n, D.n, a, e, Slots<1>{});
        if (A.has_up) {
            const float* up = (const float*)A.up + batch * A.casc_stride;
            const Pack32<V> c = *reinterpret_cast<const Pack32<V>*>(up + ((qi * (uint32_t)A.nd + k) * LB + (uint32_t)l));
#pragma unroll
            for (int i = 0; i < V; ++i) r.I[i] = fmaf(r.T[i], c.v[i], r.I[i]);
        }
#pragma unroll
        for (int i = 0; i < V; ++i) sum[i] += r.I[i];
    }
#pragma unroll
    for (int i = 0; i < V; ++i) red[wave][i][lane] = tap ? (0.25f * q.w) * sum[i] : 0.0f;
    __syncthreads();
    if constexpr (OUT == kOutMean) {
        if (wave != 0) return;
        float* out = (float*)A.out + batch * A.casc_stride;
        Pack32<V> c;
#pragma unroll
        for (int i = 0; i < V; ++i)
            c.v[i] = (red[0][i][lane] + red[1][i][lane]) + (red[2][i][lane] + red[3][i][lane]);
        const uint32_t o = ((uint32_t)(v * A.full_px + u) * (uint32_t)(A.nd / 4) + cone) * LB + (uint32_t)l;
        if (active) *reinterpret_cast<Pack32<V>*>(out + o) = c;
    } else {
        // J of PW probes x LB wavelengths, probes fastest over the threads
        // (cascade 0: rows along x)
        for (int j = (int)threadIdx.x; j < PW * LB; j += kBlock) {
            const int p = j & (PW - 1), jl = j / PW, i = jl % V, jlane = p * LPR + jl / V;
            const int jal = (int)bs * tw + (p & (tw - 1)), jas = (int)bl * A.th + (p >> A.tw_log2);
            const int ju = 2 * ((int)tx * A.tile_x + (swap ? jas : jal)) + pu;
            const int jv = 2 * ((int)tz * A.tile_z + (swap ? jal : jas)) + pv;
            const int lam = (int)batch * LB + jl;
            if (ju < A.full_px && jv < A.full_pz && lam < A.n_wave)
                A.J[(int64_t)lam * A.ncell + (int64_t)jv * A.full_px + ju] =
                    (red[0][i][jlane] + red[1][i][jlane]) + (red[2][i][jlane] + red[3][i][jlane]);
        }
    }
}

// Arguments of a march by 4 probes x 16 lanes per wavefront over a cascade
// (geometry and launch order; n_blocks = 0 when nothing is flagged). plain:
// every probe in plain order.
LaunchArgs row_args(const LevelDesc& L, const LevelTable& T, int32_t nx, int32_t nz, bool plain);

}  // namespace tab
}  // namespace rcx
