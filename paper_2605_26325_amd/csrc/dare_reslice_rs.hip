// Directionality-aware reslice at interpolation radius R = 2..8 voxels (Sec. 2.1 "Reslicing",
// Eq. 1, Eq. 2, Fig. 2; the paper times radii of 0.125, 0.25 and 0.5 mm).
//
// Every pixel blends the voxels within L-infinity distance R of its position with tent weights
// prod_a max(0, 1 - |c_a - v_a| / R), (2R)^3 voxels per pixel, each voxel's value being its
// direction blend V_v = sum_b w_b c_vb a_vb / sum_b w_b c_vb over the surviving bins.
//
// The tents are not summed per pixel.  A tent of integer half-width R has its corners on whole
// voxels, so along each axis it is linear between two neighbouring lattice points, and the sums
// over voxels, N(c) = sum_v t_v(c) V_v and D(c) = sum_v t_v(c) over the valid voxels, are
// trilinear in every unit cell: they are the trilinear interpolation of their own values at the
// cell's 8 corners.  At a lattice point g the weights are products of the whole numbers
// R - |g_a - v_a| (the common factor R^-3 cancels in N / D), so N and D on the lattice are
// separable convolutions of 2R - 1 taps per axis.  A tile computes
//   voxels   V_v of every voxel its pixels reach, once, into LDS (NaN where not valid);
//   lattice  N and D at the cells' corners by three passes of 2R - 1 taps in LDS, along the
//            dominant axis of the normal first (the axis whose extent shrinks most);
//   pixels   N and D interpolated from 8 corners, and their quotient.
// D at a lattice point is a whole number (at most R^6 < 2^24) and exact in FP32, and a pixel is
// assigned exactly when a voxel with positive weight is valid, as in the direct sum: a corner's
// weight is positive where the voxel range of its tents adds to the pixel's.  A lattice value
// with positive weight for a pixel does not depend on the tile (every voxel within its tents is in
// the pixel's reach and so staged, and taps are added in a fixed order), so a request gives the
// same bits alone and in a batch, whatever the tile edge.
//
// One workgroup takes a 16 x 16 tile, in one piece if its voxel box fits the LDS budget and in
// pieces of 8, 4, 2 or 1 pixels squared if not (coarse output pitch).  A single pixel's box
// always fits.
#include <algorithm>

#include "dare_reslice_dev.h"
#include "dare_staged.h"

namespace dare {

namespace {

template <int R>
struct WideLimits {
    // The pool holds V and, in the place it leaves, the second pass's output; and beside them the
    // cube list and, in its place, the outputs of the first and third pass.  A 16 x 16 tile at half
    // a voxel per pixel has at most 11 lattice points per axis, however it lies.  Up to radius 6
    // the pool is a little less than that takes, so that more workgroups fit a CU: 6, 5, 4, 2, 2 at
    // R = 2..6 (a 512 x 512 slice has 4 tiles per CU; at R = 4 the full pool allowed 3 workgroups,
    // a second round, and 39 us per slice against 27); the steepest tiles then go in pieces.
    static constexpr int kLattice = 11, kEdge = kLattice + 2 * R - 2;
    static constexpr int kFull = (kEdge * kEdge * kEdge + 2 * kLattice * kEdge * kEdge + 11) / 4 * 4;   // V, first pass
    static constexpr int kPool = R == 2 ? 5400 : R == 3 ? 6600 : R == 4 ? 8900 : R == 5 ? 14800 : R == 6 ? 17600 : kFull;
    static constexpr int kSlots = R <= 4 ? 1024 : 2048;     // (box brick, bin) table entries: one pixel's, at 64 bins
    static constexpr int kThreads = R <= 4 ? 256 : 512;     // boxes of 10000 voxels: two workgroups per CU
    static_assert(kPool % 4 == 0 && kPool >= 8 * R * R * R + 16 * R * R + 8, "a single pixel's box fits");
    static_assert(((2 * R + 6) / 8 + 1) * ((2 * R + 6) / 8 + 1) * ((2 * R + 6) / 8 + 1) * kMaxBins <= kSlots, "and its slots");
};

// A list entry packs a 2 x 2 x 2 cube's place in its brick (6 bits), its box brick (9) and its
// coordinates among the box's cubes (5 each).
constexpr int kBoxBricks = 511, kBoxEdge = 60;

template <int DT, int R>
struct WideLds {
    SetupLds sh;
    int lat[3], len[3];                                      // the whole tile's lattice points
    float c0[3];
    int nlist;
    alignas(16) int slot[WideLimits<R>::kSlots];             // [box brick][bin], rows of kactp
    float2 scale[DT == DARE_FP8_E4M3 ? WideLimits<R>::kSlots : 1];
    alignas(16) float pool[WideLimits<R>::kPool];
};

// x / d for 0 <= x < 2^20 through the hardware reciprocal: (x + 1/2) / d lies at least 1/(2 d) from a
// whole number, further than the products' rounding (relative 2^-22) moves it.  One reciprocal to set
// up, where the multiplier of an exact integer division takes some 25 instructions of every wave:
// a piece divides by eight different numbers.
struct FloatDiv {
    float r, h;
    __device__ __forceinline__ explicit FloatDiv(int d) : r(__builtin_amdgcn_rcpf((float)d)), h(0.5f * r) {}
    __device__ __forceinline__ int operator()(int x) const { return (int)__builtin_fmaf((float)x, r, h); }
};

// Minimum over the four lanes of a quad.
__device__ __forceinline__ int quad_min(int x) {
    x = min(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true));
    return min(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true));
}

// The lattice points of a tile's cells: `lat` the lowest cell floor, `len` lattice points per
// axis; c0 the first pixel's position.  Positions are rounded sums and products, so they rise (or
// fall) with i and with j each, and the corner pixels' cells bound every pixel's exactly.  The
// lanes of each quad take the four corners.
__device__ __forceinline__ void tile_cells(const SlicePos& q, int i0, int j0, int i1, int j1, int (&lat)[3],
                                           int (&len)[3], float (&c0)[3]) {
    const int k = threadIdx.x & 3;
    double c[3];
    pixel_coords(q, (k & 1) ? i1 : i0, (k & 2) ? j1 : j0, c);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int f = (int)fmin(fmax(floor(c[a]), -1048576.0), 1048576.0);
        lat[a] = ui(quad_min(f));
        len[a] = -ui(quad_min(-f)) - lat[a] + 2;
        c0[a] = uf((float)c[a]);   // lane 0 of the wave: the first pixel
    }
}

// Does a tile with these lattice extents fit the LDS budget?
template <int R>
__device__ __forceinline__ bool wide_fits(const int (&len)[3], int dax, int kactp) {
    using L = WideLimits<R>;
    const int pax = dax == 0 ? 1 : 0, qax = dax == 2 ? 1 : 2;
    int l[3], v[3], nbb = 1, ncubes = 1;
    bool small = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        l[a] = min(len[a], 64);
        v[a] = l[a] + 2 * R - 2;
        nbb *= (v[a] + 6) / 8 + 1;
        ncubes *= v[a] / 2 + 1;
        small = small && v[a] <= kBoxEdge;
    }
    const int ld = pick3(l, dax), lp = pick3(l, pax), vp = pick3(v, pax), vq = pick3(v, qax);
    const int nv = v[0] * v[1] * v[2], p1 = 2 * ld * vp * vq, p2 = 2 * ld * lp * vq;
    return small && max(nv, p2) + max(ncubes, p1) + 8 <= L::kPool && nbb <= kBoxBricks && nbb * kactp <= L::kSlots;
}

// One tile piece of pixels, workgroup-uniform.
struct Piece {
    int i0, j0, ni, nj;
    int lat[3], len[3];     // lattice points
    int lo[3], dim[3];      // voxel box (may leave the grid)
    int blo[3], bdim[3];    // its in-grid bricks
    float c0[3];
};

// Voxels phase, first part: the cubes of 2 x 2 x 2 voxels (one 64-byte line of FP32 pairs, 32 bytes
// of BF16) that may hold a voxel in reach, one thread per cube, z fastest as in the bricks; those
// that pass are listed in that order, with one LDS atomic per wave.
template <int DT, int R, int NT>
__device__ __forceinline__ void list_cubes(const VolView& vv, const Piece& t, WideLds<DT, R>& L, int* list) {
    float m[3], fu[3], fw[3], l1m = 0.0f, l1u = 0.0f, l1w = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        m[a] = uf(L.sh.fm[a]);
        fu[a] = uf(L.sh.fu[a]);
        fw[a] = uf(L.sh.fw[a]);
        l1m += fabsf(m[a]);
        l1u += fabsf(fu[a]);
        l1w += fabsf(fw[a]);
    }
    // a voxel within L-infinity distance R of a pixel p of the tile satisfies |m.(v - p)| < R |m|_1,
    // and its lateral offsets exceed the tile's extent by less than R |u|_1, R |w|_1; a cube's voxels
    // lie within 1/2 of its centre (the margins cover FP32 rounding of coordinates up to the grid's
    // size and the pose rigidity tolerance)
    const float slop = 2e-3f + 1e-6f * (float)(max(vv.n[0], max(vv.n[1], vv.n[2])) + 64);
    const float reach = (float)R + 0.5f;
    const float thr_n = reach * l1m + slop, thr_u = reach * l1u + 0.02f + slop, thr_v = reach * l1w + 0.02f + slop;
    const float hi_u = (float)(t.ni - 1) * uf(L.sh.lu) + thr_u, hi_v = (float)(t.nj - 1) * uf(L.sh.lw) + thr_v;
    int c_lo[3], c_n[3];      // the cubes of the box inside the grid
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c_lo[a] = max(t.lo[a], 0) >> 1;
        c_n[a] = ((min(t.lo[a] + t.dim[a], vv.n[a]) - 1) >> 1) - c_lo[a] + 1;
    }
    const int n = c_n[0] * c_n[1] * c_n[2];
    const FloatDiv dz(c_n[2]), dy(c_n[1]);
    for (int base = 0; base < n; base += NT) {
        const int e = base + (int)threadIdx.x;
        const int exy = dz(e), cx = dy(exy);
        const int c[3] = {c_lo[0] + cx, c_lo[1] + exy - cx * c_n[1], c_lo[2] + e - exy * c_n[2]};
        float dn = 0.0f, du = 0.0f, dv = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float d = (float)(2 * c[a]) + 0.5f - t.c0[a];
            dn += m[a] * d;
            du += fu[a] * d;
            dv += fw[a] * d;
        }
        const bool pass =
            e < n && fabsf(dn) < thr_n && du > -thr_u && du < hi_u && dv > -thr_v && dv < hi_v;
        const unsigned long long mask = __ballot(pass);
        int first = 0;
        if ((threadIdx.x & 63) == 0 && mask) first = atomicAdd(&L.nlist, __popcll(mask));
        first = ui(first);
        if (pass) {
            const int box = (((c[2] >> 2) - t.blo[2]) * t.bdim[1] + (c[1] >> 2) - t.blo[1]) * t.bdim[0] + (c[0] >> 2) - t.blo[0];
            list[first + __popcll(mask & ((1ull << (threadIdx.x & 63)) - 1ull))] =
                (brick_local(2 * c[0], 2 * c[1], 2 * c[2]) >> 3) | box << 6 | (c[0] - (t.lo[0] >> 1)) << 15 |
                (c[1] - (t.lo[1] >> 1)) << 20 | (c[2] - (t.lo[2] >> 1)) << 25;
        }
    }
}

// Voxels phase, second part: the listed cubes' voxels, eight lanes per cube (so a wave reads whole
// lines of a bin), their surviving bins gathered and blended into V_v, NaN when none holds a
// sample.  U voxels of NB bins per thread and round: their pair loads are all issued before any is
// used; a pair with no slot is skipped and adds nothing.  With one surviving bin its weight cancels
// and is taken as 1 (it may underflow); V_v is then the stored value itself, unrounded.
template <int DT, int R, int NT>
__device__ __forceinline__ void gather_wide(const VolView& vv, const Piece& t, int dax, WideLds<DT, R>& L,
                                            const int* list, float* V, int kact, int kactp) {
    using PT = Pair<DT>;
    using T = typename PT::T;
    constexpr int U = 2, NB = 8;
    const gptr<const T> data = global((const T*)vv.data);
    const uint32_t cap = (uint32_t)ui((int)vv.cap);
    const int nvox = 8 * ui(L.nlist);
    const bool one = kact == 1;
    // V's strides per axis, the lane's place in a cube, and the in-grid part of the box
    const int pax = dax == 0 ? 1 : 0;
    const int vd = pick3(t.dim, dax), vdp = vd * pick3(t.dim, pax);
    int str[3], off[3], r0[3], rn[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        str[a] = a == dax ? 1 : (a == pax ? vd : vdp);
        off[a] = (((int)threadIdx.x >> a) & 1) - (t.lo[a] & 1);
        r0[a] = max(-t.lo[a], 0);
        rn[a] = min(t.dim[a], vv.n[a] - t.lo[a]) - r0[a];
    }
    for (int base = 0; base < nvox; base += U * NT) {
        int row[U], loc[U], vi[U];
        bool ok[U];
        float A[U], B[U], first[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * NT + (int)threadIdx.x;
            const uint32_t ent = (uint32_t)list[min(i, nvox - 1) >> 3];
            const int x = 2 * (int)((ent >> 15) & 31) + off[0], y = 2 * (int)((ent >> 20) & 31) + off[1],
                      z = 2 * (int)(ent >> 25) + off[2];
            ok[u] = i < nvox && (unsigned)(x - r0[0]) < (unsigned)rn[0] && (unsigned)(y - r0[1]) < (unsigned)rn[1] &&
                    (unsigned)(z - r0[2]) < (unsigned)rn[2];
            vi[u] = x * str[0] + y * str[1] + z * str[2];
            row[u] = (int)__umul24((ent >> 6) & 511, (uint32_t)kactp);
            loc[u] = (int)(ent & 63) << 3 | ((int)threadIdx.x & 7);
            A[u] = B[u] = first[u] = 0.0f;
        }
        for (int k0 = 0; k0 < kact; k0 += NB) {
            int sl[U][NB];
            T pr[U][NB];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int g = 0; g < NB; g += 4) {
                    const int4 s4 = *reinterpret_cast<const int4*>(&L.slot[row[u] + k0 + g]);
                    sl[u][g] = s4.x;
                    sl[u][g + 1] = s4.y;
                    sl[u][g + 2] = s4.z;
                    sl[u][g + 3] = s4.w;
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int g = 0; g < NB; ++g) {
                    pr[u][g] = T{};
                    if ((uint32_t)sl[u][g] < cap) pr[u][g] = *(const T*)&data[((size_t)sl[u][g] << 9) | (uint32_t)loc[u]];
                }
#pragma unroll
            for (int g = 0; g < NB; ++g) {
                const float w = uf(L.sh.act_w[k0 + g]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float2 sc = make_float2(0.0f, 0.0f);
                    if constexpr (DT == DARE_FP8_E4M3) sc = L.scale[row[u] + k0 + g];
                    float a, c;
                    PT::decode(pr[u][g], sc, a, c);
                    if (g == 0) first[u] = a;
                    const float wc = w * c;
                    A[u] = __builtin_fmaf(wc, a, A[u]);
                    B[u] = B[u] + wc;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u]) V[vi[u]] = B[u] > 0.0f ? (one ? first[u] : A[u] / B[u]) : __builtin_nanf("");
    }
}

// Four neighbouring lattice points of one axis: 2R - 1 taps R - |k - (R - 1)| each, from the
// 2R + 2 inputs that `in(j, x, c)` gives (numerator x, denominator c), added in order of j.
template <int R, class In>
__device__ __forceinline__ void taps4(In&& in, float2 (&o)[4]) {
#pragma unroll
    for (int b = 0; b < 4; ++b) o[b] = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < 2 * R + 2; ++j) {
        float x, c;
        in(j, x, c);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int k = j - b;
            if (k < 0 || k > 2 * R - 2) continue;
            const float w = (float)(R - (k > R - 1 ? k - (R - 1) : R - 1 - k));
            o[b].x = __builtin_fmaf(w, x, o[b].x);
            o[b].y = __builtin_fmaf(w, c, o[b].y);
        }
    }
}

// The pixels of a piece from the lattice sums P3[q][p][d].
template <int DT, int R, int DAX, int NT>
__device__ __forceinline__ void pixels_wide(const VolView& vv, const SlicePos& q, const SliceArgs& s, const Piece& t,
                                            int edge, const float2* P3) {
    constexpr int PAX = DAX == 0 ? 1 : 0, QAX = DAX == 2 ? 1 : 2;
    const int ld = t.len[DAX], lp = t.len[PAX];
    const int shift = __builtin_ctz(edge);
    const gptr<float> out = global(s.out);
    for (int idx = (int)threadIdx.x; idx < edge * edge; idx += NT) {
        const int li = idx & (edge - 1), lj = idx >> shift;
        if (li >= t.ni || lj >= t.nj) continue;
        const int i = t.i0 + li, j = t.j0 + lj;
        double c[3];
        pixel_coords(q, i, j, c);
        float val = __builtin_nanf("");
        if (c[0] > -(double)R && c[0] < (double)(vv.n[0] - 1 + R) && c[1] > -(double)R &&
            c[1] < (double)(vv.n[1] - 1 + R) && c[2] > -(double)R && c[2] < (double)(vv.n[2] - 1 + R)) {
            // per axis: the nearer corner (base) and the weight w <= 1/2 of the other one.
            // lerp(base, other) = base + w (other - base) is then positive whenever a corner with
            // positive weight is, and loses nothing where both corners hold the same (D away from the
            // borders).  The first axis in FP32, the others and the quotient in FP64, so that the
            // result is rounded once more only.
            int b[3], step[3];
            double w[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double fl = floor(c[a]), f = c[a] - fl;
                const bool up = f > 0.5;
                // the cell lies in the box; the clamp only keeps the LDS reads in bounds
                b[a] = min(max((int)fl - t.lat[a], 0), t.len[a] - 2) + (up ? 1 : 0);
                step[a] = up ? -1 : 1;
                w[a] = up ? fl + 1.0 - c[a] : f;
            }
            const float2* cell = P3 + (b[QAX] * lp + b[PAX]) * ld + b[DAX];
            const int sd = step[DAX], sp = step[PAX] * ld, sq = step[QAX] * lp * ld;
            auto lerp = [](float2 lo, float2 hi, float x) {
                return make_float2(__builtin_fmaf(x, hi.x - lo.x, lo.x), __builtin_fmaf(x, hi.y - lo.y, lo.y));
            };
            double2 r[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float2* e = cell + (k >> 1) * sq + (k & 1) * sp;
                const float2 x = lerp(e[0], e[sd], (float)w[DAX]);
                r[k] = make_double2((double)x.x, (double)x.y);
            }
            auto lerp2 = [](double2 lo, double2 hi, double x) {
                return make_double2(__builtin_fma(x, hi.x - lo.x, lo.x), __builtin_fma(x, hi.y - lo.y, lo.y));
            };
            const double2 nd = lerp2(lerp2(r[0], r[1], w[PAX]), lerp2(r[2], r[3], w[PAX]), w[QAX]);
            if (nd.y > 1e-30) {   // the quotient from an FP32 reciprocal and one correction
                const double inv = (double)(1.0f / (float)nd.y), q0 = nd.x * inv;
                val = (float)__builtin_fma(__builtin_fma(-q0, nd.y, nd.x), inv, q0);
            } else if (nd.y > 0.0) {   // beyond the FP32 reciprocal's range
                val = (float)(nd.x / nd.y);
            }
        }
        out[(size_t)j * s.W + i] = val;
    }
}

// A piece with nothing in reach, or of a request with no surviving bin: NaN.
template <int NT>
__device__ __forceinline__ void nan_piece(const SliceArgs& s, int i0, int j0, int ni, int nj) {
    const gptr<float> out = global(s.out);
    for (int idx = (int)threadIdx.x; idx < 256; idx += NT) {
        const int li = idx & 15, lj = idx >> 4;
        if (li < ni && lj < nj) out[(size_t)(j0 + lj) * s.W + (i0 + li)] = __builtin_nanf("");
    }
}

// One staged piece of a tile (edge x edge pixels at most), `t`'s pixels, lattice and c0 set.
template <int DT, int R, int NT>
__device__ __forceinline__ void wide_piece(const VolView& vv, const SlicePos& q, const SliceArgs& s, Piece& t,
                                           int edge, int dax, int kact, int kactp, WideLds<DT, R>& L) {
    const int tid = (int)threadIdx.x;
    bool empty = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        t.lo[a] = t.lat[a] - (R - 1);
        t.dim[a] = t.len[a] + 2 * R - 2;
        const int lo = max(t.lo[a], 0), hi = min(t.lo[a] + t.dim[a], vv.n[a]) - 1;
        t.blo[a] = lo >> 3;
        t.bdim[a] = (hi >> 3) - t.blo[a] + 1;
        empty = empty || lo > hi;
    }
    if (empty) {
        nan_piece<NT>(s, t.i0, t.j0, t.ni, t.nj);
        return;
    }
    const int pax = dax == 0 ? 1 : 0, qax = dax == 2 ? 1 : 2;
    const int vd = pick3(t.dim, dax), vp = pick3(t.dim, pax), vq = pick3(t.dim, qax);
    const int ld = pick3(t.len, dax), lp = pick3(t.len, pax), lq = pick3(t.len, qax);
    const int nv = vd * vp * vq;
    float* V = L.pool;
    float2* P2 = reinterpret_cast<float2*>(L.pool);
    float* side = L.pool + ((max(nv, 2 * ld * lp * vq) + 3) & ~3);
    int* list = reinterpret_cast<int*>(side);
    float2* P1 = reinterpret_cast<float2*>(side);
    // slots: the table entry of every (box brick, bin) pair, -1 past the surviving bins; a thread's
    // first read is in flight during the classification
    const int nsl = t.bdim[0] * t.bdim[1] * t.bdim[2] * kactp;
    const FloatDiv dk(kactp), dx(t.bdim[0]), dy(t.bdim[1]);
    auto slot_of = [&](int e) {
        const int bb = dk(e), k = e - bb * kactp;
        if (e >= nsl || k >= kact) return -1;
        const int byz = dx(bb), bx = bb - byz * t.bdim[0];
        const int bz = dy(byz), by = byz - bz * t.bdim[1];
        const int64_t brick = ((int64_t)(t.blo[2] + bz) * vv.nby + (t.blo[1] + by)) * vv.nbx + (t.blo[0] + bx);
        return (int)global(vv.table)[(int64_t)L.sh.act_bin[k] * vv.nbricks + brick];
    };
    auto put_slot = [&](int e, int slot) {
        if (e >= nsl) return;
        L.slot[e] = slot;
        if constexpr (DT == DARE_FP8_E4M3) L.scale[e] = slot >= 0 ? vv.scales[slot] : make_float2(0.0f, 0.0f);
    };
    const int slot0 = slot_of(tid);
    {   // every voxel starts NaN; the gather overwrites those it reaches
        const float nan = __builtin_nanf("");
        for (int e = 4 * tid; e < nv; e += 4 * NT) *reinterpret_cast<float4*>(&V[e]) = make_float4(nan, nan, nan, nan);
    }
    if (tid == 0) L.nlist = 0;
    __syncthreads();
    list_cubes<DT, R, NT>(vv, t, L, list);
    put_slot(tid, slot0);
    for (int e = tid + NT; e < nsl; e += NT) put_slot(e, slot_of(e));
    __syncthreads();
    gather_wide<DT, R, NT>(vv, t, dax, L, list, V, kact, kactp);
    __syncthreads();
    {   // along d: V -> P1[q][p][g]
        const int nb = (ld + 3) >> 2, n = vp * vq * nb;
        const FloatDiv db(nb);
        for (int x = tid; x < n; x += NT) {
            const int col = db(x), b = x - col * nb, base = col * vd + 4 * b, left = vd - 1 - 4 * b;
            float2 o[4];
            taps4<R>([&](int j, float& num, float& den) {
                const float v = V[base + min(j, left)];
                const bool ok = v == v;
                num = ok ? v : 0.0f;
                den = ok ? 1.0f : 0.0f;
            }, o);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (4 * b + k < ld) P1[col * ld + 4 * b + k] = o[k];
        }
    }
    __syncthreads();
    {   // along p: P1 -> P2[q][gp][g]
        const int nb = (lp + 3) >> 2, n = vq * nb * ld;
        const FloatDiv dl(ld), db(nb);
        for (int x = tid; x < n; x += NT) {
            const int r = dl(x), g = x - r * ld, cq = db(r), b = r - cq * nb;
            const int base = (cq * vp + 4 * b) * ld + g, left = vp - 1 - 4 * b;
            float2 o[4];
            taps4<R>([&](int j, float& num, float& den) {
                const float2 v = P1[base + min(j, left) * ld];
                num = v.x;
                den = v.y;
            }, o);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (4 * b + k < lp) P2[(cq * lp + 4 * b + k) * ld + g] = o[k];
        }
    }
    __syncthreads();
    {   // along q: P2 -> P3[gq][gp][g], in P1's place
        const int nb = (lq + 3) >> 2, plane = lp * ld, n = nb * plane;
        const FloatDiv dp(plane);
        for (int x = tid; x < n; x += NT) {
            const int b = dp(x), g = x - b * plane, base = 4 * b * plane + g, left = vq - 1 - 4 * b;
            float2 o[4];
            taps4<R>([&](int j, float& num, float& den) {
                const float2 v = P2[base + min(j, left) * plane];
                num = v.x;
                den = v.y;
            }, o);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (4 * b + k < lq) P1[base + k * plane] = o[k];
        }
    }
    __syncthreads();
    switch (dax) {
        case 0: pixels_wide<DT, R, 0, NT>(vv, q, s, t, edge, P1); break;
        case 1: pixels_wide<DT, R, 1, NT>(vv, q, s, t, edge, P1); break;
        default: pixels_wide<DT, R, 2, NT>(vv, q, s, t, edge, P1); break;
    }
}

// Part `part` of `parts` of a 16 x 16 tile at radius R: the whole tile is part 0's if it fits in one
// piece, else the parts take the pieces in turn.
template <int DT, int R, int NT>
__device__ __forceinline__ void wide_tile(const VolDev* __restrict__ vd, const SliceArgs& s, int unit, int part,
                                          int parts, WideLds<DT, R>& L) {
    const int ty = unit / s.tiles_x, tx = unit - ty * s.tiles_x;
    const int i0 = tx * kTile, j0 = ty * kTile;
    const int ni = min(kTile, s.W - i0), nj = min(kTile, s.H - j0);
    const VolView vv = view_of(vd);
    SlicePos q;
    {   // the bins on wave 0, the plane's frame on wave 1 and the tile's lattice points on wave 2, at once
        double T[12];
        slice_pose(vd, s, T);
        load_pos(vd, T, s, q);
        if (threadIdx.x < 64) {
            const int n = slice_gates(vd, s, L.sh, T);
            pad_bins(L.sh, n);
            if (n == 1 && threadIdx.x == 0) L.sh.act_w[0] = 1.0f;   // it cancels
        } else if (threadIdx.x == 64) {
            slice_frame(vd, s, T, L.sh);
        } else if (threadIdx.x >= 128 && threadIdx.x < 192) {
            int lat[3], len[3];
            float c0[3];
            tile_cells(q, i0, j0, i0 + ni - 1, j0 + nj - 1, lat, len, c0);
            if (threadIdx.x == 128) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    L.lat[a] = lat[a];
                    L.len[a] = len[a];
                    L.c0[a] = c0[a];
                }
            }
        }
    }
    __syncthreads();
    const int kact = ui(L.sh.kact), kactp = (kact + 7) & ~7, dax = ui(L.sh.dax);
    if (kact == 0) {
        if (part == 0) nan_piece<NT>(s, i0, j0, ni, nj);
        return;
    }
    Piece t;
    t.i0 = i0;
    t.j0 = j0;
    t.ni = ni;
    t.nj = nj;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        t.lat[a] = ui(L.lat[a]);
        t.len[a] = ui(L.len[a]);
        t.c0[a] = uf(L.c0[a]);
    }
    if (wide_fits<R>(t.len, dax, kactp)) {
        if (part == 0) wide_piece<DT, R, NT>(vv, q, s, t, kTile, dax, kact, kactp, L);
        return;
    }
    // a tile out of reach of the grid as a whole (a view much larger than the volume)
    bool out = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) out = out || t.lat[a] - (R - 1) >= vv.n[a] || t.lat[a] + t.len[a] + R - 2 < 0;
    if (out) {
        if (part == 0) nan_piece<NT>(s, i0, j0, t.ni, t.nj);
        return;
    }
    // the largest piece whose box fits wherever it falls (a single pixel's does)
    int edge = kTile / 2;
    for (; edge > 1; edge >>= 1) {
        int len[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double ex = fabs(q.sx * q.e0[a]), ey = fabs(q.sy * q.e1[a]);
            const double place = fabs(q.t[a]) + fabs(q.o[a]) + (double)s.W * ex + (double)s.H * ey;
            len[a] = ui(piece_points(edge, (ex + ey) * q.inv_h, place * q.inv_h));
        }
        if (wide_fits<R>(len, dax, kactp)) break;
    }
    const int shift = __builtin_ctz(kTile / edge), across = 1 << shift;
    for (int k = part; k < across * across; k += parts) {
        const int x = (k & (across - 1)) * edge, y = (k >> shift) * edge;
        if (x >= t.ni || y >= t.nj) continue;
        Piece u;
        u.i0 = i0 + x;
        u.j0 = j0 + y;
        u.ni = min(edge, t.ni - x);
        u.nj = min(edge, t.nj - y);
        tile_cells(q, u.i0, u.j0, u.i0 + u.ni - 1, u.j0 + u.nj - 1, u.lat, u.len, u.c0);
        wide_piece<DT, R, NT>(vv, q, s, u, edge, dax, kact, kactp, L);
        __syncthreads();
    }
}

}  // namespace

template <int DT, int R>
__global__ void __launch_bounds__(WideLimits<R>::kThreads) k_reslice_rs(const VolDev* __restrict__ vd, SliceArgs s,
                                                                        int parts) {
    __shared__ WideLds<DT, R> L;
    const int b = xcd_remap(blockIdx.x, gridDim.x), unit = b / parts;
    wide_tile<DT, R, WideLimits<R>::kThreads>(vd, s, unit, b - unit * parts, parts, L);
}

// Batched form, grid-stride: the first counts[2] of the (request, tile) units take counts[3]
// workgroups each, the others one.  Every tile computes its own setup, so a request's result is
// the one it gets alone.
template <int DT, int R>
__global__ void __launch_bounds__(WideLimits<R>::kThreads) k_reslice_rs_batch(const BatchReq* __restrict__ reqs,
                                                                              const int2* __restrict__ units,
                                                                              const int* __restrict__ counts) {
    __shared__ WideLds<DT, R> L;
    // coarse units times parts is a few workgroups per CU more than the units at most: 32 bits
    const uint32_t parts = (uint32_t)max(counts[3], 1), coarse = (uint32_t)counts[2] * parts;
    const uint32_t n = coarse + (uint32_t)(counts[0] - counts[2]);
    for (uint32_t b = blockIdx.x; b < n; b += gridDim.x) {
        const bool c = b < coarse;
        const uint32_t u = c ? b / parts : b - coarse + (uint32_t)counts[2], part = c ? b - u * parts : 0;
        const int r = ui(units[u].x), t = ui(units[u].y);
        wide_tile<DT, R, WideLimits<R>::kThreads>(reqs[r].vol, reqs[r].s, t, (int)part, c ? (int)parts : 1, L);
        __syncthreads();
    }
}

int64_t staged_tiles(int W, int H) { return (int64_t)((W + kTile - 1) / kTile) * ((H + kTile - 1) / kTile); }

#define DARE_DISPATCH_R(radius, MACRO)                          \
    switch (radius) {                                           \
        case 2: MACRO(2); break;                                \
        case 3: MACRO(3); break;                                \
        case 4: MACRO(4); break;                                \
        case 5: MACRO(5); break;                                \
        case 6: MACRO(6); break;                                \
        case 7: MACRO(7); break;                                \
        case 8: MACRO(8); break;                                \
        default: return hipErrorInvalidValue;                   \
    }

template <int DT>
static hipError_t launch_one(const VolDev* vd, int radius, const SliceArgs& s, int parts, hipStream_t stream) {
    const dim3 grid((unsigned)(staged_tiles(s.W, s.H) * parts));
#define S(R) hipLaunchKernelGGL((k_reslice_rs<DT, R>), grid, dim3(WideLimits<R>::kThreads), 0, stream, vd, s, \
                                parts)
    DARE_DISPATCH_R(radius, S)
#undef S
    return hipGetLastError();
}

template <int DT>
static hipError_t launch_many(int radius, const BatchReq* reqs, const int2* units, const int* counts, int grid,
                              hipStream_t stream) {
#define B(R)                                                                                                       \
    hipLaunchKernelGGL((k_reslice_rs_batch<DT, R>), dim3(grid), dim3(WideLimits<R>::kThreads), 0, stream, reqs,   \
                       units, counts)
    DARE_DISPATCH_R(radius, B)
#undef B
    return hipGetLastError();
}

// A single request whose output is too coarse for a tile to stage in one piece (its extent beyond
// about 10 voxels) has its tiles' pieces spread over workgroups, up to 64 workgroups per CU in all:
// few tiles of a coarse view meet the grid, and those hold most of its work.  512 x 512 pixels 16
// voxels apart at R = 2, 6, 8: 287, 467, 727 us per slice with 8 workgroups per CU, 87, 163, 245 us
// with 64.
hipError_t launch_reslice_staged(const VolDev* vd, int dtype, int radius, const SliceArgs& s, double pitch_vox,
                                 hipStream_t stream) {
    const int parts = tile_parts(staged_tiles(s.W, s.H), tile_pieces(pitch_vox));
#define L(D) return launch_one<D>(vd, radius, s, parts, stream)
    DARE_DISPATCH_DT(dtype, L)
#undef L
}

hipError_t launch_reslice_staged_batch(int dtype, int radius, const BatchReq* reqs, const int2* units,
                                       const int* counts, int grid, hipStream_t stream) {
#define L(D) return launch_many<D>(radius, reqs, units, counts, grid, stream)
    DARE_DISPATCH_DT(dtype, L)
#undef L
}

// The unit entries a workspace holds for a request.  Above radius 4 that is one for 4 pixels, more
// than its tiles: what a workspace must hold, and so which batches a given one admits, is part of
// what callers have sized for.
int64_t batch_units(int radius, int W, int H) {
    return radius <= 4 ? staged_tiles(W, H) : ((int64_t)W * H + 3) / 4;
}

}  // namespace dare
