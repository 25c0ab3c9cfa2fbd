// Volume reconstruction kernels (Sec. 2.1 "Volume reconstruction", Fig. 1):
// frame pose composition, direction-bin assignment, brick occupancy and
// allocation, nearest-voxel accumulation and finalisation into the stored
// precision.  Positions are FP64 with no contraction so that every
// nearest-voxel decision is reproducible; sums and counts are exact integers
// accumulated with 64-bit atomics, so the result is independent of order.
#include <math.h>

#include <algorithm>

#include "dare_codec.h"
#include "dare_frames.h"
#include "dare_internal.h"
#include "dare_patches.h"

#pragma clang fp contract(off)

namespace dare {

namespace {

__device__ __forceinline__ double dot3(const double* a, const double* b) {
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}

// Pointers by address space: constant (what a whole workgroup reads and no running kernel
// writes: scalar loads) and global (per-lane accesses and atomics: global, not flat, operations).
template <class T>
using cptr = const __attribute__((address_space(4))) T*;
template <class T>
using gptr = __attribute__((address_space(1))) T*;

// What the per-pixel kernels read of the volume header, through scalar loads.
struct PixelView {
    double origin[3], inv_h;
    int nx, ny, nz, nbx, nby;
    int64_t nbricks;
    const FrameDesc* frames;
    const int32_t* frame_bin;
    int32_t* table;
};

__device__ __forceinline__ PixelView pixel_view(const VolDev* vd) {
    const cptr<VolDev> c = (cptr<VolDev>)vd;
    PixelView v;
#pragma unroll
    for (int a = 0; a < 3; ++a) v.origin[a] = c->origin[a];
    v.inv_h = c->inv_h;
    v.nx = c->nx;
    v.ny = c->ny;
    v.nz = c->nz;
    v.nbx = c->nbx;
    v.nby = c->nby;
    v.nbricks = c->nbricks;
    v.frames = c->frames;
    v.frame_bin = c->frame_bin;
    v.table = c->table;
    return v;
}

// Frame f's placement (translation and raw columns; the unit axes are not needed here), through
// scalar loads: a workgroup works on one frame.
__device__ __forceinline__ FrameDesc frame_uniform(const PixelView& v, int f) {
    const cptr<FrameDesc> p = (cptr<FrameDesc>)v.frames + f;
    FrameDesc d;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        d.t[a] = p->t[a];
        d.e0[a] = p->e0[a];
        d.e1[a] = p->e1[a];
        d.xh[a] = 0.0;
        d.nh[a] = 0.0;
    }
    d.pad = 0.0;
    return d;
}

__device__ __forceinline__ int64_t brick_entry(const PixelView& v, int b, int vx, int vy, int vz) {
    return (int64_t)b * v.nbricks + ((int64_t)(vz >> 3) * v.nby + (vy >> 3)) * v.nbx + (vx >> 3);
}

__device__ __forceinline__ int64_t brick_entry(const VolDev* vd, int b, int vx, int vy, int vz) {
    return (int64_t)b * vd->nbricks + ((int64_t)(vz >> 3) * vd->nby + (vy >> 3)) * vd->nbx + (vx >> 3);
}

// The per-pixel passes take patches of 1024 pixels (dare_patches.h), one per workgroup, four pixels
// per thread.  A wave's 64 lanes are an 8 x 8 block of the image at a time, not 64 pixels of a row:
// the block falls on 8 x 8 neighbouring voxels of a brick or four, whose accumulators lie in whole
// 64-byte cubes of 2 x 2 x 2, where a row of 64 touches 32 cubes in 9 bricks.

// Patch (column and row) and frame of this workgroup in a flat grid of the patches of every
// frame.  Workgroups are dealt to the 8 XCDs round-robin; when a frame's patches are a multiple of
// 8, XCD x takes the x-th eighth of every frame's patches (a band of image rows).  Frames of a
// sweep are near-parallel, so a band of rows falls on the same part of the volume frame after
// frame, and each XCD's L2 keeps the accumulators of its own part instead of all eight sharing
// every line.  The launch covers frames f0, f0 + 1, ...
struct Patch {
    int x, y, f;
};
__device__ __forceinline__ Patch frame_patch(const PatchShape& s, int f0) {
    const int g = blockIdx.x, np = s.nx * s.ny;
    int f, p;
    if ((np & 7) == 0) {
        const int per = np >> 3, k = g >> 3;
        f = k / per;
        p = (g & 7) * per + (k - f * per);
    } else {
        f = g / np;
        p = g - f * np;
    }
    const int y = p / s.nx;
    return Patch{p - y * s.nx, y, f0 + f};
}

// Pixel b (0..3) of this thread in its patch.
__device__ __forceinline__ PatchPixel patch_pixel(const PatchShape& s, const Patch& p, int b) {
    return patch_pixel(s, p.x, p.y, (int)(threadIdx.x >> 6) * 4 + b, (int)threadIdx.x & 63);
}

// The (bin, brick) entry and the place in the brick of the four pixels of this thread: entry -1
// where the pixel lies outside the image or the grid.  Linear-array frames have one bin; a fan
// frame's columns take the bin of their sector's descriptor.
template <bool FAN>
struct FramePixels {
    PixelView v;
    FrameDesc fd;
    int bin;
    const FanArgs* fan;
    int first, w;          // fan: the frame's first descriptor, columns

    __device__ __forceinline__ FramePixels(const VolDev* vd, const FanArgs* fan_, int f, int w_) : fan(fan_), w(w_) {
        v = pixel_view(vd);
        first = FAN ? f * fan->sectors : f;
        fd = frame_uniform(v, first);   // a frame's descriptors share its placement
        bin = *((cptr<int32_t>)v.frame_bin + first);
    }
    __device__ __forceinline__ int64_t entry(int i, int j, int h, double sx, double sy, int& local) const {
        int vx = 0, vy = 0, vz = 0;
        local = 0;
        if (i >= w || j >= h) return -1;
        int b = bin;
        bool ok;
        if constexpr (FAN) {
            ok = fan_voxel(&fd, v.origin, v.inv_h, v.nx, v.ny, v.nz, *fan, i, j, vx, vy, vz);
            b = ((gptr<const int32_t>)v.frame_bin)[first + i * fan->sectors / w];
        } else {
            ok = frame_voxel(&fd, v.origin, v.inv_h, v.nx, v.ny, v.nz, i, j, sx, sy, vx, vy, vz);
        }
        local = brick_local(vx, vy, vz);
        return ok ? brick_entry(v, b, vx, vy, vz) : -1;
    }
};

}  // namespace

// K1: T = P . C per frame (row-major, summed left to right), rigidity check of P.
__global__ void k_compose_frames(VolDev* vd, const float* __restrict__ poses, int n) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= n) return;
    FrameDesc d;
    if (!compose_frame(poses + (size_t)f * 16, vd->calib, vd->normal_axis, d)) atomicOr(&vd->st.bad_pose, kBadPose);
    vd->frames[f] = d;
}

// K2: leader clustering of frame orientations, frames in order, by one workgroup.  The
// sequential rule (an entry joins its best qualifying bin, else opens a new one, else, with the
// codebook full, joins its best bin overall) only changes the codebook when an entry opens a bin.
// So chunks of consecutive entries are tested in parallel against the current codebook, one entry
// per thread, which keeps its best bins so far; every entry before the chunk's first opener is
// final, the opener takes the next bin, and the entries after it test that one bin more.  Identical
// results in n / 512 passes over the codebook and at most max_bins tests of one bin.  Bound: the
// chain of FP64 dot products and barriers of one workgroup; 2400 (frame, sector) entries that open
// 64 bins take 59 us, against 283 with the whole codebook tested again after every opener and 98
// with the opener found by an LDS minimum over all lanes and its vectors read after a second barrier.
constexpr int kAssign = 512;
__global__ void __launch_bounds__(kAssign) k_assign_bins(VolDev* vd, int n, int K0) {
    __shared__ double rep[kMaxBins][6];   // per bin: representative normal, then in-plane axis
    // per wave: its first entry that would open a bin (kAssign: none) and that entry's vectors; one
    // copy is written while the other may still be read, so a round has one barrier
    __shared__ int s_first[2][kAssign / 64];
    __shared__ double s_cand[2][kAssign / 64][6];
    __shared__ int s_sat;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    if (tid < K0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            rep[tid][a] = vd->rep_n[tid][a];
            rep[tid][3 + a] = vd->rep_x[tid][a];
        }
    }
    if (tid == 0) s_sat = vd->st.saturated;
    int K = K0, turn = 0;
    const double ct = vd->cos_tol;
    const int kmax = vd->max_bins;
    __syncthreads();
    for (int base = 0; base < n; base += kAssign) {
        const int f = base + tid;
        double nf[3] = {0, 0, 0}, xf[3] = {0, 0, 0};
        int best = -1, any = -1;
        double best_s = -INFINITY, any_s = -INFINITY;
        if (f < n) {
            const FrameDesc* fd = vd->frames + f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                nf[a] = fd->nh[a];
                xf[a] = fd->xh[a];
            }
        }
        auto test = [&](int b, const double* r) {   // strict > keeps the lowest index on ties
            const double rn[3] = {r[0], r[1], r[2]};
            const double rx[3] = {r[3], r[4], r[5]};
            const double dn = dot3(nf, rn);
            const double di = fabs(dot3(xf, rx));
            const double sc = dn + di;
            if (sc > any_s) {
                any_s = sc;
                any = b;
            }
            if (dn >= ct && di >= ct && sc > best_s) {
                best_s = sc;
                best = b;
            }
        };
        for (int b = 0; b < K; ++b) test(b, rep[b]);
        for (;; turn ^= 1) {   // every entry before the round's opener is final
            const uint64_t open = __ballot(f < n && best < 0 && K < kmax);
            const int first = open ? wave * 64 + __builtin_ctzll(open) : kAssign;
            if ((tid & 63) == 0) s_first[turn][wave] = first;
            if (tid == first) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    s_cand[turn][wave][a] = nf[a];
                    s_cand[turn][wave][3 + a] = xf[a];
                }
            }
            __syncthreads();
            int p = kAssign;
#pragma unroll
            for (int w = 0; w < kAssign / 64; ++w) p = min(p, s_first[turn][w]);
            if (p == kAssign) break;
            if (tid == p) {
                best = K;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    rep[K][a] = nf[a];
                    rep[K][3 + a] = xf[a];
                }
            }
            if (tid > p) test(K, s_cand[turn][p >> 6]);
            ++K;
        }
        turn ^= 1;   // the copy just read stays as it is through the next chunk's first round
        __syncthreads();
        if (f < n) {
            vd->frame_bin[f] = best >= 0 ? best : any;
            if (best < 0) s_sat = 1;   // only with the codebook full
        }
    }
    __syncthreads();
    if (tid >= K0 && tid < K) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            vd->rep_n[tid][a] = rep[tid][a];
            vd->rep_x[tid][a] = rep[tid][3 + a];
        }
    }
    if (tid == 0) {
        vd->st.K = K;
        vd->st.saturated = s_sat;
    }
}

// Marks entry e; returns what this call was first to do: kNew, the entry's mark (-1 -> -2), or
// kDirty, the flag of a resident brick (its slot in `slot`).  The caller appends either to its
// list.  The first reads are at agent scope: through the caches an XCD would keep its stale copy
// and go on to the atomic every time.
enum Marked { kSeen, kNew, kDirty };
__device__ __forceinline__ Marked mark_entry(VolDev* vd, int64_t e, int& slot) {
    const gptr<int32_t> te = (gptr<int32_t>)vd->table + e;
    const int cur = __hip_atomic_load(te, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    slot = cur;
    if (cur == -1) {
        int expected = -1;
        return __hip_atomic_compare_exchange_strong(te, &expected, -2, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT) ? kNew : kSeen;
    }
    if (cur < 0) return kSeen;
    const gptr<uint32_t> fl = (gptr<uint32_t>)vd->dirty_flags + cur;
    return __hip_atomic_load(fl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u &&
                   __hip_atomic_exchange(fl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u ? kDirty : kSeen;
}

// The k-th new entry or dirty slot of the batch into its list.
__device__ __forceinline__ void append_new(VolDev* vd, uint32_t k, int64_t e) {
    if (k < vd->cap) ((gptr<int32_t>)vd->new_list)[k] = (int32_t)e;
}
__device__ __forceinline__ void append_dirty(VolDev* vd, uint32_t k, int slot) {
    ((gptr<int32_t>)vd->dirty_list)[k] = slot;
}
__device__ __forceinline__ void mark_one(VolDev* vd, int64_t e) {
    int slot;
    if (e > INT32_MAX) {
        atomicOr(&vd->st.bad_pose, kBadEntry);
        return;
    }
    const Marked m = mark_entry(vd, e, slot);
    if (m == kNew) append_new(vd, atomicAdd(&vd->st.new_count, 1u), e);
    if (m == kDirty) append_dirty(vd, atomicAdd(&vd->st.dirty_count, 1u), slot);
}

// K3a: mark every (bin, brick) that a pixel of the batch lands in.  A lane whose left or upper
// neighbour in the wave's block holds the same entry leaves it to that lane; what remains goes
// into a set of the workgroup's entries in LDS (about 40 for 1024 pixels), which its threads then
// mark side by side, and a workgroup takes its places in the two lists with one addition each.
// What bounds the pass is what crosses the XCDs: additions to the lists' counters above all (a
// counter takes one about every 5 ns; one per wave made 1490 us of 1800 frames of 256^2, one per
// workgroup 480), then the chain of a mark's read, exchange and store, gone through once per 1024
// pixels (2730 us when the four blocks marked in turn).  One mark per run of a 64-pixel row, each
// with its own addition, took 1190 us; 30 frames of 512^2 into resident bricks 254 -> 71 us.
// An entry that finds no place in 24 steps is marked at once, which a whole wave waits for: with 8
// steps a set two thirds full (20 x 20 pixels 5 voxels apart) turned enough of them away for a call
// of 1200 frames to take 136 us, not 113; 24 are no slower where the set is full (a pixel a brick).
constexpr int kMarkSet = 256;
template <bool FAN>
__device__ __forceinline__ void mark_patch(VolDev* vd, int w, int h, const PatchShape& shape, double sx, double sy, const FanArgs* fan, int f0) {
    __shared__ int set[kMarkSet];
    __shared__ uint32_t count[2], first[2];   // the workgroup's new entries and dirty slots
    if (threadIdx.x < 2) count[threadIdx.x] = 0u;
    for (int k = threadIdx.x; k < kMarkSet; k += 256) set[k] = -1;
    const Patch p = frame_patch(shape, f0);
    const FramePixels<FAN> px(vd, fan, p.f, w);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    bool past = false;            // a pixel in an entry that the lists' 32 bits do not hold
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        int local;
        const PatchPixel at = patch_pixel(shape, p, b);
        const int64_t entry = px.entry(at.i, at.j, h, sx, sy, local);
        past = past || entry > INT32_MAX;
        const int e = (uint64_t)entry > (uint64_t)INT32_MAX ? -1 : (int)entry;
        const int left = __shfl_up(e, 1), up = __shfl_up(e, 8);
        bool mine = e >= 0 && !(lane >= 1 && left == e) && !(lane >= 8 && up == e);
        if (mine) {
            uint32_t at = ((uint32_t)e * 2654435761u) >> 24;
            for (int probe = 0; probe < 24; ++probe, at = (at + 1) & (kMarkSet - 1)) {
                const int was = atomicCAS(&set[at], -1, e);
                mine = was != -1 && was != e;
                if (!mine) break;
            }
            if (mine) mark_one(vd, e);   // no free place for it
        }
    }
    if (__ballot(past) && lane == 0) atomicOr(&vd->st.bad_pose, kBadEntry);
    __syncthreads();
    const int e = set[threadIdx.x];
    int slot = -1;
    const Marked m = e >= 0 ? mark_entry(vd, e, slot) : kSeen;
    // places in the lists: one addition to each counter per workgroup that has any
    const unsigned long long nm = __ballot(m == kNew), dm = __ballot(m == kDirty);
    const unsigned long long below = (1ull << lane) - 1ull;
    uint32_t base_n = 0, base_d = 0;
    if (lane == 0 && nm) base_n = atomicAdd(&count[0], (uint32_t)__popcll(nm));
    if (lane == 0 && dm) base_d = atomicAdd(&count[1], (uint32_t)__popcll(dm));
    // lane 0's values, taken while the whole wave is active
    const uint32_t at_n = __builtin_amdgcn_readfirstlane(base_n) + __popcll(nm & below);
    const uint32_t at_d = __builtin_amdgcn_readfirstlane(base_d) + __popcll(dm & below);
    __syncthreads();
    if (threadIdx.x < 2 && count[threadIdx.x])
        first[threadIdx.x] = atomicAdd(threadIdx.x ? &vd->st.dirty_count : &vd->st.new_count, count[threadIdx.x]);
    __syncthreads();
    if (m == kNew) append_new(vd, first[0] + at_n, e);
    if (m == kDirty) append_dirty(vd, first[1] + at_d, slot);
}

__global__ void __launch_bounds__(256) k_mark_pixels(VolDev* vd, int w, int h, PatchShape shape, double sx, double sy,
                                                     int f0) {
    mark_patch<false>(vd, w, h, shape, sx, sy, nullptr, f0);
}

// Fan probes: one frame descriptor per (frame, sector), each with the frame's pose and the
// sector's in-plane direction, so that the bin assignment runs over them as over frames.
__global__ void k_compose_fan(VolDev* vd, const float* __restrict__ poses, int n, FanArgs fan, int width) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n * fan.sectors) return;
    const int f = k / fan.sectors;
    FrameDesc d;
    if (!compose_frame(poses + (size_t)f * 16, vd->calib, 2, d)) atomicOr(&vd->st.bad_pose, kBadPose);
    fan_sector_axis(d, fan, width, k - f * fan.sectors);
    vd->frames[k] = d;
}

// K3a for fan frames.
__global__ void __launch_bounds__(256) k_mark_fan(VolDev* vd, int w, int h, PatchShape shape, FanArgs fan, int f0) {
    mark_patch<true>(vd, w, h, shape, 0.0, 0.0, &fan, f0);
}

// Undo the marks of a rejected batch and restore the codebook size.
__global__ void k_rollback(VolDev* vd, uint32_t new_count, uint32_t dirty_count, int K0, int sat0) {
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < new_count && k < vd->cap) vd->table[vd->new_list[k]] = -1;
    if (k < dirty_count) vd->dirty_flags[vd->dirty_list[k]] = 0u;
    if (k == 0) {
        vd->st.new_count = 0u;
        vd->st.dirty_count = 0u;
        vd->st.K = K0;
        vd->st.saturated = sat0;
        vd->st.bad_pose = 0;
    }
}

// K3b: give each marked entry the next pool slot, zero its accumulators and
// queue it for finalisation.
__global__ void __launch_bounds__(256) k_alloc(VolDev* vd, uint32_t new_count, uint32_t used,
                                               uint32_t dirty_count) {
    const uint32_t k = blockIdx.x;
    const uint32_t slot = used + k;
    unsigned long long* acc = vd->acc + (size_t)slot * kBrickVox;
    acc[threadIdx.x] = 0ull;
    acc[threadIdx.x + 256] = 0ull;
    if (threadIdx.x == 0) {
        vd->table[vd->new_list[k]] = (int32_t)slot;
        vd->dirty_flags[slot] = 1u;
        vd->dirty_list[dirty_count + k] = (int32_t)slot;
        if (k == 0) {
            vd->st.used = used + new_count;
            vd->st.dirty_count = dirty_count + new_count;
            vd->st.new_count = 0u;
        }
    }
}

// Pixels of one voxel among a wave's 8 x 8 block are added up before they go to memory: halving
// steps along the rows, then across them, each lane taking over its partner's sum where both hold
// the same (slot, voxel); `place` of a lane taken over becomes -1.  Steps are skipped once no
// lane has such a partner (frames at a voxel per pixel: one comparison).
template <int D>
__device__ __forceinline__ int lane_plus(int x) {   // lane + D's value, D within a row of 16 lanes
    return __builtin_amdgcn_update_dpp(0, x, 0x100 + D, 0xF, 0xF, true);
}
template <int D>
__device__ __forceinline__ bool merge_step(int lane, int& place, int local, uint32_t& add) {
    int op, ol;
    uint32_t oa;
    if constexpr (D < 16) {
        op = lane_plus<D>(place);
        ol = lane_plus<D>(local);
        oa = (uint32_t)lane_plus<D>((int)add);
    } else {
        op = __shfl_down(place, D);
        ol = __shfl_down(local, D);
        oa = (uint32_t)__shfl_down((int)add, D);
    }
    const bool take = (lane & (2 * D - 1)) < D && (D >= 8 || (lane & (D - 1)) == 0) && place >= 0 && op == place && ol == local;
    const unsigned long long m = __ballot(take);
    if (take) add += oa;
    if ((m >> ((lane - D) & 63)) & 1ull && lane >= D) place = -1;
    return m != 0;
}
__device__ __forceinline__ void merge_pixels(int& place, int local, uint32_t& add) {
    const int lane = threadIdx.x & 63;
    if (merge_step<1>(lane, place, local, add) && merge_step<2>(lane, place, local, add)) merge_step<4>(lane, place, local, add);
    if (merge_step<8>(lane, place, local, add) && merge_step<16>(lane, place, local, add)) merge_step<32>(lane, place, local, add);
}

// K4: add each pixel's intensity and a count to its (bin, voxel).  Bound by the rate at which
// memory takes the atomic requests (all go past the L2s, which do not share lines between XCDs):
// 37 M requests of up to 64 bytes for the 100 M in-grid pixels of 1800 frames of 256^2, 1660 us.  With
// the wave's 64 pixels along a row instead of an 8 x 8 block it was 2730 us.  Merging pixels of one
// voxel first takes 300 fan frames (about 6 pixels a voxel) from 523 to 188 us.
template <bool FAN>
__device__ __forceinline__ void accumulate_patch(const VolDev* __restrict__ vd, const uint8_t* __restrict__ frames,
                                                 int w, int h, const PatchShape& shape, double sx, double sy,
                                                 const FanArgs* fan, int f0) {
    const Patch p = frame_patch(shape, f0);
    const FramePixels<FAN> px(vd, fan, p.f, w);
    const gptr<unsigned long long> acc = (gptr<unsigned long long>)((cptr<VolDev>)vd)->acc;
    const gptr<const uint8_t> img = (gptr<const uint8_t>)frames + (size_t)p.f * w * h;
    // the four pixels and their table entries, all loads in flight together (a lane without a
    // voxel reads entry 0 of each, and drops what it reads)
    int64_t e[4];
    int local[4], slot[4];
    uint32_t inten[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const PatchPixel at = patch_pixel(shape, p, b);
        e[b] = px.entry(at.i, at.j, h, sx, sy, local[b]);
        inten[b] = img[e[b] >= 0 ? (size_t)at.j * w + at.i : 0];
        slot[b] = ((gptr<const int32_t>)px.v.table)[e[b] >= 0 ? e[b] : 0];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        // slot < 0 is unreachable: every entry hit was marked and allocated
        int place = e[b] >= 0 ? slot[b] : -1;
        uint32_t add = inten[b] << 8 | 1u;   // sum and count of up to 64 pixels
        merge_pixels(place, local[b], add);
        if (place >= 0)
            __hip_atomic_fetch_add(acc + (size_t)place * kBrickVox + local[b],
                                   ((unsigned long long)(add >> 8) << 32) | (add & 255u), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void __launch_bounds__(256) k_accumulate(const VolDev* __restrict__ vd, const uint8_t* __restrict__ frames,
                                                    int w, int h, PatchShape shape, double sx, double sy, int f0) {
    accumulate_patch<false>(vd, frames, w, h, shape, sx, sy, nullptr, f0);
}

// K4 for fan frames.
__global__ void __launch_bounds__(256) k_accumulate_fan(const VolDev* __restrict__ vd,
                                                        const uint8_t* __restrict__ frames, int w, int h,
                                                        PatchShape shape, FanArgs fan, int f0) {
    accumulate_patch<true>(vd, frames, w, h, shape, 0.0, 0.0, &fan, f0);
}

// K5: exact sums -> stored (value, count) pairs of every dirty slot.
template <int DT>
__global__ void __launch_bounds__(256) k_finalize(VolDev* vd) {
    __shared__ float red[2][4];
    const int slot = vd->dirty_list[blockIdx.x];
    const unsigned long long* acc = vd->acc + (size_t)slot * kBrickVox;
    float a[2], c[2];
    uint32_t C[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const unsigned long long u = acc[threadIdx.x + 256 * k];
        C[k] = (uint32_t)(u & 0xFFFFFFFFull);
        const uint32_t S = (uint32_t)(u >> 32);
        c[k] = (float)C[k];
        a[k] = C[k] ? (float)S / c[k] : 0.0f;
    }
    const size_t base = (size_t)slot * kBrickVox;
    const float inv = 1.0f / 127.5f;
    if constexpr (DT == DARE_F32) {
        float2* d = (float2*)vd->data + base;
#pragma unroll
        for (int k = 0; k < 2; ++k) d[threadIdx.x + 256 * k] = make_float2(a[k], c[k]);
    } else if constexpr (DT == DARE_BF16 || DT == DARE_F16) {
        uint32_t* d = (uint32_t*)vd->data + base;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t q = 0u, qc = 0u;
            if (C[k]) {
                const float x = (a[k] - 127.5f) * inv;
                if constexpr (DT == DARE_BF16) {
                    q = f32_to_bf16_rne(x);
                    qc = f32_to_bf16_rne(c[k]);
                } else {
                    q = f32_to_f16_rne(x);
                    qc = f32_to_f16_rne(fminf(c[k], 65504.0f));
                }
            }
            d[threadIdx.x + 256 * k] = q | (qc << 16);
        }
    } else {
        // per-brick scales: largest |a - 127.5| and largest count over occupied voxels
        float m = 0.0f, cm = 0.0f;
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (C[k]) {
                m = fmaxf(m, fabsf(a[k] - 127.5f));
                cm = fmaxf(cm, c[k]);
            }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            m = fmaxf(m, __shfl_xor(m, off));
            cm = fmaxf(cm, __shfl_xor(cm, off));
        }
        if ((threadIdx.x & 63) == 0) {
            red[0][threadIdx.x >> 6] = m;
            red[1][threadIdx.x >> 6] = cm;
        }
        __syncthreads();
        m = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
        cm = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
        const float s = fmaxf(m / 448.0f, 9.5367431640625e-07f);   // floor 2^-20
        const float t = cm > 0.0f ? cm / 448.0f : 1.0f;
        uint16_t* d = (uint16_t*)vd->data + base;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t q = 0u, qc = 0u;
            if (C[k]) {
                q = f32_to_e4m3_rne((a[k] - 127.5f) / s);
                qc = f32_to_e4m3_rne(c[k] / t);
            }
            d[threadIdx.x + 256 * k] = (uint16_t)(q | (qc << 8));
        }
        if (threadIdx.x == 0) vd->scales[slot] = make_float2(s, t);
    }
    if (threadIdx.x == 0) {
        vd->dirty_flags[slot] = 0u;
        if (blockIdx.x == 0) vd->st.dirty_count = 0u;
    }
}

// Marks (-2) of a rejected batch that did not fit the new-entry list.
__global__ void k_clear_marks(int32_t* t, int64_t n) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        if (t[k] == -2) t[k] = -1;
}

__global__ void k_table_fill(int32_t* t, int64_t n) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        t[k] = -1;
}

// Test hooks: dense (bin, z, y, x) arrays <-> the bricked pool.
__global__ void k_dense_mark(VolDev* vd, const uint32_t* __restrict__ C, int K) {
    const int64_t nvox = (int64_t)vd->nx * vd->ny * vd->nz;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nvox * K;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (C[k] == 0u) continue;
        const int b = (int)(k / nvox);
        int64_t r = k - b * nvox;
        const int vx = (int)(r % vd->nx);
        r /= vd->nx;
        const int vy = (int)(r % vd->ny);
        const int vz = (int)(r / vd->ny);
        mark_one(vd, brick_entry(vd, b, vx, vy, vz));
    }
}

__global__ void k_dense_scatter(const VolDev* vd, const uint32_t* __restrict__ S, const uint32_t* __restrict__ C,
                                int K) {
    const int64_t nvox = (int64_t)vd->nx * vd->ny * vd->nz;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nvox * K;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (C[k] == 0u) continue;
        const int b = (int)(k / nvox);
        int64_t r = k - b * nvox;
        const int vx = (int)(r % vd->nx);
        r /= vd->nx;
        const int vy = (int)(r % vd->ny);
        const int vz = (int)(r / vd->ny);
        const int slot = vd->table[brick_entry(vd, b, vx, vy, vz)];
        vd->acc[(size_t)slot * kBrickVox + brick_local(vx, vy, vz)] =
            ((unsigned long long)S[k] << 32) | (unsigned long long)C[k];
    }
}

// Every voxel's exact sum and count as dense arrays.  A wave takes a row of 8 bricks along x (64
// voxels; 4, 2 or 1 bricks where the grid is that narrow, and as many more rows of y at a time) and
// stores it row by row, so that the waves of a workgroup, at consecutive rows of bricks, fill long
// runs in order; its loads go cube by cube, so each line of a brick is read once.  Bound by the bytes
// (3.5 GB written and 2 GB read for 26 bins of 256^3): 1150 us, 4.8 TB/s; a thread per voxel index,
// with its 64-bit divisions, took 2610 us, and rows of 8 bricks stored 64 rows apart (8 waves' worth
// of scattered 256-byte pieces) 3930 us.  6 bins of 8 x 256 x 256, the whole call: 29 us, 51 in rows
// of 64, 39 by voxel index.
template <int LW>                           // log2 of the voxels along x
__global__ void __launch_bounds__(256) k_download_sums(const VolDev* __restrict__ vd, uint32_t* __restrict__ S,
                                                       uint32_t* __restrict__ C, int64_t first, int64_t items) {
    constexpr int kRows = 64 >> LW, kSteps = 8 / kRows;             // rows of y at a time, and how often
    constexpr int kLoads = LW == 6 ? 16 : 8, kZ = kLoads / kSteps;   // in flight at a time
    int64_t g = first + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // (bin, bz, by, row of bricks)
    if (g >= items) return;
    const int nx = vd->nx, ny = vd->ny, nz = vd->nz, nxr = (nx + (1 << LW) - 1) >> LW;
    const int lane = threadIdx.x & 63;
    const int vx = (int)(g % nxr) * (1 << LW) + (lane & ((1 << LW) - 1)), dy = lane >> LW;
    g /= nxr;
    const int y0 = (int)(g % vd->nby) * 8;
    g /= vd->nby;
    const int z0 = (int)(g % vd->nbz) * 8, bin = (int)(g / vd->nbz);
    const bool in = vx < nx;
    const int slot = in ? vd->table[brick_entry(vd, bin, vx, y0, z0)] : -1;
    const gptr<const unsigned long long> acc = (gptr<const unsigned long long>)vd->acc + (size_t)max(slot, 0) * kBrickVox;
#pragma unroll 1
    for (int z = 0; z < 8; z += kZ) {
        unsigned long long u[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            u[k] = 0ull;
            if (slot >= 0) u[k] = acc[brick_local(vx, k / kZ * kRows + dy, z + k % kZ)];
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int step = k % kSteps, dz = k / kSteps;
            const int vz = z0 + z + dz, vy = y0 + step * kRows + dy;
            const unsigned long long x = u[step * kZ + dz];
            if (!in || vy >= ny || vz >= nz) continue;
            const size_t at = (((size_t)bin * nz + vz) * ny + vy) * nx + vx;
            // written once, read by no kernel here: past the caches
            __builtin_nontemporal_store((uint32_t)(x >> 32), S + at);
            __builtin_nontemporal_store((uint32_t)(x & 0xFFFFFFFFull), C + at);
        }
    }
}

template <int DT>
__global__ void k_download_storage(const VolDev* vd, float* __restrict__ A, float* __restrict__ Cout, int K) {
    using P = Pair<DT>;
    const int64_t nvox = (int64_t)vd->nx * vd->ny * vd->nz;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nvox * K;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(k / nvox);
        int64_t r = k - b * nvox;
        const int vx = (int)(r % vd->nx);
        r /= vd->nx;
        const int vy = (int)(r % vd->ny);
        const int vz = (int)(r / vd->ny);
        const int slot = vd->table[brick_entry(vd, b, vx, vy, vz)];
        float a = 0.0f, c = 0.0f;
        if (slot >= 0) {
            const typename P::T p = ((const typename P::T*)vd->data)[(size_t)slot * kBrickVox + brick_local(vx, vy, vz)];
            const float2 s = DT == DARE_FP8_E4M3 ? vd->scales[slot] : make_float2(0.0f, 0.0f);
            P::decode(p, s, a, c);
            if (!(c > 0.0f)) { a = 0.0f; c = 0.0f; }
        }
        A[k] = a;
        Cout[k] = c;
    }
}

__global__ void k_copy_probe(const uint4* __restrict__ src, uint4* __restrict__ dst, uint64_t n) {
    for (uint64_t k = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; k < n; k += (uint64_t)gridDim.x * blockDim.x)
        dst[k] = src[k];
}

// ---------------------------------------------------------------------------- launchers

static inline int grid_for(int64_t n, int block, int cap = 65536) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    return (int)(g > cap ? cap : g);
}

hipError_t launch_compose_frames(const VolDev* vd, const float* poses, int n, hipStream_t stream) {
    hipLaunchKernelGGL(k_compose_frames, dim3((n + 63) / 64), dim3(64), 0, stream, const_cast<VolDev*>(vd), poses, n);
    return hipGetLastError();
}

hipError_t launch_assign_bins(VolDev* vd, int n, int K0, hipStream_t stream) {
    hipLaunchKernelGGL(k_assign_bins, dim3(1), dim3(kAssign), 0, stream, vd, n, K0);
    return hipGetLastError();
}

hipError_t launch_mark_pixels(const VolDev* vd, int n, int w, int h, double sx, double sy, hipStream_t stream) {
    const PatchShape shape = patch_shape(w, h);
    const int np = shape.nx * shape.ny, fc = frames_per_launch(n, shape);
    for (int f0 = 0; f0 < n; f0 += fc)
        hipLaunchKernelGGL(k_mark_pixels, dim3(np * std::min(fc, n - f0)), dim3(256), 0, stream,
                           const_cast<VolDev*>(vd), w, h, shape, sx, sy, f0);
    return hipGetLastError();
}

hipError_t launch_compose_fan(const VolDev* vd, const float* poses, int n, const FanArgs& fan, int width,
                              hipStream_t stream) {
    const int m = n * fan.sectors;
    hipLaunchKernelGGL(k_compose_fan, dim3((m + 63) / 64), dim3(64), 0, stream, const_cast<VolDev*>(vd), poses, n, fan,
                       width);
    return hipGetLastError();
}

hipError_t launch_mark_fan(const VolDev* vd, int n, int w, int h, const FanArgs& fan, hipStream_t stream) {
    const PatchShape shape = patch_shape(w, h);
    const int np = shape.nx * shape.ny, fc = frames_per_launch(n, shape);
    for (int f0 = 0; f0 < n; f0 += fc)
        hipLaunchKernelGGL(k_mark_fan, dim3(np * std::min(fc, n - f0)), dim3(256), 0, stream,
                           const_cast<VolDev*>(vd), w, h, shape, fan, f0);
    return hipGetLastError();
}

hipError_t launch_accumulate_fan(const VolDev* vd, const uint8_t* frames, int n, int w, int h, const FanArgs& fan,
                                 hipStream_t stream) {
    const PatchShape shape = patch_shape(w, h);
    const int np = shape.nx * shape.ny, fc = frames_per_launch(n, shape);
    for (int f0 = 0; f0 < n; f0 += fc)
        hipLaunchKernelGGL(k_accumulate_fan, dim3(np * std::min(fc, n - f0)), dim3(256), 0, stream, vd, frames, w, h,
                           shape, fan, f0);
    return hipGetLastError();
}

hipError_t launch_rollback(VolDev* vd, uint32_t new_count, uint32_t dirty_count, int K0, int sat0,
                           hipStream_t stream) {
    const uint32_t m = new_count > dirty_count ? new_count : dirty_count;
    hipLaunchKernelGGL(k_rollback, dim3(grid_for(m ? m : 1, 256)), dim3(256), 0, stream, vd, new_count,
                       dirty_count, K0, sat0);
    return hipGetLastError();
}

hipError_t launch_alloc(VolDev* vd, uint32_t new_count, uint32_t used, uint32_t dirty_count, hipStream_t stream) {
    if (new_count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_alloc, dim3(new_count), dim3(256), 0, stream, vd, new_count, used, dirty_count);
    return hipGetLastError();
}

hipError_t launch_accumulate(const VolDev* vd, const uint8_t* frames, int n, int w, int h, double sx, double sy,
                             hipStream_t stream) {
    const PatchShape shape = patch_shape(w, h);
    const int np = shape.nx * shape.ny, fc = frames_per_launch(n, shape);
    for (int f0 = 0; f0 < n; f0 += fc)
        hipLaunchKernelGGL(k_accumulate, dim3(np * std::min(fc, n - f0)), dim3(256), 0, stream, vd, frames, w, h,
                           shape, sx, sy, f0);
    return hipGetLastError();
}

hipError_t launch_finalize(VolDev* vd, int dtype, uint32_t dirty_count, hipStream_t stream) {
    if (dirty_count == 0) return hipSuccess;
    switch (dtype) {
        case DARE_F32: hipLaunchKernelGGL(k_finalize<DARE_F32>, dim3(dirty_count), dim3(256), 0, stream, vd); break;
        case DARE_BF16: hipLaunchKernelGGL(k_finalize<DARE_BF16>, dim3(dirty_count), dim3(256), 0, stream, vd); break;
        case DARE_F16: hipLaunchKernelGGL(k_finalize<DARE_F16>, dim3(dirty_count), dim3(256), 0, stream, vd); break;
        case DARE_FP8_E4M3:
            hipLaunchKernelGGL(k_finalize<DARE_FP8_E4M3>, dim3(dirty_count), dim3(256), 0, stream, vd);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_clear_marks(int32_t* table, int64_t n, hipStream_t stream) {
    hipLaunchKernelGGL(k_clear_marks, dim3(grid_for(n, 256, 4096)), dim3(256), 0, stream, table, n);
    return hipGetLastError();
}

hipError_t launch_table_fill(int32_t* table, int64_t n, hipStream_t stream) {
    hipLaunchKernelGGL(k_table_fill, dim3(grid_for(n, 256, 4096)), dim3(256), 0, stream, table, n);
    return hipGetLastError();
}

hipError_t launch_dense_mark(const VolDev* vd, const uint32_t* C, int K, hipStream_t stream) {
    hipLaunchKernelGGL(k_dense_mark, dim3(4096), dim3(256), 0, stream, const_cast<VolDev*>(vd), C, K);
    return hipGetLastError();
}

hipError_t launch_dense_scatter(const VolDev* vd, const uint32_t* S, const uint32_t* C, int K, hipStream_t stream) {
    hipLaunchKernelGGL(k_dense_scatter, dim3(4096), dim3(256), 0, stream, vd, S, C, K);
    return hipGetLastError();
}

hipError_t launch_download_sums(const VolDev* vd, uint32_t* S, uint32_t* C, int K, int nx, int ny, int nz,
                                hipStream_t stream) {
    const int lw = nx <= 8 ? 3 : nx <= 16 ? 4 : nx <= 32 ? 5 : 6;
    const int64_t rows = (int64_t)((nx + (1 << lw) - 1) >> lw) * ((ny + 7) / 8) * ((nz + 7) / 8), items = rows * K;
    auto* const kernel = lw == 3 ? k_download_sums<3> : lw == 4 ? k_download_sums<4> : lw == 5 ? k_download_sums<5> : k_download_sums<6>;
    const int64_t most = (int64_t)1 << 25;   // waves per launch: a launch takes at most 2^32 - 1 threads
    for (int64_t first = 0; first < items; first += most)
        hipLaunchKernelGGL(kernel, dim3((unsigned)((std::min(most, items - first) + 3) / 4)), dim3(256), 0, stream, vd, S, C,
                           first, std::min(items, first + most));
    return hipGetLastError();
}

hipError_t launch_download_storage(const VolDev* vd, int dtype, float* A, float* C, int K, int, int, int,
                                   hipStream_t stream) {
    switch (dtype) {
        case DARE_F32: hipLaunchKernelGGL(k_download_storage<DARE_F32>, dim3(4096), dim3(256), 0, stream, vd, A, C, K); break;
        case DARE_BF16: hipLaunchKernelGGL(k_download_storage<DARE_BF16>, dim3(4096), dim3(256), 0, stream, vd, A, C, K); break;
        case DARE_F16: hipLaunchKernelGGL(k_download_storage<DARE_F16>, dim3(4096), dim3(256), 0, stream, vd, A, C, K); break;
        case DARE_FP8_E4M3:
            hipLaunchKernelGGL(k_download_storage<DARE_FP8_E4M3>, dim3(4096), dim3(256), 0, stream, vd, A, C, K);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_copy_probe(const void* src, void* dst, uint64_t n, hipStream_t stream) {
    const uint64_t n16 = n / 16;
    hipLaunchKernelGGL(k_copy_probe, dim3(grid_for((int64_t)n16, 256, 256 * 64)), dim3(256), 0, stream,
                       (const uint4*)src, (uint4*)dst, n16);
    return hipGetLastError();
}

}  // namespace dare
