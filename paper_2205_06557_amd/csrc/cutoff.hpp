// cutoff.hpp -- ion-ion forces with a cutoff distance and switching function
// (the paper's option for long domains, Section 4).
//
// The pair energy phi(r) = C e^-r / r is multiplied by the smooth step
// S(r) = 1 - 6x^5 + 15x^4 - 10x^3, x = clamp((r - r_sw) / (r_cut - r_sw), 0, 1),
// and the force is -d(phi S)/dr; S and S' vanish from r_cut on, so pairs
// beyond the cutoff contribute exactly zero without a branch.
//
// Every step the ions are sorted into layers along z and, within a layer,
// along a Hilbert curve over the cross section, so that 64 consecutive ions
// fill a compact box (layers of about the side of a cube of 64 ions; the
// order within a bin is by ion, so it, and with it every floating-point sum,
// is deterministic):
//   cut_bin_kernel       bin of each ion, its arrival number there (atomic)
//   cut_scan_kernel      per layer, prefix sum over its bins
//   cut_start_kernel     first slot of each layer
//   cut_place_kernel     ions to their bins' slots, in arrival order
//   cut_order_kernel     slots of a bin in ion order; sorted positions
//   cut_box_kernel       bounding box of every 64 sorted ions
// Pairs are then taken once each (as in pairsym.hpp): a block of 256
// consecutive sorted ions (tile I) meets the sorted tiles J = I .. J1 - 1,
// where J1 ends at the last source of the layers within reach above its own
// (pair_cut_kernel).  A pair within r_cut with its lower member in tile I has
// its upper member there.  From their boxes, 64 targets and 64 sources are
// skipped where none are within r_cut and take the plain term where all are
// within r_sw.  The totals go to int64 fixed-point accumulators indexed by
// sorted slot; pair_cut_epilogue writes the accelerations back to the ions'
// own slots.
#pragma once

#include "kernels.hpp"
#include "pairsym.hpp"

namespace odk {

constexpr int kMaxSlabs = 1024;

struct CutArgs {
    int nslab;        // slabs that od_get_cutoff_info counts in
    int nblk;         // blocks of 256 ions
    int reach;        // slabs on either side that can hold a source within r_cut
    int nlay, lreach; // sort layers along z; layers above that can hold one
    int side;         // cells of the cross section per axis, a power of two
    float z0;         // lower end of the domain, -H/2
    float inv_w;      // 1 / slab width
    float inv_l;      // 1 / layer width
    float x0, inv_c;  // -R, 1 / cell width
    float rsw;        // start of the switching interval
    float inv_sw;     // 1 / (r_cut - r_sw)
    float skip2, plain2;    // squared box distances beyond and below which a term is zero or plain
};

// Device buffers of the sort.
struct CutBufs {
    int* key;         // [N] bin of each ion
    int* arr;         // [N] arrival number
    int* temp;        // [N] ions by slot, in arrival order
    int* count;       // [nlay * side^2] ions per bin; zero between steps
    int* rel;         // [nlay][side^2 + 1] bin starts within the layer
    int* lay;         // [nlay + 1] first slot of each layer
    int* slab_total;  // [nslab], zero between steps
    int* slab_start;  // [nslab + 1]
    float* box;       // [6][4 nblk] min x, y, z, max x, y, z of 64 sorted ions
};

__device__ __forceinline__ int cut_bin(float z, float z0, float inv, int n)
{
    return min(max((int)((z - z0) * inv), 0), n - 1);
}

// Position along the Hilbert curve through side x side cells: the textbook loop
// from coordinates to distance, a quadrant per bit, turned and mirrored so that
// the next one starts in the corner where this one is entered.
__device__ __forceinline__ int hilbert(int side, int x, int y)
{
    int d = 0;
    for (int s = side >> 1; s > 0; s >>= 1) {
        const int rx = (x & s) != 0, ry = (y & s) != 0;
        d += s * s * ((3 * rx) ^ ry);
        if (!ry) {
            if (rx) {
                x = s - 1 - x;
                y = s - 1 - y;
            }
            const int t = x;
            x = y;
            y = t;
        }
    }
    return d;
}

__global__ __launch_bounds__(256) void cut_bin_kernel(const float* __restrict__ x, long long plane, int N, CutArgs c,
                                                      CutBufs b)
{
    __shared__ int hist[kMaxSlabs];
    for (int s = threadIdx.x; s < c.nslab; s += 256) hist[s] = 0;
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x, at = min(i, N - 1);
    const float z = x[2 * plane + at];
    const int cx = cut_bin(x[at], c.x0, c.inv_c, c.side), cy = cut_bin(x[plane + at], c.x0, c.inv_c, c.side);
    const int key = cut_bin(z, c.z0, c.inv_l, c.nlay) * c.side * c.side + hilbert(c.side, cx, cy);
    const int arr = arrive(b.count, key, i < N);
    if (i < N) {
        b.key[i] = key;
        b.arr[i] = arr;
        atomicAdd(&hist[cut_bin(z, c.z0, c.inv_w, c.nslab)], 1);
    }
    __syncthreads();
    for (int s = threadIdx.x; s < c.nslab; s += 256)
        if (hist[s]) atomicAdd(&b.slab_total[s], hist[s]);
}

// Exclusive prefix sum of n values in_k to out[0 .. n], by one block of 256.
template <typename In>
__device__ __forceinline__ void cut_prefix(int n, In in, int* __restrict__ out)
{
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int carry = 0;
    for (int k0 = 0; k0 < n; k0 += 256) {
        const int k = k0 + threadIdx.x, v = k < n ? in(k) : 0;
        int s = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(s, d, 64);
            if (lane >= d) s += u;
        }
        if (lane == 63) wsum[wv] = s;
        __syncthreads();
        int before = carry;
        for (int w = 0; w < wv; ++w) before += wsum[w];
        if (k < n) out[k] = before + s - v;
        carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

__global__ __launch_bounds__(256) void cut_scan_kernel(CutArgs c, CutBufs b)
{
    const int cells = c.side * c.side;
    int* cnt = b.count + (long long)blockIdx.x * cells;
    cut_prefix(cells, [&](int k) { const int v = cnt[k]; cnt[k] = 0; return v; },
               b.rel + (long long)blockIdx.x * (cells + 1));
}

// Block 0: first slot of each layer; block 1: of each slab, as if sorted by it.
__global__ __launch_bounds__(256) void cut_start_kernel(CutArgs c, CutBufs b)
{
    const int cells = c.side * c.side;
    if (blockIdx.x == 0)
        cut_prefix(c.nlay, [&](int k) { return b.rel[(long long)k * (cells + 1) + cells]; }, b.lay);
    else
        cut_prefix(c.nslab, [&](int k) { const int v = b.slab_total[k]; b.slab_total[k] = 0; return v; }, b.slab_start);
}

__device__ __forceinline__ int cut_first(const CutArgs& c, const CutBufs& b, int key, int& n)
{
    const int cells = c.side * c.side, l = key / cells, k = key - l * cells;
    const int* rel = b.rel + (long long)l * (cells + 1) + k;
    n = rel[1] - rel[0];
    return b.lay[l] + rel[0];
}

__global__ __launch_bounds__(256) void cut_place_kernel(int N, CutArgs c, CutBufs b)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    int n;
    b.temp[cut_first(c, b, b.key[i], n) + b.arr[i]] = i;
}

__global__ __launch_bounds__(256) void cut_order_kernel(const float* __restrict__ x, long long plane, int N, CutArgs c,
                                                        CutBufs b, float* __restrict__ xs, int* __restrict__ idx)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= N) return;
    const int i = b.temp[t];
    int n;
    const int first = cut_first(c, b, b.key[i], n);
    const int to = first + count_below(b.temp + first, n, i);
    idx[to] = i;
    xs[to] = x[i];
    xs[plane + to] = x[plane + i];
    xs[2 * plane + to] = x[2 * plane + i];
}

__global__ __launch_bounds__(256) void cut_box_kernel(const float* __restrict__ xs, long long plane, int N, CutArgs c,
                                                      CutBufs b)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    float lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = t < N ? xs[k * plane + t] : 3.0e38f;
        hi[k] = t < N ? lo[k] : -3.0e38f;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            lo[k] = fminf(lo[k], __shfl_xor(lo[k], d, 64));
            hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], d, 64));
        }
    }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            b.box[k * 4 * c.nblk + t / 64] = lo[k];
            b.box[(k + 3) * 4 * c.nblk + t / 64] = hi[k];
        }
}

// The pair terms.  Switched: with t = 1 - 2x, S = 1/2 + (15 t - 10 t^3 + 3 t^5) / 16
// and -S' = 15 (1 - t^2)^2 / (8 (r_cut - r_sw)), the term is
// e^-r / r^2 ((1 + 1/r) S - S'); both are exactly zero at t = -1.
struct CutPlain {
    __device__ __forceinline__ float operator()(float dx, float dy, float dz) const
    {
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        const float ri = __builtin_amdgcn_rsqf(r2);
        const float e = __builtin_amdgcn_exp2f(r2 * ri * -1.4426950408889634f);
        const float ri2 = ri * ri;
        return fmaf(ri2, ri, ri2) * e;
    }
};

struct CutSwitched {
    float t0, t1, ds;           // 1 + 2 r_sw / w, -2 / w, 15 / (8 w) for w = r_cut - r_sw
    __device__ __forceinline__ float operator()(float dx, float dy, float dz) const
    {
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        const float ri = __builtin_amdgcn_rsqf(r2);
        const float r = r2 * ri;
        const float e = __builtin_amdgcn_exp2f(r * -1.4426950408889634f);
        const float t = __builtin_amdgcn_fmed3f(fmaf(r, t1, t0), -1.0f, 1.0f);
        const float tt = t * t, v = fmaf(-t, t, 1.0f);
        const float S = fmaf(t, fmaf(tt, fmaf(tt, 0.1875f, -0.625f), 0.9375f), 0.5f);
        return (ri * ri * e) * fmaf(ri, S, fmaf(ds * v, v, S));
    }
};

// One lane's target against the 64 sources of a sub-tile, with the reactions
// on them (see sym_item).  Sorted neighbours put an ion's largest terms into
// one sum, so it goes to 64 bits after each sub-tile (after a whole tile the
// accelerations' relative error was 2.6e-7 instead of 1.2e-7).
template <typename Pair>
__device__ __forceinline__ void cut_subtile(const float4* base, float xi, float yi, float zi, const Pair& pair,
                                            double s[3], float j[3])
{
    float ax = 0.0f, ay = 0.0f, az = 0.0f, jx = 0.0f, jy = 0.0f, jz = 0.0f;
#pragma unroll 16
    for (int k = 0; k < 64; ++k) {
        const float4 q = base[k];                 // source (lane + k) mod 64
        const float dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
        const float f = pair(dx, dy, dz);
        ax = fmaf(f, dx, ax);
        ay = fmaf(f, dy, ay);
        az = fmaf(f, dz, az);
        jx = fmaf(-f, dx, rotate_down(jx));
        jy = fmaf(-f, dy, rotate_down(jy));
        jz = fmaf(-f, dz, rotate_down(jz));
    }
    s[0] += (double)ax;
    s[1] += (double)ay;
    s[2] += (double)az;
    j[0] = jx; j[1] = jy; j[2] = jz;
}

// Switched forces, each pair once: block (I, y) takes sorted tile I against
// the tiles I + y, I + y + gridDim.y, ... up to the end of the layers within
// reach above its last ion; the sums go to fix (planes Npad apart, sorted
// slots).  Bound by FP32 issue, 31 slots per pair evaluated.  With slabs of
// r_cut / 16 in ion order, one block to a tile and the switched term
// throughout, a pair sum took 20.1 ms at 2^19 ions of the long domain (r_sw =
// 3, r_cut = 4), 6.1 at 2^17 and 1.47 at 2^14 (64 blocks), against 15.1, 3.5
// and 0.20.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8, 8)))
void pair_cut_kernel(const float* __restrict__ xs_sorted, CutBufs b, unsigned long long* __restrict__ fix, PairArgs p,
                     CutArgs c, Ctl* __restrict__ ctl)
{
    static_assert(BLOCK == 256, "four waves of 64");
    __shared__ float4 src[4][128];
    __shared__ float jpart[4][3][BLOCK];
    if (!p.ion_ion) return;
    const long long P = p.Npad;
    const int N = p.N, I = blockIdx.x;
    const float *X = xs_sorted, *Y = X + P, *Z = Y + P;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = I * BLOCK + threadIdx.x;
    const float xi = X[i], yi = Y[i], zi = Z[i];
    const int l_hi = cut_bin(Z[min((I + 1) * BLOCK, N) - 1], c.z0, c.inv_l, c.nlay);
    const int J1 = (b.lay[min(l_hi + c.lreach + 1, c.nlay)] + BLOCK - 1) / BLOCK;
    const CutPlain plain;
    const CutSwitched switched{fmaf(2.0f * c.rsw, c.inv_sw, 1.0f), -2.0f * c.inv_sw, 1.875f * c.inv_sw};
    // lanes 4 w + s (and again from lane 16 on): the boxes of wave w's targets
    // and of sub-tile s, so that every wave knows all sixteen
    const int G = 4 * c.nblk;
    float lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = b.box[k * G + 4 * I + (lane >> 2 & 3)];
        hi[k] = b.box[(k + 3) * G + 4 * I + (lane >> 2 & 3)];
    }
    double s[3] = {0.0, 0.0, 0.0};
    for (int J = I + blockIdx.y; J < J1; J += gridDim.y) {
        float mn = 0.0f, mx = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float l = b.box[k * G + 4 * J + (lane & 3)], h = b.box[(k + 3) * G + 4 * J + (lane & 3)];
            const float gap = fmaxf(fmaxf(l - hi[k], lo[k] - h), 0.0f), span = fmaxf(h - lo[k], hi[k] - l);
            mn = fmaf(gap, gap, mn);
            mx = fmaf(span, span, mx);
        }
        const unsigned near = J == I ? 0xffffu : (unsigned)__ballot(!(mn > c.skip2)) & 0xffffu;
        const unsigned all = (unsigned)__ballot(mx < c.plain2) & 0xffffu;
        if (!near) continue;
        __syncthreads();
        {
            const int j = J * BLOCK + threadIdx.x;
            const float4 q = make_float4(X[j], Y[j], Z[j], 0.0f);
            src[wv][lane] = q;
            src[wv][lane + 64] = q;
        }
        __syncthreads();
        if (J == I) {
            for (int k0 = 0; k0 < BLOCK; k0 += 16) {
                float a[3] = {0.0f, 0.0f, 0.0f};
                for (int k = k0; k < k0 + 16; ++k) {
                    const float4 q = src[k >> 6][k & 63];
                    const float dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
                    float f = switched(dx, dy, dz);
                    f = k == (int)threadIdx.x ? 0.0f : f;
                    a[0] = fmaf(f, dx, a[0]);
                    a[1] = fmaf(f, dy, a[1]);
                    a[2] = fmaf(f, dz, a[2]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) s[k] += (double)a[k];
            }
        } else {
            for (int st = 0; st < 4; ++st) {
                if (!(near >> (4 * wv + st) & 1)) continue;
                float j[3];
                if (all >> (4 * wv + st) & 1)
                    cut_subtile(&src[st][lane], xi, yi, zi, plain, s, j);
                else
                    cut_subtile(&src[st][lane], xi, yi, zi, switched, s, j);
                // after 64 rotations lane l holds source (l + 63) mod 64
                const int sid = st * 64 + ((lane + 63) & 63);
#pragma unroll
                for (int k = 0; k < 3; ++k) jpart[wv][k][sid] = j[k];
            }
            __syncthreads();
            const unsigned waves = near >> wv & 0x1111u;        // that met this thread's source
            const int j = J * BLOCK + threadIdx.x;
            if (waves && j < N)
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    double v = 0.0;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        if (waves >> (4 * w) & 1) v += (double)jpart[w][k][threadIdx.x];
                    atomicAdd(&fix[k * P + j], to_fixed(v, p.sym_scale, &ctl->status));
                }
        }
    }
    if (i < N)
#pragma unroll
        for (int k = 0; k < 3; ++k) atomicAdd(&fix[k * P + i], to_fixed(s[k], p.sym_scale, &ctl->status));
}

// Per sorted slot: converts the totals, adds the pair_epilogue terms and
// writes the acceleration to the ion's own slot; clears the totals.
__global__ __launch_bounds__(256) void pair_cut_epilogue(const float* __restrict__ xs_sorted,
                                                         const int* __restrict__ idx,
                                                         unsigned long long* __restrict__ fix,
                                                         float* __restrict__ acc, PairArgs p,
                                                         DustSet ds, Ctl* __restrict__ ctl)
{
    __shared__ double red[4][kMaxDust][3];
    const int Npad = p.Npad;
    const int i = blockIdx.x * 256 + threadIdx.x;
    const bool live = i < p.N;
    const float xi = xs_sorted[i], yi = xs_sorted[Npad + i], zi = xs_sorted[2 * Npad + i];
    double v[3];
    for (int c = 0; c < 3; ++c) {
        unsigned long long* a = &fix[(long long)c * Npad + i];
        v[c] = live ? from_fixed(*a, p.sym_scale) : 0.0;
        *a = 0ull;
    }
    pair_epilogue<256>(xi, yi, zi, live ? idx[i] : 0, live, p.Cd * v[0], p.Cd * v[1], p.Cd * v[2], true,
                       p, ds, ctl, acc, acc + Npad, acc + 2 * Npad, red);
}

}  // namespace odk
