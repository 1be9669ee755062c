// mesh.hpp -- the all-pairs ion-ion sum of large systems, split into near
// pairs and a smooth far part on a grid (the split and its constants:
// meshplan.hpp).  The direct sum costs N^2 / 2 pair terms however far apart
// the ions are; here a pair is evaluated one by one only within r_c (a few ion
// spacings) and everything else is a few thousand operations per ion, all of
// it in 64 bits.
//
// Launch sequence of one step (all sizes fixed by the plan, so that a step can
// be captured):
//   mesh_bin_kernel      sort bin of every ion: column of kx x kx cells, slice
//                        along z; arrival number within the bin (atomic)
//   mesh_scan_kernel     per column, prefix sum over its bins
//   mesh_cols_kernel     prefix over columns, each padded to whole groups of 16;
//                        what the split would cost with the ions where they are
//   mesh_place_kernel    ion index to its bin's slots, in arrival order
//   mesh_order_kernel    slots of a bin put in ion order (arrival order depends
//                        on scheduling, ion order does not); sorted positions
//   mesh_box_kernel      bounding box of every 8 sorted ions
//   mesh_spread_kernel   charges to the grid, one brick of cells per block
//                        (64-bit MFMA; bricks in LDS as int64, order-free)
//   mesh_sum_kernel      overlapping brick margins added
//   mesh_conv_kernel     Gaussian convolutions along x, y and z (64-bit MFMA)
//   mesh_gather_kernel   far acceleration of every ion, from bricks in LDS
//   mesh_near_kernel     near pairs; totals to the fixed-point planes that the
//                        step's tail reads
//   mesh_direct_kernel   the direct sum instead, where the ions do not suit the
//                        grid: some lie outside the domain (od_set_state may
//                        put them there; they leave it in that step), or so many
//                        lie so close together that the split would cost more
// Which of the two it is, the first three find out on the device, so that it
// holds for every replay of a captured step too; the kernels of the other
// return at once.
// Every sum has a fixed order or is an integer sum: results are reproducible
// bit for bit.
#pragma once

#include "kernels.hpp"
#include "meshplan.hpp"
#include "pairsym.hpp"

namespace odk {

// One system's direct sum, for the steps that call for it.
struct MeshDirect {
    const long long* cost;      // MeshBufs::cost
    long long cost_max;
    const float* x;             // positions and totals, their planes equally far apart
    unsigned long long* fix;
    SymRuns runs;
    int N;
    double scale;
    int* status;
};

// Device buffers of one system's split: its own (mesh_own) and the scratch of
// a step (mesh_scratch), which systems that step one after another share.
struct MeshBufs {
    int* count;            // own: [bins] ions per bin; zero between steps
    double* green;         // own: [m.M][ng] Green's tables
    long long* cost;       // own: [3] near pairs, mark of ions outside the domain, fullest column; see mesh_skip
    MeshDirect* direct;    // own: see mesh_direct_kernel
    float* near0;          // own: constant term of the near polynomial (mesh_zero_kernel)
    int* key;              // [N] sort bin of each ion
    int* arr;              // [N] arrival number in the bin
    int* rel;              // [columns][nzb + 1] bin starts within the column
    int* col;              // [columns + 1] first slot of each column
    int* temp;             // [cap] ions in arrival order, -1 where a column is padded
    int* idx;              // [cap] ion of each sorted slot, -1 for padding
    float4* s;             // [cap] sorted positions
    float* box;            // [6][cap / 8] min x, y, z, max x, y, z of 8 sorted ions
    double* far;           // [3][cap] far part by sorted slot
    double* q;             // grid charges
    double* phi;           // far potential on the grid
    double* t1;            // convolution scratch, mc grids each
    double* t2;
    unsigned long long* brick;  // brick sums (shares t1's memory)
    int mc;                // Gaussians per convolution pass
};

__device__ __forceinline__ int mesh_cell(double x, double lo, double inv_h, int nc)
{
    return (int)fmin(fmax(floor((x - lo) * inv_h), 0.0), (double)(nc - 1));
}

__device__ __forceinline__ int mesh_zbin(double z, const MeshArgs& m)
{
    return (int)fmin(fmax(floor((z + m.Hh) * (m.inv_h * kMeshZsub)), 0.0), (double)(m.nzb - 1));
}

constexpr long long kMeshNever = 1ll << 61;

// Whether the step is summed directly.  Asked where a kernel waits for other
// loads anyway.
__device__ __forceinline__ bool mesh_skip(const long long* cost, long long most) { return cost[0] + cost[2] > most; }

// Sort bin of every ion; also marks every slot empty, and whether ions lie
// outside the domain (by more than the rounding of one on its surface).
__global__ __launch_bounds__(256) void mesh_bin_kernel(const float* __restrict__ x, long long plane, MeshArgs m,
                                                       MeshBufs b)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < m.cap) b.temp[i] = -1;
    const bool live = i < m.N;
    const int at = live ? i : 0;
    const double px = x[at], py = x[plane + at], pz = x[2 * plane + at];
    if (fmax(fabs(px), fabs(py)) > m.R * (1.0 + 1e-6) || fabs(pz) > m.Hh * (1.0 + 1e-6)) b.cost[1] = kMeshNever;
    const int cx = mesh_cell(px, -m.R, m.inv_h, m.nc[0]) / kMeshKx;
    const int cy = mesh_cell(py, -m.R, m.inv_h, m.nc[1]) / kMeshKx;
    const int key = (cy * m.ncx + cx) * m.nzb + mesh_zbin(pz, m);
    const int arr = arrive(b.count, key, live);
    if (!live) return;
    b.key[i] = key;
    b.arr[i] = arr;
}

// One block per column: bin starts relative to the column; clears the counts.
// Block 0 passes the step's mark on.
__global__ __launch_bounds__(256) void mesh_scan_kernel(MeshArgs m, MeshBufs b)
{
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        b.cost[0] = b.cost[1];
        b.cost[1] = b.cost[2] = 0;
    }
    int* cnt = b.count + (long long)blockIdx.x * m.nzb;
    int* rel = b.rel + (long long)blockIdx.x * (m.nzb + 1);
    int carry = 0;
    for (int k0 = 0; k0 < m.nzb; k0 += 256) {
        const int k = k0 + threadIdx.x;
        const int v = k < m.nzb ? cnt[k] : 0;
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
        if (k < m.nzb) {
            rel[k] = before + s - v;
            cnt[k] = 0;
        }
        carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) rel[m.nzb] = carry;
}

// What the split would cost with the ions where they are: pairs of the ions of
// every column, in slabs as high as a brick, with those of the columns and slabs
// within r_c, and the fullest of them.  Cell k of this thread, then every
// `threads` further on.
__device__ __forceinline__ void mesh_cost(const MeshArgs& m, const MeshBufs& b, int k, int threads)
{
    const int ns = (m.nzb + kMeshSlab - 1) / kMeshSlab, cells = m.ncx * m.ncy * ns;
    auto ions = [&](int c, int z0, int z1) {
        const int* rel = b.rel + (long long)c * (m.nzb + 1);
        return rel[min(z1 * kMeshSlab, m.nzb)] - rel[max(z0, 0) * kMeshSlab];
    };
    constexpr int reach = (int)(kMeshRatio / kMeshKx + 1.0);
    long long near = 0, top = 0;
    for (; k < cells; k += threads) {
        const int c = k / ns, z = k - c * ns, cx = c % m.ncx, cy = c / m.ncx, n = ions(c, z, z + 1);
        // without branches, so that the loads are in flight together
        int w = 0;
#pragma unroll
        for (int dy = -reach; dy <= reach; ++dy)
#pragma unroll
            for (int dx = -reach; dx <= reach; ++dx) {
                const int x = min(max(cx + dx, 0), m.ncx - 1), y = min(max(cy + dy, 0), m.ncy - 1);
                const int q = ions(y * m.ncx + x, z - 1, z + 2);
                w += x == cx + dx && y == cy + dy ? q : 0;
            }
        near += (long long)n * w;
        top = max(top, (long long)(n * (kMeshColumnNs / kMeshPairNs)));
    }
    near = wave_sum(near);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) top = max(top, __shfl_xor(top, d, 64));
    if ((threadIdx.x & 63) == 0 && near > 0) {
        atomicAdd((unsigned long long*)&b.cost[0], (unsigned long long)near);
        atomicMax((unsigned long long*)&b.cost[2], (unsigned long long)top);
    }
}

// Block 0: first slot of each column; the others: the step's cost.
__global__ __launch_bounds__(1024) void mesh_cols_kernel(MeshArgs m, MeshBufs b)
{
    __shared__ int wsum[16];
    if (blockIdx.x > 0) {
        // one wave of each: the loads are scattered, and few of them to a compute unit at a time
        if (threadIdx.x < 64) mesh_cost(m, b, (blockIdx.x - 1) * 64 + threadIdx.x, (gridDim.x - 1) * 64);
        return;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ncol = m.ncx * m.ncy;
    int carry = 0;
    for (int k0 = 0; k0 < ncol; k0 += 1024) {
        const int k = k0 + threadIdx.x;
        const int v = k < ncol ? (b.rel[(long long)k * (m.nzb + 1) + m.nzb] + kMeshTile - 1) / kMeshTile * kMeshTile : 0;
        int s = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(s, d, 64);
            if (lane >= d) s += u;
        }
        if (lane == 63) wsum[wv] = s;
        __syncthreads();
        int before = carry, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wv) before += wsum[w];
            all += wsum[w];
        }
        if (k < ncol) b.col[k] = before + s - v;
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) b.col[ncol] = carry;
}

__device__ __forceinline__ int mesh_bin_start(const MeshArgs& m, const MeshBufs& b, int key)
{
    const int c = key / m.nzb;
    return b.col[c] + b.rel[(long long)c * (m.nzb + 1) + (key - c * m.nzb)];
}

__global__ __launch_bounds__(256) void mesh_place_kernel(MeshArgs m, MeshBufs b)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < m.N) b.temp[mesh_bin_start(m, b, b.key[i]) + b.arr[i]] = i;
}

// Slot order within a bin by ion index; sorted positions.  Padding slots stand
// outside the domain, more than r_c from every ion and near enough that the
// near part's rounding at r_c times their distance is nothing.
__global__ __launch_bounds__(256) void mesh_order_kernel(const float* __restrict__ x, long long plane, MeshArgs m,
                                                         MeshBufs b)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (mesh_skip(b.cost, m.cost_max) | (t >= b.col[m.ncx * m.ncy])) return;
    const int i = b.temp[t];
    if (i < 0) {
        b.idx[t] = -1;
        b.s[t] = make_float4((float)m.R + 2.0f, (float)m.R + 2.0f, (float)m.Hh + 2.0f, 0.0f);
        return;
    }
    const int key = b.key[i];
    const int c = key / m.nzb, z = key - c * m.nzb;
    const int* rel = b.rel + (long long)c * (m.nzb + 1);
    const int s0 = b.col[c] + rel[z], s1 = b.col[c] + rel[z + 1];
    const int to = s0 + count_below(b.temp + s0, s1 - s0, i);
    b.idx[to] = i;
    b.s[to] = make_float4(x[i], x[plane + i], x[2 * plane + i], 0.0f);
}

// Bounding box of every 8 sorted ions (empty: an inverted box).
__global__ __launch_bounds__(256) void mesh_box_kernel(MeshArgs m, MeshBufs b)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (mesh_skip(b.cost, m.cost_max) | (t >= b.col[m.ncx * m.ncy])) return;     // a multiple of 16
    const bool live = b.idx[t] >= 0;
    const int ns = m.cap / kMeshSub;
    const float4 p = b.s[t];
    const float at[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float v = at[c];
        float lo = live ? v : 1.0e30f, hi = live ? v : -1.0e30f;
#pragma unroll
        for (int d = 1; d < kMeshSub; d <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, d, 64));
            hi = fmaxf(hi, __shfl_xor(hi, d, 64));
        }
        if ((threadIdx.x & (kMeshSub - 1)) == 0) {
            b.box[(long long)c * ns + t / kMeshSub] = lo;
            b.box[(long long)(c + 3) * ns + t / kMeshSub] = hi;
        }
    }
}

// Window weights of the ten nodes around a coordinate u cells from its cell's
// lower edge, and their derivatives along the axis per cell when DER; z = ((u + 4 - k) / 5.
template <bool DER>
__device__ __forceinline__ double mesh_window(const MeshArgs& m, double u, int k, double& der)
{
    const double z = (u + (4.0 - k)) * 0.2;
    const double s = fma(-2.0 * z, z, 1.0);
    double p = m.win[kMeshWDeg], d = 0.0;
#pragma unroll
    for (int j = kMeshWDeg - 1; j >= 0; --j) {
        if (DER) d = fma(d, s, p);
        p = fma(p, s, m.win[j]);
    }
    if (DER) der = d * (-0.8 * z);             // ds/dz = -4 z, dz = 1/5 per cell
    return p;
}

// A brick is 4 x 4 columns of 4 x 4 cells and 7 cells along z; the ions of one
// column reach 13 x 13 x 16 of its nodes.
constexpr int kMeshReach = kMeshKx + kMeshP - 1;        // 13
constexpr int kMeshThreads = 512;
static_assert(kMeshReach <= 16 && kMeshBz + kMeshP - 1 == 16, "one MFMA tile spans a column's nodes");

typedef double mesh4 __attribute__((ext_vector_type(4)));

// Cells of a brick's column k and its ions' slots.
struct MeshColumn {
    int x, y, z;        // first cells
    int s0, s1;         // slots
};

__device__ __forceinline__ MeshColumn mesh_column(const MeshArgs& m, const MeshBufs& b, int k)
{
    MeshColumn c;
    const int bx = blockIdx.x % m.nbx, by = blockIdx.x / m.nbx % m.nby, bz = blockIdx.x / (m.nbx * m.nby);
    const int cx = bx * kMeshG + k % kMeshG, cy = by * kMeshG + k / kMeshG;
    c.x = cx * kMeshKx;
    c.y = cy * kMeshKx;
    c.z = bz * kMeshBz;
    c.s0 = c.s1 = 0;
    if (cx < m.ncx && cy < m.ncy) {
        const int col = cy * m.ncx + cx;
        const int* rel = b.rel + (long long)col * (m.nzb + 1);
        c.s0 = b.col[col] + rel[c.z * kMeshZsub];
        c.s1 = b.col[col] + rel[min((c.z + kMeshBz) * kMeshZsub, m.nzb)];
    }
    return c;
}

// Fixed point of the grid charges: weights are at most 1, so a node holds
// fewer than 2^26 of them.
constexpr double kMeshScale = 68719476736.0;    // 2^36

// Spreads the charges of one brick's ions onto its nodes.  A wave takes a
// column's ions 16 at a time, computes their weights on the column's nodes
// (zero outside an ion's ten) and contracts over the ions,
//   node[y][x][z] += sum_ions (w_x w_y) w_z,
// 13 tiles of 16 x 16; a column's sums are added to the brick's in LDS as int64
// (exact, so the order of the waves does not matter).  Adding every weight to
// LDS instead, 1,000 additions an ion, was bound by the LDS's 2 additions per
// clock: 135 us at 2^17 ions, 241 at 2^18 and 630 at 2^20, against 120, 171 and 505.
// Now the waves wait for one another's steps, 1.2 to 1.8 to a SIMD: vector
// issue 0.31, matrix cores 0.22 and LDS 0.08 of the cycles at 2^20.
__global__ __launch_bounds__(kMeshThreads) void mesh_spread_kernel(MeshArgs m, MeshBufs b)
{
    extern __shared__ unsigned long long grid[];
    __shared__ double wt[kMeshThreads / 64][16][3][16];
    const bool skip = mesh_skip(b.cost, m.cost_max);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c16 = lane & 15, q = lane >> 4;
    for (int k = threadIdx.x; k < kMeshNodes; k += kMeshThreads) grid[k] = 0ull;
    if (skip) return;
    __syncthreads();
    const int waves = kMeshThreads / 64;
    for (int k = blockIdx.y * waves + wv; k < kMeshG * kMeshG; k += gridDim.y * waves) {
        const MeshColumn c = mesh_column(m, b, k);
        if (c.s0 >= c.s1) continue;
        mesh4 acc[kMeshReach];
#pragma unroll
        for (int t = 0; t < kMeshReach; ++t) acc[t] = mesh4{0.0, 0.0, 0.0, 0.0};
        for (int k0 = c.s0; k0 < c.s1; k0 += 16) {
            __builtin_amdgcn_wave_barrier();
            for (int e = lane; e < 16 * 48; e += 64) {
                const int ion = e / 48, j = e - ion * 48, axis = j >> 4, node = j & 15;
                const float4 p = b.s[min(k0 + ion, c.s1 - 1)];
                const double v = axis == 0 ? p.x : axis == 1 ? p.y : p.z, lo = axis == 2 ? -m.Hh : -m.R;
                const int cell = mesh_cell(v, lo, m.inv_h, axis == 2 ? m.nc[2] : m.nc[0]);
                const int n = node - (cell - (axis == 0 ? c.x : axis == 1 ? c.y : c.z));
                double dummy;
                const double w = mesh_window<false>(m, (v - lo) * m.inv_h - cell, n, dummy);
                wt[wv][ion][axis][node] = n >= 0 && n < kMeshP && k0 + ion < c.s1 ? w : 0.0;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double (*w)[16] = wt[wv][4 * s + q];
                const double wx = w[0][c16], wz = w[2][c16];
#pragma unroll
                for (int t = 0; t < kMeshReach; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(wx * w[1][t], wz, acc[t], 0, 0, 0);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        unsigned long long* to = grid + (k / kMeshG * kMeshKx) * kMeshLx + k % kMeshG * kMeshKx + c16 * kMeshLx * kMeshLx;
#pragma unroll
        for (int t = 0; t < kMeshReach; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * r + q < kMeshReach)
                    __hip_atomic_fetch_add(&to[t * kMeshLx + 4 * r + q],
                                           (unsigned long long)__double2ll_rn(acc[t][r] * kMeshScale),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    unsigned long long* o = b.brick + ((long long)blockIdx.x * gridDim.y + blockIdx.y) * kMeshNodes;
    for (int k = threadIdx.x; k < kMeshNodes; k += kMeshThreads) o[k] = grid[k];
}

// Grid charges: a node lies in at most two bricks along x and y and three
// along z.
__global__ __launch_bounds__(256) void mesh_sum_kernel(MeshArgs m, MeshBufs b)
{
    const long long v = (long long)blockIdx.x * 256 + threadIdx.x;
    const int nx = m.n[0], ny = m.n[1], nz = m.n[2];
    if (v >= (long long)nx * ny * nz) return;
    const int x = (int)(v % nx), y = (int)(v / nx % ny), z = (int)(v / ((long long)nx * ny));
    constexpr int bc = kMeshG * kMeshKx;
    long long s = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int bz = z / kMeshBz - i, oz = z - bz * kMeshBz;
        if (bz < 0 || bz >= m.nbz || oz >= kMeshLz) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int by = y / bc - j, oy = y - by * bc;
            if (by < 0 || by >= m.nby || oy >= kMeshLx) continue;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int bx = x / bc - k, ox = x - bx * bc;
                if (bx < 0 || bx >= m.nbx || ox >= kMeshLx) continue;
                const unsigned long long* q = b.brick + ((long long)(bz * m.nby + by) * m.nbx + bx) * m.parts * kMeshNodes +
                                              (oz * kMeshLx + oy) * kMeshLx + ox;
                for (int p = 0; p < m.parts; ++p) s += (long long)q[(long long)p * kMeshNodes];
            }
        }
    }
    b.q[v] = (double)s / kMeshScale;
}

// Green's tables, once per system (block m): the one-dimensional kernel g_m
// on the grid whose product with two windows is e^(-t_m^2 x^2).  Its symbol is
// the least-squares one, (sum over the alias images of W^2 G) / (sum of W^2)^2
// with W the window's and G the Gaussian's transform (wave numbers per cell).
constexpr int kMeshNk = 768;

__global__ __launch_bounds__(256) void mesh_green_kernel(MeshArgs m, double i0_beta, double* __restrict__ green)
{
    __shared__ double sym[kMeshNk];
    __shared__ double part[4][64];
    const double th = m.th[blockIdx.x];
    for (int j = threadIdx.x; j < kMeshNk; j += 256) {
        double num = 0.0, den = 0.0;
        for (int a = -2; a <= 2; ++a) {
            const double k = kPi * ((j + 0.5) / kMeshNk + 2.0 * a);
            const double q = kMeshBeta * kMeshBeta - 0.25 * kMeshP * kMeshP * k * k;
            const double r = sqrt(fabs(q));
            const double w = r < 1e-6 ? 1.0 : (q > 0.0 ? sinh(r) : sin(r)) / r;
            const double w2 = w * w * (kMeshP * kMeshP / (i0_beta * i0_beta));
            num += w2 * (sqrt(kPi) / th) * exp(-0.25 * k * k / (th * th));
            den += w2;
        }
        sym[j] = num / (den * den) / kMeshNk;
    }
    __syncthreads();
    const int n = blockIdx.y * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
    double s = 0.0;
    if (n < max(m.n[0], m.n[2]))
        for (int j = q * (kMeshNk / 4); j < (q + 1) * (kMeshNk / 4); ++j)
            s = fma(sym[j], cospi((double)((2 * j + 1) * n % (4 * kMeshNk)) / (2.0 * kMeshNk)), s);
    part[q][threadIdx.x & 63] = s;
    __syncthreads();
    if (q == 0 && n < m.ng)
        green[(long long)blockIdx.x * m.ng + n] = ((part[0][n & 63] + part[1][n & 63]) + part[2][n & 63]) + part[3][n & 63];
}

// One axis of the Gaussian convolutions: a product with the symmetric Toeplitz
// matrix g[|i - k|], 64-bit MFMA.  The matrix is symmetric about its centre
// too, so the sums and differences of a line's mirrored values,
// e_k = v_k + v_(n-1-k) and o_k = v_k - v_(n-1-k), are carried by matrices of
// half the size, g[|i - k|] +- g[n - 1 - i - k], and give the mirrored results
// as (E +- O) / 2: half the products.  A wave computes NT x 16 such rows of 16
// grid lines.  AXIS 0 and 1 apply Gaussian m0 + blockIdx.z; AXIS 2 sums over
// Gaussians m0 .. m0 + mc - 1 with their weights (add: on top of what out
// holds).  144 us for the three axes at 2^17 ions, where whole lines took 233.
// The matrix cores are busy for 0.41 to 0.43 of the cycles at 2^20 ions and 0.18
// to 0.30 at 2^17, vector issue for 0.3: what binds is the way of an operand
// from memory, with the 1 to 2.5 waves a SIMD that the accumulators leave room
// for (operands loaded a step ahead, or products left out, gained nothing).
// v_mfma_f64_16x16x4_f64 operands, lane l: A[l % 16][l / 16],
// B[l / 16][l % 16], D[4 r + l / 16][l % 16].
template <int AXIS, int NT>
__global__ __launch_bounds__(256) void mesh_conv_kernel(MeshArgs m, const double* __restrict__ in,
                                                        double* __restrict__ out,
                                                        const double* __restrict__ green, const long long* cost,
                                                        int m0, int mc, int add)
{
    typedef double d4 __attribute__((ext_vector_type(4)));
    extern __shared__ double tab[];
    const bool skip = mesh_skip(cost, m.cost_max);
    const int nx = m.n[0], ny = m.n[1], nz = m.n[2];
    const int len = AXIS == 0 ? nx : AXIS == 1 ? ny : nz, half = (len + 1) / 2;
    const int lines = AXIS == 0 ? ny * nz : AXIS == 1 ? nx * nz : nx * ny;
    const long long vol = (long long)nx * ny * nz;
    const long long sk = AXIS == 0 ? 1 : AXIS == 1 ? nx : (long long)nx * ny;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int line = (blockIdx.x * 4 + wv) * 16 + (lane & 15);
    const int ln = min(line, lines - 1);
    const long long base = AXIS == 0 ? (long long)ln * nx
                         : AXIS == 1 ? (long long)(ln / nx) * nx * ny + ln % nx : ln;
    const int i0 = blockIdx.y * (16 * NT), kq = lane >> 4;
    d4 even[NT], odd[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) even[t] = odd[t] = d4{0.0, 0.0, 0.0, 0.0};
    const int first = AXIS == 2 ? 0 : blockIdx.z, count = AXIS == 2 ? mc : 1;
    for (int g = first; g < first + count; ++g) {
        const double w = AXIS == 2 ? m.w[m0 + g] : 1.0;
        __syncthreads();
        for (int k = threadIdx.x; k < m.ng; k += 256) tab[k] = 0.5 * w * green[(long long)(m0 + g) * m.ng + k];
        if (skip) return;
        __syncthreads();
        const double* src = in + (AXIS == 0 ? 0 : g * vol) + base;
        for (int k0 = 0; k0 < half; k0 += 16) {
            double e[4], o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 4 * u + kq, mk = len - 1 - k;
                const double v = k < half ? src[k * sk] : 0.0, x = k < mk ? src[mk * sk] : 0.0;
                e[u] = v + x;                   // the centre of an odd line counts once
                o[u] = v - x;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 4 * u + kq;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int i = i0 + 16 * t + (lane & 15);
                    const double a = tab[abs(i - k)], c = tab[abs(len - 1 - i - k)];
                    even[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a + c, e[u], even[t], 0, 0, 0);
                    odd[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a - c, o[u], odd[t], 0, 0, 0);
                }
            }
        }
    }
    if (line >= lines) return;
    double* dst = out + (AXIS == 2 ? 0 : first * vol) + base;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + 16 * t + 4 * r + kq, mi = len - 1 - i;
            if (i >= half) continue;
            const double p = even[t][r] + odd[t][r], q = even[t][r] - odd[t][r];
            dst[i * sk] = p + (AXIS == 2 && add ? dst[i * sk] : 0.0);
            if (mi != i) dst[mi * sk] = q + (AXIS == 2 && add ? dst[mi * sk] : 0.0);
        }
}

// Launches one axis for Gaussians m0 .. m0 + mc - 1.
template <int AXIS>
inline void mesh_conv(const MeshArgs& m, const MeshBufs& b, const double* in, double* out, int m0, int mc, hipStream_t st)
{
    const int len = m.n[AXIS], tiles = ((len + 1) / 2 + 15) / 16;
    const long long lines = (long long)m.n[0] * m.n[1] * m.n[2] / len;
    const unsigned gx = (unsigned)((lines + 63) / 64), gz = AXIS == 2 ? 1 : mc;
    const size_t lds = (size_t)m.ng * 8;
    // several row tiles to a wave share the loaded lines; one where that would leave SIMDs idle
    const int nt = (long long)gx * 4 * gz * ((tiles + 2) / 3) < 4096 ? 1 : tiles % 3 == 0 || tiles > 4 ? 3 : 2;
    const dim3 grid(gx, (tiles + nt - 1) / nt, gz);
    if (nt == 1)
        mesh_conv_kernel<AXIS, 1><<<grid, 256, lds, st>>>(m, in, out, b.green, b.cost, m0, mc, m0 > 0);
    else if (nt == 2)
        mesh_conv_kernel<AXIS, 2><<<grid, 256, lds, st>>>(m, in, out, b.green, b.cost, m0, mc, m0 > 0);
    else
        mesh_conv_kernel<AXIS, 3><<<grid, 256, lds, st>>>(m, in, out, b.green, b.cost, m0, mc, m0 > 0);
}

// Far part of every ion's raw pair sum, minus the gradient of the gridded
// potential: a thread per ion, the brick's nodes in LDS.  The window's
// derivative is taken of the normalised interpolant (sum w phi / sum w), which
// makes a constant potential exactly force free: the mean potential is 1e4
// times what matters here.  Bound by the LDS reads, one per node and ion (87 us
// at 2^17 ions, 465 at 2^20): the LDS is busy for 0.67 of the cycles at 2^20,
// 0.41 of them with bank conflicts, at 1.7 waves a SIMD.  The z weights as 64-bit MFMA products over a
// column's ions, as in the spread, took 155 and 660 us: half of each tile is
// nodes outside an ion's ten.
__global__ __launch_bounds__(kMeshThreads) void mesh_gather_kernel(MeshArgs m, MeshBufs b)
{
    extern __shared__ double node[];
    __shared__ int start[kMeshG * kMeshG], pre[kMeshG * kMeshG + 1];
    const bool skip = mesh_skip(b.cost, m.cost_max);
    const int x0 = blockIdx.x % m.nbx * kMeshG * kMeshKx, y0 = blockIdx.x / m.nbx % m.nby * kMeshG * kMeshKx,
              z0 = blockIdx.x / (m.nbx * m.nby) * kMeshBz;
    if (threadIdx.x < kMeshG * kMeshG) {
        const MeshColumn c = mesh_column(m, b, threadIdx.x);
        start[threadIdx.x] = c.s0;
        pre[threadIdx.x + 1] = c.s1 - c.s0;
    }
    if (threadIdx.x == 0) pre[0] = 0;
    if (skip) return;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int c = 0; c < kMeshG * kMeshG; ++c) pre[c + 1] += pre[c];
    for (int k = threadIdx.x; k < kMeshNodes; k += kMeshThreads) {
        const int x = x0 + k % kMeshLx, y = y0 + k / kMeshLx % kMeshLx, z = z0 + k / (kMeshLx * kMeshLx);
        node[k] = x < m.n[0] && y < m.n[1] && z < m.n[2] ? b.phi[((long long)z * m.n[1] + y) * m.n[0] + x] : 0.0;
    }
    __syncthreads();
    const int group = (threadIdx.x >> 6) * gridDim.y + blockIdx.y;
    for (int k = group * 64 + (threadIdx.x & 63); k < pre[kMeshG * kMeshG]; k += gridDim.y * kMeshThreads) {
        int c = 0;
        while (pre[c + 1] <= k) ++c;
        const int t = start[c] + (k - pre[c]);
        const float4 p = b.s[t];
        const double px = p.x, py = p.y, pz = p.z;
        const int cx = mesh_cell(px, -m.R, m.inv_h, m.nc[0]), cy = mesh_cell(py, -m.R, m.inv_h, m.nc[1]),
                  cz = mesh_cell(pz, -m.Hh, m.inv_h, m.nc[2]);
        const double ux = (px + m.R) * m.inv_h - cx, uy = (py + m.R) * m.inv_h - cy,
                     uz = (pz + m.Hh) * m.inv_h - cz;
        double wx[kMeshP], dx[kMeshP], wy[kMeshP], dy[kMeshP];
        double sx = 0.0, tx = 0.0, sy = 0.0, ty = 0.0;
#pragma unroll
        for (int j = 0; j < kMeshP; ++j) {
            wx[j] = mesh_window<true>(m, ux, j, dx[j]);
            wy[j] = mesh_window<true>(m, uy, j, dy[j]);
            sx += wx[j]; tx += dx[j];
            sy += wy[j]; ty += dy[j];
        }
        const double qx = tx / sx, qy = ty / sy;
#pragma unroll
        for (int j = 0; j < kMeshP; ++j) {
            dx[j] = fma(-qx, wx[j], dx[j]);
            dy[j] = fma(-qy, wy[j], dy[j]);
        }
        const int base = ((cz - z0) * kMeshLx + (cy - y0)) * kMeshLx + (cx - x0);
        double fx = 0.0, fy = 0.0, fz = 0.0, pw = 0.0, sz = 0.0, tz = 0.0;
#pragma unroll 1
        for (int jz = 0; jz < kMeshP; ++jz) {
            double dz;
            const double wz = mesh_window<true>(m, uz, jz, dz);
            int at = base + jz * (kMeshLx * kMeshLx);
            double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
            for (int jy = 0; jy < kMeshP; ++jy) {
                double r0 = 0.0, r1 = 0.0;
#pragma unroll
                for (int jx = 0; jx < kMeshP; ++jx) {
                    const double v = node[at + jx];
                    r0 = fma(v, dx[jx], r0);
                    r1 = fma(v, wx[jx], r1);
                }
                a0 = fma(r0, wy[jy], a0);
                a1 = fma(r1, dy[jy], a1);
                a2 = fma(r1, wy[jy], a2);
                at += kMeshLx;
            }
            fx = fma(a0, wz, fx);
            fy = fma(a1, wz, fy);
            fz = fma(a2, dz, fz);
            pw = fma(a2, wz, pw);
            sz += wz;
            tz += dz;
        }
        fz = fma(-tz / sz, pw, fz);
        b.far[t] = -fx * m.inv_h;
        b.far[m.cap + t] = -fy * m.inv_h;
        b.far[2 * (long long)m.cap + t] = -fz * m.inv_h;
    }
}

// Near part of the pair term at squared distance r2: (1 + r) e^-r / r^3 - f_L.
// Beyond r_c it is evaluated at r_c, where it vanishes.
__device__ __forceinline__ float mesh_near_f(const MeshArgs& m, float near0, float r2)
{
    const float y = __builtin_amdgcn_fmed3f(r2, 0.0f, m.rc2);
    const float ri = __builtin_amdgcn_rsqf(y);
    const float s = fmaf(y, m.irc2, 1.0f);
    float p = m.near[kMeshNearDeg];
#pragma unroll
    for (int d = kMeshNearDeg - 1; d > 0; --d) p = fmaf(p, s, m.near[d]);
    p = fmaf(p, s, near0);
    const float ri2 = ri * ri;
    const float e = __builtin_amdgcn_exp2f((y * ri) * -1.4426950408889634f);
    return fmaf(fmaf(ri2, ri, ri2), e, -p);
}

// Constant term of the near polynomial that makes mesh_near_f vanish at r_c as
// the hardware rounds it (once per system): every pair beyond r_c within a
// box contributes that value, so what is left of it adds up.
__global__ void mesh_zero_kernel(MeshArgs m, float* near0)
{
    float c = m.near[0];
    for (int k = 0; k < 4; ++k) c += mesh_near_f(m, c, m.rc2);
    if (threadIdx.x == 0) *near0 = c;
}

// Near pairs.  A block of S waves takes 64 sorted ions, as four groups of 16
// with a box each; quarter q of every wave holds group q's targets.
//
// Search: the waves share the columns within r_c of the groups' boxes and list
// in LDS, per group, the boxes of 8 ions within r_c of the group's.  Then the
// waves take the listed boxes of each group two at a time: the quarter's lanes
// load the 16 sources (the next ones while the present are worked on), pass
// them through LDS and read them back one by one, the same for the quarter.
// FP32 terms, FP64 sums of every 16.
//
// Bound by FP32 issue (31 slots a pair; 0.93 of the cycles at 2^20 ions, 0.79
// at 2^17), so what counts is how few pairs
// beyond r_c are evaluated: 3.3 times the pairs within r_c with groups of 16
// and boxes of 8, 5.8 with 64 and 16 and wider columns, whose sources could be
// scalar loads: at 2^20 ions 2.9 ms with r_c = 0.39, where the wider search
// took 3.7 ms with 0.33; 1.86 ms with the present r_c of 0.29.
constexpr int kMeshList = 64;       // boxes a wave lists per group in a round
constexpr int kMeshCand = 64;       // candidate columns per group of a round

template <int S>
__global__ __launch_bounds__(64 * S) __attribute__((amdgpu_waves_per_eu(6, 8)))
void mesh_near_kernel(MeshArgs m, const float4* __restrict__ pos, const float* __restrict__ box,
                      const int* __restrict__ rel_, const int* __restrict__ col, const int* __restrict__ idx,
                      const double* __restrict__ far, const float* __restrict__ near0_, const long long* cost,
                      unsigned long long* __restrict__ fix, long long fstride, double scale, int* status)
{
    __shared__ int seg[S][4][kMeshList];            // boxes listed by each wave
    __shared__ int list[4][S * kMeshList];          // the same, one after the other
    __shared__ int listed[4][S];
    __shared__ int full[S];
    __shared__ int2 cand[4][kMeshCand];
    __shared__ float4 src[S][64];
    __shared__ double part[S][3][64];
    const bool skip = mesh_skip(cost, m.cost_max);
    const int total = col[m.ncx * m.ncy];
    // consecutive tiles share sources: give each of the 8 XCDs a run of them
    const int tiles = (total + 63) / 64, per = (tiles + 7) / 8;
    const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (skip | ((int)(blockIdx.x >> 3) >= per) | (tile >= tiles)) return;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, l16 = lane & 15;
    const int slot = tile * 64 + lane;
    const bool here = slot < total;                 // the same for a group
    const float4 me = pos[here ? slot : 0];
    const int ns = m.cap / kMeshSub;
    float lo[3], hi[3];                             // the group's box
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float2 l = *(const float2*)&box[(long long)c * ns + (tile * 4 + q) * 2];
        const float2 h = *(const float2*)&box[(long long)(c + 3) * ns + (tile * 4 + q) * 2];
        lo[c] = here ? fminf(l.x, l.y) : 1.0e30f;
        hi[c] = here ? fmaxf(h.x, h.y) : -1.0e30f;
    }
    const float R = (float)m.R, icw = 1.0f / m.cw, slack = 1.0e-4f * m.rc, near0 = near0_[0];
    double sx = 0.0, sy = 0.0, sz = 0.0;

    // where the search goes on: candidate columns from c0, candidate t0, its box o0 (t0, o0 per
    // group and wave)
    int c0 = 0, t0 = 0, o0 = 0;
    bool fresh = true;
    for (;;) {
        if (fresh) {
            // candidate columns of each group: slots within r_c along z, as runs of boxes.
            // Thread t works for group t % 4, whose box it needs
            __syncthreads();
            const int g = threadIdx.x & 3;
            float glo[3], ghi[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                glo[c] = __shfl(lo[c], g * 16, 64);
                ghi[c] = __shfl(hi[c], g * 16, 64);
            }
            auto column = [&](float v, int nc) { return (int)fminf(fmaxf(floorf((v + R) * icw), 0.0f), (float)(nc - 1)); };
            const int x0 = column(glo[0] - m.rc, m.ncx), x1 = column(ghi[0] + m.rc, m.ncx);
            const int y0 = column(glo[1] - m.rc, m.ncy), y1 = column(ghi[1] + m.rc, m.ncy);
            const int nx = x1 - x0 + 1, all = nx > 0 && y1 >= y0 && glo[2] <= ghi[2] ? nx * (y1 - y0 + 1) : 0;
            for (int t = threadIdx.x >> 2; t < kMeshCand; t += 16 * S) {
                int2 e = make_int2(0, 0);
                if (c0 + t < all) {
                    const int cx = x0 + (c0 + t) % nx, cy = y0 + (c0 + t) / nx;
                    // the outer columns also hold ions that sit on the boundary to rounding
                    const float gx = fmaxf(0.0f, fmaxf(cx * m.cw - R - ghi[0], glo[0] - ((cx + 1) * m.cw - R)) - slack);
                    const float gy = fmaxf(0.0f, fmaxf(cy * m.cw - R - ghi[1], glo[1] - ((cy + 1) * m.cw - R)) - slack);
                    const float left = m.rc2 - gx * gx - gy * gy;
                    if (left > 0.0f) {
                        const float dz = sqrtf(left) + slack;
                        const int c = cy * m.ncx + cx;
                        const int* rel = rel_ + (long long)c * (m.nzb + 1);
                        const int s0 = rel[mesh_zbin(glo[2] - dz, m)], s1 = rel[mesh_zbin(ghi[2] + dz, m) + 1];
                        if (s1 > s0) {
                            const int first = (col[c] + s0) / kMeshSub;
                            e = make_int2(first, (col[c] + s1 + kMeshSub - 1) / kMeshSub - first);
                        }
                    }
                }
                cand[g][t] = e;
            }
            __syncthreads();
            t0 = wv;
            o0 = 0;
        }
        // this wave's candidates of each group, 16 boxes at a time
        int n = 0;
        bool stop = false;
        while (__any(t0 < kMeshCand && !stop)) {
            bool keep = false;
            int sub = 0;
            const bool on = t0 < kMeshCand && !stop;
            int2 e = make_int2(0, 0);
            if (on) {
                e = cand[q][t0];
                sub = e.x + o0 + l16;
                if (o0 + l16 < e.y) {
                    const float gx = fmaxf(0.0f, fmaxf(box[sub] - hi[0], lo[0] - box[3ll * ns + sub]));
                    const float gy = fmaxf(0.0f, fmaxf(box[ns + sub] - hi[1], lo[1] - box[4ll * ns + sub]));
                    const float gz = fmaxf(0.0f, fmaxf(box[2ll * ns + sub] - hi[2], lo[2] - box[5ll * ns + sub]));
                    keep = gx * gx + gy * gy + gz * gz < m.rc2;
                }
            }
            const unsigned mask = (unsigned)(__ballot(keep) >> (q * 16)) & 0xffffu;
            const int k = __popc(mask);
            if (on) {
                if (n + k > kMeshList) {
                    stop = true;                    // the list is full: go on here in the next round
                } else {
                    if (keep) seg[wv][q][n + __popc(mask & ((1u << l16) - 1u))] = sub;
                    n += k;
                    o0 += 16;
                    if (o0 >= e.y) {
                        t0 += S;
                        o0 = 0;
                    }
                }
            }
        }
        if (l16 == 0) listed[q][wv] = n;
        const bool again = __any(stop);
        if (lane == 0) full[wv] = again;
        __syncthreads();
        // one list per group
        int before = 0, count = 0, unfinished = 0;
#pragma unroll
        for (int w = 0; w < S; ++w) {
            const int k = listed[q][w];
            before += w < wv ? k : 0;
            count += k;
            unfinished |= full[w];
        }
        for (int k = l16; k < n; k += 16) list[q][before + k] = seg[wv][q][k];
        __syncthreads();
        // two boxes at a time; the last of an odd number is paired with a point beyond r_c
        const float far_point = (float)m.R + 2.0f;
        auto load = [&](int k) {
            const int e = 2 * k + (l16 >> 3);
            float4 p = make_float4(far_point, far_point, far_point, 0.0f);
            int from = -1;
            if (e < count) {
                from = list[q][e] * kMeshSub + (l16 & 7);
                p = pos[from];
            }
            p.w = __builtin_bit_cast(float, from);
            return p;
        };
        const int batches = (count + 1) / 2;
        float4 next = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (wv < batches) next = load(wv);
        for (int k = wv; k < batches; k += S) {
            src[wv][lane] = next;
            const bool own = __any(__builtin_bit_cast(int, next.w) >> 4 == slot >> 4);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (k + S < batches) next = load(k + S);
            float ax = 0.0f, ay = 0.0f, az = 0.0f;
            if (own) {
#pragma unroll 4
                for (int u = 0; u < 16; ++u) {
                    const float4 p = src[wv][q * 16 + u];
                    const float dx = me.x - p.x, dy = me.y - p.y, dz = me.z - p.z;
                    float f = mesh_near_f(m, near0, fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
                    f = __builtin_bit_cast(int, p.w) == slot ? 0.0f : f;
                    ax = fmaf(f, dx, ax);
                    ay = fmaf(f, dy, ay);
                    az = fmaf(f, dz, az);
                }
            } else {
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const float4 p = src[wv][q * 16 + u];
                    const float dx = me.x - p.x, dy = me.y - p.y, dz = me.z - p.z;
                    const float f = mesh_near_f(m, near0, fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
                    ax = fmaf(f, dx, ax);
                    ay = fmaf(f, dy, ay);
                    az = fmaf(f, dz, az);
                    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            sx += (double)ax;
            sy += (double)ay;
            sz += (double)az;
        }
        fresh = !unfinished;
        if (fresh) {
            c0 += kMeshCand;
            // further candidate columns of any group?
            bool more = false;
            const float w = 2.0f * m.rc;
            if (lo[2] <= hi[2])
                more = (floorf((hi[0] - lo[0] + w) * icw) + 2.0f) * (floorf((hi[1] - lo[1] + w) * icw) + 2.0f) > (float)c0;
            if (!__any(more)) break;
        }
        __syncthreads();
    }
    part[wv][0][lane] = sx;
    part[wv][1][lane] = sy;
    part[wv][2][lane] = sz;
    __syncthreads();
    if (wv != 0 || !here) return;
    const int i = idx[slot];
    if (i < 0) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double t = part[0][c][lane];
#pragma unroll
        for (int w = 1; w < S; ++w) t += part[w][c][lane];
        fix[c * fstride + i] = to_fixed(t + far[(long long)c * m.cap + slot], scale, status);
    }
}

// Direct sums of the systems whose step calls for it, as pair_sym_kernel has
// them (the same items, so the same totals).  A launch of one round of blocks
// that take the items in turn.  For the choice, this launch and the asks of the
// others, a step pays 4 to 7 us (313 -> 320 us at 40,960 ions, 424 -> 428 at
// 2^16, 620 -> 624 at 2^17).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(kSymWaves, 8)))
void mesh_direct_kernel(const MeshDirect* __restrict__ table, int systems, long long plane)
{
    __shared__ float4 src[4][128];
    __shared__ float jpart[4][3][BLOCK];
    for (int k = 0; k < systems; ++k) {
        if (!mesh_skip(table[k].cost, table[k].cost_max)) continue;
        const MeshDirect d = table[k];
        SymPlace at{0, 0};
        SymItem it;
        for (int n = blockIdx.x; sym_item_at(d.runs, n, at, it); n += gridDim.x)
            sym_dispatch<BLOCK>(d.x, d.x + plane, d.x + 2 * plane, d.N, it.rows, it.I, it.J0, it.J1, 0, 4, d.fix,
                                plane, d.scale, d.status, src, jpart, PlainPair{});
    }
}

inline hipError_t mesh_direct_launch(const MeshDirect* table, int systems, long long plane, int cus, hipStream_t st)
{
    mesh_direct_kernel<256><<<cus * kSymWaves, 256, 0, st>>>(table, systems, plane);
    return hipGetLastError();
}

// Convolution scratch: with 120, 200, 400 and 1,200 MB (fewer passes over the
// 14 Gaussians) a pair sum took 1.15, 1.13, 1.11 and 1.11 ms at 2^18 ions, 5.18,
// 4.40, 4.26 and 4.27 at 2^20.
constexpr int kMeshScratchMb = 400;

// Cuts buffers from an arena at `base` (null: only adds up their size).
struct MeshArena {
    char* base;
    size_t at = 0;
    template <typename T>
    void take(T** p, size_t bytes)
    {
        *p = (T*)(base ? base + at : nullptr);
        at += (bytes + 255) / 256 * 256;
    }
};

inline size_t mesh_own(const MeshArgs& m, char* base, MeshBufs& b)
{
    MeshArena a{base};
    a.take(&b.count, (size_t)m.ncx * m.ncy * m.nzb * 4);
    a.take(&b.green, (size_t)m.M * m.ng * 8);
    a.take(&b.near0, 4);
    a.take(&b.cost, 3 * sizeof(long long));
    a.take(&b.direct, sizeof(MeshDirect));
    return a.at;
}

inline size_t mesh_scratch(const MeshArgs& m, char* base, MeshBufs& b)
{
    MeshArena a{base};
    const size_t ncol = (size_t)m.ncx * m.ncy, cap = (size_t)m.cap, v = (size_t)m.n[0] * m.n[1] * m.n[2];
    a.take(&b.key, (size_t)m.N * 4);
    a.take(&b.arr, (size_t)m.N * 4);
    a.take(&b.rel, ncol * (m.nzb + 1) * 4);
    a.take(&b.col, (ncol + 1) * 4);
    a.take(&b.temp, cap * 4);
    a.take(&b.idx, cap * 4);
    a.take(&b.s, cap * 16);
    a.take(&b.box, 6 * (cap / kMeshSub) * 4);
    a.take(&b.far, 3 * cap * 8);
    a.take(&b.q, v * 8);
    a.take(&b.phi, v * 8);
    // convolution scratch: as many Gaussians at a time as fit
    b.mc = (int)std::min<size_t>(m.M, std::max<size_t>(1, ((size_t)kMeshScratchMb << 20) / (16 * v)));
    const int passes = (m.M + b.mc - 1) / b.mc;
    b.mc = (m.M + passes - 1) / passes;
    const size_t conv = 2 * (size_t)b.mc * v * 8, brick = (size_t)m.nbx * m.nby * m.nbz * m.parts * kMeshNodes * 8;
    a.take(&b.t1, std::max(conv, brick));
    b.t2 = b.t1 ? b.t1 + (size_t)b.mc * v : nullptr;
    b.brick = (unsigned long long*)b.t1;
    return a.at;
}

// Clears the bin counts and marks and computes the Green's tables (once per system).
inline hipError_t mesh_start(const MeshArgs& m, const MeshBufs& b, hipStream_t st)
{
    constexpr int lds = kMeshNodes * 8;
    hipError_t e = hipFuncSetAttribute((const void*)mesh_spread_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)mesh_gather_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess) e = hipMemsetAsync(b.count, 0, (size_t)m.ncx * m.ncy * m.nzb * 4, st);
    if (e == hipSuccess) e = hipMemsetAsync(b.cost, 0, 3 * sizeof(long long), st);
    if (e != hipSuccess) return e;
    mesh_zero_kernel<<<1, 64, 0, st>>>(m, b.near0);
    mesh_green_kernel<<<dim3(m.M, (m.ng + 63) / 64), 256, 0, st>>>(m, mesh_i0(kMeshBeta), b.green);
    return hipGetLastError();
}

// The pair sum of one step: positions x (planes `plane` apart) to the
// fixed-point totals fix (planes `fstride` apart).
inline hipError_t mesh_launch(const MeshArgs& m, const MeshBufs& b, const float* x, long long plane,
                              unsigned long long* fix, long long fstride, double scale, int* status, hipStream_t st)
{
    const int gi = (m.N + 255) / 256, gc = (m.cap + 255) / 256, ncol = m.ncx * m.ncy;
    const long long v = (long long)m.n[0] * m.n[1] * m.n[2];
    mesh_bin_kernel<<<gc, 256, 0, st>>>(x, plane, m, b);
    mesh_scan_kernel<<<ncol, 256, 0, st>>>(m, b);
    mesh_cols_kernel<<<1 + std::min(1024, (ncol * ((m.nzb + kMeshSlab - 1) / kMeshSlab) + 63) / 64), 1024, 0, st>>>(m, b);
    mesh_place_kernel<<<gi, 256, 0, st>>>(m, b);
    mesh_order_kernel<<<gc, 256, 0, st>>>(x, plane, m, b);
    mesh_box_kernel<<<gc, 256, 0, st>>>(m, b);
    const int bricks = m.nbx * m.nby * m.nbz;
    constexpr size_t lds = kMeshNodes * 8;
    mesh_spread_kernel<<<dim3(bricks, m.parts), kMeshThreads, lds, st>>>(m, b);
    mesh_sum_kernel<<<(unsigned)((v + 255) / 256), 256, 0, st>>>(m, b);
    for (int m0 = 0; m0 < m.M; m0 += b.mc) {
        const int mc = std::min(b.mc, m.M - m0);
        mesh_conv<0>(m, b, b.q, b.t1, m0, mc, st);
        mesh_conv<1>(m, b, b.t1, b.t2, m0, mc, st);
        mesh_conv<2>(m, b, b.t2, b.phi, m0, mc, st);
    }
    mesh_gather_kernel<<<dim3(bricks, m.gparts), kMeshThreads, lds, st>>>(m, b);
    const int tiles = (m.cap / 64 + 7) / 8 * 8;
    if (m.cap / 64 >= 8192)
        mesh_near_kernel<4><<<tiles, 256, 0, st>>>(m, b.s, b.box, b.rel, b.col, b.idx, b.far, b.near0, b.cost, fix,
                                                   fstride, scale, status);
    else
        mesh_near_kernel<8><<<tiles, 512, 0, st>>>(m, b.s, b.box, b.rel, b.col, b.idx, b.far, b.near0, b.cost, fix,
                                                   fstride, scale, status);
    return hipGetLastError();
}

}  // namespace odk
