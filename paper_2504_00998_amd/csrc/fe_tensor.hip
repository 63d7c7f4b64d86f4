// The step kernel in tensor-product form (FP64): Y = alpha (H~ - c) X - beta Ym1
// in one launch, without cell colours.
//
// On the structured box the assembled 1/2 M^-1/2 K M^-1/2 is a sum of three
// products of one-dimensional operators, K (x) M (x) M + M (x) K (x) M +
// M (x) M (x) K, because the cell matrix is one (Sec. 2.3: tensor-product
// Lagrange basis on GLL nodes) and M^-1/2 is a product of per-axis factors.
// Applied axis by axis it takes about 7 (p + 2) multiply-adds per value
// instead of the dense cell product's (p + 1)^6 / p^3 (42 against 244 at
// p = 4, 56 against 545 at p = 6), which leaves the step bound by HBM.
//
// A workgroup owns a column of tiles: BX x BY cells in the x-y plane (their
// low-face-closed nodes), 16 vectors, a range of cell layers along z.  It
// walks the z planes of nodes upwards.  Per plane:
//  - x stage: a lane holds two vectors of XC cells of one x row of the plane
//    (and of the cell before them, as a vertex node takes both cells it belongs
//    to), loaded from global memory two planes ahead, and forms M_x u, K_x u
//    and the diagonal terms (v - c) u for its output nodes into LDS;
//  - y stage: a lane holds one vector and x position of a cell's p rows, reads
//    the two from LDS along y and forms A = M_y M_x u and
//    B = (K_y M_x + M_y K_x) u;
//  - z stage: A and B are added into the p + 1 output planes of the cell
//    layer, kept in registers, times the entries of K_z and M_z; the plane's
//    own diagonal and previous-iterate terms join them, and after the last
//    plane of a layer its p planes are stored.
// The x stage and the y-z stages run in waves of their own, a plane apart:
// the x waves write plane g + 1 into one of two LDS buffers while the y-z
// waves take plane g from the other, with one barrier per plane.  Each kind
// then holds only its own registers (the x waves two planes of X rows in
// flight, the y-z waves the output planes); with all stages in every wave and
// two barriers per plane, the p = 4 slab below took 3.81 ms a step.
// Every output is summed by one lane in one order: no atomics, no partial
// sums in memory, the same bits on every run, and independent of the vectors
// beside it.  Each value of X, the previous iterate and Y moves once, but for
// the X rows of the halo (a cell before and a node after the tile along x
// and y), which the neighbouring workgroups of the same XCD read at about the
// same time (12.07 GB counted per step of the p = 4 slab, 10.81 without a halo).
//
// What bounds it up to p = 4 is memory: with all arithmetic taken out the p = 4
// slab's step was 4 % faster, without the X rows 37 %.  X comes in 16-byte requests
// because a request of any width costs the address unit about the same (with
// 8-byte ones it was busy 79 % of the time).  Above p = 4 the registers leave
// room for few waves and the latency of a plane's stages shows (p = 6: the waves
// wait 51 % of their cycles, the address units are busy 32 % of the time, no LDS
// conflicts, 6.05 GB counted per step for 5.41 at 3.9 TB/s).  On rows that share
// 128-byte lines the halo rows come from HBM again (p = 5, 200 vectors: a
// product reads 7.2 GB for a block of 3.2).
//
// Measured, ms per recurrence step (two blocks read, one written), against the
// kernels it replaces as the FP64 default: p = 4, 24x24x48 cells, 256 vectors
// 2.48 (the table kernel 4.73) = 4.4 TB/s of the 24 bytes per value, of 5.9 that
// two reads and a write stream at; p = 6, 16x16x32 cells, 128 vectors 1.57
// (5.53); p = 5, 20x20x40 cells, 200 vectors 3.16 (8.79); p = 3, 24x24x48 cells,
// 100 vectors 0.50 (1.45); p = 2, 30x30x60 cells, 100 vectors 0.29 (1.09); the
// Bloch mode on the p = 4 slab with 128 complex vectors 2.55 (7.4, the table kernel
// with dense k.G products).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "fe_internal.h"

namespace fe {

namespace {

// Entries of the one-dimensional cell matrices that differ: K and M are
// symmetric and equal to themselves with both indices reversed.
constexpr int sym_key(int p, int i, int j) {
    int best = i * 16 + j;
    const int a[3] = {j * 16 + i, (p - i) * 16 + p - j, (p - j) * 16 + p - i};
    for (int q = 0; q < 3; ++q) best = a[q] < best ? a[q] : best;
    return best;
}
constexpr int sym_id(int p, int i, int j) {
    const int key = sym_key(p, i, j);
    int n = 0;
    for (int a = 0; a <= p; ++a)
        for (int b = 0; b <= p; ++b)
            if (sym_key(p, a, b) == a * 16 + b) {
                if (a * 16 + b == key) return n;
                ++n;
            }
    return -1;
}
constexpr int sym_count(int p) {
    int n = 0;
    for (int a = 0; a <= p; ++a)
        for (int b = 0; b <= p; ++b) n += sym_key(p, a, b) == a * 16 + b;
    return n;
}

// Off-diagonal entries of the one-dimensional advection matrix above the
// diagonal that differ: it is antisymmetric, and equal to itself reflected in
// the other diagonal.  (Its diagonal is zero but for the ends, which cancel
// between the two cells of a vertex.)
constexpr int anti_key(int p, int i, int j) {
    const int a = i * 16 + j, b = (p - j) * 16 + p - i;
    return a < b ? a : b;
}
constexpr int anti_id(int p, int i, int j) {
    const int key = anti_key(p, i, j);
    int n = 0;
    for (int a = 0; a <= p; ++a)
        for (int b = a + 1; b <= p; ++b)
            if (anti_key(p, a, b) == a * 16 + b) {
                if (a * 16 + b == key) return n;
                ++n;
            }
    return -1;
}
constexpr int anti_count(int p) {
    int n = 0;
    for (int a = 0; a <= p; ++a)
        for (int b = a + 1; b <= p; ++b) n += anti_key(p, a, b) == a * 16 + b;
    return n;
}

}  // namespace

struct TensorAxis {
    int K;     // ncell * p: the period, or the last node of a Dirichlet axis
    int nfree;
    int per;   // -1: periodic, 0: Dirichlet, 1 (single vectors only): zero-Neumann
    int ncell;
};

template <int P, bool CPX> struct TensorParams {
    const double *X, *Ym1, *v;
    double *Y;
    int64_t px, py, pm, pv;           // plane strides in bytes
    uint32_t rx, ry, rm, rv;          // plane byte ranges (0: absent)
    uint32_t ldx, ldy, ldm;           // row strides in bytes
    double alpha, nba, shift;         // nba = -beta / alpha
    int N, ntx, nty, nzc, layers, items, per_xcd;
    int gw;                           // column groups side by side in the order of the items
    TensorAxis ax[3];
    double M[sym_count(P)], K[sym_count(P)], M2, K2;  // M2, K2: the vertex entries of two cells
    double GX[CPX ? anti_count(P) : 1], GY[CPX ? anti_count(P) : 1];  // k_x, k_y times the advection matrix
};

namespace {

constexpr uint32_t kAbsent = 0x80000000u;  // a byte offset past every plane: reads zeros, stores nothing
constexpr int kRawBuffer = 0x00020000;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef double Pair __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return __builtin_bit_cast(double, w);
}
__device__ __forceinline__ Pair buf_load2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    return __builtin_bit_cast(Pair, w);
}
__device__ __forceinline__ void buf_store(double x, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, voff, soff, 0);
}

// Free index of node g of an axis, or -1 where it is a Dirichlet node or
// lies outside the mesh (masks instead of branches: a branch in the walk over
// the planes would let the compiler defer the planes' sums past it).
__device__ __forceinline__ int free_node(const TensorAxis &a, int g) {
    const int lo = g + (a.K & (g >> 31)), w = lo - (a.K & ~((lo - a.K) >> 31));
    const int per = w | ~((w - a.K) >> 31);             // -1 from K on
    const int f = g - 1, dir = f | ~((f - (a.K - 1)) >> 31);  // -1 from node K on, and at node 0
    return ((per & a.per) | (dir & ~a.per)) | ((g + a.K) >> 31);
}

// The rows of plane f of a block (none for f < 0) as a buffer.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_of(const void *base, int64_t stride, uint32_t range, int f) {
    const int some = ~(f >> 31);
    return __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)base + (int64_t)(f & some) * stride), (short)0,
                                             (int)(range & (uint32_t)some), kRawBuffer);
}

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS as byte addresses, so that every access is one address register of its
// plane plus an immediate offset: left to index an array, the compiler keeps
// the address of every row past the immediate range in a register of its own.
typedef __attribute__((address_space(3))) double LdsDouble;
typedef __attribute__((address_space(3))) Pair LdsPair;
__device__ __forceinline__ LdsDouble *lds_at(uint32_t bytes) {
    asm volatile("" : "+v"(bytes));
    return (LdsDouble *)(uintptr_t)bytes;
}

// The value of the lane beside this one in its pair (the other half of a
// complex vector).
__device__ __forceinline__ double neighbour(double x) {
    const u32x2 w = __builtin_bit_cast(u32x2, x);
    u32x2 o;
    o.x = (uint32_t)__builtin_amdgcn_mov_dpp((int)w.x, 0xB1, 0xF, 0xF, true);
    o.y = (uint32_t)__builtin_amdgcn_mov_dpp((int)w.y, 0xB1, 0xF, 0xF, true);
    return __builtin_bit_cast(double, o);
}

// A sum that is formed by here (the compiler may not defer it).
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// A uniform value that the compiler forms again where it is used, rather than
// hold every multiple of it in registers for the whole walk.
template <class T> __device__ __forceinline__ void opaque(T &x) { asm volatile("" : "+s"(x)); }

// The compiler's scheduler does not move instructions across (it would
// raise the registers alive at once past the budget).
__device__ __forceinline__ void stage_end() { __builtin_amdgcn_sched_barrier(0); }

template <int I, int E, class F> __device__ __forceinline__ void unroll(F &&f) {
    if constexpr (I < E) {
        f(std::integral_constant<int, I>{});
        unroll<I + 1, E>(f);
    }
}

}  // namespace

template <int P, int BX, int BY, int XC> struct TensorShape {
    static constexpr int NV = 16;
    static constexpr int WX = BX * P, RY = (BY + 1) * P + 1;
    static constexpr int CW = (WX * BY * NV + 63) / 64;          // y-z waves: a lane one vector
    static constexpr int XI = RY * (BX / XC);                    // x items (row, XC cells): a lane two vectors
    static constexpr int XW = (XI + 7) / 8;                      // x waves
    static constexpr int T = 64 * (CW + XW);
    static constexpr int RS = WX * NV;                           // row stride
    static constexpr int BUF = 2 * RY * RS + BY * P * RS;        // M_x u, K_x u and (v - c) u of one plane
    static constexpr int VN = (XC * P + 7) / 8;                  // v requests of a lane
    static constexpr int VI = 8 * VN;                            // v of one item, in LDS
    static constexpr int LDS = 2 * BUF + XW * 8 * VI;
    static_assert(BX % XC == 0, "whole items in a tile's row");
    static_assert(T <= 1024, "threads of a workgroup");
    static_assert(LDS * 8 <= 160 * 1024, "LDS of a workgroup");
};

// CPX: the Bloch-k mode, columns complex vectors as interleaved (re, im)
// pairs.  The operator gains -i (k_x G (x) M (x) M + k_y M (x) G (x) M), and
// -i g (x_r + i x_i) = g x_i - i g x_r: in the x stage, whose lanes hold pairs,
// G_x u of the other half joins K_x u; in the y stage G_y M_x u of a lane's own
// column goes to its neighbour.
template <int P, int BX, int BY, int XC, int OCC, bool CPX>
__global__ __launch_bounds__((TensorShape<P, BX, BY, XC>::T)) __attribute__((amdgpu_waves_per_eu(OCC)))
void tensor_step_kernel(TensorParams<P, CPX> k) {
    typedef TensorShape<P, BX, BY, XC> S;
    constexpr int NV = S::NV, WX = S::WX, RY = S::RY, RS = S::RS, NX = (XC + 1) * P + 1;
    __shared__ __align__(16) double lds[S::LDS];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsDouble *)lds;

    // workgroups go round the eight XCDs; each XCD takes a contiguous eighth of
    // the items, neighbouring tiles of one column group next to each other, so
    // that its L2 serves the halo rows that they share
    const int item = (int)(blockIdx.x & 7) * k.per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= k.per_xcd || item >= k.items) return;  // whole workgroup
    int rest = item;
    const int gl = rest % k.gw;
    rest /= k.gw;
    const int tx = rest % k.ntx;
    rest /= k.ntx;
    const int ty = rest % k.nty;
    rest /= k.nty;
    const int zc = rest % k.nzc, grp = rest / k.nzc * k.gw + gl;
    if (grp * NV >= k.N) return;  // whole workgroup: past the last group
    const int cx0 = tx * BX, cy0 = ty * BY, cz0 = zc * k.layers, cz1 = min(cz0 + k.layers, k.ax[2].ncell);
    // the planes walked: from the layer before the first (its planes reach the
    // first vertex plane) to the vertex plane that closes the last; a first
    // layer on a Dirichlet face has none before it
    const int l0 = k.ax[2].per || cz0 > 0 ? cz0 - 1 : cz0;
    const int g0 = l0 * P, g1 = cz1 * P;

    const int tid = threadIdx.x, vec = tid % NV, col = grp * NV + vec;
    const bool live = col < k.N;
    const uint32_t cb = (uint32_t)col * 8u;
    // the entries of the one-dimensional matrices, in scalar registers for the
    // walk up to p = 4 (3 for complex vectors); above they do not fit beside the planes' descriptors
    // and are read again (from the scalar cache) in every plane
    typedef TensorParams<P, CPX> Params;
    typedef const __attribute__((address_space(4))) double *Entries;
    Entries cf = (Entries)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
                           offsetof(Params, M));
    constexpr bool RELOAD = P >= 5 || (CPX && P == 4);
    constexpr int NG = anti_count(P);
    constexpr int NS = sym_count(P);
#define TM(i, j) cf[sym_id(P, (i), (j))]
#define TK(i, j) cf[NS + sym_id(P, (i), (j))]
#define TM2 cf[2 * NS]
#define TK2 cf[2 * NS + 1]
#define TGX(i, j) ((i) < (j) ? cf[2 * NS + 2 + anti_id(P, (i), (j))] : -cf[2 * NS + 2 + anti_id(P, (j), (i))])
#define TGY(i, j) ((i) < (j) ? cf[2 * NS + 2 + NG + anti_id(P, (i), (j))] : -cf[2 * NS + 2 + NG + anti_id(P, (j), (i))])

    if (__builtin_amdgcn_readfirstlane(tid) >= 64 * S::CW) {
        // x waves: row xrow of the tile's input rows, cells xs XC .. + XC, vectors
        // 2 sub and 2 sub + 1 of the group (lanes past the last item repeat it:
        // the same values to the same places)
        const int xt = tid - 64 * S::CW, sub = xt % 8, xitem = min(xt / 8, S::XI - 1), xrow = xitem % RY, xs = xitem / RY;
        const uint32_t xb = (uint32_t)(grp * NV + 2 * sub) * 8u;
        uint32_t xoff[NX];
        const int fy = free_node(k.ax[1], cy0 * P - P + xrow);
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int fx = free_node(k.ax[0], (cx0 + xs * XC - 1) * P + j);
            // (the odd vector of a pair whose even one is the block's last reads
            // what lies beside the block, within the plane's range, or zero)
            xoff[j] = grp * NV + 2 * sub < k.N && fy >= 0 && fx >= 0 ? (uint32_t)(fy * k.ax[0].nfree + fx) * k.ldx + xb : kAbsent;
        }
        const uint32_t out = lds0 + 8 * (xrow * RS + xs * XC * P * NV + 2 * sub);  // the item's first output
        // the diagonal terms of the rows that the tile's cells own
        const bool orow = xrow >= P && xrow < P + BY * P;
        const uint32_t dout = lds0 + 8 * (2 * RY * RS + (xrow - P) * RS + xs * XC * P * NV + 2 * sub);
        // v of the item's nodes: lane sub requests nodes sub, sub + 8, ..; the
        // item's lanes share them through LDS (the first node is none on a
        // Dirichlet face: its X reads zero and no output takes its term)
        const uint32_t vlds = lds0 + 8 * (2 * S::BUF + xt / 8 * S::VI);
        uint32_t voff[S::VN];
#pragma unroll
        for (int q = 0; q < S::VN; ++q) {
            const int j = sub + 8 * q, fx = (cx0 + xs * XC) * P - 1 - k.ax[0].per + j;
            voff[q] = orow && fy >= 0 && fx >= 0 && j < XC * P ? (uint32_t)((fy * k.ax[0].nfree + fx) * 8) : kAbsent;
        }
        // X rows of node plane g, and its v (none past the last plane)
        auto issue_x = [&](int g, Pair (&x)[NX]) {
            const __amdgpu_buffer_rsrc_t r = plane_of(k.X, k.px, k.rx, free_node(k.ax[2], g) | ((g1 - g) >> 31));
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                const uint32_t o = xoff[j];
                x[j] = buf_load2(r, o, 0);
            }
        };
        double v[S::VN];
        auto issue_v = [&](int g) {
            const __amdgpu_buffer_rsrc_t r = plane_of(k.v, k.pv, k.rv, free_node(k.ax[2], g) | ((g1 - g) >> 31));
#pragma unroll
            for (int q = 0; q < S::VN; ++q) {
                const uint32_t o = voff[q];
                v[q] = buf_load(r, o, 0);
            }
        };
        auto stage = [&](const Pair (&x)[NX], int buf) {
            if constexpr (RELOAD) opaque(cf);
            {
                LdsDouble *const w = lds_at(vlds + 8 * sub);
#pragma unroll
                for (int q = 0; q < S::VN; ++q) w[8 * q] = v[q] - k.shift;
            }
            LdsDouble *const o = lds_at(out + 8 * buf);
#pragma unroll
            for (int c = 0; c < XC; ++c)
                unroll<0, P>([&](auto II) {
                    constexpr int i = decltype(II)::value;
                    Pair m, q;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        double mm = (i == 0 ? TM2 : TM(i, 0)) * x[(c + 1) * P][h];
                        double qq = (i == 0 ? TK2 : TK(i, 0)) * x[(c + 1) * P][h];
                        if constexpr (i == 0)
                            unroll<0, P>([&](auto JQ) {
                                constexpr int j = decltype(JQ)::value;
                                mm = __builtin_fma(TM(P, j), x[c * P + j][h], mm);
                                qq = __builtin_fma(TK(P, j), x[c * P + j][h], qq);
                                if constexpr (CPX) {
                                    const double g = TGX(P, j);
                                    qq = __builtin_fma(h ? -g : g, x[c * P + j][1 - h], qq);
                                }
                            });
                        unroll<1, P + 1>([&](auto JQ) {
                            constexpr int j = decltype(JQ)::value;
                            mm = __builtin_fma(TM(i, j), x[(c + 1) * P + j][h], mm);
                            qq = __builtin_fma(TK(i, j), x[(c + 1) * P + j][h], qq);
                        });
                        if constexpr (CPX)
                            unroll<0, P + 1>([&](auto JQ) {
                                constexpr int j = decltype(JQ)::value;
                                if constexpr (i != j) {
                                    const double g = TGX(i, j);
                                    qq = __builtin_fma(h ? -g : g, x[(c + 1) * P + j][1 - h], qq);
                                }
                            });
                        m[h] = mm;
                        q[h] = qq;
                    }
                    *(LdsPair *)(o + (c * P + i) * NV) = m;
                    *(LdsPair *)(o + (c * P + i) * NV + RY * RS) = q;
                });
            if (orow) {
                LdsDouble *const d = lds_at(dout + 8 * buf), *const w = lds_at(vlds);
#pragma unroll
                for (int j = 0; j < XC * P; ++j) {
                    const double t = w[j];
                    *(LdsPair *)(d + j * NV) = Pair{t * x[P + j][0], t * x[P + j][1]};
                }
            }
        };
        Pair xa[NX], xb2[NX];
        issue_v(g0);
        issue_x(g0, xa);
        issue_x(g0 + 1, xb2);
        for (int g = g0;;) {
            stage(xa, 0);
            stage_end();
            issue_v(g + 1);
            issue_x(g + 2, xa);
            lds_barrier();
            stage_end();
            if (++g > g1) break;
            stage(xb2, S::BUF);
            stage_end();
            issue_v(g + 1);
            issue_x(g + 2, xb2);
            lds_barrier();
            stage_end();
            if (++g > g1) break;
        }
        return;
    }

    // y-z waves: x position yx, cell yc of the tile
    const int slot = tid / NV, yx = slot % WX, yc = slot / WX;
    uint32_t oy[2], om[2];  // byte offsets of rows 0 and 1 of the cell in a plane of Y and Ym1
    {
        const bool in = live && yc < BY && cx0 + yx / P < k.ax[0].ncell && cy0 + yc < k.ax[1].ncell;
        const int fx = free_node(k.ax[0], cx0 * P + yx);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int fy = free_node(k.ax[1], (cy0 + yc) * P + r);
            // (row 1 of a degree-1 cell is not one of its outputs)
            const bool ok = in && fx >= 0 && fy >= 0 && r < P;
            const uint32_t row = (uint32_t)(fy * k.ax[0].nfree + fx);
            oy[r] = ok ? row * k.ldy + cb : kAbsent;
            om[r] = ok ? row * k.ldm + cb : kAbsent;
        }
    }
    // the first row that the cell's vertex takes, and the cell's diagonal terms
    const uint32_t in = lds0 + 8 * (min(yc, BY - 1) * P * RS + yx * NV + vec);
    const uint32_t din = lds0 + 8 * (2 * RY * RS + min(yc, BY - 1) * P * RS + yx * NV + vec);

    const double sign = vec & 1 ? -1.0 : 1.0;  // of the other half's G u in a re and an im column

    // planes of the previous iterate in flight: two where the registers
    // allow and a layer's planes take the two sets in turn
    constexpr int DEPTH = P == 2 || P == 4 ? 2 : 1;
    double acc[P + 1][P], vm[DEPTH][P];
#pragma unroll
    for (int i = 0; i <= P; ++i)
#pragma unroll
        for (int r = 0; r < P; ++r) acc[i][r] = 0.0;

    // the rows of plane g of the previous iterate, where its outputs are
    // this workgroup's
    auto issue = [&](int g, double (&o)[P]) {
        const int f = free_node(k.ax[2], g) | ((g - cz0 * P) >> 31) | ((g1 - 1 - g) >> 31);
        const __amdgpu_buffer_rsrc_t bm = plane_of(k.Ym1, k.pm, k.rm, f);
        uint32_t sm = (uint32_t)k.ax[0].nfree * k.ldm;
        opaque(sm);
        unroll<0, P>([&](auto QQ) {
            constexpr int q = decltype(QQ)::value;
            const uint32_t b = om[q ? 1 : 0];
            o[q] = buf_load(bm, b, (q ? q - 1 : 0) * sm);
        });
    };

    // one node plane: J its place in its layer (0: the vertex plane that
    // opens layer l and closes l - 1); g its node index; flush: the outputs
    // of the layer that it closes are this workgroup's
    auto plane = [&](auto JJ, int g, bool flush) {
        constexpr int J = decltype(JJ)::value;
        if constexpr (RELOAD) opaque(cf);
        lds_barrier();
        stage_end();
        const uint32_t buf = (g - g0) & 1 ? 8 * S::BUF : 0;
        const LdsDouble *lp = lds_at(in + buf), *lq = lp + RY * RS;
        // the plane's diagonal and previous-iterate terms, to the output
        // plane that it is (the vertex plane's sums are still in place P)
        constexpr int JO = J == 0 ? P : J;
        const LdsDouble *ld = lds_at(din + buf);
#pragma unroll
        for (int r = 0; r < P; ++r)
            acc[JO][r] = __builtin_fma(k.nba, vm[J % DEPTH][r], acc[JO][r] + ld[r * RS]);
#pragma unroll
        for (int r = 0; r < P; ++r) pin(acc[JO][r]);
        stage_end();
        issue(g + DEPTH, vm[J % DEPTH]);
        double A[P], B[P], C[CPX ? P : 1];
        unroll<0, 2 * P + 1>([&](auto RR) {
            constexpr int r = decltype(RR)::value, j = r - P;
            // (bounds the LDS reads in flight)
            if constexpr (P >= 4 && r == P) stage_end();
            const double pr = lp[r * RS], qr = lq[r * RS];
            unroll<0, (j < 0 ? 1 : P)>([&](auto II) {
                constexpr int i = decltype(II)::value;
                // the entries of M and K between row r and output row i
                const double mm = j < 0 ? TM(P, r) : j == 0 && i == 0 ? TM2 : TM(i, j < 0 ? 0 : j);
                const double kk = j < 0 ? TK(P, r) : j == 0 && i == 0 ? TK2 : TK(i, j < 0 ? 0 : j);
                if constexpr (r == (i == 0 ? 0 : P)) {
                    A[i] = mm * pr;
                    B[i] = __builtin_fma(mm, qr, kk * pr);
                } else {
                    A[i] = __builtin_fma(mm, pr, A[i]);
                    B[i] = __builtin_fma(kk, pr, __builtin_fma(mm, qr, B[i]));
                }
                if constexpr (CPX) {
                    if constexpr (r == (i == 0 ? 0 : P)) C[i] = (j < 0 ? TGY(P, r) : TGY(i, 0)) * pr;
                    else if constexpr (j < 0) C[i] = __builtin_fma(TGY(P, r), pr, C[i]);
                    else if constexpr (j != i) C[i] = __builtin_fma(TGY(i, j), pr, C[i]);
                }
            });
        });
        if constexpr (CPX) {
#pragma unroll
            for (int r = 0; r < P; ++r) B[r] = __builtin_fma(sign, neighbour(C[r]), B[r]);
        }
        stage_end();
        // z stage
        if constexpr (J > 0) {
            unroll<0, P + 1>([&](auto II) {
                constexpr int i = decltype(II)::value;
#pragma unroll
                for (int r = 0; r < P; ++r)
                    acc[i][r] = __builtin_fma(TK(i, J), A[r], __builtin_fma(TM(i, J), B[r], acc[i][r]));
            });
        } else {
            // plane by plane, so that an output's registers are free for the
            // next layer's
            unroll<0, P + 1>([&](auto II) {
                constexpr int i = decltype(II)::value;
                if constexpr (i < P) {
                    const __amdgpu_buffer_rsrc_t by =
                        plane_of(k.Y, k.py, k.ry, free_node(k.ax[2], g - P + i) | (flush ? 0 : -1));
                    uint32_t sy = (uint32_t)k.ax[0].nfree * k.ldy;
                    opaque(sy);
                    unroll<0, P>([&](auto QQ) {
                        constexpr int r = decltype(QQ)::value;
                        const double t = __builtin_fma(TK(i, P), A[r], __builtin_fma(TM(i, P), B[r], acc[i][r]));
                        const uint32_t o = oy[r ? 1 : 0];
                        buf_store(k.alpha * t, by, o, (r ? r - 1 : 0) * sy);
                    });
                }
#pragma unroll
                for (int r = 0; r < P; ++r)
                    acc[i][r] = i == 0 ? __builtin_fma(TK2, A[r], __builtin_fma(TM2, B[r], acc[P][r]))
                                       : __builtin_fma(TK(i, 0), A[r], TM(i, 0) * B[r]);
#pragma unroll
                for (int r = 0; r < P; ++r) pin(acc[i][r]);
                stage_end();
            });
        }
#pragma unroll
        for (int i = 0; i <= P; ++i)
#pragma unroll
            for (int r = 0; r < P; ++r) pin(acc[i][r]);
        stage_end();
    };

    issue(g0, vm[0]);
    if constexpr (DEPTH == 2) issue(g0 + 1, vm[1]);
    for (int l = l0;; ++l) {
        plane(std::integral_constant<int, 0>{}, l * P, l > cz0);
        if (l == cz1) break;
        unroll<1, P>([&](auto JJ) { plane(JJ, l * P + decltype(JJ)::value, false); });
    }
#undef TM
#undef TK
#undef TM2
#undef TK2
#undef TGX
#undef TGY
}

// Cell layers per workgroup along z: as many workgroups as keep the chip busy
// in whole rounds, each paying the p planes of the layer below its first.
static int layers_per_group(int64_t columns, int ncz, int p, int64_t slots) {
    int best = ncz;
    double cost = 0.0;
    for (int nz = 1; nz <= ncz; ++nz) {
        const int layers = (ncz + nz - 1) / nz;
        if (nz > 1 && (ncz + layers - 1) / layers != nz) continue;
        const double rounds = std::ceil((double)(columns * nz) / (double)slots);
        const double c = rounds * (layers * p + p + 2);
        if (nz == 1 || c < cost) {
            cost = c;
            best = layers;
        }
    }
    return best;
}

template <int P, int BX, int BY, int XC, int OCC, bool CPX>
static hipError_t launch_tensor_p(const fe_mesh *m, const StepArgs &a, hipStream_t s) {
    typedef TensorShape<P, BX, BY, XC> S;
    // workgroups the chip holds at once
    static const int resident = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, reinterpret_cast<const void *>(&tensor_step_kernel<P, BX, BY, XC, OCC, CPX>), S::T, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();
            return 256;
        }
        return std::max(1, per_cu) * std::max(1, cus);
    }();
    TensorParams<P, CPX> k;
    const int64_t plane = m->nf[0] * m->nf[1];
    k.X = a.X;
    k.Y = a.Y;
    k.Ym1 = a.Ym1 ? a.Ym1 : a.X;
    k.v = a.v ? a.v : m->d_v;
    const int64_t ldm = a.Ym1 ? a.ldm : a.ldx;
    k.ldx = (uint32_t)(a.ldx * 8);
    k.ldy = (uint32_t)(a.ldy * 8);
    k.ldm = (uint32_t)(ldm * 8);
    k.px = plane * a.ldx * 8;
    k.py = plane * a.ldy * 8;
    k.pm = plane * ldm * 8;
    k.pv = plane * 8;
    // a plane's byte range: its last row ends at the block's last column
    k.rx = (uint32_t)(((plane - 1) * a.ldx + a.N) * 8);
    k.ry = (uint32_t)(((plane - 1) * a.ldy + a.N) * 8);
    k.rm = a.Ym1 ? (uint32_t)(((plane - 1) * ldm + a.N) * 8) : 0u;
    k.rv = (uint32_t)k.pv;
    k.alpha = a.alpha;
    k.nba = a.Ym1 ? -a.beta / a.alpha : 0.0;
    k.shift = a.shift;
    k.N = (int)a.N;
    for (int d = 0; d < 3; ++d) {
        k.ax[d].K = m->ncell[d] * m->p;
        k.ax[d].nfree = (int)m->nf[d];
        k.ax[d].per = m->bc[d] == FE_BC_PERIODIC ? -1 : 0;
        k.ax[d].ncell = m->ncell[d];
    }
    for (int i = 0; i <= P; ++i)
        for (int j = 0; j <= P; ++j) {
            k.M[sym_id(P, i, j)] = m->axisM[(size_t)i * (P + 1) + j];
            k.K[sym_id(P, i, j)] = m->axisK[(size_t)i * (P + 1) + j];
        }
    if constexpr (CPX)
        for (int i = 0; i <= P; ++i)
            for (int j = i + 1; j <= P; ++j) {
                k.GX[anti_id(P, i, j)] = m->kvec[0] * m->axisG[(size_t)i * (P + 1) + j];
                k.GY[anti_id(P, i, j)] = m->kvec[1] * m->axisG[(size_t)i * (P + 1) + j];
            }
    k.M2 = 2.0 * m->axisM[0];
    k.K2 = 2.0 * m->axisK[0];
    k.ntx = (m->ncell[0] + BX - 1) / BX;
    k.nty = (m->ncell[1] + BY - 1) / BY;
    const int64_t groups = (a.N + S::NV - 1) / S::NV, columns = (int64_t)k.ntx * k.nty * groups;
    k.layers = layers_per_group(columns, m->ncell[2], P, resident);
    k.nzc = (m->ncell[2] + k.layers - 1) / k.layers;
    // Rows off the 128-byte lines put the ends of two groups' segments into one
    // line; then all groups of a tile go to one XCD side by side, so that its
    // L2 joins their halves (p = 4, 24x24x48 cells, ms per step, tiles / groups
    // next to each other: ld 258 5.24 / 2.81, ld 100 1.86 / 1.30, but ld 256,
    // where the tiles' halo rows are what is shared, 2.44 / 2.85).
    const bool lines = ((k.ldx | k.ldy | k.ldm | (uint32_t)(uintptr_t)a.X | (uint32_t)(uintptr_t)a.Y | (uint32_t)(uintptr_t)k.Ym1) & 127) == 0;
    k.gw = lines ? 1 : (int)groups;
    const int64_t items = columns / groups * ((groups + k.gw - 1) / k.gw * k.gw) * k.nzc;
    if (items > (1 << 28)) return hipErrorInvalidValue;
    k.items = (int)items;
    k.per_xcd = (int)((items + 7) / 8);
    const unsigned blocks = (unsigned)(8 * k.per_xcd);
    hipLaunchKernelGGL((tensor_step_kernel<P, BX, BY, XC, OCC, CPX>), dim3(blocks), dim3(S::T), 0, s, k);
    return hipGetLastError();
}

// Tile shapes (BX, BY cells, XC cells per x item, waves per SIMD), the fastest
// of six to ten each on the slabs above (ms per step on whole / ragged
// 128-byte rows): p = 4 (2, 4) 2.50 / 1.25, (2, 3) 2.46 / 1.30, (3, 3) 2.45 /
// 1.35, (4, 2) 2.55 / 1.28, (2, 2) 2.65 / 1.59; p = 6 (1, 2) 1.56 / 0.78, (2, 2)
// 1.70 / 0.84, (2, 1) 1.71 / 0.88; p = 5 (1, 4) 2.27 / 3.16, (2, 2) 2.31 / 3.22,
// (1, 2) 2.87 / 3.37; p = 3 (2, 6) 0.39 / 0.49, (2, 4) 0.40 / 0.51, (4, 3) 0.42 /
// 0.53; p = 7 (1, 1) 0.60 / 0.66, (1, 2) 0.68 / 0.71.  Two waves on a cell's rows
// (half the output planes each) were no faster at any degree.
template <int P> hipError_t launch_tensor_degree(const fe_mesh *m, const StepArgs &a, hipStream_t s) {
#define FE_TENSOR(PP, BX, BY, XC, OCC)                                             \
    if constexpr (P == PP)                                                         \
        return a.S ? launch_tensor_p<PP, BX, BY, XC, OCC, true>(m, a, s) : launch_tensor_p<PP, BX, BY, XC, OCC, false>(m, a, s);
    FE_TENSOR(1, 4, 8, 2, 4)
    FE_TENSOR(2, 3, 6, 3, 4)
    FE_TENSOR(3, 2, 6, 2, 3)
    FE_TENSOR(4, 2, 4, 2, 3)
    FE_TENSOR(5, 1, 4, 1, 3)
    FE_TENSOR(6, 1, 2, 1, 2)
    FE_TENSOR(7, 1, 1, 1, 2)
#undef FE_TENSOR
}

// ------------------------------------------------------------ single vectors
// The same step for one column (Lanczos, conjugate gradients): the lanes run
// over the nodes.  A workgroup owns BX x BY cells and a range of layers, its
// planes of X go through LDS (coalesced along x, one plane ahead in registers),
// the x stage takes a cell of a row a lane, the y-z stages an x position of a
// cell a lane; two barriers a plane.  Bound by the chain of a plane (about
// 1.7 us: LDS, barrier, x stage, LDS, barrier, y and z stages): a vector of
// 1.8 M nodes is in the caches, and the ranges along z are as short as one layer
// so that the chip is filled, at the price of the layer below each being walked
// again.  us per product, cell products with a second launch that adds them up
// or the coloured cell kernel / this one: p = 4 24x24x48 cells 97 / 23.4, p = 3
// 80 / 13.3.  From 24x24x6 to x24 cells 17-18 us, 48x48x96 96 us.  Tiles of 4x4
// to 16x4 cells and 2 or 4 planes of X ahead took 24.5-30 us at p = 4.
//
// NEU: some axis is zero-Neumann.  The even extension over such a face
// satisfies the same equations with whole vertex masses, in which the face
// node's scaled value is sqrt(2) times as large and its result 1/sqrt(2): X is
// reflected and multiplied when it is loaded, the sums when they are stored.
// DOT: the bare product H0 x (no diagonal term or previous iterate, alpha 1), and
// part[workgroup] = sum over its outputs of x times y; a layer's own x waits in
// LDS for the layer to close.
template <int P, int BX, int BY> struct TensorVecShape {
    static constexpr int WX = BX * P, RX = (BX + 1) * P + 1, RY = (BY + 1) * P + 1;
    static constexpr int YI = WX * BY, XI = RY * BX;       // y-z and x items
    static constexpr int T = ((YI > XI ? YI : XI) + 63) / 64 * 64;
    static constexpr int XR = (XI + T - 1) / T, LR = (RX * RY + T - 1) / T;
    static constexpr int XS = RX | 1, LW = WX | 1;         // odd row strides in LDS
    static constexpr int LDS = RY * XS + 2 * RY * LW;
    static_assert(T <= 1024, "threads of a workgroup");
};

template <int P> struct TensorVecParams {
    const double *X, *Ym1, *v;
    double *Y;
    int64_t px, py, pm, pv;
    uint32_t rx, ry, rm, rv, ldx, ldy, ldm;
    double alpha, nba, shift;
    int ntx, nty, nzc, layers, last;  // last: closing layer along z (the cell count, or one more on a Neumann axis)
    TensorAxis ax[3];
    const double *done;               // DOT: nonzero, nothing to do
    double *part;
    double M[sym_count(P)], K[sym_count(P)], M2, K2;
};

namespace {

constexpr int kNeumann = 1;  // TensorAxis.per of a zero-Neumann axis

// free_node with zero-Neumann axes (the even extension over their faces)
template <bool NEU> __device__ __forceinline__ int free_node_n(const TensorAxis &a, int g) {
    if constexpr (NEU) {
        if (a.per == kNeumann) {
            int f = g < 0 ? -g : g;
            f = f > a.K ? 2 * a.K - f : f;
            return f < 0 ? -1 : f;
        }
    }
    return free_node(a, g);
}
// whether node g (of the axis itself) is on a zero-Neumann face
template <bool NEU> __device__ __forceinline__ bool on_neumann_face(const TensorAxis &a, int g) {
    return NEU && a.per == kNeumann && (g == 0 || g == a.K);
}
// whether node g of the extension is one on a zero-Neumann face: on an axis of
// one cell the nodes -K and 2 K that it reaches are the opposite face's
template <bool NEU> __device__ __forceinline__ bool is_neumann_face(const TensorAxis &a, int g) {
    return on_neumann_face<NEU>(a, g) || (NEU && a.per == kNeumann && (g == -a.K || g == 2 * a.K));
}
// whether node g of cell c is one of the axis' outputs
template <bool NEU> __device__ __forceinline__ bool axis_output(const TensorAxis &a, int c, int g) {
    if (NEU && a.per == kNeumann) return g <= a.K;
    return c < a.ncell && free_node(a, g) >= 0;
}

}  // namespace

template <int P, int BX, int BY, bool NEU, bool DOT>
__global__ __launch_bounds__((TensorVecShape<P, BX, BY>::T))
void tensor_vec_kernel(TensorVecParams<P> k) {
    typedef TensorVecShape<P, BX, BY> S;
    constexpr int T = S::T, WX = S::WX, RX = S::RX, RY = S::RY, XS = S::XS, LW = S::LW, LR = S::LR;
    __shared__ double lds[S::LDS + (DOT ? P * P * T : 0)];
    double *const lx = lds, *const lp = lds + RY * XS, *const lq = lp + RY * LW;
    if constexpr (DOT) {
        if (*k.done != 0.0) return;  // whole grid
    }
    int rest = (int)blockIdx.x;
    const int tx = rest % k.ntx;
    rest /= k.ntx;
    const int ty = rest % k.nty, zc = rest / k.nty;
    const int cx0 = tx * BX, cy0 = ty * BY, cz0 = zc * k.layers, cz1 = min(cz0 + k.layers, k.last);
    const int l0 = k.ax[2].per != 0 || cz0 > 0 ? cz0 - 1 : cz0, g1 = cz1 * P;
    const uint32_t cb = blockIdx.y * 8u;  // the column
    const int tid = threadIdx.x;
    constexpr double R2 = 1.4142135623730951, H2 = 0.70710678118654757;

    // loads: element tid + T q of the tile's RX x RY nodes
    uint32_t off[LR];
    double in_scale[NEU ? LR : 1];
#pragma unroll
    for (int q = 0; q < LR; ++q) {
        const int idx = tid + T * q, row = idx / RX, cx = idx % RX;
        const int gx = cx0 * P - P + cx, gy = cy0 * P - P + row;
        const int fx = free_node_n<NEU>(k.ax[0], gx), fy = free_node_n<NEU>(k.ax[1], gy);
        off[q] = idx < RX * RY && fx >= 0 && fy >= 0 ? (uint32_t)(fy * k.ax[0].nfree + fx) * k.ldx + cb : kAbsent;
        if constexpr (NEU)
            in_scale[q] = (is_neumann_face<NEU>(k.ax[0], gx) ? R2 : 1.0) * (is_neumann_face<NEU>(k.ax[1], gy) ? R2 : 1.0);
    }
    // y-z item: x position yx, cell yc
    const int yx = tid % WX, yc = min(tid / WX, BY - 1);
    uint32_t oy[2], om[2], ov[2];
    double out_scale[NEU ? 2 : 1], inv_scale[NEU ? 2 : 1];
    {
        const int gx = cx0 * P + yx;
        const bool in = tid < S::YI && axis_output<NEU>(k.ax[0], cx0 + yx / P, gx);
        const int fx = free_node_n<NEU>(k.ax[0], gx);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int gy = (cy0 + yc) * P + r, fy = free_node_n<NEU>(k.ax[1], gy);
            const bool ok = in && r < P && axis_output<NEU>(k.ax[1], cy0 + yc, gy);
            const uint32_t row = (uint32_t)(fy * k.ax[0].nfree + fx);
            oy[r] = ok ? row * k.ldy + cb : kAbsent;
            om[r] = ok ? row * k.ldm + cb : kAbsent;
            ov[r] = ok ? row * 8u : kAbsent;
            if constexpr (NEU) {
                const bool ex = on_neumann_face<NEU>(k.ax[0], gx), ey = on_neumann_face<NEU>(k.ax[1], gy);
                out_scale[r] = (ex ? H2 : 1.0) * (ey ? H2 : 1.0);
                inv_scale[r] = (ex ? R2 : 1.0) * (ey ? R2 : 1.0);
            }
        }
    }
#define TM(i, j) k.M[sym_id(P, (i), (j))]
#define TK(i, j) k.K[sym_id(P, (i), (j))]
    double acc[P + 1][P], xr[LR], vm[DOT ? 1 : P], vv[DOT ? 1 : P], dot = 0.0;
    double *const lk = lds + S::LDS + tid;
#pragma unroll
    for (int i = 0; i <= P; ++i)
#pragma unroll
        for (int r = 0; r < P; ++r) acc[i][r] = 0.0;
    auto outside = [&](int g) { return ((g - cz0 * P) >> 31) | ((g1 - 1 - g) >> 31) | ((k.ax[2].K - g) >> 31); };
    auto issue_x = [&](int g) {
        const __amdgpu_buffer_rsrc_t r = plane_of(k.X, k.px, k.rx, free_node_n<NEU>(k.ax[2], g) | ((g1 - g) >> 31));
#pragma unroll
        for (int q = 0; q < LR; ++q) {
            const uint32_t o = off[q];
            xr[q] = buf_load(r, o, 0);
        }
    };
    auto issue_base = [&](int g) {
        if constexpr (DOT) return;
        const int f = free_node_n<NEU>(k.ax[2], g) | outside(g);
        const __amdgpu_buffer_rsrc_t bm = plane_of(k.Ym1, k.pm, k.rm, f), bv = plane_of(k.v, k.pv, k.rv, f);
        const uint32_t sm = (uint32_t)k.ax[0].nfree * k.ldm, sv = (uint32_t)k.ax[0].nfree * 8u;
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const uint32_t a = om[r ? 1 : 0], b = ov[r ? 1 : 0], q = r ? r - 1 : 0;
            vm[r] = buf_load(bm, a, q * sm);
            vv[r] = buf_load(bv, b, q * sv);
        }
    };
    auto plane = [&](auto JJ, int g, bool flush) {
        constexpr int J = decltype(JJ)::value;
        // (faces are vertex planes)
        const double zin = J == 0 && is_neumann_face<NEU>(k.ax[2], g) ? R2 : 1.0;
#pragma unroll
        for (int q = 0; q < LR; ++q) {
            const int idx = tid + T * q, row = idx / RX, cx = idx % RX;
            if (idx < RX * RY) lx[row * XS + cx] = NEU ? xr[q] * (in_scale[q] * zin) : xr[q];
        }
        lds_barrier();
        issue_x(g + 1);
#pragma unroll
        for (int q = 0; q < S::XR; ++q) {
            const int it = tid + T * q, row = it % RY, c = it / RY;
            if (it < S::XI) {
                const double *x = lx + row * XS + c * P;
                double *o = lp + row * LW + c * P;
                double u[2 * P + 1];
#pragma unroll
                for (int j = 0; j <= 2 * P; ++j) u[j] = x[j];
                unroll<0, P>([&](auto II) {
                    constexpr int i = decltype(II)::value;
                    double m = (i == 0 ? k.M2 : TM(i, 0)) * u[P], t = (i == 0 ? k.K2 : TK(i, 0)) * u[P];
                    if constexpr (i == 0)
                        unroll<0, P>([&](auto JQ) {
                            constexpr int j = decltype(JQ)::value;
                            m = __builtin_fma(TM(P, j), u[j], m);
                            t = __builtin_fma(TK(P, j), u[j], t);
                        });
                    unroll<1, P + 1>([&](auto JQ) {
                        constexpr int j = decltype(JQ)::value;
                        m = __builtin_fma(TM(i, j), u[P + j], m);
                        t = __builtin_fma(TK(i, j), u[P + j], t);
                    });
                    o[i] = m;
                    o[RY * LW + i] = t;
                });
            }
        }
        constexpr int JO = J == 0 ? P : J;
        const double *const own = lx + (P + yc * P) * XS + P + yx;
        double bx[DOT ? P : 1];
#pragma unroll
        for (int r = 0; r < P; ++r) {
            if constexpr (DOT) {
                bx[r] = own[r * XS];
            } else {
                double pm = vm[r];
                if constexpr (NEU) pm *= inv_scale[r ? 1 : 0] * zin;
                acc[JO][r] = __builtin_fma(k.nba, pm, __builtin_fma(vv[r] - k.shift, own[r * XS], acc[JO][r]));
            }
        }
        issue_base(g + 1);
        lds_barrier();
        double A[P], B[P];
        unroll<0, 2 * P + 1>([&](auto RR) {
            constexpr int r = decltype(RR)::value, j = r - P;
            const double pr = lp[(yc * P + r) * LW + yx], qr = lq[(yc * P + r) * LW + yx];
            unroll<0, (j < 0 ? 1 : P)>([&](auto II) {
                constexpr int i = decltype(II)::value;
                const double mm = j < 0 ? TM(P, r) : j == 0 && i == 0 ? k.M2 : TM(i, j < 0 ? 0 : j);
                const double kk = j < 0 ? TK(P, r) : j == 0 && i == 0 ? k.K2 : TK(i, j < 0 ? 0 : j);
                if constexpr (r == (i == 0 ? 0 : P)) {
                    A[i] = mm * pr;
                    B[i] = __builtin_fma(mm, qr, kk * pr);
                } else {
                    A[i] = __builtin_fma(mm, pr, A[i]);
                    B[i] = __builtin_fma(kk, pr, __builtin_fma(mm, qr, B[i]));
                }
            });
        });
        if constexpr (J > 0) {
            unroll<0, P + 1>([&](auto II) {
                constexpr int i = decltype(II)::value;
#pragma unroll
                for (int r = 0; r < P; ++r)
                    acc[i][r] = __builtin_fma(TK(i, J), A[r], __builtin_fma(TM(i, J), B[r], acc[i][r]));
            });
        } else {
            unroll<0, P + 1>([&](auto II) {
                constexpr int i = decltype(II)::value;
                if constexpr (i < P) {
                    const int go = g - P + i;
                    const int f = free_node_n<NEU>(k.ax[2], go) | (flush ? outside(go) : -1);
                    const __amdgpu_buffer_rsrc_t by = plane_of(k.Y, k.py, k.ry, f);
                    const uint32_t sy = (uint32_t)k.ax[0].nfree * k.ldy;
                    const double zs = i == 0 && on_neumann_face<NEU>(k.ax[2], go) ? H2 : 1.0;
#pragma unroll
                    for (int r = 0; r < P; ++r) {
                        double t = __builtin_fma(TK(i, P), A[r], __builtin_fma(TM(i, P), B[r], acc[i][r]));
                        const uint32_t o = oy[r ? 1 : 0], q = r ? r - 1 : 0;
                        if constexpr (NEU) t *= out_scale[r ? 1 : 0] * zs;
                        const double y = DOT ? t : k.alpha * t;
                        buf_store(y, by, o, q * sy);
                        if constexpr (DOT) {
                            double x = lk[(i * P + r) * T];
                            if constexpr (NEU) x *= out_scale[r ? 1 : 0] * zs;
                            dot += o != kAbsent && f >= 0 ? x * y : 0.0;
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < P; ++r)
                    acc[i][r] = i == 0 ? __builtin_fma(k.K2, A[r], __builtin_fma(k.M2, B[r], acc[P][r]))
                                       : __builtin_fma(TK(i, 0), A[r], TM(i, 0) * B[r]);
            });
        }
        if constexpr (DOT) {
#pragma unroll
            for (int r = 0; r < P; ++r) lk[(J * P + r) * T] = bx[r];
        }
#pragma unroll
        for (int i = 0; i <= P; ++i)
#pragma unroll
            for (int r = 0; r < P; ++r) pin(acc[i][r]);
    };
    issue_x(l0 * P);
    issue_base(l0 * P);
    for (int l = l0;; ++l) {
        plane(std::integral_constant<int, 0>{}, l * P, l > cz0);
        if (l == cz1) break;
        unroll<1, P>([&](auto JJ) { plane(JJ, l * P + decltype(JJ)::value, false); });
    }
    if constexpr (DOT) {
        // fixed-order sum over the workgroup
        __syncthreads();
        lds[tid] = dot;
        __syncthreads();
        for (int w = 512; w > 0; w >>= 1) {
            if (tid < w && tid + w < T) lds[tid] += lds[tid + w];
            __syncthreads();
        }
        if (tid == 0) k.part[blockIdx.x] = lds[0];
    }
#undef TM
#undef TK
}

template <int P, int BX, int BY, bool NEU, bool DOT>
static hipError_t launch_vec_p(const fe_mesh *m, const StepArgs &a, hipStream_t s, const double *done, double *part,
                               int max_parts, int *nparts) {
    typedef TensorVecShape<P, BX, BY> S;
    static const int resident = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, reinterpret_cast<const void *>(&tensor_vec_kernel<P, BX, BY, NEU, DOT>), S::T, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();
            return 256;
        }
        return std::max(1, per_cu) * std::max(1, cus);
    }();
    TensorVecParams<P> k;
    const int64_t plane = m->nf[0] * m->nf[1], ldm = a.Ym1 ? a.ldm : a.ldx;
    k.X = a.X;
    k.Y = a.Y;
    k.Ym1 = a.Ym1 ? a.Ym1 : a.X;
    k.v = a.v ? a.v : m->d_v;
    k.ldx = (uint32_t)(a.ldx * 8);
    k.ldy = (uint32_t)(a.ldy * 8);
    k.ldm = (uint32_t)(ldm * 8);
    k.px = plane * a.ldx * 8;
    k.py = plane * a.ldy * 8;
    k.pm = plane * ldm * 8;
    k.pv = plane * 8;
    k.rx = (uint32_t)(((plane - 1) * a.ldx + a.N) * 8);
    k.ry = (uint32_t)(((plane - 1) * a.ldy + a.N) * 8);
    k.rm = a.Ym1 ? (uint32_t)(((plane - 1) * ldm + a.N) * 8) : 0u;
    k.rv = (uint32_t)k.pv;
    k.alpha = a.alpha;
    k.nba = a.Ym1 ? -a.beta / a.alpha : 0.0;
    k.shift = a.shift;
    int cells[3];  // with the one past a Neumann axis' last, whose only output is the face
    for (int d = 0; d < 3; ++d) {
        k.ax[d].K = m->ncell[d] * m->p;
        k.ax[d].nfree = (int)m->nf[d];
        k.ax[d].per = m->bc[d] == FE_BC_PERIODIC ? -1 : m->bc[d] == FE_BC_NEUMANN ? kNeumann : 0;
        k.ax[d].ncell = m->ncell[d];
        cells[d] = m->ncell[d] + (m->bc[d] == FE_BC_NEUMANN ? 1 : 0);
    }
    for (int i = 0; i <= P; ++i)
        for (int j = 0; j <= P; ++j) {
            k.M[sym_id(P, i, j)] = m->axisM[(size_t)i * (P + 1) + j];
            k.K[sym_id(P, i, j)] = m->axisK[(size_t)i * (P + 1) + j];
        }
    k.M2 = 2.0 * m->axisM[0];
    k.K2 = 2.0 * m->axisK[0];
    k.ntx = (cells[0] + BX - 1) / BX;
    k.nty = (cells[1] + BY - 1) / BY;
    k.last = cells[2];
    k.layers = layers_per_group((int64_t)k.ntx * k.nty * a.N, k.last, P, resident);
    // (with partial sums: longer ranges where there would be too many)
    while (DOT && k.layers < k.last && (int64_t)k.ntx * k.nty * ((k.last + k.layers - 1) / k.layers) > max_parts) ++k.layers;
    k.nzc = (k.last + k.layers - 1) / k.layers;
    const int64_t blocks = (int64_t)k.ntx * k.nty * k.nzc;
    if (DOT) {
        // (more tiles than partial sums: nothing is launched)
        *nparts = blocks > max_parts ? 0 : (int)blocks;
        if (*nparts == 0) return hipSuccess;
    }
    if (blocks > (1 << 30)) return hipErrorInvalidValue;
    k.done = done;
    k.part = part;
    hipLaunchKernelGGL((tensor_vec_kernel<P, BX, BY, NEU, DOT>), dim3((unsigned)blocks, (unsigned)a.N), dim3(S::T), 0, s, k);
    return hipGetLastError();
}

template <int P>
hipError_t launch_vec_degree(const fe_mesh *m, const StepArgs &a, hipStream_t s, const double *done, double *part,
                             int max_parts, int *nparts) {
    constexpr int BX = P == 1 ? 32 : P == 2 ? 16 : P <= 4 ? 8 : 4, BY = 8;
    const bool neu = m->bc[0] == FE_BC_NEUMANN || m->bc[1] == FE_BC_NEUMANN || m->bc[2] == FE_BC_NEUMANN;
    if (part)
        return neu ? launch_vec_p<P, BX, BY, true, true>(m, a, s, done, part, max_parts, nparts)
                   : launch_vec_p<P, BX, BY, false, true>(m, a, s, done, part, max_parts, nparts);
    return neu ? launch_vec_p<P, BX, BY, true, false>(m, a, s, nullptr, nullptr, 0, nullptr)
               : launch_vec_p<P, BX, BY, false, false>(m, a, s, nullptr, nullptr, 0, nullptr);
}

// Every degree in one object, or with FE_TENSOR_DEGREE that one: the unrolled
// walks take the compiler longer than the rest of the library, so build.py
// compiles the degrees side by side.
#define FE_DEGREE(PP)                                                                                              \
    template hipError_t launch_tensor_degree<PP>(const fe_mesh *, const StepArgs &, hipStream_t);                  \
    template hipError_t launch_vec_degree<PP>(const fe_mesh *, const StepArgs &, hipStream_t, const double *, double *, int, int *);
#ifdef FE_TENSOR_DEGREE
FE_DEGREE(FE_TENSOR_DEGREE)
#else
FE_DEGREE(1)
FE_DEGREE(2)
FE_DEGREE(3)
FE_DEGREE(4)
FE_DEGREE(5)
FE_DEGREE(6)
FE_DEGREE(7)
#endif
#undef FE_DEGREE

}  // namespace fe
