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
//  - x stage: a lane holds one vector of one x row of the plane (the tile's
//    cells and the cell before them, as a vertex node takes both cells it
//    belongs to), loaded from global memory one plane ahead, and forms M_x u
//    and K_x u for its output nodes into LDS;
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
// flight, the y-z waves the output planes), so four waves fit a SIMD at
// p = 4; with both stages in every wave, 168 registers and two barriers per
// plane, the p = 4 slab below took 3.81 ms a step instead of 2.76.
// Every output is summed by one lane in one order: no atomics, no partial
// sums in memory, the same bits on every run, and independent of the vectors
// beside it.  Each value of X, the previous iterate and Y moves once, but for
// the X rows of the halo (a cell before and a node after the tile along x
// and y), which the neighbouring workgroups of the same XCD read at about the
// same time.
//
// Measured, ms per recurrence step (two blocks read, one written), against the
// kernels it replaces as the FP64 default: p = 4, 24x24x48 cells, 256 vectors
// 2.76 (the table kernel 4.73) = 3.9 TB/s of the 24 bytes per value, of 5.9
// that two reads and a write stream at; p = 6, 16x16x32 cells, 128 vectors 2.49
// (5.53); p = 5, 20x20x40 cells, 200 vectors 3.52 (8.79); p = 3, 24x24x48 cells,
// 100 vectors 0.66 (1.45); p = 2, 30x30x60 cells, 100 vectors 0.40 (1.09).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
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

}  // namespace

struct TensorAxis {
    int K;     // ncell * p: the period, or the last node of a Dirichlet axis
    int nfree;
    int per;   // -1: periodic, 0: Dirichlet
    int ncell;
};

template <int P> struct TensorParams {
    const double *X, *Ym1, *v;
    double *Y;
    int64_t px, py, pm, pv;           // plane strides in bytes
    uint32_t rx, ry, rm, rv;          // plane byte ranges (0: absent)
    uint32_t ldx, ldy, ldm;           // row strides in bytes
    double alpha, nba, shift;         // nba = -beta / alpha
    int N, ntx, nty, nzc, layers, items, per_xcd;
    TensorAxis ax[3];
    double M[sym_count(P)], K[sym_count(P)], M2, K2;  // M2, K2: the vertex entries of two cells
};

namespace {

constexpr uint32_t kAbsent = 0x80000000u;  // a byte offset past every plane: reads zeros, stores nothing
constexpr int kRawBuffer = 0x00020000;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return __builtin_bit_cast(double, w);
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

// A sum that is formed by here (the compiler may not defer it).
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// A uniform value that the compiler forms again where it is used, rather than
// hold every multiple of it in registers for the whole walk.
__device__ __forceinline__ void opaque(uint32_t &x) { asm volatile("" : "+s"(x)); }

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
    static constexpr int CW = (WX * BY * NV + 63) / 64;          // y-z waves
    static constexpr int XI = RY * (BX / XC);                    // x items (row, XC cells)
    static constexpr int XW = (XI * NV + 63) / 64;               // x waves
    static constexpr int T = 64 * (CW + XW);
    static constexpr int RS = WX * NV + (WX % 2 ? 0 : NV);       // row stride: an odd number of 128-byte lines
    static constexpr int BUF = 2 * RY * RS;                      // M_x u and K_x u of one plane
    static constexpr int LDS = 2 * BUF;
    static_assert(BX % XC == 0, "whole items in a tile's row");
    static_assert(T <= 1024, "threads of a workgroup");
    static_assert(LDS * 8 <= 160 * 1024, "LDS of a workgroup");
};

template <int P, int BX, int BY, int XC, int OCC>
__global__ __launch_bounds__((TensorShape<P, BX, BY, XC>::T)) __attribute__((amdgpu_waves_per_eu(OCC)))
void tensor_step_kernel(TensorParams<P> k) {
    typedef TensorShape<P, BX, BY, XC> S;
    constexpr int NV = S::NV, WX = S::WX, RY = S::RY, RS = S::RS, NX = (XC + 1) * P + 1;
    __shared__ double lds[S::LDS];

    const int item = (int)(blockIdx.x & 7) * k.per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= k.per_xcd || item >= k.items) return;  // whole workgroup
    int rest = item;
    const int tx = rest % k.ntx;
    rest /= k.ntx;
    const int ty = rest % k.nty;
    rest /= k.nty;
    const int zc = rest % k.nzc, grp = rest / k.nzc;
    const int cx0 = tx * BX, cy0 = ty * BY, cz0 = zc * k.layers, cz1 = min(cz0 + k.layers, k.ax[2].ncell);
    // the planes walked: from the layer before the first (its planes reach the
    // first vertex plane) to the vertex plane that closes the last; a first
    // layer on a Dirichlet face has none before it
    const int l0 = k.ax[2].per || cz0 > 0 ? cz0 - 1 : cz0;
    const int g0 = l0 * P, g1 = cz1 * P;

    const int tid = threadIdx.x, vec = tid % NV, col = grp * NV + vec;
    const bool live = col < k.N;
    const uint32_t cb = (uint32_t)col * 8u;
#define TM(i, j) k.M[sym_id(P, (i), (j))]
#define TK(i, j) k.K[sym_id(P, (i), (j))]

    if (__builtin_amdgcn_readfirstlane(tid) >= 64 * S::CW) {
        // x waves: row xrow of the tile's input rows, cells xs XC .. + XC (lanes
        // past the last item repeat it: the same values to the same places)
        const int xitem = min((tid - 64 * S::CW) / NV, S::XI - 1), xrow = xitem % RY, xs = xitem / RY;
        uint32_t xoff[NX];
        const int fy = free_node(k.ax[1], cy0 * P - P + xrow);
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int fx = free_node(k.ax[0], (cx0 + xs * XC - 1) * P + j);
            xoff[j] = live && fy >= 0 && fx >= 0 ? (uint32_t)(fy * k.ax[0].nfree + fx) * k.ldx + cb : kAbsent;
        }
        double *const out = lds + xrow * RS + xs * XC * P * NV + vec;  // the item's first output
        // X rows of node plane g (none past the last)
        auto issue = [&](int g, double (&x)[NX]) {
            const __amdgpu_buffer_rsrc_t rs = plane_of(k.X, k.px, k.rx, free_node(k.ax[2], g) | ((g1 - g) >> 31));
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                const uint32_t o = xoff[j];
                x[j] = buf_load(rs, o, 0);
            }
        };
        auto stage = [&](const double (&x)[NX], double *o) {
#pragma unroll
            for (int c = 0; c < XC; ++c)
                unroll<0, P>([&](auto II) {
                    constexpr int i = decltype(II)::value;
                    double m = (i == 0 ? k.M2 : TM(i, 0)) * x[(c + 1) * P];
                    double q = (i == 0 ? k.K2 : TK(i, 0)) * x[(c + 1) * P];
                    if constexpr (i == 0)
                        unroll<0, P>([&](auto JQ) {
                            constexpr int j = decltype(JQ)::value;
                            m = __builtin_fma(TM(P, j), x[c * P + j], m);
                            q = __builtin_fma(TK(P, j), x[c * P + j], q);
                        });
                    unroll<1, P + 1>([&](auto JQ) {
                        constexpr int j = decltype(JQ)::value;
                        m = __builtin_fma(TM(i, j), x[(c + 1) * P + j], m);
                        q = __builtin_fma(TK(i, j), x[(c + 1) * P + j], q);
                    });
                    o[(c * P + i) * NV] = m;
                    o[(c * P + i) * NV + RY * RS] = q;
                });
        };
        double xa[NX], xb[NX];
        issue(g0, xa);
        issue(g0 + 1, xb);
        for (int g = g0;;) {
            stage(xa, out);
            stage_end();
            issue(g + 2, xa);
            lds_barrier();
            stage_end();
            if (++g > g1) break;
            stage(xb, out + S::BUF);
            stage_end();
            issue(g + 2, xb);
            lds_barrier();
            stage_end();
            if (++g > g1) break;
        }
        return;
    }

    // y-z waves: x position yx, cell yc of the tile
    const int slot = tid / NV, yx = slot % WX, yc = slot / WX;
    uint32_t ox[2], oy[2], om[2], ov[2];  // byte offsets of rows 0 and 1 of the cell
    {
        const bool in = live && yc < BY && cx0 + yx / P < k.ax[0].ncell && cy0 + yc < k.ax[1].ncell;
        const int fx = free_node(k.ax[0], cx0 * P + yx);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int fy = free_node(k.ax[1], (cy0 + yc) * P + r);
            // (row 1 of a degree-1 cell is not one of its outputs)
            const bool ok = in && fx >= 0 && fy >= 0 && r < P;
            const uint32_t row = (uint32_t)(fy * k.ax[0].nfree + fx);
            ox[r] = ok ? row * k.ldx + cb : kAbsent;
            oy[r] = ok ? row * k.ldy + cb : kAbsent;
            om[r] = ok ? row * k.ldm + cb : kAbsent;
            ov[r] = ok ? row * 8u : kAbsent;
        }
    }
    const double *in = lds + min(yc, BY - 1) * P * RS + yx * NV + vec;  // the first row that the cell's vertex takes

    double acc[P + 1][P], vx[P], vm[P], vv[P];
#pragma unroll
    for (int i = 0; i <= P; ++i)
#pragma unroll
        for (int r = 0; r < P; ++r) acc[i][r] = 0.0;

    // the rows of plane g for its diagonal and previous-iterate terms, where
    // its outputs are this workgroup's
    auto issue = [&](int g, bool own) {
        const int f = free_node(k.ax[2], g) | (own ? 0 : -1);
        const __amdgpu_buffer_rsrc_t bx = plane_of(k.X, k.px, k.rx, f), bm = plane_of(k.Ym1, k.pm, k.rm, f),
                                     bv = plane_of(k.v, k.pv, k.rv, f);
        uint32_t sx = (uint32_t)k.ax[0].nfree * k.ldx, sm = (uint32_t)k.ax[0].nfree * k.ldm, sv = (uint32_t)k.ax[0].nfree * 8u;
        opaque(sx);
        opaque(sm);
        opaque(sv);
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const uint32_t a = ox[r ? 1 : 0], b = om[r ? 1 : 0], c = ov[r ? 1 : 0], q = r ? r - 1 : 0;
            vx[r] = buf_load(bx, a, q * sx);
            vm[r] = buf_load(bm, b, q * sm);
            vv[r] = buf_load(bv, c, q * sv);
        }
    };

    // one node plane: J its place in its layer (0: the vertex plane that opens
    // layer l and closes l - 1); g its node index; flush: the outputs of the
    // layer that it closes are this workgroup's; nown: so are those of the
    // next plane
    auto plane = [&](auto JJ, int g, bool flush, bool nown) {
        constexpr int J = decltype(JJ)::value;
        lds_barrier();
        stage_end();
        const double *lp = in + ((g - g0) & 1 ? S::BUF : 0), *lq = lp + RY * RS;
        double A[P], B[P];
        unroll<0, 2 * P + 1>([&](auto RR) {
            constexpr int r = decltype(RR)::value;
            const double pr = lp[r * RS], qr = lq[r * RS];
            if constexpr (r < P) {
                if constexpr (r == 0) {
                    A[0] = TM(P, 0) * pr;
                    B[0] = __builtin_fma(TM(P, 0), qr, TK(P, 0) * pr);
                } else {
                    A[0] = __builtin_fma(TM(P, r), pr, A[0]);
                    B[0] = __builtin_fma(TK(P, r), pr, __builtin_fma(TM(P, r), qr, B[0]));
                }
            } else {
                constexpr int j = r - P;
                unroll<0, P>([&](auto II) {
                    constexpr int i = decltype(II)::value;
                    if constexpr (j == 0 && i == 0) {
                        A[0] = __builtin_fma(k.M2, pr, A[0]);
                        B[0] = __builtin_fma(k.K2, pr, __builtin_fma(k.M2, qr, B[0]));
                    } else if constexpr (j == 0) {
                        A[i] = TM(i, 0) * pr;
                        B[i] = __builtin_fma(TM(i, 0), qr, TK(i, 0) * pr);
                    } else {
                        A[i] = __builtin_fma(TM(i, j), pr, A[i]);
                        B[i] = __builtin_fma(TK(i, j), pr, __builtin_fma(TM(i, j), qr, B[i]));
                    }
                });
            }
        });
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
            unroll<0, P>([&](auto II) {
                constexpr int i = decltype(II)::value;
                const __amdgpu_buffer_rsrc_t by =
                    plane_of(k.Y, k.py, k.ry, free_node(k.ax[2], g - P + i) | (flush ? 0 : -1));
                uint32_t sy = (uint32_t)k.ax[0].nfree * k.ldy;
                opaque(sy);
#pragma unroll
                for (int r = 0; r < P; ++r) {
                    const double t = __builtin_fma(TK(i, P), A[r], __builtin_fma(TM(i, P), B[r], acc[i][r]));
                    const uint32_t o = oy[r ? 1 : 0], q = r ? r - 1 : 0;
                    buf_store(k.alpha * t, by, o, q * sy);
                }
            });
#pragma unroll
            for (int r = 0; r < P; ++r)
                acc[0][r] = __builtin_fma(k.K2, A[r], __builtin_fma(k.M2, B[r], acc[P][r]));
            unroll<1, P + 1>([&](auto II) {
                constexpr int i = decltype(II)::value;
#pragma unroll
                for (int r = 0; r < P; ++r) acc[i][r] = __builtin_fma(TK(i, 0), A[r], TM(i, 0) * B[r]);
            });
        }
#pragma unroll
        for (int r = 0; r < P; ++r)
            acc[J][r] = __builtin_fma(k.nba, vm[r], __builtin_fma(vv[r] - k.shift, vx[r], acc[J][r]));
#pragma unroll
        for (int i = 0; i <= P; ++i)
#pragma unroll
            for (int r = 0; r < P; ++r) pin(acc[i][r]);
        stage_end();
        issue(g + 1, nown);
        stage_end();
    };

    issue(g0, l0 >= cz0);
    for (int l = l0;; ++l) {
        const bool own = l >= cz0 && l < cz1;
        plane(std::integral_constant<int, 0>{}, l * P, l > cz0, P > 1 ? own : l + 1 >= cz0 && l + 1 < cz1);
        if (l == cz1) break;
        unroll<1, P>([&](auto JJ) {
            constexpr int j = decltype(JJ)::value;
            plane(JJ, l * P + j, false, j + 1 < P ? own : l + 1 >= cz0 && l + 1 < cz1);
        });
    }
#undef TM
#undef TK
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

template <int P, int BX, int BY, int XC, int OCC>
static hipError_t launch_tensor_p(const fe_mesh *m, const StepArgs &a, hipStream_t s) {
    typedef TensorShape<P, BX, BY, XC> S;
    // workgroups the chip holds at once
    static const int resident = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, reinterpret_cast<const void *>(&tensor_step_kernel<P, BX, BY, XC, OCC>), S::T, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();
            return 256;
        }
        return std::max(1, per_cu) * std::max(1, cus);
    }();
    TensorParams<P> k;
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
    k.M2 = 2.0 * m->axisM[0];
    k.K2 = 2.0 * m->axisK[0];
    k.ntx = (m->ncell[0] + BX - 1) / BX;
    k.nty = (m->ncell[1] + BY - 1) / BY;
    const int64_t groups = (a.N + S::NV - 1) / S::NV, columns = (int64_t)k.ntx * k.nty * groups;
    k.layers = layers_per_group(columns, m->ncell[2], P, resident);
    k.nzc = (m->ncell[2] + k.layers - 1) / k.layers;
    const int64_t items = columns * k.nzc;
    if (items > (1 << 28)) return hipErrorInvalidValue;
    k.items = (int)items;
    k.per_xcd = (int)((items + 7) / 8);
    hipLaunchKernelGGL((tensor_step_kernel<P, BX, BY, XC, OCC>), dim3((unsigned)(8 * k.per_xcd)), dim3(S::T), 0, s, k);
    return hipGetLastError();
}

// Whether the tensor-product form applies: no zero-Neumann axis (M^-1/2 of a
// node is then a product of factors of its local indices, the same in every
// cell), a plane of every block within the 31 bits of its buffer requests,
// and a recurrence whose beta / alpha is a number.
bool tensor_applies(const fe_mesh *m, const StepArgs &a) {
    if (m->axisM.empty() || a.S) return false;
    const int64_t plane = m->nf[0] * m->nf[1], ld = std::max(std::max(a.ldx, a.ldy), a.Ym1 ? a.ldm : (int64_t)0);
    if (ld > (int64_t)0x7FFFFFFF / 8 / plane) return false;
    if (a.N >= (int64_t)1 << 31) return false;
    return a.alpha != 0.0 && std::isfinite(a.beta / a.alpha);
}

// Where it is the default.  It is faster than the cell kernels at every size
// measured (DESIGN has the table), so the line is drawn by what else holds:
// the default of the other degrees on a few cells, and of one or two vectors
// up to a mesh of the size where Lanczos and CG spend time on the product,
// are documented to equal the one-cell kernel (variant 1) bit for bit.  The
// rule looks at the number of vectors, not of real columns, so that a complex
// block at the Gamma point takes the kernel of its real and imaginary parts.
bool tensor_default(const fe_mesh *m, const StepArgs &a) {
    const int64_t vectors = a.vectors ? a.vectors : a.N;
    if (vectors < 3) return false;
    return m->p == 3 || m->p == 4 || m->ncells >= 64;
}

hipError_t launch_tensor(const fe_mesh *m, const StepArgs &a, hipStream_t s) {
    switch (m->p) {
    case 1: return launch_tensor_p<1, 8, 4, 2, 4>(m, a, s);
    case 2: return launch_tensor_p<2, 8, 2, 2, 4>(m, a, s);
    case 3: return launch_tensor_p<3, 4, 3, 2, 4>(m, a, s);
    case 4: return launch_tensor_p<4, 4, 2, 2, 4>(m, a, s);
    case 5: return launch_tensor_p<5, 3, 2, 3, 3>(m, a, s);
    case 6: return launch_tensor_p<6, 2, 2, 2, 3>(m, a, s);
    case 7: return launch_tensor_p<7, 2, 1, 2, 2>(m, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fe
