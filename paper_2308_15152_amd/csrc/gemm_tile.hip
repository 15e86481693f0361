// The tile kernel's instances and the choice among them (tile_gemm.hpp has
// the kernel).
//
// It takes whole tiles that are too few for the full-tile kernel to fill the
// device, ragged products, products with unaligned rows and the accumulate
// form with its transposed operands.
#include "tile_gemm.hpp"
#include "tile_launch.h"

namespace sgemm_emu {
namespace tile {

namespace {

template <class CF>
__global__ __launch_bounds__(CF::NT, CF::W) void gemm_tile_kernel(Params p) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[CF::LDS_BYTES];
    run<CF>(p, smem);
}

// What a shape costs, to rank the shapes by; not times.  A workgroup takes
// `first` per chunk when it has a CU to itself, and `chunk` for each of those
// that share one (at most `fit` do), plus `ends` for filling the pipeline and
// storing C.  Fitted to the order of the shapes' times (scaled as microseconds)
// on 160 products from 16 x 64^3 to 6000^2 x 960, odd sizes and transposed
// operands among them: the shape chosen is 0.9% slower than the best one on
// average, 15% at worst.  The estimate is below the time where all CUs run, whose
// clock falls under the products, most of all for 128 x 256 (8 x 1001 x 999 x
// 1003 35 for 57 us, 4096^3 with B stored n x k 317 for 370, 32 x 512^3 20 for
// 29).  (Without the shapes with k groups 2%: the waves of one group go through
// reads, products and split in step, and a second group fills the gaps: 1024^3
// 16.4 -> 13.9 us, 2048^3 64 -> 55, 4 x 256 x 256 x 4096 54 -> 32.)
struct Cost {
    int bm, bn, kg, fit;
    double first, chunk, ends;
};
constexpr Cost kCosts[NONE] = {
    {64, 64, 1, 4, 0.55, 0.357, 0.97},    // T64
    {64, 64, 2, 2, 0.34, 0.298, 3.78},    // T64_K2
    {64, 64, 4, 1, 0.29, 0.290, 5.07},    // T64_K4
    {128, 64, 1, 2, 0.54, 0.420, 5.75},   // T128x64
    {128, 64, 2, 1, 0.52, 0.515, 3.02},   // T128x64_K2
    {128, 128, 1, 2, 0.67, 0.576, 4.37},  // T128
    {128, 128, 2, 1, 0.58, 0.584, 5.68},  // T128_K2
    {128, 256, 1, 1, 0.93, 0.933, 4.80},  // T128x256
};
constexpr double kCus = 256;

double cost(const Cost& c, const Problem& p) {
    const double tiles = (double)((p.m + c.bm - 1) / c.bm) * ((p.n + c.bn - 1) / c.bn) * p.batch;
    const int chunks = (p.k + BK - 1) / BK;
    const double steps = (double)((chunks + c.kg - 1) / c.kg) * c.kg;
    const double here = __builtin_ceil(tiles / kCus);  // workgroups of the busiest CU
    if (here <= c.fit) {
        const double chunk = here * c.chunk > c.first ? here * c.chunk : c.first;
        return steps * chunk + c.ends * (1 + 0.5 * (here - 1));
    }
    const double n = tiles / kCus + (c.fit == 1 ? 0.5 : 0.25);
    // the ends overlap other workgroups' chunks, or, with one on the CU, wait
    // for C besides (1024 x 256^3 with C: 128 x 128 209 us, 128 x 256 235;
    // without 195 / 174)
    const double ends = c.ends * (c.fit > 1 ? 0.6 : p.C ? 1.5 : 1.0);
    return (n > c.fit ? n : c.fit) * (steps * c.chunk + ends);
}

// Workgroups of the shape that one launch holds: it stays below 2^31
// work-items.
int64_t max_tasks(int threads) { return (int64_t(1) << 31) / threads - 1; }

bool fits(const Cost& c, const Problem& p) {
    // the tiles of one item go out in one launch
    const int threads = 256 * c.kg * (c.bm * c.bn > 128 * 128 ? 2 : 1);
    const int64_t tiles = (int64_t)cdiv(p.m, c.bm) * cdiv(p.n, c.bn);
    if (tiles > max_tasks(threads)) return false;
    // only the smallest tile has an EDGE form
    if (c.bm + c.bn > 128 && (p.m < c.bm || p.n < c.bn)) return false;
    return offsets_fit(p.a_kc, c.bm, p.lda) && offsets_fit(p.b_kc, c.bn, p.ldb) &&
           offsets_fit(true, c.bm, p.ldd + c.bn) &&
           (p.C == nullptr || offsets_fit(true, c.bm, p.ldc + c.bn));
}

template <class CF>
hipError_t launch_cfg(const Problem& a, hipStream_t stream) {
    Params p;
    p.m = a.m;
    p.n = a.n;
    p.k = a.k;
    p.A = a.A;
    p.lda = a.lda;
    p.sa = a.sa;
    p.B = a.B;
    p.ldb = a.ldb;
    p.sb = a.sb;
    p.C = a.C;
    p.ldc = a.ldc;
    p.sc = a.sc;
    p.D = a.D;
    p.ldd = a.ldd;
    p.sd = a.sd;
    p.tiles_m = cdiv(a.m, CF::BM);
    p.tiles_n = cdiv(a.n, CF::BN);
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    if (tiles > max_tasks(CF::NT)) return hipErrorInvalidConfiguration;
    const int64_t items_per_launch = max_tasks(CF::NT) / tiles;
    for (int64_t i0 = 0; i0 < a.batch; i0 += items_per_launch) {
        const int64_t items = a.batch - i0 < items_per_launch ? a.batch - i0 : items_per_launch;
        p.ntasks = (int)(items * tiles);
        p.item0 = (int)i0;
        hipLaunchKernelGGL(gemm_tile_kernel<CF>, dim3((unsigned)p.ntasks), dim3(CF::NT), 0, stream,
                           p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool A_KC, bool B_KC, bool ADD>
hipError_t launch_shape(const Problem& a, Shape shape, hipStream_t s) {
    const bool edge = a.m < 64 || a.n < 64;
    switch (shape) {
        case T64:
            return edge ? launch_cfg<Cfg<64, 64, 2, 2, 1, 4, A_KC, B_KC, ADD, true>>(a, s)
                        : launch_cfg<Cfg<64, 64, 2, 2, 1, 4, A_KC, B_KC, ADD, false>>(a, s);
        case T64_K2:
            return edge ? launch_cfg<Cfg<64, 64, 2, 2, 2, 4, A_KC, B_KC, ADD, true>>(a, s)
                        : launch_cfg<Cfg<64, 64, 2, 2, 2, 4, A_KC, B_KC, ADD, false>>(a, s);
        case T64_K4:
            return edge ? launch_cfg<Cfg<64, 64, 2, 2, 4, 4, A_KC, B_KC, ADD, true>>(a, s)
                        : launch_cfg<Cfg<64, 64, 2, 2, 4, 4, A_KC, B_KC, ADD, false>>(a, s);
        case T128x64: return launch_cfg<Cfg<128, 64, 2, 2, 1, 2, A_KC, B_KC, ADD, false>>(a, s);
        case T128x64_K2:
            return launch_cfg<Cfg<128, 64, 2, 2, 2, 2, A_KC, B_KC, ADD, false>>(a, s);
        case T128: return launch_cfg<Cfg<128, 128, 2, 2, 1, 2, A_KC, B_KC, ADD, false>>(a, s);
        case T128_K2: return launch_cfg<Cfg<128, 128, 2, 2, 2, 2, A_KC, B_KC, ADD, false>>(a, s);
        case T128x256:
            return launch_cfg<Cfg<128, 256, 2, 4, 1, 2, A_KC, B_KC, ADD, false>>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

Shape choose(const Problem& p) {
    const int lim = 1 << 30;  // row, column and k indices are formed in 32 bits
    if (p.m < 1 || p.n < 1 || p.k < 1 || p.m >= lim || p.n >= lim || p.k >= lim) return NONE;
    if ((!p.a_kc && p.m < 4) || (!p.b_kc && p.n < 4)) return NONE;
    Shape best = NONE;
    double best_time = 0;
    for (int s = 0; s < NONE; ++s) {
        if (!fits(kCosts[s], p)) continue;
        const double t = cost(kCosts[s], p);
        if (best == NONE || t < best_time) {
            best = (Shape)s;
            best_time = t;
        }
    }
    return best;
}

Shape far_rows(const Problem& p) {
    const Cost& c = kCosts[T128x256];
    if (p.acc || !p.a_kc || p.b_kc || offsets_fit(true, c.bm, p.ldd + c.bn)) return NONE;
    Problem near = p;
    near.ldd = p.n;
    return choose(near) != NONE && fits(c, near) ? T128x256_FAR : NONE;
}

hipError_t launch(const Problem& p, Shape shape, hipStream_t stream) {
    if (shape == T128x256_FAR)
        return launch_cfg<Cfg<128, 256, 2, 4, 1, 2, true, false, false, false, true>>(p, stream);
    if (shape == NONE) return hipErrorInvalidValue;
    if (!p.acc && (!p.a_kc || p.b_kc || p.C)) return hipErrorInvalidValue;
    if (p.a_kc && !p.b_kc)
        return p.acc ? launch_shape<true, false, true>(p, shape, stream)
                   : launch_shape<true, false, false>(p, shape, stream);
    if (p.a_kc) return launch_shape<true, true, true>(p, shape, stream);
    return p.b_kc ? launch_shape<false, true, true>(p, shape, stream)
                  : launch_shape<false, false, true>(p, shape, stream);
}

Form form(Shape shape) {
    if (shape == NONE) return {0, 0, 0};
    if (shape == T128x256_FAR) shape = T128x256;
    return {kCosts[shape].bm, kCosts[shape].bn, kCosts[shape].kg};
}

}  // namespace tile
}  // namespace sgemm_emu
