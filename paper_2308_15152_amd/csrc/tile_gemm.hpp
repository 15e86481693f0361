// The tile kernel: one BM x BN tile of D = op(A) op(B) (+ C) per workgroup,
// for operands of any layout, size and alignment (Sec. 4.4; batched form of
// Sec. 4.4.2).  Products without and with C, ragged, unaligned or too few
// tiles for the full-tile kernel, run on it.
//
// Per k chunk of 32 every thread loads its part of both operands into
// registers with 16-byte loads along the direction in which the operand is
// contiguous, splits the values there and writes hi and lo to LDS, so each
// element is split once per workgroup; the waves read ready operand vectors
// and run three MFMAs per 32 x 32 block and 16-wide k step.
//
// An operand is K-contiguous (A stored m x k, B stored n x k) or
// M/N-contiguous (A stored k x m, B stored k x n).  In terms of its index
// "line" (a row of op(A), a column of op(B)):
//   K-contiguous    a unit is 8 consecutive k of one line (two loads); LDS
//                   planes of 64-byte lines, piece q (8 halves) of line r at
//                   q ^ ((r ^ (r >> 2)) & 3); fragments are 16-byte reads.
//   M/N-contiguous  a quad is 4 consecutive lines of one k (one load); LDS
//                   planes [k][lines], fragments by gfx950's transposing read
//                   (two 8-byte reads).  Quad q of k sits at q ^ 8 (k & 3)
//                   when a k row is 256 bytes or more; a k row of 64 lines
//                   (128 bytes) is half of that, so two k rows share the 64
//                   banks and bit 1 of k decides alone: q ^ 8 ((k >> 1) & 1).
// Both layouts keep reads and writes on distinct banks.
//
// Sizes.  The last tile of a row or column of tiles is moved back so that it
// ends with the matrix: it computes some outputs again and stores only its
// own.  No load then needs a bound in m or n.  (A matrix smaller than one
// tile, EDGE: lines past the end repeat the last line, or the last quad,
// whose values the split puts in place.)  A k tail is the first chunk of the
// loop: loads past the operand's end return zero (the buffer descriptor ends
// there) and what belongs to the next line is zeroed before the split.
// Loads are buffer loads, which need 4-byte alignment only.
//
// Pipeline: two LDS stages and two register stages, as in the full-tile
// kernel: iteration c issues the products of chunk c, splits chunk c + 1 into
// LDS, issues the loads of chunk c + 3 and meets one barrier that orders LDS
// only.  Chunk indices past the end are clamped, so every load of the loop is
// unconditional.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

#include "mfmae/frag.hpp"
#include "mfmae/tcec.hpp"
#include "tiling.hpp"

namespace sgemm_emu {
namespace tile {

using mfmae::f32x16_t;
using mfmae::half8_t;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 32;
constexpr int kNontemporal = 2;            // cache policy of buffer stores
constexpr uint32_t kPastEnd = 0x80000000;  // no buffer offset in use reaches this

struct Params {
    int m, n, k;
    const float* A;
    int64_t lda, sa;
    const float* B;
    int64_t ldb, sb;
    const float* C;  // added to the product; null: nothing
    int64_t ldc, sc;
    float* D;
    int64_t ldd, sd;
    int tiles_m, tiles_n;
    int ntasks;  // (items of this launch) x (tiles per item)
    int item0;
};

// BM x BN tiles, KG groups of WAVES_M x WAVES_N waves that share the tile's
// chunks, at least W waves per SIMD; A_KC / B_KC: the operand is K-contiguous;
// ADD: C is added; EDGE: m < BM or n < BN; FAR: D's rows are too far apart for
// 32-bit offsets (nothing is added then).
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int KG_, int W_, bool A_KC_, bool B_KC_,
          bool ADD_, bool EDGE_, bool FAR_ = false>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, KG = KG_;
    static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, W = W_;
    static constexpr bool A_KC = A_KC_, B_KC = B_KC_, ADD = ADD_, EDGE = EDGE_, FAR = FAR_;
    static_assert(!(ADD && FAR), "C would need 64-bit offsets too");
    static constexpr int GROUP = 64 * WAVES_M * WAVES_N;  // threads of a group
    static constexpr int NT = KG * GROUP;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    static constexpr int TM = WM / 32, TN = WN / 32;
    static constexpr int STAGE_BYTES = 4 * BK * (BM + BN);
    static constexpr int LDS_BYTES = KG * 2 * STAGE_BYTES;
    // the other groups' accumulators, handed to the first one at the end
    static_assert((KG - 1) * BM * BN * 8 <= LDS_BYTES, "accumulators in LDS");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "blocks");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

// Transposing 8-byte LDS read (ds_read_b64_tr_b16): in a group of 16 lanes,
// lane 4i + c receives element c of the reads of lanes i, i + 4, i + 8, i + 12.
__device__ inline half4_t read_tr(const unsigned char* p) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p)));
}

__device__ inline void split_quad(const f32x4& v, half4_t& hi, half4_t& lo) {
    mfmae::tcec::half2_t h0, l0, h1, l1;
    mfmae::tcec::split_pair(v[0], v[1], h0, l0);
    mfmae::tcec::split_pair(v[2], v[3], h1, l1);
    hi = half4_t{h0[0], h0[1], h1[0], h1[1]};
    lo = half4_t{l0[0], l0[1], l1[0], l1[1]};
}

// One operand of a tile: LINES lines by BK k per chunk, staged by a group of
// NT threads, of which this is `tid`.
template <int LINES, bool KC, int NT, bool EDGE>
struct Operand {
    static constexpr int LOADS = LINES * BK / 4 / NT;  // 16-byte loads per thread and chunk
    static constexpr int PLANE = 2 * BK * LINES;       // bytes of one binary16 plane
    static constexpr int QUADS = LINES / 4;            // quads of one k
    static constexpr int PASS = KC ? NT / 4 : NT / QUADS;  // lines (k) covered by one pass
    static_assert(LOADS * 4 * NT == LINES * BK && LOADS >= 1, "staging");
    static_assert(!KC || LOADS % 2 == 0, "K-contiguous units are two loads");
    // the swizzles repeat every 16 lines and every 4 k
    static_assert(KC ? PASS % 16 == 0 : PASS % 4 == 0, "passes keep the swizzle");

    struct Regs {
        f32x4 v[LOADS];
    };

    int tid;
    const float* base;  // first line of the tile at k = 0
    int64_t ld;
    int64_t span;       // floats from base to the operand's end
    uint32_t off;       // bytes from a chunk's corner to the thread's first load
    uint32_t edge_off[KC ? LOADS / 2 : 1];  // EDGE, K-contiguous: each unit's own
    int shift;          // EDGE, M/N-contiguous: values to drop from the thread's quads
    int lds;            // byte offset of the thread's first store in a plane

    __device__ static int swizzle(int k) { return LINES >= 128 ? 8 * (k & 3) : 8 * ((k >> 1) & 1); }
    __device__ static int piece(int r, int q) { return r * 64 + 16 * (q ^ ((r ^ (r >> 2)) & 3)); }
    __device__ static int quad(int k, int q) { return k * 2 * LINES + 8 * (q ^ swizzle(k)); }

    // p: the operand's element (line 0, k 0); the tile starts at line l0 of
    // `lines`, and there are k elements along k.
    __device__ void init(int tid_, const float* p, int64_t ld_, int l0, int lines, int k) {
        tid = tid_;
        ld = ld_;
        if constexpr (KC) {
            base = p + l0 * ld;
            span = (lines - 1 - l0) * ld + k;
            const int r = tid >> 2, q = tid & 3;
            off = (uint32_t)(r * ld + 8 * q) * 4u;
            lds = piece(r, q);
            if constexpr (EDGE) {
#pragma unroll
                for (int u = 0; u < LOADS / 2; ++u)
                    edge_off[u] =
                        (uint32_t)(min(r + u * PASS, lines - 1 - l0) * ld + 8 * q) * 4u;
            }
        } else {
            base = p + l0;
            span = (k - 1) * ld + lines - l0;
            const int kk = tid / QUADS, q = tid % QUADS;
            int c = 4 * q;
            if constexpr (EDGE) {
                c = min(c, lines - l0 - 4);  // lines >= 4
                // the quad over the edge drops the values before its own
                shift = 4 * q < lines - l0 ? 4 * q - c : 0;
            }
            off = (uint32_t)(kk * ld + c) * 4u;
            lds = quad(kk, q);
        }
    }

    // Loads of the chunk at k0.  TAIL: the descriptor ends with the operand.
    template <bool TAIL>
    __device__ void load(Regs& r, int k0) const {
        const int64_t at = KC ? k0 : k0 * ld;
        const int64_t left = span - at;  // floats; positive
        const int records =
            TAIL ? (int)(uint32_t)(left < (int64_t(1) << 30) ? 4 * left : int64_t(0xffffffff)) : -1;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(base + at), 0, records, 0x00020000);
        const uint32_t pass = (uint32_t)ld * (4u * PASS);  // bytes; under 2^31 (offsets_fit)
        if constexpr (KC) {
#pragma unroll
            for (int u = 0; u < LOADS / 2; ++u) {
                // (the scalar offset takes no part in the bounds check)
                const uint32_t o = EDGE ? edge_off[u] : TAIL ? off + pass * (uint32_t)u : off;
                const int s = EDGE || TAIL ? 0 : (int)(pass * (uint32_t)u);
                r.v[2 * u] = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, s, 0));
                r.v[2 * u + 1] = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16, s, 0));
            }
        } else {
#pragma unroll
            for (int u = 0; u < LOADS; ++u)
                r.v[u] = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                               rs, TAIL ? off + pass * (uint32_t)u : off,
                               TAIL ? 0 : (int)(pass * (uint32_t)u), 0));
        }
    }

    // Zero what lies at k >= count of the chunk.
    __device__ void mask(Regs& r, int count) const {
#pragma unroll
        for (int u = 0; u < LOADS; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int kk = KC ? 8 * (tid & 3) + 4 * (u & 1) + e : tid / QUADS + u * PASS;
                if (kk >= count) r.v[u][e] = 0.0f;
            }
    }

    // Split the chunk into its hi and lo planes at `plane`.
    __device__ void store(const Regs& r, unsigned char* plane) const {
        if constexpr (KC) {
#pragma unroll
            for (int u = 0; u < LOADS / 2; ++u) {
                const f32x4 &a = r.v[2 * u], &b = r.v[2 * u + 1];
                const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
                half8_t hi, lo;
                mfmae::tcec::split8(x, hi, lo);
                unsigned char* q = plane + lds + u * PASS * 64;
                *reinterpret_cast<half8_t*>(q) = hi;
                *reinterpret_cast<half8_t*>(q + PLANE) = lo;
            }
        } else {
#pragma unroll
            for (int u = 0; u < LOADS; ++u) {
                f32x4 v = r.v[u];
                if constexpr (EDGE) {
                    if (shift & 1) v = f32x4{v[1], v[2], v[3], v[3]};
                    if (shift & 2) v = f32x4{v[2], v[3], v[3], v[3]};
                }
                half4_t hi, lo;
                split_quad(v, hi, lo);
                unsigned char* q = plane + lds + u * PASS * 2 * LINES;
                *reinterpret_cast<half4_t*>(q) = hi;
                *reinterpret_cast<half4_t*>(q + PLANE) = lo;
            }
        }
    }

    // Operand vector of the 32 lines from `line` on, k step s (16 k), of the
    // plane: lane (j, g) holds k = 16 s + 8 g .. + 7 of line j.
    __device__ static half8_t frag(const unsigned char* plane, int line, int s) {
        const int l = threadIdx.x & 63;
        if constexpr (KC)
            return *reinterpret_cast<const half8_t*>(plane + piece(line + (l & 31), 2 * s + (l >> 5)));
        // lane 16 G + sl reads k = 8 (G / 2) + sl / 4 (+ 4 for the second
        // half) at quad 4 (G % 2) + sl % 4 of the block
        const int sl = l & 15, G = l >> 4;
        const int kl = 16 * s + 8 * (G >> 1) + (sl >> 2);
        const unsigned char* q = plane + quad(kl, (line >> 2) + 4 * (G & 1) + (sl & 3));
        const half4_t h0 = read_tr(q), h1 = read_tr(q + 4 * 2 * LINES);  // k + 4: same swizzle
        return half8_t{h0[0], h0[1], h0[2], h0[3], h1[0], h1[1], h1[2], h1[3]};
    }
};

// Barrier that orders LDS accesses only: outstanding global loads stay in
// flight across it.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class CF>
using OperandA = Operand<CF::BM, CF::A_KC, CF::GROUP, CF::EDGE>;
template <class CF>
using OperandB = Operand<CF::BN, CF::B_KC, CF::GROUP, CF::EDGE>;

template <class CF>
__device__ inline void compute(f32x16_t (&acc)[CF::TM][CF::TN], f32x16_t (&cor)[CF::TM][CF::TN],
                               const unsigned char* buf, int wrow, int wcol) {
    using OA = OperandA<CF>;
    using OB = OperandB<CF>;
    const unsigned char* a = buf;
    const unsigned char* b = buf + 2 * OA::PLANE;
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
        half8_t ahi[CF::TM], alo[CF::TM], bhi[CF::TN], blo[CF::TN];
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm) {
            ahi[tm] = OA::frag(a, wrow + 32 * tm, s);
            alo[tm] = OA::frag(a + OA::PLANE, wrow + 32 * tm, s);
        }
#pragma unroll
        for (int tn = 0; tn < CF::TN; ++tn) {
            bhi[tn] = OB::frag(b, wcol + 32 * tn, s);
            blo[tn] = OB::frag(b + OB::PLANE, wcol + 32 * tn, s);
        }
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
                acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ahi[tm], bhi[tn], acc[tm][tn],
                                                                     0, 0, 0);
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
                cor[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(alo[tm], bhi[tn], cor[tm][tn],
                                                                     0, 0, 0);
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
                cor[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ahi[tm], blo[tn], cor[tm][tn],
                                                                     0, 0, 0);
    }
}

// Ask the scheduler to interleave the chunk's MFMAs with the VALU work of
// the split, four instructions each.
template <class CF>
__device__ inline void interleave() {
#pragma unroll
    for (int i = 0; i < 3 * (BK / 16) * CF::TM * CF::TN; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
    }
}

template <bool V>
struct Bool {
    static constexpr bool value = V;
};

template <class CF>
__device__ __forceinline__ void run(const Params& p, unsigned char* smem) {
    using OA = OperandA<CF>;
    using OB = OperandB<CF>;
    const int task = xcd_task(blockIdx.x, gridDim.x);
    if (task >= p.ntasks) return;  // the whole workgroup leaves together
    const int tiles = p.tiles_m * p.tiles_n;
    const int item = task / tiles;
    const TileRC rc = grouped_tile(task - item * tiles, p.tiles_m, p.tiles_n);
    // first output of the tile's own, and first one computed
    const int m_own = rc.tm * CF::BM, n_own = rc.tn * CF::BN;
    const int m0 = max(0, min(m_own, p.m - CF::BM));
    const int n0 = max(0, min(n_own, p.n - CF::BN));
    const int64_t it = (int64_t)item + p.item0;

    OA oa;
    OB ob;
    const int gwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = gwave / (CF::WAVES_M * CF::WAVES_N);  // the wave's group
    const int wave = gwave % (CF::WAVES_M * CF::WAVES_N);
    const int tid = threadIdx.x % CF::GROUP;
    oa.init(tid, p.A + it * p.sa, p.lda, m0, p.m, p.k);
    ob.init(tid, p.B + it * p.sb, p.ldb, n0, p.n, p.k);

    const int l = threadIdx.x & 63;
    const int g = l >> 5, j = l & 31;
    const int wrow = (wave / CF::WAVES_N) * CF::WM;
    const int wcol = (wave % CF::WAVES_N) * CF::WN;

    // Whether the whole tile is the workgroup's own.  Otherwise a lane whose
    // output does not exist or belongs to another tile gets an offset past
    // the descriptor's end: its load returns zero, its store is dropped.
    const bool whole = m0 == m_own && n0 == n_own && m0 + CF::BM <= p.m && n0 + CF::BN <= p.n;
    // Calls f(tm, tn, e, lane offset, scalar offset), the bytes in C or D
    // from the wave's corner, for every accumulator element.
    auto outputs = [&](int64_t ld, auto masked, auto f) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)(4 * g * ld + j) * 4u;
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn) {
                const int row0 = m0 + wrow + 32 * tm + 4 * g, col = n0 + wcol + 32 * tn + j;
                const bool own_col = (col >= n_own) & (col < p.n);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = 8 * (e >> 2) + (e & 3);
                    const bool own = own_col & (row0 + r >= m_own) & (row0 + r < p.m);
                    f(tm, tn, e, (!decltype(masked)::value | own) ? off : kPastEnd,
                      (int)((uint32_t)((32 * tm + r) * ld + 32 * tn) * 4u));
                }
            }
    };

    f32x16_t acc[CF::TM][CF::TN], cor[CF::TM][CF::TN];
#pragma unroll
    for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < CF::TN; ++tn)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[tm][tn][e] = 0.0f;
                cor[tm][tn][e] = 0.0f;
            }
    // Chunks: the k tail, if there is one, then the whole chunks; group kg
    // takes chunks kg, kg + KG, ...
    const int tail = p.k % BK;
    const int lead = tail ? 1 : 0;
    const int nc = p.k / BK + lead;  // >= 1
    const int last = nc - 1;
    const int mine = (nc - kg + CF::KG - 1) / CF::KG;  // chunks of this group
    const int steps = (nc + CF::KG - 1) / CF::KG;      // of the first group, the most
    const int all = nc / CF::KG;                       // steps in which every group has a chunk
    // k of the group's i-th chunk (clamped; not the first chunk of all)
    auto k_of = [&](int i) { return BK * (min(i * CF::KG + kg, last) - lead); };
    typename OA::Regs a0, a1;
    typename OB::Regs b0, b1;
    const int kfirst = min(kg, last) > 0 ? k_of(0) : tail ? p.k - tail : 0;
    const int ksecond = last > 0 ? k_of(1) : kfirst;
    oa.template load<true>(a0, kfirst);
    ob.template load<true>(b0, kfirst);
    oa.template load<true>(a1, ksecond);
    ob.template load<true>(b1, ksecond);
    if (tail && kg == 0) {
        oa.mask(a0, tail);
        ob.mask(b0, tail);
    }
    unsigned char* buf0 = smem + kg * 2 * CF::STAGE_BYTES;
    unsigned char* buf1 = buf0 + CF::STAGE_BYTES;
    auto store = [&](const typename OA::Regs& a, const typename OB::Regs& b, unsigned char* buf)
                     __attribute__((always_inline)) {
        oa.store(a, buf);
        ob.store(b, buf + 2 * OA::PLANE);
    };
    auto load = [&](typename OA::Regs& a, typename OB::Regs& b, int i)
                    __attribute__((always_inline)) {
        oa.template load<false>(a, k_of(i));
        ob.template load<false>(b, k_of(i));
    };
    store(a0, b0, buf0);
    if (steps == 1) {  // nothing past the first chunk
        lds_barrier();
        if (mine > 0) compute<CF>(acc, cor, buf0, wrow, wcol);
    } else {
        load(a0, b0, 2);
        lds_barrier();
        // step i: chunk i is in LDS, i + 1 and i + 2 in registers or in flight
        int i = 0;
        for (; i + 2 <= all; i += 2) {
            compute<CF>(acc, cor, buf0, wrow, wcol);
            store(a1, b1, buf1);
            load(a1, b1, i + 3);
            interleave<CF>();
            lds_barrier();
            compute<CF>(acc, cor, buf1, wrow, wcol);
            store(a0, b0, buf0);
            load(a0, b0, i + 4);
            interleave<CF>();
            lds_barrier();
        }
        // at most two more steps, the second one not for every group
        if (i < mine) compute<CF>(acc, cor, buf0, wrow, wcol);
        if (i + 1 < steps) {
            store(a1, b1, buf1);
            lds_barrier();
            if (i + 1 < mine) compute<CF>(acc, cor, buf1, wrow, wcol);
        }
    }

    // The groups' sums, main and correction apart, added up by the first
    // group, in the order of the groups.
    if constexpr (CF::KG > 1) {
        constexpr int VECS = CF::TM * CF::TN * 8;  // 16-byte pieces per thread
        f32x4* sums = reinterpret_cast<f32x4*>(smem);
        auto piece = [&](int group, int v) -> f32x4& {
            return sums[((group - 1) * VECS + v) * CF::GROUP + tid];
        };
        lds_barrier();  // the stages are read
        if (kg > 0) {
#pragma unroll
            for (int v = 0; v < VECS; ++v) {
                const int b = v >> 3, e = 4 * (v & 3);
                const f32x16_t& x = v & 4 ? cor[b / CF::TN][b % CF::TN] : acc[b / CF::TN][b % CF::TN];
                piece(kg, v) = f32x4{x[e], x[e + 1], x[e + 2], x[e + 3]};
            }
        }
        lds_barrier();
        if (kg > 0) return;
#pragma unroll
        for (int o = 1; o < CF::KG; ++o)
#pragma unroll
            for (int v = 0; v < VECS; ++v) {
                const int b = v >> 3, e = 4 * (v & 3);
                f32x16_t& x = v & 4 ? cor[b / CF::TN][b % CF::TN] : acc[b / CF::TN][b % CF::TN];
                const f32x4 y = piece(o, v);
#pragma unroll
                for (int t = 0; t < 4; ++t) x[e + t] += y[t];
            }
    }

    // main + C + corr * 2^-11, C in the registers the staged chunks have left.
    // (C in the accumulators from the start spilled 50 registers per lane:
    // 4096 x 128^3 with 128 x 128 tiles 225 us against 189, 1024 x 256^3
    // 268 / 209.)  The rounding error of main + C joins the correction, so
    // that the result is rounded once, as when C starts the main sum.
    if (CF::ADD && p.C) {
        __builtin_amdgcn_sched_barrier(0);  // not ahead of the groups' sums
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(p.C + it * p.sc + (int64_t)(m0 + wrow) * p.ldc + n0 + wcol), 0,
            (int)kPastEnd, 0x00020000);
        f32x16_t add[CF::TM][CF::TN];
        auto get = [&](int tm, int tn, int e, uint32_t v, int s) __attribute__((always_inline)) {
            add[tm][tn][e] =
                __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rc, v, s, 0));
        };
        if (whole) outputs(p.ldc, Bool<false>{}, get);
        else outputs(p.ldc, Bool<true>{}, get);
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    // two-sum (Knuth): a + c = s + err exactly, except where
                    // a step overflows
                    const float a = acc[tm][tn][e], c = add[tm][tn][e];
                    const float s = a + c, t = s - a;
                    const float err = (a - (s - t)) + (c - t);
                    acc[tm][tn][e] =
                        s + __builtin_fmaf(cor[tm][tn][e], mfmae::tcec::kLoScaleInv,
                                           __builtin_isfinite(err) ? err : 0.0f);
                }
    } else {
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    acc[tm][tn][e] =
                        __builtin_fmaf(cor[tm][tn][e], mfmae::tcec::kLoScaleInv, acc[tm][tn][e]);
    }

    // D is not read again here: where the tile's rows are whole 128-byte lines
    // it is stored nontemporally (4096 x 128^3 158 against 166 us, 1024 x 256^3
    // 174 / 192).  Otherwise the pieces of a line meet in the L2 (8 x 1001 x 999
    // x 1003 64 against 56 us, 174 x 651 x 2213 x 128 611 / 488).
    float* const Di = p.D + it * p.sd + (int64_t)(m0 + wrow) * p.ldd + n0 + wcol;
    if constexpr (CF::FAR) {
#pragma unroll
        for (int tm = 0; tm < CF::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < CF::TN; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = 32 * tm + 4 * g + 8 * (e >> 2) + (e & 3), c = 32 * tn + j;
                    const int row = m0 + wrow + r, col = n0 + wcol + c;
                    if ((col >= n_own) & (col < p.n) & (row >= m_own) & (row < p.m))
                        Di[r * p.ldd + c] = acc[tm][tn][e];
                }
        return;
    }
    const __amdgpu_buffer_rsrc_t rd =
        __builtin_amdgcn_make_buffer_rsrc(Di, 0, (int)kPastEnd, 0x00020000);
    const bool lines = ((uintptr_t)Di % 128 == 0) & (p.ldd % 32 == 0);
    auto put = [&](auto nontemporal) __attribute__((always_inline)) {
        return [&](int tm, int tn, int e, uint32_t v, int s) __attribute__((always_inline)) {
            const float d = acc[tm][tn][e];
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, d), rd, v, s,
                                                  decltype(nontemporal)::value ? kNontemporal : 0);
        };
    };
    if (whole & lines) outputs(p.ldd, Bool<false>{}, put(Bool<true>{}));
    else if (whole) outputs(p.ldd, Bool<false>{}, put(Bool<false>{}));
    else outputs(p.ldd, Bool<true>{}, put(Bool<false>{}));
}

// Whether the byte offsets of an operand of `lines` lines per tile stay below
// 2^31, so that no buffer offset depends on how the hardware treats the top
// bit of a 32-bit offset.
inline bool offsets_fit(bool kc, int lines, int64_t ld) {
    return (kc ? (lines * ld + BK) * 4 : (BK * ld + lines) * 4) < (int64_t)kPastEnd;
}

}  // namespace tile
}  // namespace sgemm_emu
