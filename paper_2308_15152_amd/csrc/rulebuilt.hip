// Batched products with a rule-built left operand, n = 64, in emulated FP32
// (Sec. 4.4).  The 64 x 64 left matrix is never read from memory: its MFMA
// A-operand fragments are built in registers from a rule.
//
//   Householder (Sec. 4.2.1, eq. householder; foreach_ij of Sec. 4.2):
//     C = (I - 2 u u^T) B.  For every A-operand element it holds, a lane
//     evaluates h_ij = fmaf(-2 u_i, u_j, delta_ij) and splits it into hi/lo.
//     Per 16-wide k step one foreach_ij over the A-operand map fills both
//     32-row blocks (the index computation is shared by the two fragments,
//     and -2 u_i of the lane's rows is computed once), which is what keeps
//     rule-built fragments cheaper than a trip through memory.  The baseline
//     forms every entry once into LDS and loads the fragments from there.
//   Givens (Sec. 4.3.1; map of Sec. 4.3):
//     C = G(i, j, theta) B with G the identity except G_ii = G_jj = c,
//     G_ij = -s, G_ji = s.  With (i, j) embedded at compile time the fragments
//     are filled with zeros and the nonzero entries are set through map():
//     (row, col) -> (lane, element), which folds to constants.  With (i, j)
//     kernel arguments each lane asks instead which words of the two rows it
//     holds take an entry (a compare and a select per word; map() at run time
//     took a select per element of every entry).  The baseline writes G to LDS
//     and loads the fragments from there.
//
// One wavefront handles one batch item and up to 64 columns of B, in two
// 32-column blocks, or in one if at most 32 columns are left (CB): products of
// few columns are bound by the vector instructions of building the left
// operand and of splitting B, not by HBM traffic (B read once, C written once)
// as those of 64 are.  262,144 items with 24 columns: 1100 us with two blocks,
// half empty, and one value split at a time.
// B is read straight from global memory into the B-operand registers.  When
// rows allow 8-byte accesses the two 32-column blocks interleave their
// columns, so for a fixed k the 32 lanes of a half-wave read one 256-byte row
// segment with one 8-byte load each (and C is written the same way); otherwise
// lane l holds column l % 32 of each block (128-byte segments).  Loads and
// stores are buffer accesses on the item's corner: a scalar row offset and a
// lane offset, which for a lane without a column lies past the descriptor's
// end (its loads return zero, its stores are dropped).  Row pitches of 2^22
// floats and more, which 32-bit offsets don't reach, take 64-bit pointers (FAR,
// up to the 2^27 floats of B that the entry points take; 20,000 items side by
// side in such rows of B, 32 / 64 / 94 / 65 columns 67 / 133 / 214 / 191 us, two
// blocks of single columns for all 89 / 136 / 231 / 191).
#include "internal.h"
#include "mfmae/frag.hpp"
#include "mfmae/tcec.hpp"
#include "sgemm_emu.h"
#include "tiling.hpp"

namespace sgemm_emu {

using mfmae::f32x16_t;
using mfmae::half8_t;
using mfmae::Shape32;
using mfmae::Use;

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
using FragA = mfmae::fragment<Shape32, Use::A, _Float16>;

struct RuleParams {
    int ncols;
    // Householder: u_b = u + b su (64 values)
    const float* u;
    int64_t su;
    // Givens: c_b = c[b scs], s_b = s[b scs]; rotation plane (gi, gj)
    const float* c;
    const float* s;
    int64_t scs;
    int gi, gj;
    const float* B;
    int64_t ldb, sb;
    float* C;
    int64_t ldc, sc;
    int batch;      // items of this launch
    int64_t item0;  // first item of this launch
};

constexpr int kWaves = 4;  // waves (tasks) per workgroup

// ---------------------------------------------------------------------------
// Left-operand builders.  build(s, hh, hl) produces the hi and lo fragments
// of rows 32 tm .. 32 tm + 31, columns (k) 16 s .. 16 s + 15 of the 64 x 64
// left matrix, for tm = 0, 1.
// ---------------------------------------------------------------------------

struct HouseholderRule {
    // u arrives in one coalesced load, u_l in lane l; the entries the map
    // asks for are read from the lane that holds them (cross-lane reads, no
    // memory access), so building H adds no vector-memory instructions
    float ulane;
    float urow[2];  // -2 u_i of the lane's row in each 32-row block

    __device__ void init(const RuleParams& p, int64_t item, unsigned char*) {
        ulane = p.u[item * p.su + (threadIdx.x & 63)];
        mfmae::foreach_ij<FragA>([&](int e, int i, int) {
            if (e == 0) {
                urow[0] = -2.0f * __shfl(ulane, i);
                urow[1] = -2.0f * __shfl(ulane, 32 + i);
            }
        });
    }

    __device__ void build(int s, half8_t (&hh)[2], half8_t (&hl)[2]) const {
        float h[2][8];
        mfmae::foreach_ij<FragA>([&](int e, int i, int jj) {
            const int gj = 16 * s + jj;
            const float uj = __shfl(ulane, gj);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                // the diagonal crosses block tm in its own two k steps only
                const float delta = s >> 1 == tm && 32 * tm + i == gj ? 1.0f : 0.0f;
                h[tm][e] = mfmae::tcec::as_fp32(__builtin_fmaf(urow[tm], uj, delta));
            }
        });
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) mfmae::tcec::split8(h[tm], hh[tm], hl[tm]);
    }
};

// Set element (r, q) of the 64 x 64 matrix held as fragments f[tm] (rows
// 32 tm .., columns 16 s ..) to v, if it falls in k step s: the lane that
// map() names writes element `elem` of fragment r / 32.  With r and q
// compile-time constants every test folds away but the lane compare.
__device__ inline void set_entry(FragA (&f)[2], int s, int r, int q, _Float16 v) {
    if ((q >> 4) != s) return;
    int lane, elem;
    mfmae::map<FragA>(lane, elem, r & 31, q & 15);
    if ((int)(threadIdx.x & 63) != lane) return;
    const int tm = r >> 5;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < FragA::num_elements; ++e)
            if (t == tm && e == elem) f[t].x[e] = v;
}

// Givens rotation through map(), the plane (I, J) a compile-time constant.
template <int I, int J>
struct GivensMapRule {
    static constexpr int gi = I, gj = J;
    _Float16 ch, cl, sh, sl, nsh, nsl;  // hi/lo of c, s and -s

    __device__ void init(const RuleParams& p, int64_t item, unsigned char*) {
        const float c = p.c[item * p.scs];
        const float s = p.s[item * p.scs];
        mfmae::tcec::split(c, ch, cl);
        mfmae::tcec::split(s, sh, sl);
        mfmae::tcec::split(-s, nsh, nsl);
    }

    __device__ void build(int s, half8_t (&hh)[2], half8_t (&hl)[2]) const {
        FragA fh[2], fl[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            mfmae::fill(fh[t], (_Float16)0.0f);
            mfmae::fill(fl[t], (_Float16)0.0f);
        }
        // ones on the part of the diagonal in this k step (hi 1, lo 0)
#pragma unroll
        for (int d = 0; d < 16; ++d) set_entry(fh, s, 16 * s + d, 16 * s + d, (_Float16)1.0f);
        // the rotation entries (c overrides the diagonal one)
        set_entry(fh, s, gi, gi, ch);
        set_entry(fl, s, gi, gi, cl);
        set_entry(fh, s, gj, gj, ch);
        set_entry(fl, s, gj, gj, cl);
        set_entry(fh, s, gi, gj, nsh);
        set_entry(fl, s, gi, gj, nsl);
        set_entry(fh, s, gj, gi, sh);
        set_entry(fl, s, gj, gi, sl);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            hh[t] = mfmae::pack(fh[t]);
            hl[t] = mfmae::pack(fl[t]);
        }
    }
};

// Givens rotation with the plane as kernel arguments.  Where map() would find
// the lane and element of each nonzero entry, a lane asks the same of the two
// rows it holds (r = 32 tm + l % 32): the diagonal entry, 1 or c, and in rows
// i and j one more, -s or s.  An operand row is 32 words of two halves, word
// 8 s + 4 (l / 32) + w in the lane's registers of k step s, so placing an
// entry is one compare and one select per word: 560 vector instructions per
// wave with 64 columns, 1270 with a select per element of every entry.
struct GivensArgRule {
    uint32_t diag[2], diag_lo[2];  // the entry's hi and lo, in their half of the word
    uint32_t off[2], off_lo[2];
    int diag_word[2], off_word[2];  // the word of the row that holds it

    __device__ void init(const RuleParams& p, int64_t item, unsigned char*) {
        const float c = p.c[item * p.scs];
        const float s = p.s[item * p.scs];
        const int l = threadIdx.x & 63;
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const int r = 32 * tm + (l & 31);
            const bool in_i = r == p.gi, in_j = r == p.gj;
            put(in_i || in_j ? c : 1.0f, r, diag[tm], diag_lo[tm], diag_word[tm]);
            put(in_i ? -s : in_j ? s : 0.0f, in_i ? p.gj : p.gi, off[tm], off_lo[tm],
                off_word[tm]);
            if (!in_i && !in_j) off_word[tm] = -1;
        }
    }

    __device__ static void put(float v, int col, uint32_t& hi, uint32_t& lo, int& word) {
        _Float16 h, x;
        mfmae::tcec::split(v, h, x);
        hi = (uint32_t)__builtin_bit_cast(uint16_t, h) << (16 * (col & 1));
        lo = (uint32_t)__builtin_bit_cast(uint16_t, x) << (16 * (col & 1));
        word = col >> 1;
    }

    __device__ void build(int s, half8_t (&hh)[2], half8_t (&hl)[2]) const {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const int first = 8 * s + 4 * ((threadIdx.x & 63) >> 5);
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            u32x4 h, x;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const bool o = off_word[tm] == first + w;
                h[w] = o ? off[tm] : 0u;
                x[w] = o ? off_lo[tm] : 0u;
                if (s >> 1 == tm) {
                    const bool d = diag_word[tm] == first + w;
                    h[w] |= d ? diag[tm] : 0u;
                    x[w] |= d ? diag_lo[tm] : 0u;
                }
            }
            hh[tm] = __builtin_bit_cast(half8_t, h);
            hl[tm] = __builtin_bit_cast(half8_t, x);
        }
    }
};

// Baselines: the left matrix is written to the wave's own 16 KiB of LDS
// (hi and lo planes) and the fragments are loaded from there, as a fragment
// API without rule-built fragments requires.  Rows of 64 halves (128 bytes,
// 8 pieces of 8 halves); piece p of row r is stored at position
// p ^ ((r ^ (r >> 3)) & 7), so that the 32 rows a fragment load touches
// spread over all banks.
struct LdsOperand {
    unsigned char* hi;  // [64 rows][128 bytes]
    unsigned char* lo;

    __device__ static int off(int r, int p) { return r * 128 + 16 * (p ^ ((r ^ (r >> 3)) & 7)); }

    __device__ void bind(unsigned char* lds) {
        hi = lds;
        lo = lds + 64 * 128;
    }

    __device__ void build(int s, half8_t (&hh)[2], half8_t (&hl)[2]) const {
        const int l = threadIdx.x & 63;
        const int p = 2 * s + (l >> 5);  // k = 16 s + 8 (l / 32) + e
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const int o = off(32 * tm + (l & 31), p);
            hh[tm] = *reinterpret_cast<const half8_t*>(hi + o);
            hl[tm] = *reinterpret_cast<const half8_t*>(lo + o);
        }
    }
};

// Givens baseline: zero both planes, then lane r writes G_rr (c at i and j,
// else 1) and lanes 0 and 1 the two off-diagonal entries.
struct GivensLdsRule : LdsOperand {
    __device__ void init(const RuleParams& p, int64_t item, unsigned char* lds) {
        const int l = threadIdx.x & 63;
        bind(lds);
        const float c = p.c[item * p.scs];
        const float s = p.s[item * p.scs];
        // zero both planes: 64 rows x 8 pieces, 8 pieces per lane
        const half8_t z = {};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int piece = 64 * t + l;
            *reinterpret_cast<half8_t*>(hi + off(piece >> 3, piece & 7)) = z;
            *reinterpret_cast<half8_t*>(lo + off(piece >> 3, piece & 7)) = z;
        }
        // A wave's LDS accesses complete in the order they are issued; the
        // fences keep the compiler from reordering the zeros, these entries
        // and the loads in build().
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        auto put = [&](int r, int q, float v) {
            _Float16 vh, vl;
            mfmae::tcec::split(v, vh, vl);
            const int o = off(r, q >> 3) + 2 * (q & 7);
            *reinterpret_cast<_Float16*>(hi + o) = vh;
            *reinterpret_cast<_Float16*>(lo + o) = vl;
        };
        put(l, l, (l == p.gi || l == p.gj) ? c : 1.0f);
        if (l == 0) put(p.gi, p.gj, -s);
        if (l == 1) put(p.gj, p.gi, s);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
};

// Householder baseline: every entry h_ij = fmaf(-2 u_i, u_j, delta_ij) is
// formed once, split, and written to LDS; lane l forms 8 pieces of 8
// entries (rows (64 t + l) / 8, t = 0..7).
struct HouseholderLdsRule : LdsOperand {
    __device__ void init(const RuleParams& p, int64_t item, unsigned char* lds) {
        const int l = threadIdx.x & 63;
        bind(lds);
        // u as in the register-built rule: one coalesced load, entries read
        // from the lane that holds them
        const float ulane = p.u[item * p.su + l];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int piece = 64 * t + l;
            const int r = piece >> 3, q0 = 8 * (piece & 7);
            const float ur = -2.0f * __shfl(ulane, r);
            float h[8];
#pragma unroll
            for (int v = 0; v < 8; ++v)
                h[v] = mfmae::tcec::as_fp32(
                    __builtin_fmaf(ur, __shfl(ulane, q0 + v), (r == q0 + v) ? 1.0f : 0.0f));
            half8_t vh, vl;
            mfmae::tcec::split8(h, vh, vl);
            *reinterpret_cast<half8_t*>(hi + off(r, piece & 7)) = vh;
            *reinterpret_cast<half8_t*>(lo + off(r, piece & 7)) = vl;
        }
        // the fragment loads in build() read what other lanes wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
};

// ---------------------------------------------------------------------------
// The common body: one wave = one item and one group of up to 32 CB columns.
// PAIR: the two 32-column blocks interleave their columns (column j of
// block cb is c0 + 2 j + cb), so one 8-byte load of a B row and one 8-byte
// store of a C row serve both blocks (buffer accesses: 4-byte alignment is
// enough); needs an even number of columns.  Otherwise block cb holds columns
// c0 + 32 cb + j.
// ---------------------------------------------------------------------------
constexpr uint32_t kPastEnd = 0x80000000;  // no buffer offset in use reaches this

typedef f32x2 far_x2 __attribute__((aligned(4)));  // a pair in rows of any alignment

// One B or C item from column c0 on: rows ld apart, the lane's first column
// (and, PAIR, its neighbour) or both of its columns.
template <int CB, bool PAIR, bool FAR, int STREAM>
struct Rows {
    // cache policies: nontemporal, as neither B nor C is touched twice here
    static constexpr int kLoad = STREAM == 2 ? 2 : 0, kStore = STREAM ? 2 : 0;

    float* p;
    int64_t ld;
    uint32_t off[CB];  // bytes from the item's corner to (lane row, column)
    int64_t far[CB];   // FAR: the same in floats
    bool ok[CB];

    // The lane's rows are `row` and what a scalar row offset adds to it.
    __device__ void init(float* base, int64_t ld_, int row, int ncols) {
        p = base;
        ld = ld_;
        const int j = threadIdx.x & 31;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int col = PAIR ? 2 * j : 32 * cb + j;
            ok[cb] = col < ncols;
            // a lane without a column reads the last one (and stores nothing),
            // without a branch; with two single columns a test per load is faster
            if constexpr (FAR) far[cb] = row * ld + (ok[cb] ? col : ncols - (PAIR ? 2 : 1));
            else off[cb] = ok[cb] ? (uint32_t)(row * ld + col) * 4u : kPastEnd;
        }
    }

    __device__ __amdgpu_buffer_rsrc_t rsrc() const {
        return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)kPastEnd, 0x00020000);
    }

    __device__ void load(int row, float (&x)[CB]) const {
        const int s = (int)((uint32_t)ld * 4u * (uint32_t)row);
        if constexpr (FAR) {
#pragma unroll
            for (int cb = 0; cb < CB; cb += PAIR ? 2 : 1) {
                const float* q = (p + row * ld) + far[cb];
                if constexpr (PAIR) {
                    const far_x2 v = *reinterpret_cast<const far_x2*>(q);
                    x[0] = v[0];
                    x[1] = v[1];
                } else {
                    x[cb] = CB == 1 || ok[cb] ? *q : 0.0f;
                }
            }
        } else if constexpr (PAIR) {
            const f32x2 v = __builtin_bit_cast(
                f32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc(), off[0], s, kLoad));
            x[0] = v[0];
            x[1] = v[1];
        } else {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                x[cb] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rsrc(), off[cb], s, kLoad));
        }
    }

    __device__ void store(int row, const float (&x)[CB]) const {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const int s = (int)((uint32_t)ld * 4u * (uint32_t)row);
        if constexpr (FAR) {
#pragma unroll
            for (int cb = 0; cb < CB; cb += PAIR ? 2 : 1) {
                float* q = (p + row * ld) + far[cb];
                if (!ok[cb]) continue;
                if constexpr (PAIR) *reinterpret_cast<far_x2*>(q) = far_x2{x[0], x[1]};
                else *q = x[cb];
            }
        } else if constexpr (PAIR) {
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, f32x2{x[0], x[1]}),
                                                  rsrc(), off[0], s, kStore);
        } else {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x[cb]), rsrc(),
                                                      off[cb], s, kStore);
        }
    }
};

// AHEAD: see below.
template <class Rule, int CB, bool PAIR, bool FAR, int STREAM, bool AHEAD = CB == 1>
__device__ __forceinline__ void rule64_group(const RuleParams& p, const Rule& rule, int64_t item,
                                             int c0) {
    const int l = threadIdx.x & 63;
    Rows<CB, PAIR, FAR, STREAM> B, C;
    // operand rows 8 (l / 32) + .., accumulator rows 4 (l / 32) + ..
    B.init(const_cast<float*>(p.B + item * p.sb + c0), p.ldb, 8 * (l >> 5), p.ncols - c0);
    C.init(p.C + item * p.sc + c0, p.ldc, 4 * (l >> 5), p.ncols - c0);

    // B of the whole group: lane l holds rows 16 s + 8 (l / 32) + e of k step s.
    // With one block (AHEAD) all of it goes out ahead of the products (the
    // scheduling barrier keeps it there: 262,144 items of 24 columns 585 us
    // against 621); with two the scheduler's order, one k step at a time, is the
    // better one (64 columns 1536 us against 1663), and for a last group of one
    // block beside waves with two (32,336 items of 95 columns 309 against 369).
    float x[4][CB][8];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v[CB];
            B.load(16 * s + e, v);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) x[s][cb][e] = v[cb];
        }
    if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);

    f32x16_t acc[2][CB], cor[2][CB];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        half8_t bh[CB], bl[CB], hh[2], hl[2];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) mfmae::tcec::split8(x[s][cb], bh[cb], bl[cb]);
        rule.build(s, hh, hl);
        const f32x16_t zero = {};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                acc[tm][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                    hh[tm], bh[cb], s == 0 ? zero : acc[tm][cb], 0, 0, 0);
                cor[tm][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                    hl[tm], bh[cb], s == 0 ? zero : cor[tm][cb], 0, 0, 0);
                cor[tm][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hh[tm], bl[cb], cor[tm][cb],
                                                                     0, 0, 0);
            }
    }

    // C = main + corr * 2^-11; element e of a block is row
    // 8 (e / 4) + 4 (l / 32) + e % 4 of it.
#pragma unroll
    for (int tm = 0; tm < 2; ++tm)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            float v[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                v[cb] = __builtin_fmaf(cor[tm][cb][e], mfmae::tcec::kLoScaleInv, acc[tm][cb][e]);
            C.store(32 * tm + 8 * (e >> 2) + (e & 3), v);
        }
}

// The workgroup's place in the batch: 32 consecutive ones on each XCD of every
// 256 dispatched together (in order where no whole 256 are left).
__device__ inline int xcd_blocks(int b, int G) {
    return (b | 255) < G ? (b & ~255) + (b & 7) * 32 + ((b & 255) >> 3) : b;
}

// CB: 32-column blocks of a wave's group.  A last group of up to 32 columns
// takes one block, unless its rows are read in pairs: those pieces of B and C
// lines are best moved in the same step as their neighbours (32,680 items of
// 94 columns 306 us, with one block 441).
template <class Rule, int CB, bool PAIR, bool FAR, int STREAM>
__device__ __forceinline__ void rule64_body(const RuleParams& p, unsigned char* lds) {
    // wave index as a wave-uniform (scalar) value, so that the per-item base
    // pointers live in SGPRs
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Every XCD takes one contiguous range of the batch, or, with one block, 32
    // workgroups in a row of every 256: 64 columns 1491 against 1536 us in
    // dispatch order (1426 with streaming stores, 1387 with streaming loads
    // too), 40,000 items of 444 columns 1690 / 1974, 24 columns 574 / 585.
    const int wg = CB == 1 ? xcd_blocks(blockIdx.x, gridDim.x) : xcd_task(blockIdx.x, gridDim.x);
    const int64_t task = (int64_t)wg * kWaves + wave;
    const int ngroups = (p.ncols + 32 * CB - 1) / (32 * CB);
    const int64_t local = task / ngroups;
    const int c0 = (int)(task - local * ngroups) * 32 * CB;
    if (local >= p.batch) return;  // whole wave; the kernels have no barrier
    const int64_t item = local + p.item0;
    Rule rule;
    rule.init(p, item, lds);
    if (CB > 1 && !PAIR && p.ncols - c0 <= 32)
        rule64_group<Rule, 1, false, FAR, STREAM, false>(p, rule, item, c0);
    else rule64_group<Rule, CB, PAIR, FAR, STREAM>(p, rule, item, c0);
}

// One block per wave leaves registers for four waves per SIMD.
template <int CB, bool PAIR, bool FAR, int STREAM>
__global__ __launch_bounds__(64 * kWaves, CB == 1 ? 4 : 2) void householder64_kernel(RuleParams p) {
    rule64_body<HouseholderRule, CB, PAIR, FAR, STREAM>(p, nullptr);
}

template <int CB, bool PAIR, bool FAR, int STREAM>
__global__ __launch_bounds__(64 * kWaves, 2) void householder64_lds_kernel(RuleParams p) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kWaves][2 * 64 * 128];
    rule64_body<HouseholderLdsRule, CB, PAIR, FAR, STREAM>(p, lds[threadIdx.x >> 6]);
}

template <class Rule, int CB, bool PAIR, bool FAR, int STREAM>
__global__ __launch_bounds__(64 * kWaves, CB == 1 ? 4 : 2) void givens64_kernel(RuleParams p) {
    rule64_body<Rule, CB, PAIR, FAR, STREAM>(p, nullptr);
}

template <int CB, bool PAIR, bool FAR, int STREAM>
__global__ __launch_bounds__(64 * kWaves, 2) void givens64_lds_kernel(RuleParams p) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kWaves][2 * 64 * 128];
    rule64_body<GivensLdsRule, CB, PAIR, FAR, STREAM>(p, lds[threadIdx.x >> 6]);
}

// Launch `kernel` over the batch in pieces below 2^31 work-items (the
// dispatch packet counts work-items in 32 bits).
template <class K>
hipError_t launch_rule(K kernel, int cols, RuleParams p, int64_t batch, hipStream_t stream) {
    const int64_t ngroups = (p.ncols + cols - 1) / cols;
    const int64_t max_blocks = (int64_t(1) << 31) / (64 * kWaves) - 1;
    const int64_t items_per_launch = max_blocks * kWaves / ngroups;
    if (items_per_launch == 0) return hipErrorInvalidConfiguration;
    for (int64_t i0 = 0; i0 < batch; i0 += items_per_launch) {
        const int64_t items = batch - i0 < items_per_launch ? batch - i0 : items_per_launch;
        p.batch = (int)items;
        p.item0 = i0;
        const int64_t blocks = (items * ngroups + kWaves - 1) / kWaves;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * kWaves), 0, stream, p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Byte offsets of 64 rows and 64 columns below kPastEnd.
bool near(const RuleParams& p) { return p.ldb < (1 << 22) && p.ldc < (1 << 22); }

// Bytes of B and C.
double bytes(const RuleParams& p, int64_t batch) {
    return 256.0 * p.ncols * (batch + (p.sb ? batch : 1));
}

// What of B and C is streamed past the caches where their rows are whole
// 128-byte lines (otherwise the pieces of a line meet there: 40,000 items of 444
// columns 1690 us against 2263 streamed).  2: loads and stores; 1: the stores
// alone, from 96 MB to the 256 MiB of the last-level cache, which may hold B from
// the kernel that wrote it.  Reflectors of 256 columns, streamed / stores streamed
// / nothing streamed, B in the cache: 88 MB 14.4 / 14.7 / 17.9 us (rotations 13.0 /
// 14.9 / 18.7), 96 MB 16.8 / 15.5 / 18.7, 160 MB 29.7 / 24.5 / 29.4; B not there:
// 88 MB 19.8 / 20.6 / 23.8, 160 MB 32.2 / 32.8 / 36.9; 64 columns, 320 MB 62 / - / 71.
int streams(const RuleParams& p, int64_t batch) {
    const bool lines = ((uintptr_t)p.B % 128 == 0) && ((uintptr_t)p.C % 128 == 0) &&
                       p.ldb % 32 == 0 && p.ldc % 32 == 0 && p.sb % 32 == 0 && p.sc % 32 == 0 &&
                       p.ncols % 32 == 0;
    const double size = bytes(p, batch);
    return !lines ? 0 : size >= 96e6 && size <= double(1 << 28) ? 1 : 2;
}

// Whether the columns of an even number are read in pairs: not where the
// second group of 65 to 96 columns, half empty in pairs, comes from the caches
// (614 items of 80 columns, 24 MB, 7.3 us against 8.0 in pairs; 1228 items,
// 48 MB, 12.5 / 12.3).
bool pairs(const RuleParams& p, int64_t batch) {
    return p.ncols % 2 == 0 && !(p.ncols > 64 && p.ncols <= 96 && bytes(p, batch) <= 40e6);
}

// Launches KERNEL(CB, PAIR, FAR, STREAM), a kernel instance, by shape and
// strides.
#define SGEMM_EMU_RULE_LAUNCH(KERNEL)                                                             \
    (!near(p)                 ? SGEMM_EMU_RULE_FAR(KERNEL)                                        \
     : p.ncols <= 32          ? launch_rule(KERNEL(1, false, false, 0), 32, p, batch, stream)     \
     : streams(p, batch) == 2 ? launch_rule(KERNEL(2, true, false, 2), 64, p, batch, stream)      \
     : streams(p, batch) == 1 ? launch_rule(KERNEL(2, true, false, 1), 64, p, batch, stream)      \
     : pairs(p, batch)        ? launch_rule(KERNEL(2, true, false, 0), 64, p, batch, stream)      \
                              : launch_rule(KERNEL(2, false, false, 0), 64, p, batch, stream))
#define SGEMM_EMU_RULE_FAR(KERNEL)                                                                \
    (p.ncols <= 32            ? launch_rule(KERNEL(1, false, true, 0), 32, p, batch, stream)      \
     : p.ncols % 2 == 0       ? launch_rule(KERNEL(2, true, true, 0), 64, p, batch, stream)       \
                              : launch_rule(KERNEL(2, false, true, 0), 64, p, batch, stream))

// The rotation planes (i, j) with a compile-time instance of the Givens
// kernel.
#define SGEMM_EMU_GIVENS_PLANES(X) X(5, 37) X(37, 5) X(0, 1) X(31, 32) X(62, 63)

template <class Rule>
hipError_t launch_givens(const RuleParams& p, int64_t batch, hipStream_t stream) {
#define SGEMM_EMU_KERNEL(CB, PAIR, FAR, STREAM) givens64_kernel<Rule, CB, PAIR, FAR, STREAM>
    return SGEMM_EMU_RULE_LAUNCH(SGEMM_EMU_KERNEL);
#undef SGEMM_EMU_KERNEL
}

}  // namespace

bool givens_embedded(int i, int j) {
#define SGEMM_EMU_GIVENS_TEST(I, J) \
    if (i == I && j == J) return true;
    SGEMM_EMU_GIVENS_PLANES(SGEMM_EMU_GIVENS_TEST)
#undef SGEMM_EMU_GIVENS_TEST
    return false;
}

hipError_t launch_householder64(const HouseholderArgs& a, hipStream_t stream) {
    RuleParams p{};
    p.ncols = a.ncols;
    p.u = a.u;
    p.su = a.su;
    p.B = a.B;
    p.ldb = a.ldb;
    p.sb = a.sb;
    p.C = a.C;
    p.ldc = a.ldc;
    p.sc = a.sc;
    const int64_t batch = a.batch;
#define SGEMM_EMU_KERNEL(CB, PAIR, FAR, STREAM) householder64_kernel<CB, PAIR, FAR, STREAM>
#define SGEMM_EMU_LDS_KERNEL(CB, PAIR, FAR, STREAM) householder64_lds_kernel<CB, PAIR, FAR, STREAM>
    if (a.mode == SGEMM_EMU_HOUSEHOLDER_LDS) return SGEMM_EMU_RULE_LAUNCH(SGEMM_EMU_LDS_KERNEL);
    return SGEMM_EMU_RULE_LAUNCH(SGEMM_EMU_KERNEL);
#undef SGEMM_EMU_KERNEL
#undef SGEMM_EMU_LDS_KERNEL
}

hipError_t launch_givens64(const GivensArgs& a, hipStream_t stream) {
    RuleParams p{};
    p.ncols = a.ncols;
    p.c = a.c;
    p.s = a.s;
    p.scs = a.scs;
    p.gi = a.i;
    p.gj = a.j;
    p.B = a.B;
    p.ldb = a.ldb;
    p.sb = a.sb;
    p.C = a.C;
    p.ldc = a.ldc;
    p.sc = a.sc;
    const int64_t batch = a.batch;
    if (a.mode == SGEMM_EMU_GIVENS_EMBEDDED) {
#define SGEMM_EMU_GIVENS_CASE(I, J) \
    if (p.gi == I && p.gj == J) return launch_givens<GivensMapRule<I, J>>(p, batch, stream);
        SGEMM_EMU_GIVENS_PLANES(SGEMM_EMU_GIVENS_CASE)
#undef SGEMM_EMU_GIVENS_CASE
        return hipErrorInvalidValue;
    }
#define SGEMM_EMU_LDS_KERNEL(CB, PAIR, FAR, STREAM) givens64_lds_kernel<CB, PAIR, FAR, STREAM>
    if (a.mode == SGEMM_EMU_GIVENS_LDS) return SGEMM_EMU_RULE_LAUNCH(SGEMM_EMU_LDS_KERNEL);
#undef SGEMM_EMU_LDS_KERNEL
    return launch_givens<GivensArgRule>(p, batch, stream);
}

}  // namespace sgemm_emu
