// Batched inclusive scan y_j = sum_{i <= j} x_i of every row, as the product
// x^T U with the upper-triangular all-ones U (Sec. 4.1, eq. scan-mat, rule
// u-rule), in emulated FP32 (Sec. 4.4).
//
// A wavefront scans a run of consecutive values, 1024 (a block) at a time.
// The block is read as a 32 x 32 matrix Z of 32 consecutive segments
// (Z[n][k] is value 32 n + k of the block) and scanned in two levels:
//   * within segments, as the transposed product S^T = U^T Z^T: U^T's
//     32 x 32 block is the A operand, built once per wave with foreach_ij
//     from the rule (element (i, k) of U^T is [k <= i]) and never stored; Z
//     is the B operand (two 16-wide k steps, split into hi and lo in
//     registers).  U's entries are 0 and 1, whose lo parts are 0, so the
//     correction reduces to U^T lo(Z^T): four MFMAs per block;
//   * across segments, an exclusive scan of the 32 segment totals over the
//     lanes (five shuffle steps), plus the running total of the row's
//     earlier blocks, added to every value of the segment.
//
// Every block, whole or not, aligned or not, moves between memory and
// registers in four 1 KiB instructions of 16 bytes per lane, on a buffer
// descriptor that ends where the row does: a dword past the end reads as
// zero and is not written, and the accesses need 4-byte alignment only, so
// one path serves every length, row stride and base.  (The bytes are
// regrouped into the operand layout, and back, through LDS.)  The blocks of
// a wave's whole rows form one sequence with the loads of the next kBuf
// blocks in flight while the current one is multiplied.
//
// Rows (scan_kernel, one wave per 1 to 4 whole rows; scan_short_kernel, 32 rows
// of up to 32 values at a time) fill the device when there are many of them.  A
// few long rows are cut into parts instead, one wave each, in three launches on
// the stream that need no memory but Y:
//   scan_total_kernel  each part's plain FP32 sum, left in the part's last
//                      output;
//   scan_chain_kernel  those sums scanned along each row, which makes them
//                      the final outputs at those places;
//   scan_part_kernel   every other output: the part scanned as above from
//                      the output just before it.  The part's own last value
//                      is neither read nor written, so Y may be X.
// A part is read twice and written once; with 128 MB in the last-level
// cache the second read does not go to HBM.
#include "internal.h"
#include "mfmae/frag.hpp"
#include "mfmae/tcec.hpp"

namespace sgemm_emu {

namespace {

using mfmae::f32x16_t;
using mfmae::half8_t;
using mfmae::Shape32;
using mfmae::Use;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
using FragA = mfmae::fragment<Shape32, Use::A, _Float16>;

constexpr int kWaves = 4;
constexpr int kBlock = 1024;  // values scanned at a time
// Magnitudes from here on round to infinity as binary16: their split is
// (infinity, NaN), and so is every sum it enters.
constexpr float kSplitEnd = 65520.0f;
// Block buffers per wave.  Two of them and four waves per SIMD (101 VGPRs)
// against four and three (137): 131,072 rows of 2048 take 361 against 397 us
// (5.9 TB/s), of 512 values 77 against 83, of 200 60 against 68.  With one
// buffer rows of 2048 gain 10 us more, but 65,536 of 4096 lose 22.
constexpr int kBuf = 2;

// The 16 values lane (n, g) holds of a block as B operand: block values
// 32 n + 16 s + 8 g + v, s = 0, 1, v = 0..7.
struct Block {
    float x[2][8];
};

// A block as loaded: lane l holds values 256 i + 4 l .. + 3, i = 0..3, so
// every load instruction reads 1 KiB of consecutive values.
struct Raw {
    f32x4 v[4];
};

// Descriptor of the first `count` floats at p (at most one block): loads past
// them return zero and stores past them are dropped, dword by dword (raw
// buffer, no stride; the fourth word as for every gfx9 raw buffer).
__device__ inline __amdgpu_buffer_rsrc_t block_rsrc(const float* p, int count) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0,
                                             4 * max(0, min(count, kBlock)), 0x00020000);
}

__device__ inline void load_block(Raw& b, const float* p, int count) {
    const __amdgpu_buffer_rsrc_t r = block_rsrc(p, count);
    const int off = 16 * (threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        b.v[i] = __builtin_bit_cast(f32x4,
                                    __builtin_amdgcn_raw_buffer_load_b128(r, off + 1024 * i, 0, 0));
}

// The wave's LDS copy of one block: segment n (32 values) at 36 n floats.
// With this pitch the 16-byte accesses of the operand and accumulator
// layouts (lanes n = 0..15 at 36 n + c) fall on distinct banks.
constexpr int kSegPitch = 36;
constexpr int kStageFloats = 32 * kSegPitch;

__device__ inline int staged(int value) { return kSegPitch * (value >> 5) + (value & 31); }

// Regroup a contiguous block into the operand layout through the wave's
// LDS buffer (other lanes' values: ordered by the wave fence).
__device__ inline void to_operand(const Raw& r, float* buf, Block& b) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(buf + staged(256 * i + 4 * l)) = r.v[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    const float* q = buf + kSegPitch * (l & 31) + 8 * (l >> 5);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(q + 16 * s);
        const f32x4 v1 = *reinterpret_cast<const f32x4*>(q + 16 * s + 4);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            b.x[s][v] = v0[v];
            b.x[s][v + 4] = v1[v];
        }
    }
}

// U^T's diagonal block for k step s: element (i, kk) is [16 s + kk <= i];
// hi only (lo is 0 for 0 and 1).
__device__ inline void upper_ones(half8_t (&Ut)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
        mfmae::foreach_ij<FragA>([&](int e, int i, int kk) {
            Ut[s][e] = (16 * s + kk <= i) ? (_Float16)1.0f : (_Float16)0.0f;
        });
}

// Scans within the block's segments: accumulator element e of lane (n, g) is
// value 8 (e / 4) + 4 g + e % 4 of segment n.
__device__ inline void scan_segments(const Block& b, const half8_t (&Ut)[2], float (&z)[16]) {
    f32x16_t acc, cor;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        acc[e] = 0.0f;
        cor[e] = 0.0f;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        half8_t xh, xl;
        mfmae::tcec::split8(b.x[s], xh, xl);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ut[s], xh, acc, 0, 0, 0);
        cor = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ut[s], xl, cor, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = __builtin_fmaf(cor[e], mfmae::tcec::kLoScaleInv, acc[e]);
}

// y = carry + scan of the block; carry becomes the row's running total
// after it.  Accumulator element e of lane (n, g) is block value
// 32 n + 8 (e / 4) + 4 g + e % 4.
__device__ inline void scan_block(const Block& b, const half8_t (&Ut)[2], float& carry,
                                  float (&y)[16]) {
    const int l = threadIdx.x & 63;
    const int n = l & 31;
    float z[16];
    scan_segments(b, Ut, z);
    // segment totals: the last value of segment n is element 15 of lane
    // 32 + n; inclusive scan of the totals over n (both half-waves hold it)
    float incl = __shfl(z[15], 32 + n, 64);
#pragma unroll
    for (int d = 1; d < 32; d *= 2) {
        const float u = __shfl_up(incl, d, 32);
        if (n >= d) incl += u;
    }
    const float before = __shfl_up(incl, 1, 32);  // total of segments 0..n-1
    const float offset = n == 0 ? carry : carry + before;
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = offset + z[e];
    carry = carry + __shfl(incl, 31, 64);
}

// Outputs in the accumulator layout, regrouped through the wave's LDS
// buffer and stored as four contiguous 1 KiB instructions, nontemporal: y
// is not read again (measured 2.7% faster; streaming loads too, 374 -> 486 us
// on 131,072 rows of 2048).
__device__ inline void store_block(float* p, int count, const float (&y)[16], float* buf) {
    constexpr int kNontemporal = 2;
    const int l = threadIdx.x & 63;
    float* q = buf + kSegPitch * (l & 31) + 4 * (l >> 5);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");  // operand reads done
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(q + 8 * g) = f32x4{y[4 * g], y[4 * g + 1], y[4 * g + 2],
                                                     y[4 * g + 3]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    const __amdgpu_buffer_rsrc_t r = block_rsrc(p, count);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(u32x4, *reinterpret_cast<const f32x4*>(buf + staged(256 * i + 4 * l))),
            r, 16 * l + 1024 * i, 0, kNontemporal);
}

// Scan `nrows` runs of `len` values each, run r at x + r ldx, into y + r ldy,
// every run starting from `carry0`: one sequence of blocks, kBuf of them in
// flight.  Loads are unconditional (past the end they re-read the last
// block) and the first round of steps is peeled, so the loop is entered with
// the same memory operations pending as on every later iteration and the
// wait before each block covers that block's loads only.
__device__ __forceinline__ void scan_rows(const float* x, int64_t ldx, float* y, int64_t ldy, int nrows,
                                 int len, float carry0, float* sb) {
    half8_t Ut[2];
    upper_ones(Ut);

    const int nb = (len - 1) / kBlock + 1;  // blocks per run
    const int64_t nf = (int64_t)nrows * nb;
    int64_t lf = 0;  // load cursor: block lf of the sequence, block lblk of its run
    int lblk = 0;
    auto load_next = [&](Raw& b) __attribute__((always_inline)) {
        load_block(b, x + (int64_t)lblk * kBlock, len - lblk * kBlock);
        if (lf + 1 < nf) {
            ++lf;
            if (++lblk == nb) {
                lblk = 0;
                x += ldx;
            }
        }
    };
    float carry = carry0;
    int blk = 0;  // block of the run that is scanned next
    auto scan_next = [&](const Raw& r) __attribute__((always_inline)) {
        Block b;
        float out[16];
        to_operand(r, sb, b);
        scan_block(b, Ut, carry, out);
        store_block(y + (int64_t)blk * kBlock, len - blk * kBlock, out, sb);
        if (++blk == nb) {
            blk = 0;
            y += ldy;
            carry = carry0;
        }
    };
    // the scheduling barrier keeps each step's reload in place, so the
    // blocks really are loaded kBuf steps ahead
    auto step = [&](Raw& r) __attribute__((always_inline)) {
        scan_next(r);
        load_next(r);
        __builtin_amdgcn_sched_barrier(0);
    };
    Raw buf[kBuf];
#pragma unroll
    for (int i = 0; i < kBuf; ++i) load_next(buf[i]);
    int64_t f = 0;
    if (nf >= kBuf) {
#pragma unroll
        for (int i = 0; i < kBuf; ++i) step(buf[i]);
        for (f = kBuf; f + kBuf <= nf; f += kBuf) {
#pragma unroll
            for (int i = 0; i < kBuf; ++i) step(buf[i]);
        }
    }
    // buf[i] holds block f + i for the remaining blocks
#pragma unroll
    for (int i = 0; i < kBuf - 1; ++i)
        if (f + i < nf) scan_next(buf[i]);
}

__global__ __launch_bounds__(64 * kWaves, 4) void scan_kernel(ScanArgs p, int rows_per_wave) {
    __shared__ __attribute__((aligned(16))) float stage[kWaves][kStageFloats];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r0 = ((int64_t)blockIdx.x * kWaves + wave) * rows_per_wave;
    if (r0 >= p.rows) return;  // whole wave; no barrier below
    scan_rows(p.X + r0 * p.ldx, p.ldx, p.Y + r0 * p.ldy, p.ldy,
              (int)min((int64_t)rows_per_wave, p.rows - r0), p.len, 0.0f, stage[wave]);
}

// Rows of at most one segment: 32 rows are the segments of one block, so a
// wave scans them with the four products of a block and nothing crosses the
// segments (1,000,000 rows of 1 / 8 / 32 values 13 / 16 / 44 us, a block per row
// 431 / 424 / 426).  Loads and stores go straight between memory and the operand
// and accumulator layouts, lane (n, g) of row n, in 16-byte pieces of 4-byte
// alignment; what a piece holds of the next row is dropped, and the descriptor
// ends with the last row.
constexpr int kShort = 32;

// Byte offsets of 32 rows stay below 2^31.
inline bool short_rows(const ScanArgs& a) {
    return a.len <= kShort && a.ldx < (1 << 24) && a.ldy < (1 << 24);
}

__global__ __launch_bounds__(64 * kWaves) void scan_short_kernel(ScanArgs p, int groups) {
    constexpr uint32_t kPastEnd = 0x80000000;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63, n = l & 31, g = l >> 5;
    half8_t Ut[2];
    upper_ones(Ut);
    for (int i = 0; i < groups; ++i) {
        const int64_t r0 = (((int64_t)blockIdx.x * kWaves + wave) * groups + i) * 32;
        if (r0 >= p.rows) return;
        const int rows = (int)min((int64_t)32, p.rows - r0);
        const bool row = n < rows;
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(p.X + r0 * p.ldx), 0, (int)(4 * ((rows - 1) * p.ldx + p.len)),
            0x00020000);
        Block b;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = 16 * s + 8 * g + 4 * h;
                const f32x4 v = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                               rx, row && c < p.len ? 4 * (uint32_t)(n * p.ldx + c) : kPastEnd, 0,
                               0));
#pragma unroll
                for (int e = 0; e < 4; ++e) b.x[s][4 * h + e] = c + e < p.len ? v[e] : 0.0f;
            }
        float z[16];
        scan_segments(b, Ut, z);
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
            p.Y + r0 * p.ldy, 0, (int)(4 * ((rows - 1) * p.ldy + p.len)), 0x00020000);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = 8 * q + 4 * g;
            const uint32_t at = 4 * (uint32_t)(n * p.ldy + c);
            // (0 + z: the offset of a row's first segment)
            const u32x4 v = __builtin_bit_cast(u32x4, f32x4{0.0f + z[4 * q], 0.0f + z[4 * q + 1],
                                                            0.0f + z[4 * q + 2],
                                                            0.0f + z[4 * q + 3]});
            const bool whole = row && c + 4 <= p.len;
            __builtin_amdgcn_raw_buffer_store_b128(v, ry, whole ? at : kPastEnd, 0, 0);
#pragma unroll
            for (int e = 0; e < 3; ++e)
                __builtin_amdgcn_raw_buffer_store_b32(
                    v[e], ry, row && !whole && c + e < p.len ? at + 4 * e : kPastEnd, 0, 0);
        }
    }
}

// Part `part` of a row cut into parts of `blocks` blocks: its first value and
// its number of values (the last part of a row may be shorter).
struct Part {
    int64_t row;
    int part, first, count;
};

__device__ inline Part part_of(const ScanArgs& p, int blocks, int nparts, int64_t task) {
    Part q;
    q.row = task / nparts;
    q.part = (int)(task - q.row * nparts);
    q.first = q.part * blocks * kBlock;  // < len: fits
    q.count = min(blocks * kBlock, p.len - q.first);
    return q;
}

__global__ __launch_bounds__(64 * kWaves) void scan_total_kernel(ScanArgs p, int blocks,
                                                                 int nparts) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t task = (int64_t)blockIdx.x * kWaves + wave;
    if (task >= p.rows * nparts) return;
    const Part q = part_of(p, blocks, nparts, task);
    const float* x = p.X + q.row * p.ldx + q.first;
    constexpr int kAhead = 4;  // blocks in flight; past the end they read as zero
    f32x4 sum[4] = {};
    float peak = 0.0f;
    for (int c = 0; c < q.count; c += kAhead * kBlock) {
        Raw r[kAhead];
#pragma unroll
        for (int b = 0; b < kAhead; ++b) load_block(r[b], x + c + b * kBlock, q.count - c - b * kBlock);
#pragma unroll
        for (int b = 0; b < kAhead; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sum[i] += r[b].v[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) peak = fmaxf(peak, fabsf(r[b].v[i][e]));
            }
    }
    const f32x4 s = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    float total = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int d = 32; d > 0; d /= 2) total += __shfl_xor(total, d, 64);
    // A value the split does not represent makes the rest of its row NaN, as
    // in a scan of whole rows (a NaN is in the sum already).
    if (__any(!(peak < kSplitEnd))) total = __builtin_nanf("");
    if ((threadIdx.x & 63) == 0) p.Y[q.row * p.ldy + q.first + q.count - 1] = total;
}

// One wave per row: the sums of its parts, 64 at a time.
__global__ __launch_bounds__(64) void scan_chain_kernel(ScanArgs p, int blocks, int nparts) {
    const int l = threadIdx.x;
    float* y = p.Y + (int64_t)blockIdx.x * p.ldy;
    float carry = 0.0f;
    for (int s0 = 0; s0 < nparts; s0 += 64) {
        const bool in = s0 + l < nparts;
        const int64_t end = (int64_t)(s0 + l + 1) * blocks * kBlock;
        float* at = y + min(end, (int64_t)p.len) - 1;
        float t = in ? *at : 0.0f;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const float u = __shfl_up(t, d, 64);
            if (l >= d) t += u;
        }
        t += carry;
        if (in) *at = t;
        carry = __shfl(t, 63, 64);
    }
}

__global__ __launch_bounds__(64 * kWaves, 4) void scan_part_kernel(ScanArgs p, int blocks,
                                                                   int nparts) {
    __shared__ __attribute__((aligned(16))) float stage[kWaves][kStageFloats];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t task = (int64_t)blockIdx.x * kWaves + wave;
    if (task >= p.rows * nparts) return;
    const Part q = part_of(p, blocks, nparts, task);
    if (q.count == 1) return;  // its one output is final
    float* y = p.Y + q.row * p.ldy + q.first;
    const float before = q.part == 0 ? 0.0f : y[-1];
    scan_rows(p.X + q.row * p.ldx + q.first, 0, y, 0, 1, q.count - 1, before, stage[wave]);
}

}  // namespace

// Rows a wave takes.  Short rows share the wave's set-up, and two rows that fill
// two blocks its buffers; other rows are better spread over more waves
// (131,072 rows, 1 / 2 / 4 rows per wave: 100 values 66 / 68 / 59 us, 512 88 /
// 84 / 79, 1000 170 / 187 / 192, 1537 297 / 322 / 333, 1920 351 / 358, 1984
// 359 / 358, 2000 372 / 369, 2040 407 / 435, 2048 369 to 382 / 360 to 363 / 364;
// 65,536 rows of 4096: 362 / 366 / 407).
static int64_t rows_per_wave(int64_t rows, int len) {
    const int64_t best = len <= 512 ? 4 : len > 2 * kBlock - kBlock / 16 && len <= 2 * kBlock ? 2 : 1;
    const int64_t fill = rows / 8192;  // and at least that many waves
    return fill < 1 ? 1 : fill < best ? fill : best;
}

hipError_t launch_scan(const ScanArgs& a, hipStream_t stream) {
    const int64_t nb = (a.len - 1) / kBlock + 1;
    if (short_rows(a)) {
        // up to 4 groups of 32 rows per wave, and at least 8192 waves
        const int64_t all = (a.rows + 31) / 32;
        const int64_t groups = all < 2 * 8192 ? 1 : all < 4 * 8192 ? 2 : 4;
        // one launch stays below 2^31 work-items
        const int64_t max_rows = ((int64_t(1) << 31) / (64 * kWaves) - 1) * kWaves * groups * 32;
        for (int64_t r0 = 0; r0 < a.rows; r0 += max_rows) {
            ScanArgs c = a;
            c.rows = a.rows - r0 < max_rows ? a.rows - r0 : max_rows;
            c.X = a.X + r0 * a.ldx;
            c.Y = a.Y + r0 * a.ldy;
            const int64_t per = 32 * groups * kWaves;
            hipLaunchKernelGGL(scan_short_kernel, dim3((unsigned)((c.rows + per - 1) / per)),
                               dim3(64 * kWaves), 0, stream, c, (int)groups);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // A wave takes about 1 us per block of its row whatever the others do, so
    // nb us for whole rows until they fill the device; in parts a scan takes
    // 16 us (three launches) or 1.5 times the whole rows' memory time, if
    // that is longer.  Measured, whole / parts: 16 blocks 19.6 / 17.4 us for
    // 128 and for 512 rows; 64 blocks 68 / 17 us for 128 rows, 68 / 65 for
    // 512, 84 / 127 for 1024; 8 blocks 11 / 16 us.
    if (a.rows < 512 && nb >= 16) {
        // about 4096 parts in all (16 waves per CU), of at least 4 blocks
        const int64_t per_row = (4096 + a.rows - 1) / a.rows;
        int64_t blocks = (nb + per_row - 1) / per_row;
        if (blocks < 4) blocks = 4;
        const int nparts = (int)((nb + blocks - 1) / blocks);
        const dim3 grid((unsigned)((a.rows * nparts + kWaves - 1) / kWaves));
        hipLaunchKernelGGL(scan_total_kernel, grid, dim3(64 * kWaves), 0, stream, a, (int)blocks,
                           nparts);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(scan_chain_kernel, dim3((unsigned)a.rows), dim3(64), 0, stream, a,
                           (int)blocks, nparts);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(scan_part_kernel, grid, dim3(64 * kWaves), 0, stream, a, (int)blocks,
                           nparts);
        return hipGetLastError();
    }
    // one launch stays below 2^31 work-items (the dispatch packet counts
    // work-items in 32 bits); more rows take several launches, each on its
    // own range of rows
    const int64_t rpw = rows_per_wave(a.rows, a.len);
    const int64_t max_blocks = (int64_t(1) << 31) / (64 * kWaves) - 1;
    const int64_t rows_per_launch = max_blocks * kWaves * rpw;
    for (int64_t r0 = 0; r0 < a.rows; r0 += rows_per_launch) {
        ScanArgs c = a;
        c.rows = a.rows - r0 < rows_per_launch ? a.rows - r0 : rows_per_launch;
        c.X = a.X + r0 * a.ldx;
        c.Y = a.Y + r0 * a.ldy;
        const int64_t waves = (c.rows + rpw - 1) / rpw;
        const int64_t blocks = (waves + kWaves - 1) / kWaves;
        hipLaunchKernelGGL(scan_kernel, dim3((unsigned)blocks), dim3(64 * kWaves), 0, stream, c,
                           (int)rpw);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace sgemm_emu
