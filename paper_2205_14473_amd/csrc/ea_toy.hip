// ea_toy.hip -- the toy problem of Section V-A on the device:
// f(x) = E_xi || A x - (x* + xi) ||^2, whose gradient for a noise draw xi_i is
// g_i = 2 A^T (A x - x* - xi_i).  Products are summed in binary64 and each g
// rounded once to binary32, like the oracle.
//
// Two launches for both entry points:
//   1. residual: res[k] = (A x)[k] - x*[k], one wave per row of A (it also
//      clears the counter of the second launch);
//   2. toy_round_kernel: a block owns 32 or 64 columns and all rows of A.  The sums
//      of all workers (and the noise-free one) over the rows are one matrix
//      product, (r - xi_i)^T A, and run on the f64 matrix cores
//      (v_mfma_f64_16x16x4: 16 outputs x 16 columns x 4 rows), operands
//      straight from global memory into registers: each of the 16 waves takes
//      every 16th group of 16 rows, and the 16 partial sums of an output are
//      added in wave order through LDS.  The last block to finish adds the
//      blocks' partial squared norms of the noise-free gradient (lane l those
//      of blocks l, l+64, ..., then the wave's sum); no block waits.
//
// ea_toy_grad writes the gradients and stops there.  ea_toy_step fuses the
// producer into the round (quantizers without scales: Example 2, full
// precision): half a wave (a wave with 64 columns) holds worker i's gradient
// for the block's columns and runs its side of the round (Adam at the worker,
// the code, the residual); its codes fill an 8-bit (16-bit) slice of each
// message word (the block's columns are 8 or 16 lanes of one 256-element
// chunk).  The last wave adds the
// workers' dequantized values in ascending order and runs the server side.
// The gradient is not written to HBM unless asked for (g_out).  Both entry
// points sum in the same order, so their gradients agree bit for bit.
#include "ea_launch.hpp"

#include <type_traits>

namespace ea {

namespace {

constexpr int kResWaves = 4;                    // rows per residual block
constexpr int kResAhead = 4;                    // chunks of a row loaded together

// A descriptor over at most the next 2 GiB of a larger array (bytes: what is
// left of it).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t window(const void* p, int64_t bytes)
{
    const int64_t cap = 0x7FFFFFF0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(bytes < cap ? bytes : cap), kRawBuffer);
}

// Bound by the read of A (d = 8192: 38 us, 7.0 TB/s, A fitting the memory-side
// cache in part); at d = 500 by one memory
// latency, so the loads of up to four 256-element chunks of the row go out
// together.  A product of two binary32 values is exact in binary64.
__global__ __launch_bounds__(kResWaves * kWave) void toy_residual_kernel(int64_t d, const float* __restrict__ A,
                                                                         const float* __restrict__ xs,
                                                                         const float* __restrict__ x,
                                                                         double* __restrict__ res,
                                                                         uint32_t* __restrict__ counter)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;
    const int64_t k = (int64_t)blockIdx.x * kResWaves + wave_id();
    if (k >= d) return;
    const __amdgpu_buffer_rsrc_t row = window(A + k * d, d * 4), xr = window(x, d * 4);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j = 0; j < (int)d; j += kResAhead * kChunk) {
        ea_u4v av[kResAhead], xv[kResAhead];
#pragma unroll
        for (int u = 0; u < kResAhead; ++u) {
            const int off = (j + u * kChunk) * 4 + lane_id() * 16;     // past the row's end: zeros
            av[u] = __builtin_amdgcn_raw_buffer_load_b128(row, off, 0, 0);
            xv[u] = __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kResAhead; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                s[c] = fma((double)__uint_as_float(av[u][c]), (double)__uint_as_float(xv[u][c]), s[c]);
    }
    const double sum = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
    if (lane_id() == 0) res[k] = sum - (double)xs[k];
}

// ---------------------------------------------------------------------------
// The fused toy round.
// ---------------------------------------------------------------------------
constexpr int kTRWaves = 16;                   // waves per block
constexpr int kTROut = 16;                     // column sums per pass: workers + the noise-free one
constexpr int kTRWorkers = kTROut - 1;         // workers per pass
constexpr int kTRRows = 16;                    // rows per group: four matrix instructions deep
typedef double ea_d4v __attribute__((ext_vector_type(4)));

// Bits 0, 4, 8, ..., 28 of x gathered into bits 0..7.
__device__ __forceinline__ uint32_t every_fourth_bit(uint32_t x)
{
    x &= 0x11111111u;
    x = (x | (x >> 3)) & 0x03030303u;
    x = (x | (x >> 6)) & 0x000F000Fu;
    return (x | (x >> 12)) & 0x000000FFu;
}

// Code and dequantized value of one element for a quantizer without scales.
__device__ __forceinline__ void toy_code(const QDev& q, float p, uint32_t& code, float& deq)
{
    if (q.kind == Q_NONE) {
        code = __float_as_uint(p);
        deq = p;
    } else {
        code = code_of<QRt>(q, p, 0.0f, 0u);
        deq = lut_entry<QRt>(q, (int32_t)code);
    }
}

// The block's COLS columns are lanes l0..l0+COLS/4-1 of a chunk, all four
// slots.  With 32 columns each half of the wave holds them for one message
// (msg may be null: nothing to store for that half); with 64 the wave holds
// one message's.  Bit plane p of slot s is a slice of COLS/4 bits (whole
// bytes) of message word (4 chunk + s) b + p; lane s b + p of the half or wave
// stores it.  Raw values (b = 32) are stored as the binary32 element itself.
// The last column block clears the rest of its chunk's words.
template <int COLS>
__device__ __forceinline__ void toy_store_codes(const QDev& q, uint64_t* __restrict__ msg, int64_t c0, bool in,
                                                bool last, uint32_t code)
{
    using Slice = std::conditional_t<COLS == 32, uint8_t, uint16_t>;
    const int hl = lane_id() & (COLS - 1);
    if (q.kind == Q_NONE) {
        if (msg != nullptr && in) reinterpret_cast<uint32_t*>(msg)[c0 + hl] = code;
        return;
    }
    const int b = q.bits;
    constexpr int kSlices = kChunk / COLS;                     // slices of a word
    const int at = (int)(c0 / COLS) & (kSlices - 1);
    Slice* words = reinterpret_cast<Slice*>(msg + (c0 >> 8) * 4 * b) + at;
    for (int first = 0; first < 4 * b; first += COLS) {        // twice for 9-bit codes on 32 columns
        const int j = first + hl;
        const int s = (j >= b ? 1 : 0) + (j >= 2 * b ? 1 : 0) + (j >= 3 * b ? 1 : 0);
        const int p = j - s * b;
        uint32_t lo = 0u, hi = 0u;                             // the plane's bits of columns 0-31 and 32-63
        for (int pl = 0; pl < b; ++pl) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(in && ((code >> pl) & 1u) != 0u);
            const bool upper = COLS == 32 && lane_id() >= 32;
            lo = pl == p ? (upper ? (uint32_t)(m >> 32) : (uint32_t)m) : lo;
            if (COLS == 64) hi = pl == p ? (uint32_t)(m >> 32) : hi;
        }
        if (msg != nullptr && j < 4 * b) {
            words[j * kSlices] = (Slice)(every_fourth_bit(lo >> s) | (COLS == 64 ? every_fourth_bit(hi >> s) << 8 : 0u));
            if (last)
                for (int r = 1; r < kSlices - at; ++r) words[j * kSlices + r] = 0;
        }
    }
}

struct ToyArgs {
    int64_t d;
    int32_t N, placement;
    float beta1, beta2, lr;
    QDev qw, qs;
    const float* A;
    const double* res;      // r = A x - x*
    const float* xi;        // [N][d]
    float *x, *e_w, *m_w, *v_w, *m, *v, *e_s;
    uint64_t *wcodes, *scodes;
    double* part;           // [blocks] partial squared norms of the noise-free gradient
    uint32_t* counter;      // blocks done (cleared by the residual launch)
    int32_t nblk;           // column blocks
    double* grad_sq;        // nullable
    float* g_out;           // nullable: [N][d] the workers' gradients, for checking
};

// ROUND: the round follows the gradients; without it the kernel only writes
// the gradients to g_out (ea_toy_grad) and the norm.
//
// Bound by the second read of A where it is large, by two memory latencies,
// the reduction and the round's own chain at d = 500.  The vector form this
// replaced read each residual as a broadcast from LDS for every 64 columns
// (128 bytes of LDS a row and wave against 16 multiply-adds), which bound it
// at any size, and split the rows over blocks that met through global memory;
// a matrix operand instead holds 64 different residuals, and a block walks all
// rows.  CT 16-column tiles a block, two or four: message slices are whole
// bytes, and with two a row's piece is one 128-byte line.  The groups whose
// loads are in flight are as many as paid: at two tiles two sets of one (one
// set of three 99 us a step at d = 8192, three sets of one 94, against 92), at
// four one set of two.  Measured, 10 workers, a whole step, before and after:
// d = 500 22.4 -> 13.9 us, 4096 122 -> 39.6 us, 8192 334 -> 92-101 us (A read
// twice 5.3-5.9 TB/s), 16384 1025 -> 394 us (5.5 TB/s), 40000 4.70 -> 2.37 ms (5.4 TB/s);
// 20 workers (two passes) at d = 1557 103 -> 26 us.
template <int CT, int SETS, int AHEAD, bool ROUND>
__global__ __launch_bounds__(kTRWaves * kWave) void toy_round_kernel(ToyArgs a)
{
    constexpr int COLS = 16 * CT;
    typedef float ea_fv __attribute__((ext_vector_type(CT)));
    // the waves' partial sums: [wave][output][column]
    __shared__ __attribute__((aligned(16))) double big[kTRWaves * kTROut * COLS];
    __shared__ float xfer[kTRWorkers * COLS];
    // Consecutive blocks go to the 8 XCDs in turn; each XCD takes a run of
    // adjacent column blocks, which share lines when d is not a multiple of
    // 32, so that a line is fetched into one L2.
    const int per = (a.nblk + 7) / 8;
    const int blk = ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8;
    if (blk >= a.nblk || (int)blockIdx.x / 8 >= per) return;       // the whole block leaves
    const int lane = lane_id();
    const int w = wave_id();
    const int64_t d = a.d;
    const int64_t c0 = (int64_t)blk * COLS;
    const bool last = blk == a.nblk - 1;
    const bool atw = a.placement == AT_WORKER;
    constexpr int kServer = kTRWaves - 1;
    const bool server = w == kServer && lane < COLS;
    const int64_t col = c0 + (lane & (COLS - 1));
    const bool in = col < d;
    // With 32 columns two outputs share a wave and the upper half of the block
    // has none; with 64 wave o holds output o.
    const auto norm_wave = [](int nw) { return COLS == 32 ? kTRWaves / 2 : nw; };
    double norm_sq = 0.0;
    float acc = 0.0f;                              // the server's sum of dequantized messages
    float sm = 0.0f, sv = 0.0f, se = 0.0f, sx = 0.0f;
    // Operand lanes: n = lane % 16 is the output (residuals) or the columns
    // CT n .. CT n + CT - 1 (A; column CT n + c belongs to matrix tile c),
    // q = lane / 16 the four rows 4q..4q+3 of a group.
    const int n16 = lane & 15, q4 = (lane >> 4) * 4;
    int offA[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) offA[j] = (int)(((q4 + j) * d + CT * n16) * 4);
    const __amdgpu_buffer_rsrc_t rres = window(a.res, d * 8), rxi = window(a.xi, (int64_t)a.N * d * 4);
    const int ngroups = (int)((d + kTRRows - 1) / kTRRows);

    for (int g0 = 0; g0 < a.N; g0 += kTRWorkers) {
        const int nw = a.N - g0 < kTRWorkers ? a.N - g0 : kTRWorkers;
        const bool first = g0 == 0;                // output nw is the noise-free gradient (first pass)
        // outputs past the workers take no noise: their offset lies past xi
        const int offX = n16 < nw ? (int)(((int64_t)(g0 + n16) * d + q4) * 4) : 0x7FFFFFF0;
        ea_d4v s[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) s[c] = ea_d4v{0.0, 0.0, 0.0, 0.0};
        struct Group {
            ea_fv a[4];                            // A, rows 4q + j
            ea_u4v x, r0, r1;                      // noise and residuals of the same rows
        };
        const auto load = [&](int grp, Group& f) {
            const int64_t k0 = (int64_t)(grp < ngroups ? grp : 0) * kTRRows;
            // rows past d read as zeros past the end of A; columns past d
            // read what follows and are not used
            const __amdgpu_buffer_rsrc_t rA = window(a.A + k0 * d + c0, grp < ngroups ? ((d - k0) * d - c0) * 4 : 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (CT == 2)
                    f.a[j] = __builtin_bit_cast(ea_fv, __builtin_amdgcn_raw_buffer_load_b64(rA, offA[j], 0, 0));
                else
                    f.a[j] = __builtin_bit_cast(ea_fv, __builtin_amdgcn_raw_buffer_load_b128(rA, offA[j], 0, 0));
            }
            f.x = __builtin_amdgcn_raw_buffer_load_b128(rxi, n16 < nw ? offX + (int)k0 * 4 : offX, 0, 0);
            f.r0 = __builtin_amdgcn_raw_buffer_load_b128(rres, ((int)k0 + q4) * 8, 0, 0);
            f.r1 = __builtin_amdgcn_raw_buffer_load_b128(rres, ((int)k0 + q4) * 8 + 16, 0, 0);
        };
        const auto sum = [&](int grp, const Group& f) {
            const bool full = (int64_t)(grp + 1) * kTRRows <= d;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t lo = j < 2 ? f.r0[2 * j] : f.r1[2 * j - 4];
                const uint32_t hi = j < 2 ? f.r0[2 * j + 1] : f.r1[2 * j - 3];
                double val = join(hi, lo) - (double)__uint_as_float(f.x[j]);
                // past d the noise read is another worker's: zero, so that not
                // even an infinity there meets the zeros of A
                if (!full) val = (int64_t)grp * kTRRows + q4 + j < d ? val : 0.0;
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    s[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(val, (double)f.a[j][c], s[c], 0, 0, 0);
            }
        };
        // A ring of SETS sets of AHEAD groups: while one set is summed, the
        // others' loads are in flight.
        Group f[SETS][AHEAD];
        constexpr int kStep = kTRWaves * AHEAD;
#pragma unroll
        for (int i = 0; i < SETS - 1; ++i)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) load(w + i * kStep + u * kTRWaves, f[i][u]);
        for (int grp0 = w; grp0 < ngroups; grp0 += SETS * kStep) {
#pragma unroll
            for (int i = 0; i < SETS; ++i) {
                const int grp = grp0 + i * kStep;
                if (grp >= ngroups) break;
#pragma unroll
                for (int u = 0; u < AHEAD; ++u)
                    load(grp + (SETS - 1) * kStep + u * kTRWaves, f[(i + SETS - 1) % SETS][u]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < AHEAD; ++u)
                    if (grp + u * kTRWaves < ngroups) sum(grp + u * kTRWaves, f[i][u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // After the sums, thread (o, column) holds output o of the pass.  Its
        // rows and the server's (only this block writes them) are loaded here
        // and arrive during the reduction; loaded before the sums they took
        // registers from the groups in flight.  (The 64-column kernel spills 11
        // VGPRs to scratch all the same, once a pass outside the sums.)
        const int o = (int)threadIdx.x / COLS;
        const int64_t wrow = (int64_t)(g0 + (o < nw ? o : 0)) * d + (in ? col : d - 1);
        float e0 = 0.0f, m0 = 0.0f, v0 = 0.0f;
        if (ROUND && o < nw) {
            e0 = a.e_w[wrow];
            if (atw) {
                m0 = a.m_w[wrow];
                v0 = a.v_w[wrow];
            }
        }
        if (ROUND && server && in && g0 + kTRWorkers >= a.N) {
            if (!atw) {
                sm = a.m[col];
                sv = a.v[col];
            }
            se = a.e_s[col];
            sx = a.x[col];
        }
        if (!first) __syncthreads();               // the previous pass's sums have been read
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // result lane l, register i: output l/16 + 4i, column l%16 of its tile
#pragma unroll
            for (int c = 0; c < CT; c += 2) {
                double2* slot = reinterpret_cast<double2*>(big + (w * kTROut + (lane >> 4) + 4 * i) * COLS + CT * n16 + c);
                *slot = make_double2(s[c][i], s[c + 1][i]);
            }
        }
        __syncthreads();
        if (o < kTROut) {                          // whole waves
            double tot = 0.0;
#pragma unroll
            for (int u = 0; u < kTRWaves; ++u) tot += big[(u * kTROut + o) * COLS + (lane & (COLS - 1))];
            const double gd = 2.0 * tot;
            const bool mine = o < nw;
            // worker g0 + o (Algorithm 2 with Adam at the worker, else g + e)
            const float g = (float)gd;
            if (mine && in && a.g_out != nullptr) a.g_out[wrow] = g;
            if constexpr (ROUND) {
                float p;
                if (atw) {
                    const float vk = a.beta2 * v0 + (1.0f - a.beta2) * (g * g);
                    const float mk = a.beta1 * m0 + (1.0f - a.beta1) * g;
                    p = (vk > 0.0f ? a.lr * (mk / sqrtf(vk)) : 0.0f) + e0;
                    if (mine && in) {
                        a.m_w[wrow] = mk;
                        a.v_w[wrow] = vk;
                    }
                } else {
                    p = g + e0;
                }
                uint32_t code;
                float dq;
                toy_code(a.qw, p, code, dq);
                if (mine && in) a.e_w[wrow] = a.qw.ef ? p - dq : 0.0f;
                toy_store_codes<COLS>(a.qw, mine ? a.wcodes + (int64_t)(g0 + o) * a.qw.words : nullptr, c0, in, last, code);
                if (mine) xfer[o * COLS + (lane & (COLS - 1))] = dq;
            }
        }
        // the noise-free gradient's square, on a wave without a worker
        if (first && w == norm_wave(nw) && a.grad_sq != nullptr) {
            double tot = 0.0;
#pragma unroll
            for (int u = 0; u < kTRWaves; ++u) tot += big[(u * kTROut + nw) * COLS + (lane & (COLS - 1))];
            const double gd = 2.0 * tot;
            norm_sq = lane < COLS && in ? gd * gd : 0.0;
        }
        if constexpr (ROUND) {
            __syncthreads();
            if (server) {
                float dq[kTRWorkers];              // all the reads first
#pragma unroll
                for (int i = 0; i < kTRWorkers; ++i) dq[i] = xfer[i * COLS + lane];
#pragma unroll
                for (int i = 0; i < kTRWorkers; ++i)
                    if (i < nw) acc = acc + dq[i];
            }
        }
    }

    if (ROUND && w == kServer) {                   // lanes past the columns store nothing
        // Algorithm 1: average, [Adam at the server], residual, quantize, apply
        const float fN = (float)a.N;
        const bool pow2 = (a.N & (a.N - 1)) == 0;
        const float avg = pow2 ? acc * (1.0f / fN) : acc / fN;
        float u = avg;
        if (!atw) {
            const float vk = a.beta2 * sv + (1.0f - a.beta2) * (avg * avg);
            const float mk = a.beta1 * sm + (1.0f - a.beta1) * avg;
            u = vk > 0.0f ? a.lr * (mk / sqrtf(vk)) : 0.0f;
            if (server && in) {
                a.m[col] = mk;
                a.v[col] = vk;
            }
        }
        const float q = u + se;
        uint32_t code;
        float dq;
        toy_code(a.qs, q, code, dq);
        if (server && in) {
            a.e_s[col] = a.qs.ef ? q - dq : 0.0f;
            a.x[col] = sx - dq;
        }
        toy_store_codes<COLS>(a.qs, server ? a.scodes : nullptr, c0, in, last, code);
    }

    // The block's share of ||grad F||^2.  The last block to get here adds the
    // shares: lane l those of blocks l, l+64, ... in order (loaded side by
    // side), then the wave's sum.  The order rests on this chip's rules, not on
    // the memory model, in which relaxed atomics publish nothing: agent-scope
    // stores are written through to where every XCD's agent-scope loads read,
    // past the L2s, and the store has completed there when vmcnt is 0, so the
    // wait puts the share before the count; the loads depend on the count.
    // (What the model asks for, a release fence, would write back the XCD's
    // whole L2, and its acquire drop it.)
    if (w == norm_wave(a.N < kTRWorkers ? a.N : kTRWorkers) && a.grad_sq != nullptr) {
        const double sq = wave_sum(norm_sq);
        unsigned long long* bits = reinterpret_cast<unsigned long long*>(a.part);
        uint32_t done = 0;
        if (lane == 0) {
            __hip_atomic_store(bits + blk, (unsigned long long)__double_as_longlong(sq), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            done = __hip_atomic_fetch_add(a.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        done = (uint32_t)uniform((int)done);
        if (done == (uint32_t)a.nblk - 1) {
            asm volatile("" ::: "memory");
            double share = 0.0;
            for (int b = lane; b < a.nblk; b += kWave)
                share += __longlong_as_double(
                    (long long)__hip_atomic_load(bits + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            const double all = wave_sum(share);
            if (lane == 0) *a.grad_sq = all;
        }
    }
}

}  // namespace

// Columns per block: 64 once such blocks fill the 256 CUs (each block then
// reads the residuals and the noise for twice the columns: d = 16384, 10
// workers 394 against 431 us a step), 32 below (d = 8192 92 against 130 us, d =
// 2075 22 against 30: half the CUs would have no block), and 64 up to 64
// parameters, a single block either way.
int toy_cols(int64_t d)
{
    return d > 64 && (d + 63) / 64 < 256 ? 32 : 64;
}

// The two launches use r (d doubles), a partial norm per column block and the
// counter of blocks done (a 32-bit word): 70 KB at d = 8192.  The size that
// callers are told stays the one they always were: r, a norm for each 64 columns, a
// 32-bit word for each and one more, and, while there are at most 512 groups of 64 columns
// (d <= 32768), two to eight sets of sixteen 64-column sums for each; never less than
// is used, since 32-column blocks end at d = 16320.
int64_t toy_workspace_bytes(int64_t d)
{
    const int64_t cols64 = (d + kWave - 1) / kWave;
    int64_t sets = (d + kWave - 1) / kWave;
    if (sets > 8) sets = 8;
    if (sets > 1024 / cols64) sets = 1024 / cols64;
    if (sets >= 2) {
        const int64_t rows = ((d + sets - 1) / sets + kWave - 1) / kWave * kWave;
        sets = (d + rows - 1) / rows;
    } else {
        sets = 0;
    }
    if (sets < 2) sets = 0;
    return (d + cols64 + (cols64 + 2) / 2 + cols64 * sets * 16 * kWave) * (int64_t)sizeof(double);
}

namespace {

// The residual launch (which also clears the counter), then the round
// kernel, with the round (ROUND) or writing the gradients only.
template <bool ROUND>
hipError_t launch_toy(ToyArgs& a, const float* xs, const float* x, void* workspace, hipStream_t s)
{
    const int64_t d = a.d;
    const int cols = toy_cols(d);
    a.nblk = (int32_t)((d + cols - 1) / cols);
    double* res = static_cast<double*>(workspace);
    a.res = res;
    a.part = res + d;
    a.counter = reinterpret_cast<uint32_t*>(res + d + a.nblk);
    hipLaunchKernelGGL(toy_residual_kernel, dim3((unsigned)((d + kResWaves - 1) / kResWaves)),
                       dim3(kResWaves * kWave), 0, s, d, a.A, xs, x, res, a.counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((a.nblk + 7) / 8 * 8)), block(kTRWaves * kWave);
    if (cols == 32)
        hipLaunchKernelGGL((toy_round_kernel<2, 2, 1, ROUND>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((toy_round_kernel<4, 1, 2, ROUND>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_toy_grad(int64_t d, int32_t N, const float* A, const float* xs, const float* xi, const float* x,
                           float* g, double* grad_sq, void* workspace, hipStream_t s)
{
    ToyArgs a{};
    a.d = d;
    a.N = N;
    a.A = A;
    a.xi = xi;
    a.g_out = g;
    a.grad_sq = grad_sq;
    return launch_toy<false>(a, xs, x, workspace, s);
}

hipError_t launch_toy_step(const StepArgs& sa, const float* A, const float* xs, const float* xi, double* grad_sq,
                           float* g_out, void* workspace, hipStream_t s)
{
    ToyArgs a{};
    a.d = sa.d;
    a.N = sa.N;
    a.placement = sa.placement;
    a.beta1 = sa.beta1;
    a.beta2 = sa.beta2;
    a.lr = sa.lr;
    a.qw = sa.qw;
    a.qs = sa.qs;
    a.A = A;
    a.xi = xi;
    a.x = sa.x;
    a.e_w = sa.e_w;
    a.m_w = sa.m_w;
    a.v_w = sa.v_w;
    a.m = sa.m;
    a.v = sa.v;
    a.e_s = sa.e_s;
    a.wcodes = sa.wcodes;
    a.scodes = sa.scodes;
    a.grad_sq = grad_sq;
    a.g_out = g_out;
    return launch_toy<true>(a, xs, sa.x, workspace, s);
}

}  // namespace ea
