// ea_kernels.hip -- the generic and fully specialized fused-round kernels,
// the split calls' kernels, and the launchers (dispatch to the kernel that
// matches a configuration).  The round itself is in ea_round.hpp.
#include "ea_round.hpp"

namespace ea {

namespace {

// A block's partial norm from its waves' (each a tile's), in wave order.
__device__ __forceinline__ void store_block_part(double part, int norm, double* out)
{
    __shared__ double red[kWavesPerBlock];
    if (lane_id() == 0) red[wave_id()] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = red[0];
        for (int w = 1; w < kWavesPerBlock; ++w) tot = norm == S_MAX ? fmax(tot, red[w]) : tot + red[w];
        *out = tot;
    }
}

// Partial norms of the workers' inputs p, one per worker (i0 + blockIdx.y, its
// row of a.g etc.) and block of tiles, without writing any state (one-bucket Q_w).
template <int C>
__global__ __launch_bounds__(kBlock) void worker_partials_kernel(StepArgs args, int i0)
{
    const StepArgs a = with_step(args);
    const int64_t i = i0 + (int)blockIdx.y, row = i * a.d;
    TilePos t;
    double part = 0.0;
    if (tile_pos<C>(a, t)) {
        WorkerRows<C> r;
        float4 p[C];
        // without the hint: the round reads the same rows next
        load_worker<C, -1, false>(
            a, worker_span<-1>(a, a.g + row, a.e_w + row, a.m_w + row, a.v_w + row, t.base, t.left), 0, r);
        worker_p<C, -1>(a, r, p);
        part = tile_partial<C>(a.qw, p);
    }
    store_block_part(part, a.qw.norm, a.wpart + i * a.wnp + blockIdx.x);
}

// Partial norms of q = u + e_s, one per tile as the fused round leaves them
// (one-bucket Q_s, split call): the same partials, added in the same order,
// make the split call's scale the round's to the last bit.
template <int C>
__global__ __launch_bounds__(kBlock) void server_partials_kernel(StepArgs a)
{
    TilePos t;
    if (!tile_pos<C>(a, t)) return;
    const Row u = row_of(a.ubuf + t.base, t.left), e = row_of(a.e_s + t.base, t.left);
    float4 q[C];
#pragma unroll
    for (int ch = 0; ch < C; ++ch) q[ch] = add4(ld4<false>(u, ch), ld4<false>(e, ch));
    const double part = tile_partial<C>(a.qs, q);
    if (lane_id() == 0) a.spart[t.tile] = part;
}

// Reduce partials to one scale per vector: block v handles part[v*nparts ..
// (v+1)*nparts) and writes out[v*out_stride].  One block per vector, so bound
// by latency: 16 waves with eight loads of each thread in flight (5,395 tiles
// 7.3 -> 4.6 us against 4 waves with one).
constexpr int kFinalWaves = 16;
__global__ __launch_bounds__(kFinalWaves * kWave) void finalize_kernel(const double* __restrict__ part, int64_t nparts,
                                                                       int32_t norm, int64_t n,
                                                                       float* __restrict__ out, int64_t out_stride)
{
    __shared__ double red[kFinalWaves];
    const double* pv = part + (int64_t)blockIdx.x * nparts;
    constexpr int U = 8;
    double acc = 0.0;
    for (int64_t j0 = threadIdx.x; j0 < nparts; j0 += U * kFinalWaves * kWave) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = j0 + (int64_t)u * kFinalWaves * kWave;
            v[u] = pv[j < nparts ? j : j0];
            v[u] = j < nparts ? v[u] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = norm == S_MAX ? fmax(acc, v[u]) : acc + v[u];
    }
    if (norm == S_MAX) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc = fmax(acc, __shfl_xor(acc, o, kWave));
    } else {
        acc = wave_sum(acc);
    }
    if (lane_id() == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = red[0];
        for (int w = 1; w < kFinalWaves; ++w) tot = norm == S_MAX ? fmax(tot, red[w]) : tot + red[w];
        out[(int64_t)blockIdx.x * out_stride] = scale_from(norm, tot, (float)tot, n);
    }
}

__global__ void fill_kernel(float* __restrict__ p, int64_t n, float value)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

__global__ void advance_kernel(uint32_t* t_dev)
{
    if (threadIdx.x == 0) t_dev[0] = t_dev[0] + 1u;
}

int64_t grid_of(const StepArgs& a)
{
    return (a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
}

// Dispatch on C to a generic kernel template instance.
#define EA_DISPATCH(KERNEL, C, GRID, STREAM, ...)                                                    \
    do {                                                                                           \
        switch (C) {                                                                               \
        case 1: hipLaunchKernelGGL((KERNEL<1>), dim3(GRID), dim3(kBlock), 0, STREAM, __VA_ARGS__); break; \
        case 2: hipLaunchKernelGGL((KERNEL<2>), dim3(GRID), dim3(kBlock), 0, STREAM, __VA_ARGS__); break; \
        case 4: hipLaunchKernelGGL((KERNEL<4>), dim3(GRID), dim3(kBlock), 0, STREAM, __VA_ARGS__); break; \
        case 8: hipLaunchKernelGGL((KERNEL<8>), dim3(GRID), dim3(kBlock), 0, STREAM, __VA_ARGS__); break; \
        default: return hipErrorInvalidValue;                                                      \
        }                                                                                          \
    } while (0)

// Specialized fused rounds: (chunks per tile, worker traits, server traits,
// placement), chosen when the configuration matches exactly.
using SignQ8 = QCt<Q_SCALED_SIGN, 1, S_L1, 8>;
using SignQ4 = QCt<Q_SCALED_SIGN, 1, S_L1, 4>;
using SignQ2 = QCt<Q_SCALED_SIGN, 1, S_L1, 2>;
using Stoch4L2Q2 = QCt<Q_STOCH, 4, S_L2, 2>;
using Stoch2MaxQ2 = QCt<Q_STOCH, 2, S_MAX, 2>;
using Stoch2MaxQ4 = QCt<Q_STOCH, 2, S_MAX, 4>;
using TopKQ2 = QCt<Q_TOPK, 1, S_MAX, 2>;
using RandKQ2 = QCt<Q_RANDK, 1, S_MAX, 2>;

struct Special {
    int C;
    int wkind, wbits, wnorm, wcpb;
    int skind, sbits, snorm, scpb;
    int placement;
    void (*kernel)(StepArgs);
    int tiles;                  // tiles per block of `kernel`
};

#define EA_SPECIAL(CC, QWT, QST, PLC)                                                               \
    Special{CC, QWT::kind(QDev{}), QWT::bits(QDev{}), QWT::norm(QDev{}), QWT::cpb(QDev{}),         \
            QST::kind(QDev{}), QST::bits(QDev{}), QST::norm(QDev{}), QST::cpb(QDev{}), PLC,         \
            step_kernel<CC, QWT, QST, PLC>, round_tiles_per_block(CC, PLC == AT_SERVER)}

const Special kSpecials[] = {
    EA_SPECIAL(2, Stoch4L2Q2, Stoch4L2Q2, AT_SERVER),
    EA_SPECIAL(2, Stoch4L2Q2, Stoch4L2Q2, AT_WORKER),
    EA_SPECIAL(2, Stoch2MaxQ2, Stoch2MaxQ2, AT_SERVER),
    EA_SPECIAL(2, Stoch2MaxQ2, Stoch2MaxQ2, AT_WORKER),
    EA_SPECIAL(8, SignQ8, SignQ8, AT_SERVER),
    EA_SPECIAL(8, SignQ8, SignQ8, AT_WORKER),
    EA_SPECIAL(4, Stoch2MaxQ4, SignQ4, AT_SERVER),
    EA_SPECIAL(4, Stoch2MaxQ4, SignQ4, AT_WORKER),
    EA_SPECIAL(2, SignQ2, SignQ2, AT_SERVER),
    EA_SPECIAL(2, TopKQ2, TopKQ2, AT_SERVER),
    EA_SPECIAL(2, RandKQ2, RandKQ2, AT_SERVER),
};

const Special* find_special(const StepArgs& a, int C)
{
    for (const Special& s : kSpecials) {
        if (s.C == C && s.placement == a.placement && s.wkind == a.qw.kind && s.wbits == a.qw.bits &&
            s.wnorm == a.qw.norm && s.wcpb == a.qw.cpb && s.skind == a.qs.kind && s.sbits == a.qs.bits &&
            s.snorm == a.qs.norm && s.scpb == a.qs.cpb)
            return &s;
    }
    return nullptr;
}

// The specialized tables' entry for quantizer q at tile size C, when one
// matches: tiles of one bucket of q each, of any size for full precision and
// for Example 2 with 4- or 5-bit codes, of two chunks for a quantizer with one
// bucket over the whole vector.  The rest of these takes the generic kernels:
// Example 2 with other code widths (40M parameters, 16 workers: 3 bits 2376 us
// and 8 bits 3021, against 1620 for 4 bits), and one-bucket workers beside
// server buckets of 256, 1024 or 2048 elements (18.1M, 16 workers: 1180, 1555
// and 1980 us, against 1078 beside 512).  find_half keys on the worker
// quantizer (the fused round and the split worker calls); the split server
// calls key on the server's.
const HalfKernel* find_half_for(const QDev& q, int C)
{
    const bool sparse = q.kind == Q_TOPK || q.kind == Q_RANDK;
    if (q.cpb != 0 && q.cpb != C) return nullptr;
    const int norm = q.cpb == 0 || sparse ? S_MAX : q.norm;   // as the tables write it
    for (int wide = 0; wide < 2; ++wide) {
        int n = 0;
        const HalfKernel* t = wide ? (C <= 2 ? half_kernels_wide_c12(&n) : half_kernels_wide_c48(&n))
                            : C == 1 ? half_kernels_c1(&n) : C == 2 ? half_kernels_c2(&n)
                            : C == 4 ? half_kernels_c4(&n) : C == 8 ? half_kernels_c8(&n) : nullptr;
        for (int i = 0; i < n; ++i) {
            const HalfKernel& h = t[i];
            if (h.C == C && h.wkind == q.kind && h.wbits == q.bits && h.wnorm == norm && h.wcpb == q.cpb) return &h;
        }
    }
    return nullptr;
}

const HalfKernel* find_half(const StepArgs& a, int C)
{
    return find_half_for(a.qw, C);
}

// A fully specialized kernel for a wide tile with the same quantizer on both
// sides and Adam at the server, when one matches.
const SymKernel* find_sym(const StepArgs& a, int C)
{
    if (a.placement != AT_SERVER || (C != 4 && C != 8)) return nullptr;
    const QDev& w = a.qw;
    const QDev& v = a.qs;
    if (w.kind != v.kind || w.bits != v.bits || w.norm != v.norm || w.cpb != v.cpb || w.cpb != C) return nullptr;
    int n = 0;
    const SymKernel* t = C == 4 ? sym_kernels_c4(&n) : sym_kernels_c8(&n);
    for (int i = 0; i < n; ++i)
        if (t[i].kind == w.kind && t[i].bits == w.bits && t[i].norm == w.norm && t[i].cpb == w.cpb) return &t[i];
    return nullptr;
}

// Waves per block of a fused-round launch: one per worker up to the tile's
// limit, and at least one per tile of the block, since wave k serves tile k
// (with fewer workers than tiles the other waves only serve).  Fully
// specialized 8-chunk tiles serve a whole-tile server bucket, or a
// sparsifier's server side, on C waves, one chunk each (SplitServe,
// SparseServe), so their blocks have C waves
// at least.
int step_waves(const StepArgs& a, int C, int K, const Special* sp, const SymKernel* sk, size_t limit)
{
    int G = round_waves(a.N, C, K, limit, a.placement);
    if (G < K) G = K;
    const bool scaled = a.qs.cpb == C &&
                        (a.qs.kind == Q_SCALED_SIGN || a.qs.kind == Q_STOCH || a.qs.kind == Q_DET);
    const bool sparse = a.qs.kind == Q_TOPK || a.qs.kind == Q_RANDK;
    const bool split = (sp || sk) && C == 8 && (scaled || sparse);
    return split && G < C ? C : G;
}

// Rows whose byte length is not a multiple of 128 share a cache line between
// adjacent tiles.  Launches of one tile per block then deal runs
// of this many adjacent tiles to each XCD (block_slot): ResNet-18-sized
// round 0.2930 -> 0.2847 ms (runs of 8: 0.2880, 32: 0.2863).  With two
// tiles per block the pair's shared line is inside the block already, and
// runs measured slower (ResNet-50-sized 2.108 -> 2.155-2.187 ms).
#ifndef EA_XCD_RUN
#define EA_XCD_RUN 16
#endif

// LDS that a block of G waves asks for at least.  Full-precision rounds have no
// arithmetic to hide, and the more of their blocks a CU holds the less of HBM
// they reach: two 8-wave blocks or their like, and not a third beside two that
// end.  With Adam at two workers and more at any size (8 workers, 1M parameters
// 51.6 -> 50.9 us, 16M 913 -> 901, 40M 2128 -> 2086; one worker, 355M 3264 ->
// 3308); with Adam at the server, where a
// block's waves wait longer for each other, once the rows are long (8 workers,
// 40M 1138 -> 1090, 4 workers, 110M 1948 -> 1891, but 4M 125.7 -> 128.4).  Blocks
// of more than 8 waves fill a CU by themselves, and the kernels with codes need
// the others (Example 2, 8 workers, 40M 941 -> 1273).
size_t least_lds(const StepArgs& a, int C, int G)
{
    const bool full = a.qw.kind == Q_NONE && C == 2 && G <= 8;
    const bool pays = a.placement == AT_WORKER ? a.N > 1 : a.N * a.d >= (int64_t)1 << 28;
    return full && pays ? (size_t)G * 8000 : 0;
}

// One dispatch covers at most 2^32 - 1 work-items, and the fused kernels run
// up to four threads per element (one-chunk tiles, 16 waves, one tile per
// block), so a round is launched in pieces of at most this many blocks (2^30
// threads): one piece up to d = 2^28 in that shape, 2^30 in the BERT-sized
// one.  Pieces are multiples of 128 blocks, so the XCD runs of block_slot
// keep their groups.
constexpr int64_t kMaxLaunchBlocks = (int64_t)1 << 20;

}  // namespace

// The round's kernel: one specialized for both quantizers and the placement
// when one matches, else one specialized for the worker quantizer, else the
// generic one.  One launch takes every tile.
hipError_t launch_step(const StepArgs& a, int C, hipStream_t s)
{
    const size_t limit = lds_limit_bytes();
    const Special* sp = find_special(a, C);
    const SymKernel* sk = sp ? nullptr : find_sym(a, C);
    const HalfKernel* hk = sp || sk ? nullptr : find_half(a, C);
    const int K = sp ? sp->tiles : sk ? sk->tiles : hk ? hk->tiles : kernel_tiles(C, -1, false);
    const int G = step_waves(a, C, K, sp, sk, limit);
    StepArgs b = a;
    const int bufs = handoff_bufs(a.N, C, G, K, limit);
    b.one_buffer = bufs == 1 ? 1 : 0;
    b.xcd_run = (a.d * 4) % 128 != 0 && K == 1 ? EA_XCD_RUN : 1;
    const dim3 block((unsigned)(G * kWave));
    size_t lds = round_lds_bytes(a.N, C, G, K, bufs);
    if (hk && lds < least_lds(a, C, G)) lds = least_lds(a, C, G);
    const int64_t nblocks = (a.ntiles + K - 1) / K;
    for (int64_t b0 = 0; b0 < nblocks; b0 += kMaxLaunchBlocks) {
        const dim3 grid((unsigned)(nblocks - b0 < kMaxLaunchBlocks ? nblocks - b0 : kMaxLaunchBlocks));
        b.tile0 = b0 * K;
        if (sp || sk || hk) {
            hipLaunchKernelGGL(sp ? sp->kernel : sk ? sk->kernel : hk->kernel, grid, block, lds, s, b);
        } else {
            switch (C) {
            case 1: hipLaunchKernelGGL((step_kernel<1, QRt, QRt, -1>), grid, block, lds, s, b); break;
            case 2: hipLaunchKernelGGL((step_kernel<2, QRt, QRt, -1>), grid, block, lds, s, b); break;
            case 4: hipLaunchKernelGGL((step_kernel<4, QRt, QRt, -1>), grid, block, lds, s, b); break;
            case 8: hipLaunchKernelGGL((step_kernel<8, QRt, QRt, -1>), grid, block, lds, s, b); break;
            default: return hipErrorInvalidValue;
            }
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_worker_partials(const StepArgs& a, int C, int nworkers, hipStream_t s)
{
    // in pieces of at most 2^30 threads, as the round (or of one worker)
    const int64_t per = ((int64_t)1 << 22) / grid_of(a);
    for (int i0 = 0; i0 < nworkers;) {
        const int ny = per < 1 ? 1 : per < nworkers - i0 ? (int)per : nworkers - i0;
        const dim3 grid((unsigned)grid_of(a), (unsigned)ny);
        EA_DISPATCH(worker_partials_kernel, C, grid, s, a, i0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        i0 += ny;
    }
    return hipSuccess;
}

hipError_t launch_server_partials(const StepArgs& a, int C, hipStream_t s)
{
    EA_DISPATCH(server_partials_kernel, C, grid_of(a), s, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const double* part, int64_t nparts, int32_t norm, int64_t n, float* out,
                           int64_t out_stride, int nvec, hipStream_t s)
{
    hipLaunchKernelGGL(finalize_kernel, dim3(nvec), dim3(kFinalWaves * kWave), 0, s, part, nparts, norm, n, out,
                       out_stride);
    return hipGetLastError();
}

// The split calls on the worker side use a kernel specialized for the worker
// quantizer when one matches, else the generic one.
hipError_t launch_worker(const StepArgs& a, int C, hipStream_t s)
{
    const HalfKernel* hk = find_half(a, C);
    if (hk) {
        hipLaunchKernelGGL(hk->worker, dim3((unsigned)grid_of(a)), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    EA_DISPATCH(worker_kernel, C, grid_of(a), s, a);
    return hipGetLastError();
}

hipError_t launch_aggregate(const StepArgs& a, int C, hipStream_t s)
{
    if (const HalfKernel* hk = find_half(a, C)) {
        hipLaunchKernelGGL(hk->aggregate, dim3((unsigned)grid_of(a)), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    EA_DISPATCH(aggregate_kernel, C, grid_of(a), s, a);
    return hipGetLastError();
}

// The split server calls take the worker-specialized tables' kernels for the
// server quantizer when it is one of theirs.
hipError_t launch_server(const StepArgs& a, int C, hipStream_t s)
{
    const HalfKernel* hk = find_half_for(a.qs, C);
    if (hk) {
        hipLaunchKernelGGL(hk->server, dim3((unsigned)grid_of(a)), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    EA_DISPATCH(server_kernel, C, grid_of(a), s, a);
    return hipGetLastError();
}

hipError_t launch_apply(const StepArgs& a, int C, hipStream_t s)
{
    const HalfKernel* hk = find_half_for(a.qs, C);
    if (hk) {
        hipLaunchKernelGGL(hk->apply, dim3((unsigned)grid_of(a)), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    EA_DISPATCH(apply_kernel, C, grid_of(a), s, a);
    return hipGetLastError();
}

hipError_t launch_advance(uint32_t* t_dev, hipStream_t s)
{
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(kWave), 0, s, t_dev);
    return hipGetLastError();
}

hipError_t launch_fill(float* p, int64_t n, float value, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 1023) / 1024;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, value);
    return hipGetLastError();
}

}  // namespace ea
