// gl_lib.hip -- kernels and C ABI of the oblate transit light-curve library.
//
// One gl_lightcurve_batch call (all on the caller's stream):
//   k_prep      one thread per parameter set: domain checks, derived constants
//               (projected ellipse from eqs. dx, dy1, dy2, orbit, limb darkening),
//               CSR segment checks, number of workgroups per set.
//   k_scan      one workgroup: exclusive scan of those counts (CSR only, more
//               than 256 sets: k_prep's one workgroup scans fewer itself).
//   k_flux      everything else in one launch: window, classification, flux
//               integrals and averages (see "the fused pass").
// A surrogate batch adds the network's inference and k_net_sum, a likelihood
// batch the likelihood kernel.  A batch too large for one launch runs as
// passes over ranges of its sets.  The launches are captured once into a HIP
// graph and replayed while the arguments stay the same.
//
// The paper's own integrator (gl_lightcurve_batch_snap) runs k_prep, k_scan,
//   k_window    outputs whose exposure cannot overlap the star are written as
//               1; a mask of the others is kept per 64 outputs, and
//   k_snap      which integrates those.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "gl.h"
#include "gl_device.h"
#include "gl_index.h"
#include "gl_internal.h"
#include "gl_room.h"

namespace {

constexpr int kChunk = 64;
constexpr int kScanThreads = 1024;

constexpr int kCensus = 11;

// Counters that every wavefront of a launch adds to are split into kShards
// shards on lines of their own (one address for all of them serialises the
// atomics at L2); the host sums them.
constexpr int kShards = 64;

struct alignas(128) LineCount {
    unsigned long long v;
    unsigned long long pad[15];
};

struct Counters {
    unsigned long long total_chunks;  // own grids: workgroups or chunks (k_prep, k_scan)
    unsigned int status;              // bit 0: invalid set, bit 1: bad CSR segment, bit 2: non-finite time
    unsigned int pad;
    // arcs accepted at the arc rule's last level above its tolerance, summed
    // over every batch since gl_ctx_get_unconverged last read it
    unsigned long long unconverged;
    unsigned long long net_total;     // rows the current pass's network batch asks for
    unsigned long long net_most;      // and the most a pass of this context asked for
    double ll_norm;                   // likelihood batches on a shared grid: sum log(sigma) + (N/2) log(2 pi)
    // work census (census launches only): in-window sub-samples, whole-on-star,
    // intersecting, in-window but off the star, trapezoid nodes of the rigorous
    // rule, arc-rule evaluations, roots found, limb arcs, nodes of the
    // near-limb rule, ellipse arcs, arcs accepted unconverged
    LineCount census[kCensus][kShards];
    LineCount sur[3][kShards];        // surrogate batches: in-window sub-samples, of those
                                      // reaching the disk, of those accepted by the gate
    LineCount clocks[7][kShards];     // timed batches: wavefront clocks of the fused pass's stages
};

// Outputs per workgroup of the fused pass on a CSR grid: within [128, most], and
// 2 most sub-samples (2048 own grids of mixed supersampling, most = 2048: 1070
// us at 2048 sub-samples, where a workgroup's fixed part shows, 1029 at 4096,
// 1070 at 8192 and 1208 at 16384, where the last ones hold the launch up; with
// the smaller ones at the end, see most_of, 971 at 4096 and 947 at 8192).
constexpr int kFluxMinRange = 128;
// Fewer outputs where the workgroups would not fill the chip: a range is halved as
// often as the launch has room for (flux_halvings), down to kFluxFew sub-samples
// (768: 16 sets of 3000 x 3 60 us, 44 at 512; 256: 256 sets of 1000 x 3 57, 50 at 512).
constexpr int kFluxFew = 512;
__host__ __device__ __forceinline__ int flux_halved(int range, int nss, int halvings)
{
    for (int h = 0; h < halvings && range * nss > kFluxFew; ++h) range = ((range >> 1) + 1) & ~1;
    return range;
}

__device__ __forceinline__ int flux_range_of(int most, int nss, int halvings)
{
    int r = kFluxMinRange;
    while (r * nss <= most && 2 * r <= most) r *= 2;
    return flux_halved(r, nss, halvings);
}

// The last eighth of a batch's own grids takes workgroups a quarter as large,
// which evens out the launch's end (2048 own grids: 1006 us without, 987; a
// shared grid's smaller workgroups cost more than its end: 246 -> 286 us for
// 4096 sets of 1009).
__device__ __forceinline__ int most_of(int most, int64_t s, int64_t n_sets)
{
    return s < n_sets - n_sets / 8 ? most : most / 4;
}

// ---------------------------------------------------------------- kernels
// A batch runs as one or more passes over consecutive ranges of its
// parameter sets (the whole pipeline per pass); `ld` is the row stride of the
// parameter block, `first` / `last` mark the batch's first and last pass
// (CSR end checks).
// SHAPE 0: the oblate block (GL_NPARAM rows), 1: general ellipsoids, 2: MCMC
// walkers (converted to the oblate block); one instance per block kind.
template <int SHAPE>
__global__ void k_prep(const double* __restrict__ params, int64_t ld, int64_t n_sets,
                       const int64_t* __restrict__ offsets, int64_t n_times,
                       const int32_t* __restrict__ n_ss, const double* __restrict__ t_exp,
                       gl::SetConst* __restrict__ sc, int64_t* __restrict__ seg_begin,
                       int64_t* __restrict__ seg_len, int64_t* __restrict__ chunk_off,
                       Counters* __restrict__ ctr, int64_t cps_shared, int first, int last,
                       gl::SetConst* __restrict__ sph, const double* __restrict__ sigma,
                       int64_t n_sigma, double* __restrict__ norm, int fused_range, int halvings, int64_t scan_most,
                       int clear)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s == 0) ctr->net_total = 0ull;
    if (clear) {  // the counters of census, surrogate and timed batches
        const int64_t step = (int64_t)gridDim.x * blockDim.x;
        for (int64_t i = s; i < (int64_t)(kCensus + 3) * kShards; i += step) {
            const int64_t r = i / kShards, j = i % kShards;
            (r < kCensus ? ctr->census[r][j] : ctr->sur[r - kCensus][j]).v = 0ull;
        }
        for (int64_t i = s; i < (int64_t)7 * kShards; i += step) ctr->clocks[i / kShards][i % kShards].v = 0ull;
    }
    if (norm && blockIdx.x == gridDim.x - 1) {
        // the extra last workgroup: a shared grid's likelihood normalisation
        // sum log(sigma) + (N/2) log(2 pi), in a fixed order
        __shared__ double part[256 / 64];
        double acc = 0.0;
        for (int64_t i = threadIdx.x; i < n_sigma; i += blockDim.x) acc += log(sigma[i]);
        for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0)
            norm[0] = ((part[0] + part[1]) + (part[2] + part[3])) + 0.5 * (double)n_sigma * 1.8378770664093454836;
        return;
    }
    int64_t count = 0;
    if (s < n_sets) {
        constexpr int rows = SHAPE == 1 ? gl::kEllParams : GL_NPARAM;
        double p[rows];
#pragma unroll
        for (int i = 0; i < rows; ++i) p[i] = params[(int64_t)i * ld + s];
        if (SHAPE == 2) {
            double w[gl::kWalkParams];
#pragma unroll
            for (int i = 0; i < gl::kWalkParams; ++i) w[i] = p[i];
            gl::walker_to_params(w, p);
        }
        const int nss = n_ss ? n_ss[s] : 1;
        const double te = t_exp ? t_exp[s] : 0.0;
        gl::SetConst c;
        bool ok;
        if constexpr (SHAPE == 1) ok = gl::make_set_const_ell(p, te, nss, c);
        else ok = gl::make_set_const(p, te, nss, c);
        int64_t b, e;
        unsigned int flag = ok ? 0u : 1u;
        if (offsets) {
            b = offsets[s];
            e = offsets[s + 1];
            bool seg_ok = (b >= 0) && (e >= b) && (e <= n_times);
            if (s == 0 && first) seg_ok = seg_ok && (b == 0);
            if (s == n_sets - 1 && last) seg_ok = seg_ok && (e == n_times);
            if (!seg_ok) {
                b = 0;
                e = 0;
                flag |= 2u;
            }
        } else {
            b = s * n_times;
            e = b + n_times;
        }
        if (flag) atomicOr(&ctr->status, flag);
        sc[s] = c;
        if (sph) sph[s] = gl::sphere_of(c);
        // (the fused pass takes a shared grid's places from the set's number)
        if (offsets || !fused_range) {
            seg_begin[s] = b;
            seg_len[s] = e - b;
        }
        if (cps_shared > 0) {
            // shared grid, every set has cps_shared chunks: the exclusive scan in
            // closed form (no k_scan launch)
            chunk_off[s] = s * cps_shared;
            if (s == n_sets - 1) {
                chunk_off[n_sets] = n_sets * cps_shared;
                ctr->total_chunks = (unsigned long long)(n_sets * cps_shared);
            }
        } else if (offsets) {
            const int64_t per = fused_range ? flux_range_of(most_of(fused_range, s, n_sets), ok ? nss : 1, halvings) : kChunk;
            count = (e - b + per - 1) / per;
            if (!scan_most) chunk_off[s] = count;
        }
    }
    if (scan_most) {
        // one workgroup holds every set: k_scan's work here (its launch took
        // 2.6 us and the gap before it of the 38 that 37 locked sets of 700
        // outputs took)
        __shared__ int64_t sums[256 / 64];
        int64_t incl = count;
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t v = __shfl_up((long long)incl, d);
            if ((threadIdx.x & 63) >= d) incl += v;
        }
        if ((threadIdx.x & 63) == 63) sums[threadIdx.x >> 6] = incl;
        __syncthreads();
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) incl += sums[w];
        if (s < n_sets) chunk_off[s] = incl - count;
        if (s == n_sets - 1) {
            if (incl > scan_most) {  // as in k_scan
                atomicOr(&ctr->status, 2u);
                incl = 0;
            }
            chunk_off[n_sets] = incl;
            ctr->total_chunks = (unsigned long long)incl;
        }
    }
}

// exclusive scan of chunk_off[0..n) in place; chunk_off[n] = total.  A total
// above the workspace capacity (only possible when CSR offsets decrease and
// later segments overlap earlier ones) schedules no work and is reported.
__global__ void __launch_bounds__(kScanThreads)
k_scan(int64_t* __restrict__ chunk_off, int64_t n, int64_t max_chunks, Counters* __restrict__ ctr)
{
    __shared__ int64_t part[kScanThreads];
    const int tid = threadIdx.x;
    const int64_t per = (n + kScanThreads - 1) / kScanThreads;
    const int64_t lo = std::min<int64_t>(n, per * tid), hi = std::min<int64_t>(n, lo + per);
    int64_t sum = 0;
    for (int64_t i = lo; i < hi; ++i) sum += chunk_off[i];
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < kScanThreads; d <<= 1) {
        const int64_t v = (tid >= d) ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t run = part[tid] - sum;  // exclusive prefix of this thread's range
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t v = chunk_off[i];
        chunk_off[i] = run;
        run += v;
    }
    if (tid == kScanThreads - 1) {
        int64_t total = part[tid];
        if (total > max_chunks) {
            atomicOr(&ctr->status, 2u);
            total = 0;
        }
        chunk_off[n] = total;
        ctr->total_chunks = (unsigned long long)total;
    }
}

__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)(v & 0xffffffffll));
    const unsigned int hi = __builtin_amdgcn_readfirstlane((unsigned int)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Set bits of m below the calling lane (mbcnt: no lane mask is kept live).
__device__ __forceinline__ int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Adds a wave's census counts (one atomic per counter).
__device__ __forceinline__ void census_add(Counters* ctr, int idx, unsigned long long v)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(&ctr->census[idx][blockIdx.x % kShards].v, v);
}

// Adds a wave's count of unconverged arcs (and to the census in census launches).
__device__ __forceinline__ void unconverged_add(Counters* ctr, int v, bool census)
{
    unsigned long long u = (unsigned long long)v;
    for (int d = 32; d >= 1; d >>= 1) u += __shfl_xor(u, d);
    if ((threadIdx.x & 63) == 0 && u) {
        atomicAdd(&ctr->unconverged, u);
        if (census) atomicAdd(&ctr->census[10][blockIdx.x % kShards].v, u);
    }
}

// ---------------------------------------------------------------- the paper's integrator
// Window test: outputs whose exposure cannot overlap the star are written as
// 1 (NaN for an invalid set or a non-finite time); a 64-bit mask of the others
// and the chunk's set are kept.

// One time grid for every set: one wavefront per kWinGrid consecutive chunks
// of one set (bx = ceil(chunks per set / kWinGrid) wavefronts per set, set
// major);
// every time load is issued before the first test, and lane k keeps chunk k's
// mask for one store of all of them.
constexpr int kWinGrid = gl::kWinGridChunks;

__global__ void __launch_bounds__(64)
k_window_grid(const double* __restrict__ times, int64_t n_times, int64_t cps,
              const gl::SetConst* __restrict__ sc, Counters* __restrict__ ctr,
              unsigned long long* __restrict__ masks, int* __restrict__ chunk_set,
              double* __restrict__ out)
{
    const int lane = threadIdx.x;
    int64_t s, lc0;  // the set and its first chunk here
    int nk;
    gl::window_grid_block(blockIdx.x, cps, kWinGrid, s, lc0, nk);
    const int64_t ob = s * n_times;  // the set's first output (its segment start)
    const gl::SetConst& S = sc[s];
    double t[kWinGrid];
#pragma unroll
    for (int k = 0; k < kWinGrid; ++k) {
        const int64_t pos = (lc0 + k) * kChunk + lane;
        t[k] = (k < nk && pos < n_times) ? times[pos] : 0.0;
    }
    const bool valid = S.valid;
    const double reach = S.half_win + 0.5 * S.t_exp;
    unsigned long long my_mask = 0ull;
#pragma unroll
    for (int k = 0; k < kWinGrid; ++k) {
        const int64_t pos = (lc0 + k) * kChunk + lane;
        bool work = false;
        if (k < nk && pos < n_times) {
            if (!valid || !gl::finite_d(t[k])) {
                out[ob + pos] = __builtin_nan("");
                if (valid) atomicOr(&ctr->status, 4u);
            } else {
                work = fabs(gl::phase_time(S, t[k])) < reach;
                // streamed past the caches: the 1s are never read back
                if (!work) __builtin_nontemporal_store(1.0, out + ob + pos);
            }
        }
        const unsigned long long m = __ballot(work);
        if (lane == k) my_mask = m;
    }
    const int64_t c = s * cps + lc0 + lane;  // lane k: chunk k
    if (lane < nk) {
        masks[c] = my_mask;
        chunk_set[c] = (int)s;
    }
}

// CSR segments: one wavefront per group of kWinChunks consecutive chunks (their
// memory operations overlap), the set of the first chunk found by binary
// search and stepped along from there.
constexpr int kWinChunks = gl::kWinCsrChunks;

__global__ void __launch_bounds__(256)
k_window(const double* __restrict__ times, int64_t n_sets,
         const gl::SetConst* __restrict__ sc, const int64_t* __restrict__ seg_begin,
         const int64_t* __restrict__ seg_len, const int64_t* __restrict__ chunk_off,
         Counters* __restrict__ ctr, unsigned long long* __restrict__ masks,
         int* __restrict__ chunk_set, double* __restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t total = (int64_t)ctr->total_chunks;
    const int64_t g = (int64_t)blockIdx.x * 4 + wv;
    const int64_t c_first = g * kWinChunks;
    int64_t s = 0;
    if (c_first < total) s = uniform64(gl::set_of_chunk(chunk_off, n_sets, c_first));
#pragma unroll
    for (int k = 0; k < kWinChunks; ++k) {
        const int64_t c = c_first + k;
        if (c >= total) continue;
        while (s + 1 < n_sets && chunk_off[s + 1] <= c) ++s;  // uniform
        const int64_t pos = (c - chunk_off[s]) * kChunk + lane;  // position in the segment
        const bool in_seg = pos < seg_len[s];
        const int64_t i = seg_begin[s] + pos;
        const gl::SetConst& S = sc[s];
        bool work = false;
        if (in_seg) {
            const double t = times[i];
            if (!S.valid || !gl::finite_d(t)) {
                out[i] = __builtin_nan("");
                if (S.valid) atomicOr(&ctr->status, 4u);
            } else {
                const double tau = gl::phase_time(S, t);
                work = fabs(tau) < S.half_win + 0.5 * S.t_exp;
                if (!work) __builtin_nontemporal_store(1.0, out + i);
            }
        }
        const unsigned long long m = __ballot(work);
        if (lane == 0) {
            masks[c] = m;
            chunk_set[c] = (int)s;
        }
    }
}

// The paper's integrator over a batch, a workgroup per chunk of 64 outputs
// (wavefront w takes every fourth in-window output from the w-th on): the
// centres of an output's sub-samples are found one per lane, then each
// sub-sample that reaches the disk is integrated by the whole wavefront (node
// i on lane i mod 64, Simpson weight 4 on odd nodes: odd lanes, 2 on even),
// the three sums reduced across the lanes; outputs are box-averaged in FP64
// (the sub-samples off the disk first, then the others in order).  node_cs:
// cos and sin of 2 pi i / n_nodes.
constexpr int kSnapWaves = 4;

__global__ void __launch_bounds__(64 * kSnapWaves)
k_snap(const double* __restrict__ times, int shared_grid, const gl::SetConst* __restrict__ sc,
       const int64_t* __restrict__ seg_begin, const int64_t* __restrict__ chunk_off, const Counters* __restrict__ ctr,
       const unsigned long long* __restrict__ masks, const int* __restrict__ chunk_set, int n_nodes,
       const float2* __restrict__ node_cs, double* __restrict__ out)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t total = (int64_t)ctr->total_chunks;
    const float wt = (lane & 1) ? 4.0f : 2.0f;
    for (int64_t c = blockIdx.x; c < total; c += gridDim.x) {
        unsigned long long M = (unsigned long long)uniform64((int64_t)masks[c]);
        if (!M) continue;
        for (int w = 0; w < wv; ++w) M &= M - 1ull;  // this wavefront's outputs: the wv-th, wv+4-th, ...
        if (!M) continue;
        const int64_t s = uniform64(chunk_set[c]);
        const gl::SetConst& S = sc[s];
        const gl::ChunkPos cp = gl::chunk_pos(shared_grid != 0, seg_begin[s], c - chunk_off[s]);
        const int nss = S.n_ss;
        const double inv_nss = 1.0 / (double)nss;
        const float A = (float)S.A, B = (float)S.B, C = (float)S.C;
        const double reach2 = (1.0 + S.k) * (1.0 + S.k);
        const float k0 = (float)S.c0, k1 = (float)S.c1 * (2.0f / 3.0f), k2 = (float)S.c2;
        const float scale = (float)(gl::kTwoPi / 3.0) / (float)n_nodes * (float)S.inv_phi;
        while (M) {
            const int o = __builtin_ctzll(M);  // the output (a lane of the chunk)
            for (int w = 0; w < kSnapWaves && M; ++w) M &= M - 1ull;
            const double t = times[cp.time0 + o];
            // lane j: sub-sample j's centre and whether its ellipse can reach the disk
            double x0 = 0.0, y0 = 0.0;
            bool on = false;
            if (lane < nss) {
                on = gl::centre_at(S, t + (((double)lane + 0.5) * inv_nss - 0.5) * S.t_exp, x0, y0);
                on = on && x0 * x0 + y0 * y0 < reach2;
            }
            const unsigned long long todo = __ballot(on);
            double sum = (double)(nss - __popcll(todo));  // sub-samples off the disk: flux 1
            // then, in order of j, the flux of every sub-sample that reaches the disk
            for (int j = 0; j < nss; ++j) {
                if (!((todo >> j) & 1ull)) continue;
                const float xc = (float)__shfl(x0, j), yc = (float)__shfl(y0, j);
                float sf = 0.0f, sl = 0.0f, sq = 0.0f;
                for (int i = lane; i < n_nodes; i += 64) {
                    const float2 q = node_cs[i];
                    float ff, fl, fq;
                    gl::snap_node(A, B, C, xc, yc, q.x, q.y, ff, fl, fq);
                    sf += ff;
                    sl += fl;
                    sq += fq;
                }
                sf *= wt;
                sl *= wt;
                sq *= wt;
                for (int d = 32; d >= 1; d >>= 1) {
                    sf += __shfl_xor(sf, d);
                    sl += __shfl_xor(sl, d);
                    sq += __shfl_xor(sq, d);
                }
                sum += (double)(1.0f - (k0 * sf + k1 * sl + k2 * sq) * scale);
            }
            if (lane == 0) out[cp.out0 + o] = sum * inv_nss;
        }
    }
}

// cos and sin of 2 pi i / n, i < n (from the double-precision functions)
__global__ void k_snap_nodes(int n, float2* __restrict__ cs)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double sn, c;
    sincos(gl::kTwoPi * (double)i / (double)n, &sn, &c);
    cs[i] = float2{(float)c, (float)sn};
}

// ---------------------------------------------------------------- the fused pass
// The whole batch after k_prep in one launch.  A workgroup takes R consecutive
// outputs of one set (its constants are wavefront-uniform), 1024 at a time:
//   window    outputs whose exposure cannot overlap the star are written as 1
//             (NaN for an invalid set or a non-finite time), the others'
//             positions collected in LDS.  Bound by the stores: two outputs
//             per lane and 2048 behind one test, 512 sets of 65536 outputs in
//             90 us (268 MB; 44 for a plain fill), 113 with one output per lane
//             and three branches each;
//   classify  their sub-samples, up to kUnit at a time: time, ellipse centre
//             and class per thread; counting sort by class and rule order in
//             LDS, so that the 64 entries a wavefront takes next are alike;
//   evaluate  tiles of 64 sorted entries, handed out by an LDS counter, the
//             long ones first: crossing ellipses (quartic, closed forms and
//             one arc rule per lane) and whole ellipses (periodic trapezoid);
//             those near the inner tangency, whose rules are long, share an
//             entry between 4 lanes;
//   declined  what the direct rules do not fit (about one sample in 10^4 up to
//             k = 0.2, up to a tenth above k = 0.5), by the general path, 64 of a
//             unit's per wavefront (a whole output per wavefront instead, its
//             sub-samples on as many lanes: 7.6 ms, not 0.54, for 2048 sets of
//             1000 outputs, k 0.95 to 0.999);
//   average   each output's sub-samples in order, straight to `out`.
// Nothing but the inputs and the outputs touches memory.  (The work-list
// pipeline this replaces ran the same stages as eleven launches over lists in
// memory: on the walker batch their traffic, launch gaps and tails were about
// as long as the arithmetic, and a batch of 64 walkers was all gaps.)
// Bound by FP64 issue where transits fill the grid (2048 own grids, 20 M
// outputs: vector units busy about 80 % of the time, 2412 us by the pipeline, 890
// here), by the stores where they do not (512 sets of 65536 outputs, 268 MB:
// 152 us, here 81), by latency at one set of 1000 (90 us, here 16).
// Sizes by the workgroup's wavefronts (see flux_waves): four, or one for many
// sets of a few outputs.
template <int WAVES>
struct FluxSize {
    static constexpr int unit = 256 * WAVES;  // sub-samples sorted at once
    static constexpr int range = WAVES == 1 ? 128 : 4096;  // outputs per workgroup at most
    static constexpr int round = WAVES == 1 ? 128 : 2048;  // outputs whose times are loaded at once
    static_assert(range <= 64 * 128 && range % round == 0 && round % (128 * WAVES) == 0, "128 outputs per lane");
};
constexpr int kFluxWaves = 4;
// two neighbouring outputs: times and fluxes are 8-byte aligned (a 16-byte
// access needs 4 here)
typedef double pair2 __attribute__((ext_vector_type(2), aligned(8)));
// sort buckets, longest first: ellipses near the inner tangency (an arc beyond
// ~172 degrees either side or none), crossing ones in four steps of their arc's length, then
// whole ellipses by falling trapezoid order (the longest few together: 32
// buckets, five bits)
constexpr int kBWide = 0, kBHard = 1, kBWhole = 5;
constexpr int kFluxBuckets = 32;
constexpr int kBTop = kFluxBuckets - kBWhole + 3;  // half orders from here on share a bucket
// Lanes per entry of the first bucket, whose rules are the longest: always the
// same number, so that a sample's bits do not depend on how many others its
// unit holds.  All lanes of an entry set it up, so it has to be the few with
// long rules: with the limit on the arc at cos(delta) = -0.82 2048 own grids take 1016 us,
// 945 at -0.98, 934 at -0.99 and 926 at -1; 64 walkers of 1009 x 3 32.5 at -0.98, 31.6
// at -0.99 and 35.3 at -1.  (One lane when they are many, up to 4 when they
// are few, by the unit: 938 and 32.7, and 48 sets of 1009 x 3 34.6, not 23.5.)
constexpr int kWideLanes = 4;

__device__ __forceinline__ int flux_bucket(int cls, float key)
{
    if (cls >= 0) return kBWhole + kBTop - std::min(cls, kBTop);
    return key < -0.99f ? kBWide : key < -0.5f ? kBHard : key < 0.0f ? kBHard + 1 : key < 0.5f ? kBHard + 2 : kBHard + 3;
}

// Issue priority of the stages that wait for memory, LDS and each other (window,
// classification, sorting, averages): the evaluation's long runs of arithmetic,
// at 0, fill what they leave.  4096 sets of 3000 x 15 sub-samples: 149 us at one
// priority for all, 147 with the classification alone ahead, 139 with them all
// (2 and 3 are the same), 155 with the evaluation ahead.
constexpr int kPrioLatency = 1;

// stages of the fused pass whose wavefront clocks a timed batch adds up
enum { C_WINDOW, C_CLASSIFY, C_TRAP, C_HARD, C_ARCS, C_DECLINED, C_AVERAGE, kClocks };

// What a fused pass runs: oblate planets, general ellipsoids, or oblate planets
// with the gated surrogate.
enum { M_OBLATE, M_ELLIPSOID, M_SURROGATE };

// The gate and the network's rows of a surrogate pass.
struct NetArgs {
    const float* table;        // calibrated scaled-error bound per bin (< 0: never accept)
    const uint8_t* zero;       // per bin: 1 = the sphere alone (no network)
    double k;                  // safety / tolerance
    const gl::SetConst* sph;   // sphere constants per set
    uint16_t* x;               // rows: BF16 features,
    int64_t* slot;             //   output (-1: none),
    double* scale;             //   residual scale over the output's sub-samples,
    float* y;                  //   and what the network makes of them
    int64_t cap;               // rows that fit
};

// The gate on one sub-sample whose planet touches the disk: false when it has
// to be exact.  `on`: the sample counts as on the disk; `net`: the residual
// (scale times the network's output on `feat`) is to be added to the sphere's.
template <class SH>
__device__ __forceinline__ bool gate(const NetArgs& N, const SH& S, double x0, double y0, bool& on, bool& net, float* feat,
                                     double& scale)
{
    int bin;
    net = false;
    on = x0 * x0 + y0 * y0 < (1.0 + S.k) * (1.0 + S.k) && gl::sur_encode(S, x0, y0, feat, scale, bin);
    if (!on) return false;
    const float tb = N.table[bin];
    if (!(tb >= 0.f && N.k * (double)tb * scale <= 1.0)) return false;
    net = N.zero[bin] == 0;
    return true;
}

// One declined sub-sample by the general path, from its centre (a locked set's:
// cosine and sine of its phase).  Out of line: it needs far more registers and
// stack than the rest, for one sample in 10^4 up to k = 0.2, and for up to a
// tenth of them above 0.5.
struct FluxU {
    double F;
    int unconv;
};
template <bool CENSUS, int MODE>
__device__ __attribute__((noinline)) FluxU flux_declined(const gl::SetConst& S, double px, double py, int* tally)
{
    gl::SetConst L;
    const bool lock = MODE == M_ELLIPSOID && S.locked;
    const double x0 = lock ? S.xb * px : px, y0 = lock ? S.d * py : py;
    if (lock) gl::lock_turned(S, py, px, L);
    const gl::SetConst& s = lock ? L : S;
    if (CENSUS) {
        gl::Census ct;
        int cls = gl::CLS_OUT;
        const double d = gl::occulted_hard<gl::Census>(s, x0, y0, &cls, ct);
        tally[cls == gl::CLS_FULL ? 1 : cls == gl::CLS_PARTIAL ? 2 : 3] += 1;
        if (cls == gl::CLS_PARTIAL) tally[9] += 1;
        tally[8] += ct.trap_nodes;
        tally[5] += ct.arcs;
        tally[6] += ct.iters;
        tally[7] += ct.limbs;
        return {1.0 - d, (int)ct.unconv};
    }
    gl::NoCensus nc;
    const double d = gl::occulted_hard<gl::NoCensus>(s, x0, y0, nullptr, nc);
    return {1.0 - d, (int)nc.unconv};
}

// The sets of CSR blocks: block blk belongs to the set s with off[s] <= blk <
// off[s + 1]; 64 probes per step, one per lane.
__device__ __forceinline__ int64_t set_of_block(const int64_t* __restrict__ off, int64_t n_sets, int64_t blk)
{
    const int lane = threadIdx.x & 63;
    int64_t lo = 0, hi = n_sets;  // off[lo] <= blk < off[hi]
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + 63) / 64;
        const int64_t at = lo + step * lane;
        const unsigned long long m = __ballot(at < hi && off[at < hi ? at : lo] <= blk);
        const int j = 63 - __builtin_clzll(m);  // lane 0 always holds
        const int64_t nlo = lo + step * j;
        hi = std::min(hi, nlo + step);
        lo = nlo;
    }
    return uniform64(lo);
}

// A value read through the constant address space: with a wavefront-uniform
// address a scalar load, whatever the kernel stores elsewhere (the sets'
// constants never change during the launch; as plain global loads they count
// as possibly overwritten by the outputs and go to vector registers, 40 of
// them per lane).
template <class T>
__device__ __forceinline__ T sload(const T* p)
{
    return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// Index i (wavefront-uniform), unknown to the optimiser: what is read at it is
// read again rather than held in registers across a loop.
__device__ __forceinline__ int fresh(int i)
{
    i = __builtin_amdgcn_readfirstlane(i);
    asm volatile("" : "+s"(i));
    return i;
}

// The same for a value that differs from lane to lane.
__device__ __forceinline__ int fresh_v(int i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// The set's shadow and its limb-darkening law.
struct SetView : gl::Shape {
    double c0, c1, c2, inv_phi;
};

__device__ __forceinline__ SetView set_view(const gl::SetConst* __restrict__ sc, int si)
{
    const gl::SetConst* s = sc + fresh(si);
    SetView v;
    v.A = sload(&s->A);
    v.B = sload(&s->B);
    v.C = sload(&s->C);
    v.AC = sload(&s->AC);
    v.M2 = sload(&s->M2);
    v.K3 = sload(&s->K3);
    v.K4 = sload(&s->K4);
    v.k = sload(&s->k);
    v.zA = sload(&s->zA);
    v.zC0 = sload(&s->zC0);
    v.c0 = sload(&s->c0);
    v.c1 = sload(&s->c1);
    v.c2 = sload(&s->c2);
    v.inv_phi = sload(&s->inv_phi);
    return v;
}

__device__ __forceinline__ gl::Orbit orbit_view(const gl::SetConst* __restrict__ sc, int si)
{
    const gl::SetConst* s = sc + fresh(si);
    return gl::Orbit{sload(&s->xb), sload(&s->d), sload(&s->w_orb), sload(&s->P), sload(&s->t0), sload(&s->inv_P)};
}

// The set's tidally locked body.
__device__ __forceinline__ gl::Lock lock_view(const gl::SetConst* __restrict__ sc, int si)
{
    const gl::SetConst* s = sc + fresh(si);
    gl::Lock v;
#pragma unroll
    for (int i = 0; i < 9; ++i) v.rot[i] = sload(&s->rot[i]);
#pragma unroll
    for (int i = 0; i < 3; ++i) v.ax2[i] = sload(&s->ax2[i]);
    v.sb = sload(&s->sb);
    v.cb = sload(&s->cb);
    return v;
}

// What the gate needs of a set.
struct GateView {
    double k, AC, sx, sy, c1, c2;
};

__device__ __forceinline__ GateView gate_view(const gl::SetConst* __restrict__ sc, int si)
{
    const gl::SetConst* s = sc + fresh(si);
    return GateView{sload(&s->k), sload(&s->AC), sload(&s->sx), sload(&s->sy), sload(&s->c1), sload(&s->c2)};
}

// Planet centre at time t as the classification takes it.
__device__ __forceinline__ bool flux_centre(const gl::SetConst* __restrict__ sc, int si, double t, double& x0, double& y0)
{
    const gl::Orbit ob = orbit_view(sc, si);
    const bool small = fma(1.5, sload(&sc[si].t_exp), sload(&sc[si].half_win)) * ob.w_orb < 0.0625;
    return small ? gl::centre_small(ob, t, x0, y0) : gl::centre_at(ob, t, x0, y0);
}

// The sphere of equal projected area.
__device__ __forceinline__ gl::Shape sphere_shape(double AC)
{
    const double r = gl::sqrt_nn(AC), r2 = r * r;
    return gl::Shape{r, 0.0, r, r2, 2.0 * r2, 0.0, 0.0, r, 0.0, r2 - 1.0};
}

struct FluxArgs {
    const double* times;
    int64_t n_sets, n_times;
    const gl::SetConst* sc;
    const int64_t* seg_begin;  // CSR
    const int64_t* seg_len;    // CSR
    const int64_t* blk_off;    // CSR: first block of each set, and the total
    Counters* ctr;
    double* out;
    int range;                 // outputs per workgroup (CSR: at most, see flux_range_of)
    int halvings;              // and how often it may be halved (flux_halved)
    unsigned int per_set;      // shared grid: workgroups per set, at most
    unsigned int row;          // workgroups per row of the launch's grid (gl::flux_row)
    NetArgs net;               // surrogate passes
};

// Where workgroup blk's outputs are: set, count (0: none), times and fluxes.
struct FluxPlace {
    int set, n;
    const double* times;
    double* out;
};

// Consecutive workgroups run on the eight XCDs in turn, and the sets' transits
// mostly lie at one place of their grids: with an even number of workgroups
// per set the heavy ones would all meet on the same XCDs, so set s starts at
// its workgroup s (512 sets of 65536 outputs: 508 us without).
__device__ __forceinline__ int64_t turned(int64_t r, int64_t set, int64_t count)
{
    if (count & 1) return r;
    const unsigned int c = (unsigned int)count, m = (unsigned int)r + (unsigned int)set % c;
    return m >= c ? m - c : m;
}

__device__ __forceinline__ FluxPlace flux_place(const FluxArgs& A, unsigned int blk)
{
    FluxPlace p{0, 0, nullptr, nullptr};
    if (A.blk_off) {
        if ((int64_t)blk >= A.blk_off[A.n_sets]) return p;
        const int64_t s = set_of_block(A.blk_off, A.n_sets, blk);
        p.set = __builtin_amdgcn_readfirstlane((int)s);
        const int range = flux_range_of(most_of(A.range, s, A.n_sets), A.sc[s].valid ? A.sc[s].n_ss : 1, A.halvings);
        const int64_t b0 = uniform64(A.blk_off[s]), count = uniform64(A.blk_off[s + 1]) - b0;
        const int64_t r0 = turned((int64_t)blk - b0, s, count) * __builtin_amdgcn_readfirstlane(range);
        const int64_t first = uniform64(A.seg_begin[s]) + r0;
        p.n = (int)std::min<int64_t>(range, uniform64(A.seg_len[s]) - r0);
        p.times = A.times + first;
        p.out = A.out + first;
    } else {
        unsigned int q = blk / A.per_set;
        if ((int64_t)q >= A.n_sets) return p;
        int range = A.range;
        int64_t r = blk - q * A.per_set;
        if (A.halvings) {
            // the sets' first workgroups first: those that their n_ss leaves
            // without outputs come last, beside the others' work (64 walkers of
            // 1009 x 3: 36.6 us set by set); turned by one set in each round, or
            // all of a heavy set's would meet on one XCD (16 sets of 3000 x 64:
            // 249 us)
            const unsigned int n = (unsigned int)A.n_sets, i = blk / n, k = blk - i * n + i % n;
            r = i;
            q = k >= n ? k - n : k;
            // (n_ss together with the constants that the window test reads next)
            const gl::SetConst* sp = A.sc + q;
            const int nss = sload(&sp->n_ss);
            const double t0 = sload(&sp->t0), win = sload(&sp->half_win);
            asm volatile("" ::"s"(nss), "s"(t0), "s"(win));
            range = flux_halved(range, std::min(std::max(nss, 1), 64), A.halvings);
        } else {
            r = turned(r, q, A.per_set);
        }
        const int64_t r0 = r * range;
        p.set = (int)q;
        p.n = (int)std::max<int64_t>(std::min<int64_t>(range, A.n_times - r0), 0);
        p.times = A.times + r0;
        p.out = A.out + ((int64_t)q * A.n_times + r0);
    }
    p.n = __builtin_amdgcn_readfirstlane(p.n);
    return p;
}

// A surrogate batch's output whose network rows found no room, exactly: by one
// wavefront, a sub-sample per lane.
__device__ __forceinline__ void exact_output(const FluxArgs& A, const FluxPlace& pl, int pos, int& unconv)
{
    const gl::SetConst& S = A.sc[pl.set];
    const int lane = threadIdx.x & 63, nss = S.n_ss;
    double F = 1.0, x, y, d;
    if (lane < nss &&
        flux_centre(A.sc, pl.set, fma(fma((double)lane + 0.5, 1.0 / (double)nss, -0.5), S.t_exp, pl.times[pos]), x, y)) {
        if (gl::occulted_direct(S, S.c0, S.c1, S.c2, S.inv_phi, x, y, d)) {
            F = 1.0 - d;
        } else {
            const FluxU r = flux_declined<false, M_OBLATE>(S, x, y, nullptr);
            F = r.F;
            unconv += r.unconv;
        }
    }
    double sum = 0.0;
    for (int j = 0; j < nss; ++j) sum += __shfl(F, j);
    if (lane == 0) pl.out[pos] = sum / (double)nss;
}

// MODE M_ELLIPSOID: a batch of general ellipsoids.  A tidally locked set's shadow turns with
// the orbit: its samples keep the sine and cosine of their phase in LDS in the
// place of the centre, and rebuild centre and shadow (lock_shape) where they
// are classified and where they are evaluated (2048 sets of 1500 outputs, half
// of them locked: 1031 us by the work lists with a 21-node rule per arc, 235
// here; three wavefronts per SIMD instead of four cost 11 %, two 38 %).
template <bool CENSUS, bool TIMED, int MODE, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, 4) k_flux(FluxArgs A)
{
    GL_AS_WRITTEN
    constexpr int kThreads = 64 * WAVES, kUnit = FluxSize<WAVES>::unit, kRange = FluxSize<WAVES>::range, kRound = FluxSize<WAVES>::round;
    __shared__ double fx[kUnit], fy[kUnit];        // ellipse centres; fx then holds the fluxes
    __shared__ unsigned short ord[kUnit + 128];    // sorted entries: index | order << 10
    // in-window outputs of the range, per 128 of them the even ones, then the odd
    __shared__ unsigned long long masks[kRange / 64];
    __shared__ unsigned short win[kRange];             // their offsets in it
    __shared__ int cnt[64];
    __shared__ unsigned short dec[kUnit];          // entries that the direct rules declined
    __shared__ int n_wide, n_hard, n_whole, next_tile, n_dec, any_nonet;
    // surrogate: outputs without room for their rows; rows per 64 entries; the unit's first row
    __shared__ unsigned int nonet[MODE == M_SURROGATE ? kRange / 32 : 1];
    __shared__ int net_n[kUnit / 64 + 1];
    __shared__ long long net_at;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    __builtin_amdgcn_s_setprio(kPrioLatency);
    const FluxPlace pl = flux_place(A, blockIdx.y * A.row + blockIdx.x);
    if (pl.n <= 0) return;
    const int si = pl.set, n_range = pl.n;
    const double* const times = pl.times;
    double* const out = pl.out;
    int tally[CENSUS ? kCensus : 1] = {};
    unsigned long long clk[TIMED ? kClocks : 1] = {}, t_last = TIMED ? __builtin_readcyclecounter() : 0ull;
    int unconv = 0;
    auto lap = [&](int stage) {
        if (TIMED) {
            const unsigned long long t = __builtin_readcyclecounter();
            clk[stage] += t - t_last;
            t_last = t;
        }
    };
    if (MODE == M_SURROGATE && tid < kRange / 32) nonet[tid] = 0u;
    unsigned int n_sub = 0u, n_on = 0u, n_acc = 0u;  // surrogate: in window, on the disk, accepted
    if (tid == 0) any_nonet = 0;
    {
        // window
        const gl::SetConst* sp = A.sc + fresh(si);
        const double t0 = sload(&sp->t0), P = sload(&sp->P), inv_P = sload(&sp->inv_P);
        const double reach = fma(0.5, sload(&sp->t_exp), sload(&sp->half_win));
        const bool valid = sload(&sp->valid) != 0, locked = MODE == M_ELLIPSOID && sload(&sp->locked) != 0;
        bool any = false;
        auto phase = [&](double v) {  // phase_time; not a number unless v is finite
            const double dt = v - t0;
            return fabs(fma(-P, rint(dt * inv_P), dt));
        };
        for (int k0 = 0; k0 < n_range; k0 += kRound) {
            constexpr int nk = kRound / 128 / WAVES;
            pair2 t[nk];
            if (valid && k0 + kRound <= n_range) {
                // a whole round out of transit, the usual one where transits
                // are rare: one test, then stores alone, streamed past the
                // caches (the 1s are never read back)
                double a[2 * nk];
                bool in = false;
                const int pos = k0 + 128 * wv + 2 * lane;
#pragma unroll
                for (int k = 0; k < nk; ++k) t[k] = *(const pair2*)(times + pos + 128 * WAVES * k);
#pragma unroll
                for (int k = 0; k < nk; ++k) {
                    a[2 * k] = phase(t[k].x);
                    a[2 * k + 1] = phase(t[k].y);
                }
#pragma unroll
                for (int k = 0; k < 2 * nk; ++k) in |= !(a[k] >= reach);
                if (!__ballot(in)) {
#pragma unroll
                    for (int k = 0; k < nk; ++k)
                        __builtin_nontemporal_store(pair2{1.0, 1.0}, (pair2*)(out + pos + 128 * WAVES * k));
                    if (lane < 2 * nk) masks[(k0 >> 6) + (lane >> 1) * (2 * WAVES) + 2 * wv + (lane & 1)] = 0ull;
                    continue;
                }
            } else {
#pragma unroll
                for (int k = 0; k < nk; ++k) {
                    const int pos = k0 + 128 * (k * WAVES + wv) + 2 * lane;
                    t[k] = pair2{pos < n_range ? times[pos] : 0.0, pos + 1 < n_range ? times[pos + 1] : 0.0};
                }
            }
            unsigned int odd = 0u;  // groups of 128 with a value that is not finite, or of an invalid set
#pragma unroll
            for (int k = 0; k < nk; ++k) {
                const int g = k0 + 128 * (k * WAVES + wv), pos = g + 2 * lane;
                unsigned long long m0 = 0ull, m1 = 0ull;
                if (g < n_range) {
                    const double a0 = phase(t[k].x), a1 = phase(t[k].y);
                    const bool on0 = pos < n_range, on1 = pos + 1 < n_range;
                    const bool w0 = on0 && a0 < reach, w1 = on1 && a1 < reach;
                    m0 = __ballot(w0);
                    m1 = __ballot(w1);
                    if (!valid || __ballot(__builtin_isunordered(a0, a1))) {
                        odd |= 1u << k;
                    } else {
                        if (on0 && !w0) __builtin_nontemporal_store(1.0, out + pos);
                        if (on1 && !w1) __builtin_nontemporal_store(1.0, out + pos + 1);
                    }
                }
                any |= (m0 | m1) != 0ull;
                if (lane == 0) {
                    masks[g >> 6] = m0;
                    masks[(g >> 6) + 1] = m1;
                }
            }
            if (odd) {
#pragma unroll 1
                for (int k = 0; k < nk; ++k) {
                    if (!((odd >> k) & 1u)) continue;
                    const int g = k0 + 128 * (k * WAVES + wv);
#pragma unroll 1
                    for (int i = 0; i < 2; ++i) {
                        const int pos = g + 2 * lane + i;
                        const double v = pos < n_range ? times[pos] : 0.0;
                        const bool ok = valid && gl::finite_d(v), w = pos < n_range && ok && phase(v) < reach;
                        if (pos < n_range && !w) out[pos] = ok ? 1.0 : __builtin_nan("");
                        if (valid && !ok) atomicOr(&A.ctr->status, 4u);
                        const unsigned long long m = __ballot(w);
                        if (lane == 0) masks[(g >> 6) + i] = m;
                    }
                }
            }
        }
        any = any && valid;
        if (!__syncthreads_or(any)) {
            lap(C_WINDOW);
            if (TIMED && lane == 0) atomicAdd(&A.ctr->clocks[C_WINDOW][blockIdx.x % kShards].v, clk[C_WINDOW]);
            return;
        }
        // positions of the in-window outputs, in order, 128 outputs per lane
        // (masks beyond the range's last round were not written)
        const bool mine = lane < (n_range + kRound - 1) / kRound * (kRound / 128);
        int incl = mine ? __popcll(masks[2 * lane]) + __popcll(masks[2 * lane + 1]) : 0;
        const bool some = incl != 0;
        for (int d = 1; d < kRange / 128; d <<= 1) {
            const int v = __shfl_up(incl, d);
            if (lane >= d) incl += v;
        }
        const int n_in = __shfl(incl, kRange / 128 - 1);
        // (those with any are few and neighbours where transits are rare)
        int turn = 0;
        for (unsigned long long nz = __ballot(some); nz; nz &= nz - 1ull)
            if ((turn++ & (WAVES - 1)) == wv) {
                const int g = __builtin_ctzll(nz);
                const unsigned long long m0 = masks[2 * g], m1 = masks[2 * g + 1];
                const int first = __builtin_amdgcn_readlane(incl, g) - __popcll(m0) - __popcll(m1);
                const int at = first + lanes_below(m0) + lanes_below(m1), w0 = (int)((m0 >> lane) & 1ull);
                if (w0) win[at] = (unsigned short)(128 * g + 2 * lane);
                if ((m1 >> lane) & 1ull) win[at + w0] = (unsigned short)(128 * g + 2 * lane + 1);
            }
        const int nss = sload(&sp->n_ss);
        const double inv_nss = 1.0 / (double)nss;
        const float inv_nss_f = 1.0f / (float)nss;
        const int n_all = __builtin_amdgcn_readfirstlane(n_in);
        // outputs per unit: as few units as hold them, of equal size
        const int n_units = (n_all + kUnit / nss - 1) / (kUnit / nss), per_unit = (n_all + n_units - 1) / n_units;
        if (CENSUS && tid == 0) tally[0] += n_all * nss;
        lap(C_WINDOW);
        for (int o0 = 0; o0 < n_all; o0 += per_unit) {
            const int no = std::min(per_unit, n_all - o0), N = no * nss;
            const int tid = fresh_v(threadIdx.x), lane = tid & 63;
            // classify
            if (tid < 64) cnt[tid] = 0;
            if (tid == 0) next_tile = n_dec = 0;
            __syncthreads();
            double ts[4];
            int jj[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = k * kThreads + tid;
                ts[k] = 0.0;
                jj[k] = 0;
                if (e < N) {
                    // e / nss for e < 1024, nss <= 64 from a float product (exact floor)
                    const int o = (int)(((float)e + 0.5f) * inv_nss_f);
                    jj[k] = e - o * nss;
                    ts[k] = times[win[o0 + o]];
                }
            }
            const SetView S = set_view(A.sc, si);
            const gl::Orbit ob = orbit_view(A.sc, si);
            const double t_exp = sload(&A.sc[si].t_exp);
            // every phase of the window within 1/16 (planets beyond ~17 stellar radii)
            const bool small = fma(1.5, t_exp, sload(&A.sc[si].half_win)) * ob.w_orb < 0.0625;
            auto centre = [&](double t, double& x, double& y) {
                if (small) return gl::centre_small(ob, t, x, y);
                asm volatile("");  // (the general path not ahead of the branch)
                return gl::centre_at(ob, t, x, y);
            };
            static_assert(kFluxBuckets <= 32, "five bits");
            int place[4];  // bucket and rank in it
            unsigned short val[4];
            bool net[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = k * kThreads + tid;
                val[k] = 0;
                net[k] = false;
                bool sphere = false;
                int b = -1;
                if (e < N) {
                    if (MODE == M_SURROGATE) n_sub += 1;
                    const double tt = fma(fma((double)jj[k] + 0.5, inv_nss, -0.5), t_exp, ts[k]);
                    double px, py;  // centre, or cosine and sine of the phase
                    float key = 0.0f;
                    int c = gl::kOffDisk;
                    if (MODE == M_ELLIPSOID && locked) {
                        gl::phase_at(ob, tt, small, py, px);
                        if (px > 0.0)
                            c = gl::direct_class(gl::lock_shape(lock_view(A.sc, si), py, px), ob.xb * px, ob.d * py, key);
                    } else if (centre(tt, px, py)) {
                        if (MODE == M_SURROGATE) {
                            float feat[gl::kSurFeat];
                            double scale;
                            bool on;
                            sphere = gate(A.net, gate_view(A.sc, si), px, py, on, net[k], feat, scale);
                            n_on += on;
                            n_acc += sphere;
                            if (sphere) {
                                c = gl::direct_class(sphere_shape(S.AC), px, py, key);
                                // (its row still needs the centre)
                                if (net[k] && c == gl::kOffDisk) c = gl::kHard;
                            } else {
                                c = gl::direct_class(S, px, py, key);
                            }
                        } else {
                            c = gl::direct_class(S, px, py, key);
                        }
                    }
                    if (c == gl::kOffDisk) {
                        fx[e] = 1.0;
                        if (CENSUS) tally[3] += 1;
                    } else {
                        fx[e] = px;
                        fy[e] = py;
                        b = flux_bucket(c, key);
                        val[k] = (unsigned short)(e | (c > 0 ? (c - 1) << 10 : 0) | (sphere ? 0x8000 : 0));
                    }
                }
                place[k] = b;
                if (MODE == M_SURROGATE) {
                    const unsigned long long mn = __ballot(net[k]);
                    if (lane == 0) net_n[k * WAVES + wv] = __popcll(mn);
                }
            }
            // ranks in the buckets: the lanes that share a lane's bucket from
            // five ballots, one atomic by the lowest of them (neighbouring
            // sub-samples are mostly alike: an atomic per entry would meet up
            // to 64 others on one address; one bucket after another is a chain
            // of as many LDS round trips)
            int at[4], peer[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int b = place[k];
                const unsigned long long on = __ballot(b >= 0);
                unsigned int lo = (unsigned int)on, hi = (unsigned int)(on >> 32);
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const unsigned long long one = __ballot((b >> q) & 1);
                    const unsigned int mine = (unsigned int)((b << (31 - q)) >> 31);  // all ones or none
                    lo &= ~((unsigned int)one ^ mine);
                    hi &= ~((unsigned int)(one >> 32) ^ mine);
                }
                const unsigned long long same = lo | ((unsigned long long)hi << 32);
                peer[k] = lanes_below(same);
                at[k] = 0;
                if (b >= 0 && peer[k] == 0) at[k] = atomicAdd(&cnt[b], __popcll(same));
                peer[k] |= __builtin_ctzll(same | (1ull << 63)) << 8;  // and the lowest of them
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int base = __shfl(at[k], peer[k] >> 8);
                if (place[k] >= 0) place[k] |= (base + (peer[k] & 255)) << 8;
            }
            __syncthreads();
            if (tid < 64) {
                // first positions: wide entries, then (from a tile's start) the
                // other crossing ones, then (from a tile's start) the whole ones
                const int c = lane < kFluxBuckets ? cnt[lane] : 0;
                int incl = c;
                for (int d = 1; d < 64; d <<= 1) {
                    const int v = __shfl_up(incl, d);
                    if (lane >= d) incl += v;
                }
                const int cw = __shfl(c, kBWide), ch = __shfl(incl, kBWhole - 1) - cw, ct = __shfl(incl, 63) - cw - ch;
                const int pw = (cw + 63) & ~63, ph = (ch + 63) & ~63;
                const int first = lane == kBWide ? 0 : lane < kBWhole ? pw + incl - c - cw : pw + ph + incl - c - cw - ch;
                cnt[lane] = first;
                if (MODE == M_SURROGATE) {
                    // rows of the network: one range per unit, in entry order
                    const int nn = lane < kUnit / 64 ? net_n[lane] : 0;
                    int inc = nn;
                    for (int d = 1; d < kUnit / 64; d <<= 1) {
                        const int v = __shfl_up(inc, d);
                        if (lane >= d) inc += v;
                    }
                    const int total = __shfl(inc, kUnit / 64 - 1);
                    if (lane < kUnit / 64) net_n[lane] = inc - nn;
                    if (lane == 0) {
                        net_n[kUnit / 64] = total;
                        net_at = total ? (long long)atomicAdd(&A.ctr->net_total, (unsigned long long)total) : 0;
                    }
                }
                if (lane == 0) {
                    n_wide = cw;
                    n_hard = ch;
                    n_whole = ct;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (place[k] >= 0) ord[cnt[place[k] & 255] + (place[k] >> 8)] = val[k];
            if (MODE == M_SURROGATE && net_n[kUnit / 64] > 0) {
                const int64_t at = (int64_t)net_at;
                const bool fits = at + net_n[kUnit / 64] <= A.net.cap;
#pragma unroll 1
                for (int k = 0; k < 4; ++k) {
                    const bool mine = k == 0 ? net[0] : k == 1 ? net[1] : k == 2 ? net[2] : net[3];
                    const unsigned long long mn = __ballot(mine);
                    if (!mine) continue;
                    const int e = k * kThreads + tid, o = win[o0 + (int)(((float)e + 0.5f) * inv_nss_f)];
                    const int64_t row = at + net_n[k * WAVES + wv] + lanes_below(mn);
                    if (!fits) {
                        // no room: the output is exact, a slot below the end is empty
                        atomicOr(&nonet[o >> 5], 1u << (o & 31));
                        any_nonet = 1;
                        if (row < A.net.cap) {
                            A.net.slot[row] = -1;
                            for (int i = 0; i < gl::kSurFeat; ++i) A.net.x[row * gl::kSurFeat + i] = 0;
                        }
                        continue;
                    }
                    // the centre is still in LDS: the features again from it
                    float feat[gl::kSurFeat];
                    double scale;
                    int bin;
                    gl::sur_encode(gate_view(A.sc, si), fx[e], fy[e], feat, scale, bin);
                    unsigned int w[gl::kSurFeat / 2];
                    for (int i = 0; i < gl::kSurFeat / 2; ++i)
                        w[i] = (unsigned)gl::f2bf_rne(feat[2 * i]) | ((unsigned)gl::f2bf_rne(feat[2 * i + 1]) << 16);
                    uint4* dst = reinterpret_cast<uint4*>(A.net.x + row * gl::kSurFeat);
                    dst[0] = uint4{w[0], w[1], w[2], w[3]};
                    dst[1] = uint4{w[4], w[5], w[6], w[7]};
                    A.net.slot[row] = (pl.out - A.out) + o;
                    A.net.scale[row] = scale * inv_nss;
                }
            }
            __syncthreads();
            lap(C_CLASSIFY);
            // evaluate
            __builtin_amdgcn_s_setprio(0);
            const int cw = __builtin_amdgcn_readfirstlane(n_wide), ch = __builtin_amdgcn_readfirstlane(n_hard),
                      ct = __builtin_amdgcn_readfirstlane(n_whole);
            const int tw = (cw + 63 / kWideLanes) / (64 / kWideLanes), pw = (cw + 63) & ~63, th = (ch + 63) >> 6, tt = (ct + 63) >> 6;
            for (;;) {
                int tile = 0;
                const int lane = fresh_v(threadIdx.x) & 63;
                if (lane == 0) tile = atomicAdd(&next_tile, 1);
                tile = __builtin_amdgcn_readfirstlane(tile);
                const SetView S = set_view(A.sc, si);
                if (tile >= tw + th + tt) break;
                // shadow and centre of an entry
                auto entry = [&](int v, double& x0, double& y0) {
                    const int e = v & 1023;
                    x0 = fx[e];
                    y0 = fy[e];
                    if (MODE == M_SURROGATE && (v & 0x8000)) return sphere_shape(S.AC);
                    if (!(MODE == M_ELLIPSOID && locked)) return (gl::Shape)S;
                    const gl::Shape sh = gl::lock_shape(lock_view(A.sc, si), y0, x0);
                    x0 *= sload(&A.sc[si].xb);
                    y0 *= sload(&A.sc[si].d);
                    return sh;
                };
                if (tile < tw + th) {
                    // crossing ellipses: G lanes per entry
                    const bool wide = tile < tw;
                    const int G = wide ? kWideLanes : 1;
                    const int g = lane & (G - 1);
                    const int i = wide ? (64 * tile + lane) / kWideLanes : 64 * (tile - tw) + lane;
                    auto reduce = [&](double v) {
                        for (int d = 1; d < G; d <<= 1) v += __shfl_xor(v, d);
                        return v;
                    };
                    if (i < (wide ? cw : ch)) {
                        const int v0 = ord[i + (wide ? 0 : pw)], e = v0 & 1023;
                        double x0, y0;
                        const gl::Shape sh = entry(v0, x0, y0);
                        gl::DirectArc T;
                        const int st = gl::direct_arc(sh, S.c0, S.c1, S.c2, S.inv_phi, x0, y0, T);
                        lap(C_HARD);
                        double F = 1.0;
                        bool ok = st == gl::DIRECT_OFF;
                        if (st == gl::DIRECT_ARC) {
                            double v;
                            int n = T.N;
                            for (int rep = 0; rep < 2 && !ok; ++rep) {
                                ok = gl::arc_rule(T, n, g, G, v, reduce);
                                if (CENSUS && g == 0) tally[5] += 1;
                                n *= 2;
                            }
                            F = fma(S.c1 * S.inv_phi * (1.0 / 3.0), v, 1.0 - T.base);
                            if (CENSUS && g == 0 && ok) {
                                tally[2] += 1;
                                tally[6] += 4;
                                tally[7] += 1;
                                tally[9] += 1;
                            }
                        } else if (st == gl::DIRECT_DECLINED) {
                            gl::DirectWhole Wh;
                            ok = gl::direct_whole(sh, x0, y0, Wh);
                            if (ok) {
                                const double sl = gl::whole_rule(Wh, g, G, reduce);
                                F = 1.0 - gl::direct_whole_delta(sh, S.c0, S.c1, S.c2, S.inv_phi, x0, y0, sl);
                                if (CENSUS && g == 0) {
                                    tally[1] += 1;
                                    tally[8] += 2 * Wh.h;
                                }
                            }
                        } else if (CENSUS && g == 0) {
                            tally[3] += 1;
                        }
                        // (a declined sample keeps its centre)
                        if (g == 0) {
                            if (ok) fx[e] = F;
                            else dec[atomicAdd(&n_dec, 1)] = (unsigned short)v0;
                        }
                    }
                    lap(C_ARCS);
                } else {
                    const int i = lane + ((tile - tw - th) << 6);
                    if (i < ct) {
                        const int v = ord[i + pw + (th << 6)], e = v & 1023, h = ((v >> 10) & 31) + 1;
                        double x0, y0;
                        const gl::Shape sh = entry(v, x0, y0);
                        fx[e] = 1.0 - gl::direct_whole_delta(sh, S.c0, S.c1, S.c2, S.inv_phi, x0, y0, gl::whole_lin(sh, x0, y0, h));
                        if (CENSUS) {
                            tally[1] += 1;
                            tally[4] += 2 * h;
                        }
                    }
                    lap(C_TRAP);
                }
            }
            __syncthreads();
            if (const int nd = __builtin_amdgcn_readfirstlane(n_dec); __builtin_expect(nd, 0)) {
                // declined
                for (int i = fresh_v(threadIdx.x); i < nd; i += kThreads) {
                    const int v = dec[i], e = v & 1023;
                    const gl::SetConst* s = (MODE == M_SURROGATE && (v & 0x8000) ? A.net.sph : A.sc) + si;
                    const FluxU r = flux_declined<CENSUS, MODE>(*s, fx[e], fy[e], tally);
                    fx[e] = r.F;
                    unconv += r.unconv;
                }
                __syncthreads();
                lap(C_DECLINED);
            }
            __builtin_amdgcn_s_setprio(kPrioLatency);
            // average
            for (int o = fresh_v(threadIdx.x); o < no; o += kThreads) {
                double sum = 0.0;
                for (int j = 0; j < nss; ++j) sum += fx[o * nss + j];
                const int w = win[o0 + o];
                if (MODE != M_SURROGATE || !((nonet[w >> 5] >> (w & 31)) & 1u)) out[w] = sum / (double)nss;
            }
            __syncthreads();
            lap(C_AVERAGE);
        }
    }
    if (MODE == M_SURROGATE && __builtin_amdgcn_readfirstlane(any_nonet)) {
        int turn = 0;
        for (int w = 0; w < kRange / 32; ++w)
            for (unsigned int bits = __builtin_amdgcn_readfirstlane(nonet[w]); bits; bits &= bits - 1u)
                if ((turn++ & (WAVES - 1)) == wv) exact_output(A, pl, 32 * w + __builtin_ctz(bits), unconv);
        lap(C_DECLINED);
    }
    if (CENSUS)
        for (int i = 0; i < kCensus; ++i) census_add(A.ctr, i, (unsigned long long)tally[i]);
    if (MODE == M_SURROGATE) {
        const unsigned int c[3] = {n_sub, n_on, n_acc};
        for (int i = 0; i < 3; ++i) {
            unsigned int v = c[i];
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
            if (lane == 0 && v) atomicAdd(&A.ctr->sur[i][blockIdx.x % kShards].v, (unsigned long long)v);
        }
    }
    if (TIMED && lane == 0)
        for (int i = 0; i < kClocks; ++i) atomicAdd(&A.ctr->clocks[i][blockIdx.x % kShards].v, clk[i]);
    if (__ballot(unconv > 0)) unconverged_add(A.ctr, unconv, CENSUS);
}

// Adds the network's residuals to the outputs: the rows of an output are
// consecutive (one unit's, in entry order), its first row's thread adds them.
// One thread tells the host how many rows the pass asked for.
// (Only a store crosses to host memory: a load from there is a bus round trip.)
__global__ void k_net_sum(Counters* __restrict__ ctr, NetArgs N, double* __restrict__ out,
                          unsigned long long* __restrict__ rows)
{
    const int64_t want = (int64_t)ctr->net_total, n = std::min(want, N.cap);
    if (blockIdx.x == 0 && threadIdx.x == 0 && ctr->net_most < (unsigned long long)want) {
        ctr->net_most = (unsigned long long)want;
        if (rows) *rows = (unsigned long long)want;
    }
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) {
        const int64_t slot = N.slot[g];
        if (slot < 0 || (g > 0 && N.slot[g - 1] == slot)) continue;
        double sum = 0.0;
        for (int64_t i = g; i < n && N.slot[i] == slot; ++i) sum = fma(N.scale[i], (double)N.y[i], sum);
        out[slot] += sum;
    }
}

}  // namespace

// ---------------------------------------------------------------- context
// Timing events of one pass: its start, the ends of set-up and of the fused
// pass, and the pass's end (surrogate batches: after the network).
enum { E_START, E_SETUP, E_FUSED, E_END, kEvPerPass };

// Passes: a batch of more outputs or workgroups than one launch should hold
// runs as up to kMaxPasses passes over equal ranges of its parameter sets.
// Results do not depend on the split (every sub-sample and output is computed
// by itself).
constexpr int kMaxPasses = 8;
constexpr int64_t kPassOut = (int64_t)1 << 26;     // outputs one pass aims at
constexpr int64_t kPassBlocks = (int64_t)1 << 23;  // and workgroups (a launch holds fewer than 2^32 threads)

struct gl_ctx {
    int device = 0;
    int n_cu = 256;
    // the launch plan's four values, kept for gl_ctx_set_plan and its kin (the
    // fused pass takes its grid from the batch)
    int waves_per_cu = 16, waves_trap = 16, waves_classify = 24, waves_gk = 20;
    bool use_graph = true;
    char err[256] = {};  // last host-side error (fixed buffer: error paths allocate nothing)
    // workspace
    gl::SetConst* sc = nullptr;
    gl::SetConst* sc_sph = nullptr;  // equal-area spheres (surrogate batches)
    NetArgs net{};                   // rows of the network (surrogate batches)
    bool net_full = false;           // no memory for more of them
    unsigned long long* rows = nullptr;      // the most rows a pass asked for (pinned host memory)
    unsigned long long* rows_dev = nullptr;
    int64_t* seg_begin = nullptr;
    int64_t* seg_len = nullptr;
    int64_t* chunk_off = nullptr;
    int64_t cap_sets = 0;
    unsigned long long* masks = nullptr;
    int* chunk_set = nullptr;
    int64_t cap_chunks = 0;
    Counters* ctr = nullptr;
    // graph cache
    hipGraphExec_t gexec = nullptr;
    hipGraph_t graph = nullptr;
    struct Key {
        const double* params;
        int64_t n_sets;
        const double* times;
        const int64_t* offsets;
        int64_t n_times;
        const int32_t* n_ss;
        const double* t_exp;
        double* out;
        void* stream;
        void* ws;
        int passes;
        int shape;
        const double* data;
        const double* sigma;
        double* chi2;
        double* loglike;
    } key{};
    bool have_graph = false;
    // the paper's integrator: cos / sin of its nodes (snap_n of them, room for snap_cap)
    float2* snap_cs = nullptr;
    int snap_cap = 0, snap_n = 0;
    int64_t mem_total = 0;
    int passes = 1;  // passes of the current batch
    // timing of the next t_left batches: launched directly (the HIP runtime
    // a torch process loads rejects event records captured into a graph),
    // one set of stage events per pass, read right after the batch
    int t_left = 0, t_pass = 0, t_batches = 0;
    hipEvent_t* ev = nullptr;  // kEvPerPass x kMaxPasses
    double t_stage[GL_NSTAGES] = {};
    double t_comp = 0.0, t_pipe = 0.0;
};

namespace {

gl_status fail(gl_ctx* ctx, gl_status st, const char* what, hipError_t e = hipSuccess)
{
    if (ctx) {
        if (e != hipSuccess) std::snprintf(ctx->err, sizeof(ctx->err), "%s: %s", what, hipGetErrorString(e));
        else std::snprintf(ctx->err, sizeof(ctx->err), "%s", what);
    }
    return st;
}

#define GL_HIP(call, what)                                                   \
    do {                                                                     \
        hipError_t e_ = (call);                                              \
        if (e_ != hipSuccess) return fail(ctx, GL_ERR_DEVICE, what, e_);     \
    } while (0)

void drop_graph(gl_ctx* ctx)
{
    if (ctx->gexec) (void)hipGraphExecDestroy(ctx->gexec);
    if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
    ctx->gexec = nullptr;
    ctx->graph = nullptr;
    ctx->have_graph = false;
}

void free_ws(gl_ctx* ctx)
{
    (void)hipFree(ctx->sc);
    (void)hipFree(ctx->sc_sph);
    (void)hipFree(ctx->seg_begin);
    (void)hipFree(ctx->seg_len);
    (void)hipFree(ctx->chunk_off);
    (void)hipFree(ctx->masks);
    (void)hipFree(ctx->chunk_set);
    ctx->sc = ctx->sc_sph = nullptr;
    ctx->seg_begin = ctx->seg_len = ctx->chunk_off = nullptr;
    ctx->masks = nullptr;
    ctx->chunk_set = nullptr;
    ctx->cap_sets = ctx->cap_chunks = 0;
}

gl_status ensure_ws(gl_ctx* ctx, int64_t n_sets, int64_t n_chunks)
{
    if (n_sets > ctx->cap_sets) {
        drop_graph(ctx);
        GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
        (void)hipFree(ctx->sc);
        (void)hipFree(ctx->sc_sph);
        (void)hipFree(ctx->seg_begin);
        (void)hipFree(ctx->seg_len);
        (void)hipFree(ctx->chunk_off);
        ctx->sc = ctx->sc_sph = nullptr;
        ctx->seg_begin = ctx->seg_len = ctx->chunk_off = nullptr;
        ctx->cap_sets = 0;
        const int64_t cap = std::max<int64_t>(n_sets, 1024);
        if (hipMalloc(&ctx->sc, sizeof(gl::SetConst) * cap) != hipSuccess ||
            hipMalloc(&ctx->sc_sph, sizeof(gl::SetConst) * cap) != hipSuccess ||
            hipMalloc(&ctx->seg_begin, sizeof(int64_t) * cap) != hipSuccess ||
            hipMalloc(&ctx->seg_len, sizeof(int64_t) * cap) != hipSuccess ||
            hipMalloc(&ctx->chunk_off, sizeof(int64_t) * (cap + 1)) != hipSuccess) {
            free_ws(ctx);
            return fail(ctx, GL_ERR_NOMEM, "workspace allocation (sets)");
        }
        ctx->cap_sets = cap;
    }
    if (n_chunks > ctx->cap_chunks) {
        drop_graph(ctx);
        GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
        (void)hipFree(ctx->masks);
        (void)hipFree(ctx->chunk_set);
        ctx->masks = nullptr;
        ctx->chunk_set = nullptr;
        ctx->cap_chunks = 0;
        const int64_t cap = std::max<int64_t>(n_chunks, 4096);
        if (hipMalloc(&ctx->masks, sizeof(unsigned long long) * cap) != hipSuccess ||
            hipMalloc(&ctx->chunk_set, sizeof(int) * cap) != hipSuccess) {
            free_ws(ctx);
            return fail(ctx, GL_ERR_NOMEM, "workspace allocation (chunks)");
        }
        ctx->cap_chunks = cap;
    }
    return GL_OK;
}

struct Batch {
    const double* params;
    int64_t n_sets;
    const double* times;
    const int64_t* offsets;
    int64_t n_times;
    const int32_t* n_ss;
    const double* t_exp;
    double* out;
    hipStream_t stream;
    int64_t max_chunks;
    int64_t ld = 0;          // row stride of params (the whole batch's n_sets)
    int first = 1, last = 1;  // first / last pass of the batch
    int range = 128;         // outputs per workgroup of the fused pass
    int halvings = 0;        // how often they may be halved
    int waves = kFluxWaves;  // its wavefronts
    // surrogate batches (net != NULL): the gate and the network
    gl_mlp* net = nullptr;
    const float* gate_table = nullptr;
    const uint8_t* gate_zero = nullptr;
    double gate_k = 0.0;
    int shape = 0;  // 0: oblate parameter block, 1: general ellipsoids, 2: MCMC walkers
    // MCMC glue (gl_loglike_batch): the per-walker likelihood of out against
    // data / sigma after the light curves
    const double* data = nullptr;
    const double* sigma = nullptr;
    double* chi2 = nullptr;
    double* loglike = nullptr;
};

// ctx may be NULL (no message is kept)
gl_status check_batch(gl_ctx* ctx, Batch& b)
{
    if (ctx) ctx->err[0] = 0;
    if (!b.params || !b.times || !b.out) return fail(ctx, GL_ERR_NULL, "params, times and out are required");
    if (b.n_sets < 1) return fail(ctx, GL_ERR_SIZE, "n_sets must be >= 1");
    if (b.n_sets > (int64_t)INT32_MAX) return fail(ctx, GL_ERR_SIZE, "n_sets too large");
    if (b.offsets) {
        if (b.n_times < 0) return fail(ctx, GL_ERR_SIZE, "CSR n_times must be >= 0");
        b.max_chunks = b.n_times / kChunk + b.n_sets;
    } else {
        if (b.n_times < 1) return fail(ctx, GL_ERR_SIZE, "n_times must be >= 1");
        const int64_t cps = (b.n_times + kChunk - 1) / kChunk;
        if (b.n_sets > ((int64_t)1 << 62) / std::max<int64_t>(b.n_times, 1))
            return fail(ctx, GL_ERR_SIZE, "n_sets * n_times overflows");
        b.max_chunks = cps * b.n_sets;
        if ((cps + kWinGrid - 1) / kWinGrid * b.n_sets > (int64_t)INT32_MAX)
            return fail(ctx, GL_ERR_SIZE, "batch too large for one window launch");
    }
    if (b.max_chunks > ((int64_t)1 << 40)) return fail(ctx, GL_ERR_SIZE, "batch too large");
    b.ld = b.n_sets;
    return GL_OK;
}

gl_status check_args(gl_ctx* ctx, Batch& b)
{
    if (!ctx) return GL_ERR_NULL;
    return check_batch(ctx, b);
}

// Window test over all chunks (fills the out-of-window outputs, chunk masks).
void launch_window(gl_ctx* ctx, const Batch& b, hipStream_t st)
{
    if (!b.offsets) {
        const int64_t cps = (b.n_times + kChunk - 1) / kChunk;
        const int64_t bx = (cps + kWinGrid - 1) / kWinGrid;
        hipLaunchKernelGGL(k_window_grid, dim3((unsigned)(bx * b.n_sets)), dim3(64), 0, st, b.times,
                           b.n_times, cps, ctx->sc, ctx->ctr, ctx->masks, ctx->chunk_set, b.out);
    } else {
        const int64_t groups = (b.max_chunks + kWinChunks - 1) / kWinChunks;
        hipLaunchKernelGGL(k_window, dim3((unsigned)((groups + 3) / 4)), dim3(256), 0, st, b.times,
                           b.n_sets, ctx->sc, ctx->seg_begin, ctx->seg_len, ctx->chunk_off,
                           ctx->ctr, ctx->masks, ctx->chunk_set, b.out);
    }
}

// A timing event (timed batches are launched directly, never captured); on
// failure the context's error names the pass and the event.
gl_status record_event(gl_ctx* ctx, hipEvent_t ev, hipStream_t s, int e)
{
    const hipError_t r = hipEventRecord(ev, s);
    if (r == hipSuccess) return GL_OK;
    char what[64];
    std::snprintf(what, sizeof(what), "timing event %d of pass %d", e, ctx->t_pass - 1);
    return fail(ctx, GL_ERR_DEVICE, what, r);
}

// Wavefronts per workgroup of the fused pass.  A workgroup's outputs are one set's,
// so many sets of a few outputs leave four wavefronts mostly idle: with one,
// four times as many sets are on the chip at once.  Its chain is longer, so the
// sub-samples of a set must be few or the sets several times what the chip holds
// (4096); without n_ss the outputs are the sub-samples, with it (its values are
// on the device) fewer outputs qualify.  One wavefront against four, us:
//   65536 sets of 1 output: 138, 454; of 10: 245, 593 (x 64: 1061, 1140); of 32:
//   295, 629 (x 15: 1060, 1023); of 64 x 5: 874, 876; of 128: 413, 714; 16384 of 10: 83, 162 (x 64:
//   339, 309); of 32 x 15: 326, 278; 4096 of 1: 25, 43 (x 64: 53, 56); of 10 x 64:
//   155, 118; of 128: 58, 63; 1024 of 10: 29, 26.
int flux_waves(const Batch& b)
{
    const int64_t n = b.offsets ? b.n_times : b.n_sets * b.n_times;
    const int64_t most = b.n_ss ? std::min<int64_t>(FluxSize<1>::range, b.n_sets / 1024) : FluxSize<1>::range;
    return b.n_sets >= 4096 && n <= most * b.n_sets ? 1 : kFluxWaves;
}

// Outputs per workgroup of the fused pass (CSR: at most): enough workgroups to
// fill the chip (1024 are resident) four times over, at most 4096 outputs each
// (512 sets of 65536: 91 us at 2048, 89 at 4096; 2048 own grids: 971 and 947;
// want 8192 workgroups and 4096 sets of 1009 x 3 leave half a tile of 64 in
// each: 460 us, not 260; as few as 64 outputs each and 64 walkers of 1009 x 3
// take 38 us, not 33).
// An own grid's workgroups shrink with its supersampling (flux_range_of), so
// half as many outputs' worth of them are asked for (3 M outputs: 351 us at
// 4096, 315 at 2048; 333 sets of 1777 shared times: 62 us at 4096, 74 at 2048).
constexpr int kFluxTop = FluxSize<kFluxWaves>::range, kFluxWant = 4096, kFluxWantOwn = 2048;
int flux_range(const Batch& b)
{
    if (b.waves == 1) return b.offsets ? FluxSize<1>::range : (int)((b.n_times + 63) / 64 * 64);
    const int64_t n = b.offsets ? b.n_times / kFluxWantOwn : b.n_sets * b.n_times / kFluxWant;
    int r = kFluxMinRange;
    while (2 * r <= n && r < kFluxTop) r *= 2;
    if (b.offsets) return r;
    // a set's workgroups of equal length, and none for a short remainder
    const int64_t per_set = std::max<int64_t>((b.n_times + kFluxTop - 1) / kFluxTop, (b.n_times + r / 4) / r);
    return (int)(((b.n_times + per_set - 1) / per_set + 63) / 64 * 64);
}

// Workgroups of one pass (CSR: an upper bound, the sets' ranges are known on
// the device only).
int64_t flux_blocks(const Batch& b)
{
    const int least = flux_halved(b.offsets ? kFluxMinRange : b.range, 64, b.halvings);
    return b.offsets ? b.n_times / least + b.n_sets : (b.n_times + least - 1) / least * b.n_sets;
}

// How often the workgroups' ranges may be halved (the device knows n_ss, and how
// often it pays; the workgroups left over end at once): to at most 4096 workgroups,
// four times what the chip holds.  A workgroup's units follow one another, so
// few sets of many sub-samples were a long chain on a part of the chip: 16 sets of
// 1000 x 15 100 us without, 58 with, of 1000 x 64 292 and 94, one of 3000 x 64 144
// and 25; to at most 2048, 64 sets of 3000 x 15 133, not 108.
constexpr int64_t kFluxFill = 4096;
int flux_halvings(Batch b)
{
    if (!b.n_ss || b.waves == 1) return 0;
    b.halvings = 0;
    int h = 0;
    for (int64_t n = 2 * flux_blocks(b); n <= kFluxFill && h < 4; n *= 2) ++h;
    return h;
}

template <bool CENSUS, int WAVES>
auto flux_kernel(const Batch& b, bool timed)
{
    return b.net          ? (timed ? k_flux<false, true, M_SURROGATE, WAVES> : k_flux<false, false, M_SURROGATE, WAVES>)
           : b.shape == 1 ? (timed ? k_flux<false, true, M_ELLIPSOID, WAVES> : k_flux<CENSUS, false, M_ELLIPSOID, WAVES>)
                          : (timed ? k_flux<false, true, M_OBLATE, WAVES> : k_flux<CENSUS, false, M_OBLATE, WAVES>);
}

// One pass of the exact path: set-up, then the fused pass.
template <bool CENSUS>
gl_status enqueue_flux(gl_ctx* ctx, const Batch& b)
{
    hipStream_t st = b.stream;
    hipEvent_t* ev = nullptr;
    if (!CENSUS && ctx->t_left > 0 && ctx->ev && ctx->t_pass < kMaxPasses) {
        ev = ctx->ev + kEvPerPass * ctx->t_pass;
        ctx->t_pass++;
    }
    if (ev && record_event(ctx, ev[E_START], st, E_START) != GL_OK) return GL_ERR_DEVICE;
    const bool shared = b.offsets == nullptr;
    // with a likelihood on a shared grid, an extra workgroup of the first
    // pass forms its normalisation
    const bool norm = b.data && shared && b.first;
    const bool scan_here = !shared && b.n_sets <= 256;
    // single wavefronts where no workgroup has to work together: more compute
    // units share the sets' scattered stores (4096 sets: 6.4 -> 5.8 us, with the
    // surrogate's spheres 10.3 -> 6.2)
    const unsigned prep_threads = norm || scan_here ? 256u : 64u;
    const unsigned prep_blocks = (unsigned)((b.n_sets + prep_threads - 1) / prep_threads) + (norm ? 1u : 0u);
    auto prep = b.shape == 1 ? k_prep<1> : b.shape == 2 ? k_prep<2> : k_prep<0>;
    FluxArgs A{};
    A.times = b.times;
    A.n_sets = b.n_sets;
    A.n_times = b.n_times;
    A.sc = ctx->sc;
    A.ctr = ctx->ctr;
    A.out = b.out;
    A.range = b.range;
    A.halvings = b.halvings;
    const int64_t grid = flux_blocks(b);
    A.per_set = (unsigned int)(shared ? grid / b.n_sets : 0);
    A.row = gl::flux_row(grid);
    hipLaunchKernelGGL(prep, dim3(prep_blocks), dim3(prep_threads), 0, st, b.params, b.ld, b.n_sets, b.offsets, b.n_times,
                       b.n_ss, b.t_exp, ctx->sc, ctx->seg_begin, ctx->seg_len, ctx->chunk_off, ctx->ctr,
                       (int64_t)0, b.first, b.last, b.net ? ctx->sc_sph : nullptr, b.sigma, b.n_times,
                       norm ? &ctx->ctr->ll_norm : nullptr, (int)b.range, b.halvings, scan_here ? grid : (int64_t)0,
                       b.first && (CENSUS || ev || b.net));
    if (!shared) {
        if (!scan_here) hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, st, ctx->chunk_off, b.n_sets, grid, ctx->ctr);
        A.seg_begin = ctx->seg_begin;
        A.seg_len = ctx->seg_len;
        A.blk_off = ctx->chunk_off;
    }
    if (ev && record_event(ctx, ev[E_SETUP], st, E_SETUP) != GL_OK) return GL_ERR_DEVICE;
    if (b.net) {
        A.net = ctx->net;
        A.net.table = b.gate_table;
        A.net.zero = b.gate_zero;
        A.net.k = b.gate_k;
        A.net.sph = ctx->sc_sph;
    }
    const bool timed = ev != nullptr;
    auto flux = b.waves == 1 ? flux_kernel<CENSUS, 1>(b, timed) : flux_kernel<CENSUS, kFluxWaves>(b, timed);
    hipLaunchKernelGGL(flux, dim3(A.row, (unsigned)((grid + A.row - 1) / A.row)), dim3(64 * b.waves), 0, st, A);
    if (ev && record_event(ctx, ev[E_FUSED], st, E_FUSED) != GL_OK) return GL_ERR_DEVICE;
    if (b.net) {
        gl_net::infer(b.net, A.net.x, A.net.cap, &ctx->ctr->net_total, A.net.y, st);
        hipLaunchKernelGGL(k_net_sum, dim3((unsigned)(ctx->n_cu * 8)), dim3(256), 0, st, ctx->ctr, A.net, b.out, ctx->rows_dev);
    }
    if (ev && record_event(ctx, ev[E_END], st, E_END) != GL_OK) return GL_ERR_DEVICE;
    GL_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

void free_net(gl_ctx* ctx)
{
    NetArgs& N = ctx->net;
    (void)hipFree(N.x);  // (with what follows it, see ensure_net)
    N = NetArgs{};
}

// Room for the network's rows (gl::net_rows).  Units that find none are
// evaluated exactly; so a context that has some goes on with it where no more
// can be had, and does not ask again.
gl_status ensure_net(gl_ctx* ctx, int64_t n_out)
{
    static_assert(gl::kNetRowBytes == sizeof(uint16_t) * gl::kSurFeat + sizeof(int64_t) + sizeof(double) + sizeof(float), "a row");
    NetArgs& N = ctx->net;
    const int64_t want = gl::net_rows(n_out, (int64_t) * (const volatile unsigned long long*)ctx->rows, N.cap, ctx->mem_total);
    if (want <= N.cap || (ctx->net_full && N.cap > 0)) return GL_OK;
    drop_graph(ctx);
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    // one allocation: a first batch waits for each (4096 sets of 3000 x 15, first
    // pass on a new context: 362 us, 437 with four)
    void* rows = N.x;
    void** const slots[] = {&rows};
    const int64_t bytes[] = {gl::kNetRowBytes * want};
    const bool ok = gl::replace_all(
        slots, bytes,
        [](int64_t n) {
            void* p = nullptr;
            return hipMalloc(&p, (size_t)n) == hipSuccess ? p : nullptr;
        },
        [](void* p) { (void)hipFree(p); });
    if (!ok) {
        (void)hipGetLastError();
        if (N.cap == 0) return fail(ctx, GL_ERR_NOMEM, "network rows");
        ctx->net_full = true;
        return GL_OK;
    }
    N.x = (uint16_t*)rows;
    N.slot = (int64_t*)(N.x + gl::kSurFeat * want);
    N.scale = (double*)(N.slot + want);
    N.y = (float*)(N.scale + want);
    N.cap = want;
    return GL_OK;
}

// Plans a batch's passes and sizes the workspace for them (may wait for the
// device and reallocate; never called inside a stream capture).
gl_status prepare_batch(gl_ctx* ctx, Batch& b)
{
    // passes over equal ranges of sets, so that no launch covers more than
    // about kPassOut outputs or kPassBlocks workgroups
    b.waves = flux_waves(b);
    b.range = flux_range(b);
    b.halvings = flux_halvings(b);
    const int64_t n = b.offsets ? b.n_times : b.n_sets * b.n_times;
    const int64_t blocks = flux_blocks(b);
    const int64_t want = std::max((n + kPassOut - 1) / kPassOut, (blocks + kPassBlocks - 1) / kPassBlocks);
    // (every pass over own grids launches the whole batch's bound on workgroups:
    // two are enough without a network, whose rows a pass bounds)
    const int64_t most = b.offsets && !b.net ? 2 : kMaxPasses;
    ctx->passes = (int)std::max<int64_t>(1, std::min<int64_t>({most, b.n_sets, want}));
    const gl_status st = ensure_ws(ctx, b.n_sets, 1);
    return st == GL_OK && b.net ? ensure_net(ctx, n) : st;
}

// Enqueues every pass of a prepared batch (inside a stream capture when
// called from one).
gl_status run_batch(gl_ctx* ctx, const Batch& b, bool census)
{
    gl_status st = GL_OK;
    const int T = ctx->passes;
    ctx->t_pass = 0;
    for (int p = 0; p < T; ++p) {
        const int64_t a = b.n_sets * p / T, e = b.n_sets * (p + 1) / T;
        Batch q = b;
        q.params = b.params + a;
        q.n_sets = e - a;
        q.n_ss = b.n_ss ? b.n_ss + a : nullptr;
        q.t_exp = b.t_exp ? b.t_exp + a : nullptr;
        if (b.offsets) {
            q.offsets = b.offsets + a;
        } else {
            q.out = b.out + a * b.n_times;
        }
        q.first = p == 0;
        q.last = p == T - 1;
        st = census ? enqueue_flux<true>(ctx, q) : enqueue_flux<false>(ctx, q);
        if (st != GL_OK) return st;
    }
    return GL_OK;
}

gl_status enqueue(gl_ctx* ctx, const Batch& b, bool census = false)
{
    gl_status st = run_batch(ctx, b, census);
    if (st != GL_OK) return st;
    if (b.data) {
        // a shared grid's normalisation came from the first pass's k_prep
        const double* norm = b.offsets ? nullptr : &ctx->ctr->ll_norm;
        gl_mcmc::launch_loglike(b.out, b.n_sets, b.offsets, b.n_times, b.data, b.sigma, norm, b.chi2, b.loglike,
                                b.stream);
    }
    GL_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

// After a timed batch (t_pass passes recorded): waits for its stream and adds
// its stage times, the compute time (end of set-up to the end) and the pipeline
// time (start to end).
gl_status finish_timed(gl_ctx* ctx, hipStream_t s)
{
    if (ctx->t_left <= 0 || ctx->t_pass <= 0) return GL_OK;
    GL_HIP(hipStreamSynchronize(s), "hipStreamSynchronize");
    // the fused pass is one launch: its time is shared out by the clocks
    // its wavefronts spent in each stage
    LineCount c[kClocks * kShards];
    GL_HIP(hipMemcpy(c, ctx->ctr->clocks, sizeof(c), hipMemcpyDeviceToHost), "hipMemcpy");
    double part[kClocks] = {}, total = 0.0;
    for (int i = 0; i < kClocks; ++i)
        for (int j = 0; j < kShards; ++j) part[i] += (double)c[i * kShards + j].v;
    for (int i = 0; i < kClocks; ++i) total += part[i];
    for (int p = 0; p < ctx->t_pass; ++p) {
        hipEvent_t* ev = ctx->ev + kEvPerPass * p;
        float prep = 0.0f, flux = 0.0f, net = 0.0f;
        GL_HIP(hipEventElapsedTime(&prep, ev[E_START], ev[E_SETUP]), "hipEventElapsedTime");
        GL_HIP(hipEventElapsedTime(&flux, ev[E_SETUP], ev[E_FUSED]), "hipEventElapsedTime");
        GL_HIP(hipEventElapsedTime(&net, ev[E_FUSED], ev[E_END]), "hipEventElapsedTime");
        ctx->t_stage[0] += prep;
        for (int i = 0; i < kClocks; ++i) ctx->t_stage[1 + i] += total > 0.0 ? flux * part[i] / total : 0.0;
        ctx->t_stage[8] += net;
        ctx->t_comp += flux + net;
        ctx->t_pipe += prep + flux + net;
    }
    ctx->t_batches++;
    ctx->t_left--;
    ctx->t_pass = 0;
    return GL_OK;
}

bool same_key(const gl_ctx::Key& a, const gl_ctx::Key& b)
{
    return std::memcmp(&a, &b, sizeof(a)) == 0;
}

}  // namespace

extern "C" {

gl_status gl_ctx_create(gl_ctx** out, int device)
{
    if (!out) return GL_ERR_NULL;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return GL_ERR_DEVICE;
    if (hipSetDevice(device) != hipSuccess) return GL_ERR_DEVICE;
    gl_ctx* ctx = new (std::nothrow) gl_ctx();
    if (!ctx) return GL_ERR_NOMEM;
    ctx->device = device;
    hipDeviceProp_t prop{};
    if (hipGetDeviceProperties(&prop, device) == hipSuccess) {
        if (prop.multiProcessorCount > 0) ctx->n_cu = prop.multiProcessorCount;
        ctx->mem_total = (int64_t)prop.totalGlobalMem;
    }
    if (ctx->mem_total <= 0) ctx->mem_total = (int64_t)1 << 34;
    if (hipMalloc(&ctx->ctr, sizeof(Counters)) != hipSuccess) {
        delete ctx;
        return GL_ERR_NOMEM;
    }
    if (hipHostMalloc((void**)&ctx->rows, sizeof(*ctx->rows), hipHostMallocMapped) != hipSuccess ||
        hipHostGetDevicePointer((void**)&ctx->rows_dev, ctx->rows, 0) != hipSuccess) {
        if (ctx->rows) (void)hipHostFree(ctx->rows);
        (void)hipFree(ctx->ctr);
        delete ctx;
        return GL_ERR_NOMEM;
    }
    *ctx->rows = 0ull;
    if (hipMemset(ctx->ctr, 0, sizeof(Counters)) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {
        (void)hipHostFree(ctx->rows);
        (void)hipFree(ctx->ctr);
        delete ctx;
        return GL_ERR_DEVICE;
    }
    *out = ctx;
    return GL_OK;
}

void free_timing(gl_ctx* ctx)
{
    if (ctx->ev)
        for (int i = 0; i < kEvPerPass * kMaxPasses; ++i) (void)hipEventDestroy(ctx->ev[i]);
    delete[] ctx->ev;
    ctx->ev = nullptr;
    ctx->t_left = ctx->t_pass = ctx->t_batches = 0;
    for (int k = 0; k < GL_NSTAGES; ++k) ctx->t_stage[k] = 0.0;
    ctx->t_comp = ctx->t_pipe = 0.0;
}

void gl_ctx_destroy(gl_ctx* ctx)
{
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    free_timing(ctx);
    drop_graph(ctx);
    free_ws(ctx);
    (void)hipFree(ctx->ctr);
    (void)hipFree(ctx->snap_cs);
    if (ctx->rows) (void)hipHostFree(ctx->rows);
    free_net(ctx);
    delete ctx;
}

}  // extern "C"

namespace {

// The exact path for either parameter block: plans and sizes the batch, then
// replays the captured pipeline (captured again when the arguments change).
gl_status lightcurve(gl_ctx* ctx, Batch& b)
{
    const double* params = b.params;
    const int64_t n_sets = b.n_sets;
    const double* times = b.times;
    const int64_t* offsets = b.offsets;
    const int64_t n_times = b.n_times;
    const int32_t* n_ss = b.n_ss;
    const double* t_exp = b.t_exp;
    double* out = b.out;
    void* stream = (void*)b.stream;
    gl_status st = check_args(ctx, b);
    if (st != GL_OK) return st;
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    st = prepare_batch(ctx, b);
    if (st != GL_OK) return st;
    // the legacy default stream cannot be captured: launch directly there,
    // as timed batches are (their events stay out of graphs)
    const bool timed = ctx->t_left > 0;
    if (!ctx->use_graph || stream == nullptr || timed) {
        st = enqueue(ctx, b);
        if (st != GL_OK) return st;
        return timed ? finish_timed(ctx, b.stream) : GL_OK;
    }
    gl_ctx::Key k{};
    k.params = params;
    k.n_sets = n_sets;
    k.times = times;
    k.offsets = offsets;
    k.n_times = n_times;
    k.n_ss = n_ss;
    k.t_exp = t_exp;
    k.out = out;
    k.stream = stream;
    k.ws = ctx->sc;
    k.passes = ctx->passes;
    k.shape = b.shape;
    k.data = b.data;
    k.sigma = b.sigma;
    k.chi2 = b.chi2;
    k.loglike = b.loglike;
    if (!ctx->have_graph || !same_key(k, ctx->key)) {
        drop_graph(ctx);
        GL_HIP(hipStreamBeginCapture(b.stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
        gl_status est = enqueue(ctx, b);
        hipGraph_t g = nullptr;
        hipError_t ee = hipStreamEndCapture(b.stream, &g);
        if (est != GL_OK) {
            if (g) (void)hipGraphDestroy(g);
            return est;
        }
        if (ee != hipSuccess) return fail(ctx, GL_ERR_DEVICE, "hipStreamEndCapture", ee);
        hipGraphExec_t ex = nullptr;
        hipError_t ie = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        if (ie != hipSuccess) {
            (void)hipGraphDestroy(g);
            return fail(ctx, GL_ERR_DEVICE, "hipGraphInstantiate", ie);
        }
        ctx->graph = g;
        ctx->gexec = ex;
        ctx->key = k;
        ctx->have_graph = true;
    }
    GL_HIP(hipGraphLaunch(ctx->gexec, b.stream), "hipGraphLaunch");
    return GL_OK;
}

}  // namespace

extern "C" {

gl_status gl_lightcurve_batch(gl_ctx* ctx, const double* params, int64_t n_sets,
                              const double* times, const int64_t* offsets, int64_t n_times,
                              const int32_t* n_ss, const double* t_exp, double* out,
                              void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    return lightcurve(ctx, b);
}

gl_status gl_lightcurve_batch_ellipsoid(gl_ctx* ctx, const double* params, int64_t n_sets,
                                        const double* times, const int64_t* offsets, int64_t n_times,
                                        const int32_t* n_ss, const double* t_exp, double* out,
                                        void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    b.shape = 1;
    return lightcurve(ctx, b);
}

gl_status gl_loglike_batch(gl_ctx* ctx, const double* walkers, int64_t n_walkers, const double* times,
                           const int64_t* offsets, int64_t n_times, const int32_t* n_ss, const double* t_exp,
                           const double* data, const double* sigma, double* model, double* chi2, double* loglike,
                           void* stream)
{
    if (!ctx) return GL_ERR_NULL;
    ctx->err[0] = 0;
    if (!walkers || !data || !sigma || !model || (!chi2 && !loglike))
        return fail(ctx, GL_ERR_NULL, "walkers, data, sigma, model and chi2 or loglike are required");
    Batch b{walkers, n_walkers, times, offsets, n_times, n_ss, t_exp, model, (hipStream_t)stream, 0};
    b.shape = 2;  // k_prep converts the walker block
    b.data = data;
    b.sigma = sigma;
    b.chi2 = chi2;
    b.loglike = loglike;
    return lightcurve(ctx, b);
}

gl_status gl_ctx_sync_status(gl_ctx* ctx)
{
    if (!ctx) return GL_ERR_NULL;
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    unsigned int status = 0;
    GL_HIP(hipMemcpy(&status, &ctx->ctr->status, sizeof(status), hipMemcpyDeviceToHost), "hipMemcpy");
    if (status) {
        GL_HIP(hipMemset(&ctx->ctr->status, 0, sizeof(status)), "hipMemset");
        GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
        std::snprintf(ctx->err, sizeof(ctx->err), "%s%s%s", (status & 1u) ? "invalid parameter set; " : "",
                      (status & 2u) ? "invalid CSR segment; " : "", (status & 4u) ? "non-finite time; " : "");
        return GL_ERR_DOMAIN;
    }
    return GL_OK;
}

const char* gl_ctx_last_error(const gl_ctx* ctx)
{
    return ctx ? ctx->err : "null context";
}

gl_status gl_ctx_get_plan(const gl_ctx* ctx, int* waves_per_cu)
{
    if (!ctx) return GL_ERR_NULL;
    if (waves_per_cu) *waves_per_cu = ctx->waves_per_cu;
    return GL_OK;
}

gl_status gl_ctx_get_stage_plan(const gl_ctx* ctx, int* classify, int* hard, int* trap, int* gk)
{
    if (!ctx) return GL_ERR_NULL;
    if (classify) *classify = ctx->waves_classify;
    if (hard) *hard = ctx->waves_per_cu;
    if (trap) *trap = ctx->waves_trap;
    if (gk) *gk = ctx->waves_gk;
    return GL_OK;
}

gl_status gl_ctx_set_stage_plan(gl_ctx* ctx, int classify, int hard, int trap, int gk)
{
    if (!ctx) return GL_ERR_NULL;
    if (classify < 1 || classify > 64 || hard < 1 || hard > 64 || trap < 1 || trap > 64 || gk < 1 || gk > 64)
        return fail(ctx, GL_ERR_SIZE, "waves per CU in [1, 64]");
    ctx->waves_classify = classify;
    ctx->waves_per_cu = hard;
    ctx->waves_trap = trap;
    ctx->waves_gk = gk;
    drop_graph(ctx);
    return GL_OK;
}

gl_status gl_ctx_set_plan(gl_ctx* ctx, int waves_per_cu)
{
    if (!ctx) return GL_ERR_NULL;
    if (waves_per_cu < 1 || waves_per_cu > 64) return fail(ctx, GL_ERR_SIZE, "waves_per_cu in [1, 64]");
    ctx->waves_per_cu = waves_per_cu;
    return GL_OK;
}

gl_status gl_ctx_set_graph(gl_ctx* ctx, int on)
{
    if (!ctx) return GL_ERR_NULL;
    if (!on) drop_graph(ctx);
    ctx->use_graph = on != 0;
    return GL_OK;
}

}  // extern "C"

namespace {

// The fused pass takes its grid from the batch, so there is nothing to search:
// the batch runs once (the workspace is sized and the outputs are written) and
// the plan stays.
gl_status autotune(gl_ctx* ctx, Batch b)
{
    const gl_status st = lightcurve(ctx, b);
    if (st != GL_OK) return st;
    GL_HIP(hipStreamSynchronize(b.stream), "hipStreamSynchronize");
    return GL_OK;
}

}  // namespace

extern "C" {

gl_status gl_autotune(gl_ctx* ctx, const double* params, int64_t n_sets, const double* times,
                      const int64_t* offsets, int64_t n_times, const int32_t* n_ss,
                      const double* t_exp, double* out, void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    return autotune(ctx, b);
}

gl_status gl_autotune_ellipsoid(gl_ctx* ctx, const double* params, int64_t n_sets, const double* times,
                                const int64_t* offsets, int64_t n_times, const int32_t* n_ss,
                                const double* t_exp, double* out, void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    b.shape = 1;
    return autotune(ctx, b);
}

gl_status gl_ctx_set_timing(gl_ctx* ctx, int n_slots)
{
    if (!ctx) return GL_ERR_NULL;
    if (n_slots < 0 || n_slots > 10000) return fail(ctx, GL_ERR_SIZE, "n_slots in [0, 10000]");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    free_timing(ctx);
    drop_graph(ctx);  // the next batch is captured with (or without) its timing events
    if (n_slots == 0) return GL_OK;
    // one event set per pass (a timed batch is read before the next one)
    ctx->ev = new (std::nothrow) hipEvent_t[kEvPerPass * kMaxPasses];
    if (!ctx->ev) return fail(ctx, GL_ERR_NOMEM, "timing events");
    for (int i = 0; i < kEvPerPass * kMaxPasses; ++i) {
        if (hipEventCreate(&ctx->ev[i]) != hipSuccess) {
            for (int j = 0; j < i; ++j) (void)hipEventDestroy(ctx->ev[j]);
            delete[] ctx->ev;
            ctx->ev = nullptr;
            return fail(ctx, GL_ERR_DEVICE, "hipEventCreate");
        }
    }
    ctx->t_left = n_slots;
    return GL_OK;
}

gl_status gl_ctx_get_stage_timing(gl_ctx* ctx, double* stage_ms, int* n)
{
    if (!ctx) return GL_ERR_NULL;
    if (stage_ms)
        for (int k = 0; k < GL_NSTAGES; ++k) stage_ms[k] = ctx->t_stage[k];
    if (n) *n = ctx->t_batches;
    for (int k = 0; k < GL_NSTAGES; ++k) ctx->t_stage[k] = 0.0;
    ctx->t_comp = ctx->t_pipe = 0.0;
    ctx->t_batches = 0;
    return GL_OK;
}

gl_status gl_ctx_get_timing(gl_ctx* ctx, double* compute_ms, double* pipeline_ms, int* n)
{
    if (!ctx) return GL_ERR_NULL;
    if (compute_ms) *compute_ms = ctx->t_comp;
    if (pipeline_ms) *pipeline_ms = ctx->t_pipe;
    if (n) *n = ctx->t_batches;
    for (int k = 0; k < GL_NSTAGES; ++k) ctx->t_stage[k] = 0.0;
    ctx->t_comp = ctx->t_pipe = 0.0;
    ctx->t_batches = 0;
    return GL_OK;
}

gl_status gl_ctx_set_capacity(gl_ctx* ctx, int64_t sub_samples, int64_t hard_samples, int64_t arcs)
{
    if (!ctx) return GL_ERR_NULL;
    if (sub_samples < 0 || hard_samples < 0 || arcs < 0 || sub_samples > (1 << 27) - 1 ||
        hard_samples > INT32_MAX / 2 || arcs > INT32_MAX / 2)
        return fail(ctx, GL_ERR_SIZE, "capacities: 0 (default) or sub <= 2^27 - 1, hard and arcs <= 2^30 - 1");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    drop_graph(ctx);
    return GL_OK;
}

gl_status gl_census(gl_ctx* ctx, const double* params, int64_t n_sets, const double* times,
                    const int64_t* offsets, int64_t n_times, const int32_t* n_ss,
                    const double* t_exp, double* out, void* stream, int64_t* counts)
{
    if (!counts) return GL_ERR_NULL;
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    gl_status st = check_args(ctx, b);
    if (st != GL_OK) return st;
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    st = prepare_batch(ctx, b);
    if (st != GL_OK) return st;
    st = enqueue(ctx, b, true);
    if (st != GL_OK) return st;
    GL_HIP(hipStreamSynchronize(b.stream), "hipStreamSynchronize");
    std::vector<LineCount> c((size_t)kCensus * kShards);
    GL_HIP(hipMemcpy(c.data(), ctx->ctr->census, sizeof(LineCount) * c.size(), hipMemcpyDeviceToHost), "hipMemcpy");
    for (int i = 0; i < kCensus; ++i) {
        unsigned long long t = 0;
        for (int j = 0; j < kShards; ++j) t += c[(size_t)i * kShards + j].v;
        counts[i] = (int64_t)t;
    }
    return GL_OK;
}

gl_status gl_flop_model(int64_t* per_item)
{
    if (!per_item) return GL_ERR_NULL;
    per_item[0] = gl::kFlopSample;
    per_item[1] = gl::kFlopWhole;
    per_item[2] = gl::kFlopPartial;
    per_item[3] = 0;
    per_item[4] = gl::kFlopTrapNode;
    per_item[5] = gl::kFlopGKPiece;
    per_item[6] = gl::kFlopIter;
    per_item[7] = gl::kFlopLimb;
    per_item[8] = gl::kFlopTrapNode;
    per_item[9] = gl::kFlopArc;
    per_item[10] = 0;  // unconverged arcs: their pieces are already counted
    return GL_OK;
}

gl_status gl_lightcurve_batch_snap(gl_ctx* ctx, int n_nodes, const double* params, int64_t n_sets,
                                   const double* times, const int64_t* offsets, int64_t n_times,
                                   const int32_t* n_ss, const double* t_exp, double* out, void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    gl_status st = check_args(ctx, b);
    if (st != GL_OK) return st;
    if (n_nodes < 4 || n_nodes > (1 << 20) || n_nodes % 2) return fail(ctx, GL_ERR_SIZE, "n_nodes even in [4, 2^20]");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    st = ensure_ws(ctx, n_sets, b.max_chunks);
    if (st != GL_OK) return st;
    hipStream_t s = b.stream;
    const int shared = b.offsets ? 0 : 1;
    const int64_t cps_shared = shared ? (b.n_times + kChunk - 1) / kChunk : 0;
    hipLaunchKernelGGL(k_prep<0>, dim3((unsigned)((n_sets + 255) / 256)), dim3(256), 0, s, params, n_sets, n_sets,
                       offsets, n_times, n_ss, t_exp, ctx->sc, ctx->seg_begin, ctx->seg_len, ctx->chunk_off, ctx->ctr,
                       cps_shared, 1, 1, (gl::SetConst*)nullptr, (const double*)nullptr, (int64_t)0, (double*)nullptr, 0, 0, (int64_t)0, 0);
    if (!shared)
        hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, s, ctx->chunk_off, n_sets, b.max_chunks, ctx->ctr);
    launch_window(ctx, b, s);
    if (n_nodes > ctx->snap_cap) {
        GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
        (void)hipFree(ctx->snap_cs);
        ctx->snap_cs = nullptr;
        ctx->snap_cap = 0;
        if (hipMalloc(&ctx->snap_cs, sizeof(float2) * n_nodes) != hipSuccess) return fail(ctx, GL_ERR_NOMEM, "node table");
        ctx->snap_cap = n_nodes;
        ctx->snap_n = 0;
    }
    if (ctx->snap_n != n_nodes) {
        hipLaunchKernelGGL(k_snap_nodes, dim3((unsigned)((n_nodes + 255) / 256)), dim3(256), 0, s, n_nodes, ctx->snap_cs);
        ctx->snap_n = n_nodes;
    }
    // a workgroup per chunk (the dispatcher balances chunks of unequal work)
    const unsigned grid = (unsigned)std::min<int64_t>(b.max_chunks, (int64_t)INT32_MAX);
    hipLaunchKernelGGL(k_snap, dim3(grid), dim3(64 * kSnapWaves), 0, s, times, shared, ctx->sc, ctx->seg_begin,
                       ctx->chunk_off, ctx->ctr, ctx->masks, ctx->chunk_set, n_nodes, ctx->snap_cs, out);
    GL_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

gl_status gl_ctx_get_overflow(gl_ctx* ctx, int64_t* fused_chunks, int* passes)
{
    if (!ctx || !fused_chunks) return GL_ERR_NULL;
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    *fused_chunks = 0;  // no work lists: nothing can overflow them
    if (passes) *passes = ctx->passes;
    return GL_OK;
}

gl_status gl_ctx_get_unconverged(gl_ctx* ctx, int64_t* n_arcs)
{
    if (!ctx || !n_arcs) return GL_ERR_NULL;
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    unsigned long long u = 0;
    GL_HIP(hipMemcpy(&u, &ctx->ctr->unconverged, sizeof(u), hipMemcpyDeviceToHost), "hipMemcpy");
    if (u) {
        GL_HIP(hipMemset(&ctx->ctr->unconverged, 0, sizeof(u)), "hipMemset");
        GL_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    }
    *n_arcs = (int64_t)u;
    return GL_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- allocation-free batch
// For callers that cannot allocate device memory (code under stream capture,
// tight serving loops): the whole exact path with its workspace carved out of
// one file-scope device array.  Every call on a device shares that device's
// array: calls that overlap on one device race.
namespace {

constexpr int64_t kStaticSets = 16384;              // parameter sets per call
constexpr int64_t kStaticChunks = (int64_t)1 << 18;  // 64-output chunks per call (16.7 M outputs)
constexpr int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

// byte offsets of the parts of the array
constexpr int64_t kOffCtr = 0;
constexpr int64_t kOffSc = align256(kOffCtr + (int64_t)sizeof(Counters));
constexpr int64_t kOffSegB = align256(kOffSc + kStaticSets * (int64_t)sizeof(gl::SetConst));
constexpr int64_t kOffSegL = align256(kOffSegB + kStaticSets * 8);
constexpr int64_t kOffChOff = align256(kOffSegL + kStaticSets * 8);
constexpr int64_t kScratchBytes = align256(kOffChOff + (kStaticSets + 1) * 8);
static_assert(kScratchBytes <= ((int64_t)6 << 20), "allocation-free workspace above its stated 6 MiB");

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of `scratch` and CU count, per device (found once per
// device, with that device current, on the first call there).
constexpr int kMaxDevices = 64;
unsigned char* g_scratch_dev[kMaxDevices] = {};
int g_scratch_cu[kMaxDevices] = {};
std::mutex g_scratch_mu;

}  // namespace

extern "C" gl_status gl_lightcurve_batch_noalloc(const double* params, int64_t n_sets, const double* times,
                                                 const int64_t* offsets, int64_t n_times, const int32_t* n_ss,
                                                 const double* t_exp, double* out, void* stream)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    gl_status st = check_batch(nullptr, b);
    if (st != GL_OK) return st;
    if (n_sets > kStaticSets || b.max_chunks > kStaticChunks) return GL_ERR_SIZE;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GL_ERR_DEVICE;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_dev[dev]) {
            void* ptr = nullptr;
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GL_ERR_DEVICE;
            int ncu = 0;
            if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
                ncu = 256;
            g_scratch_cu[dev] = ncu;
            g_scratch_dev[dev] = (unsigned char*)ptr;
        }
    }
    unsigned char* base = g_scratch_dev[dev];
    gl_ctx c;  // on the stack, pointing into this device's array only (it owns no memory)
    c.device = dev;
    c.n_cu = g_scratch_cu[dev];
    c.use_graph = false;
    c.ctr = (Counters*)(base + kOffCtr);
    c.sc = (gl::SetConst*)(base + kOffSc);
    c.seg_begin = (int64_t*)(base + kOffSegB);
    c.seg_len = (int64_t*)(base + kOffSegL);
    c.chunk_off = (int64_t*)(base + kOffChOff);
    c.cap_sets = kStaticSets;
    c.passes = 1;
    // (nothing to clear: k_prep writes the counters this call reads, and the
    // status is not reported)
    b.waves = flux_waves(b);
    b.range = flux_range(b);
    b.halvings = flux_halvings(b);
    return enqueue_flux<false>(&c, b);
}

// ---------------------------------------------------------------- surrogate path
namespace {

// One sample per parameter set: features, scaled residual target
// (F_oblate - F_sphere) / scale, both fluxes, the scale and the bin.
__global__ void k_sur_samples(const double* __restrict__ params, int64_t n, const double* __restrict__ times,
                              float* __restrict__ feat, float* __restrict__ target, double* __restrict__ f_obl,
                              double* __restrict__ f_sph, double* __restrict__ scale_out,
                              int* __restrict__ bin_out, Counters* __restrict__ ctr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double p[GL_NPARAM];
    for (int r = 0; r < GL_NPARAM; ++r) p[r] = params[(int64_t)r * n + i];
    gl::SetConst S;
    float fe[gl::kSurFeat];
    for (int r = 0; r < gl::kSurFeat; ++r) fe[r] = 0.f;
    double Fo = 1.0, Fs = 1.0, sc = 0.0;
    int bin = -1;
    gl::NoCensus nc;
    if (!gl::make_set_const(p, 0.0, 1, S) || !gl::finite_d(times[i])) {
        atomicOr(&ctr->status, 1u);
        Fo = Fs = __builtin_nan("");
    } else {
        double x0, y0;
        if (gl::centre_at(S, times[i], x0, y0) && gl::sur_encode(S, x0, y0, fe, sc, bin)) {
            Fo = 1.0 - gl::occulted<gl::NoCensus>(S, x0, y0, nullptr, nc);
            const gl::SetConst C = gl::sphere_of(S);
            Fs = 1.0 - gl::occulted<gl::NoCensus>(C, x0, y0, nullptr, nc);
        }
    }
    unconverged_add(ctr, nc.unconv, false);
    for (int r = 0; r < gl::kSurFeat; ++r) feat[i * gl::kSurFeat + r] = fe[r];
    target[i] = bin >= 0 ? (float)((Fo - Fs) / sc) : 0.f;
    if (f_obl) f_obl[i] = Fo;
    if (f_sph) f_sph[i] = Fs;
    if (scale_out) scale_out[i] = sc;
    if (bin_out) bin_out[i] = bin;
}

// Counter-based uniform draws in [0, 1): SplitMix64 of (seed, sample, column)
__device__ __forceinline__ double u01(uint64_t seed, int64_t i, int col)
{
    uint64_t z = seed ^ ((uint64_t)i * 0xd1342543de82ef95ull) ^ ((uint64_t)(col + 1) * 0x9e3779b97f4a7c15ull);
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return (double)(z >> 11) * 0x1.0p-53;
}

// Training / calibration draws from the walker priors: k ~ U[0.05, 0.12],
// f ~ U[0, 0.9], theta ~ U[0, pi], phi ~ U[0, 2 pi), b ~ U[0, 0.9],
// a/R* ~ U[100, 300], q1, q2 ~ U[0, 1], P = 500 d, t0 = 0; one time per
// sample uniform in +-window * T14 (the transit duration of the sphere of
// radius k, T14 = (P / pi) asin(sqrt((1 + k)^2 - b^2) / (a/R* sin i)),
// sin i = sqrt(1 - (b / a/R*)^2)).
__global__ void k_sur_draw(uint64_t seed, int64_t n, double window, double* __restrict__ params,
                           double* __restrict__ times)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double k = 0.05 + 0.07 * u01(seed, i, 0);
    const double f = 0.9 * u01(seed, i, 1);
    const double th = gl::kPi * u01(seed, i, 2);
    const double ph = gl::kTwoPi * u01(seed, i, 3);
    const double b = 0.9 * u01(seed, i, 4);
    const double ars = 100.0 + 200.0 * u01(seed, i, 5);
    const double q1 = u01(seed, i, 6), q2 = u01(seed, i, 7);
    const double P = 500.0;
    const double sini = sqrt(1.0 - (b / ars) * (b / ars));
    const double t14 = P / gl::kPi * asin(fmin(1.0, sqrt((1.0 + k) * (1.0 + k) - b * b) / (ars * sini)));
    const double vals[GL_NPARAM] = {k, f, th, ph, b, ars, P, 0.0, q1, q2};
    for (int r = 0; r < GL_NPARAM; ++r) params[(int64_t)r * n + i] = vals[r];
    times[i] = (2.0 * u01(seed, i, 8) - 1.0) * window * t14;
}

constexpr int kKeepBlock = 1024;  // rows per block of the on-star compaction

// rows with bin >= 0 per block of kKeepBlock rows
__global__ void __launch_bounds__(256) k_keep_count(const int* __restrict__ bin, int64_t n, int64_t* __restrict__ cnt)
{
    __shared__ int red[4];
    const int64_t r0 = (int64_t)blockIdx.x * kKeepBlock;
    int c = 0;
    for (int k = threadIdx.x; k < kKeepBlock; k += 256)
        if (r0 + k < n && bin[r0 + k] >= 0) ++c;
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// exclusive scan of a[0..n) in place, a[n] = total (one workgroup)
__global__ void __launch_bounds__(kScanThreads) k_excl_scan(int64_t* __restrict__ a, int64_t n)
{
    __shared__ int64_t part[kScanThreads];
    const int tid = threadIdx.x;
    const int64_t per = (n + kScanThreads - 1) / kScanThreads;
    const int64_t lo = std::min<int64_t>(n, per * tid), hi = std::min<int64_t>(n, lo + per);
    int64_t sum = 0;
    for (int64_t i = lo; i < hi; ++i) sum += a[i];
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < kScanThreads; d <<= 1) {
        const int64_t v = (tid >= d) ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t run = part[tid] - sum;
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t v = a[i];
        a[i] = run;
        run += v;
    }
    if (tid == kScanThreads - 1) a[n] = part[tid];
}

// the rows with bin >= 0, in order, as BF16 features and FP32 targets
__global__ void __launch_bounds__(256)
k_keep_write(const float* __restrict__ feat, const float* __restrict__ target, const int* __restrict__ bin, int64_t n,
             const int64_t* __restrict__ off, uint16_t* __restrict__ X, float* __restrict__ T)
{
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * kKeepBlock;
    int64_t base = off[blockIdx.x];
    for (int k0 = 0; k0 < kKeepBlock; k0 += 256) {
        const int64_t r = r0 + k0 + threadIdx.x;
        const bool keep = r < n && bin[r] >= 0;
        const unsigned long long m = __ballot(keep);
        if (lane == 0) wsum[wv] = __popcll(m);
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wv; ++w) before += wsum[w];
        if (keep) {
            const int64_t o = base + before + lanes_below(m);
            for (int f = 0; f < gl::kSurFeat; ++f) X[o * gl::kSurFeat + f] = gl::f2bf_rne(feat[r * gl::kSurFeat + f]);
            T[o] = target[r];
        }
        base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
}

// Calibration: per bin the largest |prediction - target| of the network and
// of the zero predictor (float bits of non-negative values order like
// integers, so an integer maximum is exact and order-independent) and the
// sample count
__global__ void k_sur_calib(const float* __restrict__ pred, const float* __restrict__ target,
                            const int* __restrict__ bin, int64_t n, unsigned int* __restrict__ err_net,
                            unsigned int* __restrict__ err_zero, int* __restrict__ counts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || bin[i] < 0) return;
    auto up = [](double e) {  // rounded up to float
        float x = (float)e;
        if ((double)x < e) x = __uint_as_float(__float_as_uint(x) + 1u);
        return __float_as_uint(x);
    };
    const double t = (double)target[i];
    atomicMax(&err_net[bin[i]], up(fabs((double)pred[i] - t)));
    atomicMax(&err_zero[bin[i]], up(fabs(t)));
    atomicAdd(&counts[bin[i]], 1);
}

// table[b] = the smaller calibrated bound of the two predictors (the zero
// predictor only, with zero_only), -1 where fewer than min_count samples
// fell; zero[b] = 1 where the sphere alone is taken
__global__ void k_sur_finalize(const unsigned int* __restrict__ err_net, const unsigned int* __restrict__ err_zero,
                               const int* __restrict__ counts, int min_count, int zero_only, float* __restrict__ table,
                               uint8_t* __restrict__ zero)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= gl::kSurBins) return;
    const float en = __uint_as_float(err_net[b]), ez = __uint_as_float(err_zero[b]);
    const bool z = zero_only || ez <= en;
    zero[b] = z ? 1 : 0;
    table[b] = counts[b] >= min_count ? (z ? ez : en) : -1.0f;
}

}  // namespace

struct gl_surrogate {
    int device = 0;
    gl_mlp* net = nullptr;
    float* table = nullptr;      // device [kSurBins]
    uint8_t* zero = nullptr;     // device [kSurBins]
    int32_t* counts = nullptr;   // device [kSurBins]
    gl_surrogate_config cfg{};
};

namespace {

void sur_free(gl_surrogate* s)
{
    if (!s) return;
    (void)hipSetDevice(s->device);
    (void)hipDeviceSynchronize();
    gl_mlp_destroy(s->net);
    (void)hipFree(s->table);
    (void)hipFree(s->zero);
    (void)hipFree(s->counts);
    delete s;
}

gl_status sur_alloc(gl_ctx* ctx, const gl_surrogate_config& cfg, gl_surrogate** out)
{
    gl_surrogate* s = new (std::nothrow) gl_surrogate();
    if (!s) return fail(ctx, GL_ERR_NOMEM, "surrogate");
    s->device = ctx->device;
    s->cfg = cfg;
    gl_status st = gl_mlp_create(&s->net, ctx->device, cfg.batch);
    if (st != GL_OK) {
        delete s;
        return fail(ctx, st, "surrogate network");
    }
    if (hipMalloc(&s->table, sizeof(float) * gl::kSurBins) != hipSuccess ||
        hipMalloc(&s->zero, gl::kSurBins) != hipSuccess ||
        hipMalloc(&s->counts, sizeof(int32_t) * gl::kSurBins) != hipSuccess) {
        sur_free(s);
        return fail(ctx, GL_ERR_NOMEM, "surrogate tables");
    }
    *out = s;
    return GL_OK;
}

// He-uniform initial weights, zero biases, from a seeded host generator
void init_weights(uint64_t seed, float* w)
{
    uint64_t z = seed * 0x2545f4914f6cdd1dull + 1ull;
    auto next = [&z]() {
        z += 0x9e3779b97f4a7c15ull;
        uint64_t x = z;
        x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
        x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
        return (double)((x ^ (x >> 31)) >> 11) * 0x1.0p-53;
    };
    const int dims[6] = {GL_MLP_DIN, GL_MLP_WIDTH, GL_MLP_WIDTH, GL_MLP_WIDTH, GL_MLP_WIDTH, 1};
    int64_t o = 0;
    for (int l = 0; l < 5; ++l) {
        const int a = dims[l], b = dims[l + 1];
        const double lim = b != 1 ? std::sqrt(6.0 / a) : std::sqrt(3.0 / a);
        for (int64_t e = 0; e < (int64_t)a * b; ++e) w[o++] = (float)((2.0 * next() - 1.0) * lim);
        for (int e = 0; e < b; ++e) w[o++] = 0.0f;
    }
}

}  // namespace

extern "C" {

void gl_surrogate_config_default(gl_surrogate_config* c)
{
    if (!c) return;
    c->n_train = 20000000;
    c->n_calib = 1000000;
    c->epochs = 4;
    c->batch = 8192;
    c->lr = 2e-3f;
    c->lr_final = 1e-4f;
    c->safety = 4.0;
    c->min_bin_count = 200;
    c->window = 0.6;
    c->seed = 5;
    c->zero_predictor = 0;
}

gl_status gl_surrogate_samples(gl_ctx* ctx, const double* params, const double* times, int64_t n,
                               float* feat, float* target, double* f_obl, double* f_sph,
                               double* scale, int32_t* bin, void* stream)
{
    if (!ctx) return GL_ERR_NULL;
    ctx->err[0] = 0;
    if (!params || !times || !feat || !target) return fail(ctx, GL_ERR_NULL, "params, times, feat, target");
    if (n < 1) return fail(ctx, GL_ERR_SIZE, "n >= 1");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    hipLaunchKernelGGL(k_sur_samples, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, (hipStream_t)stream,
                       params, n, times, feat, target, f_obl, f_sph, scale, bin, ctx->ctr);
    GL_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

int gl_surrogate_num_bins(void) { return gl::kSurBins; }

gl_status gl_surrogate_train(gl_ctx* ctx, const gl_surrogate_config* cfg_in, gl_surrogate** out,
                             float* loss_history, void* stream)
{
    if (!ctx || !cfg_in || !out) return GL_ERR_NULL;
    *out = nullptr;
    ctx->err[0] = 0;
    const gl_surrogate_config cfg = *cfg_in;
    if (cfg.batch < 64 || cfg.batch % 64 || cfg.batch > (1 << 20) || cfg.epochs < 1 || cfg.epochs > 1000 ||
        cfg.n_train < cfg.batch || cfg.n_train > ((int64_t)1 << 31) || cfg.n_calib < 1 ||
        cfg.n_calib > ((int64_t)1 << 31) || !(cfg.lr > 0.f) || !(cfg.lr_final > 0.f) || !(cfg.safety > 0.0) ||
        cfg.min_bin_count < 1 || !(cfg.window > 0.0))
        return fail(ctx, GL_ERR_SIZE, "surrogate configuration out of range");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    hipStream_t st = (hipStream_t)stream;
    gl_surrogate* s = nullptr;
    gl_status rs = sur_alloc(ctx, cfg, &s);
    if (rs != GL_OK) return rs;
    std::vector<float> w0(gl_mlp_num_params());
    init_weights(cfg.seed + 2, w0.data());
    if (cfg.zero_predictor) std::fill(w0.begin(), w0.end(), 0.0f);
    rs = gl_mlp_set_weights(s->net, w0.data(), (int64_t)w0.size());
    if (rs != GL_OK) {
        sur_free(s);
        return fail(ctx, rs, "surrogate weights");
    }
    // sample buffers, sized for the larger of the two draws
    const int64_t nmax = std::max(cfg.n_train, cfg.n_calib);
    const int64_t nblk = (nmax + kKeepBlock - 1) / kKeepBlock;
    double *prm = nullptr, *tms = nullptr, *scl = nullptr;
    float *feat = nullptr, *tgt = nullptr, *Tk = nullptr, *pred = nullptr, *hist = nullptr;
    int *bin = nullptr;
    int64_t* koff = nullptr;
    uint16_t* Xk = nullptr;
    unsigned int *en = nullptr, *ez = nullptr;
    bool ok = hipMalloc(&prm, sizeof(double) * GL_NPARAM * nmax) == hipSuccess &&
              hipMalloc(&tms, sizeof(double) * nmax) == hipSuccess &&
              hipMalloc(&scl, sizeof(double) * nmax) == hipSuccess &&
              hipMalloc(&feat, sizeof(float) * gl::kSurFeat * nmax) == hipSuccess &&
              hipMalloc(&tgt, sizeof(float) * nmax) == hipSuccess && hipMalloc(&Tk, sizeof(float) * nmax) == hipSuccess &&
              hipMalloc(&pred, sizeof(float) * nmax) == hipSuccess &&
              hipMalloc(&hist, sizeof(float) * cfg.epochs) == hipSuccess &&
              hipMalloc(&bin, sizeof(int) * nmax) == hipSuccess &&
              hipMalloc(&koff, sizeof(int64_t) * (nblk + 1)) == hipSuccess &&
              hipMalloc(&Xk, sizeof(uint16_t) * gl::kSurFeat * nmax) == hipSuccess &&
              hipMalloc(&en, sizeof(unsigned int) * gl::kSurBins) == hipSuccess &&
              hipMalloc(&ez, sizeof(unsigned int) * gl::kSurBins) == hipSuccess;
    auto release = [&]() {
        void* b[] = {prm, tms, scl, feat, tgt, Tk, pred, hist, bin, koff, Xk, en, ez};
        for (void* q : b) (void)hipFree(q);
    };
    if (!ok) {
        release();
        sur_free(s);
        return fail(ctx, GL_ERR_NOMEM, "surrogate sample buffers");
    }
    auto draw = [&](uint64_t seed, int64_t n) {
        hipLaunchKernelGGL(k_sur_draw, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, seed, n, cfg.window, prm, tms);
        hipLaunchKernelGGL(k_sur_samples, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, prm, n, tms, feat, tgt,
                           nullptr, nullptr, scl, bin, ctx->ctr);
    };
    // training: the samples on the star, compacted in order
    int64_t n_keep = 0;
    if (!cfg.zero_predictor) {
        draw(cfg.seed, cfg.n_train);
        const int64_t nb = (cfg.n_train + kKeepBlock - 1) / kKeepBlock;
        hipLaunchKernelGGL(k_keep_count, dim3((unsigned)nb), dim3(256), 0, st, bin, cfg.n_train, koff);
        hipLaunchKernelGGL(k_excl_scan, dim3(1), dim3(kScanThreads), 0, st, koff, nb);
        hipLaunchKernelGGL(k_keep_write, dim3((unsigned)nb), dim3(256), 0, st, feat, tgt, bin, cfg.n_train, koff, Xk, Tk);
        ok = hipMemcpyAsync(&n_keep, koff + nb, sizeof(int64_t), hipMemcpyDeviceToHost, st) == hipSuccess &&
             hipStreamSynchronize(st) == hipSuccess && hipMemsetAsync(hist, 0, sizeof(float) * cfg.epochs, st) == hipSuccess;
        if (ok && n_keep >= cfg.batch) {
            rs = gl_net::train_rows(s->net, Xk, Tk, n_keep, cfg.epochs, cfg.batch, cfg.lr, cfg.lr_final, cfg.seed, hist, st);
            if (rs != GL_OK) ok = false;
        } else if (ok) {
            rs = GL_ERR_SIZE;
            ok = false;
        }
    }
    // calibration on fresh draws: the network's and the zero predictor's
    // largest scaled error per bin, and the counts
    if (ok) {
        draw(cfg.seed + 1, cfg.n_calib);
        const int64_t nc = cfg.n_calib;
        ok = hipMemsetAsync(en, 0, sizeof(unsigned int) * gl::kSurBins, st) == hipSuccess &&
             hipMemsetAsync(ez, 0, sizeof(unsigned int) * gl::kSurBins, st) == hipSuccess &&
             hipMemsetAsync(s->counts, 0, sizeof(int32_t) * gl::kSurBins, st) == hipSuccess;
        if (ok) {
            rs = gl_mlp_forward(s->net, feat, nc, pred, st);
            if (rs != GL_OK) ok = false;
        }
        if (ok) {
            hipLaunchKernelGGL(k_sur_calib, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, pred, tgt, bin, nc, en, ez,
                               s->counts);
            hipLaunchKernelGGL(k_sur_finalize, dim3((gl::kSurBins + 255) / 256), dim3(256), 0, st, en, ez, s->counts,
                               cfg.min_bin_count, cfg.zero_predictor, s->table, s->zero);
            ok = hipGetLastError() == hipSuccess && hipStreamSynchronize(st) == hipSuccess;
            if (ok && loss_history) {
                if (cfg.zero_predictor) std::fill(loss_history, loss_history + cfg.epochs, 0.0f);
                else ok = hipMemcpy(loss_history, hist, sizeof(float) * cfg.epochs, hipMemcpyDeviceToHost) == hipSuccess;
            }
        }
    }
    release();
    if (!ok) {
        sur_free(s);
        return fail(ctx, rs != GL_OK ? rs : GL_ERR_DEVICE,
                    rs == GL_ERR_SIZE ? "too few training samples on the star for one batch" : "surrogate training");
    }
    *out = s;
    return GL_OK;
}

void gl_surrogate_destroy(gl_surrogate* s) { sur_free(s); }

gl_status gl_surrogate_get(const gl_surrogate* s, float* params, int64_t n_params, float* table, uint8_t* zero_bins,
                           int32_t* counts, int n_bins)
{
    if (!s) return GL_ERR_NULL;
    if (n_bins != gl::kSurBins || (params && n_params != gl_mlp_num_params())) return GL_ERR_SIZE;
    if (hipSetDevice(s->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return GL_ERR_DEVICE;
    if (params && gl_mlp_get_weights(s->net, params, n_params) != GL_OK) return GL_ERR_DEVICE;
    if (table && hipMemcpy(table, s->table, sizeof(float) * n_bins, hipMemcpyDeviceToHost) != hipSuccess)
        return GL_ERR_DEVICE;
    if (zero_bins && hipMemcpy(zero_bins, s->zero, n_bins, hipMemcpyDeviceToHost) != hipSuccess) return GL_ERR_DEVICE;
    if (counts && hipMemcpy(counts, s->counts, sizeof(int32_t) * n_bins, hipMemcpyDeviceToHost) != hipSuccess)
        return GL_ERR_DEVICE;
    return GL_OK;
}

gl_status gl_surrogate_config_of(const gl_surrogate* s, gl_surrogate_config* cfg)
{
    if (!s || !cfg) return GL_ERR_NULL;
    *cfg = s->cfg;
    return GL_OK;
}

gl_status gl_surrogate_save(const gl_surrogate* s, const char* path)
{
    if (!s || !path) return GL_ERR_NULL;
    const int np = gl_mlp_num_params();
    std::vector<float> w(np), m(np), v(np), table(gl::kSurBins);
    std::vector<uint8_t> zero(gl::kSurBins);
    std::vector<int32_t> counts(gl::kSurBins);
    int64_t step = 0;
    gl_status st = gl_surrogate_get(s, w.data(), np, table.data(), zero.data(), counts.data(), gl::kSurBins);
    if (st != GL_OK) return st;
    st = gl_net::get_state(s->net, m.data(), v.data(), &step);
    if (st != GL_OK) return st;
    return gl_surrogate_file_write(path, &s->cfg, w.data(), m.data(), v.data(), step, np, table.data(), zero.data(),
                                   counts.data(), gl::kSurBins);
}

gl_status gl_surrogate_load(gl_ctx* ctx, gl_surrogate** out, const char* path)
{
    if (!ctx || !out || !path) return GL_ERR_NULL;
    *out = nullptr;
    ctx->err[0] = 0;
    const int np = gl_mlp_num_params();
    std::vector<float> w(np), m(np), v(np), table(gl::kSurBins);
    std::vector<uint8_t> zero(gl::kSurBins);
    std::vector<int32_t> counts(gl::kSurBins);
    int64_t step = 0;
    gl_surrogate_config cfg{};
    gl_status st = gl_surrogate_file_read(path, &cfg, w.data(), m.data(), v.data(), &step, np, table.data(),
                                          zero.data(), counts.data(), gl::kSurBins);
    if (st != GL_OK) return fail(ctx, st, "surrogate file");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    gl_surrogate* s = nullptr;
    st = sur_alloc(ctx, cfg, &s);
    if (st != GL_OK) return st;
    if (gl_mlp_set_weights(s->net, w.data(), np) != GL_OK || gl_net::set_state(s->net, m.data(), v.data(), step) != GL_OK ||
        hipMemcpy(s->table, table.data(), sizeof(float) * gl::kSurBins, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->zero, zero.data(), gl::kSurBins, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->counts, counts.data(), sizeof(int32_t) * gl::kSurBins, hipMemcpyHostToDevice) != hipSuccess) {
        sur_free(s);
        return fail(ctx, GL_ERR_DEVICE, "surrogate upload");
    }
    *out = s;
    return GL_OK;
}

gl_status gl_lightcurve_batch_surrogate(gl_ctx* ctx, const gl_surrogate* s, double tol, const double* params,
                                        int64_t n_sets, const double* times, const int64_t* offsets, int64_t n_times,
                                        const int32_t* n_ss, const double* t_exp, double* out, void* stream,
                                        int64_t* n_sub_out, int64_t* n_fallback_out)
{
    Batch b{params, n_sets, times, offsets, n_times, n_ss, t_exp, out, (hipStream_t)stream, 0};
    gl_status st = check_args(ctx, b);
    if (st != GL_OK) return st;
    if (!s) return fail(ctx, GL_ERR_NULL, "surrogate required");
    if (!(tol > 0.0)) return fail(ctx, GL_ERR_SIZE, "tol > 0");
    if (s->device != ctx->device) return fail(ctx, GL_ERR_STATE, "surrogate on another device");
    GL_HIP(hipSetDevice(ctx->device), "hipSetDevice");
    b.net = s->net;
    b.gate_table = s->table;
    b.gate_zero = s->zero;
    b.gate_k = s->cfg.safety / tol;
    st = prepare_batch(ctx, b);
    if (st != GL_OK) return st;
    st = run_batch(ctx, b, false);
    if (st != GL_OK) return st;
    st = finish_timed(ctx, b.stream);
    if (st != GL_OK) return st;
    if (n_sub_out || n_fallback_out) {
        unsigned long long c[3] = {0ull, 0ull, 0ull};  // in window, reaching the disk, accepted
        std::vector<LineCount> sh((size_t)3 * kShards);
        GL_HIP(hipStreamSynchronize(b.stream), "hipStreamSynchronize");
        GL_HIP(hipMemcpy(sh.data(), ctx->ctr->sur, sizeof(LineCount) * sh.size(), hipMemcpyDeviceToHost), "hipMemcpy");
        for (int r = 0; r < 3; ++r)
            for (int j = 0; j < kShards; ++j) c[r] += sh[(size_t)r * kShards + j].v;
        if (n_sub_out) *n_sub_out = (int64_t)c[0];
        if (n_fallback_out) *n_fallback_out = (int64_t)(c[1] - c[2]);
    }
    return GL_OK;
}

const char* gl_version(void) { return "0.1.0"; }

}  // extern "C"
