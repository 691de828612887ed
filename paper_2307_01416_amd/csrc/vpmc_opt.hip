// Spot-weight optimisation on influence matrices (the plan-optimisation
// step that consumes the 13-scenario matrices, Methods E).  The iterations run
// on the entries in structure voxels, renumbered to 0 .. nstruct - 1.  Per
// iteration:
//   forward  D_s = A_s^T w : one workgroup per (voxel chunk, scenario) sums
//            the row segments that fall in its chunk into int64 fixed-point
//            LDS accumulators (order-independent, so bit-reproducible), then
//            turns the chunk's dose into the objective residual;
//   gradient g_j = sum_s A_s[j,:] r_s : one wavefront per row piece, FP64 sums
//            in a fixed order;
//   update   a wavefront per spot (power iteration for the step size,
//            projected FISTA); per workgroup it leaves partial sums of the
//            next sweep's bound, which every forward workgroup adds up itself.
#include <hip/hip_runtime.h>

#include <math.h>

#include "vpmc_internal.hpp"

namespace vpmc {

namespace {

constexpr int kOptThreads = 256;
constexpr int kUpdThreads = 1024;
constexpr int kFwdThreads = 512;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ void set_err(unsigned *err, unsigned bit) {
    __hip_atomic_fetch_or(err, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// CSR row of (scenario s, spot j)
__device__ __forceinline__ long long csr_row(const OptDev &O, int s, int j) {
    return (long long)s * O.row_stride + O.row_offset + j;
}

// A wavefront's unit of the index passes: a piece of a row if the rows are cut
// into pieces, else a whole row.
__device__ __forceinline__ bool row_unit(const OptDev &O, int &r, long long &b, long long &e) {
    const long long u = (long long)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6);
    if (O.units) {
        if (u >= O.n_units) return false;
        const OptPiece q = O.units[u];
        r = __builtin_amdgcn_readfirstlane(q.row);
        b = q.begin;
        e = q.begin + q.len;
        return true;
    }
    if (u >= (long long)O.n_scen * O.n_spots) return false;
    r = (int)u;
    const long long crow = csr_row(O, r / O.n_spots, r % O.n_spots);
    b = O.row_ptr[crow];
    e = O.row_ptr[crow + 1];
    return true;
}

// Pass 1 over the rows: entries per (scenario, chunk), validation of the
// columns and values.  A segment is a maximal run of a
// row's entries inside one voxel chunk; it starts at every entry whose chunk
// differs from its predecessor's.
__global__ void __launch_bounds__(kOptThreads) opt_count_kernel(OptDev O, unsigned long long *cnt, unsigned *err) {
    int r;
    long long b, e;
    if (!row_unit(O, r, b, e)) return;
    const int s = r / O.n_spots;
    const int lane = lane_id();
    int carry = -1;
    for (long long i0 = b; i0 < e; i0 += 64) {
        const long long i = i0 + lane;
        const bool valid = i < e;
        int ck = -2;
        if (valid) {
            const int c = O.col[i];
            const float a = O.val[i];
            if ((unsigned)c >= (unsigned)O.nvox) set_err(err, 1u);
            else ck = c >> O.bits;
            if (!isfinite(a)) set_err(err, 2u);
        }
        int prev = __shfl_up(ck, 1);
        if (lane == 0) prev = carry;
        // entries per (scenario, chunk): one add per segment start, of the
        // segment's entry count inside this window; continuing segments add
        // the rest at the next window's lane 0
        const bool start = valid && ck >= 0 && (ck != prev || lane == 0);
        const unsigned long long m = __ballot(start);
        if (start) {
            const unsigned long long above = m & ~((2ull << lane) - 1ull);
            const long long stop = above ? i0 + (__ffsll((long long)above) - 1) : (i0 + 64 < e ? i0 + 64 : e);
            atomicAdd(&cnt[(size_t)s * O.nchunks + ck], (unsigned long long)(stop - i));
        }
        carry = __shfl(ck, 63);
    }
}

// Exclusive scan of n counts into off[0..n] by one workgroup, a tile of one
// count per thread at a time (with a run of counts per thread, 66 560 counts
// were 615 us); the counts are cleared (they serve next as the emit pass's
// cursors).
__global__ void __launch_bounds__(kUpdThreads) opt_scan_kernel(unsigned long long *cnt, unsigned long long *off, size_t n) {
    __shared__ unsigned long long part[2][kUpdThreads / 64];
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    unsigned long long before = 0;
    int flip = 0;
    for (size_t k0 = 0; k0 < n; k0 += kUpdThreads, flip ^= 1) {
        const size_t k = k0 + threadIdx.x;
        const unsigned long long own = k < n ? cnt[k] : 0ull;
        unsigned long long sum = own;
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned long long o = __shfl_up(sum, d);
            if (lane >= d) sum += o;
        }
        if (lane == 63) part[flip][w] = sum;
        __syncthreads();
        unsigned long long total = 0;
        for (int q = 0; q < kUpdThreads / 64; ++q) {
            if (q == w) sum += total;
            total += part[flip][q];
        }
        if (k < n) {
            off[k] = before + sum - own;
            cnt[k] = 0ull;
        }
        before += total;
    }
    if (threadIdx.x == 0) off[n] = before;
}

// Structure voxels: per 64 voxels a mask of those with a structure bit, with
// the structure voxels before it inside its block of 4096 (opt_rank_kernel
// adds those of earlier blocks).  The masks of 10.5 M voxels are 2.6 MB and stay
// in L2, where the row passes below look every entry up; the host loops and
// copies over all voxels that built a 42 MB index took 12 ms.  `keep` gets a
// copy for the comparison of a later call.
__global__ void __launch_bounds__(kOptThreads) opt_mask_kernel(const uint8_t *roi, int nvox, OptMask *mask,
                                                               unsigned long long *cnt, uint8_t *keep) {
    __shared__ unsigned wsum[4];
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    const size_t word0 = (size_t)blockIdx.x * 64 + (size_t)w * 16;
    unsigned long long mine = 0;   // lane k < 16: mask of word word0 + k
    uint8_t m[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const size_t v = (word0 + k) * 64 + lane;
        m[k] = v < (size_t)nvox ? roi[v] : (uint8_t)0;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const size_t v = (word0 + k) * 64 + lane;
        if (v < (size_t)nvox) keep[v] = m[k];
        const unsigned long long bits = __ballot(m[k] != 0);
        if (lane == k) mine = bits;
    }
    unsigned sum = (unsigned)__popcll(mine);
    const unsigned own = sum;
    for (int d = 1; d < 16; d <<= 1) {
        const unsigned o = __shfl_up(sum, d);
        if (lane >= d) sum += o;
    }
    if (lane == 15) wsum[w] = sum;
    __syncthreads();
    unsigned before = sum - own;
    for (int q = 0; q < w; ++q) before += wsum[q];
    if (lane < 16 && (word0 + lane) * 64 < (size_t)nvox) mask[word0 + lane] = OptMask{mine, before, 0u};
    if (threadIdx.x == 0) cnt[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

__device__ __forceinline__ uint32_t rank_of(const OptMask &m, int v) {
    return m.before + (uint32_t)__popcll(m.bits & ((1ull << (v & 63)) - 1ull));
}

// masks' ranks over all blocks, and the structure bits of each structure voxel
__global__ void __launch_bounds__(kOptThreads) opt_rank_kernel(const uint8_t *roi, int nvox, OptMask *mask,
                                                               const unsigned long long *off, uint8_t *sroi) {
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    const size_t word0 = (size_t)blockIdx.x * 64 + (size_t)w * 16;
    const uint32_t before = (uint32_t)off[blockIdx.x];
    for (int k = 0; k < 16; ++k) {
        const size_t v = (word0 + k) * 64 + lane;
        if ((word0 + k) * 64 >= (size_t)nvox) break;
        OptMask m = mask[word0 + k];
        m.before += before;
        if (m.bits >> lane & 1ull) sroi[rank_of(m, (int)v)] = roi[v];
        if (lane == 0) mask[word0 + k].before = m.before;
    }
}

__global__ void __launch_bounds__(kOptThreads) opt_roi_same_kernel(const uint8_t *a, const uint8_t *b, int nvox,
                                                                   unsigned *err) {
    bool diff = false;
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < (size_t)nvox; v += (size_t)gridDim.x * blockDim.x)
        diff |= a[v] != b[v];
    if (__ballot(diff) && lane_id() == 0) set_err(err, 1u);
}

// Restriction to the structures: the objective and its gradient involve only
// voxels with a structure bit, so the iterations run on the rows' entries in
// those voxels.  A workgroup per row, each wavefront on one of kRoiParts parts
// of it (a row of 11 000 entries by one wavefront was a chain of 175 loads:
// 390 and 480 us for 87 M entries, with the parts and four loads in flight 150
// and 200).  Count pass (also validates every entry and takes the largest |a|
// of the whole row) and copy pass (entries kept in row order, columns
// renumbered to structure voxels).
constexpr int kRoiThreads = 64 * kRoiParts;

__device__ __forceinline__ void roi_part(long long &b, long long &e) {
    const long long per = ((e - b + 64 * kRoiParts - 1) / (64 * kRoiParts)) * 64;
    b = b + per * (long long)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    e = b + per < e ? b + per : e;
}

__global__ void __launch_bounds__(kRoiThreads) opt_roi_count_kernel(OptDev O, const OptMask *mask, unsigned *rcnt,
                                                                    unsigned *err) {
    __shared__ float wmax[kRoiParts];
    for (int r = (int)blockIdx.x; r < O.n_scen * O.n_spots; r += (int)gridDim.x) {
        const int s = r / O.n_spots, j = r - s * O.n_spots;
        const long long crow = csr_row(O, s, j);
        long long b = O.row_ptr[crow], e = O.row_ptr[crow + 1];
        roi_part(b, e);
        const int lane = lane_id();
        float amax = 0.0f;
        unsigned kept = 0, bad = 0;
        for (long long i = b + lane; i < e; i += 256) {
            int c[4];
            float a[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = i + 64 * u < e;
                c[u] = in ? O.col[i + 64 * u] : 0;
                a[u] = in ? O.val[i + 64 * u] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i + 64 * u >= e) continue;
                if ((unsigned)c[u] >= (unsigned)O.nvox) bad |= 1u;
                else kept += (unsigned)(mask[c[u] >> 6].bits >> (c[u] & 63)) & 1u;
                if (!isfinite(a[u])) bad |= 2u;
                else amax = fmaxf(amax, fabsf(a[u]));
            }
        }
        if (bad) set_err(err, bad);
        for (int o = 32; o > 0; o >>= 1) {
            amax = fmaxf(amax, __shfl_xor(amax, o));
            kept += __shfl_xor(kept, o);
        }
        if (lane == 0) {
            wmax[threadIdx.x >> 6] = amax;
            rcnt[(size_t)r * kRoiParts + (threadIdx.x >> 6)] = kept;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int q = 1; q < kRoiParts; ++q) amax = fmaxf(amax, wmax[q]);
            O.amax[r] = amax;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kRoiThreads) opt_roi_copy_kernel(OptDev O, const OptMask *mask, const unsigned *rcnt,
                                                                   const long long *rptr, int32_t *ccol, float *cval) {
    for (int r = (int)blockIdx.x; r < O.n_scen * O.n_spots; r += (int)gridDim.x) {
        const int s = r / O.n_spots, j = r - s * O.n_spots;
        const long long crow = csr_row(O, s, j);
        long long b = O.row_ptr[crow], e = O.row_ptr[crow + 1];
        roi_part(b, e);
        const int lane = lane_id();
        const long long o1 = rptr[r + 1];
        long long out = rptr[r];
        for (unsigned q = 0; q < threadIdx.x >> 6; ++q) out += rcnt[(size_t)r * kRoiParts + q];
        for (long long i0 = b; i0 < e; i0 += 256) {
            int c[4];
            float a[4];
            OptMask m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long i = i0 + 64 * u + lane;
                c[u] = i < e ? O.col[i] : -1;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                m[u] = (unsigned)c[u] < (unsigned)O.nvox ? mask[c[u] >> 6] : OptMask{0ull, 0u, 0u};
                const bool keep = m[u].bits >> (c[u] & 63) & 1ull;
                a[u] = keep ? O.val[i0 + 64 * u + lane] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool keep = m[u].bits >> (c[u] & 63) & 1ull;
                const unsigned long long k = __ballot(keep);
                const long long pos = out + __popcll(k & ((1ull << lane) - 1ull));
                if (keep && pos < o1) {
                    ccol[pos] = (int32_t)rank_of(m[u], c[u]);
                    cval[pos] = a[u];
                }
                out += __popcll(k);
            }
        }
    }
}

// Pass 2 over the rows: the entries of every segment of a 64-entry window go,
// as one block, into the entry range of its (scenario, chunk) list: key (spot <<
// bits | voxel - chunk base) and value.  The segments' first lanes claim their
// blocks in one step (a claim per segment after the other was 31 us for one
// row of 1000 entries in chunks of 32 voxels).  The order of blocks inside a
// list does not matter (the dose sums are integers).
__global__ void __launch_bounds__(kOptThreads) opt_emit_kernel(OptDev O, const unsigned long long *off,
                                                               unsigned long long *cur, uint32_t *bkey, float *bval) {
    int r;
    long long b, e;
    if (!row_unit(O, r, b, e)) return;
    const int s = r / O.n_spots, j = r - s * O.n_spots;
    const int lane = lane_id();
    const uint32_t hi = (uint32_t)j << O.bits, low = (1u << O.bits) - 1u;
    for (long long i0 = b; i0 < e; i0 += 64) {
        const long long i = i0 + lane;
        const bool valid = i < e;
        int c = -1, ck = -2;
        float a = 0.0f;
        if (valid) {
            c = O.col[i];
            a = O.val[i];
            if ((unsigned)c < (unsigned)O.nvox) ck = c >> O.bits;
        }
        const int prev = __shfl_up(ck, 1);
        const bool start = valid && ck >= 0 && (lane == 0 || ck != prev);
        const unsigned long long m = __ballot(start);
        unsigned long long pos = ~0ull;
        if (start) {
            const unsigned long long above = m & ~((2ull << lane) - 1ull);
            const long long stop = above ? i0 + (__ffsll((long long)above) - 1) : (i0 + 64 < e ? i0 + 64 : e);
            const size_t list = (size_t)s * O.nchunks + ck;
            pos = off[list] + atomicAdd(&cur[list], (unsigned long long)(stop - i));
            if (pos + (unsigned long long)(stop - i) > off[list + 1]) pos = ~0ull;   // cannot happen after a consistent count pass
        }
        const unsigned long long at = m & ((2ull << lane) - 1ull);
        const int first = at ? 63 - __clzll((long long)at) : lane;
        pos = __shfl(pos, first);
        if (valid && ck >= 0 && at && pos != ~0ull) {
            pos += (unsigned long long)(lane - first);
            bkey[pos] = hi | ((uint32_t)c & low);
            bval[pos] = a;
        }
    }
}

// Block-wide sum in a fixed order, the same in every thread.
template <int N>
__device__ double block_sum(double v, double *red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < N / 64; ++q) t += red[q];
    return t;
}

// fixed-point exponent of a sweep over vector w of bound sum_j |w_j| max|A_s[j,:]|:
// 2^m bound < 2^60, so every int64 sum stays in range
__device__ __forceinline__ int scale_exp(double bnd) {
    int ex = 0;
    if (!(bnd > 0.0)) return 0;
    (void)frexp(bnd, &ex);
    return 60 - ex;
}

// Forward sweep of one (scenario, chunk) item of the work list (items in
// decreasing entry count).  mode 0: objective residual and objective partial;
// mode 1: residual M D of the power iteration (M = the target and organ
// weights); mode 2: as mode 0 and the dose into dose_out.
__global__ void __launch_bounds__(kFwdThreads) opt_forward_kernel(OptDev O, const double *w, int mode, float *dose_out) {
    __shared__ unsigned long long acc[1 << kOptMaxBits];
    __shared__ double red[kFwdThreads / 64];
    const OptWork item = O.work[blockIdx.x];
    const int s = (int)(item.list / (unsigned)O.nchunks), c = (int)(item.list - (unsigned)s * O.nchunks);
    const int chunk = 1 << O.bits;
    const long long base = (long long)c << O.bits;
    const int nv = (int)(O.nvox - base < chunk ? O.nvox - base : chunk);
    for (int v = threadIdx.x; v < chunk; v += kFwdThreads) acc[v] = 0ull;
    // the bound of this sweep: the update's partials of scenario s
    double bnd = 0.0;
    for (int k = threadIdx.x; k < O.n_part; k += kFwdThreads) bnd += O.bpart[(size_t)s * O.n_part + k];
    bnd = block_sum<kFwdThreads>(bnd, red);
    const int m2 = scale_exp(bnd);
    const double sc = ldexp(1.0, m2), isc = ldexp(1.0, -m2);
    const long long e0 = item.begin, e1 = item.begin + item.len;
    const uint32_t *bk = O.bkey;
    const float *bv = O.bval;
    const uint32_t low = (uint32_t)chunk - 1u;
    long long e = e0 + threadIdx.x;
    for (; e + 3 * kFwdThreads < e1; e += 4 * kFwdThreads) {
        uint32_t k[4];
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            k[u] = bk[e + u * kFwdThreads];
            a[u] = bv[e + u * kFwdThreads];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = k[u] >> O.bits;
            if (j < (uint32_t)O.n_spots) {
                const double t = rint(w[j] * sc * (double)a[u]);
                atomicAdd(&acc[k[u] & low], (unsigned long long)(long long)t);
            }
        }
    }
    if (e < e1) {   // the rest in one step, not one load after the other
        uint32_t k[3];
        float a[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const bool in = e + u * kFwdThreads < e1;
            k[u] = in ? bk[e + u * kFwdThreads] : ~0u;
            a[u] = in ? bv[e + u * kFwdThreads] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const uint32_t j = k[u] >> O.bits;
            if (e + u * kFwdThreads < e1 && j < (uint32_t)O.n_spots) {
                const double t = rint(w[j] * sc * (double)a[u]);
                atomicAdd(&acc[k[u] & low], (unsigned long long)(long long)t);
            }
        }
    }
    __syncthreads();
    double f = 0.0;
    float *res = O.rstruct ? O.rstruct + (size_t)s * O.nvox + base : nullptr;
    const unsigned char *roi = O.roi + base;
    for (int v = threadIdx.x; v < nv; v += kFwdThreads) {
        const double D = (double)(long long)acc[v] * isc;
        const unsigned m = roi[v];
        double r = 0.0;
        if (mode == 1) {
            const double mw = ((m & 1u) ? O.w_target : 0.0) + ((m & 2u) ? O.w_oar : 0.0);
            r = mw * D;
        } else {
            if (m & 1u) {
                const double d = D - O.d_presc;
                r += O.w_target * d;
                f += O.w_target * d * d;
            }
            if (m & 2u) {
                const double d = D > O.d_max ? D - O.d_max : 0.0;
                r += O.w_oar * d;
                f += O.w_oar * d * d;
            }
            if (mode == 2 && dose_out) dose_out[(size_t)s * O.nvox + base + v] = (float)D;
        }
        if (res) res[v] = (float)r;
    }
    if (mode == 1) return;
    f = block_sum<kFwdThreads>(f, red);
    if (threadIdx.x == 0) O.fpart[blockIdx.x] = f;
}

// Gradient sweep: a wavefront per piece (at most kOptMaxPiece consecutive
// entries of one row), FP64 products of FP32 values (exact) summed per lane
// in entry order, then over lanes by a fixed butterfly; pieces of a row are
// summed in order by the update.
__global__ void __launch_bounds__(kOptThreads) opt_grad_kernel(OptDev O) {
    const long long p = (long long)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6);
    if (p >= O.n_pieces) return;
    const OptPiece q = O.piece[p];
    const int r = __builtin_amdgcn_readfirstlane(q.row);
    const int s = r / O.n_spots;
    // columns renumbered to structure voxels: the residual gathered is the
    // compact one (n_scen x nstruct floats, cache-resident)
    const float *res = O.rstruct + (size_t)s * O.nvox;
    const int lane = lane_id();
    const long long e = q.begin + q.len;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    long long i = q.begin + lane;
    for (; i + 192 < e; i += 256) {
        int c[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = O.col[i + 64 * u];
            v[u] = O.val[i + 64 * u];
        }
        float rr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) rr[u] = (unsigned)c[u] < (unsigned)O.nvox ? res[c[u]] : 0.0f;
        a0 = fma((double)v[0], (double)rr[0], a0);
        a1 = fma((double)v[1], (double)rr[1], a1);
        a2 = fma((double)v[2], (double)rr[2], a2);
        a3 = fma((double)v[3], (double)rr[3], a3);
    }
    if (i < e) {   // the rest in one step, not one load after the other
        int c[3];
        float v[3], rr[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const bool in = i + 64 * u < e;
            c[u] = in ? O.col[i + 64 * u] : -1;
            v[u] = in ? O.val[i + 64 * u] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) rr[u] = (unsigned)c[u] < (unsigned)O.nvox ? res[c[u]] : 0.0f;
        a0 = fma((double)v[0], (double)rr[0], a0);
        a1 = fma((double)v[1], (double)rr[1], a1);
        a2 = fma((double)v[2], (double)rr[2], a2);
    }
    double a = (a0 + a1) + (a2 + a3);
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
    if (lane == 0) O.gpart[p] = a;
}

// Sum over scenarios of A_s[j,:] r_s by one wavefront, the same in every lane:
// 64 >> shift lanes' groups of 2^shift take a row each, their lanes every
// 2^shift-th of its pieces, and a fixed butterfly sums the lanes.
__device__ double row_gradient(const OptDev &O, int j) {
    const int shift = O.n_scen <= 4 ? 4 : O.n_scen <= 16 ? 2 : 0;
    const int lane = lane_id();
    double g = 0.0;
    for (int s = lane >> shift; s < O.n_scen; s += 64 >> shift) {
        const size_t r = (size_t)s * O.n_spots + j;
        const long long p1 = O.piece_off[r + 1];
#pragma unroll 4
        for (long long p = O.piece_off[r] + (lane & ((1 << shift) - 1)); p < p1; p += 1 << shift) g += O.gpart[p];
    }
    for (int o = 32; o > 0; o >>= 1) g += __shfl_xor(g, o);
    return g;
}

// Objective over the forward sweep's partials, fixed order.
__device__ double objective(const OptDev &O, double *red) {
    const size_t n = (size_t)O.n_work;
    double f = 0.0;
    for (size_t k = threadIdx.x; k < n; k += kOptThreads) f += O.fpart[k];
    return block_sum<kOptThreads>(f, red) / (double)O.n_scen;
}

// A wavefront per spot, n_part workgroups over the spots.  Modes: kOptPowerInit
// (z = 1), kOptPower (g and its and z's square sums), kOptPowerNorm
// (lam = |g|/|z|, z = g/|g|), kOptFistaInit (L = 1.05 lam, x = max(x, 0), y = x),
// kOptFista (x+ = P(y - g/L), y = x+ + beta (x+ - x)), kOptFinalPrep (x as it
// is), kOptFinal (the objective alone).  A workgroup more (kOptFista,
// kOptFinal) sums the objective of the sweep into hist[it].  Each workgroup
// leaves sum_j |w_j| max|A_s[j,:]| over its spots for the next sweep's scale.
// One workgroup over all spots, a thread per spot, was 33 us for 600 spots and
// 13 scenarios (a chain of loads per spot, then 13 block sums), more than the
// gradient itself.
__global__ void __launch_bounds__(kOptThreads) opt_update_kernel(OptDev O, int mode, double beta, int it,
                                                                 double *hist) {
    __shared__ double red[kOptThreads / 64];
    if ((int)blockIdx.x == O.n_part || mode == kOptFinal) {
        const double F = objective(O, red);
        if (threadIdx.x == 0 && hist) hist[it] = F;
        return;
    }
    const int n = O.n_spots, lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int j0 = (int)blockIdx.x * (kOptThreads / 64) + wave, dj = O.n_part * (kOptThreads / 64);
    const double g_scale = 2.0 / (double)O.n_scen;
    double *gg = O.sq, *zz = O.sq + O.n_part;
    const double *w = mode == kOptPowerInit || mode == kOptPower || mode == kOptPowerNorm ? O.z
                      : mode == kOptFinalPrep ? O.x : O.y;
    if (mode == kOptPower) {
        double sg = 0.0, sz = 0.0;
        for (int j = j0; j < n; j += dj) {
            const double g = row_gradient(O, j) * g_scale;
            if (lane == 0) O.gvec[j] = g;
            sg += g * g;
            sz += O.z[j] * O.z[j];
        }
        sg = block_sum<kOptThreads>(lane == 0 ? sg : 0.0, red);
        sz = block_sum<kOptThreads>(lane == 0 ? sz : 0.0, red);
        if (threadIdx.x == 0) {
            gg[blockIdx.x] = sg;
            zz[blockIdx.x] = sz;
        }
        return;
    }
    double gn = 0.0, lam = 0.0;
    if (mode == kOptPowerNorm) {
        double sg = 0.0, sz = 0.0;
        for (int k = threadIdx.x; k < O.n_part; k += kOptThreads) {
            sg += gg[k];
            sz += zz[k];
        }
        gn = sqrt(block_sum<kOptThreads>(sg, red));
        const double zn = sqrt(block_sum<kOptThreads>(sz, red));
        lam = zn > 0.0 ? gn / zn : 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0) O.scal[kOptLam] = lam;
    }
    if (mode == kOptFistaInit && blockIdx.x == 0 && threadIdx.x == 0) O.scal[kOptL] = 1.05 * O.scal[kOptLam];
    const double L = mode == kOptFista ? O.scal[kOptL] : 0.0;
    double bnd = 0.0;   // of scenario `lane`
    for (int j = j0; j < n; j += dj) {   // every lane has the spot's values
        const double am = lane < O.n_scen ? (double)O.amax[(size_t)lane * n + j] : 0.0;
        const double x = O.x[j], y = O.y[j];
        double wj = x;
        if (mode == kOptPowerInit) wj = 1.0;
        if (mode == kOptPowerNorm) wj = gn > 0.0 ? O.gvec[j] / gn : O.z[j];
        if (mode == kOptFistaInit) wj = x > 0.0 ? x : 0.0;
        if (mode == kOptFista) {
            const double g = row_gradient(O, j) * g_scale;
            double xn = L > 0.0 ? y - g / L : y;
            xn = xn > 0.0 ? xn : 0.0;
            wj = xn + beta * (xn - x);
            if (lane == 0) O.x[j] = xn;
        }
        if (lane == 0) {
            if (mode == kOptPowerInit || mode == kOptPowerNorm) O.z[j] = wj;
            if (mode == kOptFistaInit) O.x[j] = wj;
            if (mode == kOptFistaInit || mode == kOptFista) O.y[j] = wj;
        }
        bnd += fabs(wj) * am;
    }
    __shared__ double wb[kOptThreads / 64][64];
    for (int s0 = 0;;) {
        const int s = s0 + lane;
        wb[wave][lane] = bnd;
        __syncthreads();   // also: the other lanes may read what lane 0 wrote
        if (wave == 0 && s < O.n_scen) {
            for (int q = 1; q < kOptThreads / 64; ++q) bnd += wb[q][lane];
            O.bpart[(size_t)s * O.n_part + blockIdx.x] = bnd;
        }
        if ((s0 += 64) >= O.n_scen) break;
        __syncthreads();
        bnd = 0.0;
        if (s0 + lane < O.n_scen)
            for (int j = j0; j < n; j += dj) bnd += fabs(w[j]) * (double)O.amax[(size_t)(s0 + lane) * n + j];
    }
}

}  // namespace

namespace {

int unit_blocks(const OptDev &O) {
    const long long n = O.units ? O.n_units : (long long)O.n_scen * O.n_spots;
    return (int)((n * 64 + kOptThreads - 1) / kOptThreads);
}

}  // namespace

hipError_t opt_build_count(const OptDev &O, unsigned long long *cnt, unsigned *err, hipStream_t st) {
    if (unit_blocks(O) == 0) return hipSuccess;
    hipLaunchKernelGGL(opt_count_kernel, dim3(unit_blocks(O)), dim3(kOptThreads), 0, st, O, cnt, err);
    return hipGetLastError();
}

hipError_t opt_structures(const uint8_t *roi, int nvox, OptMask *mask, unsigned long long *cnt,
                          unsigned long long *off, uint8_t *keep, uint8_t *sroi, hipStream_t st) {
    const unsigned blocks = (unsigned)(((long long)nvox + 4095) / 4096);
    hipLaunchKernelGGL(opt_mask_kernel, dim3(blocks), dim3(kOptThreads), 0, st, roi, nvox, mask, cnt, keep);
    hipLaunchKernelGGL(opt_scan_kernel, dim3(1), dim3(kUpdThreads), 0, st, cnt, off, (size_t)blocks);
    hipLaunchKernelGGL(opt_rank_kernel, dim3(blocks), dim3(kOptThreads), 0, st, roi, nvox, mask, off, sroi);
    return hipGetLastError();
}

hipError_t opt_roi_same(const uint8_t *a, const uint8_t *b, int nvox, unsigned *err, hipStream_t st) {
    const unsigned blocks = (unsigned)std::min<long long>(((long long)nvox + kOptThreads - 1) / kOptThreads, 4096);
    hipLaunchKernelGGL(opt_roi_same_kernel, dim3(blocks), dim3(kOptThreads), 0, st, a, b, nvox, err);
    return hipGetLastError();
}

hipError_t opt_roi_count(const OptDev &O, const OptMask *mask, unsigned *rcnt, unsigned *err, hipStream_t st) {
    hipLaunchKernelGGL(opt_roi_count_kernel, dim3((unsigned)std::min(O.n_scen * O.n_spots, 1 << 20)), dim3(kRoiThreads), 0, st, O, mask,
                       rcnt, err);
    return hipGetLastError();
}

hipError_t opt_roi_copy(const OptDev &O, const OptMask *mask, const unsigned *rcnt, const long long *rptr,
                        int32_t *ccol, float *cval, hipStream_t st) {
    hipLaunchKernelGGL(opt_roi_copy_kernel, dim3((unsigned)std::min(O.n_scen * O.n_spots, 1 << 20)), dim3(kRoiThreads), 0, st, O, mask,
                       rcnt, rptr, ccol, cval);
    return hipGetLastError();
}

hipError_t opt_build_scan(unsigned long long *cnt, unsigned long long *off, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(opt_scan_kernel, dim3(1), dim3(kUpdThreads), 0, st, cnt, off, n);
    return hipGetLastError();
}

hipError_t opt_build_emit(const OptDev &O, const unsigned long long *off, unsigned long long *cur, uint32_t *bkey,
                          float *bval, hipStream_t st) {
    if (unit_blocks(O) == 0) return hipSuccess;
    hipLaunchKernelGGL(opt_emit_kernel, dim3(unit_blocks(O)), dim3(kOptThreads), 0, st, O, off, cur, bkey, bval);
    return hipGetLastError();
}

hipError_t opt_forward(const OptDev &O, const double *w, int mode, float *dose_out, hipStream_t st) {
    if (O.n_work == 0) return hipSuccess;
    hipLaunchKernelGGL(opt_forward_kernel, dim3((unsigned)O.n_work), dim3(kFwdThreads), 0, st, O, w, mode, dose_out);
    return hipGetLastError();
}

hipError_t opt_gradient(const OptDev &O, hipStream_t st) {
    if (O.n_pieces == 0) return hipSuccess;
    const long long blocks = (O.n_pieces * 64 + kOptThreads - 1) / kOptThreads;
    hipLaunchKernelGGL(opt_grad_kernel, dim3((unsigned)blocks), dim3(kOptThreads), 0, st, O);
    return hipGetLastError();
}

hipError_t opt_update(const OptDev &O, int mode, double beta, int it, double *hist, hipStream_t st) {
    const int blocks = mode == kOptFinal ? 1 : O.n_part + (mode == kOptFista ? 1 : 0);
    hipLaunchKernelGGL(opt_update_kernel, dim3(blocks), dim3(kOptThreads), 0, st, O, mode, beta, it, hist);
    return hipGetLastError();
}

}  // namespace vpmc
