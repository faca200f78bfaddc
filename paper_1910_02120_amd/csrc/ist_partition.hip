// Partition and merge kernels: neuron index tables, block gather/scatter.
//
// Section 2.1 "Constructing Subnets" / Appendix A of the IST paper: subnet s owns
// the block H_l^s of each hidden layer and gets W_l[H_l^s, H_{l-1}^s].  Inside a
// subnet the order of neurons does not change the function it computes, so the
// packed layout keeps each block sorted by neuron id: gathers then walk the full
// matrix in ascending address order.  ist_subnet_export undoes the sort.
#include "ist_internal.h"

namespace ist {

// 16-byte load of data that is read exactly once (a row of the full matrix on its way into the
// subnets): non-temporal, measured 6.3 .. 6.9 TB/s against 5.7 .. 6.2 TB/s for plain loads
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 ld_stream(const uint4 *p)
{
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return uint4{v.x, v.y, v.z, v.w};
}

// ----------------------------------------------------------------------------
// index tables
// ----------------------------------------------------------------------------
// All tables of up to kMaxPermJobs hidden layers in one launch, a workgroup per (layer, subnet).  The subnet's neuron ids
// are set as bits of an LDS mask; the packed position of an id is then the number of bits below it: bits of earlier words
// (prefix sums) plus bits of its own.  Ids are taken in windows of kPermWindow, so that any width fits.  (Measured against
// an inverse permutation followed by a compaction, two launches: three layers of 65536 neurons, 8 subnets, 50 -> 17 us;
// two layers of 128 neurons 9.3 -> 4.0 us.)
constexpr int kPermThreads = 1024, kPermWindow = 262144, kPermWords = kPermWindow / 32;
__global__ __launch_bounds__(kPermThreads) void k_perm_tables(PermJobs jobs, int32_t *err)
{
    __shared__ uint32_t bits[kPermWords];
    __shared__ int32_t before[kPermWords];
    __shared__ int32_t wave_sum[kPermThreads / 64];
    const PermJob &job = jobs.job[blockIdx.y];
    const int32_t *__restrict__ perm = job.perm;
    const int32_t S = jobs.S, s = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // subnet s owns the permutation positions [p_lo, p_hi): N = q S + r, the first r blocks one wider; its packed positions
    // are s * w + 0 .. w - 1, those beyond its own width hold no neuron
    const int64_t N = job.N, w = job.w, words = (N + 31) / 32;
    const int64_t qn = N / S, rn = N % S;
    const int64_t ws = qn + (s < rn ? 1 : 0);
    const int64_t p_lo = (int64_t)s * qn + (s < rn ? s : rn), p_hi = p_lo + ws, pack0 = (int64_t)s * w;
    for (int64_t q = ws + threadIdx.x; q < w; q += kPermThreads) job.sorted[pack0 + q] = -1;
    int base = 0;   // members below the window
    for (int64_t w0 = 0; w0 < words; w0 += kPermWords) {
        const int nw = (int)(words - w0 < kPermWords ? words - w0 : kPermWords);
        for (int i = threadIdx.x; i < nw; i += kPermThreads) bits[i] = 0u;
        __syncthreads();
        for (int64_t p = p_lo + threadIdx.x; p < p_hi; p += kPermThreads) {
            const int64_t c = perm[p];
            if (c < 0 || c >= N) { if (w0 == 0) atomicOr(err, 1); continue; }
            const int64_t i = (c >> 5) - w0;
            if (i >= 0 && i < nw) atomicOr(&bits[i], 1u << (c & 31));
        }
        __syncthreads();
        // prefix sums: a thread owns `per` consecutive words
        const int per = (nw + kPermThreads - 1) / kPermThreads, i0 = (int)threadIdx.x * per;
        int own = 0;
        for (int i = i0; i < i0 + per && i < nw; ++i) own += __popc(bits[i]);
        int scan = own;
#pragma unroll
        for (int o = 1; o < 64; o *= 2) {
            const int v = __shfl_up(scan, o);
            if (lane >= o) scan += v;
        }
        if (lane == 63) wave_sum[wave] = scan;
        __syncthreads();
        int run = base + scan - own, total = 0;
        for (int i = 0; i < kPermThreads / 64; ++i) {
            run += i < wave ? wave_sum[i] : 0;
            total += wave_sum[i];
        }
        for (int i = i0; i < i0 + per && i < nw; ++i) { before[i] = run; run += __popc(bits[i]); }
        __syncthreads();
        for (int i = threadIdx.x; i < nw; i += kPermThreads) {
            job.mask[(int64_t)s * words + w0 + i] = bits[i];
            job.rank[(int64_t)s * words + w0 + i] = before[i];
        }
        for (int64_t p = p_lo + threadIdx.x; p < p_hi; p += kPermThreads) {
            const int64_t c = perm[p];
            const int64_t i = (c >> 5) - w0;
            if (c < 0 || c >= N || i < 0 || i >= nw) continue;
            const int64_t q = before[i] + __popc(bits[i] & ((1u << (c & 31)) - 1u));
            if (q < ws) {   // always true: at most ws ids were set
                const int32_t P = (int32_t)(pack0 + q);
                job.sorted[P] = (int32_t)c;
                job.slot[c] = P;
                job.p2q[p] = P;
            }
        }
        base += total;
        __syncthreads();
    }
}

hipError_t launch_perm_tables(const PermJobs &jobs, int32_t *err, hipStream_t st)
{
    if (jobs.njobs < 1 || jobs.njobs > kMaxPermJobs) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_perm_tables, dim3((unsigned)jobs.S, (unsigned)jobs.njobs), dim3(kPermThreads), 0, st, jobs, err);
    return hipGetLastError();
}

// checked mode: the inverse permutation, and whether it is one
__global__ void k_perm_invert(const int32_t *__restrict__ perm, int32_t *__restrict__ invpos, int64_t N)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int32_t c = perm[p];
    if (c >= 0 && c < N) invpos[c] = (int32_t)p;
}

__global__ void k_perm_check(const int32_t *__restrict__ perm, const int32_t *__restrict__ invpos,
                             int64_t N, int32_t *err)
{
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    int32_t p = invpos[c];
    if (p < 0 || p >= N || perm[p] != (int32_t)c) atomicOr(err, 2);
}

hipError_t launch_perm_check(const int32_t *perm, int32_t *invpos, int64_t N, int32_t *err, hipStream_t st)
{
    const dim3 grid((unsigned)((N + 255) / 256));
    hipLaunchKernelGGL(k_perm_invert, grid, dim3(256), 0, st, perm, invpos, N);
    hipLaunchKernelGGL(k_perm_check, grid, dim3(256), 0, st, perm, invpos, N, err);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// first layer of sparse inputs
// ----------------------------------------------------------------------------
// Transposed first layer for sparse inputs: sub[g][c][q] <-> W[rows[g*nr+q]][c].
// 64x64 tiles staged through LDS so both sides move along their contiguous axis.
template <typename E, bool SCATTER>
__global__ __launch_bounds__(256) void k_rows_transposed(E *__restrict__ W, int64_t ld,
                                                         E *__restrict__ sub,
                                                         const int32_t *__restrict__ rows,
                                                         int64_t nr, int64_t nc)
{
    __shared__ E tile[64][65];
    const int g = blockIdx.z;
    const int64_t q0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 64 x 4
    E *pack = sub + (int64_t)g * nr * nc;                     // [nc][nr]
    if (!SCATTER) {
        for (int i = ty; i < 64; i += 4) {
            int64_t q = q0 + i, c = c0 + tx;
            if (q < nr && c < nc) {
                const int64_t r = rows[g * nr + q];   // -1: a packed position without a neuron
                tile[i][tx] = r >= 0 ? W[r * ld + c] : E(0);
            }
        }
        __syncthreads();
        for (int i = ty; i < 64; i += 4) {
            int64_t c = c0 + i, q = q0 + tx;
            if (q < nr && c < nc) pack[c * nr + q] = tile[tx][i];
        }
    } else {
        for (int i = ty; i < 64; i += 4) {
            int64_t c = c0 + i, q = q0 + tx;
            if (q < nr && c < nc) tile[tx][i] = pack[c * nr + q];
        }
        __syncthreads();
        for (int i = ty; i < 64; i += 4) {
            int64_t q = q0 + i, c = c0 + tx;
            if (q < nr && c < nc) {
                const int64_t r = rows[g * nr + q];
                if (r >= 0) W[r * ld + c] = tile[i][tx];
            }
        }
    }
}

// The same for 2-byte elements with wider accesses: a tile of 64 rows x 128 columns; the packed
// side moves 16 bytes per lane (8 consecutive q of one column), the full matrix 4 bytes per lane.
// A row of W starts at an arbitrary element (odd row lengths), so a row's aligned 4-byte words are
// staged in LDS with the row's one-element misalignment kept, and the transposing side reads
// column c of row q at position mis_q + c.  Words that straddle the tile's column range are
// written element by element on merge (their other half belongs to a neighbour).
constexpr int kTrQ = 64, kTrC = 128;
template <bool SCATTER>
__global__ __launch_bounds__(256) void k_rows_transposed16(uint16_t *__restrict__ W, int64_t ld,
                                                           uint16_t *__restrict__ sub, const int32_t *__restrict__ rows,
                                                           int64_t nr, int64_t nc, int64_t ncx, int64_t nqy, int32_t G)
{
    __shared__ uint32_t tile[kTrQ][kTrC / 2 + 2];
    __shared__ int64_t start[kTrQ];                         // element index of (row, c0) in W
    // Tiles are numbered column tile fastest, then row tile, then subnet (ncx * nqy * G of them), and the 8 XCDs
    // (workgroup index mod 8) each take one contiguous eighth of that list: a row piece of 256 bytes starts at an
    // arbitrary address, so the tiles left and right of a column boundary share a 128-byte line of every row, and as
    // neighbours on one XCD they meet it in the same L2 (the second fetch and the two partial writes of a merge stop
    // there) instead of each going to memory for it.  The grid holds 8 * ceil(tiles / 8) workgroups.
    const int64_t total = ncx * nqy * G, chunk = (total + 7) >> 3;
    const int64_t L = (int64_t)(blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
    if (L >= total) return;                                 // (whole workgroups, before any barrier)
    const int64_t cx = L % ncx, rest = L / ncx;
    const int g = (int)(rest / nqy);
    const int64_t q0 = (rest % nqy) * kTrQ, c0 = cx * kTrC;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    uint16_t *pack = sub + (int64_t)g * nr * nc;            // [nc][nr]
    uint32_t *W32 = reinterpret_cast<uint32_t *>(W);
    if (threadIdx.x < kTrQ) {
        const int64_t q = q0 + threadIdx.x;
        const int64_t r = q < nr ? rows[g * nr + q] : -1;
        start[threadIdx.x] = r >= 0 ? r * ld + c0 : -2;     // (even: such a position's row of the tile has no misalignment)
    }
    __syncthreads();
    const int64_t ncol = nc - c0 < kTrC ? nc - c0 : kTrC;   // valid columns of this tile
    // ---- packed side <-> LDS: thread (crow, lq) owns 8 consecutive q of one column ----
    auto packed_side = [&]() {
        const int lq = threadIdx.x & 7;
#pragma unroll
        for (int pass = 0; pass < kTrC / 32; ++pass) {
            const int crow = (threadIdx.x >> 3) + 32 * pass;
            if (crow >= ncol) continue;
            uint16_t *dst = pack + (c0 + crow) * nr + q0 + lq * 8;
            const bool full = q0 + lq * 8 + 8 <= nr;
            if (SCATTER) {
                uint16_t v[8];
                if (full) __builtin_memcpy(v, __builtin_assume_aligned(dst, 16), 16);
                else
                    for (int j = 0; j < 8; ++j) v[j] = q0 + lq * 8 + j < nr ? dst[j] : (uint16_t)0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int qi = lq * 8 + j;
                    reinterpret_cast<uint16_t *>(tile[qi])[(start[qi] & 1) + crow] = v[j];
                }
            } else {
                uint16_t v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int qi = lq * 8 + j;
                    v[j] = reinterpret_cast<const uint16_t *>(tile[qi])[(start[qi] & 1) + crow];
                }
                if (full) __builtin_memcpy(__builtin_assume_aligned(dst, 16), v, 16);
                else
                    for (int j = 0; j < 8; ++j)
                        if (q0 + lq * 8 + j < nr) dst[j] = v[j];
            }
        }
    };
    if (SCATTER) { packed_side(); __syncthreads(); }
    if (!SCATTER) {
        // all 16 row passes' words are requested before any is stored to LDS; a word outside the
        // tile's columns is read from word 0 of W instead (no branch around the loads)
        uint32_t v[kTrQ / 4];
#pragma unroll
        for (int pass = 0; pass < kTrQ / 4; ++pass) {
            const int64_t e0 = start[pass * 4 + ty];
            const int mis = (int)(e0 & 1);
            const int64_t lo = 2 * tx - mis;
            const int64_t e = e0 + lo;                      // first element of the word
            const bool ok = e0 >= 0 && lo < ncol;           // (W holds an even number of elements: it ends on a word)
            v[pass] = W32[ok ? (e >> 1) : 0];
        }
#pragma unroll
        for (int pass = 0; pass < kTrQ / 4; ++pass)         // a packed position without a neuron (start < 0) is zeros
            tile[pass * 4 + ty][tx] = start[pass * 4 + ty] >= 0 ? v[pass] : 0u;
        // the 65th word of a misaligned row
        for (int i = threadIdx.x; i < kTrQ; i += 256) {
            const int64_t e0 = start[i];
            if (e0 >= 0 && (e0 & 1) && kTrC - 1 < ncol) tile[i][kTrC / 2] = W32[(e0 + kTrC - 1) >> 1];
        }
        __syncthreads();
        packed_side();
        return;
    }
    // ---- merge: LDS -> full matrix, 4 rows per pass, one aligned word per lane (+1 spill word) ----
#pragma unroll
    for (int pass = 0; pass < kTrQ / 4; ++pass) {
        const int qi = pass * 4 + ty;
        const int64_t e0 = start[qi];
        if (e0 < 0) continue;
        const int mis = (int)(e0 & 1);
        const int64_t w0 = (e0 - mis) >> 1;                 // first word of the staged range
        for (int k = tx; k < kTrC / 2 + 1; k += 64) {       // second trip: only lane 0 (word 64)
            const int64_t lo = 2 * k - mis, hi = lo + 1;    // tile columns held by word k
            if (hi < 0 || lo >= ncol) continue;
            const bool whole = lo >= 0 && hi < ncol;
            if (whole) {
                W32[w0 + k] = tile[qi][k];
            } else {
                const uint16_t *t16 = reinterpret_cast<const uint16_t *>(tile[qi]);
                if (lo >= 0 && lo < ncol) W[e0 + lo] = t16[2 * k];
                if (hi >= 0 && hi < ncol) W[e0 + hi] = t16[2 * k + 1];
            }
        }
    }
}

// ----------------------------------------------------------------------------
// column-partitioned blocks (middle and last layers)
// ----------------------------------------------------------------------------
// Middle layers (rows and columns both partitioned), LDS-staged: one workgroup per packed
// row walks the source row in chunks of kMidChunk elements.  A chunk is read (and, for
// merge, written back) with 16-byte accesses along its memory order; the kept elements of
// the chunk are the contiguous range [rank(c0), rank(c0 + chunk)) of the packed row (the
// column list is ascending), so the packed side is read/written contiguously as well and
// the permutation happens in LDS.  HBM sees whole lines once in each direction.
constexpr int kMidChunk = 8192;
template <bool SCATTER>
__global__ __launch_bounds__(256) void k_mid_lds(uint16_t *__restrict__ W, int64_t ld, uint16_t *__restrict__ sub,
                                                 const int32_t *__restrict__ slotr,
                                                 const int32_t *__restrict__ cols,
                                                 const int32_t *__restrict__ rank, int64_t words, int64_t nr,
                                                 int64_t nc, int64_t N_in, int32_t G)
{
    using E = uint16_t;
    constexpr int EPC = 16 / sizeof(E);
    constexpr int PER = kMidChunk / EPC / 256;   // 16-byte pieces per thread and chunk
    __shared__ __attribute__((aligned(16))) E buf[kMidChunk];
    // workgroups follow the rows of the full matrix, so the rows in flight are neighbours
    const int64_t P = slotr[blockIdx.x];
    if (P < 0 || P >= nr * G) return;   // only with tables built from a non-permutation
    const int g = (int)(P / nr);
    uint4 *full = reinterpret_cast<uint4 *>(W + (int64_t)blockIdx.x * ld);
    E *pack = sub + P * nc;
    const int32_t *cg = cols + (int64_t)g * nc;
    const int32_t *rg = rank + (int64_t)g * words;
    const int64_t row_pieces = N_in / EPC;
    uint4 nxt[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t c = threadIdx.x + 256 * u;
        nxt[u] = c < row_pieces ? (SCATTER ? full[c] : ld_stream(full + c)) : uint4{0, 0, 0, 0};
    }
    for (int64_t c0 = 0; c0 < N_in; c0 += kMidChunk) {
        const int64_t cend = c0 + kMidChunk < N_in ? c0 + kMidChunk : N_in;
        int64_t qlo = rg[c0 >> 5];
        int64_t qhi = cend < N_in ? rg[cend >> 5] : nc;
        qlo = qlo < 0 ? 0 : (qlo > nc ? nc : qlo);
        qhi = qhi < qlo ? qlo : (qhi > nc ? nc : qhi);
#pragma unroll
        for (int u = 0; u < PER; ++u) reinterpret_cast<uint4 *>(buf)[threadIdx.x + 256 * u] = nxt[u];
        __syncthreads();
        // the next chunk's loads fly while this one is permuted
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t c = (c0 + kMidChunk) / EPC + threadIdx.x + 256 * u;
            nxt[u] = c < row_pieces ? (SCATTER ? full[c] : ld_stream(full + c)) : uint4{0, 0, 0, 0};
        }
        for (int64_t q = qlo + threadIdx.x; q < qhi; q += 256) {
            const int64_t off = (int64_t)cg[q] - c0;
            if (off >= 0 && off < cend - c0) {   // always true for tables built from a permutation
                if (SCATTER) buf[off] = pack[q]; else pack[q] = buf[off];
            }
        }
        __syncthreads();
        if (SCATTER) {
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int64_t c = c0 / EPC + threadIdx.x + 256 * u;
                if (c < row_pieces) full[c] = reinterpret_cast<const uint4 *>(buf)[threadIdx.x + 256 * u];
            }
            __syncthreads();
        }
    }
}

// Last layer (every row belongs to all subnets, columns partitioned): one workgroup
// per row stages the row in LDS, so that the row is read/written along its memory
// order and every packed block row is written/read as 16-byte pieces; the column
// permutation happens inside LDS (a packed position without a column, -1, reads as zero and is skipped on the way back).
// VEC: the row of the full matrix moves in 16-byte pieces as well.
template <typename E, bool SCATTER, bool VEC>
__global__ __launch_bounds__(256) void k_last_lds(E *__restrict__ W, int64_t ld, E *__restrict__ sub,
                                                  const int32_t *__restrict__ sorted, int64_t nr,
                                                  int64_t nc, int32_t G)
{
    constexpr int EPC = 16 / sizeof(E);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    E *row = reinterpret_cast<E *>(lds_raw);
    const int64_t i = blockIdx.x;
    E *const full = W + i * ld;
    const int64_t nunit = (int64_t)G * nc / EPC;
    if (!SCATTER) {
        if (VEC) {
            for (int64_t c = threadIdx.x; c < ld / EPC; c += blockDim.x)
                reinterpret_cast<uint4 *>(row)[c] = ld_stream(reinterpret_cast<const uint4 *>(full) + c);
        } else {
            for (int64_t c = threadIdx.x; c < ld; c += blockDim.x) row[c] = full[c];
        }
        __syncthreads();
        for (int64_t u = threadIdx.x; u < nunit; u += blockDim.x) {
            const int64_t P0 = u * EPC;
            const int64_t g = P0 / nc, q0 = P0 % nc;
            E e[EPC];
#pragma unroll
            for (int j = 0; j < EPC; ++j) {
                const int32_t c = sorted[P0 + j];     // (no branch around the LDS access)
                const E v = row[c >= 0 ? c : 0];
                e[j] = c >= 0 ? v : E(0);
            }
            uint4 o;
            __builtin_memcpy(&o, e, 16);
            *reinterpret_cast<uint4 *>(sub + ((int64_t)g * nr + i) * nc + q0) = o;
        }
    } else {
        for (int64_t u = threadIdx.x; u < nunit; u += blockDim.x) {
            const int64_t P0 = u * EPC;
            const int64_t g = P0 / nc, q0 = P0 % nc;
            uint4 o = *reinterpret_cast<const uint4 *>(sub + ((int64_t)g * nr + i) * nc + q0);
            E e[EPC];
            __builtin_memcpy(e, &o, 16);
#pragma unroll
            for (int j = 0; j < EPC; ++j) {
                const int32_t c = sorted[P0 + j];
                row[c >= 0 ? c : ld] = e[j];          // (one spare element behind the row takes what is skipped)
            }
        }
        __syncthreads();
        if (VEC) {
            for (int64_t c = threadIdx.x; c < ld / EPC; c += blockDim.x)
                reinterpret_cast<uint4 *>(full)[c] = reinterpret_cast<const uint4 *>(row)[c];
        } else {
            for (int64_t c = threadIdx.x; c < ld; c += blockDim.x) full[c] = row[c];
        }
    }
}

// bytes any kernel has to move at cache-line granularity: the rows a block touches are read whole, and rewritten whole on
// merge when their columns are partitioned
static double line_bytes(const CopyArgs &a, bool merge)
{
    const double sub_b = (double)a.G * a.nr * a.nc * a.esz;
    const double rows_b = (a.rows ? (double)a.G * a.nr : (double)a.N_out) * a.N_in * a.esz;
    return !a.cols ? 2.0 * sub_b : (merge && a.rows ? 2.0 * rows_b + sub_b : rows_b + sub_b);
}

static bool copy_aligned(const CopyArgs &a)
{
    const int64_t epc = 16 / a.esz;
    return reinterpret_cast<uintptr_t>(a.W) % 16 == 0 && reinterpret_cast<uintptr_t>(a.sub) % 16 == 0 && a.ld % epc == 0 &&
           a.N_in % epc == 0;
}

// Layers that get a launch of their own; all others share one launch per phase (k_row_jobs).
//   transposed first layer: always.
//   middle layer: bf16 from 64 MiB on (8192 x 8192, 8 subnets, partition / merge 25 / 52 us alone, 31 / 62 us shared; wide
//   stress network 1.85 / 3.58 ms per layer alone, 2.5 / 4.7 ms shared).  f32 layers share a launch at every size: 4-byte
//   accesses keep up with the memory (8192 x 8192, 8 subnets, partition / merge / re-sampling with everything else of the
//   phase 66 / 110 / 147 us against 83 / 120 / 176 us; 16384 x 16384 257 / 441 / 530 against 260 / 493 / 595 us).
//   last layer: from 4096 rows on (8000 x 1024 bf16 21 / 17 us alone, 24 / 25 us shared; 400,000 x 256 f32 154 / 169 us alone,
//   810 / 1323 us shared: a workgroup per short row); below, a launch costs more than the better kernel gains.
static bool copy_alone(const CopyArgs &a)
{
    if (a.transposed) return true;
    if (!a.cols) return false;
    const int64_t all_rows = a.nr * a.G;
    if (a.rows)
        return copy_aligned(a) && a.esz == 2 && (double)a.N_out * a.N_in * a.esz >= 64.0 * (1 << 20) && a.N_in == a.ld && a.N_in % 32 == 0 &&
               all_rows == a.N_out && a.nc * a.G == a.N_in && all_rows < 0x7fffffffLL;
    return a.nr >= 4096 && reinterpret_cast<uintptr_t>(a.sub) % 16 == 0 && a.N_in == a.ld && a.N_in * a.esz < 65536 &&
           a.nr < 0x7fffffffLL;   // (packed rows are whole 16-byte pieces)
}

template <typename E, bool SCATTER>
static hipError_t copy_typed(const CopyArgs &a, hipStream_t st)
{
    E *W = static_cast<E *>(a.W);
    E *sub = static_cast<E *>(a.sub);
    const double line_b = line_bytes(a, SCATTER);
    if (a.transposed) {
        tag_kernel(SCATTER ? "k_rows_transposed<scatter>" : "k_rows_transposed<gather>", 0.0, line_b);
        if (sizeof(E) == 2 && reinterpret_cast<uintptr_t>(W) % 4 == 0 && reinterpret_cast<uintptr_t>(sub) % 16 == 0 &&
            a.nr % 8 == 0 && ((int64_t)a.nr * a.nc) % 8 == 0 && a.N_out * a.N_in % 2 == 0) {
            const int64_t ncx = (a.nc + kTrC - 1) / kTrC, nqy = (a.nr + kTrQ - 1) / kTrQ;
            const int64_t wgs = 8 * ((ncx * nqy * a.G + 7) / 8);
            if (wgs < 0x7fffffffLL) {
                hipLaunchKernelGGL((k_rows_transposed16<SCATTER>), dim3((unsigned)wgs), dim3(256), 0, st,
                                   reinterpret_cast<uint16_t *>(W), a.ld, reinterpret_cast<uint16_t *>(sub), a.rows, a.nr, a.nc,
                                   ncx, nqy, a.G);
                return hipGetLastError();
            }
        }
        dim3 grid((unsigned)((a.nc + 63) / 64), (unsigned)((a.nr + 63) / 64), (unsigned)a.G);
        hipLaunchKernelGGL((k_rows_transposed<E, SCATTER>), grid, dim3(256), 0, st, W, a.ld, sub,
                           a.rows, a.nr, a.nc);
    } else if (a.rows) {
        tag_kernel(SCATTER ? "k_mid_lds<scatter>" : "k_mid_lds<gather>", 0.0, line_b);
        if constexpr (sizeof(E) == 2)
            hipLaunchKernelGGL(k_mid_lds<SCATTER>, dim3((unsigned)(a.nr * a.G)), dim3(256), 0, st, W, a.ld, sub, a.slotr,
                               a.cols, a.rankc, a.wordsc, a.nr, a.nc, a.N_in, a.G);
    } else {   // the last layer's columns cover 0 .. N_in - 1 exactly once over the G subnets
        int th = (int)(a.N_in * a.esz / 16);
        th = th < 64 ? 64 : (th > 256 ? 256 : (th + 63) / 64 * 64);
        tag_kernel(SCATTER ? "k_last_lds<scatter>" : "k_last_lds<gather>", 0.0, line_b);
        const size_t lds = (size_t)(a.N_in * (int64_t)sizeof(E) / 16 * 16 + 16);   // the row and a spare element
        if (copy_aligned(a))
            hipLaunchKernelGGL((k_last_lds<E, SCATTER, true>), dim3((unsigned)a.nr), dim3(th), lds, st, W, a.ld, sub, a.cols,
                               a.nr, a.nc, a.G);
        else
            hipLaunchKernelGGL((k_last_lds<E, SCATTER, false>), dim3((unsigned)a.nr), dim3(th), lds, st, W, a.ld, sub, a.cols,
                               a.nr, a.nc, a.G);
    }
    return hipGetLastError();
}

hipError_t launch_partition_copy(const CopyArgs &a, hipStream_t st)
{
    return a.esz == 2 ? copy_typed<uint16_t, false>(a, st) : copy_typed<uint32_t, false>(a, st);
}
hipError_t launch_merge_copy(const CopyArgs &a, hipStream_t st)
{
    return a.esz == 2 ? copy_typed<uint16_t, true>(a, st) : copy_typed<uint32_t, true>(a, st);
}

// ----------------------------------------------------------------------------
// re-sampling between rounds: merge of the old partition and partition by the new permutation in
// one pass over the full matrix (the row that merge writes is the row partition would read back)
// ----------------------------------------------------------------------------
// large bf16 middle layers: k_mid_lds with both directions on the staged chunk
__global__ __launch_bounds__(256) void k_resample_mid(uint16_t *__restrict__ W, int64_t ld, const uint16_t *__restrict__ sub_old,
                                                      uint16_t *__restrict__ sub_new, const int32_t *__restrict__ slotr_old,
                                                      const int32_t *__restrict__ slotr_new,
                                                      const int32_t *__restrict__ cols_old,
                                                      const int32_t *__restrict__ cols_new,
                                                      const int32_t *__restrict__ rank_old,
                                                      const int32_t *__restrict__ rank_new, int64_t words, int64_t nr,
                                                      int64_t nc, int64_t N_in, int32_t G)
{
    using E = uint16_t;
    constexpr int EPC = 16 / sizeof(E);
    constexpr int PER = kMidChunk / EPC / 256;
    __shared__ __attribute__((aligned(16))) E buf[kMidChunk];
    const int64_t Po = slotr_old[blockIdx.x], Pn = slotr_new[blockIdx.x];
    if (Po < 0 || Po >= nr * G || Pn < 0 || Pn >= nr * G) return;
    const int go = (int)(Po / nr), gn = (int)(Pn / nr);
    uint4 *full = reinterpret_cast<uint4 *>(W + (int64_t)blockIdx.x * ld);
    const E *pack_old = sub_old + Po * nc;
    E *pack_new = sub_new + Pn * nc;
    const int32_t *co = cols_old + (int64_t)go * nc, *cn = cols_new + (int64_t)gn * nc;
    const int32_t *ro = rank_old + (int64_t)go * words, *rn = rank_new + (int64_t)gn * words;
    const int64_t row_pieces = N_in / EPC;
    auto clampq = [&](int64_t q) { return q < 0 ? (int64_t)0 : (q > nc ? nc : q); };
    uint4 nxt[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t c = threadIdx.x + 256 * u;
        nxt[u] = c < row_pieces ? full[c] : uint4{0, 0, 0, 0};
    }
    for (int64_t c0 = 0; c0 < N_in; c0 += kMidChunk) {
        const int64_t cend = c0 + kMidChunk < N_in ? c0 + kMidChunk : N_in;
        const int64_t qlo_o = clampq(ro[c0 >> 5]), qhi_o = cend < N_in ? clampq(ro[cend >> 5]) : nc;
        const int64_t qlo_n = clampq(rn[c0 >> 5]), qhi_n = cend < N_in ? clampq(rn[cend >> 5]) : nc;
#pragma unroll
        for (int u = 0; u < PER; ++u) reinterpret_cast<uint4 *>(buf)[threadIdx.x + 256 * u] = nxt[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t c = (c0 + kMidChunk) / EPC + threadIdx.x + 256 * u;
            nxt[u] = c < row_pieces ? full[c] : uint4{0, 0, 0, 0};
        }
        for (int64_t q = qlo_o + threadIdx.x; q < qhi_o; q += 256) {
            const int64_t off = (int64_t)co[q] - c0;
            if (off >= 0 && off < cend - c0) buf[off] = pack_old[q];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t c = c0 / EPC + threadIdx.x + 256 * u;
            if (c < row_pieces) full[c] = reinterpret_cast<const uint4 *>(buf)[threadIdx.x + 256 * u];
        }
        for (int64_t q = qlo_n + threadIdx.x; q < qhi_n; q += 256) {
            const int64_t off = (int64_t)cn[q] - c0;
            if (off >= 0 && off < cend - c0) pack_new[q] = buf[off];
        }
        __syncthreads();
    }
}

// Fused merge(old) + partition(new) of a layer with a launch of its own; *fused = false when there is none and the caller
// has to run the two copies one after the other (the transposed first layer; the last layer, every line of which is owned:
// merge and partition each move it once already, and one workgroup touching the blocks of both buffers in all S subnets
// measured slower than the two passes).
hipError_t launch_resample_copy(const CopyArgs &o, const CopyArgs &n, bool *fused, hipStream_t st)
{
    *fused = !o.transposed && o.rows && o.cols && copy_aligned(o) && copy_aligned(n);
    if (!*fused) return hipSuccess;
    tag_kernel("k_resample_mid", 0.0, line_bytes(o, true) + (double)o.G * o.nr * o.nc * o.esz);
    hipLaunchKernelGGL(k_resample_mid, dim3((unsigned)(o.nr * o.G)), dim3(256), 0, st, static_cast<uint16_t *>(o.W), o.ld,
                       static_cast<const uint16_t *>(o.sub), static_cast<uint16_t *>(n.sub), o.slotr, n.slotr, o.cols, n.cols,
                       o.rankc, n.rankc, o.wordsc, o.nr, o.nc, o.N_in, o.G);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// every other layer and all biases of a phase in one launch
// ----------------------------------------------------------------------------
// Sum of up to 64 values as a balanced pairwise tree over the index (neighbours first, then pairs
// of pairs, ...); missing leaves are +0, which leaves every partial sum unchanged.
template <typename F>
__device__ inline float tree_sum64(int count, F value)
{
    float v[64];
#pragma unroll
    for (int s = 0; s < 64; ++s) v[s] = s < count ? value(s) : 0.0f;
#pragma unroll
    for (int d = 1; d < 64; d *= 2)
#pragma unroll
        for (int s = 0; s + d < 64; s += 2 * d) v[s] = v[s] + v[s + d];
    return v[0];
}

// (pairwise-tree sum over the G subnet copies) * (1/G).  With G a power of two and identical copies every step is
// exact: merging an untrained partition returns the bias bit for bit.  Two tree levels of 64 cover G <= 4096.
template <typename D>
__device__ inline typename D::T bias_mean(const typename D::T *sub, int64_t n, int64_t i, int32_t G)
{
    float acc;
    if (G <= 8) {   // the same tree, without its 56 zero leaves
        float v[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = s < G ? D::ld(sub + (int64_t)s * n + i) : 0.0f;
        acc = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    } else if (G <= 64) {
        acc = tree_sum64(G, [&](int s) { return D::ld(sub + (int64_t)s * n + i); });
    } else {
        const int chunks = (G + 63) / 64;
        acc = tree_sum64(chunks, [&](int c) {
            const int left = G - 64 * c;
            return tree_sum64(left < 64 ? left : 64, [&](int s) { return D::ld(sub + (int64_t)(64 * c + s) * n + i); });
        });
    }
    return D::cvt(acc * (1.0f / (float)G));
}

// i = lo + tid, lo + tid + nt, ... below hi, U of them at a time: all loads of a batch are issued before its first store
// (one after the other they would each wait out a trip to memory)
template <int U, typename V, typename Load, typename Store>
__device__ inline void batched(int64_t lo, int64_t hi, int tid, int nt, Load load, Store store)
{
    for (int64_t i = lo + tid; i < hi; i += (int64_t)U * nt) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * nt < hi) v[u] = load(i + u * nt);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * nt < hi) store(i + u * nt, v[u]);
    }
}

// Columns [c0, cend) of a row of the full matrix, in LDS, <-> the packed row of one subnet, whose kept elements of that range
// are the contiguous positions [rank(c0), rank(cend)) (a packed position without a column, cols = -1, reads as zero and is
// skipped on the way out; such positions come last).
template <typename E> struct ColVal { int32_t c; E v; };
template <typename E, bool TO_PACK>
__device__ inline void permute_range(E *buf, int64_t c0, int64_t cend, int64_t N_in, E *pack, const int32_t *cols,
                                     const int32_t *rank, int64_t nc, int tid, int nt)
{
    int64_t qlo = rank[c0 >> 5], qhi = cend < N_in ? rank[cend >> 5] : nc;
    qlo = qlo < 0 ? 0 : (qlo > nc ? nc : qlo);
    qhi = qhi < qlo ? qlo : (qhi > nc ? nc : qhi);
    batched<8, ColVal<E>>(qlo, qhi, tid, nt,
                          [&](int64_t q) { return ColVal<E>{cols[q], TO_PACK ? E(0) : pack[q]}; },
                          [&](int64_t q, ColVal<E> x) {
                              const bool in = x.c >= c0 && x.c < cend;   // false for an empty position (and for tables of a
                              if (TO_PACK) pack[q] = in ? buf[x.c - c0] : E(0);   // non-permutation)
                              else if (in) buf[x.c - c0] = x.v;
                          });
}

// MERGE: the old subnets' entries go into W; PART: the new subnets are cut from W (after the merge, when both).  A workgroup
// owns a row of W, or kRowChunk columns of it, from its first read to its last write, so a phase needs no order among
// workgroups.
//   whole rows (first layer): the packed row <-> the row of W, through registers when both;
//   middle and last layer: the columns pass through LDS - read unless every entry is overwritten (merge of the last layer),
//   patched by the old owner(s), written back, read by the new owner(s); in the last layer a wave per owner.
// Small layers are a chain of latencies, not of bytes: everything that does not depend on each other is requested together.
constexpr int kRowChunk = 4096;
template <typename D, bool MERGE, bool PART>
__global__ __launch_bounds__(256) void k_row_jobs(RowJobs a)
{
    using E = typename D::T;
    constexpr int EPC = 16 / sizeof(E);
    __shared__ __attribute__((aligned(16))) E buf[kRowChunk];
    int ji = 0;
    while (ji + 1 < a.njobs && (int)blockIdx.x >= a.job[ji + 1].blk0) ++ji;
    const RowJob j = a.job[ji];
    const int64_t b = (int)blockIdx.x - j.blk0;
    const int tid = threadIdx.x;
    E *W = static_cast<E *>(j.W);
    const E *so = static_cast<const E *>(j.sub_old);
    E *sn = static_cast<E *>(j.sub_new);
    if (j.kind == ROW_BIAS_HIDDEN) {   // 256 packed positions of the new (merge alone: of the old) subnets
        const int64_t P = b * 256 + tid;
        if (P >= j.nr * a.G) return;
        const int64_t r = (PART ? j.rows_new : j.rows_old)[P];
        if (r < 0) { if (PART) sn[P] = E(0); return; }
        E v;
        if (MERGE) { v = so[PART ? (int64_t)j.slot_old[r] : P]; W[r] = v; } else v = W[r];
        if (PART) sn[P] = v;
        return;
    }
    if (j.kind == ROW_BIAS_OUT) {      // mean of the copies; one copy for every subnet
        const int64_t i = b * 256 + tid;
        if (i >= j.N_out) return;
        if (MERGE) W[i] = bias_mean<D>(so, j.N_out, i, a.G);
        if (PART) {
            const E v = W[i];
            for (int g = 0; g < a.G; ++g) sn[(int64_t)g * j.N_out + i] = v;
        }
        return;
    }
    if (b >= (int64_t)j.N_out * j.chunks) {   // packed rows without a neuron (blocks of unequal width) are zeros
        if (!PART) return;
        const int64_t pads = j.nr * a.G - j.N_out, qn = j.N_out / a.G, rn = j.N_out % a.G;
        for (int64_t i = b - (int64_t)j.N_out * j.chunks; i < pads; i += j.pad_blocks) {
            const int64_t p0 = j.nr - qn - 1, p1 = j.nr - qn, wide = rn * p0;   // pads of a wider / narrower block
            const int64_t s = i < wide ? i / p0 : rn + (i - wide) / p1;
            const int64_t q = i < wide ? qn + 1 + i % p0 : qn + (i - wide) % p1;
            E *pack = sn + (s * j.nr + q) * j.nc;
            for (int64_t c = tid; c < j.nc; c += 256) pack[c] = E(0);
        }
        return;
    }
    const int64_t r = j.chunks == 1 ? b : b / j.chunks;   // row of W
    const int64_t all = j.nr * a.G;
    E *full = W + r * j.ld;
    int64_t Po = -1, Pn = -1;
    if (j.kind != ROW_LAST) {          // (a table of a non-permutation may name no valid position: nothing to do then)
        if (MERGE) { Po = j.slot_old[r]; if (Po < 0 || Po >= all) return; }
        if (PART) { Pn = j.slot_new[r]; if (Pn < 0 || Pn >= all) return; }
    }
    if (j.kind == ROW_WHOLE) {
        const E *src = MERGE ? so + Po * j.nc : full;
        E *dst = PART ? sn + Pn * j.nc : nullptr;
        if (j.vec)
            batched<4, uint4>(0, j.nc / EPC, tid, 256,
                              [&](int64_t c) { return ld_stream(reinterpret_cast<const uint4 *>(src) + c); },
                              [&](int64_t c, uint4 v) {
                                  if (MERGE) reinterpret_cast<uint4 *>(full)[c] = v;
                                  if (PART) reinterpret_cast<uint4 *>(dst)[c] = v;
                              });
        else
            batched<8, E>(0, j.nc, tid, 256, [&](int64_t c) { return src[c]; },
                          [&](int64_t c, E v) {
                              if (MERGE) full[c] = v;
                              if (PART) dst[c] = v;
                          });
        return;
    }
    const int64_t c0 = (b - r * j.chunks) * kRowChunk, cend = c0 + kRowChunk < j.N_in ? c0 + kRowChunk : j.N_in;
    uint4 *const full4 = reinterpret_cast<uint4 *>(full + c0), *const buf4 = reinterpret_cast<uint4 *>(buf);
    const int64_t n4 = (cend - c0) / EPC;
    if (!(MERGE && j.kind == ROW_LAST)) {
        if (j.vec) batched<4, uint4>(0, n4, tid, 256, [&](int64_t c) { return full4[c]; }, [&](int64_t c, uint4 v) { buf4[c] = v; });
        else batched<8, E>(c0, cend, tid, 256, [&](int64_t c) { return full[c]; }, [&](int64_t c, E v) { buf[c - c0] = v; });
        __syncthreads();
    }
    const int lane = tid & 63, wave = tid >> 6;
    if (MERGE) {
        if (j.kind == ROW_MIDDLE) {
            const int64_t g = Po / j.nr;
            permute_range<E, false>(buf, c0, cend, j.N_in, const_cast<E *>(so) + Po * j.nc, j.cols_old + g * j.nc,
                                    j.rank_old + g * j.words, j.nc, tid, 256);
        } else {
            for (int g = wave; g < a.G; g += 4)
                permute_range<E, false>(buf, c0, cend, j.N_in, const_cast<E *>(so) + ((int64_t)g * j.nr + r) * j.nc,
                                        j.cols_old + (int64_t)g * j.nc, j.rank_old + g * j.words, j.nc, lane, 64);
        }
        __syncthreads();
        if (j.vec) batched<4, uint4>(0, n4, tid, 256, [&](int64_t c) { return buf4[c]; }, [&](int64_t c, uint4 v) { full4[c] = v; });
        else batched<8, E>(c0, cend, tid, 256, [&](int64_t c) { return buf[c - c0]; }, [&](int64_t c, E v) { full[c] = v; });
    }
    if (PART) {
        if (j.kind == ROW_MIDDLE) {
            const int64_t g = Pn / j.nr;
            permute_range<E, true>(buf, c0, cend, j.N_in, sn + Pn * j.nc, j.cols_new + g * j.nc, j.rank_new + g * j.words,
                                   j.nc, tid, 256);
        } else {
            for (int g = wave; g < a.G; g += 4)
                permute_range<E, true>(buf, c0, cend, j.N_in, sn + ((int64_t)g * j.nr + r) * j.nc,
                                       j.cols_new + (int64_t)g * j.nc, j.rank_new + g * j.words, j.nc, lane, 64);
        }
    }
}

template <typename D>
static void launch_row_jobs_typed(const RowJobs &a, bool merge, bool part, dim3 grid, hipStream_t st)
{
    if (merge && part) hipLaunchKernelGGL((k_row_jobs<D, true, true>), grid, dim3(256), 0, st, a);
    else if (merge) hipLaunchKernelGGL((k_row_jobs<D, true, false>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_row_jobs<D, false, true>), grid, dim3(256), 0, st, a);
}

// o: the old subnets (merge), n: the new ones (partition), either may be null
bool copy_has_own_launch(const CopyArgs *o, const CopyArgs *n) { return copy_alone(o ? *o : *n); }

bool add_row_job(RowJobs &a, const CopyArgs *o, const CopyArgs *n)
{
    const CopyArgs &c = o ? *o : *n;
    if (a.njobs == kMaxRowJobs) return false;
    RowJob j{};
    j.kind = !c.cols ? ROW_WHOLE : (c.rows ? ROW_MIDDLE : ROW_LAST);
    j.W = c.W; j.ld = c.ld; j.nr = c.nr; j.nc = c.nc; j.N_out = c.N_out; j.N_in = c.N_in; j.words = c.wordsc;
    if (o) { j.sub_old = o->sub; j.slot_old = o->slotr; j.cols_old = o->cols; j.rank_old = o->rankc; }
    if (n) { j.sub_new = n->sub; j.slot_new = n->slotr; j.cols_new = n->cols; j.rank_new = n->rankc; }
    j.vec = copy_aligned(c) && (!o || copy_aligned(*o)) && (!n || copy_aligned(*n));
    const int64_t pads = n && c.rows ? c.nr * c.G - c.N_out : 0;
    j.pad_blocks = (int32_t)(pads < 1024 ? pads : 1024);
    j.chunks = j.kind == ROW_WHOLE ? 1 : (int32_t)((c.N_in + kRowChunk - 1) / kRowChunk);
    const int64_t blocks = a.blocks + c.N_out * j.chunks + j.pad_blocks;
    if (blocks > 0x7fffffffLL) return false;
    j.blk0 = (int32_t)a.blocks;
    a.blocks = blocks;
    a.bytes[j.kind] += o && n ? line_bytes(*o, true) + (double)c.G * c.nr * c.nc * c.esz : line_bytes(c, o != nullptr);
    a.job[a.njobs++] = j;
    return true;
}

bool add_bias_job(RowJobs &a, void *b, const void *sub_old, void *sub_new, const CopyArgs *o, const CopyArgs *n)
{
    const CopyArgs &c = o ? *o : *n;
    const int64_t blocks = a.blocks + ((c.rows ? c.nr * c.G : c.N_out) + 255) / 256;
    if (a.njobs == kMaxRowJobs || blocks > 0x7fffffffLL) return false;
    RowJob j{};
    j.kind = c.rows ? ROW_BIAS_HIDDEN : ROW_BIAS_OUT;
    j.W = b; j.sub_old = sub_old; j.sub_new = sub_new; j.nr = c.nr; j.N_out = c.N_out;
    if (o) { j.rows_old = o->rows; j.slot_old = o->slotr; }
    if (n) { j.rows_new = n->rows; j.slot_new = n->slotr; }
    j.blk0 = (int32_t)a.blocks;
    a.blocks = blocks;
    a.bytes[3] += (double)c.esz * (c.rows ? (o && n ? 3 : 2) * c.N_out : (double)(c.G + 1) * c.N_out);
    a.job[a.njobs++] = j;
    return true;
}

hipError_t launch_row_jobs(const RowJobs &a, bool merge, bool part, int dtype, hipStream_t st)
{
    if (a.njobs == 0 || a.blocks == 0) return hipSuccess;
    if (a.blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    tag_kernel(merge && part ? "k_row_jobs<resample>" : (merge ? "k_row_jobs<scatter>" : "k_row_jobs<gather>"), 0.0,
               a.bytes[0] + a.bytes[1] + a.bytes[2] + a.bytes[3]);
    const dim3 grid((unsigned)a.blocks);
    if (dtype == IST_BF16) launch_row_jobs_typed<BF16>(a, merge, part, grid, st);
    else launch_row_jobs_typed<F32>(a, merge, part, grid, st);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// export one subnet block in permutation order
// ----------------------------------------------------------------------------
template <typename E>
__global__ void k_export(const E *__restrict__ sub, E *__restrict__ dst, int64_t nr, int64_t nc, int64_t pr, int64_t pc,
                         const int32_t *__restrict__ p2q_r, int64_t perm_r, int64_t pack_r,
                         const int32_t *__restrict__ p2q_c, int64_t perm_c, int64_t pack_c, bool transposed)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nr * nc) return;
    int64_t i = idx / nc, j = idx % nc;
    int64_t qi = p2q_r ? (int64_t)p2q_r[perm_r + i] - pack_r : i;
    int64_t qj = p2q_c ? (int64_t)p2q_c[perm_c + j] - pack_c : j;
    if (qi < 0 || qi >= pr || qj < 0 || qj >= pc) return;
    dst[idx] = transposed ? sub[qj * pr + qi] : sub[qi * pc + qj];
}

hipError_t launch_export(const void *sub, void *dst, int64_t nr, int64_t nc, int64_t pr, int64_t pc,
                         const int32_t *p2q_r, int64_t perm_r, int64_t pack_r, const int32_t *p2q_c,
                         int64_t perm_c, int64_t pack_c, bool transposed, int esz, hipStream_t st)
{
    int64_t n = nr * nc;
    if (n == 0) return hipSuccess;
    dim3 grid((unsigned)((n + 255) / 256));
    if (esz == 2)
        hipLaunchKernelGGL(k_export<uint16_t>, grid, dim3(256), 0, st, (const uint16_t *)sub, (uint16_t *)dst, nr, nc, pr,
                           pc, p2q_r, perm_r, pack_r, p2q_c, perm_c, pack_c, transposed);
    else
        hipLaunchKernelGGL(k_export<uint32_t>, grid, dim3(256), 0, st, (const uint32_t *)sub, (uint32_t *)dst, nr, nc, pr,
                           pc, p2q_r, perm_r, pack_r, p2q_c, perm_c, pack_c, transposed);
    return hipGetLastError();
}

}  // namespace ist
