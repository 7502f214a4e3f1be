// The chain plan of the triangular solves.  With a random ordering the lowest-ranked rows
// hold most of the dependency chain (their walks end at one another): a 64^3 grid has 836
// levels, of which the first 135,000 of its 262,144 rows hold nine tenths, and a level costs
// about one store-to-load latency (1.2-1.5 us).  The chain rows are cut into blocks, and with
// X, the inverse of a block's diagonal block of Y (unit lower triangular, sparse), a block
// takes two dependent steps however deep it is:
//   forward:   c_i = w_i / D_i - sum over row i of Y on slots before the block of z,
//              z_i = sum over row i of X of c
//   backward:  c_i = r_node(i) - sum over row i of Y^T on slots past the block of w,
//              w_i = sum over column i of X of c
// Both are rows of one longer triangular system in (c of a block, z of it, c of the next,
// ...), which the same sync-free kernel substitutes: m chain rows make 2 m rows.
// (Where the first rows past the head are short the solves do without: see the rule of the
// build.)  33 blocks of 131,072 rows, one application without and with the plan, in us: 128^3
// 2,847 and 2,176, 64^3 1,050 and 757, geometric graph of 2M nodes 8,054 and 6,100; the plan
// adds 2 ms to the 109.6 ms build of 128^3.  Dense inverses of blocks of 2,048 rows instead
// (16.8 MB a block and direction) came to 2,375, 850 and 6,142.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "factor.hpp"

namespace srw {

namespace {

constexpr int BLOCK = 256;
constexpr int WAVES = BLOCK / 64;
constexpr int BLOCK_MAX = 8192;     // rows of a block (bits of a wave's mask in LDS)
constexpr int ROW_MAX = 1024;       // entries of a row of X
constexpr int POOL_CHUNK = 1024;    // entries a wave takes from the pool at once
constexpr int X_GRID = 1024;        // workgroups of k_chain_x: its waves keep pool chunks
constexpr int64_t POOL_PER_ROW = 64;
constexpr int LISTS = 4;            // rows of X a wave reads at once
constexpr int DEPTH_MIN = 12;       // levels of a block from which two steps are fewer by enough

// Rows of the block that starts at slot s.  An eighth of the slots before it: about 20
// levels deep and 25 entries to a row of X on 3D grids wherever it lies (64^3: 20, 21, 21
// levels and 28, 27, 20 entries at slots 8,192, 16,384, 32,768; twice the rows: 37, 34, 33
// levels and 168, 153, 109 entries).
int64_t block_rows(int64_t s, int shrink)
{
    return std::min<int64_t>(std::max<int64_t>(s / 8 / 64 * 64, 512), BLOCK_MAX) >> shrink;
}

__global__ void k_chain_blocks(int64_t m, int nblk, const int32_t* __restrict__ bnd,
                               int32_t* __restrict__ lo, int32_t* __restrict__ hi)
{
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= m) return;
    int a = 0, b = nblk;  // bnd[a] <= i < bnd[b]
    while (b - a > 1) {
        const int k = (a + b) / 2;
        if (bnd[k] <= i) a = k;
        else b = k;
    }
    lo[i] = bnd[a];
    hi[i] = bnd[b];
}

// In-block entries of the chain rows' rows of Y: their number (len), or with iptr, their
// chain rows and values in row order.  One wave per row.
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_chain_entries(int64_t h, int64_t m,
                                                         const int64_t* __restrict__ ptr,
                                                         const int32_t* __restrict__ col,
                                                         const T* __restrict__ val,
                                                         const int32_t* __restrict__ lo,
                                                         int32_t* __restrict__ len,
                                                         const int64_t* __restrict__ iptr,
                                                         int32_t* __restrict__ icol,
                                                         T* __restrict__ ival)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6);
    if (i >= m) return;  // whole wave
    const int64_t first = h + lo[i], e = ptr[h + i + 1];
    int n = 0;
    for (int64_t qb = ptr[h + i]; qb < e; qb += 64) {
        const int64_t q = qb + lane;
        const int32_t c = q < e ? col[q] : -1;
        const bool in = c >= first;
        const uint64_t mask = ballot(in);
        if (iptr && in) {
            const int64_t o = iptr[i] + n + __popcll(mask & ((1ull << lane) - 1ull));
            icol[o] = (int32_t)(c - h);
            ival[o] = val[q];
        }
        n += __popcll(mask);
    }
    if (!iptr && lane == 0) len[i] = n;
}

__global__ void k_set_end(int64_t* ptr, const int32_t* __restrict__ len, int64_t m)
{
    ptr[m] = m > 0 ? ptr[m - 1] + len[m - 1] : 0;
}

__global__ void k_chain_keys(int64_t m, const int32_t* __restrict__ lev, uint32_t* __restrict__ key,
                             uint32_t* __restrict__ val)
{
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= m) return;
    key[i] = (uint32_t)lev[i];
    val[i] = (uint32_t)i;
}

// beg[k] = first of the m sorted keys >= k, k = 0 .. n
__global__ void k_key_begin(int64_t n, const uint32_t* __restrict__ key, int64_t m,
                            int64_t* __restrict__ beg)
{
    const int64_t k = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (k > n) return;
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((int64_t)key[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    beg[k] = lo;
}

// Rows of X of one level's chain rows: X_i = e_i - sum over the in-block entries q of row i
// of Y of Y_iq X_q, the X_q being rows of lower levels (earlier launches).  One wave per
// row: the union of the rows' columns as bits in LDS (columns of the block), a prefix sum
// over their words, then the rows' values added in the order of the entries at the place
// of their column: a fixed order, and columns ascending.
// A row is a few dependent reads of lists made by other waves; thousands of rows in flight
// hide them.
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_chain_x(
    int64_t lbeg, int64_t lend, const uint32_t* __restrict__ rows, const int64_t* __restrict__ iptr,
    const int32_t* __restrict__ icol, const T* __restrict__ ival, const int32_t* __restrict__ blo,
    int64_t* xbeg, int32_t* xlen, int32_t* xc, int32_t* xr, T* xv, int64_t cap,
    unsigned long long* pool, int64_t* wave_cur, int32_t* wave_left, int* err)
{
    constexpr int WORDS = BLOCK_MAX / 32;
    __shared__ uint32_t mask_[WAVES][WORDS];
    __shared__ uint32_t pre_[WAVES][WORDS];
    __shared__ double acc_[WAVES][ROW_MAX];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t* mask = mask_[wv];
    uint32_t* pre = pre_[wv];
    double* acc = acc_[wv];
    const int64_t wid = (int64_t)blockIdx.x * WAVES + wv;
    int64_t cur = wave_cur[wid];
    int32_t left = wave_left[wid];
    for (int64_t k = lbeg + wid; k < lend; k += (int64_t)gridDim.x * WAVES) {
        const int32_t i = (int32_t)rows[k], b0 = blo[i];
        const int words = (i - b0) / 32 + 1;
        const int64_t q0 = iptr[i], q1 = iptr[i + 1];
        for (int w = lane; w < words; w += 64) mask[w] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (lane == 0) atomicOr(&mask[(i - b0) >> 5], 1u << ((i - b0) & 31));
        for (int64_t qb = q0; qb < q1; qb += 64) {
            const int nq = (int)(q1 - qb < 64 ? q1 - qb : 64);
            const int32_t q = lane < nq ? icol[qb + lane] : 0;
            const int64_t xb = lane < nq ? xbeg[q] : 0;
            const int32_t xn = lane < nq ? xlen[q] : 0;
            for (int j = 0; j < nq; j += LISTS) {
                int64_t b[LISTS];
                int n[LISTS], c[LISTS];
#pragma unroll
                for (int u = 0; u < LISTS; ++u) {
                    b[u] = __shfl(xb, (j + u) & 63);
                    n[u] = j + u < nq ? __shfl(xn, (j + u) & 63) : 0;
                    c[u] = lane < n[u] ? xc[b[u] + lane] - b0 : 0;
                }
#pragma unroll
                for (int u = 0; u < LISTS; ++u) {
                    if (lane < n[u]) atomicOr(&mask[c[u] >> 5], 1u << (c[u] & 31));
                    for (int t = lane + 64; t < n[u]; t += 64) {
                        const int e = xc[b[u] + t] - b0;
                        atomicOr(&mask[e >> 5], 1u << (e & 31));
                    }
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        int total = 0;
        for (int w0 = 0; w0 < words; w0 += 64) {
            const int w = w0 + lane;
            const int n = w < words ? __popc(mask[w]) : 0;
            int sum = n;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int up = __shfl_up(sum, off);
                if (lane >= off) sum += up;
            }
            if (w < words) pre[w] = (uint32_t)(total + sum - n);
            total += __shfl(sum, 63);
        }
        bool ok = total <= ROW_MAX;
        if (ok && left < total) {
            unsigned long long at = 0;
            if (lane == 0) at = atomicAdd(pool, (unsigned long long)POOL_CHUNK);
            cur = (int64_t)__shfl(at, 0);
            left = POOL_CHUNK;
            ok = cur + POOL_CHUNK <= cap;
            if (!ok) left = 0;
        }
        if (!ok) {  // the caller makes smaller blocks, or does without
            if (lane == 0) {
                atomicOr(err, 1);
                xbeg[i] = 0;
                xlen[i] = 0;
            }
            continue;
        }
        auto place = [&](int c) { return (int)pre[c >> 5] + __popc(mask[c >> 5] & ((1u << (c & 31)) - 1u)); };
        for (int t = lane; t < total; t += 64) acc[t] = 0.0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        for (int64_t qb = q0; qb < q1; qb += 64) {
            const int nq = (int)(q1 - qb < 64 ? q1 - qb : 64);
            const int32_t q = lane < nq ? icol[qb + lane] : 0;
            const double y = lane < nq ? (double)ival[qb + lane] : 0.0;
            const int64_t xb = lane < nq ? xbeg[q] : 0;
            const int32_t xn = lane < nq ? xlen[q] : 0;
            for (int j = 0; j < nq; j += LISTS) {
                int64_t b[LISTS];
                int n[LISTS], c[LISTS];
                double x[LISTS];
#pragma unroll
                for (int u = 0; u < LISTS; ++u) {
                    b[u] = __shfl(xb, (j + u) & 63);
                    n[u] = j + u < nq ? __shfl(xn, (j + u) & 63) : 0;
                    c[u] = lane < n[u] ? xc[b[u] + lane] - b0 : 0;
                    x[u] = lane < n[u] ? (double)xv[b[u] + lane] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < LISTS; ++u) {
                    const double yj = __shfl(y, (j + u) & 63);
                    if (lane < n[u]) acc[place(c[u])] += yj * x[u];
                    for (int t = lane + 64; t < n[u]; t += 64)
                        acc[place(xc[b[u] + t] - b0)] += yj * (double)xv[b[u] + t];
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                }
            }
        }
        for (int w = lane; w < words; w += 64) {
            uint32_t bits = mask[w];
            int at = (int)pre[w];
            while (bits) {
                const int c = 32 * w + __ffs(bits) - 1;
                bits &= bits - 1u;
                xc[cur + at] = b0 + c;
                xr[cur + at] = i;
                xv[cur + at] = (T)(b0 + c == i ? 1.0 : -acc[at]);
                ++at;
            }
        }
        if (lane == 0) {
            xbeg[i] = cur;
            xlen[i] = total;
        }
        cur += total;
        left -= total;
    }
    if (lane == 0) {
        wave_cur[wid] = cur;
        wave_left[wid] = left;
    }
}

// Keys (column) and pool places of X's entries, row by row.
__global__ __launch_bounds__(BLOCK) void k_chain_x_keys(int64_t m, const int64_t* __restrict__ xptr,
                                                        const int64_t* __restrict__ xbeg,
                                                        const int32_t* __restrict__ xlen,
                                                        const int32_t* __restrict__ xc,
                                                        uint32_t* __restrict__ key,
                                                        uint32_t* __restrict__ idx)
{
    const int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 4;
    if (i >= m) return;
    const int64_t b = xbeg[i], o = xptr[i];
    for (int t = threadIdx.x & 15; t < xlen[i]; t += 16) {
        key[o + t] = (uint32_t)xc[b + t];
        idx[o + t] = (uint32_t)(b + t);
    }
}

// Lengths, places and nodes of the 2 m rows of either direction, in the order they are
// substituted: block [a, b) takes the rows 2 a .. 2 b - 1 forward (c, then z) and, the
// blocks in descending order, 2 (m - b) .. 2 (m - a) - 1 backward (c, then w; slots
// descending).  A row's place is its slot (z, w) or n + its chain row (c).
__global__ void k_chain_shape(int64_t n, int64_t h, int64_t m, const int32_t* __restrict__ blo,
                              const int32_t* __restrict__ bhi, const int64_t* __restrict__ fptr,
                              const int64_t* __restrict__ bptr, const int32_t* __restrict__ bcol,
                              const int32_t* __restrict__ ilen, const int32_t* __restrict__ xlen,
                              const int64_t* __restrict__ tbeg, const int32_t* __restrict__ slot_node,
                              int32_t* __restrict__ flen, int32_t* __restrict__ blen,
                              int32_t* __restrict__ fpos, int32_t* __restrict__ bpos,
                              int32_t* __restrict__ fnode, int32_t* __restrict__ bnode)
{
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= m) return;
    const int64_t a = blo[i], b = bhi[i], s = h + i;
    const int32_t node = slot_node[s];
    const int64_t fc = a + i, fz = b + i;
    const int64_t bc = 2 * (m - b) + (b - 1 - i), bw = bc + (b - a);
    flen[fc] = (int32_t)(fptr[s + 1] - fptr[s]) - ilen[i];
    flen[fz] = xlen[i];
    int64_t lo = bptr[s], hi = bptr[s + 1];  // slots descend along a row of Y^T
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (bcol[mid] >= h + b) lo = mid + 1;
        else hi = mid;
    }
    blen[bc] = (int32_t)(lo - bptr[s]);
    blen[bw] = (int32_t)(tbeg[i + 1] - tbeg[i]);
    fpos[fc] = bpos[bc] = (int32_t)(n + i);
    fpos[fz] = bpos[bw] = (int32_t)s;
    fnode[fc] = fnode[fz] = bnode[bc] = bnode[bw] = node;
}

// Entries of the 2 m forward rows, one wave per chain row.
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_chain_fill_f(
    int64_t n, int64_t h, int64_t m, const int32_t* __restrict__ blo, const int32_t* __restrict__ bhi,
    const int64_t* __restrict__ ptr, const int32_t* __restrict__ col, const T* __restrict__ val,
    const int64_t* __restrict__ xbeg, const int32_t* __restrict__ xlen, const int32_t* __restrict__ xc,
    const T* __restrict__ xv, const int64_t* __restrict__ optr, int32_t* __restrict__ ocol,
    T* __restrict__ oval)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6);
    if (i >= m) return;  // whole wave
    const int64_t first = h + blo[i], e = ptr[h + i + 1];
    int64_t o = optr[blo[i] + i];
    for (int64_t qb = ptr[h + i]; qb < e; qb += 64) {
        const int64_t q = qb + lane;
        const int32_t c = q < e ? col[q] : INT_MAX;
        const bool out = c < first;
        const uint64_t mask = ballot(out);
        if (out) {
            const int64_t at = o + __popcll(mask & ((1ull << lane) - 1ull));
            ocol[at] = c;
            oval[at] = val[q];
        }
        o += __popcll(mask);
    }
    o = optr[bhi[i] + i];
    const int64_t b = xbeg[i];
    for (int t = lane; t < xlen[i]; t += 64) {
        ocol[o + t] = (int32_t)(n + xc[b + t]);
        oval[o + t] = -xv[b + t];
    }
}

// Entries of the 2 m backward rows, one wave per chain row.
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_chain_fill_b(
    int64_t n, int64_t h, int64_t m, const int32_t* __restrict__ blo, const int32_t* __restrict__ bhi,
    const int64_t* __restrict__ ptr, const int32_t* __restrict__ col, const T* __restrict__ val,
    const int64_t* __restrict__ tbeg, const uint32_t* __restrict__ tidx, const int32_t* __restrict__ xr,
    const T* __restrict__ xv, const int64_t* __restrict__ optr, int32_t* __restrict__ ocol,
    T* __restrict__ oval)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6);
    if (i >= m) return;  // whole wave
    const int64_t a = blo[i], b = bhi[i];
    const int64_t bc = 2 * (m - b) + (b - 1 - i), bw = bc + (b - a);
    const int64_t q = ptr[h + i], o = optr[bc], len = optr[bc + 1] - o;
    for (int64_t t = lane; t < len; t += 64) {
        ocol[o + t] = col[q + t];
        oval[o + t] = val[q + t];
    }
    const int64_t z = optr[bw];
    for (int64_t t = tbeg[i] + lane; t < tbeg[i + 1]; t += 64) {
        const uint32_t x = tidx[t];
        ocol[z + t - tbeg[i]] = (int32_t)(n + xr[x]);
        oval[z + t - tbeg[i]] = -xv[x];
    }
}

unsigned rows_grid(int64_t m) { return (unsigned)((m + WAVES - 1) / WAVES); }

template <typename T>
int build(srw_factor* F, int64_t h, int64_t m, int shrink, Arena& keep, Arena& tmp, int64_t* pinned,
          hipStream_t s, bool* too_big)
{
    const int64_t n = F->n;
    const unsigned g = (unsigned)grid_for(m, BLOCK);
    *too_big = false;
    std::vector<int32_t> bnd(1, 0);
    while (bnd.back() < m)
        bnd.push_back((int32_t)std::min<int64_t>(m, bnd.back() + block_rows(h + bnd.back(), shrink)));
    int32_t* dbnd = tmp.alloc<int32_t>(bnd.size());
    int32_t* blo = tmp.alloc<int32_t>(m);
    int32_t* bhi = tmp.alloc<int32_t>(m);
    int32_t* ilen = tmp.alloc<int32_t>(m);
    int32_t* xlen = tmp.alloc<int32_t>(m);
    int64_t* iptr = tmp.alloc<int64_t>(m + 1);
    int64_t* xbeg = tmp.alloc<int64_t>(m);
    int64_t* xptr = tmp.alloc<int64_t>(m + 1);
    int64_t* tbeg = tmp.alloc<int64_t>(m + 1);
    int32_t* lev = tmp.alloc<int32_t>(m);
    uint32_t* key = tmp.alloc<uint32_t>(m);
    uint32_t* key2 = tmp.alloc<uint32_t>(m);
    uint32_t* val = tmp.alloc<uint32_t>(m);
    uint32_t* val2 = tmp.alloc<uint32_t>(m);
    void* rt = tmp.alloc<char>(radix_tmp_bytes(m));
    void* st = tmp.alloc<char>(scan_tmp_bytes(2 * m));
    const int64_t cap = m * POOL_PER_ROW;
    int32_t* xc = tmp.alloc<int32_t>(cap);
    int32_t* xr = tmp.alloc<int32_t>(cap);
    T* xv = tmp.alloc<T>(cap);
    int64_t* wcur = tmp.alloc<int64_t>(X_GRID * WAVES);
    int32_t* wleft = tmp.alloc<int32_t>(X_GRID * WAVES);
    int64_t* misc = tmp.alloc<int64_t>(2);  // pool, error
    int64_t* lbeg = tmp.alloc<int64_t>(258);
    if (tmp.last != hipSuccess) return SRW_E_NOMEM;
    SRW_HIP(hipMemcpyAsync(dbnd, bnd.data(), bnd.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    SRW_HIP(hipMemsetAsync(wleft, 0, X_GRID * WAVES * sizeof(int32_t), s));
    SRW_HIP(hipMemsetAsync(wcur, 0, X_GRID * WAVES * sizeof(int64_t), s));
    SRW_HIP(hipMemsetAsync(misc, 0, 2 * sizeof(int64_t), s));
    k_chain_blocks<<<g, BLOCK, 0, s>>>(m, (int)bnd.size() - 1, dbnd, blo, bhi);
    k_chain_entries<T><<<rows_grid(m), BLOCK, 0, s>>>(h, m, F->fptr, F->fcol, (const T*)F->fval, blo, ilen,
                                                      nullptr, nullptr, nullptr);
    SRW_HIP(exclusive_scan_i32_to_i64(ilen, iptr, m, st, s));
    k_set_end<<<1, 1, 0, s>>>(iptr, ilen, m);
    SRW_HIP(hipMemcpyAsync(&pinned[0], iptr + m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipStreamSynchronize(s));  // (bnd is read too)
    int32_t* icol = tmp.alloc<int32_t>(pinned[0]);
    T* ival = tmp.alloc<T>(pinned[0]);
    if (!icol || !ival) return SRW_E_NOMEM;
    k_chain_entries<T><<<rows_grid(m), BLOCK, 0, s>>>(h, m, F->fptr, F->fcol, (const T*)F->fval, blo, ilen, iptr,
                                                      icol, ival);
    SRW_HIP(hipGetLastError());
    int32_t depth = 0;
    const int lst = row_levels(m, nullptr, iptr, icol, lev, &depth, s);
    if (lst) return lst;
    if (depth > 256 || depth < DEPTH_MIN) {
        *too_big = depth > 256;
        return SRW_OK;
    }
    uint32_t *ko, *vo;
    k_chain_keys<<<g, BLOCK, 0, s>>>(m, lev, key, val);
    SRW_HIP(radix_sort_u32(key, val, key2, val2, m, 8, rt, &ko, &vo, s));
    k_key_begin<<<2, BLOCK, 0, s>>>(depth, ko, m, lbeg);
    std::vector<int64_t> lhost((size_t)depth + 1);
    SRW_HIP(hipMemcpyAsync(lhost.data(), lbeg, ((size_t)depth + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipStreamSynchronize(s));
    for (int32_t l = 0; l < depth; ++l) {
        const unsigned gx = (unsigned)std::min<int64_t>(X_GRID, rows_grid(lhost[l + 1] - lhost[l]));
        k_chain_x<T><<<gx, BLOCK, 0, s>>>(lhost[l], lhost[l + 1], vo, iptr, icol, ival, blo, xbeg, xlen, xc, xr, xv,
                                          cap, (unsigned long long*)misc, wcur, wleft, (int*)(misc + 1));
    }
    SRW_HIP(exclusive_scan_i32_to_i64(xlen, xptr, m, st, s));
    k_set_end<<<1, 1, 0, s>>>(xptr, xlen, m);
    SRW_HIP(hipMemcpyAsync(&pinned[0], xptr + m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipMemcpyAsync(&pinned[1], misc + 1, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipStreamSynchronize(s));
    if (pinned[1]) {
        *too_big = true;
        return SRW_OK;
    }
    const int64_t nx = pinned[0];
    uint32_t* xk = tmp.alloc<uint32_t>(nx);
    uint32_t* xk2 = tmp.alloc<uint32_t>(nx);
    uint32_t* xi = tmp.alloc<uint32_t>(nx);
    uint32_t* xi2 = tmp.alloc<uint32_t>(nx);
    void* rx = tmp.alloc<char>(radix_tmp_bytes(nx));
    int32_t* flen = tmp.alloc<int32_t>(2 * m);
    int32_t* blen = tmp.alloc<int32_t>(2 * m);
    ChainPlan& C = F->chain;
    C.fptr = keep.alloc<int64_t>(2 * m + 1);
    C.bptr = keep.alloc<int64_t>(2 * m + 1);
    C.fpos = keep.alloc<int32_t>(2 * m);
    C.bpos = keep.alloc<int32_t>(2 * m);
    C.fnode = keep.alloc<int32_t>(2 * m);
    C.bnode = keep.alloc<int32_t>(2 * m);
    if (tmp.last != hipSuccess || keep.last != hipSuccess) return SRW_E_NOMEM;
    k_chain_x_keys<<<(unsigned)grid_for(16 * m, BLOCK), BLOCK, 0, s>>>(m, xptr, xbeg, xlen, xc, xk, xi);
    int bits = 8;
    while (((int64_t)1 << bits) < m) bits += 8;
    SRW_HIP(radix_sort_u32(xk, xi, xk2, xi2, nx, bits, rx, &ko, &vo, s));
    k_key_begin<<<(unsigned)grid_for(m + 1, BLOCK), BLOCK, 0, s>>>(m, ko, nx, tbeg);
    k_chain_shape<<<g, BLOCK, 0, s>>>(n, h, m, blo, bhi, F->fptr, F->bptr, F->bcol, ilen, xlen, tbeg, F->slot_node,
                                      flen, blen, C.fpos, C.bpos, C.fnode, C.bnode);
    SRW_HIP(exclusive_scan_i32_to_i64(flen, C.fptr, 2 * m, st, s));
    k_set_end<<<1, 1, 0, s>>>(C.fptr, flen, 2 * m);
    SRW_HIP(exclusive_scan_i32_to_i64(blen, C.bptr, 2 * m, st, s));
    k_set_end<<<1, 1, 0, s>>>(C.bptr, blen, 2 * m);
    SRW_HIP(hipMemcpyAsync(&pinned[0], C.fptr + 2 * m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipMemcpyAsync(&pinned[1], C.bptr + 2 * m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SRW_HIP(hipStreamSynchronize(s));
    C.fcol = keep.alloc<int32_t>(pinned[0]);
    C.fval = keep.alloc<T>(pinned[0]);
    C.bcol = keep.alloc<int32_t>(pinned[1]);
    C.bval = keep.alloc<T>(pinned[1]);
    if (keep.last != hipSuccess) return SRW_E_NOMEM;
    k_chain_fill_f<T><<<rows_grid(m), BLOCK, 0, s>>>(n, h, m, blo, bhi, F->fptr, F->fcol, (const T*)F->fval, xbeg,
                                                     xlen, xc, xv, C.fptr, C.fcol, (T*)C.fval);
    k_chain_fill_b<T><<<rows_grid(m), BLOCK, 0, s>>>(n, h, m, blo, bhi, F->bptr, F->bcol, (const T*)F->bval, tbeg,
                                                     vo, xr, xv, C.bptr, C.bcol, (T*)C.bval);
    SRW_HIP(hipGetLastError());
    C.h = h;
    C.m = m;
    return SRW_OK;
}

}  // namespace

int chain_build(srw_factor* F, int64_t h, int64_t m, Arena& keep, int64_t* pinned, hipStream_t s)
{
    if (F->n + m > INT32_MAX || m * POOL_PER_ROW > INT32_MAX) return SRW_OK;  // 32-bit places
    for (int shrink = 0; shrink <= 2; ++shrink) {
        Arena tmp, own;
        bool too_big = false;
        const int st = F->precision == SRW_FP32 ? build<float>(F, h, m, shrink, own, tmp, pinned, s, &too_big)
                                                : build<double>(F, h, m, shrink, own, tmp, pinned, s, &too_big);
        (void)hipStreamSynchronize(s);
        tmp.release();
        if (st != SRW_OK) {
            own.release();
            F->chain = ChainPlan{};
            if (st != SRW_E_NOMEM) return st;
            (void)hipGetLastError();  // no memory for a plan: the solves do without
            return SRW_OK;
        }
        keep.blocks.insert(keep.blocks.end(), own.blocks.begin(), own.blocks.end());
        if (!too_big) return SRW_OK;
    }
    return SRW_OK;
}

}  // namespace srw
