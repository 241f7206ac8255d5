// Device kernels of the PDHG library (gfx950, wave64).
//
// One PDHG iteration (Algorithm 1 inner loop, diagonal steps from the
// preconditioner) is two bandwidth-bound passes:
//   column pass over the CSC copy:  g = c_hat - A^T y,
//       x+ = proj_[l,u](x - t D_c^2 g),  x_bar = 2 x+ - x     (primal step)
//   row pass over the CSR:          y+ = proj_Y(y + s D_r^2 (b - A x_bar))
//                                                             (dual step)
// Both passes use the same tile kernel: a workgroup streams a contiguous
// run of nonzeros (coalesced, non-temporal so the gathered vector keeps the
// L2), multiplies by the gathered vector into LDS, then reduces each row
// with a power-of-two group of lanes sized to the tile's row count and
// applies the fused projection epilogue.  Rows longer than a tile are cut
// into segments whose partial sums a small combine kernel adds in a fixed
// order, so no floating-point atomics are used anywhere and every result is
// bitwise reproducible.
//
// Every R iterations a check (FP64 accumulation) evaluates the relative KKT
// errors of Section 2.2 and the restart quantities; a one-workgroup-per-
// instance decision kernel reduces them in a fixed order and sets status,
// restart and step sizes in FP64 on the device.  With restarts to the
// average the epilogues also fold every iterate into running means, a
// second check evaluates the means, and the decision takes the better of
// the two points.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "scylla_internal.h"
#include "kernels.h"

namespace scy {

// ------------------------------------------------------------------ utils
// The hardware hands consecutive workgroups to the 8 XCDs in turn; map them
// so every XCD works on one contiguous range of tiles (neighbouring tiles
// share cache lines of the row-side vectors in that XCD's L2).
__device__ __forceinline__ int xcd_tile(int b, int nb)
{
    const int xcd = b & 7, local = b >> 3;
    const int per = nb >> 3, rem = nb & 7;
    const int base = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
    return base + local;
}

template <class V>
__device__ __forceinline__ V wave_sum_width(V v, int width)
{
    for (int off = width >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, width);
    return v;
}

// v of the lane that CTRL pairs this one with (data-parallel primitives: a
// register operand modifier, against an LDS round trip for a shuffle).
template <int CTRL, class V>
__device__ __forceinline__ V dpp_pair(V v)
{
    if constexpr (sizeof(V) == 8) {
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
        return __hiloint2double(hi, lo);
    } else {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
    }
}

// Sum over aligned groups of `width` lanes (a power of two), in every lane:
// neighbours, pairs of neighbours, then mirrored halves, whose lanes hold
// equal partial sums.
template <class V>
__device__ __forceinline__ V group_sum(V v, int width)
{
    if (width < 2) return v;
    v += dpp_pair<0xb1>(v);  // quad lanes 1 0 3 2
    if (width < 4) return v;
    v += dpp_pair<0x4e>(v);  // quad lanes 2 3 0 1
    if (width < 8) return v;
    v += dpp_pair<0x141>(v);  // mirror of 8 lanes
    if (width < 16) return v;
    v += dpp_pair<0x140>(v);  // mirror of 16 lanes
    if (width < 32) return v;
    v += __shfl_xor(v, 16, 64);
    if (width < 64) return v;
    return v + __shfl_xor(v, 32, 64);
}

// Fixed-order block sum (result valid in thread 0).
template <class V, int NT>
__device__ __forceinline__ V block_sum(V v, V *red)
{
    v = wave_sum_width(v, 64);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) red[w] = v;
    __syncthreads();
    V s = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) s += red[q];
    }
    return s;
}

// Fixed-order block sum of two values (results valid in thread 0); red
// holds 2 * NT / 64 doubles.  Every thread of the block must call it.
template <int NT>
__device__ __forceinline__ void block_sum2(double &a, double &b, double *red)
{
    a = wave_sum_width(a, 64);
    b = wave_sum_width(b, 64);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) {
        red[2 * w] = a;
        red[2 * w + 1] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) {
            sa += red[2 * q];
            sb += red[2 * q + 1];
        }
        a = sa;
        b = sb;
    }
}

// Fixed-order block sums of N values to out[N] (one thread each); red holds
// NT / 64 * N doubles.  One barrier, where a block sum per value takes two.
template <int NT, int N>
__device__ __forceinline__ void block_sums(const double (&acc)[N], double *red, double *out)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double v = group_sum(acc[k], 64);
        if (l == 0) red[N * w + k] = v;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) s += red[N * q + threadIdx.x];
        out[threadIdx.x] = s;
    }
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h)
{
    return __uint_as_float(((uint32_t)h) << 16);
}

// Loads of the streamed matrix words / values (read once per pass).
template <int FMT>
struct Entry {
    uint32_t w;
    float f;
    double d;
};

// A matrix entry load: non-temporal (streamed past the caches), or with
// FMT_CACHED in the format a plain load, which the device's last-level
// (Infinity) cache keeps across iterations when an iteration's data fits.
template <int FMT, class T>
__device__ __forceinline__ T mat_load(const T *p)
{
    if constexpr ((FMT & FMT_CACHED) != 0) return *p;
    else return __builtin_nontemporal_load(p);
}

template <int FMT, class A>
__device__ __forceinline__ void load_entry(const MatView &M, int e, uint32_t &w, A &a)
{
    constexpr int F = FMT & ~(FMT_CACHED | FMT_SORTED);
    w = mat_load<FMT>(M.ent + e);
    if constexpr (F == FMT_BF16) {
        a = (A)bf16_to_f32(mat_load<FMT>((const uint16_t *)M.val + e));
    } else if constexpr (F == FMT_F32) {
        a = (A)mat_load<FMT>((const float *)M.val + e);
    } else if constexpr (F == FMT_F64) {
        a = (A)mat_load<FMT>((const double *)M.val + e);
    } else {
        a = (A)0;
    }
}

template <int FMT, class A>
__device__ __forceinline__ int decode_entry(const MatView &M, uint32_t w, A &a)
{
    if constexpr ((FMT & ~(FMT_CACHED | FMT_SORTED)) == FMT_PACKED) {
        a = (A)((int32_t)w >> M.shift);
        return (int)(w & M.mask);
    } else {
        return (int)w;
    }
}

// Entries e0 + q NT + tid < e1 of a tile, q < EPT, in registers; at[q]: the
// place of an entry's product in the tile (its own, or with FMT_SORTED the one
// kept beside it).
template <class A, int FMT, int NT, int EPT>
__device__ __forceinline__ void load_tile(const MatView &M, int e0, int e1, uint32_t (&w)[EPT], A (&a)[EPT],
                                          int (&at)[EPT])
{
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = e0 + q * NT + (int)threadIdx.x;
        w[q] = 0;
        a[q] = (A)0;
        at[q] = e - e0;
        if (e < e1) {
            load_entry<FMT, A>(M, e, w[q], a[q]);
            if constexpr ((FMT & FMT_SORTED) != 0) at[q] = mat_load<FMT>(M.pos + e);
        }
    }
}

// prod[place] = a_e * vec[idx_e] of the loaded entries.
template <class A, class GV, int FMT, int NT, int EPT>
__device__ __forceinline__ void tile_products(const MatView &M, const GV *__restrict__ vec, int e0, int e1,
                                              const uint32_t (&w)[EPT], A (&a)[EPT], const int (&at)[EPT], A *prod)
{
    const int tid = threadIdx.x;
    A g[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = e0 + q * NT + tid;
        g[q] = (A)0;
        if (e < e1) {
            const int idx = decode_entry<FMT, A>(M, w[q], a[q]);
            g[q] = (A)vec[idx];
        }
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = e0 + q * NT + tid;
        if (e < e1) prod[at[q]] = a[q] * g[q];
    }
}

// Stage prod[e - e0] = a_e * vec[idx_e] for e in [e0, e1), e1 - e0 <= NT*EPT.
template <class A, class GV, int FMT, int NT, int EPT>
__device__ __forceinline__ void stage_products(const MatView &M, const GV *__restrict__ vec, int e0,
                                               int e1, A *prod)
{
    uint32_t w[EPT];
    A a[EPT];
    int at[EPT];
    load_tile<A, FMT, NT, EPT>(M, e0, e1, w, a, at);
    tile_products<A, GV, FMT, NT, EPT>(M, vec, e0, e1, w, a, at, prod);
}

// ------------------------------------------------------------ epilogues
// Operands of one row's epilogue, loaded before the LDS barrier so their
// latency overlaps the matrix stream.
template <class V>
struct RowOps {
    V own, rhs, diag2, lo, hi, q;
    V avg;      // running mean (restart to the average)
    double ax;  // running A x (adaptive steps)
    uint8_t sense;
};

// Bounds shared by every column of an instance (binary problems, say): the
// column pass reads them once per workgroup instead of twice per column.
template <class V>
struct InstBounds {
    bool uni;
    V lo, hi;
};

template <class V, int DIR>
__device__ __forceinline__ InstBounds<V> inst_bounds(const PassArgs<V> &p, int inst)
{
    InstBounds<V> b{false, (V)0, (V)0};
    if (DIR == DIR_COL && p.ibnd) {
        b.lo = p.ibnd[2 * inst];
        b.hi = p.ibnd[2 * inst + 1];
        b.uni = b.lo == b.lo;
    }
    return b;
}

template <class V, int DIR>
__device__ __forceinline__ void load_ops(const PassArgs<V> &p, int i, RowOps<V> &o, const InstBounds<V> &ib)
{
    o.own = p.own[i];
    o.rhs = p.rhs[i];
    o.diag2 = p.diag2[i];
    if (p.avg) o.avg = p.avg[i];
    if (DIR == DIR_COL) {
        if (ib.uni) {
            o.lo = ib.lo;
            o.hi = ib.hi;
        } else {
            o.lo = p.lo[i];
            o.hi = p.hi[i];
        }
        if (p.q) o.q = p.q[i];
    } else {
        o.sense = p.sense[i];
        if (p.adapt) o.ax = p.ax[i];
    }
}

// The fused epilogue: primal step (column pass) or dual step (row pass) of
// Algorithm 1 for row i given its sum; with adaptive steps it also adds
// this row's terms of the step-size estimate to ip.  Adaptive steps change
// what the row pass gathers: the column pass stores dx = x+ - x in `bar`,
// the row pass's sum is then (A dx)_i, and (A x_bar)_i = (A x)_i + 2 (A dx)_i
// with the running FP64 (A x)_i.
// Iterates in the running average of restart-to-average once this
// iteration's is folded in (the iterates produced since the last restart),
// or 0 without an average.
template <class V>
__device__ __forceinline__ V avg_count(const PassArgs<V> &p, const InstState &S, int jw)
{
    return p.avg ? (V)(S.k + jw + 1 - S.kr) : (V)0;
}

// Folds the new iterate value v of entry i into the running mean (the first
// iterate after a restart starts it).
template <class V>
__device__ __forceinline__ void fold_avg(const PassArgs<V> &p, int i, V v, V avg, V acnt)
{
    if (acnt > (V)0) p.avg[i] = acnt == (V)1 ? v : avg + (v - avg) / acnt;
}

template <class V, int DIR>
__device__ __forceinline__ void apply_ops(const PassArgs<V> &p, int i, V sum, V step, bool copy_ref,
                                          const RowOps<V> &o, double (&ip)[2], V acnt)
{
    if (DIR == DIR_COL) {
        V xn = o.own + step * o.diag2 * (sum - o.rhs);
        if (p.q) xn /= (V)1 + step * o.diag2 * o.q;  // exact prox of q x^2 / 2
        xn = xn < o.lo ? o.lo : xn;
        xn = xn > o.hi ? o.hi : xn;
        if (copy_ref) p.own_ref[i] = o.own;
        p.bar[i] = p.adapt ? xn - o.own : (V)2 * xn - o.own;
        p.own[i] = xn;
        fold_avg(p, i, xn, o.avg, acnt);
        if (p.adapt) {
            const double d = (double)xn - (double)o.own;
            ip[0] += d * d / (double)o.diag2;
        }
    } else {
        // residual b_i - (A x_bar)_i; with adaptive steps sum = (A dx)_i
        const V res = p.adapt ? (V)((double)o.rhs - (o.ax + 2.0 * (double)sum)) : o.rhs - sum;
        V v = o.own + step * o.diag2 * res;
        if (o.sense == 'G') v = v > (V)0 ? v : (V)0;
        else if (o.sense == 'L') v = v < (V)0 ? v : (V)0;
        if (copy_ref) p.own_ref[i] = o.own;
        p.own[i] = v;
        fold_avg(p, i, v, o.avg, acnt);
        if (p.adapt) {
            const double dy = (double)v - (double)o.own;
            ip[0] += dy * dy / (double)o.diag2;
            ip[1] += dy * (double)sum;
            p.ax[i] = o.ax + (double)sum;
        }
    }
}

// Lanes per row for a tile of `nrows` rows: the largest power of two (<= 64)
// with nrows * L <= NT.
template <int NT>
__device__ __forceinline__ int lanes_per_row(int nrows)
{
    int L = 1;
    while (L < 64 && nrows * (L << 1) <= NT) L <<= 1;
    return L;
}

// Nonzeros [e0, e1) and, for a tile of whole rows, the rows of a normal tile.
struct TileRange {
    int e0, e1, rows;
};

__device__ __forceinline__ TileRange tile_range(const int4 &T)
{
    if (T.w >= 0) return {T.x, T.y, 0};
    const int e0 = ~T.w;
    return {e0, e0 + (T.y >> TILE_ROW_BITS), T.y & ((1 << TILE_ROW_BITS) - 1)};
}

// ------------------------------------------------------- iteration pass
template <class V, int FMT, int DIR, int NT, int EPT, bool EARLY>
__device__ __forceinline__ void pass_tile(const PassArgs<V> &p, const int jw)
{
    constexpr int CH = NT * EPT;
    __shared__ V prod[CH];
    __shared__ V red[NT / 64];
    __shared__ double red2[2 * NT / 64];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int4 T = p.tiles[t];
    // EARLY (one instance): the entries go out before the state is read, so a
    // workgroup waits for three loads in a row (tile, entries, gather), not
    // for five (state and row pointers between); with too few workgroups to
    // cover them they are most of its time (32 adaptive FP64 iterations of a
    // 200k x 400k LP 1.82 -> 1.61 ms, 64 FP32 ones of a 300k x 600k LP 3.10 ->
    // 2.96 ms).  Batches read the state first: their stopped instances would
    // load in vain.
    const int r0 = T.x;
    const TileRange R = tile_range(T);
    uint32_t w[EPT];
    V a[EPT];
    int at[EPT];
    if constexpr (EARLY) load_tile<V, FMT, NT, EPT>(p.M, R.e0, R.e1, w, a, at);
    const InstState &S = p.st[T.z];
    if (S.status != ST_RUN || jw >= S.nrun) return;
    if constexpr (!EARLY) load_tile<V, FMT, NT, EPT>(p.M, R.e0, R.e1, w, a, at);
    const bool copy_ref = (jw == 0) && (S.restart_now != 0);
    const V step = DIR == DIR_COL ? (V)S.t : (V)S.s;
    const V acnt = avg_count(p, S, jw);
    const int tid = threadIdx.x;
    const InstBounds<V> ib = inst_bounds<V, DIR>(p, T.z);
    if (T.w >= 0) {  // one segment of a long row: partial sum only
        tile_products<V, V, FMT, NT, EPT>(p.M, p.gvec, R.e0, R.e1, w, a, at, prod);
        __syncthreads();
        V s = 0;
        for (int q = tid; q < R.e1 - R.e0; q += NT) s += prod[q];
        s = block_sum<V, NT>(s, red);
        if (tid == 0) {
            p.seg[T.w] = s;
            if (p.adapt) p.ipart[2 * t] = p.ipart[2 * t + 1] = 0.0;
        }
        return;
    }
    double ip[2] = {0.0, 0.0};
    const int nrows = R.rows, e0 = R.e0;
    const int L = lanes_per_row<NT>(nrows);
    const int groups = NT / L, lane = tid & (L - 1);
    // first row of this lane group: bounds and epilogue operands up front
    int r = tid / L;
    int rb = 0, re = 0;
    RowOps<V> ops;
    if (r < nrows) {
        rb = p.M.ptr[r0 + r] - e0;
        re = p.M.ptr[r0 + r + 1] - e0;
        if (lane == 0) load_ops<V, DIR>(p, r0 + r, ops, ib);
    }
    tile_products<V, V, FMT, NT, EPT>(p.M, p.gvec, e0, R.e1, w, a, at, prod);
    __syncthreads();
    for (; r < nrows; r += groups) {
        V s = 0;
        for (int q = rb + lane; q < re; q += L) s += prod[q];
        if (L > 1) s = wave_sum_width(s, L);
        if (lane == 0) apply_ops<V, DIR>(p, r0 + r, s, step, copy_ref, ops, ip, acnt);
        const int rn = r + groups;
        if (rn < nrows) {
            rb = p.M.ptr[r0 + rn] - e0;
            re = p.M.ptr[r0 + rn + 1] - e0;
            if (lane == 0) load_ops<V, DIR>(p, r0 + rn, ops, ib);
        }
    }
    if (p.adapt) {
        block_sum2<NT>(ip[0], ip[1], red2);
        if (tid == 0) {
            p.ipart[2 * t] = ip[0];
            p.ipart[2 * t + 1] = ip[1];
        }
    }
}

template <class V, int FMT, int DIR, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_pass(const PassArgs<V> p, const int jw)
{
    pass_tile<V, FMT, DIR, NT, EPT, true>(p, jw);
}

// The same over a batch (entries loaded once the instance is known to run).
template <class V, int FMT, int DIR, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_pass_batch(const PassArgs<V> p, const int jw)
{
    pass_tile<V, FMT, DIR, NT, EPT, false>(p, jw);
}

// ------------------------------------------------------- sorted tiles
// One workgroup per normal tile: its entries in the order of the index they
// gather (bitonic sort in LDS of index and place), so that the lanes of a
// wave gather from the same or neighbouring cache lines.  Random gathers are
// bound by the requests that the L2s take, one a nonzero; in a tile of 8192
// entries over a vector of 1 MB two lanes share a 128-byte line, over 100 KB
// ten.  The products still go to their place in row order, so every sum is
// what it is without sorting, bit for bit.  Measured, both passes of an
// iteration: 64 uneven LPs (9M nonzeros, vectors of 4-400 KB) 72 -> 43 us, a
// skewed LP of 9.4M (column pass over 1 MB) 85 -> 71 us, 64 20k x 40k
// instances (row pass) 109 -> 81 us; the 1M x 2M LP's columns (4 MB) 119 -> 116
// us; nothing at 2M nonzeros in FP64 (40 us), a loss where long rows cut
// into segments keep most of the chip busy only in small tiles.
template <int FMT>
__global__ __launch_bounds__(1024) void k_sort_tiles(const MatView M, const int4 *tiles, int cap, uint32_t *ent,
                                                     void *val, uint16_t *pos)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    unsigned long long *key = reinterpret_cast<unsigned long long *>(lds_raw);  // [cap], a power of two
    const TileRange R = tile_range(tiles[blockIdx.x]);
    const int n = R.e1 - R.e0;
    for (int i = threadIdx.x; i < cap; i += 1024) {
        unsigned long long k = ~0ull;
        if (i < n) {
            uint32_t w = M.ent[R.e0 + i];
            if constexpr (FMT == FMT_PACKED) w &= M.mask;
            k = (unsigned long long)w << 16 | (unsigned)i;
        }
        key[i] = k;
    }
    for (int size = 2; size <= cap; size <<= 1)
        for (int step = size >> 1; step > 0; step >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < cap / 2; t += 1024) {
                const int lo = 2 * t - (t & (step - 1)), hi = lo + step;
                const unsigned long long a = key[lo], b = key[hi];
                if ((a > b) == ((lo & size) == 0)) {
                    key[lo] = b;
                    key[hi] = a;
                }
            }
        }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 1024) {
        const int p = (int)(key[i] & 0xffff);
        ent[R.e0 + i] = M.ent[R.e0 + p];
        pos[R.e0 + i] = (uint16_t)p;
        if constexpr (FMT == FMT_F64) ((double *)val)[R.e0 + i] = ((const double *)M.val)[R.e0 + p];
    }
}

// ------------------------------------------- gather-blocked pass (partials)
// Tile of block b (bits 24.. of T.z) of a gather-blocked orientation: row
// sums over the block's nonzeros go to P[b * rows + i] (A = V for the
// iteration, double for the check); long sub-rows go to segment slots.
template <class V, class A, int FMT, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_bpart(const PassArgs<V> p, const int jw, const int check)
{
    constexpr int CH = NT * EPT;
    __shared__ A prod[CH];
    __shared__ A red[NT / 64];
    const int4 T = p.tiles[blockIdx.x];
    const int inst = T.z & 0xffffff, b = T.z >> 24;
    const InstState &S = p.st[inst];
    if (S.status != ST_RUN || (!check && jw >= S.nrun)) return;
    const int tid = threadIdx.x;
    A *P = (A *)(check ? (void *)p.P64 : (void *)p.P);
    if (T.w >= 0) {
        stage_products<A, V, FMT, NT, EPT>(p.M, p.gvec, T.x, T.y, prod);
        __syncthreads();
        A s = 0;
        for (int q = tid; q < T.y - T.x; q += NT) s += prod[q];
        s = block_sum<A, NT>(s, red);
        A *seg = (A *)(check ? (void *)p.seg64 : (void *)p.seg);
        if (tid == 0) seg[T.w] = s;
        return;
    }
    const int32_t *ptr = p.bptr + (size_t)b * (p.rows + 1);
    const int r0 = T.x, nrows = T.y - T.x;
    const int e0 = ptr[r0], e1 = ptr[T.y];
    const int L = lanes_per_row<NT>(nrows);
    const int groups = NT / L, lane = tid & (L - 1);
    int r = tid / L;
    int rb = 0, re = 0;
    if (r < nrows) {
        rb = ptr[r0 + r] - e0;
        re = ptr[r0 + r + 1] - e0;
    }
    stage_products<A, V, FMT, NT, EPT>(p.M, p.gvec, e0, e1, prod);
    __syncthreads();
    A *Pb = P + (size_t)b * p.rows;
    for (; r < nrows; r += groups) {
        A s = 0;
        for (int q = rb + lane; q < re; q += L) s += prod[q];
        if (L > 1) s = wave_sum_width(s, L);
        if (lane == 0) Pb[r0 + r] = s;
        const int rn = r + groups;
        if (rn < nrows) {
            rb = ptr[r0 + rn] - e0;
            re = ptr[r0 + rn + 1] - e0;
        }
    }
}

// Combine of a blocked orientation (one thread per row, 256 rows of one
// instance per workgroup): sum the B block partials in block order, then the
// fused epilogue.
template <class V, int DIR>
__global__ __launch_bounds__(256) void k_bcombine(const PassArgs<V> p, const int jw)
{
    __shared__ double red2[8];
    const int4 T = p.ctiles[blockIdx.x];
    const InstState &S = p.st[T.z];
    if (S.status != ST_RUN || jw >= S.nrun) return;
    const int i = T.x + threadIdx.x;
    const InstBounds<V> ib = inst_bounds<V, DIR>(p, T.z);
    double ip[2] = {0.0, 0.0};
    if (i < T.y) {
        const bool copy_ref = (jw == 0) && (S.restart_now != 0);
        RowOps<V> ops;
        load_ops<V, DIR>(p, i, ops, ib);
        V s = 0;
        const int nb = p.bq ? p.bq[T.z] : p.B;
        for (int b = 0; b < nb; ++b) s += p.P[(size_t)b * p.rows + i];
        apply_ops<V, DIR>(p, i, s, DIR == DIR_COL ? (V)S.t : (V)S.s, copy_ref, ops, ip, avg_count(p, S, jw));
    }
    if (p.adapt) {
        block_sum2<256>(ip[0], ip[1], red2);
        if (threadIdx.x == 0) {
            p.ipart[2 * blockIdx.x] = ip[0];
            p.ipart[2 * blockIdx.x + 1] = ip[1];
        }
    }
}

// ------------------------------------------- LDS-staged pass (small instances)
// When an instance's whole gathered vector fits in LDS, one workgroup copies
// it there once and then walks a run of sub-tiles of that instance (whole
// rows, <= NT*EPT nonzeros each): every gather is an LDS read.  The loop is
// software-pipelined: the coalesced loads of sub-tile t+1's nonzeros are in
// flight while sub-tile t's rows are reduced and updated.
// Workgroup barrier that orders LDS accesses only: global loads issued
// before it stay in flight (__syncthreads also waits for them, which would
// serialise the prefetch of the next sub-tile with the current one).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Copies src[0, n) into LDS by NT threads in 16-byte words, U in flight per
// thread (a plain strided loop would wait for each load before its LDS
// store).  The copy starts at `base` (16-byte aligned LDS) shifted by the
// source's misalignment, so that every word is aligned on both sides, and
// the copied vector begins at the returned pointer (dst[k] = src[k], k < n;
// base needs n values + LDS_COPY_SLACK bytes).
// The words may start up to 12 bytes before src, inside the same buffer
// (device buffers are 256-byte aligned); the tail is copied value by value.
template <int NT, int U, class V>
__device__ __forceinline__ V *copy_to_lds_vec(V *base, const V *__restrict__ src, int n)
{
    constexpr int W = 16 / sizeof(V);
    typedef V VW __attribute__((ext_vector_type(W)));
    const int mis = (int)(((uintptr_t)src & 15) / sizeof(V));
    const V *asrc = src - mis;
    const int words = (mis + n) / W;
    const int tid = threadIdx.x;
    for (int k0 = 0; k0 < words; k0 += NT * U) {
        VW t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * NT + tid;
            if (k < words) t[u] = reinterpret_cast<const VW *>(asrc)[k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * NT + tid;
            if (k < words) reinterpret_cast<VW *>(base)[k] = t[u];
        }
    }
    for (int k = words * W + tid; k < mis + n; k += NT) base[k] = asrc[k];
    return base + mis;
}

template <class V, int FMT, int NT, int EPT>
__device__ __forceinline__ void spass_load(const MatView &M, int e0, int e1, uint32_t (&w)[EPT], V (&a)[EPT])
{
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = e0 + q * NT + (int)threadIdx.x;
        w[q] = 0;
        a[q] = (V)0;
        if (e < e1) load_entry<FMT, V>(M, e, w[q], a[q]);
    }
}

template <class V, int FMT, int DIR, int NT, int EPT, bool PF>
__global__ __launch_bounds__(NT) void k_spass(const PassArgs<V> p, const int jw)
{
    constexpr int CH = NT * EPT;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    V *prod = reinterpret_cast<V *>(lds_raw);  // [CH]
    V *sv = prod + CH;                         // [gathered length]
    const int4 T = p.tiles[xcd_tile(blockIdx.x, gridDim.x)];  // {sub0, sub1, inst | slice << 24, kind}
    // kind -1: a whole instance's gathered vector in LDS, fused epilogue;
    // kind -2: one slice of it, partial sums to xP (added by the combine)
    const bool part = T.w == -2;
    const int inst = T.z & 0xffffff, sl = T.z >> 24;
    const InstState &S = p.st[inst];
    if (S.status != ST_RUN || jw >= S.nrun) return;
    const bool copy_ref = (jw == 0) && (S.restart_now != 0);
    const V step = DIR == DIR_COL ? (V)S.t : (V)S.s;
    const V acnt = avg_count(p, S, jw);
    const int tid = threadIdx.x;
    const InstBounds<V> ib = inst_bounds<V, DIR>(p, inst);
    MatView M = p.M;
    const int4 *sub = p.sub;
    int g0 = p.gofs[inst], glen = p.gofs[inst + 1] - g0;
    V *Ps = nullptr;
    if (part) {
        M = p.X;
        M.ptr = p.X.ptr + (size_t)sl * (p.rows + 1);
        sub = p.xsub;
        const int Sq = p.xSq[inst];
        const int lo = (int)(((int64_t)glen * sl) / Sq), hi = (int)(((int64_t)glen * (sl + 1)) / Sq);
        g0 += lo;
        glen = hi - lo;
        Ps = p.xP + (size_t)sl * p.rows;
    }
    double ip[2] = {0.0, 0.0};
    // Descriptors of the first SPASS_DMAX sub-tiles (first row, end row,
    // first and end nonzero) go to LDS with the vector, so that starting
    // the next sub-tile's loads needs no dependent global reads.
    __shared__ int sdesc[4][SPASS_DMAX];
    for (int u = tid; u < T.y - T.x && u < SPASS_DMAX; u += NT) {
        const int4 d = sub[T.x + u];
        sdesc[0][u] = d.x;
        sdesc[1][u] = d.y;
        sdesc[2][u] = M.ptr[d.x];
        sdesc[3][u] = M.ptr[d.y];
    }
    // sub-tile state (nonzeros in registers one sub-tile ahead; with PF also
    // this thread's first row bounds and epilogue operands)
    int4 D = sub[T.x];
    int e0 = M.ptr[D.x], e1 = M.ptr[D.y];
    uint32_t w[EPT];
    V a[EPT];
    spass_load<V, FMT, NT, EPT>(M, e0, e1, w, a);
    int L = 1, r = 0, rb = 0, re = 0;
    RowOps<V> ops;
    if (PF) {
        L = lanes_per_row<NT>(D.y - D.x);
        r = tid / L;
        if (r < D.y - D.x) {
            rb = M.ptr[D.x + r] - e0;
            re = M.ptr[D.x + r + 1] - e0;
            if (!part && (tid & (L - 1)) == 0) load_ops<V, DIR>(p, D.x + r, ops, ib);
        }
    }
    sv = copy_to_lds_vec<NT, 8>(sv, p.gvec + g0, glen);
    lds_barrier();
    for (int t = T.x; t < T.y; ++t) {
        // products of sub-tile t from the registers
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            const int e = e0 + q * NT + tid;
            if (e < e1) {
                const int idx = decode_entry<FMT, V>(M, w[q], a[q]);
                prod[e - e0] = a[q] * sv[idx - g0];
            }
        }
        const int r0c = D.x, nrows = D.y - D.x, e0c = e0;
        int Lc, rc, rbc, rec;
        RowOps<V> opc;
        if (PF) {
            Lc = L;
            rc = r;
            rbc = rb;
            rec = re;
            opc = ops;
        } else {
            Lc = lanes_per_row<NT>(nrows);
            rc = tid / Lc;
            rbc = rec = 0;
            if (rc < nrows) {
                rbc = M.ptr[r0c + rc] - e0c;
                rec = M.ptr[r0c + rc + 1] - e0c;
                if (!part && (tid & (Lc - 1)) == 0) load_ops<V, DIR>(p, r0c + rc, opc, ib);
            }
        }
        lds_barrier();
        // sub-tile t+1's nonzeros (and with PF its row bounds and operands)
        // are in flight during this reduction
        if (t + 1 < T.y) {
            const int u = t + 1 - T.x;
            if (u < SPASS_DMAX) {
                D.x = sdesc[0][u];
                D.y = sdesc[1][u];
                e0 = sdesc[2][u];
                e1 = sdesc[3][u];
            } else {
                D = sub[t + 1];
                e0 = M.ptr[D.x];
                e1 = M.ptr[D.y];
            }
            spass_load<V, FMT, NT, EPT>(M, e0, e1, w, a);
            if (PF) {
                L = lanes_per_row<NT>(D.y - D.x);
                r = tid / L;
                if (r < D.y - D.x) {
                    rb = M.ptr[D.x + r] - e0;
                    re = M.ptr[D.x + r + 1] - e0;
                    if (!part && (tid & (L - 1)) == 0) load_ops<V, DIR>(p, D.x + r, ops, ib);
                }
            }
        }
        const int groups = NT / Lc, lane = tid & (Lc - 1);
        for (; rc < nrows; rc += groups) {
            V sum = 0;
            for (int q = rbc + lane; q < rec; q += Lc) sum += prod[q];
            if (Lc > 1) sum = wave_sum_width(sum, Lc);
            if (lane == 0) {
                if (part) Ps[r0c + rc] = sum;
                else apply_ops<V, DIR>(p, r0c + rc, sum, step, copy_ref, opc, ip, acnt);
            }
            const int rn = rc + groups;
            if (rn < nrows) {
                rbc = M.ptr[r0c + rn] - e0c;
                rec = M.ptr[r0c + rn + 1] - e0c;
                if (!part && lane == 0) load_ops<V, DIR>(p, r0c + rn, opc, ib);
            }
        }
        lds_barrier();
    }
    if (p.adapt && !part) {
        // the product buffer is free after the last barrier
        block_sum2<NT>(ip[0], ip[1], reinterpret_cast<double *>(lds_raw));
        if (tid == 0) {
            const int t = xcd_tile(blockIdx.x, gridDim.x);
            p.ipart[2 * t] = ip[0];
            p.ipart[2 * t + 1] = ip[1];
        }
    }
}

// ------------------------------------------ direct LDS-staged pass
// For instances whose whole gathered vector fits in LDS with nothing beside
// it: a workgroup copies the instance's vector to LDS once, then each group
// of L lanes reduces whole rows straight from their nonzeros (streamed from
// global memory, gathered from LDS), DPASS_R rows at a time, combines its
// lanes with shuffles and applies the fused epilogue; each lane takes K
// nonzeros of a row per round (K = 16 / L for the plan's lanes per row L,
// between 2 and 8, so a row of up to 16 nonzeros is one round).  The row bounds of
// the next DPASS_R rows load while the current ones are reduced, so each
// step waits for one round trip (the nonzeros).  Without a product buffer
// the vector may fill the LDS.  Tile {r0, r1, inst, L}; within a row each
// lane adds its nonzeros in order and the lanes combine in a fixed tree, so
// the result is reproducible for a given plan.
constexpr int DPASS_R = 4;

template <class V, int FMT, int K>
__device__ __forceinline__ V direct_row_chunk(const MatView &M, const V *sv, int g0, int e, int e1, int L)
{
    uint32_t w[K];
    V a[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int ee = e + k * L;
        w[k] = 0;
        a[k] = (V)0;
        if (ee < e1) load_entry<FMT, V>(M, ee, w[k], a[k]);
    }
    V s = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (e + k * L < e1) {
            const int idx = decode_entry<FMT, V>(M, w[k], a[k]);
            s += a[k] * sv[idx - g0];
        }
    }
    return s;
}

template <class V, int FMT, int DIR, int NT, int K>
__global__ __launch_bounds__(NT) void k_dpass(const PassArgs<V> p, const int jw)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ double red2[2 * NT / 64];
    V *sv = reinterpret_cast<V *>(lds_raw);
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int4 T = p.dtiles[t];
    const InstState &S = p.st[T.z];
    if (S.status != ST_RUN || jw >= S.nrun) return;
    const bool copy_ref = (jw == 0) && (S.restart_now != 0);
    const V step = DIR == DIR_COL ? (V)S.t : (V)S.s;
    const V acnt = avg_count(p, S, jw);
    const InstBounds<V> ib = inst_bounds<V, DIR>(p, T.z);
    const int tid = threadIdx.x, L = T.w, lane = tid & (L - 1), groups = NT / L;
    const int g0 = p.gofs[T.z], glen = p.gofs[T.z + 1] - g0;
    // bounds of this lane group's first DPASS_R rows, then the vector copy
    int nb0[DPASS_R], nb1[DPASS_R];
    const int first = T.x + tid / L;
#pragma unroll
    for (int u = 0; u < DPASS_R; ++u) {
        const int r = first + u * groups;
        nb0[u] = nb1[u] = 0;
        if (r < T.y) {
            nb0[u] = p.M.ptr[r];
            nb1[u] = p.M.ptr[r + 1];
        }
    }
    sv = copy_to_lds_vec<NT, 8>(sv, p.gvec + g0, glen);
    lds_barrier();
    double ip[2] = {0.0, 0.0};
    for (int base = first; base < T.y; base += DPASS_R * groups) {
        int b0[DPASS_R], b1[DPASS_R];
#pragma unroll
        for (int u = 0; u < DPASS_R; ++u) {
            b0[u] = nb0[u];
            b1[u] = nb1[u];
        }
        // nonzeros of the current rows (first K per lane of each)
        uint32_t w[DPASS_R][K];
        V a[DPASS_R][K];
#pragma unroll
        for (int u = 0; u < DPASS_R; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int e = b0[u] + lane + k * L;
                w[u][k] = 0;
                a[u][k] = (V)0;
                if (e < b1[u]) load_entry<FMT, V>(p.M, e, w[u][k], a[u][k]);
            }
        RowOps<V> ops[DPASS_R];
        if (lane == 0) {
#pragma unroll
            for (int u = 0; u < DPASS_R; ++u)
                if (base + u * groups < T.y) load_ops<V, DIR>(p, base + u * groups, ops[u], ib);
        }
        // bounds of the next rows load meanwhile
#pragma unroll
        for (int u = 0; u < DPASS_R; ++u) {
            const int r = base + (DPASS_R + u) * groups;
            nb0[u] = nb1[u] = 0;
            if (r < T.y) {
                nb0[u] = p.M.ptr[r];
                nb1[u] = p.M.ptr[r + 1];
            }
        }
#pragma unroll
        for (int u = 0; u < DPASS_R; ++u) {
            V sum = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (b0[u] + lane + k * L < b1[u]) {
                    const int idx = decode_entry<FMT, V>(p.M, w[u][k], a[u][k]);
                    sum += a[u][k] * sv[idx - g0];
                }
            }
            // rows longer than K per lane: further rounds
            for (int c = lane + K * L; b0[u] + c < b1[u]; c += K * L)
                sum += direct_row_chunk<V, FMT, K>(p.M, sv, g0, b0[u] + c, b1[u], L);
            if (L > 1) sum = wave_sum_width(sum, L);
            const int r = base + u * groups;
            if (lane == 0 && r < T.y) apply_ops<V, DIR>(p, r, sum, step, copy_ref, ops[u], ip, acnt);
        }
    }
    if (p.adapt) {
        block_sum2<NT>(ip[0], ip[1], red2);
        if (tid == 0) {
            p.ipart[2 * t] = ip[0];
            p.ipart[2 * t + 1] = ip[1];
        }
    }
}

// Sum of a long row's n segment partials, COMB_L lanes (in every lane): a row
// of 25k nonzeros has 49 segments, read one after another by one thread they
// took 7.8 us of a skewed 9.4M-nonzero LP's 92 us iteration.
constexpr int COMB_L = 16, COMB_ROWS = 256 / COMB_L;

template <class A>
__device__ __forceinline__ A segment_sum(const A *seg, int n)
{
    A s = 0;
    for (int k = threadIdx.x & (COMB_L - 1); k < n; k += COMB_L) s += seg[k];
    return group_sum(s, COMB_L);
}

// Long sub-rows of a blocked orientation: P[b][row] = sum of its segments.
template <class V, class A>
__global__ __launch_bounds__(256) void k_bseg(const PassArgs<V> p, const int jw, const int check)
{
    const int q = blockIdx.x * COMB_ROWS + threadIdx.x / COMB_L;
    if (q >= p.nlong) return;
    const int4 L = p.longs[q];
    const int inst = L.w & 0xffffff, b = L.w >> 24;
    const InstState &S = p.st[inst];
    if (S.status != ST_RUN || (!check && jw >= S.nrun)) return;
    const A *seg = (const A *)(check ? (const void *)p.seg64 : (const void *)p.seg);
    const A s = segment_sum(seg + L.y, L.z);
    if ((threadIdx.x & (COMB_L - 1)) != 0) return;
    A *P = (A *)(check ? (void *)p.P64 : (void *)p.P);
    P[(size_t)b * p.rows + L.x] = s;
}

// Long rows: add the segment partials, then the epilogue.
template <class V, int DIR>
__global__ __launch_bounds__(256) void k_combine(const PassArgs<V> p, const int jw)
{
    const int q = blockIdx.x * COMB_ROWS + threadIdx.x / COMB_L;
    if (q >= p.nlong) return;
    const int4 L = p.longs[q];
    const InstState &S = p.st[L.w];
    if (S.status != ST_RUN || jw >= S.nrun) return;
    const bool copy_ref = (jw == 0) && (S.restart_now != 0);
    const InstBounds<V> ib = inst_bounds<V, DIR>(p, L.w);
    const V s = segment_sum(p.seg + L.y, L.z);
    if ((threadIdx.x & (COMB_L - 1)) != 0) return;
    RowOps<V> ops;
    load_ops<V, DIR>(p, L.x, ops, ib);
    double ip[2] = {0.0, 0.0};
    apply_ops<V, DIR>(p, L.x, s, DIR == DIR_COL ? (V)S.t : (V)S.s, copy_ref, ops, ip, avg_count(p, S, jw));
    if (p.adapt) {
        p.iplong[2 * q] = ip[0];
        p.iplong[2 * q + 1] = ip[1];
    }
}

// ------------------------------------------------------------ KKT check
// Per-row / per-column FP64 contributions (Section 2.2, original problem).
//   row i : q0 = r_p,i^2, q1 = b_i y_i, q2 = ((y_i - yr_i) / d_r,i)^2
//   col j : q0 = r_d,j^2, q1 = c_j x_j, q2 = l_j max(lam_j,0) + u_j min(lam_j,0),
//           q3 = ((x_j - xr_j) / d_c,j)^2
template <class V>
__device__ __forceinline__ void row_terms(const PassArgs<V> &p, int i, double ax, double q[CHK])
{
    const double b = p.rhs64[i];
    const uint8_t sn = p.sense[i];
    double r;
    if (sn == 'G') r = fmax(b - ax, 0.0);
    else if (sn == 'L') r = fmax(ax - b, 0.0);
    else r = b - ax;
    const double y = (double)p.own[i];
    const double dy = (y - (double)p.own_ref[i]) / p.d64[i];
    q[0] += r * r;
    q[1] += b * y;
    q[2] += dy * dy;
    // moves since the previous check: v = y - y_prev, A d = A x - (A x)_prev
    // (the check of the running average has none)
    if (!p.own_prev) return;
    const double v = y - (double)p.own_prev[i];
    const double vp = sn == 'G' ? fmax(v, 0.0) : (sn == 'L' ? fmin(v, 0.0) : v);
    const double ad = ax - p.prod_prev[i];
    const double viol = sn == 'G' ? fmax(-ad, 0.0) : (sn == 'L' ? fmax(ad, 0.0) : ad);
    q[4] += b * v;
    q[5] += (v - vp) * (v - vp);
    q[6] += viol * viol;
    p.own_prev[i] = p.own[i];
    p.prod_prev[i] = ax;
}

template <class V>
__device__ __forceinline__ void col_terms(const PassArgs<V> &p, int j, double aty, double q[CHK])
{
    // with a diagonal Hessian: reduced cost c + Q x - A^T y, primal objective
    // + x^T Q x / 2, dual objective - x^T Q x / 2 (kept with the bound terms)
    const double x = (double)p.own[j];
    const double qx = p.q64 ? p.q64[j] * x : 0.0;
    const double g = p.rhs64[j] + qx - aty;
    const double l = p.lo64[j], u = p.hi64[j];
    const bool lf = isfinite(l), uf = isfinite(u);
    double lam;
    if (lf && uf) lam = g;
    else if (lf) lam = fmax(g, 0.0);
    else if (uf) lam = fmin(g, 0.0);
    else lam = 0.0;
    const double rd = g - lam;
    const double dx = (x - (double)p.own_ref[j]) / p.d64[j];
    q[0] += rd * rd;
    q[1] += p.rhs64[j] * x + 0.5 * qx * x;
    if (lf && lam > 0.0) q[2] += l * lam;
    if (uf && lam < 0.0) q[2] += u * lam;
    q[2] -= 0.5 * qx * x;
    q[3] += dx * dx;
    // moves since the previous check: A^T v = A^T y - (A^T y)_prev, d = x - x_prev
    // (the check of the running average has none)
    if (!p.own_prev) return;
    const double w = aty - p.prod_prev[j];
    double rl;
    if (lf && uf) rl = -w;
    else if (lf) rl = fmax(-w, 0.0);
    else if (uf) rl = fmin(-w, 0.0);
    else rl = 0.0;
    q[4] += (w + rl) * (w + rl);
    if (lf && rl > 0.0) q[5] += l * rl;
    if (uf && rl < 0.0) q[5] += u * rl;
    const double d = x - (double)p.own_prev[j];
    q[6] += p.rhs64[j] * d;
    double bv;
    if (lf && uf) bv = d;
    else if (lf) bv = fmin(d, 0.0);
    else if (uf) bv = fmax(d, 0.0);
    else bv = 0.0;
    q[7] += bv * bv;
    if (p.q64) q[7] += (p.q64[j] * d) * (p.q64[j] * d);
    p.own_prev[j] = p.own[j];
    p.prod_prev[j] = aty;
}

template <class V, int FMT, int DIR, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_check(const PassArgs<V> p)
{
    constexpr int CH = NT * EPT;
    __shared__ double prod[CH];
    __shared__ double red[NT / 64 * CHK];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int4 T = p.tiles[t];
    const InstState &S = p.st[T.z];
    if (S.status != ST_RUN) return;
    const TileRange R = tile_range(T);
    const int e0 = R.e0, e1 = R.e1;
    // row check gathers x (not x_bar), column check gathers y
    stage_products<double, V, FMT, NT, EPT>(p.M, p.gvec, e0, e1, prod);
    __syncthreads();
    const int tid = threadIdx.x;
    if (T.w >= 0) {
        // a segment's row terms are added once by the combine kernel; its own
        // tile slot contributes nothing
        double s = 0;
        for (int q = tid; q < e1 - e0; q += NT) s += prod[q];
        s = block_sum<double, NT>(s, red);
        if (tid == 0) {
            p.seg64[T.w] = s;
            for (int k = 0; k < CHK; ++k) p.part[CHK * t + k] = 0.0;
        }
        return;
    }
    const int r0 = T.x, nrows = R.rows;
    int L = 1;
    while (L < 64 && nrows * (L << 1) <= NT) L <<= 1;
    const int groups = NT / L, lane = tid & (L - 1);
    double q[CHK] = {};
    for (int r = tid / L; r < nrows; r += groups) {
        const int rb = p.M.ptr[r0 + r] - e0, re = p.M.ptr[r0 + r + 1] - e0;
        double s = 0;
        for (int k = rb + lane; k < re; k += L) s += prod[k];
        if (L > 1) s = wave_sum_width(s, L);
        if (lane == 0) {
            if (DIR == DIR_COL) {
                col_terms(p, r0 + r, s, q);
            } else {
                row_terms(p, r0 + r, s, q);
                if (p.adapt) p.ax[r0 + r] = s;  // A x of the current point (FP64)
            }
        }
    }
    block_sums<NT, CHK>(q, red, p.part + CHK * (size_t)t);
}

template <class V, int DIR>
__global__ __launch_bounds__(256) void k_combine_check(const PassArgs<V> p)
{
    const int qi = blockIdx.x * COMB_ROWS + threadIdx.x / COMB_L;
    if (qi >= p.nlong) return;
    const int4 L = p.longs[qi];
    const InstState &S = p.st[L.w];
    if (S.status != ST_RUN) return;
    const double s = segment_sum(p.seg64 + L.y, L.z);
    if ((threadIdx.x & (COMB_L - 1)) != 0) return;
    double q[CHK] = {};
    if (DIR == DIR_COL) {
        col_terms(p, L.x, s, q);
    } else {
        row_terms(p, L.x, s, q);
        if (p.adapt) p.ax[L.x] = s;
    }
    for (int k = 0; k < CHK; ++k) p.lpart[CHK * qi + k] = q[k];
}

// Check combine of a blocked orientation: FP64 row sums from the block
// partials, row / column KKT terms, fixed-order sum per combine tile.
template <class V, int DIR>
__global__ __launch_bounds__(256) void k_bcombine_check(const PassArgs<V> p)
{
    __shared__ double red[4 * CHK];
    const int ct = blockIdx.x;
    const int4 T = p.ctiles[ct];
    const InstState &S = p.st[T.z];
    if (S.status != ST_RUN) return;
    const int i = T.x + threadIdx.x;
    double q[CHK] = {};
    if (i < T.y) {
        double s = 0;
        for (int b = 0; b < p.B; ++b) s += p.P64[(size_t)b * p.rows + i];
        if (DIR == DIR_COL) {
            col_terms(p, i, s, q);
        } else {
            row_terms(p, i, s, q);
            if (p.adapt) p.ax[i] = s;
        }
    }
    block_sums<256, CHK>(q, red, p.part + CHK * (size_t)ct);
}

// ------------------------------------------------------------- decision
// Termination test (Section 2.2), infeasibility certificates, restart rule
// and primal-weight update in FP64 for one instance, from the check window's
// reduced sums tot = {||r_p||^2, b^T y, ||dy~||^2, ||r_d||^2, c^T x, bound
// terms, ||dx~||^2, b^T v, |v - proj_Y v|^2, |row violation of A d|^2,
// |A^T v + lam|^2, ray bound terms, c^T d, |bound violation of d|^2}.
constexpr int NTOT = 14;

// Relative KKT error of a check's totals (Section 2.2): rho_p, rho_d,
// rho_g, P, D and E = max of the three (NaN when one is not finite).
struct Kkt {
    double rho_p, rho_d, rho_g, P, D, E;
};

__device__ __forceinline__ Kkt kkt_of(const InstState &S, const double tot[NTOT])
{
    Kkt r;
    r.rho_p = sqrt(tot[0]) / (1.0 + S.bnorm);
    r.rho_d = sqrt(tot[3]) / (1.0 + S.cnorm);
    r.P = tot[4];
    r.D = tot[1] + tot[5];
    r.rho_g = fabs(r.P - r.D) / (1.0 + fabs(r.P) + fabs(r.D));
    r.E = fmax(r.rho_p, fmax(r.rho_d, r.rho_g));
    if (!isfinite(r.rho_p) || !isfinite(r.rho_d) || !isfinite(r.rho_g)) r.E = NAN;
    return r;
}

// The decision at a check.  totA: the totals of the running average
// (restart to the average), or null.  The candidate is the average when
// its error is below the current iterate's; its error drives termination,
// the restart rule and E_prev, a restart or an OPTIMAL / iteration-limit
// stop takes it (take_avg), and infeasibility and stalling look at the
// current iterate.
__device__ void decide_state(InstState &S, const double tot[NTOT], const double *totA, int R)
{
    const int64_t k = S.k + S.nrun;
    S.k = k;
    S.nrun = 0;
    S.restart_now = 0;
    S.take_avg = 0;
    const Kkt cur = kkt_of(S, tot);
    if (!isfinite(cur.E)) {
        S.rho_p = cur.rho_p;
        S.rho_d = cur.rho_d;
        S.rho_g = cur.rho_g;
        S.pobj = cur.P;
        S.dobj = cur.D;
        S.rel = cur.E;
        S.status = ST_NUM;
        return;
    }
    // the average exists once an iterate was produced since the last restart
    bool use_avg = false;
    Kkt avg = cur;
    if (totA && S.avg_on && k > S.kr) {
        avg = kkt_of(S, totA);
        use_avg = avg.E < cur.E;
    }
    const Kkt &c = use_avg ? avg : cur;
    const double E = c.E;
    S.rho_p = c.rho_p;
    S.rho_d = c.rho_d;
    S.rho_g = c.rho_g;
    S.pobj = c.P;
    S.dobj = c.D;
    S.rel = E;
    if (E <= S.tol) {
        S.take_avg = use_avg;
        S.status = ST_OPT;
        return;
    }
    if (S.infeas_tol > 0.0 && k > 0) {
        // a dual ray certifies primal infeasibility, a primal ray dual
        // infeasibility (moves since the previous check)
        const double rho = tot[7] + tot[11], rres = sqrt(tot[8] + tot[10]);
        if (rho > 0.0 && rres <= S.infeas_tol * rho) { S.status = ST_PINF; return; }
        const double cd = tot[12], pviol = sqrt(tot[9] + tot[13]);
        if (cd < 0.0 && pviol <= -S.infeas_tol * cd) { S.status = ST_DINF; return; }
    }
    if (S.stall_tol > 0.0) {
        // bounds stalling (Algorithm 1's inner-loop exit): neither objective
        // bound of the current iterate moved by more than stall_tol
        // (1 + |value|) since the previous check, stall_checks times in a row
        if (k > 0) {
            const bool moved = fabs(cur.P - S.pprev) > S.stall_tol * (1.0 + fabs(cur.P)) ||
                               fabs(cur.D - S.dprev) > S.stall_tol * (1.0 + fabs(cur.D));
            S.nstall = moved ? 0 : S.nstall + 1;
            if (S.nstall >= S.stall_checks) { S.status = ST_STALL; return; }
        }
        S.pprev = cur.P;
        S.dprev = cur.D;
    }
    if (k >= S.k_limit) {
        S.take_avg = use_avg;
        S.status = ST_ITER;
        return;
    }
    if (S.force_stop) { S.status = ST_TIME; return; }
    if (k == 0) {
        S.Er = E;
        S.kr = 0;
        S.restart_now = 1;
    } else if (S.restart_on) {
        const bool fire = (E <= 0.2 * S.Er) || (E <= 0.8 * S.Er && E > S.Ep) ||
                          ((double)(k - S.kr) >= 0.36 * (double)k);
        if (fire) {
            // distances of the candidate to the last restart point
            const double *tc = use_avg ? totA : tot;
            const double dx = sqrt(tc[6]), dy = sqrt(tc[2]);
            if (dx > 1e-10 && dy > 1e-10) {
                S.omega = exp(0.5 * log(dy / dx) + 0.5 * log(S.omega));
                S.t = S.eta / S.omega;
                S.s = S.eta * S.omega;
            }
            S.Er = E;
            S.kr = k;
            S.restarts += 1;
            S.restart_now = 1;
            S.take_avg = use_avg;
        }
    }
    S.Ep = E;
    const int64_t left = S.k_limit - k;
    S.nrun = (int32_t)(left < (int64_t)R ? left : (int64_t)R);
}


// One workgroup per instance: fixed-order FP64 reduction of the check
// partials, then termination (Section 2.2), restart and primal-weight
// update, all in FP64.  Bound by latency: the partials of a large LP's 10-25k
// tiles an orientation are read by one compute unit, so 1024 threads take
// DECIDE_U tiles each at a time, and the sums share their barriers (256
// threads, one tile after another and two barriers a sum: 28 us for the
// 1M x 2M LP, 48 us for a skewed one of 9.4M nonzeros, 14 us for a 5k x 10k
// one with the averages).
constexpr int DECIDE_NT = 1024, DECIDE_U = 4;

// Adds the N partials of the slots [lo, hi) whose index in a slot starts at
// from.
template <int N>
__device__ __forceinline__ void decide_add(const double *part, int lo, int hi, int from, double *acc)
{
    for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += DECIDE_NT * DECIDE_U) {
        double v[DECIDE_U][N];
#pragma unroll
        for (int u = 0; u < DECIDE_U; ++u) {
            const int t = t0 + u * DECIDE_NT;
#pragma unroll
            for (int k = 0; k < N; ++k) v[u][k] = t < hi ? part[CHK * (size_t)t + from + k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < DECIDE_U; ++u)
#pragma unroll
            for (int k = 0; k < N; ++k) acc[k] += v[u][k];
    }
}

// tot layout as in decide_state: rows {0, 1, 2} and {7, 8, 9}, columns
// {3, 4, 5, 6} and {10, 11, 12, 13}.
__device__ __forceinline__ void decide_totals(const InstInfo &I, const double *rpart, const double *lrpart,
                                              const double *cpart, const double *lcpart, double *red, double *tot)
{
    double acc[NTOT] = {};
    for (int half = 0; half < 2; ++half) {
        double r[3] = {}, c[4] = {};
        decide_add<3>(rpart, I.rt0, I.rt1, 4 * half, r);
        decide_add<3>(lrpart, I.lr0, I.lr1, 4 * half, r);
        decide_add<4>(cpart, I.ct0, I.ct1, 4 * half, c);
        decide_add<4>(lcpart, I.lc0, I.lc1, 4 * half, c);
        for (int k = 0; k < 3; ++k) acc[7 * half + k] = r[k];
        for (int k = 0; k < 4; ++k) acc[7 * half + 3 + k] = c[k];
    }
    block_sums<DECIDE_NT, NTOT>(acc, red, tot);
    __syncthreads();
}

__global__ __launch_bounds__(DECIDE_NT) void k_decide(const DecideArgs d)
{
    __shared__ double red[DECIDE_NT / 64 * NTOT], tot[NTOT], tot2[NTOT];
    const int inst = blockIdx.x;
    InstState &S = d.st[inst];
    if (S.status != ST_RUN) {
        // stopped on the average at an earlier check: it has been taken
        if (threadIdx.x == 0) S.take_avg = 0;
        return;
    }
    const InstInfo I = d.info[inst];
    decide_totals(I, d.rpart, d.lrpart, d.cpart, d.lcpart, red, tot);
    // the same reduction over the running average's check
    if (d.rpart2) decide_totals(I, d.rpart2, d.lrpart2, d.cpart2, d.lcpart2, red, tot2);
    if (threadIdx.x != 0) return;
    decide_state(S, tot, d.rpart2 ? tot2 : nullptr, d.R);
    if (S.status != ST_RUN) d.mirror[inst] = S;
}

// ------------------------------------------------------- adaptive steps
// Step-size rule after the k-th iteration (k counted from 1 over the call),
// in FP64 (Algorithm 1's step-size update, read as PDLP's adaptive rule
// without retries): eta_bar = (omega |dx~|^2 + |dy~|^2 / omega) / (2 |dy^T A dx|),
// eta <- min((1 - (k+1)^-0.3) eta_bar, (1 + (k+1)^-0.6) eta); eta_bar is
// infinite when the interaction is 0, and eta is kept when the move is 0.
// p6, p3: (k+1)^-0.6 and (k+1)^-0.3.
__device__ __forceinline__ void adapt_step(InstState &S, double nx, double ny, double inter, double p6, double p3)
{
    if (!(nx + ny > 0.0)) return;
    const double grow = (1.0 + p6) * S.eta;
    double eta = grow;
    if (inter != 0.0) {
        const double ebar = (S.omega * nx + ny / S.omega) / (2.0 * fabs(inter));
        const double shrink = (1.0 - p3) * ebar;
        eta = shrink < grow ? shrink : grow;
    }
    S.eta = eta;
    S.t = eta / S.omega;
    S.s = eta * S.omega;
}

// One workgroup per instance: fixed-order FP64 sums of the iteration
// partials of both passes (slot ranges in InstInfo::ir), then the rule.  A
// launch an iteration, bound by its latency: the partials of both passes load
// together, STEP_U of each a thread at a time, the last wave forms the rule's
// powers meanwhile, and the three sums share a barrier (one sum after the
// other and the powers behind them: 6.5 us an iteration of a 5k x 10k LP).
constexpr int STEP_NT = 1024, STEP_SUM = STEP_NT - 64, STEP_U = 4;

__global__ __launch_bounds__(STEP_NT) void k_step(const StepArgs a)
{
    __shared__ double red[3 * STEP_NT / 64], tot[3], pw[2];
    const int inst = blockIdx.x, tid = threadIdx.x;
    InstState &S = a.st[inst];
    if (S.status != ST_RUN || a.jw >= S.nrun) return;
    const InstInfo &I = a.info[inst];
    double acc[3] = {};
    if (tid >= STEP_SUM) {
        if (tid < STEP_SUM + 2) {
            const double k1 = (double)(S.k + a.jw + 1) + 1.0;
            pw[tid - STEP_SUM] = pow(k1, tid == STEP_SUM ? -0.6 : -0.3);
        }
    } else {
        const double2 *cip = reinterpret_cast<const double2 *>(a.cip), *rip = reinterpret_cast<const double2 *>(a.rip);
        for (int r = 0; r < 3; ++r) {
            const int c0 = I.ir[1][r][0], c1 = I.ir[1][r][1], r0 = I.ir[0][r][0], r1 = I.ir[0][r][1];
            const int len = max(c1 - c0, r1 - r0);
            for (int q0 = tid; q0 < len; q0 += STEP_SUM * STEP_U) {
                double2 c[STEP_U], v[STEP_U];
#pragma unroll
                for (int u = 0; u < STEP_U; ++u) {
                    const int q = q0 + u * STEP_SUM;
                    c[u] = c0 + q < c1 ? cip[c0 + q] : double2{0.0, 0.0};
                    v[u] = r0 + q < r1 ? rip[r0 + q] : double2{0.0, 0.0};
                }
#pragma unroll
                for (int u = 0; u < STEP_U; ++u) {
                    acc[0] += c[u].x;
                    acc[1] += v[u].x;
                    acc[2] += v[u].y;
                }
            }
        }
    }
    block_sums<STEP_NT, 3>(acc, red, tot);
    __syncthreads();
    if (tid == 0) adapt_step(S, tot[0], tot[1], tot[2], pw[0], pw[1]);
}

// --------------------------------------------- fused window (tiny instances)
// One workgroup per instance runs up to nwin check windows -- FP64 KKT check,
// decision, then up to R iterations -- with the instance's matrix (both
// orientations, decoded to local index + value) and vectors held in LDS and
// workgroup barriers between the passes.  Used when every instance of the
// handle fits in LDS; it removes the per-pass launch latency that dominates
// such instances, and with many windows a launch also the reload of the
// instance and the host's turn per window.  No workgroup ever waits for
// another.
template <class V>
struct TinyLds {
    int *rptr, *cptr, *rcol, *ccol;
    V *zero;  // element 0 of the dynamic LDS, holds zero
    V *rval, *cval, *x, *xb, *xr, *c, *l, *u, *dc2, *q, *y, *yr, *b, *dr2;
    double *ax;
    uint8_t *sense;
};

template <class V>
__device__ __forceinline__ TinyLds<V> tiny_carve(unsigned char *base, int m, int n, int rnnz, int cnnz)
{
    TinyLds<V> t;
    unsigned char *q = base;
    auto take = [&](size_t bytes) {
        unsigned char *p = q;
        q += (bytes + 15) & ~(size_t)15;
        return p;
    };
    t.zero = (V *)take(sizeof(V));
    t.rptr = (int *)take(4 * (size_t)(m + 1));
    t.cptr = (int *)take(4 * (size_t)(n + 1));
    t.rcol = (int *)take(4 * (size_t)rnnz);
    t.ccol = (int *)take(4 * (size_t)cnnz);
    t.rval = (V *)take(sizeof(V) * (size_t)rnnz);
    t.cval = (V *)take(sizeof(V) * (size_t)cnnz);
    t.x = (V *)take(sizeof(V) * (size_t)n);
    t.xb = (V *)take(sizeof(V) * (size_t)n);
    t.xr = (V *)take(sizeof(V) * (size_t)n);
    t.c = (V *)take(sizeof(V) * (size_t)n);
    t.l = (V *)take(sizeof(V) * (size_t)n);
    t.u = (V *)take(sizeof(V) * (size_t)n);
    t.dc2 = (V *)take(sizeof(V) * (size_t)n);
    t.q = (V *)take(sizeof(V) * (size_t)n);
    t.y = (V *)take(sizeof(V) * (size_t)m);
    t.yr = (V *)take(sizeof(V) * (size_t)m);
    t.b = (V *)take(sizeof(V) * (size_t)m);
    t.dr2 = (V *)take(sizeof(V) * (size_t)m);
    t.ax = (double *)take(8 * (size_t)m);
    t.sense = (uint8_t *)take((size_t)m);
    return t;
}

// A lane's share of one row (column) of the fused window, in registers: its
// entries lane, lane + L, ... of the row, at most K, as value and byte offset
// of what they gather in the dynamic LDS (the address of the read, so that an
// entry costs one LDS read and one multiplication; as 16-bit element indices
// the unpacking took most of a pass's instructions).  Slots beyond the lane's
// entries gather offset 0, which holds zero (so the sums need no masks, and
// 0 * 0 is added, never 0 * inf).
template <class V, int K>
struct LaneRow {
    uint32_t off[K];
    V val[K];
    int wcnt;  // the most entries of any lane of the wave
};

template <class V, int K>
__device__ __forceinline__ void lane_row_load(LaneRow<V, K> &r, const int *ptr, const int *col, const V *val,
                                              uint32_t vec0, int row, bool on, int lane, int L)
{
    const int e0 = on ? ptr[row] + lane : 0, e1 = on ? ptr[row + 1] : 0;
    int cnt = e0 < e1 ? (e1 - e0 + L - 1) / L : 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool in = k < cnt;
        const int e = in ? e0 + k * L : 0;  // (element 0 is read in any case)
        const uint32_t j = (uint32_t)col[e];
        const V v = val[e];
        r.off[k] = in ? vec0 + j * (uint32_t)sizeof(V) : 0;
        r.val[k] = in ? v : (V)0;
    }
    for (int off = 32; off > 0; off >>= 1) cnt = max(cnt, __shfl_xor(cnt, off, 64));
    r.wcnt = __builtin_amdgcn_readfirstlane(cnt);
}

// sum of val * (what lds + off holds) over the row's lanes; the gathers of
// four slots go out before the first product waits.
template <class V, int K>
__device__ __forceinline__ V lane_row_dot(const LaneRow<V, K> &r, const unsigned char *lds, int L)
{
    V s = 0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 4)
        if (k0 < r.wcnt) {
            V g[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) g[k] = *reinterpret_cast<const V *>(lds + r.off[k0 + k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) s += r.val[k0 + k] * g[k];
        }
    return group_sum(s, L);
}

// The decision, by one thread, and the step rule's powers, as calls: inlined,
// their logarithms and powers take the registers that the iterations need.
__device__ __attribute__((noinline)) void tiny_decide(InstState *S, const double *tot, int R)
{
    decide_state(*S, tot, nullptr, R);
}

__device__ __attribute__((noinline)) double tiny_power(double base, double e) { return pow(base, e); }

constexpr int TINY_NT = 1024;
// Entries of a row that a lane can hold in registers (of the 128 a thread of
// a 1024-thread workgroup has, an entry takes 2 in FP32 and 3 in FP64).
template <class V>
constexpr int TINY_K = sizeof(V) == 8 ? 8 : 16;

// Lanes of a row (column) of the fused window, of `rows` with at most `longest`
// entries.  A pass is bound by instruction issue: its update costs a wave
// about as much as 20 entries, so the rows take five eighths of the threads at
// most (two or three waves a SIMD) rather than all of them, and more lanes only
// where their entries would not fit the registers.  Set covers of 20 x 50 to
// 600 x 200, an iteration with its share of the checks: with all threads
// 0.84-1.06 us, with five eighths 0.75-0.94 (200 x 500: 1.01 -> 0.88 in FP32,
// 1.03 -> 0.90 in FP64; equal where both give the same lanes, from 230 x 575);
// adaptive steps 2.65-3.27 -> 2.51-2.98.  Three quarters of the threads differ
// from five eighths at 350 columns only (0.87 against 0.82).  One half is up to
// 0.1 us faster below 130 rows or 320 columns and equal above.
template <class V>
__device__ __forceinline__ int tiny_lanes(int rows, int longest)
{
    int L = lanes_per_row<TINY_NT / 8 * 5>(rows);
    while (L < 64 && longest > TINY_K<V> * L && rows * (L << 1) <= TINY_NT) L <<= 1;
    return L;
}

// Scratch of the fused window in static LDS (its dynamic LDS leaves 1024 B).
struct TinyShared {
    InstState S;
    double red[4 * TINY_NT / 64];
    double tot[NTOT + 2];
    double power[2];  // of the step rule, (k+1)^-0.6 and (k+1)^-0.3
    int nrun, restart, longest[2];
    double t, s;
};

// Sums of acc over the workgroup into sh.tot, four at a time, waves in order.
__device__ __forceinline__ void tiny_totals(double (&acc)[NTOT], TinyShared &sh)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int k0 = 0; k0 < NTOT; k0 += 4) {
#pragma unroll
        for (int k = k0; k < k0 + 4 && k < NTOT; ++k) {
            const double v = group_sum(acc[k], 64);
            if (l == 0) sh.red[4 * w + k - k0] = v;
        }
        __syncthreads();
        if (threadIdx.x < 4) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < TINY_NT / 64; ++q) s += sh.red[4 * q + threadIdx.x];
            sh.tot[k0 + threadIdx.x] = s;
        }
        __syncthreads();
    }
}

// Adaptive steps of the fused window, before an iteration's passes: two lanes
// of the last wave form the rule's powers for it (iteration number k1 - 1)
// while the others work.
__device__ __forceinline__ void tiny_powers(TinyShared &sh, int tid, double k1)
{
    if (tid >= TINY_NT - 2) sh.power[tid - (TINY_NT - 2)] = tiny_power(k1, tid == TINY_NT - 2 ? -0.6 : -0.3);
}

// And after them: the sums of the moves, and the rule.  (Two sums with two
// barriers each and both powers behind them made 5.8 us an iteration of a 200 x
// 500 set cover, against 3.0 us.)
__device__ __forceinline__ void tiny_step(TinyShared &sh, int tid, double nx, double ny, double inter)
{
    const double acc[3] = {nx, ny, inter};
    block_sums<TINY_NT, 3>(acc, sh.red, sh.tot);
    __syncthreads();
    if (tid == 0) {
        adapt_step(sh.S, sh.tot[0], sh.tot[1], sh.tot[2], sh.power[0], sh.power[1]);
        sh.t = sh.S.t;
        sh.s = sh.S.s;
    }
    __syncthreads();
}

// nrun PDHG iterations (Algorithm 1), column pass, barrier, row pass, with
// every row and column spread over at most one group of lanes: entries and
// epilogue operands sit in registers, LDS holds only what is gathered (x_bar
// and y), so a pass is one round of LDS gathers, a few data-parallel adds and
// the update.  Bound by LDS latency and gather throughput.  With every operand
// read from LDS in a chain (pointers, entry, gather, operands) an iteration of
// a 200 x 500 set cover took 1.5 us in FP64 and 256 of them (FP32, 192
// iterations) 740 us a solve; now 0.7 us and 430 us.
template <class V, int K, bool ADAPT>
__device__ __forceinline__ void tiny_iters_reg(const TinyArgs<V> &a, const TinyLds<V> &L, TinyShared &sh, int tid, int m,
                                               int n, int Lc, int Lr)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int j = tid / Lc, i = tid / Lr;
    const bool jon = j < n, ion = i < m;
    // waves without a column (row) go straight to the barrier
    const bool jwave = __any(jon), iwave = __any(ion);
    const bool jw = jon && (tid & (Lc - 1)) == 0, iw = ion && (tid & (Lr - 1)) == 0;
    LaneRow<V, K> C, R;
    lane_row_load<V, K>(C, L.cptr, L.ccol, L.cval, (uint32_t)((L.y - L.zero) * sizeof(V)), j, jon, tid & (Lc - 1), Lc);
    lane_row_load<V, K>(R, L.rptr, L.rcol, L.rval, (uint32_t)((L.xb - L.zero) * sizeof(V)), i, ion, tid & (Lr - 1), Lr);
    V x = 0, c = 0, lo = 0, hi = 0, dc2 = 0, q = 0, y = 0, b = 0, dr2 = 0;
    double ax = 0.0;
    uint8_t sn = 'E';
    if (jon) {
        x = L.x[j];
        c = L.c[j];
        lo = L.l[j];
        hi = L.u[j];
        dc2 = L.dc2[j];
        q = L.q[j];
    }
    if (ion) {
        y = L.y[i];
        b = L.b[i];
        dr2 = L.dr2[i];
        sn = L.sense[i];
        ax = L.ax[i];
    }
    if (sh.restart) {
        if (jw) L.xr[j] = x;
        if (iw) L.yr[i] = y;
    }
    const int nrun = sh.nrun;
    V t = (V)sh.t, sd = (V)sh.s;
    for (int it = 0; it < nrun; ++it) {
        double nx = 0.0, ny = 0.0, inter = 0.0;
        if (ADAPT) tiny_powers(sh, tid, (double)(sh.S.k + it + 1) + 1.0);
        if (jwave) {
            const V aty = lane_row_dot<V, K>(C, lds_raw, Lc);
            V xn = x + t * dc2 * (aty - c);
            if (a.q) xn /= (V)1 + t * dc2 * q;
            xn = xn < lo ? lo : xn;
            xn = xn > hi ? hi : xn;
            if (jw) L.xb[j] = ADAPT ? xn - x : (V)2 * xn - x;  // adaptive: the move dx
            if (ADAPT && jw) {
                const double d = (double)xn - (double)x;
                nx = d * d / (double)dc2;
            }
            x = xn;
        }
        __syncthreads();
        if (iwave) {
            const V axb = lane_row_dot<V, K>(R, lds_raw, Lr);
            // adaptive: axb = (A dx)_i and (A x_bar)_i = (A x)_i + 2 (A dx)_i
            const V res = ADAPT ? (V)((double)b - (ax + 2.0 * (double)axb)) : b - axb;
            V v = y + sd * dr2 * res;
            if (sn == 'G') v = v > (V)0 ? v : (V)0;
            else if (sn == 'L') v = v < (V)0 ? v : (V)0;
            if (iw) L.y[i] = v;
            if (ADAPT) {
                if (iw) {
                    const double dy = (double)v - (double)y;
                    ny = dy * dy / (double)dr2;
                    inter = dy * (double)axb;
                }
                ax += (double)axb;
            }
            y = v;
        }
        __syncthreads();
        if (ADAPT) {
            tiny_step(sh, tid, nx, ny, inter);
            t = (V)sh.t;
            sd = (V)sh.s;
        }
    }
    if (jw) L.x[j] = x;
    __syncthreads();
}

// The same iterations with the matrix read from LDS: more rows or columns
// than threads, or a row with more entries than its lanes hold.
template <class V>
__device__ __forceinline__ void tiny_iters_lds(const TinyArgs<V> &a, const TinyLds<V> &L, TinyShared &sh, int tid, int m,
                                               int n)
{
    constexpr int NT = TINY_NT;
    const int nrun = sh.nrun;
    V t = (V)sh.t, sd = (V)sh.s;
    // lane groups: a power of two of lanes per column / row, as many as fit
    const int Lc = lanes_per_row<NT>(n), Lr = lanes_per_row<NT>(m);
    const int lc = tid & (Lc - 1), lr = tid & (Lr - 1);
    for (int it = 0; it < nrun; ++it) {
        const bool copy_ref = it == 0 && sh.restart != 0;
        double nx = 0.0, ny = 0.0, inter = 0.0;
        if (a.adapt) tiny_powers(sh, tid, (double)(sh.S.k + it + 1) + 1.0);
        for (int j = tid / Lc; j < n; j += NT / Lc) {
            V aty = 0;
            for (int e = L.cptr[j] + lc; e < L.cptr[j + 1]; e += Lc) aty += L.cval[e] * L.y[L.ccol[e]];
            if (Lc > 1) aty = group_sum(aty, Lc);
            if (lc == 0) {
                const V xj = L.x[j];
                V xn = xj + t * L.dc2[j] * (aty - L.c[j]);
                if (a.q) xn /= (V)1 + t * L.dc2[j] * L.q[j];
                xn = xn < L.l[j] ? L.l[j] : xn;
                xn = xn > L.u[j] ? L.u[j] : xn;
                if (copy_ref) L.xr[j] = xj;
                L.xb[j] = a.adapt ? xn - xj : (V)2 * xn - xj;  // adaptive: the move dx
                L.x[j] = xn;
                if (a.adapt) {
                    const double d = (double)xn - (double)xj;
                    nx += d * d / (double)L.dc2[j];
                }
            }
        }
        __syncthreads();
        for (int i = tid / Lr; i < m; i += NT / Lr) {
            V axb = 0;
            for (int e = L.rptr[i] + lr; e < L.rptr[i + 1]; e += Lr) axb += L.rval[e] * L.xb[L.rcol[e]];
            if (Lr > 1) axb = group_sum(axb, Lr);
            if (lr == 0) {
                const V yi = L.y[i];
                // adaptive: axb = (A dx)_i and (A x_bar)_i = (A x)_i + 2 (A dx)_i
                const V res = a.adapt ? (V)((double)L.b[i] - (L.ax[i] + 2.0 * (double)axb)) : L.b[i] - axb;
                V v = yi + sd * L.dr2[i] * res;
                const uint8_t sn = L.sense[i];
                if (sn == 'G') v = v > (V)0 ? v : (V)0;
                else if (sn == 'L') v = v < (V)0 ? v : (V)0;
                if (copy_ref) L.yr[i] = yi;
                L.y[i] = v;
                if (a.adapt) {
                    const double dy = (double)v - (double)yi;
                    ny += dy * dy / (double)L.dr2[i];
                    inter += dy * (double)axb;
                    L.ax[i] += (double)axb;
                }
            }
        }
        __syncthreads();
        if (a.adapt) {
            tiny_step(sh, tid, nx, ny, inter);
            t = (V)sh.t;
            sd = (V)sh.s;
        }
    }
}

template <class V, int FMT>
__global__ __launch_bounds__(TINY_NT) void k_tiny(const TinyArgs<V> a, const int R, const int nwin)
{
    constexpr int NT = TINY_NT, K = TINY_K<V>;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ TinyShared sh;
    static_assert(sizeof(TinyShared) + TINY_ZERO <= 1024, "static LDS of the fused window");
    const int inst = blockIdx.x, tid = threadIdx.x;
    if (a.st[inst].status != ST_RUN) return;
    const InstInfo &I = a.info[inst];
    const int m = I.row1 - I.row0, n = I.col1 - I.col0;
    const int re0 = a.R.ptr[I.row0], rnnz = a.R.ptr[I.row1] - re0;
    const int ce0 = a.C.ptr[I.col0], cnnz = a.C.ptr[I.col1] - ce0;
    const TinyLds<V> L = tiny_carve<V>(lds_raw, m, n, rnnz, cnnz);
    if (tid == 0) {
        sh.S = a.st[inst];
        *L.zero = (V)0;
    }
    // ---- load the instance into LDS
    for (int i = tid; i <= m; i += NT) L.rptr[i] = a.R.ptr[I.row0 + i] - re0;
    for (int j = tid; j <= n; j += NT) L.cptr[j] = a.C.ptr[I.col0 + j] - ce0;
    for (int e = tid; e < rnnz; e += NT) {
        uint32_t w;
        V v;
        load_entry<FMT, V>(a.R, re0 + e, w, v);
        L.rcol[e] = decode_entry<FMT, V>(a.R, w, v) - I.col0;
        L.rval[e] = v;
    }
    for (int e = tid; e < cnnz; e += NT) {
        uint32_t w;
        V v;
        load_entry<FMT, V>(a.C, ce0 + e, w, v);
        L.ccol[e] = decode_entry<FMT, V>(a.C, w, v) - I.row0;
        L.cval[e] = v;
    }
    for (int j = tid; j < n; j += NT) {
        const int g = I.col0 + j;
        L.x[j] = a.x[g];
        L.xb[j] = a.xbar[g];
        L.xr[j] = a.xr[g];
        L.c[j] = a.c[g];
        L.l[j] = a.l[g];
        L.u[j] = a.u[g];
        L.dc2[j] = a.dc2[g];
        L.q[j] = a.q ? a.q[g] : (V)0;
    }
    for (int i = tid; i < m; i += NT) {
        const int g = I.row0 + i;
        L.y[i] = a.y[g];
        L.yr[i] = a.yr[g];
        L.b[i] = a.b[g];
        L.dr2[i] = a.dr2[g];
        L.sense[i] = a.sense[g];
    }
    __syncthreads();
    // lanes per column and row, and whether every lane's share fits registers
    if (tid < 2) sh.longest[tid] = 0;
    __syncthreads();
    for (int j = tid; j < n; j += NT) atomicMax(&sh.longest[0], L.cptr[j + 1] - L.cptr[j]);
    for (int i = tid; i < m; i += NT) atomicMax(&sh.longest[1], L.rptr[i + 1] - L.rptr[i]);
    __syncthreads();
    const int Lc = tiny_lanes<V>(n, sh.longest[0]), Lr = tiny_lanes<V>(m, sh.longest[1]);
    const bool regs = n <= NT && m <= NT && sh.longest[0] <= K * Lc && sh.longest[1] <= K * Lr;
    int win = 0;
    for (; win < nwin; ++win) {
        // the thread index behind a barrier for the optimiser: addresses made
        // from it are not kept in registers from window to window (they are
        // enough to spill)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lc = tid & (Lc - 1), lr = tid & (Lr - 1);
        // ---- FP64 KKT check of the current point (Section 2.2)
        double acc[NTOT] = {};
        for (int i = tid / Lr; i < m; i += NT / Lr) {
            // (operands in global memory first: they load during the sum)
            const int gi = I.row0 + i;
            const bool head = lr == 0;
            const double bb = head ? a.b64[gi] : 0.0, drow = head ? a.dr64[gi] : 1.0;
            const double yprev = head ? (double)a.yp[gi] : 0.0, axprev = head ? a.axp[gi] : 0.0;
            double ax = 0.0;
            for (int e = L.rptr[i] + lr; e < L.rptr[i + 1]; e += Lr) ax += (double)L.rval[e] * (double)L.x[L.rcol[e]];
            ax = group_sum(ax, Lr);
            if (!head) continue;
            const uint8_t sn = L.sense[i];
            double r;
            if (sn == 'G') r = fmax(bb - ax, 0.0);
            else if (sn == 'L') r = fmax(ax - bb, 0.0);
            else r = bb - ax;
            const double yy = (double)L.y[i];
            const double dy = (yy - (double)L.yr[i]) / drow;
            L.ax[i] = ax;  // A x of the current point in FP64 (adaptive steps)
            acc[0] += r * r;
            acc[1] += bb * yy;
            acc[2] += dy * dy;
            // moves since the previous check (infeasibility certificates)
            const double v = yy - yprev;
            const double vp = sn == 'G' ? fmax(v, 0.0) : (sn == 'L' ? fmin(v, 0.0) : v);
            const double ad = ax - axprev;
            const double viol = sn == 'G' ? fmax(-ad, 0.0) : (sn == 'L' ? fmax(ad, 0.0) : ad);
            acc[7] += bb * v;
            acc[8] += (v - vp) * (v - vp);
            acc[9] += viol * viol;
            a.yp[gi] = L.y[i];
            a.axp[gi] = ax;
        }
        for (int j = tid / Lc; j < n; j += NT / Lc) {
            const int g = I.col0 + j;
            const bool head = lc == 0;
            const double cc = head ? a.c64[g] : 0.0, lo = head ? a.l64[g] : 0.0, hi = head ? a.u64[g] : 0.0;
            const double dcol = head ? a.dc64[g] : 1.0, qj = head && a.q64 ? a.q64[g] : 0.0;
            const double xprev = head ? (double)a.xp[g] : 0.0, atyprev = head ? a.atyp[g] : 0.0;
            double aty = 0.0;
            for (int e = L.cptr[j] + lc; e < L.cptr[j + 1]; e += Lc) aty += (double)L.cval[e] * (double)L.y[L.ccol[e]];
            aty = group_sum(aty, Lc);
            if (!head) continue;
            const double xq = (double)L.x[j];
            const double qx = a.q64 ? qj * xq : 0.0;
            const double gr = cc + qx - aty;
            const bool lf = isfinite(lo), uf = isfinite(hi);
            double lam;
            if (lf && uf) lam = gr;
            else if (lf) lam = fmax(gr, 0.0);
            else if (uf) lam = fmin(gr, 0.0);
            else lam = 0.0;
            const double rd = gr - lam;
            const double dx = (xq - (double)L.xr[j]) / dcol;
            acc[3] += rd * rd;
            acc[4] += cc * xq + 0.5 * qx * xq;
            if (lf && lam > 0.0) acc[5] += lo * lam;
            if (uf && lam < 0.0) acc[5] += hi * lam;
            acc[5] -= 0.5 * qx * xq;
            acc[6] += dx * dx;
            const double w = aty - atyprev;
            double rl;
            if (lf && uf) rl = -w;
            else if (lf) rl = fmax(-w, 0.0);
            else if (uf) rl = fmin(-w, 0.0);
            else rl = 0.0;
            acc[10] += (w + rl) * (w + rl);
            if (lf && rl > 0.0) acc[11] += lo * rl;
            if (uf && rl < 0.0) acc[11] += hi * rl;
            const double d = xq - xprev;
            acc[12] += cc * d;
            double bv;
            if (lf && uf) bv = d;
            else if (lf) bv = fmin(d, 0.0);
            else if (uf) bv = fmax(d, 0.0);
            else bv = 0.0;
            acc[13] += bv * bv;
            if (a.q64) acc[13] += (qj * d) * (qj * d);
            a.xp[g] = L.x[j];
            a.atyp[g] = aty;
        }
        tiny_totals(acc, sh);
        if (tid == 0) {
            tiny_decide(&sh.S, sh.tot, R);
            sh.nrun = sh.S.status == ST_RUN ? sh.S.nrun : 0;
            sh.restart = sh.S.restart_now;
            sh.t = sh.S.t;
            sh.s = sh.S.s;
        }
        __syncthreads();
        if (sh.nrun == 0) break;
        if (!regs) tiny_iters_lds<V>(a, L, sh, tid, m, n);
        else if (a.adapt) tiny_iters_reg<V, K, true>(a, L, sh, tid, m, n, Lc, Lr);
        else tiny_iters_reg<V, K, false>(a, L, sh, tid, m, n, Lc, Lr);
    }
    if (tid == 0) {
        a.st[inst] = sh.S;
        if (sh.S.status != ST_RUN) a.mirror[inst] = sh.S;
    }
    if (win == 0) return;
    // ---- write the iterates back
    for (int j = tid; j < n; j += NT) {
        const int g = I.col0 + j;
        a.x[g] = L.x[j];
        a.xbar[g] = L.xb[j];
        a.xr[g] = L.xr[j];
    }
    for (int i = tid; i < m; i += NT) {
        const int g = I.row0 + i;
        a.y[g] = L.y[i];
        a.yr[g] = L.yr[i];
    }
}

template <class V>
void launch_tiny(const TinyArgs<V> &a, int fmt, int count, int R, int nwin, size_t shmem, hipStream_t s,
                 bool prepare)
{
    auto run = [&](auto fn) {
        if (prepare) (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)shmem);
        else hipLaunchKernelGGL(fn, dim3(count), dim3(1024), shmem, s, a, R, nwin);
    };
    if constexpr (sizeof(V) == 8) {
        run(k_tiny<V, FMT_F64>);
    } else {
        if (fmt == FMT_PACKED) run(k_tiny<V, FMT_PACKED>);
        else if (fmt == FMT_BF16) run(k_tiny<V, FMT_BF16>);
        else run(k_tiny<V, FMT_F32>);
    }
}

// Restart to the average: copies the running mean over the iterate where the
// decision took it (restart, OPTIMAL or iteration-limit stop); blocks
// workgroups an instance.  The next decision clears the flag.  The restart
// reference is copied from the new iterate by the next iteration, as for any
// restart.
template <class V>
__global__ __launch_bounds__(256) void k_take_avg(const InstState *st, const InstInfo *info, V *x, V *y, const V *xa,
                                                  const V *ya, double *ax, const double *axa, int blocks)
{
    const int inst = blockIdx.x / blocks, first = (blockIdx.x % blocks) * 256 + threadIdx.x, step = blocks * 256;
    if (!st[inst].take_avg) return;
    const InstInfo &I = info[inst];
    for (int j = I.col0 + first; j < I.col1; j += step) x[j] = xa[j];
    for (int i = I.row0 + first; i < I.row1; i += step) {
        y[i] = ya[i];
        if (ax) ax[i] = axa[i];
    }
}

__global__ void k_force_stop(InstState *st, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count && st[i].status == ST_RUN) st[i].force_stop = 1;
}

// ---------------------------------------------------------------- setup
// One round of the preconditioner, rows and columns in one launch: every
// d_r,i (d_c,j) of the last round is divided by the square root of its row's
// (column's) largest |d_r a d_c| (mode 0) or of their sum (mode 1) where that
// is positive; null: all ones.  LR / LC lanes per row / column.  The setup of a
// small LP is bound by its launches: four a round (two reductions, two updates)
// and one for each vector's cast or clearing made 68, 190 us of a 1.2 ms
// one-shot solve.
template <int FMT>
__device__ __forceinline__ void scale_one(const MatView &M, int row, int lane, int L, const double *drow,
                                          const double *dcol, double *out, int mode)
{
    const int e1 = M.ptr[row + 1];
    const double dr = drow ? drow[row] : 1.0;
    double acc = 0.0;
    for (int e = M.ptr[row] + lane; e < e1; e += L) {
        uint32_t w;
        double a;
        load_entry<FMT, double>(M, e, w, a);
        const int idx = decode_entry<FMT, double>(M, w, a);
        const double v = fabs(dr * a * (dcol ? dcol[idx] : 1.0));
        acc = mode == 0 ? fmax(acc, v) : acc + v;
    }
    for (int off = L >> 1; off > 0; off >>= 1) {
        const double o = __shfl_xor(acc, off, 64);
        acc = mode == 0 ? fmax(acc, o) : acc + o;
    }
    if (lane == 0) out[row] = acc > 0.0 ? dr / sqrt(acc) : dr;
}

template <int FMT>
__global__ __launch_bounds__(256) void k_scale_round(const ScaleArgs a)
{
    const bool rows = (int)blockIdx.x < a.rblocks;
    const int L = rows ? a.LR : a.LC, first = rows ? (int)blockIdx.x : (int)blockIdx.x - a.rblocks;
    const int i = first * (256 / L) + (int)threadIdx.x / L, lane = threadIdx.x & (L - 1);
    if (rows) {
        if (i < a.M) scale_one<FMT>(a.R, i, lane, L, a.dr, a.dc, a.dr_new, a.mode);
    } else {
        if (i < a.N) scale_one<FMT>(a.C, i, lane, L, a.dc, a.dr, a.dc_new, a.mode);
    }
}

// The vectors of a new handle in one launch: path-precision copies of the
// problem, squared preconditioner, iterates and checkpoints cleared.
template <class V>
__global__ __launch_bounds__(256) void k_setup_vectors(const SetupArgs<V> a)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < a.N) {
        a.c[k] = (V)a.c64[k];
        a.l[k] = (V)a.l64[k];
        a.u[k] = (V)a.u64[k];
        a.dc2[k] = (V)(a.dc64[k] * a.dc64[k]);
        a.x[k] = a.xbar[k] = a.xr[k] = a.xp[k] = (V)0;
        a.atyp[k] = 0.0;
    }
    if (k < a.M) {
        a.b[k] = (V)a.b64[k];
        a.dr2[k] = (V)(a.dr64[k] * a.dr64[k]);
        a.y[k] = a.yr[k] = a.yp[k] = (V)0;
        a.ax[k] = a.axp[k] = 0.0;
    }
}

// Per-instance norms of the current objective c_hat and of b: ||b||,
// ||c_hat||, and the cold-start primal weight ||D_c c_hat|| / ||D_r b|| (or 1).
//
// Bound by memory: 16 B per column (and per row, when the rows are summed).
// One workgroup per instance read a 300k x 600k LP's 14 MB in 1.05 ms and a
// 20k x 40k instance's in 75 us (latency of one CU's loads), so an instance
// is cut into norm_blocks() pieces of about NORM_CHUNK entries, one workgroup
// each, and the last of them adds the partial sums in a fixed order.  With that,
// and the sums of the instances that changed only, a new objective and a warm
// re-solve of 64 iterations of the 300k x 600k LP went from 4.80 to 3.73 ms,
// 64 objective updates and a re-solve of 64 20k x 40k instances from 11.5 to
// 7.4 ms (pieces of 8192; at 2048, with the pump's objective made in the same
// launch, the latter's update kernels take 0.4 ms less again; without a second
// launch for the sum of the pieces 4.80 -> 4.68 ms, and 32 updates and a
// re-solve of 16 5k x 10k instances 1.155 -> 1.106 ms).  The pieces depend on
// the instance alone, so a batch and a single solve agree bit for bit.  An
// instance of one piece is finished by its only workgroup.
__device__ __forceinline__ void norm_finish(InstState &S, const double s[4], bool rows)
{
    if (rows) {
        S.bnorm = sqrt(s[0]);
        S.bscale = sqrt(s[1]);
    }
    S.cnorm = sqrt(s[2]);
    const double cs = sqrt(s[3]);
    S.omega0 = (cs > 0.0 && S.bscale > 0.0) ? cs / S.bscale : 1.0;
}

// Sums v^2 and (d v)^2 over [lo, hi), four strides of the workgroup at a time.
__device__ __forceinline__ void norm_sums(const double *v, const double *d, int lo, int hi, double &s, double &t)
{
    for (int i0 = lo + (int)threadIdx.x; i0 < hi; i0 += 4 * 256) {
        double a[4], w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 256;
            a[u] = i < hi ? v[i] : 0.0;
            w[u] = i < hi ? d[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double x = w[u] * a[u];
            s += a[u] * a[u];
            t += x * x;
        }
    }
}

// The same over columns whose objective is the pump's (Algorithm 1, objective
// update), written on the way: c_hat_j = a kappa c_j + (1 - a) g_j, g_j = +1 /
// -1 from the rounding bit, 0 for continuous columns; bits count from j0.
template <class V>
__device__ __forceinline__ void blend_sums(const BlendArgs &B, double *c, const double *d, int j0, int lo, int hi,
                                           double &s, double &t)
{
    for (int i0 = lo + (int)threadIdx.x; i0 < hi; i0 += 4 * 256) {
        double w[4], co[4];
        bool up[4], in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = i0 + u * 256, q = j - j0;
            const bool on = j < hi;
            w[u] = on ? d[j] : 0.0;
            co[u] = on ? B.c_orig[j] : 0.0;
            up[u] = on && ((B.xbits[q >> 3] >> (q & 7)) & 1);
            in[u] = on && (!B.ibits || ((B.ibits[q >> 3] >> (q & 7)) & 1));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = i0 + u * 256;
            if (j >= hi) continue;
            const double g = in[u] ? (up[u] ? -1.0 : 1.0) : 0.0;
            const double v = B.a * B.kappa * co[u] + (1.0 - B.a) * g;
            c[j] = v;
            ((V *)B.cv)[j] = (V)v;
            const double x = w[u] * v;
            s += v * v;
            t += x * x;
        }
    }
}

// The same over a new objective, read where the host staged it (src counts
// from j0) and written on the way: a copy, a cast and the sums in one launch.
template <class V>
__device__ __forceinline__ void staged_sums(const double *src, double *c, V *cv, const double *d, int j0, int lo, int hi,
                                            double &s, double &t)
{
    for (int i0 = lo + (int)threadIdx.x; i0 < hi; i0 += 4 * 256) {
        double v[4], w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = i0 + u * 256;
            v[u] = j < hi ? src[j - j0] : 0.0;
            w[u] = j < hi ? d[j] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = i0 + u * 256;
            if (j >= hi) continue;
            c[j] = v[u];
            cv[j] = (V)v[u];
            const double x = w[u] * v[u];
            s += v[u] * v[u];
            t += x * x;
        }
    }
}

// How a norm launch gets the objective.
enum { NORM_KEEP = 0, NORM_BLEND = 1, NORM_STAGED = 2 };

// One workgroup a piece of the instances [q0, q1), partial sums to its place in
// part, or the norms themselves when it is an instance's only one.  The
// workgroup that counts itself last in done[q] adds the pieces of q and
// clears the count (nobody waits); the fences order the partial sums before the
// count across the XCDs' L2s.
// NORM_BLEND / NORM_STAGED: the objective is written first (V: path precision).
template <class V, int SRC>
__global__ __launch_bounds__(256) void k_norm_part(const NormArgs a, const BlendArgs B)
{
    __shared__ double red[4 * 4], sum[4];
    __shared__ int last;
    int q = a.q0, blk = (int)blockIdx.x, first = 0;
    if (a.off) {  // the instance that holds the piece
        const int at = a.off[q] + blk;
        for (int hi = a.q1; hi - q > 1;) {
            const int mid = q + (hi - q) / 2;
            if (a.off[mid] <= at) q = mid;
            else hi = mid;
        }
        first = a.off[q];
        blk = at - first;
    } else if (a.q1 - q > 1) {
        q += blk;
        blk = 0;
    }
    const InstInfo &I = a.info[q];
    const int m = I.row1 - I.row0, n = I.col1 - I.col0;
    const int nb = norm_blocks(m, n);
    double *const part = a.part + 4 * (size_t)first;
    double acc[4] = {};
    if (a.rows)
        norm_sums(a.b, a.dr, I.row0 + (int)((int64_t)m * blk / nb), I.row0 + (int)((int64_t)m * (blk + 1) / nb),
                  acc[0], acc[1]);
    const int lo = I.col0 + (int)((int64_t)n * blk / nb), hi = I.col0 + (int)((int64_t)n * (blk + 1) / nb);
    if constexpr (SRC == NORM_BLEND) blend_sums<V>(B, a.c, a.dc, I.col0, lo, hi, acc[2], acc[3]);
    else if constexpr (SRC == NORM_STAGED)
        staged_sums<V>(B.c_orig, a.c, (V *)B.cv, a.dc, I.col0, lo, hi, acc[2], acc[3]);
    else norm_sums(a.c, a.dc, lo, hi, acc[2], acc[3]);
    block_sums<256, 4>(acc, red, nb == 1 ? sum : part + 4 * (size_t)blk);
    if (nb == 1) {
        __syncthreads();
        if (threadIdx.x == 0) norm_finish(a.st[q], sum, a.rows != 0);
        return;
    }
    if (threadIdx.x < 4) __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(a.done + q, 1) == nb - 1;
    __syncthreads();
    if (!last || threadIdx.x >= 64) return;
    __threadfence();
    double s[4] = {};
    for (int b = threadIdx.x; b < nb; b += 64) {
        const double *p = part + 4 * (size_t)b;
        for (int k = 0; k < 4; ++k) s[k] += p[k];
    }
    for (int k = 0; k < 4; ++k) s[k] = group_sum(s[k], 64);
    if (threadIdx.x == 0) {
        a.done[q] = 0;
        norm_finish(a.st[q], s, a.rows != 0);
    }
}

template <class V>
__global__ void k_cast(const double *src, V *dst, int len)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < len) dst[i] = (V)src[i];
}

// Start points: proj_[l,u](v) of column j and proj_Y(v) of a row.
template <class V>
__device__ __forceinline__ V project_x(V v, const V *l, const V *u, int j)
{
    v = v < l[j] ? l[j] : v;
    return v > u[j] ? u[j] : v;
}

template <class V>
__device__ __forceinline__ V project_y(V v, uint8_t sense)
{
    if (sense == 'G') return v > (V)0 ? v : (V)0;
    if (sense == 'L') return v < (V)0 ? v : (V)0;
    return v;
}

// x on [clo, clo + nc) and y on [rlo, rlo + nr), both in place.
template <class V>
__global__ __launch_bounds__(256) void k_project(V *x, const V *l, const V *u, int clo, int nc, V *y,
                                                 const uint8_t *sense, int rlo, int nr)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < nc) x[clo + i] = project_x(x[clo + i], l, u, clo + i);
    if (i < nr) y[rlo + i] = project_y(y[rlo + i], sense[rlo + i]);
}

// Start of a solve in one launch: thread q sets instance q's state (and its
// host mirror), and the threads of the start ranges project the start points
// (zeroed first on a cold start).  States set on the host cost two copies
// and two waits before the first window, ~60 us a solve.
template <class V>
__global__ __launch_bounds__(256) void k_begin(const BeginArgs<V> a)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < a.chi - a.clo) {
        const int j = a.clo + i;
        a.x[j] = project_x(a.warm ? a.x[j] : (V)0, a.l, a.u, j);
    }
    if (i < a.rhi - a.rlo) {
        const int r = a.rlo + i;
        a.y[r] = project_y(a.warm ? a.y[r] : (V)0, a.sense[r]);
    }
    if (i >= a.count) return;
    InstState &S = a.st[i];
    int64_t lim = a.iter_limit;
    if (a.limits) {
        const int64_t own = a.limits[i];
        if (own <= 0) {  // takes no part
            if (S.status == ST_RUN) S.status = ST_ITER;
            a.mirror[i] = S;
            return;
        }
        if (own < lim) lim = own;
    }
    const double omega = (a.warm && S.omega > 0.0) ? S.omega : S.omega0;
    S.status = ST_RUN;
    S.nrun = 0;
    S.restarts = 0;
    S.restart_now = 0;
    S.restart_on = a.restarts;
    S.avg_on = a.avg;
    S.take_avg = 0;
    S.force_stop = 0;
    S.k = 0;
    S.k_limit = lim;
    S.kr = 0;
    S.omega = omega;
    S.eta = a.eta;
    S.t = a.eta / omega;
    S.s = a.eta * omega;
    S.tol = a.tol;
    S.infeas_tol = a.infeas_tol;
    S.stall_tol = a.stall_tol;
    S.stall_checks = a.stall_checks;
    S.nstall = 0;
    S.pprev = S.dprev = 0.0;
    S.Er = S.Ep = 0.0;
    S.rel = S.rho_p = S.rho_d = S.rho_g = S.pobj = S.dobj = 0.0;
    a.mirror[i] = S;
}

template <class V>
void launch_begin(const BeginArgs<V> &a, hipStream_t s)
{
    int len = a.count;
    if (a.chi - a.clo > len) len = a.chi - a.clo;
    if (a.rhi - a.rlo > len) len = a.rhi - a.rlo;
    hipLaunchKernelGGL(k_begin<V>, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, a);
}

// Warm start from device memory, in three launches and one wait: the values
// are checked (flag |= 1: a NaN in x, |= 2: a non-finite y), then written only
// if the flag stayed clear, then the flag goes to the host and is cleared for
// the next call.
__global__ __launch_bounds__(256) void k_start_check(const double *x, int n, const double *y, int m, int *flag)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    int bad = 0;
    if (x && k < n && isnan(x[k])) bad |= 1;
    if (y && k < m && !isfinite(y[k])) bad |= 2;
    if (bad) atomicOr(flag, bad);
}

template <class V>
__global__ __launch_bounds__(256) void k_start_set(const StartArgs<V> a)
{
    if (*a.flag) return;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < a.n) a.x[k] = project_x(a.x0 ? (V)a.x0[k] : a.x[k], a.l, a.u, k);
    if (k < a.m) a.y[k] = project_y(a.y0 ? (V)a.y0[k] : a.y[k], a.sense[k]);
    if (a.omega && k < a.count && a.omega[k] > 0.0) a.st[k].omega = a.omega[k];
}

__global__ void k_start_flag(int *flag, int *host)
{
    *host = *flag;
    *flag = 0;
}

template <class V>
void launch_start(const StartArgs<V> &a, int *host_flag, hipStream_t s)
{
    const int nx = a.x0 ? a.n : 0, ny = a.y0 ? a.m : 0, given = nx > ny ? nx : ny;
    if (given > 0)
        hipLaunchKernelGGL(k_start_check, dim3((unsigned)((given + 255) / 256)), dim3(256), 0, s, a.x0, nx, a.y0, ny,
                           a.flag);
    int len = a.n > a.m ? a.n : a.m;
    if (a.count > len) len = a.count;
    hipLaunchKernelGGL(k_start_set<V>, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_start_flag, dim3(1), dim3(1), 0, s, a.flag, host_flag);
}

// ------------------------------------------------ MIP feasibility
// Algorithm 1 tests the PDHG point itself before rounding it: x is
// MIP-feasible when every row holds within tol (1 + |b_i|), every x_j lies
// within tol of [l_j, u_j] and every integer x_j within tol of an integer.
// Row activities are FP64 sums of a_ij x_j (MIP_L lanes per row, MIP_U entries
// a lane at a time: at 16 lanes a row of 11 nonzeros left a load in flight a
// lane, 115 us for 64 20k x 40k instances against 31 us for a pass); a
// non-finite value counts as a violation.  Flags: 1 = violated.
constexpr int MIP_L = 4, MIP_U = 4;

template <class V, int FMT>
__global__ __launch_bounds__(256) void k_mip_rows(const MatView M, int rows, const V *__restrict__ x,
                                                  const double *__restrict__ b, const uint8_t *__restrict__ sense,
                                                  double tol, uint8_t *__restrict__ bad)
{
    const int row = blockIdx.x * (256 / MIP_L) + threadIdx.x / MIP_L;
    const int lane = threadIdx.x & (MIP_L - 1);
    // whole lane groups leave together, so the sums below only involve lanes
    // that are still running
    if (row >= rows) return;
    const int e1 = M.ptr[row + 1];
    double acc = 0.0;
    for (int e0 = M.ptr[row] + lane; e0 < e1; e0 += MIP_L * MIP_U) {
        uint32_t w[MIP_U];
        double a[MIP_U];
        int j[MIP_U];
        V g[MIP_U];
#pragma unroll
        for (int u = 0; u < MIP_U; ++u) {
            const int e = e0 + u * MIP_L;
            w[u] = 0;
            a[u] = 0.0;
            if (e < e1) load_entry<FMT, double>(M, e, w[u], a[u]);
        }
#pragma unroll
        for (int u = 0; u < MIP_U; ++u) {
            j[u] = decode_entry<FMT, double>(M, w[u], a[u]);
            if (e0 + u * MIP_L < e1) g[u] = x[j[u]];
        }
#pragma unroll
        for (int u = 0; u < MIP_U; ++u)
            if (e0 + u * MIP_L < e1) acc += a[u] * (double)g[u];
    }
    acc = group_sum(acc, MIP_L);
    if (lane == 0) {
        const double bi = b[row], t = tol * (1.0 + fabs(bi));
        const uint8_t sn = sense[row];
        bool ok = isfinite(acc);
        if (sn != 'L') ok = ok && acc >= bi - t;
        if (sn != 'G') ok = ok && acc <= bi + t;
        bad[row] = ok ? 0 : 1;
    }
}

// is_int null: every column is integer.
template <class V>
__global__ void k_mip_cols(const V *__restrict__ x, const double *__restrict__ l, const double *__restrict__ u,
                           const uint8_t *__restrict__ is_int, double tol, int n, uint8_t *__restrict__ bad)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const double v = (double)x[j];
    bool ok = v >= l[j] - tol && v <= u[j] + tol;
    if (!is_int || is_int[j]) ok = ok && fabs(v - rint(v)) <= tol;
    bad[j] = ok ? 0 : 1;
}

// Whether one of the flags [lo, hi) is set, as this thread sees them: aligned
// words of 16 flags, the ends flag by flag (flag by flag throughout, one
// workgroup took 60 us for 60k flags an instance).
__device__ __forceinline__ uint32_t any_flag(const uint8_t *__restrict__ f, int lo, int hi)
{
    uint32_t any = 0;
    const int a = (int)(((uintptr_t)(f + lo) + 15) / 16 * 16 - (uintptr_t)(f + lo));
    const int first = lo + a < hi ? lo + a : hi, words = (hi - first) / 16, last = first + 16 * words;
    for (int i = lo + (int)threadIdx.x; i < first; i += 256) any |= f[i];
    const uint4 *w = reinterpret_cast<const uint4 *>(f + first);
    for (int i = threadIdx.x; i < words; i += 256) {
        const uint4 v = w[i];
        any |= v.x | v.y | v.z | v.w;
    }
    for (int i = last + (int)threadIdx.x; i < hi; i += 256) any |= f[i];
    return any;
}

// One workgroup per instance: feasible[inst] = no violated row or column.
__global__ __launch_bounds__(256) void k_mip_reduce(const InstInfo *__restrict__ info, const uint8_t *__restrict__ rbad,
                                                    const uint8_t *__restrict__ cbad, uint8_t *__restrict__ feasible)
{
    const InstInfo &I = info[blockIdx.x];
    const uint32_t any = any_flag(rbad, I.row0, I.row1) | any_flag(cbad, I.col0, I.col1);
    const int bad = __syncthreads_or(any != 0);
    if (threadIdx.x == 0) feasible[blockIdx.x] = bad ? 0 : 1;
}

// ------------------------------------------------------ host launchers
template <class V, int FMT, int DIR, int NT, int EPT>
static void launch_pass_t(const PassArgs<V> &p, int jw, hipStream_t s)
{
    if (p.early) hipLaunchKernelGGL((k_pass<V, FMT, DIR, NT, EPT>), dim3(p.ntiles), dim3(NT), 0, s, p, jw);
    else hipLaunchKernelGGL((k_pass_batch<V, FMT, DIR, NT, EPT>), dim3(p.ntiles), dim3(NT), 0, s, p, jw);
}

template <class V, int FMT, int DIR, int NT, int EPT>
static void launch_check_t(const PassArgs<V> &p, hipStream_t s)
{
    hipLaunchKernelGGL((k_check<V, FMT, DIR, NT, EPT>), dim3(p.ntiles), dim3(NT), 0, s, p);
}

// ept: nonzeros per thread of 256-thread tile workgroups (tiles of 256 ept
// nonzeros); -8 / -16: the tiles of ept 8 / 16 run by 1024-thread
// workgroups, 2 / 4 nonzeros per thread (a thread then has at most one row
// of a tile).
template <class V, int FMT, int DIR>
static void dispatch_pass(const PassArgs<V> &p, int ept, int jw, bool check, hipStream_t s)
{
    switch (ept) {
    case -8:
        check ? launch_check_t<V, FMT, DIR, 1024, 2>(p, s) : launch_pass_t<V, FMT, DIR, 1024, 2>(p, jw, s);
        break;
    case -16:
        check ? launch_check_t<V, FMT, DIR, 1024, 4>(p, s) : launch_pass_t<V, FMT, DIR, 1024, 4>(p, jw, s);
        break;
    case 1:
        check ? launch_check_t<V, FMT, DIR, 256, 1>(p, s) : launch_pass_t<V, FMT, DIR, 256, 1>(p, jw, s);
        break;
    case 2:
        check ? launch_check_t<V, FMT, DIR, 256, 2>(p, s) : launch_pass_t<V, FMT, DIR, 256, 2>(p, jw, s);
        break;
    case 4:
        check ? launch_check_t<V, FMT, DIR, 256, 4>(p, s) : launch_pass_t<V, FMT, DIR, 256, 4>(p, jw, s);
        break;
    case 8:
        check ? launch_check_t<V, FMT, DIR, 256, 8>(p, s) : launch_pass_t<V, FMT, DIR, 256, 8>(p, jw, s);
        break;
    default:
        check ? launch_check_t<V, FMT, DIR, 256, 16>(p, s) : launch_pass_t<V, FMT, DIR, 256, 16>(p, jw, s);
        break;
    }
}

// The same over sorted tiles (4096 or 8192 nonzeros, 1024 threads).
template <class V, int FMT, int DIR>
static void dispatch_sorted(const PassArgs<V> &p, int ept, int jw, bool check, hipStream_t s)
{
    if (ept == -16)
        check ? launch_check_t<V, FMT, DIR, 1024, 4>(p, s) : launch_pass_t<V, FMT, DIR, 1024, 4>(p, jw, s);
    else
        check ? launch_check_t<V, FMT, DIR, 1024, 8>(p, s) : launch_pass_t<V, FMT, DIR, 1024, 8>(p, jw, s);
}

void launch_sort_tiles(const MatView &M, int fmt, const int4 *tiles, int ntiles, int ept, uint32_t *ent, void *val,
                       uint16_t *pos, hipStream_t s)
{
    if (ntiles <= 0) return;
    const int cap = 1024 * ept;
    if (fmt == FMT_F64) {
        (void)hipFuncSetAttribute((const void *)k_sort_tiles<FMT_F64>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  8 * cap);
        hipLaunchKernelGGL(k_sort_tiles<FMT_F64>, dim3(ntiles), dim3(1024), 8 * cap, s, M, tiles, cap, ent, val, pos);
    } else {
        (void)hipFuncSetAttribute((const void *)k_sort_tiles<FMT_PACKED>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  8 * cap);
        hipLaunchKernelGGL(k_sort_tiles<FMT_PACKED>, dim3(ntiles), dim3(1024), 8 * cap, s, M, tiles, cap, ent, val, pos);
    }
}

template <class V, class A, int FMT>
static void dispatch_bpart(const PassArgs<V> &p, int ept, int jw, int check, hipStream_t s)
{
    const dim3 g(p.ntiles), b(256);
    switch (ept) {
    case -8: hipLaunchKernelGGL((k_bpart<V, A, FMT, 1024, 2>), g, dim3(1024), 0, s, p, jw, check); break;
    case -16: hipLaunchKernelGGL((k_bpart<V, A, FMT, 1024, 4>), g, dim3(1024), 0, s, p, jw, check); break;
    case 2: hipLaunchKernelGGL((k_bpart<V, A, FMT, 256, 2>), g, b, 0, s, p, jw, check); break;
    case 4: hipLaunchKernelGGL((k_bpart<V, A, FMT, 256, 4>), g, b, 0, s, p, jw, check); break;
    case 8: hipLaunchKernelGGL((k_bpart<V, A, FMT, 256, 8>), g, b, 0, s, p, jw, check); break;
    default: hipLaunchKernelGGL((k_bpart<V, A, FMT, 256, 16>), g, b, 0, s, p, jw, check); break;
    }
}

// Calls f(std::integral_constant<int, F>{}) with F the FP32 storage format
// fmt, with or without the FMT_CACHED flag.
template <class Fn>
static void fp32_format(int fmt, Fn &&f)
{
    const bool c = (fmt & FMT_CACHED) != 0;
    switch (fmt & ~FMT_CACHED) {
    case FMT_PACKED:
        if (c) f(std::integral_constant<int, FMT_PACKED | FMT_CACHED>{});
        else f(std::integral_constant<int, FMT_PACKED>{});
        break;
    case FMT_BF16:
        if (c) f(std::integral_constant<int, FMT_BF16 | FMT_CACHED>{});
        else f(std::integral_constant<int, FMT_BF16>{});
        break;
    default:
        if (c) f(std::integral_constant<int, FMT_F32 | FMT_CACHED>{});
        else f(std::integral_constant<int, FMT_F32>{});
        break;
    }
}

template <class V, class A>
static void bpart_fmt(const PassArgs<V> &p, int fmt, int ept, int jw, int check, hipStream_t s)
{
    if constexpr (sizeof(V) == 8) {
        dispatch_bpart<V, A, FMT_F64>(p, ept, jw, check, s);
    } else {
        fp32_format(fmt, [&](auto fc) { dispatch_bpart<V, A, decltype(fc)::value>(p, ept, jw, check, s); });
    }
}

template <class V>
void launch_pass(const PassArgs<V> &p, int fmt, int dir, int ept, int jw, bool check, bool blocked, hipStream_t s)
{
    if (blocked) {
        if (p.ntiles > 0) {
            if (check) bpart_fmt<V, double>(p, fmt, ept, jw, 1, s);
            else bpart_fmt<V, V>(p, fmt, ept, jw, 0, s);
        }
        if (p.nlong > 0) {
            const int nb = (p.nlong + COMB_ROWS - 1) / COMB_ROWS;
            if (check) hipLaunchKernelGGL((k_bseg<V, double>), dim3(nb), dim3(256), 0, s, p, jw, 1);
            else hipLaunchKernelGGL((k_bseg<V, V>), dim3(nb), dim3(256), 0, s, p, jw, 0);
        }
        if (p.nctiles > 0) {
            const dim3 g(p.nctiles), b(256);
            if (check) {
                if (dir == DIR_COL) hipLaunchKernelGGL((k_bcombine_check<V, DIR_COL>), g, b, 0, s, p);
                else hipLaunchKernelGGL((k_bcombine_check<V, DIR_ROW>), g, b, 0, s, p);
            } else {
                if (dir == DIR_COL) hipLaunchKernelGGL((k_bcombine<V, DIR_COL>), g, b, 0, s, p, jw);
                else hipLaunchKernelGGL((k_bcombine<V, DIR_ROW>), g, b, 0, s, p, jw);
            }
        }
        return;
    }
    if (p.ntiles > 0) {
        if (fmt & FMT_SORTED) {
            // (packed words in FP32, or FP64: the formats that are sorted)
            if constexpr (sizeof(V) == 8) {
                if (fmt & FMT_CACHED) {
                    constexpr int F = FMT_F64 | FMT_CACHED | FMT_SORTED;
                    if (dir == DIR_COL) dispatch_sorted<V, F, DIR_COL>(p, ept, jw, check, s);
                    else dispatch_sorted<V, F, DIR_ROW>(p, ept, jw, check, s);
                } else {
                    constexpr int F = FMT_F64 | FMT_SORTED;
                    if (dir == DIR_COL) dispatch_sorted<V, F, DIR_COL>(p, ept, jw, check, s);
                    else dispatch_sorted<V, F, DIR_ROW>(p, ept, jw, check, s);
                }
            } else if (fmt & FMT_CACHED) {
                constexpr int F = FMT_PACKED | FMT_CACHED | FMT_SORTED;
                if (dir == DIR_COL) dispatch_sorted<V, F, DIR_COL>(p, ept, jw, check, s);
                else dispatch_sorted<V, F, DIR_ROW>(p, ept, jw, check, s);
            } else {
                constexpr int F = FMT_PACKED | FMT_SORTED;
                if (dir == DIR_COL) dispatch_sorted<V, F, DIR_COL>(p, ept, jw, check, s);
                else dispatch_sorted<V, F, DIR_ROW>(p, ept, jw, check, s);
            }
        } else if constexpr (sizeof(V) == 8) {
            if (fmt & FMT_CACHED) {
                constexpr int F = FMT_F64 | FMT_CACHED;
                if (dir == DIR_COL) dispatch_pass<V, F, DIR_COL>(p, ept, jw, check, s);
                else dispatch_pass<V, F, DIR_ROW>(p, ept, jw, check, s);
            } else {
                if (dir == DIR_COL) dispatch_pass<V, FMT_F64, DIR_COL>(p, ept, jw, check, s);
                else dispatch_pass<V, FMT_F64, DIR_ROW>(p, ept, jw, check, s);
            }
        } else {
            fp32_format(fmt, [&](auto fc) {
                constexpr int F = decltype(fc)::value;
                if (dir == DIR_COL) dispatch_pass<V, F, DIR_COL>(p, ept, jw, check, s);
                else dispatch_pass<V, F, DIR_ROW>(p, ept, jw, check, s);
            });
        }
    }
    if (p.nlong > 0) {
        const int nb = (p.nlong + COMB_ROWS - 1) / COMB_ROWS;
        if (check) {
            if (dir == DIR_COL) hipLaunchKernelGGL((k_combine_check<V, DIR_COL>), dim3(nb), dim3(256), 0, s, p);
            else hipLaunchKernelGGL((k_combine_check<V, DIR_ROW>), dim3(nb), dim3(256), 0, s, p);
        } else {
            if (dir == DIR_COL) hipLaunchKernelGGL((k_combine<V, DIR_COL>), dim3(nb), dim3(256), 0, s, p, jw);
            else hipLaunchKernelGGL((k_combine<V, DIR_ROW>), dim3(nb), dim3(256), 0, s, p, jw);
        }
    }
}

template <class V, int FMT, int DIR, int EPT, bool PF>
static void staged_v(const PassArgs<V> &p, int jw, size_t shmem, hipStream_t s, bool prepare)
{
    auto fn = k_spass<V, FMT, DIR, SPASS_NT, EPT, PF>;
    if (prepare) {
        (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        return;
    }
    hipLaunchKernelGGL(fn, dim3(p.ntiles), dim3(SPASS_NT), shmem, s, p, jw);
}

template <class V, int FMT, int DIR>
static void staged_t(const PassArgs<V> &p, int variant, int jw, size_t shmem, hipStream_t s, bool prepare)
{
    // variant bits: 1 = prefetch row bounds and operands, 2 = 8 nonzeros per
    // thread (else 4)
    switch (variant & 3) {
    case 0: staged_v<V, FMT, DIR, 4, false>(p, jw, shmem, s, prepare); break;
    case 1: staged_v<V, FMT, DIR, 4, true>(p, jw, shmem, s, prepare); break;
    case 2: staged_v<V, FMT, DIR, 8, false>(p, jw, shmem, s, prepare); break;
    default: staged_v<V, FMT, DIR, 8, true>(p, jw, shmem, s, prepare); break;
    }
}

template <class V>
void launch_staged(const PassArgs<V> &p, int fmt, int dir, int variant, int jw, size_t shmem, hipStream_t s,
                   bool prepare)
{
    if (!prepare && p.ntiles <= 0) return;
    if constexpr (sizeof(V) == 8) {
        if (dir == DIR_COL) staged_t<V, FMT_F64, DIR_COL>(p, variant, jw, shmem, s, prepare);
        else staged_t<V, FMT_F64, DIR_ROW>(p, variant, jw, shmem, s, prepare);
    } else {
        fp32_format(fmt, [&](auto fc) {
            constexpr int F = decltype(fc)::value;
            if (dir == DIR_COL) staged_t<V, F, DIR_COL>(p, variant, jw, shmem, s, prepare);
            else staged_t<V, F, DIR_ROW>(p, variant, jw, shmem, s, prepare);
        });
    }
}

template <class V, int FMT, int DIR, int K>
void direct_k(const PassArgs<V> &p, int jw, size_t shmem, hipStream_t s, bool prepare)
{
    auto fn = k_dpass<V, FMT, DIR, DPASS_NT, K>;
    if (prepare) {
        (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        return;
    }
    hipLaunchKernelGGL(fn, dim3(p.ndtiles), dim3(DPASS_NT), shmem, s, p, jw);
}

template <class V, int FMT, int DIR>
void direct_t(const PassArgs<V> &p, int k, int jw, size_t shmem, hipStream_t s, bool prepare)
{
    if (k <= 2) direct_k<V, FMT, DIR, 2>(p, jw, shmem, s, prepare);
    else if (k <= 4) direct_k<V, FMT, DIR, 4>(p, jw, shmem, s, prepare);
    else direct_k<V, FMT, DIR, 8>(p, jw, shmem, s, prepare);
}

template <class V>
void launch_direct(const PassArgs<V> &p, int fmt, int dir, int k, int jw, size_t shmem, hipStream_t s,
                   bool prepare)
{
    if (!prepare && p.ndtiles <= 0) return;
    if constexpr (sizeof(V) == 8) {
        if (dir == DIR_COL) direct_t<V, FMT_F64, DIR_COL>(p, k, jw, shmem, s, prepare);
        else direct_t<V, FMT_F64, DIR_ROW>(p, k, jw, shmem, s, prepare);
    } else {
        fp32_format(fmt, [&](auto fc) {
            constexpr int F = decltype(fc)::value;
            if (dir == DIR_COL) direct_t<V, F, DIR_COL>(p, k, jw, shmem, s, prepare);
            else direct_t<V, F, DIR_ROW>(p, k, jw, shmem, s, prepare);
        });
    }
}

template <class V>
void launch_combine(const PassArgs<V> &p, int dir, int jw, hipStream_t s)
{
    if (p.nctiles <= 0) return;
    const dim3 g(p.nctiles), b(256);
    if (dir == DIR_COL) hipLaunchKernelGGL((k_bcombine<V, DIR_COL>), g, b, 0, s, p, jw);
    else hipLaunchKernelGGL((k_bcombine<V, DIR_ROW>), g, b, 0, s, p, jw);
}

void launch_step(const StepArgs &a, int count, hipStream_t s)
{
    if (count > 0) hipLaunchKernelGGL(k_step, dim3(count), dim3(STEP_NT), 0, s, a);
}

void launch_decide(const DecideArgs &d, int count, hipStream_t s)
{
    hipLaunchKernelGGL(k_decide, dim3(count), dim3(DECIDE_NT), 0, s, d);
}

template <class V>
void launch_take_avg(const InstState *st, const InstInfo *info, V *x, V *y, const V *xa, const V *ya, double *ax,
                     const double *axa, int count, int longest, hipStream_t s)
{
    // about 2048 columns a workgroup, at most 256 workgroups an instance (a
    // workgroup for each of a 5k x 10k instance took 7 us), and all in all no
    // more than 2^20 beyond one an instance: a grid is limited to 2^32 threads,
    // and with that many instances the others fill the chip
    if (count <= 0) return;
    int blocks = (longest + 2047) / 2048;
    blocks = std::min({blocks, 256, (1 << 20) / count});
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_take_avg<V>, dim3((unsigned)count * (unsigned)blocks), dim3(256), 0, s, st, info, x, y, xa, ya, ax, axa,
                       blocks);
}

void launch_force_stop(InstState *st, int count, hipStream_t s)
{
    hipLaunchKernelGGL(k_force_stop, dim3((count + 255) / 256), dim3(256), 0, s, st, count);
}

void launch_scale_round(ScaleArgs a, int fmt, hipStream_t s)
{
    auto blocks = [](int len, int L) { return (len + 256 / L - 1) / (256 / L); };
    a.rblocks = blocks(a.M, a.LR);
    const dim3 g((unsigned)(a.rblocks + blocks(a.N, a.LC))), b(256);
    switch (fmt) {
    case FMT_PACKED: hipLaunchKernelGGL(k_scale_round<FMT_PACKED>, g, b, 0, s, a); break;
    case FMT_BF16: hipLaunchKernelGGL(k_scale_round<FMT_BF16>, g, b, 0, s, a); break;
    case FMT_F32: hipLaunchKernelGGL(k_scale_round<FMT_F32>, g, b, 0, s, a); break;
    default: hipLaunchKernelGGL(k_scale_round<FMT_F64>, g, b, 0, s, a); break;
    }
}

template <class V>
void launch_setup_vectors(const SetupArgs<V> &a, hipStream_t s)
{
    const int len = a.N > a.M ? a.N : a.M;
    if (len > 0) hipLaunchKernelGGL(k_setup_vectors<V>, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, a);
}

void launch_norms(const NormArgs &a, hipStream_t s)
{
    if (a.q1 <= a.q0) return;
    hipLaunchKernelGGL((k_norm_part<double, NORM_KEEP>), dim3((unsigned)a.pieces), dim3(256), 0, s, a, BlendArgs{});
}

template <class V>
void launch_blend(const NormArgs &a, const BlendArgs &b, hipStream_t s)
{
    hipLaunchKernelGGL((k_norm_part<V, NORM_BLEND>), dim3((unsigned)a.pieces), dim3(256), 0, s, a, b);
}

template <class V>
void launch_objective(const NormArgs &a, const double *src, V *cv, hipStream_t s)
{
    BlendArgs b{};
    b.c_orig = src;
    b.cv = cv;
    hipLaunchKernelGGL((k_norm_part<V, NORM_STAGED>), dim3((unsigned)a.pieces), dim3(256), 0, s, a, b);
}

// dst = src, dst_v = src in the path precision.
template <class V>
__global__ __launch_bounds__(256) void k_put(const double *src, double *dst, V *dst_v, int len)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    const double v = src[i];
    dst[i] = v;
    dst_v[i] = (V)v;
}

template <class V>
void launch_put(const double *src, double *dst, V *dst_v, int len, hipStream_t s)
{
    if (len > 0)
        hipLaunchKernelGGL(k_put<V>, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, src, dst, dst_v, len);
}

template <class V>
void launch_cast(const double *src, V *dst, int len, hipStream_t s)
{
    if (len > 0) hipLaunchKernelGGL(k_cast<V>, dim3((len + 255) / 256), dim3(256), 0, s, src, dst, len);
}

template <class V>
void launch_project(V *x, const V *l, const V *u, int clo, int chi, V *y, const uint8_t *sense, int rlo, int rhi,
                    hipStream_t s)
{
    const int nc = chi - clo, nr = rhi - rlo, len = nc > nr ? nc : nr;
    if (len > 0)
        hipLaunchKernelGGL(k_project<V>, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, x, l, u, clo, nc, y, sense,
                           rlo, nr);
}

template <class V>
void launch_mip_check(const MatView &M, int fmt, int m, int n, int count, const InstInfo *info, const V *x,
                      const double *b, const uint8_t *sense, const double *l, const double *u,
                      const uint8_t *is_int, double tol, uint8_t *rbad, uint8_t *cbad, uint8_t *feasible,
                      hipStream_t s)
{
    if (m > 0) {
        dim3 g((m + 256 / MIP_L - 1) / (256 / MIP_L)), bl(256);
        if constexpr (sizeof(V) == 8) {
            hipLaunchKernelGGL((k_mip_rows<V, FMT_F64>), g, bl, 0, s, M, m, x, b, sense, tol, rbad);
        } else {
            switch (fmt) {
            case FMT_PACKED: hipLaunchKernelGGL((k_mip_rows<V, FMT_PACKED>), g, bl, 0, s, M, m, x, b, sense, tol, rbad); break;
            case FMT_BF16: hipLaunchKernelGGL((k_mip_rows<V, FMT_BF16>), g, bl, 0, s, M, m, x, b, sense, tol, rbad); break;
            default: hipLaunchKernelGGL((k_mip_rows<V, FMT_F32>), g, bl, 0, s, M, m, x, b, sense, tol, rbad); break;
            }
        }
    }
    if (n > 0)
        hipLaunchKernelGGL(k_mip_cols<V>, dim3((n + 255) / 256), dim3(256), 0, s, x, l, u, is_int, tol, n, cbad);
    if (count > 0) hipLaunchKernelGGL(k_mip_reduce, dim3(count), dim3(256), 0, s, info, rbad, cbad, feasible);
}

#define SCY_INST(V)                                                                                    \
    template void launch_tiny<V>(const TinyArgs<V> &, int, int, int, int, size_t, hipStream_t, bool);  \
    template void launch_staged<V>(const PassArgs<V> &, int, int, int, int, size_t, hipStream_t, bool); \
    template void launch_pass<V>(const PassArgs<V> &, int, int, int, int, bool, bool, hipStream_t);    \
    template void launch_combine<V>(const PassArgs<V> &, int, int, hipStream_t);                       \
    template void launch_direct<V>(const PassArgs<V> &, int, int, int, int, size_t, hipStream_t, bool); \
    template void launch_setup_vectors<V>(const SetupArgs<V> &, hipStream_t);                          \
    template void launch_take_avg<V>(const InstState *, const InstInfo *, V *, V *, const V *, const V *, \
                                     double *, const double *, int, int, hipStream_t);                      \
    template void launch_begin<V>(const BeginArgs<V> &, hipStream_t);                                  \
    template void launch_start<V>(const StartArgs<V> &, int *, hipStream_t);                           \
    template void launch_cast<V>(const double *, V *, int, hipStream_t);                               \
    template void launch_project<V>(V *, const V *, const V *, int, int, V *, const uint8_t *, int, int, \
                                    hipStream_t);                                                      \
    template void launch_blend<V>(const NormArgs &, const BlendArgs &, hipStream_t);                   \
    template void launch_objective<V>(const NormArgs &, const double *, V *, hipStream_t);             \
    template void launch_put<V>(const double *, double *, V *, int, hipStream_t);                      \
    template void launch_mip_check<V>(const MatView &, int, int, int, int, const InstInfo *, const V *, \
                                      const double *, const uint8_t *, const double *, const double *, \
                                      const uint8_t *, double, uint8_t *, uint8_t *, uint8_t *, hipStream_t);
SCY_INST(float)
SCY_INST(double)

}  // namespace scy
