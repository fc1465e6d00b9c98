// Device tables of a batched call (pairs, their splits, the product's groups),
// built on the device from a compact description.
//
// A pair's entries take 176 bytes, which went up as chains of 3 KB
// kernel-argument copies, 7 us each one after the other: 37 copies (270 us)
// ahead of the first kernel for 1024 pairs.  Everything in them follows from
// the pairs' sizes (4 bytes a pair) by prefix sums, and the product's
// largest-first order (2 bytes); row offsets, split counts, Philox words and
// split owners follow from the position unless the call's differ.  One copy per
// 512 pairs and one work-group's scans, 512 pairs at a time (bound by their
// latency: 6 us for 64 pairs, 18 us for 1024).  The call of 1024 pairs at d = 256
// with 200 splits each went from 1175 to 925 us.
#include "hbt_launch.h"

namespace hbt {

constexpr int kTabThreads = 512;

// Exclusive prefix sum over the work-group; every thread gets the total.
__device__ __forceinline__ int64_t tab_scan(int64_t x, int64_t* sh, int64_t* total) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    long long v = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    __syncthreads();  // the previous scan's readers are done with sh
    if (lane == 63) sh[wave] = v;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kTabThreads / 64; ++q) {
        const int64_t t = sh[q];
        before += q < wave ? t : 0;
        all += t;
    }
    *total = all;
    return before + v - x;
}

template <typename T>
__device__ __forceinline__ T tab_at(const TableArgs& A, int32_t off, int64_t i) {
    return ((const T*)(A.blob + off))[i];
}
// entry i of an index list of 2 or 4 bytes an entry
__device__ __forceinline__ int tab_index(const TableArgs& A, int32_t off, int64_t i, bool narrow) {
    return narrow ? (int)tab_at<uint16_t>(A, off, i) : (int)tab_at<uint32_t>(A, off, i);
}

__global__ __launch_bounds__(kTabThreads) void k_build_tables(TableArgs A) {
    __shared__ int64_t sh[kTabThreads / 64];
    const int t = threadIdx.x;
    int64_t tot;
    // 1. shared clouds: one run of storage each
    {
        int64_t row = 0, zrow = 0, chunk = 0;
        for (int c0 = 0; c0 < A.nclouds; c0 += kTabThreads) {
            const int c = c0 + t;
            const bool in = c < A.nclouds;
            const int64_t m = in ? tab_at<uint32_t>(A, A.o_cloud_rows, c) : 0;
            const int64_t Np = (m + kRowPad - 1) / kRowPad * kRowPad;
            const int64_t r = row + tab_scan(m, sh, &tot);
            row += tot;
            const int64_t z = zrow + tab_scan(Np, sh, &tot);
            zrow += tot;
            const int64_t k = chunk + tab_scan(Np / kSumChunkY, sh, &tot);
            chunk += tot;
            if (in) {
                const int64_t first = A.o_offset >= 0 ? tab_at<int64_t>(A, A.o_offset, c) : A.offset0 + r;
                PairDesc cd = {};
                cd.X = cd.Y = A.base + first * A.row_bytes;
                cd.m = (int32_t)m;
                cd.Np = (int32_t)Np;
                cd.Wp = (int32_t)(Np / 32);
                cd.zrow0 = cd.zrow_y = z;
                cd.nxc = (int32_t)(Np / kRowPad);
                cd.cx0 = cd.cx1 = cd.cy0 = (int32_t)k;
                cd.cy1 = (int32_t)(k + Np / kSumChunkY);
                A.cdesc[c] = cd;
            }
        }
        __syncthreads();  // the clouds' entries are read below
    }
    // 2. pairs and their splits
    int64_t row = 0, zrow = 0, coef = 0, chunk = 0, xoct = 0, srow = 0, word = 0, nbig = 0, bigrow = 0;
    for (int p0 = 0; p0 < A.npairs; p0 += kTabThreads) {
        const int p = p0 + t;
        const bool in = p < A.npairs;
        PairDesc pd = {};
        int64_t B = 0;
        int owner = p;
        if (in) {
            B = A.o_splits >= 0 ? tab_at<uint32_t>(A, A.o_splits, p) : A.splits0;
            if (A.o_owner >= 0) owner = (int)tab_at<uint32_t>(A, A.o_owner, p);
            pd.pair_index = A.o_index >= 0 ? tab_at<uint32_t>(A, A.o_index, p) : A.index0 + (uint32_t)p;
            if (A.nclouds) {
                const PairDesc cx = A.cdesc[tab_index(A, A.o_pair_x, p, A.narrow_clouds)];
                const PairDesc cy = A.cdesc[tab_index(A, A.o_pair_y, p, A.narrow_clouds)];
                pd.X = cx.X;
                pd.Y = cy.X;
                pd.n = cx.m;
                pd.m = cy.m;
                pd.Np = cx.Np + cy.Np;
                pd.zrow0 = cx.zrow0;
                pd.zrow_y = cy.zrow0;
                pd.nxc = cx.Np / kRowPad;
                pd.ygap = cx.Np - cx.m;
                pd.cx0 = cx.cx1;
                pd.cx1 = cx.cy1;
                pd.cy0 = cy.cx1;
                pd.cy1 = cy.cy1;
            } else {
                const uint32_t nm = tab_at<uint32_t>(A, A.o_sizes, p);
                pd.n = (int32_t)(nm & 0xffffu);
                pd.m = (int32_t)(nm >> 16);
                pd.Np = (pd.n + pd.m + kRowPad - 1) / kRowPad * kRowPad;
                pd.nxc = pd.Np / kRowPad;
            }
            pd.Wp = pd.Np / 32;
            pd.flip = pd.m < pd.n ? 1 : 0;
        }
        const int64_t nx = in ? (pd.n + kSumChunk - 1) / kSumChunk : 0;
        const int64_t ny = in ? pd.Np / kSumChunkY - pd.n / kSumChunkY : 0;
        pd.coef0 = coef + tab_scan(pd.n, sh, &tot);
        coef += tot;
        if (!A.nclouds) {
            const int64_t r = row + tab_scan(pd.n + pd.m, sh, &tot);
            row += tot;
            pd.zrow0 = pd.zrow_y = zrow + tab_scan(pd.Np, sh, &tot);
            zrow += tot;
            pd.cx0 = (int32_t)(chunk + tab_scan(nx + ny, sh, &tot));
            chunk += tot;
            pd.cx1 = pd.cy0 = (int32_t)(pd.cx0 + nx);
            pd.cy1 = (int32_t)(pd.cx1 + ny);
            pd.xoct0 = xoct + tab_scan(in ? x_octets(pd.n) : 0, sh, &tot);
            xoct += tot;
            if (in) {
                const int64_t first = A.o_offset >= 0 ? tab_at<int64_t>(A, A.o_offset, p) : A.offset0 + r;
                pd.X = A.base + first * A.row_bytes;
                pd.Y = A.base + (first + pd.n) * A.row_bytes;
            }
        }
        BlockPair b;
        b.mrow0 = srow + tab_scan(B, sh, &tot);
        srow += tot;
        b.mword0 = word + tab_scan(owner == p ? B * pd.Wp : 0, sh, &tot);
        word += tot;
        b.perm_base = A.perm_base;
        b.nb = (int32_t)B;
        b.owner = owner;
        b.n = pd.n;
        b.m = pd.m;
        b.Wp = pd.Wp;
        b.pair_index = pd.pair_index;
        b.ygap = pd.ygap;
        const bool big = in && pd.Np > kQuadItems;
        const int64_t kb = nbig + tab_scan(big ? 1 : 0, sh, &tot);
        nbig += tot;
        const int64_t rb = bigrow + tab_scan(big ? B : 0, sh, &tot);
        bigrow += tot;
        if (big) {
            A.big_pair[kb] = p;
            A.big_row0[kb] = rb;
        }
        if (in) {
            A.pairs[p] = pd;
            A.bp[p] = b;
            A.Btot[p] = B;
            A.nflag[p] = 0u;
            A.sstat[p] = 0;
            A.ticket[p] = 0u;
            if (A.rcnt) A.rcnt[p] = 0u;
        }
        __syncthreads();
        if (in && owner != p) A.bp[p].mword0 = A.bp[owner].mword0;  // an earlier pair's masks
    }
    if (t == 0 && (A.npairs & 1)) A.nflag[A.npairs] = 0u;  // the odd word (a single pair's ticket)
    // 3. the product's groups: ngw of the wide tiles, then the others, tiles
    //    numbered from 0 in each
    for (int part = 0; part < 2; ++part) {
        const int g0 = part ? A.ngw : 0, g1 = part ? A.ngroups : A.ngw;
        const int width = part ? A.width_narrow : A.width_wide;
        int64_t tile = 0;
        for (int gb = g0; gb < g1; gb += kTabThreads) {
            const int g = gb + t;
            GemmGroup q = {0, 0, 0};
            if (g < g1) {
                q.pair = tab_index(A, A.o_order, g, A.narrow_order);
                const int64_t B = A.o_splits >= 0 ? tab_at<uint32_t>(A, A.o_splits, q.pair) : A.splits0;
                q.nbt = (int32_t)((B + width - 1) / width);
            }
            q.tile0 = tile + tab_scan((int64_t)q.nbt * A.nslot, sh, &tot);
            tile += tot;
            if (g < g1) A.groups[g] = q;
        }
    }
}

hipError_t launch_build_tables(const TableArgs& A, hipStream_t s) {
    if (A.npairs < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_build_tables, dim3(1), dim3(kTabThreads), 0, s, A);
    return hipGetLastError();
}

}  // namespace hbt
