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
// latency: 6.1 us for 64 pairs, 16 for 1024).  The call of 1024 pairs at d = 256
// with 200 splits each went from 1175 to 925 us.
#include "hbt_launch.h"

namespace hbt {

constexpr int kTabThreads = 512;

template <typename T>
__device__ __forceinline__ T tab_at(const TableArgs& A, int32_t off, int64_t i) {
    return ((const T*)(A.blob + off))[i];
}
// entry i of an index list of 2 or 4 bytes an entry
__device__ __forceinline__ int tab_index(const TableArgs& A, int32_t off, int64_t i, bool narrow) {
    return narrow ? (int)tab_at<uint16_t>(A, off, i) : (int)tab_at<uint32_t>(A, off, i);
}

__global__ __launch_bounds__(kTabThreads) void k_build_tables(TableArgs A) {
    constexpr int kScans = 9;  // of a pair
    __shared__ int64_t sh[kScans][kTabThreads / 64];
    const int t = threadIdx.x;
    // 1. shared clouds: one run of storage each
    {
        int64_t row = 0, zrow = 0, chunk = 0;
        for (int c0 = 0; c0 < A.nclouds; c0 += kTabThreads) {
            const int c = c0 + t;
            const bool in = c < A.nclouds;
            const int64_t m = in ? tab_at<uint32_t>(A, A.o_cloud_rows, c) : 0;
            const int64_t Np = (m + kRowPad - 1) / kRowPad * kRowPad;
            int64_t x[3] = {m, Np, Np / kSumChunkY}, tot[3];
            block_scan<kTabThreads>(x, sh, tot);
            const int64_t r = row + x[0], z = zrow + x[1], k = chunk + x[2];
            row += tot[0];
            zrow += tot[1];
            chunk += tot[2];
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
        const bool big = in && pd.Np > kQuadItems;
        int64_t x[kScans] = {pd.n, pd.n + pd.m, pd.Np, nx + ny, in ? x_octets(pd.n) : 0,
                             B, owner == p ? B * pd.Wp : 0, big ? 1 : 0, big ? B : 0}, tot[kScans];
        block_scan<kTabThreads>(x, sh, tot);
        pd.coef0 = coef + x[0];
        coef += tot[0];
        if (!A.nclouds) {
            pd.zrow0 = pd.zrow_y = zrow + x[2];
            pd.cx0 = (int32_t)(chunk + x[3]);
            pd.cx1 = pd.cy0 = (int32_t)(pd.cx0 + nx);
            pd.cy1 = (int32_t)(pd.cx1 + ny);
            pd.xoct0 = xoct + x[4];
            if (in) {
                const int64_t first = A.o_offset >= 0 ? tab_at<int64_t>(A, A.o_offset, p) : A.offset0 + row + x[1];
                pd.X = A.base + first * A.row_bytes;
                pd.Y = A.base + (first + pd.n) * A.row_bytes;
            }
        }
        row += tot[1];
        zrow += tot[2];
        chunk += tot[3];
        xoct += tot[4];
        BlockPair b;
        b.mrow0 = srow + x[5];
        b.mword0 = word + x[6];
        b.perm_base = A.perm_base;
        b.nb = (int32_t)B;
        b.owner = owner;
        b.n = pd.n;
        b.m = pd.m;
        b.Wp = pd.Wp;
        b.pair_index = pd.pair_index;
        b.ygap = pd.ygap;
        const int64_t kb = nbig + x[7], rb = bigrow + x[8];
        srow += tot[5];
        word += tot[6];
        nbig += tot[7];
        bigrow += tot[8];
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
    int64_t wide = 0, narrow = 0;
    for (int gb = 0; gb < A.ngroups; gb += kTabThreads) {
        const int g = gb + t;
        GemmGroup q = {0, 0, 0};
        if (g < A.ngroups) {
            const int width = g < A.ngw ? A.width_wide : A.width_narrow;
            q.pair = tab_index(A, A.o_order, g, A.narrow_order);
            const int64_t B = A.o_splits >= 0 ? tab_at<uint32_t>(A, A.o_splits, q.pair) : A.splits0;
            q.nbt = (int32_t)((B + width - 1) / width);
        }
        const int64_t tiles = (int64_t)q.nbt * A.nslot;
        int64_t x[2] = {g < A.ngw ? tiles : 0, g < A.ngw ? 0 : tiles}, tot[2];
        block_scan<kTabThreads>(x, sh, tot);
        q.tile0 = g < A.ngw ? wide + x[0] : narrow + x[1];
        wide += tot[0];
        narrow += tot[1];
        if (g < A.ngroups) A.groups[g] = q;
    }
}

hipError_t launch_build_tables(const TableArgs& A, hipStream_t s) {
    if (A.npairs < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_build_tables, dim3(1), dim3(kTabThreads), 0, s, A);
    return hipGetLastError();
}

}  // namespace hbt
