// Random splits of the pooled set into groups of sizes (n, m): the "randomly
// partition Z" step of Algorithm 1 / the sign-matrix rows of Algorithm 2,
// stored as a 0/1 bit mask of group 1.
//
// Split b of a pair puts in group 1 the n items first in the order
// (P_i, S_i, i): P_i an 8-bit primary key, S_i a 32-bit secondary key, both
// from Philox4x32-10 (counter (i/16, b, pair, 0) and (i/4, b, pair, 1)).
// Selection without a sort: a 256-bin histogram of P finds the byte theta
// holding rank n-1; items with P < theta are in; the ~N/256 items with
// P == theta are ranked by (S_i, i) and the first n - #{P < theta} join.
// Only those bucket items ever need a secondary key.
//
// Two kernels: pairs of up to kQuadItems pooled items are drawn four split rows
// a wavefront, larger pairs one; a launch of both kinds of pairs runs both, each
// skipping the other's rows.  Waves of a work-group are independent and
// synchronise only within themselves.
#include <atomic>

#include "hbt_launch.h"

namespace hbt {

__device__ __forceinline__ uint32_t word_of(uint4 w, int k) {
    return k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
}

// Per-wave LDS carve-up (bytes), for pairs with up to max_np pooled rows:
// the 256-bin histogram, the bucket items (index, secondary key) and the
// split's mask row.
// (The 256-bin histograms live in a static array, one per wave, so that a
// bin's LDS address is the key times 4 plus a constant.)
struct SplitLds {
    int cidx, ckey, mlds, total;
    __host__ __device__ SplitLds(int max_np) {
        cidx = 0;
        ckey = cidx + 4 * kCandCap;
        mlds = ckey + 4 * kCandCap;
        total = mlds + max_np / 8;
    }
};
constexpr int kSplitWaves = 4;          // waves (split rows) per work-group
constexpr int kSplitStaticLds = kSplitWaves * (1024 + 4);

// hist[W][key] += 1 for the 16 keys of a block.  The wave's histogram offset
// W * 1024 goes into the LDS instruction's immediate offset, so that a key
// costs one VALU operation (its byte times 4) besides the LDS add.  (Written
// as inline asm: with plain atomics the compiler merges the four waves' code
// paths and adds the offset in a register.  An add without return writes no
// register, and one wave's LDS operations complete in issue order, so the
// later reads of the histogram see every add.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF>
__device__ __forceinline__ void lds_inc(uint32_t addr, uint32_t one) {
    asm volatile("ds_add_u32 %0, %1 offset:%2" : : "v"(addr), "v"(one), "i"(OFF) : "memory");
}
// The LDS word's value before adding one to it (a place in a list), waited for
// here: with atomicAdd the compiler elects one lane and counts the others, more
// vector instructions than the one or two lanes that usually want a place.
__device__ __forceinline__ uint32_t lds_take(uint32_t* word) {
    uint32_t pos;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(pos)
                 : "v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)word), "v"(1u)
                 : "memory");
    return pos;
}
#pragma clang diagnostic pop
template <int W>
__device__ __forceinline__ void count_block(uint32_t (*hist)[256], uint4 w) {
    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)&hist[0][0];
    const uint32_t one = 1u;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        lds_inc<W * 1024>(base + (((word_of(w, j >> 2) >> (8 * (j & 3))) & 0xffu) << 2), one);
}

// The bits 7 of the four bytes of each of a block's words (f(word) in w.x .. w.w
// order), gathered to 16 bits: bit 4 q + b from byte b of word q, item 4 q + b of
// the block.  Per word, one product moves its four bits to the top nibble (the
// partial products fall on distinct bits, so nothing carries into it) and one
// funnel shift appends the nibble.
template <typename F>
__device__ __forceinline__ uint32_t gather_bits7(uint4 w, F f) {
    uint32_t acc = 0u;
#pragma unroll
    for (int q = 3; q >= 0; --q)
        acc = __builtin_amdgcn_alignbit(acc, (f(word_of(w, q)) & 0x80808080u) * 0x00204081u, 28);
    return acc;
}

// Bit j of the result = [key j of the block < theta] (theta4: theta in every
// byte), four bytes at a time: for each byte x and t = theta,
//   x < t  <=>  (x7 = 0 and t7 = 1) or (x7 = t7 and (x & 127) < (t & 127)),
// where (x & 127) + (128 - (t & 127)) has bit 7 set exactly when
// (x & 127) >= (t & 127) (no carry leaves the byte); one three-input logic
// operation combines the three conditions in bit 7.
__device__ __forceinline__ uint32_t below_theta(uint4 w, uint32_t theta4) {
    const uint32_t k = 0x80808080u - (theta4 & 0x7f7f7f7fu);  // per byte 128 - (t & 127)
    // truth table of (~x & t) | (~(x ^ t) & ~s) over the operands (x, t, s)
    constexpr unsigned kTT = ((~0xF0u & 0xCCu) | (~(0xF0u ^ 0xCCu) & ~0xAAu)) & 0xffu;
    return gather_bits7(w, [&](uint32_t x) {
        return __builtin_amdgcn_bitop3_b32(x, theta4, (x & 0x7f7f7f7fu) + k, (unsigned char)kTT);
    });
}

// Bit j of the result = [key j of the block == theta].
__device__ __forceinline__ uint32_t equal_theta(uint4 w, uint32_t theta4) {
    return gather_bits7(w, [&](uint32_t x) {
        const uint32_t y = x ^ theta4;
        return ~(((y & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y);
    });
}

// A finished mask row from LDS to memory.
__device__ __forceinline__ void write_mask_row(uint32_t* out, const uint32_t* mlds, const BlockPair& pd) {
    const int lane = threadIdx.x & 63;
    if (pd.ygap == 0) {
        for (int w = lane; w < pd.Wp; w += 64) out[w] = mlds[w];
        return;
    }
    // two-run storage: X's items keep their positions, Y's move ygap
    // positions on (X's padding in between); n + ygap is a multiple of 128
    const int ys = pd.n + pd.ygap;
    for (int w = lane; w < pd.Wp; w += 64) {
        uint32_t x;
        if (32 * w < ys) {
            x = mlds[w] & range_bits(w, 0, pd.n);
        } else {
            const int p0 = 32 * w - pd.ygap, q = p0 >> 5, sh = p0 & 31;
            const uint32_t a = mlds[q], b = q + 1 < pd.Wp ? mlds[q + 1] : 0u;
            x = sh ? (a >> sh) | (b << (32 - sh)) : a;
            x &= range_bits(w, ys, ys + pd.m);
        }
        out[w] = x;
    }
}

// Philox block c of split b: the primary keys of items 16c .. 16c+15 as 16
// little-endian bytes.
__device__ __forceinline__ uint4 primary_block(int c, uint32_t b, uint32_t pair, uint32_t k0, uint32_t k1) {
    return philox4x32_10(make_uint4((uint32_t)c, b, pair, 0u), k0, k1);
}
// The pair's last block holds lim (1 .. 16) items; the keys past them become
// 0xFF: they are taken out of the histogram's top bin afterwards and never enter
// group 1.
__device__ __forceinline__ uint4 pad_block(uint4 w, int lim) {
    auto fill = [&](int base) {  // wave-uniform
        const int v = lim - base;
        return v >= 4 ? 0u : v <= 0 ? 0xffffffffu : 0xffffffffu << (8 * v);
    };
    return make_uint4(w.x | fill(0), w.y | fill(4), w.z | fill(8), w.w | fill(12));
}

// One split row.  R > 0: each lane keeps its (at most R) Philox blocks in
// registers between the histogram and the classification pass (pairs with N
// <= 1024 R); R == 0: the blocks are generated again.
template <int R>
__device__ __forceinline__ void split_row(const BlockPair& pd, int p, int64_t row, int max_np, uint32_t key0,
                                          uint32_t key1, uint32_t* __restrict__ mask, int32_t* sstat,
                                          uint32_t (*hist_all)[256], uint32_t* nlist, unsigned char* smem) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, N = pd.n + pd.m;
    const SplitLds L(max_np);
    unsigned char* base = smem + wave * L.total;
    uint32_t* hist = hist_all[wave];
    uint32_t* cidx = (uint32_t*)(base + L.cidx);
    uint32_t* ckey = (uint32_t*)(base + L.ckey);
    uint32_t* mlds = (uint32_t*)(base + L.mlds);
    const uint32_t b = pd.perm_base + (uint32_t)(row - pd.mrow0);
    const int n = pd.n;
    const int nc = (N + 15) >> 4;       // Philox blocks holding items
    const int nw = pd.Wp * 2;           // blocks covering the padded mask row (Np / 16)
    const int niter = (nw + 63) >> 6;   // wave-uniform

    ((uint4*)hist)[lane] = make_uint4(0u, 0u, 0u, 0u);
    if (lane == 0) *nlist = 0u;
    wave_sync();
    // 1. primary keys and their histogram
    constexpr int RK = R > 0 ? R : 1;
    uint4 key[RK];
    auto gen_count = [&](int k) {
        const int c = 64 * k + lane;
        uint4 w = make_uint4(0u, 0u, 0u, 0u);
        if (c < nc) {
            w = primary_block(c, b, pd.pair_index, key0, key1);
            if (c == nc - 1) w = pad_block(w, N - 16 * (nc - 1));
            switch (wave) {  // wave-uniform
                case 0: count_block<0>(hist_all, w); break;
                case 1: count_block<1>(hist_all, w); break;
                case 2: count_block<2>(hist_all, w); break;
                default: count_block<3>(hist_all, w); break;
            }
        }
        return w;
    };
    if constexpr (R > 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) key[k] = k < niter ? gen_count(k) : make_uint4(0u, 0u, 0u, 0u);
    } else {
        for (int k = 0; k < niter; ++k) (void)gen_count(k);
    }
    wave_sync();
    // 2. theta = the byte value holding rank n-1 (0-based); below = #{P < theta};
    //    the padding keys are taken out of bin 255 first
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = hist[4 * lane + j];
    if (lane == 63) h[3] -= (uint32_t)(16 * nc - N);
    const uint32_t sum = h[0] + h[1] + h[2] + h[3];
    const uint32_t incl = wave_incl_scan(sum);
    const uint32_t excl = incl - sum;
    const bool owner = excl < (uint32_t)n && (uint32_t)n <= incl;
    uint32_t theta = 0, below = 0, bucket = 0;
    if (owner) {
        uint32_t acc = excl;
        bool found = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!found && acc + h[j] >= (uint32_t)n) {
                theta = 4 * lane + j;
                below = acc;
                bucket = h[j];
                found = true;
            }
            acc += h[j];
        }
    }
    const uint64_t own = __ballot(owner);
    const int src = __ffsll((unsigned long long)own) - 1;
    theta = __builtin_amdgcn_readlane(theta, src);
    below = __builtin_amdgcn_readlane(below, src);
    bucket = __builtin_amdgcn_readlane(bucket, src);
    const uint32_t need = (uint32_t)n - below;
    if (bucket > (uint32_t)kCandCap) {  // not seen in practice (expected size N / 256)
        if (lane == 0) atomicExch(&sstat[p], (int)HBT_ERR_INTERNAL);
        uint32_t* out = const_cast<uint32_t*>(mask_row(mask, pd, row, pd.Wp));
        for (int w = lane; w < pd.Wp; w += 64) out[w] = 0u;  // an empty group: nothing to gather
        return;
    }
    // 3. classification: each lane builds the 16 bits "P < theta" of its
    //    block, two neighbouring lanes form one 32-bit mask word; blocks that
    //    hold a byte equal to theta (a few per split) list those items
    const uint32_t theta4 = theta * 0x01010101u;
    // (the items of two rounds' blocks at a time, in any order: a rank does not
    // depend on the list's)
    auto classify = [&](int k, uint4 w) {
        const int c = 64 * k + lane;
        uint32_t lt = below_theta(w, theta4), eq = equal_theta(w, theta4);
        if (64 * k + 64 >= nc) {  // the round with the last block: its padding keys and the lanes past it
            if (c == nc - 1) eq &= (2u << (N - 16 * (nc - 1) - 1)) - 1u;
            if (c >= nc) {
                lt = 0u;
                eq = 0u;
            }
        }
        // lane ^ 1's bits (quad_perm [1,0,3,2])
        const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)lt, 0xB1, 0xF, 0xF, false);
        if (!(lane & 1) && c < nw) mlds[c >> 1] = lt | (nb << 16);
        return eq;
    };
    auto list_items = [&](int k, uint32_t eq) {  // bits 0-15 of round k, 16-31 of round k + 1
        while (eq) {
            const uint32_t t = (uint32_t)__ffs(eq) - 1u;
            cidx[lds_take(nlist)] = (uint32_t)(16 * (64 * k + lane)) + (t >> 4) * 1024u + (t & 15u);
            eq &= eq - 1u;
        }
    };
    if constexpr (R > 0) {
#pragma unroll
        for (int k = 0; k < R; k += 2)
            if (k < niter) {  // wave-uniform
                uint32_t eq = classify(k, key[k]);
                if (k + 1 < R && k + 1 < niter) eq |= classify(k + 1, key[k + 1 < R ? k + 1 : k]) << 16;
                list_items(k, eq);
            }
    } else {
        for (int k = 0; k < niter; ++k) {
            const int c = 64 * k + lane;
            uint4 w = make_uint4(0u, 0u, 0u, 0u);
            if (c < nc) w = primary_block(c, b, pd.pair_index, key0, key1);
            if (c == nc - 1) w = pad_block(w, N - 16 * (nc - 1));
            list_items(k, classify(k, w));
        }
    }
    wave_sync();
    const uint32_t cnt = bucket;
    // 4. secondary keys of the bucket items; 5. the `need` bucket items first in
    //    (S, i) order join group 1.  With at most 64 bucket items (the usual
    //    case: about N / 256) each lane holds one and ranks it against the
    //    others through lane broadcasts; larger buckets rank through LDS.
    if (cnt <= 64) {
        uint32_t sk = 0xffffffffu, ik = 0xffffffffu;
        if ((uint32_t)lane < cnt) {
            ik = cidx[lane];
            const uint4 w = philox4x32_10(make_uint4(ik >> 2, b, pd.pair_index, 1u), key0, key1);
            sk = word_of(w, ik & 3);
        }
        // (S, i) order as one 64-bit key
        const uint64_t key = ((uint64_t)sk << 32) | ik;
        uint32_t rank = 0;
        for (uint32_t q = 0; q < cnt; ++q) {
            const uint64_t k2 = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(sk, q) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane(ik, q);
            rank += k2 < key;
        }
        if ((uint32_t)lane < cnt && rank < need) atomicOr(&mlds[ik >> 5], 1u << (ik & 31));
    } else {
        for (uint32_t k = lane; k < cnt; k += 64) {
            const uint32_t i = cidx[k];
            const uint4 w = philox4x32_10(make_uint4(i >> 2, b, pd.pair_index, 1u), key0, key1);
            ckey[k] = word_of(w, i & 3);
        }
        wave_sync();
        for (uint32_t k = lane; k < cnt; k += 64) {
            const uint32_t sk = ckey[k], ik = cidx[k];
            uint32_t rank = 0;
            for (uint32_t q = 0; q < cnt; ++q) {
                const uint32_t s2 = ckey[q], i2 = cidx[q];
                rank += (s2 < sk) || (s2 == sk && i2 < ik);
            }
            if (rank < need) atomicOr(&mlds[ik >> 5], 1u << (ik & 31));
        }
    }
    wave_sync();
    write_mask_row(const_cast<uint32_t*>(mask_row(mask, pd, row, pd.Wp)), mlds, pd);
}

// Wave g draws the g-th of the rows [row0, rows): of all pairs, or of the nbig
// pairs listed in big_pair (their rows before each in big_row0), the pairs of
// more than skip_wp mask words a row in a call that also has smaller ones
// (without the list, as in a pipelined call, the wave of a smaller pair's row
// returns).
template <int R>
__global__ __launch_bounds__(64 * kSplitWaves) void k_split_masks(const BlockPair* __restrict__ bp, int npairs,
                                                                  int64_t rows, int max_np, uint32_t key0,
                                                                  uint32_t key1, uint32_t* __restrict__ mask,
                                                                  int32_t* sstat, int64_t row0, int skip_wp,
                                                                  double pairs_per_row,
                                                                  const int32_t* __restrict__ big_pair,
                                                                  const int64_t* __restrict__ big_row0, int nbig) {
    __shared__ uint32_t hist_all[kSplitWaves][256];
    __shared__ uint32_t nlist_all[kSplitWaves];
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t row = (int64_t)blockIdx.x * kSplitWaves + wave + row0;
    if (row >= rows) return;
    int p;
    if (big_pair) {
        const int k = place_of_row(nbig, row, pairs_per_row, [&](int q) { return big_row0[q]; },
                                   [&](int q) { return (int64_t)bp[big_pair[q]].nb; });
        p = big_pair[k];
        row += bp[p].mrow0 - big_row0[k];
    } else {
        p = pair_of_row(bp, npairs, row, pairs_per_row);
    }
    const BlockPair pd = bp[p];  // the pair's sizes, mask row width and index (not a PairDesc)
    // another pair's rows, or the other kernel, draw these masks (wave-uniform)
    if (pd.owner != p || pd.Wp <= skip_wp) return;
    split_row<R>(pd, p, row, max_np, key0, key1, mask, sstat, hist_all, &nlist_all[wave], smem);
}

// ---------------------------------------------------------------------------
// Four split rows per wave, for pairs of up to kQuadItems pooled items: 16
// lanes a row (lane 16 r + t draws blocks t, t + 16, ... of row r), so a pair of
// 128 items takes one round of 32 lanes instead of four of 8; the four histograms
// are scanned at once; and the rows' bucket items share one list and one
// secondary draw, ranked by (row, S, i).  Bound by VALU issue (920 vector
// instructions a wave at 760 items, one per SIMD every 4.3 cycles).  2.5 million
// rows of 200 to 2000 items: 1.06 ms, and 0.11 ms for the other kernel's skipping
// of them, against 2.5 ms with one wave a row (620 instructions each, and as long
// again waiting for the search of its pair).
// ---------------------------------------------------------------------------
constexpr int kQuad = 4;
constexpr int kListCap = 320;  // bucket items of a wave's rows (about 4 N / 256 <= 32 of them)
static_assert(12 * kListCap <= kQuad * 1024, "the list and its keys take the histograms' words");

// hist[key] += 1 for the 16 keys of a block, the histogram at LDS address hb (a
// multiple of 1024).
__device__ __forceinline__ void count_block_at(uint32_t hb, uint4 w) {
    const uint32_t one = 1u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t x = word_of(w, q);
        lds_inc<0>(((x << 2) & 0x3fcu) | hb, one);
        lds_inc<0>(((x >> 6) & 0x3fcu) | hb, one);
        lds_inc<0>(((x >> 14) & 0x3fcu) | hb, one);
        lds_inc<0>(((x >> 22) & 0x3fcu) | hb, one);
    }
}

// Split rows row .. row + nr - 1 (nr <= 4) of pair p, of at most 16 K blocks.
template <int K>
__device__ __forceinline__ void split_rows(const BlockPair& pd, int p, int64_t row, int nr, uint32_t key0,
                                           uint32_t key1, uint32_t* __restrict__ mask, int32_t* sstat,
                                           uint32_t (*hist)[256], uint4* meta, uint32_t* mlds) {
    int lane = threadIdx.x & 63, N = pd.n + pd.m;
    // nothing of these rows stays in registers across the caller's loop
    asm volatile("" : "+v"(lane), "+s"(N), "+s"(key0), "+s"(key1));
    const int r4 = lane >> 4, t = lane & 15;
    const uint32_t b0 = pd.perm_base + (uint32_t)(row - pd.mrow0);
    const int Wp = pd.Wp;
    const uint32_t n = (uint32_t)pd.n;
    const int nc = (N + 15) >> 4, nw = Wp * 2;  // blocks with items, and of a mask row
    const int lim = N - 16 * (nc - 1);          // items of the last block
    const bool live = r4 < nr;
    const uint32_t hb = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)hist + 1024u * (uint32_t)r4;
#pragma unroll
    for (int i = 0; i < kQuad; ++i) ((uint4*)hist)[64 * i + lane] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
    // 1. primary keys and their histograms
    uint4 key[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        key[k] = make_uint4(0u, 0u, 0u, 0u);
        if (16 * k < nc) {  // wave-uniform
            const int c = 16 * k + t;
            if (live && c < nc) {
                key[k] = primary_block(c, b0 + (uint32_t)r4, pd.pair_index, key0, key1);
                if (c == nc - 1) key[k] = pad_block(key[k], lim);
                count_block_at(hb, key[k]);
            }
        }
    }
    wave_sync();
    // 2. theta, the items below it and its bucket, per row: lane t of row r's 16
    //    lanes holds bins 16 t .. 16 t + 15 (the padding keys taken out of bin 255)
    {
        uint32_t h[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = ((const uint4*)hist[r4])[4 * t + i];
            h[4 * i] = v.x;
            h[4 * i + 1] = v.y;
            h[4 * i + 2] = v.z;
            h[4 * i + 3] = v.w;
        }
        const uint32_t pad = (uint32_t)(16 * nc - N);
        if (t == 15) h[15] -= pad;
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += h[i];
        int v = (int)sum;  // inclusive scan over the 16 lanes
        v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
        const uint32_t incl = (uint32_t)v, excl = incl - sum;
        if (live && excl < n && n <= incl) {  // one lane per row
            uint32_t acc = excl, below = excl, cnt = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc += h[i];
                const bool lt = acc < n;
                cnt += lt;
                below = lt ? acc : below;
            }
            const uint32_t theta = 16u * (uint32_t)t + cnt;
            const uint32_t bucket = hist[r4][theta] - (theta == 255u ? pad : 0u);
            meta[r4] = make_uint4(theta * 0x01010101u, n - below, bucket, 0u);
        } else if (!live && t == 0) {
            meta[r4] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    wave_sync();
    const uint32_t c0 = __builtin_amdgcn_readfirstlane(meta[0].z), c1 = __builtin_amdgcn_readfirstlane(meta[1].z),
                   c2 = __builtin_amdgcn_readfirstlane(meta[2].z), c3 = __builtin_amdgcn_readfirstlane(meta[3].z);
    uint32_t* out = const_cast<uint32_t*>(mask_row(mask, pd, row, Wp));
    if (c0 + c1 + c2 + c3 > (uint32_t)kListCap) {  // not seen in practice, as in k_split_masks
        if (lane == 0) atomicExch(&sstat[p], (int)HBT_ERR_INTERNAL);
        for (int w = lane; w < nr * Wp; w += 64) out[w] = 0u;  // empty groups: nothing to gather
        return;
    }
    // 3. classification: each lane builds the 16 bits "P < theta" of its block,
    //    two neighbouring lanes one mask word; the bucket items go to the list
    //    (row << 16 | item) in any order
    uint32_t* list = hist[0];
    const uint32_t listed = c0 + c1 + c2 + c3;
    uint32_t* nlist = &meta[0].w;
    const uint32_t theta4 = meta[r4].x;
    uint32_t* mrow = mlds + r4 * Wp + (t >> 1);
    uint32_t eq2 = 0u;  // two rounds' items equal to theta
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (16 * k < nw) {  // wave-uniform
            const int c = 16 * k + t;
            uint32_t lt = below_theta(key[k], theta4), eq = equal_theta(key[k], theta4);
            if (!live) eq = 0u;
            if (16 * k + 16 >= nc) {  // the round with the last block: its padding keys and the lanes past it
                if (c == nc - 1) eq &= (2u << (lim - 1)) - 1u;
                if (c >= nc) {
                    lt = 0u;
                    eq = 0u;
                }
            }
            // lane ^ 1's bits (quad_perm [1,0,3,2])
            const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)lt, 0xB1, 0xF, 0xF, false);
            if (!(lane & 1) && live && c < nw) mrow[8 * k] = lt | (nb << 16);
            eq2 |= eq << (16 * (k & 1));
        }
        if (k & 1) {  // the items of two rounds
            while (eq2) {
                const uint32_t j = (uint32_t)__ffs(eq2) - 1u;
                list[lds_take(nlist)] =
                    ((uint32_t)r4 << 16) | (uint32_t)(256 * (k - 1) + 16 * t) + (j >> 4) * 256u + (j & 15u);
                eq2 &= eq2 - 1u;
            }
        }
    }
    wave_sync();
    // 4., 5. secondary keys; an item's rank among all listed ones in (row, S, i)
    //    order, less the bucket items of the rows before, is its rank in its row,
    //    and the first `need` of a row join group 1
    auto key_of = [&](uint32_t e) {
        const uint32_t i = e & 0xffffu, s = e >> 16;
        const uint4 w = philox4x32_10(make_uint4(i >> 2, b0 + s, pd.pair_index, 1u), key0, key1);
        return ((uint64_t)s << 48) | ((uint64_t)word_of(w, i & 3) << 16) | i;
    };
    auto join = [&](uint32_t e, uint32_t rank) {
        const uint32_t i = e & 0xffffu, s = e >> 16;
        const uint32_t before = (s > 0 ? c0 : 0u) + (s > 1 ? c1 : 0u) + (s > 2 ? c2 : 0u);
        if (rank - before < meta[s].y) atomicOr(&mlds[(int)s * Wp + (int)(i >> 5)], 1u << (i & 31));
    };
    if (listed <= 64u) {  // the usual case: ranks through lane broadcasts
        uint32_t e = 0;
        uint64_t ky = ~0ull;
        if ((uint32_t)lane < listed) {
            e = list[lane];
            ky = key_of(e);
        }
        uint32_t rank = 0;
        for (uint32_t q = 0; q < listed; ++q) {
            const uint64_t k2 = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(ky >> 32), q) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ky, q);
            rank += k2 < ky;
        }
        if ((uint32_t)lane < listed) join(e, rank);
    } else {  // through LDS
        uint64_t* lkey = (uint64_t*)(list + kListCap);
        for (uint32_t q = lane; q < listed; q += 64) lkey[q] = key_of(list[q]);
        wave_sync();
        for (uint32_t k = lane; k < listed; k += 64) {
            const uint64_t ky = lkey[k];
            uint32_t rank = 0;
            for (uint32_t q = 0; q < listed; ++q) rank += lkey[q] < ky;
            join(list[k], rank);
        }
    }
    wave_sync();
    if (pd.ygap == 0) {  // the rows are one run
        for (int w = lane; w < nr * Wp; w += 64) out[w] = mlds[w];
    } else {
        for (int i = 0; i < nr; ++i) write_mask_row(out + i * Wp, mlds + i * Wp, pd);
    }
}

// Wave g takes the split rows 4 g .. 4 g + 3, those of one pair together; rows
// of pairs of more than 16 K blocks are left to k_split_masks.
// At most 64 registers: with six of its work-groups on a CU (wg_per_cu), a wave
// of the column sums (112 registers) still fits each SIMD.  The mask rows' LDS is
// dynamic for the compiler's count of resident waves.
template <int K>
__global__ __launch_bounds__(64 * kSplitWaves, 8) void k_split_quads(const BlockPair* __restrict__ bp, int npairs,
                                                                  int64_t rows, uint32_t key0, uint32_t key1,
                                                                  uint32_t* __restrict__ mask, int32_t* sstat,
                                                                  int64_t row0, double pairs_per_row) {
    __shared__ __attribute__((aligned(1024))) uint32_t hist_all[kSplitWaves][kQuad][256];
    __shared__ uint4 meta_all[kSplitWaves][kQuad];
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint32_t(*mlds_all)[kQuad * 8 * K] = (uint32_t(*)[kQuad * 8 * K])smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t row = ((int64_t)blockIdx.x * kSplitWaves + wave) * kQuad + row0;
    const int64_t end = row + kQuad < rows ? row + kQuad : rows;
    while (row < end) {
        const int p = pair_of_row(bp, npairs, row, pairs_per_row);
        const BlockPair pd = bp[p];  // the pair's sizes, mask row width and index (not a PairDesc)
        const int64_t pend = pd.mrow0 + pd.nb;
        const int nr = (int)((pend < end ? pend : end) - row);
        if (pd.owner == p && pd.Wp <= 8 * K) {  // else another pair's rows, or the other kernel, draw these masks
            split_rows<K>(pd, p, row, nr, key0, key1, mask, sstat, hist_all[wave], meta_all[wave], mlds_all[wave]);
            wave_sync();
        }
        row += nr;
    }
}

// LDS of one CU (160 KB on MI355X), from the device.
static size_t lds_per_cu() {
    static std::atomic<size_t> v{0};
    size_t x = v.load(std::memory_order_relaxed);
    if (!x) {
        int dev = 0, a = 0;
        x = (hipGetDevice(&dev) == hipSuccess &&
             hipDeviceGetAttribute(&a, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) == hipSuccess &&
             a > 0) ? (size_t)a : 163840;
        v.store(x, std::memory_order_relaxed);
    }
    return x;
}

size_t split_lds_limit() {
    static size_t lim = 0;
    if (!lim) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
            lim = (size_t)v;
        else
            lim = 65536;
    }
    return lim;
}

// Rounds of the four-row kernel.
constexpr int kQuadRounds = 8, kQuadRoundsSmall = 4;
static_assert(kQuadItems == 256 * kQuadRounds, "16 blocks of 16 items a round");

size_t split_lds_per_block(int max_np) { return (size_t)kSplitWaves * SplitLds(max_np).total + kSplitStaticLds; }

hipError_t launch_split_masks(const BlockPair* bp, int npairs,
                              int64_t rows, int min_np, int max_np, uint64_t seed, uint32_t* mask,
                              int32_t* sstat, int wg_per_cu, hipStream_t s, SplitBig big, int64_t row0,
                              int64_t total_rows) {
    if (rows <= row0) return hipSuccess;
    if (total_rows < rows) total_rows = rows;
    const size_t share = wg_per_cu > 0 ? lds_per_cu() / (size_t)wg_per_cu : 0;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    // At most 64 KB of LDS per work-group (of four split rows): the one limit of calls of
    // every size, checked before either kernel; a cap of one or two work-groups per CU
    // is past it.
    const SplitLds L(max_np);
    size_t lds = (size_t)kSplitWaves * L.total;
    if (share > lds + kSplitStaticLds) lds = share - kSplitStaticLds;
    if (lds + kSplitStaticLds > 65536 || lds + kSplitStaticLds > split_lds_limit()) return hipErrorInvalidValue;
    const dim3 block(64 * kSplitWaves);
    const double ppr = (double)npairs / (double)total_rows;
    if (min_np <= kQuadItems) {
        const int64_t per_wg = (int64_t)kSplitWaves * kQuad;
        const dim3 grid((unsigned)((rows - row0 + per_wg - 1) / per_wg));
        auto go = [&](auto kern, int K) {
            const size_t fixed = (size_t)kSplitWaves * kQuad * (1024 + 16), rows_lds = (size_t)kSplitWaves * kQuad * 32 * K;
            hipLaunchKernelGGL(kern, grid, block, share > fixed + rows_lds ? share - fixed : rows_lds, s, bp, npairs, rows, k0, k1, mask,
                               sstat, row0, ppr);
        };
        if (max_np <= 256 * kQuadRoundsSmall) go(k_split_quads<kQuadRoundsSmall>, kQuadRoundsSmall);
        else go(k_split_quads<kQuadRounds>, kQuadRounds);
        if (max_np <= kQuadItems) return hipGetLastError();
    }
    const int skip_wp = min_np <= kQuadItems ? kQuadItems / 32 : 0;
    if (!skip_wp) big = SplitBig{};
    double per_row = ppr;
    if (big.pair) {
        if (big.rows < 1) return hipErrorInvalidValue;
        per_row = (double)big.count / (double)big.rows;
        rows = big.rows;
        row0 = 0;
    }
    const dim3 grid((unsigned)((rows - row0 + kSplitWaves - 1) / kSplitWaves));
    // registers for the keys of the largest pair: R blocks of 16 per lane
    const int r = (max_np + 1023) / 1024;
#define HBT_SPLIT(RR)                                                                                             \
    hipLaunchKernelGGL(k_split_masks<RR>, grid, block, lds, s, bp, npairs, rows, max_np, k0, k1, mask, sstat, row0, \
                       skip_wp, per_row, big.pair, big.row0, big.count)
    if (r <= 4) HBT_SPLIT(4);
    else if (r <= 8) HBT_SPLIT(8);
    else if (r <= 12) HBT_SPLIT(12);
    else if (r <= 16) HBT_SPLIT(16);
    else HBT_SPLIT(0);
#undef HBT_SPLIT
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// explicit masks: copy + validate (exactly n items, no bits at or beyond N)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy_masks(const uint32_t* __restrict__ user,
                                                    int64_t rows, int N, int n, int Wp,
                                                    uint32_t* __restrict__ mask, int32_t* sstat) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const int W = (N + 31) >> 5;
    int pc = 0;
    bool bad = false;
    for (int w = lane; w < Wp; w += 64) {
        uint32_t x = w < W ? user[row * W + w] : 0u;
        if (w == W - 1 && (N & 31)) {
            bad |= (x >> (N & 31)) != 0u;
        }
        pc += __popc(x);
        mask[row * Wp + w] = x;
    }
    for (int o = 32; o > 0; o >>= 1) pc += __shfl_xor(pc, o, 64);
    const bool anybad = __ballot(bad) != 0;
    if (lane == 0 && (pc != n || anybad)) atomicExch(sstat, (int)HBT_ERR_MASK);
}

hipError_t launch_copy_masks(const uint32_t* user, int64_t user_row0, int64_t rows, int N, int n,
                             int Wp, uint32_t* mask, int32_t* sstat, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int W = (N + 31) >> 5;
    hipLaunchKernelGGL(k_copy_masks, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s,
                       user + user_row0 * W, rows, N, n, Wp, mask, sstat);
    return hipGetLastError();
}

__global__ void k_export_masks(const uint32_t* __restrict__ mask, int64_t rows, int Wp, int W,
                               uint32_t* __restrict__ out) {
    const int64_t total = rows * W;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = k / W;
        out[k] = mask[r * Wp + (k - r * W)];
    }
}

hipError_t launch_export_masks(const uint32_t* mask, int64_t rows, int Wp, int W, uint32_t* out,
                               hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    int64_t g = (rows * W + 255) / 256;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_export_masks, dim3((unsigned)g), dim3(256), 0, s, mask, rows, Wp, W, out);
    return hipGetLastError();
}

}  // namespace hbt
