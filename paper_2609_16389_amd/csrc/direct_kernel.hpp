// Register-direct kernel: C = A * B for products with few output tiles, a
// short K, or operands in any layout (16-bit inputs, fp32 accumulate, fp32
// out).
//
// No operand passes through LDS.  A workgroup is WN x KW waves; a wave owns
// a (16 FM) x (16 NV) block of C over every KW-th 64-wide slab of K, and
// loads its operands straight into the registers the MFMAs read:
//   A  lane l reads row l % 16 of each 16-row block, 16 bytes (8 k);
//   B  lane l reads the NV columns from NV (l % 16), in each of 8 rows (k) of
//      its k group l / 16; the 8 rows are transposed in registers (one
//      v_perm per two values), so that NV MFMAs follow, MFMA j taking the
//      columns NV c + j, c = 0 .. 15.
// Within a slab of 64, sub-step s (0, 1) of lane group g covers the k of
// 16 g + 8 s .. + 7, so that the two A loads of a lane are the two halves of
// 32 contiguous bytes.  (Any assignment of k to lanes is a valid MFMA
// operand as long as A and B agree on it.)  A half of the next slab is loaded
// as soon as the same half of the current one has been read.
// The waves never wait for each other before the K loop is over: then the
// KW partial blocks are added through LDS, in ascending wave order, each
// wave finishing its share of the block.
//
// Loads need no alignment but the element's: rows of any leading dimension
// are read in place.  Every load stays inside the operands: rows past M and
// columns past N are read from the last valid place (a lane whose columns
// run over N reads the last NV columns and stores those of its own), and
// the slab that runs over K is read from the last 8 values of a row and the
// last row, shifted and zeroed.  That needs N and K of at least 8.
//
// What bounds it: with few rows, the bytes of B (16 x 14336 x 4096, 117 MB:
// 24.8 us, 4.7 TB/s, against 30.1 for 128 x 128 tiles through LDS, whose A
// tile is 7/8 padding and whose pipeline keeps 32 KiB in flight per CU; here
// 8 waves hold 9 KiB each).  With few tiles, latency: 256^3 3.7 us against
// 6.0, 1000^3 9.5 against 20.9 (256 workgroups against 64).  With many tiles
// the L1 path, through which every wave pulls its own operands (64 x 128: 43
// flop per byte), where the LDS tiles win: 2048^3 33 us against 27 (12.8M L1
// accesses against the wave-pair tile's 5.2M; the L1's data return is the
// busiest unit, 60% of the time, the matrix cores 17%).  Odd
// rows cost a slab 1.2-1.5 times its time (each 16-byte load then straddles
// dwords); a copy of the operands costs more: 16 x 10376 x 8656 with odd
// rows 42 us against 157.  A K split over the waves of a workgroup first,
// because their partials meet in LDS, and over workgroups only until the
// CUs are busy.
#pragma once

#include "gemm_kernel.hpp"

namespace xgemm_dev {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// NV 16-bit values as dwords
template <int NV>
struct DirectVec {
    typedef uint32_t T __attribute__((ext_vector_type(NV / 2)));
};

// 16-byte units of the accumulator block per lane
template <int FM, int NV>
constexpr int direct_units()
{
    return FM * NV;
}

// LDS bytes of the partial blocks (none where no wave shares a block).
template <int FM, int NV, int WN, int KW>
constexpr int direct_lds_bytes()
{
    return KW > 1 ? WN * KW * direct_units<FM, NV>() * 1024 : 0;
}

// Eight 16-bit values shifted down by `sh` elements (sh >= 8: all zero),
// zeros entering at the top.
__host__ __device__ __forceinline__ u32x4 shift8_down(u32x4 v, int sh)
{
    uint64_t lo = v.x | ((uint64_t)v.y << 32), hi = v.z | ((uint64_t)v.w << 32);
    if (sh >= 4) {
        lo = hi;
        hi = 0;
        sh -= 4;
    }
    if (sh >= 4) {
        lo = 0;
        sh = 0;
    }
    const int b = 16 * sh;
    if (b > 0) {
        lo = (lo >> b) | (hi << (64 - b));
        hi >>= b;
    }
    u32x4 r = {(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    return r;
}

// K split over workgroups: add up the `split` partial blocks of a tile without
// a second launch.  Each workgroup publishes its block (s: the UW units of
// this wave, in the accumulators' layout; rows past M are left out) with
// device-scope stores and counts itself in once they have completed; the last
// one reads the others' and adds all in ascending K order, whichever of them
// it is, into s.  True for that one, which stores C and leaves the counter
// zero.  No workgroup waits for another.  (A second launch summing the
// partials took 2.8 to 4.9 us of 10 to 28 and 2.7 us of host time.)
template <int WN, int U, int UW, class Ops>
__host__ __device__ __forceinline__ bool combine(const Ops &ops, const GemmParams &p, int tile, int ks, int wn, int wk,
                                                 int m0, int g, int H, int lane, int tid, f32x4 (&s)[UW])
{
    constexpr int BLOCK = WN * U * 256;             // floats of a partial block
    float *const base = p.part + (int64_t)tile * p.split * BLOCK;
    auto row_of = [&](int v) {
        const int u = wk * UW + v;
        return m0 + u / (4 * H) * 16 + 4 * g + u / H % 4;
    };
    const uint32_t off = (uint32_t)(((wn * U + wk * UW) * 64 + lane) * 16);
    {
        const auto own = ops.rsrc(base + (int64_t)ks * BLOCK);
#pragma unroll
        for (int v = 0; v < UW; ++v)
            if (row_of(v) < p.M)
                ops.buf_store4_dev(own, off + v * 1024, 0, s[v]);
    }
    ops.stores_done();
    ops.sync();
    int found = 0;
    if (tid == 0)
        found = ops.flag_add(p.count + tile, 1);
    ops.lds_write4(ops.lds(), found, tid == 0);
    ops.sync();
    if (ops.uniform(ops.lds_read4(ops.lds())) != p.split - 1)
        return false;
    if (tid == 0)
        ops.flag_store(p.count + tile, 0);
    constexpr int QB = UW >= 8 ? 4 : UW >= 2 ? 8 : 16;   // partial blocks in flight
    f32x4 t[UW];
    for (int q0 = 0; q0 < p.split; q0 += QB) {
        f32x4 x[QB][UW];
#pragma unroll
        for (int b = 0; b < QB; ++b)
            if (q0 + b < p.split && q0 + b != ks) {
                const auto r = ops.rsrc(base + (int64_t)(q0 + b) * BLOCK);
#pragma unroll
                for (int v = 0; v < UW; ++v)
                    if (row_of(v) < p.M)
                        x[b][v] = ops.buf_load4_dev(r, off + v * 1024, 0);
            }
#pragma unroll
        for (int b = 0; b < QB; ++b)
            if (q0 + b < p.split) {
#pragma unroll
                for (int v = 0; v < UW; ++v) {
                    const f32x4 y = q0 + b == ks ? s[v] : x[b][v];
                    t[v] = q0 + b == 0 ? y : t[v] + y;
                }
            }
    }
#pragma unroll
    for (int v = 0; v < UW; ++v)
        s[v] = t[v];
    return true;
}

// One workgroup (id `block` of `nblocks`), as seen by thread `tid`.  NT: B is
// read with streaming loads.
template <int FM, int NV, int WN, int KW, int DT, bool NT, class Ops>
__host__ __device__ __forceinline__ void direct_tile(const Ops &ops, const GemmParams &p_in, int block, int nblocks,
                                                     int tid)
{
    static_assert(NV == 4 || NV == 8, "columns per lane");
    constexpr int BM = 16 * FM, TN = 16 * NV, BN = TN * WN;
    constexpr int SLAB = 64;
    constexpr int H = NV / 4;                       // 16-byte units per row of a lane's block
    typedef typename DirectVec<NV>::T bvec;

    int tm, tn, ks, local;
    const GemmParams p = map_tile(p_in, block, nblocks, tm, tn, ks, local);
    const int m0 = tm * BM;
    const int kbeg = ks * p.k_chunk;
    const int kend = min(p.K, kbeg + p.k_chunk);
    const int lane = tid & 63;
    const int wave = ops.uniform(tid >> 6);
    const int wk = wave % KW, wn = wave / KW;
    const int g = lane >> 4, r16 = lane & 15;
    const int nw = tn * BN + wn * TN;               // first column of the wave
    const int col = nw + NV * r16;                  // first column of the lane
    const int cb = min(col, p.N - NV);              // first column it reads
    const int64_t lda = p.lda, ldb = p.ldb;

    uint32_t a_off[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i)
        a_off[i] = (uint32_t)((min(16 * i + r16, p.M - 1 - m0) * lda + 16 * g) * 2);
    const uint32_t b_off = (uint32_t)((16 * g * ldb + cb) * 2);
    const char *const Ab = (const char *)(p.A + (int64_t)m0 * lda);
    const char *const Bb = (const char *)p.B;

    f32x4 acc[FM][NV];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[i][j][e] = 0.0f;

    u32x4 a[2][FM];
    bvec b[2][8];

    // sub-step S of the slab at k0 (wholly inside K)
    auto load = [&]<int S>(int k0) {
        const char *const as = Ab + (int64_t)k0 * 2 + 16 * S;
        const char *const bs = Bb + ((int64_t)k0 + 8 * S) * ldb * 2;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            b[S][r] = NT ? ops.template gload_any_nt<NV / 2>(bs + r * ldb * 2, b_off)
                         : ops.template gload_any<NV / 2>(bs + r * ldb * 2, b_off);
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a[S][i] = ops.template gload_any<4>(as, a_off[i]);
    };
    // the same for the slab that runs over K: row pieces that would pass K
    // are read from its last 8 values and shifted into place, rows of B past
    // K are read from its last row; what lies past K becomes zero
    auto load_tail = [&]<int S>(int k0) {
        const int k = k0 + 16 * g + 8 * S;
        const int ka = min(k, p.K - 8);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int kr = min(k + r, p.K - 1);
            b[S][r] = ops.template gload_any<NV / 2>(Bb + (int64_t)k0 * ldb * 2,
                                                          (uint32_t)(((int64_t)(kr - k0) * ldb + cb) * 2));
            if (k + r >= p.K)
#pragma unroll
                for (int d = 0; d < NV / 2; ++d)
                    b[S][r][d] = 0u;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            // (ka may lie before k0: the row's offset holds 16 g already)
            const u32x4 v = ops.template gload_any<4>(Ab, a_off[i] + (uint32_t)(ka - 16 * g) * 2u);
            a[S][i] = shift8_down(v, k - ka);
        }
    };
    auto compute = [&]<int S>() {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            u32x4 f;
#pragma unroll
            for (int d = 0; d < 4; ++d)
                f[d] = ops.pair16(b[S][2 * d][j / 2], b[S][2 * d + 1][j / 2], j & 1);
#pragma unroll
            for (int i = 0; i < FM; ++i)
                acc[i][j] = ops.template mfma<DT>(a[S][i], f, acc[i][j]);
        }
    };
    // compute a slab; NEXT: load the slab at k0 into each half once it is read
    auto slab = [&]<bool NEXT>(int k0) {
        compute.template operator()<0>();
        ops.fence();
        if constexpr (NEXT)
            load.template operator()<0>(k0);
        ops.fence();
        compute.template operator()<1>();
        ops.fence();
        if constexpr (NEXT)
            load.template operator()<1>(k0);
        ops.fence();
    };
    const int nfull = (kend - kbeg) / SLAB;         // slabs wholly inside the range
    int left = nfull > wk ? (nfull - 1 - wk) / KW + 1 : 0;   // this wave's
    int k = kbeg + wk * SLAB;
    if (left > 0) {
        load.template operator()<0>(k);
        load.template operator()<1>(k);
        while (--left > 0) {
            k += KW * SLAB;
            slab.template operator()<true>(k);
        }
        slab.template operator()<false>(0);
    }
    if (kbeg + nfull * SLAB < kend && nfull % KW == wk) {
        load_tail.template operator()<0>(kbeg + nfull * SLAB);
        load_tail.template operator()<1>(kbeg + nfull * SLAB);
        slab.template operator()<false>(0);
    }

    // acc[i][j][e] is C[m0 + 16 i + 4 g + e][cb + j].  Unit (i, e, h): the 4
    // columns from cb + 4 h of row 16 i + 4 g + e.
    const OutView ov = out_view<BM, BN>(p, ks, local, m0, tn * BN);
    float *const Cb = ov.base;
    const int64_t ldc = ov.ld;
    auto unit = [&](int i, int e, int h) {
        f32x4 v = {acc[i][4 * h][e], acc[i][4 * h + 1][e], acc[i][4 * h + 2][e], acc[i][4 * h + 3][e]};
        return v;
    };
    auto store = [&](int row, int h, f32x4 v) {
        if (row >= p.M)
            return;
        float *const c = Cb + (int64_t)row * ldc + cb + 4 * h;
        if (cb == col) {
            ops.store4(c, v);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (cb + 4 * h + j >= col)          // the lane's own columns
                    ops.store1(c + j, v[j]);
        }
    };
    // the two units of a row; where the whole block lies inside C, rearranged
    // between the lanes so that a store instruction writes 256 contiguous
    // bytes of a row, not every other 16
    const bool whole = nw + TN <= p.N;
    auto store_row = [&](int row, f32x4 v0, f32x4 v1) {
        if (whole) {
            ops.line_pair(v0, v1);
            if (row < p.M) {
                float *const c = Cb + (int64_t)row * ldc + nw + 8 * (r16 & 7) + 4 * (r16 >> 3);
                ops.store4(c, v0);
                ops.store4(c + 64, v1);
            }
        } else {
            store(row, 0, v0);
            store(row, 1, v1);
        }
    };
    if constexpr (KW == 1) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + 16 * i + 4 * g + e;
                if constexpr (H == 2)
                    store_row(row, unit(i, e, 0), unit(i, e, 1));
                else
                    store(row, 0, unit(i, e, 0));
            }
    } else {
        constexpr int U = direct_units<FM, NV>();
        constexpr int UW = U / KW;                  // units each wave finishes
        static_assert(U % KW == 0, "whole units per wave");
        char *const mine = ops.lds() + (wave * U * 64 + lane) * 16;
#pragma unroll
        for (int u = 0; u < U; ++u)
            ops.lds_write16(mine + u * 1024, __builtin_bit_cast(u32x4, unit(u / (4 * H), u / H % 4, u % H)));
        ops.sync();
        const char *const all = ops.lds() + (wn * KW * U * 64 + lane) * 16;
        f32x4 s[UW];
#pragma unroll
        for (int v = 0; v < UW; ++v) {
            const int u = wk * UW + v;
            s[v] = __builtin_bit_cast(f32x4, ops.read16(all + u * 1024));
#pragma unroll
            for (int w = 1; w < KW; ++w)
                s[v] += __builtin_bit_cast(f32x4, ops.read16(all + (w * U + u) * 1024));
        }
        if (p.count && !combine<WN, U, UW>(ops, p, local, ks, wn, wk, m0, g, H, lane, tid, s))
            return;
#pragma unroll
        for (int v = 0; v < UW; v += (UW % H == 0 ? H : 1)) {
            const int u = wk * UW + v;
            const int row = m0 + u / (4 * H) * 16 + 4 * g + u / H % 4;
            if constexpr (H == 2 && UW % 2 == 0)
                store_row(row, s[v], s[v + 1]);
            else
                store(row, u % H, s[v]);
        }
    }
}

template <int FM, int NV, int WN, int KW, int DT, bool NT>
__global__ void __launch_bounds__(WN * KW * 64, FM *NV <= 8 ? 4 : FM *NV <= 16 ? 2 : 1)
gemm_kernel_direct(GemmParams p_in)
{
    constexpr int LDS = direct_lds_bytes<FM, NV, WN, KW>();
    __shared__ __attribute__((aligned(16))) char smem[LDS > 0 ? LDS : 16];
    const int w = linear_block();
    if (w >= p_in.grid)
        return;
    const DeviceOps ops{smem};
    direct_tile<FM, NV, WN, KW, DT, NT>(ops, p_in, w, p_in.grid, threadIdx.x);
}

}  // namespace xgemm_dev
