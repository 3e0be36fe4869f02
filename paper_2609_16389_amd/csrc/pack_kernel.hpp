// Copies of 16-bit GEMM operands into the library's workspace.
//
// The pipelined GEMM kernels load whole 16-byte chunks of A and B rows
// straight into LDS, so they need 16-byte aligned rows, K a multiple of 8
// and B rows readable to a multiple of 8 columns.  An operand that is not
// laid out that way is copied once per call into a dense, zero-padded
// buffer that is: rows x cols with cols the logical width rounded up to a
// multiple of 8.  The padding is zero, so padded K positions contribute
// exactly zero to every product; padded columns of B only feed outputs that
// are never stored.
//
// Bound by HBM bandwidth once an operand is tens of MB: both operands of
// 8191^3 (537 MB read and written) take 104 us, 5.2 TB/s, where one launch
// per operand staging rows in LDS took about 125 us each; 593 x 256 x 50003
// (170 MB) 28.6 us, and the whole call 77 against 124.  Below that, by the
// launch and one memory latency: 2047^3 11.1 us for both against 8.0 + 8.4.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xgemm_dev {

typedef uint32_t pack_u32x4 __attribute__((ext_vector_type(4)));

// One operand's copy: dst[b * dst_stride + r * ldd + c] = src[b * src_stride
// + r * lds + c] for r < src_rows and c < src_cols, and 0 elsewhere in each
// of the `batch` rows x (8 * cols8) destinations.  dst and dst_stride keep
// every destination 16-byte aligned, ldd is a multiple of 8; src is 2-byte
// aligned with any leading dimension and batch stride.
struct PackOperand {
    const uint16_t *src;
    uint16_t *dst;
    int64_t lds, src_stride, ldd, dst_stride;
    int src_rows, src_cols;
    int rows, cols8, batch;
    int blocks;  // workgroups that copy it (0: nothing to copy)
};

constexpr int kPackChunks = 2;                    // chunks of 8 values per thread and pass
constexpr int kPackBlock = 256 * kPackChunks;     // chunks per workgroup and pass

// Both operands of a call in one launch: workgroups [0, a.blocks) copy a, the
// next b.blocks copy b.  A thread moves one 16-byte destination chunk per
// load and store, its source read at element alignment, and has kPackChunks
// loads in flight before it stores; there is no staging and no barrier.  The
// chunks of all rows are numbered through, so that short rows fill the
// workgroups as well as long ones; a thread divides once per pass and then
// steps 256 chunks on by additions.  Loads start on 4-byte boundaries: a
// 16-byte load at an odd element costs about twice one on a dword boundary,
// so an odd source is read one element early and shifted.  (Not the first
// chunk, before which there may be no element.)
__global__ void __launch_bounds__(256) pack16(PackOperand a, PackOperand b)
{
    struct __attribute__((packed, aligned(4))) any {
        pack_u32x4 v;
    };
    const bool second = (int)blockIdx.x >= a.blocks;
    const PackOperand p = second ? b : a;
    const int block = second ? (int)blockIdx.x - a.blocks : (int)blockIdx.x;
    const int64_t rows = (int64_t)p.batch * p.rows;   // of the stacked destinations
    const int64_t chunks = rows * p.cols8;
    const uint32_t cols8 = (uint32_t)p.cols8;
    const uint32_t step_rows = 256u / cols8, step_cols = 256u % cols8;
    for (int64_t q0 = (int64_t)block * kPackBlock; q0 < chunks; q0 += (int64_t)p.blocks * kPackBlock) {
        const int64_t row0 = q0 / p.cols8;
        const uint32_t first = (uint32_t)(q0 - row0 * p.cols8) + threadIdx.x;
        int64_t row = row0 + first / cols8;
        uint32_t c = first % cols8;
        pack_u32x4 v[kPackChunks];
        uint16_t *d[kPackChunks];
#pragma unroll
        for (int i = 0; i < kPackChunks; ++i) {
            d[i] = nullptr;
            if (row < rows) {
                int64_t bt = 0, r = row;
                if (p.batch > 1) {
                    bt = rows <= 0xffffffffll ? (int64_t)((uint32_t)row / (uint32_t)p.rows) : row / p.rows;
                    r = row - bt * p.rows;
                }
                const int col = (int)c * 8;
                d[i] = p.dst + bt * p.dst_stride + r * p.ldd + col;
                const uint16_t *const s = p.src + bt * p.src_stride + r * p.lds + col;
                if (r < p.src_rows && col + 8 <= p.src_cols && (row | c) != 0) {
                    // 16 bytes from the 4-byte boundary at or before s
                    const bool odd = (uintptr_t)s & 2;
                    v[i] = ((const any *)(s - (odd ? 1 : 0)))->v;
                    if (odd) {
                        const uint32_t last = s[7];
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            v[i][e] = (v[i][e] >> 16) | (v[i][e + 1] << 16);
                        v[i][3] = (v[i][3] >> 16) | (last << 16);
                    }
                } else {
                    uint32_t h[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        h[e] = r < p.src_rows && col + e < p.src_cols ? (uint32_t)s[e] : 0u;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[i][e] = h[2 * e] | (h[2 * e + 1] << 16);
                }
            }
            row += step_rows;
            c += step_cols;
            if (c >= cols8) {
                c -= cols8;
                ++row;
            }
        }
#pragma unroll
        for (int i = 0; i < kPackChunks; ++i)
            if (d[i])
                *(pack_u32x4 *)d[i] = v[i];
    }
}

}  // namespace xgemm_dev
