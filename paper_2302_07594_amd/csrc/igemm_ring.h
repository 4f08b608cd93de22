// Ring kernel: the mid-size products (a few hundred rows over wide B, odd
// sizes and odd leading dimensions, lowered convolutions, short k) that are
// neither large enough for the direct and packed kernels' one-workgroup-per-
// compute-unit pipelines nor small enough for the small-output kernel.
//
// What bounds these products is not the matrix cores but the way from L2 to
// LDS: a compute unit keeps 84 to 100 line requests in flight whatever the
// number of stages (rocprofv3's request latency over time; three or seven
// k-tiles in flight make no difference), so what counts is how few requests
// bring a tile and how little else the waves issue. Hence:
//   * A and B move into LDS as they lie in memory, k-tile by k-tile, into a
//     ring of NST stages. B is turned k-contiguous by the LDS transpose reads
//     (ds_read_b64_tr_b8) on the way to the matrix cores, not by byte permutes
//     on the way in (the fused tiles' way). A's rows in a k-tile are 128 bytes
//     (BK = 128 int8, 64 int16): one request a row, where 64-byte rows took two
//     (int8 2048 x 4096 x 4096 54 us against 62 when it was chosen);
//   * int8 operands whose rows start at 4-byte addresses (REG = false) go by
//     buffer DMA (buffer_load_dwordx4 ... lds). Rows beyond m, and rows of B
//     beyond the k range, lie outside the resources and land as zeros, so no
//     k or m tail needs a branch or a mask;
//   * other alignments and int16 (REG = true) go through registers, two k-tiles
//     ahead, with unaligned 16-byte loads. int16 is split into its limbs
//     there, once per element (the split after LDS, once per fragment and
//     wave, cost the same matrix work twice the vector instructions: (4096,
//     4096, 1024) 90 us against 105), and the LDS writes of tile kt + 1 are
//     issued between the matrix instructions of tile kt. Only k-tiles that
//     reach beyond the k range or a matrix's end are apart: they go first, and
//     take bounded loads where they touch the end;
//   * AM = 1: A is the IM2ROW matrix of a convolution (Sec. 4.2) whose
//     channel rows are whole 16-byte chunks, each chunk inside one filter tap.
// Two or more workgroups share a compute unit (one, int16 128 x 128). Against
// the fused tiles that took these products (us a call, operands in the caches):
// int8 512 x 4096 x 4096 17.8 from 30.0, 1000 x 3001 x 1777 19.1 from 44.6; int16
// 777 x 1111 x 2049 21.8 from 30.6, 1536^3 24.0 from 45.2.
//
// int16 exactness (limb identity): with h = x >> 8, l' = (x & 255) - 128,
//   sum_p x_p y_p = 65536 S_hh + 256 (S_hl' + S_l'h) + S_l'l'
//                   + 128 R + 128 c + 16384 K
// with R and c the row's and the column's sums of 256 h + l' over the K = BK
// (k-tiles) positions the workgroup multiplies. It holds for whatever values A
// has beyond its k range as long as B is zero there, so padding needs no masks.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "igemm.h"
#include "igemm_device.h"
#include "igemm_internal.h"
#include "igemm_lds.h"

namespace igemm {
namespace ring {

using namespace lds;

enum { EPI_ADD = 0, EPI_ATOMIC = 1, EPI_SRS = 2 };

__device__ __forceinline__ u32 div_by(u32 x, DivU32 dv) {
    const u32 t = __umulhi(x, dv.mul);
    return (t + ((x - t) >> dv.s1)) >> dv.s2;
}

// 16-byte chunk c of LDS row r sits at c ^ swz(r). A rows of 64 bytes (int8,
// 64 k) or 128 (int8, 128 k; int16, 64 high limbs and 64 low limbs): the
// fragment reads (32 rows at one chunk) are free of bank conflicts. B rows (one
// k) of 64, 128 or 256 bytes (int16: high limbs, then low limbs): a transpose
// read takes 8 consecutive rows x 32 bytes per 32 lanes, which the swizzle
// spreads over all 64 banks. The low row bits move the highest chunk bit, so
// that the split int16 chunks, written as half rows, also spread.
template <int RA>
__device__ __forceinline__ int swz_a(int row) {
    static_assert(RA == 64 || RA == 128, "A rows of 64 or 128 bytes");
    if constexpr (RA == 128) return 4 * ((row >> 1) & 1) + (row & 4) / 2 + ((row >> 3) & 1);
    else return ((row >> 1) ^ (row >> 2)) & 3;
}
template <int RB>
__device__ __forceinline__ int swz_b(int row) {
    static_assert(RB == 64 || RB == 128 || RB == 256, "B rows of 64, 128 or 256 bytes");
    if constexpr (RB == 64) return 2 * ((row >> 2) & 1);
    else if constexpr (RB == 128) return 4 * ((row >> 1) & 1) + 2 * ((row >> 2) & 1);
    else return 8 * (row & 1) + 4 * ((row >> 1) & 1) + 2 * ((row >> 2) & 1);
}

// 16 bytes at any address.
__device__ __forceinline__ v4i load_u16(const char *p) {
    v4i v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// The 16 bytes at base + off (off >= 0) of a matrix that ends at base + end, with
// zeros past its end; reads only inside the matrix. One load, moved back inside
// the matrix and shifted into place, with no branch, so that the loads of
// several chunks are in flight together; it runs past the end of a row into the
// next one, whose values end up in columns or against rows that the caller
// discards. (Bounded by the row's end instead, rows of fewer than 16 bytes went
// a byte at a time, 2.4 us a k-tile: int8 10000 x 8 x 256 7.9 us, now 5.3.)
// tiny: the whole matrix has fewer than 16 bytes (uniform).
__device__ __forceinline__ v4i load_edge(const char *base, int off, int end, bool tiny) {
    if (!tiny) {
        const int o = min(off, end - 16), b = off - o;  // b bytes to drop, >= 0
        const v4i v = load_u16(base + o);
        const u32 w0 = (u32)v.x, w1 = (u32)v.y, w2 = (u32)v.z, w3 = (u32)v.w;
        // Whole words, then bytes, in 32 bits: a 64-bit shift whose amount is
        // in the last register a kernel has allocated takes v0 instead (measured
        // on gfx950: rows shifted by their lane's number of bits), and the
        // compiler keeps it out of that register on gfx90a only.
        const bool s1 = (b & 4) != 0, s2 = (b & 8) != 0, s4 = b >= 16;
        const u32 t0 = s1 ? w1 : w0, t1 = s1 ? w2 : w1, t2 = s1 ? w3 : w2, t3 = s1 ? 0u : w3;
        const u32 u0 = s4 ? 0u : (s2 ? t2 : t0), u1 = s4 ? 0u : (s2 ? t3 : t1);
        const u32 u2 = s4 || s2 ? 0u : t2, u3 = s4 || s2 ? 0u : t3;
        return v4i{(int)__builtin_amdgcn_alignbyte(u1, u0, (u32)b),
                   (int)__builtin_amdgcn_alignbyte(u2, u1, (u32)b),
                   (int)__builtin_amdgcn_alignbyte(u3, u2, (u32)b),
                   (int)__builtin_amdgcn_alignbyte(0u, u3, (u32)b)};
    }
    u32 w[4] = {0u, 0u, 0u, 0u};
#pragma unroll 1
    for (int i = 0; i < 16 && off + i < end; ++i) {
        const u32 x = (u32)(uint8_t)base[off + i] << (8 * (i & 3));
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] |= (i >> 2) == q ? x : 0u;
    }
    return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

typedef u32 v4u __attribute__((ext_vector_type(4)));

// Words of a raw buffer resource of `bytes` bytes at p.
__device__ __forceinline__ v4u resource(const char *p, u32 bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    v4u r;
    r.x = (u32)__builtin_amdgcn_readfirstlane((int)(u32)a);
    r.y = (u32)__builtin_amdgcn_readfirstlane((int)(u32)(a >> 32)) & 0xffffu;
    r.z = (u32)__builtin_amdgcn_readfirstlane((int)bytes);
    r.w = 0x00020000u;
    return r;
}

// One wave-wide DMA: lane i's 16 bytes at offset voff of the resource (the
// whole offset, since the range check may leave scalar offsets out) to LDS
// address lds + 16 i. Inline assembly, because the compiler's waits do not
// follow DMA data that is used a loop iteration later: the kernel counts its
// own (the kernel makes no other use of M0).
__device__ __forceinline__ void dma(u32 voff, v4u rs, u32 lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                 ::"v"(voff), "s"(rs), "s"(lds)
                 : "memory");
}

// ES: operand bytes; BM x BN: C tile of the workgroup, WM x WN of a wave; BK:
// k elements per tile; NST: ring stages; OCC: workgroups per compute unit the
// registers are held to. EPI_SRS: int16 C += srs(A B), one block of k, epi =
// shift | round_half_up << 8.
template <int ES, int BM, int BN, int WM, int WN, int BK, int NST, int OCC, int AM, bool REG,
          int EPI>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64,
                                  OCC *((BM / WM) * (BN / WN)) / 4)
igemm_ring(const char *__restrict__ A, int64_t lda, const char *__restrict__ B, int64_t ldb,
           int32_t *__restrict__ C, int64_t ldc, int m, int n, int k, int kchunk, int tiles_m,
           int tiles_n, ConvGeom g, int epi) {
    typedef Mfma<32> M;
    typedef typename M::acc_t acc_t;
    constexpr int NACC = ES == 2 ? 3 : 1;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int WGN = BN / WN, NW = (BM / WM) * WGN;
    constexpr int RA = BK * ES, RB = BN * ES;
    constexpr int APL = BM * RA, BPL = BK * RB, STAGE = APL + BPL;
    constexpr int RPA = 1024 / RA, RPB = 1024 / RB;  // rows per 1 KB block
    static_assert(APL % (1024 * NW) == 0 && BPL % (1024 * NW) == 0, "1 KB blocks per wave");
    constexpr int DPA = APL / 1024 / NW, DPB = BPL / 1024 / NW, DPW = DPA + DPB;
    constexpr int KS = BK / 32;  // sub-steps of 32 k
    static_assert(NST >= 2 && (NST - 2) * DPW < 64, "outstanding DMA count");
    static_assert(!REG || NST == 2, "two stages through registers");
    static_assert(ES == 1 || REG, "int16 is split on its way through registers");
    static_assert(ES == 1 || WGN >= 2, "int16: 2 x 2 waves share the sums");
    // int16: a sum per row and column of the tile; the int16-output update keeps
    // two terms of each (below).
    constexpr int NSUM = ES == 2 ? (BM + BN) * (EPI == EPI_SRS ? 2 : 1) : 4;
    static_assert(OCC * (NST * STAGE + 4 * NSUM) <= 160 * 1024, "LDS");

    __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];
    __shared__ __attribute__((aligned(16))) int sums[NSUM];

    // Named up front so that the argument loads issue together.
    asm volatile("" ::"s"(A), "s"(lda), "s"(B), "s"(ldb), "s"(C), "s"(ldc), "s"(m), "s"(n),
                 "s"(k), "s"(kchunk), "s"(tiles_m), "s"(tiles_n), "s"(gridDim.x), "s"(epi));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;

    // Workgroup -> (k slice, tile). Workgroup ids go to the eight XCDs in
    // turn: renumber them so that each XCD takes a contiguous range, walked in
    // groups of eight tile rows, so that the tiles that run together on one
    // XCD share A rows and B columns in its L2.
    int bid = blockIdx.x;
    {
        const int G = gridDim.x, q = G >> 3, r = G & 7, x = bid & 7;
        bid = x * q + min(x, r) + (bid >> 3);
    }
    const int tiles = tiles_m * tiles_n;
    const int z = bid / tiles, t = bid - z * tiles;
    constexpr int GROUP = 8;
    const int span = GROUP * tiles_n;
    const int first_m = (t / span) * GROUP;
    const int gsize = min(tiles_m - first_m, GROUP);
    const int tm = first_m + (t % span) % gsize, tn = (t % span) / gsize;
    const int m0 = tm * BM, n0 = tn * BN;
    const int kbeg = z * kchunk, kend = min(k, kbeg + kchunk);
    const int klen = kend - kbeg;  // >= 1 (planner)
    const int nkt = (klen + BK - 1) / BK;

    // ---- C: resource at the tile's corner ------------------------------------
    // It ends at the last valid element of the tile's rows, and columns past n
    // get an offset beyond any range (loads give zero, stores are dropped), so
    // the update needs no branches. The planner keeps BM rows of C below 2 GiB.
    constexpr int CE = EPI == EPI_SRS ? 2 : 4;
    const int mrows = min(m - m0, BM);
    const int ldc_b = (int)ldc * CE;
    const __amdgpu_buffer_rsrc_t Crs = __builtin_amdgcn_make_buffer_rsrc(
        (char *)C + ((int64_t)m0 * ldc + n0) * CE, 0, (mrows - 1) * ldc_b + min(n - n0, BN) * CE,
        0x00020000);
    u32 c_vo[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int lc = wn0 + 32 * j + M::out_col(lane);
        c_vo[j] = n0 + lc < n ? (u32)((wm0 + M::out_row(lane, 0)) * ldc_b + lc * CE) : 0x80000000u;
    }
    auto c_off = [&](int i, int j, int r) __attribute__((always_inline)) -> u32 {
        return c_vo[j] + (u32)((32 * i + M::out_row(0, r)) * ldc_b);
    };

    // ---- staging geometry ----------------------------------------------------
    // Lane i of 1 KB block b moves 16 bytes: chunk i % (RA / 16) of A's row
    // b RPA + i / (RA / 16), B likewise. By DMA they land at LDS bytes
    // [16 i, 16 i + 16) of the block, so the lane fetches the logical chunk that
    // the swizzle puts there; through registers the store swizzles.
    int a_row[DPA], a_lc[DPA], b_row[DPB], b_lc[DPB];
#pragma unroll
    for (int d = 0; d < DPA; ++d) {
        a_row[d] = (wave * DPA + d) * RPA + lane / (RA / 16);
        a_lc[d] = (lane % (RA / 16)) ^ (REG ? 0 : swz_a<RA>(a_row[d]));
    }
#pragma unroll
    for (int d = 0; d < DPB; ++d) {
        b_row[d] = (wave * DPB + d) * RPB + lane / (RB / 16);
        b_lc[d] = (lane % (RB / 16)) ^ (REG ? 0 : swz_b<RB>(b_row[d]));
    }
    const int lda_b = (int)(lda * ES), ldb_b = (int)(ldb * ES);
    const char *a_base = AM == 1 ? A : A + ((int64_t)m0 * lda + kbeg) * ES;
    const char *b_base = B + ((int64_t)kbeg * ldb + n0) * ES;

    // IM2ROW: the output pixel of each of this lane's A rows, decoded once:
    // first input row and column of its window, and the window's byte offset
    // in X (a row past m gets a window outside the image).
    int cv_y[AM == 1 ? DPA : 1], cv_x[AM == 1 ? DPA : 1], cv_o[AM == 1 ? DPA : 1];
    if constexpr (AM == 1) {
#pragma unroll
        for (int d = 0; d < DPA; ++d) {
            const u32 p = (u32)(m0 + a_row[d]);
            const u32 img = div_by(p, g.by_ohw);
            const u32 rem = p - img * (u32)g.ohw;
            const u32 oy = div_by(rem, g.by_ow), ox = rem - oy * (u32)g.ow;
            const bool ok = p < (u32)m;
            cv_y[d] = ok ? (int)oy * g.sh - g.ph : -(1 << 30);
            cv_x[d] = (int)ox * g.sw - g.pw;
            // (modulo 2^32: exact where the tap is inside the image)
            cv_o[d] = (int)((((img * (u32)g.h + (u32)cv_y[d]) * (u32)g.w + (u32)cv_x[d]) *
                             (u32)g.c) * (u32)ES);
        }
    }
    // Byte offset in X of chunk d of k-tile kt, 0x80000000 (outside X) where
    // the tap falls outside the image or the chunk beyond k.
    auto conv_off = [&](int d, int kt) __attribute__((always_inline)) -> u32 {
        const int e = kt * BK + a_lc[d] * (16 / ES);
        const u32 p = (u32)(kbeg + e);
        const u32 tap = div_by(p, g.by_c);
        const int ci = (int)(p - tap * (u32)g.c);
        const u32 fy = div_by(tap, g.by_s);
        const int dy = (int)fy * g.dh, dx = (int)(tap - fy * (u32)g.s) * g.dw;
        const bool in = e < klen && (u32)(cv_y[d] + dy) < (u32)g.h &&
                        (u32)(cv_x[d] + dx) < (u32)g.w;
        return in ? (u32)cv_o[d] + (u32)((dy * g.w + dx) * g.c + ci) * (u32)ES : 0x80000000u;
    };

    const u32 lds0 = (u32)(uintptr_t)(const __attribute__((address_space(3))) char *)smem;

    // ---- DMA staging -----------------------------------------------------------
    u32 a_vo[DPA], b_vo[DPB];
    v4u Ars = {0u, 0u, 0u, 0u}, Brs = {0u, 0u, 0u, 0u};
    if constexpr (!REG) {
        // The resources end at the last row's last element of the window
        // (rounded up to the dword); rows of B past the k range lie beyond.
        if constexpr (AM == 1) {
            Ars = resource(A, (u32)g.x_bytes);
        } else {
            Ars = resource(a_base, (u32)(((mrows - 1) * lda_b + (k - kbeg) * ES + 3) & ~3));
        }
        Brs = resource(b_base, (u32)(((klen - 1) * ldb_b + (n - n0) * ES + 3) & ~3));
#pragma unroll
        for (int d = 0; d < DPA; ++d)
            a_vo[d] = a_row[d] < mrows ? (u32)(a_row[d] * lda_b + 16 * a_lc[d]) : 0x80000000u;
#pragma unroll
        for (int d = 0; d < DPB; ++d) b_vo[d] = (u32)(b_row[d] * ldb_b + 16 * b_lc[d]);
    }
    // k-tile kt into stage s. Tiles past the range are issued too, on empty
    // resources (no memory traffic), so that every wave always counts DPW
    // DMAs per tile.
    auto issue = [&](int kt, int s) __attribute__((always_inline)) {
        const bool in = kt < nkt;
        v4u ar = Ars, br = Brs;
        ar.z = in ? ar.z : 0u;
        br.z = in ? br.z : 0u;
        const u32 as = in ? (u32)(kt * RA) : 0u;
        const u32 bs = in ? (u32)(kt * BK) * (u32)ldb_b : 0u;
        const u32 base = lds0 + (u32)(s * STAGE);
#pragma unroll
        for (int d = 0; d < DPA; ++d) {
            u32 o;
            if constexpr (AM == 1) o = conv_off(d, kt);
            else o = a_vo[d] + as;
            dma(o, ar, base + (u32)((wave * DPA + d) * 1024));
        }
#pragma unroll
        for (int d = 0; d < DPB; ++d)
            dma(b_vo[d] + bs, br, base + (u32)(APL + (wave * DPB + d) * 1024));
    };

    // ---- register staging -------------------------------------------------------
    // k-tiles [0, nwhole) are read without checks: every k of the tile lies in
    // the range and the last row's last 16 bytes (which may run past n into
    // the next row) before B's end. The others, usually one, are read up to the
    // matrices' ends, with B's rows beyond the range set to zero, and multiplied
    // first, while the first whole tiles are on the way (the order of k does not
    // change the sums).
    typedef v4i regs_a[REG ? DPA : 1];
    typedef v4i regs_b[REG ? DPB : 1];
    int nwhole = 0;
    bool a_tiny = false, b_tiny = false;
    if constexpr (REG) {
        a_tiny = ((int64_t)(m - 1) * lda + k) * ES < 16;
        b_tiny = ((int64_t)(k - 1) * ldb + n) * ES < 16;
        const int64_t b_avail = (int64_t)(k - 1 - kbeg) * ldb_b + (int64_t)(n - n0) * ES - RB;
        int64_t rows = b_avail < 0 ? 0 : b_avail / ldb_b + 1;  // rows readable in full
        if (rows > klen) rows = klen;
        nwhole = (int)rows / BK;
    }
    const __amdgpu_buffer_rsrc_t Xrs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)A, 0, AM == 1 ? g.x_bytes : 0, 0x00020000);
    auto load = [&](regs_a &va, regs_b &vb, int kt) __attribute__((always_inline)) {
        if constexpr (REG) {
            const char *ak = a_base + (int64_t)kt * RA;
            const char *bk = b_base + (int64_t)kt * BK * ldb_b;
#pragma unroll
            for (int d = 0; d < DPA; ++d) {
                if constexpr (AM == 1)
                    va[d] = __builtin_amdgcn_raw_buffer_load_b128(Xrs, conv_off(d, kt), 0, 0);
                else
                    va[d] = load_u16(ak + (u32)(min(a_row[d], mrows - 1) * lda_b + 16 * a_lc[d]));
            }
#pragma unroll
            for (int d = 0; d < DPB; ++d)
                vb[d] = load_u16(bk + (u32)(b_row[d] * ldb_b + 16 * b_lc[d]));
        }
    };
    auto load_checked = [&](regs_a &va, regs_b &vb, int kt) __attribute__((always_inline)) {
        if constexpr (REG) {
            const int k0 = kt * BK, left = klen - k0;  // k positions left, >= 1
            const char *ak = a_base + (int64_t)kt * RA;
            const char *bk = b_base + (int64_t)k0 * ldb_b;
            // Ends of the matrices, from here (offsets in the windows are below
            // 2^31). A tile inside both takes plain loads, all in flight at once;
            // the others, in the last row or column of tiles, bounded ones.
            const int a_end = (int)min(((int64_t)(m - 1 - m0) * lda + (k - kbeg - k0)) * ES,
                                       (int64_t)0x7fffffff);
            const int b_end = (int)min(((int64_t)(k - 1 - kbeg - k0) * ldb + (n - n0)) * ES,
                                       (int64_t)0x7fffffff);
            int a_off[DPA], b_off[DPB];
#pragma unroll
            for (int d = 0; d < DPA; ++d)
                a_off[d] = min(a_row[d], mrows - 1) * lda_b + 16 * a_lc[d];
#pragma unroll
            for (int d = 0; d < DPB; ++d)
                b_off[d] = min(b_row[d], left - 1) * ldb_b + 16 * b_lc[d];
            if ((AM == 1 || (mrows - 1) * lda_b + RA <= a_end) &&
                (left - 1) * ldb_b + RB <= b_end) {
#pragma unroll
                for (int d = 0; d < DPA; ++d) {
                    if constexpr (AM == 1)
                        va[d] = __builtin_amdgcn_raw_buffer_load_b128(Xrs, conv_off(d, kt), 0, 0);
                    else
                        va[d] = load_u16(ak + a_off[d]);
                }
#pragma unroll
                for (int d = 0; d < DPB; ++d) vb[d] = load_u16(bk + b_off[d]);
            } else {
#pragma unroll
                for (int d = 0; d < DPA; ++d) {
                    if constexpr (AM == 1)
                        va[d] = __builtin_amdgcn_raw_buffer_load_b128(Xrs, conv_off(d, kt), 0, 0);
                    else
                        va[d] = load_edge(ak, a_off[d], a_end, a_tiny);
                }
#pragma unroll
                for (int d = 0; d < DPB; ++d) vb[d] = load_edge(bk, b_off[d], b_end, b_tiny);
            }
#pragma unroll
            for (int d = 0; d < DPB; ++d)
                if (b_row[d] >= left) vb[d] = v4i{0, 0, 0, 0};
        }
    };
    // int16 is split here, once per element: a chunk's 8 elements become 8
    // bytes of the row's high half and 8 of its low half.
    auto store = [&](const regs_a &va, const regs_b &vb, int s) __attribute__((always_inline)) {
        if constexpr (REG) {
            char *sa = smem + s * STAGE, *sb = sa + APL;
            auto put = [&](char *row, int swz, int half, int lc, v4i v)
                           __attribute__((always_inline)) {
                if constexpr (ES == 1) {
                    *(v4i *)(row + 16 * (lc ^ swz)) = v;
                } else {
                    const u32 x = (u32)v.x, y = (u32)v.y, z = (u32)v.z, w = (u32)v.w;
                    const int c = lc >> 1, o = 8 * (lc & 1);
                    *(uint2 *)(row + 16 * (c ^ swz) + o) = make_uint2(hi4(y, x), hi4(w, z));
                    *(uint2 *)(row + 16 * ((c + half) ^ swz) + o) =
                        make_uint2(lo4(y, x), lo4(w, z));
                }
            };
#pragma unroll
            for (int d = 0; d < DPA; ++d)
                put(sa + a_row[d] * RA, swz_a<RA>(a_row[d]), RA / 32, a_lc[d], va[d]);
#pragma unroll
            for (int d = 0; d < DPB; ++d)
                put(sb + b_row[d] * RB, swz_b<RB>(b_row[d]), RB / 32, b_lc[d], vb[d]);
        }
    };

    // ---- fragments and matrix instructions ------------------------------------
    // A: lane row fr = lane % 32 of each 32-row block, k chunk q = 2 ks +
    // lane / 32 of 16 elements. B: transpose reads, group gq = lane / 16 covers
    // columns 16 (gq % 2) + [0, 16) of a 32-column block and k chunk 2 ks +
    // gq / 2; lane u = lane % 16 addresses k row 16 q + 8 r + u / 2 (r < 2) at
    // columns 8 (u % 2). int16: limb plane p (0 high, 1 low) of either.
    constexpr int P = ES;
    const int fr = lane & 31, gq = lane >> 4, u = lane & 15;
    int a_rd[KS][P], b_rd[P][TN];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int row = wm0 + fr, krow = 16 * (gq >> 1) + (u >> 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            a_rd[ks][p] =
                row * RA + 16 * ((p * (RA / 32) + 2 * ks + (lane >> 5)) ^ swz_a<RA>(row));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int cb = p * BN + wn0 + 32 * j + 16 * (gq & 1) + 8 * (u & 1);
            b_rd[p][j] = APL + krow * RB + 16 * ((cb >> 4) ^ swz_b<RB>(krow)) + (cb & 15);
        }
    }
    acc_t acc[NACC][TM][TN];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < M::REGS; ++r) acc[a][i][j][r] = 0;
    // int16: limb sums of this wave's share, its rows of A or its columns of
    // B: each row by one wave, each column by one or, with four waves across a
    // tile, two (to the same value).
    constexpr int NPS = ES == 2 ? (TM > TN ? TM : TN) : 1;
    int sum_h[NPS], sum_l[NPS];
#pragma unroll
    for (int i = 0; i < NPS; ++i) sum_h[i] = sum_l[i] = 0;

    auto tile = [&](auto rows_c, int s) __attribute__((always_inline)) {
        constexpr bool ROWS = decltype(rows_c)::value != 0;
        const char *st = smem + s * STAGE;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            v4i a[P][TM], b[P][TN];
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    // (the swizzle repeats every 8 rows)
                    const char *q = st + b_rd[p][j] + ks * 32 * RB;
                    const v2i x = tr8(q), y = tr8(q + 8 * RB);
                    b[p][j] = v4i{x.x, x.y, y.x, y.y};
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    a[p][i] = *(const v4i *)(st + a_rd[ks][p] + i * 32 * RA);
            }
            // (int16: hh, hl', l'l', l'h over all blocks in turn, so that the two
            // products of one accumulator lie apart)
#pragma unroll
            for (int x = 0; x < P * P; ++x) {
                constexpr int pa[4] = {0, 0, 1, 1}, pb[4] = {0, 1, 1, 0}, pc[4] = {0, 1, 2, 1};
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[pc[x]][i][j] = M::mma(a[pa[x]][i], b[pb[x]][j], acc[pc[x]][i][j]);
            }
            if constexpr (ES == 2) {
#pragma unroll
                for (int i = 0; i < (ROWS ? TM : TN); ++i)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        sum_h[i] = sum4((u32)(ROWS ? a[0][i] : b[0][i])[x], sum_h[i]);
                        sum_l[i] = sum4((u32)(ROWS ? a[1][i] : b[1][i])[x], sum_l[i]);
                    }
            }
        }
    };

    // ---- C ahead of the k loop ---------------------------------------------------
    // The read of C overlaps the first tiles' loads where registers are there
    // for it (16 per 32 x 32 block); the register-staged form reads it after
    // the loop.
    constexpr bool PRE = EPI != EPI_ATOMIC && !REG;
    int32_t cv[EPI == EPI_ATOMIC ? 1 : TM][EPI == EPI_ATOMIC ? 1 : TN][M::REGS];
    auto load_c = [&](int i) __attribute__((always_inline)) {
        if constexpr (EPI != EPI_ATOMIC) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < M::REGS; ++r) {
                    if constexpr (EPI == EPI_SRS)
                        cv[i][j][r] = (int32_t)(int16_t)__builtin_amdgcn_raw_buffer_load_b16(
                            Crs, c_off(i, j, r), 0, 0);
                    else
                        cv[i][j][r] =
                            __builtin_amdgcn_raw_buffer_load_b32(Crs, c_off(i, j, r), 0, 0);
                }
        }
    };
    if constexpr (PRE)
#pragma unroll
        for (int i = 0; i < TM; ++i) load_c(i);

    // ---- k loop ---------------------------------------------------------------------
    auto run = [&](auto rows_c) __attribute__((always_inline)) {
        if constexpr (!REG) {
#pragma unroll
            for (int s = 0; s < NST - 1; ++s) issue(s, s);
            int s = 0;
            for (int kt = 0; kt < nkt; ++kt) {
                // tile kt has landed when at most the NST - 2 later tiles' DMAs
                // are outstanding; every read of the stage freed below is done
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NST - 2) * DPW)
                             : "memory");
                issue(kt + NST - 1, s == 0 ? NST - 1 : s - 1);
                tile(rows_c, s);
                s = s == NST - 1 ? 0 : s + 1;
            }
            // no DMA may land in LDS that the next workgroup owns
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
            regs_a va0, va1;
            regs_b vb0, vb1;
            if (nwhole > 0) load(va0, vb0, 0);
            if (nwhole > 1) load(va1, vb1, 1);
            for (int kt = nwhole; kt < nkt; ++kt) {
                regs_a va;
                regs_b vb;
                load_checked(va, vb, kt);
                store(va, vb, 1);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                tile(rows_c, 1);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            // Tile kt goes through stage kt % 2 and register set kt % 2. The
            // store of tile kt + 1 is interleaved with the matrix instructions
            // of tile kt (past the last tile it writes a stage nobody reads).
            if (nwhole > 0) store(va0, vb0, 0);
            if (nwhole > 2) load(va0, vb0, 2);
            auto step = [&](regs_a &va, regs_b &vb, int kt, auto par) __attribute__((always_inline)) {
                constexpr int S = decltype(par)::value;
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                tile(rows_c, S);
                store(va, vb, 1 - S);
                constexpr int NM = KS * TM * TN * P * P, NR = P * (TM + 2 * TN);
                constexpr int NW_ = P * DPW, NV = ES == 2 ? 6 * DPW + 8 * KS * NPS : 0;
                __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, (NR * (KS - 1) + NM - 1) / NM, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, (NV + NM - 1) / NM, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, (NW_ + NM - 1) / NM, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (kt + 3 < nwhole) load(va, vb, kt + 3);
            };
            for (int kt = 0; kt < nwhole; kt += 2) {
                step(va1, vb1, kt, ic<0>{});
                if (kt + 1 >= nwhole) break;
                step(va0, vb0, kt + 1, ic<1>{});
            }
        }
    };
    const bool rows_wave = ES == 2 && (wave / WGN) % WGN == wave % WGN;
    if constexpr (ES == 2) {
        if (rows_wave) run(ic<1>{});
        else run(ic<0>{});
    } else {
        run(ic<0>{});
    }

    // ---- update of C ------------------------------------------------------------------
    if constexpr (!PRE)
#pragma unroll
        for (int i = 0; i < TM; ++i) load_c(i);
    if constexpr (ES == 2) {
        // Lanes l and l + 32 hold complementary k chunks of one row or column.
#pragma unroll
        for (int i = 0; i < NPS; ++i) {
            // sum of the 256 h + l' (the 128 per element goes into the constant)
            const int w = 256 * sum_h[i] + sum_l[i], v = w + __shfl_xor(w, 32);
            if (lane < 32 && i < (rows_wave ? TM : TN)) {
                const int at = rows_wave ? wm0 + 32 * i + lane : BM + wn0 + 32 * i + lane;
                if constexpr (EPI == EPI_SRS) {
                    sums[at] = v >> 1;
                    sums[BM + BN + at] = 128 * (v & 1);
                } else {
                    sums[at] = v;
                }
            }
        }
        __syncthreads();
    }
    const int kmul = BK * nkt;  // k positions multiplied
    // int16 conversion, in 32-bit arithmetic (the planner keeps a block of the
    // update at most 2^14 elements long). int16 operands: with x = S_x + R / 2
    // + c / 2 and l = S_ll + 128 (R % 2 + c % 2) + 16384 K (|x|, |l| < 2^31)
    // the product is
    //   v = 2^16 z + 2^8 (y mod 2^8) + l mod 2^8,  y = x + floor(l / 2^8),
    //   z = S_hh + floor(y / 2^8).
    // Shifts up to 15: z outside int16 saturates the result whatever its
    // value (by more than the rounding unit), so clamped to int16 it gives v in
    // 32 bits, the unit is added with saturation (beyond 2^31 the result
    // saturates too), then the shift. Shifts from 16 on drop the low 16 bits:
    // (z + rounding) >> (shift - 16), where the rounding of shift 16 is bit 15
    // of v; shift 0 needs neither rounding nor a shift. R / 2 and 128 (R % 2) of a
    // row, and of a column, are formed once, where the sum is, and read from
    // LDS: the conversion was almost half of the kernel's vector instructions,
    // which bound it (rocprofv3: 12.1 million, 40 % of the cycles, against 17 %
    // for the matrix cores); with both, and operands that are not cached, (4096,
    // 4096, 290) 45.8 us to 43.5, (4065, 670, 1213) in blocks of 290 53.7 to 52.4.
    // int8: v fits in 30 bits; shifts above 31 act as 31, and the rounding unit
    // of 31 already rounds every v to 0.
    const int shift = epi & 0xff;
    const bool round = ((epi >> 8) & 1) != 0 && shift > 0;
    auto update = [&](auto mode_c) __attribute__((always_inline)) {
        constexpr bool WIDE = decltype(mode_c)::value == 1;  // shift >= 16
        constexpr bool NOSH = decltype(mode_c)::value == 2;  // shift 0
        const int sh = ES == 1 ? min(shift, 31) : (WIDE ? shift - 16 : shift);
        const int half = round && sh > 0 ? (int)(1u << (sh - 1)) : 0;
        const int bit15 = round && sh == 0 ? 1 : 0;  // WIDE: shift 16
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int rowt[M::REGS], rowl[M::REGS];
            auto row_terms = [&](int (&t)[M::REGS], int at) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < M::REGS; r += 4) {
                    const int4 q = *(const int4 *)(sums + at + wm0 + 32 * i + M::out_row(lane, r));
                    t[r] = q.x;
                    t[r + 1] = q.y;
                    t[r + 2] = q.z;
                    t[r + 3] = q.w;
                }
            };
            if constexpr (ES == 2) row_terms(rowt, 0);
            if constexpr (ES == 2 && EPI == EPI_SRS) row_terms(rowl, BM + BN);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int colt = ES == 2 ? sums[BM + wn0 + 32 * j + M::out_col(lane)] : 0;
                const int coll =
                    ES == 2 && EPI == EPI_SRS
                        ? sums[BM + BN + BM + wn0 + 32 * j + M::out_col(lane)] + 16384 * kmul
                        : 0;
#pragma unroll
                for (int r = 0; r < M::REGS; ++r) {
                    const int a0 = acc[0][i][j][r];
                    if constexpr (EPI == EPI_SRS) {
                        int t;
                        if constexpr (ES == 1) {
                            t = (a0 + half) >> sh;
                        } else {
                            const int l = acc[2][i][j][r] + rowl[r] + coll;
                            const int y = acc[1][i][j][r] + rowt[r] + colt + (l >> 8);
                            const int z = a0 + (y >> 8);
                            if constexpr (WIDE) {
                                t = (z + half + ((y >> 7) & bit15)) >> sh;
                            } else {
                                const u32 zc = (u32)min(max(z, -32768), 32767);
                                const u32 v = perm(zc, perm((u32)y, (u32)l, 0x0c0c0400u),
                                                   0x05040100u);
                                t = NOSH ? (int)v
                                         : __builtin_elementwise_add_sat((int)v, half) >> sh;
                            }
                        }
                        t = min(max(t, -32768), 32767);
                        __builtin_amdgcn_raw_buffer_store_b16(
                            (unsigned short)(u32)(cv[i][j][r] + t), Crs, c_off(i, j, r), 0, 0);
                    } else {
                        u32 v = (u32)a0;
                        if constexpr (ES == 2)
                            v = 65536u * v + 256u * (u32)acc[1][i][j][r] +
                                (u32)acc[2][i][j][r] + 128u * ((u32)rowt[r] + (u32)colt) +
                                16384u * (u32)kmul;
                        if constexpr (EPI == EPI_ATOMIC) {
                            const int lr = wm0 + 32 * i + M::out_row(lane, r);
                            const int lc = wn0 + 32 * j + M::out_col(lane);
                            if (m0 + lr < m && n0 + lc < n)
                                atomicAdd(C + (int64_t)(m0 + lr) * ldc + (n0 + lc), (int)v);
                        } else {
                            __builtin_amdgcn_raw_buffer_store_b32((int)((u32)cv[i][j][r] + v),
                                                                  Crs, c_off(i, j, r), 0, 0);
                        }
                    }
                }
            }
        }
    };
    if (EPI == EPI_SRS && ES == 2 && shift >= 16)
        update(ic<1>{});
    else if (EPI == EPI_SRS && ES == 2 && shift == 0)
        update(ic<2>{});
    else
        update(ic<0>{});
}

}  // namespace ring
}  // namespace igemm
