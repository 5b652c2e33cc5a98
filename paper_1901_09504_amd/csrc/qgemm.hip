// The expanded layer (Eq. 2 over the expanded channel set) on int8 codes: an NT GEMM
// acc[i,n] = sum_k Xq[i,k] * Wq[n,k] on the matrix cores (v_mfma_i32_32x32x32_i8, int32
// accumulation, exact), with the trailing scale factors of Eq. 1 applied in the epilogue.
//
// Both operands are K-contiguous, so a lane's MFMA operand is 16 consecutive bytes of one
// row.  A workgroup computes a BM x BN tile; per K-step of 64 or 128 bytes the BM + BN row
// segments go from global memory straight into LDS (no staging registers), into a ring of
// buffers (long K) or all at once (short K).  LDS rows are BK bytes = 16-byte chunks whose
// index is XOR-swizzled with the row so that the 16-byte fragment reads of consecutive rows fall
// in different banks.  K is padded with zero codes to a multiple of 64 by the producers, so the
// K loop has no tail; zeros add nothing to an integer sum.
#include <atomic>
#include <type_traits>

#include "ocs_internal.h"

namespace ocs {

// LDS rows are BK bytes = BK/16 chunks of 16 bytes.  The chunk index is XOR-ed with a function
// of the row chosen so that the 16-byte reads of 8 (and of 16) consecutive rows at one K offset
// land in distinct bank groups.
template <int BK>
__device__ __forceinline__ int swz(int row, int chunk) {
    if (BK == 64) return chunk ^ (((row >> 2) & 3) ^ (row & 2));
    return chunk ^ (((row >> 1) & 7) ^ ((row & 1) << 2));
}

// index clamped into [0, n): index arrays and edge rows never send a load out of bounds
__device__ __forceinline__ int col_clamp(int v, int n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Renumber them so
// that consecutive tile ids (which share an X row panel) run on the same XCD.
__device__ __forceinline__ unsigned xcd_remap(unsigned w, unsigned total) {
    const unsigned q = total / 8, r = total % 8;
    const unsigned xcd = w % 8, local = w / 8;
    return xcd * q + (xcd < r ? xcd : r) + local;
}

// ---------------------------------------------------------------------------------------------
// The operands move global -> LDS directly (global_load_lds_dwordx4): no staging registers and no
// LDS write instructions, which on this chip cost as much LDS time as the fragment reads (the LDS
// takes ~73 B/clk of writes against ~190 B/clk of 16-byte reads).
// One such instruction fills 1 KB of LDS, lane l at byte 16*l of the wave's block (the block
// base travels in M0 and is wave-uniform), so the XOR swizzle is applied on the global side:
// the lane that fills chunk slot c of row r fetches chunk c ^ f(r) of that row.  NBUF LDS
// buffers form the prefetch ring; a wave waits for its own loads of the next step with vmcnt
// (loads return in order), and the step's barrier then makes every wave's part visible.
// ---------------------------------------------------------------------------------------------
template <int N_>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N_ >= 0 && N_ < 64, "vmcnt is a 6-bit counter");
    // s_waitcnt simm16: vmcnt[3:0], expcnt[6:4], lgkmcnt[11:8], vmcnt[5:4] in bits 15:14
    __builtin_amdgcn_s_waitcnt((N_ & 15) | (7 << 4) | (15 << 8) | ((N_ >> 4) << 14));
}

// The next layer's code of an accumulator, in the low byte: dequantized, ReLU, Eq. 1.  lo: -qmax, or 0
// with a ReLU (inv >= 0, so max(y, 0) inv clamped to +-qmax is y inv clamped to [0, qmax]).
__device__ __forceinline__ unsigned out_code_bits(int a, float scale, float lo, float inv, float qmax) {
    const float y = (float)a * scale;
    float p = y * inv;
    p = __builtin_amdgcn_fmed3f(p, lo, qmax);
    return __float_as_uint(p + 12582912.0f);           // round half to even; low byte = code
}

// Copies the next layer wants of this workgroup's output columns: entries (j << 8 | column
// inside the workgroup's BN columns) for every appended column N + j whose source lies in
// [col0, col0 + BN).  Built once per workgroup (a handful of entries: a few percent of BN).
constexpr int kDupCap = 512;
template <int NT>
__device__ __forceinline__ void build_dup_list(const Requant& rq, int N, int col0, int BN_, int* list,
                                               int* count) {
    if (rq.Yq == nullptr || rq.s_next <= 0) return;   // uniform over the grid
    if (threadIdx.x == 0) *count = 0;
    __syncthreads();
    for (int t = threadIdx.x; t < rq.s_next; t += NT) {
        int src = rq.chan_src[N + t];
        src = src < 0 ? 0 : (src >= N ? N - 1 : src);
        const int local = src - col0;
        if (local >= 0 && local < BN_) {
            const int k = atomicAdd(count, 1);
            if (k < kDupCap) list[k] = (t << 8) | local;
        }
    }
    __syncthreads();
}

// ROWS x WN accumulators of one wave, staged row-major in its piece of LDS, go out to memory.
// rbase / cbase: global row and column of the staged block's corner; wcol: its first column
// inside the workgroup's tile.  fp32 (and the optional int32 dump): lane = (row, four
// consecutive columns), 16-byte stores.  Codes: lane = (row, sixteen consecutive columns),
// again 16-byte stores.  STRIDE: accumulators from one staged row to the next.
template <int ROWS, int WN, int STRIDE = WN>
__device__ __forceinline__ void emit_staged_rows(const int32_t* stage, int lane, int rbase, int cbase,
                                                 int wcol, int M, int N, float scale,
                                                 float* __restrict__ Y, int64_t ldy,
                                                 int32_t* __restrict__ acc_out, int64_t ldacc,
                                                 bool vec_y, bool vec_a, const Requant& rq, float inv,
                                                 const int* dup_list, int dup_n, bool pad_writer, bool whole = false) {
    constexpr int LPR = WN / 4;            // lanes per row (8, 16 or 32)
    constexpr int SLOTS = ROWS * LPR;      // 16-byte reads of the block
    static_assert(SLOTS % 64 == 0 && 64 % LPR == 0, "whole waves of slots, whole rows of lanes");
    // whole: the workgroup's tile lies inside the output, as nearly all of a large one's do: no bounds, no
    // branch between the stores (for the tile, not per wave: where the last columns of a row share a line
    // with the next row's first, waves that run ahead of each other cost more, 100000 x 100 19 against 16.5 us)
    if (whole && rq.Yq == nullptr && acc_out == nullptr && vec_y) {
        float* yp = Y + (int64_t)(rbase + lane / LPR) * ldy + cbase + (lane % LPR) * 4;
        const int64_t step = (int64_t)(64 / LPR) * ldy;
#pragma unroll
        for (int it = 0; it < SLOTS / 64; ++it) {
            const i32x4 a = *reinterpret_cast<const i32x4*>(&stage[(it * (64 / LPR) + lane / LPR) * STRIDE + (lane % LPR) * 4]);
            f32x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (float)a[e] * scale;
            __builtin_nontemporal_store(y, reinterpret_cast<f32x4*>(yp + it * step));
        }
        return;
    }
    if (rq.Yq == nullptr || acc_out != nullptr) {
#pragma unroll
        for (int it = 0; it < SLOTS / 64; ++it) {
            const int idx = it * 64 + lane;
            const int rr = idx / LPR, cc = (idx % LPR) * 4;
            const i32x4 a = *reinterpret_cast<const i32x4*>(&stage[rr * STRIDE + cc]);
            const int r = rbase + rr, c = cbase + cc;
            if (r >= M || c >= N) continue;
            if (rq.Yq == nullptr) {
                float* yp = Y + (int64_t)r * ldy + c;
                if (vec_y && c + 3 < N) {
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = (float)a[e] * scale;
                    __builtin_nontemporal_store(y, reinterpret_cast<f32x4*>(yp));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < N) yp[e] = (float)a[e] * scale;
                }
            }
            if (acc_out) {
                int32_t* ap = acc_out + (int64_t)r * ldacc + c;
                if (vec_a && c + 3 < N) {
                    *reinterpret_cast<i32x4*>(ap) = a;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < N) ap[e] = a[e];
                }
            }
        }
    }
    if (rq.Yq == nullptr) return;

    const float lo = rq.relu ? 0.0f : -rq.qmax;
    constexpr int LPR16 = WN / 16;         // lanes per row, sixteen columns each (2, 4 or 8)
    constexpr int SLOTS16 = ROWS * LPR16;
#pragma unroll
    for (int it = 0; it < (SLOTS16 + 63) / 64; ++it) {
        const int idx = it * 64 + lane;
        if (idx >= SLOTS16) break;
        const int rr = idx / LPR16, cc = (idx % LPR16) * 16;
        const int r = rbase + rr, c = cbase + cc;
        unsigned w[4];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const i32x4 a = *reinterpret_cast<const i32x4*>(&stage[rr * STRIDE + cc + 4 * g4]);
            w[g4] = pack4(out_code_bits(a[0], scale, lo, inv, rq.qmax), out_code_bits(a[1], scale, lo, inv, rq.qmax),
                          out_code_bits(a[2], scale, lo, inv, rq.qmax), out_code_bits(a[3], scale, lo, inv, rq.qmax));
        }
        if (r >= M || c >= N) continue;
        int8_t* qp = rq.Yq + (int64_t)r * rq.ldyq + c;      // 16-byte aligned: ldyq % 16 == 0, c % 16 == 0
        if (c + 15 < N) {
            i32x4 v;
            v[0] = (int)w[0]; v[1] = (int)w[1]; v[2] = (int)w[2]; v[3] = (int)w[3];
            *reinterpret_cast<i32x4*>(qp) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (c + e < N) qp[e] = (int8_t)((w[e >> 2] >> (8 * (e & 3))) & 0xFFu);
        }
    }
    // copies for the channels the next layer splits: the wave that holds the source column writes
    // appended column N + j; (row, copy) pairs over the lanes, rows first
    for (int idx = lane; idx < ROWS * dup_n; idx += 64) {
        const int e = dup_list[idx / ROWS], rr = idx % ROWS, r = rbase + rr;
        const int local = (e & 0xFF) - wcol;
        if (local >= 0 && local < WN && r < M)
            rq.Yq[(int64_t)r * rq.ldyq + N + (e >> 8)] = (int8_t)out_code_bits(stage[rr * STRIDE + local], scale, lo, inv, rq.qmax);
    }
    // the pad columns of the code tensor (past the last copy) are zero codes: written by one wave
    // of the last tile column, a lane walking the dwords of its row; the first dword of a row may begin
    // with the last copies, and then takes its bytes one by one
    if (pad_writer) {
        static_assert(64 % ROWS == 0, "whole rows of lanes");
        const int64_t c0 = (int64_t)N + rq.s_next;
        const int r = rbase + lane % ROWS;
        if (r < M) {
            int8_t* row = rq.Yq + (int64_t)r * rq.ldyq;                  // ldyq % 16 == 0: whole dwords
            for (int64_t c = (c0 & ~(int64_t)3) + 4 * (lane / ROWS); c < rq.ldyq; c += 4 * (64 / ROWS)) {
                if (c >= c0) {
                    *reinterpret_cast<int*>(row + c) = 0;
                } else {
                    for (int64_t e = c0; e < c + 4; ++e) row[e] = 0;
                }
            }
        }
    }
}

// One wave's accumulators through its piece of LDS to memory.  As 4-byte stores straight from the
// registers a CU retires ~16 B/clk (measured: the output-bound shapes then run at half the HBM write
// rate); turned through LDS a lane stores 16 bytes that follow its neighbours' along a row.  Only this
// wave touches its piece and a wave's LDS accesses execute in issue order, so no barrier is needed.
//   fp32 (RQ false): products taken with the activations as the first operand; a lane holds one column
//   of a 32 x 32 block and 16 of its rows.  SROWS (8 or 32) rows of the wave's whole width are staged at
//   a time, so that a row's stores follow each other (staged 32 columns at a time 802816 x 256 from 64
//   channels takes 134 us, not 127, and rows of 100 outputs, which share lines, 27, not 17).
//   Codes (RQ): products taken with the weights as the first operand; a lane holds ONE row of a block and
//   four times four consecutive columns, so the stage (32 x 32, rows 36 words apart: different banks)
//   takes a quarter of the writes, and every lane turns 16 of its values into codes.  With 8 staged rows
//   of 64 columns half of the lanes had none: 3x3 64 -> 64 at 100352 pixels 33 -> 22 us with the tile
//   that passes the same 8 MB on.
constexpr int kCodeStride = 36;
template <bool RQ, int WN, int SROWS>
constexpr int stage_bytes() { return RQ ? 32 * kCodeStride * 4 : SROWS * WN * 4; }   // per wave
template <bool RQ, int TM, int TN, int SROWS>
__device__ __forceinline__ void emit_tile(const i32x16 (&acc)[TM][TN], int32_t* stage, int lane, int rbase, int cbase,
                                          int wcol, int M, int N, float scale, float* __restrict__ Y, int64_t ldy,
                                          int32_t* __restrict__ acc_out, int64_t ldacc, const Requant& rq, float inv,
                                          const int* dup_list, int dup_n, bool pad_writer, bool whole) {
    constexpr int WN = 32 * TN;
    const bool vec_y = (reinterpret_cast<uintptr_t>(Y) % 16 == 0) && (ldy % 4 == 0);
    const bool vec_a = acc_out != nullptr && (reinterpret_cast<uintptr_t>(acc_out) % 16 == 0) && (ldacc % 4 == 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if constexpr (RQ) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    i32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e];
                    *reinterpret_cast<i32x4*>(&stage[(lane & 31) * kCodeStride + q * 8 + (lane >> 5) * 4]) = v;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                emit_staged_rows<32, 32, kCodeStride>(stage, lane, rbase + i * 32, cbase + j * 32, wcol + j * 32, M, N,
                                                      scale, Y, ldy, acc_out, ldacc, vec_y, vec_a, rq, inv, dup_list,
                                                      dup_n, pad_writer && j == TN - 1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();   // the reads are issued before the next block's writes
            }
        } else {
            constexpr int Q = 4 * SROWS / 32;      // accumulator quads of a lane per staged block
            // (one address and constant offsets; with the lane's part inside the index the compiler formed eight addresses by
            // OR and half of the writes came singly: 1x1 1024 -> 256 at 25088 rows, both launches, 40.35 us so, 40.30 now,
            // convolutions of 28 x 28 and 16 channels up to 4 %)
            int32_t* at = stage + (lane >> 5) * 4 * WN + (lane & 31);
#pragma unroll
            for (int q0 = 0; q0 < 4; q0 += Q) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < Q; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            at[(q * 8 + e) * WN + j * 32] = acc[i][j][(q0 + q) * 4 + e];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                emit_staged_rows<SROWS, WN>(stage, lane, rbase + i * 32 + q0 * 8, cbase, wcol, M, N, scale, Y, ldy, acc_out,
                                            ldacc, vec_y, vec_a, Requant{}, 0.0f, nullptr, 0, false, whole);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// one product of the tile: the operand that leads decides what a lane of the result holds (see emit_tile)
template <bool RQ>
__device__ __forceinline__ i32x16 mfma_tile(i32x4 x, i32x4 w, i32x16 acc) {
    return RQ ? __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, acc, 0, 0, 0)
              : __builtin_amdgcn_mfma_i32_32x32x32_i8(x, w, acc, 0, 0, 0);
}

__device__ __forceinline__ float requant_inv(const Requant& rq, bool writer) {
    if (rq.Yq == nullptr) return 0.0f;
    const float T = *rq.thr;
    if (writer && rq.scale_out != nullptr) {
        rq.scale_out[0] = T;
        rq.scale_out[1] = T / rq.qmax;
    }
    if (!(T > 0.0f)) return 0.0f;
    return __builtin_fminf(__fdiv_rn(rq.qmax, T), 3.402823466e+38f);
}

// Geometry of a convolution whose lowering to the GEMM is done by the A-operand loader itself
// (CONV variant below): the un-lowered activation codes Aq [B, H, W, ldc] (ldc bytes per pixel,
// a multiple of 16: the expanded channels first, zero padding after), kernel kh x kw, output
// Ho x Wo.  K is walked tap by tap in 16-byte chunks: chunk G of a row is chunk G % cpp of tap
// G / cpp, cpp = ldc / 16 chunks per pixel, so a lane's 16 bytes are 16 consecutive channels of
// one input pixel.  Taps that fall outside the image, and the chunks that pad K up to a whole
// K-step after the last tap, read a row of zeros instead.
struct ConvGeom {
    const int8_t* zero;   // at least BK bytes of zeros
    int H, W, kh, kw, cpp, stride, pad, Ho, Wo;
    int64_t ldc;
};

// K split across workgroups: `parts` workgroups share one output tile, each walks its own slice of
// the K-steps, stores its int32 accumulators in partials[tile][part] (in the register layout, so
// that the stores and the loads are whole 1 KB wave accesses) and signs in at counters[tile]; the
// one that signs in last adds the others' accumulators to its own (integer sums: any order gives
// the same bits) and runs the epilogue.  Nobody waits for anybody.  A counter wraps back to zero
// with the last arrival (atomicInc), so the counters only have to be zero once.
struct SplitK {
    int32_t* partials = nullptr;   // [tiles][parts][BM * BN]
    unsigned* counters = nullptr;  // [tiles], zero between launches
    int parts = 1;
};

// Sixteen zero codes: what a row "holds" past its pitch.  With a short K the rows of the operands
// need not fill their last K-step (a 68-byte row in an 80-byte pitch, walked as 128 bytes): the
// 16-byte pieces that lie past the pitch are fetched from here instead of from the next row.
__device__ __align__(16) int8_t zero_chunk[16] = {};   // (not declared const: it must stay in the global address space, like the rows it stands in for)

// MASK: the pitches may end inside the last K-step (see zero_chunk); every request then checks
// its piece against the pitch.
// BOUNDED: stores with bounds whatever the tile, in an instance of its own (see run_dma).
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int NBUF, bool RQ = false, bool CONV = false,
          bool SPLIT = false, bool MASK = false, bool BOUNDED = false>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64) void qgemm_dma_kernel(
    const int8_t* __restrict__ Xq, int64_t ldx, const int8_t* __restrict__ Wq, int64_t ldw, int M,
    int N, int ksteps_all, const float* __restrict__ scale_x, const float* __restrict__ scale_w,
    int32_t* __restrict__ acc_out, int64_t ldacc, float* __restrict__ Y, int64_t ldy, int tiles_n,
    unsigned total_tiles, ConvGeom cg, Requant rq, SplitK sk) {
    constexpr int NW = WAVES_M * WAVES_N;  // waves (4, 8 or 16)
    constexpr int NT = NW * 64;
    static_assert(NW == 4 || NW == 8 || NW == 16, "4, 8 or 16 waves");
    static_assert(!SPLIT || !CONV, "K split across workgroups: plain GEMM");
    static_assert(!MASK || (!SPLIT && !CONV), "pitch shorter than the K walk: plain GEMM");
    static_assert(BK == 64 || BK == 128, "K-step of 64 or 128 bytes");
    static_assert(NBUF >= 3, "ring of at least three buffers");
    constexpr int CPR = BK / 16;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int A_LOADS = BM * CPR / NT, B_LOADS = BN * CPR / NT;  // per wave & step
    constexpr int LPS = A_LOADS + B_LOADS;
    static_assert(A_LOADS >= 1 && B_LOADS >= 1, "tile too small");
    static_assert((NBUF - 2) * LPS < 64, "prefetch ring exceeds the vmcnt range");
    constexpr int KS = BK / 32;

    // one array: the A ring, then the B ring; the epilogue reuses all of it
    constexpr int RING_BYTES = NBUF * (BM + BN) * BK;
    __shared__ __align__(1024) int8_t lds[RING_BYTES];
    __shared__ int dup_list[RQ ? kDupCap : 1];
    __shared__ int dup_count;
    int8_t (*lds_a)[BM * BK] = reinterpret_cast<int8_t (*)[BM * BK]>(&lds[0]);
    int8_t (*lds_b)[BN * BK] = reinterpret_cast<int8_t (*)[BN * BK]>(&lds[NBUF * BM * BK]);

    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // SPLIT: the parts of a tile are neighbours in the renumbered order, so they run on one XCD
    // and their partial sums meet in its L2
    const unsigned vwg = xcd_remap(blockIdx.x, SPLIT ? total_tiles * (unsigned)sk.parts : total_tiles);
    const unsigned tile = SPLIT ? vwg / (unsigned)sk.parts : vwg;
    const int part = SPLIT ? (int)(vwg % (unsigned)sk.parts) : 0;
    const int kbeg = SPLIT ? (int)((int64_t)part * ksteps_all / sk.parts) : 0;
    const int ksteps = SPLIT ? (int)((int64_t)(part + 1) * ksteps_all / sk.parts) - kbeg : ksteps_all;
    const int bm = (int)(tile / tiles_n), bn = (int)(tile % tiles_n);
    const int row0 = bm * BM, col0 = bn * BN;

    // Load u of this wave fills LDS block (u*4 + wave): slots p = block*64 + lane, row p / CPR,
    // chunk slot p % CPR, which receives global chunk slot ^ f(row).
    const int8_t* a_src[A_LOADS];
    const int8_t* b_src[B_LOADS];
    // CONV: output pixel of each row this lane loads (top-left input coordinate of its window,
    // byte offset of that input pixel, which may lie outside the tensor and is then never used),
    // and the tap position (ky, kx, chunk in pixel) of the chunk this lane will request next for
    // that row: chunk kt*CPR + (its swizzled chunk slot) of the row's K extent.
    int a_iy0[CONV ? A_LOADS : 1], a_ix0[CONV ? A_LOADS : 1];
    int a_ky[CONV ? A_LOADS : 1], a_kx[CONV ? A_LOADS : 1], a_cin[CONV ? A_LOADS : 1];
    int a_zoff[CONV ? A_LOADS : 1];
    int a_piece[MASK ? A_LOADS : 1], b_piece[MASK ? B_LOADS : 1];   // MASK: the lane's piece of K-step 0
    const int a_pieces = (int)(ldx / 16), b_pieces = (int)(ldw / 16);
#pragma unroll
    for (int u = 0; u < A_LOADS; ++u) {
        int pslot = (u * NW + wave) * 64 + lane, r = pslot / CPR, c = pslot % CPR;
        if (MASK) a_piece[u] = swz<BK>(r, c);
        int gr = row0 + r;
        gr = gr < M ? gr : M - 1;  // rows past the edge re-read the last row; never stored
        if (CONV) {
            const int per_img = cg.Ho * cg.Wo;
            const int b = gr / per_img, rem = gr - b * per_img;
            const int yo = rem / cg.Wo, xo = rem - yo * cg.Wo;
            a_iy0[u] = yo * cg.stride - cg.pad;
            a_ix0[u] = xo * cg.stride - cg.pad;
            a_src[u] = Xq + (((int64_t)b * cg.H + a_iy0[u]) * cg.W + a_ix0[u]) * cg.ldc;
            a_zoff[u] = swz<BK>(r, c) * 16;
            int cin = swz<BK>(r, c), kx = 0, ky = 0;
            while (cin >= cg.cpp) {
                cin -= cg.cpp;
                if (++kx == cg.kw) { kx = 0; ++ky; }
            }
            a_cin[u] = cin;
            a_kx[u] = kx;
            a_ky[u] = ky;
        } else {
            a_src[u] = Xq + (int64_t)gr * ldx + swz<BK>(r, c) * 16 + (int64_t)kbeg * BK;
        }
    }
    int c_kt = 0;   // CONV: K-step the next request is for (stops at the last one)
#pragma unroll
    for (int u = 0; u < B_LOADS; ++u) {
        int pslot = (u * NW + wave) * 64 + lane, r = pslot / CPR, c = pslot % CPR;
        int gr = col0 + r;
        gr = gr < N ? gr : N - 1;
        b_src[u] = Wq + (int64_t)gr * ldw + swz<BK>(r, c) * 16 + (int64_t)kbeg * BK;
        if (MASK) b_piece[u] = swz<BK>(r, c);
    }

    // The load is issued through inline assembly on purpose: issued through the compiler's
    // builtin, every later LDS read is preceded by a wait for ALL outstanding loads (the
    // compiler cannot tell which LDS bytes a load fills), which would serialise the ring.
    // The waits are placed by hand instead (wait_vmcnt below); the kernel has no other loads
    // in flight until the epilogue, which starts after a wait for zero.
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds_a0 = (unsigned)(uintptr_t)(lptr_t)&lds_a[0][0];  // LDS byte addresses
    const unsigned lds_b0 = (unsigned)(uintptr_t)(lptr_t)&lds_b[0][0];
#else
    const unsigned lds_a0 = 0, lds_b0 = 0;
#endif
    auto dma16 = [&](const int8_t* g, unsigned lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
        // the block base is the same for every lane of the wave; M0 wants it in a scalar register
        const unsigned m0 = __builtin_amdgcn_readfirstlane(lds_addr);
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                     :
                     : "v"(g), "s"(m0)
                     : "memory");
#else
        (void)g;
        (void)lds_addr;
#endif
    };
    auto fetch = [&](int kt, int buf) {   // K index clamped: surplus steps refetch the last one
        const int kl = kt < ksteps ? kt : ksteps - 1;
        const int64_t koff = (int64_t)kl * BK;
        if (CONV) {
            // requests arrive in K order, so each lane keeps the tap position of its chunk
            // incrementally; it stops at the last step, which surplus requests repeat
            const bool advance = c_kt + 1 < ksteps;
#pragma unroll
            for (int u = 0; u < A_LOADS; ++u) {
                const int iy = a_iy0[u] + a_ky[u], ix = a_ix0[u] + a_kx[u];
                const bool inside = a_ky[u] < cg.kh && (unsigned)iy < (unsigned)cg.H &&
                                    (unsigned)ix < (unsigned)cg.W;
                const int8_t* src =
                    inside ? a_src[u] + ((int64_t)a_ky[u] * cg.W + a_kx[u]) * cg.ldc + a_cin[u] * 16
                           : cg.zero + a_zoff[u];
                dma16(src, lds_a0 + buf * (BM * BK) + (u * NW + wave) * 1024);
                if (advance) {
                    int cin = a_cin[u] + CPR, kx = a_kx[u], ky = a_ky[u];
                    while (cin >= cg.cpp) {
                        cin -= cg.cpp;
                        if (++kx == cg.kw) { kx = 0; ++ky; }
                    }
                    a_cin[u] = cin;
                    a_kx[u] = kx;
                    a_ky[u] = ky;
                }
            }
            if (advance) ++c_kt;
        } else {
#pragma unroll
            for (int u = 0; u < A_LOADS; ++u)
                dma16(!MASK || kl * CPR + a_piece[u] < a_pieces ? a_src[u] + koff : zero_chunk,
                      lds_a0 + buf * (BM * BK) + (u * NW + wave) * 1024);
        }
#pragma unroll
        for (int u = 0; u < B_LOADS; ++u)
            dma16(!MASK || kl * CPR + b_piece[u] < b_pieces ? b_src[u] + koff : zero_chunk,
                  lds_b0 + buf * (BN * BK) + (u * NW + wave) * 1024);
    };

    i32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    const int frag_row = lane & 31, frag_half = lane >> 5;
    i32x4 af[2][TM], bf[2][TN];
    auto read_slice = [&](int buf, int ks, i32x4 (&a)[TM], i32x4 (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int r = wm * WM + i * 32 + frag_row;
            a[i] = *reinterpret_cast<const i32x4*>(
                &lds_a[buf][r * BK + swz<BK>(r, ks * 2 + frag_half) * 16]);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int r = wn * WN + j * 32 + frag_row;
            b[j] = *reinterpret_cast<const i32x4*>(
                &lds_b[buf][r * BK + swz<BK>(r, ks * 2 + frag_half) * 16]);
        }
    };
    auto multiply = [&](i32x4 (&a)[TM], i32x4 (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = mfma_tile<RQ>(a[i], b[j], acc[i][j]);
    };

    // Step kt multiplies out of buffer kt % NBUF.  At its start it requests step kt+NBUF-1 into
    // the buffer step kt-1 used (every wave finished reading it before the previous barrier).
    // Before its last slice it waits until only the loads of steps kt+2.. are outstanding,
    // takes the barrier, and requests slice 0 of step kt+1.
    auto step = [&](int buf, int kt) {
        fetch(kt + NBUF - 1, (buf + NBUF - 1) % NBUF);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) {
                read_slice(buf, ks + 1, af[(ks + 1) & 1], bf[(ks + 1) & 1]);
            } else {
                wait_vmcnt<(NBUF - 2) * LPS>();
                __syncthreads();
                read_slice((buf + 1) % NBUF, 0, af[0], bf[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(af[ks & 1], bf[ks & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int p = 0; p < NBUF - 1; ++p) fetch(p, p);
    if constexpr (RQ) build_dup_list<NT>(rq, N, col0, BN, dup_list, &dup_count);   // behind the first requests
    wait_vmcnt<(NBUF - 2) * LPS>();
    __syncthreads();
    read_slice(0, 0, af[0], bf[0]);

    const int gsteps = ksteps;
    int kt0 = 0;
    for (; kt0 + NBUF <= gsteps; kt0 += NBUF) {
#pragma unroll
        for (int p = 0; p < NBUF; ++p) step(p, kt0 + p);
    }
#pragma unroll
    for (int p = 0; p < NBUF; ++p)
        if (kt0 + p < gsteps) step(p, kt0 + p);
    wait_vmcnt<0>();  // surplus (clamped) loads must land before the ring is reused below
    __syncthreads();  // every wave has read its last fragments: the rings are free

    if constexpr (SPLIT) {
        // The partial sums cross between workgroups that may sit on different XCDs, each with an
        // L2 of its own.  They are stored and loaded as device-coherent accesses (the sc1 bit:
        // written through to, and read from, the memory side of the L2s), which needs no cache
        // maintenance: a device-scope fence instead writes back and invalidates a whole L2 per
        // workgroup (measured: 120 us instead of 42 on the 512-channel 3x3 layer).  Order: stores,
        // wait until they are acknowledged, barrier, one arrival per workgroup.
        __shared__ unsigned arrival;
        constexpr int WAVE_VEC = TM * TN * 4 * 64;   // 16-byte groups of one wave's accumulators
        i32x4* mine = reinterpret_cast<i32x4*>(sk.partials + ((size_t)tile * sk.parts + part) * (size_t)(BM * BN)) +
                      (size_t)wave * WAVE_VEC + lane;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    i32x4 v;
                    v[0] = acc[i][j][4 * vg]; v[1] = acc[i][j][4 * vg + 1];
                    v[2] = acc[i][j][4 * vg + 2]; v[3] = acc[i][j][4 * vg + 3];
                    i32x4* dst = mine + ((i * TN + j) * 4 + vg) * 64;
#if defined(__HIP_DEVICE_COMPILE__)
                    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(dst), "v"(v) : "memory");
#else
                    *dst = v;
#endif
                }
        wait_vmcnt<0>();          // every store of this wave has been acknowledged
        __syncthreads();
        if (threadIdx.x == 0) arrival = atomicInc(sk.counters + tile, (unsigned)sk.parts - 1u);
        __syncthreads();
        if (arrival != (unsigned)sk.parts - 1u) return;   // not the last one: done (no barrier follows)
        for (int q = 0; q < sk.parts; ++q) {
            if (q == part) continue;
            const i32x4* theirs = reinterpret_cast<const i32x4*>(
                                      sk.partials + ((size_t)tile * sk.parts + q) * (size_t)(BM * BN)) +
                                  (size_t)wave * WAVE_VEC + lane;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    i32x4 v0, v1, v2, v3;
                    const i32x4* src = theirs + ((i * TN + j) * 4) * 64;
#if defined(__HIP_DEVICE_COMPILE__)
                    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v0) : "v"(src) : "memory");
                    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v1) : "v"(src + 64) : "memory");
                    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v2) : "v"(src + 128) : "memory");
                    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v3) : "v"(src + 192) : "memory");
                    // the sums below must not be scheduled ahead of the wait: they take their
                    // operands from it
                    asm volatile("s_waitcnt vmcnt(0)" : "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3) : : "memory");
#else
                    v0 = src[0]; v1 = src[64]; v2 = src[128]; v3 = src[192];
#endif
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[i][j][e] += v0[e];
                        acc[i][j][4 + e] += v1[e];
                        acc[i][j][8 + e] += v2[e];
                        acc[i][j][12 + e] += v3[e];
                    }
                }
        }
    }

    // epilogue, through a private piece of the free ring
    constexpr int STAGE = RING_BYTES / NW / 16 * 16;     // (far apart: a wave's piece of the ring)
    static_assert(STAGE >= stage_bytes<RQ, WN, 32>(), "ring too small for the staging areas");
    int32_t* stage = reinterpret_cast<int32_t*>(&lds[wave * STAGE]);
    const float scale = scale_x[1] * scale_w[1];
    const float inv = RQ ? requant_inv(rq, (SPLIT ? tile == 0 : blockIdx.x == 0) && threadIdx.x == 0) : 0.0f;
    const int dup_n = RQ && rq.s_next > 0 ? (dup_count < kDupCap ? dup_count : kDupCap) : 0;
    // Whole tiles without bounds, but for the 128 x 128 tile with 64-byte steps (1024 outputs and more), whose waves then run their
    // stores ahead of each other.  With bounds / without, us: up to 384 bytes of K ahead without (50176 x 1024 x 330 54.0 / 50.7);
    // longer, behind (8192 x 8192 x 538 89.6 / 93.4, 50176 x 1024 x 538 60.3 / 61.9, 16384 x 8192 x 900 251 / 262) until the codes
    // of X are some 56 MB (100000 x 1024 x 538, 58 MB, 117.6 / 118.9, by 2048 229 / 224; x 660 194 / 181; 70000 x 1024 x 900 151 /
    // 142, x 660 95.9 / 97.6).
    constexpr bool HELD = !CONV && !MASK && BM == 128 && BN == 128 && BK == 64;
    const bool whole = !BOUNDED && row0 + BM <= M && col0 + BN <= N && (!HELD || ksteps_all <= 6 || (int64_t)M * ksteps_all >= 900000);
    emit_tile<RQ, TM, TN, 32>(acc, stage, lane, row0 + wm * WM, col0 + wn * WN, wn * WN, M, N, scale, Y, ldy, acc_out, ldacc, rq,
                      inv, dup_list, dup_n, RQ && bn == tiles_n - 1 && wn == 0, whole);
}

// ---------------------------------------------------------------------------------------------
// Short-K variant: the whole K extent of the tile's operands (ksteps steps of 64 bytes) is
// requested into LDS up front, with no ring and no surplus requests, multiplied after ONE wait
// and barrier, and the workgroup keeps no more LDS than that (dynamic size).  For the layers
// with a few hundred input channels the GEMM is a stream of 4*N output bytes per row: what
// matters there is how many workgroups a CU holds, so that one's request latency hides behind
// the others' stores.  Per K-step the LDS holds BM rows of A, then BN rows of B, 64 bytes each,
// chunk-swizzled like the ring kernel's.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void lds_dma16(const int8_t* g, unsigned lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
    const unsigned m0 = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(g), "s"(m0)
                 : "memory");
#else
    (void)g;
    (void)lds_addr;
#endif
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool RQ>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64) void qgemm_wholek_kernel(
    const int8_t* __restrict__ Xq, int64_t ldx, const int8_t* __restrict__ Wq, int64_t ldw, int M,
    int N, int ksteps, const float* __restrict__ scale_x, const float* __restrict__ scale_w,
    int32_t* __restrict__ acc_out, int64_t ldacc, float* __restrict__ Y, int64_t ldy, int tiles_n,
    unsigned total_tiles, int dup_off, Requant rq) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int ROWS = BM + BN;          // LDS rows per K-step
    constexpr int STEP_BYTES = ROWS * 64;
    constexpr int BLOCKS = ROWS / 16;      // 1 KB pieces per K-step, 16 rows each
    static_assert(BM % 16 == 0 && BN % 16 == 0, "a 1 KB piece must not straddle the operands");
    static_assert(WM % 32 == 0 && WN % 32 == 0 && TM >= 1 && TN >= 1, "wave tile of 32x32 blocks");

    // No static LDS here: at 320 bytes of K a 128x128 tile's operands are exactly half of a
    // CU's LDS, and a few bytes more would halve the workgroups a CU holds.  The table of the
    // next layer's copies follows the operands, and only when the epilogue needs it.
    extern __shared__ __align__(1024) int8_t dlds[];
    int* dup_list = reinterpret_cast<int*>(&dlds[dup_off]);   // used only when dup_off > 0
    int* dup_count = dup_list + kDupCap;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&dlds[0];
#else
    const unsigned lds0 = 0;
#endif

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const unsigned tile = xcd_remap(blockIdx.x, total_tiles);
    const int bm = (int)(tile / tiles_n), bn = (int)(tile % tiles_n);
    const int row0 = bm * BM, col0 = bn * BN;

    // piece b of a K-step: LDS rows 16b .. 16b+15; lane l fills row 16b + l/4, chunk slot l%4
    // (a row's pitch may end inside the last K-step: pieces past it come from zero_chunk)
    for (int b = wave; b < BLOCKS; b += NW) {
        const int r = b * 16 + (lane >> 2), c = lane & 3;
        const int8_t* rowp;
        int piece, pieces;                 // this lane's 16-byte piece of K-step 0; pieces in the pitch
        if (r < BM) {
            int gr = row0 + r;
            gr = gr < M ? gr : M - 1;      // rows past the edge re-read the last row; never stored
            rowp = Xq + (int64_t)gr * ldx;
            piece = swz<64>(r, c);
            pieces = (int)(ldx / 16);
        } else {
            int gr = col0 + (r - BM);
            gr = gr < N ? gr : N - 1;
            rowp = Wq + (int64_t)gr * ldw;
            piece = swz<64>(r - BM, c);
            pieces = (int)(ldw / 16);
        }
        for (int kt = 0; kt < ksteps; ++kt, piece += 4)
            lds_dma16(piece < pieces ? rowp + piece * 16 : zero_chunk, lds0 + kt * STEP_BYTES + b * 1024);
    }

    i32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    if (RQ && dup_off > 0) build_dup_list<NW * 64>(rq, N, col0, BN, dup_list, dup_count);   // behind the requests
    wait_vmcnt<0>();
    __syncthreads();

    const int frag_row = lane & 31, frag_half = lane >> 5;
    for (int kt = 0; kt < ksteps; ++kt) {
        const int8_t* base = &dlds[kt * STEP_BYTES];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            i32x4 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = wm * WM + i * 32 + frag_row;
                a[i] = *reinterpret_cast<const i32x4*>(
                    &base[r * 64 + swz<64>(r, ks * 2 + frag_half) * 16]);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = wn * WN + j * 32 + frag_row;
                b[j] = *reinterpret_cast<const i32x4*>(
                    &base[(BM + r) * 64 + swz<64>(r, ks * 2 + frag_half) * 16]);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = mfma_tile<RQ>(a[i], b[j], acc[i][j]);
        }
    }
    __syncthreads();  // the operands are dead: their LDS becomes the staging area

    // epilogue as in the ring kernel
    int32_t* stage = reinterpret_cast<int32_t*>(&dlds[wave * stage_bytes<RQ, WN, 8>()]);
    const float scale = scale_x[1] * scale_w[1];
    const float inv = RQ ? requant_inv(rq, blockIdx.x == 0 && tid == 0) : 0.0f;
    const int dup_n = RQ && dup_off > 0 ? (*dup_count < kDupCap ? *dup_count : kDupCap) : 0;
    emit_tile<RQ, TM, TN, 8>(acc, stage, lane, row0 + wm * WM, col0 + wn * WN, wn * WN, M, N, scale, Y, ldy, acc_out, ldacc, rq,
                      inv, dup_list, dup_n, RQ && bn == tiles_n - 1 && wn == 0, row0 + BM <= M && col0 + BN <= N);
}

// ---------------------------------------------------------------------------------------------
// Few tiles: the K extent dealt over the waves of a workgroup.  A layer of a few rows (one time step
// of a recurrent layer, a small batch) has too few tiles for the chip, and a tile's walk along K with
// a barrier per step is then one long chain on a handful of compute units.  Here every wave computes
// the WHOLE tile over its own 64-byte steps of K (step `wave`, `wave` + NW, ...; neighbouring waves
// share a row's lines): its operands go global -> LDS into a ring of its own (NBUF steps, the layout
// and swizzle of the whole-K kernel), which only this wave fills and reads, so the loop has no
// barrier and the waves drift as their requests come back.  The NW partial tiles then meet in LDS:
// one barrier, every wave sums its rows over the NW copies (integer sums: any order gives the same
// bits) and stores them.
// What bounds it: the latency of a wave's few requests, the sum over the partial tiles and the launch
// itself.  Operands straight into registers instead (no LDS on the way) was slower from a few hundred
// bytes of K on: a lane's 16 bytes of its own row cost the L1 a look-up per lane, where the LDS form
// asks for four lanes' worth of a row at once (64 x 256 x 2420: 7.0 against 4.1 us).
// ---------------------------------------------------------------------------------------------
template <int TM, int TN, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void qgemm_slice_kernel(
    const int8_t* __restrict__ Xq, int64_t ldx, const int8_t* __restrict__ Wq, int64_t ldw, int M,
    int N, int ksteps, const float* __restrict__ scale_x, const float* __restrict__ scale_w,
    int32_t* __restrict__ acc_out, int64_t ldacc, float* __restrict__ Y, int64_t ldy, int tiles_m, int tiles_n,
    int rows_first, Requant rq) {
    constexpr int BM = 32 * TM, BN = 32 * TN;
    constexpr int LPS = (BM + BN) / 16;                           // 1 KB requests of a step: 16 rows each
    constexpr int STEP = (BM + BN) * 64;
    constexpr int RING = NBUF * STEP;                             // LDS of a wave: its ring, then its partial tile
    constexpr int EW = BM * BN / 256 < NW ? BM * BN / 256 : NW;   // waves that store: at least 64 x 4 outputs each
    constexpr int ROWS = BM / EW;
    static_assert(EW * ROWS == BM && ROWS * BN % 256 == 0, "whole waves of 16-byte outputs");
    static_assert(RING >= BM * BN * 4, "a wave's partial tile replaces its ring");
    static_assert((NBUF - 1) * LPS < 64, "prefetch ring exceeds the vmcnt range");
    static_assert(NBUF >= 2 && NBUF <= 4, "waits below");
    static_assert(BN <= 256, "a dup_list entry holds the column in 8 bits");
    extern __shared__ __align__(1024) int8_t slds[];
    int* dup_list = reinterpret_cast<int*>(slds + NW * RING);     // only with copies to write
    int* dup_count = dup_list + kDupCap;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&slds[0];
#else
    const unsigned lds0 = 0;
#endif

    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // uniform: the step counts below are scalar
    const unsigned tile = xcd_remap(blockIdx.x, (unsigned)tiles_m * (unsigned)tiles_n);
    // tiles that share the larger operand's panel follow each other on one XCD
    const int bm = rows_first ? (int)(tile % (unsigned)tiles_m) : (int)(tile / (unsigned)tiles_n);
    const int bn = rows_first ? (int)(tile / (unsigned)tiles_m) : (int)(tile % (unsigned)tiles_n);
    const int row0 = bm * BM, col0 = bn * BN;

    // request q of a step: lane l fills row 16q + l/4, chunk slot l%4 of the step's image (A rows, then
    // B rows); the swizzle depends on the row's low four bits only, so a lane's piece is the same in all
    const int piece = swz<64>(lane >> 2, lane & 3);
    const int8_t* src[LPS];
#pragma unroll
    for (int q = 0; q < LPS; ++q) {
        const int r = q * 16 + (lane >> 2);
        src[q] = q * 16 < BM ? Xq + (int64_t)col_clamp(row0 + r, M) * ldx          // (rows past the edge are never stored)
                             : Wq + (int64_t)col_clamp(col0 + r - BM, N) * ldw;
    }
    // a row's pitch may end inside the last K-step: pieces past it come from zero_chunk
    const int a_end = (int)(ldx / 16), b_end = (int)(ldw / 16);
    const unsigned ring0 = lds0 + (unsigned)wave * RING;
    const int8_t* ring = slds + wave * RING;
    const int trips = (ksteps - wave + NW - 1) / NW;              // this wave's steps (none: its tile is zero)
    auto fetch = [&](int it, int buf) {
        const int p = (it * NW + wave) * 4 + piece;
#pragma unroll
        for (int q = 0; q < LPS; ++q)
            lds_dma16(p < (q * 16 < BM ? a_end : b_end) ? src[q] + (int64_t)p * 16 : zero_chunk,
                      ring0 + (unsigned)(buf * STEP + q * 1024));
    };

    i32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

#pragma unroll
    for (int u = 0; u + 1 < NBUF; ++u)
        if (u < trips) fetch(u, u);
    if (rq.Yq != nullptr && rq.s_next > 0) build_dup_list<NW * 64>(rq, N, col0, BN, dup_list, dup_count);

    const int frag_row = lane & 31, frag_half = lane >> 5;
    for (int it0 = 0; it0 < trips; it0 += NBUF) {
#pragma unroll
        for (int u = 0; u < NBUF; ++u) {
            const int it = it0 + u;
            if (it >= trips) break;
            const int left = trips - 1 - it;                      // this wave's steps after this one
            if (left >= NBUF - 1) {
                // the buffer requested into was read by the step before: its reads have returned
                __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
                fetch(it + NBUF - 1, (u + NBUF - 1) % NBUF);
                wait_vmcnt<(NBUF - 1) * LPS>();
            } else if (NBUF > 3 && left == 2) {
                wait_vmcnt<(NBUF > 3 ? 2 : 0) * LPS>();
            } else if (NBUF > 2 && left == 1) {
                wait_vmcnt<(NBUF > 2 ? 1 : 0) * LPS>();
            } else {
                wait_vmcnt<0>();
            }
            asm volatile("" ::: "memory");                        // no read of the step above its wait
            const int8_t* base = ring + u * STEP;
            i32x4 a[2][TM], b[2][TN];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int r = i * 32 + frag_row;
                    a[ks][i] = *reinterpret_cast<const i32x4*>(&base[r * 64 + swz<64>(r, ks * 2 + frag_half) * 16]);
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int r = j * 32 + frag_row;
                    b[ks][j] = *reinterpret_cast<const i32x4*>(&base[(BM + r) * 64 + swz<64>(r, ks * 2 + frag_half) * 16]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);                    // all reads on their way before the first product
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
        }
    }
    // every request of this wave has landed and every read has returned (the last step waited for
    // both): the ring takes the partial tile
    constexpr int PSTRIDE = RING / 4;
    int32_t* part = reinterpret_cast<int32_t*>(slds);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                part[wave * PSTRIDE + (i * 32 + (v >> 2) * 8 + frag_half * 4 + (v & 3)) * BN + j * 32 + frag_row] = acc[i][j][v];
    __syncthreads();
    if (wave >= EW) return;                       // no barrier follows

    int32_t* stage = part + wave * (ROWS * BN);   // this wave's rows of copy 0: the sum goes there
#pragma unroll
    for (int o = 0; o < ROWS * BN / 256; ++o) {
        i32x4 sum = *reinterpret_cast<const i32x4*>(&stage[(o * 64 + lane) * 4]);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const i32x4 v = *reinterpret_cast<const i32x4*>(&stage[w * PSTRIDE + (o * 64 + lane) * 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += v[e];
        }
        *reinterpret_cast<i32x4*>(&stage[(o * 64 + lane) * 4]) = sum;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const float scale = scale_x[1] * scale_w[1];
    const float inv = requant_inv(rq, blockIdx.x == 0 && tid == 0);
    const int dup_n = (rq.Yq != nullptr && rq.s_next > 0) ? (*dup_count < kDupCap ? *dup_count : kDupCap) : 0;
    const bool vec_y = (reinterpret_cast<uintptr_t>(Y) % 16 == 0) && (ldy % 4 == 0);
    const bool vec_a = acc_out != nullptr && (reinterpret_cast<uintptr_t>(acc_out) % 16 == 0) && (ldacc % 4 == 0);
    emit_staged_rows<ROWS, BN>(stage, lane, row0 + wave * ROWS, col0, 0, M, N, scale, Y, ldy, acc_out, ldacc, vec_y,
                               vec_a, rq, inv, dup_list, dup_n, rq.Yq != nullptr && bn == tiles_n - 1);
}

// ---------------------------------------------------------------------------------------------
// A whole layer of few tiles as one launch: the sliced kernel above with X2 in its loader.  A wave's
// step of the activations is 64 floats of the tile's rows, requested as 16 bytes per lane (16 lanes
// share a row's 256 bytes) into registers, NBUF - 1 steps ahead like the weight codes' ring; it is
// put on the grid with X2's arithmetic (code_bits, pack4), written as dwords into a piece of LDS that
// only this wave uses, in the layout the matrix cores read, and multiplied.  Appended columns, the
// columns that do not fill a last step and the padding come through a table of their source columns,
// built in LDS behind the first requests: such a step gathers its floats one by one (5 % of K at the
// paper's ratios).  The codes also go to memory as ocs_split_act leaves them, every K-step written by
// one of the workgroups that share the rows.  A per-batch grid's threshold is folded from the max|X|
// pass's maxima, or, for small contiguous X, looked for by every workgroup, behind the same requests.
// Tiles are 32 rows high: the workgroups of a row of tiles each repeat the quantization of its rows, so
// width is what saves work.
// What bounds it: the smallest by latency (requests, the gather behind the table, the sum over the
// waves), the longest by the floats every workgroup draws again (rows x K x 4 bytes a compute unit).
// Passes one after the other, two launches / one, us: 64 x 256 -> 256 per batch 9.2 / 6.4, 1 x 3000 -> 6000 8.9 / 6.3, 700 x
// 256 -> 256 8.9 / 6.3, 1000 x 147 -> 64 per batch 11.3 / 8.6; the kernels alone, in a graph, 6.4 / 5.3, 7.1 / 5.6, 5.9 / 4.9,
// 7.9 / 7.2.  Accumulators, codes, scales and outputs are bit for bit those of the two calls.
// ---------------------------------------------------------------------------------------------
struct SliceLayer {
    const float* X;
    int64_t ldx;
    int M, N, K, C, g, Kexp;
    const int32_t* chan_src;
    const float* thr;          // n_max == 0 and self == 0: the threshold; else the n_max maxima
    int n_max;
    int64_t self;              // values of contiguous X to look through (0: none)
    float clip, qmax;
    int8_t* Xq;
    int64_t ldq;
    float* scale_x;
    const int8_t* Wq;
    int64_t ldw;
    const float* scale_w;
    int32_t* acc_out;
    int64_t ldacc;
    float* Y;
    int64_t ldy;
    int ksteps, kmain;         // K-steps of 64 columns; those that lie inside X's rows
    int tiles_m, tiles_n, rows_first;
};
// LDS of a wave: slots of weight codes and the step's activation codes, then its partial tile
template <int TN, int SLOTS>
constexpr int slice_layer_wave_bytes() {
    const int operands = SLOTS * 32 * TN * 64 + 32 * 64, partial = 32 * 32 * TN * 4;
    return operands > partial ? operands : partial;
}
// A_PER: requests of a step of X, four rows each (the rows above 4 A_PER of a tile are not there).  NBUF: steps in the ring.
// EARLY: the first step of appended columns has a slot of its own and is requested ahead of the others.
template <int TN, int A_PER, int NW, int NBUF, bool EARLY>
__global__ __launch_bounds__(NW * 64) void slice_layer_kernel(SliceLayer p) {
    constexpr int BM = 32, BN = 32 * TN;
    constexpr int LPS = BN / 16;                                  // requests of a step of W: 16 rows each
    constexpr int RING = slice_layer_wave_bytes<TN, NBUF + (EARLY ? 1 : 0)>();
    constexpr int EW = BM * BN / 256 < NW ? BM * BN / 256 : NW;   // waves that store (see the sliced kernel)
    constexpr int ROWS = BM / EW;
    static_assert(EW * ROWS == BM && ROWS * BN % 256 == 0, "whole waves of 16-byte outputs");
    static_assert((NBUF - 1) * (LPS + A_PER) < 64, "look-ahead exceeds the vmcnt range");
    static_assert(A_PER >= 1 && A_PER <= 8 && (NBUF == 2 || NBUF == 3), "rows of the tile, ring");
    extern __shared__ __align__(1024) int8_t slds[];
    int* tail_col = reinterpret_cast<int*>(slds + NW * RING);     // source column of every column past the whole steps (-1: zero code)
    const int tail_cols = (p.ksteps - p.kmain) * 64;
    float* red = reinterpret_cast<float*>(tail_col + tail_cols);  // NW floats
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&slds[0];
#else
    const unsigned lds0 = 0;
#endif
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned tile = xcd_remap(blockIdx.x, (unsigned)p.tiles_m * (unsigned)p.tiles_n);
    const int bm = p.rows_first ? (int)(tile % (unsigned)p.tiles_m) : (int)(tile / (unsigned)p.tiles_n);
    const int bn = p.rows_first ? (int)(tile / (unsigned)p.tiles_m) : (int)(tile % (unsigned)p.tiles_n);
    const int row0 = bm * BM, col0 = bn * BN;

    // weight codes: as in the sliced kernel (rows past the edge are never stored; pieces past the pitch are zeros)
    const int piece = swz<64>(lane >> 2, lane & 3);
    const int8_t* wsrc[LPS];
#pragma unroll
    for (int q = 0; q < LPS; ++q) wsrc[q] = p.Wq + (int64_t)col_clamp(col0 + q * 16 + (lane >> 2), p.N) * p.ldw;
    const int w_end = (int)(p.ldw / 16);
    int8_t* ring = slds + wave * RING;
    int8_t* codes = ring + (RING - BM * 64) / 16 * 16;            // behind the slots
    const unsigned ring0 = lds0 + (unsigned)wave * RING;
    // activations: request u of a step is row 4u + lane / 16, columns 4 (lane % 16) .. + 3.  Offsets from the tile's first
    // row in floats: below 2^29 (the caller's limit on ldx)
    const float* xb = p.X + (int64_t)row0 * p.ldx;
    const int c4 = (lane & 15) * 4;
    unsigned xrow[A_PER];
#pragma unroll
    for (int u = 0; u < A_PER; ++u) xrow[u] = (unsigned)(col_clamp(row0 + u * 4 + (lane >> 4), p.M) - row0) * (unsigned)p.ldx;
    // this wave's steps: those inside X's rows, kt = wave, wave + NW, ... below kmain, then the others
    const int trips = p.kmain > wave ? (p.kmain - wave + NW - 1) / NW : 0;
    const int tail0 = trips * NW + wave;

    auto fetch_w = [&](int kt, int slot) {
        const int q0 = kt * 4 + piece;
#pragma unroll
        for (int q = 0; q < LPS; ++q)
            lds_dma16(q0 < w_end ? wsrc[q] + (int64_t)q0 * 16 : zero_chunk, ring0 + (unsigned)(slot * BN * 64 + q * 1024));
    };
    // (surplus requests repeat the wave's last step: no condition around a load, or the compiler waits for those under way.
    // The weight codes first: requests return in order, so whoever has a step's activations has its weight codes.)
    auto fetch = [&](int it, int slot, f32x4 (&a)[A_PER]) {
        const int kt = (it < trips ? it : trips - 1) * NW + wave;
        fetch_w(kt, slot);
#pragma unroll
        for (int u = 0; u < A_PER; ++u) a[u] = *reinterpret_cast<const f32x4u*>(xb + (xrow[u] + (unsigned)(kt * 64 + c4)));
    };

    f32x4 av[NBUF][A_PER];
    if (trips > 0) {
#pragma unroll
        for (int u = 0; u + 1 < NBUF; ++u) fetch(u, u, av[u]);
    }
    if (EARLY && tail0 < p.ksteps) fetch_w(tail0, NBUF);
    // the table, and the threshold, behind the first requests
    for (int e = tid; e < tail_cols; e += NW * 64) {
        const int k = p.kmain * 64 + e;
        int col = -1;
        if (k < p.K) col = k;
        else if (k < p.Kexp) {
            const int j = k / p.g;
            col = col_clamp(p.chan_src[j], p.C) * p.g + (k - j * p.g);
        }
        tail_col[e] = col;
    }
    float T;
    if (p.n_max == 0 && p.self == 0) {
        T = *p.thr;
    } else {
        float m = 0.0f;
        for (int i = tid; i < p.n_max; i += NW * 64) m = fmaxf(m, p.thr[i]);
        const int n4 = (int)(p.self / 4);
        constexpr int UN = 8;
        for (int i0 = tid; i0 < n4; i0 += UN * NW * 64) {
            f32x4 v[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int i = i0 + u * NW * 64;
                v[u] = reinterpret_cast<const f32x4u*>(p.X)[i < n4 ? i : n4 - 1];
            }
#pragma unroll
            for (int u = 0; u < UN; ++u)
                m = fmaxf(fmaxf(fmaxf(m, fabsf(v[u][0])), fmaxf(fabsf(v[u][1]), fabsf(v[u][2]))), fabsf(v[u][3]));
        }
        if ((int64_t)tid < p.self - 4 * (int64_t)n4) m = fmaxf(m, fabsf(p.X[4 * n4 + tid]));
        const unsigned w = wave_umax32(__float_as_uint(m));
        if (lane == 0) red[wave] = __uint_as_float(w);
        T = 0.0f;
    }
    __syncthreads();
    if (p.n_max != 0 || p.self != 0) {
        float m = red[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, red[w]);
        T = p.clip * m;
    }
    const float inv = inv_step_of(T, p.qmax);
    if (blockIdx.x == 0 && tid == 0) {
        p.scale_x[0] = T;
        p.scale_x[1] = T / p.qmax;
    }

    i32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0;

    const int frag_row = lane & 31, frag_half = lane >> 5;
    int8_t* qrow = p.Xq + (int64_t)row0 * p.ldq;
    // A step's floats onto the grid, into LDS and, by one of the workgroups that share the rows, to memory.
    // keep: the bytes that are codes (the others are zero)
    auto quantize = [&](int kt, const f32x4 (&a)[A_PER], unsigned keep) {
        unsigned q4[A_PER];
#pragma unroll
        for (int q = 0; q < A_PER; ++q) {
            q4[q] = keep & pack4(code_bits(a[q][0], inv, p.qmax), code_bits(a[q][1], inv, p.qmax),
                                 code_bits(a[q][2], inv, p.qmax), code_bits(a[q][3], inv, p.qmax));
            const int r = q * 4 + (lane >> 4);
            *reinterpret_cast<unsigned*>(codes + r * 64 + swz<64>(r, (lane & 15) >> 2) * 16 + (lane & 3) * 4) = q4[q];
        }
        if (kt % p.tiles_n == bn && kt * 64 + c4 < p.ldq) {
#pragma unroll
            for (int q = 0; q < A_PER; ++q) {
                const int r = q * 4 + (lane >> 4);
                if (row0 + r < p.M) *reinterpret_cast<unsigned*>(qrow + (int64_t)r * p.ldq + kt * 64 + c4) = q4[q];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto multiply = [&](int slot) {
        const int8_t* base = ring + slot * (BN * 64);
        i32x4 a[2], b[2][TN];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a[ks] = *reinterpret_cast<const i32x4*>(&codes[frag_row * 64 + swz<64>(frag_row, ks * 2 + frag_half) * 16]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = j * 32 + frag_row;
                b[ks][j] = *reinterpret_cast<const i32x4*>(&base[r * 64 + swz<64>(r, ks * 2 + frag_half) * 16]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();                          // the reads are issued before the next step's writes
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[ks][j], acc[j], 0, 0, 0);
    };
    auto gather = [&](int kt, f32x4 (&a)[A_PER], unsigned& keep) {
        const i32x4 cols = *reinterpret_cast<const i32x4*>(&tail_col[(kt - p.kmain) * 64 + c4]);
        keep = 0xFFFFFFFFu;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (cols[e] < 0) keep &= ~(0xFFu << (8 * e));
#pragma unroll
        for (int u = 0; u < A_PER; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[u][e] = xb[xrow[u] + (unsigned)(cols[e] < 0 ? 0 : cols[e])];
    };

    f32x4 at[A_PER];
    unsigned keep = 0;
    if (EARLY && tail0 < p.ksteps) gather(tail0, at, keep);
    auto step = [&](int it, auto slot) {
        constexpr int u = decltype(slot)::value, next = (u + NBUF - 1) % NBUF;
        // the slot requested into was read by the step before: its reads have returned
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);                        // (no arithmetic on the step's floats ahead of the requests)
        fetch(it + NBUF - 1, next, av[next]);
        wait_vmcnt<(NBUF - 1) * (LPS + A_PER)>();                 // this step's requests are back
        asm volatile("" ::: "memory");                            // no read of the step above its wait
        __builtin_amdgcn_sched_barrier(0);
        quantize(it * NW + wave, av[u], 0xFFFFFFFFu);
        multiply(u);
    };
    // (whole rounds of the ring without a way out, or the compiler's own waits assume the shortest way through)
    int it0 = 0;
    for (; it0 + NBUF <= trips; it0 += NBUF) {
        step(it0, std::integral_constant<int, 0>{});
        step(it0 + 1, std::integral_constant<int, 1>{});
        if constexpr (NBUF > 2) step(it0 + 2, std::integral_constant<int, NBUF - 1>{});
    }
    if (it0 < trips) {
        step(it0, std::integral_constant<int, 0>{});
        if constexpr (NBUF > 2)
            if (it0 + 1 < trips) step(it0 + 1, std::integral_constant<int, 1>{});
    }
    for (int kt = tail0; kt < p.ksteps; kt += NW) {
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));       // lgkmcnt(0): the slot's last reads have returned
        asm volatile("" ::: "memory");
        const bool early = EARLY && kt == tail0;
        if (!early) {
            wait_vmcnt<0>();                                      // (surplus requests into the slot)
            fetch_w(kt, NBUF - 1);
            gather(kt, at, keep);
        }
        wait_vmcnt<0>();
        asm volatile("" ::: "memory");
        quantize(kt, at, keep);
        multiply(early ? NBUF : NBUF - 1);
    }
    wait_vmcnt<0>();                              // surplus requests have landed: the slots take the partial tile
    // the padding of the code rows past the last K-step
    if (bn == 0) {
        const int c0 = p.ksteps * 64, n4 = p.ldq > c0 ? (int)((p.ldq - c0) / 4) : 0;
        const int rows = p.M - row0 < BM ? p.M - row0 : BM;
        for (int i = tid; i < rows * n4; i += NW * 64) {
            const int r = i / n4;
            *reinterpret_cast<unsigned*>(qrow + (int64_t)r * p.ldq + c0 + 4 * (i - r * n4)) = 0u;
        }
    }
    // every wave puts its partial tile over its own operands, whose reads have returned
    constexpr int PSTRIDE = RING / 4;
    int32_t* part = reinterpret_cast<int32_t*>(slds);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            part[wave * PSTRIDE + ((v >> 2) * 8 + frag_half * 4 + (v & 3)) * BN + j * 32 + frag_row] = acc[j][v];
    __syncthreads();
    if (wave >= EW) return;                       // no barrier follows

    int32_t* stage = part + wave * (ROWS * BN);   // this wave's rows of copy 0: the sum goes there
#pragma unroll
    for (int o = 0; o < ROWS * BN / 256; ++o) {
        i32x4 sum = *reinterpret_cast<const i32x4*>(&stage[(o * 64 + lane) * 4]);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const i32x4 v = *reinterpret_cast<const i32x4*>(&stage[w * PSTRIDE + (o * 64 + lane) * 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += v[e];
        }
        *reinterpret_cast<i32x4*>(&stage[(o * 64 + lane) * 4]) = sum;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const float scale = (T / p.qmax) * p.scale_w[1];
    const bool vec_y = (reinterpret_cast<uintptr_t>(p.Y) % 16 == 0) && (p.ldy % 4 == 0);
    const bool vec_a = p.acc_out != nullptr && (reinterpret_cast<uintptr_t>(p.acc_out) % 16 == 0) && (p.ldacc % 4 == 0);
    emit_staged_rows<ROWS, BN>(stage, lane, row0 + wave * ROWS, col0, 0, p.M, p.N, scale, p.Y, p.ldy, p.acc_out, p.ldacc,
                               vec_y, vec_a, Requant{}, 0.0f, nullptr, 0, false);
}

// ---------------------------------------------------------------------------------------------
// Convolution of unit stride whose output has the input's size (kh = 2 pad + 1 = kw, the body of the
// paper's networks): the lowering as address arithmetic in LDS.  The BM output pixels of a tile are
// consecutive in the flattened image, so the input pixels that all taps together need are one
// contiguous run of BM + 2 pad (W + 1) pixels.  The workgroup fetches that run once (the ring kernel
// above fetches every pixel once per tap, 9 times for a 3x3) and keeps it; a tap of an output row is
// then the run's pixel (row + ky W + kx), read straight into the matrix cores' operand.  Taps outside
// the image read 16 zero bytes instead: one bit per tap and row, worked out once.  K runs tap by tap in
// 16-byte pieces as in the tap-major weights, which pass through a ring of 128-byte K-steps (one
// barrier each); a pixel takes an odd number of pieces in LDS, so that consecutive pixels start in
// different banks.
// What bounds it (32 x 56 x 56 x 64 -> 64 with codes out, 16.8 us): 33 vector instructions per matrix instruction, the
// addresses of the taps and the epilogue, fill 61 % of the busy compute units' cycles, the matrix cores 15 %, waits
// 23 % of the waves'; several workgroups per compute unit hide one another's fill and epilogue.
// ---------------------------------------------------------------------------------------------
constexpr int kPatchMaxTaps = 25;

template <int BM, int BN, int WAVES_M, int WAVES_N, int NBUF, bool RQ>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64) void qconv_patch_kernel(
    const int8_t* __restrict__ Aq, const int8_t* __restrict__ Wt, int64_t ldw, int M, int N, int ksteps,
    int H, int W, int kw, int pad, int cpp, int P16, unsigned magic_p16, int pixels,
    const float* __restrict__ scale_x, const float* __restrict__ scale_w, int32_t* __restrict__ acc_out,
    int64_t ldacc, float* __restrict__ Y, int64_t ldy, int tiles_n, unsigned total_tiles, int ring_off,
    int dup_off, Requant rq) {
    // cpp: 16-byte pieces of a pixel in memory; P16 >= cpp: in LDS; pixels: length of the run
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int BK = 128, KS = BK / 32;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
    constexpr int B_LOADS = BN * (BK / 16) / (NW * 64);
    static_assert(B_LOADS >= 1 && B_LOADS * NW * 64 == BN * (BK / 16), "the waves tile a step of the weights");
    static_assert(NBUF >= 3 && (NBUF - 2) * B_LOADS < 64, "ring of at least three buffers");
    static_assert(TM >= 1 && TN >= 1 && TM * 32 * WAVES_M == BM && TN * 32 * WAVES_N == BN, "32 x 32 blocks");
    extern __shared__ __align__(1024) int8_t plds[];
    int* dup_list = reinterpret_cast<int*>(plds + dup_off);       // only with copies to write
    int* dup_count = dup_list + kDupCap;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&plds[0];
#else
    const unsigned lds0 = 0;
#endif
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const unsigned tile = xcd_remap(blockIdx.x, total_tiles);
    const int bm = (int)(tile / (unsigned)tiles_n), bn = (int)(tile % (unsigned)tiles_n);
    const int row0 = bm * BM, col0 = bn * BN;
    const int kh = kw, taps = kh * kw;

    // weights first (the multiply waits for both): request u of a step as in the ring kernel
    const int8_t* b_src[B_LOADS];
    int b_piece[B_LOADS];
    const int b_pieces = (int)(ldw / 16);
#pragma unroll
    for (int u = 0; u < B_LOADS; ++u) {
        const int pslot = (u * NW + wave) * 64 + lane, r = pslot / (BK / 16), c = pslot % (BK / 16);
        b_src[u] = Wt + (int64_t)col_clamp(col0 + r, N) * ldw;    // (rows past the edge are never stored)
        b_piece[u] = swz<BK>(r, c);
    }
    auto fetch = [&](int kt, int buf) {     // surplus steps (past the last) come from zero_chunk
        const unsigned base = lds0 + (unsigned)(ring_off + buf * (BN * BK));
#pragma unroll
        for (int u = 0; u < B_LOADS; ++u) {
            const int piece = kt * (BK / 16) + b_piece[u];
            lds_dma16(piece < b_pieces ? b_src[u] + (int64_t)piece * 16 : zero_chunk, base + (unsigned)(u * NW + wave) * 1024);
        }
    };
#pragma unroll
    for (int p = 0; p < NBUF - 1; ++p) fetch(p, p);
    // the run of input pixels: piece i of the image in LDS = piece i % P16 of pixel i / P16 of the run
    // (pixels before the first or past the last one of the tensor are clamped: no valid tap reads them)
    const int lo = row0 - pad * W - pad;
    const int pieces = pixels * P16;
    for (int b = wave; b * 64 < pieces; b += NW) {
        const unsigned i = (unsigned)(b * 64 + lane);
        unsigned q = __umulhi(i, magic_p16);                      // floor(i / P16), at most one low
        unsigned c = i - q * (unsigned)P16;
        if (c >= (unsigned)P16) { ++q; c -= (unsigned)P16; }
        const bool ok = (int)q < pixels && (int)c < cpp;
        lds_dma16(ok ? Aq + ((int64_t)col_clamp(lo + (int)q, M) * cpp + c) * 16 : zero_chunk, lds0 + (unsigned)b * 1024);
    }
    const int zero_off = ring_off - 16;                           // 16 zero bytes behind the run
    if (tid < 4) *reinterpret_cast<int*>(plds + zero_off + 4 * tid) = 0;

    // per row of this lane: one bit per tap that lies inside the image
    const int frag_row = lane & 31, frag_half = lane >> 5;
    unsigned ok_taps[TM];
    int row_off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = wm * WM + i * 32 + frag_row;
        const int gr = col_clamp(row0 + r, M);
        const int yx = gr % (H * W), y = yx / W, x = yx - y * W;
        unsigned m = 0;
        for (int t = 0, ky = 0, kx = 0; t < taps; ++t) {
            if ((unsigned)(y + ky - pad) < (unsigned)H && (unsigned)(x + kx - pad) < (unsigned)W) m |= 1u << t;
            if (++kx == kw) { kx = 0; ++ky; }
        }
        ok_taps[i] = m;
        row_off[i] = r * P16 * 16;
    }
    if (RQ && dup_off > 0) build_dup_list<NW * 64>(rq, N, col0, BN, dup_list, dup_count);   // behind the requests

    i32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    // This lane's piece of the K extent: piece `frag_half` of the first slice, two further on with every
    // slice; `off` = its place relative to the row's first pixel of the run.
    int tap = 0, kx = 0, cin = frag_half, off = frag_half * 16;
    const int next_pixel = (P16 - cpp) * 16, next_row = (W - kw) * P16 * 16;
    auto advance = [&]() {
        cin += 2;
        off += 32;
        if (cin >= cpp) {                                         // (cpp >= 2: at most one tap further)
            cin -= cpp;
            off += next_pixel;
            ++tap;
            if (++kx == kw) { kx = 0; off += next_row; }
        }
    };
    i32x4 af[2][TM], bf[2][TN];
    auto read_slice = [&](int buf, int ks, i32x4 (&a)[TM], i32x4 (&b)[TN]) {
        // (taps past the last one, where K is padded to whole steps: no bit set)
        const bool in = tap < taps;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const bool ok = in && ((ok_taps[i] >> (tap & 31)) & 1u);
            a[i] = *reinterpret_cast<const i32x4*>(plds + (ok ? row_off[i] + off : zero_off));
        }
        const int8_t* bb = plds + ring_off + buf * (BN * BK);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int r = wn * WN + j * 32 + frag_row;
            b[j] = *reinterpret_cast<const i32x4*>(&bb[r * BK + swz<BK>(r, ks * 2 + frag_half) * 16]);
        }
        advance();
    };
    wait_vmcnt<0>();
    __syncthreads();
    read_slice(0, 0, af[0], bf[0]);
    // Step kt as in the ring kernel: its weights' successor NBUF-1 steps on is requested into the buffer
    // of step kt-1, the fragments of a slice are read while the slice before it is multiplied, and the
    // barrier in front of the next step's first slice comes before the last multiply of this one.
    for (int kt0 = 0; kt0 < ksteps; kt0 += NBUF) {
#pragma unroll
        for (int p = 0; p < NBUF; ++p) {
            const int kt = kt0 + p;
            if (kt >= ksteps) break;
            fetch(kt + NBUF - 1, (p + NBUF - 1) % NBUF);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks + 1 < KS) {
                    read_slice(p, ks + 1, af[(ks + 1) & 1], bf[(ks + 1) & 1]);
                } else {
                    wait_vmcnt<(NBUF - 2) * B_LOADS>();
                    __syncthreads();
                    read_slice((p + 1) % NBUF, 0, af[0], bf[0]);      // (after the last step: zeros, not used)
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = mfma_tile<RQ>(af[ks & 1][i], bf[ks & 1][j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    wait_vmcnt<0>();    // surplus requests must land before their LDS is reused
    __syncthreads();

    // epilogue as in the ring kernel
    int32_t* stage = reinterpret_cast<int32_t*>(&plds[wave * stage_bytes<RQ, WN, 8>()]);
    const float scale = scale_x[1] * scale_w[1];
    const float inv = RQ ? requant_inv(rq, blockIdx.x == 0 && tid == 0) : 0.0f;
    const int dup_n = RQ && dup_off > 0 ? (*dup_count < kDupCap ? *dup_count : kDupCap) : 0;
    emit_tile<RQ, TM, TN, 8>(acc, stage, lane, row0 + wm * WM, col0 + wn * WN, wn * WN, M, N, scale, Y, ldy, acc_out, ldacc, rq,
                      inv, dup_list, dup_n, RQ && bn == tiles_n - 1 && wn == 0, row0 + BM <= M && col0 + BN <= N);
}

constexpr int64_t kWholeKMaxLds = 160 * 1024;  // LDS of one CU
constexpr int kMaxDevices = 64;

int compute_units() {
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    int n = cached[dev].load(std::memory_order_acquire);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cached[dev].store(n, std::memory_order_release);
    }
    return n;
}

// ---------------------------------------------------------------------------------------------
// Split + quantize + GEMM in one launch: the A operand is the fp32 activation matrix X [M, C*g]
// itself.  A workgroup takes 128 rows of X and all N <= 256 output columns, walks K in steps of
// 64 source columns, and per step turns its 128 x 64 floats (16-byte loads, two steps ahead, held
// in registers) into codes on the static grid (Eq. 1, the arithmetic of the streaming pass) and
// writes them into LDS in the layout the matrix cores read; the weight codes of the step come
// through registers as well.  The expanded layer's appended channels (the activation side of
// Eq. 3: un-scaled copies) cost no memory traffic at all: the copy of a column is the byte that
// was just written into LDS, so after each step the copies whose sources lie in it are moved,
// byte by byte, into a second LDS area laid out as the K-steps that follow the C*g columns, and
// those steps are multiplied last.  The code tensor Xq never exists in memory: 4 bytes read per
// element of X and 4 written per output, instead of 4 + 1 and 1 + 4 for the two launches.
//
// Per-workgroup set-up: the appended columns e = 0 .. s*g-1 (expanded column C*g + e, source
// column chan_src[C + e/g]*g + e%g) are bucketed by the K-step of their source (counts, prefix,
// fill: three short LDS passes).
// ---------------------------------------------------------------------------------------------
constexpr int kFusedMaxBM = 128;
constexpr int kFusedMaxTail = 2048;    // appended columns s*g
constexpr int kFusedMaxK = 8192;       // unexpanded columns C*g

struct FusedLds {
    int a_off, b_off, tail_off, first_off, cursor_off, ent_off, total;
};
static FusedLds fused_lds(int BM, int BN, int ksteps_main, int tail_steps, int T) {
    FusedLds l;
    l.a_off = 0;
    l.b_off = 2 * BM * 64;
    l.tail_off = l.b_off + 2 * BN * 64;
    l.first_off = l.tail_off + tail_steps * BM * 64;
    l.cursor_off = l.first_off + (ksteps_main + 2) * 4;
    l.ent_off = l.cursor_off + (ksteps_main + 1) * 4;
    l.total = l.ent_off + (T > 0 ? T : 1) * 4;
    return l;
}

template <int BN, int BM, int NT, int WPE, int SETS>
__global__ __launch_bounds__(NT, WPE) void split_act_qgemm_kernel(
    const float* __restrict__ X, int64_t ldx, int M, int C, int g, int s,
    const int32_t* __restrict__ chan_src, const float* __restrict__ thr, float qmax,
    const int8_t* __restrict__ Wq, int64_t ldw, int N, int ksteps_main, int ksteps_all, int rem,
    const float* __restrict__ scale_w, float* __restrict__ scale_x_out, int32_t* __restrict__ acc_out,
    int64_t ldacc, float* __restrict__ Y, int64_t ldy, FusedLds L, int bm_stride) {
    // bm_stride: rows between consecutive workgroups' first rows (<= BM): a workgroup owns rows
    // row0 .. row0 + bm_stride - 1 and the rest of its BM rows are idle (nothing fetched or stored).
    // ksteps_main: whole 64-column steps of X; rem: the columns of X left over after them (< 64).
    // They and the appended columns form the steps ksteps_main .. ksteps_all-1, which are assembled
    // in LDS (`tail`): the left-over columns are quantized straight into its first step.
    constexpr int NW = NT / 64;
    constexpr int A_PER = BM * 16 / NT;        // 16-byte loads of X per thread and step (64 floats x BM rows)
    constexpr int WAVES_M = BM / 32, WAVES_N = NW / WAVES_M, WN = BN / WAVES_N, TN = WN / 32;
    static_assert(A_PER >= 1 && A_PER * NT == BM * 16 && WAVES_M * WAVES_N == NW && TN >= 1 && TN * 32 * WAVES_N == BN,
                  "the threads tile a step of X, the waves tile the outputs in 32 x 32 blocks");
    constexpr int B_SLOTS = BN * 4, B_PER = (B_SLOTS + NT - 1) / NT;
    static_assert(BN == 64 || BN == 128 || BN == 256, "64, 128 or 256 output columns");
    static_assert(NW * 8 * WN * 4 <= 2 * BM * 64 + 2 * BN * 64, "the epilogue's staging area is the operand buffers");

    extern __shared__ __align__(1024) int8_t flds[];
    int8_t* a_buf = flds + L.a_off;
    int8_t* b_buf = flds + L.b_off;
    int8_t* tail = flds + L.tail_off;
    int* first = reinterpret_cast<int*>(flds + L.first_off);     // [ksteps_main + 2]
    int* cursor = reinterpret_cast<int*>(flds + L.cursor_off);   // [ksteps_main + 1]
    int* ent = reinterpret_cast<int*>(flds + L.ent_off);         // [T]: (e << 6) | source column inside its step

    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int row0 = (int)blockIdx.x * bm_stride;
    const int row_end = row0 + bm_stride < M ? row0 + bm_stride : M;
    const int T = s * g, tail_steps = ksteps_all - ksteps_main;

    // A: the step's BM x 16 float4 numbered row-major; load i of thread t is number i*NT + t, so each
    // load instruction of a wave covers four rows' whole 256 bytes
    const float* a_src[A_PER];
    unsigned a_ok = 0;  // bit i: load i of this thread lies in a row the workgroup owns
    int a_dst[A_PER];   // byte offset of the resulting code dword inside an A buffer
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        const int f = i * NT + tid, r = f >> 4, f4 = f & 15;
        int gr = row0 + r;
        if (gr < row_end) a_ok |= 1u << i;
        gr = gr < row_end ? gr : row_end - 1;          // rows past the workgroup's own are never fetched or stored
        a_src[i] = X + (int64_t)gr * ldx + f4 * 4;
        a_dst[i] = r * 64 + swz<64>(r, f4 >> 2) * 16 + (f4 & 3) * 4;
    }
    // B: 16-byte piece (slot & 3) of the step of weight row (slot >> 2)
    static_assert(B_PER * NT == B_SLOTS, "every thread moves the same number of weight pieces");
    const int8_t* b_src[B_PER];
    int b_dst[B_PER], b_piece[B_PER];
    const int b_pieces = (int)(ldw / 16);
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
        const int slot = u * NT + tid, n = slot >> 2, c = slot & 3;
        const int gn = col_clamp(n, N);
        b_src[u] = Wq + (int64_t)gn * ldw;
        b_piece[u] = c;
        b_dst[u] = n * 64 + swz<64>(n, c) * 16;
    }

    // SETS register sets in rotation: while one is processed, the next SETS-1 steps are on their way
    static_assert(SETS == 2 || SETS == 3, "one or two steps ahead");
    f32x4 av[SETS][A_PER];
    i32x4 bv[SETS][B_PER];
    auto load_step = [&](int kt, f32x4 (&a)[A_PER], i32x4 (&b)[B_PER]) {
        // Every lane issues the same loads at every step, whatever the step holds for it: a lane with
        // nothing to fetch (steps past the columns of X, pieces past a pitch, left-over columns that
        // do not exist) reads the 16 zero bytes instead, which costs one request per wave.  With no
        // branch around any load, the number of loads in flight is known at every wait, and the
        // waits let the two steps that are on their way stay on their way.
        const bool main_step = kt < ksteps_main, rest_step = kt == ksteps_main && rem > 0;
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int c0 = ((i * NT + tid) & 15) * 4;
            // left-over columns: a float4 that would cross the row's end starts four floats before
            // the end instead, and is shifted into place afterwards (nothing is read past the row)
            const bool ok = (a_ok >> i) & 1u;
            const bool whole = ok && (main_step || (rest_step && c0 + 3 < rem));
            const bool part = ok && rest_step && c0 < rem && !whole;
            const float* src = whole ? a_src[i] + (int64_t)kt * 64
                                     : (part ? a_src[i] + (int64_t)kt * 64 - c0 + (rem - 4)
                                             : reinterpret_cast<const float*>(zero_chunk));
            a[i] = *reinterpret_cast<const f32x4u*>(src);     // (shifted when it is used, not here)
        }
#pragma unroll
        for (int u = 0; u < B_PER; ++u) {
            const int piece = kt * 4 + b_piece[u];
            // a pitch may end inside the last K-step: what the row lacks counts as zero codes
            b[u] = *reinterpret_cast<const i32x4*>(kt < ksteps_all && piece < b_pieces ? b_src[u] + piece * 16
                                                                                       : zero_chunk);
        }
    };
    load_step(0, av[0], bv[0]);
    if (SETS == 3) load_step(1, av[1], bv[1]);

    // set-up behind the first requests: clear the appended steps, bucket the appended columns
    {
        i32x4 z = {0, 0, 0, 0};
        for (int o = tid; o < tail_steps * (BM * 64 / 16); o += NT) reinterpret_cast<i32x4*>(tail)[o] = z;
        for (int k = tid; k <= ksteps_main + 1; k += NT) first[k] = 0;
        __syncthreads();
        for (int e = tid; e < T; e += NT) {
            const int j = e / g, t = e - j * g;
            const int col = col_clamp(chan_src[C + j], C) * g + t;
            atomicAdd(&first[(col >> 6) + 1], 1);
        }
        __syncthreads();
        if (tid == 0) {
            int run = 0;
            for (int k = 0; k <= ksteps_main; ++k) {
                run += first[k + 1];
                first[k + 1] = run;
            }
        }
        __syncthreads();
        for (int k = tid; k <= ksteps_main; k += NT) cursor[k] = first[k];
        __syncthreads();
        for (int e = tid; e < T; e += NT) {
            const int j = e / g, t = e - j * g;
            const int col = col_clamp(chan_src[C + j], C) * g + t;
            const int pos = atomicAdd(&cursor[col >> 6], 1);
            ent[pos] = (e << 6) | (col & 63);
        }
        // (the first step's barrier completes the table before anyone reads it)
    }

    const float Tx = *thr;
    const float inv = inv_step_of(Tx, qmax);
    if (scale_x_out != nullptr && blockIdx.x == 0 && tid == 0) {
        scale_x_out[0] = Tx;
        scale_x_out[1] = Tx / qmax;
    }

    i32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0;
    const int frag_row = lane & 31, frag_half = lane >> 5;

    auto process = [&](int kt, const f32x4 (&a)[A_PER], const i32x4 (&b)[B_PER]) {
        const int buf = kt & 1;
        int8_t* ab = a_buf + buf * (BM * 64);
        int8_t* bb = b_buf + buf * (BN * 64);
        const bool main_step = kt < ksteps_main;
        const bool rest_step = kt == ksteps_main && rem > 0;     // holds the left-over columns of X
        if (main_step || rest_step) {
#pragma unroll
            for (int i = 0; i < A_PER; ++i) {
                const unsigned q4 = pack4(code_bits(a[i][0], inv, qmax), code_bits(a[i][1], inv, qmax),
                                          code_bits(a[i][2], inv, qmax), code_bits(a[i][3], inv, qmax));
                if (main_step) {
                    *reinterpret_cast<unsigned*>(ab + a_dst[i]) = q4;
                } else {
                    // into the first assembled step, byte by byte where the dword also holds copies.
                    // A float4 that straddled the row's end was fetched as columns rem-4 .. rem-1:
                    // this lane's column c0 + e is its element c0 + e - (rem - 4)
                    const int c0 = ((i * NT + tid) & 15) * 4;
                    if (c0 + 3 < rem) {
                        *reinterpret_cast<unsigned*>(tail + a_dst[i]) = q4;
                    } else {
                        const int d = c0 - (rem - 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (c0 + e < rem) tail[a_dst[i] + e] = (int8_t)((q4 >> (8 * (e + d))) & 0xFFu);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < B_PER; ++u) *reinterpret_cast<i32x4*>(bb + b_dst[u]) = b[u];
        __syncthreads();
        const int8_t* am = main_step ? ab : tail + (kt - ksteps_main) * (BM * 64);
        if (main_step || rest_step) {
            // the copies whose sources this step holds: one byte per (copy, row), to expanded column
            // C*g + e, which is column rem + e of the assembled steps
            const int e0 = first[kt], n = first[kt + 1] - e0;
            for (int idx = tid; idx < n * BM; idx += NT) {
                const int q = idx / BM, r = idx - q * BM;
                const int en = ent[e0 + q], e = rem + (en >> 6), c = en & 63;
                const int8_t code = am[r * 64 + swz<64>(r, c >> 4) * 16 + (c & 15)];
                const int te = e & 63;
                tail[(e >> 6) * (BM * 64) + r * 64 + swz<64>(r, te >> 4) * 16 + (te & 15)] = code;
            }
            if (rest_step) __syncthreads();    // this very step may hold some of those copies
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int ra = wm * 32 + frag_row;
            const i32x4 fa = *reinterpret_cast<const i32x4*>(&am[ra * 64 + swz<64>(ra, ks * 2 + frag_half) * 16]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int rb = wn * WN + j * 32 + frag_row;
                const i32x4 fb = *reinterpret_cast<const i32x4*>(&bb[rb * 64 + swz<64>(rb, ks * 2 + frag_half) * 16]);
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb, acc[j], 0, 0, 0);
            }
        }
    };

    for (int kt0 = 0; kt0 < ksteps_all; kt0 += SETS) {
#pragma unroll
        for (int p = 0; p < SETS; ++p) {
            const int kt = kt0 + p;
            if (kt < ksteps_all) {
                load_step(kt + SETS - 1, av[(p + SETS - 1) % SETS], bv[(p + SETS - 1) % SETS]);
                process(kt, av[p], bv[p]);
            }
        }
    }
    __syncthreads();   // the operand buffers are dead: they become the staging area

    int32_t* stage = reinterpret_cast<int32_t*>(flds + wave * (8 * WN * 4));
    const float scale = (Tx / qmax) * scale_w[1];
    const bool vec_y = (reinterpret_cast<uintptr_t>(Y) % 16 == 0) && (ldy % 4 == 0);
    const bool vec_a = acc_out != nullptr && (reinterpret_cast<uintptr_t>(acc_out) % 16 == 0) && (ldacc % 4 == 0);
    const Requant none{};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                stage[((lane >> 5) * 4 + e) * WN + j * 32 + (lane & 31)] = acc[j][q * 4 + e];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        emit_staged_rows<8, WN>(stage, lane, row0 + wm * 32 + q * 8, wn * WN, wn * WN, row_end, N, scale, Y, ldy,
                                acc_out, ldacc, vec_y, vec_a, none, 0.0f, nullptr, 0, false);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Where the one launch is ahead of the two (graph replays of the same shape, two launches / one).  It walks a
// row tile serially, so it needs tiles for every compute unit, the more the longer the rows and the more
// outputs the plain GEMM can spread instead:
//   N <= 128   K = 512, N = 64: 1.07 at 16384 rows; shorter rows are ahead from the smallest call on.  From 448 values
//              64 rows per compute unit, from 768 values 128.
//   N > 128    K = 1024, N = 256: 0.91 at 32768 rows, 1.10 at 50176; K = 2304: 0.25 at 1000.  More than 256 values:
//              156 rows per compute unit; up to 256 it is the short calls that save (their launch), 64 rows each.
// Below 128 values the pass over X is short either way and the output dominates.
bool split_act_qgemm_pays(int64_t M, int C, int g, int s, int64_t N, int64_t ldx) {
    const int64_t K = (int64_t)C * g, cus = compute_units();
    if (!split_act_qgemm_fits(M, C, g, s, N, ldx) || K < 128) return false;
    if (N <= 128) return K < 448 || M >= (K < 768 ? 64 : 128) * cus;
    return K <= 256 ? M <= 64 * cus : M >= 156 * cus;
}

bool split_act_qgemm_fits(int64_t M, int C, int g, int s, int64_t N, int64_t ldx) {
    const int64_t K = (int64_t)C * g, T = (int64_t)s * g;
    (void)ldx;
    return M >= 1 && M <= 0x7FFFFFFF - kFusedMaxBM && K >= 64 && K <= kFusedMaxK && T <= kFusedMaxTail && N >= 1 &&
           N <= 256;
}

template <int BN, int BM, int NT, int WPE, int SETS>
static hipError_t run_split_act_qgemm(const float* X, int64_t ldx, int64_t M, int C, int g, int s,
                                      const int32_t* chan_src, const float* thr, float qmax, const int8_t* Wq,
                                      int64_t ldw, int64_t N, int64_t Kexp, const float* scale_w,
                                      float* scale_x_out, int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy,
                                      hipStream_t stream) {
    const int ksteps_main = (int)((int64_t)C * g / 64), ksteps_all = (int)ceil_div(Kexp, 64);
    const int rem = (int)((int64_t)C * g - (int64_t)ksteps_main * 64);
    const FusedLds L = fused_lds(BM, BN, ksteps_main, ksteps_all - ksteps_main, s * g);
    if (L.total > kWholeKMaxLds) return hipErrorInvalidValue;
    static std::atomic<bool> opted_in[kMaxDevices];
    if (L.total > 65536) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&split_act_qgemm_kernel<BN, BM, NT, WPE, SETS>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    // When the row tiles would not even fill the chip's workgroup slots once, fewer rows per
    // workgroup and a workgroup in every slot: the pass is bound by what a compute unit can draw
    // from memory, so idle matrix rows cost nothing and idle compute units do (392 tiles of 128
    // rows on 512 slots: 134 -> 122 us on the 256-channel 3x3 layers at 14 x 14, batch 256).
    int64_t stride = BM;
    {
        int wpc = (int)(kWholeKMaxLds / L.total);
        wpc = wpc > WPE ? WPE : (wpc < 1 ? 1 : wpc);
        const int64_t slots = (int64_t)compute_units() * wpc;
        const int ts = tuning().fused_stride;
        if (ts > 0 && ts <= BM) stride = ts;
        else if (ts != 0 && ceil_div(M, BM) < slots) stride = ceil_div(M, slots);
        if (stride < BM / 2) stride = BM / 2;      // (never more than half of a tile idle)
    }
    return launch_kernel(kTimeGemm, split_act_qgemm_kernel<BN, BM, NT, WPE, SETS>, dim3((unsigned)ceil_div(M, stride)),
                         dim3(NT), (unsigned)L.total, stream, X, ldx, (int)M, C, g, s, chan_src, thr, qmax,
                         Wq, ldw, (int)N, ksteps_main, ksteps_all, rem, scale_w, scale_x_out, acc_out, ldacc, Y, ldy, L,
                         (int)stride);
}

hipError_t launch_split_act_qgemm(const float* X, int64_t ldx, int64_t M, int C, int g, int s,
                                  const int32_t* chan_src, const float* thr, float qmax, const int8_t* Wq,
                                  int64_t ldw, int64_t N, int64_t Kexp, const float* scale_w, float* scale_x_out,
                                  int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream) {
    if (!split_act_qgemm_fits(M, C, g, s, N, ldx)) return hipErrorInvalidValue;
#define OCS_FUSED_ARGS X, ldx, M, C, g, s, chan_src, thr, qmax, Wq, ldw, N, Kexp, scale_w, scale_x_out, acc_out, ldacc, Y, ldy, stream
    // Measured on the paper's layer shapes at batch 256.  Up to 128 output columns: workgroups of 64
    // rows on 4 waves, three or four of them per compute unit, each with its own barriers (10-20 %
    // ahead of 128-row ones).  256 columns: the weight codes a workgroup pulls per step weigh as much
    // as 64 rows of X, and 128 rows on 8 waves are ahead, except on very tall X, where two 64-row
    // workgroups per compute unit win.  One step of look-ahead everywhere: a second one was level or
    // behind (its registers cost a workgroup per compute unit).
    const int v = tuning().fused_variant;     // tests: 1 / 2 force the 64- / 128-row shape for N > 128
    if (N <= 64) return run_split_act_qgemm<64, 64, 256, 4, 2>(OCS_FUSED_ARGS);
    if (N <= 128) return run_split_act_qgemm<128, 64, 256, 3, 2>(OCS_FUSED_ARGS);
    if (v == 1 || (v != 2 && M >= 131072)) return run_split_act_qgemm<256, 64, 512, 4, 2>(OCS_FUSED_ARGS);
    return run_split_act_qgemm<256, 128, 512, 2, 2>(OCS_FUSED_ARGS);
#undef OCS_FUSED_ARGS
}

// ---------------------------------------------------------------------------------------------
// The layer of many rows as one launch with two kinds of waves (ocs_forward; codes included).  The two launches write every code
// and read it back; in the row-tile kernel above every wave requests, quantizes, meets the others and multiplies in turn, one
// step of X ahead, and with the codes written as well it is behind the two (25088 x 1024 -> 256 55.9 us against 39.4).  Here
// NQ waves only quantize: they hold no accumulators, so a step of 128 columns of X is on its way in their registers, each
// register requested again as soon as it is read (with two steps they spill: 57 us).  Floats through LDS instead cost it as much
// again as the fragments do (25088 x 1024 -> 256 39.8 us).  The other waves multiply, and request the weight codes straight
// into LDS ahead of their step: neither kind waits for the other's memory, and a step costs one barrier.  A workgroup of 64 rows on
// every compute unit; the next tile's first steps are requested before the last one's outputs are written.  Two steps of the weights, not
// one, are what 64 rows need, whose steps are half as long as their way from the L2 (12544 x 2304 -> 256, static grid: two launches
// 37.1 us, one step ahead 38.0, two 35.1, three 34.7; per batch 54.2, 52, 45.4); two steps of X, or half as many waves that
// quantize, are level or behind.  Where K is short it is 128 rows and one step (launch_panel_layer).
// The copies of the split channels are moved byte by byte, by the wave that quantizes their rows, into the steps that follow X's
// whole ones (`tail`), next to the columns left over after those; the tail is multiplied last.
// Bounded by what the compute units draw from memory: X, codes and outputs at 4.7 TB/s (25088 x 1024 -> 256 40.5 us as two launches,
// 32.7), 4.6 (12544 x 2304 -> 256 37.1 -> 34), 5.8 behind a max|X| pass that left X in the last-level
// cache (the same per batch 57.5 -> 45.0 with that pass).  12544 x 2304 -> 256, 34.0 us in a graph: 32.5 without the products, 30.1
// without the weights' requests, 28.2 without the stores of the codes, 23.2 without X's requests.
// ---------------------------------------------------------------------------------------------
struct PanelLayer {
    const float* X;
    int64_t ldx;
    int M, C, g, s;
    const int32_t* chan_src;
    const float* thr;          // the threshold (n_max == 0), or n_max maxima
    int n_max;
    float clip, qmax;
    int8_t* Xq;
    int64_t ldq;
    float* scale_x;
    const int8_t* Wq;
    int64_t ldw;
    int N;
    const float* scale_w;
    int32_t* acc_out;
    int64_t ldacc;
    float* Y;
    int64_t ldy;
    int kmain, kall, rem;      // whole steps of X; steps with the tail; X's columns after the whole steps
    int stride, rpw;           // rows of a workgroup (<= BM) and of each of its quantizing waves
    int tail_off, list_off, stage_off, tiles;
};

constexpr int kPanelMaxTail = 256;     // appended columns s*g
constexpr int kPanelStep = 128;        // columns of a step: whole lines of codes
// Steps of weight codes in LDS: 128 rows multiply for as long as a step is on its way (with three, 256 outputs 2-6 % behind, fewer level).
constexpr int panel_wbuf(int BM) { return BM >= 128 ? 2 : 3; }

template <int BM, int BN, int NQ, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__((NQ + WAVES_M * WAVES_N) * 64) void panel_layer_kernel(PanelLayer p) {
    constexpr int NM = WAVES_M * WAVES_N, WBUF = panel_wbuf(BM);
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
    constexpr int BK = kPanelStep, CPR = BK / 16, LG = 7;    // 16-byte pieces of a row of codes, BK = 1 << LG
    constexpr int LPR = BK / 4, RPL = 64 / LPR;              // X: lanes per row, rows per request
    constexpr int RPW = BM / NQ, LA = RPW / RPL;             // rows and requests of a step per quantizing wave
    constexpr int LB = BN * BK / 1024 / NM;                  // requests of a step of W per multiplying wave
    static_assert(TM >= 1 && TN >= 1 && TM * 32 * WAVES_M == BM && TN * 32 * WAVES_N == BN && LA >= 1 && LB >= 1, "tile");
    static_assert(NQ + NM <= 16, "waves of a workgroup");

    extern __shared__ __align__(1024) int8_t plds[];
    int8_t* codes = plds;
    int8_t* wring = codes + 2 * BM * BK;
    int8_t* tail = plds + p.tail_off;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&plds[0];
#else
    const unsigned lds0 = 0;
#endif
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tail_steps = p.kall - p.kmain, nx = p.kmain + (p.rem > 0 ? 1 : 0);
    // Rows of whole 4096 bytes: from the same step on in every workgroup, all addresses under way are alike in their low bits, and
    // meet on few of the memory's channels.  Each workgroup begins at another step (25088 x 1024 -> 256 37.9 -> 35.0 us), scattered,
    // since the channel also depends on the higher bits: with step = workgroup mod steps 32768 x 2048, a megabyte apart, took 108 us
    // for 75.  Other pitches spread by themselves and gain from rows read in one direction (200000 x 256 70.6 us, 89.4 turned).
    const int turn = p.kmain > 0 && p.ldx % 1024 == 0 ? (int)((blockIdx.x * 2654435761u >> 16) % (unsigned)p.kmain) : 0;
    auto step_of = [&](int it) -> int { return it >= p.kmain ? it : (it + turn < p.kmain ? it + turn : it + turn - p.kmain); };
    const bool multiplier = wave >= NQ;
    const int mw = multiplier ? wave - NQ : 0;

    // the barrier of a step: LDS accesses of this wave done, requests to memory still on their way
    auto step_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // the threshold, folded from its maxima by each wave for itself: no barrier before the first step
    auto threshold = [&]() -> float {
        if (p.n_max == 0) return *p.thr;
        float m = 0.0f;
        for (int i0 = lane; i0 < p.n_max; i0 += 256) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = p.thr[i0 + 64 * u < p.n_max ? i0 + 64 * u : p.n_max - 1];
            m = fmaxf(fmaxf(fmaxf(m, v[0]), fmaxf(v[1], v[2])), v[3]);
        }
        return p.clip * __uint_as_float(wave_umax32(__float_as_uint(m)));
    };

    if (multiplier) {
        // W: request u of multiplying wave f fills block u * NM + f of the step (the swizzle is the same for every u)
        static_assert(NM % 2 == 0, "the blocks of a wave begin at rows of one parity");
        unsigned wsrc[LB];
        const int w_end = (int)(p.ldw / 16);
        const int wpiece = swz<BK>((mw * 64 + lane) / CPR, lane % CPR);
#pragma unroll
        for (int u = 0; u < LB; ++u)                         // (at most 256 rows, ldw < 2^23)
            wsrc[u] = (unsigned)col_clamp(((u * NM + mw) * 64 + lane) / CPR, p.N) * (unsigned)p.ldw;
        const unsigned w0 = lds0 + (unsigned)(2 * BM * BK + mw * 1024);
        auto fetch_w = [&](int kt) {
            const int q = step_of(kt) * CPR + wpiece;
            const int8_t* base = p.Wq + (int64_t)q * 16;
            const unsigned slot = w0 + (unsigned)((WBUF == 2 ? kt & 1 : kt % WBUF) * (BN * BK));
#pragma unroll
            for (int u = 0; u < LB; ++u) lds_dma16(q < w_end ? base + wsrc[u] : zero_chunk, slot + u * (NM * 1024));
        };
        auto first_weights = [&]() {
#pragma unroll
            for (int k = 0; k < WBUF - 1; ++k)
                if (k < p.kall) fetch_w(k);
        };
        first_weights();
        const int wm = mw / WAVES_N, wn = mw % WAVES_N;
        const int frag_row = lane & 31, frag_half = lane >> 5;
        int32_t* stage = reinterpret_cast<int32_t*>(plds + p.stage_off) + mw * (8 * WN);
        i32x16 acc[TM][TN];
        i32x4 fa[2][TM], fb[2][TN];
        for (int tile = (int)blockIdx.x; tile < p.tiles; tile += (int)gridDim.x) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
            for (int kt = 0; kt < p.kall; ++kt) {
                // this wave's part of the step's weight codes (behind them only those of later steps)
                if (WBUF > 2 && kt + WBUF - 2 < p.kall) wait_vmcnt<(WBUF - 2) * LB>();
                else wait_vmcnt<0>();
                step_barrier();
                const int8_t* am = kt < p.kmain ? codes + (kt & 1) * (BM * BK) : tail + (kt - p.kmain) * (BM * BK);
                const int8_t* wb = wring + (WBUF == 2 ? kt & 1 : kt % WBUF) * (BN * BK);
                auto read_slice = [&](int ks) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int r = wm * WM + i * 32 + frag_row;
                        fa[ks & 1][i] = *reinterpret_cast<const i32x4*>(&am[r * BK + swz<BK>(r, ks * 2 + frag_half) * 16]);
                    }
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int r = wn * WN + j * 32 + frag_row;
                        fb[ks & 1][j] = *reinterpret_cast<const i32x4*>(&wb[r * BK + swz<BK>(r, ks * 2 + frag_half) * 16]);
                    }
                };
                read_slice(0);
                __builtin_amdgcn_sched_barrier(0);
                if (kt + WBUF - 1 < p.kall) fetch_w(kt + WBUF - 1);      // into the slot multiplied before this barrier
#pragma unroll
                for (int ks = 0; ks < BK / 32; ++ks) {
                    if (ks + 1 < BK / 32) read_slice(ks + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_tile<false>(fa[ks & 1][i], fb[ks & 1][j], acc[i][j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            step_barrier();                                      // the tile's operands have been read: the next one's may come
            if (tile + (int)gridDim.x < p.tiles) first_weights();
            const int row0 = tile * p.stride, row_end = row0 + p.stride < p.M ? row0 + p.stride : p.M;
            const float scale = (threshold() / p.qmax) * p.scale_w[1];
            emit_tile<false, TM, TN, 8>(acc, stage, lane, row0 + wm * WM, wn * WN, wn * WN, row_end, p.N, scale, p.Y, p.ldy,
                                        p.acc_out, p.ldacc, Requant{}, 0.0f, nullptr, 0, false, row0 + BM <= row_end && BN <= p.N);
        }
        return;
    }

    // the appended columns' sources, up to ET a lane: expanded column C g + e is a copy of column col[e / 64] of lane e % 64
    constexpr int ET = kPanelMaxTail / 64;
    const int T = p.s * p.g;
    int col[ET];
#pragma unroll
    for (int q = 0; q < ET; ++q) {
        const int e = q * 64 + lane, j = e / p.g;
        col[q] = e < T ? col_clamp(p.chan_src[p.C + j], p.C) * p.g + (e - j * p.g) : -1;
    }
    const float Tx = threshold();
    const float inv = inv_step_of(Tx, p.qmax);
    if (blockIdx.x == 0 && tid == 0) {
        p.scale_x[0] = Tx;
        p.scale_x[1] = Tx / p.qmax;
    }
    int* list = reinterpret_cast<int*>(plds + p.list_off) + wave * kPanelMaxTail;
    const int c4 = (lane % LPR) * 4;
    int own;                                                 // rows of the tile this wave quantizes (none: <= 0)
    unsigned xoff[LA], qoff[LA];                             // bytes from the tile's first row of X, of the codes (ldx, ldq < 2^23)
    int at[LA];                                              // this lane's four codes inside a step's buffer
    const char* xbase;
    char* qbase;
    f32x4 av[LA];
    auto load_x = [&](int kt, int u) -> f32x4 {
        const bool main_step = kt < p.kmain, rest = kt == p.kmain && c4 < p.rem;
        // left-over columns: four floats that would cross the row's end start four before it (K >= 64) and are shifted into
        // place when they are used; nothing to request: sixteen zero bytes
        const int off = rest && c4 + 3 >= p.rem ? p.rem - 4 - c4 : 0;
        const float* src = main_step || rest ? reinterpret_cast<const float*>(xbase + (int64_t)step_of(kt) * (4 * BK) + xoff[u]) + off
                                             : reinterpret_cast<const float*>(zero_chunk);
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(src));
    };
    // X: request u of a step covers RPL rows of the wave, LPR lanes each.  Rows that do not exist repeat the last one that
    // does, codes and all, so that no request and no write has a condition; a wave without any row does nothing.
    auto begin = [&](int tile) {
        const int row0 = tile * p.stride, row_end = row0 + p.stride < p.M ? row0 + p.stride : p.M;
        own = row_end - row0 - wave * p.rpw;
        own = own < p.rpw ? own : p.rpw;
        xbase = reinterpret_cast<const char*>(p.X + (int64_t)row0 * p.ldx);
        qbase = reinterpret_cast<char*>(p.Xq + (int64_t)row0 * p.ldq);
        if (own <= 0) return;
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            int r = u * RPL + lane / LPR;
            r = wave * p.rpw + (r < own ? r : own - 1);
            xoff[u] = ((unsigned)r * (unsigned)p.ldx + (unsigned)c4) * 4u;
            qoff[u] = (unsigned)r * (unsigned)p.ldq + (unsigned)c4;
            at[u] = r * BK + swz<BK>(r, c4 >> 4) * 16 + (c4 & 15);
        }
#pragma unroll
        for (int u = 0; u < LA; ++u) av[u] = load_x(0, u);
    };
    auto code4 = [&](const f32x4& v) -> unsigned {
        return pack4(code_bits(v[0], inv, p.qmax), code_bits(v[1], inv, p.qmax), code_bits(v[2], inv, p.qmax), code_bits(v[3], inv, p.qmax));
    };
    auto quantize = [&](int it, int u, const f32x4& v) {
        const unsigned q4 = code4(v);
        *reinterpret_cast<unsigned*>(codes + (it & 1) * (BM * BK) + at[u]) = q4;
        __builtin_nontemporal_store(q4, reinterpret_cast<unsigned*>(qbase + (int64_t)step_of(it) * BK + qoff[u]));
    };
    // The copies of this wave's rows whose sources step it holds (a wave's LDS accesses execute in order: no barrier)
    auto copies = [&](int it) {
        const int step = step_of(it);
        int n = 0;
#pragma unroll
        for (int q = 0; q < ET; ++q) {
            const bool here = (col[q] >> LG) == step;          // (-1 >> LG is no step)
            const unsigned long long m = __ballot(here);
            const int to = n + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
            if (here) list[to] = ((q * 64 + lane) << LG) | (col[q] & (BK - 1));
            n += __popcll(m);
        }
        const int8_t* am = it < p.kmain ? codes + (it & 1) * (BM * BK) : tail;
        for (int idx = lane; idx < n * RPW; idx += 64) {
            const int en = list[idx / RPW], r = wave * p.rpw + idx % RPW, e = p.rem + (en >> LG), c = en & (BK - 1), te = e & (BK - 1);
            if (idx % RPW < own)
                tail[(e >> LG) * (BM * BK) + r * BK + swz<BK>(r, te >> 4) * 16 + (te & 15)] =
                    am[r * BK + swz<BK>(r, c >> 4) * 16 + (c & 15)];
        }
    };

    begin((int)blockIdx.x);
    for (int tile = (int)blockIdx.x; tile < p.tiles; tile += (int)gridDim.x) {
        const bool live = own > 0;
        if (live) {                                          // this wave's rows of the tail
            for (int o = lane; o < tail_steps * RPW * CPR; o += 64) {
                const int k = o / (RPW * CPR), r = o / CPR % RPW, c = o % CPR;
                const i32x4 z = {0, 0, 0, 0};
                if (r < own) *reinterpret_cast<i32x4*>(&tail[k * (BM * BK) + (wave * p.rpw + r) * BK + c * 16]) = z;
            }
        }
        int it = 0;
        if (live && p.kmain >= 2) {
            // steps whose requests ahead are whole ones, without a condition; the first of them by itself: the requests and
            // writes under way are then the same number on every way into the loop, and its waits no stricter than they must be
            auto step = [&]() {
#pragma unroll
                for (int u = 0; u < LA; ++u) {
                    quantize(it, u, av[u]);
                    av[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(xbase + (int64_t)step_of(it + 1) * (4 * BK) + xoff[u]));
                    __builtin_amdgcn_sched_barrier(0);       // (or the arithmetic of later requests, and its waits, move ahead)
                }
                // (the tail is read behind a later barrier: with 128 rows the copies are made while the others multiply, 25088 x 1024 -> 256
                // 34.2 -> 32.7 us; with 64 the next step waits for them, 12544 x 2304 -> 256 per batch 45.2 -> 46.7)
                if (BM < 128) copies(it);
                step_barrier();
                if (BM >= 128) copies(it);
                __builtin_amdgcn_sched_barrier(0);
                ++it;
            };
            step();
            while (it + 2 <= p.kmain) step();
        }
        for (; it < nx; ++it) {
            if (live && it < p.kmain) {
#pragma unroll
                for (int u = 0; u < LA; ++u) {
                    quantize(it, u, av[u]);
                    av[u] = load_x(it + 1, u);
                }
                copies(it);
            } else if (live) {
#pragma unroll
                for (int u = 0; u < LA; ++u) {
                    const unsigned q4 = code4(av[u]);
                    if (c4 + 3 < p.rem) {
                        *reinterpret_cast<unsigned*>(tail + at[u]) = q4;
                    } else {
                        const int d = c4 - (p.rem - 4);      // (fetched as columns rem - 4 .. rem - 1)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (c4 + e < p.rem) tail[at[u] + e] = (int8_t)((q4 >> (8 * (e + d))) & 0xFFu);
                    }
                }
                copies(it);
            }
            step_barrier();
        }
        // what follows the whole steps of a row: left-over columns, copies, and zeros up to the pitch (this wave's rows of the
        // tail are complete)
        if (live) {
            const int pieces = (int)(p.ldq / 16) - p.kmain * CPR;
            for (int idx = lane; idx < own * pieces; idx += 64) {
                const int r = wave * p.rpw + idx / pieces, c = idx % pieces;
                i32x4 q = {0, 0, 0, 0};
                if (c < tail_steps * CPR)
                    q = *reinterpret_cast<const i32x4*>(&tail[(c / CPR) * (BM * BK) + r * BK + swz<BK>(r, c % CPR) * 16]);
                *reinterpret_cast<i32x4*>(qbase + (int64_t)r * p.ldq + (int64_t)p.kmain * BK + c * 16) = q;
            }
        }
        if (tile + (int)gridDim.x < p.tiles) begin(tile + (int)gridDim.x);
        for (; it < p.kall + 1; ++it) step_barrier();                    // the tail's steps, and the last of the operands
    }
}

template <int BM, int BN, int NQ, int WAVES_M>
static int64_t panel_lds(int64_t tail_steps, PanelLayer* p) {
    constexpr int BK = kPanelStep, WBUF = panel_wbuf(BM);
    const int64_t tail = (2 * BM + WBUF * BN) * BK, list = tail + tail_steps * BM * BK, end = list + NQ * kPanelMaxTail * 4;
    // With three steps of weights the epilogue's stage is the last of their slots: the next tile's first steps go to the others,
    // and that one is requested only behind a barrier that every wave reaches after its epilogue.
    constexpr int STAGE = WAVES_M * 8 * BN * 4;
    static_assert(WBUF == 2 || STAGE <= BN * BK, "the stage fits a step of weights");
    if (p != nullptr) {
        p->tail_off = (int)tail;
        p->list_off = (int)list;
        p->stage_off = (int)(WBUF > 2 ? tail - BN * BK : end);
    }
    return WBUF > 2 ? end : end + STAGE;
}

template <int BM, int BN, int NQ, int WAVES_M, int WAVES_N>
static hipError_t run_panel(PanelLayer p, hipStream_t stream) {
    constexpr int BK = kPanelStep;
    const int64_t K = (int64_t)p.C * p.g, Kexp = (int64_t)(p.C + p.s) * p.g;
    p.kmain = (int)(K / BK);
    p.kall = (int)ceil_div(Kexp, BK);
    p.rem = (int)(K - (int64_t)p.kmain * BK);
    const int64_t o = panel_lds<BM, BN, NQ, WAVES_M>(p.kall - p.kmain, &p);
    if (o > kWholeKMaxLds) return hipErrorInvalidValue;
    static std::atomic<bool> opted_in[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!opted_in[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&panel_layer_kernel<BM, BN, NQ, WAVES_M, WAVES_N>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
        if (e != hipSuccess) return e;
        opted_in[dev].store(true, std::memory_order_release);
    }
    // a workgroup on every compute unit, rounds of tiles as even as they can be, no more than half of a tile idle
    const int64_t slots = compute_units(), rounds = ceil_div(p.M, slots * BM);
    int64_t st = ceil_div(p.M, slots * rounds);
    st = st < BM / 2 ? BM / 2 : (st > BM ? BM : st);
    p.stride = (int)st;
    p.rpw = (int)ceil_div(st, NQ);
    p.tiles = (int)ceil_div(p.M, st);
    return launch_kernel(kTimeGemm, panel_layer_kernel<BM, BN, NQ, WAVES_M, WAVES_N>,
                         dim3((unsigned)(p.tiles < slots ? p.tiles : slots)), dim3((NQ + WAVES_M * WAVES_N) * 64), (unsigned)o, stream, p);
}

static bool panel_fits(int64_t ldx, int64_t M, int C, int g, int s, int64_t ldq, int64_t ldw, int64_t N) {
    const int64_t K = (int64_t)C * g, T = (int64_t)s * g, pitch = (int64_t)1 << 23;      // (offsets of 128 rows in 32 bits)
    if (K < 64 || T > kPanelMaxTail || N > 256 || M > 0x7FFFFFFF - 256 || ldx >= pitch || ldq >= pitch || ldw >= pitch) return false;
    const int64_t tail_steps = ceil_div(K + T, kPanelStep) - K / kPanelStep;
    return tail_steps <= 2;                              // (what the widest instance has LDS for)
}

hipError_t launch_panel_layer(const float* X, int64_t ldx, int64_t M, int C, int g, int s, const int32_t* chan_src,
                              const float* thr, int n_max, float clip, float qmax, int8_t* Xq, int64_t ldq,
                              float* scale_x, const int8_t* Wq, int64_t ldw, int64_t N, const float* scale_w,
                              int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream) {
    PanelLayer p;
    p.X = X; p.ldx = ldx; p.M = (int)M; p.C = C; p.g = g; p.s = s;
    p.chan_src = chan_src; p.thr = thr; p.n_max = n_max; p.clip = clip; p.qmax = qmax;
    p.Xq = Xq; p.ldq = ldq; p.scale_x = scale_x; p.Wq = Wq; p.ldw = ldw; p.N = (int)N; p.scale_w = scale_w;
    p.acc_out = acc_out; p.ldacc = ldacc; p.Y = Y; p.ldy = ldy;
    // Tiles of 128 rows where K is short: half of the steps, each twice as long.  Time with 64 rows / with 128 where the rule takes these (layers in a graph,
    // inputs rotating, K = 384 to 1280, 50 to 256 outputs, 100 to 2500 rows per compute unit; rounds: of 64-row tiles):
    //   up to 64 outputs     static, more than 20 rounds 1.00-1.04; per batch 0.97-1.05
    //   65 to 128            static, 2 rounds 0.95-1.09, 6 and more 0.98-1.08; per batch 0.98-1.08
    //   more                 2 rounds 0.97-1.15 static (1024 columns 0.94-1.06), 0.96-1.06 per batch; 4 and more 0.97-1.10, 0.99-1.08
    // An odd count leaves the last round of 128 rows half empty (5 rounds 0.89-0.99).  Outputs that share lines between rows lose by taller tiles (100
    // outputs, 6 rounds and more 0.95-1.00; 110, 2 rounds 0.93-0.99).  More columns: 896 0.95-1.02, 128 outputs of 768 static 0.92-1.01, 1536 to 4608 in 2
    // rounds 0.89-1.05; per batch up to 128 outputs 1024 to 3456 0.92-1.03, 4608 0.96-1.06, 9216 in 2 rounds 1.00-1.06.  With 64 rows throughout
    // 512 -> 128 takes 19.7 / 161 / 362 us at 25563 / 281563 / 639963 rows, 18.8 / 154 / 334 so.
    const int64_t K = (int64_t)C * g, rounds = ceil_div(M, 64 * compute_units());
    const bool even = rounds % 2 == 0, lines = N % 32 == 0;
    bool tall;
    if (N <= 128 && n_max > 0) tall = K <= (N > 64 ? 768 : 704) || (K > 4608 && rounds == 2);
    else if (N <= 64) tall = K <= 576 && rounds > 20 && lines;
    else if (N <= 128) tall = K <= 704 && ((rounds == 2 && N % 4 == 0) || (lines && ((rounds > 5 && even) || rounds > 12)));
    else tall = K <= (rounds == 2 ? 1280 : 768) && (even || rounds > 16);
    tall = tall && rounds > 1;
    if (N <= 64) return tall ? run_panel<128, 64, 8, 4, 2>(p, stream) : run_panel<64, 64, 8, 2, 2>(p, stream);
    if (N <= 128) return tall ? run_panel<128, 128, 8, 2, 4>(p, stream) : run_panel<64, 128, 8, 2, 4>(p, stream);
    return tall ? run_panel<128, 256, 8, 2, 4>(p, stream) : run_panel<64, 256, 8, 2, 4>(p, stream);
}

// Where the one launch is ahead of the two: ranges of two / one in time over 64, 128 and 256 outputs, copies 5 % (2 % in 3x3 layers), static grid, passes
// queued back to back with the inputs rotating and the same in a graph; "again": a graph on one input again; in brackets passes queued with a
// per-batch grid.
//   rows per compute unit, K = 384 to 640: 28 and 32 0.99-1.29, again 1.04-1.14 (0.99-1.11); 36 to 64 1.15-1.60, again 1.10-1.64
//                (1.06-1.30); 66 and 80, a second round of a few rows, 0.96-1.07; 98 to 128 1.07-1.41, again 1.11-1.28 (1.04-1.22); 130 and 144
//                1.06-1.19, again 0.98-1.10; 160 to 191 1.11-1.25, again 1.02-1.13; 192 to 400 1.11-1.33, again 1.00-1.20 (1.05-1.24).
//                K = 768 to 1152: 36 1.00-1.25; 44 to 64 1.10-1.72, again 1.07-1.55 (1.09-1.49); 66 and 80 0.86-1.13, again 0.82-1.03; 96 0.96-1.18;
//                98 to 128 1.02-1.43, again 0.98-1.18 (1.12-1.21); 130 and 144 0.97-1.16, again 0.91-1.05; 160 to 191 1.04-1.22, again
//                0.98-1.12; 192 to 400 1.09-1.29, again 1.01-1.29 (1.06-1.29).
//                K = 2304: 28 and 32 0.92-1.04; 36 1.00-1.14, again 0.96-1.10; 44 to 64 1.05-1.31, again 1.00-1.16 (1.11-1.28); 66 and 80
//                0.86-1.03; 98 to 128 1.03-1.14, again 1.01-1.14 (1.15-1.25); 130 to 191 1.08-1.24; 192 to 400 1.17-1.24 (1.14-1.25).
//                K = 3456 and 4608: 44 and 48 1.00-1.21, again up to 128 outputs 1.01-1.09, 256 0.93-0.99 (1.14-1.25); 52 to 64 1.06-1.29, again
//                0.99-1.29; 98 to 300 1.15-1.28 (1.16-1.30).  K = 6912 and 9216: 40 to 200 1.15-1.35 (1.13-1.36).  (129 to 191 rows would
//                gain with long K and lose with short: left to the two.)
//   columns      K = 192: 48 and 64 1.20-1.44, 98 to 300 0.80-1.16 (0.90-1.09); 256 1.17-1.49, 0.89-1.19; 320 1.25-1.58, 0.95-1.23.
//   copies       moved byte by byte: a quarter of the columns 1.02-1.50, again 0.93-1.50 (0.99-1.24); half 0.96-1.36, again 0.88-1.36
//                (0.94-1.15).
//   whole lines  rows that begin inside one share it with their neighbour's last step, which reads it again: K = 400, 98 rows and more 1.01-1.11
//                (0.98-1.04), K = 1000 1.05-1.15, again 1.00-1.13.
//   pitch        rows that do not follow each other (32 values between them): K = 384 and 512 1.07-1.58 (0.98-1.15), K = 1024 1.07-1.27
//                (1.06-1.26).
bool panel_layer_pays(const float* X, int64_t ldx, int64_t M, int C, int g, int s, int64_t ldq, int64_t ldw, int64_t N) {
    const int mode = tuning().panel_layer;
    if (mode == 0 || !panel_fits(ldx, M, C, g, s, ldq, ldw, N)) return false;
    if (mode > 0) return true;
    const int64_t K = (int64_t)C * g, cus = compute_units();
    const bool one_round = M <= 64 * cus && M >= (K <= 640 ? 36 : (K > 2304 && N > 128 ? 52 : 44)) * cus;      // (of 64-row tiles)
    if (K < 384 || K % 64 != 0 || ldx % 32 != 0 || reinterpret_cast<uintptr_t>(X) % 128 != 0) return false;
    if (5 * (int64_t)s * g > K || (ldx != K && K < 1024)) return false;
    return one_round || (M >= 98 * cus && M <= 128 * cus) || M >= 192 * cus;
}

// ---------------------------------------------------------------------------------------------
// The layer of short code rows (up to OCS_SHORT_K bytes) as one launch, codes included (ocs_forward, ocs_conv_forward_requant): the
// streaming pass's one shot with the whole-K GEMM behind it.  The two launches write every code and read it back, and at this
// length of K neither has much else to do.  A workgroup of four waves takes 64 rows of X, requests all of them at once (U 16-byte loads
// a lane; nothing waits before the last is on its way) with all weight codes straight into LDS ahead of them, quantizes into the
// operand image in LDS, assembles the rows' tails there (left-over columns, copies, padding; the streaming pass's table), writes the
// image out as one block of whole 16-byte pieces, multiplies, and ends: no loop over tiles, so that the dispatcher keeps the chip inside one window
// that slides over X.  The image lies in LDS by steps of 32 bytes of K (one matrix instruction's), a step's rows one after the other with
// their two pieces exchanged every eight rows, the steps 32 bytes further apart: the reads of sixteen rows and the dwords a wave
// writes along a row of X fall in different banks.  The weights lie in the whole-K kernel's 64-byte steps: requested by 32 bytes of a row
// they cost the L1 twice the look-ups (401408 x 147 -> 64 71.5 us, 100352 x 256 -> 64 33.9).
// Bounded by HBM and the issue of vector instructions: X, codes and outputs at 6.1 TB/s where they are the traffic (401408 x 147 -> 64 88.5 ->
// 67.8 us for the layer, 802816 x 64 -> 64 86.8 -> 69.5), 5.0 where the launch is short (100352 x 256 -> 64 36.6 -> 30.8; with the next
// layer's codes as its output 38.8 -> 31.7).  By counters behind a max|X| pass the first reads 242 MB and writes 186 in 65 us (6.6 TB/s with what the
// last-level cache holds), 82 % of the vector issue in use, 9 % of the busy cycles bank conflicts of its tails; the last 55 % and 2 %.  X is read past the caches'
// replacement (with plain loads 74.6 and 80.8 us of the first two).  128 rows on eight waves: 74.9 and 72.1, 100352 x 256 -> 64 39.0;
// fewer workgroups on a compute unit (three, two): 71 and 84, 80 and 95.
// ---------------------------------------------------------------------------------------------
struct RowsLayer {
    const float* X;
    int64_t ldx;
    int M, C, g, s;
    const int32_t* chan_src;
    const float* thr;          // the threshold (n_max == 0), or n_max maxima
    int n_max;
    float clip, qmax;
    int8_t* Xq;
    int64_t ldq;
    float* scale_x;
    const int8_t* Wq;
    int64_t ldw;
    int N;
    const float* scale_w;
    int32_t* acc_out;
    int64_t ldacc;
    float* Y;
    int64_t ldy;
    int steps;                                      // 32-byte steps of a row
    unsigned magic_qc, magic_td, magic_pc;          // floor(2^32 / n): X's dwords, a tail's dwords, a code row's pieces
    int w_off, tab_off, dup_off, red_off;
    int flat;                                       // outputs leave as one block of a workgroup's rows
};


// item / n by the multiply (at most one low, corrected here), remainder in rem
__device__ __forceinline__ int div_magic(int item, int n, unsigned magic, int& rem) {
    unsigned q = __umulhi((unsigned)item, magic);
    unsigned r = (unsigned)item - q * (unsigned)n;
    if (r >= (unsigned)n) { ++q; r -= (unsigned)n; }
    rem = (int)r;
    return (int)q;
}

constexpr int kRowsBM = 64, kRowsNT = 256;             // rows and lanes of a workgroup: WAVES 2 x 2
constexpr int kRowsStep = kRowsBM * 32 + 32;            // a step of the image
// where byte 16 * piece of row r begins inside its 32 bytes
__device__ __forceinline__ int rows_swz(int r, int piece) { return ((piece ^ (r >> 3)) & 1) << 4; }

template <int BN, int U, bool RQ>
__global__ __launch_bounds__(kRowsNT) void rows_layer_kernel(RowsLayer p, Requant rq) {
    constexpr int BM = kRowsBM, NT = kRowsNT, NW = NT / 64, WN = BN / 2, TN = WN / 32, STEP = kRowsStep;
    // (no static LDS: beside a block aligned to 1024 bytes it takes as many)
    extern __shared__ __align__(1024) int8_t rlds[];
    float* red = reinterpret_cast<float*>(rlds + p.red_off);
    int* tab = reinterpret_cast<int*>(rlds + p.tab_off);
    int* dup_list = reinterpret_cast<int*>(rlds + p.dup_off);     // only with copies to write
    int* dup_count = dup_list + kDupCap;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) int8_t* lptr_t;
    const unsigned lds0 = (unsigned)(uintptr_t)(lptr_t)&rlds[0];
#else
    const unsigned lds0 = 0;
#endif
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = (int)blockIdx.x * BM;
    const int rows = p.M - row0 < BM ? p.M - row0 : BM;
    const int K = p.C * p.g, Ke = (p.C + p.s) * p.g, Q = K / 4, rem = K - 4 * Q, Qc = Q + (rem > 0 ? 1 : 0);
    const int TD = p.steps * 8 - Q;                             // dwords of a row's tail

    // weights: piece b of a 64-byte step = rows 16b .. 16b+15, as in the whole-K kernel
    {
        const int w_pieces = (int)(p.ldw / 16);
        for (int b = wave; b < BN / 16; b += NW) {
            const int r = b * 16 + (lane >> 2);
            const int8_t* rowp = p.Wq + (int64_t)(r < p.N ? r : p.N - 1) * p.ldw;
            int piece = swz<64>(r, lane & 3);
            for (int kt = 0; 2 * kt < p.steps; ++kt, piece += 4)
                lds_dma16(piece < w_pieces ? rowp + piece * 16 : zero_chunk, lds0 + (unsigned)(p.w_off + (kt * BN + b * 16) * 64));
        }
    }
    // the threshold or this lane's first of the maxima, and the tail's sources: all requested ahead of X, without a condition
    const float first = p.thr[tid < p.n_max ? tid : 0];
    const float step_w = p.scale_w[1];
    int tsrc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = 4 * Q + tid + i * NT;
        tsrc[i] = p.chan_src != nullptr ? p.chan_src[k >= K && k < Ke ? k / p.g : 0] : 0;
    }
    // item i of X = dword i % Qc of row i / Qc; a row's last, partial one is fetched as its last four floats
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int d;
        const int r = div_magic(tid + u * NT, Qc, p.magic_qc, d);
        const bool ok = r < rows;
        const float* src = p.X + (int64_t)(row0 + (ok ? r : 0)) * p.ldx + (ok ? (d < Q ? 4 * d : K - 4) : 0);
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(src));
    }
    // a tail's sources as places in the image (step and byte inside it; the row's exchange turns bit 4), -1: a zero code
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + i * NT, k = 4 * Q + e;
        if (e < 4 * TD) {
            int col = k < K ? k : -1;
            if (k >= K && k < Ke) col = col_clamp(tsrc[i], p.C) * p.g + k % p.g;
            tab[e] = col < 0 ? -1 : (col >> 5) * STEP + (col & 31);
        }
    }
    float T = first;
    if (p.n_max > 0) {
        float m = first;
        for (int i = tid + NT; i < p.n_max; i += NT) m = fmaxf(m, p.thr[i]);
        const unsigned w = wave_umax32(__float_as_uint(m));        // maxima of magnitudes: non-negative
        if (lane == 0) red[wave] = __uint_as_float(w);
        __syncthreads();
        T = red[0];
#pragma unroll
        for (int k = 1; k < NW; ++k) T = fmaxf(T, red[k]);
        T *= p.clip;
    }
    const float inv = inv_step_of(T, p.qmax), step_x = T / p.qmax;
    if (blockIdx.x == 0 && tid == 0) {
        p.scale_x[0] = T;
        p.scale_x[1] = step_x;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int d;
        const int r = div_magic(tid + u * NT, Qc, p.magic_qc, d);
        if (r >= BM) continue;
        unsigned q4 = pack4(code_bits(v[u][0], inv, p.qmax), code_bits(v[u][1], inv, p.qmax),
                            code_bits(v[u][2], inv, p.qmax), code_bits(v[u][3], inv, p.qmax));
        if (d >= Q) q4 >>= 8 * (4 - rem);
        *reinterpret_cast<unsigned*>(rlds + (d >> 3) * STEP + r * 32 + (((d & 7) * 4) ^ rows_swz(r, 0))) = q4;
    }
    __syncthreads();
    for (int it = tid; it < BM * TD; it += NT) {
        int td;
        const int r = div_magic(it, TD, p.magic_td, td);
        const i32x4 at = *reinterpret_cast<const i32x4*>(&tab[4 * td]);
        const int8_t* irow = rlds + r * 32;
        unsigned q4 = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned byte = (unsigned)(unsigned char)irow[at[e] < 0 ? 0 : at[e] ^ rows_swz(r, 0)];
            q4 |= (at[e] < 0 ? 0u : byte) << (8 * e);
        }
        const int d = Q + td;
        *reinterpret_cast<unsigned*>(rlds + (d >> 3) * STEP + r * 32 + (((d & 7) * 4) ^ rows_swz(r, 0))) = q4;
    }
    if constexpr (RQ) {
        if (p.dup_off > 0) build_dup_list<NT>(rq, p.N, 0, BN, dup_list, dup_count);
    }
    wait_vmcnt<0>();                                              // the weights (requested ahead of X: long there)
    __syncthreads();
    // the codes: one block of whole pieces
    {
        const int pc = (int)(p.ldq / 16);
        int8_t* out = p.Xq + (int64_t)row0 * p.ldq;
        for (int it = tid; it < rows * pc; it += NT) {
            int c;
            const int r = div_magic(it, pc, p.magic_pc, c);
            i32x4 q = {0, 0, 0, 0};                               // (a pitch longer than the image)
            if (c < 2 * p.steps) q = *reinterpret_cast<const i32x4*>(rlds + (c >> 1) * STEP + r * 32 + rows_swz(r, c));
            __builtin_nontemporal_store(q, reinterpret_cast<i32x4*>(out + (int64_t)it * 16));
        }
    }
    const int wm = wave >> 1, wn = wave & 1, frag_row = lane & 31, frag_half = lane >> 5;
    i32x16 acc[1][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][j][e] = 0;
    const int ra = wm * 32 + frag_row, piece = rows_swz(frag_row, frag_half);     // (the exchange repeats every 16 rows)
    for (int st = 0; st < p.steps; ++st) {
        const i32x4 a = *reinterpret_cast<const i32x4*>(rlds + st * STEP + ra * 32 + piece);
        const int8_t* wb = rlds + p.w_off + ((st >> 1) * BN + wn * WN + frag_row) * 64 + swz<64>(frag_row, (st & 1) * 2 + frag_half) * 16;
        i32x4 b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const i32x4*>(wb + j * 2048);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[0][j] = mfma_tile<RQ>(a, b[j], acc[0][j]);
    }
    __syncthreads();                                              // image and weights have been read: their LDS is the stage
    if constexpr (!RQ && BN <= 128) {
        if (p.flat) {
            float* out = reinterpret_cast<float*>(rlds);
            const float scale = step_x * step_w;
            const int col = wn * WN + (lane & 31);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (col + j * 32 >= p.N) continue;
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    out[(wm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * p.N + col + j * 32] = (float)acc[0][j][e] * scale;
            }
            __syncthreads();
            float* y = p.Y + (int64_t)row0 * p.N;                 // (64 rows: whole pieces of 16 bytes; fewer end the tensor)
            const int n = rows * p.N;
            for (int it = 4 * tid; it + 3 < n; it += 4 * NT)
                __builtin_nontemporal_store(*reinterpret_cast<const f32x4*>(out + it), reinterpret_cast<f32x4*>(y + it));
            if (tid < (n & 3)) y[(n & ~3) + tid] = out[(n & ~3) + tid];
            return;
        }
    }
    int32_t* stage = reinterpret_cast<int32_t*>(&rlds[wave * stage_bytes<RQ, WN, 8>()]);
    const float inv_next = RQ ? requant_inv(rq, blockIdx.x == 0 && tid == 0) : 0.0f;
    const int dup_n = RQ && p.dup_off > 0 ? (*dup_count < kDupCap ? *dup_count : kDupCap) : 0;
    emit_tile<RQ, 1, TN, 8>(acc, stage, lane, row0 + wm * 32, wn * WN, wn * WN, p.M, p.N, step_x * step_w, p.Y, p.ldy, p.acc_out,
                            p.ldacc, rq, inv_next, dup_list, dup_n, RQ && wn == 0, row0 + BM <= p.M && BN <= p.N);
}

// LDS of a launch: the image and the weights (or the epilogue's stage), the table of the tail's sources, the list of the next
// layer's copies, a word per wave for the maxima.  p (may be null) receives the offsets.
template <int BN, bool RQ>
static int64_t rows_layer_lds(int64_t K, int64_t steps, int s_next, RowsLayer* p) {
    const int64_t w = round_up(steps * kRowsStep, 1024), operands = w + (steps + 1) / 2 * BN * 64;
    const int64_t staging = p != nullptr && p->flat ? (int64_t)kRowsBM * 4 * p->N : (kRowsNT / 64) * stage_bytes<RQ, BN / 2, 8>();
    const int64_t tab = round_up(operands > staging ? operands : staging, 16), dup = tab + 16 * (steps * 8 - K / 4);
    const bool list = RQ && s_next > 0;
    const int64_t red = dup + (list ? (kDupCap + 1) * 4 : 0);
    if (p != nullptr) {
        p->w_off = (int)w;
        p->tab_off = (int)tab;
        p->dup_off = list ? (int)dup : 0;
        p->red_off = (int)red;
    }
    return red + (kRowsNT / 64) * 4;
}
constexpr int64_t kRowsMaxLds = 65536;                            // (what no kernel has to opt into)

template <int BN, int U, bool RQ>
static hipError_t run_rows(RowsLayer p, const Requant& rq, hipStream_t stream) {
    const int64_t K = (int64_t)p.C * p.g;
    auto magic_of = [](int64_t n) {          // floor(2^32 / n), or 2^32 - 1 for n = 1
        const uint64_t m = (((uint64_t)1) << 32) / (uint64_t)(n > 0 ? n : 1);
        return (unsigned)(m > 0xFFFFFFFFull ? 0xFFFFFFFFull : m);
    };
    p.magic_qc = magic_of(ceil_div(K, 4));
    p.magic_td = magic_of(p.steps * 8 - K / 4);
    p.magic_pc = magic_of(p.ldq / 16);
    const int64_t lds = rows_layer_lds<BN, RQ>(K, p.steps, rq.s_next, &p);
    if (lds > kRowsMaxLds) return hipErrorInvalidValue;
    return launch_kernel(kTimeGemm, rows_layer_kernel<BN, U, RQ>, dim3((unsigned)ceil_div(p.M, kRowsBM)), dim3(kRowsNT), (unsigned)lds,
                         stream, p, rq);
}
template <int BN, bool RQ>
static hipError_t run_rows_loads(const RowsLayer& p, const Requant& rq, hipStream_t stream) {
    const int64_t need = ceil_div(ceil_div((int64_t)p.C * p.g, 4), 4);   // 16-byte loads a lane
    if (need <= 4) return run_rows<BN, 4, RQ>(p, rq, stream);
    if (need <= 7) return run_rows<BN, 7, RQ>(p, rq, stream);
    if (need <= 10) return run_rows<BN, 10, RQ>(p, rq, stream);
    if constexpr (BN <= 128) {
        if (need <= 13) return run_rows<BN, 13, RQ>(p, rq, stream);
        if (need <= 16) return run_rows<BN, 16, RQ>(p, rq, stream);
        if (need <= 20) return run_rows<BN, 20, RQ>(p, rq, stream);
    }
    return hipErrorInvalidValue;
}

// Shapes it serves: what the table, the loads of a lane and 64 KB of LDS hold.
static bool rows_layer_fits(int64_t M, int C, int g, int s, int64_t ldq, int64_t N, const Requant& rq) {
    const int64_t K = (int64_t)C * g, steps = ceil_div(K + (int64_t)s * g, 32);
    if (K < 4 || steps > 10 || ldq > round_up(32 * steps, 64) || N > 256 || M > 0x7FFFFFFF - kRowsBM) return false;
    if (rq.Yq != nullptr)
        return N <= 64 ? rows_layer_lds<64, true>(K, steps, rq.s_next, nullptr) <= kRowsMaxLds
                       : N <= 128 && rows_layer_lds<128, true>(K, steps, rq.s_next, nullptr) <= kRowsMaxLds;
    if (N <= 128) return rows_layer_lds<128, false>(K, steps, 0, nullptr) <= kRowsMaxLds;
    return K <= 160 && rows_layer_lds<256, false>(K, steps, 0, nullptr) <= kRowsMaxLds;
}
// Where the one launch is ahead of the two: ranges of two / one in time at so many rows per compute unit, over passes queued back to back, the
// same in a graph, and a graph on one input again, all with a static grid; in brackets passes queued with a per-batch grid.  Copies 5 % (1 and
// 25 % alike).
//   rows      from sixteen on, where the layer of few tiles ends.  Up to 128 outputs, 64 to 256 columns of X: 32 to 130 1.01-1.9 (1.01-1.34), 130 to
//             400 0.97-1.75 (0.96-1.44), 784 to 10000 0.97-1.56 (1.01-1.42).
//   columns   few columns at many rows: codes and outputs are all there is, and a workgroup's 64 rows are a few requests.  K = 4 to 20: 784
//             1.02-1.48 (0.97-1.23), 1568 0.95-1.21 (0.93-1.12), 3136 0.85-1.24 (0.86-1.12), 6000 0.84-1.17 (0.79-1.12).  K = 24 to 56: 2200
//             0.97-1.36 (1.04-1.26), 3136 0.95-1.33 (0.93-1.25), 4400 0.91-1.32 (0.81-1.30).  Codes of the next layer out: K = 4 to 20 784
//             1.09-1.40 (1.01-1.29), 2200 0.93-1.20, 6000 0.84-1.15; 24 and more 0.98-1.48 (1.04-1.45).
//   rounds    more than 256 columns leave a compute unit two workgroups, 128 rows a round.  Up to 64 outputs 125 1.21-1.56, 130 0.93-1.06
//             (0.92-0.95), 140 0.96-1.15 (0.95-1.04), 150 0.98-1.12, 160 1.03-1.13.  Where the two launches' tiles come out even: 185
//             1.09-1.22, 196 0.94-1.07 (0.94-1.03), 210 0.97-1.10 (0.98-1.03), 230 1.02-1.14; codes out and more than 64 outputs 196 1.04-1.10.
//             Outputs in whole lines, which the two launches store best: 64 of them 217 0.91-0.96, 232 0.93-0.99 (0.94-0.98), 250 0.97-1.04, 262 0.97-1.02,
//             280 0.99-1.07; 128 129 0.95-1.01, 140 1.00-1.04, 217 0.95-1.02, 225 0.97-1.04, 232 1.00-1.07. 241 to 256 columns and 128 outputs 193 0.91-0.94 (0.99),
//             201 to 204 0.96-0.99 (0.99-1.02), 210 (1.03).
//   outputs   more than 128: rows of outputs that begin anywhere cost the two launches more than the one.  N % 4 != 0: 16 0.81-1.34, 24
//             0.99-1.29, 49 and more 1.02-1.60 (1.01-1.53).  N % 4 == 0, passes queued: 16 to 49 1.04-1.48 (1.02-1.35); in a graph up to 128 code
//             bytes 16 0.89-1.22 (up to 48 columns, or 64 and more than 192 outputs, 0.95-1.22), 24 0.96-1.16, 32 0.98-1.21; longer 16 0.81-0.97, 32
//             0.92-1.08, 49 0.99-1.18.  From there on up to 128 code bytes 0.95-1.55 (1.00-1.52); longer and N % 16 == 0, whole lines that a
//             launch of its own keeps up best, up to 240 outputs 64 to 128 1.05-1.34, 129 to 250 0.89-1.11 (0.89-1.07), more
//             0.80-1.12; other N % 4 == 0 140 0.95-1.18 (0.92-1.09), 196 and more 1.03-1.40.  256 outputs 0.95-1.13 (1.00-1.12).
//             More than 2^26 output values, us two / one: 802816 x 64 -> 256 179 / 188, 400000 x 48 -> 256 88.4 / 92.0, 800000 x 64 -> 160 136 / 145.
//   codes     of the next layer out: up to 64 columns 16 1.02-1.45; 96 and 128 16 0.89-1.34, with more than 64 outputs 20 0.95-1.34, 32 1.00-1.30;
//             more 32 0.93-1.61, 40 1.06-1.69 (1.01-1.30).
bool rows_layer_pays(int64_t M, int C, int g, int s, int64_t ldq, int64_t N, bool captured, const Requant& rq) {
    const int mode = tuning().rows_layer;
    if (mode == 0 || !rows_layer_fits(M, C, g, s, ldq, N, rq)) return false;
    if (mode > 0) return true;
    const int64_t cus = compute_units(), K = (int64_t)C * g, Kexp = K + (int64_t)s * g;
    const bool codes = rq.Yq != nullptr;
    auto between = [&](int64_t lo, int64_t hi) { return M > lo * cus && M <= hi * cus; };
    if (M > 784 * cus && K < 24) return false;
    if (M > 2200 * cus && K < 64 && !codes) return false;
    if (K > 256 && N <= 64 && between(128, 150)) return false;
    if (K > 256 && (N <= 64 || !codes) && between(190, 215)) return false;
    if (K > 256 && (N == 64 || N == 128) && !codes && (between(215, N == 64 ? 270 : 225) || (N == 128 && between(128, 134)))) return false;
    if (K > 240 && N == 128 && !codes && between(190, 206)) return false;
    if (codes) return M >= (K > 128 ? 48 : (K > 64 && N > 64 ? 32 : 16)) * cus;
    if (N <= 128) return M >= 16 * cus;
    if (M * N > (int64_t)1 << 26) return false;
    if (Kexp > 128 && N <= 240 && N % 4 == 0 && (between(128, 160) || (N % 16 == 0 && M > 128 * cus))) return false;
    int64_t least = Kexp > 128 && N % 4 != 0 ? 24 : 16;
    if (captured) {
        if (N % 4 != 0) least = 24;
        else if (Kexp > 128) least = 48;
        else least = K <= 48 || (K <= 64 && N > 192) ? 16 : 32;
    }
    return M >= least * cus;
}

hipError_t launch_rows_layer(const float* X, int64_t ldx, int64_t M, int C, int g, int s, const int32_t* chan_src, const float* thr,
                             int n_max, float clip, float qmax, int8_t* Xq, int64_t ldq, float* scale_x, const int8_t* Wq, int64_t ldw,
                             int64_t N, const float* scale_w, int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy,
                             hipStream_t stream, const Requant& rq) {
    RowsLayer p;
    p.X = X; p.ldx = ldx; p.M = (int)M; p.C = C; p.g = g; p.s = s;
    p.chan_src = chan_src; p.thr = thr; p.n_max = n_max; p.clip = clip; p.qmax = qmax;
    p.Xq = Xq; p.ldq = ldq; p.scale_x = scale_x; p.Wq = Wq; p.ldw = ldw; p.N = (int)N; p.scale_w = scale_w;
    p.acc_out = acc_out; p.ldacc = ldacc; p.Y = Y; p.ldy = ldy;
    p.steps = (int)ceil_div((int64_t)(C + s) * g, 32);
    // Rows of outputs that share lines leave through LDS as the one block that a workgroup's 64 rows are: stored row by row a line's parts come from several
    // instructions and waves, apart in time (us, row by row / as a block; past the caches' replacement row by row is 1.4 to 3 times as long): 332763 x
    // 64 -> 63 static 58.0 / 34.3, 511963 x 44 -> 94 105 / 53.4, x 64 -> 100 77 / 65; N % 4 != 0 1.03-2.06 in time, from 48 on 1.00-1.30,
    // 40 and 44 0.96-1.10, whole lines are stored as they are.
    p.flat = rq.Yq == nullptr && acc_out == nullptr && N % 32 != 0 && (N % 4 != 0 || N >= 48) && N <= 128 && ldy == N &&
             reinterpret_cast<uintptr_t>(Y) % 16 == 0;
    if (rq.Yq != nullptr) return N <= 64 ? run_rows_loads<64, true>(p, rq, stream) : run_rows_loads<128, true>(p, rq, stream);
    if (N <= 64) return run_rows_loads<64, false>(p, rq, stream);
    if (N <= 128) return run_rows_loads<128, false>(p, rq, stream);
    return run_rows_loads<256, false>(p, rq, stream);
}

// Dynamic LDS of a whole-K launch: operands (or the epilogue's staging area, if larger) and,
// when the output goes to the next layer as codes with copies, the table of those copies
// behind them (*dup_off = its byte offset, 0 = none).
template <int BM, int BN, int WAVES_M, int WAVES_N>
static int64_t wholek_lds_bytes(int64_t N, int64_t Kpad, const Requant& rq, int* dup_off = nullptr) {
    const int64_t operands = (Kpad / 64) * (BM + BN) * 64;
    const int64_t staging = (int64_t)WAVES_M * WAVES_N * (rq.Yq != nullptr ? stage_bytes<true, BN / WAVES_N, 8>() : stage_bytes<false, BN / WAVES_N, 8>());
    int64_t lds = operands > staging ? operands : staging;
    // Three of the 128 x 128 workgroups per compute unit, not four, and two where one tile holds a row of the
    // output: the store streams of more cost more than they hide (inside the pass, behind the launch that
    // wrote the codes: 802816 x 256 from 64 channels 189 us with three, 191 with four, 196 with two; 300000 x
    // 100 from 64 channels 54 with two, 58 with three, 60 with four; the GEMM alone, this floor against none:
    // 400000 x 200 x 68 109.9 / 114 us, 802816 x 256 x 68 133.2 / 135.2, 300000 x 128 x 68 29.1 / 29.5 and 300000 x 70 x 68
    // 39.9 / 39.6, 128 x 135 31.5 / 31.7, 128 x 269 52.8 / 52.6, 100000 x 256 x 269 level).
    const int64_t floor = N <= 128 ? 54 * 1024 : 41 * 1024;
    if (BM == 128 && BN == 128 && lds < floor) lds = floor;
    int off = 0;
    if (rq.Yq != nullptr && rq.s_next > 0) {
        off = (int)round_up(lds, 16);
        lds = off + (kDupCap + 1) * 4;
    }
    if (dup_off) *dup_off = off;
    return lds;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool RQ>
static hipError_t run_wholek_as(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw,
                             int64_t M, int64_t N, int64_t Kpad, const float* scale_x,
                             const float* scale_w, int32_t* acc_out, int64_t ldacc, float* Y,
                             int64_t ldy, hipStream_t stream, const Requant& rq) {
    int dup_off = 0;
    const int64_t lds = wholek_lds_bytes<BM, BN, WAVES_M, WAVES_N>(N, Kpad, rq, &dup_off);
    if (Kpad < 64 || Kpad % 64 != 0 || lds > kWholeKMaxLds) return hipErrorInvalidValue;
    // more than 64 KB of dynamic LDS has to be opted into, once per kernel and device (setting
    // it twice from two threads is harmless)
    static std::atomic<bool> opted_in[kMaxDevices];
    int dev = 0;
    if (lds > 65536) {
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(
                reinterpret_cast<const void*>(&qgemm_wholek_kernel<BM, BN, WAVES_M, WAVES_N, RQ>),
                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;   // one workgroup per tile: grid.x
    return launch_kernel(kTimeGemm, qgemm_wholek_kernel<BM, BN, WAVES_M, WAVES_N, RQ>,
                         dim3((unsigned)total), dim3(WAVES_M * WAVES_N * 64), (unsigned)lds, stream,
                         Xq, ldx, Wq, ldw, (int)M, (int)N, (int)(Kpad / 64), scale_x, scale_w,
                         acc_out, ldacc, Y, ldy, (int)tiles_n, (unsigned)total, dup_off, rq);
}
template <int BM, int BN, int WAVES_M, int WAVES_N>
static hipError_t run_wholek(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw,
                             int64_t M, int64_t N, int64_t Kpad, const float* scale_x,
                             const float* scale_w, int32_t* acc_out, int64_t ldacc, float* Y,
                             int64_t ldy, hipStream_t stream, const Requant& rq) {
    const auto run = rq.Yq != nullptr ? run_wholek_as<BM, BN, WAVES_M, WAVES_N, true> : run_wholek_as<BM, BN, WAVES_M, WAVES_N, false>;
    return run(Xq, ldx, Wq, ldw, M, N, Kpad, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq);
}

// The K extent dealt over the waves.  Any K extent and pitch the GEMM accepts.
template <int TM, int TN, int NW, int NBUF>
static hipError_t run_slice(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw, int64_t M, int64_t N,
                            int64_t Kpad, const float* scale_x, const float* scale_w, int32_t* acc_out,
                            int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream, const Requant& rq) {
    constexpr int BM = 32 * TM, BN = 32 * TN;
    const unsigned lds = (unsigned)(NW * NBUF * (BM + BN) * 64 + (rq.Yq != nullptr && rq.s_next > 0 ? (kDupCap + 1) * 4 : 0));
    if (Kpad < 64 || Kpad % 64 != 0) return hipErrorInvalidValue;
    if (lds > 65536) {
        static std::atomic<bool> opted_in[kMaxDevices];
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&qgemm_slice_kernel<TM, TN, NW, NBUF>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;   // one workgroup per tile: grid.x
    return launch_kernel(kTimeGemm, qgemm_slice_kernel<TM, TN, NW, NBUF>, dim3((unsigned)total), dim3(NW * 64), lds,
                         stream, Xq, ldx, Wq, ldw, (int)M, (int)N, (int)(Kpad / 64), scale_x, scale_w, acc_out,
                         ldacc, Y, ldy, (int)tiles_m, (int)tiles_n, N > M ? 1 : 0, rq);
}

// The waves' parts, the table of the columns past the whole steps and the maxima of the waves.
template <int TN, int NW, int NBUF, bool EARLY>
static int64_t slice_layer_lds(int64_t tail_cols) {
    return NW * slice_layer_wave_bytes<TN, NBUF + (EARLY ? 1 : 0)>() + tail_cols * 4 + NW * 4;
}

template <int TN, int A_PER, int NW, int NBUF, bool EARLY>
static hipError_t run_slice_layer(SliceLayer p, hipStream_t stream) {
    const int64_t bytes = slice_layer_lds<TN, NW, NBUF, EARLY>((p.ksteps - p.kmain) * 64);
    if (bytes > kWholeKMaxLds) return hipErrorInvalidValue;
    const unsigned lds = (unsigned)bytes;
    if (lds > 65536) {
        static std::atomic<bool> opted_in[kMaxDevices];
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&slice_layer_kernel<TN, A_PER, NW, NBUF, EARLY>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    p.tiles_m = (int)ceil_div(p.M, 32);
    p.tiles_n = (int)ceil_div(p.N, 32 * TN);
    p.rows_first = p.N > p.M ? 1 : 0;
    return launch_kernel(kTimeGemm, slice_layer_kernel<TN, A_PER, NW, NBUF, EARLY>, dim3((unsigned)(p.tiles_m * p.tiles_n)), dim3(NW * 64),
                         lds, stream, p);
}

// Columns of the one-launch layer's tile in units of 32 (0: more tiles than compute units).
static int slice_layer_tile(int64_t M, int64_t N) {
    const int64_t cus = compute_units(), tiles_m = ceil_div(M, 32);
    for (int tn = 1; tn <= 4; tn *= 2)
        if (tiles_m * ceil_div(N, 32 * tn) <= cus) return tn;
    return 0;
}
constexpr int kSliceLayerTail = 4096;      // columns of the table in LDS (16 KB)

// Whether an instance of launch_slice_layer takes the shape: a tile, 32-bit offsets, and the LDS of the tile's instance (the
// wider two have room for 4088 columns of the table).
static bool slice_layer_fits(int tile, int C, int g, int s, int64_t ldx) {
    const int64_t K = (int64_t)C * g, tail = round_up((int64_t)(C + s) * g, 64) - K / 64 * 64, pitch = (int64_t)1 << 23;
    if (ldx >= pitch || K >= pitch || tail > kSliceLayerTail) return false;
    switch (tile) {
        case 1: return slice_layer_lds<1, 8, 3, true>(tail) <= kWholeKMaxLds;
        case 2: return slice_layer_lds<2, 8, 3, true>(tail) <= kWholeKMaxLds;
        case 4: return slice_layer_lds<4, 8, 2, false>(tail) <= kWholeKMaxLds;
        default: return false;
    }
}

// Where the one launch is ahead of the two.  A workgroup draws and quantizes its rows of X again, and gathers the appended columns
// value by value, each step of them past a wave's first waiting for its requests: both grow with the size, what the launch saves
// does not.  A launch less saves 3 us of the host's time, so the line lies higher where the host launches than in a captured graph.
// Two launches / one, the ratio: a graph on inputs outside the caches; a graph on the same input again; passes launched one after
// the other (the range over static grid and per batch, 10 to 4000 outputs, copies 5 % of the channels):
//   values of X in a row of tiles  8192: 0.98-1.30, 1.07-1.25, 1.29-1.50; 12288: 1.02-1.20, 1.04-1.22, 1.36-1.49; 16384: 0.89-1.06,
//                0.95-1.12, 1.18-1.49; 24576: 0.81-1.05, 0.93-1.11, 1.12-1.49; 32000: 0.62-0.97, 0.77-1.08, 0.74-1.39
//   tiles of 128 columns           8192: 1.10-1.13, 1.11-1.18, 1.28-1.38; 12800: 0.99-1.22, 0.98-1.36, 1.11-1.49; 16384: 0.86-1.15,
//                0.91-1.28, 1.04-1.40; 20480: 0.88-1.24, 0.94-1.37, 1.03-1.40; 22528: 0.87-1.17, 0.91-1.24, 0.99-1.37; 24576: 0.80, 0.91, 0.99
//   a row of K = 4000: 0.97-1.15, 1.09-1.20, 1.29; 6000: 0.89-1.14, 1.01-1.19, 1.04; 8000: 0.84, 1.00, 1.01; 16000: 0.71, 0.83, 0.85
//   copies, 8192 values: half of the channels 1.02, 1.04, 1.36, all of them 0.85, 0.86, 1.24 (tiles of 128 columns 0.96, 0.97, 1.25
//                and 0.92, 0.92, 1.16); 12288: a quarter 0.90, 1.00, 1.22, half 0.88, 0.93, 1.12; four steps of them for a wave
//                (2000 to 2048 columns) 0.77, 0.78, 0.91, eight 0.64, 0.55, 0.58
// So an appended column counts as two, and a wave has at most two steps of them.
SliceLayerPays slice_layer_pays(int64_t M, int C, int g, int s, int64_t N, int64_t ldx) {
    const int64_t K = (int64_t)C * g, rows = M < 32 ? M : 32, values = rows * (K + 2 * (int64_t)s * g);
    const int mode = tuning().slice_layer;
    if (mode == 0 || (mode < 0 && values > 27648)) return {false, false};
    const int tile = slice_layer_tile(M, N);
    if (!slice_layer_fits(tile, C, g, s, ldx)) return {false, false};
    if (mode > 0) return {true, true};
    if (round_up((int64_t)(C + s) * g, 64) - K / 64 * 64 > 1024) return {false, false};
    return {values <= (tile == 4 ? 22528 : 27648) && K <= 6144, values <= (tile == 4 ? 10240 : 13312) && K <= 4096};
}

hipError_t launch_slice_layer(const float* X, int64_t ldx, int64_t M, int C, int g, int s, const int32_t* chan_src,
                              const float* thr, int n_max, int64_t self, float clip, float qmax, int8_t* Xq, int64_t ldq,
                              float* scale_x, const int8_t* Wq, int64_t ldw, int64_t N, const float* scale_w,
                              int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream) {
    SliceLayer p;
    p.X = X; p.ldx = ldx; p.M = (int)M; p.N = (int)N;
    p.K = C * g; p.C = C; p.g = g; p.Kexp = (C + s) * g;
    p.chan_src = chan_src; p.thr = thr; p.n_max = n_max; p.self = self; p.clip = clip; p.qmax = qmax;
    p.Xq = Xq; p.ldq = ldq; p.scale_x = scale_x; p.Wq = Wq; p.ldw = ldw; p.scale_w = scale_w;
    p.acc_out = acc_out; p.ldacc = ldacc; p.Y = Y; p.ldy = ldy;
    p.ksteps = (int)ceil_div(p.Kexp, 64);
    p.kmain = p.K / 64;
    const int rows = (int)(M < 32 ? M : 32);
    switch (slice_layer_tile(M, N)) {
        case 1:
            if (rows <= 8) return run_slice_layer<1, 2, 8, 3, true>(p, stream);
            if (rows <= 16) return run_slice_layer<1, 4, 8, 3, true>(p, stream);
            if (rows <= 24) return run_slice_layer<1, 6, 8, 3, true>(p, stream);
            return run_slice_layer<1, 8, 8, 3, true>(p, stream);
        case 2: return run_slice_layer<2, 8, 8, 3, true>(p, stream);
        case 4: return run_slice_layer<4, 8, 8, 2, false>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int NBUF, bool MASK = false>
static hipError_t run_dma(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw, int64_t M,
                          int64_t N, int64_t Kpad, const float* scale_x, const float* scale_w,
                          int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy,
                          hipStream_t stream, const Requant& rq) {
    // without MASK the kernel walks whole K-steps of every row
    if (!MASK && (ldx < Kpad || ldw < Kpad)) return hipErrorInvalidValue;
    // the kernel clamps its K index to ksteps - 1: it must never be launched with no K-step
    if (Kpad < BK || Kpad % BK != 0) return hipErrorInvalidValue;
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;   // one workgroup per tile: grid.x
    // A single round of 256 x 128 tiles gains nothing from stores without bounds and pays for the code of both forms
    // (1x1 1024 -> 256 at 25088 rows, both launches, 40.17 against 40.30 us, LSTM gates at 700 rows 29.06 against 29.25); in
    // several rounds they hide behind the next tile (100000 x 512 x 500 65.3 with, 63.6 without, 40000 x 256 x 1500 32.6 / 31.2).
    constexpr bool BOTH = BM == 256 && BN == 128 && BK == 128 && !MASK;
    const auto plain = BOTH && total <= compute_units() ? qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, false, false, false, MASK, BOTH>
                                                        : qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, false, false, false, MASK>;
    const auto kernel = rq.Yq != nullptr ? qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, true, false, false, MASK> : plain;
    return launch_kernel(kTimeGemm, kernel,
                         dim3((unsigned)total), dim3(WAVES_M * WAVES_N * 64), 0, stream, Xq, ldx, Wq, ldw, (int)M,
                         (int)N, (int)(Kpad / BK), scale_x, scale_w, acc_out, ldacc, Y, ldy,
                         (int)tiles_n, (unsigned)total, ConvGeom{}, rq, SplitK{});
}

// Arrival counters of the K split: part of the library's device image (zero when the module is
// loaded, and every launch leaves the counters it used at zero again), one copy per GPU.  A launch
// takes one slot of kSplitSlotTiles counters, slots handed out in turn, so that launches on
// different streams do not share counters unless more than kSplitSlots of them are in flight on
// one GPU.  In host code the array's name is only a handle: the device address is looked up once
// per device and only that address goes to a launch.
constexpr int kSplitSlotTiles = 128;
constexpr int kSplitSlots = 512;
static __device__ unsigned splitk_counters[kSplitSlotTiles * kSplitSlots];

static hipError_t splitk_counter_slot(unsigned** out) {
    static std::atomic<unsigned*> addr[kMaxDevices];
    static std::atomic<unsigned> cursor[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    unsigned* p = addr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        void* sym = nullptr;
        e = hipGetSymbolAddress(&sym, HIP_SYMBOL(splitk_counters));
        if (e != hipSuccess) return e;
        if (sym == nullptr) return hipErrorInvalidSymbol;
        p = static_cast<unsigned*>(sym);
        addr[dev].store(p, std::memory_order_release);
    }
    const unsigned slot = cursor[dev].fetch_add(1u, std::memory_order_relaxed) % (unsigned)kSplitSlots;
    *out = p + (size_t)slot * kSplitSlotTiles;
    return hipSuccess;
}

// The split kernel's tile is 256 x 256 (64-byte K-steps, ring of four).
constexpr int kSplitBM = 256, kSplitBN = 256;

// 0 when the shape cannot be split this way (more tiles than a counter slot holds, or fewer than
// one K-step per part).
size_t qgemm_split_workspace_bytes(int64_t M, int64_t N, int64_t Kpad, int parts) {
    const int64_t tiles = ceil_div(M, kSplitBM) * ceil_div(N, kSplitBN);
    if (parts < 2 || parts > 16 || tiles > kSplitSlotTiles || Kpad / 64 < parts) return 0;
    return (size_t)tiles * parts * kSplitBM * kSplitBN * sizeof(int32_t);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int NBUF>
static hipError_t run_dma_split(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw, int64_t M,
                                int64_t N, int64_t Kpad, const float* scale_x, const float* scale_w,
                                int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream,
                                const Requant& rq, int parts, void* partials) {
    if (Kpad < BK || Kpad % BK != 0 || parts < 2 || Kpad / BK < parts) return hipErrorInvalidValue;
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > kSplitSlotTiles) return hipErrorInvalidValue;
    SplitK sk;
    sk.partials = static_cast<int32_t*>(partials);
    sk.parts = parts;
    hipError_t e = splitk_counter_slot(&sk.counters);
    if (e != hipSuccess) return e;
    return launch_kernel(kTimeGemm, qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, false, false, true>,
                         dim3((unsigned)(total * parts)), dim3(WAVES_M * WAVES_N * 64), 0, stream, Xq, ldx, Wq,
                         ldw, (int)M, (int)N, (int)(Kpad / BK), scale_x, scale_w, acc_out, ldacc, Y, ldy,
                         (int)tiles_n, (unsigned)total, ConvGeom{}, rq, sk);
}

// The same kernel with the lowering of a convolution done by its A-operand loader.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NBUF>
static hipError_t run_dma_conv(const int8_t* Aq, const int8_t* Wt, int64_t ldw, int64_t M, int64_t N,
                               int64_t Kpad, const ConvGeom& cg, const float* scale_x,
                               const float* scale_w, int32_t* acc_out, int64_t ldacc, float* Y,
                               int64_t ldy, hipStream_t stream, const Requant& rq) {
    constexpr int BK = 64;
    if (Kpad < BK || Kpad % BK != 0 || cg.ldc % 16 != 0 || cg.cpp < 1) return hipErrorInvalidValue;
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;   // one workgroup per tile: grid.x
    const auto kernel = rq.Yq != nullptr ? qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, true, true>
                                         : qgemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, BK, NBUF, false, true>;
    return launch_kernel(kTimeGemm, kernel,
                         dim3((unsigned)total), dim3(WAVES_M * WAVES_N * 64), 0, stream, Aq, cg.ldc, Wt,
                         ldw, (int)M, (int)N, (int)(Kpad / BK), scale_x, scale_w, acc_out, ldacc, Y,
                         ldy, (int)tiles_n, (unsigned)total, cg, rq, SplitK{});
}

// The convolution whose taps are read from one run of pixels in LDS: unit stride, output of the input's
// size, at least two 16-byte pieces per pixel.  LDS = the run, 16 zero bytes, the ring of weight steps, the
// table of the next layer's copies.
struct PatchPlan {
    int P16 = 0, pixels = 0, ring_off = 0, dup_off = 0;
    int64_t lds = 0;
};
template <int BM, int BN, int NW, int NBUF>
static PatchPlan patch_plan(int W, int pad, int cpp, const Requant& rq) {
    PatchPlan p;
    const int64_t pixels = (int64_t)BM + 2 * (int64_t)pad * (W + 1), P16 = cpp | 1;
    if (pixels * P16 * 16 > kWholeKMaxLds) return p;              // lds == 0: does not fit
    p.P16 = (int)P16;
    p.pixels = (int)pixels;
    p.ring_off = (int)(round_up(pixels * P16, 64) * 16 + 1024);   // whole requests, then a block that ends in the zeros
    int64_t lds = (int64_t)p.ring_off + NBUF * BN * 128;
    const int64_t staging = (int64_t)NW * stage_bytes<true, BN, 8>() > (int64_t)NW * stage_bytes<false, BN, 8>()
                                ? (int64_t)NW * stage_bytes<true, BN, 8>() : (int64_t)NW * stage_bytes<false, BN, 8>();
    if (lds < staging) lds = staging;
    if (rq.Yq != nullptr && rq.s_next > 0) {
        p.dup_off = (int)lds;
        lds += (kDupCap + 1) * 4;
    }
    if (lds <= kWholeKMaxLds) p.lds = lds;
    return p;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NBUF, bool RQ>
static hipError_t run_patch(const int8_t* Aq, const int8_t* Wt, int64_t ldw, int64_t M, int64_t N, const ConvGeom& cg,
                            const PatchPlan& p, const float* scale_x, const float* scale_w, int32_t* acc_out,
                            int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream, const Requant& rq) {
    if (p.lds <= 0 || p.lds > kWholeKMaxLds || cg.cpp < 2 || cg.kh != cg.kw || cg.kh * cg.kw > kPatchMaxTaps)
        return hipErrorInvalidValue;
    if (p.lds > 65536) {
        static std::atomic<bool> opted_in[kMaxDevices];
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&qconv_patch_kernel<BM, BN, WAVES_M, WAVES_N, NBUF, RQ>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWholeKMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    const int64_t tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;   // one workgroup per tile: grid.x
    const int ksteps = (int)ceil_div((int64_t)cg.kh * cg.kw * cg.ldc, 128);
    const unsigned magic = (unsigned)((((uint64_t)1) << 32) / (uint64_t)p.P16);   // P16 >= 3
    return launch_kernel(kTimeGemm, qconv_patch_kernel<BM, BN, WAVES_M, WAVES_N, NBUF, RQ>, dim3((unsigned)total),
                         dim3(WAVES_M * WAVES_N * 64), (unsigned)p.lds, stream, Aq, Wt, ldw, (int)M, (int)N, ksteps,
                         cg.H, cg.W, cg.kw, cg.pad, cg.cpp, p.P16, magic, p.pixels, scale_x, scale_w, acc_out, ldacc, Y,
                         ldy, (int)tiles_n, (unsigned)total, p.ring_off, p.dup_off, rq);
}

// Whether the run's 256 x 128 tile is ahead of the 128 x 128 ring tile: at most one per compute unit, most of the units
// busy, and taps of enough 16-byte pieces (cpp) that the address arithmetic per tap weighs little; an even number of pieces
// takes one more in LDS, an odd one none.  3x3 layers at 14 x 14, 256 outputs, fp32 / codes out, run against ring in us:
//   cpp 17 (256 channels) 170 tiles 23.1 / 25.9 against 25.2 / 27.1, 246 tiles 25.9 / 27.7 against 30.2 / 32.8
//   cpp 13 (190)          150 tiles 19.8 / 22.5 against 21.0 / 22.1, 246 tiles 21.9 / 23.1 against 24.3 / 26.8
//   cpp 16 (240)          170 tiles 21.8 / 24.3 against 20.5 / 22.5, 200 tiles 22.6 / 24.8 against 22.5 / 24.5
//   cpp 9  (128, 28 x 28) 190 tiles 17.2 / 19.3 against 16.4 / 17.6, 245 tiles 18.2 / 20.1 against 18.6 / 20.2
//   cpp 5  (64, 28 x 28)  190 tiles 14.2 / 15.8 against 13.6 / 13.8, 245 tiles 14.5 / 16.2 against 13.4 / 14.5
static bool run_pays(int64_t tiles, int64_t cus, int64_t cpp, int64_t N, bool codes) {
    if (tiles > cus) return false;
    if (cpp < 13) return cpp >= 9 && 20 * tiles >= 19 * cus;
    if (4 * tiles >= 3 * cus) return true;
    if (cpp % 2 == 0 || N % 128 != 0) return false;
    return codes ? (cpp >= 17 ? 9 * tiles >= 5 * cus : 5 * tiles >= 3 * cus) : 2 * tiles > cus;
}

hipError_t launch_qconv(const int8_t* Aq, int64_t ldc, int B, int H, int W, int kh, int kw, int stride,
                        int pad, const int8_t* Wt, int64_t ldw, int64_t N, const float* scale_x,
                        const float* scale_w, int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy,
                        hipStream_t stream, const Requant& rq) {
    ConvGeom cg;
    cg.Ho = (H + 2 * pad - kh) / stride + 1;
    cg.Wo = (W + 2 * pad - kw) / stride + 1;
    cg.H = H;
    cg.W = W;
    cg.kh = kh;
    cg.kw = kw;
    cg.cpp = (int)(ldc / 16);
    cg.stride = stride;
    cg.pad = pad;
    cg.ldc = ldc;
    cg.zero = Wt + N * ldw;            // the row of zeros that follows the N weight rows
    const int64_t M = (int64_t)B * cg.Ho * cg.Wo;
    const int64_t Kpad = ldw;          // kh*kw*ldc rounded up to a whole K-step
    if (Kpad < (int64_t)kh * kw * ldc) return hipErrorInvalidValue;
    int tile = tuning().gemm_tile;
#define OCS_CONV_ARGS Aq, Wt, ldw, M, N, Kpad, cg, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq
#define OCS_PATCH(BM_, BN_, WM_, WN_, NB_)                                                                          \
    do {                                                                                                            \
        const PatchPlan pp = patch_plan<BM_, BN_, WM_ * WN_, NB_>(W, pad, cg.cpp, rq);                              \
        if (pp.lds > 0)                                                                                             \
            return (rq.Yq != nullptr ? run_patch<BM_, BN_, WM_, WN_, NB_, true>                                     \
                                     : run_patch<BM_, BN_, WM_, WN_, NB_, false>)(                                  \
                Aq, Wt, ldw, M, N, cg, pp, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq);                   \
    } while (0)
    if (tile < 0 && kh == 1 && kw == 1 && stride == 1 && pad == 0)
        // nothing to lower: the GEMM's own kernels (what a weight row holds past the pixel's codes is zero)
        return launch_qgemm(Aq, ldc, Wt, ldw, M, N, Kpad, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq);
    // Measured on 3x3 layers (us, ring 128 x 128 of before -> now).  Up to one 64 x 64 tile per compute
    // unit (two, for more than 64 outputs) that ring tile: 2 x 28 x 28 x 128 -> 128 11.8 -> 9.0, 4 x 7 x 7 x 512 -> 512
    // 27.1 -> 20.8.  Up to 64 outputs the run in LDS: 32 x 56 x 56 x 64 -> 64 19.7 -> 13.8 (fp32 out), 24.7 -> 16.5
    // (codes out), with 256 rows a tile once that gives every compute unit one, 128 below (16 images: 13.5 -> 10.9);
    // 256 as well where the run of 128 rows is so long that a compute unit holds one workgroup and there are more
    // of them than units (16 x 56 x 56 x 256 -> 64 ring 23.2, 128 rows 24.9, 256 rows 19.0; where those do not fit, the ring).
    // More outputs: the run's tile of 256 x 128 where run_pays() says so, else the ring.
    const int64_t cus = compute_units();
    const bool patch = stride == 1 && kh == kw && kh == 2 * pad + 1 && kh * kw <= kPatchMaxTaps && cg.cpp >= 2;
    if (tile < 0) {
        const int64_t t64 = ceil_div(M, 64) * ceil_div(N, 64), t256 = ceil_div(M, 256) * ceil_div(N, 128);
        if (t64 <= (N <= 64 ? cus : 2 * cus)) tile = 7;
        else if (patch && N <= 64) {
            const bool one_each = 2 * patch_plan<128, 64, 8, 3>(W, pad, cg.cpp, rq).lds > kWholeKMaxLds;
            tile = ceil_div(M, 256) >= cus || (one_each && ceil_div(M, 128) > cus) ? 31 : 30;
        }
        else if (patch && run_pays(t256, cus, cg.cpp, N, rq.Yq != nullptr)) tile = 32;
    }
    if (patch) {       // (a run too long for LDS: the ring)
        if (tile == 30) OCS_PATCH(128, 64, 4, 2, 3);
        if (tile == 31) OCS_PATCH(256, 64, 4, 2, 3);
        if (tile == 32) OCS_PATCH(256, 128, 4, 2, 3);
    }
    if (tile >= 30) tile = -1;
#undef OCS_PATCH
    // measured on the stem and the 3x3 layers of the paper's networks: the 128x128 ring tile is level
    // with or ahead of the larger ones (the loader's per-lane tap bookkeeping grows with the rows
    // a lane loads; a 128-byte K-step, which doubles them, was 15-90 % slower) and, from 64
    // output channels on, ahead of the 128x64 one as well
    if (tile < 0) tile = N < 64 ? 6 : 9;
    switch (tile) {
        case 6: return run_dma_conv<128, 64, 2, 2, 6>(OCS_CONV_ARGS);
        case 7: return run_dma_conv<64, 64, 2, 2, 6>(OCS_CONV_ARGS);
        case 10: return run_dma_conv<256, 128, 4, 2, 4>(OCS_CONV_ARGS);
        case 12: return run_dma_conv<256, 256, 2, 4, 4>(OCS_CONV_ARGS);
        default: return run_dma_conv<128, 128, 4, 2, 4>(OCS_CONV_ARGS);
    }
#undef OCS_CONV_ARGS
}

// Channel-major codes [N, ldq] (column j*g + t) -> tap-major [N + 1, ldt] (column t*ldc + j,
// zero for j >= E and for columns past g*ldc), the extra row all zeros.  One lane per byte quad.
__global__ __launch_bounds__(kThreads) void tap_major_kernel(const int8_t* __restrict__ Wq, int64_t ldq,
                                                             int64_t N, int E, int g, int64_t ldc,
                                                             int64_t ldt, int8_t* __restrict__ Wt) {
    const int64_t quads_per_row = ldt / 4;
    const int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (o >= (N + 1) * quads_per_row) return;
    const int64_t n = o / quads_per_row;
    const int64_t k = (o - n * quads_per_row) * 4;     // ldc % 4 == 0: a quad stays inside one tap
    const int t = (int)(k / ldc);
    const int j0 = (int)(k - (int64_t)t * ldc);
    unsigned packed = 0;
    if (n < N && t < g) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = j0 + e;
            const int code = j < E ? Wq[n * ldq + (int64_t)j * g + t] : 0;
            packed |= ((unsigned)code & 0xFFu) << (8 * e);
        }
    }
    reinterpret_cast<unsigned*>(Wt)[o] = packed;
}

hipError_t launch_tap_major(const int8_t* Wq, int64_t ldq, int64_t N, int E, int g, int64_t ldc,
                            int8_t* Wt, hipStream_t stream) {
    const int64_t ldt = round_up((int64_t)g * ldc, 64);
    const int64_t total = (N + 1) * (ldt / 4);
    if (ceil_div(total, kThreads) > 0x7FFFFFFF) return hipErrorInvalidValue;   // one lane per byte quad: grid.x
    tap_major_kernel<<<dim3((unsigned)ceil_div(total, kThreads)), kThreads, 0, stream>>>(Wq, ldq, N, E, g,
                                                                                       ldc, ldt, Wt);
    return hipGetLastError();
}

#define OCS_GEMM_ARGS Xq, ldx, Wq, ldw, M, N, Kpad, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq
#define OCS_GEMM_ARGS128 Xq, ldx, Wq, ldw, M, N, K128, scale_x, scale_w, acc_out, ldacc, Y, ldy, stream, rq

hipError_t launch_qgemm(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw, int64_t M,
                        int64_t N, int64_t Kpad, const float* scale_x, const float* scale_w,
                        int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy,
                        hipStream_t stream, const Requant& rq) {
    int tile = tuning().gemm_tile;
    if (tile < 0) {
        // Too few tiles for the chip: the smallest tiles that still give every compute unit at most one
        // workgroup, with K dealt over its waves; with 64 x 64 tiles and a long K the ring kernel's waves
        // share their fragments and its four workgroups' worth of look-ahead wins.  Launched one after
        // the other (a launch that does nothing takes 2.9 us this way), against what the rules below
        // pick: 20 x 6000 x 3150 10.2 -> 6.3 us, 64 x 256 x 269 4.9 -> 3.1, 700 x 256 x 2420 9.4 -> 4.4,
        // 1500 x 256 x 2420 10.2 -> 5.5, 64 x 6000 x 3150 11.6 -> 8.1, 1000 x 512 x 4842 18.0 -> 10.4,
        // 3000 x 256 x 269 5.4 -> 4.7, 3000 x 256 x 2420 11.0 -> 8.3 (ring), 12544 x 64 x 600 5.5 -> 4.3
        // (ring).  Beyond one workgroup per compute unit the next larger tile is ahead every time.
        const int64_t cus = compute_units();
        const int64_t t3264 = ceil_div(M, 32) * ceil_div(N, 64), t6432 = ceil_div(M, 64) * ceil_div(N, 32);
        if (ceil_div(M, 32) * ceil_div(N, 32) <= cus) tile = 26;
        else if (t3264 <= cus || t6432 <= cus) tile = t6432 < t3264 ? 28 : 27;
        else if (ceil_div(M, 64) * ceil_div(N, 64) <= cus) tile = Kpad <= 320 ? 29 : 7;
    }
    // A pitch that is not a whole number of 64-byte K-steps, or shorter than the K extent rounded
    // up to one (allowed up to 320 bytes of K), is something only the whole-K kernel and the sliced ones walk.
    const bool ring_ok = ldx % 64 == 0 && ldw % 64 == 0 && ldx >= Kpad && ldw >= Kpad;
    if (!ring_ok && !(tile >= 26 && tile <= 29) && Kpad > 320) {
        // (a 1x1 convolution on pixels of any number of 16-byte pieces: the ring tiles that check every
        // request against the pitch)
        const int64_t K128 = round_up(Kpad, 128);
        if (tile == 7) return run_dma<64, 64, 2, 2, 64, 6, true>(OCS_GEMM_ARGS);
        if (N <= 64) return run_dma<128, 64, 2, 2, 128, 3, true>(OCS_GEMM_ARGS128);
        if (ceil_div(M, 256) * ceil_div(N, 128) >= 128) return run_dma<256, 128, 4, 2, 128, 3, true>(OCS_GEMM_ARGS128);
        return run_dma<128, 128, 4, 2, 128, 3, true>(OCS_GEMM_ARGS128);
    }
    if (!ring_ok && Kpad <= 320) {
        // (the 128 x 128 ring variant checks its requests against the pitch for this case: a very
        // wide N is better served by the ring kernel's tile order, see below)
        if (tile == 9 || (tile < 0 && N >= 1024))
            return run_dma<128, 128, 4, 2, 64, 4, true>(OCS_GEMM_ARGS);
        if (tile != 16 && tile != 17 && tile != 18 && tile != 19 && !(tile >= 26 && tile <= 29)) tile = N <= 64 ? 17 : (N >= 512 ? (Kpad <= 192 ? 17 : 19) : 16);
    }
    if (tile < 0) {
        // Measured on MI355X over the layer shapes of the paper's networks.  What a CU can draw is
        // set by the line requests its L1 can have outstanding times their latency, so requests
        // count, not bytes: the largest tile that still gives most CUs a workgroup wins, a K-step
        // of one whole 128-byte line per row beats two half-line steps, and workgroups of 8 waves
        // beat 4.  Up to 320 bytes of K the layer is a stream of output rows and the whole-K kernel
        // wins (1.2-1.5x), except that a very wide N is better served by the ring kernel's tile
        // order (one L2 fill of an X row panel for all its N tiles).  With N >= 256 and enough
        // tiles, 256 columns per tile halve the reads of X.
        const int64_t t256 = ceil_div(M, 256) * ceil_div(N, 128);
        const int64_t t256sq = ceil_div(M, 256) * ceil_div(N, 256);
        if (Kpad <= 320) tile = N <= 64 ? 17 : (N >= 1024 ? 9 : (N >= 512 ? (Kpad <= 192 ? 17 : 19) : 16));   // (512 outputs from
                                        // 128 channels: the 128 x 64 tile, 70 against 83 us at M = 200,704)
        else if (N <= 64) tile = 24;    // 128 x 64 with whole-line (128-byte) K-steps: 134 against 155 us on
                                        // the 64 -> 64 3x3 layers at M = 802,816
        else if (Kpad >= 1024) {
            // Long K: rounds of the chip times what a tile costs.  A compute unit holds one workgroup of any of
            // these tiles, so the launch takes as many rounds as tiles / compute units, rounded up; a 256 x 256
            // tile takes 1.75 times as long as a 256 x 128 one, a 128 x 128 one 0.6 times (inside the pass, us:
            // 2000 x 2000 x 2000 22.4 -> 17.9 with 256 of the small ones; 6000 x 3000 x 3000 112 -> 94 with three
            // rounds of the middle ones instead of two of the large; 25088 x 256 x 1076 40.6 / 41.7 / 46.5, 50176 x 256
            // x 1076 78 / 81 / 76, 12544 x 256 x 2358 62 / 58 / 77 for middle / small / large).
            const int64_t t128 = ceil_div(M, 128) * ceil_div(N, 128), t192 = ceil_div(M, 192) * ceil_div(N, 128), cus = compute_units();
            const int64_t large = 35 * ceil_div(t256sq, cus), middle = 20 * ceil_div(t256, cus), small = 12 * ceil_div(t128, cus);
            if (N >= 256 && large < middle && large <= small) tile = 12;
            else if (middle <= small && ldx >= round_up(Kpad, 128) && ldw >= round_up(Kpad, 128) && t192 <= cus &&
                     ceil_div(M, 192) * 192 <= ceil_div(M, 256) * 256 &&
                     (32 * t192 <= 29 * cus || Kpad >= (N <= 256 ? 2048 : 1344)))
                // 192 x 128 where that is still one round and walks no more rows: the compute units the middle size leaves
                // idle get a tile, each a quarter smaller (both launches, us: 700 x 6000 x 3150, 188 tiles for 141, 28.8 -> 25.1;
                // 800 x 5000 x 4200 35.2 -> 30.8; 1400 x 3000 x 3150 29.6 -> 26.5; 9000 x 512 x 1076 22.9 -> 21.4; 40000 x 100 x
                // 1575 68.3 -> 67.3; with 576 rows walked for 512, 400 x 8000 x 3150 22.5 -> 23.2).  The tiles together ask for more than
                // the middle size's: where nearly every compute unit has one and K is short, that is what counts, on some chips more than on
                // others (24576 x 256 x 1110 36.6 -> 40.0, another 35.0 -> 34.0; 24576 x 256 x 2397 70 -> 70, 3932 x 1500 x 1260 22.9 -> 24.3,
                // 16181 x 300 x 1257 level; 12167 x 512 x 1396 31.0 -> 30.2, 5729 x 1024 x 1381 23.5 -> 21.8, 22000 x 256 x 1575, 230 tiles,
                // 45.3 -> 45.0)
                tile = 33;
            else if (middle <= small)
                // the middle size as 128 x 256 for a very long K and fewer tiles than compute units: X rows asked for
                // by two tiles, not four (43-46 against 45-47 us on the 512 -> 512 3x3 layers at M = 12544)
                tile = N >= 512 && t256 < cus && Kpad >= 4096 ? 25 : 11;
            else tile = 23;       // 128-byte K-steps when the operands allow them
        }
        else if (N >= 1024) tile = 9;     // (launched alone on cold operands the 256 x 256 tile
                                                         // is ahead here; behind the pass that wrote the codes
                                                         // it is 7-18 % behind)
        else if (N >= 512 && t256sq >= 512) tile = 12;
        else if (t256 >= 128) tile = 11;                 // N = 256 with K below 1024 included (89 against 92 us)
        else tile = 23;   // 128-byte K-steps when the operands allow them
    }
    // A 128-byte K-step needs a K extent that is a multiple of 128.  The extent is the codes
    // rounded up to 64; when both leading dimensions hold 64 bytes more, those are zero padding
    // on both operands (the producers' contract) and the walk may include them.
    const int64_t K128 = round_up(Kpad, 128);
    const bool k128 = K128 == Kpad || (ldx >= K128 && ldw >= K128);
    // Tile variants by id (the dispatcher above picks 7, 9, 11, 12, 16, 17, 19, 23 to 29 or 33, a convolution 30 to 32 as well; the others
    // are kept selectable because the parity tests run every kernel family through them).
    switch (tile) {
        case 6: return run_dma<128, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS);
        case 7: return run_dma<64, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS);
        case 9: return run_dma<128, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);    // 8 waves
        case 10: return run_dma<256, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);   // 8 waves
        case 11: return k128 ? run_dma<256, 128, 4, 2, 128, 3>(OCS_GEMM_ARGS128)  // 8 waves
                             : run_dma<256, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);
        case 12: return run_dma<256, 256, 2, 4, 64, 4>(OCS_GEMM_ARGS);   // 8 waves
        case 14: return run_dma<256, 256, 4, 4, 64, 4>(OCS_GEMM_ARGS);   // 16 waves
        // whole-K variants; a K extent too long for them falls back to a ring variant
#define OCS_WHOLEK(BM_, BN_, WM_, WN_, FALLBACK)                                                   \
    (wholek_lds_bytes<BM_, BN_, WM_, WN_>(N, Kpad, rq) <= kWholeKMaxLds                                   \
         ? run_wholek<BM_, BN_, WM_, WN_>(OCS_GEMM_ARGS)                                            \
         : FALLBACK)
        case 16: return OCS_WHOLEK(128, 128, 4, 2, (run_dma<128, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS)));
        case 17: return OCS_WHOLEK(128, 64, 4, 1, (run_dma<128, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS)));
        case 18: return OCS_WHOLEK(64, 64, 2, 2, (run_dma<64, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS)));
        case 19: return OCS_WHOLEK(128, 256, 2, 4, (run_dma<128, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS)));
#undef OCS_WHOLEK
        case 23: return k128 ? run_dma<128, 128, 4, 2, 128, 3>(OCS_GEMM_ARGS128)
                             : run_dma<128, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);
        case 24: return k128 ? run_dma<128, 64, 2, 2, 128, 3>(OCS_GEMM_ARGS128)
                             : run_dma<128, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS);
        case 25: return k128 ? run_dma<128, 256, 2, 4, 128, 3>(OCS_GEMM_ARGS128)
                             : run_dma<256, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);
        case 33: return k128 ? run_dma<192, 128, 2, 4, 128, 3>(OCS_GEMM_ARGS128) : run_dma<128, 128, 4, 2, 64, 4>(OCS_GEMM_ARGS);
        // K dealt over eight waves; any pitch
        case 26: return run_slice<1, 1, 8, 4>(OCS_GEMM_ARGS);    // 32 x 32
        case 27: return run_slice<1, 2, 8, 3>(OCS_GEMM_ARGS);    // 32 x 64
        case 28: return run_slice<2, 1, 8, 3>(OCS_GEMM_ARGS);    // 64 x 32
        case 29: return run_slice<2, 2, 8, 2>(OCS_GEMM_ARGS);    // 64 x 64
        default: return run_dma<64, 64, 2, 2, 64, 6>(OCS_GEMM_ARGS);
    }
}

hipError_t launch_qgemm_split(const int8_t* Xq, int64_t ldx, const int8_t* Wq, int64_t ldw, int64_t M,
                              int64_t N, int64_t Kpad, const float* scale_x, const float* scale_w,
                              int32_t* acc_out, int64_t ldacc, float* Y, int64_t ldy, hipStream_t stream,
                              int parts, void* partials) {
    return run_dma_split<kSplitBM, kSplitBN, 2, 4, 64, 4>(Xq, ldx, Wq, ldw, M, N, Kpad, scale_x, scale_w,
                                                         acc_out, ldacc, Y, ldy, stream, Requant{}, parts,
                                                         partials);
}

}  // namespace ocs
