// libhot: one sampled Bayesian linear layer with the weight draw fused into the contraction
// (arxiv 2604.04736, Algorithm 1 / 2: reparameterisation line followed by ForwardPass, for the
// case that the layer is a Linear):
//     y_s = x (mu_W + sigma_W (.) eps_s)^T + (mu_b + sigma_b (.) eps_s^b)        for every local sample s
// The sampled weights do not exist in memory (but for the bf16 pieces that a caller's workspace may hold at many rows,
// linear_planes.h): a wave draws the eps of a 16-output x 32-input tile
// in registers (Philox + Box-Muller on the vector ALU), forms w = fma(sigma, eps, mu) and feeds
// it straight to the matrix cores as the B operand of v_mfma_f32_16x16x4_f32, while the minibatch
// x is the A operand.  mu_W and sigma_W are read once per block of rows and sample chunk; eps for
// weight (o, k) is the draw of flat parameter index weight_offset + o*K + k, i.e. exactly the value
// hot_forward_rng would put into w for the same hot_rng.
//
// Lane roles inside a wave (MFMA 16x16x4: lane l supplies A[m = l%16][kk = l/16] and
// B[kk = l/16][n = l%16], and receives D[4*(l/16) + r][l%16] in register r): lane (j, n) owns the
// eight consecutive inputs k = kb + 8j .. kb + 8j + 7 of output column n (two draws of four), and,
// as an A lane, the same eight inputs of row m = n of x.  MFMA number i of a 32-input block then
// takes element i of every lane's eight: the contraction index is merely enumerated in a different
// order, and every 128-byte line of mu_W, sigma_W and x is consumed by one iteration.
//
// Kernels of this file, by regime:
//   forward   hot_linear_forward_kernel        up to 32 rows, and layers that do not fill the chip: every wave draws what it multiplies
//             hot_linear_forward_rows_kernel   from 256 rows: four waves x 64 rows share every draw through LDS; where neither of the
//                                              next two runs (fewer than 128 inputs, operands beyond their 32-bit offsets)
//             hot_linear_slab_kernel           many rows on layers that fill the chip: 256 to 1024 rows x 32 to 128 outputs per
//                                              workgroup, x loaded straight into LDS, the drawn weights shared through it, bf16 pieces
//                                              on v_mfma_f32_32x32x16_bf16 (128 rows: v_mfma_f32_32x32x2_f32); also input gradients
//             hot_linear_deep_kernel           tens to hundreds of rows, and more where it is faster: a wave holds all rows of its
//                                              workgroup, the waves split the contraction; also the input gradients
//   backward  hot_linear_wgrad_kernel          weight and bias gradients (per-sample G never stored); variants for
//                                              few tiles (waves split the rows), many rows (operands prefetched,
//                                              two output groups per wave), tiles dealt out by XCD
//             hot_linear_wgrad_tile_kernel     the same for large layers: 128 inputs x 128 outputs per workgroup, x and dy
//                                              cut into bf16 pieces once and shared through LDS
//             hot_linear_wgrad_row_parts_kernel  the same for smaller layers and many rows, with a workspace: the rows cut into
//                                              parts, bf16 pieces straight from memory, no LDS before the last sum
//             hot_linear_xgrad_kernel          input gradients where few workgroups are left to it: up to 16 waves split a sum
//             hot_linear_xgrad_rows_kernel     input gradients from 256 rows: shared draws, as in the forward kernel; with a
//                                              workspace from 129 rows on in parts (both where the forward kernels above do not run)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hot.h"
#include "vec.h"
#include "draw.h"

namespace {

constexpr int kMaxWaves = 16;  // waves of a workgroup; they split the input dimension among themselves
constexpr int kColsPerWave = 16;
constexpr int kRowsPerTile = 16;
constexpr int kInputsPerIter = 32;

// More row tiles need more registers per lane: such workgroups are limited to fewer waves.
constexpr int max_waves(int rb) { return rb >= 4 ? 4 : (rb >= 2 ? 8 : kMaxWaves); }

// Four samples' accumulators are live together only where the register file holds them without spills.
constexpr bool four_samples_fit(int rb, bool per_sample_x) { return rb == 2 || (rb == 1 && !per_sample_x); }

// The matrix pipeline writes the registers of an accumulator over several passes after the instruction has
// issued, and only wait states keep a following read from seeing the old value.  The compiler inserts them,
// but left them out where a branch lay between the last matrix instruction and the first read of its result:
// in one kernel variant the register written last came back stale (one row's product missing from one
// column of the weight gradients; found by comparing launch shapes on random layer sizes).  Every run of
// matrix instructions whose results are read next therefore ends here: 32 wait states that the scheduler
// may not move, more than any of these instructions needs.
__device__ __forceinline__ void mfma_results_settle()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// So that no read of a result can be written without those wait states: the accumulator registers of the
// matrix instructions are private to MfmaAcc, which hands them out only against an MfmaSettled, and constructing
// one of those issues the wait states.  Construct it behind the last mac() of a run; one serves all accumulators.
struct MfmaSettled {
    __device__ __forceinline__ MfmaSettled() { mfma_results_settle(); }
    MfmaSettled(const MfmaSettled &) = delete;
    MfmaSettled &operator=(const MfmaSettled &) = delete;
};

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

template <class V, int N>
class MfmaAcc {
    V v_;

public:
    __device__ __forceinline__ MfmaAcc()
    {
#pragma unroll
        for (int i = 0; i < N; ++i) v_[i] = 0.0f;
    }
    // v += a (x) b over the instruction's contraction block
    __device__ __forceinline__ void mac(float a, float b)
    {
        if constexpr (N == 4) v_ = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, v_, 0, 0, 0);
        else v_ = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, v_, 0, 0, 0);
    }
    // the same over sixteen contraction indices of bf16 operands (32 x 32 blocks only)
    __device__ __forceinline__ void mac(bf8 a, bf8 b) { v_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, v_, 0, 0, 0); }
    __device__ __forceinline__ V read(const MfmaSettled &) const { return v_; }
};
typedef MfmaAcc<f4, 4> Acc16x16;        // v_mfma_f32_16x16x4_f32: four result registers per lane
typedef MfmaAcc<f16v, 16> Acc32x32;     // v_mfma_f32_32x32x2_f32: sixteen

__device__ __forceinline__ float pick4_of(f4 v, int c) { return c == 0 ? v[0] : (c == 1 ? v[1] : (c == 2 ? v[2] : v[3])); }

struct LinearArgs {
    long rows, in_features, out_features, ldx;
    long x_sample_stride;   // floats between the inputs of consecutive samples (0: one input for all)
    int s_loc;
    int s_chunk;            // hot_linear_forward_kernel: samples per layer of the grid along z
    long weight_quad0;   // (weight_offset) / 4
    long bias_quad0;     // (bias_offset) / 4
    const float *x, *mu_w, *sigma_w, *mu_b, *sigma_b;
    float *y;
    Rng rng;
};

// A workgroup owns 16 output columns and 16*RB rows; its waves take the 32-input blocks round-robin
// and their partial tiles are added through LDS in wave order (deterministic).  XS: every sample has
// its own input (a layer inside the network); its rows are then loaded per sample, right before
// that sample's draw, whose arithmetic covers their latency.
template <int RB, int ST, bool XS>
__global__ void __launch_bounds__(64 * max_waves(RB), RB >= 4 ? 2 : 1)
hot_linear_forward_kernel(LinearArgs a)
{
    extern __shared__ float partial[];   // [waves - 1][ST * RB * 4][64]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long o = (long)blockIdx.x * kColsPerWave + n;
    const long r0 = (long)blockIdx.y * (kRowsPerTile * RB);
    const bool o_ok = o < O;
    const float *mu_row = a.mu_w + (o_ok ? o : 0) * K;
    const float *sg_row = a.sigma_w + (o_ok ? o : 0) * K;
    const long quad_row = a.weight_quad0 + ((o_ok ? o : 0) * K >> 2);
    // grid z: the samples in chunks of s_chunk (a multiple of ST)
    const int s_lo = (int)blockIdx.z * a.s_chunk, s_hi = s_lo + a.s_chunk < a.s_loc ? s_lo + a.s_chunk : a.s_loc;

    for (int s0 = s_lo; s0 < s_hi; s0 += ST) {
        Acc16x16 mm[ST][RB];

        for (long kb = (long)wave * kInputsPerIter; kb < K; kb += (long)waves * kInputsPerIter) {
            const long k = kb + 8 * j;
            f4 m4[2], sd4[2], xa[RB][2];
            bool ok[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                ok[h] = o_ok && (k + 4 * h < K);
                m4[h] = ok[h] ? load4<true, false>(mu_row + k + 4 * h) : f4{0.0f, 0.0f, 0.0f, 0.0f};
                sd4[h] = ok[h] ? load4<true, false>(sg_row + k + 4 * h) : f4{0.0f, 0.0f, 0.0f, 0.0f};
                if constexpr (!XS) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const long row = r0 + kRowsPerTile * rb + n;
                        xa[rb][h] = (row < R && k + 4 * h < K) ? load4<true, false>(a.x + row * a.ldx + k + 4 * h)
                                                                : f4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                }
            }
#pragma unroll
            for (int st = 0; st < ST; ++st) {
                if (s0 + st < s_hi) {             // uniform over the wave
                    if constexpr (XS) {
                        const float *xs = a.x + (size_t)(s0 + st) * (size_t)a.x_sample_stride;
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) {
                                const long row = r0 + kRowsPerTile * rb + n;
                                xa[rb][h] = (row < R && k + 4 * h < K) ? load4<true, false>(xs + row * a.ldx + k + 4 * h)
                                                                        : f4{0.0f, 0.0f, 0.0f, 0.0f};
                            }
                    }
                    f4 w4[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        w4[h] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                        if (ok[h]) {
                            const f4 e = eps_quad(quad_row + ((k + 4 * h) >> 2), s0 + st, a.rng);
#pragma unroll
                            for (int c = 0; c < 4; ++c) w4[h][c] = __builtin_fmaf(sd4[h][c], e[c], m4[h][c]);
                        }
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb)
                                mm[st][rb].mac(xa[rb][h][c], w4[h][c]);
                }
            }
        }
        const MfmaSettled settled;
        f4 acc[ST][RB];
#pragma unroll
        for (int st = 0; st < ST; ++st)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[st][rb] = mm[st][rb].read(settled);

        if (waves > 1) {
            __syncthreads();            // the previous chunk's readers are done with the buffer
            if (wave > 0) {
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            partial[((wave - 1) * (ST * RB * 4) + (st * RB + rb) * 4 + r) * 64 + lane] = acc[st][rb][r];
            }
            __syncthreads();
            if (wave == 0) {
                for (int v = 1; v < waves; ++v)
#pragma unroll
                    for (int st = 0; st < ST; ++st)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                acc[st][rb][r] += partial[((v - 1) * (ST * RB * 4) + (st * RB + rb) * 4 + r) * 64 + lane];
            }
        }
        if (wave != 0) continue;        // wave 0 holds the complete tile and writes it

#pragma unroll
        for (int st = 0; st < ST; ++st) {
            if (s0 + st < s_hi) {
                float bias = 0.0f;
                if (a.mu_b && o_ok) {
                    const f4 e = eps_quad(a.bias_quad0 + (o >> 2), s0 + st, a.rng);
                    const int c = (int)(o & 3);
                    const float ev = c == 0 ? e[0] : (c == 1 ? e[1] : (c == 2 ? e[2] : e[3]));
                    bias = __builtin_fmaf(a.sigma_b[o], ev, a.mu_b[o]);
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const long row = r0 + kRowsPerTile * rb + 4 * j + r;
                        if (row < R && o_ok) a.y[((size_t)(s0 + st) * (size_t)R + (size_t)row) * (size_t)O + (size_t)o] = acc[st][rb][r] + bias;
                    }
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// The same layer for many rows (hundreds and more: a transformer layer's tokens).  In the kernel above
// every wave draws the weights of its own 16 x 32 tile and uses them for at most 64 rows, so from a few
// hundred rows on the vector ALUs spend more time drawing than the matrix cores multiplying (the two do
// not overlap on this chip).  Here the four waves of a workgroup take 64 rows each (256 rows per
// workgroup) and SHARE every draw through LDS: per iteration of 64 inputs each of the 256 threads draws
// one quad of the 16-output x 64-input weight tile and stores it in LDS; after one barrier every wave
// reads its B operands from there (16-byte reads; the 272-byte row pitch spreads the 16 output rows over
// the banks) and multiplies its own 64 rows: 64 matrix instructions per drawn quad instead of 16.  The
// LDS tile is double-buffered, so one barrier per iteration suffices: a buffer is overwritten two
// iterations later, behind the barrier of the iteration in between, which a wave passes only after it
// has finished reading.  eps, lane roles inside a wave and the order of the contraction index are those
// of the kernel above (MFMA number i of a 32-input block takes element i of every lane's eight inputs).
// ---------------------------------------------------------------------------------
constexpr int kRowsKernelWaves = 4;
constexpr int kRowsKernelRows = 64 * kRowsKernelWaves;   // rows per workgroup
constexpr int kRowsKernelInputs = 64;                    // inputs per iteration: one drawn quad per thread
constexpr int kRowsKernelPitch = kRowsKernelInputs + 4;  // floats per output row of the LDS tile

template <int ST, int NO, bool XS>
__global__ void __launch_bounds__(64 * kRowsKernelWaves)
hot_linear_forward_rows_kernel(LinearArgs a)
{
    // NO column tiles of 16 outputs per workgroup.  More tiles reuse every loaded row of x more often but
    // cost accumulators: with two samples in flight one tile is fastest (86-90 TFLOP/s on 4096^3 and
    // 8192^2 x 1024; two and four tiles leave one wave per SIMD and reach 75-90), a single sample affords two
    // tiles (81 against 64 TFLOP/s).
    __shared__ __attribute__((aligned(16))) float tile[2][ST][NO * 16 * kRowsKernelPitch];
    // x is loaded with consecutive lanes on consecutive addresses (lane (n, j): inputs kb + 4 n .. + 3
    // of a row 4 q + j) and brought into the operand layout (lane (n, j): row n) through a wave's own 32 rows
    // of LDS, half a tile at a time: loading in the operand layout, where every lane of a 16-byte load sits
    // in another row, made the loads of x cost a third of the kernel's time (89 -> 105 TFLOP/s on 4096^3 with
    // the lane pattern alone).
    __shared__ __attribute__((aligned(16))) float turn[kRowsKernelWaves][32 * kRowsKernelPitch];
    static_assert(!XS || ST == 1, "one input per sample: one sample per pass");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long o0 = (long)blockIdx.x * (kColsPerWave * NO);
    const long r0 = (long)blockIdx.y * kRowsKernelRows + (long)wave * 64;
    // as a drawing thread: quad dq of the 16 quads of outputs o0 + dn, o0 + dn + 16, ... in every iteration
    const int dn = (int)threadIdx.x >> 4, dq = (int)threadIdx.x & 15;

    for (int s0 = 0; s0 < a.s_loc; s0 += ST) {
        Acc16x16 mm[ST][4][NO];

        int buf = 0;
        for (long kb = 0; kb < K; kb += kRowsKernelInputs, buf ^= 1) {
            // this wave's rows of x (shared input): row 16 rb + n, inputs kb + 32 blk + 8 j + 4 h .. + 3
            f4 xa[4][2][2];
            f4 xg[4][4];          // as loaded: row 16 rb + 4 q + j, inputs kb + 4 n .. + 3
            {
                const float *xs = XS ? a.x + (size_t)s0 * (size_t)a.x_sample_stride : a.x;     // XS: the pass's one sample
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const long row = r0 + kRowsPerTile * rb + 4 * q + j, k = kb + 4 * n;
                        xg[rb][q] = (row < R && k < K) ? load4<true, false>(xs + row * a.ldx + k) : f4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
            }
            // draw this thread's quads for every sample of the chunk and put them into the tile
            const long kd = kb + 4 * dq;
#pragma unroll
            for (int no = 0; no < NO; ++no) {
                const long o_draw = o0 + 16 * no + dn;
                const bool draw_ok = o_draw < O && kd < K;
                const f4 m4 = draw_ok ? load4<true, false>(a.mu_w + o_draw * K + kd) : f4{0.0f, 0.0f, 0.0f, 0.0f};
                const f4 sd4 = draw_ok ? load4<true, false>(a.sigma_w + o_draw * K + kd) : f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    f4 w4 = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (draw_ok && s0 + st < a.s_loc) {
                        const f4 e = eps_quad(a.weight_quad0 + ((o_draw * K + kd) >> 2), s0 + st, a.rng);
#pragma unroll
                        for (int c = 0; c < 4; ++c) w4[c] = __builtin_fmaf(sd4[c], e[c], m4[c]);
                    }
                    *reinterpret_cast<f4 *>(&tile[buf][st][(16 * no + dn) * kRowsKernelPitch + 4 * dq]) = w4;
                }
            }
            {
                // Two halves of 32 rows through the wave's own LDS rows.  Only this wave touches them and the LDS
                // executes a wave's instructions in order, so no barrier is needed, only the program order.  It
                // happens ahead of the workgroup's barrier: a wave that drew faster turns its x while it would wait.
                float *mine = turn[wave];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
#pragma unroll
                    for (int r2 = 0; r2 < 2; ++r2)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<f4 *>(&mine[(16 * r2 + 4 * q + j) * kRowsKernelPitch + 4 * n]) = xg[2 * half + r2][q];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                    for (int r2 = 0; r2 < 2; ++r2)
#pragma unroll
                        for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                            for (int h = 0; h < 2; ++h)
                                xa[2 * half + r2][blk][h] =
                                    *reinterpret_cast<const f4 *>(&mine[(16 * r2 + n) * kRowsKernelPitch + 32 * blk + 8 * j + 4 * h]);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            }
            __syncthreads();
#pragma unroll
            for (int st = 0; st < ST; ++st) {
                if (s0 + st < a.s_loc) {          // uniform over the workgroup
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int no = 0; no < NO; ++no) {
                                const f4 wq = *reinterpret_cast<const f4 *>(&tile[buf][st][(16 * no + n) * kRowsKernelPitch + 32 * blk + 8 * j + 4 * h]);
#pragma unroll
                                for (int c = 0; c < 4; ++c)
#pragma unroll
                                    for (int rb = 0; rb < 4; ++rb)
                                        mm[st][rb][no].mac(xa[rb][blk][h][c], wq[c]);
                            }
                }
            }
        }
        const MfmaSettled settled;
        f4 acc[ST][4][NO];
#pragma unroll
        for (int st = 0; st < ST; ++st)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int no = 0; no < NO; ++no) acc[st][rb][no] = mm[st][rb][no].read(settled);
        __syncthreads();        // the chunk's last reads are done before the next chunk's first draw lands in buffer 0

#pragma unroll
        for (int st = 0; st < ST; ++st) {
            if (s0 + st < a.s_loc) {
#pragma unroll
                for (int no = 0; no < NO; ++no) {
                    const long o = o0 + 16 * no + n;
                    const bool o_ok = o < O;
                    float bias = 0.0f;
                    if (a.mu_b && o_ok) {
                        const f4 e = eps_quad(a.bias_quad0 + (o >> 2), s0 + st, a.rng);
                        const int c = (int)(o & 3);
                        const float ev = c == 0 ? e[0] : (c == 1 ? e[1] : (c == 2 ? e[2] : e[3]));
                        bias = __builtin_fmaf(a.sigma_b[o], ev, a.mu_b[o]);
                    }
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const long row = r0 + kRowsPerTile * rb + 4 * j + r;
                            if (row < R && o_ok) a.y[((size_t)(s0 + st) * (size_t)R + (size_t)row) * (size_t)O + (size_t)o] = acc[st][rb][no][r] + bias;
                        }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// The same layer for hundreds to thousands of rows.  On this chip the fp32 matrix instructions and the vector ALU do not
// run side by side (the fp32 matrix rate equals the packed fp32 vector rate: the same multipliers serve both; measured
// with the two kinds of work in different waves of one SIMD, the times add), so every cycle spent drawing is lost to
// the contraction, and the share of the draw is 81 / (rows per workgroup): a third at 256 rows, a seventh at 512.  Here
// a workgroup of eight waves owns 512 rows (64 per wave) x 32 to 128 outputs (one of sixteen: 1024 rows x 64 outputs; one
// of four: 256 rows x 32 or 64); per step of 16 contraction indices a thread draws at most ONE quad of the weight tile
// (two samples per pass: the second half of the drawing threads takes the second sample).
// x never passes through registers: each wave sends for the 16 inputs of its own 64 rows with buffer loads that write
// straight into LDS (lane l of an instruction leaves its 16 bytes at the instruction's LDS address + 16 l, zeros for an
// offset outside the window), into a region that only this wave reads, so x needs no barrier at all.  Rows are 64 bytes
// there without padding; so that the operand reads (lane = row, 16 bytes at a fixed input) still spread over all banks,
// the quad q of row r sits at position q ^ swizzle(r) of its row, which the loading lanes arrange by choosing which
// quad of memory they fetch.  The drawn weight tile is shared by the waves and laid out the same way.
// One barrier per step, in its middle.  A step on tile i (buffers i % 2):
//     read the operands of the second half (inputs 8 .. 15) of tile i;  matrix instructions of the first half, whose
//     operands are in registers already;  wait for everything sent for a step ago, barrier (every wave has now read
//     tile i, and tile i + 1 is complete);  draw tile i + 2 into the weight buffer just freed, send for mu, sigma of
//     tile i + 3 (registers) and for x of tile i + 2 (the x region just freed);  matrix instructions of the second half,
//     with the reads of the first-half operands of tile i + 1 issued ahead of their last quarter.
// Behind the barrier nothing waits for LDS or memory: loads have a whole step of matrix instructions to arrive, and
// the first matrix instruction behind it has its operands.  (The kernel this replaces kept both tiles in padded
// LDS arrays filled through registers and met at a barrier at the end of every step, behind which every wave first
// had to read its operands: 105-115 TFLOP/s where this one reaches 130.)
// The matrix instruction is v_mfma_f32_32x32x2_f32: lanes 0-31 hold inputs k .. k + 3 of their row or output, lanes
// 32-63 inputs k + 4 .. k + 7; instruction i takes element i of both operands, so the contraction index is enumerated
// in another order, identically on both sides.  All global accesses go through range-checked windows (see vec.h).
// ---------------------------------------------------------------------------------
constexpr int kComputeUnits = 256;
constexpr int kXcds = 8;
constexpr int kSlabRows = 512;               // rows per workgroup of eight waves (sixteen: twice as many, four: half)
constexpr int kSlabK = 16;                   // contraction indices per step
constexpr unsigned kOutside = 0xFFFFFFF0u;   // a byte offset beyond any window

// (LDS pointers keep their address space through the call: as generic pointers they would become flat accesses)
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f4 lds_f4;
typedef __attribute__((address_space(3))) void lds_void;

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) unsigned short lds_ushort;
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u2 lds_u2;
typedef __attribute__((address_space(3))) bf8 lds_bf8;

// The kernel's products on the bf16 matrix instruction (v_mfma_f32_32x32x16_bf16: sixteen contraction indices in half
// the cycles that v_mfma_f32_32x32x2_f32 takes for two) at the accuracy of fp32: a float is the exact sum of three
// pieces of at most eight significant bits each, x = x1 + x2 + x3 up to 2^-25 |x| (each piece is the remainder rounded
// to bf16, both remainders are exact), each piece is a bf16 number, and a product of two pieces is exact in the fp32
// accumulator.  x w = x1 w1 + (x1 w2 + x2 w1) + (x1 w3 + x2 w2 + x3 w1) + terms below 2^-24 |x w|: six products, summed
// from the smallest on.  The matrix pipe does 6 x 32 = 192 cycles of work per 32 x 32 x 16 block instead of 512.

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

// the pieces of two floats, each piece pair packed in one register (v_cvt_pk_bf16_f32 rounds to nearest even)
__device__ __forceinline__ void split2_bf16(float x0, float x1, unsigned &p1, unsigned &p2, unsigned &p3)
{
    p1 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{x0, x1}, bf2));
    const float r0 = x0 - __builtin_bit_cast(float, p1 << 16), r1 = x1 - __builtin_bit_cast(float, p1 & 0xFFFF0000u);
    p2 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{r0, r1}, bf2));
    const float s0 = r0 - __builtin_bit_cast(float, p2 << 16), s1 = r1 - __builtin_bit_cast(float, p2 & 0xFFFF0000u);
    p3 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{s0, s1}, bf2));
}

// the pieces of eight floats (a then b), packed as the matrix instruction takes them
__device__ __forceinline__ void split8_bf16(const f4 &a, const f4 &b, bf8 &p1, bf8 &p2, bf8 &p3)
{
    u4 q1, q2, q3;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x0 = j < 2 ? a[2 * j] : b[2 * j - 4], x1 = j < 2 ? a[2 * j + 1] : b[2 * j - 3];
        unsigned t1, t2, t3;
        split2_bf16(x0, x1, t1, t2, t3);
        q1[j] = t1;
        q2[j] = t2;
        q3[j] = t3;
    }
    p1 = __builtin_bit_cast(bf8, q1);
    p2 = __builtin_bit_cast(bf8, q2);
    p3 = __builtin_bit_cast(bf8, q3);
}

// What the kernel works on: out_s[row][n] = sum_c in_s[row][c] W_s(n, c) + bias_s[n] with W_s drawn.  Forward (TR = false):
// in = x, c runs over the layer's inputs, n over its outputs, weight (n, c) has flat index n * C + c (the generator's
// quads run along c).  Input gradients (TR = true): in = dy, c runs over the layer's outputs, n over its inputs, weight
// (n, c) has flat index c * N + n (the quads run along n: a drawn quad goes into four rows of the tile), no bias.
struct SlabArgs {
    long rows, contract, outs;   // R, C, N
    long ld_in;                  // pitch of the rows of `in`
    long in_sample_stride;       // floats between the inputs of consecutive samples (0: one input for all)
    int s_begin, s_end;          // the local samples of this launch: workgroups with blockIdx.z = p take those of pass p
    long weight_quad0, bias_quad0;
    const float *in, *mu_w, *sigma_w, *mu_b, *sigma_b;
    float *out;                  // [S_loc, R, N] packed
    Rng rng;
};

__device__ __forceinline__ void everything_arrived_then_barrier()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// position of a row's quads in LDS: quad q of row r (r counted within a block of 16) is stored as quad q ^ slab_swizzle(r);
// any 8 and any 16 consecutive rows then put a given q into different banks
__device__ __forceinline__ int slab_swizzle(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }

// WAVES: 4, 8 or 16 waves of 64 rows each (16: half the draw per row again; their registers then allow 64 outputs and one
// sample; 4: for layers that 512 rows per workgroup fill badly: twice the draw per row, but up to four such workgroups
// share a compute unit, one's matrix instructions covering what the others wait for); CBW: blocks of 32 outputs per
// workgroup (every wave multiplies its 64 rows by all of them); ST samples per pass (they share the input tile); OWN:
// every sample has an input of its own (then ST = 1).
// RBW: blocks of 32 rows per wave; one only with four waves (128 rows per workgroup, for 65 to 128 rows: half the matrix
// work per draw again).
template <int WAVES, int CBW, int ST, bool OWN, bool TR, int RBW = 2, bool BF = (RBW == 2)>
__global__ void __launch_bounds__(64 * WAVES, CBW * ST <= 2 ? (BF && WAVES != 16 ? 3 : 4) : 2)
hot_linear_slab_kernel(SlabArgs a)
{
    static_assert(ST == 1 || ST == 2, "one or two samples per pass");
    static_assert(!OWN || ST == 1, "one input per sample: one sample per pass");
    static_assert(WAVES == 8 || ((WAVES == 16 || WAVES == 4) && CBW * ST <= 2), "sixteen waves have 128 registers each, and so have four: four such workgroups share a compute unit");
    static_assert(RBW == 2 || (RBW == 1 && WAVES == 4), "32 rows per wave only in workgroups of four waves");
    constexpr int WROWS = 32 * RBW, OUTS = 32 * CBW, KS = kSlabK;
    constexpr int XW = WROWS * KS;           // floats of a wave's region of x
    constexpr int WT = OUTS * KS;            // floats of one sample's weight tile
    constexpr int NX = WROWS / 16;           // load instructions per wave and step
    constexpr int QUADS = ST * OUTS * 4;     // quads drawn per step
    constexpr bool EVERY = QUADS == 64 * WAVES;
    static_assert(QUADS <= 64 * WAVES && QUADS % 64 == 0, "whole waves draw");
    __shared__ __attribute__((aligned(16))) float xs0[WAVES * XW], xs1[WAVES * XW];
    // (BF: three planes of bf16 pieces instead of one of floats)
    __shared__ __attribute__((aligned(16))) float ws0[ST * WT * (BF ? 3 : 2) / 2], ws1[ST * WT * (BF ? 3 : 2) / 2];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int C = (int)a.contract, N = (int)a.outs, R = (int)a.rows;
    const int n0 = (int)blockIdx.x * OUTS, r0 = (int)blockIdx.y * (WROWS * WAVES);

    // reading operands: lane (l32, half) holds, for half-step k8, inputs 8 k8 + 4 half .. + 3 of row / output l32 of a block of 32
    int op_off[2];
#pragma unroll
    for (int k8 = 0; k8 < 2; ++k8) op_off[k8] = (l32 >> 4) * 256 + (4 * (l32 & 15) + ((2 * k8 + half) ^ slab_swizzle(l32 & 15))) * 4;

    // loading x: instruction j of a step brings rows 16 j .. 16 j + 15 of this wave's 64, lane l the quad that belongs at position l
    const int lq = (lane & 3) ^ slab_swizzle(lane >> 2);
    const int x_cols = C - 4 * lq;           // this lane's quad exists in the step that starts at cb0 while cb0 < x_cols
    unsigned x_first[NX];
    bool x_ok[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const long row = (long)r0 + wave * WROWS + 16 * j + (lane >> 2);
        x_ok[j] = row < R;
        x_first[j] = (unsigned)((row * a.ld_in + 4 * lq) * 4);
    }
    // drawing: sample d_st of the pass, quad d_idx of the step's tile: outputs n0 + d_n (.. + 3 if TR), contraction
    // indices cb0 + d_c (.. + 3 if not TR)
    const bool draws = t < QUADS;
    const int d_st = t / (OUTS * 4), d_idx = t % (OUTS * 4);
    const int d_n = TR ? 4 * (d_idx % (OUTS / 4)) : d_idx >> 2;
    const int d_c = TR ? d_idx / (OUTS / 4) : 4 * (d_idx & 3);
    const bool d_ok = draws && n0 + d_n < N;
    const int d_cols = C - d_c;
    const long d_flat = TR ? (long)d_c * N + n0 + d_n : (long)(n0 + d_n) * C + d_c;
    const unsigned w_step = TR ? (unsigned)(KS * N * 4) : (unsigned)(KS * 4);      // bytes from one step's quad to the next
    int d_put[TR ? 4 : 1];                   // where the drawn weights go in the tile (floats; BF: bytes within a plane)
    if constexpr (BF) {
        // A plane holds, per sample and output, 32 bytes: two chunks of eight bf16, chunk h with the contraction indices
        // 4 h .. 4 h + 3 and 8 + 4 h .. 8 + 4 h + 3 (what lanes 32 h .. 32 h + 31 feed to one matrix instruction), stored
        // as chunk h ^ bit 3 of the output (so that 16 consecutive outputs spread over all banks).
        const int h = (d_c >> 2) & 1, part = d_c >> 3;
#pragma unroll
        for (int e = 0; e < (TR ? 4 : 1); ++e)
            d_put[e] = (d_st * OUTS + d_n + e) * 32 + ((h ^ (((d_n + e) >> 3) & 1)) << 4) + part * 8 + (TR ? (d_c & 3) * 2 : 0);
    } else if constexpr (!TR) d_put[0] = d_st * WT + (4 * d_n + ((d_c >> 2) ^ slab_swizzle(d_n & 15))) * 4;
    else {
#pragma unroll
        for (int e = 0; e < 4; ++e) d_put[e] = d_st * WT + (4 * (d_n + e) + ((d_c >> 2) ^ slab_swizzle((d_n + e) & 15))) * 4 + (d_c & 3);
    }
    const window_t mu_win = window(a.mu_w, (unsigned)((long)C * N * 4)), sg_win = window(a.sigma_w, (unsigned)((long)C * N * 4));
    const unsigned in_bytes = (unsigned)((((long)R - 1) * a.ld_in + C) * 4);
    lds_float *const X0 = (lds_float *)xs0, *const X1 = (lds_float *)xs1, *const W0 = (lds_float *)ws0, *const W1 = (lds_float *)ws1;

    const int s0 = a.s_begin + (int)blockIdx.z * ST, s_hi = a.s_end;      // this workgroup's pass: samples s0 .. s0 + ST - 1 below s_hi
    {
        const window_t in_win = window(OWN ? a.in + (size_t)s0 * (size_t)a.in_sample_stride : a.in, in_bytes);
        Acc32x32 mm[ST][RBW][CBW];

        unsigned x_off[NX], w_off = (unsigned)(d_flat * 4);
#pragma unroll
        for (int j = 0; j < NX; ++j) x_off[j] = x_first[j];
        long d_quad = a.weight_quad0 + (d_flat >> 2);

        const bool d_live = d_ok && s0 + d_st < s_hi;

        // sends for mu and sigma of this thread's quad of the step that starts at cb0 (every call advances one step)
        f4 m4, sd4;
        auto ask_w = [&](int cb0) {
            const int off = (int)((d_ok && cb0 < d_cols) ? w_off : kOutside);
            m4 = window_load4<false>(mu_win, off);
            sd4 = window_load4<false>(sg_win, off);
            w_off += w_step;
        };
        // draws that quad and puts it into the tile (every call advances one step; zeros beyond the layer's edges)
        auto put_w = [&](int cb0, lds_float *wsb) {
            // (Beyond the layer's edges mu and sigma have arrived as zeros.  Without the inner branch the scheduler may set the draw
            // between matrix instructions; where only some waves draw the branch is faster: sixteen waves, 1024 x 8192^2 forward
            // 1430 against 1495 us, but for the input gradients 1540 against 1480.)
            if (EVERY || draws) {
                f4 w4 = {0.0f, 0.0f, 0.0f, 0.0f};
                if (EVERY || (WAVES == 16 && TR) || (d_live && cb0 < d_cols)) {
                    const f4 e = eps_quad(d_quad, s0 + d_st, a.rng);
#pragma unroll
                    for (int c = 0; c < 4; ++c) w4[c] = __builtin_fmaf(sd4[c], e[c], m4[c]);
                }
                if constexpr (BF) {
                    // three bf16 pieces of every weight (see split2_bf16): a quad along the contraction is 8 bytes per plane
                    unsigned pc[3][2];
                    split2_bf16(w4[0], w4[1], pc[0][0], pc[1][0], pc[2][0]);
                    split2_bf16(w4[2], w4[3], pc[0][1], pc[1][1], pc[2][1]);
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) {
                        lds_char *plane = (lds_char *)wsb + pl * (ST * OUTS * 32);
                        if constexpr (!TR) *(lds_u2 *)(plane + d_put[0]) = u2{pc[pl][0], pc[pl][1]};
                        else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) *(lds_ushort *)(plane + d_put[e]) = (unsigned short)(pc[pl][e >> 1] >> (16 * (e & 1)));
                        }
                    }
                } else if constexpr (!TR) *(lds_f4 *)(wsb + d_put[0]) = w4;
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) wsb[d_put[e]] = w4[e];
                }
                d_quad += TR ? (long)(KS / 4) * N : KS / 4;
            }
        };
        // sends for this wave's rows of the step that starts at cb0, straight into its region of xsb (every call advances one step)
        auto ask_x = [&](int cb0, lds_float *xsb) {
            const bool col_ok = cb0 < x_cols;
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(in_win, (lds_void *)(xsb + wave * XW + j * 256), 16,
                                                         (int)((x_ok[j] && col_ok) ? x_off[j] : kOutside), 0, 0, 0);
                x_off[j] += KS * 4;
            }
        };
        f4 xa[2][RBW], wb[2][ST][CBW];      // operand registers of the two half-steps
        auto read_ops = [&](int k8, const lds_float *xsb, const lds_float *wsb) {
            const volatile lds_f4 *xp = (const volatile lds_f4 *)(xsb + wave * XW + op_off[k8]);
            const volatile lds_f4 *wp = (const volatile lds_f4 *)(wsb + op_off[k8]);
#pragma unroll
            for (int rb = 0; rb < RBW; ++rb) xa[k8][rb] = xp[rb * 128];
            if constexpr (!BF) {
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int cb = 0; cb < CBW; ++cb) wb[k8][st][cb] = wp[(st * WT + cb * 512) / 4];
            }
        };
        auto multiply = [&](int k8, int i0, int i1) {
#pragma unroll
            for (int i = i0; i < i1; ++i)
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
                        for (int cb = 0; cb < CBW; ++cb) mm[st][rb][cb].mac(xa[k8][rb][i], wb[k8][st][cb][i]);
        };
        // BF: one step on the bf16 matrix instruction.  The operands of the step are read (x as floats, the weights
        // as their three planes), x is cut into its pieces, and six products per block of 32 x 32 leave out only the
        // terms below 2^-24 of the full product; then the barrier, behind which the buffers just read are refilled.
        // AHEAD: both row blocks are cut first, every block of weights is read once for the two of them, one block ahead of its
        // products, and consecutive instructions go to different accumulators; it takes 24 to 36 registers more.  Measured:
        // 64 output-samples in four waves 82 -> 77 us (16640 x 192 x 768), 128 in eight 246 -> 218 (7260 x 540 x 2160) and 267 -> 244
        // (its transpose's input gradients), the input gradients of sixteen 1541 -> 1490 (1024 x 8192^2); but the forward call's
        // sixteen waves spill (1439 -> 1488) and narrower tiles of eight, three waves to a SIMD, lose 3 %.
        constexpr bool AHEAD = WAVES == 4 || CBW * ST == 4 || (WAVES == 16 && TR);
        auto read_b = [&](int at, const lds_float *wsb, bf8 (&b)[3]) {      // at = st * CBW + cb
            const volatile lds_bf8 *wp = (const volatile lds_bf8 *)((const lds_char *)wsb + ((at / CBW * OUTS + at % CBW * 32 + l32) * 32 + ((half ^ ((l32 >> 3) & 1)) << 4)));
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) b[pl] = wp[pl * ST * OUTS * 2];
        };
        auto step_bf = [&](int cb0, lds_float *xsb, lds_float *wsb) {
            read_ops(0, xsb, wsb);
            read_ops(1, xsb, wsb);
            if constexpr (AHEAD) {
                constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
                bf8 b[2][3], p[RBW][3];
                read_b(0, wsb, b[0]);
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb) split8_bf16(xa[0][rb], xa[1][rb], p[rb][0], p[rb][1], p[rb][2]);
#pragma unroll
                for (int at = 0; at < ST * CBW; ++at) {
                    if (at + 1 < ST * CBW) read_b(at + 1, wsb, b[(at + 1) & 1]);
#pragma unroll
                    for (int i = 0; i < 6; ++i)
#pragma unroll
                        for (int rb = 0; rb < RBW; ++rb) mm[at / CBW][rb][at % CBW].mac(p[rb][PA[i]], b[at & 1][PB[i]]);
                }
            } else {
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb) {
                    bf8 a1, a2, a3;
                    split8_bf16(xa[0][rb], xa[1][rb], a1, a2, a3);
#pragma unroll
                    for (int st = 0; st < ST; ++st)
#pragma unroll
                        for (int cb = 0; cb < CBW; ++cb) {
                            const volatile lds_bf8 *wp = (const volatile lds_bf8 *)((const lds_char *)wsb + ((st * OUTS + cb * 32 + l32) * 32 + ((half ^ ((l32 >> 3) & 1)) << 4)));
                            const bf8 b1 = wp[0], b2 = wp[ST * OUTS * 2], b3 = wp[2 * ST * OUTS * 2];
                            mm[st][rb][cb].mac(a3, b1);
                            mm[st][rb][cb].mac(a2, b2);
                            mm[st][rb][cb].mac(a1, b3);
                            mm[st][rb][cb].mac(a2, b1);
                            mm[st][rb][cb].mac(a1, b2);
                            mm[st][rb][cb].mac(a1, b1);
                        }
                }
            }
            everything_arrived_then_barrier();
            put_w(cb0 + 2 * KS, wsb);
            ask_w(cb0 + 3 * KS);
            ask_x(cb0 + 2 * KS, xsb);
        };
        auto step = [&](int cb0, lds_float *xsb, lds_float *wsb, const lds_float *xsn, const lds_float *wsn) {
            read_ops(1, xsb, wsb);
            multiply(0, 0, 4);
            everything_arrived_then_barrier();
            put_w(cb0 + 2 * KS, wsb);
            ask_w(cb0 + 3 * KS);
            ask_x(cb0 + 2 * KS, xsb);
            multiply(1, 0, 3);
            read_ops(0, xsn, wsn);
            multiply(1, 3, 4);
        };

        ask_x(0, X0);
        ask_x(KS, X1);
        ask_w(0);
        put_w(0, W0);
        ask_w(KS);
        put_w(KS, W1);
        ask_w(2 * KS);
        everything_arrived_then_barrier();
        if constexpr (BF) {
            for (int cb0 = 0; cb0 < C; cb0 += 2 * KS) {
                step_bf(cb0, X0, W0);
                step_bf(cb0 + KS, X1, W1);
            }
        } else {
            read_ops(0, X0, W0);
            for (int cb0 = 0; cb0 < C; cb0 += 2 * KS) {      // (an odd number of steps is followed by one on zeros)
                step(cb0, X0, W0, X1, W1);
                step(cb0 + KS, X1, W1, X0, W0);
            }
        }
        const MfmaSettled settled;

        // result register i of a 32 x 32 block: row 8 (i / 4) + 4 (lane / 32) + i % 4, column lane % 32
        int r0w = r0 + wave * WROWS + 4 * half, n0l = n0 + l32;
        asm volatile("" : "+v"(r0w), "+v"(n0l));       // (so that the offsets below are formed here, not ahead of the loop)
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            if (s0 + st < s_hi) {
                const window_t out_win = window(a.out + (size_t)(s0 + st) * (size_t)R * (size_t)N, (unsigned)((long)R * N * 4));
#pragma unroll
                for (int cb = 0; cb < CBW; ++cb) {
                    const int n = n0l + 32 * cb;
                    const bool n_ok = n < N;
                    float bias = 0.0f;
                    if (!TR && a.mu_b && n_ok) {
                        const f4 e = eps_quad(a.bias_quad0 + (n >> 2), s0 + st, a.rng);
                        bias = __builtin_fmaf(a.sigma_b[n], pick4_of(e, n & 3), a.mu_b[n]);
                    }
#pragma unroll
                    for (int rb = 0; rb < RBW; ++rb) {
                        const f16v acc = mm[st][rb][cb].read(settled);
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int row = r0w + 32 * rb + 8 * (i >> 2) + (i & 3);
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, acc[i] + bias), out_win,
                                                                  (n_ok && row < R) ? (int)(((unsigned)row * (unsigned)N + (unsigned)n) * 4u) : (int)kOutside, 0, 0);
                        }
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// Tens to hundreds of rows.  The kernel above shares a drawn weight among waves that hold 64 rows each and meet at a barrier
// in every step; with few rows its workgroups are few or its waves idle, and what runs instead draws every weight once per 64 or
// 256 rows, on the fp32 instruction.  Here ONE wave holds all rows of a workgroup (32 RB, 64 to 320) x 32 CB outputs, and the four
// waves take turns on the contraction, 16 indices at a time: every weight is drawn and cut into pieces by one lane, every
// element of x by one lane, nothing is shared, and no wave waits for another before their tiles are added up at the end.
// Products, layouts and lane roles are those of the kernel above (bf16 pieces; x by buffer loads straight into LDS, 64 bytes per
// row, the weights through three planes there), but all of it is the wave's own, so program order and counts of outstanding
// loads replace the barriers.  Per block of 32 rows: the pieces of the next block are cut and a twelfth or so of the next step's
// quads is drawn between the matrix instructions of this one; a block's place in LDS is sent for again, for the next step, as
// soon as its values are in registers.  What bounds it: vector and matrix work, which on this chip overlap only in
// part (256 x 8192^2: 172 TFLOP/s of fp32 work, the library's bf16 product at six products each would do 202), and the last round
// of workgroups.  Two outputs' width (CB = 2) halves the cutting of x per product but leaves one wave per SIMD; RB = 10 with
// CB = 2 does not fit the registers.  RB is even: a block's two operand registers alternate.
// ---------------------------------------------------------------------------------
constexpr int kDeepWaves = 4;
constexpr long kDeepStep = kSlabK * kDeepWaves;     // contraction indices that the waves take together
constexpr unsigned kFarOutside = 0x80000000u;      // a byte offset beyond any window of this kernel, also with a tile's rows added

struct DeepArgs {
    long rows, contract, outs;
    long ld_in, in_sample_stride;
    long contract_per_part;      // multiple of 16 * kDeepWaves
    int parts, n_begin, samples;
    int items, per_xcd;          // tiles of the launch, and per XCD
    long part_stride;            // floats between the parts' outputs
    long weight_quad0, bias_quad0;
    const float *in, *mu_w, *sigma_w, *mu_b, *sigma_b;
    float *out;
    Rng rng;
};

template <int N>
__device__ __forceinline__ void wait_for_all_but()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N < 63 ? N : 63) : "memory");
}

// Philox in pieces (rounds R0 .. R1 - 1 of philox4x32_10), so that a draw can be spread over a loop
template <int R0, int R1>
__device__ __forceinline__ void philox_rounds(u4 &c, unsigned k0, unsigned k1)
{
    constexpr unsigned kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
#pragma unroll
    for (int r = R0; r < R1; ++r) {
        const unsigned long long p0 = (unsigned long long)kM0 * c[0], p1 = (unsigned long long)kM1 * c[2];
        const unsigned n0 = xor3((unsigned)(p1 >> 32), c[1], k0 + (unsigned)r * kW0);
        const unsigned n2 = xor3((unsigned)(p0 >> 32), c[3], k1 + (unsigned)r * kW1);
        c[1] = (unsigned)p1;
        c[3] = (unsigned)p0;
        c[0] = n0;
        c[2] = n2;
    }
}

// An infinite factor, and one beyond the largest bf16 number, has no bf16 pieces: the products of what they give are NaN.  So where
// a sum of the kernel below is NaN (`again`) it is formed again from fp32 products, over the indices c_lo .. c_hi - 1.  First over
// the inputs without pieces alone, which the OUTS lanes of a row look for together: an infinity or NaN among them decides the sum
// (an infinite weight beside an infinite input, which could make it NaN, is not looked for), and few draws are needed (300 x 2160 x 8640 x 2 samples with one infinity in every row 11.9 -> 0.9 ms).  All of it is formed
// only where that leaves it open.  Called by whole waves (in: the row of the lane, also of lanes beyond the outputs).
template <bool TR, int OUTS, class Args>
__device__ __forceinline__ float deep_plain_sum(const Args &a, const float *in, int s, int n, int c_lo, int c_hi, bool again)
{
    auto weight = [&](int c) -> float {
        const long flat = TR ? (long)c * a.outs + n : (long)n * a.contract + c;
        return __builtin_fmaf(a.sigma_w[flat], pick4_of(eps_quad(a.weight_quad0 + (flat >> 2), s, a.rng), (int)(flat & 3)), a.mu_w[flat]);
    };
    constexpr float kMostBf16 = 3.3895313892515355e38f;
    const int lane = threadIdx.x & 63;
    float sum = 0.0f;
#pragma unroll 1
    for (int c = c_lo; c < c_hi; c += 4 * OUTS) {
        const int mine = c + 4 * (lane % OUTS);          // (whole quads: c_lo, c_hi and the rows are multiples of four)
        f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (mine < c_hi) v = load4<true, false>(in + mine);
        const bool has_pieces = __builtin_fabsf(v[0]) <= kMostBf16 && __builtin_fabsf(v[1]) <= kMostBf16 &&
                                __builtin_fabsf(v[2]) <= kMostBf16 && __builtin_fabsf(v[3]) <= kMostBf16;
        unsigned long long quads = __builtin_amdgcn_ballot_w64(!has_pieces);
        if (OUTS == 32) quads = lane & 32 ? quads >> 32 : quads & 0xFFFFFFFFull;
#pragma unroll 1
        for (; again && quads != 0 && sum == sum; quads &= quads - 1) {
            const int q = c + 4 * __builtin_ctzll(quads);
#pragma unroll 1
            for (int i = q; i < q + 4; ++i)
                if (!(__builtin_fabsf(in[i]) <= kMostBf16)) sum = __builtin_fmaf(in[i], weight(i), sum);
        }
        if (__builtin_amdgcn_ballot_w64(again && sum == sum) == 0) break;
    }
    if (!again || sum != sum || __builtin_isinf(sum)) return sum;
    sum = 0.0f;
#pragma unroll 1
    for (int c = c_lo; c < c_hi && sum == sum; ++c) sum = __builtin_fmaf(in[c], weight(c), sum);
    return sum;
}

// (in a file of its own; it uses the windows, the draw, the pieces and the sums above)
}  // namespace
#include "linear_planes.h"
namespace {

template <int RB, int CB, bool TR>
__global__ void __launch_bounds__(64 * kDeepWaves, RB * CB <= 2 ? 4 : RB * CB <= 4 ? 3 : (RB * CB <= 8 ? 2 : 1))
hot_linear_deep_kernel(DeepArgs a)
{
    static_assert(RB % 2 == 0, "the operand registers of a step's last block and of the next step's first differ");
    constexpr int KS = kSlabK, ROWS = 32 * RB, OUTS = 32 * CB, QW = 2 * CB;     // QW: quads a lane draws per step
    constexpr int XW = ROWS * KS, WW = OUTS * KS * 3 / 2;                        // floats of a wave's x and of its three planes of weights
    constexpr int RP = OUTS + 1;                                                 // pitch of a row block on its way out
    constexpr int LDS_LOOP = XW + WW, LDS_OUT = 32 * RP;
    __shared__ __attribute__((aligned(16))) float lds[kDeepWaves * (LDS_LOOP > LDS_OUT ? LDS_LOOP : LDS_OUT)];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int C = (int)a.contract, N = (int)a.outs, R = (int)a.rows;
    // The list of tiles (row blocks fastest, then samples, then parts, then outputs) is cut into one contiguous range per XCD:
    // the workgroups that need the same mu and sigma run at about the same time behind one L2.
    const int row_tiles = (R + ROWS - 1) / ROWS;
    const int item = ((int)blockIdx.x % kXcds) * a.per_xcd + (int)blockIdx.x / kXcds;
    if ((int)blockIdx.x / kXcds >= a.per_xcd || item >= a.items) return;         // the whole workgroup
    const int s = item / row_tiles % a.samples, part = item / (row_tiles * a.samples) % a.parts;
    const int n0 = a.n_begin + item / (row_tiles * a.samples * a.parts) * OUTS, r0 = item % row_tiles * ROWS;
    const int c_lo = part * (int)a.contract_per_part, c_hi = c_lo + (int)a.contract_per_part < C ? c_lo + (int)a.contract_per_part : C;
    lds_float *const X = (lds_float *)lds + wave * LDS_LOOP, *const W = X + XW;

    // operand reads of x: quads half and 2 + half of row l32 of a block
    int op_off[2];
#pragma unroll
    for (int k8 = 0; k8 < 2; ++k8) op_off[k8] = (l32 >> 4) * 256 + (4 * (l32 & 15) + ((2 * k8 + half) ^ slab_swizzle(l32 & 15))) * 4;
    const int wb_off = l32 * 32 + ((half ^ ((l32 >> 3) & 1)) << 4);              // bytes within a plane and block of 32 outputs
    // loads of x: an instruction brings 16 rows x 16 indices
    const int lq = (lane & 3) ^ slab_swizzle(lane >> 2);
    const unsigned in_bytes = (unsigned)((((long)R - 1) * a.ld_in + C) * 4);
    const window_t in_win = window(a.in + (size_t)s * (size_t)a.in_sample_stride, in_bytes);
    const window_t mu_win = window(a.mu_w, (unsigned)((long)C * N * 4)), sg_win = window(a.sigma_w, (unsigned)((long)C * N * 4));
    const int my_row = r0 + (lane >> 2);        // (of the first 16)
    const unsigned x_pitch16 = (unsigned)(16 * a.ld_in * 4);
    const unsigned x_lane = (unsigned)(((long)my_row * a.ld_in + 4 * lq) * 4);

    // drawing.  Not TR: quad i of the lane is output n0 + 16 i + lane / 4, indices 4 (lane % 4) .. + 3 of the step.  TR: outputs
    // n0 + 4 (lane % (8 CB)) .. + 3, index QW (lane / (8 CB)) + i.
    const int d_n = TR ? 4 * (lane % (8 * CB)) : lane >> 2;
    const int d_c = TR ? QW * (lane / (8 * CB)) : 4 * (lane & 3);
    int d_put;
    {
        const int h = (d_c >> 2) & 1, prt = d_c >> 3;
        d_put = d_n * 32 + ((h ^ ((d_n >> 3) & 1)) << 4) + prt * 8 + (TR ? (d_c & 3) * 2 : 0);
    }
    auto d_flat = [&](int i, int cb) -> long {
        return TR ? (long)(cb + d_c + i) * N + n0 + d_n : (long)(n0 + 16 * i + d_n) * C + cb + d_c;
    };
    auto d_ok = [&](int i, int cb) -> bool { return TR ? (n0 + d_n < N && cb + d_c + i < c_hi) : (n0 + 16 * i + d_n < N && cb + d_c < c_hi); };

    f4 m4[QW], sd4[QW];
    auto ask_w = [&](int i, int cb) {
        const int off = (int)(d_ok(i, cb) ? (unsigned)(d_flat(i, cb) * 4) : kOutside);
        m4[i] = window_load4<false>(mu_win, off);
        sd4[i] = window_load4<false>(sg_win, off);
    };
    u4 ph;
    f4 wprev;
    unsigned held[3][4];
    // piece t of the step's drawing: rounds 0-4, rounds 5-9, the rest of quad t / 3; then sends for what the quad needs a step later
    auto draw_piece = [&](int t, int cb) {
        const int i = t / 3;
        if (t % 3 == 0) {
            const long quad = a.weight_quad0 + (d_flat(i, cb) >> 2);
            ph = u4{(unsigned)((unsigned long long)quad & 0xFFFFFFFFull), (unsigned)((unsigned long long)quad >> 32),
                    a.rng.first_sample + (unsigned)s, a.rng.step};
            philox_rounds<0, 5>(ph, a.rng.k0, a.rng.k1);
        } else if (t % 3 == 1) {
            philox_rounds<5, 10>(ph, a.rng.k0, a.rng.k1);
        } else {
            const f4 e = eps_from_words(ph);
            f4 w4;
#pragma unroll
            for (int c = 0; c < 4; ++c) w4[c] = __builtin_fmaf(sd4[i][c], e[c], m4[i][c]);
            if constexpr (!TR) {
                unsigned pc[3][2];
                split2_bf16(w4[0], w4[1], pc[0][0], pc[1][0], pc[2][0]);
                split2_bf16(w4[2], w4[3], pc[0][1], pc[1][1], pc[2][1]);
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *(lds_u2 *)((lds_char *)W + pl * (OUTS * 32) + d_put + i * 16 * 32) = u2{pc[pl][0], pc[pl][1]};
            } else {
                if ((i & 1) == 0) wprev = w4;
                else {
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4) {
                        unsigned p1, p2, p3;
                        split2_bf16(wprev[e4], w4[e4], p1, p2, p3);
                        if constexpr (CB == 2) {
                            if (i == 1) {
                                held[0][e4] = p1;
                                held[1][e4] = p2;
                                held[2][e4] = p3;
                            } else {
                                *(lds_u2 *)((lds_char *)W + 0 * (OUTS * 32) + d_put + e4 * 32) = u2{held[0][e4], p1};
                                *(lds_u2 *)((lds_char *)W + 1 * (OUTS * 32) + d_put + e4 * 32) = u2{held[1][e4], p2};
                                *(lds_u2 *)((lds_char *)W + 2 * (OUTS * 32) + d_put + e4 * 32) = u2{held[2][e4], p3};
                            }
                        } else {
                            typedef __attribute__((address_space(3))) unsigned lds_unsigned;
                            *(lds_unsigned *)((lds_char *)W + 0 * (OUTS * 32) + d_put + e4 * 32) = p1;
                            *(lds_unsigned *)((lds_char *)W + 1 * (OUTS * 32) + d_put + e4 * 32) = p2;
                            *(lds_unsigned *)((lds_char *)W + 2 * (OUTS * 32) + d_put + e4 * 32) = p3;
                        }
                    }
                }
            }
        }
    };
    // sends for block rb of the step that starts at cb
    auto ask_x = [&](int rb, int cb) {
        // (rows beyond the last lie behind the window, which ends with it; indices beyond the part's end are moved there)
        const unsigned base = cb + 4 * lq < c_hi ? x_lane + (unsigned)cb * 4u : kFarOutside;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(in_win, (lds_void *)(X + (2 * rb + j) * 256), 16,
                                                     (int)(base + (unsigned)(2 * rb + j) * x_pitch16), 0, 0, 0);
    };
    auto read_x = [&](int rb, f4 &lo, f4 &hi) {
        lo = *(const volatile lds_f4 *)(X + op_off[0] + rb * 512);
        hi = *(const volatile lds_f4 *)(X + op_off[1] + rb * 512);
    };
    bf8 b[CB][3];
    auto read_w = [&] {
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) b[c][pl] = *(const volatile lds_bf8 *)((const lds_char *)W + pl * (OUTS * 32) + c * 1024 + wb_off);
    };

    Acc32x32 mm[RB][CB];
    const int first = c_lo + KS * wave, stride = KS * kDeepWaves;
    if (first < c_hi) {
#pragma unroll
        for (int i = 0; i < QW; ++i) ask_w(i, first);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) ask_x(rb, first);
#pragma unroll
        for (int t = 0; t < 3 * QW; ++t) draw_piece(t, first);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < QW; ++i) ask_w(i, first + stride);
        wait_for_all_but<0>();
        f4 raw[2][2];
        read_x(0, raw[0][0], raw[0][1]);
        read_x(1 % RB, raw[1][0], raw[1][1]);
        bf8 cur[3], nxt[3];
        asm volatile("" : "+v"(raw[0][0]), "+v"(raw[0][1])::"memory");
        ask_x(0, first + stride);
        split8_bf16(raw[0][0], raw[0][1], cur[0], cur[1], cur[2]);
        for (int cb = first; cb < c_hi; cb += stride) {
            read_w();
            // (the weights of this step are in registers before the next ones overwrite them: the LDS executes a wave's
            // instructions in order)
            asm volatile("" ::: "memory");
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                // here: pieces of block rb in cur; block rb + 1 on its way into raw[(rb + 1) % 2].  Sent for since the two loads of
                // block rb + 2: those of the RB - 1 blocks behind it (and mu, sigma), so that many may be outstanding.
                f4 &lo = raw[(rb + 1) & 1][0], &hi = raw[(rb + 1) & 1][1];
                asm volatile("" : "+v"(lo), "+v"(hi)::"memory");          // (has arrived: its place may be refilled)
                const int ahead = rb + 1;
                if (ahead < RB) ask_x(ahead, cb + stride);
                else ask_x(0, cb + 2 * stride);
                wait_for_all_but<2 * (RB - 1)>();
                f4 nlo, nhi;
                read_x((rb + 2) % RB, nlo, nhi);
                __builtin_amdgcn_sched_barrier(0);
                split8_bf16(lo, hi, nxt[0], nxt[1], nxt[2]);
#pragma unroll
                for (int t = 0; t < 3 * QW; ++t)
                    if (t * RB / (3 * QW) == rb) draw_piece(t, cb + stride);
                constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int c = 0; c < CB; ++c) mm[rb][c].mac(cur[PA[p]], b[c][PB[p]]);
                __builtin_amdgcn_sched_barrier(0);
                // (the parameters of the quads drawn above are dead: send for those of the step after next)
#pragma unroll
                for (int t = 2; t < 3 * QW; t += 3)
                    if (t * RB / (3 * QW) == rb) ask_w(t / 3, cb + 2 * stride);
                cur[0] = nxt[0];
                cur[1] = nxt[1];
                cur[2] = nxt[2];
                raw[rb & 1][0] = nlo;
                raw[rb & 1][1] = nhi;
            }
        }
    }
    wait_for_all_but<0>();          // (what was sent for beyond the last step must not land in the sums below)
    const MfmaSettled settled;

    const int col = (int)threadIdx.x % OUTS, n = n0 + col;
    float bias = 0.0f;
    if (!TR && a.mu_b && n < N) bias = __builtin_fmaf(a.sigma_b[n], pick4_of(eps_quad(a.bias_quad0 + (n >> 2), s, a.rng), n & 3), a.mu_b[n]);
    float *const dst = a.out + (size_t)part * (size_t)a.part_stride + (size_t)s * (size_t)R * (size_t)N;
    bool special = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        __syncthreads();
        lds_float *mine = (lds_float *)lds + wave * (32 * RP);
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const f16v acc = mm[rb][c].read(settled);
#pragma unroll
            for (int g = 0; g < 16; ++g) mine[(8 * (g >> 2) + 4 * half + (g & 3)) * RP + 32 * c + l32] = acc[g];
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < OUTS / 8; ++it) {
            const int row = it * (256 / OUTS) + (int)threadIdx.x / OUTS;
            float v[kDeepWaves];
#pragma unroll
            for (int w = 0; w < kDeepWaves; ++w) v[w] = ((const lds_float *)lds)[w * (32 * RP) + row * RP + col];
            const int at = r0 + 32 * rb + row;
            if (at < R && n < N) {
                const float sum = (v[0] + v[1]) + (v[2] + v[3]) + bias;
                special |= sum != sum;
                dst[(size_t)at * (size_t)N + (size_t)n] = sum;
            }
        }
    }
    // (a loop of its own, so that no accumulator lives through it: each thread looks at what it stored)
    if (__builtin_amdgcn_ballot_w64(special) != 0) {
#pragma unroll 1
        for (int i = 0; i < RB * (OUTS / 8); ++i) {
            const int at = r0 + i * (256 / OUTS) + (int)threadIdx.x / OUTS;
            const bool mine = at < R && n < N;
            float *const y = dst + (size_t)(mine ? at : r0) * (size_t)N + (size_t)(mine ? n : n0);
            const bool again = mine && *y != *y;
            if (__builtin_amdgcn_ballot_w64(again) == 0) continue;
            const float *in = a.in + (size_t)s * (size_t)a.in_sample_stride + (size_t)(at < R ? at : r0) * (size_t)a.ld_in;
            const float sum = deep_plain_sum<TR, OUTS>(a, in, s, n, c_lo, c_hi, again);
            if (again) *y = sum + bias;
        }
    }
}

template <int RB, int CB, bool TR>
void deep_go(hipStream_t s, DeepArgs a, int samples, int n_begin, int n_end)
{
    const long items = (n_end - n_begin + 32 * CB - 1) / (32 * CB) * ((a.rows + 32 * RB - 1) / (32 * RB)) * a.parts * samples;
    a.n_begin = n_begin;
    a.samples = samples;
    a.items = (int)items;
    a.per_xcd = (int)((items + kXcds - 1) / kXcds);
    hot_linear_deep_kernel<RB, CB, TR><<<dim3((unsigned)(kXcds * a.per_xcd)), dim3(64 * kDeepWaves), 0, s>>>(a);
}

// The shapes of the kernel above and what they cost: microseconds per step of a workgroup with 1 .. `resident` workgroups on its
// compute unit (as many as registers and LDS admit), and of a round of workgroups besides its steps (the first loads, the sums
// through LDS, the stores).  Measured on layers of 3 to 128 steps; the model ranks shapes, and picks the number of parts.
struct DeepShape {
    int rb, cb, resident;
    double us[4];
    double start;
};
constexpr DeepShape kDeepShapes[] = {{2, 1, 4, {1.05, 1.9, 2.3, 2.9}, 4.0}, {4, 1, 3, {1.1, 2.05, 2.8}, 5.0}, {6, 1, 2, {1.5, 2.7}, 6.0}, {8, 1, 2, {1.75, 3.8}, 7.0},
                                     {10, 1, 1, {2.3}, 9.0}, {6, 2, 1, {2.6}, 11.0}, {8, 2, 1, {3.0}, 13.0}, {4, 2, 2, {2.1, 3.9}, 6.0}};
constexpr int kDeepCodes = sizeof(kDeepShapes) / sizeof(kDeepShapes[0]);
constexpr int kDeepCodesTr = kDeepCodes - 1;        // (the last one's transposed draw spills its registers)

struct DeepPlan {
    int code;               // index into kDeepShapes, -1: none
    int rest_code;          // the shape of the outputs n_cut .. N - 1, which would start a round of their own (-1: one launch)
    long n_cut;
    int parts;
    long contract_per_part;
    double cost;            // what shapes and parts are ranked by
};

inline double deep_cost(const DeepShape &h, long wgs, long steps)
{
    const long round = (long)kComputeUnits * h.resident, full = wgs / round, left = wgs % round;
    double t = (double)full * ((double)steps * h.us[h.resident - 1] + 5.0);
    if (left) t += (double)steps * h.us[(left + kComputeUnits - 1) / kComputeUnits - 1] + 5.0;
    return t + 4.0;
}

// Where it runs, measured against the other kernels on 60 layer shapes: forward from 33 rows on (64 x 2160 x 8640 x 2 samples 133 ->
// 83 us, 300: 638 -> 215, 256 x 8192^2 592 -> 403, 64 x 1024^2 x 8 93 -> 22; at 16 rows 59 -> 79, so fewer stay), input gradients from
// 65 (below, the other kernel draws as few weights and has more waves: 0.87-1.04x), both given two (four) steps of contraction per
// wave and, without parts, 100 workgroups for the input gradients (below, the other kernel's up to sixteen waves per tile win:
// 200 x 192 x 768 27 -> 32).  Where the kernel above runs too, the faster one by the two models (deep_beats_slab).
constexpr long kDeepMinRows = 33, kDeepMinRowsTr = 65;
constexpr long kDeepMinContract = 128, kDeepMinContractTr = 256, kDeepMinWorkgroupsTr = 100;
constexpr int kDeepMaxParts = 16;
constexpr int64_t kDeepMaxBytes = (int64_t)256 << 20;
constexpr long kDeepMostTiles = (1L << 24) - kXcds;

// Whether the kernel can take a problem of R rows, C contraction indices and N outputs, and is worth a look there.
inline bool deep_fits(long R, long C, long N, long ld_in, int S, bool tr)
{
    if (R < (tr ? kDeepMinRowsTr : kDeepMinRows) || C < (tr ? kDeepMinContractTr : kDeepMinContract) || S > 65535) return false;
    constexpr long kIndexMost = 1L << 29;                // (so that the products below stay within 64 bits)
    if (R > kIndexMost || C > kIndexMost || N > kIndexMost || ld_in > kIndexMost) return false;
    const unsigned long long lim = 0x7FFFFFF0ull;
    if ((unsigned long long)(R + 640) * ld_in * 4 >= lim || (unsigned long long)(C + 256) * (N + 64) * 4 >= 2 * lim) return false;
    // One workgroup of 256 threads per tile, in one dimension of the grid, which holds fewer than 2^32 threads.  (Parts need not be
    // counted: what they leave in the workspace bounds them to far fewer tiles.)
    return (N + 31) / 32 * ((R + 63) / 64) <= kDeepMostTiles / S;
}

// ws_bytes: as in wgrad_shape (0: no parts); least_parts: the fewest parts allowed
inline DeepPlan deep_plan(long R, long C, long N, long ld_in, int S, bool tr, int64_t ws_bytes, int least_parts)
{
    DeepPlan best = {-1, -1, 0, 1, 0, 0.0};
    if (!deep_fits(R, C, N, ld_in, S, tr)) return best;
    const int64_t block_bytes = (int64_t)S * R * N * (int64_t)sizeof(float);
    const int64_t budget = ws_bytes < 0 || ws_bytes > kDeepMaxBytes ? kDeepMaxBytes : ws_bytes;
    for (int i = 0; i < (tr ? kDeepCodesTr : kDeepCodes); ++i) {
        const DeepShape &h = kDeepShapes[i];
        const long row_tiles = (R + 32 * h.rb - 1) / (32 * h.rb), col_tiles = (N + 32 * h.cb - 1) / (32 * h.cb);
        const long per_col = row_tiles * S;             // workgroups of one column of tiles
        for (int parts = least_parts; parts <= (tr ? kDeepMaxParts : 1); ++parts) {
            if (parts > 1 && parts * block_bytes > budget) break;
            const long per_part = ((C + parts - 1) / parts + kDeepStep - 1) / kDeepStep * kDeepStep;
            if (parts > 1 && (per_part * (parts - 1) >= C || per_part < 2 * kDeepStep)) continue;
            if (tr && parts == 1 && col_tiles * per_col < kDeepMinWorkgroupsTr) continue;
            double cost = deep_cost(h, col_tiles * per_col * parts, per_part / kDeepStep);
            if (parts > 1) cost += 4.0 + (double)(parts + 1) * (double)block_bytes / 4e6;
            if (best.code < 0 || cost < best.cost) best = DeepPlan{i, -1, N, parts, per_part, cost};
        }
        if (least_parts > 1) continue;
        // whole rounds of this shape, and what is left over in the shape that does it fastest
        const long steps = (C + kDeepStep - 1) / kDeepStep, round = (long)kComputeUnits * h.resident;
        const long main_tiles = col_tiles * per_col / round * round / per_col;
        if (main_tiles < 1 || main_tiles >= col_tiles) continue;
        const double main_cost = deep_cost(h, main_tiles * per_col, steps);
        const long n_cut = main_tiles * 32 * h.cb;
        for (int j = 0; j < (tr ? kDeepCodesTr : kDeepCodes); ++j) {
            const DeepShape &r = kDeepShapes[j];
            const double cost = main_cost + deep_cost(r, (N - n_cut + 32 * r.cb - 1) / (32 * r.cb) * ((R + 32 * r.rb - 1) / (32 * r.rb)) * S, steps);
            if (best.code >= 0 && cost < best.cost) best = DeepPlan{i, j, n_cut, 1, steps * kDeepStep, cost};
        }
    }
    return best;
}

template <bool TR>
void deep_launch(int code, hipStream_t s, const DeepArgs &a, int samples, long n0, long n1)
{
    switch (code) {
    case 0: return deep_go<2, 1, TR>(s, a, samples, (int)n0, (int)n1);
    case 1: return deep_go<4, 1, TR>(s, a, samples, (int)n0, (int)n1);
    case 2: return deep_go<6, 1, TR>(s, a, samples, (int)n0, (int)n1);
    case 3: return deep_go<8, 1, TR>(s, a, samples, (int)n0, (int)n1);
    case 4: return deep_go<10, 1, TR>(s, a, samples, (int)n0, (int)n1);
    case 5: return deep_go<6, 2, TR>(s, a, samples, (int)n0, (int)n1);
    case 6: return deep_go<8, 2, TR>(s, a, samples, (int)n0, (int)n1);
    default:
        if constexpr (!TR) deep_go<4, 2, false>(s, a, samples, (int)n0, (int)n1);
    }
}

template <bool TR>
void deep_run(const DeepPlan &p, hipStream_t s, DeepArgs a, int samples)
{
    a.parts = p.parts;
    a.contract_per_part = p.contract_per_part;
    deep_launch<TR>(p.code, s, a, samples, 0, p.n_cut);
    if (p.rest_code >= 0) deep_launch<TR>(p.rest_code, s, a, samples, p.n_cut, a.outs);
}

// Whether the kernel above can address this problem (its windows take 32-bit byte offsets, its indices are 32-bit).
inline bool slab_kernel_fits(long rows, long contract, long outs, long ld_in)
{
    const unsigned long long lim = 0xFFFFFFF0ull;
    return (unsigned long long)((rows + 2 * kSlabRows) * ld_in + contract) * 4 < lim && (unsigned long long)(contract + 4 * kSlabK) * outs * 4 < lim &&
           (unsigned long long)(rows + 2 * kSlabRows) * (outs + 128) * 4 < lim && (rows + kSlabRows - 1) / kSlabRows <= 65535;
}

constexpr int kSlabMinRows = 512;             // below, the kernels whose workgroups hold 256 rows
// Least share of the chip's time that the tiles of a launch must fill, measured against the kernels for fewer rows on 130
// layer shapes.  Forward with a shared x: wins from 0.6 on (1.1-2x; between 0.45 and 0.6 anything from 0.73x to 1.2x).
// Forward with one x per sample, where the other kernel is weaker: from 0.45 on (1.4-1.5x between 0.45 and 0.6).  Input
// gradients, whose other kernel packs several 256-row workgroups into a compute unit: from 0.72 on (1.0-1.3x), and from
// 0.6 on where the tiles of 32 inputs are the best shape (1.0-1.2x there; the wider shapes 0.95-0.97x).
constexpr double kSlabMinFillForward = 0.6, kSlabMinFillForwardOwnX = 0.45, kSlabMinFillInputGrad = 0.72, kSlabMinFillInputGradNarrow = 0.6;

// A launch shape of the kernel above and what it costs.  One workgroup per compute unit runs at a time (two of the narrow
// ones, at half speed each), so a launch takes its number of rounds times the time of a workgroup, which per step is, per
// block of 32 outputs and sample, about 2050 cycles of matrix instructions for 512 rows plus 325 of drawing, and
// 600 for the barrier and what else does not overlap; the wider tile also loads x half as often.  The constants are
// fitted to timings of 130 layer shapes; the model only has to rank the shapes of one layer.
struct SlabShape {
    int waves;      // 4, 8 or 16; 0: none
    int cbw;        // blocks of 32 outputs per workgroup
    double cost;
    int rbw = 2;    // blocks of 32 rows per wave (one: four waves of 32 rows, for 65 to 128 rows)
    double fill = 1.0;      // four-wave shapes: the share of its compute units' workgroup slots that the launch fills
};

// Four waves: 256 rows x 32 or 64 output-samples.  Up to four such workgroups share a compute unit and run at the rate of
// its matrix pipes together (measured per step and workgroup: 2700 cycles for 64 output-samples, 1600 for 32, whose x is
// re-read twice as often), one alone at that plus 600.  Against the kernels on the fp32 instruction they win from a fill of 0.52
// of the compute units' last workgroup on (measured on 160 layer shapes of 256 to 7260 rows: 1.1-2.2x from there, 0.3-0.9x below);
// against the kernel for tens to hundreds of rows deep_beats_slab decides.
constexpr double kSlab4MinFill = 0.52;
constexpr long kSlab4MinRows = 129;
// From 65 to 128 rows the four waves take 32 rows each: half the matrix work per draw again, measured per step and
// workgroup 1850 cycles for 64 output-samples and 1170 for 32, 300 more for one alone on its compute unit.  The kernel for tens to
// hundreds of rows takes most of these layers; to this shape remain few inputs and many outputs (110 x 100 x 8192 x 2, below
// 128 inputs, or where deep_beats_slab prefers it).  A narrow workgroup alone on its compute unit (one wave per SIMD) loses
// (96 x 4096^2: 0.87x), so the shapes of 32 output-samples need two workgroups per compute unit.
constexpr long kSlab4HalfMinRows = 65;
constexpr double kSlab4HalfMinFill = 0.52;

inline SlabShape slab_shape4(long rows, long outs, long passes, int st)
{
    SlabShape best = {0, 0, 0.0};
    if (passes < 1 || passes > 65535 || rows < kSlab4HalfMinRows) return best;
    const bool half = rows <= 128;
    const long tile_rows = half ? 128 : 256;
    for (int cbw = st == 2 ? 1 : 2; cbw >= 1; cbw /= 2) {
        const long col_tiles = (outs + 32 * cbw - 1) / (32 * cbw), wgs = col_tiles * ((rows + tile_rows - 1) / tile_rows) * passes;
        const long per_cu = (wgs + kComputeUnits - 1) / kComputeUnits;
        const double exact = (double)outs / (32 * cbw) * (double)rows / (double)tile_rows * (double)passes;
        if (exact < (half ? kSlab4HalfMinFill : kSlab4MinFill) * (double)(per_cu * kComputeUnits)) continue;
        if (half && cbw * st == 1 && wgs < 2 * kComputeUnits) continue;
        const double wide = half ? 1850.0 : 2700.0, narrow = half ? 1170.0 : 1600.0;
        const double cost = (double)per_cu * (cbw * st == 2 ? wide : narrow) + (per_cu == 1 ? (half ? 300.0 : 600.0) : 0.0);
        if (best.waves == 0 || cost < best.cost) best = SlabShape{4, cbw, cost, half ? 1 : 2, exact / (double)(per_cu * kComputeUnits)};
    }
    return best;
}

// the cheapest of the eight-wave shapes with `st` samples per pass and tiles of 32 * narrow .. 32 * wide outputs
inline SlabShape slab_shape8(long rows, long outs, long passes, int st, int narrow, int wide)
{
    SlabShape best = {0, 0, 0.0};
    if (passes < 1 || passes > 65535) return best;
    const long row_blocks = (rows + kSlabRows - 1) / kSlabRows;
    for (int cbw = wide; cbw >= narrow; cbw /= 2) {
        const long wgs = ((outs + 32 * cbw - 1) / (32 * cbw)) * row_blocks * passes;
        // (two narrow workgroups share a compute unit and cover part of each other's waits: about 5 % by measurement)
        const double cost = (double)((wgs + kComputeUnits - 1) / kComputeUnits) * (2375.0 * cbw * st + 600.0) * (cbw * st <= 2 ? 0.95 : 1.0);
        if (best.waves == 0 || cost < best.cost) best = SlabShape{8, cbw, cost};
    }
    return best;
}

// sixteen waves: 1024 rows x 64 outputs, one sample per pass
inline SlabShape slab_shape16(long rows, long outs, long passes)
{
    if (passes < 1 || passes > 65535 || rows <= kSlabRows) return SlabShape{0, 0, 0.0};
    const long wgs = ((outs + 63) / 64) * ((rows + 2 * kSlabRows - 1) / (2 * kSlabRows)) * passes;
    // (measured on layers that both shapes fill: 0.966 of the time of 512 rows x 64 outputs x 2 samples)
    return SlabShape{16, 2, (double)((wgs + kComputeUnits - 1) / kComputeUnits) * 9750.0};
}

// what the samples of a launch would cost on a chip they fill evenly
inline double slab_full(long rows, long outs, long samples)
{
    return (double)rows / kSlabRows * (double)outs / 32.0 * (double)samples * 2375.0 / kComputeUnits;
}

// Launches it for the samples s_begin .. s_end - 1, ST per pass, one pass per layer of the grid along z.
template <int WAVES, int CBW, int ST, bool OWN, bool TR, int RBW = 2>
void slab_go(hipStream_t s, SlabArgs a, int s_begin, int s_end)
{
    a.s_begin = s_begin;
    a.s_end = s_end;
    const dim3 grid((unsigned)((a.outs + 32 * CBW - 1) / (32 * CBW)), (unsigned)((a.rows + 32 * RBW * WAVES - 1) / (32 * RBW * WAVES)),
                    (unsigned)((s_end - s_begin + ST - 1) / ST));
    hot_linear_slab_kernel<WAVES, CBW, ST, OWN, TR, RBW><<<grid, dim3(64 * WAVES), 0, s>>>(a);
}

// one sample per pass, in the shape chosen
template <bool OWN, bool TR>
void slab_go_singles(const SlabShape &shape, hipStream_t s, const SlabArgs &a, int s_begin, int s_end)
{
    if (shape.waves == 16) slab_go<16, 2, 1, OWN, TR>(s, a, s_begin, s_end);
    else if (shape.waves == 4 && shape.rbw == 1 && shape.cbw == 2) slab_go<4, 2, 1, OWN, TR, 1>(s, a, s_begin, s_end);
    else if (shape.waves == 4 && shape.rbw == 1) slab_go<4, 1, 1, OWN, TR, 1>(s, a, s_begin, s_end);
    else if (shape.waves == 4 && shape.cbw == 2) slab_go<4, 2, 1, OWN, TR>(s, a, s_begin, s_end);
    else if (shape.waves == 4) slab_go<4, 1, 1, OWN, TR>(s, a, s_begin, s_end);
    else if (shape.cbw == 4) slab_go<8, 4, 1, OWN, TR>(s, a, s_begin, s_end);
    else if (shape.cbw == 2) slab_go<8, 2, 1, OWN, TR>(s, a, s_begin, s_end);
    else slab_go<8, 1, 1, OWN, TR>(s, a, s_begin, s_end);
}

// the cheaper of the shapes with one sample per pass, or none where the chip would stand too empty
// (min_fill_narrow: the bar where that shape has tiles of 32 outputs)
inline SlabShape slab_shape_singles(long rows, long outs, long samples, double min_fill, double min_fill_narrow)
{
    SlabShape best = {0, 0, 0.0};
    if (rows >= kSlabMinRows) {
        best = slab_shape8(rows, outs, samples, 1, 1, 4);
        const SlabShape tall = slab_shape16(rows, outs, samples);
        if (tall.waves && (!best.waves || tall.cost < best.cost)) best = tall;
        const double bar = best.waves == 8 && best.cbw == 1 ? min_fill_narrow : min_fill;
        if (best.waves && slab_full(rows, outs, samples) < bar * best.cost) best.waves = 0;
    }
    const SlabShape small = slab_shape4(rows, outs, samples, 1);
    if (small.waves && (!best.waves || small.cost < best.cost)) best = small;
    return best;
}

// How the forward call runs a layer on the kernel above: pairs of samples that share x (samples 0 .. 2 * pairs - 1) in
// `two` and the samples behind them one at a time in `one`; neither where the layer is left to the kernels for fewer rows.
struct SlabForwardPlan {
    int pair_samples;     // samples that go two to a pass
    SlabShape two, one;   // (waves == 0: not used)
};

inline SlabForwardPlan slab_forward_plan(const hot_linear_desc *d)
{
    SlabForwardPlan p = {0, SlabShape{0, 0, 0.0}, SlabShape{0, 0, 0.0}};
    if (d->rows < kSlab4HalfMinRows || !slab_kernel_fits(d->rows, d->in_features, d->out_features, d->ldx)) return p;
    const int S = d->s_local;
    if (d->x_sample_stride != 0 || S == 1) {
        const double bar = d->x_sample_stride != 0 ? kSlabMinFillForwardOwnX : kSlabMinFillForward;
        p.one = slab_shape_singles(d->rows, d->out_features, S, bar, bar);
        return p;
    }
    // two samples to a pass and an odd last one on its own (512-row or 256-row workgroups), or every sample on its own in the
    // tall shape: whichever is cheapest among those that fill the chip well enough
    const int pairs = S / 2, odd = S & 1;
    const SlabShape none = {0, 0, 0.0}, free = {8, 0, 0.0};
    double best = 0.0;
    if (d->rows >= kSlabMinRows) {
        const SlabShape two = slab_shape8(d->rows, d->out_features, pairs, 2, 1, 2);
        const SlabShape last = odd ? slab_shape8(d->rows, d->out_features, 1, 1, 1, 4) : free;
        const SlabShape tall = slab_shape16(d->rows, d->out_features, S);
        const double full = slab_full(d->rows, d->out_features, S);
        if (tall.waves && (!two.waves || !last.waves || tall.cost < two.cost + last.cost)) {
            if (full >= kSlabMinFillForward * tall.cost) {
                p.one = tall;
                best = tall.cost;
            }
        } else if (two.waves && last.waves && full >= kSlabMinFillForward * (two.cost + last.cost)) {
            p.pair_samples = 2 * pairs;
            p.two = two;
            p.one = odd ? last : none;
            best = two.cost + last.cost;
        }
    }
    const SlabShape two4 = slab_shape4(d->rows, d->out_features, pairs, 2);
    const SlabShape last4 = odd ? slab_shape4(d->rows, d->out_features, 1, 1) : free;
    if (two4.waves && last4.waves && (best == 0.0 || two4.cost + last4.cost < best)) {
        p.pair_samples = 2 * pairs;
        p.two = two4;
        p.one = odd ? last4 : none;
    }
    return p;
}

// ... and the input gradients (dy is the input, read in 16-byte quads: rows of dy must allow that)
inline SlabShape slab_input_grad_shape(const hot_linear_desc *d, bool dy_aligned)
{
    if (d->rows < kSlab4HalfMinRows || (d->out_features & 3) != 0 || !dy_aligned ||
        !slab_kernel_fits(d->rows, d->out_features, d->in_features, d->out_features))
        return SlabShape{0, 0, 0.0};
    return slab_shape_singles(d->rows, d->in_features, d->s_local, kSlabMinFillInputGrad, kSlabMinFillInputGradNarrow);
}

constexpr DeepPlan kNoDeepPlan = {-1, -1, 0, 1, 0, 0.0};

// What a plan takes, in microseconds, to compare it with other kernels: shapes are ranked with 5 us for the start of every round,
// as they were measured; here it is the shape's own.  And every column of tiles reads the whole input: one that the L2 caches cannot
// hold (inputs: how many differ among the samples) comes at 5.3 TB/s (1387 x 1964 x 540 x 8 samples with inputs of their own: 1.5 GB,
// 296 us, where the steps alone would take 188; 2019 x 2108 x 768 x 2: 0.82 GB, 149 us).
constexpr double kInputTooLarge = 20e6, kInputBytesPerUs = 5.3e6;

inline double deep_time(const DeepPlan &p, long R, long C, long N, long S, long inputs)
{
    long col_tiles = 0;
    double t = p.cost;
    auto add = [&](int code, long n) {
        const DeepShape &h = kDeepShapes[code];
        const long cols = (n + 32 * h.cb - 1) / (32 * h.cb), wgs = cols * ((R + 32 * h.rb - 1) / (32 * h.rb)) * S * p.parts;
        const long round = (long)kComputeUnits * h.resident;
        t += (double)((wgs + round - 1) / round) * (h.start - 5.0);
        col_tiles += cols;
    };
    add(p.code, p.n_cut);
    if (p.rest_code >= 0) add(p.rest_code, N - p.n_cut);
    const double bytes = (double)R * (double)C * 4.0;
    const double reads = bytes * (double)inputs > kInputTooLarge ? bytes * (double)(S * col_tiles) / kInputBytesPerUs : 0.0;
    return t > reads ? t : reads;
}

// What a launch of the slab kernel takes, in microseconds: a unit of its cost times its steps of 16 indices is 0.32 ns, more or less
// of it by shape, fitted to 200 layers of 65 to 3500 rows and 128 to 4096 inputs (st: samples per pass).
inline double slab_time(const SlabShape &h, int st, long contract)
{
    if (!h.waves) return 0.0;
    const int wide = h.cbw * st;
    double share = 1.1, start = 5.0;                                     // 256 rows x 32 outputs
    if (h.waves == 4 && h.rbw == 1) start = 6.0;                         // 128 rows
    else if (h.waves == 4 && st == 2) share = 0.78, start = 7.0;
    else if (h.waves == 4 && wide == 2) share = 0.86, start = 10.0;
    else if (h.waves == 8 && wide == 1) share = h.cost > 3000.0 ? 1.0 : 1.3, start = 6.0;       // (1.3: alone on its compute unit)
    else if (h.waves == 8 && wide == 2) share = 0.92, start = 7.0;
    else if (h.waves == 8) share = 0.8, start = 11.0;
    else if (h.waves == 16) share = 0.85, start = 18.0;
    return share * h.cost * (double)((contract + kSlabK - 1) / kSlabK) * 3.2e-4 + start;
}

// Whether the kernel for tens to hundreds of rows takes a layer that the slab kernel could take (slab: that one's time, 0: it could
// not), unless the models are too close to tell.  Of 1000 layers where either runs they leave three more than 6 % behind the faster
// (245 x 644 x 6107 x 2 samples: 42 us against 38); with the kernel for fewer rows up to 704 rows always, layers of few inputs and many
// outputs lost (493 x 236 x 8192 x 4: 94 against 67, 658 x 192 x 8048 x 4 134 against 74).
inline bool deep_beats_slab(const DeepPlan &p, long R, long C, long N, long S, long inputs, double slab)
{
    return p.code >= 0 && (slab == 0.0 || deep_time(p, R, C, N, S, inputs) < 0.96 * slab);
}

// Whether a forward call is left to the first kernel above: where that has at most one workgroup (64 rows x 16 outputs, one
// sample) per compute unit.  A workgroup of either waits for one dependent chain per step there, and the first kernel's
// four waves step over 128 indices in 1.3 us, those of the kernel for tens to hundreds of rows over 64 in 1.0 to 1.6.  Measured
// on 360 layers: up to 256 workgroups 1.2x on average (63 x 6480 x 1172 x 1: 82 us against 135, 312 x 6816 x 72 x 1 86 against 139;
// at worst 0.95x), from 257 to 512 0.9x, but for long sums (52 x 8192 x 6264 x 1: 214 against 237, 769 x 7712 x 252 x 2 150 against
// 171, 71 x 2804 x 2048 x 2 55 against 60; one sample up to 5000 inputs 1.05x the other way).
inline bool few_first_kernel_workgroups(const hot_linear_desc *d)
{
    const long gx = (d->out_features + kColsPerWave - 1) / kColsPerWave, gy = (d->rows + 4 * kRowsPerTile - 1) / (4 * kRowsPerTile);
    if (gx > 2 * kComputeUnits || gy > 2 * kComputeUnits) return false;
    const long wgs = gx * gy * d->s_local;
    return wgs <= kComputeUnits || (wgs <= 2 * kComputeUnits && d->s_local <= 2 && d->in_features > (d->s_local == 2 ? 2500 : 6000));
}

inline DeepPlan deep_forward_plan(const hot_linear_desc *d)
{
    if (few_first_kernel_workgroups(d)) return kNoDeepPlan;
    const DeepPlan p = deep_plan(d->rows, d->in_features, d->out_features, d->ldx, d->s_local, false, 0, 1);
    if (p.code < 0) return p;
    const SlabForwardPlan slab = slab_forward_plan(d);
    const double time = slab_time(slab.two, 2, d->in_features) + slab_time(slab.one, 1, d->in_features);
    return deep_beats_slab(p, d->rows, d->in_features, d->out_features, d->s_local, d->x_sample_stride != 0 ? d->s_local : 1, time) ? p : kNoDeepPlan;
}

// Whether planes of drawn weights (linear_planes.h) stand in for a launch of the slab kernel that takes `slab` microseconds by its
// model: where a workspace holds them, unless they are slower by the models.  (Their sums are the bf16 slab kernel's bit for bit;
// layers of the 128-row slab shapes on the fp32 instruction stay where they are.)  Of 9600 forward products that this and the
// next rule take, drawn over the range, planes are 1.32 times as fast on average, 62 slower by more than 3 % (0.83 at worst, 4317 x 128 x 4302 x 8; 7260 x 2160 x
// 540 x 2 samples 312 -> 190 us, 13300 x 180 x 216 x 4 94 -> 42); the slab model is 10 % below the time in the middle, hence the factor; under 40 us the second launch and the draw of
// wide layers show (213 x 120 x 5072 x 4: 19 -> 30).
// Up to kPlanesFewRows rows that model is right in the middle, and tiles smaller than 256 x 256 are taken only where the models see them ahead:
// with the factor 46 of 229 forward products were slower by more than 3 % (219 x 304 x 1406 x 16 samples 35 -> 44 us, 444 x 1832 x 4769 x 8 432 ->
// 493, 153 x 224 x 6932 x 8 54 -> 61), without it 11 are, by 3 to 8 % but for one; of 199 backward passes, their input gradients from planes, 14 (222 x
// 7776 x 832 x 3 184 -> 203) and none; the products given back were 6 % faster on average.  The tiles of 256 x 256 were behind on none of 16 there.  One
// sample below 8.3 us by the model: its two launches take longer than that (719 x 96 x 1536 8.9 -> 11.4, 3031 x 96 x 375 9.3 -> 10.9, 1381 x 120 x 862
// 10.6 -> 11.6; from there on 3596 x 148 x 311 12.7 -> 12.0).
constexpr double kPlanesMost = 1.11, kPlanesMostFewRows = 1.0, kPlanesMostShort = 0.75, kPlanesShort = 40.0, kPlanesLeastAlone = 8.3;
constexpr long kPlanesFewRows = 512;

inline PlanePlan planes_instead(long R, long C, long N, int S, bool tr, double slab, int64_t ws_bytes)
{
    const PlanePlan p = plane_plan(R, C, N, S, tr, false);
    const bool few = R <= kPlanesFewRows && p.code >= 0 && !plane_shape_large(kPlaneShapes[p.code]);
    const double most = p.time < kPlanesShort ? kPlanesMostShort : few ? kPlanesMostFewRows : kPlanesMost;
    if (!tr && S == 1 && p.time < kPlanesLeastAlone) return kNoPlanePlan;
    return p.code >= 0 && (ws_bytes < 0 || p.bytes <= ws_bytes) && p.time < most * slab ? p : kNoPlanePlan;
}

// ... and for a forward launch of the kernel for tens to hundreds of rows, with the small products apart.  (826 x 5136 x 1275 x 4: 338 -> 280, 1363 x 2188 x
// 1272 x 3 199 -> 142; where the models are closer than this the two are level, 300 x 2160 x 8640 x 2 227 and 226, of which 64 are the draw at 5.8 TB/s.)  The two narrow tiles have the long sums, where the models know less, and under 40 us it is as above.
// The larger tiles of that kernel (eight blocks of 32 x 32 and more, code 3 on) are further from its model: beside fewer than kApartFewOutputs outputs nearer lines than kApartMostFew lost
// (of 527 products 8, 2707 x 6776 x 83 x 7 samples 195 -> 236 us, 5288 x 3168 x 97 x 4 122 -> 136; the others there gained 6 %), and with more outputs
// those of 32 outputs, one workgroup to a compute unit (codes 3 and 4), read rows that are in the L2 already, a third faster than it says: 604 x 7984 x 968 x 4
// 283 -> 370 and 631 x 1984 x 559 x 7 80 -> 86 where the models see 0.73.  Of the 527, 483 are left, one slower by more than 3 % (was 11).
constexpr double kApartMost = 0.9, kApartMostNarrow = 0.75, kApartMostFew = 0.84, kApartMostTall = 0.7;
constexpr long kApartFewOutputs = 450;

inline PlanePlan planes_forward_plan(const hot_linear_desc *d, int64_t ws_bytes)
{
    if (ws_bytes == 0) return kNoPlanePlan;
    if (const DeepPlan deep = deep_forward_plan(d); deep.code >= 0) {
        if (!slab_kernel_fits(d->rows, d->in_features, d->out_features, d->ldx)) return kNoPlanePlan;        // (32-bit offsets)
        const PlanePlan p = plane_plan(d->rows, d->in_features, d->out_features, d->s_local, false, true);
        const double time = deep_time(deep, d->rows, d->in_features, d->out_features, d->s_local, d->x_sample_stride != 0 ? d->s_local : 1);
        double most = p.code >= 0 && kPlaneShapesApart[p.code].rb == 1 ? kApartMostNarrow : kApartMost;
        if (deep.code >= 3 && d->out_features < kApartFewOutputs) most = std::min(most, kApartMostFew);
        if (p.time < kPlanesShort) most *= kPlanesMostShort;
        else if ((deep.code == 3 || deep.code == 4) && d->out_features >= kApartFewOutputs) most = std::min(most, kApartMostTall);
        return p.code >= 0 && (ws_bytes < 0 || p.bytes <= ws_bytes) && p.time < most * time ? p : kNoPlanePlan;
    }
    const SlabForwardPlan slab = slab_forward_plan(d);
    if ((!slab.two.waves && !slab.one.waves) || (slab.two.waves && slab.two.rbw == 1) || (slab.one.waves && slab.one.rbw == 1)) return kNoPlanePlan;
    return planes_instead(d->rows, d->in_features, d->out_features, d->s_local, false,
                          slab_time(slab.two, 2, d->in_features) + slab_time(slab.one, 1, d->in_features), ws_bytes);
}

template <int RB, bool XS>
void linear_go_st(int st, dim3 grid, int waves, hipStream_t s, const LinearArgs &a)
{
    const dim3 block(64 * waves);
    const size_t lds = waves > 1 ? (size_t)(waves - 1) * (size_t)(st * RB * 4) * 64 * sizeof(float) : 0;
    if constexpr (four_samples_fit(RB, XS)) {
        if (st == 4) { hot_linear_forward_kernel<RB, 4, XS><<<grid, block, lds, s>>>(a); return; }
    }
    if (st >= 2) hot_linear_forward_kernel<RB, 2, XS><<<grid, block, lds, s>>>(a);
    else hot_linear_forward_kernel<RB, 1, XS><<<grid, block, lds, s>>>(a);
}

template <int RB>
void linear_go(int st, dim3 grid, int waves, hipStream_t s, const LinearArgs &a)
{
    // (one sample has one input: 129 x 3648 x 540 x 1 51 -> 47 us)
    if (a.x_sample_stride != 0 && a.s_loc > 1) linear_go_st<RB, true>(st, grid, waves, s, a);
    else linear_go_st<RB, false>(st, grid, waves, s, a);
}


// ---------------------------------------------------------------------------------
// Backward.  Weight gradients: a wave owns 16 outputs x 64 inputs and contracts over the rows with
// the TRANSPOSED product P_s[k][o] = sum_r x_s[r][k] dy_s[r][o] (x as the A operand, dy as B).  A lane
// loads four consecutive inputs of a row of x at once and hands element i to matrix instruction i, so
// that register c of the four accumulators holds four consecutive inputs k of one output o: exactly one
// quad of the generator, drawn once per sample, and one 16-byte access to mu, sigma and the two
// gradient arrays.  Input gradients: dx_s^T[k][r] = sum_o W_s[o][k] dy_s[r][o] with
// the drawn weights as the A operand; MFMA number i of a step takes element i of every lane's
// quad (as in the forward kernel), so result register rr of the four accumulators again holds
// four consecutive inputs and dx is written with 16-byte stores.
// ---------------------------------------------------------------------------------
struct LinearGradArgs {
    long rows, in_features, out_features, ldx, x_sample_stride;
    int s_loc;
    long weight_quad0, bias_quad0;
    double g, k;            // scaling of the data part and of the KL part of the gradients
    const float *x, *dy, *mu_w, *sigma_w, *mu_b, *sigma_b;
    float *gmu_w, *gsig_w, *gmu_b, *gsig_b, *dx;
    float *ws;              // PARTS kernels: partial sums [part][gm, gs][O*K + O]
    long rows_per_part;     // PARTS kernels: rows of one part, a multiple of 16
    int x_parts;            // input gradients for many rows: parts the outputs are cut into (1: dx written directly)
    long outs_per_part;     // outputs of one such part, a multiple of 16; partial dx blocks go to ws[part][S][R][K]
    Rng rng;
};

__device__ __forceinline__ float pick4(f4 v, int c) { return c == 0 ? v[0] : (c == 1 ? v[1] : (c == 2 ? v[2] : v[3])); }

// The four lanes (j = 0..3, same n) of a 16-lane column each hold four quads q[0..3], lane j's quad t
// belonging to position 16 j + 4 t of a 64-wide block.  Afterwards lane j's quad t belongs to position
// 16 t + 4 j: a store of quad t then covers 64 contiguous bytes per 16-lane column instead of four separate
// 16-byte pieces (the memory system wants whole 64-byte words).  A 4 x 4 transpose over j in four rounds of
// lane shuffles; every lane of the wave must call it.
__device__ __forceinline__ void transpose_quads_over_j(f4 (&q)[4], int j, int n)
{
    f4 out[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int give = (j - d) & 3, from = (((j + d) & 3) << 4) | n, slot = (j + d) & 3;
        f4 v = q[0];
#pragma unroll
        for (int t = 1; t < 4; ++t)
            if (give == t) v = q[t];
        f4 r;
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = __shfl(v[c], from);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (slot == t) out[t] = r;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) q[t] = out[t];
}

// grad_mu, grad_sigma of one parameter from its sums over the samples (gradient and averaging lines
// of Algorithm 2; d KL / d mu = mu, d KL / d sigma = sigma - 1/sigma).  In single precision: six operations per
// parameter.  An fp64 form (the flat sample layer's, which is bound by memory) cost these kernels, bound by vector
// arithmetic at few rows, about 1000 cycles per 16 x 64 tile, 40 % of a draw (8192^2 at 16 rows: weight gradients
// 0.289 -> 0.271 ms; at 1024 rows 127.6 -> 130 TFLOP/s); each term is rounded once more, 1e-7 of its magnitude.
__device__ __forceinline__ void finish_pair(float sum_g, float sum_ge, float m, float sd, float g, float k,
                                            float &gm, float &gs)
{
    const float kl_m = k != 0.0f ? k * m : 0.0f;
    const float kl_s = k != 0.0f ? k * (sd - __builtin_amdgcn_rcpf(sd)) : 0.0f;
    gm = __builtin_fmaf(g, sum_g, kl_m);
    gs = __builtin_fmaf(g, sum_ge, kl_s);
}

constexpr int kWgradWaves = 4;       // waves per workgroup when every wave has a tile of its own
constexpr int kWgradMaxSplit = 8;    // most waves that share one tile (60 KiB of LDS for their partial sums)
constexpr int kWgradRowsPerIter = 16;
constexpr int kWgradDeepRows = 128;  // from this many rows on operands are prefetched one row block ahead
constexpr int kWgradWideRows = 512;  // from this many rows on a wave may own several output groups
constexpr int kWgradMaxParts = 16;    // most row parts of a run with a workspace
constexpr int kWgradPartials = 34;   // per lane: 16 + 16 weight-gradient sums and the two bias sums

// SPLIT = false: the four waves of a workgroup own one tile each.  SPLIT = true (layers with few
// tiles and many rows): the waves of a workgroup share one tile, take the 16-row blocks round-robin,
// apply each sample's eps to their own partial product (the gradient is linear in it) and add their
// sums through LDS in wave order at the end.  DEEP (many rows): operands of the next row block are
// fetched while the current one multiplies; it costs a wave per SIMD, which the few-row shapes need more.
// OB: 16-output groups per tile.  At many rows the kernel is bound by the 16-byte loads of x (with them
// taken out it runs at 100-119 TFLOP/s instead of 60-80, with the loads of dy taken out nothing changes);
// two output groups per wave use every loaded quad of x twice.
//
// Workgroups go to the eight XCDs round-robin and each XCD has an L2 of its own, so the tiles are dealt
// out by XCD: the list of tiles, ordered so that the larger of the two operands changes slowest (output
// groups outermost when O >= K: dy is the larger one; input groups outermost otherwise), is cut into eight
// contiguous ranges, one per XCD.  The larger operand then enters one L2 only (two at a range boundary) and
// the smaller one each L2 once, where the plain order had every XCD stream both (40 % L2 misses at 7260
// rows).  Only locality depends on the round-robin placement, not the result.
constexpr int wgrad_max_split(int ob) { return kWgradMaxSplit / ob; }   // at most 60 KiB of LDS

template <bool SPLIT, bool DEEP, int OB, bool PARTS = false>
__global__ void __launch_bounds__(64 * (SPLIT ? wgrad_max_split(OB) : kWgradWaves), 1)
hot_linear_wgrad_kernel(LinearGradArgs a)
{
    extern __shared__ float partial[];   // SPLIT: [waves - 1][OB][kWgradPartials][64]
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: tile and trip counts stay scalar
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long k_groups = (K + 63) / 64;
    const long o_tiles = ((O + 15) / 16 + OB - 1) / OB, tiles = k_groups * o_tiles, per_xcd = (tiles + kXcds - 1) / kXcds;
    const long xcd = blockIdx.x % kXcds, nth = blockIdx.x / kXcds;      // nth workgroup of its XCD
    const long local = SPLIT ? nth : nth * kWgradWaves + wave;
    const long tile = xcd * per_xcd + local;
    // no such tile: a whole workgroup (SPLIT) or a whole wave of a kernel without barriers leaves
    if (local >= per_xcd || tile >= tiles) return;
    const bool outputs_outermost = O >= K;
    const long o0 = (outputs_outermost ? tile / k_groups : tile % o_tiles) * (16 * OB);
    const long k0 = (outputs_outermost ? tile % k_groups : tile / o_tiles) * 64;
    long o[OB];
    bool o_ok[OB];
#pragma unroll
    for (int b = 0; b < OB; ++b) {
        o[b] = o0 + 16 * b + n;
        o_ok[b] = o[b] < O;
    }
    const bool bias_tile = a.mu_b != nullptr && k0 == 0;     // uniform over the wave: this tile also owns its outputs' biases
    // PARTS: workgroup (x, y) owns the rows of part y only and leaves its sums in the workspace
    const long r_lo = PARTS ? (long)blockIdx.y * a.rows_per_part : 0;
    const long r_hi = PARTS ? (r_lo + a.rows_per_part < R ? r_lo + a.rows_per_part : R) : R;
    const long row_first = r_lo + (SPLIT ? (long)wave * kWgradRowsPerIter : 0);
    const long row_step = SPLIT ? (long)waves * kWgradRowsPerIter : kWgradRowsPerIter;

    // gm[b][t], gs[b][t]: the sums for the generator quad of inputs k0 + 16 j + 4 t .. + 3 of output o[b]
    f4 gm[OB][4], gs[OB][4];
    float gb_m[OB], gb_s[OB];
#pragma unroll
    for (int b = 0; b < OB; ++b) {
#pragma unroll
        for (int t = 0; t < 4; ++t) gm[b][t] = gs[b][t] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        gb_m[b] = gb_s[b] = 0.0f;
    }
    const long k_lane = k0 + 4 * n;          // as an A lane: the four inputs k_lane .. k_lane + 3 of a row, one 16-byte load
    const bool k_lane_ok = k_lane < K;

    for (int s = 0; s < a.s_loc; ++s) {
        const float *xs = a.x + (size_t)s * (size_t)a.x_sample_stride;
        const float *dys = a.dy + (size_t)s * (size_t)R * (size_t)O;
        // matrix instruction i of a row block takes element i of every lane's four inputs, so P[.][i] collects
        // the inputs k0 + 4 m + i (m = 0..15) and register c of P[.][i] is input k0 + 16 j + 4 c + i: the four
        // P[.][.][c] are the four consecutive inputs of one generator quad
        Acc16x16 mm[OB][4], mm_b[OB];
        // Whole blocks of 16 rows first, with nothing in the loop but the loads, the offset increments and the
        // matrix instructions: lanes outside the layer (o >= O, inputs >= K) read a valid address instead, which
        // only reaches rows and columns of P that are never stored.  The last, partial block is predicated per
        // row: rows beyond the last one must contribute zeros, they are summed over.
        constexpr int Q = kWgradRowsPerIter / 4;
        long pd[OB][Q], px[Q];      // offsets, not pointers: the loads stay global loads
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int b = 0; b < OB; ++b) pd[b][q] = (row_first + 4 * q + j) * O + (o_ok[b] ? o[b] : O - 1);
            px[q] = (row_first + 4 * q + j) * a.ldx + (k_lane_ok ? k_lane : 0);
        }
        const long d_step = row_step * O, x_step = row_step * a.ldx;
        const long full = r_hi - row_first >= kWgradRowsPerIter ? (r_hi - kWgradRowsPerIter - row_first) / row_step + 1 : 0;
        auto multiply = [&](const float (&bv)[OB][Q], const f4 (&av)[Q]) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int b = 0; b < OB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        mm[b][i].mac(av[q][i], bv[b][q]);
            if (bias_tile) {             // column sums of dy: the same contraction against ones
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int b = 0; b < OB; ++b) mm_b[b].mac(1.0f, bv[b][q]);
            }
        };
        if constexpr (DEEP) {
            // Two register sets of operands.  Every fetch is unconditional (behind a branch around loads the
            // compiler waits for all of them at the join): past the last whole block the offsets stop moving
            // and that block is simply read again.
            float bA[OB][Q], bB[OB][Q];
            f4 aA[Q], aB[Q];
            long fetched = 0;
            auto fetch = [&](float (&bv)[OB][Q], f4 (&av)[Q]) {
                ++fetched;
                const long dd = fetched < full ? d_step : 0, dx = fetched < full ? x_step : 0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
#pragma unroll
                    for (int b = 0; b < OB; ++b) {
                        bv[b][q] = dys[pd[b][q]];
                        pd[b][q] += dd;
                    }
                    av[q] = load4<true, false>(xs + px[q]);
                    px[q] += dx;
                }
            };
            if (full > 0) {
                fetch(bA, aA);
                for (long it = 0; it < full; it += 2) {
                    fetch(bB, aB);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(bA, aA);
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(bA, aA);
                    __builtin_amdgcn_sched_barrier(0);
                    if (it + 1 < full) multiply(bB, aB);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {        // on to the partial block
#pragma unroll
                    for (int b = 0; b < OB; ++b) pd[b][q] += d_step;
                    px[q] += x_step;
                }
            }
        } else {
            for (long it = 0; it < full; ++it) {
                float bv[OB][Q];
                f4 av[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
#pragma unroll
                    for (int b = 0; b < OB; ++b) {
                        bv[b][q] = dys[pd[b][q]];
                        pd[b][q] += d_step;
                    }
                    av[q] = load4<true, false>(xs + px[q]);
                    px[q] += x_step;
                }
                __builtin_amdgcn_sched_barrier(0);      // all loads first, one wait
                multiply(bv, av);
            }
        }
        const long rb = row_first + full * row_step;
        if (rb < r_hi) {
            float bv[OB][Q];
            f4 av[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const bool r_ok = rb + 4 * q + j < r_hi;
#pragma unroll
                for (int b = 0; b < OB; ++b) bv[b][q] = r_ok ? dys[pd[b][q]] : 0.0f;
                av[q] = r_ok ? load4<true, false>(xs + px[q]) : f4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            multiply(bv, av);
        }
        const MfmaSettled settled;
        f4 P[OB][4], Pb[OB];
#pragma unroll
        for (int b = 0; b < OB; ++b) {
#pragma unroll
            for (int i = 0; i < 4; ++i) P[b][i] = mm[b][i].read(settled);
            Pb[b] = mm_b[b].read(settled);
        }
        if (row_first < r_hi) {          // a wave without rows has nothing to add (uniform over the wave)
#pragma unroll
            for (int b = 0; b < OB; ++b) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const long col = k0 + 16 * j + 4 * t;
                    if (o_ok[b] && col < K) {
                        const f4 e = eps_quad(a.weight_quad0 + ((o[b] * K + col) >> 2), s, a.rng);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            gm[b][t][c] += P[b][c][t];
                            gs[b][t][c] = __builtin_fmaf(P[b][c][t], e[c], gs[b][t][c]);
                        }
                    }
                }
                if (bias_tile && o_ok[b]) {      // every register of Pb holds sum_r dy_s[r][o]
                    const f4 e = eps_quad(a.bias_quad0 + (o[b] >> 2), s, a.rng);
                    gb_m[b] += Pb[b][0];
                    gb_s[b] = __builtin_fmaf(Pb[b][0], pick4(e, (int)(o[b] & 3)), gb_s[b]);
                }
            }
        }
    }

    if constexpr (SPLIT) {
        if (wave > 0) {
#pragma unroll
            for (int b = 0; b < OB; ++b) {
                float *mine = partial + (size_t)((wave - 1) * OB + b) * kWgradPartials * 64 + lane;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        mine[(t * 4 + c) * 64] = gm[b][t][c];
                        mine[(16 + t * 4 + c) * 64] = gs[b][t][c];
                    }
                mine[32 * 64] = gb_m[b];
                mine[33 * 64] = gb_s[b];
            }
        }
        __syncthreads();
        if (wave != 0) return;
        for (int v = 1; v < waves; ++v)
#pragma unroll
            for (int b = 0; b < OB; ++b) {
                const float *theirs = partial + (size_t)((v - 1) * OB + b) * kWgradPartials * 64 + lane;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        gm[b][t][c] += theirs[(t * 4 + c) * 64];
                        gs[b][t][c] += theirs[(16 + t * 4 + c) * 64];
                    }
                gb_m[b] += theirs[32 * 64];
                gb_s[b] += theirs[33 * 64];
            }
    }

    // A lane holds the 16 consecutive inputs k0 + 16 j .. + 15 of its output: the four lanes of an output
    // exchange quads so that store t covers the 64 contiguous bytes k0 + 16 t .. + 15 of every row.
#pragma unroll
    for (int b = 0; b < OB; ++b) {
        transpose_quads_over_j(gm[b], j, n);
        transpose_quads_over_j(gs[b], j, n);
        if constexpr (PARTS) {          // the raw sums of this part; hot_linear_wgrad_finish_kernel adds the parts up
            const long per = O * K + ((O + 3) & ~3L);       // a multiple of 4 floats: quads stay 16-byte aligned
            float *mine = a.ws + (size_t)blockIdx.y * 2 * (size_t)per;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const long col = k0 + 16 * t + 4 * j;
                if (o_ok[b] && col < K) {
                    store4<true, false>(mine + o[b] * K + col, gm[b][t]);
                    store4<true, false>(mine + per + o[b] * K + col, gs[b][t]);
                }
            }
            if (bias_tile && j == 0 && o_ok[b]) {
                mine[O * K + o[b]] = gb_m[b];
                mine[per + O * K + o[b]] = gb_s[b];
            }
            continue;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const long col = k0 + 16 * t + 4 * j;
            if (o_ok[b] && col < K) {
                const long at = o[b] * K + col;
                const f4 m4 = load4<true, false>(a.mu_w + at), sd4 = load4<true, false>(a.sigma_w + at);
                f4 om, os;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float u, v;
                    finish_pair(gm[b][t][c], gs[b][t][c], m4[c], sd4[c], (float)a.g, (float)a.k, u, v);
                    om[c] = u;
                    os[c] = v;
                }
                store4<true, false>(a.gmu_w + at, om);
                store4<true, false>(a.gsig_w + at, os);
            }
        }
        if (bias_tile && j == 0 && o_ok[b]) {
            float u, v;
            finish_pair(gb_m[b], gb_s[b], a.mu_b[o[b]], a.sigma_b[o[b]], (float)a.g, (float)a.k, u, v);
            a.gmu_b[o[b]] = u;
            a.gsig_b[o[b]] = v;
        }
    }
}

// Adds the parts of a PARTS run in their order and finishes the gradients: thread q owns quad q of the
// O*K weights (K is a multiple of 4, so a quad never leaves its row), the first O threads also one bias.
__global__ void __launch_bounds__(256)
hot_linear_wgrad_finish_kernel(LinearGradArgs a, int parts)
{
    const long K = a.in_features, O = a.out_features, per = O * K + ((O + 3) & ~3L);
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q < O * K / 4) {
        f4 gm = {0.0f, 0.0f, 0.0f, 0.0f}, gs = gm;
        for (int p = 0; p < parts; ++p) {
            const float *theirs = a.ws + (size_t)p * 2 * (size_t)per;
            const f4 u = load4<true, false>(theirs + 4 * q), v = load4<true, false>(theirs + per + 4 * q);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                gm[c] += u[c];
                gs[c] += v[c];
            }
        }
        const f4 m4 = load4<true, false>(a.mu_w + 4 * q), sd4 = load4<true, false>(a.sigma_w + 4 * q);
        f4 om, os;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float u, v;
            finish_pair(gm[c], gs[c], m4[c], sd4[c], (float)a.g, (float)a.k, u, v);
            om[c] = u;
            os[c] = v;
        }
        store4<true, false>(a.gmu_w + 4 * q, om);
        store4<true, false>(a.gsig_w + 4 * q, os);
    }
    if (a.mu_b != nullptr && q < O) {
        float gm = 0.0f, gs = 0.0f;
        for (int p = 0; p < parts; ++p) {
            const float *theirs = a.ws + (size_t)p * 2 * (size_t)per;
            gm += theirs[O * K + q];
            gs += theirs[per + O * K + q];
        }
        float u, v;
        finish_pair(gm, gs, a.mu_b[q], a.sigma_b[q], (float)a.g, (float)a.k, u, v);
        a.gmu_b[q] = u;
        a.gsig_b[q] = v;
    }
}

// The PARTS run: every tile once per part (grid y), then the finish kernel.
template <int OB>
void wgrad_go_parts(long tiles, int waves, int parts, hipStream_t s, const LinearGradArgs &a)
{
    const long per_xcd = (tiles + kXcds - 1) / kXcds;
    const size_t lds = (size_t)(waves - 1) * OB * kWgradPartials * 64 * sizeof(float);
    hot_linear_wgrad_kernel<true, true, OB, true><<<dim3((unsigned)(kXcds * per_xcd), (unsigned)parts), dim3(64 * waves), lds, s>>>(a);
    const long quads = a.out_features * a.in_features / 4;
    const long threads = quads > a.out_features ? quads : a.out_features;
    hot_linear_wgrad_finish_kernel<<<dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s>>>(a, parts);
}

template <bool SPLIT, bool DEEP, int OB>
void wgrad_go(long tiles, int waves, hipStream_t s, const LinearGradArgs &a)
{
    const long per_xcd = (tiles + kXcds - 1) / kXcds;      // the kernel deals the tiles out by XCD
    const long wgs = SPLIT ? per_xcd : (per_xcd + kWgradWaves - 1) / kWgradWaves;
    const size_t lds = SPLIT ? (size_t)(waves - 1) * OB * kWgradPartials * 64 * sizeof(float) : 0;
    hot_linear_wgrad_kernel<SPLIT, DEEP, OB><<<dim3((unsigned)(kXcds * wgs)), dim3(64 * waves), lds, s>>>(a);
}

// ---------------------------------------------------------------------------------
// Weight gradients of large layers.  The kernel above gives a wave a tile of 16-32 outputs x 64 inputs, about 10
// flops per byte it loads: at thousands of rows the second-level caches cannot feed that (the matrix pipes were 42 %
// busy).  Here a workgroup of four waves owns 128 inputs x 128 outputs and takes 16 rows of x and of dy at a time.
// Every element is loaded and cut into its three bf16 pieces ONCE in the workgroup (by a lane that holds eight rows of two
// columns, i.e. whole operands of the matrix instruction) and shared through LDS; a wave multiplies 64 inputs x 64 outputs as
// 2 x 2 blocks with x as the A operand and dy as the B operand, so result registers 4 q .. 4 q + 3 of a lane are the inputs
// 8 q + 4 (lane / 32) .. + 3 of output lane % 32: one generator quad, as above.  Two samples have accumulators of their own (128
// registers), and two workgroups share a compute unit and cover each other's draws.
// What bounds it: matrix and vector instructions, which overlap only in part, at the clock that the card's power leaves (1024 x
// 8192^2 x 2: matrix pipes 55-60 % busy at 1.7 GHz, 211 TFLOP/s of fp32 work per further row), and at a few hundred rows the draw
// (43 us of 196 at 300 x 2160 x 8640 x 2) and the 16 bytes per weight of mu, sigma and the gradients.  Measured against its
// predecessor, which sent fp32 rows straight into LDS, had every wave cut its operands itself (176 instead of 88 vector instructions per
// 24 matrix instructions), and waited for memory sixteen times per tile on the way out, in turn, nothing else between the calls: 1024 x 8192^2 x 2 1691 -> 1506 us
// (between the other kernels of a pass, at the clock that those leave, 1790 -> 1660 to 1700), 160 x 8192^2 x 2 522 -> 402, 300 x 2160 x 8640 x 2 222 -> 196,
// 200 x 4096^2 x 2 157 -> 126; of 1100 layers of 140 to 2000 tiles, edges of every width among them, 0.86 of the time in the middle and none slower, though blocks of 32 x 32
// outside the layer are multiplied too.  21 registers are spilled (72 bytes of scratch per lane).  On the way (1024 x 8192^2 x 2): the same with the vector instructions where the
// scheduler put them, in rows, 1680; with fixed places 1650; rows of x and dy sent for two steps ahead 1560; the way out
// without waits 1502.  Three sets of rows under way instead of two (steps in threes): 1566, with 51 registers spilled.
// ---------------------------------------------------------------------------------
constexpr int kTileSide = 128;        // inputs and outputs per workgroup
constexpr int kTileRows = 16;         // rows per step
constexpr int kTileBuffer = 2 * kTileSide * kTileRows * 6;      // bytes of the cut columns of a step: four blocks of 32 columns of x, four of dy, three planes each
constexpr int kTurnPitch = 36;        // floats per row of a wave's 32 x 32 block on its way out (16-byte aligned rows)


// The weight gradients of a wave's 64 inputs x 64 outputs (from k0, o0) that the tile kernel left as NaN, again from fp32 products on
// the matrix instruction: an infinite factor, and one whose pieces overflow, leaves NaN where those give infinity or a number.
// Rows straight from memory, a block of 32 x 32 at a time and only those that hold a NaN.  Called by whole waves.  What it takes is
// bounded by the layer: every gradient again (a row of dy that is NaN) makes 1024 x 2560 x 2560 x 2 samples 0.21 -> 1.4 ms, 300 x 2160 x
// 8640 x 2 0.24 -> 1.4, 2048 x 4096 x 4096 x 2 0.8 -> 5.5 (a lane to each sum and a load to each factor: 36, 17 and 159).
__device__ __forceinline__ void wgrad_tile_again(const LinearGradArgs &a, long o0, long k0)
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const long K = a.in_features, O = a.out_features;
    const int R = (int)a.rows;
#pragma unroll 1
    for (int n = 0; n < 4; ++n) {
        const long k = k0 + 32 * (n >> 1), o = o0 + 32 * (n & 1) + l32;
        auto inside = [&](int q) { return o < O && k + 8 * q + 4 * half < K; };
        auto at = [&](int q) { return o * K + k + 8 * q + 4 * half; };
        unsigned bad = 0;                       // bit 4 q + c: weight (o, k + 8 q + 4 half + c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (inside(q)) {
                const f4 om = load4<true, false>(a.gmu_w + at(q)), os = load4<true, false>(a.gsig_w + at(q));
#pragma unroll
                for (int c = 0; c < 4; ++c) bad |= (om[c] != om[c] || os[c] != os[c] ? 1u : 0u) << (4 * q + c);
            }
        if (__builtin_amdgcn_ballot_w64(bad != 0) == 0) continue;
        float gm[16] = {}, gs[16] = {};
#pragma unroll 1
        for (int s = 0; s < a.s_loc; ++s) {
            // (columns outside the layer and rows behind the last take the nearest ones; the latter count as zeros)
            const float *x = a.x + (size_t)s * (size_t)a.x_sample_stride + (size_t)(k + l32 < K ? k + l32 : K - 1);
            const float *dy = a.dy + (size_t)s * (size_t)R * (size_t)O + (size_t)(o < O ? o : O - 1);
            Acc32x32 m;
#pragma unroll 1
            for (int r0 = half; r0 < R + half; r0 += 16) {
                float xv[8], dv[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int r = r0 + 2 * t, from = r < R ? r : R - 1;
                    xv[t] = x[(size_t)from * (size_t)a.ldx];
                    dv[t] = dy[(size_t)from * (size_t)O];
                    xv[t] = r < R ? xv[t] : 0.0f;
                    dv[t] = r < R ? dv[t] : 0.0f;
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) m.mac(xv[t], dv[t]);
            }
            const MfmaSettled settled;
            const f16v p = m.read(settled);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (inside(q)) {
                    const f4 e = eps_quad(a.weight_quad0 + (at(q) >> 2), s, a.rng);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        gm[4 * q + c] += p[4 * q + c];
                        gs[4 * q + c] = __builtin_fmaf(p[4 * q + c], e[c], gs[4 * q + c]);
                    }
                }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (inside(q)) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (bad >> (4 * q + c) & 1u)
                        finish_pair(gm[4 * q + c], gs[4 * q + c], a.mu_w[at(q) + c], a.sigma_w[at(q) + c], (float)a.g, (float)a.k, a.gmu_w[at(q) + c], a.gsig_w[at(q) + c]);
            }
    }
}

template <int N>
struct Number {
    static constexpr int value = N;
};

// lds: three buffers of kTileBuffer bytes, the cut columns of x and behind them those of dy.  Returns whether the wave left a NaN.
__device__ __forceinline__ bool wgrad_tile_body(const LinearGradArgs &a, lds_char *lds, long o0, long k0)
{
    constexpr int WK = 2;                                         // 2 x 2 waves of 64 inputs x 64 outputs
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int wk = wave % WK, wo = wave / WK;
    const long K = a.in_features, O = a.out_features, R = a.rows;

    const bool bias_tile = a.mu_b != nullptr && k0 == 0;          // this workgroup also sums dy over the rows

    // As a loading wave: waves 0 and 1 take the even and the odd rows of x, waves 2 and 3 those of dy; a lane two columns, eight
    // rows of a step, which make whole operands of the matrix instruction.  Rows behind the last lie outside the window and
    // arrive as zeros; what columns outside the layer bring is never stored.
    const bool of_x = wave < 2;
    const int odd = wave & 1;
    const unsigned pitch = (unsigned)((of_x ? a.ldx : O) * 4);
    const unsigned bytes = (unsigned)((of_x ? (R - 1) * a.ldx + K : R * O) * 4);
    const float *const from = of_x ? a.x : a.dy;
    const size_t from_stride = of_x ? (size_t)a.x_sample_stride : (size_t)R * (size_t)O;
    const unsigned lane_off = (unsigned)(((of_x ? k0 : o0) + 2 * lane) * 4);
    // Column m of a block of 32 lies in slot m / 2 of its plane's half if m is even, 16 + (m / 2 ^ 2) if odd: sixteen lanes then write a
    // run of 256 bytes, and the lanes that a 16-byte read serves together (0-3, 12-15, 20-27 and the others; found by counting
    // conflicts, 33 % of the LDS cycles with ^ 12, 1 % with ^ 2) meet all banks.
    const int put_block = (of_x ? 0 : kTileBuffer / 2) + (lane >> 4) * 3072 + odd * 512;
    const int put_at = put_block + (lane & 15) * 16, put_at1 = put_block + (16 + ((lane & 15) ^ 2)) * 16;
    const int slot = (l32 & 1) ? 16 + ((l32 >> 1) ^ 2) : l32 >> 1;
    const int x_get = wk * 2 * 3072 + half * 512 + slot * 16, d_get = kTileBuffer / 2 + wo * 2 * 3072 + half * 512 + slot * 16;
    // steps of 16 rows, in pairs (the last one may run on zeros); those of the second sample follow those of the first without a gap
    const int rows = (int)R, steps = (rows + 2 * kTileRows - 1) / (2 * kTileRows) * 2;

    f2 raw[2][8];                // the rows of two steps under way
    auto load = [&](int i, f2 (&raw)[8], int s0, bool two) {
        const bool second = i >= steps;
        const int row = second ? (two ? (i - steps) * kTileRows : rows) : i * kTileRows;
        const window_t win = window(from + (size_t)(two && second ? s0 + 1 : s0) * from_stride, bytes);
        const unsigned at = (unsigned)((row < rows ? row : rows) + odd) * pitch;
#pragma unroll
        for (int p = 0; p < 8; ++p) raw[p] = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(win, (int)(lane_off + (at + 2 * p * pitch)), 0, 0));
    };
    // Cutting, in sixteen turns (see split2_bf16): pair n % 4 of rows of column n / 4, first its first piece and remainders, then the rest;
    // behind a column's last turn its three operands go to LDS.
    unsigned p1[4], p2[4], p3[4];
    float r0, r1;
    auto cut = [&](int turn, const f2 (&raw)[8], lds_char *buffer) {
        const int n = turn >> 1, e = n >> 2, j = n & 3;
        if ((turn & 1) == 0) {
            p1[j] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{raw[2 * j][e], raw[2 * j + 1][e]}, bf2));
            r0 = raw[2 * j][e] - __builtin_bit_cast(float, p1[j] << 16);
            r1 = raw[2 * j + 1][e] - __builtin_bit_cast(float, p1[j] & 0xFFFF0000u);
            return;
        }
        p2[j] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{r0, r1}, bf2));
        const float s0 = r0 - __builtin_bit_cast(float, p2[j] << 16), s1 = r1 - __builtin_bit_cast(float, p2[j] & 0xFFFF0000u);
        p3[j] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{s0, s1}, bf2));
        if (j < 3) return;
        lds_char *const to = buffer + (e ? put_at1 : put_at);
        *(lds_bf8 *)to = __builtin_bit_cast(bf8, u4{p1[0], p1[1], p1[2], p1[3]});
        *(lds_bf8 *)(to + 1024) = __builtin_bit_cast(bf8, u4{p2[0], p2[1], p2[2], p2[3]});
        *(lds_bf8 *)(to + 2048) = __builtin_bit_cast(bf8, u4{p3[0], p3[1], p3[2], p3[3]});
    };
    auto add_columns = [&](const f2 (&raw)[8], float (&sb)[2]) {
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int e = 0; e < 2; ++e) sb[e] += raw[p][e];
    };
    bf8 av[2][3], bv[2][3];
    auto get_x = [&](int pl, const lds_char *buffer) {
#pragma unroll
        for (int i = 0; i < 2; ++i) av[i][pl] = *(const volatile lds_bf8 *)(buffer + x_get + i * 3072 + pl * 1024);
    };
    auto get_d = [&](int pl, const lds_char *buffer) {
#pragma unroll
        for (int j = 0; j < 2; ++j) bv[j][pl] = *(const volatile lds_bf8 *)(buffer + d_get + j * 3072 + pl * 1024);
    };
    // One step on tile i.  Barrier: every wave has read tile i - 1, and tile i + 1 is in LDS.  Beside the products, tile i + 2 is cut and
    // put where tile i - 1 was, tile i + 4 is sent for, and every piece of an operand is read as soon as the last product that
    // needs its predecessor has been issued, so that one set of registers suffices.  The six products come as everywhere, the three small
    // ones first and the large one last (with a3 b1 behind it, which let every piece be read a step ahead, the sums were 1.004 times as far from 64 bits on 1100
    // layers, 1.02 on those of 136 rows, and 0.5 % faster); a2 b2 is first of all, since it is the one that needs neither a1 nor b1, which are read
    // meanwhile.  The order is fixed by hand, a few vector instructions behind every matrix instruction: left to the scheduler they
    // stand in rows, and the matrix pipes idle behind them.
    auto step = [&](f2 (&raw)[8], int i, const lds_char *now, const lds_char *next, lds_char *free, int s0, bool two, Acc32x32 (&mm)[2][2], float (&sb)[2][2]) {
        constexpr int PA[6] = {1, 0, 2, 1, 0, 0}, PB[6] = {1, 2, 0, 0, 1, 0};
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 24; ++n) {
            const int g = n >> 2, bi = n >> 1 & 1, bj = n & 1;
            mm[bi][bj].mac(av[bi][PA[g]], bv[bj][PB[g]]);
            if (n < 16) cut(n, raw, free);
            if (n == 0) {
                get_x(0, now);
                get_d(0, now);
            }
            if (n == 8) get_d(2, next);
            if (n == 12) get_x(2, next);
            if (n == 16) {
                if (bias_tile && !of_x) {
                    if (i + 2 < steps) add_columns(raw, sb[0]);
                    else add_columns(raw, sb[1]);
                }
                load(i + 4, raw, s0, two);
                get_x(1, next);
            }
            if (n == 20) get_d(1, next);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the steps i .. i_end - 1 of a sample (an even number), `at` the buffer of step i
    auto all_steps = [&](int i, int i_end, int &at, int s0, bool two, Acc32x32 (&mm)[2][2], float (&sb)[2][2]) {
#pragma unroll 1
        for (; i < i_end; i += 2) {
            const int b1 = at == 2 * kTileBuffer ? 0 : at + kTileBuffer, b2 = b1 == 2 * kTileBuffer ? 0 : b1 + kTileBuffer;
            step(raw[0], i, lds + at, lds + b1, lds + b2, s0, two, mm, sb);
            step(raw[1], i + 1, lds + b1, lds + b2, lds + at, s0, two, mm, sb);
            at = b2;
        }
    };

    // Two samples at a time, each with accumulators of its own: P_s = sum_r x_s[r] (x) dy_s[r], whose sum and whose sum
    // weighted with eps_s leave together (one draw per sample and weight).  Further pairs of samples add to what the
    // pairs before left in the gradient arrays (the same thread holds the same weights every time); the last pair
    // applies the scale and the KL part.
    float gb_m = 0.0f, gb_s = 0.0f;
    float special = 0.0f;                    // NaN once this lane has left a NaN (or an infinity, which only costs a look) in the last pass
    lds_float *const mine = (lds_float *)lds + wave * 64 * kTurnPitch;         // for turning a block of either sample on its way out
    for (int s0 = 0; s0 < a.s_loc; s0 += 2) {
        const bool two = s0 + 1 < a.s_loc, first = s0 == 0, last = s0 + 2 >= a.s_loc;
        Acc32x32 m0[2][2], m1[2][2];
        float sb[2][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};         // (tile 0 counts for sample s0, whose steps follow)
        // (the accumulators are not alive yet: four steps' rows are sent for at once)
        f2 first2[2][8];
        load(0, first2[0], s0, two);
        load(1, first2[1], s0, two);
        load(2, raw[0], s0, two);
        load(3, raw[1], s0, two);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int turn = 0; turn < 16; ++turn) cut(turn, first2[i], lds + i * kTileBuffer);
            if (bias_tile && !of_x) add_columns(first2[i], sb[0]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        get_x(1, lds);
        get_d(1, lds);
        get_d(2, lds);
        get_x(2, lds);
        int at = 0;
        all_steps(0, steps, at, s0, two, m0, sb);
        if (two) all_steps(steps, 2 * steps, at, s0, two, m1, sb);
        everything_arrived_then_barrier();       // every wave is done with the buffers
        const MfmaSettled settled;
        special = 0.0f;                      // (not kept through the row loops)

        // Out: a block of 32 x 32 goes through the wave's own LDS (which executes a wave's instructions in order, so no barrier), after which
        // a lane holds quads of consecutive inputs, eight lanes 128 contiguous bytes of a row of the gradients.  Two quads at a time: their
        // eps are drawn, the products of both samples combined, the gradients finished and stored.  mu and sigma of the next two are
        // sent for ahead of the draw: loads and stores complete in order on this chip, so a load asked for where it is needed waits for
        // the stores before it (sixteen such waits, one behind the other, were most of the time at a few hundred rows).  All through
        // range-checked windows, without branches, behind which every outstanding access would have to be waited for.
        int ov = (int)o0 + 64 * wo, kv = (int)k0 + 64 * wk;
        asm volatile("" : "+v"(ov), "+v"(kv));         // (so that the addresses below are formed here, not ahead of the row loops)
        const int oe = __builtin_amdgcn_readfirstlane(ov), ke = __builtin_amdgcn_readfirstlane(kv);
        const long corner = (long)oe * K + ke;
        const unsigned win_bytes = (unsigned)(64 * K * 4);
        const window_t mu_win = window(a.mu_w + corner, win_bytes), sg_win = window(a.sigma_w + corner, win_bytes);
        const window_t gm_win = window(a.gmu_w + corner, win_bytes), gs_win = window(a.gsig_w + corner, win_bytes);
        const long quad_corner = a.weight_quad0 + (corner >> 2);
        // turn n: block n / 4 (inputs 32 (n / 8), outputs 32 (n / 4 % 2)), rows 8 (n % 4) .. + 7 of it
        auto offset = [&](int n) {
            const int row = 32 * (n >> 2 & 1) + 8 * (n & 3) + (lane >> 3), col = 32 * (n >> 3) + 4 * (lane & 7);
            return oe + row < (int)O && ke + col < (int)K ? (unsigned)((row * K + col) * 4) : kOutside;
        };
        auto finish = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value != 0;         // these are the only samples
            f4 m4[2], sd4[2], next_m4[2], next_sd4[2];
            auto ask = [&](int n) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    next_m4[e] = window_load4<false>(mu_win, offset(n + e));
                    next_sd4[e] = window_load4<false>(sg_win, offset(n + e));
                }
            };
            if (PLAIN || last) ask(0);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const f16v p0 = m0[b >> 1][b & 1].read(settled), p1 = m1[b >> 1][b & 1].read(settled);      // (p1 is zero without a second sample)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    *reinterpret_cast<lds_f4 *>(mine + l32 * kTurnPitch + 8 * q + 4 * half) = f4{p0[4 * q], p0[4 * q + 1], p0[4 * q + 2], p0[4 * q + 3]};
                    *reinterpret_cast<lds_f4 *>(mine + (32 + l32) * kTurnPitch + 8 * q + 4 * half) = f4{p1[4 * q], p1[4 * q + 1], p1[4 * q + 2], p1[4 * q + 3]};
                }
#pragma unroll 1
                for (int n = 4 * b; n < 4 * b + 4; n += 2) {
                    if (PLAIN || last) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            m4[e] = next_m4[e];
                            sd4[e] = next_sd4[e];
                        }
                        ask(n + 2 < 16 ? n + 2 : n);
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const unsigned off = offset(n + e);
                        const lds_float *const turned = mine + (8 * ((n + e) & 3) + (lane >> 3)) * kTurnPitch + 4 * (lane & 7);
                        const f4 q0 = *reinterpret_cast<const lds_f4 *>(turned), q1 = *reinterpret_cast<const lds_f4 *>(turned + 32 * kTurnPitch);
                        const long quad = quad_corner + (off >> 4);
                        const f4 e0 = eps_quad(quad, s0, a.rng);
                        f4 om = q0, os;
#pragma unroll
                        for (int c = 0; c < 4; ++c) os[c] = q0[c] * e0[c];
                        if (two) {
                            const f4 e1 = eps_quad(quad, s0 + 1, a.rng);
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                om[c] += q1[c];
                                os[c] = __builtin_fmaf(q1[c], e1[c], os[c]);
                            }
                        }
                        if (!PLAIN && !first) {
                            om += window_load4<false>(gm_win, off);
                            os += window_load4<false>(gs_win, off);
                        }
                        if (PLAIN || last) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                float pm, ps;
                                finish_pair(om[c], os[c], m4[e][c], sd4[e][c], (float)a.g, (float)a.k, pm, ps);
                                om[c] = pm;
                                os[c] = ps;
                            }
                        }
                        window_store4<false>(gm_win, off, om);
                        window_store4<false>(gs_win, off, os);
                        // (a product that is not finite shows in os)
                        const float look = __builtin_fmaf(os[3], 0.0f, __builtin_fmaf(os[2], 0.0f, __builtin_fmaf(os[1], 0.0f, os[0] * 0.0f)));
                        special += off != kOutside ? look : 0.0f;
                    }
                }
            }
        };
        if (first && last) finish(Number<1>());
        else finish(Number<0>());
        everything_arrived_then_barrier();
        if (bias_tile) {                         // the column sums of the even and of the odd rows meet in LDS
            lds_float *const sums = (lds_float *)lds;
            if (!of_x) {
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int e = 0; e < 2; ++e) sums[(n * 2 + odd) * kTileSide + 2 * lane + e] = sb[n][e];
            }
            everything_arrived_then_barrier();
            const long o = o0 + t;
            if (t < kTileSide && o < O) {
                const float t0 = sums[t] + sums[kTileSide + t];
                gb_m += t0;
                gb_s = __builtin_fmaf(t0, pick4(eps_quad(a.bias_quad0 + (o >> 2), s0, a.rng), (int)(o & 3)), gb_s);
                if (two) {
                    const float t1 = sums[2 * kTileSide + t] + sums[3 * kTileSide + t];
                    gb_m += t1;
                    gb_s = __builtin_fmaf(t1, pick4(eps_quad(a.bias_quad0 + (o >> 2), s0 + 1, a.rng), (int)(o & 3)), gb_s);
                }
            }
            everything_arrived_then_barrier();   // (the buffers go back to the rows of the next pair)
        }
    }
    if (bias_tile && t < kTileSide && o0 + t < O) {
        float p, r;
        finish_pair(gb_m, gb_s, a.mu_b[o0 + t], a.sigma_b[o0 + t], (float)a.g, (float)a.k, p, r);
        a.gmu_b[o0 + t] = p;
        a.gsig_b[o0 + t] = r;
    }
    return __builtin_amdgcn_ballot_w64(special != special) != 0;
}

__global__ void __launch_bounds__(256, 2)
hot_linear_wgrad_tile_kernel(LinearGradArgs a)
{
    constexpr int TK = kTileSide, TO = kTileSide;
    // (at the end every wave turns its blocks on their way out there)
    __shared__ __attribute__((aligned(16))) char buffers[3 * kTileBuffer];
    static_assert(3 * kTileBuffer >= 4 * 64 * kTurnPitch * 4, "two blocks of each wave");
    lds_char *const lds = (lds_char *)buffers;
    const long K = a.in_features, O = a.out_features;
    const long k_tiles = (K + TK - 1) / TK, o_tiles = (O + TO - 1) / TO;
    const long tiles = k_tiles * o_tiles, per_xcd = (tiles + kXcds - 1) / kXcds;
    const long xcd = blockIdx.x % kXcds, nth = blockIdx.x / kXcds;      // the tiles are dealt out by XCD as above
    const long tile = xcd * per_xcd + nth;
    if (nth >= per_xcd || tile >= tiles) return;          // the whole workgroup
    // The tile list runs through bands of eight rows of tiles, column by column inside a band, so that the 64 tiles an
    // XCD works on at a time are about 8 x 8 and share 16 columns of x and dy in its L2 (listed row by row they were
    // 2 x 32 and shared 34).
    const long band = tile / (8 * k_tiles), bands = o_tiles / 8;
    const long height = band < bands ? 8 : o_tiles - 8 * bands, within = tile - (band < bands ? band : bands) * 8 * k_tiles;
    const long o0 = (8 * (band < bands ? band : bands) + within % height) * TO;
    const long k0 = (within / height) * TK;
    if (wgrad_tile_body(a, lds, o0, k0)) {
        // (the arguments read once more, so that none is kept for this through the row loops; the last barrier's wait covers the wave's own stores)
        unsigned long long args = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
#ifdef __OPTIMIZE__       // (without optimisation nothing is kept anyhow, and the address is in no scalar register)
        asm volatile("" : "+s"(args));
#endif
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        wgrad_tile_again(*reinterpret_cast<const LinearGradArgs *>(args), o0 + 64 * (wave / 2), k0 + 64 * (wave % 2));
    }
}

// Whether the kernel above can address this problem (its windows take 32-bit byte offsets).  Any number of outputs: a quad of dy
// that reaches over the end of a row brings columns that are never stored, loads need an alignment of 4 bytes only, and the check at
// the end of the window is per 4 bytes.  (Where such layers take it: wgrad_shape.)
inline bool wgrad_tile_fits(const hot_linear_desc *d)
{
    const unsigned long long lim = 0xFFFFFFF0ull;
    return (unsigned long long)((d->rows + kTileRows) * d->ldx + d->in_features) * 4 < lim &&
           (unsigned long long)(d->rows + kTileRows) * d->out_features * 4 < lim;
}

inline long wgrad_tile_count(const hot_linear_desc *d)
{
    return ((d->in_features + kTileSide - 1) / kTileSide) * ((d->out_features + kTileSide - 1) / kTileSide);
}

void wgrad_tile_go(hipStream_t s, const LinearGradArgs &a, long tiles)
{
    const long per_xcd = (tiles + kXcds - 1) / kXcds;
    hot_linear_wgrad_tile_kernel<<<dim3((unsigned)(kXcds * per_xcd)), dim3(256), 0, s>>>(a);
}

// ---------------------------------------------------------------------------------
// Weight gradients of layers with few tiles and many rows, given a workspace: the rows are cut into parts for different
// workgroups, as in the PARTS runs of the first kernel above, but the products are formed from bf16 pieces (see
// split2_bf16), and what a part leaves in the workspace is the raw product P_s of each sample: eps is drawn once per
// weight and sample by the finish kernel instead of once per part and wave.
//
// A wave owns a tile of 128 x 64 (BIG x SMALL blocks of 32; XBIG: 128 inputs x 64 outputs, else 64 inputs x 128 outputs) and
// takes 16 rows at a time, the four waves of a workgroup round-robin over the rows of its part.  Lane (l32, half) reads rows
// 8 half .. 8 half + 7 of the step at the four (two) consecutive columns 4 l32 .. (2 l32 ..) of the larger (smaller) operand: whole rows of
// 512 (256) contiguous bytes per load, and element i of what it read is the lane's operand of block i, so that nothing
// passes through LDS and no wave waits for another before the end.  Two waves share a SIMD (128 accumulators and 60
// registers of pieces each) and one's cutting into pieces (about 1060 vector cycles a step) runs beside the other's
// matrix instructions (1540).  The larger operand is cut first and its next rows are sent for at once, the smaller
// one block by block.  At the end the waves' tiles are added through LDS in a fixed order.
// ---------------------------------------------------------------------------------
constexpr int kRowPartWaves = 4;
constexpr int kRowPartRows = 16;                          // rows per wave and step
constexpr int kRowPartBig = 4, kRowPartSmall = 2;         // blocks of 32 per side of a wave's tile

template <int N>
struct Floats;
template <>
struct Floats<2> {
    typedef f2 V;
    static __device__ __forceinline__ V load(window_t w, unsigned off) { return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(w, (int)off, 0, 0)); }
};
template <>
struct Floats<4> {
    typedef f4 V;
    static __device__ __forceinline__ V load(window_t w, unsigned off) { return window_load4<false>(w, off); }
};

// floats of one part's share of the workspace: per sample the weights, then the biases (a multiple of four, so that quads stay aligned)
inline __host__ __device__ long row_part_floats(long K, long O, int s_loc) { return (O * K + ((O + 3) & ~3L)) * s_loc; }

// (XBIG spills seven registers, 32 bytes of scratch per lane.)
template <bool XBIG>
__global__ void __launch_bounds__(64 * kRowPartWaves, 2)
hot_linear_wgrad_row_parts_kernel(LinearGradArgs a, int parts, int chunk)
{
    constexpr int NB = kRowPartBig, NS = kRowPartSmall, KB = XBIG ? NB : NS, OB = XBIG ? NS : NB;
    constexpr int TK = 32 * KB, TO = 32 * OB, PITCH = TK + 4;
    typedef Floats<NB> LB;
    typedef Floats<NS> LS;
    __shared__ __attribute__((aligned(16))) float turn[kRowPartWaves][32 * PITCH];
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long k_tiles = (K + TK - 1) / TK, o_tiles = (O + TO - 1) / TO, tiles = k_tiles * o_tiles;
    // the list of (part, sample, tile), tiles changing fastest, is cut into one contiguous range per XCD: workgroups that read the
    // same rows share an L2
    const long all = tiles * a.s_loc * parts, per_xcd = (all + kXcds - 1) / kXcds;
    const long xcd = blockIdx.x % kXcds, nth = blockIdx.x / kXcds, item = xcd * per_xcd + nth;
    if (nth >= per_xcd || item >= all) return;          // the whole workgroup
    const long tile = item % tiles, ps = item / tiles;
    const int s = (int)(ps % a.s_loc);
    const long part = ps / a.s_loc;
    const long o0 = (O >= K ? tile / k_tiles : tile % o_tiles) * TO, k0 = (O >= K ? tile % k_tiles : tile / o_tiles) * TK;
    const long r_lo = part * a.rows_per_part, r_hi = r_lo + a.rows_per_part < R ? r_lo + a.rows_per_part : R;
    const bool bias_tile = a.mu_b != nullptr && k0 == 0;

    // Windows end behind the part's last row, so that rows beyond it arrive as zeros.  (Columns beyond the layer read some other
    // element of the operand, which only reaches accumulators that are never stored.)
    const window_t x_win = window(a.x + (size_t)s * (size_t)a.x_sample_stride, (unsigned)(((r_hi - 1) * a.ldx + K) * 4));
    const window_t d_win = window(a.dy + (size_t)s * (size_t)R * (size_t)O, (unsigned)(r_hi * O * 4));
    const window_t b_win = XBIG ? x_win : d_win, s_win = XBIG ? d_win : x_win;
    const unsigned x_pitch = (unsigned)(a.ldx * 4), d_pitch = (unsigned)(O * 4);
    const unsigned b_pitch = XBIG ? x_pitch : d_pitch, s_pitch = XBIG ? d_pitch : x_pitch;
    const unsigned row0 = (unsigned)(r_lo + kRowPartRows * wave + 8 * half);
    unsigned b_off = row0 * b_pitch + (unsigned)((XBIG ? k0 : o0) * 4 + 4 * NB * l32);
    unsigned s_off = row0 * s_pitch + (unsigned)((XBIG ? o0 : k0) * 4 + 4 * NS * l32);

    // The instruction rounds its accumulations downwards (the mean error is -1.4e-7 of the mean magnitude at 8191 rows, for sums of either
    // sign), and what all parts and samples lose in one direction adds up.  So every other wave takes its products with the
    // opposite sign, and its tile is subtracted.
    const float sign = wave & 1 ? -1.0f : 1.0f;
    float col_sum[OB];
#pragma unroll
    for (int j = 0; j < OB; ++j) col_sum[j] = 0.0f;
    typename LB::V br[8];
    typename LS::V sr[8];
    auto ask_big = [&] {
#pragma unroll
        for (int t = 0; t < 8; ++t) br[t] = LB::load(b_win, b_off + (unsigned)t * b_pitch);
        b_off += (unsigned)(kRowPartRows * kRowPartWaves) * b_pitch;
    };
    auto ask_small = [&] {
#pragma unroll
        for (int t = 0; t < 8; ++t) sr[t] = LS::load(s_win, s_off + (unsigned)t * s_pitch);
        s_off += (unsigned)(kRowPartRows * kRowPartWaves) * s_pitch;
    };
    ask_big();
    ask_small();
    // A long part is added up in chunks of `chunk` rows (a multiple of 64), each into accumulators of its own and then to what the
    // chunks before left in the workspace (the same thread holds the same sums every time).  What is sent for beyond the end
    // of a chunk are the first rows of the next.
    for (long c_lo = r_lo; c_lo < r_hi; c_lo += chunk) {
        const long c_hi = c_lo + chunk < r_hi ? c_lo + chunk : r_hi;
        Acc32x32 mm[NB][NS];
        for (long r = c_lo + kRowPartRows * wave; r < c_hi; r += kRowPartRows * kRowPartWaves) {       // uniform over the wave
            if (bias_tile) {
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int j = 0; j < OB; ++j) col_sum[j] += XBIG ? sr[t][j % NS] : br[t][j];
            }
            bf8 b1[NB], b2[NB], b3[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i)
                split8_bf16(f4{br[0][i], br[1][i], br[2][i], br[3][i]}, f4{br[4][i], br[5][i], br[6][i], br[7][i]}, b1[i], b2[i], b3[i]);
            ask_big();
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                bf8 c1, c2, c3;
                split8_bf16(f4{sr[0][j], sr[1][j], sr[2][j], sr[3][j]} * sign, f4{sr[4][j], sr[5][j], sr[6][j], sr[7][j]} * sign, c1, c2, c3);
                if (j == NS - 1) ask_small();
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    // (x is the A operand: its index runs over the registers of a result)
                    auto mac = [&](const bf8 &b, const bf8 &c) {
                        if constexpr (XBIG) mm[i][j].mac(b, c);
                        else mm[i][j].mac(c, b);
                    };
                    mac(b3[i], c1);
                    mac(b2[i], c2);
                    mac(b1[i], c3);
                    mac(b2[i], c1);
                    mac(b1[i], c2);
                    mac(b1[i], c1);
                }
            }
        }
        const MfmaSettled settled;

        // result register 4 q + c of a block: input index 8 q + 4 half + c, output index l32; input k0 + KB index + i, output o0 + OB index + j
        float *const P = a.ws + (size_t)part * (size_t)row_part_floats(K, O, a.s_loc) + (size_t)s * (size_t)(O * K);
#pragma unroll
        for (int j = 0; j < OB; ++j) {
            float *mine = turn[wave];
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                const int m = 8 * (g >> 2) + 4 * half + (g & 3);
                typename Floats<KB>::V v;
#pragma unroll
                for (int i = 0; i < KB; ++i) v[i] = XBIG ? mm[i][j % NS].read(settled)[g] : mm[j][i % NS].read(settled)[g];
                *reinterpret_cast<typename Floats<KB>::V *>(mine + l32 * PITCH + KB * m) = v;
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < KB; ++it) {
                const int idx = it * 64 * kRowPartWaves + (int)threadIdx.x, row = idx / (TK / 4), quad = idx % (TK / 4);
                f4 of_wave[kRowPartWaves], sum;
#pragma unroll
                for (int v = 0; v < kRowPartWaves; ++v) of_wave[v] = *reinterpret_cast<const f4 *>(turn[v] + row * PITCH + 4 * quad);
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] = (of_wave[0][c] - of_wave[1][c]) + (of_wave[2][c] - of_wave[3][c]);
                const long o = o0 + OB * row + j, k = k0 + 4 * quad;
                if (o < O && k < K) {
                    if (c_lo != r_lo) sum += load4<true, false>(P + o * K + k);
                    store4<true, false>(P + o * K + k, sum);
                }
            }
            __syncthreads();
        }
    }
    if (bias_tile) {            // uniform over the workgroup
#pragma unroll
        for (int j = 0; j < OB; ++j) {
            const float both = col_sum[j] + __shfl_xor(col_sum[j], 32);
            if (half == 0) turn[wave][OB * l32 + j] = both;
        }
        __syncthreads();
        if (threadIdx.x < TO && o0 + (long)threadIdx.x < O) {
            float sum = turn[0][threadIdx.x];
#pragma unroll
            for (int v = 1; v < kRowPartWaves; ++v) sum += turn[v][threadIdx.x];
            a.ws[(size_t)part * (size_t)row_part_floats(K, O, a.s_loc) + (size_t)a.s_loc * (size_t)(O * K) +
                 (size_t)s * (size_t)((O + 3) & ~3L) + (size_t)o0 + threadIdx.x] = sum;
        }
    }
}

// Quad q of a sample's sums where the parts add up to NaN: parts that hold a NaN (an infinite factor, and one whose pieces overflow, leaves
// one) are formed again there, from fp32 products.  A wave's lanes read consecutive quads of a row of x and the same factor of dy.
// A row of dy that is NaN, late in a part, makes 7260 x 2160 x 540 x 2 samples 0.22 -> 0.60 ms and 16640 x 192 x 768 x 2 0.086 -> 0.23; in
// the kernel above, a lane to each sum with rows across its lanes, it was 25.7 and 4.7.
__device__ __forceinline__ f4 row_parts_again(const LinearGradArgs &a, int s, long q, int parts, const float *theirs, size_t per_part)
{
    const long K = a.in_features, O = a.out_features, o = 4 * q / K, k = 4 * q - o * K;
    const float *x = a.x + (size_t)s * (size_t)a.x_sample_stride + (size_t)k, *dy = a.dy + (size_t)s * (size_t)a.rows * (size_t)O + (size_t)o;
    f4 P = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int p = 0; p < parts; ++p) {
        f4 u = load4<true, false>(theirs + (size_t)p * per_part);
        if (u[0] != u[0] || u[1] != u[1] || u[2] != u[2] || u[3] != u[3]) {
            const long lo = p * a.rows_per_part, hi = lo + a.rows_per_part < a.rows ? lo + a.rows_per_part : a.rows;
            f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
            bool open = true;                   // a sum that is to be formed again is not NaN so far
#pragma unroll 1
            for (long r = lo; r < hi && open; r += 4) {
                f4 xv[4];
                float dv[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const size_t from = (size_t)(r + t < hi ? r + t : hi - 1);
                    xv[t] = load4<true, false>(x + from * (size_t)a.ldx);
                    dv[t] = dy[from * (size_t)O];
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (r + t < hi) v[c] = __builtin_fmaf(dv[t], xv[t][c], v[c]);
                open = false;
#pragma unroll
                for (int c = 0; c < 4; ++c) open |= u[c] != u[c] && v[c] == v[c];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) u[c] = u[c] != u[c] ? v[c] : u[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) P[c] += u[c];
    }
    return P;
}

// Adds the parts in a fixed order, draws eps and finishes the gradients: thread q owns quad q of the O*K weights, the threads
// behind them one quad of biases each.  A thread sends for eight parts at a time and draws eps behind the first of them.  What bounds it: memory
// and the draw; with few parts, on large layers, how many waves hide the one behind the other.  So PARTS of them, up to kRowPartUnrolled,
// are a kernel of their own (0: more): no load is made twice, and mu and sigma, which up to then would be held through the draw, come last
// (64 registers, seven waves to a SIMD, against 83 and five).  The whole weight gradients, before eight parts were sent for at a
// time, with eight for all, and now: one part 380 x 416 x 4580 x 2 samples 33.3 / 35.5 / 32.8 us, 157 x 1660 x 876 x 4 31.6 / 35.6 / 30.6;
// two 850 x 4032 x 372 x 1 31.1 / 34.4 / 31.3; five 1184 x 168 x 4004 x 1 25.2 / 27.0 / 25.3; fourteen 16640 x 192 x 768 x 2 73.8 / 69.2 / 69.5;
// of 3700 layers with parts the second was more than 3 % behind the first on 530; this is on none of 4900.
constexpr int kRowPartUnrolled = 8;

template <int PARTS>
__global__ void __launch_bounds__(64)
hot_linear_wgrad_row_parts_finish_kernel(LinearGradArgs a, int n_parts)
{
    const int parts = PARTS ? PARTS : n_parts;
    const long K = a.in_features, O = a.out_features, quads = O * K / 4, O4 = (O + 3) & ~3L;
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool weights = q < quads;
    const long b = q - quads;                   // bias quad
    if (!weights && (a.mu_b == nullptr || 4 * b >= O)) return;
    const size_t per_part = (size_t)row_part_floats(K, O, a.s_loc), per_sample = (size_t)(weights ? O * K : O4);
    const float *first = a.ws + (weights ? (size_t)q * 4 : (size_t)a.s_loc * (size_t)(O * K) + (size_t)b * 4);
    f4 gm = {0.0f, 0.0f, 0.0f, 0.0f}, gs = gm;
    const size_t mine = weights ? (size_t)q * 4 : 0;
    f4 m4, sd4;
    if constexpr (PARTS == 0) {
        m4 = load4<true, false>(a.mu_w + mine);
        sd4 = load4<true, false>(a.sigma_w + mine);
    }
    for (int s = 0; s < a.s_loc; ++s) {
        const float *theirs = first + (size_t)s * per_sample;
        // (four running sums, so that neither the additions nor their roundings form one long chain)
        f4 of[4], P, e;
#pragma unroll
        for (int v = 0; v < 4; ++v) of[v] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        constexpr int B = PARTS ? PARTS : 8;
        for (int p0 = 0; p0 < parts; p0 += B) {
            f4 u[B];
#pragma unroll
            for (int v = 0; v < B; ++v) u[v] = load4<true, false>(theirs + (size_t)(p0 + v < parts ? p0 + v : parts - 1) * per_part);
            if (p0 == 0) e = eps_quad(weights ? a.weight_quad0 + q : a.bias_quad0 + b, s, a.rng);
#pragma unroll
            for (int v = 0; v < B; ++v)
#pragma unroll
                for (int c = 0; c < 4; ++c) of[v & 3][c] += p0 + v < parts ? u[v][c] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) P[c] = (of[0][c] + of[1][c]) + (of[2][c] + of[3][c]);
        if (weights && (P[0] != P[0] || P[1] != P[1] || P[2] != P[2] || P[3] != P[3])) P = row_parts_again(a, s, q, parts, theirs, per_part);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            gm[c] += P[c];
            gs[c] = __builtin_fmaf(P[c], e[c], gs[c]);
        }
    }
    if (weights) {
        if constexpr (PARTS != 0) {
            m4 = load4<true, false>(a.mu_w + mine);
            sd4 = load4<true, false>(a.sigma_w + mine);
        }
        f4 om, os;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float u, v;
            finish_pair(gm[c], gs[c], m4[c], sd4[c], (float)a.g, (float)a.k, u, v);
            om[c] = u;
            os[c] = v;
        }
        store4<true, false>(a.gmu_w + 4 * q, om);
        store4<true, false>(a.gsig_w + 4 * q, os);
        return;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const long o = 4 * b + c;
        if (o < O) {
            float u, v;
            finish_pair(gm[c], gs[c], a.mu_b[o], a.sigma_b[o], (float)a.g, (float)a.k, u, v);
            a.gmu_b[o] = u;
            a.gsig_b[o] = v;
        }
    }
}

// How the two kernels above run a layer; parts == 0: they do not.
struct RowPartsPlan {
    int parts;
    long rows_per_part;
    long chunks;        // in which a part is added up
    bool xbig;
};

template <bool XBIG>
inline long row_part_tiles(const hot_linear_desc *d)
{
    constexpr int tk = 32 * (XBIG ? kRowPartBig : kRowPartSmall), to = 32 * (XBIG ? kRowPartSmall : kRowPartBig);
    return ((d->in_features + tk - 1) / tk) * ((d->out_features + to - 1) / to);
}

// Where they run, measured against the first kernel above with a workspace, 40 shapes: 16640 x 192 x 768 150 -> 74 us,
// 7260 x 2160 x 540 382 -> 205, 1024 x 540 x 2160 96 -> 52, 300 x 540 x 2160 41 -> 28, 513 x 2160 x 2160 x 8 samples 478 -> 293;
// below 300 rows they win once rows x samples reach 600 (256 x 192 x 768 x 4: 20 -> 17 us) and lose below that (256 x 1024^2 x 2:
// 24 -> 28, 129 x 8192 x 1024 x 1: 43 -> 52), and at a hundred rows and less (64 x 128^2 x 4: 15 -> 18).  Layers of 512 tiles of
// 128 x 128 and more stay with the kernel above this one: level with it (0.96-1.08x), it needs no workspace.
constexpr long kRowPartMinRows = 129, kRowPartAlwaysRows = 300, kRowPartMinRowSamples = 600;
constexpr long kRowPartMinWeights = 8192, kRowPartAnyWeightsRows = 512;     // (one or two tiles need that many rows to be worth two launches)
// From 8192 to 2^18 weights the products are too few to pay for a second launch with one or two samples and fewer than 1200 rows
// of them (581 x 540 x 380 x 1: 13.3 against 15.2 us, 317 x 124 x 1448 x 2 14.0 against 15.2; of 90 such layers 1.03x on
// average), nor do they where half of every tile has no outputs (544 x 7756 x 32 x 2: 18.2 against 20.4).  From 8192 rows on the
// other kernel cuts the rows of up to 2^17 weights into four parts, from 16384 on its waves outnumber the chip's slots: between
// them it is as fast on one sample (8300 x 192 x 128 x 1: 23.3 against 25.9, 12000 x 100 x 300 level, 16640 x 192^2 42.9 against 31.0).
constexpr long kRowPartFewRowSamples = 1200, kRowPartManyWeights = 1L << 18;
constexpr long kRowPartNarrow = 32, kRowPartNarrowRows = 1000;
constexpr long kRowPartOneSampleRows = 8192, kRowPartOneSampleRowsEnd = 12000, kRowPartOneSampleWeights = 1L << 17;
constexpr long kRowPartMaxTileCount = 512;
// Rows of dy may start at any multiple of 4 bytes: a load of 8 or 16 bytes needs no more, a quad that reaches over the end of a row only
// brings columns that are never stored, and behind the window's end the hardware's check is per 4 bytes.  (104 layers with outputs even
// but no multiple of four, 129 to 16640 rows: 1.02-3.0x against the first kernel, 8809 x 1108 x 30 x 2 samples 0.95x and 884 x 100 x 26 x 1
// 0.97x, at 0.3-0.97 of its distance from 64 bits.)  Odd numbers of outputs still go to that kernel.  Nothing in this one stands against
// them, and on 45 such layers it was 1.06-2.8x as fast at 0.4-0.98 of the distance; their route has not been changed yet.
constexpr int kRowPartMaxParts = 64;
constexpr int64_t kRowPartMaxBytes = (int64_t)256 << 20, kRowPartSmallBytes = (int64_t)8 << 20;
// Errors grow with the rows that a wave adds up, 2-norm against 64 bits at 16640 x 192 x 768: 2.7e-7 with 297, 2.0e-7 with 152 (the fp32
// instruction with 260: 3.1e-7).  From 8192 rows on, where the first kernel also cuts many parts, a wave's sums leave its
// registers after at most 208 rows.
constexpr long kRowPartLongRows = 8192, kRowPartLongMost = 208, kRowPartFineRows = 64;

inline bool row_parts_suit(const hot_linear_desc *d)
{
    if (d->rows < kRowPartMinRows || (d->rows < kRowPartAlwaysRows && d->rows * d->s_local < kRowPartMinRowSamples)) return false;
    if (d->rows < kRowPartAnyWeightsRows && d->in_features * d->out_features < kRowPartMinWeights) return false;
    if ((d->out_features & 1) || wgrad_tile_count(d) >= kRowPartMaxTileCount) return false;
    if (const long weights = d->in_features * d->out_features; weights > kRowPartMinWeights) {
        if (weights < kRowPartManyWeights && d->s_local <= 2 && d->rows * d->s_local < kRowPartFewRowSamples) return false;
        if (d->out_features <= kRowPartNarrow && d->rows < kRowPartNarrowRows && d->s_local <= 4) return false;
        if (weights < kRowPartOneSampleWeights && d->s_local == 1 && d->rows >= kRowPartOneSampleRows && d->rows < kRowPartOneSampleRowsEnd) return false;
    }
    const unsigned long long lim = 0xFFFFFFF0ull;           // 32-bit byte offsets
    const unsigned long long reach = (unsigned long long)d->rows + 2 * kRowPartRows * kRowPartWaves;
    return (reach * d->ldx + d->in_features) * 4 < lim && reach * d->out_features * 4 < lim;
}

inline int64_t wgrad_part_bytes(const hot_linear_desc *d)
{
    return 2 * (d->out_features * d->in_features + ((d->out_features + 3) & ~(int64_t)3)) * (int64_t)sizeof(float);
}

// What the parts may take: as much as the first kernel's sixteen, for small layers up to 8 MiB.
inline int64_t row_parts_budget(const hot_linear_desc *d)
{
    const int64_t sixteen = kWgradMaxParts * wgrad_part_bytes(d), most = sixteen > kRowPartSmallBytes ? sixteen : kRowPartSmallBytes;
    return most < kRowPartMaxBytes ? most : kRowPartMaxBytes;
}

// (a wave to a workgroup, so that few reach every compute unit)
template <int PARTS>
void row_parts_finish_go(int parts, long threads, hipStream_t s, const LinearGradArgs &a)
{
    const dim3 grid((unsigned)((threads + 63) / 64)), block(64);
    if (parts > kRowPartUnrolled) return hot_linear_wgrad_row_parts_finish_kernel<0><<<grid, block, 0, s>>>(a, parts);
    if (parts == PARTS) return hot_linear_wgrad_row_parts_finish_kernel<PARTS><<<grid, block, 0, s>>>(a, parts);
    if constexpr (PARTS > 1) row_parts_finish_go<PARTS - 1>(parts, threads, s, a);
}

void row_parts_go(const RowPartsPlan &p, hipStream_t s, const LinearGradArgs &a, long tiles)
{
    const long per_xcd = (tiles * a.s_loc * p.parts + kXcds - 1) / kXcds;
    const dim3 grid((unsigned)(kXcds * per_xcd)), block(64 * kRowPartWaves);
    const long step_rows = kRowPartRows * kRowPartWaves, chunk = ((p.rows_per_part + p.chunks - 1) / p.chunks + step_rows - 1) / step_rows * step_rows;
    if (p.xbig) hot_linear_wgrad_row_parts_kernel<true><<<grid, block, 0, s>>>(a, p.parts, (int)chunk);
    else hot_linear_wgrad_row_parts_kernel<false><<<grid, block, 0, s>>>(a, p.parts, (int)chunk);
    const long threads = a.out_features * a.in_features / 4 + (a.mu_b ? (a.out_features + 3) / 4 : 0);
    row_parts_finish_go<kRowPartUnrolled>(p.parts, threads, s, a);
}

// A wave's finished 64-input x 16*RB-row tile of one sample's dx goes to memory.  Register rr of accumulator
// i is input k0 + 16 j + 4 rr + i of row r0 + 16 rb + n; the lanes of a row exchange quads so that each store
// covers 64 contiguous bytes of the row.  Every lane of the wave must call it.
template <int RB>
__device__ __forceinline__ void store_dx_tile(const f4 (&acc)[RB][4], float *dx, int s, long r0, long k0, int j, int n,
                                              const LinearGradArgs &a)
{
    const long K = a.in_features, R = a.rows;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const long row = r0 + kRowsPerTile * rb + n;
        f4 q[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) q[rr] = f4{acc[rb][0][rr], acc[rb][1][rr], acc[rb][2][rr], acc[rb][3][rr]};
        transpose_quads_over_j(q, j, n);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const long col = k0 + 16 * t + 4 * j;
            if (row < R && col < K)
                store4<true, false>(dx + ((size_t)s * (size_t)R + (size_t)row) * (size_t)K + (size_t)col, q[t]);
        }
    }
}

// A workgroup owns 64 inputs x 16*RB rows of one sample's dx; its waves take the outputs in blocks
// of sixteen, round-robin, and their partial tiles are added through LDS in wave order.
constexpr int kXgradOutputsPerStep = 16;
template <int RB>
__global__ void __launch_bounds__(64 * max_waves(RB), RB >= 4 ? 2 : 1)
hot_linear_xgrad_kernel(LinearGradArgs a)
{
    extern __shared__ float partial[];   // [waves - 1][RB * 16][64]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long k0 = (long)blockIdx.x * 64, r0 = (long)blockIdx.y * (kRowsPerTile * RB);
    const int s = blockIdx.z;
    const float *dys = a.dy + (size_t)s * (size_t)R * (size_t)O;
    const long kq = k0 + 4 * n;          // this lane's quad of inputs (as an A lane)
    const bool k_ok = kq < K;

    Acc16x16 mm[RB][4];

    // dy is read as quads of four consecutive outputs (lane (n, j): outputs ob + 4 j .. + 3 of row n; dword
    // alignment suffices), and matrix instruction (c, i) takes element c of them against element i of the
    // weight quad of output ob + 4 j + c: one 16-byte load per row block where single values took four loads.
    // Rows beyond R read row R - 1: they only reach accumulator columns that are never stored.
    long at[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const long row = r0 + kRowsPerTile * rb + n;
        at[rb] = (row < R ? row : R - 1) * O + 4 * j;
    }
    for (long ob = (long)wave * kXgradOutputsPerStep; ob < O; ob += (long)waves * kXgradOutputsPerStep) {
        f4 m4[4], sd4[4], dyq[RB];
        bool ok[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long o = ob + 4 * j + c;
            ok[c] = k_ok && o < O;
            m4[c] = ok[c] ? load4<true, false>(a.mu_w + o * K + kq) : f4{0.0f, 0.0f, 0.0f, 0.0f};
            sd4[c] = ok[c] ? load4<true, false>(a.sigma_w + o * K + kq) : f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if (ob + kXgradOutputsPerStep <= O) {        // uniform over the wave
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) dyq[rb] = load4<false, false>(dys + at[rb] + ob);
        } else {                                     // last, partial step: outputs beyond O contribute zeros
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < 4; ++c) dyq[rb][c] = ob + 4 * j + c < O ? dys[at[rb] + ob + c] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f4 w4 = {0.0f, 0.0f, 0.0f, 0.0f};
            if (ok[c]) {
                const long o = ob + 4 * j + c;
                const f4 e = eps_quad(a.weight_quad0 + ((o * K + kq) >> 2), s, a.rng);
#pragma unroll
                for (int i = 0; i < 4; ++i) w4[i] = __builtin_fmaf(sd4[c][i], e[i], m4[c][i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    mm[rb][i].mac(w4[i], dyq[rb][c]);
        }
    }
    const MfmaSettled settled;
    f4 acc[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[rb][i] = mm[rb][i].read(settled);

    if (waves > 1) {
        if (wave > 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
                        partial[((wave - 1) * (RB * 16) + (rb * 4 + i) * 4 + rr) * 64 + lane] = acc[rb][i][rr];
        }
        __syncthreads();
        if (wave == 0) {
            for (int v = 1; v < waves; ++v)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr)
                            acc[rb][i][rr] += partial[((v - 1) * (RB * 16) + (rb * 4 + i) * 4 + rr) * 64 + lane];
        }
    }
    if (wave != 0) return;

    store_dx_tile<RB>(acc, a.dx, s, r0, k0, j, n, a);
}

// ---------------------------------------------------------------------------------
// Input gradients for many rows: as in the forward kernel for many rows, the four waves of a workgroup
// take up to 64 rows each and share every draw through LDS.  A workgroup owns 64 inputs x 256 rows of one
// sample's dx and walks over the outputs 16 at a time: each of its 256 threads draws one quad of the
// 16-output x 64-input weight tile (wave c, lane (m, j): output ob + 4 j + c, inputs k0 + 4 m .. + 3) into
// LDS, and after one barrier every wave reads the four quads of its lane position and multiplies its own
// 64 rows: 64 matrix instructions per drawn quad instead of 16.  A lane reads dy as quads of four
// consecutive outputs (one 16-byte load per row block and iteration; dy needs dword alignment only) and
// matrix instruction (c, i) takes element c of the dy quads against element i of weight quad c: the
// contraction index is only enumerated in another order.  Tile double-buffered, one barrier per iteration,
// as in the forward kernel; accumulators and epilogue are those of the kernel above.
// ---------------------------------------------------------------------------------
constexpr int kXgradRowsKernelOutputs = 16;    // outputs per iteration: one drawn quad per thread
constexpr int kXgradMaxParts = 16;             // most parts the outputs are cut into with a workspace

// RB: 16-row blocks per wave (a workgroup owns 64 RB rows); fewer of them where 256-row workgroups would be too few.
template <int RB>
__global__ void __launch_bounds__(256)
hot_linear_xgrad_rows_kernel(LinearGradArgs a)
{
    __shared__ __attribute__((aligned(16))) float tile[2][4 * 64 * 4];     // [buffer][c][j][m] quads
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    // with a workspace the outputs may be cut into parts for different workgroups (grid x = input groups x parts):
    // this one contracts over the outputs o_lo .. o_hi - 1 only and leaves its block in the workspace
    const long k_groups = (K + 63) / 64;
    const long part = (long)blockIdx.x / k_groups, k0 = ((long)blockIdx.x % k_groups) * 64;
    const long o_lo = a.x_parts > 1 ? part * a.outs_per_part : 0;
    const long o_hi = a.x_parts > 1 && o_lo + a.outs_per_part < O ? o_lo + a.outs_per_part : O;
    const long r0 = ((long)blockIdx.y * 4 + wave) * (kRowsPerTile * RB);
    const int s = blockIdx.z;
    const float *dys = a.dy + (size_t)s * (size_t)R * (size_t)O;
    const long kq = k0 + 4 * n;          // this lane's quad of inputs (as a drawing thread and as an A lane)
    const bool k_ok = kq < K;

    Acc16x16 mm[RB][4];
    // rows beyond R read row R - 1 instead: they only reach columns of the accumulators that are never stored
    long at[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const long row = r0 + kRowsPerTile * rb + n;
        at[rb] = (row < R ? row : R - 1) * O + 4 * j;
    }

    int buf = 0;
    for (long ob = o_lo; ob < o_hi; ob += kXgradRowsKernelOutputs, buf ^= 1) {
        const long o_draw = ob + 4 * j + wave;
        const bool draw_ok = k_ok && o_draw < o_hi;
        f4 w4 = {0.0f, 0.0f, 0.0f, 0.0f};
        f4 dyq[RB];
        if (ob + kXgradRowsKernelOutputs <= o_hi) {      // uniform
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) dyq[rb] = load4<false, false>(dys + at[rb] + ob);
        } else {                                         // last, partial step: outputs beyond O contribute zeros
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < 4; ++c) dyq[rb][c] = ob + 4 * j + c < o_hi ? dys[at[rb] + ob + c] : 0.0f;
        }
        if (draw_ok) {
            const f4 m4 = load4<true, false>(a.mu_w + o_draw * K + kq), sd4 = load4<true, false>(a.sigma_w + o_draw * K + kq);
            const f4 e = eps_quad(a.weight_quad0 + ((o_draw * K + kq) >> 2), s, a.rng);
#pragma unroll
            for (int c = 0; c < 4; ++c) w4[c] = __builtin_fmaf(sd4[c], e[c], m4[c]);
        }
        *reinterpret_cast<f4 *>(&tile[buf][((wave * 4 + j) * 16 + n) * 4]) = w4;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const f4 wq = *reinterpret_cast<const f4 *>(&tile[buf][((c * 4 + j) * 16 + n) * 4]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    mm[rb][i].mac(wq[i], dyq[rb][c]);
        }
    }
    const MfmaSettled settled;
    f4 acc[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[rb][i] = mm[rb][i].read(settled);

    float *dst = a.x_parts > 1 ? a.ws + (size_t)part * (size_t)a.s_loc * (size_t)R * (size_t)K : a.dx;
    store_dx_tile<RB>(acc, dst, s, r0, k0, j, n, a);
}

// dx = the sum of the parts' blocks in the workspace, in part order; one quad per thread.
__global__ void __launch_bounds__(256)
hot_linear_dx_sum_kernel(float *__restrict__ dx, const float *__restrict__ ws, long quads, int parts)
{
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q >= quads) return;
    f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int p = 0; p < parts; ++p) {
        const f4 v = load4<true, false>(ws + (size_t)p * (size_t)quads * 4 + (size_t)q * 4);
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[c] += v[c];
    }
    store4<true, false>(dx + (size_t)q * 4, sum);
}

// ---------------------------------------------------------------------------------
// Few rows (at most 32) with the input gradients wanted: both gradients in ONE pass over the weights.  The kernels
// above each draw every eps of the layer, and at few rows the draw is most of their time (four generator quads
// per lane and 16 x 64 tile: about 2600 vector cycles, against 512 matrix cycles per 16 rows and product); here a
// wave draws the quads of its tile once per sample and uses them for both products.  No drawn value has to move
// between lanes for that: with dy as the A operand and element i of a lane's quad of x as the B operand, result
// register rr of accumulator i is G[ob + 4 j + rr][k0 + 4 n + i], so lane (n, j) receives the weight gradients of
// exactly the four quads (outputs ob + 4 j + c, inputs k0 + 4 n .. + 3) that the input-gradient kernel has it draw.
//
// A workgroup of four waves owns 64 inputs (its strip of x waits in LDS) and one part of the outputs; its waves
// take that part's 16-output tiles round-robin, and the accumulators of every sample's dx stay in registers over
// the whole loop (16 RB per sample and lane: that bounds rows x samples).  Per tile and sample: dy of the tile
// (once per operand layout), the draw, G = dy^T x, sum_s G and sum_s G eps in registers, w = mu + sigma eps in
// the registers of eps, dx += dy w; the loads of a sample (and of the tile's mu, sigma) are issued before its draw.  After the last
// sample the tile's gradients are finished and stored, 256 contiguous bytes per output row.  At the end the
// waves' dx tiles are added through LDS in wave order and go to the workspace as this part's block (straight to
// dx if the layer has one part); hot_linear_dx_sum_kernel adds the blocks in part order.  No atomics.
// ---------------------------------------------------------------------------------
constexpr int kOnePassWaves = 4;
constexpr int kOnePassMaxRows = 32;
constexpr int kOnePassAccumulators = 8;     // most (16-row blocks) x (samples) whose dx accumulators a lane holds

template <int RB, int SMAX>
__global__ void __launch_bounds__(64 * kOnePassWaves, RB * SMAX <= 4 ? 2 : 1)
hot_linear_backward_one_pass_kernel(LinearGradArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float strip[];   // [copies of x][16 RB rows][64 inputs]; at the end [waves - 1][16 RB][64]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long k0 = (long)blockIdx.x * 64;
    const long part = blockIdx.y;
    const long o_lo = part * a.outs_per_part;
    const long o_hi = o_lo + a.outs_per_part < O ? o_lo + a.outs_per_part : O;
    const long kq = k0 + 4 * n;             // this lane's quad of inputs
    const bool k_ok = kq < K;
    const bool bias_strip = a.mu_b != nullptr && blockIdx.x == 0;    // this strip's workgroups also own the biases of their outputs
    constexpr int kStripQuads = 16 * RB * 16;
    const float gf = (float)a.g, kf = (float)a.k;

    // rows beyond R and inputs beyond K enter as zeros: they are summed over
    const int copies = a.x_sample_stride != 0 ? a.s_loc : 1;
    for (int at = threadIdx.x; at < copies * kStripQuads; at += 64 * kOnePassWaves) {
        const int copy = at / kStripQuads, rest = at % kStripQuads, row = rest >> 4, q = rest & 15;
        f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < R && k0 + 4 * q < K)
            v = load4<true, false>(a.x + (size_t)copy * (size_t)a.x_sample_stride + (size_t)row * (size_t)a.ldx + (size_t)(k0 + 4 * q));
        *reinterpret_cast<f4 *>(strip + (size_t)at * 4) = v;
    }
    __syncthreads();

    // dx: register rr of mx[s][rb][i] is input k0 + 16 j + 4 rr + i of row 16 rb + n of sample s
    Acc16x16 mx[SMAX][RB][4];

    // Lanes outside the layer (outputs >= O, inputs >= K) read a valid address instead; what they read is never used.
    auto fetch_parameters = [&](long ob, f4 (&m)[4], f4 (&sd)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long o = ob + 4 * j + c;
            const long at = (o < O ? o : O - 1) * K + (k_ok ? kq : 0);
            m[c] = load4<true, false>(a.mu_w + at);
            sd[c] = load4<true, false>(a.sigma_w + at);
        }
    };

    // dy of a tile and sample, once per operand layout: as the A operand of G (lane (n, j): output ob + n, rows 4 q + j; rows
    // beyond R are zeros) and as the B operand of dx (row 16 rb + n, outputs ob + 4 j .. + 3; rows beyond R read row R - 1,
    // which only reaches columns of the accumulators that are never stored; outputs beyond O must be zeros)
    auto fetch_dy = [&](long ob, int s, float (&dya)[4 * RB], f4 (&dyq)[RB]) {
        const float *dys = a.dy + (size_t)s * (size_t)R * (size_t)O;
        const long o_a = ob + n < O ? ob + n : O - 1;
#pragma unroll
        for (int q = 0; q < 4 * RB; ++q) {      // (rows beyond R: row R - 1 for now; zeroed where the values are used, behind the draw)
            const long row = 4 * q + j;
            dya[q] = dys[(row < R ? row : R - 1) * O + o_a];
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const long row = 16 * rb + n;
            const float *at = dys + (row < R ? row : R - 1) * O + ob + 4 * j;
            if (ob + 16 <= O) dyq[rb] = load4<false, false>(at);       // uniform over the wave
            else {
#pragma unroll
                for (int c = 0; c < 4; ++c) dyq[rb][c] = ob + 4 * j + c < O ? at[c] : 0.0f;
            }
        }
    };

    // The loads of a tile's first sample and of its mu, sigma are issued at the end of the tile before, ahead of that
    // tile's stores: loads and stores complete in order, and a wait for a load issued behind the stores would also wait
    // until the gradients have reached memory.  A wave without tiles fetches a valid tile and uses nothing.
    const long ob_first = o_lo + 16 * wave;
    f4 m4[4], sd4[4];
    float dya0[4 * RB];
    f4 dyq0[RB];
    fetch_parameters(ob_first < o_hi ? ob_first : o_lo, m4, sd4);
    fetch_dy(ob_first < o_hi ? ob_first : o_lo, 0, dya0, dyq0);
    for (long ob = ob_first; ob < o_hi; ob += 16 * kOnePassWaves) {
        bool ok[4];
        long quad[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long o = ob + 4 * j + c;
            ok[c] = k_ok && o < O;
            quad[c] = a.weight_quad0 + (((o < O ? o : O - 1) * K + (k_ok ? kq : 0)) >> 2);
        }
        f4 gm[4], gs[4], gbm = {0.0f, 0.0f, 0.0f, 0.0f}, gbs = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < 4; ++c) gm[c] = gs[c] = f4{0.0f, 0.0f, 0.0f, 0.0f};

#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
            if (s < a.s_loc) {                  // uniform over the grid
                float dya[4 * RB];
                f4 dyq[RB];
                if (s == 0) {
#pragma unroll
                    for (int q = 0; q < 4 * RB; ++q) dya[q] = dya0[q];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) dyq[rb] = dyq0[rb];
                } else {
                    fetch_dy(ob, s, dya, dyq);
                }
                // every load of this sample, the rows of x from LDS among them, is on its way before its draw, whose
                // arithmetic covers their latency
                const float *xs = strip + (a.x_sample_stride != 0 ? s : 0) * (kStripQuads * 4);
                constexpr bool kEarlyX = RB * SMAX <= 2;        // (registers for it only in the lightest shape)
                f4 xq[4 * RB];
                if constexpr (kEarlyX) {
#pragma unroll
                    for (int q = 0; q < 4 * RB; ++q) xq[q] = *reinterpret_cast<const f4 *>(xs + (4 * q + j) * 64 + 4 * n);
                }
                __builtin_amdgcn_sched_barrier(0);
                f4 e[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) e[c] = eps_quad(quad[c], s, a.rng);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 4 * RB; ++q)
                    if (4 * q + j >= R) dya[q] = 0.0f;

                Acc16x16 mg[4], mb;
#pragma unroll
                for (int q = 0; q < 4 * RB; ++q) {
                    if constexpr (!kEarlyX) xq[q] = *reinterpret_cast<const f4 *>(xs + (4 * q + j) * 64 + 4 * n);
#pragma unroll
                    for (int i = 0; i < 4; ++i) mg[i].mac(dya[q], xq[q][i]);
                }
                if (bias_strip) {               // column sums of dy: the same contraction against ones
#pragma unroll
                    for (int q = 0; q < 4 * RB; ++q) mb.mac(dya[q], 1.0f);
                }
                f4 P[4], Pb;
                {
                    const MfmaSettled settled;
#pragma unroll
                    for (int i = 0; i < 4; ++i) P[i] = mg[i].read(settled);
                    Pb = mb.read(settled);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        gm[c][i] += P[i][c];
                        gs[c][i] = __builtin_fmaf(P[i][c], e[c][i], gs[c][i]);
                    }
                if (bias_strip) {               // register rr of Pb: sum_r dy_s[r][ob + 4 j + rr], the four outputs of one generator quad
                    const f4 eb = eps_quad(a.bias_quad0 + ((ob + 4 * j) >> 2), s, a.rng);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        gbm[rr] += Pb[rr];
                        gbs[rr] = __builtin_fmaf(Pb[rr], eb[rr], gbs[rr]);
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) e[c][i] = ok[c] ? __builtin_fmaf(sd4[c][i], e[c][i], m4[c][i]) : 0.0f;
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) mx[s][rb][i].mac(e[c][i], dyq[rb][c]);
            }
        }

        // the tile's gradients; then the next tile's loads into the registers they leave; then the stores
        f4 om[4], os[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float u, v;
                finish_pair(gm[c][i], gs[c][i], m4[c][i], sd4[c][i], gf, kf, u, v);
                om[c][i] = u;
                os[c][i] = v;
            }
        f4 ob_m = {0.0f, 0.0f, 0.0f, 0.0f}, ob_s = {0.0f, 0.0f, 0.0f, 0.0f};
        if (bias_strip) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const long o = ob + 4 * j + rr < O ? ob + 4 * j + rr : O - 1;
                float u, v;
                finish_pair(gbm[rr], gbs[rr], a.mu_b[o], a.sigma_b[o], gf, kf, u, v);
                ob_m[rr] = u;
                ob_s[rr] = v;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        {
            const long ob_next = ob + 16 * kOnePassWaves < o_hi ? ob + 16 * kOnePassWaves : ob;
            fetch_parameters(ob_next, m4, sd4);
            fetch_dy(ob_next, 0, dya0, dyq0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (ok[c]) {
                const long at = (ob + 4 * j + c) * K + kq;
                store4<true, false>(a.gmu_w + at, om[c]);
                store4<true, false>(a.gsig_w + at, os[c]);
            }
        }
        if (bias_strip && n == 0) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const long o = ob + 4 * j + rr;
                if (o < O) {
                    a.gmu_b[o] = ob_m[rr];
                    a.gsig_b[o] = ob_s[rr];
                }
            }
        }
    }

    __syncthreads();        // every wave is done with the strip of x: its LDS now carries the waves' partial tiles
    float *dst = a.x_parts > 1 ? a.ws + (size_t)part * (size_t)a.s_loc * (size_t)R * (size_t)K : a.dx;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        if (s < a.s_loc) {
            f4 acc[RB][4];
            {
                const MfmaSettled settled;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[rb][i] = mx[s][rb][i].read(settled);
            }
            if (wave > 0) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr)
                            strip[((wave - 1) * (RB * 16) + (rb * 4 + i) * 4 + rr) * 64 + lane] = acc[rb][i][rr];
            }
            __syncthreads();
            if (wave == 0) {
                for (int v = 1; v < kOnePassWaves; ++v)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr)
                                acc[rb][i][rr] += strip[((v - 1) * (RB * 16) + (rb * 4 + i) * 4 + rr) * 64 + lane];
                store_dx_tile<RB>(acc, dst, s, 0, k0, j, n, a);
            }
            __syncthreads();    // the next sample's tiles overwrite these
        }
    }
}

// ---------------------------------------------------------------------------------
// The same one pass for more rows (33 to 128): the four waves of a workgroup split the ROWS (16 RBW each) and share
// every draw.  Per 16-output x 64-input tile and sample, wave c draws quad c of every lane position (output
// ob + 4 j + c, inputs k0 + 4 n .. + 3), forms w = mu + sigma eps and leaves it in LDS; behind a barrier every wave reads
// the four quads of its lane position, which are exactly its A operands of dx += dy w for its own rows, and multiplies
// G = dy^T x over its own rows; the partial G of the waves meet in LDS, and behind a second barrier wave c adds
// those of quad c in wave order and applies the eps that it drew itself.  A wave so holds the dx accumulators of its
// own rows only (16 RBW per sample) and one quad's gradient sums: few registers, several workgroups per compute
// unit, which take turns at the barriers.  No reduction of dx at the end: every wave stores its own rows.
// ---------------------------------------------------------------------------------
constexpr int kSplitRowsWaves = 4;

template <int RBW, int SMAX>
__global__ void __launch_bounds__(64 * kSplitRowsWaves, 2)
hot_linear_backward_split_rows_kernel(LinearGradArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    // [4][64] quads of drawn weights; [4 waves][5][64] quads of partial G (the fifth: column sums of dy); then the strip of x
    float *const wt = lds, *const gp = lds + 4 * 64 * 4, *const strip = gp + kSplitRowsWaves * 5 * 64 * 4;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, j = lane >> 4;
    const long K = a.in_features, O = a.out_features, R = a.rows;
    const long k0 = (long)blockIdx.x * 64;
    const long part = blockIdx.y;
    const long o_lo = part * a.outs_per_part;
    const long o_hi = o_lo + a.outs_per_part < O ? o_lo + a.outs_per_part : O;
    const long kq = k0 + 4 * n;
    const bool k_ok = kq < K;
    const bool bias_strip = a.mu_b != nullptr && blockIdx.x == 0;
    const float gf = (float)a.g, kf = (float)a.k;
    constexpr int kRows = 16 * RBW * kSplitRowsWaves;       // rows of the workgroup
    constexpr int kStripQuads = kRows * 16;
    const int r0 = 16 * RBW * wave;                         // this wave's rows

    const int copies = a.x_sample_stride != 0 ? a.s_loc : 1;
    for (int at = threadIdx.x; at < copies * kStripQuads; at += 64 * kSplitRowsWaves) {
        const int copy = at / kStripQuads, rest = at % kStripQuads, row = rest >> 4, q = rest & 15;
        f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < R && k0 + 4 * q < K)
            v = load4<true, false>(a.x + (size_t)copy * (size_t)a.x_sample_stride + (size_t)row * (size_t)a.ldx + (size_t)(k0 + 4 * q));
        *reinterpret_cast<f4 *>(strip + (size_t)at * 4) = v;
    }
    __syncthreads();

    // dx of this wave's rows: register rr of mx[s][rb][i] is input k0 + 16 j + 4 rr + i of row r0 + 16 rb + n
    Acc16x16 mx[SMAX][RBW][4];

    for (long ob = o_lo; ob < o_hi; ob += 16) {         // every wave walks every tile of the part
        // this wave's quad of the tile
        const long o_own = ob + 4 * j + wave;
        const bool ok = k_ok && o_own < O;
        const long at_own = (o_own < O ? o_own : O - 1) * K + (k_ok ? kq : 0);
        const f4 m4 = load4<true, false>(a.mu_w + at_own), sd4 = load4<true, false>(a.sigma_w + at_own);
        const long quad = a.weight_quad0 + (at_own >> 2);
        f4 gm = {0.0f, 0.0f, 0.0f, 0.0f}, gs = {0.0f, 0.0f, 0.0f, 0.0f};
        float gbm = 0.0f, gbs = 0.0f;

#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
            if (s < a.s_loc) {                  // uniform over the grid
                const float *dys = a.dy + (size_t)s * (size_t)R * (size_t)O;
                // dy of the tile and this wave's rows, once per operand layout (as in the kernel above), and the rows of x
                float dya[4 * RBW];
                f4 dyq[RBW], xq[4 * RBW];
                const long o_a = ob + n < O ? ob + n : O - 1;
#pragma unroll
                for (int q = 0; q < 4 * RBW; ++q) {
                    const long row = r0 + 4 * q + j;
                    dya[q] = dys[(row < R ? row : R - 1) * O + o_a];
                }
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb) {
                    const long row = r0 + 16 * rb + n;
                    const float *at = dys + (row < R ? row : R - 1) * O + ob + 4 * j;
                    if (ob + 16 <= O) dyq[rb] = load4<false, false>(at);       // uniform over the wave
                    else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) dyq[rb][c] = ob + 4 * j + c < O ? at[c] : 0.0f;
                    }
                }
                const float *xs = strip + (a.x_sample_stride != 0 ? s : 0) * (kStripQuads * 4);
#pragma unroll
                for (int q = 0; q < 4 * RBW; ++q) xq[q] = *reinterpret_cast<const f4 *>(xs + (r0 + 4 * q + j) * 64 + 4 * n);
                __builtin_amdgcn_sched_barrier(0);      // all of it on its way before the draw

                const f4 e = eps_quad(quad, s, a.rng);
                f4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = ok ? __builtin_fmaf(sd4[i], e[i], m4[i]) : 0.0f;
                *reinterpret_cast<f4 *>(wt + (wave * 64 + lane) * 4) = w;
                __syncthreads();        // the tile's four quads per lane position are there (and the sums below have been read)

                f4 wq[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) wq[c] = *reinterpret_cast<const f4 *>(wt + (c * 64 + lane) * 4);
#pragma unroll
                for (int q = 0; q < 4 * RBW; ++q)
                    if (r0 + 4 * q + j >= R) dya[q] = 0.0f;      // rows beyond R are summed over: zeros
                Acc16x16 mg[4], mb;
#pragma unroll
                for (int q = 0; q < 4 * RBW; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mg[i].mac(dya[q], xq[q][i]);
                if (bias_strip) {
#pragma unroll
                    for (int q = 0; q < 4 * RBW; ++q) mb.mac(dya[q], 1.0f);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int rb = 0; rb < RBW; ++rb) mx[s][rb][i].mac(wq[c][i], dyq[rb][c]);
                {
                    const MfmaSettled settled;
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const f4 p = {mg[0].read(settled)[rr], mg[1].read(settled)[rr], mg[2].read(settled)[rr], mg[3].read(settled)[rr]};
                        *reinterpret_cast<f4 *>(gp + ((wave * 5 + rr) * 64 + lane) * 4) = p;
                    }
                    if (bias_strip) *reinterpret_cast<f4 *>(gp + ((wave * 5 + 4) * 64 + lane) * 4) = mb.read(settled);
                }
                __syncthreads();        // the waves' partial sums are there (and every wave has read the drawn quads)

                f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int v = 0; v < kSplitRowsWaves; ++v) {
                    const f4 p = *reinterpret_cast<const f4 *>(gp + ((v * 5 + wave) * 64 + lane) * 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] += p[i];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gm[i] += sum[i];
                    gs[i] = __builtin_fmaf(sum[i], e[i], gs[i]);
                }
                if (bias_strip) {       // element rr of the fifth quad: sum over the wave's rows of dy_s[r][ob + 4 j + rr]; this wave's output: rr = wave
                    float col = 0.0f;
#pragma unroll
                    for (int v = 0; v < kSplitRowsWaves; ++v)
                        col += pick4(*reinterpret_cast<const f4 *>(gp + ((v * 5 + 4) * 64 + lane) * 4), wave);
                    const f4 eb = eps_quad(a.bias_quad0 + ((ob + 4 * j) >> 2), s, a.rng);
                    gbm += col;
                    gbs = __builtin_fmaf(col, pick4(eb, wave), gbs);
                }
            }
        }

        if (ok) {
            f4 om, os;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float u, v;
                finish_pair(gm[i], gs[i], m4[i], sd4[i], gf, kf, u, v);
                om[i] = u;
                os[i] = v;
            }
            store4<true, false>(a.gmu_w + o_own * K + kq, om);
            store4<true, false>(a.gsig_w + o_own * K + kq, os);
        }
        if (bias_strip && n == 0 && o_own < O) {
            float u, v;
            finish_pair(gbm, gbs, a.mu_b[o_own], a.sigma_b[o_own], gf, kf, u, v);
            a.gmu_b[o_own] = u;
            a.gsig_b[o_own] = v;
        }
    }

    float *dst = a.x_parts > 1 ? a.ws + (size_t)part * (size_t)a.s_loc * (size_t)R * (size_t)K : a.dx;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        if (s < a.s_loc) {
            f4 acc[RBW][4];
            {
                const MfmaSettled settled;
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[rb][i] = mx[s][rb][i].read(settled);
            }
            store_dx_tile<RBW>(acc, dst, s, r0, k0, j, n, a);
        }
    }
}

// Launch shape of the two kernels above; rb == 0: the layer goes to the two separate kernels.
struct OnePassPlan {
    int rb, smax;       // split: 16-row blocks per wave; else per workgroup.  smax: samples a lane holds accumulators for
    bool split;         // the waves split the rows and share the draws
    long parts, outs_per_part;
};

// Where the waves split the rows: 33 to 128 rows, one or two samples, half a million weights.  Measured against the two
// separate kernels at 2 samples: 33 rows 1.33x at 2160 x 8640, 64 rows 1.39-1.47x at 516 x 2100 and 2160 x 8640, 1.16x at 8192^2;
// at 100 and 128 rows those have become faster since the row limit was set (0.63x at 100 x 516 x 2100, 0.71-0.75x at 2160 x 8640,
// 0.87-0.90x at 8192^2 and 540 x 2160): an open end.  Slower on smaller layers, whose few tiles leave the barriers
// exposed, and with four samples (two waves per SIMD).  Up to 64 rows it also beats a wave drawing whole tiles for all rows.
constexpr int kSplitRowsFrom = kOnePassMaxRows + 1, kSplitRowsMaxRows = 128;
constexpr long kSplitRowsMinWeights = 512 * 1024;

// ws_bytes as in wgrad_shape
OnePassPlan one_pass_plan(const hot_linear_desc *d, bool input_gradients, int64_t ws_bytes)
{
    OnePassPlan p{0, 0, false, 1, 0};
    if (!input_gradients || d->rows > kSplitRowsMaxRows) return p;
    int rb, smax;
    bool split = false;
    long budget;        // workgroups that fill the chip once
    if (d->rows >= kSplitRowsFrom) {
        if (d->s_local > 2 || d->in_features * d->out_features < kSplitRowsMinWeights) return p;
        split = true;
        rb = d->rows > 64 ? 2 : 1;
        smax = 2;
        budget = 768;       // (three workgroups share a compute unit)
    } else {
        rb = d->rows > 16 ? 2 : 1;
        smax = d->s_local <= 2 ? 2 : (d->s_local <= 4 ? 4 : 8);
        if (d->s_local > 8 || rb * smax > kOnePassAccumulators) return p;
        budget = rb * smax <= 4 ? 512 : 256;    // (the lighter shapes fit two workgroups on a compute unit)
    }
    const long strips = (d->in_features + 63) / 64, tiles = (d->out_features + 15) / 16;
    // Workgroups for every compute unit from the strips of inputs alone where the strips are that many; fewer strips cut
    // the outputs into parts (a part keeps a tile per wave, four tiles where the waves share them), whose blocks of dx go
    // through the workspace.
    long parts = budget / strips;
    if (parts > tiles / 4) parts = tiles / 4;
    if (parts > 65535) parts = 65535;
    if (parts < 1) parts = 1;
    const int64_t block_bytes = (int64_t)d->s_local * d->rows * d->in_features * (int64_t)sizeof(float);
    if (parts > 1 && ws_bytes >= 0 && parts * block_bytes > ws_bytes) parts = ws_bytes / block_bytes;
    if (parts <= 1) {
        // no workspace (or one too small for two blocks): only where the strips alone nearly fill the chip
        if (strips < 200) return p;
        parts = 1;
    }
    p.outs_per_part = (tiles + parts - 1) / parts * 16;
    p.parts = (d->out_features + p.outs_per_part - 1) / p.outs_per_part;       // every part begins below O
    p.rb = rb;
    p.smax = smax;
    p.split = split;
    return p;
}

template <int RB, int SMAX>
void one_pass_go(const OnePassPlan &p, hipStream_t s, const LinearGradArgs &a)
{
    const size_t strip_bytes = (size_t)SMAX * 16 * RB * 64 * sizeof(float);
    const size_t tiles_bytes = (size_t)(kOnePassWaves - 1) * 16 * RB * 64 * sizeof(float);
    const dim3 grid((unsigned)((a.in_features + 63) / 64), (unsigned)p.parts);
    hot_linear_backward_one_pass_kernel<RB, SMAX><<<grid, dim3(64 * kOnePassWaves), strip_bytes > tiles_bytes ? strip_bytes : tiles_bytes, s>>>(a);
}

template <int RBW, int SMAX>
void split_rows_go(const OnePassPlan &p, hipStream_t s, const LinearGradArgs &a)
{
    const int copies = a.x_sample_stride != 0 ? a.s_loc : 1;
    const size_t lds = ((size_t)(4 + kSplitRowsWaves * 5) * 64 * 4 + (size_t)copies * 16 * RBW * kSplitRowsWaves * 64) * sizeof(float);
    const dim3 grid((unsigned)((a.in_features + 63) / 64), (unsigned)p.parts);
    hot_linear_backward_split_rows_kernel<RBW, SMAX><<<grid, dim3(64 * kSplitRowsWaves), lds, s>>>(a);
}

template <int RB>
void xgrad_go(dim3 grid, int waves, hipStream_t s, const LinearGradArgs &a)
{
    const size_t lds = waves > 1 ? (size_t)(waves - 1) * (size_t)(RB * 16) * 64 * sizeof(float) : 0;
    hot_linear_xgrad_kernel<RB><<<grid, dim3(64 * waves), lds, s>>>(a);
}

// Input gradients for many rows on too few workgroups of 256 rows (few 64-input groups, around a thousand
// rows): with a workspace the contraction over the outputs is cut into parts (1024 x 540 x 2160: 72
// workgroups, 0.15 ms with 64-row workgroups instead).  Returns the number of parts, 1 for none.
// ws_bytes as in wgrad_shape.
inline long xgrad_outs_per_part(const hot_linear_desc *d, int parts)
{
    return ((d->out_features + parts - 1) / parts + kXgradRowsKernelOutputs - 1) / kXgradRowsKernelOutputs * kXgradRowsKernelOutputs;
}

int xgrad_parts(const hot_linear_desc *d, int64_t ws_bytes)
{
    if (ws_bytes == 0 || d->rows < kSlab4MinRows) return 1;
    const long k_groups = (d->in_features + 63) / 64, gy = (d->rows + 255) / 256;
    const long wgs = k_groups * gy * d->s_local;
    if (wgs >= 256 || gy > 65535) return 1;
    const int64_t block_bytes = (int64_t)d->s_local * d->rows * d->in_features * (int64_t)sizeof(float);
    int parts = 1;
    // up to two workgroups per compute unit; a part keeps at least 64 outputs (four steps)
    while (parts < kXgradMaxParts && wgs * parts < 512 && d->out_features >= 64L * (2 * parts) &&
           (ws_bytes < 0 || (int64_t)(2 * parts) * block_bytes <= ws_bytes))
        parts *= 2;
    // (the parts must all exist: the last one begins below O)
    while (parts > 1 && xgrad_outs_per_part(d, parts) * (parts - 1) >= d->out_features) parts /= 2;
    return parts;
}

// The launch shapes of the two kernels above without parts: 64 * rb rows per workgroup of the kernel whose waves share the
// draws (rb == 0: it does not run), 16 * rb rows and `waves` shares of the contraction of the other.
struct XgradShape {
    int rb, waves;
    long gy;            // row blocks
};

inline XgradShape xgrad_rows_shape(const hot_linear_desc *d)
{
    // Rows per workgroup: 64 x cand.  All workgroups of these shapes are resident at once and those that share a
    // compute unit share its SIMDs, so the kernel takes (most workgroups on one compute unit) x (one workgroup's
    // work): per step 512 x cand matrix cycles per wave plus about 900 for the draw and the rest.  The count that
    // minimises the product wins: 7260 rows x 540 inputs x 2 samples are 522 workgroups of 256 rows (three on ten
    // compute units, two on the others: a third of the chip's time idle) but 684 of 192 rows (0.48 -> 0.40 ms).
    XgradShape best = {0, 1, 0};
    long best_cost = 0;
    const long k_groups = (d->in_features + 63) / 64;
    for (int cand = d->rows >= 256 ? 4 : 0; cand >= 1; --cand) {
        const long gy = (d->rows + 64 * cand - 1) / (64 * cand);
        const long wgs = k_groups * gy * d->s_local;
        if (gy > 65535 || wgs < 256) continue;     // (none fits: the other kernel, 15 % faster than 64-row workgroups there)
        const long cost = ((wgs + 255) / 256) * (512L * cand + 900);
        if (best.rb == 0 || cost < best_cost) {
            best = XgradShape{cand, 1, gy};
            best_cost = cost;
        }
    }
    return best;
}

inline XgradShape xgrad_shape(const hot_linear_desc *d)
{
    // Row tiles per workgroup: more of them share each drawn weight, fewer of them give more
    // workgroups and more waves per workgroup.  Take the most sharing that still puts a wave on
    // every SIMD of the chip (1024), else whatever yields the most waves.
    const long k_groups = (d->in_features + 63) / 64;
    const long o_blocks = (d->out_features + kXgradOutputsPerStep - 1) / kXgradOutputsPerStep;
    XgradShape best = {1, 1, 0};
    long most = -1;
    for (int cand = d->rows > 32 ? 4 : (d->rows > 16 ? 2 : 1); cand >= 1; cand >>= 1) {
        const long gy = (d->rows + kRowsPerTile * cand - 1) / (kRowsPerTile * cand);
        int waves = 1;
        while (waves < max_waves(cand) && k_groups * gy * d->s_local * waves < 8192 && 2L * waves <= o_blocks &&
               (size_t)(2 * waves - 1) * (size_t)(cand * 16) * 64 * sizeof(float) <= 65536)
            waves *= 2;
        const long total = k_groups * gy * d->s_local * waves;
        if (total > most) {
            most = total;
            best = XgradShape{cand, waves, gy};
        }
        if (total >= 1024) break;
    }
    return best;
}

// Whether the slab kernel takes the input gradients (where the kernel for tens to hundreds of rows does not).  A four-wave launch
// that leaves a quarter of its slots empty gives way to the parts of the kernel above where a workspace allows them.  Of the layers that
// still come here (short contractions on few inputs: 362 x 872 x 248 x 8, 905 x 504 x 584 x 3) the slab kernel would be the faster one
// by now (the whole call 0.75-0.90 of the time on 40 of them), but its sums are whole: 1.1-1.2 times as far from 64 bits.
inline bool xgrad_by_slab(const SlabShape &one, int parts_at_hand)
{
    return one.waves && !(parts_at_hand > 1 && one.waves == 4 && one.fill < 0.75);
}

// Whether the kernel for tens to hundreds of rows takes the input gradients (dy is its input, read in 16-byte quads).  Its four waves
// and the parts share an output's sum.  In bf16 pieces, with six roundings to 16 products, a sum ends 0.83-0.88 times as far from
// 64 bits as on the fp32 instruction in as many shares (measured at 33 to 2500 rows), so it needs as many shares as the kernel
// has that would run otherwise: with four against sixteen (81 x 2048 x 3624) the distance was 4.7e-7 against 2.8e-7.
inline DeepPlan deep_input_grad_plan(const hot_linear_desc *d, bool dy_aligned, int64_t ws_bytes)
{
    if ((d->out_features & 3) != 0 || !dy_aligned ||
        !deep_fits(d->rows, d->out_features, d->in_features, d->out_features, d->s_local, true))
        return kNoDeepPlan;
    const SlabShape slab = slab_input_grad_shape(d, true);
    const int parts_at_hand = xgrad_parts(d, ws_bytes);
    const int shares = xgrad_by_slab(slab, parts_at_hand) ? 1 : parts_at_hand > 1 ? parts_at_hand : xgrad_rows_shape(d).rb ? 1 : xgrad_shape(d).waves;
    const DeepPlan p = deep_plan(d->rows, d->out_features, d->in_features, d->out_features, d->s_local, true, ws_bytes,
                                 (shares + kDeepWaves - 1) / kDeepWaves);
    if (p.code < 0) return p;
    return deep_beats_slab(p, d->rows, d->out_features, d->in_features, d->s_local, d->s_local, slab_time(slab, 1, d->out_features)) ? p : kNoDeepPlan;
}

inline PlanePlan planes_input_grad_plan(const hot_linear_desc *d, bool dy_aligned, int64_t ws_bytes)
{
    if (ws_bytes == 0 || deep_input_grad_plan(d, dy_aligned, ws_bytes).code >= 0) return kNoPlanePlan;
    const SlabShape slab = slab_input_grad_shape(d, dy_aligned);
    if (slab.rbw == 1 || !xgrad_by_slab(slab, xgrad_parts(d, ws_bytes))) return kNoPlanePlan;
    return planes_instead(d->rows, d->out_features, d->in_features, d->s_local, true, slab_time(slab, 1, d->out_features), ws_bytes);
}

// Launch shape of the weight-gradient kernel.
struct WgradShape {
    long tiles, rows_per_part;
    int ob, split, parts;
    bool deep;
    bool tile;      // the kernel with tiles of 128 x 128 instead (no parts; the other fields do not apply)
};

// ws_bytes: what the caller's workspace holds (0: none; a negative value: as much as wanted, for the size query)
// wide_through_parts: count on eight row parts when deciding for two output groups per tile
WgradShape wgrad_shape_with(const hot_linear_desc *d, int64_t ws_bytes, bool wide_through_parts)
{
    WgradShape w;
    w.tile = false;
    const long k_groups = (d->in_features + 63) / 64;
    const long o_groups = (d->out_features + kColsPerWave - 1) / kColsPerWave;
    w.deep = d->rows >= kWgradDeepRows;
    // two output groups per tile where that still leaves a wave for every SIMD twice over after the row split
    // (four per tile were measured too: 90 against 95 TFLOP/s at 4096^2 x 1024, their registers spill)
    const long wide_waves = k_groups * ((o_groups + 1) / 2) * wgrad_max_split(2) * (wide_through_parts ? 8 : 1);
    w.ob = (d->rows >= kWgradWideRows && d->out_features >= 32 && wide_waves >= 2048) ? 2 : 1;
    w.tiles = k_groups * ((o_groups + w.ob - 1) / w.ob);
    // few tiles and many rows: let several waves share a tile (each then draws the tile's eps itself)
    // (up to a wave on every SIMD twice over; beyond that only while a wave keeps a thousand rows: finer pieces
    // even out the last round of waves, but every piece draws eps and adds through LDS again)
    w.split = 1;
    while (w.split < wgrad_max_split(w.ob) && d->rows >= 2L * w.split * kWgradRowsPerIter &&
           (w.tiles * w.split < 2048 || (w.tiles * w.split < 6144 && d->rows >= 1024L * w.split)))
        w.split *= 2;
    // Still too few waves for the chip (the tiles are few and a workgroup cannot hold more waves), or a number
    // of waves that fills the last round of the chip's 2048 wave slots (two per SIMD) badly: with a workspace
    // the rows are cut into parts for different workgroups, whose sums a second kernel adds in part order.
    // Measured: 1152 waves -> 4 or 8 parts (0.25 -> 0.19 ms), 2448 -> 2 parts (0.47 -> 0.42 ms; 4 parts lose),
    // 2048 -> none (2 parts: 0.19 -> 0.21 ms).  A wave keeps at least 128 rows.
    w.parts = 1;
    w.rows_per_part = 0;
    const long waves = w.tiles * w.split, last_round = waves % 2048;
    const bool fills_its_rounds = waves >= 2048 && (last_round == 0 || last_round > 1536);
    if (w.deep && ws_bytes != 0 && w.split == wgrad_max_split(w.ob) && !fills_its_rounds) {
        int parts = 1;
        while (parts < kWgradMaxParts && waves * parts < 4096 && d->rows >= 256L * w.split * (2 * parts) &&
               (ws_bytes < 0 || (int64_t)(2 * parts) * wgrad_part_bytes(d) <= ws_bytes))
            parts *= 2;
        if (parts > 1) {
            w.parts = parts;
            w.rows_per_part = ((d->rows + parts - 1) / parts + kWgradRowsPerIter - 1) / kWgradRowsPerIter * kWgradRowsPerIter;
        }
    }
    return w;
}

// the least tiles with which the tile kernel takes outputs that are no multiple of four (measured in wgrad_shape)
inline long wgrad_tile_ragged_tiles(long rows) { return rows >= 450 ? 230 : rows >= 208 ? 320 : 1100; }

// the shape of the kernel above
WgradShape wgrad_first_shape(const hot_linear_desc *d, int64_t ws_bytes)
{
    if (ws_bytes != 0 && d->rows >= 8192) {     // with parts, smaller layers afford the wide tiles too (16640 x 192 x 768: 51 -> 57 TFLOP/s)
        const WgradShape w = wgrad_shape_with(d, ws_bytes, true);
        if (w.parts > 1) return w;              // (else the workspace was too small for that)
    }
    return wgrad_shape_with(d, ws_bytes, false);
}

WgradShape wgrad_shape(const hot_linear_desc *d, int64_t ws_bytes)
{
    // Large layers at hundreds of rows and more: the kernel with tiles of 128 x 128.  Two workgroups share a compute
    // unit, so 512 tiles make a round, and a last round that is nearly empty costs as much as a full one; since the
    // kernel multiplies bf16 pieces it wins all the same (measured against the kernel above at 160 to 7260 rows: 1156
    // tiles 1.2-1.6x, 520 to 576 tiles 1.05-1.5x), and from 140 tiles and 256 rows on too (144 to 306 tiles 1.0-1.4x;
    // 128 tiles 0.8-0.95x, 85 tiles 0.5-0.8x: those stay with the kernel above, whose smaller tiles and row split fill
    // the chip better, as do few-tile layers whose rows a workspace spreads over the chip).
    const long tile_count = wgrad_tile_count(d);
    const bool fills = tile_count >= 512 || (tile_count >= 140 && d->rows >= 256 && !(ws_bytes != 0 && d->rows >= 8192));
    // Rows of dy off the 16-byte grid: only where the kernel above adds up all rows in one sum too (there this one is 0.82-0.88 times as far
    // from 64 bits; against two shorter sums 1.2 times, 1517 x 6448 x 1397 x 4 samples 5.0e-7 and 6.2e-7, against four 1.85 times), and
    // where it is faster.  From 450 rows and 230 tiles on 1.03-2.1x (788 x 1340 x 3429 x 3 290 -> 244 us, 473 x 5560 x 6805 x 2 1246 ->
    // 584; 455 x 272 x 8421 x 4, 198 tiles, 143 -> 155; 440 x 3964 x 1051 x 1, 279, 57 -> 60), from 208 rows and 320 tiles on 1.01-1.8x (212 x 1632 x 5714 x 4 242 -> 210; 332 x
    // 788 x 4859 x 2, 266 tiles, 76 -> 86), with fewer rows from 1100 tiles on 1.04-1.5x (134 x 7800 x 1149 x 3, 549, 122 -> 159).
    const WgradShape first = wgrad_first_shape(d, ws_bytes);
    const bool suits = (d->out_features & 3) == 0 || (first.split * first.parts == 1 && tile_count >= wgrad_tile_ragged_tiles(d->rows));
    if (wgrad_tile_fits(d) && d->rows >= kSlab4MinRows && fills && suits) {
        WgradShape w = wgrad_shape_with(d, 0, false);
        w.parts = 1;
        w.rows_per_part = 0;
        w.tile = true;
        return w;
    }
    return first;
}

// Most rows that a wave of the row parts may add up in one sum.  In as many rows the bf16 pieces are 0.75-0.85 times as far from 64
// bits as the fp32 instruction, so with 3/2 of the rows that a wave of the kernel adds up that would run otherwise they are not
// farther (533 x 920 x 464 x 3 samples, four waves against eight: 1.8e-7 in one sum, 1.3e-7 in two, that kernel 1.6e-7; 6151 x
// 2048 x 632 x 3: 6.1e-7, 4.3e-7 and 5.0e-7); up to 64 rows they are level.
inline long row_parts_most_rows(const hot_linear_desc *d, int64_t ws_bytes)
{
    const WgradShape w = wgrad_shape(d, ws_bytes);
    long most = d->rows;            // (the tile kernel adds up all rows in one such sum)
    if (!w.tile) most = (d->rows + (long)w.split * w.parts - 1) / ((long)w.split * w.parts) * 3 / 2;
    if (d->rows >= kRowPartLongRows && most > kRowPartLongMost) most = kRowPartLongMost;
    return most < kRowPartFineRows ? kRowPartFineRows : most / kRowPartRows * kRowPartRows;
}

// the best plan whose parts fit into `budget` bytes, with at most `most` rows to a wave's sum
inline RowPartsPlan row_parts_within(const hot_linear_desc *d, int64_t budget, long most)
{
    RowPartsPlan p = {0, 0, 1, false};
    const long tall = row_part_tiles<true>(d), wide = row_part_tiles<false>(d);
    p.xbig = tall <= wide;
    const long tiles = p.xbig ? tall : wide;
    const int64_t part_bytes = row_part_floats(d->in_features, d->out_features, d->s_local) * (int64_t)sizeof(float);
    // The number of parts whose rounds of workgroups (two per compute unit; a last round of one per compute unit runs its
    // workgroups faster) times steps per workgroup is least; a workgroup's start, its sums through LDS (once per chunk) and its
    // share of the finish kernel take about as long as four steps.  At least 128 rows to a part.
    const long step_rows = kRowPartRows * kRowPartWaves;
    double best = 0.0;
    for (int parts = 1; parts <= kRowPartMaxParts && parts * part_bytes <= budget && (parts == 1 || d->rows >= 128L * parts); ++parts) {
        const long rows = ((d->rows + parts - 1) / parts + kRowPartRows - 1) / kRowPartRows * kRowPartRows;
        if (rows * (parts - 1) >= d->rows) continue;       // (the parts must all exist)
        const long wgs = tiles * d->s_local * parts, last = wgs % 512;
        const double rounds = (double)(wgs / 512) + (last == 0 ? 0.0 : (last <= 256 ? 0.65 : 1.0));
        const long chunks = (rows + most * kRowPartWaves - 1) / (most * kRowPartWaves);
        const double cost = rounds * ((double)((rows + step_rows - 1) / step_rows) + 4.0 * (double)chunks);
        if (p.parts == 0 || cost < best) {
            best = cost;
            p.parts = parts;
            p.rows_per_part = rows;
            p.chunks = chunks;
        }
    }
    return p;
}

// ws_bytes: what the caller's workspace holds (negative: as much as wanted, for the size query).  With less than half of the
// parts it wants the chip would stand too empty: then the first kernel runs, which needs no workspace to split the rows.
inline RowPartsPlan row_parts_plan(const hot_linear_desc *d, int64_t ws_bytes)
{
    const RowPartsPlan none = {0, 0, 1, false};
    if (ws_bytes == 0 || !row_parts_suit(d)) return none;
    const long most = row_parts_most_rows(d, ws_bytes);
    const RowPartsPlan wanted = row_parts_within(d, row_parts_budget(d), most);
    const int64_t part_bytes = row_part_floats(d->in_features, d->out_features, d->s_local) * (int64_t)sizeof(float);
    if (ws_bytes < 0 || wanted.parts * part_bytes <= ws_bytes) return wanted;
    const RowPartsPlan p = row_parts_within(d, ws_bytes, most);
    return 2 * p.parts >= wanted.parts ? p : none;
}

}  // namespace

extern "C" {

int hot_linear_launch_shape(const hot_linear_desc *d, int which)
{
    if (!d || d->rows < 1 || d->in_features < 4 || (d->in_features & 3) || d->out_features < 1 || d->s_local < 1) return HOT_EINVAL;
    if (d->ldx < d->in_features || (d->ldx & 3) || d->x_sample_stride < 0 || which < 0 || which > 2) return HOT_EINVAL;
    if (d->out_features > (INT64_MAX / 8) / d->in_features || d->rows > (INT64_MAX / 8) / d->ldx) return HOT_EINVAL;
    if (which == 2) {
        const OnePassPlan p = one_pass_plan(d, true, -1);
        return p.rb ? (p.split ? 100 : 0) + 10 * p.rb + p.smax : 0;
    }
    auto code = [](const SlabShape &h, int st) { return h.waves ? 100 * (h.rbw == 1 ? 2 : h.waves) + 10 * h.cbw + st : 0; };
    if (which == 1) return deep_input_grad_plan(d, true, 0).code >= 0 ? 0 : code(slab_input_grad_shape(d, true), 1);
    if (deep_forward_plan(d).code >= 0) return 0;
    const SlabForwardPlan p = slab_forward_plan(d);
    return p.two.waves ? code(p.two, 2) + 1000 * (p.one.waves ? p.one.cbw : 0) : code(p.one, 1);
}

int64_t hot_linear_kernel_shape(const hot_linear_desc *d, int which, int64_t workspace_bytes)
{
    if (const int plain = hot_linear_launch_shape(d, 0); plain < 0) return plain;
    if (which < 0 || which > 2) return HOT_EINVAL;
    if (which == 2) {
        const RowPartsPlan p = row_parts_plan(d, workspace_bytes);
        return p.parts ? 1000 * (int64_t)p.chunks + 10 * p.parts + (p.xbig ? 1 : 0) : 0;
    }
    const DeepPlan p = which == 0 ? deep_forward_plan(d) : deep_input_grad_plan(d, true, workspace_bytes);
    auto code = [](int i) { return i < 0 ? 0 : 10 * kDeepShapes[i].rb + kDeepShapes[i].cb; };
    return p.code < 0 ? 0 : 1000000 * (int64_t)p.parts + 1000 * code(p.rest_code) + code(p.code);
}

int hot_linear_planes_shape(const hot_linear_desc *d, int which, int64_t workspace_bytes)
{
    if (const int plain = hot_linear_launch_shape(d, 0); plain < 0) return plain;
    if (which < 0 || which > 1) return HOT_EINVAL;
    const PlanePlan p = which == 0 ? planes_forward_plan(d, workspace_bytes) : planes_input_grad_plan(d, true, workspace_bytes);
    if (p.code < 0) return 0;
    const PlaneShape &h = p.apart ? kPlaneShapesApart[p.code] : kPlaneShapes[p.code];
    return (p.apart ? 100 : 0) + 10 * h.rb + h.cb;
}

int64_t hot_linear_planes_workspace_bytes(const hot_linear_desc *d, int which)
{
    if (const int plain = hot_linear_launch_shape(d, 0); plain < 0) return plain;
    if (which < 0 || which > 1) return HOT_EINVAL;
    if (which == 0) return planes_forward_plan(d, -1).bytes;
    const PlanePlan p = planes_input_grad_plan(d, true, -1);
    // (not where memory handed over for this alone would take the weight gradients off the kernel that they run on without any)
    if (p.bytes > 0 && hot_linear_backward_workspace_bytes(d) == 0 && wgrad_shape(d, p.bytes).tile != wgrad_shape(d, 0).tile) return 0;
    return p.bytes;
}

int64_t hot_linear_backward_workspace_bytes(const hot_linear_desc *d)
{
    if (!d || d->rows < 1 || d->in_features < 4 || (d->in_features & 3) || d->out_features < 1 || d->s_local < 1) return HOT_EINVAL;
    if (d->out_features > (INT64_MAX / 64) / d->in_features) return HOT_EINVAL;
    if (d->rows > (INT64_MAX / 64) / d->in_features || d->rows * d->in_features > (INT64_MAX / 64) / d->s_local) return HOT_EINVAL;
    const WgradShape w = wgrad_shape(d, -1);
    const int64_t for_weights = w.parts > 1 ? (int64_t)w.parts * wgrad_part_bytes(d) : 0;
    const DeepPlan deep = deep_input_grad_plan(d, true, -1);
    // (a dy off the 16-byte grid goes to the kernel whose waves share the draws: enough for its parts too)
    const int deep_parts = deep.code >= 0 ? deep.parts : 1, other_parts = xgrad_parts(d, -1);
    const int x_parts = deep_parts > other_parts ? deep_parts : other_parts;
    const int64_t for_inputs = x_parts > 1 ? (int64_t)x_parts * d->s_local * d->rows * d->in_features * (int64_t)sizeof(float) : 0;
    int64_t most = for_weights > for_inputs ? for_weights : for_inputs;     // the two kernels use it one after the other
    if (const RowPartsPlan plan = row_parts_plan(d, -1); plan.parts) {
        // (a power of two of the first kernel's parts where that is at most sixteen of them: so many the call has always asked for)
        const int64_t for_parts = plan.parts * row_part_floats(d->in_features, d->out_features, d->s_local) * (int64_t)sizeof(float);
        int64_t ask = 2 * wgrad_part_bytes(d);
        while (ask < for_parts) ask *= 2;
        if (ask > kWgradMaxParts * wgrad_part_bytes(d)) ask = for_parts;
        if (ask > most) most = ask;
    }
    // (whether input gradients will be asked for the query does not know: enough for either way)
    if (const OnePassPlan plan = one_pass_plan(d, true, -1); plan.rb && plan.parts > 1) {
        const int64_t for_one_pass = plan.parts * (int64_t)d->s_local * d->rows * d->in_features * (int64_t)sizeof(float);
        if (for_one_pass > most) most = for_one_pass;
    }
    return most;
}

int hot_linear_forward_rng_ws(const hot_linear_desc *d, const hot_rng *rng, const float *x, const float *mu_w,
                              const float *sigma_w, const float *mu_b, const float *sigma_b, float *y, void *workspace,
                              int64_t workspace_bytes, void *stream)
{
    if (!d || !x || !mu_w || !sigma_w || !y) return HOT_EINVAL;
    if (workspace && (workspace_bytes < 0 || !aligned16(workspace))) return HOT_EINVAL;
    if ((mu_b == nullptr) != (sigma_b == nullptr)) return HOT_EINVAL;
    if (d->rows < 1 || d->in_features < 4 || (d->in_features & 3) || d->out_features < 1 || d->s_local < 1) return HOT_EINVAL;
    if (d->ldx < d->in_features || (d->ldx & 3) || d->weight_offset < 0 || (d->weight_offset & 3)) return HOT_EINVAL;
    if (d->reserved != 0 || d->x_sample_stride < 0 || (d->x_sample_stride & 3)) return HOT_EINVAL;
    if (d->x_sample_stride != 0 && (d->rows > INT64_MAX / d->ldx || d->x_sample_stride < d->rows * d->ldx ||
                                    d->x_sample_stride > INT64_MAX / 4 / d->s_local))
        return HOT_EINVAL;
    if (mu_b && (d->bias_offset < 0 || (d->bias_offset & 3))) return HOT_EINVAL;
    if (!aligned16(x) || !aligned16(mu_w) || !aligned16(sigma_w) || !aligned4(y)) return HOT_EINVAL;
    if (mu_b && (!aligned4(mu_b) || !aligned4(sigma_b))) return HOT_EINVAL;
    if (d->out_features > (INT64_MAX / 8) / d->in_features) return HOT_EINVAL;
    Rng r;
    if (!make_rng(rng, d->s_local, r)) return HOT_EINVAL;

    LinearArgs a;
    a.rows = d->rows;
    a.in_features = d->in_features;
    a.out_features = d->out_features;
    a.ldx = d->ldx;
    a.x_sample_stride = d->x_sample_stride;
    a.s_loc = d->s_local;
    a.s_chunk = d->s_local;
    a.weight_quad0 = d->weight_offset >> 2;
    a.bias_quad0 = mu_b ? d->bias_offset >> 2 : 0;
    a.x = x;
    a.mu_w = mu_w;
    a.sigma_w = sigma_w;
    a.mu_b = mu_b;
    a.sigma_b = sigma_b;
    a.y = y;
    a.rng = r;

    hipStream_t s = static_cast<hipStream_t>(stream);
    // Given scratch, many rows: the weights drawn once into it.
    if (const PlanePlan plan = planes_forward_plan(d, workspace ? workspace_bytes : 0); plan.code >= 0) {
        SlabArgs b;
        b.rows = d->rows;
        b.contract = d->in_features;
        b.outs = d->out_features;
        b.ld_in = d->ldx;
        b.in_sample_stride = d->x_sample_stride;
        b.s_begin = b.s_end = 0;
        b.weight_quad0 = a.weight_quad0;
        b.bias_quad0 = a.bias_quad0;
        b.in = x;
        b.mu_w = mu_w;
        b.sigma_w = sigma_w;
        b.mu_b = mu_b;
        b.sigma_b = sigma_b;
        b.out = y;
        b.rng = r;
        planes_run<false>(plan, s, b, d->s_local, static_cast<char *>(workspace));
        return hot_detail::note_hip(hipGetLastError());
    }
    if (const DeepPlan plan = deep_forward_plan(d); plan.code >= 0) {
        DeepArgs b;
        b.rows = d->rows;
        b.contract = d->in_features;
        b.outs = d->out_features;
        b.ld_in = d->ldx;
        b.in_sample_stride = d->x_sample_stride;
        b.part_stride = 0;
        b.n_begin = 0;
        b.weight_quad0 = a.weight_quad0;
        b.bias_quad0 = a.bias_quad0;
        b.in = x;
        b.mu_w = mu_w;
        b.sigma_w = sigma_w;
        b.mu_b = mu_b;
        b.sigma_b = sigma_b;
        b.out = y;
        b.rng = r;
        deep_run<false>(plan, s, b, d->s_local);
        return hot_detail::note_hip(hipGetLastError());
    }
    // Many rows on a layer that fills the chip with its tiles: the kernel that stages x and the
    // drawn weights through LDS.  Samples that share x go two to a pass (they share every loaded row), an odd last one,
    // a single one and samples with inputs of their own one to a pass with tiles twice as wide.
    if (const SlabForwardPlan plan = slab_forward_plan(d); plan.two.waves || plan.one.waves) {
        SlabArgs b;
        b.rows = d->rows;
        b.contract = d->in_features;
        b.outs = d->out_features;
        b.ld_in = d->ldx;
        b.in_sample_stride = d->x_sample_stride;
        b.s_begin = b.s_end = 0;
        b.weight_quad0 = a.weight_quad0;
        b.bias_quad0 = a.bias_quad0;
        b.in = x;
        b.mu_w = mu_w;
        b.sigma_w = sigma_w;
        b.mu_b = mu_b;
        b.sigma_b = sigma_b;
        b.out = y;
        b.rng = r;
        if (plan.two.waves == 4 && plan.two.rbw == 1) slab_go<4, 1, 2, false, false, 1>(s, b, 0, plan.pair_samples);
        else if (plan.two.waves == 4) slab_go<4, 1, 2, false, false>(s, b, 0, plan.pair_samples);
        else if (plan.two.waves) {
            if (plan.two.cbw == 2) slab_go<8, 2, 2, false, false>(s, b, 0, plan.pair_samples);
            else slab_go<8, 1, 2, false, false>(s, b, 0, plan.pair_samples);
        }
        if (plan.one.waves) {
            if (d->x_sample_stride != 0) slab_go_singles<true, false>(plan.one, s, b, plan.pair_samples, d->s_local);
            else slab_go_singles<false, false>(plan.one, s, b, plan.pair_samples, d->s_local);
        }
        return hot_detail::note_hip(hipGetLastError());
    }
    // Many rows (from 256) and at least 128 workgroups of 256 rows: the kernel whose waves share every draw
    // through LDS (measured against the first kernel: 1.05-1.4x from there on, slower below).  Two samples per
    // pass and one column tile when several samples share x; a single sample, and samples with inputs of
    // their own (one per pass), afford two column tiles.
    {
        const bool xs = d->x_sample_stride != 0;
        const int no = (d->s_local == 1 || xs) ? 2 : 1;      // one sample per pass: its x loads serve two column tiles
        const long gx = (d->out_features + kColsPerWave * no - 1) / (kColsPerWave * no);
        const long gy = (d->rows + kRowsKernelRows - 1) / kRowsKernelRows;
        if (d->rows >= 256 && gx * gy >= 128 && gx <= 0x7fffffffL && gy <= 65535) {
            const dim3 grid((unsigned)gx, (unsigned)gy), block(64 * kRowsKernelWaves);
            if (xs) hot_linear_forward_rows_kernel<1, 2, true><<<grid, block, 0, s>>>(a);
            else if (no == 2) hot_linear_forward_rows_kernel<1, 2, false><<<grid, block, 0, s>>>(a);
            else hot_linear_forward_rows_kernel<2, 1, false><<<grid, block, 0, s>>>(a);
            return hot_detail::note_hip(hipGetLastError());
        }
    }
    // rows per workgroup: 16, 32 or 64 (one, two or four MFMA row tiles share every drawn weight)
    const int rb = d->rows > 32 ? 4 : (d->rows > 16 ? 2 : 1);
    // samples whose accumulators are live together (they share the loads of mu_W, sigma_W and x)
    int st = d->s_local >= 4 && four_samples_fit(rb, d->x_sample_stride != 0) ? 4 : (d->s_local >= 2 ? 2 : 1);
    const long gx = (d->out_features + kColsPerWave - 1) / kColsPerWave;
    const long gy = (d->rows + kRowsPerTile * rb - 1) / (kRowsPerTile * rb);
    if (gx > 0x7fffffffL || gy > 65535) return HOT_EINVAL;
    // waves per workgroup: enough to give every SIMD of the chip several waves, bounded by the
    // number of 32-input blocks and by 64 KiB of LDS for the partial tiles
    const long k_blocks = (d->in_features + kInputsPerIter - 1) / kInputsPerIter;
    int waves = 1;
    while (waves < max_waves(rb) && gx * gy * waves < 8192 && 2L * waves <= k_blocks &&
           (size_t)(2 * waves - 1) * (size_t)(st * rb * 4) * 64 * sizeof(float) <= 65536)
        waves *= 2;
    // Small layers leave most of the chip idle while one workgroup draws its samples one after the other (1 x 96 x 128 x 16
    // samples: eight workgroups, 28 us of dependent instructions): the samples then go to workgroups of their own, one each while all
    // waves fit on the chip at two per SIMD, else in as many chunks as do.
    const long waves_all = gx * gy * waves;
    // (a second wave per SIMD gains the four-tile workgroups nothing: their pairs of samples stay together.  Of the workgroups of sixteen
    // waves one runs on a compute unit at a time, four waves to a SIMD: they may be as many as the compute units.  With 128 before:
    // 8000 x 2000 x 2 samples x 16 rows 67.7 -> 49.8 us, 5000 x 1100 x 4 77 -> 41, 700 x 540 x 8 16.0 -> 10.4, 2048^2 x 2 20.7 -> 15.5; beyond
    // 256 a second round begins: 280, 2048 x 2240 x 2, 19.9 -> 24.2.)
    const bool sixteen = rb == 1 && waves == kMaxWaves;
    const long room = sixteen ? (long)kMaxWaves * kComputeUnits : rb == 4 && d->s_local == 2 ? 1024 : 2048;
    a.s_chunk = (d->s_local + st - 1) / st * st;
    if (waves_all * d->s_local <= room) {
        st = 1;
        a.s_chunk = 1;
    } else if (2 * waves_all <= room) {
        const int chunks = (int)(room / waves_all), per = (d->s_local + chunks - 1) / chunks;
        if (sixteen && per < st) st = per > 1 ? 2 : 1;
        a.s_chunk = (per + st - 1) / st * st;
    }
    const dim3 grid((unsigned)gx, (unsigned)gy, (unsigned)((d->s_local + a.s_chunk - 1) / a.s_chunk));
    if (rb == 4) linear_go<4>(st, grid, waves, s, a);
    else if (rb == 2) linear_go<2>(st, grid, waves, s, a);
    else linear_go<1>(st, grid, waves, s, a);
    return hot_detail::note_hip(hipGetLastError());
}

int hot_linear_forward_rng(const hot_linear_desc *d, const hot_rng *rng, const float *x, const float *mu_w,
                           const float *sigma_w, const float *mu_b, const float *sigma_b, float *y, void *stream)
{
    return hot_linear_forward_rng_ws(d, rng, x, mu_w, sigma_w, mu_b, sigma_b, y, nullptr, 0, stream);
}

int hot_linear_backward_rng_ws(const hot_linear_desc *d, int32_t s_total, double dataset_size, uint32_t flags,
                               const hot_rng *rng, const float *x, const float *dy, const float *mu_w,
                               const float *sigma_w, const float *mu_b, const float *sigma_b, float *grad_mu_w,
                               float *grad_sigma_w, float *grad_mu_b, float *grad_sigma_b, float *dx, void *workspace,
                               int64_t workspace_bytes, void *stream)
{
    if (!d || !x || !dy || !mu_w || !sigma_w || !grad_mu_w || !grad_sigma_w) return HOT_EINVAL;
    if (workspace && (workspace_bytes < 0 || !aligned16(workspace))) return HOT_EINVAL;
    if ((mu_b == nullptr) != (sigma_b == nullptr) || (mu_b == nullptr) != (grad_mu_b == nullptr) ||
        (mu_b == nullptr) != (grad_sigma_b == nullptr))
        return HOT_EINVAL;
    if (d->rows < 1 || d->in_features < 4 || (d->in_features & 3) || d->out_features < 1 || d->s_local < 1) return HOT_EINVAL;
    if (d->ldx < d->in_features || (d->ldx & 3) || d->weight_offset < 0 || (d->weight_offset & 3)) return HOT_EINVAL;
    if (d->reserved != 0 || d->x_sample_stride < 0 || (d->x_sample_stride & 3)) return HOT_EINVAL;
    if (d->x_sample_stride != 0 && (d->rows > INT64_MAX / d->ldx || d->x_sample_stride < d->rows * d->ldx ||
                                    d->x_sample_stride > INT64_MAX / 4 / d->s_local))
        return HOT_EINVAL;
    if (mu_b && (d->bias_offset < 0 || (d->bias_offset & 3))) return HOT_EINVAL;
    if (s_total < d->s_local || !(dataset_size > 0.0) || !(dataset_size < 1.0 / 0.0)) return HOT_EINVAL;
    if (flags != HOT_REDUCE_SUM && flags != HOT_REDUCE_MEAN && flags != HOT_REDUCE_NONE) return HOT_EINVAL;
    if (!aligned16(x) || !aligned16(mu_w) || !aligned16(sigma_w) || !aligned16(grad_mu_w) || !aligned16(grad_sigma_w) ||
        !aligned4(dy) || (dx && !aligned16(dx)))
        return HOT_EINVAL;
    if (mu_b && (!aligned4(mu_b) || !aligned4(sigma_b) || !aligned4(grad_mu_b) || !aligned4(grad_sigma_b))) return HOT_EINVAL;
    if (d->out_features > (INT64_MAX / 8) / d->in_features) return HOT_EINVAL;
    // element offsets into dy and dx must fit: S_loc * R * max(O, K)
    const int64_t widest = d->out_features > d->in_features ? d->out_features : d->in_features;
    if (d->rows > (INT64_MAX / 8) / widest || d->rows * widest > (INT64_MAX / 8) / d->s_local) return HOT_EINVAL;
    // the grid of the input-gradient kernel is (64-input groups, row blocks, samples): checked here so that
    // a refused call has launched nothing
    if (dx && (d->s_local > 65535 || (d->rows + kRowsPerTile - 1) / kRowsPerTile > 65535)) return HOT_EINVAL;
    Rng r;
    if (!make_rng(rng, d->s_local, r)) return HOT_EINVAL;

    LinearGradArgs a;
    a.rows = d->rows;
    a.in_features = d->in_features;
    a.out_features = d->out_features;
    a.ldx = d->ldx;
    a.x_sample_stride = d->x_sample_stride;
    a.s_loc = d->s_local;
    a.weight_quad0 = d->weight_offset >> 2;
    a.bias_quad0 = mu_b ? d->bias_offset >> 2 : 0;
    if (flags == HOT_REDUCE_NONE) {
        a.g = 1.0;
        a.k = 1.0 / dataset_size;
    } else if (flags == HOT_REDUCE_MEAN) {
        a.g = 1.0 / (double)d->s_local;
        a.k = 1.0 / dataset_size;
    } else {
        a.g = 1.0 / (double)s_total;
        a.k = (double)d->s_local / ((double)s_total * dataset_size);
    }
    a.x = x;
    a.dy = dy;
    a.mu_w = mu_w;
    a.sigma_w = sigma_w;
    a.mu_b = mu_b;
    a.sigma_b = sigma_b;
    a.gmu_w = grad_mu_w;
    a.gsig_w = grad_sigma_w;
    a.gmu_b = grad_mu_b;
    a.gsig_b = grad_sigma_b;
    a.dx = dx;
    a.ws = nullptr;
    a.rows_per_part = 0;
    a.x_parts = 1;
    a.outs_per_part = 0;
    a.rng = r;
    hipStream_t s = static_cast<hipStream_t>(stream);

    const long k_groups = (d->in_features + 63) / 64;
    const long o_groups = (d->out_features + kColsPerWave - 1) / kColsPerWave;
    if (k_groups * o_groups > 0x7fffff00L) return HOT_EINVAL;      // the grid may exceed the number of tiles by a few workgroups
    // Few rows and input gradients wanted: both gradients in one pass over the weights, every eps drawn once.
    if (const OnePassPlan plan = one_pass_plan(d, dx != nullptr, workspace ? workspace_bytes : 0); plan.rb) {
        a.ws = static_cast<float *>(workspace);
        a.x_parts = (int)plan.parts;
        a.outs_per_part = plan.outs_per_part;
        if (plan.split) {
            if (plan.rb == 2) split_rows_go<2, 2>(plan, s, a);
            else split_rows_go<1, 2>(plan, s, a);
        } else if (plan.rb == 2 && plan.smax == 2) one_pass_go<2, 2>(plan, s, a);
        else if (plan.rb == 2) one_pass_go<2, 4>(plan, s, a);
        else if (plan.smax == 2) one_pass_go<1, 2>(plan, s, a);
        else if (plan.smax == 4) one_pass_go<1, 4>(plan, s, a);
        else one_pass_go<1, 8>(plan, s, a);
        if (plan.parts > 1) {
            const long quads = (long)d->s_local * d->rows * d->in_features / 4;
            hot_linear_dx_sum_kernel<<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s>>>(dx, a.ws, quads, (int)plan.parts);
        }
        return hot_detail::note_hip(hipGetLastError());
    }
    const WgradShape shape = wgrad_shape(d, workspace ? workspace_bytes : 0);
    if (const RowPartsPlan plan = row_parts_plan(d, workspace ? workspace_bytes : 0); plan.parts) {
        a.ws = static_cast<float *>(workspace);
        a.rows_per_part = plan.rows_per_part;
        row_parts_go(plan, s, a, plan.xbig ? row_part_tiles<true>(d) : row_part_tiles<false>(d));
    } else if (shape.tile) {
        wgrad_tile_go(s, a, wgrad_tile_count(d));
    } else {
        const long tiles = shape.tiles;
        const int split = shape.split, ob = shape.ob;
        const bool deep = shape.deep;
        if (shape.parts > 1) {
            a.ws = static_cast<float *>(workspace);
            a.rows_per_part = shape.rows_per_part;
            if (ob == 2) wgrad_go_parts<2>(tiles, split, shape.parts, s, a);
            else wgrad_go_parts<1>(tiles, split, shape.parts, s, a);
        } else if (split > 1) {
            if (ob == 2) wgrad_go<true, true, 2>(tiles, split, s, a);
            else if (deep) wgrad_go<true, true, 1>(tiles, split, s, a);
            else wgrad_go<true, false, 1>(tiles, split, s, a);
        } else {
            if (ob == 2) wgrad_go<false, true, 2>(tiles, kWgradWaves, s, a);
            else if (deep) wgrad_go<false, true, 1>(tiles, kWgradWaves, s, a);
            else wgrad_go<false, false, 1>(tiles, kWgradWaves, s, a);
        }
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return hot_detail::note_hip(e);
    if (!dx) return HOT_OK;

    const int parts_at_hand = xgrad_parts(d, workspace ? workspace_bytes : 0);
    if (const DeepPlan plan = deep_input_grad_plan(d, aligned16(dy), workspace ? workspace_bytes : 0); plan.code >= 0) {
        DeepArgs b;
        b.rows = d->rows;
        b.contract = d->out_features;
        b.outs = d->in_features;
        b.ld_in = d->out_features;
        b.in_sample_stride = d->rows * d->out_features;
        b.part_stride = (long)d->s_local * d->rows * d->in_features;
        b.n_begin = 0;
        b.weight_quad0 = a.weight_quad0;
        b.bias_quad0 = 0;
        b.in = dy;
        b.mu_w = mu_w;
        b.sigma_w = sigma_w;
        b.mu_b = b.sigma_b = nullptr;
        b.out = plan.parts > 1 ? static_cast<float *>(workspace) : dx;
        b.rng = r;
        deep_run<true>(plan, s, b, d->s_local);
        if (plan.parts > 1) {
            const long quads = b.part_stride / 4;
            hot_linear_dx_sum_kernel<<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s>>>(dx, b.out, quads, plan.parts);
        }
        return hot_detail::note_hip(hipGetLastError());
    }
    // Many rows on a layer whose dx fills the chip with the tiles of the slab kernel: the kernel of the forward pass
    // with dy as its input and the weight tile drawn transposed (rows of dy are read in 16-byte quads).
    if (const SlabShape one = slab_input_grad_shape(d, aligned16(dy)); xgrad_by_slab(one, parts_at_hand)) {
        SlabArgs b;
        b.rows = d->rows;
        b.contract = d->out_features;
        b.outs = d->in_features;
        b.ld_in = d->out_features;
        b.in_sample_stride = d->rows * d->out_features;
        b.s_begin = b.s_end = 0;
        b.weight_quad0 = a.weight_quad0;
        b.bias_quad0 = 0;
        b.in = dy;
        b.mu_w = mu_w;
        b.sigma_w = sigma_w;
        b.mu_b = b.sigma_b = nullptr;
        b.out = dx;
        b.rng = r;
        if (const PlanePlan planes = planes_input_grad_plan(d, aligned16(dy), workspace ? workspace_bytes : 0); planes.code >= 0)
            planes_run<true>(planes, s, b, d->s_local, static_cast<char *>(workspace));
        else slab_go_singles<true, true>(one, s, b, 0, d->s_local);
        return hot_detail::note_hip(hipGetLastError());
    }
    // many rows: the workgroup-shared draw
    if (const int x_parts = parts_at_hand; x_parts > 1) {
        // too few 256-row workgroups: the outputs are cut into parts, summed from the workspace afterwards
        a.ws = static_cast<float *>(workspace);
        a.x_parts = x_parts;
        a.outs_per_part = xgrad_outs_per_part(d, x_parts);
        const long gy_c = (d->rows + 255) / 256;
        hot_linear_xgrad_rows_kernel<4><<<dim3((unsigned)(k_groups * x_parts), (unsigned)gy_c, (unsigned)d->s_local), dim3(256), 0, s>>>(a);
        const long quads = (long)d->s_local * d->rows * d->in_features / 4;
        hot_linear_dx_sum_kernel<<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s>>>(dx, a.ws, quads, x_parts);
        return hot_detail::note_hip(hipGetLastError());
    }
    if (const XgradShape h = xgrad_rows_shape(d); h.rb) {
        const dim3 grid((unsigned)k_groups, (unsigned)h.gy, (unsigned)d->s_local);
        if (h.rb == 4) hot_linear_xgrad_rows_kernel<4><<<grid, dim3(256), 0, s>>>(a);
        else if (h.rb == 3) hot_linear_xgrad_rows_kernel<3><<<grid, dim3(256), 0, s>>>(a);
        else if (h.rb == 2) hot_linear_xgrad_rows_kernel<2><<<grid, dim3(256), 0, s>>>(a);
        else hot_linear_xgrad_rows_kernel<1><<<grid, dim3(256), 0, s>>>(a);
        return hot_detail::note_hip(hipGetLastError());
    }
    const XgradShape h = xgrad_shape(d);
    const dim3 grid((unsigned)k_groups, (unsigned)h.gy, (unsigned)d->s_local);
    if (h.rb == 4) xgrad_go<4>(grid, h.waves, s, a);
    else if (h.rb == 2) xgrad_go<2>(grid, h.waves, s, a);
    else xgrad_go<1>(grid, h.waves, s, a);
    return hot_detail::note_hip(hipGetLastError());
}

int hot_linear_backward_rng(const hot_linear_desc *d, int32_t s_total, double dataset_size, uint32_t flags,
                            const hot_rng *rng, const float *x, const float *dy, const float *mu_w,
                            const float *sigma_w, const float *mu_b, const float *sigma_b, float *grad_mu_w,
                            float *grad_sigma_w, float *grad_mu_b, float *grad_sigma_b, float *dx, void *stream)
{
    return hot_linear_backward_rng_ws(d, s_total, dataset_size, flags, rng, x, dy, mu_w, sigma_w, mu_b, sigma_b, grad_mu_w,
                                      grad_sigma_w, grad_mu_b, grad_sigma_b, dx, nullptr, 0, stream);
}

}  // extern "C"
