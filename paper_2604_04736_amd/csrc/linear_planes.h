// Part of linear.hip: products with drawn weights that lie in memory as bf16 pieces.
//
// At thousands of rows every tile of rows of the slab kernel draws its weights again, and every tile of outputs cuts x again:
// 7260 x 2160 x 540 forward on tiles of 512 x 32 cuts every element of x seventeen times, and its matrix pipes ran 30 % of the time.
// Given a workspace the weights are therefore drawn and cut ONCE, by hot_linear_draw_planes_kernel, into three planes of bf16 in
// the order in which the lanes of the matrix instruction take them, and hot_linear_planes_kernel multiplies: a wave reads its
// weight operands straight from memory into registers (1 KB per instruction, no LDS, no address arithmetic), x is cut once per
// workgroup and shared through LDS.  Products, their order and the order of the contraction are the slab kernel's, so results
// are the same bit for bit.  Layers of the kernel for tens to hundreds of rows, whose four waves share a sum, come here with the five
// small products of every pair of factors in accumulators of their own (APART): the large ones then take one rounding per
// step instead of six, and the sums end 0.76-0.80 times as far from 64 bits as that kernel's (190 layers).  Measured (two samples, product kernel + draw): 7260 x 2160 x 540 forward 325 -> 181 + 5 us, its input
// gradients 270 -> 171 + 8, 16640 x 192 x 768 80 -> 60 + 4 and 96 -> 59 + 5.
#ifndef HOT_LINEAR_PLANES_H
#define HOT_LINEAR_PLANES_H

namespace {

constexpr long kPlaneBytes = 1024;               // one piece of a block: 32 outputs x 16 contraction indices
constexpr long kBlockBytes = 3 * kPlaneBytes;

inline __host__ __device__ long plane_steps(long contract) { return (contract + kSlabK - 1) / kSlabK; }
inline __host__ __device__ long plane_blocks(long outs) { return (outs + 31) / 32; }

struct PlaneDrawArgs {
    long contract, outs;         // C, N
    int steps, blocks;
    int samples, s_chunk;
    long sample_bytes;           // of the planes of one sample
    long weight_quad0;
    const float *mu_w, *sigma_w;
    char *planes;
    Rng rng;
};

constexpr int kDrawWaves = 4;

// Planes of a sample: [step of 16 contraction indices][block of 32 outputs][piece][lane l: 16 bytes], lane l the output l % 32 and
// the indices 4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3 of the step with h = l / 32; zeros beyond the layer's edges.  What bounds it: the
// draw (8.7e11 eps/s) and the stores, six bytes per weight and sample.  A thread makes whole 16-byte lanes.  Along the contraction a store
// instruction then covers runs of 128 bytes, eight outputs; across it (TR) a thread holds four neighbouring outputs, so an instruction
// stores 16 bytes in every 64 and four of them fill the lines together: 8192^2 x 2 samples take 330 us (4.1 TB/s) against 253 (5.3).  Both gradients' orders come from the same rows of mu and sigma: along the
// contraction (forward) a thread draws two quads, across it (TR, input gradients) the eight quads of 4 outputs x 8 indices.

template <bool TR>
__global__ void __launch_bounds__(64 * kDrawWaves)
hot_linear_draw_planes_kernel(PlaneDrawArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int C = (int)a.contract, N = (int)a.outs;
    const window_t mu_win = window(a.mu_w, (unsigned)((long)C * N * 4)), sg_win = window(a.sigma_w, (unsigned)((long)C * N * 4));
    const int s_lo = (int)blockIdx.z * a.s_chunk, s_hi = s_lo + a.s_chunk < a.samples ? s_lo + a.s_chunk : a.samples;
    constexpr int QS = TR ? 8 : 2;               // quads a thread draws per sample
    // Not TR: lane = (output l / 8 of the wave's eight, step l % 8 / 2 of four, half l % 2); quads half and half + 2 of the step.
    // TR: lane = (quad l % 32 of 128 outputs, half l / 32), the wave's own step; contraction indices 4 half .. + 3 and 8 + 4 half .. + 3.
    const int step = TR ? (int)blockIdx.y * kDrawWaves + wave : (int)blockIdx.x * 4 + (lane >> 1 & 3);
    const int half = TR ? lane >> 5 : lane & 1;
    const int n = TR ? (int)blockIdx.x * 128 + 4 * (lane & 31) : (int)blockIdx.y * 32 + wave * 8 + (lane >> 3);
    if (step >= a.steps || n >= 32 * a.blocks) return;
    f4 m4[QS], sd4[QS];
    long quad[QS];
#pragma unroll
    for (int i = 0; i < QS; ++i) {
        const int c = TR ? step * kSlabK + 4 * half + (i & 3) + 8 * (i >> 2) : step * kSlabK + 4 * half + 8 * i;
        const bool ok = c < C && n < N;
        const long flat = TR ? (long)c * N + n : (long)n * C + c;
        const int off = (int)(ok ? (unsigned)(flat * 4) : kOutside);
        m4[i] = window_load4<false>(mu_win, off);
        sd4[i] = window_load4<false>(sg_win, off);
        quad[i] = a.weight_quad0 + (flat >> 2);
    }
    char *const at = a.planes + ((size_t)step * (size_t)a.blocks + (size_t)(n >> 5)) * kBlockBytes + (half * 32 + (n & 31)) * 16;
    for (int s = s_lo; s < s_hi; ++s) {
        f4 w4[QS];
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            const f4 e = eps_quad(quad[i], s, a.rng);
#pragma unroll
            for (int c = 0; c < 4; ++c) w4[i][c] = __builtin_fmaf(sd4[i][c], e[c], m4[i][c]);
        }
        char *const to = at + (size_t)s * (size_t)a.sample_bytes;
#pragma unroll
        for (int e = 0; e < (TR ? 4 : 1); ++e) {
            bf8 p[3];
            if constexpr (TR) split8_bf16(f4{w4[0][e], w4[1][e], w4[2][e], w4[3][e]}, f4{w4[4][e], w4[5][e], w4[6][e], w4[7][e]}, p[0], p[1], p[2]);
            else split8_bf16(w4[0], w4[1], p[0], p[1], p[2]);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<bf8 *>(to + pl * kPlaneBytes + e * 16) = p[pl];
        }
    }
}

// What it works on is the slab kernel's product (see SlabArgs).  Four waves as 2 x 2, each with RB x CB blocks of 32 x 32; x goes
// through two LDS buffers with one barrier per step, in the middle of its matrix instructions, so that behind the barrier
// nobody waits: the products of the second half have their operands, and those of the next step are read meanwhile.  The
// operands of a step are a second set of registers.  XOR 12 on the second half's rows spreads the eight-byte stores and the
// sixteen-byte reads of a plane over the banks.  What bounds it: the matrix pipes at the clock that the card's power leaves
// (1.3-1.9 GHz; pipes busy 70-80 %), vector instructions between them and the last round of workgroups.  Larger tiles cut x and
// read weights less often, smaller ones fill the chip: kPlaneShapes.
struct PlaneArgs {
    long rows, contract, outs;   // R, C, N
    long ld_in, in_sample_stride;
    int steps, blocks;
    long sample_bytes;
    int row_tiles, col_tiles, items, per_xcd;
    int rows_first;              // neighbouring workgroups: 1 the row tiles of a column, 0 the column tiles of a row
    long bias_quad0;
    long weight_quad0;           // (APART, for sums that are formed again)
    const float *in, *mu_w, *sigma_w, *mu_b, *sigma_b;
    const char *planes;
    float *out;                  // [S, R, N]
    Rng rng;
};

template <int RB, int CB, int OCC, bool APART>
__global__ void __launch_bounds__(256, OCC)
hot_linear_planes_kernel(PlaneArgs a)
{
    constexpr int KS = kSlabK, ROWS = 64 * RB, OUTS = 64 * CB;
    __shared__ __attribute__((aligned(16))) float xs0[ROWS * KS * 3 / 2], xs1[ROWS * KS * 3 / 2];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wr = wave >> 1, wc = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;
    const int C = (int)a.contract, N = (int)a.outs, R = (int)a.rows;
    const int item = ((int)blockIdx.x % kXcds) * a.per_xcd + (int)blockIdx.x / kXcds;
    if ((int)blockIdx.x / kXcds >= a.per_xcd || item >= a.items) return;         // the whole workgroup
    const int tiles = a.row_tiles * a.col_tiles, s = item / tiles, tile = item % tiles;
    const int rt = a.rows_first ? tile % a.row_tiles : tile / a.col_tiles, ct = a.rows_first ? tile / a.row_tiles : tile % a.col_tiles;
    const int r0 = rt * ROWS, n0 = ct * OUTS;
    lds_char *const X0 = (lds_char *)(lds_float *)xs0, *const X1 = (lds_char *)(lds_float *)xs1;

    // x: this thread's quads are row 64 j + t / 4, indices 4 (t % 4) .. + 3 of a step; rows beyond the last repeat it (nothing of theirs is stored)
    const int q = t & 3;
    const window_t in_win = window(a.in + (size_t)s * (size_t)a.in_sample_stride, (unsigned)((((long)R - 1) * a.ld_in + C) * 4));
    unsigned x_off[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int row = r0 + 64 * j + (t >> 2);
        x_off[j] = (unsigned)(((long)(row < R ? row : R - 1) * a.ld_in + 4 * q) * 4);
    }
    // ... which go, cut, to the block of row / 32, half q % 2, eight bytes of the lane's sixteen
    const int x_h = q & 1, x_put = (t >> 7) * 3 * 1024 + (x_h * 32 + (((t >> 2) & 31) ^ (12 * x_h))) * 16 + (q >> 1) * 8;
    const int x_get = wr * RB * 3 * 1024 + (half * 32 + (l32 ^ (12 * half))) * 16;

    // the weights: straight from memory into operand registers
    const unsigned step_bytes = (unsigned)(a.blocks * kBlockBytes);
    const window_t w_win = window(reinterpret_cast<const float *>(a.planes + (size_t)s * (size_t)a.sample_bytes), (unsigned)(a.steps * (long)step_bytes));
    unsigned w_off = (unsigned)((n0 / 32 + wc * CB) * kBlockBytes + lane * 16);

    f4 xr[RB];
    auto ask_x = [&](int cb0) {
        const bool ok = cb0 + 4 * q < C;
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            xr[j] = window_load4<false>(in_win, ok ? x_off[j] : kOutside);
            x_off[j] += KS * 4;
        }
    };
    auto put_x = [&](int j, lds_char *to) {
        unsigned pc[3][2];
        split2_bf16(xr[j][0], xr[j][1], pc[0][0], pc[1][0], pc[2][0]);
        split2_bf16(xr[j][2], xr[j][3], pc[0][1], pc[1][1], pc[2][1]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *(lds_u2 *)(to + x_put + (2 * j * 3 + pl) * 1024) = u2{pc[pl][0], pc[pl][1]};
    };
    bf8 av[2][RB][3], bv[2][CB][3];
    auto get_x = [&](int u, int rb, const lds_char *from) {
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) av[u][rb][pl] = *(const volatile lds_bf8 *)(from + x_get + (rb * 3 + pl) * 1024);
    };
    auto ask_w = [&](int u, int cb) {
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) bv[u][cb][pl] = __builtin_bit_cast(bf8, window_load4<false>(w_win, w_off + cb * (unsigned)kBlockBytes + pl * 1024u));
    };
    Acc32x32 mm[RB][CB], small[APART ? RB : 1][APART ? CB : 1];

    // One step on tile i, whose operands are in registers (set u).  First half: x of tile i + 1 is cut and put into LDS, its weights and
    // x of tile i + 2 are sent for; barrier; second half: the operands of tile i + 1 are read.
    auto step = [&](int u, int cb0, lds_char *to) {
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
        constexpr int GROUPS = 6 * CB, MID = GROUPS / 2;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int cb = g / 6, i = g % 6;
            // what is done beside the products of this group
            if (g < CB) {
                if (g == 0) w_off += step_bytes;
                ask_w(u ^ 1, g);
            }
#pragma unroll
            for (int j = 0; j < RB; ++j)
                if (g == 1 + j * (MID - 1) / RB) put_x(j, to);
            if (g == MID - 1) ask_x(cb0 + 2 * KS);
            if (g == MID) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (g == MID + rb) get_x(u ^ 1, rb, to);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if constexpr (APART) (i < 5 ? small : mm)[rb][cb].mac(av[u][rb][PA[i]], bv[u][cb][PB[i]]);
                else mm[rb][cb].mac(av[u][rb][PA[i]], bv[u][cb][PB[i]]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    ask_x(0);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) ask_w(0, cb);
#pragma unroll
    for (int j = 0; j < RB; ++j) put_x(j, X0);
    ask_x(KS);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) get_x(0, rb, X0);
    for (int cb0 = 0; cb0 < C; cb0 += 2 * KS) {          // (an odd number of steps is followed by one on zeros)
        step(0, cb0, X1);
        step(1, cb0 + KS, X0);
    }
    const MfmaSettled settled;

    int r0w = r0 + wr * 32 * RB + 4 * half, n0l = n0 + wc * 32 * CB + l32;
    asm volatile("" : "+v"(r0w), "+v"(n0l));       // (so that the offsets below are formed here, not ahead of the loop)
    const window_t out_win = window(a.out + (size_t)s * (size_t)R * (size_t)N, (unsigned)((long)R * N * 4));
    auto bias_of = [&](int n) {
        return a.mu_b && n < N ? __builtin_fmaf(a.sigma_b[n], pick4_of(eps_quad(a.bias_quad0 + (n >> 2), s, a.rng), n & 3), a.mu_b[n]) : 0.0f;
    };
    [[maybe_unused]] bool special = false;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int n = n0l + 32 * cb;
        const bool n_ok = n < N;
        const float bias = bias_of(n);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            f16v acc = mm[rb][cb].read(settled);
            if constexpr (APART) acc += small[rb][cb].read(settled);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = r0w + 32 * rb + 8 * (i >> 2) + (i & 3);
                const float sum = acc[i] + bias;
                if constexpr (APART) special |= n_ok && row < R && sum != sum;
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, sum), out_win,
                                                      (n_ok && row < R) ? (int)(((unsigned)row * (unsigned)N + (unsigned)n) * 4u) : (int)kOutside, 0, 0);
            }
        }
    }
    // (where the other kernel forms sums again that the pieces leave as NaN, so does this one: each lane looks at what it stored)
    if constexpr (APART) {
        if (__builtin_amdgcn_ballot_w64(special) == 0) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        float *const y0 = a.out + (size_t)s * (size_t)R * (size_t)N;
#pragma unroll 1
        for (int k = 0; k < RB * CB * 16; ++k) {
            const int i = k & 15, row = r0w + 32 * ((k >> 4) % RB) + 8 * (i >> 2) + (i & 3), n = n0l + 32 * ((k >> 4) / RB);
            const bool mine = row < R && n < N;
            float *const y = y0 + (mine ? (size_t)row * (size_t)N + (size_t)n : 0);
            const bool again = mine && *y != *y;
            if (__builtin_amdgcn_ballot_w64(again) == 0) continue;
            const float *in = a.in + (size_t)s * (size_t)a.in_sample_stride + (size_t)(row < R ? row : R - 1) * (size_t)a.ld_in;
            const float sum = deep_plain_sum<false, 32>(a, in, s, n, 0, C, again);
            if (again) *y = sum + bias_of(n);
        }
    }
}

// ---------------------------------------------------------------------------------
// Host side.  What a shape costs, in microseconds: once; per round of workgroups; per step of 16 contraction indices with 1 .. `resident`
// workgroups on a compute unit (as many as its registers admit); and per workgroup to a compute unit on average, a step and as a
// whole (the card's power and memory, which the workgroups share).  Fitted to 300 products of 128 to 16640 rows, 24 to 8192
// contraction indices and 24 to 8551 outputs (within 6 %); the shape that the model picks is 0.5 % behind the fastest on average, 15 % at
// worst.  Tiles of 256 x 256 (302 products of 400 to 12000 rows, within 8 %) hold 256 accumulators, one wave to a SIMD, and are what large
// products take: 4096^3 x 2 samples 1270 -> 1139 us, 1005 x 7052 x 6900 x 2 1314 -> 1094.  Nothing covers such a workgroup's start and end, so they
// are taken from kPlaneLongSteps steps on and where the model sees them ahead by kPlaneLargeAhead (by the bare model 1000 products: with under 300
// indices 0.91 times as fast, 0.96 with 300 to 400, 1.00 with 500 to 600, 1.03 with 700 to 800, 1.08 from 1200 on; whole backward passes 0.97
// to 1.04).  256 x 192 were hardly ever ahead of both of their neighbours.
struct PlaneShape {
    int rb, cb, resident;
    double once, round, us[6], share, each;
};
constexpr PlaneShape kPlaneShapes[] = {{3, 3, 1, 1.6, 5.9, {0.849}, 0.375, 1.57},
                                       {2, 2, 2, 3.1, 1.2, {0.463, 0.878}, 0.133, 1.44},
                                       {2, 3, 2, 3.0, 2.6, {0.60, 1.213}, 0.202, 1.75},
                                       {1, 3, 3, 3.1, 0.0, {0.441, 0.766, 1.185}, 0.082, 1.34},
                                       {2, 1, 4, 2.7, 0.0, {0.357, 0.563, 0.871, 1.159}, 0.065, 0.75},
                                       {3, 1, 3, 3.4, 0.0, {0.464, 0.761, 1.175}, 0.119, 1.2},
                                       {1, 1, 6, 0.0, 0.0, {0.297, 0.303, 0.425, 0.594, 0.747, 0.817}, 0.079, 0.49},
                                       {4, 4, 1, 0.0, 5.6, {1.185}, 0.821, 10.1}};
constexpr bool plane_shape_large(const PlaneShape &h) { return h.rb * h.cb == 16; }       // (256 x 256, the last shape)
constexpr long kPlaneLongSteps = 40;
constexpr double kPlaneLargeAhead = 1.03;
constexpr int kPlaneCodes = sizeof(kPlaneShapes) / sizeof(kPlaneShapes[0]);
// The same with two sets of accumulators (190 products of 64 to 7800 rows, within 5 %, 0.8 % behind the fastest on average).
constexpr PlaneShape kPlaneShapesApart[] = {{2, 2, 2, 2.1, 2.3, {0.45, 0.805}, 0.17, 0.98},
                                            {2, 3, 1, 0.7, 5.5, {0.581}, 0.282, 0.61},
                                            {1, 3, 2, 2.2, 0.5, {0.443, 0.764}, 0.085, 1.54},
                                            {1, 1, 5, 0.3, 0.0, {0.305, 0.305, 0.364, 0.538, 0.614}, 0.085, 0.84}};
constexpr int kPlaneCodesApart = sizeof(kPlaneShapesApart) / sizeof(kPlaneShapesApart[0]);

// Most bytes of planes (below 2 GiB, since offsets into a sample's are 32 bits).  Beyond the 256 MiB of the memory-side cache they are
// still faster than drawing in every tile: on 42 layers of 256 to 900 MiB 1.14 times forward, 1.12 the whole backward pass, none
// slower (1337 x 3744 x 6132 x 2 forward 802 -> 625 us, 2048 x 8192^2 x 1 1365 -> 1242, 1024 x 8192^2 x 2 1379 -> 1338).  With the small products
// apart, for layers of fewer rows, it was not measured and stays at what that cache holds.
constexpr int64_t kPlanesMostBytes = (int64_t)1024 << 20, kPlanesMostBytesApart = (int64_t)256 << 20;
constexpr long kPlanesMostTiles = (1L << 24) - kXcds;        // (one grid dimension holds fewer than 2^32 threads)

struct PlanePlan {
    int code;            // index into kPlaneShapes or kPlaneShapesApart, -1: none
    bool apart;
    int64_t bytes;       // of the planes of all samples
    double time;         // microseconds, the draw included
};
constexpr PlanePlan kNoPlanePlan = {-1, false, 0, 0.0};

inline PlanePlan plane_plan(long R, long C, long N, int S, bool tr, bool apart)
{
    const long steps = plane_steps(C), blocks = plane_blocks(N);
    if (S > 65535 || steps > 4 * 65535 || blocks > 65535 || steps > (apart ? kPlanesMostBytesApart : kPlanesMostBytes) / kBlockBytes / blocks / S)
        return kNoPlanePlan;
    PlanePlan best = {-1, apart, steps * blocks * S * kBlockBytes, 0.0};
    for (int i = 0; i < (apart ? kPlaneCodesApart : kPlaneCodes); ++i) {
        const PlaneShape &h = apart ? kPlaneShapesApart[i] : kPlaneShapes[i];
        const long wgs_of_sample = ((R + 64 * h.rb - 1) / (64 * h.rb)) * ((N + 64 * h.cb - 1) / (64 * h.cb));
        if (wgs_of_sample > kPlanesMostTiles / S) continue;
        const long wgs = wgs_of_sample * S, round = (long)kComputeUnits * h.resident, full = wgs / round, left = wgs % round;
        const double taken = (double)(steps + (steps & 1));          // (steps go in pairs)
        double t = h.once + (double)full * (taken * h.us[h.resident - 1] + h.round);
        if (left) t += taken * h.us[(left + kComputeUnits - 1) / kComputeUnits - 1] + h.round;
        t += (double)wgs / kComputeUnits * (taken * h.share + h.each);
        const bool large = plane_shape_large(h);
        if (large && steps < kPlaneLongSteps) continue;
        if (best.code < 0 || (large ? kPlaneLargeAhead : 1.0) * t < best.time) {
            best.code = i;
            best.time = t;
        }
    }
    best.time += (tr ? 5.0 : 4.0) + (double)C * (double)N * (double)S * (tr ? 2.4e-6 : 2.0e-6);
    return best;
}

template <int RB, int CB, int OCC, bool APART = false>
void planes_go(hipStream_t s, PlaneArgs a, int samples)
{
    a.row_tiles = (int)((a.rows + 64 * RB - 1) / (64 * RB));
    a.col_tiles = (int)((a.outs + 64 * CB - 1) / (64 * CB));
    a.items = a.row_tiles * a.col_tiles * samples;
    a.per_xcd = (a.items + kXcds - 1) / kXcds;
    hot_linear_planes_kernel<RB, CB, OCC, APART><<<dim3((unsigned)(kXcds * a.per_xcd)), dim3(256), 0, s>>>(a);
}

// Draws the planes of all samples into `planes` (p.bytes of them) and multiplies.
template <bool TR>
void planes_run(const PlanePlan &p, hipStream_t s, const SlabArgs &b, int samples, char *planes)
{
    PlaneDrawArgs d;
    d.contract = b.contract;
    d.outs = b.outs;
    d.steps = (int)plane_steps(b.contract);
    d.blocks = (int)plane_blocks(b.outs);
    d.samples = samples;
    d.sample_bytes = (long)d.steps * d.blocks * kBlockBytes;
    d.weight_quad0 = b.weight_quad0;
    d.mu_w = b.mu_w;
    d.sigma_w = b.sigma_w;
    d.planes = planes;
    d.rng = b.rng;
    const unsigned gx = (unsigned)(TR ? (d.blocks + 3) / 4 : (d.steps + 3) / 4), gy = (unsigned)(TR ? (d.steps + kDrawWaves - 1) / kDrawWaves : d.blocks);
    // the samples of a weight in one thread, which loads mu and sigma once, where that leaves four workgroups to a compute unit
    const long chunks = (long)gx * gy >= 4 * kComputeUnits ? 1 : samples;
    d.s_chunk = (int)((samples + chunks - 1) / chunks);
    hot_linear_draw_planes_kernel<TR><<<dim3(gx, gy, (unsigned)chunks), dim3(64 * kDrawWaves), 0, s>>>(d);

    PlaneArgs a;
    a.rows = b.rows;
    a.contract = b.contract;
    a.outs = b.outs;
    a.ld_in = b.ld_in;
    a.in_sample_stride = b.in_sample_stride;
    a.steps = d.steps;
    a.blocks = d.blocks;
    a.sample_bytes = d.sample_bytes;
    // Neighbouring workgroups, which run at the same time behind one L2, share the larger operand (1024 x 8192^2: 1336 -> 1238 us on tiles of 128 x 128)
    a.rows_first = 6 * b.outs > 4 * b.rows;
    a.bias_quad0 = b.bias_quad0;
    a.weight_quad0 = b.weight_quad0;
    a.in = b.in;
    a.mu_w = b.mu_w;
    a.sigma_w = b.sigma_w;
    a.mu_b = b.mu_b;
    a.sigma_b = b.sigma_b;
    a.planes = planes;
    a.out = b.out;
    a.rng = b.rng;
    if constexpr (!TR) {
        if (p.apart) switch (p.code) {
            case 0: return planes_go<2, 2, 2, true>(s, a, samples);
            case 1: return planes_go<2, 3, 1, true>(s, a, samples);
            case 2: return planes_go<1, 3, 2, true>(s, a, samples);
            default: return planes_go<1, 1, 2, true>(s, a, samples);
            }
    }
    switch (p.code) {
    case 0: return planes_go<3, 3, 1>(s, a, samples);
    case 1: return planes_go<2, 2, 2>(s, a, samples);
    case 2: return planes_go<2, 3, 2>(s, a, samples);
    case 3: return planes_go<1, 3, 2>(s, a, samples);
    case 4: return planes_go<2, 1, 2>(s, a, samples);
    case 5: return planes_go<3, 1, 2>(s, a, samples);
    case 6: return planes_go<1, 1, 2>(s, a, samples);
    default: return planes_go<4, 4, 1>(s, a, samples);
    }
}

}  // namespace

#endif  // HOT_LINEAR_PLANES_H
