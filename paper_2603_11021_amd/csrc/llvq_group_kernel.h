// Closed-form group scales (paper App. J): per row i the Hessian-weighted least-squares gains of its fixed blocks,
// (M_i + lambda I) s_i = r_i with M_i[p][q] = Wq_{i,p} H_{pq} Wq_{i,q}^T and r_i[p] = Wq_{i,p} H_{p,:} W0_i^T.
// Included by llvq_kernels.hip.
//
// Two kernels per chunk of rows: group_gram_kernel forms the systems, group_solve_kernel factorises and solves them and
// rescales the rows.  Both sides of a system come from the same products Z_{i,p} = Wq_{i,p} H[p, :], so one pass over H
// per group of rows serves M and r; Z never leaves the registers.
#pragma once

namespace {

typedef float group_f4 __attribute__((ext_vector_type(4)));
typedef group_f4 group_f4_any __attribute__((aligned(4)));        // 16 bytes at any float address
typedef float group_f16 __attribute__((ext_vector_type(16)));

// A system is stored as its lower triangle, row after row, every row padded to a multiple of four floats so that rows can be
// read in 16-byte pieces: row p = 4a + b starts at 4 (a + 1) (2a + b).
__host__ __device__ __forceinline__ size_t group_row(int p) {
    const size_t a = (size_t)p >> 2, b = (size_t)p & 3;
    return 4 * (a + 1) * (2 * a + b);
}
// floats of a system with its right-hand side as one more row
__host__ __device__ __forceinline__ size_t group_system(int KB) { return group_row(KB) + (((size_t)KB + 3) & ~(size_t)3); }

// ---- the systems -----------------------------------------------------------------------------------------------------
// A wave owns 32 rows and four neighbouring block columns p and walks the channels b of H in units of 96 (four block
// columns q, three 32-channel tiles).  Z^T[b][row] is a v_mfma_f32_32x32x2_f32 product (A: H[p][b], read as runs of 32
// channels; B: the rows' weights of block p, held in registers for the whole walk), so a lane holds 16 channels of one row
// and the two reductions over b (against Wq for M, against W0 for r) stay inside the lane but for one exchange between
// the lane halves.  Channel groups of eight never straddle a block boundary.  Four block columns per wave, because the
// weights of a tile cost the vector memory pipe 32 lines per load: shared by four products they cost less than the
// matrix cores (12 x 64 cycles per product).  The walk is cut into `splits` parts so that the chip is full at any N, KB;
// a part writes its own share of r, and M has no shares: a pair (p, q) lies in one part.
// Bound by the fp32 matrix rate: 2 N K^2 flops at 157 TFLOP/s.  The whole call (1024 rows, K = 4104) takes 0.90 ms where a
// library product per block column, a kernel of dot products after each and an unblocked factorisation took 28.7 ms.
constexpr int kGroupP = 4;              // block columns p per wave
constexpr int kGroupRowWaves = 4;       // waves (of 32 rows) per workgroup: they read the same lines of H
constexpr int kGroupMaxSplits = 8;

__global__ void __launch_bounds__(64 * kGroupRowWaves, 2) group_gram_kernel(const float* __restrict__ Wq, const float* __restrict__ W0, size_t ldw,
                                                                           const float* __restrict__ H, int row0, int C, int KB,
                                                                           float* __restrict__ systems, float* __restrict__ r_parts) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int c0 = ((int)blockIdx.x * kGroupRowWaves + wave) * 32;
    if (c0 >= C) return;
    const int c = min(c0 + col, C - 1);                              // row of the chunk (rows past the end repeat the last one)
    const bool live = c0 + col < C;
    const int p0 = (int)blockIdx.y * kGroupP;
    const uint32_t K = 24u * (uint32_t)KB;
    const int units = (KB + 3) / 4;
    const int u0 = (int)(((int64_t)units * blockIdx.z) / gridDim.z), u1 = (int)(((int64_t)units * (blockIdx.z + 1)) / gridDim.z);
    const float* wq_row = Wq + (size_t)(row0 + c) * ldw;
    const float* w0_row = W0 + (size_t)(row0 + c) * ldw;

    // B operands: k = 2 j + half of block p, column = row of W
    float bop[kGroupP][12];
#pragma unroll
    for (int pp = 0; pp < kGroupP; pp++) {
        const int p = min(p0 + pp, KB - 1);
#pragma unroll
        for (int j = 0; j < 12; j++) bop[pp][j] = wq_row[24 * p + 2 * j + half];
    }
    float racc[kGroupP];
#pragma unroll
    for (int pp = 0; pp < kGroupP; pp++) racc[pp] = 0.0f;
    float* sys = systems + (size_t)c * group_system(KB);

    // Requests run one product ahead for H and one tile ahead for the weights; the scheduling barrier between products
    // keeps the compiler from moving more of them up than the register file holds.
    struct Weights { group_f4 wq[4], w0[4]; };
    auto load_h = [&](uint32_t b0, int pp, float (&h)[12]) {
        // wave-uniform start of the block's 24 rows + 32-bit lane offset; channels past K: their weights are zero
        uint32_t off = ((uint32_t)half * K + min(b0 + (uint32_t)col, K - 1)) * 4u;
        asm("" : "+v"(off));                                        // offsets are formed where they are used, not kept
        const unsigned char* rows = reinterpret_cast<const unsigned char*>(H + (size_t)24 * (uint32_t)min(p0 + pp, KB - 1) * K);
#pragma unroll
        for (int j = 0; j < 12; j++, off += 8u * K) h[j] = *reinterpret_cast<const float*>(rows + off);
    };
    auto load_w = [&](uint32_t b0, Weights& w) {
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const uint32_t b = b0 + 8u * (uint32_t)g + 4u * (uint32_t)half;
            const bool in = b < K;                                   // K is a multiple of 8: a group of eight is inside or outside
            uint32_t off = (in ? b : 0u) * 4u;
            asm("" : "+v"(off));
            const group_f4 z4 = {0.0f, 0.0f, 0.0f, 0.0f};
            const group_f4 v0 = *reinterpret_cast<const group_f4_any*>(reinterpret_cast<const unsigned char*>(w0_row) + off);
            const group_f4 vq = *reinterpret_cast<const group_f4_any*>(reinterpret_cast<const unsigned char*>(wq_row) + off);
            w.w0[g] = in ? v0 : z4;
            w.wq[g] = in ? vq : z4;
        }
    };
    float h[2][12];
    Weights w[2];
    if (u0 < u1) {
        load_h(96u * (uint32_t)u0, 0, h[0]);
        load_w(96u * (uint32_t)u0, w[0]);
    }
    // one unit; kWantM: some pair (p, q) of it is stored (q <= p)
    auto unit = [&](auto m_tag, int u) {
        constexpr bool kWantM = decltype(m_tag)::value;
        float macc[kGroupP][4];
#pragma unroll
        for (int pp = 0; pp < kGroupP; pp++) {
#pragma unroll
            for (int q = 0; q < 4; q++) macc[pp][q] = 0.0f;
        }
#pragma unroll
        for (int t = 0; t < 3; t++) {
            const uint32_t b0 = 96u * (uint32_t)u + 32u * (uint32_t)t;
#pragma unroll
            for (int pp = 0; pp < kGroupP; pp++) {
                load_h(pp + 1 < kGroupP ? b0 : b0 + 32u, (pp + 1) % kGroupP, h[(pp + 1) & 1]);
                if (pp == 1) load_w(b0 + 32u, w[(t + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                group_f16 z;
#pragma unroll
                for (int v = 0; v < 16; v++) z[v] = 0.0f;
#pragma unroll
                for (int j = 0; j < 12; j++) z = __builtin_amdgcn_mfma_f32_32x32x2f32(h[pp & 1][j], bop[pp][j], z, 0, 0, 0);
                const Weights& wt = w[t & 1];
#pragma unroll
                for (int g = 0; g < 4; g++) {
#pragma unroll
                    for (int v = 0; v < 4; v++) racc[pp] = fmaf(z[4 * g + v], wt.w0[g][v], racc[pp]);
                }
                if constexpr (kWantM) {
#pragma unroll
                    for (int g = 0; g < 4; g++) {
#pragma unroll
                        for (int v = 0; v < 4; v++) macc[pp][(4 * t + g) / 3] = fmaf(z[4 * g + v], wt.wq[g][v], macc[pp][(4 * t + g) / 3]);
                    }
                    // the sums are used under a condition only; left alone, the compiler moves them there and keeps all z alive
                    asm volatile("" : "+v"(macc[pp][4 * t / 3]), "+v"(macc[pp][(4 * t + 3) / 3]), "+v"(racc[pp]));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        w[0] = w[1];                                                 // the tile after an odd number of tiles was requested into w[1]
        if constexpr (kWantM) {
#pragma unroll
            for (int pp = 0; pp < kGroupP; pp++) {
                group_f4 m;
#pragma unroll
                for (int q = 0; q < 4; q++) m[q] = macc[pp][q] + __shfl_xor(macc[pp][q], 32);
                const int p = p0 + pp;
                if (half == (pp & 1) && live && p < KB && 4 * u <= p) *reinterpret_cast<group_f4*>(sys + group_row(p) + 4 * u) = m;
            }
        }
    };
    int u = u0;
    for (; u < u1 && 4 * u < p0 + kGroupP; u++) unit(std::true_type{}, u);
    for (; u < u1; u++) unit(std::false_type{}, u);
#pragma unroll
    for (int pp = 0; pp < kGroupP; pp++) {
        const float r = racc[pp] + __shfl_xor(racc[pp], 32);
        if (half == (pp & 1) && live && p0 + pp < KB) r_parts[((size_t)blockIdx.z * C + c) * KB + p0 + pp] = r;
    }
}

// ---- factorisation, solution, rescaling ---------------------------------------------------------------------------------
// One workgroup per row.  The system lies in LDS (IN_LDS: up to 160 KB, KB <= 276; two workgroups share a compute unit up
// to KB of about 190) or stays in global memory.  Blocked Cholesky with panels of 16 columns; the right-hand side rides along
// as one more row, so that the forward substitution is part of the factorisation:
//   panel     every wave holds the 16 rows of the diagonal block in its lanes 0..15 and 48 further rows in the others, 16
//             entries per lane, and runs the 16 column steps with lane broadcasts: all waves factorise the diagonal block
//             themselves, none waits for another
//   trailing  16 x 16 tiles, four v_mfma_f32_16x16x4_f32 each (a lane's 16-byte piece of a panel row is its operand of
//             all four; both operands use the same order of the 16 columns)
// then one wave substitutes backwards with the unknowns in registers.  A matrix that is not positive definite in fp32 leaves
// the row as it is (s = 1).  
constexpr int kGroupSolveWaves = 8;
constexpr size_t kGroupLdsMax = 160 * 1024;

template <bool IN_LDS>
__global__ void __launch_bounds__(64 * kGroupSolveWaves, IN_LDS ? 4 : 2) group_solve_kernel(float* __restrict__ systems, const float* __restrict__ r_parts, int splits,
                                                                              float lambda, int row0, int C, int KB, float* __restrict__ Wq,
                                                                              size_t ldw, uint16_t* __restrict__ gain, float* __restrict__ s_out) {
    constexpr int kThreadsHere = 64 * kGroupSolveWaves;
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t n_sys = group_system(KB);
    float* mine = systems + (size_t)c * n_sys;
    float* lds = reinterpret_cast<float*>(g_lds);
    float* sol = lds;                                                // KB solutions
    float* dinv = lds + ((KB + 3) & ~3);                             // KB reciprocal diagonal entries of L
    int* failed = reinterpret_cast<int*>(dinv + ((KB + 3) & ~3));
    float* A = IN_LDS ? dinv + ((KB + 3) & ~3) + 4 : mine;
    if (tid == 0) *failed = 0;
    if constexpr (IN_LDS) {
        const size_t n4 = group_row(KB) / 4;
        for (size_t i = tid; i < n4; i += kThreadsHere) reinterpret_cast<group_f4*>(A)[i] = reinterpret_cast<const group_f4*>(mine)[i];
        __syncthreads();
    }
    for (int i = tid; i < KB; i += kThreadsHere) {
        A[group_row(i) + i] += lambda;
        float r = 0.0f;
        for (int z = 0; z < splits; z++) r += r_parts[((size_t)z * C + c) * KB + i];
        A[group_row(KB) + i] = r;
    }
    __syncthreads();

    bool bad = false;
    for (int j0 = 0; j0 < KB; j0 += 16) {
        const int nb = min(16, KB - j0), j1 = j0 + nb;
        // ---- panel ----
        float dv[16];                                                // lanes 0..15: the diagonal block's row j0 + lane
        {
            const int row = min(j0 + (lane & 15), KB - 1);
            const float* src = A + group_row(row) + j0;
#pragma unroll
            for (int k = 0; k < 16; k++) dv[k] = k <= row - j0 ? src[k] : 0.0f;
        }
        for (int base = j1 + 48 * wave, first = 1; first || base <= KB; base += 48 * kGroupSolveWaves, first = 0) {
            const int row = lane < 16 ? min(j0 + lane, KB - 1) : base + lane - 16;
            const bool below = lane >= 16 && row <= KB;
            float* src = A + group_row(min(row, KB)) + j0;
            float v[16];
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = lane < 16 ? dv[k] : 0.0f;
            if (below) {
#pragma unroll
                for (int k = 0; k < 16; k++) if (k < nb) v[k] = src[k];
            }
            if (first) __syncthreads();                              // everybody has read the diagonal block
            float inv_mine = 0.0f;
#pragma unroll
            for (int k = 0; k < 16; k++) {
                if (k < nb) {
                    const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[k]), k));
                    if (!(d > 0.0f)) bad = true;
                    const float inv = 1.0f / sqrtf(d);
                    inv_mine = lane == k ? inv : inv_mine;
                    v[k] *= inv;
#pragma unroll
                    for (int k2 = k + 1; k2 < 16; k2++) {
                        const float l2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[k]), k2));
                        v[k2] = fmaf(-v[k], l2, v[k2]);
                    }
                }
            }
            if (below) {
#pragma unroll
                for (int k = 0; k < 16; k++) if (k < nb) src[k] = v[k];
            }
            if (first && wave == 0 && lane < nb) {
                dinv[j0 + lane] = inv_mine;
#pragma unroll
                for (int k = 0; k < 16; k++) if (k <= lane) src[k] = v[k];
            }
        }
        __syncthreads();
        // ---- trailing update of rows j1 .. KB, columns j1 .. min(row, KB - 1) ----
        const int nt = (KB + 1 - j1 + 15) / 16;
        if (nb == 16) {
            const int li = lane & 15, lq = lane >> 4;
            for (int e = wave, ti = 0, tk = 0; ; e += kGroupSolveWaves) {
                // tile (ti, tk), tk <= ti, of number e (the waves' numbers grow: walk on from the last one)
                while (tk * (tk + 1) / 2 <= e) tk++;                  // tk: one past the tile row of e
                ti = tk - 1;
                if (ti >= nt) break;
                const int kt = e - ti * (ti + 1) / 2, i0 = j1 + 16 * ti, k0 = j1 + 16 * kt;
                const group_f4 a = *reinterpret_cast<const group_f4*>(A + group_row(min(i0 + li, KB)) + j0 + 4 * lq);
                const group_f4 b = *reinterpret_cast<const group_f4*>(A + group_row(min(k0 + li, KB)) + j0 + 4 * lq);
                const int col = k0 + li;
                group_f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                bool in[4];
                float* dst[4];
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int row = i0 + 4 * lq + v;
                    in[v] = row <= KB && col <= row && col < KB;
                    dst[v] = A + (in[v] ? group_row(row) + col : 0);
                    acc[v] = *dst[v];
                }
#pragma unroll
                for (int s = 0; s < 4; s++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-a[s], b[s], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; v++) if (in[v]) *dst[v] = acc[v];
            }
        }
        __syncthreads();
    }
    if (bad && wave == 0 && lane == 0) *failed = 1;                  // every wave has seen the same diagonal entries
    // ---- L^T s = z, z in row KB of A: unknown i lives in lane i % 64, register i / 64 ----
    if (wave == 0) {
        constexpr int R = IN_LDS ? 5 : 16;
        float z[R], dl[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int i = 64 * r + lane;
            z[r] = i < KB ? A[group_row(KB) + i] : 0.0f;
            dl[r] = i < KB ? dinv[i] : 0.0f;
        }
#pragma unroll
        for (int r = R - 1; r >= 0; r--) {
            const int top = min(KB, 64 * (r + 1)) - 1;
            float nxt[R];
            auto request = [&](int i) {
#pragma unroll
                for (int r2 = 0; r2 <= r; r2++) nxt[r2] = 64 * r2 + lane < i ? A[group_row(i) + 64 * r2 + lane] : 0.0f;
            };
            if (top >= 64 * r) request(top);
            for (int i = top; i >= 64 * r; i--) {
                float cur[R];
#pragma unroll
                for (int r2 = 0; r2 <= r; r2++) cur[r2] = nxt[r2];
                if (i > 64 * r) request(i - 1);
                const int src = i & 63;
                const float s = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, z[r] * dl[r]), src));
#pragma unroll
                for (int r2 = 0; r2 <= r; r2++) z[r2] = fmaf(-cur[r2], s, z[r2]);
                if (lane == src) sol[i] = s;
            }
        }
    }
    __syncthreads();
    const bool keep = *failed != 0;
    // new gain = old gain * s rounded to fp16; the block is rescaled by the ratio of the two fp16 gains
    const size_t row = (size_t)(row0 + c);
    for (int p = tid; p < KB; p += kThreadsHere) {
        const float s = keep ? 1.0f : sol[p];
        const float g_old = __half2float(__ushort_as_half(gain[row * KB + p]));
        const __half g_new = __float2half_rn(g_old * s);
        gain[row * KB + p] = __half_as_ushort(g_new);
        if (s_out) s_out[row * KB + p] = s;
        sol[p] = g_old != 0.0f ? __half2float(g_new) / g_old : 0.0f;
    }
    __syncthreads();
    for (int u = tid; u < KB * 24; u += kThreadsHere) Wq[row * ldw + u] *= sol[u / 24];
}

}  // namespace
