// Kernels of the run-time specialized evaluator (compiled with hipRTC).
//
// The skeleton is the one of the packed evaluators (kernels_packed.hpp), one
// lane per energy sample, but every table walk is replaced by the diagram's own
// straight-line code: the generated part that precedes this file defines, in
// namespace amijit, the sizes NE (energies), NI (loops), NG (lines), NX
// (external slots), L (distinct leaves), D (distinct denominators), G (groups),
// the leaf kinds kBose[L], and the functions
//   lines            K_j = sum_l alpha_jl k_l (+ external q), per component
//   line_trig        sin K_j, cos K_j from those of the k_l and q by angle addition
//   leaf_args        x_l = sum_i c_li E_i                        (Sec. 2.2)
//   taylor_leaves    f_l -> its Taylor coefficient T_j (poles of higher order, Eq. (5))
//   group_sums_c     the group sums at complex leaves (complex energies)
//   group_sums       FT_g = sum_{t in g} s_t prod_{l in t} f_l     (Sec. 2.3)
//   den_args         D_k = e_k . E + a_k . w                        (Sec. 2.2)
//   group_products   R_g = prod_{k in g} 1/D_k
//   den_cotangents   U_k = sum_{g contains k} u_g
//   den_scatter      dL/dE_i += e_ki Re(U_k rho_k), dL/dw_x += a_kx U_k rho_k
//   leaf_cotangents  dL/df_l = sum_{t contains l} dL/dFT_g(t) s_t prod_{l' != l} f_l'
//   leaf_scatter     dL/dE_i += sum_l c_li v_l
//   line_scatter     dL/dk_l += sum_j alpha_jl dL/dK_j
// With every index a constant, all per-sample state lives in registers: no
// LDS beyond the block reduction, no table reads, no scalar bit tests.
// Partial sums are written per wave (no LDS, no barrier), column by column
// (a.nrows = blocks x waves per block rows), in the column order of the packed
// evaluators, so the same reduction kernels finish them.
#pragma once

#include "jit_tiles.hpp"

// AMI_JIT_BLOCK lanes per block (the host launches with the same value);
// AMI_JIT_KERNELS selects the forward (1), the adjoint (2), the Monte-Carlo
// integrator (4), the forward at complex energies (8), the two passes of the
// two-pass forward (16, 32), the frequency and leaf passes of the adjoint of
// large solutions (64, 128), the adjoint at complex energies (256), the two
// passes of the forward at complex energies (512, 1024), the frequency and
// leaf passes of the adjoint at complex energies (2048, 4096), or a sum of
// them, or, alone, the block adjoint (8192; for several rows, where that is apart,
// 65536; at complex energies 16384) or the block forward (32768)

// Small calls (a.fin_cols > 0): the last block to arrive adds the partial sums of
// all blocks, in the order of the reduction kernel that large calls launch (64
// rows at a time, then those totals in row order: the same bits).  NW waves per
// block, each with its columns, 16 loads in flight.  last: a word of the kernel's
// LDS.  The second launch this saves bounds such calls on
// the host: order 2, 300 samples 14.4 -> 11.3 us, the adjoint of 10^4 21.5 -> 18.5.
// Every wave's rows are in L2 before the barrier, and released to the device before
// the block is counted (ROCm 7.2's compiler counts without waiting for the
// write-back, so the wait is explicit); the block that completes the count resets it
// for the next launch on the stream.
typedef __attribute__((address_space(3))) unsigned *LdsWord;
typedef __attribute__((address_space(1))) double *GlobalDouble;

// Where the total of column c goes (null: nowhere).  By selections alone: ROCm 7.2's
// compiler loses fin_t from the branches of the nested conditional.
__device__ __forceinline__ GlobalDouble finish_target(const ami::KArgs &a, int c) {
    const uint64_t scalar[3] = {reinterpret_cast<uint64_t>(a.fin_beta), reinterpret_cast<uint64_t>(a.fin_mu),
                                reinterpret_cast<uint64_t>(a.fin_t)};
    uint64_t p = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) p |= scalar[j] & (0 - static_cast<uint64_t>(c == j));
    const uint64_t w = reinterpret_cast<uint64_t>(a.fin_w), sum = reinterpret_cast<uint64_t>(a.fin_sum);
    const uint64_t in_w = 0 - static_cast<uint64_t>(c >= ami::kAdjScalars && w != 0);
    const uint64_t in_sum = 0 - static_cast<uint64_t>(c >= a.fin_grad);
    p |= (w + 8 * static_cast<int64_t>(c - ami::kAdjScalars)) & in_w;
    p = (p & ~in_sum) | ((sum + 8 * static_cast<int64_t>(c - a.fin_grad)) & in_sum);
    return reinterpret_cast<GlobalDouble>(p);
}

template <int NW>
__device__ __forceinline__ void finish_sums(const ami::KArgs &a, LdsWord last) {
    if (a.fin_cols == 0) return;
    const unsigned blocks = gridDim.x * gridDim.y;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned before = 0;
        if (blocks > 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __builtin_amdgcn_s_waitcnt(0);
            before = __hip_atomic_fetch_add(a.fin_ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        }
        const bool whole = before == blocks - 1;
        *last = whole;
        if (whole && blocks > 1) __hip_atomic_store(a.fin_ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(*last)) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double *cols = a.gpartial ? a.gpartial : a.partial;
    const int rows = static_cast<int>(a.nrows), chunks = (rows + 63) >> 6;
    const int todo = a.fin_cols > wave ? (a.fin_cols - wave + NW - 1) / NW * chunks : 0;
    int lc = wave, lk = 0, c = wave, k = 0;     // column and chunk of the next load and of the next addend
    double total = 0.0;
    for (int p = 0; p < todo; p += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int row = 64 * lk + lane;
            v[u] = p + u < todo && row < rows ? cols[lc * rows + row] : 0.0;
            if (++lk == chunks) {
                lk = 0;
                lc += NW;
            }
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (p + u >= todo) break;
            total += ami::wave_sum(0.0 + v[u]);
            if (++k < chunks) continue;
            const GlobalDouble dst = finish_target(a, c);
            if (lane == 0 && dst) *dst = total;
            total = 0.0;
            k = 0;
            c += NW;
        }
    }
}

// The one-pass and block forwards run blocks (tile, part of the rows): every part
// forms the tile's leaves and group sums again, and takes an even number of
// rows; the host launches no empty part.
#define AMI_JIT_ROW_PART(f0, f1)                                                    \
    const int per = ((a.n_f + static_cast<int>(gridDim.y) - 1) / static_cast<int>(gridDim.y) + 1) & ~1; \
    const int f0 = static_cast<int>(blockIdx.y) * per;                                      \
    const int f1 = f0 + per < a.n_f ? f0 + per : a.n_f;

#if AMI_JIT_KERNELS & 1
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_fwd(ami::KArgs a) {
    __shared__ unsigned word;
    if (a.n_f == 1) {
        amijit::fwd_tile<AMI_JIT_HUB, true>(a, blockIdx.x, 0, 1);
    } else {
        AMI_JIT_ROW_PART(f0, f1)
        amijit::fwd_tile<AMI_JIT_HUB, false>(a, blockIdx.x, f0, f1);
    }
    finish_sums<AMI_JIT_BLOCK / 64>(a, (LdsWord)&word);
}
#endif

#if AMI_JIT_ADJ_WAVES > 0
#define AMI_JIT_ADJ_ATTR __attribute__((amdgpu_waves_per_eu(AMI_JIT_ADJ_WAVES)))
#else
#define AMI_JIT_ADJ_ATTR
#endif

#if AMI_JIT_KERNELS & 2

extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) AMI_JIT_ADJ_ATTR void ami_jit_adj(ami::KArgs a) {
    __shared__ double park[amijit::kParkCols > 0 ? amijit::kParkCols * AMI_JIT_BLOCK : 1];
    const int64_t s = static_cast<int64_t>(blockIdx.x) * AMI_JIT_BLOCK + threadIdx.x;
    double in[amijit::NIN];
    amijit::load_inputs<AMI_JIT_HUB>(a, s < a.n_e ? s : a.n_e - 1, in);
    if (a.n_f == 1) amijit::adj_tile<AMI_JIT_HUB, true>(a, blockIdx.x, park, in);
    else amijit::adj_tile<AMI_JIT_HUB, false>(a, blockIdx.x, park, in);
    finish_sums<AMI_JIT_BLOCK / 64>(a, (LdsWord)park);
}
#endif

#if AMI_JIT_KERNELS & 4
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_mc(ami::KArgs a) {
    amijit::mc_block<AMI_JIT_HUB>(a);
}
#endif

#if AMI_JIT_KERNELS & 8
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_cfwd(ami::KArgs a) {
    __shared__ unsigned word;
    AMI_JIT_ROW_PART(f0, f1)
    amijit::cfwd_tile(a, blockIdx.x, f0, f1);
    finish_sums<AMI_JIT_BLOCK / 64>(a, (LdsWord)&word);
}
#endif

#if AMI_JIT_KERNELS & 256
#if AMI_JIT_CADJ_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_CADJ_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_cadj(ami::KArgs a) {
    __shared__ double park[amijit::kParkS ? 2 * amijit::L * AMI_JIT_BLOCK : 1];
    amijit::cadj_tile(a, blockIdx.x, park);
    finish_sums<AMI_JIT_BLOCK / 64>(a, (LdsWord)park);
}
#endif

#if AMI_JIT_KERNELS & 512
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_csums(ami::KArgs a) {
    amijit::csums_tile(a, blockIdx.x);
}
#endif

#if AMI_JIT_KERNELS & 1024
// the grid of ami_jit_freq: (tile, frequency) blocks dealt over the XCDs
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_cfreq(ami::KArgs a) {
    const int64_t b = blockIdx.x, local = b >> 3;
    const int f = static_cast<int>(local % a.n_f);
    const int64_t tile = 8 * (local / a.n_f) + (b & 7);
    if (tile * AMI_JIT_BLOCK >= a.n_chunk) return;
    amijit::cfreq_tile(a, tile, f);
}
#endif

// occupancy floors of the large adjoint's passes (waves per SIMD; 0: none)
#ifndef AMI_JIT_ADJF_WAVES
#define AMI_JIT_ADJF_WAVES 2
#endif
#ifndef AMI_JIT_ADJL_WAVES
#define AMI_JIT_ADJL_WAVES 2
#endif
#if AMI_JIT_KERNELS & 64
#if AMI_JIT_ADJF_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_ADJF_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_adjf(ami::KArgs a) {
    amijit::adjf_tile(a, blockIdx.x);
}
#endif

#if AMI_JIT_KERNELS & 128
#if AMI_JIT_ADJL_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_ADJL_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_adjl(ami::KArgs a) {
    __shared__ double park[amijit::kParkCols > 0 ? amijit::kParkCols * AMI_JIT_BLOCK : 1];
    amijit::adjl_tile<AMI_JIT_HUB>(a, blockIdx.x, park);
}
#endif

#ifndef AMI_JIT_SUMS_WAVES
#define AMI_JIT_SUMS_WAVES 0
#endif
#if AMI_JIT_KERNELS & 16
#if AMI_JIT_SUMS_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_SUMS_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_sums(ami::KArgs a) {
    amijit::sums_tile<AMI_JIT_HUB>(a, blockIdx.x);
}
#endif

#if AMI_JIT_KERNELS & 32
// One block per (tile, frequency row) in a one-dimensional grid: block b runs
// on the XCD b mod 8 (the dispatcher deals blocks round-robin over the eight
// XCDs), and the n_f blocks of a tile are consecutive on that XCD, so a
// tile's stored group sums come from HBM once and from the XCD's L2 for the
// other frequency rows.  Blocks past the last tile (the tile count rounded up
// to a multiple of 8) return at once.
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_freq(ami::KArgs a) {
    const int64_t b = blockIdx.x, local = b >> 3;
    const int f = static_cast<int>(local % a.n_f);
    const int64_t tile = 8 * (local / a.n_f) + (b & 7);
    if (tile * AMI_JIT_BLOCK >= a.n_chunk) return;
    amijit::freq_tile(a, tile, f);
}
#endif

#if AMI_JIT_KERNELS & 2048
#if AMI_JIT_ADJF_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_ADJF_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_cadjf(ami::KArgs a) {
    amijit::cadjf_tile(a, blockIdx.x);
}
#endif

#if AMI_JIT_KERNELS & 4096
#if AMI_JIT_CADJL_WAVES > 0
__attribute__((amdgpu_waves_per_eu(AMI_JIT_CADJL_WAVES)))
#endif
extern "C" __global__ __launch_bounds__(AMI_JIT_BLOCK) void ami_jit_cadjl(ami::KArgs a) {
    amijit::cadjl_tile(a, blockIdx.x);
}
#endif

#if AMI_JIT_KERNELS & (8192 | 65536)
// 64 samples per block of NW waves; two waves per SIMD (one alone issues an
// FP64 instruction every eight cycles instead of four): two blocks of four
// waves, or one of eight, on a CU
extern "C" __global__ __launch_bounds__(64 * amijit::NW) __attribute__((amdgpu_waves_per_eu(2))) void ami_jit_badj(ami::KArgs a) {
    __shared__ double sm[64 * amijit::kBlockCols];
    const int64_t tile = (a.s0 >> 6) + blockIdx.x;      // s0: the launch's first sample
    constexpr amijit::Rows rows = !amijit::kRowsApart ? amijit::ANY_ROWS
                                  : AMI_JIT_KERNELS & 65536 ? amijit::SEVERAL_ROWS : amijit::ONE_ROW;
    amijit::badj_tile<AMI_JIT_HUB, rows>(a, tile, sm);
    finish_sums<amijit::NW>(a, (LdsWord)sm);
}
#endif

#if AMI_JIT_KERNELS & 16384
extern "C" __global__ __launch_bounds__(64 * amijit::NW) __attribute__((amdgpu_waves_per_eu(2))) void ami_jit_bcadj(ami::KArgs a) {
    __shared__ double sm[64 * amijit::kBlockCols];
    const int64_t tile = (a.s0 >> 6) + blockIdx.x;      // s0: the launch's first sample
    if constexpr (amijit::kRowsApart) {
        if (a.n_f == 1) amijit::bcadj_tile<amijit::ONE_ROW>(a, tile, sm);
        else amijit::bcadj_tile<amijit::SEVERAL_ROWS>(a, tile, sm);
    } else {
        amijit::bcadj_tile<amijit::ANY_ROWS>(a, tile, sm);
    }
    finish_sums<amijit::NW>(a, (LdsWord)sm);
}
#endif

#if AMI_JIT_KERNELS & 32768
extern "C" __global__ __launch_bounds__(64 * amijit::NW) __attribute__((amdgpu_waves_per_eu(2))) void ami_jit_bfwd(ami::KArgs a) {
    __shared__ double sm[64 * amijit::kBlockCols];
    const int64_t tile = (a.s0 >> 6) + blockIdx.x;      // s0: the launch's first sample
    AMI_JIT_ROW_PART(f0, f1)
    amijit::bfwd_tile<AMI_JIT_HUB>(a, tile, f0, f1, sm);
    finish_sums<amijit::NW>(a, (LdsWord)sm);
}
#endif
