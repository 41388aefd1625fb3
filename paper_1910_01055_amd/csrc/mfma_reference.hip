// Measurement aid for the whole-network int8 kernels (Sec. 3.1 actor inference): the inner loop of the
// pipelined wide kernel and nothing else, so that a benchmark can report what the matrix cores sustain in that
// loop shape on the operands it is given -- the ceiling of k_mlp_wide's passes on this machine.
//
// One workgroup of 8 wavefronts per CU owns 64 activation rows of K = 1024 in LDS.  64 of K are, for a wavefront, sixteen
// 16x16x64 MFMAs (four halves of its two 32-feature tiles x four 16-row tiles) on 4 KiB of weight operands read L2 -> registers in
// operand order, two such steps in flight, and on four activation operands read from LDS one step ahead, each behind its last use:
// 32 KiB of weights and 128 MFMAs per CU, the ratio at which a CU's vector memory path (64 B/clock) and its matrix cores (8192 op/clock)
// are both saturated.  No epilogue, no barrier, no output but the accumulators of
// workgroup 0, which a test checks.  The matrix cores' clock under load depends on the operands (a loop on
// zeros runs about a third faster than one on random bytes), which is why the operands are arguments.
#include <atomic>

#include "kernels.hpp"

namespace aq {
namespace {

constexpr int RPF = 2;      // steps of 64 of K whose weights are in flight per wavefront
constexpr int RLD = 1040;   // LDS row stride in bytes (K + 16: rows 16 bytes apart in the banks)
// LDS asked for: more than half of a CU's 160 KiB, so that every CU holds one workgroup, as under k_mlp_wide
constexpr int RLDS = 96 * 1024;
static_assert(64 * RLD <= RLDS, "the activation rows fit");

typedef int rv4i __attribute__((ext_vector_type(4)));

// weights: 16 feature tiles x 64 k-steps (of 32) x 1 KiB; wavefront w owns tiles 2w and 2w + 1 and walks their 64 k-steps
// round and round, two at a time.  acts: 64 rows x 1024 bytes, walked 32 k-steps round and round.
template <bool STREAM>
__global__ __launch_bounds__(512) void k_mfma_reference(const char* __restrict__ weights, const int8_t* __restrict__ acts,
                                                        int ksteps, int32_t* __restrict__ acc_out) {
    extern __shared__ __align__(16) int8_t x[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < 64 * 64; i += 512) {  // 16-byte pieces
        const int m = i >> 6, k16 = i & 63;
        *(rv4i*)(x + m * RLD + 16 * k16) = *(const rv4i*)(acts + m * 1024 + 16 * k16);
    }
    __syncthreads();
    const int b16 = lane & 15, g = lane >> 4;  // batch row and k-group (operands) / feature quad (results)
    const int8_t* xrow = x + b16 * RLD + g * 16;
    const char* wp = weights + (size_t)(2 * wave) * 64 * 1024 + (g >> 1) * 1024 + (b16 + 32 * (g & 1)) * 16;
    auto wload = [&](int h, int step) { return *(const rv4i*)(wp + (h >> 1) * 64 * 1024 + step * 2048 + 256 * (h & 1)); };
    rv4i wreg[RPF][4], xf[4], c[4][4];
#pragma unroll
    for (int p = 0; p < RPF; ++p)
#pragma unroll
        for (int h = 0; h < 4; ++h) wreg[p][h] = wload(h, p);
#pragma unroll
    for (int r = 0; r < 4; ++r) xf[r] = *(const rv4i*)(xrow + r * 16 * RLD);
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[h][r] = rv4i{0, 0, 0, 0};
    const int steps = ksteps >> 1;
    for (int k = 0; k < steps; k += RPF) {
#pragma unroll
        for (int p = 0; p < RPF; ++p) {
            const int8_t* const nx = xrow + ((k + p + 1) & 15) * 64;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
#pragma unroll
                for (int h = 0; h < 4; ++h) c[h][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wreg[p][h], xf[r], c[h][r], 0, 0, 0);
                xf[r] = *(const rv4i*)(nx + r * 16 * RLD);
            }
            if (STREAM) {
#pragma unroll
                for (int h = 0; h < 4; ++h) wreg[p][h] = wload(h, (k + p + RPF) & 31);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // workgroup 0's accumulators, [wave][feature tile][row tile][register][lane] of 32 x 32 tiles: register q of lane l is feature
    // 8 (q / 4) + 4 (l / 32) + q % 4, row l % 32; the other workgroups computed the same values
    if (blockIdx.x == 0) {
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = 4 * (2 * (h & 1) + (g >> 1)) + i, l = 32 * (g & 1) + 16 * (r & 1) + b16;
                    acc_out[(((wave * 2 + (h >> 1)) * 2 + (r >> 1)) * 16 + q) * 64 + l] = c[h][r][i];
                }
    }
}

}  // namespace

aq_status launch_mfma_reference(const void* d_weights, const void* d_acts, int ksteps, bool stream_weights, int workgroups,
                                int32_t* d_acc, hipStream_t st) {
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)k_mfma_reference<true>, hipFuncAttributeMaxDynamicSharedMemorySize, RLDS)) ||
            hip_failed(hipFuncSetAttribute((const void*)k_mfma_reference<false>, hipFuncAttributeMaxDynamicSharedMemorySize, RLDS)))
            return AQ_EHIP;
        attr_set = true;
    }
    if (stream_weights)
        hipLaunchKernelGGL((k_mfma_reference<true>), dim3((unsigned)workgroups), dim3(512), RLDS, st, (const char*)d_weights,
                           (const int8_t*)d_acts, ksteps, d_acc);
    else
        hipLaunchKernelGGL((k_mfma_reference<false>), dim3((unsigned)workgroups), dim3(512), RLDS, st, (const char*)d_weights,
                           (const int8_t*)d_acts, ksteps, d_acc);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq
