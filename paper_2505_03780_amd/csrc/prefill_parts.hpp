// Prefill whose keys are cut into parts over workgroups: the records that the parts leave, and their merge.
#pragma once
#include "kernel_params.hpp"

namespace attn {
namespace {

// Record of a part of a 32-row block: 32 * HD unnormalised outputs, then (reference, sum) of every row.
template <int HD>
constexpr int kRecordFloats = 32 * (HD + 2);

constexpr int kMergeThreads = 256;
template <int HD>
constexpr int kMergeBlocks = 32 * HD / 4 / kMergeThreads;  // workgroups of a merge kernel per 32-row block

// Four merged outputs: element i of `outputs` in each of `n_parts` records from `rec` on, of the row whose (reference, sum) is pair
// `row`.  Up to eight records at a time, so that a thread takes one or a few round trips.  A part in which the row sees no
// key has sum 0.
template <int HD>
__device__ __forceinline__ float4 merge_records(const float *rec, int n_parts, int i, int row)
{
    float M = -INFINITY, L = 0.f;
    float4 acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int kBlock = 8;
    for (int b = 0; b < n_parts; b += kBlock) {
        float2 ml[kBlock];
        float4 o[kBlock];
#pragma unroll
        for (int j = 0; j < kBlock; ++j) {  // (past the last part: that part again, cleared below)
            const float *r = rec + (int64_t)(b + j < n_parts ? b + j : n_parts - 1) * kRecordFloats<HD>;
            ml[j] = *(const float2 *)(r + 32 * HD + 2 * row);
            o[j] = *(const float4 *)(r + 4 * i);
        }
        // Cleared, not weighted with zero: the last part may hold an infinity.  (Real records are weighted whatever they hold, as the
        // unsplit kernels weight every key: zero times infinity is NaN in both.)
#pragma unroll
        for (int j = 1; j < kBlock; ++j)
            if (b + j >= n_parts) {
                ml[j] = float2{-INFINITY, 0.f};
                o[j] = float4{0.f, 0.f, 0.f, 0.f};
            }
        float m_new = M;
#pragma unroll
        for (int j = 0; j < kBlock; ++j) m_new = ml[j].y > 0.f ? fmaxf(m_new, ml[j].x) : m_new;
        const float keep = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - m_new);
        M = m_new;
        L *= keep;
        acc.x *= keep, acc.y *= keep, acc.z *= keep, acc.w *= keep;
#pragma unroll
        for (int j = 0; j < kBlock; ++j) {
            const float f = ml[j].y > 0.f ? __builtin_amdgcn_exp2f(ml[j].x - M) : 0.f;
            L += ml[j].y * f;
            acc.x += o[j].x * f, acc.y += o[j].y * f, acc.z += o[j].z * f, acc.w += o[j].w * f;
        }
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;  // (a query without a visible key gets zeros)
    return float4{acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
}

}  // namespace
}  // namespace attn
