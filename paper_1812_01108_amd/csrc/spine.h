// The spine of a lane's residues (omega, phi, psi transforms), and the
// spine-only pass of the recomputing adjoints, shared by the backbone and
// full-atom kernels.
#pragma once
#include "scan.h"

namespace a2c {

namespace {

struct ResidueIn {
    float co, so, cp, sp, cs, ss;  // cos/sin of omega, phi, psi
};

// Spine angles (phi, psi, omega) of a lane's K residues, 0 past the chunk.
template <int K>
struct SpineAngles {
    float phi[K], psi[K], om[K];
};

template <int K>
__device__ __forceinline__ SpineAngles<K> load_spine_angles(const float *__restrict__ ang,
                                                            int64_t R, int64_t rs, int cnt)
{
    SpineAngles<K> a;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        a.phi[j] = j < cnt ? ang[rs + j] : 0.f;
        a.psi[j] = j < cnt ? ang[R + rs + j] : 0.f;
        a.om[j] = j < cnt ? ang[2 * R + rs + j] : 0.f;
    }
    return a;
}

// Lane-serial spine aggregate of K residues (reset at chain heads), with one
// polar step.  first_head: the lane's first residue that starts a chain (K:
// none).
template <int K>
__device__ __forceinline__ Aff fa_lane_aggregate(const SpineAngles<K> &a, int cnt, uint32_t hm,
                                                 const BBParams &P, ResidueIn (&in)[K],
                                                 int &first_head)
{
    Aff m = aff_identity();
    first_head = K;
    const float(&phi)[K] = a.phi;
    const float(&psi)[K] = a.psi;
    const float(&om)[K] = a.om;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < K; ++j)
        ok = ok && sincos_fast_ok(om[j]) && sincos_fast_ok(phi[j]) && sincos_fast_ok(psi[j]);
    if (__all(ok)) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            sincos_fast(phi[j], in[j].sp, in[j].cp);
            sincos_fast(psi[j], in[j].ss, in[j].cs);
            sincos_fast(om[j], in[j].so, in[j].co);
        }
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            sincos_accurate(phi[j], in[j].sp, in[j].cp);
            sincos_accurate(psi[j], in[j].ss, in[j].cs);
            sincos_accurate(om[j], in[j].so, in[j].co);
        }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j < cnt) {
            if ((hm >> j) & 1u) {
                m = aff_identity();
                if (first_head == K) first_head = j;
            }
            aff_apply_transform(m, P.ct[0], P.st[0], P.d[0], in[j].co, in[j].so);
            aff_apply_transform(m, P.ct[1], P.st[1], P.d[1], in[j].cp, in[j].sp);
            aff_apply_transform(m, P.ct[2], P.st[2], P.d[2], in[j].cs, in[j].ss);
        }
    }
    aff_orthonormalise(m);
    return m;
}

// Spine aggregates for the recomputing adjoints whose windows cannot wait on
// each other in both directions (a chain over more than kMaxAhead + 1 windows):
// a spine-only pass over the same windows publishes each window's aggregate
// (the product of its spine transforms from its last chain head, or its
// start, to its end) as tagged words and waits on nothing; the adjoint, last
// window first, then composes the aggregates of the windows its first chain
// spans, all complete by then (lb_carry_in).
template <int K, int LB>
__global__ __launch_bounds__(LB) void spine_aggregate_kernel(
    const float *__restrict__ ang, const uint32_t *__restrict__ head_bits,
    const int32_t *__restrict__ wstart, uint64_t *__restrict__ status, int64_t R, BBParams P)
{
    __shared__ FwdShared sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = blockIdx.x;
    const int64_t ts = wstart[t], te = wstart[t + 1];
    const int nact = (int)((te - ts + kWave * K - 1) / (kWave * K));
    const bool active = wave < nact;
    const int64_t rs = ts + (int64_t)threadIdx.x * K;
    const int cnt = (int)max((int64_t)0, min((int64_t)K, te - rs));
    const uint32_t hm = lane_head_mask<K>(head_bits, rs, te, cnt);
    uint64_t prev = 0;
    if (wave == 0) prev = lb_load(status + t * kLbWords);
    ResidueIn in[K];
    int first_head = K;
    Aff m = aff_identity();
    if (active) m = fa_lane_aggregate<K>(load_spine_angles<K>(ang, R, rs, cnt), cnt, hm, P, in,
                                         first_head);
    const uint64_t heads = __builtin_amdgcn_ballot_w64(first_head < K);
    if (active) {
        aff_wave_scan<false>(m, heads, kWave, lane);
        if (lane == kWave - 1) {
            aff_store(sh.tot[wave], m);
            sh.tot_flag[wave] = heads != 0ull ? 1 : 0;
        }
    }
    __syncthreads();
    if (wave != 0) return;
    Aff tw = aff_identity();
    bool tf = false;
    if (lane < nact) {
        tw = aff_load(sh.tot[lane]);
        tf = sh.tot_flag[lane] != 0;
    }
    const uint64_t th = __builtin_amdgcn_ballot_w64(tf);
    aff_wave_scan<true>(tw, th, nact, lane);
    if (lane == nact - 1) aff_store(sh.pre[0], tw);
    wave_lds_sync();
    const uint32_t tag = (uint32_t)(__builtin_amdgcn_readfirstlane((uint32_t)(prev >> 32))) + 1u;
    if (lane < kLbWords) lb_store(status + t * kLbWords + lane, tag, sh.pre[0][lane]);
}

// The spine pass over the windows of schedule S (at most C = 64 W K residues
// each), with more residues per lane where C allows (8 or 4 per lane, fewer
// waves): the per-residue walk is cheap and the scan is shared by more
// residues.
inline void launch_spine_pass(const float *ang, const uint32_t *head_bits, const Sched &S,
                              int64_t R, const BBParams &bb, hipStream_t s)
{
    const int64_t C = (int64_t)kWave * S.K * S.W;
    const dim3 grid(S.n_win);
    if (C % (kWave * 8) == 0)
        hipLaunchKernelGGL((spine_aggregate_kernel<8, 512>), grid, dim3(C / 8), 0, s, ang,
                           head_bits, S.d_wstart, S.d_status_fwd, R, bb);
    else if (C % (kWave * 4) == 0)
        hipLaunchKernelGGL((spine_aggregate_kernel<4, 1024>), grid, dim3(C / 4), 0, s, ang,
                           head_bits, S.d_wstart, S.d_status_fwd, R, bb);
    else if (C % (kWave * 2) == 0)
        hipLaunchKernelGGL((spine_aggregate_kernel<2, 1024>), grid, dim3(C / 2), 0, s, ang,
                           head_bits, S.d_wstart, S.d_status_fwd, R, bb);
    else
        hipLaunchKernelGGL((spine_aggregate_kernel<1, 1024>), grid, dim3(C), 0, s, ang, head_bits,
                           S.d_wstart, S.d_status_fwd, R, bb);
}

}  // namespace

}  // namespace a2c
