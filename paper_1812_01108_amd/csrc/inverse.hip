// Inverse map: Cartesian coordinates -> dihedral angles, the step before the
// forward map in a pipeline (targets, initial angles).  The angle of the
// transform placing atom i is the IUPAC torsion about the bond into atom i,
// (i-2, i-1, i, i+1) ("Backbone model" section), so per residue j
//   omega_j = torsion(CA_{j-1}, C_{j-1}, N_j, CA_j),
//   phi_j   = torsion(C_{j-1}, N_j, CA_j, C_j),
//   psi_j   = torsion(N_j, CA_j, C_j, N_{j+1}),
// with the identity start frame's virtual atoms C_{-1} = origin and
// CA_{-1} = (-1, 0, 0) at a chain start; psi of a chain's last residue moves
// no atom and is written as 0.  Side chains ("Full-atom model" section): the
// transform of side frame f carries chi_{f+1}, so
//   chi_{f+1} = torsion(grandparent origin, parent origin, origin of f, D),
// the grandparent of side frame 0 being N and its parent CA, and D an atom
// that lies at y = 0, z < 0 in frame f's own coordinates (where the
// transform puts the next frame's origin, and where the residue table puts
// the atom that defines the last chi): its torsion is exactly the frame's
// angle.  The quadruples are read off the converted residue table on the
// host; chi planes a residue lacks are written as 0.
#include "a2c_internal.h"

#include <algorithm>
#include <cmath>

namespace a2c {

// Per residue type, the residue slots of the points the chi torsions run over:
// N, CA, the side frames' origins in order and the atom D of the last frame,
// so that chi_{f+1} is the torsion of points f .. f + 3; and in byte 7 the
// mask of the chis the type has (bit f) and whose atoms the table names.
void build_chi_points(const FATable &T, uint8_t (&out)[A2C_NUM_RESIDUE_TYPES][8])
{
    for (int t = 0; t < A2C_NUM_RESIDUE_TYPES; ++t) {
        const FAType &ft = T.t[t];
        uint8_t *q = out[t];
        for (int i = 0; i < 8; ++i) q[i] = 0;
        q[1] = 1;
        for (int f = 0; f < ft.n_side; ++f) {
            q[2 + f] = (uint8_t)ft.origin_slot[3 + f];
            bool named = f + 1 < ft.n_side;
            if (!named) {
                const int k = 3 + f;
                for (int i = 0; i < ft.fcount[k] && !named; ++i) {
                    const int s = ft.fbegin[k] + i;
                    const float x = ft.atom[s].x, y = ft.atom[s].y, z = ft.atom[s].z;
                    const float r = std::sqrt(x * x + y * y + z * z);
                    if (r > 0.f && std::fabs(y) <= 1e-5f * r && z < -1e-3f * r) {
                        q[3 + f] = (uint8_t)ft.atom[s].slot;
                        named = true;
                    }
                }
            }
            if (named && ft.side_chi[f]) q[7] |= (uint8_t)(1u << f);
        }
    }
}

namespace {

struct P3 {
    float x, y, z;
};

// atan2 for the torsions.  Octant reduction: t = min(|x|, |y|) / max(|x|, |y|)
// in [0, 1] (reciprocal by v_rcp_f32), atan t = t (a0 + a1 t^2 + ... + a6 t^12)
// with coefficients fitted for this library by a discrete minimax
// (Lawson-weighted least squares) in double and rounded to float32 (maximum
// error 3.3e-7 rad evaluated in float32), then pi/2 - a where |y| > |x|,
// pi - a where x < 0, and the sign of y.  NaN in gives NaN; (0, 0) gives 0.
__device__ __forceinline__ float atan2_poly(float y, float x)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
    const float t = mx > 0.f ? mn * __builtin_amdgcn_rcpf(mx) : 0.f;
    const float t2 = t * t;
    float p = 6.81179157e-03f;
    p = fmaf(p, t2, -3.36042158e-02f);
    p = fmaf(p, t2, 7.96236694e-02f);
    p = fmaf(p, t2, -1.32333413e-01f);
    p = fmaf(p, t2, 1.98078156e-01f);
    p = fmaf(p, t2, -3.33173692e-01f);
    p = fmaf(p, t2, 9.99996126e-01f);
    float a = p * t;
    a = ay > ax ? 1.57079637f - a : a;
    a = x < 0.f ? 3.14159274f - a : a;
    a = copysignf(a, y);
    return (x != x || y != y) ? x + y : a;
}

__device__ __forceinline__ P3 sub(P3 a, P3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }

__device__ __forceinline__ P3 cross(P3 a, P3 b)
{
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// Torsions over consecutive points: for p0-p1-p2-p3 with bonds b1, b2, b3 the
// IUPAC angle is atan2(|b2| b1 . (b2 x b3), (b1 x b2) . (b2 x b3)).  |b2| only
// scales the first argument, so the 1-ulp hardware square root is enough.  A
// walk along a chain of points keeps the last two bonds and their normal, so
// that the next point costs one bond and one normal.
struct TorsionWalk {
    P3 b1, b2, n1;
    __device__ __forceinline__ void start(P3 first, P3 second)
    {
        b1 = first;
        b2 = second;
        n1 = cross(b1, b2);
    }
    // the torsion about b2 onto the bond b3, which the walk then moves along
    __device__ __forceinline__ float next(P3 b3)
    {
        const P3 n2 = cross(b2, b3);
        const float len = __builtin_amdgcn_sqrtf(b2.x * b2.x + b2.y * b2.y + b2.z * b2.z);
        const float y = len * (b1.x * n2.x + b1.y * n2.y + b1.z * n2.z);
        const float x = n1.x * n2.x + n1.y * n2.y + n1.z * n2.z;
        b1 = b2;
        b2 = b3;
        n1 = n2;
        return atan2_poly(y, x);
    }
};

__device__ __forceinline__ bool head_bit(const uint32_t *__restrict__ bits, int64_t r)
{
    return (bits[r >> 5] >> (r & 31)) & 1u;
}

constexpr int kInvThreads = 256;  // residues per workgroup

// One lane per residue.  The workgroup's atoms, with one residue on either
// side (the neighbours' backbone atoms), are staged once through LDS with
// coalesced loads, every load issued before the first store; the torsions
// then read LDS, where an atom's x, y, z lie side by side (one address per
// point; the odd stride keeps the coalesced side free of conflicts).  Staged:
// residues [max(r0 - 1, 0), min(r0 + 257, R)), at most 258 residues of at most
// kAtoms atoms each; rows of 256 atoms past the range are skipped as a whole.
// Bound by the memory: 1.68 M full-atom residues, 223 MB with the atoms no
// torsion needs (they share cache lines with those that do; 235 MB counted), in
// 44.3 us, 5.0 TB/s, the rate of a device copy; 52.6 us before, with 630 VALU instructions
// per wave (549 now: shared bonds and normals) and seven useless rows of loads
// per thread.  128 residues per workgroup 47.9 us, 64 52.2, 512 46.6.
// NT: large plans write the angles with non-temporal stores (46.3 -> 44.3 us);
// small ones leave them in the caches for whatever reads them next.
template <bool FA, bool NT>
__global__ __launch_bounds__(kInvThreads) void inverse_kernel(
    const float *__restrict__ xyz, float *__restrict__ ang, const uint32_t *__restrict__ head_bits,
    const int32_t *__restrict__ res_aoff, const uint8_t *__restrict__ seq,
    const uint8_t *__restrict__ chi_points, int64_t R, int64_t A)
{
    constexpr int kAtoms = FA ? A2C_MAX_RESIDUE_ATOMS : 3;
    constexpr int kStage = (kInvThreads + 2) * kAtoms;
    constexpr int kPer = (kStage + kInvThreads - 1) / kInvThreads;
    // sized to the largest staged range of any workgroup of this plan
    extern __shared__ float stage[];
    const int tid = (int)threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kInvThreads;
    const int64_t rlo = r0 > 0 ? r0 - 1 : 0;
    const int64_t rhi = r0 + kInvThreads + 1 < R ? r0 + kInvThreads + 1 : R;
    // atom indices fit in int32: a plan holds at most INT32_MAX / 16 residues
    const int lo = FA ? res_aoff[rlo] : (int)(3 * rlo);
    const int hi = FA ? res_aoff[rhi] : (int)(3 * rhi);
    const float *__restrict__ px = xyz + lo;
    const float *__restrict__ py = xyz + A + lo;
    const float *__restrict__ pz = xyz + 2 * A + lo;
    const int n_st = __builtin_amdgcn_readfirstlane(hi - lo);
    const int64_t r = r0 + tid;
    const int64_t rc = r < R ? r : R - 1;
    const bool head = head_bit(head_bits, rc), last = head_bit(head_bits, rc + 1);
    // neighbours: the previous residue is staged unless r is a chain head,
    // the next one unless r ends its chain (then r's own atoms stand in and
    // the angle is replaced below)
    const int64_t rp = head ? rc : rc - 1, rn = last ? rc : rc + 1;
    const int a = (FA ? res_aoff[rc] : (int)(3 * rc)) - lo;
    const int pa = (FA ? res_aoff[rp] : (int)(3 * rp)) - lo;
    const int na = (FA ? res_aoff[rn] : (int)(3 * rn)) - lo;
    uint2 q{};
    if (FA) q = *reinterpret_cast<const uint2 *>(chi_points + 8 * seq[rc]);
    {
        float vx[kPer], vy[kPer], vz[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (j * kInvThreads < n_st) {
                const int k = min(tid + j * kInvThreads, n_st - 1);
                vx[j] = px[k]; vy[j] = py[k]; vz[j] = pz[k];
            }
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (j * kInvThreads < n_st) {
                const int k = 3 * min(tid + j * kInvThreads, n_st - 1);
                stage[k] = vx[j]; stage[k + 1] = vy[j]; stage[k + 2] = vz[j];
            }
    }
    __syncthreads();
    if (r >= R) return;
    auto pt = [&](int k) -> P3 { return {stage[3 * k], stage[3 * k + 1], stage[3 * k + 2]}; };
    const P3 n = pt(a), ca = pt(a + 1), c = pt(a + 2);
    const P3 pca = head ? P3{-1.f, 0.f, 0.f} : pt(pa + 1);
    const P3 pc = head ? P3{0.f, 0.f, 0.f} : pt(pa + 2);
    auto put = [&](int64_t i, float v) {
        if constexpr (NT) __builtin_nontemporal_store(v, ang + i);
        else ang[i] = v;
    };
    const P3 nca = sub(ca, n);
    TorsionWalk w;
    w.start(sub(pc, pca), sub(n, pc));
    put(2 * R + r, w.next(nca));
    put(r, w.next(sub(c, ca)));
    const float psi = w.next(sub(pt(na), c));
    put(R + r, last ? 0.f : psi);
    if (FA) {
        // chis a type lacks repeat its own atoms and are written as 0
        const uint32_t mask = q.y >> 24;
        P3 at = pt(a + (int)((q.x >> 16) & 255u));
        w.start(nca, sub(at, ca));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const P3 to = pt(a + (int)((k == 0 ? q.x >> 24 : q.y >> (8 * (k - 1))) & 255u));
            const float v = w.next(sub(to, at));
            at = to;
            put((3 + k) * R + r, (mask >> k) & 1u ? v : 0.f);
        }
    }
}

}  // namespace

// The most atoms any workgroup of the inverse map stages.
int32_t inverse_stage_atoms(const a2c_plan &p)
{
    int32_t most = 0;
    for (int64_t r0 = 0; r0 < p.R; r0 += kInvThreads) {
        const int64_t rlo = r0 > 0 ? r0 - 1 : 0;
        const int64_t rhi = r0 + kInvThreads + 1 < p.R ? r0 + kInvThreads + 1 : p.R;
        most = std::max(most, p.model == A2C_BACKBONE
                                  ? (int32_t)(3 * (rhi - rlo))
                                  : p.res_atom_off[rhi] - p.res_atom_off[rlo]);
    }
    return most;
}

}  // namespace a2c

using namespace a2c;

extern "C" a2c_status a2c_coords_to_angles(a2c_plan *p, const float *d_coords, float *d_angles,
                                           void *stream)
{
    if (!p) {
        set_error("plan is NULL");
        return A2C_ERR_INVALID_ARG;
    }
    if (p->R == 0) return A2C_OK;
    if (!d_coords || !d_angles) {
        set_error("NULL coords or angles");
        return A2C_ERR_INVALID_ARG;
    }
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != p->device) {
        set_error("current device is not the plan's device");
        return A2C_ERR_STATE;
    }
    const dim3 grid((unsigned)((p->R + kInvThreads - 1) / kInvThreads)), block(kInvThreads);
    hipStream_t s = (hipStream_t)stream;
    const size_t lds = 3 * (size_t)p->inv_stage_atoms * sizeof(float);
    const auto kernel = p->model == A2C_BACKBONE
                            ? (p->nt_grad ? inverse_kernel<false, true> : inverse_kernel<false, false>)
                            : (p->nt_grad ? inverse_kernel<true, true> : inverse_kernel<true, false>);
    hipLaunchKernelGGL(kernel, grid, block, lds, s, d_coords, d_angles, p->d_head_bits,
                       p->d_res_atom_off, p->d_seq, p->d_chi_points, p->R, p->A);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? A2C_OK : hip_fail(e, "inverse map launch");
}
