// Full-atom model ("Full-atom model" section of the paper) on gfx950.
//
// The spine N -> CA -> C of every residue is the backbone chain (same three
// transforms, same segmented affine scan); each residue then hangs its side
// chain off the CA frame through a fixed rotation R' and a chain of up to
// four side frames M_f = M_parent R(chi_f, theta_f, d_f), and places every
// atom as r = M_frame r°.  One lane owns K consecutive residues:
//   forward : lane aggregate of the 3K spine transforms -> window prefix scan
//             on a quarter of the waves -> the lane re-walks its residues from
//             its prefix frame, building spine and side frames and emitting
//             atoms;
//   adjoint : the same walk yields frame origins and axes; per residue the
//             side-frame subtree wrenches give the chi gradients (side frames
//             form a chain, so a suffix over frames), the residue's N, CA
//             (+ side chain) and C (+ O) group wrenches feed a block reverse
//             scan over residues, and u . (S_m - o x S_g) gives phi, psi,
//             omega -- Eq. FAMBackward summed over subtrees in O(N).
// In the adjoint the atom positions either come from the forward's output
// (axes from bond vectors) or are recomputed from the angles.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "scan.h"
#include "spine.h"

namespace a2c {

// ------------------------------------------------------------------ host

namespace {

struct V3 {
    double x, y, z;
};
V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
V3 add(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
V3 scale(V3 a, double s) { return {a.x * s, a.y * s, a.z * s}; }
V3 cross(V3 a, V3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }
double norm(V3 a) { return std::sqrt(a.x * a.x + a.y * a.y + a.z * a.z); }

// Natural extension reference frame placement (Parsons et al., J. Comput.
// Chem. 26, 2005): the point d with |d - c| = bond, angle(b, c, d) = angle
// and torsion(a, b, c, d) = torsion.
V3 nerf(V3 a, V3 b, V3 c, double bond, double angle, double torsion)
{
    V3 bc = sub(c, b);
    bc = scale(bc, 1.0 / norm(bc));
    V3 n = cross(sub(b, a), bc);
    n = scale(n, 1.0 / norm(n));
    const V3 m = cross(n, bc);
    const double dx = -bond * std::cos(angle);
    const double dy = bond * std::sin(angle) * std::cos(torsion);
    const double dz = bond * std::sin(angle) * std::sin(torsion);
    return add(c, add(scale(bc, dx), add(scale(m, dy), scale(n, dz))));
}

a2c_status bad_table(int t, const std::string &msg)
{
    set_error("residue table, type " + std::to_string(t) + ": " + msg);
    return A2C_ERR_INVALID_ARG;
}

}  // namespace

// Validate a residue table and convert it to float32 constants (r° of every
// atom in its frame, side-frame transforms).  spine_d: bond lengths of the
// spine frames N, CA, C (their predecessor distances).  Host only.
a2c_status convert_residue_table(const a2c_residue_table *table, const double spine_d[3],
                                 FATable &T)
{
    const double pi = 3.14159265358979323846, d2r = pi / 180.0;
    std::memset(&T, 0, sizeof(T));
    for (int t = 0; t < A2C_NUM_RESIDUE_TYPES; ++t) {
        const a2c_residue_def &rd = table->residues[t];
        FAType &ft = T.t[t];
        if (rd.n_atoms < 3 || rd.n_atoms > A2C_MAX_RESIDUE_ATOMS)
            return bad_table(t, "n_atoms must be 3..14");
        if (rd.n_side_frames < 0 || rd.n_side_frames > A2C_MAX_SIDE_FRAMES)
            return bad_table(t, "n_side_frames must be 0..4");
        ft.n_atoms = rd.n_atoms;
        ft.n_side = rd.n_side_frames;
        double fd[7] = {spine_d[0], spine_d[1], spine_d[2], 0, 0, 0, 0};
        for (int f = 0; f < rd.n_side_frames; ++f) {
            const a2c_side_frame &sf = rd.frames[f];
            if (sf.parent != (f == 0 ? 1 : 3 + f - 1))
                return bad_table(t, "side frame " + std::to_string(f) +
                                        " must hang off CA (frame 0) or the previous side frame");
            if (sf.chi != 0 && sf.chi != f + 1)
                return bad_table(t, "side frame " + std::to_string(f) + " must use chi" +
                                        std::to_string(f + 1) + " or a fixed torsion");
            if (f > 0 && sf.pre_rotation_deg != 0.0)
                return bad_table(t, "only side frame 0 may have a pre-rotation");
            if (!(std::isfinite(sf.bond) && sf.bond > 0) ||
                !(std::isfinite(sf.bond_angle_deg) && sf.bond_angle_deg > 0 &&
                  sf.bond_angle_deg < 180))
                return bad_table(t, "side frame geometry out of range");
            ft.side_chi[f] = sf.chi ? 1 : 0;
            unit_pair(pi - sf.bond_angle_deg * d2r, ft.ct[f], ft.st[f]);
            ft.d[f] = (float)sf.bond;
            ft.inv_d[f] = (float)(1.0 / sf.bond);
            fd[3 + f] = sf.bond;
            if (f == 0) unit_pair(sf.pre_rotation_deg * d2r, ft.pre_c, ft.pre_s);
        }
        const int nframes = 3 + rd.n_side_frames;
        for (int k = 0; k < 7; ++k) ft.origin_slot[k] = -1;
        V3 local[A2C_MAX_RESIDUE_ATOMS];
        for (int a = 0; a < rd.n_atoms; ++a) {
            const a2c_atom_def &ad = rd.atoms[a];
            if (ad.frame < 0 || ad.frame >= nframes) return bad_table(t, "atom frame out of range");
            if (a < 3 && !(ad.frame == a && ad.kind == A2C_ATOM_ORIGIN))
                return bad_table(t, "atoms 0, 1, 2 must be N, CA, C at the spine frame origins");
            if (ad.kind == A2C_ATOM_ORIGIN) {
                if (ft.origin_slot[ad.frame] >= 0) return bad_table(t, "two atoms at one frame origin");
                ft.origin_slot[ad.frame] = a;
                local[a] = {0, 0, 0};
            } else if (ad.kind == A2C_ATOM_AZIMUTH) {
                const double ang = ad.angle_deg * d2r, z = ad.torsion_deg * d2r;
                local[a] = {-ad.bond * std::cos(ang), ad.bond * std::sin(ang) * std::sin(z),
                            -ad.bond * std::sin(ang) * std::cos(z)};
            } else if (ad.kind == A2C_ATOM_ZMATRIX) {
                V3 r[3];
                for (int q = 0; q < 3; ++q) {
                    const int i = ad.ref[q];
                    if (i == -1) r[q] = {-fd[ad.frame], 0, 0};
                    else if (i >= 0 && i < a && rd.atoms[i].frame == ad.frame) r[q] = local[i];
                    else return bad_table(t, "z-matrix reference must be an earlier atom of the "
                                             "same frame or -1");
                }
                local[a] = nerf(r[0], r[1], r[2], ad.bond, ad.angle_deg * d2r, ad.torsion_deg * d2r);
            } else {
                return bad_table(t, "unknown atom kind");
            }
            if (!std::isfinite(local[a].x) || !std::isfinite(local[a].y) || !std::isfinite(local[a].z))
                return bad_table(t, "atom position not finite");
        }
        for (int k = 0; k < nframes; ++k)
            if (ft.origin_slot[k] < 0) return bad_table(t, "every frame needs an atom at its origin");
        // each frame's list starts with its origin atom (the kernels place it
        // at the frame's translation without a product)
        int n = 0;
        for (int k = 0; k < 7; ++k) {
            ft.fbegin[k] = n;
            for (int pass = 0; pass < 2; ++pass)
                for (int a = 0; a < rd.n_atoms; ++a)
                    if (rd.atoms[a].frame == k && (a == ft.origin_slot[k]) == (pass == 0)) {
                        ft.atom[n].slot = a;
                        ft.atom[n].x = (float)local[a].x;
                        ft.atom[n].y = (float)local[a].y;
                        ft.atom[n].z = (float)local[a].z;
                        ++n;
                    }
            ft.fcount[k] = n - ft.fbegin[k];
        }
    }
    return A2C_OK;
}

// The kernels' form of the converted table: per type the side frames'
// constants, the slots of their origin atoms, and the other ("extra") atoms
// in the order the walk meets them (N, CA, the side frames in order, C).
static void build_device_table(const FATable &T, FADevTable &D)
{
    static const int walk[7] = {0, 1, 3, 4, 5, 6, 2};  // frame at each position of the walk
    std::memset(&D, 0, sizeof(D));
    for (int t = 0; t < A2C_NUM_RESIDUE_TYPES; ++t) {
        const FAType &ft = T.t[t];
        FADevType &d = D.t[t];
        d.pre_c = ft.pre_c;
        d.pre_s = ft.pre_s;
        d.counts = (uint32_t)ft.n_side << 28;
        float *inv = &d.inv_d.x;
        for (int f = 0; f < ft.n_side; ++f) {
            d.fr[f] = float4{ft.ct[f], ft.st[f], ft.d[f], ft.side_chi[f] ? 1.f : 0.f};
            inv[f] = ft.inv_d[f];
            d.origin |= (uint32_t)ft.origin_slot[3 + f] << (8 * f);
        }
        int n = 0;
        for (int i = 0; i < 7; ++i) {
            const int k = walk[i];
            // a frame's list starts with its origin atom
            for (int a = 1; a < ft.fcount[k]; ++a) d.ex[n++] = ft.atom[ft.fbegin[k] + a];
            if (ft.fcount[k] > 1) d.counts |= (uint32_t)(ft.fcount[k] - 1) << (4 * i);
        }
    }
}

a2c_status build_fullatom_tables(a2c_plan *p, const a2c_residue_table *table)
{
    FATable &T = p->fa_host;
    const double spine_d[3] = {p->bb.d[0], p->bb.d[1], p->bb.d[2]};
    const a2c_status st = convert_residue_table(table, spine_d, T);
    if (st != A2C_OK) return st;
    build_device_table(T, p->fa_dev);
    // atom offsets
    p->res_atom_off.assign((size_t)p->R + 1, 0);
    for (int64_t r = 0; r < p->R; ++r)
        p->res_atom_off[r + 1] = p->res_atom_off[r] + T.t[p->seq[r]].n_atoms;
    p->A = p->res_atom_off[p->R];
    p->chain_atom_off.resize(p->n_chains + 1);
    for (int32_t c = 0; c <= p->n_chains; ++c)
        p->chain_atom_off[c] = p->res_atom_off[p->res_off[c]];
    return A2C_OK;
}

}  // namespace a2c

extern "C" a2c_status a2c_residue_table_info(const a2c_residue_table *table, int32_t *n_atoms,
                                            float *local_xyz)
{
    using namespace a2c;
    if (!table) {
        set_error("table is NULL");
        return A2C_ERR_INVALID_ARG;
    }
    // default backbone bond lengths for the spine predecessors
    const double spine_d[3] = {1.329, 1.458, 1.525};
    FATable T;
    const a2c_status st = convert_residue_table(table, spine_d, T);
    if (st != A2C_OK) return st;
    for (int t = 0; t < A2C_NUM_RESIDUE_TYPES; ++t) {
        const FAType &ft = T.t[t];
        if (n_atoms) n_atoms[t] = ft.n_atoms;
        if (local_xyz)
            for (int q = 0; q < ft.n_atoms; ++q) {
                float *o = local_xyz + 3 * (A2C_MAX_RESIDUE_ATOMS * t + ft.atom[q].slot);
                o[0] = ft.atom[q].x; o[1] = ft.atom[q].y; o[2] = ft.atom[q].z;
            }
    }
    return A2C_OK;
}

namespace a2c {

// ---------------------------------------------------------------- device

namespace {

// The constant table into LDS in 16-byte pieces: loads first (issued ahead of
// the window's inputs, so that the copy waits for nothing else), then the
// stores, which a barrier of the caller closes.  Rounds past the end are
// skipped as a whole; inside the last one indices are clamped (those threads
// rewrite the last piece with the value it already gets).
constexpr int kTabPieces = sizeof(FADevTable) / 16;
constexpr int kTabRounds = (kTabPieces + kWave - 1) / kWave;

typedef int Piece __attribute__((ext_vector_type(4)));

struct TableCopy {
    Piece v[kTabRounds];
};

__device__ __forceinline__ TableCopy table_load(const FADevTable *__restrict__ g)
{
    static_assert(sizeof(FADevTable) % 16 == 0, "the table copies in 16-byte pieces");
    TableCopy c;
    const Piece *src = reinterpret_cast<const Piece *>(g);
#pragma unroll
    for (int u = 0; u < kTabRounds; ++u)
        if (u * (int)blockDim.x < kTabPieces)
            c.v[u] = src[min((int)(threadIdx.x + u * blockDim.x), kTabPieces - 1)];
    return c;
}

__device__ __forceinline__ void table_store(FADevTable &tab, const TableCopy &c)
{
    Piece *dst = reinterpret_cast<Piece *>(&tab);
#pragma unroll
    for (int u = 0; u < kTabRounds; ++u)
        if (u * (int)blockDim.x < kTabPieces)
            dst[min((int)(threadIdx.x + u * blockDim.x), kTabPieces - 1)] = c.v[u];
}

// M <- M Rx(b): the fixed pre-rotation of side frame 0
__device__ __forceinline__ void aff_rot_x(Aff &m, float c, float s)
{
    const float a0 = c * m.r01 + s * m.r02, a1 = c * m.r11 + s * m.r12, a2 = c * m.r21 + s * m.r22;
    const float b0 = c * m.r02 - s * m.r01, b1 = c * m.r12 - s * m.r11, b2 = c * m.r22 - s * m.r21;
    m.r01 = a0; m.r11 = a1; m.r21 = a2;
    m.r02 = b0; m.r12 = b1; m.r22 = b2;
}

// A wave's atom run [A0, A0 + n): atom e (relative to A0).  In the per-wave
// LDS stage (LDS = true) its x, y, z lie side by side (one 12-byte access per
// atom; the copies take four atoms, three 16-byte accesses, per lane); for schedules whose stage does not fit the LDS the run is global
// memory itself, in planes ns apart.
struct F3 {
    float x, y, z;
};

template <bool LDS>
struct Atoms {
    float *st;
    int64_t ns;
    __device__ __forceinline__ F3 get(int e) const
    {
        if constexpr (LDS) return *reinterpret_cast<const F3 *>(st + 3 * e);
        else return F3{st[e], st[ns + e], st[2 * ns + e]};
    }
    __device__ __forceinline__ void put(int e, float x, float y, float z) const
    {
        if constexpr (LDS) *reinterpret_cast<F3 *>(st + 3 * e) = F3{x, y, z};
        else { st[e] = x; st[ns + e] = y; st[2 * ns + e] = z; }
    }
};

// Coalesced copies between a global run (3 planes, plane stride A) and the
// wave's stage, in pieces of kPiece atoms of a lane: kPiece consecutive floats
// of each plane, 3 kPiece in the stage.  kRows rows of 64 pieces at a time: a
// batch's loads are all issued before its first store.  Rows past the run's
// whole pieces are skipped (n is wave-uniform), inside the last one indices
// are clamped; the atoms after the last whole piece go one per lane.  A run
// starts at any atom, so its planes are aligned to a float only; the stage is
// aligned to a piece.  A quarter of the accesses of one atom per lane, and no
// bank conflicts at 12 floats a lane: 4096 chains of 50..2000 residues, forward
// 123.3 to 119.5 us, fused step 207 to 204 us; pieces of two atoms 121.7 and
// 206 us; rows for 512 instead of 768 atoms at once 119.4 and 208 us.
constexpr int kPiece = 4;
constexpr int kRows = 3;
typedef float PieceLds __attribute__((ext_vector_type(kPiece)));
typedef float PieceMem __attribute__((ext_vector_type(kPiece), aligned(4)));

struct RunRows {
    PieceLds v0[kRows], v1[kRows], v2[kRows];
};

// Rows from piece `base` on of np.
__device__ __forceinline__ RunRows rows_load(const float *__restrict__ src, int64_t A, int64_t A0,
                                             int base, int np)
{
    const int lane = threadIdx.x & 63;
    const float *s0 = src + A0, *s1 = src + A + A0, *s2 = src + 2 * A + A0;
    RunRows r;
#pragma unroll
    for (int u = 0; u < kRows; ++u)
        if (base + u * kWave < np) {
            const int e = kPiece * min(base + lane + u * kWave, np - 1);
            r.v0[u] = *reinterpret_cast<const PieceMem *>(s0 + e);
            r.v1[u] = *reinterpret_cast<const PieceMem *>(s1 + e);
            r.v2[u] = *reinterpret_cast<const PieceMem *>(s2 + e);
        }
    return r;
}

__device__ __forceinline__ void rows_to_lds(const RunRows &r, float *st, int base, int np)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < kRows; ++u)
        if (base + u * kWave < np) {
            PieceLds *q = reinterpret_cast<PieceLds *>(st) + 3 * min(base + lane + u * kWave, np - 1);
            float a[3 * kPiece];
#pragma unroll
            for (int i = 0; i < kPiece; ++i) {
                a[3 * i] = r.v0[u][i];
                a[3 * i + 1] = r.v1[u][i];
                a[3 * i + 2] = r.v2[u][i];
            }
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                PieceLds w;
#pragma unroll
                for (int i = 0; i < kPiece; ++i) w[i] = a[h * kPiece + i];
                q[h] = w;
            }
        }
}

// A run of n atoms: its first rows and the atoms after its last whole piece,
// and then (run_to_lds) the rest.
struct RunStart {
    RunRows rows;
    F3 tail;
};

__device__ __forceinline__ RunStart run_start(const float *__restrict__ src, int64_t A, int64_t A0,
                                              int n)
{
    RunStart r;
    r.rows = rows_load(src, A, A0, 0, n / kPiece);
    const int e = n / kPiece * kPiece + (int)(threadIdx.x & 63);
    if (e < n) r.tail = F3{src[A0 + e], src[A + A0 + e], src[2 * A + A0 + e]};
    return r;
}

__device__ __forceinline__ void run_to_lds(const RunStart &r, float *st,
                                           const float *__restrict__ src, int64_t A, int64_t A0,
                                           int n)
{
    const int np = n / kPiece;
    rows_to_lds(r.rows, st, 0, np);
    const int e = np * kPiece + (int)(threadIdx.x & 63);
    if (e < n) *reinterpret_cast<F3 *>(st + 3 * e) = r.tail;
    for (int base = kRows * kWave; base < np; base += kRows * kWave)
        rows_to_lds(rows_load(src, A, A0, base, np), st, base, np);
}

__device__ __forceinline__ void lds_to_run(const float *st, float *__restrict__ dst, int64_t A,
                                           int64_t A0, int n)
{
    const int lane = threadIdx.x & 63;
    float *o0 = dst + A0, *o1 = dst + A + A0, *o2 = dst + 2 * A + A0;
    const int np = n / kPiece;
    for (int base = 0; base < np; base += kRows * kWave) {
        PieceLds w[kRows][3];
#pragma unroll
        for (int u = 0; u < kRows; ++u)
            if (base + u * kWave < np) {
                const PieceLds *q =
                    reinterpret_cast<const PieceLds *>(st) + 3 * min(base + lane + u * kWave, np - 1);
#pragma unroll
                for (int h = 0; h < 3; ++h) w[u][h] = q[h];
            }
#pragma unroll
        for (int u = 0; u < kRows; ++u)
            if (base + u * kWave < np) {
                const int e = kPiece * min(base + lane + u * kWave, np - 1);
                PieceLds x, y, z;
#pragma unroll
                for (int i = 0; i < kPiece; ++i) {
                    x[i] = w[u][(3 * i) / kPiece][(3 * i) % kPiece];
                    y[i] = w[u][(3 * i + 1) / kPiece][(3 * i + 1) % kPiece];
                    z[i] = w[u][(3 * i + 2) / kPiece][(3 * i + 2) % kPiece];
                }
                *reinterpret_cast<PieceMem *>(o0 + e) = x;
                *reinterpret_cast<PieceMem *>(o1 + e) = y;
                *reinterpret_cast<PieceMem *>(o2 + e) = z;
            }
    }
    const int e = np * kPiece + lane;
    if (e < n) {
        o0[e] = st[3 * e];
        o1[e] = st[3 * e + 1];
        o2[e] = st[3 * e + 2];
    }
}

struct ChunkRange {
    int64_t cs, ce;
    int nact;
};

// Per-lane bookkeeping of one window.
template <int K>
struct LaneRun {
    int64_t rs, rbase, A0;
    int cnt, nres, natoms;
    bool active;
    uint32_t hm, lm;
};

template <int K>
__device__ __forceinline__ LaneRun<K> lane_run(const ChunkRange &k,
                                               const uint32_t *__restrict__ head_bits,
                                               const int32_t *__restrict__ res_aoff)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    LaneRun<K> L;
    L.rbase = k.cs + (int64_t)wave * kWave * K;
    L.active = wave < k.nact;
    L.nres = L.active ? (int)min((int64_t)kWave * K, k.ce - L.rbase) : 0;
    L.rs = k.cs + (int64_t)threadIdx.x * K;
    L.cnt = (int)max((int64_t)0, min((int64_t)K, k.ce - L.rs));
    L.hm = lane_head_mask<K>(head_bits, L.rs, k.ce, L.cnt);
    L.lm = lane_head_mask<K>(head_bits, L.rs + 1, k.ce + 1, L.cnt);
    // (waves past the window's end: no atoms, and no branch around the loads)
    const int64_t rb = min(L.rbase, k.ce);
    L.A0 = __builtin_amdgcn_readfirstlane(res_aoff[rb]);
    L.natoms = __builtin_amdgcn_readfirstlane(res_aoff[rb + L.nres]) - (int)L.A0;
    return L;
}

// Per-residue inputs of a lane, read right after the window's bookkeeping so
// that their latency overlaps the spine scan instead of stalling the walk:
// residue type, first atom and (ANG) the seven angles (chi planes are read
// for every residue; a residue without chi f ignores plane f).
template <int K, bool ANG>
struct LaneRes {
    int type[K];
    int aoff[K];
    float phi[ANG ? K : 1], psi[ANG ? K : 1], om[ANG ? K : 1];
    float chi[ANG ? K : 1][4];
};

template <int K, bool ANG>
__device__ __forceinline__ LaneRes<K, ANG> load_lane_res(const LaneRun<K> &L,
                                                         const uint8_t *__restrict__ seq,
                                                         const int32_t *__restrict__ res_aoff,
                                                         const float *__restrict__ ang, int64_t R)
{
    LaneRes<K, ANG> lr;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const bool v = j < L.cnt;
        const int64_t r = v ? L.rs + j : 0;
        lr.type[j] = v ? seq[r] : 0;
        lr.aoff[j] = v ? res_aoff[r] : 0;
        if (ANG) {
            lr.phi[j] = v ? ang[r] : 0.f;
            lr.psi[j] = v ? ang[R + r] : 0.f;
            lr.om[j] = v ? ang[2 * R + r] : 0.f;
#pragma unroll
            for (int f = 0; f < 4; ++f) lr.chi[j][f] = v ? ang[(3 + f) * R + r] : 0.f;
        }
    }
    return lr;
}

// ------------------------------------------------------- entering frames
// The spine scan of a window.  Every lane forms the product of its K residues'
// spine transforms (its unit) and leaves it in LDS; the window's first waves
// then take four units per lane (256 per wave), scan them, hand frames across
// the window's edges and leave the frame entering every unit in its place.
// The wave scan costs some 370 VALU instructions however many residues a lane
// holds, so it runs on a quarter of the waves, and a window of four waves
// needs no scan across waves; everything per residue stays spread over all
// lanes.
//
// 256 units take one block of 3 x 4 x 65 16-byte pieces: piece part of unit
// 4 l + j sits at (4 part + j) 65 + l, so that neither the spine lanes (l
// consecutive) nor the unit lanes (j fastest) meet bank conflicts.
constexpr int kGroup = 4;                        // units per spine lane
constexpr int kSpineUnits = kWave * kGroup;      // units per spine wave
constexpr int kFrameBlock = 3 * kGroup * 65 * 4; // floats
using SpineShared = FwdSharedOf<kMaxWaves / kGroup>;

inline size_t frame_bytes(int waves)
{
    return (size_t)((waves + kGroup - 1) / kGroup) * kFrameBlock * sizeof(float);
}

__device__ __forceinline__ void frame_put(float *frames, int block, int i, const Aff &m)
{
    float4 *q = reinterpret_cast<float4 *>(frames + block * kFrameBlock);
    q[i] = float4{m.r00, m.r10, m.r20, m.r01};
    q[i + kGroup * 65] = float4{m.r11, m.r21, m.r02, m.r12};
    q[i + 2 * kGroup * 65] = float4{m.r22, m.t0, m.t1, m.t2};
}

__device__ __forceinline__ Aff frame_get(const float *frames, int block, int i)
{
    const float4 *q = reinterpret_cast<const float4 *>(frames + block * kFrameBlock);
    const float4 u = q[i], v = q[i + kGroup * 65], w = q[i + 2 * kGroup * 65];
    Aff m;
    m.r00 = u.x; m.r10 = u.y; m.r20 = u.z; m.r01 = u.w;
    m.r11 = v.x; m.r21 = v.y; m.r02 = v.z; m.r12 = v.w;
    m.r22 = w.x; m.t0 = w.y; m.t1 = w.z; m.t2 = w.w;
    return m;
}

// The frame entering each lane's unit.  unit: the product of the lane's spine
// transforms since its last chain head (the identity for an empty lane);
// head: a chain starts in the lane; n_units: lanes holding residues.  Every
// thread of the block calls it; flags (kMaxWaves words) and frames
// (frame_bytes) are LDS.  LINK as in block_prefix_windows.  The frames are free again after the caller's next
// barrier.
template <bool LINK>
__device__ __forceinline__ Aff entering_frame(const Aff &unit, bool head, int n_units,
                                              float *frames, uint64_t (&flags)[kMaxWaves],
                                              SpineShared &sh, float (&carry_sh)[12],
                                              uint64_t *__restrict__ status, int64_t t,
                                              int64_t first, uint64_t prev, bool published)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int block = wave / kGroup;
    const int at = (lane & 3) * 65 + (wave % kGroup) * (kWave / kGroup) + (lane >> 2);
    const uint64_t heads_u = __builtin_amdgcn_ballot_w64(head);
    if (wave * kWave < n_units) {
        frame_put(frames, block, at, unit);
        if (lane == 0) flags[wave] = heads_u;
    }
    __syncthreads();
    const int ns = (n_units + kSpineUnits - 1) / kSpineUnits;  // spine waves
    const bool spine = wave < ns;
    Aff m = aff_identity();
    uint32_t hm = 0;  // chain heads in the lane's four units
    if (spine) {
        // the other waves of the workgroup wait for this part
        __builtin_amdgcn_s_setprio(3);
        const int w = kGroup * wave + (lane >> 4);  // the wave holding the lane's units
        const int u0 = wave * kSpineUnits + kGroup * lane;
        if (u0 < n_units) {
            hm = (uint32_t)(flags[w] >> (4 * (lane & 15))) & 15u;
            const bool any = __builtin_amdgcn_ballot_w64(hm != 0u) != 0ull;
            m = frame_get(frames, wave, lane);
#pragma unroll
            for (int j = 1; j < kGroup; ++j) {
                // units past the last one hold nothing (their waves may not
                // have run): they leave the aggregate alone
                if (u0 + j < n_units) {
                    const Aff b = frame_get(frames, wave, j * 65 + lane);
                    const Aff c = aff_compose(m, b);
                    if (any) m = aff_select((hm >> j) & 1u, b, c);
                    else m = c;
                }
            }
        }
        // the fixed rotations repeat every residue, so their float32 rounding
        // drifts the scale of long products coherently; one polar step per
        // lane aggregate removes that drift
        aff_orthonormalise(m);
    }
    const uint64_t heads = __builtin_amdgcn_ballot_w64(hm != 0u);
    Aff cur = block_prefix_windows<LINK>(m, heads, ns, spine, sh, carry_sh, status, t, first, prev,
                                         published);
    if (spine) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const Aff b = frame_get(frames, wave, j * 65 + lane);
            frame_put(frames, wave, j * 65 + lane, cur);
            if (j + 1 < kGroup) {
                const Aff c = aff_compose(cur, b);
                const bool h = (hm >> j) & 1u;
                if (__builtin_amdgcn_ballot_w64(h) != 0ull) cur = aff_select(h, b, c);
                else cur = c;
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    return frame_get(frames, block, at);
}

// cos/sin of a lane's spine angles.
template <int K>
__device__ __forceinline__ void lane_sincos(const LaneRes<K, true> &lr, ResidueIn (&in)[K])
{
    bool ok = true;
#pragma unroll
    for (int j = 0; j < K; ++j)
        ok = ok && sincos_fast_ok(lr.om[j]) && sincos_fast_ok(lr.phi[j]) && sincos_fast_ok(lr.psi[j]);
    if (__all(ok)) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            sincos_fast(lr.om[j], in[j].so, in[j].co);
            sincos_fast(lr.phi[j], in[j].sp, in[j].cp);
            sincos_fast(lr.psi[j], in[j].ss, in[j].cs);
        }
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            sincos_accurate(lr.om[j], in[j].so, in[j].co);
            sincos_accurate(lr.phi[j], in[j].sp, in[j].cp);
            sincos_accurate(lr.psi[j], in[j].ss, in[j].cs);
        }
    }
}

// The lane's unit: the product of its residues' spine transforms since its
// last chain head (the identity for an empty lane).
template <int K>
__device__ __forceinline__ Aff spine_unit(const ResidueIn (&in)[K], const LaneRun<K> &L,
                                          const BBParams &P)
{
    Aff m = aff_identity();
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j < L.cnt) {
            const bool h = (L.hm >> j) & 1u;
            if (j == 0 || h) m = aff_first_transform(P.ct[0], P.st[0], P.d[0], in[j].co, in[j].so);
            else aff_apply_transform(m, P.ct[0], P.st[0], P.d[0], in[j].co, in[j].so);
            aff_apply_transform(m, P.ct[1], P.st[1], P.d[1], in[j].cp, in[j].sp);
            aff_apply_transform(m, P.ct[2], P.st[2], P.d[2], in[j].cs, in[j].ss);
        }
    }
    return m;
}

// ------------------------------------------------------------- the walk
// A residue type's list of extra atoms (not at a frame's origin) as the walk
// consumes it: N, CA, the side frames in order, C.
struct TypeAt {
    const FADevType *ft;
    uint32_t counts, origin;
    int n_side;
    const FAAtom *ex;  // next extra atom
};

__device__ __forceinline__ TypeAt type_at(const FADevTable &tab, int type)
{
    TypeAt t;
    t.ft = &tab.t[type];
    t.counts = t.ft->counts;
    t.origin = t.ft->origin;
    t.n_side = (int)(t.counts >> 28);
    t.ex = t.ft->ex;
    return t;
}

// Extra atoms in position i of the walk (0 N, 1 CA, 2 + f side frame f, 6 C).
__device__ __forceinline__ int extra_count(const TypeAt &t, int i)
{
    return (int)((t.counts >> (4 * i)) & 15u);
}

// Every extra atom of one frame placed by F: op(e, x, y, z).
template <typename Op>
__device__ __forceinline__ void walk_extras(TypeAt &t, int n, const Aff &F, int aloc, Op &&op)
{
    for (int i = 0; i < n; ++i) {
        const FAAtom at = t.ex[i];
        float x, y, z;
        aff_point(F, at.x, at.y, at.z, x, y, z);
        op(aloc + at.slot, x, y, z);
    }
    t.ex += n;
}

// Side frame f from the one before it (chi: its torsion; a frame without one
// takes 0 whatever the plane holds).
__device__ __forceinline__ void side_step(Aff &sf, const FADevType &ft, int f, float chi)
{
    const float4 g = ft.fr[f];  // ct, st, d, 1 where the frame has a chi
    const float a = g.w != 0.f ? chi : 0.f;
    float c, s;
    if (__all(sincos_fast_ok(a))) sincos_fast(a, s, c);
    else sincos_accurate(a, s, c);
    aff_apply_transform(sf, g.x, g.y, g.z, c, s);
}

// All atoms of one residue from the frame before it (cur, advanced to the
// residue's C frame): spine transforms omega, phi, psi, and the side chain
// branching off the CA frame.  Each frame's first atom is its origin: the
// frame's translation, no product.  Of the side frames' extra atoms nearly all
// belong to a residue's last frame, so those run in one loop after the
// frames, as long as the largest of the wave's lanes has atoms, whichever
// frame is its last (8 rounds for random sequences, where a loop per frame to
// the table's largest count took 15 for the 2.5 a residue has on average).
template <bool LDS>
__device__ __forceinline__ void fa_emit_residue(const FADevTable &tab, int type, Aff &cur,
                                                const ResidueIn &in, const float (&chi)[4],
                                                const BBParams &P, const Atoms<LDS> &out, int aloc)
{
    TypeAt t = type_at(tab, type);
    auto put = [&](int e, float x, float y, float z) { out.put(e, x, y, z); };
    aff_apply_transform(cur, P.ct[0], P.st[0], P.d[0], in.co, in.so);
    put(aloc, cur.t0, cur.t1, cur.t2);
    walk_extras(t, extra_count(t, 0), cur, aloc, put);
    aff_apply_transform(cur, P.ct[1], P.st[1], P.d[1], in.cp, in.sp);
    put(aloc + 1, cur.t0, cur.t1, cur.t2);
    walk_extras(t, extra_count(t, 1), cur, aloc, put);
    if (t.n_side > 0) {
        Aff sf = cur;
        aff_rot_x(sf, t.ft->pre_c, t.ft->pre_s);
        int last = 0;  // extra atoms of the last side frame
#pragma unroll
        for (int f = 0; f < A2C_MAX_SIDE_FRAMES; ++f) {
            if (f < t.n_side) {
                side_step(sf, *t.ft, f, chi[f]);
                put(aloc + (int)((t.origin >> (8 * f)) & 255u), sf.t0, sf.t1, sf.t2);
                last = extra_count(t, 2 + f);
                if (f + 1 < t.n_side && last > 0) walk_extras(t, last, sf, aloc, put);
            }
        }
        walk_extras(t, last, sf, aloc, put);
    }
    aff_apply_transform(cur, P.ct[2], P.st[2], P.d[2], in.cs, in.ss);
    put(aloc + 2, cur.t0, cur.t1, cur.t2);
    walk_extras(t, extra_count(t, 6), cur, aloc, put);
}

// Forward over windows of the packed batch (window t: residues
// [wstart[t], wstart[t + 1]), at most C = 64 W K): the spine scan leaves the
// frame entering every residue in LDS (frames handed across window edges by
// window look-back); then every lane walks its residues, building the spine
// and side frames and writing each atom into the wave's LDS stage, which is
// copied out with coalesced stores (STG; otherwise, for schedules whose stage
// does not fit the LDS, straight to global memory).  The stage takes the
// frames' place once every lane holds its own.
// Bound by VALU issue and waits in turn: 1082 instructions per wave of 64
// residues at K = 1 (60 us of issue for 2.16 M residues in some 110 us, where
// the 301 MB it moves would take 59), 16 waves per CU (the LDS stages).  The spine scan
// on a quarter of the waves, one loop over the last frame's atoms and 12-byte
// stage accesses took 2000 chains of 50..2000 residues from 59.7 to 51.5 us at
// (1, 4), 500 chains of 151 from 11.9 to 10.7 us at (1, 6).
// LINK = false: windows of whole chains, none of which needs another's frame
// (no words read or written: forward and adjoint of 64 chains of 300 17.05 to
// 16.4 us); true: fixed windows.
template <int K, int LB, bool LINK, bool STG>
__global__ __launch_bounds__(LB) void fa_forward_flat_kernel(
    const float *__restrict__ ang, float *__restrict__ xyz, const uint32_t *__restrict__ head_bits,
    const int32_t *__restrict__ wstart, int32_t cap, const int32_t *__restrict__ res_aoff,
    const uint8_t *__restrict__ seq, const FADevTable *__restrict__ gtab,
    const int32_t *__restrict__ look_first,
    uint64_t *__restrict__ status, int64_t R, int64_t A, BBParams P, int stage_atoms)
{
    extern __shared__ __align__(16) float stage_mem[];
    __shared__ __align__(16) FADevTable tab;
    __shared__ SpineShared sh;
    __shared__ float carry_sh[12];
    __shared__ uint64_t unit_flags[kMaxWaves];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = blockIdx.x;
    ChunkRange k;
    window_range<LINK>(wstart, cap, R, t, k.cs, k.ce);
    k.nact = (int)((k.ce - k.cs + kWave * K - 1) / (kWave * K));
    const TableCopy tc = table_load(gtab);
    uint64_t prev = 0;
    int64_t first = t;
    if (LINK && wave == 0) {
        prev = lb_load(status + t * kLbWords);
        first = look_first[t];
    }
    const LaneRun<K> L = lane_run<K>(k, head_bits, res_aoff);
    const LaneRes<K, true> lr = load_lane_res<K, true>(L, seq, res_aoff, ang, R);
    table_store(tab, tc);
    ResidueIn in[K];
    Aff unit = aff_identity();
    if (L.active) {
        lane_sincos<K>(lr, in);
        unit = spine_unit<K>(in, L, P);
    }
    const int n_units = (int)((k.ce - k.cs + K - 1) / K);
    Aff cur = entering_frame<LINK>(unit, L.hm != 0u, n_units, stage_mem, unit_flags, sh, carry_sh,
                                   status, t, first, prev, false);
    if (STG) __syncthreads();  // the stage takes the frames' place
    if (!L.active) return;
    float *st = stage_mem + (size_t)wave * 3 * stage_atoms;
    const Atoms<STG> out = STG ? Atoms<STG>{st, 0} : Atoms<STG>{xyz + L.A0, A};
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j < L.cnt) {
            if ((L.hm >> j) & 1u) cur = aff_identity();
            fa_emit_residue<STG>(tab, lr.type[j], cur, in[j], lr.chi[j], P, out,
                                 lr.aoff[j] - (int)L.A0);
        }
    }
    if (STG) {
        wave_lds_sync();
        lds_to_run(st, xyz, A, L.A0, L.natoms);
    }
}

// Torque bookkeeping of one rotation axis (a spine node or a side frame):
// the derivative of sum g.r over the atoms a rotation about the axis u
// through o moves is u . (m - o x g) = u . m - v . g with v = u x o, summed
// over the wrenches (g, m) of the atom groups it moves.  It is linear in the
// wrench, so the wrenches of the residue's groups an axis moves are summed
// and folded into c once the residue is walked, and the wrench S of
// everything after the residue enters later as c + u . S.m - v . S.g.
// 7 floats per axis.
struct NodeGrad {
    float c, u0, u1, u2, v0, v1, v2;
};

// What a residue keeps across the block scan: its three spine nodes and W,
// the residue's whole wrench (for earlier residues of the lane).
struct SpineGrad {
    NodeGrad n, ca, cc;
    Wrench W;
};

__device__ __forceinline__ NodeGrad node_at(float ox, float oy, float oz, float ux, float uy,
                                            float uz)
{
    NodeGrad g;
    g.c = 0.f;
    g.u0 = ux; g.u1 = uy; g.u2 = uz;
    // explicit FMAs: no contraction left to the compiler here
    g.v0 = fmaf(uy, oz, -(uz * oy));
    g.v1 = fmaf(uz, ox, -(ux * oz));
    g.v2 = fmaf(ux, oy, -(uy * ox));
    return g;
}

// the axis of frame F: its x axis through its origin
__device__ __forceinline__ NodeGrad node_of_frame(const Aff &F)
{
    return node_at(F.t0, F.t1, F.t2, F.r00, F.r10, F.r20);
}

__device__ __forceinline__ float node_torque(const NodeGrad &g, const Wrench &S)
{
    float t = fmaf(g.u0, S.m0, g.c);
    t = fmaf(g.u1, S.m1, t);
    t = fmaf(g.u2, S.m2, t);
    t = fmaf(-g.v0, S.g0, t);
    t = fmaf(-g.v1, S.g1, t);
    return fmaf(-g.v2, S.g2, t);
}

__device__ __forceinline__ void node_fold(NodeGrad &g, const Wrench &w) { g.c = node_torque(g, w); }

// An angle gradient: a non-temporal store when nt (large plans).
__device__ __forceinline__ void grad_store(float *p, float v, bool nt)
{
    if (nt) out_store<true>(p, v);
    else out_store<false>(p, v);
}

__device__ __forceinline__ void fa_store_grads(float *__restrict__ gang, int64_t R, int64_t r,
                                               const SpineGrad &sp, const Wrench &S_after,
                                               Wrench &S_out, bool nt)
{
    grad_store(&gang[R + r], node_torque(sp.cc, S_after), nt);
    grad_store(&gang[r], node_torque(sp.ca, S_after), nt);
    grad_store(&gang[2 * R + r], node_torque(sp.n, S_after), nt);
    Wrench S = S_after;
    wrench_add(S, sp.W);
    S_out = S;
}

// The adjoint's per-atom step where the frames are recomputed: the wrench of
// the atom at (x, y, z) for its staged upstream gradient, or (GM = kGradMse)
// for the loss gradient 2 (r - t) of its staged target, which the position
// then replaces (the stage ends up holding the coordinates); the loss takes
// |r - t|^2.
template <int GM, bool STG>
struct AtomForce {
    Atoms<STG> g, out;
    bool write;
    float loss;
    __device__ __forceinline__ void operator()(Wrench &w, int e, float x, float y, float z)
    {
        const F3 s = g.get(e);
        if constexpr (GM == kGradMse) {
            const float dx = x - s.x, dy = y - s.y, dz = z - s.z;
            loss += dx * dx + dy * dy + dz * dz;
            wrench_add_point(w, x, y, z, 2.f * dx, 2.f * dy, 2.f * dz);
            if (write) out.put(e, x, y, z);
        } else {
            wrench_add_point(w, x, y, z, s.x, s.y, s.z);
        }
    }
};

// Backward over windows of the packed batch: the side chains' subtree sums
// give the chi gradients, the spine groups feed a reverse scan over residues
// (window look-ahead for the wrench of later windows), and
// u . (S_m - o x S_g) gives phi, psi, omega.
// RECOMPUTE: frames from the angles.  Window t publishes its spine aggregate,
// takes the frames of the earlier windows its first chain spans, then
// publishes its wrench and adds those of the later windows its last chain
// runs into; a wrench waits only on aggregates and those on nothing, so the
// windows go in order and a launch progresses as long as the device holds the
// at most kMaxAhead + 1 workgroups a chain spans at once.  For longer chains
// (spined) a spine pass has published the aggregates and the windows go last
// to first (LEADS: as many workgroups more, dispatched first, publish them
// instead of the pass).  Otherwise positions and axes from the forward's coordinates, last
// window first (rev; in order where the windows hold whole chains).
// GM = kGradMse (with RECOMPUTE): g points at a target t and the upstream
// gradient is 2 (r - t), formed from the recomputed positions (the fused
// training step); xyz_out (may be NULL) receives the positions, loss_out
// (may be NULL) the batch's sum of |r - t|^2 (lb_loss_commit).
// Bound as the forward, with 1699 instructions per wave at (1, 8) (94 us of
// issue for 2.16 M residues recomputing, 366 MB, in some 150 us).  Without the
// spine pass before it (6.5 us on 512 chains of 50..2000 residues), with the
// spine scan on a quarter of the waves, the extra atoms in one loop and the
// first rows of the gradients loaded ahead of the scan, the recomputing form
// went from 87.1 to 67.0 us on 2000 such chains at (1, 4) and from 31.4 to
// 20.8 us on 512, the fused step from 116 to 90.1 and 38.3 to 30.1 us; from
// coordinates 12.7 to 9.1 us on 64 chains of 300 at (1, 6).
// nt: the angle gradients go out with non-temporal stores (large plans).
// STG: atoms go through the per-wave LDS stage; otherwise global memory is
// addressed directly (schedules whose stage does not fit the LDS).
// LINK: as in the forward.
template <int K, bool RECOMPUTE, int LB, int GM, bool LINK, bool STG, bool LEADS = false>
__global__ __launch_bounds__(LB) void fa_backward_flat_kernel(
    const float *__restrict__ ang, const float *__restrict__ xyz, const float *__restrict__ g,
    float *__restrict__ gang, float *__restrict__ xyz_out, float *__restrict__ loss_out,
    const uint32_t *__restrict__ head_bits, const int32_t *__restrict__ wstart, int32_t cap,
    const int32_t *__restrict__ res_aoff, const uint8_t *__restrict__ seq,
    const FADevTable *__restrict__ gtab, uint64_t *__restrict__ status_fwd,
    const int32_t *__restrict__ look_fwd,
    const int32_t *__restrict__ look_last, uint64_t *__restrict__ status, int64_t R, int64_t A,
    BBParams P, int stage_atoms, int32_t rev, int32_t spined, int32_t nt)
{
    static_assert(GM == kGradLoad || RECOMPUTE, "the fused step recomputes the frames");
    extern __shared__ __align__(16) float stage_mem[];
    __shared__ __align__(16) FADevTable tab;
    __shared__ SpineShared shf;
    __shared__ BwdShared shb;
    __shared__ float fcarry_sh[12];
    __shared__ float rcarry_sh[6];
    __shared__ uint64_t unit_flags[kMaxWaves];
    __shared__ float loss_tot[GM == kGradMse ? kMaxWaves : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool lead = LEADS && is_lead();
    const int64_t t = LEADS ? window_with_leads()
                      : LINK && rev ? reverse_window(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    ChunkRange k;
    window_range<LINK>(wstart, cap, R, t, k.cs, k.ce);
    k.nact = (int)((k.ce - k.cs + kWave * K - 1) / (kWave * K));
    const TableCopy tc = table_load(gtab);
    uint64_t prev = 0, prev_f = 0, prev_l = 0;
    int64_t last = t, first = t;
    if (wave == 0) {
        if constexpr (LINK) {
            prev = lb_load(status + t * kLbWords);
            last = look_last[t];
            if (RECOMPUTE) {
                prev_f = lb_load(LEADS && !lead ? status + t * kLbWords + kLbLeadWord
                                                   : status_fwd + t * kLbWords);
                first = lead ? t : look_fwd[t];
            }
        }
        if (GM == kGradMse && loss_out) prev_l = lb_load(status + t * kLbWords + kLbLossWord);
    }
    const LaneRun<K> L = lane_run<K>(k, head_bits, res_aoff);
    const LaneRes<K, RECOMPUTE> lr = load_lane_res<K, RECOMPUTE>(L, seq, res_aoff, ang, R);
    // the wave's upstream gradients (or targets): the first rows are under
    // way during the spine scan
    constexpr int planes = RECOMPUTE ? 3 : 6;
    float *st = stage_mem + (size_t)wave * planes * stage_atoms;
    float *stx = st + 3 * stage_atoms;  // coordinates (coordinate mode)
    RunStart gr;
    if (STG && L.active && !lead) gr = run_start(g, A, L.A0, L.natoms);
    table_store(tab, tc);
    Aff cur = aff_identity();
    ResidueIn in[K];
    if constexpr (RECOMPUTE) {
        Aff unit = aff_identity();
        if (L.active) {
            lane_sincos<K>(lr, in);
            unit = spine_unit<K>(in, L, P);
        }
        const int n_units = (int)((k.ce - k.cs + K - 1) / K);
        if (LEADS && !lead) prev_f = lead_tag(status, t, prev_f);
        cur = entering_frame<LINK>(unit, L.hm != 0u, n_units, stage_mem, unit_flags, shf,
                                   fcarry_sh, status_fwd, t, first, prev_f,
                                   LEADS ? !lead : spined != 0);
        if (LEADS && lead) return;
    }
    __syncthreads();  // the stage takes the frames' place; the table is complete
    if (STG && L.active) {
        run_to_lds(gr, st, g, A, L.A0, L.natoms);
        if (!RECOMPUTE)
            run_to_lds(run_start(xyz, A, L.A0, L.natoms), stx, xyz, A, L.A0, L.natoms);
    }
    // the C atom before the lane's first residue (coordinate mode): in
    // the staged run for lanes > 0, from global memory for lane 0
    float pcx = 0.f, pcy = 0.f, pcz = 0.f;
    if (!RECOMPUTE && lane == 0 && L.cnt > 0 && !(L.hm & 1u)) {
        const int64_t ac = res_aoff[L.rs - 1] + 2;
        pcx = xyz[ac]; pcy = xyz[A + ac]; pcz = xyz[2 * A + ac];
    }
    SpineGrad sp[K];
    Wrench agg = wrench_zero();
    bool f_end = false;
    // upstream gradient (or target), coordinates in, positions out
    const Atoms<STG> ga = STG ? Atoms<STG>{st, 0} : Atoms<STG>{const_cast<float *>(g) + L.A0, A};
    const Atoms<STG> xa = STG ? Atoms<STG>{stx, 0} : Atoms<STG>{const_cast<float *>(xyz) + L.A0, A};
    const Atoms<STG> oa = STG ? ga : Atoms<STG>{xyz_out + L.A0, A};
    AtomForce<GM, STG> force{ga, oa, xyz_out != nullptr, 0.f};
    if (L.active) {
        wave_lds_sync();
        // first atom of the residue before the lane: the previous lane's last
        const int prev_aoff = __builtin_amdgcn_mov_dpp(lr.aoff[K - 1], kDppWaveShr1, 0xf, 0xf, true);
        if (!RECOMPUTE && lane > 0 && L.cnt > 0 && !(L.hm & 1u)) {
            const F3 p = xa.get(prev_aoff + 2 - (int)L.A0);
            pcx = p.x; pcy = p.y; pcz = p.z;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (j < L.cnt) {
                TypeAt ty = type_at(tab, lr.type[j]);
                const int aloc = lr.aoff[j] - (int)L.A0;
                const bool head = (L.hm >> j) & 1u;
                // each group's wrench goes to the axes that move it once the
                // residue is walked (N: every group; CA: its own, the side
                // chain, C's; C: its own; side frame f: frames f and after)
                SpineGrad gq;
                NodeGrad sc[A2C_MAX_SIDE_FRAMES];
                Wrench wn = wrench_zero(), wca = wrench_zero(), wc = wrench_zero();
                Wrench ws[A2C_MAX_SIDE_FRAMES];
                Wrench side = wrench_zero();  // starts as the last frame's extra atoms
                if constexpr (RECOMPUTE) {
                    auto into = [&](Wrench &w) {
                        return [&](int e, float x, float y, float z) { force(w, e, x, y, z); };
                    };
                    if (head) cur = aff_identity();
                    aff_apply_transform(cur, P.ct[0], P.st[0], P.d[0], in[j].co, in[j].so);
                    gq.n = node_of_frame(cur);
                    force(wn, aloc, cur.t0, cur.t1, cur.t2);
                    walk_extras(ty, extra_count(ty, 0), cur, aloc, into(wn));
                    aff_apply_transform(cur, P.ct[1], P.st[1], P.d[1], in[j].cp, in[j].sp);
                    gq.ca = node_of_frame(cur);
                    force(wca, aloc + 1, cur.t0, cur.t1, cur.t2);
                    walk_extras(ty, extra_count(ty, 1), cur, aloc, into(wca));
                    if (ty.n_side > 0) {
                        Aff sf = cur;
                        aff_rot_x(sf, ty.ft->pre_c, ty.ft->pre_s);
                        int n_last = 0;
#pragma unroll
                        for (int f = 0; f < A2C_MAX_SIDE_FRAMES; ++f) {
                            if (f < ty.n_side) {
                                side_step(sf, *ty.ft, f, lr.chi[j][f]);
                                sc[f] = node_of_frame(sf);
                                ws[f] = wrench_zero();
                                force(ws[f], aloc + (int)((ty.origin >> (8 * f)) & 255u), sf.t0,
                                      sf.t1, sf.t2);
                                n_last = extra_count(ty, 2 + f);
                                if (f + 1 < ty.n_side && n_last > 0)
                                    walk_extras(ty, n_last, sf, aloc, into(ws[f]));
                            }
                        }
                        walk_extras(ty, n_last, sf, aloc, into(side));
                    }
                    aff_apply_transform(cur, P.ct[2], P.st[2], P.d[2], in[j].cs, in[j].ss);
                    gq.cc = node_of_frame(cur);
                    force(wc, aloc + 2, cur.t0, cur.t1, cur.t2);
                    walk_extras(ty, extra_count(ty, 6), cur, aloc, into(wc));
                } else {
                    auto add = [&](Wrench &w, int e) {
                        const F3 p = xa.get(e), q = ga.get(e);
                        wrench_add_point(w, p.x, p.y, p.z, q.x, q.y, q.z);
                        return p;
                    };
                    auto extras = [&](int n, Wrench &w) {
                        for (int i = 0; i < n; ++i) add(w, aloc + ty.ex[i].slot);
                        ty.ex += n;
                    };
                    const F3 pn = add(wn, aloc);
                    extras(extra_count(ty, 0), wn);
                    const F3 pa = add(wca, aloc + 1);
                    extras(extra_count(ty, 1), wca);
                    const F3 pc = add(wc, aloc + 2);
                    if (head) { pcx = 0.f; pcy = 0.f; pcz = 0.f; }
                    gq.n = node_at(pn.x, pn.y, pn.z, (pn.x - pcx) * P.inv_d[0],
                                   (pn.y - pcy) * P.inv_d[0], (pn.z - pcz) * P.inv_d[0]);
                    gq.ca = node_at(pa.x, pa.y, pa.z, (pa.x - pn.x) * P.inv_d[1],
                                    (pa.y - pn.y) * P.inv_d[1], (pa.z - pn.z) * P.inv_d[1]);
                    gq.cc = node_at(pc.x, pc.y, pc.z, (pc.x - pa.x) * P.inv_d[2],
                                    (pc.y - pa.y) * P.inv_d[2], (pc.z - pa.z) * P.inv_d[2]);
                    F3 pp = pa;
                    int n_last = 0;
#pragma unroll
                    for (int f = 0; f < A2C_MAX_SIDE_FRAMES; ++f) {
                        if (f < ty.n_side) {
                            const float inv = (&ty.ft->inv_d.x)[f];
                            ws[f] = wrench_zero();
                            const F3 o = add(ws[f], aloc + (int)((ty.origin >> (8 * f)) & 255u));
                            sc[f] = node_at(o.x, o.y, o.z, (o.x - pp.x) * inv, (o.y - pp.y) * inv,
                                            (o.z - pp.z) * inv);
                            pp = o;
                            n_last = extra_count(ty, 2 + f);
                            if (f + 1 < ty.n_side && n_last > 0) extras(n_last, ws[f]);
                        }
                    }
                    extras(n_last, side);
                    extras(extra_count(ty, 6), wc);
                    pcx = pc.x; pcy = pc.y; pcz = pc.z;
                }
                // side frame f moves frames f and after: their wrench, summed
                // from the last frame back, folds into each axis once
#pragma unroll
                for (int f = A2C_MAX_SIDE_FRAMES - 1; f >= 0; --f) {
                    if (f < ty.n_side) {
                        wrench_add(side, ws[f]);
                        node_fold(sc[f], side);
                    }
                }
                node_fold(gq.cc, wc);      // C: the C group (with O)
                wrench_add(wca, side);
                wrench_add(wca, wc);
                node_fold(gq.ca, wca);     // CA: its group, the side chain, the C group
                gq.W = wn;
                wrench_add(gq.W, wca);
                node_fold(gq.n, gq.W);     // N: the whole residue
                // chi gradients are complete here (their subtrees end in the residue)
#pragma unroll
                for (int f = 0; f < A2C_MAX_SIDE_FRAMES; ++f)
                    grad_store(&gang[(3 + f) * R + L.rs + j],
                               (f < ty.n_side && ty.ft->fr[f].w != 0.f) ? sc[f].c : 0.f, nt != 0);
                sp[j] = gq;
                if (!f_end) wrench_add(agg, gq.W);
                if ((L.lm >> j) & 1u) f_end = true;
            }
        }
        wave_lds_sync();
        if (STG && GM == kGradMse && xyz_out) {
            lds_to_run(st, xyz_out, A, L.A0, L.natoms);  // the stage now holds r
            wave_lds_sync();
        }
    }
    Wrench S = block_suffix_windows<LINK>(agg, __builtin_amdgcn_ballot_w64(f_end), k.nact, L.active,
                                          shb, rcarry_sh, status, t, last, prev);
    if (L.active) {
#pragma unroll
        for (int j = K - 1; j >= 0; --j) {
            if (j < L.cnt) {
                if ((L.lm >> j) & 1u) S = wrench_zero();
                fa_store_grads(gang, R, L.rs + j, sp[j], S, S, nt != 0);
            }
        }
    }
    if constexpr (GM == kGradMse) {
        if (loss_out)
            lb_loss_commit(force.loss, status, t, LEADS ? gridDim.x >> 1 : gridDim.x, prev_l,
                           loss_out, loss_tot);
    }
}

// Dynamic LDS of a launch: the waves' stages, whose place the frames entering the
// units take first (no frames: the adjoint from coordinates; stage_atoms 0:
// direct I/O).
size_t fa_lds_bytes(FaForm form, int32_t W, int64_t stage_atoms)
{
    const size_t plane = (size_t)W * stage_atoms * sizeof(float);
    return form == FaForm::coords ? 6 * plane : std::max(3 * plane, frame_bytes(W));
}

template <int K, int LB, bool STG>
hipError_t fa_fwd_kl(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s)
{
    const size_t lds = fa_lds_bytes(FaForm::forward, p.fs.W, STG ? p.fs.fa_stage_atoms : 0);
    hipLaunchKernelGGL((p.fs.whole_chains ? fa_forward_flat_kernel<K, LB, false, STG>
                                          : fa_forward_flat_kernel<K, LB, true, STG>),
                       dim3(p.fs.n_win), dim3(p.fs.W * kWave), lds, s, ang, xyz, p.d_head_bits,
                       p.fs.d_wstart, p.fs.cap(), p.d_res_atom_off, p.d_seq, p.d_fa, p.fs.d_look,
                       p.fs.d_status, p.R, p.A, p.bb, p.fs.fa_stage_atoms);
    return hipGetLastError();
}

template <int K, bool STG>
hipError_t fa_fwd_ks(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s)
{
    const int threads = p.fs.W * kWave;
    if (threads <= 256) return fa_fwd_kl<K, 256, STG>(p, ang, xyz, s);
    if (threads <= kLbSmall) return fa_fwd_kl<K, kLbSmall, STG>(p, ang, xyz, s);
    return fa_fwd_kl<K, kLbLarge, STG>(p, ang, xyz, s);
}

template <int K>
hipError_t fa_fwd_k(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s)
{
    if (!p.fs.d_look) return hipErrorInvalidValue;
    return p.fs.fa_unstaged ? fa_fwd_ks<K, false>(p, ang, xyz, s) : fa_fwd_ks<K, true>(p, ang, xyz, s);
}

template <int K, bool RECOMPUTE, int LB, int GM, bool STG>
void fa_bwd_launch(const a2c_plan &p, const float *ang, const float *xyz, const float *g,
                   float *gang, hipStream_t s, float *xyz_out, float *loss_out)
{
    const Sched &S = p.bs;
    const bool pass = RECOMPUTE && S.pass();
    if (pass) launch_spine_pass(ang, p.d_head_bits, S, p.R, p.bb, s);
    const size_t lds = fa_lds_bytes(RECOMPUTE ? FaForm::recompute : FaForm::coords, S.W,
                                    STG ? S.fa_stage_atoms : 0);
    const bool rev = RECOMPUTE ? pass : !S.whole_chains;
    auto kernel = S.whole_chains ? fa_backward_flat_kernel<K, RECOMPUTE, LB, GM, false, STG>
                                 : fa_backward_flat_kernel<K, RECOMPUTE, LB, GM, true, STG>;
    if constexpr (RECOMPUTE && K == 1 && STG)
        if (S.leads) kernel = fa_backward_flat_kernel<K, RECOMPUTE, LB, GM, true, STG, true>;
    hipLaunchKernelGGL(kernel, dim3(RECOMPUTE ? S.linked_groups() : S.n_win), dim3(S.W * kWave), lds,
                       s, ang, xyz, g, gang, xyz_out, loss_out,
                       p.d_head_bits, S.d_wstart, S.cap(), p.d_res_atom_off, p.d_seq, p.d_fa,
                       S.d_status_fwd, S.d_look_fwd, S.d_look, S.d_status, p.R, p.A, p.bb,
                       S.fa_stage_atoms, rev ? 1 : 0, pass ? 1 : 0, p.nt_grad ? 1 : 0);
}

// mode 0: adjoint from coordinates, 1: recompute, 2: fused squared-distance step
template <int K, int MODE, bool STG>
void fa_bwd_dispatch(const a2c_plan &p, const float *ang, const float *xyz, const float *g,
                     float *gang, hipStream_t s, float *xyz_out, float *loss_out)
{
    constexpr bool RC = MODE != 0;
    constexpr int GM = MODE == 2 ? kGradMse : kGradLoad;
    const int threads = p.bs.W * kWave;
    if (threads <= 256) fa_bwd_launch<K, RC, 256, GM, STG>(p, ang, xyz, g, gang, s, xyz_out, loss_out);
    else if (threads <= kLbSmall)
        fa_bwd_launch<K, RC, kLbSmall, GM, STG>(p, ang, xyz, g, gang, s, xyz_out, loss_out);
    else fa_bwd_launch<K, RC, kLbLarge, GM, STG>(p, ang, xyz, g, gang, s, xyz_out, loss_out);
}

template <int K, int MODE>
hipError_t fa_bwd_mode(const a2c_plan &p, const float *ang, const float *xyz, const float *g,
                       float *gang, hipStream_t s, float *xyz_out = nullptr,
                       float *loss_out = nullptr)
{
    if (p.bs.fa_unstaged) fa_bwd_dispatch<K, MODE, false>(p, ang, xyz, g, gang, s, xyz_out, loss_out);
    else fa_bwd_dispatch<K, MODE, true>(p, ang, xyz, g, gang, s, xyz_out, loss_out);
    return hipGetLastError();
}

template <int K>
hipError_t fa_mse_k(const a2c_plan &p, const float *ang, const float *tgt, float *xyz,
                    float *loss_out, float *gang, hipStream_t s)
{
    return fa_bwd_mode<K, 2>(p, ang, nullptr, tgt, gang, s, xyz, loss_out);
}

template <int K>
hipError_t fa_bwd_k(const a2c_plan &p, const float *ang, const float *xyz, const float *g,
                    float *gang, hipStream_t s)
{
    return xyz && p.bs.fa_from_coords ? fa_bwd_mode<K, 0>(p, ang, xyz, g, gang, s)
               : fa_bwd_mode<K, 1>(p, ang, xyz, g, gang, s);
}

}  // namespace

hipError_t launch_fa_forward_scan(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s)
{
    switch (p.fs.K) {
    case 1: return fa_fwd_k<1>(p, ang, xyz, s);
    case 2: return fa_fwd_k<2>(p, ang, xyz, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fa_backward_scan(const a2c_plan &p, const float *ang, const float *xyz,
                                   const float *g, float *gang, hipStream_t s)
{
    switch (p.bs.K) {
    case 1: return fa_bwd_k<1>(p, ang, xyz, g, gang, s);
    case 2: return fa_bwd_k<2>(p, ang, xyz, g, gang, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fa_mse_step(const a2c_plan &p, const float *ang, const float *tgt, float *xyz,
                              float *loss_out, float *gang, hipStream_t s)
{
    switch (p.bs.K) {
    case 1: return fa_mse_k<1>(p, ang, tgt, xyz, loss_out, gang, s);
    case 2: return fa_mse_k<2>(p, ang, tgt, xyz, loss_out, gang, s);
    default: return hipErrorInvalidValue;
    }
}

template <int K, int LB, bool LINK>
static const void *staged_kernel(FaForm form)
{
    switch (form) {
    case FaForm::forward: return (const void *)fa_forward_flat_kernel<K, LB, LINK, true>;
    case FaForm::coords:
        return (const void *)fa_backward_flat_kernel<K, false, LB, kGradLoad, LINK, true>;
    case FaForm::recompute:
        return (const void *)fa_backward_flat_kernel<K, true, LB, kGradLoad, LINK, true>;
    case FaForm::mse: break;
    }
    return (const void *)fa_backward_flat_kernel<K, true, LB, kGradMse, LINK, true>;
}

template <int K, bool LINK>
static const void *staged_kernel(FaForm form, int32_t W)
{
    const int threads = W * kWave;
    return threads <= 256        ? staged_kernel<K, 256, LINK>(form)
           : threads <= kLbSmall ? staged_kernel<K, kLbSmall, LINK>(form)
                                 : staged_kernel<K, kLbLarge, LINK>(form);
}

// The kernel's own LDS and registers come from the loaded code: literals here
// went stale when a kernel changed (the forward over whole chains takes 68
// registers, seven waves a SIMD, the linked one 74, six).  LDS is handed out in
// pieces of 1280 bytes; a SIMD has 512 registers a lane, given in eights, and
// runs at most eight waves.  A workgroup counts as one wave on each SIMD, or as
// many as the fullest holds when its waves are dealt out over the four (five
// waves at four a SIMD: two workgroups; 4096 chains of 50..2000 recomputing 253
// us, 149 at eight waves).
FaHeld fa_held(FaForm form, int32_t K, int32_t W, bool whole_chains, int64_t stage_atoms)
{
    constexpr size_t kCuLds = 160 * 1024, kGranule = 1280;
    constexpr int32_t kSimdRegisters = 512, kSimdWaves = 8, kSimds = 4;
    const size_t dynamic = fa_lds_bytes(form, W, stage_atoms);
    hipFuncAttributes a{};
    const void *kernel = K == 1 ? whole_chains ? staged_kernel<1, false>(form, W)
                                               : staged_kernel<1, true>(form, W)
                         : whole_chains ? staged_kernel<2, false>(form, W)
                                        : staged_kernel<2, true>(form, W);
    if (dynamic > (size_t)kMaxDynamicLds) return {0, 0};
    if (hipFuncGetAttributes(&a, kernel) != hipSuccess) {
        (void)hipGetLastError();  // not for the next launch to report
        return {0, 0};
    }
    const size_t group = (dynamic + a.sharedSizeBytes + kGranule - 1) / kGranule * kGranule;
    const int32_t simd = std::min(kSimdWaves, kSimdRegisters / std::max(8, (a.numRegs + 7) / 8 * 8));
    return {(int32_t)(kCuLds / group), simd / ((W + kSimds - 1) / kSimds)};
}

template <typename F>
static void allow_lds(F kernel)
{
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kMaxDynamicLds);
}

template <int K, int LB, bool LINK>
static void allow_lds_kll()
{
    allow_lds(fa_forward_flat_kernel<K, LB, LINK, true>);
    allow_lds(fa_backward_flat_kernel<K, false, LB, kGradLoad, LINK, true>);
    allow_lds(fa_backward_flat_kernel<K, true, LB, kGradLoad, LINK, true>);
    allow_lds(fa_backward_flat_kernel<K, true, LB, kGradMse, LINK, true>);
    if constexpr (K == 1 && LINK) {
        allow_lds(fa_backward_flat_kernel<K, true, LB, kGradLoad, LINK, true, true>);
        allow_lds(fa_backward_flat_kernel<K, true, LB, kGradMse, LINK, true, true>);
    }
}

template <int K, int LB>
static void allow_lds_kl()
{
    allow_lds_kll<K, LB, false>();
    allow_lds_kll<K, LB, true>();
}

void fa_allow_large_lds()
{
    static bool done = false;
    if (done) return;
    allow_lds_kl<1, 256>();
    allow_lds_kl<2, 256>();
    allow_lds_kl<1, kLbSmall>();
    allow_lds_kl<2, kLbSmall>();
    allow_lds_kl<1, kLbLarge>();
    allow_lds_kl<2, kLbLarge>();
    done = true;
}

}  // namespace a2c
