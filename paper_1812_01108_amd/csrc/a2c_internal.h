// Internal declarations shared by the host API and the kernel files.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "a2c.h"
#include "schedule.h"

namespace a2c {

constexpr int kWave = 64;
constexpr int kMaxWaves = 16;
constexpr int kMaxChunks = 64;        // chunks of 64 W K residues per tile
// dynamic LDS allowed to the full-atom kernels (160 KB per workgroup on
// gfx950, less the static tables)
constexpr int kMaxDynamicLds = 136 * 1024;
// Launch-bound classes of the scan kernels: a workgroup of up to 8 waves (512
// lanes) leaves a kernel up to 256 VGPRs, one of 16 waves 128 (the backbone
// forward and the adjoint that recomputes its frames on windows ask for four
// waves per SIMD, 128 VGPRs, in either class).  Launchers pick the class from
// the schedule's wave count.
constexpr int kLbSmall = 512, kLbLarge = 1024;
// Source of the upstream coordinate gradient in the recompute adjoints: read
// from memory, or 2 (r - t) of the squared distance to a target (the fused
// training step).
constexpr int kGradLoad = 0, kGradMse = 1;
// Window look-back: tagged 64-bit words per tile aggregate (a 3x4 affine)
constexpr int kLbWords = 12;
// LRMSD: atoms per segment (one workgroup of 256 lanes, 16 atoms per lane)
constexpr int kLrSegAtoms = 4096;
// LRMSD gradient pieces: four atoms per thread of a 256-thread workgroup
constexpr int kLrPieceAtoms = 1024;

// Backbone slot constants in float32, slot order N (omega), CA (phi), C (psi).
// (ct, st) is a float32 pair chosen so that ct^2 + st^2 is as close to 1 as
// float32 allows near (cos theta, sin theta), which keeps the repeated fixed
// rotations from drifting in scale along long chains.
struct BBParams {
    float ct[3], st[3], d[3], inv_d[3];
};

// Full-atom constants of one residue type.  Frames: 0 N, 1 CA, 2 C (spine,
// backbone geometry) and 3 + f for side frame f; side frames form a chain
// CA -> 0 -> 1 -> ... (frame f hangs off f-1), frame 0 through a fixed
// rotation about CA's x axis.  Atoms are grouped by frame.
// One atom of a residue type: position in its frame and output slot, packed
// so that a kernel reads it from LDS in one 16-byte access.
struct alignas(16) FAAtom {
    float x, y, z;
    int32_t slot;
};

struct FAType {
    int32_t n_atoms;
    int32_t n_side;
    int32_t side_chi[4];            // 1: torsion chi_{f+1} (plane 3 + f); 0: fixed 0
    float pre_c, pre_s;             // fixed rotation of side frame 0
    float ct[4], st[4], d[4], inv_d[4];
    int32_t fbegin[7], fcount[7];   // atoms of frame k in the sorted lists
    int32_t origin_slot[7];         // residue slot of the atom at frame k's origin
    FAAtom atom[A2C_MAX_RESIDUE_ATOMS];   // sorted by frame
};

struct FATable {
    FAType t[A2C_NUM_RESIDUE_TYPES];
};

// The same as the kernels read it, 272 bytes per type: an odd number of
// 16-byte pieces, so that lanes reading the same field of different types
// spread over the LDS banks.
struct alignas(16) FADevType {
    float4 fr[4];                   // side frame f: cos, sin theta, d, 1 where it has a chi
    float4 inv_d;                   // 1 / d of the side frames
    float pre_c, pre_s;             // fixed rotation of side frame 0
    uint32_t origin;                // byte f: residue slot of side frame f's origin atom
    uint32_t counts;                // nibble i < 7: extra atoms at position i of the walk (N,
                                    // CA, side frames 0..3, C); nibble 7: side frames
    FAAtom ex[A2C_MAX_RESIDUE_ATOMS - 3];  // extra atoms (not at a frame's origin), walk order
};
static_assert(sizeof(FADevType) == 272, "odd number of 16-byte pieces");

struct FADevTable {
    FADevType t[A2C_NUM_RESIDUE_TYPES];
};

// Windows ahead of its own that a window of a recomputing adjoint may wait
// on.  A launch whose windows wait ahead progresses only where the device (a
// partition, a masked stream, what other work leaves of it) holds all of them
// at once: 8 workgroups, as the adjoints that take their windows last to first
// need too (reverse_window).  In batches with a chain over more windows the
// spine aggregates are published first, by leads or a spine pass, and the
// windows then go last to first.
constexpr int kMaxAhead = 7;

// One scan schedule: K residues per lane, W waves per workgroup, and the
// layouts built for them, in chunks of C = 64 W K residues.
//   - windows of at most C residues with look tables (every kernel but the
//     backbone adjoint that recomputes the frames).  They hold whole chains
//     where every chain fits in one and that packs well, and are fixed,
//     [t C, t C + C), otherwise;
//   - own windows (the backbone fused step): whole chains wherever every chain
//     fits in one;
//   - for that adjoint, whose chunk may differ (rec: the default adjoint
//     schedule has one of its own), windows of whole chains as well, or, where
//     a chain is longer than a chunk, tiles: chains of at most one chunk packed
//     whole, a longer chain alone.
// n_tiles is what the schedule reports: windows, or for the backbone adjoint
// the tiles its own chunk C would take.
struct Sched {
    int32_t K = 4, W = 4, n_tiles = 0;
    int32_t n_win = 0;                   // windows (0: none)
    int32_t *d_wstart = nullptr;         // n_win + 1 window boundaries (residues)
    bool whole_chains = false;           // every window holds whole chains (no
                                         // window waits on another)
    int32_t *d_look = nullptr;           // n_win: forward, the first window whose
                                         // aggregate window t composes; adjoint, the
                                         // last window whose wrench it adds (t: none)
    uint64_t *d_status = nullptr;        // n_win x kLbWords tagged words
    // recomputing adjoints on fixed windows: each window's spine aggregate in
    // its own tagged words; a window composes those of the windows its first
    // chain spans (from d_look_fwd[t] to t - 1)
    int32_t *d_look_fwd = nullptr;       // n_win, first window to compose
    uint64_t *d_status_fwd = nullptr;    // n_win x kLbWords tagged words
    bool spined = false;                 // a chain spans more than kMaxAhead + 1 windows,
    bool leads = false;                  // and leads publish the aggregates (else a pass)
    int32_t fa_stage_atoms = 0;          // per-wave staging (floats per plane)
    bool fa_unstaged = false;            // stage too large for the LDS: direct I/O
    bool fa_from_coords = false;         // the adjoint given coordinates reads them
    int32_t n_own = 0;                   // own windows
    int32_t *d_own_wstart = nullptr;     // n_own + 1 boundaries
    uint64_t *d_own_status = nullptr;    // n_own x kLbWords tagged words (loss shares)
    Shape rec{4, 4};                     // backbone adjoint that recomputes the frames
    bool rec_chunked = false;            // tiles, a chain longer than a chunk
    int32_t n_rec = 0;                   // its windows or tiles
    int32_t *d_rec_wstart = nullptr;     // n_rec + 1 boundaries
    int32_t *d_tile_res = nullptr;       // n_rec (first, end) residue pairs, longest first
    int32_t cap() const { return kWave * K * W; }  // residues of a fixed window
    bool pass() const { return spined && !leads; }
    int32_t linked_groups() const { return leads ? 2 * n_win : n_win; }
};

}  // namespace a2c

struct a2c_plan {
    a2c_model model;
    int device = 0;
    int n_cu = 0;                        // compute units of the device
    int32_t n_chains = 0;
    int64_t R = 0, A = 0;
    int32_t max_len = 0;
    std::vector<int32_t> res_off;        // n_chains + 1
    std::vector<int32_t> chain_atom_off; // n_chains + 1
    std::vector<int32_t> res_atom_off;   // R + 1
    std::vector<uint8_t> seq;
    // schedules: fs for the forward, bs for the adjoint and the fused step
    a2c::Sched fs, bs;
    // device tables of schedules that were replaced: a graph captured before
    // the change still launches with them, so they live until the plan does
    std::vector<void *> retired;
    // store-vs-recompute threshold: the forward's coordinates (12 bytes per
    // atom) are kept for the adjoint while they fit; 0 = always recompute
    size_t mem_budget = 0;
    // the schedules the plan starts with, and the chunk its backbone adjoint
    // that recomputes the frames has under them (build_sched: the same pair
    // always brings the same chunk)
    a2c::Shape def_fwd{0, 0}, def_adj{0, 0}, def_rec{0, 0};
    // the adjoints write the angle gradients, and the inverse map the angles,
    // with non-temporal stores (at least kNtGradBytes of them)
    bool nt_grad = false;
    // device tables
    uint32_t *d_head_bits = nullptr;     // bit r: residue r starts a chain (bit R set)
    int32_t *d_res_off = nullptr;        // chain residue offsets (plain form)
    int32_t *d_res_atom_off = nullptr;   // R + 1 (full-atom)
    uint8_t *d_seq = nullptr;            // R (full-atom)
    a2c::FADevTable *d_fa = nullptr;     // full-atom constants
    a2c::BBParams bb{};
    a2c::FATable fa_host{};
    a2c::FADevTable fa_dev{};
    // LRMSD segments (the sums): runs of at most kLrSegAtoms atoms of one
    // chain; pieces (the gradient): runs of at most kLrPieceAtoms
    int32_t lr_n_seg = 0;
    std::vector<int32_t> lr_seg_atom;    // lr_n_seg + 1 first atoms (last = A)
    std::vector<int32_t> lr_seg_origin;  // lr_n_seg first atom of each segment's chain
    std::vector<int32_t> lr_chain_seg;   // n_chains + 1 first segment of each chain
    int32_t lr_n_piece = 0;
    std::vector<int32_t> lr_piece_atom;  // lr_n_piece + 1 first atoms (last = A)
    std::vector<int32_t> lr_piece_chain; // lr_n_piece chain of each piece
    int32_t inv_stage_atoms = 0;         // most atoms a workgroup of the inverse map stages
    uint8_t *d_chi_points = nullptr;     // [20][8] points of the chi torsions (full-atom)
    int32_t *d_lr_seg_atom = nullptr;
    int32_t *d_lr_seg_origin = nullptr;
    int32_t *d_lr_chain_seg = nullptr;
    int32_t *d_lr_piece_atom = nullptr;
    int32_t *d_lr_piece_chain = nullptr;
};

namespace a2c {

// Angle gradients of at least this many bytes are written with non-temporal
// stores: nothing in a training step reads them before the next step, and
// on large batches their cache lines would otherwise evict coordinates and
// upstream gradients that the step reads again.  Below it the cached stores
// are faster (the whole step then stays in the caches).
constexpr size_t kNtGradBytes = (size_t)4 << 20;

void set_error(const std::string &msg);
// the checks a2c_plan_set_schedule (and the adjoint setter) makes on (K, W),
// without the device; the forward setter's checks (K = 8 too for the backbone)
a2c_status check_schedule_args(const a2c_plan *p, int32_t K, int32_t W);
a2c_status check_forward_schedule_args(const a2c_plan *p, int32_t K, int32_t W);
hipError_t launch_fill_zero(float *x, int64_t n, hipStream_t s);
// float32 (cos t, sin t) pair with squared norm closest to 1
void unit_pair(double t, float &c, float &s);
a2c_status hip_fail(hipError_t e, const char *what);

// Launchers (each returns hipSuccess or the launch error)
// quat: the comparison form with the quaternion + translation scan state
hipError_t launch_bb_forward_scan(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s,
                                  bool quat = false);
hipError_t launch_bb_backward_scan(const a2c_plan &p, const float *ang, const float *xyz,
                                   const float *g, float *gang, hipStream_t s);
hipError_t launch_bb_forward_plain(const a2c_plan &p, const float *ang, float *xyz, float *ws,
                                   hipStream_t s);
hipError_t launch_bb_backward_plain(const a2c_plan &p, const float *ang, const float *g,
                                    float *gang, const float *ws, hipStream_t s);
// loss (may be NULL): receives sum |r - t|^2, from the windows' shares, which
// travel in the adjoint's tagged words (lb_loss_commit)
hipError_t launch_bb_mse_step(const a2c_plan &p, const float *ang, const float *tgt, float *xyz,
                              float *loss, float *gang, hipStream_t s);
hipError_t launch_fa_mse_step(const a2c_plan &p, const float *ang, const float *tgt, float *xyz,
                              float *loss, float *gang, hipStream_t s);
hipError_t launch_fa_forward_scan(const a2c_plan &p, const float *ang, float *xyz, hipStream_t s);
hipError_t launch_fa_backward_scan(const a2c_plan &p, const float *ang, const float *xyz,
                                   const float *g, float *gang, hipStream_t s);
// Workgroups of a staged full-atom launch that a compute unit holds at once, by
// its LDS and by its registers (both 0 where the stage does not fit), for the
// kernel that the launch takes; stage_atoms as in Sched.
enum class FaForm { forward, coords, recompute, mse };
struct FaHeld {
    int32_t by_lds, by_registers;
};
FaHeld fa_held(FaForm form, int32_t K, int32_t W, bool whole_chains, int64_t stage_atoms);
void build_lrmsd_segments(a2c_plan &p);
void build_chi_points(const FATable &T, uint8_t (&out)[A2C_NUM_RESIDUE_TYPES][8]);
int32_t inverse_stage_atoms(const a2c_plan &p);
size_t lrmsd_workspace_bytes(const a2c_plan &p);
// device address of the no-allocation LRMSD scratch on `device` (current)
a2c_status lrmsd_scratch_setup(int device);
void fa_allow_large_lds();
void bb_allow_large_lds();

}  // namespace a2c
