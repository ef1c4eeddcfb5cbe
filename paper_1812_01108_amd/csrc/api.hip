// Host side of the C ABI declared in include/a2c.h: argument validation,
// plan construction (tile packing, head bits, geometry constants, full-atom
// tables) and kernel dispatch.  No call here that can be captured allocates
// or synchronises.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "a2c_internal.h"

namespace a2c {

namespace {
thread_local std::string g_last_error;

a2c_status fail(a2c_status st, const std::string &msg)
{
    g_last_error = msg;
    return st;
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }
bool valid_angle(double v) { return std::isfinite(v) && v > 0.0 && v < 180.0; }

a2c_status upload(void **dst, const void *src, size_t bytes, hipStream_t s)
{
    if (*dst) {
        (void)hipFree(*dst);
        *dst = nullptr;
    }
    if (bytes == 0) return A2C_OK;
    hipError_t e = hipMalloc(dst, bytes);
    if (e != hipSuccess) return hip_fail(e, "hipMalloc");
    e = hipMemcpyAsync(*dst, src, bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    return A2C_OK;
}

// The device tables a schedule owns.
std::vector<void *> sched_tables(const Sched &S)
{
    return {S.d_tile_res, S.d_wstart,     S.d_look,      S.d_status, S.d_look_fwd, S.d_status_fwd,
            S.d_own_wstart, S.d_own_status, S.d_rec_wstart};
}

void forget_tables(Sched &S)
{
    S.d_tile_res = S.d_wstart = S.d_look = S.d_look_fwd = S.d_own_wstart = nullptr;
    S.d_rec_wstart = nullptr;
    S.d_status = S.d_status_fwd = S.d_own_status = nullptr;
}

void free_sched(Sched &S)
{
    for (void *q : sched_tables(S)) (void)hipFree(q);
    forget_tables(S);
}

// Boundaries of windows of at most `cap` residues that hold whole chains,
// packed greedily in order (none for an empty batch or where a chain is
// longer than cap).  Zero-length chains take no space.
std::vector<int64_t> whole_chain_starts(const a2c_plan *p, int64_t cap)
{
    std::vector<int64_t> st;
    if (p->R == 0 || p->max_len > cap) return st;
    st.push_back(0);
    int64_t cur = 0;  // residues in the open window
    for (size_t c = 0; c + 1 < p->res_off.size(); ++c) {
        const int64_t L = p->res_off[c + 1] - p->res_off[c];
        if (L == 0) continue;
        if (cur + L > cap) {
            st.push_back(p->res_off[c]);
            cur = 0;
        }
        cur += L;
    }
    st.push_back(p->R);
    return st;
}

// Window boundaries for windows of at most `cap` residues (n_win + 1
// entries; none for an empty batch).  Where every chain fits in a window and
// packing whole chains greedily, in order, takes at most 1/8 more windows
// than cutting the batch into fixed windows [t cap, t cap + cap), or no more
// windows than the device has CUs (a launch that leaves CUs idle anyway),
// the windows hold whole chains: no chain crosses a window edge and no window
// waits on another (whole_chains is set).  Otherwise the fixed windows,
// wherever the chains fall.  Zero-length chains take no space.
std::vector<int64_t> window_starts(const a2c_plan *p, int64_t cap, bool &whole_chains)
{
    std::vector<int64_t> st = whole_chain_starts(p, cap);
    whole_chains = false;
    if (p->R == 0) return st;
    const int64_t n_fixed = (p->R + cap - 1) / cap;
    const int64_t n_whole = (int64_t)st.size() - 1;
    if (!st.empty() && (n_whole <= n_fixed + n_fixed / 8 || n_whole <= p->n_cu)) {
        whole_chains = true;
        return st;
    }
    st.clear();
    for (int64_t b = 0; b < p->R; b += cap) st.push_back(b);
    st.push_back(p->R);
    return st;
}

// The window holding residue r (starts as from window_starts).
int32_t window_of(const std::vector<int64_t> &starts, int64_t r)
{
    return (int32_t)(std::upper_bound(starts.begin(), starts.end() - 1, r) - starts.begin()) - 1;
}

// kLbWords tagged words for each of n windows, at tag 0.
a2c_status new_words(uint64_t *&d_status, int64_t n, hipStream_t s)
{
    const size_t words = (size_t)std::max<int64_t>(1, n) * kLbWords * sizeof(uint64_t);
    hipError_t e = hipMalloc((void **)&d_status, words);
    if (e == hipSuccess) e = hipMemsetAsync(d_status, 0, words, s);
    return e == hipSuccess ? A2C_OK : hip_fail(e, "look-back words");
}

// Look-back table and tagged words of the windows given by starts.  Forward
// (look_back): for each window t the first window whose aggregate its
// carry-in needs, i.e. the window holding the head of the chain its first
// residue belongs to (t itself when a chain starts there).  Adjoint: the last
// window whose wrench it adds, i.e. the window holding the end of the chain
// of its last residue (t itself when a chain ends there).  long_span is set
// where a window looks more than kMaxAhead windows away.  The tagged words
// start at tag 0.
a2c_status build_windows(const a2c_plan *p, const std::vector<int64_t> &starts, bool look_back,
                         int32_t *&d_look, uint64_t *&d_status, int32_t &n_win, bool &long_span,
                         hipStream_t s)
{
    const int64_t n = starts.empty() ? 0 : (int64_t)starts.size() - 1;
    std::vector<int32_t> look((size_t)n);
    size_t c = 0;  // non-empty chain holding the residue: res_off[c] <= r < res_off[c + 1]
    for (int64_t t = 0; t < n; ++t) {
        const int64_t r = look_back ? starts[(size_t)t] : starts[(size_t)t + 1] - 1;
        while (p->res_off[c + 1] <= r) ++c;
        look[(size_t)t] =
            window_of(starts, look_back ? p->res_off[c] : (int64_t)p->res_off[c + 1] - 1);
        if (std::abs((int64_t)look[(size_t)t] - t) > kMaxAhead) long_span = true;
    }
    n_win = (int32_t)n;
    a2c_status st = upload((void **)&d_look, look.data(), look.size() * sizeof(int32_t), s);
    if (st != A2C_OK) return st;
    return new_words(d_status, n, s);
}

// The window boundaries as int32 on the device.
a2c_status upload_starts(const std::vector<int64_t> &starts, int32_t *&d_wstart, hipStream_t s)
{
    std::vector<int32_t> v(starts.begin(), starts.end());
    return upload((void **)&d_wstart, v.data(), v.size() * sizeof(int32_t), s);
}

// Greedy packing of whole chains, in order, into tiles: chains of at most one
// chunk (`cap` residues) share tiles of at most `cap` residues; a longer chain
// gets a tile of its own, which the kernels walk chunk by chunk.  Zero-length
// chains produce nothing and never open a tile.
std::vector<int32_t> pack_tiles(const std::vector<int32_t> &off, int64_t cap)
{
    std::vector<int32_t> tiles;
    const size_t n = off.size() - 1;
    int64_t cur = 0;
    tiles.push_back(0);
    for (size_t c = 0; c < n; ++c) {
        const int64_t L = off[c + 1] - off[c];
        if (L == 0) continue;
        if (cur > 0 && (cur + L > cap || L > cap)) {
            tiles.push_back(off[c]);
            cur = 0;
        }
        cur += L;
        if (L > cap) {  // a long chain closes its own tile
            tiles.push_back(off[c + 1]);
            cur = 0;
        }
    }
    if (cur > 0) tiles.push_back(off[n]);
    if (tiles.size() == 1) tiles.clear();  // no residues
    return tiles;
}

// The most atoms of one wave's run of `run` residues in the windows `starts`,
// in whole pieces of the kernels' copies (four atoms).
int64_t most_run_atoms(const a2c_plan &p, const std::vector<int64_t> &starts, int64_t run)
{
    int64_t most = 1;
    for (size_t t = 0; t + 1 < starts.size(); ++t)
        for (int64_t rb = starts[t]; rb < starts[t + 1]; rb += run) {
            const int64_t re = std::min<int64_t>(rb + run, starts[t + 1]);
            most = std::max<int64_t>(most, p.res_atom_off[re] - p.res_atom_off[rb]);
        }
    return (most + 3) / 4 * 4;
}

// Whether leads publish the spine aggregates of a launch of n windows that
// needs them published first: where the device holds both halves of the launch
// at once (four waves, four workgroups a CU); more windows take a spine pass,
// which has eight residues per lane.  Built for one residue per lane.
// Recomputing adjoint and fused step at (1, 4), us, with the pass and with
// leads: full-atom, one chain of 6000 17.9 and 19.9, 13.9 and 15.9; 40 of
// 1500..6000 (508 windows) 20.1 and 22.8, 16.5 and 19.1; 60 (790) 24.1 and
// 26.8, 23.3 and 26.2; 150 (1911) 44.3 and 48.5, 45.1 and 50.4.  Backbone fused
// step, one chain of 6000 15.1 and 10.8, 40 (508) 18.3 and 16.2, 60 (790) 21.4
// and 20.7.
bool lead_windows(const a2c_plan &p, int64_t n) { return n <= 2 * (int64_t)p.n_cu; }

// Layouts of a schedule (see Sched).
enum SchedRole { kRoleForward, kRoleAdjoint };

a2c_status build_sched(const a2c_plan *p, int32_t K, int32_t W, Sched &out, hipStream_t s,
                       SchedRole role)
{
    const int64_t cap = (int64_t)kWave * W * K;  // residues per chunk
    if (p->max_len > cap * kMaxChunks)
        return fail(A2C_ERR_UNSUPPORTED, "a chain of " + std::to_string(p->max_len) +
                                             " residues needs more than " +
                                             std::to_string(kMaxChunks) + " chunks of " +
                                             std::to_string(cap) + " residues");
    Sched S;
    S.K = K;
    S.W = W;
    const std::vector<int64_t> starts = window_starts(p, cap, S.whole_chains);
    if (p->model == A2C_FULLATOM) {
        // per-wave LDS stage of three planes (the adjoint from coordinates
        // stages six where they fit): the most atoms of one wave's run of
        // 64 K residues
        const int64_t most = most_run_atoms(*p, starts, (int64_t)kWave * K);
        if ((size_t)W * 3 * most * sizeof(float) > (size_t)kMaxDynamicLds)
            S.fa_unstaged = true;  // atoms straight to global memory
        else
            S.fa_stage_atoms = (int32_t)most;
        // the form from coordinates stages six planes; where they do not fit,
        // the recomputing form (three planes) computes the same gradient, and
        // where their LDS leaves the launch more than one round it is the
        // faster one: (1, 4), us from coordinates and recomputing: 64 x 300 9.1
        // and 13.2, 1000 chains of 100 10.5 and 13.8, 512 of 50..2000 24.4 and
        // 20.0, 4096 of them 206 and 141
        S.fa_from_coords =
            S.fa_unstaged ||
            (int64_t)starts.size() - 1 <=
                (int64_t)fa_held(FaForm::coords, K, W, S.whole_chains, most).by_lds * p->n_cu;
    }
    const bool fwd = role == kRoleForward;
    bool ignored = false;
    a2c_status st = upload_starts(starts, S.d_wstart, s);
    if (st == A2C_OK)
        st = build_windows(p, starts, fwd, S.d_look, S.d_status, S.n_win, ignored, s);
    S.n_tiles = S.n_win;
    if (st == A2C_OK && !fwd) {
        // the recomputing adjoints: the spine aggregates' words and the
        // windows whose aggregates each window composes (the fused step's
        // loss shares travel in the adjoint's own tagged words)
        int32_t n2 = 0;
        st = build_windows(p, starts, true, S.d_look_fwd, S.d_status_fwd, n2, S.spined, s);
        S.leads = S.spined && K == 1 && !S.fa_unstaged && lead_windows(*p, S.n_win);
    }
    if (st == A2C_OK && !fwd && p->model == A2C_BACKBONE && p->R > 0) {
        const std::vector<int64_t> own = whole_chain_starts(p, cap);
        if (!own.empty()) {
            S.n_own = (int32_t)own.size() - 1;
            st = upload_starts(own, S.d_own_wstart, s);
            if (st == A2C_OK) st = new_words(S.d_own_status, S.n_own, s);
        }
        // the chunk of the recomputing adjoint: the schedule's own, but for the
        // default pair, whether it is the plan's first schedule or set again
        S.rec = Shape{K, W} == p->def_adj ? p->def_rec : Shape{K, W};
        const int64_t rec_cap = (int64_t)kWave * S.rec.W * S.rec.K;
        const std::vector<int64_t> rec = whole_chain_starts(p, rec_cap);
        S.rec_chunked = rec.empty();
        if (st == A2C_OK && !S.rec_chunked) {
            S.n_rec = (int32_t)rec.size() - 1;
            st = upload_starts(rec, S.d_rec_wstart, s);
        } else if (st == A2C_OK) {
            // (first, end) residue pairs, longest tile first: tiles are
            // independent, and dispatching the long ones first keeps them out
            // of the tail of the launch
            const std::vector<int32_t> tiles = pack_tiles(p->res_off, rec_cap);
            S.n_rec = (int32_t)tiles.size() - 1;
            std::vector<int32_t> order(S.n_rec);
            for (int32_t t = 0; t < S.n_rec; ++t) order[t] = t;
            std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
                return tiles[a + 1] - tiles[a] > tiles[b + 1] - tiles[b];
            });
            std::vector<int32_t> pairs(2 * (size_t)S.n_rec);
            for (int32_t t = 0; t < S.n_rec; ++t) {
                pairs[2 * t] = tiles[order[t]];
                pairs[2 * t + 1] = tiles[order[t] + 1];
            }
            st = upload((void **)&S.d_tile_res, pairs.data(), pairs.size() * sizeof(int32_t), s);
        }
        S.n_tiles = S.rec == Shape{K, W} ? S.n_rec
                                         : (int32_t)pack_tiles(p->res_off, cap).size() - 1;
    }
    // the host tables above are read by the copies until here
    const hipError_t e = hipStreamSynchronize(s);
    if (st == A2C_OK && e != hipSuccess) st = hip_fail(e, "hipStreamSynchronize");
    if (st != A2C_OK) {
        free_sched(S);
        return st;
    }
    out = S;
    return A2C_OK;
}

// A replaced schedule's device tables stay allocated until the plan is
// destroyed: a graph captured before the change still launches with them.
void retire_sched(a2c_plan *p, Sched &S)
{
    for (void *q : sched_tables(S))
        if (q) p->retired.push_back(q);
    forget_tables(S);
}

// Replace one of the plan's schedules; on failure it stays as it was.  The
// old tables are retired (kept until the plan is destroyed), or freed at once
// when retire_old is false: the autotuner's own candidates, which no graph
// can have captured.
a2c_status set_sched(a2c_plan *p, Sched &dst, int32_t K, int32_t W, hipStream_t s,
                     bool retire_old = true)
{
    Sched S;
    const a2c_status st = build_sched(p, K, W, S, s, &dst == &p->fs ? kRoleForward : kRoleAdjoint);
    if (st != A2C_OK) return st;
    if (retire_old) retire_sched(p, dst);
    else free_sched(dst);
    dst = S;
    return A2C_OK;
}

// Both schedules (forward, and adjoint / fused step) to (K, W).
a2c_status apply_schedule(a2c_plan *p, int32_t K, int32_t W, hipStream_t s,
                          bool retire_old = true)
{
    Sched f, b;
    a2c_status st = build_sched(p, K, W, f, s, kRoleForward);
    if (st != A2C_OK) return st;
    st = build_sched(p, K, W, b, s, kRoleAdjoint);
    if (st != A2C_OK) {
        free_sched(f);
        return st;
    }
    if (retire_old) {
        retire_sched(p, p->fs);
        retire_sched(p, p->bs);
    } else {
        free_sched(p->fs);
        free_sched(p->bs);
    }
    p->fs = f;
    p->bs = b;
    return A2C_OK;
}

// ------------------------------------------------------ default schedules
// Rules on the batch's residues R and longest chain, from timing every
// schedule on batches of 150 to 3 M residues (one MI355X, launches back to
// back in a graph; microseconds below).  Few residues want few per lane (the
// walk over them is a serial chain, and waves are short in supply), many want
// more (the wave scan costs the same whatever a lane holds).

int32_t waves_for(int64_t len, int32_t K)
{
    return (int32_t)std::max<int64_t>(1, (len + (int64_t)kWave * K - 1) / (kWave * K));
}

// The fewest waves, from `least` to `most`, at which windows of whole chains
// are no more than the device has CUs (one round, nothing handed over);
// `least` where none is.  1000 chains of 100, K = 1: adjoint 5.9 at W = 2, 4.6
// at W = 8; full-atom forward 11.5 and 10.8.
int32_t pack_waves(const a2c_plan &p, int32_t K, int32_t least, int32_t most)
{
    for (int32_t W = least; W <= most; ++W) {
        const std::vector<int64_t> st = whole_chain_starts(&p, (int64_t)kWave * K * W);
        if (!st.empty() && (int64_t)st.size() - 1 <= p.n_cu) return W;
    }
    return least;
}

// Whether a full-atom launch of schedule (K, W) is one round of workgroups: the
// LDS and the registers let the device hold all of them at once.
bool one_round(const a2c_plan &p, int32_t K, int32_t W, FaForm form)
{
    const int64_t run = (int64_t)kWave * K;
    const auto holds = [&](int64_t n_win, bool whole, int64_t run_atoms) {
        const FaHeld h = fa_held(form, K, W, whole, run_atoms);
        return n_win <= (int64_t)std::min(h.by_lds, h.by_registers) * p.n_cu;
    };
    // the least there can be, before the windows are laid out
    const int64_t least = (p.R + run * W - 1) / (run * W);
    const int64_t mean_atoms = run * p.A / std::max<int64_t>(1, p.R);
    if (!holds(least, true, mean_atoms) && !holds(least, false, mean_atoms)) return false;
    bool whole;
    const std::vector<int64_t> st = window_starts(&p, run * W, whole);
    return holds((int64_t)st.size() - 1, whole, most_run_atoms(p, st, run));
}

// Whether some chain runs over more than kMaxAhead + 1 fixed windows of `cap`
// residues, so that the recomputing adjoints need the spine aggregates first.
bool spans_far(const a2c_plan &p, int64_t cap)
{
    if (p.max_len <= kMaxAhead * cap) return false;
    for (size_t c = 0; c + 1 < p.res_off.size(); ++c)
        if (p.res_off[c + 1] > p.res_off[c] &&
            (p.res_off[c + 1] - 1) / cap - p.res_off[c] / cap > kMaxAhead)
            return true;
    return false;
}

// Waves of the recomputing adjoints where chains run over several windows, at
// one residue per lane: four, or eight where that saves the spine pass, which
// costs more than eight waves do (leads cost less).  Full-atom, recomputing and
// fused step, us: 512 chains of 50..2000 25.7 and 31.8 at W = 4 with the pass,
// 19.8 and 26.3 at W = 8; 4096 of them 149 and 206, 146 and 199; where eight
// need the pass too (100 of 1500..6000) 37.0 and 41.1 at W = 4, 39.2 and 42.6
// at W = 8; with leads (128 of 50..2000) 14.6 and 17.1 at W = 4, 14.9 and 17.4
// at W = 8.
int32_t linked_waves(const a2c_plan &p)
{
    const int64_t four = 4 * kWave, eight = 8 * kWave;
    if (!spans_far(p, four) || lead_windows(p, (p.R + four - 1) / four)) return 4;
    return spans_far(p, eight) ? 4 : 8;
}

// A launch just over one round takes nearly two: `s` if it is one round, else
// the fewest residues per lane (one, up to most_K) and waves that make it one
// (adjoint: and whose windows wait no further ahead than kMaxAhead where those
// of `s` do not), else `s`.
// Forward: 2000
// chains of 151, 1573 windows at W = 3 23.2, 500 of four chains at W = 10 15.9;
// 580 chains of 50..2000, 24.3 at W = 4, 16.8 at W = 6.  Recomputing adjoint:
// 550 of them, 30.8 at (1, 4), 23.7 at (2, 3).
Shape prefer_one_round(const a2c_plan &p, Shape s, int32_t most_K, FaForm form)
{
    if (one_round(p, s.K, s.W, form)) return s;
    const auto far = [&](int32_t K, int32_t W) { return spans_far(p, (int64_t)kWave * K * W); };
    const bool near_only = form != FaForm::forward && !far(s.K, s.W);
    // (two residues per lane and more than eight waves spill)
    for (int32_t K = 1; K <= most_K; ++K)
        for (int32_t W = 2; W <= kMaxWaves / K; ++W)
            if (one_round(p, K, W, form) && !(near_only && far(K, W)))
                return {K, W};
    return s;
}

Shape default_forward(const a2c_plan &p)
{
    const int64_t R = p.R;
    if (p.model == A2C_FULLATOM) {
        // one residue per lane; four waves (eight for batches of several
        // rounds: 150 chains of 1000..6000 29.9 and 28.3, 4096 of 50..2000
        // 124.7 and 119.9; 2000 of 151 23.2 and 24.2), and one window for a
        // chain of up to 512 where that fits one round (64 x 300: 10.5 at
        // W = 4, 9.2 at W = 6)
        const int32_t whole = waves_for(p.max_len, 1);
        const Shape s{1, whole <= 8 ? pack_waves(p, 1, whole, 8)
                                    : std::min<int32_t>(R > 400000 ? 8 : 4, whole)};
        return prefer_one_round(p, s, 1, FaForm::forward);
    }
    // a batch of a few chunks keeps a chunk that holds its longest chain
    if (p.max_len > 1024 && p.max_len <= 4096 && R <= 4 * 4096) return {4, waves_for(p.max_len, 4)};
    // 150 residues 7.0 at K = 4, 4.6 at K = 1; 256 x 700 8.4 at (4, 3), 7.3 at
    // (2, 6); 700 chains of 20..1000 10.5 at (4, 4), 10.1 at (2, 12); 1500 of
    // them 13.1 at (4, 4), 15.0 at (2, 8)
    const int32_t K = R <= 16384 ? 1 : R <= 393216 ? 2 : 4;
    const int32_t whole = waves_for(p.max_len, K);
    // a chain of more waves than this is handed between smaller windows
    // instead: 48 chains of 1500..6000 12.5 at (4, 16), 8.6 at (2, 8); 8 of
    // 1500..4000 11.3 and 6.8 at (1, 4)
    const int32_t most = K == 1 ? 16 : K == 2 ? 8 : 4;
    if (whole > most) return {K, K == 2 ? 8 : 4};
    return {K, pack_waves(p, K, whole, most)};
}

Shape default_adjoint(const a2c_plan &p, Shape &rec)
{
    const int64_t R = p.R;
    if (p.model == A2C_FULLATOM) {
        // as the forward, but four waves for large batches too
        const int32_t whole = waves_for(p.max_len, 1);
        rec = {1, whole <= 8 ? pack_waves(p, 1, whole, 8) : linked_waves(p)};
        if (whole <= 8 && rec.W > 4 && (int64_t)kWave * rec.W * p.n_cu < R) rec.W = 4;
        return rec = prefer_one_round(p, rec, 2, FaForm::mse);
    }
    // from coordinates: 256 x 700 7.2 at (4, 3), 5.2 at (1, 12); 700 chains of
    // 20..1000 9.2 at (4, 4), 8.3 at (2, 8); 6000 of them 41.4 and 41.9 at
    // (4, 8), which takes the recomputing adjoint from 57.7 to 51.1 (packing
    // whole chains leaves 12 % of its lanes idle instead of 26)
    Shape s;
    s.K = R <= 196608 ? 1 : R <= 524288 ? 2 : 4;
    const int32_t whole = waves_for(p.max_len, s.K);
    const int32_t most = s.K == 1 ? 16 : 8;
    if (s.K == 4) s.W = 8;
    else if (whole <= most) s.W = pack_waves(p, s.K, whole, most);
    // long chains: 48 of 1500..6000, from coordinates 10.7 at (4, 16), 6.6 at
    // (2, 8), fused step 22.1 and 14.6; 8 of 1500..4000, 5.3 and 11.6 at (1, 4)
    else if (R <= 65536) s.W = linked_waves(p);
    else s = {2, 8};
    // the adjoint that recomputes the frames hands nothing over: a chunk that
    // holds the longest chain, up to 4096, and beyond that the one whose
    // chunk walk is fastest (48 chains of 1500..6000: 73 at (4, 16), which
    // spills, 46 at (4, 8), 66 at (2, 8))
    if (waves_for(p.max_len, s.K) <= most) rec = s;
    else if (p.max_len <= 4096) rec = {4, std::max(waves_for(p.max_len, 4), 4)};
    else rec = {4, 8};
    if (waves_for(p.max_len, rec.K) > rec.W && p.max_len <= 4096)
        rec.W = waves_for(p.max_len, rec.K);
    return s;
}

// The most residues a chain may have under `s` is kMaxChunks chunks: more
// waves, then more residues per lane, until the longest chain fits
// (plan_create has already rejected longer ones).
void fit_longest(const a2c_plan &p, Shape &s, int32_t most_K)
{
    while ((int64_t)p.max_len > (int64_t)kWave * s.W * s.K * kMaxChunks) {
        if (s.W < kMaxWaves) s.W = std::min<int32_t>(kMaxWaves, 2 * s.W);
        else if (s.K < most_K) s.K *= 2;
        else break;
    }
}

a2c_status default_schedules(a2c_plan *p, hipStream_t s)
{
    const int32_t most_K = p->model == A2C_BACKBONE ? 4 : 2;
    Shape rec{};
    Shape f = default_forward(*p), b = default_adjoint(*p, rec);
    fit_longest(*p, f, most_K);
    fit_longest(*p, b, most_K);
    fit_longest(*p, rec, most_K);
    p->def_fwd = f;
    p->def_adj = b;
    p->def_rec = rec;
    a2c_status st = build_sched(p, f.K, f.W, p->fs, s, kRoleForward);
    if (st == A2C_OK) st = build_sched(p, b.K, b.W, p->bs, s, kRoleAdjoint);
    return st;
}

bool check_device(const a2c_plan *p)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    return dev == p->device;
}

}  // namespace

// The float32 (c, s) pair within +-2 ulps of (cos t, sin t) whose squared
// norm is closest to 1 (ties broken by the angle error).  Independent
// rounding of cos and sin leaves c^2 + s^2 - 1 ~ 1e-7, a scale error that
// every residue repeats; the pair search makes it ~1e-9.
void unit_pair(double t, float &c_out, float &s_out)
{
    const float c0 = (float)std::cos(t), s0 = (float)std::sin(t);
    double best = std::numeric_limits<double>::infinity();
    c_out = c0;
    s_out = s0;
    float cs[5], ss[5];
    cs[2] = c0;
    ss[2] = s0;
    cs[3] = std::nextafter(c0, 2.f); cs[4] = std::nextafter(cs[3], 2.f);
    cs[1] = std::nextafter(c0, -2.f); cs[0] = std::nextafter(cs[1], -2.f);
    ss[3] = std::nextafter(s0, 2.f); ss[4] = std::nextafter(ss[3], 2.f);
    ss[1] = std::nextafter(s0, -2.f); ss[0] = std::nextafter(ss[1], -2.f);
    for (float c : cs)
        for (float s : ss) {
            const double e = std::fabs((double)c * c + (double)s * s - 1.0) +
                             1e-3 * std::fabs(std::atan2((double)s, (double)c) - t);
            if (e < best) {
                best = e;
                c_out = c;
                s_out = s;
            }
        }
}

// The forward setter's checks: the backbone forward also takes K = 8.
a2c_status check_forward_schedule_args(const a2c_plan *p, int32_t K, int32_t W)
{
    if (p->model == A2C_BACKBONE && K == 8) {
        if (W < 1 || W > kMaxWaves) return fail(A2C_ERR_INVALID_ARG, "waves_per_group must be 1..16");
        return A2C_OK;
    }
    return check_schedule_args(p, K, W);
}

// The checks a2c_plan_set_schedule makes on (K, W), without the device.
a2c_status check_schedule_args(const a2c_plan *p, int32_t K, int32_t W)
{
    if (!(K == 1 || K == 2 || K == 4))
        return fail(A2C_ERR_INVALID_ARG, "res_per_lane must be 1, 2 or 4");
    if (p->model == A2C_FULLATOM && K == 4)
        return fail(A2C_ERR_INVALID_ARG, "the full-atom kernels take res_per_lane 1 or 2");
    if (W < 1 || W > kMaxWaves) return fail(A2C_ERR_INVALID_ARG, "waves_per_group must be 1..16");
    return A2C_OK;
}

namespace {
__global__ void fill_zero_kernel(float *x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.f;
}
}  // namespace

// A kernel, not hipMemsetAsync: callers may capture it in a graph.
hipError_t launch_fill_zero(float *x, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n);
    return hipGetLastError();
}

void set_error(const std::string &msg) { g_last_error = msg; }

a2c_status hip_fail(hipError_t e, const char *what)
{
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return A2C_ERR_HIP;
}

a2c_status build_fullatom_tables(a2c_plan *p, const a2c_residue_table *table);

a2c_status plan_apply_adjoint_schedule(a2c_plan *p, int32_t K, int32_t W, hipStream_t s,
                                       bool retire_old)
{
    return set_sched(p, p->bs, K, W, s, retire_old);
}

a2c_status plan_apply_forward_schedule(a2c_plan *p, int32_t K, int32_t W, hipStream_t s,
                                       bool retire_old)
{
    return set_sched(p, p->fs, K, W, s, retire_old);
}

}  // namespace a2c

using namespace a2c;

extern "C" {

const char *a2c_version(void) { return "a2c 0.1 gfx950"; }

const char *a2c_status_string(int32_t st)
{
    switch (st) {
    case A2C_OK: return "ok";
    case A2C_ERR_INVALID_ARG: return "invalid argument";
    case A2C_ERR_UNSUPPORTED: return "unsupported";
    case A2C_ERR_WORKSPACE: return "workspace missing or too small";
    case A2C_ERR_HIP: return "HIP runtime error";
    case A2C_ERR_STATE: return "invalid state";
    }
    return "unknown status";
}

const char *a2c_last_error(void) { return g_last_error.c_str(); }

void a2c_plan_destroy(a2c_plan *p)
{
    if (!p) return;
    free_sched(p->fs);
    free_sched(p->bs);
    for (void *q : p->retired) (void)hipFree(q);
    (void)hipFree(p->d_head_bits);
    (void)hipFree(p->d_res_off);
    (void)hipFree(p->d_res_atom_off);
    (void)hipFree(p->d_seq);
    (void)hipFree(p->d_fa);
    (void)hipFree(p->d_chi_points);
    (void)hipFree(p->d_lr_seg_atom);
    (void)hipFree(p->d_lr_seg_origin);
    (void)hipFree(p->d_lr_chain_seg);
    (void)hipFree(p->d_lr_piece_atom);
    (void)hipFree(p->d_lr_piece_chain);
    delete p;
}

a2c_status a2c_plan_create(a2c_plan **out, int32_t model_id, int32_t n_chains,
                           const int32_t *h_res_offsets, const uint8_t *h_seq,
                           const a2c_backbone_geometry *geom, const a2c_residue_table *table,
                           size_t mem_budget_bytes, void *stream)
{
    if (!out) return fail(A2C_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (model_id != A2C_BACKBONE && model_id != A2C_FULLATOM)
        return fail(A2C_ERR_INVALID_ARG, "unknown model");
    const a2c_model model = (a2c_model)model_id;
    if (n_chains < 0) return fail(A2C_ERR_INVALID_ARG, "n_chains < 0");
    if (!h_res_offsets) return fail(A2C_ERR_INVALID_ARG, "h_res_offsets is NULL");
    if (h_res_offsets[0] != 0) return fail(A2C_ERR_INVALID_ARG, "h_res_offsets[0] != 0");
    int32_t max_len = 0;
    for (int32_t c = 0; c < n_chains; ++c) {
        const int64_t L = (int64_t)h_res_offsets[c + 1] - h_res_offsets[c];
        if (L < 0)
            return fail(A2C_ERR_INVALID_ARG,
                        "h_res_offsets decreases at chain " + std::to_string(c));
        max_len = std::max<int32_t>(max_len, (int32_t)L);
    }
    const int64_t R = h_res_offsets[n_chains];
    if (R > (int64_t)std::numeric_limits<int32_t>::max() / 16)
        return fail(A2C_ERR_UNSUPPORTED, "too many residues for int32 atom offsets");
    const int32_t max_tile = kMaxChunks * kWave * kMaxWaves * (model == A2C_BACKBONE ? 4 : 2);
    if (max_len > max_tile)
        return fail(A2C_ERR_UNSUPPORTED, "chain longer than " + std::to_string(max_tile) +
                                             " residues");
    if (model == A2C_FULLATOM) {
        if (!table) return fail(A2C_ERR_INVALID_ARG, "full-atom plan needs a residue table");
        if (R > 0 && !h_seq) return fail(A2C_ERR_INVALID_ARG, "full-atom plan needs h_seq");
        for (int64_t r = 0; r < R; ++r)
            if (h_seq[r] >= A2C_NUM_RESIDUE_TYPES)
                return fail(A2C_ERR_INVALID_ARG, "residue code " + std::to_string(h_seq[r]) +
                                                     " >= 20 at residue " + std::to_string(r));
    }
    a2c_backbone_geometry g = {1.458, 1.525, 1.329, 111.2, 116.2, 121.7};
    if (geom) g = *geom;
    if (!finite_pos(g.bond_n_ca) || !finite_pos(g.bond_ca_c) || !finite_pos(g.bond_c_n) ||
        !valid_angle(g.angle_n_ca_c) || !valid_angle(g.angle_ca_c_n) ||
        !valid_angle(g.angle_c_n_ca))
        return fail(A2C_ERR_INVALID_ARG, "backbone geometry out of range");

    hipStream_t s = (hipStream_t)stream;
    a2c_plan *p = new a2c_plan();
    p->model = model;
    p->n_chains = n_chains;
    p->R = R;
    p->max_len = max_len;
    p->mem_budget = mem_budget_bytes;
    p->res_off.assign(h_res_offsets, h_res_offsets + n_chains + 1);
    // slot constants (N, CA, C): bond to the previous atom and the bond angle
    // at the previous atom; theta = pi - angle
    const double pi = 3.14159265358979323846;
    const double bond[3] = {g.bond_c_n, g.bond_n_ca, g.bond_ca_c};
    const double angle[3] = {g.angle_ca_c_n, g.angle_c_n_ca, g.angle_n_ca_c};
    for (int k = 0; k < 3; ++k) {
        unit_pair(pi - angle[k] * (pi / 180.0), p->bb.ct[k], p->bb.st[k]);
        p->bb.d[k] = (float)bond[k];
        p->bb.inv_d[k] = (float)(1.0 / bond[k]);
    }

    a2c_status st = A2C_OK;
    if (model == A2C_BACKBONE) {
        p->A = 3 * R;
        p->chain_atom_off.resize(n_chains + 1);
        for (int32_t c = 0; c <= n_chains; ++c) p->chain_atom_off[c] = 3 * h_res_offsets[c];
    } else {
        p->seq.assign(h_seq, h_seq + R);
        st = build_fullatom_tables(p, table);
        if (st != A2C_OK) {
            a2c_plan_destroy(p);
            return st;
        }
    }
    p->inv_stage_atoms = inverse_stage_atoms(*p);
    p->nt_grad = (size_t)R * (model == A2C_BACKBONE ? 3 : 7) * sizeof(float) >= kNtGradBytes;
    // host tables are complete: now the device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        a2c_plan_destroy(p);
        return hip_fail(e, "hipGetDevice");
    }
    p->device = dev;
    e = hipDeviceGetAttribute(&p->n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) {
        a2c_plan_destroy(p);
        return hip_fail(e, "hipDeviceGetAttribute");
    }
    // chain-head bits, padded by two words so a lane may read one word past
    std::vector<uint32_t> bits((size_t)((R + 64) / 32 + 2), 0u);
    for (int32_t c = 0; c < n_chains; ++c)
        if (h_res_offsets[c + 1] > h_res_offsets[c])
            bits[h_res_offsets[c] >> 5] |= 1u << (h_res_offsets[c] & 31);
    bits[R >> 5] |= 1u << (R & 31);
    st = upload((void **)&p->d_head_bits, bits.data(), bits.size() * sizeof(uint32_t), s);
    if (st == A2C_OK)
        st = upload((void **)&p->d_res_off, p->res_off.data(), p->res_off.size() * sizeof(int32_t), s);
    if (st == A2C_OK && model == A2C_FULLATOM) {
        st = upload((void **)&p->d_res_atom_off, p->res_atom_off.data(),
                    p->res_atom_off.size() * sizeof(int32_t), s);
        if (st == A2C_OK) st = upload((void **)&p->d_seq, p->seq.data(), p->seq.size(), s);
        if (st == A2C_OK) st = upload((void **)&p->d_fa, &p->fa_dev, sizeof(FADevTable), s);
        if (st == A2C_OK) {
            uint8_t chi[A2C_NUM_RESIDUE_TYPES][8];
            build_chi_points(p->fa_host, chi);
            st = upload((void **)&p->d_chi_points, chi, sizeof(chi), s);
        }
    }
    if (st == A2C_OK) {
        build_lrmsd_segments(*p);
        st = upload((void **)&p->d_lr_seg_atom, p->lr_seg_atom.data(),
                    p->lr_seg_atom.size() * sizeof(int32_t), s);
        if (st == A2C_OK)
            st = upload((void **)&p->d_lr_seg_origin, p->lr_seg_origin.data(),
                        p->lr_seg_origin.size() * sizeof(int32_t), s);
        if (st == A2C_OK)
            st = upload((void **)&p->d_lr_chain_seg, p->lr_chain_seg.data(),
                        p->lr_chain_seg.size() * sizeof(int32_t), s);
        if (st == A2C_OK)
            st = upload((void **)&p->d_lr_piece_atom, p->lr_piece_atom.data(),
                        p->lr_piece_atom.size() * sizeof(int32_t), s);
        if (st == A2C_OK)
            st = upload((void **)&p->d_lr_piece_chain, p->lr_piece_chain.data(),
                        p->lr_piece_chain.size() * sizeof(int32_t), s);
    }
    if (st == A2C_OK) st = lrmsd_scratch_setup(dev);
    if (st == A2C_OK) {
        if (model == A2C_FULLATOM) fa_allow_large_lds();
        else bb_allow_large_lds();
    }
    if (st == A2C_OK) {
        st = default_schedules(p, s);
    }
    if (st != A2C_OK) {
        a2c_plan_destroy(p);
        return st;
    }
    *out = p;
    return A2C_OK;
}

a2c_status a2c_plan_sizes(const a2c_plan *p, int64_t *n_res, int64_t *n_atoms)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (n_res) *n_res = p->R;
    if (n_atoms) *n_atoms = p->A;
    return A2C_OK;
}

a2c_status a2c_plan_atom_offsets(const a2c_plan *p, int32_t *h_chain_atom_offsets,
                                 int32_t *h_res_atom_offsets)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (h_chain_atom_offsets)
        std::memcpy(h_chain_atom_offsets, p->chain_atom_off.data(),
                    p->chain_atom_off.size() * sizeof(int32_t));
    if (h_res_atom_offsets) {
        if (p->model == A2C_BACKBONE)
            for (int64_t r = 0; r <= p->R; ++r) h_res_atom_offsets[r] = (int32_t)(3 * r);
        else
            std::memcpy(h_res_atom_offsets, p->res_atom_off.data(),
                        p->res_atom_off.size() * sizeof(int32_t));
    }
    return A2C_OK;
}

a2c_status a2c_plan_keep_coords(const a2c_plan *p, int32_t *keep)
{
    if (!p || !keep) return fail(A2C_ERR_INVALID_ARG, "plan or keep is NULL");
    *keep = (uint64_t)p->A * 3 * sizeof(float) <= (uint64_t)p->mem_budget && p->mem_budget > 0
                ? 1 : 0;
    return A2C_OK;
}

a2c_status a2c_plan_workspace_bytes(const a2c_plan *p, int32_t v, size_t *bytes)
{
    if (!p || !bytes) return fail(A2C_ERR_INVALID_ARG, "plan or bytes is NULL");
    if (v == A2C_SCAN || v == A2C_SCAN_QUAT) *bytes = 0;
    else if (v == A2C_PLAIN) *bytes = (size_t)p->A * 12 * sizeof(float);
    else return fail(A2C_ERR_INVALID_ARG, "unknown variant");
    return A2C_OK;
}

a2c_status a2c_plan_set_schedule(a2c_plan *p, int32_t K, int32_t W, void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    const a2c_status sa = check_schedule_args(p, K, W);
    if (sa != A2C_OK) return sa;
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    return apply_schedule(p, K, W, (hipStream_t)stream);
}

a2c_status a2c_plan_set_adjoint_schedule(a2c_plan *p, int32_t K, int32_t W, void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    const a2c_status sa = check_schedule_args(p, K, W);
    if (sa != A2C_OK) return sa;
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    return set_sched(p, p->bs, K, W, (hipStream_t)stream);
}

a2c_status a2c_plan_set_forward_schedule(a2c_plan *p, int32_t K, int32_t W, void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    const a2c_status sa = check_forward_schedule_args(p, K, W);
    if (sa != A2C_OK) return sa;
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    return set_sched(p, p->fs, K, W, (hipStream_t)stream);
}

a2c_status a2c_plan_get_schedule(const a2c_plan *p, int32_t *K, int32_t *W, int32_t *n_tiles)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (K) *K = p->fs.K;
    if (W) *W = p->fs.W;
    if (n_tiles) *n_tiles = p->fs.n_tiles;
    return A2C_OK;
}

a2c_status a2c_plan_get_adjoint_schedule(const a2c_plan *p, int32_t *K, int32_t *W,
                                         int32_t *n_tiles)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (K) *K = p->bs.K;
    if (W) *W = p->bs.W;
    if (n_tiles) *n_tiles = p->bs.n_tiles;
    return A2C_OK;
}

a2c_status a2c_forward(a2c_plan *p, int32_t v, const float *d_angles, float *d_coords,
                       void *d_workspace, void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (v != A2C_SCAN && v != A2C_PLAIN && v != A2C_SCAN_QUAT)
        return fail(A2C_ERR_INVALID_ARG, "unknown variant");
    if (v == A2C_PLAIN && p->model != A2C_BACKBONE)
        return fail(A2C_ERR_UNSUPPORTED, "the plain form is the backbone comparison only");
    if (v == A2C_SCAN_QUAT && p->model != A2C_BACKBONE)
        return fail(A2C_ERR_UNSUPPORTED, "the quaternion scan state is a backbone comparison only");
    if (p->R == 0) return A2C_OK;
    if (!d_angles || !d_coords) return fail(A2C_ERR_INVALID_ARG, "NULL angles or coords");
    if (v == A2C_PLAIN && !d_workspace)
        return fail(A2C_ERR_WORKSPACE, "the plain form stores M_i in the workspace");
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (v == A2C_PLAIN) e = launch_bb_forward_plain(*p, d_angles, d_coords, (float *)d_workspace, s);
    else if (p->model == A2C_BACKBONE)
        e = launch_bb_forward_scan(*p, d_angles, d_coords, s, v == A2C_SCAN_QUAT);
    else e = launch_fa_forward_scan(*p, d_angles, d_coords, s);
    if (e != hipSuccess) return hip_fail(e, "forward launch");
    return A2C_OK;
}

a2c_status a2c_backward(a2c_plan *p, int32_t v, const float *d_angles, const float *d_coords,
                        const float *d_grad_coords, float *d_grad_angles, void *d_workspace,
                        void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (v == A2C_SCAN_QUAT)
        return fail(A2C_ERR_UNSUPPORTED, "the quaternion scan state is a forward comparison only");
    if (v != A2C_SCAN && v != A2C_PLAIN) return fail(A2C_ERR_INVALID_ARG, "unknown variant");
    if (v == A2C_PLAIN && p->model != A2C_BACKBONE)
        return fail(A2C_ERR_UNSUPPORTED, "the plain form is the backbone comparison only");
    if (p->R == 0) return A2C_OK;
    if (!d_grad_coords || !d_grad_angles)
        return fail(A2C_ERR_INVALID_ARG, "NULL grad_coords or grad_angles");
    if (!d_angles) return fail(A2C_ERR_INVALID_ARG, "NULL angles");
    if (v == A2C_PLAIN && !d_workspace)
        return fail(A2C_ERR_WORKSPACE, "the plain backward reads the M_i its forward stored");
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (v == A2C_PLAIN)
        e = launch_bb_backward_plain(*p, d_angles, d_grad_coords, d_grad_angles,
                                     (const float *)d_workspace, s);
    else if (p->model == A2C_BACKBONE)
        e = launch_bb_backward_scan(*p, d_angles, d_coords, d_grad_coords, d_grad_angles, s);
    else
        e = launch_fa_backward_scan(*p, d_angles, d_coords, d_grad_coords, d_grad_angles, s);
    if (e != hipSuccess) return hip_fail(e, "backward launch");
    return A2C_OK;
}

a2c_status a2c_mse_step(a2c_plan *p, const float *d_angles, const float *d_target,
                        float *d_coords, float *d_loss, float *d_grad_angles, void *stream)
{
    if (!p) return fail(A2C_ERR_INVALID_ARG, "plan is NULL");
    if (p->R == 0) {  // the loss of an empty batch is 0 (one fill kernel, capturable)
        if (!d_loss) return A2C_OK;
        if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
        const hipError_t e = launch_fill_zero(d_loss, 1, (hipStream_t)stream);
        return e == hipSuccess ? A2C_OK : hip_fail(e, "loss fill launch");
    }
    if (!d_angles || !d_target || !d_grad_angles)
        return fail(A2C_ERR_INVALID_ARG, "NULL angles, target or grad_angles");
    if (!check_device(p)) return fail(A2C_ERR_STATE, "current device is not the plan's device");
    hipStream_t s = (hipStream_t)stream;
    const hipError_t e =
        p->model == A2C_BACKBONE
            ? launch_bb_mse_step(*p, d_angles, d_target, d_coords, d_loss, d_grad_angles, s)
            : launch_fa_mse_step(*p, d_angles, d_target, d_coords, d_loss, d_grad_angles, s);
    if (e != hipSuccess) return hip_fail(e, "training step launch");
    return A2C_OK;
}

}  // extern "C"
