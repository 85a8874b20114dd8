// Internal layout shared by the host runtime and the HIP kernels of libexs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace exs {

constexpr int kWave = 64;
constexpr int kMaxAtoms = 128;   // bits of one exclusion / moving mask row
constexpr int kMaxRot = 32;
constexpr int kMaxTopK = 32;
constexpr int kMaxWavesPerWg = 8;
constexpr int kMaxThreadsPerWg = kMaxWavesPerWg * kWave;
constexpr int kXcds = 8;   // accelerator complex dies of an MI355X, each with its own L2

// Work queues of a persistent launch: the workgroups of XCD x start on queue x % n_queues and
// move on to the others once it is drained.  Three layouts of the order:
//  * one queue, longest first, for one pocket: what runs last is short.  (Cut into queues, the one of
//    the longest ligands ends in long ones too: 230 ligands of up to 90 atoms 1,377 us, 903 in one
//    queue; 1,000 of up to 60 3.13 and 2.93 ms.)
//  * spread: kXcds queues, contiguous pocket-major runs of equal cost, each longest first.  For
//    launches whose pockets hold fewer ligands each than the device has in flight: an XCD's
//    workgroups keep to one or two pockets (6,000 ligands over 5 pockets of 96^3 x 8, FP32: 15.3 ms,
//    15.8 pocket by pocket, 26.5 in one queue longest first).
//  * pocket-major: kPocketMajorQueues queues, each pocket by pocket, longest first within a
//    pocket, so that few pockets are in use at a time and their texel blocks stay in the L2s and
//    the shared last-level cache (4,000 ligands over 4 pockets of 128^3 x 8, BF16: 12.2 ms, 13.0 in
//    one such queue, 13.2 spread).
constexpr int kMaxWorkQueues = kXcds;
// The queues' counters lie a line apart: what workgroups ask of one line is served one after another,
// about 10 ns each.
constexpr int kQueueStride = 32;
constexpr int kQueueInts = kMaxWorkQueues * kQueueStride;
constexpr int kPocketMajorQueues = 2;
constexpr int kInflightWaves = 256 * 4 * 3;   // CUs x SIMDs x dock-kernel waves per SIMD
struct QueuePlan {
    int n_queues;
    bool pocket_major;
};
// Layout for n_ligands ligands over n_pockets distinct pockets, waves_per_ligand waves each
// (orientations / 64, whatever the launch's lanes: the threshold is an empirical one in that unit).
inline QueuePlan queue_plan(int64_t n_ligands, int n_pockets, int waves_per_ligand) {
    if (n_pockets <= 1) return {1, false};
    const int64_t inflight = kInflightWaves / (waves_per_ligand > 0 ? waves_per_ligand : 1);
    if (n_ligands >= inflight * n_pockets) return {kPocketMajorQueues, true};
    return {kXcds, false};
}

// Turn tables: for S in {8, 16, 32}, cos then sin of 2*pi*s/S at offset trig_offset(S).
constexpr int kTrigEntries = 2 * (8 + 16 + 32);
__host__ __device__ constexpr int trig_offset(int S) { return S == 8 ? 0 : (S == 16 ? 16 : 48); }

// cos(2 pi m / S) for 0 <= m <= S/4, FP64 values rounded to FP32 (RNE).  Every turn
// 2 pi s / S of the torsion sweep has cos and sin equal to +-qcos(m) for some m, so the
// unrolled sweep needs S/4 + 1 constants and the signs fold into FMA source modifiers.
// upload_trig_tables() checks these literals against the host's FP64 cos.
template <int S> __host__ __device__ __forceinline__ constexpr float qcos(int m);
template <> __host__ __device__ __forceinline__ constexpr float qcos<8>(int m) {
    return m == 0 ? 1.0f : (m == 1 ? 0x1.6a09e6p-1f : 0.0f);
}
template <> __host__ __device__ __forceinline__ constexpr float qcos<16>(int m) {
    return m == 0 ? 1.0f : m == 1 ? 0x1.d906bcp-1f : m == 2 ? 0x1.6a09e6p-1f
         : m == 3 ? 0x1.87de2ap-2f : 0.0f;
}
template <> __host__ __device__ __forceinline__ constexpr float qcos<32>(int m) {
    return m == 0 ? 1.0f : m == 1 ? 0x1.f6297cp-1f : m == 2 ? 0x1.d906bcp-1f
         : m == 3 ? 0x1.a9b662p-1f : m == 4 ? 0x1.6a09e6p-1f : m == 5 ? 0x1.1c73b4p-1f
         : m == 6 ? 0x1.87de2ap-2f : m == 7 ? 0x1.8f8b84p-3f : 0.0f;
}
// cos and sin of 2 pi s / S, 0 <= s < S, from the quarter-period table.
template <int S> __host__ __device__ __forceinline__ constexpr float kcos(int s) {
    constexpr int Q = S / 4;
    const int q = s / Q, r = s % Q;
    return q == 0 ? qcos<S>(r) : q == 1 ? -qcos<S>(Q - r) : q == 2 ? -qcos<S>(r) : qcos<S>(Q - r);
}
template <int S> __host__ __device__ __forceinline__ constexpr float ksin(int s) {
    constexpr int Q = S / 4;
    const int q = s / Q, r = s % Q;
    return q == 0 ? qcos<S>(Q - r) : q == 1 ? qcos<S>(r) : q == 2 ? -qcos<S>(Q - r) : -qcos<S>(r);
}

// One packed ligand (caller order).
struct LigInfo {
    int32_t atom_base;   // first atom in the packed atom arrays
    int32_t rot_base;    // first rotatable bond in the packed bond arrays
    int16_t n;           // atoms
    int16_t nrot;        // rotatable bonds
    int16_t pocket;      // index into the job's pocket table
    int16_t pad;
    float cost;          // relative search cost, for longest-first ordering
    int32_t pad2[3];
};
static_assert(sizeof(LigInfo) == 32, "LigInfo layout");

// One pocket as the kernels see it.
struct GridDesc {
    const void* tex;       // gather layout, one channel every chan_bytes: per node the four texels
                           // of its y-z square, 16 B in FP32, 8 B in BF16/FP16, x fastest
    const float* master;   // FP32 master texels [C][nz][ny][nx] (FP64 rescoring)
    int nx, ny, nz, channels;
    float ox, oy, oz, inv_h;   // origin and 1/spacing, FP32
    float cx, cy, cz, pad;     // pocket centre (grid centre), FP32
    float ux_hi, uy_hi, uz_hi, pad1;  // largest floats below N-1 per axis (grid-unit clamp)
    double h, dox, doy, doz;   // FP64 geometry for the rescoring
    double dcx, dcy, dcz, dpad;
    int32_t chan_bytes;        // bytes of one channel of the gather layout
    int32_t master_chan_bytes; // bytes of one FP32 channel
    int32_t storage;           // EXS_F32 / EXS_BF16 / EXS_F16
    int32_t tex_row, tex_slice;   // entries of a row and of a slice of the gather layout
    int32_t pad3;
};

// Serving: the results of one iteration's ligands in contiguous host memory (one record per
// ligand, then coordinates and torsion bytes at host-computed offsets).
struct ResultRec {
    float score;
    int32_t k;
    int32_t tau;
    int32_t pad;
    double score64;
};

// Dynamic LDS of a dock workgroup (byte offsets): the turn table, the ligand's topology (ref ..
// topk relative to lig), the waves' best (score, orientation), and per wave its poses, clash difference arrays, queue of crossing pairs and torsions
// (diff, queue, theta relative to the wave's part).  Sized by the launch's largest ligand: LDS decides how many waves fit on a CU.
struct DockLds {
    int32_t lig;
    int32_t ref, excl, rmask, ruv, mc, perm, perm_stride, e64, topk;
    int32_t rec;
    int32_t waves, wave_bytes, diff, queue, theta;
    int32_t total;
};
__host__ __device__ inline int lds_align(int x) { return (x + 15) & ~15; }
inline DockLds dock_lds(int n_max, int rot_max, int top_k, int waves, int lanes, int S) {
    DockLds d;
    const int no = kWave / lanes;
    int at = lds_align(2 * S * 4);
    d.lig = at;
    int p = 32;                                   // lig, n, nrot, pocket, atom_base, rot_base
    d.ref = p; p += 16 * n_max;
    d.excl = p; p += 16 * n_max;
    d.rmask = p; p += 16 * rot_max;
    d.e64 = p; p += lds_align(8 * top_k);
    d.topk = p; p += lds_align(4 * top_k);
    d.ruv = p; p += lds_align(4 * rot_max);
    d.mc = p; p += lds_align(4 * rot_max);
    d.perm = p;
    d.perm_stride = (n_max + 3) & ~3;
    p += lds_align(d.perm_stride * rot_max);
    at += p;
    d.rec = at; at += lds_align(8 * waves);
    d.waves = at;
    p = lds_align(12 * n_max * no);               // the poses (the FP64 ones of the top_k, 24 n_max, fit)
    d.diff = p; p += lds_align(2 * S * no);
    d.queue = p; p += 13 * kWave;
    d.theta = p; p += lds_align(rot_max * no);
    d.wave_bytes = p;
    d.total = at + waves * d.wave_bytes;
    return d;
}
constexpr size_t kMaxLdsBytes = 160 * 1024;   // gfx950 LDS per workgroup
constexpr int kDockStaticLds = 16;                      // the dock kernel's static words
constexpr int kDockLdsBytes = (int)kMaxLdsBytes - 256;   // dynamic LDS beside them
// Words in front of a scratch slot's poses: a part's best score, orientation and tau, then its
// torsions from word 4.
constexpr int kSlotHead = 4 + kMaxRot;

// Shape of a dock launch: lanes per orientation, waves of a workgroup, workgroups per ligand.
struct DockShape {
    int lanes = 4, waves = 1, parts = 1;
    bool pair = false;   // two waves search the same orientations: one looks up, one counts clashes
    DockLds lds{};
    int64_t slot_floats(int n_max) const { return kSlotHead + ((int64_t)waves + (parts > 1 ? 1 : 0)) * 3 * n_max; }
};
// What the shape of a launch is chosen by: its ligands, the largest one, and the mean work of one of
// their orientations (turns, offsets and the rest, in ligand_cost's units).
struct LaunchWork {
    int n_lig = 0, beside = 0;   // beside: ligands of another launch on the chip
    bool sorted = true;          // the ligands come longest first, in every queue
    int64_t n_atoms = 0;
    int n_max = 1, rot_max = 0;
    double turn = 0.0, offset = 0.0, rest = 0.0;
    double bonds = 0.0;          // of it the bonds': turns and clash pairs
    double steps = 0.0;          // bonds taken one after another: of every pass
};
DockShape dock_shape(const LaunchWork& w, int K, int S, int top_k, int cus);

// Sums over ligands from which the mean work follows for any search settings.
struct WorkSums {
    double ligands = 0, atoms = 0, square = 0, moving = 0, pairs = 0;   // square: n^2; moving, pairs: over the bonds
    double bonds = 0;
    void add(int n, const int16_t* m, int nrot) {
        ligands += 1;
        atoms += n;
        square += (double)n * n;
        bonds += nrot;
        for (int b = 0; b < nrot; ++b) {
            moving += m[b];
            pairs += (double)m[b] * (n - m[b]);
        }
    }
    void add(const WorkSums& o) {
        ligands += o.ligands;
        atoms += o.atoms;
        square += o.square;
        moving += o.moving;
        pairs += o.pairs;
        bonds += o.bonds;
    }
    LaunchWork mean(int S, int P, int T) const {
        LaunchWork w;
        const double per = ligands > 0 ? 1.0 / ligands : 0.0;
        w.turn = 40.0 * P * S * moving * per;
        w.offset = 40.0 * P * (T > 1 ? T : 0) * atoms * per;
        w.rest = (80.0 * atoms + 20.0 * (square + P * pairs)) * per;
        w.bonds = w.turn + 20.0 * P * pairs * per;
        w.steps = P * bonds * per;
        return w;
    }
};

// Everything one dock launch reads and writes.
struct DockArgs {
    // packed ligand batch
    const LigInfo* info;
    const float4* ref;        // [A] centred input coords, type in .w (int bits)
    const double* ref64;      // [A*3] centred input coords in FP64 (rescoring)
    const uint4* excl;        // [A] bit j: pair (i, j) excluded (bond distance <= 3, or i == j)
    const uint32_t* rot_uv;   // [R] u | v << 16, u on atom 0's side
    const uint4* rot_mask;    // [R] atoms that turn with the bond
    const int32_t* order;     // ligands in processing order (pocket-major, longest first within)
    int32_t n_order;          // ligands in this launch
    int32_t n_tiles;          // workgroups' worth of work: n_order times parts
    // pockets
    const GridDesc* grids;
    // search settings
    const float* rot32;       // [K][9] orientation matrices, row-major
    const double* rot64;      // [K][9]
    const int32_t* order_k;   // [K] the orientations in the order the chunks take them
    int32_t K, S, P, T;
    float step, cut2, pen, pad0;
    double step64, cut2_64, pen64;
    int32_t top_k;
    int32_t parts;            // workgroups that share a ligand's chunks
    int32_t n_max;            // atoms of the largest ligand in the launch
    int32_t persistent;
    DockLds lds;
    // scratch slots, one per workgroup (parts > 1: one per tile): kSlotHead words, with parts > 1
    // the part's pose [n_max][3], then [waves][n_max][3]
    float* scratch;
    int64_t slot_floats;
    int32_t* tile_counter;    // persistent launches: next tile of each queue [n_queues][kQueueStride]
    int32_t* done;            // parts > 1: finished parts of each position of `order`, zeroed
    // persistent launches: n_queues + 1 positions in `order`, queue q = [qb[q], qb[q+1]);
    // a workgroup takes tiles from queue (its XCD index mod n_queues) first, then from the
    // others.  Null, or n_queues = 1: one queue over the whole order.
    const int32_t* queue_bounds;
    int32_t n_queues;
    int32_t beside;           // persistent launches: another launch may hold the workgroups back
    // outputs (indexed by caller ligand / rotatable-bond index)
    float* orient_score;      // [L*K]
    uint8_t* orient_theta;    // [R*K], element (rot_base+b)*K + k
    int32_t* orient_tau;      // [L*K], tau packed as 3 signed bytes
    float* best_score;        // [L]
    int32_t* best_k;          // [L]
    float* best_coords;       // [A*3]
    uint8_t* best_theta;      // [R]
    int32_t* best_tau;        // [L]
    double* best_score64;     // [L]   (top_k > 0)
    int32_t* topk_k;          // [L*top_k]
    float* topk_score;        // [L*top_k] FP32 search score
    double* topk_score64;     // [L*top_k]
    uint8_t* topk_theta;      // [R*top_k], element (rot_base+b)*top_k + t
    int32_t* topk_tau;        // [L*top_k]
    // ranking of the final poses (rank_keep > 0)
    float rank_thr2;          // RMSD threshold squared (A^2)
    int32_t rank_keep;        // ranked poses kept per ligand
    int32_t* n_clusters;      // [L]
    int32_t* ranked;          // [L*rank_keep] orientation indices, leaders first
    float* final_xyz;         // [A*3][K] final pose of every orientation (rank_keep > 0)
    // second-stage rescoring of the ranked poses (rescore2 > 0; needs rank_keep > 0)
    int32_t rescore2;
    int32_t pad2;
    const uint32_t* rot_ac;   // [R] a | c << 16 (0xffff: none): dihedral neighbours of u and v
    double eps2, w2;          // contact well depth, torsion weight of the second-stage score
    double* score2;           // [L*rank_keep] second-stage score of each ranked pose
    int32_t* best2_k;         // [L] orientation of the lowest second-stage score
    double* best2;            // [L] that score
    // serving iterations (res_rec non-null): each ligand's finish also writes its result to the
    // iteration's result buffer (mapped host memory), at position j = res_slot[l]: the record
    // res_rec[j], coordinates from res_coords + 3 res_adst[j], torsion bytes from
    // res_theta + res_rdst[j]; no kernel runs after the search
    const int32_t* res_slot;  // [L] position of each ligand in its iteration's work list
    const int32_t* res_adst;  // [work list]
    const int32_t* res_rdst;  // [work list]
    ResultRec* res_rec;
    float* res_coords;
    uint8_t* res_theta;
};

// LDS words of a ranking block: a head of rank, state and score per pose, the leader bits, the
// list of uncovered poses and the waves' shares of it (to a multiple of 4 words), then the
// coordinates of 8 candidate leaders (rank_row_words rows each, n_max the launch's largest ligand).
constexpr int kRankWaves = 4;
constexpr int kRankRowBatch = 16;   // pose rows a sweep loads at once; a candidate's rows are padded to it
__host__ __device__ inline int rank_row_words(int n_max) {
    return (3 * n_max + kRankRowBatch - 1) / kRankRowBatch * kRankRowBatch;
}
__host__ __device__ inline int rank_head_words(int K) {
    return (4 * K + (K + 31) / 32 + kRankWaves + 2 + 3) & ~3;
}
__host__ __device__ inline int rank_lds_words(int K, int n_max) {
    return rank_head_words(K) + 8 * (rank_row_words(n_max) + 4);
}

// A ligand's topology in the LDS of the second-stage rescoring.
struct LigLds {
    float4 ref[kMaxAtoms];     // centred reference coordinates, type in .w
    uint4 excl[kMaxAtoms];     // exclusion rows
    uint4 rmask[kMaxRot];      // moving masks
    uint32_t ruv[kMaxRot];     // u | v << 16
    int32_t lig, n, nrot, pocket;
    int32_t atom_base, rot_base, pad0, pad1;
};

// Launchers (dock_misc.hip).
hipError_t launch_dock(const DockArgs& a, int storage, const DockShape& sh, int n_blocks, hipStream_t st);
// Gather layout of a pocket channel: entries of four texels (16 B in FP32, 8 B in 16 bits), entry
// (x, y, z) at z * slice + y * row + x, x < nx, y < ny-1, z < nz-1.
// The L1 serves a quad of lanes in one cycle unless two of them want the same bank of different
// lines (or more than two lines), and rows of whole lines put every y and z of one x in the same
// banks.  So rows and slices are padded to 6 and 3 entries past whole lines in FP32, to 12 and 9 in
// 16 bits: of all paddings these conflict least over the quads of the turns and offsets (counted on
// the CPU, cycles per quad, before and after: offsets 2.0 / 1.5 FP32, 2.0 / 1.4 16-bit; turns 2.3 /
// 1.9 and 2.9 / 2.0).  A grid that the padding would take past the limits of a channel's offsets
// goes without.
struct GatherLayout {
    int32_t row, slice;     // entries
    int64_t bytes;          // of a channel
};
inline GatherLayout gather_layout(int nx, int ny, int nz, int storage) {
    const int64_t eb = storage == 0 ? 16 : 8, line = 128 / eb;
    auto pad = [line](int64_t v, int64_t rest) { return v + (rest + line - v % line) % line; };
    const int64_t row = pad(nx, storage == 0 ? 6 : 12), slice = pad(row * (ny - 1), storage == 0 ? 3 : 9);
    const int64_t bytes = slice * (nz - 1) * eb;
    if (slice < (int64_t)1 << 24 && bytes <= INT32_MAX) return {(int32_t)row, (int32_t)slice, bytes};
    const int64_t plain = (int64_t)nx * (ny - 1);
    return {nx, (int32_t)plain, plain * (nz - 1) * eb};
}
hipError_t launch_expand_grid(const float* src, void* dst, int nx, int ny, int nz, int channels,
                              int storage, const GatherLayout& g, hipStream_t st);
// Gather probe over the pocket `gd` (device pointer) in `storage`: blocks x 256 lanes, nb
// (8, 16 or 32) independent lookups per round.
hipError_t launch_gather_probe(const GridDesc* gd, int storage, int nb, int64_t blocks, int per_lane,
                               float half, float walk, uint32_t seed, float* out, hipStream_t st);
// Unfolding of `n_lig` packed ligands in place (ref, ref64), S turns per bond, `passes` passes;
// turns [passes * R] receives the kept turns (or null).
// The waves take the ligands in `order` (a permutation of 0..n_lig-1, longest first).
hipError_t launch_unfold(const LigInfo* info, float4* ref, double* ref64, const uint32_t* rot_uv,
                         const uint4* rot_mask, int32_t* turns, const int32_t* order, int n_lig, int R,
                         int S, int passes, hipStream_t st);
// Ranking of the final poses of `n_lig` ligands (rank_keep > 0), one block per ligand, the
// ligands taken in `order` (a permutation of 0..n_lig-1, longest first).
hipError_t launch_rank(const DockArgs& a, int n_lig, int64_t n_atoms, const int32_t* order, hipStream_t st);
// Second-stage rescoring of the ranked poses of `n_lig` ligands, one block of waves per ligand,
// the ligands taken in `order`.
hipError_t launch_rescore2(const DockArgs& a, int n_lig, const int32_t* order, hipStream_t st);
hipError_t launch_zero_ints(int* p, int n, hipStream_t st);
// dst[0..n) = src[0..n), zero[0..nz) = 0 and slot[src[lig + j]] = j for j < n_lig, one kernel;
// src may be mapped host memory (a kernel reads it over the bus, so no copy call is queued).
hipError_t launch_stage_ints(const int32_t* src, int32_t* dst, int n, int* zero, int nz, int lig,
                             int n_lig, int32_t* slot, hipStream_t st);
// *flag |= 1 if a texel is not finite, |= 2 if one overflows the 16-bit storage (storage 1, 2).
hipError_t launch_check_texels(const float* v, int64_t count, int storage, int* flag, hipStream_t st);
// K orientation matrices [K][9] (row-major), FP32 and (unless r64 is null) FP64, and the order in
// which the chunks take the orientations [K]; clears zero[0 .. n_zero) (launch counters) as well.
hipError_t launch_orientation_table(int K, float* r32, double* r64, int32_t* order_k, int32_t* zero, int n_zero,
                                    hipStream_t st);
hipError_t upload_trig_tables();
const void* dock_kernel_fn(int storage, int S, int lanes);

}  // namespace exs
