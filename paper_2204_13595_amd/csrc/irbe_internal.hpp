// Internal declarations of the HIP implementation: the handle, the launch
// helpers and the kernel entry points shared between the translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "irbe.h"

namespace irbe {

// Error-word bits set by kernels and read back at the next waiting call
// (ERR_SHELL_ROW: no error, the next build is to take 32-bit shell entries).
enum : uint32_t { ERR_NONFINITE = 1u, ERR_CORE_CAP = 2u, ERR_SHELL_CAP = 4u, ERR_SHELL_ROW = 8u };

// Shell lists as masks. The list build takes blocks of up to 32 consecutive
// atoms of one cell row (slot_of: an atom's block); a block's candidates, in
// canonical order, fill words of 32 in half words of 16 (words[2 (slot * cap + w)
// + q]: the sorted index of the first candidate of half q of word w, the others
// follow it; nw[slot] words), and S(i) is
// one bit per candidate (mask[i * cap + w], zero up to the next multiple of four
// words): member r is the (r + 1)-th set bit.
struct ShellMasks {
    const uint32_t* mask;
    const int32_t* words;
    const int32_t* nw;
    const int32_t* slot_of;
    int cap;  // words per row, a multiple of 4, at most kMaskMaxWords
};
constexpr int kMaskMaxWords = 2048;
constexpr int kMaskTableWords = 256;  // words per row up to which a wavefront keeps an atom's masks and bases in LDS

constexpr int kBlock = 256;          // threads per block of the per-atom kernels
constexpr int kReduceBlock = 256;    // threads of the deterministic final reductions
constexpr int kPairPartials = 16;    // FP64 values per block of the pair kernel
constexpr int kLjArgTypes = 4;       // LJ tables of up to this many types are kernel arguments
constexpr int kMaxTypesGrad = 4;     // LJ parameter gradients: n_types <= 4
// atoms per wavefront in the cooperative pair kernels: the adjoint, the forward
// kernel with list-drawn batches, and the forward kernel with stencil sampling
constexpr int kAtomsPerWave = 8;
constexpr int kAtomsPerWaveList = 4;   // full lists
constexpr int kAtomsPerWaveSplit = 8;  // split lists (the optimum with compact shell lists; the same with
                                       // 32-bit ones, so that the per-block sums and results do not change)
constexpr int kAtomsPerWaveStencil = 16;
// Shell-adjoint transpose: scatter records staged per block in LDS, then
// bucketed by destination cell row (y, z) and reduced per row.
constexpr int kBucketRowLds = 2048;  // atoms of a row accumulated in LDS (the rest: device atomics)
constexpr int kBucketRecF = 1200;    // staged records per block (budget), FP32
constexpr int kBucketRecD = 600;     // staged records per block (budget), FP64
constexpr int kBucketRecMaxF = 2048; // staged records per block (LDS limit), FP32
constexpr int kBucketRecMaxD = 1024; // staged records per block (LDS limit), FP64
constexpr int kBucketMaxKeys = 256;  // (source row, destination row) keys per block
constexpr int kBucketSlack = 64;     // records of spare capacity per destination row

// Per-k constants of the force kernels: k (3), then coefficient products.
template <typename real>
struct KForce {
    real kx, ky, kz;
    real a;  // ke c_l Im(rho_l)
    real b;  // ke c_l Re(rho_l)
    real pad0, pad1, pad2;
};

template <typename real>
struct KAdj {
    real kx, ky, kz;
    real ar, ai;  // ke c_l A_l
    real rr, ri;  // ke c_l rho_l
    real pad;
};

// LJ pair table entry: force 48 eps s^12, 24 eps s^6; energy 4 eps s^12, 4 eps s^6;
// the term acts at r^2 < rc2 (the largest finite value without a cutoff) and its
// energy is lowered by esh there (the shifted-truncated form).
template <typename real>
struct LJ {
    real a12, b6, rc2, esh, c12, c6;
};

struct Geometry {
    int32_t n_c = 0;
    int32_t reach = 0;      // R: shell stencil half-width in cells
    int32_t lo = 0, hi = 0; // shell stencil offsets per axis, inclusive
    uint64_t t_core = 0, t_shell = 0;  // membership at force time: r <= r_core, r <= r_shell
    // list thresholds: C(i) D^2 <= tl_core, S(i) tl_lo < D^2 <= tl_shell (the
    // above without a skin; with one, r_core + skin, r_core - skin, r_shell + skin)
    uint64_t tl_core = 0, tl_lo = 0, tl_shell = 0;
    bool skin = false;      // lists built with a skin: entries tested at force time
    double inv_l = 0.0;
    double quantum = 0.0;   // L / 2^32
    int64_t n_cells = 0;
};

// What a list build produces: split core and shell lists, one full list, the
// core list alone (the shell batch of stencil sampling is drawn from the
// stencil's cells), or split lists with a skin, where S(i) starts at its own
// threshold below C(i)'s end (the two lists overlap).
enum { kListsSplit = 0, kListsFull = 1, kListsCoreOnly = 2, kListsSplitSkin = 3 };

// Arguments of k_list_blocks.
struct ListBlockArgs {
    int n_c, lo, span, G, cap_core, cap_shell;
    uint64_t t_out, t_in, t_lo;      // squared radii (quanta): outer list, C(i), inner end of S(i) with a skin
    float tu_out, tu_in, tu_lo;      // the same in the units of the test
    float unit;                      // units per quantum
    float inv_span;                  // 1 / span
    float r_in;                      // C(i)'s radius in units, with a margin
    float tf_hi;                     // t_out with the margin of the row pruning
    float band_valu;                 // error bound of the vector-unit distances
    const uint4* spos;
    const int32_t* cell_start;
    const uint32_t* bound;
    const int32_t* blk_start;        // first atom + 1 of every block slot (0: unused)
    const int2* sxr;
    const int32_t* xidx;             // excluded partners (caller ids) and the caller ids' sorted indices
    const int32_t* rank;
    const int32_t* smol;             // molecule ids
    int32_t* sxidx;                  // the partners' sorted indices, written by the build (not with ids)
    int32_t *core, *ncore, *shell, *nshell, *maxcnt;
    uint32_t* err;
    // shell lists as masks (ShellMasks)
    uint32_t* mask;
    int32_t *words, *nw, *slot_of;
    int cap_words;
    int max_row;                     // candidates of a stencil row beyond which ERR_SHELL_ROW is set
};

// Stencil and segments of the block list build: segments of G cells of a cell
// row, gpr per row; narrow: the stencil does not wrap the box.
struct ListBlockShape {
    int reach, lo, span, G, gpr;
    bool narrow;
};

}  // namespace irbe

struct irbe_ctx {
    irbe_config cfg{};
    hipStream_t stream = nullptr;
    int device = 0;
    bool fp64 = false;
    bool full_list = false;
    bool stencil = false;             // shell batch drawn from the stencil's cells (no shell list)
    size_t real_size = 4;
    irbe::Geometry geo;
    std::string last_error;

    // k table
    int32_t kM = 0;
    double kH = 0.0, kS = 0.0;

    // state
    bool have_system = false;
    bool have_lists = false;
    int32_t cap_core = 0, cap_shell = 0;
    // longest core / shell (or stencil) list of the last build whose lengths the
    // host has seen: exact after a waiting build, possibly stale after the
    // asynchronous ones (which only read them back when they have completed), so
    // only choices of speed use them; sizes that must hold every list use
    // shell_bound()
    int32_t max_core = 0, max_shell = 0;
    bool lists_sized = false;         // a waiting build has sized the list rows
    int32_t* chk_host = nullptr;      // pinned [4]: error word, max core, max shell, max mask words of the last build
    hipEvent_t chk_event = nullptr;   // recorded after the copy into chk_host
    bool chk_pending = false;         // chk_host awaits a completed copy
    // Upper bound on every atom's shell (or full, or stencil) list length.
    int32_t shell_bound() const { return stencil ? max_shell : cap_shell; }
    uint64_t last_force_step = 0;
    bool have_force_step = false;
    std::vector<double> lj_sigma_host, lj_eps_host;

    // device memory, all owned by the handle
    uint32_t* err = nullptr;          // error word
    int32_t* maxcnt = nullptr;        // [3] max core / shell count and mask words of the last build
    uint64_t* ktab = nullptr;         // [2M+1]
    void* q_orig = nullptr;           // real[N]
    int32_t* type_orig = nullptr;     // [N]
    int32_t* mol_orig = nullptr;      // [N]
    void* lj = nullptr;               // LJ<real>[n_t^2]
    void* lj_raw = nullptr;           // real[2 n_t^2]: sigma, eps
    int32_t* xoff = nullptr;          // [N+1] exclusion partners per atom (caller ids)
    int32_t* xidx = nullptr;
    int32_t* sxidx = nullptr;         // [n_excl] xidx entries as sorted indices (rebuilt with the cells)
    int2* sxr = nullptr;              // [N] sorted atom's range (first, count) in sxidx
    int64_t n_excl = 0;
    int32_t max_excl = 0;             // most excluded partners of an atom
    double* sumq2 = nullptr;          // [1]
    double* q2part = nullptr;

    uint4* sq = nullptr;              // [N] quantized position + cell, caller order
    int32_t* cell_count = nullptr;    // [n_cells]
    int32_t* cell_start = nullptr;    // [n_cells + 1]
    uint32_t* cell_bound = nullptr;   // [n_c + 1] first fixed-point coordinate of each cell row/column
    std::vector<int32_t*> scan_levels;
    std::vector<int64_t> scan_sizes;
    int32_t* blk_start = nullptr;     // [list_block_slots] first atom + 1 of the blocks of the list build
    int32_t* perm = nullptr;          // [N] sorted -> caller id
    int32_t* rank = nullptr;          // [N] caller id -> sorted
    uint4* spos = nullptr;            // [N] sorted {sx, sy, sz, type} (FP32: at the last build)
    uint4* spk = nullptr;             // [N] sorted packed records of the list build
    int32_t* brow = nullptr;          // [N] cell (z << 16 | y) at the build of each sorted atom (lists with a skin)
    uint4* spq = nullptr;             // [N] sorted {sx, sy, sz, FP32 charge with the type in its low 4 bits}
                                      //     (FP32 evaluations; the FP64 ones read spos and sq_r)
    void* sq_r = nullptr;             // real[N] sorted charges (FP32: at the last build)
    int32_t* smol = nullptr;          // [N] sorted molecule ids

    int32_t* core = nullptr;          // [N * cap_core]
    int32_t* ncore = nullptr;         // [N]
    int32_t* shell = nullptr;         // [N * cap_shell] sorted indices, or (masks) [N * cap_words] mask words
    bool masks = false;               // the shell rows are allocated as masks (ShellMasks)
    bool masks_ok = true;             // cleared for good once a build found a crowded stencil row or a block of too many words
    int32_t cap_words = 0;            // words per mask row
    int32_t* blk_words = nullptr;     // [2 * list_block_slots * cap_words] first candidate of the blocks' half words
    int32_t* blk_nw = nullptr;        // [list_block_slots] words of the blocks
    int32_t* slot_of = nullptr;       // [N] block of each sorted atom
    irbe::ShellMasks shell_masks() const { return {(const uint32_t*)shell, blk_words, blk_nw, slot_of, cap_words}; }
    int32_t* nshell = nullptr;        // [N]

    void* fsr = nullptr;              // real[3N] sorted short-range (+ excluded-pair) force
    double* pair_part = nullptr;      // [nb * kPairPartials]
    double* fcorr = nullptr;          // [3]
    double* pair_slices = nullptr;    // [256 * 12] first-stage sums of pair_part
    double* ev_pair = nullptr;        // [kPairPartials] reduced pair partials

    int4* kvec = nullptr;             // [P]
    double* kcoef = nullptr;          // [4P]: kx, ky, kz, c_l
    double* rho_part = nullptr;       // [2 * P * nb_rho] (x2 for the adjoint A)
    bool rho_wide = false;            // structure factors in the widest shape always (fewest partial sums)
    double* rho = nullptr;            // [2P]
    double* Avec = nullptr;           // [2P]
    void* kforce = nullptr;           // KForce<real>[P]
    void* kadj = nullptr;             // KAdj<real>[P]

    void* gs = nullptr;               // real[3N] sorted dL/dF
    double* gpart = nullptr;          // [nb * 3]
    double* gmean = nullptr;          // [3]
    void* gself = nullptr;            // real[3N]
    void* gscat = nullptr;            // real[3N]
    void* gqself = nullptr;           // real[N]
    void* gqscat = nullptr;           // real[N]
    double* ljpart = nullptr;         // [nb * 2 * kMaxTypesGrad^2]
    double* lj_slices = nullptr;      // [256 * 2 * kMaxTypesGrad^2] first-stage sums of ljpart
    int64_t adj_nb = 0;               // blocks of the last pair-adjoint launch
    int64_t pair_nb = 0;              // blocks of the last pair-force launch
    int64_t part_blocks = 0;          // capacity (blocks) of pair_part and ljpart
    unsigned long long* bk_cursor = nullptr;  // [2 n_c^2] records reserved per destination row, then max |record|
    void* bk_c = nullptr;             // real[4 * bk_total] shell-adjoint records: dL/dr_j (3), dL/dq_j
    uint16_t* bk_j = nullptr;         // [bk_total] record's atom, relative to its row's first atom
    int64_t bk_total = 0;             // allocated records
    unsigned long long* adj_atomics = nullptr;  // [1] shell-adjoint records of the last backward added by atomics
    bool adj_all_atomic = false;      // the last backward added every shell-adjoint record by atomics
    uint16_t* ranks = nullptr;        // [N * p_stride] shell batch ranks of the current step
    int32_t* batch_j = nullptr;       // [N * p_stride] the drawn atoms (sorted index) of the current ranks (with
                                      // stencil sampling -1: i or i's molecule), for the adjoint and read-back:
                                      // written by the forward for the backward that follows it, or decoded
                                      // (stencil ranks, compact shell lists); allocated on first use
    bool batch_j_valid = false;       // batch_j holds the decode of the current ranks
    bool batch_j_fwd = false;         // ... written by a forward (not by a decode for the backward)
    bool keep_batch = false;          // the next forward writes batch_j (the last forward had a backward)
    bool fwd_pending = false;         // a forward ran and no backward has followed it yet
    bool adj_used_batch = false;      // the last backward read batch_j instead of the ranks and shell rows
    int32_t* scell = nullptr;         // [N] stencil sampling: cell of each sorted atom at the last build
    uint32_t* draw_bits = nullptr;    // Floyd bitmaps in device memory for lists too long for LDS
    size_t draw_bits_words = 0;
    int32_t p_stride = 0;
    bool ranks_valid = false;         // ranks hold the draw of ranks_step for the current lists
    uint64_t ranks_step = 0;

    // per-stage event timing (irbe_enable_timing)
    bool timing = false;
    struct Pending {
        int stage;
        hipEvent_t start, stop;
    };
    std::vector<Pending> pending;
    hipEvent_t open_start = nullptr;
    double stage_ms[IRBE_N_STAGES] = {};
    int64_t stage_n[IRBE_N_STAGES] = {};

    std::vector<void*> owned;
};

namespace irbe {

int64_t blocks_for(int64_t n, int block);
int64_t rho_blocks(const irbe_ctx* h);

// Launchers (all on the handle's stream). Each returns the HIP status of the launch.
hipError_t launch_fill_i32(hipStream_t s, int32_t* p, int32_t v, int64_t n);
hipError_t launch_fill_bytes0(hipStream_t s, void* p, size_t bytes);
hipError_t launch_bin(irbe_ctx* h, const void* pos);
// Positions and charges of a force evaluation, and the k-vectors of `step`.
hipError_t launch_requantize(irbe_ctx* h, const void* pos, uint64_t step);
hipError_t launch_build_lists(irbe_ctx* h);
// Mean atoms per cell below which the list build takes one lane per atom. Build + forces
// (100 draws), lanes against blocks, 400,000 atoms: 1.3 per cell 314 + 182 and 336 + 296 us,
// 2: 365 + 271 and 318 + 372, 3: 476 + 293 and 321 + 372, 4: 544 + 356 and 317 + 374, 8:
// 724 + 463 and 325 + 378; full lists, 3: 436 + 198 and 488 + 198, 5: 579 + 291 and 530 + 283.
// The lanes' lists of indices make the cheaper forces, which counts where lists are kept; the
// blocks build small boxes faster at any density (30,000 atoms, 3: 235 + 37 and 54 + 46).
constexpr double kLaneMaxPerCell = 4.0;
// True when it does (k_build_lists_lanes); else the blocks below.
bool lists_by_lanes(const irbe_ctx* h);
// The block form of the list build (k_list_blocks) and the block slots it takes.
hipError_t launch_list_blocks(irbe_ctx* h);
// Most excluded partners of an atom up to which the build clears them from its masks one
// by one (and writes their sorted indices on the way); beyond, by molecule ids (and the
// indices in a launch of their own). One by one against ids, build of 96,000 atoms in
// molecules of 3: 138 and 189 us, of 100: 196 and 215, of 200: 269 and 254, of 400: 470
// and 382, of 4,000: 3,932 and 1,678.
constexpr int kPartnersMost = 200;
bool exclusions_by_id(const irbe_ctx* h);
ListBlockShape list_block_shape(const Geometry& geo, bool core_only);
int64_t list_block_slots(const Geometry& geo, bool core_only, int64_t n);
hipError_t launch_rho(irbe_ctx* h, const void* grad, bool with_adjoint);
hipError_t launch_pair_forces(irbe_ctx* h, uint64_t step, bool ev);
// True when the shell batch draw of the current lists keeps its Floyd bitmaps in
// LDS (lists of at most 16,384 entries); false when it needs device memory.
bool draw_bitmaps_in_lds(const irbe_ctx* h);
hipError_t launch_pair_reduce(irbe_ctx* h, bool ev);
hipError_t launch_kspace_forces(irbe_ctx* h, void* force);
hipError_t launch_energy_finalize(irbe_ctx* h, double* ev);
hipError_t launch_sum_q2(irbe_ctx* h);
template <typename real>
hipError_t launch_store_lj(irbe_ctx* h, const LJ<real>* tab, const real* raw);
hipError_t launch_gather_grad(irbe_ctx* h, const void* grad);
hipError_t launch_pair_adjoint(irbe_ctx* h, uint64_t step, bool want_q, bool want_lj);
// Grow the shell-adjoint record buckets to hold `records` records.
hipError_t ensure_buckets(irbe_ctx* h, int64_t records);
// Stencil sampling: allocate the read-back array of the decoded batch, and fill it.
hipError_t ensure_batch_atoms(irbe_ctx* h);
// Words per mask row that this handle's shell lists take (an estimate with a
// margin), 0 when they are stored as 32-bit indices.
int mask_words_wanted(const irbe_ctx* h);
// Whether mask rows of `words` words, more than kMaskTableWords, are preferred to 32-bit indices.
bool long_masks(const irbe_ctx* h, double words);
// Device-memory Floyd bitmaps of at least `words` 32-bit words.
hipError_t ensure_draw_bits(irbe_ctx* h, size_t words);
hipError_t launch_stencil_decode(irbe_ctx* h);
hipError_t launch_kspace_adjoint(irbe_ctx* h, const void* grad, void* grad_pos, void* grad_q, double* grad_lj);

}  // namespace irbe
