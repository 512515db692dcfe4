// Internal data structures shared by the host side and the gfx950 kernels of
// libislf.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/islf.h"

namespace islf {

constexpr int kBlock = 256;          // threads per workgroup of the update kernels
constexpr int kAccSlots = 64;        // spread of the per-sweep partial-sum atomics
constexpr int kClasses = 4;          // bulk, x = 0, x = Lx-1, one-layer film
constexpr int kThrPerClass = 16;     // index u*8 + cnt, cnt in 0..6
constexpr int kThrEntries = kClasses * kThrPerClass;
constexpr int kPadEntry = kThrEntries - 1;   // class 3, u = 1, cnt = 7: never a real site
constexpr int kMaxMarch = 256;       // x planes one thread may march through per entry
constexpr int kNoAllocMaxReps = 8192;   // live replicas islf_means_noalloc serves per call

// One item of work for one replica.  j counts 8-byte columns of one
// sublattice row (int8 format: 8 sites) or 32-bit words of one sublattice
// row (bit-packed: 32 sites).
// Main tile (kind 0, rows 2 .. Ly-2): a box of rows/columns starting at
// (x0, y0, j0) whose extent is the replica's tile shape, or (linear tile
// shape, i8_tj = 0) the columns [y0, j0) of a plane's main rows in row-major
// order, marched through nsteps x planes from x0 (a launch plan may cut a
// tile into pieces along x).
// Seam-slab tile (kind 1, rows Ly-1, 0, 1): x0 = first x pair p (planes p and
// Lx-1-p), y0 = number of consecutive pairs, j0 = first column,
// nsteps = number of columns.
enum { ITEM_MAIN = 0, ITEM_SLAB = 1 };
struct Entry {
    int32_t rep, x0, y0, j0;
    int32_t nsteps, kind;
};

// Launch kinds of a run of sweeps and their flags.
enum { KIND_A = 0, KIND_B = 1, KIND_F = 2 };
enum { FLAG_PREV = 1, FLAG_FOLD = 2 };   // A: do the previous sweep's phase 3; B: fold its record

// Read-only description of a replica as the kernels see it.
struct RepDesc {
    uint8_t *spins;        // int8 format: byte 1 = up, 0 = down; rows of RB = 2*Hp bytes (even z, odd z)
                           // bit-packed: rows of 2*Wq uint32 words (even z, odd z)
    islf_obs *rec;         // ring of cap per-sweep records
    long long *acc;        // 2 x kAccSlots x 4 partial sums (double-buffered by t & 1)
    uint64_t thr[kThrEntries];  // acceptance thresholds, index class*16 + u*8 + cnt
    uint32_t thr_m1[kThrEntries];  // thr - 1 (accept iff u <= thr_m1) where thr >= 1
    int32_t dpack[kThrEntries];    // change of (B, M) on a flip: dB + 65536 * dM
    uint64_t never_mask;           // bit i set when thr[i] == 0 (no draw can accept)
    uint32_t thr_q[4];             // bulk class without a bulk field: thr - 1 by aligned neighbours <= 3, 4, 5, 6
    int32_t sym;                   // 1: the bulk class depends on that number alone (thr_q holds it)
    int32_t Lx, Ly, Lz;
    int32_t C;             // Philox groups of 8 consecutive z per row, ceil(Lz/8)
    int32_t K;             // int8 8-byte columns per sublattice row, ceil(Lz/16)
    int32_t Hp;            // int8 bytes per sublattice row, 8*K
    int32_t RB;            // int8 row stride in bytes, 2*Hp
    int32_t Wq;            // bit-packed words per sublattice row, ceil(Lz/64)
    int32_t seam_reflect;  // 1: the y seam maps x -> Lx-1-x
    int32_t seam_invert;   // 1: the y seam carries eps = -1
    uint32_t key0, key1, replica, cap;
    int32_t fmt;                   // islf_spin_format
    int32_t i8_tj, i8_ty, i8_mx;   // main tiles: columns x rows per workgroup (0 x 0: linear), x planes marched
    double J, H, h1, hn;           // for energies (Eq. 1)
};

// Mutable per-replica state (device memory).
struct RepState {
    long long cur[4];      // observables after the last completed sweep
    uint32_t t;            // completed sweeps
    uint32_t live;
    uint32_t pad_[2];
};

// Persistent-kernel synchronisation words (device memory, zero-initialised).
// Two-level grid barrier state.  Blocks arrive at their group's counter; the
// last arrival of a group arrives at the top counter, waits for all groups,
// then bumps its group's release counter, which the group's other blocks
// poll.  Every counter only changes through read-modify-write atomics and is
// re-zeroed by a fill kernel before each persistent launch; each sits on its
// own 128-byte line.
// 256 blocks per group (3 to 5 groups at the usual grids) measured best:
// 2-5% over 32, 64 or one flat group of 1024
constexpr int kBarrierGroup = 256;    // blocks per group
constexpr int kMaxGroups = 16;        // up to 4096 blocks
struct SyncLine {
    unsigned long long v;
    unsigned long long pad_[15];
};
struct GridSync {
    SyncLine top;
    SyncLine error;
    SyncLine arrive[kMaxGroups];
    SyncLine release[kMaxGroups];
};

// Team form of the persistent kernel: every workgroup serves one replica
// (its team), and a team's workgroups meet at a barrier of their own (an
// arrival and a release counter per replica slot, each on its own line,
// re-zeroed before each launch), so replicas do not wait for each other.
struct TeamInfo {
    int32_t rep;    // replica slot
    int32_t rank;   // 0 .. size-1 inside the team (rank 0 folds the records)
    int32_t size;   // workgroups of the team
    int32_t pad_;
};

// ---------------------------------------------------------------------------
// Resident form (islf_resident.hip): a launch keeps its replicas' spins in
// LDS, one bit per site, for all of its sweeps.
// ---------------------------------------------------------------------------
constexpr int kResThreads = 1024;      // threads per workgroup: 4 waves per SIMD, one workgroup per CU
constexpr int kResMaxSweeps = 256;     // sweeps one launch may run
constexpr int kResStaticLds = 11392;    // LDS bytes beside the lattice: pair tables, thresholds, control words
constexpr int kResFineChunk = 16;       // words of a chunk in the fine form
enum { RES_WORDS, RES_GROUPS, RES_FINE };   // how a launch's words go to lanes: see k_resident
constexpr int kSmallTasks = 2;         // four-site groups a lane of the small form may hold per phase

// Tables of a share, as the host writes them: its planes in the order of
// update (those sent to x neighbours first, free surfaces last) and its rows
// (by row set).  Slots are positions in LDS: two runs of planes, each with a
// halo plane on both sides (one run: the whole film or the middle).
enum { PL_ODD = 1, PL_X0 = 2, PL_XL = 4, PL_SEND = 16 };   // x odd; x = 0; x = Lx-1; sent to outer j = 0, 1, inner j = 0, 1
struct ResPlane {
    int16_t slot, x, mirror, flags;   // mirror: slot of plane Lx-1-x
};
enum { RW_ODD = 1, RW_LAST = 2, RW_ROW0 = 4, RW_DOWN = 8, RW_UP = 16 };   // y odd; y = Ly-1; y = 0; sent down, up
struct ResRow {
    int32_t y;
    int16_t lr, flags;
};
// A row set: entries r0 .. r0 + n - 1 of the row table.
struct ResRows {
    int32_t r0, n;
    uint32_t m, m_w;              // ceil(2^32 / d) of d = n and of d = n * whole words of a row
    int32_t whole, part;          // chunks of whole words, of partial last words
    int32_t seam;                 // holds row y = 0 or Ly-1
};
enum { RES_EDGE = 0, RES_SEAM = 1, RES_INNER = 2, RES_ROW0 = 3 };
// A stage of a sweep ends with a workgroup barrier.  It updates chunks
// [c0, c1) of up to three row sets (whole words are numbered before partial
// ones) and takes in the neighbours' mail of one or two phases.
struct ResPart {
    int16_t set, phase;
    int32_t c0, c1;
};
struct ResStage {
    ResPart part[3];
    int32_t mail, mail_row0;      // phase 0 or 1 of the main rows / phase 2 or 3 of row 0 taken in, -1 none
};
enum { HAS_Y = 1, HAS_OUTER = 2, HAS_INNER = 4 };   // neighbours of a share

// One workgroup's share of one replica: R consecutive rows of the y ring
// starting at row y0 (all z) in planes xa .. xa+n1-1 and their mirror images
// (n2 = n1), or in the middle planes xa .. Lx-1-xa (n2 = 0; all planes when
// xa = 0).  A replica's P shares form a cluster.  Planes come in mirrored
// pairs and the shares that hold row 0 also hold rows Ly-1 and 1, so that the
// y seam joins sites of one share whatever the boundary, and only row 0's own
// x neighbours sit in other shares during phases 2 and 3.  Local rows are
// 1 .. R; local rows 0 and R+1 and the halo planes are copies of the
// neighbouring shares' edges, or 0 beyond a free surface.
struct ResJob {
    int32_t rep, P;
    int32_t id;                   // its slot in the per-sweep sums (a replica's shares are consecutive)
    int32_t y0, R;
    int32_t ls, lr0;              // local rows of y = Ly-1 and y = 0 (0: not in this share)
    int32_t xa, n1, n2;
    int32_t has;                  // HAS_*
    int32_t planes, rows;         // offsets of its tables
    int32_t n_edge, n_head, n_tail;   // planes sent to x neighbours; surface planes among the first / at the end
    ResRows set[4];               // edge rows (sent to the y neighbours), rows Ly-1 and 1 beside row 0 (where they
                                  // are no edge rows), interior rows, and row 0 (phases 2 and 3)
    int32_t stages;               // 2, or 4 in a share with row 0
    ResStage stage[4];
    int32_t Wf, ng;               // whole words of a sublattice row; 4-site groups of a partial last word
    uint32_t m_c;                 // ceil(2^32 / d) of d = 4-site groups of a row,
    uint32_t m_q, m_f;            // of d = words of a row, of d = R * words of a row
    // mailboxes (64-bit words).  This share's: two slots (by phase & 1) of
    // `slot` words, the faces it has one after the other: y from below and
    // from above (plane, word), x from the outer share (run of lower x, of
    // upper x) and from the inner one (local row - 1, word).  The neighbours'
    // faces that it fills: out_y below, above; out_x outer, inner.
    uint32_t in, slot, out_y[2], out_x[2];
};
// A replica of a resident launch and its jobs job0 .. job0 + P - 1.
struct ResRep {
    int32_t rep, job0, P, pad_;
};
// Launch state of the resident form (device memory, zero-initialised; the
// last workgroup of each closing kernel resets it).
struct ResSync {
    unsigned int count;    // cluster workgroups that have started
    unsigned int pad0_[31];
    unsigned int state;    // RES_WAIT, RES_GO (all are resident) or RES_ABORT
    unsigned int pad1_[31];
    unsigned int done;     // closing kernel: workgroups finished
    unsigned int epoch;    // mailbox epoch of the next launch
    unsigned int ended;    // cluster launches (and marked runs of the chain) that have ended, and those
    unsigned int aborts;   // called off by the census; the host sees both in HOST_ENDED, HOST_ABORTS
    unsigned int pad2_[28];
};
// Words of the context's pinned memory that show them (word 0 is the error
// word that calls bring back, results start at word 8).
enum { HOST_ENDED = 1, HOST_ABORTS = 2 };
enum { RES_WAIT = 0, RES_GO = 1, RES_ABORT = 2 };
// Arguments of a resident launch and its closing kernel.
struct ResLaunch {
    const RepDesc *descs;
    RepState *st;
    const ResJob *jobs;          // workgroup b runs jobs first[b] .. first[b+1]-1
    const int *first;
    const ResPlane *planes;
    const ResRow *rows;
    const ResRep *reps;
    int grid, njobs, members, nreps;   // members: cluster workgroups of the grid
    uint32_t n;                  // sweeps
    int check_error;             // leave at once if the context's error word is raised (persistent form)
    ResSync *rs;
    GridSync *sync;
    int4 *part;                  // n x njobs sums
    unsigned long long *mbox;
    unsigned long long *host;    // where the context shows its HOST_* words
};

}  // namespace islf
