// step.h -- kernel argument blocks and launchers of the step (host + device).
#pragma once

#include "common.h"
#include "event_log.h"

namespace sfqed {

// step kernels: 8 waves per block, two blocks per CU (the emission tables take
// ~78 KiB of LDS per block), so four waves per SIMD; the FP32 count kernels
// are held to the register budget of that occupancy (the FP64 ones keep their
// tables in HBM and are limited by registers instead).  The lepton write
// kernel runs one block per CU (see kWriteThreads).
constexpr int kStepThreads = 512;
constexpr int kStepWavesPerSimd = 4;
// photons merged inside the step: photons per thread and per tile of the count pass
constexpr int kMergedItems = 4;
constexpr int kMergedTile = kStepThreads * kMergedItems;
// lepton work queue: counters per launch and kernel (see wq_take)
constexpr int kQueueParts = 8;
constexpr int kQueueStride = 16;  // 64-bit words between counters: one 128-byte line each
constexpr int kQueueWords = kQueueParts * kQueueStride;
constexpr uint32_t kChunkMin = 256, kChunkMax = 8192;
// How a lepton launch of n particles deals them out to its waves (see wq_take):
// every wave owns `pieces` pieces of `piece` particles, dealt in turn; the last
// `rest` particles come from the counters.  Up to kOwnMax particles per wave
// the waves own everything.
struct WqPlan {
  uint32_t n, waves, piece, pieces, rest, chunk_div;
};
constexpr uint32_t kOwnMax = 512;
__host__ __device__ inline WqPlan wq_plan(uint32_t n, uint32_t waves) {
  WqPlan p;
  p.n = n;
  p.waves = waves;
  const uint32_t per = (uint32_t)(((uint64_t)n + waves - 1) / waves);
  if (per <= kOwnMax) {
    p.pieces = per <= 64 ? 1 : (per + 63) / 64;
    const uint64_t all = (uint64_t)waves * p.pieces;
    p.piece = (uint32_t)((n + all - 1) / all);
    p.rest = 0;
  } else {
    p.piece = 64;
    p.pieces = per / 128;
    p.rest = n - waves * p.pieces * 64;
  }
  p.chunk_div = 2 * (waves / kQueueParts > 0 ? waves / kQueueParts : 1);
  return p;
}

// The lepton write kernel runs one block of kWriteThreads per CU (four waves
// per SIMD, one copy of the LDS tables).  Its child records are staged per
// lane in LDS, kLinePieces 16-byte pieces (a 64-byte half line) at a time, and
// written by kLinePieces lanes per half line: a store instruction then covers
// 16 half lines instead of 64 scattered pieces.  A lane's slot has one spare
// piece so that neighbouring slots start in different banks.
constexpr int kWriteThreads = 1024;
constexpr int kLinePieces = 4;
constexpr int kLineShift = 2;  // log2(kLinePieces)
constexpr int kLineSlot = kLinePieces + 1;
constexpr size_t kLineStageBytes = (size_t)kWriteThreads * kLineSlot * 16;
constexpr size_t kMaxLdsBytes = 163840;  // LDS per work-group on gfx950
// byte offset of the line slots in the write kernel's dynamic LDS: after the
// source table and, for FP32, the staged rate and CDF tables
__host__ __device__ constexpr size_t line_stage_offset(size_t src_bytes, int fp32, int rate_n, int cdf_n) {
  return (src_bytes + (fp32 ? 8 * (size_t)rate_n + 4 * (size_t)cdf_n : 0) + 15) / 16 * 16;
}
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kMergeThreads = 256;
constexpr int kMergeItems = 8;
constexpr int kMergeTile = kMergeThreads * kMergeItems;

// device statistics words
constexpr int kStatMaxEvents = 0;
constexpr int kStatCapped = 1;
constexpr int kStatEventParticles = 2;  // + 0 leptons, + 1 photons
constexpr int kStatBadRoot = 4;         // a record's root named no particle of the ensemble
constexpr int kStatLogNeed = 5;         // largest event log a lepton launch needed (bytes)
constexpr int kStatReplays = 6;         // lepton launches written from the event log
constexpr int kStatReruns = 7;          // lepton launches written by the direct write kernel
constexpr int kStatLogOwn = 8;          // the same as kStatLogNeed with a first block for every wave
constexpr int kStatWords = 9;

// Event log of the lepton count pass, replayed by the write pass
// (k_replay_lepton and k_replay_events in step.hip; format in event_log.h).
// Each wave of the count launch writes its own sequence of trip records into
// blocks of one pool: handed out one by one, or its first block by its own index
// and further ones handed out (log_own_blocks); log_ctl words of the launch:
// blocks handed out, overflow flag, the sum of the waves' tallies.
constexpr int kLogUsed = 0, kLogOverflow = 1, kLogTally = 2;
// bytes of one lane's slot: an event's z and h in the step's dtype, or a
// finished particle's optical depth (FP64)
template <typename T>
constexpr uint32_t log_slot_bytes() {
  return 2u * (uint32_t)sizeof(T);
}

// A launch covers up to two source ranges ("parts"): electrons and positrons
// go together (part 0 e-, part 1 e+), photons alone (part 0).  Particle k of
// the launch is particle begin[0] + k of part 0 for k < n0, else particle
// begin[1] + k - n0 of part 1, so the append order is that of separate
// launches for the two species, one after the other.
// Per-lane choice of launch constants: the step kernels copy the arrays of
// both source ranges and the fields of the three species into this table in
// LDS when they start (see step.hip); it precedes the tables in the dynamic LDS.
enum SrcWord : int { kPx, kPy, kPz, kX, kY, kZ, kW, kTau, kId, kAlive, kNev, kRec, kPos, kBegin, kSrcWords };
enum FieldWord : int { kEx, kEy, kEz, kBx, kBy, kBz, kStride, kFieldCount, kFieldWords };
struct SrcTable {
  uint64_t part[2][kSrcWords];    // the two source ranges of the launch
  uint64_t field[3][kFieldWords];  // the fields of each species
  uint64_t stats;                  // the launch's statistics words (device address)
  uint64_t pad;                    // to a multiple of 16 bytes
};
static_assert(sizeof(SrcTable) % 16 == 0, "LDS layout");

// FP64 step kernels copy the Chebyshev coefficients of the rate to LDS when the
// table has at most 64 segments (9 KiB a block; the default range of chi, 1e-7
// to 1e5, has 56): a trip's eighteen 8-byte gathers through L2 become LDS reads.
// Lepton count passes of a step of 2e5 particles 1.82 ms (1.87 before), photons'
// 0.32 (0.35).  Wider tables are read from memory as before: copying more would
// cost blocks per CU for chi that the particles hardly span.
constexpr int kChebStaged = 64;
__host__ __device__ constexpr bool cheb_staged(int nseg) { return nseg <= kChebStaged; }

template <typename T>
struct StepArgs {
  SpeciesView<T> src[2];  // the input ensemble of each part (from_main)
  Rec<T>* src_rec[2];     // or its appended records
  T* src_pos[2];          // their positions (4 per record) or null
  int64_t begin[2];       // first particle of each part in its source
  int32_t species;        // species of part 0 (0 e-, 2 photon); part 1 is species + 1
  int32_t from_main;      // 1: sources are the input ensemble (root = species << 30 | index)
  int64_t n0, n;          // particles of part 0; of the launch
  FieldView<T> f[3];
  Rec<T>* out_rec[2];  // leptons: out[0] photons; photons: out[0] e-, out[1] e+
  T* out_pos[2];
  int64_t out_cap;
  int32_t* counts;     // [n]
  int64_t* offsets;    // [n]
  int32_t* list;       // [n]
  const int64_t* list_len;
  WqPlan wq;            // leptons: how the count pass deals out its particles
  int32_t block_waves;  // and how many waves of each block get any
  unsigned long long* queue;  // work counters of the count, then the write kernel: 2 x kQueueWords, zero at launch
  unsigned long long* stats;
  double dt;
  uint64_t seed;
  uint32_t step;
  int32_t emission, pair, push, positions, write_nev;
  double gamma_min;
  int64_t max_events;
  TableView tab;
  // photons merged inside the step (k_count_photon_merged): survivors of an
  // appended range go straight into the main photon arrays
  SpeciesView<T> dst;               // the main photons
  int64_t dst_cap;                  // their capacity (nothing is written at or past it)
  int64_t* dst_cursor;              // photons in dst so far: read by the first tile, set by the last
  uint64_t* dst_state;              // look-back words, one per tile of kMergedTile photons
  uint32_t dst_epoch;
  unsigned long long* dst_ticket;   // tile counter, zero at launch
  int64_t* pair_cursor;             // pairs appended so far (the scan's cursor of a photon launch)
  // a merged range sized on the device: photons [n_base, min(*n_dev, n_cap)) of
  // the append buffer (the photon cursor after the round's lepton launch), so
  // that the host need not read the cursor back first; null: n photons
  const int64_t* n_dev;
  int64_t n_base, n_cap;
  int64_t list_cap;                 // entries of list and offsets (events past it are not listed)
  // lepton launches: the count pass's event log, replayed by the write pass
  char* log_pool;                   // log blocks
  uint64_t log_cap;                 // bytes of log_pool (0: the count pass only measures the log)
  uint64_t* log_head;               // per wave of the count launch: 1 + byte offset of its first block, 0 = none
  unsigned long long* log_ctl;      // the launch's log words (kLogUsed, kLogOverflow, kLogTally), zero at launch
  int32_t log_on;                   // 1: the count pass logs; the replay writes unless the log overflowed
  uint32_t log_own;                 // first blocks of the pool that belong to the waves by their index (wq.waves or 0)
  int64_t* offsets_k;               // first-child offset of every particle of the launch (from the scan)
};

struct ScanArgs {
  const int32_t* counts;
  int64_t n;
  int64_t* offsets;
  int32_t* list;
  int64_t* cursor;    // in: append count before the launch; out: after
  int64_t* list_len;
  uint64_t* state_c;  // look-back words, one per tile
  uint64_t* state_f;
  uint32_t epoch;
  unsigned long long* ticket;  // zero at launch
  int64_t num_tiles;
  unsigned long long* event_particles;  // += number of particles with events
  int64_t* offsets_k;  // or null: the first-child offset of every particle
};

template <typename T>
struct MergeArgs {
  SpeciesView<T> main;
  const Rec<T>* app;
  const T* app_pos;
  int64_t n_main, n_app;
  int32_t positions;
  uint64_t* state;
  uint32_t epoch;
  unsigned long long* ticket;
  int64_t num_tiles;
  int64_t* out_count;
};

// resampling after the merge (see step.hip)
constexpr int kLevelThreads = 256;
constexpr int kLevelBlocks = 1024;      // fixed: the sums do not depend on the size of the launch
constexpr uint32_t kResampleJ = 0xFFFFFFFDu;  // Philox counter word of the thinning draw
constexpr int kLevelDevicePasses = 8;   // threshold passes queued without waiting for the host
constexpr int kLevelMaxPasses = 100;    // a solve stops there

// Device state of one species' threshold solve (written by k_level_step or k_level_solve, read
// by the next pass and by the host).
struct LevelState {
  double wt;        // current threshold weight (0: no thinning)
  double eligible;  // particles that pass the filter
  double total;     // their total weight
  int64_t kept;     // particles after the compaction (written by k_resample)
  int32_t done, iterations;
  int32_t started, pad;  // the first pass has been made
};

// One pass of the threshold solves, for the species with solve[k] set.
template <typename T>
struct LevelArgs {
  SpeciesView<T> s[3];
  int64_t n[3], target[3];
  int32_t solve[3];
  double e_min2;      // squared energy threshold of photons (0: no filter)
  uint64_t* mask;     // a bit per photon, set by the first pass: it passes the filter
  LevelState* state;  // [3]
  double* part;       // [3][kLevelBlocks][4] the blocks' sums
  unsigned long long* tickets;  // [3] of the compaction that follows, cleared by the first pass
};

// The solve in one launch (k_level_solve): 256 blocks of 1024 threads, which
// hold the weights of the kLevelBlocks x kLevelThreads threads above in LDS, a
// slot of 4 bytes per particle of a thread.  35 slots and the trees' scratch are
// 158 of a CU's 160 KiB; species with ceil(n / 262144) slots in all above that
// (9.2e6 particles) take the two kernels per pass, as do parts of a chip with
// fewer CUs than blocks.
constexpr int kSolveThreads = 1024;
constexpr int kSolveBlocks = kLevelBlocks * kLevelThreads / kSolveThreads;
constexpr int kSolveGroups = kSolveThreads / kLevelThreads;
constexpr int kSolveSlots = 35;
constexpr int kSolvePasses = 32;
static_assert(kSolveBlocks == 256 && kSolveGroups == 4, "k_level_solve: 16 x 16 blocks, 16 sums a species and block");
// words of `sync`: the compaction's tickets, whether a block has left, the
// barrier's counters (a line each), eight words per pass; all zero at launch
constexpr int kSolveLeft = 8, kSolveCounters = 16, kSolveWords = kSolveCounters + 16 * 17;
constexpr int kSolveSyncWords = kSolveWords + 8 * kSolvePasses;
template <typename T>
struct SolveArgs {
  LevelArgs<T> lv;
  unsigned long long* sync;
  uint64_t wait;     // longest wait at a barrier, in ticks of 10 ns
  int32_t slots[3];  // per species
};

template <typename T>
struct ResampleArgs {
  SpeciesView<T> s;
  int64_t n;
  int32_t photon, positions;
  double e_min2;  // squared energy threshold of photons (0: no filter)
  uint64_t seed;
  uint32_t step;
  uint64_t* state;
  uint32_t epoch;
  unsigned long long* ticket;
  int64_t num_tiles;
};

// One launch compacts up to three species: block b works on species k for
// first_block[k] <= b < first_block[k + 1] (a species without a filter or target
// has no blocks; the blocks of one that keeps everything return at once).
template <typename T>
struct ResampleLaunch {
  ResampleArgs<T> a[3];
  int64_t first_block[3];
  int32_t solve[3];
  int32_t forced;     // 0: nothing is done unless the solves of all these species have finished
  LevelState* state;  // [3]: the thresholds
};

// The records of both lepton species behind the particles of their arrays.
template <typename T>
struct AppendArgs {
  SpeciesView<T> dst[2];
  int64_t at[2];  // first free place
  const Rec<T>* rec[2];
  const T* pos[2];  // or null
  int64_t n[2];
};

// The photon write pass and, in a merged step, the appending of the round's
// lepton records (ap.n zero: none).
template <typename T>
struct WritePhotonArgs {
  StepArgs<T> step;
  AppendArgs<T> ap;
  int32_t ap_blocks;  // set by the launch
};
static_assert(sizeof(WritePhotonArgs<double>) <= 4096, "kernel arguments");
constexpr int kAppendBlocks = 1024;  // at most, of kStepThreads threads

template <typename T, bool kPhoton>
hipError_t launch_count(const StepArgs<T>& a, int grid, size_t lds, hipStream_t st);
template <typename T>
hipError_t launch_count_photon_merged(const StepArgs<T>& a, int grid, size_t lds, hipStream_t st);
template <typename T>
hipError_t launch_write_photon(WritePhotonArgs<T>& a, int grid, size_t lds, hipStream_t st);
template <typename T>
hipError_t launch_write(const StepArgs<T>& a, int grid, size_t lds, hipStream_t st, bool stage);
template <typename T>
hipError_t launch_replay(const StepArgs<T>& a, int grid, hipStream_t st);
hipError_t launch_scan(const ScanArgs& s, hipStream_t st);
template <typename T>
hipError_t launch_merge_photons(const MergeArgs<T>& a, hipStream_t st);
template <typename T>
hipError_t launch_level_pass(const LevelArgs<T>& a, int first, hipStream_t st);
template <typename T>
hipError_t launch_level_solve(const SolveArgs<T>& a, hipStream_t st);
template <typename T>
hipError_t launch_resample(const ResampleLaunch<T>& a, int64_t tiles, hipStream_t st);
hipError_t launch_count_alive(const uint8_t* alive, int64_t n, unsigned long long* out, hipStream_t st);
template <typename T>
hipError_t launch_count_alive_rec(const Rec<T>* rec, int64_t n, unsigned long long* out, hipStream_t st);
template <typename T>
hipError_t launch_append_records(const AppendArgs<T>& a, hipStream_t st);
// particles of [0, n) with a non-finite momentum, position, weight, optical
// depth or field component are added to *bad (validate.hip)
template <typename T>
hipError_t launch_count_nonfinite(const SpeciesView<T>& s, const FieldView<T>& f, int64_t n,
                                  unsigned long long* bad, hipStream_t st);
template <typename T>
hipError_t launch_init_tau(double* tau, const uint64_t* id, int64_t n, uint64_t seed, uint32_t step, hipStream_t st);
template <typename T>
hipError_t launch_eval_rate(const TableView& tab, int process, const T* chi, const T* e, T* out, int64_t n,
                            hipStream_t st);
template <typename T>
hipError_t launch_eval_particles(const TableView& tab, int species, const T* px, const T* py, const T* pz,
                                 const FieldView<T>& f, int64_t n, T* chi, T* w, hipStream_t st);
template <typename T>
hipError_t launch_sample(const TableView& tab, int process, const T* chi, const uint32_t* k, T* out, int64_t n,
                         hipStream_t st);


}  // namespace sfqed
