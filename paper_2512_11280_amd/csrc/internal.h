// Host-side declarations shared by the translation units of libadasd.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/adasd.h"
#include <hip/hip_ext.h>

#include "device_common.h"

namespace adasd {

constexpr int kWideCap = 512;       // list capacity from which the decision stage is launched with a workgroup per position
constexpr int kSumsMin = 4096;      // list length from which the state's running sums are kept (a longer list is no longer added up)
constexpr int kWideMin = 384;       // list length from which a sequence actually uses them
constexpr int kMaxSplit = 64;        // vocabulary slices per row: a fold takes one record per lane
constexpr int kMaxSampleSplit = 128; // vocabulary slices per sequence of the token kernel's form for long rows
constexpr int kXchgWords = 3;        // 64-bit hand-off words per record (records.h)
constexpr int kWaitPolls = 16384;    // polls (2.5 ms, 3.4 with a thousand waiting) before a workgroup stops waiting for the words of others
// How the drafting and token kernels wait for the slices' records: as many polls, or as the tests have it: the last slice of few rows
// gives up at once, or the records count as not there when they are.
enum WordWait : int32_t { kWaits = kWaitPolls, kGivesUp = 0, kNotThere = -1 };

// Where the rows of one call live.  which = 0: target, 1: draft.
struct RowMap {
  const char* base[2];
  int64_t seq_stride[2], pos_stride[2];  // elements
  const int32_t* draft_len;              // [B] or null
  const uint8_t* active;                 // [B] or null (draft-entropy mode)
  const int32_t* slots;                  // [B*K] or null: the candidate positions inside their windows, packed
                                         // (window position first, sequence second), -1 behind them
  int32_t K;                             // k_max; 0 selects draft-entropy mode (one row per sequence)
  int32_t B, V;
};

struct Workspace {
  float4* part1;      // [rows][kMaxSplit]   (m, s, u, -) partial log-sum-exp states of the two-kernel path; with the single-read
                      // statistics kernel, which has none, the HistRecords of the sequences
  int32_t* ticket1;   // [kTicket1Len]       arrival words of the drafting kernel (see Arrivals), zero between calls
  RowResult* rows;    // [rows]
  float2* part2;      // [positions][kMaxSplit] partial KL sums (p side, q side), log2 units
  int32_t* ticket2;   // [kTicket2Len]       arrival counters of the long-history decision kernel, zero between calls
  SamplePlan* plan;   // [B]
  Top2* part3;        // [B][kMaxSampleSplit]
  int32_t* ticket3;   // [kTicket3Len]       the same of the token kernel
  uint64_t* xchg;     // [positions][kMaxSplit][kXchgWords] self-validating hand-off words (records.h), zero between kernels:
                      // slice records of the single-read statistics kernel (cleared by the decision kernel), of the drafting
                      // kernel [rows] and of the token kernel [sequences] (cleared by the workgroup that folds them; where it takes
                      // the decisions too, in slots that the statistics kernel left unused)
  PosRecord* pos_rec; // [positions] outcomes of the positions (long-history decision kernel)
  float2* tok;        // [positions] logits of the drafted tokens (looked up by the JS kernel or by the column shards)
  int32_t* slots;     // [positions] packed list of the positions inside their windows (ragged calls)
  size_t bytes;
};

// Region offsets depend only on the size of the workspace (not on the shape of the call), so calls of
// different shapes can share one workspace: counters and hand-off words are always found where the
// previous call left them zeroed.  Returns the number of positions the workspace can serve.
size_t workspace_bytes_for(size_t positions);
size_t workspace_layout(size_t ws_bytes, Workspace* ws, void* base);

// Arrival counters of different rows / sequences sit on different 128-byte lines while the array is long
// enough (read-modify-writes on one line are served one after the other, whatever word they hit).
__host__ __device__ inline int ticket_stride(int count, int capacity) {
  int st = count > 0 ? capacity / count : 32;
  return st > 32 ? 32 : (st < 1 ? 1 : st);
}
constexpr int kTicket1Len = 65536, kTicket2Len = 32768, kTicket3Len = 32768;

struct DraftOut {     // draft-entropy epilogue
  const float* T_G;
  float* H_out;
  uint8_t* stop_out;
  int32_t force_stop; // step + 1 >= k_max
  WordWait wait;      // for the slices' records (see hand_off)
};

struct DraftDraw {    // token draw of a drafting step (x_i ~ q_i)
  uint32_t seed_lo, seed_hi;
  const uint32_t* seq_id;
  const uint32_t* round;
  uint32_t round0;
  uint32_t step;
  int32_t* token_out;
  uint32_t* status;   // may be null
};
// One drafting call: entropy and stop flag of each row, and with `draw` the drawn token (one kernel)
hipError_t launch_draft_step(const RowMap& map, int dt, const Workspace& ws, const DraftOut& dout,
                             const DraftDraw* draw /* or null */, hipStream_t st);

struct VerifyOut {
  float* H_p;
  float* H_q;
  float* d_js;
  // With both set, the JS kernel also looks up the two logits of each position's drafted token and leaves
  // them in tok[position], so the decision kernel does not start with a chain of two dependent loads.
  const int32_t* tokens;   // [positions] or null
  float2* tok;             // [positions] or null
};

// Kernel launches go through launch_kernel: while kernel timing is enabled and a timing scope is open,
// the launch carries a pair of events that the dispatch itself stamps at its start and end (the same
// timestamps a profiler reports), so the measured durations hold no launch or queueing time.
bool profile_take_events(hipEvent_t* start, hipEvent_t* stop);
template <class Kernel, class... Args>
inline void launch_kernel(Kernel kernel, dim3 grid, dim3 block, hipStream_t st, Args... args) {
  hipEvent_t e0, e1;
  if (profile_take_events(&e0, &e1))
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, e0, e1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

int pick_split(int rows, int V, int dt);

// Slices per row of the drafting and token scans.  Up to 896 rows: as few vectors per thread (turns) as keep every
// workgroup resident (seven on each of 256 compute units) and the slices within the limit of the hand-off words.  With more
// rows that would be one slice per row, which leaves compute units with three workgroups beside others with four, or
// a nearly empty second round: up to eight rounds then, in slices of four turns at least.  B rows of 128256, one slice
// per row / eight rounds (kernel, us): token bf16 B=897 177 / 117, 1200 214 / 158, 1793 302 / 223; drafted tokens bf16
// 127 / 115, 160 / 156, 240 / 224; entropies float 92 / 81, 105 / 108, 153 / 159 (four rounds: 86, 108, 159).  Rows of
// 5003, which stay in one slice: token B=1793 15 us, in more slices 20.
constexpr int kResidentGroups = 1792;
inline int scan_split(int rows, int V, int dt, int slices = kMaxSplit) {
  const int epv = dt == ADASD_BF16 ? 8 : 4, nv = (V + epv - 1) / epv;
  const bool many = rows > kResidentGroups / 2;
  const int64_t most = many ? 8 * kResidentGroups : kResidentGroups;
  for (int turns = many ? 4 : 1;; ++turns) {
    const int S = (nv + turns * kBlock - 1) / (turns * kBlock);
    if (S == 1 || (S <= slices && (int64_t)S * rows <= most)) return S;
  }
}

// The same for the token scan.  Rows of more than 65536 vectors (four turns of a workgroup in each of 64 slices) are cut
// into up to 128 slices, more than there are hand-off words, and take the form of the kernel for those: a few sequences'
// slices do not fill the chip.  One sequence (kernel, us), 64 slices / 128: 400000 float 8.3 / 7.7, 1048576 bf16 11.1 / 9.0,
// 1048576 float 13.4 / 9.4, 4194304 bf16 33 / 19, float 41 / 20.
constexpr int kLongRow = 65536;
inline int token_split(int rows, int V, int dt) {
  const int epv = dt == ADASD_BF16 ? 8 : 4, nv = (V + epv - 1) / epv;
  return scan_split(rows, V, dt, nv > kLongRow ? kMaxSampleSplit : kMaxSplit);
}

// Who folds the slices' records of a drafting or token scan: of a few rows the workgroup of the last slice, which waits for the
// others' words; else the last one to add to the row's count, which costs a round trip more (records.h).  Whole calls (us), waiting /
// the last to add: drafting 1 x 32000 float 4.6 / 5.0, 64 x 32000 6.7 / 7.1, 64 x 128256 bf16 12.0 / 12.4, 128 x 128256 17.6 / 18.0,
// 512 x 32000 float 18.3 / 18.8, a round of 16 x 2 x 32000 15.1 / 15.7.  The line is not where that ends: those who wait hold a
// place on the chip per row, and where the slices are a multiple of eight all of them on one die, which has 160 to 224 (five to
// seven workgroups on each of 32 compute units).  More than 64 would keep a good part of a die from the work of other streams.
// (Workgroups of a die start in order, those of different dies need not, and other streams' work may come between: whoever is
// waited for has mostly started, but nothing here relies on it.)
constexpr int kFewRows = 64;
__host__ __device__ inline bool few_rows(int rows) { return rows <= kFewRows; }

// Whether a scan over slices of `chunk` vectors leaves out the logits that cannot win any more (sample_device.h): from four
// groups of 256 logits per wavefront on.  The first groups are looked at in any case, and the test costs a wavefront
// about a tenth of what looking at a group costs.  Rows of 128256, without / with (kernel, us): drafting bf16, 32 rows (3.9 groups) 9.8 / 9.8,
// 64 (6) 13.7 / 13.0, 128 (9.7) 21.8 / 18.5, 256 (18) 34.7 / 26.3, 896 (63) 109 / 77; float, 32 (3) 10.4 / 11.0, 64 (4.8) 15.1 / 14.2,
// 128 (9) 22.7 / 19.0; token bf16, 8 (2) 6.0 / 6.5, 64 (6) 13.9 / 13.6, 128 (9.7) 21.8 / 18.7, 256 (18) 37.1 / 29.2.
// Rows in which little or nothing falls out cost no more than without: drafting 128 x 152064 bf16, logits rising along the row
// 23.9 / 23.2; masked but for the last 1000 29.1 / 22.5, but for one in a thousand 25.5 / 20.1.
constexpr int kPruneGroups = 4;
inline bool scan_prunes(int chunk, int dt) { return chunk * (dt == ADASD_BF16 ? 2 : 1) >= kPruneGroups * kBlock; }

// Ragged windows: the positions i < draft_len[b] of all sequences, packed into slots[0 .. n) in the order
// (window position, sequence), -1 in the remaining slots up to B*K (one small kernel).
hipError_t launch_pack_slots(const int32_t* draft_len, int B, int K, int32_t* slots, hipStream_t st);

// plain streaming read (diagnostics): one word per workgroup goes to `sink`
size_t stream_read_groups(size_t bytes);
hipError_t launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t st);

hipError_t launch_rowstats(const RowMap& map, int dt, int rows, int S, const Workspace& ws, hipStream_t st);
// Single-read statistics kernel: T threads per workgroup, NB vectors per thread and row, S slices per position.
// It leaves what the two-kernel path leaves (rows, entropies, per-slice JS sums, the drafted tokens' logits)
// plus the hand-off words of the positions it worked on, which the decision kernel clears (DecideArgs::xchg_split).
bool fused_plan(const RowMap& map, int dt, int* T_out, int* NB_out, int* S_out);
struct HistRecord;
struct HistArgs {       // the lists of a call's sequences (history_device.h), or rec == null: nothing to form
  const float* LA;
  const float* LR;
  const int32_t* nA;
  const int32_t* nR;
  const double* mom;    // as DecideArgs::mom
  HistRecord* rec;      // [B]
  int32_t cap, B, bw_rule;
};

struct UpdateArgs {
  int32_t B, K, cap;
  float* T_G;
  double* ent_sum;
  int32_t* ent_cnt;
  float* LA;
  float* LR;
  int32_t* nA;
  int32_t* nR;
  double* mom;          // [B,4] running sums of the lists about their first elements, or null
  const int32_t* n_accept;
  const int32_t* draft_len;
  const float* H_q;
  const float* d_js;
  float d_eps;
  uint32_t* status;
};
struct DecideArgs {
  RowMap map;
  int32_t dt;
  int32_t jsd_split;   // > 0: the distances are still per-slice partial sums of the JS kernel (that many per position)
  int32_t xchg_split;  // > 0: the single-read statistics kernel ran with that many slices: its hand-off words are cleared here
  const int32_t* draft_tokens;
  // state (device pointers, may be null)
  int32_t cap;
  const float* LA;
  const float* LR;
  const int32_t* nA;
  const int32_t* nR;
  const double* mom;    // [B,4] running sums of the lists about their first elements, or null: add them up here
  const HistRecord* hist;   // [B], left by the statistics launch, or null: the lists' constants are formed here
  uint32_t seed_lo, seed_hi;
  const uint32_t* seq_id;
  const uint32_t* round;
  uint32_t round0;
  int32_t reject_rule, kde_min_n, bw_rule, relaxed_off;
  const float2* tok;    // non-null: (z_p(x), z_q(x)) of every position's drafted token; the logits are then not read
  int32_t base_test;    // 1: match test of the verification loop, replacement from p without the drafted token
  int32_t list_update;  // 1: the accepted list grows inside the loop
  float d_eps;          // filter of the in-loop appends
  // outputs
  int32_t* n_accept;
  float* H_p;
  float* H_q;
  float* d_js;
  float* p_accept;
  uint8_t* accept_mask;
  uint32_t* status;
};
hipError_t launch_stats_fused(const RowMap& map, int dt, int T, int NB, int S, int wait_polls,
                              const Workspace& ws, const VerifyOut& vout, const HistArgs& hist, hipStream_t st);
// upd.B > 0: the round is also applied to the state (the update step) by the same kernel
hipError_t launch_decide(const DecideArgs& a, const UpdateArgs& upd, const Workspace& ws, hipStream_t st);
// JS distance: per-slice partial sums (the decision kernel adds them up), rows and entropies
// S_fold: slice records per row that the kernel folds into the normalisers (S for a whole-vocabulary call)
hipError_t launch_jsd(const RowMap& map, int dt, int S, int S_fold, const Workspace& ws, const VerifyOut& vout,
                      hipStream_t st);

// ---- column-sharded verification: records exchanged between the shards (float4 each)
hipError_t launch_shard_fold_rows(const RowMap& map, int S, const Workspace& ws, float4* triples_out, hipStream_t st);
hipError_t launch_shard_scatter_rows(const float4* triples_all, int G, int rows, const Workspace& ws, hipStream_t st);
hipError_t launch_shard_fold_pos(const RowMap& map, int dt, int S, const Workspace& ws, const int32_t* draft_tokens,
                                 int col_begin, float4* pos_out, hipStream_t st);
hipError_t launch_shard_prepare(const RowMap& map, const float4* pos_all, int G, const Workspace& ws, float* H_p,
                                float* H_q, hipStream_t st);

struct SampleArgs {
  RowMap map;
  int32_t dt;
  uint32_t seed_lo, seed_hi;
  const uint32_t* seq_id;
  const uint32_t* round;
  uint32_t round0;
  int32_t* next_token;
  uint32_t* status;
  WordWait wait;        // for the slices' records (see hand_off)
};
hipError_t launch_shard_sample(const SampleArgs& a, int S, int col0, const Workspace& ws, float4* top_out, hipStream_t st);
hipError_t launch_shard_pick(int B, int G, const float4* top_all, const Workspace& ws, int32_t* next_token,
                             uint32_t* status, float* tau_out, hipStream_t st);
hipError_t launch_shard_refine(const SampleArgs& a, int S, int col0, const float* tau, int exact, const Workspace& ws,
                               void* cand_out, hipStream_t st);
hipError_t launch_shard_settle(const SampleArgs& a, int G, float* tau, const void* cand_all, const Workspace& ws,
                               hipStream_t st);
// Whether the decisions of a round are taken inside the token kernel, S slices per sequence (sample.hip): up to so many workgroups.
constexpr int kMergeGroups = 512, kMergeInLoop = 256;      // (256 compute units)
bool merges_decisions(const DecideArgs& d, int S);
hipError_t launch_decide_sample(const DecideArgs& d, const UpdateArgs& upd, const SampleArgs& a, int S, const Workspace& ws, hipStream_t st);
hipError_t launch_sample(const SampleArgs& a, int S, const Workspace& ws, hipStream_t st);

hipError_t launch_update(const UpdateArgs& a, hipStream_t st);
hipError_t launch_state_refresh(const UpdateArgs& a, hipStream_t st);
hipError_t launch_state_init(const UpdateArgs& a, hipStream_t st);
hipError_t launch_state_refresh(const UpdateArgs& a, hipStream_t st);
hipError_t launch_zero(void* p, size_t bytes, hipStream_t st);

}  // namespace adasd
