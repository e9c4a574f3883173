// Host-side lowering of one decode step into per-CU task queues, and the
// static check that must accept a schedule before it is launched.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/amk.h"

namespace amk {

// Largest number of GEMV output rows one task may own: the kernel keeps one
// fp32 partial per row and streaming wave in LDS.
constexpr int kMaxJobsPerTask = 1024;
// Largest number of position splits per KV head (one combine lane per split).
constexpr int kMaxAttnSplits = 64;
// Counters a wide stage signals (task i counter i mod k); its consumers wait
// on all of them, so the producers' increments spread over k counter lines.
constexpr int kStageCounters = 4;

// Derived shape of a validated config.
struct Shape {
  int H = 0, L = 0, nq = 0, nkv = 0, hd = 0, I = 0, V = 0, max_seq = 0;
  int fmt = 0, tied = 0;
  int qgroup = 0;        // W4A16: input columns per scale (0 for the other formats)
  int group = 0;         // query heads per KV head
  int half = 0;          // hd / 2: RoPE row pairs per head
  int units = 0;         // (nq + 2 nkv) * half: q/k/v row-pair units
  int gunits = 0;        // (group + 2) * half: units of one KV group
  int q_units = 0;       // nq * half
  int npg = 0;           // QKV tasks per KV group
  int nsplit = 0;        // attention position splits per KV head (long schedule)
  int max_jobs = 0;      // GEMV rows per task cap
  int short_context = 0; // steps with pos + 1 <= short_context use the short schedule
  int tiny_context = 0;  // steps with pos + 1 <= tiny_context use the tiny schedule
  int assign = 0;        // AMK_ASSIGN_ROUND_ROBIN or AMK_ASSIGN_LPT
  float theta = 0.f, eps = 0.f;
};

// Number of tasks of a GEMV stage over `items` items of `jobs_per_item` rows:
// one per CU (at most one per item), more if the row cap requires.
int stage_tasks(int items, int jobs_per_item, int n_cu, int max_jobs);

// Validates the config (shape family, divisibility, 16-byte row alignment)
// and fills *s.  Returns AMK_OK or AMK_ERR_INVALID_ARGUMENT / _UNSUPPORTED
// with a message.
int derive_shape(const amk_config_t* cfg, const amk_tuning_t* tuning, int n_cu, Shape* s,
                 std::string* why);

struct Schedule {
  std::vector<amk_task_t> tasks;   // sorted by (cu, seq)
  std::vector<int32_t> queue_start;// n_cu + 1 offsets into tasks
  int n_counters = 0;
  int n_lm_slots = 0;              // argmax partial slots (one per LM-head task)
};

// Defaults of amk_tuning_t.short_context and .tiny_context.  us a step by the
// position, with either schedule:
//  tiny / short   Llama-3-8B bf16: 0 2732 / 2780, 3 2777 / 2782, 5 2808 / 2780;
//                 8B W8A16: 0 1681 / 1745, 4 1741 / 1746, 5 1757 / 1746;
//                 Llama-3.2-1B W8A16: 0 557 / 583, 4 584 / 583, 5 591 / 583;
//                 TinyLlama bf16: 0 690 / 746, 5 737 / 747, 6 748 / 747;
//                 SmolLM2 bf16: 0 542 / 619, 5 590 / 618, 7 613 / 619.
//                 Even near 3, 4, 4, 6 and past 7: 6 loses up to 1.4% at positions
//                 4 and 5 of the larger shapes and gains up to 12% before.
//  short / long   8B bf16: 255 2877 / 2914, 300 2885 / 2914, 400 2939 / 2915;
//                 8B W8A16: 255 1845 / 1866, 300 1858 / 1866, 400 1910 / 1865;
//                 Llama-3.2-1B W8A16: 300 612 / 633, 400 632 / 634, 600 653 / 634;
//                 TinyLlama bf16: 400 840 / 861, 600 880 / 864;
//                 SmolLM2 bf16: 400 710 / 739, 600 751 / 741.
//                 Even between 310 and 560: 256 lies below all of them.
constexpr int kDefaultShortContext = 256;
constexpr int kDefaultTinyContext = 6;

// Deterministic lowering of one decode step onto n_cu queues, schedule
// variant AMK_SCHEDULE_SHORT or AMK_SCHEDULE_LONG.
Schedule build_schedule(const Shape& s, int n_cu, int variant);

// Which head a QKV unit belongs to: kind 0 = query head `head`, 1 = K head,
// 2 = V head (head = KV group); i = row-pair index within the head.
struct UnitHead {
  int kind, head, i;
};
UnitHead unit_head(const Shape& s, int u);

// Static check (never throws).  Fills *rep; returns true iff accepted.
bool check_schedule(const Shape& s, int n_cu, const amk_task_t* tasks, int n_tasks,
                    int n_counters, amk_check_report_t* rep);

// Sorts tasks by (cu, seq) and computes queue offsets (tasks must be checked).
void finalize_queues(std::vector<amk_task_t>* tasks, int n_cu, std::vector<int32_t>* queue_start);

// Number of rows (jobs) a GEMV task computes; 0 for non-GEMV ops.
int task_jobs(const Shape& s, const amk_task_t& t);

}  // namespace amk
