// One batch-1 Llama decode step as ONE persistent cooperative kernel for
// gfx950 (MI355X): one workgroup per CU walks its host-built task queue
// (paper §3 Algorithm alg:sm) and orders itself against other CUs only
// through monotonic counters (paper §4 "Synchronization model").
//
// Workgroup layout (512 threads = 8 wave64s):
//   wave 0      "sync wave": waits on counters (agent-scope acquire), reduces
//               the streaming waves' partial row sums, applies the fused
//               epilogue (RMSNorm scale, RoPE + KV append, SwiGLU, residual,
//               int8 row scale, argmax), writes every result other CUs read,
//               then releases and signals.
//   waves 1..7  "streaming waves": stream the task's weight rows from HBM in
//               16-byte-per-lane vectors through a ring of registers and
//               reduce them against the LDS activation (int4 weights: with
//               their fp16 group scales, dequantised in the dot product); they
//               also load the task's input into LDS after the wait (one round
//               trip), and the last one stages task records and prepares
//               epilogues ahead.
//   all waves   run attention and inline continuations.
//
// Per task the workgroup passes three barriers:
//   B1a  the sync wave's counter wait is satisfied (or the launch aborts)
//   B1b  the input activation is in LDS (GEMV tasks)
//   B2   the task's compute is done (partials in LDS / attention stored)
// after which the sync wave stores, releases and signals the task's results
// while the other waves go on to the next task.  A task with a chain counter
// passes B3 after its signal: if that signal completed its counter (it is the
// last producer of this launch) every wave then runs that counter's inline
// task: a KV group's whole attention after its QKV tasks, or the merge of a KV
// group's attention splits.  Each wave drains its own stores, the workgroup
// meets at B4 and the sync wave releases and signals the chain counter.
//
// The weight stream does not stop at a task's end: while a streaming wave
// consumes the last granules of one task it already issues the first ones of
// the next GEMV task of its queue (weights depend on nothing), so they travel
// while the epilogue, the signal, the wait and the input load go on.  For that
// the last wave keeps the next tasks' records and layer pointers in LDS
// (struct Slot), loaded two and three tasks ahead: read when needed, each was
// a chain of two cold scalar loads between a task's end and its successor's
// first weight load.
//
// Every result another workgroup reads is stored coherent at agent scope
// (write-through past the XCD's L2), so releasing it takes only a drain of
// the storing wave's own stores before the counter increment: no L2
// writeback.  Only the sync wave waits on counters (acquire: agent-scope
// polls, then plain loads with no cache invalidation, see
// acquire_after_poll) and increments them; streaming waves never drain while
// their weight loads are in flight.
// Lane reductions use DPP (VALU latency) rather than LDS permutes.
//
// No MFMA in the GEMVs: a batch-1 GEMV is a matrix-vector product, bound by HBM
// bandwidth.  The attention scores, of four to eight query heads against each K
// row, are matrix products and use it.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "device.h"
#include "schedule.h"

namespace amk {

constexpr int NT = 512;       // threads per workgroup
constexpr int NW = NT / 64;   // waves
constexpr int NSW = NW - 1;   // streaming waves
constexpr int GRAN = 1024;    // bytes per wave-wide 16-B-per-lane load
// Granules each streaming wave keeps in flight (registers): slots, each
// refilled as soon as it is consumed.  28 KiB a CU; more only lengthens every
// queue that polls, inputs and result stores pass through.  Llama-3-8B shape,
// us a step with 4 / 5 / 6 / 8: bf16 pos 0 2808 / 2834 / 2836 / 2856, W8A16
// pos 100 1826 / 1818 / 1823 / 1841, W4A16 pos 2000 1755 / 1785 / 1827 / 1792.
constexpr int RING = 4;
// int4 columns per granule, and per lane (one 16-byte load of 32 nibbles)
constexpr int GRAN4 = 2 * GRAN;
constexpr int LANE4 = 32;

// A task record and its layer's pointers, staged in LDS ahead of their task.
struct Slot {
  amk_task_t t;
  DevLayer ly;
};
constexpr int NSLOT = 4;  // tasks idx .. idx + 3
static_assert(sizeof(amk_task_t) == 64 && sizeof(DevLayer) == 128, "one dword per lane: 16 lanes a record, 32 a layer");

struct Ctl {
  Slot slot[NSLOT];
  OpGeom geom[kOps];            // per op, from the model record
  float4 prep[2][64];           // the prepared epilogue of the task to come (struct Fast), a lane per item
  float ssq[NSW];               // per-wave sum of squares of the task input
  int abort;
  int cont;                     // this task runs its chain counter's inline task
};

// ---------------------------------------------------------------- memory helpers
// Pointers read out of the model record are generic; casting them to the
// global (1) or constant (4) address space makes the compiler emit global_*
// vector accesses and scalar s_load reads instead of flat accesses, which
// would also count against the LDS wait counter.
#define AMK_GLOBAL __attribute__((address_space(1)))
#define AMK_CONST __attribute__((address_space(4)))
// Raw storage of the same size as T (native vector types copy through any
// address space; HIP's vector structs do not).
template <int N> struct Bits;
template <> struct Bits<2> { typedef unsigned short T; };
template <> struct Bits<4> { typedef unsigned int T; };
template <> struct Bits<8> { typedef unsigned int T __attribute__((ext_vector_type(2))); };
template <> struct Bits<16> { typedef unsigned int T __attribute__((ext_vector_type(4))); };

template <typename T>
__device__ __forceinline__ T ldg(const void* p) {
  using B = typename Bits<sizeof(T)>::T;
  return __builtin_bit_cast(T, *(const AMK_GLOBAL B*)p);
}
// Load of data that is read once per step (weight rows): non-temporal, so the
// stream does not push the vectors, counters and records that workgroups share
// out of the L2.
template <typename T>
__device__ __forceinline__ T ldnt(const void* p) {
  using B = typename Bits<sizeof(T)>::T;
  return __builtin_bit_cast(T, __builtin_nontemporal_load((const AMK_GLOBAL B*)p));
}
template <typename T>
__device__ __forceinline__ void stg(void* p, const T& v) {
  using B = typename Bits<sizeof(T)>::T;
  *(AMK_GLOBAL B*)p = __builtin_bit_cast(B, v);
}
// Store of a published result: coherent at agent scope (written through the
// XCD's L2), so a producer releases its results by draining its stores
// (s_waitcnt vmcnt(0)) before the counter increment, with no L2 writeback.
__device__ __forceinline__ void stc(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stc(uint16_t* p, uint16_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stc(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stc(float2* p, float2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T ldc(const void* p) {
  using B = typename Bits<sizeof(T)>::T;
  return __builtin_bit_cast(T, *(const AMK_CONST B*)p);
}

// ---------------------------------------------------------------- numeric helpers
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float i8f(uint32_t w, int k) { return (float)(int8_t)(w >> (8 * k)); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ const T* unip(const T* p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = (uint32_t)uni((int)(uint32_t)u), hi = (uint32_t)uni((int)(uint32_t)(u >> 32));
  return (const T*)((uint64_t)hi << 32 | lo);
}
// Wait until every global load and store this wave issued has completed
// (s_waitcnt vmcnt(0)).  A barrier does not wait for them, so waves that
// store results another CU reads drain before the barrier that precedes the
// sync wave's agent-scope release.
__device__ __forceinline__ void drain_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// DPP lane moves.  Control codes: quad_perm [1,0,3,2] = 0xb1, [2,3,0,1] = 0x4e,
// row_mirror = 0x140, row_half_mirror = 0x141, row_bcast15 = 0x142,
// row_bcast31 = 0x143.  Lanes outside row_mask receive 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}

// Exchanges with lane ^ 16 and lane ^ 32 through the gfx950 row swaps: with
// both operands v, v_permlane16_swap returns (v[l], v[l ^ 16]) in even rows
// of 16 lanes and (v[l ^ 16], v[l]) in odd rows (v_permlane32_swap likewise
// for halves of 32), so one swap and one VALU op combine the two lanes.
__device__ __forceinline__ float xor16_add(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float xor16_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32_add(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float xor32_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Sum over groups of N consecutive lanes (N in 2, 4, 8, 16, 32); every lane of
// a group receives its group's sum.
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(N == 2 || N == 4 || N == 8 || N == 16 || N == 32, "group size");
  v += dpp<0xb1>(v);
  if constexpr (N >= 4) v += dpp<0x4e>(v);
  if constexpr (N >= 8) v += dpp<0x141>(v);
  if constexpr (N >= 16) v += dpp<0x140>(v);
  if constexpr (N >= 32) v = xor16_add(v);
  return v;
}
template <int N>
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp<0xb1>(v));
  if constexpr (N >= 4) v = fmaxf(v, dpp<0x4e>(v));
  if constexpr (N >= 8) v = fmaxf(v, dpp<0x141>(v));
  if constexpr (N >= 16) v = fmaxf(v, dpp<0x140>(v));
  if constexpr (N >= 32) v = xor16_max(v);
  return v;
}

// Sum over the lanes l ^ k*G of a wave (G = 8, 16 or 32: the lanes that
// share l mod G), returned to every lane.
template <int G>
__device__ __forceinline__ float across_sum(float v) {
  static_assert(G == 8 || G == 16 || G == 32 || G == 64, "group stride");
  if constexpr (G == 8) v += dpp<0x128>(v);  // row_ror:8 = lane ^ 8 within a row of 16
  if constexpr (G <= 16) v = xor16_add(v);
  if constexpr (G <= 32) v = xor32_add(v);
  return v;
}
// Full-wave sum / max, returned to every lane.
__device__ __forceinline__ float wave_sum(float v) {
  v = group_sum<16>(v);
  v += dpp<0x142, 0xa>(v);  // rows 1, 3 += last lane of rows 0, 2
  v += dpp<0x143, 0xc>(v);  // rows 2, 3 += lane 31
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  v = group_max<16>(v);
  v = xor16_max(v);
  v = xor32_max(v);
  return v;
}

// The model record is read where it lies, in the kernel-argument segment
// (uniform scalar loads through the constant cache), through a pointer that
// reopen() makes anew for the compiler at every task: held by value, its
// fields were all loaded at the kernel's start and some 260 of them lived in
// spill lanes.
typedef const AMK_CONST DevModel& ModelRef;
__device__ __forceinline__ const AMK_CONST DevModel* reopen(const AMK_CONST DevModel* p) {
  uint64_t u = (uint64_t)p;
  asm volatile("" : "+s"(u));
  return (const AMK_CONST DevModel*)u;
}

__device__ __forceinline__ bool is_gemv(int op) {
  return op == AMK_OP_QKV || op == AMK_OP_O || op == AMK_OP_GATEUP || op == AMK_OP_DOWN ||
         op == AMK_OP_LMHEAD;
}
__device__ __forceinline__ bool is_normed(int op) {
  return op == AMK_OP_QKV || op == AMK_OP_GATEUP || op == AMK_OP_LMHEAD;
}

// ---------------------------------------------------------------- LDS regions
// The task's input activation act[] is padded: element i sits at
// act_at(i) = i + 4 (i / 64), one unused float4 after every 64 floats.  A
// lane of a GEMV granule reads 8, 16 or 32 consecutive elements (bf16, int8,
// int4 weights) with float4 loads, so lanes start 32, 64 or 128 bytes apart
// and, unpadded, many lanes of one LDS access start in the same bank group
// (measured on the Llama-3-8B shape: int4 weights decode 1.3x slower
// unpadded); the padding staggers them.  A lane's elements stay inside one
// 64-float block, so its loads keep immediate offsets, and a granule's start
// c * E (E a multiple of 64) moves to c * E * 17 / 16.
// After act[]:
//   stat[...]               static epilogue data of a task of more than 64 items
//                           (epi_stat gives the layout)
//   res[...]                residual rows of the last O / down task
//   part[...]               the streaming waves' row partials / attention scratch
//   xsum[...]               W4A16: xsum[i] = sum of act[32 i .. 32 i + 31]
__device__ __forceinline__ int act_at(int i) { return i + ((i >> 6) << 2); }
// act_at(c * E + j) for a granule of E elements (a multiple of 64), j < E
template <int E>
__device__ __forceinline__ int act_gran(int c, int j) { return c * (E + E / 16) + act_at(j); }

struct Lds {
  float* act;
  float* stat;
  float* res;
  float* part;
  float* xsum;
};

// ---------------------------------------------------------------- GEMV task geometry
struct Gemv {
  int nj = 0;          // rows (jobs)
  int gpr = 1;         // granules per row
  int quant = 0;       // rows in the handle's quantised format (a tied LM head is bf16)
  int G = 0;           // total granules = nj * gpr
};

// QKV unit u: head slot u / (d/2) counts KV group by KV group, each group
// holding its query heads, then its K head, then its V head.
__device__ __forceinline__ void unit_head(ModelRef m, int u, int* mat, int* head) {
  const int slot = u >> m.half_log2;
  const int g = (int)__umulhi((uint32_t)slot, m.gq2_magic);  // slot / gq2
  const int r = slot - g * m.gq2;
  if (r < m.group) { *mat = W_Q; *head = g * m.group + r; }
  else { *mat = r == m.group ? W_K : W_V; *head = g; }
}

__device__ __forceinline__ int task_jobs_dev(int op, int n) {
  return (op == AMK_OP_QKV || op == AMK_OP_GATEUP) ? 2 * n : n;
}

__device__ __forceinline__ Gemv gemv_geom(const Ctl& ctl, int op, int n) {
  Gemv g;
  g.gpr = uni(ctl.geom[op].gpr);
  g.quant = uni(ctl.geom[op].quant);
  g.nj = task_jobs_dev(op, n);
  g.G = g.nj * g.gpr;
  return g;
}

// Granule range of streaming wave sw: [sw*G/NSW, (sw+1)*G/NSW).  G * NSW
// stays far below 2^31 (rows per task <= 1024, granules per row <= 64).
__device__ __forceinline__ int wave_gbegin(int G, int sw) { return (int)((uint32_t)(G * sw) / NSW); }

// The issue side of a wave's weight stream: the next granule to load, walking
// the rows of one task.  Rows are visited in job order: single-matrix tasks
// step one row at a time; gate / up and QKV tasks alternate between two rows
// (gate and up; the RoPE pair i, i + d/2), so the row after next is always the
// current one plus `step`.  A QKV stream that reaches the end of a head looks
// up the next one.
struct Stream {
  const uint8_t *cur = nullptr, *nxt = nullptr;    // the current row and the one after it
  const uint8_t *scur = nullptr, *snxt = nullptr;  // W4A16: their group scales
  uint32_t step = 0, sstep = 0;
  int c = 0;        // granule of the current row
  int gpr = 1;
  int lastb = 0;    // bytes of a row's last granule
  int quant = 0;
  int left = 0;     // granules of this wave's range not issued yet
  int hleft = 0;    // jobs left in the QKV head, the current one included
  int unit = 0;     // QKV: first unit of the next head
  int slot = 0;     // the task's LDS slot
};

template <int FMT>
__device__ __forceinline__ void stream_head(Stream& s, ModelRef m, const Ctl& ctl, int u, int odd) {
  int mat, head;
  unit_head(m, u, &mat, &head);
  const int i = u & (m.half - 1);
  const OpGeom& og = ctl.geom[AMK_OP_QKV];
  const uint32_t rb = (uint32_t)uni(og.row_bytes);
  const uint8_t* base = unip((const uint8_t*)ctl.slot[s.slot].ly.w[mat]);
  const uint8_t* lo = base + (size_t)(head * m.hd + i) * rb;
  const uint8_t* hi = lo + (size_t)m.half * rb;
  s.cur = odd ? hi : lo;
  s.nxt = odd ? lo + rb : hi;
  if constexpr (FMT == AMK_WEIGHTS_W4A16) {
    const uint32_t srow = (uint32_t)uni(og.srow);
    const uint8_t* sb = unip((const uint8_t*)ctl.slot[s.slot].ly.s[mat]);
    const uint8_t* slo = sb + (size_t)(head * m.hd + i) * srow;
    const uint8_t* shi = slo + (size_t)m.half * srow;
    s.scur = odd ? shi : slo;
    s.snxt = odd ? slo + srow : shi;
  }
  s.unit = u - i + m.half;
  s.hleft = 2 * (m.half - i) - odd;
}

// Start of streaming wave sw's range in the task at LDS slot k; returns its
// first job and granule, and the number of granules in s.left.
template <int FMT>
__device__ __forceinline__ void stream_begin(Stream& s, ModelRef m, const Ctl& ctl, int k, int sw, int* j0,
                                             int* c0) {
  const Slot& sl = ctl.slot[k];
  const int op = uni(sl.t.op), begin = uni(sl.t.begin), n = uni(sl.t.end) - begin;
  const OpGeom& og = ctl.geom[op];
  const uint32_t rb = (uint32_t)uni(og.row_bytes), magic = (uint32_t)uni(og.magic);
  s.slot = k;
  s.gpr = uni(og.gpr);
  s.lastb = uni(og.lastb);
  s.quant = uni(og.quant);
  const int G = task_jobs_dev(op, n) * s.gpr;
  const int g0 = wave_gbegin(G, sw);
  s.left = wave_gbegin(G, sw + 1) - g0;
  // g0 / gpr with magic = ceil(2^32 / gpr) (0 for gpr = 1)
  int j = magic ? (int)__umulhi((uint32_t)g0, magic) : g0;
  s.c = g0 - j * s.gpr;
  *j0 = j;
  *c0 = s.c;
  s.hleft = 0x7fffffff;
  if (op == AMK_OP_QKV) {
    s.step = rb;
    if constexpr (FMT == AMK_WEIGHTS_W4A16) s.sstep = (uint32_t)uni(og.srow);
    stream_head<FMT>(s, m, ctl, begin + (j >> 1), j & 1);
    return;
  }
  const bool pair = op == AMK_OP_GATEUP;
  const int mat = op == AMK_OP_O ? W_O : op == AMK_OP_DOWN ? W_D : W_G;
  const uint8_t* a = op == AMK_OP_LMHEAD ? (const uint8_t*)m.lm_w : unip((const uint8_t*)sl.ly.w[mat]);
  if (pair) {
    const uint8_t* b = unip((const uint8_t*)sl.ly.w[W_U]);
    const size_t off = (size_t)(begin + (j >> 1)) * rb;
    s.step = rb;
    s.cur = (j & 1) ? b + off : a + off;
    s.nxt = (j & 1) ? a + off + rb : b + off;
  } else {
    s.step = 2 * rb;
    s.cur = a + (size_t)(begin + j) * rb;
    s.nxt = s.cur + rb;
  }
  if constexpr (FMT == AMK_WEIGHTS_W4A16) {
    // rows of another format load a valid address instead of scales
    const uint32_t srow = (uint32_t)uni(og.srow);
    const uint8_t* sa = !s.quant ? s.cur : op == AMK_OP_LMHEAD ? (const uint8_t*)m.lm_s : unip((const uint8_t*)sl.ly.s[mat]);
    if (!s.quant) {
      s.scur = s.snxt = sa;
      s.sstep = 0;
    } else if (pair) {
      const uint8_t* sb = unip((const uint8_t*)sl.ly.s[W_U]);
      const size_t off = (size_t)(begin + (j >> 1)) * srow;
      s.sstep = srow;
      s.scur = (j & 1) ? sb + off : sa + off;
      s.snxt = (j & 1) ? sa + off + srow : sb + off;
    } else {
      s.sstep = 2 * srow;
      s.scur = sa + (size_t)(begin + j) * srow;
      s.snxt = s.scur + srow;
    }
  }
}

// Load the stream's next granule (under W4A16 with the fp16 scale of each
// lane's 32 columns; one group holds whole lanes) and step on.  The load is
// unconditional, so in the steady loop the compiler counts outstanding loads
// exactly and waits for just the oldest one (a load under a branch makes it
// drain the whole ring).  It is non-temporal: with plain loads the Llama-3-8B
// shape takes 2996 us instead of 2805 (bf16, pos 0), 1930 instead of 1791
// (W8A16, pos 100).  Past the end of the range one 16-byte vector of the
// last granule is read again and never used, and lanes past the end of a short
// row re-read the granule's start, which consume() drops.
template <int FMT>
__device__ __forceinline__ void stream_issue(Stream& s, uint4& buf, uint32_t& sc, ModelRef m, const Ctl& ctl,
                                             int lane) {
  uint32_t o = (uint32_t)lane * 16;
  const uint32_t lim = s.left <= 0 ? 16u : s.c == s.gpr - 1 ? (uint32_t)s.lastb : (uint32_t)GRAN;
  o = o < lim ? o : 0;
  buf = ldnt<uint4>(s.cur + (size_t)(uint32_t)(s.c * GRAN) + o);
  if constexpr (FMT == AMK_WEIGHTS_W4A16) sc = ldg<uint16_t>(s.scur + 2 * ((uint32_t)(s.c * GRAN4 + 2 * o) >> m.qglog2));
  if (--s.left > 0 && ++s.c == s.gpr) {
    s.c = 0;
    if (--s.hleft == 0) {
      stream_head<FMT>(s, m, ctl, s.unit, 0);
    } else {
      const uint8_t* t = s.cur + s.step;
      s.cur = s.nxt;
      s.nxt = t;
      if constexpr (FMT == AMK_WEIGHTS_W4A16) {
        const uint8_t* u = s.scur + s.sstep;
        s.scur = s.snxt;
        s.snxt = u;
      }
    }
  }
}

// The consume side: the next granule of the wave's range to reduce.
struct Work {
  int j = 0, c = 0;     // job and granule
  int left = 0;         // granules not consumed yet
  int gpr = 1, lastb = 0, quant = 0;
  float acc = 0.f;
};

template <int FMT>
__device__ __forceinline__ float dot_gran(const uint4 v, const float* __restrict__ act, int c, int lane, int quant,
                                          float acc) {
  if (FMT != AMK_WEIGHTS_W8A16 || !quant) {
    const float* x = act + act_gran<GRAN / 2>(c, lane * 8);
    const float4 a = *reinterpret_cast<const float4*>(x);
    const float4 b = *reinterpret_cast<const float4*>(x + 4);
    acc = fmaf(bf_lo(v.x), a.x, acc); acc = fmaf(bf_hi(v.x), a.y, acc);
    acc = fmaf(bf_lo(v.y), a.z, acc); acc = fmaf(bf_hi(v.y), a.w, acc);
    acc = fmaf(bf_lo(v.z), b.x, acc); acc = fmaf(bf_hi(v.z), b.y, acc);
    acc = fmaf(bf_lo(v.w), b.z, acc); acc = fmaf(bf_hi(v.w), b.w, acc);
  } else {
    const float* x = act + act_gran<GRAN>(c, lane * 16);
    const float4 a = *reinterpret_cast<const float4*>(x);
    const float4 b = *reinterpret_cast<const float4*>(x + 4);
    const float4 d = *reinterpret_cast<const float4*>(x + 8);
    const float4 e = *reinterpret_cast<const float4*>(x + 12);
    acc = fmaf(i8f(v.x, 0), a.x, acc); acc = fmaf(i8f(v.x, 1), a.y, acc);
    acc = fmaf(i8f(v.x, 2), a.z, acc); acc = fmaf(i8f(v.x, 3), a.w, acc);
    acc = fmaf(i8f(v.y, 0), b.x, acc); acc = fmaf(i8f(v.y, 1), b.y, acc);
    acc = fmaf(i8f(v.y, 2), b.z, acc); acc = fmaf(i8f(v.y, 3), b.w, acc);
    acc = fmaf(i8f(v.z, 0), d.x, acc); acc = fmaf(i8f(v.z, 1), d.y, acc);
    acc = fmaf(i8f(v.z, 2), d.z, acc); acc = fmaf(i8f(v.z, 3), d.w, acc);
    acc = fmaf(i8f(v.w, 0), e.x, acc); acc = fmaf(i8f(v.w, 1), e.y, acc);
    acc = fmaf(i8f(v.w, 2), e.z, acc); acc = fmaf(i8f(v.w, 3), e.w, acc);
  }
  return acc;
}

// One int4 granule: the lane's 32 columns [c * 2048 + 32 lane, + 32) of one
// row, times their group scale s.  Word d of the lane's 16 bytes holds
// columns 8d .. 8d + 3 in its low nibbles and 8d + 4 .. 8d + 7 in its high
// nibbles, as unsigned code + 8.  Masked (and the high ones shifted down)
// into the low nibble of each byte, a byte n read as an FP8 E4M3 value
// (exponent field 0 or 1, bias 7) is exactly n * 2^-9, so one
// v_cvt_pk_f32_fp8 turns two nibbles into floats.  Every product and partial
// sum then carries the exact factor 2^-9, which rounding commutes with, so
// the sum equals the plain fp32 one bit for bit once the factor is taken
// out.  The zero point leaves sum (code + 8) x - 8 sum x, with sum x over the
// 32 columns precomputed.
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot_gran4(const uint4 v, uint32_t sbits, const float* __restrict__ act,
                                           const float* __restrict__ xsum, int c, int lane, bool valid, float acc) {
  const float* x = act + act_gran<GRAN4>(c, lane * LANE4);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  // all 32 activations and their sum are read before any product, so the
  // LDS latency is paid once per granule
  float4 xv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) xv[i] = *reinterpret_cast<const float4*>(x + 4 * i);
  const float xs = xsum[c * (GRAN4 / LANE4) + lane];
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const float4 a = xv[2 * d], b = xv[2 * d + 1];
    const int l = (int)(w[d] & 0x0f0f0f0fu), h = (int)((w[d] >> 4) & 0x0f0f0f0fu);
    const f32x2 l01 = __builtin_amdgcn_cvt_pk_f32_fp8(l, false), l23 = __builtin_amdgcn_cvt_pk_f32_fp8(l, true);
    const f32x2 h01 = __builtin_amdgcn_cvt_pk_f32_fp8(h, false), h23 = __builtin_amdgcn_cvt_pk_f32_fp8(h, true);
    lo = fmaf(l01.x, a.x, lo); lo = fmaf(l01.y, a.y, lo);
    lo = fmaf(l23.x, a.z, lo); lo = fmaf(l23.y, a.w, lo);
    hi = fmaf(h01.x, b.x, hi); hi = fmaf(h01.y, b.y, hi);
    hi = fmaf(h23.x, b.z, hi); hi = fmaf(h23.y, b.w, hi);
  }
  const float u = (lo + hi) * 512.f;                             // sum of (code + 8) x
  const float p = fmaf(-8.f, xs, u);                             // sum of code x
  const float s = (float)__builtin_bit_cast(_Float16, (uint16_t)sbits);
  return valid ? fmaf(s, p, acc) : acc;
}

// Reduce one granule; a finished row's wave-reduced partial goes to part[j].
template <int FMT>
__device__ __forceinline__ void consume(Work& w, const uint4& buf, uint32_t sc, const Lds& L, float* __restrict__ part,
                                        int lane) {
  if (w.left <= 0) return;
  --w.left;
  const bool last = w.c == w.gpr - 1;
  const bool valid = !last || lane * 16 < w.lastb;
  if (FMT == AMK_WEIGHTS_W4A16 && w.quant) {
    w.acc = dot_gran4(buf, sc, L.act, L.xsum, w.c, lane, valid, w.acc);
  } else {
    const float r = dot_gran<FMT>(buf, L.act, w.c, lane, w.quant, w.acc);
    w.acc = valid ? r : w.acc;
  }
  ++w.c;
  if (last) {
    const float r = wave_sum(w.acc);
    if (lane == 0) part[w.j] = r;
    w.acc = 0.f;
    w.c = 0;
    ++w.j;
  }
}

// ---------------------------------------------------------------- sync wave: counters
// Acquire after a counter poll.  The polls are agent-coherent loads; what they
// order is then read with plain loads, with no cache invalidation:
//  - every vector another workgroup reads (residual stream, q, attention
//    records and output, SwiGLU output, argmax partials, the KV row at pos) is
//    written at most once per launch, and read only after all its producers
//    signalled;
//  - the launch's own acquire has invalidated every cached copy of earlier
//    launches' data;
//  - no cache line holds parts of two such vectors (256-byte strides).
// Producers' row ranges are not line-aligned: several producers, often on
// different XCDs, write parts of one 128-byte line.  This relies on the L2
// keeping written-through bytes with a byte mask: a store does not make the
// rest of its line valid, so a later read of the line by a CU of that XCD
// fetches the other producers' bytes from memory.  (The SmolLM2-shaped
// decoder, whose residual tasks own 2 or 3 rows, puts up to 16 producers in
// one line and decodes 32 greedy steps in agreement with the oracle.)
// So a line a workgroup finds in its L1 or its XCD's L2 was fetched after the
// producers had released all of it, and the XCD's L2 serves one fetch of an
// input vector to all its CUs instead of one per CU.  The fence only keeps
// the compiler from moving those loads above the poll; the hardware issues
// them after it, since leaving the poll loop depends on the loaded value.
__device__ __forceinline__ void acquire_after_poll() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

// What a wait needs, prepared one task ahead: lanes past n_wait poll the first
// counter too and never block, so the loads are unconditional and the compiler
// counts them exactly.
struct Poll {
  const uint32_t* p = nullptr;
  uint32_t target = 0;
  int nw = 0;
};
__device__ __forceinline__ Poll poll_for(ModelRef m, const amk_task_t& t, uint32_t epoch, int lane) {
  Poll w;
  w.nw = uni(t.n_wait);
  const int wl = lane < w.nw ? lane : 0;
  const int c = w.nw ? t.wait_counter[wl] : 0;
  w.p = m.counters + ((size_t)c * kCounterReplicas + blockIdx.x % kCounterReplicas) * kCounterStride;
  w.target = epoch * (uint32_t)t.wait_count[wl];
  return w;
}

// One poll in flight, the abort words every 8 (device) and 64 (host) spins: a
// second poll in flight or an abort word loaded at every spin queues before the
// poll that counts (Llama-3-8B bf16 pos 0: 2801 us a step with two polls, 2743
// so; tiny decoder 98.7 and 93.8).
__device__ __forceinline__ bool wait_deps(ModelRef m, const Poll& w, uint64_t deadline, int lane, uint64_t* tr) {
  const int nw = w.nw;
  if (nw == 0) return uni(__hip_atomic_load(m.dev_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0;
  for (uint32_t spins = 1;; ++spins) {
    const uint32_t v = __hip_atomic_load(w.p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t now = wall_clock64();
    if (__all(lane >= nw || (int32_t)(v - w.target) >= 0)) break;
    int code = 0;
    if ((spins & 7u) == 0 && uni(__hip_atomic_load(m.dev_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return false;
    // host-mapped flag: read over the bus, so only every 64 spins
    if ((spins & 63u) == 0 && uni(__hip_atomic_load(m.host_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)))
      code = AMK_ERR_ABORTED;
    else if (now > deadline)
      code = AMK_ERR_TIMEOUT;
    if (code) {
      if (lane == 0) {
        // plain stores (no read-modify-write over the bus); if two
        // workgroups stop at once, either code is a valid report
        __hip_atomic_store(m.host_status, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(m.dev_abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  if (tr && lane == 0) stg<uint64_t>(tr + AMK_TRACE_SATISFIED, (uint64_t)wall_clock64());
  acquire_after_poll();
  return true;
}

// This lane's copy of a counter (lanes past the copies: none).
__device__ __forceinline__ uint32_t* counter_copy(ModelRef m, int counter, int lane) {
  if (counter < 0 || lane >= kCounterReplicas) return nullptr;
  return m.counters + ((size_t)counter * kCounterReplicas + lane) * kCounterStride;
}

__device__ __forceinline__ void release_signal(uint32_t* copy) {
  drain_vmem();  // every published store of this wave is coherent at agent scope
  if (copy) __hip_atomic_fetch_add(copy, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Release, increment a counter, and report whether this increment brought it
// to `target` (the last producer of this launch).  The caller that gets true
// acquires before reading what the other producers released.
__device__ __forceinline__ bool release_signal_last(uint32_t* copy, uint32_t target) {
  drain_vmem();
  uint32_t old = 0;
  // copy 0's return value orders the producers
  if (copy) old = __hip_atomic_fetch_add(copy, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
  return (int32_t)(old + 1u - target) == 0;
}

// ---------------------------------------------------------------- per-row static data
// Data of a GEMV task that does not depend on this launch's results and is
// needed only in its epilogue: int8 row scales, RoPE factors, the layer-0
// embedding rows of the residual.  For a task of at most 64 items (rows, or
// row pairs) the last streaming wave loads it two tasks ahead, so nobody waits
// for these cold loads; for larger tasks (LM head) the sync wave loads it in
// the task itself, while the others compute.
struct RowStat {
  float a = 0.f, b = 0.f;  // int8 scales of the item's row(s)
  float c = 0.f, s = 0.f;  // QKV: RoPE factors;  layer-0 O: c = the embedding value
};

// Static data of item i of the task at slot sl.
__device__ __forceinline__ RowStat row_stat(ModelRef m, const Slot& sl, int op, int quant, int i, int token,
                                            int pos) {
  RowStat r;
  if (op == AMK_OP_QKV) {
    const int u = i, k = u & (m.half - 1);
    if (quant) {
      int mat, head;
      unit_head(m, u, &mat, &head);
      const float* s = (const float*)sl.ly.s[mat] + head * m.hd + k;
      r.a = ldg<float>(s);
      r.b = ldg<float>(s + m.half);
    }
    const float2 cs = ldg<float2>(m.rope + (size_t)pos * m.half + k);
    r.c = cs.x;
    r.s = cs.y;
  } else if (op == AMK_OP_GATEUP) {
    if (quant) {
      r.a = ldg<float>((const float*)sl.ly.s[W_G] + i);
      r.b = ldg<float>((const float*)sl.ly.s[W_U] + i);
    }
  } else {
    if (quant) {
      const void* s = op == AMK_OP_LMHEAD ? m.lm_s : sl.ly.s[op == AMK_OP_O ? W_O : W_D];
      r.a = ldg<float>((const float*)s + i);
    }
    if (op == AMK_OP_O && sl.t.layer == 0) r.c = bf16f(ldg<uint16_t>(m.embed + (size_t)token * m.H + i));
  }
  return r;
}

// ---------------------------------------------------------------- input activation (streaming waves)
// The task input moves into LDS in one round trip: chunk q of 64 float4s goes
// through streaming wave q mod 7 (the sync wave meanwhile prepares the
// epilogue).  Normed inputs are stored as x * gain, with each wave's sum of
// x^2 in ctl.ssq; the GEMV result is scaled by 1/sqrt(mean(x^2) + eps) in the
// epilogue (RMSNorm folded into the consumer).  The gains depend on nothing,
// so they are loaded before the wait (load_gain).  Under W4A16 each 32-column
// block's sum of the stored values goes to xsum (8 lanes hold one block).
constexpr int NGAIN = 4;  // chunks a wave preloads the gains of

__device__ __forceinline__ void load_gain(const uint16_t* gain, int n4, int sw, int lane, uint2 (&gv)[NGAIN]) {
#pragma unroll
  for (int i = 0; i < NGAIN; ++i)
    if ((sw + NSW * i) * 64 < n4) gv[i] = ldg<uint2>(gain + 4 * (size_t)min((sw + NSW * i) * 64 + lane, n4 - 1));
}

template <int FMT, int NB, bool NORM>
__device__ __forceinline__ float input_batch(const float* src, const uint2* gv, int q0, int n4, const Lds& L, int lane) {
  float4 xv[NB];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NB; ++i) xv[i] = ldg<float4>(src + 4 * (size_t)min((q0 + NSW * i) * 64 + lane, n4 - 1));
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int v = (q0 + NSW * i) * 64 + lane;
    float4 x = xv[i];
    if constexpr (NORM) {
      if (v < n4) {
        ss = fmaf(x.x, x.x, ss); ss = fmaf(x.y, x.y, ss); ss = fmaf(x.z, x.z, ss); ss = fmaf(x.w, x.w, ss);
      }
      x = make_float4(x.x * bf_lo(gv[i].x), x.y * bf_hi(gv[i].x), x.z * bf_lo(gv[i].y), x.w * bf_hi(gv[i].y));
    }
    if (v < n4) *reinterpret_cast<float4*>(L.act + act_at(v * 4)) = x;
    if constexpr (FMT == AMK_WEIGHTS_W4A16) {
      // lanes 8k .. 8k + 7 hold one block, all in range or all out
      const float blk = group_sum<8>((x.x + x.y) + (x.z + x.w));
      if (v < n4 && (lane & 7) == 0) L.xsum[v >> 3] = blk;
    }
  }
  return ss;
}

template <int FMT>
__device__ __forceinline__ void load_input(const float* src, int n4, const Lds& L, int sw, int lane) {
  const int nc = (n4 + 63) / 64;
  const int n = (nc - sw + NSW - 1) / NSW;  // chunks of this wave
  if (n <= 0) return;
  if (n == 1) input_batch<FMT, 1, false>(src, nullptr, sw, n4, L, lane);
  else if (n == 2) input_batch<FMT, 2, false>(src, nullptr, sw, n4, L, lane);
  else if (n <= 4) input_batch<FMT, 4, false>(src, nullptr, sw, n4, L, lane);
  else
    for (int q = sw; q < nc; q += 8 * NSW) input_batch<FMT, 8, false>(src, nullptr, q, n4, L, lane);
}

template <int FMT>
__device__ __forceinline__ void load_input_normed(const float* src, const uint16_t* src_bf, const uint16_t* gain, int n4,
                                                  uint2 (&gv)[NGAIN], const Lds& L, Ctl& ctl, int sw, int lane) {
  const int nc = (n4 + 63) / 64;
  const int n = (nc - sw + NSW - 1) / NSW;
  float ss = 0.f;
  if (src_bf) {  // layer 0: the embedding row
    for (int q = sw; q < nc; q += NSW) {
      const int v = q * 64 + lane, vc = min(v, n4 - 1);
      const uint2 r = ldg<uint2>(src_bf + (size_t)vc * 4), g = ldg<uint2>(gain + (size_t)vc * 4);
      float4 x = make_float4(bf_lo(r.x), bf_hi(r.x), bf_lo(r.y), bf_hi(r.y));
      if (v < n4) {
        ss = fmaf(x.x, x.x, ss); ss = fmaf(x.y, x.y, ss); ss = fmaf(x.z, x.z, ss); ss = fmaf(x.w, x.w, ss);
      }
      x = make_float4(x.x * bf_lo(g.x), x.y * bf_hi(g.x), x.z * bf_lo(g.y), x.w * bf_hi(g.y));
      if (v < n4) *reinterpret_cast<float4*>(L.act + act_at(v * 4)) = x;
      if constexpr (FMT == AMK_WEIGHTS_W4A16) {
        const float blk = group_sum<8>((x.x + x.y) + (x.z + x.w));
        if (v < n4 && (lane & 7) == 0) L.xsum[v >> 3] = blk;
      }
    }
  } else if (n == 1) {
    ss = input_batch<FMT, 1, true>(src, gv, sw, n4, L, lane);
  } else if (n == 2) {
    ss = input_batch<FMT, 2, true>(src, gv, sw, n4, L, lane);
  } else if (n > 2) {
    ss = input_batch<FMT, NGAIN, true>(src, gv, sw, n4, L, lane);
    for (int q = sw + NSW * NGAIN; q < nc; q += NSW) {  // hidden sizes past 7168
      const uint2 g1[1] = {ldg<uint2>(gain + 4 * (size_t)min(q * 64 + lane, n4 - 1))};
      ss += input_batch<FMT, 1, true>(src, g1, q, n4, L, lane);
    }
  }
  ss = wave_sum(ss);
  if (lane == 0) ctl.ssq[sw] = ss;
}

__device__ __forceinline__ float input_rs(ModelRef m, const Ctl& ctl) {
  float ss = 0.f;
#pragma unroll
  for (int w = 0; w < NSW; ++w) ss += ctl.ssq[w];
  return 1.0f / sqrtf(ss / (float)m.H + m.eps);
}

// ---------------------------------------------------------------- row sums of a GEMV task
// Granule boundaries of the streaming waves, computed while they compute.
struct Ranges {
  int b[NSW + 1];
};
__device__ __forceinline__ Ranges wave_ranges(const Gemv& g) {
  Ranges r;
#pragma unroll
  for (int sw = 0; sw <= NSW; ++sw) r.b[sw] = wave_gbegin(g.G, sw);
  return r;
}

// Wave sw's partial of row j lies at part[sw + j]: the waves' ranges follow each
// other and neighbours share at most one row, so no two partials share a word.
__device__ __forceinline__ float row_sum(const float* part, const Gemv& g, const Ranges& wr, int j) {
  const int lo = j * g.gpr, hi = lo + g.gpr;
  // every wave's slot is read (all reads in flight at once), the ones of
  // waves that wrote nothing for row j are dropped: a wave with an empty
  // range wrote nothing, even if its start lies inside the row
  float v[NSW];
#pragma unroll
  for (int sw = 0; sw < NSW; ++sw) v[sw] = part[sw + j];
  float s = 0.f;
#pragma unroll
  for (int sw = 0; sw < NSW; ++sw) s += max(wr.b[sw], lo) < min(wr.b[sw + 1], hi) ? v[sw] : 0.f;
  return s;
}

// ---------------------------------------------------------------- sync wave: epilogues
// What the sync wave holds for the epilogue of a task of more than 64 items.
struct Epi {
  Gemv g;
  Ranges wr;
  float rs;         // RMSNorm factor of normed inputs
  int layer, begin, end, aux;
};
// Residual rows cached in LDS: x buffer index and row range.
struct Res {
  int buf = -1, lo = 0, hi = 0;
};

// Static data of item i in LDS: per item four floats for QKV, two for gate / up (a, b) and for the residual
// ops (a, c), one for the LM head (a).
template <int OP>
__device__ __forceinline__ RowStat epi_stat(const Epi& e, const Lds& L, int i) {
  RowStat r;
  const int k = i - e.begin;
  if constexpr (OP == AMK_OP_QKV) {
    const float4 v = *reinterpret_cast<const float4*>(L.stat + 4 * k);
    r.a = v.x; r.b = v.y; r.c = v.z; r.s = v.w;
  } else if constexpr (OP == AMK_OP_GATEUP) {
    r.a = L.stat[2 * k]; r.b = L.stat[2 * k + 1];
  } else if constexpr (OP == AMK_OP_O) {
    r.a = L.stat[2 * k]; r.c = L.stat[2 * k + 1];
  } else {
    r.a = L.stat[k];
  }
  return r;
}
__device__ __forceinline__ void put_stat(const Lds& L, int op, int k, const RowStat& r) {
  if (op == AMK_OP_QKV) {
    *reinterpret_cast<float4*>(L.stat + 4 * k) = make_float4(r.a, r.b, r.c, r.s);
  } else if (op == AMK_OP_LMHEAD) {
    L.stat[k] = r.a;
  } else {
    L.stat[2 * k] = r.a;
    L.stat[2 * k + 1] = op == AMK_OP_GATEUP ? r.b : r.c;
  }
}

__device__ __forceinline__ void epi_qkv(ModelRef m, const Epi& e, const Lds& L, int pos, uint16_t* kv,
                                        int lane) {
  const int l = e.layer;
  for (int u = e.begin + lane; u < e.end; u += 64) {
    const int j0 = 2 * (u - e.begin);
    float y0 = row_sum(L.part, e.g, e.wr, j0) * e.rs;
    float y1 = row_sum(L.part, e.g, e.wr, j0 + 1) * e.rs;
    const RowStat st = epi_stat<AMK_OP_QKV>(e, L, u);
    if (m.fmt == AMK_WEIGHTS_W8A16) {
      y0 *= st.a;
      y1 *= st.b;
    }
    int mat, head;
    unit_head(m, u, &mat, &head);
    const int i = u & (m.half - 1);
    if (mat != W_V) {
      const float a = y0 * st.c - y1 * st.s;
      const float b = y1 * st.c + y0 * st.s;
      y0 = a;
      y1 = b;
    }
    if (mat == W_Q) {
      float* qd = m.q + (size_t)l * m.qs + (size_t)head * m.hd;
      stc(qd + i, y0);
      stc(qd + i + m.half, y1);
    } else {
      const int which = (mat == W_K) ? 0 : 1;
      uint16_t* dst = kv + (((size_t)(l * 2 + which) * m.nkv + head) * m.max_seq + pos) * m.hd;
      stc(dst + i, f2bf(y0));
      stc(dst + i + m.half, f2bf(y1));
    }
  }
}

// O and down projections: x_out = x_in + W y, with x_in rows taken from LDS
// when this workgroup's previous residual task produced exactly those rows.
__device__ __forceinline__ void epi_residual(ModelRef m, const Epi& e, Res& res, int op, const Lds& L, int lane) {
  const int xin = op == AMK_OP_O ? 2 * e.layer : 2 * e.layer + 1;
  const bool cached = res.buf == xin && res.lo == e.begin && res.hi == e.end;
  for (int r = e.begin + lane; r < e.end; r += 64) {
    float y = row_sum(L.part, e.g, e.wr, r - e.begin);
    const RowStat st = epi_stat<AMK_OP_O>(e, L, r);
    if (m.fmt == AMK_WEIGHTS_W8A16) y *= st.a;
    const float x = xin == 0 ? st.c : cached ? L.res[r - e.begin] : ldg<float>(m.x + (size_t)xin * m.xs + r);
    const float o = x + y;
    stc(m.x + (size_t)(xin + 1) * m.xs + r, o);
    L.res[r - e.begin] = o;
  }
  res.buf = xin + 1;
  res.lo = e.begin;
  res.hi = e.end;
}

__device__ __forceinline__ void epi_gateup(ModelRef m, const Epi& e, const Lds& L, int lane) {
  for (int r = e.begin + lane; r < e.end; r += 64) {
    const int j = 2 * (r - e.begin);
    float gv = row_sum(L.part, e.g, e.wr, j) * e.rs;
    float uv = row_sum(L.part, e.g, e.wr, j + 1) * e.rs;
    if (m.fmt == AMK_WEIGHTS_W8A16) {
      const RowStat st = epi_stat<AMK_OP_GATEUP>(e, L, r);
      gv *= st.a;
      uv *= st.b;
    }
    const float silu = gv / (1.0f + __expf(-gv));
    stc(m.a + (size_t)e.layer * m.as + r, silu * uv);
  }
}

// LM head: logits + per-task argmax partial (lowest index on ties).  A NaN
// logit never wins a comparison; it records the sticky status
// AMK_ERR_NONFINITE, so the step's next token is reported as meaningless
// instead of silently skipping it.
__device__ __forceinline__ void epi_lmhead(ModelRef m, const Epi& e, const Lds& L, float* logits, int lane) {
  float best = -INFINITY;
  int besti = 0x7fffffff;
  bool nan = false;
  for (int r = e.begin + lane; r < e.end; r += 64) {
    float y = row_sum(L.part, e.g, e.wr, r - e.begin) * e.rs;
    if (m.lm_fmt == AMK_WEIGHTS_W8A16) y *= epi_stat<AMK_OP_LMHEAD>(e, L, r).a;
    stc(logits + r, y);
    nan |= y != y;
    if (y > best || (y == best && r < besti)) { best = y; besti = r; }
  }
  if (__any(nan) && lane == 0)
    __hip_atomic_store(m.host_status, (int32_t)AMK_ERR_NONFINITE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o);
    const int oi = __shfl_xor(besti, o);
    if (ob > best || (ob == best && oi < besti)) { best = ob; besti = oi; }
  }
  if (lane == 0) stc(reinterpret_cast<float2*>(m.argp + 2 * e.aux), make_float2(best, __int_as_float(besti)));
}

// Epilogue of a task of at most 64 items, one item per lane, in two halves.
// Everything that does not need the row sums (addresses, which waves' partials
// count, factors) is prepared by the last streaming wave while the task before
// it is handed over, and left in ctl.prep; after B2, on the path every consumer
// waits for, the sync wave only sums the partials, scales and stores.  (In one
// piece on the sync wave the epilogue took 0.65-0.85 us of a 4.2 us stage of
// the tiny decoder; so it takes 0.24-0.36 us of a stage in the short and long
// schedules, and 0.8-1.2 us with the drain and the signal in the tiny one.)
struct Fast {
  float f0, f1;      // int8 scales (1 otherwise)
  float c, s;        // RoPE factors, or the layer-0 residual in c
  uint64_t d0;       // where the (first) result goes, then
  uint32_t d1;       // the second one's distance in bytes
  uint32_t bits;     // 7 bits of waves whose partial of the first row counts, 7 of the second's, then:
  enum { WIDE = 1 << 14, ROT = 1 << 15 };  // fp32 result (appended K / V: bf16); RoPE applies (q and K)
};
static_assert(sizeof(Fast) == 32, "two float4s");

__device__ __forceinline__ uint32_t row_bits(const Gemv& g, const Ranges& wr, int j) {
  const int lo = j * g.gpr, hi = lo + g.gpr;
  uint32_t b = 0;
#pragma unroll
  for (int sw = 0; sw < NSW; ++sw) b |= max(wr.b[sw], lo) < min(wr.b[sw + 1], hi) ? 1u << sw : 0u;
  return b;
}

__device__ __forceinline__ Fast fast_prepare(ModelRef m, const Ctl& ctl, const amk_task_t& t, int op, const RowStat& st,
                                             int pos, uint16_t* kv, int lane) {
  Fast f;
  const int layer = uni(t.layer), begin = uni(t.begin), n = uni(t.end) - begin;
  const int i = begin + min(lane, n - 1);
  const bool pair = op == AMK_OP_QKV || op == AMK_OP_GATEUP;
  const Gemv g = gemv_geom(ctl, op, n);
  const Ranges wr = wave_ranges(g);
  f.bits = row_bits(g, wr, pair ? 2 * lane : lane);
  if (pair) f.bits |= row_bits(g, wr, 2 * lane + 1) << NSW;
  const bool int8 = m.fmt == AMK_WEIGHTS_W8A16;
  f.f0 = int8 ? st.a : 1.f;
  f.f1 = int8 ? st.b : 1.f;
  f.c = st.c;
  f.s = st.s;
  f.d1 = 0;
  if (op == AMK_OP_QKV) {
    int mat, head;
    unit_head(m, i, &mat, &head);
    const int k = i & (m.half - 1);
    if (mat != W_V) f.bits |= Fast::ROT;
    if (mat == W_Q) {
      f.bits |= Fast::WIDE;
      f.d0 = (uint64_t)(m.q + (size_t)layer * m.qs + (size_t)head * m.hd + k);
      f.d1 = (uint32_t)m.half * 4;
    } else {
      f.d0 = (uint64_t)(kv + (((size_t)(layer * 2 + (mat == W_K ? 0 : 1)) * m.nkv + head) * m.max_seq + pos) * m.hd + k);
      f.d1 = (uint32_t)m.half * 2;
    }
  } else if (op == AMK_OP_GATEUP) {
    f.d0 = (uint64_t)(m.a + (size_t)layer * m.as + i);
  } else {
    f.d0 = (uint64_t)(m.x + (size_t)(2 * layer + (op == AMK_OP_O ? 1 : 2)) * m.xs + i);
  }
  return f;
}

__device__ __forceinline__ float masked_sum(const float* part, uint32_t bits, int j) {
  uint32_t v[NSW];
#pragma unroll
  for (int sw = 0; sw < NSW; ++sw) v[sw] = __float_as_uint(part[sw + j]);
  float s = 0.f;
#pragma unroll
  for (int sw = 0; sw < NSW; ++sw) s += __uint_as_float(v[sw] & (uint32_t)((int)(bits << (31 - sw)) >> 31));
  return s;
}

__device__ __forceinline__ void fast_finish(int op, int n, const Fast& f, float rs, const Lds& L, int lane) {
  if (lane >= n) return;
  if (op == AMK_OP_QKV) {
    const float y0 = masked_sum(L.part, f.bits, 2 * lane) * rs * f.f0;
    const float y1 = masked_sum(L.part, f.bits >> NSW, 2 * lane + 1) * rs * f.f1;
    const bool rot = f.bits & Fast::ROT;
    const float a = rot ? y0 * f.c - y1 * f.s : y0;
    const float b = rot ? y1 * f.c + y0 * f.s : y1;
    if (f.bits & Fast::WIDE) {
      stc((float*)f.d0, a);
      stc((float*)(f.d0 + f.d1), b);
    } else {
      stc((uint16_t*)f.d0, f2bf(a));
      stc((uint16_t*)(f.d0 + f.d1), f2bf(b));
    }
  } else if (op == AMK_OP_GATEUP) {
    const float gv = masked_sum(L.part, f.bits, 2 * lane) * rs * f.f0;
    const float uv = masked_sum(L.part, f.bits >> NSW, 2 * lane + 1) * rs * f.f1;
    const float silu = gv / (1.0f + __expf(-gv));
    stc((float*)f.d0, silu * uv);
  } else {
    const float o = f.c + masked_sum(L.part, f.bits, lane) * f.f0;
    stc((float*)f.d0, o);
    L.res[lane] = o;
  }
}

__device__ __forceinline__ void argmax_final(ModelRef m, int begin, int end, int lane) {
  float best = -INFINITY;
  int besti = 0x7fffffff;
  for (int s = begin + lane; s < end; s += 64) {
    const float2 vi = ldg<float2>(m.argp + 2 * s);
    const int i = __float_as_int(vi.y);
    if (vi.x > best || (vi.x == best && i < besti)) { best = vi.x; besti = i; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o);
    const int oi = __shfl_xor(besti, o);
    if (ob > best || (ob == best && oi < besti)) { best = ob; besti = oi; }
  }
  if (lane == 0) stc(m.next_token, besti);
}

// ---------------------------------------------------------------- attention (all 8 waves)
// Geometry of the attention of one KV group, shared with the host's LDS
// sizing.  HD: head dim; GM: largest query group handled.  A tile is 16 K/V
// rows; a wave holds up to T tiles per pass with all their loads in flight, so
// one pass of the workgroup covers T * 16 * NW rows (384 for groups of at
// most four heads).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int HD, int GM>
struct AttnGeom {
  static constexpr int T = GM == 4 ? 3 : HD == 64 ? 2 : 1;  // what the registers hold
  static constexpr int HS = GM / 4;      // sets of four query heads
  static constexpr int KL = HD / 32;     // 16-byte loads per lane of a K tile, and of a V tile
  static constexpr int VR = 512 / HD;    // rows per V load
  static constexpr int RP = T * 16 * NW;
  // LDS scratch (floats): per-wave accumulators red[NW][GM][HD] and running
  // (max, sum) stat[NW][GM][2]; a wave's softmax weights lie in its part of
  // red until it stores its accumulators; the split merge reuses the region
  static constexpr int SCRATCH = NW * GM * HD + 2 * NW * GM;
  static constexpr int MERGE = GM * 64 + 4 * NT;
  static constexpr int LDS = SCRATCH > MERGE ? SCRATCH : MERGE;
  static_assert(GM % 4 == 0 && T * 16 * GM <= GM * HD, "the weights of a pass fit a wave's part of red");
};

__device__ __forceinline__ float row_elem(const uint4& v, int e) {
  const uint32_t w = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
  return (e & 1) ? bf_hi(w) : bf_lo(w);
}

// Attention of the query heads of KV group g over positions [j0, j1) of
// layer `layer` (j1 > j0), scores q.k / sqrt(d), max-subtracted softmax,
// V-weighted sum (paper §2 "Kernel authoring and attention" names the
// flash-decoding family this follows).  Every wave keeps its own running
// max / sum / accumulators over the rows it loads (online softmax, no
// barrier inside the position loop); the waves merge through LDS at the end.
//
// Scores on the matrix cores: a tile's 16 K rows are the A operand of
// v_mfma_f32_16x16x32_bf16 as they lie in the cache (lane l: row l % 16, 16
// bytes), the B operand holds four query heads, each fp32 query cut into three
// bf16 parts of 8 significant bits in columns h, 4 + h and 8 + h (columns 12
// to 15 are zero).  Cut by truncation the three parts add up to the fp32 value
// exactly, and a product of two 8-bit significands is exact in fp32, so the
// sums differ from fp32 products only in their order.  On the vector units
// the scores took 24 of 39 instructions per row.  The later parts are often 0
// and the last columns always, and 0 times an infinite K element is NaN: those
// columns count only where they are finite, and the first part's column, whose
// parts are 0 only where the query is, then gives the +-inf or NaN of the fp32
// product (a K row with a score of -inf has weight 0).
// The queries are pre-multiplied by log2(e) / sqrt(d), so scores and
// maxima are in log2 units and each softmax weight is one exp2: the same
// weights as exp(q.k / sqrt(d) - max), up to fp32 rounding.  The weights
// stay fp32 (through LDS, where a V row's lanes read all heads at once).
// `record`: store per head (m, l, unnormalised acc) at dst[h * (kPartHead +
// d)], else the normalised output at dst[h * d].  Stores are issued by every
// wave; the caller drains them.
template <int HD, int GM>
__device__ __forceinline__ void attention(ModelRef m, int layer, int g, int j0, int j1, const uint16_t* __restrict__ kv,
                                          float* __restrict__ qs, float* __restrict__ scr, float* __restrict__ dst,
                                          bool record, int wave, int lane) {
  using A = AttnGeom<HD, GM>;
  constexpr int T = A::T, HS = A::HS, KL = A::KL, VR = A::VR, RP = A::RP, LPR = HD / 8;
  const int G = m.group;
  const int n = j1 - j0;
  const int col = lane & 15, quad = lane >> 4;
  const int sub = lane / LPR, c = lane % LPR;  // V: row within a load, 8-dim block
  const size_t hs = (size_t)m.max_seq * HD;
  // uniform bases, of row w0, and 32-bit byte offsets per lane from them; the
  // bases move on every WINDOW rows (a head's rows may take more than 2^32 bytes)
  constexpr int WINDOW = 1 << 16;
  static_assert((WINDOW + RP) * (2 * HD) < 1 << 30, "byte offsets from the bases");
  const uint8_t* Kp = (const uint8_t*)(kv + ((size_t)(layer * 2 + 0) * m.nkv + g) * hs + (size_t)j0 * HD);
  const uint8_t* Vp = (const uint8_t*)(kv + ((size_t)(layer * 2 + 1) * m.nkv + g) * hs + (size_t)j0 * HD);
  float* red = scr;                   // [NW][GM][HD]
  float* stat = scr + NW * GM * HD;   // [NW][GM][2]
  float* wts = red + wave * GM * HD;  // this wave's weights: [HS][T * 16 rows][4 heads]

  float m_run[HS], l_run[HS], acc[GM][8];
#pragma unroll
  for (int s = 0; s < HS; ++s) {
    m_run[s] = -INFINITY;
    l_run[s] = 0.f;
  }
#pragma unroll
  for (int h = 0; h < GM; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.f;

  const bool active = wave * 16 < n;  // this wave has rows
  // Long splits load their rows past the caches like the weights.  us a step,
  // plain / non-temporal, with the rows cold (three models decoded in turn):
  // Llama-3.2-1B W8A16, 64 / 96 / 129 rows a split: 637 / 640, 656 / 649, 667 /
  // 656; TinyLlama bf16, 48 / 64 / 96: 871 / 874, 880 / 875, 909 / 898; SmolLM2
  // bf16, 32 / 64 / 96: 743 / 748, 760 / 749, 785 / 766.  Where one context is
  // decoded on, the memory-side cache holds its rows until they outgrow its 256
  // MB, and plain loads win: the same at 96 rows 644 / 651, 888 / 899 and 756 /
  // 768, at 128 rows 648 / 654, 893 / 904 and 763 / 773; 8B bf16 at 96 and 256
  // rows (403 and 1074 MB) 2983 / 2957 and 3072 / 3053.  At 96 rows what the
  // cold rows gain outweighs or equals what the cached ones lose.  A group's rows
  // in one task (no record) are slower non-temporally at any length (SmolLM2,
  // 201 rows: 656 / 672; 8B, 8192: 6246 / 6725).
  const bool nt = record && n >= 96;
  // a thread's queries (one or two of the group's G * HD), loaded ahead of the
  // rows; each is cut once and its parts go to qs[part][G * HD] as bf16
  const int tid = wave * 64 + lane;
  const float* qp = m.q + (size_t)layer * m.qs + (size_t)(g * G) * HD;
  const float qscale = m.attn_scale * 1.4426950408889634f;  // log2(e) / sqrt(d)
  // what columns past the first part's never add to a score: NaN and infinities
  // (v_cmp_class bits 0 to 2 and 9)
  const int not_first = col < 4 ? 0 : 0x207;
  constexpr int QN = GM * HD > NT ? 2 : 1;
  float qv[QN];
#pragma unroll
  for (int i = 0; i < QN; ++i) qv[i] = ldg<float>(qp + min(tid + i * NT, G * HD - 1));
  bf16x8 qf[HS][KL];

  int w0 = 0;
  for (int p0 = 0; p0 < n; p0 += RP) {
    if (p0 - w0 >= WINDOW) {
      Kp += (size_t)(p0 - w0) * (2 * HD);
      Vp += (size_t)(p0 - w0) * (2 * HD);
      w0 = p0;
    }
    // tile t of this wave: rows p0 + (t * NW + wave) * 16 ..; rows past the
    // range re-read its last row, whose weight is set to 0
    uint4 kr[T][KL], vr[T][KL];
    auto load_v = [&](int t, int tb) {
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        const uint32_t vo = (uint32_t)((min(tb + j * VR + sub, n - 1) - w0) * (2 * HD) + c * 16);
        vr[t][j] = nt ? ldnt<uint4>(Vp + vo) : ldg<uint4>(Vp + vo);
      }
    };
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int tb = p0 + (t * NW + wave) * 16;
      if (tb < n) {
        const uint32_t ko = (uint32_t)((min(tb + col, n - 1) - w0) * (2 * HD) + quad * 16);
#pragma unroll
        for (int kb = 0; kb < KL; ++kb) kr[t][kb] = nt ? ldnt<uint4>(Kp + ko + kb * 64) : ldg<uint4>(Kp + ko + kb * 64);
        if (t == 0) load_v(t, tb);
      }
    }
    if (p0 == 0) {
      uint16_t* qb = reinterpret_cast<uint16_t*>(qs);
#pragma unroll
      for (int i = 0; i < QN; ++i) {
        const float x = qv[i] * qscale;
        const float y = x - __uint_as_float(__float_as_uint(x) & 0xffff0000u);
        const float z = y - __uint_as_float(__float_as_uint(y) & 0xffff0000u);
        if (tid + i * NT < G * HD) {
          qb[tid + i * NT] = (uint16_t)(__float_as_uint(x) >> 16);
          qb[G * HD + tid + i * NT] = (uint16_t)(__float_as_uint(y) >> 16);
          qb[2 * G * HD + tid + i * NT] = (uint16_t)(__float_as_uint(z) >> 16);
        }
      }
      __syncthreads();
      // column col: part col / 4 of head col % 4 of the set, dims kb * 32 +
      // quad * 8 ..; no such part or head: zero
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        const int h = s * 4 + (col & 3), part = col >> 2;
        const bool on = part < 3 && h < G;
        const uint16_t* qf0 = qb + (on ? part * G + h : 0) * HD + quad * 8;
#pragma unroll
        for (int kb = 0; kb < KL; ++kb) {
          const uint4 v = *reinterpret_cast<const uint4*>(qf0 + kb * 32);
          qf[s][kb] = __builtin_bit_cast(bf16x8, make_uint4(on ? v.x : 0, on ? v.y : 0, on ? v.z : 0, on ? v.w : 0));
        }
      }
    }
    f32x4 sv[HS][T];
    float mx[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) mx[s] = -INFINITY;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int tb = p0 + (t * NW + wave) * 16;
      if (tb < n) {
#pragma unroll
        for (int s = 0; s < HS; ++s) {
          f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kb = 0; kb < KL; ++kb)
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[t][kb]), qf[s][kb], d, 0, 0, 0);
          // lane: column col, rows quad * 4 + i; add the parts' columns
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float v = __builtin_amdgcn_classf(d[i], not_first) ? 0.f : d[i];
            v += dpp<0x128>(v);  // row_ror:8
            v += dpp<0x124>(v);  // row_ror:4
            v = tb + quad * 4 + i < n ? v : -INFINITY;
            sv[s][t][i] = v;
            mx[s] = fmaxf(mx[s], v);
          }
        }
      }
    }
    // the V rows past the first tile take the K rows' registers
#pragma unroll
    for (int t = 1; t < T; ++t)
      if (p0 + (t * NW + wave) * 16 < n) load_v(t, p0 + (t * NW + wave) * 16);
    // one online-softmax update per head (lane's head: col % 4 of the set)
    float alpha[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) {
      const float m_new = fmaxf(m_run[s], xor32_max(xor16_max(mx[s])));
      // a wave that has seen no row keeps (-inf, 0, 0)
      const float mref = m_new == -INFINITY ? 0.f : m_new;
      alpha[s] = __builtin_amdgcn_exp2f(m_run[s] - mref);
      float ls = 0.f;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if (p0 + (t * NW + wave) * 16 < n) {
          float w[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            w[i] = __builtin_amdgcn_exp2f(sv[s][t][i] - mref);
            ls += w[i];
          }
          // the four columns of a head hold the same weights: column 4 i + h
          // stores row quad * 4 + i, so the tile lies linear in lane order
          const int i = col >> 2;
          wts[(s * T + t) * 64 + lane] = i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : w[3];
        }
      }
      l_run[s] = l_run[s] * alpha[s] + ls;
      m_run[s] = m_new;
    }
    if (p0 > 0) {
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        const float al = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha[h / 4]), h & 3));
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] *= al;
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (p0 + (t * NW + wave) * 16 < n) {
#pragma unroll
        for (int j = 0; j < KL; ++j) {
          float vf[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) vf[e] = row_elem(vr[t][j], e);
#pragma unroll
          for (int s = 0; s < HS; ++s) {
            const float4 w = *reinterpret_cast<const float4*>(wts + (s * T + t) * 64 + (j * VR + sub) * 4);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              acc[4 * s][e] = fmaf(w.x, vf[e], acc[4 * s][e]);
              acc[4 * s + 1][e] = fmaf(w.y, vf[e], acc[4 * s + 1][e]);
              acc[4 * s + 2][e] = fmaf(w.z, vf[e], acc[4 * s + 2][e]);
              acc[4 * s + 3][e] = fmaf(w.w, vf[e], acc[4 * s + 3][e]);
            }
          }
        }
      }
    }
  }

  // per wave: sum the accumulators over the row groups, two registers to one
  // at each exchange, which leaves dims c * 8 + 2 * quad + {0, 1} of every head
  // to a lane; then merge the waves
#pragma unroll
  for (int s = 0; s < HS; ++s) l_run[s] = across_sum<16>(l_run[s]);
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    if (h < G) {
      if (active) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if constexpr (LPR == 8) acc[h][e] += dpp<0x128>(acc[h][e]);  // row_ror:8
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[h][e]), __float_as_uint(acc[h][e + 4]), false, false);
          v[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[e]), __float_as_uint(v[e + 2]), false, false);
          v[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        *reinterpret_cast<float2*>(red + (wave * GM + h) * HD + c * 8 + 2 * quad) = make_float2(v[0], v[1]);
      }
      if (lane == (h & 3)) {
        stat[(wave * GM + h) * 2] = m_run[h / 4];
        stat[(wave * GM + h) * 2 + 1] = l_run[h / 4];
      }
    }
  }
  __syncthreads();
  for (int i = wave * 64 + lane; i < G * HD; i += NT) {
    const int h = i / HD, d = i - h * HD;
    float2 ml[NW];
    float r[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      ml[w] = *reinterpret_cast<const float2*>(stat + (w * GM + h) * 2);
      r[w] = red[(w * GM + h) * HD + d];
    }
    float M = ml[0].x;
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, ml[w].x);
    // rows that all score -inf leave (-inf, 0, 0), which weighs 0 in a merge
    const float mref = M == -INFINITY ? 0.f : M;
    float l = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // a wave without rows left (-inf, 0) and no accumulators
      const float f = __builtin_amdgcn_exp2f(ml[w].x - mref);
      l = fmaf(f, ml[w].y, l);
      o = fmaf(f, ml[w].x == -INFINITY ? 0.f : r[w], o);
    }
    if (record) {
      float* rec = dst + h * (kPartHead + HD);
      stc(rec + kPartHead + d, o);
      // the record's maximum in natural-log units, as the split merge reads it
      if (d == 0) stc(reinterpret_cast<float2*>(rec), make_float2(M * 0.6931471805599453f, l));
    } else {
      stc(dst + h * HD + d, o / l);
    }
  }
}

// Attention of every query head over positions [0, pos] (pos < AMK_TINY_MAX)
// into act[h * HD + d]: the input of an O task of the tiny schedule, which
// computes it itself instead of waiting for an attention stage.  Each wave
// takes HR heads per round; lane owns head dims [lane * DPL, (lane + 1) * DPL).
// All q / K / V loads of a round go out before any arithmetic, once per KV
// group.
template <int HD, int FMT>
__device__ __forceinline__ void attention_all(ModelRef m, int layer, int pos, const uint16_t* __restrict__ kv,
                                              float* __restrict__ act, float* __restrict__ xsum, int wave,
                                              int lane) {
  constexpr int DPL = HD / 64;
  constexpr int HR = 4;
  constexpr int T = AMK_TINY_MAX;
  const int n = pos + 1;
  const size_t hs = (size_t)m.max_seq * HD;
  // the HR heads of a round share one KV group when the group size is a
  // multiple of HR (heads h0.. h0 + HR - 1 with h0 a multiple of HR)
  const int group = m.group;
  const bool one_group = (group & (HR - 1)) == 0;
  const float scale = m.attn_scale;
  for (int h0 = wave * HR; h0 < m.nq; h0 += NW * HR) {
    float qv[HR][DPL];
    uint32_t kr[HR][T] = {}, vr[HR][T] = {};  // DPL bf16 values per row (the low half only when DPL == 1)
#pragma unroll
    for (int i = 0; i < HR; ++i) {
      const int h = min(h0 + i, m.nq - 1);
      const int g = (int)__umulhi((uint32_t)h, m.group_magic) + (group == 1 ? h : 0);  // h / group
      const float* qh = m.q + (size_t)layer * m.qs + (size_t)h * HD + lane * DPL;
      const uint16_t* Kp = kv + ((size_t)(layer * 2) * m.nkv + g) * hs + lane * DPL;
      const uint16_t* Vp = kv + ((size_t)(layer * 2 + 1) * m.nkv + g) * hs + lane * DPL;
      if constexpr (DPL == 2) {
        const float2 q2 = ldg<float2>(qh);
        qv[i][0] = q2.x;
        qv[i][1] = q2.y;
      } else {
        qv[i][0] = ldg<float>(qh);
      }
      // one load per KV group (the other heads of the group copy it below)
      if (i > 0 && one_group) continue;
#pragma unroll
      for (int p = 0; p < T; ++p) {
        if (p < n) {
          if constexpr (DPL == 2) {
            kr[i][p] = ldg<uint32_t>(Kp + p * HD);
            vr[i][p] = ldg<uint32_t>(Vp + p * HD);
          } else {
            kr[i][p] = ldg<uint16_t>(Kp + p * HD);
            vr[i][p] = ldg<uint16_t>(Vp + p * HD);
          }
        }
      }
    }
    if (one_group) {
#pragma unroll
      for (int i = 1; i < HR; ++i)
#pragma unroll
        for (int p = 0; p < T; ++p) {
          kr[i][p] = kr[0][p];
          vr[i][p] = vr[0][p];
        }
    }
#pragma unroll
    for (int i = 0; i < HR; ++i) {
      float mrun = -INFINITY, l = 0.f, acc[DPL];
#pragma unroll
      for (int j = 0; j < DPL; ++j) acc[j] = 0.f;
#pragma unroll
      for (int p = 0; p < T; ++p) {
        if (p < n) {
          float d = qv[i][0] * bf_lo(kr[i][p]);
          if constexpr (DPL == 2) d = fmaf(qv[i][1], bf_hi(kr[i][p]), d);
          d = wave_sum(d) * scale;
          const float mn = fmaxf(mrun, d);
          const float mref = mn == -INFINITY ? 0.f : mn;  // only scores of -inf so far: weight 0
          const float alpha = __expf(mrun - mref), e = __expf(d - mref);
          l = l * alpha + e;
          acc[0] = fmaf(e, bf_lo(vr[i][p]), acc[0] * alpha);
          if constexpr (DPL == 2) acc[1] = fmaf(e, bf_hi(vr[i][p]), acc[1] * alpha);
          mrun = mn;
        }
      }
      const int h = h0 + i;
      if (h < m.nq) {
        const float inv = 1.0f / l;
        float blk = 0.f;
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
          const float o = acc[j] * inv;
          act[act_at(h * HD + lane * DPL + j)] = o;
          blk += o;
        }
        if constexpr (FMT == AMK_WEIGHTS_W4A16) {
          // W4A16 block sums: 32 / DPL lanes hold one 32-column block
          blk = group_sum<32 / DPL>(blk);
          if ((lane & (32 / DPL - 1)) == 0) xsum[(h * HD + lane * DPL) >> 5] = blk;
        }
      }
    }
  }
}

// Number of position splits with work at `pos` (split s covers positions
// [s * chunk, (s + 1) * chunk) of 0..pos).
__device__ __forceinline__ int active_splits(ModelRef m, int pos, int* chunk_out) {
  const int n_pos = pos + 1;
  const int chunk = (n_pos + m.nsplit - 1) / m.nsplit;
  if (chunk_out) *chunk_out = chunk;
  return (n_pos + chunk - 1) / chunk;
}

// Merge the S (> 1) split records of KV group g into the normalised output of
// its query heads: o_h = sum_s exp(m_s - M) acc_s / sum_s exp(m_s - M) l_s.
// All waves: first the per-(head, split) weights, then every thread sums a
// float4 of the output over a share of the splits with all its loads in
// flight, then the shares are added through LDS.
template <int HD, int GM>
__device__ __forceinline__ void merge_splits(ModelRef m, int layer, int g, int S, float* scr, int wave,
                                             int lane) {
  const int G = m.group;
  const int rec = G * (kPartHead + HD);
  const float* base = m.part + (size_t)layer * m.ps + (size_t)g * m.nsplit * rec;
  float* wts = scr;                                        // [GM][64]
  float4* red = reinterpret_cast<float4*>(scr + GM * 64);  // [SP][E4]
  const int E4 = G * HD / 4;                               // float4s of output
  const int t = wave * 64 + lane;
  // NT / E4 threads share an output: sp'th share of the splits
  constexpr int SPMAX = 4 * NT / HD;
  int SP = 1;
#pragma unroll
  for (int k = 2; k <= SPMAX; ++k)
    if (k * E4 <= NT) SP = k;
  int sp = 0;
#pragma unroll
  for (int k = 1; k < SPMAX; ++k)
    if (t >= k * E4) sp = k;
  const int o4 = t - sp * E4;
  const int h = (4 * o4) / HD, d = 4 * o4 - h * HD;
  const float* src = base + h * (kPartHead + HD) + kPartHead + d;
  const bool on = sp < SP && o4 < E4;
  float2 ml = make_float2(-INFINITY, 0.f);
  if (wave < G && lane < S) ml = ldg<float2>(base + (size_t)lane * rec + wave * (kPartHead + HD));
  // the first accumulators travel together with the maxima
  float4 v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int s = sp + k * SP;
    v[k] = on && s < S ? ldg<float4>(src + (size_t)s * rec) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (wave < G) {
    const float M = wave_max(ml.x);
    const float w = lane < S ? __expf(ml.x - M) : 0.f;
    const float inv = 1.0f / wave_sum(w * ml.y);
    wts[wave * 64 + lane] = w * inv;
  }
  __syncthreads();
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = sp;;) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int s = s0 + k * SP;
      const float w = s < S ? wts[h * 64 + s] : 0.f;
      a.x = fmaf(w, v[k].x, a.x); a.y = fmaf(w, v[k].y, a.y);
      a.z = fmaf(w, v[k].z, a.z); a.w = fmaf(w, v[k].w, a.w);
    }
    s0 += 8 * SP;
    if (s0 >= S) break;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int s = s0 + k * SP;
      v[k] = on && s < S ? ldg<float4>(src + (size_t)s * rec) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  if (on) red[sp * E4 + o4] = a;
  __syncthreads();
  if (t < E4) {
    float4 o = red[t];
    for (int k = 1; k < SP; ++k) {
      const float4 w = red[k * E4 + t];
      o.x += w.x; o.y += w.y; o.z += w.z; o.w += w.w;
    }
    float* od = m.o + (size_t)layer * m.qs + (size_t)g * G * HD + 4 * t;
    stc(od, o.x); stc(od + 1, o.y); stc(od + 2, o.z); stc(od + 3, o.w);
  }
}

// ---------------------------------------------------------------- the kernel
// TINY: the kernel of the tiny-context schedule, whose O tasks compute the
// attention themselves; the other kernel runs the short and long schedules
// (attention tasks, the inline attention or split merge of a chain counter).
// Each carries only its own attention code, so the tiny one stays within
// 64 KiB of code: the instruction cache then holds it whole, where a larger
// kernel's lines evict each other depending on where the code lies
// (identical machine code measured 20-50 us apart per 8B step at different
// offsets, with instruction-cache misses rising from 6 to 100 thousand per
// step).  Each instantiation starts on a 64 KiB boundary, so its placement
// does not depend on the code size of the others.
template <int HD, int GM, int FMT, bool TINY>
__global__ void __launch_bounds__(NT, 1) __attribute__((aligned(65536)))
amk_decode_kernel(DevModel model, int32_t token, int32_t pos, uint32_t epoch, uint16_t* __restrict__ kv,
                  float* __restrict__ logits, uint64_t timeout_ticks) {
  constexpr int R = RING;
  extern __shared__ float4 lds4[];
  __shared__ Ctl ctl;
  const AMK_CONST DevModel* mp = (const AMK_CONST DevModel*)__builtin_amdgcn_kernarg_segment_ptr();  // `model`
  Lds L;
  L.act = reinterpret_cast<float*>(lds4);
  L.stat = L.act + mp->lds_act;
  L.res = L.stat + mp->lds_stat;
  L.part = L.res + mp->lds_res;
  L.xsum = L.part + mp->lds_scr;

  const int wave = uni(threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  const int sw = wave - 1;
  const uint64_t deadline = wall_clock64() + timeout_ticks;  // on this workgroup's clock from its start
  uint64_t* const trace = mp->trace;

  const int qb = ldc<int32_t>(mp->queue_start + blockIdx.x), qe = ldc<int32_t>(mp->queue_start + blockIdx.x + 1);
  if (qb >= qe) return;

  // ---- records, layer pointers and static data, staged ahead in LDS by the
  // last streaming wave: dword `lane` of a record in lanes 0..15, dword
  // `lane - 16` of a layer entry in lanes 16..47
  typedef uint32_t __attribute__((may_alias)) dword;  // the records are read back as their own types
  auto slot_dw = [&](int k) { return reinterpret_cast<dword*>(&ctl.slot[k & (NSLOT - 1)]); };
  auto rec_dw = [&](int idx) { return (const uint32_t*)(mp->tasks + min(idx, qe - 1)); };
  auto stat_for = [&](int idx) {  // static data of this lane's item of task idx
    const Slot& sl = ctl.slot[idx & (NSLOT - 1)];
    const int op = uni(sl.t.op), begin = uni(sl.t.begin), n = uni(sl.t.end) - begin;
    RowStat r;
    if (is_gemv(op) && n <= 64 && lane < n)
      r = row_stat(*mp, sl, op, FMT == AMK_WEIGHTS_W8A16 && uni(ctl.geom[op].quant), begin + lane, token, pos);
    return r;
  };
  auto prepare = [&](int idx, const RowStat& r) {  // the epilogue of task idx
    const amk_task_t& t = ctl.slot[idx & (NSLOT - 1)].t;
    const int op = uni(t.op);
    if (!is_gemv(op) || op == AMK_OP_LMHEAD || uni(t.end) - uni(t.begin) > 64) return;
    const Fast f = fast_prepare(*mp, ctl, t, op, r, pos, kv, lane);
    ctl.prep[0][lane] = make_float4(f.f0, f.f1, f.c, f.s);
    ctl.prep[1][lane] = make_float4(__uint_as_float((uint32_t)f.d0), __uint_as_float((uint32_t)(f.d0 >> 32)),
                                    __uint_as_float(f.d1), __uint_as_float(f.bits));
  };
  uint32_t stage = 0;  // staging wave: a dword of record idx + 3 or layer idx + 2
  RowStat nst;         // and static data of task idx + 1
  auto stage_load = [&](int idx) {  // record idx, layer idx - 1
    const uint32_t* lp = (const uint32_t*)(mp->layers + uni(ctl.slot[(idx - 1) & (NSLOT - 1)].t.layer));
    stage = ldg<uint32_t>(lane < 16 ? rec_dw(idx) + lane : lp + min(lane - 16, 31));
  };
  if (wave == 1) {
    constexpr int N = sizeof(ctl.geom) / 4;
    static_assert(N <= 64, "one dword per lane");
    const AMK_CONST uint32_t* geom = (const AMK_CONST uint32_t*)mp->geom;
    if (lane < N) reinterpret_cast<dword*>(ctl.geom)[lane] = geom[lane];
  } else if (wave == NW - 1) {
    // the first three records (48 lanes), then the layers of the first two
    if (lane < 48) slot_dw(qb + (lane >> 4))[lane & 15] = ldg<uint32_t>(rec_dw(qb + (lane >> 4)) + (lane & 15));
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const int k = qb + (lane >> 5);
    const uint32_t* lp = (const uint32_t*)(mp->layers + ctl.slot[k & (NSLOT - 1)].t.layer);
    slot_dw(k)[16 + (lane & 31)] = ldg<uint32_t>(lp + (lane & 31));
  }
  for (int i = threadIdx.x; i < mp->lds_act; i += NT) L.act[i] = 0.f;
  if (threadIdx.x == 0) {
    ctl.abort = 0;
    ctl.cont = 0;
  }
  __syncthreads();

  // ---- a streaming wave's ring of granules, its issue side, and the task
  // whose first granules the ring holds
  uint4 buf[R] = {};
  uint32_t sc[R] = {};  // W4A16 group scales (unused otherwise)
  Stream is;
  int ring = -1, nj = 0, nc = 0, nn = 0;  // first job, granule and count of the wave's range in task `ring`
  auto ring_begin = [&](int idx) {
    stream_begin<FMT>(is, *mp, ctl, idx & (NSLOT - 1), sw, &nj, &nc);
    nn = is.left;
    ring = idx;
  };
  // empties the ring; called where its registers serve attention tasks, which
  // also tells the compiler that they are free there
  auto ring_drop = [&]() {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      buf[k] = make_uint4(0, 0, 0, 0);
      sc[k] = 0;
    }
    ring = -1;
  };
  // fills an empty ring: a range shorter than the ring loads only what it has
  // (the loads are waited for together with the input that follows them)
  auto ring_fill = [&]() {
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (is.left > 0) stream_issue<FMT>(is, buf[k], sc[k], *mp, ctl, lane);
  };

  Poll poll;  // sync wave: the wait of the task to come
  Res res;
  if (wave == 0) {
    poll = poll_for(*mp, ctl.slot[qb & (NSLOT - 1)].t, epoch, lane);
  } else if (wave == NW - 1) {
    prepare(qb, stat_for(qb));
    nst = stat_for(qb + 1);
    stage_load(qb + 3);
  }

  for (int idx = qb; idx < qe; ++idx) {
    mp = reopen(mp);
    asm volatile("" : "+v"(lane));  // nor is what follows from the lane kept in registers over all tasks
    ModelRef m = *mp;
    const Slot& sl = ctl.slot[idx & (NSLOT - 1)];
    uint64_t* tr = trace ? trace + (size_t)idx * AMK_TRACE_FIELDS : nullptr;

    // ---- B1a: the sync wave's counter wait; meanwhile the other waves load
    // what depends on nothing: the task's first weights, unless the ring holds
    // them already, and the gains of a normed input
    bool ok = true;
    if (wave == 0) {
      if (tr && lane == 0) stg<uint64_t>(tr + AMK_TRACE_WAIT_BEGIN, (uint64_t)wall_clock64());
      ok = uni(wait_deps(m, poll, deadline, lane, tr)) != 0;
      if (!ok && lane == 0) ctl.abort = 1;
      if (tr && lane == 0) stg<uint64_t>(tr + AMK_TRACE_WAIT_END, (uint64_t)wall_clock64());
    }
    const int op = uni(sl.t.op), layer = uni(sl.t.layer), begin = uni(sl.t.begin), end = uni(sl.t.end);
    const int aux = uni(sl.t.aux), chain = uni(sl.t.chain_counter);
    const bool gemv = is_gemv(op);
    const bool normed = is_normed(op);
    const int next = idx + 1;
    uint2 gv[NGAIN] = {};
    const uint16_t *gain = nullptr, *src_bf = nullptr;
    const float* src = nullptr;
    int n4 = 0;
    float* mypart = nullptr;
    bool next_gemv = false;
    if (wave != 0 && gemv) {
      if (ring != idx) {
        ring_begin(idx);
        ring_fill();
      }
      if (normed) {
        gain = op == AMK_OP_QKV ? unip(sl.ly.attn_norm) : op == AMK_OP_GATEUP ? unip(sl.ly.mlp_norm) : m.final_norm;
        n4 = m.H >> 2;
        load_gain(gain, n4, sw, lane, gv);
        const int xi = op == AMK_OP_QKV ? 2 * layer : op == AMK_OP_GATEUP ? 2 * layer + 1 : 2 * m.L;
        if (xi == 0) src_bf = m.embed + (size_t)token * m.H;
        src = m.x + (size_t)xi * m.xs;
      } else if (op == AMK_OP_DOWN) {
        src = m.a + (size_t)layer * m.as;
        n4 = m.I >> 2;
      } else {
        src = m.o + (size_t)layer * m.qs;
        n4 = (m.nq * HD) >> 2;
      }
      mypart = L.part + sw;
      next_gemv = next < qe && is_gemv(uni(ctl.slot[next & (NSLOT - 1)].t.op));
    }
    __syncthreads();

    uint32_t* sig = nullptr;
    if (wave == 0) {
      sig = counter_copy(m, uni(sl.t.signal_counter), lane);
      if (next < qe) poll = poll_for(m, ctl.slot[next & (NSLOT - 1)].t, epoch, lane);
    }
    // the attention scratch: behind the queries in the activation region (free
    // then) where the partials region has no room for it
    float* scr = m.scr_at ? L.act + m.scr_at : L.part;
    int active = 0;  // attention splits with work at `pos`
    auto traced = [&](int field) {
      if (tr && wave == 0 && lane == 0) stg<uint64_t>(tr + field, (uint64_t)wall_clock64());
    };
    auto publish = [&]() {  // sync wave: results stored
      traced(AMK_TRACE_PUBLISHED);
      if (chain >= 0) {
        // the producer that completes the counter runs its inline task: a QKV
        // task's group has npg producers, an attention split's nsplit
        const uint32_t producers = op == AMK_OP_QKV ? (uint32_t)m.npg : (uint32_t)m.nsplit;
        const bool cont = release_signal_last(sig, epoch * producers);
        if (cont) acquire_after_poll();
        if (lane == 0) ctl.cont = cont;
      } else {
        release_signal(sig);
      }
      traced(AMK_TRACE_SIGNALLED);
      if (tr && lane == 0) stg<uint64_t>(tr + AMK_TRACE_CHAINED, 0ull);
    };

    if (gemv) {
      // ---- B1b: the input activation; the sync wave prepares the epilogue
      Epi e;
      Fast f;
      float rs = 1.f;
      const bool small = end - begin <= 64 && op != AMK_OP_LMHEAD;
      if (wave != 0) {
        if (normed) load_input_normed<FMT>(src, src_bf, gain, n4, gv, L, ctl, sw, lane);
        else if (!TINY || op == AMK_OP_DOWN) load_input<FMT>(src, n4, L, sw, lane);
      }
      if constexpr (TINY) {
        if (op == AMK_OP_O) attention_all<HD, FMT>(m, layer, pos, kv, L.act, L.xsum, wave, lane);
      }
      if (wave == 0) {
        if (small) {
          const float4 a = ctl.prep[0][lane], b = ctl.prep[1][lane];
          f.f0 = a.x; f.f1 = a.y; f.c = a.z; f.s = a.w;
          f.d0 = (uint64_t)__float_as_uint(b.y) << 32 | __float_as_uint(b.x);
          f.d1 = __float_as_uint(b.z);
          f.bits = __float_as_uint(b.w);
          if (op == AMK_OP_O || op == AMK_OP_DOWN) {
            const int xin = 2 * layer + (op == AMK_OP_DOWN);
            if (xin != 0) {
              if (res.buf == xin && res.lo == begin && res.hi == end) f.c = L.res[min(lane, end - begin - 1)];
              else f.c = ldg<float>(m.x + (size_t)xin * m.xs + begin + min(lane, end - begin - 1));
            }
            res.buf = xin + 1;
            res.lo = begin;
            res.hi = end;
          }
        } else {
          e.layer = layer; e.begin = begin; e.end = end; e.aux = aux;
          e.g = gemv_geom(ctl, op, end - begin);
          e.wr = wave_ranges(e.g);
        }
      }
      __syncthreads();
      traced(AMK_TRACE_INPUT_READY);

      // ---- compute
      bool fill = false;  // the ring takes the next task's granules after B2
      if (wave == 0) {
        if (normed) rs = input_rs(m, ctl);
        if (!small) {
          e.rs = rs;
          for (int i = begin + lane; i < end; i += 64)
            put_stat(L, op, i - begin, row_stat(m, sl, op, FMT == AMK_WEIGHTS_W8A16 && e.g.quant, i, token, pos));
        }
      } else {
        Work w;
        w.j = nj; w.c = nc; w.left = nn;
        w.gpr = is.gpr; w.lastb = is.lastb; w.quant = is.quant;
        // blocks of R granules; the last one of several already refills the
        // ring with the next task's granules
        const int nblk = max(1, (nn + R - 1) / R);
        fill = next_gemv && nblk == 1;
        const int full = next_gemv && nblk > 1 ? nblk : nblk - 1;
        for (int b = 0; b < full; ++b) {
          if (b == nblk - 1) ring_begin(next);
#pragma unroll
          for (int k = 0; k < R; ++k) {
            consume<FMT>(w, buf[k], sc[k], L, mypart, lane);
            stream_issue<FMT>(is, buf[k], sc[k], m, ctl, lane);
          }
        }
        if (full < nblk) {
#pragma unroll
          for (int k = 0; k < R; ++k) consume<FMT>(w, buf[k], sc[k], L, mypart, lane);
        }
        if (w.c != 0) {
          const float r = wave_sum(w.acc);
          if (lane == 0) mypart[w.j] = r;
        }
      }
      __syncthreads();  // B2: partials in LDS
      traced(AMK_TRACE_COMPUTE_END);
      if (wave == 0) {
        if (!ok) return;
        if (small) {
          fast_finish(op, end - begin, f, rs, L, lane);
        } else {
          switch (op) {
            case AMK_OP_QKV: epi_qkv(m, e, L, pos, kv, lane); break;
            case AMK_OP_O: case AMK_OP_DOWN: epi_residual(m, e, res, op, L, lane); break;
            case AMK_OP_GATEUP: epi_gateup(m, e, L, lane); break;
            default: epi_lmhead(m, e, L, logits, lane); break;
          }
        }
        publish();
      } else {
        if (uni(ctl.abort)) return;
        if (fill) {
          ring_begin(next);
          ring_fill();
        }
      }
    } else {
      if (uni(ctl.abort)) return;
      traced(AMK_TRACE_INPUT_READY);
      if constexpr (!TINY) {
        if (op == AMK_OP_ATTN) {
          int chunk = 0;
          active = active_splits(m, pos, &chunk);
          // a split with no positions at `pos` has no work
          if (begin < active) {
            // one split: the normalised output directly; several: a partial record
            const int j0 = begin * chunk, j1 = min(pos + 1, j0 + chunk);
            const int rec = m.group * (kPartHead + HD);
            float* dst = active == 1 ? m.o + (size_t)layer * m.qs + (size_t)aux * m.group * HD
                                     : m.part + (size_t)layer * m.ps + ((size_t)aux * m.nsplit + begin) * rec;
            attention<HD, GM>(m, layer, aux, j0, j1, kv, L.act, scr, dst, active > 1, wave, lane);
            drain_vmem();
          }
          ring_drop();
        }
      }
      __syncthreads();  // B2: attention results stored
      traced(AMK_TRACE_COMPUTE_END);
      if (wave == 0) {
        if (op == AMK_OP_ARGMAX) argmax_final(m, begin, end, lane);
        publish();
      }
    }
    if (wave == NW - 1) {
      // the staged dwords and static data arrive in LDS, the next ones set out
      if (lane < 48) slot_dw(lane < 16 ? idx + 3 : idx + 2)[lane] = stage;
      prepare(next, nst);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      nst = stat_for(idx + 2);
      stage_load(idx + 4);
    }

    // ---- inline task of the chain counter (all waves; never in the tiny schedule)
    if constexpr (!TINY) {
      if (chain >= 0) {
        __syncthreads();  // B3: results released and signalled
        if (uni(ctl.cont)) {
          if (op == AMK_OP_QKV) {
            float* dst = m.o + (size_t)layer * m.qs + (size_t)aux * m.group * HD;
            attention<HD, GM>(m, layer, aux, 0, pos + 1, kv, L.act, scr, dst, false, wave, lane);
          } else if (active > 1) {
            merge_splits<HD, GM>(m, layer, aux, active, scr, wave, lane);
          }
          ring_drop();
          drain_vmem();
          __syncthreads();  // B4: inline results stored
          if (wave == 0) {
            release_signal(counter_copy(m, chain, lane));
            if (tr && lane == 0) stg<uint64_t>(tr + AMK_TRACE_CHAINED, (uint64_t)wall_clock64());
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------- read probe
// Grid-stride streaming read, four 16-byte loads in flight per thread.
__global__ void __launch_bounds__(NT) amk_read_kernel(const uint4* __restrict__ p, int64_t n16,
                                                      uint32_t* __restrict__ sink) {
  const int64_t stride = (int64_t)gridDim.x * NT;
  int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  uint32_t acc = 0;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    const uint4 a = ldg<uint4>(p + i), b = ldg<uint4>(p + i + stride);
    const uint4 c = ldg<uint4>(p + i + 2 * stride), d = ldg<uint4>(p + i + 3 * stride);
    acc ^= a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ d.x ^ d.y ^ d.z ^ d.w;
  }
  for (; i < n16; i += stride) {
    const uint4 a = ldg<uint4>(p + i);
    acc ^= a.x ^ a.y ^ a.z ^ a.w;
  }
  sink[(size_t)blockIdx.x * NT + threadIdx.x] = acc;
}

extern "C" int amk_internal_read_probe(const void* buf, int64_t bytes, int32_t blocks, uint32_t* sink,
                                       void* stream) {
  hipLaunchKernelGGL(amk_read_kernel, dim3(blocks), dim3(NT), 0, (hipStream_t)stream, (const uint4*)buf, bytes / 16,
                     sink);
  return hipGetLastError() == hipSuccess ? AMK_OK : AMK_ERR_DEVICE;
}

// ---------------------------------------------------------------- static scratch
// Device memory of a handle made by amk_create_static (its task tables,
// counters, activations, RoPE table and status words): one array per device,
// held from the library's first use on that device until the process ends.
// In host code `scratch` only names the array; its device address on each
// device comes from hipGetSymbolAddress and is used everywhere instead.
static __device__ __align__(256) unsigned char scratch[AMK_STATIC_SCRATCH_BYTES];

extern "C" int amk_internal_static_scratch(int device, void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  if (!ptr || !bytes || device < 0 || device >= kMaxDevices) return AMK_ERR_INVALID_ARGUMENT;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return AMK_ERR_DEVICE;
    }
    addr[device] = p;
  }
  *ptr = addr[device];
  *bytes = sizeof(scratch);
  return AMK_OK;
}

// ---------------------------------------------------------------- host side
template <int HD, int GM, bool TINY>
static const void* kernel_ptr(int fmt) {
  if (fmt == AMK_WEIGHTS_W4A16) return (const void*)amk_decode_kernel<HD, GM, AMK_WEIGHTS_W4A16, TINY>;
  return fmt == AMK_WEIGHTS_W8A16 ? (const void*)amk_decode_kernel<HD, GM, AMK_WEIGHTS_W8A16, TINY>
                                  : (const void*)amk_decode_kernel<HD, GM, AMK_WEIGHTS_BF16, TINY>;
}

template <int HD, int GM>
static const void* kernel_ptr(int fmt, bool tiny) {
  return tiny ? kernel_ptr<HD, GM, true>(fmt) : kernel_ptr<HD, GM, false>(fmt);
}

static const void* kernel_for(int head_dim, int group, int fmt, bool tiny) {
  const bool small = group <= 4;
  if (head_dim == 64) return small ? kernel_ptr<64, 4>(fmt, tiny) : kernel_ptr<64, 8>(fmt, tiny);
  return small ? kernel_ptr<128, 4>(fmt, tiny) : kernel_ptr<128, 8>(fmt, tiny);
}

extern "C" int amk_internal_threads(void) { return NT; }
extern "C" int amk_internal_static_lds(void) { return (int)sizeof(Ctl); }

// Floats of LDS scratch the attention and split merge of one task need (in
// the partials region).
extern "C" int amk_internal_attn_scratch(int group, int head_dim) {
  const bool small = group <= 4;
  if (head_dim == 64) return small ? AttnGeom<64, 4>::LDS : AttnGeom<64, 8>::LDS;
  return small ? AttnGeom<128, 4>::LDS : AttnGeom<128, 8>::LDS;
}

// Both kernels of the shape and format (tiny schedule and the others).
extern "C" int amk_internal_prepare(int head_dim, int group, int fmt, int lds_bytes) {
  for (const bool tiny : {true, false}) {
    const hipError_t e = hipFuncSetAttribute(kernel_for(head_dim, group, fmt, tiny),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return AMK_ERR_DEVICE;
  }
  return AMK_OK;
}

// Largest number of co-resident workgroups per CU for this LDS size that
// both kernels of the shape and format reach.
extern "C" int amk_internal_occupancy(int head_dim, int group, int fmt, int lds_bytes, int* blocks_per_cu) {
  int least = 0;
  for (const bool tiny : {true, false}) {
    int n = 0;
    const hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel_for(head_dim, group, fmt, tiny), NT, lds_bytes);
    if (e != hipSuccess) return AMK_ERR_DEVICE;
    least = tiny ? n : (n < least ? n : least);
  }
  *blocks_per_cu = least;
  return AMK_OK;
}

extern "C" int amk_internal_launch(const DevModel* m, int32_t tiny, int32_t token, int32_t pos, uint32_t epoch,
                                   uint16_t* kv, float* logits, uint64_t timeout_ticks, void* stream) {
  DevModel mm = *m;
  void* args[] = {&mm, &token, &pos, &epoch, &kv, &logits, &timeout_ticks};
  hipError_t e = hipLaunchCooperativeKernel(kernel_for(m->hd, m->group, m->fmt, tiny != 0), dim3(m->n_cu), dim3(NT), args,
                                            (unsigned)m->lds_bytes, (hipStream_t)stream);
  return e == hipSuccess ? AMK_OK : AMK_ERR_DEVICE;
}

}  // namespace amk
