// gfx950 kernel that runs a graph's merge program (merge.cpp), one scenario
// per lane: every lane of a wavefront executes the same instruction list, so
// a visited op's durations and finish times are whole 256-byte rows, and only
// the deferred ops run at places that differ between lanes.
//
// The event replay, which every lane runs in its own order, is bound by its
// divergent accesses (one per lane and load); here they are left only to the
// deferred ops, and the kernel is bound by the instruction stream of the one
// wavefront that a SIMD has.  BERT (16 workers), 262144 scenarios, by counters:
// 1024 blocks for 1024 SIMDs (31 KB of LDS allow five blocks a CU, and the 4096
// tiles go evenly to four); a wavefront issues in 45 % of its cycles and waits
// in 49 %, for LDS hardly ever; an op costs it 29 VALU, 22 scalar, 7 branch and
// 2.5 LDS instructions; HBM traffic is 16.4 GB, 1.18 times the durations and
// finish times.  Replays with finish times, before and after: BERT (16
// workers), 262144 scenarios, 35.0 -> 7.2 ms; ResNet-50 (8 workers), 65536
// scenarios, 7.8 -> 2.9 ms; BERT with gaps and delays, 20000 scenarios, 9.9 ->
// 3.5 ms; with generated durations, 262144 scenarios, 28.2 -> 10.4 ms.
//
// State per lane, [slot][64], in LDS: every resource's free time, the values
// the program keeps, and of each deferred chain its first waiting op's ready
// time, duration and (where the chain has a follower) its partner's duration,
// and the number of its ops run.  An op released while others of its chain
// wait goes to global scratch (ready time and duration), which also takes the
// finish times of deferred ops until the end of the tile, when they are
// written out as rows.  That scratch is the part of a set where the event
// replay keeps its heaps, all ones between calls, so a set holds no more for
// it.
//
// Instructions come in frames of up to 8 of one type, one register each (lane
// 8 u + f holds word f of instruction u), four frames to a group.  Pure frames
// hold consecutive visits of one resource all of whose predecessors ran on it
// (local visits): such an op starts when the resource is free, so the frame is
// a running sum, checked against the cluster's smallest deferred ready time.
// Frames of other visits that no deferred op can precede, of maxima and of
// releases hold instructions independent of one another, so their LDS reads
// go out together.  The rest runs one instruction at a time.
#include <algorithm>
#include <cstring>
#include <utility>
#include <vector>

#include "philox.hpp"
#include "sim.hpp"

namespace mlsim {

namespace {

constexpr uint32_t kI32Max = 0x7fffffffu;
constexpr uint32_t kNever = 0xffffffffu;
constexpr int kMgFrame = 8;   // instructions per frame
constexpr int kMgGroup = 4;   // frames per group
constexpr int kMgPad = 2;     // empty groups after the last (read ahead)
constexpr int kMgNone = 0, kMgPureT = 1, kMgStatic = 2, kMgMaxT = 3, kMgReleaseT = 4, kMgMixed = 5;  // frame types
constexpr int kMgPure = 3;    // local visits in a row that make a pure frame
// most LDS of a block.  Near it a CU has two wavefronts, and the program is still
// 2.2 times (65536 scenarios) to 3.7 times (16384) as fast as the event list
// (ResNet-50, 16 workers, 58 KB); larger programs are not taken
constexpr size_t kMgLdsMax = 64 * 1024;
// instruction flags, above the kind: more than two operands; the one operand
// is the free time that the visit before left
constexpr uint32_t kMgWide = 8, kMgNext = 16;

typedef int32_t i32x32 __attribute__((ext_vector_type(32)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));

template <class T>
using lptr = __attribute__((address_space(3))) T *;
template <class T>
using cptr = const __attribute__((address_space(4))) T *;

struct MgArgs {
  int64_t n_scen;
  const int32_t *dur;
  uint32_t ldb_dur;  // bytes from one row to the next
  int32_t *makespan;
  int32_t *finish;   // [n_ops] rows (FIN)
  uint32_t ldb_fin;
  int32_t *status;
  int32_t *prev;     // PREV: rows like finish: the op that ran before each op on its resource, -1: none
  uint32_t *state;   // [blocks][2][n_def][64] deferred ops: ready then finish times, durations
  const int32_t *dev;  // DEV: [2R] gaps, output delays
  int dev_gap, dev_delay;
  DurGen gen;          // GEN
};

// a use of a group's rows and of a later one's instructions: the wait for them lands here
__device__ __forceinline__ void mg_settle(i32x32 &v, i32x4 &w) { asm volatile("" : "+v"(v), "+v"(w)); }
template <class V>
__device__ __forceinline__ V mg_use(V v) {
  asm volatile("" : "+v"(v));
  return v;
}
using mg_gptr = __attribute__((address_space(1))) char *;
using mg_gint = __attribute__((address_space(1))) int32_t;

// GEN: durations generated from a.gen; DEV: gaps and output delays; PREV: the
// op each resource ran before is recorded; FIN: finish times are written.
// Lanes past the last scenario replay it and write its results again.
template <bool GEN, bool DEV, bool PREV, bool FIN>
__global__ __launch_bounds__(kWave) void k_merge(MergeTable T, MgArgs a) {
  extern __shared__ uint32_t mg_lds[];
  const int lane = threadIdx.x;
  const int NC = T.n_chain, R = T.R;
  const lptr<uint32_t> S = (lptr<uint32_t>)mg_lds + lane;
  const lptr<uint32_t> head = S + (size_t)T.head_slot * kWave;       // first ready time per chain
  const lptr<uint32_t> hdur = head + (size_t)NC * kWave;             // that op's duration
  const lptr<uint32_t> haux = hdur + (size_t)NC * kWave;             // its partner's
  const lptr<uint16_t> at = (lptr<uint16_t>)(mg_lds + (size_t)T.slots * kWave) + lane;  // ops run per chain
  const lptr<uint16_t> ran = at + (size_t)NC * kWave;                // PREV: last row per resource
  // ops released per chain: the same in every lane (a chain that follows
  // another has as many as that one has run)
  const lptr<uint16_t> rel = (lptr<uint16_t>)(mg_lds + (size_t)T.slots * kWave) + ((size_t)NC + (PREV ? R : 0)) * kWave;
  uint32_t *vr = a.state + (size_t)blockIdx.x * 2 * T.n_def * kWave + lane;
  uint32_t *vd = vr + (size_t)T.n_def * kWave;
  const int2 *def = (const int2 *)T.def;
  const cptr<i32x4> chain = (cptr<i32x4>)T.chain;  // {first deferred index, resource, follower, leader}
  const int32_t *insw = T.ins;
  const bool keep_fin = FIN || T.force;

  for (int64_t tile = blockIdx.x; tile * kWave < a.n_scen; tile += gridDim.x) {
    const int64_t s0 = tile * kWave;
    const bool active = s0 + lane < a.n_scen;
    const int col = active ? lane : (int)(a.n_scen - 1 - s0);
    const int64_t G = GEN ? a.gen.scen0 + s0 + col : 0;
    const int32_t *brow = GEN ? gen_knob_row(a.gen, G) : nullptr;
    const uint32_t g_lo = (uint32_t)G, g_hi = (uint32_t)((uint64_t)G >> 32);
    for (int r = 0; r < R; ++r) S[r * kWave] = 0;
    if (PREV)
      for (int r = 0; r < R; ++r) ran[r * kWave] = 0xffffu;
    for (int i = T.head_slot; i < T.zero_slot; ++i) S[i * kWave] = kNever;
    S[T.zero_slot * kWave] = 0;
    S[T.inf_slot * kWave] = kNever;
    for (int c = 0; c < NC; ++c) at[c * kWave] = rel[c] = 0;
    uint32_t mx = 0;
    int32_t dmin = 1;
    // this tile's columns
    const mg_gptr dur0 = (mg_gptr)(a.dur + s0 + col), fin0 = (mg_gptr)(a.finish + s0 + col),
                  prev0 = (mg_gptr)(a.prev + s0 + col);
    uint32_t ldb_dur = a.ldb_dur, ldb_fin = a.ldb_fin;
    asm("" : "+v"(ldb_dur), "+v"(ldb_fin));  // in vector registers, where the multiply-adds take them

    // a finish on resource r frees it and reaches its successors (DEV); both
    // saturated at 2^31, which still makes a later finish overflow
    auto model = [&](uint32_t fin, int r, uint32_t &avail, uint32_t &arr) __attribute__((always_inline)) {
      if (a.dev_gap) {
        const uint32_t y = fin + (uint32_t)a.dev[r];
        avail = y < kI32Max + 1u ? y : kI32Max + 1u;
      }
      if (a.dev_delay) {
        const uint32_t y = fin + (uint32_t)a.dev[R + r];
        arr = y < kI32Max + 1u ? y : kI32Max + 1u;
      }
    };

    // Runs deferred ops of chains [c0, c1) in key order: with force until
    // chain fc has run more than fx ops, else while the smallest key is below
    // (K, id); rf is resource r's free time.  Each round every lane that still
    // has one to run runs one and moves one of its chains forward, so the loops
    // end.  Returns the smallest ready time left.  One chain, or two on
    // different resources, stay in registers meanwhile.
    auto finish_deferred = [&](int x, int r, uint32_t fin) __attribute__((always_inline)) {
      if (keep_fin) vr[(size_t)x * kWave] = fin;
      if (PREV) {
        const uint32_t h = ran[r * kWave];
        ran[r * kWave] = (uint16_t)mg_use(def[x].x);
        vd[(size_t)x * kWave] = h == 0xffffu ? kNever : h;
      }
    };
    auto below = [&](uint32_t t, int x, uint32_t K, int id) __attribute__((always_inline)) -> bool {
      bool less = t < K;
      const bool tie = t == K && t != kNever;
      if (__ballot(tie)) {  // equal ready times: the lower id
        if (tie) less = mg_use(def[x].y) < id;
      }
      return less;
    };
    auto run_one = [&](int c, bool force, uint32_t K, int id, int fx, int r, uint32_t &rf)
        __attribute__((always_inline)) -> uint32_t {
      const i32x4 C = chain[c];
      uint32_t t = head[c * kWave], d = hdur[c * kWave];
      int pos = at[c * kWave];
      const int rl = rel[c];
      uint32_t rfc = C.y == r ? rf : S[C.y * kWave];
      auto goes = [&]() { return force ? pos <= fx && t != kNever : below(t, C.x + pos, K, id); };
      bool go = goes();
      while (__ballot(go)) {
        // ops of the chain that wait behind the first, four at a time
        uint32_t nt[4], nd[4];
        const bool more = go && pos + 1 < rl;
        const bool any = __ballot(more) != 0;
        if (any) {
          if (more) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const size_t x = (size_t)(C.x + (pos + 1 + i < rl ? pos + 1 + i : rl - 1)) * kWave;
              nt[i] = vr[x];
              nd[i] = vd[x];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              nt[i] = mg_use(nt[i]);
              nd[i] = mg_use(nd[i]);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (go) {
            const uint32_t fin = (t > rfc ? t : rfc) + d;
            uint32_t avail = fin, out = fin;
            if (DEV) model(fin, C.y, avail, out);
            rfc = avail;
            mx = fin > mx ? fin : mx;
            finish_deferred(C.x + pos, C.y, fin);
            ++pos;
            t = pos < rl ? nt[i] : kNever;
            d = nd[i];
          }
          go = go && goes();
          if (!any || !__ballot(go)) break;
        }
      }
      head[c * kWave] = t;
      hdur[c * kWave] = d;
      at[c * kWave] = (uint16_t)pos;
      if (C.y == r)
        rf = rfc;
      else
        S[C.y * kWave] = rfc;
      return t;
    };
    auto run_two = [&](int c, bool force, uint32_t K, int id, int fx, int fc, int r, uint32_t &rf)
        __attribute__((always_inline)) -> uint32_t {
      const i32x4 C[2] = {chain[c], chain[c + 1]};
      uint32_t t[2], d[2], aux[2], rfc[2];
      int pos[2], rl[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        t[k] = head[(c + k) * kWave];
        d[k] = hdur[(c + k) * kWave];
        aux[k] = C[k].z >= 0 ? haux[(c + k) * kWave] : 0u;
        pos[k] = at[(c + k) * kWave];
        rl[k] = C[k].w >= 0 ? at[C[k].w * kWave] : rel[c + k];
        rfc[k] = C[k].y == r ? rf : S[C[k].y * kWave];
      }
      auto second = [&]() {  // the second chain's op comes first
        bool less = t[1] < t[0];
        const bool tie = t[1] == t[0] && t[0] != kNever;
        if (__ballot(tie)) {
          if (tie) less = mg_use(def[C[1].x + pos[1]].y) < mg_use(def[C[0].x + pos[0]].y);
        }
        return less;
      };
      for (;;) {
        bool some = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const bool mine = second() == (k == 1);
          bool go = force ? (fc == c ? pos[0] : pos[1]) <= fx && t[k] != kNever : below(t[k], C[k].x + pos[k], K, id);
          go = go && mine;
          if (!__ballot(go)) continue;
          some = true;
          if (go) {
            const uint32_t fin = (t[k] > rfc[k] ? t[k] : rfc[k]) + d[k];
            uint32_t avail = fin, out = fin;
            if (DEV) model(fin, C[k].y, avail, out);
            rfc[k] = avail;
            mx = fin > mx ? fin : mx;
            if (C[k].z >= 0) {  // the partner, released at the arrival
              rl[1 - k] = pos[k] + 1;
              if (pos[1 - k] == pos[k]) {
                t[1 - k] = out;
                d[1 - k] = aux[k];
              } else {
                vr[(size_t)(C[1 - k].x + pos[k]) * kWave] = out;
                vd[(size_t)(C[1 - k].x + pos[k]) * kWave] = aux[k];
              }
            }
            finish_deferred(C[k].x + pos[k], C[k].y, fin);
            ++pos[k];
            t[k] = kNever;
            if (pos[k] < rl[k]) {  // the next op of the chain waits already
              const size_t x = (size_t)(C[k].x + pos[k]) * kWave;
              t[k] = vr[x];
              d[k] = vd[x];
              if (C[k].z >= 0) aux[k] = mg_use(vd[(size_t)(C[1 - k].x + pos[k]) * kWave]);
              t[k] = mg_use(t[k]);
              d[k] = mg_use(d[k]);
            }
          }
        }
        if (!some) break;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        head[(c + k) * kWave] = t[k];
        hdur[(c + k) * kWave] = d[k];
        if (C[k].z >= 0) haux[(c + k) * kWave] = aux[k];
        at[(c + k) * kWave] = (uint16_t)pos[k];
        if (C[k].y == r)
          rf = rfc[k];
        else
          S[C[k].y * kWave] = rfc[k];
      }
      return t[0] < t[1] ? t[0] : t[1];
    };
    auto run_many = [&](int c0, int c1, bool force, uint32_t K, int id, int fx, int fc)
        __attribute__((always_inline)) -> uint32_t {
      for (;;) {
        uint32_t t = kNever;
        int c = c0, beg = 0, r = 0, fo = -1, le = -1;
        for (int k = c0; k < c1; ++k) {
          const uint32_t y = head[k * kWave];
          const i32x4 Ck = chain[k];
          bool less = y < t;
          const bool tie = y == t && y != kNever;
          if (__ballot(tie)) {
            if (tie) less = mg_use(def[Ck.x + at[k * kWave]].y) < mg_use(def[beg + at[c * kWave]].y);
          }
          t = less ? y : t;
          c = less ? k : c;
          beg = less ? Ck.x : beg;
          r = less ? Ck.y : r;
          fo = less ? Ck.z : fo;
          le = less ? Ck.w : le;
        }
        const int pos = at[c * kWave];
        const bool go = force ? at[fc * kWave] <= fx && t != kNever : below(t, beg + pos, K, id);
        if (!__ballot(go)) return t;
        if (go) {
          const uint32_t rfree = S[r * kWave], d = hdur[c * kWave];
          const int rl = le >= 0 ? at[le * kWave] : rel[c], x = beg + pos, np = pos + 1;
          const uint32_t fin = (t > rfree ? t : rfree) + d;
          uint32_t avail = fin, out = fin;
          if (DEV) model(fin, r, avail, out);
          S[r * kWave] = avail;
          mx = fin > mx ? fin : mx;
          at[c * kWave] = (uint16_t)np;
          int fbeg = 0;
          if (fo >= 0) {
            const uint32_t pd = haux[c * kWave];
            fbeg = mg_use(T.chain[fo * 4]);
            if (at[fo * kWave] == pos) {
              head[fo * kWave] = out;
              hdur[fo * kWave] = pd;
            } else {
              vr[(size_t)(fbeg + pos) * kWave] = out;
              vd[(size_t)(fbeg + pos) * kWave] = pd;
            }
          }
          uint32_t nt = kNever;
          if (np < rl) {
            nt = mg_use(vr[(size_t)(x + 1) * kWave]);
            hdur[c * kWave] = mg_use(vd[(size_t)(x + 1) * kWave]);
            if (fo >= 0) haux[c * kWave] = mg_use(vd[(size_t)(fbeg + np) * kWave]);
          }
          head[c * kWave] = nt;
          finish_deferred(x, r, fin);
        }
      }
    };
    auto run = [&](int c0, int c1, bool force, uint32_t K, int id, int fx, int fc, int r, uint32_t &rf)
        __attribute__((always_inline)) -> uint32_t {
      if (c1 - c0 == 1) return run_one(c0, force, K, id, fx, r, rf);
      if (c1 - c0 == 2 && chain[c0].y != chain[c0 + 1].y) return run_two(c0, force, K, id, fx, fc, r, rf);
      S[r * kWave] = rf;
      const uint32_t m = run_many(c0, c1, force, K, id, fx, fc);
      rf = S[r * kWave];
      return m;
    };

    // this lane's entry of a row (one 64-bit multiply-add)
    auto entry = [&](mg_gptr base, uint32_t row, uint32_t ldb) __attribute__((always_inline)) {
      return (mg_gint *)(base + (uint64_t)row * ldb);
    };
    auto load_group = [&](int g) -> i32x4 {
      i32x4 q;
#pragma unroll
      for (int j = 0; j < kMgGroup; ++j) q[j] = insw[((size_t)g * kMgGroup + j) * kWave + lane];
      return q;
    };
    auto load_rows = [&](i32x4 q, i32x32 &dv) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kMgGroup; ++j)
#pragma unroll
        for (int u = 0; u < kMgFrame; ++u) {
          const uint32_t row = (uint32_t)__builtin_amdgcn_readlane(q[j], u * 8);
          dv[j * kMgFrame + u] = GEN ? brow[row] : *entry(dur0, row, ldb_dur);
        }
    };
#define MG_FIELD(u, f) ((uint32_t)__builtin_amdgcn_readlane(q, (u) * 8 + (f)))
    auto operands = [&](int32_t q, int u, uint32_t w1) __attribute__((always_inline)) -> uint32_t {
      const uint32_t w3 = MG_FIELD(u, 3);
      const uint32_t x0 = S[(w3 & 0xffffu) * kWave], x1 = S[(w3 >> 16) * kWave];
      uint32_t t = x0 > x1 ? x0 : x1;
      if (w1 & kMgWide) {
        const uint32_t w4 = MG_FIELD(u, 4);
        const uint32_t x2 = S[(w4 & 0xffffu) * kWave], x3 = S[(w4 >> 16) * kWave];
        const uint32_t y = x2 > x3 ? x2 : x3;
        t = y > t ? y : t;
      }
      return t;
    };
    auto duration = [&](int32_t d, uint32_t row) __attribute__((always_inline)) -> int32_t {
      if (GEN) d = gen_duration(d, g_lo, g_hi, row, a.gen.key0, a.gen.key1, a.gen.noise);
      dmin = d < dmin ? d : dmin;
      return d;
    };
    // local visits start at free times: not with delays, when an arrival may lie after them
    const bool local_ok = !(DEV && a.dev_delay);

    // Finish times of a frame's visits go out when the next frame starts: one
    // in-order counter covers loads and stores, and so no wait for a group's
    // rows covers a store just issued.
    uint32_t fv[kMgFrame];
    int32_t pv[kMgFrame];       // PREV: the rows that ran before
    int32_t qs = 0;             // the frame they belong to
    uint32_t todo = 0;          // how many of them
    auto flush = [&]() __attribute__((always_inline)) {
      if (!FIN) return;
      auto put = [&](int u) __attribute__((always_inline)) {
        const uint32_t row = (uint32_t)__builtin_amdgcn_readlane(qs, u * 8);
        *entry(fin0, row, ldb_fin) = (int32_t)fv[u];
        if (PREV) *entry(prev0, row, ldb_fin) = pv[u] == 0xffff ? -1 : pv[u];
      };
      if (todo == kMgFrame) {
#pragma unroll
        for (int u = 0; u < kMgFrame; ++u) put(u);
      } else {
#pragma unroll
        for (int u = 0; u < kMgFrame - 1; ++u)
          if ((uint32_t)u < todo) put(u);
      }
      todo = 0;
    };

    // one frame q of k instructions, whose rows are dv[base ...]
    auto frame = [&](int32_t q, const i32x32 &dv, int base) __attribute__((always_inline)) {
      const uint32_t h = MG_FIELD(0, 7);  // count, type, results that are read
      const int k = (int)(h & 15u), type = (int)(h >> 4 & 7u);
      int u0 = 0;  // instructions done
      flush();
      if (type == kMgPureT && local_ok) {
        const int r = (int)(MG_FIELD(0, 2) >> 16);
        const uint32_t keep = h >> 16;
        uint32_t rf = S[r * kWave];
        uint32_t m = S[(MG_FIELD(0, 5) & 0xffffu) * kWave];
        const uint32_t gap = DEV && a.dev_gap ? (uint32_t)a.dev[r] : 0u;
        int32_t before = PREV ? ran[r * kWave] : 0;
        // four at a time (the last ones padded with zero durations): a
        // deferred op may come first only where the least ready time is not
        // above the free time before the last of them
        auto four = [&](auto g0) __attribute__((always_inline)) -> bool {
          constexpr int g = decltype(g0)::value;
          const int left = k - g;
          if (left <= 0) return false;
          int32_t d[4];
          uint32_t fin[4], x = rf, lastx = rf;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            d[j] = dv[base + g + j];
            if (GEN) d[j] = gen_duration(d[j], g_lo, g_hi, MG_FIELD(g + j, 0), a.gen.key0, a.gen.key1, a.gen.noise);
          }
          int32_t dm = d[0];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (j > 0 && left <= j) d[j] = 0;
            lastx = j == 0 || left > j ? x : lastx;
            fin[j] = x + (uint32_t)d[j];
            x = fin[j];
            if (DEV && (j == 0 || left > j)) {
              const uint32_t y = fin[j] + gap;
              x = y < kI32Max + 1u ? y : kI32Max + 1u;
            }
            if (j > 0) dm = left > j && d[j] < dm ? d[j] : dm;
          }
          if (__ballot(m <= lastx)) return false;
          dmin = dm < dmin ? dm : dmin;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (!DEV || j == 0 || left > j) mx = fin[j] > mx ? fin[j] : mx;
            fv[g + j] = fin[j];
          }
          rf = x;
          if (keep >> g & 15u) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (keep >> (g + j) & 1u) S[(MG_FIELD(g + j, 2) & 0xffffu) * kWave] = fin[j];
          }
          u0 = left < 4 ? k : g + 4;
          return true;
        };
        if (four(std::integral_constant<int, 0>{})) four(std::integral_constant<int, 4>{});
        if (PREV) {
#pragma unroll
          for (int u = 0; u < kMgFrame; ++u) {
            pv[u] = before;
            before = (int32_t)MG_FIELD(u, 0);
          }
          if (u0 > 0) ran[r * kWave] = (uint16_t)MG_FIELD(u0 - 1, 0);
        }
        qs = q;
        todo = (uint32_t)u0;
        if (u0 < k) {  // one at a time from where a deferred op may come first
          const int ms = (int)(MG_FIELD(0, 5) & 0xffffu);
#pragma unroll 1
          for (; u0 < k; ++u0) {
            const uint32_t w1 = MG_FIELD(u0, 1), row = MG_FIELD(u0, 0);
            if (__ballot(m <= rf)) {
              const uint32_t t = !DEV && (w1 & kMgNext) ? rf : operands(q, u0, w1);
              if (__ballot(m <= t))
                m = run((int)(w1 >> 8 & 0x7ffu), (int)(w1 >> 20), false, t, (int)(MG_FIELD(u0, 5) >> 16), 0, 0, r, rf);
            }
            const uint32_t fin = rf + (uint32_t)duration(dv[base + u0], row);
            rf = fin;
            if (DEV) {
              const uint32_t y = fin + gap;
              rf = y < kI32Max + 1u ? y : kI32Max + 1u;
            }
            mx = fin > mx ? fin : mx;
            if (keep >> u0 & 1u) S[(MG_FIELD(u0, 2) & 0xffffu) * kWave] = fin;
            if (FIN) *entry(fin0, row, ldb_fin) = (int32_t)fin;
            if (PREV) {
              const int32_t p = ran[r * kWave];
              ran[r * kWave] = (uint16_t)row;
              *entry(prev0, row, ldb_fin) = p == 0xffff ? -1 : p;
            }
          }
          S[ms * kWave] = m;
        }
        S[r * kWave] = rf;
      } else if (type == kMgStatic) {
#pragma unroll
        for (int g = 0; g < kMgFrame; g += 4) {
          if (g >= k) break;
          uint32_t t[4], rf[4], out[4], res[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t w2 = MG_FIELD(g + j, 2);
            out[j] = w2 & 0xffffu;
            res[j] = w2 >> 16;
            rf[j] = S[res[j] * kWave];
            if (PREV) pv[g + j] = ran[(g + j < k ? res[j] : 0u) * kWave];
            t[j] = operands(q, g + j, MG_FIELD(g + j, 1));  // (of a next, 0: it starts at the free time)
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (j > 0 && g + j >= k) break;
            const uint32_t fin = (t[j] > rf[j] ? t[j] : rf[j]) +
                                 (uint32_t)duration(dv[base + g + j], GEN ? MG_FIELD(g + j, 0) : 0);
            uint32_t avail = fin, arr = fin;
            if (DEV) model(fin, (int)res[j], avail, arr);
            S[res[j] * kWave] = avail;
            S[out[j] * kWave] = arr;
            mx = fin > mx ? fin : mx;
            fv[g + j] = fin;
            if (PREV) ran[res[j] * kWave] = (uint16_t)MG_FIELD(g + j, 0);
          }
        }
        qs = q;
        todo = (uint32_t)k;
        u0 = k;
      } else if (type == kMgMaxT) {
#pragma unroll
        for (int g = 0; g < kMgFrame; g += 4) {
          if (g >= k) break;
          uint32_t t[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) t[j] = operands(q, g + j, MG_FIELD(g + j, 1));
#pragma unroll
          for (int j = 0; j < 4; ++j) S[(MG_FIELD(g + j, 2) & 0xffffu) * kWave] = t[j];  // absent ones: a slot nobody reads
        }
        u0 = k;
      } else if (type == kMgReleaseT) {
        // (a load, if any, then its release) twice four: other chains, other clusters
#pragma unroll
        for (int g = 0; g < kMgFrame; g += 4) {
          if (g >= k) break;
          uint32_t t[4], m[4];
          int pos[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            t[j] = operands(q, g + j, MG_FIELD(g + j, 1));
            m[j] = S[(MG_FIELD(g + j, 5) & 0xffffu) * kWave];
            pos[j] = at[(MG_FIELD(g + j, 6) >> 16) * kWave];
          }
          int32_t aux = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (j > 0 && g + j >= k) break;
            const int32_t d = duration(dv[base + g + j], GEN ? MG_FIELD(g + j, 0) : 0);
            if ((MG_FIELD(g + j, 1) & 7u) == (uint32_t)kMgLoad) {
              aux = d;
              continue;
            }
            const uint32_t w6 = MG_FIELD(g + j, 6);
            const int x = (int)(w6 & 0xffffu), xc = (int)(w6 >> 16);
            rel[xc] = (uint16_t)(x + 1);
            if (pos[j] == x) {  // the chain's first waiting op
              head[xc * kWave] = t[j];
              hdur[xc * kWave] = (uint32_t)d;
              if (T.aux) haux[xc * kWave] = (uint32_t)aux;
              S[(MG_FIELD(g + j, 5) & 0xffffu) * kWave] = t[j] < m[j] ? t[j] : m[j];
            } else {
              const i32x4 C = chain[xc];
              vr[(size_t)(C.x + x) * kWave] = t[j];
              vd[(size_t)(C.x + x) * kWave] = (uint32_t)d;
              if (C.z >= 0) vd[(size_t)(chain[C.z].x + x) * kWave] = (uint32_t)aux;
            }
          }
        }
        u0 = k;
      }
      // the others
#pragma unroll 1
      for (int u = u0; u < k; ++u) {
        const uint32_t w1 = MG_FIELD(u, 1), w2 = MG_FIELD(u, 2), w5 = MG_FIELD(u, 5), w6 = MG_FIELD(u, 6);
        const int kind = (int)(w1 & 7u), r = (int)(w2 >> 16), c0 = (int)(w1 >> 8 & 0x7ffu), c1 = (int)(w1 >> 20);
        const int ms = (int)(w5 & 0xffffu);
        uint32_t rf = S[r * kWave];
        const uint32_t m = S[ms * kWave];
        uint32_t t = operands(q, u, w1);
        if (!DEV && (w1 & kMgNext)) t = rf;
        const bool force = kind == kMgForce;
        const int x = (int)(w6 & 0xffffu), xc = (int)(w6 >> 16);
        const uint32_t bound = kind == kMgDrain ? kNever : t;
        uint64_t wait = __ballot(m <= bound);
        if (force) wait = __ballot(at[xc * kWave] <= x);
        if (wait && c0 < c1) {
          S[ms * kWave] = run(c0, c1, force, bound, (int)(w5 >> 16), x, xc, r, rf);
          S[r * kWave] = rf;
        }
        if (kind == kMgVisit) {
          const uint32_t row = MG_FIELD(u, 0);
          const uint32_t fin = (t > rf ? t : rf) + (uint32_t)duration(dv[base + u], row);
          uint32_t avail = fin, arr = fin;
          if (DEV) model(fin, r, avail, arr);
          S[r * kWave] = avail;
          S[(w2 & 0xffffu) * kWave] = arr;
          mx = fin > mx ? fin : mx;
          if (FIN) *entry(fin0, row, ldb_fin) = (int32_t)fin;
          if (PREV) {
            const int32_t p = ran[r * kWave];
            ran[r * kWave] = (uint16_t)row;
            *entry(prev0, row, ldb_fin) = p == 0xffff ? -1 : p;
          }
        } else if (force) {
          const uint32_t fin = mg_use(vr[(size_t)(chain[xc].x + x) * kWave]);
          uint32_t avail, arr = fin;
          if (DEV) model(fin, r, avail, arr);
          S[(w2 & 0xffffu) * kWave] = arr;
        }
      }
    };
    // While a group runs, the next one's rows and the instructions of the one
    // after are on their way.
    i32x4 qa = load_group(0), qb = load_group(1);
    i32x32 da, db;
    load_rows(qa, da);
    mg_settle(da, qb);
#pragma unroll 1
    for (int g = 0; g < T.n_group; ++g) {
      i32x4 qc = load_group(g + 2);
      load_rows(qb, db);
#pragma unroll 1
      for (int j = 0; j < kMgGroup; ++j) frame(j == 0 ? qa[0] : j == 1 ? qa[1] : j == 2 ? qa[2] : qa[3], da, j * kMgFrame);
      mg_settle(db, qc);
      qa = qb;
      qb = qc;
      da = db;
    }
    flush();
#undef MG_FIELD
    // the deferred ops' finish times (and, PREV, the rows that ran before)
    if (FIN) {
      const cptr<i32x2> defc = (cptr<i32x2>)T.def;
      for (int x0 = 0; x0 < T.n_def; x0 += 8) {
        uint32_t y[8], z[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const size_t i = (size_t)(x0 + j < T.n_def ? x0 + j : x0) * kWave;
          y[j] = vr[i];
          if (PREV) z[j] = vd[i];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (x0 + j >= T.n_def) break;
          const uint32_t row = (uint32_t)defc[x0 + j].x;
          *entry(fin0, row, ldb_fin) = (int32_t)y[j];
          if (PREV) *entry(prev0, row, ldb_fin) = (int32_t)z[j];
        }
      }
    }
    const int32_t st = dmin < 1 ? SIM_ST_BAD_DUR : mx > kI32Max ? SIM_ST_OVERFLOW : 0;
    if (active) {
      a.makespan[s0 + lane] = st ? -1 : (int32_t)mx;
      if (a.status) a.status[s0 + lane] = st;
    }
  }
  for (int x = 0; x < 2 * T.n_def; ++x) vr[(size_t)x * kWave] = kNever;  // all ones again
}

using MgKernel = void (*)(MergeTable, MgArgs);
template <bool FIN>
MgKernel mg_kernel_of(bool gen, bool dev, bool prev) {
  if (gen) return k_merge<true, false, false, FIN>;
  if (prev) return k_merge<false, false, true, true>;
  return dev ? k_merge<false, true, false, FIN> : k_merge<false, false, false, FIN>;
}
MgKernel mg_kernel(bool gen, bool dev, bool prev, bool fin) {
  return fin ? mg_kernel_of<true>(gen, dev, prev) : mg_kernel_of<false>(gen, dev, prev);
}

// (One chain's places at least: a free time that overflowed may equal kNever,
// the least ready time where a cluster defers nothing, and the search among its
// no chains then reads the first chain's place before it finds none.  A test
// for that in the frames of local visits costs BERT 2 %.)
size_t mg_lds_bytes(const MergeTable &T, bool prev) {
  return ((size_t)T.slots * 4 + std::max<size_t>(T.n_chain, 1) * 2 + (prev ? (size_t)T.R * 2 : 0)) * kWave +
         (size_t)T.n_chain * 2;
}

}  // namespace

// The device form of a program: frames of instructions, deferred ops, chains.
void pack_merge(const MergeProgram &P, std::vector<int32_t> &ins, std::vector<int32_t> &def,
                std::vector<int32_t> &chain, MergeTable &T) {
  const size_t n = P.ins.size();
  auto u16s = [](int32_t lo, int32_t hi) { return (int32_t)((uint32_t)(lo & 0xffff) | ((uint32_t)hi << 16)); };
  ins.clear();
  auto frame = [&](size_t i0, size_t k, int type) {
    // absent instructions read 0 and write a slot nobody reads
    std::vector<int32_t> w(kWave, 0);
    for (int u = 0; u < kMgFrame; ++u) {
      w[u * 8 + 1] = kMgMax;
      w[u * 8 + 2] = u16s(P.sink_slot, P.sink_slot);
      w[u * 8 + 3] = w[u * 8 + 4] = u16s(P.zero_slot, P.zero_slot);
      w[u * 8 + 5] = P.inf_slot;
    }
    uint32_t read = 0;
    for (size_t u = 0; u < k; ++u) {
      const MergeIns &I = P.ins[i0 + u];
      const MergeCluster c = I.cluster < 0 ? MergeCluster{0, 0, -1} : P.cluster[I.cluster];
      const bool wide = I.p[2] != P.zero_slot || I.p[3] != P.zero_slot;
      const uint32_t f = (uint32_t)I.kind | (wide ? kMgWide : 0u) | (I.next ? kMgNext : 0u);
      const bool d = I.kind == kMgRelease || I.kind == kMgLoad || I.kind == kMgForce;
      const int32_t xc = d ? P.def[I.x].chain : 0;
      const int32_t v[8] = {std::max(I.row, 0), (int32_t)(f | (uint32_t)c.beg << 8 | (uint32_t)c.end << 20),
                            u16s(I.out, I.res), u16s(I.p[0], I.p[1]), u16s(I.p[2], I.p[3]),
                            u16s(c.min_slot < 0 ? P.inf_slot : c.min_slot, I.id),
                            u16s(d ? I.x - P.chain[xc].beg : 0, xc), 0};
      for (int j = 0; j < 8; ++j) w[u * 8 + j] = v[j];
      read |= (I.out != P.sink_slot ? 1u : 0u) << u;
    }
    w[7] = (int32_t)((uint32_t)k | (uint32_t)type << 4 | read << 16);
    ins.insert(ins.end(), w.begin(), w.end());
  };
  auto type_of = [&](const MergeIns &I) {
    return I.kind == kMgMax ? kMgMaxT : I.kind == kMgRelease || I.kind == kMgLoad ? kMgReleaseT
           : I.kind == kMgVisit && I.cluster < 0 ? kMgStatic : kMgMixed;
  };
  auto pure_run = [&](size_t i) {  // local visits of one resource from i on
    size_t j = i;
    while (j < n && P.ins[j].local && P.ins[j].res == P.ins[i].res) ++j;
    return j - i;
  };
  // instruction y does not depend on x before it, and (x and y visits or
  // releases) touches no state of its
  auto apart = [&](const MergeIns &x, const MergeIns &y) {
    for (int32_t p : y.p)
      if (p == x.out && p != P.zero_slot) return false;
    for (int32_t p : x.p)
      if (p == y.out && p != P.zero_slot) return false;
    if (x.out == y.out && x.out != P.sink_slot) return false;
    if (x.kind == kMgVisit) return x.res != y.res;
    return x.kind == kMgMax || x.cluster != y.cluster || (x.kind == kMgLoad && y.kind == kMgRelease);
  };
  size_t frames = 0, run_end = 0;
  for (size_t i = 0; i < n; ++frames) {
    size_t k = pure_run(i);
    int type = kMgPureT;
    if (k >= (size_t)kMgPure) run_end = i + k;  // its last frame may be short
    if (i >= run_end) {
      type = type_of(P.ins[i]);
      for (k = 1; i + k < n && type_of(P.ins[i + k]) == type && pure_run(i + k) < (size_t)kMgPure; ++k) {
        bool free = true;
        for (size_t j = 0; j < k && type != kMgMixed; ++j) free = free && apart(P.ins[i + j], P.ins[i + k]);
        if (!free) break;
      }
    }
    k = std::min<size_t>(k, kMgFrame);
    // a load stays with its release, in one half of the frame
    if (type == kMgReleaseT) {
      size_t half = 0;
      for (size_t j = 0; j < k; ++j) {
        if (P.ins[i + j].kind == kMgLoad && (j % 4 == 3 || j + 1 >= k)) {
          half = j;
          break;
        }
        half = j + 1;
      }
      k = half;
    }
    frame(i, k, type);
    i += k;
  }
  T.n_group = (int32_t)((frames + kMgGroup - 1) / kMgGroup);
  while (frames++ < ((size_t)T.n_group + kMgPad) * kMgGroup) frame(0, 0, kMgNone);
  def.clear();
  T.force = T.aux = 0;
  for (const MergeIns &I : P.ins) T.force |= I.kind == kMgForce;
  for (const MergeDef &d : P.def) {
    def.push_back(d.row);
    def.push_back(d.id);
  }
  chain.clear();
  for (const MergeChain &c : P.chain) {
    const int32_t w[4] = {c.beg, c.res, c.follow, c.lead};
    T.aux |= c.follow >= 0;
    chain.insert(chain.end(), w, w + 4);
  }
  T.n_def = (int32_t)P.def.size();
  T.n_chain = (int32_t)P.chain.size();
  T.slots = P.slots;
  T.head_slot = P.head_slot;
  T.zero_slot = P.zero_slot;
  T.inf_slot = P.inf_slot;
}

// Persistent grids of the merge kernel (plain, generated, device model,
// recording predecessors) whose deferred ops' state fits `bytes`; none when
// one block's LDS or state is too large.
int plan_merge(const sim_graph *g, int cus, size_t bytes, int32_t (&blocks)[4]) {
  std::fill(blocks, blocks + 4, 0);
  const size_t per = std::max<size_t>((size_t)2 * g->mg.n_def * kWave * 4, 1);
  if (!g->mg.n_group || mg_lds_bytes(g->mg, true) > kMgLdsMax || mg_lds_bytes(g->mg_dev, false) > kMgLdsMax ||
      per > bytes)
    return SIM_OK;
  for (int k = 0; k < 4; ++k) {
    const MergeTable &T = k == 2 ? g->mg_dev : g->mg;
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, mg_kernel(k == 1, k == 2, k == 3, true), kWave,
                                                     mg_lds_bytes(T, k == 3)) != hipSuccess)
      return SIM_E_HIP;
    blocks[k] = (int32_t)std::min<size_t>((size_t)std::max(occ, 1) * cus, bytes / per);
  }
  return SIM_OK;
}

int launch_merge(const sim_graph *g, char *scr, int64_t n_scen, const int32_t *dur, int64_t ld_dur, int32_t *makespan,
                 int32_t *finish, int64_t ld_fin, int32_t *status, int32_t *prev, const DurGen *gen,
                 const int32_t *dev, bool has_gap, bool has_delay, hipStream_t stream) {
  const int64_t fit = g->plan.mg_blocks[gen ? 1 : dev ? 2 : prev ? 3 : 0];
  MgArgs a{n_scen, dur, (uint32_t)(ld_dur * 4), makespan, finish, (uint32_t)(ld_fin * 4), status, prev,
           (uint32_t *)(scr + g->scratch_ev_heap_off), dev, has_gap, has_delay, DurGen{}};
  if (gen) a.gen = *gen;
  // every block takes the same number of tiles (within one)
  const int64_t tiles = (n_scen + kWave - 1) / kWave, rounds = (tiles + fit - 1) / fit;
  MergeTable T = dev ? g->mg_dev : g->mg;
  void *args[] = {&T, &a};
  if (hipLaunchKernel((const void *)mg_kernel(gen != nullptr, dev != nullptr, prev != nullptr, finish != nullptr),
                      dim3((unsigned)((tiles + rounds - 1) / rounds)), dim3(kWave), args,
                      mg_lds_bytes(T, prev != nullptr), stream) != hipSuccess)
    return SIM_E_HIP;
  return hipGetLastError() == hipSuccess ? SIM_OK : SIM_E_HIP;
}

}  // namespace mlsim
