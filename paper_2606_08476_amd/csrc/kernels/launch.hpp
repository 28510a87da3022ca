// Kernel parameter blocks and host-side launchers (implemented in the .hip
// files). Only the C ABI layer calls these, after validating everything.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <unistd.h>

#include <mutex>

namespace fck {

// Orders the uses of a view's own partial slots: every use waits, on its
// stream, for the event the last use on that stream's device recorded, so uses
// on several streams or threads follow one another instead of racing. A view
// bound again on another device has its slots there and starts an event of that
// device's (an event is recorded on its own device only). Hold `mu` from wait()
// to used().
struct SlotGuard {
  std::mutex mu;

  hipError_t wait(hipStream_t s) {
    int cur = 0;
    if (const hipError_t e = hipGetDevice(&cur); e != hipSuccess) return e;
    dev_ = cur;
    if (s)
      if (const hipError_t e = hipStreamGetDevice(s, &dev_); e != hipSuccess) return e;
    if (dev_ < 0 || dev_ >= kDevices) return hipErrorInvalidDevice;
    hipEvent_t& ev = last_[dev_];
    if (ev) return hipStreamWaitEvent(s, ev, 0);
    if (dev_ != cur)
      if (const hipError_t e = hipSetDevice(dev_); e != hipSuccess) return e;
    const hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) ev = nullptr;
    pid_ = getpid();
    if (dev_ != cur) (void)hipSetDevice(cur);
    return e;
  }

  hipError_t used(hipStream_t s) { return hipEventRecord(last_[dev_], s); }

  // (no HIP call in a forked process that drops a view it inherited)
  ~SlotGuard() {
    if (pid_ != getpid()) return;
    for (hipEvent_t ev : last_)
      if (ev) (void)hipEventDestroy(ev);
  }

 private:
  static constexpr int kDevices = 64;
  hipEvent_t last_[kDevices] = {};  // by device, made by the first use there
  int dev_ = 0;                     // the stream's device in wait()
  pid_t pid_ = 0;                   // of the process that made the events
};

struct FwdParams {
  const uint16_t* q;        // [t_q, hq, d] bf16
  const uint16_t* k_recv;   // [t_r, hkv, d]
  const uint16_t* v_recv;
  const uint16_t* k_loc;    // [t_q, hkv, d]
  const uint16_t* v_loc;
  const int32_t* items;     // 8 int32 per item, in launch order: q0 q1 r0 r1 l0 l1 ldiag seg
  int32_t n_items;
  int32_t hq, hkv, group, head_chunks;
  float scale_log2;         // softmax scale * log2(e)
  // outputs; final: o_bf16 (+ o_f32 if non-null) + lse; partial: o_f32 + lse
  uint16_t* o_bf16;
  float* o_f32;
  float* lse;               // [hq, t_q]
  int32_t t_q;
  // both partials at once (non-null o_f32_recv): items carry a received and
  // a local range; the received partial goes to o_f32_recv/lse_recv, the
  // local one to o_f32/lse; with final output, the two are merged in the
  // kernel (o_f32_recv is then a workspace, lse_recv unused) and the final
  // O/LSE written as for the one-pass final output
  float* o_f32_recv;
  float* lse_recv;
  // split views (non-zero chunk: key tiles per chunk). With slots: `units` are
  // the chunks, last field the slot; slots of 128 x d floats and 128 LSEs per
  // KV head and head chunk, merged per entry of `comb` (q0 q1 first-slot
  // received-chunks local-chunks 0 0 0) into the final output, or for the
  // partial passes into each source's partial: the local one to o_f32/lse, the
  // received one to o_f32_recv/lse_recv, either null if not asked for; these
  // use the view's own slots, guard[0] for the local chunks' and guard[1] for
  // the received ones'. Without slots (partial passes): `items`, a workgroup
  // per query tile merging its chunks itself.
  int32_t chunk;
  const int32_t* units;
  int32_t n_units;
  float* slots;
  float* slot_lse;
  const int32_t* comb;
  int32_t n_comb;
  SlotGuard* guard[2];
};

struct BwdParams {
  const uint16_t* q;        // [t_q, hq, d]
  const uint16_t* dout;     // [t_q, hq, d]
  const float* lse;         // [hq, t_q] natural log
  const float* delta;       // [hq, t_q] rowsum(dO * O)
  const uint16_t* k_loc;
  const uint16_t* v_loc;
  const uint16_t* k_recv;
  const uint16_t* v_recv;
  const int32_t* items;     // 8 int32 per item, in launch order: k0 k1 q0 q1 qfull src seg slot
  const int32_t* lim;       // [t_q] receive index end per query
  const int32_t* qfirst;    // per item, per 32-key wave: first query row that sees it
  float* part_k;            // [slots, hkv, 128, d] partial dK/dV of split key tiles
  float* part_v;
  int32_t n_items;
  int32_t hq, hkv, group;
  float scale;
  float* dk_loc;            // [t_q, hkv, d] fp32
  float* dv_loc;
  float* dk_recv;           // [t_r, hkv, d] fp32
  float* dv_recv;
  int32_t t_q;
  float* dq;                // [t_q, hq, d] fp32, added into (atomic pass only)
};

struct DqParams {
  const uint16_t* q;        // [t_q, hq, d]
  const uint16_t* dout;     // [t_q, hq, d]
  const float* lse;         // [hq, t_q] natural log
  const float* delta;       // [hq, t_q]
  const uint16_t* k_recv;
  const uint16_t* v_recv;
  const uint16_t* k_loc;
  const uint16_t* v_loc;
  const int32_t* items;     // fused forward items, in launch order: q0 q1 r0 r1 l0 l1 ldiag seg
  int32_t n_items;
  int32_t hq, hkv, group, head_chunks;
  float scale;
  float* dq;                // [t_q, hq, d] fp32, written
  int32_t t_q;
  // split key ranges (non-null part): the items are parts, the last field is
  // the partial slot (-1: the whole range, written to dq directly); slots of
  // 128 x d floats per KV head and head chunk, summed per entry of `comb`
  // (q0 q1 first-slot slot-count 0 0 0 0) in slot order
  float* part;
  const int32_t* comb;
  int32_t n_comb;
};

hipError_t launch_fwd(const FwdParams& p, int d, int heads_per_tile, bool final_out,
                      hipStream_t s);
hipError_t launch_bwd_dq(const DqParams& p, int d, int heads_per_tile, hipStream_t s);
hipError_t launch_bwd(const BwdParams& p, int d, hipStream_t s);
// dK/dV with dQ added into p.dq by atomics (p.dq zeroed beforehand)
hipError_t launch_bwd_atomic(const BwdParams& p, int d, hipStream_t s);
// dK/dV and dQ in one launch (dK/dV workgroups first)
hipError_t launch_bwd_grid(const BwdParams& bp, const DqParams& dp, int d, int heads_per_tile,
                           hipStream_t s);
hipError_t launch_bwd_reduce(const int32_t* entries, int32_t n, const float* part_k,
                             const float* part_v, int32_t hkv, int32_t d, float* dk_loc,
                             float* dv_loc, float* dk_recv, float* dv_recv, hipStream_t s);
// delta = rowsum(dout * o), o the fp32 o_f32 when non-null, else the bf16
// o; with a non-null dq_zero, also zeroes that [t, h, d] fp32 tensor (the
// atomic backward's dQ) in the same pass
hipError_t launch_bwd_preprocess(const uint16_t* o, const float* o_f32, const uint16_t* dout,
                                 float* delta, int32_t t, int32_t h, int32_t d, float* dq_zero,
                                 hipStream_t s);
hipError_t launch_fill_zero(float* x, int64_t n, hipStream_t s);
hipError_t launch_lse_merge(const float* o_a, const float* lse_a, const float* o_b,
                            const float* lse_b, int32_t t, int32_t h, int32_t d, uint16_t* o_bf16,
                            float* o_f32, float* lse_out, hipStream_t s);
// rows r0 .. r1-1 of the concatenation (local rows 0 .. t_q-1, then the
// receive set)
hipError_t launch_kv_gather(const uint16_t* k, const uint16_t* v, const int32_t* q_gpos,
                            const int32_t* recv_gpos, int32_t t_q, int32_t t_r, int64_t r0,
                            int64_t r1, int32_t row_elems,
                            uint16_t* k_loc, uint16_t* v_loc, uint16_t* k_recv, uint16_t* v_recv,
                            hipStream_t s);

}  // namespace fck
