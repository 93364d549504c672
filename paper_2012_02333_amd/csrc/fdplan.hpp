// Per-instance plans of the full-definition path (shared by single and batched calls).
#pragma once

#include <array>
#include <cstring>
#include <utility>
#include <vector>

#include "engine.hpp"

namespace cqc {

struct FdInstancePlan {
  CutInfo cut;
  NetLayout net;
  std::vector<size_t> conv_off;  // per entry: converted copy (or SIZE_MAX)
  size_t end = 0;
};

// Plans of one-instance calls, kept per thread.  A plan depends on the cut, the
// entry dtype and the arithmetic alone and takes about 5 us of host time, twice
// per one-shot call (workspace size, then the call) and once per call of a loop
// over prepared circuits - as long as the kernels of a small one.  The key is
// the whole cut description by value; pointers are checked on every call.
struct PlanKey {
  int32_t len = 0;   // 0: not to be kept
  std::array<int32_t, 5 + CQC_MAX_SUB + 2 * CQC_MAX_CUTS + CQC_MAX_FD_QUBITS> v;
  bool operator==(const PlanKey &o) const {
    return len == o.len && std::memcmp(v.data(), o.v.data(), sizeof(int32_t) * (size_t)len) == 0;
  }
};
// Descriptions that do not look valid get no key: planning reports the error.
inline PlanKey plan_key(const cqc_cut &c, cqc_dtype in_t, Acc acc) {
  PlanKey k;
  if (c.n_qubits < 1 || c.n_qubits > CQC_MAX_FD_QUBITS || c.n_sub < 1 || c.n_sub > CQC_MAX_SUB || c.n_cuts < 0 ||
      c.n_cuts > CQC_MAX_CUTS || !c.f || !c.out_qubit || (c.n_cuts > 0 && (!c.edge_up || !c.edge_down)))
    return k;
  int64_t sum = 0;
  for (int i = 0; i < c.n_sub; ++i) sum += c.f[i];
  if (sum != c.n_qubits) return k;
  int n = 0;
  auto add = [&](const int32_t *p, int count) {
    for (int i = 0; i < count; ++i) k.v[n++] = p[i];
  };
  const int32_t head[5] = {c.n_qubits, c.n_sub, c.n_cuts, (int32_t)in_t, (int32_t)acc};
  add(head, 5);
  add(c.f, c.n_sub);
  add(c.edge_up, c.n_cuts);
  add(c.edge_down, c.n_cuts);
  add(c.out_qubit, c.n_qubits);
  k.len = n;
  return k;
}
// The last few plans of a thread; a returned plan stays valid until the
// thread's next put.
template <typename P> class PlanMemo {
 public:
  const P *find(const PlanKey &k) const {
    for (const auto &s : slots_)
      if (k.len && s.first == k) return &s.second;
    return nullptr;
  }
  const P *put(const PlanKey &k, P &&p) {
    auto &s = slots_[next_];
    next_ = (next_ + 1) % slots_.size();
    s.first = k;
    s.second = std::move(p);
    return &s.second;
  }

 private:
  std::array<std::pair<PlanKey, P>, 4> slots_;
  size_t next_ = 0;
};

Status precision_acc(cqc_precision prec, Acc *acc);
Status check_dtype(cqc_dtype t);
// out_optional: inst.out may be NULL (a cross-entropy batch that does not
// keep p); every other pointer is required when need_ptrs is set.
Status plan_fd_instance(const cqc_instance &in, cqc_dtype in_t, Acc acc, size_t base, bool need_ptrs,
                        FdInstancePlan *out, bool out_optional = false);
// The plan of a one-instance call, from the thread's memo where it has it.
Status fd_plan_one(const cqc_instance &in, cqc_dtype in_t, cqc_dtype out_t, cqc_precision prec, bool need_ptrs,
                   const FdInstancePlan **plan, Acc *acc_out);
Status fd_plans(const cqc_instance *inst, int32_t n_inst, cqc_dtype in_t, cqc_dtype out_t,
                cqc_precision prec, bool need_ptrs, std::vector<FdInstancePlan> *plans, Acc *acc_out,
                bool out_optional = false);

}  // namespace cqc
