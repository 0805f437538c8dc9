// Host-side check of a batched pass's launch plan (tests/test_host_plan.py builds it): a plan whose
// recorded launches hold no product must be refused or have the device lists its grouped launches read.
#include "dmpt_api.hip"

int main() {
  dmpt_ctx c = new dmpt_ctx_s();
  BatchedPlan plan;
  Op cg, ew;
  cg.cg = true;
  cg.ca.n = 128 * 128;
  cg.ca.batch = 1;
  ew.ew = true;
  ew.ewop = EwOp::Account;
  ew.ea = ew_account(nullptr, nullptr, 1, nullptr);
  plan.ops = {{cg, ew}, {cg, ew}};
  std::vector<void*> owned;
  const dmpt_status st = build_plan(c, plan, owned);
  const bool lists = plan.d_cglist && plan.d_ewlist && plan.d_start;
  std::printf("plan without products: status %d, lists %d\n", (int)st, (int)lists);
  const bool ok = st != DMPT_OK || lists;
  for (void* p : owned) dev_free(c, p);
  delete c;
  std::puts(ok ? "plan driver: ok" : "plan driver: launches would read null lists");
  return ok ? 0 : 1;
}
