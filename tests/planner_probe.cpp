// Prints what the planner makes of a tensor list, one JSON object: built and run on the CPU by tests/planner.py.
// Arguments: kind hidden_padded P lstm_hidden n_bank head_folded groups n_cu apply (0 none, 1 strip, 2 narrow); standard input: "rows cols" per tensor.
#include <cstdio>
#include <cstdlib>
#include <utility>
#include <vector>

#include "lopt_plan.h"

int main(int argc, char** argv) {
  if (argc != 10) return 2;
  lopt::PlanOptions o;
  o.kind = atoi(argv[1]);
  o.HP = atoi(argv[2]);
  o.P = atoi(argv[3]);
  o.lstm_hidden = atoi(argv[4]);
  o.n_bank = atoi(argv[5]);
  o.head_folded = atoi(argv[6]) != 0;
  o.groups_override = atoi(argv[7]);
  o.n_cu = atoi(argv[8]);
  o.apply = (lopt::ApplyTiles)atoi(argv[9]);
  std::vector<lopt_tensor_desc> d;
  long long m, n;
  while (scanf("%lld %lld", &m, &n) == 2) {
    lopt_tensor_desc x{};
    x.ndim = 2; x.rows = m; x.cols = n;
    d.push_back(x);
  }
  lopt::Plan pl;
  lopt::build_plan(o, d.size(), d.data(), &pl);
  std::vector<std::pair<int, long long>> runs;   // heights of the apply tiles in table order, run by run
  for (const auto& t : pl.atiles) {
    if (runs.empty() || runs.back().first != t.rows) runs.push_back({t.rows, 0});
    runs.back().second++;
  }
  printf("{\"ws_floats\": %llu, \"table_bytes\": %zu, \"n_tiles\": %zu, \"n_rcitems\": %zu, \"n_rcshort\": %zu, \"n_rctiles\": %zu, \"n_atiles\": %zu, "
         "\"short_list\": %d, \"groups\": %d, \"fold_finalize\": %d, \"lstm_ahead\": %d, \"keep\": %d, \"keep_off\": %d, \"keep_line\": %d, \"backwards\": %d, "
         "\"strip_ordinary\": %d, \"off_grid_nt\": %d, \"atile_runs\": [",
         (unsigned long long)pl.ws_floats, lopt::table_bytes(pl), pl.tiles.size(), pl.rcitems.size(), pl.rcshort.size(), pl.rctiles.size(),
         pl.atiles.size(), pl.short_list, pl.groups, pl.fold_finalize, pl.oLstmZ != 0, pl.keep, pl.keep_off, pl.keep_line, pl.backwards,
         pl.strip_ordinary, pl.off_grid_nt);
  const char* sep = "";
  for (const auto& h : runs) { printf("%s[%d, %lld]", sep, h.first, h.second); sep = ", "; }
  printf("], \"tensors\": [");
  for (size_t i = 0; i < d.size(); ++i) {
    const lopt::TensorDev& T = pl.tensors[i];
    printf("%s{\"TR\": %d, \"nrt\": %d, \"nct\": %d, \"nrblk\": %d, \"ncblk\": %d, \"state_bytes\": %zu, "
           "\"regions\": [%llu, %llu, %llu, %llu, %llu, %llu, %llu, %llu, %llu]}", i ? ", " : "", T.TR, T.nrt, T.nct, T.nrpart, T.ncpart,
           pl.state_bytes[i], (unsigned long long)T.oRowPart, (unsigned long long)T.oColPart, (unsigned long long)T.oRR,
           (unsigned long long)T.oRC, (unsigned long long)T.oRcPart, (unsigned long long)T.oStatPart, (unsigned long long)T.oStats,
           (unsigned long long)T.oScale, (unsigned long long)T.oPrep);
  }
  printf("]}\n");
  return 0;
}
