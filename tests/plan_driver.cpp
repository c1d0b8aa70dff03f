// Prints the launch plan and the load kind of the configurations on standard
// input, one a line: "plan U G D S blocks work bf16 agg list_ints splits npr cold"
// or "loads own others units prompt" (bytes).
#include <stdio.h>
#include <string.h>

#include "raas_internal.h"

int main() {
    char line[256];
    while (fgets(line, sizeof line, stdin)) {
        int U, G, D, S, blocks, work, bf16, agg, list, splits, npr, cold;
        double own, others;
        if (sscanf(line, "plan %d %d %d %d %d %d %d %d %d %d %d %d", &U, &G, &D, &S, &blocks, &work, &bf16, &agg, &list,
                   &splits, &npr, &cold) == 12) {
            const raas::StepPlan p = raas::plan_step(U, G, D, S, blocks * raas::kBlockTokens, work, bf16 != 0, agg, false,
                                                     list, splits, npr, 1, cold != 0);
            printf("%d %d %d %d\n", p.waves, p.nsplit, p.pool_scratch ? 1 : 0, p.fused ? 1 : 0);
        } else if (sscanf(line, "loads %lf %lf %d %d", &own, &others, &U, &npr) == 4) {
            printf("%d\n", raas::non_temporal_loads(own, others, U, npr != 0) ? 1 : 0);
        } else {
            fprintf(stderr, "bad line: %s", line);
            return 1;
        }
    }
    return 0;
}
