// The division of products on the fused large-batch kernel and the rules that choose between it and the others, for tests on the CPU:
// reads "M K b batch work_bytes" per line, writes "taken ntiles nj blocks waves steps parts copy_bytes gemm_pays static_dense".
#include <cstdio>

#include "../../paper_2402_10517_amd/csrc/kernels.h"

int main()
{
    apgemv::GemvArgs a = {};
    while (std::scanf("%d %d %d %d %zu", &a.M, &a.K, &a.b, &a.batch, &a.work_bytes) == 5) {
        const apgemv::FusedPlan p = apgemv::fused_plan(a);
        std::printf("%d %d %d %d %d %d %d %zu %d %d\n", (int)apgemv::gemm_fused_ok(a), p.ntiles, p.nj, p.blocks, p.waves, p.steps, p.parts,
                    p.copy_bytes, (int)apgemv::gemm_fused_pays(a), (int)apgemv::static_dense_pays(a));
    }
    return 0;
}
