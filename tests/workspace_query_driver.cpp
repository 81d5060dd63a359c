// pg_chain_workspace_bytes over descriptors whose sizes nothing has validated: an answer or an error, no overflow in the planner behind it.
// Built with UndefinedBehaviorSanitizer; CPU only.
#include "../include/pygraph_hip.h"

#include <cstdio>
#include <vector>

int main() {
    const long long sizes[] = {1, 8, 2048, 1ll << 31, 1ll << 40, 1ll << 62, -1, 0x7fffffffffffffffll};
    for (int op = PG_ADD; op <= PG_SCALE_BIAS_RELU; op++)
        for (int dtype : {PG_F32, PG_BF16})
            for (long long rows : sizes)
                for (long long cols : sizes)
                    for (long long n : sizes) {
                        std::vector<pg_kernel_desc> k(3);
                        for (int i = 0; i < 3; i++) {        // each reads what the one before wrote
                            k[i] = pg_kernel_desc{};
                            k[i].op = op; k[i].dtype = dtype; k[i].rows = rows; k[i].cols = cols; k[i].n = n; k[i].m = i ? n : 0; k[i].inner = cols;
                            k[i].out = {PG_REF_INT, i & 1};
                            const int n_in = op == PG_GELU ? 1 : op == PG_SCALE_BIAS_RELU ? 3 : 2;
                            for (int j = 0; j < n_in; j++) k[i].in[j] = i && j < 2 && !(op == PG_GEMV && j == 0) ? pg_ref{PG_REF_INT, (i + 1) & 1} : pg_ref{PG_REF_EXT, 0};
                        }
                        const pg_tensor_desc t[2] = {{dtype, 0, 64}, {dtype, 0, 64}};
                        size_t need = 0;
                        if (pg_chain_workspace_bytes(k.data(), 3, t, 1, t, 2, &need) == PG_OK && need == 0) return 1;
                    }
    std::printf("workspace queries: ok\n");
    return 0;
}
