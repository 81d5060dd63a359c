// The total of the matrices that a chain's GEMVs read (chain_weight_bytes): each once, whichever kind of tensor it is and however many GEMVs
// read it; one that GEMVs of several sizes read counts with the largest.  And the shapes whose kernel depends on it: those with a form that takes
// weights by non-temporal loads, which is the slower one where rows share cache lines and, from 81 rows on, for few outputs.  CPU only.
#include <array>

#include "../paper_2503_19779_amd/csrc/chain.hip"

int main() {
    int failures = 0;
    auto total = [&](std::vector<std::array<long long, 4>> gemvs) {          // {operand kind, index, n, cols}
        pg_chain c;
        c.ext.resize(2); c.ints.resize(2); c.w.resize(2);
        for (const auto& g : gemvs) {
            pg_kernel_desc d{};
            d.op = PG_GEMV; d.dtype = PG_BF16; d.rows = 1; d.n = g[2]; d.cols = g[3];
            d.in[0] = pg_ref{(int32_t)g[0], (int32_t)g[1]};
            c.k.push_back(d);
        }
        pg_kernel_desc other{};
        other.op = PG_GELU; other.dtype = PG_BF16; other.n = 1 << 20; other.in[0] = pg_ref{PG_REF_WEIGHT, 1};
        c.k.push_back(other);
        return chain_weight_bytes(&c);
    };
    auto check = [&](const char* what, long long got, long long want) {
        if (got != want) { std::printf("%s: %lld bytes, not %lld\n", what, got, want); failures++; }
    };
    for (int kind : {PG_REF_WEIGHT, PG_REF_EXT, PG_REF_INT}) {
        check("one matrix, forty readers", total(std::vector<std::array<long long, 4>>(40, {kind, 0, 2048, 2048})), 2048 * 2048 * 2);
        check("two matrices, one by two sizes", total({{kind, 0, 64, 32}, {kind, 1, 16, 8}, {kind, 0, 128, 32}, {kind, 0, 8, 8}}), (128 * 32 + 16 * 8) * 2);
    }
    check("the same index of three kinds", total({{PG_REF_WEIGHT, 0, 8, 8}, {PG_REF_EXT, 0, 8, 8}, {PG_REF_INT, 0, 8, 8}}), 3 * 8 * 8 * 2);
    check("no GEMV", total({}), 0);
    for (long long rows : {40, 64, 80, 81, 100, 128})
        for (long long n : {64, 255, 256, 2048}) for (long long cols : {520, 576, 768, 1000, 1024, 1088, 1280, 1500, 1536, 1544, 1928, 1984, 2000, 2048}) {
            if (rows < 81 && cols <= 1024) continue;             // a form that is the same for all chains
            pgk::Shape s;
            s.rows = rows; s.n = n; s.cols = cols;
            pgk::Launch merged, alone;
            pgk::plan_gemv_epilogue(s, false, &merged);
            if (!pgk::plan(PG_GEMV, PG_BF16, 0, s, &alone)) failures++;
            for (const auto& l : {merged, alone})
                if ((l.fn_beyond_cache != nullptr) != (cols % 64 == 0 && (rows < 81 || n >= 256))) {
                    std::printf("%lld rows of %lld columns, %lld outputs: %s form for weights beyond the cache\n", rows, cols, n, l.fn_beyond_cache ? "a" : "no");
                    failures++;
                }
        }
    if (!failures) std::printf("weight bytes: ok\n");
    return failures != 0;
}
