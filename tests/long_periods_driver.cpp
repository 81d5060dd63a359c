// A second operand with a period longer than the tensor, of 2^32 elements and more: the argument blocks of every form an add or mul can take
// hold periods of 32 bits, which such a period does not fit; element for element is the same.  CPU only, over made-up addresses.
#include "../paper_2503_19779_amd/csrc/chain.hip"

namespace {
int failures = 0;
void check(const char* what, long long m, long long n) {
    if (m != n) { std::printf("%s: period %lld, not %lld\n", what, m, n); failures++; }
}

pg_kernel_desc desc(int op, int out, pg_ref a, pg_ref b, long long n, long long m) {
    pg_kernel_desc d{};
    d.op = op; d.dtype = PG_BF16; d.out = {PG_REF_INT, out}; d.in[0] = a; d.in[1] = b; d.n = n; d.m = m; d.rows = 1;
    return d;
}

void run(const std::vector<pg_kernel_desc>& k, long long n, long long m) {
    const pg_tensor_desc ext[2] = {{PG_BF16, 0, n}, {PG_BF16, 0, m}}, w = {PG_BF16, 0, n * n};
    std::vector<pg_tensor_desc> ints(4, pg_tensor_desc{PG_BF16, 0, n});
    const void* wp = reinterpret_cast<const void*>(0x600000000000ull);
    size_t need = 0;
    pg_chain* c = nullptr;
    if (pg_chain_workspace_bytes(k.data(), (int)k.size(), ext, 2, ints.data(), 4, &need) || pg_chain_build(k.data(), (int)k.size(), ext, 2, ints.data(), 4, &wp, &w, 1, reinterpret_cast<void*>(0x700000000000ull), need, &c)) {
        std::printf("not built: %s\n", pg_last_error());
        failures++;
        return;
    }
    for (size_t i = 0; i < k.size(); i++)
        if (k[i].op == PG_ADD || k[i].op == PG_MUL) check("on its own", c->rec[i].a_eager.ew.m, n);
    auto all = segment_dispatches(c, c->seg[0], kGraphTable, 0);
    for (size_t g = 0; g < all.size(); g++) {
        const MergeGroup& grp = c->seg[0].groups[g];
        if (grp.k1 - grp.k0 < 2) continue;
        if (grp.head) {
            const auto* e = reinterpret_cast<const pgk::GemvEpiArgs*>(all[g].args.data());
            for (int i = 0; i < e->n_epi; i++) check("behind a GEMV", e->ph[i].m, n);
        } else if (grp.chain) {
            const auto* e = reinterpret_cast<const pgk::ChainArgs*>(all[g].args.data());
            for (int i = 0; i < grp.k1 - grp.k0; i++) check("in a chain", e->m[i], n);
        } else if (!grp.carry && !grp.sbr) {
            const auto* e = reinterpret_cast<const pgk::MergedArgs*>(all[g].args.data());
            for (int i = 0; i < e->n_phase; i++) if ((e->ph[i].meta & 0xffu) != PG_GELU) check("in a run", e->ph[i].m, n);
        }
    }
    std::printf("%zu kernels in %zu dispatches\n", k.size(), all.size());
    if (all.size() >= k.size()) failures++;
    pg_chain_destroy(c);
}
}  // namespace

int main() {
    const pg_ref none = {PG_REF_NONE, 0}, x = {PG_REF_EXT, 0}, b = {PG_REF_EXT, 1};
    auto in = [](int i) { return pg_ref{PG_REF_INT, i}; };
    for (long long m : {(1ll << 32), (1ll << 32) + 8, (1ll << 33) + 1, 1025ll}) {
        const long long n = 1024;
        run({desc(PG_ADD, 0, x, b, n, m), desc(PG_MUL, 0, in(0), b, n, m), desc(PG_ADD, 1, in(0), b, n, m)}, n, m);                  // a chain
        run({desc(PG_ADD, 0, x, b, n, m), desc(PG_MUL, 1, x, b, n, m), desc(PG_ADD, 2, in(0), in(1), n, n), desc(PG_MUL, 3, in(1), b, n, m)}, n, m);
        pg_kernel_desc v = desc(PG_GEMV, 0, {PG_REF_WEIGHT, 0}, x, n, 0);
        v.cols = n;
        run({v, desc(PG_GELU, 0, in(0), none, n, 0), desc(PG_ADD, 1, in(0), b, n, m)}, n, m);
    }
    if (!failures) std::printf("long periods: ok\n");
    return failures != 0;
}
