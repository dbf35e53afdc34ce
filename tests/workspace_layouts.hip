// The workspace layouts of the library (host code only; nothing here runs on a GPU).  Prints one line per check that failed,
// then "checked <n>".
#include <cstdio>
#include "../paper_2306_16354_amd/csrc/slhc_api.hip"

static long checked = 0;

// The row order clusters its pivots, as many as the data asks for up to Pmax, in a workspace laid out for Pmax of them: every
// number keeps within it.
static void pivots(int64_t N, int32_t d)
{
    OrderWs o{};
    Carver c(nullptr);
    o.carve(c, N, d, true);
    for (int P = o.P1; P <= o.Pmax; P += o.Pmax > 1000 ? o.Pmax / 500 : 1) {
        if (P < 2) continue;
        const int32_t kp = P - 1 < NESTED_K ? P - 1 : NESTED_K;
        const SlhcWs w(nullptr, P, d, kp, false, o.nested_bytes);
        const KnnWs k(nullptr, P, d, false, kp, w.knn_most);
        if (w.bytes > o.nested_bytes || !k.near.ok) std::printf("pivots N=%lld d=%d P=%d: %zu of %zu bytes, engine %d\n", (long long)N, d, P, w.bytes, o.nested_bytes, k.near.ok);
        ++checked;
    }
}

int main()
{
    for (int64_t N : {512, 700, 5000, 24576, 60000, 100000, 200000, 250000, 300000, 320000, 500000, 1000000, 2000000, 4000000, 7000000})
        for (int32_t d : {4, 32, 64, 128}) pivots(N, d);
    std::printf("checked %ld\n", checked);
    return 0;
}
