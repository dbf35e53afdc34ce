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
        if (w.bytes > o.nested_bytes || !w.knn->near.ok) std::printf("pivots N=%lld d=%d P=%d: %zu of %zu bytes, engine %d\n", (long long)N, d, P, w.bytes, o.nested_bytes, w.knn->near.ok);
        ++checked;
    }
}

// A layout keeps within the bytes it is given, from the least there can be to what the size functions report, and takes as many
// where it is laid out as where it is only measured; `engine`: whether the half-precision engine is part of it, and at least one
// panel's worth of batch.
template <typename L>
static void limits(const char* what, long long a, long long b, long long c, L&& layout_at)
{
    bool engine = false;
    auto layout = [&](size_t most, bool* e) {
        bool e2 = false;
        const size_t bytes = layout_at(nullptr, most, e), there = layout_at(reinterpret_cast<void*>((size_t)1 << 40), most, &e2);
        if (bytes != there || *e != e2) std::printf("%s %lld %lld %lld: %zu bytes measured, %zu laid out\n", what, a, b, c, bytes, there);
        return bytes;
    };
    const size_t least = layout(0, &engine), full = layout(NO_LIMIT, &engine);
    const bool has_engine = engine;
    auto check = [&](size_t most, bool want) {
        bool e = false;
        const size_t bytes = layout(most, &e);
        if (bytes > most || (want && e != has_engine)) std::printf("%s %lld %lld %lld: %zu bytes in %zu (least %zu, full %zu), engine %d\n", what, a, b, c, bytes, most, least, full, e);
        ++checked;
    };
    check(least, false);
    for (int i = 1; i < 200; ++i) check(least + (size_t)((double)(full - least) * i / 200), false);
    if (full > least) check(full - 1, false);
    check(full, true);
    check(full + 12345, true);
    std::printf("least %s %lld %lld %lld %zu\n", what, a, b, c, least);
}

int main()
{
    struct Shape { int64_t N; int32_t d, k; };
    for (const Shape x : {Shape{2, 1, 1}, Shape{700, 4, 3}, Shape{4096, 16, 16}, Shape{20011, 50, 10}, Shape{100000, 64, 32}, Shape{250000, 784, 16},
                          Shape{1000000, 128, 32}, Shape{2000000, 32, 8}, Shape{100000000, 8, 8}}) {
        const int32_t dw = working_columns(x.N, x.d);
        const size_t head = padded_copy_bytes(x.N, x.d);
        limits("knn", x.N, x.d, x.k, [&](void* at, size_t most, bool* e) {
            const KnnWs w(at, x.N, dw, true, x.k, false, most == NO_LIMIT ? most : most > head ? most - head : 0);
            *e = w.near.ok;
            return head + w.bytes;
        });
        limits("slhc", x.N, x.d, x.k, [&](void* at, size_t most, bool* e) {
            const SlhcWs w(at, x.N, dw, x.k, true, most == NO_LIMIT ? most : most > head ? most - head : 0);
            *e = w.knn->near.ok;
            return head + w.bytes;
        });
    }
    struct Search { int64_t m, n; int32_t d; };
    for (const Search x : {Search{1, 1, 1}, Search{10, 2000000, 64}, Search{1000, 100000, 128}, Search{1000, 4000, 30}, Search{20000, 500000, 256}, Search{200000, 3000, 20}})
        limits("fused", x.m, x.n, x.d, [&](void* at, size_t most, bool* e) {
            float *hq, *hy; unsigned long long* keys;
            NearWs near;
            const size_t bytes = fused_1nn_layout(at, x.m, x.n, x.d, &hq, &hy, &keys, &near, most);
            *e = near.ok;
            return bytes;
        });
    for (const Search x : {Search{0, 100, 4}, Search{1, 2, 1}, Search{10000, 100000, 64}, Search{10, 1000000, 64}, Search{50, 2000, 8}, Search{300000, 300000, 128}})
        limits("cross", x.n, x.d, x.m, [&](void* at, size_t most, bool* e) {
            const CrossWs w(at, x.n, x.d, x.m, most);
            *e = w.near.ok;
            return w.bytes;
        });
    for (int64_t N : {512, 700, 5000, 24576, 60000, 100000, 200000, 250000, 300000, 320000, 500000, 1000000, 2000000, 4000000, 7000000})
        for (int32_t d : {4, 32, 64, 128}) pivots(N, d);
    std::printf("checked %ld\n", checked);
    return 0;
}
