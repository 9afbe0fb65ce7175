// Host audit of the tiles of the direct form and of the batched kernel
// (paper_2609_06449_amd/csrc/tile_addr.h): for every launch that the splits of N
// allow, every workgroup, thread and item, with the functions the kernels call:
//   - the LDS exchange of every stage: each slot inside the buffer, written once,
//     and every item read from where it was stored (both thread orders, one and
//     two groups); the factors that pass B keeps in the buffer fit it;
//   - pass A reads every item of x once, pass B writes every item of y once, and
//     ws is written and read once each, the item (k, c) where pass B expects it;
//   - indexes into the factor tables lie inside them and name the exponent they
//     stand for; no index wraps the 32 bits it is formed in.
// Prints one line per launch kind and exits non-zero on the first failure.
#include "tile_addr.h"

#include <cstdio>
#include <cstdlib>
#include <vector>

using namespace paco;

namespace {

#define CHECK(cond, ...)                                       \
    do {                                                       \
        if (!(cond)) {                                         \
            std::printf("FAIL %s:%d: ", __FILE__, __LINE__);   \
            std::printf(__VA_ARGS__);                          \
            std::printf("\n");                                 \
            std::exit(1);                                      \
        }                                                      \
    } while (0)

// Items the tile functions are given, by thread: as tile_load and tile_stage.
template <int L, int LTG, int H, bool JF>
struct Tile {
    static constexpr int E = tile_items(L), NT = (1 << (L + LTG)) / E, LT = LTG + (H == 2 ? 1 : 0);
    static constexpr int buffer = tile_lds(L, LT, H) - tile_tw(L);

    // f(t, row) for the first stage's operands
    template <class F>
    static void loads(F f)
    {
        constexpr int LR = stage_log2radix(L, 0), R = 1 << LR, NB = E / R, LJ = L - LR;
        for (int tid = 0; tid < NT; ++tid)
            for (int i = 0; i < NB; ++i) {
                const int g = tid + i * NT;
                for (int r = 0; r < R; ++r) f(tile_col<LTG, LJ, JF>(g), tile_idx<LTG, LJ, JF>(g) + (r << LJ));
            }
    }
    // f(t, row) for the last stage's outputs
    template <class F>
    static void stores(F f)
    {
        constexpr int S = stage_count(L) - 1, LR = stage_log2radix(L, S), R = 1 << LR, NB = E / R, LJ = L - LR;
        constexpr int LNS = stage_log2ns(L, S);
        for (int tid = 0; tid < NT; ++tid)
            for (int i = 0; i < NB; ++i) {
                const int g = tid + i * NT;
                for (int r = 0; r < R; ++r) f(tile_col<LTG, LJ, JF>(g), tile_idx<LTG, LJ, JF>(g) + (r << LNS));
            }
    }
    // the exchange between stage S and the next
    template <int S>
    static void exchange()
    {
        if constexpr (S + 1 < stage_count(L)) {
            constexpr int LR = stage_log2radix(L, S), R = 1 << LR, LNS = stage_log2ns(L, S), NB = E / R, LJ = L - LR;
            constexpr int LR2 = stage_log2radix(L, S + 1), R2 = 1 << LR2, NB2 = E / R2, LNR2 = L - LR2;
            std::vector<int> at(buffer, -1);
            for (int tid = 0; tid < NT; ++tid)
                for (int i = 0; i < NB; ++i) {
                    const int g = tid + i * NT, t = tile_col<LTG, LJ, JF>(g), j = tile_idx<LTG, LJ, JF>(g);
                    const int d = stage_dest<LNS, LR>(j);
                    for (int r = 0; r < R; ++r) {
                        const int row = d + (r << LNS), a = tile_slot<L, LTG, JF>(row, t);
                        CHECK(a >= 0 && a < buffer, "L %d LTG %d: store to slot %d of %d", L, LTG, a, buffer);
                        CHECK(at[a] < 0, "L %d LTG %d: slot %d stored twice", L, LTG, a);
                        at[a] = (t << L) + row;
                    }
                }
            for (int tid = 0; tid < NT; ++tid)
                for (int i = 0; i < NB2; ++i) {
                    const int g = tid + i * NT, t = tile_col<LTG, LNR2, JF>(g), j = tile_idx<LTG, LNR2, JF>(g);
                    for (int r = 0; r < R2; ++r) {
                        const int row = j + (r << LNR2), a = tile_slot<L, LTG, JF>(row, t);
                        CHECK(a >= 0 && a < buffer && at[a] == (t << L) + row, "L %d LTG %d: slot %d is another item's", L, LTG, a);
                    }
                }
            exchange<S + 1>();
        }
    }
    static void audit()
    {
        CHECK(NT >= 1 && NT <= 1024 && NT == tile_threads(L, LT, H), "L %d LTG %d: %d threads", L, LTG, NT);
        std::vector<char> in(size_t(1) << (L + LTG)), out(in.size());
        loads([&](int t, int row) { ++in[(size_t(t) << L) + row]; });
        stores([&](int t, int row) { ++out[(size_t(t) << L) + row]; });
        for (char c : in) CHECK(c == 1, "L %d LTG %d: an operand read %d times", L, LTG, c);
        for (char c : out) CHECK(c == 1, "L %d LTG %d: an output stored %d times", L, LTG, c);
        exchange<0>();
        std::printf("ok   tile 2^%d x 2^%d, %d group(s), %s fastest, %d threads\n", L, LT, H, JF ? "index" : "column", NT);
    }
};

// index a 32-bit expression gave, against the exact one and the buffer
uint64_t at32(uint32_t idx, uint64_t exact, uint64_t n, const char *what)
{
    CHECK(exact == idx && exact < n, "%s: %u for %llu of %llu", what, idx, (unsigned long long)exact, (unsigned long long)n);
    return exact;
}

// Pass A over tile `tile` of 2^LT columns; ws[item] = place of (k, c) + 1.
template <int L, int LT, int H>
void pass_a(int l2, int lb, uint32_t tile, std::vector<char> &x, std::vector<uint32_t> &ws)
{
    const uint64_t N = uint64_t(1) << (L + l2);
    const uint32_t col0 = tile << LT;
    typedef Tile<L, LT - (H == 2), H, false> T;
    T::loads([&](int t, int row) {
        const uint32_t i = addr::pass_a_load(uint32_t(row), uint32_t(t * H), l2);
        for (int h = 0; h < H; ++h) ++x[at32(col0 + i + h, (uint64_t(row) << l2) + col0 + t * H + h, N, "pass A load")];
        CHECK(H == 1 || (i + col0) % 2 == 0, "pass A: a 16-byte load off its alignment");
    });
    T::stores([&](int t, int k) {
        for (int h = 0; h < H; ++h) {
            const uint32_t c = col0 + uint32_t(t * H);
            const uint32_t i = addr::pass_a_store(uint32_t(k), c, l2, lb) + (uint32_t(h) << lb);
            CHECK(i < N && !ws[i], "pass A: item %u of ws stored twice or outside", i);
            ws[i] = ((uint32_t(k) << l2) + c + h) + 1;
        }
    });
}

// Pass B over tile `tile` of 2^LT columns k.
template <int L, int LT, int H>
void pass_b(int l1, int log2Lo, uint32_t tile, std::vector<uint32_t> &ws, std::vector<char> &y)
{
    const int lN = L + l1;
    const uint64_t N = uint64_t(1) << lN;
    const uint32_t col0 = tile << LT;
    typedef Tile<L, LT - (H == 2), H, false> T;
    CHECK((16 << LT) <= T::buffer, "pass B: %d factors in %d slots", 16 << LT, T::buffer);
    T::loads([&](int t, int row) {
        const uint32_t i = addr::pass_b_load(uint32_t(row), uint32_t(t * H), LT);
        CHECK(H == 1 || i % 2 == 0, "pass B: a 16-byte load off its alignment");
        for (int h = 0; h < H; ++h) {
            const uint64_t a = (uint64_t(col0) << L) + i + h;
            const uint32_t k = col0 + uint32_t(t * H + h);
            CHECK(a < N && ws[a] == (k << L) + uint32_t(row) + 1, "pass B: item %llu of ws is not (%u, %d)", (unsigned long long)a, k, row);
            ws[a] = 0;
            // w_N^{-k row} = w_N^{-k j} w_{16 M1}^{-k r}, row = j + r 2^(L-4)
            const uint32_t j = uint32_t(row) & ((1u << (L - 4)) - 1u), r = uint32_t(row) >> (L - 4);
            const uint32_t cw = addr::pass_b_cw(k, r, l1), e = addr::pass_b_top(k, j, lN);
            CHECK(cw < (16u << l1) && e < N, "pass B: factor outside its table");
            CHECK((e >> log2Lo) < (N >> log2Lo) && ((e + (uint64_t(cw) << (L - 4))) & (N - 1)) == ((uint64_t(k) * row) & (N - 1)),
                  "pass B: factors of (%u, %d)", k, row);
        }
    });
    T::stores([&](int t, int row) {
        const uint32_t i = addr::pass_b_store(uint32_t(row), uint32_t(t * H), l1);
        CHECK(H == 1 || (i + col0) % 2 == 0, "pass B: a 16-byte store off its alignment");
        for (int h = 0; h < H; ++h) ++y[at32(col0 + i + h, (uint64_t(row) << l1) + col0 + t * H + h, N, "pass B store")];
    });
}

template <class A, class B>
void audit_passes(const char *what, int l1, int l2, uint32_t tiles_a, uint32_t tiles_b, A a, B b)
{
    const size_t N = size_t(1) << (l1 + l2);
    std::vector<char> x(N), y(N);
    std::vector<uint32_t> ws(N);
    for (uint32_t g = 0; g < tiles_a; ++g) a(g, tiles_a, x, ws);
    for (size_t i = 0; i < N; ++i) CHECK(x[i] == 1 && ws[i], "%s 2^%d x 2^%d: pass A at item %zu", what, l1, l2, i);
    for (uint32_t g = 0; g < tiles_b; ++g) b(g, tiles_b, ws, y);
    for (size_t i = 0; i < N; ++i) CHECK(y[i] == 1 && !ws[i], "%s 2^%d x 2^%d: pass B at item %zu", what, l1, l2, i);
    std::printf("ok   %s 2^%d x 2^%d (%u + %u tiles)\n", what, l1, l2, tiles_a, tiles_b);
}

// Calls f with L as a constant.
template <class F>
void with_length(int l, F f)
{
    switch (l) {
    case 7: f(std::integral_constant<int, 7>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    case 9: f(std::integral_constant<int, 9>()); break;
    case 10: f(std::integral_constant<int, 10>()); break;
    case 11: f(std::integral_constant<int, 11>()); break;
    case 12: f(std::integral_constant<int, 12>()); break;
    default: CHECK(false, "no pass of 2^%d points", l);
    }
}

int log2lo(int lN) { return (lN + 1) / 2; }

template <bool MFMA>
void audit_direct(int l1, int l2)
{
    const uint32_t ta = 1u << (l2 - tile_cols(l1, MFMA)), tb = 1u << (l1 - tile_cols(l2, MFMA));
    audit_passes(MFMA ? "direct, split MFMA" : "direct", l1, l2, ta, tb,
                 [&](uint32_t g, uint32_t n, auto &x, auto &ws) {
                     with_length(l1, [&](auto L) {
                         pass_a<L, tile_cols(L, MFMA), tile_groups(L)>(l2, tile_cols(l2, MFMA), uint32_t(tile_order(g, n)), x, ws);
                     });
                 },
                 [&](uint32_t g, uint32_t n, auto &ws, auto &y) {
                     with_length(l2, [&](auto L) {
                         pass_b<L, tile_cols(L, MFMA), tile_groups(L)>(l1, log2lo(l1 + l2), uint32_t(tile_order(g, n)), ws, y);
                     });
                 });
}

template <bool COH>
void audit_batch(int l1, int l2)
{
    constexpr int H = COH ? 1 : 2;
    audit_passes(COH ? "batch, shared queue" : "batch, queue per XCD", l1, l2, 1u << (l2 - pass_lt(l1, COH)),
                 1u << (l1 - pass_lt(l2, COH)),
                 [&](uint32_t g, uint32_t, auto &x, auto &ws) {
                     with_length(l1, [&](auto L) {
                         if constexpr (L <= kBatchPassMax) pass_a<L, pass_lt(L, COH), H>(l2, pass_lt(l2, COH), g, x, ws);
                     });
                 },
                 [&](uint32_t g, uint32_t, auto &ws, auto &y) {
                     with_length(l2, [&](auto L) {
                         if constexpr (L <= kBatchPassMax) pass_b<L, pass_lt(L, COH), H>(l1, log2lo(l1 + l2), g, ws, y);
                     });
                 });
}

// Transforms of one workgroup: the single kernels, then the batch's tasks of 256 and 512 threads.
template <int L>
void audit_chips()
{
    if constexpr (L <= 13) {
        Tile<L, 0, 1, true>::audit();
        if constexpr (L <= 12) Tile<L, small_lt(L, 8), 1, true>::audit();
        Tile<L, small_lt(L, 9), 1, true>::audit();
        audit_chips<L + 1>();
    }
}
template <int L>
void audit_pass_tiles()
{
    if constexpr (L <= 12) {
        Tile<L, tile_cols(L, false) - (tile_groups(L) == 2), tile_groups(L), false>::audit();
        if constexpr (L == 7) Tile<L, tile_cols(L, true), 1, false>::audit();
        if constexpr (L <= kBatchPassMax) {
            Tile<L, pass_lt(L, false) - 1, 2, false>::audit();
            Tile<L, pass_lt(L, true), 1, false>::audit();
        }
        audit_pass_tiles<L + 1>();
    }
}

}  // namespace

int main()
{
    audit_chips<2>();
    Tile<13, 0, 2, true>::audit();  // 2^14 points, 512 threads
    Tile<13, 1, 1, true>::audit();  // the same by 1024
    audit_pass_tiles<7>();
    // every split of a single plan, by the rule that picks it
    for (int lN = kDirectChipLog2 + 1; lN <= kDirectMaxLog2; ++lN) {
        std::vector<int> seen(lN + 1);
        for (int l1 = 1; l1 < lN; ++l1) {
            const int a = direct_l1(l1, lN - l1);
            CHECK(a >= 7 && a <= 12 && lN - a >= 7 && lN - a <= 11, "a split of 2^%d", lN);
            if (!seen[a]++) audit_direct<false>(a, lN - a);
        }
    }
    for (int l1 = 7; l1 <= 11; ++l1)
        for (int l2 = 7; l2 <= 11; ++l2) audit_direct<true>(l1, l2);
    int splits = 0;
    for (int l1 = 1; l1 <= 20; ++l1)
        for (int l2 = 1; l1 + l2 <= 20; ++l2)
            if (batch_split(l1, l2)) {
                audit_batch<false>(l1, l2);
                audit_batch<true>(l1, l2);
                ++splits;
            }
    std::printf("tile audit passed (%d splits of the batch)\n", splits);
    return 0;
}
