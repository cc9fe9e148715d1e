// Host-only check of the streamed lists of the tiled products.
//
// Builds the format with the library's own builder (this file includes the
// library source; no GPU is touched) and walks it as the kernel does: chunk by
// chunk along every wave's stream, lists ending inside chunks, rows moved on by
// the deltas from the base rows.  Checks that
//   * every chunk, list and LDS index stays inside its array;
//   * no row is touched by two lanes of a list, padding included, except the
//     spare zero of lanes without entries;
//   * the row sums, taken entry by entry in FP32, are bit for bit those of the
//     CSR rows summed slab by slab in their own order.
// Prints one line per case and "ok" at the end; exits 1 after a failure.
#include "../../paper_1601_08201_amd/csrc/sgtv_api.hip"

#include <cstdio>
#include <map>

namespace {

struct Csr {
    int64_t n_rows = 0, n_cols = 0;
    std::vector<int64_t> rp;
    std::vector<int32_t> ci;
    std::vector<float> v;
};

uint64_t lcg(uint64_t &s) {
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    return s >> 33;
}

// about per_row entries a row; every 17th row empty; with runs, every 7th row
// falls into a few columns (long runs of one row in one list)
Csr make_csr(int64_t n_rows, int64_t n_cols, int per_row, uint64_t seed, bool runs) {
    Csr m;
    m.n_rows = n_rows;
    m.n_cols = n_cols;
    m.rp.push_back(0);
    uint64_t s = seed;
    for (int64_t r = 0; r < n_rows; ++r) {
        const int k = r % 17 == 5 ? 0 : static_cast<int>(lcg(s) % (2 * per_row + 1));
        for (int e = 0; e < k; ++e) {
            int32_t c = static_cast<int32_t>(lcg(s) % n_cols);
            if (runs && r % 7 == 0) c = static_cast<int32_t>((r * 13 + e) % std::min<int64_t>(n_cols, 40));
            m.ci.push_back(c);
            m.v.push_back(e % 29 == 11 ? 0.0f : static_cast<float>(lcg(s) % 1000 + 1) / 997.0f);
        }
        m.rp.push_back(static_cast<int64_t>(m.ci.size()));
    }
    return m;
}

int failures = 0;

#define CHECK(cond, ...)                                     \
    do {                                                     \
        if (!(cond)) {                                       \
            std::printf("FAIL %s:%d: ", __FILE__, __LINE__); \
            std::printf(__VA_ARGS__);                        \
            std::printf("\n");                               \
            ++failures;                                      \
            return;                                          \
        }                                                    \
    } while (0)

// want: 1 the streamed format must be built, 0 it must be refused, -1 either
void check_case(const char *name, const Csr &m, TileParams t, int want) {
    PackedTiled T;
    CHECK(pack_tiled(T, m.n_rows, m.n_cols, m.rp, m.ci, m.v, t, true) == SGTV_OK, "%s: packing failed", name);
    const sgtv::TileMap &map = T.map;
    const bool streamed = map.idx24 == sgtv::kIdxStream;
    CHECK(want < 0 || streamed == (want == 1), "%s: format %d", name, map.idx24);
    if (!streamed) {
        std::printf("%s: not streamed\n", name);
        return;
    }
    const int W = t.waves, C = sgtv::kStreamChunk;
    const int64_t RB = static_cast<int64_t>(W) * t.rw, n_tiles = map.n_rb * map.ns;
    const int64_t n_streams = n_tiles * W, n_lists = n_streams * map.cbs_max;
    const int64_t acc = (RB + 3) / 4 * 4, lds = acc + t.cb + 4;
    CHECK(static_cast<size_t>(lds) * 4 <= map.lds_bytes() && map.lds_bytes() <= 163840, "%s: LDS", name);
    CHECK(map.pad == n_streams + 1 && static_cast<int64_t>(T.poff.size()) == n_streams + 1 + 32 * n_lists &&
              static_cast<int64_t>(T.goff.size()) == n_lists + 1,
          "%s: offset arrays", name);
    const uint16_t *bases = reinterpret_cast<const uint16_t *>(T.poff.data() + map.pad);
    const uint16_t *idx = reinterpret_cast<const uint16_t *>(T.pk.data());
    const int64_t n_chunks = static_cast<int64_t>(T.pk.size()) / 256;
    CHECK(T.v32.size() == static_cast<size_t>(n_chunks) * C * 64, "%s: value array", name);
    const uint32_t cmask = (1u << map.cbits) - 1;
    CHECK(static_cast<uint32_t>(t.cb) <= cmask, "%s: column bits", name);
    std::vector<float> x(static_cast<size_t>(m.n_cols));
    uint64_t s = 99;
    for (float &v : x) v = static_cast<float>(lcg(s) % 4000) / 1234.0f;
    std::vector<float> got(static_cast<size_t>(map.ns * m.n_rows), -1.0f), ref(got.size(), 0.0f);
    int64_t groups = 0;
    for (int64_t tile = 0; tile < n_tiles; ++tile) {
        const int slab = static_cast<int>(tile % map.ns);
        const int ncbs = map.slab_begin[slab + 1] - map.slab_begin[slab];
        std::vector<float> L(static_cast<size_t>(lds), 0.0f);
        for (int w = 0; w < W; ++w) {
            const int64_t c0 = T.poff[tile * W + w], c1 = T.poff[tile * W + w + 1];
            CHECK(0 <= c0 && c0 <= c1 && c1 < n_chunks, "%s: chunks of a stream", name);   // a spare one follows
            int64_t g = 0;
            for (int c = 0; c < ncbs; ++c) {
                const int64_t list = (tile * map.cbs_max + c) * W + w;
                const int64_t end = T.goff[list];
                CHECK(end >= g && end <= (c1 - c0) * C, "%s: list end", name);
                std::map<int64_t, int> owner;
                for (int lane = 0; lane < 64; ++lane) {
                    int64_t row = static_cast<int64_t>(w) * t.rw + bases[list * 64 + lane];
                    CHECK(g == end || row < lds, "%s: base row", name);
                    for (int64_t k = g; k < end; ++k) {
                        const int64_t ch = c0 + k / C, e = k % C;
                        const uint32_t code = idx[(ch * 64 + lane) * C + e];
                        const float a = T.v32[((ch * 2 + e / 4) * 64 + lane) * 4 + e % 4];
                        const int64_t col = code & cmask;
                        row += code >> map.cbits;
                        CHECK(col <= t.cb && (col < t.cb || a == 0.0f), "%s: column", name);
                        const bool spare = row == acc + t.cb + 1;
                        CHECK((row >= w * t.rw && row < (w + 1) * t.rw) || (spare && col == t.cb), "%s: row", name);
                        auto it = owner.find(row);
                        CHECK(spare || it == owner.end() || it->second == lane, "%s: a row in two lanes", name);
                        owner[row] = lane;
                        const int64_t j = (map.slab_begin[slab] + c) * static_cast<int64_t>(t.cb) + col;
                        CHECK(col == t.cb || j < m.n_cols, "%s: column past the matrix", name);
                        L[row] = std::fmaf(a, col == t.cb ? 0.0f : x[j], L[row]);
                    }
                }
                groups += end - g;
                g = end;
            }
            CHECK((g + C - 1) / C == c1 - c0, "%s: stream length", name);
        }
        const int64_t r0 = tile / map.ns * RB;
        for (int64_t i = 0; i < RB && r0 + i < m.n_rows; ++i)
            got[slab * m.n_rows + r0 + i] = L[T.slot.empty() ? i : T.slot[tile * RB + i]];
    }
    for (int64_t r = 0; r < m.n_rows; ++r)
        for (int slab = 0; slab < map.ns; ++slab)
            for (int b = map.slab_begin[slab]; b < map.slab_begin[slab + 1]; ++b)
                for (int64_t k = m.rp[r]; k < m.rp[r + 1]; ++k)
                    if (m.ci[k] / t.cb == b) {
                        float &y = ref[slab * m.n_rows + r];
                        y = std::fmaf(m.v[k], x[m.ci[k]], y);
                    }
    CHECK(std::memcmp(got.data(), ref.data(), sizeof(float) * got.size()) == 0, "%s: row sums differ", name);
    std::printf("%s: streamed, %d column bits, %zu entries in %lld groups\n", name, map.cbits, m.ci.size(),
                static_cast<long long>(groups));
}

}  // namespace

int main() {
    const Csr a = make_csr(5000, 3000, 20, 1, false);
    check_case("dealt rows", a, TileParams{64, 4, 512, 2}, 1);
    check_case("too few column blocks", a, TileParams{64, 4, 1024, 2}, 0);
    check_case("14 column bits", make_csr(5000, 9000, 60, 1, false), TileParams{128, 4, 3000, 1}, 1);
    check_case("a block too wide for one read", a, TileParams{64, 1, 3000, 1}, 0);
    check_case("odd block width", a, TileParams{100, 4, 1023, 2}, 0);
    check_case("16 waves, 3 slabs", a, TileParams{128, 16, 256, 3}, -1);
    const Csr b = make_csr(3000, 4000, 24, 2, true);
    check_case("long row runs", b, TileParams{64, 8, 512, 1}, -1);
    const Csr thin = make_csr(20000, 600000, 8, 3, false);
    check_case("too sparse", thin, TileParams{16000, 2, 2048, 2}, 0);
    const Csr f = make_csr(40000, 20000, 60, 7, false);
    check_case("2048 rows per wave, all of the LDS", f, TileParams{2048, 16, 8188, 1}, 1);
    check_case("1500 rows per wave", f, TileParams{1500, 3, 1400, 3}, 1);
    Csr e;
    e.n_rows = 300;
    e.n_cols = 500;
    e.rp.assign(301, 0);
    check_case("no entries", e, TileParams{64, 4, 128, 1}, 1);
    check_case("one row", make_csr(1, 4000, 900, 5, false), TileParams{64, 4, 256, 2}, -1);
    check_case("one column", make_csr(3000, 1, 1, 6, false), TileParams{64, 4, 4, 1}, -1);
    uint64_t rs = 4321;
    for (int k = 0; k < 24 && !failures; ++k) {
        const Csr m = make_csr(1 + lcg(rs) % 12000, 1 + lcg(rs) % 30000, 1 + lcg(rs) % 40, 100 + k, k % 3 == 0);
        const int rws[] = {64, 100, 512, 1024, 1025, 2048}, cbs[] = {12, 1000, 4096, 8188, 16380};
        TileParams t{rws[lcg(rs) % 6], 1 + static_cast<int>(lcg(rs) % 16), cbs[lcg(rs) % 5],
                     1 + static_cast<int>(lcg(rs) % 4)};
        if (t.rw > 1024 && t.cb > 8188) t.cb = 8188;
        while (tile_lds_bytes(t, true) > 163840) t.cb /= 8, t.cb = std::max(4, t.cb / 4 * 4);
        t.ns = static_cast<int>(std::min<int64_t>(t.ns, (m.n_cols + t.cb - 1) / t.cb));
        char name[120];
        std::snprintf(name, sizeof name, "random %d: rw %d, waves %d, cb %d, ns %d", k, t.rw, t.waves, t.cb, t.ns);
        check_case(name, m, t, -1);
    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
