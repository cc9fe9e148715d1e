// Host-only checks of the choices that the library makes before it launches
// anything (this file includes the library source; no GPU is touched):
//   * arrays are used in place only where they are device memory of the GPU that
//     reads them;
//   * a tiled copy that ends in 32-bit lists (streaming refused, tiles too tall and
//     wide for 24 bits) gives the row sums, walked as the kernel does;
//   * a small scan's second copy is left out where it would be mostly padding, and
//     the memory estimate follows the formats that are taken;
//   * the automatic schedule of sparse matrices ends in streamed lists, that of a
//     matrix whose entries lie in a band takes lower tiles.
// Prints one line per case and "ok" at the end; exits 1 after a failure.
#include "../../paper_1601_08201_amd/csrc/sgtv_api.hip"

#include <cstdio>
#include <set>

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

// len(r) entries in row r, in uniform columns; band: in a tenth of the columns
// that moves on with the row
template <class Len>
Csr make_csr(int64_t n_rows, int64_t n_cols, uint64_t seed, Len len, bool band = false) {
    Csr m;
    m.n_rows = n_rows;
    m.n_cols = n_cols;
    m.rp.push_back(0);
    uint64_t s = seed;
    for (int64_t r = 0; r < n_rows; ++r) {
        for (int64_t e = len(r); e > 0; --e) {
            m.ci.push_back(static_cast<int32_t>(band ? r * (n_cols - n_cols / 10) / n_rows + lcg(s) % (n_cols / 10)
                                                     : lcg(s) % n_cols));
            m.v.push_back(static_cast<float>(lcg(s) % 1000 + 1) / 997.0f);
        }
        std::sort(m.ci.begin() + m.rp.back(), m.ci.end());
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

void check_memory() {
    hipPointerAttribute_t a{};
    a.type = hipMemoryTypeDevice;
    a.device = 1;
    CHECK(lies_on(a, 1), "own memory");
    CHECK(!lies_on(a, 0), "another GPU's memory");
    for (const hipMemoryType t : {hipMemoryTypeHost, hipMemoryTypeManaged, hipMemoryTypeUnregistered}) {
        a.type = t;
        CHECK(!lies_on(a, 1), "memory type %d", static_cast<int>(t));
    }
    std::printf("memory in place\n");
}

// The 32-bit lists of a copy as tiled_body walks them: groups of 64 lanes (four
// groups a batch, the rest one by one), row sums read through the slot table.
void check_lists32(const char *name, const Csr &m, TileParams t) {
    PackedTiled T;
    CHECK(pack_tiled(T, m.n_rows, m.n_cols, m.rp, m.ci, m.v, t, true) == SGTV_OK, "%s: packing failed", name);
    const sgtv::TileMap &M = T.map;
    CHECK(M.idx24 == 0, "%s: format %d", name, M.idx24);
    const int64_t RB = static_cast<int64_t>(M.waves) * M.rw;
    std::vector<double> ref(static_cast<size_t>(m.n_rows * M.ns), 0.0), got(ref.size(), 0.0);
    std::vector<int> slab_of;
    for (int k = 0; k < M.ns; ++k) slab_of.insert(slab_of.end(), M.slab_begin[k + 1] - M.slab_begin[k], k);
    for (int64_t r = 0; r < m.n_rows; ++r)
        for (int64_t k = m.rp[r]; k < m.rp[r + 1]; ++k)
            ref[slab_of[m.ci[k] / M.cb] * m.n_rows + r] += m.v[k] * static_cast<double>(m.ci[k] % 97 + 1);
    for (int64_t tile = 0; tile < M.n_rb * M.ns; ++tile) {
        const int64_t rb = tile / M.ns;
        const int slab = static_cast<int>(tile % M.ns);
        std::vector<double> acc(static_cast<size_t>(M.waves) * (M.rw + 1), 0.0);
        for (int c = M.slab_begin[slab]; c < M.slab_begin[slab + 1]; ++c)
            for (int w = 0; w < M.waves; ++w) {
                const int64_t L = (tile * M.cbs_max + (c - M.slab_begin[slab])) * M.waves + w;
                const int64_t base = static_cast<int64_t>(T.goff[L]) * 64, ng = T.goff[L + 1] - T.goff[L];
                for (int64_t g = 0; g < ng; ++g) {
                    std::set<int> rows;
                    for (int lane = 0; lane < 64; ++lane) {
                        const int64_t pos = g < ng / 4 * 4 ? base + g / 4 * 256 + lane * 4 + g % 4 : base + g * 64 + lane;
                        const int row = T.pk[pos] >> 16, col = T.pk[pos] & 0xFFFF;
                        CHECK(row <= M.rw && (row == M.rw || rows.insert(row).second), "%s: two lanes on a row", name);
                        if (row < M.rw)
                            acc[w * (M.rw + 1) + row] +=
                                T.v32[pos] * static_cast<double>((static_cast<int64_t>(c) * M.cb + col) % 97 + 1);
                    }
                }
            }
        for (int64_t i = 0; i < RB && rb * RB + i < m.n_rows; ++i) {
            const int64_t s = T.slot.empty() ? i : T.slot[tile * RB + i];
            got[slab * m.n_rows + rb * RB + i] = acc[s / M.rw * (M.rw + 1) + s % M.rw];
        }
    }
    for (size_t i = 0; i < ref.size(); ++i)
        CHECK(std::fabs(got[i] - ref[i]) <= 1e-9 * (1.0 + std::fabs(ref[i])), "%s: row %lld", name,
              static_cast<long long>(i) % static_cast<long long>(m.n_rows));
    // saved copies of this format with dealt rows are refused
    const int64_t goff = 4 * static_cast<int64_t>(T.goff.size());
    CHECK(tiles_consistent(M, goff, 0, 0) && !tiles_consistent(M, goff, 0, 2 * M.n_rb * M.ns * RB), "%s: sizes", name);
    std::printf("%s: 32-bit lists\n", name);
}

// The automatic schedule of a product and the format its copy gets.
void check_automatic(const char *name, const Csr &m, int want, int tallest) {
    const int64_t nnz = m.rp[m.n_rows];
    const LoadMap loads = load_map(m.n_rows, m.n_cols, m.rp, m.ci);
    const TileParams t = choose_tiles(m.n_rows, m.n_cols, nnz, 4, 0, 0, 0, 0, true, &loads);
    const TileParams even = choose_tiles(m.n_rows, m.n_cols, nnz, 4, 0, 0, 0, 0);
    PackedTiled T;
    CHECK(pack_tiled(T, m.n_rows, m.n_cols, m.rp, m.ci, m.v, t, true) == SGTV_OK, "%s: packing failed", name);
    const double bytes = 4.0 * (T.pk.size() + T.v32.size() + T.goff.size() + T.poff.size());
    std::printf("%s: %d x %d, %d slabs (even entries: %d x %d, %d), format %d, %.2f bytes an entry\n", name, t.rw, t.cb,
                t.ns, even.rw, even.cb, even.ns, T.map.idx24, bytes / nnz);
    CHECK(want < 0 || T.map.idx24 == want, "%s: format %d", name, T.map.idx24);
    CHECK(t.rw <= tallest, "%s: %d rows per wave", name, t.rw);
    if (tallest >= 2048) CHECK(t.rw == even.rw && t.cb == even.cb && t.ns == even.ns, "%s: not the even schedule", name);
}

void check_rules() {
    // the pipelined loops read 32-bit lists: the schedule is not the modelled one
    const TileParams p = choose_tiles(1 << 20, 1 << 21, 1 << 26, 4, 0, 0, 0, 0, false);
    CHECK(p.rw == 1024 && p.cb == 16380 && p.ns == 4, "pipelined loop: %d x %d, %d", p.rw, p.cb, p.ns);
    // two column blocks are not streamed: 24-bit lists must fit
    for (const int64_t rows : {int64_t(3000000), int64_t(5000000), int64_t(9000000)}) {
        const TileParams t = choose_tiles(rows, 30000, 20 * rows, 4, 0, 0, 0, 0);
        CHECK(sgtv::idx24_fits(t.rw, t.cb), "30000 columns: %d x %d", t.rw, t.cb);
    }
    std::printf("rules of the schedule\n");
}

// len(j) entries in voxel j of a scan of ny x nx x Q, in uniform measurements:
// does it get the second copy of a small scan
// (want 1, 0; -1 either)?
template <class Len>
void check_small(const char *name, int64_t I, int ny, int nx, int Q, int want, Len len, bool even = true) {
    const Csr t = make_csr(static_cast<int64_t>(ny) * nx * Q, I, 11, len);
    std::vector<int64_t> rp, lrp = t.rp;
    std::vector<int32_t> ci;
    std::vector<float> v;
    transpose_csr(t.n_rows, I, t.rp, t.ci, t.v, rp, ci, v);
    sgtv_ctx_s c;
    Packed PK;
    CHECK(pack_system(&c, PK, I, ny, nx, Q, rp.data(), ci.data(), v.data(), rp.back(), SGTV_F32, nullptr, 0, SGTV_HOST) ==
              SGTV_OK, "%s: packing failed", name);
    const double tiles = 8.0 * (PK.fwd.v32.size() + PK.back.v32.size());
    const double copy = 8.0 * (PK.rsv32.size() + PK.csv32.size());
    std::printf("%s: %lld entries, tiles %.1f MB, second copy %.1f MB\n", name, static_cast<long long>(rp.back()),
                tiles / 1e6, copy / 1e6);
    CHECK(want < 0 || PK.S->small() == (want == 1), "%s: %s", name, want ? "no second copy" : "a second copy");
    CHECK(copy <= 3.3 * tiles + 1048576.0, "%s: second copy of %.0f MB", name, copy / 1e6);
    if (!even) return;
    // the estimate of the memory that is held, within a quarter
    double held = 4.0 * (3 * t.n_rows + 8 * t.n_rows + 4 * t.n_rows + 3 * I) + 4.0 * (PK.fpart_floats + PK.bpart_floats) +
                  8.0 * (PK.rsv32.size() + PK.csv32.size()) + 1048576.0;
    for (const PackedTiled *T : {&PK.fwd, &PK.back})
        held += 4.0 * (T->pk.size() + T->v32.size() + T->goff.size() + T->poff.size()) + 2.0 * T->slot.size();
    const double est = static_cast<double>(sgtv_workspace_bytes(I, t.n_rows, rp.back(), SGTV_F32));
    std::printf("%s: held %.1f MB, estimate %.1f MB, formats %d %d\n", name, held / 1e6, est / 1e6, PK.fwd.map.idx24,
                PK.back.map.idx24);
    CHECK(std::fabs(est - held) <= 0.25 * held, "%s: estimate", name);
}

void check_format(const char *name, const Csr &m, TileParams t, int want) {
    PackedTiled T;
    CHECK(pack_tiled(T, m.n_rows, m.n_cols, m.rp, m.ci, m.v, t, true) == SGTV_OK, "%s: packing failed", name);
    CHECK(T.map.idx24 == want, "%s: format %d", name, T.map.idx24);
    CHECK(tiles_consistent(T.map, 4 * T.goff.size(), 4 * T.poff.size(), 2 * T.slot.size()), "%s: sizes", name);
    std::printf("%s: format %d\n", name, want);
}

}  // namespace

int main() {
    check_memory();
    check_rules();
    const int S = sgtv::kIdxStream;
    // the shapes that tests/test_gpu_stream.py takes for streamed ones
    check_format("13 bits, full block", make_csr(30000, 19926, 1, [](int64_t) { return 16; }), TileParams{64, 16, 4092, 1}, S);
    check_format("14 bits, widest block, back", make_csr(35420, 50000, 1, [](int64_t) { return 24; }),
                 TileParams{100, 16, 16380, 1}, S);
    check_format("all of the LDS", make_csr(60000, 32768, 1, [](int64_t) { return 13; }), TileParams{2048, 16, 8188, 1}, S);
    check_format("narrow blocks, slabs", make_csr(3001, 3003, 1, [](int64_t) { return 16; }), TileParams{65, 4, 256, 3}, S);
    check_format("one wave, back", make_csr(930, 700, 1, [](int64_t) { return 9; }), TileParams{300, 1, 100, 1}, S);
    check_format("one row, three blocks", make_csr(1, 768, 1, [](int64_t) { return 768; }), TileParams{64, 16, 256, 1}, S);
    check_small("16 a voxel", 4096, 16, 16, 32, 1, [](int64_t) { return 16; });
    check_small("24 a voxel", 8192, 9, 41, 54, 1, [](int64_t) { return 24; });
    check_small("9 a voxel", 131072, 64, 64, 64, 1, [](int64_t) { return 9; });
    check_small("1 a voxel", 131072, 64, 64, 64, 1, [](int64_t) { return 1; });
    check_small("1 a voxel, 20000 measurements", 20000, 128, 128, 128, 1, [](int64_t) { return 1; });
    check_small("32 a voxel", 131072, 64, 64, 64, 0, [](int64_t) { return 32; });
    check_small("8 a voxel, 128 x 128 x 64", 524288, 128, 128, 64, 0, [](int64_t) { return 8; });
    check_small("8 a voxel, 128^3", 1 << 20, 128, 128, 128, 0, [](int64_t) { return 8; });
    check_small("16 a voxel, 60 x 100 x 100", 600000, 60, 100, 100, 0, [](int64_t) { return 16; });
    check_small("3 a voxel, 100 x 100 x 100", 400000, 100, 100, 100, 0, [](int64_t) { return 3; });
    check_small("24 a voxel, 77 x 101 x 40", 150001, 77, 101, 40, 0, [](int64_t) { return 24; });
    check_small("one entry", 1, 1, 1, 1, 1, [](int64_t) { return 1; });
    check_small("150 in every 64th voxel, 2 in the others", 131072, 64, 64, 64, 0,
                [](int64_t j) { return j % 64 ? 2 : 150; }, false);
    check_small("150 in every 64th voxel", 131072, 64, 128, 100, 0, [](int64_t j) { return j % 64 ? 0 : 150; }, false);
    check_small("40 in every 64th voxel, 2 in the others", 131072, 64, 64, 64, 1, [](int64_t j) { return j % 64 ? 2 : 40; }, false);
    check_small("60 in every 16th voxel, 4 in the others", 131072, 64, 64, 64, -1,
                [](int64_t j) { return j % 16 ? 4 : 60; }, false);
    check_automatic("128 x 128 x 64, 4 a voxel", make_csr(524288, 1048576, 3, [](int64_t) { return 8; }), S, 2048);
    check_automatic("128 x 128 x 64, 4 a voxel, back", make_csr(1048576, 524288, 3, [](int64_t) { return 4; }), S, 2048);
    check_automatic("128^3, 4 a voxel", make_csr(1 << 20, 1 << 21, 3, [](int64_t) { return 8; }), S, 2048);
    check_automatic("128^3, 8 a voxel", make_csr(1 << 20, 1 << 21, 3, [](int64_t) { return 16; }), S, 2048);
    check_automatic("128^3, 8 a voxel, back", make_csr(1 << 21, 1 << 20, 3, [](int64_t) { return 8; }), S, 2048);
    check_automatic("128^3, 16 a voxel", make_csr(1 << 20, 1 << 21, 4, [](int64_t) { return 32; }), S, 2048);
    check_automatic("100 x 100 x 110, 16 a voxel", make_csr(800000, 1100000, 5, [](int64_t) { return 22; }), S, 2048);
    check_automatic("120 x 110 x 90, 20 a voxel, back", make_csr(1188000, 1000000, 6, [](int64_t) { return 20; }), S, 2048);
    check_automatic("128 x 128 x 64, 8 a voxel", make_csr(524288, 1048576, 7, [](int64_t) { return 16; }), S, 2048);
    check_automatic("128^3, 8 a voxel in a band", make_csr(1 << 20, 1 << 21, 9, [](int64_t) { return 16; }, true), S, 1024);
    check_automatic("64^3, 32 a voxel in a band", make_csr(131072, 262144, 9, [](int64_t) { return 64; }, true), -1, 256);
    check_automatic("96^3, 16 a voxel", make_csr(442368, 884736, 8, [](int64_t) { return 32; }), -1, 2048);
    check_lists32("even rows", make_csr(40000, 50000, 1, [](int64_t) { return 3; }), TileParams{1500, 16, 15000, 2});
    check_lists32("uneven rows", make_csr(60001, 70001, 2, [](int64_t r) { return r % 9 == 4 ? 0 : 1 + r % 70; }),
                  TileParams{1400, 16, 16000, 3});
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
