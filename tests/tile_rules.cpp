// Rules of the several-gates-per-sweep path (tile.h) that hold without a GPU.
//
//   tile_rules layout     the programs lie at multiples of 16 bytes
//   tile_rules short      short lists: one sweep, or one for each gate
//   tile_rules strings    few strings on many small rows: sweeps by x or tiles
//   tile_rules single     gates in sweeps of their own get the list's matrices
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../paper_2511_19291_amd/csrc/tile.h"

namespace sv {
void launch_tile_adj(const TileAdjArgs&, int, int, hipStream_t) {}
void launch_sum_slots(const double*, int, int, double*, hipStream_t) {}
void launch_tile(const TileArgs&, int, int, hipStream_t) {}
void fail(sv_status, const std::string& msg)
{
    std::fprintf(stderr, "%s\n", msg.c_str());
    std::abort();
}
void hip_check(hipError_t, const char*) {}
const DeviceInfo& device_info()
{
    static DeviceInfo d;
    d.cu_count = 256;
    return d;
}
}  // namespace sv

// The kernels read headers and matrices as 16-byte words from `words` on; the
// kernel arguments themselves lie at a multiple of 16.
static int layout()
{
    const size_t run = offsetof(sv::TileArgs, words), adj = offsetof(sv::TileAdjArgs, words);
    std::printf("words at %zu and %zu\n", run, adj);
    // the matrices of a list for every row are found past 2^31 floats (16000 U3 on 16384 rows)
    if (sizeof(sv::TileGate::mat) < 8) return 1;
    return run % 16 == 0 && adj % 16 == 0 && alignof(sv::TileArgs) % 16 == 0 && alignof(sv::TileAdjArgs) % 16 == 0 ? 0 : 1;
}

// Gates that share no sweep get the matrix that the list keeps for them: it is
// scaled by what the gates before it left over, and the gates behind it count on
// that. Every kind of matrix comes back as it was appended, but for that scale
// and the rounding; and over a list with many lone gates the norm stays within
// one rounding.
static int single()
{
    using sv::cd;
    const double c = std::cos(0.3), s = std::sin(0.3);
    // kinds: general, real, imaginary off-diagonal, phases, exchange, 4 x 4; one matrix or two
    for (int kind = 0; kind < 9; ++kind)
        for (int rows = 1; rows <= 2; ++rows) {
            const int k = kind >= 6 ? 2 : 1, D = 1 << k, targets[2] = {7, 3}, control = 9, nc = kind == 4;
            std::vector<cd> ms;
            for (int r = 0; r < rows; ++r) {
                const double a = 0.4 + r, ca = std::cos(a), sa = std::sin(a);
                const cd p = std::polar(1.0, 0.3 + r);
                std::vector<cd> m(D * D);
                if (kind == 0) m = {ca, -sa * p, sa, ca * p};
                if (kind == 1) m = {ca, -sa, sa, ca};
                if (kind == 2) m = {ca, cd(0, -sa), cd(0, -sa), ca};
                if (kind == 3) m = {std::conj(p), 0.0, 0.0, p};
                if (kind == 4) m = {1.0, 0.0, 0.0, p};
                if (kind == 5) m = {0.0, 1.0, 1.0, 0.0};
                if (kind == 6) for (int i = 0; i < 4; ++i) m[5 * i] = std::polar(1.0, 0.2 * i * i + r);
                if (kind == 7) m[0] = m[6] = m[9] = m[15] = 1.0;
                if (kind == 8) m = {ca, 0, 0, -sa * p, 0, ca, -sa, 0, 0, sa, ca, 0, sa, 0, 0, ca * p};
                ms.insert(ms.end(), m.begin(), m.end());
            }
            sv::TileList list;
            sv::tile_append(list, k, targets, nc, &control, ms.data(), rows, 0);
            const sv::TileGate& g = list.gates[0];
            for (int r = 0; r < (g.per_row ? rows : 1); ++r) {
                cd m[16];
                sv::tile_matrix(list, g, r, m);
                if (g.k == 0) {                       // a phase on the all-ones pattern
                    if (std::abs(m[0] - ms[r * D * D + D * D - 1]) > 2e-7) return 1;
                    continue;
                }
                for (int i = 0; i < D * D; ++i)
                    if (std::abs(m[i] - ms[r * D * D + i]) > 2e-7) return 1;
            }
        }
    // rotations on twelve qubits, and one on a thirteenth, which is left alone
    int differ = 0;
    for (int count = 24; count <= 200; ++count) {
        sv::TileList list;
        const int n = 13, last = 12;
        const cd rx[4] = {c, cd(0, -s), cd(0, -s), c};
        for (int i = 0; i < count; ++i) {
            const int q = i % 12;
            sv::tile_append(list, 1, &q, 0, nullptr, rx, 1, i);
        }
        sv::tile_append(list, 1, &last, 0, nullptr, rx, 1, count);
        const float* want = list.pool.data() + list.gates[count].mat;
        int lone = 0;
        bool same = true;
        sv::tile_run(sv::Rows{nullptr, nullptr, 1, 1, 1ull << n}, n, list, nullptr, [&](const sv::TileGate& g) {
            cd m[16];
            sv::tile_matrix(list, g, 0, m);
            ++lone;
            same = same && g.op == count && (float)m[0].real() == want[0] && (float)m[1].imag() == want[1];
            differ += want[0] != (float)c || want[1] != (float)-s;
        });
        if (lone != 1 || !same) return 1;
    }
    return differ > 0 ? 0 : 1;                        // (the scale is seen at all)
}

// Lists of a few gates, each of which touches 2^-controls of the state: whether
// they share a sweep. The sides are as measured on an MI355X, where one of them
// is clearly the faster.
static int short_lists()
{
    const struct {
        int n, gates, controls, rows;
        bool own_rows, together;
    } cases[] = {
        // two gates: 18.5 against 29.4 us, 17.9 : 21.3, 17.0 : 18.3
        {22, 2, 3, 1, false, false}, {20, 2, 3, 1, false, false}, {10, 2, 3, 1, false, false},
        // 18.0 : 19.2, 17.4 : 18.9, 7.9 : 6.9 (among others), 17.5 : 16.3
        {18, 2, 1, 1, false, false}, {16, 2, 1, 1, false, false}, {10, 2, 1, 1, false, true}, {4, 2, 0, 1, false, true},
        // two CX: 167 : 202, 88 : 100, 47 : 52, 26 : 28.6, 38.8 : 43.7 (behind a reset); 10.3 : 9.1 at 21 qubits
        {26, 2, 1, 1, false, false}, {25, 2, 1, 1, false, false}, {24, 2, 1, 1, false, false}, {23, 2, 1, 1, false, false},
        {22, 2, 1, 1, false, false}, {21, 2, 1, 1, false, true},
        // three CX: 249 : 203, 23.3 : 14.5, 9.5 : 6.8; three with three controls 9.9 : 16.2 on 22
        {26, 3, 1, 1, false, true}, {22, 3, 1, 1, false, true}, {12, 3, 1, 1, false, true}, {22, 3, 3, 1, false, false},
        {21, 3, 3, 1, false, false},
        // without controls: 321 : 198, 26 : 14, 12.8 : 8.5
        {26, 2, 0, 1, false, true}, {22, 2, 0, 1, false, true}, {20, 2, 0, 1, false, true},
        // matrices per row take a launch per row
        {12, 2, 0, 8, true, true}, {14, 2, 2, 3, true, true}, {20, 3, 1, 8, true, true},
        // long lists
        {26, 40, 3, 1, false, true}};
    const sv::cd u[4] = {0.8, sv::cd(0.0, -0.6), sv::cd(0.0, -0.6), 0.8};
    for (const auto& k : cases) {
        sv::TileList list;
        std::vector<sv::cd> ms;
        for (int r = 0; r < (k.own_rows ? k.rows : 1); ++r) ms.insert(ms.end(), u, u + 4);
        for (int i = 0; i < k.gates; ++i) {
            const int target = i % 3, controls[3] = {k.n - 1, k.n - 2, k.n - 3};
            sv::tile_append(list, 1, &target, k.controls, controls, ms.data(), k.own_rows ? k.rows : 1, i);
        }
        sv::TilePlannerHandle plan(list, k.n, k.rows);
        sv::TileSweep w;
        if (!plan.next(w) || (int)w.gates.size() != k.gates) return 1;
        if (w.single == k.together) {
            std::printf("%d qubits, %d rows, %d gates with %d controls: %s\n", k.n, k.rows, k.gates, k.controls,
                        w.single ? "a sweep each" : "one sweep");
            return 1;
        }
    }
    return 0;
}

// Sets of strings with as many x as strings (or two, or one): whether they go into
// a tile sweep, as measured on an MI355X where one side is clearly the faster.
static int strings()
{
    const struct {
        int n, rows, count, xs;
        bool tiles;
    } cases[] = {
        // 276 us by x, 367 in tiles; 389 : 480; 66 : 74
        {6, 60000, 2, 2, false}, {6, 60000, 3, 3, false}, {6, 8000, 2, 2, false}, {9, 60000, 3, 3, false}, {7, 60000, 5, 5, false}, {4, 60000, 8, 2, false},
        // 45 : 37, 149 : 125, 2657 : 2236, 28 : 25
        {6, 1000, 3, 3, true}, {6, 8000, 5, 5, true}, {6, 60000, 20, 20, true}, {6, 100, 2, 2, true},
        // 1125 : 353; single rows of any width
        {13, 20000, 3, 3, true}, {8, 1, 2, 2, true}, {12, 1, 3, 3, true}, {24, 1, 2, 2, true},
        // one x: 21.5 : 23.3 at 8 qubits, 32.2 : 24.9 at 20
        {8, 1, 8, 1, false}, {20, 1, 8, 1, true},
        // x wider than a tile
        {16, 1, 300, 0, false}, {24, 1, 300, 0, false}};
    for (const auto& k : cases) {
        std::vector<uint64_t> x(k.count), z(k.count);
        for (int i = 0; i < k.count; ++i) {
            x[i] = k.xs ? 1 + i % k.xs : (1ull << k.n) - 1 - (i % 2);
            z[i] = k.xs ? i / k.xs : i;
        }
        std::vector<sv::PauliSweep> sweeps;
        std::vector<int> rest;
        sv::plan_pauli_tiles(k.n, k.rows, x.data(), z.data(), k.count, sweeps, rest);
        size_t placed = rest.size();
        for (const auto& w : sweeps) placed += w.terms.size();
        if (placed != (size_t)k.count || rest.empty() != k.tiles) {
            std::printf("%d qubits, %d rows, %d strings of %d x: %zu by x\n", k.n, k.rows, k.count, k.xs, rest.size());
            return 1;
        }
    }
    return 0;
}

int main(int argc, char** argv)
{
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "layout")) return layout();
    if (!std::strcmp(argv[1], "short")) return short_lists();
    if (!std::strcmp(argv[1], "strings")) return strings();
    if (!std::strcmp(argv[1], "single")) return single();
    return 2;
}
