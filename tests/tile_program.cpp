// Executes the programs of the several-gates-per-sweep path (tile.h) on the
// CPU in double precision and compares them with the gates applied one by one.
// Random lists of every kind the planner distinguishes: general, real,
// imaginary off-diagonal, phases, exchanges, 4 x 4; 0..3 controls anywhere;
// one matrix or one per row.
//
//   tile_program FIRST_SEED SEEDS COMPUTE_UNITS
// COMPUTE_UNITS decides between three and four register bits.
#include <algorithm>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../paper_2511_19291_amd/csrc/tile.h"

using sv::cd;
using sv::TileArgs;

static std::vector<cd> psi;
static int cu_count = 256;
static int launches = 0;

static uint32_t element(uint32_t index)
{
    uint32_t e = 0;
    for (int b = 0; b < sv::kTileMaxBits; ++b)
        if ((index >> b) & 1) e ^= (1u << b) ^ (b >= 4 ? sv::kTileSwz[b - 4] : 0u);
    return e;
}

static float as_float(uint32_t w)
{
    float f;
    std::memcpy(&f, &w, 4);
    return f;
}

static cd entry(const uint32_t* m, int i) { return cd(as_float(m[2 * i]), as_float(m[2 * i + 1])); }

// One workgroup: tile `tile` of row a.row0 + y.
static void run_tile(const TileArgs& a, int R, uint32_t tile, int y)
{
    const int T = a.T, M = 1 << R, threads = 1 << (T - R);
    uint64_t base = tile;
    for (int i = 0; i < T; ++i) base = ((base >> a.pos[i]) << (a.pos[i] + 1)) | (base & ((1ull << a.pos[i]) - 1));
    auto place = [&](uint32_t e) {
        uint64_t o = (uint64_t)(a.row0 + y) * a.N + base;
        for (int b = 0; b < T; ++b)
            if ((e >> b) & 1) o += 1ull << a.pos[b];
        return o;
    };
    std::vector<cd> lds(1 << sv::kTileMaxBits), out(1 << sv::kTileMaxBits);
    for (uint32_t e = 0; e < (1u << T); ++e) lds[element(e)] = psi[place(e)];
    const uint32_t* pc = a.words;
    for (int r = 0; r < a.nrounds; ++r) {
        const uint32_t r0 = pc[0];
        const int steps = r0 & 255, nouter = (r0 >> 8) & 255;
        const bool mapped = (r0 >> 18) & 1;
        const uint32_t* first = pc + sv::kTileRoundWords + (mapped ? sv::kTileMapWords + ((nouter + 3) & ~3) : 0);
        const uint32_t* end = first;
        std::vector<char> written(1 << sv::kTileMaxBits, 0);
        for (int t = 0; t < threads; ++t) {
            auto columns = [&](int c, int c2) {
                uint32_t v = 0;
                for (int k = 0; k < T - R; ++k)
                    if ((t >> k) & 1) v ^= ((k < 8 ? pc[c + k / 2] : pc[c2 + (k - 8) / 2]) >> (16 * (k & 1))) & 0xffff;
                return v;
            };
            auto reg = [&](int c, int j) {
                uint32_t v = 0;
                for (int k = 0; k < R; ++k)
                    if ((j >> k) & 1) v ^= (pc[c + k / 2] >> (16 * (k & 1))) & 0xffff;
                return v;
            };
            uint32_t tix = 0;
            for (int k = 0; k < T - R; ++k)
                if ((t >> k) & 1) tix |= 1u << (((k < 8 ? pc[7] : pc[9]) >> (4 * (k & 7))) & 15);
            const uint32_t* ps = first;
            cd own = 1.0;
            auto lanes = [&](const uint32_t* h) {
                const uint32_t ctl = (h[0] >> 16) & 0xfff;
                return (tile & h[1]) == h[1] && (tix & ctl) == ctl;
            };
            auto phase = [&](const uint32_t* h, int j) {
                const int nfree = (h[3] >> 16) & 3;
                auto bit = [&](int i) {
                    const int at = (h[3] >> (8 * i)) & 255, where = (h[3] >> (20 + 2 * i)) & 3;
                    return (int)(((where == sv::kPlaceReg ? (uint32_t)j : where == sv::kPlaceThread ? tix : tile) >> at) & 1);
                };
                return entry(a.words + (h[2] & 0xffff) + (h[2] >> 16) * y,
                             nfree == 0 ? 0 : nfree == 1 ? bit(0) : 2 * bit(0) + bit(1));
            };
            for (int g = r0 >> 24; g > 0; --g, ps += sv::kTileHeadWords)
                if (lanes(ps)) own *= ps[0] & sv::TF_SIGN ? cd(-1.0) : phase(ps, 0);
            const uint32_t at = columns(1, 8);
            cd x[16];
            for (int j = 0; j < M; ++j) x[j] = lds[at ^ reg(5, j)];
            uint32_t flips = 0;
            for (int g = 0; g < steps; ++g, ps += sv::kTileHeadWords) {
                const uint32_t* h = ps;
                auto one_target = [&](int b, const cd (&m)[4], auto&& on) {
                    for (int j = 0; j < M; ++j)
                        if (!((j >> b) & 1) && on(j)) {
                            const cd u = x[j], v = x[j | 1 << b];
                            x[j] = m[0] * u + m[1] * v;
                            x[j | 1 << b] = m[2] * u + m[3] * v;
                        }
                };
                if (h[0] & sv::TF_LAYER) {
                    for (int b = 0; b < R; ++b) {
                        if (!((h[0] >> (8 + b)) & 1)) continue;
                        const uint32_t* w = a.words + h[2] * y + 4 * ((h[1] >> (8 * b)) & 255);
                        cd m[4] = {};
                        for (int i = 0; i < 4; ++i) {
                            if (h[0] & sv::TF_DENSE) m[i] = entry(w, i);
                            if (h[0] & sv::TF_REAL) m[i] = as_float(w[i]);
                            if (h[0] & sv::TF_IMOFF) m[i] = i == 0 || i == 3 ? cd(as_float(w[i])) : cd(0.0, as_float(w[i]));
                        }
                        if (h[0] & sv::TF_DIAG) m[0] = entry(w, 0), m[3] = entry(w, 1);
                        one_target(b, m, [](int) { return true; });
                    }
                    continue;
                }
                const uint32_t rcm = (h[0] >> 8) & 15;
                const uint32_t* w = a.words + (h[2] & 0xffff) + (h[2] >> 16) * y;
                auto on = [&](int j) { return lanes(h) && ((uint32_t)j & rcm) == rcm; };
                if (h[0] & sv::TF_SIGN) flips ^= (tile & h[1]) == h[1] ? h[3] : 0u;
                if (h[0] & sv::TF_APPLY) {
                    for (int j = 0; j < M; ++j)
                        if ((flips >> j) & 1) x[j] = -x[j];
                    flips = 0;
                }
                if (h[0] & sv::TF_LANE_SIGN)
                    for (int j = 0; j < M; ++j)
                        if (lanes(h) && ((h[3] >> j) & 1)) x[j] = -x[j];
                if (h[0] & sv::TF_PHASE)
                    for (int j = 0; j < M; ++j)
                        if (on(j)) x[j] *= phase(h, j);
                if (h[0] & sv::TF_CTRL) {
                    const cd m[4] = {entry(w, 0), entry(w, 1), entry(w, 2), entry(w, 3)};
                    one_target(__builtin_ctz(h[3]), m, on);
                }
                if (h[0] & sv::TF_DENSE2) {
                    static const int hi[] = {1, 2, 2, 3, 3, 3}, lo[] = {0, 0, 1, 0, 1, 2};
                    const int A = hi[__builtin_ctz(h[3])], B = lo[__builtin_ctz(h[3])];
                    for (int j = 0; j < M; ++j) {
                        if (((j >> A) & 1) || ((j >> B) & 1) || !on(j)) continue;
                        cd v[4];
                        for (int i = 0; i < 4; ++i) v[i] = x[j | (i >> 1) << A | (i & 1) << B];
                        for (int i = 0; i < 4; ++i) {
                            cd s = 0.0;
                            for (int q = 0; q < 4; ++q) s += entry(w, 4 * i + q) * v[q];
                            x[j | (i >> 1) << A | (i & 1) << B] = s;
                        }
                    }
                }
            }
            if (flips) std::abort();
            end = ps;
            uint32_t to = at;
            if (mapped) {
                to = columns(12, 16) ^ pc[19];
                for (int i = 0; i < nouter; ++i)
                    if ((tile >> (pc[20 + i] & 31)) & 1) to ^= pc[20 + i] >> 16;
            }
            for (int j = 0; j < M; ++j) {
                const uint32_t d = to ^ reg(mapped ? 17 : 5, j);
                if (d >= (1u << sv::kTileMaxBits) || written[d]) std::abort();
                written[d] = 1;
                out[d] = own * x[j];
            }
        }
        lds = out;
        pc = end;
    }
    if (pc - a.words > a.nwords || a.nwords > sv::kTileWords) std::abort();
    for (uint32_t e = 0; e < (1u << T); ++e) psi[place(e)] = lds[element(e)];
}

namespace sv {
void launch_tile_adj(const TileAdjArgs&, int, int, hipStream_t) { std::abort(); }
void launch_sum_slots(const double*, int, int, double*, hipStream_t) { std::abort(); }
void launch_tile(const TileArgs& a, int rows, int reg_bits, hipStream_t)
{
    ++launches;
    for (int y = 0; y < rows; ++y)
        for (uint32_t t = 0; t < (1u << (__builtin_ctzll(a.N) - a.T)); ++t) run_tile(a, reg_bits, t, y);
}
void fail(sv_status, const std::string& msg)
{
    std::fprintf(stderr, "%s\n", msg.c_str());
    std::abort();
}
void hip_check(hipError_t, const char*) {}
const DeviceInfo& device_info()
{
    static DeviceInfo d;
    d.cu_count = cu_count;
    return d;
}
}  // namespace sv

struct Gate {
    int k, t[2], nc, c[3], nm;
    std::vector<cd> ms;
};

static void apply(const Gate& g, int rows, uint64_t N, std::vector<cd>& v)
{
    const int D = 1 << g.k;
    for (int r = 0; r < rows; ++r)
        for (uint64_t b = 0; b < N; ++b) {
            bool skip = false;
            for (int j = 0; j < g.nc; ++j) skip |= !((b >> g.c[j]) & 1);
            for (int j = 0; j < g.k; ++j) skip |= (b >> g.t[j]) & 1;
            if (skip) continue;
            cd x[4];
            auto at = [&](int i) {
                uint64_t o = b;
                for (int j = 0; j < g.k; ++j)
                    if ((i >> (g.k - 1 - j)) & 1) o |= 1ull << g.t[j];
                return r * N + o;
            };
            for (int i = 0; i < D; ++i) x[i] = v[at(i)];
            for (int i = 0; i < D; ++i) {
                cd s = 0.0;
                for (int q = 0; q < D; ++q) s += g.ms[(g.nm > 1 ? r * D * D : 0) + i * D + q] * x[q];
                v[at(i)] = s;
            }
        }
}

// The scale of a list's matrices as the kernels get them, and as each would be
// rounded by itself: logarithms, summed over the uncontrolled gates; per row.
static int norms()
{
    const double kRounding = std::ldexp(1.01, -24);
    std::mt19937 rng(1);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    double angle = 0.0, most = 0.0;               // the angle whose rounded rotation scales most
    for (int i = 1; i <= 400; ++i) {
        const double a = 0.0005 * i, c = (float)std::cos(a), s = (float)std::sin(a), e = std::abs(c * c + s * s - 1.0) / 2;
        if (e > most) {
            most = e;
            angle = a;
        }
    }
    for (int mode = 0; mode < 5; ++mode) {
        const int rows = mode == 4 ? 3 : 1;
        sv::TileList list;
        double alone = 0.0;
        for (int i = 0; i < 3000; ++i) {
            std::vector<cd> ms;
            for (int r = 0; r < rows; ++r) {
                const double a = mode < 2 ? angle : 3.0 * u(rng), c = std::cos(a), s = std::sin(a);
                const cd p = std::polar(1.0, 3.0 * u(rng)), q = std::polar(1.0, 3.0 * u(rng));
                if (mode == 0 || mode == 4) ms.insert(ms.end(), {c, cd(0, -s), cd(0, -s), c});
                else if (mode == 1) ms.insert(ms.end(), {c, -s, s, c});
                else if (mode == 2) ms.insert(ms.end(), {c, -s * p, s * q, c * p * q});
                else ms.insert(ms.end(), {std::conj(p), 0.0, 0.0, p});
            }
            if (mode == 0) alone += 0.5 * std::log(std::pow((double)(float)std::cos(angle), 2) + std::pow((double)(float)std::sin(angle), 2));
            const int t = i % 6;
            sv::tile_append(list, 1, &t, 0, nullptr, ms.data(), rows, i);
        }
        if (mode == 0 && std::abs(alone) < 1000 * kRounding * 0.3) return 1;      // the list would drift
        for (int r = 0; r < rows; ++r) {
            double sum = 0.0;
            for (const sv::TileGate& g : list.gates) {
                const int words = g.kind == sv::TK_DENSE ? 8 : 4;
                const float* w = list.pool.data() + g.mat + (g.per_row ? r * words : 0);
                double s = 0.0;
                for (int i = 0; i < words; ++i) s += (double)w[i] * w[i];
                sum += 0.5 * std::log(s / 2);
            }
            std::printf("mode %d row %d: %.3g\n", mode, r, sum);
            if (list.gates.size() != 3000 || std::abs(sum) > kRounding) return 1;
        }
    }
    return 0;
}

int main(int argc, char** argv)
{
    if (argc == 2) return norms();
    if (argc != 4) return 2;
    const int first = std::atoi(argv[1]), count = std::atoi(argv[2]);
    cu_count = std::atoi(argv[3]);
    double worst = 0.0;
    for (int seed = first; seed < first + count; ++seed) {
        std::mt19937 rng(seed);
        std::uniform_real_distribution<double> u(-1.0, 1.0);
        const int n = 4 + rng() % 11, rows = 1 + rng() % 3, gates = 1 + rng() % 120;
        const uint64_t N = 1ull << n;
        std::vector<cd> want(rows * N);
        for (cd& v : want) v = cd(u(rng), u(rng));
        psi = want;
        sv::TileList list;
        std::vector<Gate> all;
        for (int i = 0; i < gates; ++i) {
            Gate g{};
            g.k = 1 + (rng() % 4 == 0);
            std::vector<int> q(n);
            for (int j = 0; j < n; ++j) q[j] = j;
            std::shuffle(q.begin(), q.end(), rng);
            g.nc = rng() % 8 == 0 ? 3 : rng() % 2 ? rng() % 2 : rng() % 3;
            if (g.k + g.nc > n) g.nc = 0;
            for (int j = 0; j < g.k; ++j) g.t[j] = q[j];
            for (int j = 0; j < g.nc; ++j) g.c[j] = q[g.k + j];
            g.nm = rows > 1 && rng() % 4 == 0 ? rows : 1;
            const int D = 1 << g.k, kind = rng() % 8;
            for (int r = 0; r < g.nm; ++r) {
                std::vector<cd> m(D * D);
                auto unitary = [&](bool real) {      // Gram-Schmidt
                    for (cd& v : m) v = cd(u(rng), real ? 0.0 : u(rng));
                    for (int a = 0; a < D; ++a) {
                        for (int b = 0; b < a; ++b) {
                            cd s = 0.0;
                            for (int c = 0; c < D; ++c) s += m[a * D + c] * std::conj(m[b * D + c]);
                            for (int c = 0; c < D; ++c) m[a * D + c] -= s * m[b * D + c];
                        }
                        double s = 0.0;
                        for (int c = 0; c < D; ++c) s += std::norm(m[a * D + c]);
                        for (int c = 0; c < D; ++c) m[a * D + c] /= std::sqrt(s);
                    }
                };
                if (kind < 2) unitary(false);
                else if (kind == 2) unitary(true);
                else if (kind == 3) for (int a = 0; a < D; ++a) m[a * D + a] = std::polar(1.0, 3.0 * u(rng));
                else if (kind <= 5) {
                    for (int a = 0; a < D; ++a) m[a * D + a] = 1.0;
                    m[D * D - 1] = kind == 4 ? cd(-1.0) : std::polar(1.0, 3.0 * u(rng));
                } else if (kind == 6) {
                    if (D == 2) m[1] = m[2] = 1.0;
                    else m[0] = m[6] = m[9] = m[15] = 1.0;
                } else if (D == 2) {
                    const double a = 3.0 * u(rng);
                    m[0] = m[3] = std::cos(a);
                    m[1] = m[2] = cd(0.0, -std::sin(a));
                } else unitary(false);
                g.ms.insert(g.ms.end(), m.begin(), m.end());
            }
            sv::tile_append(list, g.k, g.t, g.nc, g.c, g.ms.data(), g.nm, i);
            all.push_back(g);
        }
        for (const Gate& g : all) apply(g, rows, N, want);
        sv::tile_run(sv::Rows{nullptr, nullptr, rows, rows, N}, n, list, nullptr, [&](int op) { apply(all[op], rows, N, psi); });
        double err = 0.0;
        for (size_t i = 0; i < want.size(); ++i) err = std::max(err, std::abs(want[i] - psi[i]));
        worst = std::max(worst, err / std::sqrt((double)N));
        // the matrices are complex64: 2^-24 per entry and gate
        if (!(err <= 120 * 8 * 6e-8 * std::sqrt(2.0 * N))) {
            std::printf("seed %d: n %d, %d rows, %d gates: off by %g\n", seed, n, rows, gates, err);
            return 1;
        }
    }
    std::printf("ok: %d lists, %d programs, worst %g\n", count, launches, worst);
    return 0;
}
