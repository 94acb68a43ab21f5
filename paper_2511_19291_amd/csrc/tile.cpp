// tile.cpp -- host side of the several-gates-per-sweep path (tile.h): which
// gates a sweep takes, how they fall into rounds, and the program the kernel
// reads.
#include <algorithm>
#include <array>
#include <cstring>
#include <functional>

#include "tile.h"

namespace sv {

namespace {

// floats of one matrix by TileKind (multiples of four: read as 16-byte words)
constexpr int kMatFloats[] = {8, 4, 4, 4, 8, 4, 0, 32, 0};

// Lowest qubits that every tile of a larger state holds: runs of 2^5
// amplitudes = 256 contiguous bytes. With runs of one line (2^4) a tile has a
// qubit more to choose and lists need fewer sweeps (27-qubit brickwork 19 instead
// of 23), which take as much longer: 21.7 ms against 21.9 (0.7 % between runs),
// the step of the 25-qubit ring 18.6 against 19.3 (3 %), 20-qubit brickwork 0.69
// against 0.71 (4 %).
constexpr int kRunBits = 5;

// Ready gates looked at for each register bit of a round: the choice costs
// host time, which small states do not hide, and more of them find the same
// rounds on layered circuits.
constexpr int kRoundOptions = 4;

// The gates that can be applied next, as a set of qubits grows. On each
// qubit consecutive gates that are diagonal there (controls, phases) form one
// group, whose gates commute on that qubit; any other gate is a group of its
// own. A gate is ready when its group is the current one on each of its
// qubits.
class Frontier {
public:
    Frontier(const TileList& l, const std::vector<int>& ids, int n) : n_(n)
    {
        const int G = (int)ids.size();
        use_.resize(G);
        stamp_.assign(G, 0);
        std::vector<char> last_z(n, 0);
        for (int i = 0; i < G; ++i) {
            const TileGate& g = l.gates[ids[i]];
            Use& u = use_[i];
            const bool diag = g.kind == TK_DIAG1 || g.kind == TK_DIAG2;
            // a derivative is formed on register amplitudes
            if (g.deriv) u.need |= 1ull << g.targets[0];
            u.map = g.kind == TK_MAP;
            auto add = [&](int q, bool z) {
                if (start_[q].empty() || !(z && last_z[q])) {
                    start_[q].push_back((uint32_t)item_[q].size());
                    last_z[q] = z;
                }
                item_[q].push_back((uint32_t)i);
                u.q[u.n] = (uint8_t)q;
                u.grp[u.n++] = (uint32_t)start_[q].size() - 1;
            };
            for (int j = 0; j < g.nc; ++j) add(g.controls[j], true);
            for (int j = 0; j < g.k; ++j) {
                add(g.targets[j], diag);
                if (!diag) u.need |= 1ull << g.targets[j];
            }
        }
        for (int q = 0; q < n; ++q) at_.open(*this, q, 0);
        left_ = G;
    }

    int left() const { return left_; }

    // Which gates a call may place: any, all but index maps, index maps only.
    enum Kinds { kAny, kNoMaps, kMaps };

    // Place every gate that can be applied with the qubits of S; they are
    // appended (as positions in ids) to `out`.
    void take(uint64_t S, std::vector<int>& out, Kinds kinds)
    {
        kinds_ = kinds;
        ++now_;
        queue_.clear();
        for (int q = 0; q < n_; ++q) push_group(q);
        const size_t first = out.size();
        close(S, &out);
        for (size_t i = first; i < out.size(); ++i) stamp_[out[i]] = kDone;
        left_ -= (int)(out.size() - first);
    }

    // Grow S to at most `width` qubits, each time by the qubits of the ready
    // gate, among the `most` earliest, that lets the most gates be placed per
    // qubit (ties: the earliest), placing them.
    uint64_t grow(uint64_t S, int width, std::vector<int>& out, Kinds kinds, int most)
    {
        take(S, out, kinds);
        for (;;) {
            const int room = width - __builtin_popcountll(S);
            if (room <= 0 || left_ == 0) return S;
            tried_.clear();
            for (int q = 0; q < n_; ++q) {
                const uint32_t c = at_.cur[q];
                if (c >= start_[q].size()) continue;
                const uint32_t end = c + 1 < start_[q].size() ? start_[q][c + 1] : (uint32_t)item_[q].size();
                for (uint32_t i = start_[q][c]; i < end; ++i) {
                    const uint32_t g = item_[q][i];
                    const uint64_t more = use_[g].need & ~S;
                    if (stamp_[g] == kDone || !more || !allowed(g) || !ready(g)) continue;
                    if (__builtin_popcountll(more) > room) continue;
                    auto it = std::find_if(tried_.begin(), tried_.end(), [&](const Option& o) { return o.more == more; });
                    if (it == tried_.end()) tried_.push_back(Option{more, g});
                    else it->gate = std::min(it->gate, g);
                }
            }
            if (tried_.empty()) return S;
            std::sort(tried_.begin(), tried_.end(), [](const Option& a, const Option& b) { return a.gate < b.gate; });
            if ((int)tried_.size() > most) tried_.resize(most);
            uint64_t best = tried_[0].more;
            double best_gain = -1.0;
            if (tried_.size() > 1)
                for (const Option& o : tried_) {
                    const double gain = (double)gain_of(S | o.more, o.gate) / __builtin_popcountll(o.more);
                    if (gain > best_gain) {
                        best = o.more;
                        best_gain = gain;
                    }
                }
            S |= best;
            take(S, out, kinds);
        }
    }

private:
    static constexpr uint32_t kDone = ~0u;
    struct Use {
        int n = 0;
        uint8_t q[5];
        uint32_t grp[5];
        bool map = false;
        uint64_t need = 0;
    };
    struct At {
        uint32_t cur[64], rem[64];
        void open(const Frontier& f, int q, uint32_t grp)
        {
            cur[q] = grp;
            const auto& st = f.start_[q];
            rem[q] = grp >= st.size() ? 0
                     : (grp + 1 < st.size() ? st[grp + 1] : (uint32_t)f.item_[q].size()) - st[grp];
        }
    };

    struct Undo {
        int q;
        uint32_t cur, rem;
    };

    bool allowed(uint32_t g) const { return kinds_ == kAny || use_[g].map == (kinds_ == kMaps); }

    bool ready(uint32_t g) const
    {
        const Use& u = use_[g];
        for (int j = 0; j < u.n; ++j)
            if (at_.cur[u.q[j]] != u.grp[j]) return false;
        return true;
    }

    void push_group(int q)
    {
        const uint32_t c = at_.cur[q];
        if (c >= start_[q].size()) return;
        const uint32_t end = c + 1 < start_[q].size() ? start_[q][c + 1] : (uint32_t)item_[q].size();
        for (uint32_t i = start_[q][c]; i < end; ++i) queue_.push_back(item_[q][i]);
    }

    // Apply what the queue leads to; returns the number of gates with
    // non-diagonal targets among them.
    int close(uint64_t S, std::vector<int>* out)
    {
        int count = 0;
        for (size_t h = 0; h < queue_.size(); ++h) {
            const uint32_t g = queue_[h];
            const Use& u = use_[g];
            if (stamp_[g] == kDone || stamp_[g] == now_ || (u.need & ~S) || !allowed(g) || !ready(g)) continue;
            stamp_[g] = now_;
            if (out) out->push_back((int)g);
            if (u.need) ++count;
            for (int j = 0; j < u.n; ++j) {
                const int q = u.q[j];
                if (!out) undo_.push_back(Undo{q, at_.cur[q], at_.rem[q]});
                if (--at_.rem[q] == 0) {
                    at_.open(*this, q, at_.cur[q] + 1);
                    push_group(q);
                }
            }
        }
        return count;
    }

    int gain_of(uint64_t S, uint32_t g)
    {
        undo_.clear();
        ++now_;
        queue_.clear();
        const Use& u = use_[g];
        for (int j = 0; j < u.n; ++j) push_group(u.q[j]);
        const int count = close(S, nullptr);
        for (size_t i = undo_.size(); i-- > 0;) {
            at_.cur[undo_[i].q] = undo_[i].cur;
            at_.rem[undo_[i].q] = undo_[i].rem;
        }
        return count;
    }

    int n_;
    int left_ = 0;
    std::vector<Use> use_;
    std::vector<uint32_t> stamp_;
    uint32_t now_ = 0;
    Kinds kinds_ = kAny;
    std::array<std::vector<uint32_t>, 64> item_, start_;
    At at_;
    std::vector<uint32_t> queue_;
    struct Option {
        uint64_t more;
        uint32_t gate;
    };
    std::vector<Option> tried_;
    std::vector<Undo> undo_;
};

int tile_bits(int n) { return std::min(n, kTileMaxBits); }

}  // namespace

bool tile_applies(int n) { return n >= kTileRegBits; }

namespace {

// A matrix rounded to FP32 scales every state by 1 + some 1e-8, a list of
// gates by the sum of these: 1e-6 after hundreds of rotations, four times that
// in the derivatives of a backward. So each matrix that is not exact is scaled
// first by what the gates before it left over (`drift`, a logarithm of the norm),
// which keeps the sum within one rounding. Only matrices that every amplitude
// takes part in (no controls) are counted and scaled; a gate that runs in a
// sweep of its own takes its scaled matrix along (tile_matrix).
void keep_norm(cd* m, int count, double& drift)
{
    double want = 0.0, got = 0.0;
    bool exact = true;
    const double f = 1.0 - drift;
    for (int i = 0; i < count; ++i) {
        exact = exact && (double)(float)m[i].real() == m[i].real() && (double)(float)m[i].imag() == m[i].imag();
        want += std::norm(m[i]);
        const double re = (float)(f * m[i].real()), im = (float)(f * m[i].imag());
        got += re * re + im * im;
    }
    if (exact) return;
    const double left = drift + 0.5 * std::log(got / want);          // `got` holds the factor f
    if (!(std::abs(left) < 1e-6)) return;              // not finite, or not a rounding
    for (int i = 0; i < count; ++i) m[i] *= f;
    drift = left;
}

}  // namespace

void tile_append(TileList& l, int k, const int* targets, int nc, const int* controls, const cd* ms, int nm, int op,
                 int deriv)
{
    const int D = 1 << k;
    bool diag = true, ident = true, ones = true, sign = true, exch = true, real = true, imoff = true;
    for (int r = 0; r < nm; ++r) {
        const cd* m = ms + (size_t)r * D * D;
        for (int i = 0; i < D; ++i)
            for (int j = 0; j < D; ++j) {
                const cd v = m[i * D + j];
                const bool last = i == D - 1 && j == D - 1;
                if (i != j && v != cd(0.0)) diag = false;
                if (v != cd(i == j ? 1.0 : 0.0)) ident = false;
                if (i == j && !last && v != cd(1.0)) ones = false;
                if (last && v != cd(-1.0)) sign = false;
                const int swapped = k == 1 ? 1 - i : (i == 1 ? 2 : i == 2 ? 1 : i);
                if (v != cd(j == swapped ? 1.0 : 0.0)) exch = false;
                if (v.imag() != 0.0) real = false;
                if (i == j ? v.imag() != 0.0 : v.real() != 0.0) imoff = false;
            }
    }
    if (ident && !deriv) return;
    // the generator decides what a gate with a derivative commutes with, also
    // where its matrix is the identity
    if (deriv && deriv != TD_Z) diag = false;
    TileGate g{};
    g.deriv = deriv;
    g.k = k;
    for (int j = 0; j < k; ++j) g.targets[j] = targets[j];
    g.nc = nc;
    for (int j = 0; j < nc; ++j) g.controls[j] = controls[j];
    g.op = op;
    g.mat = l.pool.size();
    g.per_row = nm > 1;
    if (diag && ones && !deriv) {
        for (int j = 0; j < k; ++j) g.controls[g.nc++] = targets[j];
        g.k = 0;
        g.kind = sign ? TK_SIGN : TK_ONES;
    } else if (diag && !(deriv && nc > 0)) {
        g.kind = k == 1 ? TK_DIAG1 : TK_DIAG2;
    } else if (exch && nc <= 2 - k && !deriv) {
        g.kind = TK_MAP;
    } else if (k == 2) {
        g.kind = TK_DENSE2;
    } else {
        g.kind = nc > 0 ? TK_DENSE : real ? TK_REAL : imoff ? TK_IMOFF : TK_DENSE;
    }
    if (kMatFloats[g.kind] == 0) g.per_row = false;
    if (g.per_row) l.row_drift.resize(std::max<size_t>(l.row_drift.size(), nm), 0.0);
    for (int r = 0; r < (g.per_row ? nm : 1); ++r) {
        cd m[16];
        std::copy(ms + (size_t)r * D * D, ms + (size_t)(r + 1) * D * D, m);
        // uncontrolled: every amplitude takes part
        if (nc == 0 && g.k > 0) keep_norm(m, D * D, g.per_row ? l.row_drift[r] : l.drift);
        auto put = [&](cd v) {
            l.pool.push_back((float)v.real());
            l.pool.push_back((float)v.imag());
        };
        switch (g.kind) {
        case TK_REAL:
            for (int i = 0; i < 4; ++i) l.pool.push_back((float)m[i].real());
            break;
        case TK_IMOFF:
            for (int i = 0; i < 4; ++i) l.pool.push_back((float)(i == 0 || i == 3 ? m[i].real() : m[i].imag()));
            break;
        case TK_DIAG1: case TK_DIAG2:
            for (int i = 0; i < D; ++i) put(m[i * D + i]);
            break;
        case TK_ONES:
            put(m[D * D - 1]);
            put(0.0);
            break;
        case TK_DENSE: case TK_DENSE2:
            for (int i = 0; i < D * D; ++i) put(m[i]);
            break;
        default: break;
        }
    }
    l.gates.push_back(g);
}

void tile_matrix(const TileList& l, const TileGate& g, int r, cd* m)
{
    const int D = 1 << g.k;
    const float* w = l.pool.data() + g.mat + (g.per_row ? (size_t)r * kMatFloats[g.kind] : 0);
    std::fill(m, m + D * D, cd(0.0));
    switch (g.kind) {
    case TK_DENSE: case TK_DENSE2:
        for (int i = 0; i < D * D; ++i) m[i] = cd(w[2 * i], w[2 * i + 1]);
        break;
    case TK_REAL:
        for (int i = 0; i < 4; ++i) m[i] = w[i];
        break;
    case TK_IMOFF:
        for (int i = 0; i < 4; ++i) m[i] = i == 0 || i == 3 ? cd(w[i]) : cd(0.0, w[i]);
        break;
    case TK_DIAG1: case TK_DIAG2:
        for (int i = 0; i < D; ++i) m[i * D + i] = cd(w[2 * i], w[2 * i + 1]);
        break;
    case TK_ONES: m[0] = cd(w[0], w[1]); break;
    case TK_SIGN: m[0] = -1.0; break;
    case TK_MAP:                      // X, or SWAP
        if (g.k == 1) m[1] = m[2] = 1.0;
        else m[0] = m[6] = m[9] = m[15] = 1.0;
        break;
    default: break;
    }
}

// ------------------------------------------------------------ sweeps

// In us of this card, both sides measured as lists of two and three gates. A
// launch of its own takes 2.7 and its part of the state at 7.0 TB/s, no less than
// 3.3 (a U3 on 20 / 23 / 26 qubits: 6.4, 23, 160); a tile sweep 4 and every
// amplitude at 5.5 TB/s (20 / 23 / 26 qubits: 7, 28, 199), and no less than 6.5,
// from 2^16 amplitudes on 7.5: two gates on 18 qubits take 18.0 by themselves,
// 19.2 in one sweep when waited for (8.0 : 7.3 among others of their kind), on 10
// qubits 16.7 : 17.0 (7.5 : 6.9), on 16 17.4 : 18.9. Gates of several controls cost a program more
// (two X with three: 17.0 : 18.3 on 10 qubits, 18.5 : 29.4 on 22). Two CX on 26
// qubits: 167 : 202, on 22 behind a reset 39 : 44, on 21 10.3 : 9.1. Three gates:
// 19.1 : 17.3, 10.4 : 7.3 on 10 qubits.
bool tile_apart(const TileList& l, const int* gates, int count, int n, int rows)
{
    constexpr int kFullLine = 4;
    const double moved = 16.0 * (double)((uint64_t)rows << n);
    double own = 0.0, tile = std::max(moved < (1 << 20) ? 6.5 : 7.5, 4.0 + moved / 5.5e6);
    for (int i = 0; i < count; ++i) {
        const TileGate& g = l.gates[gates ? gates[i] : i];
        double part = 1.0;
        for (int j = 0; j < g.nc; ++j)
            if (g.controls[j] >= kFullLine) part *= 0.5;       // lower ones leave every line touched
        const int launches = g.per_row ? rows : 1;
        own += std::max(3.3 * launches, 2.7 * launches + part * moved / 7.0e6);
        if (g.nc + g.k > 2) tile += 0.5;
    }
    return own < tile;
}

struct TilePlanner {
    const TileList& l;
    int n, rows;
    std::vector<int> all;
    Frontier front;

    static std::vector<int> iota(size_t m)
    {
        std::vector<int> v(m);
        for (size_t i = 0; i < m; ++i) v[i] = (int)i;
        return v;
    }
    TilePlanner(const TileList& list, int nq, int nr)
        : l(list), n(nq), rows(nr), all(iota(list.gates.size())), front(l, all, nq)
    {
    }

    bool next(TileSweep& s)
    {
        s.gates.clear();
        s.single = false;
        if (front.left() == 0) return false;
        const int T = tile_bits(n);
        uint64_t S = T == n ? (n >= 64 ? ~0ull : (1ull << n) - 1) : (1ull << kRunBits) - 1;
        S = front.grow(S, T, s.gates, Frontier::kAny, 64);
        // unused room: the lowest other qubits (longer runs)
        for (int q = 0; q < n && __builtin_popcountll(S) < T; ++q) S |= 1ull << q;
        s.qubits = S;
        s.single = separate(s);
        return true;
    }

    // Whether the gates of a sweep go faster by sweeps of their own: one gate
    // always, a few that each touch a small part of the state often.
    bool separate(const TileSweep& s) const
    {
        if (s.gates.size() == 1) return true;
        if (s.gates.size() > 16) return false;
        return tile_apart(l, s.gates.data(), (int)s.gates.size(), n, rows);
    }
};

TilePlannerHandle::TilePlannerHandle(const TileList& l, int n, int rows) : p(new TilePlanner(l, n, rows)) {}
TilePlannerHandle::~TilePlannerHandle() { delete p; }
bool TilePlannerHandle::next(TileSweep& s) { return p->next(s); }

// ------------------------------------------------------------ programs

namespace {

uint32_t swizzled(int b) { return (1u << b) ^ (b >= 4 ? kTileSwz[b - 4] : 0u); }

// A sweep's places: tile bit of each qubit, bit of the tile's index for the others.
struct Places {
    int T;
    int tile_bit[64];
    int outer_bit[64];
    uint8_t pos[kTileMaxBits];
    Places(int n, uint64_t S)
    {
        T = 0;
        int o = 0;
        for (int q = 0; q < n; ++q) {
            tile_bit[q] = outer_bit[q] = -1;
            if ((S >> q) & 1) {
                pos[T] = (uint8_t)q;
                tile_bit[q] = T++;
            } else {
                outer_bit[q] = o++;
            }
        }
        for (int b = T; b < kTileMaxBits; ++b) pos[b] = 0;
    }
};

// The words of one round: register bits (tile bits, ascending) and the
// thread bits, the first four chosen so that 16 neighbouring lanes reach 16
// different 8-byte banks.
struct Round {
    int nreg;
    int reg[kTileRegBits];
    uint32_t reg_mask;
    int nthr;
    int thr[kTileMaxBits];
    Round(const Places& pl, uint64_t regs, int R)
    {
        nreg = nthr = 0;
        reg_mask = 0;
        for (int b = 0; b < pl.T; ++b)
            if ((regs >> pl.pos[b]) & 1) reg_mask |= 1u << b;
        // fewer targets than registers: the highest free tile bits (the low
        // ones stay with the lanes)
        for (int b = pl.T - 1; b >= 0 && __builtin_popcount(reg_mask) < R; --b) reg_mask |= 1u << b;
        uint32_t span[4] = {0, 0, 0, 0};
        std::vector<int> late;
        for (int b = 0; b < pl.T; ++b) {
            if ((reg_mask >> b) & 1) {
                reg[nreg++] = b;
                continue;
            }
            uint32_t v = swizzled(b) & 15u;
            for (int i = 3; i >= 0; --i)
                if ((v >> i) & 1) {
                    if (span[i]) v ^= span[i];
                    else break;
                }
            if (v && nthr < 4) {
                span[31 - __builtin_clz(v)] = v;
                thr[nthr++] = b;
            } else {
                late.push_back(b);
            }
        }
        for (int b : late) thr[nthr++] = b;
    }
    void words(int ngates, uint32_t* w) const
    {
        std::memset(w, 0, kTileRoundWords * sizeof(uint32_t));
        w[0] = (uint32_t)ngates;
        for (int k = 0; k < nthr; ++k) {
            w[k < 8 ? 1 + k / 2 : 8] |= swizzled(thr[k]) << (16 * (k & 1));
            w[k < 8 ? 7 : 9] |= (uint32_t)thr[k] << (4 * (k & 7));
        }
        for (int k = 0; k < nreg; ++k) w[5 + k / 2] |= swizzled(reg[k]) << (16 * (k & 1));
    }
    int reg_index(int tile_bit) const { return __builtin_popcount(reg_mask & ((1u << tile_bit) - 1)); }
};

int value_count(const TileGate& g) { return g.deriv == TD_NONE ? 0 : g.deriv == TD_GENERAL ? 8 : 1; }

// Collects rounds until the kernel arguments are full, then launches.
class Emitter {
public:
    // launch(args, rows, derivative gates in the order of their values, last)
    using Launch = std::function<void(const TileArgs&, int, const std::vector<int>&, bool)>;

    Emitter(const Rows& rows, int n, const TileList& l, uint64_t S, int R, Launch launch, int max_values = kAdjValues)
        : rows_(rows), l_(l), pl_(n, S), R_(R), launch_(std::move(launch)), min_rows_(std::min(rows.nrows, kMinRows)),
          max_values_(max_values)
    {
        std::memset(&a_, 0, sizeof(a_));
        a_.p0 = rows.p0;
        a_.p1 = rows.p1;
        a_.N = rows.N;
        a_.nrow0 = rows.nrow0;
        a_.T = pl_.T;
        std::memcpy(a_.pos, pl_.pos, sizeof(a_.pos));
    }

    // A round: gates on the register qubits `regs`, then index maps.
    void round(uint64_t regs, std::vector<int> gates, const std::vector<int>& maps)
    {
        const Round r(pl_, regs, R_);
        by_level(r, gates);
        if (!room(kTileRoundWords + kTileHeadWords + kMatFloats[TK_DENSE2])) flush();
        open(r);
        for (int gi : gates)
            if (!add(gi)) {
                flush();
                open(r);
                add(gi);
            }
        if (maps.empty()) return;
        const Map m = compose(maps);
        const int words = kTileMapWords + (((int)m.outer.size() + 3) & ~3);
        if (!room(words)) {
            flush();
            open(r);
        }
        rounds_.back().map = m;
        rounds_.back().mapped = true;
        prog_ += words;
    }

    void flush(bool last = false)
    {
        if (prog_ == 0 && !last) return;
        int rows_per = std::min(rows_.nrows, kMaxRows);
        if (per_row_) rows_per = std::min(rows_per, (kTileWords - prog_ - shared_) / per_row_);
        for (int r0 = 0; r0 < rows_.nrows; r0 += rows_per) {
            const int nr = std::min(rows_per, rows_.nrows - r0);
            fill(r0, nr);
            a_.row0 = r0;
            launch_(a_, nr, values_, last);
        }
        rounds_.clear();
        prog_ = shared_ = per_row_ = nvalues_ = 0;
    }

private:
    // per-row matrices: a launch takes at least this many rows (of a larger batch)
    static constexpr int kMinRows = 8;
    static constexpr int kMaxRows = 16384;
    // Gates in the order of their depth on the register bits, those of a kind
    // together: gates of one depth act on different bits (or commute), so
    // they share steps.
    void by_level(const Round& r, std::vector<int>& gates)
    {
        int level[kTileRegBits] = {0, 0, 0, 0};
        bool phase[kTileRegBits] = {false, false, false, false};   // the level's gates are diagonal on the bit
        order_.clear();
        for (int gi : gates) {
            const TileGate& g = l_.gates[gi];
            const bool diag = g.kind >= TK_DIAG1 && g.kind <= TK_SIGN;
            int at = 0;
            auto look = [&](int q, bool z) {
                if (!in_registers(r, q)) return;
                const int b = r.reg_index(pl_.tile_bit[q]);
                // gates diagonal on a bit share its level with each other
                at = std::max(at, level[b] + (z && phase[b] ? 0 : 1));
            };
            for (int j = 0; j < g.k; ++j) look(g.targets[j], diag);
            for (int j = 0; j < g.nc; ++j) look(g.controls[j], true);
            auto set = [&](int q, bool z) {
                if (!in_registers(r, q)) return;
                const int b = r.reg_index(pl_.tile_bit[q]);
                phase[b] = z && (phase[b] || at > level[b]);
                level[b] = at;
            };
            for (int j = 0; j < g.k; ++j) set(g.targets[j], diag);
            for (int j = 0; j < g.nc; ++j) set(g.controls[j], true);
            // sign flips with and without a thread control apart
            int lane = 0;
            if (g.kind == TK_SIGN)
                for (int j = 0; j < g.nc; ++j)
                    if (pl_.tile_bit[g.controls[j]] >= 0 && !in_registers(r, g.controls[j])) lane = 1;
            order_.push_back({at * 16 + g.kind + (lane ? 4 : 0), gi});
        }
        std::stable_sort(order_.begin(), order_.end(),
                         [](const std::pair<int, int>& a, const std::pair<int, int>& b) { return a.first < b.first; });
        for (size_t i = 0; i < gates.size(); ++i) gates[i] = order_[i].second;
    }

    // A step: a layer of one kind (gate on each register bit, -1 none) or one
    // other gate.
    struct Step {
        int layer;                    // kind, -1: not a layer
        bool per_row;
        int gate[kTileRegBits];
    };
    // An affine map of the tile's index: new index = XOR of the columns of the
    // old index's set bits, of those of the set outer bits, and a constant.
    struct Map {
        uint32_t col[kTileMaxBits];
        std::vector<std::pair<int, uint32_t>> outer;
        uint32_t constant;
    };
    struct Entry {
        Round r;
        std::vector<int> thread;      // phases without a register bit
        std::vector<Step> steps;
        int last[kTileRegBits];       // last step on each register bit
        bool sign, phase, mapped;
        Map map;
    };

    Map compose(const std::vector<int>& maps) const
    {
        struct Form { uint32_t tile, outer, one; } f[kTileMaxBits];
        for (int t = 0; t < pl_.T; ++t) f[t] = Form{1u << t, 0, 0};
        for (int gi : maps) {
            const TileGate& g = l_.gates[gi];
            Form& t = f[pl_.tile_bit[g.targets[0]]];
            if (g.k == 2) {
                std::swap(t, f[pl_.tile_bit[g.targets[1]]]);
            } else if (g.nc == 0) {
                t.one ^= 1u;
            } else if (pl_.tile_bit[g.controls[0]] >= 0) {
                const Form& c = f[pl_.tile_bit[g.controls[0]]];
                t.tile ^= c.tile;
                t.outer ^= c.outer;
                t.one ^= c.one;
            } else {
                t.outer ^= 1u << pl_.outer_bit[g.controls[0]];
            }
        }
        Map m{};
        uint32_t outer = 0;
        for (int t = 0; t < pl_.T; ++t) {
            for (int i = 0; i < pl_.T; ++i) m.col[i] |= ((f[t].tile >> i) & 1u) << t;
            m.constant |= f[t].one << t;
            outer |= f[t].outer;
        }
        for (; outer; outer &= outer - 1) {
            const int o = __builtin_ctz(outer);
            uint32_t col = 0;
            for (int t = 0; t < pl_.T; ++t) col |= ((f[t].outer >> o) & 1u) << t;
            m.outer.push_back({o, col});
        }
        return m;
    }

    static uint32_t element(uint32_t index)
    {
        uint32_t e = 0;
        for (; index; index &= index - 1) e ^= swizzled(__builtin_ctz(index));
        return e;
    }

    bool room(int more) const { return prog_ + shared_ + per_row_ * min_rows_ + more <= kTileWords; }

    void open(const Round& r)
    {
        rounds_.push_back(Entry{r, {}, {}, {-1, -1, -1, -1}, false, false, false, {}});
        prog_ += kTileRoundWords;
    }

    bool in_registers(const Round& r, int q) const
    {
        return pl_.tile_bit[q] >= 0 && ((r.reg_mask >> pl_.tile_bit[q]) & 1);
    }

    // Uncontrolled one-target gates of one kind on different register bits
    // share a step: the first such layer after everything on the gate's qubit.
    bool add(int gi)
    {
        const TileGate& g = l_.gates[gi];
        Entry& e = rounds_.back();
        const int mw = kMatFloats[g.kind];
        const int words = g.per_row ? mw * min_rows_ : mw;
        const int values = value_count(g);
        if (nvalues_ + values > max_values_) return false;
        if (g.kind <= TK_DIAG1 && g.nc == 0 && in_registers(e.r, g.targets[0])) {
            const int b = e.r.reg_index(pl_.tile_bit[g.targets[0]]);
            int at = e.last[b] + 1;
            while (at < (int)e.steps.size() && !(e.steps[at].layer == g.kind && e.steps[at].per_row == g.per_row)) ++at;
            const bool fresh = at == (int)e.steps.size();
            if (!room(words + (fresh ? kTileHeadWords : 0))) return false;
            if (fresh) {
                e.steps.push_back(Step{g.kind, g.per_row, {-1, -1, -1, -1}});
                prog_ += kTileHeadWords;
            }
            e.steps[at].gate[b] = gi;
            e.last[b] = at;
        } else {
            if (!room(words + kTileHeadWords)) return false;
            bool any = false;
            auto touch = [&](int q) {
                if (!in_registers(e.r, q)) return;
                any = true;
                e.last[e.r.reg_index(pl_.tile_bit[q])] = (int)e.steps.size();
            };
            for (int j = 0; j < g.k; ++j) touch(g.targets[j]);
            for (int j = 0; j < g.nc; ++j) touch(g.controls[j]);
            if (any) {
                e.steps.push_back(Step{-1, g.per_row, {gi, -1, -1, -1}});
            } else {
                (g.kind == TK_SIGN ? e.sign : e.phase) = true;
                e.thread.push_back(gi);
            }
            prog_ += kTileHeadWords;
        }
        (g.per_row ? per_row_ : shared_) += mw;
        nvalues_ += values;
        return true;
    }

    void fill(int r0, int nr)
    {
        int pc = 0, mat = prog_;
        a_.nrounds = (int)rounds_.size();
        values_.clear();
        for (const Entry& e : rounds_) {
            uint32_t* rw = a_.words + pc;
            e.r.words((int)e.steps.size(), rw);
            rw[0] |= (uint32_t)e.thread.size() << 24 | (uint32_t)e.sign << 16 | (uint32_t)e.phase << 17 | (uint32_t)e.mapped << 18;
            pc += kTileRoundWords;
            if (e.mapped) {
                const int no = (int)e.map.outer.size();
                rw[0] |= (uint32_t)no << 8;
                std::memset(rw + 12, 0, (kTileMapWords + ((no + 3) & ~3)) * sizeof(uint32_t));
                for (int k = 0; k < e.r.nthr; ++k) rw[12 + k / 2] |= element(e.map.col[e.r.thr[k]]) << (16 * (k & 1));
                for (int k = 0; k < e.r.nreg; ++k) rw[17 + k / 2] |= element(e.map.col[e.r.reg[k]]) << (16 * (k & 1));
                rw[19] = element(e.map.constant);
                for (int i = 0; i < no; ++i)
                    rw[20 + i] = (uint32_t)e.map.outer[i].first | element(e.map.outer[i].second) << 16;
                pc += kTileMapWords + ((no + 3) & ~3);
            }
            for (int gi : e.thread) {
                const TileGate& g = l_.gates[gi];
                uint32_t* h = a_.words + pc;
                pc += kTileHeadWords;
                header(e.r, g, h);
                h[2] = (uint32_t)mat | (g.per_row ? (uint32_t)kMatFloats[g.kind] << 16 : 0u);
                for (int r = 0; r < (g.per_row ? nr : 1); ++r) mat += matrix(g, r0 + r, a_.words + mat);
            }
            uint32_t* sign = nullptr;
            for (const Step& s : e.steps) {
                uint32_t* h = a_.words + pc;
                pc += kTileHeadWords;
                const int nm = s.per_row ? nr : 1;
                int stride = 0;
                if (s.layer >= 0) {
                    if (sign) sign[0] |= TF_APPLY;
                    sign = nullptr;
                    h[0] = TF_LAYER | (uint32_t)(TF_DENSE << s.layer);
                    h[1] = 0;
                    for (int b = 0; b < R_; ++b)
                        if (s.gate[b] >= 0) {
                            const TileGate& g = l_.gates[s.gate[b]];
                            h[0] |= 1u << (8 + b);
                            h[1] |= (uint32_t)((mat + stride) / 4) << (8 * b);
                            stride += kMatFloats[g.kind];
                        }
                    h[2] = s.per_row ? (uint32_t)stride : 0u;
                    h[3] = 0;
                    for (int b = 0; b < R_; ++b)
                        if (s.gate[b] >= 0 && l_.gates[s.gate[b]].deriv) derivative(s.gate[b], b, h);
                } else {
                    const TileGate& g = l_.gates[s.gate[0]];
                    stride = kMatFloats[g.kind];
                    header(e.r, g, h);
                    if (g.deriv) derivative(s.gate[0], __builtin_ctz(h[3]), h);
                    // the last of consecutive sign flips applies them
                    if (sign && !(h[0] & TF_SIGN)) sign[0] |= TF_APPLY;
                    sign = h[0] & TF_SIGN ? h : nullptr;
                    h[2] = (uint32_t)mat | (s.per_row ? (uint32_t)stride << 16 : 0u);
                }
                for (int r = 0; r < nm; ++r)
                    for (int b = 0; b < R_; ++b)
                        if (s.gate[b] >= 0) mat += matrix(l_.gates[s.gate[b]], r0 + r, a_.words + mat);
            }
            if (sign) sign[0] |= TF_APPLY;
        }
        a_.nwords = mat;
    }

    void derivative(int gi, int bit, uint32_t* h)
    {
        h[0] |= TF_DERIV;
        h[3] |= (uint32_t)l_.gates[gi].deriv << (8 + 4 * bit);
        values_.push_back(gi);
    }

    void header(const Round& rd, const TileGate& g, uint32_t* h) const
    {
        uint32_t rb = 0, rcm = 0, tctl = 0, octl = 0, places = 0, ats = 0;
        for (int j = 0; j < g.nc; ++j) {
            const int b = pl_.tile_bit[g.controls[j]];
            if (b < 0) octl |= 1u << pl_.outer_bit[g.controls[j]];
            else if (in_registers(rd, g.controls[j])) rcm |= 1u << rd.reg_index(b);
            else tctl |= 1u << b;
        }
        for (int j = 0; j < g.k; ++j) {
            const int b = pl_.tile_bit[g.targets[j]];
            const bool reg = in_registers(rd, g.targets[j]);
            const int at = reg ? rd.reg_index(b) : b >= 0 ? b : pl_.outer_bit[g.targets[j]];
            if (reg) rb |= 1u << at;
            places |= (uint32_t)(reg ? kPlaceReg : b >= 0 ? kPlaceThread : kPlaceOuter) << (2 * j);
            ats |= (uint32_t)at << (8 * j);
        }
        // place of a pair of register bits
        static constexpr int kPair[] = {0, 0, 0, 0, 0, 1, 2, 0, 0, 3, 4, 0, 5};
        uint32_t flag = 0;
        h[3] = rb;
        switch (g.kind) {
        case TK_SIGN:
            flag = tctl && rcm ? TF_LANE_SIGN : TF_SIGN;
            h[3] = 0;
            for (uint32_t j = 0; j < (1u << R_); ++j) h[3] |= (uint32_t)((j & rcm) == rcm) << j;
            break;
        case TK_DIAG1: case TK_DIAG2: case TK_ONES:
            flag = TF_PHASE;
            h[3] = ats | (uint32_t)g.k << 16 | places << 20;
            break;
        case TK_DENSE2:
            flag = TF_DENSE2;
            h[3] = 1u << kPair[rb];
            break;
        default: flag = TF_CTRL; break;
        }
        h[0] = TF_OTHER | flag | rcm << 8 | tctl << 16;
        h[1] = octl;
    }

    // Row r's matrix of g; returns its words. A 4 x 4 is written with the
    // higher tile bit as its index's most significant bit.
    int matrix(const TileGate& g, int r, uint32_t* dst) const
    {
        const int mw = kMatFloats[g.kind];
        const float* src = l_.pool.data() + g.mat + (g.per_row ? (size_t)r * mw : 0);
        if (g.kind != TK_DENSE2 || pl_.tile_bit[g.targets[0]] > pl_.tile_bit[g.targets[1]]) {
            std::memcpy(dst, src, mw * sizeof(float));
            return mw;
        }
        constexpr int sw[4] = {0, 2, 1, 3};
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j)
                std::memcpy(dst + 2 * (4 * i + j), src + 2 * (4 * sw[i] + sw[j]), 2 * sizeof(float));
        return mw;
    }

    Rows rows_;
    const TileList& l_;
    Places pl_;
    int R_;
    Launch launch_;
    int min_rows_, max_values_;
    TileArgs a_;
    std::vector<Entry> rounds_;
    std::vector<std::pair<int, int>> order_;
    std::vector<int> values_;         // gates with derivatives, in the order of their values
    int prog_ = 0, shared_ = 0, per_row_ = 0, nvalues_ = 0;
};

// The gates (positions in the list) of a sweep over the qubits S as rounds.
void emit_rounds(Emitter& em, int n, const TileList& l, const std::vector<int>& gates, uint64_t S, int R)
{
    Frontier f(l, gates, n);
    std::vector<int> at, maps, carry, now, later;
    while (f.left() > 0) {
        at.clear();
        const uint64_t regs = f.grow(0, R, at, Frontier::kNoMaps, kRoundOptions);
        const size_t local = at.size();
        f.take(S, at, Frontier::kMaps);
        maps.clear();
        uint64_t changed = 0;         // qubits that a later gate changes
        for (size_t i = local; i < at.size(); ++i) {
            maps.push_back(gates[at[i]]);
            for (int j = 0; j < l.gates[maps.back()].k; ++j) changed |= 1ull << l.gates[maps.back()].targets[j];
        }
        now = carry;
        for (size_t i = 0; i < local; ++i) now.push_back(gates[at[i]]);
        // A phase on register qubits that nothing behind it in the round waits
        // for is left to the next round, where its qubits are the threads' and
        // it costs one operation instead of one per amplitude.
        carry.clear();
        if (f.left() > 0) {
            later.clear();
            for (size_t i = now.size(); i-- > 0;) {
                const TileGate& g = l.gates[now[i]];
                uint64_t qs = 0;
                for (int j = 0; j < g.k; ++j) qs |= 1ull << g.targets[j];
                if (g.kind < TK_DIAG1 || g.kind > TK_SIGN || g.deriv) {
                    changed |= qs;
                    continue;
                }
                for (int j = 0; j < g.nc; ++j) qs |= 1ull << g.controls[j];
                if ((qs & regs) && !(qs & changed)) {
                    later.push_back(now[i]);
                    now[i] = -1;
                }
            }
            now.erase(std::remove(now.begin(), now.end(), -1), now.end());
            carry.assign(later.rbegin(), later.rend());
        }
        em.round(regs, now, maps);
    }
}

}  // namespace

int tile_sweep(const Rows& rows, int n, const TileList& l, const TileSweep& s, hipStream_t st)
{
    // Few workgroups: half as many amplitudes per thread, so that a compute unit
    // holds twice the waves of its one or two tiles (20-qubit brickwork,
    // one tile per unit: 24.8 us a sweep instead of 26.4; 27 qubits: 1043
    // instead of 904, from the rounds over three bits instead of four).
    const uint64_t groups = (1ull << (n - tile_bits(n))) * rows.nrows;
    const int R = groups <= 2 * (uint64_t)device_info().cu_count ? kTileRegBits - 1 : kTileRegBits;
    int launches = 0;
    Emitter em(rows, n, l, s.qubits, R,
               [&](const TileArgs& a, int nr, const std::vector<int>&, bool) {
                   launch_tile(a, nr, R, st);
                   launches += a.row0 == 0;
               });
    emit_rounds(em, n, l, s.gates, s.qubits, R);
    em.flush();
    return launches;
}

bool tile_adjoint_applies(int n) { return n >= kTileRegBits; }

int tile_values(const TileList& l)
{
    int v = 0;
    for (const TileGate& g : l.gates) v += value_count(g);
    return v;
}

void tile_adjoint(float2* psi, float2* lam, int n, int rows, const TileList& l, const double* coeff, int coeff_stride,
                  double* out, std::vector<int>& order, hipStream_t st)
{
    constexpr int R = kTileRegBits - 1;
    TileAdjArgs a{};
    a.psi = psi;
    a.lam = lam;
    a.coeff = coeff;
    a.coeff_stride = coeff_stride;
    a.out = out;
    a.out_stride = tile_values(l) + 2;
    a.N = 1ull << n;
    a.T = n;
    a.first = 1;
    order.clear();
    const Rows rr{psi, psi, rows, rows, 1ull << n};
    const uint64_t S = (1ull << n) - 1;
    Emitter em(rr, n, l, S, R, [&](const TileArgs& t, int nr, const std::vector<int>& gates, bool last) {
        a.row0 = t.row0;
        a.nrounds = t.nrounds;
        a.nwords = t.nwords;
        a.nvalues = 0;
        for (int gi : gates) a.nvalues += value_count(l.gates[gi]);
        a.last = last;
        std::memcpy(a.words, t.words, sizeof(a.words));
        launch_tile_adj(a, 1, nr, st);
        if (t.row0 + nr < rows) return;
        order.insert(order.end(), gates.begin(), gates.end());
        a.value0 += a.nvalues;
        a.first = 0;
        a.coeff = nullptr;            // lambda lies in memory from here on
    });
    std::vector<int> all(l.gates.size());
    for (size_t i = 0; i < all.size(); ++i) all[i] = (int)i;
    emit_rounds(em, n, l, all, S, R);
    em.flush(true);
}

namespace {

// Workgroups per row of a sweep: two per compute unit over all rows (their
// LDS), each taking several tiles, so that values are summed over few parts.
int adjoint_grid(uint64_t tiles, int rows)
{
    const uint64_t most = 2 * (uint64_t)device_info().cu_count;
    while (tiles > 1 && tiles * rows > most) tiles /= 2;
    return (int)tiles;
}

}  // namespace

uint64_t tile_adjoint_parts(int rows)
{
    return (uint64_t)kAdjTileValues * std::max<uint64_t>(2 * (uint64_t)device_info().cu_count, rows);
}

void tile_adjoint_sweep(float2* psi, float2* lam, int n, int rows, const TileList& l, const TileSweep& s, double* part,
                        double* out, std::vector<TileValues>& values, hipStream_t st)
{
    constexpr int R = kTileRegBits - 1;
    TileAdjArgs a{};
    a.psi = psi;
    a.lam = lam;
    a.out = part;
    a.N = 1ull << n;
    const Rows rr{psi, psi, rows, rows, a.N};
    Emitter em(
        rr, n, l, s.qubits, R,
        [&](const TileArgs& t, int nr, const std::vector<int>& gates, bool) {
            a.T = t.T;
            a.row0 = t.row0;
            a.nrounds = t.nrounds;
            a.nwords = t.nwords;
            a.nvalues = 0;
            for (int gi : gates) a.nvalues += value_count(l.gates[gi]);
            std::memcpy(a.pos, t.pos, sizeof(a.pos));
            std::memcpy(a.words, t.words, sizeof(a.words));
            const int grid = adjoint_grid(a.N >> a.T, nr);
            launch_tile_adj(a, grid, nr, st);
            if (a.nvalues == 0) return;
            const uint64_t at = values.empty() ? 0 : values.back().at + (uint64_t)values.back().rows * values.back().nvalues;
            launch_sum_slots(part, grid, nr * a.nvalues, out + at, st);
            values.push_back(TileValues{t.row0, nr, a.nvalues, at, gates});
        },
        kAdjTileValues);
    emit_rounds(em, n, l, s.gates, s.qubits, R);
    em.flush();
}

// ------------------------------------------------------------ Pauli strings

bool pauli_tile_applies(int n) { return n >= 4; }

void plan_pauli_tiles(int n, int rows, const uint64_t* x, const uint64_t* z, int count, std::vector<PauliSweep>& sweeps,
                      std::vector<int>& rest)
{
    // runs of 2^4 amplitudes (whole 128-byte lines) leave the tile eight
    // qubits of the strings' choice
    constexpr uint64_t kRun = 15;
    const int T = tile_bits(n);
    std::vector<int> left;
    left.reserve(count);
    rest.clear();
    for (int i = 0; i < count; ++i) (__builtin_popcountll(x[i] | kRun) > std::max(T, 4) ? rest : left).push_back(i);
    auto imag = [&](int i) { return __builtin_popcountll(x[i] & z[i]) & 1; };
    std::stable_sort(left.begin(), left.end(), [&](int a, int b) {
        return x[a] != x[b] ? x[a] < x[b] : imag(a) < imag(b);
    });
    while (!left.empty()) {
        uint64_t S = T == n ? (1ull << n) - 1 : kRun;
        for (int i : left)
            if (__builtin_popcountll(S | x[i]) <= T) S |= x[i];
        for (int q = 0; q < n && __builtin_popcountll(S) < T; ++q) S |= 1ull << q;
        const Places pl(n, S);
        std::vector<int> take, keep;
        for (int i : left) ((x[i] & ~S) || (int)take.size() == kPauliTerms ? keep : take).push_back(i);
        left.swap(keep);
        // One sweep by x (at most 8 strings) does as well for one string, and
        // for one x below 20 qubits, where the launch is all: 19.6 us against
        // 20.2 at 8 qubits for a string, 21.5 against 23.3 for 8; at 20 qubits
        // 8 strings take 32.2 and 24.9, at 28 qubits 754 and 438. Nor do a few
        // strings pay for a workgroup and its tile on each of thousands of small
        // rows: a row costs the tile 2.4 ns more than it costs a sweep by x, and
        // each of these 5 us and 0.3 ns a row; both read the rows, once or each
        // time (60000 rows of 6 qubits, 2 / 3 / 8 strings of as many x: 276 /
        // 389 / 1006 us by x, 367 / 480 / 996 in one tile sweep; 8000 rows 66 /
        // 87 / 216 and 74 / 92 / 162).
        int by_x = 0;                 // sweeps by x
        for (size_t k = 0, same = 0; k < take.size(); ++k) {
            same = k && x[take[k]] == x[take[k - 1]] ? same + 1 : 0;
            by_x += same % 8 == 0;
        }
        const double read = 8.0 * (double)(1ull << n) / 8.0e6;       // us a row
        if (take.size() == 1 || (n < 20 && take.size() <= 8 && by_x == 1) ||
            (take.size() <= 8 && by_x > 1 && 5.0 + rows * (2.4e-3 + read) > by_x * (5.0 + rows * (0.3e-3 + read)))) {
            rest.insert(rest.end(), take.begin(), take.end());
            continue;
        }
        sweeps.emplace_back();
        PauliSweep& s = sweeps.back();
        std::memset(&s.args, 0, sizeof(s.args));
        s.args.T = T;
        s.args.N = 1ull << n;
        std::memcpy(s.args.pos, pl.pos, sizeof(s.args.pos));
        s.args.nterms = (int)take.size();
        auto tile_bits_of = [&](uint64_t m) {
            uint32_t b = 0;
            for (uint64_t r = m & S; r; r &= r - 1) b |= 1u << pl.tile_bit[__builtin_ctzll(r)];
            return b;
        };
        uint32_t* w = s.args.words;
        uint32_t* head = nullptr;
        for (size_t k = 0; k < take.size(); ++k) {
            const int i = take[k];
            if (k == 0 || x[i] != x[take[k - 1]] || imag(i) != imag(take[k - 1])) {
                head = w++;
                *head = tile_bits_of(x[i]) | (uint32_t)imag(i) << 12;
                ++s.args.ngroups;
            }
            *head += 1u << 16;
            // the amplitudes of a thread differ in the tile's top bits; with
            // x, those without its top bit
            const uint32_t xt = tile_bits_of(x[i]);
            uint32_t zt = tile_bits_of(z[i]), outer = 0, flips = 0;
            if (xt) {
                const uint32_t below = (1u << (31 - __builtin_clz(xt))) - 1;
                zt = (zt & below) | ((zt >> 1) & ~below);
            }
            for (uint64_t r = z[i] & ~S; r; r &= r - 1) outer |= 1u << pl.outer_bit[__builtin_ctzll(r)];
            for (uint32_t j = 0; j < 16; ++j) flips |= (uint32_t)(__builtin_popcount(j & (zt >> (T - 4))) & 1) << j;
            // Re[i^y c]: Re c, -Im c, -Re c, Im c
            const int y = __builtin_popcountll(x[i] & z[i]) & 3;
            w[0] = flips | (zt & ((1u << (T - 4)) - 1)) << 16 | (uint32_t)(y == 1 || y == 2) << 29;
            w[1] = outer;
            w += 2;
        }
        s.terms = take;
    }
}

}  // namespace sv
