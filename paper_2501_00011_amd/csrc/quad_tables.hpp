// Tables of the four-cells-per-wavefront solver: a cell is a row of 16 lanes,
// so every operation list is cut into rounds of 16 (one operation per lane)
// whose structure -- how many terms, what becomes of the sum -- is the same on
// every lane.  Nothing of that structure is then read, tested or selected per
// lane, as it is in the op streams of the one-cell-per-wavefront solver.
// (Part of the mechanism compiler: included by mech_compile.cpp alone.)
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <numeric>

#include "mcc_internal.hpp"

namespace mcc {
namespace {

// Tables of records are stored record by record as 16-byte vectors, [vector]
// [lane], so that the lanes of a row read consecutive bytes.
template <class T>
std::vector<uint32_t> by_vector(const std::vector<T> &recs)
{
    constexpr size_t nv = sizeof(T) / 16;
    std::vector<uint32_t> out(recs.size() * nv * 4);
    for (size_t r = 0; r < recs.size() / kQLanes; ++r)
        for (size_t i = 0; i < kQLanes; ++i)
            for (size_t v = 0; v < nv; ++v)
                std::memcpy(&out[((r * nv + v) * kQLanes + i) * 4],
                            reinterpret_cast<const char *>(&recs[r * kQLanes + i]) + 16 * v, 16);
    return out;
}

struct Term {
    double coef;
    int src;
};

std::map<int, double> net(const mcc_mech_desc *d, int j)
{
    std::map<int, double> nu;
    for (int q = d->reac_ptr[j]; q < d->reac_ptr[j + 1]; ++q) nu[d->reac_idx[q]] -= 1.0;
    for (int q = d->prod_ptr[j]; q < d->prod_ptr[j + 1]; ++q) nu[d->prod_idx[q]] += d->prod_yield[q];
    return nu;
}

// Newton-matrix records of a set of entries (dst -> terms, diagonal?): sorted
// by length so that the 16 lanes of a round have chains of about one length.
struct NmEntry {
    int dst;
    bool diag;
    std::vector<Term> terms;
};

void emit_nm(std::vector<NmEntry> es, std::vector<QNmRec> *recs, int *n_recs, int *first_two, int *first_one)
{
    QNmRec none{};
    for (int q = 0; q < 4; ++q) none.src[q] = kQZero, none.dst[q] = kQTrash;
    int n = 0;
    auto add = [&](const std::vector<QNmRec> &lanes) {
        recs->insert(recs->end(), lanes.begin(), lanes.end());
        ++n;
    };
    std::vector<NmEntry> one, two, more[2];
    for (auto &e : es) {
        if (!e.diag && e.terms.size() == 1) one.push_back(e);
        else if (!e.diag && e.terms.size() == 2) two.push_back(e);
        else more[e.diag].push_back(e);
    }
    for (int diag = 0; diag < 2; ++diag) {  // the long chains first
        auto &v = more[diag];
        std::stable_sort(v.begin(), v.end(), [](const NmEntry &a, const NmEntry &b) { return a.terms.size() > b.terms.size(); });
        for (size_t r = 0; r < v.size(); r += kQLanes) {
            const size_t len = std::max<size_t>(1, (v[r].terms.size() + 3) / 4);
            for (size_t b = 0; b < len; ++b) {
                std::vector<QNmRec> lanes(kQLanes, none);
                for (int i = 0; i < kQLanes && r + i < v.size(); ++i) {
                    const NmEntry &e = v[r + i];
                    for (size_t q = 0; q < 4 && 4 * b + q < e.terms.size(); ++q) {
                        lanes[i].coef[q] = e.terms[4 * b + q].coef;
                        lanes[i].src[q] = (uint16_t)e.terms[4 * b + q].src;
                    }
                    lanes[i].dst[0] = (uint16_t)e.dst;
                }
                for (QNmRec &l : lanes) l.dst[3] = b + 1 < len ? kQNmMore : (diag ? kQNmDiag : kQNmLast);
                add(lanes);
            }
        }
    }
    auto fours = [&]() {
        while (n % 4) add(std::vector<QNmRec>(kQLanes, none));
    };
    while (n % 4) {
        std::vector<QNmRec> pad(kQLanes, none);
        for (QNmRec &l : pad) l.dst[3] = kQNmLast;
        add(pad);
    }
    *first_two = n;
    for (size_t r = 0; r < two.size(); r += 2 * kQLanes) {
        std::vector<QNmRec> lanes(kQLanes, none);
        for (size_t q = r; q < std::min(two.size(), r + 2 * kQLanes); ++q) {
            QNmRec &l = lanes[(q - r) % kQLanes];
            const int h = (int)((q - r) / kQLanes);
            for (int x = 0; x < 2; ++x) {
                l.coef[2 * h + x] = two[q].terms[x].coef;
                l.src[2 * h + x] = (uint16_t)two[q].terms[x].src;
            }
            l.dst[h] = (uint16_t)two[q].dst;
        }
        add(lanes);
    }
    fours();
    *first_one = n;
    for (size_t r = 0; r < one.size(); r += 4 * kQLanes) {
        std::vector<QNmRec> lanes(kQLanes, none);
        for (size_t q = r; q < std::min(one.size(), r + 4 * kQLanes); ++q) {
            QNmRec &l = lanes[(q - r) % kQLanes];
            const int h = (int)((q - r) / kQLanes);
            l.coef[h] = one[q].terms[0].coef;
            l.src[h] = (uint16_t)one[q].terms[0].src;
            l.dst[h] = (uint16_t)one[q].dst;
        }
        add(lanes);
    }
    fours();
    *n_recs = n;
    for (int a = 0; a < kQAhead; ++a) add(std::vector<QNmRec>(kQLanes, none));
}

}  // namespace

void build_quad(const mcc_mech_desc *d, HostTables *t)
{
    QuadTables &q = t->quad;
    q = QuadTables{};
    const int N = t->N, R = t->R, L = kQLanes;
    // Shapes: everything dense in registers (no tail chosen, at most 32
    // species), or a 32-row tail in registers behind a sparse front of at
    // most 64 positions.
    if (t->transposed || R == 0) return;
    if (t->M == 0 && N <= 32 && R <= 8 * L) {
        q.F = 0;
        q.TB = N <= 16 ? 1 : 2;
        q.NC = N <= 16 ? 16 : N <= 24 ? 24 : 32;
    } else if (t->M == 32 && N > 32 && N - 32 <= 64 && R <= 16 * L) {
        q.F = N - 32;
        q.TB = 2;
        q.NC = 32;
    } else {
        return;
    }
    const int F = q.F;
    q.Mt = N - F;
    q.FB = (F + L - 1) / L;
    q.NB = q.TB + q.FB;
    auto block_of = [&](int p) { return p >= F ? q.FB + (p - F) / L : p / L; };
    auto lane_of = [&](int p) { return p >= F ? (p - F) % L : p % L; };
    q.vsp.assign((size_t)q.NB * L, -1);
    for (int p = 0; p < N; ++p) q.vsp[(size_t)block_of(p) * L + lane_of(p)] = t->perm[p];

    // ---- partials and Jacobian terms per entry (positions) ------------------
    struct Part { int j, slot, s; };
    std::vector<Part> parts;
    for (int j = 0; j < R; ++j)
        for (int l = d->reac_ptr[j]; l < d->reac_ptr[j + 1]; ++l) parts.push_back({j, l - d->reac_ptr[j], d->reac_idx[l]});
    const int P = (int)parts.size();
    std::map<std::pair<int, int>, std::vector<Term>> jac;  // (row, column) -> terms (src = partial)
    for (int p = 0; p < N; ++p) jac[{p, p}];
    for (int a = 0; a < P; ++a)
        for (const auto &kv : net(d, parts[a].j))
            if (kv.second != 0.0) jac[{t->iperm[kv.first], t->iperm[parts[a].s]}].push_back({kv.second, a});

    // The factors' entries: those with a term, and what the elimination fills.
    // (Not the pattern of the Jacobian, which counts every participant of a
    // reaction: a species that it needs and gives back, or a product of yield
    // zero, has no term there, and an entry that is neither assembled nor
    // updated would be read without a value.)
    std::vector<std::vector<char>> lp(N, std::vector<char>(N, 0));
    for (const auto &kv : jac) lp[kv.first.first][kv.first.second] = 1;
    for (int i = F; i < N; ++i)
        for (int j = F; j < N; ++j) lp[i][j] = 1;
    for (int k = 0; k < F; ++k)
        for (int i = k + 1; i < N; ++i)
            if (lp[i][k])
                for (int j = k + 1; j < N; ++j) lp[i][j] |= lp[k][j];

    // ---- local memory -------------------------------------------------------
    // [fixed cells][entries of the first part][of the second, fill last]
    // [scratch][y]; the staged tail entries take the second part's place until
    // it is assembled, and the rate partials reach down from the end of the
    // scratch into its fill.
    const int tm = (kMaxOrder + 1) * (kMaxOrder + 1);
    std::vector<std::vector<int>> at(N, std::vector<int>(N, -1));
    int lu_end = 0, scratch = 0, n_first = 0, n_second = 0;  // ends of the regions
    std::vector<int> fills[2];
    std::map<std::pair<int, int>, int> staged;
    // the first pivot that updates entry (i, j), if any; whether one before k does
    std::vector<std::vector<int>> updates(N, std::vector<int>(N, N));
    for (int x = N - 1; x >= 0; --x)
        for (int i = x + 1; i < N; ++i)
            if (lp[i][x])
                for (int j = x + 1; j < N; ++j)
                    if (lp[x][j]) updates[i][j] = x;
    auto before = [&](int i, int j, int k) { return updates[i][j] < k; };
    std::vector<std::vector<char>> assembled(N, std::vector<char>(N, 0));
    for (const auto &kv : jac) assembled[kv.first.first][kv.first.second] = 1;
    // Entries by the smaller of row and column, the front's with those that are
    // assembled; the tail's by whether they are, or the first pivot that updates them.
    std::vector<int> front_at(N + 1, 0), front_assembled(N + 1, 0), tail_at_pivot(N + 1, 0);
    int tail_assembled = 0;
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            if (std::min(i, j) < F && lp[i][j]) {
                front_at[std::min(i, j)]++;
                front_assembled[std::min(i, j)] += assembled[i][j];
            } else if (i >= F && j >= F) {
                if (assembled[i][j]) tail_assembled++;
                else tail_at_pivot[updates[i][j]]++;
            }
        }
    const int n_front = std::accumulate(front_at.begin(), front_at.end(), 0);
    // Sets the ends of the regions for a split; returns the doubles they take.
    auto size = [&](int split) {
        const auto upto = [&](const std::vector<int> &v) { return std::accumulate(v.begin(), v.begin() + split, 0); };
        n_first = kQFirst + upto(front_at);
        n_second = kQFirst + n_front;
        const int n_held = n_first + std::accumulate(front_assembled.begin() + split, front_assembled.end(), 0);
        const int ns = n_first + tail_assembled + upto(tail_at_pivot);
        lu_end = std::max(n_second, ns);
        const int held = std::max(n_held, ns);  // the partials stay above this
        scratch = std::max({R, tm, P - (lu_end - held)});
        return lu_end + scratch;
    };
    // Split: as many pivots as fit without taking more local memory, while a
    // pivot's tail update is small enough that its share of LU units (one
    // multiply-add of two gathered operands per 16 updates) is cheaper than the
    // dense update of the tail in registers (64 multiply-adds, any pivot).
    q.split = 0;
    q.m0 = std::max(0, F - L);
    const int room = size(0);
    for (int k = 0; k < q.m0; ++k) {
        int r = 0, cc = 0;
        for (int i = F; i < N; ++i) r += lp[i][k], cc += lp[k][i];
        if (r * cc > 160 || size(k + 1) > room) break;
        q.split = k + 1;
    }
    size(q.split);
    {
        int n = kQFirst;
        for (int part = 0; part < 2; ++part)
            for (int fill = 0; fill < 2; ++fill)
                for (int i = 0; i < N; ++i)
                    for (int j = 0; j < N; ++j)
                        if (lp[i][j] && std::min(i, j) < F && (std::min(i, j) >= q.split) == (part == 1) &&
                            (assembled[i][j] == 0) == (fill == 1)) {
                            if (fill && before(i, j, q.m0)) fills[part].push_back(n);
                            at[i][j] = n++;
                        }
        int ns = n_first;  // tail entries of the Jacobian, and those the first part's pivots update
        for (int i = F; i < N; ++i)
            for (int j = F; j < N; ++j)
                if (assembled[i][j] || before(i, j, q.split)) {
                    if (!assembled[i][j]) fills[0].push_back(ns);
                    staged[{i, j}] = ns++;
                }
    }
    q.off_r = lu_end;
    const int off_p = lu_end + scratch - P;
    q.off_y = lu_end + scratch;
    const int total = q.off_y + F + q.TB * L;
    q.stride = (total + 15) / 16 * 16;
    if (q.stride / 16 % 2 == 0) q.stride += 16;  // an odd multiple of 16 doubles: neighbour cells start on other banks
    // Three wavefronts' cells have to fit a compute unit's local memory.  One
    // cell / four cells a wavefront, ms, 10,000 cells: with 16 cells there 123 /
    // 93 (72 species, 136 reactions), 135 / 98 (80, 136); with 12, 141 / 128 (72,
    // 151), 165 / 164 (84, 159), 158 / 154 (88, 132), 146 / 136 (96, 144), and
    // 4,000 cells, a second round on 256 compute units, 69.5 / 66.9, 77.9 / 88.4,
    // 80.1 / 84.4, 73.9 / 74.9; with 8 cells 505 / 601 (96, 201).
    if ((int64_t)q.stride * 8 * kQCells * 3 > kQLdsBytes) return;
    auto yid = [&](int species) { return q.off_y + t->iperm[species]; };

    // ---- reactions -----------------------------------------------------------
    q.n_rx = (R + L - 1) / L;
    QRx idle{};
    idle.r = kQTrash;
    for (int x = 0; x < 3; ++x) idle.y[x] = kQOne, idle.d[x] = kQTrash;
    q.rx.assign((size_t)(q.n_rx + 2 * kQAhead) * L, idle);
    for (int j = 0; j < R; ++j)
        for (int l = d->reac_ptr[j]; l < d->reac_ptr[j + 1]; ++l)
            q.rx[j].y[l - d->reac_ptr[j]] = (uint16_t)yid(d->reac_idx[l]);
    for (int j = 0; j < R; ++j) q.rx[j].r = (uint16_t)(q.off_r + j);
    for (int a = 0; a < P; ++a) q.rx[parts[a].j].d[parts[a].slot] = (uint16_t)(off_p + a);

    // ---- f gather: two terms per block and iteration ---------------------------
    std::vector<std::vector<Term>> rows(N);
    for (int j = 0; j < R; ++j)
        for (const auto &kv : net(d, j))
            if (kv.second != 0.0) rows[t->iperm[kv.first]].push_back({kv.second, q.off_r + j});
    size_t longest = 0;
    for (auto &r : rows) longest = std::max(longest, r.size());
    q.fg_iters = (int)std::max<size_t>(2, (longest + 3) / 4 * 2);  // an even number
    q.nbp = (q.NB + 3) / 4 * 4;
    q.fg_coef.assign((size_t)(q.fg_iters + kQAhead) * q.NB * L * 2, 0.0);
    q.fg_idx.assign((size_t)(q.fg_iters + kQAhead) * L * q.nbp * 2, (uint16_t)kQZero);
    for (int p = 0; p < N; ++p)
        for (size_t x = 0; x < rows[p].size(); ++x) {
            const size_t it = x / 2;
            q.fg_coef[((it * q.NB + block_of(p)) * L + lane_of(p)) * 2 + x % 2] = rows[p][x].coef;
            q.fg_idx[((it * L + lane_of(p)) * q.nbp + block_of(p)) * 2 + x % 2] = (uint16_t)rows[p][x].src;
        }

    // ---- Newton matrix ---------------------------------------------------------
    std::vector<NmEntry> set[2];
    for (const auto &kv : jac) {
        const int i = kv.first.first, j = kv.first.second;
        NmEntry e;
        e.diag = i == j;
        e.terms = kv.second;
        for (Term &x : e.terms) x.src += off_p;
        const bool tail = i >= F && j >= F;
        e.dst = tail ? staged[{i, j}] : at[i][j];
        set[!tail && std::min(i, j) >= q.split].push_back(e);
    }
    for (int s = 0; s < 2; ++s) emit_nm(set[s], &q.nm[s], &q.nm_recs[s], &q.nm_two[s], &q.nm_one[s]);
    const int te = q.TB * q.NC;  // a multiple of 8
    q.tmap.assign((size_t)te * L, (uint16_t)kQZero);
    for (const auto &kv : staged) {
        const int i = kv.first.first - F, j = kv.first.second - F, e = i / L * q.NC + j;
        q.tmap[((size_t)(e / 8) * L + i % L) * 8 + e % 8] = (uint16_t)kv.second;
    }
    for (int part = 0; part < 2; ++part) {
        const int nf = (int)fills[part].size();
        q.n_fill[part] = (nf + 8 * L - 1) / (8 * L);
        q.fill[part].assign((size_t)(q.n_fill[part] + 1) * L * 8, (uint16_t)kQTrash);
        for (int e = 0; e < nf; ++e) q.fill[part][((size_t)(e / (8 * L)) * L + e % L) * 8 + e / L % 8] = (uint16_t)fills[part][e];
    }

    // ---- front LU: every entry formed once, when its operands are final --------
    // (left-looking: a_ij - sum_{q < min(i,j)} l_iq u_qj, then times 1 / u_jj
    // below the diagonal, reciprocal on it).  Entries whose operands are final
    // after the same number of steps form a level.
    // The first part's levels also hold the staged tail entries' sums over its
    // pivots.
    struct Ent { int i, j; std::vector<int> q; };
    QLuUnit nop{};
    for (int e = 0; e < kQLuEnt; ++e) nop.dst[e] = kQTrash, nop.scale[e] = kQOne;
    for (int s = 0; s < kQLuSteps; ++s)
        for (int e = 0; e < kQLuEnt; ++e) nop.lu[s][e][0] = nop.lu[s][e][1] = kQZero;
    std::vector<std::vector<int>> lev(N, std::vector<int>(N, 0));
    auto place = [&](int i, int j) { return i >= F && j >= F ? staged.at({i, j}) : at[i][j]; };
    for (int part = 0; part < 2; ++part) {
        std::map<int, std::vector<Ent>> levels[2];  // off the diagonal, on it
        int maxlev = 0;
        auto form = [&](int i, int j, int kmax, int base) {
            Ent e{i, j, {}};
            int l = base;
            for (int x = 0; x < kmax; ++x)
                if (lp[i][x] && lp[x][j]) {
                    e.q.push_back(x);
                    l = std::max({l, lev[i][x], lev[x][j]});
                }
            const bool tail = std::min(i, j) >= q.m0;  // a tail or middle entry: only the sum over the earlier pivots
            const bool op = (i >= j && !tail) || !e.q.empty();  // an untouched U, tail or middle entry stays as assembled
            if (!tail) lev[i][j] = l + (op ? 1 : 0);
            if (op) {
                levels[i == j && !tail][l + 1].push_back(e);
                maxlev = std::max(maxlev, l + 1);
            }
        };
        for (int k = part ? q.split : 0; k < (part ? q.m0 : q.split); ++k) {
            for (int j = k; j < N; ++j)
                if (lp[k][j]) form(k, j, k, 0);
            for (int i = k + 1; i < N; ++i)
                if (lp[i][k]) form(i, k, k, lev[k][k]);
        }
        if (part == 0)
            for (const auto &kv : staged) form(kv.first.first, kv.first.second, q.split, 0);
        else
            for (int i = q.m0; i < N; ++i)
                for (int j = q.m0; j < N; ++j)
                    if (lp[i][j] && std::min(i, j) < F) form(i, j, q.m0, 0);
        for (int l = 1; l <= maxlev; ++l) {
            // rounds of 16 entries, the diagonals apart (U and L together: a U entry is scaled by 1), longest first
            std::vector<std::pair<std::vector<Ent>, bool>> all;
            for (int dg = 1; dg >= 0; --dg) {
                std::vector<Ent> &v = levels[dg][l];
                std::stable_sort(v.begin(), v.end(), [](const Ent &a, const Ent &b) { return a.q.size() > b.q.size(); });
                for (size_t r = 0; r < v.size(); r += L)
                    all.push_back({std::vector<Ent>(v.begin() + r, v.begin() + std::min(v.size(), r + L)), dg != 0});
            }
            std::stable_sort(all.begin(), all.end(), [](const auto &a, const auto &b) { return a.first[0].q.size() > b.first[0].q.size(); });
            for (size_t r = 0; r < all.size(); r += kQLuEnt) {
                const int ne = (int)std::min<size_t>(kQLuEnt, all.size() - r);
                const size_t steps = all[r].first[0].q.size();
                const size_t units = std::max<size_t>(1, (steps + kQLuSteps - 1) / kQLuSteps);
                for (size_t u = 0; u < units; ++u) {
                    const size_t s0 = u * kQLuSteps, ns = std::min<size_t>(kQLuSteps, steps - std::min(steps, s0));
                    uint32_t fl = (uint32_t)ns;
                    for (int e = 0; e < ne; ++e)
                        if (all[r + e].second) fl |= kQLuD << e;
                    if (u > 0) fl |= kQLuCont;
                    if (u + 1 < units) fl |= kQLuMore;
                    std::vector<QLuUnit> lanes(L, nop);
                    for (int i = 0; i < L; ++i)
                        for (int e = 0; e < ne; ++e) {
                            const auto &rd = all[r + e].first;
                            if (i >= (int)rd.size()) continue;
                            const Ent &x = rd[i];
                            lanes[i].dst[e] = (uint16_t)place(x.i, x.j);
                            if (x.i > x.j && x.j < q.m0) lanes[i].scale[e] = (uint16_t)at[x.j][x.j];
                            for (size_t s = 0; s < ns && s0 + s < x.q.size(); ++s) {
                                lanes[i].lu[s][e][0] = (uint16_t)at[x.i][x.q[s0 + s]];
                                lanes[i].lu[s][e][1] = (uint16_t)at[x.q[s0 + s]][x.j];
                            }
                        }
                    q.lu.insert(q.lu.end(), lanes.begin(), lanes.end());
                    q.lu_flags.push_back(fl);
                    q.n_lu[part]++;
                }
            }
        }
        if (q.n_lu[part] % 2) {  // an even number of units
            q.lu.insert(q.lu.end(), L, nop);
            q.lu_flags.push_back(0);
            q.n_lu[part]++;
        }
    }
    for (int a = 0; a < kQAhead; ++a) {
        q.lu.insert(q.lu.end(), L, nop);
        q.lu_flags.push_back(0);
    }

    // ---- Schur complement of the second part: a pivot's L in the tail rows, its U in the tail columns
    auto off = [&](int i, int j) { return (uint16_t)(i < N && j < N && lp[i][j] ? at[i][j] : kQZero); };
    q.schur.assign((size_t)(q.m0 - q.split + 2 * kQAhead) * L, QSchur{});  // kQZero is 0
    for (int k = q.split; k < q.m0; ++k)
        for (int i = 0; i < L; ++i)
            for (int b = 0; b < 2; ++b) {
                q.schur[(size_t)(k - q.split) * L + i].l[b] = off(F + 16 * b + i, k);
                q.schur[(size_t)(k - q.split) * L + i].u[b] = off(k, F + 16 * b + i);
            }

    // ---- middle pivots: their rows (lane m0 + i) in the middle and tail columns, 48
    // registers, then the tail rows (two blocks) in the middle columns.  Loaded: the
    // entries that hold a value (assembled, or updated by an earlier pivot); stored:
    // every structural entry, in the places the sweeps read.
    if (F > 0) {
        q.mid_load.assign((size_t)kQMid * L, (uint16_t)kQZero);
        q.mid_store.assign((size_t)kQMid * L, (uint16_t)kQTrash);
        for (int e = 0; e < kQMid; ++e)
            for (int i = 0; i < L; ++i) {
                const bool u = e < 48;
                const int row = u ? (q.m0 + i < F ? q.m0 + i : N) : F + (e - 48) / 16 * L + i;
                const int mc = u ? e : (e - 48) % 16;  // middle column, or 16 + tail column
                const int col = mc < 16 ? (q.m0 + mc < F ? q.m0 + mc : N) : F + mc - 16;
                const size_t w = ((size_t)(e / 8) * L + i) * 8 + e % 8;
                if (u && row == N && mc == i) q.mid_load[w] = (uint16_t)kQOne;  // beyond the front: an identity row
                if (row >= N || col >= N || !lp[row][col]) continue;
                if (assembled[row][col] || before(row, col, q.m0)) q.mid_load[w] = (uint16_t)at[row][col];
                q.mid_store[w] = (uint16_t)at[row][col];
            }
    }

    // ---- sweep maps ------------------------------------------------------------
    // fwd: for every half block of front columns (8 of them), the L entries of
    // the rows of the front blocks from that column's block on, then of the
    // tail blocks.  bwt: for every half block of tail columns, last first, the
    // U entries of the front blocks' rows.  bwf: for every half block of front
    // columns, last first, the strictly upper U entries of the rows of the
    // front blocks up to its own.  Vectors of eight columns: [vector][lane][8].
    auto vec = [&](std::vector<uint16_t> *out, int rb, int c0, bool tail_cols, bool lower) {
        for (int i = 0; i < L; ++i)
            for (int c = 0; c < 8; ++c) {
                const int col = tail_cols ? F + c0 + c : c0 + c;
                const int row = rb >= q.FB ? F + (rb - q.FB) * L + i : rb * L + i;
                const bool in = col < (tail_cols ? N : F) && row < (rb >= q.FB ? N : F) && (lower ? row > col : row < col);
                out->push_back(in ? off(row, col) : (uint16_t)kQZero);
            }
    };
    for (int h = 0; h < 2 * q.FB; ++h)
        for (int b = h / 2; b < q.NB; ++b) vec(&q.fwd, b, 8 * h, false, true);
    for (int h = 2 * q.TB - 1; h >= 0; --h)
        for (int b = 0; b < q.FB; ++b) vec(&q.bwt, b, 8 * h, true, false);
    for (int h = 2 * q.FB - 1; h >= 0; --h)
        for (int b = 0; b <= h / 2; ++b) vec(&q.bwf, b, 8 * h, false, false);
    for (int s = 0; s < 2; ++s) q.nm_dev[s] = by_vector(q.nm[s]);
    q.lu_dev = by_vector(q.lu);
    q.dmap.assign((size_t)std::max(1, q.FB) * L, (uint16_t)kQOne);
    for (int k = 0; k < F; ++k) q.dmap[k] = (uint16_t)at[k][k];
    q.ok = true;
}

// One cell of the quad solver on the host, phase by phase as the kernel runs
// them (16 lanes in turn; within one LU unit every operand is read before any
// result is written).  Counts index violations and reads of cells that were
// never written in this evaluation.
int emulate_quad(const HostTables &t, const double *k, const double *y_species, double c, const double *b_species,
                 double *f_species, double *x_species)
{
    const QuadTables &q = t.quad;
    const int L = kQLanes, F = q.F, TB = q.TB, NC = q.NC;
    int bad = 0;
    std::vector<double> mem((size_t)q.stride, NAN);  // NaN: never written
    auto rd = [&](int a) {
        if (a < 0 || a >= q.stride || a == kQTrash) return ++bad, 0.0;
        return mem[a];
    };
    auto wr = [&](int a, double v) {
        if (a < 0 || a >= q.stride || a == kQZero || a == kQOne) ++bad;
        else mem[a] = v;
    };
    mem[kQZero] = 0.0;
    mem[kQOne] = 1.0;
    for (int b = 0; b < q.NB; ++b)
        for (int i = 0; i < L; ++i) {
            const int s = q.vsp[b * L + i];
            wr(q.off_y + (b < q.FB ? b * L : F + (b - q.FB) * L) + i, s >= 0 ? y_species[s] : 0.0);
        }
    auto kj = [&](int j) { return j < t.R ? k[j] : 0.0; };
    // f
    const int nr = (int)q.rx.size();  // idle lanes and rounds write to the write-only cell
    for (int j = 0; j < nr; ++j) wr(q.rx[j].r, kj(j) * rd(q.rx[j].y[0]) * rd(q.rx[j].y[1]) * rd(q.rx[j].y[2]));
    for (int b = 0; b < q.NB; ++b)
        for (int i = 0; i < L; ++i) {
            double acc = 0.0;
            for (int it = 0; it < q.fg_iters; ++it)
                for (int x = 0; x < 2; ++x)
                    acc += q.fg_coef[(((size_t)it * q.NB + b) * L + i) * 2 + x] *
                           rd(q.fg_idx[(((size_t)it * L + i) * q.nbp + b) * 2 + x]);
            if (q.vsp[b * L + i] >= 0) f_species[q.vsp[b * L + i]] = acc;
        }
    // rate partials and the Newton matrix
    for (int j = 0; j < nr; ++j) {
        const double ya = rd(q.rx[j].y[0]), yb = rd(q.rx[j].y[1]), yc = rd(q.rx[j].y[2]);
        const double kc = -c * kj(j);
        wr(q.rx[j].d[0], kc * yb * yc);
        wr(q.rx[j].d[1], kc * ya * yc);
        wr(q.rx[j].d[2], kc * ya * yb);
    }
    std::vector<double> T((size_t)TB * NC * L, 0.0);
    auto tat = [&](int rb, int col, int i) -> double & { return T[((size_t)rb * NC + col) * L + i]; };
    int unit = 0;
    for (int s = 0; s < 2; ++s) {
        std::vector<double> acc(L, 0.0);
        for (int r = 0; r < q.nm_recs[s]; ++r)
            for (int i = 0; i < L; ++i) {
                const QNmRec &e = q.nm[s][(size_t)r * L + i];
                double x[4];
                for (int a = 0; a < 4; ++a) x[a] = rd(e.src[a]);
                if (r >= q.nm_one[s])
                    for (int a = 0; a < 4; ++a) wr(e.dst[a], e.coef[a] * x[a]);
                else if (r >= q.nm_two[s])
                    for (int a = 0; a < 2; ++a) wr(e.dst[a], e.coef[2 * a] * x[2 * a] + e.coef[2 * a + 1] * x[2 * a + 1]);
                else {
                    for (int a = 0; a < 4; ++a) acc[i] += e.coef[a] * x[a];
                    if (e.dst[3] != q.nm[s][(size_t)r * L].dst[3]) ++bad;
                    if (e.dst[3] != kQNmMore) {
                        wr(e.dst[0], e.dst[3] == kQNmDiag ? 1.0 + acc[i] : acc[i]);
                        acc[i] = 0.0;
                    }
                }
            }
        for (size_t e = 0; e < (size_t)q.n_fill[s] * L * 8; ++e) wr(q.fill[s][e], 0.0);
        std::vector<double> sum(kQLuEnt * L, 0.0), res(kQLuEnt * L);
        for (int n = 0; n < q.n_lu[s]; ++n, ++unit) {
            const uint32_t fl = q.lu_flags[unit];
            for (int i = 0; i < L; ++i) {
                const QLuUnit &e = q.lu[(size_t)unit * L + i];
                for (int x = 0; x < kQLuEnt; ++x) {
                    double a = fl & kQLuCont ? sum[kQLuEnt * i + x] : (e.dst[x] == kQTrash ? 0.0 : rd(e.dst[x]));
                    for (int st = 0; st < (int)(fl & 15); ++st) a -= rd(e.lu[st][x][0]) * rd(e.lu[st][x][1]);
                    sum[kQLuEnt * i + x] = a;
                    res[kQLuEnt * i + x] = fl & (kQLuD << x) ? 1.0 / a : a * rd(e.scale[x]);
                }
            }
            if (!(fl & kQLuMore))
                for (int i = 0; i < L; ++i)
                    for (int x = 0; x < kQLuEnt; ++x) wr(q.lu[(size_t)unit * L + i].dst[x], res[kQLuEnt * i + x]);
        }
        if (s == 0)
            for (int e = 0; e < TB * NC; ++e)
                for (int i = 0; i < L; ++i) tat(e / NC, e % NC, i) = rd(q.tmap[((size_t)(e / 8) * L + i) * 8 + e % 8]);
    }
    // Schur complement, dense tail
    for (int p = 0; p < q.m0 - q.split; ++p)
        for (int rb = 0; rb < TB; ++rb)
            for (int i = 0; i < L; ++i)
                for (int col = 0; col < NC; ++col)
                    tat(rb, col, i) -= rd(q.schur[(size_t)p * L + i].l[rb]) * rd(q.schur[(size_t)p * L + col % L].u[col / L]);
    if (F > 0) {
        std::vector<double> mr((size_t)kQMid * L);
        auto um = [&](int col, int i) -> double & { return mr[(size_t)col * L + i]; };
        auto lt = [&](int b, int col, int i) -> double & { return mr[(size_t)(48 + 16 * b + col) * L + i]; };
        for (int e = 0; e < kQMid; ++e)
            for (int i = 0; i < L; ++i) mr[(size_t)e * L + i] = rd(q.mid_load[((size_t)(e / 8) * L + i) * 8 + e % 8]);
        for (int p = 0; p < F - q.m0; ++p) {
            const double inv = 1.0 / um(p, p);
            for (int i = p + 1; i < L; ++i) {
                um(p, i) *= inv;
                for (int col = p + 1; col < 48; ++col) um(col, i) -= um(p, i) * um(col, p);
            }
            for (int b = 0; b < 2; ++b)
                for (int i = 0; i < L; ++i) {
                    lt(b, p, i) *= inv;
                    for (int col = p + 1; col < 16; ++col) lt(b, col, i) -= lt(b, p, i) * um(col, p);
                    for (int col = 0; col < 32; ++col) tat(b, col, i) -= lt(b, p, i) * um(16 + col, p);
                }
            um(p, p) = inv;
        }
        for (int e = 0; e < kQMid; ++e)
            for (int i = 0; i < L; ++i) wr(q.mid_store[((size_t)(e / 8) * L + i) * 8 + e % 8], mr[(size_t)e * L + i]);
    }
    std::vector<double> dinv((size_t)TB * L, 1.0);
    for (int p = 0; p < q.Mt; ++p) {
        const int pb = p / L, pl = p % L;
        const double inv = 1.0 / tat(pb, p, pl);
        dinv[p] = inv;
        for (int rb = pb; rb < TB; ++rb)
            for (int i = 0; i < L; ++i) {
                if (rb == pb && i <= pl) continue;
                const double l = tat(rb, p, i) * inv;
                tat(rb, p, i) = l;
                for (int col = p + 1; col < NC; ++col) tat(rb, col, i) -= l * tat(pb, col, pl);
            }
    }
    // solve
    std::vector<double> b((size_t)q.NB * L, 0.0);
    for (int e = 0; e < q.NB * L; ++e)
        if (q.vsp[e] >= 0) b[e] = b_species[q.vsp[e]];
    auto field = [&](const std::vector<uint16_t> &m, size_t v, int i, int cc) { return rd(m[(v * L + i) * 8 + cc]); };
    const size_t bt = (size_t)q.FB * L;  // the tail's part of b
    size_t v = 0;
    for (int h = 0; h < 2 * q.FB; ++h) {
        const int nb = q.NB - h / 2;
        for (int cc = 0; cc < 8; ++cc) {
            const double x = b[(size_t)(h / 2) * L + (h % 2) * 8 + cc];
            for (int w = 0; w < nb; ++w)
                for (int i = 0; i < L; ++i) b[(size_t)(h / 2 + w) * L + i] -= field(q.fwd, v + w, i, cc) * x;
        }
        v += nb;
    }
    for (int p = 0; p < q.Mt; ++p)
        for (int rb = p / L; rb < TB; ++rb)
            for (int i = 0; i < L; ++i)
                if (rb > p / L || i > p % L) b[bt + rb * L + i] -= tat(rb, p, i) * b[bt + p];
    v = 0;
    for (int h = 2 * TB - 1; h >= 0; --h) {
        for (int cc = 7; cc >= 0; --cc) {
            const int p = 8 * h + cc;
            if (p >= q.Mt) continue;
            const double x = b[bt + p] * dinv[p];
            for (int rb = 0; rb <= p / L; ++rb)
                for (int i = 0; i < L; ++i)
                    if (rb < p / L || i < p % L) b[bt + rb * L + i] -= tat(rb, p, i) * x;
            for (int w = 0; w < q.FB; ++w)
                for (int i = 0; i < L; ++i) b[(size_t)w * L + i] -= field(q.bwt, v + w, i, cc) * x;
            b[bt + p] = x;
        }
        v += q.FB;
    }
    v = 0;
    for (int h = 2 * q.FB - 1; h >= 0; --h) {
        for (int cc = 7; cc >= 0; --cc) {
            const int kcol = 8 * h + cc;
            if (kcol >= F) continue;
            const double x = b[kcol] * rd(q.dmap[kcol]);
            for (int w = 0; w <= h / 2; ++w)
                for (int i = 0; i < L; ++i) b[(size_t)w * L + i] -= field(q.bwf, v + w, i, cc) * x;
            b[kcol] = x;
        }
        v += h / 2 + 1;
    }
    for (int e = 0; e < q.NB * L; ++e)
        if (q.vsp[e] >= 0) x_species[q.vsp[e]] = b[e];
    return bad;
}

}  // namespace mcc
