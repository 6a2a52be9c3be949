// Host-side self-test of the transform schedules (wht_plan.h), compiled with the host compiler only.
// For every (schedule, log2 d) the library instantiates it checks that
//   - every stage runs exactly once (matrix-core bits included) and only on register-resident bits,
//   - in every phase (thread, register) -> element is a bijection onto [0, d),
//   - the LDS address map is injective, keeps 16-byte groups together, is additive over disjoint
//     bit sets and stays inside the token's region,
//   - the first and last phases give each lane whole 16-byte vectors, contiguous across >= 8 lanes,
//   - for the matrix-core schedule, the first layout is the MFMA operand layout the kernels assume
//     (registers = bits 0,1,2,9,tile bits; lanes = bits 3..8),
// and it emulates the whole schedule on the CPU (registers + an LDS array, phase by phase, in forward
// and in reverse order, the matrix-core rounds as butterflies on their bits) against a direct +-1
// sum on small sizes.
// Prints one line per configuration; exit status 0 iff all pass.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "wht_plan.h"

using namespace wht;

typedef unsigned (*PhysFn)(unsigned);
static unsigned phys_plain(unsigned i) { return lds_phys_plain(i); }
static unsigned phys_rot(unsigned i) { return lds_phys_rot(i); }

static unsigned thread_elem(const PhaseDesc& p, int n, int e, unsigned t) {
    unsigned off = 0;
    for (int k = 0; k < n - e; ++k) off |= ((t >> k) & 1u) << p.tb[k];
    return off;
}

static void butterfly_bits(std::vector<double>& a, unsigned bits) {
    const unsigned D = (unsigned)a.size();
    for (unsigned b = 0; (1u << b) < D; ++b) {
        if (!((bits >> b) & 1u)) continue;
        for (unsigned i = 0; i < D; ++i)
            if (!((i >> b) & 1u)) {
                const double u = a[i], w = a[i | (1u << b)];
                a[i] = u + w; a[i | (1u << b)] = u - w;
            }
    }
}

static bool check(const char* kind, const PlanDesc& pl, PhysFn phys, unsigned words, bool verbose) {
    const int n = pl.n, e = pl.e, v = pl.v;
    const unsigned D = 1u << n, E = 1u << e, T = 1u << (n - e);
    bool ok = plan_is_complete(pl);
    // address map
    std::vector<char> used(words, 0);
    for (unsigned i = 0; i < D; ++i) {
        const unsigned a = phys(i);
        if (a >= words || used[a]) ok = false; else used[a] = 1;
        if ((i & 3u) == 0 && ((a & 3u) != 0 || phys(i + 3) != a + 3)) ok = false;
    }
    for (int p = 0; p < pl.nphase; ++p) {
        std::vector<char> seen(D, 0);
        for (unsigned t = 0; t < T; ++t)
            for (unsigned r = 0; r < E; ++r) {
                const unsigned a = thread_elem(pl.ph[p], n, e, t), b = reg_elem_offset(pl.ph[p], e, (int)r);
                if (a & b) ok = false;
                const unsigned el = a | b;
                if (el >= D || seen[el]) ok = false; else seen[el] = 1;
                if (phys(el) != phys(a) + phys(b)) ok = false;
            }
    }
    // global layouts: vector bits in the low register bits, low thread bits follow on
    for (int p : {0, pl.nphase - 1}) {
        for (int q = 0; q < v; ++q) if (pl.ph[p].rb[q] != q) ok = false;
        int run = 0;
        while (run < n - e && pl.ph[p].tb[run] == v + run) ++run;
        if (n - e > 0 && run < ((n - e) < 3 ? (n - e) : 3)) ok = false;   // >= 128 contiguous bytes
    }
    if (pl.mfma_bits) {
        // operand layout of the matrix-core rounds
        const PhaseDesc& f = pl.ph[0];
        if (pl.mfma_bits != 0x3ffu || v != 3) ok = false;
        if (f.rb[0] != 0 || f.rb[1] != 1 || f.rb[2] != 2 || f.rb[3] != 9) ok = false;
        for (int q = 4; q < e; ++q) if (f.rb[q] != 10 + (q - 4)) ok = false;
        for (int k = 0; k < 6; ++k) if (f.tb[k] != 3 + k) ok = false;
        // every layout keeps lanes on bits 3..8, so the exchange is between waves only
        for (int p = 0; p < pl.nphase; ++p)
            for (int k = 0; k < 6; ++k) if (pl.ph[p].tb[k] != 3 + k) ok = false;
    }
    if (pl.lane_bits) {
        // wave schedule: lane positions 0..5 carry element bits v.. in the first layout, positions 0..3
        // in every layout; position k's DPP partner differs in element bit v+k and in no other
        const int L = n - e < 6 ? n - e : 6;
        for (int k = 0; k < L; ++k) if (pl.ph[0].tb[k] != v + k) ok = false;
        for (int p = 0; p < pl.nphase; ++p)
            for (int k = 0; k < L && k < 4; ++k) if (pl.ph[p].tb[k] != v + k) ok = false;
        const unsigned partner[4] = {1, 2, 7, 8};
        for (int k = 0; k < L && k < 4; ++k) {
            if (!((pl.lane_bits >> (v + k)) & 1u)) ok = false;
            for (unsigned l = 0; l < 64; ++l)
                if ((wave_lane_to_bits(l, L) ^ wave_lane_to_bits(l ^ partner[k], L)) != (1u << k)) ok = false;
        }
        // the second layout is the first with lane positions 4 (5) and register bits e-1 (e-2) exchanged;
        // the third with wave positions and register bits v, v+1 exchanged: nothing else moves
        for (int p = 1; p < pl.nphase; ++p) {
            PhaseDesc x = pl.ph[p - 1];
            if (p == 1)
                for (int k = 4; k < L; ++k) { const int b = x.tb[k]; x.tb[k] = x.rb[e - 1 - (k - 4)]; x.rb[e - 1 - (k - 4)] = b; }
            else
                for (int k = 0; k < n - e - 6; ++k) { const int b = x.tb[6 + k]; x.tb[6 + k] = x.rb[v + k]; x.rb[v + k] = b; }
            for (int q = 0; q < e; ++q) if (x.rb[q] != pl.ph[p].rb[q]) ok = false;
            for (int k = 0; k < n - e; ++k) if (x.tb[k] != pl.ph[p].tb[k]) ok = false;
        }
    }
    // emulate on the CPU for small d
    if (n <= 12) {
        for (int reverse = 0; reverse < 2; ++reverse) {
            std::vector<double> x(D), lds(words, NAN), want(D);
            for (unsigned i = 0; i < D; ++i) x[i] = std::sin(0.37 * i + 1.0) + (i % 7) * 0.25;
            want = x;
            butterfly_bits(want, D - 1);
            if (n <= 9) {       // and the direct sum itself on the smallest sizes
                for (unsigned j = 0; j < D; ++j) {
                    double s = 0;
                    for (unsigned k = 0; k < D; ++k) s += (__builtin_popcount(j & k) & 1) ? -x[k] : x[k];
                    if (std::fabs(s - want[j]) > 1e-9 * (1 + std::fabs(s))) ok = false;
                }
            }
            // the matrix-core rounds come first going forward (on the data as loaded) ...
            if (!reverse) butterfly_bits(x, pl.mfma_bits | pl.lane_bits);
            std::vector<std::vector<double>> reg(T, std::vector<double>(E));
            for (int s = 0; s < pl.nphase; ++s) {
                const int p = reverse ? pl.nphase - 1 - s : s;
                const PhaseDesc& ph = pl.ph[p];
                for (unsigned t = 0; t < T; ++t) {
                    const unsigned base = thread_elem(ph, n, e, t);
                    for (unsigned r = 0; r < E; ++r) {
                        const unsigned el = base | reg_elem_offset(ph, e, (int)r);
                        reg[t][r] = (s == 0) ? x[el] : lds[phys(el)];
                    }
                    for (int q = 0; q < e; ++q) {
                        if (!((ph.stages >> ph.rb[q]) & 1u)) continue;
                        for (unsigned r = 0; r < E; ++r)
                            if (!((r >> q) & 1u)) {
                                const double a = reg[t][r], b = reg[t][r | (1u << q)];
                                reg[t][r] = a + b; reg[t][r | (1u << q)] = a - b;
                            }
                    }
                }
                // write-back happens after every thread has read (the barrier in the kernel)
                for (unsigned t = 0; t < T; ++t) {
                    const unsigned base = thread_elem(ph, n, e, t);
                    for (unsigned r = 0; r < E; ++r)
                        lds[phys(base | reg_elem_offset(ph, e, (int)r))] = reg[t][r];
                }
            }
            std::vector<double> got(D);
            for (unsigned j = 0; j < D; ++j) got[j] = lds[phys(j)];
            // ... and last in reverse (on the registers of the first layout)
            if (reverse) butterfly_bits(got, pl.mfma_bits | pl.lane_bits);
            double worst = 0, big = 0;
            for (unsigned j = 0; j < D; ++j) {
                worst = std::fmax(worst, std::fabs(got[j] - want[j]));
                big = std::fmax(big, std::fabs(want[j]));
            }
            if (!(worst <= 1e-9 * big)) ok = false;
        }
    }
    std::printf("%-9s n=%2d e=%d v=%d phases=%d lds_words=%u %s\n", kind, n, e, v, pl.nphase, words,
                ok ? "ok" : "FAIL");
    if (verbose || !ok)
        for (int p = 0; p < pl.nphase; ++p) {
            std::printf("   phase %d regs:", p);
            for (int q = 0; q < e; ++q) std::printf(" %d", pl.ph[p].rb[q]);
            std::printf("  stages 0x%x  threads:", pl.ph[p].stages);
            for (int k = 0; k < n - e; ++k) std::printf(" %d", pl.ph[p].tb[k]);
            std::printf("\n");
        }
    return ok;
}

// Rows of 12 * 2^m elements: the layouts must be bijections onto the token's elements (or the two tokens of
// 768), the exchange must go through the LDS words the kernels use, and the two rounds -- emulated from the operand
// words the kernels load and the 16x16x32 product's lane layout -- with the stages after them must equal the definition
//     out[j] = sum_k P12[j / L][k / L] * (-1)^popcount(j & k & (L - 1)) * x[k],   L = 2^m,
// in forward order (rounds first) and in reverse.
typedef std::vector<std::vector<double>> Regs;         // [lane of the token's waves][24]

// D[i][j] += sum_k A[i][k] B[k][j]:  A: lane i + 16 (k / 8), element k % 8;  B: lane j + 16 (k / 8), element
// k % 8;  D: lane j + 16 (i / 4), register i % 4.  Operands hold 8 values of each of the 64 lanes.
static void product(const double (&A)[64][8], const double (&B)[64][8], double (&D)[64][4]) {
    for (int i = 0; i < 16; ++i)
        for (int j = 0; j < 16; ++j)
            for (int k = 0; k < 32; ++k)
                D[j + 16 * (i / 4)][i % 4] += A[i + 16 * (k / 8)][k % 8] * B[j + 16 * (k / 8)][k % 8];
}

static double word_value(unsigned word, int odd) {
    const unsigned h = odd ? word >> 16 : word & 0xffffu;
    return h == 0u ? 0.0 : (h == 0x3F80u ? 1.0 : (h == 0xBF80u ? -1.0 : NAN));
}

static void twelve_rounds(std::vector<double>* lanes, int m) {        // one wave: 64 x 24 registers
    double d1[3][2][64][4] = {}, out[64][24] = {};
    for (int v = 0; v < 3; ++v)
        for (int h = 0; h < 2; ++h) {
            double A[64][8], B[64][8];
            for (int l = 0; l < 64; ++l)
                for (int e = 0; e < 8; ++e) {
                    A[l][e] = lanes[l][8 * v + e];
                    B[l][e] = word_value(twelve_round1_word(l, h, e / 2), e & 1);
                }
            product(A, B, d1[v][h]);
        }
    for (int h = 0; h < 2; ++h)
        for (int pair = 0; pair < 2; ++pair) {
            double A[64][8], B[64][8], S[64][8], main[64][4] = {}, shared[64][4] = {};
            for (int l = 0; l < 64; ++l)
                for (int e = 0; e < 8; ++e) {
                    A[l][e] = d1[(e / 4) == pair ? pair : 2][h][l][e % 4];
                    B[l][e] = word_value(twelve_round2_word(l, pair, false, e / 2, m), e & 1);
                    S[l][e] = word_value(twelve_round2_word(l, pair, true, e / 2, m), e & 1);
                }
            product(A, B, main);
            product(A, S, shared);
            for (int l = 0; l < 64; ++l)
                for (int i = 0; i < 4; ++i) {
                    out[l][8 * pair + 4 * h + i] += main[l][i];
                    out[l][16 + 4 * h + i] += shared[l][i];
                }
        }
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 24; ++i)       // the stage on r6, which the product has done for vector 2
            lanes[l][i] = m == 6 || i >= 16 ? out[l][i] : (i < 8 ? out[l][i] + out[l][8 + i] : out[l][i - 8] - out[l][i]);
}

// a - b in the upper of two places of one vector, a + b in the lower (the kernels' DPP stages, signs resolved)
static void lane_stage(Regs& r, int pos) {
    const Regs old = r;
    for (unsigned t = 0; t < r.size(); ++t)
        for (int i = 0; i < 24; ++i) {
            const double own = old[t][i], other = old[t ^ (1u << pos)][i];
            r[t][i] = ((t >> pos) & 1u) ? other - own : own + other;
        }
}

// The exchange as the kernels do it: every thread puts its registers, four at a time, into the LDS words of one
// layout and gets them from those of the other.  Words inside the region, 16-byte aligned, written once, all read.
static bool twelve_exchange(Regs& r, int w, bool put_last) {
    std::vector<double> lds(twelve_exchange_words(w), NAN);
    bool ok = true;
    for (bool get : {false, true})
        for (unsigned t = 0; t < r.size(); ++t) {
            const unsigned lane = t & 63u, wave = t >> 6;
            const LaneWave to = twelve_swap(lane, wave, w);
            const unsigned at = get == put_last ? twelve_place(to.lane, to.wave) : twelve_place(lane, wave);
            for (unsigned i = 0; i < 24; i += 4) {
                const unsigned word = at + twelve_exchange_reg((int)i, w);
                if (word % 4 != 0 || word + 4 > lds.size()) return false;
                for (unsigned k = 0; k < 4; ++k) {
                    if (!get && !std::isnan(lds[word + k])) ok = false;
                    if (get) { r[t][i + k] = lds[word + k]; lds[word + k] = NAN; }
                    else lds[word + k] = r[t][i + k];
                    if (std::isnan(r[t][i + k])) ok = false;
                }
            }
        }
    return ok;
}

// In place (y = x, dx = dy): without an exchange between them, no wave may store what another has still to fetch.
static bool check_twelve_in_place(int m) {
    const int w = twelve_wave_bits(m);
    const unsigned D = 12u << m, tokens = m == 6 ? 2 : 1;
    std::vector<unsigned> fetched(tokens * D, 0), stored(tokens * D, 0);        // by element: bit set of the waves
    for (unsigned wave = 0; wave < 1u << w; ++wave)
        for (unsigned lane = 0; lane < 64; ++lane)
            for (int vec = 0; vec < 3; ++vec) {
                const unsigned token = m == 6 ? twelve_pair(lane, vec) * D : 0u;
                const LaneWave to = twelve_swap(lane, wave, w);
                for (unsigned i = 0; i < 8; ++i) {
                    fetched[token + twelve_elem(lane, wave, vec, m) + i] |= 1u << wave;
                    stored[token + twelve_elem(to.lane, to.wave, vec, m) + i] |= 1u << wave;
                }
            }
    bool crossed = false, ok = true;
    for (unsigned e = 0; e < tokens * D; ++e) {
        if (__builtin_popcount(stored[e]) != 1) ok = false;           // stored once
        if (fetched[e] & ~stored[e]) crossed = true;
    }
    if (crossed && w == 0) ok = false;
    std::printf("in place  row=%u crossed=%d %s\n", D, crossed, ok ? "ok" : "FAIL");
    return ok;
}

static bool check_twelve(int m) {
    const unsigned L = 1u << m, D = 12 * L;
    const int w = twelve_wave_bits(m);
    const unsigned W = 1u << w, T = 64 * W, tokens = m == 6 ? 2 : 1;
    bool ok = true;
    auto place = [&](unsigned t) { return LaneWave{t & 63u, t >> 6}; };
    auto elem = [&](unsigned t, int vec, bool last) {           // index within the wave's tokens
        LaneWave p = place(t);
        if (last) p = twelve_swap(p.lane, p.wave, w);
        return twelve_elem(p.lane, p.wave, vec, m) + (m == 6 ? twelve_pair(p.lane, vec) * D : 0u);
    };
    for (bool last : {false, true}) {
        std::vector<int> hit(D * tokens, 0);
        for (unsigned t = 0; t < T; ++t)
            for (int vec = 0; vec < 3; ++vec)
                for (int i = 0; i < 8; ++i) {
                    const unsigned e = elem(t, vec, last) + i;
                    if (e >= D * tokens) { ok = false; continue; }
                    ++hit[e];
                }
        for (int h : hit) if (h != 1) ok = false;
    }
    std::vector<int> column(12 * (L + 16), 0);
    for (unsigned t = 0; t < T; ++t) {
        const LaneWave p = place(t), q = twelve_swap(p.lane, p.wave, w), back = twelve_swap(q.lane, q.wave, w);
        if (back.lane != p.lane || back.wave != p.wave || q.wave >= W) ok = false;
    }
    for (unsigned e = 0; e < D; ++e)
        if (twelve_column(e, m) >= column.size() || column[twelve_column(e, m)]++) ok = false;
    std::vector<double> x(D * tokens), want(D * tokens, 0.0);
    uint32_t rng = 12345u + (uint32_t)m;
    for (double& v : x) { rng = rng * 1664525u + 1013904223u; v = (double)((int)(rng >> 24) - 128); }   // exact in double
    for (unsigned tok = 0; tok < tokens; ++tok) {
        std::vector<double> z(x.begin() + tok * D, x.begin() + (tok + 1) * D);
        for (unsigned s = 1; s < L; s *= 2)                    // Sylvester stages inside every block
            for (unsigned k = 0; k < D; ++k)
                if (!(k & s)) { const double a = z[k], c = z[k + s]; z[k] = a + c; z[k + s] = a - c; }
        for (unsigned j = 0; j < D; ++j)
            for (unsigned k = 0; k < 12; ++k)
                want[tok * D + j] += (((paley12_minus_row(j / L) >> k) & 1u) ? -1 : 1) * z[k * L + j % L];
    }
    for (int reverse = 0; reverse < 2; ++reverse) {
        Regs r(T, std::vector<double>(24));
        for (unsigned t = 0; t < T; ++t)
            for (int i = 0; i < 24; ++i) r[t][i] = x[elem(t, i / 8, reverse != 0) + i % 8];
        auto rounds = [&] { for (unsigned wave = 0; wave < W; ++wave) twelve_rounds(&r[64 * wave], m); };
        auto exchange = [&] { if (w > 0) ok = twelve_exchange(r, w, reverse != 0) && ok; };
        auto wave_stages = [&] { for (int k = 0; k < w; ++k) lane_stage(r, twelve_lane_pos(k)); };
        if (!reverse) { rounds(); exchange(); wave_stages(); }
        else          { wave_stages(); exchange(); rounds(); }
        for (unsigned t = 0; t < T; ++t)
            for (int i = 0; i < 24; ++i)
                if (r[t][i] != want[elem(t, i / 8, reverse == 0) + i % 8]) ok = false;
    }
    std::printf("twelve    n=%2d row=%u waves=%u %s\n", m + 4, D, W, ok ? "ok" : "FAIL");
    return ok;
}

int main(int argc, char** argv) {
    if (argc > 1 && std::string(argv[1]) == "--p12") {     // print the order-12 factor, rows of +/-
        for (unsigned r = 0; r < 12; ++r) {
            for (unsigned c = 0; c < 12; ++c) std::putchar(((paley12_minus_row(r) >> c) & 1u) ? '-' : '+');
            std::putchar('\n');
        }
        return 0;
    }
    bool ok = true;
    const bool verbose = argc > 1;
    for (int m = 6; m <= 10; ++m) ok = check_twelve(m) && ok;
    for (int m = 6; m <= 10; ++m) ok = check_twelve_in_place(m) && ok;
    for (int v : {2, 3})
        for (int n = 5; n <= (v == 2 ? 13 : 14); ++n) {
            const PlanDesc pl = make_wave_plan(n, wave_log_e(n, v), v);
            ok = check("wave", pl, phys_plain, 1u << n, verbose) && ok;
        }
    for (int n = 10; n <= 14; ++n)
        for (int backward = 0; backward < 2; ++backward) {
            if (backward && mfma_log_tiles(n, true) == mfma_log_tiles(n, false)) continue;
            const PlanDesc pl = make_mfma_plan(n, mfma_log_tiles(n, backward != 0));
            ok = check("mfma", pl, phys_rot, 1u << n, verbose) && ok;
        }
    return ok ? 0 : 1;
}
