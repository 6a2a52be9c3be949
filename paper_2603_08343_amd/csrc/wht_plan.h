// Compile-time schedule of one token's fast Walsh-Hadamard transform across a group of threads.
//
// A token has d = 2^n elements.  It is held by 2^(n-e) threads, 2^e values per thread, in float32
// registers.  A butterfly stage on element-index bit b (paper Fig. 2: pairs whose indices differ by
// the stride 2^b) costs one add or subtract per element when bit b is a bit of the *register*
// index, so the schedule is a short list of layouts ("phases"); each phase names which e element
// bits are register-resident, the stages run on those, and between phases bits change places: through
// LDS, or by swaps between the lanes of a wave.  Stages commute (they act on different index bits), so any
// order gives H_raw x.
//
// The first and the last layout keep element bits 0..v-1 in registers (2^v elements = one 16-byte
// global vector) and give the lowest thread bits the next element bits, so that global loads and
// stores are 16 bytes per lane and contiguous across lanes.
#pragma once

namespace wht {

constexpr int kMaxRegBits = 6;
constexpr int kMaxBits = 16;
constexpr int kMaxPhases = 5;

struct PhaseDesc {
    int rb[kMaxRegBits];   // rb[q]: element-index bit carried by bit q of the register index
    int tb[kMaxBits];      // tb[k]: element-index bit carried by bit k of the thread index
    unsigned stages;       // element bits butterflied while the token is in this layout
};

struct PlanDesc {
    int n, e, v, nphase;
    unsigned mfma_bits;    // element bits transformed by the matrix-core rounds (in the first layout)
    unsigned lane_bits;    // element bits transformed between lanes, by DPP operands (wave schedule)
    PhaseDesc ph[kMaxPhases];
};


constexpr unsigned reg_mask(const PhaseDesc& p, int e) {
    unsigned m = 0;
    for (int q = 0; q < e; ++q) m |= 1u << p.rb[q];
    return m;
}

constexpr void fill_thread_bits(PhaseDesc& p, int n, int e) {
    const unsigned inreg = reg_mask(p, e);
    int k = 0;
    for (int b = 0; b < n; ++b)
        if (!((inreg >> b) & 1u)) p.tb[k++] = b;
    for (; k < kMaxBits; ++k) p.tb[k] = 0;
}

// Element offset contributed by register index r in a phase.
constexpr unsigned reg_elem_offset(const PhaseDesc& p, int e, int r) {
    unsigned off = 0;
    for (int q = 0; q < e; ++q)
        if ((r >> q) & 1) off |= 1u << p.rb[q];
    return off;
}

// Every element bit must be butterflied exactly once over the phases.
constexpr bool plan_is_complete(const PlanDesc& pl) {
    unsigned seen = pl.mfma_bits | pl.lane_bits;
    for (int p = 0; p < pl.nphase; ++p) {
        if (seen & pl.ph[p].stages) return false;
        if (pl.ph[p].stages & ~reg_mask(pl.ph[p], pl.e)) return false;
        seen |= pl.ph[p].stages;
    }
    return seen == (1u << pl.n) - 1u;
}

// Every layout keeps element bits 0 and 1 in the low register bits: four consecutive values, one 16-byte
// LDS access.
constexpr bool plan_keeps_vectors(const PlanDesc& pl) {
    for (int p = 0; p < pl.nphase; ++p)
        if (pl.ph[p].rb[0] != 0 || pl.ph[p].rb[1] != 1) return false;
    return true;
}

// ---- the matrix-core schedule (bfloat16 I/O, d >= 1024) ---------------------------------------
//
// H_32 applied along five element bits is a 32x32 (+-1) matrix product, which the MFMA unit does
// with exact products and float32 accumulation.  Two such rounds cover bits 0..9:
//   round 1 contracts bits {0,1,2,8,9}: each lane feeds 8 consecutive elements (one 16-byte global
//           vector, bits 0..2), the lane's upper half selects bit 8, the two instructions bit 9;
//           the 32 rows are bits 3..7 (lanes 0..31 read 512 contiguous bytes);
//   round 2 contracts bits {3..7}: the accumulator layout of round 1 has those bits in the register
//           index and the lane's upper half, which is exactly an A-operand layout again.
// After round 2 every lane holds 8 consecutive elements per 16 registers -- the layout it loaded
// in -- so the rounds map the first layout onto itself and leave d/1024 = 2^(t+w) sub-transforms to
// combine: t "tile" bits in registers (2^t MFMA tiles per wave), w bits across the waves of the
// token.  One LDS exchange brings up to 1+t of the wave bits into registers (in place of the first
// layout's upper register bits, whose stages are done); a token of more than 2^(1+t) waves takes a
// second exchange for the rest.
//   first layout : registers (0,1,2, 9, 10..10+t-1), lanes (3..8), waves (10+t..n-1)
//   next layouts : registers (0,1,2, the upper register bits of the previous layout that are not
//                  replaced, the wave bits brought in), lanes (3..8), waves (everything else)
constexpr PlanDesc make_mfma_plan(int n, int t) {
    PlanDesc pl{};
    const int e = 4 + t, v = 3, w = n - 10 - t, c = 1 + t;
    pl.n = n; pl.e = e; pl.v = v; pl.nphase = 0;
    pl.mfma_bits = (1u << 10) - 1u;
    PhaseDesc first{};
    first.rb[0] = 0; first.rb[1] = 1; first.rb[2] = 2; first.rb[3] = 9;
    for (int k = 0; k < t; ++k) first.rb[4 + k] = 10 + k;
    first.stages = 0;
    for (int k = 0; k < t; ++k) first.stages |= 1u << (10 + k);
    fill_thread_bits(first, n, e);
    pl.ph[pl.nphase++] = first;
    PhaseDesc prev = first;
    for (int done = 0; done < w;) {
        const int take = (w - done) < c ? (w - done) : c;
        PhaseDesc next{};
        next.rb[0] = 0; next.rb[1] = 1; next.rb[2] = 2;
        int q = 3;
        for (int k = take; k < c; ++k) next.rb[q++] = prev.rb[3 + k];     // kept upper register bits
        next.stages = 0;
        for (int k = 0; k < take; ++k) {
            const int bit = n - w + done + k;
            next.rb[q++] = bit;
            next.stages |= 1u << bit;
        }
        fill_thread_bits(next, n, e);
        pl.ph[pl.nphase++] = next;
        prev = next;
        done += take;
    }
    return pl;
}

// tiles per wave (log2) used for a given log2 d.  At d = 2^14 the forward pass takes four tiles per
// wave (64 values per thread, one exchange), the backward pass two (32 values per thread, two
// exchanges): its per-thread state (alpha', dalpha, dbeta) does not fit next to 64 values.
constexpr int mfma_log_tiles(int logd, bool backward) {
    return logd <= 10 ? 0 : ((logd >= 14 && !backward) ? 2 : 1);
}

// For a few tokens per launch (one token group per workgroup): as few tiles per wave as the schedule
// allows, i.e. as many waves per token, which shortens each wave's chain of dependent instructions.
constexpr int mfma_log_tiles_few(int logd) { return logd <= 12 ? 0 : 1; }

// ---- the wave schedule: a token inside one wave (or two, four), hardly any LDS in the transform -----
//
// A token lies on 2^L lanes of one wave (L = n - e <= 6), 2^e values per lane, and a wave holds
// 2^(6-L) tokens; a token that does not fit (n - e = 6 + w) lies on 2^w whole waves.  Element bits
// v .. v+5 are the lane bits, v+6 .. v+5+w the wave bits, the rest register bits:
//   lane positions 0..3 : butterflied in place, the partner's value read through a DPP operand;
//   lane positions 4, 5 : exchanged with the top register bits (one permlane16/32 swap per register
//                         pair) and then butterflied in registers.  The second layout is therefore
//                         the first one with element bits v+4 <-> n-1 (and v+5 <-> n-2) exchanged;
//   wave bits           : exchanged with register bits v, v+1 through LDS, the only re-deal there is.
// The stages run in the order 0 .. v+3, v+6 .. n-1, v+5, v+4 whatever e is (w = 0), so that two
// kernels with different values per lane give the same bits.
constexpr PlanDesc make_wave_plan(int n, int e, int v) {
    PlanDesc pl{};
    const int T = n - e, L = T < 6 ? T : 6, w = T - L;
    pl.n = n; pl.e = e; pl.v = v; pl.nphase = 1; pl.mfma_bits = 0; pl.lane_bits = 0;
    for (int k = 0; k < L && k < 4; ++k) pl.lane_bits |= 1u << (v + k);
    PhaseDesc first{};
    for (int q = 0; q < v; ++q) first.rb[q] = q;
    for (int q = v; q < e; ++q) first.rb[q] = n - (e - v) + (q - v);
    first.stages = reg_mask(first, e);
    fill_thread_bits(first, n, e);
    pl.ph[0] = first;
    unsigned done = first.stages;
    if (L > 4) {
        PhaseDesc next = first;
        for (int k = 4; k < L; ++k) {
            next.rb[e - 1 - (k - 4)] = first.tb[k];
            next.tb[k] = first.rb[e - 1 - (k - 4)];
        }
        next.stages = reg_mask(next, e) & ~done;
        done |= next.stages;
        pl.ph[pl.nphase++] = next;
    }
    if (w > 0) {
        PhaseDesc last = pl.ph[pl.nphase - 1];
        for (int k = 0; k < w; ++k) {
            const int lane = last.rb[v + k];
            last.rb[v + k] = last.tb[6 + k];
            last.tb[6 + k] = lane;
        }
        last.stages = reg_mask(last, e) & ~done;
        pl.ph[pl.nphase++] = last;
    }
    return pl;
}

// Lane <-> element bits at lane positions 0..3.  The DPP operands at hand pair lane l with l ^ 1,
// l ^ 2, l ^ 7 and l ^ 8; with c the element bits of a lane, l = c0*1 ^ c1*2 ^ c2*7 ^ c3*8.
constexpr unsigned wave_lane_to_bits(unsigned l, int L) {
    return L >= 3 ? l ^ ((l >> 2) & 1u) ^ ((l >> 1) & 2u) : l;
}

// The layout needs a register bit above the vector bits for every lane position above 3, and for
// every wave bit.
constexpr bool wave_fits(int n, int e, int v) {
    const int T = n - e, L = T < 6 ? T : 6, w = T - L;
    return T >= 0 && w <= 2 && e <= kMaxRegBits && e >= v && (L <= 4 || e - v >= L - 4) && e - v >= w;
}
// log2(values per lane): at least eight lanes per token where the vectors allow it (128 contiguous
// bytes), 16 values if the token then fits a wave, 32 on up to four waves beyond that (64 for the
// widest bfloat16 row).
constexpr int wave_log_e(int n, int v) {
    int e = n - 3 < 4 ? n - 3 : 4;
    if (e < v) e = v;
    if (n - e > 6) ++e;
    while (!wave_fits(n, e, v)) ++e;
    return e;
}

// ---- rows of 12 * 2^m elements (bfloat16, m = 6..10) --------------------------------------------
//
// Element e = b * 2^m + r, block b = 0..11.  H_raw = P12 (x) S_{2^m}: the order-12 matrix across the
// blocks, Sylvester stages on the bits of r.  A wave holds 1536 elements, three 16-byte vectors (8
// consecutive elements, r bits 0..2) per lane and no empty place:
//   vectors 0, 1: rows of blocks 0..7,   lane = b0 b1 r3 b2 r4 r5 (bit 0 first), the vector's number is "pair"
//   vector  2   : rows of blocks 8..11,  lane = b0 b1 r3 pair r4 r5
// "pair" is r6, or for m = 6 the second of the wave's two tokens.  Bits r7.. are the wave's number within
// the token.  Two matrix-core rounds of 16x16x32 products transform r0..r5 and the blocks in place:
//   round 1 contracts the 32 values (r0 r1 r2 r4 r5) of every row, 16 rows a product: rows change places
//           with columns, and the rows' index (block, r3) is then in the registers and lane bits 4, 5;
//   round 2 contracts the 24 values (block, r3): a row's operand is 16 values of vector 0 or 1 and its half
//           of vector 2's, the other half multiplied by zeros; results of blocks 8..11 of both halves are
//           accumulated side by side into vector 2, for m > 6 with the stage on r6 between them done by the
//           signs of that product.
// So the products unpack and pack the odd quarter: no vector or lane is idle anywhere else, where a row
// padded to 16 blocks left a quarter of the lanes and of every instruction's work empty.
constexpr int twelve_wave_bits(int m) { return m > 7 ? m - 7 : 0; }      // log2(waves per token)
constexpr unsigned twelve_block(unsigned lane, int vec) {
    return (lane & 3u) | (vec == 2 ? 8u : ((lane >> 3) & 1u) << 2);
}
constexpr unsigned twelve_pair(unsigned lane, int vec) { return vec == 2 ? (lane >> 3) & 1u : (unsigned)vec; }
// First element of the vector a lane holds in the first layout (m = 6: within its own token).
constexpr unsigned twelve_elem(unsigned lane, unsigned wave, int vec, int m) {
    return (twelve_block(lane, vec) << m) | (((lane >> 2) & 1u) << 3) | ((lane >> 4) << 4) |
           (m > 6 ? twelve_pair(lane, vec) << 6 : 0u) | (wave << 7);
}
// The last layout (tokens of several waves): wave bits k = 0, 1, 2 exchanged with lane positions 0, 1, 3,
// where their stages run through DPP operands.  Its own inverse.
constexpr int twelve_lane_pos(int k) { return k < 2 ? k : 3; }
struct LaneWave { unsigned lane, wave; };
constexpr LaneWave twelve_swap(unsigned lane, unsigned wave, int w) {
    LaneWave s{lane, wave};
    for (int k = 0; k < w; ++k) {
        const int p = twelve_lane_pos(k);
        const unsigned x = ((lane >> p) ^ (wave >> k)) & 1u;
        s.lane ^= x << p;
        s.wave ^= x << k;
    }
    return s;
}
// Exchange region of a token: one block of 64 16-byte places per (four registers, wave), and 16 bytes more, so
// that the lanes of a scattered access differ in their banks.  Every thread puts in the order of one layout and
// gets in the order of the other.
constexpr unsigned kTwelveBlockWords = 64u * 4u + 4u;
constexpr unsigned twelve_place(unsigned lane, unsigned wave) { return wave * kTwelveBlockWords + lane * 4u; }
constexpr unsigned twelve_exchange_words(int w) { return 6u * (kTwelveBlockWords << w); }
// Registers I .. I+3 of a thread.
constexpr unsigned twelve_exchange_reg(int I, int w) { return (I / 4) * (kTwelveBlockWords << w); }
// Column sums in LDS: 16 words more after every block, for the same reason.
constexpr unsigned twelve_column(unsigned e, int m) { return e + 16u * (e >> m); }

// P12: symmetric order-12 Hadamard matrix (Paley's second construction over GF(5)), first row and
// column +1.  Bit c of row r's mask is set where P12[r][c] = -1.
// The twelve masks 0x000 0x556 0x3ca 0x96c 0xf22 0x5b8 0xc8e 0x6e4 0x23e 0xb94 0x8f2 0xe58 are packed
// five to a 64-bit word and picked out with shifts: on the GPU a table indexed at run time would be
// a memory load, and the kernels build their matrix operand from this on every launch.
constexpr unsigned paley12_minus_row(unsigned r) {
    const unsigned long long word = r < 5u ? 0x0f2296c3ca556000ull : (r < 10u ? 0x0b9423e6e4c8e5b8ull : 0xe588f2ull);
    const unsigned k = r < 5u ? r : (r < 10u ? r - 5u : r - 10u);
    return (unsigned)(word >> (12u * k)) & 0xfffu;
}
constexpr bool paley12_packing_matches() {
    constexpr unsigned rows[12] = {0x000, 0x556, 0x3ca, 0x96c, 0xf22, 0x5b8,
                                   0xc8e, 0x6e4, 0x23e, 0xb94, 0x8f2, 0xe58};
    for (unsigned r = 0; r < 12u; ++r)
        if (paley12_minus_row(r) != rows[r]) return false;
    return true;
}
static_assert(paley12_packing_matches(), "packed P12 masks");
// Operand words of the rounds' matrices for a lane: bf16 pairs, elements 2*word and 2*word + 1 of the lane's 8
// (matrix row k = 8 * (lane / 16) + element, column j = lane % 16).  Built on every launch, so in few operations.
constexpr unsigned kBothSigns = 0x80008000u;
// Round 1, output half `half`: column j stands for (r0 r1 | r4 r5) = (j0 j1 | j2 j3), half for r2, row k for
// (r0 r1 r2 r4 r5); the sign is the parity of row & column.
constexpr unsigned twelve_round1_word(unsigned lane, int half, int word) {
    const unsigned j = lane & 15u, both = (j >> 2) & (lane >> 4), base = (both ^ (both >> 1)) & 1u;      // r4, r5
    const unsigned first = 0x3F803F80u | (base << 15) | ((base ^ j) << 31);                             // r0: element 1
    const unsigned r1 = (word & 1) && (j & 2u) ? kBothSigns : 0u;
    return first ^ r1 ^ ((word & 2) && half ? kBothSigns : 0u);
}
// Round 2 on the rows of `pair`, results for vectors 0 / 1 (shared = false) or 2.  Matrix rows: the four registers
// of vector `pair` and of vector 2, in this order for pair 0 and in the other for pair 1 (the registers then lie
// side by side as 0, 2, 1 and both operands are slices of them); lanes of vector 2 that belong to the other
// pair are zero.  Columns of vector 2 that do are zero for m = 6, and else hold the stage on r6: minus where both
// the row and the column are of pair 1.
constexpr unsigned twelve_round2_word(unsigned lane, int pair, bool shared, int word, int m) {
    const unsigned j = lane & 15u, g = lane >> 4;
    const bool second = (word >> 1) != pair;                     // registers of vector 2
    const unsigned wrong_column = shared && m == 6 ? (j >> 3) ^ (unsigned)pair : 0u;
    const unsigned wrong_row = second ? (g >> 1) ^ (unsigned)pair : 0u;
    const unsigned keep = ((wrong_column | wrong_row) & 1u) - 1u;               // all ones or none
    const unsigned flip = (g & (j >> 2) & 1u) ^ (shared && pair && m > 6 ? (j >> 3) & 1u : 0u);      // r3, r6
    const unsigned minus = paley12_minus_row(twelve_block(j, shared ? 2 : 0)) ^ ((0u - flip) & 0xfffu);
    const unsigned at = (second ? minus >> 8 : minus >> (4u * (g >> 1))) >> (2 * (word & 1));
    return (0x3F803F80u | (((at << 15) | (at << 30)) & kBothSigns)) & keep;
}

// ---- LDS address maps -------------------------------------------------------------------------
// Both are linear in the bits of i (phys(a | b) = phys(a) + phys(b) for disjoint a, b) and keep four
// consecutive elements in one aligned 16-byte group.

// Wave schedule: at float32, where the exchange between waves serves d = 4096 and 8192, lane l's 16 bytes
// follow lane l-1's in every layout and the plain index is free of bank conflicts.  (bfloat16 rows of several
// waves, which run here only when the matrix-core schedule is switched off, have a lane stride of 32 bytes
// and do conflict.)
constexpr unsigned lds_phys_plain(unsigned i) { return i; }

// Matrix-core schedule: both layouts give lane l the 8 elements starting at 8*l (+ multiples of
// 512) as two 16-byte accesses.  Moving element bit 2 above the six lane bits makes each of those
// accesses contiguous across the wave (lane stride 16 bytes): no padding, no bank conflicts.
constexpr unsigned lds_phys_rot(unsigned i) {
    return (i & 3u) | (((i >> 3) & 63u) << 2) | (((i >> 2) & 1u) << 8) | (i & ~511u);
}

}  // namespace wht
