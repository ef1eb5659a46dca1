// Multicanonical Metropolis sweeps (Sec. II, Eq. (2)) with per-attempt minimum and
// round-trip bookkeeping (Sec. III) and per-sweep histograms.
//
// Mapping: one lane = one walker; one wave = 64 walkers of one realization, which
// share its couplings (wave-uniform, scalar registers) and its threshold table
// (LDS). A walker's lattice stays in VGPRs for the whole launch, bit-packed by
// colour and plane (see nfm_internal.hpp).
//
// What bounds it (MI355X, 2.4 GHz): instruction issue. With several waves per SIMD a vector
// instruction takes 4.2 cycles of the SIMD (adds, ands, ors, xors of vector registers and right
// shifts 2.3), whatever it does: the 32 x 32 -> 64 bit product costs no more than a compare. A wave
// alone on its SIMD issues one instruction of any kind per 4.5 (4-byte encodings) or 5.5 cycles
// (8-byte). So an attempt is written for its instruction count: 19.1 vector instructions at L = 8
// (16 products and 18 xors for four random words, 6 for the decision, 1 for the running extremes,
// the rest block preparation), 14.4 in the tempering form. Measured, after per-site gathering products
// and a plane index resolved by compares and selects: L = 8 x 4096 realizations 81.5 -> 72.5 us per
// sweep (power-law rounds), tempering 70.9 -> 53.9 us.
//
// The sweep order is checkerboard: all sites of colour 0, then colour 1. The
// neighbours of a site all have the other colour, so at the start of each
// (colour, plane) block the number u of unsatisfied bonds of every site of the
// block is fixed; it is computed for the whole block at once with word-parallel
// bit operations (six flag strings and a bit-sliced adder). The attempts then run
// one after the other, since each acceptance reads the walker's current energy.
//
// Files: this header holds a wave's work (sweep_wave, generate_words); sweep_size.hip the kernels
// of one lattice size, sweep_queue.hip the persistent kernels over mixed sizes, sweep.hip the
// choice between them.
//
// Kernel forms: k_sweeps (one wave per workgroup; compact or expanded table, speculative or
// plain, tempering), k_sweeps_ws (the sampling wave plus a generator wave that supplies its
// random words through LDS) and k_sweeps_queue (persistent, over a batch of mixed sizes). All
// forms draw the same words for the same attempts, so their results are identical.
#pragma once
#include <type_traits>
#include <utility>

#include "kernels.hpp"
#include "philox.hpp"

namespace nfm {

// f(0), ..., f(N - 1) with each index a compile-time constant (operands of the instruction sequences
// below are immediates that depend on it).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Blocks. The sites of one colour are taken a block at a time: a plane, or at L = 4, whose planes
// hold eight sites of a colour, all four planes, so that a block fills a 32-bit word. The plane
// strings of a block lie one after the other in its string.
template <int L>
struct Geo {
  static constexpr int F = field_bits(L);
  static constexpr int NWP = plane_words(L);   // words of a block's string
  static constexpr int H = L / 2;              // sites of one colour per row
  static constexpr int N = L * L * L;
  static constexpr int ZB = L == 4 ? 4 : 1;    // planes per block
  static constexpr int LB = L / ZB;            // blocks per colour
  static constexpr int QP = L * L / 2;         // sites of one colour per plane
  static constexpr int Q = ZB * QP;            // sites per block
  static constexpr int NGP = (QP + 3) / 4;     // generator groups (four sites) per plane
  static constexpr int NG = ZB * NGP;          // per block
  static constexpr int PB = L * F;             // bits of a plane string
  static constexpr int BITS = ZB * PB;         // bits of a block string
  static_assert(ZB == 1 || (QP % 4 == 0 && BITS == 32), "blocks of several planes: whole groups, one word");

  // Masks of one string word. A word holds whole rows, an even number of them where a string has
  // several, so one mask serves every word (bits beyond the string are zero in the spins and
  // couplings and stay zero): bits [lo, lo + width) of the field of every row y with
  // y % 2 == parity (parity 2: of every row).
  static constexpr uint32_t fields(int lo, int width, int parity = 2) {
    uint32_t m = 0;
    for (int y = 0; y < BITS / F && (y + 1) * F <= 32; ++y)
      for (int b = lo; b < lo + width; ++b)
        if (parity == 2 || y % 2 == parity) m |= 1u << (y * F + b);
    return m;
  }
  // bits [lo, lo + width) of every plane string of a one-word block
  static constexpr uint32_t plane_bits(int lo, int width) {
    uint32_t m = 0;
    for (int z = 0; z < ZB; ++z)
      for (int b = lo; b < lo + width; ++b) m |= 1u << (z * PB + b);
    return m;
  }
};

// Three-input bit operations as one instruction each: exclusive or, majority.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Rows y + 1 and y - 1 of every field of a plane-colour string (periodic).
template <int L>
__device__ __forceinline__ void shift_rows(const uint32_t* O, uint32_t* up, uint32_t* dn) {
  using G = Geo<L>;
  constexpr int F = G::F, NWP = G::NWP, TOP = G::BITS - 32 * (NWP - 1);   // bits of the last word
  if constexpr (G::ZB > 1) {
    up[0] = ((O[0] >> F) & G::plane_bits(0, G::PB - F)) | ((O[0] << (G::PB - F)) & G::plane_bits(G::PB - F, F));
    dn[0] = ((O[0] << F) & G::plane_bits(F, G::PB - F)) | ((O[0] >> (G::PB - F)) & G::plane_bits(0, F));
  } else if constexpr (NWP == 1) {
    if constexpr (TOP == 32) {
      up[0] = __builtin_amdgcn_alignbit(O[0], O[0], F);
      dn[0] = __builtin_amdgcn_alignbit(O[0], O[0], 32 - F);
    } else {
      constexpr uint32_t ALL = (1u << (TOP & 31)) - 1u;
      up[0] = ((O[0] >> F) | (O[0] << (TOP - F))) & ALL;
      dn[0] = ((O[0] << F) | (O[0] >> (TOP - F))) & ALL;
    }
  } else {
#pragma unroll
    for (int w = 0; w + 1 < NWP; ++w) {
      up[w] = __builtin_amdgcn_alignbit(O[w + 1], O[w], F);
      dn[w + 1] = __builtin_amdgcn_alignbit(O[w + 1], O[w], 32 - F);
    }
    if constexpr (TOP == 32) {
      up[NWP - 1] = __builtin_amdgcn_alignbit(O[0], O[NWP - 1], F);
      dn[0] = __builtin_amdgcn_alignbit(O[0], O[NWP - 1], 32 - F);
    } else {
      constexpr uint32_t ALL = (1u << (TOP & 31)) - 1u;
      up[NWP - 1] = (O[NWP - 1] >> F) | ((O[0] << (TOP - F)) & ALL);
      dn[0] = (O[0] << F) | (O[NWP - 1] >> (TOP - F));
      dn[NWP - 1] &= ALL;
    }
  }
}

__device__ __forceinline__ int floor_div4(int a) { return a >= 0 ? a / 4 : -((-a + 3) / 4); }
__device__ __forceinline__ int ceil_div4(int a) { return -floor_div4(-a); }

// Bookkeeping window of the round-trip state: while lo <= B <= hi an attempt cannot change it
// (B = (k - row0) * 32 for level k). The walker's minimum and new-minimum flag do not depend on the
// order of the attempts, so they are taken from each group's lowest B instead; only a group in
// which some walker reached the bound its state waits for is replayed in order.
struct Window {
  int lo, hi;
};

// Groups of four attempts between two window checks of an L x L x L lattice. Each check costs the
// extremes of the levels since the last one, a compare and a branch, and a replay covers every
// attempt since then: a lone wave on its SIMD (the largest lattices) gains from longer intervals,
// several waves per SIMD whose walkers often reach a bound (small lattices, first rounds) from
// shorter ones. L = 12 with 8 groups instead of 4 gains 1 to 3 % under settled tables (512 waves alone
// 88.4 -> 86.8 us per sweep) and loses in the first rounds (1446 waves, 48 sweeps: 7.7 -> 8.1 ms).
template <int L>
constexpr int check_groups() { return L >= 10 ? 4 : 2; }

__device__ __forceinline__ Window make_window(int state, int Bbot, int Btop) {
  constexpr int INF = 1 << 29;
  Window w;
  w.lo = (state == 1) ? Bbot + 32 : -INF;   // at or after the top: waiting for the bottom
  w.hi = (state == 1) ? INF : Btop - 32;    // before the first top, or after a bottom: for the top
  return w;
}

// Exact round-trip bookkeeping of one attempt (Sec. III): E >= e_top <=> B >= Btop and
// E <= e_bot <=> B <= Bbot.
struct Track {
  int Bmin, state, newmin;   // Bmin, newmin: folded from the running minimum (see sweep_wave)
  uint32_t trips;
  uint64_t t_first, t_last;
};

// SELECTS: without branches, for L = 2, where in most replays some lane takes each branch (1.73 us per
// sweep with branches, 1.58 without); beyond, a replay is for one lane or two, and the branches that no
// lane takes are skipped (L = 8 x 4096 production of 500 sweeps: 37.6 ms with branches, 38.0 without).
template <bool SELECTS>
__device__ __forceinline__ void track_attempt(Track& tr, int B, uint64_t tau, int Bbot, int Btop) {
  if constexpr (SELECTS) {
    const bool top = B >= Btop;
    const bool trip = top & (tr.state == 2), first = top & (tr.state == 0);
    const bool bottom = (B <= Bbot) & (tr.state == 1);
    tr.trips += trip ? 1u : 0u;
    tr.t_last = trip ? tau : tr.t_last;
    tr.t_first = first ? tau : tr.t_first;
    tr.state = top ? 1 : bottom ? 2 : tr.state;
  } else if (B >= Btop) {
    if (tr.state == 2) {
      tr.trips += 1;
      tr.t_last = tau;
    }
    if (tr.state == 0) tr.t_first = tau;
    tr.state = 1;
  } else if (B <= Bbot && tr.state == 1) {
    tr.state = 2;
  }
}

// Round-trip bookkeeping on energies, applied once per sweep (parallel tempering: a
// configuration's energy is examined after each Metropolis phase).
struct TrackE {
  int Emin, state, newmin;
  uint32_t trips;
  uint64_t t_first, t_last;
};

__device__ __forceinline__ void track_energy(TrackE& tr, int E, uint64_t tau, int e_bot, int e_top) {
  tr.Emin = min(tr.Emin, E);
  tr.newmin = E < e_bot ? 1 : tr.newmin;
  const bool top = E >= e_top;
  const bool trip = top & (tr.state == 2), first = top & (tr.state == 0);
  const bool bottom = (E <= e_bot) & (tr.state == 1);
  tr.trips += trip ? 1u : 0u;
  tr.t_last = trip ? tau : tr.t_last;
  tr.t_first = first ? tau : tr.t_first;
  tr.state = top ? 1 : bottom ? 2 : tr.state;
}

__device__ __forceinline__ int lds_load_i32(uint32_t byte_addr) {
  return *(const __attribute__((address_space(3))) int*)(uintptr_t)byte_addr;
}
__device__ __forceinline__ uint32_t read_row(uint32_t byte_addr) {
  return *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)byte_addr;
}
__device__ __forceinline__ void lds_store_i32(uint32_t byte_addr, int v) {
  *(__attribute__((address_space(3))) int*)(uintptr_t)byte_addr = v;
}
typedef uint32_t lds_v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 lds_load_u32x4(uint32_t byte_addr) {
  const lds_v4u q = *(const __attribute__((address_space(3))) lds_v4u*)(uintptr_t)byte_addr;
  return u32x4{{q.x, q.y, q.z, q.w}};
}
__device__ __forceinline__ void lds_store_u32x4(uint32_t byte_addr, const u32x4& w) {
  const lds_v4u q = {w.v[0], w.v[1], w.v[2], w.v[3]};
  *(__attribute__((address_space(3))) lds_v4u*)(uintptr_t)byte_addr = q;
}

// Warp-specialized form (expanded table only): a workgroup of two waves, the sampling wave and
// a generator wave that computes the random words of the sampling wave's walkers two blocks
// ahead into a ring of three block slots in LDS (16 bytes per walker and group of four sites),
// after the sampling wave's table, couplings and histogram. Both waves meet at one barrier per
// block. The generator's work leaves the sampling wave's instruction stream, and the two waves
// share a SIMD's issue slots where one wave per SIMD would leave them idle.
template <int L>
__host__ __device__ constexpr uint32_t ws_slot_bytes() {
  return (uint32_t)Geo<L>::NG * 64u * 16u;
}
__host__ __device__ inline uint32_t ws_ring_base(int K, int jk_words_L, int hist_n) {
  return ((uint32_t)K * 32u + 4u * (uint32_t)jk_words_L + 4u * (uint32_t)hist_n + 15u) & ~15u;
}

// Byte form of a block's level steps. The steps of four sites sit in the bytes of one
// word: D holds m << 5 (sign-extended: the level change 32 m), A holds 4 (m & 7), the entry's
// offset in its table row. The sub-dword operand forms read a byte inside the add and the or
// that need it, so a site costs no instruction to gather its step: what is left per site is its
// share of the expansion from bit planes to bytes (35 instructions for 32 sites, most of them
// shifts and ands, which issue at twice the rate of multiplies and three-operand forms).
__device__ __forceinline__ int add_step(int B, uint32_t D, int byte) { return B + (int)(int8_t)(D >> (8 * byte)); }
template <int byte>
__device__ __forceinline__ uint32_t or_entry(uint32_t A, int R) {   // table address: row R, entry in A's byte
  uint32_t an;
  asm("v_or_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_%3"
      : "=v"(an)
      : "v"(R), "v"(A), "n"(byte));
  return an;
}

// Acceptance of one attempt and its effect on the state, as one instruction sequence: the
// comparison r <= th' of the random word with the on-chip threshold (th' = thr - 1, or 0 for
// thr = 0, or 2^32 - 1 for always, so that r <= th' <=> thr = 2^32 - 1 or r < max(thr, 1)) sets VCC, which then selects the new level and is shifted into the flip word F
// (F = 2F + accepted). The two instructions between the comparison and the first reader of
// VCC are the distance the hardware needs between a VALU write of VCC and a VALU read of it;
// they are the level after acceptance (B, the row offset of the level, 32 per level, plus byte
// cb of D) and, where two levels wait for it, a step of the running extremes (EXT 1: minimum,
// 2: maximum of x and the levels t0, t1; 0: none).
// an: byte nb of A, the next site's entry offset; addr receives its table address.
// XT: every level has its own row on chip, so the row is the level and needs no clamp.
#define NFM_DECIDE(MID, CLAMP, ROW)                                                                  \
  asm volatile("v_cmp_le_u32_e32 vcc, %[rc], %[th]\n\t"                                              \
               "v_add_u32_sdwa %[Bacc], %[B], sext(%[D]) dst_sel:DWORD dst_unused:UNUSED_PAD "        \
               "src0_sel:DWORD src1_sel:BYTE_%[cb]\n\t" MID "\n\t"                                   \
               "v_cndmask_b32_e32 %[Bn], %[B], %[Bacc], vcc\n\t"                                     \
               "v_addc_co_u32_e32 %[F], vcc, %[F], %[F], vcc\n\t" CLAMP                              \
               "v_or_b32_sdwa %[an], " ROW ", %[A] dst_sel:DWORD dst_unused:UNUSED_PAD "             \
               "src0_sel:DWORD src1_sel:BYTE_%[nb]"                                                 \
               : [Bn] "=&v"(Bn), [Rn] "=&v"(Rn), [F] "+&v"(F), [Bacc] "=&v"(Bacc), [an] "=&v"(an), [x] "+&v"(x) \
               : [rc] "v"(rc), [th] "v"(th), [D] "v"(D), [A] "v"(A), [B] "v"(B), [Bmax] "v"(vBmax),  \
                 [t0] "v"(t0), [t1] "v"(t1), [cb] "n"(cb), [nb] "n"(nb)                              \
               : "vcc")
template <bool XT, int EXT, int cb, int nb>
__device__ __forceinline__ void decide_bytes(uint32_t rc, uint32_t th, uint32_t D, uint32_t A, int vBmax, int t0, int t1,
                                             int& B, int& R, uint32_t& F, uint32_t& addr, int& x) {
  int Bacc, Bn, Rn;
  uint32_t an;
  if constexpr (XT) {
    if constexpr (EXT == 0) NFM_DECIDE("s_nop 0", "", "%[Bn]");
    if constexpr (EXT == 1) NFM_DECIDE("v_min3_i32 %[x], %[x], %[t0], %[t1]", "", "%[Bn]");
    if constexpr (EXT == 2) NFM_DECIDE("v_max3_i32 %[x], %[x], %[t0], %[t1]", "", "%[Bn]");
    R = Bn;
  } else {
    if constexpr (EXT == 0) NFM_DECIDE("s_nop 0", "v_med3_i32 %[Rn], %[Bn], 0, %[Bmax]\n\t", "%[Rn]");
    if constexpr (EXT == 1)
      NFM_DECIDE("v_min3_i32 %[x], %[x], %[t0], %[t1]", "v_med3_i32 %[Rn], %[Bn], 0, %[Bmax]\n\t", "%[Rn]");
    if constexpr (EXT == 2)
      NFM_DECIDE("v_max3_i32 %[x], %[x], %[t0], %[t1]", "v_med3_i32 %[Rn], %[Bn], 0, %[Bmax]\n\t", "%[Rn]");
    R = Rn;
  }
  B = Bn;
  addr = an;
}
#undef NFM_DECIDE

// Tempering: the decisions of a group of up to four sites, q0 .. q0 + 3 of a block, shifted into F in
// site order (a zero for each bit of a field beyond its row). The comparisons come first, so that
// each acceptance mask is old enough when it is shifted in.
template <int H, int FB, int Q, int q0>
__device__ __forceinline__ void accept_group(const u32x4& rnd, const uint32_t (&th)[4], uint32_t& F) {
  constexpr bool four = q0 + 4 <= Q;
  // the group's only inner row end (rows of three or more sites), -1 if none
  constexpr int e0 = H - 1 - q0 % H;
  constexpr int brk = (FB > H && e0 < 3 && q0 + e0 + 1 < Q) ? e0 : -1;
  if constexpr (four) {
#define NFM_ACC4(S0, S1, S2)                                                                            \
  asm volatile("v_cmp_le_u32_e64 %[a], %[r0], %[t0]\n\tv_cmp_le_u32_e64 %[b], %[r1], %[t1]\n\t"           \
               "v_cmp_le_u32_e64 %[c], %[r2], %[t2]\n\tv_cmp_le_u32_e32 vcc, %[r3], %[t3]\n\t"            \
               "v_addc_co_u32_e64 %[F], %[a], %[F], %[F], %[a]\n\t" S0                                  \
               "v_addc_co_u32_e64 %[F], %[b], %[F], %[F], %[b]\n\t" S1                                  \
               "v_addc_co_u32_e64 %[F], %[c], %[F], %[F], %[c]\n\t" S2                                  \
               "v_addc_co_u32_e32 %[F], vcc, %[F], %[F], vcc"                                           \
               : [F] "+&v"(F), [a] "=&s"(ma), [b] "=&s"(mb), [c] "=&s"(mc)                               \
               : [r0] "v"(rnd.v[0]), [r1] "v"(rnd.v[1]), [r2] "v"(rnd.v[2]), [r3] "v"(rnd.v[3]),         \
                 [t0] "v"(th[0]), [t1] "v"(th[1]), [t2] "v"(th[2]), [t3] "v"(th[3]), [pad] "n"(FB - H)  \
               : "vcc")
    uint64_t ma, mb, mc;
    if constexpr (brk == 0) NFM_ACC4("v_lshlrev_b32_e32 %[F], %[pad], %[F]\n\t", "", "");
    else if constexpr (brk == 1) NFM_ACC4("", "v_lshlrev_b32_e32 %[F], %[pad], %[F]\n\t", "");
    else if constexpr (brk == 2) NFM_ACC4("", "", "v_lshlrev_b32_e32 %[F], %[pad], %[F]\n\t");
    else NFM_ACC4("", "", "");
#undef NFM_ACC4
  } else {
    // the last two sites of a block (L = 2, 6, 10)
    uint64_t ma;
    if constexpr (brk == 0)
      asm volatile("v_cmp_le_u32_e64 %[a], %[r0], %[t0]\n\tv_cmp_le_u32_e32 vcc, %[r1], %[t1]\n\ts_nop 0\n\t"
                   "v_addc_co_u32_e64 %[F], %[a], %[F], %[F], %[a]\n\tv_lshlrev_b32_e32 %[F], %[pad], %[F]\n\t"
                   "v_addc_co_u32_e32 %[F], vcc, %[F], %[F], vcc"
                   : [F] "+&v"(F), [a] "=&s"(ma)
                   : [r0] "v"(rnd.v[0]), [r1] "v"(rnd.v[1]), [t0] "v"(th[0]), [t1] "v"(th[1]), [pad] "n"(FB - H)
                   : "vcc");
    else
      asm volatile("v_cmp_le_u32_e64 %[a], %[r0], %[t0]\n\tv_cmp_le_u32_e32 vcc, %[r1], %[t1]\n\ts_nop 0\n\t"
                   "v_addc_co_u32_e64 %[F], %[a], %[F], %[F], %[a]\n\t"
                   "v_addc_co_u32_e32 %[F], vcc, %[F], %[F], vcc"
                   : [F] "+&v"(F), [a] "=&s"(ma)
                   : [r0] "v"(rnd.v[0]), [r1] "v"(rnd.v[1]), [t0] "v"(th[0]), [t1] "v"(th[1])
                   : "vcc");
  }
  constexpr int qe = four ? q0 + 3 : q0 + 1;   // a row that ends with the group, not with the word
  if constexpr (FB > H && qe % H == H - 1 && qe + 1 < Q && (((qe + 1) / H) * FB) % 32 != 0) F <<= (FB - H);
}

// Paired form: the thresholds of a site for both outcomes of the site before it (rej, acc) are read
// before that one is decided; prev, its acceptance of all lanes, selects. The read is off the chain
// then: two attempts share its latency. Returns this attempt's acceptance. The two instructions after
// the comparison are the distance its mask needs: the shift of prev into F (SHIFT) and a step of the
// running extremes (EXT as in decide_bytes) where there is one to do.
#define NFM_PAIRED(S1, S2, ROW)                                                                     \
  asm volatile("v_cndmask_b32_e64 %[th], %[rej], %[acc], %[prev]\n\tv_cmp_le_u32_e64 %[m], %[rc], %[th]\n\t" S1 \
               "\n\t" S2 "\n\tv_cndmask_b32_e64 %[Bn], %[B], %[Bacc], %[m]" ROW                      \
               : [Bn] "=&v"(Bn), [Rn] "=&v"(Rn), [th] "=&v"(th), [m] "=&s"(m), [F] "+&v"(F), [x] "+&v"(x) \
               : [rc] "v"(rc), [rej] "v"(rej), [acc] "v"(acc), [prev] "s"(prev), [Bacc] "v"(Bacc), [B] "v"(B), \
                 [R] "v"(R), [Racc] "v"(Racc), [t0] "v"(t0), [t1] "v"(t1)                            \
               : "vcc")
#define NFM_PAIRED_EXT(S1, ROW)                                                           \
  do {                                                                                    \
    if constexpr (EXT == 0) NFM_PAIRED(S1, "s_nop 0", ROW);                               \
    if constexpr (EXT == 1) NFM_PAIRED(S1, "v_min3_i32 %[x], %[x], %[t0], %[t1]", ROW);   \
    if constexpr (EXT == 2) NFM_PAIRED(S1, "v_max3_i32 %[x], %[x], %[t0], %[t1]", ROW);   \
  } while (0)
template <bool XT, bool SHIFT, int EXT>
__device__ __forceinline__ uint64_t decide_paired(uint32_t rc, uint32_t rej, uint32_t acc, uint64_t prev, int Bacc,
                                                  int Racc, int t0, int t1, int& B, int& R, uint32_t& F, int& x) {
  int Bn, Rn = 0;
  uint32_t th;
  uint64_t m;
  if constexpr (XT) {   // the row is the level
    if constexpr (SHIFT) NFM_PAIRED_EXT("v_addc_co_u32_e64 %[F], vcc, %[F], %[F], %[prev]", "");
    else NFM_PAIRED_EXT("s_nop 0", "");
    R = Bn;
  } else {              // the row moves with the level (R, Racc: clamped beforehand)
    if constexpr (SHIFT)
      NFM_PAIRED_EXT("v_addc_co_u32_e64 %[F], vcc, %[F], %[F], %[prev]",
                     "\n\tv_cndmask_b32_e64 %[Rn], %[R], %[Racc], %[m]");
    else
      NFM_PAIRED_EXT("s_nop 0", "\n\tv_cndmask_b32_e64 %[Rn], %[R], %[Racc], %[m]");
    R = Rn;
  }
  B = Bn;
  return m;
}
#undef NFM_PAIRED_EXT
#undef NFM_PAIRED
__device__ __forceinline__ void accept_shift(uint64_t mask, uint32_t& F) {
  asm volatile("v_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(F) : "s"(mask) : "vcc");
}

// Exchange threshold of slots (s, s+1) whose energies differ by 4d (Eq. (8)): q^d rounded down
// to a multiple of 2^-32 (0xFFFFFFFF = always, d <= 0), q = exp(4 (beta_{s+1} - beta_s)) given by
// the host, raised to d by binary powering (one FP64 product per bit and per squaring, lowest bit
// first) -- products only, so the host reproduces every value bit for bit.
__device__ __forceinline__ uint32_t pt_swap_threshold(double q, int d) {
  if (d <= 0) return 0xFFFFFFFFu;
  double r = 1.0, b = q;
  while (d > 0) {
    if (d & 1) r = r * b;
    b = b * b;
    d >>= 1;
  }
  return r >= 1.0 ? 0xFFFFFFFFu : (uint32_t)floor(ldexp(r, 32));
}

__device__ __forceinline__ int clamp_row(int B, int Bmax) {
  int R;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(R) : "v"(B), "s"(Bmax));
  return R;
}

// Where the random words come from.
//   kGenVector   all rounds on the vector unit
//   kGenScalar   the uniform half of rounds 0-2 on the scalar unit (free where other waves fill the
//                vector unit meanwhile, an issue slot per instruction where a wave is alone)
//   kGenStaged   that half for all groups of a sweep at once, one group per lane, into LDS at the
//                sweep's start (staged_words): a group then costs one broadcast read
//   kGenWave     a generator wave beside the sampling wave
enum Gen { kGenVector, kGenScalar, kGenStaged, kGenWave };

// kGenStaged, LDS after the histogram: per group of four sites in sweep order {hi(M0 c0) ^ k1_0,
// hi(p) ^ k0_2, lo(p) ^ k0_3, -}, p = M1 n2 of round 2, and two entries more for the reads ahead.
template <int L>
__host__ __device__ constexpr uint32_t staged_bytes() {
  return (uint32_t)(2 * Geo<L>::LB * Geo<L>::NG + 2) * 16u;
}
__host__ __device__ inline uint32_t staged_base(uint32_t hbase, int hist_n) {
  return (hbase + 4u * (uint32_t)hist_n + 15u) & ~15u;
}

// PT = false: multicanonical sweeps; the table row follows the walker's level.
// PT = true: parallel tempering (Sec. II, Eq. (8)); each wave of 64 walkers holds floor(64/M)
// sets of M configurations (lanes g M .. g M + M - 1; the remaining lanes idle at slot 0, outside
// exchanges and bookkeeping), the row is the configuration's temperature slot, and after every
// sweep the slots (s, s+1) with s = t (mod 2) try an exchange. Temperatures are per realization.
// SPEC (multicanonical): the thresholds of both outcomes of an attempt are read before it is decided
// (the speculative forms and, beside a generator wave, the paired one).
// XT (multicanonical; SPEC beside a generator wave only): the table is expanded on chip to one row per level of
// the realization (rows outside the stored range repeat its edge rows, as the clamp would), so
// the row of a level is the level itself and the decision needs no clamp.
template <int L, bool SPEC, bool PT, bool XT, Gen GEN, bool ROLL = (L >= 8)>
__device__ __forceinline__ void sweep_wave(const SweepArgs& A, int wave) {
  using G = Geo<L>;
  constexpr int NWP = G::NWP, Q = G::Q, N = G::N, H = G::H, FB = G::F, ZB = G::ZB, LB = G::LB, NG = G::NG;
  // A block's level steps: bit planes m0, m1, m2 of each string word, expanded to byte words one
  // string word at a time.
  constexpr int NBLK = 3 * NWP;
  constexpr bool kRolled = ROLL && LB > 2;
  constexpr int kZUnroll = kRolled ? 1 : LB;
  constexpr bool WS = GEN == kGenWave, SU = GEN == kGenScalar, PS = GEN == kGenStaged;
  static_assert(!(PT && SPEC), "the tempering row does not depend on the decision");
  static_assert(!(PT && (PS || WS)), "the staged words and the generator wave serve the multicanonical form");
  static_assert(!(XT && PT), "the expanded table is for the multicanonical form");
  static_assert(!(XT && SPEC) || WS, "the speculative form with the expanded table runs beside a generator wave");
  static_assert(!WS || XT, "the generator wave serves the expanded-table form");
  int lane = (int)(threadIdx.x & 63u);
  // In the persistent kernel every item starts from opaque values: what follows from them would
  // otherwise be computed once, before the item loop, for all sizes and kept in registers.
  if constexpr (ROLL) asm volatile("" : "+v"(lane));
  const int r = A.wave_real[wave];
  const int wl = A.wave_wl[wave] + lane;
  const RealInfo& RI = A.reals[r];
  const int e_base = RI.e_base, walkers = RI.walkers, K = RI.K;
  const int row0 = (PT || XT) ? 0 : RI.row0, rows = PT ? A.pt_M : (XT ? K : RI.rows);
  const int e_bot = RI.e_bot, e_top = RI.e_top;
  const uint32_t real_id = RI.real_id;
  const int64_t gw = RI.walker_off + wl;

  // LDS (the kernel's only LDS, so it starts at address 0):
  //   [0, rows*32)        threshold table, each row permuted from u-order to m-order: entry j
  //                       holds the threshold of the step m = j (j < 4) or m = j - 8 (j > 4),
  //                       as th' of the decision (r <= th');
  //   tempering only      energies by slot, exchange decisions, exchange counters (3 x 256 B);
  //   then                the realization's couplings in the kernel layout;
  //   multicanonical only the launch's histogram over a window of levels around the table rows
  //   (all K levels where that costs no occupancy: walkers leave the rows in both directions,
  //   above the top where W is constant and below the lowest known level in the first rounds),
  //   flushed to HBM once at the end; levels outside the window are counted in HBM directly.
  const uint32_t sE = (uint32_t)rows * 32u, sD = sE + 256u, sAcc = sD + 256u;
  const uint32_t jbase = PT ? sAcc + 256u : sE;
  const uint32_t hbase = jbase + 4u * (uint32_t)jk_words(L);
  const int hlo = max(0, row0 - A.hist_margin), hn = A.hist_n;
  {
    const uint32_t* gt = A.tables + RI.table_off;
    for (int e = lane; e < rows * 8; e += 64) {
      const int jj = e & 7;
      const int u = jj < 4 ? 3 - jj : (jj == 4 ? 7 : 11 - jj);
      int gr = e >> 3;   // row of the stored table
      if constexpr (XT) gr = min(max(gr - RI.row0, 0), RI.rows - 1);
      const uint32_t v = PT ? A.pt_metro[((int64_t)r * kMaxReplicas + gr) * 8 + u] : gt[gr * 8 + u];
      const uint32_t vp = (v == 0xFFFFFFFFu) ? v : (v ? v - 1u : 0u);
      *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)(e * 4) = vp;
    }
    const uint32_t* jg = A.jk + RI.jk_off;
    if constexpr (ZB == 1) {
      for (int e = lane; e < jk_words(L); e += 64) lds_store_i32(jbase + 4u * (uint32_t)e, (int)jg[e]);
    } else {
      for (int e = lane; e < 12; e += 64) {   // (colour, bond): the plane strings of the block
        uint32_t v = 0;
        for (int z = 0; z < ZB; ++z) v |= jg[(e / 6 * L + z) * 6 + e % 6] << (z * G::PB);
        lds_store_i32(jbase + 4u * (uint32_t)e, (int)v);
      }
    }
  }
  if constexpr (PT) {
    lds_store_i32(sAcc + 4u * (uint32_t)lane, 0);
  } else {
    for (int e = lane; e < hn; e += 64) lds_store_i32(hbase + 4u * (uint32_t)e, 0);
  }
  __syncthreads();

  // walker state -> registers. One array per (colour, word) so that each stays small
  // enough to live in VGPRs under a dynamic plane index.
  // (Arrays of more than eight elements: a dynamic index into eight or fewer compiles to a chain
  // of compares and selects, about 50 a block at L = 8, into more to an indexed register move.)
  constexpr int LA = (kRolled && LB <= 8) ? 9 : LB;
  uint32_t a00[LA], a01[LA], a02[LA], a10[LA], a11[LA], a12[LA];
  auto lat = [&](int c, int w) -> uint32_t* {
    return c == 0 ? (w == 0 ? a00 : w == 1 ? a01 : a02) : (w == 0 ? a10 : w == 1 ? a11 : a12);
  };
  static_assert(NWP <= 3, "block strings of at most 3 words");
  {
    const uint32_t* sp = A.spins + RI.spin_off + wl;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int w = 0; w < NWP; ++w)
#pragma unroll
        for (int b = 0; b < LB; ++b) {
          uint32_t v = 0;
#pragma unroll
          for (int z = 0; z < ZB; ++z)
            v |= sp[(int64_t)((c * L + b * ZB + z) * NWP + w) * walkers] << (ZB > 1 ? z * G::PB : 0);
          lat(c, w)[b] = v;
        }
  }
  // tempering: this lane's set within the wave (floor(lane / M)), its first lane, its index in
  // the realization; lanes beyond the last whole set idle
  uint32_t pt_base = 0, pt_set = 0;
  bool pt_active = false;
  if constexpr (PT) {
    const uint32_t sw = __umulhi((uint32_t)lane, A.pt_minv);
    pt_active = sw < (uint32_t)A.pt_spw;
    pt_base = sw * (uint32_t)A.pt_M;
    pt_set = (uint32_t)(A.wave_wl[wave] >> 6) * (uint32_t)A.pt_spw + sw;
    asm volatile("" : "+v"(pt_base), "+v"(pt_set));
  }
  const int E0 = A.ws.E[gw];
  int E = E0;        // tempering: the energy, updated per attempt
  int slot = 0;      // tempering: the temperature slot
  int B;
  Track tr;
  TrackE te;
  if constexpr (PT) {
    slot = A.pt_slot[gw];
    B = slot * 32;
    te.Emin = A.ws.E_min[gw];
    te.state = A.ws.rt_state[gw];
    te.newmin = A.ws.new_min[gw];
    te.trips = 0;
    te.t_first = A.ws.t_first[gw];
    te.t_last = A.ws.t_last[gw];
  } else {
    B = ((E0 - e_base) / 4 - row0) * 32;
    tr.Bmin = ((A.ws.E_min[gw] - e_base) / 4 - row0) * 32;
    tr.state = A.ws.rt_state[gw];
    tr.newmin = A.ws.new_min[gw];
    tr.trips = 0;
    tr.t_first = A.ws.t_first[gw];
    tr.t_last = A.ws.t_last[gw];
  }

  const int Bmax = (rows - 1) * 32;
  const int Btop = (ceil_div4(e_top - e_base) - row0) * 32;    // E >= e_top  <=> B >= Btop
  const int Bbot = (floor_div4(e_bot - e_base) - row0) * 32;   // E <= e_bot  <=> B <= Bbot
  const int Bnm = (ceil_div4(e_bot - e_base) - 1 - row0) * 32; // E <  e_bot  <=> B <= Bnm
  Window win;
  if constexpr (!PT) win = make_window(tr.state, Bbot, Btop);
  int R = clamp_row(B, Bmax);   // the table row in use: B clamped to the stored rows
  int vBmax;                    // Bmax in a vector register (an operand of the decision sequence)
  asm volatile("v_mov_b32 %0, %1" : "=v"(vBmax) : "s"(Bmax));

  uint32_t key0 = (uint32_t)A.walker_seed, key1 = (uint32_t)(A.walker_seed >> 32);
  if constexpr (ROLL) asm volatile("" : "+s"(key0), "+s"(key1));
  // Round keys in VGPRs: uniform values, but keeping them out of the scalar file leaves room for
  // the per-plane coupling words and constants without spilling scalar registers. (Not needed
  // when a generator wave supplies the words.)
  PhiloxKeysV kv;
  if constexpr (!WS) kv = philox_round_keys_v<SU || PS ? 3 : 0>(key0, key1);
  uint32_t ctr3 = ((uint32_t)wl << 8) | (PT ? kTagPT : kTagAcc);

  // Level steps of the sites of block (c, z) from the other colour's spins and the couplings: the
  // three bits of m = 3 - u as bit planes (V[3w + k] = bit k of string word w). The other colour does
  // not change while colour c is updated, so the block after the current one is prepared while the
  // current one runs.
  // Own: the block's spins; O, Zp, Zm: the other colour's in planes z, z + 1, z - 1.
  auto block_steps = [&](int c, int z, const uint32_t (&Own)[NWP], const uint32_t (&O)[NWP], const uint32_t (&Zp)[NWP],
                         const uint32_t (&Zm)[NWP], uint32_t (&V)[NBLK]) __attribute__((always_inline)) {
    const uint32_t jz = jbase + 4u * (uint32_t)((c * LB + z) * 6 * NWP);
    uint32_t Jw[6][NWP];
    {
      // 6 NWP words, 8-byte aligned: read as pairs, all issued before the first use
      uint64_t jv[3 * NWP];
#pragma unroll
      for (int k = 0; k < 3 * NWP; ++k)
        jv[k] = *(const __attribute__((address_space(3))) uint64_t*)(uintptr_t)(jz + 8u * (uint32_t)k);
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int w = 0; w < NWP; ++w) {
          const int e = k * NWP + w;
          Jw[k][w] = (uint32_t)(jv[e >> 1] >> (32 * (e & 1)));
        }
    }
    uint32_t Yp[NWP], Ym[NWP];
    shift_rows<L>(O, Yp, Ym);
    // The x-neighbour that is not in the site's own field position: j + 1 in rows whose sites have
    // odd x (phi = 1), j - 1 in the others, periodic within the field.
    const bool odd0 = ((c + z) & 1) != 0;   // row 0 has phi = 1
    const uint32_t mp = odd0 ? G::fields(0, G::H - 1, 0) : G::fields(0, G::H - 1, 1);
    const uint32_t mpw = odd0 ? G::fields(G::H - 1, 1, 0) : G::fields(G::H - 1, 1, 1);
    const uint32_t mm = odd0 ? G::fields(1, G::H - 1, 1) : G::fields(1, G::H - 1, 0);
    const uint32_t mmw = odd0 ? G::fields(0, 1, 1) : G::fields(0, 1, 0);
    uint32_t m0[NWP], m1[NWP], m2[NWP];
#pragma unroll
    for (int w = 0; w < NWP; ++w) {
      const uint32_t Xo = G::H == 1 ? O[w] : ((O[w] >> 1) & mp) | ((O[w] << (G::H - 1)) & mpw) | ((O[w] << 1) & mm) |
                          ((O[w] >> (G::H - 1)) & mmw);
      const uint32_t Up = ZB > 1 ? __builtin_amdgcn_alignbit(O[w], O[w], G::PB & 31) : Zp[w];
      const uint32_t Dn = ZB > 1 ? __builtin_amdgcn_alignbit(O[w], O[w], (32 - G::PB) & 31) : Zm[w];
      // flags: bit set <=> bond unsatisfied (S_i xor S_j xor [J = -1])
      const uint32_t f1 = xor3(Own[w], Up, Jw[0][w]), f2 = xor3(Own[w], Dn, Jw[1][w]);
      const uint32_t f3 = xor3(Own[w], Yp[w], Jw[2][w]), f4 = xor3(Own[w], Ym[w], Jw[3][w]);
      const uint32_t f5 = xor3(Own[w], O[w], Jw[4][w]), f6 = xor3(Own[w], Xo, Jw[5][w]);
      // Bit-sliced u = f1 + ... + f6, delivered as the level step m = 3 - u in 3-bit two's
      // complement: m = (7 - u) ^ 4, i.e. bits (~u0, ~u1, u2).
      const uint32_t s1 = xor3(f1, f2, f3), k1 = maj3(f1, f2, f3);
      const uint32_t s2 = xor3(f4, f5, f6), k2 = maj3(f4, f5, f6);
      const uint32_t t0 = s1 & s2;
      m0[w] = ~(s1 ^ s2);
      m1[w] = __builtin_amdgcn_bitop3_b32(k1, k2, t0, 0x69);
      m2[w] = maj3(k1, k2, t0);
    }
#pragma unroll
    for (int w = 0; w < NWP; ++w) {
      V[3 * w] = m0[w];
      V[3 * w + 1] = m1[w];
      V[3 * w + 2] = m2[w];
      asm volatile("" : "+v"(V[3 * w]), "+v"(V[3 * w + 1]), "+v"(V[3 * w + 2]));
    }
  };
  // Planes of the lattice by a dynamic index (a rolled plane loop).
  auto plane = [&](int c, int z, uint32_t (&v)[NWP]) __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < NWP; ++w) v[w] = lat(c, w)[z];
  };
  // Byte words of string word w: the site at bit b of the word is byte b >> 3 of A[b & 7] (4 (m & 7))
  // and D[b & 7] (m << 5). Planes are merged to pairs, pairs to nibbles (m in bits 1..3 of the
  // nibble), and the low and high nibbles of each byte masked out.
  auto expand = [&](const uint32_t (&V)[NBLK], int w, uint32_t (&A)[8], uint32_t (&D)[8]) __attribute__((always_inline)) {
    const uint32_t m0 = V[3 * w], m1 = V[3 * w + 1], m2 = V[3 * w + 2];
    if constexpr (Q == 2) {   // two sites, bits 0 and 1 (the bytes above them are not read)
      const uint32_t v0 = (m0 & 1u) | ((m1 << 1) & 2u) | (m2 << 2);
      const uint32_t v1 = ((m0 >> 1) & 1u) | (m1 & 2u) | ((m2 << 1) & ~3u);
      D[0] = v0 << 5;
      D[1] = v1 << 5;
      A[0] = (v0 << 2) & 0x1Cu;
      A[1] = (v1 << 2) & 0x1Cu;
      return;
    }
    const uint32_t P0 = (m0 & 0x55555555u) | ((m1 << 1) & 0xAAAAAAAAu);   // sites 2i: bits 2i, 2i+1
    const uint32_t P1 = ((m0 >> 1) & 0x55555555u) | (m1 & 0xAAAAAAAAu);   // sites 2i + 1
    const uint32_t W[4] = {((P0 << 1) & 0x77777777u) | ((m2 << 3) & 0x88888888u),    // sites 4i
                           ((P1 << 1) & 0x77777777u) | ((m2 << 2) & 0x88888888u),    // sites 4i + 1
                           ((P0 >> 1) & 0x77777777u) | ((m2 << 1) & 0x88888888u),    // sites 4i + 2
                           ((P1 >> 1) & 0x77777777u) | (m2 & 0x88888888u)};          // sites 4i + 3
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      D[k] = (W[k] << 4) & 0xE0E0E0E0u;
      D[k + 4] = W[k] & 0xE0E0E0E0u;
      A[k] = D[k] >> 3;
      A[k + 4] = D[k + 4] >> 3;
    }
  };
  // entry offset of a block's first site (byte 0)
  auto first_entry = [&](const uint32_t (&V)[NBLK]) __attribute__((always_inline)) -> uint32_t {
    return ((V[0] << 2) & 4u) | ((V[1] << 3) & 8u) | ((V[2] << 4) & 16u);
  };
  // Generator counter of group g (four sites) of block (c, z) in sweep t.
  auto group_ctr = [&](int c, int z, int g, uint64_t t) __attribute__((always_inline)) -> PhiloxRun {
    return PhiloxRun{((uint32_t)(c * L + z * ZB + g / G::NGP) << 8) | (uint32_t)(g % G::NGP), (uint32_t)t, real_id, ctr3};
  };
  // first generator round of the next group that runs beside attempt i of a group
  constexpr auto round_of = [](int i) constexpr { return SU || PS ? (i == 0 ? 0 : 2 + 2 * i) : (i < 3 ? 3 * i - i / 2 : 2 + 2 * i); };
  static_assert(round_of(0) == 0 && round_of(4) == 10, "ten rounds a group");
  // The generator runs one group ahead: pr holds the words of the next group of four sites, and
  // its rounds are spread over the attempts of the group before it (also across blocks and colours,
  // and but for the staged form across sweeps), so that they fill the wait for each threshold read.
  PhiloxRun pr{};
  if constexpr (!WS && !PS) {
    pr = group_ctr(0, 0, 0, A.t0);
    if constexpr (SU) philox_rounds_u<0, 3>(pr, key0, key1);
    philox_rounds<SU ? 3 : 0, 10>(pr, kv);
  }
  // Staged form. With c0, t, real_id uniform and c3 the walker's word, rounds 0-2 leave: n2 = A ^ c3,
  // q = M1 n2, n0' = hi(q) ^ K1, r = M0 n0', n0'' = lo(q) ^ X2, n2'' = hi(r) ^ P3, n3'' = lo(r), and
  // round 3's first word takes X3 for its uniform part; A, X2, X3 are the staged words, K1 is
  // constant and P3 constant in a sweep.
  constexpr uint32_t PM0 = 0xD2511F53u, PM1 = 0xCD9E8D57u, PW0 = 0x9E3779B9u, PW1 = 0xBB67AE85u;
  const uint32_t sbase = PS ? staged_base(hbase, hn) : 0u;
  uint32_t ps_K1 = 0, ps_P3 = 0, ps_addr = 0;   // ps_addr: staged words of the current block
  u32x4 ps_next{};                              // staged words of the next group
  if constexpr (PS) ps_K1 = (PM1 * real_id) ^ (key0 + PW0);
  auto stage_sweep = [&](uint64_t t) __attribute__((always_inline)) {
    const uint32_t n0 = __umulhi(PM1, real_id) ^ (uint32_t)t ^ key0;
    const uint32_t H0 = __umulhi(PM0, n0) ^ (key1 + PW1);
    ps_P3 = (PM0 * n0) ^ (key1 + 2u * PW1);
    for (int e = lane; e < 2 * LB * NG; e += 64) {
      const int cb = e / NG, g = e % NG;   // block c LB + b, group within it
      const uint32_t c0 = ((uint32_t)(cb * ZB + g / G::NGP) << 8) | (uint32_t)(g % G::NGP);
      const uint64_t p0 = (uint64_t)PM0 * c0;
      const uint64_t p = (uint64_t)PM1 * (H0 ^ (uint32_t)p0);
      const u32x4 w{{(uint32_t)(p0 >> 32) ^ key1, (uint32_t)(p >> 32) ^ (key0 + 2u * PW0),
                     (uint32_t)p ^ (key0 + 3u * PW0), 0u}};
      lds_store_u32x4(sbase + (uint32_t)e * 16u, w);
    }
    asm volatile("" ::: "memory");
  };
  // rounds 0-3 of the group whose staged words are w
  auto staged_rounds = [&](const u32x4& w) __attribute__((always_inline)) {
    const uint64_t q = (uint64_t)PM1 * (w.v[0] ^ ctr3);
    const uint64_t r = (uint64_t)PM0 * ((uint32_t)(q >> 32) ^ ps_K1);
    const uint64_t p0 = (uint64_t)PM0 * ((uint32_t)q ^ w.v[1]);
    const uint64_t p1 = (uint64_t)PM1 * ((uint32_t)(r >> 32) ^ ps_P3);
    pr.c0 = (uint32_t)(p1 >> 32) ^ w.v[2];
    pr.c1 = (uint32_t)p1;
    pr.c2 = xor3((uint32_t)(p0 >> 32), (uint32_t)r, kv.k1[3]);
    pr.c3 = (uint32_t)p0;
  };
  // Warp-specialized form: the words of block b sit in ring slot b mod 3; rw holds the next
  // group's words, read one group ahead.
  const uint32_t rbase = WS ? ws_ring_base(K, jk_words(L), hn) : 0u;
  auto ring = [&](uint32_t slot, int g) __attribute__((always_inline)) -> uint32_t {
    return rbase + slot * ws_slot_bytes<L>() + (uint32_t)(g * 64 + lane) * 16u;
  };
  uint32_t rslot = 0, rslot_n = 1;
  u32x4 rw{};
  if constexpr (WS) rw = lds_load_u32x4(ring(0, 0));

  // Running extremes of the walker's level since its round-trip state last changed (multicanonical).
  // Nothing in between reached the bound the state waits for, so a check compares them with the
  // window; the minimum folds into the walker's record when they restart and at the launch's end.
  constexpr int kFar = 1 << 29;
  int bmin = kFar, bmax = -kFar;
  auto fold_minimum = [&]() __attribute__((always_inline)) {
    tr.Bmin = min(tr.Bmin, bmin);
    tr.newmin = (bmin <= Bnm) ? 1 : tr.newmin;   // E < e_bot <=> B <= Bnm
    bmin = kFar;
    bmax = -kFar;
  };
  for (uint32_t s = 0; s < A.n_sweeps; ++s) {
    const uint64_t t = A.t0 + s;
    const uint64_t tau0 = t * (uint64_t)N + 1u;
    if constexpr (PS) {
      // this sweep's staged words, then the first group's random words (not run ahead across sweeps:
      // the table holds one sweep)
      stage_sweep(t);
      ps_addr = sbase;
      staged_rounds(lds_load_u32x4(ps_addr));
      philox_rounds<4, 10>(pr, kv);
      ps_next = lds_load_u32x4(ps_addr + 16u);
    }
    // The counter is opaque in each sweep where planes are unrolled beyond L = 4, in the tempering form
    // and in the persistent kernel: products that depend on the group and the walker alone would otherwise be kept in
    // registers for all groups (L = 6: over 256 of them, one wave per SIMD).
    if constexpr (ROLL || L == 6 || PT) asm volatile("" : "+v"(ctr3));
    int es0 = 0, es1 = 0, es2 = 0;   // tempering: bit counts of the accepted steps' planes
    static_for<2>([&](auto cc) __attribute__((always_inline)) {
      constexpr int c = decltype(cc)::value;
      uint32_t Vc[NBLK];
      // own spins of plane z, the other colour's in planes z and z + 1: each plane is read once
      uint32_t Cw[NWP], Oc[NWP], On[NWP];
      {
        uint32_t Ob[NWP];
        plane(c, 0, Cw);
        plane(1 - c, 0, Oc);
        plane(1 - c, LB > 1 ? 1 : 0, On);
        plane(1 - c, LB - 1, Ob);
        block_steps(c, 0, Cw, Oc, On, Ob, Vc);
      }
      // the colour's first threshold; later ones are read by the attempt before, across block ends
      // (tempering: a group ahead within a block)
      uint32_t th_fly = 0, addr_cur = 0;
      uint32_t thg[4] = {0, 0, 0, 0};   // tempering: the thresholds of the group to come
      if constexpr (!PT) th_fly = read_row(or_entry<0>(first_entry(Vc), R));
      uint32_t th_acc = th_fly;   // paired form: th_fly after a rejection, th_acc after an acceptance
      uint64_t accepted = 0;      // of the attempt before
      // thresholds of group g of a block (byte words of its string word)
      auto group_thresholds = [&](const uint32_t (&Aw)[8], auto gt) __attribute__((always_inline)) {
        constexpr int g = decltype(gt)::value;
        static_for<(4 * g + 4 <= Q) ? 4 : Q - 4 * g>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value, q = 4 * g + i, p = (q / H) * FB + q % H;
          thg[i] = read_row(or_entry<(p >> 3) & 3>(Aw[p & 7], R));
        });
      };
      // small lattices: planes unrolled (static register indices); larger ones: a plane loop
      // whose dynamic index selects registers of the per-(colour, word) arrays
#pragma unroll kZUnroll
      for (int z = 0; z < LB; ++z) {
        const bool has_next = z + 1 < LB;
        // The next block's steps (and the entry offset of its first site), prepared once this
        // block's planes are all expanded: its registers then need no copies at the loop's end.
        uint32_t Vn[NBLK], Cn[NWP], Onn[NWP], An = 0;
        auto prepare_next = [&]() __attribute__((always_inline)) {
          if (has_next) {
            plane(c, z + 1, Cn);
            plane(1 - c, z + 2 < LB ? z + 2 : 0, Onn);
            block_steps(c, z + 1, Cn, On, Onn, Oc, Vn);
            An = first_entry(Vn);
          }
        };
        uint32_t Ac[8], Dc[8];   // byte words of the string word in progress
        expand(Vc, 0, Ac, Dc);
        if constexpr (NWP == 1 && !PT) prepare_next();
        if constexpr (PT) group_thresholds(Ac, std::integral_constant<int, 0>{});
        const uint64_t tau_blk = tau0 + (uint64_t)(c * (N / 2) + z * Q);
        // Acceptance bits are shifted into F in site order, with a zero for every bit of a
        // field beyond the row's H sites, and applied to the plane-colour string once per word.
        uint32_t F = 0;
        // levels after each attempt since the last window check (kCheckGroups groups of four)
        constexpr int kCheckGroups = check_groups<L>();
        int Bq[4 * kCheckGroups];
        static_for<NG>([&](auto gc) __attribute__((always_inline)) {
          constexpr int g = decltype(gc)::value;
          u32x4 rnd;
          if constexpr (WS) {
            // this group's words, and the read of the next group's (in this block, or the first
            // group of the next block, whose slot the generator filled before the last barrier)
            rnd = rw;
            rw = lds_load_u32x4(g + 1 < NG ? ring(rslot, g + 1) : ring(rslot_n, 0));
          } else {
            rnd = u32x4{{pr.c0, pr.c1, pr.c2, pr.c3}};
            // the next group: in this block, the next block, the other colour or the next sweep
            if constexpr (PS) {}
            else if (g + 1 < NG) pr = group_ctr(c, z, g + 1, t);
            else if (has_next) pr = group_ctr(c, z + 1, 0, t);
            else if (c == 0) pr = group_ctr(1, 0, 0, t);
            else pr = group_ctr(0, 0, 0, t + 1);
          }
          constexpr int n_att = (4 * g + 4 <= Q) ? 4 : Q - 4 * g;
          if constexpr (PT) {
            // The rows are fixed for the sweep, so the group's decisions are independent of each
            // other: the next group's generator call and threshold reads, then this group's
            // decisions. String words end with a group.
            constexpr int p0 = (4 * g / H) * FB + (4 * g) % H, w = p0 >> 5;
            constexpr int qe = 4 * g + n_att - 1, pe = (qe / H) * FB + qe % H;
            static_assert(L <= 2 || NWP == 1 || (H * 32 / FB) % 4 == 0, "string words end with a group");
            constexpr bool word_end = qe + 1 == Q || (((qe + 1) / H) * FB + (qe + 1) % H) >> 5 != w;
            const uint32_t th[4] = {thg[0], thg[1], thg[2], thg[3]};
            uint32_t M[3];   // planes of this word's steps, for the energy
            M[0] = Vc[3 * w];
            M[1] = Vc[3 * w + 1];
            M[2] = Vc[3 * w + 2];
            if constexpr (g + 1 < NG) {
              if constexpr (word_end) expand(Vc, w + 1, Ac, Dc);
              group_thresholds(Ac, std::integral_constant<int, g + 1>{});
            }
            if constexpr (SU) {
              philox_rounds_u<0, 3>(pr, key0, key1);
              philox_rounds<3, 10>(pr, kv);
            } else {
              philox_rounds<0, 10>(pr, kv);
            }
            if constexpr (g + 1 == NG) prepare_next();
            accept_group<H, FB, Q, 4 * g>(rnd, th, F);
            if constexpr (word_end) {
              const uint32_t flips = __builtin_bitreverse32(F) >> (31 - (pe & 31));
              Cw[w] ^= flips;
              // accepted steps' energy: 4 (popc(m0) + 2 popc(m1) - 4 popc(m2)) over the flips
              es0 += __popc(flips & M[0]);
              es1 += __popc(flips & M[1]);
              es2 += __popc(flips & M[2]);
              F = 0;
            }
          } else {
          static_for<n_att>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value, q = 4 * g + i;
            constexpr int y = q / H, j = q % H;
            constexpr int p = y * FB + j, w = p >> 5;
            constexpr int qn = q + 1 < Q ? q + 1 : 0;                    // the next site, its string word
            constexpr int pn = (qn / H) * FB + qn % H, wn = pn >> 5;
            constexpr bool last_in_word = (q + 1 == Q) || wn != w;
            constexpr int a = 4 * (g % kCheckGroups) + i;                // attempts since the check
            // generator rounds of the next group, spread over this group's attempts
            auto rounds = [&]() __attribute__((always_inline)) {
              if constexpr (!WS) {
                // SU: rounds 0-2 act on a counter whose words 0..2 are still uniform, so their
                // uniform parts go to the scalar unit (two of their six products are left, so round
                // 3 joins them: four products an attempt)
                if constexpr (SU && i == 0) {
                  philox_rounds_u<0, 3>(pr, key0, key1);
                  philox_rounds<3, 4>(pr, kv);
                } else if constexpr (PS && i == 0) {
                  const u32x4 w = ps_next;
                  ps_next = lds_load_u32x4(ps_addr + (uint32_t)(g + 2) * 16u);
                  staged_rounds(w);
                } else {
                  philox_rounds<round_of(i), round_of(i + 1)>(pr, kv);
                }
              }
            };
            if constexpr (SPEC) {
              const uint32_t rc = rnd.v[i];
              const int Bacc = add_step(B, Dc[p & 7], (p >> 3) & 3);
              const int Racc = XT ? Bacc : clamp_row(Bacc, Bmax);
              if constexpr (last_in_word && q + 1 < Q) {
                expand(Vc, wn, Ac, Dc);
                if constexpr (wn == NWP - 1) prepare_next();
              }
              const uint32_t Aq = q + 1 < Q ? Ac[pn & 7] : An;
              uint32_t n_rej = 0, n_acc = 0;
              if (q + 1 < Q || has_next) {
                n_rej = read_row(or_entry<(pn >> 3) & 3>(Aq, R));
                n_acc = read_row(or_entry<(pn >> 3) & 3>(Aq, Racc));
              }
              __builtin_amdgcn_sched_barrier(0);   // the reads go out before anything else
              rounds();
              // the attempt before is shifted into F here, but for the last of a row with unused bits
              // and of a word, which are shifted in at once
              constexpr bool kAtOnce = last_in_word || (j == H - 1 && FB > H);
              constexpr bool kShift = q > 0 && j > (FB > H ? 0 : -1) && (p & 31) > 0;
              if constexpr (a >= 2 && a % 2 == 0)
                accepted = decide_paired<XT, kShift, 1>(rc, th_fly, th_acc, accepted, Bacc, Racc, Bq[a - 2], Bq[a - 1], B,
                                                        R, F, bmin);
              else if constexpr (a >= 3)
                accepted = decide_paired<XT, kShift, 2>(rc, th_fly, th_acc, accepted, Bacc, Racc, Bq[a - 3], Bq[a - 2], B,
                                                        R, F, bmax);
              else
                accepted = decide_paired<XT, kShift, 0>(rc, th_fly, th_acc, accepted, Bacc, Racc, B, B, B, R, F, bmin);
              if constexpr (kAtOnce) accept_shift(accepted, F);
              th_fly = n_rej;
              th_acc = n_acc;
            } else {
              // (1) the threshold of this site, read by the previous decision at the address it
              //     computed
              const uint32_t th = th_fly;
              const uint32_t Dq = Dc[p & 7];
              // the next string word's bytes, in time for the address of its first site
              if constexpr (last_in_word && q + 1 < Q) {
                expand(Vc, wn, Ac, Dc);
                if constexpr (wn == NWP - 1) prepare_next();
              }
              // (2) independent work: generator rounds of the next group. Empty volatile
              //     statements pin the order: they are ordered with the decision, and the
              //     rounds' outputs pass through the second one. The first takes only the words
              //     the round's products do not read: a VALU read of a register an asm statement
              //     wrote costs a wait state, and uniform words stay scalar.
              if constexpr ((!SU && !PS) || i > 0) asm volatile("" : "+v"(pr.c1), "+v"(pr.c3));
              rounds();
              const uint32_t rc = rnd.v[i];
              asm volatile("" : "+v"(pr.c0), "+v"(pr.c1), "+v"(pr.c2), "+v"(pr.c3));
              // (3) the decision, the next site's table address and its read, issued before the
              //     bookkeeping and flips that follow
              constexpr int cb = (p >> 3) & 3, nb = (pn >> 3) & 3;
              const uint32_t Aq = q + 1 < Q ? Ac[pn & 7] : An;
              if constexpr (a >= 2 && a % 2 == 0)
                decide_bytes<XT, 1, cb, nb>(rc, th, Dq, Aq, vBmax, Bq[a - 2], Bq[a - 1], B, R, F, addr_cur, bmin);
              else if constexpr (a >= 3)
                decide_bytes<XT, 2, cb, nb>(rc, th, Dq, Aq, vBmax, Bq[a - 3], Bq[a - 2], B, R, F, addr_cur, bmax);
              else
                decide_bytes<XT, 0, cb, nb>(rc, th, Dq, Aq, vBmax, B, B, B, R, F, addr_cur, bmin);
              if (q + 1 < Q || has_next) th_fly = read_row(addr_cur);
            }
            Bq[a] = B;
            // end of a row inside the word: zeros for the field's unused bits; end of the word
            // (or of the string): apply the flips
            if constexpr (last_in_word) {
              Cw[w] ^= __builtin_bitreverse32(F) >> (31 - (p & 31));
              F = 0;
            } else if constexpr (j == H - 1 && FB > H) {
              F <<= (FB - H);
            }
          });
          // a short last group: the generator rounds its missing attempts would have run
          if constexpr (!WS && n_att < 4) philox_rounds<round_of(n_att), 10>(pr, kv);
          // Every kCheckGroups-th group (and at the block's end): if an attempt since the last check
          // reached the bound the round-trip state waits for, replay those attempts' state exactly.
          if constexpr (g % kCheckGroups == kCheckGroups - 1 || g + 1 == NG) {
            constexpr int g0 = g - g % kCheckGroups;                   // first group since the check
            constexpr int cnt = 4 * (g - g0) + n_att;                  // attempts since the check (even)
            // the decisions have taken in the levels of all attempts but the last pair
            bmin = min(bmin, min(Bq[cnt - 2], Bq[cnt - 1]));
            bmax = max(bmax, max(Bq[cnt - 2], Bq[cnt - 1]));
            if (bmin < win.lo || bmax > win.hi) {
#pragma unroll
              for (int k = 0; k < cnt; ++k)
                track_attempt<L == 2>(tr, Bq[k], tau_blk + (uint64_t)(4 * g0 + k), Bbot, Btop);
              win = make_window(tr.state, Bbot, Btop);
              fold_minimum();
            }
          }
          }
        });
#pragma unroll
        for (int w = 0; w < NWP; ++w) lat(c, w)[z] = Cw[w];
        if constexpr (PS) ps_addr += 16u * NG;
        if constexpr (WS) {
          // this block's words are consumed: the generator may refill their slot
          __syncthreads();
          rslot = rslot_n;
          rslot_n = rslot_n == 2u ? 0u : rslot_n + 1u;
        }
        if (has_next) {
#pragma unroll
          for (int k = 0; k < NBLK; ++k) Vc[k] = Vn[k];
#pragma unroll
          for (int w = 0; w < NWP; ++w) {
            Oc[w] = On[w];
            On[w] = Onn[w];
            Cw[w] = Cn[w];
          }
        }
      }
    });
    if constexpr (PT) E += 4 * (es0 + 2 * es1 - 4 * es2);
    if constexpr (PT) {
      // end of the Metropolis phase: bookkeeping with stamp (t + 1) N, trace
      const int M = A.pt_M;
      const bool active = pt_active;
      if (active) track_energy(te, E, (t + 1u) * (uint64_t)N, e_bot, e_top);
      if (t - A.trace_t0 < (uint64_t)A.trace_cap && (uint64_t)(gw - A.trace_w0) < (uint64_t)A.trace_nw)
        A.trace[(gw - A.trace_w0) * A.trace_cap + (int64_t)(t - A.trace_t0)] = E;
      // exchange phase: slots (s, s+1), s = t (mod 2), of each set of M lanes
      const uint32_t base = pt_base;
      lds_store_i32(sE + 4u * (base + (uint32_t)slot), E);
      __syncthreads();
      const int par = (int)(t & 1u);
      const bool lower = active && ((slot & 1) == par) && (slot + 1 < M);
      const bool upper = active && (slot >= 1) && (((slot - 1) & 1) == par);
      int dec = 0;
      if (lower) {
        const int Eh = lds_load_i32(sE + 4u * (base + (uint32_t)slot + 1u));
        const int d = (Eh - E) / 4;   // energies of one realization share their residue mod 4
        const uint32_t th = pt_swap_threshold(A.pt_q[(int64_t)r * kMaxReplicas + slot], d);
        const uint32_t set = pt_set;   // set index within the realization
        u32x4 rr;
        if constexpr (GEN == kGenVector) {   // all round keys are in registers
          PhiloxRun pe{(uint32_t)(slot >> 2), (uint32_t)t, real_id, (set << 8) | kTagSwap};
          philox_rounds<0, 10>(pe, kv);
          rr = u32x4{{pe.c0, pe.c1, pe.c2, pe.c3}};
        } else {
          rr = philox4x32_10((uint32_t)(slot >> 2), (uint32_t)t, real_id, (set << 8) | kTagSwap, key0, key1);
        }
        const int k4 = slot & 3;
        const uint32_t rw = k4 == 0 ? rr.v[0] : k4 == 1 ? rr.v[1] : k4 == 2 ? rr.v[2] : rr.v[3];
        dec = min(rw, 0xFFFFFFFEu) < th ? 1 : 0;
        lds_store_i32(sD + 4u * (base + (uint32_t)slot), dec);
        if (dec) {
          const uint32_t ca = sAcc + 4u * (base + (uint32_t)slot);
          lds_store_i32(ca, lds_load_i32(ca) + 1);
        }
      }
      __syncthreads();
      int nslot = slot;
      if (lower && dec) nslot = slot + 1;
      if (upper && lds_load_i32(sD + 4u * (base + (uint32_t)slot - 1u))) nslot = slot - 1;
      slot = nslot;
      B = slot * 32;
      R = B;
      __syncthreads();
    } else {
      // end of sweep: histogram (on chip) and trace
      const int k = (B >> 5) + row0;
      const uint32_t kh = (uint32_t)(k - hlo);
      if (kh < (uint32_t)hn && k < K)
        __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t*)(uintptr_t)(hbase + 4u * kh), 1u,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      else if ((uint32_t)k < (uint32_t)K)  // always true for exact energies
        atomicAdd(A.hist + RI.level_off + k, 1ULL);
      if (t - A.trace_t0 < (uint64_t)A.trace_cap && (uint64_t)(gw - A.trace_w0) < (uint64_t)A.trace_nw)
        A.trace[(gw - A.trace_w0) * A.trace_cap + (int64_t)(t - A.trace_t0)] = e_base + 4 * k;
    }
  }

  // registers -> walker state
  {
    uint32_t* sp = A.spins + RI.spin_off + wl;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int w = 0; w < NWP; ++w)
#pragma unroll
        for (int b = 0; b < LB; ++b)
#pragma unroll
          for (int z = 0; z < ZB; ++z)
            sp[(int64_t)((c * L + b * ZB + z) * NWP + w) * walkers] =
                ZB > 1 ? (lat(c, w)[b] >> (z * G::PB)) & ((1u << (G::PB & 31)) - 1u) : lat(c, w)[b];
  }
  if constexpr (PT) {
    A.ws.E[gw] = E;
    A.ws.E_min[gw] = te.Emin;
    A.ws.rt_state[gw] = te.state;
    A.ws.new_min[gw] = te.newmin;
    A.ws.rt_count[gw] += te.trips;
    A.ws.t_first[gw] = te.t_first;
    A.ws.t_last[gw] = te.t_last;
    A.pt_slot[gw] = slot;
    // exchange counters of the pairs (s, s+1) of this lane's set, s = lane index in the set
    const int M = A.pt_M;
    const int cidx = (int)((uint32_t)lane - pt_base);
    if (pt_active && cidx < M - 1)   // global set index: walker offsets of realizations are multiples of 64
      A.pt_acc[(int64_t)(RI.walker_off / 64 * A.pt_spw + pt_set) * (M - 1) + cidx] +=
          (uint64_t)lds_load_i32(sAcc + 4u * (uint32_t)lane);
  } else {
    // the launch's histogram counts (at most 64 walkers x 2^20 sweeps per level)
    __syncthreads();
    for (int e = lane; e < hn; e += 64) {
      const uint32_t c = (uint32_t)lds_load_i32(hbase + 4u * (uint32_t)e);
      if (c) atomicAdd(A.hist + RI.level_off + hlo + e, (unsigned long long)c);   // c > 0: hlo + e < K
    }
    fold_minimum();
    A.ws.E[gw] = e_base + 4 * ((B >> 5) + row0);
    A.ws.E_min[gw] = e_base + 4 * ((tr.Bmin >> 5) + row0);
    A.ws.rt_state[gw] = tr.state;
    A.ws.new_min[gw] = tr.newmin;
    A.ws.rt_count[gw] += tr.trips;
    A.ws.t_first[gw] = tr.t_first;
    A.ws.t_last[gw] = tr.t_last;
  }
}

// The generator wave of the warp-specialized form: the words of every group of every block of
// the launch (blocks in sweep order: sweep, colour, plane), two blocks ahead of the sampling
// wave. It meets the sampling wave at the same barriers: after the tables are staged, at the end
// of every block, before the histogram flush.
template <int L>
__device__ __forceinline__ void generate_words(const SweepArgs& A, int wave) {
  constexpr int NG = Geo<L>::NG, ZB = Geo<L>::ZB, LB = Geo<L>::LB;
  const int lane = (int)(threadIdx.x & 63u);
  const RealInfo& RI = A.reals[A.wave_real[wave]];
  const uint32_t ctr3 = ((uint32_t)(A.wave_wl[wave] + lane) << 8) | kTagAcc, real_id = RI.real_id;
  const uint32_t key0 = (uint32_t)A.walker_seed, key1 = (uint32_t)(A.walker_seed >> 32);
  const uint32_t rbase = ws_ring_base(RI.K, jk_words(L), A.hist_n);
  // blocks in the sampling wave's order; (t, cz = c LB + block) names the block to be written next
  const uint32_t nb = (uint32_t)A.n_sweeps * 2u * (uint32_t)LB;   // at most 2^20 sweeps per launch
  uint32_t t = (uint32_t)A.t0, cz = 0;
  auto advance = [&]() __attribute__((always_inline)) {
    if (++cz == 2u * (uint32_t)LB) {
      cz = 0;
      ++t;
    }
  };
  auto fill = [&](uint32_t slot) __attribute__((always_inline)) {
    for (int g = 0; g < NG; ++g) {
      const uint32_t pl = cz * (uint32_t)ZB + (uint32_t)(g / Geo<L>::NGP);   // c L + z of the group's plane
      const u32x4 w = philox4x32_10_u((pl << 8) | (uint32_t)(g % Geo<L>::NGP), t, real_id, ctr3, key0, key1);
      lds_store_u32x4(rbase + slot * ws_slot_bytes<L>() + (uint32_t)(g * 64 + lane) * 16u, w);
    }
  };
  if (nb > 0u) fill(0u);
  advance();
  if (nb > 1u) fill(1u);
  advance();
  __syncthreads();   // tables staged, blocks 0 and 1 written
  uint32_t slot = 2;
  for (uint32_t b = 0; b < nb; ++b) {
    if (b + 2u < nb) fill(slot);   // block b + 2
    advance();
    slot = slot == 2u ? 0u : slot + 1u;
    __syncthreads();   // the sampling wave has finished block b
  }
  __syncthreads();     // before the sampling wave's histogram flush
}

}  // namespace nfm
