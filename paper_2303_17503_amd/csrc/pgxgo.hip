// pgxgo.hip -- batched Go environment step for AMD MI355X (gfx950, wave64), C ABI in include/pgxgo.h.
//
// What is computed: the Go environment of the Pgx paper (arXiv 2303.17503): Fig. 2 (init/step API,
// legal_action_mask, observation, current_player), Table 1 (9x9x17 / 82 actions, 19x19x17 / 362 actions),
// Appendix C "Go" (Tromp-Taylor area scoring, komi for White, 8x2 history planes + colour plane, pass is
// the last action, rewards +1/-1/0), Sec. 4.1 (random policy, auto-reset on termination).
//
// How it is mapped to the machine (nothing of this is in the paper, whose implementation is XLA-generated):
//   * One board row per lane.  A wavefront holds W = 63/(N+1) boards (3 at 19x19, 6 at 9x9): board j owns
//     lanes j*(N+1)+1 .. j*(N+1)+N, and lanes j*(N+1) stay all-zero "sentinel rows", so a one-lane DPP
//     wave shift moves every row to its north/south neighbour and brings zeros in from off the board.
//   * Stones are row bitboards (bit c = column c).  East/west neighbours are register shifts, north/south
//     neighbours are DPP shifts; a flood-fill step is a handful of VALU instructions for all W boards at once.
//   * Facts about a whole board (a move is legal, ...) come from a ballot masked with the lane segment of the board,
//     counts (liberties of the chains a move touches) from one sum per board in LDS; every lane of the board then holds
//     the same answer.
//   * The state keeps, besides the stones, the set of stones whose chain has exactly one liberty
//     ("atari sets").  With them captures, the ko test and the whole legal mask are stencils; only the
//     chains touched by the move are re-flooded (the merged chain and at most four opposing neighbours),
//     a flood stops as soon as two liberties have been seen, and several growth steps are taken per
//     (comparatively expensive) look at the liberties.
//   * The emission takes the history point-major: 16 bits per point = 8 plies x (black, white), two points per
//     dword, so a ply is one shift-and-insert per dword and the [N][N][17] byte observation is produced by
//     building the 17-bit-per-point bit stream of a board in LDS and expanding 16 bits -> 16 bytes per
//     lane through a 256-entry LDS table, stored as aligned 16-byte vectors.
//   * HBM layout: a game's state is one run of bytes (State); at 19x19 the history lies there position by position, so
//     that a ply writes the new position over the oldest one instead of every point's history.
//   * Kernels: go_step_kernel (one ply per launch, optionally drawing the next random action),
//     go_rollout_kernel (T plies per launch, state in registers), go_step_slots_kernel (tree search: step
//     from and to arbitrary state slots), go_step_superko_kernel (one ply with the positional-superko rule:
//     Zobrist keys in per-game open-addressing tables), plus small set-up / export / import kernels.
//   * Small batches are stepped by teams of wavefronts per group of boards (go_step_team_kernel, go_step_superko_team_kernel).
//   * How many boards a launch puts into a wavefront (1 .. W) is chosen per launch: W for throughput at large
//     batches, fewer at small batches where the slowest board of a wavefront and its serial output rounds
//     decide the latency.
//   * Output stores: every store instruction of a wavefront covers whole 128-byte lines (wave_common.hpp), and
//     the kind of store -- through the L2, with the non-temporal hint, ordinary -- is chosen per launch from the
//     bytes it writes and from whether it overwrites the previous launch's buffers (store_kind_for).  The
//     line-padded output pitches make a wavefront's stream consist of whole lines only.
//   * Recordings that outgrow the memory-side cache are written in time slots, in the order of their addresses (Pace).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "pgxgo.h"
#include "wave_common.hpp"

namespace {

using namespace pgxwave;

thread_local int g_last_hip = 0;

#define HIPCHK(expr)                                   \
  do {                                                 \
    hipError_t e_ = (expr);                            \
    if (e_ != hipSuccess) {                            \
      g_last_hip = (int)e_;                            \
      return PGXGO_EHIP;                               \
    }                                                  \
  } while (0)

constexpr int kWavesPerBlock = kBlockThreads / 64;   // of the kernels without teams: the wavefronts share the lookup table and no more; this only shapes the launch


// ------------------------------------------------------------------------------------------------
// geometry
// ------------------------------------------------------------------------------------------------
template <int N>
struct Geo {
  static constexpr int P = N * N;
  static constexpr int A = P + 1;
  static constexpr int STRIDE = N + 1;        // lanes per board, one of them the zero sentinel row
  static constexpr int W = 63 / STRIDE;       // boards per wavefront
  static constexpr int HD = (N + 1) / 2;      // history dwords per row, two points per dword
  static constexpr bool RINGED = N > 16;      // how the history lies in memory, see State
  static constexpr int CUR = RINGED ? 2 : 1;  // dwords of a row's stones and atari set
  static constexpr int TAIL = RINGED ? HD - 8 : HD - 4;   // history dwords of a row beyond its first part
  static constexpr int HIST = RINGED ? 8 : 4;             // dwords of that first part
  static constexpr uint32_t FULL = (1u << N) - 1u;
  static constexpr int OBS = P * 17;          // observation bytes per board
  static constexpr int ROWBITS = N * 17;      // observation bits contributed by one row
  static constexpr int NR = (ROWBITS + 31) / 32;       // dwords of one row's bit string
  static constexpr int NI = ROWBITS / 32 - 1;          // dwords 1..NI of the shifted string are never shared with another row
  static constexpr int OBS_PAD = (OBS + 127) / 128 * 128;   // the pitches at which every board starts on a 128-byte line
  static constexpr int A_PAD = (A + 127) / 128 * 128;
  static constexpr int OBS_DW = ((OBS_PAD + 15 + 31) / 32 + 3) / 4 * 4;   // LDS dwords of one board's bit stream (+ up to 15 lead bits)
  static constexpr int MASK_DW = ((A + 15 + 31) / 32 + 3) / 4 * 4;
  static constexpr int GAME = (N * (CUR + TAIL + HIST) + 3) / 4 * 4;   // dwords of a game's state, whole 16-byte groups
  static constexpr size_t row_bytes = (size_t)(HD + 4) * 4;   // room per row in the caller's state buffer
  static_assert(GAME * 4 <= N * row_bytes, "the state fits the size the caller was told");
  // lanes holding the rows of board slot j
  static constexpr uint64_t seg(int j) { return ((1ull << N) - 1ull) << (j * STRIDE + 1); }
};

// per-board scalars, one 16-byte record per environment
//   x: ko point or -1     y: steps[0:16) | passes[16:18) | white_to_move[18] | terminated[19] | black_player[20] | head[21:24) (State)
//   z: episode            w: illegal actions received
struct Meta {
  int ko, steps, passes, wtm, term, bp;
  int head;              // where the ring of positions begins (State)
  uint32_t episode, illegal;
};
__device__ __forceinline__ Meta unpack_meta(uint4 v) {
  Meta m;
  m.ko = (int)v.x;
  m.steps = v.y & 0xFFFF; m.passes = (v.y >> 16) & 3; m.wtm = (v.y >> 18) & 1; m.term = (v.y >> 19) & 1; m.bp = (v.y >> 20) & 1; m.head = (v.y >> 21) & 7;
  m.episode = v.z; m.illegal = v.w;
  return m;
}
__device__ __forceinline__ uint4 pack_meta(const Meta& m) {
  uint4 v;
  v.x = (uint32_t)m.ko;
  v.y = (uint32_t)m.steps | ((uint32_t)m.passes << 16) | ((uint32_t)m.wtm << 18) | ((uint32_t)m.term << 19) | ((uint32_t)m.bp << 20) | ((uint32_t)m.head << 21);
  v.z = m.episode; v.w = m.illegal;
  return v;
}

// all 4-neighbours of the set x (bits beyond column N-1 may be set; callers intersect with on-board sets)
// (kept(v): v is wanted by itself.  The ORs of a dilation are built as two halves, each of which ends in one that takes the neighbouring
// lane's row as an operand; as one expression the compiler moves the two rows into registers first and ORs three at a time, two
// instructions more.)
__device__ __forceinline__ uint32_t kept(uint32_t v) {
  asm volatile("" ::"v"(v));
  return v;
}
__device__ __forceinline__ uint32_t dilate(uint32_t x) {
  const uint32_t a = kept(from_lane_below(x) | (x << 1)), b = kept(from_lane_above(x) | (x >> 1));
  return a | b;
}
// the set and all its 4-neighbours, as two halves
__device__ __forceinline__ Halves grown(uint32_t x) {
  const uint32_t sideways = kept((x << 1) | x);
  return Halves{kept(from_lane_below(x) | sideways), kept(from_lane_above(x) | (x >> 1))};
}
__device__ __forceinline__ uint32_t grown_in(uint32_t x, uint32_t S) { const Halves h = grown(x); return (h.a | h.b) & S; }

// Size class of a board-wide set given by its row words: exactly one element / two or more.
__device__ __forceinline__ void board_count(uint32_t w, uint32_t seglo, uint32_t seghi, bool& one, bool& two) {
  const uint64_t nz = ballot(w != 0u), mu = ballot((w & (w - 1u)) != 0u);
  const int c = __popc((uint32_t)nz & seglo) + __popc((uint32_t)(nz >> 32) & seghi);
  two = (((uint32_t)mu & seglo) | ((uint32_t)(mu >> 32) & seghi)) != 0u || c >= 2;
  one = !two && c == 1;
}

// connected component(s) of `seed`, a part of S, inside S
__device__ __forceinline__ uint32_t flood_plain(uint32_t seed, uint32_t S) {
  uint32_t F = seed;
  for (;;) {   // three growth steps per convergence test: the test (ballot, scalar branch) costs as much as a step
    F = grown_in(F, S);
    F = grown_in(F, S);
    uint32_t G = grown_in(F, S);
    bool ch = G != F;
    F = G;
    if (ballot(ch) == 0ull) break;
  }
  return F;
}

// ------------------------------------------------------------------------------------------------
// lane bookkeeping
// ------------------------------------------------------------------------------------------------
template <int N>
struct Lane {
  int lane, j, r, b;     // lane id, board slot in the wavefront, row, index of the board in the call (outputs, actions)
  int slot;              // index of the environment whose state this board is (= b except in the slot kernels)
  int some;              // an environment that exists, near this one's: what a lane without a board loads in its place
  bool valid;            // this lane holds a real row of a real board
  bool boardok;          // slot j holds a real board (also true for its sentinel lane)
  uint32_t seglo, seghi; // lanes of the rows of this lane's board
  uint32_t full;         // FULL on valid lanes, else 0
  // wb: boards this launch puts into a wavefront (1 .. W; fewer than W trades lanes for latency at small batches)
  __device__ __forceinline__ Lane(int wave, int lane_, int B, int wb = Geo<N>::W) {
    using G = Geo<N>;
    lane = lane_;
    j = lane / G::STRIDE;
    int rr = lane - j * G::STRIDE;
    r = rr - 1;
    b = wave * wb + j;
    slot = b;
    some = wave * wb < B ? wave * wb : 0;
    boardok = (j < wb) && (b < B);
    valid = boardok && rr >= 1;
    uint64_t seg = (j < wb) ? (((1ull << N) - 1ull) << (j * G::STRIDE + 1)) : 0ull;
    seglo = (uint32_t)seg; seghi = (uint32_t)(seg >> 32);
    full = valid ? G::FULL : 0u;
  }
};

template <int N>
struct Row {                      // per-lane registers: one row of one board
  uint32_t bk, wt, ab, aw;        // stones and atari sets (stones of chains with exactly one liberty)
  uint32_t ko;                    // the ko point, if it is in this row (place_ko)
};

// ------------------------------------------------------------------------------------------------
// The state of a game in memory, GAME dwords in a row, so that a game met by itself (tree search) is a few neighbouring lines:
//   hist   the history, HIST dwords per row, see below
//   tail   TAIL more dwords per row of it
//   cur    the row's stones and atari set, CUR dwords (an atari stone has its stone's colour, so one set serves both)
// The emission wants the history point by point (Points): 16 bits per point, bit 2i = black i plies ago, bit 2i+1 = white.  Held like
// that in memory a ply rewrites every point that changed within the last eight.
//   9x9: it is held like that, hist is one 16-byte vector per row (columns 0 .. 7), tail column 8, and those that changed are
//     written.
//   19x19 (RINGED): columns 0 .. 15 are held position by position, a dword per row and position (ring_word); the position i plies
//     ago is number (head + i) mod 8, head being kept with the game's scalars, so that a ply overwrites the oldest one and moves
//     the head.  tail holds columns 16 .. 18 point by point.  A ply writes 20 bytes of a row; with everything point by point it was
//     56, or the changed ones of four pieces.  Turning positions into points costs about as many instructions as pushing them did
//     (exchange_columns_and_positions).  Bytes moved per ply of 65536 games 571 -> 521 MB; us per ply, before / since, with what
//     else changed then (this order of a game's pieces, packed atari sets, state_store_kind): 16384 games 20.0 / 19.5, 28000 36.3 / 34.1,
//     65536 81.5 / 78.2, without observation 30.1 / 27.5, 16384 with superko 28.5 / 27.3; 36000 to 40000 games have lost 1 % (44.6
//     / 45.0, 49.1 / 49.7), and plies of one wavefront for everything where its chain counts up to 1.5 % (6489 games 11.2 / 11.35).  At 9x9, where hardly a byte leaves the caches, a ring is 3 to 7 % slower than this.
// As planes over all games instead (every piece one run of all games) a search, which takes games from anywhere, is 3 to 7 % slower
// and 40000 games 5 % faster.
// ------------------------------------------------------------------------------------------------
template <int N>
struct State {                    // where one row of one game lies
  uint32_t *hist, *tail, *cur;
  static constexpr int NEXT = N;  // dwords from one position of the ring to the next
  __device__ __forceinline__ State(uint32_t* base, const Lane<N>& L) {
    using G = Geo<N>;
    // a lane without a row of its own gets some row of the state: its loads need no branch, and it stores nothing.  (A row near
    // by: with the same one for all wavefronts 256 games of 9x9 took 0.1 us more.)
    uint32_t* game = base + (size_t)(uint32_t)(L.boardok ? L.slot : L.some) * G::GAME;
    const int r = L.r > 0 ? L.r : 0;
    hist = game + r * (G::RINGED ? 1 : G::HIST); tail = game + N * G::HIST + r * G::TAIL; cur = game + N * (G::HIST + G::TAIL) + r * G::CUR;
  }
};
template <int N>
struct History {                  // per-lane registers: the history of one row as it lies in memory
  uint32_t s[Geo<N>::HIST], tail[Geo<N>::TAIL];
  uint32_t changed;               // not RINGED: bit 0 / 1 set = hist / tail differs from what memory holds
};
template <int N>
struct Points {                   // column 2j in the low half of h[j], column 2j+1 in the high half
  uint32_t h[Geo<N>::HD];
};

template <int N>
__device__ __forceinline__ void load_row(uint32_t* state, const Lane<N>& L, Row<N>& R) {
  using G = Geo<N>;
  const State<N> S(state, L);
  uint2 v = make_uint2(0u, 0u);
  if constexpr (G::CUR == 2) v = *(const uint2*)S.cur;
  else v.x = *S.cur;
  // black, white and atari set, N bits each, from bit 0 on (a lane without a row: empty)
  const uint32_t at = G::CUR == 2 ? v.y >> (2 * N - 32) : v.x >> (2 * N);
  R.bk = v.x & L.full;
  R.wt = (G::CUR == 2 ? __builtin_amdgcn_alignbit(v.y, v.x, N) : v.x >> N) & L.full;
  R.ab = at & R.bk; R.aw = at & R.wt;
  R.ko = 0u;
}
// (what a lane without a row gets is some other row's history: nothing is done with it)
template <int N>
__device__ __forceinline__ void load_history(uint32_t* state, const Lane<N>& L, History<N>& H) {
  using G = Geo<N>;
  const State<N> S(state, L);
  if constexpr (G::RINGED) {
#pragma unroll
    for (int k = 0; k < 8; ++k) H.s[k] = S.hist[k * S.NEXT];
    const uint2 v = *(const uint2*)S.tail;
    H.tail[0] = v.x; H.tail[1] = v.y;
  } else {
    const uint4 v = *(const uint4*)S.hist;
    H.s[0] = v.x; H.s[1] = v.y; H.s[2] = v.z; H.s[3] = v.w;
    H.tail[0] = *S.tail;
  }
  H.changed = 0u;
}
// The scalars of this lane's game (of some game in a lane without one: every use of them asks for a real board first)
template <int N>
__device__ __forceinline__ uint4 load_meta(const uint4* meta, const Lane<N>& L) { return meta[L.boardok ? L.slot : L.some]; }
// ST: kind of the stores (store_small)
template <int N, int ST = kStorePlain>
__device__ __forceinline__ void store_row(const State<N>& S, const Row<N>& R) {
  const uint32_t at = R.ab | R.aw;
  if constexpr (Geo<N>::CUR == 2) store_small<ST>((uint2*)S.cur, make_uint2(R.bk | (R.wt << N), (R.wt >> (32 - N)) | (at << (2 * N - 32))));
  else store_small<ST>(S.cur, R.bk | (R.wt << N) | (at << (2 * N)));
}
template <int N, int ST = kStorePlain>
__device__ __forceinline__ void store_tail(const State<N>& S, const History<N>& H) {
  if constexpr (Geo<N>::TAIL == 2) store_small<ST>((uint2*)S.tail, make_uint2(H.tail[0], H.tail[1]));
  else store_small<ST>(S.tail, H.tail[0]);
}
// the whole history, the whole state of a row
template <int N>
__device__ __forceinline__ void store_history(uint32_t* state, const Lane<N>& L, const History<N>& H) {
  if (!L.valid) return;
  const State<N> S(state, L);
  store_tail<N>(S, H);
  if constexpr (Geo<N>::RINGED) {
#pragma unroll
    for (int k = 0; k < 8; ++k) S.hist[k * S.NEXT] = H.s[k];
  } else *(uint4*)S.hist = make_uint4(H.s[0], H.s[1], H.s[2], H.s[3]);
}
template <int N>
__device__ __forceinline__ void store_all(uint32_t* state, const Lane<N>& L, const Row<N>& R, const History<N>& H) {
  if (L.valid) store_row<N>(State<N>(state, L), R);
  store_history<N>(state, L, H);
}

// A row's stones with the colours side by side: bits 2j / 2j+1 = black / white at column 2j (lo), at column 2j+1 (hi)
struct Pairs {
  uint32_t lo, hi;
};
__device__ __forceinline__ Pairs pairs_of(uint32_t bk, uint32_t wt) {
  return Pairs{(bk & 0x55555555u) | ((wt & 0x55555555u) << 1), ((bk >> 1) & 0x55555555u) | (wt & 0xAAAAAAAAu)};
}
__device__ __forceinline__ uint32_t pair_dword(const Pairs& p, int j) { return ((p.lo >> (2 * j)) & 3u) | (((p.hi >> (2 * j)) & 3u) << 16); }   // of columns 2j, 2j+1
// columns 0 .. 15 of a row as a dword of the ring: the even ones in the low half, the odd ones in the high half
__device__ __forceinline__ uint32_t ring_word(const Pairs& p) { return (p.lo & 0xFFFFu) | (p.hi << 16); }

// Exchanges, in eight dwords, bit k of the dword's index with bit k + 1 of the bit position within a half (k = 0, 1, 2).  Applied to
// the ring dwords of eight positions, whose halves hold column pair j at bits 2j and 2j+1, it gives in dword j the two bits of
// position i at 2i and 2i+1: Points.  It is its own inverse.
__device__ __forceinline__ void exchange_columns_and_positions(uint32_t (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = x[i], b = x[i + 4];
    x[i] = __builtin_amdgcn_perm(b, a, 0x06020400u);        // bytes a0 b0 a2 b2
    x[i + 4] = __builtin_amdgcn_perm(b, a, 0x07030501u);    // bytes a1 b1 a3 b3
  }
#pragma unroll
  for (int d = 2; d >= 1; d >>= 1) {
    const uint32_t mask = d == 2 ? 0x0F0F0F0Fu : 0x33333333u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & d) continue;
      const uint32_t a = x[i], b = x[i + d];
      x[i] = (a & mask) | ((b << (2 * d)) & ~mask);
      x[i + d] = ((a >> (2 * d)) & mask) | (b & ~mask);
    }
  }
}
// both halves of x rotated right by 2 * head bits
__device__ __forceinline__ uint32_t rotate_halves(uint32_t x, int head) {
  typedef unsigned short halves __attribute__((ext_vector_type(2)));
  const unsigned short right = (unsigned short)(2 * head), left = (unsigned short)((16 - 2 * head) & 15);
  const halves v = __builtin_bit_cast(halves, x);
  return __builtin_bit_cast(uint32_t, (halves)((v >> halves{right, right}) | (v << halves{left, left})));
}
template <int N>
__device__ __forceinline__ Points<N> points_of(const History<N>& H, int head) {
  using G = Geo<N>;
  Points<N> Q;
  uint32_t x[G::HIST];
#pragma unroll
  for (int k = 0; k < G::HIST; ++k) x[k] = H.s[k];
  if constexpr (G::RINGED) {
    exchange_columns_and_positions(x);
#pragma unroll
    for (int k = 0; k < G::HIST; ++k) x[k] = rotate_halves(x[k], head);
  }
#pragma unroll
  for (int j = 0; j < G::HD; ++j) Q.h[j] = j < G::HIST ? x[j < G::HIST ? j : 0] : H.tail[j < G::HIST ? 0 : j - G::HIST];
  return Q;
}
// the inverse, with the ring's head at 0
template <int N>
__device__ __forceinline__ History<N> history_of(const Points<N>& Q) {
  using G = Geo<N>;
  History<N> H;
#pragma unroll
  for (int k = 0; k < G::HIST; ++k) H.s[k] = Q.h[k];
  if constexpr (G::RINGED) exchange_columns_and_positions(H.s);
#pragma unroll
  for (int k = 0; k < G::TAIL; ++k) H.tail[k] = Q.h[G::HIST + k];
  H.changed = ~0u;
  return H;
}

// a6: the position (bk, wt) becomes the newest one of a board that moved
// (which: all ones on a board that moved, else 0.  A mask and not a condition: the compiler would make branches of it, 4 % of a rollout)
__device__ __forceinline__ uint32_t mask_of(bool which) { return in_place(which ? ~0u : 0u); }
__device__ __forceinline__ uint32_t pushed(uint32_t h, const Pairs& p, int j, uint32_t which) {
  const uint32_t v = ((h << 2) & 0xFFFCFFFCu) | pair_dword(p, j);
  return (v & which) | (h & ~which);
}
template <int N>
__device__ __forceinline__ void push_points(Points<N>& Q, uint32_t bk, uint32_t wt, bool moved) {
  const Pairs p = pairs_of(bk, wt);
  const uint32_t which = mask_of(moved);
#pragma unroll
  for (int j = 0; j < Geo<N>::HD; ++j) Q.h[j] = pushed(Q.h[j], p, j, which);
}
template <int N>
__device__ __forceinline__ void push_history(History<N>& H, int& head, uint32_t bk, uint32_t wt, bool moved) {
  using G = Geo<N>;
  const Pairs p = pairs_of(bk, wt);
  const uint32_t which = mask_of(moved);
  if constexpr (G::RINGED) {
    const uint32_t word = ring_word(p);
    if (moved) head = (head + 7) & 7;
    const int at = moved ? head : 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) H.s[k] = k == at ? word : H.s[k];
  } else {
    uint32_t dif = 0u;
#pragma unroll
    for (int k = 0; k < G::HIST; ++k) { const uint32_t v = pushed(H.s[k], p, k, which); dif |= v ^ H.s[k]; H.s[k] = v; }
    H.changed |= dif ? 1u : 0u;
  }
#pragma unroll
  for (int k = 0; k < G::TAIL; ++k) { const uint32_t v = pushed(H.tail[k], p, G::HIST + k, which); H.changed |= v != H.tail[k] ? 2u : 0u; H.tail[k] = v; }
}
// The history as a rollout keeps it from ply to ply: by points for the emission, or, AS_STORED, as the ring that memory holds
template <int N, bool AS_STORED>
__device__ __forceinline__ Points<N> kept_history(const History<N>& H, int head) {
  if constexpr (!AS_STORED) return points_of<N>(H, head);
  Points<N> Q;
#pragma unroll
  for (int j = 0; j < Geo<N>::HD; ++j) Q.h[j] = j < Geo<N>::HIST ? H.s[j < Geo<N>::HIST ? j : 0] : H.tail[j < Geo<N>::HIST ? 0 : j - Geo<N>::HIST];
  return Q;
}
template <int N, bool AS_STORED>
__device__ __forceinline__ void push_kept(Points<N>& Q, int& head, uint32_t bk, uint32_t wt, bool moved) {
  using G = Geo<N>;
  if constexpr (!AS_STORED) return push_points<N>(Q, bk, wt, moved);
  const Pairs p = pairs_of(bk, wt);
  const uint32_t word = ring_word(p), which = mask_of(moved);
  if (moved) head = (head + 7) & 7;
  const int at = moved ? head : 8;
#pragma unroll
  for (int k = 0; k < G::HD; ++k) Q.h[k] = k < G::HIST ? (k == at ? word : Q.h[k]) : pushed(Q.h[k], p, k, which);
}
template <int N, bool AS_STORED>
__device__ __forceinline__ History<N> history_of_kept(const Points<N>& Q, int& head) {
  if constexpr (!AS_STORED) { head = 0; return history_of<N>(Q); }
  History<N> H;
#pragma unroll
  for (int k = 0; k < Geo<N>::HIST; ++k) H.s[k] = Q.h[k];
#pragma unroll
  for (int k = 0; k < Geo<N>::TAIL; ++k) H.tail[k] = Q.h[Geo<N>::HIST + k];
  H.changed = ~0u;
  return H;
}
template <int N>
__device__ __forceinline__ void clear_points(Points<N>& Q) {
#pragma unroll
  for (int j = 0; j < Geo<N>::HD; ++j) Q.h[j] = 0u;
}
template <int N>
__device__ __forceinline__ void clear_history(History<N>& H) {
#pragma unroll
  for (int k = 0; k < Geo<N>::HIST; ++k) H.s[k] = 0u;
#pragma unroll
  for (int k = 0; k < Geo<N>::TAIL; ++k) H.tail[k] = 0u;
  H.changed = ~0u;
}
// Kind of the state's stores in a launch whose outputs are stored as OUT.  A launch whose outputs go past the caches is so large that its
// state does not stay in them either, and what it leaves dirty in the L2s (32 MB) would have to be written back at its end: written
// through, 65536 games of 19x19 81.6 -> 79.8 us, 40000 52.6 -> 48.1.  Smaller launches lose 1 to 5 % that way.
constexpr int state_store_kind(int out) { return out == kStoreStreamWhole ? kStoreThrough : kStorePlain; }

// What a ply changes of a row in memory, after push_history and clear_history: nothing unless the board moved or was re-initialised.
template <int N, int ST>
__device__ __forceinline__ void store_ply(uint32_t* state, const Lane<N>& L_, const Row<N>& R, const History<N>& H, int head, bool moved, bool reset) {
  Lane<N> L = L_;
  L.slot = in_place(L.slot); L.r = in_place(L.r);   // (the addresses anew: kept from the loads on they cost the superko kernels registers they do not have)
  if (L.valid && (moved || reset)) {
    const State<N> S(state, L);
    store_row<N, ST>(S, R);
    if constexpr (Geo<N>::RINGED) {
      store_tail<N, ST>(S, H);
      store_small<ST>(&S.hist[head * S.NEXT], ring_word(pairs_of(R.bk, R.wt)));   // zero after a reset, as the others are below
    } else {
      if (H.changed & 1u) store_small<ST>((uint4*)S.hist, make_uint4(H.s[0], H.s[1], H.s[2], H.s[3]));
      if (H.changed & 2u) store_tail<N, ST>(S, H);
    }
  }
  if constexpr (Geo<N>::RINGED) {
    if (ballot(reset) != 0ull && L.valid && reset) {
      const State<N> S(state, L);
#pragma unroll
      for (int k = 0; k < 8; ++k) store_small<ST>(&S.hist[k * S.NEXT], 0u);
    }
  }
}

// the ko point of the loaded scalars as a row word
template <int N>
__device__ __forceinline__ void place_ko(const Lane<N>& L, Row<N>& R, const Meta& m) {
  const int kr = m.ko / N, kc = m.ko - kr * N;
  R.ko = (m.ko >= 0 && L.valid && L.r == kr) ? (1u << kc) : 0u;
}

// legal points of the player to move (Fig. 2 legal_action_mask, pass excluded): empty, not the ko point, and
// next to an empty point, or to an own chain that is not in atari, or to an opposing chain that is
template <int N>
__device__ __forceinline__ uint32_t legal_row(const Lane<N>& L, const Row<N>& R, int wtm) {
  uint32_t E = L.full & ~(R.bk | R.wt);
  uint32_t own = wtm ? R.wt : R.bk, opp = wtm ? R.bk : R.wt;
  uint32_t aown = wtm ? R.aw : R.ab, aopp = wtm ? R.ab : R.aw;
  uint32_t support = E | (own & ~aown) | (opp & aopp);
  return E & ~R.ko & dilate(support);
}

// Legal mask bytes [N*N+1] of every board of the wavefront.  TIGHT: the pitch is the dense one (N*N+1) or the
// line-padded one (A_PAD); the boards of a wavefront are then one contiguous run of bytes, pad bytes included, and
// are staged and written as one stream (the pad bytes as zeros); otherwise board by board, pad bytes untouched.
// FIRST_AS_EDGE: see emit_bytes.
template <int N, bool TIGHT, int ST = kStorePlain, bool FIRST_AS_EDGE = false>
__device__ __forceinline__ void emit_mask(const Lane<N>& L, uint32_t legal, int wave, int B, uint8_t* mask, int64_t mask_pitch,
                                          uint32_t* lds_mask, const uint2* lut, int wb = Geo<N>::W) {
  using G = Geo<N>;
  static_assert(G::W * G::MASK_DW <= 64 && (15 + G::W * G::A_PAD + 31) / 32 <= 64, "mask staging is cleared by one store per lane");
  constexpr bool tight = TIGHT;   // the caller guarantees mask_pitch == N*N+1 or A_PAD
  const uint32_t stride = (uint32_t)mask_pitch;
  const int j = in_place(L.j), row = in_place(L.r);
  const int b0 = wave * wb;
  const int nb = B - b0 < wb ? B - b0 : wb;   // boards of this wavefront
  lds_mask[L.lane] = 0u;
  wave_lds_fence();
  if (L.valid) {
    uint32_t* reg;
    uint32_t head;
    if constexpr (tight) { head = (uint32_t)((uintptr_t)(mask + (int64_t)b0 * mask_pitch) & 15u) + __umul24((uint32_t)j, stride); reg = lds_mask; }
    else { head = (uint32_t)((uintptr_t)(mask + (int64_t)L.b * mask_pitch) & 15u); reg = lds_mask + j * G::MASK_DW; }
    const uint32_t o = head + (uint32_t)(N * row), q = o >> 5, s = o & 31u;
    atomicOr(&reg[q], legal << s);
    if (s + N > 32u) atomicOr(&reg[q + 1], legal >> (32u - s));
    if (L.r == 0) { const uint32_t o2 = head + G::P; atomicOr(&reg[o2 >> 5], 1u << (o2 & 31u)); }   // pass is always legal
  }
  wave_lds_fence();
  if constexpr (tight) {
    emit_bytes<G::W * G::A_PAD, ST, 4, FIRST_AS_EDGE>(lds_mask, lut, mask + (int64_t)b0 * mask_pitch, (uint32_t)nb * stride, L.lane);
  } else {
#pragma unroll
    for (int jj = 0; jj < G::W; ++jj)
      if (jj < nb) emit_bytes<G::A, ST, 4, FIRST_AS_EDGE>(lds_mask + jj * G::MASK_DW, lut, mask + (int64_t)(b0 + jj) * mask_pitch, G::A, L.lane);
  }
  wave_lds_fence();
}

// The observation's bits of one row: 17 bits per point, the point's history halfword seen by the mover (pairs swapped when White
// moves), then the colour bit (Appendix C "Go", Observation); a row is N such pieces back to back.
template <int N>
__device__ __forceinline__ void obs_string(uint32_t (&S)[Geo<N>::NR], const uint32_t (&h)[Geo<N>::HD], int wtm) {
  using G = Geo<N>;
#pragma unroll
  for (int k = 0; k < G::NR; ++k) S[k] = 0u;
  const uint32_t cb = wtm ? 0u : 1u;
  const uint32_t swap = wtm ? 1u : 0u;
#pragma unroll
  for (int jd = 0; jd < G::HD; ++jd) {
    uint32_t w = h[jd];
    w = ((w >> swap) & 0x55555555u) | ((w << swap) & 0xAAAAAAAAu);
    uint32_t lo17 = (w & 0xFFFFu) | (cb << 16);
    uint32_t hi17 = (2 * jd + 1 < N) ? ((w >> 16) | (cb << 16)) : 0u;
    uint32_t low32 = lo17 | (hi17 << 17), high2 = hi17 >> 15;
    const int pos = 34 * jd, k = pos >> 5, sh = pos & 31;
    S[k] |= low32 << sh;
    if (k + 1 < G::NR) S[k + 1] |= sh ? ((low32 >> (32 - sh)) | (high2 << sh)) : high2;
  }
}
template <int N>
__device__ __forceinline__ void clear_obs_stream(uint32_t* lds_obs, int lane) {
  using G = Geo<N>;
  uint4* z = (uint4*)lds_obs;
  const uint32_t zero = in_place(0u);
  constexpr int NZ = G::W * G::OBS_DW / 4;
#pragma unroll
  for (int i = 0; i < (NZ + 63) / 64; ++i)
    if (i * 64 + 63 < NZ || i * 64 + lane < NZ) z[i * 64 + lane] = make_uint4(zero, zero, zero, zero);
}
// Puts a row's bits at bit offset o of the (cleared) stream.  Written as a left shift by u = 1..32 from dword (o-u)/32 on, every
// shifted dword is one funnel shift of two neighbours of S (a shift by 0 would need a special case): T[i] = bits of dword q+i;
// T[0] and T[NI+1..NR] may share their dword with the rows next door.
template <int N>
__device__ __forceinline__ void put_obs_string(uint32_t* reg, const uint32_t (&S)[Geo<N>::NR], uint32_t o) {
  using G = Geo<N>;
  const uint32_t u1 = (o + 31u) & 31u;            // u - 1
  reg += (int32_t)(o - 1u - u1) >> 5;             // dword -1 only when o = 0, and then T[0] = 0 is not written
  const uint32_t sh = 31u - u1;                   // right shift of the (S[i], S[i-1]) pair that equals the left shift by u
  {
    const uint32_t t0 = __builtin_amdgcn_alignbit(S[0], 0u, sh);
    if (t0) atomicOr(&reg[0], t0);
  }
#pragma unroll
  for (int i = 1; i <= G::NR; ++i) {
    const uint32_t hi = (i < G::NR) ? S[i] : 0u;
    const uint32_t t = __builtin_amdgcn_alignbit(hi, S[i - 1], sh);
    if (i <= G::NI) reg[i] = t;
    else if (t) atomicOr(&reg[i], t);
  }
}

// Observation bytes [N][N][17] of every board of the wavefront from the history words h of its rows.  MOST, FIRST_AS_EDGE: see emit_bytes.
template <int N, bool TIGHT, int ST = kStorePlain, int MOST = 4, bool FIRST_AS_EDGE = false>
__device__ __forceinline__ void emit_obs(const Lane<N>& L, const uint32_t (&h)[Geo<N>::HD], int wtm, int wave, int B, uint8_t* obs,
                                         int64_t obs_pitch, uint32_t* lds_obs, const uint2* lut, int wb = Geo<N>::W) {
  using G = Geo<N>;
  static_assert((15 + G::W * G::OBS_PAD + 31) / 32 <= G::W * G::OBS_DW, "one stream for all boards fits the staging area");
  constexpr bool tight = TIGHT;   // the caller guarantees obs_pitch == N*N*17 or OBS_PAD (see emit_mask)
  const uint32_t stride = (uint32_t)obs_pitch;
  const int j = in_place(L.j), row = in_place(L.r);
  const int b0 = wave * wb;
  const int nb = B - b0 < wb ? B - b0 : wb;
  uint32_t S[G::NR];
  obs_string<N>(S, h, wtm);
  clear_obs_stream<N>(lds_obs, L.lane);
  wave_lds_fence();
  if (L.valid) {
    uint32_t* reg;
    uint32_t head;
    if constexpr (tight) { head = (uint32_t)((uintptr_t)(obs + (int64_t)b0 * obs_pitch) & 15u) + __umul24((uint32_t)j, stride); reg = lds_obs; }
    else { head = (uint32_t)((uintptr_t)(obs + (int64_t)L.b * obs_pitch) & 15u); reg = lds_obs + j * G::OBS_DW; }
    put_obs_string<N>(reg, S, head + (uint32_t)(G::ROWBITS * row));
  }
  wave_lds_fence();
  if constexpr (tight) {
    emit_bytes<G::W * G::OBS_PAD, ST, MOST, FIRST_AS_EDGE>(lds_obs, lut, obs + (int64_t)b0 * obs_pitch, (uint32_t)nb * stride, L.lane);
  } else {
#pragma unroll
    for (int jj = 0; jj < G::W; ++jj)
      if (jj < nb) emit_bytes<G::OBS, ST, MOST, FIRST_AS_EDGE>(lds_obs + jj * G::OBS_DW, lut, obs + (int64_t)(b0 + jj) * obs_pitch, G::OBS, L.lane);
  }
  wave_lds_fence();
}

template <int N, bool TIGHT, int ST = kStorePlain, bool FIRST_AS_EDGE = false>
__device__ __forceinline__ void emit_outputs(const Lane<N>& L, const Points<N>& Q, uint32_t legal, int wtm, int wave, int B,
                                             uint8_t* mask, int64_t mask_pitch, uint8_t* obs, int64_t obs_pitch,
                                             uint32_t* lds_mask, uint32_t* lds_obs, const uint2* lut, int wb = Geo<N>::W) {
  if (mask) emit_mask<N, TIGHT, ST, FIRST_AS_EDGE>(L, legal, wave, B, mask, mask_pitch, lds_mask, lut, wb);
  if (obs) emit_obs<N, TIGHT, ST, 4, FIRST_AS_EDGE>(L, Q.h, wtm, wave, B, obs, obs_pitch, lds_obs, lut, wb);
}

// ------------------------------------------------------------------------------------------------
// uniform random legal action: the k-th legal action in ascending order, k = hash mod legal_count
// ------------------------------------------------------------------------------------------------
template <int N>
struct Draw {
  bool pass, point;    // the same in every lane of the board; neither = the environment is still waiting for its start time (action -1)
  uint32_t bit;        // the drawn point in the lane of its row, else 0
  int pos, src;        // its column, in that lane; that lane
  // the action is known to one lane of the board: that of the drawn point, else that of the first row
  __device__ __forceinline__ bool known(const Lane<N>& L) const { return point ? bit != 0u : L.valid && L.r == 0; }
  __device__ __forceinline__ int action(const Lane<N>& L) const { return pass ? Geo<N>::P : point ? L.r * N + pos : -1; }
  // row and column for every lane of the board when `point` (called by all lanes of the wavefront)
  __device__ __forceinline__ int row(const Lane<N>& L) const { return src - (L.j * Geo<N>::STRIDE + 1); }
  __device__ __forceinline__ int column() const { return __shfl(pos, src); }
};

template <int N>
__device__ __forceinline__ Draw<N> draw_action(const Lane<N>& L, uint32_t legal, uint32_t hash, bool wait) {   // hash: env_hash(seed, 0, L.b, t)
  const uint32_t cnt = __popc(legal);
  // legal points in the rows above this one, and on the whole board, from ballots of the bits of cnt
  uint32_t before = 0u, total = 1u;   // pass is always legal
#pragma unroll
  for (int k = 0; (1 << k) <= N; ++k) {
    const uint64_t m = ballot(((cnt >> k) & 1u) != 0u);
    const uint32_t lo = (uint32_t)m & L.seglo, hi = (uint32_t)(m >> 32) & L.seghi;
    before += __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)) << k;
    total += (uint32_t)(__popc(lo) + __popc(hi)) << k;
  }
  const uint32_t k = remainder_of(hash, total);
  // position of the (n+1)-th set bit of the row word by halving (meaningful in the row that holds it)
  uint32_t n = k - before, w = legal, pos = 0u;
#pragma unroll
  for (int width = N > 16 ? 16 : 8; width >= 1; width >>= 1) {
    const uint32_t c = __popc(w & ((1u << width) - 1u));
    if (n >= c) { n -= c; w >>= width; pos += width; }
  }
  const bool mine = L.valid && k >= before && k < before + cnt;
  const uint64_t sel = ballot(mine);
  const uint32_t slo = (uint32_t)sel & L.seglo, shi = (uint32_t)(sel >> 32) & L.seghi;
  const int src = slo ? __ffs(slo) - 1 : 31 + __ffs(shi);   // lane of the chosen row (any lane when pass is drawn)
  Draw<N> d;
  d.pass = !wait && k == total - 1u;
  d.point = !wait && k != total - 1u;
  d.bit = mine && d.point ? 1u << pos : 0u;
  d.pos = (int)pos; d.src = src & 63;
  return d;
}
template <int N>
__device__ __forceinline__ Draw<N> draw_action(const Lane<N>& L, uint32_t legal, uint32_t seed, uint32_t t, bool wait) {
  return draw_action<N>(L, legal, env_hash(seed, 0u, (uint32_t)L.b, t), wait);
}

// ------------------------------------------------------------------------------------------------
// one ply for every board of the wavefront (steps a2-a8); registers in, registers out
// ------------------------------------------------------------------------------------------------
struct Rules {
  uint32_t seed;
  int komi_x2, max_steps, auto_reset;
};

// What a requested action amounts to for a board (the same in every lane of the board).
struct Move {
  bool skip;      // leave the board alone
  bool frozen;    // the game had ended before (no auto-reset): nothing changes, terminated is reported
  bool is_pass, playing, illegal;
  int pr, pc;     // the point when `playing`
  uint32_t bit;   // the same as a row word: in the lane of its row, else 0
  __device__ __forceinline__ void forbid() { playing = false; illegal = true; pr = -100; pc = 0; bit = 0u; }
};
template <int N>
__device__ __forceinline__ uint32_t bit_of(const Lane<N>& L, bool on, int pr, int pc) { return L.valid && on && L.r == pr ? 1u << pc : 0u; }

// a1/a2.  want_pass / want_point(pr,pc), bit_in = that point as a row word: the requested action; anything else is illegal.
// GATE: check the point against the mover's legal set (not needed for actions drawn from that set).
template <int N, bool GATE>
__device__ __forceinline__ Move gate_move(const Lane<N>& L, const Row<N>& R, const Meta& m, bool skip, bool want_pass, bool want_point,
                                          uint32_t bit_in, int pr_in, int pc_in) {
  Move mv;
  mv.skip = skip;
  mv.frozen = !skip && m.term;
  const bool live = !skip && !mv.frozen;
  mv.is_pass = live && want_pass;
  const bool on_board = live && want_point;
  mv.playing = on_board;
  if (GATE) {
    const uint32_t legal_now = legal_row<N>(L, R, m.wtm);
    mv.playing = on_board && board_any((legal_now & bit_in) != 0u, L.seglo, L.seghi);
  }
  mv.illegal = live && !mv.is_pass && !mv.playing;
  mv.pr = mv.playing ? pr_in : -100;
  mv.pc = mv.playing ? pc_in : 0;
  mv.bit = mv.playing ? bit_in : 0u;
  return mv;
}

// a8: back to the initial state of the next episode (Sec. 4.1); the seat is drawn anew.  The history is the caller's to clear.
template <int N>
__device__ __forceinline__ void reset_board(const Lane<N>& L, Row<N>& R, Meta& m, uint32_t seed) {
  R.bk = R.wt = R.ab = R.aw = R.ko = 0u;
  m.ko = -1; m.steps = 0; m.passes = 0; m.wtm = 0; m.term = 0;
  m.episode += 1;
  m.bp = (int)(env_hash(seed, 1u, (uint32_t)in_place(L.slot), m.episode) & 1u);
}

// ------------------------------------------------------------------------------------------------
// Board-wide sums through LDS: every row lane adds its value to its board's 8-byte cell, every lane reads the sum back
// (a wavefront's LDS operations execute in program order, so no barrier is needed).  A board has two cells, used in turn: each sum leaves
// the other one cleared for the next.
// (The sums used to be ballots masked with the board's lanes, per flood and per lane: 39 instructions for a look at one flood,
// against 14 and one round trip to LDS for all five.)
// ------------------------------------------------------------------------------------------------
constexpr int kBlindSteps = 4;   // growth steps between two looks at the liberties (9x9 and 19x19: 2 and 3 are slower, 6 the same)
constexpr int kTallyCells = 16;  // of a wavefront: two for each of up to eight boards (Geo::W of them, and the lanes beyond)
struct TallyCells {
  uint64_t cell[kTallyCells];
};
class Tally {
  uint64_t* cells_;   // of the block
  uint32_t at_;       // the present one of the wavefront's first board, the same in every lane
  uint32_t board_;
  __device__ __forceinline__ uint64_t* present() const { return cells_ + (at_ + board_); }

 public:
  // later: it is cleared by a call, before the first sum
  template <int N>
  __device__ __forceinline__ Tally(TallyCells* of_block, int wavefront, const Lane<N>& L, bool later = false)
      : cells_(of_block->cell), at_((uint32_t)(kTallyCells * wavefront)), board_((uint32_t)L.j) {
    static_assert(63 / Geo<N>::STRIDE < kTallyCells / 2, "a cell for every board and for the lanes beyond them");
    if (!later) clear();
  }
  __device__ __forceinline__ void clear() {
    present()[0] = 0u;
    present()[kTallyCells / 2] = 0u;
    wave_lds_fence();
  }
  // the sum of v over the rows of this lane's board (called by all lanes)
  __device__ __forceinline__ uint64_t operator()(uint64_t v) {
    __hip_atomic_fetch_add(present(), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    const uint64_t sum = __hip_atomic_load(present(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    at_ ^= (uint32_t)(kTallyCells / 2);
    __hip_atomic_store(present(), (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    return sum;
  }
};

// The five floods of a ply (the new stone's chain and its four opposing neighbours) side by side.  At 9x9 a dword holds a row
// of three floods in fields of ten bits (the tenth is always zero in the sets the floods run in, so that nothing crosses
// between fields), which makes two words of five, and the sixth field has room for the flood that takes chains out of the mover's
// atari set; at 19x19 every flood has its own word, and a word no board of the wavefront needs any more is left out.  Liberty counts are fields of ten bits in both cases: floods 0-2 in the low half of the sum, 3
// and 4 in the high half.
// What bounds a ply of few games is this chain of instructions (one wavefront per SIMD issues one every four cycles).  Against
// five separate floods with a ballot each: 9x9 x 5001 games, 64 plies in one launch without observation 192 -> 118 us; 9x9 x
// 4096, one launch per ply 7.4 -> 6.0 us, x 256 6.3 -> 5.4; 19x19 x 1000, draw and ply 9.9 -> 9.2.  Both words' growth side by side, the sixth flood in
// place of a loop of its own, a draw with one slow product instead of four (remainder_of) and the end of a game out of the way of the usual ply:
// the same 64 plies, by teams since, 88.4 -> 82.6; 8 plies of 9x9 x 4096 39.5 -> 38.6.
template <int N>
struct Floods {
  static constexpr bool PACKED = N == 9;
  static constexpr int WORDS = PACKED ? 2 : 5;
  static_assert(N * N < 512, "a count and the bias below fit a field");
  static constexpr uint32_t kOnes = 1u | (1u << 10) | (1u << 20);
  static __device__ __forceinline__ void spread(uint32_t (&w)[WORDS], uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, uint32_t x4, uint32_t x5) {
    if constexpr (PACKED) { w[0] = x0 | (x1 << 10) | (x2 << 20); w[1] = x3 | (x4 << 10) | (x5 << 20); }
    else { w[0] = x0; w[1] = x1; w[2] = x2; w[3] = x3; w[4] = x4; }
  }
  static __device__ __forceinline__ uint32_t sixth(const uint32_t (&w)[WORDS]) { return w[1] >> 20; }   // PACKED only
  // kBlindSteps growth steps of both words and the halves of one more
  static __device__ __forceinline__ void grow_both(uint32_t (&F)[WORDS], const uint32_t (&S)[WORDS], Halves& d0, Halves& d1) {
    static_assert(kBlindSteps == 4, "what grow_pair does");
    grow_pair(F[0], F[1], S[0], S[1], d0, d1);
  }
  // puts the counts of word k's floods into this row's fields
  static __device__ __forceinline__ void count(int k, uint32_t w, uint32_t& lo, uint32_t& hi) {
    if constexpr (PACKED) {
      if (k == 0) lo = __popc(w & 0x3FFu) + (__popc(w & (0x3FFu << 10)) << 10) + (__popc(w >> 20) << 20);
      else hi = __popc(w & 0x3FFu) + (__popc(w >> 10) << 10);
    } else {
      uint32_t& half = k < 3 ? lo : hi;
      const int at = 10 * (k < 3 ? k : k - 3);
      half = (half & ~(0x3FFu << at)) | (__popc(w) << at);
    }
  }
  static __device__ __forceinline__ uint32_t all(uint32_t x, int bit) { return (uint32_t)((int32_t)(x << (31 - bit)) >> 31); }   // every bit = bit `bit` of x
  // bit 9 of every field whose value is at least `least` (1 or 2)
  static __device__ __forceinline__ uint32_t reached(uint32_t fields, uint32_t least) { return (fields + kOnes * (512u - least)) & (kOnes << 9); }
  // takes the floods that have seen two liberties out of the sets of stones just reached
  static __device__ __forceinline__ void undecided(uint32_t (&open)[WORDS], uint64_t libs) {
    const uint32_t lo = reached((uint32_t)libs, 2u), hi = reached((uint32_t)(libs >> 32), 2u);
    if constexpr (PACKED) {
      open[0] &= ~(lo - (lo >> 9)); open[1] &= ~(hi - (hi >> 9));
    } else {
      open[0] &= ~all(lo, 9); open[1] &= ~all(lo, 19); open[2] &= ~all(lo, 29); open[3] &= ~all(hi, 9); open[4] &= ~all(hi, 19);
    }
  }
  // adds the chains with exactly one liberty to the atari sets
  static __device__ __forceinline__ void atari(const uint32_t (&F)[WORDS], uint64_t libs, uint32_t& aown, uint32_t& aopp) {
    const uint32_t lo = reached((uint32_t)libs ^ kOnes, 1u) ^ (kOnes << 9), hi = reached((uint32_t)(libs >> 32) ^ kOnes, 1u) ^ (kOnes << 9);
    if constexpr (PACKED) {
      const uint32_t a = F[0] & (lo - (lo >> 9)), b = F[1] & (hi - (hi >> 9));
      aown |= a & 0x1FFu;
      aopp |= ((a >> 10) & 0x1FFu) | (a >> 20) | (b & 0x1FFu) | (b >> 10);
    } else {
      aown |= F[0] & all(lo, 9);
      aopp |= (F[1] & all(lo, 19)) | (F[2] & all(lo, 29)) | (F[3] & all(hi, 9)) | (F[4] & all(hi, 19));
    }
  }
};

// What one ply did to a board (the same in every lane of the board, but for `captured`)
struct Ply {
  float rew0, rew1;    // rewards by player id
  bool moved;          // a stone was placed or the player passed: the history takes the new position
  bool flag;           // the terminated output: the game ended in this ply, or had ended before
  bool reset;          // the board was re-initialised by auto-reset
  uint32_t captured;   // the stones this ply removed, this row's
};

// a3-a5, a7 and a8 for every board of the wavefront; registers in, registers out.  a6, the history, is the caller's: clear() is
// called, with the lanes concerned, where a board is re-initialised (a push of the then empty board leaves a cleared history as it is).
struct NothingToClear {
  __device__ __forceinline__ void operator()() const {}
};
// RARE_IN_LINE: the end of a game stands among the rest.  Out of the way it saves the usual ply its jumps, each of them a fetch (9x9, rollouts by single wavefronts, in
// line / out of it: 200 plies of 300 games 194.6 / 189.5 us, 16 of 18000 71.6 / 71.3), but go_rollout_kernel at 19x19 then needs two registers more than it has.
// SIXTH: the flood that clears the mover's atari set runs in the sixth field where there is one, us a ply of 9x9 in a loop of its own / there: x 6000 5.55 / 5.52, x 65536
// without observation 14.46 / 14.38, with the rule at play time x 512 6.51 / 6.45, x 16384 9.67 / 9.63.  With the rule in the mask by single wavefronts the loop is faster at every size:
// two boards per wavefront x 512 7.99 / 8.20, pitches of its own x 1000 8.90 / 9.07, x 20000 14.45 / 14.66, x 50000 without observation 19.38 / 19.65 (search the same:
// 64 entries 11.1 either way, 1024 14.9).
template <int N, bool RARE_IN_LINE = false, bool SIXTH = Floods<N>::PACKED, class Clear = NothingToClear>
__device__ __forceinline__ Ply apply_move(const Lane<N>& L, Row<N>& R, Meta& m, const Rules& cfg, const Move& mv, Tally& tally, Clear&& clear = Clear{}) {
  Ply out;
  using G = Geo<N>;
  const bool playing = mv.playing, is_pass = mv.is_pass, illegal = mv.illegal, frozen = mv.frozen;
  const uint32_t pbit = mv.bit;
  const int wtm0 = m.wtm;
  float rew0 = 0.f, rew1 = 0.f;
  out.captured = 0u;

  // ---- a3-a5: place the stone, capture, update the atari sets, ko ----------------------------------------
  if (ballot(playing) != 0ull) {
    uint32_t own = wtm0 ? R.wt : R.bk, opp = wtm0 ? R.bk : R.wt;
    uint32_t aown = wtm0 ? R.aw : R.ab, aopp = wtm0 ? R.ab : R.aw;
    // (a sentinel lane may get a bit too: none of the sets they are intersected with has stones there)
    const uint32_t nbN = from_lane_above(pbit), nbS = from_lane_below(pbit), nbW = pbit >> 1, nbE = (pbit << 1) & G::FULL;
    const uint32_t nb = nbN | nbS | nbW | nbE;
    const uint32_t friends = nb & own;   // own stones next to the new one
    own |= pbit;
    // opposing chains in atari that touch the new stone lose their last liberty
    int ko_new = -1;
    uint32_t ko_bit = 0u;
    const uint32_t capseed = nb & aopp;
    uint32_t released = nb;   // own chains in atari next to these points stop being that: the new stone joins them, or they gain a liberty
    if (ballot(capseed != 0u) != 0ull) {
      const uint32_t cap = flood_plain(capseed, aopp);
      if (playing) out.captured = cap;
      opp &= ~cap; aopp &= ~cap;
      released |= dilate(cap);
      // simple ko: exactly one stone taken by a stone without friends whose only liberty is the vacated point.  One tally of the
      // stones taken, the new stone's friends and liberties, and the points of the neighbours taken.
      const uint32_t around = (friends | (nb & ~(own | opp))) & L.full;
      const uint32_t where = capseed ? (uint32_t)(L.r * N + __ffs(capseed) - 1) : 0u;
      const uint64_t sum = tally((uint64_t)(__popc(cap) | (__popc(around) << 16)) | ((uint64_t)where << 32));
      if ((uint32_t)sum == 0x10001u) { ko_new = (int)(sum >> 32); ko_bit = cap; }
    }
    const uint32_t E = L.full & ~(own | opp);
    const uint32_t clrseed = released & aown;
    if (!SIXTH && ballot(clrseed != 0u) != 0ull) aown &= ~flood_plain(clrseed, aown);   // (else below)
    // Liberty class of the new stone's chain (flood 0, through own stones) and of the surviving opposing neighbour chains,
    // which lost the liberty just filled (floods 1-4, through opposing stones).  A flood is decided as soon as two
    // liberties are known; one that converges with a single liberty has found a whole chain in atari.
    using FL = Floods<N>;
    uint32_t F[FL::WORDS], S[FL::WORDS], EE[FL::WORDS];
    FL::spread(F, pbit, nbN & opp, nbS & opp, nbW & opp, nbE & opp, SIXTH ? clrseed : 0u);
    FL::spread(S, own, opp, opp, opp, opp, aown);
    FL::spread(EE, E, E, E, E, E, 0u);   // (the sixth flood counts no liberties and so runs until it stops growing)
    uint64_t libs;                 // liberties seen per flood, FL::count's fields
    uint32_t lo = 0u, hi = 0u;     // this row's part of them
    uint32_t open[FL::WORDS];
    bool run[FL::WORDS];   // a flood of this word is under way in some board of the wavefront
#pragma unroll
    for (int k = 0; k < FL::WORDS; ++k) run[k] = FL::PACKED || ballot(F[k] != 0u) != 0ull;
    for (;;) {
      [[maybe_unused]] Halves both[2];
      if constexpr (FL::PACKED) FL::grow_both(F, S, both[0], both[1]);
#pragma unroll
      for (int k = 0; k < FL::WORDS; ++k) {
        open[k] = 0u;
        if (!run[k]) continue;
        if constexpr (!FL::PACKED) {
#pragma unroll
          for (int i = 0; i < kBlindSteps; ++i) F[k] = grown_in(F[k], S[k]);
        }
        const Halves D = FL::PACKED ? both[FL::PACKED ? k : 0] : grown(F[k]);   // (every flood lies in its S, and S has no point of EE)
        const uint32_t G_ = (D.a | D.b) & S[k];
        open[k] = G_ ^ F[k];
        FL::count(k, (D.a | D.b) & EE[k], lo, hi);
        F[k] = G_;
      }
      libs = tally((uint64_t)lo | ((uint64_t)hi << 32));
      FL::undecided(open, libs);
      bool any = false;
      if constexpr (FL::PACKED) any = ballot((open[0] | open[1]) != 0u) != 0ull;
      else {
#pragma unroll
        for (int k = 0; k < FL::WORDS; ++k) { run[k] = ballot(open[k] != 0u) != 0ull; any = any || run[k]; }
      }
      if (!any) break;
    }
    if constexpr (SIXTH) aown &= ~FL::sixth(F);
    FL::atari(F, libs, aown, aopp);
    if (playing) {
      m.ko = ko_new; R.ko = ko_bit;
      R.bk = wtm0 ? opp : own; R.wt = wtm0 ? own : opp;
      R.ab = wtm0 ? aopp : aown; R.aw = wtm0 ? aown : aopp;
    }
  }
  const bool moved = playing || is_pass;
  if (is_pass) { m.ko = -1; R.ko = 0u; m.passes += 1; }
  if (playing) m.passes = 0;
  if (moved) {
    m.steps += 1;
    m.wtm ^= 1;
  }
  // ---- a7: termination and Tromp-Taylor area score ------------------------------------------------------
  const bool score = moved && (m.passes >= 2 || m.steps >= cfg.max_steps);
  const bool ended = score || illegal;
  out.reset = ended && cfg.auto_reset != 0;
  out.moved = moved; out.flag = ended || frozen;
  const bool usual = ballot(ended) == 0ull;
  if (RARE_IN_LINE ? usual : __builtin_expect(usual, true)) { out.rew0 = 0.f; out.rew1 = 0.f; return out; }
  if (ballot(score) != 0ull) {
    const uint32_t E = L.full & ~(R.bk | R.wt);
    const uint32_t rb = flood_plain(E & dilate(R.bk), E);
    const uint32_t rw = flood_plain(E & dilate(R.wt), E);
    // per-board sum of (black area - white area) of the rows, from ballots of the bits of a biased row value
    const uint32_t v = (uint32_t)(__popc(R.bk | (rb & ~rw)) - __popc(R.wt | (rw & ~rb)) + N);   // 0 .. 2N
    int sum = -N * N;
#pragma unroll
    for (int k = 0; (1 << k) <= 2 * N; ++k) {
      const uint64_t mk = ballot(((v >> k) & 1u) != 0u);
      sum += (__popc((uint32_t)mk & L.seglo) + __popc((uint32_t)(mk >> 32) & L.seghi)) << k;
    }
    if (score) {
      int d = 2 * sum - cfg.komi_x2;   // komi counts for White
      float s = d > 0 ? 1.f : (d < 0 ? -1.f : 0.f);
      rew0 = m.bp == 0 ? s : -s;
      rew1 = -rew0;
    }
  }
  if (illegal) {  // the offender loses at once, the position stays
    const int mover = wtm0 ? 1 - m.bp : m.bp;
    rew0 = mover == 0 ? -1.f : 1.f;
    rew1 = -rew0;
    m.illegal += 1;
  }
  if (ended) {
    m.term = 1;
    if (cfg.auto_reset) { reset_board<N>(L, R, m, cfg.seed); clear(); }   // a8 (Sec. 4.1)
  }
  out.rew0 = rew0; out.rew1 = rew1;
  return out;
}

// ------------------------------------------------------------------------------------------------
// the step kernel: one launch = one ply of every environment
// ------------------------------------------------------------------------------------------------
struct StepArgs {            // what is not needed before the first loads
  float* rew;
  uint8_t* term;
  uint8_t* mask;
  uint8_t* obs;
  int64_t mask_pitch, obs_pitch;
  int store_kind;            // kind of the output stores, by the bytes the launch writes (store_kind_for)
  Rules rules;
  // fused sampler
  uint32_t sample_seed, sample_t;
  int32_t* next_actions;
};

template <int N, bool SAMPLE, bool TIGHT, int ST>
__global__ void __launch_bounds__(64 * kWavesPerBlock, 6) go_step_kernel(uint32_t* state, uint4* meta, const int32_t* actions, const int32_t* start_t, int B,
                                                                        int wb, uint32_t eighth, StepArgs a) {   // wb: boards per wavefront of this launch
  using G = Geo<N>;
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs_all[kWavesPerBlock][G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask_all[kWavesPerBlock][64];
  __shared__ TallyCells tally_all[kWavesPerBlock];
  __shared__ uint2 lut[256];
  const int wib = wave_in_block();
  const int wave = piece_of_block(eighth) * kWavesPerBlock + wib;
  const Lane<N> L(wave, threadIdx.x & 63, B, wb);   // in a wavefront beyond the batch no lane is valid

  // the loads are issued first and fly while the block fills its lookup table
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  load_history<N>(state, L, H);
  const uint4 meta_raw = load_meta<N>(meta, L);
  const int act_raw = actions[L.boardok ? L.b : L.some], act = L.boardok ? act_raw : -1;
  // loaded here and not where it is used: a load after the output stores would have to wait for them (one counter);
  // looked at only after the table is filled, so that no wait for a load comes before the barrier
  const int32_t start_raw = (SAMPLE && L.boardok && start_t) ? start_t[L.b] : INT32_MIN;
  in_scalar_registers(a.rew, a.term, a.mask, a.obs, a.mask_pitch, a.obs_pitch, a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset);
  if (SAMPLE) in_scalar_registers(a.sample_seed, a.sample_t, a.next_actions);
  fill_spread_table(lut);
  if (wave * wb >= B) return;   // whole wavefront idle; there is no block-wide barrier anywhere below
  const bool wait_start = (int64_t)a.sample_t < (int64_t)held_back(start_raw);
  Meta m = unpack_meta(meta_raw);
  place_ko<N>(L, R, m);

  // a1/a2: decode the action and gate it
  const bool skip = !L.boardok || act == -1;
  const bool in_range = act >= 0 && act < G::P;
  const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
  const Move mv = gate_move<N, true>(L, R, m, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc);

  // a3-a8
  Tally tally(tally_all, wib, L);
  const Ply ply = apply_move<N>(L, R, m, a.rules, mv, tally, [&]() { clear_history<N>(H); });
  push_history<N>(H, m.head, R.bk, R.wt, ply.moved);
  if (!skip && L.valid && L.r == 0) {
    *(float2*)(a.rew + 2 * (size_t)L.b) = make_float2(ply.rew0, ply.rew1);
    store_small<ST>(&a.term[L.b], (uint8_t)(ply.flag ? 1 : 0));
  }

  // ---- a10 / a9: observation and legal mask of the player now to move ---------------------------------------
  if (a.obs) emit_obs<N, TIGHT, ST>(L, points_of<N>(H, m.head).h, m.wtm, wave, B, a.obs, a.obs_pitch, lds_obs_all[wib], lut, wb);
  const uint32_t legal = legal_row<N>(L, R, m.wtm);
  if (a.mask) emit_mask<N, TIGHT, ST>(L, legal, wave, B, a.mask, a.mask_pitch, lds_mask_all[wib], lut, wb);

  // ---- a11: store the state --------------------------------------------------------------------------------
  store_ply<N, state_store_kind(ST)>(state, L, R, H, m.head, ply.moved, ply.reset);
  if (!skip && L.valid && L.r == 0) store_small<state_store_kind(ST)>(&meta[L.b], pack_meta(m));
  if (SAMPLE) {
    const Draw<N> d = draw_action<N>(L, legal, a.sample_seed, a.sample_t, wait_start);
    if (d.known(L)) a.next_actions[L.b] = d.action(L);
  }
}

// ------------------------------------------------------------------------------------------------
// The same ply by TEAMS, for batches that leave most of the machine empty.  A block is a team: four wavefronts that share one
// group of boards.  One applies the rules; the others load what they need meanwhile and, once it has left the new position in LDS,
// one of them writes the mask, one the observation, one draws the next action, and the first stores the state.
// A ply of few games is bound by the chain of instructions of a wavefront that has its SIMD to itself (one every four to five cycles, some
// 1000 of them at 9x9 and 1200 at 19x19): a team's chain is the state's load, the gate and the rules, and then the longest of
// four shorter ones (9x9 x 256 games: a wavefront lives 6600 instead of 9150 cycles).  What the observation's wavefront can do ahead it
// does while the rules run.  Figures, and where the line to the other kernel lies: boards_per_step_team.
// ------------------------------------------------------------------------------------------------
// What the wavefront that applies the rules leaves for the other three: every lane its row, the board's facts in the bits beyond
// column N-1.
template <int N>
struct HandOver {
  static_assert(N <= 20, "flags fit beside a row");
  uint4 v;
  static __device__ __forceinline__ HandOver of(const Row<N>& R, const Meta& m, const Ply& ply) {
    return HandOver{make_uint4(R.bk | (ply.moved ? 1u << 29 : 0u) | (ply.reset ? 1u << 30 : 0u) | ((uint32_t)m.wtm << 31), R.wt, R.ab | R.aw, R.ko)};
  }
  __device__ __forceinline__ Row<N> row() const {
    const uint32_t bk = v.x & Geo<N>::FULL;
    return Row<N>{bk, v.y, v.z & bk, v.z & v.y, v.w};
  }
  __device__ __forceinline__ bool moved() const { return (v.x >> 29) & 1u; }
  __device__ __forceinline__ bool reset() const { return (v.x >> 30) & 1u; }
  __device__ __forceinline__ int wtm() const { return (int)(v.x >> 31); }
  __device__ __forceinline__ uint32_t legal(const Lane<N>& L) const { return legal_row<N>(L, row(), wtm()); }
};
enum TeamRole { kTeamRules = 0, kTeamMask = 1, kTeamDraw = 2, kTeamObs = 3, kTeamWaves = 4 };

// The observation of a team: everything but the ply's own changes is put into the stream beforehand, as if the position were to
// stay as it is (a pass), and the points that do change are corrected in it.  A board for which that was wrong (skipped, illegal, ended)
// has the wavefront build its stream anew.
template <int N, int ST, class Wait>
__device__ __forceinline__ void team_obs(const Lane<N>& L, const Row<N>& before, Points<N> Q, const Meta& m, const uint4* hand, int group, int B, uint8_t* obs,
                                         int64_t obs_pitch, uint32_t* lds_obs, const uint2* lut, int wb, Wait&& wait_for_hand_over) {
  using G = Geo<N>;
  const uint32_t stride = (uint32_t)obs_pitch;
  const int b0 = group * wb, nb = B - b0 < wb ? B - b0 : wb;
  uint8_t* const dst = obs + (int64_t)b0 * obs_pitch;
  const uint32_t at = (uint32_t)((uintptr_t)dst & 15u) + __umul24((uint32_t)L.j, stride) + (uint32_t)(G::ROWBITS * L.r);
  auto build = [&](const Points<N>& P, int wtm) {
    uint32_t S[G::NR];
    obs_string<N>(S, P.h, wtm);
    clear_obs_stream<N>(lds_obs, L.lane);
    wave_lds_fence();
    if (L.valid) put_obs_string<N>(lds_obs, S, at);
    wave_lds_fence();
  };
  Points<N> next = Q;
  push_points<N>(next, before.bk, before.wt, true);
  build(next, m.wtm ^ 1);
  wait_for_hand_over();
  const HandOver<N> in{hand[L.lane]};
  const Row<N> R = in.row();
  const bool as_expected = in.moved() && !in.reset();   // then the other player is to move
  if (ballot(L.valid && !as_expected) != 0ull) {
    if (in.reset()) clear_points<N>(Q);
    push_points<N>(Q, R.bk, R.wt, in.moved());
    build(Q, in.wtm());
  } else {
    const uint32_t db = R.bk ^ before.bk, dw = R.wt ^ before.wt;
    uint32_t d = db | dw;
    while (ballot(d != 0u) != 0ull) {   // the stone played, and those it took
      if (d) {
        const int c = __ffs(d) - 1;
        const uint32_t black = (db >> c) & 1u, white = (dw >> c) & 1u;
        const uint32_t bits = in.wtm() ? white | (black << 1) : black | (white << 1);   // mover's stone, opponent's stone
        const uint32_t o = at + 17u * (uint32_t)c, q = o >> 5, sh = o & 31u;
        atomicXor(&lds_obs[q], bits << sh);
        if (sh == 31u) atomicXor(&lds_obs[q + 1], bits >> 1);
        d &= d - 1u;
      }
    }
    wave_lds_fence();
  }
  emit_bytes<G::W * G::OBS_PAD, ST>(lds_obs, lut, dst, (uint32_t)nb * stride, L.lane);
}

template <int N, bool SAMPLE, int ST>
__global__ void __launch_bounds__(64 * kTeamWaves) go_step_team_kernel(uint32_t* state, uint4* meta, const int32_t* actions, const int32_t* start_t, int B,
                                                                       int wb, uint32_t eighth, StepArgs a) {   // wb: boards per team
  using G = Geo<N>;
  static_assert(64 * kTeamWaves == kBlockThreads, "the table is filled by one entry per thread");
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs[G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask[64];
  __shared__ TallyCells tally_cells;
  __shared__ uint2 lut[256];
  __shared__ uint4 hand[64];
  const int group = piece_of_block(eighth);
  if (group * wb >= B) return;   // the whole block
  const int role = wave_in_block();
  const Lane<N> L(group, threadIdx.x & 63, B, wb);
  auto fill_table = [&]() { const uint32_t x = threadIdx.x; lut[x] = make_uint2(spread4(x & 15u), spread4(x >> 4)); };

  if (role == kTeamRules) {
    rules_first(eighth);
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    const uint4 meta_raw = load_meta<N>(meta, L);
    const int act_raw = actions[L.boardok ? L.b : L.some], act = L.boardok ? act_raw : -1;
    load_history<N>(state, L, H);
    in_scalar_registers(a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset, a.rew, a.term);
    fill_table();
    Meta m = unpack_meta(meta_raw);
    place_ko<N>(L, R, m);
    const bool skip = !L.boardok || act == -1;
    const bool in_range = act >= 0 && act < G::P;
    const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
    const Move mv = gate_move<N, true>(L, R, m, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc);
    Tally tally(&tally_cells, 0, L);
    const Ply ply = apply_move<N>(L, R, m, a.rules, mv, tally, [&]() { clear_history<N>(H); });
    hand[L.lane] = HandOver<N>::of(R, m, ply).v;
    __syncthreads();
    push_history<N>(H, m.head, R.bk, R.wt, ply.moved);
    store_ply<N, kStorePlain>(state, L, R, H, m.head, ply.moved, ply.reset);
    if (!skip && L.valid && L.r == 0) {
      meta[L.b] = pack_meta(m);
      *(float2*)(a.rew + 2 * (size_t)L.b) = make_float2(ply.rew0, ply.rew1);
      a.term[L.b] = (uint8_t)(ply.flag ? 1 : 0);   // (neighbouring teams write bytes of one line: through the L2 it goes to memory with each of them)
    }
  } else if (role == kTeamMask) {
    in_scalar_registers(a.mask, a.mask_pitch);
    fill_table();
    __syncthreads();
    if (a.mask) emit_mask<N, true, ST>(L, HandOver<N>{hand[L.lane]}.legal(L), group, B, a.mask, a.mask_pitch, lds_mask, lut, wb);
  } else if (role == kTeamDraw) {
    const int32_t start_raw = (SAMPLE && L.boardok && start_t) ? start_t[L.b] : INT32_MIN;
    in_scalar_registers(a.sample_seed, a.sample_t, a.next_actions);
    fill_table();
    const uint32_t hash = in_place(env_hash(a.sample_seed, 0u, (uint32_t)L.b, a.sample_t));
    __syncthreads();
    if (SAMPLE) {
      const Draw<N> d = draw_action<N>(L, HandOver<N>{hand[L.lane]}.legal(L), hash, (int64_t)a.sample_t < (int64_t)start_raw);
      if (d.known(L)) a.next_actions[L.b] = d.action(L);
    }
  } else if (a.obs) {
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    load_history<N>(state, L, H);
    const Meta m = unpack_meta(load_meta<N>(meta, L));
    in_scalar_registers(a.obs, a.obs_pitch);
    fill_table();
    team_obs<N, ST>(L, R, points_of<N>(H, m.head), m, hand, group, B, a.obs, a.obs_pitch, lds_obs, lut, wb, [] { __syncthreads(); });
  } else {
    fill_table();
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------------
// positional superko (Appendix C "Go": Tromp-Taylor rules, whose repetition rule forbids a play that recreates
// an earlier whole-board position of the game).  Two readings, chosen by `mode`: 2 = the rule proper, the legal mask
// leaves such plays out; 1 = looked at only when the move is played (the offender loses like for any illegal
// action) while the mask keeps showing the simple-ko set.
//
// Every position is summarised by two 32-bit Zobrist keys, one per colour (XOR of one key per stone of that colour,
// updated from the stones that changed), and its two stone counts.  A play by colour c always gives a position with
// exactly one more stone of colour c, so the earlier positions a play can recreate are those whose count of c is
// (current count + 1): the per-game table (open addressing, linear probing, 8-byte entries = the two keys) holds
// every position twice, once on the probe chain of (black, its black count) and once on that of (white, its white
// count).  Per ply that costs one chain walk to find where the new position goes and one for the next mover's
// forbidden plays.  The latter needs no loop over the legal points: an earlier position q can be recreated by the
// mover's play on p only if q's key of the mover's colour differs from the current one by exactly the key of a stone
// on p, and the stone keys come from an invertible mixer, so every lane inverts the difference of the entry it holds
// and sees at once whether it is a stone key at all (a random 32-bit value is one with probability 2^-22).  Only for
// such an entry -- a genuine near-repetition -- is the rest checked: the other colour's keys must differ by nothing
// (a play that takes nothing) or by exactly the keys of the chains the play takes.  The forbidden plays found when a
// position arises are kept with the game (two points, or a marker to look again), so the next ply's legality gate
// and the getters need no table access.
// Equality of positions = equality of the 64 key bits; the empty board (keys 0,0 = an empty slot) is never stored
// and can never be recreated.
// ------------------------------------------------------------------------------------------------
template <int N>
struct Zt {
  static constexpr int LOG2 = N == 19 ? 11 : 9;
  static constexpr uint32_t SLOTS = 1u << LOG2;
  static constexpr uint32_t MASK = SLOTS - 1u;
  static constexpr uint32_t WIN = N >= 16 ? 16u : 8u;   // slots a board's row lanes look at per round: one aligned 128- or 64-byte piece of the table
  static_assert(SLOTS > 2u * (2u * N * N + 9u), "two entries per position (ply cap + the imported history window) always leave empty slots");
};

// key of a stone: an invertible function of 2*point + colour + 1 (colour 0 black / 1 white)
__device__ __forceinline__ uint32_t zkey(uint32_t point, uint32_t colour) { return mixer(0x9E3779B9u * (2u * point + colour + 1u)); }
// 2*point + colour + 1 for a stone key, anything else for other values
__device__ __forceinline__ uint32_t zkey_inverse(uint32_t x) {
  x ^= x >> 16; x *= 0x43021123u;               // the mixer's steps undone in reverse order (odd multipliers are invertible mod 2^32)
  x ^= (x >> 15) ^ (x >> 30); x *= 0x1d69e2a5u;
  x ^= x >> 16;
  return x * 0x144cbc89u;                        // 0x9E3779B9^-1
}

// Keys (x: black stones, y: white stones) and stone counts of a game's current position, and the plays that would
// recreate an earlier position (fw: two points in 16 bits each, kNoPoint = none; kLookAgain in the low half = more than
// two, to be found by walking the table again).  The same in every lane of the board.
struct SkGame {
  uint2 key;
  int nb, nw;
  uint32_t fw;
};
constexpr uint32_t kNoPoint = 0xFFFFu, kLookAgain = 0xFFFEu;
__device__ __forceinline__ SkGame sk_unpack(uint4 v) {
  SkGame g;
  g.key = make_uint2(v.x, v.y); g.nb = (int)(v.z & 0xFFFFu); g.nw = (int)(v.z >> 16); g.fw = v.w;
  return g;
}
__device__ __forceinline__ uint4 sk_pack(const SkGame& g) { return make_uint4(g.key.x, g.key.y, (uint32_t)g.nb | ((uint32_t)g.nw << 16), g.fw); }
__device__ __forceinline__ SkGame sk_fresh() {   // a game on the empty board
  SkGame g;
  g.key = make_uint2(0u, 0u); g.nb = 0; g.nw = 0; g.fw = kNoPoint | (kNoPoint << 16);
  return g;
}

// a table entry is the position's two keys; (0,0) is an empty slot
__device__ __forceinline__ bool sk_real(uint2 e) { return (e.x | e.y) != 0u; }
// start of the probe chain of the positions whose count of `colour` stones is `count`
template <int N>
__device__ __forceinline__ uint32_t sk_home(int colour, int count) {
  return (((uint32_t)(2 * count + colour + 1) * 0x9E3779B1u) >> (32 - Zt<N>::LOG2)) & ~(Zt<N>::WIN - 1u);
}
// the same for the play-time reading (mode 1), where a position has one entry, on the chain of its two stone counts
template <int N>
__device__ __forceinline__ uint32_t sk_home_counts(int nb, int nw) {
  return (((uint32_t)((nb << 10) + nw + 1) * 0x9E3779B1u) >> (32 - Zt<N>::LOG2)) & ~(Zt<N>::WIN - 1u);
}
// Table accesses go to the device-coherent level: a wavefront of the rollout kernel reads in a later ply what its own
// lanes wrote in an earlier one.
__device__ __forceinline__ uint2 tab_load(const uint2* p) {
  const unsigned long long v = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void tab_store(uint2* p, uint2 e) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)e.x | ((unsigned long long)e.y << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// orders a wavefront's earlier global-memory accesses before its later ones as seen by its own lanes
__device__ __forceinline__ void wave_mem_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// XOR of the keys of the stones of row r: x over the black bits, y over the white bits
template <int N>
__device__ __forceinline__ uint2 row_keys(int r, uint32_t black, uint32_t white) {
  uint2 acc = make_uint2(0u, 0u);
  for (uint32_t d = black; d; d &= d - 1u) acc.x ^= zkey((uint32_t)(r * N + __ffs(d) - 1), 0u);
  for (uint32_t d = white; d; d &= d - 1u) acc.y ^= zkey((uint32_t)(r * N + __ffs(d) - 1), 1u);
  return acc;
}

// every lane of a board receives the XOR of v over the board's rows; scratch = 2*W dwords of the wavefront's LDS
template <int N>
__device__ __forceinline__ uint2 board_xor(const Lane<N>& L, uint2 v, uint32_t* scratch) {
  using G = Geo<N>;
  if (L.lane < 2 * G::W) scratch[L.lane] = 0u;
  wave_lds_fence();
  if (L.valid && (v.x | v.y) != 0u) { atomicXor(&scratch[2 * L.j], v.x); atomicXor(&scratch[2 * L.j + 1], v.y); }
  wave_lds_fence();
  uint2 out = make_uint2(0u, 0u);
  if (L.j < G::W) out = make_uint2(scratch[2 * L.j], scratch[2 * L.j + 1]);
  wave_lds_fence();
  return out;
}

// number of set bits of a board-wide set given by its row words, known to every lane of the board
template <int N>
__device__ __forceinline__ int board_popcount(const Lane<N>& L, uint32_t w) {
  const uint32_t v = __popc(w);
  int sum = 0;
#pragma unroll
  for (int k = 0; (1 << k) <= N; ++k) {
    const uint64_t mk = ballot(((v >> k) & 1u) != 0u);
    sum += (__popc((uint32_t)mk & L.seglo) + __popc((uint32_t)(mk >> 32) & L.seghi)) << k;
  }
  return sum;
}

// The WIN table slots from `home` on, one per row lane, loaded ahead of their use (home = ~0u: nothing loaded)
struct SkWin {
  uint32_t home;
  uint2 e;
};
template <int N>
__device__ __forceinline__ SkWin sk_window(const Lane<N>& L, const uint2* tab, uint32_t home, bool want) {
  SkWin w;
  w.home = want ? home : ~0u;
  w.e = make_uint2(1u, 0u);   // neither empty nor a real entry
  if (L.valid && want && (uint32_t)L.r < Zt<N>::WIN) w.e = tab_load(&tab[(home + (uint32_t)L.r) & Zt<N>::MASK]);
  return w;
}

// Walks the probe chain that starts at `home` (the same for every lane of a board; active = this board takes part),
// WIN slots per round, one per row lane, until the chain's first empty slot.  visit(e, look) is called once per round
// by every lane of the wavefront with the lane's entry (look = the lane holds a slot of an active board's chain).
// free_slot = the first empty slot other than `taken` (a slot this ply has filled already; ~0u = none); ok = found,
// which is always the case since the table is never full.  pre: a window loaded earlier, used when it starts at `home`.
template <int N, class V>
__device__ __forceinline__ void sk_walk(const Lane<N>& L, const uint2* tab, uint32_t home, bool active, const SkWin& pre, uint32_t taken, V&& visit,
                                        bool& ok, uint32_t& free_slot) {
  using G = Geo<N>;
  constexpr uint32_t WIN = Zt<N>::WIN;
  const uint64_t seg = ((uint64_t)L.seghi << 32) | L.seglo;
  ok = false; free_slot = 0u;
  bool done = !active;
  uint32_t base = home;
  for (uint32_t round = 0; round < Zt<N>::SLOTS / WIN + 1u; ++round) {
    if (ballot(!done) == 0ull) break;
    const bool look = L.valid && (uint32_t)L.r < WIN && !done;
    uint2 e = make_uint2(1u, 0u);
    const uint32_t slot = (base + (uint32_t)L.r) & Zt<N>::MASK;
    const bool from_pre = round == 0u && pre.home == base;
    if (look && from_pre) e = pre.e;
    if (ballot(look && !from_pre) != 0ull) {   // a branch of the whole wavefront: most walks end in the window loaded ahead
      if (look && !from_pre) e = tab_load(&tab[slot]);
      // the wait for this load stays inside the branch: after it, it would also be a wait for the caller's output stores
      asm volatile("" : "+v"(e.x), "+v"(e.y));
    }
    if (look && slot == taken && (e.x | e.y) == 0u) e = make_uint2(1u, 0u);
    visit(e, look);
    const uint64_t em = ballot(look && (e.x | e.y) == 0u) & seg;
    if (!done) {
      if (em) { free_slot = (base + (uint32_t)(__ffsll((long long)em) - 1 - (L.j * G::STRIDE + 1))) & Zt<N>::MASK; ok = true; done = true; }
      else base += WIN;
    }
  }
}

// What placing a stone does to the game's key set (the same in every lane of the board).
struct SkPly {
  uint2 key;        // keys and counts of the position after the ply (meaningful for a board that placed a stone)
  int nb, nw;
  bool ok;          // free_a is valid
  uint32_t free_a;  // where the position goes on the chain of the mover's colour
};

// After the rules have been applied to a board that placed a stone (colour c, stones `captured` taken): the new
// position's keys and counts, and the free slot on its first chain.
template <int N>
__device__ __forceinline__ SkPly sk_look(const Lane<N>& L, const uint2* tab, const SkGame& g, int c, const Move& mv, uint32_t captured,
                                         const SkWin& pre, uint32_t* scratch) {
  SkPly s;
  const bool played = mv.playing;
  const uint32_t kp = zkey((uint32_t)(played ? mv.pr * N + mv.pc : 0), (uint32_t)c);
  int ncap = 0;
  uint2 dk = make_uint2(0u, 0u);
  if (ballot(captured != 0u) != 0ull) {   // the captured stones have the other colour
    ncap = board_popcount<N>(L, captured);
    dk = board_xor<N>(L, row_keys<N>(L.r, c ? captured : 0u, c ? 0u : captured), scratch);
  }
  const int own1 = (c ? g.nw : g.nb) + 1, opp1 = (c ? g.nb : g.nw) - ncap;
  s.key = make_uint2(g.key.x ^ (c ? 0u : kp) ^ dk.x, g.key.y ^ (c ? kp : 0u) ^ dk.y);
  s.nb = c ? opp1 : own1; s.nw = c ? own1 : opp1;
  sk_walk<N>(L, tab, sk_home<N>(c, own1), played, pre, ~0u, [](uint2, bool) {}, s.ok, s.free_a);
  return s;
}

// Writes the position of a board that placed a stone into the table (both chains) and makes it the game's current one.
// tab_r: the table the chains are read from; tab_w: the one the entries go to (they differ only while the slot kernel
// copies a game from one slot to another).
template <int N>
__device__ __forceinline__ void sk_insert(const Lane<N>& L, const uint2* tab_r, uint2* tab_w, SkGame& g, const SkPly& s, bool insert, int c,
                                          const SkWin& pre) {
  if (ballot(insert) == 0ull) return;
  bool ok_c;
  uint32_t free_c;
  const int opp1 = c ? s.nb : s.nw;   // count of the colour that did not move
  sk_walk<N>(L, tab_r, sk_home<N>(c ^ 1, opp1), insert, pre, s.ok ? s.free_a : ~0u, [](uint2, bool) {}, ok_c, free_c);
  if (insert) { g.key = s.key; g.nb = s.nb; g.nw = s.nw; }
  if (insert && L.valid && L.r == 0 && sk_real(s.key)) {
    if (s.ok) tab_store(&tab_w[s.free_a], s.key);
    if (ok_c) tab_store(&tab_w[free_c], s.key);
  }
  wave_mem_fence();
}

// Whether the mover's (colour c2) play on point p would recreate the earlier position whose keys differ from the
// current ones by d_other in the other colour (on = this board has such a candidate); returns the play as row words.
template <int N>
__device__ __forceinline__ uint32_t sk_forbidden_play(const Lane<N>& L, const Row<N>& R, int c2, int p, uint32_t d_other, bool on, uint32_t legal_s,
                                                      uint32_t* scratch) {
  const int pr = on ? p / N : -100, pc = on ? p - (p / N) * N : 0;
  const uint32_t pb = (L.valid && L.r == pr) ? (1u << pc) : 0u;
  const bool legal = on && board_any((legal_s & pb) != 0u, L.seglo, L.seghi);   // an occupied, suicidal or ko point is out anyway
  const uint32_t aopp = c2 ? R.ab : R.aw;
  const uint32_t seed = legal ? (dilate(pb) & aopp) : 0u;    // the opposing chains in atari next to the play are what it takes
  const bool takes = board_any(seed != 0u, L.seglo, L.seghi);
  uint32_t kt = 0u;
  if (ballot(takes) != 0ull) {
    const uint32_t taken = flood_plain(seed, aopp);
    const uint2 k = board_xor<N>(L, row_keys<N>(L.r, c2 ? taken : 0u, c2 ? 0u : taken), scratch);
    kt = c2 ? k.x : k.y;
  }
  return (legal && kt == d_other) ? pb : 0u;
}

// The plays of the player to move that would recreate an earlier position of the game (row words): one walk of the
// chain of the positions with one more stone of the mover's colour than now.  KO_IN_ROW: R's ko bit is up to date and m.ko is not looked at.
template <int N, bool KO_IN_ROW = false>
__device__ __forceinline__ uint32_t sk_forbidden(const Lane<N>& L, const uint2* tab, const SkGame& g, const Row<N>& R, const Meta& m, bool active,
                                                 const SkWin& pre, uint32_t* scratch) {
  uint32_t forb = 0u;
  if (ballot(active) == 0ull) return forb;
  const uint64_t seg = ((uint64_t)L.seghi << 32) | L.seglo;
  const int c2 = m.wtm, n2 = c2 ? g.nw : g.nb;
  bool ok;
  uint32_t fs;
  sk_walk<N>(L, tab, sk_home<N>(c2, n2 + 1), active, pre, ~0u,
             [&](uint2 e, bool look) {
               // is (entry xor current) in the mover's colour the key of one stone of that colour?
               const uint32_t u = zkey_inverse(c2 ? e.y ^ g.key.y : e.x ^ g.key.x) - 1u;   // 2*point + colour for a stone key
               const uint32_t d_other = c2 ? e.x ^ g.key.x : e.y ^ g.key.y;
               uint64_t pend = ballot(look && sk_real(e) && u < 2u * N * N && (int)(u & 1u) == c2);
               if (pend == 0ull) return;          // nearly always: no earlier position is one stone of the mover's away
               Row<N> now = R;   // (its ko bit from the scalars: not held through the table work, which needs the registers)
               if constexpr (!KO_IN_ROW) place_ko<N>(L, now, m);
               const uint32_t legal_s = legal_row<N>(L, now, m.wtm);
               while (pend != 0ull) {             // one candidate per board per turn
                 const uint64_t mine = pend & seg;
                 const bool on = mine != 0ull;
                 const int src = on ? (__ffsll((long long)mine) - 1) : L.lane;
                 const int p = __shfl((int)(u >> 1), src);
                 const uint32_t dq = (uint32_t)__shfl((int)d_other, src);
                 pend &= ~ballot(on && L.lane == src);
                 forb |= sk_forbidden_play<N>(L, R, c2, p, dq, on, legal_s, scratch);
               }
             },
             ok, fs);
  return forb;
}

// the forbidden plays kept with a game -> row words of this lane's board
template <int N>
__device__ __forceinline__ uint32_t sk_forb_rows(const Lane<N>& L, uint32_t fw) {
  const uint32_t p1 = fw & 0xFFFFu, p2 = fw >> 16;
  uint32_t out = 0u;
  if (L.valid && p1 < (uint32_t)(N * N) && (int)(p1 / N) == L.r) out |= 1u << (p1 % N);
  if (L.valid && p2 < (uint32_t)(N * N) && (int)(p2 / N) == L.r) out |= 1u << (p2 % N);
  return out;
}
// row words -> the form kept with the game (the same in every lane of the board)
template <int N>
__device__ __forceinline__ uint32_t sk_forb_word(const Lane<N>& L, uint32_t forb) {
  using G = Geo<N>;
  uint32_t fw = kNoPoint | (kNoPoint << 16);
  if (ballot(forb != 0u) == 0ull) return fw;   // nearly always
  const uint64_t seg = ((uint64_t)L.seghi << 32) | L.seglo;
  const int cnt = board_popcount<N>(L, forb);
  uint32_t rest = forb;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint64_t mine = ballot(rest != 0u) & seg;
    const int src = mine ? (__ffsll((long long)mine) - 1) : L.lane;
    const int col = __shfl((int)(__ffs(rest) - 1), src);
    const uint32_t p = mine ? (uint32_t)((src - (L.j * G::STRIDE + 1)) * N + col) : kNoPoint;
    fw = k == 0 ? ((fw & 0xFFFF0000u) | p) : ((fw & 0xFFFFu) | (p << 16));
    if (L.lane == src) rest &= rest - 1u;
  }
  if (cnt > 2) fw = kLookAgain | (kNoPoint << 16);
  return fw;
}
// The forbidden plays of the position the kernel has just loaded: from the game's record, or (more than two of them
// were found when the position arose) by walking the table again.
template <int N>
__device__ __forceinline__ uint32_t sk_forb_loaded(const Lane<N>& L, const uint2* tab, const SkGame& g, const Row<N>& R, const Meta& m, const SkWin& pre,
                                                   uint32_t* scratch) {
  uint32_t forb = sk_forb_rows<N>(L, g.fw);
  const bool again = L.boardok && (g.fw & 0xFFFFu) == kLookAgain;
  if (ballot(again) != 0ull) {
    const uint32_t f2 = sk_forbidden<N>(L, tab, g, R, m, again, pre, scratch);
    if (again) forb = f2;
  }
  return forb;
}

// all lanes of the wavefront clear the tables of the boards flagged by their row-0 lane (auto-reset); `game` = the
// index of this lane's board among the handle's tables
template <int N>
__device__ __forceinline__ void sk_clear_tables(const Lane<N>& L, bool flagged, uint2* zt, int game) {
  for (uint64_t q = ballot(flagged && L.valid && L.r == 0); q; q &= q - 1ull) {
    const size_t bb = (size_t)__shfl(game, __ffsll((long long)q) - 1);
    uint4* t4 = (uint4*)(zt + bb * Zt<N>::SLOTS);
    for (uint32_t i = L.lane; i < Zt<N>::SLOTS / 2u; i += 64u) t4[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  wave_mem_fence();
}

// Steps a2-a8 of one ply with the repetition rule for every board of the wavefront: the requested move passes the
// legality gate only if it is not one of the position's forbidden plays (`forb`, updated to those of the new position),
// the new position goes into the table, an auto-reset clears it.  tab_r / tab_w / game: see sk_insert, sk_clear_tables.
// GATE as in gate_move.  Out: as apply_move.
// board_final(moved, reset) is called once the rows and scalars of the new position (an auto-reset included) are final: the
// caller brings its history up to date there, emits the observation and may store the state.  EARLY: before the table work, so that those stores are
// under way while the walks go on (measured: 25.1 -> 23.8 us per ply in the rollout kernel; in the one-launch-per-ply
// kernel it is 1 us slower than calling it afterwards, hence the choice).
template <int N, bool GATE, bool EARLY, class Hook>
__device__ __forceinline__ void sk_step_core(const Lane<N>& L, Row<N>& R, Meta& m, SkGame& g, uint32_t& forb, const Rules& rules, bool skip, bool want_pass,
                                             bool want_point, uint32_t bit_in, int pr_in, int pc_in, const uint2* tab_r, uint2* tab_w, uint2* zt, int game,
                                             uint32_t* scratch, Tally& tally, Ply& ply, bool pre_a_loaded, const SkWin& pre_a, Hook&& board_final) {
  const int c = m.wtm, own = c ? g.nw : g.nb, opp = c ? g.nb : g.nw;
  Move mv = gate_move<N, GATE>(L, R, m, skip, want_pass, want_point, bit_in, pr_in, pc_in);
  // a play the simple rules allow but the repetition rule forbids is an illegal action
  const bool repeats = mv.playing && board_any((mv.bit & forb) != 0u, L.seglo, L.seghi);
  if (repeats) mv.forbid();
  // The chains this ply needs start at slots known before the rules run when the move takes nothing (most do): the
  // loads fly while the rules run.  pre[0]: one more stone of the mover's colour (where the new position goes);
  // pre[1]: one more stone of the other colour (the next mover's forbidden plays); pre[2]: as many stones of the
  // other colour as now (the new position's second entry).
  SkWin pre[3];
  if (pre_a_loaded) pre[0] = pre_a;
  else pre[0] = sk_window<N>(L, tab_r, sk_home<N>(c, own + 1), mv.playing);
  pre[1] = sk_window<N>(L, tab_r, sk_home<N>(c ^ 1, opp + 1), mv.playing || mv.is_pass);
  pre[2] = sk_window<N>(L, tab_r, sk_home<N>(c ^ 1, opp), mv.playing);
  Rules r0 = rules;
  r0.auto_reset = 0;   // the reset happens below, after the table work
  // go_step_superko_kernel clears the tally here, with the windows on their way, and not where it unpacks the state, before the walks (19x19, us a ply there / here:
  // x 16384 26.57 / 26.42, x 20000 32.41 / 32.25, x 24000 38.8 / 38.6; small batches the same).
  if constexpr (GATE && !EARLY) tally.clear();
  ply = apply_move<N, false, Floods<N>::PACKED && !GATE>(L, R, m, r0, mv, tally);
  const bool do_reset = !skip && !mv.frozen && m.term && rules.auto_reset != 0;
  if (do_reset) reset_board<N>(L, R, m, rules.seed);   // a board that is reset takes no part in the table work below
  ply.reset = do_reset;
  if constexpr (EARLY) {
    // The windows have to be in registers before the caller's stores are issued: loads and stores share one counter,
    // and a wait for these loads placed after the stores would wait for the stores as well.
    asm volatile("" ::"v"(pre[0].e.x), "v"(pre[0].e.y), "v"(pre[1].e.x), "v"(pre[1].e.y), "v"(pre[2].e.x), "v"(pre[2].e.y));
    board_final(ply.moved, do_reset);
  }
  const SkPly s = sk_look<N>(L, tab_r, g, c, mv, ply.captured, pre[0], scratch);
  sk_insert<N>(L, tab_r, tab_w, g, s, mv.playing && !do_reset, c, pre[2]);
  // the forbidden plays change with the position and with the player to move; otherwise they stay
  const bool moved = (mv.playing || mv.is_pass) && !do_reset;
  const uint32_t fresh = sk_forbidden<N>(L, tab_r, g, R, m, moved, pre[1], scratch);
  if (moved) forb = fresh;
  if (do_reset) { g = sk_fresh(); forb = 0u; }
  sk_clear_tables<N>(L, do_reset, zt, game);
  if constexpr (!EARLY) board_final(ply.moved, do_reset);
}

// The same for the reading in which the rule is looked at only for the move that is played (mode 1): no sets of
// forbidden plays are kept, and a position has ONE table entry, on the chain of its two stone counts (so that it is
// found whoever recreates it).  One table window read and one 8-byte store per game-ply instead of three and two.
// pre: the chain's first window for a play that takes nothing, loaded by the caller as early as it can (home = ~0u:
// not loaded).  Two orders:
//   POST = false (the rollout kernel, whose state lives in registers): the position the requested play would give is
//     known before the rules run -- it takes exactly the opposing chains in atari next to it -- so its keys are looked
//     up first; a hit turns the play into an illegal action.
//   POST = true (one launch per ply, where every wavefront would wait for the window before it can do anything else):
//     the rules run first, on the assumption that the play repeats nothing, board_final(moved, reset) is called (the observation is
//     under way), and the look-up follows; after a hit (rare) restore(R, m, which) brings back the state as loaded for
//     the boards flagged and the history as loaded for all, the ply is applied again as an illegal action and board_final is
//     called once more: the same wavefront overwrites what it stored the first time.
template <int N, bool GATE, bool POST, class Hook, class Restore>
__device__ __forceinline__ void sk_step_core_play(const Lane<N>& L, Row<N>& R, Meta& m, SkGame& g, const Rules& rules, bool skip, bool want_pass,
                                                  bool want_point, uint32_t bit_in, int pr_in, int pc_in, const uint2* tab_r, uint2* tab_w, uint2* zt, int game,
                                                  uint32_t* scratch, Tally& tally, Ply& ply, const SkWin& pre, Hook&& board_final, Restore&& restore) {
  const int c = m.wtm, own1 = (c ? g.nw : g.nb) + 1;
  const uint64_t seg = ((uint64_t)L.seghi << 32) | L.seglo;
  Move mv = gate_move<N, GATE>(L, R, m, skip, want_pass, want_point, bit_in, pr_in, pc_in);
  Rules r0 = rules;
  r0.auto_reset = 0;   // the reset happens below, together with the table's
  bool do_reset = false;
  if constexpr (POST) {
    ply = apply_move<N>(L, R, m, r0, mv, tally);
    do_reset = !skip && !mv.frozen && m.term && rules.auto_reset != 0;
    if (do_reset) reset_board<N>(L, R, m, rules.seed);
    // The window has to be in registers before the caller's stores are issued: loads and stores share one counter.
    asm volatile("" ::"v"(pre.e.x), "v"(pre.e.y));
    board_final(ply.moved, do_reset);   // on the assumption that nothing repeats; done again below if something does
  }
  // the stones the play takes: known from the rules (POST), else the opposing chains in atari next to it
  uint32_t taken = 0u;
  if constexpr (POST) taken = ply.captured;
  else {
    const uint32_t aopp = c ? R.ab : R.aw;
    const uint32_t seed = dilate(mv.bit) & aopp;
    if (ballot(seed != 0u) != 0ull) taken = flood_plain(seed, aopp);
  }
  int ncap = 0;
  uint2 dk = make_uint2(0u, 0u);
  if (ballot(taken != 0u) != 0ull) {   // about one ply in ten
    ncap = board_popcount<N>(L, taken);
    dk = board_xor<N>(L, row_keys<N>(L.r, c ? taken : 0u, c ? 0u : taken), scratch);
  }
  const int opp1 = (c ? g.nb : g.nw) - ncap;
  const int nb1 = c ? opp1 : own1, nw1 = c ? own1 : opp1;
  const uint32_t kp = zkey((uint32_t)(mv.playing ? mv.pr * N + mv.pc : 0), (uint32_t)c);
  const uint2 key = make_uint2(g.key.x ^ (c ? 0u : kp) ^ dk.x, g.key.y ^ (c ? kp : 0u) ^ dk.y);
  bool hit = false, ok;
  uint32_t free_slot;
  sk_walk<N>(L, tab_r, sk_home_counts<N>(nb1, nw1), mv.playing, pre, ~0u,
             [&](uint2 e, bool look) { if ((ballot(look && e.x == key.x && e.y == key.y) & seg) != 0ull) hit = true; }, ok, free_slot);
  const bool repeats = mv.playing && hit;
  if (repeats) mv.forbid();
  if constexpr (!POST) {
    ply = apply_move<N>(L, R, m, r0, mv, tally);
    do_reset = !skip && !mv.frozen && m.term && rules.auto_reset != 0;
    if (do_reset) reset_board<N>(L, R, m, rules.seed);
    board_final(ply.moved, do_reset);
  } else if (ballot(repeats) != 0ull) {
    restore(R, m, repeats);   // the boards that repeat get the state as loaded back
    Move again = mv;          // the other boards of the wavefront keep what the first pass gave them: for them, a skipped ply
    if (!repeats) { again.skip = true; again.frozen = false; again.is_pass = false; again.playing = false; again.illegal = false; again.pr = -100; again.pc = 0; again.bit = 0u; }
    const Ply second = apply_move<N>(L, R, m, r0, again, tally);
    if (repeats) {
      ply = second;
      do_reset = rules.auto_reset != 0;   // the illegal action has ended the game
      if (do_reset) reset_board<N>(L, R, m, rules.seed);
    }
    board_final(ply.moved, do_reset);
  }
  ply.reset = do_reset;
  if (mv.playing && !do_reset) {
    if (L.valid && L.r == 0 && ok && sk_real(key)) tab_store(&tab_w[free_slot], key);
    g.key = key; g.nb = nb1; g.nw = nw1;
  }
  if (do_reset) g = sk_fresh();
  wave_mem_fence();
  sk_clear_tables<N>(L, do_reset, zt, game);
}
// the window the next play of the game looks at first (mode 1), if that play takes nothing
template <int N>
__device__ __forceinline__ SkWin sk_window_play(const Lane<N>& L, const uint2* tab, const SkGame& g, const Meta& m, bool want) {
  return sk_window<N>(L, tab, sk_home_counts<N>(g.nb + (m.wtm ? 0 : 1), g.nw + (m.wtm ? 1 : 0)), want);
}

// One ply with the repetition rule.  Same steps as go_step_kernel.
// MODE: 1 = the rule is looked at when the move is played, 2 = honoured by the legal mask
template <int N, bool TIGHT, int ST, int MODE>
__global__ void __launch_bounds__(64 * kWavesPerBlock, 6) go_step_superko_kernel(uint32_t* state, uint4* meta, const int32_t* actions, const int32_t* start_t,
                                                                                uint4* zcur, int B, int wb, uint32_t eighth, uint2* zt, StepArgs a) {
  using G = Geo<N>;
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs_all[kWavesPerBlock][G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask_all[kWavesPerBlock][64];
  __shared__ TallyCells tally_all[kWavesPerBlock];
  __shared__ uint2 lut[256];
  const int wib = wave_in_block();
  const int wave = piece_of_block(eighth) * kWavesPerBlock + wib;
  const Lane<N> L(wave, threadIdx.x & 63, B, wb);
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  load_history<N>(state, L, H);
  const uint4 meta_raw = load_meta<N>(meta, L);
  const int act_raw = actions[L.boardok ? L.b : L.some], act = L.boardok ? act_raw : -1;
  const uint4 g_raw = zcur[L.boardok ? L.b : L.some];
  const int32_t start_raw = (a.next_actions && L.boardok && start_t) ? start_t[L.b] : INT32_MIN;
  in_scalar_registers(a.rew, a.term, a.mask, a.obs, a.mask_pitch, a.obs_pitch, a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset);
  fill_spread_table(lut);   // (nothing loaded above is looked at before this barrier)
  if (wave * wb >= B) return;
  const bool wait_start = (int64_t)a.sample_t < (int64_t)held_back(start_raw);
  SkGame g = L.boardok ? sk_unpack(g_raw) : sk_fresh();
  Meta m = unpack_meta(meta_raw);
  place_ko<N>(L, R, m);
  uint2* tab = zt + (size_t)(L.boardok ? L.b : 0) * Zt<N>::SLOTS;

  const bool skip = !L.boardok || act == -1;
  const bool in_range = act >= 0 && act < G::P;
  const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
  SkWin none;
  none.home = ~0u; none.e = make_uint2(1u, 0u);
  uint32_t forb = 0u;
  Ply ply;
  // a6, a10 (mode 1 still holds the row and the table window: a fourth round at once, at 9x9 a third, would spill)
  auto board_final = [&](bool moved, bool reset) {
    push_history<N>(H, m.head, R.bk, R.wt, moved);
    if (reset) clear_history<N>(H);
    if (a.obs) emit_obs<N, TIGHT, ST, MODE == 1 ? (N == 9 ? 2 : 3) : 4>(L, points_of<N>(H, m.head).h, m.wtm, wave, B, a.obs, a.obs_pitch, lds_obs_all[wib], lut, wb);
  };
  if constexpr (MODE == 1) {
    const SkWin pre = sk_window_play<N>(L, tab, g, m, !skip);
    Tally tally(tally_all, wib, L);   // (ahead of the window: 19x19 x 20000 30.5 us and not 30.1, x 24000 35.3 and not 34.8, 9x9 x 30001 13.54 and not 13.42)
    sk_step_core_play<N, true, true>(L, R, m, g, a.rules, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc, tab, tab, zt, L.b, lds_mask_all[wib], tally, ply, pre,
                                     board_final, [&](Row<N>& Rr, Meta& mr, bool which) {   // the state is stored below: memory still holds it as loaded
                                       Row<N> T;
                                       load_row<N>(state, L, T);
                                       load_history<N>(state, L, H);
                                       const Meta as_loaded = unpack_meta(load_meta<N>(meta, L));
                                       mr.head = as_loaded.head;
                                       place_ko<N>(L, T, as_loaded);
                                       if (which) { Rr = T; mr = as_loaded; }
                                     });
  } else {
    forb = sk_forb_loaded<N>(L, tab, g, R, m, none, lds_mask_all[wib]);
    Tally tally(tally_all, wib, L, true);
    sk_step_core<N, true, false>(L, R, m, g, forb, a.rules, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc, tab, tab, zt, L.b, lds_mask_all[wib], tally, ply, false, none, board_final);
    g.fw = sk_forb_word<N>(L, forb);
  }
  constexpr int STATE_ST = MODE == 1 && N == 9 ? kStorePlain : state_store_kind(ST);   // (mode 1 at 9x9 has no registers left for the other kind)
  store_ply<N, STATE_ST>(state, L, R, H, m.head, ply.moved, ply.reset);   // a11
  if (!skip && L.valid && L.r == 0) {
    store_small<STATE_ST>(&meta[L.b], pack_meta(m));
    *(float2*)(a.rew + 2 * (size_t)L.b) = make_float2(ply.rew0, ply.rew1);
    store_small<ST>(&a.term[L.b], (uint8_t)(ply.flag ? 1 : 0));
  }

  place_ko<N>(L, R, m);
  const uint32_t legal = legal_row<N>(L, R, m.wtm) & ~(MODE == 2 ? forb : 0u);
  if (a.mask) emit_mask<N, TIGHT, ST>(L, legal, wave, B, a.mask, a.mask_pitch, lds_mask_all[wib], lut, wb);
  if (!skip && L.valid && L.r == 0) zcur[L.b] = sk_pack(g);
  if (a.next_actions) {
    const Draw<N> dr = draw_action<N>(L, legal, a.sample_seed, a.sample_t, wait_start);
    if (dr.known(L)) a.next_actions[L.b] = dr.action(L);
  }
}

// ------------------------------------------------------------------------------------------------
// The same by teams (go_step_team_kernel), for the rule proper (mode 2): one wavefront applies the rules and stores the state, one has the
// table -- its windows are loaded while the rules run -- and then the mask and the draw, which need what it finds, and one has the observation.
// What bounds the other kernel is that all of this stands in a row in one wavefront.  Figures, and which plies go this way: boards_per_superko_team.
// ------------------------------------------------------------------------------------------------
template <int N, bool OBS, int ST>
__global__ void __launch_bounds__(64 * (OBS ? 3 : 2)) go_step_superko_team_kernel(uint32_t* state, uint4* meta, const int32_t* actions, const int32_t* start_t, uint4* zcur,
                                                                                  int B, int wb, uint32_t eighth, uint2* zt, StepArgs a) {   // wb: boards per team
  using G = Geo<N>;
  constexpr uint32_t THREADS = 64u * (OBS ? 3u : 2u);
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs[OBS ? G::W * G::OBS_DW : 4];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask[64];
  __shared__ TallyCells tally_cells;
  __shared__ uint2 lut[256];
  __shared__ uint4 hand[64];
  const int group = piece_of_block(eighth);
  if (group * wb >= B) return;   // the whole block
  const int role = wave_in_block();
  const Lane<N> L(group, threadIdx.x & 63, B, wb);
  const int game = L.boardok ? L.b : L.some;
  auto fill_table = [&]() {
#pragma unroll
    for (uint32_t x = threadIdx.x; x < 256u; x += THREADS) lut[x] = make_uint2(spread4(x & 15u), spread4(x >> 4));
  };
  SkWin none;
  none.home = ~0u; none.e = make_uint2(1u, 0u);

  if (role == 0) {   // the rules
    rules_first(eighth);
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    const uint4 meta_raw = load_meta<N>(meta, L);
    const int act_raw = actions[game], act = L.boardok ? act_raw : -1;
    const uint4 g_raw = zcur[game];
    load_history<N>(state, L, H);
    in_scalar_registers(a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset, a.rew, a.term);
    fill_table();
    Meta m = unpack_meta(meta_raw);
    place_ko<N>(L, R, m);
    const bool skip = !L.boardok || act == -1;
    const bool in_range = act >= 0 && act < G::P;
    const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
    Move mv = gate_move<N, true>(L, R, m, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc);
    const SkGame g = L.boardok ? sk_unpack(g_raw) : sk_fresh();
    const uint32_t forb = sk_forb_loaded<N>(L, zt + (size_t)game * Zt<N>::SLOTS, g, R, m, none, (uint32_t*)hand);
    if (mv.playing && board_any((mv.bit & forb) != 0u, L.seglo, L.seghi)) mv.forbid();
    Tally tally(&tally_cells, 0, L);
    const Ply ply = apply_move<N>(L, R, m, a.rules, mv, tally, [&]() { clear_history<N>(H); });
    hand[L.lane] = HandOver<N>::of(R, m, ply).v;
    __syncthreads();
    push_history<N>(H, m.head, R.bk, R.wt, ply.moved);
    store_ply<N, kStorePlain>(state, L, R, H, m.head, ply.moved, ply.reset);
    if (!skip && L.valid && L.r == 0) {
      meta[L.b] = pack_meta(m);
      *(float2*)(a.rew + 2 * (size_t)L.b) = make_float2(ply.rew0, ply.rew1);
      a.term[L.b] = (uint8_t)(ply.flag ? 1 : 0);
    }
  } else if (role == 1) {   // the table, the mask, the draw
    Row<N> before;
    const uint4 meta_raw = load_meta<N>(meta, L), g_raw = zcur[game];
    const int act_raw = actions[game], act = L.boardok ? act_raw : -1;
    const int32_t start_raw = (a.next_actions && L.boardok && start_t) ? start_t[L.b] : INT32_MIN;
    load_row<N>(state, L, before);
    in_scalar_registers(a.mask, a.mask_pitch, a.sample_seed, a.sample_t, a.next_actions);
    fill_table();
    Meta m = unpack_meta(meta_raw);
    SkGame g = L.boardok ? sk_unpack(g_raw) : sk_fresh();
    uint2* const tab = zt + (size_t)game * Zt<N>::SLOTS;
    // the windows of sk_step_core, for a play that is legal and takes nothing
    const int c = m.wtm, own = c ? g.nw : g.nb, opp = c ? g.nb : g.nw;
    const bool may_play = act >= 0 && act < G::P && !m.term;
    const SkWin pre_a = sk_window<N>(L, tab, sk_home<N>(c, own + 1), may_play);
    const SkWin pre_forb = sk_window<N>(L, tab, sk_home<N>(c ^ 1, opp + 1), may_play || (act == G::P && !m.term));
    const SkWin pre_b = sk_window<N>(L, tab, sk_home<N>(c ^ 1, opp), may_play);
    const uint32_t hash = in_place(env_hash(a.sample_seed, 0u, (uint32_t)L.b, a.sample_t));
    // here before the other wavefront stores the next position, which it does once it has handed it over
    asm volatile("" ::"v"(before.bk), "v"(before.wt));
    __syncthreads();
    const HandOver<N> in{hand[L.lane]};
    const Row<N> R = in.row();
    const bool moved = in.moved() && !in.reset(), played = moved && act != G::P;
    Move mv;
    mv.playing = played;
    mv.pr = played ? act / N : -100; mv.pc = played ? act - (act / N) * N : 0;
    const uint32_t captured = !played ? 0u : c ? before.bk & ~R.bk : before.wt & ~R.wt;
    const SkPly s = sk_look<N>(L, tab, g, c, mv, captured, pre_a, lds_mask);
    sk_insert<N>(L, tab, tab, g, s, played, c, pre_b);
    // the forbidden plays change with the position and with the player to move; otherwise they stay, where they fit the record, and are found anew where not
    m.wtm = in.wtm();
    const bool find = moved || (L.boardok && !in.reset() && (g.fw & 0xFFFFu) == kLookAgain);
    const uint32_t found = sk_forbidden<N, true>(L, tab, g, R, m, find, pre_forb, lds_mask);
    const uint32_t forb = in.reset() ? 0u : find ? found : sk_forb_rows<N>(L, g.fw);
    if (in.reset()) g = sk_fresh();
    sk_clear_tables<N>(L, in.reset(), zt, L.b);
    g.fw = sk_forb_word<N>(L, forb);
    const uint32_t legal = legal_row<N>(L, R, in.wtm()) & ~forb;
    if (a.mask) emit_mask<N, true, ST>(L, legal, group, B, a.mask, a.mask_pitch, lds_mask, lut, wb);
    if (act != -1 && L.valid && L.r == 0) zcur[L.b] = sk_pack(g);
    if (a.next_actions) {
      const Draw<N> d = draw_action<N>(L, legal, hash, (int64_t)a.sample_t < (int64_t)start_raw);
      if (d.known(L)) a.next_actions[L.b] = d.action(L);
    }
  } else if constexpr (OBS) {
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    load_history<N>(state, L, H);
    const Meta m = unpack_meta(load_meta<N>(meta, L));
    in_scalar_registers(a.obs, a.obs_pitch);
    fill_table();
    team_obs<N, ST>(L, R, points_of<N>(H, m.head), m, hand, group, B, a.obs, a.obs_pitch, lds_obs, lut, wb, [] { __syncthreads(); });
  }
}

// Fills the tables from what the state still carries: the 8 history positions and the current one (set-up, import),
// and finds the current position's forbidden plays.  The tables must have been cleared by an earlier launch.
template <int N>
__global__ void __launch_bounds__(64) go_superko_rebuild_kernel(uint32_t* state, const uint4* meta, int B, uint2* zt, uint4* zcur, int mode) {
  __shared__ uint32_t scratch[64];
  const Lane<N> L(blockIdx.x, threadIdx.x, B);
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  load_history<N>(state, L, H);
  const Meta m = unpack_meta(load_meta<N>(meta, L));
  place_ko<N>(L, R, m);
  const Points<N> Q = points_of<N>(H, m.head);
  uint2* tab = zt + (size_t)(L.boardok ? L.b : 0) * Zt<N>::SLOTS;
  SkWin none;
  none.home = ~0u; none.e = make_uint2(1u, 0u);
  SkGame g = sk_fresh();
  for (int i = 8; i >= 0; --i) {   // history position i-1 (oldest first), then i = 0: the current stones
    uint32_t black = R.bk, white = R.wt;
    if (i > 0) {
      black = 0u; white = 0u;
#pragma unroll
      for (int col = 0; col < N; ++col) {
        const uint32_t hw = (Q.h[col >> 1] >> ((col & 1) * 16)) & 0xFFFFu;
        black |= ((hw >> (2 * (i - 1))) & 1u) << col;
        white |= ((hw >> (2 * (i - 1) + 1)) & 1u) << col;
      }
    }
    uint2 k = make_uint2(0u, 0u);
    if (L.valid) k = row_keys<N>(L.r, black, white);
    g.key = board_xor<N>(L, k, scratch);
    g.nb = board_popcount<N>(L, black); g.nw = board_popcount<N>(L, white);
    const uint2 entry = g.key;
    bool hit = false, ok_a, ok_b = false;
    uint32_t free_a, free_b = 0u;
    // mode 1: one entry on the chain of the two counts; mode 2: one on the chain of each colour's count
    sk_walk<N>(L, tab, mode == 1 ? sk_home_counts<N>(g.nb, g.nw) : sk_home<N>(0, g.nb), L.boardok, none, ~0u,
               [&](uint2 e, bool look) { hit = hit || (look && e.x == entry.x && e.y == entry.y); }, ok_a, free_a);
    const bool found = board_any(hit, L.seglo, L.seghi) || !sk_real(entry);   // the empty board is never stored
    if (mode != 1) sk_walk<N>(L, tab, sk_home<N>(1, g.nw), L.boardok && !found, none, ok_a ? free_a : ~0u, [](uint2, bool) {}, ok_b, free_b);
    if (L.valid && L.r == 0) {
      if (!found && ok_a) tab_store(&tab[free_a], entry);
      if (!found && ok_b) tab_store(&tab[free_b], entry);
    }
    __threadfence();   // the next round's look-ups must see these inserts
  }
  if (mode != 1) g.fw = sk_forb_word<N>(L, sk_forbidden<N>(L, tab, g, R, m, L.boardok, none, scratch));
  if (L.valid && L.r == 0) zcur[L.b] = sk_pack(g);
}

__global__ void go_zero_kernel(uint4* p, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ------------------------------------------------------------------------------------------------
// the slot kernel (tree search): entry i reads the state of slot src[i], applies actions[i] (all -1 when
// actions is null: a plain copy) and writes the result to slot dst[i]; outputs go to row i.
// ------------------------------------------------------------------------------------------------
struct SlotArgs {       // what is not needed before the first loads
  float* rew;           // [n][2] or null
  uint8_t* term;        // [n] or null; 255 marks an entry whose slot index was out of range
  uint8_t* mask;        // [n][mask_pitch] or null
  uint8_t* obs;         // [n][obs_pitch] or null
  int64_t mask_pitch, obs_pitch;
  Rules rules;
  uint2* zt;            // positional superko (SK kernels): per-slot tables, per-slot current keys, mode 1 / 2
  uint4* zcur;
  int sk_mode;
};

// SK: the positional-superko rule is on; a game that moves to another slot takes its key table along.
template <int N, bool TIGHT, int SK, int ST = kStorePlain>
__global__ void __launch_bounds__(64 * kWavesPerBlock, SK ? 4 : 6) go_step_slots_kernel(const int32_t* src_slots, const int32_t* dst_slots, const int32_t* actions,
                                                                                      uint32_t* state, uint4* meta, int pool, int n, uint32_t eighth, SlotArgs a) {
  // pool: number of state slots (the handle's batch), n: entries of this call
  using G = Geo<N>;
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs_all[kWavesPerBlock][G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask_all[kWavesPerBlock][64];
  __shared__ TallyCells tally_all[kWavesPerBlock];
  __shared__ uint2 lut[256];
  const int wib = wave_in_block();
  const int wave = piece_of_block(eighth) * kWavesPerBlock + wib;
  Lane<N> L(wave, threadIdx.x & 63, n);
  const int src = L.boardok ? src_slots[L.b] : 0, dst = L.boardok ? dst_slots[L.b] : 0;
  const bool in_pool = src >= 0 && src < pool && dst >= 0 && dst < pool;
  const bool bad = L.boardok && !in_pool;
  if (bad) { L.boardok = false; L.valid = false; L.full = 0u; }   // the entry becomes inert: no state access, no outputs
  L.slot = src; L.some = 0;   // (a lane without an entry loads from slot 0, whatever another entry may be doing with it, and uses nothing of that)
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  load_history<N>(state, L, H);
  const uint4 meta_raw = load_meta<N>(meta, L);
  const int act = (L.boardok && actions) ? actions[L.b] : -1;
  in_scalar_registers(a.rew, a.term, a.mask, a.obs, a.mask_pitch, a.obs_pitch, a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset);
  fill_spread_table(lut);
  if (wave * G::W >= n) return;
  Meta m = unpack_meta(meta_raw);
  place_ko<N>(L, R, m);
  L.slot = dst;   // from here on the board is environment dst (seat draw on reset, state store)

  const bool skip = !L.boardok || act == -1;
  const bool in_range = act >= 0 && act < G::P;
  const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
  Ply ply;
  uint32_t forb = 0u;
  Tally tally(tally_all, wib, L);
  auto board_final = [&](bool moved, bool reset) {   // a6, a10
    push_history<N>(H, m.head, R.bk, R.wt, moved);
    if (reset) clear_history<N>(H);
    if (a.obs) emit_obs<N, TIGHT, ST>(L, points_of<N>(H, m.head).h, m.wtm, wave, n, a.obs, a.obs_pitch, lds_obs_all[wib], lut);
  };
  if constexpr (!SK) {
    const Move mv = gate_move<N, true>(L, R, m, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc);
    ply = apply_move<N>(L, R, m, a.rules, mv, tally);
  } else {
    const int sslot = L.boardok ? src : 0, dslot = L.boardok ? dst : 0;
    SkGame g = L.boardok ? sk_unpack(a.zcur[sslot]) : sk_fresh();
    const uint2* tab_r = a.zt + (size_t)sslot * Zt<N>::SLOTS;   // nothing writes to a source slot's table during the call
    uint2* tab_w = a.zt + (size_t)dslot * Zt<N>::SLOTS;
    for (uint64_t q = ballot(L.valid && L.r == 0 && src != dst); q; q &= q - 1ull) {   // all lanes copy one table after the other
      const int ln = __ffsll((long long)q) - 1;
      const uint4* from = (const uint4*)(a.zt + (size_t)__shfl(sslot, ln) * Zt<N>::SLOTS);
      uint4* to = (uint4*)(a.zt + (size_t)__shfl(dslot, ln) * Zt<N>::SLOTS);
      for (uint32_t i = L.lane; i < Zt<N>::SLOTS / 2u; i += 64u) to[i] = from[i];
    }
    __threadfence();   // the copied tables are in place before entries are added to them or they are cleared
    SkWin none;
    none.home = ~0u; none.e = make_uint2(1u, 0u);
    if constexpr (SK == 1) {
      const SkWin pre = sk_window_play<N>(L, tab_r, g, m, !skip);
      sk_step_core_play<N, true, true>(L, R, m, g, a.rules, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc, tab_r, tab_w, a.zt, dslot, lds_mask_all[wib], tally, ply, pre,
                                       board_final, [&](Row<N>& Rr, Meta& mr, bool which) {   // the source slot still holds the state as loaded
                                         Lane<N> Ls = L;
                                         Ls.slot = src;
                                         Row<N> T;
                                         load_row<N>(state, Ls, T);
                                         load_history<N>(state, Ls, H);
                                         const Meta as_loaded = unpack_meta(meta[sslot]);
                                         mr.head = as_loaded.head;
                                         place_ko<N>(L, T, as_loaded);
                                       if (which) { Rr = T; mr = as_loaded; }
                                       });
    } else {
      forb = sk_forb_loaded<N>(L, tab_r, g, R, m, none, lds_mask_all[wib]);
      sk_step_core<N, true, true>(L, R, m, g, forb, a.rules, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc, tab_r, tab_w, a.zt, dslot, lds_mask_all[wib], tally, ply, false, none, board_final);
      g.fw = sk_forb_word<N>(L, forb);
    }
    if (L.valid && L.r == 0) a.zcur[dslot] = sk_pack(g);
    if constexpr (SK != 2) forb = 0u;   // the mask shows the simple-ko set unless the rule proper is on
  }
  if ((threadIdx.x & 63) == L.j * G::STRIDE + 1 && L.j < G::W && L.b < n) {   // row-0 lane of the entry, inert or not
    if (bad) { if (a.term) store_small<ST>(&a.term[L.b], (uint8_t)255); }
    else {
      // a copied entry (action -1) reports what a skipped step reports for a fresh handle: no reward, and its terminated state
      if (a.rew) *(float2*)(a.rew + 2 * (size_t)L.b) = skip ? make_float2(0.f, 0.f) : make_float2(ply.rew0, ply.rew1);
      if (a.term) store_small<ST>(&a.term[L.b], (uint8_t)(skip ? m.term : (ply.flag ? 1 : 0)));
    }
  }
  const uint32_t legal = legal_row<N>(L, R, m.wtm) & ~forb;
  if constexpr (!SK) board_final(ply.moved, ply.reset);
  if (a.mask) emit_mask<N, TIGHT, ST>(L, legal, wave, n, a.mask, a.mask_pitch, lds_mask_all[wib], lut);
  store_all<N>(state, L, R, H);
  if (L.valid && L.r == 0) meta[dst] = pack_meta(m);
}

// ------------------------------------------------------------------------------------------------
// The same by teams (go_step_team_kernel): one wavefront applies the rules and stores the new state, one writes the mask, one the
// observation.  Figures, and which calls go this way: boards_per_slot_team.
// ------------------------------------------------------------------------------------------------
template <int N, bool OBS, int ST>
__global__ void __launch_bounds__(64 * (OBS ? 3 : 2)) go_step_slots_team_kernel(const int32_t* src_slots, const int32_t* dst_slots, const int32_t* actions, uint32_t* state,
                                                                                uint4* meta, int pool, int n, int wb, uint32_t eighth, SlotArgs a) {   // wb: boards per team
  using G = Geo<N>;
  constexpr uint32_t THREADS = 64u * (OBS ? 3u : 2u);
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs[OBS ? G::W * G::OBS_DW : 4];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask[64];
  __shared__ TallyCells tally_cells;
  __shared__ uint2 lut[256];
  __shared__ uint4 hand[64];
  const int group = piece_of_block(eighth);
  if (group * wb >= n) return;   // the whole block
  const int role = wave_in_block();
  Lane<N> L(group, threadIdx.x & 63, n, wb);
  const int entry = L.boardok ? L.b : L.some;   // (a lane without an entry loads the team's first one: no branch around a load)
  const int src = src_slots[entry], dst = dst_slots[entry];
  auto fill_table = [&]() {
#pragma unroll
    for (uint32_t x = threadIdx.x; x < 256u; x += THREADS) lut[x] = make_uint2(spread4(x & 15u), spread4(x >> 4));
  };
  const bool in_pool = src >= 0 && src < pool && dst >= 0 && dst < pool;
  const bool bad = L.boardok && !in_pool;
  if (bad) { L.boardok = false; L.valid = false; L.full = 0u; }   // the entry becomes inert: no state access, no outputs
  L.slot = src; L.some = 0;

  if (role == 0) {
    rules_first(eighth);
    const int act_raw = actions[entry];
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    const uint4 meta_raw = load_meta<N>(meta, L);
    load_history<N>(state, L, H);
    in_scalar_registers(a.rew, a.term, a.rules.seed, a.rules.komi_x2, a.rules.max_steps, a.rules.auto_reset);
    fill_table();
    const int act = L.boardok ? act_raw : -1;
    Meta m = unpack_meta(meta_raw);
    place_ko<N>(L, R, m);
    L.slot = dst;   // from here on the board is environment dst (seat draw on reset, state store)
    const bool skip = !L.boardok || act == -1;
    const bool in_range = act >= 0 && act < G::P;
    const int pr = in_range ? act / N : 0, pc = in_range ? act - (act / N) * N : 0;
    const Move mv = gate_move<N, true>(L, R, m, skip, act == G::P, in_range, bit_of<N>(L, in_range, pr, pc), pr, pc);
    Tally tally(&tally_cells, 0, L);
    const Ply ply = apply_move<N>(L, R, m, a.rules, mv, tally, [&]() { clear_history<N>(H); });
    hand[L.lane] = HandOver<N>::of(R, m, ply).v;
    __syncthreads();
    push_history<N>(H, m.head, R.bk, R.wt, ply.moved);
    store_all<N>(state, L, R, H);
    if (L.valid && L.r == 0) meta[dst] = pack_meta(m);
    if (L.lane == L.j * G::STRIDE + 1 && L.j < wb && L.b < n) {   // row-0 lane of the entry, inert or not
      if (bad) { if (a.term) a.term[L.b] = (uint8_t)255; }
      else {
        // a copied entry (action -1) reports what a skipped step reports for a fresh handle: no reward, and its terminated state
        if (a.rew) *(float2*)(a.rew + 2 * (size_t)L.b) = skip ? make_float2(0.f, 0.f) : make_float2(ply.rew0, ply.rew1);
        if (a.term) a.term[L.b] = (uint8_t)(skip ? m.term : (ply.flag ? 1 : 0));
      }
    }
  } else if (role == 1) {
    in_scalar_registers(a.mask, a.mask_pitch);
    fill_table();
    __syncthreads();
    if (a.mask) emit_mask<N, true, ST>(L, HandOver<N>{hand[L.lane]}.legal(L), group, n, a.mask, a.mask_pitch, lds_mask, lut, wb);
  } else if constexpr (OBS) {
    Row<N> R;
    History<N> H;
    load_row<N>(state, L, R);
    load_history<N>(state, L, H);
    const Meta m = unpack_meta(load_meta<N>(meta, L));
    in_scalar_registers(a.obs, a.obs_pitch);
    fill_table();
    team_obs<N, ST>(L, R, points_of<N>(H, m.head), m, hand, group, n, a.obs, a.obs_pitch, lds_obs, lut, wb, [] { __syncthreads(); });
  }
}

// ------------------------------------------------------------------------------------------------
// the rollout kernel: one launch = `steps` plies of uniform random legal play of every environment.  The
// state stays in registers between plies; each ply's outputs go to slice (i mod slices) of the caller's
// trajectory buffers.
// ------------------------------------------------------------------------------------------------
struct RolloutArgs {
  uint32_t* state;
  uint4* meta;
  int B;
  int wb;               // boards per wavefront of this launch
  Rules rules;
  int steps, slices;
  uint32_t seed, t0;
  const int32_t* start_t;
  int32_t* actions;     // [slices][B] or null
  float* rew;           // [slices][B][2] or null
  uint8_t* term;        // [slices][B] or null
  uint8_t* mask;        // [slices][B][mask_pitch] or null
  uint8_t* obs;         // [slices][B][obs_pitch] or null
  int64_t mask_pitch, obs_pitch;
  uint2* zt;            // positional superko (SK kernels): per-game tables, per-game current keys, mode 1 / 2
  uint4* zcur;
  int sk_mode;
  PaceArgs pace;
};

// The rate that the slots of a paced rollout are laid out for (us for plies of 19x19 x 16384 games, recorded, with 6.3 / 6.35 / 6.4 / 6.45 /
// 6.5 / 6.6 TB/s: 16 plies 281.2 / 280.4 / 277.8 / 276.1 / 275.3 / 276.0, 64 plies 1092 / 1084 / 1076 / 1069 / 1061 / 1145; two steps below
// the best, since above it the gain is soon lost)
constexpr double kPaceBytesPerSecond = 6.4e12;
// Ticks until the first slot with the repetition rule, whose first ply looks at the tables beforehand (with 0 / 2 us: 8 plies of 30001 games, which
// run in generations, 327 / 324; 16 of 16384 351 / 346)
constexpr uint32_t kPaceFirstSuperko = 200u;

// The registers hold a game's state from ply to ply, and 80 of them (six wavefronts per SIMD) are just enough for it and a ply's own values.
// What a ply derives from the lane's place alone is therefore computed anew every ply (in_place): kept from one to the next it pushed
// 8 to 16 registers out to memory, and every one read back between the outputs waited for all output stores under way (20 plies in
// place by this kernel, which teams have taken over since unless a handle asks for it: 19x19 x 16384 games 307 -> 281 us, x 65536 1141 -> 1043;
// with pitches that are neither dense nor padded 367 -> 326).
// SK: 0 = simple ko only, 1 / 2 = positional superko at play time / in the legal mask.  PACED: recordings that go to DRAM, see Pace;
// their stores carry the non-temporal hint as well (16 plies of 19x19 x 16384 games at 6.2 TB/s: 286 us with it, 344 without).
// AS_STORED (19x19, no observation, and then never PACED): the history stays a ring.  Turned into points and back, which only the emission
// needs, a launch of one ply of 16384 games took 14.8 instead of 13.5 us, of 50000 29.5 instead of 25.8 (14.0 and 28.0 when memory held points too);
// as a choice at run time it costs rollouts with observation up to 1.5 %.
template <int N, bool TIGHT, int SK, bool PACED, bool AS_STORED = false>
__global__ void __launch_bounds__(64 * kWavesPerBlock, SK ? 4 : 6) go_rollout_kernel(RolloutArgs a) {
  using G = Geo<N>;
  static_assert(!AS_STORED || (G::RINGED && !PACED), "a ring is kept where memory holds one, and nothing is emitted from it");
  constexpr int ST = PACED ? kStoreStreamWhole : kStoreThroughWhole;
  // In place the ends of a wavefront's streams are better left to the L2: ordinary stores to the same lines meet there from ply to ply and
  // do not go to memory each time.  With dense pitches a stream hardly ever starts on a line; with line-padded ones every stream does,
  // and its first 1 KB counts as an end all the same (20 plies of 16384 games by this kernel: 2.14 -> 1.94 GB leave the L2, 313 -> 282 us; x
  // 65536 1154 -> 1043 us).  9x9 x 16384, where a wavefront writes half as much, gains nothing.
  constexpr bool FIRST_AS_EDGE = N == 19 && TIGHT && !PACED;
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs_all[kWavesPerBlock][G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask_all[kWavesPerBlock][64];
  __shared__ TallyCells tally_all[kWavesPerBlock];
  __shared__ uint2 lut[256];
  const int wib = wave_in_block();
  Pace pace(PACED, PACED ? Pace::now() : 0, a.pace, (blockIdx.x >> 3) * kWavesPerBlock + wib, (gridDim.x >> 3) * kWavesPerBlock, SK ? kPaceFirstSuperko : 0u);
  fill_spread_table(lut);
  const int wave = piece_of_block() * kWavesPerBlock + wib;
  if (wave * a.wb >= a.B) return;
  const Lane<N> L0(wave, threadIdx.x & 63, a.B, a.wb);
  Row<N> R;
  Points<N> Q;
  Meta m = unpack_meta(load_meta<N>(a.meta, L0));
  {
    History<N> H;
    load_row<N>(a.state, L0, R);
    load_history<N>(a.state, L0, H);
    Q = kept_history<N, AS_STORED>(H, m.head);
    place_ko<N>(L0, R, m);
  }
  const int64_t start = (L0.boardok && a.start_t) ? (int64_t)a.start_t[L0.b] : INT64_MIN;
  uint32_t legal = legal_row<N>(L0, R, m.wtm);
  SkGame g = sk_fresh();
  uint2* tab = nullptr;
  uint32_t forb = 0u;
  if constexpr (SK) {
    if (L0.boardok) g = sk_unpack(a.zcur[L0.b]);
    tab = a.zt + (size_t)(L0.boardok ? L0.b : 0) * Zt<N>::SLOTS;
    SkWin none;
    none.home = ~0u; none.e = make_uint2(1u, 0u);
    if constexpr (SK != 1) forb = sk_forb_loaded<N>(L0, tab, g, R, m, none, lds_mask_all[wib]);
    if constexpr (SK == 2) legal &= ~forb;
  }
  // mode 1: the window the next ply looks at, loaded one ply ahead
  SkWin ahead;
  ahead.home = ~0u; ahead.e = make_uint2(1u, 0u);
  if constexpr (SK == 1) ahead = sk_window_play<N>(L0, tab, g, m, L0.boardok);
  int slice = 0;
  for (int i = 0; i < a.steps; ++i) {   // the same trip count for every wavefront
    Lane<N> L = L0;
    if (!TIGHT) L.lane = in_place(L.lane);   // (board-by-board emission holds more)
    Tally tally(tally_all, wib, L);          // (anew every ply: which cell is next is nothing to hold through the loop)
    const uint32_t t = a.t0 + (uint32_t)i;
    const bool wait = (int64_t)t < start;
    const Draw<N> d = draw_action<N>(L, legal, a.seed, t, wait);
    const bool skip = !L.boardok || wait;
    const size_t sb = (size_t)slice * a.B;
    if (a.actions && d.known(L)) a.actions[sb + L.b] = d.action(L);
    Ply ply;
    const int dr = d.row(L), dc = SK ? d.column() : 0;
    if constexpr (!SK) {
      ply = apply_move<N, N == 19>(L, R, m, a.rules, gate_move<N, false>(L, R, m, skip, d.pass, d.point, d.bit, 0, 0), tally,
                          [&]() { clear_points<N>(Q); });
      push_kept<N, AS_STORED>(Q, m.head, R.bk, R.wt, ply.moved);
      legal = legal_row<N>(L, R, m.wtm);
    } else {
      SkWin none;
      none.home = ~0u; none.e = make_uint2(1u, 0u);
      uint8_t* const obs_t = a.obs ? a.obs + (size_t)slice * a.B * a.obs_pitch : nullptr;
      auto board_final = [&](bool moved, bool reset) {
        push_kept<N, AS_STORED>(Q, m.head, R.bk, R.wt, moved);
        if (reset) clear_points<N>(Q);
        if constexpr (PACED) pace.wait();
        if (obs_t) emit_obs<N, TIGHT, ST, 4, FIRST_AS_EDGE>(L, Q.h, m.wtm, wave, a.B, obs_t, a.obs_pitch, lds_obs_all[wib], lut, a.wb);
      };
      if constexpr (SK == 1) {
        sk_step_core_play<N, false, false>(L, R, m, g, a.rules, skip, d.pass, d.point, d.bit, dr, dc, tab, tab, a.zt, L.b, lds_mask_all[wib], tally, ply,
                                           ahead, board_final, [](Row<N>&, Meta&, bool) {});
        ahead = sk_window_play<N>(L, tab, g, m, L.boardok);
      } else {
        sk_step_core<N, false, true>(L, R, m, g, forb, a.rules, skip, d.pass, d.point, d.bit, dr, dc, tab, tab, a.zt, L.b, lds_mask_all[wib], tally, ply, false, none, board_final);
      }
      legal = legal_row<N>(L, R, m.wtm) & ~(SK == 2 ? forb : 0u);
    }
    if (L.valid && L.r == 0) {
      const size_t e = sb + L.b;
      // a waiting environment reports the values a skipped step call leaves behind at the start: zeros
      if (a.rew) *(float2*)(a.rew + 2 * e) = skip ? make_float2(0.f, 0.f) : make_float2(ply.rew0, ply.rew1);
      if (a.term) a.term[e] = (uint8_t)((!skip && ply.flag) ? 1 : 0);
    }
    if constexpr (PACED && !SK) pace.wait();
    emit_outputs<N, TIGHT, ST, FIRST_AS_EDGE>(L, Q, legal, m.wtm, wave, a.B, a.mask ? a.mask + sb * a.mask_pitch : nullptr, a.mask_pitch,
                    (!SK && a.obs) ? a.obs + sb * a.obs_pitch : nullptr, a.obs_pitch, lds_mask_all[wib], lds_obs_all[wib], lut, a.wb);
    wave_lds_fence();
    slice = slice + 1 == a.slices ? 0 : slice + 1;
  }
  const Lane<N> L1(wave, in_place(L0.lane), a.B, a.wb);   // (anew: where a game's state lies is nothing to hold through the loop)
  store_all<N>(a.state, L1, R, history_of_kept<N, AS_STORED>(Q, m.head));
  if (L1.valid && L1.r == 0) a.meta[L1.b] = pack_meta(m);
  if constexpr (SK) {
    if constexpr (SK != 1) g.fw = sk_forb_word<N>(L0, forb);
    if (L0.valid && L0.r == 0) a.zcur[L0.b] = sk_pack(g);
  }
}

// ------------------------------------------------------------------------------------------------
// The same plies by teams (go_step_team_kernel): one wavefront draws and applies the rules, ply after ply; it leaves each position in
// LDS, in one of two places in turn, and goes on with the next ply while the others write the outputs of this one.
// A ply's chain is then a draw and the rules alone: of the 5200 cycles that a wavefront by itself takes for a ply of one 9x9 board, with its
// observation, 3200 are left.  The hand-over waits for the next draw, by when the writes to LDS are done, and the other wavefronts hash for the draws: 64 plies
// of 9x9 x 5001 games without observation 82.6 -> 81.8 us.  Figures, and which rollouts go this way: boards_per_rollout_team.
// ------------------------------------------------------------------------------------------------
// (team_barrier orders nothing in memory.  So rows and history are written by the wavefront that has read them itself.  The
// scalars are read by two; the one with the history writes them, when the other, which has needed all of them for its first ply, has handed
// over the new ones in LDS.)
constexpr int rollout_team_waves(bool with_obs) { return with_obs ? 3 : 2; }
// SK: 0 = simple ko only, 1 / 2 = positional superko at play time / in the legal mask, whose table is the business of the wavefront with the rules
template <int N, bool OBS, int SK>
__global__ void __launch_bounds__(64 * rollout_team_waves(OBS)) go_rollout_team_kernel(RolloutArgs a) {   // a.wb: boards per team
  using G = Geo<N>;
  constexpr int WAVES = rollout_team_waves(OBS), ST = kStoreThroughWhole;
  constexpr bool FIRST_AS_EDGE = N == 19;   // as in go_rollout_kernel
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs[OBS ? G::W * G::OBS_DW : 4];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask[64];
  __shared__ TallyCells tally_cells;
  __shared__ uint2 lut[256];
  __shared__ uint4 hand[2][64];
  __shared__ uint4 scalars[2][G::W];   // per board: rewards, terminated
  __shared__ int32_t drawn[2][8];
  __shared__ uint32_t hashes[4][64];      // of the draws, computed by the wavefront with the mask three plies ahead
  __shared__ uint4 scalars_after[G::W];   // the game's record as the launch leaves it
  __shared__ uint32_t legal_of[SK == 2 ? 2 : 1][64];   // SK = 2: what the position alone does not say
  __shared__ uint32_t sk_scratch[SK ? 64 : 1];
  const int group = piece_of_block();
  if (group * a.wb >= a.B) return;   // the whole block
  const int role = wave_in_block();
  const Lane<N> L(group, threadIdx.x & 63, a.B, a.wb);
  for (uint32_t x = threadIdx.x; x < 256u; x += 64u * WAVES) lut[x] = make_uint2(spread4(x & 15u), spread4(x >> 4));

  if (role == 0) {   // the draws and the rules
    rules_first(gridDim.x >> 3);
    Row<N> R;
    load_row<N>(a.state, L, R);
    Meta m = unpack_meta(load_meta<N>(a.meta, L));
    place_ko<N>(L, R, m);
    const int64_t start = (L.boardok && a.start_t) ? (int64_t)a.start_t[L.b] : INT64_MIN;
    uint32_t legal = legal_row<N>(L, R, m.wtm);
    for (uint32_t k = 0; k < 2u; ++k) hashes[k][L.lane] = env_hash(a.seed, 0u, (uint32_t)L.b, a.t0 + k);   // (plies 0 and 1 are drawn before the other's come)
    Tally tally(&tally_cells, 0, L);
    SkGame g = sk_fresh();
    uint2* tab = nullptr;
    uint32_t forb = 0u;
    SkWin none, ahead;
    none.home = ~0u; none.e = make_uint2(1u, 0u);
    if constexpr (SK) {
      if (L.boardok) g = sk_unpack(a.zcur[L.b]);
      tab = a.zt + (size_t)(L.boardok ? L.b : 0) * Zt<N>::SLOTS;
      if constexpr (SK == 1) ahead = sk_window_play<N>(L, tab, g, m, L.boardok);
      else { forb = sk_forb_loaded<N>(L, tab, g, R, m, none, sk_scratch); legal &= ~forb; }
    }
    for (int i = 0; i < a.steps; ++i) {
      const uint32_t t = a.t0 + (uint32_t)i;
      const bool wait = (int64_t)t < start;
      const Draw<N> d = draw_action<N>(L, legal, hashes[i & 3][L.lane], wait);
      if (i) team_barrier();   // hands over the ply before: what it left in LDS is there by now, and nobody waits for that
      const bool skip = !L.boardok || wait;
      if (d.known(L)) drawn[i & 1][L.j] = d.action(L);
      Ply ply;
      if constexpr (!SK) ply = apply_move<N>(L, R, m, a.rules, gate_move<N, false>(L, R, m, skip, d.pass, d.point, d.bit, 0, 0), tally);
      else {
        const int dr = d.row(L), dc = d.column();
        auto nothing = [](bool, bool) {};   // (history and observation are the others')
        if constexpr (SK == 1) {
          sk_step_core_play<N, false, false>(L, R, m, g, a.rules, skip, d.pass, d.point, d.bit, dr, dc, tab, tab, a.zt, L.b, sk_scratch, tally, ply, ahead, nothing, [](Row<N>&, Meta&, bool) {});
          ahead = sk_window_play<N>(L, tab, g, m, L.boardok);
        } else
          sk_step_core<N, false, false>(L, R, m, g, forb, a.rules, skip, d.pass, d.point, d.bit, dr, dc, tab, tab, a.zt, L.b, sk_scratch, tally, ply, false, none, nothing);
      }
      hand[i & 1][L.lane] = HandOver<N>::of(R, m, ply).v;
      // a waiting environment reports the values a skipped step call leaves behind at the start: zeros
      if (L.valid && L.r == 0) scalars[i & 1][L.j] = make_uint4(skip ? 0u : __float_as_uint(ply.rew0), skip ? 0u : __float_as_uint(ply.rew1), !skip && ply.flag ? 1u : 0u, 0u);
      legal = legal_row<N>(L, R, m.wtm) & ~(SK == 2 ? forb : 0u);
      if constexpr (SK == 2) legal_of[i & 1][L.lane] = legal;
    }
    team_barrier();
    if constexpr (SK) {
      if constexpr (SK == 2) g.fw = sk_forb_word<N>(L, forb);
      if (L.valid && L.r == 0) a.zcur[L.b] = sk_pack(g);
    }
    if (L.valid) {
      store_row<N>(State<N>(a.state, L), R);
      m.head = 0;
      if (L.r == 0) scalars_after[L.j] = pack_meta(m);
    }
    team_barrier();
  } else {   // 1: the mask and the scalars; 2: the observation; the last of them keeps the history
    const bool history = role == WAVES - 1, observe = OBS && role == 2;
    Points<N> Q;
    if (history) {
      History<N> H;
      load_history<N>(a.state, L, H);
      Q = points_of<N>(H, unpack_meta(load_meta<N>(a.meta, L)).head);
    }
    int slice = 0;
    if (role == 1) hashes[2][L.lane] = env_hash(a.seed, 0u, (uint32_t)L.b, a.t0 + 2u);
    for (int i = 0; i < a.steps; ++i) {
      team_barrier();
      const HandOver<N> in{hand[i & 1][L.lane]};
      const size_t sb = (size_t)slice * a.B;
      if (role == 1) {
        hashes[(i + 3) & 3][L.lane] = env_hash(a.seed, 0u, (uint32_t)L.b, a.t0 + (uint32_t)i + 3u);   // (in the place of ply i - 1's; the other may be drawing ply i + 2)
        if (L.valid && L.r == 0) {
          const size_t e = sb + L.b;
          const uint4 v = scalars[i & 1][L.j];
          if (a.actions) a.actions[e] = drawn[i & 1][L.j];
          if (a.rew) *(float2*)(a.rew + 2 * e) = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
          if (a.term) a.term[e] = (uint8_t)v.z;
        }
        if (a.mask) emit_mask<N, true, ST, FIRST_AS_EDGE>(L, SK == 2 ? legal_of[SK == 2 ? i & 1 : 0][L.lane] : in.legal(L), group, a.B, a.mask + sb * a.mask_pitch, a.mask_pitch, lds_mask, lut, a.wb);
      }
      if (history) {
        const Row<N> R = in.row();
        if (in.reset()) clear_points<N>(Q);
        push_points<N>(Q, R.bk, R.wt, in.moved());
      }
      if constexpr (OBS) {
        if (observe) emit_obs<N, true, ST, 4, FIRST_AS_EDGE>(L, Q.h, in.wtm(), group, a.B, a.obs + sb * a.obs_pitch, a.obs_pitch, lds_obs, lut, a.wb);
      }
      slice = slice + 1 == a.slices ? 0 : slice + 1;
    }
    team_barrier();
    if (history) {
      store_history<N>(a.state, L, history_of<N>(Q));
      if (L.valid && L.r == 0) a.meta[L.b] = scalars_after[L.j];   // (this wavefront has taken the ring's beginning from there)
    }
  }
}

// ------------------------------------------------------------------------------------------------
// auxiliary kernels
// ------------------------------------------------------------------------------------------------
// SK: the legal mask leaves out the plays that would recreate an earlier position (positional superko, mode 2)
template <int N, bool TIGHT, bool SK>
__global__ void __launch_bounds__(64 * kWavesPerBlock) go_emit_kernel(uint32_t* state, const uint4* meta, int B, uint8_t* mask,
                                                                      int64_t mask_pitch, uint8_t* obs, int64_t obs_pitch, const uint2* zt,
                                                                      const uint4* zcur) {
  using G = Geo<N>;
  __shared__ __attribute__((aligned(16))) uint32_t lds_obs_all[kWavesPerBlock][G::W * G::OBS_DW];
  __shared__ __attribute__((aligned(16))) uint32_t lds_mask_all[kWavesPerBlock][64];
  __shared__ uint2 lut[256];
  fill_spread_table(lut);
  const int wib = wave_in_block();
  const int wave = piece_of_block() * kWavesPerBlock + wib;
  if (wave * G::W >= B) return;
  const Lane<N> L(wave, threadIdx.x & 63, B);
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  if (obs) load_history<N>(state, L, H);
  Meta m = unpack_meta(load_meta<N>(meta, L));
  place_ko<N>(L, R, m);
  uint32_t legal = legal_row<N>(L, R, m.wtm);
  if constexpr (SK) {
    if (mask) {
      const SkGame g = L.boardok ? sk_unpack(zcur[L.b]) : sk_fresh();
      SkWin none;
      none.home = ~0u; none.e = make_uint2(1u, 0u);
      legal &= ~sk_forb_loaded<N>(L, zt + (size_t)(L.boardok ? L.b : 0) * Zt<N>::SLOTS, g, R, m, none, lds_mask_all[wib]);
    }
  }
  if (mask) emit_mask<N, TIGHT>(L, legal, wave, B, mask, mask_pitch, lds_mask_all[wib], lut);
  if (obs) emit_obs<N, TIGHT>(L, points_of<N>(H, m.head).h, m.wtm, wave, B, obs, obs_pitch, lds_obs_all[wib], lut);
}

// k-th legal action of the current position, same row-per-lane mapping as the step kernel
template <int N, bool SK>
__global__ void __launch_bounds__(64 * kWavesPerBlock) go_random_actions_kernel(uint32_t* state, const uint4* meta, const int32_t* start_t,
                                                                                int32_t* actions, int B, uint32_t seed, uint32_t t, uint32_t eighth,
                                                                                const uint2* zt, const uint4* zcur) {
  using G = Geo<N>;
  __shared__ uint32_t sk_scratch[SK ? kWavesPerBlock : 1][64];
  const int wave = piece_of_block(eighth) * kWavesPerBlock + wave_in_block();
  if (wave * G::W >= B) return;
  const Lane<N> L(wave, threadIdx.x & 63, B);
  Row<N> R;
  load_row<N>(state, L, R);
  Meta m = unpack_meta(load_meta<N>(meta, L));
  place_ko<N>(L, R, m);
  uint32_t legal = legal_row<N>(L, R, m.wtm);
  if constexpr (SK) {
    const SkGame g = L.boardok ? sk_unpack(zcur[L.b]) : sk_fresh();
    SkWin none;
    none.home = ~0u; none.e = make_uint2(1u, 0u);
    legal &= ~sk_forb_loaded<N>(L, zt + (size_t)(L.boardok ? L.b : 0) * Zt<N>::SLOTS, g, R, m, none, sk_scratch[wave_in_block()]);
  }
  const bool wait = L.boardok && start_t && (int64_t)t < (int64_t)start_t[L.b];
  const Draw<N> d = draw_action<N>(L, legal, seed, t, wait);
  if (d.known(L)) actions[L.b] = d.action(L);
}

// new episode for every environment: empty board, Black to move, seat from the hash
template <int N>
__global__ void go_reset_kernel(uint32_t* state, uint4* meta, float* rew, uint8_t* term, int B, uint32_t seed, int first) {
  using G = Geo<N>;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  constexpr int share = (G::GAME + N - 1) / N;   // of a game's dwords for each of its N threads
  if (i < (size_t)B * N) {
    const int r = (int)(i % N);
#pragma unroll
    for (int k = 0; k < share; ++k)
      if (share * r + k < G::GAME) state[i / N * G::GAME + share * r + k] = 0u;
  }
  if (i < (size_t)B) {
    Meta m;
    if (first) { m.episode = 0u; m.illegal = 0u; }
    else { Meta old = unpack_meta(meta[i]); m.episode = old.episode + 1u; m.illegal = old.illegal; }
    m.ko = -1; m.steps = 0; m.passes = 0; m.wtm = 0; m.term = 0; m.head = 0;
    m.bp = (int)(env_hash(seed, 1u, (uint32_t)i, m.episode) & 1u);
    meta[i] = pack_meta(m);
    rew[2 * i] = 0.f; rew[2 * i + 1] = 0.f; term[i] = 0;
  }
}

template <int N>
__global__ void go_current_player_kernel(const uint4* meta, int B, uint8_t* dst) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  Meta m = unpack_meta(meta[b]);
  dst[b] = (uint8_t)(m.wtm ? 1 - m.bp : m.bp);
}

struct CanonArgs {
  int8_t* board; int8_t* history; int32_t* ko; int8_t* to_play; int32_t* steps; int8_t* passes;
  uint8_t* terminated; uint8_t* black_player; uint32_t* episode; uint32_t* illegal;
};

template <int N>
__global__ void __launch_bounds__(64) go_export_kernel(uint32_t* state, const uint4* meta, int B, CanonArgs c) {
  using G = Geo<N>;
  const Lane<N> L(blockIdx.x, threadIdx.x, B);
  Row<N> R;
  History<N> H;
  load_row<N>(state, L, R);
  load_history<N>(state, L, H);
  if (!L.valid) return;
  const Meta m = unpack_meta(meta[L.b]);
  const Points<N> Q = points_of<N>(H, m.head);
  const size_t cell0 = (size_t)L.b * G::P + (size_t)L.r * N;
#pragma unroll
  for (int col = 0; col < N; ++col) {
    if (c.board) c.board[cell0 + col] = (int8_t)((int)((R.bk >> col) & 1u) - (int)((R.wt >> col) & 1u));
    if (c.history) {
      uint32_t hw = (Q.h[col >> 1] >> ((col & 1) * 16)) & 0xFFFFu;
      for (int i = 0; i < 8; ++i)
        c.history[((size_t)L.b * 8 + i) * G::P + (size_t)L.r * N + col] = (int8_t)((int)((hw >> (2 * i)) & 1u) - (int)((hw >> (2 * i + 1)) & 1u));
    }
  }
  if (L.r == 0) {
    if (c.ko) c.ko[L.b] = m.ko;
    if (c.to_play) c.to_play[L.b] = (int8_t)(m.wtm ? -1 : 1);
    if (c.steps) c.steps[L.b] = m.steps;
    if (c.passes) c.passes[L.b] = (int8_t)m.passes;
    if (c.terminated) c.terminated[L.b] = (uint8_t)m.term;
    if (c.black_player) c.black_player[L.b] = (uint8_t)m.bp;
    if (c.episode) c.episode[L.b] = m.episode;
    if (c.illegal) c.illegal[L.b] = m.illegal;
  }
}

// canonical arrays -> private state; the atari sets are rebuilt chain by chain
template <int N>
__global__ void __launch_bounds__(64) go_import_kernel(uint32_t* state, uint4* meta, float* rew, uint8_t* term, int B, CanonArgs c) {
  using G = Geo<N>;
  const Lane<N> L(blockIdx.x, threadIdx.x, B);
  Row<N> R;
  Points<N> Q;
#pragma unroll
  for (int k = 0; k < G::HD; ++k) Q.h[k] = 0u;
  R.bk = R.wt = R.ab = R.aw = R.ko = 0u;
  Meta m;
  m.head = 0;
  m.ko = -1; m.steps = 0; m.passes = 0; m.wtm = 0; m.term = 0; m.bp = 0; m.episode = 0u; m.illegal = 0u;
  if (L.boardok) {
    Meta old = unpack_meta(meta[L.b]);
    m.illegal = old.illegal;
    m.ko = c.ko[L.b]; m.wtm = c.to_play[L.b] < 0 ? 1 : 0; m.steps = c.steps[L.b] & 0xFFFF; m.passes = c.passes[L.b] & 3;
    m.term = c.terminated[L.b] ? 1 : 0; m.bp = c.black_player[L.b] & 1; m.episode = c.episode[L.b];
  }
  if (L.valid) {
    const size_t cell0 = (size_t)L.b * G::P + (size_t)L.r * N;
    for (int col = 0; col < N; ++col) {
      int v = c.board[cell0 + col];
      if (v > 0) R.bk |= 1u << col; else if (v < 0) R.wt |= 1u << col;
      uint32_t hw = 0u;
      for (int i = 0; i < 8; ++i) {
        int hv = c.history[((size_t)L.b * 8 + i) * G::P + (size_t)L.r * N + col];
        if (hv > 0) hw |= 1u << (2 * i); else if (hv < 0) hw |= 1u << (2 * i + 1);
      }
#pragma unroll
      for (int k = 0; k < G::HD; ++k) if (k == (col >> 1)) Q.h[k] |= hw << ((col & 1) * 16);
    }
  }
  const uint32_t E = L.full & ~(R.bk | R.wt);
  uint32_t visited = 0u;
  for (;;) {
    // next unvisited stone of every board, its whole chain, its liberty class
    const uint32_t rest = (R.bk | R.wt) & ~visited;
    const uint64_t has = ballot(rest != 0u);
    if (has == 0ull) break;
    const uint64_t mine = has & (((uint64_t)L.seghi << 32) | L.seglo);
    const bool first = mine != 0ull && (__ffsll((long long)mine) - 1) == L.lane;
    const uint32_t seed = first ? (rest & (0u - rest)) : 0u;
    const bool black = board_any((seed & R.bk) != 0u, L.seglo, L.seghi);
    const uint32_t F = flood_plain(seed, black ? R.bk : R.wt);
    bool one, two;
    board_count(dilate(F) & E, L.seglo, L.seghi, one, two);
    visited |= F;
    if (one) { if (black) R.ab |= F; else R.aw |= F; }
  }
  store_all<N>(state, L, R, history_of<N>(Q));
  if (L.valid && L.r == 0) {
    meta[L.b] = pack_meta(m);
    rew[2 * (size_t)L.b] = 0.f; rew[2 * (size_t)L.b + 1] = 0.f; term[L.b] = (uint8_t)m.term;
  }
}

__global__ void lane_shift_probe_kernel(const uint32_t* in, uint32_t* out) {
  uint32_t x = in[threadIdx.x];
  out[threadIdx.x] = from_lane_below(x);
  out[64 + threadIdx.x] = from_lane_above(x);
}

__global__ void __launch_bounds__(256) remainder_probe_kernel(const uint32_t* n, const uint32_t* d, uint32_t* out, uint32_t count) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < count) out[i] = remainder_of(n[i], d[i]);
}

// Measurement helpers: a plain fill with 16-byte stores (the practical write ceiling of the machine on the same
// buffers the step kernel writes) and an empty kernel (the gap between dependent launches on one stream).
template <int ST>
__global__ void __launch_bounds__(256) fill_probe_kernel(uint4* __restrict__ dst, size_t n16, uint32_t value) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte store per thread
  if (i < n16) store16<ST>(&dst[i], make_uint2(value, value), make_uint2(value, value));
}
__global__ void empty_probe_kernel() {}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

template <int N>
size_t state_bytes_for(int B, size_t* off_meta, size_t* off_rew, size_t* off_term) {
  using G = Geo<N>;
  size_t o = 0;
  o += align_up((size_t)B * N * G::row_bytes, 256);
  if (off_meta) *off_meta = o;
  o += align_up((size_t)B * sizeof(uint4), 256);
  if (off_rew) *off_rew = o;
  o += align_up((size_t)B * 2 * sizeof(float), 256);
  if (off_term) *off_term = o;
  o += align_up((size_t)B, 256);
  return o;
}

}  // namespace

struct pgxgo_ctx {
  int B, N;
  int wb;        // boards per wavefront used by the step and rollout launches (1 .. W)
  bool automatic;   // wb is this library's choice; then teams take the batches that suit them (boards_per_step_team, boards_per_rollout_team)
  uint32_t seed;
  int komi_x2, max_steps, auto_reset;
  int64_t obs_pitch, mask_pitch;
  hipStream_t stream;
  uint32_t* state;
  uint4* meta;
  float* rew_int;
  uint8_t* term_int;
  uint8_t* mask_out;
  uint8_t* obs_out;
  float* rew_out;
  uint8_t* term_out;
  const uint8_t* mask_written;   // the buffers the last step (or bind) call wrote mask and observation to
  const uint8_t* obs_written;
  uint2* zt;     // positional superko: per-game key tables, or null when the rule is off
  uint4* zcur;   // key and stone counts of every game's current position
  int sk_mode;   // 0 off, 1 enforced when the move is played, 2 honoured by the legal mask
};

namespace {

template <int N>
int launch_reset(pgxgo_ctx* h, int first) {
  const size_t n = (size_t)h->B * N;
  const int threads = 256;
  const unsigned blocks = (unsigned)((n + threads - 1) / threads);
  hipLaunchKernelGGL(go_reset_kernel<N>, dim3(blocks), dim3(threads), 0, h->stream, h->state, h->meta, h->rew_out, h->term_out, h->B, h->seed,
                     first);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
unsigned waves_for(int B) { return (unsigned)((B + Geo<N>::W - 1) / Geo<N>::W); }
template <int N>
unsigned blocks_for(int B) { return ((waves_for<N>(B) + kWavesPerBlock - 1) / kWavesPerBlock + 7u) & ~7u; }   // a multiple of 8: piece_of_block
unsigned blocks_for_wb(int B, int wb) { return (((unsigned)((B + wb - 1) / wb) + kWavesPerBlock - 1) / kWavesPerBlock + 7u) & ~7u; }

// Kind of the output stores of a one-launch-per-ply kernel by the bytes the launch writes: up to 48 MB everything written
// through the L2 (us for 4 launches, against whole lines only: 19x19 x 6001 games, 39 MB, 39.6 / 39.9, as entries of a search
// x 5500 37.9 / 39.3; 9x9 x 24000, 35 MB, 38.0 / 40.4; above the line 19x19 x 9000, 58 MB, 50.5 / 50.0); from there to the size
// of the memory-side cache write-through for whole lines only (16384 games: 20.7 against 22.1 us per ply with ordinary stores);
// beyond what that cache holds of them beside the state the non-temporal hint on top (us per ply, whole lines written through / with the
// hint: 19x19 x 28000 games, 182 MB, 34.1 / 38.3; x 36000, 234 MB, 47.8 / 46.1; x 40000 55 / 48; x 48000 77 / 61; x 65536 114 / 80; with
// superko x 40000 86 / 62; 9x9 x 160000, 233 MB, 49.7 / 49.9; x 200000 67 / 62).  Rollouts use kStoreThroughWhole at every size
// unless they are paced (by single wavefronts, 16384 games: 14.4 against 16.5 us per ply, 65536 games: 53.8 against 60.2 us; in place the
// non-temporal hint is slower at every size).
// in_place: the launch overwrites the buffers the previous one wrote, whose lines are then still in the memory-side
// cache.  In the middle range a launch into other buffers (a caller that records a trajectory) has to reach DRAM and
// is faster with the hint as well (16384 games: 23.9 us per ply against 25.4 with ordinary stores and 25.9 with
// write-through alone).
constexpr size_t kWriteThroughUpTo = (size_t)48 << 20, kNonTemporalFrom = (size_t)220 << 20;
int store_kind_for(size_t out_bytes, bool in_place) {
  if (out_bytes <= kWriteThroughUpTo) return kStoreThrough;
  if (out_bytes <= kNonTemporalFrom) return in_place ? kStoreThroughWhole : kStoreStreamWhole;
  return kStoreStreamWhole;
}
size_t output_bytes_per_ply(const pgxgo_ctx* h, bool with_mask, bool with_obs) {
  return (size_t)h->B * ((with_mask ? (size_t)h->mask_pitch : 0) + (with_obs ? (size_t)h->obs_pitch : 0));
}

// What a launch takes is decided by the SIMD (of 1024) with the most wavefronts, and by how many boards share a wavefront's floods
// and output rounds.  So: the smallest number of wavefronts per SIMD that W boards per wavefront allow, and then the fewest boards
// per wavefront that need no more (measured per ply, one launch per ply: 9x9 x 2048 games 5.3 us with 2 boards, 7.0 with 1, 5.9
// with 6; x 4096 5.7 with 4, 8.9 with 1; x 8192 6.5 with 4, 6.8 with 6, 7.9 with 2; x 7001 6.1 with 4, 6.4 with 6; 19x19 x 3072
// 7.4 with 3, 10.0 with 1; 32 plies of 9x9 x 8192 in one launch 106 us with 4, 116 with 6).  At 19x19 that would be two boards
// instead of W = 3 from 3073 to 4096 games, and there three are kept: two save 2 to 4 % of a ply per launch (8 of x 3300 65.7 / 67.9 us, x 4096
// 67.7 / 69.5) but cost 7 to 10 % of a rollout in place (20 plies of x 3300 102.0 / 94.4, x 4096 103.2 / 95.7; recorded 2 to 4 %), and a
// handle has one count for both.
template <int N>
int auto_boards_per_wavefront(int B) {
  if (N == 19 && B > 1024 * Geo<N>::W) return Geo<N>::W;   // (beyond 4096 games the rule gives W by itself)
  const int per_simd = (int)(((int64_t)B + 1024 * Geo<N>::W - 1) / (1024 * Geo<N>::W));
  return (int)(((int64_t)B + 1024 * (int64_t)per_simd - 1) / (1024 * (int64_t)per_simd));
}

// both output pitches are the dense or the line-padded ones: the kernels treat a wavefront's boards as one run of bytes
// (with the line-padded pitch the pad bytes belong to that run and are written as zeros)
template <int N>
bool tight_pitches(const pgxgo_ctx* h) {
  using G = Geo<N>;
  return (h->mask_pitch == G::A || h->mask_pitch == G::A_PAD) && (h->obs_pitch == G::OBS || h->obs_pitch == G::OBS_PAD);
}

// Boards per team of four wavefronts (go_step_team_kernel) for batches that are faster that way, else 0.  A team is worth while as long as
// the machine has wavefront slots to spare: up to four teams per compute unit at 9x9 (us per ply, one wavefront for all / teams: 256
// games 4.60 / 3.72, 1024 4.94 / 4.16, 2048 4.95 / 4.55, 4096 5.21 / 4.99; beyond it is one or the other by turns, four boards to a team 4500 5.56 /
// 5.40, 5000 5.49 / 5.53, 6000 5.59 / 5.70, 6500 5.95 / 5.80, 7500 6.03 / 6.26, 8192 6.03 / 6.35) and eight at 19x19, where the
// observation is four times as long (256 games 5.96 / 4.63, 1000 6.47 / 5.66, 2048 7.18 / 6.08, 4096 8.79 / 7.50, 5500 9.57 / 8.57, 8192
// 12.0 / 12.4; without observation 1000 5.34 / 4.79, 4096 6.27 / 6.05, 5500 6.48 / 6.54).  Boards: as few as keep the teams at one to two per
// compute unit (9x9 x 256 with 1 / 2 / 4 boards 3.72 / 3.77 / 3.97, x 1024 4.63 / 4.16 / 4.30, x 2048 5.8 / 4.78 / 4.55; 19x19 x 400 with 1 / 3
// 5.09 / 5.33, x 700 5.46 / 5.42, x 2048 7.52 / 6.08).
template <int N>
int boards_per_step_team(int B) {
  if (N == 9) return B <= 384 ? 1 : B <= 1024 ? 2 : B <= 4096 ? 4 : 0;
  return B <= 512 ? 1 : B <= 2048 * Geo<N>::W ? Geo<N>::W : 0;
}
constexpr int kTeamsWithoutObservation = 1366;   // 19x19: more teams only pay with the observation
// boards per team of a step of this handle, or 0: one wavefront for everything
template <int N>
int step_team(const pgxgo_ctx* h, bool with_obs) {
  if (!h->automatic || h->zt || !tight_pitches<N>(h)) return 0;
  const int wb = boards_per_step_team<N>(h->B);
  return wb && (with_obs || (h->B + wb - 1) / wb <= kTeamsWithoutObservation) ? wb : 0;
}
// Outputs of a team launch up to this many bytes are stored the ordinary way (9x9 x 256 games 3.72 us against 3.83 written through, 19x19 x 400, 2.6
// MB, 5.09 / 5.13, without observation x 2048 5.24 / 5.36), beyond it through the L2 (9x9 x 2048, 3 MB, 4.63 / 4.55; 19x19 x 1000 6.10 / 5.66).
constexpr size_t kTeamPlainUpTo = (size_t)5 << 19;

// Boards per team of three wavefronts of a ply with the repetition rule in the mask (go_step_superko_team_kernel), or 0: one wavefront for
// everything.  us per ply, one wavefront / teams: 19x19 x 256 games 8.36 / 6.2, 1000 9.33 / 7.14, 3000 10.4 / 8.6, 5000 12.3 / 10.2, 8000 15.1 / 13.6, 10000 17.2 / 15.5,
// 12000 18.8 / 19.6, 16384 26.1 / 29.7; without observation 256 7.9 / 6.0, 5000 9.1 / 8.8, 10000 11.4 / 11.0, 12000 11.8 / 11.9; 9x9 x 256 8.0 / 6.05, 1000 9.0 /
// 7.05, 4096 9.6 / 8.2, 8192 10.6 / 9.5, 16384 12.8 / 12.2, 24000 14.7 / 15.1; without observation 4096 8.6 / 7.8, 16384 11.1 / 11.05.  The line lies farther out
// than without the rule (boards_per_step_team), as there is more to do beside the outputs.  Boards: 9x9 with 1 / 4 / 6 256 6.05 / 6.34 / 6.77, 1000 7.29 /
// 7.05 / 7.37, 5001 13.8 / 8.65 / 8.53; 19x19 with 1 / 3 256 6.24 / 6.57, 512 6.74 / 6.73, 1000 7.46 / 7.14.
template <int N>
int boards_per_superko_team(int B) {
  if (N == 9) return B <= 384 ? 1 : B <= 4096 ? 4 : B <= 16384 ? 6 : 0;
  return B <= 384 ? 1 : B <= 10240 ? Geo<N>::W : 0;
}
constexpr int superko_team_waves(bool with_obs) { return with_obs ? 3 : 2; }
template <int N>
int superko_team(const pgxgo_ctx* h) { return h->automatic && h->zt && h->sk_mode == 2 && tight_pitches<N>(h) ? boards_per_superko_team<N>(h->B) : 0; }

template <int N, bool TIGHT, bool SK>
void launch_emit_as(pgxgo_ctx* h, uint8_t* mask, uint8_t* obs) {
  hipLaunchKernelGGL((go_emit_kernel<N, TIGHT, SK>), dim3(blocks_for<N>(h->B)), dim3(64 * kWavesPerBlock), 0, h->stream, h->state, h->meta, h->B, mask,
                     h->mask_pitch, obs, h->obs_pitch, h->zt, h->zcur);
}

template <int N>
int launch_emit(pgxgo_ctx* h, uint8_t* mask, uint8_t* obs) {
  const bool tight = tight_pitches<N>(h), sk = h->zt && h->sk_mode == 2;   // only then does the rule change the mask
  if (tight && sk) launch_emit_as<N, true, true>(h, mask, obs);
  else if (tight) launch_emit_as<N, true, false>(h, mask, obs);
  else if (sk) launch_emit_as<N, false, true>(h, mask, obs);
  else launch_emit_as<N, false, false>(h, mask, obs);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
int launch_step(pgxgo_ctx* h, const int32_t* actions, bool sample, uint32_t seed, uint32_t t, const int32_t* start_t, int32_t* next) {
  StepArgs a;
  a.rew = h->rew_out; a.term = h->term_out;
  a.mask = h->mask_out; a.obs = h->obs_out; a.mask_pitch = h->mask_pitch; a.obs_pitch = h->obs_pitch;
  a.rules.seed = h->seed; a.rules.komi_x2 = h->komi_x2; a.rules.max_steps = h->max_steps; a.rules.auto_reset = h->auto_reset;
  a.sample_seed = seed; a.sample_t = t; a.next_actions = next;
  a.store_kind = store_kind_for(output_bytes_per_ply(h, h->mask_out != nullptr, h->obs_out != nullptr),
                                h->mask_out == h->mask_written && h->obs_out == h->obs_written);
  h->mask_written = h->mask_out; h->obs_written = h->obs_out;
  const dim3 grid(blocks_for_wb(h->B, h->wb)), block(64 * kWavesPerBlock);
  const bool tight = tight_pitches<N>(h);
  const int wb = step_team<N>(h, h->obs_out != nullptr);
  if (wb) {
    const dim3 tgrid((unsigned)((h->B + wb - 1) / wb + 7) & ~7u);
    const bool plain = output_bytes_per_ply(h, h->mask_out != nullptr, h->obs_out != nullptr) <= kTeamPlainUpTo;
    auto team = [&](auto sample_c, auto st_c) {
      hipLaunchKernelGGL((go_step_team_kernel<N, decltype(sample_c)::value, decltype(st_c)::value>), tgrid, block, 0, h->stream, h->state, h->meta, actions, start_t,
                         h->B, wb, tgrid.x / 8, a);
    };
    using Plain = std::integral_constant<int, kStorePlain>;
    using Through = std::integral_constant<int, kStoreThrough>;
    if (sample && plain) team(std::true_type{}, Plain{});
    else if (sample) team(std::true_type{}, Through{});
    else if (plain) team(std::false_type{}, Plain{});
    else team(std::false_type{}, Through{});
    HIPCHK(hipGetLastError());
    return PGXGO_OK;
  }
  if (h->zt && !sample) a.next_actions = nullptr;
  const int sk_wb = superko_team<N>(h);
  if (sk_wb) {
    const dim3 teams((unsigned)((h->B + sk_wb - 1) / sk_wb + 7) & ~7u);
    auto team = [&](auto obs_c, auto st_c) {
      constexpr bool O = decltype(obs_c)::value;
      hipLaunchKernelGGL((go_step_superko_team_kernel<N, O, decltype(st_c)::value>), teams, dim3(64 * superko_team_waves(O)), 0, h->stream, h->state, h->meta, actions, start_t, h->zcur, h->B, sk_wb,
                         teams.x / 8, h->zt, a);
    };
    using Plain = std::integral_constant<int, kStorePlain>;
    using Through = std::integral_constant<int, kStoreThrough>;
    const bool plain = output_bytes_per_ply(h, a.mask != nullptr, a.obs != nullptr) <= kTeamPlainUpTo;
    if (a.obs && plain) team(std::true_type{}, Plain{});
    else if (a.obs) team(std::true_type{}, Through{});
    else if (plain) team(std::false_type{}, Plain{});
    else team(std::false_type{}, Through{});
    HIPCHK(hipGetLastError());
    return PGXGO_OK;
  }
  if (h->zt) {
    auto sk = [&](auto tight_c, auto mode_c) {
      constexpr bool T = decltype(tight_c)::value;
      constexpr int M = decltype(mode_c)::value;
      if (a.store_kind == kStoreThrough) hipLaunchKernelGGL((go_step_superko_kernel<N, T, kStoreThrough, M>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->zcur, h->B, h->wb, grid.x / 8, h->zt, a);
      else if (a.store_kind == kStoreThroughWhole) hipLaunchKernelGGL((go_step_superko_kernel<N, T, kStoreThroughWhole, M>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->zcur, h->B, h->wb, grid.x / 8, h->zt, a);
      else hipLaunchKernelGGL((go_step_superko_kernel<N, T, kStoreStreamWhole, M>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->zcur, h->B, h->wb, grid.x / 8, h->zt, a);
    };
    using M1 = std::integral_constant<int, 1>;
    using M2 = std::integral_constant<int, 2>;
    if (tight && h->sk_mode == 1) sk(std::true_type{}, M1{});
    else if (tight) sk(std::true_type{}, M2{});
    else if (h->sk_mode == 1) sk(std::false_type{}, M1{});
    else sk(std::false_type{}, M2{});
    HIPCHK(hipGetLastError());
    return PGXGO_OK;
  }
  auto go = [&](auto sample_c, auto tight_c) {
    constexpr bool S = decltype(sample_c)::value, T = decltype(tight_c)::value;
    if (a.store_kind == kStoreThrough) hipLaunchKernelGGL((go_step_kernel<N, S, T, kStoreThrough>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->B, h->wb, grid.x / 8, a);
    else if (a.store_kind == kStoreThroughWhole) hipLaunchKernelGGL((go_step_kernel<N, S, T, kStoreThroughWhole>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->B, h->wb, grid.x / 8, a);
    else hipLaunchKernelGGL((go_step_kernel<N, S, T, kStoreStreamWhole>), grid, block, 0, h->stream, h->state, h->meta, actions, start_t, h->B, h->wb, grid.x / 8, a);
  };
  if (sample && tight) go(std::true_type{}, std::true_type{});
  else if (sample) go(std::true_type{}, std::false_type{});
  else if (tight) go(std::false_type{}, std::true_type{});
  else go(std::false_type{}, std::false_type{});
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
int launch_random(pgxgo_ctx* h, uint32_t seed, uint32_t t, const int32_t* start_t, int32_t* actions) {
  if (h->zt && h->sk_mode == 2)
    hipLaunchKernelGGL((go_random_actions_kernel<N, true>), dim3(blocks_for<N>(h->B)), dim3(64 * kWavesPerBlock), 0, h->stream, h->state, h->meta, start_t,
                       actions, h->B, seed, t, blocks_for<N>(h->B) / 8, h->zt, h->zcur);
  else
    hipLaunchKernelGGL((go_random_actions_kernel<N, false>), dim3(blocks_for<N>(h->B)), dim3(64 * kWavesPerBlock), 0, h->stream, h->state, h->meta, start_t,
                       actions, h->B, seed, t, blocks_for<N>(h->B) / 8, h->zt, h->zcur);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

// calls f with the rollout kernel's TIGHT and SK for this handle as compile-time constants
template <int N, class F>
void with_rollout_variant(const pgxgo_ctx* h, F&& f) {
  auto by_mode = [&](auto tight_c) {
    if (!h->zt) f(tight_c, std::integral_constant<int, 0>{});
    else if (h->sk_mode == 1) f(tight_c, std::integral_constant<int, 1>{});
    else f(tight_c, std::integral_constant<int, 2>{});
  };
  if (tight_pitches<N>(h)) by_mode(std::true_type{});
  else by_mode(std::false_type{});
}

// (with the repetition rule a rollout is never as fast as the cache: 16384 games, 2 to 8 slices, 2 to 80 plies, 0.72 to 0.97 with slots)
template <int N>
PaceArgs rollout_pace(const pgxgo_ctx* h, int steps, int slices, bool with_mask, bool with_obs) {
  PaceArgs p;
  with_rollout_variant<N>(h, [&](auto tight_c, auto sk_c) {
    // bytes written per game and ply: the whole record with the dense and the line-padded pitches, else without the pad
    constexpr bool T = decltype(tight_c)::value;
    const int64_t mask_bytes = T ? h->mask_pitch : Geo<N>::A, obs_bytes = T ? h->obs_pitch : Geo<N>::OBS;
    const double game_bytes = (double)((with_mask ? mask_bytes : 0) + (with_obs ? obs_bytes : 0));
    p = pace_args<go_rollout_kernel<N, T, decltype(sk_c)::value, true>>(h->B, h->wb, game_bytes, steps, slices,
                                                                           decltype(sk_c)::value ? 0.0 : 2.0, kPaceBytesPerSecond, kWavesPerBlock);
  });
  return p;
}

// Boards per team of a rollout (go_rollout_team_kernel), or 0 where one wavefront for everything is faster.  us for 16 plies in place, one
// wavefront / teams: 9x9 x 256 games 42.2 / 25.1, 1000 43.5 / 28.3, 5001 53.4 / 35.9, 12000 64.5 / 55.5, without observation x 1000 32.6 /
// 27.6, 5001 35.9 / 31.5; 19x19 x 400 60.3 / 34.0, 1500 72 / 39, 4000 81 / 66, 8192 121 / 114, 16384 227 / 212, 28000 377 / 353, 65536
// 836 / 797, without observation x 400 41.5 / 33.7, 8192 67 / 63.  A single ply gains too little (19x19 x 8192 14.4 / 15.8).
// A launch of teams takes longer to get going, the more of them a compute unit has to hold and the more generations of them there are, and
// needs plies to make up for it.  Time of teams over time of one wavefront, outputs that are not in the caches:
//  * 9x9, whose teams of six the machine holds up to 15360 games of: 2 plies 0.95 x 12288, 1.03 x 13312, 1.09 x 15360; 3 plies 0.96 x 13312, 0.99
//    x 14336, 1.02 x 15360; 4 plies 0.96 x 14336; 5 plies 0.99 x 15360; so 1024 games more for every ply.  Beyond, 8 plies 0.975 x 15616, 1.00 x
//    16384, 1.02 x 17408, 1.07 x 18432 (12 to 64 plies are the same), and again ahead where one wavefront for everything needs a fourth on
//    every SIMD: 8 plies 0.91 x 18433, 0.99 x 20480, 6 plies 0.98 x 19456, 1.006 x 20480, 4 plies 1.03 x 20480.
//  * 9x9 without observation: 2 plies 1.00 x 8000, 1.02 x 9000, 1.04 x 10000, 1.03 x 20480; 3 plies 0.98 x 13000, 1.02 x 14336; 16 plies 0.97 x 16384.
//  * 19x19 without observation: 2 plies 0.98 x 3072, 1.05 x 4000; 3 plies 0.99 x 4096, 1.01 x 5120, 1.04 x 5500; 4 plies 1.00 x 7000, 1.045 x 8192;
//    8 plies 0.99 x 7000, 1.025 x 8192, 1.00 x 10240; 16 / 32 plies 1.00 / 0.975 x 8192, 0.97 x 10240; beyond 3584 teams, x 11000, 1.08.
//  * 19x19: 2 plies 0.98 x 26000, 1.04 x 27648, 1.08 x 30720 (outputs in the cache 0.97, 1.00, 1.00), 3 plies 0.97 x 26000, 1.015 x 27648, 1.04 x
//    30720 (0.96, 0.99, 0.99), 4 plies 1.01 x 30720 (0.98); from 16 plies on teams win at every size.  Two slices written in turn, together more
//    than the memory-side cache, are slower by teams up to 6 plies (3 / 4 / 6 plies 0.94 / 0.98 / 0.94 x 22000, 0.95 / 1.03 / 1.00 x 23000, 1.06 /
//    1.07 / 1.015 x 27000; three slices 0.96 x 27000).
// Boards as in boards_per_step_team; 19x19 without observation, where the mask is short, spreads further (1000 games with 1 / 3 37.5 / 40.4).
template <int N>
int boards_per_rollout_team(int B, int steps, int slices, bool with_obs) {
  if (steps < 2) return 0;
  constexpr int K = 1024;
  int most;   // games
  if (N == 9 && with_obs) most = steps < 8 ? std::min(10 + steps, 15) * K : 16 * K;
  else if (N == 9) most = steps == 2 ? 8 * K : steps == 3 ? 13 * K : 20 * K;
  else if (!with_obs) most = steps < 4 ? (1 + steps) * K : steps < 16 ? 7 * K : 3584 * Geo<N>::W;
  else if (steps >= 16) most = B;
  else most = slices == 2 && steps < 7 ? 22 * K : steps < 4 ? (24 + steps) * K : 30 * K;
  const bool ahead_again = N == 9 && with_obs && steps >= 6 && B > 18 * K && B <= 20 * K;
  if (B > most && !ahead_again) return 0;
  if (N == 9) return B <= 384 ? 1 : B <= K ? 2 : B <= 4 * K ? 4 : 6;
  return with_obs ? (B <= 512 ? 1 : 3) : B <= K ? 1 : B <= 2 * K ? 2 : 3;
}

// The same with the repetition rule, whose table work stays with the rules and so weighs against teams.  us, one wavefront / teams: mode 1, 16 plies,
// 9x9 x 256 games 50.7 / 31.6, 5001 66.4 / 42.5, 19x19 x 1000 69.2 / 43.5, 4000 91.7 / 66.3; mode 2 9x9 x 256 68.6 / 51.2, 5001 97.4 / 77.8, 19x19 x 1000 85.3 /
// 64.0, 2000 99.5 / 68.8; without observation mode 1 9x9 x 5001 47.7 / 41.1, 19x19 x 1000 48.5 / 42.0, mode 2 75.8 / 71.0 x 4096 and 64.8 / 62.2.  Time of teams over
// time of one wavefront at the lines: with observation, where the machine holds the teams at once, mode 1 2 / 6 plies 0.90 / 0.80 x 9216, 1.16 / 1.05 x 10240
// (19x19 0.86 / 0.79 x 4608, 1.13 / 1.02 x 5120), mode 2 0.94 / 0.89 x 7000, 4 plies 1.16 x 8000 (19x19 0.89 / 0.78 x 3500, 1.04 x 4000).  Without it a launch of few
// plies does not make up for the teams' start: mode 1 2 plies 1.00 x 8192, 3 plies 0.97 x 12288 (19x19 0.96 x 4096, 1.01 x 6144), 6 plies 0.97 x 6144;
// mode 2 2 to 6 plies 0.93 to 1.04, 16 plies 0.94 x 4096, 0.99 x 8000 (19x19 0.96 x 4000, 0.97 x 6000).
template <int N>
int boards_per_superko_rollout_team(int B, int steps, bool with_obs, int mode) {
  constexpr int K = 1024;
  int most;   // games
  if (with_obs) most = steps < 2 ? 0 : (mode == 1 ? 1536 : 1152) * Geo<N>::W;
  else if (mode == 1) most = steps < 3 ? 0 : N == 9 ? 12 * K : steps < 4 ? 4 * K : 6 * K;
  else most = steps < 8 ? 0 : 6 * K;
  if (B > most) return 0;
  if (N == 9) return B <= 384 ? 1 : B <= K ? 2 : B <= 4 * K ? 4 : 6;
  return B <= 512 ? 1 : 3;
}
// boards per team of such a rollout of this handle, or 0: one wavefront for everything
template <int N>
int rollout_team(const pgxgo_ctx* h, int steps, int slices, bool with_mask, bool with_obs, const PaceArgs& pace) {
  if (!h->automatic || pace.ply || !tight_pitches<N>(h)) return 0;
  if (h->zt && !with_mask && !with_obs) return 0;   // (nothing to take off the wavefront with the rules: 300 plies of 9x9 x 5001, mode 2, 1.17 / 1.34 ms)
  return h->zt ? boards_per_superko_rollout_team<N>(h->B, steps, with_obs, h->sk_mode) : boards_per_rollout_team<N>(h->B, steps, slices, with_obs);
}
template <int N>
int team_of(const pgxgo_ctx* h, int steps, int slices, bool with_mask, bool with_obs) {   // steps = 0: of a step
  return steps ? rollout_team<N>(h, steps, slices, with_mask, with_obs, rollout_pace<N>(h, steps, slices, with_mask, with_obs)) : h->zt ? superko_team<N>(h) : step_team<N>(h, with_obs);
}

template <int N>
int launch_rollout(pgxgo_ctx* h, RolloutArgs& a) {
  const dim3 grid(blocks_for_wb(h->B, h->wb)), block(64 * kWavesPerBlock);
  a.pace = rollout_pace<N>(h, a.steps, a.slices, a.mask != nullptr, a.obs != nullptr);
  const int team = rollout_team<N>(h, a.steps, a.slices, a.mask != nullptr, a.obs != nullptr, a.pace);
  if (team) {
    a.wb = team;
    const dim3 teams((unsigned)(((int64_t)h->B + team - 1) / team + 7) & ~7u);
    auto go = [&](auto sk_c) {
      constexpr int M = decltype(sk_c)::value;
      if (a.obs) hipLaunchKernelGGL((go_rollout_team_kernel<N, true, M>), teams, dim3(64 * rollout_team_waves(true)), 0, h->stream, a);
      else hipLaunchKernelGGL((go_rollout_team_kernel<N, false, M>), teams, dim3(64 * rollout_team_waves(false)), 0, h->stream, a);
    };
    if (!h->zt) go(std::integral_constant<int, 0>{});
    else if (h->sk_mode == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
    HIPCHK(hipGetLastError());
    return PGXGO_OK;
  }
  with_rollout_variant<N>(h, [&](auto tight_c, auto sk_c) {
    constexpr bool T = decltype(tight_c)::value;
    constexpr int M = decltype(sk_c)::value;
    if (a.pace.ply) hipLaunchKernelGGL((go_rollout_kernel<N, T, M, true>), grid, block, 0, h->stream, a);
    else if (Geo<N>::RINGED && !a.obs) hipLaunchKernelGGL((go_rollout_kernel<N, T, M, false, Geo<N>::RINGED>), grid, block, 0, h->stream, a);
    else hipLaunchKernelGGL((go_rollout_kernel<N, T, M, false>), grid, block, 0, h->stream, a);
  });
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

// Boards per team of a search call of n entries (go_step_slots_team_kernel), 0 where one wavefront for everything is as fast.  The chain is
// that of a ply with two more loads ahead of it, and the lines lie where they lie for plies (us per call, one wavefront / teams: 9x9 x 256
// entries 4.38 / 3.26, 1024 4.51 / 3.47, 4096 4.66 / 4.11, without observation 256 3.38 / 3.11, 4096 3.63 / 3.36; 19x19 x 256 5.40 / 3.76, 1000
// 5.60 / 4.28, 4096 8.61 / 7.47, 5500 9.50 / 8.83, without observation 256 3.86 / 3.24).  Without observation teams have drawn level with
// one wavefront at 4096 entries of 19x19, out of 16384 games in progress 5.45 / 5.49, and are 2 to 5 % behind from there to the line
// (5500 5.77 / 5.98).  What bounds such a call now is the loads' chain (slot, state) and the rules.  Mere copies
// have no chain to shorten and stay with the other kernel, calls with the repetition rule too.
template <int N>
int boards_per_slot_team(int n) { return boards_per_step_team<N>(n); }

template <int N>
int launch_slots(pgxgo_ctx* h, int n, const int32_t* src, const int32_t* actions, const int32_t* dst, const SlotArgs& a) {
  const dim3 grid(blocks_for<N>(n)), block(64 * kWavesPerBlock);
  const bool tight = tight_pitches<N>(h), sk = h->zt != nullptr;
  const size_t out_bytes = (size_t)n * ((a.mask ? (size_t)a.mask_pitch : 0) + (a.obs ? (size_t)a.obs_pitch : 0));
  const int wb = tight && !sk && h->automatic && actions ? boards_per_slot_team<N>(n) : 0;
  if (wb) {
    const dim3 teams((unsigned)((n + wb - 1) / wb + 7) & ~7u);
    auto team = [&](auto obs_c, auto st_c) {
      constexpr bool O = decltype(obs_c)::value;
      hipLaunchKernelGGL((go_step_slots_team_kernel<N, O, decltype(st_c)::value>), teams, dim3(64 * (O ? 3 : 2)), 0, h->stream, src, dst, actions, h->state, h->meta, h->B,
                         n, wb, teams.x / 8, a);
    };
    using Plain = std::integral_constant<int, kStorePlain>;
    using Through = std::integral_constant<int, kStoreThrough>;
    const bool plain = out_bytes <= kTeamPlainUpTo;
    if (a.obs && plain) team(std::true_type{}, Plain{});
    else if (a.obs) team(std::true_type{}, Through{});
    else if (plain) team(std::false_type{}, Plain{});
    else team(std::false_type{}, Through{});
    HIPCHK(hipGetLastError());
    return PGXGO_OK;
  }
  if (tight && sk && h->sk_mode == 1) hipLaunchKernelGGL((go_step_slots_kernel<N, true, 1>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (tight && sk) hipLaunchKernelGGL((go_step_slots_kernel<N, true, 2>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (tight && store_kind_for(out_bytes, true) == kStoreThrough) hipLaunchKernelGGL((go_step_slots_kernel<N, true, 0, kStoreThrough>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (tight && store_kind_for(out_bytes, true) == kStoreThroughWhole) hipLaunchKernelGGL((go_step_slots_kernel<N, true, 0, kStoreThroughWhole>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (tight) hipLaunchKernelGGL((go_step_slots_kernel<N, true, 0, kStoreStreamWhole>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (sk && h->sk_mode == 1) hipLaunchKernelGGL((go_step_slots_kernel<N, false, 1>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else if (sk) hipLaunchKernelGGL((go_step_slots_kernel<N, false, 2>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  else hipLaunchKernelGGL((go_step_slots_kernel<N, false, 0>), grid, block, 0, h->stream, src, dst, actions, h->state, h->meta, h->B, n, grid.x / 8, a);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
int launch_export(pgxgo_ctx* h, const CanonArgs& c) {
  hipLaunchKernelGGL(go_export_kernel<N>, dim3(waves_for<N>(h->B)), dim3(64), 0, h->stream, h->state, h->meta, h->B, c);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
int launch_import(pgxgo_ctx* h, const CanonArgs& c) {
  hipLaunchKernelGGL(go_import_kernel<N>, dim3(waves_for<N>(h->B)), dim3(64), 0, h->stream, h->state, h->meta, h->rew_out, h->term_out, h->B,
                     c);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

template <int N>
size_t superko_bytes_for(int B, size_t* off_cur) {
  size_t o = align_up((size_t)B * Zt<N>::SLOTS * sizeof(uint2), 256);
  if (off_cur) *off_cur = o;
  return o + align_up((size_t)B * sizeof(uint4), 256);
}

// clears the tables, then (rebuild) fills them from the history window of the current state
template <int N>
int launch_superko_refresh(pgxgo_ctx* h, bool rebuild) {
  const size_t n16 = superko_bytes_for<N>(h->B, nullptr) / 16;
  const unsigned blocks = (unsigned)((n16 + 255) / 256 < 65536 ? (n16 + 255) / 256 : 65536);
  hipLaunchKernelGGL(go_zero_kernel, dim3(blocks), dim3(256), 0, h->stream, (uint4*)h->zt, n16);
  HIPCHK(hipGetLastError());
  if (rebuild) {
    hipLaunchKernelGGL(go_superko_rebuild_kernel<N>, dim3(waves_for<N>(h->B)), dim3(64), 0, h->stream, h->state, h->meta, h->B, h->zt, h->zcur, h->sk_mode);
    HIPCHK(hipGetLastError());
  }
  return PGXGO_OK;
}

#define DISPATCH_N(h, call19, call9) ((h)->N == 19 ? (call19) : (call9))

// validates the arguments of an init call and fills the handle; launches nothing
int fill_ctx(pgxgo_ctx* h, int32_t batch, int32_t board_size, uint32_t seed, const pgxgo_opts* opts, void* state_dev, size_t state_bytes) {
  if (batch <= 0 || (board_size != 9 && board_size != 19) || !state_dev) return PGXGO_EINVAL;
  if (((uintptr_t)state_dev & 255u) != 0) return PGXGO_EINVAL;
  const int P = board_size * board_size;
  pgxgo_opts o;
  if (opts) o = *opts;
  else { o.komi_x2 = 15; o.max_steps = 0; o.auto_reset = 0; o.obs_pitch = 0; o.mask_pitch = 0; o.stream = nullptr; }
  if (o.max_steps == 0) o.max_steps = 2 * P;
  if (o.max_steps < 1 || o.max_steps > 65535) return PGXGO_EINVAL;
  if (o.obs_pitch == 0) o.obs_pitch = P * 17;
  if (o.mask_pitch == 0) o.mask_pitch = P + 1;
  if (o.obs_pitch < P * 17 || o.mask_pitch < P + 1) return PGXGO_EINVAL;
  size_t off_meta, off_rew, off_term;
  const size_t need = board_size == 19 ? state_bytes_for<19>(batch, &off_meta, &off_rew, &off_term)
                                       : state_bytes_for<9>(batch, &off_meta, &off_rew, &off_term);
  if (state_bytes < need) return PGXGO_EINVAL;
  *h = pgxgo_ctx{};
  h->B = batch; h->N = board_size; h->seed = seed;
  h->wb = board_size == 19 ? auto_boards_per_wavefront<19>(batch) : auto_boards_per_wavefront<9>(batch);
  h->automatic = true;
  h->komi_x2 = o.komi_x2; h->max_steps = o.max_steps; h->auto_reset = o.auto_reset ? 1 : 0;
  h->obs_pitch = o.obs_pitch; h->mask_pitch = o.mask_pitch;
  h->stream = (hipStream_t)o.stream;
  uint8_t* base = (uint8_t*)state_dev;
  h->state = (uint32_t*)base;
  h->meta = (uint4*)(base + off_meta);
  h->rew_int = (float*)(base + off_rew);
  h->term_int = base + off_term;
  h->mask_out = nullptr; h->obs_out = nullptr; h->rew_out = h->rew_int; h->term_out = h->term_int;
  h->mask_written = nullptr; h->obs_written = nullptr;
  return PGXGO_OK;
}

// State of the handle made by pgxgo_init_static (callers that cannot allocate device memory).  In host code the
// array's name is only a stand-in: its device address comes from hipGetSymbolAddress, once per device.
constexpr int kMaxStaticDevices = 16;
void* g_scratch_ptr[kMaxStaticDevices] = {};
pgxgo_ctx g_static_ctx[kMaxStaticDevices] = {};

}  // namespace

static __device__ __align__(256) unsigned char scratch[PGXGO_STATIC_STATE_BYTES];

extern "C" {

size_t pgxgo_state_bytes(int32_t batch, int32_t board_size) {
  if (batch <= 0) return 0;
  if (board_size == 19) return state_bytes_for<19>(batch, nullptr, nullptr, nullptr);
  if (board_size == 9) return state_bytes_for<9>(batch, nullptr, nullptr, nullptr);
  return 0;
}

int32_t pgxgo_boards_per_wavefront(int32_t n) { return n == 19 ? Geo<19>::W : n == 9 ? Geo<9>::W : 0; }
int32_t pgxgo_num_actions(int32_t n) { return (n == 19 || n == 9) ? n * n + 1 : 0; }
int32_t pgxgo_obs_bytes(int32_t n) { return (n == 19 || n == 9) ? n * n * 17 : 0; }

int pgxgo_init(pgxgo_t* out, int32_t batch, int32_t board_size, uint32_t seed, const pgxgo_opts* opts, void* state_dev, size_t state_bytes) {
  if (!out) return PGXGO_EINVAL;
  *out = nullptr;
  if (!state_dev) return PGXGO_EINVAL;
  pgxgo_ctx* h = (pgxgo_ctx*)calloc(1, sizeof(pgxgo_ctx));
  if (!h) return PGXGO_ENOMEM;
  int rc = fill_ctx(h, batch, board_size, seed, opts, state_dev, state_bytes);
  if (rc == PGXGO_OK) rc = DISPATCH_N(h, launch_reset<19>(h, 1), launch_reset<9>(h, 1));
  if (rc == PGXGO_OK) {
    hipError_t e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) { g_last_hip = (int)e; rc = PGXGO_EHIP; }
  }
  if (rc != PGXGO_OK) { free(h); return rc; }
  *out = h;
  return PGXGO_OK;
}

int pgxgo_init_static(pgxgo_t* out, int32_t batch, int32_t board_size, uint32_t seed, const pgxgo_opts* opts) {
  if (!out) return PGXGO_EINVAL;
  *out = nullptr;
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxStaticDevices) return PGXGO_EINVAL;
  if (!g_scratch_ptr[dev]) {   // once per device, with that device current: each GPU holds its own copy of the array
    void* ptr = nullptr;
    HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr || ((uintptr_t)ptr & 255u) != 0) return PGXGO_EINVAL;
    g_scratch_ptr[dev] = ptr;
  }
  if (batch <= 0 || (board_size != 9 && board_size != 19)) return PGXGO_EINVAL;
  const size_t need = board_size == 19 ? state_bytes_for<19>(batch, nullptr, nullptr, nullptr) : state_bytes_for<9>(batch, nullptr, nullptr, nullptr);
  if (need > (size_t)PGXGO_STATIC_STATE_BYTES) return PGXGO_ELIMIT;
  pgxgo_ctx* h = &g_static_ctx[dev];
  const int rc = fill_ctx(h, batch, board_size, seed, opts, g_scratch_ptr[dev], (size_t)PGXGO_STATIC_STATE_BYTES);
  if (rc != PGXGO_OK) return rc;
  // everything the handle reads is (re)written by this launch: rows, scalars, rewards, terminated flags of `batch` games
  const int rc2 = DISPATCH_N(h, launch_reset<19>(h, 1), launch_reset<9>(h, 1));
  if (rc2 != PGXGO_OK) return rc2;
  *out = h;
  return PGXGO_OK;
}

int pgxgo_destroy(pgxgo_t h) {
  if (!h) return PGXGO_EINVAL;
  if (h >= g_static_ctx && h < g_static_ctx + kMaxStaticDevices) return PGXGO_OK;   // a static handle owns no host memory
  free(h);
  return PGXGO_OK;
}

int pgxgo_reset(pgxgo_t h) {
  if (!h) return PGXGO_EINVAL;
  int rc = DISPATCH_N(h, launch_reset<19>(h, 0), launch_reset<9>(h, 0));
  if (rc != PGXGO_OK) return rc;
  if (h->zt) {   // empty tables; the rebuild pass writes the per-game records of the fresh games
    rc = DISPATCH_N(h, launch_superko_refresh<19>(h, true), launch_superko_refresh<9>(h, true));
    if (rc != PGXGO_OK) return rc;
  }
  if (h->mask_out || h->obs_out) return DISPATCH_N(h, launch_emit<19>(h, h->mask_out, h->obs_out), launch_emit<9>(h, h->mask_out, h->obs_out));
  return PGXGO_OK;
}

int pgxgo_bind_outputs(pgxgo_t h, uint8_t* mask_dev, uint8_t* obs_dev, float* rewards_dev, uint8_t* terminated_dev) {
  if (!h) return PGXGO_EINVAL;
  float* new_rew = rewards_dev ? rewards_dev : h->rew_int;
  uint8_t* new_term = terminated_dev ? terminated_dev : h->term_int;
  if (new_rew != h->rew_out) HIPCHK(hipMemcpyAsync(new_rew, h->rew_out, (size_t)h->B * 2 * sizeof(float), hipMemcpyDeviceToDevice, h->stream));
  if (new_term != h->term_out) HIPCHK(hipMemcpyAsync(new_term, h->term_out, (size_t)h->B, hipMemcpyDeviceToDevice, h->stream));
  h->rew_out = new_rew; h->term_out = new_term;
  h->mask_out = mask_dev; h->obs_out = obs_dev;
  h->mask_written = mask_dev; h->obs_written = obs_dev;
  if (mask_dev || obs_dev) return DISPATCH_N(h, launch_emit<19>(h, mask_dev, obs_dev), launch_emit<9>(h, mask_dev, obs_dev));
  return PGXGO_OK;
}

int pgxgo_set_output_buffers(pgxgo_t h, uint8_t* mask_dev, uint8_t* obs_dev, float* rewards_dev, uint8_t* terminated_dev) {
  if (!h) return PGXGO_EINVAL;
  h->mask_out = mask_dev; h->obs_out = obs_dev;
  h->rew_out = rewards_dev ? rewards_dev : h->rew_int;
  h->term_out = terminated_dev ? terminated_dev : h->term_int;
  return PGXGO_OK;
}

int pgxgo_emit(pgxgo_t h, uint8_t* mask_dev, uint8_t* obs_dev) {
  if (!h || (!mask_dev && !obs_dev)) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_emit<19>(h, mask_dev, obs_dev), launch_emit<9>(h, mask_dev, obs_dev));
}

int pgxgo_step(pgxgo_t h, const int32_t* actions_dev) {
  if (!h || !actions_dev) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_step<19>(h, actions_dev, false, 0u, 0u, nullptr, nullptr), launch_step<9>(h, actions_dev, false, 0u, 0u, nullptr, nullptr));
}

int pgxgo_step_sample(pgxgo_t h, const int32_t* actions_dev, uint32_t seed, uint32_t t, const int32_t* start_t_dev, int32_t* next_actions_dev) {
  if (!h || !actions_dev || !next_actions_dev || next_actions_dev == actions_dev) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_step<19>(h, actions_dev, true, seed, t, start_t_dev, next_actions_dev),
                    launch_step<9>(h, actions_dev, true, seed, t, start_t_dev, next_actions_dev));
}

int pgxgo_rollout(pgxgo_t h, int32_t steps, int32_t slices, uint32_t seed, uint32_t t0, const int32_t* start_t_dev, int32_t* actions_dev,
                  float* rewards_dev, uint8_t* terminated_dev, uint8_t* mask_dev, uint8_t* obs_dev) {
  if (!h || steps < 0 || slices < 1) return PGXGO_EINVAL;
  if (steps == 0) return PGXGO_OK;
  RolloutArgs a;
  a.state = h->state; a.meta = h->meta; a.B = h->B; a.wb = h->wb;
  a.rules.seed = h->seed; a.rules.komi_x2 = h->komi_x2; a.rules.max_steps = h->max_steps; a.rules.auto_reset = h->auto_reset;
  a.steps = steps; a.slices = slices; a.seed = seed; a.t0 = t0; a.start_t = start_t_dev;
  a.actions = actions_dev; a.rew = rewards_dev; a.term = terminated_dev; a.mask = mask_dev; a.obs = obs_dev;
  a.mask_pitch = h->mask_pitch; a.obs_pitch = h->obs_pitch;
  a.zt = h->zt; a.zcur = h->zcur; a.sk_mode = h->sk_mode;
  return DISPATCH_N(h, launch_rollout<19>(h, a), launch_rollout<9>(h, a));
}

int pgxgo_rollout_in_time_slots(pgxgo_t h, int32_t steps, int32_t slices, int32_t with_mask, int32_t with_obs, int64_t* games_at_once) {
  if (!h || steps < 0 || slices < 1) return PGXGO_EINVAL;
  const PaceArgs p = DISPATCH_N(h, rollout_pace<19>(h, steps, slices, with_mask != 0, with_obs != 0), rollout_pace<9>(h, steps, slices, with_mask != 0, with_obs != 0));
  if (games_at_once) *games_at_once = (int64_t)8 * p.held * h->wb;
  return p.ply != 0u ? 1 : 0;
}

int pgxgo_boards_per_team(pgxgo_t h, int32_t steps, int32_t slices, int32_t with_mask, int32_t with_obs, int32_t* wavefronts) {
  if (!h || steps < 0 || slices < 1) return PGXGO_EINVAL;
  const int wb = DISPATCH_N(h, team_of<19>(h, steps, slices, with_mask != 0, with_obs != 0), team_of<9>(h, steps, slices, with_mask != 0, with_obs != 0));
  if (wavefronts) *wavefronts = !wb ? 1 : steps ? rollout_team_waves(with_obs != 0) : h->zt ? superko_team_waves(with_obs != 0) : (int)kTeamWaves;
  return wb;
}

int pgxgo_step_slots(pgxgo_t h, int32_t n, const int32_t* src_slots_dev, const int32_t* actions_dev, const int32_t* dst_slots_dev,
                     uint8_t* mask_dev, uint8_t* obs_dev, float* rewards_dev, uint8_t* terminated_dev) {
  if (!h || n < 0 || n > h->B || !src_slots_dev || !dst_slots_dev) return PGXGO_EINVAL;
  if (n == 0) return PGXGO_OK;
  SlotArgs a;
  a.rew = rewards_dev; a.term = terminated_dev; a.mask = mask_dev; a.obs = obs_dev; a.mask_pitch = h->mask_pitch; a.obs_pitch = h->obs_pitch;
  a.rules.seed = h->seed; a.rules.komi_x2 = h->komi_x2; a.rules.max_steps = h->max_steps; a.rules.auto_reset = h->auto_reset;
  a.zt = h->zt; a.zcur = h->zcur; a.sk_mode = h->sk_mode;
  return DISPATCH_N(h, launch_slots<19>(h, n, src_slots_dev, actions_dev, dst_slots_dev, a), launch_slots<9>(h, n, src_slots_dev, actions_dev, dst_slots_dev, a));
}

int pgxgo_copy_slots(pgxgo_t h, int32_t n, const int32_t* src_slots_dev, const int32_t* dst_slots_dev) {
  return pgxgo_step_slots(h, n, src_slots_dev, nullptr, dst_slots_dev, nullptr, nullptr, nullptr, nullptr);
}

int pgxgo_random_actions(pgxgo_t h, uint32_t seed, uint32_t t, const int32_t* start_t_dev, int32_t* actions_dev) {
  if (!h || !actions_dev) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_random<19>(h, seed, t, start_t_dev, actions_dev), launch_random<9>(h, seed, t, start_t_dev, actions_dev));
}

int pgxgo_legal_mask(pgxgo_t h, uint8_t* dst_dev) {
  if (!h || !dst_dev) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_emit<19>(h, dst_dev, nullptr), launch_emit<9>(h, dst_dev, nullptr));
}

int pgxgo_observe(pgxgo_t h, uint8_t* dst_dev) {
  if (!h || !dst_dev) return PGXGO_EINVAL;
  return DISPATCH_N(h, launch_emit<19>(h, nullptr, dst_dev), launch_emit<9>(h, nullptr, dst_dev));
}

int pgxgo_rewards(pgxgo_t h, float* dst_dev) {
  if (!h || !dst_dev) return PGXGO_EINVAL;
  if (dst_dev != h->rew_out) HIPCHK(hipMemcpyAsync(dst_dev, h->rew_out, (size_t)h->B * 2 * sizeof(float), hipMemcpyDeviceToDevice, h->stream));
  return PGXGO_OK;
}

int pgxgo_terminated(pgxgo_t h, uint8_t* dst_dev) {
  if (!h || !dst_dev) return PGXGO_EINVAL;
  if (dst_dev != h->term_out) HIPCHK(hipMemcpyAsync(dst_dev, h->term_out, (size_t)h->B, hipMemcpyDeviceToDevice, h->stream));
  return PGXGO_OK;
}

int pgxgo_current_player(pgxgo_t h, uint8_t* dst_dev) {
  if (!h || !dst_dev) return PGXGO_EINVAL;
  const int threads = 256;
  if (h->N == 19) hipLaunchKernelGGL(go_current_player_kernel<19>, dim3((h->B + threads - 1) / threads), dim3(threads), 0, h->stream, h->meta, h->B, dst_dev);
  else hipLaunchKernelGGL(go_current_player_kernel<9>, dim3((h->B + threads - 1) / threads), dim3(threads), 0, h->stream, h->meta, h->B, dst_dev);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

int pgxgo_export_state(pgxgo_t h, int8_t* board_dev, int8_t* history_dev, int32_t* ko_dev, int8_t* to_play_dev, int32_t* steps_dev,
                       int8_t* passes_dev, uint8_t* terminated_dev, uint8_t* black_player_dev, uint32_t* episode_dev, uint32_t* illegal_dev) {
  if (!h) return PGXGO_EINVAL;
  CanonArgs c = {board_dev, history_dev, ko_dev, to_play_dev, steps_dev, passes_dev, terminated_dev, black_player_dev, episode_dev, illegal_dev};
  return DISPATCH_N(h, launch_export<19>(h, c), launch_export<9>(h, c));
}

int pgxgo_import_state(pgxgo_t h, const int8_t* board_dev, const int8_t* history_dev, const int32_t* ko_dev, const int8_t* to_play_dev,
                       const int32_t* steps_dev, const int8_t* passes_dev, const uint8_t* terminated_dev, const uint8_t* black_player_dev,
                       const uint32_t* episode_dev) {
  if (!h || !board_dev || !history_dev || !ko_dev || !to_play_dev || !steps_dev || !passes_dev || !terminated_dev || !black_player_dev ||
      !episode_dev)
    return PGXGO_EINVAL;
  CanonArgs c = {(int8_t*)board_dev, (int8_t*)history_dev, (int32_t*)ko_dev, (int8_t*)to_play_dev, (int32_t*)steps_dev, (int8_t*)passes_dev,
                 (uint8_t*)terminated_dev, (uint8_t*)black_player_dev, (uint32_t*)episode_dev, nullptr};
  int rc = DISPATCH_N(h, launch_import<19>(h, c), launch_import<9>(h, c));
  if (rc != PGXGO_OK) return rc;
  if (h->zt) {
    rc = DISPATCH_N(h, launch_superko_refresh<19>(h, true), launch_superko_refresh<9>(h, true));
    if (rc != PGXGO_OK) return rc;
  }
  if (h->mask_out || h->obs_out) return DISPATCH_N(h, launch_emit<19>(h, h->mask_out, h->obs_out), launch_emit<9>(h, h->mask_out, h->obs_out));
  return PGXGO_OK;
}

int pgxgo_set_boards_per_wavefront(pgxgo_t h, int32_t boards) {
  if (!h) return PGXGO_EINVAL;
  const int wmax = h->N == 19 ? Geo<19>::W : Geo<9>::W;
  if (boards < 0 || boards > wmax) return PGXGO_EINVAL;
  h->wb = boards ? boards : (h->N == 19 ? auto_boards_per_wavefront<19>(h->B) : auto_boards_per_wavefront<9>(h->B));
  h->automatic = boards == 0;   // a number that is asked for is had
  return h->wb;
}

size_t pgxgo_superko_bytes(int32_t batch, int32_t board_size) {
  if (batch <= 0) return 0;
  if (board_size == 19) return superko_bytes_for<19>(batch, nullptr);
  if (board_size == 9) return superko_bytes_for<9>(batch, nullptr);
  return 0;
}

int pgxgo_enable_superko(pgxgo_t h, int32_t mode, void* table_dev, size_t table_bytes) {
  if (!h || mode < 0 || mode > 2) return PGXGO_EINVAL;
  if (mode == 0 || !table_dev) {
    if (mode != 0) return PGXGO_EINVAL;
    h->zt = nullptr; h->zcur = nullptr; h->sk_mode = 0;
  } else {
    if (((uintptr_t)table_dev & 255u) != 0 || h->max_steps > 2 * h->N * h->N) return PGXGO_EINVAL;
    size_t off_cur;
    const size_t need = h->N == 19 ? superko_bytes_for<19>(h->B, &off_cur) : superko_bytes_for<9>(h->B, &off_cur);
    if (table_bytes < need) return PGXGO_EINVAL;
    h->zt = (uint2*)table_dev;
    h->zcur = (uint4*)((uint8_t*)table_dev + off_cur);
    h->sk_mode = mode;
    const int rc = DISPATCH_N(h, launch_superko_refresh<19>(h, true), launch_superko_refresh<9>(h, true));
    if (rc != PGXGO_OK) { h->zt = nullptr; h->zcur = nullptr; h->sk_mode = 0; return rc; }
  }
  // the bound mask follows the rule in force from now on
  if (h->mask_out) return DISPATCH_N(h, launch_emit<19>(h, h->mask_out, nullptr), launch_emit<9>(h, h->mask_out, nullptr));
  return PGXGO_OK;
}

int pgxgo_sync(pgxgo_t h) {
  if (!h) return PGXGO_EINVAL;
  HIPCHK(hipStreamSynchronize(h->stream));
  return PGXGO_OK;
}

const char* pgxgo_strerror(int code) {
  switch (code) {
    case PGXGO_OK: return "ok";
    case PGXGO_EINVAL: return "invalid argument";
    case PGXGO_EHIP: return "HIP runtime error";
    case PGXGO_ENOMEM: return "out of host memory";
    case PGXGO_ELIMIT: return "size beyond the limit of the library's static buffer";
    default: return "unknown error";
  }
}

int pgxgo_last_hip_error(void) { return g_last_hip; }

int pgxgo_fill_probe(void* dst_dev, size_t nbytes, uint32_t value, int32_t kind, void* stream) {
  if (!dst_dev || ((uintptr_t)dst_dev & 15u) != 0 || (nbytes & 15u) != 0 || kind < 0 || kind > 2) return PGXGO_EINVAL;
  if (nbytes == 0) return PGXGO_OK;
  const size_t n16 = nbytes / 16;
  if ((n16 + 255) / 256 > 0x7FFFFFFFull) return PGXGO_EINVAL;
  const dim3 grid((unsigned)((n16 + 255) / 256)), block(256);
  if (kind == 0) hipLaunchKernelGGL(fill_probe_kernel<kStorePlain>, grid, block, 0, (hipStream_t)stream, (uint4*)dst_dev, n16, value);
  else if (kind == 1) hipLaunchKernelGGL(fill_probe_kernel<kStoreStream>, grid, block, 0, (hipStream_t)stream, (uint4*)dst_dev, n16, value);
  else hipLaunchKernelGGL(fill_probe_kernel<kStoreThrough>, grid, block, 0, (hipStream_t)stream, (uint4*)dst_dev, n16, value);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

int pgxgo_empty_probe(void* stream, int32_t count) {
  if (count < 0) return PGXGO_EINVAL;
  for (int32_t i = 0; i < count; ++i) hipLaunchKernelGGL(empty_probe_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

int pgxgo_lane_shift_probe(const uint32_t* in_dev, uint32_t* out_dev, void* stream) {
  if (!in_dev || !out_dev) return PGXGO_EINVAL;
  hipLaunchKernelGGL(lane_shift_probe_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, in_dev, out_dev);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

int pgxgo_remainder_probe(const uint32_t* n_dev, const uint32_t* d_dev, uint32_t* out_dev, int32_t count, void* stream) {
  if (!n_dev || !d_dev || !out_dev || count <= 0) return PGXGO_EINVAL;
  hipLaunchKernelGGL(remainder_probe_kernel, dim3(((unsigned)count + 255u) / 256u), dim3(256), 0, (hipStream_t)stream, n_dev, d_dev, out_dev, (uint32_t)count);
  HIPCHK(hipGetLastError());
  return PGXGO_OK;
}

}  // extern "C"
