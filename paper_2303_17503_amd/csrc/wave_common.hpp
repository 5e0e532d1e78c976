// wave_common.hpp -- wavefront-level building blocks shared by the game kernels of this library (gfx950, wave64).
//
// Mapping they serve: one board row per lane, several boards per wavefront separated by all-zero sentinel
// lanes, so that a one-lane DPP shift brings every row its north / south neighbour; board-wide facts come from
// ballots masked with the board's lane segment; byte outputs (legal mask, observation planes; Fig. 2 and
// Table 1 of the Pgx paper, arXiv 2303.17503) are staged as a bit stream in LDS and expanded 16 bits ->
// 16 bytes per lane through a 256-entry LDS table.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "remainder.hpp"

namespace pgxwave {

// counter-based hash of (seed, tag, env, t); tag 0 = action draw, tag 1 = seat draw (t = episode)
__device__ __forceinline__ uint32_t mixer(uint32_t x) {
  x ^= x >> 16; x *= 0x7feb352du;
  x ^= x >> 15; x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}
__device__ __forceinline__ uint32_t env_hash(uint32_t seed, uint32_t tag, uint32_t env, uint32_t t) {
  return mixer(mixer(mixer(seed + 0x9E3779B9u * (tag + 1u)) ^ env) ^ t);
}

// index of the calling wavefront within its block, as a value the compiler knows to be the same in every lane
// (so that everything derived from it -- output addresses, trip counts -- is computed once per wavefront)
__device__ __forceinline__ int wave_in_block() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Which piece of the batch a block works on.  The hardware hands the blocks of a launch to the chip's eight dies (each
// with an L2 of its own) round-robin by block index; with piece = block index, neighbouring stretches of every array
// would be written through eight different L2s, and a 128-byte line shared by the output runs of two neighbouring
// blocks would reach memory as two partial writes.  Block i takes piece (i mod 8) * (blocks / 8) + i / 8 instead, so
// that each die reads and writes one contiguous eighth of the batch and such lines leave one L2 whole (65536 games of
// 19x19: 85.5 -> 82.5 us per ply; 16384 games: 20.4 -> 20.15).  The grid must be a multiple of 8 blocks (pieces
// beyond the batch are idle).
__device__ __forceinline__ int piece_of_block(uint32_t eighth) { return (int)(blockIdx.x & 7u) * (int)eighth + (int)(blockIdx.x >> 3); }   // eighth: blocks / 8
__device__ __forceinline__ int piece_of_block() { return piece_of_block(gridDim.x >> 3); }

// Threads of a block of the board kernels (4 wavefronts), as a constant: the launch's own block size would be another load from
// the kernel's arguments ahead of everything else.
constexpr int kBlockThreads = 256;

// The kernels of one ply per launch take what the first loads need (pointers to state and actions, batch, boards per wavefront,
// blocks per eighth) as plain leading arguments, which the hardware puts into scalar registers before the first instruction
// (the build asks for it: -amdgpu-kernarg-preload-count); from the argument struct they came by four dependent loads, 1500
// cycles before the first state load was under way.  The rest of the arguments is loaded while the state is on its way.

// ------------------------------------------------------------------------------------------------
// Pacing of recorded rollouts.  A rollout whose plies go to fresh memory writes at the rate of DRAM, and DRAM is faster when
// the lines being written at any one time lie close together: thousands of wavefronts that each write their own 18 to 31 KB run
// whenever they have one reach 5.0 TB/s, the same runs written in the order of their addresses 6.3 TB/s.  So every wavefront
// gets a time slot per ply: wavefront i of the n that share an eighth of the batch (piece_of_block) starts its stores of ply s no
// earlier than (s + i / n) * T after it began, T being the time in which memory takes one ply's outputs.  Nothing but time
// depends on it: a wavefront that is late goes ahead at once, and the wait ends by the clock.
// Measured with a skeleton of the kernel's stores, 16 slices of 100 MB, 5 us of other work per ply: 337 us without slots,
// 331 / 259 / 284 / 309 us with T for 7.2 / 6.5 / 5.9 / 5.4 TB/s; staggering only the first ply gains nothing.
// ------------------------------------------------------------------------------------------------
// A batch of more wavefronts than the machine holds at once runs in generations: those of a later one start one after the
// other as their predecessors end, in step already, and share the time of as many as they are.
struct PaceArgs {
  uint32_t ply;    // T of a full generation (or of the whole batch if that is smaller), in 1/256 ticks of the constant 100 MHz clock; 0: not paced
  uint32_t held;   // wavefronts of an eighth that the machine holds at once
};
struct Pace {
  int64_t slot;      // when this wavefront may write its next ply, in 1/256 ticks of the constant 100 MHz clock
  uint32_t ply;      // T in the same unit
  __device__ __forceinline__ static int64_t now() {   // (the same in every lane, which the compiler does not know of the clock)
    const uint64_t t = __builtin_amdgcn_s_memrealtime() << 8;
    return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)t) |
                     ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(t >> 32)) << 32));
  }
  // begin: now() as the kernel begins.  index: this wavefront among the `eighth` wavefronts that write to the same eighth of the batch.  first:
  // when the first of them may write, in ticks after `begin`.  From the kernel's beginning: the loads of the state and the first ply, 4 to 5 us, then pass within the
  // slots of those that are to write early, who go ahead late, and not ahead of all slots (16 plies of 19x19 x 16384 games 285.8 -> 281.2
  // us, 8 of Hex x 262144, whose first slot lies 1 us later, 206.1 -> 202.4; each us later costs one).
  __device__ __forceinline__ Pace(bool on, int64_t begin, PaceArgs a, uint32_t index, uint32_t eighth, uint32_t first) : slot(0), ply(a.ply) {
    if (!on) return;
    slot = begin + ((int64_t)first << 8);
    if (eighth <= a.held) slot += (int64_t)((uint64_t)ply * index / eighth);
    else if (index < a.held) slot += (int64_t)((uint64_t)ply * index / a.held);
    else if (index >= eighth / a.held * a.held) ply = (uint32_t)((uint64_t)ply * (eighth % a.held) / a.held);
  }
  __device__ __forceinline__ void wait() {
    for (int i = 0; i < 8192 && now() < slot; ++i) __builtin_amdgcn_s_sleep(2);   // 128 cycles a turn
    slot += ply;
  }
};
// PaceArgs::held of a kernel (256 compute units; the kernel's registers and LDS decide); looked up once, 0 = unknown
template <auto KERNEL>
inline uint32_t waves_held_per_eighth(int waves_per_block) {
  static const int blocks = [&] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)KERNEL, 64 * waves_per_block, 0) == hipSuccess) return n;
    (void)hipGetLastError();   // the launch that follows is sound all the same and must not be reported as failed
    return 0;
  }();
  return (uint32_t)(blocks * 32 * waves_per_block);
}
// The pace of a rollout of `steps` plies into buffers of `slices` slices, of which min(steps, slices) are written; game_bytes: bytes
// per game and ply, wb: games per wavefront.  A rollout is paced if memory sets its speed:
//  * Lines that are written once have to outgrow the 256 MB memory-side cache, batches that run in generations counted whole (without
//    / with slots: 19x19 x 16384, 107 MB per ply, 2 slices 38.1 / 44.3 us, 3 slices 65.2 / 61.8, 16 slices 358 / 281; 2 slices of 65536
//    200 / 161).
//  * Where the plies rewrite slices (steps > slices), much of what they rewrite is still in the cache.  So the slices of the games on the
//    machine have to outgrow it by more, the more is rewritten: by `rewrite` times the rewritten share of the plies (time with slots over
//    time without, 19x19: 4 slices of 16384 games, 426 MB, 0.85 for 4 plies, 1.06 for 6, 1.11 for 40; 6 slices 0.93 for 12, 0.99 for 18,
//    1.07 for 60; 8 slices 0.84 to 0.92; 4 slices of 65536, 479 MB on the machine, 0.88 for 4 plies, 1.17 for 12, 1.28 for 40), and
//    hardly by more if the machine is not full (8 slices of 8000, 416 MB, 0.80 for 8 plies, 0.98 for 40; 16 of 9x9 x 20000, 467 MB, 0.83
//    to 0.86).
//  * A ply has to hold enough bytes for memory and not its own instructions to set the pace (20 MB of 19x19 x 3000 games: 271 / 284
//    us for 64 plies; 29 MB of 9x9 x 20000: 282 / 206 for 40; 18 MB of Hex x 30000: 359 / 349 for 64).
template <auto KERNEL>
inline PaceArgs pace_args(int B, int wb, double game_bytes, int steps, int slices, double rewrite, double bytes_per_second, int waves_per_block) {
  constexpr double kMB = 1048576.0;
  PaceArgs p;
  p.ply = 0u;
  p.held = waves_held_per_eighth<KERNEL>(waves_per_block);
  const double together = 8.0 * p.held * wb, at_once = B < together ? B : together, written = steps < slices ? steps : slices;
  const double rewritten = steps > slices ? 1.0 - (double)slices / steps : 0.0;
  if (B < 0.7 * together && rewrite > 0.5) rewrite = 0.5;
  const double footprint = (rewritten * rewrite > 0.0 ? at_once : (double)B) * game_bytes * written;
  if (written < 2.0 || footprint < 280.0 * kMB * (1.0 + rewrite * rewritten) || at_once * game_bytes < 23.0 * kMB) return p;
  p.ply = (uint32_t)(at_once * game_bytes * (256.0 * 1e8 / bytes_per_second));
  return p;
}

// ------------------------------------------------------------------------------------------------
// cross-lane primitives.  All of them must be called with every lane of the wavefront active.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t from_lane_below(uint32_t x) {  // lane i receives lane i-1, lane 0 receives 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t from_lane_above(uint32_t x) {  // lane i receives lane i+1, lane 63 receives 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
}
// A set and its neighbours, as two halves that are yet to be joined.
struct Halves {
  uint32_t a, b;
};
// Four growth steps of f0 within s0 and of f1 within s1 (rows of floods, whose neighbours are one bit or one lane away) and the halves of one
// more of each.  Word by word a step is five instructions and an idle one: the compiler keeps two instructions between a value and the DPP
// instruction that takes it, and one word has nothing to put there.  (The sets are read again after the floods are written, so a flood that
// starts as its whole set has to be kept out of the set's register.)
__device__ __forceinline__ void grow_pair(uint32_t& f0, uint32_t& f1, uint32_t s0, uint32_t s1, Halves& d0, Halves& d1) {
#define PGX_HALVES                                                                                                           \
  "v_lshl_or_b32 %2, %0, 1, %0\n\tv_lshrrev_b32_e32 %3, 1, %0\n\tv_lshl_or_b32 %4, %1, 1, %1\n\tv_lshrrev_b32_e32 %5, 1, %1\n\t" \
  "v_or_b32_dpp %2, %0, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"                                             \
  "v_or_b32_dpp %3, %0, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"                                             \
  "v_or_b32_dpp %4, %1, %4 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"                                             \
  "v_or_b32_dpp %5, %1, %5 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define PGX_STEP PGX_HALVES "v_bitop3_b32 %0, %2, %6, %3 bitop3:0xc8\n\tv_bitop3_b32 %1, %4, %7, %5 bitop3:0xc8\n\t"   // (first | third) & second
  asm(PGX_STEP PGX_STEP PGX_STEP PGX_STEP PGX_HALVES
      : "+&v"(f0), "+&v"(f1), "=&v"(d0.a), "=&v"(d0.b), "=&v"(d1.a), "=&v"(d1.b)
      : "v"(s0), "v"(s1));
#undef PGX_STEP
#undef PGX_HALVES
}
// The lanes where p holds.  (HIP's own ballot takes an int: a condition that is already a lane mask goes through a register and back.)
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// A fact about a whole board, known to every lane of the board: does `pred` hold in any of its rows?
// (seglo/seghi = the lanes holding the rows of the calling lane's board)
__device__ __forceinline__ bool board_any(bool pred, uint32_t seglo, uint32_t seghi) {
  const uint64_t m = ballot(pred);
  return (((uint32_t)m & seglo) | ((uint32_t)(m >> 32) & seghi)) != 0u;
}

// Returns v; keeps the compiler from evaluating anything that depends on a loaded value before this point (it
// would otherwise move the first use, and with it the wait for the load, up to the load itself).
__device__ __forceinline__ int32_t held_back(int32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Returns v; what is derived from the result is computed at this place and not ahead of a loop around it (a value kept through a
// loop costs a register in all of it).
template <class T>
__device__ __forceinline__ T in_place(T v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Has the wavefront-uniform values v in scalar registers from here on (the compiler would otherwise load kernel arguments one
// by one where they are first needed, each time with a wait of its own).
__device__ __forceinline__ void in_scalar_registers() {}
template <class V, class... T>
__device__ __forceinline__ void in_scalar_registers(const V& v, const T&... rest) {
  asm volatile("" ::"s"(v));
  in_scalar_registers(rest...);
}

// LDS traffic between the lanes of one wavefront needs no hardware barrier (a wavefront's LDS operations
// execute in program order); this only keeps the compiler from moving accesses across the hand-over.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Teams: a block whose wavefronts share one group of boards, one for the rules, the others for the outputs.
// Everything the wavefronts of a block wrote to LDS is there for all of them.  (Unlike __syncthreads this does not wait for their output
// stores as well, and it orders nothing in memory.)
__device__ __forceinline__ void team_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// The wavefront with the rules goes first where its SIMD has a team's other wavefront to issue from as well (more than one team per compute unit,
// 256) and no second one with rules (up to one team per SIMD, 1024): the team waits for it.  eighth: teams / 8.  us, without / with: a ply of 9x9 x 4096
// 4.88 / 4.49, x 3000 4.67 / 4.51; 32 plies of 9x9 in one launch without observation x 1000 38.4 / 36.2, x 5001 43.5 / 40.8, x 6000 43.9 / 41.0, with it x 1000 37.9 / 36.1,
// x 4096 53.0 / 52.1; 16 plies of 19x19 x 1500 without observation 29.5 / 27.1, with it 32.6 / 32.0; search x 4096 of 9x9 4.18 / 4.04.  With the repetition rule: 16 plies at
// play time 9x9 x 1000 36.7 / 35.9, x 5001 46.5 / 42.0, 19x19 x 2000 53.0 / 47.9, in the mask 9x9 x 5001 80.8 / 78.7, 19x19 x 2000 82.1 / 78.8; a ply in the mask 9x9 x 4096
// 8.25 / 8.10, 19x19 x 2000 8.67 / 8.52.  Hex, 16 plies x 1500 18.0 / 17.5, x 4000 20.2 / 17.7, x 5120 20.1 / 17.7, without observation 18.3 / 17.1.
// Beyond 1024 teams the outputs, which start later, lose what the rules gain or more: 32 plies of 9x9 x 8000 61.1 / 64.3, x 15000 119 / 140; search of 19x19 x 6144
// 9.2 / 9.8; 16 plies of Hex x 16384 45.3 / 46.7.  (Not everywhere: Hex x 8192 27.6 / 26.1, with the repetition rule 16 plies of 19x19 x 3400 63.5 / 57.3.)  With one team per
// compute unit nothing is gained (16 plies of 19x19 x 256 23.0 / 23.4, at play time 38.4 / 38.6).
__device__ __forceinline__ void rules_first(uint32_t eighth) {
  if (eighth > 32u && eighth <= 128u) __builtin_amdgcn_s_setprio(3);
}

// ------------------------------------------------------------------------------------------------
// bit stream -> byte stream.  `bits` (LDS) holds bit (head+i) = byte i of the destination, head = the
// destination's offset from the previous 16-byte boundary.  Whole aligned 16-byte groups are written as
// vectors, the ragged ends byte by byte.  Lane l always writes a group whose address is l*16 modulo 128, so
// that every store instruction of the wavefront covers eight whole 128-byte lines: a 1 KB store that straddles
// line boundaries costs a quarter more time once the lines have to reach DRAM (measured with a plain fill).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t spread4(uint32_t nibble) { return (nibble * 0x00204081u) & 0x01010101u; }

// 256-entry table in LDS: entry x = the eight bytes (0/1) of the bits of x.  Filled once per block.
__device__ __forceinline__ void fill_spread_table(uint2* lut) {
  for (uint32_t x = threadIdx.x; x < 256u; x += kBlockThreads) lut[x] = make_uint2(spread4(x & 15u), spread4(x >> 4));
  __syncthreads();
}

// The 16-byte output stores.  Basic kinds:
//   kStorePlain          ordinary store (write-back in the compute die's L2);
//   kStoreStream         with the non-temporal hint, for launches that write far more than the memory-side cache
//                        holds (below that size it is slower);
//   kStoreThrough        written through the L2 to the memory-side level (`sc1`).  Lines left dirty in the L2 have to
//                        be written back when the kernel ends: a plain fill of 106 MB pays 1.3 of its 16.8 us for
//                        that.  Partial lines written this way are expensive, though;
//   kStoreStreamThrough  both modifiers.
// and two that emit_bytes resolves per store instruction: the instructions of a stream that cover whole 128-byte
// lines only (all but its first and its last two) / the others, whose lines are shared with the streams next door:
//   kStoreThroughWhole   kStoreThrough / kStorePlain
//   kStoreStreamWhole    kStoreStreamThrough / kStoreStream
// Which kind a launch uses is decided on the host from the bytes it writes (all choices measured).
// The compiler has no builtin for a 16-byte store with the `sc1` modifier, hence the instruction itself.  It is
// followed by the two wait states this hardware needs between a store of more than 8 bytes and a write to its data
// registers (the compiler inserts them for its own stores; with one wait state rows of the state were stored wrong).
constexpr int kStorePlain = 0, kStoreStream = 1, kStoreThrough = 2, kStoreThroughWhole = 3, kStoreStreamThrough = 4, kStoreStreamWhole = 5;
typedef unsigned int vec4u __attribute__((ext_vector_type(4)));
template <int KIND>
__device__ __forceinline__ void store16(uint4* p, uint2 lo, uint2 hi) {
  const vec4u v4 = {lo.x, lo.y, hi.x, hi.y};
  static_assert(KIND != kStoreThroughWhole && KIND != kStoreStreamWhole, "resolved by emit_bytes");
  if constexpr (KIND == kStorePlain) *p = make_uint4(lo.x, lo.y, hi.x, hi.y);
  else if constexpr (KIND == kStoreStream) __builtin_nontemporal_store(v4, (vec4u*)p);
  else if constexpr (KIND == kStoreStreamThrough) asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v4) : "memory");
  else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v4) : "memory");
}
// the same to base + offset + IMM bytes, base the same in every lane (no 64-bit address arithmetic per lane)
template <int KIND, int IMM>
__device__ __forceinline__ void store16_at(uint8_t* base, uint32_t offset, uint2 lo, uint2 hi) {
  static_assert(IMM >= 0 && IMM < 4096, "fits the instruction");
  const vec4u v4 = {lo.x, lo.y, hi.x, hi.y};
  if constexpr (KIND == kStoreThrough) asm volatile("global_store_dwordx4 %0, %1, %2 offset:%3 sc1\n\ts_nop 1" ::"v"(offset), "v"(v4), "s"(base), "n"(IMM) : "memory");
  else if constexpr (KIND == kStoreStreamThrough) asm volatile("global_store_dwordx4 %0, %1, %2 offset:%3 sc1 nt\n\ts_nop 1" ::"v"(offset), "v"(v4), "s"(base), "n"(IMM) : "memory");
  else store16<KIND>((uint4*)(base + offset + IMM), lo, hi);
}

// A store of 1, 4, 8 or 16 bytes, written through the L2 if its launch's other stores are (KIND kStoreThrough).  A byte stored
// the ordinary way leaves a dirty piece of a line whose other pieces have been written through, and the lines of a stream's ragged
// ends then go to memory piece by piece: with such bytes written through as well, Hex x 16384 games 55.4 -> 44.3 us for 8 plies,
// 19x19 x 4096 entries of a search 39.4 -> 35.0 for 4, 19x19 x 5000 with superko 57.0 -> 53.4 for 4.  The wider ones gain in Hex (a further
// 44.2 -> 42.8) but not in Go, where rows of the state written through cost more than they save (search x 1024 35.6 -> 37.1,
// superko x 5000 53.2 -> 66).
template <int KIND, class T>
__device__ __forceinline__ void store_small(T* p, T v) {
  static_assert(sizeof(T) == 1 || sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "a store instruction's width");
  if constexpr (KIND != kStoreThrough) *p = v;
  else if constexpr (sizeof(T) == 1) asm volatile("global_store_byte %0, %1, off sc1" ::"v"(p), "v"((uint32_t)v) : "memory");
  else if constexpr (sizeof(T) == 4) asm volatile("global_store_dword %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
  else if constexpr (sizeof(T) == 8) {
    typedef unsigned int vec2u __attribute__((ext_vector_type(2)));
    asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(__builtin_bit_cast(vec2u, v)) : "memory");
  } else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(__builtin_bit_cast(vec4u, v)) : "memory");
}

// MAXBYTES: upper bound of nbytes.  MOST: upper bound of the rounds that are under way at once.  FIRST_AS_EDGE: the first round counts as an end of the stream
// even if it covers whole lines.  LARGE: see below.  dst and nbytes must be the same in every lane.
// The groups go out in rounds of 64, counted from the 128-byte line dst lies in, three or four rounds at a time: their bits and
// table entries are all read before the first of them is stored, so that a wavefront that has its SIMD to itself waits twice for
// LDS per batch and not twice per round.  A short stream's rounds stand in a loop and keep their tests in line: a kernel of 5 us
// runs through code it has to fetch, and every jump is another fetch.  Kernels of large batches (LARGE) fetch it once for all their wavefronts
// and do better without the tests (20 plies of Hex x 262144 with the mask alone 161 -> 158 us, x 65536 71.8 -> 69.3).
template <int MAXBYTES, int ST = kStorePlain, int MOST = 4, bool FIRST_AS_EDGE = false, bool LARGE = false>
__device__ __forceinline__ void emit_bytes(const uint32_t* bits, const uint2* lut, uint8_t* dst, uint32_t nbytes, int lane) {
  constexpr int ROUNDS = (((MAXBYTES + 15) >> 4) + 7 + 63) / 64;   // groups + the at most 7 of the line before dst
  constexpr int WANTED = ROUNDS < 3 ? ROUNDS : (ROUNDS < 12 ? 3 : 4);
  constexpr int AT_ONCE = WANTED < MOST ? WANTED : MOST;
  constexpr int ST_WHOLE = ST == kStoreThroughWhole ? kStoreThrough : (ST == kStoreStreamWhole ? kStoreStreamThrough : ST);
  constexpr int ST_EDGE = ST == kStoreThroughWhole ? kStorePlain : (ST == kStoreStreamWhole ? kStoreStream : ST);
  const uint32_t head = (uint32_t)((uintptr_t)dst & 15u);
  const uint32_t q = ((uint32_t)(uintptr_t)dst >> 4) & 7u;          // position of dst's group in its line
  uint8_t* line = dst - head - 16u * q;
  const uint32_t total = head + nbytes;
  const uint32_t first = q + (head ? 1u : 0u), last = q + (total >> 4);   // whole groups first .. last-1 of the line's count
  const uint16_t* src = (const uint16_t*)bits - q;
  const uint32_t offset = 16u * (uint32_t)lane;
  // the ragged ends, one byte per lane: lanes 0-15 the bytes before the first whole group, 16-31 those after the last one
  const uint32_t eb = (uint32_t)lane & 15u, pos = (lane & 16 ? total & ~15u : 0u) + eb;
  const bool edge = lane < 32 && (lane & 16 ? eb < (total & 15u) : head != 0u && eb >= head);
  const uint32_t edge_bits = edge ? bits[pos >> 5] : 0u;
  // rounds r0 .. r0+AT_ONCE-1; INSIDE: all of them lie within the whole groups
  auto batch = [&](uint32_t r0, auto inside) {
    constexpr bool INSIDE = decltype(inside)::value;
    const uint32_t g0 = 64u * r0 + (uint32_t)lane;   // this lane's group of the batch's first round
    uint32_t v[AT_ONCE];
    uint2 a[AT_ONCE], b[AT_ONCE];
#pragma unroll
    for (uint32_t k = 0; k < AT_ONCE; ++k) {
      if constexpr (INSIDE) v[k] = src[g0 + 64u * k];
      else { const uint32_t g = g0 + 64u * k; v[k] = src[g < q ? q : (g < last ? g : last - 1u)]; }   // any group of the stream does for a lane that stores nothing
    }
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) { a[k] = lut[v[k] & 255u]; b[k] = lut[v[k] >> 8]; }
    uint8_t* out = line + 1024u * r0;
    auto store = [&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if constexpr (k < AT_ONCE) {
        const uint32_t g = g0 + 64u * k;
        if constexpr (INSIDE) store16_at<ST_WHOLE, 1024 * k>(out, offset, a[k], b[k]);
        else if (ST_WHOLE != ST_EDGE && (!FIRST_AS_EDGE || r0 + k > 0u) && 64u * (r0 + k) >= first && 64u * (r0 + k + 1u) <= last) store16_at<ST_WHOLE, 1024 * k>(out, offset, a[k], b[k]);   // (the same in every lane)
        else if (__builtin_expect(g >= first && g < last, 1)) store16_at<ST_EDGE, 1024 * k>(out, offset, a[k], b[k]);
      }
    };
    static_assert(AT_ONCE <= 4, "one base per batch");
    store(std::integral_constant<int, 0>{}); store(std::integral_constant<int, 1>{}); store(std::integral_constant<int, 2>{}); store(std::integral_constant<int, 3>{});
    __builtin_amdgcn_sched_barrier(0);
  };
  // A stream of the full length (a wavefront with all its boards) ends in its last or last but one round: the batches between the
  // first and the one with these rounds need no tests.
  constexpr int INSIDE_END = (ROUNDS < 4 * AT_ONCE && !LARGE) ? AT_ONCE : AT_ONCE + (ROUNDS - 2 - AT_ONCE) / AT_ONCE * AT_ONCE;
  if (ROUNDS == 1) {
    const uint32_t g = (uint32_t)lane;
    if (g >= first && g < last) { const uint32_t v = src[g]; store16_at<ST_EDGE, 0>(line, offset, lut[v & 255u], lut[v >> 8]); }
  } else if (INSIDE_END > AT_ONCE && __builtin_expect(last >= 64u * (uint32_t)INSIDE_END, 1)) {
    batch(0u, std::false_type{});
#pragma unroll
    for (int r0 = AT_ONCE; r0 < INSIDE_END; r0 += AT_ONCE) batch((uint32_t)r0, std::true_type{});
#pragma unroll
    for (int r0 = INSIDE_END; r0 < ROUNDS; r0 += AT_ONCE) batch((uint32_t)r0, std::false_type{});
  } else {
#pragma unroll 1
    for (uint32_t r0 = 0u; 64u * r0 < last; r0 += AT_ONCE) batch(r0, std::false_type{});
  }
  if (edge) store_small<ST_EDGE>(line + 16u * q + pos, (uint8_t)((edge_bits >> (pos & 31u)) & 1u));
}

}  // namespace pgxwave
