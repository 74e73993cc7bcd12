// Steps 1 and 4-5 in one pass: the render of Eq. (1)-(2) and, for the
// fragments whose Id is still missing, the chunk level of their hash (Id of
// Alg. 2), from the same loads.
//
// Done separately, hash and render read every byte twice. Here one wave takes
// one (slot, tensor, stripe) task: a stripe is 64 consecutive BLAKE3 chunks of
// the tensor (64 KiB) and lane k hashes chunk k, 1 KiB of consecutive bytes,
// i.e. whole rows of the tensor (a row is 64 B .. 1 KiB).
//
// A full stripe goes line by line: line k is bytes [128 k, 128 k + 128) of every
// chunk. Eight lanes hold a line, 16 bytes each, so each load and store
// instruction moves eight whole lines (a lane's own blocks, 1 KiB from its
// neighbour's, would make every 16-byte piece a line of its own to the caches),
// and rotated K leaves the registers it was loaded to for the merged cache. Only
// the hash needs a chunk in one lane: a line is transposed through 9 KiB of LDS
// per wave, and each lane compresses its chunk's two blocks. Line k + 1 is loaded
// while line k is rotated, stored and hashed. V and offset-0 K are stored
// unchanged, other K rotated by R(off) in fp64; a lane's pieces of one line of
// all rows lie in the same columns, so its angles are a few registers.
//
// What bounds it: HBM, in this access pattern. 36,864 stripes of 64 KiB copied
// by waves that walk them in lines, as many waves as here, reach 5.4-5.55 TB/s read +
// written whatever the line's width (128 to 512 B), one-wave units in address order 6.1-6.7,
// but a chunk's 16 dependent compressions keep its line open for tens of
// microseconds, so the stripes in flight (three waves per SIMD: 192 MB) cannot be
// fewer. On 4.83 GB (Qwen3-4B N=4) the kernel takes 950 us: 925 us with neither
// hash nor rotation, 1047 us when each lane loaded its own chunk's blocks and
// the output went through the LDS (246 VGPRs, two waves per SIMD).
#include <type_traits>

#include "chunk_ops.h"
#include "fused_geometry.h"
#include "rotate.h"
#include "stripe_fold.h"

namespace cm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
// Persistent grid of up to CUs x 32 blocks (fewer when the set has fewer tasks).
// Many more blocks than fit keep the end of the launch short: a block that
// starts late has few tasks (4.83 GB: 975 us; as many blocks as fit 1041 us).
constexpr int kFusedBlocksPerCu = 32;
// Three waves per SIMD (168 VGPRs: two lines and their partners, the hash state
// or the fp64 rotation) hide a line's way from HBM better than two (Qwen3-1.7B
// N=2: 84 us, with two 92 us); half-split rows of 512 bytes and more re-read
// their partner lines and would spill.
constexpr int fused_waves(int style, int rb) {
  return style == CM_ROPE_HALF && rb >= 512 ? 2 : 3;
}

template <int V>
using IC = std::integral_constant<int, V>;

// The last stripe of a tensor, where each lane moves its own blocks: ordinary
// accesses (the 16-byte pieces of a line are merged by the caches). Lines carry
// the nontemporal hint both ways: they are whole, and neither side is read again.
__device__ __forceinline__ void load_block(u32x4 (&x)[4], const uint8_t* p) {
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = *global_ptr<u32x4>(p + 16 * q);
}

__device__ __forceinline__ void store16(uint8_t* p, u32x4 v) { *(CM_GLOBAL u32x4*)p = v; }

__device__ __forceinline__ void compress_block(B3Cv& st, const u32x4 (&x)[4], uint64_t chunk,
                                               uint32_t flags) {
  uint32_t w[16];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int k = 0; k < 4; ++k) w[4 * q + k] = x[q][k];
  b3_compress_paired<0>(st, w, chunk, 64, flags);
}

// N consecutive (cos, sin) pairs j0 .. j0 + N - 1 of a slot's pair-ordered
// table (entry j = cos, sin of off * theta_j). j0 is the same on every lane,
// so the pairs are read by scalar loads (through the constant address space:
// the table is not written while the kernel runs) into scalar registers, which
// the fp64 multiply and FMA take as operands. The table address is made opaque
// first, so that the loads stay where they are used (loop-invariant loads of
// every angle of the slot hoisted out of the step loop would not fit the
// scalar registers).
#define CM_CONST __attribute__((address_space(4)))
template <int N>
__device__ __forceinline__ void pair_angles(const double* __restrict__ table, int j0, double* cs,
                                            double* sn) {
  const double* a = table;
  asm volatile("" : "+s"(a));
  const CM_CONST double* ang = (const CM_CONST double*)a;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    cs[e] = ang[2 * (j0 + e)];
    sn[e] = ang[2 * (j0 + e) + 1];
  }
}

// A wave's LDS staging area: chunk c's line at byte c * 144, piece q at + 16 q.
// The 16 bytes of padding per chunk put the pieces q of any eight consecutive
// chunks, and the eight pieces of one chunk, on distinct LDS banks.
constexpr int kStageLane = 144;
constexpr int kStageBytes = 64 * kStageLane;

// Where a task's lanes read and write. By chunk (task()): s(b), the address of
// block b of the lane's chunk; d(pos), that of block pos of the lane's current
// output row (nullptr: the row is not written); next_row(). By line (lines()):
// line_s and line_d, the source and the merged place of the lane's j-th piece of
// line k (nullptr likewise); lo is fused_line_lane(lane).
//
// Dense: fragment tensors are contiguous [H][T][row] and the merged cache is
// [2L][H][T_out][row]; a lane's chunk is 1 KiB of consecutive bytes and it
// walks its rows into the merged cache.
template <int RB>
struct DenseTask {
  static constexpr bool kSkips = false;
  const uint8_t* src;     // the lane's chunk
  uint8_t* dst;           // the lane's current row in the merged cache
  int64_t left, T, gap;
  __device__ __forceinline__ const uint8_t* s(int b) const { return src + b * 64; }
  __device__ __forceinline__ uint8_t* d(int pos) const { return dst + pos * 64; }
  __device__ __forceinline__ void next_row() { fused_next_row(dst, left, T, gap, RB); }
};

template <int RB>
struct DenseLines {
  static constexpr bool kSkips = false;
  FusedStripe st;
  const uint8_t* sbase;   // the stripe, the same on every lane
  uint8_t* dbase;         // its first row in the merged cache
  int64_t gap;
  float inv_T;
  bool straight;          // the stripe ends before the next head's rows
  __device__ __forceinline__ const uint8_t* line_s(int k, int j, uint32_t lo, int) const {
    return sbase + fused_line_step(k, j) + lo;
  }
  // the merged place of stripe byte o
  __device__ __forceinline__ uint8_t* at(uint32_t o) const {
    return dbase + (o + fused_line_gap(st, o, __builtin_ctz(RB), gap, inv_T));
  }
  __device__ __forceinline__ uint8_t* line_d(int k, int j, uint32_t lo, int) const {
    uint8_t* p = dbase + fused_line_step(k, j);
    if (straight) return p + lo;
    return p + (lo + fused_line_gap(st, fused_line_step(k, j) + lo, __builtin_ctz(RB), gap, inv_T));
  }
};

// QP: stripes of at most 16 chunks are hashed by quads of lanes (the variant
// for sets whose tensors are all shorter than one stripe).
template <bool QP>
struct DenseAddr {
  const int64_t* table;   // per fragment: a row of `stride` int64, tensor pointers from entry 1
  int64_t stride;
  uint8_t* out;
  static constexpr bool kQuadPartial = QP;
  __device__ __forceinline__ const uint8_t* stripe(int64_t i, int64_t t, int64_t sidx) const {
    return reinterpret_cast<const uint8_t*>(table[i * stride + 1 + t]) + (sidx << 16);
  }
  template <int RB>
  __device__ __forceinline__ DenseTask<RB> task(int64_t i, int64_t t, int64_t sidx, int64_t off,
                                                int64_t T, int64_t T_out, int32_t H,
                                                int64_t bytes, int lane, int) const {
    constexpr int RB_SHIFT = __builtin_ctz(RB);
    const FusedLane fl = fused_lane(bytes, sidx, lane, RB_SHIFT, T, T_out, off);
    DenseTask<RB> a;
    a.src = reinterpret_cast<const uint8_t*>(table[i * stride + 1 + t]) + fl.src;
    a.dst = out + t * (int64_t)H * T_out * RB + fl.dst;
    a.left = fl.left;
    a.T = T;
    a.gap = (T_out - T) << RB_SHIFT;   // end of a head's rows -> next head
    return a;
  }
  template <int RB>
  __device__ __forceinline__ DenseLines<RB> lines(int64_t i, int64_t t, int64_t sidx, int64_t off,
                                                  int64_t T, int64_t T_out, int32_t H, int64_t,
                                                  int, int) const {
    constexpr int RB_SHIFT = __builtin_ctz(RB);
    DenseLines<RB> a;
    a.gap = (T_out - T) << RB_SHIFT;
    a.st = fused_stripe(sidx, RB_SHIFT, T, T_out, off);
    a.sbase = stripe(i, t, sidx);
    a.dbase = out + t * (int64_t)H * T_out * RB + a.st.dst;
    a.inv_T = 1.0f / (float)T;
    a.straight = !a.st.many && a.st.wrap == 0xFFFFFFFFu;
    return a;
  }
};

// Paged: fragments and the merged cache on pages of a pool (fused_geometry.h).
// At the start of a task each lane resolves the RPC rows of its chunk, where
// each is read and where it goes, into its column of the wave's LDS table
// (entry j * 64 + lane: source row j; (RPC + j) * 64 + lane: destination).
template <int RB>
struct PagedTask {
  static constexpr bool kSkips = true;
  static constexpr int RPC = 1024 / RB;
  static constexpr int BPR = RB / 64;
  static constexpr int RB_SHIFT = __builtin_ctz(RB);
  uint8_t* slice;          // the tensor's (layer, K/V) slice of the pool
  const uint32_t* rows;    // the lane's column of the wave's table
  const uint32_t* tab;     // the wave's table
  int j;                   // the lane's current output row (the same on every lane)
  __device__ __forceinline__ const uint8_t* s(int b) const {
    return slice + ((uint64_t)rows[(b / BPR) * 64] << RB_SHIFT) + (b % BPR) * 64;
  }
  __device__ __forceinline__ uint8_t* d(int pos) const {
    const uint32_t r = rows[(RPC + j) * 64];
    return r == kPagedSkipRow ? nullptr : slice + ((uint64_t)r << RB_SHIFT) + pos * 64;
  }
  __device__ __forceinline__ void next_row() { ++j; }
  __device__ __forceinline__ const uint8_t* line_s(int k, int jj, uint32_t, int lane) const {
    const int r = fused_line_row<RB>(k, lane), c = 8 * jj + (lane >> 3);
    return slice + ((uint64_t)tab[r * 64 + c] << RB_SHIFT) + fused_line_col<RB>(k, lane);
  }
  __device__ __forceinline__ uint8_t* line_d(int k, int jj, uint32_t, int lane) const {
    const int r = fused_line_row<RB>(k, lane), c = 8 * jj + (lane >> 3);
    const uint32_t row = tab[(RPC + r) * 64 + c];
    return row == kPagedSkipRow ? nullptr
                                : slice + ((uint64_t)row << RB_SHIFT) + fused_line_col<RB>(k, lane);
  }
};

struct PagedAddr {
  uint8_t* pool;
  int64_t P;                 // pages
  int32_t b_shift;           // log2 of the rows per page
  const int64_t* table;      // per fragment {T, first}: its page ids start at blocks[first]
  const int32_t* blocks;
  const int32_t* k_table;    // merged block -> page, K and V
  const int32_t* v_table;
  uint32_t* lds;             // the block's tables: [waves][2 * RPC][64]
  static constexpr bool kQuadPartial = false;
  template <int RB>
  __device__ __forceinline__ PagedTask<RB> lines(int64_t i, int64_t t, int64_t sidx, int64_t off,
                                                 int64_t T, int64_t T_out, int32_t H,
                                                 int64_t bytes, int lane, int wave) const {
    return task<RB>(i, t, sidx, off, T, T_out, H, bytes, lane, wave);
  }
  template <int RB>
  __device__ __forceinline__ PagedTask<RB> task(int64_t i, int64_t t, int64_t sidx, int64_t off,
                                                int64_t T, int64_t, int32_t H, int64_t,
                                                int lane, int wave) const {
    constexpr int RPC = PagedTask<RB>::RPC;
    constexpr int RB_SHIFT = PagedTask<RB>::RB_SHIFT;
    PagedTask<RB> a;
    a.slice = pool + ((t * P * H) << (b_shift + RB_SHIFT));
    uint32_t* col = lds + (int64_t)wave * (2 * RPC * 64) + lane;
    a.rows = col;
    a.tab = col - lane;
    a.j = 0;
    const int64_t first = table[2 * i + 1];
    const int32_t* tab = (t & 1) ? v_table : k_table;
    wave_lds_order();                    // the task before has looked its rows up
    const int64_t q0 = (sidx * 64 + lane) * RPC;   // the chunk's first row in the tensor
    const int64_t rows = (int64_t)H * T;
    ChunkRow c = fused_chunk_row(sidx, lane, RB_SHIFT, T);
#pragma unroll
    for (int r = 0; r < RPC; ++r) {
      uint32_t sr = 0, dr = kPagedSkipRow;
      if (q0 + r < rows) paged_row_pair(blocks, first, tab, P, H, b_shift, off, c, &sr, &dr);
      col[r * 64] = sr;
      col[(RPC + r) * 64] = dr;
      fused_chunk_next(c, T);
    }
    wave_lds_order();                    // lanes look up each other's columns
    return a;
  }
};

// The chaining values of a stripe of at most 16 chunks of a dense tensor, by
// quads of lanes: lanes 4Q .. 4Q + 3 hash chunk Q (b3_chunk_quad), a chain of
// about half the latency of one lane's. On a small set such stripes are all the
// work and few waves run. stripe: the stripe's first byte; blocks: the tensor's
// 64-byte blocks. Returns words q and 4 + q of chunk Q's value in lane 4Q + q. Out
// of line: inlined, it makes the 256-byte-row kernel spill.
__device__ __attribute__((noinline)) uint2 quad_hash_stripe(const uint8_t* stripe, int64_t blocks,
                                                            int64_t sidx, bool root, int lane) {
  const int Q = lane >> 2;
  const int64_t left = blocks - (sidx * kStripeChunks + Q) * 16;
  const int nb = left <= 0 ? 0 : (left > 16 ? 16 : (int)left);
  uint32_t lo = 0, hi = 0;
  const uint8_t* c = stripe + ((int64_t)Q << 10);
  if (nb != 0)                                         // uniform over the quad
    b3_chunk_quad(lo, hi, nb, (uint64_t)(sidx * kStripeChunks + Q), root, (lane & 1) != 0,
                  (lane & 2) != 0,
                  [&](int64_t b, uint32_t (&w)[16]) { load_block64(c + b * 64, w); });
  return make_uint2(lo, hi);
}

// ESIZE: element bytes; STYLE: pairing; RB: row bytes (64 .. 1024); Addr: the
// storage of the fragments and of the merged cache.
template <int ESIZE, int STYLE, int RB, class Addr>
__device__ __forceinline__ void render_hash_body(
    const Addr& addr, int32_t n, const int64_t* __restrict__ plan,
    const int64_t* __restrict__ task_base, const double* __restrict__ angles, int32_t H,
    int32_t d, const uint8_t* __restrict__ select, int32_t level,
    const int64_t* __restrict__ base_v,
    uint8_t* __restrict__ nodes) {
  constexpr int EP = 16 / ESIZE;              // elements per 16-byte piece
  constexpr int BPR = RB / 64;                // blocks per row: 1 .. 16
  constexpr int HBK = BPR / 2;                // blocks per half row (0: a row is one block)
  constexpr bool HALF = STYLE == CM_ROPE_HALF;
  // the wave index is the same on every lane: say so, so that everything derived
  // from the task (slot, lengths, offsets, step positions, branches) stays in
  // scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * kWaves;
  // Per wave, the staging area through which a line of every chunk, loaded by
  // eight lanes each, reaches the lane that hashes the chunk.
  __shared__ __attribute__((aligned(16))) uint8_t stage_lds[kWaves][kStageBytes];
  uint8_t* stage_line = stage_lds[wave] + (lane >> 3) * kStageLane + (lane & 7) * 16;
  const uint8_t* stage_chunk = stage_lds[wave] + lane * kStageLane;
  const int lq = lane & 7;                         // piece of its lines this lane holds
  // the plan and the task bases are read on the device: a plan the host has not
  // seen is rendered as it stands (its length T_out fits the output by contract)
  const int n_u = (int)plan[CM_PLAN_NUNIQUE];
  const int64_t T_out = plan[CM_PLAN_TOUT];
  const int64_t total_tasks = task_base[n];      // 0 for a plan whose status is an error
  for (int64_t task = (int64_t)blockIdx.x * kWaves + wave; task < total_tasks; task += waves) {
    const int s = fused_slot(task_base, n_u, task);
    const int64_t i = plan[CM_PLAN_HEADER + s];
    const int64_t off = plan[CM_PLAN_HEADER + n + s];
    const int64_t T = plan[CM_PLAN_HEADER + 2 * (int64_t)n + s];
    const bool hashing = select[i] == 0;
    const int64_t bytes = (int64_t)H * T * RB;
    const int64_t stripes = stripes_of(bytes);
    const int64_t local = task - task_base[s];
    const int64_t t = local / stripes;             // tensor: 2l + kv
    const int64_t sidx = local - t * stripes;
    const bool rotate = (t & 1) == 0 && off != 0;
    const double* ang = angles + (int64_t)s * d;
    const int64_t m = chunks_of(bytes);
    const int64_t in_stripe = (bytes >> 6) - sidx * kStripeBlocks;
    const bool full = in_stripe >= kStripeBlocks;
    // a last stripe of at most 16 chunks is hashed by quads of lanes in the
    // kernel variant for sets of short tensors (kept out of the other variants:
    // the extra code changes their registers and costs the full-stripe loop)
    constexpr bool kQuadPartial = Addr::kQuadPartial;
    const bool quad_hash = kQuadPartial && hashing && !full && in_stripe <= 16 * 16;
    const uint64_t chunk = (uint64_t)sidx * kStripeChunks + lane;
    const int64_t blocks_left = (bytes >> 6) - (int64_t)chunk * 16;
    const int nb = blocks_left < 0 ? 0 : (blocks_left > 16 ? 16 : (int)blocks_left);
    B3Cv st;
    b3_init(st);
    const uint32_t root = m == 1 ? kB3Root : 0u;
    auto flags = [&](int b, int last) {
      return (b == 0 ? kB3ChunkStart : 0u) | (b == last ? (kB3ChunkEnd | root) : 0u);
    };

    // Rotation in place of block x, block bi of its row (pos of its first
    // piece: bi * 64 bytes), for the pairings a block holds by itself: both
    // halves of a 64-byte row, or interleaved pairs.
    auto rotate_own = [&](u32x4 (&x)[4], int bi) {
      if constexpr (HALF) {
        // the row is this one block: pieces 0, 1 pair with pieces 2, 3
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          double cs[EP], sn[EP];
          pair_angles<EP>(ang, q * EP, cs, sn);
          rotate_pair_half<ESIZE>(x[q], x[q + 2], cs, sn);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double cs[EP / 2], sn[EP / 2];
          pair_angles<EP / 2>(ang, (bi * 64 + 16 * q) / ESIZE / 2, cs, sn);
          x[q] = rotate_piece_il<ESIZE>(x[q], cs, sn);
        }
      }
    };
    // Rotation in place of first-half block a (block bi of its row) and its
    // second-half partner b.
    auto rotate_halves = [&](u32x4 (&a)[4], u32x4 (&b)[4], int bi) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double cs[EP], sn[EP];
        pair_angles<EP>(ang, bi * (4 * EP) + q * EP, cs, sn);
        rotate_pair_half<ESIZE>(a[q], b[q], cs, sn);
      }
    };
    // Angles of the lane's piece of line k (the sine's sign flipped on a second
    // half that is rotated by itself, see rotate_piece_half).
    constexpr int NA = HALF ? EP : EP / 2;
    auto line_angles = [&](int k, double (&cs)[NA], double (&sn)[NA]) {
      constexpr int LPR = RB >= 128 ? RB / 128 : 1;           // lines per row
      int j0;
      bool flip = false;
      if constexpr (HALF && RB >= 256) {
        j0 = ((k % (LPR / 2)) * 8 + lq) * EP;
      } else if constexpr (HALF) {
        constexpr int P = RB / 32;                            // pieces per half row
        j0 = (lq & (P - 1)) * EP;
        flip = (lq & P) != 0;
      } else {
        j0 = (RB >= 128 ? (k % LPR) * 8 + lq : lq & 3) * (EP / 2);
      }
      const CM_GLOBAL double* a = (const CM_GLOBAL double*)ang + 2 * j0;
#pragma unroll
      for (int e = 0; e < NA; ++e) {
        cs[e] = a[2 * e];
        sn[e] = flip ? -a[2 * e + 1] : a[2 * e + 1];
      }
    };
    uint32_t lo = fused_line_lane(lane);
    auto store_piece = [&](const auto& A, const u32x4& x, int k, int j) {
      uint8_t* p = A.line_d(k, j, lo, lane);
      if constexpr (std::decay_t<decltype(A)>::kSkips) {
        if (p != nullptr) st_stream(p, x);
      } else {
        st_stream(p, x);
      }
    };
    auto load_line = [&](const auto& A, u32x4 (&x)[8], int k) {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = ld16(A.line_s(k, j, lo, lane));
    };

    // A full stripe (every chunk has 16 blocks) line by line. Step k: line k of
    // every chunk (cur, loaded a step earlier) goes to the LDS for the hash; the
    // next line's loads are issued into the other buffer; the line is rotated in
    // the lanes that hold it and stored; each lane then reads its own chunk's
    // two blocks back and compresses them. Half-split pairs: in the same line
    // (rows up to 128 bytes, the partner's lane by a lane move), in the line
    // before (256: it waits in the other buffer, and the next loads are issued
    // once both are stored), or further back (re-read from the cache).
    auto full_stripe = [&](auto rotc) {
      constexpr bool ROT = decltype(rotc)::value;
      constexpr bool SPLIT = ROT && HALF && RB >= 256;   // halves in different lines
      constexpr int HL = RB >= 256 ? RB / 256 : 1;       // lines per half row
      constexpr bool KEEP = SPLIT && HL == 1;
      u32x4 xa[8], xb[8], par[8];
      const auto A = addr.template lines<RB>(i, t, sidx, off, T, T_out, H, bytes, lane, wave);
      auto step = [&](int k, u32x4 (&cur)[8], u32x4 (&oth)[8]) {
        const bool second = SPLIT && ((k / HL) & 1) != 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) launder(cur[j]);
        asm volatile("" : "+v"(lo));       // no address is kept from step to step
        // the memory accesses of a step go ahead of other waves' compressions
        // (Qwen3-1.7B N=2: 90 -> 85 us)
        __builtin_amdgcn_s_setprio(3);
        __builtin_amdgcn_sched_barrier(0);
        if (hashing) {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            *reinterpret_cast<u32x4*>(stage_line + j * 8 * kStageLane) = cur[j];
        }
        if constexpr (!KEEP) {
          if (k + 1 < 8) load_line(A, oth, k + 1);
        } else {
          if (!second && k + 1 < 8) load_line(A, oth, k + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!ROT) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            store_piece(A, cur[j], k, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else if constexpr (!SPLIT) {
          double cs[NA], sn[NA];
          line_angles(k, cs, sn);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            if constexpr (HALF)
              cur[j] = rotate_piece_half<ESIZE>(cur[j], lane_xor4<(RB >= 128 ? 4 : 2)>(cur[j]), cs, sn);
            else
              cur[j] = rotate_piece_il<ESIZE>(cur[j], cs, sn);
            store_piece(A, cur[j], k, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else if (second) {
          double cs[NA], sn[NA];
          line_angles(k, cs, sn);
          u32x4 (&first)[8] = KEEP ? oth : par;
          if constexpr (!KEEP) load_line(A, par, k - HL);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            rotate_pair_half<ESIZE>(first[j], cur[j], cs, sn);
            store_piece(A, first[j], k - HL, j);
            store_piece(A, cur[j], k, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if constexpr (KEEP) {
          __builtin_amdgcn_sched_barrier(0);
          if (second && k + 1 < 8) load_line(A, oth, k + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        if (hashing) {
          u32x4 m0[4], m1[4];
          wave_lds_order();                  // the other lanes' pieces are written
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            m0[q] = *reinterpret_cast<const u32x4*>(stage_chunk + 16 * q);
            m1[q] = *reinterpret_cast<const u32x4*>(stage_chunk + 64 + 16 * q);
          }
          wave_lds_order();                  // before the next line goes to the same LDS
          compress_block(st, m0, chunk, flags(2 * k, kB3ChunkBlocks - 1));
          compress_block(st, m1, chunk, flags(2 * k + 1, kB3ChunkBlocks - 1));
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      load_line(A, xa, 0);
#pragma nounroll
      for (int k = 0; k < 8; k += 2) {
        step(k, xa, xb);
        step(k + 1, xb, xa);
      }
    };

    // The last stripe of a tensor (a lane may own fewer than 16 blocks, or
    // none): a block at a time, its partner re-read when it is needed, each lane
    // storing its own blocks; at most one stripe per tensor, so it is kept
    // short in registers.
    auto partial = [&](auto rotc) {
      constexpr bool ROT = decltype(rotc)::value;
      u32x4 x[4], par[4];
      auto A = addr.template task<RB>(i, t, sidx, off, T, T_out, H, bytes, lane, wave);
      constexpr bool SKIPS = decltype(A)::kSkips;   // rows that are not written
      for (int b = 0; b < nb; ++b) {
        const int pos = b & (BPR - 1);
        load_block(x, A.s(b));
        if (ROT && HALF && BPR > 1 && pos >= HBK) load_block(par, A.s(b - HBK));
        if (hashing && !quad_hash) compress_block(st, x, chunk, flags(b, nb - 1));
        bool out = true;
        if (ROT) {
          if (HALF && BPR > 1) {
            if (pos >= HBK) rotate_halves(par, x, pos - HBK);
            else out = false;                     // stored with its partner
          } else {
            rotate_own(x, pos);
          }
        }
        if (out && (!SKIPS || A.d(0) != nullptr)) {
          if (ROT && HALF && BPR > 1) {
            uint8_t* dp = A.d(pos - HBK);
#pragma unroll
            for (int q = 0; q < 4; ++q) store16(dp + 16 * q, par[q]);
          }
          uint8_t* dx = A.d(pos);
#pragma unroll
          for (int q = 0; q < 4; ++q) store16(dx + 16 * q, x[q]);
        }
        if (pos == BPR - 1) A.next_row();
      }
    };

    // The last stripe of a short tensor, at most 16 chunks, in the variant for sets
    // of such tensors: the wave takes it piece by piece in memory order, eight KiB
    // in flight, rotated like the unit render's pieces. (By chunk, a block at a time,
    // each lane waits for 16 loads one after the other: tensors of 8 and 12
    // chunks, four of each, this kernel 27.5 us so and 20.6 us this way, the whole
    // path 46.3 and 39.6 us. The limit of 16 chunks is the quad hash's; a longer
    // stripe is hashed from the registers it is rendered in.)
    auto short_stripe = [&](auto rotc) {
      constexpr bool ROT = decltype(rotc)::value;
      if constexpr (kQuadPartial) {
      constexpr int PPR = RB / 16, P = RB / 32;        // pieces per row and per half row
      const auto A = addr.template lines<RB>(i, t, sidx, off, T, T_out, H, bytes, lane, wave);
      const uint32_t end = (uint32_t)(in_stripe * 64);
      const int cp = lane & (PPR - 1);
      double cs[NA], sn[NA];
      if constexpr (ROT) {
        const bool flip = HALF && (cp & P) != 0;
        const CM_GLOBAL double* a = (const CM_GLOBAL double*)ang +
                                    2 * (HALF ? (cp & (P - 1)) * EP : cp * (EP / 2));
#pragma unroll
        for (int e = 0; e < NA; ++e) {
          cs[e] = a[2 * e];
          sn[e] = flip ? -a[2 * e + 1] : a[2 * e + 1];
        }
      }
      for (uint32_t o0 = lane * 16; o0 - lane * 16 < end; o0 += 8192) {
        u32x4 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t o = o0 + 1024 * k;
          x[k] = u32x4{0u, 0u, 0u, 0u};
          if (o < end) x[k] = ld16(A.sbase + o);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t o = o0 + 1024 * k;
          u32x4 y = x[k];
          if constexpr (ROT && HALF) {
            const u32x4 partner = lane_xor4<P>(x[k]);  // every lane takes part
            y = rotate_piece_half<ESIZE>(x[k], partner, cs, sn);
          } else if constexpr (ROT) {
            y = rotate_piece_il<ESIZE>(x[k], cs, sn);
          }
          if (o < end) st_stream(A.at(o), y);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      }
    };
    bool rendered = false;
    if constexpr (kQuadPartial) {
      if (!full && in_stripe <= 16 * 16 && (quad_hash || !hashing)) {
        if (rotate) short_stripe(std::true_type{});
        else short_stripe(std::false_type{});
        rendered = true;
      }
    }
    if (rendered) {
    } else if (!full) {
      if (rotate) partial(std::true_type{});
      else partial(std::false_type{});
    } else if constexpr (!kQuadPartial) {
      if (rotate) full_stripe(std::true_type{});
      else full_stripe(std::false_type{});
    }
    if (hashing) {
      const int64_t left = m - sidx * kStripeChunks;
      const int cnt = (int)(left < kStripeChunks ? left : kStripeChunks);
      uint32_t* fold = reinterpret_cast<uint32_t*>(stage_lds[wave]);
      if constexpr (kQuadPartial) {
        if (quad_hash) {
          const uint2 w = quad_hash_stripe(addr.stripe(i, t, sidx), bytes >> 6, sidx, m == 1, lane);
          fold[(lane >> 2) * 8 + (lane & 3)] = w.x;
          fold[(lane >> 2) * 8 + 4 + (lane & 3)] = w.y;
        }
      }
      if (!quad_hash) put_cv(fold, st, lane);
      stripe_nodes<0>(fold, cnt, level, stripes == 1, lane,
                      nodes + (base_v[i] + t * nodes_at(m, level) +
                               ((sidx * kStripeChunks) >> level)) * 32);
      wave_lds_order();                  // the next task's lines go to the same LDS
    }
  }
}

template <int ESIZE, int STYLE, int RB, bool QP = false>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(fused_waves(STYLE, RB)))) void render_hash_kernel(
    const int64_t* __restrict__ table, int64_t stride, int32_t n, const int64_t* __restrict__ plan,
    const int64_t* __restrict__ task_base, const double* __restrict__ angles, int32_t H,
    int32_t d, const uint8_t* __restrict__ select, int32_t level,
    const int64_t* __restrict__ base_v,
    uint8_t* __restrict__ nodes, uint8_t* __restrict__ out) {
  render_hash_body<ESIZE, STYLE, RB>(DenseAddr<QP>{table, stride, out}, n, plan, task_base,
                                     angles, H, d, select, level, base_v, nodes);
}

// The pool is read (fragment pages) and written (the merged cache's fresh
// pages) through the same pointer.
template <int ESIZE, int STYLE, int RB>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(fused_waves(STYLE, RB)))) void paged_hash_render_kernel(
    uint8_t* pool, int64_t P, int32_t b_shift, const int64_t* __restrict__ table,
    const int32_t* __restrict__ blocks, const int32_t* __restrict__ k_table,
    const int32_t* __restrict__ v_table, int32_t n, const int64_t* __restrict__ plan,
    const int64_t* __restrict__ task_base, const double* __restrict__ angles, int32_t H,
    int32_t d, const uint8_t* __restrict__ select, int32_t level,
    const int64_t* __restrict__ base_v,
    uint8_t* __restrict__ nodes) {
  __shared__ uint32_t rows_lds[kWaves * 2 * (1024 / RB) * 64];
  render_hash_body<ESIZE, STYLE, RB>(
      PagedAddr{pool, P, b_shift, table, blocks, k_table, v_table, rows_lds}, n, plan, task_base,
      angles, H, d, select, level, base_v, nodes);
}

// Calls go(IC<RB>) for the row size of the set.
template <class Go>
__host__ inline void dispatch_row(int64_t row_bytes, Go&& go) {
  switch ((int)row_bytes) {
    case 64: return go(IC<64>{});
    case 128: return go(IC<128>{});
    case 256: return go(IC<256>{});
    case 512: return go(IC<512>{});
    default: return go(IC<1024>{});
  }
}

}  // namespace

hipError_t launch_render_hash(const SetDesc& s, const HashLayout& hlay, const RenderLayout& rlay,
                              const int64_t* plan_dev, double base, int32_t style,
                              const uint8_t* select, uint8_t* digests, void* out, uint8_t* ws,
                              hipStream_t stream, bool tables_ready, bool prep_ready,
                              const Copies* ct) {
  uint8_t* hws = ws;
  uint8_t* rws = ws + align_up(hlay.bytes, kWsAlign);
  hipError_t e = hipSuccess;
  if (!tables_ready && (e = launch_hash_prep(s, hlay, hws, stream)) != hipSuccess) return e;
  if (!prep_ready && (e = launch_render_prep(s, rlay, plan_dev, s.n, base, style,
                                             (int32_t)kStripeBlocks, select, rws, stream)) !=
                         hipSuccess)
    return e;
  const uint8_t* hsel = rws + rlay.off_hsel;  // 0: slot delivery whose Id is computed here
  {
    const int64_t* base_tab = reinterpret_cast<const int64_t*>(hws + hlay.off_tables) +
                              (int64_t)hlay.stripe_level * (s.n + 1);
    const int64_t* tasks = reinterpret_cast<const int64_t*>(rws + rlay.off_tiles);
    const double* angles = reinterpret_cast<const double*>(rws + rlay.off_angles);
    // the task count is known on the device only; the tasks of every delivery
    // (hlay.tasks) bound it. A persistent grid of a few workgroups per CU, or
    // fewer when there are fewer tasks, strides over it.
    const int64_t cap = (int64_t)device_cu_count() * kFusedBlocksPerCu;
    const int64_t want = (hlay.tasks + kWaves - 1) / kWaves;
    const dim3 grid((uint32_t)(want < cap ? (want > 0 ? want : 1) : cap));
    ScopedTiming tm(K_RENDER_HASH, stream);
    uint8_t* nodes = hws + hlay.off_buf0;
    uint8_t* o = reinterpret_cast<uint8_t*>(out);
    bool short_tensors = true;
    for (int i = 0; i < s.n && short_tensors; ++i)
      short_tensors = s.T(i) * token_bytes_of(s) < kStripeBlocks * 64;
    auto go = [&](auto rbc) {
      constexpr int RB = decltype(rbc)::value;
      auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, stream, s.table_dev, s.stride, s.n,
                           plan_dev, tasks, angles, s.H, s.d, hsel, hlay.stripe_level, base_tab, nodes, o);
      };
      auto pick = [&](auto qpc) {
        constexpr bool QP = decltype(qpc)::value;
        if (s.esize == 2) {
          if (style == CM_ROPE_HALF) launch(render_hash_kernel<2, CM_ROPE_HALF, RB, QP>);
          else launch(render_hash_kernel<2, CM_ROPE_INTERLEAVED, RB, QP>);
        } else {
          if (style == CM_ROPE_HALF) launch(render_hash_kernel<4, CM_ROPE_HALF, RB, QP>);
          else launch(render_hash_kernel<4, CM_ROPE_INTERLEAVED, RB, QP>);
        }
      };
      // every tensor shorter than one stripe (rows up to 256 bytes): every task
      // is a tensor's only, partial stripe, hashed by quads of lanes
      if constexpr (RB <= 256) {
        if (short_tensors) {
          pick(std::true_type{});
          return;
        }
      }
      pick(std::false_type{});
    };
    dispatch_row(s.row_bytes, go);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_hash_tree(s, hlay, hsel, 0, digests, hws, stream, ct);
}

hipError_t launch_paged_render_hash(const PagedDesc& p, const HashLayout& hlay,
                                    const RenderLayout& rlay, const int64_t* plan_dev, double base,
                                    int32_t style, const uint8_t* select, const int32_t* k_table,
                                    const int32_t* v_table, uint8_t* digests, uint8_t* ws,
                                    hipStream_t stream, bool prep_ready) {
  const SetDesc& s = p.s;
  uint8_t* hws = ws;
  uint8_t* rws = ws + align_up(hlay.bytes, kWsAlign);
  hipError_t e = hipSuccess;
  if (!prep_ready && (e = launch_hash_prep(s, hlay, hws, stream)) != hipSuccess) return e;
  if (!prep_ready && (e = launch_render_prep(s, rlay, plan_dev, s.n, base, style,
                                             (int32_t)kStripeBlocks, select, rws, stream)) !=
                         hipSuccess)
    return e;
  const uint8_t* hsel = rws + rlay.off_hsel;  // 0: slot delivery whose Id is computed here
  {
    const int64_t* base_tab = reinterpret_cast<const int64_t*>(hws + hlay.off_tables) +
                              (int64_t)hlay.stripe_level * (s.n + 1);
    const int64_t* tasks = reinterpret_cast<const int64_t*>(rws + rlay.off_tiles);
    const double* angles = reinterpret_cast<const double*>(rws + rlay.off_angles);
    const int64_t cap = (int64_t)device_cu_count() * kFusedBlocksPerCu;
    const int64_t want = (hlay.tasks + kWaves - 1) / kWaves;
    const dim3 grid((uint32_t)(want < cap ? (want > 0 ? want : 1) : cap));
    ScopedTiming tm(K_PAGED_HASH_RENDER, stream);
    uint8_t* nodes = hws + hlay.off_buf0;
    uint8_t* pool = static_cast<uint8_t*>(p.pool);
    auto go = [&](auto rbc) {
      constexpr int RB = decltype(rbc)::value;
      auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, stream, pool, p.pages, p.b_shift,
                           s.table_dev, p.blocks_dev, k_table, v_table, s.n, plan_dev, tasks,
                           angles, s.H, s.d, hsel, hlay.stripe_level, base_tab, nodes);
      };
      if (s.esize == 2) {
        if (style == CM_ROPE_HALF) launch(paged_hash_render_kernel<2, CM_ROPE_HALF, RB>);
        else launch(paged_hash_render_kernel<2, CM_ROPE_INTERLEAVED, RB>);
      } else {
        if (style == CM_ROPE_HALF) launch(paged_hash_render_kernel<4, CM_ROPE_HALF, RB>);
        else launch(paged_hash_render_kernel<4, CM_ROPE_INTERLEAVED, RB>);
      }
    };
    dispatch_row(s.row_bytes, go);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_hash_tree(s, hlay, hsel, 0, digests, hws, stream);
}

}  // namespace cm
