// Hybrid-mask verify+draft attention (Sec. 4.1) at full fp32 precision.
//
// This is the fp32 path (and the path for bf16 shapes the bf16 matrix-core kernel does not take):
// inputs enter the products as they are (bf16 widened exactly), every product and sum is fp32,
// exponentials are accurate expf, so that an fp32 call stays within 1e-5 of the fp64 definition.
//
// Both contractions run on the fp32 matrix instruction v_mfma_f32_16x16x4_f32, whose rate (64 FLOP
// per clock and SIMD, 154 TFLOP/s measured on a large product) bounds the kernel: 64 tile rows need
// 128 FLOP per cached byte.  One work-group of four waves handles up to 64 tile rows (a tile row is
// one new row of one query head of the KV head's group) of one (sequence, KV head, KV chunk) and
// streams that chunk's keys 32 at a time through LDS, double buffered, the next tile's loads in
// flight (in registers) while a tile is multiplied:
//   S^T = K Q^T   A = K rows from LDS, B = Q held in registers for the whole chunk; a lane owns one
//                 query row (column of S^T, lane & 15) and keys 4 (lane >> 4) + {0..3} of each 16
//   O^T += V^T P^T  the same lane layout: P goes from the S^T registers into the B operand as it is
// Waves: 1, 2 or 4 blocks of 16 tile rows; with one or two the tile's two 16-key blocks are split
// between waves, which merge their (max, sum, O) through LDS at the end.
// The cached prefix needs no mask (every new row sees all of it, Sec. 4.1); only the ragged tail and
// the new-row tiles are masked.  A sequence of one chunk is normalised and stored; the others leave
// split partials (running max, sum, un-normalised output) that the combine kernel merges.
//
// Measured (4 sequences of 512..2048, 8 KV heads, 64 tile rows each, head dim 128, fp32; 1.64 GFLOP, 53 MB):
// 35 us a call, 47 TFLOP/s, against 283 us with scalar products on sixteen-row tiles; 16 such sequences 86 us.
// What is left: with the tile loads taken out 35 us, with the products taken out 21 us -- 408 work-groups of 128
// keys put two on some CUs and one on others, and the split partials (34 KB a work-group) are written and read once.
#include "fd_common.h"

namespace fd {

constexpr int GEN_BLOCK = 256;
constexpr int GEN_ROWS = 64;    // tile rows per work-group
constexpr int GEN_KEYS = 32;    // keys per LDS tile
typedef __attribute__((ext_vector_type(2))) float f32x2;

// Maximum over the four lanes that share lane & 15, by two register swaps instead of two trips through LDS.
__device__ __forceinline__ float quarters_max(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = fmaxf(__builtin_bit_cast(float, (unsigned)a[0]), __builtin_bit_cast(float, (unsigned)a[1]));
  const unsigned w = __builtin_bit_cast(unsigned, v);
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)b[0]), __builtin_bit_cast(float, (unsigned)b[1]));
}

// Where the longest lengths allow more work-groups of one chunk each than the chip holds at once (AttnParams::even_cus, set on the host),
// the device deals out the tiles (32 keys; those of the prefix, then those of the new rows) itself: every sequence is cut into equal
// pieces, at most as many as it has chunks of p.chunk keys, and the pieces are the first work-groups of the launch.
// A compute unit takes its tiles one after the other whether one work-group holds them or two (some 2.9 us a tile of 64 rows), so a call
// takes as long as the compute unit with the most of them: rounds of pieces, times tiles of a piece and the one that its partial weighs.  The
// piece size is the one of four, p.chunk to 7/4 of it, for which that product is least.  (A sequence has as many pieces as its prefix has chunks at most, so
// that new rows that are many against the prefix make its pieces longer than the size: 385 keys and 256 new rows with chunks of 128 keys are
// four pieces of up to six tiles.  The product counts them as the size.)  In a grid over (chunk, head, sequence) the chunks that shorter
// sequences don't have leave some compute units with three work-groups and others with one, and equal lengths end in a round of few.
// us a call, fp32, 8 KV heads, 64 tile rows, head dim 128, chunks / pieces (keys of a chunk of the automatic cut, of a piece at most):
// 3 sequences of 2992..3583 keys 59.2 / 45.7 (128, 160), 9 of 1024 55.1 / 44.9 (128, 160), 5 of 1036..1997 49.9 / 40.8 (128, 128), 5 of 512..4096
// 68.8 / 59.2 (192, 256), 16 of 512..2048 105.3 / 85.8 (320, 416), 16 of 2048 125.5 / 107.5 (320, 576); 8 of 500..2000 at head dim 64 34.9 / 31.4,
// bf16 at head dim 96 49.3 / 41.0 (128, 192); one KV head, 8 of 1000..4000, 512 tile rows 106.5 / 82.1 (320, 416).  6 of 4000 in three rounds instead
// of four 89.2 / 90.0 (192, 256).  Declared for longer sequences than there are: 16 of 60..100 with a bound of 2048 35.0 / 27.6.
// Up to two work-groups per compute unit the grid is kept: they all start at once, and where lengths differ
// little (4 of 1400..2000 keys) finding the pieces costs more than it gives, 35.6 / 36.4.
// Every wave works this out by itself, lane i for sequence i.
struct EvenPieces { SeqInfo s; uint32_t bad; int T, S, items; };           // of this lane: tiles, pieces of an item, items (heads x row tiles)
__device__ __forceinline__ EvenPieces even_pieces(const AttnParams& p) {
  EvenPieces e;
  const int lane = threadIdx.x & 63;
  e.s = SeqInfo{}; e.bad = 0; e.T = e.S = e.items = 0;
  const int c0 = p.chunk / GEN_KEYS;
  int most = 0;
  if (lane < p.B) {
    e.s = load_seq_t<false>(p, lane, &e.bad);
    e.T = (e.s.L + GEN_KEYS - 1) / GEN_KEYS + (e.s.n + GEN_KEYS - 1) / GEN_KEYS;
    e.items = p.Hkv * ((e.s.n * p.G + GEN_ROWS - 1) / GEN_ROWS);
    most = max(1, small_div((e.s.L + GEN_KEYS - 1) / GEN_KEYS + c0 - 1, inverse(c0)));
  }
  const float inv_cus = inverse(p.even_cus);
  int least = 0x7fffffff;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = c0 + (q * c0 + 3) / 4;
    const int S = min(most, small_div(e.T + c - 1, inverse(c)));
    const int cost = small_div(wave_total(e.items * S) + p.even_cus - 1, inv_cus) * (c + 1);
    if (cost < least) { least = cost; e.S = S; }
  }
  return e;
}

int attn_generic_rows_per_wg() { return GEN_ROWS; }

// NDB: head dim in blocks of 16, rounded up to 2, 4, 6 or 8 (the columns beyond D are zero in LDS and in Q).
// Column of the output block g16 (0 .. NDB - 1) that matrix row m stands for: blocks are taken four
// at a time (the rest, two, together), column = 64 (g16 / 4) + W m + g16 % 4 with W the group's
// width, so that a lane's V operands of a group are adjacent in LDS and its outputs adjacent in memory.
template <typename T, int NDB, bool EVEN>
__global__ __launch_bounds__(GEN_BLOCK, 2) void attn_generic_kernel(AttnParams p) {
  constexpr int DP = 16 * NDB;                     // padded head dim
  // LDS row pitch: a multiple of 16 bytes that is odd in units of 16, so that the 16 rows one
  // ds_read_b128 of K touches fall into 16 different slots of the 256-byte bank line
  constexpr int STR = DP + 4;
  constexpr int VEC = 16 / (int)sizeof(T);         // elements per 16-byte load
  constexpr int TPR = DP / VEC;                    // loads per row
  constexpr int NLD = (GEN_KEYS * TPR + GEN_BLOCK - 1) / GEN_BLOCK;
  constexpr int NG = (NDB + 3) / 4;                // column groups
  __shared__ __attribute__((aligned(16))) float lds[2][2][GEN_KEYS * STR];   // [buffer][K, V]

  int chunk_id, nchunks, g, rt, tile0, tile1;      // tiles of the sequence: those of its prefix, then those of its new rows
  SeqInfo s;
  if (EVEN) {
    // pieces are numbered (sequence, row tile, head, piece)
    const EvenPieces e = even_pieces(p);
    const int w = blockIdx.x;
    if (w == 0 && threadIdx.x < 64 && e.bad) flag_status(p.status, e.bad);
    const int hi = wave_incl_scan(e.items * e.S), lo = hi - e.items * e.S;
    const int at = __ffsll((long long)__ballot(lo <= w && w < hi)) - 1;
    if (at < 0) return;
    auto from = [&](int v) { return __builtin_amdgcn_readlane(v, at); };
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    s.L = from(e.s.L); s.row0 = from(e.s.row0); s.n = from(e.s.n); s.k = from(e.s.k);
    s.v = from(e.s.v); s.nb = from(e.s.nb); s.page0 = from(e.s.page0); s.npages = from(e.s.npages);
    const int tiles = from(e.T);
    nchunks = from(e.S);
    const float inv = inverse(nchunks);
    const int local = w - from(lo), unit = uniform(small_div(local, inv));
    chunk_id = uniform(local - unit * nchunks);
    rt = uniform((int)((unsigned)unit / (unsigned)p.Hkv));
    g = uniform(unit - rt * p.Hkv);
    const int a = small_div(tiles, inv), b = tiles - a * nchunks;         // (j T / S, with T = a S + b)
    tile0 = uniform(chunk_id * a + small_div(chunk_id * b, inv));
    tile1 = uniform((chunk_id + 1) * a + small_div((chunk_id + 1) * b, inv));
  } else {
    // Consecutive work-group ids go to different XCDs; rotating the chunk index by head and
    // sequence keeps any one XCD from collecting only the long (or only the short) chunks.
    chunk_id = (blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x;
    g = blockIdx.y % p.Hkv; rt = blockIdx.y / p.Hkv;
    s = load_seq(p, blockIdx.z);
    nchunks = max(1, (s.L + p.chunk - 1) / p.chunk);
    if (chunk_id >= nchunks) return;
    tile0 = chunk_id * (p.chunk / GEN_KEYS);
    tile1 = chunk_id == nchunks - 1 ? (s.L + GEN_KEYS - 1) / GEN_KEYS + (s.n + GEN_KEYS - 1) / GEN_KEYS : tile0 + p.chunk / GEN_KEYS;
  }
  const int rows_total = s.n * p.G;
  if (rt * GEN_ROWS >= rows_total) return;
  const int D = p.D, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, kq = lane >> 4;
  const T* Kc = reinterpret_cast<const T*>(p.k_cache) + (long long)g * p.sh;
  const T* Vc = reinterpret_cast<const T*>(p.v_cache) + (long long)g * p.sh;
  const T* Kn = reinterpret_cast<const T*>(p.k_new) + (long long)g * D;
  const T* Vn = reinterpret_cast<const T*>(p.v_new) + (long long)g * D;

  const int rows_here = min(GEN_ROWS, rows_total - rt * GEN_ROWS);
  // Row blocks and key split: a wave takes sixteen rows; with one or two blocks two waves share each, so that
  // small calls (up to 32 tile rows: bound by the stream, not by the products) still use the tile's halves side by side.
  const int RB = rows_here <= 16 ? 1 : (rows_here <= 32 ? 2 : 4);      // row blocks
  const int KS = RB == 4 ? 1 : 2;                                      // waves that share a row block
  const int rb = wave % RB, ks = wave / RB;
  const bool wave_works = ks < KS && rb * 16 < rows_here;
  const int my_T = rt * GEN_ROWS + rb * 16 + l15;                      // this lane's tile row
  const bool row_valid = wave_works && my_T < rows_total;
  const int my_nn = my_T / p.G, my_hq = g * p.G + my_T % p.G;
  const RowWindow win = row_window(row_valid ? my_nn : 0, s);

  const int prefix_tiles = (s.L + GEN_KEYS - 1) / GEN_KEYS;
  const int c0 = tile0 * GEN_KEYS, c1 = min(s.L, tile1 * GEN_KEYS);
  const int nt = tile1 - tile0, cached_tiles = max(0, min(prefix_tiles, tile1) - tile0);
  const int new0 = EVEN ? max(0, tile0 - prefix_tiles) * GEN_KEYS : 0;            // first new key of this work-group's new tiles (chunks: the last has them all)

  // key / page_size by a multiplication (AttnParams::page_magic): exact for keys below 2^31
  auto page_of = [&](int key) {
    return p.page_size == 1 ? key : (int)(__umulhi((unsigned)key, p.page_magic) >> p.page_magic_shift);
  };

  // ---- tile loads: thread tid takes 16-byte vectors tid + 256 i of the tile's K and V -------------
  // No load is conditional: rows past the end read the last row, columns past D the first ones, and both enter LDS as zeros.
  // (The scores of such rows are masked and Q is zero in such columns, but zero times an infinity would not be zero.)
  constexpr bool EXACT = GEN_KEYS * TPR % GEN_BLOCK == 0;
  int ld_row[NLD], ld_col[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int idx = EXACT ? tid + GEN_BLOCK * i : min(tid + GEN_BLOCK * i, GEN_KEYS * TPR - 1);
    ld_row[i] = idx / TPR; ld_col[i] = (idx % TPR) * VEC;
  }
  int pid[NLD], slot_[NLD];                        // pages and slots of this thread's rows of the next tile to load
  u32x4 rk[NLD], rv[NLD];
  auto fetch_pages = [&](int t) {
    if (t >= cached_tiles) return;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int key = min(c0 + t * GEN_KEYS + ld_row[i], c1 - 1);
      const int lp = page_of(key);
      pid[i] = p.page_indices[s.page0 + lp];
      slot_[i] = key - lp * p.page_size;
    }
  };
  auto load_tile = [&](int t) {
    if (t >= cached_tiles) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int key = min(new0 + (t - cached_tiles) * GEN_KEYS + ld_row[i], s.n - 1);
        const long long off = (long long)(s.row0 + key) * p.Hkv * D + (ld_col[i] < D ? ld_col[i] : 0);
        rk[i] = *reinterpret_cast<const u32x4*>(Kn + off); rv[i] = *reinterpret_cast<const u32x4*>(Vn + off);
      }
    } else {
      bool oob = false;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const bool bad = (unsigned)pid[i] >= (unsigned)p.num_pages;
        oob |= bad;
        const unsigned long long off = (unsigned)(bad ? 0 : pid[i]) * (unsigned long long)p.sp +
                                       (unsigned long long)(unsigned)slot_[i] * (unsigned)p.st + (unsigned)(ld_col[i] < D ? ld_col[i] : 0);
        rk[i] = *reinterpret_cast<const u32x4*>(Kc + off); rv[i] = *reinterpret_cast<const u32x4*>(Vc + off);
      }
      if (oob) flag_status(p.status, FD_DEV_PAGE_RANGE);
    }
  };
  auto put = [&](float* dst, u32x4 w) {            // one vector, widened to fp32
    if (sizeof(T) == 4) {
      *reinterpret_cast<u32x4*>(dst) = w;
    } else {
      const u32x4 a = {w[0] << 16, w[0] & 0xffff0000u, w[1] << 16, w[1] & 0xffff0000u};
      const u32x4 b = {w[2] << 16, w[2] & 0xffff0000u, w[3] << 16, w[3] & 0xffff0000u};
      *reinterpret_cast<u32x4*>(dst) = a; *reinterpret_cast<u32x4*>(dst + 4) = b;
    }
  };
  auto store_tile = [&](int t, int buf) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      put(&lds[buf][0][ld_row[i] * STR + ld_col[i]], rk[i]);
      put(&lds[buf][1][ld_row[i] * STR + ld_col[i]], rv[i]);
    }
    const int rows = t >= cached_tiles ? s.n - new0 - (t - cached_tiles) * GEN_KEYS : c1 - c0 - t * GEN_KEYS;     // that exist
    if (rows < GEN_KEYS || D < DP) {               // (over what was just written: selecting the values before costs every tile 3 %)
      const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        if (ld_row[i] >= rows || ld_col[i] >= D) {
          put(&lds[buf][0][ld_row[i] * STR + ld_col[i]], zero);
          put(&lds[buf][1][ld_row[i] * STR + ld_col[i]], zero);
        }
    }
  };

  fetch_pages(0);
  // query row of this lane: columns 16 j + 4 kq + {0..3}
  f32x4 q[NDB];
  {
    const T* qp = reinterpret_cast<const T*>(p.q) + ((long long)(s.row0 + my_nn) * p.Hq + my_hq) * D;
#pragma unroll
    for (int j = 0; j < NDB; ++j) {
      const int col = 16 * j + 4 * kq;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
      if (row_valid && col < D) {                  // D is a multiple of 8: a vector is inside or outside
        if (sizeof(T) == 4) x = *reinterpret_cast<const f32x4*>(qp + col);
        else {
          const u32x2 w = *reinterpret_cast<const u32x2*>(qp + col);
          x[0] = __uint_as_float(w[0] << 16); x[1] = __uint_as_float(w[0] & 0xffff0000u);
          x[2] = __uint_as_float(w[1] << 16); x[3] = __uint_as_float(w[1] & 0xffff0000u);
        }
      }
      q[j] = x;
    }
  }
  load_tile(0);
  fetch_pages(1);
  store_tile(0, 0);
  __syncthreads();

  float m_run = -INFINITY, l_lane = 0.f;
  f32x4 o[NDB];
#pragma unroll
  for (int b = 0; b < NDB; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A piece may be longer than a chunk, and the rounding of a sum over keys grows with the number of keys that go through one accumulator: a
  // piece is summed in parts of a chunk each, and a part that has ended waits in registers of its own.
  // 2-norm error against 64 bits over that of chunks (mean of eight calls), pieces summed in one go / in parts: 16 sequences of 2048 keys
  // at head dim 128 1.10 / 0.86, 16 of 512..2048 at head dim 32 1.08 / 0.93, one KV head with 512 tile rows at head dim 64 1.08 / 0.88,
  // 12 of 300..1200 at head dim 8 1.10 / 0.96.  us a call: 16 of 512..2048 85.3 / 85.6, 6 of 4000 88.2 / 89.5, the others within 1 %.
  const int part_tiles = p.chunk / GEN_KEYS;
  int part_end = part_tiles;
  float m_done = -INFINITY, l_done = 0.f;
  f32x4 o_done[EVEN ? NDB : 1];
  if (EVEN) {
#pragma unroll
    for (int b = 0; b < NDB; ++b) o_done[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto end_part = [&]() {                          // what is done, and the part in o and l_lane, at the reference m_run
    const float r = expf(m_done - (m_run == -INFINITY ? 0.f : m_run));               // (m_done = -inf: 0)
    l_done = l_done * r + l_lane;
#pragma unroll
    for (int b = 0; b < NDB; ++b) o_done[EVEN ? b : 0] = o_done[EVEN ? b : 0] * r + o[b];
    m_done = m_run;
  };

  for (int t = 0; t < nt; ++t) {
    if (t + 1 < nt) { load_tile(t + 1); fetch_pages(t + 2); }
    const bool is_new = t >= cached_tiles;
    const int base = is_new ? new0 + (t - cached_tiles) * GEN_KEYS : c0 + t * GEN_KEYS;
    const int end = is_new ? s.n : c1;                                  // keys at or beyond are invisible
    const bool masked = is_new || base + GEN_KEYS > end;
    const float* Ks = lds[t & 1][0];
    const float* Vs = lds[t & 1][1];
    auto block = [&](auto nkb_c, int kb0) {        // NKB 16-key blocks from kb0 on
      constexpr int NKB = decltype(nkb_c)::value;
      // K fragments are requested one 16-column step ahead of the matrix instructions that take them
      // accumulation chains per key block; four with pieces, where time is equal and the error smaller (9 sequences of 1024 keys, 64 tile
      // rows, head dim 128: chunks with two chains 3.27e-7, pieces with four 2.71e-7)
      constexpr int CHAINS = EVEN ? 4 : 2;
      f32x4 sc[NKB][CHAINS];
#pragma unroll
      for (int b = 0; b < NKB; ++b)
#pragma unroll
        for (int e = 0; e < CHAINS; ++e) sc[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* kp = Ks + (16 * kb0 + l15) * STR + 4 * kq;
      f32x4 kf[2][NKB];
#pragma unroll
      for (int b = 0; b < NKB; ++b) kf[0][b] = *reinterpret_cast<const f32x4*>(kp + 16 * b * STR);
#pragma unroll
      for (int j = 0; j < NDB; ++j) {
        if (j + 1 < NDB) {
#pragma unroll
          for (int b = 0; b < NKB; ++b) kf[(j + 1) & 1][b] = *reinterpret_cast<const f32x4*>(kp + 16 * b * STR + 16 * (j + 1));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int b = 0; b < NKB; ++b)
            sc[b][e % CHAINS] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j & 1][b][e], q[j][e], sc[b][e % CHAINS], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      // V fragments likewise, one key step (8 matrix instructions at head dim 128) ahead; the first before the softmax
      const float* vp = Vs + (16 * kb0 + 4 * kq) * STR;
      f32x4 vf[2][NG];
      auto vread = [&](int st) {                   // key step st = 4 b + e
#pragma unroll
        for (int gr = 0; gr < NG; ++gr) {
          const float* a = vp + (16 * (st >> 2) + (st & 3)) * STR + 64 * gr;
          if (NDB % 4 && gr == NG - 1) {
            const f32x2 w = *reinterpret_cast<const f32x2*>(a + 2 * l15);
            vf[st & 1][gr][0] = w[0]; vf[st & 1][gr][1] = w[1];
          } else {
            vf[st & 1][gr] = *reinterpret_cast<const f32x4*>(a + 4 * l15);
          }
        }
      };
      vread(0);
      float x[NKB][4];
#pragma unroll
      for (int b = 0; b < NKB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float sum = sc[b][0][i] + sc[b][1][i];
          if (CHAINS == 4) sum += sc[b][CHAINS - 2][i] + sc[b][CHAINS - 1][i];
          x[b][i] = sum * p.sm_scale;
        }
      if (masked) {
        RowWindow wv = win;
        if (!is_new) { wv.vr = end; wv.lo = 0; wv.hi = 0; }             // a prefix tile: the keys below the end
#pragma unroll
        for (int b = 0; b < NKB; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = base + 16 * (kb0 + b) + 4 * kq + i;
            x[b][i] = (new_key_visible(wv, key) & (key < end)) ? x[b][i] : -INFINITY;
          }
      }
      float mx = x[0][0];
#pragma unroll
      for (int b = 0; b < NKB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, x[b][i]);
      mx = quarters_max(mx);
      const float m_new = fmaxf(m_run, mx);
      const float m_sub = m_new == -INFINITY ? 0.f : m_new;             // row with nothing visible yet
      if (__any(m_new != m_run)) {
        const float alpha = expf(m_run - m_sub);                        // expf(-inf) = 0 on the first visible key
        l_lane *= alpha;
#pragma unroll
        for (int b = 0; b < NDB; ++b) o[b] *= alpha;
      }
      m_run = m_new;
#pragma unroll
      for (int b = 0; b < NKB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[b][i] = expf(x[b][i] - m_sub); l_lane += x[b][i]; }
#pragma unroll
      for (int st = 0; st < 4 * NKB; ++st) {
        if (st + 1 < 4 * NKB) vread(st + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NDB; ++c)
          o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[st & 1][c >> 2][c & 3], x[st >> 2][st & 3], o[c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (wave_works) {
      if (KS == 1) block(std::integral_constant<int, 2>{}, 0);
      else if (base + 16 * ks < end) block(std::integral_constant<int, 1>{}, ks);
    }
    if (EVEN && t + 1 == part_end && t + 1 < nt) {
      end_part();
      l_lane = 0.f;
#pragma unroll
      for (int b = 0; b < NDB; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
      part_end += part_tiles;
    }
    if (t + 1 < nt) store_tile(t + 1, (t + 1) & 1);
    __syncthreads();                               // tile t consumed, tile t + 1 visible
  }
  if (EVEN && nt > part_tiles) {
    end_part();
    l_lane = l_done;
#pragma unroll
    for (int b = 0; b < NDB; ++b) o[b] = o_done[EVEN ? b : 0];
  }

  // ---- merge the two waves of a row block (same register layout) through LDS --------------------
  if (KS == 2) {
    f32x4* xch = reinterpret_cast<f32x4*>(&lds[0][0][0]);              // [rb][NDB + 1][64]
    static_assert(sizeof(lds) >= 2 * (NDB + 1) * 64 * sizeof(f32x4), "the merge area fits the tile buffers");
    if (wave_works && ks == 1) {
#pragma unroll
      for (int b = 0; b < NDB; ++b) xch[(rb * (NDB + 1) + b) * 64 + lane] = o[b];
      xch[(rb * (NDB + 1) + NDB) * 64 + lane] = f32x4{m_run, l_lane, 0.f, 0.f};
    }
    __syncthreads();
    if (wave_works && ks == 0) {
      const f32x4 ml = xch[(rb * (NDB + 1) + NDB) * 64 + lane];
      const float m_new = fmaxf(m_run, ml[0]);
      const float m_sub = m_new == -INFINITY ? 0.f : m_new;
      const float a = expf(m_run - m_sub), b2 = expf(ml[0] - m_sub);
      l_lane = l_lane * a + ml[1] * b2;
      m_run = m_new;
#pragma unroll
      for (int b = 0; b < NDB; ++b) o[b] = o[b] * a + xch[(rb * (NDB + 1) + b) * 64 + lane] * b2;
    }
  }
  if (!wave_works || ks > 0) return;
  float l_run = l_lane + __shfl_xor(l_lane, 16);
  l_run += __shfl_xor(l_run, 32);
  if (!row_valid) return;

  // o[4 gr + c][i]: column 64 gr + W (4 kq + i) + c, i.e. 4 W adjacent columns per lane and group
  const long long orow = (long long)(s.row0 + my_nn) * p.Hq + my_hq;
  if (nchunks == 1) {
    const float inv = l_run > 0.f ? 1.0f / l_run : 0.f;
    T* op = reinterpret_cast<T*>(p.out) + orow * D;
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      constexpr int W_LAST = NDB % 4 ? NDB % 4 : 4;
      const int W = gr == NG - 1 ? W_LAST : 4;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < W; ++c) {
          const int d = 64 * gr + W * (4 * kq + i) + c;
          if (d < D) Elem<T>::store(op + d, l_run > 0.f ? o[4 * gr + c][i] * inv : 0.f);        // (as the combine kernel does)
        }
    }
    if (p.lse && kq == 0) p.lse[orow] = m_run + logf(l_run);
  } else {
    const long long slot = ((long long)chunk_id * p.total_rows + (s.row0 + my_nn)) * p.Hq + my_hq;
    float* ap = p.part_acc + slot * D;
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      constexpr int W_LAST = NDB % 4 ? NDB % 4 : 4;
      const int W = gr == NG - 1 ? W_LAST : 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = 64 * gr + W * (4 * kq + i);
        if (W == 4) { if (d < D) *reinterpret_cast<f32x4*>(ap + d) = f32x4{o[4 * gr][i], o[4 * gr + 1][i], o[4 * gr + 2][i], o[4 * gr + 3][i]}; }
        else {
#pragma unroll
          for (int c = 0; c < W; ++c) if (d + c < D) ap[d + c] = o[4 * gr + c][i];
        }
      }
    }
    if (kq == 0) { p.part_ml[slot * 2] = m_run; p.part_ml[slot * 2 + 1] = l_run; }
  }
}

// ---------------------------------------------------------------------------------------
// Combine the per-chunk partials of every (row, head) of the sequences of more than one chunk:
//   M = max_c m_c;  out = sum_c e^{m_c - M} acc_c / sum_c e^{m_c - M} l_c;  lse = M + log(sum)
// 32 lanes per (row, head), a lane owns four columns; grid (ceil(Hq / 8), max_new_rows, B).  The
// chunks are taken four at a time, their loads issued together, with a running maximum.
// ---------------------------------------------------------------------------------------
template <typename T, bool EVEN>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnParams p) {
  const int seq = blockIdx.z, nn = blockIdx.y;
  const SeqInfo s = load_seq(p, seq);
  // one chunk, and so one piece: the streaming kernel stored the rows itself.  (Before the pieces are counted: a call declared for longer
  // sequences than it has, 2 of 64..100 keys with a bound of 8192, 23.0 -> 22.2 us, 16 of 60..100 with 2048 28.7 -> 27.6.)
  if (nn >= s.n || s.L <= p.chunk) return;
  int nchunks = (s.L + p.chunk - 1) / p.chunk;
  if (EVEN) nchunks = __builtin_amdgcn_readlane(even_pieces(p).S, seq);
  if (nchunks <= 1) return;
  const int hq = blockIdx.x * 8 + (threadIdx.x >> 5), d = (threadIdx.x & 31) * 4;
  if (hq >= p.Hq || d >= p.D) return;
  const long long row = s.row0 + nn;
  const long long stride = (long long)p.total_rows * p.Hq;     // partial slots per chunk
  const long long slot0 = row * p.Hq + hq;
  float M = -INFINITY, den = 0.f;
  f32x4 num = {0.f, 0.f, 0.f, 0.f};
  constexpr int NB = 4;
  for (int ch0 = 0; ch0 < nchunks; ch0 += NB) {
    f32x2 ml[NB]; f32x4 a[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const long long sl = slot0 + min(ch0 + u, nchunks - 1) * stride;
      ml[u] = *reinterpret_cast<const f32x2*>(p.part_ml + sl * 2);
      a[u] = *reinterpret_cast<const f32x4*>(p.part_acc + sl * p.D + d);
      if (ch0 + u >= nchunks) ml[u][0] = -INFINITY;
    }
    float Mb = M;
#pragma unroll
    for (int u = 0; u < NB; ++u) Mb = fmaxf(Mb, ml[u][0]);
    const float Ms = Mb == -INFINITY ? 0.f : Mb;   // (no branch on it: the loads of the sums would move behind it)
    const float r = expf(M - Ms);                  // M = -inf: 0
    num *= r; den *= r; M = Mb;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const float w = expf(ml[u][0] - Ms);
      const bool none = ml[u][0] == -INFINITY;     // surplus, or a chunk in which no key has any weight: adds nothing, whatever its sums hold
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(w, none ? 0.f : a[u][e], num[e]);
      den = fmaf(w, none ? 0.f : ml[u][1], den);
    }
  }
  T* op = reinterpret_cast<T*>(p.out) + slot0 * p.D + d;
#pragma unroll
  for (int e = 0; e < 4; ++e) Elem<T>::store(op + e, den > 0.f ? num[e] / den : 0.f);
  if (p.lse && d == 0) p.lse[slot0] = M + logf(den);
}

template <typename T, bool EVEN>
static void launch_generic(const AttnParams& p, hipStream_t st) {
  const dim3 grid = EVEN ? dim3(p.B * p.Hkv * p.row_tiles * p.max_chunks) : dim3(p.max_chunks, p.Hkv * p.row_tiles, p.B);
  if (p.D <= 32) hipLaunchKernelGGL((attn_generic_kernel<T, 2, EVEN>), grid, dim3(GEN_BLOCK), 0, st, p);
  else if (p.D <= 64) hipLaunchKernelGGL((attn_generic_kernel<T, 4, EVEN>), grid, dim3(GEN_BLOCK), 0, st, p);
  else if (p.D <= 96) hipLaunchKernelGGL((attn_generic_kernel<T, 6, EVEN>), grid, dim3(GEN_BLOCK), 0, st, p);
  else hipLaunchKernelGGL((attn_generic_kernel<T, 8, EVEN>), grid, dim3(GEN_BLOCK), 0, st, p);
}

hipError_t run_attn_generic(const AttnParams& p, int dtype, hipStream_t st) {
  if (dtype == FD_BF16) p.even_cus > 0 ? launch_generic<bf16_t, true>(p, st) : launch_generic<bf16_t, false>(p, st);
  else p.even_cus > 0 ? launch_generic<float, true>(p, st) : launch_generic<float, false>(p, st);
  return hipGetLastError();
}

template <typename T>
static void launch_generic_combine(const AttnParams& p, hipStream_t st) {
  const dim3 grid((p.Hq + 7) / 8, p.max_new_rows, p.B);
  if (p.even_cus > 0) hipLaunchKernelGGL((attn_combine_kernel<T, true>), grid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL((attn_combine_kernel<T, false>), grid, dim3(256), 0, st, p);
}

hipError_t run_attn_combine(const AttnParams& p, int dtype, hipStream_t st) {
  if (dtype == FD_BF16) launch_generic_combine<bf16_t>(p, st);
  else launch_generic_combine<float>(p, st);
  return hipGetLastError();
}

}  // namespace fd
