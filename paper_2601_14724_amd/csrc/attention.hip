// Chunk attention for gfx950 (MFMA bf16, 64-wide waves).
//
// attn_fwd     causal GQA attention of the chunk (or query) rows over
//              [cache; new rows]: O and the per-row log-sum-exp.
// attn_colsum  attention mass W_i = sum over heads and rows of the softmax
//              probability on candidate i (Sec. 3.1, deep-layer score),
//              recomputed key-major from the row LSE so that every W_i's
//              share of a KV head (or of a range of its rows) is summed by
//              exactly one wave, in a fixed order; mass_reduce adds the shares.
//
// Query rows are packed per KV head: packed row p = r * G + g holds chunk row
// r of query head kv * G + g, so the G heads that share a KV head share every
// K/V tile, and all rows of a tile share nearly the same causal boundary.
//
// MFMA layout (v_mfma_f32_32x32x16_bf16): lane l supplies A[m = l%32][k = 8(l/32)
// .. +7] and B[k = 8(l/32) .. +7][n = l%32]; result register j of lane l holds
// D[m = 8(j/4) + 4(l/32) + j%4][n = l%32].
#include <type_traits>

#include "hermes_internal.h"
#include "score_terms.h"

namespace hermes {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s4 __attribute__((ext_vector_type(4)));

constexpr int AT = 512;                  // attention workgroup: 8 waves, two per SIMD
constexpr int BM = kAttnRowsPerBlock;    // packed rows per workgroup with one key group (8 waves x 32)
constexpr int BK = kColsumKeysPerBlock;  // candidates per sweep workgroup (4 waves x 64)
constexpr int BQS = 32;                  // packed rows per sweep tile
constexpr int KPAD = 8;                  // u16 padding of K / Q rows in LDS
constexpr int VPAD = 32;                 // u16 padding of V rows in LDS
constexpr int kAheadK = 4;               // K fragment reads issued ahead of their MFMA
// fourth word of a raw buffer descriptor on gfx9-family chips (32-bit data,
// no swizzle; the range check uses the byte count in the third word)
constexpr int kBufferWord3 = 0x00020000;
constexpr int kAheadV = 4;               // V^T fragment pairs issued ahead of their MFMA

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t f2bf(float x) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }


// 16-byte load through the global (not flat) address space, so outstanding
// prefetches are tracked by vmcnt only and never delay LDS waits.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 gload16(const uint16_t *p) {
  typedef const __attribute__((address_space(1))) u32x4 *gptr;
  const u32x4 v = *(gptr)(p);
  return uint4{v.x, v.y, v.z, v.w};
}

// ds_read_b64_tr_b16: inside each group of 16 lanes, lane j receives element
// j%4 of the 8-byte rows addressed by lanes j/4, 4 + j/4, 8 + j/4, 12 + j/4.
__device__ __forceinline__ s4 lds_tr16(const uint16_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4 *)p);
}

// Workgroups are dispatched to the 8 XCDs round-robin by linear id; this
// maps linear ids so that consecutive logical tiles (the q-tiles of one
// layer and KV head, which stream the same K/V) run on the same XCD and
// share its L2.
__device__ __forceinline__ int xcd_remap(int i, int n) {
  const int q = n / 8, r = n % 8, x = i % 8, k = i / 8;
  return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

constexpr int kCopyAhead = 4;   // pieces of K and of V a thread has in flight

// Appends: this workgroup's share (the id-th of n) of the copy of the new K/V
// rows and positions into the caches.  Nothing in the launch reads those rows
// of the caches, so the copy rides with it: a launch of its own took 4-5 us a
// layer, 20 us over 28 layers of 784 rows.  It comes last in the kernel, where
// a pass that copies nothing does not wait for the test (in front it cost a
// query 0.5 us).
// A launch of several rounds leaves it to the first round's workgroups (by
// dispatch order: one a CU), so that the others do not each wait for a load.
// 28 layers of 32768 + 3136 rows, 38 rounds: the step 1.1% slower than with the
// copy as a launch of its own when every workgroup copied, 0.1% faster now.
__device__ __forceinline__ void copy_share(const AttnArgs &a, int D, int id, int n) {
  if (id >= n) return;
  const int entries = a.st_entries, threads = blockDim.x;
  const int per = a.C * (a.Hkv * D / 8);    // 16-byte pieces of an entry's K (or V)
  // every entry has its own workgroups, or a workgroup has several entries
  const int first = n < entries ? id : id % entries, step = min(n, entries);
  const int share = n < entries ? 0 : id / entries;
  const int shares = n < entries ? 1 : (n - first + entries - 1) / entries;
  for (int j = first; j < entries; j += step) {
    const AttnEntry &en = a.e[j];
    const LayerTable &L = a.tab[en.layer];
    const int cur = en.cur, T0 = en.T0;
    const uint16_t *kn = a.kn + en.slot * a.kv_lstride, *vn = a.vn + en.slot * a.kv_lstride;
    uint16_t *kd = en.k + (int64_t)T0 * a.Hkv * D, *vd = en.v + (int64_t)T0 * a.Hkv * D;
    const int stride = shares * threads;
    for (int x0 = share * threads + threadIdx.x; x0 < per; x0 += kCopyAhead * stride) {
      uint4 kx[kCopyAhead], vx[kCopyAhead];
#pragma unroll
      for (int u = 0; u < kCopyAhead; ++u) {
        const int x = x0 + u * stride;
        if (x < per) {
          kx[u] = gload16(kn + 8 * (int64_t)x);
          vx[u] = gload16(vn + 8 * (int64_t)x);
        }
      }
#pragma unroll
      for (int u = 0; u < kCopyAhead; ++u) {
        const int x = x0 + u * stride;
        if (x < per) {
          *reinterpret_cast<uint4 *>(kd + 8 * (int64_t)x) = kx[u];
          *reinterpret_cast<uint4 *>(vd + 8 * (int64_t)x) = vx[u];
        }
        if (x < a.C) {   // (an entry has more pieces than rows)
          L.pos[cur][T0 + x] = a.pos[x];
          if (L.rpos[cur] != nullptr) L.rpos[cur][T0 + x] = a.rope_pos != nullptr ? a.rope_pos[x] : a.pos[x];
          if (L.rpos_h[cur] != nullptr) {   // M-RoPE: h and w beside t
            L.rpos_h[cur][T0 + x] = a.rope_h[x];
            L.rpos_w[cur][T0 + x] = a.rope_w[x];
          }
        }
      }
    }
  }
}

// STREAM: passes whose (entry, KV head, query tile) workgroups would not fill
// the CUs (one layer's chunk, queries, guidance prompts).  The key tiles of
// every (entry, KV head) pair, concatenated in pair order (pair k = j Hkv +
// kv, e[j].st_tiles tiles each, entry j's pairs from tile e[j].st_off), are cut
// into st_units equal ranges; unit u is nqt workgroups with consecutive ids
// (one per query tile, sharing the K/V tiles in their XCD's L2) over tiles
// [u N / U, (u + 1) N / U).  The workgroup walks its range pair by pair;
// where the range leaves a pair it writes the pair's unnormalised partial
// state (fp32 O, running maximum and row sum) to partial block (u + k)
// of its query tile (distinct for every (u, k): a later unit only covers
// later pairs) and switches to the next pair.  attn_combine merges a pair's
// blocks.  Otherwise: one workgroup per (entry, KV head, query tile) over its
// whole sequence, writing O (WRITE_O) and the row LSE.
//
// KG key groups: the workgroup's NW waves are KG groups of RG = NW / KG waves;
// a group holds all of the workgroup's 32 RG packed rows and takes every KG-th
// key tile, and the groups' states are merged through LDS at the end.  Rows a
// workgroup shrink by KG, so a launch has KG times the workgroups and each
// walks a KG-th of the keys: what a launch of few rows needs to fill the CUs,
// for KG times the K/V staging per row.
//
// SPLIT: each pair's steps are cut into e[j].st_tiles ranges of st_units steps
// (entry j's from e[j].st_off), each nqt workgroups with consecutive ids, one for
// each query tile.  Each writes its partial state as in stream mode.  A pass of
// a few rows then fills the CUs with less partial state than stream mode's
// 256-row workgroups write.  Where the packed rows fit one workgroup (a few
// tokens: decoding) no two workgroups share a key, so the pass is bound by HBM,
// and by latency where a CU has little to read: it takes workgroups of four
// waves, two a CU, so that one's start and end hide behind the other's loads.
enum { PLAIN = 0, STREAMED = 1, SPLIT = 2 };
// (WRITE_O false: at head size 64, and with four key groups, 128 registers are
// enough without spilling and two workgroups fit a CU)
template <int D, int NW, int KG, int MODE, bool WRITE_O>
__global__ __launch_bounds__(64 * NW, NW != 8 ? 2 : !WRITE_O && (D == 64 || KG == 4) ? 4 : 1)
void attn_fwd(AttnArgs a, int nqt) {
  constexpr bool STREAM = MODE == STREAMED;
  constexpr int RG = NW / KG;               // 32-row groups (waves of a key group)
  constexpr int BM = 32 * RG;               // packed rows of the workgroup
  constexpr int BN = KG <= NW / 4 ? 64 : 32;   // keys per tile
  constexpr int SUB = BN / 32;
  constexpr int NBUF = RG == 1 ? 1 : 2;     // (a tile of one wave needs no second buffer)
  constexpr int GT = 64 * RG;               // threads of a key group
  constexpr bool ONE_TILE = MODE == SPLIT && NW == 4;   // (nqt is 1, no K/V tile is shared)
  const int lin = ONE_TILE ? (int)blockIdx.x : xcd_remap(blockIdx.x, gridDim.x);
  const int qtile = lin % nqt;
  const int unit = ONE_TILE ? lin : lin / nqt;
  const int C = a.C, Hq = a.Hq, Hkv = a.Hkv;
  const int G = Hq / Hkv;
  const int P = C * G;
  const int p0 = qtile * BM;
  if (p0 >= P) return;
  const int tid = threadIdx.x % GT, wave = tid >> 6, lane = tid & 63;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / GT);
  const int half = lane >> 5, l32 = lane & 31;

  // This lane's query row (column n of the S^T tile).
  const int prow = p0 + wave * 32 + l32;
  const bool row_ok = prow < P;
  // A wave whose 32 rows all lie past P (in the last query tile of a head
  // group) still loads and stores its share of every tile and meets every
  // barrier, but issues no MFMAs.
  const bool wave_rows = __builtin_amdgcn_readfirstlane(p0 + wave * 32 < P ? 1 : 0) != 0;
  const int r = row_ok ? prow / G : 0;
  const int g = row_ok ? prow - r * G : 0;
  const int pmax = min(p0 + BM, P) - 1;

  // Pair state: entry j, KV head kv, its cache and new rows.  A key tile is BN
  // consecutive rows of [cache; new rows]; the one that holds the cache's end may
  // have rows of both.
  int j = 0, kv = 0, T0 = 0, ntiles = 0, n_pure = 0, first = 0;
  const uint16_t *q = nullptr, *kn = nullptr, *vn = nullptr, *kc = nullptr, *vc = nullptr;
  const int64_t row_stride = (int64_t)Hkv * D;
  constexpr int CH = D / 8;                 // 16-byte chunks per key row and head
  constexpr int NLD = BN * CH / GT;         // chunks per thread per tensor
  static_assert(GT % CH == 0, "a thread's chunks lie in one column");
  uint32_t cofs = 0;
  const int cstep = (int)(GT / CH * row_stride * sizeof(uint16_t));
  bf16x8 qf[D / 16];
  // STREAM: this unit's tile range over the concatenated pairs
  int x_lo = 0, x_hi = 0, u = 0;
  if constexpr (STREAM) {
    u = unit;
    // (the 64-bit divisions run on vector registers: back to scalar ones, so
    // that tile indices, loop bounds and buffer descriptors stay scalar)
    x_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)u * a.st_total / a.st_units));
    x_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)(u + 1) * a.st_total / a.st_units));
  }
  auto enter = [&](int jj, int kvv) {
    j = jj;
    kv = kvv;
    const AttnEntry &en = a.e[j];
    T0 = en.T0;
    n_pure = T0 / BN;                       // tiles wholly in the cache: no mask, one source
    ntiles = (T0 + pmax / G) / BN + 1;      // the last one a row of the block sees
    const int slot = en.slot;
    q = a.q + slot * a.q_lstride;
    kn = a.kn + slot * a.kv_lstride;
    vn = a.vn + slot * a.kv_lstride;
    kc = en.k;
    vc = en.v;
    const int h = kv * G + g;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      qf[kk] = row_ok ? *reinterpret_cast<const bf16x8 *>(q + ((int64_t)r * Hq + h) * D + 16 * kk + 8 * half)
                      : bf16x8{};
    }
    // byte offset of this thread's first chunk inside a key tile; the others
    // follow GT / CH rows apart
    cofs = (uint32_t)(((tid / CH) * row_stride + kv * D + (tid % CH) * 8) * sizeof(uint16_t));
  };
  // the pair holding concatenated tile x (STREAM) or range x (SPLIT), its
  // first one in `f`
  auto locate = [&](int x, int &jj, int &kvv, int &f) {
    // (no branch, so the search stays scalar: with a loop, or a load under a
    // condition, the loops below need 60 more vector registers and spill)
    int e = 0;
#pragma unroll
    for (int b = kMaxLayers / 2; b > 0; b >>= 1) {
      const int at = a.e[min(e + b, a.st_entries - 1)].st_off;
      e += (int)(e + b < a.st_entries) & (int)(x >= at) ? b : 0;
    }
    jj = e;
    kvv = __builtin_amdgcn_readfirstlane((x - a.e[e].st_off) / a.e[e].st_tiles);
    f = a.e[e].st_off + kvv * a.e[e].st_tiles;
  };
  if constexpr (MODE != PLAIN) {
    int jj, kvv;
    locate(STREAM ? x_lo : unit, jj, kvv, first);
    enter(jj, kvv);
  } else {
    enter(lin / (nqt * Hkv), (lin / nqt) % Hkv);
  }

  // Double-buffered K and V tiles, both row-major [key][d]; V is read
  // transposed by ds_read_b64_tr_b16.  Row pads keep the K reads (16 B per
  // lane) and the transposed V reads (4 rows x 32 B per 16 lanes) spread
  // over the LDS banks.
  // A pass for the row LSE alone has no V tiles: 200 rows on 28 layers of 2 K to 6 K
  // tokens (16 KV heads), 267 us with V loaded and stored all the same, 208 now;
  // two, four and eight key groups 335 / 504 / 531 and 229 / 214 / 302.
  __shared__ __attribute__((aligned(16)))
  uint16_t tiles[KG * NBUF * BN * (D + KPAD + (WRITE_O ? D + VPAD : 0))];
  uint16_t(*Ks)[BN][D + KPAD] = reinterpret_cast<uint16_t(*)[BN][D + KPAD]>(tiles) + kg * NBUF;
  uint16_t(*Vs)[BN][D + VPAD] =
      reinterpret_cast<uint16_t(*)[BN][D + VPAD]>(tiles + (WRITE_O ? KG * NBUF * BN * (D + KPAD) : 0)) + kg * NBUF;
  uint4 kreg[NLD], vreg[NLD];
  // Tiles load through buffer descriptors whose base is the tile's first row
  // (scalar arithmetic): each load is the descriptor plus the lane's 32-bit
  // offset, with no per-lane 64-bit address addition.
  auto load_pure = [&](int t) {
    const int64_t at = (int64_t)t * BN * row_stride;
    const __amdgpu_buffer_rsrc_t kr =
        __builtin_amdgcn_make_buffer_rsrc((void *)(kc + at), 0, 0x7FFFFFFF, kBufferWord3);
    const __amdgpu_buffer_rsrc_t vr =
        __builtin_amdgcn_make_buffer_rsrc((void *)(vc + at), 0, 0x7FFFFFFF, kBufferWord3);
#pragma unroll
    for (int uu = 0; uu < NLD; ++uu) {
      const auto kx = __builtin_amdgcn_raw_buffer_load_b128(kr, (int)cofs, uu * cstep, 0);
      kreg[uu] = uint4{kx[0], kx[1], kx[2], kx[3]};
      if constexpr (WRITE_O) {
        const auto vx = __builtin_amdgcn_raw_buffer_load_b128(vr, (int)cofs, uu * cstep, 0);
        vreg[uu] = uint4{vx[0], vx[1], vx[2], vx[3]};
      }
    }
  };
  // Any tile: a descriptor for its rows in the cache and one for its new rows,
  // each ending with the last of them, so that rows past the end (and a whole
  // tile past it) load as zeros.  Only the tile with rows of both asks lane by
  // lane which it is.  (Tiles of one source each, the cache's end padded, were one
  // tile more a pass where T0 is no multiple of 64: one row on 28 layers of 700
  // tokens, 16 KV heads, 34.5 us, 32.0 now.)
  auto load_any = [&](int t) {
    const int at0 = t * BN;
    const int n_old = max(0, min(BN, T0 - at0)), r0 = max(0, at0 - T0);
    const int n_new = max(0, min(BN - n_old, C - r0));
    const int row_bytes = (int)(row_stride * sizeof(uint16_t));
    const int64_t ofs = n_new > 0 ? r0 * row_stride : 0;
    const __amdgpu_buffer_rsrc_t kr =
        __builtin_amdgcn_make_buffer_rsrc((void *)(kn + ofs), 0, n_new * row_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t vr =
        __builtin_amdgcn_make_buffer_rsrc((void *)(vn + ofs), 0, n_new * row_bytes, kBufferWord3);
    auto load = [&](__amdgpu_buffer_rsrc_t k, __amdgpu_buffer_rsrc_t v, int uu, int skip) {
      const auto kx = __builtin_amdgcn_raw_buffer_load_b128(k, (int)cofs + uu * cstep - skip, 0, 0);
      kreg[uu] = uint4{kx[0], kx[1], kx[2], kx[3]};
      if constexpr (WRITE_O) {
        const auto vx = __builtin_amdgcn_raw_buffer_load_b128(v, (int)cofs + uu * cstep - skip, 0, 0);
        vreg[uu] = uint4{vx[0], vx[1], vx[2], vx[3]};
      }
    };
    if (n_old == 0) {
#pragma unroll
      for (int uu = 0; uu < NLD; ++uu) load(kr, vr, uu, 0);
    } else {
      const int64_t at = at0 * row_stride;
      const __amdgpu_buffer_rsrc_t ko =
          __builtin_amdgcn_make_buffer_rsrc((void *)(kc + at), 0, n_old * row_bytes, kBufferWord3);
      const __amdgpu_buffer_rsrc_t vo =
          __builtin_amdgcn_make_buffer_rsrc((void *)(vc + at), 0, n_old * row_bytes, kBufferWord3);
#pragma unroll
      for (int uu = 0; uu < NLD; ++uu) {
        if (tid / CH + uu * (GT / CH) < n_old) load(ko, vo, uu, 0);
        else load(kr, vr, uu, n_old * row_bytes);
      }
    }
  };
  // tile t holds a key that some row of the block does not see
  auto edge = [&](int t) { return (t + 1) * BN - 1 > T0 + p0 / G; };
  auto store_tile = [&](int b) {
#pragma unroll
    for (int uu = 0; uu < NLD; ++uu) {
      const int e = tid + uu * GT;
      const int kr = e / CH, ch = e % CH;
      *reinterpret_cast<uint4 *>(&Ks[b][kr][ch * 8]) = kreg[uu];
      if constexpr (WRITE_O) *reinterpret_cast<uint4 *>(&Vs[b][kr][ch * 8]) = vreg[uu];
    }
  };

  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) o[db] = f32x16{};
  float m_run = -1e30f, l_run = 0.f;
  const float c = a.scale_log2, inv_c = 1.f / c;
  float m_lim = (m_run + 8.f) * inv_c;

  // transposed-read coordinates of this lane inside its 16-lane group
  const int tr_row = 4 * half + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  // key tile t of the current pair, in LDS buffer b.
  // `masked` is a std::integral_constant: the mask code folds away per call
  // site.
  auto compute = [&](int b, int t, auto masked) {
    // S^T = K Q^T for SUB 32-key sub-tiles: lane = query row, register = key.
    f32x16 s[SUB];
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub) {
      s[sub] = f32x16{};
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8 *>(&Ks[b][sub * 32 + l32][16 * kk + 8 * half]);
        s[sub] = mfma32(kf, qf[kk], s[sub]);
      }
    }
    // Schedule: kAheadK fragment reads, then one MFMA per read, so each MFMA's
    // operand was requested kAheadK MFMAs earlier (3% faster on the 7B
    // workload than all reads first).
#pragma unroll
    for (int i = 0; i < kAheadK; ++i) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
    for (int i = 0; i < SUB * (D / 16) - kAheadK; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < kAheadK; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (masked) {
      // last key of the tile that this row sees
      const int vis = T0 + r - t * BN;
#pragma unroll
      for (int sub = 0; sub < SUB; ++sub) {
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
          const int key = sub * 32 + 8 * (jj >> 2) + 4 * half + (jj & 3);
          if (key > vis) s[sub][jj] = -INFINITY;
        }
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub) {
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) mx = fmaxf(mx, s[sub][jj]);
    }
    {
      // the other lane half's maximum (rows are split over the halves by key):
      // v_permlane32_swap exchanges the halves of a register pair, so the max
      // of its two results holds both halves' maxima in every lane
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      const float m0 = __uint_as_float(r[0]), m1 = __uint_as_float(r[1]);
      mx = m0 > m1 ? m0 : m1;   // (a compare and a select: fmaxf would first canonicalise both)
    }
    // Lazy rescaling: the running maximum only moves when a row's tile
    // maximum exceeds it by more than 2^8 (in the log2 domain), so
    // probabilities stay <= 256; the test compares the raw maximum with the
    // precomputed threshold (m_run + 8) / c.  Rare after the first tiles, so it
    // lies out of line: 28 layers of 32768 + 3136 rows 56.98 -> 56.81 ms, and
    // 0.1-0.3% on the other large calls.
    if (__builtin_expect(__any(mx > m_lim), 0)) {
      const float m_new = fmaxf(m_run, mx * c);
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      m_lim = (m_run + 8.f) * inv_c;
      l_run *= alpha;
      if constexpr (WRITE_O) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) o[db] *= alpha;
      }
    }

    bf16x8 pf[2 * SUB];
    float ls = 0.f;
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub) {
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        const float p = fast_exp2(fmaf(s[sub][jj], c, -m_run));
        ls += p;
        pf[2 * sub + (jj >> 3)][jj & 7] = static_cast<__bf16>(p);
      }
    }
    l_run += ls;
    if constexpr (!WRITE_O) return;

    // O^T += V^T P^T.  B element t of lane half hf in key group qq is key
    // 16 qq + 8 (t/4) + 4 hf + t%4; two transposed reads give the matching
    // V^T fragment (keys 16 qq + 4 hf + 0..3 and 16 qq + 8 + 4 hf + 0..3).
    // The wave streams these MFMAs at raised issue priority, so that the
    // other wave on the SIMD fills the issue cycles they leave free with its
    // softmax rather than competing with them (3% on the 7B workload).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
#pragma unroll
      for (int qq = 0; qq < 2 * SUB; ++qq) {
        const uint16_t *vp = &Vs[b][16 * qq + tr_row][32 * db + tr_col];
        const s4 lo = lds_tr16(vp);
        const s4 hi = lds_tr16(vp + 8 * (D + VPAD));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o[db] = mfma32(vf, pf[qq], o[db]);
      }
    }
    // the same for O^T += V^T P^T: two transposed reads per MFMA, kAheadV
    // MFMAs ahead
    constexpr int kPV = (D / 32) * 2 * SUB;
#pragma unroll
    for (int i = 0; i < 2 * kAheadV; ++i) __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
#pragma unroll
    for (int i = 0; i < kPV - kAheadV; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
    }
#pragma unroll
    for (int i = 0; i < kAheadV; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
    __builtin_amdgcn_s_setprio(0);
  };

  using NoMask = std::integral_constant<bool, false>;
  using Mask = std::integral_constant<bool, true>;
  // Steps [s0, s0 + n) of the current pair: step x covers tiles x KG .. x KG +
  // KG - 1, one for each key group.  Steady state: this step's tiles and the
  // next one's are pure (no branch in the body); the last pure step joins the
  // general loop, where it is unmasked.
  auto walk = [&](int s0, int n) {
    int steps = (ntiles + KG - 1) / KG, pure_steps = n_pure / KG, tile0 = kg;
    if constexpr (MODE != PLAIN) {
      steps = min(steps - s0, n);
      pure_steps = min(pure_steps - s0, steps);
      tile0 += s0 * KG;
    }
    auto tile = [&](int s) { return s * KG + tile0; };
    // the group's waves wait for their tile's stores (all groups take the same
    // steps; a group of one wave only keeps its own order)
    auto sync = [&] {
      if constexpr (RG > 1) __syncthreads();
      else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    };
    if (pure_steps > 0) load_pure(tile(0)); else load_any(tile(0));
    int s = 0;
    // two steps per trip, so that the LDS buffer of each is a constant and its
    // addresses fold into the instructions' offsets
    for (; s + 2 < pure_steps; s += 2) {
      store_tile(0);
      sync();
      load_pure(tile(s + 1));
      if (wave_rows) compute(0, tile(s), NoMask{});
      store_tile(NBUF - 1);
      sync();
      load_pure(tile(s + 2));
      if (wave_rows) compute(NBUF - 1, tile(s + 1), NoMask{});
    }
    for (; s + 1 < pure_steps; ++s) {
      store_tile(s % NBUF);
      sync();
      load_pure(tile(s + 1));
      if (wave_rows) compute(s % NBUF, tile(s), NoMask{});
    }
    for (; s < steps; ++s) {
      store_tile(s % NBUF);
      sync();
      if (s + 1 < steps) load_any(tile(s + 1));   // (zeros past the last key)
      const int t = tile(s);
      if (!wave_rows || (KG > 1 && t >= ntiles)) {
      } else if (edge(t)) {
        compute(s % NBUF, t, Mask{});
      } else {
        compute(s % NBUF, t, NoMask{});
      }
    }
  };
  // The key groups' states merge through LDS: every wave leaves its (max, sum)
  // and O there ([4-channel group][lane], as it holds them), then wave kg of a
  // row group merges the KG-th part of the channels, groups in order.  mt and
  // lsum are the merged (max, sum); fn(c, x) gets channel group c.
  constexpr int NC = D / 8;                   // 4-channel groups of a lane half
  auto own = [&](int c) {
    return float4{o[c / 4][4 * (c % 4) + 0], o[c / 4][4 * (c % 4) + 1], o[c / 4][4 * (c % 4) + 2],
                  o[c / 4][4 * (c % 4) + 3]};
  };
  auto merge = [&](float &mt, float &lsum, auto fn) {
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if constexpr (KG == 1) {
      mt = m_run;
      lsum = l_tot;
#pragma unroll
      for (int c = 0; c < NC; ++c) fn(c, own(c));
    } else {
      static_assert(NC % KG == 0 && ((WRITE_O ? NW * NC * 64 * 16 : 0) + NW * 32 * 8) <= (int)sizeof(tiles),
                    "merge state fits");
      float4 *mo = reinterpret_cast<float4 *>(tiles);
      float2 *mm = reinterpret_cast<float2 *>(mo + (WRITE_O ? NW * NC * 64 : 0));
      __syncthreads();   // all tiles are read
      if constexpr (WRITE_O) {
#pragma unroll
        for (int c = 0; c < NC; ++c) mo[((kg * RG + wave) * NC + c) * 64 + lane] = own(c);
      }
      if (half == 0) mm[(kg * RG + wave) * 32 + l32] = float2{m_run, l_tot};
      __syncthreads();
      float wt[KG];
      mt = -1e30f;
      lsum = 0.f;
#pragma unroll
      for (int x = 0; x < KG; ++x) {
        wt[x] = mm[(x * RG + wave) * 32 + l32].x;
        mt = fmaxf(mt, wt[x]);
      }
#pragma unroll
      for (int x = 0; x < KG; ++x) {
        wt[x] = fast_exp2(wt[x] - mt);
        lsum += wt[x] * mm[(x * RG + wave) * 32 + l32].y;
      }
      if constexpr (WRITE_O) {
#pragma unroll
        for (int i = 0; i < NC / KG; ++i) {
          const int c = kg * (NC / KG) + i;
          float4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int x = 0; x < KG; ++x) {
            const float4 y = mo[((x * RG + wave) * NC + c) * 64 + lane];
            t.x += wt[x] * y.x;
            t.y += wt[x] * y.y;
            t.z += wt[x] * y.z;
            t.w += wt[x] * y.w;
          }
          fn(c, t);
        }
      }
    }
  };
  // unnormalised partial state of the current pair into partial block blk.
  // Each 32-row group is stored as the wave holds it ([4-channel group][lane]),
  // so that both the stores and the combine's loads are contiguous; lanes past
  // the packed rows write nothing.
  auto flush = [&](int64_t blk) {
    const int64_t rg = blk * a.part_groups + (p0 >> 5) + wave;
    float4 *op = reinterpret_cast<float4 *>(a.opart) + rg * NC * 64 + lane;
    float mt, lsum;
    merge(mt, lsum, [&](int c, float4 x) {
      if (row_ok) op[c * 64] = x;
    });
    if (row_ok && kg == 0 && half == 0)
      *reinterpret_cast<float2 *>(a.mlpart + 2 * (rg * 32 + l32)) = float2{mt, lsum};
  };
  if constexpr (STREAM) {
    // Pair by pair over the range, each with the loops of the plain kernel (4%
    // faster than one loop over all tiles with the mask decided at run time).
    // No early exit and one way out of the loop: a return in it, or before it,
    // cost 50-70 vector registers and spilled.
    int t = x_lo - first, k = j * Hkv + kv, x = x_lo;
    do {
      const int n = min(a.e[j].st_tiles - t, x_hi - x);
      walk(t, n);
      flush(u + k);
      x += n;
      t = 0;
      ++k;
      if (x < x_hi) {
        if (kv + 1 < Hkv) enter(j, kv + 1); else enter(j + 1, 0);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) o[db] = f32x16{};
        m_run = -1e30f;
        m_lim = (m_run + 8.f) * inv_c;
        l_run = 0.f;
        __syncthreads();   // the last tile (or the merge) may still be read from the buffers that the next one takes
      }
    } while (x < x_hi);
  } else if constexpr (MODE == SPLIT) {
    walk((unit - first) * a.st_units, a.st_units);
    flush(unit);
  } else {
    walk(0, ntiles);
    uint16_t *orow = a.out + a.e[j].slot * a.q_lstride + ((int64_t)r * Hq + kv * G + g) * D + 4 * half;
    float mt, lsum;
    merge(mt, lsum, [&](int c, float4 x) {
      const float inv = 1.f / lsum;
      if (WRITE_O && row_ok)
        *reinterpret_cast<uint2 *>(orow + 8 * c) =
            uint2{(uint32_t)f2bf(x.x * inv) | ((uint32_t)f2bf(x.y * inv) << 16),
                  (uint32_t)f2bf(x.z * inv) | ((uint32_t)f2bf(x.w * inv) << 16)};
    });
    if (row_ok && a.lse != nullptr && kg == 0 && half == 0)
      a.lse[a.e[j].layer * a.lse_lstride + (int64_t)kv * P + prow] = mt + log2f(lsum);
  }
  if (a.pos != nullptr) copy_share(a, D, blockIdx.x, min((int)gridDim.x, kStreamSlots));
}

// Merge of a pair's partial blocks: m = max_s m_s, w_s = 2^(m_s - m),
// O = sum_s w_s O_s / sum_s w_s l_s, LSE = m + log2(sum_s w_s l_s).  Pair
// k = j Hkv + kv covers concatenated tiles [f, f + n); units u0 (holding
// tile f) to u1 (holding tile f + n - 1) wrote its blocks u0 + k .. u1 + k.  In
// split mode f and n count ranges and the blocks are f .. f + n - 1.
// A workgroup merges 32 channels of a 32-row group: wave w takes the blocks
// w, w + 4, ... in order, kCombineAhead of them loaded at once, and the four
// waves' sums are added in wave order.  The launch is bound by the latency of
// its loads: with one thread walking all blocks one by one, a pair's 64
// blocks took 20-31 us, now 4-6.  784 rows of one layer (40 MB of partials):
// 12.5 us with 4 loaded at once, 10.5 with 2 (more waves fit), 17 with 8.
constexpr int kCombineAhead = 2;
template <int D>
__global__ __launch_bounds__(256) void attn_combine(AttnArgs a) {
  const int j = blockIdx.z, kv = blockIdx.y;
  const int layer = a.e[j].layer;
  const int G = a.Hq / a.Hkv, P = a.C * G;
  const int rgi = blockIdx.x / (D / 32), db = blockIdx.x % (D / 32);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l32 = lane & 31, half = lane >> 5;
  // the unit whose range [u N / U, (u + 1) N / U) holds tile x
  auto unit_of = [&](int64_t x) {
    return (int)(((x + 1) * a.st_units + a.st_total - 1) / a.st_total - 1);
  };
  const int64_t f = a.e[j].st_off + (int64_t)kv * a.e[j].st_tiles;
  const int u0 = a.split ? (int)f : unit_of(f);
  const int nsp = a.split ? a.e[j].st_tiles : unit_of(f + a.e[j].st_tiles - 1) - u0 + 1;
  const int64_t rg0 = ((int64_t)u0 + (a.split ? 0 : j * a.Hkv + kv)) * a.part_groups + rgi;
  // lanes past the packed rows read the group's first row, which others read too
  const int p = rgi * 32 + l32, src = p < P ? lane : 32 * half;
  const float4 *op = reinterpret_cast<const float4 *>(a.opart) + (rg0 * (D / 8) + 4 * db) * 64 + src;
  const int64_t ostep = (int64_t)a.part_groups * (D / 8) * 64, mstep = (int64_t)a.part_groups * 32;
  const float2 *ml = reinterpret_cast<const float2 *>(a.mlpart) + rg0 * 32 + (src & 31);

  float m = -1e30f, l = 0.f;
  float4 acc[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) acc[g] = float4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = wave; s0 < nsp; s0 += 4 * kCombineAhead) {
    float2 x[kCombineAhead];
    float4 v[kCombineAhead][4];
#pragma unroll
    for (int u = 0; u < kCombineAhead; ++u) {
      const int s = s0 + 4 * u;
      if (s >= nsp) {
        x[u] = float2{-1e30f, 0.f};
#pragma unroll
        for (int g = 0; g < 4; ++g) v[u][g] = float4{0.f, 0.f, 0.f, 0.f};
        continue;
      }
      x[u] = ml[s * mstep];
#pragma unroll
      for (int g = 0; g < 4; ++g) v[u][g] = op[s * ostep + g * 64];
    }
    float mn = m;
#pragma unroll
    for (int u = 0; u < kCombineAhead; ++u) mn = fmaxf(mn, x[u].x);
    const float w0 = exp2f(m - mn);
    m = mn;
    l *= w0;
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = float4{acc[g].x * w0, acc[g].y * w0, acc[g].z * w0, acc[g].w * w0};
#pragma unroll
    for (int u = 0; u < kCombineAhead; ++u) {
      const float w = exp2f(x[u].x - m);
      l += w * x[u].y;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 y = v[u][g];
        acc[g].x += w * y.x;
        acc[g].y += w * y.y;
        acc[g].z += w * y.z;
        acc[g].w += w * y.w;
      }
    }
  }
  __shared__ float4 sacc[4][4][64];
  __shared__ float2 sml[4][64];
#pragma unroll
  for (int g = 0; g < 4; ++g) sacc[wave][g][lane] = acc[g];
  sml[wave][lane] = float2{m, l};
  __syncthreads();
  // wave w finishes the 4-channel group w
  float mt = sml[0][lane].x, lsum = 0.f;
#pragma unroll
  for (int w = 1; w < 4; ++w) mt = fmaxf(mt, sml[w][lane].x);
  float4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float2 x = sml[w][lane];
    const float4 y = sacc[w][wave][lane];
    const float e = exp2f(x.x - mt);
    lsum += e * x.y;
    t.x += e * y.x;
    t.y += e * y.y;
    t.z += e * y.z;
    t.w += e * y.w;
  }
  if (p >= P) return;
  const int r = p / G, h = kv * G + (p - r * G);
  if (a.out != nullptr) {
    const float inv = 1.f / lsum;
    uint16_t *orow = a.out + a.e[j].slot * a.q_lstride + ((int64_t)r * a.Hq + h) * D + 32 * db + 8 * wave + 4 * half;
    *reinterpret_cast<uint2 *>(orow) = uint2{(uint32_t)f2bf(t.x * inv) | ((uint32_t)f2bf(t.y * inv) << 16),
                                             (uint32_t)f2bf(t.z * inv) | ((uint32_t)f2bf(t.w * inv) << 16)};
  }
  if (a.lse != nullptr && db == 0 && wave == 0 && half == 0)
    a.lse[layer * a.lse_lstride + (int64_t)kv * P + p] = mt + log2f(lsum);
}

template <int D>
__global__ __launch_bounds__(256, 3) void attn_colsum(ColsumArgs a, int nkb) {
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int kblk = lin % nkb;
  int group = lin / nkb, split = 0;
  if (a.splits > 1) {
    split = group % a.splits;
    group /= a.splits;
  }
  const int kv_blk = group % a.Hkv;
  const int j = group / a.Hkv;
  const MassEntry &en = a.e[j];
  const int layer = en.layer;
  const int T0 = en.T0;
  const int C = a.C, Hq = a.Hq, Hkv = a.Hkv;
  const int G = Hq / Hkv;
  const int P = C * G;
  const int T = en.ncand;          // candidates: T0 + C, or T0 for a prompt
  const int k0 = kblk * BK;
  if (k0 >= T) return;

  // wave index made scalar: the loop bounds below derive from it and stay uniform
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int half = lane >> 5, l32 = lane & 31;
  // Each wave owns 64 candidates (two MFMA column blocks of 32).
  const int kw0 = k0 + wave * 64;
  int key[2], pmin[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    key[kb] = kw0 + 32 * kb + l32;
    pmin[kb] = key[kb] < T0 ? 0 : (key[kb] - T0) * G;   // first packed row that sees it
  }
  // rows below pmask_end may be invisible to some candidate of this wave
  const int pmask_end = kw0 + 63 < T0 ? 0 : (kw0 + 63 - T0) * G + 1;
  const int p_first = (k0 < T0 ? 0 : (k0 - T0) * G) & ~(BQS - 1);
  const int ntq = (P - p_first + BQS - 1) / BQS;
  // this split's share of the block's query tiles (possibly none: it then
  // writes zeros); at most 32 splits of 2^25 tiles, so 32 bits hold the products
  // (two 64-bit divisions in every workgroup, split or not, and a branch before
  // the first tile's loads: 273 us, 259 now, 28 layers of 3 K to 7 K tokens, 16 KV
  // heads, 200 prompt rows)
  int t_lo = 0, nit = ntq;
  if (a.splits > 1) {
    t_lo = split * ntq / a.splits;
    nit = (split + 1) * ntq / a.splits - t_lo;
  }
  const int p_begin = p_first + t_lo * BQS;

  const int slot = en.slot;
  const uint16_t *q = a.q + slot * a.q_lstride;
  const uint16_t *kn = a.kn + slot * a.kv_lstride;
  const uint16_t *kc = en.k;
  const float *lse_l = a.lse + layer * a.lse_lstride;
  const float c = a.scale_log2;

  // Ring of 32-row query tiles (four slots, so the slot index is a mask):
  // tile it is read by the MFMAs while tile it+2 is stored and tile it+3
  // loaded.
  __shared__ __attribute__((aligned(16))) uint16_t Qs[4][BQS][D + KPAD];
  __shared__ __attribute__((aligned(16))) float Ls[4][BQS];

  constexpr int CH = D / 8;
  constexpr int NLD = BQS * CH / 256;
  uint4 qreg[NLD];
  float lreg = INFINITY;
  auto tile_p = [&](int it) { return p_begin + it * BQS; };
  // Each thread loads NLD 16-byte pieces of one packed row of a tile (pieces
  // c and c + CH / NLD, ...), so one offset per thread serves all of them.
  // Tiles are loaded in order, so the thread's packed row p = (r, g) steps
  // by BQS per tile: r by BQS / G and g by BQS % G, plus one row when g wraps
  // past G; its byte offset moves by the matching fixed amounts.  The loads
  // go through a buffer descriptor over this slot's C chunk rows, so the
  // offset is a 32-bit register and rows past P (r >= C) lie outside the
  // descriptor's range, where the load returns zeros.
  constexpr int PPR = CH / NLD;             // pieces per thread-row group
  const int ld_row = tid / PPR, ld_c = tid % PPR;
  const __amdgpu_buffer_rsrc_t qrs =
      __builtin_amdgcn_make_buffer_rsrc((void *)q, 0, C * Hq * D * (int)sizeof(uint16_t), kBufferWord3);
  const int step_r = BQS / G, step_g = BQS - (BQS / G) * G;
  const uint32_t ostep = (uint32_t)((step_r * Hq + step_g) * D * sizeof(uint16_t));
  const uint32_t owrap = (uint32_t)((Hq - G) * D * sizeof(uint16_t));
  int ld_g;
  uint32_t ld_o;
  {
    const int p = p_begin + ld_row;
    const int r0 = p / G;
    ld_g = p - r0 * G;
    ld_o = (uint32_t)((((int64_t)r0 * Hq + kv_blk * G + ld_g) * D + ld_c * 8) * sizeof(uint16_t));
  }
  // FULL: every row of the tile is < P (no bounds test on the LSE load)
  auto load_tile = [&](int it, auto full) {
    const int pt = tile_p(it);
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(qrs, (int)(ld_o + u * PPR * 16), 0, 0);
      qreg[u] = uint4{x[0], x[1], x[2], x[3]};
    }
    ld_g += step_g;
    const bool wrap = ld_g >= G;
    ld_g -= wrap ? G : 0;
    ld_o += ostep + (wrap ? owrap : 0u);
    if (tid < BQS)
      lreg = (decltype(full)::value || pt + tid < P) ? lse_l[(int64_t)kv_blk * P + pt + tid] : INFINITY;
  };
  auto store_tile = [&](int b) {
#pragma unroll
    for (int u = 0; u < NLD; ++u)
      *reinterpret_cast<uint4 *>(&Qs[b][ld_row][(ld_c + u * PPR) * 8]) = qreg[u];
    if (tid < BQS) Ls[b][tid] = lreg;
  };

  bf16x8 kf[2][D / 16];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const bool ok = key[kb] < T;
    const uint16_t *krow = key[kb] < T0 ? kc + ((int64_t)key[kb] * Hkv + kv_blk) * D
                                        : kn + ((int64_t)(key[kb] - T0) * Hkv + kv_blk) * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
      kf[kb][kk] = ok ? __builtin_bit_cast(bf16x8, gload16(krow + 16 * kk + 8 * half)) : bf16x8{};
  }
  // S = Q K^T for one 32-row tile: lane = candidate, register = query row.
  auto scores = [&](int b, f32x16 *s) {
    s[0] = f32x16{};
    s[1] = f32x16{};
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const bf16x8 qv = *reinterpret_cast<const bf16x8 *>(&Qs[b][l32][16 * kk + 8 * half]);
      s[0] = mfma32(qv, kf[0][kk], s[0]);
      s[1] = mfma32(qv, kf[1][kk], s[1]);
    }
  };
  double wacc[2] = {0.0, 0.0};
  auto read_lse = [&](int b, float *lv) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const float4 l4 = *reinterpret_cast<const float4 *>(&Ls[b][8 * grp + 4 * half]);
      lv[4 * grp + 0] = l4.x;
      lv[4 * grp + 1] = l4.y;
      lv[4 * grp + 2] = l4.z;
      lv[4 * grp + 3] = l4.w;
    }
  };
  auto acc_masked = [&](int it, const f32x16 *s, const float *lv) {
    const int pt = tile_p(it);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float ts = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int prow = pt + 8 * (e >> 2) + 4 * half + (e & 3);
        const float p = fast_exp2(fmaf(s[kb][e], c, -lv[e]));
        ts += prow >= pmin[kb] ? p : 0.f;
      }
      wacc[kb] += (double)ts;
    }
  };
  auto acc_plain = [&](const f32x16 *s, const float *lv) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float t0 = fast_exp2(fmaf(s[kb][0], c, -lv[0]));
      float t1 = fast_exp2(fmaf(s[kb][1], c, -lv[1]));
#pragma unroll
      for (int e = 2; e < 16; e += 2) {
        t0 += fast_exp2(fmaf(s[kb][e], c, -lv[e]));
        t1 += fast_exp2(fmaf(s[kb][e + 1], c, -lv[e + 1]));
      }
      wacc[kb] += (double)(t0 + t1);
    }
  };
  // tiles [0, n_mask) touch the causal edge of this wave's candidates
  const int n_mask = min(nit, max(0, (pmask_end - p_begin + BQS - 1) / BQS));

  using Full = std::integral_constant<bool, true>;
  using Edge = std::integral_constant<bool, false>;
  // tiles [0, nfull) lie wholly below P
  const int nfull = min(nit, (P - p_begin) / BQS);
  load_tile(0, Edge{});   // (a split with no tile loads one too, so that no branch parts this from the K loads)
  store_tile(0);
  if (nit > 1) {
    load_tile(1, Edge{});
    store_tile(1);
  }
  if (nit > 2) load_tile(2, Edge{});
  __syncthreads();
  // One tile per trip, scores then probabilities: without a second score
  // buffer the kernel fits three waves per SIMD, which hide the MFMA and LDS
  // latency better than overlapping two tiles inside one wave did.
  f32x16 s_cur[2];
  auto step = [&](int it, auto masked) {
    float lv[16];
    scores(it & 3, s_cur);
    read_lse(it & 3, lv);
    if constexpr (decltype(masked)::value) acc_masked(it, s_cur, lv); else acc_plain(s_cur, lv);
    if (it + 2 < nit) {
      store_tile((it + 2) & 3);
      if (it + 3 < nit) load_tile(it + 3, Edge{});
    }
    __syncthreads();
  };
  int it = 0;
  for (; it < n_mask; ++it) step(it, std::integral_constant<bool, true>{});
  // steady state: no branches inside the body
  for (; it + 3 < nfull; ++it) {
    float lv[16];
    scores(it & 3, s_cur);
    read_lse(it & 3, lv);
    acc_plain(s_cur, lv);
    store_tile((it + 2) & 3);
    load_tile(it + 3, Full{});
    __syncthreads();
  }
  for (; it < nit; ++it) step(it, std::integral_constant<bool, false>{});
  double *part = a.wpart + (layer - a.layer0) * a.wpart_lstride + (int64_t)(kv_blk * a.splits + split) * a.wpart_hstride;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const double wsum = wacc[kb] + __shfl_xor(wacc[kb], 32);
    if (key[kb] < T && half == 0) part[key[kb]] = wsum;
  }
}

// W_i = the sum of the fp64 partials (KV heads, and within a head its splits
// of the query rows), rounded to fp32; with it, per block of kNormBlock
// candidates, the fp64 partial of the attention-score normaliser
// sum_i alpha_i W_i over the rounded W (thread order within each wave by a
// fixed butterfly, then the waves in order).  A launch with many partials has
// few candidates, one workgroup a CU at most, and is bound by the latency of
// its loads: MG = 4 groups of threads then share a candidate's partials (each
// a contiguous run, eight loads in flight; the runs are added in order).  One
// layer of 8976 candidates with 20 partials: 4.7 us, 7.7 with one group and
// one load at a time; 25 layers with 4 partials: 5.2 us with MG = 1, 9.1 with
// 4, so up to eight partials stay with one thread.
template <int MG>
__global__ __launch_bounds__(kNormBlock *MG) void mass_reduce(ColsumArgs a) {
  const int j = blockIdx.y;
  const MassEntry &en = a.e[j];
  const int layer = en.layer;
  const int T = en.ncand;
  if ((int)blockIdx.x * kNormBlock >= T) return;   // whole block past this layer's end
  __shared__ double run[MG > 1 ? MG - 1 : 1][kNormBlock];
  __shared__ double red[kNormBlock / 64];
  const int lc = threadIdx.x % kNormBlock, grp = threadIdx.x / kNormBlock;
  const int i = blockIdx.x * kNormBlock + lc;
  const int n = a.Hkv * a.splits;
  double w = 0.0;
  if (i < T) {
    const double *part = a.wpart + (layer - a.layer0) * a.wpart_lstride + i;
    const int x1 = (grp + 1) * n / MG;
    for (int x0 = grp * n / MG; x0 < x1; x0 += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = x0 + u < x1 ? part[(int64_t)(x0 + u) * a.wpart_hstride] : 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) w += v[u];
    }
  }
  if constexpr (MG > 1) {
    if (grp > 0) run[grp - 1][lc] = w;
    __syncthreads();
  }
  double m = 0.0;
  if (grp == 0) {
#pragma unroll
    for (int x = 0; x < MG - 1; ++x) w += run[x][lc];
    if (i < T) {
      const float wf = (float)w;
      en.w[i] = wf;
      m = mass_over_observers(wf, i, en.T0, a.C, en.alpha_mode);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m += __shfl_xor(m, o);
    if ((lc & 63) == 0) red[lc >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int x = 0; x < kNormBlock / 64; ++x) s += red[x];
    a.normpart[layer * a.normpart_lstride + blockIdx.x] = s;
  }
}

}  // namespace

template <int D, int KG>
static void plain_pass(const AttnArgs &a, int n_list, hipStream_t s) {
  constexpr int rows = BM / KG;
  const int nqt = (a.C * (a.Hq / a.Hkv) + rows - 1) / rows;
  const dim3 grid(nqt * a.Hkv * n_list);
  if (a.out != nullptr) hipLaunchKernelGGL((attn_fwd<D, 8, KG, PLAIN, true>), grid, dim3(AT), 0, s, a, nqt);
  else hipLaunchKernelGGL((attn_fwd<D, 8, KG, PLAIN, false>), grid, dim3(AT), 0, s, a, nqt);
}

template <int D>
static void plain_pass_of(const AttnArgs &a, int n_list, int key_groups, hipStream_t s) {
  switch (key_groups) {
    case 8: plain_pass<D, 8>(a, n_list, s); break;
    case 4: plain_pass<D, 4>(a, n_list, s); break;
    case 2: plain_pass<D, 2>(a, n_list, s); break;
    default: plain_pass<D, 1>(a, n_list, s); break;
  }
}

hipError_t launch_attention(const AttnArgs &a, int n_list, int head_dim, hipStream_t s) {
  if (head_dim == 64) plain_pass_of<64>(a, n_list, a.key_groups, s);
  else plain_pass_of<128>(a, n_list, a.key_groups, s);
  return hipGetLastError();
}

template <int D>
static hipError_t parted_pass(const AttnArgs &a, int n_list, hipStream_t s) {
  const int P = a.C * (a.Hq / a.Hkv);
  if (a.split == 2) {
    const int nqt = (P + BM / a.key_groups - 1) / (BM / a.key_groups);
    const dim3 grid(a.e[n_list].st_off * nqt);
    if (a.key_groups == 2) hipLaunchKernelGGL((attn_fwd<D, 8, 2, SPLIT, true>), grid, dim3(AT), 0, s, a, nqt);
    else if (a.key_groups == 4) hipLaunchKernelGGL((attn_fwd<D, 8, 4, SPLIT, true>), grid, dim3(AT), 0, s, a, nqt);
    else hipLaunchKernelGGL((attn_fwd<D, 8, 8, SPLIT, true>), grid, dim3(AT), 0, s, a, nqt);
  } else if (a.split == 1) {
    const dim3 grid(a.e[n_list].st_off), block(256);
    if (P <= 32) hipLaunchKernelGGL((attn_fwd<D, 4, 4, SPLIT, true>), grid, block, 0, s, a, 1);
    else if (P <= 64) hipLaunchKernelGGL((attn_fwd<D, 4, 2, SPLIT, true>), grid, block, 0, s, a, 1);
    else hipLaunchKernelGGL((attn_fwd<D, 4, 1, SPLIT, true>), grid, block, 0, s, a, 1);
  } else {
    const int nqt = (P + BM - 1) / BM;
    hipLaunchKernelGGL((attn_fwd<D, 8, 1, STREAMED, true>), dim3(a.st_units * nqt), dim3(AT), 0, s, a, nqt);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(attn_combine<D>, dim3(a.part_groups * (D / 32), a.Hkv, n_list), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_attention_parted(const AttnArgs &a, int n_list, int head_dim, hipStream_t s) {
  return head_dim == 64 ? parted_pass<64>(a, n_list, s) : parted_pass<128>(a, n_list, s);
}

hipError_t launch_colsum(const ColsumArgs &a, int n_list, int max_T, int head_dim,
                         hipStream_t s) {
  const int nkb = (max_T + BK - 1) / BK;
  dim3 grid(nkb * a.splits * a.Hkv * n_list);
  if (head_dim == 64) {
    hipLaunchKernelGGL(attn_colsum<64>, grid, dim3(256), 0, s, a, nkb);
  } else {
    hipLaunchKernelGGL(attn_colsum<128>, grid, dim3(256), 0, s, a, nkb);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 rgrid((max_T + kNormBlock - 1) / kNormBlock, n_list);
  if (a.Hkv * a.splits > 8) hipLaunchKernelGGL(mass_reduce<4>, rgrid, dim3(kNormBlock * 4), 0, s, a);
  else hipLaunchKernelGGL(mass_reduce<1>, rgrid, dim3(kNormBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace hermes
