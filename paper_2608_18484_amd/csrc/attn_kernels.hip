// Attention-side kernels of the SparsePR operator for gfx950:
//  * renormalised hard-drop block-sparse attention over the routed cells
//    (Sec. 3 eq. hard_drop; Sec. 4.3), bf16 MFMA with fp32 accumulation, or
//    an fp32 MFMA variant;
//  * exact probe rows against all keys (Sec. 4.3; App. A.2 eq.
//    app_probe_residual), split over keys and merged by log-sum-exp;
//  * the probe-fitted residual fit, correction and restore are launched from
//    here and live in fit_kernels.hip.
//
// Layout of the bf16 attention kernel.  A block of NW waves (2, or for large
// launches 3) owns up to 32 NW query rows of one query group; each wave
// owns 32 of them.
// The scores are formed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16
// (A = 32 keys x 16 dims from LDS, B = 16 dims x 32 queries held in
// registers), so every lane holds scores of ONE query and the online softmax
// needs a single cross-lane exchange (lanes l and l+32).  The probabilities
// stay in registers and feed O^T = V^T P^T directly as the B operand; V stays
// row-major in LDS and its A operand V^T comes from transposing LDS reads
// (ds_read_b64_tr_b16), the keys of each 16-key chunk taken in the order of
// the accumulator layout.
// K/V rows are gathered on load through the group-major permutation, so the
// routed K/V groups are contiguous key ranges without a physical copy.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>

#include <type_traits>

#include "device_utils.hpp"
#include "sparsepr_internal.hpp"

namespace sparsepr {

// Running maximum before any finite score.  Not -inf: keys whose scores are all
// -inf (the first tile of a key part or of a key split, say) then add nothing,
// where (-inf) - (-inf) would turn the rows they share with other keys to NaN.
constexpr float kNoMax = -FLT_MAX;

enum { MODE_SPARSE = 0, MODE_PROBE = 1, MODE_DENSE = 2 };  // MODE_DENSE: k_attn_f32 only

struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  void* out;          // MODE_DENSE: user output tensor
  float* osp;         // MODE_SPARSE: [BH][N][D] fp32
  float* part;        // MODE_PROBE: [BH][M][nsplit][D+2]
  const int4* chunks;
  const int32_t* nchunks;
  const int32_t* permq;
  const int32_t* offq;
  const int32_t* permk;
  const int2* rng;
  const int32_t* rng_cnt;
  const int32_t* probes;
  const int32_t* nprobes;
  const uint16_t* kperm;
  const uint16_t* vperm;
  // MODE_SPARSE key segment: only keys at group-major positions in
  // [seg_lo, seg_hi) are processed; (O, m, l) carry over between segments
  float* mlst;
  int seg_lo, seg_hi, seg_first, seg_last;
  int heads_per_xcd;  // MODE_SPARSE block order (see k_attn_mfma)
  int cls;            // MODE_SPARSE: class of work items of this launch
};

// Where the rows and keys of one block come from.
struct Work1 {
  int nrows;      // valid query rows (<= 32 NW)
  int nkeys;      // keys in the flat key list
  int k0;         // MODE_PROBE: first key row
  int a;          // MODE_SPARSE: query group
  int rbase;      // MODE_SPARSE: first permutation slot of the rows
  int split;      // MODE_PROBE: split index
  int tile;       // MODE_PROBE: row tile
};

template <int MODE>
__device__ __forceinline__ bool get_work(const Geom& g, const AttnArgs& A, int bh, Work1& w) {
  if (MODE == MODE_SPARSE) {
    const int cx = blockIdx.x;
    if (cx >= A.nchunks[bh * kItemClasses + kItemClasses - 1]) return false;
    const int4 c = A.chunks[(size_t)bh * g.nchunk_max + cx];
    w.a = c.x;
    w.rbase = A.offq[(size_t)bh * (g.CQt + 1) + c.x] + c.y;
    w.nrows = c.z;
    w.nkeys = c.w;
    w.k0 = 0;
    return w.nrows > 0 && w.nkeys > 0;
  } else if (MODE == MODE_PROBE) {
    const int np = A.nprobes[bh];
    w.tile = blockIdx.x;
    w.split = blockIdx.y;
    if (w.tile * 64 >= np) return false;
    w.nrows = min(64, np - w.tile * 64);
    w.k0 = w.split * g.psplit;
    w.nkeys = min(g.N - w.k0, g.psplit);
    return w.nkeys > 0;
  } else {
    w.tile = blockIdx.x;
    w.nrows = min(64, g.N - w.tile * 64);
    w.k0 = 0;
    w.nkeys = g.N;
    return w.nrows > 0;
  }
}

template <int MODE>
__device__ __forceinline__ int row_of(const Geom& g, const AttnArgs& A, int bh, const Work1& w,
                                      int r) {
  if (MODE == MODE_SPARSE) return A.permq[(size_t)bh * g.N + w.rbase + r];
  if (MODE == MODE_PROBE) return A.probes[(size_t)bh * g.M + w.tile * 64 + r];
  return w.tile * 64 + r;
}

// Source row of flat key f (f < nkeys).  MODE_SPARSE walks the routed ranges
// with a per-thread cursor that only moves forward.
struct KeyCursor {
  int j, cum;
};

template <int MODE>
__device__ __forceinline__ int key_row(const Geom& g, const AttnArgs& A, int bh, const Work1& w,
                                       int f, KeyCursor& cur, const int2* rg, int nr) {
  if (MODE != MODE_SPARSE) return w.k0 + f;
  while (cur.j < nr && f >= cur.cum + rg[cur.j].y) {
    cur.cum += rg[cur.j].y;
    ++cur.j;
  }
  return A.permk[(size_t)bh * g.N + rg[cur.j].x + (f - cur.cum)];
}

// Bank swizzle of the 16-byte chunks of a K/V tile row in LDS: chunk c of
// key r sits at position c ^ swz(r).  A 16-lane phase of a 128-bit read (the
// K operand) takes one chunk of 16 consecutive keys, and one of a transposing
// read takes two neighbouring chunks of 4 consecutive keys (two phases: four
// chunks).  With 256-byte rows (D = 128) a row spans the 64 banks once, so
// swz is a bijection of 16 consecutive keys onto the 16 chunk positions whose
// bits 2-3 differ within every aligned group of 4 keys: both reads hit
// distinct banks.  With 128-byte rows (D = 64) two keys share a bank row and
// the 3-bit form is used.
template <int D>
__device__ __forceinline__ int kv_swz(int r) {
  if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  return ((r & 3) << 1) | ((r >> 2) & 1);
}

// Vectors in memory that is only as aligned as its elements: the callers' fp32
// rows and outputs (a base pointer need not be aligned further) and the probe
// partials' rows of D + 2 floats.  gfx950 moves them by the same wide accesses.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_u __attribute__((ext_vector_type(2), aligned(2)));

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// LDS transposing read of four 16-bit values.  In every group of 16 lanes,
// lane j receives element j%4 of the 8-byte rows addressed by lanes
// j/4, j/4+4, j/4+8, j/4+12 of its group.
__device__ __forceinline__ v4i16 lds_read_tr16(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_v4i16*)(__attribute__((address_space(3))) uint16_t*)(p));
}

// Direct global->LDS copy of 16 bytes per lane: lane l's bytes land at
// m0v + 16*l, m0v being the wave-uniform LDS address, from a uniform 64-bit
// base (SGPRs) plus a 32-bit per-lane byte offset.  Issued as inline assembly
// so that the compiler adds no waits for it; callers order it with explicit
// s_waitcnt vmcnt.  Nothing else in these kernels uses M0.
__device__ __forceinline__ void g2lds16s(const void* sbase, uint32_t voff, uint32_t m0v) {
  // readfirstlane returns a signed int: widen through uint32_t so the low
  // half of the address is zero-extended, never sign-extended
  const uint64_t b = (uint64_t)(size_t)sbase;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const uint64_t sb = ((uint64_t)hi << 32) | (uint64_t)lo;
  const uint32_t m0u = (uint32_t)__builtin_amdgcn_readfirstlane(m0v);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:0"
               :
               : "v"(voff), "s"(sb), "s"(m0u)
               : "memory");
}

// Combine a value with the one held by lane l ^ 32 (the other half of the
// same query's keys) through v_permlane32_swap: swapping a register with
// itself leaves, in each lane, its own value in one result and its partner's
// in the other, so max3 / the sum of both results combine the pair.
__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Block-sparse flash attention, bf16 MFMA, fp32 accumulation.
//  * NW waves; a block owns up to 32 NW query rows (32 per wave) that share
//    one key list: the routed ranges of their query group in the
//    group-major K/V copy (MODE_SPARSE), or a contiguous slice of the original
//    K/V rows (MODE_PROBE).
//  * 32-key tiles in LDS filled by direct global->LDS 16-byte loads: one K
//    buffer, refilled with the next tile once every wave has read its score
//    operands, and two V buffers, the next tile's V loading while the current
//    one is computed; the key positions of a tile are computed two tiles
//    ahead into a ring of three slots.  The 26 KB of LDS and at most 168
//    registers per lane leave room for six blocks of two waves per CU (three
//    waves per SIMD), which hide each other's latencies better than four.
//    Blocks of three waves have LDS to spare at that occupancy: their
//    K is double-buffered too and a step has one barrier.
//  * S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_32x32x16_bf16; V^T
//    fragments come from the row-major V tile through transposing LDS reads.
//  * Online softmax in base 2 with lazy rescaling: the running maximum only
//    moves (and O, l are rescaled) when a tile's maximum exceeds it by 2^8.
template <int D, int MODE, int NW = 2>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_attn_mfma(Geom g, AttnArgs A) {
  constexpr int KT = 32, NT = 64 * NW;
  constexpr int CH = D / 8;                    // 16-byte chunks per row
  constexpr int NKS = D / 16;                  // k-steps of Q K^T
  constexpr int NDB = D / 32;                  // 32-wide blocks of O^T
  constexpr int NCP = KT * CH / 64;            // 1 KB copies per tensor per tile,
  constexpr int LPT = (NCP + NW - 1) / NW;     // at most so many per wave
  constexpr int MAXR = 128;                    // routed ranges of the segment staged in LDS
  constexpr bool K2 = NW > 2;                  // K double-buffered
  // tiles[0] = K (one buffer), tiles[1..2] = V (double-buffered), tiles[3] =
  // K's second buffer
  __shared__ __attribute__((aligned(1024))) uint16_t tiles[K2 ? 4 : 3][KT * D];
  __shared__ int spos[3][KT];
  __shared__ int2 srng[MODE == MODE_SPARSE ? MAXR : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  Work1 w;
  int bh, jq;  // K/V head, and which of its G query heads
  const uint16_t* Kp;
  const uint16_t* Vp;
  if (MODE == MODE_SPARSE) {
    // XCD-aware order: hardware block b runs on XCD b % 8, which takes the
    // items b / 8 of its share in turn, the G query heads of a K/V head one
    // after the other for each item (they read the same keys).
    //  * heads_per_xcd (K/V head count a multiple of 8): grid (8 G items, BH / 8);
    //    XCD x runs every item of K/V heads x, x + 8, ... in turn, so its L2
    //    only ever holds one head's K/V segment and all of that head's query
    //    groups reuse it.
    //  * otherwise: grid (8 G ceil(items / 8), BH); XCD x takes the contiguous
    //    slice [x*per, (x+1)*per) of each head's items.
    int cx = blockIdx.x >> 3;
    jq = cx % g.G;
    cx /= g.G;
    bh = A.heads_per_xcd ? blockIdx.y * 8 + (blockIdx.x & 7) : blockIdx.y;
    const int32_t* ends = A.nchunks + bh * kItemClasses;
    const int c0 = A.cls > 0 ? ends[A.cls - 1] : 0, nch = ends[A.cls] - c0;
    if (!A.heads_per_xcd) {
      const int per = (nch + 7) / 8;
      cx = cx < per ? (int)(blockIdx.x & 7) * per + cx : nch;
    }
    if (cx >= nch) return;
    cx += c0;
    const int4 c = A.chunks[(size_t)bh * g.nchunk_max + cx];
    w.a = c.x;
    w.rbase = A.offq[(size_t)bh * (g.CQt + 1) + c.x] + c.y;
    w.nrows = c.z;
    w.nkeys = c.w;
    w.k0 = 0;
    if (w.nrows <= 0 || w.nkeys <= 0) return;  // every routed query group has keys
    Kp = A.kperm + (size_t)bh * g.N * D;
    Vp = A.vperm + (size_t)bh * g.N * D;
  } else {
    bh = blockIdx.z % g.BH;
    jq = blockIdx.z / g.BH;
    if (!get_work<MODE>(g, A, bh, w)) return;
    const int64_t base = kv_base(g, bh);
    Kp = (const uint16_t*)A.k + base;
    Vp = (const uint16_t*)A.v + base;
  }
  const int64_t ksn = (MODE == MODE_SPARSE) ? D : g.sn;  // row stride of Kp/Vp
  const int bq = jq * g.BH + bh;  // entry of the attend outputs
  const uint16_t* Qp = (const uint16_t*)A.q + q_base(g, bh, jq);

  // query row of this lane and its B operands
  const int qr = wv * 32 + n;
  const bool qvalid = qr < w.nrows;
  const int qrow = qvalid ? row_of<MODE>(g, A, bh, w, qr) : 0;
  bf16x8 qreg[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    uint4 u = make_uint4(0, 0, 0, 0);
    if (qvalid) u = *(const uint4*)(Qp + (int64_t)qrow * g.sn + ks * 16 + h * 8);
    qreg[ks] = __builtin_bit_cast(bf16x8, u);
  }
  const bool wave_active = wv * 32 < w.nrows;

  // routed ranges of the query group (positions in the group-major K/V);
  // never read through generic pointers (flat accesses would make the
  // compiler wait for the in-flight tile loads).  Only the ranges meeting the
  // key segment [seg_lo, seg_hi) are walked, each clipped to it: ranges are
  // sorted and disjoint, so they are the run [j0, j0 + nseg) and their
  // clipped lengths sum to this launch's keys; the first MAXR of the run are
  // staged in LDS.
  typedef const __attribute__((address_space(1))) int* gptr_int;
  gptr_int grng = nullptr;
  int nr = 0, j0 = 0, nseg = 0;
  __shared__ int sred[NW][3];
  if (MODE == MODE_SPARSE) {
    grng = (gptr_int)(A.rng + ((size_t)bh * g.CQt + w.a) * g.CKt);
    nr = A.rng_cnt[(size_t)bh * g.CQt + w.a];
    int below = 0, before_end = 0, keys = 0;
    for (int i = tid; i < nr; i += NT) {
      const int2 r = make_int2(grng[2 * i], grng[2 * i + 1]);
      below += (r.x + r.y <= A.seg_lo);
      before_end += (r.x < A.seg_hi);
      keys += max(min(r.x + r.y, A.seg_hi) - max(r.x, A.seg_lo), 0);
    }
    below = wave_sum_i(below);
    before_end = wave_sum_i(before_end);
    keys = wave_sum_i(keys);
    if (lane == 0) {
      sred[wv][0] = below;
      sred[wv][1] = before_end;
      sred[wv][2] = keys;
    }
    __syncthreads();
    w.nkeys = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      j0 += sred[v][0];
      nseg += sred[v][1];
      w.nkeys += sred[v][2];
    }
    nseg -= j0;
    for (int i = tid; i < min(nseg, MAXR); i += NT)
      srng[i] = make_int2(grng[2 * (j0 + i)], grng[2 * (j0 + i) + 1]);
    __syncthreads();
  }
  auto range_at = [&](int j) -> int2 {  // clipped range j of the segment's run
    const int jj = j0 + j;
    const int2 r = (j < MAXR) ? srng[j] : make_int2(grng[2 * jj], grng[2 * jj + 1]);
    const int lo = max(r.x, A.seg_lo), hi = min(r.x + r.y, A.seg_hi);
    return make_int2(lo, hi - lo);
  };
  const int safe_pos = (MODE == MODE_SPARSE) ? (nseg > 0 ? range_at(0).x : 0) : w.k0;
  // Each of lanes 0-31 of wave 0 walks the ranges for key tid of every tile
  // with a cursor that only moves forward.  The cursor's range and the one
  // after it are kept in registers, so a tile costs no dependent LDS read
  // unless its key crosses two range boundaries; the read of the new next
  // range is only waited for at the following crossing.
  KeyCursor cur{0, 0};
  int2 cr = make_int2(0, 0), nx = make_int2(0, 0);
  if (MODE == MODE_SPARSE && tid < KT && nseg > 0) {
    cr = range_at(0);
    nx = nseg > 1 ? range_at(1) : make_int2(0, 0x7fffffff);
  }
  auto fill_pos = [&](int tt) {  // key positions of tile tt -> ring slot tt % 3
    if (tid < KT) {
      const int f = tt * KT + tid;
      int pos = safe_pos;
      if (f < w.nkeys) {
        if (MODE == MODE_SPARSE) {
          while (f >= cur.cum + cr.y) {  // f < nkeys: the run ends after f
            cur.cum += cr.y;
            ++cur.j;
            cr = nx;
            nx = cur.j + 1 < nseg ? range_at(cur.j + 1) : make_int2(0, 0x7fffffff);
          }
          pos = cr.x + (f - cur.cum);
        } else {
          pos = w.k0 + f;
        }
      }
      spos[tt % 3][tid] = pos;
    }
  };
  // LDS byte address of tiles[0] (uniform); the K buffer is there, V
  // buffer b at +(1+b)*KT*D*2
  const uint32_t lds_tiles = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)&tiles[0][0]);
  const uint32_t row_bytes = (uint32_t)(ksn * 2);
  // the copies of tile tt of one tensor into the buffer at dst
  auto issue = [&](int tt, const uint16_t* src, uint32_t dst) {
    // all positions first (one LDS wait), then the copies
    // Two waves: keys at a constant distance from the lane's first, so that one
    // register addresses the positions (with keys from the scalar wave index
    // the loop held an address per copy and read them one by one: 28.45 -> 28.27
    // ms for the sparse attention of 24 heads of 75,600 rows).  Three waves,
    // whose last round is partial, are faster by the wave index (with classes
    // 25.3 ms, this way 25.7).
    uint32_t voff[LPT];
#pragma unroll
    for (int u = 0; u < LPT; ++u) {
      const int inst = u * NW + wv;  // past NCP (uniform) in a last partial round
      const int s = (inst < NCP ? inst : 0) * 64 + lane;
      const int key = NW == 2 ? tid / CH + u * (NT / CH) : s / CH;
      const int p = NW == 2 ? tid % CH : s % CH;
      const int c8 = p ^ kv_swz<D>(key);
      voff[u] = (uint32_t)spos[tt % 3][key] * row_bytes + (uint32_t)(c8 * 16);
    }
#pragma unroll
    for (int u = 0; u < LPT; ++u)
      if (NCP % NW == 0 || u * NW + wv < NCP) g2lds16s(src, voff[u], dst + (uint32_t)((u * NW + wv) * 1024));
  };
  const uint32_t kdst = lds_tiles;
  auto vdst = [&](int b) { return lds_tiles + (uint32_t)((1 + b) * KT * D * 2); };

  const float sl2 = 1.4426950408889634f / sqrtf((float)D);
  float m_run = kNoMax, l_run = 0.f;
  f32x16 O[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
  if (MODE == MODE_SPARSE && !A.seg_first && qvalid) {
    // resume the running state left by the previous key segment
    const float* src = A.osp + ((size_t)bq * g.N + qrow) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const float4 v4 = *(const float4*)(src + db * 32 + i4 * 8 + h * 4);
        O[db][i4 * 4] = v4.x;
        O[db][i4 * 4 + 1] = v4.y;
        O[db][i4 * 4 + 2] = v4.z;
        O[db][i4 * 4 + 3] = v4.w;
      }
    const float* ml = A.mlst + ((size_t)bq * g.N + qrow) * 4;
    m_run = ml[0];
    l_run = ml[1 + h];
  }
  // s_waitcnt immediate (gfx9 encoding) waiting for lgkmcnt(0) only
  constexpr int kWaitLgkm0 = 0xC07F;
  // The Q operands and any resumed state were loaded into registers with
  // ordinary global loads.  Wait for them here, once: otherwise the
  // compiler's wait before their first use inside the loop would be a
  // vmcnt(0) on every iteration, which also waits for the next tile's loads.
  __builtin_amdgcn_s_waitcnt(0x3f70);

  const int ntile = (w.nkeys + KT - 1) / KT;
  // One step computes tile t (K in the K buffer, V in V buffer vb).  Barrier
  // A: every wave's copies of tile t have landed and every wave is done with
  // tile t-1, so V(t+1) is copied into the other V buffer; the scores read
  // the K buffer; barrier B: every wave is done with K(t), so K(t+1) is
  // copied into it while the softmax and PV of tile t run.  Plain s_barrier
  // (no fence): ordering is explicit, each wave waits for its own copies and
  // LDS accesses before a barrier.
  auto step = [&](int t, int vb) {
    const uint16_t* kt = tiles[K2 && vb ? 3 : 0];
    const uint16_t* vt = tiles[1 + vb];
    // positions first: the range walk may read global memory, and the wait
    // the compiler puts before its use also covers the copies issued
    // earlier, which are awaited next anyway
    if (t + 2 < ntile) fill_pos(t + 2);
    __builtin_amdgcn_s_waitcnt(0x3f70);  // vmcnt(0): K(t) and V(t) have landed
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    if (K2 && t + 1 < ntile) issue(t + 1, Kp, vb ? kdst : kdst + (uint32_t)(3 * KT * D * 2));
    if (t + 1 < ntile) issue(t + 1, Vp, vdst(1 - vb));
    f32x16 S;
    if (wave_active) {
#pragma unroll
      for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int c8 = (2 * ks + h) ^ kv_swz<D>(n);
        const bf16x8 kf = __builtin_bit_cast(bf16x8, *(const uint4*)(kt + (n * CH + c8) * 8));
        S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qreg[ks], S, 0, 0, 0);
      }
    }
    if (!K2) {
      // every wave's K reads are done before K(t+1) overwrites the buffer
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      __builtin_amdgcn_s_barrier();
      if (t + 1 < ntile) issue(t + 1, Kp, kdst);
    }
    if (wave_active) {
      // register i holds key (i/4)*8 + h*4 + i%4 of the tile
      float mt = -INFINITY;
      if ((t + 1) * KT > w.nkeys) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = t * KT + (i >> 2) * 8 + h * 4 + (i & 3);
          if (key >= w.nkeys) S[i] = -INFINITY;
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) mt = fmaxf(mt, S[i]);
      mt = pair_max(mt) * sl2;
      const bool need = mt > m_run + 8.f;
      if (__ballot(need)) {
        const float m_new = need ? mt : m_run;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) O[db][i] *= alpha;
      }
      // probabilities rounded to bf16 for the PV product; the row sum is
      // taken over the same rounded values (two per dot2), so O and l share
      // one set of weights
      bf16x8 P[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          P[c][e] = (__bf16)__builtin_amdgcn_exp2f(fmaf(S[c * 8 + e], sl2, -m_run));
      typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
      const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const bf16x2 pp = {P[c][e], P[c][e + 1]};
          l_run = __builtin_amdgcn_fdot2_f32_bf16(pp, one2, l_run, false);
        }
      // V^T fragments (transposing reads), after the scores are consumed so
      // that the two never hold registers together
      const int grp = lane >> 4, gl = lane & 15;
      bf16x8 vf[NDB][2];
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int dv = db * 32 + 16 * (grp & 1) + 4 * (gl & 3);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int key0 = 16 * c + 4 * h + (gl >> 2);
          const int key1 = key0 + 8;
          const v4i16 lo = lds_read_tr16(vt + (key0 * CH + ((dv >> 3) ^ kv_swz<D>(key0))) * 8 + (dv & 7));
          const v4i16 hi = lds_read_tr16(vt + (key1 * CH + ((dv >> 3) ^ kv_swz<D>(key1))) * 8 + (dv & 7));
          vf[db][c] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
      }
      // O^T += V^T P^T over the two 16-key chunks
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][c], P[c], O[db], 0, 0, 0);
    }
  };
  if (ntile > 0) fill_pos(0);
  if (ntile > 1) fill_pos(1);
  __syncthreads();
  if (ntile > 0) {
    issue(0, Kp, kdst);
    issue(0, Vp, vdst(0));
  }
  for (int t = 0; t < ntile; t += 2) {
    step(t, 0);
    if (t + 1 < ntile) step(t + 1, 1);
  }
  // every copy has landed before the block can end
  __builtin_amdgcn_s_waitcnt(0x3f70);
  if (!qvalid) return;
  const float l_tot = pair_sum(l_run);
  if (MODE == MODE_PROBE) {
    float* dst = A.part + (((size_t)bq * g.M + w.tile * 64 + qr) * g.nsplit + w.split) * (D + 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int dv = db * 32 + i4 * 8 + h * 4;
        *(f32x4_u*)(dst + dv) =
            f32x4_u{O[db][i4 * 4], O[db][i4 * 4 + 1], O[db][i4 * 4 + 2], O[db][i4 * 4 + 3]};
      }
    if (h == 0) {
      dst[D] = m_run;
      dst[D + 1] = l_tot;
    }
  } else {
    const float inv = 1.f / l_tot;
    if (!A.seg_last) {
      // hand the running state to the next key segment
      float* dst = A.osp + ((size_t)bq * g.N + qrow) * D;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int dv = db * 32 + i4 * 8 + h * 4;
          *(float4*)(dst + dv) =
              make_float4(O[db][i4 * 4], O[db][i4 * 4 + 1], O[db][i4 * 4 + 2], O[db][i4 * 4 + 3]);
        }
      float* ml = A.mlst + ((size_t)bq * g.N + qrow) * 4;
      if (h == 0) ml[0] = m_run;
      ml[1 + h] = l_run;
    } else {
      float* dst = A.osp + ((size_t)bq * g.N + qrow) * D;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int dv = db * 32 + i4 * 8 + h * 4;
          *(float4*)(dst + dv) = make_float4(O[db][i4 * 4] * inv, O[db][i4 * 4 + 1] * inv,
                                             O[db][i4 * 4 + 2] * inv, O[db][i4 * 4 + 3] * inv);
        }
    }
  }
}

// Dense flash attention, bf16 MFMA, fp32 accumulation: the tiles, swizzle and
// transposed products of k_attn_mfma for contiguous keys.  NW waves of 32 query
// rows share each 32-key tile, so the copies per row shrink with NW and their
// addresses are a uniform base plus per-lane constants.  The scores of tile
// t + 1 are formed next to the exponentials of tile t (an MFMA leaves the issue
// slots of about six VALU instructions), K and V are double-buffered and the
// copies of K(t + 2) and V(t + 1) go out at the start of step t, with one
// barrier per step.
// 24 heads of 17,160 rows at d = 128: 4.12 -> 3.52 ms (1.03 PFLOP/s); 12 of
// 4,335 at d = 64: 107 -> 92 us; 2 of 1,275 at d = 128: 35 -> 30 us.  What is
// left is the matrix pipes' sustained rate on such data: without any copies
// 3.04 ms, without copies, LDS reads and exponentials 2.9 ms, which is 1.25
// PFLOP/s; rings of three buffers changed nothing.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_dense(Geom g, AttnArgs A) {
  constexpr int KT = 32, CH = D / 8, NKS = D / 16, NDB = D / 32;
  constexpr int NCP = KT * CH / 64, CPW = NCP / NW;  // 1 KB copies per tensor and tile, per wave
  constexpr uint32_t TB = KT * D * 2;                // bytes of a tile
  static_assert(NCP % NW == 0, "copies divide among the waves");
  __shared__ __attribute__((aligned(1024))) uint16_t kt[2][KT * D], vt[2][KT * D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  // Block order: with a multiple of 8 query heads, XCD x takes heads x, x + 8,
  // ... so that its L2 holds one head's keys; otherwise blocks go head by head.
  const int tiles = (g.N + 32 * NW - 1) / (32 * NW), heads = g.BH * g.G;
  int bq, tile;
  if (heads % 8 == 0) {
    const int b = blockIdx.x >> 3;
    bq = (b / tiles) * 8 + (blockIdx.x & 7);
    tile = b % tiles;
  } else {
    bq = blockIdx.x / tiles;
    tile = blockIdx.x % tiles;
  }
  // query heads of one K/V head follow each other
  const int bh = bq / g.G, jq = bq % g.G;
  const int64_t base = kv_base(g, bh), qbase = q_base(g, bh, jq);
  const unsigned char* Kp = (const unsigned char*)((const uint16_t*)A.k + base);
  const unsigned char* Vp = (const unsigned char*)((const uint16_t*)A.v + base);
  const uint16_t* Qp = (const uint16_t*)A.q + qbase;
  const int qrow = tile * 32 * NW + wv * 32 + n;
  const bool qvalid = qrow < g.N;
  const bool wave_active = tile * 32 * NW + wv * 32 < g.N;
  bf16x8 qreg[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    uint4 u = make_uint4(0, 0, 0, 0);
    if (qvalid) u = *(const uint4*)(Qp + (int64_t)qrow * g.sn + ks * 16 + h * 8);
    qreg[ks] = __builtin_bit_cast(bf16x8, u);
  }
  constexpr int kWaitLgkm0 = 0xC07F, kWaitVm0 = 0x3f70;
  __builtin_amdgcn_s_waitcnt(kWaitVm0);

  const int ntile = (g.N + KT - 1) / KT;
  const uint32_t row_bytes = (uint32_t)(g.sn * 2);
  auto lds_of = [](const void* p) {
    return __builtin_amdgcn_readfirstlane(
        (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)p);
  };
  const uint32_t kdst = lds_of(&kt[0][0]), vdst = lds_of(&vt[0][0]);
  // this lane's key and 16-byte chunk of the wave's copies
  int ckey[CPW];
  uint32_t cchunk[CPW], voff[CPW];
#pragma unroll
  for (int u = 0; u < CPW; ++u) {
    const int s = (u * NW + wv) * 64 + lane;
    ckey[u] = s / CH;
    cchunk[u] = (uint32_t)(((s % CH) ^ kv_swz<D>(ckey[u])) * 16);
    voff[u] = (uint32_t)ckey[u] * row_bytes + cchunk[u];
  }
  auto issue = [&](int t, const unsigned char* src, uint32_t dst) {
    const unsigned char* p = src + (size_t)t * KT * row_bytes;
    const int left = g.N - t * KT;  // keys past the end repeat the last one
    if (left >= KT) {
#pragma unroll
      for (int u = 0; u < CPW; ++u) g2lds16s(p, voff[u], dst + (uint32_t)((u * NW + wv) * 1024));
    } else {
#pragma unroll
      for (int u = 0; u < CPW; ++u)
        g2lds16s(p, (uint32_t)min(ckey[u], left - 1) * row_bytes + cchunk[u],
                 dst + (uint32_t)((u * NW + wv) * 1024));
    }
  };
  const float sl2 = 1.4426950408889634f / sqrtf((float)D);
  float m_run = kNoMax, l_run = 0.f, mt = 0.f;
  f32x16 O[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
  auto scores = [&](f32x16& S, int b) {
    bf16x8 kf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      kf[ks] = __builtin_bit_cast(bf16x8, *(const uint4*)(kt[b] + (n * CH + ((2 * ks + h) ^ kv_swz<D>(n))) * 8));
#pragma unroll
    for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qreg[ks], S, 0, 0, 0);
  };
  // maximum of this lane's scores of tile t, keys past the end masked
  auto tile_max = [&](f32x16& S, int t) {
    const int left = g.N - t * KT;
    if (left < KT) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if ((i >> 2) * 8 + h * 4 + (i & 3) >= left) S[i] = -INFINITY;
    }
    mt = fmaxf(fmaxf(S[0], S[1]), S[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) mt = fmaxf(fmaxf(mt, S[i]), S[i + 1]);
    mt = fmaxf(mt, S[15]);
  };
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
  // step t: softmax and PV of tile t (scores Sc, buffer b), scores Sn of
  // tile t + 1 (past the last tile on whatever the buffer holds, unused)
  auto step = [&](int t, int b, f32x16& Sc, f32x16& Sn) {
    __builtin_amdgcn_s_waitcnt(kWaitVm0);  // this wave's copies of K(t + 1), V(t)
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    // every wave is done with K(t) and V(t - 1)
    if (t + 2 < ntile) issue(t + 2, Kp, kdst + (uint32_t)b * TB);
    if (t + 1 < ntile) issue(t + 1, Vp, vdst + (uint32_t)(1 - b) * TB);
    if (!wave_active) return;
    const float mp = pair_max(mt) * sl2;
    const bool need = mp > m_run + 8.f;
    if (__ballot(need)) {
      const float m_new = need ? mp : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[db][i] *= alpha;
    }
    scores(Sn, 1 - b);
    // probabilities rounded to bf16 for the PV product; the row sum is taken
    // over the same rounded values (two per dot2), so O and l share one set
    // of weights
    bf16x8 P[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        P[c][e] = (__bf16)__builtin_amdgcn_exp2f(fmaf(Sc[c * 8 + e], sl2, -m_run));
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 pp = {P[c][e], P[c][e + 1]};
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pp, one2, l_run, false);
      }
    const int grp = lane >> 4, gl = lane & 15;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int dv = db * 32 + 16 * (grp & 1) + 4 * (gl & 3);
        const int key0 = 16 * c + 4 * h + (gl >> 2);
        const int key1 = key0 + 8;
        const v4i16 lo = lds_read_tr16(vt[b] + (key0 * CH + ((dv >> 3) ^ kv_swz<D>(key0))) * 8 + (dv & 7));
        const v4i16 hi = lds_read_tr16(vt[b] + (key1 * CH + ((dv >> 3) ^ kv_swz<D>(key1))) * 8 + (dv & 7));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, P[c], O[db], 0, 0, 0);
      }
    tile_max(Sn, t + 1);
  };
  f32x16 S0, S1;
  issue(0, Kp, kdst);
  issue(0, Vp, vdst);
  if (ntile > 1) issue(1, Kp, kdst + TB);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __builtin_amdgcn_s_barrier();
  scores(S0, 0);
  tile_max(S0, 0);
  for (int t = 0; t < ntile; t += 2) {
    step(t, 0, S0, S1);
    if (t + 1 < ntile) step(t + 1, 1, S1, S0);
  }
  // every copy has landed before the block can end
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  if (!qvalid) return;
  const float inv = 1.f / pair_sum(l_run);
  uint16_t* dst = (uint16_t*)A.out + qbase + (int64_t)qrow * g.sn;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const int dv = db * 32 + i4 * 8 + h * 4;
      uint32_t o[2];
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const uint16_t lo = __builtin_bit_cast(uint16_t, (__bf16)(O[db][i4 * 4 + e] * inv));
        const uint16_t hi = __builtin_bit_cast(uint16_t, (__bf16)(O[db][i4 * 4 + e + 1] * inv));
        o[e >> 1] = (uint32_t)lo | ((uint32_t)hi << 16);
      }
      *(u32x2_u*)(dst + dv) = u32x2_u{o[0], o[1]};
    }
}

// Group-major copies of K and V (Sec. 4.3): position p of head bh holds row
// perm_kv[p].  Each row is moved as 16-byte pieces.
template <int D>
__global__ __launch_bounds__(256) void k_permute_kv(Geom g, const void* k, const void* v,
                                                    const int32_t* permk, uint16_t* kperm,
                                                    uint16_t* vperm) {
  constexpr int CH = D / 8, RPB = 256 / CH;
  const int bh = blockIdx.y, tid = threadIdx.x;
  const int p = blockIdx.x * RPB + tid / CH, c = tid % CH;
  if (p >= g.N) return;
  const int64_t base = kv_base(g, bh);
  const int src = permk[(size_t)bh * g.N + p];
  const uint4 kv = *(const uint4*)((const uint16_t*)k + base + (int64_t)src * g.sn + c * 8);
  const uint4 vv = *(const uint4*)((const uint16_t*)v + base + (int64_t)src * g.sn + c * 8);
  *(uint4*)(kperm + ((size_t)bh * g.N + p) * D + c * 8) = kv;
  *(uint4*)(vperm + ((size_t)bh * g.N + p) * D + c * 8) = vv;
}

// fp32 variant on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32, fp32
// products and accumulation: 157 TFLOP/s against 79 for unpacked vector FMAs).
// A block of 4 waves owns up to 64 query rows (32 when the row tile is 32 or
// the chunk is short): with 2 sets of 32 rows two waves share each set and
// halve its keys, with one set four waves quarter them, every wave taking
// each nparts-th 32-key tile; the partial (m, l, O) merge through LDS at the
// end.  As in the bf16 kernel the scores are formed transposed, S^T = K Q^T,
// so a lane's scores belong to one query and the probabilities feed
// O^T += V^T P^T from registers.
//  * Both contractions may take their terms in any order: lane (n, h) holds
//    dims 8j + 4h + 0..3 of query n, so a key operand is one 16-byte load per
//    four MFMAs; PV step i contracts the keys of score register i of both
//    halves, and V^T row m of block db is value channel m * NDB + db, so one
//    16-byte (D = 64: 8-byte) load of a value row serves every block.
//  * Operands go straight from global memory to registers: a load feeds four
//    64-cycle MFMAs, so the CU asks for 16 B/clk of K and V, far below what L1
//    and L2 deliver, and there is no LDS tile, no barrier and no transposition.
//    Loads run half a tile (2048 matrix cycles at D = 128) ahead.
// One thread per row on vector FMAs in one-wave blocks, with K/V tiles staged
// through LDS by scalar loads, took 9.97 ms for dense attention of 8 heads of
// 2,442 rows at d = 64 (1.2 TFLOP/s); this kernel 0.204 ms (60 TFLOP/s: its
// 312 blocks all run at once, 56 of the 256 CUs holding two, so that at most 61%
// of the chip works, and loads are exposed).
template <int D, int MODE>
__global__ __launch_bounds__(256, 2) void k_attn_f32(Geom g, AttnArgs A) {
  constexpr int KT = 32, NQ = D / 8, HQ = NQ / 2, NDB = D / 32;
  constexpr int NREG = 16 * NDB;
  typedef float fv __attribute__((ext_vector_type(NDB), aligned(4)));
  __shared__ float red[3][NREG + 2][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  // block's query head j of K/V head bh; attend outputs are entry bq
  const int bq = (MODE == MODE_SPARSE) ? blockIdx.y : blockIdx.z;
  const int bh = bq % g.BH, jq = bq / g.BH;
  Work1 w;
  if (!get_work<MODE>(g, A, bh, w)) return;
  const int64_t base = kv_base(g, bh), qbase = q_base(g, bh, jq);
  const float* Kp = (const float*)A.k + base;
  const float* Vp = (const float*)A.v + base;
  const float* Qp = (const float*)A.q + qbase;
  const int nsets = w.nrows > 32 ? 2 : 1, nparts = 4 / nsets;
  const int set = nsets == 2 ? wv & 1 : 0, part = nsets == 2 ? wv >> 1 : wv;
  const int qr = set * 32 + n;
  const bool qvalid = qr < w.nrows;
  const int qrow = row_of<MODE>(g, A, bh, w, qvalid ? qr : 0);
  f32x4_u q4[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) q4[j] = *(const f32x4_u*)(Qp + (int64_t)qrow * g.sn + 8 * j + 4 * h);
  const int2* rg = nullptr;
  int nr = 0;
  if (MODE == MODE_SPARSE) {
    rg = A.rng + ((size_t)bh * g.CQt + w.a) * g.CKt;
    nr = A.rng_cnt[(size_t)bh * g.CQt + w.a];
  }
  KeyCursor cur{0, 0};
  // scores are scaled into base 2 with the softmax scale's own rounding
  const float scale = 1.f / sqrtf((float)D);
  const float l2e = 1.4426950408889634f;
  float m_run = kNoMax, l_run = 0.f;
  f32x16 O[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
  const int ntile = (w.nkeys + KT - 1) / KT;
  // row of key n of tile t; keys past the end repeat the last one and are masked
  auto tile_row = [&](int t) {
    return key_row<MODE>(g, A, bh, w, min(t * KT + n, w.nkeys - 1), cur, rg, nr);
  };
  f32x4_u ka[HQ], kb[HQ];
  fv va[8], vb[8];
  auto load_k = [&](f32x4_u* dst, int row, int half) {
    const float* src = Kp + (int64_t)row * g.sn + 4 * h + half * (HQ * 8);
#pragma unroll
    for (int j = 0; j < HQ; ++j) dst[j] = *(const f32x4_u*)(src + 8 * j);
  };
  auto load_v = [&](fv* dst, int row, int half) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = half * 8 + i;
      const int r = __shfl(row, (e >> 2) * 8 + 4 * h + (e & 3));
      dst[i] = *(const fv*)(Vp + (int64_t)r * g.sn + n * NDB);
    }
  };
  f32x16 S;
  auto scores = [&](const f32x4_u* kk, int half) {
#pragma unroll
    for (int j = 0; j < HQ; ++j) {
      const f32x4_u q = q4[half * HQ + j];
      S = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[j].x, q.x, S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[j].y, q.y, S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[j].z, q.z, S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[j].w, q.w, S, 0, 0, 0);
    }
  };
  auto pv = [&](const fv* vv, int half) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int db = 0; db < NDB; ++db)
        O[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[i][db], S[half * 8 + i], O[db], 0, 0, 0);
  };
  int row = 0, nrow = 0;
  if (part < ntile) {
    row = tile_row(part);
    load_k(ka, row, 0);
  }
  for (int t = part; t < ntile; t += nparts) {
    load_k(kb, row, 1);
    const bool more = t + nparts < ntile;
    if (more) nrow = tile_row(t + nparts);
#pragma unroll
    for (int i = 0; i < 16; ++i) S[i] = 0.f;
    scores(ka, 0);
    load_v(va, row, 0);
    scores(kb, 1);
    load_v(vb, row, 1);
    const int left = w.nkeys - t * KT;  // valid keys of this tile when below KT
    float mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      S[i] = S[i] * scale * l2e;
      if (left < KT && (i >> 2) * 8 + 4 * h + (i & 3) >= left) S[i] = -INFINITY;
      mt = fmaxf(mt, S[i]);
    }
    mt = pair_max(mt);
    if (__any(mt > m_run)) {
      const float m_new = fmaxf(m_run, mt);
      const float alpha = exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[db][i] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      S[i] = exp2f(S[i] - m_run);
      l_run += S[i];
    }
    if (left < KT) {  // masked keys add nothing, whatever their row holds
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int key = (i >> 2) * 8 + 4 * h + (i & 3);
          if (key >= left) va[i][db] = 0.f;
          if (key + 16 >= left) vb[i][db] = 0.f;
        }
    }
    pv(va, 0);
    if (more) load_k(ka, nrow, 0);
    pv(vb, 1);
    row = nrow;
  }
  float l_tot = pair_sum(l_run);
  // merge the key parts of each row set into part 0
  if (part > 0) {
    float(*dst)[64] = red[nsets == 2 ? set : part - 1];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) dst[db * 16 + i][lane] = O[db][i];
    dst[NREG][lane] = m_run;
    dst[NREG + 1][lane] = l_tot;
  }
  __syncthreads();
  if (part > 0 || !qvalid) return;
  for (int p = 1; p < nparts; ++p) {
    const float(*src)[64] = red[nsets == 2 ? set : p - 1];
    const float mp = src[NREG][lane], lp = src[NREG + 1][lane];
    // a part without a finite score holds (kNoMax, 0, 0)
    const float m_new = fmaxf(m_run, mp);
    const float fa = exp2f(m_run - m_new), fb = exp2f(mp - m_new);
    m_run = m_new;
    l_tot = l_tot * fa + lp * fb;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) O[db][i] = O[db][i] * fa + src[db * 16 + i][lane] * fb;
  }
  float* dst;
  float inv = 1.f;
  if (MODE == MODE_PROBE) {
    dst = A.part + (((size_t)bq * g.M + w.tile * 64 + qr) * g.nsplit + w.split) * (D + 2);
    if (h == 0) {
      dst[D] = m_run;
      dst[D + 1] = l_tot;
    }
  } else {
    dst = (MODE == MODE_SPARSE) ? A.osp + ((size_t)bq * g.N + qrow) * D
                                : (float*)A.out + qbase + (int64_t)qrow * g.sn;
    inv = l_tot;
  }
  // register i of block db: value channel (8 (i / 4) + 4 h + i % 4) NDB + db
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    fv o;
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] = MODE == MODE_PROBE ? O[db][i] : O[db][i] / inv;
    *(fv*)(dst + ((i >> 2) * 8 + 4 * h + (i & 3)) * NDB) = o;
  }
}

// Merge the key splits of the probe rows: O = sum_s o_s 2^(m_s - m) / sum_s l_s 2^(m_s - m).
// Kernels from here on take every query head in one launch: block index
// bq = j * BH + bh is query head j of K/V head bh, whose attend outputs are
// entry bq of the [G][BH] arrays and whose plan is entry bh.
__global__ __launch_bounds__(128) void k_probe_merge(Geom g, const float* part,
                                                     const int32_t* nprobes, float* odp) {
  const int p = blockIdx.x, bq = blockIdx.y, bh = bq % g.BH, c = threadIdx.x;
  if (p >= nprobes[bh] || c >= g.dv) return;
  const int D = g.dv;
  const float* src = part + ((size_t)bq * g.M + p) * g.nsplit * (D + 2);
  // both sweeps keep the split order; unrolled so that their loads overlap
  float m = -INFINITY;
#pragma unroll 8
  for (int s = 0; s < g.nsplit; ++s) m = fmaxf(m, src[(size_t)s * (D + 2) + D]);
  float l = 0.f, o = 0.f;
#pragma unroll 8
  for (int s = 0; s < g.nsplit; ++s) {
    const float* e = src + (size_t)s * (D + 2);
    const float f = exp2f(e[D] - m);
    l += e[D + 1] * f;
    o += e[c] * f;
  }
  odp[((size_t)bq * g.M + p) * D + c] = o / l;
}

static AttnArgs make_args(const Work* w, const void* q, const void* k, const void* v, void* out) {
  AttnArgs a{};
  a.q = q;
  a.k = k;
  a.v = v;
  a.out = out;
  if (w) {
    a.osp = w->osp;
    a.part = w->part;
    a.chunks = w->chunks;
    a.nchunks = w->nchunks;
    a.permq = w->permq;
    a.offq = w->offq;
    a.permk = w->permk;
    a.rng = w->rng;
    a.rng_cnt = w->rng_cnt;
    a.probes = w->probes;
    a.nprobes = w->nprobes;
    a.kperm = w->kperm;
    a.vperm = w->vperm;
    a.mlst = w->mlst;
  }
  a.seg_lo = 0;
  a.seg_hi = 0x7fffffff;
  a.seg_first = 1;
  a.seg_last = 1;
  return a;
}

template <int D>
static void attend_d(const Geom& g, const Work& w, const void* q, const void* k, const void* v,
                     void* out, hipStream_t s, hipEvent_t* ev) {
  // every kernel takes all G * BH query heads in one launch (the attend
  // outputs are [G][BH] arrays)
  const int BQ = g.BH * g.G;
  const AttnArgs a = make_args(&w, q, k, v, out);
  if (g.bf16) {
    constexpr int CH = D / 8;
    k_permute_kv<D><<<dim3((g.N + 256 / CH - 1) / (256 / CH), g.BH), 256, 0, s>>>(
        g, k, v, w.permk, w.kperm, w.vperm);
  }
  if (ev) (void)hipEventRecord(ev[0], s);
  if (g.bf16) {
    // one launch per key segment, so that all blocks in flight read the same
    // slice of K/V and it stays in L2
    for (int sg = 0; sg < g.nseg; ++sg) {
      AttnArgs as = a;
      as.seg_lo = (int)((int64_t)g.N * sg / g.nseg);
      as.seg_hi = (int)((int64_t)g.N * (sg + 1) / g.nseg);
      as.seg_first = sg == 0;
      as.seg_last = sg == g.nseg - 1;
      as.heads_per_xcd = g.BH % 8 == 0;
      // one launch per class of work items; an item of 3 sets has at least
      // 65 rows
      auto launch = [&](auto nw, int cls, int most) {
        constexpr int NW = decltype(nw)::value;
        as.cls = cls;
        const dim3 grid = as.heads_per_xcd ? dim3(8 * g.G * most, g.BH / 8)
                                           : dim3(8 * g.G * ((most + 7) / 8), g.BH);
        if (most > 0) k_attn_mfma<D, MODE_SPARSE, NW><<<grid, 64 * NW, 0, s>>>(g, as);
      };
      if (g.classes) launch(std::integral_constant<int, 3>{}, 0, g.N / 65);
      launch(std::integral_constant<int, 2>{}, 1, g.nchunk_max);
    }
  } else {
    k_attn_f32<D, MODE_SPARSE><<<dim3(g.nchunk_max, BQ), 256, 0, s>>>(g, a);
  }
  if (ev) (void)hipEventRecord(ev[1], s);
  if (g.M > 0) {
    const dim3 gp((g.M + 63) / 64, g.nsplit, BQ);
    if (g.bf16)
      k_attn_mfma<D, MODE_PROBE><<<gp, 128, 0, s>>>(g, a);
    else
      k_attn_f32<D, MODE_PROBE><<<gp, 256, 0, s>>>(g, a);
    k_probe_merge<<<dim3(g.M, BQ), 128, 0, s>>>(g, w.part, w.nprobes, w.odp);
  }
  if (ev) (void)hipEventRecord(ev[2], s);
  launch_fit_correct(g, w, out, s, ev);
}

void launch_attend(const Geom& g, const Work& w, const void* q, const void* k, const void* v,
                   void* out, hipStream_t s, hipEvent_t* ev) {
  if (g.d == 64)
    attend_d<64>(g, w, q, k, v, out, s, ev);
  else
    attend_d<128>(g, w, q, k, v, out, s, ev);
}

template <int D>
static void dense_d(const Geom& g, const AttnArgs& a, hipStream_t s) {
  const int tiles = (g.N + 63) / 64;
  if (!g.bf16) {
    k_attn_f32<D, MODE_DENSE><<<dim3(tiles, 1, g.BH * g.G), 256, 0, s>>>(g, a);
    return;
  }
  // Four waves share a tile's copies when such blocks fill the chip twice
  // over (24 heads of 17,160 rows: 3.52 ms, with two waves 3.91); shorter
  // launches spread over twice the blocks (2 heads of 1,275 rows: 29.7 us,
  // with four waves 31.2; 12 of 4,335 at d = 64: 92 us either way), and so do
  // heads of one or three 64-row tiles, half or a quarter of whose 128-row
  // blocks would be padding (d = 128, two waves and four: 2,400 heads of 33
  // rows 22.3 and 27.1 us, 600 of 130 23.7 and 32.0, 1,200 of 192 51.6 and
  // 61.3; with five tiles either may win: 200 of 300 20.6 and 26.8, 768 of 300
  // 72.6 and 68.0).
  const int64_t heads = (int64_t)g.BH * g.G, blocks4 = (g.N + 127) / 128 * heads;
  if (blocks4 >= 512 && tiles != 1 && tiles != 3)
    k_attn_dense<D, 4><<<(unsigned)blocks4, 256, 0, s>>>(g, a);
  else
    k_attn_dense<D, 2><<<(unsigned)(tiles * heads), 128, 0, s>>>(g, a);
}

void launch_dense(const Geom& g, const void* q, const void* k, const void* v, void* out,
                  float* part, hipStream_t s) {
  (void)part;
  const AttnArgs a = make_args(nullptr, q, k, v, out);
  if (g.d == 64)
    dense_d<64>(g, a, s);
  else
    dense_d<128>(g, a, s);
}

}  // namespace sparsepr
