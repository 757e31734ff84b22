// conv_split.hip -- float32 3x3 convolution stage (stride 1, zero padding
// outside the image, folded batch-norm scale/bias, activation, optional fused
// 2x2/2 max-pool) on the bf16 matrix cores: every float32 operand is split
// exactly into three bf16 parts, 2^24 x = x0 + x1 + x2 (8 significant bits
// each, each part the nearest to what is left), and a product is the sum of six
// part products: x0 w0, x0 w1, x1 w0, x1 w1, x0 w2, x2 w0, each exact in
// float32.
//
// Why: the fp32 MFMA runs at 1/16 of the bf16 rate (157 against 2517 TFLOP/s
// dense), so six bf16 MFMAs take 3/8 of the time of the fp32 ones they
// replace.  Precision: x0 w0 is summed in one accumulator (one rounding per
// 32 products instead of one per product), the five small terms in another,
// added at the end.  Dropped are x1 w2, x2 w1 and x2 w2: |x1| <= 2^-8 |x| and
// |x2| <= 2^-17 |x|, so they are at most 2^-24 (1 + 2^-9) of a product, of
// either sign (rms 5.5e-9 of a product); parts cut off instead of rounded
// would drop up to 2^-21, always towards zero.  The factor 2^24 keeps the parts
// of every float32, the smallest subnormal's too, clear of the bf16 subnormals:
// without it parts fall below the smallest bf16 from operands of 2^-110 down.
// Relative error of a layer against 64-bit sums (leaky activations), K = 288,
// 1152 and 4608: 1.1e-7, 2.1e-7 and 4.1e-7 (the fp32 MFMA chain 2.9e-7, 5.9e-7
// and 1.2e-6).  The factor costs one multiplication a value: 0.5 to 1.5 % of the
// time of float32 networks.
//
// What the split cannot carry: infinities and NaN (their parts are not sums),
// operands from 2^104 and sums of products from 2^80 up (2^48 times that is
// past the largest float).  Sums that come out not finite are computed again in
// plain float32, on the fp32 MFMA with operands straight from memory, by their
// whole wave: one such pixel in an early layer reaches all waves of the later
// ones, so their time has to stay that of a convolution.
// 3x3 512->512 on 26x26 with a NaN in every window takes 156 us (60 without), and
// 4984 us with one output after the other on the vector ALUs.
//
// Structure: a workgroup owns a BR x BC block of conv outputs of one tile and
// BN output channels.  K runs over 32-channel chunks and, in each, the three
// filter rows ky; a step is one (chunk, ky): three taps.  Per chunk the
// (BR+2) x (BC+2) input patch is held in LDS as three planes of 64-byte rows
// (the layout of conv_patch.hip), and per step the three taps' BN weight rows
// likewise; both are double buffered.  The float32 values come through
// registers (two 16-byte loads per 8 channels), issued two steps ahead, are
// split (6.5 vector instructions per value) and written after the MFMAs of
// the step before theirs: the split of one wave runs while the other wave of
// its SIMD has the matrix core.  Per step and 128 x 64 block: 2304 matrix-core
// cycles per compute unit, ~830 vector cycles, 336 KiB of LDS traffic.
// Measured: see choose_split in run.cpp.
//
// Requires f = 3, c_in % 32 == 0, c_out % 16 == 0, byte offsets below 2^31
// within a frame's source buffer and within the weights (host-checked); a
// fused pool needs even tile origins and extents.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernel_args.h"

namespace mafat {
namespace {

// Two floats to the nearest bf16 (ties to even), packed; and its two values.
__device__ __forceinline__ unsigned near2(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ float lo_of(unsigned p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_of(unsigned p) { return __uint_as_float(p & 0xffff0000u); }

// Eight floats -> the three bf16 parts of kSplitScale times them, packed: each
// part the bf16 nearest to what the ones before it leave.  That rest is exact in
// float32, and the third part holds all of the last one.
constexpr float kSplitScale = 0x1p24f;
__device__ __forceinline__ void split8(const u32x4& lo, const u32x4& hi, u32x4 (&out)[3]) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float a = kSplitScale * __uint_as_float(w < 2 ? lo[2 * w] : hi[2 * w - 4]);
    const float b = kSplitScale * __uint_as_float(w < 2 ? lo[2 * w + 1] : hi[2 * w - 3]);
    const unsigned p0 = near2(a, b);
    const float ra = a - lo_of(p0), rb = b - hi_of(p0);
    const unsigned p1 = near2(ra, rb);
    out[0][w] = p0;
    out[1][w] = p1;
    out[2][w] = near2(ra - lo_of(p1), rb - hi_of(p1));
  }
}

template <int BR, int BC, int BM, int BN, int WGM, int WGN, bool POOL>
__global__ __launch_bounds__(64 * WGM * WGN) void conv_split_kernel(const StageArgs a) {
  if (__builtin_expect(blockIdx.y != 0, 0)) {  // the second grid row: carried band copies (row reuse)
    carried_copies();
    return;
  }
  constexpr int NWAVE = WGM * WGN, NTHR = 64 * NWAVE;
  constexpr int WM = BM / WGM, WN = BN / WGN, MT = WM / 16, NT = WN / 16;
  constexpr int PR = BR + 2, PC = BC + 2;
  constexpr int PPX = (PR * PC + 15) / 16 * 16;   // patch pixels, whole 16-row groups
  constexpr int APL = PPX * 64, BPL = 3 * BN * 64;  // bytes of one plane: a chunk's patch, a step's weight rows
  constexpr int ABUF = 3 * APL, BBUF = 3 * BPL;
  constexpr int BOFF = 2 * ABUF;
  constexpr int SINK = 2 * ABUF + 2 * BBUF;  // 16 bytes nothing reads
  constexpr int SMEM = SINK + 16;
  // Load items of a step, 8 channels each: the weights' 3 BN x 4, then a
  // third of the next chunk's patch (whole waves).
  constexpr int NBI = 12 * BN;
  constexpr int NAI = ((PPX * 4 + 2) / 3 + 63) / 64 * 64;
  constexpr int NI = (NBI + NAI + NTHR - 1) / NTHR;  // per thread
  static_assert(MT >= 1 && NT >= 1 && MT * 16 == WM && NT * 16 == WN, "wave tile");
  static_assert(BR * BC <= BM && BR % 2 == 0 && BC % 2 == 0, "block");
  static_assert(SMEM <= 160 * 1024, "LDS");
  __shared__ __align__(1024) unsigned char smem[SMEM];

  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave - wm * WGN;
  const int cin = a.cin, cout = a.cout, nchunk = cin >> 5;
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(a.w, static_cast<unsigned>(cout * 9 * cin * 4));

  KTile tl;
  const BlockPos bp = decode_block(a, &tl);
  const int nbx = (tl.cw + BC - 1) / BC;
  const int bby = div_small(bp.mb, nbx), bbx = bp.mb - bby * nbx;
  const int by0 = tl.cy0 + bby * BR, bx0 = tl.cx0 + bbx * BC;  // block origin (conv outputs)
  const int n0 = bp.nb * BN;
  const float* src = static_cast<const float*>(a.src) + bp.frame * a.src_fstride + tl.src_off;
  float* dst = static_cast<float*>(a.dst) + bp.frame * a.dst_fstride + tl.dst_off;
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(src, static_cast<unsigned>((a.src_fstride - tl.src_off) * 4));
  const auto is_b = [&](int k) { return k * NTHR + wave * 64 < NBI; };
  // Item k of this thread in the job of a step (c, g): byte offset of its 32
  // bytes (chunk 0) and its place in a plane.  Items below NBI are the weights
  // of filter row g; the next NAI bring a third of a patch, so that a chunk's
  // patch is whole one step before its first: g = 1, 2 thirds 0, 1 of chunk
  // c + 1, g = 0 third 2 of chunk c.  Which kind an item is, is the same for a
  // whole wave.  Patch pixels outside the image, outside the tile's source
  // region or past the patch, and weight rows past c_out, get bit 31 (reads as
  // zero); items past both kinds, and patch rows past PPX, go to a sink.
  const int ry0 = max(tl.cy0 - 1, 0), ry1 = min(tl.cy0 + tl.ch + 1, a.in_h);
  const int rx0 = max(tl.cx0 - 1, 0), rx1 = min(tl.cx0 + tl.cw + 1, a.in_w);
  unsigned off[NI][3];
  int place[NI][3];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int e = k * NTHR + tid;
    const int row = e >> 2, kx = row / BN, co = n0 + row - kx * BN;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      if (is_b(k)) {
        off[k][g] = co < cout ? static_cast<unsigned>(((co * 9 + g * 3 + kx) * cin + (e & 3) * 8) * 4) : 0x80000000u;
        place[k][g] = swz(row, e & 3);
      } else {
        const int idx = e - NBI, f = (g + 2) % 3 * NAI + idx, p = f >> 2;
        const int py = p / PC, px = p - py * PC;
        const int iy = by0 - 1 + py, ix = bx0 - 1 + px;
        const bool ok = idx < NAI && p < PR * PC && iy >= ry0 && iy < ry1 && ix >= rx0 && ix < rx1;
        off[k][g] = ok ? static_cast<unsigned>((((iy - tl.sy0) * tl.sw + (ix - tl.sx0)) * cin + (f & 3) * 8) * 4)
                       : 0x80000000u;
        place[k][g] = (idx < NAI && p < PPX) ? p * 64 + (((f & 3) ^ patch_key(py)) << 4) : -1;
      }
    }
  }

  // Fragment places as in conv_patch.hip.
  const int q = lane >> 4;
  int pb[MT], kq3[MT][3];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int r = wm * WM + i * 16 + (lane & 15);
    r = (r < BR * BC) ? r : (((r ^ 12) < BR * BC) ? (r ^ 12) : 0);
    int py, px;
    block_pixel<BC>(r, &py, &px);
    pb[i] = (py * PC + px) * 64;
#pragma unroll
    for (int d = 0; d < 3; ++d) kq3[i][d] = (q ^ patch_key(py + d)) << 4;
  }
  const int b_lane = swz(wn * WN + (lane & 15), q);

  f32x4 acc[NT][MT], low[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = low[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Item k of the job of step (c, g), into registers.
  u32x4 set[3][NI][2];
  auto fetch = [&](auto gc, int c) {
    constexpr int g = decltype(gc)::value;
    const int ca = g == 0 ? c : min(c + 1, nchunk - 1);  // past the last chunk: data nothing reads
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const bool w = is_b(k);
      const __amdgpu_buffer_rsrc_t rs = w ? rsb : rsa;
      const unsigned o = off[k][g] + static_cast<unsigned>((w ? c : ca) * 128);
      set[g][k][0] = buf_load16(rs, o);
      set[g][k][1] = buf_load16(rs, o + 16);
    }
  };
  auto put_item = [&](int base, int plane, int at, const u32x4 (&v)[2]) {
    u32x4 s[3];
    split8(v[0], v[1], s);
    const int d = at < 0 ? SINK : base + at;
#pragma unroll
    for (int t = 0; t < 3; ++t) *reinterpret_cast<u32x4*>(smem + d + (at < 0 ? 0 : t * plane)) = s[t];
  };
  // Writes item k of a job (bslot: its step's weight buffer, aslot: its patch's).
  auto commit = [&](auto gc, int k, int aslot, int bslot) {
    constexpr int g = decltype(gc)::value;
    const bool w = is_b(k);
    put_item(w ? BOFF + bslot * BBUF : aslot * ABUF, w ? BPL : APL, place[k][g], set[g][k]);
  };
  auto mm = [&](f32x4& d, const u32x4& x, const u32x4& w) {  // x: pixels, w: weights
    if constexpr (POOL) mma<MAFAT_BF16>(d, x, w);
    else mma<MAFAT_BF16>(d, w, x);
  };
  u32x4 xf[2][3][MT], wf[2][3][NT];
  auto read = [&](int d, int ky, int kx, const unsigned char* sa, const unsigned char* sb) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
        xf[d][t][i] = *reinterpret_cast<const u32x4*>(sa + t * APL + pb[i] + (ky * PC + kx) * 64 + kq3[i][ky]);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        wf[d][t][j] = *reinterpret_cast<const u32x4*>(sb + t * BPL + b_lane + (kx * BN + j * 16) * 64);
    }
  };
  auto mfmas = [&](int d) {
    constexpr int PX[6] = {0, 1, 0, 1, 2, 0}, PW[6] = {0, 0, 1, 1, 0, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) mm(t == 0 ? acc[j][i] : low[j][i], xf[d][PX[t]][i], wf[d][PW[t]][j]);
  };
  // A step: its three taps' MFMAs, tap by tap, each beside the LDS reads of
  // the next tap and the split of a part of the next step's job (a wave's
  // MFMAs leave its vector and LDS issue slots free), whose patch part goes to
  // patch buffer acommit.
  auto step = [&](auto gc, auto nc, int aslot, int acommit, int bslot, bool more) {
    constexpr int ky = decltype(gc)::value;
    const unsigned char* sa = smem + aslot * ABUF;
    const unsigned char* sb = smem + BOFF + bslot * BBUF;
    read(0, ky, 0, sa, sb);
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      __builtin_amdgcn_sched_barrier(0);
      if (kx < 2) read((kx + 1) & 1, ky, kx + 1, sa, sb);
#pragma unroll
      for (int k = 0; k < NI; ++k)
        if (more && 2 - (NI - 1 - k) * 3 / NI == kx) commit(nc, k, acommit, bslot ^ 1);
      mfmas(kx & 1);
      constexpr int NM = 6 * MT * NT, NR = 3 * (MT + NT);
#pragma unroll
      for (int m = 0; m < NM / 2; ++m) {
        if (kx < 2 && m < NR) __builtin_amdgcn_sched_group_barrier(0x100, NR > NM / 2 ? 2 : 1, 0);  // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // vector
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  using G0 = std::integral_constant<int, 0>;
  using G1 = std::integral_constant<int, 1>;
  using G2 = std::integral_constant<int, 2>;
  // Chunk 0's patch (its thirds 0 and 1 ahead of the jobs that bring the
  // others') and jobs.
  u32x4 first[2][NI][2];
#pragma unroll
  for (int k = 0; k < NI; ++k)
    if (!is_b(k)) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {  // off[k][g + 1]: third g
        first[g][k][0] = buf_load16(rsa, off[k][g + 1]);
        first[g][k][1] = buf_load16(rsa, off[k][g + 1] + 16);
      }
    }
  fetch(G0{}, 0);
  fetch(G1{}, 0);
  fetch(G2{}, 0);
#pragma unroll
  for (int k = 0; k < NI; ++k)
    if (!is_b(k)) {
#pragma unroll
      for (int g = 0; g < 2; ++g) put_item(0, APL, place[k][g + 1], first[g][k]);
    }
#pragma unroll
  for (int k = 0; k < NI; ++k) commit(G0{}, k, 0, 0);
  wg_barrier_writes();
  // Step (c, g): fetches the job of (c + 1, g), three steps on, and writes the
  // next step's.
  int aslot = 0, bslot = 0;
  for (int c = 0; c + 1 < nchunk; ++c) {
    fetch(G0{}, c + 1);
    step(G0{}, G1{}, aslot, aslot ^ 1, bslot, true);
    wg_barrier_writes();
    fetch(G1{}, c + 1);
    step(G1{}, G2{}, aslot, aslot ^ 1, bslot ^ 1, true);
    wg_barrier_writes();
    fetch(G2{}, c + 1);
    step(G2{}, G0{}, aslot, aslot ^ 1, bslot, true);
    wg_barrier_writes();
    aslot ^= 1;
    bslot ^= 1;
  }
  f32x4 sc[NT], bi[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int co = n0 + wn * WN + j * 16 + (POOL ? (lane & 15) : 4 * (lane >> 4));
    const int cc = co < cout ? co : 0;
    if constexpr (POOL) {
      sc[j] = f32x4{a.scale[cc], 0.f, 0.f, 0.f};
      bi[j] = f32x4{a.bias[cc], 0.f, 0.f, 0.f};
    } else {
      sc[j] = *reinterpret_cast<const f32x4*>(a.scale + cc);
      bi[j] = *reinterpret_cast<const f32x4*>(a.bias + cc);
    }
  }
  step(G0{}, G1{}, aslot, aslot ^ 1, bslot, true);
  wg_barrier_writes();
  step(G1{}, G2{}, aslot, aslot ^ 1, bslot ^ 1, true);
  wg_barrier_writes();
  step(G2{}, G0{}, aslot, aslot ^ 1, bslot, false);

  // Epilogue, from registers: folded batch-norm, activation, the fused pool.
  const float slope = act_slope(a.act);
  const int vy = tl.cy0 + tl.ch - by0, vx = tl.cx0 + tl.cw - bx0;  // valid extent of this block
  // Place of this lane's outputs of GEMM row tile i (POOL: its window's), or
  // -1 outside the tile's rectangle; channel co of tile j.
  auto row_out = [&](int i, int* py, int* px) {
    const int r = wm * WM + i * 16 + (POOL ? 4 * (lane >> 4) : (lane & 15));
    block_pixel<BC>(r, py, px);
    if (r >= BR * BC || *py >= vy || *px >= vx) return -1;
    const int oy = POOL ? (by0 + *py) >> 1 : by0 + *py, ox = POOL ? (bx0 + *px) >> 1 : bx0 + *px;
    return ((oy - tl.dy0) * tl.dw + (ox - tl.dx0)) * cout;
  };
  const auto carried = [](float v) { return fabsf(v) <= 3.4028234663852886e38f; };  // finite
  bool bad = false;
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[j][i][r] = (acc[j][i][r] + low[j][i][r]) * (1.f / kSplitScale / kSplitScale);
        bad = bad || !carried(acc[j][i][r]);
      }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {
    // What the split could not carry: this wave's sums in plain float32, on the
    // fp32 MFMA, operands straight from memory.  Tap by tap, 16 channels to four
    // MFMAs, of which the r-th takes channels 4 q + r.
    f32x4 sum[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) sum[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t = 0; t < 9; ++t) {
      const int ky = t / 3, kx = t - 3 * ky;
      unsigned xo[MT], wo[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int r = wm * WM + i * 16 + (lane & 15);
        int py, px;
        block_pixel<BC>(r, &py, &px);
        const int iy = by0 + py + ky - 1, ix = bx0 + px + kx - 1;
        const bool ok = r < BR * BC && iy >= ry0 && iy < ry1 && ix >= rx0 && ix < rx1;
        xo[i] = ok ? static_cast<unsigned>((((iy - tl.sy0) * tl.sw + (ix - tl.sx0)) * cin + 4 * q) * 4) : 0x80000000u;
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int co = n0 + wn * WN + j * 16 + (lane & 15);
        wo[j] = co < cout ? static_cast<unsigned>(((co * 9 + t) * cin + 4 * q) * 4) : 0x80000000u;
      }
#pragma unroll 1
      for (unsigned c = 0; c < static_cast<unsigned>(cin) * 4; c += 128) {  // 32 channels, their loads in flight together
        u32x4 xv[2][MT], wv[2][NT];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int i = 0; i < MT; ++i) xv[h][i] = buf_load16(rsa, xo[i] + c + 64 * h);
#pragma unroll
          for (int j = 0; j < NT; ++j) wv[h][j] = buf_load16(rsb, wo[j] + c + 64 * h);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
              for (int j = 0; j < NT; ++j) {
                const float x = __uint_as_float(xv[h][i][r]), w = __uint_as_float(wv[h][j][r]);
                sum[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(POOL ? x : w, POOL ? w : x, sum[j][i], 0, 0, 0);
              }
      }
    }
    // Sum by sum: which others share a wave follows the block shape, and that
    // the size of the launch; what an output gets must not.
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][i][r] = carried(acc[j][i][r]) ? acc[j][i][r] : sum[j][i][r];
  }
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int py, px;
    const int o = row_out(i, &py, &px);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int co = n0 + wn * WN + j * 16 + (POOL ? (lane & 15) : 4 * (lane >> 4));
      float v[4];
      if constexpr (POOL) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = fmaf(acc[j][i][k], sc[j][0], bi[j][0]);
        float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
        mx = fmaxf(mx, slope * mx);
        if (o >= 0 && co < cout) dst[o + co] = mx;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[k] = fmaf(acc[j][i][k], sc[j][k], bi[j][k]);
          v[k] = fmaxf(v[k], slope * v[k]);
        }
        if (o >= 0 && co < cout) store4<MAFAT_F32>(dst + o + co, v);
      }
    }
  }
}

template <bool POOL>
hipError_t launch_split_p(const MfmaShape& sh, const StageArgs& args, hipStream_t stream, LaunchEvents ev) {
  const dim3 grid(static_cast<unsigned>(args.total_blocks), args.copy_blocks > 0 ? 2u : 1u);
#define MAFAT_SPLIT(br_, bc_, bm_, bn_, wgm_, wgn_)                                                       \
  if (sh.br == (br_) && sh.bc == (bc_) && sh.bm == (bm_) && sh.bn == (bn_)) {                             \
    hipExtLaunchKernelGGL((conv_split_kernel<br_, bc_, bm_, bn_, wgm_, wgn_, POOL>), grid,                \
                          dim3(64 * (wgm_) * (wgn_)), 0, stream, ev.start, ev.stop, 0, args);             \
    return hipGetLastError();                                                                             \
  }
  MAFAT_SPLIT_SHAPES
#undef MAFAT_SPLIT
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_conv_split(bool pool, const MfmaShape& shape, const StageArgs& args, hipStream_t stream,
                             LaunchEvents ev) {
  if (args.total_blocks <= 0) return hipSuccess;
  return pool ? launch_split_p<true>(shape, args, stream, ev) : launch_split_p<false>(shape, args, stream, ev);
}

}  // namespace mafat
